// QR of an n x n latent by blocks of 256 columns, from Gram matrices in fp64 (the QR step of Alg. 1).
//
// A block A_J is orthogonalised against itself by Cholesky: G = A_J^T A_J in fp64 on the fp64 matrix cores, G = U^T U in one
// workgroup, Q_J = A_J U^-1 with the inverses of U's 64 x 64 diagonal blocks; then everything right of it loses its part along
// Q_J.  A second pass orthogonalises Q_J once more, against the finished columns of R and against itself by the same
// kernels, which leaves R orthogonal to rounding whenever Z's condition number is below 2^24.
//   gram64_kernel / gram64_sum_kernel   G of an m x <= 256 block: partial sums of row chunks, then their sum
//   chol64_kernel                       U and the inverses of its 64 x 64 diagonal blocks
//   block_solve_kernel                  A U^-1, rows dealt to the whole chip, with a step of refinement where U asks for it
// fp64 holds the squares of any fp32 column and resolves condition numbers of a block up to 2^22, so that a block needs no other
// factorisation beside this one.
#include "dq_internal.h"
#include "dq_wave.h"

namespace dq {
namespace {

typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int GB = kGramBlock;        // columns of a block
constexpr int GT = GB / 16;           // 16 x 16 tiles across
static_assert(kGramSums == GB / 64 * (GB / 64 + 1) / 2 * 16, "workgroups of gram64_sum_kernel, 256 entries each");
#define MFMA64(a, b, c) __builtin_amdgcn_mfma_f64_16x16x4f64((a), (b), (c), 0, 0, 0)
#define MFMA32(a, b, c) __builtin_amdgcn_mfma_f32_16x16x4f32((a), (b), (c), 0, 0, 0)

// v_mfma_f64_16x16x4: A[m = l % 16][k = l / 16], B[k = l / 16][n = l % 16], register r of the result D[m = 4 r + l / 16][n = l % 16].
// Register r of a tile that was a result is therefore the operand of the 4 k from 4 r of the same tile, as B and, transposed, as A:
// C -= P^T Q takes three such tiles as they lie.

// ---- G = A^T A ----------------------------------------------------------------------------------------------------
// A workgroup forms one 64 x 64 tile of the upper triangle over one chunk of rows, a wavefront a 32 x 32 quarter of it.
// Bound: the fp64 matrix cores (one 16 x 16 x 4 product in 64 cycles) and the latency of one chunk's loads, which come straight
// from L2 in operand layout (64 bytes a row and tile).
__device__ __forceinline__ void gram_tile(int t, int nt, int& ti, int& tj) {
    ti = 0;
    while (t >= nt - ti) { t -= nt - ti; ++ti; }
    tj = ti + t;
}

__global__ __launch_bounds__(256) void gram64_kernel(const float* __restrict__ A, long lda, int rows, int cols, int nt,
                                                     int chunk, double* __restrict__ part) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int ti, tj;
    gram_tile(blockIdx.x, nt, ti, tj);
    const int wm = (wave >> 1) * 32, wn = (wave & 1) * 32;
    if (ti == tj && wm > wn) return;      // below the diagonal
    const int r0 = blockIdx.y * chunk, r1 = r0 + chunk < rows ? r0 + chunk : rows;
    const int c = lane & 15, g = lane >> 4;
    // columns past the last are read as the last one: nobody uses what they give
    const float* pa[2];
    const float* pb[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int ca = 64 * ti + wm + 16 * i + c, cb = 64 * tj + wn + 16 * i + c;
        pa[i] = A + (long)(r0 + g) * lda + (ca < cols ? ca : cols - 1);
        pb[i] = A + (long)(r0 + g) * lda + (cb < cols ? cb : cols - 1);
    }
    f64x4 acc[2][2] = {};
    constexpr int STEP = 4;               // groups of four rows in flight
    int r = r0;
    for (; r + 4 * STEP <= r1; r += 4 * STEP) {
        float fa[STEP][2], fb[STEP][2];
#pragma unroll
        for (int s = 0; s < STEP; ++s)
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const long o = (long)(r - r0 + 4 * s) * lda;
                fa[s][i] = pa[i][o];
                fb[s][i] = pb[i][o];
            }
#pragma unroll
        for (int s = 0; s < STEP; ++s)
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j) acc[i][j] = MFMA64((double)fa[s][i], (double)fb[s][j], acc[i][j]);
    }
    for (; r < r1; r += 4) {
        const bool in = r + g < r1;
        double a[2], b[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const long o = (long)(r - r0) * lda;
            a[i] = in ? (double)pa[i][o] : 0.0;
            b[i] = in ? (double)pb[i][o] : 0.0;
        }
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) acc[i][j] = MFMA64(a[i], b[j], acc[i][j]);
    }
    double* out = part + ((long)blockIdx.y * gridDim.x + blockIdx.x) * 4096;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v) out[(wm + 16 * i + 4 * v + g) * 64 + wn + 16 * j + c] = acc[i][j][v];
}

// G (GB x GB row-major: the upper triangle and, within the 64 x 64 tiles on the diagonal, its mirror image; past the last column the
// identity) = sum of the chunks' tiles, in order.  U gets zeros below its diagonal and inv the identity, which chol64_kernel fills in.
// second.dev (second pass, else null): U and inv as they are where G = I + E is so near to I that U = I + X with X the upper half of E (half
// of its diagonal), U^-1 = I - X, to |E|^2; dev takes each workgroup's share of |E|_F^2, which decides.  T += T2 where that is asked for.
__global__ __launch_bounds__(256) void gram64_sum_kernel(const double* __restrict__ part, int chunks, int cols,
                                                         double* __restrict__ G, float* __restrict__ U, long ldu,
                                                         float* __restrict__ inv, SecondPass second) {
    __shared__ double wsum[4];
    double* const dev = second.dev;
    const int nt = (cols + 63) / 64, tiles = nt * (nt + 1) / 2;
    int ti, tj;
    gram_tile(blockIdx.x >> 4, GB / 64, ti, tj);
    const int e = (blockIdx.x & 15) * 256 + threadIdx.x;
    const int r = 64 * ti + (e >> 6), c = 64 * tj + (e & 63);
    double s = r == c ? 1.0 : 0.0;
    if (r <= c && c < cols) {
        const double* p = part + (long)(ti * nt - ti * (ti - 1) / 2 + tj - ti) * 4096 + e;
        const long stride = (long)tiles * 4096;
        s = 0.0;
        int z = 0;
        for (; z + 8 <= chunks; z += 8) {
            double v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = p[(z + u) * stride];
#pragma unroll
            for (int u = 0; u < 8; ++u) s += v[u];
        }
        for (; z < chunks; ++z) s += p[z * stride];
    }
    if (r <= c) {
        G[r * GB + c] = s;
        if (ti == tj && r < c) G[c * GB + r] = s;
    }
    const bool near = dev != nullptr;
    if (r < cols && c < cols) {
        if (near && r <= c) U[(long)r * ldu + c] = (float)(r < c ? s : 0.5 + 0.5 * s);
        if (r < c) U[(long)c * ldu + r] = 0.f;
    }
    if (ti == tj && r <= c) {
        float* o = inv + (long)ti * 4096;
        o[(r & 63) * 64 + (c & 63)] = (float)(r < c ? (near ? -s : 0.0) : (near ? 1.5 - 0.5 * s : 1.0));
        if (r < c) o[(c & 63) * 64 + (r & 63)] = 0.f;
    }
    if (!near) return;
    if (second.trows > 0 && *second.again != 0u) {
        const int q = threadIdx.x;
        if (q < cols)
            for (int i = blockIdx.x; i < second.trows; i += kGramSums) second.T[(long)i * second.ldt + q] += second.T2[(long)i * second.ldt2 + q];
    }
    const double d = r == c ? s - 1.0 : s;
    double q = r < c ? 2.0 * d * d : (r == c ? d * d : 0.0);
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) q += __shfl_xor(q, o);
    if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = q;
    __syncthreads();
    if (threadIdx.x == 0) dev[blockIdx.x] = (wsum[0] + wsum[1]) + (wsum[2] + wsum[3]);
}

__global__ __launch_bounds__(256) void second_sum_kernel(const float* __restrict__ part, int splits, long stride, long ldp, int rows,
                                                         int cols, float* __restrict__ S, long lds_, unsigned* again) {
    const int c = threadIdx.x;
    unsigned large = 0u;
    if (c < cols)
        for (int r = blockIdx.x; r < rows; r += gridDim.x) {
            const float* p = part + (long)r * ldp + c;
            float s = 0.f;
            int z = 0;
            for (; z + 4 <= splits; z += 4) {
                float v[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) v[u] = p[(z + u) * stride];
#pragma unroll
                for (int u = 0; u < 4; ++u) s += v[u];
            }
            for (; z < splits; ++z) s += p[z * stride];
            S[(long)r * lds_ + c] = s;
            if (!(fabsf(s) < 0x1p-9f)) large = 1u;
        }
    if (large) atomicOr(again, 1u);
}

// ---- U and the inverses of its 64 x 64 diagonal blocks ------------------------------------------------------------
// Right-looking Cholesky by 16 columns on twelve wavefronts, four SIMDs' turn and turn about: wavefront 0 factors the 16 x 16
// diagonal tile of a step and inverts it; the nine that do not share its SIMD hold the 136 tiles of the upper triangle in
// registers, form the step's row of U from the inverse and take it off what is left; wavefronts 4 and 8 carry W = U^-T of the current
// 64 x 64 diagonal block along.  (fp64 products and fp64 arithmetic of a SIMD's wavefronts wait for each other: with tiles on
// wavefront 0's SIMD as well its pivots take up to 8000 cycles a tile, without 3200.)  Wavefront 0 forms the one tile of the row
// that the next diagonal tile waits for by itself and goes on: one barrier a step (the inverse is there, and the tiles that the
// next step starts from); the others meet a second time, at a counter in LDS, between a step's row and its update.
// Bound: wavefront 0's chain (a pivot about 190 cycles, products and copies 2000 a tile), in the first steps the fp64 matrix cores
// of one compute unit (256 cycles a tile).
constexpr int CHOL_WAVES = 12;
constexpr int CW = 9;                             // wavefronts that hold tiles
constexpr int CSLOTS = (GT * (GT + 1) / 2 + CW - 1) / CW;
constexpr int DEFER = 4;                          // first rows that the lower right quarter takes later
constexpr int DLD = 18;                           // row stride of the diagonal tile's copy: 16-byte reads of rows without conflicts
constexpr double kRefine = 1024.0;                // (square of) the cancellation from which A U^-1 gets a step of refinement
constexpr double kIllcond = 268435456.0;          // ... and from which the block counts as ill-conditioned, 2^14 in length

struct TileMap {
    unsigned char i[CW * CSLOTS + 1], j[CW * CSLOTS + 1];
    constexpr TileMap() : i(), j() {
        int t = 0;
        for (int r = 0; r < GT; ++r)
            for (int c = r; c < GT; ++c, ++t) { i[t] = (unsigned char)r; j[t] = (unsigned char)c; }
        for (; t <= CW * CSLOTS; ++t) { i[t] = 255; j[t] = 255; }   // no tile
    }
};
__constant__ const TileMap kTiles;

template <int L>
__device__ __forceinline__ double row_lane(double v) {   // the value of lane L of this lane's row of 16
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), 0x150 + L, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), 0x150 + L, 0xF, 0xF, true);
    return __hiloint2double(hi, lo);
}
// the g-th of four values, without a branch
__device__ __forceinline__ unsigned pick(unsigned mask, unsigned a, unsigned b) { return (mask & a) | (~mask & b); }
__device__ __forceinline__ double pick4(int g, double a, double b, double c, double d) {
    const unsigned m0 = 0u - (unsigned)(g & 1), m1 = 0u - (unsigned)(g >> 1);
    auto two = [&](int v0, int v1, int v2, int v3) {
        return (int)pick(m1, pick(m0, (unsigned)v3, (unsigned)v2), pick(m0, (unsigned)v1, (unsigned)v0));
    };
    return __hiloint2double(two(__double2hiint(a), __double2hiint(b), __double2hiint(c), __double2hiint(d)),
                            two(__double2loint(a), __double2loint(b), __double2loint(c), __double2loint(d)));
}

// acc - (lane I's value of u in this lane's row of 16) v, the broadcast in the instruction; nu = -u.  (s_nop: two wait states between
// a write of nu and a read of it from another lane)
template <int I>
__device__ __forceinline__ void take_off(double& acc, double nu, double v) {
    asm("v_fmac_f64_dpp %0, %1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf" : "+v"(acc) : "v"(nu), "v"(v), "i"(I));
}
template <int P, int I>
__device__ __forceinline__ void take_off_rows(double (&d)[16], double (&x)[16], double nu, double u, double w) {
    if constexpr (I < 16) {
        take_off<I>(d[I], nu, u);
        take_off<I>(x[I], nu, w);
        take_off_rows<P, I + 1>(d, x, nu, u, w);
    }
}

// d[i], x[i]: rows of this lane's column of the symmetric tile and of the identity.  Afterwards d[p] = U[p][lane] for p <= lane, x[p] =
// W[p][lane] with W = U^-T.  piv: the pivot; least: what this lane's pivot is kept above; mine: 1 / U[lane][lane].
// The chain: pivot, reciprocal root (2^-24, and one step: 1e-15), the pivot's row, the next pivot; the rest of the row goes off the
// rows below in its shadow.
template <int P>
__device__ __forceinline__ void factor_pivots(double (&d)[16], double (&x)[16], int col, double least, double piv, double& mine) {
    asm("v_max_f64 %0, %1, %2" : "=v"(piv) : "v"(piv), "v"(row_lane<P>(least)));   // (fmax quiets both operands first)
    const double r0 = __builtin_amdgcn_rsq(piv);
    const double e = __builtin_fma(-(piv * r0), r0, 1.0), r = r0 * __builtin_fma(e, 0.5, 1.0);
    const double u = (col == P ? piv : d[P]) * r, w = x[P] * r;
    mine = col == P ? r : mine;
    d[P] = u;
    x[P] = w;
    if constexpr (P < 15) {
        const double next = row_lane<P + 1>(__builtin_fma(-u, u, d[P + 1]));   // lane P + 1's own
        double nu = -u;
        asm volatile("s_nop 1" : "+v"(nu));
        take_off_rows<P, P + 1>(d, x, nu, u, w);
        factor_pivots<P + 1>(d, x, col, least, next, mine);
    }
}

// keeps what is derived from a loop-invariant value inside the loop: twenty slots' addresses do not fit the registers
__device__ __forceinline__ int opaque(int v) {
    asm volatile("" : "+s"(v));
    return v;
}

__device__ __forceinline__ f64x4 tile_read(const double* t, int lane) {
    f64x4 v;
#pragma unroll
    for (int r = 0; r < 4; ++r) v[r] = t[64 * r + lane];
    return v;
}
__device__ __forceinline__ f64x4 inverse_read(const double* w, int c, int g) {   // the tile W^T
    f64x4 v;
#pragma unroll
    for (int r = 0; r < 4; ++r) v[r] = w[c * DLD + 4 * r + g];
    return v;
}
__device__ __forceinline__ void tile_write(double* t, int lane, f64x4 v) {
#pragma unroll
    for (int r = 0; r < 4; ++r) t[64 * r + lane] = v[r];
}
// p^T q in two sums: a product waits 105 cycles for the one before it in the same sum, 64 for one in another
__device__ __forceinline__ f64x4 tile_mul2(f64x4 p, f64x4 q) {
    f64x4 a = MFMA64(p[0], q[0], f64x4{}), b = MFMA64(p[1], q[1], f64x4{});
    a = MFMA64(p[2], q[2], a);
    b = MFMA64(p[3], q[3], b);
    return a + b;
}
__device__ __forceinline__ f64x4 tile_sub(f64x4 p, f64x4 q, f64x4 c) {   // c - p^T q (blgp negates the first operand of an fp64 product)
#pragma unroll
    for (int r = 0; r < 4; ++r) c = __builtin_amdgcn_mfma_f64_16x16x4f64(p[r], q[r], c, 0, 0, 1);
    return c;
}

// U: the block's place in the triangular factor (cols x cols, zeros below the diagonal).  inv: GB / 64 row-major 64 x 64 inverses.
// refine: set to 1 where A U^-1 needs the step of refinement, else 0.  second.dev: the sums of gram64_sum_kernel (second pass) or null;
// where they say that G is I to |E|_F < 1e-4, U and inv are there already.  started (optional) takes `value` when the kernel runs.
// The slots from `first` on, in order: a jump into code that names each slot's registers.
#define DQ_SLOT(s, BODY) case s: if constexpr (s < CSLOTS) { BODY(s) } [[fallthrough]];
#define DQ_SLOTS(first, BODY)                                                                                              \
    switch (first) {                                                                                                       \
        DQ_SLOT(0, BODY) DQ_SLOT(1, BODY) DQ_SLOT(2, BODY) DQ_SLOT(3, BODY) DQ_SLOT(4, BODY) DQ_SLOT(5, BODY)               \
        DQ_SLOT(6, BODY) DQ_SLOT(7, BODY) DQ_SLOT(8, BODY) DQ_SLOT(9, BODY) DQ_SLOT(10, BODY) DQ_SLOT(11, BODY)             \
        DQ_SLOT(12, BODY) DQ_SLOT(13, BODY) DQ_SLOT(14, BODY) DQ_SLOT(15, BODY) DQ_SLOT(16, BODY) DQ_SLOT(17, BODY)         \
        DQ_SLOT(18, BODY) DQ_SLOT(19, BODY)                                                                                \
        default: break;                                                                                                    \
    }
// a tile of row k becomes U's
#define ROW_SLOT(s)                                                                                                        \
    {                                                                                                                      \
        const int t = opaque(tij[s]), tj = t & 255;                                                                        \
        if (t >> 8 == k && tj != k && tj < nt) {                                                                           \
            acc[s] = tile_mul2(ik, acc[s]);                                                                                \
            tile_write(rowbuf + tj * 256, lane, acc[s]);                                                                   \
            if (k < DEFER && tj >= GT / 2) tile_write(keep[k] + (tj - GT / 2) * 256, lane, acc[s]);                         \
        }                                                                                                                  \
        if (CW * (s + 1) > t1) break;                                                                                      \
    }
// what is left of a tile behind row k; the two that wavefront 0 goes on from are left for it.  The lower right quarter takes rows
// 0 .. DEFER - 1 together with the DEFER rows behind them: the first steps have the most tiles.
#define UPDATE_SLOT(s)                                                                                                     \
    {                                                                                                                      \
        const int t = opaque(tij[s]), ti = t >> 8, tj = t & 255;                                                           \
        if (ti > k && tj < nt && t != 257 * (k + 1) && (k >= DEFER || ti < GT / 2)) {                                      \
            if (k < 2 * DEFER && ti >= GT / 2) {                                                                           \
                const double* first = keep[k - DEFER];                                                                     \
                acc[s] = tile_sub(tile_read(first + (ti - GT / 2) * 256, lane), tile_read(first + (tj - GT / 2) * 256, lane), acc[s]); \
            }                                                                                                              \
            acc[s] = tile_sub(tile_read(rowbuf + ti * 256, lane), tile_read(rowbuf + tj * 256, lane), acc[s]);             \
            if (t == 257 * (k + 1) + 1) tile_write(nextbuf[(k + 1) & 1], lane, acc[s]);                                    \
            if (t == 257 * (k + 2)) tile_write(diagbuf[(k + 1) & 1], lane, acc[s]);                                        \
        }                                                                                                                  \
    }
static_assert(CSLOTS <= 20 && 2 * DEFER == GT / 2, "cases of DQ_SLOTS; the quarter is up to date when its first row is due");

__global__ __launch_bounds__(64 * CHOL_WAVES) void chol64_kernel(const double* __restrict__ G, int cols, float* __restrict__ U, long ldu,
                                                     float* __restrict__ inv, unsigned* refine, unsigned* flags,
                                                     SecondPass second, unsigned long long* started, unsigned long long value) {
    __shared__ __attribute__((aligned(16))) double rowbuf[GT * 256];   // the step's row of U, tile by tile
    __shared__ __attribute__((aligned(16))) double winv[2][16 * DLD];  // W = U^-T of the step's diagonal tile; of this and the last step
    __shared__ __attribute__((aligned(16))) double udiag[GT][256];     // U's diagonal tiles
    __shared__ __attribute__((aligned(16))) double keep[DEFER][GT / 2 * 256];   // right halves of U's first rows
    __shared__ __attribute__((aligned(16))) double nextbuf[2][256];    // tiles (k, k + 1) and (k + 1, k + 1) as step k finds them
    __shared__ __attribute__((aligned(16))) double diagbuf[2][256];
    __shared__ __attribute__((aligned(16))) double dcopy[16 * DLD];    // wavefront 0's
    __shared__ int rows_done;                                          // counts them at the end of each step's row
    __shared__ double norm2[GB];                                       // squared column lengths
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 15, g = lane >> 4;
    const int nt = (cols + 15) / 16;
    const double* const dev = second.dev;
    if (dev != nullptr && tid == 0) *second.again = 0u;
    if (started != nullptr && tid == 0) __hip_atomic_store(started, value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (dev != nullptr) {
        double s = 0.0;
        for (int i = lane; i < kGramSums; i += 64) s += dev[i];
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) s += __shfl_xor(s, o);
        if (__builtin_amdgcn_readfirstlane((int)(s < 1e-8))) {
            if (tid == 0) *refine = 0u;
            return;
        }
    }
    if (tid == 0) rows_done = 0;
    if (tid < GB) {
        const double v = G[tid * (GB + 1)];
        norm2[tid] = v;
        if (!(v < 0x1p1000)) atomicOr(flags, DQ_FLAG_NONFINITE);
        if (v == 0.0) atomicOr(flags, dev == nullptr ? DQ_FLAG_SINGULAR | DQ_FLAG_ILLCOND_PANEL : DQ_FLAG_SINGULAR);
    }
    __syncthreads();
    // Three loops with the same barriers, so that none's registers are live in another.
    if (wave == 0) {
        double worst = 0.0;              // largest (length / what is left of it)^2 of this lane's columns
        f64x4 dk;                        // the diagonal tile of the step
#pragma unroll
        for (int r = 0; r < 4; ++r) dk[r] = G[(4 * r + g) * GB + c];
        f64x4 next = {}, diag = {};      // tiles (k, k + 1) and (k + 1, k + 1)
        if (nt > 1) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                next[r] = G[(4 * r + g) * GB + 16 + c];
                diag[r] = G[(16 + 4 * r + g) * GB + 16 + c];
            }
        }
        for (int k = 0; k < nt; ++k) {
#pragma unroll
            for (int r = 0; r < 4; ++r) dcopy[(4 * r + g) * DLD + c] = dk[r];
            __builtin_amdgcn_wave_barrier();       // one wavefront's LDS accesses are in order
            double d[16], x[16];
            int cc = c;
            asm volatile("" : "+v"(cc));           // sixteen comparisons and ones of the identity do not fit the registers across steps
#pragma unroll
            for (int i = 0; i < 16; i += 2) {      // a row of the symmetric tile is its column
                const double2 v = *reinterpret_cast<const double2*>(&dcopy[c * DLD + i]);
                d[i] = v.x; d[i + 1] = v.y;
            }
            const double len2 = norm2[16 * k + c];
            // what rounding leaves of a column that depends on those before it is kept above 2^-22 of its length; a column of
            // zeros keeps its pivot's reciprocal finite and its row of the inverse zero
            const double least = __builtin_fmax(len2 * 0x1p-44, 0x1p-600), one = len2 > 0.0 ? 1.0 : 0.0;
            double mine = 0.0;
#pragma unroll
            for (int i = 0; i < 16; ++i) x[i] = i == cc ? one : 0.0;
            factor_pivots<0>(d, x, cc, least, row_lane<0>(d[0]), mine);
            worst = __builtin_fmax(worst, len2 * mine * mine);
            // each row of 16 lanes writes four rows of W and of U's tile
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                winv[k & 1][(4 * g + q) * DLD + c] = pick4(g, x[q], x[4 + q], x[8 + q], x[12 + q]);
                udiag[k][(4 * g + q) * 16 + c] = pick4(g, d[q], d[4 + q], d[8 + q], d[12 + q]);
            }
            lds_barrier();                         // step k's inverse and the tiles of step k are there
            if (k + 1 < nt) {
                if (k > 0) {
                    next = tile_read(nextbuf[k & 1], lane);
                    diag = tile_read(diagbuf[k & 1], lane);
                }
                if (k == 2 * DEFER - 1) {          // what the quarter's first tile would still get in this step's update
                    const f64x4 v = tile_read(keep[DEFER - 1], lane);
                    diag = tile_sub(v, v, diag);
                }
                const f64x4 u = tile_mul2(inverse_read(winv[k & 1], c, g), next);
                dk = tile_sub(u, u, diag);
            }
        }
#pragma unroll
        for (int o = 8; o >= 1; o >>= 1) worst = __builtin_fmax(worst, __shfl_xor(worst, o));
        if (lane == 0) {
            if (dev == nullptr && worst > kIllcond) atomicOr(flags, DQ_FLAG_ILLCOND_PANEL);
            *refine = worst > kRefine ? 1u : 0u;
        }
    } else if ((wave & 3) == 0) {
        // Columns of W within the 64 x 64 block: 0 and 3 (wavefront 4), 1 and 2 (wavefront 8); slots 0 .. split - 1 are the first's rows
        // from the diagonal down, the others the second's.
        const int ja = wave == 4 ? 0 : 1, jb = wave == 4 ? 3 : 2, split = 4 - ja;
        f64x4 wacc[5] = {};
        for (int k = 0; k < nt; ++k) {
            const int kk = k & 3;
            if (kk == 0) {
#pragma unroll
                for (int s = 0; s < 5; ++s) wacc[s] = f64x4{};
            }
            lds_barrier();
            const f64x4 ik = inverse_read(winv[k & 1], c, g);
            f64x4 cur[2] = {};                     // row kk's tiles of the two columns
#pragma unroll
            for (int s = 0; s < 5; ++s) {
                const int j = s < split ? ja : jb, i = s < split ? ja + s : jb + s - split;
                if (i == kk) {
                    if (j == kk) {                 // the diagonal tile: the transposed inverse itself
#pragma unroll
                        for (int r = 0; r < 4; ++r) wacc[s][r] = winv[k & 1][(4 * r + g) * DLD + c];
                    } else {
                        wacc[s] = tile_mul2(ik, wacc[s]);
                    }
                    if (s < split) cur[0] = wacc[s];
                    else cur[1] = wacc[s];
                }
            }
            while (__hip_atomic_load(&rows_done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) < CW * (k + 1)) {}
            asm volatile("" ::: "memory");
#pragma unroll
            for (int s = 0; s < 5; ++s) {
                const int j = s < split ? ja : jb, i = s < split ? ja + s : jb + s - split;
                if (i > kk && j <= kk && k - kk + i < nt)
                    wacc[s] = tile_sub(tile_read(rowbuf + (k - kk + i) * 256, lane), s < split ? cur[0] : cur[1], wacc[s]);
            }
            if (kk == 3 || k == nt - 1) {          // out, transposed, as the inverse
                float* o = inv + (long)(k >> 2) * 4096;
#pragma unroll
                for (int s = 0; s < 5; ++s) {
                    const int j = s < split ? ja : jb, i = s < split ? ja + s : jb + s - split;
                    if (i <= kk) {
#pragma unroll
                        for (int r = 0; r < 4; ++r) o[(16 * j + c) * 64 + 16 * i + 4 * r + g] = (float)wacc[s][r];
                    }
                }
            }
        }
    } else {
        // the tiles: slot s of the w-th of these wavefronts holds tile CW s + w of the upper triangle, so that what is left is always
        // dealt evenly
        const int w = wave - 1 - wave / 4;
        f64x4 acc[CSLOTS];
        int tij[CSLOTS];                 // 256 i + j
#pragma unroll
        for (int s = 0; s < CSLOTS; ++s) {
            tij[s] = __builtin_amdgcn_readfirstlane(256 * kTiles.i[CW * s + w] + kTiles.j[CW * s + w]);
            acc[s] = f64x4{};
            const int ti = tij[s] >> 8, tj = tij[s] & 255;
            if (tj < nt) {
                const double* p = G + (16 * ti + g) * GB + 16 * tj + c;
#pragma unroll
                for (int r = 0; r < 4; ++r) acc[s][r] = p[4 * r * GB];
            }
        }
        for (int k = 0; k < nt; ++k) {
            lds_barrier();
            const f64x4 ik = inverse_read(winv[k & 1], c, g);
            // tiles t0 .. of row k, and the diagonal tile behind them, from the first slot that may hold one on
            const int t0 = k * GT - k * (k - 1) / 2, t1 = t0 + GT - k;
            DQ_SLOTS(t0 / CW, ROW_SLOT)
            // they wait for each other's tiles of the row
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            if (lane == 0) __hip_atomic_fetch_add(&rows_done, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            while (__hip_atomic_load(&rows_done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) < CW * (k + 1)) {}
            asm volatile("" ::: "memory");
            DQ_SLOTS(t1 / CW, UPDATE_SLOT)
        }
        // U
#pragma unroll
        for (int s = 0; s < CSLOTS; ++s) {
            const int ti = tij[s] >> 8, tj = tij[s] & 255;
            if (tj < nt) {
                const f64x4 u = ti == tj ? tile_read(udiag[ti], lane) : acc[s];
                float* o = U + (long)(16 * ti + g) * ldu + 16 * tj + c;
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (16 * tj + c < cols && 16 * ti + 4 * r + g <= 16 * tj + c) o[(long)(4 * r) * ldu] = (float)u[r];
            }
        }
    }
}

// ---- Q = A U^-1 ---------------------------------------------------------------------------------------------------
// RT times 16 rows a workgroup, by substitution over the 64 columns of each diagonal block: T_s = A_s - sum_i Q_i U_is, Q_s = T_s
// inv_s.  fp32 matrix instructions; U and the inverses come from L2 in operand layout, 64 rows of them a step ahead.  Where U's
// columns cancelled by more than 2^5 against each other the products with its inverse lose as much, which one step of refinement,
// Q += (A - Q U) U^-1, gives back.
// Bound: the chain of ten steps of 64 k, 16 products each per 16 rows, and two barriers a block.
constexpr int SLD = GB + 4;

template <int RT>
__device__ __forceinline__ void solve_rows(float (*buf)[SLD], const float* __restrict__ U, long ldu,
                                           const float* __restrict__ inv, int cols, int lane, int wave) {
    const int c = lane & 15, g = lane >> 4;
    const int ns = (cols + 63) / 64;
    // step kc of block s: rows 64 kc .. of U's columns of the block, or, kc == s, of the inverse
    auto fetch = [&](int s, int kc, float (&b)[16]) {
        const int col = 64 * s + 16 * wave + c;
        const float* p = kc < s ? U + (long)(64 * kc + g) * ldu + (col < cols ? col : cols - 1)
                                : inv + (long)s * 4096 + g * 64 + 16 * wave + c;
        const long step = 4 * (kc < s ? ldu : 64);
#pragma unroll
        for (int q = 0; q < 16; ++q) b[q] = p[q * step];
    };
    float b[16];
    fetch(0, 0, b);
    for (int s = 0; s < ns; ++s) {
        const int col = 64 * s + 16 * wave + c;
        const bool in = col < cols;
        f32x4 acc[RT] = {};
        for (int kc = 0; kc <= s; ++kc) {
            float nb[16];
            if (kc < s) fetch(s, kc + 1, nb);
            else if (s + 1 < ns) fetch(s + 1, 0, nb);
            if (kc == s) {
                if (s > 0) {
#pragma unroll
                    for (int t = 0; t < RT; ++t)
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            buf[16 * t + 4 * g + r][col] -= in ? acc[t][r] : 0.f;
                            acc[t][r] = 0.f;
                        }
                    __syncthreads();
                }
#pragma unroll
                for (int q4 = 0; q4 < 4; ++q4)
                    if (q4 <= wave) {      // the inverse is upper triangular
#pragma unroll
                        for (int q = 4 * q4; q < 4 * q4 + 4; ++q)
#pragma unroll
                            for (int t = 0; t < RT; ++t) acc[t] = MFMA32(buf[16 * t + c][64 * s + 4 * q + g], b[q], acc[t]);
                    }
            } else {
#pragma unroll
                for (int q = 0; q < 16; ++q)
#pragma unroll
                    for (int t = 0; t < RT; ++t) acc[t] = MFMA32(buf[16 * t + c][64 * kc + 4 * q + g], b[q], acc[t]);
            }
#pragma unroll
            for (int q = 0; q < 16; ++q) b[q] = nb[q];
        }
        __syncthreads();
#pragma unroll
        for (int t = 0; t < RT; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) buf[16 * t + 4 * g + r][col] = acc[t][r];
        __syncthreads();
    }
}

// A (rows x cols) <- A U^-1, also written to R where that is given
template <int RT>
__global__ __launch_bounds__(256) void block_solve_kernel(float* A, long lda, int rows, int cols, const float* __restrict__ U,
                                                          long ldu, const float* __restrict__ inv,
                                                          const unsigned* __restrict__ refine, float* R, long ldr) {
    constexpr int SR = 16 * RT;
    __shared__ __attribute__((aligned(16))) float a[SR][SLD];
    __shared__ __attribute__((aligned(16))) float q[SR][SLD];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int r0 = blockIdx.x * SR;
    const bool again = *refine != 0u;
    const int c4 = 4 * (tid & 63);
#pragma unroll
    for (int i = 0; i < SR / 4; ++i) {
        const int r = (tid >> 6) + 4 * i;
        float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
        if (r0 + r < rows && c4 < cols) v = load_quad(A + (long)(r0 + r) * lda + c4, cols - c4);
        *reinterpret_cast<float4*>(&q[r][c4]) = v;
        if (again) *reinterpret_cast<float4*>(&a[r][c4]) = v;
    }
    __syncthreads();
    solve_rows<RT>(q, U, ldu, inv, cols, lane, wave);
    if (again) {
        const int c = lane & 15, g = lane >> 4;
        for (int s = 0; s < (cols + 63) / 64; ++s) {          // A - Q U
            const int col = 64 * s + 16 * wave + c;
            const bool in = col < cols;
            const float* pu = U + (in ? col : cols - 1);
            f32x4 acc[RT] = {};
            for (int k = 0; k < 64 * s + 16 * (wave + 1); k += 16) {
                float b[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int row = k + 4 * u + g;
                    b[u] = in && row < cols ? pu[(long)row * ldu] : 0.f;
                }
#pragma unroll
                for (int u = 0; u < 4; ++u)
#pragma unroll
                    for (int t = 0; t < RT; ++t) acc[t] = MFMA32(q[16 * t + c][k + 4 * u + g], b[u], acc[t]);
            }
#pragma unroll
            for (int t = 0; t < RT; ++t)
#pragma unroll
                for (int r = 0; r < 4; ++r) a[16 * t + 4 * g + r][col] -= acc[t][r];
        }
        __syncthreads();
        solve_rows<RT>(a, U, ldu, inv, cols, lane, wave);
    }
#pragma unroll
    for (int i = 0; i < SR / 4; ++i) {
        const int r = (tid >> 6) + 4 * i;
        if (r0 + r >= rows || c4 >= cols) continue;
        float4 v = *reinterpret_cast<const float4*>(&q[r][c4]);
        if (again) {
            const float4 e = *reinterpret_cast<const float4*>(&a[r][c4]);
            v.x += e.x; v.y += e.y; v.z += e.z; v.w += e.w;
        }
        store_quad(A + (long)(r0 + r) * lda + c4, cols - c4, v);
        if (R != nullptr) store_quad(R + (long)(r0 + r) * ldr + c4, cols - c4, v);
    }
}

}  // namespace

// chunks of rows of a Gram product: 64 rows at least, 32 chunks at most
static int gram64_chunk(int rows) {
    int chunk = (rows + 31) / 32;
    if (chunk < 64) chunk = 64;
    return (chunk + 15) / 16 * 16;
}

size_t gram64_part_doubles(int rows, int cols) {
    const int nt = (cols + 63) / 64, chunk = gram64_chunk(rows);
    return (size_t)((rows + chunk - 1) / chunk) * (nt * (nt + 1) / 2) * 4096;
}

hipError_t launch_gram64(const float* A, long lda, int rows, int cols, double* part, double* G, float* U, long ldu, float* inv,
                         const SecondPass& second, hipStream_t s) {
    if (rows < 1 || cols < 1 || cols > GB) return hipErrorInvalidValue;
    const int nt = (cols + 63) / 64, tiles = nt * (nt + 1) / 2, chunk = gram64_chunk(rows), chunks = (rows + chunk - 1) / chunk;
    hipLaunchKernelGGL(gram64_kernel, dim3(tiles, chunks), dim3(256), 0, s, A, lda, rows, cols, nt, chunk, part);
    hipLaunchKernelGGL(gram64_sum_kernel, dim3(kGramSums), dim3(256), 0, s, part, chunks, cols, G, U, ldu, inv, second);
    return hipGetLastError();
}

hipError_t launch_second_sum(const float* part, int splits, long stride, long ldp, int rows, int cols, float* S, long lds_,
                             unsigned* again, hipStream_t s) {
    if (rows < 1 || cols < 1 || cols > GB) return hipErrorInvalidValue;
    hipLaunchKernelGGL(second_sum_kernel, dim3(rows < 2048 ? rows : 2048), dim3(GB), 0, s, part, splits, stride, ldp, rows, cols, S,
                       lds_, again);
    return hipGetLastError();
}

hipError_t launch_chol64(const double* G, int cols, float* U, long ldu, float* inv, unsigned* refine, unsigned* flags,
                         const SecondPass& second, unsigned long long* started, unsigned long long value, hipStream_t s) {
    if (cols < 1 || cols > GB) return hipErrorInvalidValue;
    hipLaunchKernelGGL(chol64_kernel, dim3(1), dim3(64 * CHOL_WAVES), 0, s, G, cols, U, ldu, inv, refine, flags, second, started,
                       value);
    return hipGetLastError();
}

// 16 rows a workgroup where that fills the chip no more than once
hipError_t launch_block_solve(float* A, long lda, int rows, int cols, const float* U, long ldu, const float* inv,
                              const unsigned* refine, float* R, long ldr, hipStream_t s) {
    if (rows < 1 || cols < 1 || cols > GB) return hipErrorInvalidValue;
    if (rows <= 4096)
        hipLaunchKernelGGL(block_solve_kernel<1>, dim3((rows + 15) / 16), dim3(256), 0, s, A, lda, rows, cols, U, ldu, inv, refine,
                           R, ldr);
    else
        hipLaunchKernelGGL(block_solve_kernel<2>, dim3((rows + 31) / 32), dim3(256), 0, s, A, lda, rows, cols, U, ldu, inv, refine,
                           R, ldr);
    return hipGetLastError();
}

}  // namespace dq
