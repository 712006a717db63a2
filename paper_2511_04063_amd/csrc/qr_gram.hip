// QR of an n x n latent by blocks of 256 columns, from Gram matrices in fp64 (the QR step of Alg. 1).
//
// A block A_J is orthogonalised against itself by Cholesky: G = A_J^T A_J in fp64 on the fp64 matrix cores, G = U^T U in one
// workgroup, Q_J = A_J U^-1 with the inverses of U's 64 x 64 diagonal blocks; then everything right of it loses its part along
// Q_J.  A second pass orthogonalises Q_J once more, against the finished columns of R and against itself by the same
// kernels, and where that finds a block ill-conditioned a third projection and a correction at the end follow: R is orthogonal to
// rounding whenever Z's condition number is below 2^24.
//   gram64_kernel / gram64_sum_kernel   G of an m x <= 256 block: partial sums of row chunks, then their sum
//   chol64_kernel                       U and the inverses of its 64 x 64 diagonal blocks
//   block_solve_kernel                  A U^-1, rows dealt to the whole chip, with a step of refinement where U asks for it
//   third_pass_kernel / correct_kernel  what the third projections mean for U, and the correction
// fp64 holds the squares of any fp32 column and resolves condition numbers of a block up to 2^22; a block beyond that is orthogonalised
// column by column in the Cholesky's workgroup.
#include "dq_chol16.h"
#include "dq_internal.h"
#include "dq_wave.h"

namespace dq {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int GB = kGramBlock;        // columns of a block
constexpr int GT = GB / 16;           // 16 x 16 tiles across
static_assert(kGramSums == GB / 64 * (GB / 64 + 1) / 2 * 16, "workgroups of gram64_sum_kernel, 256 entries each");
constexpr unsigned kDone = 2u;        // *refine
// The second pass's G = I + E.  Up to here U = I + X, and from there on its columns may have lost half their length or cancel against
// each other, and what they have left along R_<J grows as much: once more.
constexpr double kNear = 1e-8, kFar = 0.25;      // |E|_F^2
#define MFMA32(a, b, c) __builtin_amdgcn_mfma_f32_16x16x4f32((a), (b), (c), 0, 0, 0)

// ---- G = A^T A ----------------------------------------------------------------------------------------------------
// A workgroup forms one 64 x 64 tile of the upper triangle over one chunk of rows, a wavefront a 32 x 32 quarter of it.
// Bound: the fp64 matrix cores (one 16 x 16 x 4 product in 64 cycles) and the latency of one chunk's loads, which come straight
// from L2 in operand layout (64 bytes a row and tile).
__device__ __forceinline__ void gram_tile(int t, int nt, int& ti, int& tj) {
    ti = 0;
    while (t >= nt - ti) { t -= nt - ti; ++ti; }
    tj = ti + t;
}

// rows r0 .. r1 of the quarter at (wm, wn) of tile (ti, tj)
__device__ __forceinline__ void gram_rows(const float* __restrict__ A, long lda, int cols, int ti, int tj, int wm, int wn, int r0,
                                          int r1, int c, int g, f64x4 (&acc)[2][2]) {
    // columns past the last are read as the last one: nobody uses what they give
    const float* pa[2];
    const float* pb[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int ca = 64 * ti + wm + 16 * i + c, cb = 64 * tj + wn + 16 * i + c;
        pa[i] = A + (long)(r0 + g) * lda + (ca < cols ? ca : cols - 1);
        pb[i] = A + (long)(r0 + g) * lda + (cb < cols ? cb : cols - 1);
    }
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
    f64x4 acc[2][2] = {};
    gram_rows(A, lda, cols, ti, tj, wm, wn, r0, r1, c, g, acc);
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
// of its diagonal), U^-1 = I - X, to |E|^2; dev takes each workgroup's share of |E|_F^2, which decides.
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
    const double d = r == c ? s - 1.0 : s;
    double q = r < c ? 2.0 * d * d : (r == c ? d * d : 0.0);
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) q += __shfl_xor(q, o);
    if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = q;
    __syncthreads();
    if (threadIdx.x == 0) dev[blockIdx.x] = (wsum[0] + wsum[1]) + (wsum[2] + wsum[3]);
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

// U: the block's place in the triangular factor (cols x cols, zeros below the diagonal).  inv: GB / 64 row-major 64 x 64 inverses.
// refine: 1 where A U^-1 needs the step of refinement, kDone where A is Q already (a block that the Gram matrix does not hold), else 0.
// second.dev: the sums of gram64_sum_kernel (second pass) or null;
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
                                                     float* __restrict__ inv, float* A, long lda, int rows, unsigned* refine,
                                                     unsigned* flags, SecondPass second, unsigned long long* started, unsigned long long value) {
    __shared__ __attribute__((aligned(16))) double rowbuf[GT * 256];   // the step's row of U, tile by tile
    __shared__ __attribute__((aligned(16))) double winv[2][16 * CLD];  // W = U^-T of the step's diagonal tile; of this and the last step
    __shared__ __attribute__((aligned(16))) double udiag[GT][256];     // U's diagonal tiles
    __shared__ __attribute__((aligned(16))) double keep[DEFER][GT / 2 * 256];   // right halves of U's first rows
    __shared__ __attribute__((aligned(16))) double nextbuf[2][256];    // tiles (k, k + 1) and (k + 1, k + 1) as step k finds them
    __shared__ __attribute__((aligned(16))) double diagbuf[2][256];
    __shared__ __attribute__((aligned(16))) double dcopy[16 * CLD];    // wavefront 0's
    __shared__ double cancels[2];                                      // of the columns of W that wavefronts 4 and 8 carry
    __shared__ int rows_done;                                          // counts them at the end of each step's row
    __shared__ double norm2[GB];                                       // squared column lengths
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 15, g = lane >> 4;
    const int nt = (cols + 15) / 16;
    const double* const dev = second.dev;
    if (dev != nullptr && tid == 0) {
        if (second.block == 0) second.again[0] = 0u;
        second.again[second.block + 1] = 0u;
    }
    if (started != nullptr && tid == 0) __hip_atomic_store(started, value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (dev != nullptr) {
        double s = 0.0;
        for (int i = lane; i < kGramSums; i += 64) s += dev[i];
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) s += __shfl_xor(s, o);
        if (__builtin_amdgcn_readfirstlane((int)(s < kNear))) {
            if (tid == 0) *refine = 0u;
            return;
        }
        if (!(s < kFar) && second.block > 0 && tid == 0) second.again[0] = second.again[second.block] = 1u;
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
            for (int r = 0; r < 4; ++r) dcopy[(4 * r + g) * CLD + c] = dk[r];
            __builtin_amdgcn_wave_barrier();       // one wavefront's LDS accesses are in order
            double d[16], x[16];
            int cc = c;
            asm volatile("" : "+v"(cc));           // sixteen comparisons and ones of the identity do not fit the registers across steps
#pragma unroll
            for (int i = 0; i < 16; i += 2) {      // a row of the symmetric tile is its column
                const double2 v = *reinterpret_cast<const double2*>(&dcopy[c * CLD + i]);
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
            // each row of 16 lanes writes four rows of W and of U's tile
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                winv[k & 1][(4 * g + q) * CLD + c] = pick4(g, x[q], x[4 + q], x[8 + q], x[12 + q]);
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
    } else if ((wave & 3) == 0) {
        // Columns of W within the 64 x 64 block: 0 and 3 (wavefront 4), 1 and 2 (wavefront 8); slots 0 .. split - 1 are the first's rows
        // from the diagonal down, the others the second's.
        const int ja = wave == 4 ? 0 : 1, jb = wave == 4 ? 3 : 2, split = 4 - ja;
        f64x4 wacc[5] = {};
        double cancel = 0.0;
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
                        for (int r = 0; r < 4; ++r) wacc[s][r] = winv[k & 1][(4 * r + g) * CLD + c];
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
                        const double len2 = norm2[16 * (k - kk + j) + c];
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            o[(16 * j + c) * 64 + 16 * i + 4 * r + g] = (float)wacc[s][r];
                            cancel = __builtin_fmax(cancel, len2 * wacc[s][r] * wacc[s][r]);
                        }
                    }
                }
            }
        }
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) cancel = __builtin_fmax(cancel, __shfl_xor(cancel, o));
        if (lane == 0) cancels[wave >> 3] = cancel;
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
    __syncthreads();
    const double cancel = __builtin_fmax(cancels[0], cancels[1]);
    const bool slow = !(cancel < kSlow);
    if (tid == 0) {
        if (!(cancel < kIllcond)) atomicOr(flags, DQ_FLAG_ILLCOND_PANEL);
        *refine = slow ? kDone : (cancel > kRefine ? 1u : 0u);
    }
    static_assert(sizeof(keep) >= orthogonalise_lds(CHOL_WAVES, GB) * sizeof(double), "scratch of the slow way");
    if (slow) orthogonalise_slowly<CHOL_WAVES>(A, lda, rows, cols, U, ldu, &keep[0][0], flags);
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
    const unsigned mode = *refine;
    const bool again = mode == 1u;
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
    if (mode != kDone) solve_rows<RT>(q, U, ldu, inv, cols, lane, wave);
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

// ---- after a third projection ---------------------------------------------------------------------------------------
// 16 columns of U from s0 on <- (I + X) U in place, X (upper triangular) by its entries: from the first 64 rows on, so that nothing is
// read that is new.
template <class X>
__device__ __forceinline__ void upper_times_columns(const X& x, int n, float* U, long ldu, int s0) {
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int c = lane & 15, g = lane >> 4, last = s0 + 16 < n ? s0 + 16 : n, col = s0 + c < n ? s0 + c : n - 1;
    for (int b = 0; 64 * b < last; ++b) {
        const int i0 = 64 * b + 16 * wave;
        f32x4 acc = {};
#pragma unroll 8
        for (int k = i0; k < last; k += 4) acc = MFMA32(x(i0 + c, k + g), k + g < n ? U[(long)(k + g) * ldu + col] : 0.f, acc);
        __syncthreads();
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (i0 + 4 * g + r <= s0 + c && s0 + c < n) U[(long)(i0 + 4 * g + r) * ldu + s0 + c] += acc[r];
    }
}

// The workgroups from `tiles` on: U <- (I + S) U, S from the blocks' third projections.  Those before: E = R^T R - I in fp64, one 64 x 64
// tile of the upper triangle each.
__global__ __launch_bounds__(256) void third_pass_kernel(const float* __restrict__ R, long ldr, int n, int tiles, float* __restrict__ E,
                                                         long lde, const float* __restrict__ S, long lds_, float* U, long ldu,
                                                         const unsigned* __restrict__ again, unsigned* flags) {
    if (again[0] == 0u) return;
    if ((int)blockIdx.x >= tiles) {
        auto x = [&](int i, int j) -> float {
            return j < n && i < j / GB * GB && again[j / GB] != 0u ? S[(long)i * lds_ + j] : 0.f;
        };
        upper_times_columns(x, n, U, ldu, 16 * ((int)blockIdx.x - tiles));
        return;
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int ti, tj;
    gram_tile(blockIdx.x, (n + 63) / 64, ti, tj);
    const int wm = (wave >> 1) * 32, wn = (wave & 1) * 32, c = lane & 15, g = lane >> 4;
    if (ti == tj && wm > wn) return;
    f64x4 acc[2][2] = {};
    gram_rows(R, ldr, n, ti, tj, wm, wn, 0, n, c, g, acc);
    bool large = false;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int r = 64 * ti + wm + 16 * i + 4 * v + g, k = 64 * tj + wn + 16 * j + c;
                if (r > k || k >= n) continue;
                const double e = acc[i][j][v] - (r == k ? 1.0 : 0.0);
                E[(long)r * lde + k] = (float)e;
                large |= !(__builtin_fabs(e) < 0x1p-10);
            }
    if (large) atomicOr(flags, DQ_FLAG_ILLCOND_PANEL);      // R stays off by the square of it
}

// R <- R (I - X), U <- (I + X) U in place, X the upper triangle of E, half of its diagonal: R^T R = I to |E|^2.  The first workgroups
// have 16 rows of R each and go through its columns from the last 64 back.
__global__ __launch_bounds__(256) void correct_kernel(const float* __restrict__ E, long lde, int n, float* R, long ldr, float* U,
                                                      long ldu, const unsigned* __restrict__ again) {
    if (again[0] == 0u) return;
    const int strips = (n + 15) / 16;
    auto x = [&](int i, int j) -> float {
        if (i > j || j >= n) return 0.f;
        const float v = E[(long)i * lde + j];
        return i < j ? v : 0.5f * v;
    };
    if ((int)blockIdx.x >= strips) {
        upper_times_columns(x, n, U, ldu, 16 * ((int)blockIdx.x - strips));
        return;
    }
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int c = lane & 15, g = lane >> 4, s0 = 16 * blockIdx.x;
    const float* row = R + (long)(s0 + c < n ? s0 + c : n - 1) * ldr;
    for (int b = (n - 1) / 64; b >= 0; --b) {
        const int j0 = 64 * b + 16 * wave;
        f32x4 acc = {};
#pragma unroll 8
        for (int k = 0; k < j0 + 16; k += 4) acc = MFMA32(k + g < n ? row[k + g] : 0.f, x(k + g, j0 + c), acc);
        __syncthreads();
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (s0 + 4 * g + r < n && j0 + c < n) R[(long)(s0 + 4 * g + r) * ldr + j0 + c] -= acc[r];
    }
}

}  // namespace

hipError_t launch_third_pass(float* R, long ldr, int n, const float* S, long lds_, float* E, long lde, float* U, long ldu,
                             const unsigned* again, unsigned* flags, hipStream_t s) {
    if (n < 1) return hipErrorInvalidValue;
    const int strips = (n + 15) / 16, nt = (n + 63) / 64, tiles = nt * (nt + 1) / 2, more = U != nullptr ? strips : 0;
    hipLaunchKernelGGL(third_pass_kernel, dim3(tiles + more), dim3(256), 0, s, R, ldr, n, tiles, E, lde, S, lds_, U, ldu, again, flags);
    hipLaunchKernelGGL(correct_kernel, dim3(strips + more), dim3(256), 0, s, E, lde, n, R, ldr, U, ldu, again);
    return hipGetLastError();
}

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

hipError_t launch_chol64(const double* G, int cols, float* U, long ldu, float* inv, float* A, long lda, int rows, unsigned* refine,
                         unsigned* flags, const SecondPass& second, unsigned long long* started, unsigned long long value, hipStream_t s) {
    if (cols < 1 || cols > GB) return hipErrorInvalidValue;
    hipLaunchKernelGGL(chol64_kernel, dim3(1), dim3(64 * CHOL_WAVES), 0, s, G, cols, U, ldu, inv, A, lda, rows, refine, flags, second, started,
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
