// QR of an n x n latent by blocks of 256 columns, from Gram matrices in fp64 (the QR step of Alg. 1).
//
// A block A_J is orthogonalised against itself by Cholesky: G = A_J^T A_J in fp64 on the fp64 matrix cores, G = U^T U in one
// workgroup, Q_J = A_J U^-1 with the inverses of U's 64 x 64 diagonal blocks; then everything right of it loses its part along
// Q_J.  A second pass orthogonalises Q_J once more, against the finished columns of R and against itself by the same
// kernels.  Where that finds a block ill-conditioned, and where columns have vanished, the columns that are not yet orthogonal are gone
// through at the end: R is orthogonal to rounding for every finite Z, and reproduces it.
//   gram64_kernel / gram64_sum_kernel   G of an m x <= 256 block: partial sums of row chunks, then their sum
//   chol64_kernel                       U and the inverses of its 64 x 64 diagonal blocks
//   block_solve_kernel                  A U^-1, rows dealt to the whole chip
//   finish_kernel                       what the second pass may have left
// fp64 holds the squares of fp32 columns of 2^-102 to 2^120 and resolves condition numbers of a block up to 2^18 with room to spare; a block beyond that is
// orthogonalised 16 columns at a time by the workgroups of its solve.
#include <type_traits>

#include "dq_chol16.h"
#include "dq_internal.h"
#include "dq_wave.h"

namespace dq {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int GB = kGramBlock;        // columns of a block
constexpr int GT = GB / 16;           // 16 x 16 tiles across
static_assert(kGramSums == GB / 64 * (GB / 64 + 1) / 2 * 16, "workgroups of gram64_sum_kernel, 256 entries each");
// What a block's columns cancel by against each other is taken from U^-1: max over i, j of (|a_j| |U^-1[j][i]|)^2.  From kSubstitute on
// A U^-1 is formed by substitution, from kIllcond on (2^14 in length) the block is reported, from kLots on (2^18), and where a pivot has
// been raised, its Gram matrix does not hold it any more, and it is made orthonormal 16 columns at a time.
constexpr double kSubstitute = 1024.0, kIllcond = 0x1p28, kLots = 0x1p36;
// Columns shorter than 2^-102 count as zeros: the products on split operands do not see all of them, nor is 2^22 / length an fp32 number.
// From 2^120 on what is formed of them may leave fp32's range.
constexpr double kTiny = 0x1p-204, kHuge = 0x1p240;      // squared
enum : unsigned { kPlain = 0u, kSubstituted = 1u, kByLots = 2u };        // words[0] of the solve
// The second pass's G = I + E.  Up to here U = I + X, and from there on its columns may have lost half their length or cancel against
// each other, and what they have left along R_<J grows as much: finish_kernel looks at them.
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
// solve: [0] how A U^-1 is to be formed, [2..3] zeroed for it.
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
                                                     float* __restrict__ inv, unsigned* solve, unsigned* flags,
                                                     SecondPass second, unsigned long long* started, unsigned long long value) {
    __shared__ __attribute__((aligned(16))) double rowbuf[GT * 256];   // the step's row of U, tile by tile
    __shared__ __attribute__((aligned(16))) double winv[2][16 * CLD];  // W = U^-T of the step's diagonal tile; of this and the last step
    __shared__ __attribute__((aligned(16))) double udiag[GT][256];     // U's diagonal tiles
    __shared__ __attribute__((aligned(16))) double keep[DEFER][GT / 2 * 256];   // right halves of U's first rows
    __shared__ __attribute__((aligned(16))) double nextbuf[2][256];    // tiles (k, k + 1) and (k + 1, k + 1) as step k finds them
    __shared__ __attribute__((aligned(16))) double diagbuf[2][256];
    __shared__ __attribute__((aligned(16))) double dcopy[16 * CLD];    // wavefront 0's
    __shared__ double cancels[3];                                      // of the columns of W that wavefronts 4 and 8 carry; of raised pivots
    __shared__ int rows_done;                                          // counts them at the end of each step's row
    __shared__ double norm2[GB];                                       // squared column lengths
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 15, g = lane >> 4;
    const int nt = (cols + 15) / 16;
    const double* const dev = second.dev;
    for (int i = tid; i < second.clear; i += 64 * CHOL_WAVES) second.words[i] = 0u;
    if (started != nullptr && tid == 0) __hip_atomic_store(started, value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (dev != nullptr) {
        double s = 0.0;
        for (int i = lane; i < kGramSums; i += 64) s += dev[i];
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) s += __shfl_xor(s, o);
        if (__builtin_amdgcn_readfirstlane((int)(s < kNear))) {
            if (tid == 0) solve[0] = kPlain;
            return;
        }
        if (!(s < kFar) && tid == 0) second.words[0] = 1u;
    }
    if (tid == 0) rows_done = 0;
    if (tid < GB) {
        const double v = G[tid * (GB + 1)];
        norm2[tid] = v;
        if (!(v < kHuge)) atomicOr(flags, DQ_FLAG_NONFINITE);
        if (v < kTiny) atomicOr(flags, dev == nullptr ? DQ_FLAG_SINGULAR | DQ_FLAG_ILLCOND_PANEL : DQ_FLAG_SINGULAR);
    }
    __syncthreads();
    // Three loops with the same barriers, so that none's registers are live in another.
    if (wave == 0) {
        f64x4 dk;                        // the diagonal tile of the step
#pragma unroll
        for (int r = 0; r < 4; ++r) dk[r] = G[(4 * r + g) * GB + c];
        f64x4 next = {}, diag = {};      // tiles (k, k + 1) and (k + 1, k + 1)
        double raised = 0.0;
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
            // what rounding leaves of a column that depends on those before it is kept above 2^-22 of its length, and the Gram matrix
            // does not hold the block; a column of zeros gets a pivot that it does not matter beside, and its row of the inverse zero
            const bool there = len2 >= kTiny;
            const double least = there ? len2 * 0x1p-44 : 1.0, one = there ? 1.0 : 0.0;
            double mine = 0.0;
#pragma unroll
            for (int i = 0; i < 16; ++i) x[i] = i == cc ? one : 0.0;
            factor_pivots<0>(d, x, cc, least, row_lane<0>(d[0]), mine);
            raised = __builtin_fmax(raised, one * (mine * mine * least));      // 1 where the pivot was
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
#pragma unroll
        for (int o = 8; o >= 1; o >>= 1) raised = __builtin_fmax(raised, __shfl_xor(raised, o));
        if (lane == 0) cancels[2] = raised > 0.9 ? 0x1p100 : 0.0;
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
    const double cancel = __builtin_fmax(__builtin_fmax(cancels[0], cancels[1]), cancels[2]);
    if (tid == 0) {
        if (!(cancel < kIllcond)) atomicOr(flags, DQ_FLAG_ILLCOND_PANEL);
        solve[0] = !(cancel < kLots) ? kByLots : (cancel > kSubstitute ? kSubstituted : kPlain);
        solve[2] = solve[3] = 0u;
    }
}

// ---- columns that a Gram matrix does not hold, 16 at a time -------------------------------------------------------------
// A lot S goes through turns: W = M_<^T S, S -= M_< W, S^T S = U^T U (its Cholesky factor, in fp64), S <- S U^-1; the last is the one that
// finds S orthonormal.  Two for a lot of any condition that fp32 can hold, a third where rounding noise was left.  A column that has
// vanished, or of which at unit length only rounding in the span of the others was left once more, is set to zero, with its row of T: none of
// what the columns behind it have is along it.
// The workgroups of one launch do this together and wait for each other at a word in device memory, three times a turn.  They all have
// a place at the same time: at most 128 of them, two or three to a compute unit (64 units at least), and what runs on other streams ends or, if it is one
// of these kernels, fits beside them three times over.  The polls are bounded like those between streams.  They share the work by tiles of W
// (cut along the rows where there are few) and strips of 16 rows; the 16 x 16 numerics are done by all of them alike.
// Bound: the latency of these steps: a block of 256 columns 0.35 ms at 200 rows, 0.7 at 600, 1.0 at 1536, 2.2 at 4096 (by one workgroup, in
// global memory: 1.2, 4.5, 13 and 37 ms).
constexpr double kSettled = 1e-2;          // |S^T S - I|_F^2 with which a turn is a lot's last
constexpr int kTurns = 12;                 // two or three in fact
constexpr int kLotGroups = 128;            // workgroups, at most
constexpr int kLotStrips = DQ_MAX_N / 16 / kLotGroups;      // strips of 16 rows that a workgroup has room for
constexpr int kLotParts = 8;               // parts of W along the rows, at most, where it has
constexpr int kLotTiles = GT - 1;          // no more than these tiles
constexpr long long kMeetTicks = 5LL * 1000 * 1000 * 100;

struct LotShared {
    double gsum[16 * CLD], dist[4];
    float red[4][256], strip[kLotStrips][256], ut[256], u1[256], rinv[16];
    float w[kLotTiles][256];
    unsigned gone;
};

// M (rows x cols): the columns; T: before = after * T; W: cols (a multiple of 16) x 16, or kLotParts of that; gpart: 256 a workgroup.
struct LotJob {
    float* M; long ldm; int rows, cols;
    float* T; long ldt;
    float* W; double* gpart;
    int groups;
};
size_t lot_scratch_bytes(int cols, int groups) {
    const size_t lots = (cols + 15) / 16, parts = kLotParts * kLotTiles;      // tiles of W, with all their parts or alone
    return (size_t)groups * 2048 + (lots > parts ? lots : parts) * 1024;
}

struct Meeting {                           // what the other workgroups wrote before is there afterwards
    unsigned long long* arrived; int groups; unsigned* flags;
    unsigned long long due = 0;
    __device__ __forceinline__ void operator()() {
        due += groups;
        store_barrier();
        if (threadIdx.x == 0) {
            (void)__hip_atomic_fetch_add(arrived, 1ull, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
            (void)handover_wait(arrived, due, kMeetTicks, flags);
        }
        __syncthreads();
    }
};

// +1 or -1 by row and column: the bits of both well mixed
__device__ __forceinline__ float random_sign(unsigned row, unsigned col, unsigned turn) {
    unsigned h = row * 0x9E3779B1u + col * 0x85EBCA77u + turn * 0xC2B2AE3Du;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        h ^= h >> 15;
        h *= 0x2C1B3C6Du;
    }
    return (h ^ (h >> 16)) & 1u ? 1.f : -1.f;
}

// The turns of a lot of w columns S against the first 16 * tiles columns of M (no more than there are).  c0 >= 0: S is M's columns from c0 on
// and T gets its columns; returns those that have vanished.  c0 < 0: such columns become random ones by `seed`, until none is left.
// *finite: cleared, alike in all workgroups, where S is not.
__device__ __forceinline__ unsigned turn_lot(const LotJob& b, LotShared& sh, Meeting& meet, float* S, long lds_, int w, int c0, int tiles,
                                             int seed, bool* finite) {
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int wg = blockIdx.x, nwg = b.groups, rows = b.rows;
    const int depth = 16 * tiles < b.cols ? 16 * tiles : b.cols;
    const int groups = (rows + 15) / 16 < nwg ? (rows + 15) / 16 : nwg;
    int wparts = tiles > kLotTiles || tiles == 0 ? 1 : nwg / tiles;
    wparts = wparts < 1 ? 1 : (wparts > kLotParts ? kLotParts : wparts);
    const int chunk = ((rows + wparts - 1) / wparts + 15) / 16 * 16;
    const long wstride = (long)tiles * 256;
    unsigned fresh = ~0u, empty = 0u;      // columns that no turn has seen, and those that have vanished
    for (int turn = 0; turn < kTurns; ++turn) {
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));      // addresses of all phases do not fit the registers across turns
        const int lane = tid & 63, c = lane & 15, g = lane >> 4, ei = tid >> 4, ej = tid & 15;
        // W: a tile a workgroup, cut along the rows, or two side by side, whose rows share their cache lines
        auto project = [&](int t0, int r0, int r1, float* out, auto count) {
            constexpr int NT = decltype(count)::value;
            const float *pq[NT], *ps = S + (c < w ? c : 0) + (long)g * lds_;
            f32x4 acc[NT] = {};
#pragma unroll
            for (int i = 0; i < NT; ++i) {
                const int qc = 16 * (t0 + i) + c;
                pq[i] = b.M + (qc < b.cols ? qc : b.cols - 1) + (long)g * b.ldm;
            }
            int k = r0 + 4 * wave;
#pragma unroll 8
            for (; k + 4 <= r1; k += 16) {
                const float v = ps[(long)k * lds_];
#pragma unroll
                for (int i = 0; i < NT; ++i) acc[i] = MFMA32(pq[i][(long)k * b.ldm], v, acc[i]);
            }
            if (k < r1) {
                const bool in = k + g < r1;
                const float v = in ? ps[(long)k * lds_] : 0.f;
#pragma unroll
                for (int i = 0; i < NT; ++i) acc[i] = MFMA32(in ? pq[i][(long)k * b.ldm] : 0.f, v, acc[i]);
            }
#pragma unroll
            for (int i = 0; i < NT; ++i) {
                const int t = t0 + i;
                __syncthreads();
#pragma unroll
                for (int r = 0; r < 4; ++r) sh.red[wave][(4 * g + r) * 16 + c] = acc[i][r];
                __syncthreads();
                if (t < tiles)
                    out[t * 256 + tid] = ej < w && 16 * t + ei < b.cols
                                             ? (sh.red[0][tid] + sh.red[1][tid]) + (sh.red[2][tid] + sh.red[3][tid]) : 0.f;
            }
        };
        if (wparts > 1) {
            for (int item = wg; item < tiles * wparts; item += nwg) {
                const int part = item / tiles, r0 = part * chunk, r1 = r0 + chunk < rows ? r0 + chunk : rows;
                project(item % tiles, r0, r1, b.W + part * wstride, std::integral_constant<int, 1>());
            }
        } else {
            for (int t = 2 * wg; t < tiles; t += 2 * nwg) project(t, 0, rows, b.W, std::integral_constant<int, 2>());
        }
        meet();
        if (wparts > 1) {
            for (int t = 0; t < tiles; ++t) {
                float v[kLotParts], x = 0.f;
#pragma unroll
                for (int p = 0; p < kLotParts; ++p) v[p] = p < wparts ? b.W[p * wstride + t * 256 + tid] : 0.f;
#pragma unroll
                for (int p = 0; p < kLotParts; ++p) x += v[p];
                sh.w[t][tid] = x;
            }
            __syncthreads();
        }
        if (c0 >= 0)
            for (int t = wg; t < tiles; t += nwg) {                       // T's part of it
                float* const part = wparts > 1 ? sh.w[t] : sh.red[0];
                if (wparts == 1) {
                    __syncthreads();
                    part[tid] = b.W[t * 256 + tid];
                    __syncthreads();
                }
                if (ej >= w) continue;
                float* o = b.T + (long)(16 * t + ei) * b.ldt + c0 + ej;
                if (turn == 0) {
                    *o = part[tid];
                } else {
                    float x = 0.f;
                    for (int p = 0; p <= ej; ++p) x += part[ei * 16 + p] * sh.u1[p * 16 + ej];
                    *o += x;
                }
            }
        // S -= M W and S^T S, by rows
        auto strips = [&](const float* W, auto count) {
            constexpr int NZ = decltype(count)::value;
            const float* row[NZ];
            f32x4 acc[NZ] = {};
#pragma unroll
            for (int z = 0; z < NZ; ++z) {
                const int r = 16 * (wg + z * nwg) + c;
                row[z] = b.M + (long)(r < rows ? r : rows - 1) * b.ldm + 4 * g;
            }
            auto take = [&](const float4 (&a)[NZ], const float* pw) {
                const float w0 = pw[0], w1 = pw[16], w2 = pw[32], w3 = pw[48];
#pragma unroll
                for (int z = 0; z < NZ; ++z) {
                    acc[z] = MFMA32(a[z].x, w0, acc[z]);
                    acc[z] = MFMA32(a[z].y, w1, acc[z]);
                    acc[z] = MFMA32(a[z].z, w2, acc[z]);
                    acc[z] = MFMA32(a[z].w, w3, acc[z]);
                }
            };
            const float* pw = W + 4 * g * 16 + c;
            int k = 16 * wave;
#pragma unroll 4
            for (; k + 16 <= depth; k += 64) {
                float4 a[NZ];
#pragma unroll
                for (int z = 0; z < NZ; ++z) a[z] = *reinterpret_cast<const float4*>(row[z] + k);
                take(a, pw + k * 16);
            }
            if (k < depth) {
                float4 a[NZ];
#pragma unroll
                for (int z = 0; z < NZ; ++z)
                    a[z] = k + 4 * g < depth ? load_quad(row[z] + k, depth - k - 4 * g) : make_float4(0.f, 0.f, 0.f, 0.f);
                take(a, pw + k * 16);
            }
#pragma unroll
            for (int z = 0; z < NZ; ++z) {
                __syncthreads();
#pragma unroll
                for (int r = 0; r < 4; ++r) sh.red[wave][(4 * g + r) * 16 + c] = acc[z][r];
                __syncthreads();
                const int r = 16 * (wg + z * nwg) + ei;
                sh.strip[z][tid] = r < rows && ej < w ? S[(long)r * lds_ + ej] - ((sh.red[0][tid] + sh.red[1][tid]) +
                                                                                 (sh.red[2][tid] + sh.red[3][tid]))
                                                      : 0.f;
            }
        };
        const int mine = (rows - 16 * wg + 16 * nwg - 1) / (16 * nwg);    // strips of this workgroup
        if (wparts > 1) {
            if (rows <= 16 * nwg) strips(&sh.w[0][0], std::integral_constant<int, 1>());
            else strips(&sh.w[0][0], std::integral_constant<int, kLotStrips>());
        } else if (rows <= 16 * nwg) {
            strips(b.W, std::integral_constant<int, 1>());
        } else if (rows <= 32 * nwg) {
            strips(b.W, std::integral_constant<int, 2>());
        } else {
            strips(b.W, std::integral_constant<int, kLotStrips>());
        }
        __syncthreads();
        f64x4 gram = {};
        if (wave == 0)
            for (int z = 0; z < mine; ++z)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const double v = (double)sh.strip[z][64 * r + lane];
                    gram = MFMA64(v, v, gram);
                }
        if (wave == 0 && wg < groups) tile_write(b.gpart + (long)wg * 256, lane, gram);
        meet();
        double s = 0.0;
#pragma unroll 32
        for (int z = 0; z < groups; ++z) s += b.gpart[(long)z * 256 + tid];
        if (ei == ej && (ej >= w || (empty >> ej & 1u))) s = 1.0;
        sh.gsum[ei * CLD + ej] = s;
        __syncthreads();
        if (wave == 0) {
            double d[16], x[16], mine = 0.0;
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                d[i] = sh.gsum[c * CLD + i];
                x[i] = 0.0;
            }
            const double len2 = sh.gsum[c * CLD + c];
            factor_pivots<0>(d, x, c, __builtin_fmax(len2 * 0x1p-44, 0x1p-600), row_lane<0>(d[0]), mine);
            // nothing, or, at unit length, nothing but rounding: below 2^-10
            const bool gone = c < w && (!(len2 >= kTiny) || (!(fresh >> c & 1u) && mine > 0x1p10));
            const unsigned mask = (unsigned)__ballot(gone) & 0xffffu;
            if (g == 0) {
#pragma unroll
                for (int i = 0; i < 16; ++i) sh.ut[i * 16 + c] = i <= c && !(mask >> i & 1u) ? (float)d[i] : 0.f;
                sh.rinv[c] = gone ? 0.f : (float)mine;
            }
            if (lane == 0) sh.gone = mask;
        }
        // columns of zeros are as they will be, and nothing depends on them
        const bool zero = sh.gsum[ei * CLD + ei] == 0.0 || sh.gsum[ej * CLD + ej] == 0.0;
        const double e = s - (ei == ej ? 1.0 : 0.0);
        double q2 = zero && c0 >= 0 ? 0.0 : e * e;
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) q2 += __shfl_xor(q2, o);
        if (lane == 0) sh.dist[wave] = q2;
        __syncthreads();
        const double off = (sh.dist[0] + sh.dist[1]) + (sh.dist[2] + sh.dist[3]);
        if (!(off < 0x1p1000)) {
            *finite = false;
            return empty;
        }
        const unsigned gone = sh.gone;
        if (tid < 16 * kLotStrips) {                                      // S <- S U^-1, by substitution
            const int r = 16 * (wg + (tid >> 4) * nwg) + (tid & 15);
            if (r < rows) {
                const float* s1 = sh.strip[tid >> 4] + (tid & 15) * 16;
                float q[16];
#pragma unroll
                for (int k = 0; k < 16; ++k) {
                    float v = s1[k];
#pragma unroll
                    for (int i = 0; i < k; ++i) v -= q[i] * sh.ut[i * 16 + k];
                    q[k] = v * sh.rinv[k];
                    asm volatile("" ::: "memory");     // the factor does not fit the registers
                }
                if (c0 < 0 && gone != 0u) {
                    const float unit = __builtin_amdgcn_rsqf((float)rows);
                    for (int k = 0; k < 16; ++k)
                        if (gone >> k & 1u) S[(long)r * lds_ + k] = unit * random_sign(r, seed + k, turn);
                }
#pragma unroll
                for (int k = 0; k < 16; ++k)
                    if (k < w && (c0 >= 0 || !(gone >> k & 1u))) S[(long)r * lds_ + k] = q[k];
            }
        }
        if (c0 >= 0) {
            float v = sh.ut[tid];                                         // the product of the lot's factors so far
            if (turn > 0) {
                v = 0.f;
                for (int p = ei; p <= ej; ++p) v += sh.ut[ei * 16 + p] * sh.u1[p * 16 + ej];
            }
            __syncthreads();
            sh.u1[tid] = v;
            if (wg == 0 && ei <= ej && ej < w) b.T[(long)(c0 + ei) * b.ldt + c0 + ej] = v;
            empty |= gone;
        }
        meet();
        // (off: without columns of zeros)
        if (off < kSettled && (c0 >= 0 || gone == 0u)) break;
        fresh = c0 >= 0 ? 0u : gone;
    }
    return empty;
}

// ---- Q = A U^-1 ---------------------------------------------------------------------------------------------------
// RT times 16 rows a workgroup, by substitution over the 64 columns of each diagonal block: T_s = A_s - sum_i Q_i U_is, Q_s = T_s
// inv_s.  fp32 matrix instructions; U and the inverses come from L2 in operand layout, 64 rows of them a step ahead.
// Bound: the chain of ten steps of 64 k, 16 products each per 16 rows, and two barriers a block.
// Where U's columns cancel by more than 2^5 against each other the products with its inverse lose as much of R U = A.  Substitution
// column by column loses none whatever U: 16 columns at a time, a thread a row, and products for what is right of them.
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

// the same by substitution over 16 columns at a time
template <int RT>
__device__ __forceinline__ void substitute_rows(float (*buf)[SLD], float* tile, const float* __restrict__ U, long ldu, int cols, int tid) {
    const int lane = tid & 63, wave = tid >> 6, c = lane & 15, g = lane >> 4, ei = tid >> 4, ej = tid & 15;
    for (int l = 0; 16 * l < cols; ++l) {
        const int j0 = 16 * l;
        const float u = j0 + ej < cols && ei <= ej ? U[(long)(j0 + ei) * ldu + j0 + ej] : 0.f;
        tile[tid] = ei < ej ? u : (u > 0.f ? 1.f / u : 0.f);           // (zero: a column that has vanished, or one past the last)
        float b[GT / 4][4];                  // U right of the tile, 16 columns in four a wavefront
#pragma unroll
        for (int t = 0; t < GT / 4; ++t) {
            const int col = j0 + 16 * (1 + wave + 4 * t) + c;
#pragma unroll
            for (int q = 0; q < 4; ++q) b[t][q] = col < cols ? U[(long)(j0 + 4 * q + g) * ldu + col] : 0.f;
        }
        __syncthreads();
        if (tid < 16 * RT) {
            float* row = buf[tid] + j0;
            float x[16];
#pragma unroll
            for (int k = 0; k < 16; k += 4) *reinterpret_cast<float4*>(x + k) = *reinterpret_cast<const float4*>(row + k);
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                x[k] *= tile[k * 17];
#pragma unroll
                for (int i = k + 1; i < 16; ++i) x[i] -= x[k] * tile[k * 16 + i];
            }
#pragma unroll
            for (int k = 0; k < 16; k += 4) *reinterpret_cast<float4*>(row + k) = *reinterpret_cast<const float4*>(x + k);
        }
        __syncthreads();
#pragma unroll
        for (int t = 0; t < GT / 4; ++t) {
            const int c0 = j0 + 16 * (1 + wave + 4 * t);
            if (c0 >= cols) continue;
#pragma unroll
            for (int i = 0; i < RT; ++i) {
                f32x4 acc = {};
#pragma unroll
                for (int q = 0; q < 4; ++q) acc = MFMA32(buf[16 * i + c][j0 + 4 * q + g], b[t][q], acc);
#pragma unroll
                for (int r = 0; r < 4; ++r) buf[16 * i + 4 * g + r][c0 + c] -= acc[r];
            }
        }
        __syncthreads();
    }
}

// A (rows x cols) <- A U^-1, also written to R where that is given
template <int RT>
__global__ __launch_bounds__(256, RT == 1 ? 3 : 2) void block_solve_kernel(float* A, long lda, int rows, int cols, float* U, long ldu,
                                                          const float* __restrict__ inv, unsigned* words, void* scratch, float* R,
                                                          long ldr, unsigned* flags) {
    constexpr int SR = 16 * RT;
    constexpr size_t ROWS = sizeof(float) * SR * SLD, ROOM = ROWS > sizeof(LotShared) ? ROWS : sizeof(LotShared);
    __shared__ __attribute__((aligned(16))) char room[ROOM];
    __shared__ __attribute__((aligned(16))) float tile[256];
    float (*const q)[SLD] = reinterpret_cast<float (*)[SLD]>(room);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int r0 = blockIdx.x * SR;
    const unsigned mode = words[0];
    if (mode == kByLots) {
        LotShared& sh = *reinterpret_cast<LotShared*>(room);
        const int groups = (int)gridDim.x < kLotGroups ? (int)gridDim.x : kLotGroups;
        if ((int)blockIdx.x >= groups) return;
        double* const gpart = static_cast<double*>(scratch);
        const LotJob job{A, lda, rows, cols, U, ldu, reinterpret_cast<float*>(gpart + groups * 256), gpart, groups};
        Meeting meet{reinterpret_cast<unsigned long long*>(words + 2), groups, flags};
        bool finite = true;
        for (int l = 0; 16 * l < cols && finite; ++l)
            (void)turn_lot(job, sh, meet, A + 16 * l, lda, cols - 16 * l < 16 ? cols - 16 * l : 16, 16 * l, l, 0, &finite);
        if (R == nullptr) return;
        for (int r0 = 16 * blockIdx.x; r0 < rows; r0 += 16 * groups)      // (its own strips)
            for (int e = tid; e < 16 * cols; e += 256) {
                const int r = r0 + e / cols, k = e % cols;
                if (r < rows) R[(long)r * ldr + k] = A[(long)r * lda + k];
            }
        return;
    }
    const int c4 = 4 * (tid & 63);
#pragma unroll
    for (int i = 0; i < SR / 4; ++i) {
        const int r = (tid >> 6) + 4 * i;
        float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
        if (r0 + r < rows && c4 < cols) v = load_quad(A + (long)(r0 + r) * lda + c4, cols - c4);
        *reinterpret_cast<float4*>(&q[r][c4]) = v;
    }
    __syncthreads();
    if (mode == kSubstituted) substitute_rows<RT>(q, tile, U, ldu, cols, tid);
    else solve_rows<RT>(q, U, ldu, inv, cols, lane, wave);
#pragma unroll
    for (int i = 0; i < SR / 4; ++i) {
        const int r = (tid >> 6) + 4 * i;
        if (r0 + r >= rows || c4 >= cols) continue;
        const float4 v = *reinterpret_cast<const float4*>(&q[r][c4]);
        store_quad(A + (long)(r0 + r) * lda + c4, cols - c4, v);
        if (R != nullptr) store_quad(R + (long)(r0 + r) * ldr + c4, cols - c4, v);
    }
}

// ---- what the second pass may have left ------------------------------------------------------------------------------
// E = R^T R - I; then every lot of 16 columns with an entry of E above kOff, from the left, and U <- T U.  Columns that have
// vanished become, at the end and 16 at a time, random ones made orthogonal to all others.
// Where there is nothing to do 2 to 4 us.  One pair of columns parallel to 1e-5 or one column of zeros, which is E, a lot or two and their
// part of U: 0.22 and 0.47 ms at n = 1536, 0.4 and 2.2 at 4096; at 8192 12 ms, 10 of them E at 55 TFLOP/s.  Many lots: 40 us a turn at n =
// 600, 75 at 1536, 170 at 4096, from when on what 128 workgroups have under way is what bounds them.
constexpr float kOff = 7e-7f;
constexpr int kFinishGroups = 768;         // for E, at most: as many as there is room for at a time
__host__ __device__ constexpr int lot_groups_of(int n) { return (n + 15) / 16 < kLotGroups ? (n + 15) / 16 : kLotGroups; }

__global__ __launch_bounds__(256, 3) void finish_kernel(float* R, long ldr, int n, float* U, long ldu, float* T, long ldt, double* gpart,
                                                        float* spare, float* W, unsigned* words, unsigned* flags) {
    if (words[0] == 0u) return;
    const int nwg = lot_groups_of(n), all = gridDim.x;      // those beyond have their share of E and go
    constexpr int ELD = 72;                // rows of 64 two apart: 16 banks on, four rows side by side
    constexpr size_t TILES = sizeof(float) * 32 * 2 * ELD, ROOM = TILES > sizeof(LotShared) ? TILES : sizeof(LotShared);
    __shared__ __attribute__((aligned(16))) char room[ROOM];      // of E's tiles, then of the lots
    LotShared& sh = *reinterpret_cast<LotShared*>(room);
    __shared__ unsigned char todo[DQ_MAX_N / 16];
    __shared__ unsigned short dead[DQ_MAX_N / 16];     // a lot's columns that have vanished
    __shared__ int late_cols[16], late_n;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 15, g = lane >> 4, ei = tid >> 4, ej = tid & 15;
    const int wg = blockIdx.x, lots = (n + 15) / 16;
    const LotJob job{R, ldr, n, n, T, ldt, W, gpart, nwg};
    Meeting meet{reinterpret_cast<unsigned long long*>(words + 2), nwg, flags, (unsigned long long)(all - nwg)};
    // ---- the largest entry of E of every lot
    {
        // a tile of 64 x 64 a workgroup, 32 rows of R at a time through LDS, the next 32 on their way meanwhile
        const int nt = (n + 63) / 64, tiles = nt * (nt + 1) / 2, wm = (wave >> 1) * 32, wn = (wave & 1) * 32;
        float (*const rows)[2][ELD] = reinterpret_cast<float (*)[2][ELD]>(room);
        for (int t = wg; t < tiles; t += all) {
            int ti, tj;
            gram_tile(t, nt, ti, tj);
            float4 next[4];                // row tid / 16 + 16 i of the left and the right columns 4 (tid % 16) ..
            auto fetch = [&](int r0) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int r = r0 + ei + 16 * (i >> 1), k = 64 * (i & 1 ? tj : ti) + 4 * ej;
                    next[i] = r < n && k < n ? load_quad(R + (long)r * ldr + k, n - k) : make_float4(0.f, 0.f, 0.f, 0.f);
                }
            };
            double acc[2][2][4] = {};      // fp32 sums of 64 rows, summed in fp64
            f32x4 part[2][2] = {};
            fetch(0);
            for (int r0 = 0; r0 < n; r0 += 32) {
                __syncthreads();
#pragma unroll
                for (int i = 0; i < 4; ++i) *reinterpret_cast<float4*>(&rows[ei + 16 * (i >> 1)][i & 1][4 * ej]) = next[i];
                __syncthreads();
                if (r0 + 32 < n) fetch(r0 + 32);
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    float fa[2], fb[2];
#pragma unroll
                    for (int i = 0; i < 2; ++i) {
                        fa[i] = rows[4 * q + g][0][wm + 16 * i + c];
                        fb[i] = rows[4 * q + g][1][wn + 16 * i + c];
                    }
#pragma unroll
                    for (int i = 0; i < 2; ++i)
#pragma unroll
                        for (int j = 0; j < 2; ++j) part[i][j] = MFMA32(fa[i], fb[j], part[i][j]);
                }
                if ((r0 & 32) == 0 && r0 + 32 < n) continue;
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
#pragma unroll
                        for (int v = 0; v < 4; ++v) acc[i][j][v] += (double)part[i][j][v];
                        part[i][j] = f32x4{};
                    }
            }
            if (ti == tj && wm > wn) continue;
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int k = 64 * tj + wn + 16 * j + c;
                unsigned most = 0u;        // (as bits: a NaN is larger than all)
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const int r = 64 * ti + wm + 16 * i + 4 * g + v;
                        const unsigned e = __float_as_uint(fabsf((float)(acc[i][j][v] - (r == k ? 1.0 : 0.0))));
                        if (r <= k && k < n && e > most) most = e;
                    }
#pragma unroll
                for (int o = 32; o >= 1; o >>= 1) {
                    const unsigned other = (unsigned)__shfl_xor((int)most, o);
                    most = other > most ? other : most;
                }
                const int lot = 4 * tj + wn / 16 + j;
                if (lane == 0 && lot < lots) (void)atomicMax(words + 4 + lot, most);
            }
        }
    }
    if (wg >= nwg) {
        store_barrier();
        if (tid == 0) (void)__hip_atomic_fetch_add(meet.arrived, 1ull, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
        return;
    }
    meet();
    for (int l = tid; l < lots; l += 256) {
        dead[l] = 0;
        todo[l] = __hip_atomic_load(words + 4 + l, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) > __float_as_uint(kOff);
    }
    __syncthreads();
    // ---- the lots, then, behind them, the columns that have vanished
    bool finite = true;
    for (int l = 0;; ++l) {
        const bool late = l >= lots;
        int w = n - 16 * l < 16 ? n - 16 * l : 16;
        if (late) {
            if (tid == 0) {                // the next 16
                int m = 0;
                for (int i = 0; i < lots && m < 16; ++i) {
                    unsigned left = dead[i];
                    if (left == 0u) continue;
                    for (; left != 0u && m < 16; left &= left - 1u) late_cols[m++] = 16 * i + __ffs(left) - 1;
                    dead[i] = (unsigned short)left;
                }
                late_n = m;
            }
            __syncthreads();
            w = late_n;
            if (w == 0) break;
            const float unit = __builtin_amdgcn_rsqf((float)n);
            for (int r0 = 16 * wg; r0 < n; r0 += 16 * nwg)
                if (r0 + ei < n) spare[(r0 + ei) * 16 + ej] = ej < w ? unit * random_sign(r0 + ei, 16 * l + ej, kTurns) : 0.f;
            meet();
        } else if (!todo[l]) {
            continue;
        }
        const unsigned empty = turn_lot(job, sh, meet, late ? spare : R + 16 * l, late ? 16 : ldr, w, late ? -1 : 16 * l, late ? lots : l,
                                        16 * l, &finite);
        if (!finite) return;
        if (late) {
            for (int r0 = 16 * wg; r0 < n; r0 += 16 * nwg)
                if (r0 + ei < n && ej < w) R[(long)(r0 + ei) * ldr + late_cols[ej]] = spare[(r0 + ei) * 16 + ej];
            meet();
        } else if (tid == 0) {
            dead[l] = (unsigned short)empty;
            if (wg == 0 && empty != 0u) atomicOr(flags, DQ_FLAG_SINGULAR);
        }
        __syncthreads();
    }
    if (U == nullptr) return;
    // ---- U <- T U in place, 16 columns a workgroup, from the first 64 rows on: nothing is read that is new
    for (int s0 = 16 * wg; s0 < n; s0 += 16 * nwg) {
        const int last = s0 + 16 < n ? s0 + 16 : n, col = s0 + c < n ? s0 + c : n - 1;
        for (int b = 0; 64 * b < last; ++b) {
            const int i0 = 64 * b + 16 * wave;
            f32x4 acc = {};
            for (int l = i0 / 16; 16 * l < last; ++l) {
                if (!todo[l]) continue;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int i = i0 + c, k = 16 * l + 4 * q + g;
                    const float x = i <= k && k < n ? T[(long)i * ldt + k] - (i == k ? 1.f : 0.f) : 0.f;
                    acc = MFMA32(x, k < n ? U[(long)k * ldu + col] : 0.f, acc);
                }
            }
            __syncthreads();
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (i0 + 4 * g + r <= s0 + c && s0 + c < n) U[(long)(i0 + 4 * g + r) * ldu + s0 + c] += acc[r];
        }
    }
}

}  // namespace

size_t finish_scratch_bytes(int n) { return lot_scratch_bytes(n, lot_groups_of(n)) + (size_t)(n + 15) / 16 * 1024; }

hipError_t launch_finish(float* R, long ldr, int n, float* U, long ldu, float* T, long ldt, void* scratch, unsigned* words, unsigned* flags,
                         hipStream_t s) {
    if (n < 1 || n > DQ_MAX_N) return hipErrorInvalidValue;
    const int nt = (n + 63) / 64, tiles = nt * (nt + 1) / 2, most = tiles < kFinishGroups ? tiles : kFinishGroups;
    const int groups = lot_groups_of(n);
    double* gpart = static_cast<double*>(scratch);
    float* spare = reinterpret_cast<float*>(gpart + groups * 256);
    hipLaunchKernelGGL(finish_kernel, dim3(most > groups ? most : groups), dim3(256), 0, s, R, ldr, n, U, ldu, T, ldt, gpart, spare,
                       spare + (size_t)(n + 15) / 16 * 256, words, flags);
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

hipError_t launch_chol64(const double* G, int cols, float* U, long ldu, float* inv, unsigned* solve, unsigned* flags, const SecondPass& second,
                         unsigned long long* started, unsigned long long value, hipStream_t s) {
    if (cols < 1 || cols > GB) return hipErrorInvalidValue;
    hipLaunchKernelGGL(chol64_kernel, dim3(1), dim3(64 * CHOL_WAVES), 0, s, G, cols, U, ldu, inv, solve, flags, second, started,
                       value);
    return hipGetLastError();
}

// 16 rows a workgroup where that fills the chip no more than once
static int solve_groups(int rows) { return rows <= 4096 ? (rows + 15) / 16 : (rows + 31) / 32; }
size_t block_solve_scratch_bytes(int rows, int cols) { return lot_scratch_bytes(cols, solve_groups(rows) < kLotGroups ? solve_groups(rows) : kLotGroups); }

hipError_t launch_block_solve(float* A, long lda, int rows, int cols, float* U, long ldu, const float* inv, unsigned* words, void* scratch,
                              float* R, long ldr, unsigned* flags, hipStream_t s) {
    if (rows < 1 || rows > DQ_MAX_N || cols < 1 || cols > GB) return hipErrorInvalidValue;
    if (rows <= 4096)
        hipLaunchKernelGGL(block_solve_kernel<1>, dim3(solve_groups(rows)), dim3(256), 0, s, A, lda, rows, cols, U, ldu, inv, words, scratch,
                           R, ldr, flags);
    else
        hipLaunchKernelGGL(block_solve_kernel<2>, dim3(solve_groups(rows)), dim3(256), 0, s, A, lda, rows, cols, U, ldu, inv, words, scratch,
                           R, ldr, flags);
    return hipGetLastError();
}

}  // namespace dq
