// fp32 GEMM on the CDNA4 matrix cores (v_mfma_f32_32x32x2_f32), LDS-staged, double-buffered.
//
//   C (M x N) = alpha * op(A) * op(B) + beta * C
//
// Workgroup: 256 threads = 4 wavefronts; workgroup tile 128 x 128 (64 x 256 for M <= 64, 256 x 64 for N <= 64),
// wavefront tile 64 x 64 = 2 x 2 MFMA tiles of 32 x 32; K step 16.  Both operand tiles live in LDS as [k][mn]
// (mn contiguous), so every MFMA operand fetch is a conflict-free 32-float row segment.
//
// MFMA 32x32x2 f32 lane layout (lane l of 64):  A operand a = A[m = l % 32][k = l / 32],
// B operand b = B[k = l / 32][n = l % 32], accumulator register v (0..15) holds
// D[m = 8*(v/4) + 4*(l/32) + v%4][n = l % 32].
//
// This kernel serves the trailing updates of the blocked Householder QR (Alg. 2 in compact-WY form),
// the accumulation of the orthogonal factor, the fp32 X @ R / X^T @ dY products and the three products
// of the derivative through Z = R U (the last step of Alg. 1).
#include "dq_internal.h"

namespace dq {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

namespace {


struct OperandView {
    const float* p; long ld;
    int row_lim, col_lim;   // storage rows / cols that may be read (others read as 0)
    int vec;                // 16-byte vector loads allowed
    int unit_lower_cols;    // storage columns < this get the unit-lower-trapezoid treatment (0: none)
};

__device__ __forceinline__ float4 load4_guarded(const OperandView& o, int sr, int sc) {
    float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
    if (sr < o.row_lim) {
        const float* q = o.p + (long)sr * o.ld + sc;
        if (o.vec && sc + 3 < o.col_lim) {
            v = *reinterpret_cast<const float4*>(q);
        } else {
            if (sc + 0 < o.col_lim) v.x = q[0];
            if (sc + 1 < o.col_lim) v.y = q[1];
            if (sc + 2 < o.col_lim) v.z = q[2];
            if (sc + 3 < o.col_lim) v.w = q[3];
        }
        if (o.unit_lower_cols > 0) {
            float* e = reinterpret_cast<float*>(&v);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int c = sc + j;
                if (c < o.unit_lower_cols && c < o.col_lim) e[j] = (sr > c) ? e[j] : (sr == c ? 1.f : 0.f);
            }
        }
    }
    return v;
}

// KC = true : storage is (mn, k) with k contiguous  -> transposing store into LDS [k][mn]
// KC = false: storage is (k, mn) with mn contiguous -> straight 16-byte store
// ROWS = extent of the tile along mn, BK along k; every thread moves ROWS * BK / 1024 float4.
template <bool KC, int ROWS, int BK>
__device__ __forceinline__ void fetch_tile(const OperandView& o, int mn0, int k0, int tid,
                                           float4 (&frag)[ROWS * BK / 1024]) {
#pragma unroll
    for (int i = 0; i < ROWS * BK / 1024; ++i) {
        const int f = tid + 256 * i;
        if (KC) {
            const int r = f / (BK / 4), kq = (f % (BK / 4)) << 2;
            frag[i] = load4_guarded(o, mn0 + r, k0 + kq);
        } else {
            const int kr = f / (ROWS / 4), c4 = (f % (ROWS / 4)) << 2;
            frag[i] = load4_guarded(o, k0 + kr, mn0 + c4);
        }
    }
}

// The same for a tile that lies inside the operand with 16-byte aligned rows and needs no mask: plain 16-byte loads.
template <bool KC, int ROWS, int BK>
__device__ __forceinline__ void fetch_tile_inner(const float* __restrict__ p, long ld, int mn0, int k0, int tid,
                                                 float4 (&frag)[ROWS * BK / 1024]) {
#pragma unroll
    for (int i = 0; i < ROWS * BK / 1024; ++i) {
        const int f = tid + 256 * i;
        if (KC) {
            const int r = f / (BK / 4), kq = (f % (BK / 4)) << 2;
            frag[i] = *reinterpret_cast<const float4*>(p + (long)(mn0 + r) * ld + k0 + kq);
        } else {
            const int kr = f / (ROWS / 4), c4 = (f % (ROWS / 4)) << 2;
            frag[i] = *reinterpret_cast<const float4*>(p + (long)(k0 + kr) * ld + mn0 + c4);
        }
    }
}

template <bool KC, int ROWS, int BK>
__device__ __forceinline__ void stash_tile(float (*S)[ROWS + 4], int tid, const float4 (&frag)[ROWS * BK / 1024]) {
#pragma unroll
    for (int i = 0; i < ROWS * BK / 1024; ++i) {
        const int f = tid + 256 * i;
        if (KC) {
            const int r = f / (BK / 4), kq = (f % (BK / 4)) << 2;
            S[kq + 0][r] = frag[i].x;
            S[kq + 1][r] = frag[i].y;
            S[kq + 2][r] = frag[i].z;
            S[kq + 3][r] = frag[i].w;
        } else {
            const int kr = f / (ROWS / 4), c4 = (f % (ROWS / 4)) << 2;
            *reinterpret_cast<float4*>(&S[kr][c4]) = frag[i];
        }
    }
}

// C tile = alpha * acc + beta * C for the wavefront block of 32 WT x 32 WT at (m0 + wm, n0 + wn); inner: the workgroup's
// tile lies wholly inside C.
template <int WT>
__device__ __forceinline__ void store_tile(const GemmF32& g, long bz, int z, f32x16 (&acc)[WT][WT], int m0, int n0, int wm,
                                           int wn, int lrow, int lk, bool inner) {
    float* C = g.C + bz * g.batch_c + (long)z * g.split_stride;
    // the scale of the product may also carry a factor that only the device knows (a step size formed by a kernel)
    const float alpha = g.alpha_dev != nullptr ? g.alpha * *g.alpha_dev : g.alpha, beta = g.beta;
    if (inner) {
        // one base pointer per 32 x 32 block and constant row offsets from it
        float* cb[WT][WT];
#pragma unroll
        for (int i = 0; i < WT; ++i)
#pragma unroll
            for (int j = 0; j < WT; ++j) cb[i][j] = C + (long)(m0 + wm + i * 32 + 4 * lk) * g.ldc + n0 + wn + j * 32 + lrow;
        if (beta != 0.f) {
            float cin[WT][WT][16];
#pragma unroll
            for (int i = 0; i < WT; ++i)
#pragma unroll
                for (int j = 0; j < WT; ++j)
#pragma unroll
                    for (int v = 0; v < 16; ++v) cin[i][j][v] = cb[i][j][(long)(8 * (v >> 2) + (v & 3)) * g.ldc];
#pragma unroll
            for (int i = 0; i < WT; ++i)
#pragma unroll
                for (int j = 0; j < WT; ++j)
#pragma unroll
                    for (int v = 0; v < 16; ++v) acc[i][j][v] = alpha * acc[i][j][v] + beta * cin[i][j][v];
        } else {
#pragma unroll
            for (int i = 0; i < WT; ++i)
#pragma unroll
                for (int j = 0; j < WT; ++j)
#pragma unroll
                    for (int v = 0; v < 16; ++v) acc[i][j][v] *= alpha;
        }
#pragma unroll
        for (int i = 0; i < WT; ++i)
#pragma unroll
            for (int j = 0; j < WT; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) cb[i][j][(long)(8 * (v >> 2) + (v & 3)) * g.ldc] = acc[i][j][v];
    } else {
    // All reads of C are issued before the first write: interleaved they would serialise on possible aliasing and
    // expose one memory round trip per element.
    if (beta != 0.f) {
#pragma unroll
        for (int i = 0; i < WT; ++i) {
#pragma unroll
            for (int j = 0; j < WT; ++j) {
                const int col = n0 + wn + j * 32 + lrow;
                float cin[16];
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int row = m0 + wm + i * 32 + 8 * (v >> 2) + 4 * lk + (v & 3);
                    cin[v] = (row < g.M && col < g.N) ? C[(long)row * g.ldc + col] : 0.f;
                }
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[i][j][v] = alpha * acc[i][j][v] + beta * cin[v];
            }
        }
    } else {
#pragma unroll
        for (int i = 0; i < WT; ++i)
#pragma unroll
            for (int j = 0; j < WT; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[i][j][v] *= alpha;
    }
#pragma unroll
    for (int i = 0; i < WT; ++i) {
#pragma unroll
        for (int j = 0; j < WT; ++j) {
            const int col = n0 + wn + j * 32 + lrow;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int row = m0 + wm + i * 32 + 8 * (v >> 2) + 4 * lk + (v & 3);
                if (row < g.M && col < g.N) C[(long)row * g.ldc + col] = acc[i][j][v];
            }
        }
    }
    }   // guarded epilogue
}

// acc += the k in [kb, ke) of a workgroup's BM x BN tile at (m0, n0) on the fp32 matrix cores; inner: rows and block wholly
// inside the matrices, with aligned rows and out of reach of the unit-lower masks.
template <bool TA, bool TB, int BM, int BN, int WT, int BK>
__device__ __forceinline__ void multiply_f32(const OperandView& oa, const OperandView& ob, bool inner, int m0, int n0, int kb,
                                             int ke, float (*As)[BK][BM + 4], float (*Bs)[BK][BN + 4], int tid, int wm, int wn,
                                             int lrow, int lk, f32x16 (&acc)[WT][WT]) {
    const int nk = ke > kb ? (ke - kb + BK - 1) / BK : 0;
    float4 fa[BM * BK / 1024], fb[BN * BK / 1024];
    auto fetch_both = [&](int k0) {
        if (inner && k0 + BK <= ke) {
            fetch_tile_inner<!TA, BM, BK>(oa.p, oa.ld, m0, k0, tid, fa);
            fetch_tile_inner<TB, BN, BK>(ob.p, ob.ld, n0, k0, tid, fb);
        } else {
            fetch_tile<!TA, BM, BK>(oa, m0, k0, tid, fa);
            fetch_tile<TB, BN, BK>(ob, n0, k0, tid, fb);
        }
    };
    if (nk > 0) {
        fetch_both(kb);
        stash_tile<!TA, BM, BK>(As[0], tid, fa);
        stash_tile<TB, BN, BK>(Bs[0], tid, fb);
    }
    __syncthreads();
    for (int kt = 0; kt < nk; ++kt) {
        const int cur = kt & 1;
        if (kt + 1 < nk) fetch_both(kb + (kt + 1) * BK);
#pragma unroll
        for (int kk = 0; kk < BK; kk += 2) {
            float a[WT], b[WT];
#pragma unroll
            for (int i = 0; i < WT; ++i) a[i] = As[cur][kk + lk][wm + i * 32 + lrow];
#pragma unroll
            for (int j = 0; j < WT; ++j) b[j] = Bs[cur][kk + lk][wn + j * 32 + lrow];
#pragma unroll
            for (int i = 0; i < WT; ++i)
#pragma unroll
                for (int j = 0; j < WT; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i], b[j], acc[i][j], 0, 0, 0);
        }
        if (kt + 1 < nk) {
            stash_tile<!TA, BM, BK>(As[cur ^ 1], tid, fa);
            stash_tile<TB, BN, BK>(Bs[cur ^ 1], tid, fb);
        }
        __syncthreads();
    }
}

// BM x BN is the workgroup tile and WT the wavefront tile in units of 32 (wavefront tile 32*WT x 32*WT, four
// wavefronts): 128 x 128 (WT 2, waves 2 x 2), 64 x 256 (M <= 64) and 256 x 64 (N <= 64) for throughput, and
// 64 x 64 with WT 1 and a deeper K step for small latency-bound products that need many workgroups.
template <bool TA, bool TB, int BM, int BN, int WT, int BK>
__global__ __launch_bounds__(256) void gemm_f32_kernel(GemmF32 g, int tiles_m, int tiles_n, int avec, int bvec) {
    __shared__ __attribute__((aligned(16))) float As[2][BK][BM + 4];
    __shared__ __attribute__((aligned(16))) float Bs[2][BK][BN + 4];
    constexpr int WAVES_N = BN / (32 * WT);
    static_assert((BM / (32 * WT)) * WAVES_N == 4, "four wavefronts per workgroup");

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;

    // Workgroup ids are dealt round-robin to the 8 XCDs (each with its own L2): give each XCD a
    // contiguous run of tiles, and walk tiles in groups of 8 tile-rows so a run shares operand panels.
    const int nt = tiles_m * tiles_n;
    const int bid = blockIdx.x;
    const int q8 = nt >> 3, r8 = nt & 7;
    const int xcd = bid & 7;
    const int pid = xcd * q8 + (xcd < r8 ? xcd : r8) + (bid >> 3);
    const int group = 8 * tiles_n;
    const int gid = pid / group;
    const int first_m = gid * 8;
    const int gsz = (tiles_m - first_m) < 8 ? (tiles_m - first_m) : 8;
    int pid_m = first_m + (pid % group) % gsz;
    int pid_n = (pid % group) / gsz;
    if (g.b_strict_lower) {
        // The K loop of a tile starts at its column offset: tile columns are dealt out whole, longest first, so that
        // the long tiles do not start late and finish alone.
        pid_n = bid / tiles_m;
        pid_m = bid % tiles_m;
    }
    const int m0 = pid_m * BM, n0 = pid_n * BN;

    const int z = blockIdx.y;
    int kb = 0, ke = g.K;
    if (g.splits > 1) {
        kb = z * g.kchunk;
        ke = kb + g.kchunk < g.K ? kb + g.kchunk : g.K;
    }
    if (g.b_strict_lower) {
        const int lo = (n0 / BK) * BK;
        kb = kb > lo ? kb : lo;
    }
    if (g.a_upper) kb = kb > m0 ? kb : m0;

    OperandView oa, ob;
    const long bz = blockIdx.z;   // independent problem of a batched launch
    oa.p = g.A + bz * g.batch_a; oa.ld = g.lda; oa.vec = avec;
    oa.unit_lower_cols = g.a_unit_lower ? 0x7fffffff : 0;
    if (TA) { oa.row_lim = ke; oa.col_lim = g.M; } else { oa.row_lim = g.M; oa.col_lim = ke; }
    ob.p = g.B + bz * g.batch_b; ob.ld = g.ldb; ob.vec = bvec;
    ob.unit_lower_cols = g.b_unit_lower_cols;
    if (TB) { ob.row_lim = g.N; ob.col_lim = ke; } else { ob.row_lim = ke; ob.col_lim = g.N; }

    f32x16 acc[WT][WT];
#pragma unroll
    for (int i = 0; i < WT; ++i)
#pragma unroll
        for (int j = 0; j < WT; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

    const int wm = (wave / WAVES_N) * 32 * WT, wn = (wave % WAVES_N) * 32 * WT;
    const int lrow = lane & 31, lk = lane >> 5;

    // A tile whose operand rows and output block lie wholly inside the matrices, with aligned rows and out of reach
    // of the unit-lower masks, takes loaders and an epilogue without bounds checks: the checks cost more instructions
    // than the products of a short K loop.  Only a last K step that is cut short reads with checks.
    const bool inner = avec && bvec && m0 + BM <= g.M && n0 + BN <= g.N &&
                       (!g.a_unit_lower || (!TA && m0 >= ke)) && (g.b_unit_lower_cols == 0 || (TB && n0 >= ke));
    multiply_f32<TA, TB, BM, BN, WT, BK>(oa, ob, inner, m0, n0, kb, ke, As, Bs, tid, wm, wn, lrow, lk, acc);
    store_tile<WT>(g, bz, z, acc, m0, n0, wm, wn, lrow, lk, inner);
}

// ---- the same products on the bf16 matrix cores ------------------------------------------------------------------
// Every fp32 operand element is split into three bf16 terms on its way from the staging registers to LDS,
//   x = x1 + x2 + x3,  x1 = bf16(x), x2 = bf16(x - x1), x3 = bf16(x - x1 - x2)   (24 bits, both remainders exact in fp32),
// and six of the nine products of terms, (3,1) (1,3) (2,2) (2,1) (1,2) (1,1), are accumulated in fp32 (each bf16 product is
// exact there; with |x2| <= 2^-8 |x| and |x3| <= 2^-17 |x| the three left out are at most 2^-24 |a| |b| together, one fp32 rounding
// of the product, and below 2^-26 for all but a few per cent of pairs): the five small ones apart from (1,1), so that the large
// accumulator is rounded once per 16 k where the fp32 instruction rounds it 8 times.
// Bound: the fp32 matrix instructions deliver 157 TFLOP/s at most and held the kernel above at 105 to 128; six bf16 ones do
// the same work in 3/8 of the time.  Measured before / after: 8192 x 8192 x 256 with beta = 1 408 / 251 us, 4096 x 4096 x 64
// 43 / 32 us, 4096^3 1160 / 708 us (118 / 194 TFLOP/s), 2890^3 742 / 472 us; relative error against 64 bits 0.32 to 0.38 of the
// fp32 kernel's at every shape tried (0.8 to 0.87 with one accumulator for all six, at the same speed).
// 128 x 128 tiles, K step 32, four wavefronts of 64 x 64, ONE buffer of three planes per operand (60 KB) with the next K
// step's operands in registers: two workgroups share a compute unit, one splits and stores while the other multiplies.  A
// plane row holds 32 k (four 16-byte chunks) in 80 bytes, chunk c of row r stored at place c ^ (r / 16 % 4): the 8-byte stores
// of a transposed operand, whose lanes lie four rows apart, hit every bank twice, and eight consecutive rows are read without
// conflicts.  Counters at 5120^3: matrix cores 60 % busy, LDS 60 %, half of that bank conflicts.
constexpr int kX3Resident = 512;   // workgroups resident at a time: two on each of 256 compute units
constexpr int X3K = 32, X3LD = 40, X3PLANE = 128 * X3LD;   // K step; halfwords per row; per plane

__device__ __forceinline__ void split3_pair(float a, float b, uint32_t& p1, uint32_t& p2, uint32_t& p3) {
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    const f32x2 v = {a, b};
    p1 = __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
    const f32x2 r = {a - __builtin_bit_cast(float, p1 << 16), b - __builtin_bit_cast(float, p1 & 0xffff0000u)};
    p2 = __builtin_bit_cast(uint32_t, __builtin_convertvector(r, bf16x2));
    const f32x2 t = {r[0] - __builtin_bit_cast(float, p2 << 16), r[1] - __builtin_bit_cast(float, p2 & 0xffff0000u)};
    p3 = __builtin_bit_cast(uint32_t, __builtin_convertvector(t, bf16x2));
}

// four consecutive k of one row, at halfword offset `off` of a plane
__device__ __forceinline__ void split3_store4(bf16_t* S, int off, float e0, float e1, float e2, float e3) {
    uint2 q1, q2, q3;
    split3_pair(e0, e1, q1.x, q2.x, q3.x);
    split3_pair(e2, e3, q1.y, q2.y, q3.y);
    *reinterpret_cast<uint2*>(S + off) = q1;
    *reinterpret_cast<uint2*>(S + X3PLANE + off) = q2;
    *reinterpret_cast<uint2*>(S + 2 * X3PLANE + off) = q3;
}

// A thread moves four float4 of a 128 x 32 operand tile.  KC (k contiguous): row tid / 8 + 32 i, k 4 (tid % 8).  Otherwise
// the 4 x 4 block of k 4 (tid / 32) + i and rows 4 (tid % 32) .. + 3, transposed on the way to LDS.
template <bool KC>
__device__ __forceinline__ void x3_fetch(const OperandView& o, bool inner, int mn0, int k0, int tid, float4 (&q)[4]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int sr = KC ? mn0 + (tid >> 3) + 32 * i : k0 + 4 * (tid >> 5) + i;
        const int sc = KC ? k0 + 4 * (tid & 7) : mn0 + 4 * (tid & 31);
        q[i] = inner ? *reinterpret_cast<const float4*>(o.p + (long)sr * o.ld + sc) : load4_guarded(o, sr, sc);
    }
}

template <bool KC>
__device__ __forceinline__ void x3_stash(bf16_t* S, int tid, const float4 (&q)[4]) {
    if (KC) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int r = (tid >> 3) + 32 * i, c = (tid & 7) >> 1;
            split3_store4(S, r * X3LD + ((c ^ ((r >> 4) & 3)) << 3) + ((tid & 1) << 2), q[i].x, q[i].y, q[i].z, q[i].w);
        }
    } else {
        const int kb = tid >> 5, r = 4 * (tid & 31);
        const int off = r * X3LD + (((kb >> 1) ^ ((r >> 4) & 3)) << 3) + ((kb & 1) << 2);
        split3_store4(S, off, q[0].x, q[1].x, q[2].x, q[3].x);
        split3_store4(S, off + X3LD, q[0].y, q[1].y, q[2].y, q[3].y);
        split3_store4(S, off + 2 * X3LD, q[0].z, q[1].z, q[2].z, q[3].z);
        split3_store4(S, off + 3 * X3LD, q[0].w, q[1].w, q[2].w, q[3].w);
    }
}

// acc += the k in [kb, ke) of a workgroup's 128 x 128 tile at (m0, n0) from split operands (inner: as in multiply_f32)
template <bool TA, bool TB>
__device__ __forceinline__ void multiply_x3(const OperandView& oa, const OperandView& ob, bool inner, int m0, int n0, int kb,
                                            int ke, bf16_t* As, bf16_t* Bs, int tid, int wm, int wn, int lrow, int lk,
                                            f32x16 (&acc)[2][2]) {
    const int nk = ke > kb ? (ke - kb + X3K - 1) / X3K : 0;
    f32x16 low[2][2];   // the five small products of a pair of terms
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) low[i][j][v] = 0.f;
    float4 fa[4], fb[4];
    auto fetch_both = [&](int k0) {
        if (inner && k0 + X3K <= ke) {
            x3_fetch<!TA>(oa, true, m0, k0, tid, fa);
            x3_fetch<TB>(ob, true, n0, k0, tid, fb);
        } else {
            x3_fetch<!TA>(oa, false, m0, k0, tid, fa);
            x3_fetch<TB>(ob, false, n0, k0, tid, fb);
        }
    };
    if (nk > 0) fetch_both(kb);
    for (int kt = 0; kt < nk; ++kt) {
        x3_stash<!TA>(As, tid, fa);
        x3_stash<TB>(Bs, tid, fb);
        __syncthreads();
        if (kt + 1 < nk) fetch_both(kb + (kt + 1) * X3K);
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            bf16x8 a[2][3], b[2][3];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int ra = wm + i * 32 + lrow, rb = wn + i * 32 + lrow, ch = 2 * ks + lk;
                const int offa = ra * X3LD + ((ch ^ ((ra >> 4) & 3)) << 3), offb = rb * X3LD + ((ch ^ ((rb >> 4) & 3)) << 3);
#pragma unroll
                for (int p = 0; p < 3; ++p) {
                    a[i][p] = *reinterpret_cast<const bf16x8*>(As + p * X3PLANE + offa);
                    b[i][p] = *reinterpret_cast<const bf16x8*>(Bs + p * X3PLANE + offb);
                }
            }
            constexpr int PA[6] = {2, 0, 1, 1, 0, 0}, PB[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
            for (int t = 0; t < 6; ++t)
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
                        f32x16& d = t < 5 ? low[i][j] : acc[i][j];
                        d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i][PA[t]], b[j][PB[t]], d, 0, 0, 0);
                    }
        }
        __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] += low[i][j][v];
}

template <bool TA, bool TB>
__global__ __launch_bounds__(256, 2) void gemm_f32x3_kernel(GemmF32 g, int tiles_m, int tiles_n, int avec, int bvec,
                                                                 int whole, int pchunk) {
    __shared__ __attribute__((aligned(16))) bf16_t lds[6 * X3PLANE];
    bf16_t* const As = lds;
    bf16_t* const Bs = lds + 3 * X3PLANE;
    constexpr int BM = 128, BN = 128;
    static_assert(kGuardWords == 256, "one word per thread");
    const bool split = g.guard == nullptr || __syncthreads_or(g.guard[threadIdx.x] != 0u) == 0;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;

    // tile order as in the fp32 kernel; behind the first `whole` tiles the others follow in parts of pchunk k, all tiles of
    // one part side by side
    const int bid = blockIdx.x;
    const int q8 = whole >> 3, r8 = whole & 7;
    const int xcd = bid & 7;
    int pid = xcd * q8 + (xcd < r8 ? xcd : r8) + (bid >> 3);
    const int rest = tiles_m * tiles_n - whole;
    const bool in_parts = bid >= whole;
    if (in_parts) pid = whole + (bid - whole) % rest;
    const int group = 8 * tiles_n;
    const int gid = pid / group;
    const int first_m = gid * 8;
    const int gsz = (tiles_m - first_m) < 8 ? (tiles_m - first_m) : 8;
    int pid_m = first_m + (pid % group) % gsz;
    int pid_n = (pid % group) / gsz;
    if (g.b_strict_lower) {
        pid_n = bid / tiles_m;
        pid_m = bid % tiles_m;
    }
    const int m0 = pid_m * BM, n0 = pid_n * BN;

    const int z = blockIdx.y;
    int kb = 0, ke = g.K;
    if (g.splits > 1) {
        kb = z * g.kchunk;
        ke = kb + g.kchunk < g.K ? kb + g.kchunk : g.K;
    }
    if (in_parts) {
        kb = (bid - whole) / rest * pchunk;
        ke = kb + pchunk < g.K ? kb + pchunk : g.K;
    }
    if (g.b_strict_lower) kb = kb > n0 ? kb : n0;   // n0 is a multiple of the K step
    if (g.a_upper) kb = kb > m0 ? kb : m0;

    OperandView oa, ob;
    const long bz = blockIdx.z;
    oa.p = g.A + bz * g.batch_a; oa.ld = g.lda; oa.vec = avec;
    oa.unit_lower_cols = g.a_unit_lower ? 0x7fffffff : 0;
    if (TA) { oa.row_lim = ke; oa.col_lim = g.M; } else { oa.row_lim = g.M; oa.col_lim = ke; }
    ob.p = g.B + bz * g.batch_b; ob.ld = g.ldb; ob.vec = bvec;
    ob.unit_lower_cols = g.b_unit_lower_cols;
    if (TB) { ob.row_lim = g.N; ob.col_lim = ke; } else { ob.row_lim = ke; ob.col_lim = g.N; }

    f32x16 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

    const int wm = (wave >> 1) * 64, wn = (wave & 1) * 64;
    const int lrow = lane & 31, lk = lane >> 5;

    // loads without checks where the tile lies inside both operands and out of reach of their masks
    const bool inner = avec && bvec && m0 + BM <= g.M && n0 + BN <= g.N && (!g.a_unit_lower || (!TA && m0 >= ke)) &&
                       (g.b_unit_lower_cols == 0 || (TB && n0 >= ke));
    if (split) {
        multiply_x3<TA, TB>(oa, ob, inner, m0, n0, kb, ke, As, Bs, tid, wm, wn, lrow, lk, acc);
    } else {            // an operand entry has no split (see GemmF32::guard)
        constexpr int BK = 16;
        static_assert(2 * BK * (BM + 4) * sizeof(float) <= 3 * X3PLANE * sizeof(bf16_t), "both buffers in an operand's planes");
        multiply_f32<TA, TB, BM, BN, 2, BK>(oa, ob, inner, m0, n0, kb, ke, reinterpret_cast<float (*)[BK][BM + 4]>(As),
                                            reinterpret_cast<float (*)[BK][BN + 4]>(Bs), tid, wm, wn, lrow, lk, acc);
    }
    if (in_parts) {
        float* t = g.tail + (long)(bid - whole) * (BM * BN) + (wm + 4 * lk) * BN + wn + lrow;
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) t[(i * 32 + 8 * (v >> 2) + (v & 3)) * BN + j * 32] = acc[i][j][v];
        return;
    }
    store_tile<2>(g, bz, z, acc, m0, n0, wm, wn, lrow, lk, m0 + BM <= g.M && n0 + BN <= g.N);
}

// C = alpha * (sum of the parts) + beta * C for the tiles that were multiplied in parts: a workgroup takes 8 rows of a tile
__global__ __launch_bounds__(256) void x3_parts_kernel(GemmF32 g, int tiles_m, int tiles_n, int whole, int parts) {
    const int rest = tiles_m * tiles_n - whole;
    const int t = blockIdx.x >> 4, pid = whole + t;
    const int group = 8 * tiles_n;
    const int first_m = pid / group * 8;
    const int gsz = (tiles_m - first_m) < 8 ? (tiles_m - first_m) : 8;
    const int m0 = (first_m + (pid % group) % gsz) * 128, n0 = (pid % group) / gsz * 128;
    const int r = 8 * (blockIdx.x & 15) + (threadIdx.x >> 5), c = 4 * (threadIdx.x & 31);
    const float* p = g.tail + (long)t * (128 * 128) + r * 128 + c;
    float s[4] = {0.f, 0.f, 0.f, 0.f};
    for (int z = 0; z < parts; ++z) {
        const float4 v = *reinterpret_cast<const float4*>(p + (long)z * rest * (128 * 128));
        s[0] += v.x; s[1] += v.y; s[2] += v.z; s[3] += v.w;
    }
    if (m0 + r >= g.M) return;
    const float alpha = g.alpha_dev != nullptr ? g.alpha * *g.alpha_dev : g.alpha;
    float* C = g.C + (long)(m0 + r) * g.ldc + n0 + c;
#pragma unroll
    for (int e = 0; e < 4; ++e)
        if (n0 + c + e < g.N) C[e] = g.beta != 0.f ? alpha * s[e] + g.beta * C[e] : alpha * s[e];
}

__global__ __launch_bounds__(256) void splitk_reduce_kernel(const float* __restrict__ part, int splits, long stride,
                                                            long ldp, int rows, int cols, float alpha, float beta,
                                                            float* __restrict__ out, long ldo) {
    const long total = (long)rows * cols;
    for (long e = (long)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += (long)gridDim.x * blockDim.x) {
        const int r = (int)(e / cols), c = (int)(e % cols);
        float s = 0.f;
        const float* q = part + (long)r * ldp + c;
        int zz = 0;
        for (; zz + 8 <= splits; zz += 8) {     // eight independent loads in flight
            float t[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) t[u] = q[(long)(zz + u) * stride];
#pragma unroll
            for (int u = 0; u < 8; ++u) s += t[u];
        }
        for (; zz < splits; ++zz) s += q[(long)zz * stride];
        float* o = out + (long)r * ldo + c;
        float v = alpha * s;
        if (beta != 0.f) v += beta * *o;
        *o = v;
    }
}

// The same sum for rows that can be read 16 bytes at a time (cols, ldp, stride, ldo multiples of 4, aligned bases):
// one row piece of four columns per thread, no division per element, four layers in flight.
__global__ __launch_bounds__(256) void splitk_reduce4_kernel(const float* __restrict__ part, int splits, long stride,
                                                             long ldp, int rows, int cols4, float alpha, float beta,
                                                             float* __restrict__ out, long ldo) {
    const int c4 = blockIdx.x * 64 + (threadIdx.x & 63);
    if (c4 >= cols4) return;
    for (int r = blockIdx.y * 4 + (threadIdx.x >> 6); r < rows; r += gridDim.y * 4) {
        const float4* q = reinterpret_cast<const float4*>(part + (long)r * ldp) + c4;
        const long st4 = stride >> 2;
        float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
        int zz = 0;
        for (; zz + 4 <= splits; zz += 4) {
            float4 t[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) t[u] = q[(long)(zz + u) * st4];
#pragma unroll
            for (int u = 0; u < 4; ++u) { s.x += t[u].x; s.y += t[u].y; s.z += t[u].z; s.w += t[u].w; }
        }
        for (; zz < splits; ++zz) {
            const float4 t = q[(long)zz * st4];
            s.x += t.x; s.y += t.y; s.z += t.z; s.w += t.w;
        }
        float4* o = reinterpret_cast<float4*>(out + (long)r * ldo) + c4;
        float4 v = make_float4(alpha * s.x, alpha * s.y, alpha * s.z, alpha * s.w);
        if (beta != 0.f) {
            const float4 old = *o;
            v.x += beta * old.x; v.y += beta * old.y; v.z += beta * old.z; v.w += beta * old.w;
        }
        *o = v;
    }
}

}  // namespace

template <int BM, int BN, int WT, int BK>
static hipError_t launch_gemm_f32_tile(const GemmF32& g, hipStream_t s) {
    const int tiles_m = (g.M + BM - 1) / BM, tiles_n = (g.N + BN - 1) / BN;
    const int avec = ((reinterpret_cast<uintptr_t>(g.A) & 15) == 0 && (g.lda & 3) == 0 && (g.batch_a & 3) == 0) ? 1 : 0;
    const int bvec = ((reinterpret_cast<uintptr_t>(g.B) & 15) == 0 && (g.ldb & 3) == 0 && (g.batch_b & 3) == 0) ? 1 : 0;
    dim3 grid(tiles_m * tiles_n, g.splits > 1 ? g.splits : 1, g.batch > 1 ? g.batch : 1);
    dim3 block(256, 1, 1);
    if (g.ta && g.tb)
        hipLaunchKernelGGL((gemm_f32_kernel<true, true, BM, BN, WT, BK>), grid, block, 0, s, g, tiles_m, tiles_n, avec, bvec);
    else if (g.ta)
        hipLaunchKernelGGL((gemm_f32_kernel<true, false, BM, BN, WT, BK>), grid, block, 0, s, g, tiles_m, tiles_n, avec, bvec);
    else if (g.tb)
        hipLaunchKernelGGL((gemm_f32_kernel<false, true, BM, BN, WT, BK>), grid, block, 0, s, g, tiles_m, tiles_n, avec, bvec);
    else
        hipLaunchKernelGGL((gemm_f32_kernel<false, false, BM, BN, WT, BK>), grid, block, 0, s, g, tiles_m, tiles_n, avec, bvec);
    return hipGetLastError();
}

static hipError_t launch_gemm_f32x3(const GemmF32& g, hipStream_t s) {
    const int tiles_m = (g.M + 127) / 128, tiles_n = (g.N + 127) / 128;
    const int avec = ((reinterpret_cast<uintptr_t>(g.A) & 15) == 0 && (g.lda & 3) == 0 && (g.batch_a & 3) == 0) ? 1 : 0;
    const int bvec = ((reinterpret_cast<uintptr_t>(g.B) & 15) == 0 && (g.ldb & 3) == 0 && (g.batch_b & 3) == 0) ? 1 : 0;
    // 512 workgroups run at a time.  The tiles of a last round that leaves half of them idle or more are cut along K into as many
    // parts as there is room for (at least 256 k each: a part is written and read again, 128 KB per tile), summed by a
    // second launch: 2890^3, 529 tiles, 497 us whole; the fewer than 512 tiles of a product up to 2816 wide are all cut.
    const int tiles = tiles_m * tiles_n, rest = tiles % kX3Resident;
    int parts = 1;
    if (g.tail != nullptr && g.splits <= 1 && g.batch <= 1 && !g.b_strict_lower && !g.a_upper && g.K >= 768 && rest > 0) {
        parts = kX3Resident / rest;
        if (parts > g.K / 256) parts = g.K / 256;
        const long room = g.tail_floats / ((long)rest * 128 * 128);
        if (parts > room) parts = (int)room;
    }
    int whole = tiles, pchunk = 0;
    if (parts > 1) {
        whole = tiles - rest;
        pchunk = ((g.K + parts - 1) / parts + X3K - 1) / X3K * X3K;
        parts = (g.K + pchunk - 1) / pchunk;
    }
    dim3 grid(whole + (tiles - whole) * parts, g.splits > 1 ? g.splits : 1, g.batch > 1 ? g.batch : 1);
    dim3 block(256, 1, 1);
#define DQ_LAUNCH(TA, TB)                                                                                                \
    hipLaunchKernelGGL((gemm_f32x3_kernel<TA, TB>), grid, block, 0, s, g, tiles_m, tiles_n, avec, bvec, whole, pchunk)
    if (g.ta && g.tb) DQ_LAUNCH(true, true);
    else if (g.ta) DQ_LAUNCH(true, false);
    else if (g.tb) DQ_LAUNCH(false, true);
    else DQ_LAUNCH(false, false);
#undef DQ_LAUNCH
    if (whole < tiles)
        hipLaunchKernelGGL(x3_parts_kernel, dim3((tiles - whole) * 16), block, 0, s, g, tiles_m, tiles_n, whole, parts);
    return hipGetLastError();
}

// 1 = 64 x 256 tile, 2 = 256 x 64, 3 = 64 x 64 (many small workgroups), 0 = 128 x 128
static int gemm_f32_config(int M, int N, int splits) {
    const long big_tiles = (long)((M + 127) / 128) * ((N + 127) / 128) * (splits > 1 ? splits : 1);
    if (big_tiles < 96 && N <= 128) return 3;   // few output tiles: 64 x 64 tiles give more workgroups
    if (M <= 64 && N > 64) return 1;
    if (big_tiles < 96) return 3;      // would leave most compute units idle: use 64 x 64 tiles
    if (N <= 64) return 2;
    return 0;
}

bool gemm_f32_split_applies(int M, int N, int splits) { return gemm_f32_config(M, N, splits) == 0; }

int gemm_f32_tile_n(int M, int N) { return N <= 128 ? 64 : ((M <= 64) ? 256 : 128); }

hipError_t launch_gemm_f32(const GemmF32& g, hipStream_t s) {
    if (g.M <= 0 || g.N <= 0) return hipSuccess;
    switch (g.cfg >= 0 ? g.cfg : gemm_f32_config(g.M, g.N, g.splits)) {
        case 1: return launch_gemm_f32_tile<64, 256, 2, 16>(g, s);
        case 2: return launch_gemm_f32_tile<256, 64, 2, 16>(g, s);
        case 3: return launch_gemm_f32_tile<64, 64, 1, 32>(g, s);
        default:
            // a caller that allows it gets the products of this tile size from split operands
            if (g.x3) return launch_gemm_f32x3(g, s);
            return launch_gemm_f32_tile<128, 128, 2, 16>(g, s);
    }
}

hipError_t launch_splitk_reduce(const float* part, int splits, long stride, long ldp, int rows, int cols,
                                float alpha, float beta, float* out, long ldo, hipStream_t s) {
    if (rows <= 0 || cols <= 0) return hipSuccess;
    if ((cols & 3) == 0 && (ldp & 3) == 0 && (stride & 3) == 0 && (ldo & 3) == 0 &&
        (reinterpret_cast<uintptr_t>(part) & 15) == 0 && (reinterpret_cast<uintptr_t>(out) & 15) == 0) {
        const int cols4 = cols >> 2;
        int gy = (rows + 3) / 4;
        if (gy > 2048) gy = 2048;
        hipLaunchKernelGGL(splitk_reduce4_kernel, dim3((cols4 + 63) / 64, gy), dim3(256), 0, s, part, splits, stride,
                           ldp, rows, cols4, alpha, beta, out, ldo);
        return hipGetLastError();
    }
    const long total = (long)rows * cols;
    long blocks = (total + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(splitk_reduce_kernel, dim3((unsigned)blocks), dim3(256), 0, s, part, splits, stride, ldp,
                       rows, cols, alpha, beta, out, ldo);
    return hipGetLastError();
}

}  // namespace dq
