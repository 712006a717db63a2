// Batched path for small rotations, n <= 128 (per-head rotations; the "heads" workload has 64 of size 128): every problem
// of a batch runs in the same launch.
//   * heads_qr_kernel: R, U = qr(Z) for one latent per workgroup, entirely on chip.  Alg. 2 as printed:
//     column by column, the reflector is applied to the trailing columns of the matrix and accumulated into the
//     orthogonal factor in the same step (A <- H A, Q <- Q H); the signs are then fixed so that diag(U) >= 0.
//   * heads_rlg_kernel: Alg. 1, rotation and loss steps, fused for bf16 activations.  A workgroup streams 64-token tiles of X once;
//     Y = X R (R as two bf16 planes held in registers), the Whip loss and its gradient (Eq. 4) and the tile's
//     contribution to G = X^T dY are formed on chip: Y and dY never reach HBM.
//   * heads_reduce_kernel: sums the per-workgroup partial G and loss.
//   * heads_backward_kernel: the derivative through the QR and the update, one problem per workgroup, out of LDS.
#include <type_traits>

#include "dq_internal.h"
#include "dq_wave.h"


namespace dq {
namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

constexpr int HN = kHeadDim;     // largest matrix size of this path

__device__ __forceinline__ double wave_total(double v) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

__device__ __forceinline__ float lane_value(float v, int l) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}

__device__ __forceinline__ uint32_t to_bf16_rne(float f) {
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (u >> 16) | 0x40u;   // NaN stays NaN
    u += 0x7fffu + ((u >> 16) & 1u);
    return u >> 16;
}

// ------------------------------------------------------------------------------------------------ S1 + S2
// Alg. 2 with the unnormalised reflector vector: for column j, x = A[j:, j], beta = -sign(x_0) ||x||,
// u = x - beta e_0, H = I - gamma u u^T with gamma = 2 / u^T u  (the same reflection as the paper's normalised v);
// a column that is already zero below the diagonal gets H = I.
// 512 threads: four adjacent lanes ("item" i = tid / 4, part h = tid % 4) hold one column of A AND one row of Q in
// registers, lane part h owning the 4-row groups g with g % 4 == h of both.  Both get x <- x - gamma (u . x) u (the
// column only if it lies right of j), with ONE read of u from LDS for the two, the partial dot products of the four
// lanes meeting through DPP.  Columns are dealt to the items round-robin over the wavefronts (item i holds column
// 8 (i % 16) + i / 16), so that every wavefront keeps live columns to the end.  The owners of column j + 1 publish it in
// LDS at the end of step j, so a step needs one barrier; every wavefront forms the column norm itself.  Rows are handled
// in blocks of 16: blocks above the diagonal block are skipped (the block index is a template parameter, so register
// indices are static and a step runs straight-line code), the diagonal block substitutes u_0 for the raw pivot and
// zero above it.
constexpr int QS = 4;                   // lanes per column / row
constexpr int QB = 16;                  // rows per block = 4 groups, one per lane part
// NG: 4-row groups held by a thread (of its column and of its row) = blocks of 16 rows carried, 4, 6 or 8: the rest of a
// smaller matrix is zero (32 problems of order 80: 91 us with all 8 carried, 74 with 6).  Bound: the vector ALU and the
// chain of dependent operations of a step, half and half; four workgroups per problem, each with all of A and a quarter
// of Q's rows, took as long as one.

__device__ __forceinline__ int item_column(int item) { return 8 * (item & 15) + (item >> 4); }
__device__ __forceinline__ int column_item(int c) { return 16 * (c & 7) + (c >> 3); }

// rows of this thread's k-th group: 4 * (k * QS + h) .. + 3
template <int JB, int NG>
__device__ __forceinline__ void publish_from(float* cb, const float (&x)[4 * NG], int h, int j) {
#pragma unroll
    for (int k = JB; k < NG; ++k) {
        const int i = 4 * (k * QS + h);
        float4 v = make_float4(x[4 * k], x[4 * k + 1], x[4 * k + 2], x[4 * k + 3]);
        if (k == JB) {   // diagonal block: entries above the diagonal are published as zero
            v.x = i >= j ? v.x : 0.f; v.y = i + 1 >= j ? v.y : 0.f; v.z = i + 2 >= j ? v.z : 0.f; v.w = i + 3 >= j ? v.w : 0.f;
        }
        *reinterpret_cast<float4*>(cb + i) = v;
    }
}

// x <- x - gamma (u . x) u for this thread's part of its column (if live) and of its row of Q, for block row JB = j / 16
// of the pivot; u is the published column with u_0 = uj in place of the raw pivot.  LARGE: gamma times g2 in place of gamma
template <int JB, int NG, bool LARGE>
__device__ __forceinline__ void reflect_from(const float* cb, float (&xc)[4 * NG], float (&xq)[4 * NG], bool col_live,
                                             int h, int j, float uj, float gamma, float g2) {
    float4 u[NG - JB];
#pragma unroll
    for (int k = JB; k < NG; ++k) u[k - JB] = *reinterpret_cast<const float4*>(cb + 4 * (k * QS + h));
    {   // diagonal block: the pivot entry becomes u_0 (the entries above it were published as zero)
        const int i = 4 * (JB * QS + h);
        float4& v = u[0];
        v.x = i == j ? uj : v.x; v.y = i + 1 == j ? uj : v.y; v.z = i + 2 == j ? uj : v.z; v.w = i + 3 == j ? uj : v.w;
    }
    // four independent partial sums per dot product: a lone dependent chain of 32 FMAs would set the pace of the step
    float c0 = 0.f, c1 = 0.f, c2 = 0.f, c3 = 0.f, q0 = 0.f, q1 = 0.f, q2 = 0.f, q3 = 0.f;
#pragma unroll
    for (int k = JB; k < NG; ++k) {
        const float4 v = u[k - JB];
        c0 += v.x * xc[4 * k]; c1 += v.y * xc[4 * k + 1]; c2 += v.z * xc[4 * k + 2]; c3 += v.w * xc[4 * k + 3];
        q0 += v.x * xq[4 * k]; q1 += v.y * xq[4 * k + 1]; q2 += v.z * xq[4 * k + 2]; q3 += v.w * xq[4 * k + 3];
    }
    float dc = (c0 + c1) + (c2 + c3), dq = (q0 + q1) + (q2 + q3);
    dc += lane_xor<1>(dc); dq += lane_xor<1>(dq);
    dc += lane_xor<2>(dc); dq += lane_xor<2>(dq);
    const float fc = col_live ? gamma * (LARGE ? g2 * dc : dc) : 0.f;
    const float fq = gamma * (LARGE ? g2 * dq : dq);
#pragma unroll
    for (int k = JB; k < NG; ++k) {
        const float4 v = u[k - JB];
        xc[4 * k] -= fc * v.x; xc[4 * k + 1] -= fc * v.y; xc[4 * k + 2] -= fc * v.z; xc[4 * k + 3] -= fc * v.w;
        xq[4 * k] -= fq * v.x; xq[4 * k + 1] -= fq * v.y; xq[4 * k + 2] -= fq * v.z; xq[4 * k + 3] -= fq * v.w;
    }
}

#define DQ_BLOCK_SWITCH(jb, CALL)                                                                  \
    switch (jb) {                                                                                  \
        case 0: if constexpr (NG > 0) { CALL(0); } break;                                          \
        case 1: if constexpr (NG > 1) { CALL(1); } break;                                          \
        case 2: if constexpr (NG > 2) { CALL(2); } break;                                          \
        case 3: if constexpr (NG > 3) { CALL(3); } break;                                          \
        case 4: if constexpr (NG > 4) { CALL(4); } break;                                          \
        case 5: if constexpr (NG > 5) { CALL(5); } break;                                          \
        case 6: if constexpr (NG > 6) { CALL(6); } break;                                          \
        case 7: if constexpr (NG > 7) { CALL(7); } break;                                          \
        default: break;                                                                            \
    }

// FULL: n == 128, nothing to guard.
template <bool FULL, int NG>
__global__ __launch_bounds__(HN * QS) void heads_qr_kernel(const float* __restrict__ Z, long ldz, long sz,
                                                           float* __restrict__ R, long ldr, long sr,
                                                           float* __restrict__ U, long ldu, long su, int n_,
                                                           unsigned* flags) {
    const int n = FULL ? HN : n_;
    __shared__ __attribute__((aligned(16))) float cbuf[2][HN];
    __shared__ __attribute__((aligned(16))) float sgn[HN];
    const int tid = threadIdx.x, lane = tid & 63;
    const int item = tid / QS, h = tid % QS;
    const int col = item_column(item);   // this thread's column of A; its row of Q is `item`
    const float* Zp = Z + (long)blockIdx.x * sz;
    float xc[4 * NG], xq[4 * NG], mydiag = 0.f;
    // The factorisation.  Columns of norm 2^62 and more: 2 / u . u is no normal fp32 number though the squares are; they are
    // noticed (returned) and the factorisation is done again with that factor in two, which costs 3 % where it always is.
    auto factor = [&](auto large) -> bool {
        constexpr bool LARGE = decltype(large)::value;
        bool met = false;
#pragma unroll
        for (int k = 0; k < NG; ++k)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int i = 4 * (k * QS + h) + e;
                xc[4 * k + e] = (i < n && col < n) ? Zp[(long)i * ldz + col] : 0.f;
                xq[4 * k + e] = (i == item) ? 1.f : 0.f;
            }
        if (tid < HN) { cbuf[0][tid] = 0.f; cbuf[1][tid] = 0.f; }   // what lies beyond the carried blocks reads as zero
        __syncthreads();
        if (col == 0) publish_from<0, NG>(cbuf[0], xc, h, 0);
        __syncthreads();
        for (int j = 0; j < n; ++j) {           // (rows and columns from n on are zero and stay zero)
            const float* cb = cbuf[j & 1];
            // column norm below the pivot: DPP inside the rows of 16 lanes, then the four row sums through scalar registers
            const float a0 = cb[lane], a1 = cb[lane + 64];
            const float alpha = cb[j];
            float sr_ = (lane > j ? a0 * a0 : 0.f) + (lane + 64 > j ? a1 * a1 : 0.f);
            sr_ += lane_xor<1>(sr_);
            sr_ += lane_xor<2>(sr_);
            sr_ += lane_xor<4>(sr_);
            sr_ += lane_xor<8>(sr_);
            const float s = (lane_value(sr_, 0) + lane_value(sr_, 16)) + (lane_value(sr_, 32) + lane_value(sr_, 48));
            float beta = alpha;   // nothing below the pivot: H = I
            if (s != 0.f) {
                // hardware square root (1 ulp): beta only decides how exactly the column is annihilated; 2 / u . u is formed
                // from the u that is applied, so that H is orthogonal whatever the rounding of beta
                const float nrm = __builtin_amdgcn_sqrtf(alpha * alpha + s);
                beta = alpha >= 0.f ? -nrm : nrm;
                const float uj = alpha - beta;
                const float uu = fmaf(uj, uj, s);
                float gamma = 2.f * __builtin_amdgcn_rcpf(uu), g2 = 1.f;
                if (LARGE) {    // from u at a norm of 1 to 2
                    const int ex = __builtin_amdgcn_frexp_expf(nrm);
                    const float us = ldexpf(uj, -ex);
                    gamma = ldexpf(2.f * __builtin_amdgcn_rcpf(fmaf(us, us, ldexpf(s, -2 * ex))), -ex);
                    g2 = ldexpf(1.f, -ex);
                }
                met = met || !(uu < 0x1p125f);
#define DQ_CALL(JB) reflect_from<JB, NG, LARGE>(cb, xc, xq, col > j, h, j, uj, gamma, g2)
                DQ_BLOCK_SWITCH(j / QB, DQ_CALL)
#undef DQ_CALL
            }
            if (col == j) mydiag = beta;
            if (tid == 0) sgn[j] = beta >= 0.f ? 1.f : -1.f;
            if (col == j + 1) {
                float* nb = cbuf[(j + 1) & 1];
#define DQ_CALL(JB) publish_from<JB, NG>(nb, xc, h, j + 1)
                DQ_BLOCK_SWITCH((j + 1) / QB, DQ_CALL)
#undef DQ_CALL
            }
            __syncthreads();
        }
        return met;
    };
    if (factor(std::false_type{})) factor(std::true_type{});    // (the same for every thread: all see the same columns)
    if (h == 0 && col < n) {
        if (!(fabsf(mydiag) <= 3.0e38f)) atomicOr(flags, DQ_FLAG_NONFINITE);
        else if (mydiag == 0.f) atomicOr(flags, DQ_FLAG_SINGULAR);
    }
    if (U != nullptr) {   // U[i][c] = s_i A[i][c] above the diagonal, |diag| on it
        float* Up = U + (long)blockIdx.x * su;
#pragma unroll
        for (int k = 0; k < NG; ++k)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int i = 4 * (k * QS + h) + e;
                if (i < n && col < n) Up[(long)i * ldu + col] = i < col ? sgn[i] * xc[4 * k + e] : (i == col ? fabsf(mydiag) : 0.f);
            }
    }
    {                     // R[r][c] = s_c Q[r][c]
        float* Rp = R + (long)blockIdx.x * sr + (long)item * ldr;
#pragma unroll
        for (int k = 0; k < NG; ++k) {
            const int c = 4 * (k * QS + h);
            const float4 sg = *reinterpret_cast<const float4*>(sgn + c);
            const float4 v = make_float4(xq[4 * k] * sg.x, xq[4 * k + 1] * sg.y, xq[4 * k + 2] * sg.z, xq[4 * k + 3] * sg.w);
            if (item < n && c + 3 < n) {
                *reinterpret_cast<float4*>(Rp + c) = v;
            } else if (item < n) {
                if (c < n) Rp[c] = v.x;
                if (c + 1 < n) Rp[c + 1] = v.y;
                if (c + 2 < n) Rp[c + 2] = v.z;
            }
        }
    }
}
#undef DQ_BLOCK_SWITCH

// ------------------------------------------------------------------------------------------------ S3 + S4 + S5
// JB = number of 32-column blocks of the rotation (n <= 32 JB): a workgroup has JB wavefronts, wavefront w forms the columns
// [32 w, 32 w + 32) of Y and the same rows of G.  A narrower rotation thus costs its own share of the matrix-core work and
// of the registers instead of the 128-wide one's.
constexpr int TT = 64;            // tokens per tile
constexpr int DLD = TT + 8;       // halfwords per LDS row of the transposed dY tile (144 bytes)
template <int JB> constexpr int xld() { return 32 * JB + 8; }   // halfwords per LDS row of an X tile (16-byte rows, 4-bank skew)

struct XRegs { uint4 q0, q1, q2, q3; };

// A thread's share of a tile: columns [col, col + 8) of the rows row0 + 16 i.  n no multiple of 32 (not EXACT): what lies beyond
// column n is masked on the way to LDS, where the loads have arrived anyway (a test or a mask at the load waits for it there and
// then: n = 100 on 16384 tokens 134 us).  A piece that the last column cuts short is read whole, its row goes on for ldx
// elements, a multiple of 8; only that of the last row, which may end where the buffer ends, is read element by element.
template <int JB, bool EXACT>
struct XPiece {
    int col, row0;
    bool cut;
    uint4 mask;
    __device__ __forceinline__ XPiece(int n, int tid) {
        col = tid % (4 * JB) * 8;
        row0 = tid / (4 * JB);
        cut = !EXACT && col < n && col + 8 > n;
        auto m = [&](int c) { return (EXACT || c < n ? 0xffffu : 0u) | (EXACT || c + 1 < n ? 0xffff0000u : 0u); };
        mask = make_uint4(m(col), m(col + 2), m(col + 4), m(col + 6));
        if (!EXACT && col >= n) col = 0;    // (masked)
    }
};

__device__ __forceinline__ uint4 load_cut(const bf16_t* p, int count) {
    uint32_t w[4] = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int e = 0; e < 8; ++e)
        if (e < count) w[e >> 1] |= (uint32_t)p[e] << (16 * (e & 1));
    return make_uint4(w[0], w[1], w[2], w[3]);
}

// tile rows [t0, t0 + 64) of X (tokens >= tend read as zero): 4 JB threads per row, 16 bytes each; T: its rows
template <int JB, bool EXACT>
__device__ __forceinline__ XRegs fetch_x(const bf16_t* __restrict__ Xp, long ldx, int t0, int tend, int T, int n,
                                         const XPiece<JB, EXACT>& x) {
    const int row = t0 + x.row0;
    const bf16_t* p = Xp + (long)row * ldx + x.col;
    const int last = x.cut ? T - 1 : T;     // first row that is not read whole
    const int end = tend < last ? tend : last;
    XRegs r;
    r.q0 = r.q1 = r.q2 = r.q3 = make_uint4(0u, 0u, 0u, 0u);
    if (row < end) r.q0 = *reinterpret_cast<const uint4*>(p);
    if (row + 16 < end) r.q1 = *reinterpret_cast<const uint4*>(p + 16 * ldx);
    if (row + 32 < end) r.q2 = *reinterpret_cast<const uint4*>(p + 32 * ldx);
    if (row + 48 < end) r.q3 = *reinterpret_cast<const uint4*>(p + 48 * ldx);
    if (!EXACT && t0 <= T - 1 && T - 1 < t0 + TT && T == tend) {    // (uniform) the tile holds the last row
        if (x.cut && row == T - 1) r.q0 = load_cut(p, n - x.col);
        if (x.cut && row + 16 == T - 1) r.q1 = load_cut(p + 16 * ldx, n - x.col);
        if (x.cut && row + 32 == T - 1) r.q2 = load_cut(p + 32 * ldx, n - x.col);
        if (x.cut && row + 48 == T - 1) r.q3 = load_cut(p + 48 * ldx, n - x.col);
    }
    return r;
}
template <int JB, bool EXACT>
__device__ __forceinline__ void stash_x(bf16_t* Xs, int tid, XRegs r, const XPiece<JB, EXACT>& x) {
    constexpr int XLD = xld<JB>();
    bf16_t* p = Xs + (tid / (4 * JB)) * XLD + (tid % (4 * JB)) * 8;
    auto masked = [&](uint4 q) {
        return EXACT ? q : make_uint4(q.x & x.mask.x, q.y & x.mask.y, q.z & x.mask.z, q.w & x.mask.w);
    };
    *reinterpret_cast<uint4*>(p) = masked(r.q0);
    *reinterpret_cast<uint4*>(p + 16 * XLD) = masked(r.q1);
    *reinterpret_cast<uint4*>(p + 32 * XLD) = masked(r.q2);
    *reinterpret_cast<uint4*>(p + 48 * XLD) = masked(r.q3);
}

// One 64-token tile.  Wavefront w forms Y[:, 32w .. 32w+32) (two 32 x 32 accumulators), applies Eq. 4 and its
// derivative, leaves dY transposed in LDS; after the barrier it adds X_tile^T dY_tile to its 32 rows of G.
// Matrix-core operand layout (32x32x16 bf16): lane l supplies row/column (l & 31) and the 8 consecutive reduction
// indices 8 (l >> 5) ..; the 32 x 32 result holds row 8 (v >> 2) + 4 (l >> 5) + (v & 3), column (l & 31) in register v.
// EVEN: every tile holds 64 tokens; otherwise only the first `tokens` rows of the last one are tokens.
template <int JB, bool EVEN>
__device__ __forceinline__ void heads_tile(const bf16_t* Xs, bf16_t* dYs, const bf16x8 (&rhi)[2 * JB],
                                           const bf16x8 (&rlo)[2 * JB], f32x16 (&accG)[JB], double& loss, float scale,
                                           int tokens, int wave, int lrow, int lk) {
    constexpr int XLD = xld<JB>();
    f32x16 y0, y1;
#pragma unroll
    for (int v = 0; v < 16; ++v) { y0[v] = 0.f; y1[v] = 0.f; }
#pragma unroll
    for (int ks = 0; ks < 2 * JB; ++ks) {
        const bf16x8 a0 = *reinterpret_cast<const bf16x8*>(Xs + lrow * XLD + ks * 16 + lk * 8);
        const bf16x8 a1 = *reinterpret_cast<const bf16x8*>(Xs + (32 + lrow) * XLD + ks * 16 + lk * 8);
        y0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a0, rhi[ks], y0, 0, 0, 0);
        y1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1, rhi[ks], y1, 0, 0, 0);
        y0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a0, rlo[ks], y0, 0, 0, 0);
        y1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1, rlo[ks], y1, 0, 0, 0);
    }
    if (!EVEN && tokens < TT) {   // the rows behind the last token: exp(-1e30) = 0 adds nothing to the loss nor to dY
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int tok = 8 * (v >> 2) + 4 * lk + (v & 3);
            y0[v] = tok < tokens ? y0[v] : 1e30f;
            y1[v] = 32 + tok < tokens ? y1[v] : 1e30f;
        }
    }
    const int j = 32 * wave + lrow;
    float sum[4] = {0.f, 0.f, 0.f, 0.f};   // eight terms each, then to 64 bits
#pragma unroll
    for (int i = 0; i < 2; ++i) {
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const int tok0 = i * 32 + 8 * g + 4 * lk;
            float d[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float y = i == 0 ? y0[4 * g + q] : y1[4 * g + q];
                const float ex = __expf(-fabsf(y));
                sum[q] += ex;
                // scale * sgn(y) without comparisons: y * 2^150 has modulus 2 or more for every y but 0 (an overflow to
                // infinity is as good), so the median with -scale and +scale picks the signed bound; y = 0 stays 0
                const float sg = __builtin_amdgcn_fmed3f(ldexpf(y, 150), -scale, scale);
                d[q] = -sg * ex;
            }
            const f32x2 d01 = {d[0], d[1]}, d23 = {d[2], d[3]};
            const bf16x2 b01 = __builtin_convertvector(d01, bf16x2), b23 = __builtin_convertvector(d23, bf16x2);
            *reinterpret_cast<uint2*>(dYs + j * DLD + tok0) =
                make_uint2(__builtin_bit_cast(uint32_t, b01), __builtin_bit_cast(uint32_t, b23));
        }
    }
    loss += (double)((sum[0] + sum[1]) + (sum[2] + sum[3]));
    __syncthreads();
    const int ch = 32 * wave + lrow;   // this lane's row of G
#pragma unroll
    for (int kt = 0; kt < TT / 16; ++kt) {
        u32x4 au;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const uint32_t lo = Xs[(kt * 16 + lk * 8 + 2 * e) * XLD + ch];
            const uint32_t hi = Xs[(kt * 16 + lk * 8 + 2 * e + 1) * XLD + ch];
            au[e] = lo | (hi << 16);
        }
        const bf16x8 afr = __builtin_bit_cast(bf16x8, au);
#pragma unroll
        for (int jb = 0; jb < JB; ++jb) {
            const bf16x8 bfr = *reinterpret_cast<const bf16x8*>(dYs + (jb * 32 + lrow) * DLD + kt * 16 + lk * 8);
            accG[jb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(afr, bfr, accG[jb], 0, 0, 0);
        }
    }
}

// grid (splits, b): workgroup (s, p) handles tokens [s * chunk, min(T, (s+1) * chunk)) of problem p and writes its
// partial G to Gpart[(p * splits + s) * (32 JB)^2 ..] and its partial sum of exp(-|y|) to lpart[p * splits + s].
template <int JB, bool EXACT, bool EVEN>
__global__ __launch_bounds__(64 * JB, 2) void heads_rlg_kernel(const bf16_t* __restrict__ X, long ldx, long sx, int T, int n,
                                                        const float* __restrict__ R, long ldr, long sr, float scale,
                                                        float* __restrict__ Gpart, double* __restrict__ lpart,
                                                        int chunk) {
    constexpr int NP = 32 * JB;
    __shared__ __attribute__((aligned(16))) bf16_t Xs[2][TT * xld<JB>()];
    __shared__ __attribute__((aligned(16))) bf16_t dYs[NP * DLD];
    __shared__ double wsum[JB];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lrow = lane & 31, lk = lane >> 5;
    const int split = blockIdx.x, prob = blockIdx.y, splits = gridDim.x;
    const bf16_t* Xp = X + (long)prob * sx;
    const float* Rp = R + (long)prob * sr;
    const int tbeg = split * chunk;
    const int tend = (tbeg + chunk < T) ? tbeg + chunk : T;
    const int ntiles = tend > tbeg ? (tend - tbeg + TT - 1) / TT : 0;

    // this wavefront's 32 columns of R as matrix-core operands: R = hi + lo, 16 mantissa bits (zero beyond n x n)
    bf16x8 rhi[2 * JB], rlo[2 * JB];
    {
        const int j = 32 * wave + lrow;
#pragma unroll
        for (int ks = 0; ks < 2 * JB; ++ks) {
            u32x4 hi, lo;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int k = ks * 16 + lk * 8 + 2 * e;
                const float r0 = (EXACT || (k < n && j < n)) ? Rp[(long)k * ldr + j] : 0.f;
                const float r1 = (EXACT || (k + 1 < n && j < n)) ? Rp[(long)(k + 1) * ldr + j] : 0.f;
                const uint32_t h0 = to_bf16_rne(r0), h1 = to_bf16_rne(r1);
                const uint32_t l0 = to_bf16_rne(r0 - __uint_as_float(h0 << 16));
                const uint32_t l1 = to_bf16_rne(r1 - __uint_as_float(h1 << 16));
                hi[e] = h0 | (h1 << 16);
                lo[e] = l0 | (l1 << 16);
            }
            rhi[ks] = __builtin_bit_cast(bf16x8, hi);
            rlo[ks] = __builtin_bit_cast(bf16x8, lo);
        }
    }

    f32x16 accG[JB];
#pragma unroll
    for (int jb = 0; jb < JB; ++jb)
#pragma unroll
        for (int v = 0; v < 16; ++v) accG[jb][v] = 0.f;
    double lsum = 0.0;

    const XPiece<JB, EXACT> piece(n, tid);
    XRegs p0 = fetch_x<JB, EXACT>(Xp, ldx, tbeg, tend, T, n, piece);
    XRegs p1 = fetch_x<JB, EXACT>(Xp, ldx, tbeg + TT, tend, T, n, piece);
    stash_x<JB, EXACT>(Xs[0], tid, p0, piece);
    __syncthreads();
    for (int it = 0; it < ntiles; it += 2) {
        // tile `it` is in Xs[0], tile it+1 in p1; tile it+2 is requested into p0
        p0 = fetch_x<JB, EXACT>(Xp, ldx, tbeg + (it + 2) * TT, tend, T, n, piece);
        heads_tile<JB, EVEN>(Xs[0], dYs, rhi, rlo, accG, lsum, scale, tend - (tbeg + it * TT), wave, lrow, lk);
        stash_x<JB, EXACT>(Xs[1], tid, p1, piece);
        __syncthreads();
        if (it + 1 < ntiles) {
            p1 = fetch_x<JB, EXACT>(Xp, ldx, tbeg + (it + 3) * TT, tend, T, n, piece);
            heads_tile<JB, EVEN>(Xs[1], dYs, rhi, rlo, accG, lsum, scale, tend - (tbeg + (it + 1) * TT), wave, lrow, lk);
        }
        stash_x<JB, EXACT>(Xs[0], tid, p0, piece);
        __syncthreads();
    }

    float* Gp = Gpart + ((long)prob * splits + split) * (NP * NP);
#pragma unroll
    for (int jb = 0; jb < JB; ++jb)
#pragma unroll
        for (int v = 0; v < 16; ++v)
            Gp[(32 * wave + 8 * (v >> 2) + 4 * lk + (v & 3)) * NP + jb * 32 + lrow] = accG[jb][v];
    // columns from n on hold y = 0 throughout: they count nothing
    lsum = wave_total(EXACT || 32 * wave + lrow < n ? lsum : 0.0);
    if (lane == 0) wsum[wave] = lsum;
    __syncthreads();
    if (tid == 0) {
        double t = 0.0;
#pragma unroll
        for (int w = 0; w < JB; ++w) t += wsum[w];
        lpart[(long)prob * splits + split] = t;
    }
}

// grid (NP^2 / 1024, b): G[p] = sum_s Gpart[p][s] (partials NP x NP, NP = 32 ceil(n / 32));  loss[p] = scale * sum_s lpart[p][s]
__global__ __launch_bounds__(256) void heads_reduce_kernel(const float* __restrict__ Gpart, const double* __restrict__ lpart,
                                                           int splits, float scale, int n, int np, float* __restrict__ G,
                                                           long ldg, long sg, float* __restrict__ loss, unsigned* flags) {
    const int prob = blockIdx.y;
    const int e = (blockIdx.x * 256 + threadIdx.x) * 4;
    const float* src = Gpart + (long)prob * splits * (np * np) + e;
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int s0 = 0; s0 < splits; s0 += 8) {     // eight loads in flight
        float4 v[8];
#pragma unroll
        for (int k = 0; k < 8; ++k)
            v[k] = s0 + k < splits ? *reinterpret_cast<const float4*>(src + (long)(s0 + k) * (np * np)) : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int k = 0; k < 8; ++k) { acc.x += v[k].x; acc.y += v[k].y; acc.z += v[k].z; acc.w += v[k].w; }
    }
    const int r = e / np, c = e % np;
    float* o = G + (long)prob * sg + (long)r * ldg + c;
    if (r < n && c + 3 < n) {
        *reinterpret_cast<float4*>(o) = acc;
    } else if (r < n) {
        if (c < n) o[0] = acc.x;
        if (c + 1 < n) o[1] = acc.y;
        if (c + 2 < n) o[2] = acc.z;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        double t = 0.0;
        for (int s = 0; s < splits; ++s) t += lpart[(long)prob * splits + s];
        const float Lf = (float)((double)scale * t);
        loss[prob] = Lf;
        if (!(fabsf(Lf) <= 3.0e38f)) atomicOr(flags, DQ_FLAG_NONFINITE);
    }
}

// ------------------------------------------------------------------------------------------------ S6 (+ S7)
// The derivative through the QR of one problem per workgroup, out = alpha R M + beta out with
//   B = R^T G,  P = strict_lower(B - B^T),  M U^T = P
// (alpha = 1, beta = 0: dZ;  alpha = -lr, beta = 1: the updated latent).  Everything between R, G, U and the result stays in
// LDS.  64 problems of order 128: 38 us, 32 of order 80: 25 us.  Before: the inverse of U in a launch beside the gradient's,
// which held its compute units' registers (24 us alone, done 20 us after it at 64 x 128), and four batched launches, 31 us,
// nearly all of it launches, gaps and trips through memory.
// Bound: the fp32 matrix instructions of ONE compute unit (B 7 us at order 128, the triangular product, which skips its zero
// blocks, 5 us) and the chain of the solve (four blocks of 32 columns from the right, about 1 us each).  16 wavefronts, one
// 32 x 32 block each, dealt out so that every SIMD gets one of each block column (they differ in length).  LDS rows of 129
// floats: a matrix is an operand along its rows and along its columns without bank conflicts.  P and M are held transposed.
// Rows and columns from n on are zero (of U: the identity).
constexpr int HBL = HN + 1, HIL = 33;

__global__ __launch_bounds__(1024) void heads_backward_kernel(const float* R, long ldr, long sr, const float* G, long ldg,
                                                              long sg, const float* U, long ldu, long su, int n, float alpha,
                                                              float beta, float* out, long ldo, long so, unsigned* flags) {
    __shared__ float Rs[HN * HBL];
    __shared__ float Bs[HN * HBL];
    __shared__ float Xs[4 * 32 * HIL];      // inverses of the 32 x 32 diagonal blocks of U
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lrow = lane & 31, lk = lane >> 5;
    const int wi = wave >> 2, wj = (wave + wi) & 3;
    R += (long)blockIdx.x * sr;
    G += (long)blockIdx.x * sg;
    U += (long)blockIdx.x * su;
    out += (long)blockIdx.x * so;
    const int nb = (n + 31) >> 5;           // blocks of 32 that hold anything
    {
        float r[16], g[16], u[4];
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            const int e = tid + 1024 * q, i = e >> 7, c = e & 127;
            const bool in = i < n && c < n;
            r[q] = in ? R[(long)i * ldr + c] : 0.f;
            g[q] = in ? G[(long)i * ldg + c] : 0.f;
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {       // diagonal block q of U, entry (tid / 32, tid % 32)
            const int i = 32 * q + (tid >> 5), c = 32 * q + (tid & 31);
            u[q] = (i < n && c < n) ? U[(long)i * ldu + c] : (i == c ? 1.f : 0.f);
            if (i == c && u[q] == 0.f) atomicOr(flags, DQ_FLAG_SINGULAR);
        }
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            const int e = tid + 1024 * q, i = e >> 7, c = e & 127;
            Rs[i * HBL + c] = r[q];
            Bs[i * HBL + c] = g[q];
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) Xs[(32 * q + (tid >> 5)) * HIL + (tid & 31)] = u[q];
    }
    const bool live = wi < nb && wj < nb;
    const int r0 = 32 * wi + 4 * lk, cc = 32 * wj + lrow;   // accumulator v: row r0 + 8 (v / 4) + v % 4, column cc
    f32x16 acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0.f;
    __syncthreads();
    if (wave < nb) {
        // one wavefront per diagonal block: lane c solves U x = e_c from the last row up (the upper lanes repeat the lower ones)
        float* X = Xs + 32 * wave * HIL;
        float x[32];
#pragma unroll
        for (int i = 31; i >= 0; --i) {
            float t0 = i == lrow ? 1.f : 0.f, t1 = 0.f;
#pragma unroll
            for (int k = i + 1; k < 32; ++k) {
                if (k & 1) t1 -= X[i * HIL + k] * x[k];
                else t0 -= X[i * HIL + k] * x[k];
            }
            x[i] = (t0 + t1) / X[i * HIL + i];
        }
#pragma unroll
        for (int i = 0; i < 32; ++i) X[i * HIL + lrow] = x[i];   // (zero below the diagonal by itself)
    }
    if (live) {                         // B = R^T G
        for (int k0 = 0; k0 < 32 * nb; k0 += 32)
#pragma unroll
            for (int k = k0; k < k0 + 32; k += 2)
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(Rs[(k + lk) * HBL + 32 * wi + lrow], Bs[(k + lk) * HBL + cc], acc, 0, 0, 0);
    }
    __syncthreads();
#pragma unroll
    for (int v = 0; v < 16; ++v) Bs[(r0 + 8 * (v >> 2) + (v & 3)) * HBL + cc] = acc[v];
    __syncthreads();
    // P^T (k, i) = B(i, k) - B(k, i) for i > k, zero elsewhere
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const int k = r0 + 8 * (v >> 2) + (v & 3);
        acc[v] = cc > k ? Bs[cc * HBL + k] - acc[v] : 0.f;
    }
    __syncthreads();
#pragma unroll
    for (int v = 0; v < 16; ++v) Bs[(r0 + 8 * (v >> 2) + (v & 3)) * HBL + cc] = acc[v];
    // M by block columns J from the right (block rows of M^T):  M^T_J = inv(U_JJ) P^T_J,  P^T_K -= U_KJ M^T_J for K < J; both
    // only for the rows i >= 32 J of M, the columns right of there in M^T
    for (int J = nb - 1; J >= 0; --J) {
        const int cols = nb - J;            // blocks of i
        const int K = wave / cols, ib = J + wave % cols;
        const bool upd = K < J;
        // the block U_KJ of this wavefront's update: row 32 K + lrow, k = 8 q + 4 lk + 0 .. 3 in step q
        float u[16];
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int c = 32 * J + 8 * q + 4 * lk + e;
                u[4 * q + e] = (upd && c < n) ? U[(long)(32 * K + lrow) * ldu + c] : 0.f;
            }
        __syncthreads();
        if (wave < cols) {
            const int i0 = 32 * (J + wave) + lrow;
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[v] = 0.f;
#pragma unroll
            for (int k = 0; k < 32; k += 2)
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(Xs[(32 * J + lrow) * HIL + k + lk], Bs[(32 * J + k + lk) * HBL + i0], acc, 0, 0, 0);
#pragma unroll
            for (int v = 0; v < 16; ++v) Bs[(32 * J + 8 * (v >> 2) + 4 * lk + (v & 3)) * HBL + i0] = acc[v];   // own columns only
        }
        __syncthreads();
        if (upd) {
            const int i0 = 32 * ib + lrow;
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[v] = 0.f;
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(u[4 * q + e], Bs[(32 * J + 8 * q + 4 * lk + e) * HBL + i0], acc, 0, 0, 0);
#pragma unroll
            for (int v = 0; v < 16; ++v) Bs[(32 * K + 8 * (v >> 2) + 4 * lk + (v & 3)) * HBL + i0] -= acc[v];
        }
    }
    __syncthreads();
    if (!live) return;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0.f;
    for (int k0 = 32 * wj; k0 < 32 * nb; k0 += 32)      // R M; M is strictly lower triangular
#pragma unroll
        for (int k = k0; k < k0 + 32; k += 2)
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(Rs[(32 * wi + lrow) * HBL + k + lk], Bs[cc * HBL + k + lk], acc, 0, 0, 0);
    if (cc >= n) return;
    float* o = out + (long)r0 * ldo + cc;
    float old[16];
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const int r = 8 * (v >> 2) + (v & 3);
        old[v] = (beta != 0.f && r0 + r < n) ? o[(long)r * ldo] : 0.f;
    }
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const int r = 8 * (v >> 2) + (v & 3);
        if (r0 + r < n) o[(long)r * ldo] = beta != 0.f ? alpha * acc[v] + beta * old[v] : alpha * acc[v];
    }
}

}  // namespace

hipError_t launch_heads_qr(int b, int n, const float* Z, long ldz, long sz, float* R, long ldr, long sr, float* U, long ldu,
                           long su, unsigned* flags, hipStream_t s) {
    if (b < 1) return hipSuccess;
    if (n < 1 || n > HN) return hipErrorInvalidValue;
#define DQ_LAUNCH(FULL, NG)                                                                                              \
    hipLaunchKernelGGL((heads_qr_kernel<FULL, NG>), dim3(b), dim3(HN * QS), 0, s, Z, ldz, sz, R, ldr, sr, U, ldu, su, n, flags)
    if (n == HN) DQ_LAUNCH(true, 8);
    else if (n > 96) DQ_LAUNCH(false, 8);
    else if (n > 64) DQ_LAUNCH(false, 6);
    else DQ_LAUNCH(false, 4);
#undef DQ_LAUNCH
    return hipGetLastError();
}

hipError_t launch_heads_backward(int b, int n, const float* R, long ldr, long sr, const float* G, long ldg, long sg,
                                 const float* U, long ldu, long su, float alpha, float beta, float* out, long ldo, long so,
                                 unsigned* flags, hipStream_t s) {
    if (b < 1) return hipSuccess;
    if (n < 1 || n > HN) return hipErrorInvalidValue;
    hipLaunchKernelGGL(heads_backward_kernel, dim3(b), dim3(1024), 0, s, R, ldr, sr, G, ldg, sg, U, ldu, su, n, alpha, beta,
                       out, ldo, so, flags);
    return hipGetLastError();
}

// Tokens per workgroup.  It depends on T and n alone, so that a batch and its problems one by one sum in the same order; the
// partial gradient a workgroup leaves costs as much as 64 tokens of X, and few blocks in long parts leave the chip idle (one of
// 16384 tokens in eight: the general route's tiles take 47 us for it at n = 80).
//   n = 128, 96: about eight parts, 256 to 2048 tokens each: 64 blocks of 16384 tokens make 512 workgroups, two per compute unit.
//   Others above 64: the same up to 12288 tokens, from there sixteen parts of 1024 at most, us for 1 / 32 / 64 blocks of 16384 tokens in
//   eight and in sixteen: n = 80 74 / 83 / 99 and 45 / 63 / 117, n = 112 86 / 99 / 129 and 53 / 82 / 166 (element by element loads,
//   eight parts: 87 / 113 / 125, 109 / 136 / 176).  At n = 96 64 blocks would lose too much, 91 -> 109.
//   Up to 64, whose partials are small, sixteen parts, no shorter than 256 tokens above 32 (n = 64, 512 tokens, 1000 blocks: 270 us
//   a step, in parts of 128 294) and than 128 below: 1 / 32 / 64 blocks as above n = 64 61 / 67 / 79 -> 36 / 49 / 55, n = 16 57 / 70 / 76
//   -> 26 / 28 / 29.
static int heads_chunk(int T, int n) {
    const bool even = n % 32 == 0;
    const int parts = n > 64 && (even || T <= 12288) ? 8 : 16;
    const int lo = n > 64 ? 256 : (n > 32 ? 256 : 128), hi = n > 64 && even ? kHeadsChunk : (parts == 8 ? 1536 : 1024);
    const int c = (int)round_up((T + parts - 1) / parts, TT);
    return c < lo ? lo : (c < hi ? c : hi);
}
int heads_splits(int T, int n) { const int c = heads_chunk(T, n); return (T + c - 1) / c; }

hipError_t launch_heads_rlg(int b, int n, int T, const bf16_t* X, long ldx, long sx, const float* R, long ldr, long sr,
                            float scale, float* Gpart, double* lpart, float* G, long ldg, long sg, float* loss,
                            unsigned* flags, hipStream_t s) {
    if (b < 1) return hipSuccess;
    if (n < 1 || n > HN) return hipErrorInvalidValue;
    const int splits = heads_splits(T, n), chunk = heads_chunk(T, n), jb = (n + 31) / 32;
    const dim3 grid(splits, b), block(64 * jb);
#define DQ_RLG1(JB, EXACT, EVEN)                                                                                             \
    hipLaunchKernelGGL((heads_rlg_kernel<JB, EXACT, EVEN>), grid, block, 0, s, X, ldx, sx, T, n, R, ldr, sr, scale, Gpart, lpart, chunk)
#define DQ_RLG(JB)                                                                                                            \
    if (n == 32 * JB && T % TT == 0) DQ_RLG1(JB, true, true);                                                                 \
    else if (n == 32 * JB) DQ_RLG1(JB, true, false);                                                                          \
    else DQ_RLG1(JB, false, false)
    switch (jb) {
        case 1: DQ_RLG(1); break;
        case 2: DQ_RLG(2); break;
        case 3: DQ_RLG(3); break;
        default: DQ_RLG(4); break;
    }
#undef DQ_RLG
#undef DQ_RLG1
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(heads_reduce_kernel, dim3(jb * jb, b), dim3(256), 0, s, Gpart, lpart, splits, scale, n, 32 * jb, G, ldg,
                       sg, loss, flags);
    return hipGetLastError();
}

}  // namespace dq
