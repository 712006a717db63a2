// Batched path for small rotations, n <= 128 (per-head rotations; the "heads" workload has 64 of size 128): every problem
// of a batch runs in the same launch.
//   * heads_qr_kernel: R, U = qr(Z) for one latent per workgroup, entirely on chip: Cholesky of the Gram matrix in fp64, once or
//     twice, or column by column.
//   * heads_rlg_kernel: Alg. 1, rotation and loss steps, fused for bf16 activations.  A workgroup streams 64-token tiles of X once;
//     Y = X R (R as two bf16 planes held in registers), the Whip loss and its gradient (Eq. 4) and the tile's
//     contribution to G = X^T dY are formed on chip: Y and dY never reach HBM.
//   * heads_reduce_kernel: sums the per-workgroup partial G and loss.
//   * heads_backward_kernel: the derivative through the QR and the update, one problem per workgroup, out of LDS.
#include "dq_chol16.h"
#include "dq_internal.h"
#include "dq_wave.h"


namespace dq {
namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

constexpr int HN = kHeadDim;     // largest matrix size of this path
#define MFMA16(a, b, c) __builtin_amdgcn_mfma_f32_16x16x4f32((a), (b), (c), 0, 0, 0)

__device__ __forceinline__ double wave_total(double v) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

__device__ __forceinline__ uint32_t to_bf16_rne(float f) {
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (u >> 16) | 0x40u;   // NaN stays NaN
    u += 0x7fffu + ((u >> 16) & 1u);
    return u >> 16;
}

// ------------------------------------------------------------------------------------------------ S1 + S2
// R, U of one latent per workgroup, in LDS and registers: G = A^T A, G = U^T U and Q^T = U^-T A^T in fp64 on the matrix cores, which
// leaves Q^T Q = I + E at 1e-16 times the square of the condition number.  Q once more where that is not yet the identity: by the factor
// I + X with X the upper half of E where its square is rounding; by another factorisation where it is not; and Z column by column
// (householder_columns) where its Gram matrix has no factor: condition numbers from 1e8 on, columns that vanish or are spanned.
// Wavefront 0 factors the 16 x 16 diagonal tiles, the other seven hold the tiles of G's upper triangle (see chol64_kernel, which has
// more of them).  Q's rows are independent of each other, 16 to a wavefront: their transposes take the factorisation's steps as more columns
// of G would.  (In fp32 Q cost 6 us, and E, from condition numbers of 100 on, a correction and one more look, 10 to 45 us.)
// Us: U above the diagonal, below it X^T, its diagonal in dinv.
// Bound: one compute unit's fp64 matrix cores and the chain of its diagonal tiles.  Every latent column by column (1 us a column: a
// chain of barrier, norm, dot product and update) and now: 64 latents of order 128 127 / 65 us, 512 of them 269 / 134, 64 of 112 117 / 50,
// 64 of 96 89 / 38, 32 of 80 77 / 29, 64 of 64 51 / 20.  Of the 65 us: G 19, the factor 23 (eight diagonal tiles), Q about 10, E 11.
// One latent of a batch that is factored twice: 140 us at order 128; one that is taken column by column: 198.
constexpr int HW = 7;            // wavefronts that hold tiles
constexpr double kHeadsDone = 4e-14;      // |R^T R - I|_F^2 / n with which R is finished: 2e-7 (column by column it was 3.3 to 4.1e-7)
// |R^T R - I|_F^2 up to which Q (I - X), (I + X) U is taken: their product lacks X^2 U, at most 1.5e-7 of a column of Z here.
constexpr double kHeadsNear = 3e-7;

// |R^T R - I|_F^2 from which Z is taken column by column: below, no eigenvalue of R^T R is under 0.29, and another factorisation ends it.
constexpr double kHeadsFar = 0.5;

template <int NT>
struct HeadsQr {
    static constexpr int N = 16 * NT, LD = N + 4, TILES = NT * (NT + 1) / 2, SLOTS = (TILES + HW - 1) / HW, NB = (NT + 3) / 4;
    // U's tiles above the diagonal, the diagonal ones' inverses and the exchange buffers lie where Q is before and after
    static constexpr int ROW = 0, WINV = ROW + NT * (NT - 1) / 2 * 256, NEXT = WINV + NT * 16 * CLD, DIAG = NEXT + 512,
                         COPY = DIAG + 512, USED = COPY + 16 * CLD;
    static constexpr int COLUMNS = N * LD;       // floats: householder_columns has its scratch behind Q
    static constexpr int POOL = USED > (COLUMNS + 4 * HN) / 2 ? USED : (COLUMNS + 4 * HN) / 2;
};

// Alg. 2 with the unnormalised reflector vector, R and U of any finite Z: for column j, x = A[j:, j], beta = -sign(x_0) ||x||,
// u = x - beta e_0, H = I - gamma u u^T with gamma = 2 / u^T u  (the same reflection as the paper's normalised v);
// a column that is already zero below the diagonal gets H = I.  Columns are taken at a length of 1 to 2, by the power of two
// in norm2 (squared lengths of Z's), and U's get it back.
// 512 threads: four adjacent lanes ("item" i = tid / 4, part h = tid % 4) hold one column of A AND one row of Q in
// registers, lane part h owning the 4-row groups g with g % 4 == h of both.  Both get x <- x - gamma (u . x) u (the
// column only if it lies right of j), with ONE read of u from LDS for the two, the partial dot products of the four
// lanes meeting through DPP.  Columns are dealt to the items round-robin over the wavefronts (item i holds column
// 8 (i % 16) + i / 16), so that every wavefront keeps live columns to the end.  The owners of column j + 1 publish it in
// LDS at the end of step j, so a step needs one barrier; every wavefront forms the column norm itself.  Rows are handled
// in blocks of 16: blocks above the diagonal block are skipped (the block index is a template parameter, so register
// indices are static and a step runs straight-line code), the diagonal block substitutes u_0 for the raw pivot and
// zero above it.
// Bound: the vector ALU and the chain of dependent operations of a step, half and half, 1 us a column.
constexpr int QS = 4;                   // lanes per column / row
constexpr int QB = 16;                  // rows per block = 4 groups, one per lane part

__device__ __forceinline__ float lane_value(float v, int l) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}

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
// of the pivot; u is the published column with u_0 = uj in place of the raw pivot
template <int JB, int NG>
__device__ __forceinline__ void reflect_from(const float* cb, float (&xc)[4 * NG], float (&xq)[4 * NG], bool col_live,
                                             int h, int j, float uj, float gamma) {
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
    const float fc = col_live ? gamma * dc : 0.f, fq = gamma * dq;
#pragma unroll
    for (int k = JB; k < NG; ++k) {
        const float4 v = u[k - JB];
        xc[4 * k] -= fc * v.x; xc[4 * k + 1] -= fc * v.y; xc[4 * k + 2] -= fc * v.z; xc[4 * k + 3] -= fc * v.w;
        xq[4 * k] -= fq * v.x; xq[4 * k + 1] -= fq * v.y; xq[4 * k + 2] -= fq * v.z; xq[4 * k + 3] -= fq * v.w;
    }
}

#define DQ_BLOCK_SWITCH(jb, CALL)                                                                  \
    switch (jb) {                                                                                  \
        case 0: CALL(0); break;                                                                    \
        case 1: CALL(1); break;                                                                    \
        case 2: CALL(2); break;                                                                    \
        case 3: CALL(3); break;                                                                    \
        case 4: if constexpr (NT > 4) { CALL(4); } break;                                          \
        case 5: if constexpr (NT > 5) { CALL(5); } break;                                          \
        case 6: if constexpr (NT > 6) { CALL(6); } break;                                          \
        case 7: if constexpr (NT > 7) { CALL(7); } break;                                          \
        default: break;                                                                            \
    }

// Q <- R, Us <- U (on and above the diagonal; row stride HeadsQr<NT>::LD both)
template <int NT>
__device__ __noinline__ void householder_columns(const float* __restrict__ Zp, long ldz, int n, const double* norm2, float* Q, float* Us,
                                                 unsigned* flags) {
    using H = HeadsQr<NT>;
    constexpr int LD = H::LD;
    static_assert(64 * (HW + 1) == HN * QS, "an item for every column");
    float *const cbuf0 = Q + H::COLUMNS, *const sgn = cbuf0 + 2 * HN;
    const int tid = threadIdx.x, lane = tid & 63, item = tid / QS, h = tid % QS;
    const int col = 8 * (item & 15) + (item >> 4);   // this thread's column of A; its row of Q is `item`
    const double len2 = col < n ? norm2[col] : 0.0;
    const int ex = len2 > 0.0 && len2 < 0x1p1000 ? __builtin_amdgcn_frexp_exp(len2) >> 1 : 0;
    float xc[4 * NT], xq[4 * NT], mydiag = 0.f;
#pragma unroll
    for (int k = 0; k < NT; ++k)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int i = 4 * (k * QS + h) + e;
            xc[4 * k + e] = (i < n && col < n) ? ldexpf(Zp[(long)i * ldz + col], -ex) : 0.f;
            xq[4 * k + e] = (i == item) ? 1.f : 0.f;
        }
    __syncthreads();
    if (tid < 2 * HN) cbuf0[tid] = 0.f;     // what lies beyond the carried blocks reads as zero
    __syncthreads();
    if (col == 0) publish_from<0, NT>(cbuf0, xc, h, 0);
    __syncthreads();
    for (int j = 0; j < n; ++j) {           // (rows and columns from n on are zero and stay zero)
        const float* cb = cbuf0 + (j & 1) * HN;
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
            const float uj = alpha - beta, gamma = 2.f * __builtin_amdgcn_rcpf(fmaf(uj, uj, s));
#define DQ_CALL(JB) reflect_from<JB, NT>(cb, xc, xq, col > j, h, j, uj, gamma)
            DQ_BLOCK_SWITCH(j / QB, DQ_CALL)
#undef DQ_CALL
        }
        if (col == j) mydiag = beta;
        if (tid == 0) sgn[j] = beta >= 0.f ? 1.f : -1.f;
        if (col == j + 1) {
            float* nb = cbuf0 + ((j + 1) & 1) * HN;
#define DQ_CALL(JB) publish_from<JB, NT>(nb, xc, h, j + 1)
            DQ_BLOCK_SWITCH((j + 1) / QB, DQ_CALL)
#undef DQ_CALL
        }
        __syncthreads();
    }
    if (h == 0 && col < n && mydiag == 0.f) atomicOr(flags, DQ_FLAG_SINGULAR);
    // U[i][c] = s_i A[i][c] above the diagonal, |diag| on it; R[r][c] = s_c Q[r][c]
#pragma unroll
    for (int k = 0; k < NT; ++k)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int i = 4 * (k * QS + h) + e;
            if (i <= col && col < n) Us[i * LD + col] = ldexpf(i < col ? sgn[i] * xc[4 * k + e] : fabsf(mydiag), ex);
            if (item < n && i < n) Q[item * LD + i] = xq[4 * k + e] * sgn[i];
        }
}
#undef DQ_BLOCK_SWITCH

// acc[t] (16 rows, columns 64 s + 16 t ..) += row[k] M[k][.] over k >= 64 first, M upper triangular with its transpose below Us's diagonal and
// its diagonal in dinv
template <int NT>
__device__ __forceinline__ void heads_times_upper(const float* row, const float* Us, const float* dinv, int first, int s, int c, int g,
                                                  f32x4 (&acc)[4]) {
    constexpr int LD = HeadsQr<NT>::LD;
#pragma unroll 1
    for (int kb = first; kb < s; ++kb)
#pragma unroll 4
        for (int q = 0; q < 16; ++q) {
            const int k = 64 * kb + 4 * q + g;
            const float a = row[k];
#pragma unroll
            for (int t = 0; t < 4; ++t)
                if (4 * s + t < NT) acc[t] = MFMA16(a, Us[(64 * s + 16 * t + c) * LD + k], acc[t]);
        }
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        const int k = 64 * s + 4 * q + g;
        if (4 * s + q / 4 >= NT) continue;
        const float a = row[k];
#pragma unroll
        for (int t = 0; t < 4; ++t)
            if (t >= q / 4 && 4 * s + t < NT) {
                float m = Us[(64 * s + 16 * t + c) * LD + k];
                if (t == q / 4) m = 4 * (q & 3) + g < c ? m : (4 * (q & 3) + g == c ? dinv[64 * s + 16 * t + c] : 0.f);
                acc[t] = MFMA16(a, m, acc[t]);
            }
    }
}

template <int NT>
__global__ __launch_bounds__(64 * (HW + 1)) void heads_qr_kernel(const float* __restrict__ Z, long ldz, long sz, float* R, long ldr,
                                                                 long sr, float* U, long ldu, long su, int n, unsigned* flags) {
    using H = HeadsQr<NT>;
    constexpr int N = H::N, LD = H::LD, SLOTS = H::SLOTS;
    __shared__ __attribute__((aligned(16))) double pool[H::POOL];
    __shared__ __attribute__((aligned(16))) float Us[N * LD];
    __shared__ float dinv[N];
    __shared__ double norm2[N];
    __shared__ double dev[HW + 1];
    __shared__ int rows_done;
    float* const Q = reinterpret_cast<float*>(pool);
    double *const winv = pool + H::WINV, *const nextbuf = pool + H::NEXT, *const diagbuf = pool + H::DIAG,
                  *const dcopy = pool + H::COPY;
    auto tile = [&](int k, int j) { return pool + H::ROW + (k * (2 * NT - k - 1) / 2 + j - k - 1) * 256; };   // (k, j) of U
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c0 = lane & 15, g0 = lane >> 4, w = wave - 1;
    const int nt = (n + 15) / 16;
    const float* Zp = Z + (long)blockIdx.x * sz;
    float* Rp = R + (long)blockIdx.x * sr;
    float* Up = U != nullptr ? U + (long)blockIdx.x * su : nullptr;
    auto load = [&](const float* p, long ld) {        // Q <- an n x n matrix, zeros past it
        for (int e = tid; e < N * N / 4; e += 64 * (HW + 1)) {
            const int r = e / (N / 4), q = e % (N / 4) * 4;
            float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
            if (r < n && q < n) v = load_quad(p + (long)r * ld + q, n - q);
            *reinterpret_cast<float4*>(Q + r * LD + q) = v;
        }
    };
    // tile HW s + w of the upper triangle, row by row, is slot s of the w-th of the seven; 256 i + j
    int tij[SLOTS];
#pragma unroll
    for (int s = 0; s < SLOTS; ++s) {
        int t = HW * s + w, i = 0;
        while (i < NT && t >= NT - i) { t -= NT - i; ++i; }
        tij[s] = __builtin_amdgcn_readfirstlane(wave > 0 && i < NT ? 256 * i + i + t : 255);
    }
    f64x4 acc[SLOTS];
    if (tid == 0) rows_done = 0;
    load(Zp, ldz);
    bool again = false;
    for (int step = 0, rows_base = 0;; ++step) {
        int c = c0, g = g0;
        asm volatile("" : "+v"(c), "+v"(g));    // addresses of all phases do not fit the registers across steps
        __syncthreads();
        if (step > 0) {
            // ---- E = Q^T Q - I, in fp32; the tiles dealt as G's
            f32x4 e[SLOTS];
            float part = 0.f;
#pragma unroll
            for (int s = 0; s < SLOTS; ++s) {
                const int t = opaque(tij[s]), ti = t >> 8, tj = t & 255;
                e[s] = f32x4{};
                if (tj < nt) {
                    const float *pa = Q + g * LD + 16 * ti + c, *pb = Q + g * LD + 16 * tj + c;
                    f32x4 odd = {};
#pragma unroll 8
                    for (int k = 0; k < 4 * nt; k += 2) {
                        e[s] = MFMA16(pa[4 * k * LD], pb[4 * k * LD], e[s]);
                        odd = MFMA16(pa[(4 * k + 4) * LD], pb[(4 * k + 4) * LD], odd);
                    }
                    e[s] += odd;
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        if (ti == tj && 4 * g + r == c) e[s][r] = 16 * tj + c < n ? e[s][r] - 1.f : 0.f;
                        part += (ti == tj ? 1.f : 2.f) * e[s][r] * e[s][r];
                    }
                }
            }
            const double mine = wave_total((double)part);
            if (lane == 0) dev[wave] = mine;
            __syncthreads();
            const double sum = ((dev[0] + dev[1]) + (dev[2] + dev[3])) + ((dev[4] + dev[5]) + (dev[6] + dev[7]));
            if (sum < kHeadsDone * n) break;
            if (sum < kHeadsNear) {
#pragma unroll
                for (int s = 0; s < SLOTS; ++s) {
                    const int t = opaque(tij[s]), ti = t >> 8, tj = t & 255;
                    if (tj < nt)
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            const int i = 16 * ti + 4 * g + r, j = 16 * tj + c;
                            if (i < j) Us[j * LD + i] = e[s][r];
                            if (i == j) dinv[i] = 0.5f * e[s][r];
                        }
                }
                if (tid < N && tid >= 16 * nt) dinv[tid] = 0.f;
                __syncthreads();
                if (wave < NT) {                            // Q -= Q X, from the last columns on: what is read is still the old one
                    float* own = Q + (16 * wave + 4 * g) * LD + c;
#pragma unroll
                    for (int b = H::NB - 1; b >= 0; --b) {
                        f32x4 v[4] = {};
                        heads_times_upper<NT>(Q + (16 * wave + c) * LD, Us, dinv, 0, b, c, g, v);
#pragma unroll
                        for (int t = 0; t < 4; ++t)
                            if (4 * b + t < NT)
#pragma unroll
                                for (int r = 0; r < 4; ++r) own[r * LD + 64 * b + 16 * t] -= v[t][r];
                    }
                }
                // U += X U, the tiles of the upper triangle dealt as G's
                f32x4 xu[SLOTS];
#pragma unroll
                for (int s = 0; s < SLOTS; ++s) {
                    const int t = opaque(tij[s]), ti = t >> 8, tj = t & 255;
                    xu[s] = f32x4{};
                    if (tj < nt) {
                        const float *px = Us + g * LD + 16 * ti + c, *pu = Us + g * LD + 16 * tj + c;
#pragma unroll
                        for (int q = 0; q < 4; ++q) {       // X's diagonal tile
                            const int k = 4 * q + g;
                            const float x = px[(16 * ti + 4 * q) * LD], u = pu[(16 * ti + 4 * q) * LD];
                            xu[s] = MFMA16(k > c ? x : (k == c ? dinv[16 * ti + c] : 0.f), ti < tj || k <= c ? u : 0.f, xu[s]);
                        }
#pragma unroll 1
                        for (int kk = ti + 1; kk < tj; ++kk)
#pragma unroll
                            for (int q = 0; q < 4; ++q) xu[s] = MFMA16(px[(16 * kk + 4 * q) * LD], pu[(16 * kk + 4 * q) * LD], xu[s]);
                        if (ti < tj)
#pragma unroll
                            for (int q = 0; q < 4; ++q) {   // U's
                                const float u = pu[(16 * tj + 4 * q) * LD];
                                xu[s] = MFMA16(px[(16 * tj + 4 * q) * LD], 4 * q + g <= c ? u : 0.f, xu[s]);
                            }
                    }
                }
                __syncthreads();
#pragma unroll
                for (int s = 0; s < SLOTS; ++s) {
                    const int t = opaque(tij[s]), ti = t >> 8, tj = t & 255;
                    if (tj < nt)
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            const int i = 16 * ti + 4 * g + r, j = 16 * tj + c;
                            if (i <= j) Us[i * LD + j] += xu[s][r];
                        }
                }
                break;
            }
            if (!(sum < kHeadsFar) || again) {     // (again: E was below kHeadsFar and so is one of rounding now; a NaN ends here)
                householder_columns<NT>(Zp, ldz, n, norm2, Q, Us, flags);
                break;
            }
            again = true;
            // Q waits in R, U in U
            if (wave < NT)
#pragma unroll 1
                for (int t = 0; t < NT; ++t)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int i = 16 * wave + 4 * g + r, j = 16 * t + c;
                        if (i < n && j < n) {
                            Rp[(long)i * ldr + j] = Q[i * LD + j];
                            if (Up != nullptr && i <= j) Up[(long)i * ldu + j] = Us[i * LD + j];
                        }
                    }
            __threadfence_block();
        }
        // ---- G = Q^T Q in fp64, the identity past the last column
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) {
            const int t = opaque(tij[s]), ti = t >> 8, tj = t & 255;
            acc[s] = f64x4{};
            if (tj < nt) {
                const float *pa = Q + g * LD + 16 * ti + c, *pb = Q + g * LD + 16 * tj + c;
#pragma unroll 8
                for (int k = 0; k < 4 * nt; ++k) acc[s] = MFMA64((double)pa[4 * k * LD], (double)pb[4 * k * LD], acc[s]);
                if (ti == tj)
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        if (4 * r + g == c && 16 * tj + c >= n) acc[s][r] = 1.0;
            }
        }
        // ---- U^T U = G
        __syncthreads();                       // Q has been read
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) {
            const int ti = tij[s] >> 8, tj = tij[s] & 255;
            if (tj >= nt) continue;
            if (ti == tj)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (4 * r + g == c) norm2[16 * ti + c] = acc[s][r];
            if (tij[s] == 0) tile_write(dcopy, lane, acc[s]);
            if (tij[s] == 1) tile_write(nextbuf, lane, acc[s]);
            if (tij[s] == 257) tile_write(diagbuf, lane, acc[s]);
        }
        __syncthreads();
        if (tid < n) {
            const double v = norm2[tid];
            if (!(v < 0x1p256)) atomicOr(flags, DQ_FLAG_NONFINITE);      // or what U has of it may be no fp32 number
            if (v == 0.0) atomicOr(flags, DQ_FLAG_SINGULAR);
        }
        if (wave == 0) {
            f64x4 dk = tile_read(dcopy, lane);
            for (int k = 0; k < nt; ++k) {
#pragma unroll
                for (int r = 0; r < 4; ++r) dcopy[(4 * r + g) * CLD + c] = dk[r];
                __builtin_amdgcn_wave_barrier();
                double d[16], x[16];
                int cc = c;
                asm volatile("" : "+v"(cc));
#pragma unroll
                for (int i = 0; i < 16; i += 2) {
                    const double2 v = *reinterpret_cast<const double2*>(&dcopy[c * CLD + i]);
                    d[i] = v.x; d[i + 1] = v.y;
                }
                const double len2 = norm2[16 * k + c];
                const double least = __builtin_fmax(len2 * 0x1p-44, 0x1p-600), one = len2 > 0.0 ? 1.0 : 0.0;   // (see chol64_kernel)
                double mine = 0.0;
#pragma unroll
                for (int i = 0; i < 16; ++i) x[i] = i == cc ? one : 0.0;
                factor_pivots<0>(d, x, cc, least, row_lane<0>(d[0]), mine);
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int i = 4 * g + q;
                    const double xv = pick4(g, x[q], x[4 + q], x[8 + q], x[12 + q]), dv = pick4(g, d[q], d[4 + q], d[8 + q], d[12 + q]);
                    winv[(k * 16 + i) * CLD + c] = xv;
                    if (i <= c) Us[(16 * k + i) * LD + 16 * k + c] = (float)dv;
                }
                lds_barrier();
                if (k + 1 < nt) {
                    const f64x4 next = tile_read(nextbuf + (k & 1) * 256, lane), diag = tile_read(diagbuf + (k & 1) * 256, lane);
                    const f64x4 u = tile_mul2(inverse_read(winv + k * 16 * CLD, c, g), next);
                    dk = tile_sub(u, u, diag);
                }
            }
        } else {
            for (int k = 0; k < nt; ++k) {
                lds_barrier();
                const f64x4 ik = inverse_read(winv + k * 16 * CLD, c, g);
#pragma unroll
                for (int s = 0; s < SLOTS; ++s) {
                    const int t = opaque(tij[s]), tj = t & 255;
                    if (t >> 8 == k && tj != k && tj < nt) {
                        acc[s] = tile_mul2(ik, acc[s]);
                        tile_write(tile(k, tj), lane, acc[s]);
#pragma unroll
                        for (int r = 0; r < 4; ++r) Us[(16 * k + 4 * r + g) * LD + 16 * tj + c] = (float)acc[s][r];
                    }
                }
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                if (lane == 0) __hip_atomic_fetch_add(&rows_done, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                while (__hip_atomic_load(&rows_done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) < rows_base + HW * (k + 1)) {}
                asm volatile("" ::: "memory");
#pragma unroll
                for (int s = 0; s < SLOTS; ++s) {
                    const int t = opaque(tij[s]), ti = t >> 8, tj = t & 255;
                    if (ti > k && tj < nt && t != 257 * (k + 1)) {
                        acc[s] = tile_sub(tile_read(tile(k, ti), lane), tile_read(tile(k, tj), lane), acc[s]);
                        if (t == 257 * (k + 1) + 1) tile_write(nextbuf + ((k + 1) & 1) * 256, lane, acc[s]);
                        if (t == 257 * (k + 2)) tile_write(diagbuf + ((k + 1) & 1) * 256, lane, acc[s]);
                    }
                }
            }
        }
        rows_base += HW * nt;
        // ---- Q^T = U^-T A^T in fp64, 16 rows of A a wavefront, as the factorisation forms U's rows
        f64x4 x[NT];
        if (wave < nt) {
            const float* Ap = again ? Rp : Zp;
            const long lda = again ? ldr : ldz;
            const int row = 16 * wave + c;
            const float* pr = Ap + (long)(row < n ? row : 0) * lda;
            float v[NT][4];
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int r = 0; r < 4; ++r) v[t][r] = pr[16 * t + 4 * r + g < n ? 16 * t + 4 * r + g : 0];
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int r = 0; r < 4; ++r) x[t][r] = row < n && 16 * t + 4 * r + g < n ? (double)v[t][r] : 0.0;
        }
        __syncthreads();
        if (wave < nt) {
#pragma unroll
            for (int k = 0; k < NT; ++k) {
                if (NT == 4 && k >= nt) continue;      // (of the other orders NT is the number of tiles)
                x[k] = tile_mul2(inverse_read(winv + k * 16 * CLD, c, g), x[k]);
#pragma unroll
                for (int t = k + 1; t < NT; ++t) {     // (a tile past the last gives what nobody uses)
                    x[t] = tile_sub(tile_read(tile(k, t), lane), x[k], x[t]);
                    asm volatile("" ::: "memory");     // the tiles of later steps do not fit the registers
                }
            }
        }
        // what lies past the last tile
        if (nt < NT)
            for (int e = tid; e < N * N; e += 64 * (HW + 1)) {
                const int r = e / N, q = e % N;
                if (r >= 16 * nt || q >= 16 * nt) Us[r * LD + q] = 0.f;
            }
        __syncthreads();
        if (wave < NT) {
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int r = 0; r < 4; ++r) Q[(16 * wave + c) * LD + 16 * t + 4 * r + g] = wave < nt && t < nt ? (float)x[t][r] : 0.f;
        }
        if (again && Up != nullptr) {      // U <- T U with T the second factor
            f32x4 v[NT];
            if (wave < NT)
#pragma unroll
                for (int t = 0; t < NT; ++t) {
                    v[t] = f32x4{};
#pragma unroll 1
                    for (int kk = wave; kk <= t; ++kk)
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            const int k = 4 * q + g;
                            float x = Us[(16 * wave + c) * LD + 16 * kk + k];
                            if (kk == wave) x = k >= c ? x : 0.f;
                            const bool in = 16 * kk + k <= 16 * t + c && 16 * t + c < n;
                            v[t] = MFMA16(x, in ? Up[(long)(16 * kk + k) * ldu + 16 * t + c] : 0.f, v[t]);
                        }
                }
            __syncthreads();
            if (wave < NT)
#pragma unroll
                for (int t = 0; t < NT; ++t)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int i = 16 * wave + 4 * g + r, j = 16 * t + c;
                        if (i <= j) Us[i * LD + j] = v[t][r];
                    }
        }
    }
    __syncthreads();
    for (int e = tid; e < N * N / 4; e += 64 * (HW + 1)) {
        const int r = e / (N / 4), q = e % (N / 4) * 4;
        if (r >= n || q >= n) continue;
        store_quad(Rp + (long)r * ldr + q, n - q, *reinterpret_cast<const float4*>(Q + r * LD + q));
        if (Up != nullptr) {
            float4 u = *reinterpret_cast<const float4*>(Us + r * LD + q);
            u.x = q >= r ? u.x : 0.f; u.y = q + 1 >= r ? u.y : 0.f; u.z = q + 2 >= r ? u.z : 0.f; u.w = q + 3 >= r ? u.w : 0.f;
            store_quad(Up + (long)r * ldu + q, n - q, u);
        }
    }
}

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
#define DQ_LAUNCH(NT)                                                                                                    \
    hipLaunchKernelGGL((heads_qr_kernel<NT>), dim3(b), dim3(64 * (HW + 1)), 0, s, Z, ldz, sz, R, ldr, sr, U, ldu, su, n, flags)
    if (n > 112) DQ_LAUNCH(8);
    else if (n > 96) DQ_LAUNCH(7);
    else if (n > 80) DQ_LAUNCH(6);
    else if (n > 64) DQ_LAUNCH(5);
    else DQ_LAUNCH(4);
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
