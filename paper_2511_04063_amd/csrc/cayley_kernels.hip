// Elementwise pieces of Cayley SGD with momentum (Alg. 3, App. B.2), the optimiser the paper compares QR-Orth with
// (Sec. 5, optimiser comparison).  Its six n x n products run on the fp32 matrix-core GEMM; what is left are
// HBM-bound passes over n x n matrices: the momentum update, the skew-symmetrisation with the Frobenius norm that the
// step-size rule needs, the step size itself (a device scalar: no host round trip), and sums of two matrices.
#include <math.h>

#include "dq_internal.h"

namespace dq {
namespace {

// M <- beta M - G  (Alg. 3, momentum update).  This pass and the sums below move three matrices and are bound by memory: at n =
// 4096 63 us before, with a division per piece and 4-byte accesses.
__global__ __launch_bounds__(256) void cayley_momentum_kernel(float* __restrict__ M, long ldm, const float* __restrict__ G,
                                                             long ldg, int n, float beta) {
    for_quads(n, n, [&](long r, int c, int left) {
        const float4 m = load_quad(M + r * ldm + c, left), g = load_quad(G + r * ldg + c, left);
        store_quad(M + r * ldm + c, left,
                   make_float4(beta * m.x - g.x, beta * m.y - g.y, beta * m.z - g.z, beta * m.w - g.w));
    });
}

// The same with the scan of the new M for values without a split (launch_range_scan) on the way: a word per workgroup, four
// pieces of M and G in flight per lane.  (A scan of its own costs 9 us at n = 1290 to 2560.)
__global__ __launch_bounds__(1024) void cayley_momentum_scan_kernel(float* __restrict__ M, long ldm, const float* __restrict__ G,
                                                                   long ldg, int n, float beta, unsigned* __restrict__ words) {
    unsigned bad = 0u;
    const int lane = threadIdx.x & 63, whole = n >> 2;
    for (int r = blockIdx.x * 16 + (threadIdx.x >> 6); r < n; r += gridDim.x * 16) {
        float* m = M + (long)r * ldm;
        const float* g = G + (long)r * ldg;
        for (int q = lane; q < whole; q += 256) {
            float4 a[4], b[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                a[k] = b[k] = make_float4(0.f, 0.f, 0.f, 0.f);
                if (q + 64 * k < whole) {
                    a[k] = *reinterpret_cast<const float4*>(m + 4 * (q + 64 * k));
                    b[k] = *reinterpret_cast<const float4*>(g + 4 * (q + 64 * k));
                }
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const float4 v = make_float4(beta * a[k].x - b[k].x, beta * a[k].y - b[k].y, beta * a[k].z - b[k].z,
                                             beta * a[k].w - b[k].w);
                bad |= no_split(v);
                if (q + 64 * k < whole) *reinterpret_cast<float4*>(m + 4 * (q + 64 * k)) = v;
            }
        }
        if (4 * whole + lane < n) {             // at most three columns are left
            const float v = beta * m[4 * whole + lane] - g[4 * whole + lane];
            bad |= no_split(v);
            m[4 * whole + lane] = v;
        }
    }
    const bool any = __syncthreads_or(bad != 0u) != 0;
    if (threadIdx.x == 0) words[blockIdx.x] = any ? 1u : 0u;
}

// W = What - What^T (Alg. 3, skew-symmetrisation) on 32 x 32 tiles: tile (bi, bj) and its mirror are both read row-wise (coalesced)
// and the mirror is transposed through LDS.  Each block also leaves the sum of squares of the entries it wrote.
__global__ __launch_bounds__(256) void cayley_skew_kernel(const float* __restrict__ H, long ldh, int n, float* __restrict__ W,
                                                         long ldw, double* __restrict__ partials) {
    __shared__ float mirror[32][33];
    __shared__ float wsum[4];
    const int tiles = (n + 31) >> 5;
    const int bi = blockIdx.x / tiles, bj = blockIdx.x % tiles;
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
    for (int i = ty; i < 32; i += 8) {
        const int r = bj * 32 + i, c = bi * 32 + tx;        // the mirror tile (bj, bi)
        mirror[i][tx] = (r < n && c < n) ? H[(long)r * ldh + c] : 0.f;
    }
    __syncthreads();
    float acc = 0.f;
    for (int i = ty; i < 32; i += 8) {
        const int r = bi * 32 + i, c = bj * 32 + tx;
        if (r < n && c < n) {
            const float w = H[(long)r * ldh + c] - mirror[tx][i];
            W[(long)r * ldw + c] = w;
            acc += w * w;
        }
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) acc += __shfl_xor(acc, o);
    if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) partials[blockIdx.x] = ((double)wsum[0] + (double)wsum[1]) + ((double)wsum[2] + (double)wsum[3]);
}

// alpha = min(lr, 2 q / (||W||_F + eps))  (Alg. 3, step-size rule); out[0] = alpha, out[1] = alpha / 2
__global__ __launch_bounds__(1024) void cayley_alpha_kernel(const double* __restrict__ partials, int count, float lr, float q,
                                                          float eps, float* __restrict__ out) {
    // one workgroup, a chain of loads: four in flight per thread (16384 partials at n = 4096: 18 us with 256 threads and one load,
    // 5 with 1024; the few hundred of small orders are summed by 256 threads, and by lane exchanges instead of ten barriers)
    __shared__ double sh[16];
    const int nt = (int)blockDim.x;
    double t[4] = {0.0, 0.0, 0.0, 0.0};
    int i = threadIdx.x;
    for (; i + 3 * nt < count; i += 4 * nt) {
        const double a = partials[i], b = partials[i + nt], c = partials[i + 2 * nt], d = partials[i + 3 * nt];
        t[0] += a; t[1] += b; t[2] += c; t[3] += d;
    }
    for (; i < count; i += nt) t[0] += partials[i];
    double sum = (t[0] + t[1]) + (t[2] + t[3]);
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) sum += __shfl_xor(sum, o);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = sum;
    __syncthreads();
    if (threadIdx.x == 0) {
        double total = 0.0;
        for (int w = 0; w < nt / 64; ++w) total += sh[w];
        const float norm = (float)sqrt(total);
        const float cap = 2.f * q / (norm + eps);
        const float alpha = lr < cap ? lr : cap;        // a NaN norm leaves lr
        out[0] = alpha;
        out[1] = 0.5f * alpha;
    }
}

// out = A + scale B
__global__ __launch_bounds__(256) void add_scaled_kernel(float* out, long ldo, const float* A, long lda, const float* B,
                                                        long ldb, int n, float scale_host, const float* __restrict__ scale_dev) {
    const float sc = scale_dev != nullptr ? scale_host * *scale_dev : scale_host;
    for_quads(n, n, [&](long r, int c, int left) {
        const float4 x = load_quad(A + r * lda + c, left), y = load_quad(B + r * ldb + c, left);
        store_quad(out + r * ldo + c, left, make_float4(x.x + sc * y.x, x.y + sc * y.y, x.z + sc * y.z, x.w + sc * y.w));
    });
}

}  // namespace

hipError_t launch_cayley_momentum(float* M, long ldm, const float* G, long ldg, int n, float beta, unsigned* words, hipStream_t s) {
    if (words != nullptr) {
        hipLaunchKernelGGL(cayley_momentum_scan_kernel, dim3(kGuardWords), dim3(1024), 0, s, M, ldm, G, ldg, n, beta, words);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(cayley_momentum_kernel, quad_grid(n, n), dim3(256), 0, s, M, ldm, G, ldg, n, beta);
    return hipGetLastError();
}

int cayley_skew_grid(int n) {
    const int tiles = (n + 31) / 32;
    return tiles * tiles;
}

hipError_t launch_cayley_skew(const float* What, long ldh, int n, float* W, long ldw, double* partials, hipStream_t s) {
    hipLaunchKernelGGL(cayley_skew_kernel, dim3(cayley_skew_grid(n)), dim3(256), 0, s, What, ldh, n, W, ldw, partials);
    return hipGetLastError();
}

hipError_t launch_cayley_alpha(const double* partials, int count, float lr, float q, float eps, float* alpha_dev,
                               hipStream_t s) {
    hipLaunchKernelGGL(cayley_alpha_kernel, dim3(1), dim3(count <= 2048 ? 256 : 1024), 0, s, partials, count, lr, q, eps, alpha_dev);
    return hipGetLastError();
}

hipError_t launch_add_scaled(float* out, long ldo, const float* A, long lda, const float* B, long ldb, int n,
                             float scale_host, const float* scale_dev, hipStream_t s) {
    hipLaunchKernelGGL(add_scaled_kernel, quad_grid(n, n), dim3(256), 0, s, out, ldo, A, lda, B, ldb, n,
                       scale_host, scale_dev);
    return hipGetLastError();
}

}  // namespace dq
