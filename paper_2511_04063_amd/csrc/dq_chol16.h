// 16 x 16 tiles of a symmetric positive definite matrix on the fp64 matrix cores, and the Cholesky factor of one on a wavefront
// (device code only; the QR's blocks of 256 columns and the small rotations).
#pragma once

#include "dq_internal.h"

namespace dq {
namespace {

typedef double f64x4 __attribute__((ext_vector_type(4)));
#define MFMA64(a, b, c) __builtin_amdgcn_mfma_f64_16x16x4f64((a), (b), (c), 0, 0, 0)

// v_mfma_f64_16x16x4: A[m = l % 16][k = l / 16], B[k = l / 16][n = l % 16], register r of the result D[m = 4 r + l / 16][n = l % 16].
// Register r of a tile that was a result is therefore the operand of the 4 k from 4 r of the same tile, as B and, transposed, as A:
// C -= P^T Q takes three such tiles as they lie.

constexpr int CLD = 18;   // row stride of a tile whose rows are read 16 bytes at a time: no bank conflicts

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
    for (int r = 0; r < 4; ++r) v[r] = w[c * CLD + 4 * r + g];
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

}  // namespace
}  // namespace dq
