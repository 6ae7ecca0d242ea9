// tri.hpp -- both triangular inverses of one diagonal block in LDS, by one
// workgroup (four wavefronts), in FP64.
#pragma once

#include "tiles.hpp"

namespace selinv {

// Blocked by 16 (NB blocks):
//   1. the 16x16 diagonal blocks, by substitution: wavefront w takes block w;
//      lane c < 16 forms column c of (L_ww)^{-1} and lane 16 + c column c of
//      (U_ww^T)^{-1} = row c of (U_ww)^{-1}, the same forward recurrence for
//      both (the L diagonal is 1; U's diagonal enters through reciprocals
//      formed once per block);
//   2. the off-diagonal 16x16 blocks by distance d = 1, 2, 3 from the
//      diagonal, on v_mfma_f64_16x16x4 (X = L^{-1}, Y = U^{-1}):
//        X_ij = -X_ii (sum_{k=j}^{i-1} L_ik X_kj)      (i = j + d)
//        Y_ij = -Y_ii (sum_{k=i+1}^{j} U_ik Y_kj)      (j = i + d)
//      every block of one distance in parallel, one per wavefront.
// Both results live packed in one LDS tile (strict lower part: L^{-1}; upper
// part with the diagonal: U^{-1}).
template <int NB>
struct TriSmem {
    static constexpr int W = 16 * NB;
    double Ds[W][65];        // Ds[c][r] = D(o + r, o + c), identity-padded; later a panel (64 rows)
    double Xs[W][W + 1];     // Xs[c][r]: r > c: L^{-1}(r, c); r <= c: U^{-1}(r, c)
    double Ts[4][16][17];    // per-wavefront 16x16 intermediate
    double rd[W];            // 1 / U(c, c)
};

typedef double v4d_t __attribute__((ext_vector_type(4)));

// L^{-1}(r, c) and U^{-1}(r, c) read from the packed tile (zero outside the
// triangle; the unit diagonal of L^{-1} is implicit)
// (read first, selected after: a conditional read would be a branch and a wait
// of its own)
template <class SM>
__device__ __forceinline__ double linv_at(const SM &sm, int r, int c) {
    const double v = sm.Xs[c][r];
    return r > c ? v : (r == c ? 1.0 : 0.0);
}
template <class SM>
__device__ __forceinline__ double uinv_at(const SM &sm, int r, int c) {
    const double v = sm.Xs[c][r];
    return r <= c ? v : 0.0;
}

// One off-diagonal block at distance D, computed by the calling wavefront.
// The lanes feed the MFMA with A(i = lane % 16, k = lane / 16) and
// B(k = lane / 16, j = lane % 16); the result row is lane / 16 + 4 v, its
// column lane % 16 (register v of the accumulator).
template <int NB, int D, class SM>
__device__ __forceinline__ void tri_offdiag(SM &sm, int t, int lane, int wave) {
    const bool upper = t >= NB - D;
    const int i = upper ? t - (NB - D) : t + D;  // row block of the result
    const int j = upper ? i + D : t;             // column block
    const int kb = upper ? 16 * (i + 1) : 16 * j;  // contraction range [kb, kb + 16 D)
    const int li = lane & 15, lk = lane >> 4;
    v4d_t acc = {0, 0, 0, 0};
#pragma unroll
    for (int kk = 0; kk < 16 * D; kk += 4) {
        const int k = kb + kk + lk;
        // factor entry L(16 i + li, k) or U(16 i + li, k): strictly off the diagonal
        const double a = sm.Ds[k][16 * i + li];
        const int bc = 16 * j + li;
        const double x = sm.Xs[bc][k];  // U^{-1}(k, bc) or L^{-1}(k, bc)
        const double bv = upper ? (k <= bc ? x : 0.0) : (k > bc ? x : k == bc ? 1.0 : 0.0);
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a, bv, acc, 0, 0, 0);
    }
#pragma unroll
    for (int v = 0; v < 4; v++) sm.Ts[wave][lk + 4 * v][li] = acc[v];
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    v4d_t out = {0, 0, 0, 0};
#pragma unroll
    for (int kk = 0; kk < 16; kk += 4) {
        const int r = 16 * i + li, c = 16 * i + kk + lk;
        const double x = sm.Xs[c][r];
        const double a = upper ? (r <= c ? x : 0.0) : (r > c ? x : r == c ? 1.0 : 0.0);
        out = __builtin_amdgcn_mfma_f64_16x16x4f64(a, sm.Ts[wave][kk + lk][li], out, 0, 0, 0);
    }
#pragma unroll
    for (int v = 0; v < 4; v++) sm.Xs[16 * j + li][16 * i + lk + 4 * v] = -out[v];
    // the wavefront's next task overwrites Ts
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

template <int NB, int D, class SM>
__device__ __forceinline__ void tri_round(SM &sm, int lane, int wave) {
    __syncthreads();
    for (int t = wave; t < 2 * (NB - D); t += 4) tri_offdiag<NB, D>(sm, t, lane, wave);
}

// v of lane R of every group of 16 lanes (row_newbcast)
template <int R>
__device__ __forceinline__ double row_bcast(double v) {
    const int64_t b = __builtin_bit_cast(int64_t, v);
    const uint32_t lo = __builtin_amdgcn_update_dpp(0, (int)b, 0x150 + R, 0xf, 0xf, true);
    const uint32_t hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), 0x150 + R, 0xf, 0xf, true);
    return __builtin_bit_cast(double, (int64_t)(((uint64_t)hi << 32) | lo));
}

// Steps K.. of the forward recurrence x[K] *= dg(K) (DG), x[r] -= m(r, K) x[K]
// (r > K); lane r of the group holds m(r, :) and dg(r).
template <int K, int R>
__device__ __forceinline__ void tri_eliminate(const double (&m)[16], double (&x)[16]) {
    if constexpr (R < 16) {
        x[R] = fma(-row_bcast<R>(m[K]), x[K], x[R]);
        tri_eliminate<K, R + 1>(m, x);
    }
}
template <int K, bool DG>
__device__ __forceinline__ void tri_substitute(const double (&m)[16], double (&x)[16], double dg) {
    if constexpr (K < 16) {
        if constexpr (DG) x[K] *= row_bcast<K>(dg);
        if constexpr (K < 15) tri_eliminate<K, K + 1>(m, x);
        tri_substitute<K + 1, DG>(m, x, dg);
    }
}

// Both triangular inverses of the 16 NB wide block in sm.Ds (packed L \ U,
// identity-padded), with the reciprocals of U's diagonal in sm.rd, into sm.Xs.
template <int NB, class SM>
__device__ __forceinline__ void tri_invert(SM &sm, int lane, int wave) {
    if (wave < NB && lane < 32) {
        const int base = 16 * wave, c = lane & 15;
        const bool up = (lane & 16) != 0;
        // lane c of each group of 16 holds row c of its side's unit lower factor
        // (L, or U^T with the diagonal apart); row r reaches the group's other
        // lanes by DPP, so that the recurrence itself reads no LDS
        double m[16], x[16];
#pragma unroll
        for (int k = 0; k < 15; k++) m[k] = up ? sm.Ds[base + c][base + k] : sm.Ds[base + k][base + c];
        const double dg = up ? sm.rd[base + c] : 1.0;
#pragma unroll
        for (int r = 0; r < 16; r++) x[r] = r == c ? 1.0 : 0.0;
        tri_substitute<0, true>(m, x, dg);
        // the whole recurrence here, not each value's part of it under the
        // conditional store that takes it
#pragma unroll
        for (int r = 0; r < 16; r++) asm volatile("" : "+v"(x[r]));
#pragma unroll
        for (int r = 0; r < 16; r++) {
            if (!up && r > c) sm.Xs[base + c][base + r] = x[r];  // L^{-1}(r, c)
            if (up && r >= c) sm.Xs[base + r][base + c] = x[r];  // U^{-1}(c, r)
        }
    }
    if constexpr (NB >= 2) tri_round<NB, 1>(sm, lane, wave);
    if constexpr (NB >= 3) tri_round<NB, 2>(sm, lane, wave);
    if constexpr (NB >= 4) tri_round<NB, 3>(sm, lane, wave);
}

}  // namespace selinv
