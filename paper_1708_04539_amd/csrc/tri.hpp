// tri.hpp -- both triangular inverses of one diagonal block in LDS, by one
// workgroup (four wavefronts), in FP64.
#pragma once

#include "tiles.hpp"

namespace selinv {

// The block is held packed in one LDS tile, column-major: first the factors
// (strict lower part: L, upper part with the diagonal: U), then, in their
// place, the inverses (strict lower part: L^{-1}; upper part: U^{-1}).  Blocked
// by 16 (NB blocks; X = L^{-1}, Y = U^{-1}):
//   1. the 16x16 diagonal blocks, by substitution: wavefront w takes block w;
//      lane c < 16 forms column c of X_ww and lane 16 + c row c of Y_ww, the
//      same forward recurrence for both (the L diagonal is 1; U's diagonal
//      enters through reciprocals formed once per block);
//   2. the off-diagonal blocks on v_mfma_f64_16x16x4, a block row of X from
//      the top and one of Y from the bottom per round:
//        X_ij = -X_ii (sum_{k=j}^{i-1} L_ik X_kj)      i = 1, 2, 3
//        Y_ij = -Y_ii (sum_{k=i+1}^{j} U_ik Y_kj)      i = NB - 2, ...
//      A row of factor blocks is read by its own round only, so that the row's
//      results take its place after a barrier.  Odd wavefronts form Y; the
//      first pair takes the row's longest sum, the second the other one or two.
// One tile of 33 KB instead of two and a staging buffer (76 KB) lets four
// workgroups share a compute unit instead of two.
template <int NB>
struct TriSmem {
    static constexpr int W = 16 * NB;
    double M[W][W + 1];  // M[c][r]
    double rd[W];        // 1 / U(c, c)
};

// L^{-1}(r, c) and U^{-1}(r, c) read from the packed tile (zero outside the
// triangle; the unit diagonal of L^{-1} is implicit)
// (read first, selected after: a conditional read would be a branch and a wait
// of its own)
template <class SM>
__device__ __forceinline__ double linv_at(const SM &sm, int r, int c) {
    const double v = sm.M[c][r];
    return r > c ? v : (r == c ? 1.0 : 0.0);
}
template <class SM>
__device__ __forceinline__ double uinv_at(const SM &sm, int r, int c) {
    const double v = sm.M[c][r];
    return r <= c ? v : 0.0;
}

// The block of round R whose sum has LEN blocks, formed by the calling
// wavefront (upper: of Y, else of X).  The lanes feed the MFMA with
// A(i = lane % 16, k = lane / 16) and B(k = lane / 16, j = lane % 16); result
// register v holds row lane / 16 + 4 v, column lane % 16, which is the B operand
// of k step v: the sum goes into the second product as it is.
template <int NB, int R, int LEN, class SM>
__device__ __forceinline__ v4d tri_offdiag(const SM &sm, bool upper, int lane) {
    const int i = upper ? NB - 1 - R : R;          // block row
    const int j = upper ? i + LEN : R - LEN;       // block column
    const int kb = 16 * (upper ? i + 1 : j);       // contraction range [kb, kb + 16 LEN)
    const int li = lane & 15, lk = lane >> 4, c = 16 * j + li;
    v4d acc = {0, 0, 0, 0};
#pragma unroll
    for (int kk = 0; kk < 16 * LEN; kk += 4) {
        const int k = kb + kk + lk;
        const double a = sm.M[k][16 * i + li];  // factor entry, off the diagonal blocks
        double x = sm.M[c][k];                  // X(k, c) or Y(k, c)
        // the first block of a sum of X, the last one of Y, is a diagonal block
        if (kk < 16 || kk >= 16 * (LEN - 1)) x = upper ? (k <= c ? x : 0.0) : (k > c ? x : k == c ? 1.0 : 0.0);
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a, x, acc, 0, 0, 0);
    }
    v4d out = {0, 0, 0, 0};
#pragma unroll
    for (int v = 0; v < 4; v++) {
        const int r = 16 * i + li, q = 16 * i + 4 * v + lk;
        const double x = sm.M[q][r];
        const double a = upper ? (r <= q ? x : 0.0) : (r > q ? x : r == q ? 1.0 : 0.0);
        out = __builtin_amdgcn_mfma_f64_16x16x4f64(a, acc[v], out, 0, 0, 0);
    }
    return out;
}

template <int NB, int R, class SM>
__device__ __forceinline__ void tri_round(SM &sm, int lane, int wave) {
    const bool upper = wave & 1;
    v4d o1 = {0, 0, 0, 0}, o2 = {0, 0, 0, 0};
    __syncthreads();  // the rows this one needs are complete
    if (wave < 2)
        o1 = tri_offdiag<NB, R, R>(sm, upper, lane);
    else {
        if constexpr (R >= 2) o1 = tri_offdiag<NB, R, R - 1>(sm, upper, lane);
        if constexpr (R >= 3) o2 = tri_offdiag<NB, R, R - 2>(sm, upper, lane);
    }
    __syncthreads();  // this row's factors are read
    auto put = [&](const v4d &o, int len) {
        const int i = upper ? NB - 1 - R : R, j = upper ? i + len : R - len;
#pragma unroll
        for (int v = 0; v < 4; v++) sm.M[16 * j + (lane & 15)][16 * i + (lane >> 4) + 4 * v] = -o[v];
    };
    if (wave < 2)
        put(o1, R);
    else {
        if constexpr (R >= 2) put(o1, R - 1);
        if constexpr (R >= 3) put(o2, R - 2);
    }
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

// Both triangular inverses of the 16 NB wide block in sm.M (packed L \ U,
// identity-padded), with the reciprocals of U's diagonal in sm.rd, in place.
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
        for (int k = 0; k < 15; k++) m[k] = up ? sm.M[base + c][base + k] : sm.M[base + k][base + c];
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
            if (!up && r > c) sm.M[base + c][base + r] = x[r];  // X(r, c)
            if (up && r >= c) sm.M[base + r][base + c] = x[r];  // Y(c, r)
        }
    }
    if constexpr (NB >= 2) tri_round<NB, 1>(sm, lane, wave);
    if constexpr (NB >= 3) tri_round<NB, 2>(sm, lane, wave);
    if constexpr (NB >= 4) tri_round<NB, 3>(sm, lane, wave);
}

}  // namespace selinv
