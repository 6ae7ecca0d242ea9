// lu_device.hip -- kernels of the supernodal LU without pivoting on the GPU:
// the factorisation At = L U (eq. LU) that Algorithm 1 of arXiv:1708.04539
// starts from, in the block storage the selected inversion reads (the s x s
// diagonal block holding L_KK \ U_KK, the c_L x s panel L(R_L, K) and the
// c_U x s panel U(K, R_U)^T of every supernode K).
//
// The host orchestration (runtime.hip) runs the levels of the supernodal
// dependency graph from the deepest up.  Per level, in 64-column steps j0 of
// every supernode's diagonal block:
//   lu_tile_kernel   LU of the 64 x 64 tile at (j0, j0) and the inverses of
//                    its unit L and of its U;
//   grouped GEMM     the solves against the tile as products with those
//                    inverses, in place: the rows of D below the tile and of
//                    the L panel times U11^{-1}, L11^{-1} times the columns of
//                    D right of the tile, the rows of the U panel times
//                    L11^{-T};
//   grouped GEMM     the trailing updates of the block and the panels;
// then schur_scatter_kernel, which forms the Schur complement product W_K =
// -L(R_L, K) U(K, R_U) and adds it to the blocks of the ancestors.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "device_types.hpp"
#include "kernels.hpp"
#include "tiles.hpp"
#include "tri.hpp"

namespace selinv {

// vals[p] (emb == nullptr), or for complex handles the entry of the real form
// taken from the interleaved complex values: emb[p] = source << 1 | negate
__global__ __launch_bounds__(256) void scatter_values_kernel(const int64_t *__restrict__ loc,
                                                             const double *__restrict__ vals,
                                                             const int64_t *__restrict__ emb, int64_t nnz,
                                                             double *diag, double *lpan, double *upan) {
    const int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (p >= nnz) return;
    const int64_t l = gptr(loc)[p];
    const int64_t kind = l >> 60, off = l & ((int64_t(1) << 60) - 1);
    double v;
    if (emb) {
        const int64_t e = gptr(emb)[p];
        v = gptr(vals)[e >> 1];
        if (e & 1) v = -v;
    } else {
        v = gptr(vals)[p];
    }
    double *dst = kind == 0 ? diag : kind == 1 ? lpan : upan;
    gptr_w(dst)[off] = v;
}

// LU of the 16 nb wide block in sm.M (identity-padded) by one workgroup, in
// 16-column panels: one wavefront eliminates the panel with lane i holding row
// i of it in registers (the pivot row reaches the other lanes through scalar
// registers, v_readlane), the other three form the rows of U right of it, 16
// columns each (lane = column, substitution with the panel's unit L), then all
// four update the rest on v_mfma_f64_16x16x4.
__device__ __forceinline__ double lane_value(double v, int lane) {
    return __builtin_bit_cast(double, lane_value(__builtin_bit_cast(int64_t, v), lane));
}

template <class SM>
__device__ __forceinline__ void lu_factor_block(SM &sm, int nb, int lane, int wave) {
    const int li = lane & 15, lk = lane >> 4;
    for (int kb = 0; kb < nb; kb++) {
        const int k0 = 16 * kb;
        if (wave == 0) {
            double a[16];
#pragma unroll
            for (int c = 0; c < 16; c++) a[c] = sm.M[k0 + c][lane];
            // the reciprocal of the next pivot is formed as soon as its column is
            // updated, beside the updates of the other columns
            double rp = 1.0 / lane_value(a[0], k0);
#pragma unroll
            for (int k = 0; k < 15; k++) {
                double u[16];
#pragma unroll
                for (int c = k + 1; c < 16; c++) u[c] = lane_value(a[c], k0 + k);
                // rows above keep their values (l = 0); a non-finite u could
                // spoil them, but then the pivot of its column is rejected too
                const bool below = lane > k0 + k;
                const double l = below ? a[k] * rp : 0.0;
                a[k] = below ? l : a[k];
                a[k + 1] = fma(-l, u[k + 1], a[k + 1]);
                rp = 1.0 / lane_value(a[k + 1], k0 + k + 1);
#pragma unroll
                for (int c = k + 2; c < 16; c++) a[c] = fma(-l, u[c], a[c]);
            }
            if (lane > k0 + 15) a[15] *= rp;
#pragma unroll
            for (int c = 0; c < 16; c++) sm.M[k0 + c][lane] = a[c];
        }
        __syncthreads();
        if (kb + 1 == nb) break;
        if (wave > 0 && lane < 16 && kb + wave < nb) {  // block column kb + wave
            double m[16], x[16];  // row `lane` of the panel's unit L, column `lane` of the block
            double *col = sm.M[k0 + 16 * wave + lane];
#pragma unroll
            for (int r = 0; r < 16; r++) {
                m[r] = sm.M[k0 + r][k0 + lane];
                x[r] = col[k0 + r];
            }
            tri_substitute<0, false>(m, x, 1.0);
#pragma unroll
            for (int r = 1; r < 16; r++) col[k0 + r] = x[r];
        }
        __syncthreads();
        const int nt = nb - kb - 1;
        for (int t = wave; t < nt * nt; t += 4) {
            const int i = k0 + 16 + 16 * (t % nt), j = k0 + 16 + 16 * (t / nt);
            v4d acc;
#pragma unroll
            for (int v = 0; v < 4; v++) acc[v] = sm.M[j + li][i + lk + 4 * v];
#pragma unroll
            for (int kk = 0; kk < 16; kk += 4)
                acc = __builtin_amdgcn_mfma_f64_16x16x4f64(-sm.M[k0 + kk + lk][i + li], sm.M[j + li][k0 + kk + lk],
                                                           acc, 0, 0, 0);
#pragma unroll
            for (int v = 0; v < 4; v++) sm.M[j + li][i + lk + 4 * v] = acc[v];
        }
        __syncthreads();
    }
}

// The b x b tile (b = min(64, s - j0)) at (j0, j0) of the column-major s x s
// block D: its LU in place, and the inverses of its unit L and of its U into
// the same place of Linv and Uinv (the solves of the rows below it and of the
// columns right of it are products with them).  A zero or non-finite pivot
// lowers *bad to its permuted column f + j0 + k (the arithmetic goes on; the
// host reports the failure).
// Bound by the chain of 64 pivots, each a reciprocal and a rank-one update.
// One wavefront over the whole tile (64-wide rows in registers, the pivot row
// through LDS) took 36 us a launch and the inverses another 15 us in a launch
// of their own (2D 256^2); blocked by 16, both take 22 us in one launch (about
// 9 of them the pivot chain, 3.5 the rows of U, 5.5 the inverses).
__global__ __launch_bounds__(256) void lu_tile_kernel(const LuTile *__restrict__ items, int32_t *bad) {
    __shared__ TriSmem<4> sm;
    const LuTile it = items[blockIdx.x];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int s = it.s, b = min(64, s - it.j0), nb = (b + 15) / 16;
    const int64_t at = it.j0 + (int64_t)it.j0 * s;
    SELINV_GLOBAL double *D = gptr_w(it.D) + at;
    {
        // all loads in flight at once (clamped addresses), identity padding
        double v[16];
#pragma unroll
        for (int q = 0; q < 16; q++) v[q] = D[min(lane, b - 1) + (int64_t)min(wave + 4 * q, b - 1) * s];
#pragma unroll
        for (int q = 0; q < 16; q++) {
            const int c = wave + 4 * q;
            sm.M[c][lane] = (lane < b && c < b) ? v[q] : (lane == c ? 1.0 : 0.0);
        }
    }
    __syncthreads();
    lu_factor_block(sm, nb, lane, wave);
    if (tid < 64) {
        const double p = sm.M[tid][tid];
        sm.rd[tid] = 1.0 / p;
        if (tid < b && !(p != 0.0 && isfinite(p))) atomicMin(bad, it.f + it.j0 + tid);
    }
#pragma unroll
    for (int q = 0; q < 16; q++) {
        const int c = wave + 4 * q;
        if (lane < b && c < b) D[lane + (int64_t)c * s] = sm.M[c][lane];
    }
    __syncthreads();
    if (nb > 2)
        tri_invert<4>(sm, lane, wave);
    else if (nb == 2)
        tri_invert<2>(sm, lane, wave);
    else
        tri_invert<1>(sm, lane, wave);
    __syncthreads();
    SELINV_GLOBAL double *Linv = gptr_w(it.Linv) + at, *Uinv = gptr_w(it.Uinv) + at;
#pragma unroll
    for (int q = 0; q < 16; q++) {
        const int c = wave + 4 * q;
        if (lane < b && c < b) {
            Linv[lane + (int64_t)c * s] = linv_at(sm, lane, c);
            Uinv[lane + (int64_t)c * s] = uinv_at(sm, lane, c);
        }
    }
}

// One 64 x 64 tile of W_K = -L(R_L,K) U(K,R_U) (c_L x c_U) per workgroup, added
// to the blocks of the ancestors.  W_K(a, b) belongs to entry (R_L(K)[a],
// R_U(K)[b]) of At, which lies in the diagonal block of J (I = J), the L panel
// of J (I > J) or the U panel of I (I < J), I and J the supernodes of its row
// and column; the relative-index maps give its place there.  As in the gather
// of the selected inversion (the same positions, read there), the tile's row
// and column records go to LDS first; the product tile follows into LDS, then
// the diagonal and L-side entries are added with the threads along the rows
// (contiguous in the L panels) and the U-side entries along the columns
// (contiguous in the U panels).  Supernodes of one level update the same
// entries of their common ancestors, hence the atomic adds.
// Bound by the atomic adds and their scattered places.  W_K in memory between
// a product launch and a scatter launch (16 bytes an entry and a launch more a
// level) took 2.19 ms on the 3D 40^3 27-point matrix and 275 us on the 2D 256^2
// one; in one launch 1.82 ms and 187 us.
__global__ __launch_bounds__(256) void schur_scatter_kernel(const MatDev *__restrict__ mat,
                                                            const GatherTile *__restrict__ tiles, double *diag,
                                                            double *lpan, double *upan) {
    union Shared {
        DmaSmem<64, 64> g;
        double t[64][65];  // [b][a]
    };
    __shared__ Shared sm;
    double(&tileS)[64][65] = sm.t;
    __shared__ int32_t rowR[64], rowI[64], colJ[64];
    __shared__ int64_t rowUp[64], rowUoff[64], colDiag[64], colLow[64], colLoff[64];
    const GatherTile gt = tiles[xcd_tile(blockIdx.x, gridDim.x)];
    const MatDev &M = *mat;
    const SELINV_GLOBAL SnRec *sn = gptr(M.sn);
    const SELINV_GLOBAL int32_t *supof = gptr(M.supof);
    const int K = gt.K, a0 = gt.a0, b0 = gt.b0, cl = gt.cl, cu = gt.cu;
    const int64_t rl_off = sn[K].rl_off, ru_off = sn[K].ru_off;
    const int tid = threadIdx.x;
    const int na = min(64, cl - a0), nb = min(64, cu - b0);  // both >= 1
    if (tid < 64) {
        const int t = min(tid, na - 1);
        const int64_t a = rl_off + a0 + t;
        const int32_t r = gptr(M.rl)[a];
        const int64_t uo = gptr(M.u_rowoff)[a];
        const int32_t I = supof[r];
        if (tid < na) {
            rowR[tid] = r;
            rowI[tid] = I;
            rowUp[tid] = sn[I].off_u + (int64_t)(r - sn[I].f) * sn[I].cu;
            rowUoff[tid] = uo + b0;
        }
    } else if (tid < 128) {
        const int t = min(tid - 64, nb - 1);
        const int64_t bb = ru_off + b0 + t;
        const int32_t c = gptr(M.ru)[bb];
        const int64_t lo = gptr(M.l_coloff)[bb];
        const int32_t J = supof[c];
        if (tid - 64 < nb) {
            colJ[t] = J;
            colDiag[t] = sn[J].off_d + (int64_t)(c - sn[J].f) * sn[J].s - sn[J].f;
            colLow[t] = sn[J].off_l + (int64_t)(c - sn[J].f) * sn[J].cl;
            colLoff[t] = lo + a0;
        }
    }
    constexpr int PER = 64 * 64 / 256;
    {
        GemmProb p;
        p.A = lpan + sn[K].off_l;
        p.B = upan + sn[K].off_u;
        p.M = p.lda = cl;
        p.N = p.ldb = cu;
        p.K = sn[K].s;
        p.ktri = p.cpx = 0;
        AccTile<CMP_F64, 64, 64> w;
        DmaProduct<CMP_F64, 64, 64, 0, 1>::form(p, a0, b0, sm.g, w);
        __syncthreads();  // LDS free for the tile
        const int lane = tid & 63, wave = tid >> 6;
#pragma unroll
        for (int i = 0; i < 2; i++)
#pragma unroll
            for (int j = 0; j < 2; j++)
#pragma unroll
                for (int v = 0; v < 4; v++)
                    tileS[(wave & 1) * 32 + j * 16 + (lane >> 4) + 4 * v][(wave >> 1) * 32 + i * 16 + (lane & 15)] =
                        -w.a[i][j][v];
    }
    __syncthreads();
    const SELINV_GLOBAL int32_t *mapL = gptr(M.mapL);
    const SELINV_GLOBAL int32_t *mapU = gptr(M.mapU);
    {
        int kind[PER];  // 0 none, 1 diagonal block, 2 L panel
        int32_t mi[PER];
#pragma unroll
        for (int t = 0; t < PER; t++) {
            const int e = tid + 256 * t, ia = e & 63, ib = e >> 6;
            kind[t] = 0;
            if (ia < na && ib < nb) {
                const int32_t I = rowI[ia], J = colJ[ib];
                kind[t] = I == J ? 1 : (I > J ? 2 : 0);
            }
        }
#pragma unroll
        for (int t = 0; t < PER; t++) {
            const int e = tid + 256 * t, ia = e & 63, ib = e >> 6;
            mi[t] = mapL[kind[t] == 2 ? colLoff[ib] + ia : 0];
        }
#pragma unroll
        for (int t = 0; t < PER; t++) {
            const int e = tid + 256 * t, ia = e & 63, ib = e >> 6;
            if (kind[t] == 1)
                atomicAdd(diag + colDiag[ib] + rowR[ia], tileS[ib][ia]);
            else if (kind[t] == 2)
                atomicAdd(lpan + colLow[ib] + mi[t], tileS[ib][ia]);
        }
    }
    {
        bool up[PER];
        int32_t mi[PER];
#pragma unroll
        for (int t = 0; t < PER; t++) {
            const int e = tid + 256 * t, ib = e & 63, ia = e >> 6;
            up[t] = ia < na && ib < nb && rowI[ia] < colJ[ib];
        }
#pragma unroll
        for (int t = 0; t < PER; t++) {
            const int e = tid + 256 * t, ib = e & 63, ia = e >> 6;
            mi[t] = mapU[up[t] ? rowUoff[ia] + ib : 0];
        }
#pragma unroll
        for (int t = 0; t < PER; t++) {
            const int e = tid + 256 * t, ib = e & 63, ia = e >> 6;
            if (up[t]) atomicAdd(upan + rowUp[ia] + mi[t], tileS[ib][ia]);
        }
    }
}

// Zeros into the factor storage and the pivot flag to "none", in one launch
// (three fills by hipMemsetAsync, of two kernels each, and one of the flag took
// 34 us on the 2D 256^2 matrix (72 MB), this 12 us).
__global__ __launch_bounds__(256) void clear_factors_kernel(double *diag, int64_t nd, double *lpan, int64_t nl,
                                                            double *upan, int64_t nu, int32_t *bad) {
    const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x, n = gridDim.x * (int64_t)blockDim.x;
    if (t == 0) *bad = LU_NO_BAD_PIVOT;
    auto clear = [&](double *p, int64_t len) {
        typedef double v2 __attribute__((ext_vector_type(2)));
        SELINV_GLOBAL v2 *q = (SELINV_GLOBAL v2 *)p;  // every array starts 256-byte aligned
        for (int64_t i = t; i < len / 2; i += n) q[i] = v2{0.0, 0.0};
        if (t == 0 && (len & 1)) gptr_w(p)[len - 1] = 0.0;
    };
    clear(diag, nd);
    clear(lpan, nl);
    clear(upan, nu);
}

hipError_t launch_clear_factors(double *diag, int64_t nd, double *lpan, int64_t nl, double *upan, int64_t nu,
                                int32_t *bad, hipStream_t st) {
    const int64_t blocks = std::min<int64_t>(2048, (std::max(nd, std::max(nl, nu)) / 2 + 255) / 256 + 1);
    hipLaunchKernelGGL(clear_factors_kernel, dim3((unsigned)blocks), dim3(256), 0, st, diag, nd, lpan, nl, upan, nu,
                       bad);
    return hipGetLastError();
}

hipError_t launch_scatter_values(const int64_t *loc, const double *vals, const int64_t *emb, int64_t nnz,
                                 double *diag, double *lpan, double *upan, hipStream_t st) {
    if (nnz <= 0) return hipSuccess;
    hipLaunchKernelGGL(scatter_values_kernel, dim3((unsigned)((nnz + 255) / 256)), dim3(256), 0, st, loc, vals, emb,
                       nnz, diag, lpan, upan);
    return hipGetLastError();
}

hipError_t launch_lu_tiles(const LuTile *items, int count, int32_t *bad, hipStream_t st) {
    if (count <= 0) return hipSuccess;
    hipLaunchKernelGGL(lu_tile_kernel, dim3(count), dim3(256), 0, st, items, bad);
    return hipGetLastError();
}

hipError_t launch_schur_scatter(const MatDev *mat, const GatherTile *tiles, int count, double *diag, double *lpan,
                                double *upan, hipStream_t st) {
    if (count <= 0) return hipSuccess;
    hipLaunchKernelGGL(schur_scatter_kernel, dim3(count), dim3(256), 0, st, mat, tiles, diag, lpan, upan);
    return hipGetLastError();
}

}  // namespace selinv
