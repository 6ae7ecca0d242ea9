// kernels.hip -- gfx950 kernels of supernodal selected inversion
// (arXiv:1708.04539, Algorithm 1).
//
//   tri_base_kernel  diagonal 64x64 sub-blocks of (L_KK)^{-1} and (U_KK)^{-1}
//                    in FP64 (step 2 / step 4 initialisation); the rest of the
//                    triangular inverses comes from GEMM rounds.
//   (the grouped MFMA GEMM of steps 2-5 lives in gemm.hip)
//   gather_kernel    G_K = A^{-T}(R_L(K), R_U(K)) from the diagonal blocks and
//                    panels of the ancestors (Theorem 1), one 64x64 tile per
//                    workgroup with the tile's index metadata staged in LDS;
//                    entries from U-side panels are read along their
//                    contiguous dimension and transposed through LDS.
//   extract_kernel   step 6: the selected entries, one per entry of A.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "device_types.hpp"
#include "kernels.hpp"
#include "tiles.hpp"
#include "tri.hpp"

namespace selinv {


// ---------------------------------------------------------------------------
// triangular inversion, diagonal 64x64 blocks
// ---------------------------------------------------------------------------
// One workgroup (4 wavefronts) inverts both triangles of the 64x64 (16 NB
// wide) diagonal sub-block that starts at row/column o of one supernode's packed
// L_KK \ U_KK (column-major, s x s; L unit lower, U upper).  A ragged
// sub-block (s - o < 64) is padded with the identity, whose inverse stays the
// identity and is not stored.  tri_invert (tri.hpp) leaves both results packed
// in one LDS tile; they are written out with coalesced stores,
// together with the zeros of L^{-1} above the sub-block and of U^{-1} left of
// it.  The off-diagonal 64x64 blocks of the inverses come from the GEMM rounds
// of the recursive doubling (X21 = -B^{-1} C A^{-1} for L,
// X12 = -A^{-1} C B^{-1} for U).
// NB = 4 handles every 64-wide sub-block; NB = 1 and 2 (16- and 32-wide
// blocks, far less LDS) serve the supernodes of at most 16 or 32 columns
// whose normalisation runs in the same workgroup.
// Bound by the latency of a chain of small steps (load, substitution, up to 40
// dependent MFMAs, stores), so by how many workgroups share a compute unit.
// With a second LDS tile for the factors and the staged panels (76 KB, two
// workgroups) the 5683 leaf blocks of 12 grids of side 64-256 took 288 us; in
// place and with the panels in registers (33 KB, 108 VGPRs, four) 154 us, and
// the two launches of the 2D 256^2 matrix 102 -> 69 us.

// Normalisation and diagonal initialisation of a supernode with s, c_L,
// c_U <= 64, after its inverses are complete in LDS (FP64 arithmetic on
// v_mfma_f64_16x16x4, results in the storage precision).  Every product is
// formed transposed (the MFMA takes the inverse as its first operand), so
// that a lane's results run down a column of the output and the stores are
// coalesced.  Wavefront w takes rows 16 w .. of the panels and reads them
// straight into its operand registers (16 rows of one column are 128
// consecutive bytes), the L panel before the inversion's rounds, so that the
// rounds hide its latency.
template <int NB>
struct TriPanel {
    double v[4 * NB];  // pan(16 w + lane % 16, 4 q + lane / 16)
    __device__ __forceinline__ void load(const double *pan, int rows, int s, int lane, int wave) {
        if (!pan || 16 * wave >= rows) return;
        const SELINV_GLOBAL double *P = gptr(pan);
        const int m = min(16 * wave + (lane & 15), rows - 1);
#pragma unroll
        for (int q = 0; q < 4 * NB; q++) v[q] = P[m + (int64_t)min(4 * q + (lane >> 4), s - 1) * rows];
    }
};

template <int NB>
__device__ __forceinline__ void tri_fused_epilogue(TriSmem<NB> &sm, const TriItem &it, TriPanel<NB> &lp, int lane,
                                                   int wave) {
    const int s = it.s, li = lane & 15, lk = lane >> 4;
    auto put = [&](void *out, int64_t idx, double v) {
        if (it.f32out == 2)
            gptr_w((uint32_t *)out)[idx] = stored<Pk32>(v);
        else if (it.f32out)
            gptr_w((float *)out)[idx] = (float)v;
        else
            gptr_w((double *)out)[idx] = v;
    };
    // panel products: out(m, n) = sum_k pan(m, k) inv(k, n), inv(k, n) =
    // Linv(k, n) (L side) or Uinv(n, k) (U side), zero for k < n
    auto panel = [&](const TriPanel<NB> &pan, int rows, void *out, auto UPPER_) {
        constexpr bool UPPER = decltype(UPPER_)::value;
        if (16 * wave >= rows) return;
        v4d acc[NB];
#pragma unroll
        for (int nb = 0; nb < NB; nb++) acc[nb] = v4d{0, 0, 0, 0};
#pragma unroll
        for (int q = 0; q < 4 * NB; q++) {
            if (4 * q >= s) break;
            const int k = 4 * q + lk;
            const double p = k < s ? pan.v[q] : 0.0;
#pragma unroll
            for (int nb = 0; nb < NB; nb++) {
                if (16 * nb > 4 * q + 3) continue;
                const int n = 16 * nb + li;
                acc[nb] = __builtin_amdgcn_mfma_f64_16x16x4f64(UPPER ? uinv_at(sm, n, k) : linv_at(sm, k, n), p,
                                                               acc[nb], 0, 0, 0);
            }
        }
        // acc[nb][v] = out(16 w + li, 16 nb + lk + 4 v)
        const int m = 16 * wave + li;
#pragma unroll
        for (int nb = 0; nb < NB; nb++)
#pragma unroll
            for (int v = 0; v < 4; v++) {
                const int n = 16 * nb + lk + 4 * v;
                if (m < rows && n < s) put(out, m + (int64_t)n * rows, acc[nb][v]);
            }
    };
    TriPanel<NB> up;
    up.load(it.upan, it.cu, s, lane, wave);
    if (it.lpan) panel(lp, it.cl, it.Lh, std::false_type{});
    if (it.upan) panel(up, it.cu, it.Uh, std::true_type{});
    // A^{-T}(K,K) := Linv^T Uinv^T:  Zd(m, n) = sum_k Linv(k, m) Uinv(n, k),
    // k >= max(m, n); wavefront w takes rows 16 w ..
    SELINV_GLOBAL double *Zd = gptr_w(it.Zd);
    if (wave < NB && 16 * wave < s) {
        const int m = 16 * wave + li;
        v4d acc[NB];
#pragma unroll
        for (int nb = 0; nb < NB; nb++) acc[nb] = v4d{0, 0, 0, 0};
        for (int kk = 16 * wave; kk < s; kk += 4) {
            const int k = kk + lk;
            const double l = linv_at(sm, k, m);
#pragma unroll
            for (int nb = 0; nb < NB; nb++)
                if (16 * nb <= kk + 3)
                    acc[nb] = __builtin_amdgcn_mfma_f64_16x16x4f64(uinv_at(sm, 16 * nb + li, k), l, acc[nb], 0, 0, 0);
        }
#pragma unroll
        for (int nb = 0; nb < NB; nb++)
#pragma unroll
            for (int v = 0; v < 4; v++) {
                const int n = 16 * nb + lk + 4 * v;
                if (m < s && n < s) Zd[m + (int64_t)n * s] = acc[nb][v];
            }
    }
}

template <int NB>
__device__ __forceinline__ void tri_base_item(const TriItem &it, TriSmem<NB> &sm) {
    constexpr int W = 16 * NB;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int s = it.s, o = it.j0, b = min(W, s - o);
    {
        // all loads of a thread in flight at once; addresses clamped into
        // the block, the identity padding selected afterwards
        constexpr int PER = W * W / 256 > 0 ? W * W / 256 : 1;
        double v[PER];
#pragma unroll
        for (int q = 0; q < PER; q++) {
            const int e = tid + 256 * q, r = e % W, c = e / W;
            v[q] = gptr(it.D)[(int64_t)(o + min(r, b - 1)) + (int64_t)(o + min(c, b - 1)) * s];
        }
#pragma unroll
        for (int q = 0; q < PER; q++) {
            const int e = tid + 256 * q, r = e % W, c = e / W;
            if (e >= W * W) continue;
            const double d = (r < b && c < b) ? v[q] : (r == c ? 1.0 : 0.0);
            sm.M[c][r] = d;
            if (r == c) sm.rd[c] = 1.0 / d;
        }
    }
    __syncthreads();
    TriPanel<NB> lp;
    if (it.fused) lp.load(it.lpan, it.cl, s, lane, wave);
    tri_invert<NB>(sm, lane, wave);
    __syncthreads();
    if (it.fused) {
        tri_fused_epilogue<NB>(sm, it, lp, lane, wave);
        return;
    }
    if constexpr (NB == 4) {
        SELINV_GLOBAL double *Linv = gptr_w(it.Linv), *Uinv = gptr_w(it.Uinv);
        {
            const int r = lane;
#pragma unroll
            for (int q = 0; q < 16; q++) {
                const int c = wave + 4 * q;
                if (r < b && c < b) {
                    const int64_t g = (int64_t)(o + r) + (int64_t)(o + c) * s;
                    Linv[g] = linv_at(sm, r, c);
                    Uinv[g] = uinv_at(sm, r, c);
                }
            }
        }
        // zeros of L^{-1} above the sub-block and of U^{-1} left of it
        for (int c = wave; c < b; c += 4)
            for (int r = lane; r < o; r += 64) Linv[r + (int64_t)(o + c) * s] = 0.0;
        if (lane < b)
            for (int c = wave; c < o; c += 4) Uinv[(o + lane) + (int64_t)c * s] = 0.0;
    }
}

// One item per workgroup.
template <int NB>
__global__ __launch_bounds__(256) void tri_base_kernel(const TriItem *__restrict__ items) {
    __shared__ TriSmem<NB> sm;
    tri_base_item<NB>(items[blockIdx.x], sm);
}

// Items [0, count), item b + q gridDim.x to workgroup b: a launch with fewer
// workgroups than items keeps at most that many resident (the side-stream
// inversion of the leaves, beside the level chain).  The item is a call: inlined into the
// loop, the item's per-lane LDS addresses are hoisted out of it and held
// across iterations, which more than triples the kernel's registers.
template <int NB>
__device__ __attribute__((noinline)) void tri_base_item_call(const TriItem *__restrict__ items, int b,
                                                             TriSmem<NB> &sm) {
    tri_base_item<NB>(items[b], sm);
}

template <int NB>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void tri_base_loop_kernel(const TriItem *__restrict__ items, int count) {
    __shared__ TriSmem<NB> sm;
    for (int b = blockIdx.x; b < count; b += gridDim.x) {
        tri_base_item_call<NB>(items, b, sm);
        __syncthreads();  // LDS free for the next item
    }
}

// ---------------------------------------------------------------------------
// gather
// ---------------------------------------------------------------------------
template <typename T, typename TG>
__global__ __launch_bounds__(256) void gather_kernel(const MatDev *__restrict__ mats,
                                                     const GatherTile *__restrict__ tiles) {
    __shared__ GatherSmem<T> sm;
    const GatherTile tl = tiles[blockIdx.x];
    gather_tile<T, TG>(mats[tl.mat], tl, sm);
}

// ---------------------------------------------------------------------------
// split-K reduction of the step-4 products
// ---------------------------------------------------------------------------
// blockIdx.y = item; each thread one entry of C; the partial products are
// added in a fixed order, so the result does not depend on the schedule.
__global__ __launch_bounds__(256) void splitk_reduce_kernel(const ReduceItem *__restrict__ items,
                                                            const MatDev *__restrict__ mats) {
    const ReduceItem it = items[blockIdx.y];
    const int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x, mn = (int64_t)it.M * it.N;
    if (e >= mn) return;
    const int m = (int)(e % it.M), n = (int)(e / it.M);
    // complex blocks: column n of the parts is column 2n of C, which gives
    // entry (m ^ 1, 2n + 1)
    const int nc = it.cpx ? 2 * n : n;
    SELINV_GLOBAL double *C = gptr_w(it.C) + m + (int64_t)nc * it.ldc;
    const SELINV_GLOBAL double *P = gptr(it.P) + e;
    double acc = *C;
    for (int p = 0; p < it.nparts; p++) acc += P[p * it.pstride];
    *C = acc;
    const double csign = (m & 1) ? -1.0 : 1.0;
    if (it.cpx) gptr_w(it.C)[(m ^ 1) + (int64_t)(nc + 1) * it.ldc] = csign * acc;
    if (it.push_sn < 0) return;
    // the final entry (m, n) of A^{-T}(P,P) into G_K of every child K of P
    // (the children's gathers skip these entries)
    const MatDev &Md = mats[it.push_mat];
    const SELINV_GLOBAL SnRec *sn = gptr(Md.sn);
    const SELINV_GLOBAL int32_t *kp = gptr(Md.kids_ptr);
    const SELINV_GLOBAL int32_t *kids = gptr(Md.kids);
    const int Pa = it.push_sn, sP = it.M;
    for (int q = kp[Pa]; q < kp[Pa + 1]; q++) {
        const int32_t K = kids[q];
        const SELINV_GLOBAL int32_t *posL = gptr(Md.push_pos) + gptr(Md.push_off)[K];
        for (int h = 0; h < (it.cpx ? 2 : 1); h++) {
            // h = 1: the odd-column entry that this one gives
            const int a = posL[h ? (m ^ 1) : m], b = posL[sP + nc + h];
            if (a < 0 || b < 0) continue;
            const double v = h ? csign * acc : acc;
            const int64_t g = sn[K].g_off + a + (int64_t)b * sn[K].cl;
            if (it.g_f32 == 2)
                gptr_w((uint32_t *)Md.G)[g] = stored<Pk32>(v);
            else if (it.g_f32)
                gptr_w((float *)Md.G)[g] = (float)v;
            else
                gptr_w((double *)Md.G)[g] = v;
        }
    }
}

// ---------------------------------------------------------------------------
// extraction
// ---------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(256) void extract_kernel(ExtractArgs a) {
    const int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (p >= a.nnz) return;
    const int64_t loc = gptr(a.loc)[p];
    const int64_t kind = loc >> 60, off = loc & ((int64_t(1) << 60) - 1);
    double v;
    if (kind == 0)
        v = gptr(a.Zd)[off];
    else if (kind == 1)
        v = (double)gptr((const T *)a.ZL)[off];
    else
        v = (double)gptr((const T *)a.ZU)[off];
    gptr_w(a.out)[p] = v;
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
hipError_t launch_tri_base(const TriItem *items, int count, int nb, hipStream_t st, int max_groups) {
    if (count <= 0) return hipSuccess;
    if (nb != 1 && nb != 2 && nb != 4) return hipErrorInvalidValue;
    if (max_groups > 0 && max_groups < count) {
        const dim3 g(max_groups);
        if (nb == 1)
            hipLaunchKernelGGL(tri_base_loop_kernel<1>, g, dim3(256), 0, st, items, count);
        else if (nb == 2)
            hipLaunchKernelGGL(tri_base_loop_kernel<2>, g, dim3(256), 0, st, items, count);
        else
            hipLaunchKernelGGL(tri_base_loop_kernel<4>, g, dim3(256), 0, st, items, count);
    } else if (nb == 1) {
        hipLaunchKernelGGL(tri_base_kernel<1>, dim3(count), dim3(256), 0, st, items);
    } else if (nb == 2) {
        hipLaunchKernelGGL(tri_base_kernel<2>, dim3(count), dim3(256), 0, st, items);
    } else {
        hipLaunchKernelGGL(tri_base_kernel<4>, dim3(count), dim3(256), 0, st, items);
    }
    return hipGetLastError();
}

hipError_t launch_gather(int mode, const MatDev *mats, const GatherTile *tiles, int ntiles, hipStream_t st) {
    if (ntiles <= 0) return hipSuccess;
    if (mode == CMP_F64)
        hipLaunchKernelGGL((gather_kernel<double, double>), dim3(ntiles), dim3(256), 0, st, mats, tiles);
    else if (mode == CMP_F32)
        hipLaunchKernelGGL((gather_kernel<float, float>), dim3(ntiles), dim3(256), 0, st, mats, tiles);
    else
        hipLaunchKernelGGL((gather_kernel<float, Pk32>), dim3(ntiles), dim3(256), 0, st, mats, tiles);
    return hipGetLastError();
}

hipError_t launch_splitk_reduce(const ReduceItem *items, int count, int64_t max_mn, const MatDev *mats,
                                hipStream_t st) {
    if (count <= 0 || max_mn <= 0) return hipSuccess;
    hipLaunchKernelGGL(splitk_reduce_kernel, dim3((unsigned)((max_mn + 255) / 256), count), dim3(256), 0, st, items,
                       mats);
    return hipGetLastError();
}

hipError_t launch_extract(int f64, const ExtractArgs &a, hipStream_t st) {
    if (a.nnz <= 0) return hipSuccess;
    const int64_t blocks = (a.nnz + 255) / 256;
    if (f64)
        hipLaunchKernelGGL(extract_kernel<double>, dim3((unsigned)blocks), dim3(256), 0, st, a);
    else
        hipLaunchKernelGGL(extract_kernel<float>, dim3((unsigned)blocks), dim3(256), 0, st, a);
    return hipGetLastError();
}

}  // namespace selinv
