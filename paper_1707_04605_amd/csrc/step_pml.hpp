// One leap-frog step with the split-field PML in one launch: the step of step_kernels.hpp with
// per-slice coefficient arrays, the layer's load, and the update of the layer's state q.
// Included by step.hip only.
//
// The update needs p_l and q_{l-1/2} alone, as the step does, and takes workgroups of the
// same launch.  Launches that short are bound by their latency: two of them took 10.7 us a
// step (321^2 nodes x 16 columns FP32), one takes 7.8; 1,001^2 x 32 100 and 98 us.
#pragma once

#include "step_kernels.hpp"

namespace mgrt {

template <typename T>
struct PmlArgs {
    // load of node rows: p+[node][:] += sum_{k = ptr[node]}^{ptr[node + 1] - 1} coef[k] * q[ent[k]][:]
    const int32_t *__restrict__ ptr;
    const int32_t *__restrict__ ent;
    const T *__restrict__ coef;
    const T *__restrict__ q;      // q_{l-1/2}
    // the launch's first `blocks` workgroups (a multiple of 8) form q_{l+1/2}
    const uint32_t *__restrict__ rec;
    T *__restrict__ qn;
    int64_t n_ent;
    int32_t nv;                   // nodes per element
    int32_t blocks;
};

// q_{l+1/2} = (1 - dt zeta) q_{l-1/2} + dt d_k p_l|_T for every listed element-direction; VEC
// columns per lane, LPN lanes per entry.  Each entry's record [its NV nodes, dt d_k phi_a|_T
// for the NV nodes, 1 - dt zeta] (values as 1 or 2 32-bit words) is contiguous, so a
// workgroup's records are one contiguous range: the lanes copy it to LDS one word each and
// read their entry's words from there.
template <typename T, int VEC, int LPN, int NV>
__device__ __forceinline__ void pml_update(const StepArgs<T> &a, const PmlArgs<T> &m, uint32_t *rec) {
    typedef typename VecT<T, VEC>::type V;
    constexpr int VW = sizeof(T) / 4;
    constexpr int MW = NV + (NV + 1) * VW;
    constexpr int64_t BW = VEC * LPN;
    constexpr int per_block = 256 / LPN;
    const int64_t e0 = (int64_t)blockIdx.x * per_block;
    const int words = (int)min((int64_t)per_block, m.n_ent - e0) * MW;
    for (int w = threadIdx.x; w < words; w += 256) rec[w] = m.rec[e0 * MW + w];
    __syncthreads();
    const int le = threadIdx.x / LPN;
    const int64_t e = e0 + le;
    if (e >= m.n_ent) return;
    const int64_t off = (int64_t)(threadIdx.x % LPN) * VEC;
    const uint32_t *r = rec + le * MW;
    auto value = [&](int k) -> T {
        if constexpr (VW == 1) return __uint_as_float(r[k]);
        else return __hiloint2double((int)r[k + 1], (int)r[k]);
    };
    V s = value(NV + NV * VW) * *reinterpret_cast<const V *>(m.q + e * BW + off);
#pragma unroll
    for (int k = 0; k < NV; ++k)
        s += value(NV + k * VW) * *reinterpret_cast<const V *>(a.p + (int64_t)r[k] * BW + off);
    // streamed out: the step reads q_{l+1/2} only in the next launch, and dirty lines left
    // in the XCDs' L2 caches would be written back at the kernel boundary
    __builtin_nontemporal_store(s, reinterpret_cast<V *>(m.qn + e * BW + off));
}

template <typename T, int VEC, int LPN, int W, bool NT>
__global__ __launch_bounds__(256) void k_step_pml(const StepArgs<T> a, const PmlArgs<T> m) {
    typedef typename VecT<T, VEC>::type V;
    constexpr int S = 256 / LPN;
    constexpr int64_t BW = VEC * LPN;
    __shared__ uint32_t rec[S * (4 + 5 * (int)(sizeof(T) / 4))];
    if ((int)blockIdx.x < m.blocks) {
        if (m.nv == 3) pml_update<T, VEC, LPN, 3>(a, m, rec);
        else pml_update<T, VEC, LPN, 4>(a, m, rec);
        return;
    }
    const int bid = (int)blockIdx.x - m.blocks;
    const int64_t tile = a.xcd_map ? (int64_t)(bid & 7) * a.per_xcd + (bid >> 3) : (int64_t)bid;
    if (tile >= a.n_tiles) return;
    const int ln = threadIdx.x / LPN, sub = threadIdx.x % LPN;
    const int64_t node = tile * S + ln;
    if (node >= a.n) return;
    // the layer row's bounds now: its gathers come last
    const int32_t k0 = m.ptr[node], k1 = m.ptr[node + 1];
    const int64_t off = node * BW + (int64_t)sub * VEC;
    const V pc = *reinterpret_cast<const V *>(a.p + off);
    V pv;
    if constexpr (NT) pv = __builtin_nontemporal_load(reinterpret_cast<const V *>(a.pm + off));
    else pv = *reinterpret_cast<const V *>(a.pm + off);
    V inc = a.beta[node] * (pc - pv);
    const int64_t sp = a.slice_ptr[tile] + ln;
    if constexpr (W > 0) {
        int c[W];
        T v[W];
        V pj[W];
#pragma unroll
        for (int k = 0; k < W; ++k) {
            c[k] = a.cols[sp + (int64_t)k * S];
            v[k] = a.vals[sp + (int64_t)k * S];
        }
#pragma unroll
        for (int k = 0; k < W; ++k)
            pj[k] = *reinterpret_cast<const V *>(a.p + (int64_t)c[k] * BW + (int64_t)sub * VEC);
#pragma unroll
        for (int k = 0; k < W; ++k) inc += v[k] * (pj[k] - pc);
    } else {
        const int w = a.slice_w[tile];
        for (int k = 0; k < w; ++k) {
            const int cj = a.cols[sp + (int64_t)k * S];
            inc += a.vals[sp + (int64_t)k * S] *
                   (*reinterpret_cast<const V *>(a.p + (int64_t)cj * BW + (int64_t)sub * VEC) - pc);
        }
    }
    // unrolled so that several entry -> q gather chains are in flight
#pragma unroll 4
    for (int32_t k = k0; k < k1; ++k)
        inc += m.coef[k] * *reinterpret_cast<const V *>(m.q + (int64_t)m.ent[k] * BW + (int64_t)sub * VEC);
    step_tail<T, VEC, LPN, NT>(a, tile, node, ln, sub, off, pc, inc);
}

namespace {

template <typename T, int VEC, int LPN, bool NT>
void launch_step_pml_w(const StepArgs<T> &a, const PmlArgs<T> &m, int W, int64_t grid, hipStream_t s) {
    auto go = [&](auto kern) { hipLaunchKernelGGL(kern, dim3(grid + m.blocks), dim3(256), 0, s, a, m); };
    switch (W) {
    case 4: go(k_step_pml<T, VEC, LPN, 4, NT>); break;
    case 6: go(k_step_pml<T, VEC, LPN, 6, NT>); break;
    case 8: go(k_step_pml<T, VEC, LPN, 8, NT>); break;
    case 12: go(k_step_pml<T, VEC, LPN, 12, NT>); break;
    case 16: go(k_step_pml<T, VEC, LPN, 16, NT>); break;
    default: go(k_step_pml<T, VEC, LPN, 0, NT>); break;
    }
}

// the batch widths of launch_step
template <typename T>
void launch_step_pml(const StepArgs<T> &a, const PmlArgs<T> &m, int B, int W, bool nt, int64_t grid, hipStream_t s) {
    constexpr int VEC = 16 / (int)sizeof(T);
    auto go = [&](auto vec, auto lpn) {
        constexpr int VE = decltype(vec)::value, LP = decltype(lpn)::value;
        MGRT_REQUIRE(a.B == VE * LP, MGRT_E_ARG, "row stride must equal the batch width");
        if (nt) launch_step_pml_w<T, VE, LP, true>(a, m, W, grid, s);
        else launch_step_pml_w<T, VE, LP, false>(a, m, W, grid, s);
    };
    const std::integral_constant<int, VEC> v;
    if (B == 1) return go(std::integral_constant<int, 1>{}, std::integral_constant<int, 1>{});
    switch (B / VEC) {
    case 1: return go(v, std::integral_constant<int, 1>{});
    case 2: return go(v, std::integral_constant<int, 2>{});
    case 4: return go(v, std::integral_constant<int, 4>{});
    case 8: return go(v, std::integral_constant<int, 8>{});
    case 16: return go(v, std::integral_constant<int, 16>{});
    case 32: return go(v, std::integral_constant<int, 32>{});
    case 64:
        if constexpr (sizeof(T) == 8) return go(v, std::integral_constant<int, 64>{});
        [[fallthrough]];
    default: throw Error(MGRT_E_ARG, "unsupported batch width");
    }
}

}  // namespace

}  // namespace mgrt
