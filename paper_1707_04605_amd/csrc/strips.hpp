// Several leap-frog steps per launch on lexicographic 2D grids: the streaming form of
// multistep.hip's launches for meshes whose every stiffness row couples a node only to
// its left, right, lower and upper neighbour (offsets -1, +1, -nx, +nx).  Included by
// multistep.hip only.
//
// One wave advances a strip of 64 nodes (a lane each, K of them halo on either side) by K
// steps, marching along y.  At row y it loads p_l of row y and p_{l-1} of row y - 1 and
// computes step m + 1 of row y - 1 - m for m = 0 .. K - 1: the three newest rows of every
// step stay in registers, the lower and upper neighbours are the wave's own rows, the left
// and right ones its neighbour lanes (DPP, folded into the subtraction).  There is no
// barrier and no state in LDS; the row's coefficients wait in a per-wave LDS ring of K
// rows.  The state is [group][node][VEC] as in multistep.hip, and so are the arithmetic
// and its order; a missing neighbour has coefficient 0 and a finite stand-in value.
#pragma once

#include "mgrt_internal.hpp"

namespace mgrt {

namespace {

template <typename T>
struct StripArgs {
    const T *p, *pm;
    T *out_p, *out_pm;
    const T *coef;                   // [n][4]: coefficients of nodes -nx, -1, +1, +nx (0: none)
    const T *beta;
    const int32_t *row_first;        // [ny]: 1 where a node of the row has no lower neighbour
    int32_t nx, ny, strips, chunks, groups, items, halo;
    int64_t n;
    const int32_t *ld_ptr, *ld_loc, *ld_col, *ld_sid;   // per (group, tile), loc = row * 64 + lane
    const double *ld_w;
    const int32_t *tp_ptr, *tp_loc, *tp_col, *tp_dst;
    const double *tp_w;
    const double *series;
    int64_t series_len, step0;
    double *parts;
    int64_t n_parts;
    int64_t *done;
    int32_t slot;
    const int32_t *hist_of;
    T *hist, *hist2;
    int64_t hist_nh, hist_b, hist_chunk;
    int32_t hist_mode;
    T inv_dt;
    T *vel_out;
    int64_t vel_step;
};

// the value of the lane below (D = -1) or above (D = +1); the wave's end lanes get 0
template <int D>
__device__ __forceinline__ float lane_next(float x) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), D < 0 ? 0x138 : 0x130, 0xF, 0xF, true));
}
template <int D>
__device__ __forceinline__ double lane_next(double x) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(x), D < 0 ? 0x138 : 0x130, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(x), D < 0 ? 0x138 : 0x130, 0xF, 0xF, true);
    return __hiloint2double(hi, lo);
}

// EXT: 1 the run records node histories, 2 the velocity field, 0 neither
template <typename T, int VEC, int K, int EXT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void k_strips(
    const StripArgs<T> a) {
    typedef typename GroupVec<T, VEC>::type V;
    constexpr int R = K <= 1 ? 1 : K <= 2 ? 2 : K <= 4 ? 4 : K <= 6 ? 6 : 8;
    // loads of the steps: FP32 in LDS, FP64 in registers (two waves a SIMD leave 20 KB a wave)
    constexpr bool LDS_ADD = sizeof(T) == 4;
    __shared__ T cf[4][R][5][64];
    __shared__ int32_t hr[EXT == 1 ? 4 : 1][R][64];
    __shared__ T adds[LDS_ADD ? 4 : 1][LDS_ADD ? K : 1][BL_CAP], tapv[4][K][BL_CAP];    // tapv: values of the taps
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int64_t l0 = a.done[a.slot];
    if (blockIdx.x == 0 && threadIdx.x == 0) a.done[a.slot ^ 1] = l0 + K;
    const int nwg = gridDim.x;
    const int rank = (blockIdx.x & 7) * (nwg >> 3) + min((int)blockIdx.x & 7, nwg & 7) + (blockIdx.x >> 3);
    const int item = __builtin_amdgcn_readfirstlane(rank * 4 + wave);
    if (item >= a.items) return;
    const int t = item / a.groups, g = item - t * a.groups;
    const int cy = t / a.strips, sx = t - cy * a.strips;
    const int ya = (int)((int64_t)a.ny * cy / a.chunks), yb = (int)((int64_t)a.ny * (cy + 1) / a.chunks);
    const int xa = (int)((int64_t)a.nx * sx / a.strips), xb = (int)((int64_t)a.nx * (sx + 1) / a.strips);
    const int x = xa - K + lane, xc = min(max(x, 0), a.nx - 1);
    const bool xin = x == xc, xown = x >= xa && x < xb;
    const int64_t go = (int64_t)g * a.n;
    const V *gp = reinterpret_cast<const V *>(a.p) + go, *gq = reinterpret_cast<const V *>(a.pm) + go;
    V *op = reinterpret_cast<V *>(a.out_p) + go, *om = reinterpret_cast<V *>(a.out_pm) + go;
    const int64_t li = (int64_t)g * a.strips * a.chunks + t;
    const int lb = a.ld_ptr[li], nl = a.ld_ptr[li + 1] - lb;
    const int qb = a.tp_ptr[li], nq = a.tp_ptr[li + 1] - qb;

    // buffer addressing: a load's row is a scalar offset, the lane's part a constant register, and
    // a store past the buffer's end is dropped, so the loads and stores of an iteration have
    // no branches around them and the waits for a row loaded PD iterations ago count exactly.
    // Stores have no scalar offset: a store of 16 bytes per lane reads its data registers over
    // several cycles, and the compiler keeps the next write of them off only for stores without
    // one (with one, lanes 12 to 15 of every 16 got the next value now and then).
    constexpr int OOB = (int)0x80000000;
    const int rowb = a.nx * 16, bytes = (int)(a.n * 16);
    const auto rp = __builtin_amdgcn_make_buffer_rsrc((void *)gp, 0, bytes, 0x00027000);
    const auto rq = __builtin_amdgcn_make_buffer_rsrc((void *)gq, 0, bytes, 0x00027000);
    const auto rop = __builtin_amdgcn_make_buffer_rsrc((void *)op, 0, bytes, 0x00027000);
    const auto rom = __builtin_amdgcn_make_buffer_rsrc((void *)om, 0, bytes, 0x00027000);
    const int vin = xc * 16, vown = xown ? xc * 16 : OOB;
    const T *cx = a.coef + (int64_t)xc * 4, *bx = a.beta + xc;

    constexpr int PD = 3;
    V L[K][3], m1, n0[PD], n1[PD];
    typedef T C4 __attribute__((ext_vector_type(4)));
    C4 nc[PD];
    T nb[PD];
    int nh[PD] = {};
    // lane e holds entry e of the lists: a hit costs a ballot and lane reads, no memory access
    // (list positions are relative to the plan's halo; outside this launch's: -1)
    const int sh = a.halo - K;
    auto place = [&](int loc) { return (loc & 63) < sh || loc >> 6 < sh ? -1 : loc - sh * 65; };
    int lloc = -1, lcol = 0, tloc = -1, tcol = 0;
    double lw = 0.0;
    T add_of[LDS_ADD ? 1 : K] = {};
    if (lane < nl) {
        lloc = place(a.ld_loc[lb + lane]);
        lcol = a.ld_col[lb + lane];
        const double w = a.ld_w[lb + lane];
        const double *ser = a.series + (int64_t)a.ld_sid[lb + lane] * a.series_len + a.step0 + l0;
#pragma unroll
        for (int m = 0; m < K; ++m) load_value(w, ser[m], LDS_ADD ? adds[wave][m][lane] : add_of[LDS_ADD ? 0 : m]);
        lw = w;
    }
    if (lane < nq) {
        tloc = place(a.tp_loc[qb + lane]);
        tcol = a.tp_col[qb + lane];
    }
#pragma unroll
    for (int m = 0; m < K; ++m)
#pragma unroll
        for (int q = 0; q < 3; ++q)
#pragma unroll
            for (int u = 0; u < VEC; ++u) L[m][q][u] = T(0);
#pragma unroll
    for (int u = 0; u < VEC; ++u) m1[u] = T(0);
    // rows of this item, bit m: row i - 1 - m carries loads / taps / histories
    uint32_t lrows = 0, trows = 0, hrows = 0;
    // Histories: the values of an iteration's first such row (coarse nodes lie 2^L rows apart,
    // so there is hardly a second) leave with the iteration's other stores, unconditionally
    // (OOB where there is none): with stores in branches of the levels the waits for fetched
    // rows count those too, and a 64-bit remainder per row took its time (513^2 nodes x 32
    // FP32 columns, coarse nodes 8 apart: 81.7 -> 68.6 us per launch of 8 steps).
    // A launch's steps lie in one chunk of the stage.
    const int64_t hrow = EXT == 1 ? a.hist_nh * a.hist_b : 0;
    const int64_t hb = EXT == 1 ? l0 % a.hist_chunk * hrow : 0;
    T *const h1 = a.hist + hb, *const h2 = a.hist_mode == 2 ? a.hist2 + hb : nullptr;
    T *const vel0 = EXT == 2 ? a.vel_out + l0 * a.vel_step + go * VEC : nullptr;
    V hout, hvel;
#pragma unroll
    for (int u = 0; u < VEC; ++u) hout[u] = hvel[u] = T(0);
    auto fetch = [&](auto qc, int i) {
        constexpr int Q = decltype(qc)::value;
        const int y = ya - K + i, yc = min(max(y, 0), a.ny - 1);
        n0[Q] = __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b128(rp, vin, yc * rowb, 0));
        n1[Q] = __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b128(rq, vin, yc * rowb, 0));
        const int64_t rn = (int64_t)yc * a.nx;
        nc[Q] = *reinterpret_cast<const C4 *>(cx + rn * 4);
        nb[Q] = bx[rn];
        if constexpr (EXT == 1) nh[Q] = a.hist_of[rn + xc];
    };
    const int nit = yb - ya + 2 * K;
    int ifirst = 0;             // iterations up to the last that may see a row of row_first
    for (int r = lane; r < nit; r += 64) {
        const int y = ya - K + r;
        if (y >= 0 && y < a.ny && a.row_first[y]) ifirst = r + K + 1;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) ifirst = max(ifirst, __shfl_xor(ifirst, o));
    ifirst = __builtin_amdgcn_readfirstlane(ifirst);
    // in this order: the waits of the loop count the loads behind the one they wait for
    fetch(std::integral_constant<int, 0>{}, 0);
    __builtin_amdgcn_sched_barrier(0);
    fetch(std::integral_constant<int, 1>{}, 1);
    __builtin_amdgcn_sched_barrier(0);
    fetch(std::integral_constant<int, 2>{}, 2);
    __builtin_amdgcn_sched_barrier(0);
    // FIRST: rows with nodes without a lower neighbour may be among the iteration's; their
    // first term is the next neighbour there is, as in the one-step kernel's padded rows
    auto iter = [&](auto qc, auto first, int i) {
        constexpr bool FIRST = decltype(first)::value;
        constexpr int Q = decltype(qc)::value, QP = (Q + 2) % 3, QO = (Q + 1) % 3;
        const int y = ya - K + i;
        const bool in = xin && y >= 0 && y < a.ny;
        // copies with registers of their own: the fetched row's registers stay the target of
        // the next fetch (else the compiler moves rows still in flight, and waits for them)
        V m1n;
#pragma unroll
        for (int u = 0; u < VEC; ++u) {
            T x0 = n0[Q][u], x1 = n1[Q][u];
            asm volatile("" : "+v"(x0), "+v"(x1));
            L[0][Q][u] = x0;
            m1n[u] = x1;
        }
        T cw[5];
#pragma unroll
        for (int q = 0; q < 4; ++q) cw[q] = in ? nc[Q][q] : T(0);
        cw[4] = in ? nb[Q] : T(0);
#pragma unroll
        for (int q = 0; q < 5; ++q) asm volatile("" : "+v"(cw[q]));
        const int hw = EXT == 1 && xown && y >= ya && y < yb ? nh[Q] : -1;
        fetch(qc, i + PD);
        V last = m1, lastc = m1;
        int hat = OOB;
        [[maybe_unused]] const int hm = __ffs((int)hrows & ((1 << K) - 1)) - 1;
        // a level's coefficients are read one level ahead of their use
        T cv[2][5];
        auto coef = [&](int m) {
#pragma unroll
            for (int q = 0; q < 5; ++q) cv[m & 1][q] = cf[wave][(uint32_t)(i - 1 - m) % R][q][lane];
        };
        coef(0);
#pragma unroll
        for (int m = 0; m < K; ++m) {
            // row r = y - 1 - m, step m + 1; the first rows of a chunk are still incomplete
            if (i < 2 * m + 2) break;
            const int rr = i - 1 - m;
            [[maybe_unused]] const int slot = (uint32_t)rr % R;
            if (m + 1 < K) coef(m + 1);
            __builtin_amdgcn_sched_barrier(0);
            const V c = L[m][QP], dn = L[m][QO], up = L[m][Q];
            const V o = m == 0 ? m1 : L[m > 0 ? m - 1 : 0][QO];
            const T v0 = cv[m & 1][0], v1 = cv[m & 1][1], v2 = cv[m & 1][2], v3 = cv[m & 1][3], be = cv[m & 1][4];
            V inc;
            if constexpr (FIRST) {
                const bool z0 = v0 == T(0), f1 = z0 && v1 != T(0), f2 = z0 && !f1 && v2 != T(0), f3 = z0 && !f1 && !f2;
                const T vf = f1 ? v1 : f2 ? v2 : f3 ? v3 : v0;
                const T w1 = f1 ? T(0) : v1, w2 = f2 ? T(0) : v2, w3 = f3 ? T(0) : v3;
#pragma unroll
                for (int u = 0; u < VEC; ++u) {
                    const T l = lane_next<-1>(c[u]) - c[u], r = lane_next<1>(c[u]) - c[u], w = up[u] - c[u];
                    T e = dn[u] - c[u];
                    e = f1 ? l : e;
                    e = f2 ? r : e;
                    e = f3 ? w : e;
                    inc[u] = fma(w3, w, fma(w2, r, fma(w1, l, first_terms(be, c[u] - o[u], vf, e))));
                }
            } else {
#pragma unroll
                for (int u = 0; u < VEC; ++u) {
                    T s = first_terms(be, c[u] - o[u], v0, dn[u] - c[u]);
                    s = fma(v1, lane_next<-1>(c[u]) - c[u], s);
                    s = fma(v2, lane_next<1>(c[u]) - c[u], s);
                    inc[u] = fma(v3, up[u] - c[u], s);
                }
            }
            if (lrows & (1u << m)) {
                for (uint64_t b = __ballot(lloc >> 6 == rr); b; b &= b - 1) {
                    const int e = __ffsll((unsigned long long)b) - 1;
                    T add;
                    if constexpr (LDS_ADD) add = adds[wave][m][e];
                    else add = __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(add_of[m]), e),
                                                __builtin_amdgcn_readlane(__double2loint(add_of[m]), e));
                    const double w = __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(lw), e),
                                                      __builtin_amdgcn_readlane(__double2loint(lw), e));
                    const int at = __builtin_amdgcn_readlane(lloc, e) & 63, col = __builtin_amdgcn_readlane(lcol, e);
#pragma unroll
                    for (int u = 0; u < VEC; ++u)
                        if (col == u && lane == at) inc[u] = add_load(inc[u], w, add);
                }
            }
            const V out = c + inc;
            if (trows & (1u << m)) {
                for (uint64_t b = __ballot(tloc >> 6 == rr); b; b &= b - 1) {
                    const int e = __ffsll((unsigned long long)b) - 1;
                    const int at = __builtin_amdgcn_readlane(tloc, e) & 63, col = __builtin_amdgcn_readlane(tcol, e);
                    T val = out[0];
#pragma unroll
                    for (int u = 1; u < VEC; ++u)
                        if (col == u) val = out[u];
                    if (lane == at) tapv[wave][m][e] = val;
                }
            }
            if constexpr (EXT == 1) {
                if (hrows & (1u << m)) {
                    const int hx = hr[wave][slot][lane];
                    const V vel = -inc * a.inv_dt;
                    if (m == hm) {
                        hat = hx >= 0 ? (hx * (int)a.hist_b + g * VEC) * (int)sizeof(T) : OOB;
                        hout = a.hist_mode == 1 ? vel : out;
                        hvel = vel;
                    } else if (hx >= 0) {
                        const int64_t ho = m * hrow + hx * a.hist_b + (int64_t)g * VEC;
                        *reinterpret_cast<V *>(h1 + ho) = a.hist_mode == 1 ? vel : out;
                        if (h2) *reinterpret_cast<V *>(h2 + ho) = vel;
                    }
                }
            }
            if constexpr (EXT == 2) {
                typedef unsigned int U4 __attribute__((ext_vector_type(4)));
                T *vp = vel0 + m * a.vel_step;
                asm volatile("" : "+s"(vp));        // made here: K descriptors kept would spill
                const auto rv = __builtin_amdgcn_make_buffer_rsrc((void *)vp, 0, bytes, 0x00027000);
                const int vo = rr >= K && rr < nit - K ? vown + (ya - K + rr) * rowb : OOB;
                __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(U4, -inc * a.inv_dt), rv, vo, 0, 2);
            }
            if (m + 1 < K) {
                L[m + 1 < K ? m + 1 : 0][Q] = out;
            } else {
                last = out;
                lastc = c;
            }
        }
        {   // row y - K, one of the chunk's own from iteration 2 K on
            typedef unsigned int U4 __attribute__((ext_vector_type(4)));
            const int vo = i < 2 * K || i >= nit ? OOB : vown + (y - K) * rowb;
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(U4, last), rop, vo, 0, 0);
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(U4, lastc), rom, vo, 0, 0);
            if constexpr (EXT == 1) {
                const int64_t hs = max(hm, 0) * hrow;
                const auto r1 = __builtin_amdgcn_make_buffer_rsrc((void *)(h1 + hs), 0, 0x7ffffff0, 0x00027000);
                const auto r2 = __builtin_amdgcn_make_buffer_rsrc((void *)(h2 ? h2 + hs : h1), 0, 0x7ffffff0, 0x00027000);
                __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(U4, hout), r1, hat, 0, 0);
                __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(U4, hvel), r2, h2 ? hat : OOB, 0, 0);
            }
        }
        // row y's coefficients: first used by the next iteration
#pragma unroll
        for (int q = 0; q < 5; ++q) cf[wave][(uint32_t)i % R][q][lane] = cw[q];
        m1 = m1n;
        lrows = lrows << 1 | (uint32_t)(__ballot(lloc >> 6 == i) != 0);
        trows = trows << 1 | (uint32_t)(__ballot(tloc >> 6 == i) != 0);
        if constexpr (EXT == 1) {
            hr[wave][(uint32_t)i % R][lane] = hw;
            hrows = hrows << 1 | (uint32_t)(__ballot(hw >= 0) != 0);
        }
    };
    int i = 0;
    for (; i < ifirst; i += 3) {
        iter(std::integral_constant<int, 0>{}, std::true_type{}, i);
        iter(std::integral_constant<int, 1>{}, std::true_type{}, i + 1);
        iter(std::integral_constant<int, 2>{}, std::true_type{}, i + 2);
    }
    for (; i < nit; i += 3) {                   // up to two iterations past the end store nothing
        iter(std::integral_constant<int, 0>{}, std::false_type{}, i);
        iter(std::integral_constant<int, 1>{}, std::false_type{}, i + 1);
        iter(std::integral_constant<int, 2>{}, std::false_type{}, i + 2);
    }
    if (lane < nq) {
        const double w = a.tp_w[qb + lane];
        double *dst = a.parts + l0 * a.n_parts + a.tp_dst[qb + lane];
#pragma unroll
        for (int m = 0; m < K; ++m) dst[m * a.n_parts] = w * (double)tapv[wave][m][lane];
    }
}

// coef[node][slot] from the operator's slices (S = 1 << log_s rows, width W)
template <typename T>
__global__ __launch_bounds__(256) void k_strip_coef(const int32_t *__restrict__ cols, const T *__restrict__ vals,
                                                    int64_t n, int log_s, int W, int nx, T *__restrict__ coef,
                                                    int32_t *__restrict__ row_first) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    T v[4] = {T(0), T(0), T(0), T(0)};
    const int64_t sp = ((i >> log_s) * W << log_s) + (i & ((1 << log_s) - 1));
    for (int w = 0; w < W; ++w) {
        const int64_t d = cols[sp + ((int64_t)w << log_s)] - i;
        const T c = vals[sp + ((int64_t)w << log_s)];
        if (d == -nx) v[0] = c;
        else if (d == -1) v[1] = c;
        else if (d == 1) v[2] = c;
        else if (d == nx) v[3] = c;
    }
    for (int q = 0; q < 4; ++q) coef[i * 4 + q] = v[q];
    if (v[0] == T(0)) row_first[i / nx] = 1;         // every writer writes 1
}

}  // namespace

}  // namespace mgrt
