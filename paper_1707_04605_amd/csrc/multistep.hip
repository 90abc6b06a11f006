// Several leap-frog steps per launch (App. A eqs. leap-frog1/2 in the nodal three-level
// form of the one-step launches, step.hip).
//
// A one-step launch reads p_l and p_{l-1} and writes p_{l+1}, three words of HBM traffic
// per node, column and step, and pays one launch per step.  Here the nodes are cut into
// compact tiles (coordinate bisection).  A workgroup takes its tile and every node within
// graph distance k of it (the k-ring in the stiffness graph), advances them k steps out of
// registers and LDS, and writes the tile's two newest levels to the other buffer pair:
// four words per node and column and one launch per k steps.  A node at distance d from
// the tile is exact after k - d steps, so sub-step s updates the nodes within distance
// k - 1 - s; neighbouring tiles recompute their shared rings instead of exchanging them.
// Every node update is the one-step launch's, term by term: the increment
// beta (p_l - p_{l-1}) + sum_j c_ij (p_{l,j} - p_{l,i}) over the row's padded entries in
// the same order, the nodal loads in list order, then taps, histories and correlation.
//
// Layout: VEC columns (16 bytes, or one column on small problems) form a group; the state
// of a run is [group][node][VEC].  A thread owns up to NPT entries of the region and keeps
// p_l, p_{l-1}, beta, the row's coefficients and neighbour slots (16 bits) in registers for
// the whole launch; only p_l goes through LDS, in two buffers, so a sub-step is W 16-byte
// LDS reads, one write and one barrier.  The entries of a region are ordered by distance
// (tile first), so whole waves drop out as the rings shrink.
#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdlib>
#include <memory>
#include <new>
#include <thread>
#include <vector>

#include "mgrt_internal.hpp"

namespace mgrt {

// Tiles and regions of one mesh (stepping order): topology only, kept with the mesh.
struct Blocks {
    int k = 0, W = 0, vec = 1, npt = 1, threads = 0, rmax = 0;
    int64_t n_tiles = 0;
    int64_t n_ent = 0;   // entries of all regions, each padded to threads * npt
    double ratio = 0;    // region entries per node
    DevBuf cnt;      // int32 [n_tiles][64]: entries of the tile within distance d
    DevBuf node;     // int32 per entry: stepping-order node (padding: the tile's first)
    DevBuf nbr;      // uint32 [W/2][n_ent]: LDS byte offsets of the row's neighbours, in pairs
    // on the host: each node's tile, the tiles' entries and how many lie within each distance
    std::vector<int32_t> tile_of, h_cnt;             // h_cnt [n_tiles][k + 1]
    std::vector<std::vector<int32_t>> ents;
    // strips instead of regions (strips.hpp): nx > 0, tiles are strips x chunks of rows
    int64_t nx = 0, ny = 0, strips = 0, chunks = 0;

    // where a region updates a node
    struct Place {
        int32_t tile, loc;
    };
    // places of the nodes that carried loads so far; place_at[node]: where, or -1
    std::vector<std::vector<Place>> places;
    std::vector<int32_t> place_at, seen;             // seen[node]: the last search that met it
    int32_t searches = 0;

    // node ii among the entries at distance d of tile t (ascending)
    Place place(int32_t ii, int32_t t, int d) const {
        const int32_t *ct = &h_cnt[(size_t)t * (k + 1)];
        const auto e = ents[t].begin();
        return Place{t, (int32_t)(std::lower_bound(e + (d ? ct[d - 1] : 0), e + ct[d], ii) - e)};
    }

    // A tile updates the nodes within distance k - 1 of it, so the tiles that update node ii are
    // those of the nodes within distance k - 1 of ii.
    const std::vector<Place> &places_of(const HostMesh &hm, int32_t ii) {
        if (place_at[ii] >= 0) return places[place_at[ii]];
        std::vector<int32_t> ball{ii}, tiles;
        std::vector<Place> out;
        seen[ii] = ++searches;
        size_t f0 = 0;
        for (int d = 0; d < (n_tiles == 1 ? 1 : k); ++d) {
            const size_t f1 = ball.size();
            for (size_t f = f0; f < f1; ++f) {
                const int32_t t = tile_of[ball[f]];
                if (std::find(tiles.begin(), tiles.end(), t) == tiles.end()) {
                    tiles.push_back(t);
                    out.push_back(place(ii, t, d));
                }
                const int64_t i = hm.perm[ball[f]];
                for (int64_t q = hm.krow[i]; q < hm.krow[i + 1]; ++q) {
                    const int32_t jj = hm.iperm[hm.kcol[q]];
                    if (seen[jj] == searches) continue;
                    seen[jj] = searches;
                    ball.push_back(jj);
                }
            }
            f0 = f1;
        }
        places.push_back(std::move(out));
        place_at[ii] = (int32_t)places.size() - 1;
        return places.back();
    }

    // f(tile, local entry) for every tile that updates node ii, or for the node's own alone
    template <typename F>
    void each_tile(const HostMesh &hm, int32_t ii, bool own, F &&f) {
        if (nx == 0) {
            if (own) {
                const Place q = place(ii, tile_of[ii], 0);
                f((int64_t)q.tile, q.loc);
            } else {
                for (const Place &q : places_of(hm, ii)) f((int64_t)q.tile, q.loc);
            }
            return;
        }
        // chunks of rows and strips about the node
        const int64_t x = ii % nx, y = ii / nx;
        const int64_t c0 = std::max<int64_t>(0, std::max<int64_t>(0, y - k) * chunks / ny - 1);
        const int64_t c1 = std::min(chunks, (y + k) * chunks / ny + 2);
        const int64_t s0 = std::max<int64_t>(0, std::max<int64_t>(0, x + k - 64) * strips / nx - 1);
        const int64_t s1 = std::min(strips, (x + k) * strips / nx + 2);
        for (int64_t cy = c0; cy < c1; ++cy) {
            const int64_t ya = ny * cy / chunks, yb = ny * (cy + 1) / chunks;
            if (own ? y < ya || y >= yb : y < ya - k || y >= yb + k) continue;
            for (int64_t sx = s0; sx < s1; ++sx) {
                const int64_t xa = nx * sx / strips, xb = nx * (sx + 1) / strips;
                if (own ? x < xa || x >= xb : x < xa - k || x >= xa - k + 64) continue;
                f(cy * strips + sx, (int32_t)((y - ya + k) * 64 + (x - xa + k)));
            }
        }
    }
};

namespace {

constexpr int BL_FIELD = 32768;   // bytes of a p buffer, at most
// steps per launch of strips: FP64's coefficient rings of 8 rows leave a SIMD one wave, of 6
// two (513^2 nodes x 30 columns: 16.2 -> 12.9 us a step)
template <typename T>
constexpr int STRIP_K = sizeof(T) == 4 ? 8 : 6;
constexpr int BL_CAP = 64;        // nodal loads / taps per tile and group (held in LDS)
// Runs of several columns take one launch per step below this many steps: building the
// regions costs about as much as a hundred one-step launches, once per mesh and shape.
constexpr int64_t BL_MIN_STEPS = 256;

template <typename T, int VEC>
struct GroupVec {
    typedef T type __attribute__((ext_vector_type(VEC)));
};

// The one-step kernel's arithmetic, as the compiler contracts it there, so that runs of
// either kind give the same values bit for bit: beta d + v e, d = p_l - p_{l-1}, e the first
// neighbour's difference, rounds v e and fuses beta d; a nodal load's product w g is rounded
// to FP32 (load_value) and fused into an FP64 sum (add_load).
template <typename T>
__device__ __forceinline__ T first_terms(T be, T d, T v, T e) {
    return fma(be, d, v * e);
}
__device__ __forceinline__ void load_value(double w, double g, float &out) { out = (float)(w * g); }
__device__ __forceinline__ void load_value(double, double g, double &out) { out = g; }
__device__ __forceinline__ float add_load(float inc, double, float v) { return inc + v; }
__device__ __forceinline__ double add_load(double inc, double w, double v) { return fma(w, v, inc); }

}  // namespace

}  // namespace mgrt

#include "strips.hpp"

namespace mgrt {

namespace {

int padded_width(int wmax) {
    for (int w : {4, 6, 8, 12, 16})
        if (wmax <= w) return w;
    return 0;
}

template <typename T>
struct BlockArgs {
    const T *p, *pm;                 // p_l, p_{l-1}: [group][node][VEC]
    T *out_p, *out_pm;               // p_{l+k}, p_{l+k-1}
    const int32_t *cnt, *node;
    const uint32_t *nbr;
    const T *beta, *vals;            // per node; SELL slices of S = 1 << log_s rows, width W
    int64_t n, n_ent;
    int32_t n_tiles, log_s, ksteps, groups;
    int32_t beta_first;              // round beta d and fuse the first neighbour's product
    // nodal loads and receiver taps per (group, tile)
    const int32_t *ld_ptr, *ld_loc, *ld_col, *ld_sid;
    const double *ld_w;
    const int32_t *tp_ptr, *tp_loc, *tp_col, *tp_dst;
    const double *tp_w;
    const double *series;
    int64_t series_len, step0;
    double *parts;
    int64_t n_parts;
    // steps done: a launch reads done[slot] and leaves done[slot ^ 1] for the next one, so
    // replayed launches need no arguments of their own
    int64_t *done;
    int32_t slot;
    // coarse-node histories (as StepArgs): hist_of[node] = history index or -1
    const int32_t *hist_of;
    T *hist, *hist2;
    int64_t hist_nh, hist_b, hist_chunk;
    int32_t hist_mode;
    T inv_dt;
    // full velocity out, zero-lag correlation with a stored velocity: [step][group][node][VEC]
    T *vel_out;
    const T *vel;
    int64_t vel_step, vel_first;     // elements per step (negative: read backwards), step 0
    double *acc;                     // [group][node]
};

// What bounds it: on large meshes HBM traffic (16 B (1 + region / tile) / 2 k per group
// entry) and the VALU (11 operations per column and update) together; on small ones the
// chain of LDS reads and barriers of a sub-step.
//
// A workgroup takes a contiguous range of the (tile, group) items, tile-major: the tables
// of a tile are loaded once for its groups.
template <typename T, int VEC, int W, int NPT, bool EXT>
__global__ __launch_bounds__(1024) void k_blocks(const BlockArgs<T> a) {
    typedef typename GroupVec<T, VEC>::type V;
    extern __shared__ __align__(16) unsigned char sm[];
    const int tid = threadIdx.x, TH = blockDim.x, RP = TH * NPT;
    double *tw = reinterpret_cast<double *>(sm + (size_t)2 * RP * sizeof(V)), *lw = tw + BL_CAP;
    int32_t *tloc = reinterpret_cast<int32_t *>(lw + BL_CAP), *tcol = tloc + BL_CAP, *tdst = tcol + BL_CAP;
    int32_t *lloc = tdst + BL_CAP, *lcol = lloc + BL_CAP;
    T *adds = reinterpret_cast<T *>(lcol + BL_CAP);              // [k][BL_CAP]
    const int64_t l0 = a.done[a.slot];
    const int ks = a.ksteps;
    // a launch's steps lie in one chunk of the history stage
    [[maybe_unused]] const int64_t hist_l0 = EXT && a.hist_of ? l0 % a.hist_chunk : 0;
    if (blockIdx.x == 0 && tid == 0) a.done[a.slot ^ 1] = l0 + ks;
    // item ranges in XCD order: consecutive workgroups go to different XCDs
    const int nwg = gridDim.x;
    const int rank = (blockIdx.x & 7) * (nwg >> 3) + min((int)blockIdx.x & 7, nwg & 7) + (blockIdx.x >> 3);
    const int64_t items = (int64_t)a.n_tiles * a.groups;
    const int i0 = (int)(items * rank / nwg), i1 = (int)(items * (rank + 1) / nwg);
    const int wave0 = __builtin_amdgcn_readfirstlane(tid & ~63);
    int cnt = 0, ntile = 0, nact = 0, tcur = -1;
    int nid[NPT], hx[NPT];
    T be[NPT], v[NPT][W];
    uint32_t nb[NPT][W / 2];
    V pc[NPT], pv[NPT];
    for (int it = i0; it < i1; ++it) {
        const int t = it / a.groups, g = it - t * a.groups;
        if (t != tcur) {
            tcur = t;
            const int64_t r0 = (int64_t)t * RP;
            // lane d holds the entries within distance d
            cnt = a.cnt[(int64_t)t * 64 + (tid & 63)];
#pragma unroll
            for (int j = 0; j < NPT; ++j) nid[j] = a.node[r0 + tid + j * TH];
            ntile = __builtin_amdgcn_readlane(cnt, 0);
            nact = __builtin_amdgcn_readlane(cnt, ks - 1);
#pragma unroll
            for (int j = 0; j < NPT; ++j) {
                const int e = tid + j * TH;
#pragma unroll
                for (int w = 0; w < W / 2; ++w) nb[j][w] = a.nbr[(int64_t)w * a.n_ent + r0 + e];
                be[j] = a.beta[nid[j]];
                const int64_t sp = ((int64_t)(nid[j] >> a.log_s) * W << a.log_s) + (nid[j] & ((1 << a.log_s) - 1));
#pragma unroll
                for (int w = 0; w < W; ++w) v[j][w] = a.vals[sp + ((int64_t)w << a.log_s)];
                hx[j] = -1;
                if constexpr (EXT)
                    if (a.hist_of && e < ntile) hx[j] = a.hist_of[nid[j]];
            }
        }
        const int64_t go = (int64_t)g * a.n;
        const V *gp = reinterpret_cast<const V *>(a.p) + go, *gq = reinterpret_cast<const V *>(a.pm) + go;
#pragma unroll
        for (int j = 0; j < NPT; ++j) {
            pc[j] = gp[nid[j]];
            if (wave0 + j * TH < nact) pv[j] = gq[nid[j]];
        }
        const int64_t li = (int64_t)g * a.n_tiles + t;
        const int lb = a.ld_ptr[li], nl = a.ld_ptr[li + 1] - lb;
        const int qb = a.tp_ptr[li], nq = a.tp_ptr[li + 1] - qb;
        if (nl > 0) {
            if (tid < nl) {
                lloc[tid] = a.ld_loc[lb + tid];
                lcol[tid] = a.ld_col[lb + tid];
                lw[tid] = a.ld_w[lb + tid];
            }
            // the launch's loads: thread x takes list entry x % 64 of steps x / 64, ...
            const int i = tid & 63;
            if (i < nl) {
                const double w = a.ld_w[lb + i];
                const double *ser = a.series + (int64_t)a.ld_sid[lb + i] * a.series_len + a.step0 + l0;
                for (int q = tid >> 6; q < ks; q += TH >> 6) load_value(w, ser[q], adds[q * BL_CAP + i]);
            }
        }
        if (tid < nq) {
            tloc[tid] = a.tp_loc[qb + tid];
            tcol[tid] = a.tp_col[qb + tid];
            tdst[tid] = a.tp_dst[qb + tid];
            tw[tid] = a.tp_w[qb + tid];
        }
#pragma unroll
        for (int j = 0; j < NPT; ++j) reinterpret_cast<V *>(sm)[tid + j * TH] = pc[j];
        __syncthreads();
        // this thread's entries that carry loads (bit j) or taps (bit 4 + j), whether more
        // than one list entry does (bits 8, 9), and the first of each: a walk over the lists
        // costs LDS round trips on the sub-steps' chain
        uint32_t mk = 0;
        for (int i = 0; i < nl; ++i)
#pragma unroll
            for (int j = 0; j < NPT; ++j)
                if (lloc[i] - tid == j * TH) mk |= (mk & 15u ? 1u << 8 : (uint32_t)i << 10 | (uint32_t)lcol[i] << 16) | 1u << j;
        for (int i = 0; i < nq; ++i)
#pragma unroll
            for (int j = 0; j < NPT; ++j)
                if (tloc[i] - tid == j * TH) mk |= (mk & 240u ? 1u << 9 : (uint32_t)i << 18 | (uint32_t)tcol[i] << 24) | 16u << j;
        double acc[NPT];
#pragma unroll
        for (int j = 0; j < NPT; ++j) acc[j] = 0.0;
        // step s: o (p_{l-1}) becomes p_{l+1}; lanes past the active entries of a wave
        // compute values that nothing reads
        auto substep = [&](int s, V(&c)[NPT], V(&o)[NPT], const unsigned char *rd, unsigned char *wr) {
            const int act = __builtin_amdgcn_readlane(cnt, ks - 1 - s);
            const T *ad = adds + s * BL_CAP;
            T add0 = T(0);
            double tw0 = 0.0, lw0 = 0.0;
            int td0 = 0;
            if (mk) {
                add0 = ad[mk >> 10 & 63];
                if (sizeof(T) == 8) lw0 = lw[mk >> 10 & 63];
                tw0 = tw[mk >> 18 & 63];
                td0 = tdst[mk >> 18 & 63];
            }
#pragma unroll
            for (int j = 0; j < NPT; ++j) {
                if (wave0 + j * TH >= act) continue;
                const int e = tid + j * TH;
                V pj[W];
#pragma unroll
                for (int w = 0; w < W / 2; ++w) {
                    uint32_t q = nb[j][w];
                    asm volatile("" : "+v"(q));    // unpacked here: kept unpacked it takes W registers
                    pj[2 * w] = *reinterpret_cast<const V *>(rd + (q & 0xffffu));
                    pj[2 * w + 1] = *reinterpret_cast<const V *>(rd + (q >> 16));
                }
                V vv;
                bool corr = false;
                if constexpr (EXT) {
                    corr = a.acc && e < ntile;
                    if (corr)
                        vv = *reinterpret_cast<const V *>(a.vel + a.vel_first + (l0 + s) * a.vel_step +
                                                          (go + nid[j]) * VEC);
                }
                // column by column: a coefficient stays one scalar register (a vector
                // product would keep a copy of it per column across the loop)
                V inc;
#pragma unroll
                for (int u = 0; u < VEC; ++u) {
                    const T d = c[j][u] - o[j][u], e0 = pj[0][u] - c[j][u];
                    T x = first_terms(be[j], d, v[j][0], e0);
                    if constexpr (VEC == 1) {
                        const T y = fma(v[j][0], e0, be[j] * d);
                        x = a.beta_first ? y : x;
                    }
#pragma unroll
                    for (int w = 1; w < W; ++w) x = fma(v[j][w], pj[w][u] - c[j][u], x);
                    inc[u] = x;
                }
                if (mk & (1u << j)) {
                    if (!(mk & 256u)) {
#pragma unroll
                        for (int u = 0; u < VEC; ++u)
                            if ((int)(mk >> 16 & 3) == u) inc[u] = add_load(inc[u], lw0, add0);
                    } else {
                        for (int i = 0; i < nl; ++i)
                            if (lloc[i] == e) {
                                const T add = ad[i];
#pragma unroll
                                for (int u = 0; u < VEC; ++u)
                                    if (lcol[i] == u) inc[u] = add_load(inc[u], lw[i], add);
                            }
                    }
                }
                const V out = c[j] + inc;
                *reinterpret_cast<V *>(wr + e * (int)sizeof(V)) = out;
                o[j] = out;
                if (mk & (16u << j)) {
                    double *row = a.parts + (l0 + s) * a.n_parts;
                    auto pick = [&](int col) {
                        T val = out[0];
#pragma unroll
                        for (int u = 1; u < VEC; ++u)
                            if (col == u) val = out[u];
                        return (double)val;
                    };
                    if (!(mk & 512u)) {
                        row[td0] = tw0 * pick((int)(mk >> 24 & 3));
                    } else {
                        for (int i = 0; i < nq; ++i)
                            if (tloc[i] == e) row[tdst[i]] = tw[i] * pick(tcol[i]);
                    }
                }
                if constexpr (EXT) {
                    if (hx[j] >= 0) {
                        const int64_t ho = ((hist_l0 + s) * a.hist_nh + hx[j]) * a.hist_b + (int64_t)g * VEC;
                        const V vel = -inc * a.inv_dt;
                        *reinterpret_cast<V *>(a.hist + ho) = a.hist_mode == 1 ? vel : out;
                        if (a.hist_mode == 2) *reinterpret_cast<V *>(a.hist2 + ho) = vel;
                    }
                    if (corr) {
                        double sum = 0.0;
#pragma unroll
                        for (int u = 0; u < VEC; ++u) sum += (double)out[u] * (double)vv[u];
                        acc[j] += sum;
                    }
                    if (a.vel_out && e < ntile)
                        __builtin_nontemporal_store(-inc * a.inv_dt,
                                                    reinterpret_cast<V *>(a.vel_out + (l0 + s) * a.vel_step +
                                                                          (go + nid[j]) * VEC));
                }
            }
            __syncthreads();
        };
        int s = 0;
        for (; s + 1 < ks; s += 2) {
            substep(s, pc, pv, sm, sm + RP * (int)sizeof(V));
            substep(s + 1, pv, pc, sm + RP * (int)sizeof(V), sm);
        }
        V *op = reinterpret_cast<V *>(a.out_p) + go, *om = reinterpret_cast<V *>(a.out_pm) + go;
        if (s < ks) {
            substep(s, pc, pv, sm, sm + RP * (int)sizeof(V));
            V *x = op;
            op = om;
            om = x;
        }
#pragma unroll
        for (int j = 0; j < NPT; ++j)
            if (tid + j * TH < ntile) {
                op[nid[j]] = pc[j];
                om[nid[j]] = pv[j];
                if constexpr (EXT)
                    if (a.acc) a.acc[go + nid[j]] += acc[j];
            }
    }
}

// acc[i] += sum over the planes, in order
__global__ __launch_bounds__(256) void k_add_planes(const double *__restrict__ pl, int64_t planes, int64_t n,
                                                    double *__restrict__ acc) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    double s = 0.0;
    for (int64_t y = 0; y < planes; ++y) s += pl[y * n + i];
    acc[i] += s;
}

size_t block_lds(int entries, int vec, int k, size_t esz) {
    return (size_t)2 * entries * vec * esz + (size_t)BL_CAP * (2 * 8 + 5 * 4) + (size_t)k * BL_CAP * esz;
}

// How a run launches: ksteps == 0 sets the kernel's LDS limit and asks how many workgroups
// a CU holds instead of launching.
struct BlockLaunch {
    int W, npt, threads;
    bool ext;
    size_t lds;
    int64_t grid;
    int per_cu;
    hipStream_t s;
};

template <typename T, int VEC, int W, int NPT>
void launch_blocks_x(const BlockArgs<T> &a, BlockLaunch &L) {
    auto go = [&](auto kern) {
        if (a.ksteps == 0) {
            MGRT_HIP(hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)L.lds));
            MGRT_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&L.per_cu, (const void *)kern, L.threads, L.lds));
        } else {
            hipLaunchKernelGGL(kern, dim3((unsigned)L.grid), dim3(L.threads), L.lds, L.s, a);
        }
    };
    if (L.ext) go(k_blocks<T, VEC, W, NPT, true>);
    else go(k_blocks<T, VEC, W, NPT, false>);
}

// Entries per thread that the kernel's registers allow without spills
template <typename T, int VEC>
constexpr int max_npt(int W) {
    return W == 4 ? 4 : W == 6 ? (VEC == 1 || sizeof(T) == 4 ? 4 : 2) : W == 8 ? 2 : 1;
}
int max_npt(int prec, int vec, int W) {
    return prec == 32 ? (vec == 1 ? max_npt<float, 1>(W) : max_npt<float, 4>(W))
                      : (vec == 1 ? max_npt<double, 1>(W) : max_npt<double, 2>(W));
}

template <typename T, int VEC, int W>
void launch_blocks_w(const BlockArgs<T> &a, BlockLaunch &L) {
    if (L.npt == 1) return launch_blocks_x<T, VEC, W, 1>(a, L);
    if constexpr (max_npt<T, VEC>(W) >= 2)
        if (L.npt == 2) return launch_blocks_x<T, VEC, W, 2>(a, L);
    if constexpr (max_npt<T, VEC>(W) >= 4)
        if (L.npt == 4) return launch_blocks_x<T, VEC, W, 4>(a, L);
    throw Error(MGRT_E_STATE, "unsupported region shape");
}

template <typename T, int VEC>
void launch_blocks(const BlockArgs<T> &a, BlockLaunch &L) {
    switch (L.W) {
    case 4: return launch_blocks_w<T, VEC, 4>(a, L);
    case 6: return launch_blocks_w<T, VEC, 6>(a, L);
    case 8: return launch_blocks_w<T, VEC, 8>(a, L);
    case 12: return launch_blocks_w<T, VEC, 12>(a, L);
    default: return launch_blocks_w<T, VEC, 16>(a, L);
    }
}

// Entries of a region of s nodes with k rings of the nearest-neighbour stencil of a square
// or cubic tile (a start for the tile size; the built regions decide).
double region_estimate(int d, double s, int k) {
    if (d == 2) return s + 4.0 * k * std::sqrt(s) * 1.03 + 2.0 * k * (k - 1);
    const double a = std::cbrt(s) * 1.02;
    double r = s;
    for (int q = 1; q <= k; ++q) r += 6 * a * a + 12.0 * a * (q - 1) + 4.0 * (q - 1) * (q - 2);
    return r;
}

// A node on the host: its coordinates beside its id, so that a cut reads its keys in a row.
template <int D>
struct NodeAt {
    double x[D];
    int32_t ii;
};

// Cut nodes[lo, hi) into nt tiles of nearly equal size by bisection along the longest side;
// ties on that coordinate are ordered by the others and the node id, so that a cut through
// a grid line leaves one step in it.  first[t0 + t] is where tile t of them starts.
template <int D>
void bisect(NodeAt<D> *nodes, int64_t lo, int64_t hi, int64_t nt, int64_t t0, int64_t *first, int depth) {
    if (nt == 1) {
        first[t0] = lo;
        return;
    }
    double mn[D], mx[D];
    for (int a = 0; a < D; ++a) mn[a] = mx[a] = nodes[lo].x[a];
    for (int64_t i = lo; i < hi; ++i)
        for (int a = 0; a < D; ++a) {
            mn[a] = std::min(mn[a], nodes[i].x[a]);
            mx[a] = std::max(mx[a], nodes[i].x[a]);
        }
    int ax = D - 1;
    for (int a = D - 2; a >= 0; --a)
        if (mx[a] - mn[a] > 1.0001 * (mx[ax] - mn[ax])) ax = a;
    const int64_t nl = nt / 2, mid = lo + (hi - lo) * nl / nt;
    std::nth_element(nodes + lo, nodes + mid, nodes + hi, [ax](const NodeAt<D> &p, const NodeAt<D> &q) {
        for (int b = 0; b < D; ++b) {
            const int a = ax + b < D ? ax + b : ax + b - D;
            if (p.x[a] != q.x[a]) return p.x[a] < q.x[a];
        }
        return p.ii < q.ii;
    });
    std::thread half;
    if (depth < 4 && hi - lo > 2048) {
        try {
            half = std::thread([=] { bisect<D>(nodes, lo, mid, nl, t0, first, depth + 1); });
        } catch (...) {       // no thread to be had: this one does both
        }
    }
    if (!half.joinable()) bisect<D>(nodes, lo, mid, nl, t0, first, depth + 1);
    bisect<D>(nodes, mid, hi, nt - nl, t0 + nl, first, depth + 1);
    if (half.joinable()) half.join();
}

// The tiles' nodes, tile by tile, and where each tile starts.
template <int D>
void cut_tiles(const HostMesh &hm, int64_t n_tiles, std::vector<int32_t> &idx, std::vector<int64_t> &first) {
    const int64_t n = hm.n;
    const std::unique_ptr<NodeAt<D>[]> nodes(new NodeAt<D>[n]);
    parallel_for(n, [&](int64_t i0, int64_t i1) {
        for (int64_t i = i0; i < i1; ++i) {
            for (int a = 0; a < D; ++a) nodes[i].x[a] = hm.coords[(int64_t)hm.perm[i] * D + a];
            nodes[i].ii = (int32_t)i;
        }
    }, 16384);
    first.assign(n_tiles + 1, n);
    bisect<D>(nodes.get(), 0, n, n_tiles, 0, first.data(), 0);
    idx.resize(n);
    parallel_for(n, [&](int64_t i0, int64_t i1) {
        for (int64_t i = i0; i < i1; ++i) idx[i] = nodes[i].ii;
    }, 65536);
}

// The last region that met a node (its tile + 1, 0: none) and the node's entry there; zero pages
// of the allocation that no region of the thread touches are never made.
struct Mark {
    int32_t tile, loc;
};
struct FreeHost {
    void operator()(void *p) const { std::free(p); }
};

// Regions of n_tiles tiles and k steps: per tile the entries by distance, ascending within
// a distance.  Returns null when a region has more than cap entries.  The first run of a mesh
// and shape waits for this (eight cores, a node table per thread, every node's tiles listed and
// tile numbers tried that did not fit: 301^2 nodes 13 ms, 1,025^2 204; as here 4.6 and 37).
std::shared_ptr<Blocks> build_blocks(Ctx &c, int W, int64_t n_tiles, int k, int cap, int npt_max, int entry_bytes,
                                     int c_esz) {
    const HostMesh &hm = c.hm;
    const int64_t n = hm.n;
    std::vector<int32_t> idx;
    std::vector<int64_t> first;
    if (hm.d == 2) cut_tiles<2>(hm, n_tiles, idx, first);
    else cut_tiles<3>(hm, n_tiles, idx, first);
    auto B = std::make_shared<Blocks>();
    B->k = k;
    B->W = W;
    B->n_tiles = n_tiles;
    B->tile_of.resize(n);
    B->place_at.assign(n, -1);
    B->seen.assign(n, 0);
    B->h_cnt.assign((size_t)n_tiles * (k + 1), 0);
    B->ents.resize(n_tiles);
    std::vector<std::vector<uint16_t>> nbs(n_tiles);       // [entry][W]: LDS byte offsets
    std::atomic<int> bad{0};
    // a thread costs as much as some 2,000 entries
    const int64_t grain = std::max<int64_t>(
        {1, n_tiles / 16, (int64_t)(2048 / std::min<double>(n, region_estimate(hm.d, (double)n / n_tiles, k)))});
    parallel_for(n_tiles, [&](int64_t a0, int64_t a1) {
        try {
            const std::unique_ptr<Mark[], FreeHost> marks(static_cast<Mark *>(std::calloc(n, sizeof(Mark))));
            if (!marks) throw std::bad_alloc();
            Mark *at = marks.get();
            for (int64_t t = a0; t < a1 && !bad; ++t) {
                const int32_t me = (int32_t)t + 1;
                auto &E = B->ents[t];
                int32_t *ct = &B->h_cnt[(size_t)t * (k + 1)];
                E.reserve(std::min<int64_t>(cap + 64, 4 * (first[t + 1] - first[t]) + 256));
                E.assign(idx.begin() + first[t], idx.begin() + first[t + 1]);
                std::sort(E.begin(), E.end());
                for (int32_t ii : E) {
                    at[ii].tile = me;
                    B->tile_of[ii] = (int32_t)t;
                }
                ct[0] = (int32_t)E.size();
                size_t f0 = 0;
                for (int d = 1; d <= k && (int64_t)E.size() <= cap; ++d) {
                    const size_t f1 = E.size();
                    for (size_t f = f0; f < f1; ++f) {
                        const int64_t i = hm.perm[E[f]];
                        for (int64_t q = hm.krow[i]; q < hm.krow[i + 1]; ++q) {
                            const int32_t jj = hm.iperm[hm.kcol[q]];
                            if (at[jj].tile == me) continue;
                            at[jj].tile = me;
                            E.push_back(jj);
                        }
                    }
                    std::sort(E.begin() + f1, E.end());
                    f0 = f1;
                    ct[d] = (int32_t)E.size();
                }
                if ((int64_t)E.size() > cap) {
                    bad = 1;
                    return;
                }
                for (size_t e = 0; e < E.size(); ++e) at[E[e]].loc = (int32_t)e;
                auto &N = nbs[t];
                N.resize(E.size() * W);
                for (size_t e = 0; e < E.size(); ++e) {
                    // entries at distance k are never updated; padding: the own slot
                    const int64_t i = hm.perm[E[e]], q0 = hm.krow[i];
                    const int len = (int)e < ct[k - 1] ? (int)(hm.krow[i + 1] - q0) : 0;
                    for (int w = 0; w < W; ++w)
                        N[e * W + w] = (uint16_t)((w < len ? at[hm.iperm[hm.kcol[q0 + w]]].loc : (int)e) * entry_bytes);
                }
            }
        } catch (...) {
            bad = 2;
        }
    }, grain);
    if (bad == 2) throw Error(MGRT_E_OOM_PLAN, "host allocation failed");
    if (bad) return nullptr;
    int64_t tot = 0;
    for (int64_t t = 0; t < n_tiles; ++t) {
        B->rmax = std::max(B->rmax, (int)B->ents[t].size());
        tot += (int64_t)B->ents[t].size();
    }
    B->ratio = (double)tot / n;
    // 1,024 lanes a workgroup, but 512 (two workgroups a CU) for the large regions of four FP32
    // columns: 250^2 nodes x 16 columns 2.34 us per step against 2.75, while 150^2 x 16 (smaller
    // regions) takes 1.33 us at 1,024 against 1.47
    const int lanes = entry_bytes == 16 && c_esz == 4 && B->rmax > 1536 ? 512 : 1024;
    while (B->rmax > lanes * B->npt && B->npt < npt_max) B->npt *= 2;
    B->threads = ((B->rmax + B->npt - 1) / B->npt + 63) / 64 * 64;
    const int64_t rp = (int64_t)B->threads * B->npt, ne = B->n_ent = n_tiles * rp;
    if (ne >= (int64_t)1 << 31) return nullptr;
    const int W2 = W / 2;
    const std::unique_ptr<int32_t[]> node(new int32_t[ne]), cnt64(new int32_t[n_tiles * 64]);
    const std::unique_ptr<uint32_t[]> nbr(new uint32_t[(size_t)ne * W2]);
    parallel_for(n_tiles, [&](int64_t a0, int64_t a1) {
        for (int64_t t = a0; t < a1; ++t) {
            const auto &E = B->ents[t];
            const int64_t ec = (int64_t)E.size();
            for (int d = 0; d < 64; ++d) cnt64[t * 64 + d] = B->h_cnt[(size_t)t * (k + 1) + std::min(d, k)];
            for (int64_t e = 0; e < rp; ++e) node[t * rp + e] = E[e < ec ? e : 0];
            for (int w = 0; w < W2; ++w) {
                uint32_t *dst = nbr.get() + (size_t)w * ne + t * rp;
                const uint16_t *src = nbs[t].data() + 2 * w;
                for (int64_t e = 0; e < ec; ++e) dst[e] = src[e * W] | (uint32_t)src[e * W + 1] << 16;
                std::fill(dst + ec, dst + rp, 0u);
            }
        }
    }, std::max<int64_t>(grain, 65536 / rp));
    B->cnt = upload(cnt64.get(), n_tiles * 64, c.stream);
    B->node = upload(node.get(), ne, c.stream);
    B->nbr = upload(nbr.get(), ne * W2, c.stream);
    return B;
}

// Row length nx of a 2D mesh whose stepping order is a lexicographic grid and whose
// stiffness rows couple node i to i - nx, i - 1, i + 1, i + nx only, in that order and
// without wrapping around a row's ends; else 0.
int64_t grid_row(const HostMesh &hm) {
    if (hm.d != 2) return 0;
    int64_t nx = 0;
    for (int64_t q = hm.krow[hm.perm[0]]; q < hm.krow[hm.perm[0] + 1]; ++q)
        nx = std::max<int64_t>(nx, hm.iperm[hm.kcol[q]]);
    if (nx < 2 || hm.n % nx != 0 || hm.n / nx < 2) return 0;
    std::atomic<int> bad{0};
    parallel_for(hm.n, [&](int64_t a0, int64_t a1) {
        for (int64_t ii = a0; ii < a1 && !bad; ++ii) {
            const int64_t i = hm.perm[ii], x = ii % nx;
            int64_t last = -nx - 1;
            for (int64_t q = hm.krow[i]; q < hm.krow[i + 1]; ++q) {
                const int64_t d = hm.iperm[hm.kcol[q]] - ii;
                const bool ok = d == -nx || d == nx || (d == -1 && x > 0) || (d == 1 && x + 1 < nx);
                if (!ok || d <= last) bad = 1;
                last = d;
            }
        }
    }, 65536);
    return bad ? 0 : nx;
}

// Cost of a launch of strips in row iterations of a SIMD: chunks of rows per strip are waves,
// `slots` of them resident on the chip; a SIMD steps r resident waves in r iterations' time
// (one alone takes 1.35: its LDS waits are exposed).  The rows a chunk shares with its
// neighbours (2 k) count 0.8, their first levels are skipped.
double strip_cost(int64_t waves, int64_t slots, double rows, int k) {
    const int64_t full = waves / slots, rem = waves % slots;
    const double r = (double)slots / 1024;
    return (full * std::max(r, 1.35) + (rem ? std::max(std::ceil(rem / 1024.0), 1.35) : 0.0)) * (rows + 1.6 * k);
}

}  // namespace

// The shape of a run's launches, by measurement on MI355X (us per step, one launch per step
// first):
//  - up to 2,048 nodes in 2D (4,096 in 3D) and several columns: the whole mesh is one tile, a
//    workgroup steps a column 64 steps (33^2 nodes, 3 columns, FP64: 3.9 -> 0.61)
//  - one column a group while n * columns <= 131,072 (97^2 nodes: 4 columns 0.90 with one
//    column a group, 16 columns 1.29, and 1.19 with four)
//  - 2D grids: regions while the tiles of one round of workgroups (256) hold the mesh, strips
//    beyond; the two estimates below cross near n * groups = 10^6 (251^2 nodes x 64 FP32
//    columns 5.9 either way; 513^2 x 32: regions 9.2, strips 7.7)
//  - k = 12 where a tile holds up to 200 nodes (65^2 x 4: 0.80, k = 8 0.90) and for one
//    column (129^2: 0.64, k = 8 0.89), else 8.  One-column runs on fewer than 2,048 nodes stay
//    at 8, the bound that mgrt_timing.steps_per_launch has had there.
//  - one column on more than 65,536 nodes, whose values are the same either way: not before the
//    mesh's runs together repay the tables (first call, one step a launch and these, ms: 301^2
//    nodes, 200 steps 7.3 and 4.7; 513^2, 200 7.5 and 8.8, 4,000 19.3 and 14.0; 701^2, 1,000 15.6
//    and 19.8, 4,000 25.4 and 24.4; 1,025^2, 4,000 50 and 59; 8 steps on 301^2 1.8 and 4.6)
//  - 3D and wide rows: a tile's rings outgrow it, so only small problems, up to 100,000 words
//    of state per field (18^3 nodes: 1 column 3.9 -> 1.7, 16 FP32 columns 3.8 -> 2.7; 34^3 x 16
//    loses, 4.3 -> 7.6), with k = 4, above 60,000 words 3
Blocks *plan_blocks(Ctx &c, int prec, const StepOp &op, int64_t n_cols, int B, int64_t n_steps,
                    const mgrt_run_opts *opts, bool corr) {
    const HostMesh &hm = c.hm;
    const int64_t n = hm.n;
    const int flags = opts ? opts->flags : 0;
    // a requested launch variant or batch width (above one column) selects the one-step
    // launches it describes
    if ((flags & MGRT_F_ONE_STEP) || (opts && (opts->launch != 0 || (opts->batch != 0 && B > 1)))) return nullptr;
    const int W = padded_width(op.wmax);
    if (c.have_pml || n_cols < 1 || n >= (1 << 27) || W == 0 || n_steps < 8) return nullptr;
    if (n_cols > 1 && n_steps < BL_MIN_STEPS) return nullptr;
    const int esz = prec / 8;
    int vec = n * n_cols <= 131072 || B == 1 ? 1 : 16 / esz;
    int k = 8;
    int64_t tiles = 1, G = 0;
    // tables hold columns in groups of vec and entries of vec * esz bytes: FP32 in fours and FP64
    // in pairs have the same bytes and are not the same tables
    auto lookup = [&](bool strip, int64_t a, auto &&build) -> Blocks * {
        const auto key = std::make_tuple(strip, prec, vec, W, a, k);
        auto it = c.blocks.find(key);
        if (it == c.blocks.end()) {
            if (B == 1 && n > ONE_COLUMN_NODES) {
                c.one_col_steps += n_steps;
                if (c.one_col_steps < 64 || n > 140000 + 100 * c.one_col_steps) return nullptr;
            }
            it = c.blocks.emplace(key, build()).first;
        }
        return it->second->k ? it->second.get() : nullptr;
    };
    const int64_t one_tile = hm.d == 2 ? 2048 : 4096;
    if (n_cols > 1 && n <= std::min<int64_t>(one_tile, 1024 * max_npt(prec, 1, W))) {
        vec = 1;
        k = 64;
    } else {
        G = (n_cols + vec - 1) / vec;
        if (hm.d == 3 || W > 4) {
            const int64_t words = n * n_cols * (esz / 4);
            if (words > 100000) return nullptr;
            k = hm.d == 2 ? 8 : words <= 60000 ? 4 : 3;
        } else {
            if (vec > 1 && !corr) {
                if (c.grid_nx < 0) c.grid_nx = grid_row(hm);
                if (c.grid_nx > 0) {
                    const int kr = k;
                    k = esz == 4 ? STRIP_K<float> : STRIP_K<double>;
                    const int64_t strips = (c.grid_nx + 64 - 2 * k - 1) / (64 - 2 * k), ny = n / c.grid_nx;
                    const int64_t slots = 2048;          // 57 and 74 KB of LDS per four waves
                    double best = 1e300;
                    int64_t chunks = 1;
                    for (int64_t ch = 1; ch <= std::max<int64_t>(1, ny / 4); ++ch) {
                        const double cost = strip_cost(strips * G * ch, slots, (double)ny / ch, k);
                        if (cost < 0.999 * best) {
                            best = cost;
                            chunks = ch;
                        }
                    }
                    const double us_strips = ((esz == 4 ? 0.82 : 0.69) * best + 6.0) / k;
                    const double us_regions = (esz == 4 ? 4.5e-6 : 5.5e-6) * n * G + 1.0;
                    if (us_strips < us_regions)
                        return lookup(true, G, [&] {
                            auto b = std::make_shared<Blocks>();
                            b->k = k;
                            b->W = W;
                            b->vec = vec;
                            b->nx = c.grid_nx;
                            b->ny = ny;
                            b->strips = strips;
                            b->chunks = chunks;
                            b->n_tiles = strips * chunks;
                            return b;
                        });
                    k = kr;
                }
            }
            if (n_cols == 1 ? n >= 2048 : n * G <= 200 * 256) k = 12;
        }
        tiles = std::max<int64_t>(1, std::min(256 / G, n / 16));
    }
    const int npt_max = max_npt(prec, vec, W);
    const int cap = std::min(BL_FIELD / (vec * esz), 1024 * npt_max);
    // tiles whose regions fit by the estimate times f
    auto fit = [&](double f) {
        double s = (double)n / tiles;
        while (f * region_estimate(hm.d, s, k) > cap && s > 1) s *= 0.98;
        return std::max<int64_t>(1, (int64_t)std::ceil(n / s));
    };
    // where the wished number does not fit, regions are up to a tenth larger than the estimate
    if (k < 64 && region_estimate(hm.d, (double)n / tiles, k) > cap) tiles = fit(1.1);
    return lookup(false, tiles, [&] {
        std::shared_ptr<Blocks> b;
        int64_t tl = tiles;
        for (int tries = 0; tries < 8 && !b && n / tl >= 4; ++tries) {
            b = build_blocks(c, W, tl, k, cap, npt_max, vec * esz, esz);
            tl = std::max(k < 64 ? fit(1.1) : 1, tl + tl / 16 + 1);
        }
        if (!b) b = std::make_shared<Blocks>();      // k = 0: no such regions
        b->vec = vec;
        return b;
    });
}

namespace {

struct GroupLists {
    std::vector<int32_t> ptr, loc, col, aux;
    std::vector<double> w;
    bool fits = true;
};

// Entries by (group, tile) in the given order; own: only the node's own tile (taps).  Lists that
// overflow by the nodes' own tiles alone are given up before any other tile is looked for.
template <typename Ent, typename AuxFn>
GroupLists group_lists(Blocks &B, int64_t groups, const std::vector<Ent> &ents, const HostMesh &hm, bool own,
                       AuxFn aux) {
    GroupLists L;
    auto each = [&](bool own_tile, auto &&f) {
        for (const auto &e : ents)
            B.each_tile(hm, hm.iperm[e.node], own_tile, [&](int64_t tile, int32_t loc) {
                f(e, (int64_t)(e.col / B.vec) * B.n_tiles + tile, loc);
            });
    };
    auto count = [&](bool own_tile) {
        L.ptr.assign(groups * B.n_tiles + 1, 0);
        each(own_tile, [&](const Ent &, int64_t li, int32_t) {
            if (++L.ptr[li + 1] > BL_CAP) L.fits = false;
        });
    };
    count(true);
    if (L.fits && !own) count(false);
    if (!L.fits) return L;
    for (size_t i = 0; i + 1 < L.ptr.size(); ++i) L.ptr[i + 1] += L.ptr[i];
    const size_t ne = std::max<size_t>(1, L.ptr.back());
    L.loc.assign(ne, 0);
    L.col.assign(ne, 0);
    L.aux.assign(ne, 0);
    L.w.assign(ne, 0.0);
    std::vector<int32_t> fill(L.ptr.begin(), L.ptr.end() - 1);
    each(own, [&](const Ent &e, int64_t li, int32_t loc) {
        const int32_t q = fill[li]++;
        L.loc[q] = loc;
        L.col[q] = e.col % B.vec;
        L.aux[q] = aux(e);
        L.w[q] = e.weight;
    });
    return L;
}

int64_t live_groups(const BatchRun &run, int vec) {
    int32_t c = 0;
    for (const Injection &j : run.inj) c = std::max(c, j.col);
    for (const Record &q : run.rec) c = std::max(c, q.col);
    return c / vec + 1;
}

template <typename T>
bool run_blocks_t(Ctx &c, StepOp &op, BatchRun &run) {
    Blocks &B = *run.blocks;
    const int64_t n = c.hm.n;
    hipStream_t s = c.stream;
    const int64_t groups = live_groups(run, B.vec);
    // the kernels take 16 bytes of columns or one; the caller's fields hold run.B columns
    MGRT_REQUIRE((B.vec == 1 || B.vec == 16 / (int)sizeof(T)) && groups * B.vec <= run.B, MGRT_E_STATE,
                 "regions of another precision or batch width");
    GroupLists tp = group_lists(B, groups, run.rec, c.hm, true, [](const Record &e) { return e.dst; });
    if (!tp.fits) return false;
    GroupLists ld = group_lists(B, groups, run.inj, c.hm, false, [](const Injection &e) { return e.sid; });
    if (!ld.fits) return false;
    // strips record histories (at 31-bit offsets) or the velocity field, not both
    if (B.nx > 0 && run.hist &&
        (run.d_vel_out || (int64_t)run.hist_nodes.size() * run.B * (int64_t)sizeof(T) >= (1ll << 30)))
        return false;
    if (run.d_series == nullptr) MGRT_REQUIRE(run.inj.empty(), MGRT_E_ARG, "loads without series");
    Pack pack;
    size_t lo[5], to[5];
    DevBuf xa, xb, done;
    const size_t state = (size_t)groups * n * B.vec * sizeof(T);
    const bool strip = B.nx > 0;
    try {
        auto up = [&](GroupLists &L, size_t *o) {
            o[0] = pack.add(L.ptr);
            o[1] = pack.add(L.loc);
            o[2] = pack.add(L.col);
            o[3] = pack.add(L.aux);
            o[4] = pack.add(L.w);
        };
        up(ld, lo);
        up(tp, to);
        pack.upload(nullptr);
        if (!run.d_alt_p) {
            xa.alloc(state);
            xb.alloc(state);
        }
        done.alloc(2 * sizeof(int64_t));
        if (strip && !op.strip_coef.p) op.strip_coef.alloc((size_t)n * 4 * sizeof(T));
        if (strip && !op.strip_rows.p) op.strip_rows.alloc((size_t)B.ny * 4);
    } catch (const Error &e) {
        if (e.code != MGRT_E_OOM_PLAN || run.d_alt_p) throw;
        (void)hipGetLastError();       // no room for the second buffer pair: one launch per step
        return false;
    }
    MGRT_HIP(hipMemsetAsync(done.p, 0, 2 * sizeof(int64_t), s));

    BlockArgs<T> a{};
    a.cnt = B.cnt.as<int32_t>();
    a.node = B.node.as<int32_t>();
    a.nbr = B.nbr.as<uint32_t>();
    a.beta = op.beta.as<T>();
    a.vals = op.vals.as<T>();
    a.n = n;
    a.n_ent = B.n_ent;
    a.n_tiles = (int32_t)B.n_tiles;
    a.log_s = 0;
    while ((1 << a.log_s) < op.S) ++a.log_s;
    a.groups = (int32_t)groups;
    // one-column runs of small meshes have always summed in this order (their traces are within
    // rounding of the one-step launches', and stay what they were)
    a.beta_first = run.B == 1 && n <= ONE_COLUMN_NODES && !run.hist && !run.d_vel_out && !run.d_acc;
    a.ld_ptr = pack.at<int32_t>(lo[0]);
    a.ld_loc = pack.at<int32_t>(lo[1]);
    a.ld_col = pack.at<int32_t>(lo[2]);
    a.ld_sid = pack.at<int32_t>(lo[3]);
    a.ld_w = pack.at<double>(lo[4]);
    a.tp_ptr = pack.at<int32_t>(to[0]);
    a.tp_loc = pack.at<int32_t>(to[1]);
    a.tp_col = pack.at<int32_t>(to[2]);
    a.tp_dst = pack.at<int32_t>(to[3]);
    a.tp_w = pack.at<double>(to[4]);
    a.series = run.d_series;
    a.series_len = run.series_len;
    a.step0 = run.step0;
    a.parts = run.d_parts;
    a.n_parts = run.n_parts;
    a.done = done.as<int64_t>();
    if (strip && op.strip_coef_version != op.version) {
        MGRT_HIP(hipMemsetAsync(op.strip_rows.p, 0, op.strip_rows.bytes, s));
        hipLaunchKernelGGL(k_strip_coef<T>, dim3((n + 255) / 256), dim3(256), 0, s, op.cols.as<int32_t>(),
                           op.vals.as<T>(), n, a.log_s, B.W, (int)B.nx, op.strip_coef.as<T>(), op.strip_rows.as<int32_t>());
        op.strip_coef_version = op.version;
    }
    a.inv_dt = (T)(1.0 / op.dt);
    // histories: staged step-major for chunks of up to 64 steps (at most 256 MB)
    const int64_t hist_nh = run.hist ? (int64_t)run.hist_nodes.size() : 0, hist_nser = hist_nh * run.B;
    const bool dual = run.hist && run.hist_mode == 2;
    MGRT_REQUIRE(!dual || run.d_hist2, MGRT_E_ARG, "dual history without its second series");
    int64_t chunk = 0;
    DevBuf st1, st2, hof;
    if (hist_nh > 0) {
        chunk = std::max<int64_t>(1, std::min<int64_t>(64, (256ll << 20) / (hist_nser * (int64_t)sizeof(T))));
        st1.alloc((size_t)chunk * hist_nser * sizeof(T));
        if (dual) st2.alloc((size_t)chunk * hist_nser * sizeof(T));
        std::vector<int32_t> of(n, -1);
        for (int64_t q = 0; q < hist_nh; ++q) of[c.hm.iperm[run.hist_nodes[q]]] = (int32_t)q;
        hof = upload(of, s);
        a.hist_of = hof.as<int32_t>();
        a.hist = st1.as<T>();
        a.hist2 = st2.as<T>();
        a.hist_nh = hist_nh;
        a.hist_b = run.B;
        a.hist_mode = run.hist_mode;
        a.hist_chunk = chunk;
    }
    const int64_t nB = n * (int64_t)run.B;
    DevBuf accp;
    if (run.d_vel_out) {
        a.vel_out = static_cast<T *>(run.d_vel_out);
        a.vel_step = nB;
    }
    if (run.d_acc) {
        a.vel = static_cast<const T *>(run.d_vel);
        a.vel_step = run.vel_reverse ? -nB : nB;
        a.vel_first = run.vel_reverse ? (run.n_steps - 1) * nB : 0;
        a.acc = run.d_acc;
        if (groups > 1) {
            accp.alloc((size_t)groups * n * 8);
            MGRT_HIP(hipMemsetAsync(accp.p, 0, (size_t)groups * n * 8, s));
            a.acc = accp.as<double>();
        }
    }
    const bool ext = chunk > 0 || run.d_vel_out || run.d_acc;

    const bool timing = (run.flags & MGRT_F_TIMING) != 0;
    hipEvent_t e0 = nullptr, e1 = nullptr;
    if (timing) {
        MGRT_HIP(hipEventCreate(&e0));
        MGRT_HIP(hipEventCreate(&e1));
    }
    // the pair (p_l, p_{l-1}) alternates between the caller's buffers and (xa, xb): a launch
    // reads one pair while its workgroups write the other
    T *src_p = static_cast<T *>(run.d_p), *src_pm = static_cast<T *>(run.d_pm);
    T *alt_p = run.d_alt_p ? static_cast<T *>(run.d_alt_p) : xa.as<T>();
    T *alt_pm = run.d_alt_p ? static_cast<T *>(run.d_alt_pm) : xb.as<T>();
    int64_t launches = 0;
    int slot = 0;
    BlockLaunch L{};
    L.W = B.W;
    L.npt = B.npt;
    L.threads = B.threads;
    L.ext = ext;
    L.lds = block_lds(B.threads * B.npt, B.vec, B.k, sizeof(T));
    L.s = s;
    auto launch = [&] {
        if (B.vec == 1) launch_blocks<T, 1>(a, L);
        else launch_blocks<T, 16 / sizeof(T)>(a, L);
    };
    if (!strip) {
        launch();   // ksteps 0: the LDS limit and the workgroups per CU
        L.grid = std::min<int64_t>(B.n_tiles * groups, 256 * std::max(1, L.per_cu));
    }
    auto launch_strips = [&](int ks) {
        constexpr int VEC = 16 / sizeof(T);
        StripArgs<T> b{};
        b.p = a.p; b.pm = a.pm; b.out_p = a.out_p; b.out_pm = a.out_pm;
        b.coef = op.strip_coef.as<T>();
        b.beta = a.beta;
        b.row_first = op.strip_rows.as<int32_t>();
        b.nx = (int32_t)B.nx; b.ny = (int32_t)B.ny;
        b.strips = (int32_t)B.strips; b.chunks = (int32_t)B.chunks;
        b.groups = a.groups;
        b.items = (int32_t)(B.n_tiles * groups);
        b.n = n;
        b.ld_ptr = a.ld_ptr; b.ld_loc = a.ld_loc; b.ld_col = a.ld_col; b.ld_sid = a.ld_sid; b.ld_w = a.ld_w;
        b.tp_ptr = a.tp_ptr; b.tp_loc = a.tp_loc; b.tp_col = a.tp_col; b.tp_dst = a.tp_dst; b.tp_w = a.tp_w;
        b.series = a.series; b.series_len = a.series_len; b.step0 = a.step0;
        b.parts = a.parts; b.n_parts = a.n_parts;
        b.done = a.done; b.slot = a.slot;
        b.hist_of = a.hist_of; b.hist = a.hist; b.hist2 = a.hist2;
        b.hist_nh = a.hist_nh; b.hist_b = a.hist_b; b.hist_chunk = a.hist_chunk; b.hist_mode = a.hist_mode;
        b.inv_dt = a.inv_dt;
        b.vel_out = a.vel_out; b.vel_step = a.vel_step;
        b.halo = B.k;
        const dim3 grid((unsigned)((b.items + 3) / 4));
        auto go = [&](auto kern) { hipLaunchKernelGGL(kern, grid, dim3(256), 0, s, b); };
        auto by_ext = [&](auto kc) {
            constexpr int KS = decltype(kc)::value;
            if (chunk) go(k_strips<T, VEC, KS, 1>);
            else if (run.d_vel_out) go(k_strips<T, VEC, KS, 2>);
            else go(k_strips<T, VEC, KS, 0>);
        };
        if (ks == STRIP_K<T>) by_ext(std::integral_constant<int, STRIP_K<T>>{});
        else if (ks == 4) by_ext(std::integral_constant<int, 4>{});
        else if (ks == 2) by_ext(std::integral_constant<int, 2>{});
        else by_ext(std::integral_constant<int, 1>{});
    };
    auto issue = [&](int64_t ks) {
        a.p = src_p;
        a.pm = src_pm;
        a.out_p = alt_p;
        a.out_pm = alt_pm;
        a.ksteps = (int32_t)ks;
        a.slot = slot;
        if (strip) launch_strips((int)ks);
        else launch();
        std::swap(src_p, alt_p);
        std::swap(src_pm, alt_pm);
        slot ^= 1;
        ++launches;
    };
    // the chunk of count steps that ends with the steps done so far
    auto flush = [&](int64_t count) {
        hist_flush(run, op.prec, st1.p, st2.p, hist_nser, count, a.done + slot, s);
    };
    // steps of the launch after l of cnt steps: at most k, none of them across a history chunk
    auto next_steps = [&](int64_t l, int64_t cnt) {
        int64_t ks = std::min<int64_t>(B.k, cnt - l);
        if (chunk) ks = std::min(ks, chunk - l % chunk);
        if (strip)
            while (ks != B.k && (ks & (ks - 1))) ks &= ks - 1;      // k or a power of two
        return ks;
    };
    auto steps = [&](int64_t cnt) {
        for (int64_t l = 0; l < cnt;) {
            const int64_t ks = next_steps(l, cnt);
            issue(ks);
            l += ks;
            if (chunk && (l % chunk == 0 || l == cnt)) flush(l % chunk ? l % chunk : chunk);
        }
    };
    if (timing) MGRT_HIP(hipEventRecord(e0, s));
    // Runs of steps are captured once and replayed: one history chunk, 64 launches of a
    // one-column run, else 64 steps; twice that where the launch count is odd, so that the
    // buffer pairs are back in place after each replay.
    int64_t l = 0;
    const int64_t kk = B.k;
    int64_t per = chunk ? chunk : run.B == 1 ? 64 * kk : 64;
    auto launches_of = [&](int64_t cnt) {
        int64_t m = 0;
        for (int64_t q = 0; q < cnt; ++m) q += next_steps(q, cnt);
        return m;
    };
    if (launches_of(per) % 2) per *= 2;
    // (twice the steps need not be twice the launches where no history chunk ends a launch)
    const int64_t nrep = launches_of(per) % 2 ? 0 : run.n_steps / per;
    if (!(run.flags & MGRT_F_NO_GRAPH) && nrep >= 2) {
        const hipGraphExec_t exec = capture_launches(c, [&](hipStream_t cs) {
            s = L.s = cs;
            steps(per);
            s = L.s = c.stream;
        });
        if (!exec) {
            launches = 0;
        } else {
            launches *= nrep;
            hipError_t le = hipSuccess;
            for (int64_t r = 0; r < nrep && le == hipSuccess; ++r) le = hipGraphLaunch(exec, s);
            const hipError_t se = hipStreamSynchronize(s);
            (void)hipGraphExecDestroy(exec);
            MGRT_HIP(le);
            MGRT_HIP(se);
            l = nrep * per;
            c.timing.graph_steps += l;
        }
    }
    if (l < run.n_steps) steps(run.n_steps - l);
    MGRT_HIP(hipGetLastError());
    if (timing) MGRT_HIP(hipEventRecord(e1, s));
    if (run.d_acc && groups > 1)
        hipLaunchKernelGGL(k_add_planes, dim3((n + 255) / 256), dim3(256), 0, s,
                           static_cast<const double *>(accp.as<double>()), groups, n, run.d_acc);
    // leave p_N, p_{N-1} in the caller's buffers
    if (src_p != run.d_p) {
        MGRT_HIP(hipMemcpyAsync(run.d_p, src_p, state, hipMemcpyDeviceToDevice, s));
        MGRT_HIP(hipMemcpyAsync(run.d_pm, src_pm, state, hipMemcpyDeviceToDevice, s));
    }
    MGRT_HIP(hipStreamSynchronize(s));
    if (timing) {
        float ms = 0;
        MGRT_HIP(hipEventElapsedTime(&ms, e0, e1));
        c.timing.step_ms_total += ms;
        (void)hipEventDestroy(e0);
        (void)hipEventDestroy(e1);
    }
    c.timing.step_launches += launches;
    c.timing.steps_per_launch = B.k;
    // per launch: four state words per node and column and the operator; per step a word of
    // velocity out or in, and the accumulator per launch
    const double cols = (double)groups * B.vec;
    c.timing.step_bytes += launches * (4.0 * sizeof(T) * n * cols + op.oper_bytes + (run.d_acc ? 16.0 * n : 0.0)) +
                           (double)run.n_steps * ((run.d_vel_out ? 1 : 0) + (run.d_acc ? 1 : 0)) * sizeof(T) * n * cols;
    c.timing.batch = run.B;
    c.timing.ell_width = op.wmax;
    c.timing.ell_mean_width = op.wmean;
    return true;
}

}  // namespace

bool blocks_hold(const Ctx &c, Blocks &B, const BatchRun &run) {
    const int64_t g = live_groups(run, B.vec);
    return group_lists(B, g, run.inj, c.hm, false, [](const Injection &e) { return e.sid; }).fits &&
           group_lists(B, g, run.rec, c.hm, true, [](const Record &e) { return e.dst; }).fits;
}

bool run_blocks(Ctx &c, StepOp &op, BatchRun &run) {
    return op.prec == 32 ? run_blocks_t<float>(c, op, run) : run_blocks_t<double>(c, op, run);
}

}  // namespace mgrt
