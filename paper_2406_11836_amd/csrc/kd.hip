// kd.hip -- KD-tree partition of the Gaussian centres (RetinaGS Sec. 3.3).
//
// Level by level, every node's split is the floor(n/2)-th smallest centre
// coordinate (IEEE total order) on axis depth mod 3, found exactly by a radix
// select over the 32 key bits, 8 bits per pass: each pass histograms the
// digit of the members still matching the selected prefix, per node, and one
// wave per node picks the digit holding the target rank.  The first pass of a
// level moves the members to the children of the level above (coordinate <
// split: left); the third writes the few members that match 16 bits to a list,
// which the last one reads.  Leaf boxes are the intersections of the
// half-spaces along each root-to-leaf path.
//
// The fixed-size partition the paper compares against (Sec. 4.2, Table 2)
// uses the same tree with every node cut at the midpoint of its extent,
// starting from the bounding box of the centres: the leaves form a uniform
// grid.
#include <type_traits>

#include "common.hpp"

namespace rgs {

static constexpr int KD_THREADS = 256;

struct KdState {        // per node of the current level
    uint32_t prefix;    // selected high bits of the split key
    uint32_t mask;      // which bits are selected
    uint32_t k;         // rank still to find among members matching prefix
    uint32_t n;         // members of the node
};

// A pass reads a byte (the node inside its level) and a coordinate per centre and
// is bound by that: 16M centres, five levels, 0.48 ms for all levels instead of
// 1.75, when nodes took four bytes, every level read all centres five times and
// the digit of a rank was looked for by one thread.  LDS atomics on one address
// take a lane per clock, and the first levels' first digits (sign and exponent)
// are the same for most lanes: R copies of the histogram, by lane, share the 32 KB
// that the last level's 32 nodes need anyway.
static constexpr int KH_THREADS = 1024, KH_U = 4, KH_BLOCKS = 512;  // two blocks per CU: few flushes, enough loads
static constexpr int KH_LIST = 4096;   // a block's members that match 16 bits (more: the last pass reads all centres)
static constexpr int KD_MAXCNT = RGS_MAXK / 2;

struct KdList {
    uint32_t* e;    // node << 16 | low half of the key
    uint32_t* n;    // entries (above cap: incomplete, not used)
    uint32_t cap;
};

// hist[node * 256 + digit] over the members whose key matches the node's prefix.
template <int PASS>
__global__ __launch_bounds__(KH_THREADS) void k_kd_pass(const float* __restrict__ coord, const float* __restrict__ above,
                                                        uint8_t* __restrict__ node, int64_t n, int cnt, int copies,
                                                        const KdState* __restrict__ st, const float* __restrict__ split,
                                                        uint32_t* __restrict__ hist, KdList list) {
    extern __shared__ uint32_t s_h[];  // [copies][cnt][256]
    __shared__ uint32_t s_prefix[KD_MAXCNT], s_mask[KD_MAXCNT];
    __shared__ float s_split[KD_MAXCNT];
    __shared__ uint32_t s_list[PASS == 2 ? KH_LIST : 1], s_n, s_base;
    constexpr int shift = 24 - 8 * PASS;
    const int tid = threadIdx.x;
    for (int k = tid; k < copies * cnt * 256; k += KH_THREADS) s_h[k] = 0;
    if (tid < cnt) {
        s_prefix[tid] = PASS > 0 ? st[tid].prefix : 0u;
        s_mask[tid] = PASS > 0 ? st[tid].mask : 0u;
    }
    if (PASS == 0 && tid < cnt / 2) s_split[tid] = split[cnt / 2 - 1 + tid];
    if (tid == 0) s_n = 0;
    __syncthreads();
    uint32_t* h = s_h + (tid & (copies - 1)) * cnt * 256;
    const int64_t step = (int64_t)gridDim.x * KH_THREADS * KH_U;
    if (PASS == 3 && *list.n <= list.cap) {
        const int64_t m = *list.n;
        for (int64_t i = (int64_t)blockIdx.x * KH_THREADS + tid; i < m; i += (int64_t)gridDim.x * KH_THREADS) {
            const uint32_t e = list.e[i], nd = e >> 16;
            if (((e ^ s_prefix[nd]) & 0xff00u) == 0u) atomicAdd(&h[nd * 256 + (e & 0xffu)], 1u);
        }
    } else {
        for (int64_t base = (int64_t)blockIdx.x * KH_THREADS * KH_U; base < n; base += step) {
            // all loads first (a lane past the end reads the last centre and adds nothing)
            float c[KH_U], ca[KH_U];
            uint32_t nd[KH_U];
#pragma unroll
            for (int u = 0; u < KH_U; ++u) {
                const int64_t i = base + u * KH_THREADS + tid, at = i < n ? i : n - 1;
                c[u] = coord[at];
                ca[u] = PASS == 0 && cnt > 1 ? above[at] : 0.f;
                nd[u] = cnt > (PASS == 0 ? 2 : 1) ? node[at] : 0u;
            }
#pragma unroll
            for (int u = 0; u < KH_U; ++u) {
                const int64_t i = base + u * KH_THREADS + tid;
                if (i >= n) continue;
                uint32_t k = nd[u];
                if (PASS == 0 && cnt > 1) {
                    k = 2u * k + (ca[u] < s_split[k] ? 0u : 1u);
                    node[i] = (uint8_t)k;
                }
                const uint32_t key = f2key(c[u]);
                if (PASS > 0 && (key & s_mask[k]) != s_prefix[k]) continue;
                atomicAdd(&h[k * 256 + ((key >> shift) & 0xffu)], 1u);
                if (PASS == 2) {
                    const uint32_t at = atomicAdd(&s_n, 1u);
                    if (at < KH_LIST) s_list[at] = k << 16 | (key & 0xffffu);
                }
            }
        }
    }
    __syncthreads();
    for (int k = tid; k < cnt * 256; k += KH_THREADS) {
        uint32_t a = 0;
        for (int r = 0; r < copies; ++r) a += s_h[r * cnt * 256 + k];
        if (a) atomicAdd(&hist[k], a);
    }
    if (PASS == 2) {
        const uint32_t m = s_n;
        // a block that holds too many makes the list one that is not used
        if (tid == 0 && m) s_base = m <= KH_LIST ? atomicAdd(list.n, m) : atomicMax(list.n, list.cap + 1u);
        __syncthreads();
        if (m <= KH_LIST)
            for (uint32_t k = tid; k < m; k += KH_THREADS)
                if (s_base + k < list.cap) list.e[s_base + k] = s_list[k];
    }
}

__global__ void k_kd_zero(uint32_t* __restrict__ p, int m) {
    for (int k = threadIdx.x + blockIdx.x * blockDim.x; k < m; k += blockDim.x * gridDim.x) p[k] = 0;
}

__global__ void k_kd_fill_ones(uint32_t* __restrict__ p, int m) {
    for (int k = threadIdx.x + blockIdx.x * blockDim.x; k < m; k += blockDim.x * gridDim.x) p[k] = 0xffffffffu;
}

// Node bounds along the path (for empty nodes, or for every node under the
// grid rule, starting from the centres' bounding box) and the split value.
__device__ __forceinline__ void finish_node(int t, const KdState* st, float* __restrict__ split, int first, int level,
                                            const uint32_t* __restrict__ root_key) {
    const int nd = first + t;
    const int a = level % 3;
    float s;
    if (root_key) {
        // grid rule: midpoint of the node's extent inside the bounding box
        const uint32_t klo = root_key[a], khi = root_key[3 + a];
        float lo = klo == 0xffffffffu ? INFINITY : key2f(klo), hi = khi == 0u ? -INFINITY : key2f(khi);
        int c = nd;
        while (c > 0) {
            const int p = (c - 1) >> 1;
            const int dp = 31 - __builtin_clz((unsigned)(p + 1));  // depth of p
            if (dp % 3 == a) {
                if (c == 2 * p + 1) { if (split[p] < hi) hi = split[p]; }
                else { if (split[p] > lo) lo = split[p]; }
            }
            c = p;
        }
        s = (isfinite(lo) && isfinite(hi)) ? 0.5f * (lo + hi) : 0.0f;
    } else if (st[t].n > 0) {
        s = key2f(st[t].prefix);
    } else {
        float lo = -INFINITY, hi = INFINITY;
        int c = nd, d = level;
        while (c > 0) {
            int p = (c - 1) >> 1;
            --d;
            if (d % 3 == a) {
                if (c == 2 * p + 1) { if (split[p] < hi) hi = split[p]; }
                else { if (split[p] > lo) lo = split[p]; }
            }
            c = p;
        }
        if (isfinite(lo) && isfinite(hi)) s = 0.5f * (lo + hi);
        else if (isfinite(lo)) s = lo;
        else if (isfinite(hi)) s = hi;
        else s = 0.0f;
    }
    split[nd] = s;
}

__global__ void k_kd_grid_level(float* __restrict__ split, int first, int cnt, int level,
                                const uint32_t* __restrict__ root_key) {
    if ((int)threadIdx.x < cnt) finish_node(threadIdx.x, nullptr, split, first, level, root_key);
}

// One wave per node: pick the digit containing rank k, and clear the node's
// histogram for the next pass.  After the last digit, the splits.
__global__ __launch_bounds__(KH_THREADS) void k_kd_select(KdState* __restrict__ st, uint32_t* __restrict__ hist, int cnt,
                                                          int pass, float* __restrict__ split, int first, int level,
                                                          uint32_t* __restrict__ list_n) {
    __shared__ KdState s_st[KD_MAXCNT];
    const int lane = threadIdx.x & 63, shift = 24 - 8 * pass;
    for (int t = threadIdx.x >> 6; t < cnt; t += KH_THREADS / 64) {
        uint4* h4 = reinterpret_cast<uint4*>(hist + t * 256) + lane;
        const uint4 h = *h4;
        *h4 = make_uint4(0u, 0u, 0u, 0u);
        const uint32_t own = (h.x + h.y) + (h.z + h.w), incl = wave_incl_scan(own);
        KdState s = pass == 0 ? KdState{0u, 0u, 0u, 0u} : st[t];
        if (pass == 0) {
            s.n = __shfl(incl, 63, 64);
            s.k = s.n / 2;
        }
        if (s.n > 0) {
            // the lane whose four digits hold the rank
            const uint64_t above = __ballot(incl > s.k);
            const int sel = above ? (int)__builtin_ctzll(above) : 63;
            uint32_t cum = incl - own;
            int d = 4 * lane;
            if (cum + h.x <= s.k) { cum += h.x; ++d;
                if (cum + h.y <= s.k) { cum += h.y; ++d;
                    if (cum + h.z <= s.k) { cum += h.z; ++d; } } }
            s.k -= __shfl(cum, sel, 64);
            s.prefix |= (uint32_t)__shfl(d, sel, 64) << shift;
            s.mask |= 0xffu << shift;
        }
        if (lane == 0) {
            st[t] = s;
            s_st[t] = s;
        }
    }
    if (pass < 3) return;
    __syncthreads();
    if ((int)threadIdx.x < cnt) finish_node(threadIdx.x, s_st, split, first, level, nullptr);
    if (threadIdx.x == 0) *list_n = 0u;
}

// Bounding box of the centres as IEEE total-order keys: min of x, y, z then max.
__global__ __launch_bounds__(KD_THREADS) void k_kd_root_box(const float* __restrict__ means, int64_t n,
                                                            uint32_t* __restrict__ key) {
    __shared__ uint32_t s_k[6];
    if (threadIdx.x < 6) s_k[threadIdx.x] = threadIdx.x < 3 ? 0xffffffffu : 0u;
    __syncthreads();
    uint32_t mn[3] = {0xffffffffu, 0xffffffffu, 0xffffffffu}, mx[3] = {0u, 0u, 0u};
    for (int64_t i = (int64_t)blockIdx.x * KD_THREADS + threadIdx.x; i < n; i += (int64_t)gridDim.x * KD_THREADS)
        for (int a = 0; a < 3; ++a) {
            const uint32_t k = f2key(means[a * n + i]);
            mn[a] = min(mn[a], k);
            mx[a] = max(mx[a], k);
        }
    for (int a = 0; a < 3; ++a) {
        mn[a] = ~wave_max_u32(~mn[a]);
        mx[a] = wave_max_u32(mx[a]);
    }
    if ((threadIdx.x & 63) == 0)
        for (int a = 0; a < 3; ++a) {
            atomicMin(&s_k[a], mn[a]);
            atomicMax(&s_k[3 + a], mx[a]);
        }
    __syncthreads();
    if (threadIdx.x < 3) atomicMin(&key[threadIdx.x], s_k[threadIdx.x]);
    else if (threadIdx.x < 6) atomicMax(&key[threadIdx.x], s_k[threadIdx.x]);
}

__global__ void k_kd_boxes(const float* __restrict__ split, int L, float* __restrict__ lo, float* __restrict__ hi,
                           int32_t* __restrict__ counts) {
    const int K = 1 << L;
    int k = threadIdx.x;
    if (k >= K) return;
    float l[3] = {-INFINITY, -INFINITY, -INFINITY}, h[3] = {INFINITY, INFINITY, INFINITY};
    int nd = 0;
    for (int d = 0; d < L; ++d) {
        const int a = d % 3;
        const int right = (k >> (L - 1 - d)) & 1;
        if (right) { l[a] = split[nd]; nd = 2 * nd + 2; }
        else { h[a] = split[nd]; nd = 2 * nd + 1; }
    }
    for (int a = 0; a < 3; ++a) {
        lo[a * K + k] = l[a];
        hi[a * K + k] = h[a];
    }
    counts[k] = 0;
}

// Leaf of every centre (walked down the splits), per-leaf counts, ownership
// masks and per-leaf bounds (the box of the centres and the largest scale).
// Grid-stride blocks: counts and bounds are reduced in LDS (integer keys, so
// min/max are exact and order-independent; a bound is only updated by a lane that
// reads a looser one) and each block issues one global atomic per (leaf, bound)
// it touched.
// A centre lies on the near side of every cut, so with D_i >= 0 a cut can only
// take the cells of its far side out of the mask: one distance per cut instead of
// six per cell (a cell's faces are its path's last cuts per axis, and looser cuts
// of the same axis hold when the last one does, as the subtraction is monotone).
// Where a centre, D_i or a cut is not finite the faces are compared one by one.
// 16M Gaussians, 32 cells: 662 us with six comparisons per cell, three fp64
// exponentials (the largest scale is that of the largest log scale) and
// unconditional atomics; 189 now.
// A block ends with an atomic per (leaf, bound), which the other blocks' take turns
// with: 1024 blocks (1M, 8 cells: 169 us for the partition, with 2048 196) but 2048
// from 8M on, where the work counts (16M, 64 cells: 841 / 803).  With one leaf there
// would be nothing but turns, in LDS and here: there a thread keeps its own bounds (1M
// 115 -> 80 us, 16M sorted by coordinate 584 -> 178).
static unsigned leaf_blocks(int64_t n) { return n < 8000000 ? 1024u : 2048u; }

// The masks and cuts are scalar: the kernel is made for each depth.
template <int L>
__global__ __launch_bounds__(KD_THREADS) void k_kd_leaves(int64_t n, const float* __restrict__ split,
                                                          const float* __restrict__ means,
                                                          const float* __restrict__ log_scales, float d_factor,
                                                          const float* __restrict__ lo, const float* __restrict__ hi,
                                                          int32_t* __restrict__ center_cell, int32_t* __restrict__ counts,
                                                          uint32_t* __restrict__ own_mask, uint32_t* __restrict__ bounds_key) {
    __shared__ int32_t s_cnt[RGS_MAXK];
    __shared__ uint32_t s_bk[7 * RGS_MAXK];
    __shared__ float s_split[RGS_MAXK];
    __shared__ int s_plain;
    constexpr int K = 1 << L;
    using Mask = typename std::conditional<(L > 5), uint64_t, uint32_t>::type;
    if (threadIdx.x == 0) s_plain = 0;
    __syncthreads();
    for (int t = threadIdx.x; t < K; t += KD_THREADS) s_cnt[t] = 0;
    for (int t = threadIdx.x; t < K - 1; t += KD_THREADS) {
        s_split[t] = split[t];
        if (!isfinite(split[t])) s_plain = 1;
    }
    for (int t = threadIdx.x; t < 7 * K; t += KD_THREADS) s_bk[t] = (t < 3 * K) ? 0xffffffffu : 0u;
    __syncthreads();
    constexpr int Wm = (K + 31) / 32;
    const bool plain = s_plain != 0;
    // one leaf: a thread keeps its own
    uint32_t mn[3] = {0xffffffffu, 0xffffffffu, 0xffffffffu}, mx[4] = {0u, 0u, 0u, 0u};
    for (int64_t i = (int64_t)blockIdx.x * KD_THREADS + threadIdx.x; i < n; i += (int64_t)gridDim.x * KD_THREADS) {
        const float u[3] = {means[i], means[n + i], means[2 * n + i]};
        float ls = 0.f;
        if (own_mask || bounds_key) ls = fmaxf(fmaxf(log_scales[i], log_scales[n + i]), log_scales[2 * n + i]);
        int leaf = 0;
        for (int d = 0; d < L; ++d) {
            const float c = d % 3 == 0 ? u[0] : (d % 3 == 1 ? u[1] : u[2]);
            leaf = 2 * leaf + (c < s_split[(1 << d) - 1 + leaf] ? 0 : 1);
        }
        if (L > 0) atomicAdd(&s_cnt[leaf], 1);
        center_cell[i] = leaf;
        if (!own_mask && !bounds_key) continue;
        // D_i = d_factor * max scale; transcendental in fp64, rounded once
        const float smax = (float)exp((double)ls);
        const float Di = d_factor * smax;
        if (L == 0) {
            for (int a = 0; a < 3; ++a) {
                mn[a] = min(mn[a], f2key(u[a]));
                mx[a] = max(mx[a], f2key(u[a]));
            }
            mx[3] = max(mx[3], f2key(smax));
        } else if (bounds_key) {
            for (int a = 0; a < 3; ++a) {
                const uint32_t k = f2key(u[a]);
                if (k < s_bk[a * K + leaf]) atomicMin(&s_bk[a * K + leaf], k);
                if (k > s_bk[(3 + a) * K + leaf]) atomicMax(&s_bk[(3 + a) * K + leaf], k);
            }
            const uint32_t k = f2key(smax);
            if (k > s_bk[6 * K + leaf]) atomicMax(&s_bk[6 * K + leaf], k);
        }
        if (!own_mask) continue;
        Mask m = 0;
        if (!plain && Di >= 0.f && Di < INFINITY && fabsf(u[0]) < INFINITY && fabsf(u[1]) < INFINITY && fabsf(u[2]) < INFINITY) {
            m = K == 8 * (int)sizeof(Mask) ? ~Mask(0) : (Mask)(((Mask)1 << (K & 63)) - 1);
#pragma unroll
            for (int d = 0; d < L; ++d) {
                const float c = u[d % 3];
#pragma unroll
                for (int t = 0; t < (1 << d); ++t) {
                    const int w = K >> (d + 1), k0 = 2 * w * t;  // cells per side
                    const Mask left_cells = (Mask)((((Mask)1 << w) - 1) << k0), right_cells = (Mask)(left_cells << w);
                    const float cut = split[(1 << d) - 1 + t];
                    const bool left = c < cut;
                    // the far side's face: right lo - u, left u - hi
                    if (!((left ? cut - c : c - cut) <= Di)) m &= ~(left ? right_cells : left_cells);
                }
            }
        } else {
            for (int k = 0; k < K; ++k) {
                bool in = true;
                for (int a = 0; a < 3; ++a) {
                    if (!((lo[a * K + k] - u[a]) <= Di)) in = false;
                    if (!((u[a] - hi[a * K + k]) <= Di)) in = false;
                }
                if (in) m |= (Mask)1 << k;
            }
        }
        own_mask[i * Wm] = (uint32_t)m;
        if (Wm > 1) own_mask[i * Wm + 1] = (uint32_t)((uint64_t)m >> 32);
    }
    if (L == 0) {
        uint32_t r[7];
        for (int a = 0; a < 3; ++a) r[a] = ~wave_max_u32(~mn[a]);
        for (int a = 0; a < 4; ++a) r[3 + a] = wave_max_u32(mx[a]);
        if ((threadIdx.x & 63) == 0) {
            for (int a = 0; a < 3; ++a) atomicMin(&s_bk[a], r[a]);
            for (int a = 3; a < 7; ++a) atomicMax(&s_bk[a], r[a]);
        }
        if (blockIdx.x == 0 && threadIdx.x == 0) s_cnt[0] = (int32_t)n;
    }
    __syncthreads();
    for (int t = threadIdx.x; t < K; t += KD_THREADS)
        if (s_cnt[t]) atomicAdd(&counts[t], s_cnt[t]);
    if (bounds_key)
        for (int t = threadIdx.x; t < 7 * K; t += KD_THREADS) {
            const uint32_t v = s_bk[t];
            if (t < 3 * K) {
                if (v != 0xffffffffu) atomicMin(&bounds_key[t], v);
            } else if (v != 0u) {
                atomicMax(&bounds_key[t], v);
            }
        }
}

__global__ void k_kd_bounds_init(uint32_t* __restrict__ bk, int K) {
    int t = threadIdx.x;
    if (t < 7 * K) bk[t] = (t < 3 * K) ? 0xffffffffu : 0u;
}

// cell_bounds rows: min x, y, z; max x, y, z of the centres (+inf / -inf for an
// empty cell); the largest scale exp(log_scale) of the cell (0 if empty); 0.
__global__ void k_kd_bounds_final(const uint32_t* __restrict__ bk, int K, float* __restrict__ bounds) {
    int t = threadIdx.x;
    if (t >= 8 * K) return;
    if (t >= 7 * K) { bounds[t] = 0.0f; return; }
    const uint32_t k = bk[t];
    if (t < 3 * K) bounds[t] = (k == 0xffffffffu) ? INFINITY : key2f(k);
    else if (t < 6 * K) bounds[t] = (k == 0u) ? -INFINITY : key2f(k);
    else bounds[t] = (k == 0u) ? 0.0f : key2f(k);
}

size_t kd_ws_bytes(int64_t n, int L) {
    const int K = 1 << L;
    return (size_t)n * sizeof(int32_t) + 256 + (size_t)K * 256 * sizeof(uint32_t) + 256 + (size_t)K * sizeof(KdState) + 256 +
           (size_t)7 * K * sizeof(uint32_t) + 256 + 6 * sizeof(uint32_t) + 256;
}

rgs_status kd_partition(const rgs_gaussians* g, int L, float d_factor, int rule, const rgs_kdtree* kd, void* ws,
                        hipStream_t s) {
    const int64_t n = g->n;
    const int K = 1 << L;
    WsCarver c{reinterpret_cast<char*>(ws), 0, (size_t)-1};
    // the nodes' bytes and the list share four bytes per centre
    char* per = c.take<char>((size_t)(n > 0 ? n : 1) * sizeof(int32_t));
    uint8_t* node = reinterpret_cast<uint8_t*>(per);
    const size_t node_bytes = ((size_t)n + 255) & ~size_t(255);
    const size_t all = (size_t)n * sizeof(int32_t);
    KdList list{reinterpret_cast<uint32_t*>(per + node_bytes), nullptr,
                all > node_bytes ? (uint32_t)((all - node_bytes) / sizeof(uint32_t)) : 0u};
    uint32_t* hist = c.take<uint32_t>((size_t)K * 256);
    KdState* st = c.take<KdState>(K);
    uint32_t* bk = c.take<uint32_t>((size_t)7 * K);
    uint32_t* root = c.take<uint32_t>(6);
    list.n = hist + (size_t)(K > 1 ? K / 2 : 1) * 256;  // (half of the table's rows are used)
    const unsigned gridN = (unsigned)((n + KD_THREADS - 1) / KD_THREADS);
    if (rule == RGS_SPLIT_MIDPOINT) {
        // min keys start at all ones, max keys at zero; every split follows from the box
        int box_blocks = (int)((n + KD_THREADS * 16 - 1) / (KD_THREADS * 16));
        if (box_blocks > 4096) box_blocks = 4096;
        hipLaunchKernelGGL(k_kd_fill_ones, dim3(1), dim3(64), 0, s, root, 3);
        hipLaunchKernelGGL(k_kd_zero, dim3(1), dim3(64), 0, s, root + 3, 3);
        if (n > 0) hipLaunchKernelGGL(k_kd_root_box, dim3(box_blocks), dim3(KD_THREADS), 0, s, g->means, n, root);
        for (int l = 0; l < L; ++l)
            hipLaunchKernelGGL(k_kd_grid_level, dim3(1), dim3(64), 0, s, kd->split, (1 << l) - 1, 1 << l, l, root);
    } else if (L > 0) {
        hipLaunchKernelGGL(k_kd_zero, dim3(16), dim3(256), 0, s, hist, (K / 2) * 256 + 1);
        int64_t hb = (n + KH_THREADS * KH_U - 1) / (KH_THREADS * KH_U);
        const dim3 grid((unsigned)(hb < 1 ? 1 : (hb > KH_BLOCKS ? KH_BLOCKS : hb))), block(KH_THREADS), one(1);
        for (int l = 0; l < L; ++l) {
            const int first = (1 << l) - 1, cnt = 1 << l;
            const int copies = 32 / cnt > 8 ? 8 : (32 / cnt < 1 ? 1 : 32 / cnt);
            const float* coord = g->means + (int64_t)(l % 3) * n;
            const float* above = g->means + (int64_t)((l + 2) % 3) * n;  // the axis of the level above
            const size_t lds = (size_t)copies * cnt * 256 * sizeof(uint32_t);
#define RGS_KD_PASS(P)                                                                                                 \
    if (n > 0)                                                                                                         \
        hipLaunchKernelGGL(k_kd_pass<P>, grid, block, lds, s, coord, above, node, n, cnt, copies, st, kd->split, hist, \
                           list);                                                                                      \
    hipLaunchKernelGGL(k_kd_select, one, block, 0, s, st, hist, cnt, P, kd->split, first, l, list.n);
            RGS_KD_PASS(0)
            RGS_KD_PASS(1)
            RGS_KD_PASS(2)
            RGS_KD_PASS(3)
#undef RGS_KD_PASS
            RGS_LAUNCH_CHECK();
        }
    }
    hipLaunchKernelGGL(k_kd_boxes, dim3(1), dim3(64), 0, s, kd->split, L, kd->box_lo, kd->box_hi, kd->counts);
    if (kd->cell_bounds) hipLaunchKernelGGL(k_kd_bounds_init, dim3(1), dim3(448), 0, s, bk, K);
    const unsigned gridL = gridN < leaf_blocks(n) ? gridN : leaf_blocks(n);
    if (n > 0) {
        using Leaves = decltype(&k_kd_leaves<0>);
        static const Leaves leaves[7] = {k_kd_leaves<0>, k_kd_leaves<1>, k_kd_leaves<2>, k_kd_leaves<3>,
                                         k_kd_leaves<4>, k_kd_leaves<5>, k_kd_leaves<6>};
        static_assert(RGS_MAXK == 64, "one kernel per depth");
        hipLaunchKernelGGL(leaves[L], dim3(gridL), dim3(KD_THREADS), 0, s, n, kd->split, g->means, g->log_scales, d_factor,
                           kd->box_lo, kd->box_hi, kd->center_cell, kd->counts, kd->own_mask,
                           kd->cell_bounds ? bk : nullptr);
    }
    if (kd->cell_bounds) hipLaunchKernelGGL(k_kd_bounds_final, dim3(1), dim3(512), 0, s, bk, K, kd->cell_bounds);
    return launch_check();
}

}  // namespace rgs
