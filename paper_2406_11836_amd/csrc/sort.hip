// sort.hip -- device-wide exclusive scan and stable LSD radix sort (gfx950).
//
// Scan: reduce per 4096-element tile, scan the tile sums in one block, then
// scan each tile with its offset.  Tiles are staged through LDS so that
// global loads and stores stay coalesced.
//
// Radix sort: digits of up to 8 bits, least significant first.  Per pass a
// histogram kernel counts digits per tile (LDS atomics on integers), one
// block per digit scans that digit's row of the [digit][tile] table (the digit
// bases come from the row totals), and a scatter kernel ranks each key stably
// inside its tile: every wave walks its strip in order, finds the lanes
// sharing its digit with a ballot per digit bit, and keeps a running count per
// digit in LDS; keys are then reordered in LDS by digit so that the global
// writes come out as contiguous runs.  A sort of few tiles skips the row scan;
// the instance sort's first histogram comes from the emission.
#include "common.hpp"

namespace rgs {

// ------------------------------------------------------------------ scan
static constexpr int SCAN_THREADS = 256;
// Grid cap for kernels whose element count is read on the device.
static constexpr unsigned DEV_GRID = 2048;
static constexpr int SCAN_ITEMS = 16;
static constexpr int SCAN_TILE = SCAN_THREADS * SCAN_ITEMS;
static_assert(SCAN_TILE == RGS_SCAN_TILE, "callers producing tile sums use RGS_SCAN_TILE");

__device__ __forceinline__ int skew(int i) { return i + (i >> 5); }

// Block-wide exclusive scan of one value per thread; returns the block total.
__device__ uint32_t block_excl_scan_256(uint32_t v, uint32_t* s_wave /*[4]*/, uint32_t* excl) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    uint32_t inc = wave_incl_scan(v);
    if (lane == 63) s_wave[w] = inc;
    __syncthreads();
    uint32_t base = 0, tot = 0;
    for (int k = 0; k < 4; ++k) {
        uint32_t t = s_wave[k];
        if (k < w) base += t;
        tot += t;
    }
    *excl = base + inc - v;
    __syncthreads();
    return tot;
}

// marks = 1: the scanned value of entry i is 1 if in[i] != ~0 (an occupied
// entry of a table whose empty entries hold all ones), else 0.
__device__ __forceinline__ uint32_t scan_val(const uint32_t* __restrict__ in, int64_t i, int marks) {
    const uint32_t v = in[i];
    return marks ? (v != 0xffffffffu ? 1u : 0u) : v;
}

__global__ __launch_bounds__(SCAN_THREADS) void k_scan_reduce(const uint32_t* __restrict__ in, DevN dn, int marks,
                                                              uint32_t* __restrict__ partial) {
    __shared__ uint32_t s_wave[4];
    const int64_t n = dn.get();
    for (int64_t tile = blockIdx.x; tile * SCAN_TILE < n; tile += gridDim.x) {
        const int64_t base = tile * SCAN_TILE;
        // all loads first (a lane past the end reads the last entry and adds nothing)
        uint32_t v[SCAN_ITEMS];
#pragma unroll
        for (int k = 0; k < SCAN_ITEMS; ++k) {
            const int64_t i = base + k * SCAN_THREADS + threadIdx.x;
            v[k] = scan_val(in, i < n ? i : n - 1, marks);
        }
        uint32_t acc = 0;
#pragma unroll
        for (int k = 0; k < SCAN_ITEMS; ++k) acc += base + k * SCAN_THREADS + threadIdx.x < n ? v[k] : 0u;
        uint32_t ex;
        uint32_t tot = block_excl_scan_256(acc, s_wave, &ex);
        if (threadIdx.x == 0) partial[tile] = tot;
    }
}

// Exclusive scan, in place, of the sums of the first ceil(dn / tile) tiles;
// the total to *total if non-null.
// (One block: 16384 sums per round, loaded together; 100M entries have 24K sums
// of 4096, which took 32 us in rounds of 256.)
static constexpr int SP_THREADS = 1024, SP_ITEMS = 16;
__global__ __launch_bounds__(SP_THREADS) void k_scan_partials(uint32_t* __restrict__ partial, DevN dn, int64_t tile,
                                                              uint32_t* __restrict__ total) {
    __shared__ uint32_t s_w[SP_THREADS / 64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int64_t m = (dn.get() + tile - 1) / tile;
    uint32_t carry = 0;
    for (int64_t b = 0; b < m; b += SP_THREADS * SP_ITEMS) {
        const int64_t i = b + (int64_t)threadIdx.x * SP_ITEMS;
        uint32_t v[SP_ITEMS], acc = 0;
        if (i + SP_ITEMS <= m) {
#pragma unroll
            for (int k = 0; k < SP_ITEMS; k += 4) {
                const uint4 q = *reinterpret_cast<const uint4*>(partial + i + k);
                v[k] = q.x; v[k + 1] = q.y; v[k + 2] = q.z; v[k + 3] = q.w;
            }
        } else {
#pragma unroll
            for (int k = 0; k < SP_ITEMS; ++k) v[k] = i + k < m ? partial[i + k] : 0u;
        }
#pragma unroll
        for (int k = 0; k < SP_ITEMS; ++k) acc += v[k];
        const uint32_t inc = wave_incl_scan(acc);
        if (lane == 63) s_w[w] = inc;
        __syncthreads();
        uint32_t run = carry + inc - acc;
#pragma unroll
        for (int k = 0; k < SP_THREADS / 64; ++k) {
            run += k < w ? s_w[k] : 0u;
            carry += s_w[k];
        }
#pragma unroll
        for (int k = 0; k < SP_ITEMS; ++k) {
            if (i + k < m) partial[i + k] = run;
            run += v[k];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0 && total) *total = carry;
}

// The optional tail of a scan of per-pair instance counts: out[n] = total,
// and, with guard set (no host copy of the instance count), if the total
// exceeds the capacity, counters[3] = total and the pair, instance and slot
// counts are zeroed so that every later kernel of the pass finds no work;
// else (and always without guard) counters[3] = 0.
__device__ __forceinline__ void scan_tail(const ScanTail& t, uint32_t* __restrict__ out, int64_t n, uint32_t total) {
    if (!t.cnt) return;
    out[n] = total;
    if (t.guard && (int64_t)total > t.capacity) {
        t.cnt[3] = total;
        t.cnt[0] = 0u;
        t.cnt[1] = 0u;
        t.cnt[2] = 0u;
    } else {
        t.cnt[3] = 0u;
    }
}

// fold = 1: the tile sums are not scanned beforehand; every block adds up the
// sums of the tiles before its own (for at most SCAN_FOLD_TILES tiles), and
// the block of the last tile writes the total and the tail.  fold = 0: the
// partials hold the scanned tile offsets (k_scan_partials wrote the total).
__global__ __launch_bounds__(SCAN_THREADS) void k_scan_apply(const uint32_t* __restrict__ in, DevN dn, int marks,
                                                             const uint32_t* __restrict__ partial, int fold,
                                                             uint32_t* __restrict__ total, ScanTail tail,
                                                             uint32_t* __restrict__ out) {
    __shared__ uint32_t s[SCAN_TILE + SCAN_TILE / 32];
    __shared__ uint32_t s_wave[4];
    const int64_t n = dn.get();
    if (fold && n <= 0) {
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            if (total) *total = 0u;
            scan_tail(tail, out, 0, 0u);
        }
        return;
    }
    const int64_t ntiles = (n + SCAN_TILE - 1) / SCAN_TILE;
    for (int64_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        const int64_t base = tile * SCAN_TILE;
        uint32_t toff;
        if (fold) {
            uint32_t a = 0;
            for (int64_t t = threadIdx.x; t < tile; t += SCAN_THREADS) a += partial[t];
            uint32_t ex;
            toff = block_excl_scan_256(a, s_wave, &ex);  // the block total of the per-thread sums
        } else {
            toff = partial[tile];
        }
        {
            uint32_t lv[SCAN_ITEMS];
#pragma unroll
            for (int k = 0; k < SCAN_ITEMS; ++k) {
                const int64_t i = base + k * SCAN_THREADS + threadIdx.x;
                lv[k] = scan_val(in, i < n ? i : n - 1, marks);
            }
#pragma unroll
            for (int k = 0; k < SCAN_ITEMS; ++k) {
                const int li = k * SCAN_THREADS + threadIdx.x;
                s[skew(li)] = base + li < n ? lv[k] : 0u;
            }
        }
        __syncthreads();
        uint32_t v[SCAN_ITEMS], acc = 0;
        for (int k = 0; k < SCAN_ITEMS; ++k) {
            v[k] = s[skew(threadIdx.x * SCAN_ITEMS + k)];
            acc += v[k];
        }
        uint32_t ex;
        const uint32_t tsum = block_excl_scan_256(acc, s_wave, &ex);
        if (fold && tile == ntiles - 1 && threadIdx.x == 0) {
            if (total) *total = toff + tsum;
            scan_tail(tail, out, n, toff + tsum);
        }
        uint32_t run = toff + ex;
        for (int k = 0; k < SCAN_ITEMS; ++k) {
            s[skew(threadIdx.x * SCAN_ITEMS + k)] = run;
            run += v[k];
        }
        __syncthreads();
        for (int k = 0; k < SCAN_ITEMS; ++k) {
            int li = k * SCAN_THREADS + threadIdx.x;
            int64_t i = base + li;
            if (i < n) out[i] = s[skew(li)];
        }
        if (tail.first) {
            // the pair holding each group's first instance: the last whose offset is
            // not above it (entries past n hold the tile's end)
            const int64_t end0 = (int64_t)toff + tsum, end = end0 < tail.capacity ? end0 : tail.capacity;
            auto mark = [&](uint32_t* table, int64_t group, int64_t lim) {
                for (int64_t g = ((int64_t)toff + group - 1) / group + threadIdx.x; g * group < lim; g += SCAN_THREADS) {
                    const uint32_t j = (uint32_t)(g * group);
                    int p = 0;
#pragma unroll
                    for (int step = SCAN_TILE / 2; step > 0; step >>= 1)
                        if (s[skew(p + step)] <= j) p += step;
                    table[g] = (uint32_t)(base + p);
                }
            };
            mark(tail.first, RGS_RADIX_TILE, end);
            mark(tail.first_small, RGS_FIRST_GROUP, end < RGS_FOLD_KEYS ? end : RGS_FOLD_KEYS);
        }
        __syncthreads();  // LDS is reused by the next tile
    }
}

// The tail for the path with a separate scan of the tile sums (total known).
__global__ void k_scan_tail(uint32_t* __restrict__ out, ScanTail tail) {
    if (threadIdx.x != 0) return;
    scan_tail(tail, out, tail.cnt[0], tail.cnt[1]);
}

size_t scan_ws_bytes(int64_t n) {
    int64_t tiles = (n + SCAN_TILE - 1) / SCAN_TILE;
    return (size_t)(tiles + 1) * sizeof(uint32_t) + 256;
}

rgs_status scan_tile_reduce(const uint32_t* in, int64_t n, int marks, uint32_t* partial, hipStream_t s) {
    if (n <= 0) return RGS_OK;
    const int64_t tiles = (n + SCAN_TILE - 1) / SCAN_TILE;
    hipLaunchKernelGGL(k_scan_reduce, dim3((unsigned)tiles), dim3(SCAN_THREADS), 0, s, in, DevN{nullptr, n, 1, 1}, marks,
                       partial);
    return launch_check();
}

rgs_status scan_tile_sums(uint32_t* partial, DevN dn, int64_t tile, uint32_t* total, hipStream_t s) {
    hipLaunchKernelGGL(k_scan_partials, dim3(1), dim3(SP_THREADS), 0, s, partial, dn, tile, total);
    return launch_check();
}

// Up to this many tiles, the apply kernel sums the tile sums itself (one
// launch fewer); beyond it a single block scans them first.
static constexpr int64_t SCAN_FOLD_TILES = 1024;

rgs_status exclusive_scan_u32_dev(const uint32_t* in, uint32_t* out, DevN dn, int64_t n_max, uint32_t* total, void* ws,
                                  hipStream_t s, int marks, const ScanTail* tail, int sums_ready) {
    uint32_t* partial = reinterpret_cast<uint32_t*>(ws);
    const ScanTail tl = tail ? *tail : ScanTail{nullptr, 0, 0, nullptr, nullptr};
    const int64_t tiles = (n_max + SCAN_TILE - 1) / SCAN_TILE;
    const bool fold = tiles <= SCAN_FOLD_TILES;
    const unsigned grid = (unsigned)(tiles < 1 ? 1 : (dn.p && tiles > DEV_GRID ? DEV_GRID : tiles));
    if (n_max > 0 && !sums_ready)
        hipLaunchKernelGGL(k_scan_reduce, dim3(grid), dim3(SCAN_THREADS), 0, s, in, dn, marks, partial);
    if (!fold) hipLaunchKernelGGL(k_scan_partials, dim3(1), dim3(SP_THREADS), 0, s, partial, dn, (int64_t)SCAN_TILE, total);
    hipLaunchKernelGGL(k_scan_apply, dim3(grid), dim3(SCAN_THREADS), 0, s, in, dn, marks, partial, fold ? 1 : 0,
                       total, tl, out);
    if (!fold && tl.cnt) {
        // the tail after the single-block scan of the tile sums
        hipLaunchKernelGGL(k_scan_tail, dim3(1), dim3(64), 0, s, out, tl);
    }
    return launch_check();
}

rgs_status exclusive_scan_u32(const uint32_t* in, uint32_t* out, int64_t n, uint32_t* total, void* ws,
                              hipStream_t s, int marks) {
    return exclusive_scan_u32_dev(in, out, DevN{nullptr, n, 1, 1}, n, total, ws, s, marks, nullptr);
}

// ------------------------------------------------------------------ radix sort
static constexpr int RS_THREADS = 256;

// The passes of a sort: as few as 8-bit digits allow, of nearly equal widths
// (13 bits: 7 + 6, not 8 + 5), so that the runs a tile writes per digit are as
// long as they can be.  Tiles are 2048 keys; a sort of at most 64K keys takes
// 512-key tiles, since a few blocks' latency is all it costs (20k keys, four
// passes' scatters: 24 against 31 us).
// Up to RS_FOLD_TILES tiles the scatter adds up the earlier tiles' counts
// itself (no column scan launch, about 4 us).
static constexpr int64_t RS_SMALL_KEYS = 65536;
static constexpr int64_t RS_FOLD_TILES = RGS_FOLD_KEYS / RGS_RADIX_TILE;

RadixPlan radix_plan(int64_t n, int bits) {
    RadixPlan p;
    p.passes = (bits + 7) / 8;
    int left = bits;
    for (int k = 0; k < 4; ++k) {
        const int w = k < p.passes ? (left + (p.passes - k) - 1) / (p.passes - k) : 0;
        p.bits[k] = w > 0 && w < 6 ? 6 : w;
        left -= p.bits[k];
        if (left < 0) left = 0;
    }
    p.items = n <= RS_SMALL_KEYS ? 2 : RGS_RADIX_TILE / RS_THREADS;
    p.tiles = (n + RS_THREADS * p.items - 1) / (RS_THREADS * p.items);
    p.fold = p.tiles <= RS_FOLD_TILES ? 1 : 0;
    return p;
}

int radix_fold_words(int64_t capacity) {
    const int64_t small = capacity < RS_SMALL_KEYS ? capacity : RS_SMALL_KEYS;
    const int64_t a = (capacity + RGS_RADIX_TILE - 1) / RGS_RADIX_TILE, b = (small + 2 * RS_THREADS - 1) / (2 * RS_THREADS);
    const int64_t t = a > b ? a : b;
    return (int)(256 * (t < RS_FOLD_TILES ? t : RS_FOLD_TILES));
}

__device__ __forceinline__ int64_t rs_n(int64_t n, const uint32_t* n_dev) {
    return n_dev ? (int64_t)*n_dev : n;
}

// Blocks loop over tiles (with a device-side count the grid is capped and
// sized for the largest possible count, so no block is launched only to exit);
// the n-th tile a block takes (n = block + round * grid) is tile
// xcd_band(n, tiles): with a grid that is a multiple of 8 (or a single
// round) every XCD takes one contiguous band of tiles, the same number each,
// so that the tiles that write neighbouring parts of a digit's output run on
// one XCD and the cache lines their runs share are completed in one L2.
template <int BITS, int ITEMS>
__global__ __launch_bounds__(RS_THREADS) void k_rs_hist(const uint32_t* __restrict__ keys, int64_t n_host,
                                                        const uint32_t* __restrict__ n_dev, int shift, int fold,
                                                        uint32_t* __restrict__ ws_a, uint32_t* __restrict__ ws_b) {
    constexpr int NB = 1 << BITS, TILE = RS_THREADS * ITEMS;
    __shared__ uint32_t s_h[NB];
    const int64_t n = rs_n(n_host, n_dev);
    const RadixTab tab = radix_tab(n, ITEMS, fold, ws_a, ws_b);
    for (int nth = blockIdx.x; nth < tab.units; nth += gridDim.x) {
        const int unit = xcd_band(nth, tab.units);
        uint32_t run = 0;  // digit threadIdx.x's count over the unit's tiles so far
        for (int u = 0; u < tab.per; ++u) {
            const int tile = unit * tab.per + u;
            const int64_t base = (int64_t)tile * TILE;
            if (base >= n) break;  // uniform per block
            if (threadIdx.x < NB) s_h[threadIdx.x] = 0;
            __syncthreads();
            // all loads first (a lane past the end reads the last key and adds nothing)
            const uint32_t tile_n = (uint32_t)((n - base) < TILE ? (n - base) : TILE);
            const uint32_t* kp = keys + base;
            uint32_t kv[ITEMS];
#pragma unroll
            for (int k = 0; k < ITEMS; ++k) {
                const uint32_t i = k * RS_THREADS + threadIdx.x;
                kv[k] = kp[i < tile_n ? i : tile_n - 1u];
            }
#pragma unroll
            for (int k = 0; k < ITEMS; ++k) {
                const uint32_t d = (kv[k] >> shift) & (NB - 1u);
                bool add = k * RS_THREADS + threadIdx.x < tile_n;
                if (tab.per > 1) {
                    // a large sort's later digits (view, screen rows) hardly vary inside
                    // a wave, and LDS atomics on one address take a lane per clock: the
                    // two commonest-looking digits are counted by ballot
#pragma unroll
                    for (int r = 0; r < 2; ++r) {
                        const uint64_t am = __builtin_amdgcn_ballot_w64(add);
                        if (am == 0ull) break;
                        const int l = (int)__builtin_ctzll(am);
                        const uint32_t f = (uint32_t)__builtin_amdgcn_readlane((int)d, l);
                        const uint64_t m = __builtin_amdgcn_ballot_w64(add && d == f);
                        if ((int)(threadIdx.x & 63) == l) atomicAdd(&s_h[f], (uint32_t)__popcll(m));
                        add = add && d != f;
                    }
                }
                if (add) atomicAdd(&s_h[d], 1u);
            }
            __syncthreads();
            if (threadIdx.x < NB) radix_tile_counts(tab, NB, tile, threadIdx.x, s_h[threadIdx.x], run);
        }
        if (threadIdx.x < NB) radix_unit_counts(tab, NB, fold, unit, threadIdx.x, run);
        __syncthreads();
    }
}

// Per digit d (one block each): exclusive scan over units of the digit's row
// hist[d][*] into offs[d][*], and the row total into dtot[d].  The scatter
// adds the digit's base (an exclusive scan of the totals, done in LDS).
__global__ __launch_bounds__(RS_THREADS) void k_rs_colscan(int64_t n_host, const uint32_t* __restrict__ n_dev, int items,
                                                           uint32_t* __restrict__ ws_a, uint32_t* __restrict__ ws_b,
                                                           uint32_t* __restrict__ dtot) {
    __shared__ uint32_t s_wave[4];
    const RadixTab tab = radix_tab(rs_n(n_host, n_dev), items, 0, ws_a, ws_b);
    const int units = tab.units;
    const int64_t row = (int64_t)blockIdx.x * units;
    uint32_t carry = 0;
    for (int t0 = 0; t0 < units; t0 += RS_THREADS * 4) {
        uint32_t v[4], acc = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int t = t0 + threadIdx.x * 4 + k;
            v[k] = t < units ? tab.hist[row + t] : 0u;
            acc += v[k];
        }
        uint32_t ex;
        const uint32_t tot = block_excl_scan_256(acc, s_wave, &ex);
        uint32_t run = carry + ex;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int t = t0 + threadIdx.x * 4 + k;
            if (t < units) tab.offs[row + t] = run;
            run += v[k];
        }
        carry += tot;
    }
    if (threadIdx.x == 0) dtot[blockIdx.x] = carry;
}

// The value an element enters the sort with: as stored, or, for the instance
// sort's first pass, (source << 32) | position from the 4-byte source alone
// (4 + 4 bytes per instance are emitted and read instead of 4 + 8).
template <typename VIN, typename V>
__device__ __forceinline__ V rs_value(VIN v, int64_t i) {
    if constexpr (sizeof(VIN) == sizeof(V)) return (V)v;
    else return ((V)v << 32) | (V)(uint32_t)i;
}

// (A bound of five or six waves per SIMD, which the LDS would allow, spills: 47
// against 42 us per pass of 7.3M instances.)
template <typename VIN, typename V, int BITS, int ITEMS, bool FOLD>
__global__ __launch_bounds__(RS_THREADS) void k_rs_scatter(const uint32_t* __restrict__ keys_in,
                                                           const VIN* __restrict__ vals_in, int64_t n_host,
                                                           const uint32_t* __restrict__ n_dev, int shift,
                                                           uint32_t* __restrict__ ws_a, uint32_t* __restrict__ ws_b,
                                                           const uint32_t* __restrict__ dtot,
                                                           uint32_t* __restrict__ keys_out,
                                                           V* __restrict__ vals_out) {
    constexpr int NB = 1 << BITS, TILE = RS_THREADS * ITEMS;
    __shared__ uint32_t s_cnt[4][NB];   // per-wave running digit counts, then wave prefixes
    __shared__ uint32_t s_dstart[NB];   // tile-local start of each digit
    __shared__ uint32_t s_goff[NB];     // global start of each digit for this tile
    __shared__ uint32_t s_dbase[NB];    // global start of each digit
    __shared__ uint32_t s_wave[4];
    __shared__ uint32_t s_keys[TILE];
    __shared__ V s_vals[TILE];

    const int64_t n = rs_n(n_host, n_dev);
    const RadixTab tab = radix_tab(n, ITEMS, FOLD ? 1 : 0, ws_a, ws_b);
    const int tiles = (int)((n + TILE - 1) / TILE);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    if (!FOLD && (int)blockIdx.x < tiles) {  // the block has a tile (uniform per block)
        uint32_t ex;
        block_excl_scan_256(threadIdx.x < NB ? dtot[threadIdx.x] : 0u, s_wave, &ex);
        if (threadIdx.x < NB) s_dbase[threadIdx.x] = ex;
    }
    for (int nth = blockIdx.x; nth < tiles; nth += gridDim.x) {
        const int tile = xcd_band(nth, tiles);
        for (int k = threadIdx.x; k < 4 * NB; k += RS_THREADS) (&s_cnt[0][0])[k] = 0;
        __syncthreads();

        const int64_t base = (int64_t)tile * TILE;
        const uint32_t tile_n = (uint32_t)((n - base) < TILE ? (n - base) : TILE);
        const uint32_t* kp = keys_in + base;
        const VIN* vp = vals_in + base;
        const uint32_t l0 = (uint32_t)w * (64 * ITEMS) + (uint32_t)lane;  // the thread's first element of the tile
        uint32_t key[ITEMS];
        V val[ITEMS];
        uint32_t rank[ITEMS];
        // all loads first, without branches (a lane past the end reads the last element)
#pragma unroll
        for (int k = 0; k < ITEMS; ++k) {
            const uint32_t li = l0 + k * 64, lc = li < tile_n ? li : tile_n - 1u;
            key[k] = kp[lc];
            val[k] = rs_value<VIN, V>(vp[lc], base + lc);
        }
        uint32_t tot = 0, prior_tiles = 0;
        if (FOLD && threadIdx.x < NB) {
            // the tiles' counts, tile-major: the earlier tiles' sum and the total
            constexpr int FU = 32;  // loads in flight
            for (int t0 = 0; t0 < tiles; t0 += FU) {
                uint32_t x[FU];
#pragma unroll
                for (int k = 0; k < FU; ++k) x[k] = tab.hist[(t0 + k < tiles ? t0 + k : 0) * NB + threadIdx.x];
#pragma unroll
                for (int k = 0; k < FU; ++k) {
                    tot += t0 + k < tiles ? x[k] : 0u;
                    prior_tiles += t0 + k < tile ? x[k] : 0u;
                }
            }
        }
#pragma unroll
        for (int k = 0; k < ITEMS; ++k) {
            const bool valid = l0 + k * 64 < tile_n;
            const uint32_t d = (key[k] >> shift) & (NB - 1u);
            // the lanes with the same digit: per digit bit, its ballot where the lane's
            // bit is set, else the ballot's complement (sx = -1 or 0)
            const uint64_t vb = __builtin_amdgcn_ballot_w64(valid);
            uint32_t lo = (uint32_t)vb, hi = (uint32_t)(vb >> 32);
#pragma unroll
            for (int b = 0; b < BITS; ++b) {
                const uint32_t sx = (uint32_t)__builtin_amdgcn_sbfe((int)key[k], (uint32_t)(shift + b), 1u);
                const uint64_t bb = __builtin_amdgcn_ballot_w64(sx != 0u);
                lo &= ~((uint32_t)bb ^ sx);
                hi &= ~((uint32_t)(bb >> 32) ^ sx);
            }
            uint32_t prior = 0;
            if (valid) prior = s_cnt[w][d];
            const uint32_t before = __builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, 0u));
            const uint32_t all = (uint32_t)(__popc(lo) + __popc(hi));
            rank[k] = prior + before;
            // the highest lane of each digit group publishes the new count
            if (valid && before + 1u == all) s_cnt[w][d] = prior + all;
        }
        if (FOLD) {
            uint32_t ex;
            block_excl_scan_256(tot, s_wave, &ex);
            if (threadIdx.x < NB) s_goff[threadIdx.x] = ex + prior_tiles;
        }
        __syncthreads();
        {
            const int d = threadIdx.x;
            uint32_t c = 0;
            if (d < NB) {
                const uint32_t c0 = s_cnt[0][d], c1 = s_cnt[1][d], c2 = s_cnt[2][d], c3 = s_cnt[3][d];
                s_cnt[0][d] = 0;
                s_cnt[1][d] = c0;
                s_cnt[2][d] = c0 + c1;
                s_cnt[3][d] = c0 + c1 + c2;
                c = c0 + c1 + c2 + c3;
                if (!FOLD) s_goff[d] = s_dbase[d] + radix_tile_offset(tab, NB, tile, d);
            }
            uint32_t ex;
            block_excl_scan_256(c, s_wave, &ex);
            if (d < NB) {
                s_dstart[d] = ex;
                s_goff[d] -= ex;  // from here on relative to the tile's first element
            }
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < ITEMS; ++k) {
            if (l0 + k * 64 >= tile_n) continue;
            const uint32_t d = (key[k] >> shift) & (NB - 1u);
            const uint32_t p = s_dstart[d] + s_cnt[w][d] + rank[k];
            s_keys[p] = key[k];
            s_vals[p] = val[k];
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < ITEMS; ++k) {
            const uint32_t p = k * RS_THREADS + threadIdx.x;
            if (p < tile_n) {
                const uint32_t kk = s_keys[p];
                const uint32_t o = s_goff[(kk >> shift) & (NB - 1u)] + p;
                keys_out[o] = kk;
                vals_out[o] = s_vals[p];
            }
        }
        __syncthreads();  // LDS is reused by the next tile
    }
}

// A digit's counts per 512- or 2048-key tile, twice (counts and offsets), and
// its total.
size_t radix_ws_bytes(int64_t n) {
    const int64_t small = n < RS_SMALL_KEYS ? n : RS_SMALL_KEYS;
    int64_t tiles = (n + RGS_RADIX_TILE - 1) / RGS_RADIX_TILE, ts = (small + 2 * RS_THREADS - 1) / (2 * RS_THREADS);
    if (tiles < ts) tiles = ts;
    if (tiles < 2) tiles = 2;
    size_t h = (size_t)256 * tiles * sizeof(uint32_t);
    return 2 * ((h + 255) & ~size_t(255)) + 256 * sizeof(uint32_t) + 512;
}

RadixWs radix_ws(void* ws, const RadixPlan& p) {
    const size_t h = (size_t)256 * (p.tiles < 2 ? 2 : p.tiles) * sizeof(uint32_t), hpad = (h + 255) & ~size_t(255);
    char* b = reinterpret_cast<char*>(ws);
    return RadixWs{reinterpret_cast<uint32_t*>(b), reinterpret_cast<uint32_t*>(b + hpad),
                   reinterpret_cast<uint32_t*>(b + 2 * hpad)};
}

template <typename VIN, typename V, int BITS, int ITEMS>
static void radix_pass(const uint32_t* ki, const VIN* vi, uint32_t* ko, V* vo, int64_t n, const uint32_t* n_dev, int shift,
                       const RadixPlan& p, bool hist_ready, const RadixWs& w, hipStream_t s) {
    const unsigned grid = (unsigned)(n_dev && p.tiles > DEV_GRID ? DEV_GRID : p.tiles);
    if (!hist_ready)
        hipLaunchKernelGGL(HIP_KERNEL_NAME(k_rs_hist<BITS, ITEMS>), dim3(grid), dim3(RS_THREADS), 0, s, ki, n, n_dev, shift,
                           p.fold, w.a, w.b);
    if (!p.fold)
        hipLaunchKernelGGL(k_rs_colscan, dim3(1 << BITS), dim3(RS_THREADS), 0, s, n, n_dev, p.items, w.a, w.b, w.dtot);
    if (p.fold)
        hipLaunchKernelGGL(HIP_KERNEL_NAME(k_rs_scatter<VIN, V, BITS, ITEMS, true>), dim3(grid), dim3(RS_THREADS), 0, s, ki,
                           vi, n, n_dev, shift, w.a, w.b, w.dtot, ko, vo);
    else if constexpr (ITEMS > 2)  // (512-key tiles are always few)
        hipLaunchKernelGGL(HIP_KERNEL_NAME(k_rs_scatter<VIN, V, BITS, ITEMS, false>), dim3(grid), dim3(RS_THREADS), 0, s, ki,
                           vi, n, n_dev, shift, w.a, w.b, w.dtot, ko, vo);
}

template <typename VIN, typename V, int ITEMS>
static void radix_pass_bits(int bits, const uint32_t* ki, const VIN* vi, uint32_t* ko, V* vo, int64_t n,
                            const uint32_t* n_dev, int shift, const RadixPlan& p, bool hist_ready, const RadixWs& w,
                            hipStream_t s) {
    switch (bits) {
        case 6: radix_pass<VIN, V, 6, ITEMS>(ki, vi, ko, vo, n, n_dev, shift, p, hist_ready, w, s); break;
        case 7: radix_pass<VIN, V, 7, ITEMS>(ki, vi, ko, vo, n, n_dev, shift, p, hist_ready, w, s); break;
        default: radix_pass<VIN, V, 8, ITEMS>(ki, vi, ko, vo, n, n_dev, shift, p, hist_ready, w, s); break;
    }
}

// FIRST: the first pass reads 4-byte sources from the start of its value buffer
// and its histogram is in ws already (the producer wrote it).
template <typename V, bool FIRST>
static rgs_status radix_sort_impl(uint32_t* keys, V* vals, uint32_t* keys_alt, V* vals_alt, int64_t n,
                                  const uint32_t* n_dev, const RadixPlan& p, void* ws, hipStream_t s) {
    if (n <= 0) return RGS_OK;
    const RadixWs w = radix_ws(ws, p);
    const bool odd = p.passes & 1;
    uint32_t *ki = odd ? keys_alt : keys, *ko = odd ? keys : keys_alt;
    V *vi = odd ? vals_alt : vals, *vo = odd ? vals : vals_alt;
    int shift = 0;
    for (int k = 0; k < p.passes; ++k) {
        if (FIRST && k == 0) {
            const uint32_t* v32 = reinterpret_cast<const uint32_t*>(vi);
            if (p.items == 2) radix_pass_bits<uint32_t, V, 2>(p.bits[k], ki, v32, ko, vo, n, n_dev, shift, p, true, w, s);
            else radix_pass_bits<uint32_t, V, 8>(p.bits[k], ki, v32, ko, vo, n, n_dev, shift, p, true, w, s);
        } else {
            if (p.items == 2) radix_pass_bits<V, V, 2>(p.bits[k], ki, vi, ko, vo, n, n_dev, shift, p, false, w, s);
            else radix_pass_bits<V, V, 8>(p.bits[k], ki, vi, ko, vo, n, n_dev, shift, p, false, w, s);
        }
        RGS_LAUNCH_CHECK();
        shift += p.bits[k];
        uint32_t* tk = ki; ki = ko; ko = tk;
        V* tv = vi; vi = vo; vo = tv;
    }
    return RGS_OK;
}

rgs_status radix_sort_u32_u32(uint32_t* keys, uint32_t* vals, uint32_t* keys_alt, uint32_t* vals_alt, int64_t n,
                              const uint32_t* n_dev, const RadixPlan& p, void* ws, hipStream_t s) {
    return radix_sort_impl<uint32_t, false>(keys, vals, keys_alt, vals_alt, n, n_dev, p, ws, s);
}

rgs_status radix_sort_instances(uint32_t* keys, uint64_t* vals, uint32_t* keys_alt, uint64_t* vals_alt, int64_t n,
                                const uint32_t* n_dev, const RadixPlan& p, void* ws, hipStream_t s) {
    return radix_sort_impl<uint64_t, true>(keys, vals, keys_alt, vals_alt, n, n_dev, p, ws, s);
}

}  // namespace rgs
