// layout.hip -- a copy of the Gaussians grouped by the KD leaf of their
// centre (each sub-model's subset of Sec. 3.3 contiguous in memory), ordered
// inside a leaf along a Morton curve over the leaf's bounds.  Views that
// cannot see a cell then skip a contiguous index range whose parameters are
// never fetched, and Gaussians visible together share cache lines.
//
// Key = leaf << 24 | interleaved 8-bit coordinates of the centre quantised
// to the leaf's centre-bounds box; a stable radix sort on the key keeps gid
// order among equal keys, so the permutation is deterministic.
#include "common.hpp"

namespace rgs {

static constexpr int LY_THREADS = 256;

__device__ __forceinline__ uint32_t spread3_8(uint32_t v) {  // bit b of v -> bit 3b
    v &= 0xffu;
    v = (v | (v << 8)) & 0x0000f00fu;
    v = (v | (v << 4)) & 0x000c30c3u;
    v = (v | (v << 2)) & 0x00249249u;
    return v;
}

__global__ __launch_bounds__(LY_THREADS) void k_group_keys(const float* __restrict__ means,
                                                           const int32_t* __restrict__ center_cell,
                                                           const float* __restrict__ cell_bounds, int K, int64_t n,
                                                           uint32_t* __restrict__ keys, uint32_t* __restrict__ idx) {
    const int64_t i = (int64_t)blockIdx.x * LY_THREADS + threadIdx.x;
    if (i >= n) return;
    const int cell = center_cell[i];
    uint32_t code = 0;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const float lo = cell_bounds[a * K + cell], hi = cell_bounds[(3 + a) * K + cell];
        const float x = means[a * n + i];
        const float u = hi > lo ? (x - lo) / (hi - lo) : 0.0f;
        const int q = (int)fminf(fmaxf(u * 256.0f, 0.0f), 255.0f);
        code |= spread3_8((uint32_t)q) << a;
    }
    keys[i] = ((uint32_t)cell << 24) | code;
    idx[i] = (uint32_t)i;
}

// The gather out[j] = in[perm[j]] of all rows directly: bound by HBM at 8 bytes per
// (row, Gaussian) where neighbours come from neighbours; from random places each 4
// bytes read move a line.
__device__ __forceinline__ void gather_direct(const rgs_gaussians& in, const rgs_gaussians& out, int rows,
                                              const uint32_t* __restrict__ perm, int32_t* __restrict__ perm_out, int64_t j) {
    const int64_t n = in.n;
    if (j >= n) return;
    const int64_t s = perm[j];
    constexpr int U = 8;  // loads in flight
    for (int r0 = 0; r0 < rows; r0 += U) {
        float v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = r0 + u < rows ? param_row(in, n, r0 + u)[s] : 0.f;
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (r0 + u < rows) const_cast<float*>(param_row(out, n, r0 + u))[j] = v[u];
    }
    if (perm_out) perm_out[j] = (int32_t)s;
}

__global__ __launch_bounds__(LY_THREADS) void k_gather_direct(rgs_gaussians in, rgs_gaussians out, int rows,
                                                              const uint32_t* __restrict__ perm,
                                                              int32_t* __restrict__ perm_out) {
    gather_direct(in, out, rows, perm, perm_out, (int64_t)blockIdx.x * LY_THREADS + threadIdx.x);
}

// The gather out[j] = in[perm[j]] of all rows, LY_ROWS rows at a time through
// a staged copy in which the LY_ROWS values of a Gaussian are one aligned
// 64-byte line.  A direct gather reads 4 bytes per (row, Gaussian) from a
// random place and so moves a whole line for each; here the random reads are
// lines used in full and everything else is coalesced (the two transposes go
// through LDS).  Bound by HBM: per row group 4 x 4 bytes per (row, Gaussian).
// Keys, sort and gather of 16M Gaussians, SH 3 (59 rows): 16.2 ms with the direct
// gather, 3.9 ms so (floor of the rows read and written once: 1.5 ms).
// Where neighbours mostly come from neighbours the first launch gathers directly and
// the others end: with a share c near the direct gather moves about 8 c + 68 (1 - c)
// bytes per value, the staged one 16, the same at 87 %.
static constexpr int LY_ROWS = 16;
static constexpr int64_t LY_DIRECT = 131072;
static constexpr int LY_LDW = LY_ROWS + 1;  // LDS row of a Gaussian: odd, so that neither side of a transpose conflicts

__global__ __launch_bounds__(LY_THREADS) void k_stage_rows(rgs_gaussians in, rgs_gaussians out, int r0, int nr, int rows,
                                                           const uint32_t* __restrict__ perm,
                                                           int32_t* __restrict__ perm_out, float* __restrict__ stage) {
    if (perm_mostly_near(perm, in.n)) {
        if (r0 == 0) gather_direct(in, out, rows, perm, perm_out, (int64_t)blockIdx.x * LY_THREADS + threadIdx.x);
        return;
    }
    __shared__ float s[LY_THREADS * LY_LDW];
    const int64_t n = in.n, base = (int64_t)blockIdx.x * LY_THREADS;
    const int t = threadIdx.x;
    const int64_t i = base + t;
    float v[LY_ROWS];
#pragma unroll
    for (int r = 0; r < LY_ROWS; ++r) v[r] = (r < nr && i < n) ? param_row(in, n, r0 + r)[i] : 0.f;
#pragma unroll
    for (int r = 0; r < LY_ROWS; ++r) s[t * LY_LDW + r] = v[r];
    __syncthreads();
    const int64_t left = (n - base) * LY_ROWS;
#pragma unroll
    for (int k = 0; k < LY_ROWS; ++k) {
        const int e = k * LY_THREADS + t;
        if (e < left) stage[base * LY_ROWS + e] = s[(e / LY_ROWS) * LY_LDW + e % LY_ROWS];
    }
}

__global__ __launch_bounds__(LY_THREADS) void k_gather_rows(const float* __restrict__ stage, rgs_gaussians out, int r0,
                                                            int nr, const uint32_t* __restrict__ perm,
                                                            int32_t* __restrict__ perm_out) {
    if (perm_mostly_near(perm, out.n)) return;
    __shared__ float s[LY_THREADS * LY_LDW];
    const int64_t n = out.n, base = (int64_t)blockIdx.x * LY_THREADS;
    const int t = threadIdx.x;
    constexpr int Q = LY_ROWS / 4;  // float4 per Gaussian, one lane each
    float4 v[Q];
#pragma unroll
    for (int k = 0; k < Q; ++k) {
        const int e = k * LY_THREADS + t;
        const int64_t j = base + e / Q;
        v[k] = reinterpret_cast<const float4*>(stage)[(size_t)perm[j < n ? j : n - 1] * Q + e % Q];
    }
#pragma unroll
    for (int k = 0; k < Q; ++k) {
        const int e = k * LY_THREADS + t;
        float* d = s + (e / Q) * LY_LDW + 4 * (e % Q);
        d[0] = v[k].x;
        d[1] = v[k].y;
        d[2] = v[k].z;
        d[3] = v[k].w;
    }
    __syncthreads();
    const int64_t j = base + t;
    if (j >= n) return;
#pragma unroll
    for (int r = 0; r < LY_ROWS; ++r)
        if (r < nr) const_cast<float*>(param_row(out, n, r0 + r))[j] = s[t * LY_LDW + r];
    if (perm_out) perm_out[j] = (int32_t)perm[j];
}

// The sorted index stays while the rows are moved; the other sort buffers'
// place is the staged copy's.
size_t group_ws_bytes(int64_t n) {
    WsCarver c{nullptr, 0, 0};
    c.take<uint32_t>(n + 1);
    const size_t first = c.used;
    for (int k = 0; k < 3; ++k) c.take<uint32_t>(n + 1);
    c.take<char>(radix_ws_bytes(n + 1));
    WsCarver d{nullptr, first, 0};
    d.take<float>((size_t)LY_ROWS * n);
    return (c.used > d.used ? c.used : d.used) + 256;
}

rgs_status group_by_cell(const rgs_gaussians* in, const rgs_kdtree* kd, int L, const rgs_gaussians* out,
                         int32_t* perm, void* ws, size_t ws_bytes, hipStream_t s) {
    const int64_t n = in->n;
    if (n <= 0) return RGS_OK;
    if (ws_bytes < group_ws_bytes(n)) return RGS_E_ARG;
    WsCarver c{reinterpret_cast<char*>(ws), 0, ws_bytes};
    uint32_t* idx = c.take<uint32_t>(n + 1);
    WsCarver d = c;
    uint32_t* keys = c.take<uint32_t>(n + 1);
    uint32_t* keys_alt = c.take<uint32_t>(n + 1);
    uint32_t* idx_alt = c.take<uint32_t>(n + 1);
    void* rws = c.take<char>(radix_ws_bytes(n + 1));
    float* stage = d.take<float>((size_t)LY_ROWS * n);
    const unsigned grid = (unsigned)((n + LY_THREADS - 1) / LY_THREADS);
    hipLaunchKernelGGL(k_group_keys, dim3(grid), dim3(LY_THREADS), 0, s, in->means, kd->center_cell, kd->cell_bounds,
                       1 << L, n, keys, idx);
    RGS_LAUNCH_CHECK();
    // 24 + L bits: four passes, an even number, so the input starts in keys / idx
    rgs_status st = radix_sort_u32_u32(keys, idx, keys_alt, idx_alt, n, nullptr, radix_plan(n, 25 > 24 + L ? 25 : 24 + L), rws, s);
    if (st != RGS_OK) return st;
    const int rows = 11 + 3 * (in->sh_degree + 1) * (in->sh_degree + 1);
    // up to LY_DIRECT Gaussians the caches hold what is read, and launches count
    if (n <= LY_DIRECT) {
        hipLaunchKernelGGL(k_gather_direct, dim3(grid), dim3(LY_THREADS), 0, s, *in, *out, rows, idx, perm);
        return launch_check();
    }
    for (int r = 0; r < rows; r += LY_ROWS) {
        const int nr = rows - r < LY_ROWS ? rows - r : LY_ROWS;
        hipLaunchKernelGGL(k_stage_rows, dim3(grid), dim3(LY_THREADS), 0, s, *in, *out, r, nr, rows, idx, perm, stage);
        hipLaunchKernelGGL(k_gather_rows, dim3(grid), dim3(LY_THREADS), 0, s, stage, *out, r, nr, idx,
                           r == 0 ? perm : nullptr);
    }
    return launch_check();
}

}  // namespace rgs
