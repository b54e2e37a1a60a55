// render.hip -- per-cell partial blending (RetinaGS Eq. 3, Eq. 4 with the
// indicator of Eq. 6), its backward, and the per-pair gradient reduction.
//
// Forward: a 256-thread block per 16x16 tile walks the tile's slots (tile, cell) in
// merge order; wave w owns the 8x8 quadrant (w & 1, w >> 1), one pixel per lane.  The
// longest tiles are given to four blocks each, whose waves own 4x4 pixels and take
// four instances at a time.  The contribute decision d^2 <= tau uses the exact
// fp32 operation sequence the CPU oracle mirrors, on the factored form of the
// quadratic (no cancellation for elongated footprints):
//   dx = (x + 0.5) - mx, dy = (y + 0.5) - my, u = fma(k, dy, dx),
//   d^2 = fma(e dy, dy, (ca u) u).
// The conic (ca, cb, cc) = (ca, k ca, e + k cb) is rebuilt per instance where
// the quadrant test and the gradients need it.  Gaussian records are staged
// through LDS (one coalesced 64-byte record per thread) with a 4-bit mask of
// the quadrants their rectangle meets, and read
// back as wave-uniform broadcasts; a wave skips Gaussians outside its
// quadrant with a scalar branch.  A pixel stops after the contribution that
// takes its merged transmittance below eps_T; the block leaves once all its
// pixels stopped.
//
// Backward (a 128-thread block per slot, two pixels of one row per lane)
// walks each slot back to front from the largest per-pixel `last`, recovers
// the transmittance before every contribution from a reciprocal, adds each
// lane's two pixels and sums each instance's gradient over the wave's 128
// pixels with a reduce-scatter butterfly (no atomics), adds the two half-tile
// sums in a fixed order and stores one record (9 floats, 36 bytes) at the
// instance's emission position; a segmented reduction then sums each pair's
// records (contiguous by construction) in a fixed order.
#include "common.hpp"

namespace rgs {

static constexpr int RD_BATCH = 64;
static constexpr int RD_REC = 9;   // floats per backward record (36 bytes, read back contiguously)
// A pair's flag: no record (0), its entry is the sum of its records, or (pairs whose
// instances span several waves) the range of waves whose partials make it up.
static constexpr uint8_t PS_SUM = 1, PS_SPAN = 2;
static constexpr int PS_REC = 12;  // floats per per-pair / per-wave sum (48 bytes, float4-aligned)
// The backward's launch order: slots per block of its two passes, and the
// size classes (half octaves of the instances a slot is walked over)
static constexpr int SW_SLOTS = 64;
static constexpr int SW_CLS = 64;

struct SlotGeom {
    int v, px, py0, cell;
    bool ok;
};

__device__ __forceinline__ SlotGeom slot_geom(const ViewTable* __restrict__ vt, uint32_t key, int L) {
    SlotGeom g;
    const uint32_t gt = key >> L;
    const uint32_t rank = key & ((1u << L) - 1u);
    g.v = view_of_tile(vt, gt);
    const ViewParams& V = vt->v[g.v];
    const uint32_t lt = gt - V.tile_offset;
    const int tx = (int)(lt % (uint32_t)V.tiles_x), ty = (int)(lt / (uint32_t)V.tiles_x);
    const int lane = lane_id();
    g.px = tx * 16 + (lane & 15);
    g.py0 = ty * 16 + (lane >> 4);
    g.cell = V.cell_of_rank[rank];
    g.ok = true;
    return g;
}

// Quadrant mask of a Gaussian's rectangle within tile (tx, ty): bit q set iff
// the rectangle meets 8x8 quadrant q = 2 qy + qx of the 16x16 tile.
__device__ __forceinline__ uint32_t quad_mask(uint2 rr, int tx, int ty) {
    const int x0 = (int)(int16_t)(rr.x & 0xffffu) - tx * 16, x1 = (int)(int16_t)(rr.x >> 16) - tx * 16;
    const int y0 = (int)(int16_t)(rr.y & 0xffffu) - ty * 16, y1 = (int)(int16_t)(rr.y >> 16) - ty * 16;
    const uint32_t mx = ((x0 <= 7 && x1 >= 0) ? 1u : 0u) | ((x0 <= 15 && x1 >= 8) ? 2u : 0u);
    const uint32_t my = ((y0 <= 7 && y1 >= 0) ? 1u : 0u) | ((y0 <= 15 && y1 >= 8) ? 2u : 0u);
    uint32_t m = 0;
    if (my & 1u) m |= mx;
    if (my & 2u) m |= mx << 2;
    return m;
}

// Can a pixel centre of the wx-by-wy block of pixels whose first pixel is
// (x0, y0) pass the fp32 decision d^2 <= tau?  The minimum of the quadratic
// form over the box of the block's pixel centres is 0 if the mean is inside,
// else the least of its four edge minima (a convex function of one variable
// each, minimised at the clamped stationary point).  Against the fp32
// sequence used per pixel the test adds a margin of 2^-18 (ca dx^2 + cc dy^2)
// at the box's far corner, above the rounding error of both evaluations (a
// few ulp of |ca dx^2| + 2|cb dx dy| + |cc dy^2| <= 2 (ca dx^2 + cc dy^2)),
// plus 2^-20 tau: a block is only dropped when no pixel can contribute.
__device__ __forceinline__ bool box_hits(float mx, float my, float ca, float cb, float cc, float tau, float x0,
                                         float y0, float wx, float wy) {
    const float lx = (x0 + 0.5f) - mx, hx = (x0 + (wx - 0.5f)) - mx;
    const float ly = (y0 + 0.5f) - my, hy = (y0 + (wy - 0.5f)) - my;
    if (lx <= 0.0f && hx >= 0.0f && ly <= 0.0f && hy >= 0.0f) return true;
    const float ica = __builtin_amdgcn_rcpf(ca), icc = __builtin_amdgcn_rcpf(cc);
    float qmin = INFINITY;
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        const float ex = e ? hx : lx;  // vertical edge dx = ex
        const float dy = fminf(fmaxf(-(cb * ex) * icc, ly), hy);
        qmin = fminf(qmin, (ca * ex) * ex + dy * (2.0f * cb * ex + cc * dy));
        const float ey = e ? hy : ly;  // horizontal edge dy = ey
        const float dx = fminf(fmaxf(-(cb * ey) * ica, lx), hx);
        qmin = fminf(qmin, (cc * ey) * ey + dx * (2.0f * cb * ey + ca * dx));
    }
    const float far = ca * fmaxf(lx * lx, hx * hx) + cc * fmaxf(ly * ly, hy * hy);
    return qmin <= tau + 0x1p-18f * far + 0x1p-20f * tau;
}

#define RGS_DPP(v, ctrl) __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, (v)), (ctrl), 0xf, 0xf, false))

// Lane mask of a comparison (the compare writes it to scalar registers).
__device__ __forceinline__ uint64_t wmask(bool p) { return __builtin_amdgcn_ballot_w64(p); }

// 4x4 blocks of the pixel row band by .. by + 3, from column bx on, that the
// footprint can reach: bit c = block column c < 2.  The band's
// span of columns as in row_span, with the hardware's reciprocal and square
// root; the enlargement of tau and the pads at the ends are four times those of
// row_span, above the error of both the per-pixel test and these, so a block
// is only dropped when none of its pixels can contribute.
__device__ __forceinline__ uint32_t block_row_mask(float4 a, float4 b, uint2 rr, int bx, int by, bool rect_only) {
    const int x_lo = (int)(int16_t)(rr.x & 0xffffu), x_hi = (int)(int16_t)(rr.x >> 16);
    const int y_lo = (int)(int16_t)(rr.y & 0xffffu), y_hi = (int)(int16_t)(rr.y >> 16);
    const int y0 = max(by, y_lo), y1 = min(by + 3, y_hi);
    float lo = (float)x_lo, hi = (float)x_hi;
    if (!rect_only) {
        const float mx = a.x, my = a.y, ca = a.z, k = a.w, e = b.x, tau = b.z;
        const float ica = __builtin_amdgcn_rcpf(ca), ie = __builtin_amdgcn_rcpf(e), q = (k * k) * ca;
        const float rk = __builtin_amdgcn_sqrtf(fmaf(q, ie, 1.0f));
        const float taup = fmaf(tau, 0x1p-16f * (1.0f + rk), tau);
        const float dyr = -(k * __builtin_amdgcn_sqrtf((ca * taup) * (ie * __builtin_amdgcn_rcpf(e + q))));
        const float ly = ((float)y0 + 0.5f) - my, hy = ((float)y1 + 0.5f) - my;
        const float dR = fminf(fmaxf(dyr, ly), hy), dL = fminf(fmaxf(-dyr, ly), hy);
        const float xr = mx + (__builtin_amdgcn_sqrtf(fmaxf(taup - e * (dR * dR), 0.0f) * ica) - k * dR);
        const float xl = mx - (__builtin_amdgcn_sqrtf(fmaxf(taup - e * (dL * dL), 0.0f) * ica) + k * dL);
        const float pr = 0x1p-4f + 0x1p-14f * (fabsf(mx) + fabsf(xr - mx));
        const float pl = 0x1p-4f + 0x1p-14f * (fabsf(mx) + fabsf(xl - mx));
        // an end that is not finite leaves the rectangle's bound
        if (fabsf(xl) < INFINITY && fabsf(xr) < INFINITY && fabsf(dyr) < INFINITY) {
            lo = fmaxf((xl - pl) - 0.5f, lo);
            hi = fminf((xr + pr) - 0.5f, hi);
        }
    }
    // pixels lo .. hi (rounded outwards) to block columns
    const int c0 = max(((int)floorf(lo) - bx) >> 2, 0), c1 = min(((int)floorf(hi) - bx) >> 2, 1);
    if (y0 > y1 || !(lo <= hi) || c0 > c1) return 0u;
    return (2u << c1) - (1u << c0);
}

// Forward: one 256-thread block per tile, walking the tile's slots (one per
// cell that has instances there) in the view's merge order; wave w owns the
// 8x8 quadrant (w & 1, w >> 1) of the tile, one pixel per lane.  Each pixel
// carries P, the product of the T_k of the slots already done: the merged
// transmittance in front of the current cell.  Within a slot, T_k starts at
// 1 and P T_k is the merged transmittance, so a pixel stops (in this cell
// and all later ones) after the contribution that takes P T_k below eps_T:
// the plain render's early termination, which a pixel reaches in the cell
// where it happens, so cells behind an opaque front are not rendered there
// (their partial stays C = 0, T = 1, last = 0).  Records are staged 256 at a
// time in LDS, each with the quadrant mask of its rectangle so that a wave
// skips Gaussians that cannot touch its quadrant with a scalar branch.
//
// A tile's list is a serial chain, and a wave alone on its SIMD issues an
// instruction about every eight clocks (400 clocks per instance here), so the
// tiles with the longest lists were the kernel's time for small and middle
// views (300k Gaussians at 997x663: all other tiles done in 95 us, the last at
// 246).  The RF_HEAVY first tiles of the launch order are therefore given to
// four blocks each, one per quadrant, whose waves own 4x4 pixels and take four
// instances at a time: lane = 4 pixel + instance for the sigmas, the
// transmittances passed along the quad by DPP, lane = 4 pixel + channel for the
// colours, which are added instance by instance.  Every value is formed by the
// same operations in the same order as with a pixel per lane, so the results
// are the same bits and the choice is free.  A wave's list holds only the
// records whose ellipse reaches its 4x4 block.  This costs twice the
// instructions per (pixel, instance) pair, so it is not for every tile: with
// all tiles so, 300k Gaussians take 120 us and 20k at 256x256 30, but 1M at
// 1920x1080 293 instead of 212 and 16M at 3840x2160 990 instead of 550.  How many
// is a matter of the views measured, in us, before / with the first 128 / 256 / 512
// tiles: 20k at 256x256 66 / 28 / 28 / 28; 150k at 1237x823 165 / 123 / 127 / more; 300k
// at 997x663 228 / 128 / 128 / more; 1M at 1600x1060 312 / 300 / 228; 16M at 3840x2160
// 551 / 523 / 519.  A view without long tiles pays for it: 1M at 1920x1080, four
// scenes, none / 256: 206 / 213, 212 / 215, 195 / 196, 192 / 200; so does one of next to
// nothing in many cells (300 Gaussians at 500x333, 64 cells: 66 / 90).  Asking each of
// the 256 for its share of the instances first, and taking the short ones whole, costs
// as much as it saves (the three blocks that then end have waited for the tile's
// range: 218 to 221 us at 1920x1080 for any share asked).
// 64 registers keep 8 waves per SIMD (72 and 7 waves: 246 at 1920x1080).
static constexpr uint32_t RF_HEAVY = 256;

template <bool STATS>
__global__ __launch_bounds__(256, 8) void k_render_fwd(const float* __restrict__ rec,
                                                    const uint64_t* __restrict__ vals,
                                                    const uint32_t* __restrict__ slot_key,
                                                    const uint32_t* __restrict__ slot_range,
                                                    const uint32_t* __restrict__ tile_slot,
                                                    const uint32_t* __restrict__ tile_order, uint32_t n_heavy,
                                                    const ViewTable* __restrict__ vt, const float* __restrict__ box_lo,
                                                    const float* __restrict__ box_hi, float eps_T,
                                                    float* __restrict__ outC, float* __restrict__ outT,
                                                    uint32_t* __restrict__ outLast,
                                                    unsigned long long* __restrict__ stats,
                                                    float* __restrict__ image, float* __restrict__ T_final) {
    constexpr int NB = 256;
    // record NB never contributes (tau < 0): it fills a list's last group of four
    __shared__ float4 sA[NB + 1], sB[NB + 1], sCl[NB + 1];
    __shared__ uint32_t sM[NB];
    __shared__ uint2 sR[STATS ? NB : 1];
    __shared__ uint32_t s_flag[2][4];
    __shared__ __align__(8) uint16_t s_list[4][NB + 8];
    const bool heavy = blockIdx.x < 4 * n_heavy;
    const uint32_t gt = tile_order[heavy ? blockIdx.x >> 2 : blockIdx.x - 3 * n_heavy];
    const uint32_t s0 = tile_slot[gt], s1 = tile_slot[gt + 1];
    if (s0 >= s1 && !image) return;
    const int L = vt->L, K = 1 << L;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int v = view_of_tile(vt, gt);
    const ViewParams& V = vt->v[v];
    const uint32_t lt = gt - V.tile_offset;
    const int tx = (int)(lt % (uint32_t)V.tiles_x), ty = (int)(lt / (uint32_t)V.tiles_x);
    const float o0 = V.o[0], o1 = V.o[1], o2 = V.o[2];
    uint32_t n_eval = 0u, n_con = 0u;

    if (heavy) {
        const int quadr = (int)(blockIdx.x & 3u), inst = lane & 3, pix = lane >> 2;
        const int qlx = (quadr & 1) * 8, qly = (quadr >> 1) * 8;                       // the block's quadrant in the tile
        const int lx = qlx + (w & 1) * 4 + (pix & 3), ly = qly + (w >> 1) * 4 + (pix >> 2);
        const int px = tx * 16 + lx, py = ty * 16 + ly, p = ly * 16 + lx;
        const float fxp = (float)px + 0.5f, fyp = (float)py + 0.5f;
        const float dxp = (fxp - V.cx) / V.fx, dyp = (fyp - V.cy) / V.fy;
        const float D0 = (V.R[0] * dxp + V.R[3] * dyp) + V.R[6];
        const float D1 = (V.R[1] * dxp + V.R[4] * dyp) + V.R[7];
        const float D2 = (V.R[2] * dxp + V.R[5] * dyp) + V.R[8];
        const bool on_image = px < V.W && py < V.H;
        bool live = on_image;
        float P = 1.0f, M = 0.f;  // M: the merged colour's channel `inst`
        if (tid == 0) {
            sA[NB] = sCl[NB] = make_float4(0.f, 0.f, 0.f, 0.f);
            sB[NB] = make_float4(0.f, 0.f, -1.f, 0.f);
        }
        // the source of the next batch's record is loaded ahead
        uint32_t src = 0;
        const uint32_t* vhi = reinterpret_cast<const uint32_t*>(vals) + 1;  // high words: the sources
        auto next_src = [&](uint32_t at, uint32_t lim) {  // of the slot that ends at lim (past it: its last instance)
            const uint32_t i = at + (uint32_t)tid;
            src = vhi[2 * (size_t)(i < lim ? i : max(lim, 1u) - 1u)];
        };
        if (s0 < s1) next_src(slot_range[2 * s0], slot_range[2 * s0 + 1]);
        int par = 0;  // parity of the batch (its flags are read while the next one's are written)
        for (uint32_t slot = s0; slot < s1; ++slot) {
            const uint32_t key = slot_key[slot];
            const uint32_t begin = slot_range[2 * slot], end = slot_range[2 * slot + 1];
            // the tile's next slot, which need not follow in the list (a caller's table of some cells)
            const uint32_t sn = slot + 1 < s1 ? slot + 1 : slot;
            const uint32_t sn_begin = slot_range[2 * sn], sn_end = slot_range[2 * sn + 1];
            const int cell = V.cell_of_rank[key & ((1u << L) - 1u)];
            const float blo0 = box_lo[cell], blo1 = box_lo[K + cell], blo2 = box_lo[2 * K + cell];
            const float bhi0 = box_hi[cell], bhi1 = box_hi[K + cell], bhi2 = box_hi[2 * K + cell];
            // a pixel that has stopped (or is off the image) takes no contribution; one that has
            // not takes at least one, also where P was rounded to just below eps_T (a
            // contribution leaves T below 1)
            const float thr = live ? fminf(eps_T / P, 1.0f) : INFINITY;
            float T = 1.0f, C = 0.f;  // C: channel `inst`
            uint32_t last = 0u;
            bool any_alive = false;
            for (uint32_t base = begin;;) {
                const int nb = (int)((end - base) < (uint32_t)NB ? (end - base) : (uint32_t)NB);
                const uint32_t next = base + (uint32_t)nb;  // the next batch of this slot, or the next slot's first
                const float4* rp = reinterpret_cast<const float4*>(rec) + 4 * (size_t)src;
                const float4 ra = rp[0], rb = rp[1], rc = rp[2];
                const float2 rr = *reinterpret_cast<const float2*>(rp + 3);
                sA[tid] = ra;
                sB[tid] = rb;
                sCl[tid] = make_float4(rc.x, rc.y, rc.z, __uint_as_float(base - begin + (uint32_t)tid + 1u));
                const uint2 rct = make_uint2(__float_as_uint(rr.x), __float_as_uint(rr.y));
                if (STATS) sR[tid] = rct;
                uint32_t m = 0u;
                if (tid < nb) {
                    const int bx = tx * 16 + qlx, by = ty * 16 + qly;
                    m = block_row_mask(ra, rb, rct, bx, by, STATS) | (block_row_mask(ra, rb, rct, bx, by + 4, STATS) << 2);
                    m |= (__float_as_uint(rc.w) & 1u) ? 0u : 16u;  // its footprint reaches several cells
                }
                sM[tid] = m;
                const uint64_t am = wmask(!(T < thr));
                // colours are >= 0: all finite if their sum is
                const uint64_t odd_m = wmask(tid < nb && !((rc.x + rc.y) + rc.z < INFINITY));
                if (lane == 0) s_flag[par][w] = (am != 0ull ? 1u : 0u) | (odd_m != 0ull ? 2u : 0u);
                if (next < end) next_src(next, end);
                else next_src(sn_begin, sn_end);
                __syncthreads();
                const uint32_t fl = s_flag[par][0] | s_flag[par][1] | s_flag[par][2] | s_flag[par][3];
                par ^= 1;
                any_alive = (fl & 1u) != 0u;
                if (!any_alive) break;
                if (am != 0ull) {
                    int cnt = 0;
#pragma unroll
                    for (int k = 0; k < NB / 64; ++k) {
                        const uint32_t mk = sM[k * 64 + lane];
                        const bool hit = (mk >> w) & 1u;
                        const uint64_t rel = wmask(hit);
                        const int at = cnt + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(rel >> 32),
                                                                            __builtin_amdgcn_mbcnt_lo((uint32_t)rel, 0u));
                        if (hit) s_list[w][at] = (uint16_t)(((k * 64 + lane) << 4) | (mk >> 4));
                        cnt += (int)__popcll(rel);
                    }
                    if (lane < 8) s_list[w][cnt + lane] = (uint16_t)(NB << 4);
                    __builtin_amdgcn_wave_barrier();
                    uint32_t en = s_list[w][inst];
                    for (int g = 0; g < cnt; g += 4) {
                        const uint32_t ad = en & 0xfff0u;
                        const bool mul = en & 1u;
                        en = s_list[w][g + 4 + inst];
                        const float4 ac = *reinterpret_cast<const float4*>(reinterpret_cast<const char*>(sA) + ad);
                        const float4 bc = *reinterpret_cast<const float4*>(reinterpret_cast<const char*>(sB) + ad);
                        const uint32_t idx = *reinterpret_cast<const uint32_t*>(reinterpret_cast<const char*>(sCl) + ad + 12);
                        // channel `inst` of the four instances' colours (the index for lane 3, unused)
                        float cv[4];
#define RGS_QUAD(i) (uint32_t)__builtin_amdgcn_update_dpp(0, (int)ad, (i) * 0x55, 0xf, 0xf, false)
                        cv[0] = *reinterpret_cast<const float*>(reinterpret_cast<const char*>(sCl) + RGS_QUAD(0) + 4 * inst);
                        cv[1] = *reinterpret_cast<const float*>(reinterpret_cast<const char*>(sCl) + RGS_QUAD(1) + 4 * inst);
                        cv[2] = *reinterpret_cast<const float*>(reinterpret_cast<const char*>(sCl) + RGS_QUAD(2) + 4 * inst);
                        cv[3] = *reinterpret_cast<const float*>(reinterpret_cast<const char*>(sCl) + RGS_QUAD(3) + 4 * inst);
#undef RGS_QUAD
                        const float dx = fxp - ac.x, dy = fyp - ac.y;
                        const float u = fmaf(ac.w, dy, dx);  // d^2 = ca u^2 + e dy^2
                        const float d2 = fmaf(bc.x * dy, dy, (ac.z * u) * u);
                        bool con = d2 <= bc.z;
                        if (wmask(mul) != 0ull) {  // the indicator of Eq. 6, where a footprint reaches several cells
                            const float x0 = fmaf(bc.w, D0, o0), x1 = fmaf(bc.w, D1, o1), x2 = fmaf(bc.w, D2, o2);
                            const bool in = (blo0 <= x0) && (x0 < bhi0) && (blo1 <= x1) && (x1 < bhi1) && (blo2 <= x2) &&
                                            (x2 < bhi2);
                            con = con && (in || !mul);
                        }
                        const float G = __builtin_amdgcn_exp2f(d2 * -0.72134752044448170368f);  // exp(-d^2/2)
                        const float sg = con ? fminf(0.99f, bc.y * G) : 0.0f;
                        const float a = 1.0f - sg;
                        // the transmittance after each instance of the quad, one product after another
                        // (DPP reads are made by all lanes, before any selection)
                        const float t0 = T * a;
                        const float t1 = RGS_DPP(t0, 0x00) * a;
                        const float t2 = RGS_DPP(t1, 0x55) * a;
                        const float t3 = RGS_DPP(t2, 0xaa) * a;
                        const float Ta = inst < 2 ? (inst == 0 ? t0 : t1) : (inst == 2 ? t2 : t3);
                        const float sb = RGS_DPP(Ta, 0x90);    // quad_perm [0,0,1,2]
                        const float Tb = inst >= 1 ? sb : T;   // ... and before it
                        const bool on = !(Tb < thr);           // included unless the pixel stopped before it
                        if (STATS) {
                            // pairs the method must test: pixel inside the Gaussian's rectangle, not yet stopped
                            const uint2 rr2 = sR[ad < (uint32_t)(NB << 4) ? ad >> 4 : 0u];
                            const bool inr = px >= (int)(int16_t)(rr2.x & 0xffffu) && px <= (int)(int16_t)(rr2.x >> 16) &&
                                             py >= (int)(int16_t)(rr2.y & 0xffffu) && py <= (int)(int16_t)(rr2.y >> 16);
                            n_eval += on && inr && ad < (uint32_t)(NB << 4) ? 1u : 0u;
                            n_con += on && con ? 1u : 0u;
                        }
                        const float wgt = on && con ? sg * Tb : -0.0f;  // (a weight has no sign)
                        last = on && con ? idx : last;
                        const float w0 = RGS_DPP(wgt, 0x00), w1 = RGS_DPP(wgt, 0x55), w2 = RGS_DPP(wgt, 0xaa),
                                    w3 = RGS_DPP(wgt, 0xff);
                        if (__builtin_expect((fl & 2u) != 0u, 0)) {
                            // a colour of the batch is not finite: what is not included leaves C as it is
                            C = (int)__float_as_uint(w0) >= 0 ? fmaf(w0, cv[0], C) : C;
                            C = (int)__float_as_uint(w1) >= 0 ? fmaf(w1, cv[1], C) : C;
                            C = (int)__float_as_uint(w2) >= 0 ? fmaf(w2, cv[2], C) : C;
                            C = (int)__float_as_uint(w3) >= 0 ? fmaf(w3, cv[3], C) : C;
                        } else {
                            C = fmaf(w3, cv[3], fmaf(w2, cv[2], fmaf(w1, cv[1], fmaf(w0, cv[0], C))));
                        }
                        // the transmittance after the last included instance: the least of the quad's
                        // (not negative: ordered like their bits)
                        uint32_t Tn = __float_as_uint(on ? Ta : T);
                        Tn = min(Tn, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)Tn, 0xb1, 0xf, 0xf, false));
                        Tn = min(Tn, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)Tn, 0x4e, 0xf, 0xf, false));
                        T = __uint_as_float(Tn);
                        if (wmask(!(T < thr)) == 0ull) break;
                    }
                }
                __syncthreads();
                if (next >= end) break;
                base = next;
            }
            last = max(last, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)last, 0xb1, 0xf, 0xf, false));
            last = max(last, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)last, 0x4e, 0xf, 0xf, false));
            {  // lane 4 pixel + c writes component c (C, then T)
                float* o = inst < 3 ? outC + (size_t)slot * 768 + 256 * inst : outT + (size_t)slot * 256;
                o[p] = inst < 3 ? C : T;
                if (inst == 0) outLast[(size_t)slot * 256 + p] = last;
            }
            // the walk stopped in this cell: every later cell is neutral here
            live = live && !(T < eps_T / P);
            M = fmaf(P, C, M);
            P *= T;
            if (!any_alive) {
                // every pixel of the quadrant has stopped: its share of the remaining
                // slots is neutral, written without staging a record
                for (uint32_t sn = slot + 1; sn < s1; ++sn) {
                    float* o = inst < 3 ? outC + (size_t)sn * 768 + 256 * inst : outT + (size_t)sn * 256;
                    o[p] = inst < 3 ? 0.f : 1.f;
                    if (inst == 0) outLast[(size_t)sn * 256 + p] = 0u;
                }
                break;
            }
        }
        if (image && on_image) {
            const size_t HW = (size_t)V.W * V.H, at = (size_t)py * V.W + px;
            const float bgc = inst == 0 ? V.bg[0] : (inst == 1 ? V.bg[1] : V.bg[2]);
            float* o = inst < 3 ? image + 3 * (size_t)V.pix_offset + HW * inst : T_final + V.pix_offset;
            o[at] = inst < 3 ? fmaf(P, bgc, M) : P;
        }
    } else {
        const int lx = (w & 1) * 8 + (lane & 7), ly = (w >> 1) * 8 + (lane >> 3);
        const int px = tx * 16 + lx, py = ty * 16 + ly;
        // merged image (image != null): the fold of Eq. 5 over the tile's slots in
        // their order, as the merge does it from the stored partials
        float M0 = 0.f, M1 = 0.f, M2 = 0.f;
        const float fxp = (float)px + 0.5f;
        const float dxp = (fxp - V.cx) / V.fx, dyp = ((float)py + 0.5f - V.cy) / V.fy;
        const float D0 = (V.R[0] * dxp + V.R[3] * dyp) + V.R[6];
        const float D1 = (V.R[1] * dxp + V.R[4] * dyp) + V.R[7];
        const float D2 = (V.R[2] * dxp + V.R[5] * dyp) + V.R[8];
        // a stopped (or off-image) pixel samples row +inf: d^2 = inf fails every test
        bool live = px < V.W && py < V.H;
        float P = 1.0f;
        const uint32_t qbit = 1u << (w + 1);
        const int p = ly * 16 + lx;

        for (uint32_t slot = s0; slot < s1; ++slot) {
            if (slot > s0) {
                // once every pixel of the tile has stopped, the remaining slots are
                // neutral: written without staging a record (P only decreases, so
                // the tile stays stopped)
                const uint64_t lv = __ballot(live);
                if (lane == 0) s_flag[0][w] = lv != 0ull ? 1u : 0u;
                __syncthreads();
                if ((s_flag[0][0] | s_flag[0][1] | s_flag[0][2] | s_flag[0][3]) == 0u) {
                    for (uint32_t sn = slot; sn < s1; ++sn) {
                        float* on = outC + (size_t)sn * 768;
                        on[p] = 0.f;
                        on[256 + p] = 0.f;
                        on[512 + p] = 0.f;
                        outT[(size_t)sn * 256 + p] = 1.f;
                        outLast[(size_t)sn * 256 + p] = 0u;
                    }
                    break;
                }
            }
            const uint32_t key = slot_key[slot];
            const int cell = V.cell_of_rank[key & ((1u << L) - 1u)];
            const uint32_t begin = slot_range[2 * slot], end = slot_range[2 * slot + 1];
            const float blo0 = box_lo[cell], blo1 = box_lo[K + cell], blo2 = box_lo[2 * K + cell];
            const float bhi0 = box_hi[cell], bhi1 = box_hi[K + cell], bhi2 = box_hi[2 * K + cell];
            // stop once P T < eps_T, i.e. T < eps_T / P (>= eps_T: T stays normal)
            const float thr = live ? eps_T / P : 0.0f;
            float fyp = live ? (float)py + 0.5f : INFINITY;
            float T = 1.0f, C0 = 0.f, C1 = 0.f, C2 = 0.f;
            uint32_t last = 0u;
            for (uint32_t base = begin; base < end; base += NB) {
                const uint64_t alive = __ballot(fyp != INFINITY);
                if (lane == 0) s_flag[1][w] = alive != 0ull ? 1u : 0u;
                const uint32_t idx = base + tid;
                if (idx < end) {
                    const uint32_t src = (uint32_t)(vals[idx] >> 32);
                    const float4* rp = reinterpret_cast<const float4*>(rec + (size_t)src * RGS_REC_FLOATS);
                    const float4 a = rp[0];
                    const float4 b = rp[1], cl = rp[2], r4 = rp[3];
                    const uint2 rr = make_uint2(__float_as_uint(r4.x), __float_as_uint(r4.y));
                    sM[tid] = (quad_mask(rr, tx, ty) << 1) | (__float_as_uint(cl.w) & 1u);
                    sA[tid] = a;
                    sB[tid] = b;
                    sCl[tid] = cl;
                    if (STATS) sR[tid] = rr;
                }
                __syncthreads();
                if ((s_flag[1][0] | s_flag[1][1] | s_flag[1][2] | s_flag[1][3]) == 0u) break;
                const int nb = (int)((end - base) < (uint32_t)NB ? (end - base) : (uint32_t)NB);
                if (alive != 0ull) {
                    // Gaussians of this batch whose footprint can reach the wave's
                    // quadrant, walked in order (other waves hide the LDS latency);
                    // the wave leaves the batch once all its pixels have stopped
#pragma unroll
                    for (int k = 0; k < NB / 64; ++k) {
                        if (k > 0 && __ballot(fyp != INFINITY) == 0ull) break;
                        const int tl = k * 64 + lane;
                        const uint32_t mk = tl < nb ? sM[tl] : 0u;
                        uint64_t rel = __ballot((mk & qbit) != 0u);
                        const uint64_t inside = __ballot((mk & 1u) != 0u);  // footprint in one cell: no indicator test
                        while (rel) {
                            const int bit = (int)__builtin_ctzll(rel);
                            const int tc = k * 64 + bit;
                            rel &= rel - 1ull;
                            const float4 ac = sA[tc], bc = sB[tc];
                            const float dx = fxp - ac.x, dy = fyp - ac.y;
                            const float u = fmaf(ac.w, dy, dx);  // d^2 = ca u^2 + e dy^2
                            const float d2 = fmaf(bc.x * dy, dy, (ac.z * u) * u);
                            if (STATS && fyp != INFINITY) {
                                // pairs the method must test: pixel inside the Gaussian's rectangle
                                const uint2 rr = sR[tc];
                                const bool inr = px >= (int)(int16_t)(rr.x & 0xffffu) && px <= (int)(int16_t)(rr.x >> 16) &&
                                                 py >= (int)(int16_t)(rr.y & 0xffffu) && py <= (int)(int16_t)(rr.y >> 16);
                                n_eval += inr ? 1u : 0u;
                            }
                            if (!(d2 <= bc.z)) continue;
                            const float4 cl = sCl[tc];
                            if (!((inside >> bit) & 1ull)) {
                                const float x0 = fmaf(bc.w, D0, o0), x1 = fmaf(bc.w, D1, o1), x2 = fmaf(bc.w, D2, o2);
                                const bool in = (blo0 <= x0) && (x0 < bhi0) && (blo1 <= x1) && (x1 < bhi1) && (blo2 <= x2) &&
                                                (x2 < bhi2);
                                if (!in) continue;
                            }
                            if (STATS) ++n_con;
                            const float G = __builtin_amdgcn_exp2f(d2 * -0.72134752044448170368f);  // exp(-d^2/2)
                            const float sg = fminf(0.99f, bc.y * G);
                            const float wgt = sg * T;
                            C0 = fmaf(wgt, cl.x, C0);
                            C1 = fmaf(wgt, cl.y, C1);
                            C2 = fmaf(wgt, cl.z, C2);
                            T = T * (1.0f - sg);
                            last = base - begin + (uint32_t)tc + 1u;
                            if (T < thr) fyp = INFINITY;
                        }
                    }
                }
                __syncthreads();
            }
            float* oc = outC + (size_t)slot * 768;
            oc[p] = C0;
            oc[256 + p] = C1;
            oc[512 + p] = C2;
            outT[(size_t)slot * 256 + p] = T;
            outLast[(size_t)slot * 256 + p] = last;
            // the walk stopped in this cell: every later cell is neutral here
            if (live && T < thr) live = false;
            M0 = fmaf(P, C0, M0);
            M1 = fmaf(P, C1, M1);
            M2 = fmaf(P, C2, M2);
            P *= T;
        }
        if (image && px < V.W && py < V.H) {
            const size_t HW = (size_t)V.W * V.H, pix = (size_t)py * V.W + px;
            float* img = image + 3 * (size_t)V.pix_offset;
            img[pix] = fmaf(P, V.bg[0], M0);
            img[HW + pix] = fmaf(P, V.bg[1], M1);
            img[2 * HW + pix] = fmaf(P, V.bg[2], M2);
            T_final[V.pix_offset + pix] = P;
        }
    }
    if (STATS) {
        unsigned long long e = n_eval, c = n_con;
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) {
            e += __shfl_xor(e, d, 64);
            c += __shfl_xor(c, d, 64);
        }
        if (lane == 0) {
            atomicAdd(&stats[0], e);
            atomicAdd(&stats[1], c);
        }
    }
}

rgs_status render_fwd_launch(const rgs_projected* proj, const rgs_bins* bins, const ViewTable* vt, const rgs_kdtree* kd,
                             float eps_T, const rgs_partials* out, uint64_t* stats, int64_t total_tiles, hipStream_t s,
                             float* image, float* T_final) {
    if (total_tiles <= 0) return RGS_OK;
    // a pixel stops once its merged transmittance falls below max(eps_T,
    // 2^-100): the backward recovers the transmittance before each
    // contribution from the stored T_k by division, which needs T_k to stay
    // a normal fp32 number (T_k >= 0.01 eps_T / P >= 2^-107)
    eps_T = fmaxf(eps_T, RGS_T_FLOOR);
    const uint32_t heavy = (uint32_t)(total_tiles < (int64_t)RF_HEAVY ? total_tiles : (int64_t)RF_HEAVY);
    const dim3 grid((unsigned)total_tiles + 3u * heavy);
    if (stats)
        hipLaunchKernelGGL(k_render_fwd<true>, grid, dim3(256), 0, s, proj->rec, bins->vals, bins->slot_key,
                           bins->slot_range, bins->tile_slot, bins->tile_order, heavy, vt, kd->box_lo, kd->box_hi,
                           eps_T, out->C, out->T, out->last, reinterpret_cast<unsigned long long*>(stats), image,
                           T_final);
    else
        hipLaunchKernelGGL(k_render_fwd<false>, grid, dim3(256), 0, s, proj->rec, bins->vals, bins->slot_key,
                           bins->slot_range, bins->tile_slot, bins->tile_order, heavy, vt, kd->box_lo, kd->box_hi,
                           eps_T, out->C, out->T, out->last, nullptr, image, T_final);
    return launch_check();
}

// ------------------------------------------------------------------ backward
// Sum of g[0..8] over the wave: values 0..7 by reduce-scatter over lane bits
// 5, 4, 3 and a full sum over bits 2, 1, 0, so lane 8v ends with value v;
// value 8 ends in lane 63.  Bits 5 and 4 use the gfx950 lane-swap
// instructions: swapping the upper 32 lanes of x with the lower 32 lanes of y
// leaves, in both outputs, x's half where lane bit 5 is clear and y's half
// where it is set, with the partner lane's copy in the other output, so one
// add reduces over bit 5 without a select; the 16-lane swap does the same for
// bit 4.  Bit 3 is a row rotation by 8 (DPP), bits 2..0 quad permutes and a
// half-row mirror; no exchange goes through LDS.
__device__ __forceinline__ float swap32_sum(float x, float y) {
    const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, x), __builtin_bit_cast(unsigned, y),
                                                   false, false);
    unsigned a = r[0], b = r[1];
    asm volatile("" : "+v"(a), "+v"(b));  // keeps the two results apart (r[0] + r[1] otherwise folds to 2 r[0])
    return __builtin_bit_cast(float, a) + __builtin_bit_cast(float, b);
}

__device__ __forceinline__ float swap16_sum(float x, float y) {
    const auto r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(unsigned, x), __builtin_bit_cast(unsigned, y),
                                                   false, false);
    unsigned a = r[0], b = r[1];
    asm volatile("" : "+v"(a), "+v"(b));  // keeps the two results apart (r[0] + r[1] otherwise folds to 2 r[0])
    return __builtin_bit_cast(float, a) + __builtin_bit_cast(float, b);
}

__device__ __forceinline__ void wave_sum9(const float* g, int lane, float* out_v, float* out_8) {
    *out_8 = wave_sum_to_lane63(g[8]);
    float q4[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) q4[k] = swap32_sum(g[k], g[4 + k]);  // bit 5 clear keeps k, set keeps 4 + k
    const float q20 = swap16_sum(q4[0], q4[2]);                      // bit 4 clear keeps 4 h5 + 0, set + 2
    const float q21 = swap16_sum(q4[1], q4[3]);
    const bool h3 = (lane & 8) != 0;
    float q1 = (h3 ? q21 : q20) + RGS_DPP(h3 ? q20 : q21, 0x128);     // row_ror:8 = lane xor 8 within a row
    q1 += RGS_DPP(q1, 0xb1);                                          // quad_perm [1,0,3,2]
    q1 += RGS_DPP(q1, 0x4e);                                          // quad_perm [2,3,0,1]
    q1 += RGS_DPP(q1, 0x141);                                         // row_half_mirror
    *out_v = q1;
}
#undef RGS_DPP

// Backward: 128-thread block per slot.  Wave w owns the 16x8 half (rows
// 8w .. 8w + 7) of the tile and every lane two pixels of one row, eight
// columns apart (quadrants (0, w) and (1, w)): the lane adds its two pixels'
// gradient terms before the cross-lane sum, so one wave sum covers 128
// pixels.  Batches of 64 instances are walked back to front from the block's
// largest `last`; every wave sums each instance's gradient over its 128
// pixels (zero when culled or not contributing) into LDS, and the two half
// sums are added in a fixed order into the instance's record.
struct BwdPix {
    float fx, D0, D1, D2;  // sample x, ray direction
    float T, gB, gC0, gC1, gC2, gTf;
    uint32_t last;
};

// One pixel's share of an instance's gradient.  A pixel that does not
// contribute comes with d^2 = +inf: G = 0 and sigma = 0, so 1 / (1 - sigma) = 1
// exactly, T and <dC, B> stay as they are, and every term returned is zero.
struct PixTerms {
    float q, dsg_g, G, wc;
};

__device__ __forceinline__ PixTerms pix_step(BwdPix& P, float d2, float alpha, float4 cl) {
    PixTerms r;
    r.G = __builtin_amdgcn_exp2f(d2 * -0.72134752044448170368f);  // exp(-d^2/2)
    const float aG = alpha * r.G;
    const float sgm = fminf(0.99f, aG);
    const float rom = __builtin_amdgcn_rcpf(1.0f - sgm);
    const float Tb = P.T * rom;  // transmittance before this contribution
    const float dot = fmaf(P.gC2, cl.z, fmaf(P.gC1, cl.y, P.gC0 * cl.x)) - P.gB;  // <dC, c - B>
    const float dsg = rom * fmaf(P.T, dot, -P.gTf);                               // dL/dsigma
    r.wc = Tb * sgm;
    P.gB = fmaf(sgm, dot, P.gB);  // B <- B + sigma (c - B)
    P.T = Tb;
    // clamped at 0.99: no gradient to alpha or the footprint
    r.dsg_g = aG < 0.99f ? dsg : 0.0f;
    r.q = aG * r.dsg_g;
    return r;
}

template <bool STATS>
__global__ __launch_bounds__(128) void k_render_bwd(const float* __restrict__ rec,
                                                    const uint64_t* __restrict__ vals,
                                                    const uint32_t* __restrict__ slot_key,
                                                    const uint32_t* __restrict__ slot_range,
                                                    const uint32_t* __restrict__ slot_order,
                                                    const uint32_t* __restrict__ n_launch,
                                                    const ViewTable* __restrict__ vt, const float* __restrict__ box_lo,
                                                    const float* __restrict__ box_hi, const float* __restrict__ partT,
                                                    const uint32_t* __restrict__ partLast, const float* __restrict__ dC,
                                                    const float* __restrict__ dT, float* __restrict__ records,
                                                    uint32_t* __restrict__ touched,
                                                    const uint32_t* __restrict__ counters, uint32_t* __restrict__ flags,
                                                    unsigned long long* __restrict__ stats) {
    constexpr int NB = 64;
    __shared__ float4 sA[NB], sB[NB], sCl[NB];
    __shared__ uint2 sR[NB];
    __shared__ uint32_t sJ[NB];
    __shared__ float sG[2][NB][9];
    __shared__ uint32_t s_max[2];
    __shared__ uint64_t s_wrote[2];  // per wave: the batch's instances it wrote half sums for
    // the pairs' flags for the pair reduction (a byte each, where the slots' work was)
    for (uint64_t i = (uint64_t)blockIdx.x * 128u + threadIdx.x; i < ((uint64_t)counters[0] + 3u) / 4u; i += (uint64_t)gridDim.x * 128u)
        flags[i] = 0u;
    if (blockIdx.x >= *n_launch) return;
    const uint32_t slot = slot_order[blockIdx.x];
    const int L = vt->L, K = 1 << L;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const uint32_t key = slot_key[slot];
    const uint32_t gt = key >> L;
    const int v = view_of_tile(vt, gt);
    const ViewParams& V = vt->v[v];
    const uint32_t lt = gt - V.tile_offset;
    const int tx = (int)(lt % (uint32_t)V.tiles_x), ty = (int)(lt / (uint32_t)V.tiles_x);
    const int cell = V.cell_of_rank[key & ((1u << L) - 1u)];
    const uint32_t begin = slot_range[2 * slot], end = slot_range[2 * slot + 1];
    const float blo0 = box_lo[cell], blo1 = box_lo[K + cell], blo2 = box_lo[2 * K + cell];
    const float bhi0 = box_hi[cell], bhi1 = box_hi[K + cell], bhi2 = box_hi[2 * K + cell];
    const int lx = lane & 7, ly = w * 8 + (lane >> 3);
    const int py = ty * 16 + ly;
    const float fyp = (float)py + 0.5f;
    const float dyp = (fyp - V.cy) / V.fy;
    const float o0 = V.o[0], o1 = V.o[1], o2 = V.o[2];
    BwdPix P[2];
    int pxs[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int px = tx * 16 + lx + 8 * h;
        pxs[h] = px;
        P[h].fx = (float)px + 0.5f;
        const float dxp = (P[h].fx - V.cx) / V.fx;
        P[h].D0 = (V.R[0] * dxp + V.R[3] * dyp) + V.R[6];
        P[h].D1 = (V.R[1] * dxp + V.R[4] * dyp) + V.R[7];
        P[h].D2 = (V.R[2] * dxp + V.R[5] * dyp) + V.R[8];
        const int p = ly * 16 + lx + 8 * h;
        const bool valid = px < V.W && py < V.H;
        const float Tf = partT[(size_t)slot * 256 + p];
        P[h].T = Tf;
        P[h].last = valid ? partLast[(size_t)slot * 256 + p] : 0u;
        P[h].gTf = valid ? dT[(size_t)slot * 256 + p] * Tf : 0.f;
        P[h].gC0 = valid ? dC[(size_t)slot * 768 + p] : 0.f;
        P[h].gC1 = valid ? dC[(size_t)slot * 768 + 256 + p] : 0.f;
        P[h].gC2 = valid ? dC[(size_t)slot * 768 + 512 + p] : 0.f;
        // gB = <dC_k, B>, where B is the colour blended behind the current
        // instance (the suffix of Eq. 3): the only way B enters the gradient
        P[h].gB = 0.f;
    }
    uint32_t n_eval = 0u, n_con = 0u;
    const uint32_t wmax = wave_max_u32(max(P[0].last, P[1].last));
    if (lane == 0) s_max[w] = wmax;
    __syncthreads();
    const uint32_t bmax = max(s_max[0], s_max[1]);
    // instances behind every pixel's last contributor (k >= bmax) get no
    // record: their bit in `touched` stays clear and the pair reduction
    // counts them as zero
    const float hx0 = (float)(tx * 16), hy0 = (float)(ty * 16 + w * 8);
    for (int bstart = bmax == 0 ? -1 : (int)(((bmax - 1) / NB) * NB); bstart >= 0; bstart -= NB) {
        if (tid < NB && (uint32_t)bstart + tid < bmax) {
            const uint64_t vv = vals[begin + bstart + tid];
            const uint32_t src = (uint32_t)(vv >> 32);
            const float4* rp = reinterpret_cast<const float4*>(rec + (size_t)src * RGS_REC_FLOATS);
            const float4 cl = rp[2];
            const float4 a = rp[0], b = rp[1], r4 = rp[3];
            sA[tid] = a;
            sB[tid] = b;
            sCl[tid] = cl;
            sR[tid] = make_uint2(__float_as_uint(r4.x), __float_as_uint(r4.y));
            sJ[tid] = (uint32_t)vv;
        }
        __syncthreads();
        // Gaussians of this batch below the wave's largest `last` whose
        // footprint can reach the wave's half tile (each wave tests its own
        // half, one record per lane), walked back to front
        const int tl = lane;
        bool hit = (uint32_t)(bstart + tl) + 1u <= wmax && (uint32_t)(bstart + tl) < bmax;
        if (hit) {
            const float4 a = sA[tl], b = sB[tl];
            const float cb = a.w * a.z, cc = b.x + a.w * cb;  // conic from (ca, k, e)
            hit = ((quad_mask(sR[tl], tx, ty) >> (2 * w)) & 3u) &&
                  box_hits(a.x, a.y, a.z, cb, cc, b.z, hx0, hy0, 16.0f, 8.0f);
        }
        uint64_t rel = __ballot(hit);
        uint64_t wrote = 0ull;
        const uint64_t inside = __ballot(hit && (__float_as_uint(sCl[tl].w) & 1u));  // in one cell: no indicator test
        while (rel) {
            const int t = 63 - (int)__builtin_clzll(rel);
            rel &= ~(1ull << t);
            const uint32_t pos1 = (uint32_t)(bstart + t) + 1u;  // this instance's index + 1
            const float4 a = sA[t];
            const float4 b = sB[t];
            const float dy = fyp - a.y;
            const float edy = b.x * dy;
            const float dx0 = P[0].fx - a.x, dx1 = P[1].fx - a.x;
            const float u0 = fmaf(a.w, dy, dx0), u1 = fmaf(a.w, dy, dx1);  // d^2 = ca u^2 + e dy^2
            const float d20 = fmaf(edy, dy, (a.z * u0) * u0), d21 = fmaf(edy, dy, (a.z * u1) * u1);
            // contributing lanes as wave masks: one ballot per comparison (the
            // compare's own lane mask), combined in scalar registers; a lane's
            // flag is read back with an inverse ballot
            uint64_t m0 = wmask(pos1 <= P[0].last) & wmask(d20 <= b.z);
            uint64_t m1 = wmask(pos1 <= P[1].last) & wmask(d21 <= b.z);
            if (STATS) {
                // pairs the backward must re-test: pixel inside the rectangle, at or before its last contributor
                const uint2 rr = sR[t];
                const bool rowin = py >= (int)(int16_t)(rr.y & 0xffffu) && py <= (int)(int16_t)(rr.y >> 16);
                const int xl = (int)(int16_t)(rr.x & 0xffffu), xh = (int)(int16_t)(rr.x >> 16);
                n_eval += (pos1 <= P[0].last && rowin && pxs[0] >= xl && pxs[0] <= xh) ? 1u : 0u;
                n_eval += (pos1 <= P[1].last && rowin && pxs[1] >= xl && pxs[1] <= xh) ? 1u : 0u;
            }
            if ((m0 | m1) == 0ull) continue;
            const float4 cl = sCl[t];
            if (!((inside >> t) & 1ull)) {  // not interior to the cell: the indicator of Eq. 6
                const float x0 = fmaf(b.w, P[0].D0, o0), y0 = fmaf(b.w, P[0].D1, o1), z0 = fmaf(b.w, P[0].D2, o2);
                const float x1 = fmaf(b.w, P[1].D0, o0), y1 = fmaf(b.w, P[1].D1, o1), z1 = fmaf(b.w, P[1].D2, o2);
                m0 &= wmask(blo0 <= x0) & wmask(x0 < bhi0) & wmask(blo1 <= y0) & wmask(y0 < bhi1) & wmask(blo2 <= z0) &
                      wmask(z0 < bhi2);
                m1 &= wmask(blo0 <= x1) & wmask(x1 < bhi0) & wmask(blo1 <= y1) & wmask(y1 < bhi1) & wmask(blo2 <= z1) &
                      wmask(z1 < bhi2);
                if ((m0 | m1) == 0ull) continue;
            }
            const bool c0 = __builtin_amdgcn_inverse_ballot_w64(m0), c1 = __builtin_amdgcn_inverse_ballot_w64(m1);
            if (STATS) n_con += (c0 ? 1u : 0u) + (c1 ? 1u : 0u);
            // a pixel column of the wave where no lane contributes (the
            // instance reaches one quadrant of the half only) is skipped: its
            // step would leave T and <dC, B> as they are and add zeros
            const float d2c0 = c0 ? d20 : INFINITY, d2c1 = c1 ? d21 : INFINITY;
            const bool any0 = m0 != 0ull, any1 = m1 != 0ull;
            PixTerms r0 = {0.f, 0.f, 0.f, 0.f}, r1 = {0.f, 0.f, 0.f, 0.f};
            if (any0) r0 = pix_step(P[0], d2c0, b.y, cl);
            if (any1) r1 = pix_step(P[1], d2c1, b.y, cl);
            // Raw sums over the lane's two pixels; the conic and constant
            // factors are applied per instance after the reduction
            // (dL/d(d^2) = -q / 2)
            float g[9];
            const float qx0 = r0.q * dx0, qx1 = r1.q * dx1;
            g[0] = qx0 + qx1;                      // q dx
            g[1] = (r0.q + r1.q) * dy;             // q dy
            g[2] = fmaf(qx1, dx1, qx0 * dx0);      // q dx^2
            g[3] = g[0] * dy;                      // q dx dy
            g[4] = g[1] * dy;                      // q dy^2
            g[5] = fmaf(r1.dsg_g, r1.G, r0.dsg_g * r0.G);
            g[6] = fmaf(r1.wc, P[1].gC0, r0.wc * P[0].gC0);
            g[7] = fmaf(r1.wc, P[1].gC1, r0.wc * P[0].gC1);
            g[8] = fmaf(r1.wc, P[1].gC2, r0.wc * P[0].gC2);
            float sv, s8;
            wave_sum9(g, lane, &sv, &s8);
            // 32-bit LDS offsets (t * 9 in scalar registers)
            float* const gw = &sG[w][0][0];
            const uint32_t gt = (uint32_t)t * 9u;
            if ((lane & 7) == 0) gw[gt + (uint32_t)(lane >> 3)] = sv;
            if (lane == 63) gw[gt + 8u] = s8;
            wrote |= 1ull << t;
        }
        if (lane == 0) s_wrote[w] = wrote;
        __syncthreads();
        const uint64_t h0 = s_wrote[0], h1 = s_wrote[1];
        // a record for every instance that either half wrote (the others add nothing)
        if (tid < NB && (uint32_t)bstart + tid < bmax && (((h0 | h1) >> tid) & 1ull)) {
            // S_c = sum over the two halves, in a fixed order (a half that
            // wrote nothing adds zero)
            const int t = tid;
            const bool w0 = (h0 >> t) & 1ull, w1 = (h1 >> t) & 1ull;
            float S[9];
#pragma unroll
            for (int c = 0; c < 9; ++c) S[c] = (w0 ? sG[0][t][c] : 0.f) + (w1 ? sG[1][t][c] : 0.f);
            const float4 a = sA[t];
            const float cb = a.w * a.z, cc = sB[t].x + a.w * cb;  // conic from (ca, k, e)
            const uint32_t jr = sJ[t];
            float* rp = records + (size_t)jr * RD_REC;
            atomicOr(&touched[jr >> 5], 1u << (jr & 31u));
            // d mx = sum q (ca dx + cb dy), d my = sum q (cb dx + cc dy); d ca, d cb, d cc
            // carry dL/d(d^2) = -q / 2 (d cb counts the cross term twice); then d alpha, colour
            rp[0] = a.z * S[0] + cb * S[1];
            rp[1] = cb * S[0] + cc * S[1];
            rp[2] = -0.5f * S[2];
            rp[3] = -S[3];
            rp[4] = -0.5f * S[4];
            rp[5] = S[5];
            rp[6] = S[6];
            rp[7] = S[7];
            rp[8] = S[8];
        }
        __syncthreads();
    }
    if (STATS) {
        unsigned long long e = n_eval, c = n_con;
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) {
            e += __shfl_xor(e, d, 64);
            c += __shfl_xor(c, d, 64);
        }
        if (lane == 0) {
            atomicAdd(&stats[0], e);
            atomicAdd(&stats[1], c);
        }
    }
}

// Per (view, Gaussian) pair: sum of its instance records.  The records of a
// pair are contiguous (emission order), so the sum is a segmented reduction
// over the instance array, balanced over instances:
//  1. k_pair_seg: a wave takes 64 consecutive records; the pairs covering
//     them come from the wave's first pair (first_pair, written by the
//     backward's records call along with its launch order) and one coalesced
//     load of the next 64 pair offsets; a segmented inclusive scan (fixed tree of
//     shuffles) sums each pair's records within the wave.  The wave's first
//     segment (pair begun before it) and last segment (pair going on after
//     it) are kept as wave partials; a pair with a record gets its psum[rank]
//     entry and a flag: its sum if it lies in one wave, else the first and
//     last wave it spans.  Most waves of a large batch have no record (16
//     views: 73 %) and end at once.
//  2. k_pair_gather: thread per (view, Gaussian): zero if culled or without a
//     flag, else the pair's psum entry, or, for a pair spanning several waves,
//     its tail partial + whole-wave partials + head partial, in instance order.
// us, reduction + gather: 16 views, 767M instances, 5 % with a record, 55M pairs
// 4714 + 1899 -> 2286 + 1148; 1M at 1600x1060 56 + 32 -> 45 + 24; 16M at
// 3840x2160 78 + 179 -> 41 + 190 (when every pair's entry was written and read).
// first_pair[w] = the pair holding instance 64 w: each pair writes the waves
// that start inside it (one thread per pair, grid-stride over the device count).
__device__ __forceinline__ void wave_first_pairs(const uint32_t* __restrict__ pair_off,
                                                 const uint32_t* __restrict__ counters,
                                                 uint32_t* __restrict__ first_pair) {
    const int64_t np = counters[0];
    for (int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r < np; r += (int64_t)gridDim.x * blockDim.x) {
        const uint32_t b = pair_off[r], e = pair_off[r + 1];
        for (uint32_t w = (b + 63u) >> 6; (w << 6) < e; ++w) first_pair[w] = (uint32_t)r;
    }
}

__global__ __launch_bounds__(256) void k_wave_first(const uint32_t* __restrict__ pair_off,
                                                    const uint32_t* __restrict__ counters,
                                                    uint32_t* __restrict__ first_pair) {
    wave_first_pairs(pair_off, counters, first_pair);
}

__global__ __launch_bounds__(256) void k_pair_seg(const float* __restrict__ records,
                                                  const uint32_t* __restrict__ touched,
                                                  const uint32_t* __restrict__ pair_off,
                                                  const uint32_t* __restrict__ counters,
                                                  const uint32_t* __restrict__ first_pair, float* __restrict__ psum,
                                                  float* __restrict__ wpart, uint8_t* __restrict__ flags) {
    const int lane = threadIdx.x & 63;
    const int64_t w = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const uint32_t n_pairs = counters[0], n_inst = counters[1];
    const int64_t j0 = w * 64;
    if (j0 >= (int64_t)n_inst) return;  // uniform per wave
    const uint2 tw = reinterpret_cast<const uint2*>(touched)[w];
    const uint64_t has_mask = (uint64_t)tw.y << 32 | tw.x;
    if (has_mask == 0ull) return;  // no record: its pairs' entries stay empty, its partials unread
    const int64_t j = j0 + lane;
    const bool valid = j < (int64_t)n_inst;
    // the records first (they do not depend on the pair lookup); an instance
    // without a record (behind its tile's last contributors) counts as zero
    float v[9];
    const bool has = (has_mask >> lane) & 1ull;
    {
#pragma unroll
        for (int c = 0; c < 9; ++c) v[c] = 0.f;
        if (has) {
            const float* rp = records + (size_t)j * RD_REC;
#pragma unroll
            for (int c = 0; c < 9; ++c) v[c] = rp[c];
        }
    }
    const uint32_t r0 = first_pair[w];  // the pair holding instance j0
    // starts of the next 64 pairs (increasing, the tail entry included); pos =
    // how many start at or before j (at most 63: they start after j0)
    const uint32_t rk = r0 + 1u + (uint32_t)lane;
    const int64_t bk = rk <= n_pairs ? (int64_t)pair_off[rk] : INT64_MAX;
    const int64_t b_r0 = (int64_t)pair_off[r0];
    // the lanes where those pairs start, as a lane mask: a start inside the
    // wave (never at its lane 0) sets its lane's byte in the wave's 64 bytes of
    // LDS (starts are distinct; one wave's LDS operations run in order)
    __shared__ uint8_t s_flag[4][64];
    uint8_t* fl = s_flag[threadIdx.x >> 6];
    fl[lane] = 0;
    __builtin_amdgcn_wave_barrier();
    const int64_t dl = bk - j0;
    if (dl > 0 && dl < 64) fl[dl] = 1;
    __builtin_amdgcn_wave_barrier();
    const uint64_t starts = __ballot(fl[lane] != 0);
    const uint64_t le_mask = (lane == 63) ? ~0ull : ((2ull << lane) - 1ull);
    const int pos = __popcll(starts & le_mask);  // pairs after r0 starting at or before j
    const uint64_t heads = starts | 1ull;
    const int seg0 = 63 - __builtin_clzll(heads & le_mask);  // first lane of this lane's segment
    // the start and end of this lane's pair, from the starts already loaded
    const int64_t b_at = __shfl(bk, pos > 0 ? pos - 1 : 0, 64);
    const int64_t e_at = __shfl(bk, pos, 64);
    // Segmented inclusive scan: in-row steps by DPP row shifts (1, 2, 4, 8;
    // lanes shifted in from outside the row read 0), then the row broadcasts
    // of lanes 15 and 47 (into rows 1 and 3) and of lane 31 (into rows 2 and
    // 3); a lane only adds values from its own segment.
    const int row = lane >> 4;
#define RGS_SEG_STEP(ctrl, rmask, take)                                                                            \
    {                                                                                                              \
        const bool tk = (take);                                                                                    \
        _Pragma("unroll") for (int c = 0; c < 9; ++c) {                                                            \
            const float u = __builtin_bit_cast(                                                                    \
                float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v[c]), (ctrl), (rmask), 0xf, false)); \
            if (tk) v[c] += u;                                                                                     \
        }                                                                                                          \
    }
    RGS_SEG_STEP(0x111, 0xf, lane - 1 >= seg0)             // row_shr:1
    RGS_SEG_STEP(0x112, 0xf, lane - 2 >= seg0)             // row_shr:2
    RGS_SEG_STEP(0x114, 0xf, lane - 4 >= seg0)             // row_shr:4
    RGS_SEG_STEP(0x118, 0xf, lane - 8 >= seg0)             // row_shr:8
    RGS_SEG_STEP(0x142, 0xa, (row & 1) && seg0 < 16 * row)  // row_bcast:15
    RGS_SEG_STEP(0x143, 0xc, row >= 2 && seg0 < 32)         // row_bcast:31
#undef RGS_SEG_STEP
    const int pos_next = __shfl_down(pos, 1, 64);
    const bool next_valid = lane < 63 && j + 1 < (int64_t)n_inst;
    const bool seg_end = valid && (!next_valid || pos_next != pos);
    if (!seg_end) return;
    const uint32_t r = r0 + (uint32_t)pos;
    const int64_t pb = pos > 0 ? b_at : b_r0;  // the pair's instances: [pb, e_at)
    const bool began_before = pb < j0;
    const bool goes_on = e_at > j0 + 64;
    const float4 o0 = make_float4(v[0], v[1], v[2], v[3]), o1 = make_float4(v[4], v[5], v[6], v[7]),
                 o2 = make_float4(v[8], 0.f, 0.f, 0.f);
    if (has_mask & le_mask & ~((1ull << seg0) - 1ull)) {  // the segment has a record
        float4* q = reinterpret_cast<float4*>(psum + (size_t)r * PS_REC);
        if (!goes_on && !began_before) {
            q[0] = o0; q[1] = o1; q[2] = o2;
            flags[r] = PS_SUM;
        } else {
            // spans waves pb / 64 .. (e_at - 1) / 64: its sum is in the wave partials
            // (every wave with one of its records writes the same)
            q[2] = make_float4(0.f, __uint_as_float((uint32_t)(pb >> 6)), __uint_as_float((uint32_t)((e_at - 1) >> 6)), 0.f);
            flags[r] = PS_SPAN;
        }
    }
    if (began_before) {
        float4* q = reinterpret_cast<float4*>(wpart + ((size_t)w * 2 + 0) * PS_REC);
        q[0] = o0; q[1] = o1; q[2] = o2;
    }
    if (goes_on) {
        float4* q = reinterpret_cast<float4*>(wpart + ((size_t)w * 2 + 1) * PS_REC);
        q[0] = o0; q[1] = o1; q[2] = o2;
    }
}

__device__ __forceinline__ void acc_rec(const float* __restrict__ p, float4& a0, float4& a1, float& a8) {
    const float4* q = reinterpret_cast<const float4*>(p);
    const float4 x = q[0], y = q[1];
    a0.x += x.x; a0.y += x.y; a0.z += x.z; a0.w += x.w;
    a1.x += y.x; a1.y += y.y; a1.z += y.z; a1.w += y.w;
    a8 += q[2].x;
}

__global__ __launch_bounds__(256) void k_pair_gather(const float* __restrict__ psum, const float* __restrict__ wpart,
                                                     const uint32_t* __restrict__ touched,
                                                     const uint8_t* __restrict__ flags,
                                                     const uint32_t* __restrict__ count,
                                                     const int32_t* __restrict__ pair_rank,
                                                     const uint32_t* __restrict__ counters, int64_t m,
                                                     float* __restrict__ dproj) {
    const int64_t sidx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (sidx >= m) return;
    float4 a0 = make_float4(0.f, 0.f, 0.f, 0.f), a1 = a0;
    float a8 = 0.f;
    const int32_t r = count[sidx] > 0u ? pair_rank[sidx] : -1;
    if (r >= 0 && (uint32_t)r < counters[0]) {  // a pass that ran out of capacity has no pairs
        const float4* q = reinterpret_cast<const float4*>(psum + (size_t)r * PS_REC);
        const uint8_t flag = flags[r];
        if (flag == PS_SUM) {
            a0 = q[0];
            a1 = q[1];
            a8 = q[2].x;
        } else if (flag == PS_SPAN) {
            const uint32_t wb = __float_as_uint(q[2].y), we = __float_as_uint(q[2].z);
            // the range the pair reduction wrote lies in the instance array (checked all the same)
            const uint32_t nw = (uint32_t)(((uint64_t)counters[1] + 63u) >> 6);
            if (wb < we && we < nw) {
                // tail of the first wave, whole waves, head of the last one; a wave
                // without records wrote no partials
                for (uint32_t w = wb; w <= we; ++w) {
                    const uint2 tw = reinterpret_cast<const uint2*>(touched)[w];
                    if ((tw.x | tw.y) != 0u) acc_rec(wpart + ((size_t)w * 2 + (w == wb ? 1 : 0)) * PS_REC, a0, a1, a8);
                }
            }
        }
    }
    dproj[0 * m + sidx] = a0.x;
    dproj[1 * m + sidx] = a0.y;
    dproj[2 * m + sidx] = a0.z;
    dproj[3 * m + sidx] = a0.w;
    dproj[4 * m + sidx] = a1.x;
    dproj[5 * m + sidx] = a1.y;
    dproj[6 * m + sidx] = a1.z;
    dproj[7 * m + sidx] = a1.w;
    dproj[8 * m + sidx] = a8;
}

// Backward workspace for an instance capacity, at most `slots` slots and at most
// `pairs` pairs (neither can exceed the instances): 36-byte records; 48-byte
// per-pair sums; two 48-byte partials and the first pair per 64 instances; a bit
// per instance; a word per slot twice, of which the first array is the pairs'
// flag bytes later, and the launch order's class counts.  Sized by the capacity
// alone everything but the records comes to 62 bytes per instance, of which
// nothing like that is used where instances are many per pair and slot (16 views,
// 882M instances, 64M pairs, 0.8M slots: 80.3 GiB, against 33.9 GiB so).
static size_t up256(size_t b) { return (b + 255) & ~size_t(255); }

struct BwdSizes {
    size_t c, slots, pairs;
    size_t rec() const { return up256(c * RD_REC * sizeof(float)); }
    size_t psum() const { return up256(pairs * PS_REC * sizeof(float)); }
    size_t wpart() const { return up256((c + 63) / 64 * 2 * PS_REC * sizeof(float)); }
    size_t first() const { return up256((c + 63) / 64 * sizeof(uint32_t)); }
    size_t touched() const { return up256(((c + 31) / 32 + 64) * sizeof(uint32_t)); }  // bitmask + launch count
    size_t work() const { return up256((slots > (pairs + 3) / 4 ? slots : (pairs + 3) / 4) * sizeof(uint32_t)); }
    size_t order() const { return up256(slots * sizeof(uint32_t)); }
    size_t tab() const { return up256((slots + SW_SLOTS - 1) / SW_SLOTS * SW_CLS * sizeof(uint32_t)); }
    size_t all() const { return rec() + psum() + wpart() + first() + touched() + work() + order() + tab() + 256; }
};

static BwdSizes bwd_sizes(int64_t capacity, int64_t slots, int64_t pairs) {
    const int64_t c = capacity > 0 ? capacity : 1;
    auto most = [c](int64_t x) { return (size_t)(x < 1 ? 1 : (x < c ? x : c)); };
    return BwdSizes{(size_t)c, most(slots), most(pairs)};
}

size_t render_bwd_ws_bytes(int64_t capacity, int64_t slots, int64_t pairs) { return bwd_sizes(capacity, slots, pairs).all(); }

struct BwdWs {
    float *records, *psum, *wpart;
    uint32_t* first_pair;
    uint32_t* touched;  // bit j: instance j (emission position) has a record
    size_t touched_words;
    uint32_t* wcls;     // the number of slots launched (after the bitmask)
    uint32_t* work;     // per slot: instances the backward visits (its largest `last`); then the pairs' flags
    int64_t flag_words;
    uint32_t* order;    // the backward's launch order
    uint32_t* wtab;     // [blocks of SW_SLOTS slots][SW_CLS] class counts
};

__global__ __launch_bounds__(256) void k_clear_words(uint32_t* __restrict__ p, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) p[i] = 0u;
}

// A workspace of the size for the capacity alone is laid out by it, a smaller one
// by the slots and pairs; the records and the reduction see the same bytes.
static BwdWs carve_bwd(const rgs_bins* bins, int64_t pairs, void* ws, size_t ws_bytes) {
    const int64_t cap = bins->capacity;
    BwdSizes z = bwd_sizes(cap, cap, cap);
    if (ws_bytes < z.all()) z = bwd_sizes(cap, bins->slot_capacity, pairs);
    BwdWs w;
    char* p = reinterpret_cast<char*>(ws);
    w.records = reinterpret_cast<float*>(p);
    w.psum = reinterpret_cast<float*>(p += z.rec());
    w.wpart = reinterpret_cast<float*>(p += z.psum());
    w.first_pair = reinterpret_cast<uint32_t*>(p += z.wpart());
    w.touched = reinterpret_cast<uint32_t*>(p += z.first());
    w.touched_words = 2 * ((z.c + 63) / 64);  // (whole 64-instance waves)
    w.wcls = w.touched + w.touched_words;
    w.work = reinterpret_cast<uint32_t*>(p += z.touched());
    w.flag_words = (int64_t)((z.pairs + 3) / 4);
    w.order = reinterpret_cast<uint32_t*>(p += z.work());
    w.wtab = reinterpret_cast<uint32_t*>(p += z.order());
    return w;
}

// The backward's launch order: the slots by decreasing size class (half
// octaves, slot_class) of the instances the backward visits (w = the largest `last`
// over the slot's pixels: it walks instances 0 .. w - 1), so that the
// heaviest blocks start first; a slot with w = 0 (no contribution) is not
// launched.  Two passes without global atomics (which serialise on a handful
// of class counters): k_slot_work, SW_SLOTS slots (times `rounds`) per block, a wave per slot
// at a time (256 `last` values, four per lane), stores w and the block's
// class counts as one row of a table; k_slot_place, the same slots
// per block, derives every class's start and the block's offset in it from
// the table and places its slots (the order inside a class is the launch
// order only and affects no result).
static constexpr int SW_CHUNK = 16;  // slots per wave whose loads are issued together
static_assert(SW_SLOTS % (4 * SW_CHUNK) == 0, "a block's four waves take whole chunks");
static_assert(SW_CLS == 32 || SW_CLS == 64 || SW_CLS == 128, "the placement's column sums split 256 threads by class");

// Class of w > 0: 2 floor(log2 w) plus the bit below the leading one (half
// octaves; whole or quarter octaves for 32 or 128 classes).
__device__ __forceinline__ int slot_class(uint32_t w) {
    const int hb = 31 - __clz(w);
    if (SW_CLS == 32) return hb;
    if (SW_CLS == 64) return 2 * hb + (hb > 0 ? (int)((w >> (hb - 1)) & 1u) : 0);
    return 4 * hb + (hb >= 2 ? (int)((w >> (hb - 2)) & 3u) : (hb == 1 ? (int)((w & 1u) << 1) : 0));
}

// Largest u32 of the wave, into lane 63 (DPP row operations, as the sums
// above; a lane a broadcast does not reach keeps its value: max with 0).
__device__ __forceinline__ uint32_t wave_max_to_lane63(uint32_t v) {
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xb1, 0xf, 0xf, false));   // quad_perm [1,0,3,2]
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4e, 0xf, 0xf, false));   // quad_perm [2,3,0,1]
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x124, 0xf, 0xf, false));  // row_ror:4
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x128, 0xf, 0xf, false));  // row_ror:8
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false));  // row_bcast:15
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false));  // row_bcast:31
    return v;
}

// (The same launch clears the record bitmask and writes the pair reduction's
// first pair of every 64 instances, both grid-stride.)
__global__ __launch_bounds__(256) void k_slot_work(const uint32_t* __restrict__ partLast,
                                                   const uint32_t* __restrict__ counters, uint32_t* __restrict__ work,
                                                   uint32_t* __restrict__ wtab, uint32_t* __restrict__ touched,
                                                   int64_t touched_words, const uint32_t* __restrict__ pair_off,
                                                   uint32_t* __restrict__ first_pair, int rounds) {
    __shared__ uint32_t s_c[SW_CLS];
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < touched_words; i += (int64_t)gridDim.x * 256)
        touched[i] = 0u;
    wave_first_pairs(pair_off, counters, first_pair);
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    if (threadIdx.x < SW_CLS) s_c[threadIdx.x] = 0u;
    __syncthreads();
    const int64_t ns = (int64_t)counters[2];
    const int64_t base = ((int64_t)blockIdx.x * SW_SLOTS + wv * (SW_SLOTS / 4)) * rounds;
    for (int k0 = 0; k0 < SW_SLOTS / 4 * rounds; k0 += SW_CHUNK) {
        // all loads first (a slot past the count reads slot 0 and is not stored;
        // this launch has at least one slot of capacity)
        uint4 v[SW_CHUNK];
#pragma unroll
        for (int k = 0; k < SW_CHUNK; ++k) {
            const int64_t slot = base + k0 + k;
            v[k] = reinterpret_cast<const uint4*>(partLast + (slot < ns ? slot : 0) * 256)[lane];
        }
#pragma unroll
        for (int k = 0; k < SW_CHUNK; ++k) {
            const int64_t slot = base + k0 + k;
            const uint32_t m = wave_max_to_lane63(max(max(v[k].x, v[k].y), max(v[k].z, v[k].w)));
            if (lane == 63 && slot < ns) {
                work[slot] = m;
                if (m) atomicAdd(&s_c[slot_class(m)], 1u);
            }
        }
    }
    __syncthreads();
    if (threadIdx.x < SW_CLS) wtab[(size_t)blockIdx.x * SW_CLS + threadIdx.x] = s_c[threadIdx.x];
}

// n_launch: the number of launched slots (written by block 0).
__global__ __launch_bounds__(256) void k_slot_place(const uint32_t* __restrict__ work,
                                                    const uint32_t* __restrict__ counters,
                                                    const uint32_t* __restrict__ wtab, uint32_t* __restrict__ n_launch,
                                                    uint32_t* __restrict__ order, int rounds) {
    constexpr int NG = 256 / SW_CLS;  // row groups per class column
    __shared__ uint32_t s_tot[NG][SW_CLS], s_bef[NG][SW_CLS], s_base[SW_CLS], s_c[SW_CLS];
    const int t = threadIdx.x, c = t % SW_CLS, g = t / SW_CLS;
    const int64_t ns = (int64_t)counters[2];
    const int64_t per = (int64_t)SW_SLOTS * rounds;
    const int nblk = (int)((ns + per - 1) / per);
    {  // the table's column c, rows g, g + NG, ...: all blocks, and the blocks before this one
        uint32_t tot = 0, bef = 0;
        for (int r0 = g; r0 < nblk; r0 += 8 * NG) {
            uint32_t x[8];  // eight loads issued before their adds
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const int r = r0 + NG * k;
                x[k] = r < nblk ? wtab[(size_t)r * SW_CLS + c] : 0u;
            }
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                tot += x[k];
                bef += r0 + NG * k < (int)blockIdx.x ? x[k] : 0u;
            }
        }
        s_tot[g][c] = tot;
        s_bef[g][c] = bef;
    }
    if (t < SW_CLS) s_c[t] = 0u;
    __syncthreads();
    if (t < SW_CLS) {
        uint32_t tot = 0, bef = 0;
        for (int k = 0; k < NG; ++k) {
            tot += s_tot[k][t];
            bef += s_bef[k][t];
        }
        s_tot[0][t] = tot;
        s_bef[0][t] = bef;
    }
    __syncthreads();
    if (t == 0) {
        uint32_t run = 0;
        for (int k = SW_CLS - 1; k >= 0; --k) {
            s_base[k] = run + s_bef[0][k];
            run += s_tot[0][k];
        }
        if (blockIdx.x == 0) *n_launch = run;
    }
    __syncthreads();
    for (int64_t o = t; o < per; o += 256) {
        const int64_t i = (int64_t)blockIdx.x * per + o;
        const uint32_t wk = i < ns ? work[i] : 0u;
        if (wk) {
            const int k = slot_class(wk);
            order[s_base[k] + atomicAdd(&s_c[k], 1u)] = (uint32_t)i;
        }
    }
}

// The partial-render backward alone: per-instance records into the workspace.
rgs_status render_bwd_records_launch(const rgs_partials_grad* dparts, const rgs_partials* parts, const rgs_bins* bins,
                                     const rgs_projected* proj, int64_t pairs, const ViewTable* vt, const rgs_kdtree* kd,
                                     void* ws, size_t ws_bytes, uint64_t* stats, int64_t slot_bound, hipStream_t s) {
    const BwdWs w = carve_bwd(bins, pairs, ws, ws_bytes);
    // no record yet: the bitmask is cleared by a fill kernel (not a memset:
    // the call may be captured), with the launch order's first pass
    // (and the pair reduction's first pair of every 64 instances, which it
    // reads from this workspace)
    if (slot_bound <= 0) {
        const int64_t nb = ((int64_t)w.touched_words + 255) / 256;
        hipLaunchKernelGGL(k_clear_words, dim3((unsigned)(nb < 1024 ? (nb > 0 ? nb : 1) : 1024)), dim3(256), 0, s,
                           w.touched, (int64_t)w.touched_words);
        hipLaunchKernelGGL(k_clear_words, dim3(1), dim3(256), 0, s, w.work, w.flag_words);  // (the pairs' flags)
        const int64_t pb = (bins->capacity + 255) / 256;
        hipLaunchKernelGGL(k_wave_first, dim3((unsigned)(pb < 2048 ? (pb > 0 ? pb : 1) : 2048)), dim3(256), 0, s,
                           bins->pair_off, bins->counters, w.first_pair);
        return launch_check();
    }
    // every block of the placement reads the whole class table: many slots take
    // more per block, still hundreds of blocks (16 views, 825k slots: placement
    // 1551 us with 64 slots per block, now 124)
    const int rounds = slot_bound >= (1 << 20) ? 16 : (slot_bound >= (1 << 16) ? 4 : 1);
    const unsigned nblk = (unsigned)((slot_bound + SW_SLOTS * rounds - 1) / (SW_SLOTS * rounds));
    hipLaunchKernelGGL(k_slot_work, dim3(nblk), dim3(256), 0, s, parts->last, bins->counters, w.work, w.wtab, w.touched,
                       (int64_t)w.touched_words, bins->pair_off, w.first_pair, rounds);
    hipLaunchKernelGGL(k_slot_place, dim3(nblk), dim3(256), 0, s, w.work, bins->counters, w.wtab, w.wcls, w.order, rounds);
    if (stats)
        hipLaunchKernelGGL(k_render_bwd<true>, dim3((unsigned)slot_bound), dim3(128), 0, s, proj->rec, bins->vals,
                           bins->slot_key, bins->slot_range, w.order, w.wcls, vt, kd->box_lo, kd->box_hi,
                           parts->T, parts->last, dparts->dC, dparts->dT, w.records, w.touched,
                           bins->counters, w.work, reinterpret_cast<unsigned long long*>(stats));
    else
        hipLaunchKernelGGL(k_render_bwd<false>, dim3((unsigned)slot_bound), dim3(128), 0, s, proj->rec, bins->vals,
                           bins->slot_key, bins->slot_range, w.order, w.wcls, vt, kd->box_lo, kd->box_hi,
                           parts->T, parts->last, dparts->dC, dparts->dT, w.records, w.touched,
                           bins->counters, w.work, nullptr);
    return launch_check();
}

// The per-pair sums of the records in the workspace.
rgs_status pair_reduce_launch(const rgs_bins* bins, const rgs_projected* proj, int64_t n, int n_views, float* dproj,
                              void* ws, size_t ws_bytes, hipStream_t s) {
    const int64_t m = (int64_t)n_views * n;
    const BwdWs w = carve_bwd(bins, m, ws, ws_bytes);
    // one wave per 64 instances up to the capacity; waves past the device-side
    // instance count return at once
    // (the records call wrote first_pair)
    if (bins->capacity > 0) {
        hipLaunchKernelGGL(k_pair_seg, dim3((unsigned)((bins->capacity + 255) / 256)), dim3(256), 0, s, w.records,
                           w.touched, bins->pair_off, bins->counters, w.first_pair, w.psum, w.wpart,
                           reinterpret_cast<uint8_t*>(w.work));
    }
    RGS_LAUNCH_CHECK();
    if (m > 0)
        hipLaunchKernelGGL(k_pair_gather, dim3((unsigned)((m + 255) / 256)), dim3(256), 0, s, w.psum, w.wpart,
                           w.touched, reinterpret_cast<const uint8_t*>(w.work), proj->count, bins->pair_rank, bins->counters, m, dproj);
    return launch_check();
}

}  // namespace rgs
