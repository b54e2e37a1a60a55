// loss.hip -- L1 + w (1 - SSIM) on one view, forward and backward.
//
// SSIM uses an 11x11 Gaussian window (std 1.5, normalised), zero padding and
// C1 = 0.01^2, C2 = 0.03^2; the window is separable, so the local moments
// take a horizontal and a vertical 11-tap pass, both run from LDS: on 32x16
// tiles with a 5-pixel halo or, for large views, along strips of 118 columns.  E[x^2] and E[y^2] enter SSIM only through
// sigma_x^2 + sigma_y^2, so four moments are filtered: mu_x, mu_y,
// E[x^2 + y^2] and E[xy].  The backward needs d SSIM / d (mu_x, E[x^2], E[xy])
// per pixel, convolved again with the (symmetric) window.  Block partial sums
// are combined by one block in a fixed order, so the scalar is reproducible.
#include <mutex>

#include "common.hpp"

namespace rgs {

struct Win11 { float w[11]; };

static constexpr int LS_THREADS = 256;

__global__ __launch_bounds__(LS_THREADS) void k_l1_only(const float* __restrict__ x, const float* __restrict__ y, int64_t m,
                                                        float invN, float* __restrict__ dx, float* __restrict__ part) {
    __shared__ float s_w[4];
    const int64_t i = (int64_t)blockIdx.x * LS_THREADS + threadIdx.x;
    float a = 0.f;
    if (i < m) {
        const float d = x[i] - y[i];
        a = fabsf(d);
        dx[i] = (float)((d > 0.f) - (d < 0.f)) * invN;
    }
    a = wave_sum(a);
    if ((threadIdx.x & 63) == 0) s_w[threadIdx.x >> 6] = a;
    __syncthreads();
    if (threadIdx.x == 0) {
        part[2 * blockIdx.x] = (s_w[0] + s_w[1]) + (s_w[2] + s_w[3]);
        part[2 * blockIdx.x + 1] = 0.f;
    }
}

// Tiled SSIM: one 256-thread block per 32x16 output tile of one channel,
// with the 5-pixel halo staged in LDS; both separable passes run from LDS.
// (32x16 rather than 32x32: 25 KB of LDS per block instead of 41 KB, so that
// five blocks share a CU instead of three and the passes of one block
// overlap the loads of another.)  Tiles are handed out in XCD bands: a tile's
// halo rows were loaded by the tile row above it into the same L2.
static constexpr int HALO = 5;
static constexpr int TS = 32, TW = TS + 2 * HALO;       // output / staged columns (42)
static constexpr int TSY = 16, TH = TSY + 2 * HALO;     // output / staged rows (26)
static constexpr int RPT = TSY / 8;                      // output rows per thread in the vertical pass
static constexpr int VWIN = RPT + 2 * HALO;              // its window of horizontal results
// Staging: thread (column c, row group g) of TW x SG loads rows g, g + SG, ...
// of the tile with its halo (index arithmetic once per thread, not per value).
static constexpr int SG = LS_THREADS / TW;               // 6 row groups
static_assert(SG >= 1 && TW * SG <= LS_THREADS, "staging layout");
static constexpr int SR = (TH + SG - 1) / SG;            // rows per thread (5)

// Forward: SSIM map terms and d SSIM / d (mu_x, E[x^2], E[xy]) per pixel,
// plus block sums of the SSIM map and of |x - y|.
__global__ __launch_bounds__(LS_THREADS) void k_ssim_fwd_tiled(const float* __restrict__ x, const float* __restrict__ y,
                                                               int H, int W, Win11 win, float* __restrict__ d3,
                                                               float* __restrict__ part) {
    __shared__ float sx[TH * TW], sy[TH * TW];
    __shared__ float hm[4][TH * TS];
    __shared__ float s_w[2][4];
    const int tiles_x = (W + TS - 1) / TS, tiles_y = (H + TSY - 1) / TSY;
    const int b = xcd_band((int)blockIdx.x, (int)gridDim.x);  // neighbouring tiles on one XCD
    const int ch = b / (tiles_x * tiles_y);
    const int tt = b % (tiles_x * tiles_y);
    const int x0 = (tt % tiles_x) * TS, y0 = (tt / tiles_x) * TSY;
    const int64_t HW = (int64_t)H * W;
    const float* xc = x + ch * HW;
    const float* yc = y + ch * HW;
    if (threadIdx.x < TW * SG) {
        const int c = threadIdx.x % TW, g = threadIdx.x / TW;
        const int gx = x0 + c - HALO;
        const bool xin = gx >= 0 && gx < W;
        // all loads of the thread are issued before the stores
        float vx[SR], vy[SR];
#pragma unroll
        for (int i = 0; i < SR; ++i) {
            const int r = g + SG * i, gy = y0 + r - HALO;
            const bool in = r < TH && xin && gy >= 0 && gy < H;
            const int64_t gi = (int64_t)gy * W + gx;
            vx[i] = in ? xc[gi] : 0.f;
            vy[i] = in ? yc[gi] : 0.f;
        }
#pragma unroll
        for (int i = 0; i < SR; ++i) {
            const int r = g + SG * i;
            if (r < TH) {
                sx[r * TW + c] = vx[i];
                sy[r * TW + c] = vy[i];
            }
        }
    }
    __syncthreads();
    // horizontal pass: a thread takes 4 consecutive outputs of one row from a
    // 14-value window in registers (the taps of each output in the same order)
    for (int k = threadIdx.x; k < TH * (TS / 4); k += LS_THREADS) {
        const int r = k >> 3, c0 = (k & 7) * 4;
        float xv[14], yv[14], ss[14], xy[14];
#pragma unroll
        for (int j = 0; j < 14; ++j) {
            xv[j] = sx[r * TW + c0 + j];
            yv[j] = sy[r * TW + c0 + j];
            ss[j] = xv[j] * xv[j] + yv[j] * yv[j];  // products once per input, not once per tap
            xy[j] = xv[j] * yv[j];
        }
#pragma unroll
        for (int o = 0; o < 4; ++o) {
            float a0 = 0.f, a1 = 0.f, a2 = 0.f, a3 = 0.f;
#pragma unroll
            for (int t = 0; t < 11; ++t) {
                const float w = win.w[t];
                a0 = fmaf(w, xv[o + t], a0);
                a1 = fmaf(w, yv[o + t], a1);
                a2 = fmaf(w, ss[o + t], a2);
                a3 = fmaf(w, xy[o + t], a3);
            }
            const int q = r * TS + c0 + o;
            hm[0][q] = a0; hm[1][q] = a1; hm[2][q] = a2; hm[3][q] = a3;
        }
    }
    __syncthreads();
    float l1 = 0.f, ss = 0.f;
    // vertical pass: thread (column c, row group) takes RPT consecutive rows
    {
        const int c = threadIdx.x & 31, r0 = (threadIdx.x >> 5) * RPT;
        float mom[4][RPT];
#pragma unroll
        for (int mm = 0; mm < 4; ++mm) {
            float hv[VWIN];
#pragma unroll
            for (int j = 0; j < VWIN; ++j) hv[j] = hm[mm][(r0 + j) * TS + c];
#pragma unroll
            for (int o = 0; o < RPT; ++o) {
                float a = 0.f;
#pragma unroll
                for (int t = 0; t < 11; ++t) a = fmaf(win.w[t], hv[o + t], a);
                mom[mm][o] = a;
            }
        }
#pragma unroll
        for (int o = 0; o < RPT; ++o) {
            const int r = r0 + o;
            const int gy = y0 + r, gx = x0 + c;
            if (gy >= H || gx >= W) continue;
            const float mu_x = mom[0][o], mu_y = mom[1][o], ess = mom[2][o], exy = mom[3][o];
            const float C1 = 1e-4f, C2 = 9e-4f;
            const float A1 = 2.f * mu_x * mu_y + C1;
            const float A2 = 2.f * (exy - mu_x * mu_y) + C2;
            const float m2 = mu_x * mu_x + mu_y * mu_y;
            const float B1 = m2 + C1;
            const float B2 = (ess - m2) + C2;
            const float Nn = A1 * A2, Dd = B1 * B2;
            const float iD = 1.f / Dd;
            ss += Nn * iD;
            const float dN = 2.f * mu_y * A2 - 2.f * mu_y * A1;
            const float dD = 2.f * mu_x * B2 - 2.f * mu_x * B1;
            const int64_t i = ch * HW + (int64_t)gy * W + gx;
            const int64_t m = 3 * HW;
            d3[i] = (dN * Dd - Nn * dD) * iD * iD;
            d3[m + i] = -Nn * B1 * iD * iD;
            d3[2 * m + i] = 2.f * A1 * iD;
            l1 += fabsf(sx[(r + HALO) * TW + c + HALO] - sy[(r + HALO) * TW + c + HALO]);
        }
    }
    l1 = wave_sum(l1);
    ss = wave_sum(ss);
    if ((threadIdx.x & 63) == 0) { s_w[0][threadIdx.x >> 6] = l1; s_w[1][threadIdx.x >> 6] = ss; }
    __syncthreads();
    if (threadIdx.x == 0) {
        part[2 * b] = (s_w[0][0] + s_w[0][1]) + (s_w[0][2] + s_w[0][3]);
        part[2 * b + 1] = (s_w[1][0] + s_w[1][1]) + (s_w[1][2] + s_w[1][3]);
    }
}

// The final sums of the block partials in one block of NT threads: a fixed
// order of additions for a given NT (reproducible).  s_a, s_b: NT doubles of
// LDS each.
template <int NT, class P2>
__device__ __forceinline__ void loss_final_sums(const P2* __restrict__ part, int nb, float invN, float w,
                                                float* __restrict__ loss, double* s_a, double* s_b) {
    double a = 0.0, b = 0.0;
    // the same order of additions per thread as one partial at a time; the
    // loads of eight steps are issued before their adds
    constexpr int U = 8;
    int k = threadIdx.x;
    for (; k + (U - 1) * NT < nb; k += U * NT) {
        P2 pv[U];
#pragma unroll
        for (int u = 0; u < U; ++u) pv[u] = part[k + u * NT];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            a += pv[u].x;
            b += pv[u].y;
        }
    }
    for (; k < nb; k += NT) { a += part[k].x; b += part[k].y; }
    s_a[threadIdx.x] = a;
    s_b[threadIdx.x] = b;
    __syncthreads();
    for (int st = NT / 2; st > 0; st >>= 1) {
        if (threadIdx.x < st) { s_a[threadIdx.x] += s_a[threadIdx.x + st]; s_b[threadIdx.x] += s_b[threadIdx.x + st]; }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        double l = s_a[0] * (double)invN;
        if (w != 0.f) l += (double)w * (1.0 - s_b[0] * (double)invN);
        *loss = (float)l;
    }
}

static constexpr int LF_THREADS = 1024;

template <class P2>
__global__ __launch_bounds__(LF_THREADS) void k_loss_final(const P2* __restrict__ part, int nb, float invN, float w,
                                                           float* __restrict__ loss) {
    __shared__ double s_a[LF_THREADS], s_b[LF_THREADS];
    loss_final_sums<LF_THREADS, P2>(part, nb, invN, w, loss, s_a, s_b);
}

// Backward: convolve the three derivative maps with the (symmetric) window
// and combine: dL/dx = sign(x - y)/N + sc (w*g_mu + 2 x w*g_xx + y w*g_xy).
// Block 0 adds up the forward's block partials into the loss (dispatched
// first, it runs beside the tiles instead of as a launch of its own);
// blocks 1.. take the tiles.
__global__ __launch_bounds__(LS_THREADS) void k_ssim_bwd_tiled(const float* __restrict__ x, const float* __restrict__ y,
                                                               const float* __restrict__ d3, int H, int W, Win11 win,
                                                               float invN, float sc, float* __restrict__ dx,
                                                               const float* __restrict__ part, float ssim_w,
                                                               float* __restrict__ loss) {
    __shared__ __align__(16) float sd[3][TH * TW];
    __shared__ float hm[3][TH * TS];
    static_assert(sizeof(sd) >= 2 * LS_THREADS * sizeof(double), "final sums reuse the staging array");
    const int tiles_x = (W + TS - 1) / TS, tiles_y = (H + TSY - 1) / TSY;
    const int ntiles = (int)gridDim.x - 1;
    if (blockIdx.x == 0) {
        double* s2 = reinterpret_cast<double*>(&sd[0][0]);
        loss_final_sums<LS_THREADS>(reinterpret_cast<const float2*>(part), ntiles, invN, ssim_w, loss, s2, s2 + LS_THREADS);
        return;
    }
    const int b = xcd_band((int)blockIdx.x - 1, ntiles);  // neighbouring tiles on one XCD
    const int ch = b / (tiles_x * tiles_y);
    const int tt = b % (tiles_x * tiles_y);
    const int x0 = (tt % tiles_x) * TS, y0 = (tt / tiles_x) * TSY;
    const int64_t HW = (int64_t)H * W;
    const int64_t m = 3 * HW;
    if (threadIdx.x < TW * SG) {
        const int c = threadIdx.x % TW, g = threadIdx.x / TW;
        const int gx = x0 + c - HALO;
        const bool xin = gx >= 0 && gx < W;
        float v0[SR], v1[SR], v2[SR];
#pragma unroll
        for (int k = 0; k < SR; ++k) {
            const int r = g + SG * k, gy = y0 + r - HALO;
            const bool in = r < TH && xin && gy >= 0 && gy < H;
            const int64_t i = ch * HW + (int64_t)gy * W + gx;
            v0[k] = in ? d3[i] : 0.f;
            v1[k] = in ? d3[m + i] : 0.f;
            v2[k] = in ? d3[2 * m + i] : 0.f;
        }
#pragma unroll
        for (int k = 0; k < SR; ++k) {
            const int r = g + SG * k;
            if (r < TH) {
                sd[0][r * TW + c] = v0[k];
                sd[1][r * TW + c] = v1[k];
                sd[2][r * TW + c] = v2[k];
            }
        }
    }
    __syncthreads();
    for (int k = threadIdx.x; k < TH * (TS / 4); k += LS_THREADS) {
        const int r = k >> 3, c0 = (k & 7) * 4;
#pragma unroll
        for (int mm = 0; mm < 3; ++mm) {
            float v[14];
#pragma unroll
            for (int j = 0; j < 14; ++j) v[j] = sd[mm][r * TW + c0 + j];
#pragma unroll
            for (int o = 0; o < 4; ++o) {
                float a = 0.f;
#pragma unroll
                for (int t = 0; t < 11; ++t) a = fmaf(win.w[t], v[o + t], a);
                hm[mm][r * TS + c0 + o] = a;
            }
        }
    }
    __syncthreads();
    {
        const int c = threadIdx.x & 31, r0 = (threadIdx.x >> 5) * RPT;
        float gm[3][RPT];
#pragma unroll
        for (int mm = 0; mm < 3; ++mm) {
            float hv[VWIN];
#pragma unroll
            for (int j = 0; j < VWIN; ++j) hv[j] = hm[mm][(r0 + j) * TS + c];
#pragma unroll
            for (int o = 0; o < RPT; ++o) {
                float a = 0.f;
#pragma unroll
                for (int t = 0; t < 11; ++t) a = fmaf(win.w[t], hv[o + t], a);
                gm[mm][o] = a;
            }
        }
#pragma unroll
        for (int o = 0; o < RPT; ++o) {
            const int gy = y0 + r0 + o, gx = x0 + c;
            if (gy >= H || gx >= W) continue;
            const int64_t i = ch * HW + (int64_t)gy * W + gx;
            const float xv = x[i], yv = y[i];
            const float d = xv - yv;
            const float l1g = (float)((d > 0.f) - (d < 0.f)) * invN;
            dx[i] = l1g + sc * (gm[0][o] + 2.f * xv * gm[1][o] + yv * gm[2][o]);
        }
    }
}

// SSIM and its gradient in one pass: a block owns SO output columns of one
// channel and marches down seg_rows rows of them (and the 10 above and below
// that these see), a batch of SB rows at a time:
//   1 the inputs of the batch to LDS (loaded one batch ahead),
//   2 horizontal taps of the four moments, four columns per thread,
//   3 vertical taps: a thread owns a column and holds, per moment, the partial
//     sums of the ten windows in progress; a row adds its tap to each of them
//     while they move on by one (the destination of the fma is the next one),
//     and the one that leaves is a moment.  From the moments, the SSIM term and
//     its derivatives by (mu_x, E[x^2], E[xy]), which stay in LDS,
//   4, 5 the same two steps for the derivatives, and dL/dx of the row.
// The vertical halo is computed once per segment instead of once per 16 rows,
// and the derivative maps never reach memory (24 bytes per value).  What bounds it
// is vector issue: 86 % of the time at 3840x2160x3, where the loss takes 236 us
// instead of 367.  (The taps as 4x4x1 matrix products take a third of the vector issue away, but
// at 2 to 3 waves per SIMD their chains' latency takes its place: 258 us; as banded
// 16x16x4 products 279; 128 registers and 4 waves spill: 310.)
// Every tap is added in the same order as in a direct sum over the window.
static constexpr int SC = 128;                 // moment columns = threads
static constexpr int SO = SC - 2 * HALO;       // output columns (118)
static constexpr int SI = SC + 2 * HALO;       // input columns (138)
static constexpr int SB = 4;                   // rows per batch
static constexpr int SD = SC + 4;              // row of the derivative maps in LDS (read in fours beyond SO)
static constexpr int SH = 4 * ((SO + 3) / 4);  // row of their horizontal results (120)
static_assert(SB * (SC / 4) == SC && SB * (SH / 4) <= SC, "one group of four columns per thread");

// One row into the column's windows: returns the sum that is complete.
__device__ __forceinline__ float tap_down(float (&acc)[10], const Win11& win, float h) {
    const float out = fmaf(win.w[10], h, acc[9]);
#pragma unroll
    for (int j = 9; j > 0; --j) acc[j] = fmaf(win.w[j], h, acc[j - 1]);
    acc[0] = fmaf(win.w[0], h, 0.f);
    return out;
}

// Four neighbouring outputs of the horizontal taps.
__device__ __forceinline__ float4 tap_across(const float (&v)[14], const Win11& win) {
    float o[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        o[i] = 0.f;
#pragma unroll
        for (int t = 0; t < 11; ++t) o[i] = fmaf(win.w[t], v[i + t], o[i]);
    }
    return make_float4(o[0], o[1], o[2], o[3]);
}

__device__ __forceinline__ float ld_at(const float* row, uint32_t byte) {  // (a scalar base and a 32-bit offset)
    return *reinterpret_cast<const float*>(reinterpret_cast<const char*>(row) + byte);
}

__global__ __launch_bounds__(SC, 3) void k_ssim(const float* __restrict__ x, const float* __restrict__ y, int H, int W,
                                                Win11 win, int strips, int segs, int seg_rows, float invN, float sc,
                                                float* __restrict__ dx, double* __restrict__ part) {
    __shared__ __align__(16) float2 s_in[SB][SI];
    __shared__ __align__(16) float s_h[4][SB][SC];  // and the derivatives' horizontal results, [3][SB][SH]
    __shared__ __align__(16) float s_d[3][SB][SD];
    __shared__ double s_w[2][2];
    static_assert(3 * SB * SH <= 4 * SB * SC, "aliased");
    float(*s_b)[SB][SH] = reinterpret_cast<float(*)[SB][SH]>(&s_h[0][0][0]);
    const int b = xcd_band((int)blockIdx.x, (int)gridDim.x);  // neighbouring strips on one XCD
    const int strip = b % strips, seg = (b / strips) % segs, ch = b / (strips * segs);
    const int x0 = strip * SO, ys = seg * seg_rows, ye = min(ys + seg_rows, H);
    const size_t HW = (size_t)H * W;
    const float *xc = x + ch * HW, *yc = y + ch * HW;
    float* dc = dx + ch * HW;
    const int t = threadIdx.x;

    // inputs: thread t takes column t of every row, and the first 10 SB threads
    // the columns beyond; outside the image (zero padding) a clamped load is made
    // and dropped
    const int gx = x0 - 2 * HALO + t;
    const uint32_t at1 = 4u * (uint32_t)min(max(gx, 0), W - 1);
    const bool x_in = gx >= 0 && gx < W;
    const int k2 = min(t / (SI - SC), SB), c2 = SC + t % (SI - SC);
    const int gx2 = x0 - 2 * HALO + c2, gx2c = min(max(gx2, 0), W - 1);
    const bool x2_in = gx2 >= 0 && gx2 < W;
    float vx[SB], vy[SB], vx2, vy2;
    auto load = [&](int row) {
#pragma unroll
        for (int k = 0; k < SB; ++k) {
            const size_t at = (size_t)min(max(row + k, 0), H - 1) * W;
            vx[k] = ld_at(xc + at, at1);
            vy[k] = ld_at(yc + at, at1);
        }
        const size_t at2 = (size_t)min(max(row + min(k2, SB - 1), 0), H - 1) * W + gx2c;
        vx2 = xc[at2];
        vy2 = yc[at2];
    };

    float mom[4][10], der[3][10];
#pragma unroll
    for (int j = 0; j < 10; ++j) {
        mom[0][j] = mom[1][j] = mom[2][j] = mom[3][j] = 0.f;
        der[0][j] = der[1][j] = der[2][j] = 0.f;
    }
    double l1 = 0.0, ssim = 0.0;
    // moment column t, output column t
    const int gxm = x0 - HALO + t;
    const bool m_in = gxm >= 0 && gxm < W, m_own = m_in && t >= HALO && t < HALO + SO;
    const bool o_own = t < SO && x0 + t < W;
    const uint32_t ato = 4u * (uint32_t)min(x0 + t, W - 1);
    const int rows = (ye - ys) + 4 * HALO;
    load(ys - 2 * HALO);
    for (int i0 = 0; i0 < rows; i0 += SB) {
        const int row = ys - 2 * HALO + i0;  // input row of the batch; moments are 5 above, outputs 10
#pragma unroll
        for (int k = 0; k < SB; ++k) {
            const bool in = x_in && row + k >= 0 && row + k < H;
            s_in[k][t] = make_float2(in ? vx[k] : 0.f, in ? vy[k] : 0.f);
        }
        if (k2 < SB) {
            const bool in = x2_in && row + k2 >= 0 && row + k2 < H;
            s_in[k2][c2] = make_float2(in ? vx2 : 0.f, in ? vy2 : 0.f);
        }
        __syncthreads();
        {
            const int k = t / (SC / 4), c0 = 4 * (t % (SC / 4));
            float xv[14], yv[14], pv[14];
            const float4* in = reinterpret_cast<const float4*>(&s_in[k][c0]);
#pragma unroll
            for (int j = 0; j < 7; ++j) {
                const float4 q = in[j];
                xv[2 * j] = q.x, yv[2 * j] = q.y, xv[2 * j + 1] = q.z, yv[2 * j + 1] = q.w;
            }
            *reinterpret_cast<float4*>(&s_h[0][k][c0]) = tap_across(xv, win);
            *reinterpret_cast<float4*>(&s_h[1][k][c0]) = tap_across(yv, win);
#pragma unroll
            for (int j = 0; j < 14; ++j) pv[j] = xv[j] * xv[j] + yv[j] * yv[j];
            *reinterpret_cast<float4*>(&s_h[2][k][c0]) = tap_across(pv, win);
#pragma unroll
            for (int j = 0; j < 14; ++j) pv[j] = xv[j] * yv[j];
            *reinterpret_cast<float4*>(&s_h[3][k][c0]) = tap_across(pv, win);
        }
        __syncthreads();
        float ss = 0.f;
#pragma unroll
        for (int k = 0; k < SB; ++k) {
            const float mu_x = tap_down(mom[0], win, s_h[0][k][t]), mu_y = tap_down(mom[1], win, s_h[1][k][t]);
            const float ess = tap_down(mom[2], win, s_h[2][k][t]), exy = tap_down(mom[3], win, s_h[3][k][t]);
            const int gy = row + k - HALO;
            const float C1 = 1e-4f, C2 = 9e-4f;
            const float A1 = 2.f * mu_x * mu_y + C1;
            const float A2 = 2.f * (exy - mu_x * mu_y) + C2;
            const float m2 = mu_x * mu_x + mu_y * mu_y;
            const float B1 = m2 + C1;
            const float B2 = (ess - m2) + C2;
            const float Nn = A1 * A2, Dd = B1 * B2;
            const float iD = 1.f / Dd;
            ss += gy >= ys && gy < ye ? Nn * iD : 0.f;
            const float dN = 2.f * mu_y * A2 - 2.f * mu_y * A1;
            const float dD = 2.f * mu_x * B2 - 2.f * mu_x * B1;
            const float d0 = (dN * Dd - Nn * dD) * iD * iD, d1 = -Nn * B1 * iD * iD, d2 = 2.f * A1 * iD;
            const bool in = m_in && gy >= 0 && gy < H;  // zero padding of the derivatives
            s_d[0][k][t] = in ? d0 : 0.f;
            s_d[1][k][t] = in ? d1 : 0.f;
            s_d[2][k][t] = in ? d2 : 0.f;
        }
        // the next batch's inputs, and the values of this batch's outputs (read ten rows
        // earlier: they come from the cache)
        load(row + SB);
        float ox[SB], oy[SB];
#pragma unroll
        for (int k = 0; k < SB; ++k) {
            const size_t at = (size_t)min(max(row + k - 2 * HALO, 0), H - 1) * W;
            ox[k] = ld_at(xc + at, ato);
            oy[k] = ld_at(yc + at, ato);
        }
        if (i0 + SB <= 2 * HALO) continue;  // no window of the segment is complete yet
        ssim += (double)(m_own ? ss : 0.f);
        __syncthreads();
        if (t < SB * (SH / 4)) {
            const int k = t / (SH / 4), c0 = 4 * (t % (SH / 4));
#pragma unroll
            for (int mm = 0; mm < 3; ++mm) {
                const float4* in = reinterpret_cast<const float4*>(&s_d[mm][k][c0]);
                const float4 a = in[0], e = in[1], f = in[2];
                const float2 g = *reinterpret_cast<const float2*>(in + 3);
                const float v[14] = {a.x, a.y, a.z, a.w, e.x, e.y, e.z, e.w, f.x, f.y, f.z, f.w, g.x, g.y};
                *reinterpret_cast<float4*>(&s_b[mm][k][c0]) = tap_across(v, win);
            }
        }
        __syncthreads();
        float la = 0.f;
        const int to = min(t, SH - 1);
#pragma unroll
        for (int k = 0; k < SB; ++k) {
            const float g0 = tap_down(der[0], win, s_b[0][k][to]), g1 = tap_down(der[1], win, s_b[1][k][to]),
                        g2 = tap_down(der[2], win, s_b[2][k][to]);
            const int gy = row + k - 2 * HALO;
            const float xv = ox[k], yv = oy[k], d = xv - yv;
            la += gy >= ys && gy < ye ? fabsf(d) : 0.f;
            const float l1g = (float)((d > 0.f) - (d < 0.f)) * invN;
            const float o = l1g + sc * (g0 + 2.f * xv * g1 + yv * g2);
            if (gy >= ys && gy < ye && o_own)
                *reinterpret_cast<float*>(reinterpret_cast<char*>(dc + (size_t)gy * W) + ato) = o;
        }
        l1 += (double)(o_own ? la : 0.f);
    }
    for (int o = 32; o > 0; o >>= 1) {
        l1 += __shfl_down(l1, o);
        ssim += __shfl_down(ssim, o);
    }
    if ((t & 63) == 0) { s_w[t >> 6][0] = l1; s_w[t >> 6][1] = ssim; }
    __syncthreads();
    if (t < 2) part[2 * b + t] = s_w[0][t] + s_w[1][t];
}

// One marching pass from SSIM_MARCH values on, where its blocks' rows take less time
// than tiles.  Segments are as long as one round of blocks allows (3 waves per SIMD:
// 6 blocks per CU), since each computes ten rows above and below its own: 2048
// blocks, two rounds, take 302 us at 3840x2160.  So the pass takes 1.4 us per row of
// a segment and its halo, whatever the shape, and the tiles 12.8 us per million
// values: SSIM_ROW_VALUES values per row.  us for the loss, tiles / marching:
// 1920x1080 81 / 78, 2000x1200 93 / 84, 2560x1440 139 / 117, 3840x2160 347 / 230, 5000x3000
// 622 / 413, 60000x100 271 / 167, 236x20000 202 / 139; few rows or strips that go far
// beyond the width leave blocks or columns idle: 20901x131 112 / 121, 20500x100 88 / 99,
// 7000x300 81 / 84, 130x20000 125 / 138.  Smaller views (1600x1060 76 / 79, 997x663 36 / 54)
// are mostly the pass's start-up.
static constexpr int64_t SSIM_MARCH = 6000000, SSIM_ROW_VALUES = 109000;
static constexpr int SSIM_BLOCKS = 1536, SSIM_ROWS = 32;

// What callers size their workspaces by (a fixed array's largest view among
// them): three maps of the image and 3.1 pairs of sums per 512 values, of which the
// sums are used.
size_t loss_ws_bytes(int H, int W) {
    const int64_t m = 3 * (int64_t)H * W;
    const int64_t nb = (m + LS_THREADS - 1) / LS_THREADS;
    const int64_t nt = 3 * (int64_t)((W + TS - 1) / TS) * ((H + TSY - 1) / TSY);
    const int64_t np = nb > nt ? nb : nt;
    return (size_t)3 * m * sizeof(float) + (size_t)2 * np * sizeof(float) + 1024;
}

rgs_status loss_launch(const float* image, const float* target, int H, int W, float ssim_w, float* loss, float* dimg,
                       void* ws, hipStream_t s) {
    const int64_t m = 3 * (int64_t)H * W;
    const int64_t nb = (m + LS_THREADS - 1) / LS_THREADS;
    const int64_t nt = 3 * (int64_t)((W + TS - 1) / TS) * ((H + TSY - 1) / TSY);
    WsCarver c{reinterpret_cast<char*>(ws), 0, (size_t)-1};
    float* d3 = c.take<float>(3 * m);
    float* part = c.take<float>(2 * (nb > nt ? nb : nt));
    const float invN = (float)(1.0 / (double)m);
    Win11 win;
    double g[11], gs = 0.0;
    for (int k = 0; k < 11; ++k) { g[k] = exp(-((k - 5) * (k - 5)) / (2.0 * 1.5 * 1.5)); gs += g[k]; }
    for (int k = 0; k < 11; ++k) win.w[k] = (float)(g[k] / gs);
    const int strips = (W + SO - 1) / SO;
    const int most = SSIM_BLOCKS / (3 * strips) > 1 ? SSIM_BLOCKS / (3 * strips) : 1;  // segments
    int rows = (H + most - 1) / most;
    if (rows < SSIM_ROWS) rows = SSIM_ROWS;
    if (ssim_w == 0.f) {
        hipLaunchKernelGGL(k_l1_only, dim3((unsigned)nb), dim3(LS_THREADS), 0, s, image, target, m, invN, dimg, part);
        hipLaunchKernelGGL(k_loss_final<float2>, dim3(1), dim3(LF_THREADS), 0, s, reinterpret_cast<const float2*>(part),
                           (int)nb, invN, ssim_w, loss);
    } else if (m >= SSIM_MARCH && (rows + 4 * HALO) * SSIM_ROW_VALUES <= m) {
        const int segs = (H + rows - 1) / rows;
        double* sums = reinterpret_cast<double*>(ws);  // (no derivative maps here)
        hipLaunchKernelGGL(k_ssim, dim3((unsigned)(3 * strips * segs)), dim3(SC), 0, s, image, target, H, W, win, strips,
                           segs, rows, invN, -ssim_w * invN, dimg, sums);
        hipLaunchKernelGGL(k_loss_final<double2>, dim3(1), dim3(LF_THREADS), 0, s,
                           reinterpret_cast<const double2*>(sums), 3 * strips * segs, invN, ssim_w, loss);
    } else {
        hipLaunchKernelGGL(k_ssim_fwd_tiled, dim3((unsigned)nt), dim3(LS_THREADS), 0, s, image, target, H, W, win, d3, part);
        // the final sums in its block 0
        hipLaunchKernelGGL(k_ssim_bwd_tiled, dim3((unsigned)nt + 1u), dim3(LS_THREADS), 0, s, image, target, d3, H, W,
                           win, invN, -ssim_w * invN, dimg, part, ssim_w, loss);
    }
    return launch_check();
}

// Fixed workspace of the allocation-free loss entry point: one copy per
// device, held until the process ends.  Host code never passes the array's
// name to a kernel (on the host it is a stand-in, not a device address); it
// uses the address hipGetSymbolAddress returns for the current device, taken
// once per device and kept.
static __device__ __align__(256) unsigned char scratch[RGS_LOSS_SCRATCH_BYTES];

static constexpr int SCRATCH_MAX_DEVICES = 64;
static std::mutex g_scratch_mu;
static void* g_scratch_dev[SCRATCH_MAX_DEVICES];

rgs_status loss_scratch(void** out) {
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) {
        set_hip_error(e);
        return RGS_E_HIP;
    }
    if (dev < 0 || dev >= SCRATCH_MAX_DEVICES) return RGS_E_UNSUPPORTED;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_dev[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p) {
            set_hip_error(e != hipSuccess ? e : hipErrorInvalidSymbol);
            return RGS_E_HIP;
        }
        g_scratch_dev[dev] = p;
    }
    *out = g_scratch_dev[dev];
    return RGS_OK;
}

}  // namespace rgs
