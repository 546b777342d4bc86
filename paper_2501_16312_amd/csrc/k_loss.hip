// k_loss.hip -- the photometric loss of the optimisation (Sec. 3.4
// "Optimization": 3DGS's L1 + SSIM) and its gradient with respect to the
// rendered image, fused: per view and channel,
//   L = (1 - lam) mean |x - y| + lam (1 - mean s),
//   s = (2 mx my + C1)(2 sxy + C2) / ((mx^2 + my^2 + C1)(sxx + syy + C2)),
// local statistics by an 11 x 11 Gaussian window (sigma 1.5, zero padding).
//
// Two passes over 32 x 32 output tiles, each applying the separable window as
// a row pass (four neighbouring outputs of a row per thread, straight from
// global memory) and a column pass (through LDS):
//   k_ssim_fwd  five statistics -> s and its partial derivatives with respect
//               to mx, E[x^2], E[xy] (written per pixel), block sums of s and
//               |x - y|;
//   k_ssim_bwd  the window applied to those three derivative maps (the window
//               is symmetric, so it is its own adjoint) ->
//               dL/dx = (1 - lam) sign(x - y) / n - lam / n (G*A + 2 x G*B + y G*C).
//
// What bounds them, per 1080p view: the forward issues 25M VALU instructions
// (40 us of issue) for 125 MB of traffic, the backward 12.5M (20 us) for 150
// MB; together they take 79 us (119 when the inputs were staged in LDS first,
// with a barrier between).  Taller tiles: 32 x 48 as long, 32 x 64 13% longer
// (fewer waves per SIMD).
#include "linprim_common.h"

namespace linprim {

constexpr int kSsimHalo = 5;
constexpr int kRun = 4;                      // outputs of a row per thread of a row pass
constexpr int kRuns = kLossTile / kRun;      // runs per row of a tile
constexpr int kRowsIn = kLossTile + 2 * kSsimHalo;
constexpr float kC1 = 0.0001f;               // 0.01^2
constexpr float kC2 = 0.0009f;               // 0.03^2

struct SsimWindow {
    float w[11];
};

// The 14 inputs of the four outputs at columns x .. x + 3 of row y: columns
// x - 5 .. x + 8 (v[3] .. v[16]), zero outside the image.  In a tile away from
// the borders (`inner`, the same for the whole block) as five 16-byte loads from column x - 8 (x is a multiple of 4, so
// they are aligned where the rows are; the type only promises 4 bytes).
struct __attribute__((packed, aligned(4))) Float4u {
    float v[4];
};
constexpr int kIn = kRun + 2 * kSsimHalo;    // 14
template <bool INNER>
__device__ inline void load_run(const float* __restrict__ img, int W, int H, int x, int y, float (&v)[20]) {
    if (INNER) {
        const float* row = img + (int64_t)y * W + (x - 8);
#pragma unroll
        for (int k = 0; k < 5; ++k) {
            const Float4u q = *reinterpret_cast<const Float4u*>(row + 4 * k);
#pragma unroll
            for (int j = 0; j < 4; ++j) v[4 * k + j] = q.v[j];
        }
        return;
    }
    // the same five loads, moved inside the image where they would leave it:
    // a quad of columns is then in the image, beyond it, or, at the right
    // border of a width that is no multiple of 4, short of its last d columns
    const bool row_in = y >= 0 && y < H;
    const float* row = img + (int64_t)min(max(y, 0), H - 1) * W;
    if (W >= 4) {
#pragma unroll
        for (int k = 0; k < 5; ++k) {
            const int c = x - 8 + 4 * k, at = min(max(c, 0), W - 4), d = c - at;
            const Float4u q = *reinterpret_cast<const Float4u*>(row + at);
            const bool whole = row_in && d == 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) v[4 * k + j] = whole ? q.v[j] : 0.0f;
            if (row_in && d > 0 && d < 4) {
#pragma unroll
                for (int j = 0; j < 3; ++j)
                    if (c + j < W) v[4 * k + j] = row[c + j];
            }
        }
    } else {
#pragma unroll
        for (int k = 0; k < 20; ++k) {
            const int c = x - 8 + k;
            v[k] = row_in && c >= 0 && c < W ? row[c] : 0.0f;
        }
    }
}

// Different code at the end of the two forms of a row pass, so that the
// compiler does not merge their arithmetic behind the two ways of loading:
// merged, every run waits for all of its loads before the first product (four
// views of 288 x 229: 42 us apart, 46 merged).
template <bool INNER>
__device__ inline void keep_apart() {
    if (INNER) asm volatile("; inner tile");
    else asm volatile("; border tile");
}

// Tile of block b of a launch of T tiles padded to a multiple of 8 blocks:
// consecutive blocks go to different XCDs, so XCD x = b % 8 is given the tiles
// x ceil(T / 8) .. , in order, whose halos then meet in its L2 (four 1080p
// views: 342 us against 405 in plain order).
struct SsimTile {
    int x0, y0, ch;
    uint32_t index;
    bool valid, inner;   // inner: every input of the tile's row pass, in 20-column runs, is in the image
};
__device__ inline SsimTile ssim_tile(int W, int H) {
    const uint32_t tx = (uint32_t)(W + kLossTile - 1) / kLossTile, ty = (uint32_t)(H + kLossTile - 1) / kLossTile;
    const uint32_t t = (blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
    const uint32_t ch = t / (tx * ty), r = t - ch * (tx * ty);
    const uint32_t row = r / tx;
    SsimTile T;
    T.x0 = (int)(r - row * tx) * kLossTile;
    T.y0 = (int)row * kLossTile;
    T.ch = (int)ch;
    T.index = t;
    T.valid = ch < 3;
    T.inner = T.x0 >= 8 && T.x0 + kLossTile + 8 <= W && T.y0 >= kSsimHalo && T.y0 + kLossTile + kSsimHalo <= H;
    return T;
}

__device__ inline float wave_sum_f(float v) {
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// Row pass of the forward: the five statistics of every row of the tile and
// its halo, and the sum of |x - y| over the tile's own pixels.
template <int NT, bool INNER>
__device__ inline void ssim_rows(const float* __restrict__ X, const float* __restrict__ Y, int W, int H, int x0, int y0,
                                 const SsimWindow& win, float (*hs)[kRowsIn * kLossTile], float& l1) {
    for (int k = threadIdx.x; k < kRowsIn * kRuns; k += NT) {
        const int r = k / kRuns, c0 = (k % kRuns) * kRun;
        const int y = y0 - kSsimHalo + r;
        float xv[20], yv[20];
        load_run<INNER>(X, W, H, x0 + c0, y, xv);
        load_run<INNER>(Y, W, H, x0 + c0, y, yv);
        float acc[5][kRun];
#pragma unroll
        for (int q = 0; q < kRun; ++q)
#pragma unroll
            for (int m = 0; m < 5; ++m) acc[m][q] = 0.f;
#pragma unroll
        for (int i = 0; i < kIn; ++i) {
            const float a = xv[i + 3], b = yv[i + 3];
            const float aa = a * a, bb = b * b, ab = a * b;
#pragma unroll
            for (int q = 0; q < kRun; ++q) {
                const int u = i - q;     // tap of output c0 + q
                if (u < 0 || u > 10) continue;
                const float wt = win.w[u];
                acc[0][q] += wt * a;
                acc[1][q] += wt * b;
                acc[2][q] += wt * aa;
                acc[3][q] += wt * bb;
                acc[4][q] += wt * ab;
            }
        }
        // the tile's own pixels (zero beyond the image on both sides)
        if (r >= kSsimHalo && r < kSsimHalo + kLossTile) {
            float run = 0.0f;
#pragma unroll
            for (int q = 0; q < kRun; ++q)
                if (INNER || x0 + c0 + q < W) run += fabsf(xv[8 + q] - yv[8 + q]);
            l1 += run;
        }
#pragma unroll
        for (int m = 0; m < 5; ++m)
            *reinterpret_cast<float4*>(&hs[m][r * kLossTile + c0]) = make_float4(acc[m][0], acc[m][1], acc[m][2], acc[m][3]);
        keep_apart<INNER>();
    }
}

// Row pass of the backward: the three derivative maps.
template <int NT, bool INNER>
__device__ inline void ssim_rows_bwd(const float* __restrict__ dm, int64_t hw, int W, int H, int x0, int y0,
                                     const SsimWindow& win, float (*hs)[kRowsIn * kLossTile]) {
    for (int k = threadIdx.x; k < kRowsIn * kRuns; k += NT) {
        const int r = k / kRuns, c0 = (k % kRuns) * kRun;
        float v[3][20];
#pragma unroll
        for (int m = 0; m < 3; ++m) load_run<INNER>(dm + m * hw, W, H, x0 + c0, y0 - kSsimHalo + r, v[m]);
        float acc[3][kRun];
#pragma unroll
        for (int q = 0; q < kRun; ++q)
#pragma unroll
            for (int m = 0; m < 3; ++m) acc[m][q] = 0.f;
#pragma unroll
        for (int i = 0; i < kIn; ++i) {
#pragma unroll
            for (int q = 0; q < kRun; ++q) {
                const int u = i - q;
                if (u < 0 || u > 10) continue;
                const float wt = win.w[u];
#pragma unroll
                for (int m = 0; m < 3; ++m) acc[m][q] += wt * v[m][i + 3];
            }
        }
#pragma unroll
        for (int m = 0; m < 3; ++m)
            *reinterpret_cast<float4*>(&hs[m][r * kLossTile + c0]) = make_float4(acc[m][0], acc[m][1], acc[m][2], acc[m][3]);
        keep_apart<INNER>();
    }
}

template <int NT>
__global__ __launch_bounds__(NT) void k_ssim_fwd(const float* __restrict__ rgb, const float* __restrict__ target,
                                                  int W, int H, SsimWindow win, float* __restrict__ dmaps,
                                                  float* __restrict__ partial, const uint32_t* __restrict__ skip) {
    if (skip && *skip) return;
    __shared__ __attribute__((aligned(16))) float hs[5][kRowsIn * kLossTile];
    __shared__ double red[2][NT / 64];
    const SsimTile tile = ssim_tile(W, H);
    if (!tile.valid) return;
    const int ch = tile.ch, x0 = tile.x0, y0 = tile.y0;
    const int64_t hw = (int64_t)W * H;
    const float* X = rgb + ch * hw;
    const float* Y = target + ch * hw;
    float ssum = 0.f, l1 = 0.f;
    if (tile.inner)
        ssim_rows<NT, true>(X, Y, W, H, x0, y0, win, hs, l1);
    else
        ssim_rows<NT, false>(X, Y, W, H, x0, y0, win, hs, l1);
    __syncthreads();
    // column pass: a thread takes PER neighbouring rows of one column (4, or 2
    // with eight waves; lanes run along a row, so the map stores are coalesced)
    {
        constexpr int PER = kLossTile * kLossTile / NT;
        const int c = threadIdx.x % kLossTile, r0 = (threadIdx.x / kLossTile) * PER;
        float acc[5][PER];
#pragma unroll
        for (int q = 0; q < PER; ++q)
#pragma unroll
            for (int m = 0; m < 5; ++m) acc[m][q] = 0.f;
#pragma unroll
        for (int i = 0; i < PER + 10; ++i) {
            float v[5];
#pragma unroll
            for (int m = 0; m < 5; ++m) v[m] = hs[m][(r0 + i) * kLossTile + c];
#pragma unroll
            for (int q = 0; q < PER; ++q) {
                const int u = i - q;
                if (u < 0 || u > 10) continue;
                const float wt = win.w[u];
#pragma unroll
                for (int m = 0; m < 5; ++m) acc[m][q] += wt * v[m];
            }
        }
        float* dm = dmaps + (int64_t)ch * 3 * hw;
        const int x = x0 + c;
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int y = y0 + r0 + q;
            if (x >= W || y >= H) continue;
            const float mx = acc[0][q], my = acc[1][q], exx = acc[2][q], eyy = acc[3][q], exy = acc[4][q];
            const float A = 2.f * mx * my + kC1;
            const float B = 2.f * (exy - mx * my) + kC2;
            const float Cc = mx * mx + my * my + kC1;
            const float D = (exx - mx * mx) + (eyy - my * my) + kC2;
            const float icd = 1.0f / (Cc * D);
            const float sv = A * B * icd;
            const int64_t p = (int64_t)y * W + x;
            dm[p] = 2.f * my * (B - A) * icd - 2.f * mx * sv / Cc + 2.f * mx * sv / D;   // ds/dmx
            dm[hw + p] = -sv / D;                                                       // ds/dE[x^2]
            dm[2 * hw + p] = 2.f * A * icd;                                            // ds/dE[xy]
            ssum += sv;
        }
    }
    // Block sums, in a fixed order: the waves' in float, as a tree; over the waves
    // in double, rounded once.  One wave after the other in float would be further
    // off than a tree over the block (one view of 65 x 97: 3.2e-8 of the loss, rms,
    // against 2.1e-8).
    ssum = wave_sum_f(ssum);
    l1 = wave_sum_f(l1);
    if ((threadIdx.x & 63) == 0) {
        red[0][threadIdx.x >> 6] = ssum;
        red[1][threadIdx.x >> 6] = l1;
    }
    __syncthreads();
    if (threadIdx.x < 2) {
        const double* q = red[threadIdx.x];
        double t = 0.0;
#pragma unroll
        for (int w = 0; w < NT / 64; ++w) t += q[w];
        partial[2 * tile.index + threadIdx.x] = (float)t;
    }
}

template <int NT>
__global__ __launch_bounds__(NT) void k_ssim_bwd(const float* __restrict__ rgb, const float* __restrict__ target,
                                                  int W, int H, SsimWindow win, const float* __restrict__ dmaps,
                                                  float l1_scale, float ssim_scale, float* __restrict__ grad,
                                                  const uint32_t* __restrict__ skip) {
    if (skip && *skip) return;
    __shared__ __attribute__((aligned(16))) float hs[3][kRowsIn * kLossTile];
    const SsimTile tile = ssim_tile(W, H);
    if (!tile.valid) return;
    const int ch = tile.ch, x0 = tile.x0, y0 = tile.y0;
    const int64_t hw = (int64_t)W * H;
    const float* dm = dmaps + (int64_t)ch * 3 * hw;
    if (tile.inner)
        ssim_rows_bwd<NT, true>(dm, hw, W, H, x0, y0, win, hs);
    else
        ssim_rows_bwd<NT, false>(dm, hw, W, H, x0, y0, win, hs);
    const float* X = rgb + ch * hw;
    const float* Y = target + ch * hw;
    float* G = grad + ch * hw;
    // column pass: PER neighbouring rows of one column per thread, the
    // image's own pixels loaded before the barrier
    constexpr int PER = kLossTile * kLossTile / NT;
    const int c = threadIdx.x % kLossTile, r0 = (threadIdx.x / kLossTile) * PER;
    const int x = x0 + c;
    float px[PER], py[PER];
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const int y = y0 + r0 + q;
        const bool in = x < W && y < H;
        const int64_t p = (int64_t)y * W + x;
        px[q] = in ? X[p] : 0.0f;
        py[q] = in ? Y[p] : 0.0f;
    }
    __syncthreads();
    float acc[3][PER];
#pragma unroll
    for (int q = 0; q < PER; ++q)
#pragma unroll
        for (int m = 0; m < 3; ++m) acc[m][q] = 0.f;
#pragma unroll
    for (int i = 0; i < PER + 10; ++i) {
        float v[3];
#pragma unroll
        for (int m = 0; m < 3; ++m) v[m] = hs[m][(r0 + i) * kLossTile + c];
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int u = i - q;
            if (u < 0 || u > 10) continue;
            const float wt = win.w[u];
#pragma unroll
            for (int m = 0; m < 3; ++m) acc[m][q] += wt * v[m];
        }
    }
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const int y = y0 + r0 + q;
        if (x >= W || y >= H) continue;
        const float xv = px[q], yv = py[q];
        const float d = xv - yv;
        const float sg = d > 0.f ? 1.f : (d < 0.f ? -1.f : 0.f);
        G[(int64_t)y * W + x] = l1_scale * sg - ssim_scale * (acc[0][q] + 2.f * xv * acc[1][q] + yv * acc[2][q]);
    }
}

SsimWindow ssim_window() {
    SsimWindow S;
    double g[11], tot = 0.0;
    for (int t = 0; t < 11; ++t) {
        const double r = t - 5;
        g[t] = exp(-(r * r) / (2.0 * 1.5 * 1.5));
        tot += g[t];
    }
    for (int t = 0; t < 11; ++t) S.w[t] = (float)(g[t] / tot);
    return S;
}

// Up to two tiles per CU, a tile takes eight waves instead of four: the row
// pass is one round instead of two, and nothing else waits for the waves.  Four
// views, eight waves against four: 12 tiles a view (64 x 64) 40 us and 50, 216
// 42 and 52, 480 54 and 61, 576 and 720 63 and 68, 900 78 and 77, 1824 (1000 x
// 600) 128 and 123.  The line is where every CU has its two tiles at once.
constexpr int64_t kSsimFewTiles = 512;

// One view [3, H, W]: dmaps [3][3][H][W] scratch, partial [2 * 3 * tiles].
hipError_t launch_ssim_l1(const float* rgb, const float* target, int W, int H, float lam, float* dmaps,
                          float* partial, float* grad, const uint32_t* skip, hipStream_t s) {
    const SsimWindow win = ssim_window();
    const int64_t tiles = (int64_t)((W + kLossTile - 1) / kLossTile) * ((H + kLossTile - 1) / kLossTile) * 3;
    const dim3 grid((unsigned)((tiles + 7) & ~int64_t(7)));
    const float n = 3.0f * (float)W * (float)H;
#define LP_SSIM(NT_)                                                                                                \
    hipLaunchKernelGGL(k_ssim_fwd<NT_>, grid, dim3(NT_), 0, s, rgb, target, W, H, win, dmaps, partial, skip);        \
    hipLaunchKernelGGL(k_ssim_bwd<NT_>, grid, dim3(NT_), 0, s, rgb, target, W, H, win, dmaps, (1.0f - lam) / n,      \
                       lam / n, grad, skip)
    if (tiles <= kSsimFewTiles) {
        LP_SSIM(512);
    } else {
        LP_SSIM(256);
    }
#undef LP_SSIM
    return hipGetLastError();
}

}  // namespace linprim
