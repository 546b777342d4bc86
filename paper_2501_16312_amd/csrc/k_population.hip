// k_population.hip -- adaptive population control (Sec. 3.4 "Adaptive
// Population Control"; thresholds in App. G): statistics accumulated over
// the views of each step, then one densify / prune pass that compacts the
// primitives and their Adam moments into new arrays.
//
//   k_accum_stats   per primitive: add, over the views in which it touches a
//                   tile, the norm of its view-space positional gradient
//                   (left per slot by the preprocessing backward), count the
//                   views, keep the largest screen radius.
//   k_dens_count    per primitive: how many rows it leaves (0..3); block sums.
//   k_dens_scan     exclusive scan of the block sums (one block).
//   k_dens_apply    per primitive: its rows' offset (block scan) and the rows:
//                   the original or its two split children, then its clone.
#include <mutex>

#include "linprim_common.h"

namespace linprim {

__global__ __launch_bounds__(256) void k_accum_stats(int64_t n, int n_views, const uint32_t* __restrict__ tiles,
                                                     const float2* __restrict__ stats, float* __restrict__ grad_accum,
                                                     int32_t* __restrict__ count, float* __restrict__ max_radius) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    float acc = 0.0f, mr = max_radius[i];
    int cnt = 0;
    for (int v = 0; v < n_views; ++v) {
        const int64_t vs = (int64_t)v * n + i;
        if (tiles[vs] == 0) continue;
        const float2 s = stats[vs];
        acc += s.x;
        mr = fmaxf(mr, s.y);
        ++cnt;
    }
    grad_accum[i] += acc;
    count[i] += cnt;
    max_radius[i] = mr;
}

hipError_t launch_accumulate_stats(int64_t n, int32_t n_views, const ViewLayout& L, const char* vws,
                                   float* grad_accum, int32_t* count, float* max_radius, hipStream_t s) {
    if (n == 0) return hipSuccess;
    const uint32_t* tiles = reinterpret_cast<const uint32_t*>(vws + L.tiles);
    const float2* stats = reinterpret_cast<const float2*>(vws + L.stats);
    hipLaunchKernelGGL(k_accum_stats, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, n, (int)n_views, tiles,
                       stats, grad_accum, count, max_radius);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Decisions, in float32 (the precision of every input): size = longest axis
// 2 max d (octahedron) or sqrt(2) times the distance to the furthest corner
// (tetrahedron); a mean gradient above the threshold makes a candidate, a
// small candidate is cloned, a larger one split in two; transparent, too
// large or (originals only) too wide primitives are removed.
// ---------------------------------------------------------------------------
struct Decision {
    bool keep, split, clone;
    __device__ int rows() const { return (keep ? 1 : 0) + (split ? 2 : 0) + (clone ? 1 : 0); }
};

template <int ND>
__device__ inline Decision decide(int type, const float* __restrict__ d, float opacity, float acc, int cnt,
                                  float mr, const DensifyParams& dp, float extent) {
    float dm = d[0];
#pragma unroll
    for (int k = 1; k < ND; ++k) dm = fmaxf(dm, d[k]);
    const float size = (type == LINPRIM_OCTAHEDRON) ? 2.0f * dm : (float)1.41421356237309504880 * dm;
    const float avg = cnt > 0 ? acc / (float)cnt : 0.0f;
    const float max_size = dp.max_size_frac * extent;
    const bool cand = avg > dp.grad_threshold;
    const bool small = size < dp.clone_size_frac * extent;
    const bool transparent = opacity < dp.min_opacity;
    Decision D;
    const bool split = cand && !small;
    D.keep = !split && !transparent && !(size > max_size) && !(mr > dp.max_radius);
    D.split = split && !transparent && !(size / dp.shrink > max_size);
    D.clone = cand && small && !transparent && !(size > max_size);
    return D;
}

template <int ND>
__global__ __launch_bounds__(256) void k_dens_count(int type, int64_t n, const float* __restrict__ dists,
                                                    const float* __restrict__ opacity,
                                                    const float* __restrict__ grad_accum,
                                                    const int32_t* __restrict__ count,
                                                    const float* __restrict__ max_radius, DensifyParams dp,
                                                    float extent, int64_t* __restrict__ block_sums) {
    __shared__ int64_t part[256];
    const int t = threadIdx.x;
    int64_t sum = 0;
#pragma unroll
    for (int k = 0; k < kDensifyItems / 256; ++k) {
        const int64_t i = (int64_t)blockIdx.x * kDensifyItems + k * 256 + t;
        if (i < n) sum += decide<ND>(type, dists + ND * i, opacity[i], grad_accum[i], count[i], max_radius[i], dp,
                                     extent).rows();
    }
    part[t] = sum;
    __syncthreads();
    for (int off = 128; off > 0; off >>= 1) {
        if (t < off) part[t] += part[t + off];
        __syncthreads();
    }
    if (t == 0) block_sums[blockIdx.x] = part[0];
}

// Exclusive scan of nb block sums in place; block_sums[nb] = total.
__global__ __launch_bounds__(1024) void k_dens_scan(int64_t* __restrict__ block_sums, int64_t nb) {
    __shared__ int64_t s[1024];
    __shared__ int64_t carry;
    const int t = threadIdx.x;
    if (t == 0) carry = 0;
    __syncthreads();
    for (int64_t base = 0; base < nb; base += 1024) {
        const int64_t i = base + t;
        const int64_t x = i < nb ? block_sums[i] : 0;
        s[t] = x;
        __syncthreads();
        for (int off = 1; off < 1024; off <<= 1) {
            const int64_t y = t >= off ? s[t - off] : 0;
            __syncthreads();
            s[t] += y;
            __syncthreads();
        }
        if (i < nb) block_sums[i] = carry + s[t] - x;
        __syncthreads();
        if (t == 1023) carry += s[1023];
        __syncthreads();
    }
    if (t == 0) block_sums[nb] = carry;
}

// Output rows of a block, in order: the local index of the source primitive
// and what the row is to it, one word each in LDS.
enum : uint32_t { kRowKeep = 0, kRowChild0 = 1, kRowChild1 = 2, kRowClone = 3 };
constexpr int kRowShift = 10;
static_assert(kDensifyItems <= (1 << kRowShift), "local index in the low bits of a row word");

// Rows [0, R) of one field of W words: dst row r (from `dst`, the block's
// first output row) is a copy of the row's source (from `src`, the block's
// first input row), or zero unless the row is a kept primitive (`moments`:
// new primitives start with zero moments; src may be null, then all zero).
// Consecutive threads write consecutive words, four at a time where the rows
// are whole 16-byte units and both arrays are aligned; four loads in flight.
template <int W, int U>
__device__ inline void copy_rows_u(const float* __restrict__ src, float* __restrict__ dst,
                                   const uint16_t* __restrict__ rows, int R, bool moments) {
    struct alignas(4 * U) Unit {
        float w[U];
    };
    constexpr int UPR = W / U;
    const Unit* sp = reinterpret_cast<const Unit*>(src);
    Unit* dp = reinterpret_cast<Unit*>(dst);
    const int total = R * UPR;
    for (int j0 = threadIdx.x; j0 < total; j0 += 4 * 256) {
        Unit x[4];
#pragma unroll
        for (int h = 0; h < 4; ++h) {
            const int j = j0 + 256 * h;
#pragma unroll
            for (int k = 0; k < U; ++k) x[h].w[k] = 0.0f;
            if (j < total) {
                const int r = j / UPR, q = j - r * UPR;
                const uint32_t e = rows[r];
                const bool read = !moments || (sp && (e >> kRowShift) == kRowKeep);
                if (read) x[h] = sp[(e & ((1u << kRowShift) - 1)) * UPR + q];
            }
        }
#pragma unroll
        for (int h = 0; h < 4; ++h) {
            const int j = j0 + 256 * h;
            if (j < total) dp[j] = x[h];
        }
    }
}

template <int W>
__device__ inline void copy_rows(const float* src, float* dst, const uint16_t* rows, int R, bool moments) {
    if (W % 4 == 0 && ((reinterpret_cast<uintptr_t>(src) | reinterpret_cast<uintptr_t>(dst)) & 15) == 0)
        copy_rows_u<W, (W % 4 == 0 ? 4 : 1)>(src, dst, rows, R, moments);
    else
        copy_rows_u<W, 1>(src, dst, rows, R, moments);
}

// One block per kDensifyItems primitives and array set (blockIdx.y: the
// parameters, the first moments, the second moments).  The block takes its
// primitives' decisions, lists its output rows in LDS and then copies field
// by field, all threads along the rows' words.  Bound by HBM: 1M octahedra of
// degree 3 with moments (1.43 GB read and written) take 0.32 ms, 4.4 TB/s;
// they took 3.66 ms when each thread copied its own primitives' rows, 192
// bytes between lanes.  One set of arrays per block gives three times the
// blocks (977 alone would leave the last round of the chip nearly empty).
template <int ND, int SHF>
__global__ __launch_bounds__(256) void k_dens_apply(int type, int64_t n, StateSet src, StateSet dst,
                                                    const float* __restrict__ normals,
                                                    const float* __restrict__ grad_accum,
                                                    const int32_t* __restrict__ count,
                                                    const float* __restrict__ max_radius, DensifyParams dp,
                                                    float extent, const int64_t* __restrict__ block_sums) {
    constexpr int PER = kDensifyItems / 256;
    __shared__ uint16_t rows[3 * kDensifyItems];
    __shared__ uint32_t wsum[4];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int64_t b0 = (int64_t)blockIdx.x * kDensifyItems;
    // this thread's items are consecutive, so that the block's rows stay in order
    Decision D[PER];
    uint32_t mine = 0;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int64_t i = b0 + t * PER + k;
        D[k] = (i < n) ? decide<ND>(type, src.p[2] + ND * i, src.p[3][i], grad_accum[i], count[i], max_radius[i], dp,
                                    extent)
                       : Decision{false, false, false};
        mine += (uint32_t)D[k].rows();
    }
    const uint32_t incl = wave_incl_scan_u32(mine);
    if (lane == 63) wsum[wave] = incl;
    __syncthreads();
    uint32_t o = incl - mine, R = 0;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        o += (w < wave) ? wsum[w] : 0u;
        R += wsum[w];
    }
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const uint32_t e = (uint32_t)(t * PER + k);
        if (D[k].keep) rows[o++] = (uint16_t)(e | (kRowKeep << kRowShift));
        if (D[k].split) {
            rows[o++] = (uint16_t)(e | (kRowChild0 << kRowShift));
            rows[o++] = (uint16_t)(e | (kRowChild1 << kRowShift));
        }
        if (D[k].clone) rows[o++] = (uint16_t)(e | (kRowClone << kRowShift));
    }
    __syncthreads();
    const int64_t o0 = block_sums[blockIdx.x];
    const int nr = (int)R;
    if (blockIdx.y != 0) {
        // moments: fields without a destination are skipped, without a source zero
        float* const* d = (blockIdx.y == 1) ? dst.m : dst.v;
        float* const* s = (blockIdx.y == 1) ? src.m : src.v;
        auto from = [&](int f, int w) { return src.m[f] ? s[f] + b0 * w : nullptr; };
        if (dst.m[0]) copy_rows<3>(from(0, 3), d[0] + o0 * 3, rows, nr, true);
        if (dst.m[1]) copy_rows<4>(from(1, 4), d[1] + o0 * 4, rows, nr, true);
        if (dst.m[2]) copy_rows<ND>(from(2, ND), d[2] + o0 * ND, rows, nr, true);
        if (dst.m[3]) copy_rows<1>(from(3, 1), d[3] + o0, rows, nr, true);
        if (dst.m[4]) copy_rows<SHF>(from(4, SHF), d[4] + o0 * SHF, rows, nr, true);
        return;
    }
    copy_rows<SHF>(src.p[4] + b0 * SHF, dst.p[4] + o0 * SHF, rows, nr, false);
    copy_rows<4>(src.p[1] + b0 * 4, dst.p[1] + o0 * 4, rows, nr, false);
    copy_rows<1>(src.p[3] + b0, dst.p[3] + o0, rows, nr, false);
    // centres and distances, a thread per row
    for (int r = t; r < nr; r += 256) {
        const uint32_t e = rows[r], what = e >> kRowShift;
        const int64_t i = b0 + (e & ((1u << kRowShift) - 1));
        const float* mus = src.p[0] + i * 3;
        const float* d = src.p[2] + ND * i;
        float* mu = dst.p[0] + (o0 + r) * 3;
        float* dd = dst.p[2] + (o0 + r) * ND;
        if (what != kRowChild0 && what != kRowChild1) {
            for (int c = 0; c < 3; ++c) mu[c] = mus[c];
            for (int c = 0; c < ND; ++c) dd[c] = d[c];
            continue;
        }
        // children: distances / shrink; positions mu + R (d * z) along the
        // octahedron's own axes, or mu + (max d / 2) z for a tetrahedron
        const float* z = normals + (i * 2 + (what == kRowChild1 ? 1 : 0)) * 3;
        double off[3];
        if (type == LINPRIM_OCTAHEDRON) {
            const float* q = src.p[1] + 4 * i;
            double Rm[9];
            const bool rot = quat_rotation_d((double)q[0], (double)q[1], (double)q[2], (double)q[3], Rm);
            const double l[3] = {(double)d[0] * z[0], (double)d[1] * z[1], (double)d[2] * z[2]};
            for (int c = 0; c < 3; ++c)
                off[c] = rot ? Rm[3 * c] * l[0] + Rm[3 * c + 1] * l[1] + Rm[3 * c + 2] * l[2] : l[c];
        } else {
            float dm = d[0];
#pragma unroll
            for (int c = 1; c < ND; ++c) dm = fmaxf(dm, d[c]);
            for (int c = 0; c < 3; ++c) off[c] = 0.5 * (double)dm * (double)z[c];
        }
        for (int c = 0; c < 3; ++c) mu[c] = (float)((double)mus[c] + off[c]);
        for (int c = 0; c < ND; ++c) dd[c] = (float)((double)d[c] / (double)dp.shrink);
    }
}

hipError_t launch_densify_plan(int type, int64_t n, const float* dists, const float* opacity,
                               const float* grad_accum, const int32_t* count, const float* max_radius,
                               const DensifyParams& dp, float extent, int64_t* block_sums, hipStream_t s) {
    const int64_t nb = (n + kDensifyItems - 1) / kDensifyItems;
    if (nb > 0) {
        if (type == LINPRIM_OCTAHEDRON)
            hipLaunchKernelGGL(k_dens_count<3>, dim3((unsigned)nb), dim3(256), 0, s, type, n, dists, opacity,
                               grad_accum, count, max_radius, dp, extent, block_sums);
        else
            hipLaunchKernelGGL(k_dens_count<4>, dim3((unsigned)nb), dim3(256), 0, s, type, n, dists, opacity,
                               grad_accum, count, max_radius, dp, extent, block_sums);
    }
    hipLaunchKernelGGL(k_dens_scan, dim3(1), dim3(1024), 0, s, block_sums, nb);
    return hipGetLastError();
}

hipError_t launch_densify_apply(int type, int sh_degree, int64_t n, const StateSet& src, const float* normals,
                                const float* grad_accum, const int32_t* count, const float* max_radius,
                                const DensifyParams& dp, float extent, const int64_t* block_sums,
                                const StateSet& dst, hipStream_t s) {
    const int64_t nb = (n + kDensifyItems - 1) / kDensifyItems;
    if (nb == 0) return hipSuccess;
    bool moments = false;
    for (int f = 0; f < 5; ++f) moments = moments || dst.m[f];
    const dim3 grid((unsigned)nb, moments ? 3 : 1);
#define LP_DENS(ND_, SHF_)                                                                                        \
    hipLaunchKernelGGL((k_dens_apply<ND_, SHF_>), grid, dim3(256), 0, s, type, n, src, dst, normals, grad_accum, \
                       count, max_radius, dp, extent, block_sums)
#define LP_DENS_DEG(ND_)                  \
    switch (sh_degree) {                  \
        case 0: LP_DENS(ND_, 3); break;   \
        case 1: LP_DENS(ND_, 12); break;  \
        case 2: LP_DENS(ND_, 27); break;  \
        default: LP_DENS(ND_, 48); break; \
    }
    if (type == LINPRIM_OCTAHEDRON) {
        LP_DENS_DEG(3)
    } else {
        LP_DENS_DEG(4)
    }
#undef LP_DENS_DEG
#undef LP_DENS
    return hipGetLastError();
}

// Scratch of the allocation-free densify entry point: the plan's block sums
// and total, (n / kDensifyItems + 1) values, held by each device the
// library runs on until the process ends.  Host code reaches it only through
// the address hipGetSymbolAddress returns for the current device.
constexpr int64_t kDensifyScratchItems = kNoAllocMaxPrims / kDensifyItems + 8;
static __device__ __align__(256) int64_t scratch[kDensifyScratchItems];

namespace {
constexpr int kScratchDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kScratchDevices];
}  // namespace

hipError_t densify_scratch(int64_t** out) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kScratchDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        g_scratch_ptr[dev] = p;
    }
    *out = static_cast<int64_t*>(g_scratch_ptr[dev]);
    return hipSuccess;
}

}  // namespace linprim
