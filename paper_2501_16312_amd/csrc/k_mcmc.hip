// k_mcmc.hip -- LinPrim-MCMC's population steps (Sec. 3.4 "LinPrim-MCMC":
// GS-MCMC's relocation and noise applied to octahedra treated as Gaussians
// with standard deviations d / 2.6).
//
// Relocation, with caller-supplied 32-bit random numbers:
//   k_mc_count    per block of 1,024: sums of the integer weights
//                 w_i = floor(alpha_i 2^32) of live primitives (alpha > 0.005)
//                 and of the dead flags;
//   k_mc_scan     exclusive scan of both block sums (one block; only beyond
//                 kMcDirectBlocks blocks);
//   k_mc_prefix   inclusive weight prefix per primitive, list of the dead;
//                 each block adds the sums of the blocks before it itself;
//   k_mc_sample   the k-th dead primitive draws a source: the first index whose
//                 prefix exceeds floor(total r_k / 2^32) (binary search);
//                 per-source draw counts by integer atomics;
//   k_mc_sources  a source drawn c times becomes one of N = min(c + 1, 51)
//                 copies: opacity 1 - (1 - alpha)^(1/N), distances scaled to
//                 keep the composited opacity's line integral; moments reset;
//   k_mc_copy     dead primitive k <- its (updated) source; moments reset.
// Noise: k_mc_noise adds noise_lr lr s(1 - alpha) R S^2 R^T eps to the centre.
// All decisions on integers; the sampling is exact and reproducible.
#include "linprim_common.h"

namespace linprim {

constexpr float kMcDead = 0.005f;
constexpr int kMcItems = 1024;
constexpr int kMcMaxN = 51;
// Up to this many blocks of kMcItems primitives, each block of k_mc_prefix
// adds the sums of the blocks before it (8 KB of loads per block and sum at
// 1M primitives, from L2) instead of waiting for a one-block scan kernel.  The
// loads grow with the square: a relocation that draws nothing takes 19 us at 1M
// (22 with the scan kernel), 27 (33) at 2M, 46 (54) at 4M, 91 (94) at 8M.
constexpr int64_t kMcDirectBlocks = 8192;

__device__ inline uint64_t mc_weight(float a) {
    return a > kMcDead ? (uint64_t)floor((double)a * 4294967296.0) : 0ull;
}

__global__ __launch_bounds__(256) void k_mc_count(int64_t n, const float* __restrict__ opacity,
                                                  uint64_t* __restrict__ wsum, int64_t* __restrict__ dsum) {
    __shared__ uint64_t sw[256];
    __shared__ int64_t sd[256];
    const int t = threadIdx.x;
    uint64_t w = 0;
    int64_t d = 0;
#pragma unroll
    for (int k = 0; k < kMcItems / 256; ++k) {
        const int64_t i = (int64_t)blockIdx.x * kMcItems + (int64_t)t * (kMcItems / 256) + k;
        if (i < n) {
            const float a = opacity[i];
            w += mc_weight(a);
            d += a <= kMcDead ? 1 : 0;
        }
    }
    sw[t] = w;
    sd[t] = d;
    __syncthreads();
    for (int off = 128; off > 0; off >>= 1) {
        if (t < off) {
            sw[t] += sw[t + off];
            sd[t] += sd[t + off];
        }
        __syncthreads();
    }
    if (t == 0) {
        wsum[blockIdx.x] = sw[0];
        dsum[blockIdx.x] = sd[0];
    }
}

// Exclusive scans of nb block sums in place; entry nb receives the total.
__global__ __launch_bounds__(1024) void k_mc_scan(uint64_t* __restrict__ wsum, int64_t* __restrict__ dsum,
                                                  int64_t nb) {
    __shared__ uint64_t sw[1024];
    __shared__ int64_t sd[1024];
    __shared__ uint64_t cw;
    __shared__ int64_t cd;
    const int t = threadIdx.x;
    if (t == 0) {
        cw = 0;
        cd = 0;
    }
    __syncthreads();
    for (int64_t base = 0; base < nb; base += 1024) {
        const int64_t i = base + t;
        const uint64_t xw = i < nb ? wsum[i] : 0;
        const int64_t xd = i < nb ? dsum[i] : 0;
        sw[t] = xw;
        sd[t] = xd;
        __syncthreads();
        for (int off = 1; off < 1024; off <<= 1) {
            const uint64_t yw = t >= off ? sw[t - off] : 0;
            const int64_t yd = t >= off ? sd[t - off] : 0;
            __syncthreads();
            sw[t] += yw;
            sd[t] += yd;
            __syncthreads();
        }
        if (i < nb) {
            wsum[i] = cw + sw[t] - xw;
            dsum[i] = cd + sd[t] - xd;
        }
        __syncthreads();
        if (t == 1023) {
            cw += sw[1023];
            cd += sd[1023];
        }
        __syncthreads();
    }
    if (t == 0) {
        wsum[nb] = cw;
        dsum[nb] = cd;
    }
}

// Sum of a u64 over the 64 lanes of a wave (every lane gets it).
__device__ inline uint64_t mc_wave_sum(uint64_t x) {
    for (int off = 32; off >= 1; off >>= 1) x += __shfl_xor(x, off, 64);
    return x;
}

// `scanned`: wsum and dsum hold exclusive prefixes and their totals
// (k_mc_scan); otherwise the blocks' own sums, and the last block writes the
// totals after them.
__global__ __launch_bounds__(256) void k_mc_prefix(int64_t n, const float* __restrict__ opacity, bool scanned,
                                                   uint64_t* __restrict__ wsum, int64_t* __restrict__ dsum,
                                                   uint64_t* __restrict__ prefix, int32_t* __restrict__ dead_list,
                                                   int32_t* __restrict__ counts) {
    constexpr int PER = kMcItems / 256;
    __shared__ uint64_t part[4][4];   // weights and dead of the blocks before; of this block's waves
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int64_t b = blockIdx.x;
    const int64_t i0 = b * kMcItems + (int64_t)t * PER;
    uint64_t bw = 0, bd = 0;
    if (!scanned) {
        for (int64_t k = t; k < b; k += 256) {
            bw += wsum[k];
            bd += (uint64_t)dsum[k];
        }
        bw = mc_wave_sum(bw);
        bd = mc_wave_sum(bd);
    }
    uint64_t w[PER];
    bool dead[PER];
    uint64_t mw = 0;
    uint32_t md = 0;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int64_t i = i0 + k;
        const float a = i < n ? opacity[i] : 1.0f;
        w[k] = i < n ? mc_weight(a) : 0ull;
        dead[k] = i < n && a <= kMcDead;
        mw += w[k];
        md += dead[k] ? 1u : 0u;
    }
    uint64_t iw = mw;
    for (int off = 1; off < 64; off <<= 1) {
        const uint64_t y = __shfl_up(iw, off, 64);
        if (lane >= off) iw += y;
    }
    const uint32_t id = wave_incl_scan_u32(md);
    if (lane == 63) {
        part[0][wave] = bw;
        part[1][wave] = bd;
        part[2][wave] = iw;
        part[3][wave] = id;
    }
    __syncthreads();
    uint64_t run, rank;
    if (scanned) {
        run = wsum[b];
        rank = (uint64_t)dsum[b];
    } else {
        run = part[0][0] + part[0][1] + part[0][2] + part[0][3];
        rank = part[1][0] + part[1][1] + part[1][2] + part[1][3];
        if (b == (int64_t)gridDim.x - 1 && t == 0) {
            wsum[b + 1] = run + part[2][0] + part[2][1] + part[2][2] + part[2][3];
            dsum[b + 1] = (int64_t)(rank + part[3][0] + part[3][1] + part[3][2] + part[3][3]);
        }
    }
#pragma unroll
    for (int k = 0; k < 4; ++k)
        if (k < wave) {
            run += part[2][k];
            rank += part[3][k];
        }
    run += iw - mw;
    rank += id - md;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int64_t i = i0 + k;
        if (i >= n) break;
        run += w[k];
        prefix[i] = run;
        counts[i] = 0;
        if (dead[k]) dead_list[rank++] = (int32_t)i;
    }
}

// n_draws >= 0: that many draws (adding primitives); otherwise one per dead
// primitive (the device count).
__global__ __launch_bounds__(256) void k_mc_sample(int64_t n, const uint64_t* __restrict__ prefix,
                                                   const uint64_t* __restrict__ wtotal,
                                                   const int64_t* __restrict__ dtotal, int64_t n_draws,
                                                   const uint32_t* __restrict__ rnd, int32_t* __restrict__ samples,
                                                   int32_t* __restrict__ counts) {
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const uint64_t total = *wtotal;
    if (k >= (n_draws >= 0 ? n_draws : *dtotal) || total == 0) return;
    // floor(total r / 2^32), exactly
    const uint64_t r = rnd[k];
    const uint64_t t = (total >> 32) * r + (((total & 0xffffffffull) * r) >> 32);
    int64_t lo = 0, hi = n - 1;
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if (prefix[mid] > t) hi = mid; else lo = mid + 1;
    }
    samples[k] = (int32_t)lo;
    atomicAdd(counts + lo, 1);
}

// Rows of one field of W words, by the whole block: row to[r] receives the
// words of row from[r] (skipped if from is null) and its moments become zero.
// Consecutive threads take consecutive words, four at a time where the rows
// are whole 16-byte units and the arrays aligned.  to and from in LDS; no row
// is both written and read.
template <int W, int U>
__device__ inline void mc_rows_u(float* __restrict__ p, float* __restrict__ m, float* __restrict__ v,
                                 const int32_t* __restrict__ from, const int32_t* __restrict__ to, int R) {
    struct alignas(4 * U) Unit {
        float w[U];
    };
    constexpr int UPR = W / U;
    Unit* P = reinterpret_cast<Unit*>(p);
    Unit* M = reinterpret_cast<Unit*>(m);
    Unit* V = reinterpret_cast<Unit*>(v);
    Unit zero;
#pragma unroll
    for (int k = 0; k < U; ++k) zero.w[k] = 0.0f;
    for (int j = threadIdx.x; j < R * UPR; j += 256) {
        const int r = j / UPR, q = j - r * UPR;
        const int64_t d = (int64_t)to[r] * UPR + q;
        if (from) P[d] = P[(int64_t)from[r] * UPR + q];
        if (m) {
            M[d] = zero;
            V[d] = zero;
        }
    }
}

template <int W>
__device__ inline void mc_rows(const StateSet& S, int f, const int32_t* from, const int32_t* to, int R) {
    const uintptr_t a = reinterpret_cast<uintptr_t>(S.p[f]) | reinterpret_cast<uintptr_t>(S.m[f]) |
                        reinterpret_cast<uintptr_t>(S.v[f]);
    if (W % 4 == 0 && (a & 15) == 0)
        mc_rows_u<W, (W % 4 == 0 ? 4 : 1)>(S.p[f], S.m[f], S.v[f], from, to, R);
    else
        mc_rows_u<W, 1>(S.p[f], S.m[f], S.v[f], from, to, R);
}

template <int SHF>
__device__ inline void mc_all_rows(const StateSet& S, const int32_t* from, const int32_t* to, int R) {
    mc_rows<SHF>(S, 4, from, to, R);
    mc_rows<4>(S, 1, from, to, R);
    mc_rows<3>(S, 0, from, to, R);
    mc_rows<3>(S, 2, from, to, R);
    mc_rows<1>(S, 3, from, to, R);
}

// One block per kMcItems primitives: the drawn ones are listed in LDS, so
// that a few full waves run the update of the few that were drawn, and all
// threads then clear their moments along the rows' words.  (A thread per
// primitive, clearing 118 words by itself: 40 us for 50k sources of 1M, bound
// by the stores of single lanes; now 16 us.)
template <int SHF>
__global__ __launch_bounds__(256) void k_mc_sources(int64_t n, StateSet S, const int32_t* __restrict__ counts) {
    __shared__ int32_t list[kMcItems];
    __shared__ int32_t drawn[kMcItems];
    __shared__ int32_t total;
    if (threadIdx.x == 0) total = 0;
    __syncthreads();
    for (int k = 0; k < kMcItems / 256; ++k) {
        const int64_t i = (int64_t)blockIdx.x * kMcItems + k * 256 + threadIdx.x;
        const int32_t c = i < n ? counts[i] : 0;
        if (c) {
            const int32_t at = atomicAdd(&total, 1);   // any order: rows are independent
            list[at] = (int32_t)i;
            drawn[at] = c;
        }
    }
    __syncthreads();
    const int R = total;
    for (int r = threadIdx.x; r < R; r += 256) {
        const int64_t i = list[r];
        const int N = min(drawn[r] + 1, kMcMaxN);
        const double a = (double)S.p[3][i];
        double an = 1.0 - pow(1.0 - a, 1.0 / (double)N);
        an = fmin(fmax(an, (double)kMcDead), 1.0 - 1.1920928955078125e-7);
        // sum_{j=1}^{N} sum_{k=0}^{j-1} C(j-1, k) (-1)^k an^(k+1) / sqrt(k+1), as
        // it stands: summed over j first it is the N terms C(N, k+1) (-1)^k
        // an^(k+1) / sqrt(k+1), which cancel worse (alpha = 1, N = 12: 2e-14 of
        // the sum against 7e-16; N = 32: 1.8e-8 against 8e-9; N = 51: 6e-3
        // against 1e-3; other alpha, N = 28: 4e-14 rms against 1e-14)
        double denom = 0.0;
        for (int j = 1; j <= N; ++j) {
            double c = 1.0;                       // C(j-1, k)
            double p = an;                        // an^(k+1)
            for (int k = 0; k < j; ++k) {
                denom += ((k & 1) ? -c : c) * p / sqrt((double)(k + 1));
                c = c * (double)(j - 1 - k) / (double)(k + 1);
                p *= an;
            }
        }
        const double coeff = a / denom;
#pragma unroll
        for (int k = 0; k < 3; ++k) S.p[2][i * 3 + k] = (float)((double)S.p[2][i * 3 + k] * coeff);
        S.p[3][i] = (float)an;
    }
    if (S.m[0]) mc_all_rows<SHF>(S, nullptr, list, R);
}

// Draw k's target: the k-th dead primitive, or row append_base + k when
// adding (n_draws >= 0).  A block copies kMcCopyRows rows at a time, all
// threads along the rows' words (54 us for 50k rows of degree 3 with moments
// when each thread copied a whole row; now 18 us).
constexpr int kMcCopyRows = 64;
template <int SHF>
__global__ __launch_bounds__(256) void k_mc_copy(StateSet S, const int64_t* __restrict__ dtotal, int64_t n_draws,
                                                 int64_t append_base, const uint64_t* __restrict__ wtotal,
                                                 const int32_t* __restrict__ dead_list,
                                                 const int32_t* __restrict__ samples) {
    __shared__ int32_t from[kMcCopyRows], to[kMcCopyRows];
    const int64_t total = n_draws >= 0 ? n_draws : *dtotal;
    if (*wtotal == 0) return;
    for (int64_t k0 = (int64_t)blockIdx.x * kMcCopyRows; k0 < total; k0 += (int64_t)gridDim.x * kMcCopyRows) {
        const int R = (int)min((int64_t)kMcCopyRows, total - k0);
        if ((int)threadIdx.x < R) {
            const int64_t k = k0 + threadIdx.x;
            from[threadIdx.x] = samples[k];
            to[threadIdx.x] = n_draws >= 0 ? (int32_t)(append_base + k) : dead_list[k];
        }
        __syncthreads();
        mc_all_rows<SHF>(S, from, to, R);
        __syncthreads();
    }
}

__global__ __launch_bounds__(256) void k_mc_noise(int64_t n, float* __restrict__ means,
                                                  const float* __restrict__ quats, const float* __restrict__ dists,
                                                  const float* __restrict__ opacity, const float* __restrict__ eps,
                                                  double scale) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const double a = (double)opacity[i];
    const double gate = 1.0 / (1.0 + exp(-100.0 * ((1.0 - a) - 0.995)));
    double R[9];
    if (!quat_rotation_d((double)quats[4 * i], (double)quats[4 * i + 1], (double)quats[4 * i + 2],
                         (double)quats[4 * i + 3], R))
        return;
    double l[3];
    // R S^2 R^T e: into the primitive's frame, scale by (d / 2.6)^2, back
    for (int c = 0; c < 3; ++c) {
        const double e = R[c] * eps[3 * i] + R[3 + c] * eps[3 * i + 1] + R[6 + c] * eps[3 * i + 2];
        const double s = (double)dists[3 * i + c] / 2.6;
        l[c] = s * s * e;
    }
    for (int r = 0; r < 3; ++r)
        means[3 * i + r] = (float)((double)means[3 * i + r] + scale * gate * (R[3 * r] * l[0] + R[3 * r + 1] * l[1] +
                                                                             R[3 * r + 2] * l[2]));
}

// Workspace: prefix [n] u64 | wsum [nb+1] u64 | dsum [nb+1] i64 | dead [n] i32 | samples [n] i32 | counts [n] i32
// (draws when adding are at most n: the workspace of n serves both steps).
struct McLayout {
    size_t prefix, wsum, dsum, dead, samples, counts, total;
};

McLayout mc_layout(int64_t n) {
    const int64_t nb = (n + kMcItems - 1) / kMcItems;
    McLayout L;
    size_t off = 0;
    L.prefix = off; off = align256(off + (size_t)n * 8);
    L.wsum = off; off = align256(off + (size_t)(nb + 1) * 8);
    L.dsum = off; off = align256(off + (size_t)(nb + 1) * 8);
    L.dead = off; off = align256(off + (size_t)n * 4);
    L.samples = off; off = align256(off + (size_t)n * 4);
    L.counts = off; off = align256(off + (size_t)n * 4);
    L.total = off;
    return L;
}

size_t mc_workspace_bytes(int64_t n) { return mc_layout(n).total; }

// n_add < 0: relocate the dead in place; n_add >= 0: draw n_add sources
// among the first n rows and write their copies to rows n .. n + n_add - 1.
hipError_t launch_mc_relocate(int64_t n, int64_t n_add, int sh_degree, const StateSet& S, const uint32_t* rnd,
                              char* ws, hipStream_t s) {
    if (n == 0 || n_add == 0) return hipSuccess;
    const McLayout L = mc_layout(n);
    const int64_t nb = (n + kMcItems - 1) / kMcItems;
    uint64_t* prefix = (uint64_t*)(ws + L.prefix);
    uint64_t* wsum = (uint64_t*)(ws + L.wsum);
    int64_t* dsum = (int64_t*)(ws + L.dsum);
    int32_t* dead = (int32_t*)(ws + L.dead);
    int32_t* samples = (int32_t*)(ws + L.samples);
    int32_t* counts = (int32_t*)(ws + L.counts);
    hipLaunchKernelGGL(k_mc_count, dim3((unsigned)nb), dim3(256), 0, s, n, S.p[3], wsum, dsum);
    const bool scanned = nb > kMcDirectBlocks;
    if (scanned) hipLaunchKernelGGL(k_mc_scan, dim3(1), dim3(1024), 0, s, wsum, dsum, nb);
    hipLaunchKernelGGL(k_mc_prefix, dim3((unsigned)nb), dim3(256), 0, s, n, S.p[3], scanned, wsum, dsum, prefix, dead,
                       counts);
    const int64_t draws_max = n_add >= 0 ? n_add : n;
    hipLaunchKernelGGL(k_mc_sample, dim3((unsigned)((draws_max + 255) / 256)), dim3(256), 0, s, n, prefix, wsum + nb,
                       dsum + nb, n_add, rnd, samples, counts);
    // the blocks stride over the rows: of a relocation only the device knows how many
    const int64_t cb = (draws_max + kMcCopyRows - 1) / kMcCopyRows;
    const unsigned copy_blocks = (unsigned)(cb < 2048 ? cb : 2048);
#define LP_MC(SHF_)                                                                                             \
    hipLaunchKernelGGL(k_mc_sources<SHF_>, dim3((unsigned)nb), dim3(256), 0, s, n, S, counts);                  \
    hipLaunchKernelGGL(k_mc_copy<SHF_>, dim3(copy_blocks), dim3(256), 0, s, S, dsum + nb, n_add, n, wsum + nb,  \
                       dead, samples)
    switch (sh_degree) {
        case 0: LP_MC(3); break;
        case 1: LP_MC(12); break;
        case 2: LP_MC(27); break;
        default: LP_MC(48); break;
    }
#undef LP_MC
    return hipGetLastError();
}

hipError_t launch_mc_noise(int64_t n, float* means, const float* quats, const float* dists, const float* opacity,
                           const float* eps, double scale, hipStream_t s) {
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_mc_noise, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, n, means, quats, dists, opacity,
                       eps, scale);
    return hipGetLastError();
}

int64_t mc_dead_offset(int64_t n) {
    const McLayout L = mc_layout(n);
    return (int64_t)(L.dsum + ((n + kMcItems - 1) / kMcItems) * 8);
}

}  // namespace linprim
