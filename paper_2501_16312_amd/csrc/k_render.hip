// k_render.hip -- per-pixel compositing (Sec. 3.2 "Rasterization",
// "Compositing") and its backward pass (Sec. 3.4, App. E).
//
// Work decomposition (gfx950, wave64):
//   * one 64-lane wavefront per 8 x 8 pixel group; a TILE x TILE screen tile
//     has (TILE/8)^2 groups, each an independent workgroup; a lane owns one
//     pixel of its group;
//   * forward: the list is taken 32 entries at a time with their records
//     staged in LDS, and each 16-lane row of the wave walks the entries whose
//     rectangle meets its 4 x 4 quad of the group (exact rays: the whole wave
//     together where that takes hardly more steps);
//   * backward: batches of 64 entries, one vector load brings 64 primitive
//     indices and their pixel rectangles, a ballot keeps the entries whose
//     rectangle meets the group, and only those entries' 32-dword payloads are
//     read, wave-uniform, through scalar loads issued one entry ahead (no LDS,
//     no barriers), so that an entry's gradients are summed by the whole wave;
//   * a pixel is evaluated only inside the primitive's pixel rectangle, so
//     images do not depend on the tile size.
//
// Chord.  Pixel rays are parallel to the ray-space z axis, so the ray's
// chord through a convex primitive is max(0, min_up - max_lo): the lowest
// of the planes bounding the primitive from above minus the highest of the
// planes bounding it from below, evaluated at the pixel.  This equals the
// paper's exit-minus-entry Moeller-Trumbore depth difference (the entry and
// exit hits lie on the active lower and upper faces).  Octahedra keep their 8
// faces as 4 slabs (opposite faces are parallel), tetrahedra their 4 faces
// split into upper and lower sets.  Planes are stored relative to the
// centre of the primitive's pixel rectangle, so ki, kj are small exact
// half-integers.
#include "linprim_common.h"

namespace linprim {

// ---------------------------------------------------------------------------
// Wave helpers.
// ---------------------------------------------------------------------------
template <int CTRL, int ROW_MASK = 0xF>
__device__ inline float dpp_move(float src) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(src), CTRL, ROW_MASK, 0xF, false));
}

// Sum over the 64 lanes; every lane must be active.  Returns the total (uniform).
__device__ inline float wave_sum(float v) {
    v += dpp_move<0xB1>(v);          // quad_perm(1,0,3,2)
    v += dpp_move<0x4E>(v);          // quad_perm(2,3,0,1)
    v += dpp_move<0x141>(v);         // row_half_mirror
    v += dpp_move<0x140>(v);         // row_mirror: every lane holds its row sum
    v += dpp_move<0x142, 0xA>(v);    // row_bcast:15 -> rows 1 and 3
    v += dpp_move<0x143, 0x8>(v);    // row_bcast:31 -> row 3 holds the total
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}

// s_waitcnt lgkmcnt(0) (vmcnt and expcnt left at their maxima), fenced so
// that the scheduler moves no scalar load above it.
__device__ inline void smem_wait_all() {
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(0xC07F);
    __builtin_amdgcn_sched_barrier(0);
}
__device__ inline void sched_fence() { __builtin_amdgcn_sched_barrier(0); }

// Between some lanes' LDS accesses and others' of the same wave.  LDS answers a
// wave in order, so nothing has to be waited for, but the compiler knows of no
// dependence between lanes, and accesses of different types it may reorder.
__device__ inline void lds_hand_over() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

__device__ inline int wave_max_int(int v) {
    for (int off = 32; off >= 1; off >>= 1) v = max(v, __shfl_xor(v, off, 64));
    return v;
}

// Round-robin dispatch puts consecutive workgroups on different XCDs.  Deal
// out chunks of kXcdChunk consecutive waves (neighbouring tiles, which share
// primitives) round-robin instead, so each XCD's L2 sees whole chunks while
// every XCD still gets a spread of the image (tiles differ a lot in work).
constexpr int64_t kXcdChunk = 32;
__device__ inline int64_t xcd_tile(int64_t b, int64_t nb) {
    constexpr int64_t X = 8;
    const int64_t full = (nb / (X * kXcdChunk)) * (X * kXcdChunk);
    if (b >= full) return b;
    const int64_t x = b % X, k = b / X;
    return ((k / kXcdChunk) * X + x) * kXcdChunk + (k % kXcdChunk);
}

__device__ inline int find_view(const ViewInfo* __restrict__ views, int n_views, int64_t g) {
    int lo = 0, hi = n_views - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (views[mid].tile_base <= g) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// ---------------------------------------------------------------------------
// Chords.  Contraction is disabled inside so the forward and the backward
// kernels evaluate bit-identical chords; fused multiply-adds are explicit.
// ---------------------------------------------------------------------------
struct Rec {
    float s2, r, g, b, fi0, fj0, fwi, fwj;
    float p[18];
    float sigma;
    int fmap;
};

template <int KIND>
__device__ inline void load_rec(const float* __restrict__ rec, Rec& R) {
    R.s2 = rec[R_S2];
    R.r = rec[R_RGB];
    R.g = rec[R_RGB + 1];
    R.b = rec[R_RGB + 2];
    R.fi0 = rec[R_FI0];
    R.fj0 = rec[R_FJ0];
    R.fwi = rec[R_FWI];
    R.fwj = rec[R_FWJ];
    constexpr int NP = (KIND == LINPRIM_OCTAHEDRON) ? 16 : 18;
#pragma unroll
    for (int k = 0; k < NP; ++k) R.p[k] = rec[R_PLANES + k];
    R.sigma = rec[R_SIGMA];
    R.fmap = (KIND == LINPRIM_OCTAHEDRON) ? 0 : __float_as_int(rec[R_FACEMAP]);
}

// An entry's record words 4.. as a 16-lane row holds them: lane l has words
// 2 l and 2 l + 1, and an instruction takes one as its DPP operand
// (row_newbcast), so a record costs two registers and one LDS read.
template <int KIND, bool EXACT>
constexpr int rec_quads() {
    return (EXACT || KIND == LINPRIM_OCTAHEDRON) ? 6 : 7;
}
template <int W>
__device__ inline float row_word(float2 r) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int((W & 1) ? r.y : r.x), 0x150 + (W >> 1), 0xF, 0xF, true));
}
// Returns hi - lo; ih / il are the active upper / lower slot (first on ties).
template <int KIND>
__device__ inline float chord(const Rec& R, float ki, float kj, int& ih, int& il) {
#pragma clang fp contract(off)
    if (KIND == LINPRIM_OCTAHEDRON) {
        float hi = 0.f, lo = 0.f;
        ih = 0; il = 0;
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const float u = __builtin_fmaf(R.p[4 * s + 0], ki, R.p[4 * s + 1] * kj);
            const float h = u + R.p[4 * s + 2];
            const float l = u + R.p[4 * s + 3];
            if (s == 0) { hi = h; lo = l; }
            else {
                if (h < hi) { hi = h; ih = s; }
                if (l > lo) { lo = l; il = s; }
            }
        }
        return hi - lo;
    } else {
        float hi = 0.f, lo = 0.f;
        ih = 0; il = 0;
#pragma unroll
        for (int s = 0; s < 3; ++s) {
            const float h = __builtin_fmaf(R.p[3 * s + 0], ki, __builtin_fmaf(R.p[3 * s + 1], kj, R.p[3 * s + 2]));
            const float l = __builtin_fmaf(R.p[9 + 3 * s + 0], ki, __builtin_fmaf(R.p[9 + 3 * s + 1], kj, R.p[9 + 3 * s + 2]));
            if (s == 0) { hi = h; lo = l; }
            else {
                if (h < hi) { hi = h; ih = s; }
                if (l > lo) { lo = l; il = s; }
            }
        }
        return hi - lo;
    }
}

// Same chord without slot tracking (forward), from a record spread over the
// row; lo is the entry depth relative to the centre's ray-space depth.  Each
// word is taken where it is used: the compiler folds a broadcast into the
// instruction that reads it only a few instructions away.
// Broadcasts into multiply-adds are written out (the compiler leaves a move
// for each), several to a block: a register is read through DPP two wait
// states after a vector instruction wrote it.
#define LP_FMAC_ROW(acc, word, lane, x) "v_fmac_f32_dpp " acc ", " word ", " x " row_newbcast:" lane " row_mask:0xf bank_mask:0xf\n\t"
template <int KIND>
__device__ inline float chord_row(float2 r, float ki, float kj, float& lo) {
#pragma clang fp contract(off)
    if (KIND == LINPRIM_OCTAHEDRON) {
        float u0 = row_word<9>(r) * kj, u1 = row_word<13>(r) * kj, u2 = row_word<17>(r) * kj, u3 = row_word<21>(r) * kj;
        asm("s_nop 1\n\t"
            LP_FMAC_ROW("%0", "%4", "4", "%5")
            LP_FMAC_ROW("%1", "%4", "6", "%5")
            LP_FMAC_ROW("%2", "%4", "8", "%5")
            LP_FMAC_ROW("%3", "%4", "10", "%5")
            : "+v"(u0), "+v"(u1), "+v"(u2), "+v"(u3)
            : "v"(r.x), "v"(ki));
        const float h0 = u0 + row_word<10>(r), l0 = u0 + row_word<11>(r);
        const float h1 = u1 + row_word<14>(r), l1 = u1 + row_word<15>(r);
        const float h2 = u2 + row_word<18>(r), l2 = u2 + row_word<19>(r);
        const float h3 = u3 + row_word<22>(r), l3 = u3 + row_word<23>(r);
        lo = fmaxf(fmaxf(l0, l1), fmaxf(l2, l3));
        return fminf(fminf(h0, h1), fminf(h2, h3)) - lo;
    } else {
        float h0 = row_word<10>(r), h1 = row_word<13>(r), h2 = row_word<16>(r);
        float l0 = row_word<19>(r), l1 = row_word<22>(r), l2 = row_word<25>(r);
        asm("s_nop 1\n\t"
            LP_FMAC_ROW("%0", "%7", "4", "%9")
            LP_FMAC_ROW("%1", "%6", "6", "%9")
            LP_FMAC_ROW("%2", "%7", "7", "%9")
            LP_FMAC_ROW("%3", "%6", "9", "%9")
            LP_FMAC_ROW("%4", "%7", "10", "%9")
            LP_FMAC_ROW("%5", "%6", "12", "%9")
            LP_FMAC_ROW("%0", "%6", "4", "%8")
            LP_FMAC_ROW("%1", "%7", "5", "%8")
            LP_FMAC_ROW("%2", "%6", "7", "%8")
            LP_FMAC_ROW("%3", "%7", "8", "%8")
            LP_FMAC_ROW("%4", "%6", "10", "%8")
            LP_FMAC_ROW("%5", "%7", "11", "%8")
            : "+v"(h0), "+v"(h1), "+v"(h2), "+v"(l0), "+v"(l1), "+v"(l2)
            : "v"(r.x), "v"(r.y), "v"(ki), "v"(kj));
        lo = fmaxf(fmaxf(l0, l1), l2);
        return fminf(fminf(h0, h1), h2) - lo;
    }
}
// c += w rgb
__device__ inline void add_colour_row(float2 r, float w, float& c0, float& c1, float& c2) {
    asm("s_nop 1\n\t"
        LP_FMAC_ROW("%0", "%4", "0", "%5")
        LP_FMAC_ROW("%1", "%3", "1", "%5")
        LP_FMAC_ROW("%2", "%4", "1", "%5")
        : "+v"(c0), "+v"(c1), "+v"(c2)
        : "v"(r.x), "v"(r.y), "v"(w));
}

// Exact variant (no ray space): each plane k bounds the relative depth tau
// along the pixel ray at (u_k + h) / (c_k - u_k).  Per plane: u, 1/(c - u),
// the plane's upper and lower bounds (a tetrahedron face is an exit where
// c - u >= 0, an entry elsewhere; the other bound is infinite).  A plane
// parallel to the ray gives infinite (or, on its boundary, NaN) bounds,
// which the min / max reductions ignore.
struct ExactPlanes {
    float u[4], inv[4], hi[4], lo[4];
    float U, L;
};

// Plane k with u at the pixel and constant c.
template <int KIND>
__device__ inline void exact_plane(float u, float c, int k, ExactPlanes& X) {
#pragma clang fp contract(off)
    const float den = c - u;
    const float inv = __builtin_amdgcn_rcpf(den);
    X.u[k] = u;
    X.inv[k] = inv;
    if (KIND == LINPRIM_OCTAHEDRON) {
        const float ui = u * inv;
        const float t1 = ui - inv, t2 = ui + inv;
        X.hi[k] = fmaxf(t1, t2);
        X.lo[k] = fminf(t1, t2);
    } else {
        const float t = __builtin_fmaf(u, inv, inv);
        const bool ex = den >= 0.0f;
        X.hi[k] = ex ? t : INFINITY;
        X.lo[k] = ex ? -INFINITY : t;
    }
    X.U = fminf(X.U, X.hi[k]);
    X.L = fmaxf(X.L, X.lo[k]);
}

// All four, from a record spread over the row (see chord_row).
template <int KIND>
__device__ inline void exact_planes_row(float2 r, float ki, float kj, ExactPlanes& X) {
    float u0 = row_word<10>(r), u1 = row_word<14>(r), u2 = row_word<18>(r), u3 = row_word<22>(r);
    asm("s_nop 1\n\t"
        LP_FMAC_ROW("%0", "%5", "4", "%7")
        LP_FMAC_ROW("%1", "%5", "6", "%7")
        LP_FMAC_ROW("%2", "%5", "8", "%7")
        LP_FMAC_ROW("%3", "%5", "10", "%7")
        LP_FMAC_ROW("%0", "%4", "4", "%6")
        LP_FMAC_ROW("%1", "%4", "6", "%6")
        LP_FMAC_ROW("%2", "%4", "8", "%6")
        LP_FMAC_ROW("%3", "%4", "10", "%6")
        : "+v"(u0), "+v"(u1), "+v"(u2), "+v"(u3)
        : "v"(r.x), "v"(r.y), "v"(ki), "v"(kj));
    X.U = INFINITY;
    X.L = -INFINITY;
    exact_plane<KIND>(u0, row_word<11>(r), 0, X);
    exact_plane<KIND>(u1, row_word<15>(r), 1, X);
    exact_plane<KIND>(u2, row_word<19>(r), 2, X);
    exact_plane<KIND>(u3, row_word<23>(r), 3, X);
}
#undef LP_FMAC_ROW

// All four, from a whole record.
template <int KIND>
__device__ inline void exact_planes(const Rec& R, float ki, float kj, ExactPlanes& X) {
    X.U = INFINITY;
    X.L = -INFINITY;
#pragma unroll
    for (int k = 0; k < 4; ++k)
        exact_plane<KIND>(__builtin_fmaf(R.p[4 * k + 0], ki, __builtin_fmaf(R.p[4 * k + 1], kj, R.p[4 * k + 2])),
                          R.p[4 * k + 3], k, X);
}

// |D| (min exits - max entries) with rn = |D| of the pixel ray; the z_c
// factor of the chord is folded into the record's sigma.
__device__ inline float exact_chord(const ExactPlanes& X, float rn) {
#pragma clang fp contract(off)
    return (X.U - X.L) * rn;
}

// Opacity factors of a chord: e = exp(-sigma chord), 1 - o = max(e, 0.01).
__device__ inline float chord_exp(float s2, float delta) {
#pragma clang fp contract(off)
    return __builtin_amdgcn_exp2f(-(s2 * delta));
}

// |D| of the exact variant's pixel ray D = ((x + 1/2 - cx)/fx, (y + 1/2 - cy)/fy, 1).
__device__ inline float ray_norm(const ViewInfo& V, int x, int y) {
    const float rx = (float)(((double)x + 0.5 - V.cx) / V.fx);
    const float ry = (float)(((double)y + 0.5 - V.cy) / V.fy);
    return sqrtf(rx * rx + ry * ry + 1.0f);
}

// ---------------------------------------------------------------------------
// Wave placement: wave w (XCD-chunked) handles group q = w % NQ of the tile at
// position w / NQ of a render order.  The forward's: heavy tiles first, then
// the others, each part in tile order, so that consecutive positions are
// mostly neighbouring tiles.  The backward's (also taken by the exact
// variant's forward): longest lists first in classes of list length (tile
// order inside a class), so that the waves that start last are short and
// the kernel has no long tail.
// ---------------------------------------------------------------------------
struct Place {
    int v, tx, ty, gx0, gy0, W, H, q;
    int64_t g;
};

template <int TILE>
__device__ inline Place place_wave(const ViewInfo* __restrict__ views, int n_views, const uint32_t* __restrict__ order) {
    constexpr int QX = TILE / 8, NQ = QX * QX;
    const int64_t w = xcd_tile(blockIdx.x, gridDim.x);
    Place P;
    P.g = order[w / NQ];
    P.q = (int)(w % NQ);
    P.v = find_view(views, n_views, P.g);
    P.W = views[P.v].width;
    P.H = views[P.v].height;
    const int tiles_x = views[P.v].tiles_x;
    const int64_t lt = P.g - views[P.v].tile_base;
    P.tx = (int)(lt % tiles_x);
    P.ty = (int)(lt / tiles_x);
    P.gx0 = P.tx * TILE + (P.q % QX) * 8;
    P.gy0 = P.ty * TILE + (P.q / QX) * 8;
    return P;
}

__device__ inline bool rect_meets_group(int4 r, int gx0, int gy0) {
    return !(r.x > gx0 + 7 || r.z < gx0 || r.y > gy0 + 7 || r.w < gy0);
}

// One batch of up to 64 list entries starting at e0: lane l holds entry
// e0 + l's primitive index and the index of the gradient record of that
// (tile, primitive) pair and this group.
struct Batch {
    uint32_t idx;
    uint32_t off;      // gradient record index
    uint64_t mask;     // entries whose pixel rectangle meets the group
};

// Gradient records of a slot are laid out by tile of its tile rectangle
// (row-major), NQ groups per tile, from the slot's pair offset on.
__device__ inline uint32_t record_index(int4 r, int tile_shift, int tx, int ty, uint32_t prim_offset, int NQ, int q) {
    const int tx0 = r.x >> tile_shift, ty0 = r.y >> tile_shift, tx1 = r.z >> tile_shift;
    return (prim_offset + (uint32_t)((ty - ty0) * (tx1 - tx0 + 1) + (tx - tx0))) * (uint32_t)NQ + (uint32_t)q;
}

template <int NQ>
__device__ inline Batch load_batch(const float* __restrict__ base, const uint32_t* __restrict__ vals,
                                   const uint32_t* __restrict__ offs, uint32_t e0, uint32_t nb, int gx0, int gy0,
                                   int tile_shift, int tx, int ty, int q) {
    const int lane = threadIdx.x;
    Batch B;
    B.idx = 0;
    B.off = 0;
    bool rel = false;
    if ((uint32_t)lane < nb) {
        B.idx = vals[e0 + lane];
        const float* rp = base + (size_t)B.idx * kRecordWords;
        const int4 r = *reinterpret_cast<const int4*>(rp);
        rel = (NQ == 1) || rect_meets_group(r, gx0, gy0);
        B.off = record_index(r, tile_shift, tx, ty, offs[B.idx], NQ, q);
    }
    B.mask = __ballot(rel);
    return B;
}

// ---------------------------------------------------------------------------
// Forward.
// ---------------------------------------------------------------------------
// Depth maps of the appendix "Depth and Surface Reconstruction": the
// distance along the pixel ray to the entry of the first primitive at which
// the cumulative opacity exceeds 0.5.  The walk keeps that primitive's entry
// depth relative to its centre (ray space: the highest lower plane, whose
// depth axis is the distance from the camera; exact rays: the entry
// parameter tau); the centre's depth is added once per pixel afterwards.
constexpr float kDepthT = 0.5f;

// What bounds the walk is VALU issue, and most of it went to lanes that a
// primitive does not touch: with 8-pixel tiles an entry hits 3 to 6 of a
// group's 64 pixels and its rectangle meets 1.3 to 1.8 of its four quads.  So
// the rows of a wave walk their own quads' entries, each the next one set in
// its mask of the batch, and a step evaluates up to four entries at once: 0.43
// to 0.57 steps an entry.  The pixels of a quad still see the list in order,
// and blend with the same operations.  A record costs a row one 8-byte LDS
// read a lane, loaded a step ahead; its words reach the arithmetic as DPP
// broadcasts, not as registers.  Wave-uniform scalar loads, all lanes on the
// same entry (and LDS records for lists of more than 128): 93 us for 1M
// octahedra at 1080p, 568 for 16 views of 500k, 992 for 8 views of 3M; now 69,
// 358 and 570.  Large primitives, whose rectangles meet every quad, gain
// nothing from the split: 124 -> 121 us for a depth map of 500k with 2.9 quads an
// entry at 16-pixel tiles (88 with the outlines' test), and where a crowd of
// opaque ones fills every quad the step's own cost shows: a step is 44 VALU
// instructions (46 with a select for the empty mask and entries counted from 1)
// against 39 of the wave-uniform walk (20k octahedra 0.05-0.3 wide at 1080p,
// 8-pixel tiles: 57 us, now 59; 20k tetrahedra 76 and 79).
// Wider tiles first filter the list for the group, so that batches are full; a
// list of one batch is not filtered, which saves a sparse image a load and an
// LDS round trip per group (20k octahedra of a room at 3840 x 2160, 16-pixel
// tiles: 70 us filtered, 57 so, 57 before the quads; exact rays 75, 64 and 59;
// 16 views of 500k 417 and 387).  Seven waves per SIMD, but for depth maps at
// wide tiles, which would spill.
__device__ inline double centre_depth(const ViewInfo& V, const float* __restrict__ means, uint32_t prim, bool exact) {
    const double x = means[3 * (size_t)prim], y = means[3 * (size_t)prim + 1], z = means[3 * (size_t)prim + 2];
    const double t0 = V.Rw[0] * x + V.Rw[1] * y + V.Rw[2] * z + V.tw[0];
    const double t1 = V.Rw[3] * x + V.Rw[4] * y + V.Rw[5] * z + V.tw[1];
    const double t2 = V.Rw[6] * x + V.Rw[7] * y + V.Rw[8] * z + V.tw[2];
    return exact ? t2 : sqrt(t0 * t0 + t1 * t1 + t2 * t2);
}

// Whether no pixel centre of a quad can have a chord through the octahedron,
// for the quads at x = qx and qx + 4 and y = qy (bits 0 and 1).  A chord needs
// every upper plane above every lower one at the pixel; the difference of two
// planes is linear, so over the part of the quad inside the pixel rectangle it
// is at most |da| hx + |db| hy above the middle's.  One pair below zero
// everywhere drops the entry; those lines hold the edges of the primitive's
// outline.  The margin covers the rounding of both evaluations: at most 6 eps M
// in a pixel's h - l and 25 eps M here, eps = 2^-24 and M the largest
// |A| Kx + |B| Ky + |D| of a plane; 64 eps M is taken.  A NaN or an infinite M
// keeps the entry.
// Planes are read one pair at a time, in order, to take few registers.
__device__ inline uint32_t quads_missed(const float* rec, float gx, float gy, float qy) {
    const float bx = rec[4], by = rec[5], bw = rec[6], bh = rec[7];
    const float* w = rec + 8;
    const float kx = fmaxf(fabsf(fmaxf(gx - bx, -bw)), fabsf(fminf(gx + 7.0f - bx, bw)));
    const float ky = fmaxf(fabsf(fmaxf(gy - by, -bh)), fabsf(fminf(gy + 7.0f - by, bh)));
    const float y0 = fmaxf(qy - by, -bh), y1 = fminf(qy + 3.0f - by, bh);
    const float cy = 0.5f * (y0 + y1), hy = 0.5f * (y1 - y0);
    float cx[2], hx[2], least[2], m = 0.0f;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const float x0 = fmaxf(gx + 4.0f * (float)q - bx, -bw), x1 = fminf(gx + 4.0f * (float)q + 3.0f - bx, bw);
        cx[q] = 0.5f * (x0 + x1);
        hx[q] = 0.5f * (x1 - x0);
        least[q] = INFINITY;
    }
#pragma unroll
    for (int a = 0; a < 4; ++a) {
        const float p0 = w[4 * a], p1 = w[4 * a + 1], p2 = w[4 * a + 2], p3 = w[4 * a + 3];
        m = fmaxf(m, __builtin_fmaf(fabsf(p0), kx, __builtin_fmaf(fabsf(p1), ky, fmaxf(fabsf(p2), fabsf(p3)))));
#pragma unroll
        for (int b = a + 1; b < 4; ++b) {
            const float da = p0 - w[4 * b], db = p1 - w[4 * b + 1], up = p2 - w[4 * b + 3], dn = w[4 * b + 2] - p3;
            const float my = db * cy, ey = fabsf(db) * hy;
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const float mid = __builtin_fmaf(da, cx[q], my), ext = __builtin_fmaf(fabsf(da), hx[q], ey);
                least[q] = fminf(least[q], fminf((ext + mid) + up, (ext - mid) + dn));
            }
            asm volatile("" : "+v"(least[0]), "+v"(least[1]), "+v"(m) : : "memory");
        }
    }
    const float margin = -0x1p-18f * m;
    return (least[0] < margin ? 1u : 0u) | (least[1] < margin ? 2u : 0u);
}

// Batches in which some quad's row has at least this many entries test the
// outlines: the test costs a batch about four steps, and drops a third to a
// half of the steps where primitives are long and thin (a depth map of 500k
// octahedra at 16-pixel tiles, 42% of whose entries hit no pixel of the group:
// kernel 120 -> 88 us; from 16 or 25 on 88 and 94, and 41 -> 43 us from 16 on
// for a training view whose entries meet 1.8 quads).  8-pixel tiles, whose
// lists hold smaller rectangles, go without it: the registers it takes cost
// them more (1M octahedra at 1080p 71 -> 74 us, 16 views of 500k 370 -> 382), and
// so do tetrahedra, which fill more of their rectangles: 20k at 1080p, 0.05-0.3
// wide, 16-pixel tiles 76 us without it, 103 with it; 200k 74 and 103; 500k of a
// room 74 and 90.
constexpr int kOutlineSteps = 20;

// Exact rays: where the wave, walking a batch together, takes no more than
// kWaveSteps for every kRowSteps steps that its busiest row would take alone, it
// does so, with records in scalar registers: a step is 64 VALU instructions
// then, 69 with rows (20k octahedra 0.05-0.3 wide at 1080p, 8-pixel tiles: 75 us
// by rows alone, 65 so and when the wave always walked together; at 16-pixel
// tiles 79, 70 and 66; 300k of a room 33.0, 31.8 and 43; if no step may be lost,
// 68 for the crowd).  Ray space, 39 against 44, stays with the rows: crowds would
// gain (1M of a room 76 -> 72 us), but 16 views of 500k take 352 -> 378 and
// tetrahedra at 16-pixel tiles 382 -> 408.
constexpr int kRowSteps = 8, kWaveSteps = 9;

template <int TILE, int KIND, bool COUNT, bool EXACT, bool DEPTH>
__global__ __launch_bounds__(64, (DEPTH && TILE > 8) ? 6 : 7) void k_render_fwd(const ViewInfo* __restrict__ views, int n_views, int64_t n,
                                                   const float* __restrict__ payload, const uint32_t* __restrict__ vals,
                                                   const uint2* __restrict__ ranges, const Status* __restrict__ status,
                                                   uint64_t capacity, float bg0, float bg1, float bg2,
                                                   float* __restrict__ out_rgb, float* __restrict__ out_T,
                                                   int32_t* __restrict__ out_last,
                                                   unsigned long long* __restrict__ counters,
                                                   const float* __restrict__ means,
                                                   float* __restrict__ out_depth, const uint32_t* __restrict__ order) {
    __shared__ float4 store[33][8];
    float4 (*srec)[8] = store + 1;
    __shared__ uint2 queue[(TILE == 8) ? 1 : 96];   // (primitive, list position) of entries that meet the group
    if (status->n_pairs > capacity) return;
    constexpr int QX = TILE / 8, NQ = QX * QX;
    const Place P = place_wave<TILE>(views, n_views, order);
    if (P.gx0 >= P.W || P.gy0 >= P.H) return;
    const int lane = threadIdx.x, row = lane >> 4, li = lane & 15;
    // row r owns the quad (r & 1, r >> 1) of the group
    const int x = P.gx0 + 4 * (row & 1) + (li & 3), y = P.gy0 + 4 * (row >> 1) + (li >> 2);
    const bool valid = x < P.W && y < P.H;
    const float pxf = (float)x, pyf = (float)y;
    const float rn = EXACT ? ray_norm(views[P.v], x, y) : 1.0f;
    const uint2 rg = ranges[P.g];
    float T = 1.0f, C0 = 0.0f, C1 = 0.0f, C2 = 0.0f;
    int last = (int)rg.x;
    // lanes still compositing, as a wave-uniform mask (kept in scalar
    // registers; each lane's bit is read back with an inverse ballot)
    uint64_t live = __builtin_amdgcn_ballot_w64(valid);
    uint32_t ev = 0, hit = 0, term = rg.y;
    uint32_t half = 0xffffffffu;   // list position at which 1 - T first exceeds 0.5
    float half_entry = 0.0f;       // its entry depth relative to its centre
    const float* base = payload + (size_t)P.v * (size_t)n * kRecordWords;
    // counted renders count every pixel of a rectangle
    constexpr bool kOutline = NQ > 1 && KIND == LINPRIM_OCTAHEDRON && !EXACT && !COUNT;
    uint32_t seen = ~0u;           // the batch's last blended entry
    auto in_box = [&](float ki, float kj, float wi, float wj) {
        // lane masks of single compares combine in scalar registers
        return __builtin_amdgcn_ballot_w64(fabsf(ki) <= wi) & __builtin_amdgcn_ballot_w64(fabsf(kj) <= wj) & live;
    };
    // Branch-free: lanes that do not see the primitive blend with
    // 1 - o = 1 exactly, which leaves C and T unchanged.
    auto composite = [&](uint64_t m_in, float dch, float entry, float eh, uint32_t e, auto add_colour) {
        const uint64_t m_hit = m_in & __builtin_amdgcn_ballot_w64(dch > 0.0f);
        const bool hitp = __builtin_amdgcn_inverse_ballot_w64(m_hit);
        if (COUNT) {
            ev += __builtin_amdgcn_inverse_ballot_w64(m_in) ? 1u : 0u;
            hit += hitp ? 1u : 0u;
        }
        const float ex = hitp ? eh : 1.0f;
        const float onemo = fmaxf(ex, kOneMinusOMax);
        const float w = T * (1.0f - onemo);
        add_colour(w);
        if (DEPTH) {
            const bool cross = T >= kDepthT && T * onemo < kDepthT;
            half = cross ? e : half;
            half_entry = cross ? entry : half_entry;
        }
        T = T * onemo;
        seen = hitp ? e : seen;
        // T only falls where the primitive was hit
        const uint64_t stop = __builtin_amdgcn_ballot_w64(T <= kTStop) & m_hit;
        if (COUNT) term = __builtin_amdgcn_inverse_ballot_w64(stop) ? e : term;
        live &= ~stop;
    };
    // an entry of each row's own, its record spread over the row
    auto blend = [&](float2 words, uint32_t e) {
        const float ki = pxf - row_word<4>(words), kj = pyf - row_word<5>(words);
        const uint64_t m_in = in_box(ki, kj, row_word<6>(words), row_word<7>(words));
        float dch, entry = 0.0f;
        if (EXACT) {
            ExactPlanes X;
            exact_planes_row<KIND>(words, ki, kj, X);
            dch = exact_chord(X, rn);
            entry = X.L;
        } else {
            dch = chord_row<KIND>(words, ki, kj, entry);
        }
        // broadcasts run with every lane: outside the selection
        composite(m_in, dch, entry, chord_exp(row_word<0>(words), dch), e,
                  [&](float w) { add_colour_row(words, w, C0, C1, C2); });
    };
    // one entry for the whole wave, its record in scalar registers
    auto blend_together = [&](const Rec& R, uint32_t e) {
        const float ki = pxf - R.fi0, kj = pyf - R.fj0;
        const uint64_t m_in = in_box(ki, kj, R.fwi, R.fwj);
        ExactPlanes X;
        exact_planes<KIND>(R, ki, kj, X);
        const float dch = exact_chord(X, rn);
        composite(m_in, dch, X.L, chord_exp(R.s2, dch), e, [&](float w) {
            C0 = __builtin_fmaf(w, R.r, C0);
            C1 = __builtin_fmaf(w, R.g, C1);
            C2 = __builtin_fmaf(w, R.b, C2);
        });
    };
    constexpr int NQD = rec_quads<KIND, EXACT>(), NH = (NQD + 1) / 2;
    const uint32_t sl = (uint32_t)lane & 31u, q0 = ((uint32_t)lane >> 5) * NH;
    // lanes l and l + 32 bring the two halves of entry l's record
    float4 st[NH];
    auto fetch = [&](uint32_t idx) {
        const float4* rp = reinterpret_cast<const float4*>(base + (size_t)idx * kRecordWords);
#pragma unroll
        for (int k = 0; k < NH; ++k) st[k] = rp[1 + min((int)q0 + k, NQD - 1)];
    };
    // entry -1: a record no pixel lies in, for a row without one
    if (lane < 8) srec[-1][lane] = (lane == 1) ? make_float4(0.f, 0.f, -1.f, -1.f) : make_float4(0.f, 0.f, 0.f, 0.f);
    const float2* words = reinterpret_cast<const float2*>(srec[0]) + li;
    // The next up to 32 entries that meet the group: their number, their list
    // positions and primitives (lane l: entry l & 31), their records on the way.
    // A group-sized tile takes its list as it is, and so does a list of one batch
    // (the quads' masks leave out what does not meet the group); others are
    // filtered, 64 entries at a time.
    const bool whole = NQ == 1 || rg.y - rg.x <= 32u;
    uint32_t ce = rg.x, qn = 0;
    auto chunk = [&](uint32_t e) {
        const uint32_t k = whole ? sl : (uint32_t)lane;
        return (e < rg.y && k < rg.y - e) ? vals[e + k] : 0u;
    };
    uint32_t idx0 = chunk(ce), idx1 = chunk(ce + (NQ == 1 ? 32u : 64u));
    int4 rect = make_int4(0, 0, 0, 0);
    if (!whole) rect = *reinterpret_cast<const int4*>(base + (size_t)idx0 * kRecordWords);
    auto take = [&](uint32_t& pos, uint32_t& prim) {
        uint32_t n = 0;
        if (whole) {
            n = min(32u, rg.y - ce);
            pos = ce + sl;
            prim = idx0;
            ce += n;
            if (NQ == 1) {
                idx0 = idx1;
                idx1 = chunk(ce + 32);
            }
        } else {
            while (qn < 32 && ce < rg.y) {
                const bool rel = (uint32_t)lane < rg.y - ce && rect_meets_group(rect, P.gx0, P.gy0);
                const uint64_t m = __builtin_amdgcn_ballot_w64(rel);
                const uint32_t r = qn + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                                                  __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
                if (rel) queue[r] = make_uint2(idx0, ce + (uint32_t)lane);
                qn += (uint32_t)__builtin_popcountll(m);
                ce += 64;
                idx0 = idx1;
                if (ce < rg.y) rect = *reinterpret_cast<const int4*>(base + (size_t)idx0 * kRecordWords);
                idx1 = chunk(ce + 64);
            }
            lds_hand_over();
            n = min(32u, qn);
            const uint2 e = queue[sl < n ? sl : 0u], rest = queue[min(32u + (uint32_t)lane, 95u)];
            pos = e.y;
            prim = sl < n ? e.x : 0u;
            qn -= n;
            lds_hand_over();
            if ((uint32_t)lane < qn) queue[lane] = rest;
            lds_hand_over();
        }
        if (n) fetch(prim);
        return n;
    };
    uint32_t pos, prim, n_here = take(pos, prim);
    while (n_here && live) {
        // which entries' rectangles meet each quad, from the first halves
        const float4 box = st[1];
        const float bx0 = box.x - box.z, bx1 = box.x + box.z, by0 = box.y - box.w, by1 = box.y + box.w;
        const float gx = (float)P.gx0, gy = (float)P.gy0;
        const uint32_t here = n_here < 32u ? (1u << n_here) - 1u : ~0u;
        auto meets = [&](float lo, float hi, float q) {
            return (uint32_t)(__builtin_amdgcn_ballot_w64(lo <= q + 3.0f) & __builtin_amdgcn_ballot_w64(hi >= q));
        };
        const uint32_t ml = meets(bx0, bx1, gx) & here, mr = meets(bx0, bx1, gx + 4.0f) & here;
        const uint32_t mt = meets(by0, by1, gy), mb = meets(by0, by1, gy + 4.0f);
        uint32_t m0 = ml & mt, m1 = mr & mt, m2 = ml & mb, m3 = mr & mb;
#pragma unroll
        for (int k = 0; k < NH; ++k)
            if ((int)q0 + k < NQD) srec[sl][q0 + k] = st[k];
        lds_hand_over();   // other lanes read what this one staged
        if (kOutline) {
            const int steps = max(max(__builtin_popcount(m0), __builtin_popcount(m1)),
                                  max(__builtin_popcount(m2), __builtin_popcount(m3)));
            if (steps >= kOutlineSteps) {
                // lanes l and l + 32 test the upper and the lower quads of entry l
                const uint32_t missed = quads_missed(reinterpret_cast<const float*>(srec[sl]), gx, gy,
                                                           lane < 32 ? gy : gy + 4.0f);
                const uint64_t xl = __builtin_amdgcn_ballot_w64(missed & 1u), xr = __builtin_amdgcn_ballot_w64(missed & 2u);
                m0 &= ~(uint32_t)xl;
                m1 &= ~(uint32_t)xr;
                m2 &= ~(uint32_t)(xl >> 32);
                m3 &= ~(uint32_t)(xr >> 32);
            }
        }
        const uint32_t mine_q = (row & 2) ? ((row & 1) ? m3 : m2) : ((row & 1) ? m1 : m0);
        uint32_t mask = ((uint32_t)(live >> (lane & 48)) & 0xffffu) ? mine_q : 0u;
        uint32_t pos1, prim1;
        n_here = take(pos1, prim1);
        // inside the batch entries count from 0
        const uint32_t half0 = half, term0 = term;
        seen = ~0u;
        half = 0xffffffffu;
        term = ~0u;
        auto next = [&](uint32_t& e, float2& w) {
            // the lowest set bit, ~0 for none (the compiler adds a select for that)
            asm("v_ffbl_b32 %0, %1" : "=v"(e) : "v"(mask));
            mask &= mask - 1u;
            w = words[(int)e * 16];
        };
        if (EXACT) {
            uint32_t any = m0 | m1 | m2 | m3;
            const int most = max(max(__builtin_popcount(m0), __builtin_popcount(m1)),
                                 max(__builtin_popcount(m2), __builtin_popcount(m3)));
            if (any && __builtin_popcount(any) * kRowSteps <= most * kWaveSteps) {
                mask = 0;
                auto next_rec = [&](Rec& R) {
                    const int b = __builtin_ctz(any);
                    any &= any - 1u;
                    load_rec<KIND>(base + (size_t)(uint32_t)__builtin_amdgcn_readlane((int)prim, b) * kRecordWords, R);
                    return (uint32_t)b;
                };
                // Scalar loads complete out of order: wait for all in flight,
                // then issue the next record's, then blend the one waited for.
                Rec RA, RB;
                uint32_t eA = next_rec(RA), eB = 0;
                while (live) {
                    smem_wait_all();
                    const bool haveB = any != 0;
                    if (haveB) eB = next_rec(RB);
                    sched_fence();
                    blend_together(RA, eA);
                    if (!haveB || !live) break;
                    smem_wait_all();
                    const bool haveA = any != 0;
                    if (haveA) eA = next_rec(RA);
                    sched_fence();
                    blend_together(RB, eB);
                    if (!haveA) break;
                }
            }
        }
        uint32_t eA, eB;
        float2 wA, wB;
        next(eA, wA);
        next(eB, wB);
        while (live && __builtin_amdgcn_ballot_w64((int)eA >= 0)) {
            blend(wA, eA);
            next(eA, wA);
            blend(wB, eB);
            next(eB, wB);
        }
        lds_hand_over();
        auto list_pos = [&](uint32_t e) {
            return (NQ == 1) ? (uint32_t)__builtin_amdgcn_readfirstlane((int)pos) + e : (uint32_t)__shfl((int)pos, (int)(e & 31u));
        };
        const uint32_t p_last = list_pos(seen);
        last = (seen != ~0u) ? (int)p_last + 1 : last;
        if (DEPTH) {
            const uint32_t p_half = list_pos(half);
            half = (half != 0xffffffffu) ? p_half : half0;
        }
        if (COUNT) {
            const uint32_t p_term = list_pos(term);
            term = (term != ~0u) ? p_term + 1 : term0;
        }
        pos = pos1;
        prim = prim1;
    }
    unsigned long long c_it = 0, c_ev = 0, c_hit = 0;
    if (valid) {
        const int64_t p = (int64_t)y * P.W + x;
        const int64_t pix = views[P.v].pix_base + p;
        const int64_t hw = (int64_t)P.W * P.H;
        float* o = out_rgb + 3 * views[P.v].pix_base;
        o[p] = C0 + T * bg0;
        o[hw + p] = C1 + T * bg1;
        o[2 * hw + p] = C2 + T * bg2;
        out_T[pix] = T;
        out_last[pix] = last;
        if (DEPTH) {
            float dz = 0.0f;
            if (half != 0xffffffffu) {
                const double zc = centre_depth(views[P.v], means, vals[half], EXACT);
                // exact rays: camera depth z_c (1 + tau) times |D|
                dz = EXACT ? (float)((zc + zc * (double)half_entry) * (double)rn) : (float)(zc + (double)half_entry);
            }
            out_depth[pix] = dz;
        }
        if (COUNT) {
            c_it = term - rg.x;
            c_ev = ev;
            c_hit = hit;
        }
    }
    if (COUNT) {
        const float fi = wave_sum((float)c_it), fe = wave_sum((float)c_ev), fh = wave_sum((float)c_hit);
        if (lane == 0) {
            atomicAdd(counters + 0, (unsigned long long)fi);
            atomicAdd(counters + 1, (unsigned long long)fe);
            atomicAdd(counters + 2, (unsigned long long)fh);
        }
    }
}

// ---------------------------------------------------------------------------
// Backward: reverse walk recomputing transmittance.  One gradient record of
// kGradWords floats per (tile, primitive) pair and group, at
// (pair slot) * NQ + q, written for every entry whose rectangle meets the
// group (zeros if no pixel of the group reached it):
//   octahedron: [4 s + 0..3] dL/d(A_s, B_s, Dup_s, Dlo_s) for slab s
//   tetrahedron: [3 f + 0..2] dL/d(A_f, B_f, D_f) for face f
//   [16..18] dL/d rgb, [19] dL/d sigma
// ---------------------------------------------------------------------------

// One step of the backward walk for this lane's pixel, branch-free: a lane
// that does not see the primitive (not active, outside the rectangle, zero
// chord) runs the same instructions with delta = 0, o = 0, 1 - o = 1, which
// leaves T and the colour behind (GB = dL/dC . colour behind) unchanged
// exactly and yields zero terms.  Writes the lane's gradient terms of the
// entry's record into acc; returns whether the lane contributed.
template <int KIND>
__device__ inline bool bwd_step(const Rec& R, bool active, float pxf, float pyf, float G0, float G1,
                                float G2, float& T, float& GB, float (&acc)[kGradWords]) {
    const float ki = pxf - R.fi0, kj = pyf - R.fj0;
    const bool inside = active & (fabsf(ki) <= R.fwi) & (fabsf(kj) <= R.fwj);
    // chord and the active (lowest upper, highest lower) planes,
    // the first one in plane order on ties; the chord is the same
    // number the forward computed
    float dch;
    bool eh[4], el[4];
    int ih = 0, il = 0;
    if (KIND == LINPRIM_OCTAHEDRON) {
#pragma clang fp contract(off)
        float h[4], l[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const float u = __builtin_fmaf(R.p[4 * s + 0], ki, R.p[4 * s + 1] * kj);
            h[s] = u + R.p[4 * s + 2];
            l[s] = u + R.p[4 * s + 3];
        }
        const float hi = fminf(fminf(h[0], h[1]), fminf(h[2], h[3]));
        const float lo = fmaxf(fmaxf(l[0], l[1]), fmaxf(l[2], l[3]));
        dch = hi - lo;
        bool fh = false, fl = false;
#pragma unroll
        for (int s = 0; s < 3; ++s) {
            eh[s] = !fh && h[s] == hi;
            el[s] = !fl && l[s] == lo;
            fh = fh || eh[s];
            fl = fl || el[s];
        }
        eh[3] = !fh;
        el[3] = !fl;
    } else {
        dch = chord<KIND>(R, ki, kj, ih, il);
    }
    const bool contributed = inside && dch > 0.0f;
    const float delta = contributed ? dch : 0.0f;
    const float ex = contributed ? chord_exp(R.s2, delta) : 1.0f;
    const float onemo = fmaxf(ex, kOneMinusOMax);
    const float o = 1.0f - onemo;
    const float ro = __builtin_amdgcn_rcpf(onemo);
    const float Tk = T * ro;                     // transmittance in front of this primitive
    // dL/do = G . (T_k rgb - behind / (1 - o))
    const float Grgb = G0 * R.r + G1 * R.g + G2 * R.b;
    const float dLdo = Tk * Grgb - ro * GB;
    const float wk = Tk * o;
    acc[16] = G0 * wk;
    acc[17] = G1 * wk;
    acc[18] = G2 * wk;
    GB += wk * Grgb;
    T = Tk;
    // not clamped: o = 1 - exp(-sigma chord)
    const bool open = contributed && ex >= kOneMinusOMax;
    const float q = dLdo * ex;
    const float gD = open ? q * R.sigma : 0.0f;    // dL/dchord
    acc[19] = open ? q * delta : 0.0f;             // dL/dsigma
    if (KIND == LINPRIM_OCTAHEDRON) {
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const float gh = eh[s] ? gD : 0.0f;
            const float gl = el[s] ? -gD : 0.0f;
            const float d = gh + gl;
            acc[4 * s + 0] = d * ki;
            acc[4 * s + 1] = d * kj;
            acc[4 * s + 2] = gh;
            acc[4 * s + 3] = gl;
        }
    } else {
        const int fh = (R.fmap >> (2 * ih)) & 3;
        const int fl = (R.fmap >> (2 * (il + 3))) & 3;
#pragma unroll
        for (int f = 0; f < 4; ++f) {
            const float d = ((fh == f) ? gD : 0.0f) - ((fl == f) ? gD : 0.0f);
            acc[3 * f + 0] = d * ki;
            acc[3 * f + 1] = d * kj;
            acc[3 * f + 2] = d;
        }
#pragma unroll
        for (int k = 12; k < 16; ++k) acc[k] = 0.0f;
    }
    return contributed;
}

// The step of the exact variant, from a record spread over the row.
template <int KIND>
__device__ inline bool bwd_step_exact(float2 r, bool active, float pxf, float pyf, float rn, float G0, float G1,
                                      float G2, float& T, float& GB, float (&acc)[kGradWords]) {
    const float ki = pxf - row_word<4>(r), kj = pyf - row_word<5>(r);
    const bool inside = active & (fabsf(ki) <= row_word<6>(r)) & (fabsf(kj) <= row_word<7>(r));
    ExactPlanes X;
    exact_planes_row<KIND>(r, ki, kj, X);
    const float dch = exact_chord(X, rn);
    bool eh[4], el[4];
    bool fh = false, fl = false;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        eh[k] = !fh && X.hi[k] == X.U;
        el[k] = !fl && X.lo[k] == X.L;
        fh = fh || eh[k];
        fl = fl || el[k];
    }
    // broadcasts run with every lane: outside the selections
    const float ec = chord_exp(row_word<0>(r), dch);
    const bool contributed = inside && dch > 0.0f;
    const float ex = contributed ? ec : 1.0f;
    const float onemo = fmaxf(ex, kOneMinusOMax);
    const float o = 1.0f - onemo;
    const float ro = __builtin_amdgcn_rcpf(onemo);
    const float Tk = T * ro;                     // transmittance in front of this primitive
    // dL/do = G . (T_k rgb - behind / (1 - o))
    const float Grgb = G0 * row_word<1>(r) + G1 * row_word<2>(r) + G2 * row_word<3>(r);
    const float dLdo = Tk * Grgb - ro * GB;
    const float wk = Tk * o;
    acc[16] = G0 * wk;
    acc[17] = G1 * wk;
    acc[18] = G2 * wk;
    GB += wk * Grgb;
    T = Tk;
    // not clamped: o = 1 - exp(-sigma chord)
    const bool open = contributed && ex >= kOneMinusOMax;
    const float q = dLdo * ex, qs = q * row_word<26>(r);
    const float gD = open ? qs : 0.0f;             // dL/dchord
    acc[19] = open ? q * dch : 0.0f;               // dL/dsigma
    {
        // words 4 k + 0..3: dL/d(a_k, b_k, g_k, c_k); a plane bound
        // tau = (u + h) / (c - u) has dtau/du = (c + h) / (c - u)^2
        // and dtau/dc = -tau / (c - u)
        const float g = gD * rn;                   // dL/d(U - L)
        const float cw[4] = {row_word<11>(r), row_word<15>(r), row_word<19>(r), row_word<23>(r)};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const float c = cw[k];
            const float inv = X.inv[k];
            const float ge = eh[k] ? g : 0.0f, gl = el[k] ? g : 0.0f;
            float gu;
            if (KIND == LINPRIM_OCTAHEDRON) {
                // the upper bound has h = +1 where c - u >= 0, else h = -1
                const float hh = (c - X.u[k] >= 0.0f) ? 1.0f : -1.0f;
                gu = (ge * (c + hh) - gl * (c - hh)) * (inv * inv);
            } else {
                gu = (ge - gl) * (c + 1.0f) * (inv * inv);
            }
            const float gc = (gl * X.L - ge * X.U) * inv;
            const bool act = eh[k] || el[k];
            const float Gu = act ? gu : 0.0f, Gc = act ? gc : 0.0f;
            acc[4 * k + 0] = Gu * ki;
            acc[4 * k + 1] = Gu * kj;
            acc[4 * k + 2] = Gu;
            acc[4 * k + 3] = Gc;
        }
    }
    return contributed;
}

template <int TILE, int KIND>
__global__ __launch_bounds__(64) void k_render_bwd(const ViewInfo* __restrict__ views, int n_views, int64_t n,
                                                   const float* __restrict__ payload, const uint32_t* __restrict__ vals,
                                                   const uint2* __restrict__ ranges, const uint32_t* __restrict__ offsets,
                                                   const Status* __restrict__ status, uint64_t capacity, float bg0,
                                                   float bg1, float bg2, const float* __restrict__ out_T,
                                                   const int32_t* __restrict__ out_last,
                                                   const float* __restrict__ grad_rgb, float* __restrict__ grads,
                                                   const uint32_t* __restrict__ order) {
    if (status->n_pairs > capacity) return;
    constexpr int QX = TILE / 8, NQ = QX * QX;
    constexpr int SHIFT = (TILE == 8) ? 3 : (TILE == 16) ? 4 : 5;
    const Place P = place_wave<TILE>(views, n_views, order);
    if (P.gx0 >= P.W || P.gy0 >= P.H) return;
    const int lane = threadIdx.x;
    const int x = P.gx0 + (lane & 7), y = P.gy0 + (lane >> 3);
    const bool valid = x < P.W && y < P.H;
    const float pxf = (float)x, pyf = (float)y;
    const uint2 rg = ranges[P.g];
    const int64_t hw = (int64_t)P.W * P.H;
    const float* base = payload + (size_t)P.v * (size_t)n * kRecordWords;
    const uint32_t* offs = offsets + (size_t)P.v * (size_t)n;

    // GB = dL/dC . (colour behind the current step), kept as one running
    // dot product (the colour behind itself is not needed)
    float T = 1.0f, GB = 0.0f, G0 = 0.0f, G1 = 0.0f, G2 = 0.0f;
    int last = (int)rg.x;
    if (valid) {
        const int64_t p = (int64_t)y * P.W + x;
        const int64_t pix = views[P.v].pix_base + p;
        const float* gi = grad_rgb + 3 * views[P.v].pix_base;
        T = out_T[pix];
        // stay inside this tile's list whatever the caller passed
        last = min(max(out_last[pix], (int)rg.x), (int)rg.y);
        G0 = gi[p];
        G1 = gi[hw + p];
        G2 = gi[2 * hw + p];
        // the colour behind starts as T_final bg
        GB = T * (G0 * bg0 + G1 * bg1 + G2 * bg2);
    }
    const uint32_t walk_end = (uint32_t)wave_max_int(last);

    // zero records of the entries that meet the group but no pixel reached
    for (uint32_t e0 = walk_end; e0 < rg.y; e0 += 64) {
        const Batch bt = load_batch<NQ>(base, vals, offs, e0, min(64u, rg.y - e0), P.gx0, P.gy0, SHIFT, P.tx,
                                              P.ty, P.q);
        uint64_t mask = bt.mask;
        while (mask) {
            const int b = __builtin_ctzll(mask);
            mask &= mask - 1;
            const uint32_t slot = (uint32_t)__builtin_amdgcn_readlane((int)bt.off, b);
            if (lane < kGradWords) grads[(size_t)slot * kGradWords + lane] = 0.0f;
        }
    }

    const int ridx = reduce20_index(lane);   // the word of a record this lane writes
    uint32_t word = 4u * (uint32_t)ridx;
    for (uint32_t e_hi = walk_end; e_hi > rg.x;) {
        const uint32_t nb = min(64u, e_hi - rg.x);
        const uint32_t e0 = e_hi - nb;
        e_hi = e0;
        const Batch bt = load_batch<NQ>(base, vals, offs, e0, nb, P.gx0, P.gy0, SHIFT, P.tx, P.ty, P.q);
        uint64_t mask = bt.mask;
        if (!mask) continue;
        // Entries in reverse order, two record buffers used in turn, with no
        // copies.  Scalar loads complete out of order, so waiting for one buffer
        // means waiting for every scalar load in flight: wait first, then issue
        // the next record's load, then step from the buffer just waited for.
        auto next_rec = [&](Rec& R) {
            const int b = 63 - __builtin_clzll(mask);
            mask &= ~(1ull << b);
            load_rec<KIND>(base + (size_t)(uint32_t)__builtin_amdgcn_readlane((int)bt.idx, b) *
                                             kRecordWords, R);
            return b;
        };
        auto step = [&](const Rec& R, int bcur) {
            const uint32_t e = e0 + (uint32_t)bcur;
            // a lane past its last blended entry takes no part
            float acc[kGradWords];
            const bool contributed = bwd_step<KIND>(R, (int)e < last, pxf, pyf, G0, G1, G2, T, GB, acc);
            const size_t slot = (uint32_t)__builtin_amdgcn_readlane((int)bt.off, bcur);
            float outv = 0.0f;
            if (__ballot(contributed) != 0) outv = wave_reduce20(acc, lane);
            // a scalar address and the lane's offset, kept apart: a 64-bit
            // multiply-add per lane costs four issue slots
            asm("" : "+v"(word));
            if (ridx >= 0) *reinterpret_cast<float*>(reinterpret_cast<char*>(grads + slot * kGradWords) + word) = outv;
        };
        Rec RA, RB;
        int bA = next_rec(RA), bB = 0;
        while (true) {
            smem_wait_all();
            const bool haveB = mask != 0;
            if (haveB) bB = next_rec(RB);
            sched_fence();
            step(RA, bA);
            if (!haveB) break;
            smem_wait_all();
            const bool haveA = mask != 0;
            if (haveA) bA = next_rec(RA);
            sched_fence();
            step(RB, bB);
            if (!haveA) break;
        }
    }
}

// ---------------------------------------------------------------------------
// Backward of the exact variant: each 16-lane row of the wave owns one 4 x 4
// quad of the 8 x 8 group and walks, in reverse list order, only the entries
// whose rectangle meets its quad and that lie before the last blended entry
// of one of its pixels; the four rows walk independently, so a step
// evaluates up to four entries.  The list is taken in batches of kBwdBatch
// entries: the batch's records (words 4..31) are staged in LDS, a row reads
// the record of its current entry from there as the forward does (8 bytes a
// lane, the words as broadcasts), sums its 16 lanes' gradient
// terms (transposed, inside the row) and adds them to the entry's LDS
// accumulator, the rows one after the other (a fixed order); the batch's
// records are then written out, one per lane.  Same records as
// k_render_bwd.  The exact step is heavy enough that skipping the entries a
// quad does not meet pays for the LDS round trips; the ray-space step is not.
// Bound by VALU issue (85%) and, with whole records read by every lane, by LDS
// as well (80% of its cycles): 300k octahedra at 1597 x 1199, 144 -> 139 us by
// the broadcasts, 135 by the bank-masked sums.
// ---------------------------------------------------------------------------
constexpr int kBwdBatch = 32;
static_assert(kBwdBatch <= 32, "entry masks are 32-bit");

// o[j] = x[j] of lanes i and 15 - i (row mirror) or 7 - i (half-row mirror),
// and y[j] of them in the upper half of the row or half row: an add of all
// lanes, then one whose bank mask keeps to the upper halves, in place of two
// selects and an add.
template <bool ROW>
__device__ inline void fold5(const float* x, const float* y, float* o) {
    if (ROW)
        asm("s_nop 1\n\t"     // a register is read through DPP two wait states after its write
            "v_add_f32_dpp %0, %5, %5 row_mirror row_mask:0xf bank_mask:0xf\n\t"
            "v_add_f32_dpp %1, %6, %6 row_mirror row_mask:0xf bank_mask:0xf\n\t"
            "v_add_f32_dpp %2, %7, %7 row_mirror row_mask:0xf bank_mask:0xf\n\t"
            "v_add_f32_dpp %3, %8, %8 row_mirror row_mask:0xf bank_mask:0xf\n\t"
            "v_add_f32_dpp %4, %9, %9 row_mirror row_mask:0xf bank_mask:0xf\n\t"
            "v_add_f32_dpp %0, %10, %10 row_mirror row_mask:0xf bank_mask:0xc\n\t"
            "v_add_f32_dpp %1, %11, %11 row_mirror row_mask:0xf bank_mask:0xc\n\t"
            "v_add_f32_dpp %2, %12, %12 row_mirror row_mask:0xf bank_mask:0xc\n\t"
            "v_add_f32_dpp %3, %13, %13 row_mirror row_mask:0xf bank_mask:0xc\n\t"
            "v_add_f32_dpp %4, %14, %14 row_mirror row_mask:0xf bank_mask:0xc"
            : "=&v"(o[0]), "=&v"(o[1]), "=&v"(o[2]), "=&v"(o[3]), "=&v"(o[4])
            : "v"(x[0]), "v"(x[1]), "v"(x[2]), "v"(x[3]), "v"(x[4]), "v"(y[0]), "v"(y[1]), "v"(y[2]), "v"(y[3]),
              "v"(y[4]));
    else
        asm("s_nop 1\n\t"
            "v_add_f32_dpp %0, %5, %5 row_half_mirror row_mask:0xf bank_mask:0xf\n\t"
            "v_add_f32_dpp %1, %6, %6 row_half_mirror row_mask:0xf bank_mask:0xf\n\t"
            "v_add_f32_dpp %2, %7, %7 row_half_mirror row_mask:0xf bank_mask:0xf\n\t"
            "v_add_f32_dpp %3, %8, %8 row_half_mirror row_mask:0xf bank_mask:0xf\n\t"
            "v_add_f32_dpp %4, %9, %9 row_half_mirror row_mask:0xf bank_mask:0xf\n\t"
            "v_add_f32_dpp %0, %10, %10 row_half_mirror row_mask:0xf bank_mask:0xa\n\t"
            "v_add_f32_dpp %1, %11, %11 row_half_mirror row_mask:0xf bank_mask:0xa\n\t"
            "v_add_f32_dpp %2, %12, %12 row_half_mirror row_mask:0xf bank_mask:0xa\n\t"
            "v_add_f32_dpp %3, %13, %13 row_half_mirror row_mask:0xf bank_mask:0xa\n\t"
            "v_add_f32_dpp %4, %14, %14 row_half_mirror row_mask:0xf bank_mask:0xa"
            : "=&v"(o[0]), "=&v"(o[1]), "=&v"(o[2]), "=&v"(o[3]), "=&v"(o[4])
            : "v"(x[0]), "v"(x[1]), "v"(x[2]), "v"(x[3]), "v"(x[4]), "v"(y[0]), "v"(y[1]), "v"(y[2]), "v"(y[3]),
              "v"(y[4]));
}

// Sums 20 values over the 16 lanes of each row, transposed: four DPP steps
// each halve the values a lane keeps (row mirror: lane i with 15 - i, split
// on bit 3; half-row mirror: i with 7 - i, bit 2; quad swaps i with i ^ 2,
// bit 1, and i with i ^ 1, bit 0).  With base = 10 b3 + 5 b2 of the row lane
// index, a lane ends with the totals of words
//   b1 b0 = 00: base, base + 1;  01: base + 2;  10: base + 3, base + 4;
//   11: none (such a lane holds sums that nobody reads).
__device__ inline void row_reduce20(const float (&v)[20], int li, float& t0, float& t1, int& w0, int& w1) {
    const bool h3 = (li >> 3) & 1, h2 = (li >> 2) & 1, h1 = (li >> 1) & 1, h0 = li & 1;
    float a[10], b[5];
    fold5<true>(v, v + 10, a);
    fold5<true>(v + 5, v + 15, a + 5);
    fold5<false>(a, a + 5, b);
    float c[3];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const float keep = h1 ? b[j + 3] : b[j];
        const float give = h1 ? b[j] : b[j + 3];
        c[j] = keep + dpp_move<0x4E>(give);
    }
    c[2] = b[2] + dpp_move<0x4E>(b[2]);
    const float keep = h0 ? c[2] : c[0];
    const float give = h0 ? c[0] : c[2];
    t0 = keep + dpp_move<0xB1>(give);
    t1 = c[1] + dpp_move<0xB1>(c[1]);
    const int base = 10 * (int)h3 + 5 * (int)h2;
    if (!h1 && !h0) { w0 = base; w1 = base + 1; }
    else if (!h1) { w0 = base + 2; w1 = -1; }
    else if (!h0) { w0 = base + 3; w1 = base + 4; }
    else { w0 = -1; w1 = -1; }
}

template <int TILE, int KIND>
__global__ __launch_bounds__(64) void k_render_bwd_rows(const ViewInfo* __restrict__ views, int n_views, int64_t n,
                                                   const float* __restrict__ payload, const uint32_t* __restrict__ vals,
                                                   const uint2* __restrict__ ranges, const uint32_t* __restrict__ offsets,
                                                   const Status* __restrict__ status, uint64_t capacity, float bg0,
                                                   float bg1, float bg2, const float* __restrict__ out_T,
                                                   const int32_t* __restrict__ out_last,
                                                   const float* __restrict__ grad_rgb, float* __restrict__ grads,
                                                   const uint32_t* __restrict__ order) {
    __shared__ float4 srec[kBwdBatch + 1][8];         // record words 4..31
    __shared__ float sacc[kBwdBatch][kGradWords];     // gradient record accumulators
    if (status->n_pairs > capacity) return;
    constexpr int QX = TILE / 8, NQ = QX * QX;
    constexpr int SHIFT = (TILE == 8) ? 3 : (TILE == 16) ? 4 : 5;
    const Place P = place_wave<TILE>(views, n_views, order);
    if (P.gx0 >= P.W || P.gy0 >= P.H) return;
    const int lane = threadIdx.x, row = lane >> 4, li = lane & 15;
    // row r owns the quad (r & 1, r >> 1) of the group
    const int x = P.gx0 + 4 * (row & 1) + (li & 3), y = P.gy0 + 4 * (row >> 1) + (li >> 2);
    const bool valid = x < P.W && y < P.H;
    const float pxf = (float)x, pyf = (float)y;
    const float rn = ray_norm(views[P.v], x, y);
    const uint2 rg = ranges[P.g];
    const int64_t hw = (int64_t)P.W * P.H;
    const float* base = payload + (size_t)P.v * (size_t)n * kRecordWords;
    const uint32_t* offs = offsets + (size_t)P.v * (size_t)n;

    // GB = dL/dC . (colour behind the current step), kept as one running
    // dot product (the colour behind itself is not needed)
    float T = 1.0f, GB = 0.0f, G0 = 0.0f, G1 = 0.0f, G2 = 0.0f;
    int last = (int)rg.x;
    if (valid) {
        const int64_t p = (int64_t)y * P.W + x;
        const int64_t pix = views[P.v].pix_base + p;
        const float* gi = grad_rgb + 3 * views[P.v].pix_base;
        T = out_T[pix];
        // stay inside this tile's list whatever the caller passed
        last = min(max(out_last[pix], (int)rg.x), (int)rg.y);
        G0 = gi[p];
        G1 = gi[hw + p];
        G2 = gi[2 * hw + p];
        // the colour behind starts as T_final bg
        GB = T * (G0 * bg0 + G1 * bg1 + G2 * bg2);
    }
    const uint32_t walk_end = (uint32_t)wave_max_int(last);
    // each row's end: the largest last blended position of its 16 pixels
    int rlast = last;
#pragma unroll
    for (int m = 8; m >= 1; m >>= 1) rlast = max(rlast, __shfl_xor(rlast, m, 16));
    const uint32_t rend[4] = {(uint32_t)__builtin_amdgcn_readlane(rlast, 0),
                              (uint32_t)__builtin_amdgcn_readlane(rlast, 16),
                              (uint32_t)__builtin_amdgcn_readlane(rlast, 32),
                              (uint32_t)__builtin_amdgcn_readlane(rlast, 48)};

    // zero records of the entries that meet the group but no pixel reached
    for (uint32_t e0 = walk_end; e0 < rg.y; e0 += 64) {
        const Batch bt = load_batch<NQ>(base, vals, offs, e0, min(64u, rg.y - e0), P.gx0, P.gy0, SHIFT, P.tx,
                                              P.ty, P.q);
        uint64_t mask = bt.mask;
        while (mask) {
            const int b = __builtin_ctzll(mask);
            mask &= mask - 1;
            const uint32_t slot = (uint32_t)__builtin_amdgcn_readlane((int)bt.off, b);
            if (lane < kGradWords) grads[(size_t)slot * kGradWords + lane] = 0.0f;
        }
    }

    // the last record: one no pixel lies in, for a row without an entry
    if (lane < 8) srec[kBwdBatch][lane] = (lane == 1) ? make_float4(0.f, 0.f, -1.f, -1.f) : make_float4(0.f, 0.f, 0.f, 1.f);
    const float2* words = reinterpret_cast<const float2*>(srec[0]) + li;
    for (uint32_t e_hi = walk_end; e_hi > rg.x;) {
        const uint32_t nb = min((uint32_t)kBwdBatch, e_hi - rg.x);
        const uint32_t e0 = e_hi - nb;
        e_hi = e0;
        // lane l < nb stages entry e0 + l: its record, a zero accumulator, and
        // the quads whose row walks it
        bool meets = false;
        uint32_t qm = 0, off = 0;
        if ((uint32_t)lane < nb) {
            const uint32_t idx = vals[e0 + lane];
            const float* rp = base + (size_t)idx * kRecordWords;
            const int4 r = *reinterpret_cast<const int4*>(rp);
            meets = (NQ == 1) || rect_meets_group(r, P.gx0, P.gy0);
            if (meets) {
                off = record_index(r, SHIFT, P.tx, P.ty, offs[idx], NQ, P.q);
                const float4* src = reinterpret_cast<const float4*>(rp + 4);
#pragma unroll
                for (int k = 0; k < 7; ++k) srec[lane][k] = src[k];
                float4* acc4 = reinterpret_cast<float4*>(sacc[lane]);
#pragma unroll
                for (int k = 0; k < kGradWords / 4; ++k) acc4[k] = make_float4(0.f, 0.f, 0.f, 0.f);
                const uint32_t e = e0 + (uint32_t)lane;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int qx0 = P.gx0 + 4 * (q & 1), qy0 = P.gy0 + 4 * (q >> 1);
                    const bool mq = !(r.x > qx0 + 3 || r.z < qx0 || r.y > qy0 + 3 || r.w < qy0);
                    qm |= (mq && e < rend[q]) ? (1u << q) : 0u;
                }
            }
        }
        const uint32_t staged = (uint32_t)__ballot(meets);   // kBwdBatch <= 32 entries
        if (staged == 0) continue;
        const uint32_t m0 = (uint32_t)__ballot(qm & 1u), m1 = (uint32_t)__ballot(qm & 2u),
                       m2 = (uint32_t)__ballot(qm & 4u), m3 = (uint32_t)__ballot(qm & 8u);
        uint32_t mask = (row == 0) ? m0 : (row == 1) ? m1 : (row == 2) ? m2 : m3;
        lds_hand_over();   // rows read, and add to, what other lanes staged
        while (true) {
            const bool act = mask != 0;
            if (__ballot(act) == 0) break;
            // the row's next entry, in reverse order (a row without one runs
            // the step with every lane outside)
            const int bcur = act ? 31 - __builtin_clz(mask) : kBwdBatch;
            mask &= act ? ~(1u << bcur) : ~0u;
            const float2 w = words[bcur * 16];
            const uint32_t e = e0 + (uint32_t)bcur;
            float acc[kGradWords];
            const bool contributed = bwd_step_exact<KIND>(w, act && (int)e < last, pxf, pyf, rn, G0, G1, G2, T, GB, acc);
            if (__ballot(contributed) != 0) {
                float t0, t1;
                int w0, w1;
                row_reduce20(acc, li, t0, t1, w0, w1);
                // the rows one after the other: a fixed order of the additions
#pragma unroll
                for (int rr = 0; rr < 4; ++rr) {
                    if (row == rr && act) {
                        if (w0 >= 0) atomicAdd(&sacc[bcur][w0], t0);
                        if (w1 >= 0) atomicAdd(&sacc[bcur][w1], t1);
                    }
                }
            }
        }
        lds_hand_over();
        // the batch's records, one per lane
        if (meets) {
            const float4* acc4 = reinterpret_cast<const float4*>(sacc[lane]);
            float4* dst = reinterpret_cast<float4*>(grads + (size_t)off * kGradWords);
#pragma unroll
            for (int k = 0; k < kGradWords / 4; ++k) dst[k] = acc4[k];
        }
        lds_hand_over();
    }
}

// ---------------------------------------------------------------------------
// Launchers.
// ---------------------------------------------------------------------------
template <int TILE>
static dim3 wave_grid(const ViewLayout& L) {
    constexpr int NQ = (TILE / 8) * (TILE / 8);
    return dim3((unsigned)(L.n_tiles_total * NQ));
}

template <int TILE, int KIND, bool EXACT>
static void fwd_dispatch(bool count, const ViewLayout& Lv, hipStream_t s, const ViewInfo* views, int nv, int64_t n,
                         const float* payload, const uint32_t* vals, const uint2* ranges, const Status* st,
                         uint64_t cap, const float bg[3], float* rgb, float* T, int32_t* last,
                         unsigned long long* counters, const float* means, float* depth, const uint32_t* order) {
    const dim3 grid = wave_grid<TILE>(Lv);
#define LP_K(C_, D_)                                                                                              \
    hipLaunchKernelGGL((k_render_fwd<TILE, KIND, C_, EXACT, D_>), grid, dim3(64), 0, s, views, nv, n, payload, vals, \
                       ranges, st, cap, bg[0], bg[1], bg[2], rgb, T, last, counters, means, depth, order)
    if (depth) {
        if (count) LP_K(true, true); else LP_K(false, true);
    } else {
        if (count) LP_K(true, false); else LP_K(false, false);
    }
#undef LP_K
}

hipError_t launch_render_fwd_ex(const ViewLayout& L, const char* vws, const PairLayout& P, const char* pws,
                                int result_in_b, int type, bool exact, int tile, int32_t n_views, const float bg[3],
                                float* out_rgb, float* out_T, int32_t* out_last, float* out_depth,
                                const float* means, unsigned long long* counters, hipStream_t stream) {
    if (L.n_tiles_total == 0) return hipSuccess;
    const ViewInfo* views = reinterpret_cast<const ViewInfo*>(vws + L.views);
    const float* payload = reinterpret_cast<const float*>(vws + L.payload);
    const uint32_t* vals = reinterpret_cast<const uint32_t*>(pws + (result_in_b ? P.vals_b : P.vals_a));
    const uint2* ranges = reinterpret_cast<const uint2*>(vws + L.ranges);
    const Status* st = reinterpret_cast<const Status*>(vws + L.status);
    // the exact variant's heavier step runs best in the backward's order
    const uint32_t* order = reinterpret_cast<const uint32_t*>(vws + (exact ? L.order_bwd : L.order));
    const uint64_t cap = (uint64_t)P.capacity;
    const bool count = counters != nullptr;
#define LP_FWD(T_, K_, E_) fwd_dispatch<T_, K_, E_>(count, L, stream, views, n_views, L.n, payload, vals, ranges, st, \
                                                    cap, bg, out_rgb, out_T, out_last, counters, means, out_depth, order)
#define LP_FWD_T(K_, E_)                                                       \
    do {                                                                       \
        if (tile == 8) LP_FWD(8, K_, E_);                                      \
        else if (tile == 16) LP_FWD(16, K_, E_);                               \
        else LP_FWD(32, K_, E_);                                               \
    } while (0)
    if (type == LINPRIM_OCTAHEDRON) {
        if (exact) LP_FWD_T(0, true); else LP_FWD_T(0, false);
    } else {
        if (exact) LP_FWD_T(1, true); else LP_FWD_T(1, false);
    }
#undef LP_FWD_T
#undef LP_FWD
    return hipGetLastError();
}

hipError_t launch_render_fwd(const ViewLayout& L, const char* vws, const PairLayout& P, const char* pws,
                             int result_in_b, int type, bool exact, int tile, int32_t n_views, const float bg[3],
                             float* out_rgb, float* out_T, int32_t* out_last, hipStream_t stream) {
    return launch_render_fwd_ex(L, vws, P, pws, result_in_b, type, exact, tile, n_views, bg, out_rgb, out_T, out_last,
                                nullptr, nullptr, nullptr, stream);
}

template <int TILE, int KIND, bool EXACT>
static void bwd_dispatch(const ViewLayout& Lv, hipStream_t s, const ViewInfo* views, int nv, int64_t n,
                         const float* payload, const uint32_t* vals, const uint2* ranges, const uint32_t* offsets,
                         const Status* st, uint64_t cap, const float bg[3], const float* T, const int32_t* last,
                         const float* grad, float* grads, const uint32_t* order) {
    if (EXACT)
        hipLaunchKernelGGL((k_render_bwd_rows<TILE, KIND>), wave_grid<TILE>(Lv), dim3(64), 0, s, views, nv, n,
                           payload, vals, ranges, offsets, st, cap, bg[0], bg[1], bg[2], T, last, grad, grads, order);
    else
        hipLaunchKernelGGL((k_render_bwd<TILE, KIND>), wave_grid<TILE>(Lv), dim3(64), 0, s, views, nv, n,
                           payload, vals, ranges, offsets, st, cap, bg[0], bg[1], bg[2], T, last, grad, grads, order);
}

hipError_t launch_render_bwd(const ViewLayout& L, const char* vws, const PairLayout& P, char* pws, int result_in_b,
                             int type, bool exact, int tile, int32_t n_views, const float bg[3], const float* out_T,
                             const int32_t* out_last, const float* grad_rgb, hipStream_t stream) {
    if (L.n_tiles_total == 0) return hipSuccess;
    const ViewInfo* views = reinterpret_cast<const ViewInfo*>(vws + L.views);
    const float* payload = reinterpret_cast<const float*>(vws + L.payload);
    const uint32_t* vals = reinterpret_cast<const uint32_t*>(pws + (result_in_b ? P.vals_b : P.vals_a));
    const uint2* ranges = reinterpret_cast<const uint2*>(vws + L.ranges);
    const uint32_t* offsets = reinterpret_cast<const uint32_t*>(vws + L.offsets);
    const Status* st = reinterpret_cast<const Status*>(vws + L.status);
    float* grads = reinterpret_cast<float*>(pws + P.grads);
    const uint32_t* order = reinterpret_cast<const uint32_t*>(vws + L.order_bwd);
    const uint64_t cap = (uint64_t)P.capacity;
#define LP_BWD(T_, K_, E_) bwd_dispatch<T_, K_, E_>(L, stream, views, n_views, L.n, payload, vals, ranges, offsets, \
                                                    st, cap, bg, out_T, out_last, grad_rgb, grads, order)
#define LP_BWD_T(K_, E_)                                                       \
    do {                                                                       \
        if (tile == 8) LP_BWD(8, K_, E_);                                      \
        else if (tile == 16) LP_BWD(16, K_, E_);                               \
        else LP_BWD(32, K_, E_);                                               \
    } while (0)
    if (type == LINPRIM_OCTAHEDRON) {
        if (exact) LP_BWD_T(0, true); else LP_BWD_T(0, false);
    } else {
        if (exact) LP_BWD_T(1, true); else LP_BWD_T(1, false);
    }
#undef LP_BWD_T
#undef LP_BWD
    return hipGetLastError();
}

}  // namespace linprim
