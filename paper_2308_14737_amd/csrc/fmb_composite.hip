// fmb_composite.hip -- gfx950 kernels of the zero-parameter Fuzzy Metaballs renderer
// (alpha compositing, Keselman & Hebert, WACV 2024, Sec. 3.3, Eq. 9-10).
//
// Weights: w_i = T_i (1 - exp(-delta_i)), T_i = exp(-sum_j delta_j [t_j < t_i]), blended by
// Eq. (3) for depth, normals and colour; alpha is Eq. (8) as in the two-parameter model.  The
// weights enter Eq. (3) as base-2 logarithms,
//   log2 w_i = -log2(e) F_i + log2(1 - exp(-delta_i)),   F_i = sum_{t_j < t_i} delta_j,
// normalised by their running maximum like the two-parameter weights, so rays far from every
// Gaussian keep finite weights.  The strict inequality is taken literally: intersections at
// equal depth do not attenuate one another.
//
// Layout: one ray per lane, one 8 x 8 pixel tile (ViewRec's ray tiles) per wave; an item is a run of
// consecutive tiles of one view.  A scene of at most kCompTG Gaussians is staged in LDS once per item
// and block for four waves, which take the item's tiles in turn (one wave per block staged it for itself
// and left a 20-view 128 x 128 job at 320 waves: 960 -> 196 us for its step).  Of a larger scene each
// wave first bounds every Gaussian on its tile and stages those that can matter there (about 10 of 1000 on
// a clustered 480 x 270 view: a render of 13.3 ms, and 0.8 before a tile was cut over several waves); only a tile with more than kCompTG of them takes the
// scene in staged tiles.
//
// Front sums without a sort: F_i only needs the densities in front of t_i, and of those only the
// significant ones (density above 2^sig, comp_sig_log2: the rest total below 2^-36, below FP32's
// rounding of T_i).  A lane keeps its ray's significant intersections, with their depths, in
// registers and forms F_i as a sum of exact 0/1 steps over them: per pair the cost is the count of
// significant intersections around the tile (about ten on the benchmark scenes), not N.  Slots are
// filled in Gaussian order at positions uniform over the wave -- a lane for which the slot's
// Gaussian is not significant leaves density 0 there -- so that filling a slot is a register move
// and the step sums run a count uniform over the wave.
//
// Depth windows: a pass fills at most kCompSlots slots.  When more Gaussians are significant for
// the tile, a lane that meets one more than the slots hold records the nearest such depth, and the
// pass covers only the depths in front of it: the lane's window [lo, hi).  The next pass starts at
// hi, with the window's densities (and those at its lower edge, which do not attenuate one another)
// added to the lane's base sum.  Every pair is blended in the window that holds its depth.  Almost
// every tile of the benchmark scenes takes one window; a tile whose rays pass hundreds of Gaussians
// takes several, so the renderer takes any N.
//
// Backward (same layout): with z_i = log w_i and z_bar_i = wt_i (lin_i - kappa) the softmax
// adjoint (wt_i the normalised weight, lin_i the pair's share of the cotangents), delta_j enters
// z_i of every pair behind it, so
//   d_bar(log delta_j) = z_bar_j delta_j / expm1(delta_j) + delta_j (D_bar - B_j),
//   B_j = sum_{t_i > t_j} z_bar_i,   t_bar_j = wt_j tf_bar,
// and the rest is the two-parameter renderer's per-pair adjoint.  B_j is summed over the
// significant intersections (one pass over the slots' Gaussians forms their z_bar), by the same
// step sums; across windows the z_bar of the windows behind come from a first sweep.  The pairs
// left out carry normalised weights below 2^-24 of the ray's largest, and delta_j B_j is itself
// below 2^-24 of z_bar_j where every density of the ray is insignificant.  Each wave sums its pairs'
// terms over its 64 rays for every Gaussian it touches (a fixed butterfly), adds them to the item's
// record in LDS in tile order, and the records go to the deterministic finalize.
#include "fmb_device.h"

namespace fmb {

constexpr int kCompSlots = 48;  // significant intersections a lane holds per depth window
constexpr int kCompTG = 128;    // Gaussians staged per LDS tile
// Waves per SIMD the kernels are compiled for: the slots take 2 (forward) or 3 VGPRs each.  The
// forward of small scenes is held to three waves (168 VGPRs, some values spilled to scratch, within
// what the runtime keeps allocated); the others keep two and do not spill: spills above 267 bytes a lane make the runtime
// allocate scratch for every launch, which cost 0.5 ms.
constexpr int kBwdcWaves = 2, kStatcWaves = 2;
__host__ __device__ constexpr int fwdc_waves(int nw) { return nw > 1 ? 3 : 2; }

// log2(1 - exp(-delta)) with log2(delta) = d2.
__device__ __forceinline__ float log2_opacity(float delta, float d2)
{
    const float series = fmaf((float)kLog2e * delta, fmaf(delta, fmaf(delta * delta, -1.0f / 2880.0f, 1.0f / 24.0f), -0.5f), d2);
    const float direct = __builtin_amdgcn_logf(1.0f - exp2_(-(float)kLog2e * delta));
    return delta < 0.0625f ? series : direct;
}

// delta / expm1(delta) = d log(1 - exp(-delta)) / d log(delta).
__device__ __forceinline__ float opacity_slope(float delta)
{
    const float series = fmaf(delta, fmaf(delta, fmaf(delta * delta, -1.0f / 720.0f, 1.0f / 12.0f), -0.5f), 1.0f);
    const float em = exp2_(-(float)kLog2e * delta);
    const float direct = delta * em * rcp_(1.0f - em);
    return delta < 0.0625f ? series : direct;
}

// Depths are kept and compared scaled by 2^100: clamp(b - a, 0, 1) of two scaled depths is 1
// exactly when a < b and 0 when a >= b, for every pair of depths below 2^27 in magnitude whose
// difference is at least 2^-100, i.e. any two distinct depths this renderer meets.
constexpr float kDepthScale = 0x1p100f;

__device__ __forceinline__ float before(float a, float b) { return __builtin_amdgcn_fmed3f(b - a, 0.0f, 1.0f); }

// Base-2 log of the smallest significant density of a scene of n Gaussians: the densities left
// out of a front sum total less than n 2^sig <= 2^-36 (and 2^sig <= 2^-30).
__device__ __forceinline__ float comp_sig_log2(int n)
{
    const int lg = n > 1 ? 32 - __clz(n - 1) : 0;  // ceil(log2 n)
    return fminf(-30.0f, -36.0f - (float)lg);
}

// A ray whose largest base-2 log weight is at least this takes only its significant pairs: the
// others weigh less than n 2^sig <= 2^-36 together, below 2^-24 of its sum of weights.
constexpr float kCompHitLog2 = -12.0f;

// Base-2 log of the smallest normalised weight (and density) whose pair terms are evaluated: the
// weights of Eq. (9) fall off only as fast as the densities, so pairs far from a ray keep weights far
// above FP32's zero, but all pairs below 2^skip together move a ray's sums by less than
// n 2^skip <= 2^-26 of their value (and 2^skip <= 2^-40).
__device__ __forceinline__ float comp_skip_log2(int n)
{
    const int lg = n > 1 ? 32 - __clz(n - 1) : 0;  // ceil(log2 n)
    return fminf(-40.0f, -26.0f - (float)lg);
}

// The same cutoff relative to a lower bound of a ray's largest log2 density (or 0 above it): a ray of
// density sum D has a sum of weights of at least 1 - exp(-D) >= 0.63 min(1, D), so its largest weight
// is at least 2^-0.67 / n of min(1, D).  Pairs below this on every ray of a tile are pairs that each ray's
// own test against its running maximum would leave out, or whose terms a later, larger weight would
// scale below the sums' rounding.
__device__ __forceinline__ float comp_blend_log2(int n) { return comp_skip_log2(n) - 1.0f - ceil_log2(n); }

// A lane's slots: scaled depth and density of the significant intersection of the slot's
// Gaussian (density 0 where that Gaussian is not significant for the lane, or not in its window).
// They are register vectors (slots 0..31 in the first, 32..47 in the second), read at
// compile-time positions and written at the wave-uniform fill position by one indirect register
// move; slot k holds the window's k-th Gaussian in staging order, and the slots from ns on hold
// zeros.
typedef float CompV32 __attribute__((ext_vector_type(32)));
typedef float CompV16 __attribute__((ext_vector_type(16)));
static_assert(kCompSlots == 48, "the slot vectors hold 32 + 16 slots");
struct CompList {
    CompV32 t0, d0;
    CompV16 t1, d1;
};
// a value per slot (the backward's z_bar of the slots' pairs)
struct CompZ {
    CompV32 z0;
    CompV16 z1;
};

__device__ __forceinline__ float slot_t(const CompList &L, int k) { return k < 32 ? L.t0[k] : L.t1[k - 32]; }
__device__ __forceinline__ float slot_d(const CompList &L, int k) { return k < 32 ? L.d0[k] : L.d1[k - 32]; }
__device__ __forceinline__ float slot_z(const CompZ &z, int k) { return k < 32 ? z.z0[k] : z.z1[k - 32]; }

__device__ __forceinline__ void slot_set_d(CompList &L, int k, float d)
{
    if (k < 32)
        L.d0[k] = d;
    else
        L.d1[k - 32] = d;
}

__device__ __forceinline__ void slot_set(CompList &L, int k, float t, float d)
{
    if (k < 32) {
        L.t0[k] = t;
        L.d0[k] = d;
    } else {
        L.t1[k - 32] = t;
        L.d1[k - 32] = d;
    }
}

__device__ __forceinline__ void slot_set_z(CompZ &z, int k, float v)
{
    if (k < 32)
        z.z0[k] = v;
    else
        z.z1[k - 32] = v;
}

// A lane's depth window (scaled depths): pairs with lo <= t < hi are taken in the current pass;
// base sums the significant densities in front of lo, tie those at lo.
struct CompWin {
    float lo, hi, base, tie;
};

__device__ __forceinline__ void comp_clear(CompList &L)
{
    L.t0 = (CompV32)(0.0f);
    L.d0 = (CompV32)(0.0f);
    L.t1 = (CompV16)(0.0f);
    L.d1 = (CompV16)(0.0f);
}

// Step sums over the slots in use, four slots at a time (template recursion, so that every slot
// index is a compile-time register index); ns is uniform, so the early exits are scalar branches,
// and the unused slots of a group add zeros.  The even and the odd slots go to two sums (two
// independent chains).
constexpr int kSlotGroup = 4;
template <int K>
struct SlotSums {
    // sum of the densities of the slots in front of ts
    __device__ static __forceinline__ void front(const CompList &L, int ns, float ts, float &f, float &g)
    {
        if constexpr (K < kCompSlots) {
            if (K >= ns) return;
#pragma unroll
            for (int k = K; k < K + kSlotGroup; k += 2) {
                f = fmaf(before(slot_t(L, k), ts), slot_d(L, k), f);
                g = fmaf(before(slot_t(L, k + 1), ts), slot_d(L, k + 1), g);
            }
            SlotSums<K + kSlotGroup>::front(L, ns, ts, f, g);
        }
    }
    // sum of z over the slots behind ts
    __device__ static __forceinline__ void behind(const CompList &L, const CompZ &z, int ns, float ts, float &b,
                                                  float &c)
    {
        if constexpr (K < kCompSlots) {
            if (K >= ns) return;
#pragma unroll
            for (int k = K; k < K + kSlotGroup; k += 2) {
                b = fmaf(before(ts, slot_t(L, k)), slot_z(z, k), b);
                c = fmaf(before(ts, slot_t(L, k + 1)), slot_z(z, k + 1), c);
            }
            SlotSums<K + kSlotGroup>::behind(L, z, ns, ts, b, c);
        }
    }
};
static_assert(kCompSlots % kSlotGroup == 0 && kSlotGroup % 2 == 0, "whole slot groups, of pairs");

// F at scaled depth ts inside window w: base, the densities at lo (if ts > lo), and the slots
// in front of ts.
__device__ __forceinline__ float comp_front(const CompList &L, int ns, const CompWin &w, float ts)
{
    float f = ts > w.lo ? w.base + w.tie : w.base, g = 0.0f;
    SlotSums<0>::front(L, ns, ts, f, g);
    return f + g;
}

// Sum of z over the slots behind ts.
__device__ __forceinline__ float comp_behind(const CompList &L, const CompZ &z, int ns, float ts)
{
    float b = 0.0f, c = 0.0f;
    SlotSums<0>::behind(L, z, ns, ts, b, c);
    return b + c;
}

// z_bar of the slots' pairs without a normal or colour cotangent, from the slots alone: the pair's
// weight 2^(lw - M2) / S with lw = -log2(e) F + log2(1 - exp(-delta)) at the slot's depth and
// density, times (tf_bar t - kappa); 0 where the slot is empty for the lane.  A loop over the slots
// in use (each read and written by an indirect register move at the uniform index k) rather than
// one unrolled over every slot: the unrolled form, a front sum per slot, was 70 KB of the adjoint
// kernel's 118 KB of code (same speed on the benchmark scenes).
__device__ __forceinline__ float slot_zf(float f, float dl, float ts, float M2, float invS, float tfb, float kap);

__device__ __forceinline__ float slot_z_plain(const CompList &L, int ns, const CompWin &w, float M2, float invS,
                                              float tfb, float kap, float dl, float ts)
{
    if (!(dl > 0.0f)) return 0.0f;
    return slot_zf(comp_front(L, ns, w, ts), dl, ts, M2, invS, tfb, kap);
}

__device__ __forceinline__ void slots_z_plain(const CompList &L, CompZ &zs, int ns, const CompWin &w, float M2,
                                              float invS, float tfb, float kap)
{
    // (one loop per register vector, so that each writes a single vector in place)
#pragma unroll 1
    for (int k = 0; k < min(ns, 32); ++k)
        zs.z0[k] = slot_z_plain(L, ns, w, M2, invS, tfb, kap, L.d0[k], L.t0[k]);
#pragma unroll 1
    for (int k = 32; k < ns; ++k)
        zs.z1[k - 32] = slot_z_plain(L, ns, w, M2, invS, tfb, kap, L.d1[k - 32], L.t1[k - 32]);
}

// z_bar of a slot's pair from its front sum F, density and depth (0 where the slot is empty); kap is
// kappa less the pair's C_bar . c.
__device__ __forceinline__ float slot_zf(float f, float dl, float ts, float M2, float invS, float tfb, float kap)
{
    if (!(dl > 0.0f)) return 0.0f;
    const float lw = fmaf(-(float)kLog2e, f, log2_opacity(dl, __builtin_amdgcn_logf(dl)));
    return exp2_(lw - M2) * invS * fmaf(tfb, ts * (1.0f / kDepthScale), -kap);
}

// The same z_bar for a tile of one window whose pairs are all slots' (no normal cotangent;
// kap_of(k): kappa less C_bar . c of slot k's Gaussian): first every slot's front sum F into zs,
// then every slot's z_bar into its density register.  The adjoint of such a tile then takes a
// pair's front sum from zs and the sums of z_bar behind it from the density registers: the slots'
// densities are needed only for the front sums, and a second front sum per pair is saved (the
// kernel is bound by instruction issue: with a colour cotangent 141 -> 123 us for 20 views of
// 128 x 128 and 64 Gaussians).
template <class KapOf>
__device__ __forceinline__ void slots_fz_plain(CompList &L, CompZ &zs, int ns, const CompWin &w, float M2,
                                               float invS, float tfb, KapOf kap_of)
{
#pragma unroll 1
    for (int k = 0; k < min(ns, 32); ++k) zs.z0[k] = comp_front(L, ns, w, L.t0[k]);
#pragma unroll 1
    for (int k = 32; k < ns; ++k) zs.z1[k - 32] = comp_front(L, ns, w, L.t1[k - 32]);
#pragma unroll 1
    for (int k = 0; k < min(ns, 32); ++k) L.d0[k] = slot_zf(zs.z0[k], L.d0[k], L.t0[k], M2, invS, tfb, kap_of(k));
#pragma unroll 1
    for (int k = 32; k < ns; ++k)
        L.d1[k - 32] = slot_zf(zs.z1[k - 32], L.d1[k - 32], L.t1[k - 32], M2, invS, tfb, kap_of(k));
}

// The part of an 8 x 8 tile that the lane is in, of 4^cut square ones (cut 1 or 2).  The forward of a
// larger scene gives a dense view's tiles to 4 or 16 waves: a part's rays share fewer Gaussians, so
// that its wave takes fewer windows, and the slowest tile, which the launch waits for, is the sooner
// done (1000 clustered Gaussians at 270 x 480: 792 -> 400 us; at 64 x 64: 2863 -> 388 us).
__device__ __forceinline__ int comp_part(int lane, int cut)
{
    const int half = 3 - cut;
    return ((lane >> (3 + half)) << cut) + ((lane & 7) >> half);
}

// Entries of Gaussians [gb, gb + cnt) of the scene into LDS, EW float4 each: the entry, the terms
// of the m estimate (make_entry_est) and, with EW = 6, the colour.
constexpr int kCompEst = 4, kCompCol = 5;  // float4 offsets within an LDS entry
template <int EW>
__device__ __forceinline__ void comp_entry(const Params &P, int gi, const double o[3], float4 *__restrict__ dst)
{
    make_entry_est(P.means + 3 * gi, P.prec + 6 * gi, P.weights[gi], o, dst);
    if (EW == 6) dst[kCompCol] = colour_entry(P.colors + 3 * gi);
}

template <int EW, int THREADS>
__device__ __forceinline__ void comp_stage(const Params &P, const SceneRec &sr, int gb, int cnt, const double o[3],
                                           float4 *__restrict__ ents)
{
    __syncthreads();  // the previous tile is consumed
    for (int q = threadIdx.x; q < cnt; q += THREADS) comp_entry<EW>(P, sr.gauss_off + gb + q, o, &ents[EW * q]);
    __syncthreads();
}

template <int EW>
__device__ __forceinline__ Ent comp_ent(const float4 *__restrict__ ents, int i)
{
    return ent_from(ents[EW * i], ents[EW * i + 1], ents[EW * i + 2], ents[EW * i + 3]);
}

// The staged Gaussians [0, cnt) of a ray tile: lane j's upper bounds of the log2 densities of
// Gaussians j and 64 + j over the tile (tile_bounds on its box; -inf past cnt) and the least, over the
// tile's rays, of the largest log2 density, from below.
struct CompBounds {
    float hi[2];
    float low;
};

template <int EW>
__device__ __forceinline__ CompBounds comp_bounds(const float4 *__restrict__ ents, int cnt, const TileBox &tb, int lane)
{
    static_assert(kCompTG == 128, "two bounds per lane");
    CompBounds cb{{-INFINITY, -INFINITY}, -INFINITY};
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        const int i = 64 * c + lane;
        if (i < cnt) {
            const PairBounds pb = tile_bounds(comp_ent<EW>(ents, i), ents[EW * i + kCompEst], tb, (float)(-0.5 * kLog2e), 0.0f, 0.0f);
            cb.hi[c] = pb.d2_hi;
            cb.low = fmaxf(cb.low, pb.d2_lo);
        }
    }
    cb.low = wave_max_u(cb.low);
    return cb;
}

// Those whose log2 density can exceed thr, as 64-bit masks (a NaN bound keeps the Gaussian; one of weight 0,
// with a bound of -inf, is dropped also where a ray without any density makes thr -inf).
__device__ __forceinline__ void comp_masks(const CompBounds &cb, int cnt, int lane, float thr, unsigned long long mask[2])
{
#pragma unroll
    for (int c = 0; c < 2; ++c) mask[c] = wave_ballot(64 * c + lane < cnt && !(cb.hi[c] <= thr));
}

// A scene of more than kCompTG Gaussians: those whose log2 density can exceed the cutoff on a ray of the
// tile, staged in scene order with their scene-local indices in gid.  The cutoff is `thr`, or with REL
// (the forward) that or less, `rel` + min(0, the largest lower bound of the tile's log2 densities), bounded
// by the Gaussians seen so far (a superset of the final cutoff's, whose bound is returned in `low`).  The bounds are
// taken on FP32 entries (make_bound_entry); only the survivors' are formed in FP64.  Returns their
// count, which may exceed kCompTG: then the first kCompTG are staged, and the tile takes the scene in
// staged tiles.  One wave.
template <int EW, bool REL>
__device__ __forceinline__ int comp_survivors(const Params &P, const SceneRec &sr, const double o[3], float4 *__restrict__ ents,
                                              int *__restrict__ gid, const TileBox &tb, float thr, float rel, int lane, float &low)
{
    int ne = 0;
    low = -INFINITY;
    __syncthreads();  // the previous tile's entries are consumed
    for (int gb = 0; gb < sr.n; gb += 64) {
        const int gl = gb + lane;
        const bool in = gl < sr.n;
        const int gi = sr.gauss_off + (in ? gl : 0);
        Ent g;
        float4 est;
        make_bound_entry(P.means + 3 * gi, P.prec + 6 * gi, P.weights[gi], o, g, est);
        const PairBounds pb = tile_bounds(g, est, tb, (float)(-0.5 * kLog2e), 0.0f, 0.0f);
        if (REL) low = fmaxf(low, wave_max_u(in ? pb.d2_lo : -INFINITY));
        const bool keep = in && !(pb.d2_hi <= (REL ? fminf(thr, fminf(low, 0.0f) + rel) : thr));
        const unsigned long long bal = wave_ballot(keep);
        const int at = ne + __popcll(bal & ((1ull << lane) - 1ull));
        if (keep && at < kCompTG) gid[at] = gl;
        ne += __popcll(bal);
    }
    __syncthreads();
    for (int q = lane; q < min(ne, kCompTG); q += 64) comp_entry<EW>(P, sr.gauss_off + gid[q], o, &ents[EW * q]);
    __syncthreads();
    return __builtin_amdgcn_readfirstlane(ne);
}

// The slots of window w: every staged Gaussian of `mask` significant for some lane of the wave (log2
// density above sig2), with a depth behind lo for that lane, takes the next slot; the densities at lo
// go to w.tie (and each such pair, whose front sum is w.base, to on_tie(g, q, density, staged index)); a
// lane that meets one more than the slots hold lowers w.hi to its depth.  gb: the scene-local index of
// the first staged Gaussian; slot_g receives gb + the slots' staged indices.
template <int EW, class OnTie>
__device__ __forceinline__ void comp_collect_tile(const float4 *__restrict__ ents, int gb, const unsigned long long mask[2],
                                                  float v0, float v1, float v2, float hm, float sig2, int lane, CompWin &w,
                                                  CompList &L, int &ns, bool &t_inf, int *__restrict__ slot_g, OnTie on_tie)
{
    // the pair's share of the window: tie, slot or (a full list) the end of the window
    auto take = [&](const Ent &g, const Geo &q, int i) {
        const bool sig = q.d2 > sig2;
        const float ts = q.t * kDepthScale;
        const float dl = exp2_(q.d2);
        const bool tie = sig && ts == w.lo;
        if (wave_any(tie)) {
            if (tie) {
                w.tie += dl;
                on_tie(g, q, dl, i);
            }
        }
        const bool cand = sig && ts > w.lo;
        if (!wave_any(cand)) return;
        if (ns < kCompSlots) {
            slot_set(L, ns, ts, cand ? dl : 0.0f);
            t_inf = t_inf || (cand && ts == INFINITY);
            if (lane == 0) slot_g[ns] = gb + i;
            ns = __builtin_amdgcn_readfirstlane(ns + 1);
        } else if (cand) {
            w.hi = fminf(w.hi, ts);
        }
    };
    // two candidates a step, their geometry computed together (two independent chains)
#pragma unroll 1
    for (int c = 0; c < 2; ++c) {
        unsigned long long mk = mask[c];
        while (mk) {
            const int ia = 64 * c + __builtin_ctzll(mk);
            mk &= mk - 1;
            const bool two = mk != 0;
            const int ib = two ? 64 * c + __builtin_ctzll(mk) : ia;
            if (two) mk &= mk - 1;
            const Ent ga = comp_ent<EW>(ents, ia), gb2 = comp_ent<EW>(ents, ib);
            Geo qa, qb;
            pair_geo_coarse(ga, v0, v1, v2, hm, 0.0f, 0.0f, qa);
            pair_geo_coarse(gb2, v0, v1, v2, hm, 0.0f, 0.0f, qb);
            take(ga, qa, ia);
            if (two) take(gb2, qb, ib);
        }
    }
}

// All slots of window w, from the staged Gaussians of `mask` (resident) or the scene's staged tiles;
// slots at or behind w.hi are cleared (they belong to a later window).  Returns the slot count
// (uniform).
template <int EW, class OnTie>
__device__ __forceinline__ int comp_collect(const Params &P, const SceneRec &sr, const double o[3],
                                            float4 *__restrict__ ents, bool resident, const unsigned long long rmask[2],
                                            float v0, float v1, float v2, float hm, float sig2, const TileBox &tb, int lane,
                                            CompWin &w, CompList &L, int *__restrict__ slot_g, OnTie on_tie)
{
    int ns = 0;
    bool t_inf = false;  // a slot of this lane holds an infinite scaled depth
    comp_clear(L);
    for (int gb = 0; gb < (resident ? 1 : sr.n); gb += kCompTG) {
        unsigned long long mask[2] = {rmask[0], rmask[1]};
        if (!resident) {
            const int cnt = min(kCompTG, sr.n - gb);
            comp_stage<EW, 64>(P, sr, gb, cnt, o, ents);
            comp_masks(comp_bounds<EW>(ents, cnt, tb, lane), cnt, lane, sig2, mask);
        }
        comp_collect_tile<EW>(ents, gb, mask, v0, v1, v2, hm, sig2, lane, w, L, ns, t_inf, slot_g, on_tie);
    }
    // (where no lane's window was cut, only a slot at an infinite scaled depth can be at or behind hi)
    if (wave_any(w.hi != INFINITY || t_inf)) {
#pragma unroll
        for (int k = 0; k < kCompSlots; ++k) slot_set_d(L, k, slot_t(L, k) >= w.hi ? 0.0f : slot_d(L, k));
    }
    return ns;
}

// Moves window w past hi (or marks the lane done); returns true while the lane has depths left.
__device__ __forceinline__ bool comp_next(CompWin &w, const CompList &L, int ns)
{
    if (w.hi == INFINITY) {
        w.lo = INFINITY;
        return false;
    }
    float s = w.tie;
#pragma unroll
    for (int k = 0; k < kCompSlots; ++k) s += slot_d(L, k);
    w.base += s;
    w.lo = w.hi;
    w.hi = INFINITY;
    w.tie = 0.0f;
    return true;
}

// ------------------------------------------------------------------------------------
// Forward
// ------------------------------------------------------------------------------------

// NW waves per block: 4 for scenes of at most kCompTG Gaussians (staged once per item for all four, each
// wave taking every fourth tile of it), 1 for larger ones (each wave stages its own tile's survivors).
template <int F, int NW>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(fwdc_waves(NW)))) void fwdc_kernel(
    Params P, FwdOut O, const CompItem *__restrict__ items)
{
    constexpr bool NORMALS = (F & kNrm) != 0, COLOR = (F & kCol) != 0;
    constexpr int EW = COLOR ? 6 : 5;
    __shared__ float4 ents[kCompTG * EW];
    __shared__ int slot_gs[NW][kCompSlots];
    __shared__ int gid[NW == 1 ? kCompTG : 1];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    int *const slot_g = slot_gs[wave];
    const CompItem item = ld_uniform(items + blockIdx.x);
    const ViewRec vr = ld_uniform(P.views + item.view);
    const SceneRec sr = ld_uniform(P.scenes + vr.scene);
    const CamRec cam = cam_of(P, item.view);
    const float *e = cam.e, *kk = cam.k;
    double o[3];
    cam_centre(e, o);
    const float o0 = (float)o[0], o1 = (float)o[1], o2 = (float)o[2];
    const float hm = (float)(-0.5 * kLog2e);
    const float sig2 = comp_sig_log2(sr.n), skip2 = comp_skip_log2(sr.n), blend2 = comp_blend_log2(sr.n);
    if (NW > 1) comp_stage<EW, 64 * NW>(P, sr, 0, sr.n, o, ents);
    const int nt = min(item.span, vr.tiles - item.tile0);

    for (int tt = wave; tt < nt; tt += NW) {
        int row, col;
        const int loc = tile_local(vr, item.tile0 + tt, lane, row, col);
        const bool valid = loc >= 0 && (NW > 1 || item.cut == 0 || comp_part(lane, item.cut) == item.part);
        if (NW == 1 && !wave_any(valid)) continue;  // a part past the edge
        float v0, v1, v2;
        tile_ray_dir(P, vr, e, kk, valid ? loc : 0, valid ? row : 0, valid ? col : 0, v0, v1, v2);
        float at = 0.0f, dt = 0.0f;  // loss targets, loaded ahead of the epilogue
        if (O.g_depth && valid) {
            at = O.alpha_t[vr.ray_off + loc];
            dt = O.depth_t[vr.ray_off + loc];
        }
        const TileBox tc = wave_box(v0, v1, v2, valid, e);
        // the tile's Gaussians: the whole scene, or its survivors, staged (ne of them)
        int ne = sr.n;
        float low = -INFINITY;
        if (NW == 1) ne = comp_survivors<EW, true>(P, sr, o, ents, gid, tc, sig2, blend2, lane, low);
        const bool resident = NW > 1 || ne <= kCompTG;
        // the staged Gaussians that can be significant on the tile, and those that can reach the blend
        CompBounds cb{{0.0f, 0.0f}, low};
        if (resident) cb = comp_bounds<EW>(ents, ne, tc, lane);
        const float rel = fminf(cb.low, 0.0f) + blend2;
        unsigned long long smask[2] = {0, 0};
        if (resident) comp_masks(cb, ne, lane, sig2, smask);
        float M, S, T, N0, N1, N2, C0, C1, C2, D;
        auto reset = [&]() {
            M = -INFINITY;
            S = T = N0 = N1 = N2 = C0 = C1 = C2 = D = 0.0f;
        };
        reset();
        CompWin w{valid ? -INFINITY : INFINITY, INFINITY, 0.0f, 0.0f};
        CompList L;
        // blends pair (g, q) of this lane at front sum fs; ci: the staged index of its colour
        auto blend = [&](const Ent &g, Geo &q, float fs, int ci) {
            const float delta = exp2_(q.d2);
            D += delta;
            const float lw = fmaf(-(float)kLog2e, fs, log2_opacity(delta, q.d2));
            if (lw > M) {  // new running maximum: rescale the sums
                const float sc = exp2_(M - lw);
                S *= sc;
                T *= sc;
                N0 *= sc;
                N1 *= sc;
                N2 *= sc;
                C0 *= sc;
                C1 *= sc;
                C2 *= sc;
                M = lw;
            }
            const float ew = exp2_(lw - M);
            S += ew;
            T = fmaf(ew, q.t, T);
            if (NORMALS) {
                pair_refine(q);
                const PairNormal pn = pair_normal(g, q, 0.0f, 0.0f, 0.0f);
                N0 = fmaf(ew, pn.n0, N0);
                N1 = fmaf(ew, pn.n1, N1);
                N2 = fmaf(ew, pn.n2, N2);
            }
            if (COLOR) {
                const float4 cc = ents[EW * ci + kCompCol];
                C0 = fmaf(ew, cc.x, C0);
                C1 = fmaf(ew, cc.y, C1);
                C2 = fmaf(ew, cc.z, C2);
            }
        };
        const auto no_tie = [](const Ent &, const Geo &, float, int) {};
        int ns = comp_collect<EW>(P, sr, o, ents, resident, smask, v0, v1, v2, hm, sig2, tc, lane, w, L, slot_g, no_tie);

        // A tile of one window whose rays all weigh at least 2^kCompHitLog2 somewhere blends only the
        // significant pairs (the slots' Gaussians), each ray its own.  The weights are kept as logarithms and
        // added in scene order in every tile, whatever the cut of the work: the sign of an L1 loss
        // follows the last bit of a depth or colour.
        bool done = false;
        // (a ray whose densities are all below that cannot qualify: a weight is at most its density)
        float most = 0.0f;
#pragma unroll
        for (int k = 0; k < kCompSlots; ++k) most = fmaxf(most, slot_d(L, k));
        if (resident && ns > 0 && !wave_any(w.hi != INFINITY) && wave_all(!valid || most > 0x1.fp-13f)) {
            for (int s = 0; s < ns; s += 2) {  // two slots a step (two independent chains)
                const bool two = s + 1 < ns;
                const int ia = slot_g[s], ib = two ? slot_g[s + 1] : ia;
                const Ent ga = comp_ent<EW>(ents, ia), gb = comp_ent<EW>(ents, ib);
                Geo qa, qb;
                pair_geo_coarse(ga, v0, v1, v2, hm, 0.0f, 0.0f, qa);
                pair_geo_coarse(gb, v0, v1, v2, hm, 0.0f, 0.0f, qb);
                if (valid && qa.d2 > sig2) blend(ga, qa, comp_front(L, ns, w, qa.t * kDepthScale), ia);
                if (two && valid && qb.d2 > sig2) blend(gb, qb, comp_front(L, ns, w, qb.t * kDepthScale), ib);
            }
            done = wave_all(!valid || M >= kCompHitLog2);
            if (!done) reset();
        }
        // Otherwise every pair of every window (a tile that sees background or several windows).
        while (!done) {
            for (int gb = 0; gb < (resident ? 1 : sr.n); gb += kCompTG) {
                const int cnt = resident ? ne : min(kCompTG, sr.n - gb);
                if (!resident) {
                    comp_stage<EW, 64>(P, sr, gb, cnt, o, ents);
                    cb = comp_bounds<EW>(ents, cnt, tc, lane);
                }
                unsigned long long mask[2];
                comp_masks(cb, cnt, lane, rel, mask);
#pragma unroll 1
                for (int c = 0; c < 2; ++c) {
                    unsigned long long mk = mask[c];
                    while (mk) {  // two Gaussians a step (two independent chains)
                        const int ia = 64 * c + __builtin_ctzll(mk);
                        mk &= mk - 1;
                        const bool two = mk != 0;
                        const int ib = two ? 64 * c + __builtin_ctzll(mk) : ia;
                        if (two) mk &= mk - 1;
                        const Ent ga = comp_ent<EW>(ents, ia), gb2 = comp_ent<EW>(ents, ib);
                        Geo qa, qb;
                        pair_geo_coarse(ga, v0, v1, v2, hm, 0.0f, 0.0f, qa);
                        pair_geo_coarse(gb2, v0, v1, v2, hm, 0.0f, 0.0f, qb);
                        // a pair of this window whose weight (at most its density) is not below
                        // 2^skip2 of the running maximum
                        const float tsa = qa.t * kDepthScale, tsb = qb.t * kDepthScale;
                        const bool la = tsa >= w.lo && tsa < w.hi && qa.d2 - M >= skip2;
                        if (wave_any(la) && la) blend(ga, qa, comp_front(L, ns, w, tsa), ia);
                        const bool lb = two && tsb >= w.lo && tsb < w.hi && qb.d2 - M >= skip2;
                        if (wave_any(lb) && lb) blend(gb2, qb, comp_front(L, ns, w, tsb), ib);
                    }
                }
            }
            const bool more = comp_next(w, L, ns);
            if (!wave_any(more)) break;
            ns = comp_collect<EW>(P, sr, o, ents, resident, smask, v0, v1, v2, hm, sig2, tc, lane, w, L, slot_g, no_tie);
        }
        if (valid)
            write_ray<F>(P, O, item.view, vr.ray_off + loc, e, kk, o0, o1, o2, v0, v1, v2, M, S, T, N0, N1, N2, C0,
                         C1, C2, D, at, dt);
    }
}

// ------------------------------------------------------------------------------------
// Backward
// ------------------------------------------------------------------------------------

// NW waves per block as in the forward: with 4, the waves share the staged scene and each sums its
// tiles' terms into its own record, added in wave order at the end of the item.
template <int F, int NW>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(kBwdcWaves))) void bwdc_kernel(
    Params P, BwdIn I, const BwdItem *__restrict__ items, const int *__restrict__ order, float *__restrict__ partial,
    float *__restrict__ beta_partial)
{
    constexpr bool NORMALS = (F & kNrm) != 0, COLOR = (F & kCol) != 0;
    // without a normal cotangent the pairs take the offset form of the adjoint
    // (pair_adjoint_offset), which needs neither the refined peak nor r
    constexpr bool PLAIN = !NORMALS;
    constexpr int EW = COLOR ? 6 : 5;
    constexpr int REC = COLOR ? kPartialColor : kPartial;   // partial record per Gaussian
    // the sums per Gaussian: (H, Bv, L) of the offset form or the general record, then colour
    constexpr int LREC = (PLAIN ? kOffsetAcc : kPartial) + (COLOR ? 3 : 0);
    static_assert(LREC <= 16, "one 16-value wave sum per pair");
    __shared__ float4 ents[kCompTG * EW];
    // the slots' entries, for scenes beyond one LDS tile (dynamic: the four-wave form, whose scenes are
    // all resident, is launched without it)
    extern __shared__ float4 sents[];
    __shared__ float recs[NW][kCompTG * LREC];  // each wave's sums of the staged Gaussians
    __shared__ int slot_gs[NW][kCompSlots];
    __shared__ int touched[NW == 1 ? kCompTG : 1];
    __shared__ int gid[NW == 1 ? kCompTG : 1];  // scene-local indices of a tile's survivors
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    int *const slot_g = slot_gs[wave];
    float *const rec = recs[wave];
    const int it = order ? ld_uniform(order + blockIdx.x) : (int)blockIdx.x;
    const BwdItem item = ld_uniform(items + it);
    const ViewRec vr = ld_uniform(P.views + item.view);
    const SceneRec sr = ld_uniform(P.scenes + vr.scene);
    const CamRec cam = cam_of(P, item.view);
    const float *e = cam.e, *kk = cam.k;
    double o[3];
    cam_centre(e, o);
    const float o0 = (float)o[0], o1 = (float)o[1], o2 = (float)o[2];
    const float hm = (float)(-0.5 * kLog2e);
    const float sig2 = comp_sig_log2(sr.n), skip2 = comp_skip_log2(sr.n);
    const int n = sr.n;
    float *__restrict__ prec_out = partial + item.poff;
    if (NW > 1) {
        for (int q = lane; q < n * LREC; q += 64) rec[q] = 0.0f;
        comp_stage<EW, 64 * NW>(P, sr, 0, n, o, ents);
    } else {
        // the record is summed in place over the item's tiles and windows, one staged tile at a time
        for (int q = lane; q < n * REC; q += 64) prec_out[q] = 0.0f;
        __syncthreads();
    }
    const int nt = min(item.span, vr.tiles - item.ray0);

    for (int tt = wave; tt < nt; tt += NW) {
        int row, col;
        const int loc = tile_local(vr, item.ray0 + tt, lane, row, col);
        const bool valid = loc >= 0;
        float4 pr[4];
        ray_prologue<F>(P, I, item.view, vr, e, kk, o0, o1, o2, valid ? loc : 0, valid, 0.0f, 0.0f, pr, valid ? row : 0,
                        valid ? col : 0);
        const float v0 = pr[0].x, v1 = pr[0].y, v2 = pr[0].z, M2 = pr[0].w;
        const float invS = pr[1].x, tfb = pr[1].y, nb0 = pr[1].z, nb1 = pr[1].w;
        const float nb2 = pr[2].x, kap = pr[2].y, Db = pr[2].z;
        const float cb0 = pr[3].x, cb1 = pr[3].y, cb2 = pr[3].z;
        // a normalised weight 2^(lw - M2) / S is below 2^skip2 where lw < M2 + log2 S + skip2,
        // and lw is at most the log2 density
        const float wskip = valid ? M2 - __builtin_amdgcn_logf(invS) + skip2 : INFINITY;
        // the least cutoff of the wave's rays (pairs below a ray's cutoff are not taken)
        const float lim = fminf(skip2, wskip), lim_min = wave_min_u(valid ? lim : INFINITY);
        const CompWin w0{valid ? -INFINITY : INFINITY, INFINITY, 0.0f, 0.0f};
        CompWin w = w0;
        CompList L;
        CompZ zs;
        const TileBox tc = wave_box(v0, v1, v2, valid, e);
        // the tile's Gaussians: the whole scene, or its survivors, staged (ne of them)
        int ne = n;
        float low;
        if (NW == 1) ne = comp_survivors<EW, false>(P, sr, o, ents, gid, tc, fminf(sig2, lim_min), 0.0f, lane, low);
        const bool resident = NW > 1 || ne <= kCompTG;
        const bool mapped = NW == 1 && resident;  // the staged Gaussians' records are flushed per tile
        unsigned long long smask[2] = {0, 0}, fmask[2] = {0, 0};
        if (resident) {
            const CompBounds cb = comp_bounds<EW>(ents, ne, tc, lane);
            comp_masks(cb, ne, lane, sig2, smask);
            comp_masks(cb, ne, lane, lim_min, fmask);
        }
        if (mapped) {
            for (int q = lane; q < ne * LREC; q += 64) rec[q] = 0.0f;
            for (int q = lane; q < ne; q += 64) touched[q] = 0;
            __syncthreads();
        }

        // z_bar of the slots' own pairs (the lanes' significant intersections of the window)
        auto slots_z = [&](int ns) {
            zs.z0 = (CompV32)(0.0f);
            zs.z1 = (CompV16)(0.0f);
            if (PLAIN && !COLOR) {
                // z_bar = wt (tf_bar t - kappa) needs only the slot's depth and density (a colour
                // cotangent adds C_bar . c of the slot's Gaussian: the general form below)
                slots_z_plain(L, zs, ns, w, M2, invS, tfb, kap);
                return;
            }
            if (!resident) {
                __syncthreads();
                if (lane < ns) {
                    const int gi = sr.gauss_off + slot_g[lane];
                    make_entry_est(P.means + 3 * gi, P.prec + 6 * gi, P.weights[gi], o, &sents[EW * lane]);
                    if (COLOR) sents[EW * lane + kCompCol] = colour_entry(P.colors + 3 * gi);
                }
                __syncthreads();
            }
            const float4 *src = resident ? ents : sents;
            // z_bar of the lane's pair (g, q) when the slot holds it: significant and in the window
            auto own_z = [&](const Ent &g, Geo &q, int gs, int k) {
                const float ts = q.t * kDepthScale;
                const bool own = q.d2 > sig2 && ts > w.lo && ts < w.hi;
                float z = 0.0f;
                if (wave_any(own) && own) {
                    const float lw = fmaf(-(float)kLog2e, comp_front(L, ns, w, ts), log2_opacity(exp2_(q.d2), q.d2));
                    const float wt = exp2_(lw - M2) * invS;
                    float lin = tfb * q.t;
                    if (NORMALS) {
                        pair_refine(q);
                        lin += pair_normal(g, q, nb0, nb1, nb2).nN;
                    }
                    if (COLOR) {
                        const float4 cc = src[EW * gs + kCompCol];
                        lin = fmaf(cb0, cc.x, fmaf(cb1, cc.y, fmaf(cb2, cc.z, lin)));
                    }
                    z = wt * (lin - kap);
                }
                slot_set_z(zs, k, z);
            };
            for (int s = 0; s < ns; s += 2) {  // two slots a step (two independent chains)
                const bool two = s + 1 < ns;
                const int ga_i = resident ? slot_g[s] : s;
                const int gb_i = two ? (resident ? slot_g[s + 1] : s + 1) : ga_i;
                const Ent ga = comp_ent<EW>(src, ga_i), gb = comp_ent<EW>(src, gb_i);
                Geo qa, qb;
                pair_geo_coarse(ga, v0, v1, v2, hm, 0.0f, 0.0f, qa);
                pair_geo_coarse(gb, v0, v1, v2, hm, 0.0f, 0.0f, qb);
                own_z(ga, qa, ga_i, s);
                if (two) own_z(gb, qb, gb_i, s + 1);
            }
        };

        // z_bar of the significant pairs at a window's lower edge (the depth where the previous
        // window stopped): they take no slot, and their front sum is the window's base
        float ztie = 0.0f;
        auto on_tie = [&](const Ent &g, const Geo &q0, float dl, int i) {
            Geo q = q0;
            const float lw = fmaf(-(float)kLog2e, w.base, log2_opacity(dl, q.d2));
            const float wt = exp2_(lw - M2) * invS;
            float lin = tfb * q.t;
            if (NORMALS) {
                pair_refine(q);
                lin += pair_normal(g, q, nb0, nb1, nb2).nN;
            }
            if (COLOR) {
                const float4 cc = ents[EW * i + kCompCol];
                lin = fmaf(cb0, cc.x, fmaf(cb1, cc.y, fmaf(cb2, cc.z, lin)));
            }
            ztie = fmaf(wt, lin - kap, ztie);
        };
        // sum of z_bar over the window's significant pairs: the slots' and the lower edge's
        auto window_z = [&](int ns) {
            float s = ztie;
#pragma unroll
            for (int k = 0; k < kCompSlots; ++k) s += slot_z(zs, k);
            return s;
        };

        // First sweep, for tiles that take several windows: the sum of z_bar over all significant
        // intersections of each ray, so that a window knows the z_bar of the windows behind it.
        int ns = comp_collect<EW>(P, sr, o, ents, resident, smask, v0, v1, v2, hm, sig2, tc, lane, w, L, slot_g, on_tie);
        float zall = 0.0f;
        if (wave_any(w.hi != INFINITY)) {
            bool more = true;
            for (;;) {
                slots_z(ns);
                zall += window_z(ns);
                more = comp_next(w, L, ns);
                if (!wave_any(more)) break;
                ztie = 0.0f;
                ns = comp_collect<EW>(P, sr, o, ents, resident, smask, v0, v1, v2, hm, sig2, tc, lane, w, L, slot_g, on_tie);
            }
            w = w0;
            ztie = 0.0f;
            ns = comp_collect<EW>(P, sr, o, ents, resident, smask, v0, v1, v2, hm, sig2, tc, lane, w, L, slot_g, on_tie);
        }

        // A tile of one window whose rays all weigh at least 2^kCompHitLog2 somewhere (the forward's
        // test, on its stashed maximum) takes only the slots' Gaussians, each ray its own pairs.
        const bool hit_tile = resident && ns > 0 && !wave_any(w.hi != INFINITY) && wave_all(!valid || M2 >= kCompHitLog2);

        // Adjoint terms of this lane's pair (g, q) of Gaussian staged at index i (live: the lane
        // has the pair), summed over the wave and added to the Gaussian's sums rec[LREC r ...].
        // With from_slots (a tile of slots_fz_plain) the pair's front sum is fs and z_bar of the
        // slots is in the density registers.
        auto pair_terms = [&](const Ent &g, Geo &q, float ts, bool live, int i, int r, float zafter, bool from_slots,
                              float fs) {
            PairAcc acc;
            OffsetAcc oacc;
            float aC0 = 0.0f, aC1 = 0.0f, aC2 = 0.0f;
            if (live) {
                const float delta = exp2_(q.d2);
                const float lw = fmaf(-(float)kLog2e, from_slots ? fs : comp_front(L, ns, w, ts), log2_opacity(delta, q.d2));
                const float wt = exp2_(lw - M2) * invS;
                PairNormal pn{0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
                if (NORMALS) {
                    pair_refine(q);
                    pn = pair_normal(g, q, nb0, nb1, nb2);
                }
                float lin = fmaf(tfb, q.t, pn.nN);
                if (COLOR) {
                    const float4 cc = ents[EW * i + kCompCol];
                    lin = fmaf(cb0, cc.x, fmaf(cb1, cc.y, fmaf(cb2, cc.z, lin)));
                    aC0 = wt * cb0;
                    aC1 = wt * cb1;
                    aC2 = wt * cb2;
                }
                const float zb = wt * (lin - kap);
                const float bsum = zafter + (from_slots ? comp_behind(L, CompZ{L.d0, L.d1}, ns, ts)
                                                        : comp_behind(L, zs, ns, ts));
                const float db = fmaf(zb, opacity_slope(delta), delta * (Db - bsum));
                const float tb = wt * tfb;
                if (PLAIN)
                    pair_adjoint_offset(q, v0, v1, v2, tb, db, oacc);
                else
                    pair_adjoint<NORMALS>(g, q, v0, v1, v2, wt, pn, nb0, nb1, nb2, tb, db, acc);
            }
            float x[16];
            if (PLAIN) {
                offset_acc_store(oacc, x);
            } else {
                x[0] = acc.u0; x[1] = acc.u1; x[2] = acc.u2; x[3] = acc.u3; x[4] = acc.u4; x[5] = acc.u5;
                x[6] = acc.p0; x[7] = acc.p1; x[8] = acc.p2; x[9] = acc.l;
            }
            constexpr int B0 = PLAIN ? kOffsetAcc : kPartial;
#pragma unroll
            for (int c = B0; c < 16; ++c) x[c] = 0.0f;
            if (COLOR) {
                x[B0] = aC0;
                x[B0 + 1] = aC1;
                x[B0 + 2] = aC2;
            }
            const float tot = wave_sum16(x, lane);
            const int idx = wave16_index(lane);
            if ((lane & 3) == 0 && idx < LREC) rec[LREC * r + idx] += tot;
        };

        // adds the sums of the staged Gaussians that took a term to the item's record (gb: the first one's
        // scene-local index, or -1 for a tile's survivors)
        auto flush = [&](int cnt, int gb) {
            for (int qq = lane; qq < cnt; qq += 64) {
                if (!touched[qq]) continue;
                const int gl = gb >= 0 ? gb + qq : gid[qq];
                const int gg = sr.gauss_off + gl;
                float r[kPartialColor];
                if (PLAIN)
                    write_partial_offset(r, rec + LREC * qq, REC, P.prec + 6 * gg, P.means + 3 * gg, o);
                else
                    write_partial(r, rec + LREC * qq, REC, P.means + 3 * gg, o);
                float *dst = prec_out + REC * gl;
                for (int c = 0; c < REC; ++c) dst[c] += r[c];
            }
        };
        float zthrough = 0.0f;
        for (;;) {
            // (a tile of one window whose pairs are all slots': the slots keep F and z_bar)
            const bool fz = PLAIN && hit_tile;
            if (fz) {
                slots_fz_plain(L, zs, ns, w, M2, invS, tfb, [&](int k) {
                    if (!COLOR) return kap;
                    const float4 cc = ents[EW * slot_g[k] + kCompCol];
                    return kap - fmaf(cb0, cc.x, fmaf(cb1, cc.y, cb2 * cc.z));
                });
            } else {
                slots_z(ns);
                zthrough += window_z(ns);
            }
            // z_bar of the significant intersections behind this window
            const float zafter = w.hi == INFINITY ? 0.0f : zall - zthrough;

            if (hit_tile) {
                for (int s = 0; s < ns; ++s) {
                    const int ia = slot_g[s];
                    const Ent ga = comp_ent<EW>(ents, ia);
                    Geo qa;
                    pair_geo_coarse(ga, v0, v1, v2, hm, 0.0f, 0.0f, qa);
                    // the pair of slot s is the slot's own (its front sum is F of the slot)
                    const float fa = fz ? slot_z(zs, s) : 0.0f;
                    pair_terms(ga, qa, qa.t * kDepthScale, valid && qa.d2 > sig2, ia, ia, zafter, fz, fa);
                    if (mapped && lane == 0) touched[ia] = 1;
                }
            } else {
                for (int gb = 0; gb < (resident ? 1 : n); gb += kCompTG) {
                    const int cnt = min(kCompTG, n - gb);
                    unsigned long long fm[2] = {fmask[0], fmask[1]};
                    if (!resident) {
                        comp_stage<EW, 64>(P, sr, gb, cnt, o, ents);
                        for (int q = lane; q < cnt * LREC; q += 64) rec[q] = 0.0f;
                        for (int q = lane; q < cnt; q += 64) touched[q] = 0;
                        __syncthreads();
                        // only the Gaussians whose density can reach some lane's cutoff on the tile
                        comp_masks(comp_bounds<EW>(ents, cnt, tc, lane), cnt, lane, lim_min, fm);
                    }
#pragma unroll 1
                    for (int c = 0; c < 2; ++c) {
                      unsigned long long mk = fm[c];
                      while (mk) {
                        const int i = 64 * c + __builtin_ctzll(mk);
                        mk &= mk - 1;
                        const Ent ga = comp_ent<EW>(ents, i);
                        Geo qa;
                        pair_geo_coarse(ga, v0, v1, v2, hm, 0.0f, 0.0f, qa);
                        // a pair of this window with a normalised weight or a density not below 2^skip2
                        const float tsa = qa.t * kDepthScale;
                        const bool la = tsa >= w.lo && tsa < w.hi && qa.d2 >= lim;
                        if (wave_any(la)) {
                            pair_terms(ga, qa, tsa, la, i, i, zafter, false, 0.0f);
                            if (NW == 1 && lane == 0) touched[i] = 1;
                        }
                      }
                    }
                    if (!resident) {
                        __syncthreads();
                        flush(cnt, gb);
                    }
                }
            }
            const bool more = comp_next(w, L, ns);
            if (!wave_any(more)) break;
            ztie = 0.0f;
            ns = comp_collect<EW>(P, sr, o, ents, resident, smask, v0, v1, v2, hm, sig2, tc, lane, w, L, slot_g, on_tie);
        }
        if (mapped) {
            __syncthreads();
            flush(ne, -1);
        }
    }

    if (NW > 1) {
        __syncthreads();
        for (int q = threadIdx.x; q < n; q += 64 * NW) {
            const int gg = sr.gauss_off + q;
            float sum[LREC];
#pragma unroll
            for (int c = 0; c < LREC; ++c) sum[c] = recs[0][LREC * q + c];
#pragma unroll
            for (int k = 1; k < NW; ++k)
#pragma unroll
                for (int c = 0; c < LREC; ++c) sum[c] += recs[k][LREC * q + c];
            if (PLAIN)
                write_partial_offset(prec_out + REC * q, sum, REC, P.prec + 6 * gg, P.means + 3 * gg, o);
            else
                write_partial(prec_out + REC * q, sum, REC, P.means + 3 * gg, o);
        }
    }
    if (threadIdx.x < 2) beta_partial[2 * it + threadIdx.x] = 0.0f;  // the model has no blend parameters
}

// ------------------------------------------------------------------------------------
// Split statistic (Sec. 8) with the compositing weights: lbar_i = (1/M) sum_j L_j w_ji, summed
// here per item and Gaussian; the running maximum and 1/S come from the forward's stash.
// ------------------------------------------------------------------------------------

// (waves and staging as in the backward)
template <int NW>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(kStatcWaves))) void statc_kernel(
    Params P, const float *__restrict__ loss, const float *__restrict__ stash, const BwdItem *__restrict__ items,
    const int *__restrict__ order, float *__restrict__ partial)
{
    constexpr int EW = 5;
    __shared__ float4 ents[kCompTG * EW];
    __shared__ float recs[NW][kCompTG];
    __shared__ int slot_gs[NW][kCompSlots];
    __shared__ int gid[NW == 1 ? kCompTG : 1];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    int *const slot_g = slot_gs[wave];
    float *const rec = recs[wave];
    const BwdItem item = ld_uniform(items + ld_uniform(order + blockIdx.x));
    const ViewRec vr = ld_uniform(P.views + item.view);
    const SceneRec sr = ld_uniform(P.scenes + vr.scene);
    const CamRec cam = cam_of(P, item.view);
    const float *e = cam.e, *kk = cam.k;
    double o[3];
    cam_centre(e, o);
    const float hm = (float)(-0.5 * kLog2e);
    const float sig2 = comp_sig_log2(sr.n), skip2 = comp_skip_log2(sr.n);
    const int n = sr.n;
    float *__restrict__ out = partial + item.poff;
    if (NW > 1) {
        for (int q = lane; q < n; q += 64) rec[q] = 0.0f;
        comp_stage<EW, 64 * NW>(P, sr, 0, n, o, ents);
    } else {
        for (int q = lane; q < n; q += 64) out[q] = 0.0f;
        __syncthreads();
    }
    const int nt = min(item.span, vr.tiles - item.ray0);
    for (int tt = wave; tt < nt; tt += NW) {
        int row, col;
        const int loc = tile_local(vr, item.ray0 + tt, lane, row, col);
        const bool valid = loc >= 0;
        float v0, v1, v2;
        tile_ray_dir(P, vr, e, kk, valid ? loc : 0, valid ? row : 0, valid ? col : 0, v0, v1, v2);
        float M2 = INFINITY, invS = 0.0f, lr = 0.0f;
        if (valid) {
            const size_t r = (size_t)vr.ray_off + loc;
            const float4 s0 = reinterpret_cast<const float4 *>(stash)[2 * r];
            M2 = s0.x;
            invS = s0.y;
            lr = loss[r];
        }
        const float wskip = valid ? M2 - __builtin_amdgcn_logf(invS) + skip2 : INFINITY;
        const float lim_min = wave_min_u(wskip);
        CompWin w{valid ? -INFINITY : INFINITY, INFINITY, 0.0f, 0.0f};
        CompList L;
        const TileBox tc = wave_box(v0, v1, v2, valid, e);
        int ne = n;
        float low;
        if (NW == 1) ne = comp_survivors<EW, false>(P, sr, o, ents, gid, tc, fminf(sig2, lim_min), 0.0f, lane, low);
        const bool resident = NW > 1 || ne <= kCompTG;
        const bool mapped = NW == 1 && resident;
        unsigned long long smask[2] = {0, 0}, fmask[2] = {0, 0};
        if (resident) {
            const CompBounds cb = comp_bounds<EW>(ents, ne, tc, lane);
            comp_masks(cb, ne, lane, sig2, smask);
            comp_masks(cb, ne, lane, lim_min, fmask);
        }
        if (mapped) {
            for (int q = lane; q < ne; q += 64) rec[q] = 0.0f;
            __syncthreads();
        }
        const auto no_tie = [](const Ent &, const Geo &, float, int) {};
        // loss times the normalised weight of the lane's pair, summed over the wave into rec[i]
        auto term = [&](const Geo &q, bool live, float ts, int ns, int i) {
            float x = 0.0f;
            if (live) {
                const float lw = fmaf(-(float)kLog2e, comp_front(L, ns, w, ts), log2_opacity(exp2_(q.d2), q.d2));
                x = lr * (exp2_(lw - M2) * invS);
            }
            x = wave_sum_u(x);
            if (lane == 0) rec[i] += x;
        };
        for (bool first = true;; first = false) {
            const int ns = comp_collect<EW>(P, sr, o, ents, resident, smask, v0, v1, v2, hm, sig2, tc, lane, w, L, slot_g, no_tie);
            // as in the backward: a tile of one window whose rays all weigh at least 2^kCompHitLog2
            // somewhere takes only the slots' Gaussians
            if (first && resident && ns > 0 && !wave_any(w.hi != INFINITY) && wave_all(!valid || M2 >= kCompHitLog2)) {
                for (int s = 0; s < ns; ++s) {
                    const int gi = slot_g[s];
                    Geo q;
                    pair_geo_coarse(comp_ent<EW>(ents, gi), v0, v1, v2, hm, 0.0f, 0.0f, q);
                    term(q, valid && q.d2 > sig2, q.t * kDepthScale, ns, gi);
                }
                break;
            }
            for (int gb = 0; gb < (resident ? 1 : n); gb += kCompTG) {
                const int cnt = min(kCompTG, n - gb);
                unsigned long long fm[2] = {fmask[0], fmask[1]};
                if (!resident) {
                    comp_stage<EW, 64>(P, sr, gb, cnt, o, ents);
                    for (int q = lane; q < cnt; q += 64) rec[q] = 0.0f;
                    __syncthreads();
                    comp_masks(comp_bounds<EW>(ents, cnt, tc, lane), cnt, lane, lim_min, fm);
                }
#pragma unroll 1
                for (int c = 0; c < 2; ++c) {
                    unsigned long long mk = fm[c];
                    while (mk) {
                        const int i = 64 * c + __builtin_ctzll(mk);
                        mk &= mk - 1;
                        Geo q;
                        pair_geo_coarse(comp_ent<EW>(ents, i), v0, v1, v2, hm, 0.0f, 0.0f, q);
                        const float ts = q.t * kDepthScale;
                        const bool live = ts >= w.lo && ts < w.hi && q.d2 >= wskip;
                        if (wave_any(live)) term(q, live, ts, ns, i);
                    }
                }
                if (!resident) {
                    __syncthreads();
                    for (int q = lane; q < cnt; q += 64) out[gb + q] += rec[q];
                }
            }
            const bool more = comp_next(w, L, ns);
            if (!wave_any(more)) break;
        }
        if (mapped) {
            __syncthreads();
            for (int q = lane; q < ne; q += 64) out[gid[q]] += rec[q];
        }
    }
    if (NW > 1) {
        __syncthreads();
        for (int q = threadIdx.x; q < n; q += 64 * NW) {
            float sum = recs[0][q];
#pragma unroll
            for (int k = 1; k < NW; ++k) sum += recs[k][q];
            out[q] = sum;
        }
    }
}

// ------------------------------------------------------------------------------------
// Launchers
// ------------------------------------------------------------------------------------

#define FMB_COMP_DISPATCH(flags, CALL)                                                                     \
    switch (flags) {                                                                                      \
    case 0: CALL(0); break;                                                                               \
    case 1: CALL(1); break;                                                                               \
    case 2: CALL(2); break;                                                                               \
    case 3: CALL(3); break;                                                                               \
    case 4: CALL(4); break;                                                                               \
    case 5: CALL(5); break;                                                                               \
    case 6: CALL(6); break;                                                                             \
    case 7: CALL(7); break;                                                                             \
    default: return hipErrorInvalidValue;                                                                 \
    }

#define FMB_FWDC_SMALL(F_) hipLaunchKernelGGL((fwdc_kernel<F_, 4>), dim3(n_small), dim3(256), 0, st, P, O, items)
#define FMB_FWDC_BIG(F_) hipLaunchKernelGGL((fwdc_kernel<F_, 1>), dim3(n_big), dim3(64), 0, st, P, O, items + n_small)
#define FMB_BWDC_SMALL(F_)                                                                                \
    hipLaunchKernelGGL((bwdc_kernel<F_, 4>), dim3(n_small), dim3(256), 0, st, P, I, items, order, partial, beta_partial)
#define FMB_BWDC_BIG(F_)                                                                                  \
    hipLaunchKernelGGL((bwdc_kernel<F_, 1>), dim3(n_big), dim3(64), dyn, st, P, I, items, order ? order + n_small : nullptr, partial, beta_partial)

int comp_resident_max() { return kCompTG; }

// Blocks take the items in order: first the n_small items of scenes of at most kCompTG Gaussians (four
// waves per block), then the n_big of larger ones (one wave per block).
hipError_t launch_fwdc(int flags, int n_small, int n_big, hipStream_t st, const Params &P, const FwdOut &O,
                       const CompItem *items)
{
    if (n_small > 0) FMB_COMP_DISPATCH(flags, FMB_FWDC_SMALL)
    if (n_big > 0) FMB_COMP_DISPATCH(flags, FMB_FWDC_BIG)
    return hipGetLastError();
}

// order: the items' indices, the n_small of small scenes first (or NULL where they are all of one kind).
hipError_t launch_bwdc(int flags, int n_small, int n_big, hipStream_t st, const Params &P, const BwdIn &I,
                       const BwdItem *items, const int *order, float *partial, float *beta_partial)
{
    const size_t dyn = (size_t)kCompSlots * 6 * sizeof(float4);
    if (!order && n_small > 0 && n_big > 0) return hipErrorInvalidValue;
    if (n_small > 0) FMB_COMP_DISPATCH(flags, FMB_BWDC_SMALL)
    if (n_big > 0) FMB_COMP_DISPATCH(flags, FMB_BWDC_BIG)
    return hipGetLastError();
}

hipError_t launch_statc(int n_small, int n_big, hipStream_t st, const Params &P, const float *loss, const float *stash,
                        const BwdItem *items, const int *order, float *partial)
{
    if (n_small > 0)
        hipLaunchKernelGGL((statc_kernel<4>), dim3(n_small), dim3(256), 0, st, P, loss, stash, items, order, partial);
    if (n_big > 0)
        hipLaunchKernelGGL((statc_kernel<1>), dim3(n_big), dim3(64), 0, st, P, loss, stash, items, order + n_small, partial);
    return hipGetLastError();
}

}  // namespace fmb
