// fmb_kernels.hip -- gfx950 kernels of the sort-free two-parameter Fuzzy Metaballs
// renderer (Keselman & Hebert, WACV 2024, Sec. 3.1-3.2, 5, 6).
//
// Layout of the work (see fmb_internal.h):
//   * forward: one lane per ray (RPT rays per lane), Gaussians staged through LDS in
//     tiles of TG; each (view, Gaussian) entry is formed on the fly in FP64 when the
//     tile is loaded (mean relative to the camera centre as a float hi/lo pair, the
//     precision-weighted mean c = Sigma^-1 (mu - o), log2 lambda).  The softmax of the
//     blend weights (Eq. 7 in Eq. 3) runs online in FP32 registers in base 2.
//   * backward: one lane per (Gaussian, ray slot); rays of the item's span are staged
//     through LDS with their per-ray adjoint prologue; every lane recomputes its pairs
//     and accumulates its Gaussian's gradient in registers -- no per-pair cross-lane
//     reduction and no P x N storage (without a normal cotangent in the offset form of
//     pair_adjoint_offset).  Partial gradients per item are reduced deterministically by
//     the finalize kernel.
//   * a block takes one item; of a batch, whose items are uneven, in the order given by the host
//     (largest item first), so that the last blocks to start are the shortest.
//
// Per pair (ray o + t v with |v| = 1, Gaussian mu, U, lambda; mu' = mu - o):
//   a = U v, t = v.c / a.a (peak of the density along the ray, Sec. 3.1),
//   r = U (t v - mu') formed as U (t v - hi) - U lo, m = r.r, d = log lambda - m/2 (Eq. 2),
//   delta = e^d (Eq. 4), z = beta1 d - (beta2/eta) t (log of Eq. 7); where a normal is
//   needed, one Newton step on |U(t v - mu')|^2 moves r to the peak, g = U^T r =
//   Sigma^-1 x (Eq. 17).
#include "fmb_device.h"

namespace fmb {

// ------------------------------------------------------------------------------------
// Forward
// ------------------------------------------------------------------------------------

template <int BLOCK, int RPT, int TG, int F>
__global__ __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(TG > 128 ? 3 : 4))) void fwd_kernel(Params P, FwdOut O, const FwdItem *__restrict__ items,
                                                   const int *__restrict__ order)
{
    constexpr bool NORMALS = (F & kNrm) != 0;
    constexpr bool COLOR = (F & kCol) != 0, BIG = (F & kBig) != 0;
    constexpr int EW = COLOR ? 6 : 5;  // float4 per LDS entry: the entry, the m estimate terms, colour
    __shared__ float4 tile[TG * EW];
    // the upper bound of the log2 weight of each staged (Gaussian, ray tile), +inf where its density can
    // reach the cutoff: per wave, per group of 64 / RPT Gaussians, per lane
    __shared__ float hisave[BLOCK / 64][TG * RPT];
    __shared__ float4 tbox[BLOCK / 64 * RPT * 3];  // each ray tile's box (TileBox)
    // scenes beyond BLOCK Gaussians: the waves' least running maxima, their counts
    // of survivors (of two rounds in turn), and the list of survivors (a ring)
    constexpr int LIST = 2 * BLOCK;
    static_assert(TG <= BLOCK, "a round is added to fewer than TG survivors");
    __shared__ float wmin[BIG ? BLOCK / 64 : 1];
    __shared__ int wcnt[2][BIG ? BLOCK / 64 : 1];
    __shared__ int slist[BIG ? LIST : 1];
    const int it = order ? ld_uniform(order + blockIdx.x) : (int)blockIdx.x;
    const FwdItem item = ld_uniform(items + it);
    const ViewRec vr = ld_uniform(P.views + item.view);
    const SceneRec sr = ld_uniform(P.scenes + vr.scene);
    const CamRec cam = cam_of(P, item.view);
    const float *e = cam.e, *kk = cam.k;
    double o[3];
    cam_centre(e, o);
    const Blend bl = blend_of(P, vr.scene);
    const bool b1_pos = bl.b1 >= 0.0f;  // the weight bound needs beta1 >= 0
    // ray j of a lane: lane `lane` of tile tile0 + j * NW + wave (8 x 8 pixels where the view is
    // wide enough: a wave's rays stay close together, so the exact skip of zero weights below
    // is uniform over the wave more often)
    constexpr int NW = BLOCK / 64;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;

    float v0[RPT], v1[RPT], v2[RPT];
    float M[RPT], S[RPT], T[RPT], N0[RPT], N1[RPT], N2[RPT], D[RPT], C0[RPT], C1[RPT], C2[RPT];
    float at[RPT], dt[RPT];  // loss targets, loaded now so that the epilogue does not wait
    int loc[RPT];
#pragma unroll
    for (int j = 0; j < RPT; ++j) {
        int row, col;
        loc[j] = tile_local(vr, item.tile0 + j * NW + wave, lane, row, col);
        const int lc = loc[j] >= 0 ? loc[j] : 0;  // a lane past the edge takes ray 0 (not written)
        tile_ray_dir(P, vr, e, kk, lc, loc[j] >= 0 ? row : 0, loc[j] >= 0 ? col : 0, v0[j], v1[j], v2[j]);
        M[j] = -FLT_MAX;  // (not -inf: a first weight of 0 stays below it)
        S[j] = T[j] = N0[j] = N1[j] = N2[j] = D[j] = C0[j] = C1[j] = C2[j] = 0.0f;
        at[j] = dt[j] = 0.0f;
        if (O.g_depth) {
            at[j] = O.alpha_t[vr.ray_off + lc];
            dt[j] = O.depth_t[vr.ray_off + lc];
        }
    }
    // The box of each of the wave's ray tiles, for the bounds of tile_bounds: lane l bounds Gaussian
    // l / RPT on ray tile l % RPT.
    const int jl = lane % RPT;
#pragma unroll
    for (int j = 0; j < RPT; ++j) {
        const TileBox b = wave_box(v0[j], v1[j], v2[j], loc[j] >= 0, e);
        if (lane == 0) {
            tbox[3 * (wave * RPT + j)] = b.c;
            tbox[3 * (wave * RPT + j) + 1] = b.x;
            tbox[3 * (wave * RPT + j) + 2] = b.y;
        }
    }
    // lower bound over lane's tile jl, from the Gaussians bounded so far, of the running maximum
    float mlow = -INFINITY;

    // Of a scene of more than BLOCK Gaussians each is first bounded on a box around all the item's
    // tiles, BLOCK of them a round, and only those whose density can reach the cutoff there, or whose
    // weight can be above FP32's zero against the least running maximum of the item's rays so
    // far, are listed, in scene order; rounds go on until the list fills a staged tile (a round of
    // 10 000 clustered Gaussians leaves a handful: staged and bounded by themselves they took a third
    // of the kernel's instructions, 718 us against 542 for a 1920 x 1080 view).  The running
    // maxima only grow, so a Gaussian left out is one that the tests below would
    // skip when its turn came.
    // Smaller scenes stage all their Gaussians (and launches without kBig, whose scenes are all
    // small, have no list).
    const bool sparse = BIG && sr.n > BLOCK;
    TileBox ibox;
    int rb = 0, head = 0, total = sparse ? 0 : sr.n;  // next round, ring position and count of the listed
    for (bool first = true; ; first = false) {
      if (sparse && rb < sr.n && total < TG) {
        float mm = INFINITY;
#pragma unroll
        for (int j = 0; j < RPT; ++j) mm = loc[j] >= 0 ? fminf(mm, M[j]) : mm;
        mm = wave_min_u(mm);
        if (lane == 0) wmin[wave] = mm;
        __syncthreads();  // tile boxes and least maxima visible
        if (first) ibox = wave_box_of(tbox, NW * RPT, lane, e);
        float imin = INFINITY;
        for (int w = 0; w < NW; ++w) imin = fminf(imin, wmin[w]);
        do {
            const int gl = rb + (int)threadIdx.x, par = (rb / BLOCK) & 1;
            bool keep = false;
            if (gl < sr.n) {
                const int gg = sr.gauss_off + gl;
                Ent ge;
                float4 ee;
                make_bound_entry(P.means + 3 * gg, P.prec + 6 * gg, P.weights[gg], o, ge, ee);
                const PairBounds pb = tile_bounds(ge, ee, ibox, bl.hm, bl.b1, bl.nc2);
                // (written so that a NaN bound keeps the Gaussian)
                keep = !(b1_pos && pb.d2_hi < kDensSkipLog2 && pb.z_hi - imin < kSkipLog2);
            }
            const unsigned long long bal = wave_ballot(keep);
            if (lane == 0) wcnt[par][wave] = __popcll(bal);
            __syncthreads();
            int off = head + total;
            for (int w = 0; w < NW; ++w) {
                const int c = wcnt[par][w];
                off += w < wave ? c : 0;
                total += c;
            }
            if (keep) slist[(off + __popcll(bal & ((1ull << lane) - 1ull))) & (LIST - 1)] = gl;
            rb += BLOCK;
        } while (rb < sr.n && total < TG);
      }
      if (total == 0) break;
      {
        const int cnt = min(TG, total);
        if (!first || sparse) __syncthreads();  // the list visible; the previous tile is consumed
        for (int q = threadIdx.x; q < cnt; q += BLOCK) {
            const int gi = sr.gauss_off + (sparse ? slist[(head + q) & (LIST - 1)] : head + q);
            make_entry_est(P.means + 3 * gi, P.prec + 6 * gi, P.weights[gi], o, &tile[EW * q]);
            if (COLOR) tile[EW * q + 5] = colour_entry(P.colors + 3 * gi);
        }
        __syncthreads();
        // Every (Gaussian, ray tile) of the staged tile is bounded first, GP Gaussians at a time;
        // the lower bounds give the least running maximum that the tile's rays end with.  A pair is
        // taken if on some ray its density can reach 2^kDensSkipLog2 or its weight be above FP32's
        // zero.  Without beta1 >= 0 the weight bounds do not hold and every pair is taken.
        constexpr int GP = 64 / RPT;
        const TileBox bj = TileBox{tbox[3 * (wave * RPT + jl)], tbox[3 * (wave * RPT + jl) + 1], tbox[3 * (wave * RPT + jl) + 2]};
        for (int ib = 0; ib < cnt; ib += GP) {
            const int il = ib + lane / RPT;
            if (il < cnt) {
                const Ent gl = ent_from(tile[EW * il], tile[EW * il + 1], tile[EW * il + 2], tile[EW * il + 3]);
                const PairBounds pb = tile_bounds(gl, tile[EW * il + 4], bj, bl.hm, bl.b1, bl.nc2);
                // (comparisons written so that a NaN bound keeps the pair)
                hisave[wave][ib * RPT + lane] = pb.d2_hi < kDensSkipLog2 ? pb.z_hi : INFINITY;
                mlow = fmaxf(mlow, pb.z_lo);
            }
        }
#pragma unroll
        for (int off = RPT; off < 64; off <<= 1) mlow = fmaxf(mlow, __shfl_xor(mlow, off, 64));
        if (!first) {  // the maxima of the Gaussians taken so far bound too
#pragma unroll
            for (int j = 0; j < RPT; ++j) {
                const float mm = wave_min_u(loc[j] >= 0 ? M[j] : INFINITY);
                if (jl == j) mlow = fmaxf(mlow, mm);
            }
        }
        // (The running maximum itself starts below every weight, not at that bound: sums scaled to a bound round
        // otherwise than sums scaled to weights, and the sign of an L1 loss follows the last bit of a depth.
        // Starting at the bound saved 0.4 % of a step, of 16 scenes 1.6 %.)
        const float zcut = mlow + kSkipLog2;
        for (int ib = 0; ib < cnt; ib += GP) {
            const int il = ib + lane / RPT;
            bool need = false;
            if (il < cnt && bj.c.w >= 0.0f) {
                // (a weight of 0, with a bound of -inf, is passed over also where zcut is -inf)
                const float h = hisave[wave][ib * RPT + lane];
                need = !(b1_pos && (h < zcut || h == -INFINITY));
            }
            unsigned long long nm = wave_ballot(need);
          while (nm != 0ull) {
            const int k = __builtin_ctzll(nm) / RPT;
            const unsigned bits = (unsigned)(nm >> (k * RPT)) & ((1u << RPT) - 1u);
            nm &= ~((unsigned long long)((1u << RPT) - 1u) << (k * RPT));
            const int i = ib + k;
            const Ent g = ent_from(tile[EW * i], tile[EW * i + 1], tile[EW * i + 2], tile[EW * i + 3]);
            float4 cc = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            if (COLOR) cc = tile[EW * i + 5];
#pragma unroll
            for (int j = 0; j < RPT; ++j) {
                if (!((bits >> j) & 1u)) continue;  // no ray of tile j needs the pair
                Geo q;
                pair_geo_coarse(g, v0[j], v1[j], v2[j], bl.hm, bl.b1, bl.nc2, q);
                const float delta = exp2_(q.d2);
                D[j] += delta;
                // log2 of the weight relative to the running maximum, b1 d2 + (nc2 t - M)
                float zr = fmaf(bl.b1, q.d2, fmaf(bl.nc2, q.t, -M[j]));
                // A weight below 2^-150 of the running maximum is zero in FP32: its terms are
                // skipped (the branch is uniform over a wave for most distant Gaussians).
                if (zr < kSkipLog2) continue;
                pair_refine(q);
                if (zr > 0.0f) {  // new running maximum: rescale the sums (rare)
                    const float sc = exp2_(M[j] - q.z2);
                    S[j] *= sc;
                    T[j] *= sc;
                    if (NORMALS) {
                        N0[j] *= sc;
                        N1[j] *= sc;
                        N2[j] *= sc;
                    }
                    if (COLOR) {
                        C0[j] *= sc;
                        C1[j] *= sc;
                        C2[j] *= sc;
                    }
                    M[j] = q.z2;
                    zr = 0.0f;
                }
                const float ew = exp2_(zr);
                S[j] += ew;
                T[j] = fmaf(ew, q.t, T[j]);
                if (NORMALS) {
                    const float g0 = g.u00 * q.r0;
                    const float g1 = fmaf(g.u01, q.r0, g.u11 * q.r1);
                    const float g2 = fmaf(g.u02, q.r0, fmaf(g.u12, q.r1, g.u22 * q.r2));
                    const float es = ew * rsq_(fmaf(g0, g0, fmaf(g1, g1, fmaf(g2, g2, kEpsN))));
                    N0[j] = fmaf(es, g0, N0[j]);
                    N1[j] = fmaf(es, g1, N1[j]);
                    N2[j] = fmaf(es, g2, N2[j]);
                }
                if (COLOR) {
                    C0[j] = fmaf(ew, cc.x, C0[j]);
                    C1[j] = fmaf(ew, cc.y, C1[j]);
                    C2[j] = fmaf(ew, cc.z, C2[j]);
                }
            }
          }
        }
        head += cnt;
        total -= cnt;
      }
    }

    const float o0 = (float)o[0], o1 = (float)o[1], o2 = (float)o[2];
#pragma unroll
    for (int j = 0; j < RPT; ++j) {
        if (loc[j] < 0) continue;
        write_ray<F>(P, O, item.view, vr.ray_off + loc[j], e, kk, o0, o1, o2, v0[j], v1[j], v2[j], M[j], S[j],
                     T[j], N0[j], N1[j], N2[j], C0[j], C1[j], C2[j], D[j], at[j], dt[j]);
    }
}

// ------------------------------------------------------------------------------------
// Backward
// ------------------------------------------------------------------------------------


// Waves per SIMD the Gaussian-lane backward is compiled for: six (at most 80 VGPRs) where the
// variant fits without spilling, else what its registers give.
constexpr int bwd_min_waves(int F)
{
    return (F & kCol) && F != kCol ? 1 : 6;
}

template <int BLOCK, int RT, int F>
__global__ __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(bwd_min_waves(F)))) void bwd_kernel(Params P, BwdIn I, const BwdItem *__restrict__ items,
                                                   const int *__restrict__ order, float *__restrict__ partial,
                                                   float *__restrict__ beta_partial)
{
    constexpr bool NORMALS = (F & kNrm) != 0, COLOR = (F & kCol) != 0;
    // Without a normal cotangent the pairs take pair_adjoint_offset: the staged ray is
    // (v, M2) (invS, tf_bar, kappa, D_bar) (t_f, dc, 0, 0) [(Cb, 0)]; with one it is the prologue
    // as written by ray_prologue (four float4).
    constexpr bool PLAIN = !NORMALS;
    constexpr int RW = PLAIN ? (COLOR ? 4 : 3) : 4;  // float4 per staged ray
    constexpr int REC = COLOR ? kPartialColor : kPartial;  // partial record per Gaussian
    // a lane's sums: (H, Bv, L) of the offset form or the general record, then the colour sums
    constexpr int LREC = PLAIN ? kOffsetAcc + (COLOR ? 3 : 0) : REC;
    constexpr int RS = LREC + 2;                  // reduction record per lane (+ two betas)
    // the staged rays and, after an item's pair loop, the reduction records share the LDS
    constexpr int SM4 = RT * RW > BLOCK * RS / 4 ? RT * RW : (BLOCK * RS + 3) / 4;
    __shared__ float4 smem[SM4];
    float4 *rays = smem;
    float *red = reinterpret_cast<float *>(smem);
    const int tid = threadIdx.x;
    const int it = order ? ld_uniform(order + blockIdx.x) : (int)blockIdx.x;
    const BwdItem item = ld_uniform(items + it);
    const ViewRec vr = ld_uniform(P.views + item.view);
    const SceneRec sr = ld_uniform(P.scenes + vr.scene);
    const CamRec cam = cam_of(P, item.view);
    const float *e = cam.e, *kk = cam.k;
    double o[3];
    cam_centre(e, o);
    const float o0 = (float)o[0], o1 = (float)o[1], o2 = (float)o[2];
    const Blend bl = blend_of(P, vr.scene);
    const int hw = vr.h * vr.w;
    const int end = min(item.ray0 + item.span, hw);

    const int gi = tid % item.gc;
    const int slot = tid / item.gc;
    const bool active = slot < item.slots && item.g0 + gi < sr.n;
    Ent g;
    float4 cc = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    if (active) {
        const int gg = sr.gauss_off + item.g0 + gi;
        float4 q[4];
        make_entry(P.means + 3 * gg, P.prec + 6 * gg, P.weights[gg], o, q);
        g = ent_from(q[0], q[1], q[2], q[3]);
        if (COLOR) cc = colour_entry(P.colors + 3 * gg);
    }
    float aB1 = 0, aB2 = 0;
    float aC0 = 0, aC1 = 0, aC2 = 0;
    // The item's rays RT at a time: staged with their prologue, then `pair` runs over this lane's
    // rays slot, slot + slots, ... (walked by address: one induction variable).
    auto passes = [&](auto &&pair) {
        for (int r0 = item.ray0; r0 < end; r0 += RT) {
            const int cnt = min(RT, end - r0);
            __syncthreads();
            for (int q = tid; q < RT; q += BLOCK) {
                float4 pr[4];
                ray_prologue<F>(P, I, item.view, vr, e, kk, o0, o1, o2, r0 + q, q < cnt, bl.b1, bl.nc2, pr);
                if (PLAIN) {
                    rays[RW * q] = pr[0];
                    rays[RW * q + 1] = make_float4(pr[1].x, pr[1].y, pr[2].y, pr[2].z);
                    rays[RW * q + 2] = make_float4(pr[2].w, pr[3].w, 0.0f, 0.0f);
                    if (COLOR) rays[RW * q + 3] = pr[3];
                } else {
#pragma unroll
                    for (int k = 0; k < RW; ++k) rays[RW * q + k] = pr[k];
                }
            }
            __syncthreads();
            if (active) {
                const float4 *const rend = rays + RW * cnt;
                for (const float4 *rp = rays + RW * slot; rp < rend; rp += RW * item.slots) pair(rp);
            }
        }
        __syncthreads();  // every lane is done with the staged rays (the LDS is reused below)
    };
    // One pair without a normal cotangent, accumulated in the offset form.
    auto plain_pair = [&](const float4 *rp, OffsetAcc &acc) {
        const float4 x0 = rp[0], x1 = rp[1], x2 = rp[2];
        float4 x4 = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        if (COLOR) x4 = rp[3];
        const float v0 = x0.x, v1 = x0.y, v2 = x0.z;
        Geo q;
        pair_geo_coarse(g, v0, v1, v2, bl.hm, bl.b1, bl.nc2, q);
        const float delta = exp2_(q.d2);
        // normalised blend weight 2^(z2 - M) / S, with z2 - M = b1 d2 + (nc2 t - M)
        const float wt = exp2_(fmaf(bl.b1, q.d2, fmaf(bl.nc2, q.t, -x0.w))) * x1.x;
        const float tfb = x1.y;
        float lin = tfb * q.t;
        if (COLOR) {
            lin = fmaf(x4.x, cc.x, fmaf(x4.y, cc.y, fmaf(x4.z, cc.z, lin)));
            aC0 = fmaf(wt, x4.x, aC0);
            aC1 = fmaf(wt, x4.y, aC1);
            aC2 = fmaf(wt, x4.z, aC2);
        }
        const float zb = wt * (lin - x1.z);
        const float tb = fmaf(-bl.cb, zb, wt * tfb);
        const float db = fmaf(bl.b1, zb, x1.w * delta);
        aB1 = fmaf(zb, q.d2 - x2.y, aB1);
        aB2 = fmaf(zb, q.t - x2.x, aB2);
        pair_adjoint_offset(q, v0, v1, v2, tb, db, acc);
    };
    float *my = red + RS * tid;
    if (!PLAIN) {
        PairAcc acc;
        passes([&](const float4 *rp) {
            const float4 x0 = rp[0], x1 = rp[1], x2 = rp[2], x3 = rp[3];
            const float v0 = x0.x, v1 = x0.y, v2 = x0.z;
            Geo q;
            pair_geo(g, v0, v1, v2, bl.hm, bl.b1, bl.nc2, q);
            const float delta = exp2_(q.d2);
            const float wt = exp2_(q.z2 - x0.w) * x1.x;   // normalised blend weight
            const float tfb = x1.y;
            PairNormal pn{0, 0, 0, 0, 0};
            if (NORMALS) pn = pair_normal(g, q, x1.z, x1.w, x2.x);
            // softmax adjoint: z_bar = wt (tf_bar t + Nb.n + Cb.c - kappa)
            float lin = fmaf(tfb, q.t, pn.nN);
            if (COLOR) {
                lin = fmaf(x3.x, cc.x, fmaf(x3.y, cc.y, fmaf(x3.z, cc.z, lin)));
                aC0 = fmaf(wt, x3.x, aC0);
                aC1 = fmaf(wt, x3.y, aC1);
                aC2 = fmaf(wt, x3.z, aC2);
            }
            const float zb = wt * (lin - x2.y);
            // z = beta1 d - (beta2/eta) t
            const float tb = fmaf(-bl.cb, zb, wt * tfb);
            const float db = fmaf(bl.b1, zb, x2.z * delta);
            aB1 = fmaf(zb, q.d2 - x3.w, aB1);
            aB2 = fmaf(zb, q.t - x2.w, aB2);
            pair_adjoint<NORMALS>(g, q, v0, v1, v2, wt, pn, x1.z, x1.w, x2.x, tb, db, acc);
        });
        my[0] = acc.u0; my[1] = acc.u1; my[2] = acc.u2; my[3] = acc.u3; my[4] = acc.u4; my[5] = acc.u5;
        my[6] = acc.p0; my[7] = acc.p1; my[8] = acc.p2; my[9] = acc.l;
    } else {
        OffsetAcc acc;
        passes([&](const float4 *rp) { plain_pair(rp, acc); });
        offset_acc_store(acc, my);
    }

    // deterministic block reduction: Gaussian partials over the slots, betas over all lanes
    if (COLOR) {
        my[LREC - 3] = aC0; my[LREC - 2] = aC1; my[LREC - 1] = aC2;
    }
    my[LREC] = aB1; my[LREC + 1] = aB2;
    __syncthreads();
    if (slot == 0 && gi < item.gc && item.g0 + gi < sr.n) {
        float sum[LREC];
#pragma unroll
        for (int c = 0; c < LREC; ++c) sum[c] = red[RS * gi + c];
        for (int s = 1; s < item.slots; ++s) {
#pragma unroll
            for (int c = 0; c < LREC; ++c) sum[c] += red[RS * (s * item.gc + gi) + c];
        }
        const int gg = sr.gauss_off + item.g0 + gi;
        if (PLAIN)
            write_partial_offset(partial + item.poff + REC * gi, sum, REC, P.prec + 6 * gg, P.means + 3 * gg, o);
        else
            write_partial(partial + item.poff + REC * gi, sum, REC, P.means + 3 * gg, o);
    }
    if (tid < 64) {
        // lane l sums lanes l, l+64, ... in order, then a fixed butterfly over the wave
        float s1 = 0.0f, s2 = 0.0f;
        for (int k = tid; k < BLOCK; k += 64) {
            s1 += red[RS * k + LREC];
            s2 += red[RS * k + LREC + 1];
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            s1 += __shfl_xor(s1, off, 64);
            s2 += __shfl_xor(s2, off, 64);
        }
        if (tid == 0) {
            beta_partial[2 * it] = s1;
            beta_partial[2 * it + 1] = s2;
        }
    }
}

// ------------------------------------------------------------------------------------
// Backward, ray-lane layout: one lane per ray (RPT rays per lane) as in the forward pass,
// the item's Gaussians staged through LDS in tiles of TG.  For each Gaussian the lanes'
// terms are summed over the wave (butterfly) and the wave sums in LDS, over the item's ray
// tiles, so an item writes one partial record per Gaussian of its scene.  A Gaussian whose
// blend weight is exactly zero (below 2^-150 of the ray's maximum) on every ray of the wave
// takes only the density term of alpha, and one whose density is zero too is skipped.
// ------------------------------------------------------------------------------------

__device__ __forceinline__ float wave_sum(float x)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off, 64);
    return x;
}

template <int BLOCK, int RPT, int TG, int F>
__global__ __launch_bounds__(BLOCK) void bwdr_kernel(Params P, BwdIn I, const BwdItem *__restrict__ items,
                                                    const int *__restrict__ order, float *__restrict__ partial,
                                                    float *__restrict__ beta_partial)
{
    constexpr bool NORMALS = (F & kNrm) != 0, COLOR = (F & kCol) != 0;
    // without a normal cotangent the pairs take the offset form (pair_adjoint_offset)
    constexpr bool PLAIN = !NORMALS;
    constexpr int EW = COLOR ? 5 : 4;                       // float4 per LDS entry
    constexpr int REC = COLOR ? kPartialColor : kPartial;  // partial record per Gaussian
    // sums per Gaussian and wave: (H, Bv, L) of the offset form or the general record, then colour
    constexpr int LREC = PLAIN ? kOffsetAcc + (COLOR ? 3 : 0) : REC;
    constexpr int NW = BLOCK / 64;
    __shared__ float4 tile[TG * EW];
    __shared__ float wsum[NW * TG * LREC];  // per wave, per Gaussian of the tile
    __shared__ float bsum[NW * 2];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int it = order ? ld_uniform(order + blockIdx.x) : (int)blockIdx.x;
    const BwdItem item = ld_uniform(items + it);
    const ViewRec vr = ld_uniform(P.views + item.view);
    const SceneRec sr = ld_uniform(P.scenes + vr.scene);
    const CamRec cam = cam_of(P, item.view);
    const float *e = cam.e, *kk = cam.k;
    double o[3];
    cam_centre(e, o);
    const float o0 = (float)o[0], o1 = (float)o[1], o2 = (float)o[2];
    const Blend bl = blend_of(P, vr.scene);
    const int hw = vr.h * vr.w;
    const int end = min(item.ray0 + item.span, hw);
    float aB1 = 0.0f, aB2 = 0.0f;

    for (int gb = 0; gb < sr.n; gb += TG) {
        const int cnt = min(TG, sr.n - gb);
        __syncthreads();  // the previous tile's entries and sums are no longer read
        for (int q = tid; q < cnt; q += BLOCK) {
            const int gi = sr.gauss_off + gb + q;
            make_entry(P.means + 3 * gi, P.prec + 6 * gi, P.weights[gi], o, &tile[EW * q]);
            if (COLOR) tile[EW * q + 4] = colour_entry(P.colors + 3 * gi);
        }
        for (int q = tid; q < NW * TG * LREC; q += BLOCK) wsum[q] = 0.0f;
        __syncthreads();
        for (int rb = item.ray0; rb < end; rb += BLOCK * RPT) {
            float4 x0[RPT], x1[RPT], x2[RPT], x3[RPT];
#pragma unroll
            for (int j = 0; j < RPT; ++j) {
                const int local = rb + tid + j * BLOCK;
                float4 pr[4];
                ray_prologue<F>(P, I, item.view, vr, e, kk, o0, o1, o2, local, local < end, bl.b1, bl.nc2, pr);
                x0[j] = pr[0];
                x1[j] = pr[1];
                x2[j] = pr[2];
                x3[j] = pr[3];
            }
            for (int i = 0; i < cnt; ++i) {
                const Ent g = ent_from(tile[EW * i], tile[EW * i + 1], tile[EW * i + 2], tile[EW * i + 3]);
                float4 cc = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                if (COLOR) cc = tile[EW * i + 4];
                Geo q[RPT];
                float delta[RPT], wt[RPT];
                bool need_w = false, need_d = false;
#pragma unroll
                for (int j = 0; j < RPT; ++j) {
                    if (PLAIN)
                        pair_geo_coarse(g, x0[j].x, x0[j].y, x0[j].z, bl.hm, bl.b1, bl.nc2, q[j]);
                    else
                        pair_geo(g, x0[j].x, x0[j].y, x0[j].z, bl.hm, bl.b1, bl.nc2, q[j]);
                    delta[j] = exp2_(q[j].d2);
                    const bool w_on = q[j].z2 - x0[j].w >= kSkipLog2;
                    wt[j] = w_on ? exp2_(q[j].z2 - x0[j].w) * x1[j].x : 0.0f;
                    need_w |= w_on;
                    need_d |= x2[j].z * delta[j] != 0.0f;
                }
                PairAcc a;
                OffsetAcc pa;
                float aC0 = 0.0f, aC1 = 0.0f, aC2 = 0.0f;
                if (wave_any(need_w)) {
#pragma unroll
                    for (int j = 0; j < RPT; ++j) {
                        const float tfb = x1[j].y;
                        PairNormal pn{0, 0, 0, 0, 0};
                        if (NORMALS) pn = pair_normal(g, q[j], x1[j].z, x1[j].w, x2[j].x);
                        float lin = fmaf(tfb, q[j].t, pn.nN);
                        if (COLOR) {
                            lin = fmaf(x3[j].x, cc.x, fmaf(x3[j].y, cc.y, fmaf(x3[j].z, cc.z, lin)));
                            aC0 = fmaf(wt[j], x3[j].x, aC0);
                            aC1 = fmaf(wt[j], x3[j].y, aC1);
                            aC2 = fmaf(wt[j], x3[j].z, aC2);
                        }
                        const float zb = wt[j] * (lin - x2[j].y);
                        const float tb = fmaf(-bl.cb, zb, wt[j] * tfb);
                        const float db = fmaf(bl.b1, zb, x2[j].z * delta[j]);
                        aB1 = fmaf(zb, q[j].d2 - x3[j].w, aB1);
                        aB2 = fmaf(zb, q[j].t - x2[j].w, aB2);
                        if (PLAIN) {
                            pair_adjoint_offset(q[j], x0[j].x, x0[j].y, x0[j].z, tb, db, pa);
                        } else {
                            pair_adjoint<NORMALS>(g, q[j], x0[j].x, x0[j].y, x0[j].z, wt[j], pn, x1[j].z,
                                                  x1[j].w, x2[j].x, tb, db, a);
                        }
                    }
                } else if (wave_any(need_d)) {
                    // zero weight on every ray of the wave: only d(alpha)/d(delta) remains
#pragma unroll
                    for (int j = 0; j < RPT; ++j) {
                        if (PLAIN) {
                            pair_adjoint_offset(q[j], x0[j].x, x0[j].y, x0[j].z, 0.0f, x2[j].z * delta[j], pa);
                        } else {
                            const PairNormal pn{0, 0, 0, 0, 0};
                            pair_adjoint<false>(g, q[j], x0[j].x, x0[j].y, x0[j].z, 0.0f, pn, 0.0f, 0.0f, 0.0f,
                                                0.0f, x2[j].z * delta[j], a);
                        }
                    }
                } else {
                    continue;  // no term of this Gaussian on this wave's rays
                }
                float v[LREC];
                if (PLAIN) {
                    offset_acc_store(pa, v);
                } else {
                    v[0] = a.u0; v[1] = a.u1; v[2] = a.u2; v[3] = a.u3; v[4] = a.u4; v[5] = a.u5;
                    v[6] = a.p0; v[7] = a.p1; v[8] = a.p2; v[9] = a.l;
                }
                if (COLOR) {
                    v[LREC - 3] = aC0; v[LREC - 2] = aC1; v[LREC - 1] = aC2;
                }
#pragma unroll
                for (int c = 0; c < LREC; ++c) v[c] = wave_sum(v[c]);
                if (lane == 0) {
                    float *dst = wsum + (wave * TG + i) * LREC;
#pragma unroll
                    for (int c = 0; c < LREC; ++c) dst[c] += v[c];
                }
            }
        }
        __syncthreads();
        // the tile's partial records: waves summed in order, -(sum rho) mu'^T applied in double
        for (int q = tid; q < cnt; q += BLOCK) {
            float sum[LREC];
#pragma unroll
            for (int c = 0; c < LREC; ++c) sum[c] = wsum[q * LREC + c];
            for (int w = 1; w < NW; ++w) {
#pragma unroll
                for (int c = 0; c < LREC; ++c) sum[c] += wsum[(w * TG + q) * LREC + c];
            }
            const int gg = sr.gauss_off + gb + q;
            if (PLAIN)
                write_partial_offset(partial + item.poff + REC * (gb + q), sum, REC, P.prec + 6 * gg, P.means + 3 * gg, o);
            else
                write_partial(partial + item.poff + REC * (gb + q), sum, REC, P.means + 3 * gg, o);
        }
    }
    // betas: lanes summed over the wave, then the waves in order
    aB1 = wave_sum(aB1);
    aB2 = wave_sum(aB2);
    if (lane == 0) {
        bsum[2 * wave] = aB1;
        bsum[2 * wave + 1] = aB2;
    }
    __syncthreads();
    if (tid < 2) {
        float sb = 0.0f;
        for (int w = 0; w < NW; ++w) sb += bsum[2 * w + tid];
        beta_partial[2 * it + tid] = sb;
    }
}

// ------------------------------------------------------------------------------------
// Backward, tiled ray-lane layout: an item is T ray tiles of
// one view (8 x 8 pixels, see ViewRec) against every Gaussian of its scene.  The item's rays
// are staged in LDS with their adjoint prologue; each wave takes every NW-th Gaussian and walks
// the T tiles with a lane per ray, so a lane sums that Gaussian's terms over T rays before one
// scattered reduction over the wave.  A tile on which the Gaussian's blend weight is exactly
// zero on every ray takes only the density term of alpha, and one whose density is zero too
// adds nothing -- both decided uniformly over the wave (on the 16-scene batch about 58 % and
// 34 % of (tile, Gaussian) pairs).
// ------------------------------------------------------------------------------------

// With a normal cotangent the staged ray is the prologue as ray_prologue writes it (64 bytes) and the
// pair takes the general adjoint of bwd_kernel; items are then 8 tiles.

template <int BLOCK, int T, int TG, int F>
__global__ __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu((F & kNrm) ? 4 : 6))) void bwdt_kernel(
    Params P, BwdIn I, const BwdItem *__restrict__ items, const int *__restrict__ order, float *__restrict__ partial,
    float *__restrict__ beta_partial,
    unsigned long long *__restrict__ masks)
{
    constexpr bool NORMALS = (F & kNrm) != 0, COLOR = (F & kCol) != 0, BIG = (F & kBig) != 0;
    constexpr int NW = BLOCK / 64;
    constexpr int RAYS = 64 * T;
    static_assert(T <= 32 && 64 % T == 0, "a 32-bit mask of the item's ray tiles, whole tile sets per wave");
    constexpr int RW = NORMALS ? 4 : COLOR ? 3 : 2;           // float4 per staged ray
    constexpr int EW = COLOR ? 6 : 5;                         // float4 per staged Gaussian
    constexpr int LREC = (NORMALS ? kPartial : kOffsetAcc) + (COLOR ? 3 : 0);  // sums per Gaussian
    constexpr int REC = COLOR ? kPartialColor : kPartial;     // partial record per Gaussian
    // per ray: (v, M2 + log2 S), (tf_bar, D_bar, dc, t_f) [, (C_bar, C_bar . C)]
    __shared__ float4 rays[RW * RAYS];
    __shared__ float4 tbox[3 * T];            // per ray tile: its box (TileBox)
    __shared__ float tnorm[T];                // per ray tile: least M2 + log2 S over its rays
    __shared__ int tdb[T];                    // per ray tile: 1 if some ray has D_bar != 0, else 0
    __shared__ float4 ents[EW * TG];          // the Gaussian tile's entries (m estimate terms, colour)
    __shared__ float rec[LREC * TG];          // (H, Bv, L) [and the colour sums] of each Gaussian
    __shared__ float bsum[2 * NW];
    // large scenes (kBig): the list of survivors (a ring), the waves' counts of two rounds
    constexpr int LIST = 2 * BLOCK;
    static_assert(TG <= BLOCK, "a round is added to fewer than TG survivors");
    __shared__ int slist[BIG ? LIST : 1];
    __shared__ int wcnt[2][BIG ? NW : 1];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int it = order ? ld_uniform(order + blockIdx.x) : (int)blockIdx.x;
    const BwdItem item = ld_uniform(items + it);
    const ViewRec vr = ld_uniform(P.views + item.view);
    const SceneRec sr = ld_uniform(P.scenes + vr.scene);
    const CamRec cam = cam_of(P, item.view);
    const float *e = cam.e, *kk = cam.k;
    double o[3];
    cam_centre(e, o);
    const float o0 = (float)o[0], o1 = (float)o[1], o2 = (float)o[2];
    const Blend bl = blend_of(P, vr.scene);
    const bool b1_pos = bl.b1 >= 0.0f;  // the weight bound needs beta1 >= 0
    const int nt = min(item.span, vr.tiles - item.ray0);  // the item's tiles: ray0 is its first tile

    constexpr bool sparse = BIG;
    int rb = 0, head = 0, total = sparse ? 0 : sr.n;  // next round, ring position and count of the listed
    // large scenes: the item takes every slots-th 64 Gaussians of the scene, from the g0-th (words of masks)
    const int words = (sr.n + 63) / 64, part_words = sparse ? (words - item.g0 + item.slots - 1) / item.slots : 0;
    // entry q of the Gaussian tile
    auto stage = [&](int q) {
        const int gi = sr.gauss_off + (sparse ? slist[(head + q) & (LIST - 1)] : head + q);
        make_entry_est(P.means + 3 * gi, P.prec + 6 * gi, P.weights[gi], o, &ents[EW * q]);
        if (COLOR) ents[EW * q + 5] = colour_entry(P.colors + 3 * gi);
    };
    // The last threads form the first Gaussian tile's entries beside the rays' prologue, so that their
    // loads and FP64 chain share one wait (pre-culled scenes have no list yet).
    if (!sparse && BLOCK - 1 - tid < min(TG, sr.n)) stage(BLOCK - 1 - tid);
    for (int q = tid; q < RAYS; q += BLOCK) {
        int row = 0, col = 0;
        const int local = (q >> 6) < nt ? tile_local(vr, item.ray0 + (q >> 6), q & 63, row, col) : -1;
        float4 pr[4];
        ray_prologue<F>(P, I, item.view, vr, e, kk, o0, o1, o2, local >= 0 ? local : 0, local >= 0, bl.b1, bl.nc2,
                        pr, local >= 0 ? row : 0, col);
        if (NORMALS) {
#pragma unroll
            for (int k = 0; k < 4; ++k) rays[RW * q + k] = pr[k];
            continue;
        }
        // the weight 2^(z2 - M2) / S as 2^(z2 - M2 - log2 S); a ray past the edge has M2 = inf, S = inf
        rays[RW * q] = make_float4(pr[0].x, pr[0].y, pr[0].z, pr[0].w - __builtin_amdgcn_logf(pr[1].x));
        rays[RW * q + 1] = make_float4(pr[1].y, pr[2].z, pr[3].w, pr[2].w);
        if (COLOR) {
            // the colour cotangent and its product with the blended colour (kappa's colour part)
            float kc = 0.0f;
            if (local >= 0) {
                const size_t r3 = 3 * ((size_t)vr.ray_off + local);
                kc = fmaf(pr[3].x, I.color[r3], fmaf(pr[3].y, I.color[r3 + 1], pr[3].z * I.color[r3 + 2]));
            }
            rays[RW * q + 2] = make_float4(pr[3].x, pr[3].y, pr[3].z, kc);
        }
    }
    __syncthreads();
    // each ray tile's box and least normaliser, for the bound that lets a wave pass over the tiles
    // on which a Gaussian can neither weigh above FP32's zero nor add a density above
    // 2^kDensSkipLog2 (tile_bounds)
    for (int tt = wave; tt < nt; tt += NW) {
        int row, col;
        const bool ok = tile_local(vr, item.ray0 + tt, lane, row, col) >= 0;
        const float4 x0 = rays[RW * (64 * tt + lane)];
        const float dbar = NORMALS ? rays[RW * (64 * tt + lane) + 2].z : rays[RW * (64 * tt + lane) + 1].y;
        const int db_flag = wave_any(dbar != 0.0f) ? 1 : 0;
        const TileBox b = wave_box(x0.x, x0.y, x0.z, ok, e);
        const float norm = NORMALS ? x0.w - __builtin_amdgcn_logf(rays[RW * (64 * tt + lane) + 1].x) : x0.w;
        const float nmin = wave_min_u(ok ? norm : INFINITY);
        if (lane == 0) {
            tbox[3 * tt] = b.c;
            tbox[3 * tt + 1] = b.x;
            tbox[3 * tt + 2] = b.y;
            tnorm[tt] = nmin;
            tdb[tt] = db_flag;
        }
    }
    float aB1 = 0.0f, aB2 = 0.0f;
    // Each Gaussian of a large scene is first bounded on the whole item (tile_bounds on a box around
    // all its tiles, against their least normaliser), BLOCK of them a round, and only those that
    // can matter on some tile are listed, in scene order, and staged TG at a time; the others'
    // records would be zero, as the per-tile bounds would have left them, and are not written: a
    // bit per Gaussian (masks) tells the finalize which of the item's records are.  Rounds go on
    // until the list fills a staged tile.  Smaller scenes stage all their Gaussians in order.
    TileBox ibox;
    for (bool first = true; ; first = false) {
      if (sparse && rb < part_words && total < TG) {
        if (first) __syncthreads();  // boxes visible
        float inorm = INFINITY;
        for (int t = 0; t < nt; ++t) inorm = fminf(inorm, tnorm[t]);
        if (first) ibox = wave_box_of(tbox, nt, lane, e);
        do {
            const int word = item.g0 + item.slots * (rb + wave), gl = 64 * word + lane, par = (rb / NW) & 1;
            bool keep = false;
            if (gl < sr.n) {
                const int gg = sr.gauss_off + gl;
                Ent ge;
                float4 ee;
                make_bound_entry(P.means + 3 * gg, P.prec + 6 * gg, P.weights[gg], o, ge, ee);
                const PairBounds pb = tile_bounds(ge, ee, ibox, bl.hm, bl.b1, bl.nc2);
                // (written so that a NaN bound keeps the Gaussian)
                keep = !(b1_pos && pb.z_hi - inorm < kSkipLog2 && pb.d2_hi < kDensSkipLog2);
            }
            const unsigned long long bal = wave_ballot(keep);
            if (lane == 0) {
                wcnt[par][wave] = __popcll(bal);
                if (word < words) masks[item.moff + word] = bal;
            }
            __syncthreads();
            int off = head + total;
            for (int w = 0; w < NW; ++w) {
                const int c = wcnt[par][w];
                off += w < wave ? c : 0;
                total += c;
            }
            if (keep) slist[(off + __popcll(bal & ((1ull << lane) - 1ull))) & (LIST - 1)] = gl;
            rb += NW;
        } while (rb < part_words && total < TG);
      }
      if (total == 0) break;
      {
        const int cnt = min(TG, total);
        if (!first || sparse) {
            __syncthreads();  // the list visible; the previous tile's entries and sums are consumed
            for (int q = tid; q < cnt; q += BLOCK) stage(q);
        }
        __syncthreads();
        // The wave takes Gaussians i0, i0 + NW, ... and bounds GPB of them on the item's tiles in
        // one pass (lane: tile lane % T of Gaussian i0 + (lane / T) NW), then walks them in order.
        constexpr int GPB = 64 / T;
        for (int i0 = wave; i0 < cnt; i0 += GPB * NW) {
          unsigned long long tmasks;  // bits [T k, T k + T): the tiles Gaussian i0 + k NW can matter on
          {
            const int ik = i0 + (lane / T) * NW, tl = lane % T;
            bool need = false;
            if (tl < nt && ik < cnt) {
                const Ent gk = ent_from(ents[EW * ik], ents[EW * ik + 1], ents[EW * ik + 2], ents[EW * ik + 3]);
                const PairBounds pb = tile_bounds(gk, ents[EW * ik + 4], TileBox{tbox[3 * tl], tbox[3 * tl + 1], tbox[3 * tl + 2]},
                                                  bl.hm, bl.b1, bl.nc2);
                // (written so that a NaN bound keeps the tile)
                need = !(b1_pos && pb.z_hi - tnorm[tl] < kSkipLog2 && (pb.d2_hi < kDensSkipLog2 || tdb[tl] == 0));
            }
            tmasks = wave_ballot(need);
          }
          for (int k = 0; k < GPB; ++k) {
            const int i = i0 + k * NW;
            if (i >= cnt) break;
            unsigned tmask = (unsigned)(tmasks >> (T * k));
            if (T < 32) tmask &= (1u << (T % 32)) - 1u;
            if (tmask == 0u) {
                // no tile of the item takes a term of this Gaussian: its sums are zero
                if (lane < LREC) rec[LREC * i + lane] = 0.0f;
                continue;
            }
            const Ent g = ent_from(ents[EW * i], ents[EW * i + 1], ents[EW * i + 2], ents[EW * i + 3]);
            float4 cc = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            if (COLOR) cc = ents[EW * i + 5];
            OffsetAcc acc;
            PairAcc nacc;
            float aC0 = 0.0f, aC1 = 0.0f, aC2 = 0.0f;  // colour sums: wt C_bar
#pragma unroll 1
            while (tmask) {
                const int t = __builtin_ctz(tmask);
                tmask &= tmask - 1;
                const float4 x0 = rays[RW * (64 * t + lane)], x1 = rays[RW * (64 * t + lane) + 1];
                Geo q;
                if (NORMALS) {
                    pair_geo(g, x0.x, x0.y, x0.z, bl.hm, bl.b1, bl.nc2, q);
                    const float4 x2 = rays[RW * (64 * t + lane) + 2];
                    const float delta = exp2_(q.d2), dd = x2.z * delta;
                    const float zr = q.z2 - x0.w;
                    if (wave_any(!(zr < kSkipLog2))) {  // (a NaN weight shows in the sums)
                        const float4 x3 = rays[RW * (64 * t + lane) + 3];
                        const float wt = exp2_(zr) * x1.x;  // normalised blend weight
                        const float tfb = x1.y;
                        const PairNormal pn = pair_normal(g, q, x1.z, x1.w, x2.x);
                        // z_bar = wt (tf_bar t + Nb.n + Cb.c - kappa)
                        float lin = fmaf(tfb, q.t, pn.nN);
                        if (COLOR) {
                            lin = fmaf(x3.x, cc.x, fmaf(x3.y, cc.y, fmaf(x3.z, cc.z, lin)));
                            aC0 = fmaf(wt, x3.x, aC0);
                            aC1 = fmaf(wt, x3.y, aC1);
                            aC2 = fmaf(wt, x3.z, aC2);
                        }
                        const float zb = wt * (lin - x2.y);
                        const float tb = fmaf(-bl.cb, zb, wt * tfb);
                        const float db = fmaf(bl.b1, zb, dd);
                        aB1 = fmaf(zb, q.d2 - x3.w, aB1);
                        aB2 = fmaf(zb, q.t - x2.w, aB2);
                        pair_adjoint<true>(g, q, x0.x, x0.y, x0.z, wt, pn, x1.z, x1.w, x2.x, tb, db, nacc);
                    } else {
                        const PairNormal pn{0, 0, 0, 0, 0};
                        pair_adjoint<false>(g, q, x0.x, x0.y, x0.z, 0.0f, pn, 0.0f, 0.0f, 0.0f, 0.0f, dd, nacc);
                    }
                    continue;
                }
                pair_geo_coarse(g, x0.x, x0.y, x0.z, bl.hm, bl.b1, bl.nc2, q);
                // log2 of the normalised weight, and the density term D_bar delta
                const float zr = fmaf(bl.b1, q.d2, fmaf(bl.nc2, q.t, -x0.w));
                // a weight below 2^-150 rounds to zero in FP32, and a density below 2^kDensSkipLog2
                // adds nothing measurable: such a tile skips the exponential and the adjoint
                // (the density test only where no weight is left)
                const bool any_w = wave_any(zr >= kSkipLog2);
                if (any_w || wave_any(q.d2 >= kDensSkipLog2 && x1.y != 0.0f)) {
                    const float dd = x1.y * exp2_(q.d2);
                    // with zero weights on every ray of the tile only the density term remains:
                    // t_bar = 0, d_bar = D_bar delta (the offset form then adds exactly that)
                    float tb = 0.0f, db = dd;
                    if (any_w) {
                        // z_bar = wt (tf_bar t - kappa) with kappa = tf_bar t_f [+ C_bar . C, and
                        // C_bar . c added to the pair's share]
                        const float x = q.t - x1.w;
                        const float wt = exp2_(zr);
                        const float wtf = wt * x1.x;
                        float zb = wtf * x;
                        if (COLOR) {
                            const float4 x2 = rays[RW * (64 * t + lane) + 2];
                            zb = fmaf(wt, fmaf(x2.x, cc.x, fmaf(x2.y, cc.y, fmaf(x2.z, cc.z, -x2.w))), zb);
                            aC0 = fmaf(wt, x2.x, aC0);
                            aC1 = fmaf(wt, x2.y, aC1);
                            aC2 = fmaf(wt, x2.z, aC2);
                        }
                        tb = fmaf(-bl.cb, zb, wtf);
                        db = fmaf(bl.b1, zb, dd);
                        aB1 = fmaf(zb, q.d2 - x1.z, aB1);
                        aB2 = fmaf(zb, x, aB2);
                    }
                    // one accumulation for both cases, so the sums stay in their registers
                    pair_adjoint_offset(q, x0.x, x0.y, x0.z, tb, db, acc);
                }
            }
            float v[16];
            constexpr int C0 = NORMALS ? kPartial : kOffsetAcc;
            static_assert(kOffsetAcc + 3 <= 16, "one 16-value wave sum per Gaussian");
            if (NORMALS) {
                v[0] = nacc.u0; v[1] = nacc.u1; v[2] = nacc.u2; v[3] = nacc.u3; v[4] = nacc.u4; v[5] = nacc.u5;
                v[6] = nacc.p0; v[7] = nacc.p1; v[8] = nacc.p2; v[9] = nacc.l;
                v[13] = v[14] = v[15] = 0.0f;
            } else {
                offset_acc_store(acc, v);
            }
            v[C0] = aC0;
            v[C0 + 1] = aC1;
            v[C0 + 2] = aC2;
            const float tot = wave_sum16(v, lane);
            const int idx = wave16_index(lane);
            if ((lane & 3) == 0 && idx < LREC) rec[LREC * i + idx] = tot;
          }
        }
        __syncthreads();
        for (int q = tid; q < cnt; q += BLOCK) {
            const int gl = sparse ? slist[(head + q) & (LIST - 1)] : head + q;
            const int gg = sr.gauss_off + gl;
            if (NORMALS)
                write_partial(partial + item.poff + REC * gl, rec + LREC * q, REC, P.means + 3 * gg, o);
            else
                write_partial_offset(partial + item.poff + REC * gl, rec + LREC * q, REC,
                                     P.prec + 6 * gg, P.means + 3 * gg, o);
        }
        head += cnt;
        total -= cnt;
      }
    }
    // betas: lanes summed over the wave, then the waves in order
    aB1 = wave_sum(aB1);
    aB2 = wave_sum(aB2);
    if (lane == 0) {
        bsum[2 * wave] = aB1;
        bsum[2 * wave + 1] = aB2;
    }
    __syncthreads();
    if (tid < 2) {
        float sb = 0.0f;
        for (int w = 0; w < NW; ++w) sb += bsum[2 * w + tid];
        beta_partial[2 * it + tid] = sb;
    }
}

// ------------------------------------------------------------------------------------
// Finalize, deterministic, in one stage (fin_one_kernel) or two.
//   stage 1: each group of <= kGroupItems consecutive items of a chunk is summed in item
//            order in FP64 (all values of the chunk's partial record, and the betas);
//   stage 2: each chunk sums its groups in order, maps the peak-depth adjoint to the means
//            (dL/dmu = -U^T sum rho), the log-weight adjoint to the weights
//            (dL/dlambda = dL/dlog(lambda) / lambda), and the first chunk of a scene
//            reduces the scene's betas.
// ------------------------------------------------------------------------------------

// Sum n strided values src[0], src[stride], ... in index order (FP64), issuing the loads
// eight at a time so that they are in flight together; the association is fixed.
template <typename T>
__device__ __forceinline__ double ordered_sum(const T *__restrict__ src, int n, size_t stride)
{
    double s = 0.0;
    int i = 0;
    for (; i + 8 <= n; i += 8) {
        T x[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) x[k] = src[(i + k) * stride];
#pragma unroll
        for (int k = 0; k < 8; ++k) s += (double)x[k];
    }
    for (; i < n; ++i) s += (double)src[i * stride];
    return s;
}

// Gradients of Gaussian gg from its summed record sm.
__device__ __forceinline__ void fin_write(const Params &P, int gg, const double *sm, int rec, float *__restrict__ g_means,
                                          float *__restrict__ g_prec, float *__restrict__ g_weights,
                                          float *__restrict__ g_colors)
{
    const float *u = P.prec + 6 * gg;
    float *gp = g_prec + 6 * gg;
#pragma unroll
    for (int c = 0; c < 6; ++c) gp[c] = (float)sm[c];
    const double r0 = sm[6], r1 = sm[7], r2 = sm[8];
    g_means[3 * gg + 0] = (float)(-(double)u[0] * r0);
    g_means[3 * gg + 1] = (float)(-((double)u[1] * r0 + (double)u[3] * r1));
    g_means[3 * gg + 2] = (float)(-((double)u[2] * r0 + (double)u[4] * r1 + (double)u[5] * r2));
    g_weights[gg] = (float)(sm[9] / (double)P.weights[gg]);
    if (rec == kPartialColor && g_colors) {
        // colour = sigmoid(q): dL/dq = dL/dc c (1 - c)
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const double col = 1.0 / (1.0 + exp(-(double)P.colors[3 * gg + c]));
            g_colors[3 * gg + c] = (float)(sm[10 + c] * col * (1.0 - col));
        }
    }
}

// beta1_bar = sum z_bar d (d = d2 / log2 e); beta2_bar = -sum z_bar t / eta
__device__ __forceinline__ void fin_write_beta(const Params &P, int scene, int k, double sb, float *__restrict__ g_betas)
{
    g_betas[2 * scene + k] = k == 0 ? (float)(sb / kLog2e) : (float)(-sb / (double)P.eta[scene]);
}

// One stage, for scenes of at most kOneStageItems items: block (task, slice) sums the records of a
// few Gaussians (and, with the first, the betas) over all items.  Thread (k, v) of 32 x 32 adds value v of
// items k, k + 32, ... in order, then a fixed tree adds the k: one launch with every load of a value
// in flight, where the two stages below took two launches of 5 us each on small jobs (their reads of
// a few items per thread leave nothing to hide the latency).
__global__ __launch_bounds__(1024) void fin_one_kernel(Params P, const FinTask *__restrict__ tasks,
                                                       const float *__restrict__ partial,
                                                       const float *__restrict__ beta_partial, float *__restrict__ g_means,
                                                       float *__restrict__ g_prec, float *__restrict__ g_weights,
                                                       float *__restrict__ g_colors, float *__restrict__ g_betas)
{
    __shared__ double sums[32][32];
    const FinTask task = tasks[blockIdx.x];
    const int per = fin_one_gauss(task.rec), g_lo = blockIdx.y * per;
    if (g_lo >= task.gc) return;
    const int ng = min(per, task.gc - g_lo), nv = ng * task.rec;
    const int v = threadIdx.x & 31, k = threadIdx.x >> 5;
    const int nval = task.gc * task.rec, n = task.item_end - task.item_begin;
    const int nk = n > k ? (n - k + 31) / 32 : 0;  // items k, k + 32, ...
    const bool beta = v >= 30 && blockIdx.y == 0 && task.beta;
    double s = 0.0;
    if (v < nv)
        s = ordered_sum(partial + task.poff + (size_t)k * nval + g_lo * task.rec + v, nk, (size_t)32 * nval);
    else if (beta)
        s = ordered_sum(beta_partial + 2 * (task.item_begin + k) + v - 30, nk, (size_t)64);
    sums[k][v] = s;
    __syncthreads();
#pragma unroll
    for (int h = 16; h > 0; h >>= 1) {
        if (k < h) sums[k][v] += sums[k + h][v];
        __syncthreads();
    }
    if (threadIdx.x < ng)
        fin_write(P, P.scenes[task.scene].gauss_off + task.g0 + g_lo + threadIdx.x, &sums[0][task.rec * threadIdx.x], task.rec,
                  g_means, g_prec, g_weights, g_colors);
    if (k == 0 && beta) fin_write_beta(P, task.scene, v - 30, sums[0][v], g_betas);
}

// First stage: block (group, slice) sums the values slice * BLOCK + tid, + BLOCK * slices, ...
// of a group's records (a record of a whole large scene spreads over many blocks).
template <int BLOCK>
__global__ __launch_bounds__(BLOCK) void fin1_kernel(const FinGroup *__restrict__ groups,
                                                    const float *__restrict__ partial,
                                                    const float *__restrict__ beta_partial,
                                                    double *__restrict__ stage, double *__restrict__ stage_beta)
{
    const FinGroup gr = groups[blockIdx.x];
    const int tid = threadIdx.x;
    const int n = gr.item_end - gr.item_begin;
    for (int v = blockIdx.y * BLOCK + tid; v < gr.nval; v += BLOCK * gridDim.y)
        stage[gr.soff + v] = ordered_sum(partial + gr.poff + v, n, gr.nval);
    if (blockIdx.y == 0 && tid < 2)
        stage_beta[2 * blockIdx.x + tid] = ordered_sum(beta_partial + 2 * gr.item_begin + tid, n, 2);
}

// First stage of large scenes' items (FinGroup::words: 64-bit words of the items' masks): a lane per
// Gaussian sums, in item order, the records that the items wrote.  An item of 16 tiles touches a few
// per cent of 10 000 clustered Gaussians, so the stage reads the masks and little else: 197 -> 42 us for
// one 1920 x 1080 view, whose 0.8 GB of records were all written and read before.
template <int BLOCK, int REC>
__device__ __forceinline__ void fin1_sparse(const FinGroup &gr, const unsigned long long *__restrict__ masks,
                                            const float *__restrict__ partial, double *__restrict__ stage, double *sums)
{
    const int lane = threadIdx.x & 63, gc = gr.nval / REC;
    for (int base = blockIdx.y * BLOCK + (threadIdx.x & ~63); base < gc; base += BLOCK * gridDim.y) {
        const unsigned long long *mw = masks + gr.moff + base / 64;
        const float *rp = partial + gr.poff + REC * (base + lane);
        const int n = (gr.item_end - gr.item_begin) / gr.parts;
        double s[REC];
#pragma unroll
        for (int c = 0; c < REC; ++c) s[c] = 0.0;
        for (int i0 = 0; i0 < n; i0 += 64) {
            // lane l holds the word of item i0 + l
            const unsigned long long own = i0 + lane < n ? mw[(size_t)(i0 + lane) * gr.words] : 0ull;
            unsigned long long any = wave_ballot(own != 0ull);
            // Four items' records in flight, added in item order.  A lane whose record was not written
            // loads the buffer's first one instead (one cache line for all of them) and adds zero, so
            // that the loads take no branch.
            while (any) {
                float x[4][REC];
                bool mine[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int k = any ? __builtin_ctzll(any) : 0;
                    const unsigned lo = __builtin_amdgcn_readlane((unsigned)own, k), hi = __builtin_amdgcn_readlane((unsigned)(own >> 32), k);
                    mine[u] = any && base + lane < gc && ((((unsigned long long)hi << 32) | lo) >> lane & 1ull);
                    any &= any - 1;
                    const float *r = mine[u] ? rp + (size_t)(i0 + k) * gr.nval : partial;
#pragma unroll
                    for (int c = 0; c < REC; ++c) x[u][c] = r[c];
                }
#pragma unroll
                for (int u = 0; u < 4; ++u)
#pragma unroll
                    for (int c = 0; c < REC; ++c) s[c] += mine[u] ? (double)x[u][c] : 0.0;
            }
        }
        // through LDS, so that the wave writes its sums in one contiguous run
#pragma unroll
        for (int c = 0; c < REC; ++c) sums[REC * lane + c] = s[c];
        __builtin_amdgcn_wave_barrier();
        const int nv = REC * min(64, gc - base);
        for (int v = lane; v < nv; v += 64) stage[gr.soff + REC * base + v] = sums[v];
        __builtin_amdgcn_wave_barrier();
    }
}

template <int BLOCK>
__global__ __launch_bounds__(BLOCK) void fin1s_kernel(const FinGroup *__restrict__ groups, const float *__restrict__ partial,
                                                     const float *__restrict__ beta_partial,
                                                     const unsigned long long *__restrict__ masks, int rec,
                                                     double *__restrict__ stage, double *__restrict__ stage_beta)
{
    __shared__ double sums[BLOCK / 64][64 * kPartialColor];
    const FinGroup gr = groups[blockIdx.x];
    if (gr.words == 0) {  // a small scene's: every record is written
        const int n = gr.item_end - gr.item_begin;
        for (int v = blockIdx.y * BLOCK + threadIdx.x; v < gr.nval; v += BLOCK * gridDim.y)
            stage[gr.soff + v] = ordered_sum(partial + gr.poff + v, n, gr.nval);
    } else if (rec == kPartial)
        fin1_sparse<BLOCK, kPartial>(gr, masks, partial, stage, sums[threadIdx.x >> 6]);
    else
        fin1_sparse<BLOCK, kPartialColor>(gr, masks, partial, stage, sums[threadIdx.x >> 6]);
    if (blockIdx.y == 0 && threadIdx.x < 2)
        stage_beta[2 * blockIdx.x + threadIdx.x] =
            ordered_sum(beta_partial + 2 * gr.item_begin + threadIdx.x, gr.item_end - gr.item_begin, 2);
}

// Second stage: block (task, slice) finishes kFinSlice Gaussians of a chunk.
constexpr int kFinSlice = 25;

template <int BLOCK>
__global__ __launch_bounds__(BLOCK) void fin2_kernel(Params P, const FinTask *__restrict__ tasks,
                                                    const FinGroup *__restrict__ groups,
                                                    const double *__restrict__ stage,
                                                    const double *__restrict__ stage_beta,
                                                    float *__restrict__ g_means, float *__restrict__ g_prec,
                                                    float *__restrict__ g_weights, float *__restrict__ g_colors,
                                                    float *__restrict__ g_betas)
{
    __shared__ double sums[kFinSlice * kPartialColor];
    const FinTask task = tasks[blockIdx.x];
    const int g_lo = blockIdx.y * kFinSlice;
    if (g_lo >= task.gc) return;
    const int ng = min(kFinSlice, task.gc - g_lo);
    const int rec = task.rec;
    const SceneRec sr = P.scenes[task.scene];
    const int tid = threadIdx.x;
    for (int tv = tid; tv < ng * rec; tv += BLOCK) {
        const int v = g_lo * rec + tv;
        double s = 0.0;
        int gi = task.group_begin;
        for (; gi + 8 <= task.group_end; gi += 8) {
            double x[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) x[k] = stage[groups[gi + k].soff + v];
#pragma unroll
            for (int k = 0; k < 8; ++k) s += x[k];
        }
        for (; gi < task.group_end; ++gi) s += stage[groups[gi].soff + v];
        sums[tv] = s;
    }
    __syncthreads();
    if (tid < ng) fin_write(P, sr.gauss_off + task.g0 + g_lo + tid, sums + rec * tid, rec, g_means, g_prec, g_weights, g_colors);
    if (task.beta && blockIdx.y == 0 && tid < 2) {
        const double sb = ordered_sum(stage_beta + 2 * task.sgroup_begin + tid, task.sgroup_end - task.sgroup_begin, 2);
        fin_write_beta(P, task.scene, tid, sb, g_betas);
    }
}

// ------------------------------------------------------------------------------------
// Split statistic (Sec. 8): lbar_i = (1/M) sum_j L_j w_ji over a scene's M rays, w_ji the
// normalised blend weights of Eq. (3) (Eq. 7 here), read back from the forward pass's stash.
// Tiled like the backward (bwdt_kernel): an item is T ray tiles of one view against every
// Gaussian of its scene.  The rays are staged in LDS with M2 + log2 S (so that z2 minus it is the
// log2 of the normalised weight) and their loss value; each wave bounds GPB Gaussians at a time on
// the item's tiles (tile_bounds against the tile's least M2 + log2 S) and, for each Gaussian, sums
// L w over the rays of the tiles where some weight can be above FP32's zero, then reduces over the
// wave into the item's record of one float per Gaussian.  Bound by instruction issue: a bound per
// pair after the tile's found too little to skip to pay for itself (16 scenes, 12.6e6 rays:
// 224 us with it, 217 without).
// ------------------------------------------------------------------------------------

template <int BLOCK, int T, int TG>
__global__ __launch_bounds__(BLOCK) void statt_kernel(Params P, const float *__restrict__ loss,
                                                     const float *__restrict__ stash,
                                                     const BwdItem *__restrict__ items, float *__restrict__ partial)
{
    static_assert(T <= 32 && 64 % T == 0, "a 32-bit mask of the item's ray tiles, whole tile sets per wave");
    constexpr int NW = BLOCK / 64, RAYS = 64 * T, GPB = 64 / T;
    __shared__ float4 rays[RAYS];   // per ray: (v, M2 + log2 S)
    __shared__ float lossv[RAYS];   // per ray: its loss value
    __shared__ float4 tbox[3 * T];  // per ray tile: its box (TileBox)
    __shared__ float tnorm[T];      // per ray tile: least M2 + log2 S over its rays
    __shared__ float4 ents[5 * TG];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const BwdItem item = ld_uniform(items + blockIdx.x);
    const ViewRec vr = ld_uniform(P.views + item.view);
    const SceneRec sr = ld_uniform(P.scenes + vr.scene);
    const CamRec cam = cam_of(P, item.view);
    const float *e = cam.e, *kk = cam.k;
    double o[3];
    cam_centre(e, o);
    const Blend bl = blend_of(P, vr.scene);
    const bool b1_pos = bl.b1 >= 0.0f;  // the weight bounds need beta1 >= 0
    const int nt = min(T, vr.tiles - item.ray0);  // the item's tiles: ray0 is its first tile

    auto stage = [&](int gb, int q) {
        const int gi = sr.gauss_off + gb + q;
        make_entry_est(P.means + 3 * gi, P.prec + 6 * gi, P.weights[gi], o, &ents[5 * q]);
    };
    // (the first Gaussian tile beside the rays, as in the backward)
    if (BLOCK - 1 - tid < min(TG, sr.n)) stage(0, BLOCK - 1 - tid);
    for (int q = tid; q < RAYS; q += BLOCK) {
        int row = 0, col = 0;
        const int local = (q >> 6) < nt ? tile_local(vr, item.ray0 + (q >> 6), q & 63, row, col) : -1;
        float v0 = 0.0f, v1 = 0.0f, v2 = 1.0f, wo = INFINITY, lr = 0.0f;  // a ray past the edge weighs 0
        if (local >= 0) {
            tile_ray_dir(P, vr, e, kk, local, row, col, v0, v1, v2);
            const size_t r = (size_t)vr.ray_off + local;
            const float4 s0 = reinterpret_cast<const float4 *>(stash)[2 * r];
            wo = s0.x - __builtin_amdgcn_logf(s0.y);  // M2 + log2 S (s0.y = 1 / S)
            lr = loss[r];
        }
        rays[q] = make_float4(v0, v1, v2, wo);
        lossv[q] = lr;
    }
    __syncthreads();
    for (int tt = wave; tt < nt; tt += NW) {
        int row, col;
        const bool ok = tile_local(vr, item.ray0 + tt, lane, row, col) >= 0;
        const float4 x0 = rays[64 * tt + lane];
        const TileBox b = wave_box(x0.x, x0.y, x0.z, ok, e);
        const float nmin = wave_min_u(ok ? x0.w : INFINITY);
        if (lane == 0) {
            tbox[3 * tt] = b.c;
            tbox[3 * tt + 1] = b.x;
            tbox[3 * tt + 2] = b.y;
            tnorm[tt] = nmin;
        }
    }
    float *__restrict__ out = partial + item.poff;
    for (int gb = 0; gb < sr.n; gb += TG) {
        const int cnt = min(TG, sr.n - gb);
        if (gb > 0) {
            __syncthreads();  // the previous tile's entries are consumed
            for (int q = tid; q < cnt; q += BLOCK) stage(gb, q);
        }
        __syncthreads();  // staged rays, boxes and entries visible
        for (int i0 = wave; i0 < cnt; i0 += GPB * NW) {
            unsigned long long tmasks;  // bits [T k, T k + T): the tiles Gaussian i0 + k NW can weigh on
            {
                const int ik = i0 + (lane / T) * NW, tl = lane % T;
                bool need = false;
                if (tl < nt && ik < cnt) {
                    const Ent gk = ent_from(ents[5 * ik], ents[5 * ik + 1], ents[5 * ik + 2], ents[5 * ik + 3]);
                    const PairBounds pb = tile_bounds(gk, ents[5 * ik + 4], TileBox{tbox[3 * tl], tbox[3 * tl + 1], tbox[3 * tl + 2]},
                                                      bl.hm, bl.b1, bl.nc2);
                    // (written so that a NaN bound keeps the tile)
                    need = !(b1_pos && pb.z_hi - tnorm[tl] < kSkipLog2);
                }
                tmasks = wave_ballot(need);
            }
            for (int k = 0; k < GPB; ++k) {
                const int i = i0 + k * NW;
                if (i >= cnt) break;
                unsigned tmask = (unsigned)(tmasks >> (T * k));
                if (T < 32) tmask &= (1u << (T % 32)) - 1u;
                float acc = 0.0f;
                if (tmask != 0u) {
                    const Ent g = ent_from(ents[5 * i], ents[5 * i + 1], ents[5 * i + 2], ents[5 * i + 3]);
#pragma unroll 1
                    while (tmask) {
                        const int t = __builtin_ctz(tmask);
                        tmask &= tmask - 1;
                        const float4 x0 = rays[64 * t + lane];
                        Geo q;
                        pair_geo_coarse(g, x0.x, x0.y, x0.z, bl.hm, bl.b1, bl.nc2, q);
                        const float zr = fmaf(bl.b1, q.d2, fmaf(bl.nc2, q.t, -x0.w));
                        if (zr >= kSkipLog2) acc = fmaf(lossv[64 * t + lane], exp2_(zr), acc);
                    }
                    acc = wave_sum(acc);
                }
                if (lane == 0) out[gb + i] = acc;
            }
        }
    }
}

// lbar of one Gaussian of a (scene, chunk) per block: thread j adds the partial sums of items
// j, j + 256, ... in double, then a fixed tree over the threads, divided by the scene's ray
// count (the same order on every call).
__global__ __launch_bounds__(256) void stat_fin_kernel(Params P, const StatTask *__restrict__ tasks,
                                                      const BwdItem *__restrict__ items,
                                                      const float *__restrict__ partial,
                                                      const int64_t *__restrict__ rays_per_scene,
                                                      float *__restrict__ lbar)
{
    __shared__ double red[256];
    const StatTask t = tasks[blockIdx.x];
    const int g = blockIdx.y;
    if (g >= t.gc) return;  // uniform over the block
    double s = 0.0;
    for (int it = t.item_begin + (int)threadIdx.x; it < t.item_end; it += 256)
        s += (double)partial[items[it].poff + g];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
        if ((int)threadIdx.x < h) red[threadIdx.x] += red[threadIdx.x + h];
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        const SceneRec sr = P.scenes[t.scene];
        lbar[sr.gauss_off + t.g0 + g] = (float)(red[0] / (double)rays_per_scene[t.scene]);
    }
}

// Gradient of the Sec. 4 reconstruction loss (mask BCE, mask-weighted L1 depth, mask-weighted
// flow term) with respect to one render's outputs; per-block loss partials in fixed order.
constexpr int kLossBlock = 1024;

__global__ __launch_bounds__(kLossBlock) void loss_kernel(int p, const float *__restrict__ depth,
                                                         const float *__restrict__ alpha,
                                                         const float *__restrict__ flow,
                                                         const float *__restrict__ color,
                                                         const float *__restrict__ depth_t,
                                                         const float *__restrict__ alpha_t,
                                                         const float *__restrict__ flow_t,
                                                         const float *__restrict__ color_t, float w_depth,
                                                         float w_flow, int flow_norm, int flow_cols,
                                                         float w_color, float *__restrict__ g_depth, float *__restrict__ g_alpha,
                                                         float *__restrict__ g_flow, float *__restrict__ g_color,
                                                         float *__restrict__ block_loss)
{
    __shared__ float red[kLossBlock / 64];
    // 64-bit ray index: the products flow_cols r and 3 r overflow int above 5.4e8 rays
    const int64_t r = (int64_t)blockIdx.x * kLossBlock + threadIdx.x;
    const float inv_p = 1.0f / (float)p;
    float l = 0.0f;
    if (r < p) {
        const float at = alpha_t[r];
        const float a = alpha[r];
        const float ac = fminf(fmaxf(a, 1e-6f), 1.0f - 1e-6f);
        const float dd = depth[r] - depth_t[r];
        float ga, gd;
        loss_grad_ray(a, at, depth[r], depth_t[r], w_depth, inv_p, ga, gd);
        g_alpha[r] = ga;
        g_depth[r] = gd;
        l = -(at * logf(ac) + (1.0f - at) * logf(1.0f - ac)) + w_depth * at * fabsf(dd);
        if (flow) {
            for (int c = 0; c < flow_cols; ++c) {
                const float f = flow[flow_cols * r + c] - flow_t[flow_cols * r + c];
                if (flow_norm == 1) {
                    g_flow[flow_cols * r + c] = w_flow * at * (float)((f > 0.0f) - (f < 0.0f)) * inv_p;
                    l += w_flow * at * fabsf(f);
                } else {
                    g_flow[flow_cols * r + c] = 2.0f * w_flow * at * f * inv_p;
                    l += w_flow * at * f * f;
                }
            }
        }
        if (color) {
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const float dc = color[3 * r + c] - color_t[3 * r + c];
                g_color[3 * r + c] = w_color * at * (float)((dc > 0.0f) - (dc < 0.0f)) * inv_p;
                l += w_color * at * fabsf(dc);
            }
        }
        l *= inv_p;
    }
    if (block_loss) {
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) l += __shfl_xor(l, off, 64);
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = l;
        __syncthreads();
        if (threadIdx.x == 0) {
            float s = 0.0f;
            for (int k = 0; k < kLossBlock / 64; ++k) s += red[k];
            block_loss[blockIdx.x] = s;
        }
    }
}

hipError_t launch_loss(int p, const float *depth, const float *alpha, const float *flow, const float *color,
                       const float *depth_t, const float *alpha_t, const float *flow_t, const float *color_t,
                       float w_depth, float w_flow, int flow_norm, int flow_cols, float w_color, float *g_depth,
                       float *g_alpha, float *g_flow, float *g_color, float *block_loss, hipStream_t st)
{
    hipLaunchKernelGGL(loss_kernel, dim3((p + kLossBlock - 1) / kLossBlock), dim3(kLossBlock), 0, st, p, depth, alpha,
                       flow, color, depth_t, alpha_t, flow_t, color_t, w_depth, w_flow, flow_norm, flow_cols, w_color, g_depth,
                       g_alpha, g_flow, g_color, block_loss);
    return hipGetLastError();
}

__global__ void fill_int_kernel(int *p, int n, int value)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = value;
}

// Parameter validation: bit 1 non-finite, 2 weight <= 0, 4 zero diagonal of U, 8 bad beta.
__global__ void validate_kernel(Params P, int n_total, int n_scenes, int *flags)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    int f = 0;
    if (i < n_total) {
        for (int a = 0; a < 3; ++a)
            if (!isfinite(P.means[3 * i + a])) f |= 1;
        for (int a = 0; a < 6; ++a)
            if (!isfinite(P.prec[6 * i + a])) f |= 1;
        const float w = P.weights[i];
        if (!isfinite(w)) f |= 1;
        if (!(w > 0.0f)) f |= 2;
        if (P.prec[6 * i] == 0.0f || P.prec[6 * i + 3] == 0.0f || P.prec[6 * i + 5] == 0.0f) f |= 4;
    }
    if (i < n_scenes) {
        if (!isfinite(P.betas[2 * i]) || !isfinite(P.betas[2 * i + 1])) f |= 8;
    }
    if (f) atomicOr(flags, f);
}

// ------------------------------------------------------------------------------------
// Launchers
// ------------------------------------------------------------------------------------

constexpr int kBlock = 256;

struct FwdVariant {
    int rpt, tg;
};
static const FwdVariant kFwdVariants[] = {{1, 128}, {2, 128}, {2, 256}, {4, 128}};
// Backward variants: 0-2 the Gaussian-lane kernel with RT rays staged per pass; 3-5 the
// ray-lane kernel with (RPT rays per lane, TG Gaussians per tile).
static const int kBwdRT[] = {64, 128, 256};
struct BwdRayVariant {
    int rpt, tg;
};
static const BwdRayVariant kBwdRay[] = {{2, 64}, {4, 64}, {4, 128}};
constexpr int kNumBwdGauss = (int)(sizeof kBwdRT / sizeof kBwdRT[0]);
constexpr int kNumBwdRay = (int)(sizeof kBwdRay / sizeof kBwdRay[0]);
// Variants 6-8: the tiled ray-lane kernel with T ray tiles per item (Gaussians staged 64 at a time),
// without a normal cotangent.  Calls with one run the form of it that takes them, numbered 9 (not a
// variant to choose: eight waves share 8 tiles, whose rays are twice the size).  It passes over the
// pairs that the Gaussian-lane variant 2, run before, evaluated: 12 views of 203 x 150 against 60
// Gaussians 76 -> 49 us.
// (256 threads per block for variants 6 and 7; variant 8 has eight waves share an item's 16 staged
// tiles, 512 threads).  Items of scenes beyond a block's count of Gaussians are cut by the scene, 2 to 16
// tiles, and run the form for large scenes of eight waves in all three.
static const int kBwdTiles[] = {8, 16, 16, 8};
constexpr int kNumBwdTiled = (int)(sizeof kBwdTiles / sizeof kBwdTiles[0]);  // the last: normal cotangents
constexpr int kBwdTiledFirst = kNumBwdGauss + kNumBwdRay;

// F dispatch: calls body<F>() for the runtime flag set f (0..7).
#define FMB_DISPATCH_F(f, CALL)                                                                            \
    switch (f) {                                                                                           \
    case 0: CALL(0); break;   case 1: CALL(1); break;   case 2: CALL(2); break;   case 3: CALL(3); break;   \
    case 4: CALL(4); break;   case 5: CALL(5); break;   case 6: CALL(6); break;   case 7: CALL(7); break;   \
    default: return hipErrorInvalidValue;                                                                  \
    }

// ... and over the forward's flag sets with kBig (8..15).
#define FMB_DISPATCH_F16(f, CALL)                                                                          \
    if ((f) < 8) {                                                                                         \
        FMB_DISPATCH_F(f, CALL)                                                                            \
    } else {                                                                                               \
        switch (f) {                                                                                       \
        case 8: CALL(8); break;   case 9: CALL(9); break;   case 10: CALL(10); break; case 11: CALL(11); break; \
        case 12: CALL(12); break; case 13: CALL(13); break; case 14: CALL(14); break; case 15: CALL(15); break; \
        default: return hipErrorInvalidValue;                                                              \
        }                                                                                                  \
    }

template <int RPT, int TG>
static hipError_t launch_fwd_v(int f, int grid, hipStream_t st, const Params &P, const FwdOut &O,
                               const FwdItem *items, const int *order)
{
#define FMB_FWD_CALL(F)                                                                                    \
    hipLaunchKernelGGL((fwd_kernel<kBlock, RPT, TG, F>), dim3(grid), dim3(kBlock), 0, st, P, O, items, order)
    FMB_DISPATCH_F16(f, FMB_FWD_CALL)
#undef FMB_FWD_CALL
    return hipGetLastError();
}

template <int RPT, int TG>
static hipError_t launch_bwdr_v(int f, int grid, hipStream_t st, const Params &P, const BwdIn &I,
                                const BwdItem *items, const int *order, float *partial,
                                float *bpart)
{
#define FMB_BWDR_CALL(F)                                                                                   \
    hipLaunchKernelGGL((bwdr_kernel<kBlock, RPT, TG, F>), dim3(grid), dim3(kBlock), 0, st, P, I, items, order, \
                       partial, bpart)
    FMB_DISPATCH_F(f, FMB_BWDR_CALL)
#undef FMB_BWDR_CALL
    return hipGetLastError();
}

template <int RT>
static hipError_t launch_bwd_v(int f, int grid, hipStream_t st, const Params &P, const BwdIn &I,
                               const BwdItem *items, const int *order, float *partial,
                               float *bpart)
{
#define FMB_BWD_CALL(F)                                                                                    \
    hipLaunchKernelGGL((bwd_kernel<kBlock, RT, F>), dim3(grid), dim3(kBlock), 0, st, P, I, items, order, \
                       partial, bpart)
    FMB_DISPATCH_F(f, FMB_BWD_CALL)
#undef FMB_BWD_CALL
    return hipGetLastError();
}

template <int BLK, int T, int BIG>
static hipError_t launch_bwdt_v(int f, int grid, hipStream_t st, const Params &P, const BwdIn &I,
                                const BwdItem *items, const int *order, float *partial,
                                float *bpart, unsigned long long *masks)
{
#define FMB_BWDT_CALL(F)                                                                                   \
    hipLaunchKernelGGL((bwdt_kernel<BLK, T, 64, F>), dim3(grid), dim3(BLK), 0, st, P, I, items, order,   \
                       partial, bpart, masks)
    if (grid == 0) return hipSuccess;
    switch (f) {  // (no normal cotangent; BIG: kBig)
    case 0: FMB_BWDT_CALL(BIG); break;
    case kFlw: FMB_BWDT_CALL(BIG | kFlw); break;
    case kCol: FMB_BWDT_CALL(BIG | kCol); break;
    case kCol | kFlw: FMB_BWDT_CALL(BIG | kCol | kFlw); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// The form with a normal cotangent.
static hipError_t launch_bwdt_normal(int f, int grid, hipStream_t st, const Params &P, const BwdIn &I,
                                     const BwdItem *items, const int *order, float *partial,
                                     float *bpart, unsigned long long *masks)
{
    constexpr int BLK = 512, T = 8;
    if (grid == 0) return hipSuccess;
    switch (f) {
    case 1: FMB_BWDT_CALL(1); break;   case 3: FMB_BWDT_CALL(3); break;   case 5: FMB_BWDT_CALL(5); break;
    case 7: FMB_BWDT_CALL(7); break;   case 9: FMB_BWDT_CALL(9); break;   case 11: FMB_BWDT_CALL(11); break;
    case 13: FMB_BWDT_CALL(13); break; case 15: FMB_BWDT_CALL(15); break;
    default: return hipErrorInvalidValue;
    }
#undef FMB_BWDT_CALL
    return hipGetLastError();
}

int num_fwd_variants() { return (int)(sizeof kFwdVariants / sizeof kFwdVariants[0]); }
int fwd_variant_rays(int v) { return kBlock * kFwdVariants[v].rpt; }
int num_bwd_variants() { return kNumBwdGauss + kNumBwdRay + kNumBwdTiled - 1; }
int bwd_normal_variant() { return num_bwd_variants(); }
// Tiled variants 6-9: ray tiles per item (0 for the others).
int bwd_variant_tiles(int v) { return v >= kBwdTiledFirst && v <= num_bwd_variants() ? kBwdTiles[v - kBwdTiledFirst] : 0; }
// Gaussian-lane variants: rays staged per pass; others: 0.
int bwd_variant_rt(int v) { return v < kNumBwdGauss ? kBwdRT[v] : 0; }
// Ray-lane variants 3-5: rays per block tile (BLOCK * RPT); others: 0.
int bwd_variant_ray_tile(int v) { return v >= kNumBwdGauss && v < kBwdTiledFirst ? kBlock * kBwdRay[v - kNumBwdGauss].rpt : 0; }
int block_size() { return kBlock; }

// flags: bit 0 normals, 1 flow, 2 colour, 3 a scene beyond a block's count of Gaussians
hipError_t launch_fwd(int variant, int flags, int grid, hipStream_t st, const Params &P, const FwdOut &O,
                      const FwdItem *items, const int *order)
{
    switch (variant) {
    case 0: return launch_fwd_v<1, 128>(flags, grid, st, P, O, items, order);
    case 1: return launch_fwd_v<2, 128>(flags, grid, st, P, O, items, order);
    case 2: return launch_fwd_v<2, 256>(flags, grid, st, P, O, items, order);
    case 3: return launch_fwd_v<4, 128>(flags, grid, st, P, O, items, order);
    default: return hipErrorInvalidValue;
    }
}

// n_small, n_big: the items of scenes within and beyond a block's count of Gaussians, in this order (order
// may be NULL where one of them is 0); big_tiles: the most ray tiles of the latter's items.  The variants
// that are not tiled have no form for large scenes: all their items are n_small.
hipError_t launch_bwd(int variant, int flags, int n_small, int n_big, int big_tiles, hipStream_t st, const Params &P,
                      const BwdIn &I, const BwdItem *items, const int *order, float *partial, float *bpart,
                      unsigned long long *masks)
{
    const int grid = n_small;
    if (n_big > 0) {
        const int *big_order = order ? order + n_small : nullptr;
        if (variant < kBwdTiledFirst || (!order && n_small > 0) || !masks || big_tiles > 16) return hipErrorInvalidValue;
        hipError_t e;
        if (variant == bwd_normal_variant())
            e = launch_bwdt_normal(flags | kBig, n_big, st, P, I, items, big_order, partial, bpart, masks);
        else if (big_tiles <= 8)
            e = launch_bwdt_v<512, 8, kBig>(flags, n_big, st, P, I, items, big_order, partial, bpart, masks);
        else
            e = launch_bwdt_v<512, 16, kBig>(flags, n_big, st, P, I, items, big_order, partial, bpart, masks);
        if (e != hipSuccess || n_small == 0) return e;
    }
    switch (variant) {
    case 0: return launch_bwd_v<64>(flags, grid, st, P, I, items, order, partial, bpart);
    case 1: return launch_bwd_v<128>(flags, grid, st, P, I, items, order, partial, bpart);
    case 2: return launch_bwd_v<256>(flags, grid, st, P, I, items, order, partial, bpart);
    case 3: return launch_bwdr_v<2, 64>(flags, grid, st, P, I, items, order, partial, bpart);
    case 4: return launch_bwdr_v<4, 64>(flags, grid, st, P, I, items, order, partial, bpart);
    case 5: return launch_bwdr_v<4, 128>(flags, grid, st, P, I, items, order, partial, bpart);
    case 6: return launch_bwdt_v<256, 8, 0>(flags, grid, st, P, I, items, order, partial, bpart, masks);
    case 7: return launch_bwdt_v<256, 16, 0>(flags, grid, st, P, I, items, order, partial, bpart, masks);
    case 8: return launch_bwdt_v<512, 16, 0>(flags, grid, st, P, I, items, order, partial, bpart, masks);
    case 9: return launch_bwdt_normal(flags, grid, st, P, I, items, order, partial, bpart, masks);
    default: return hipErrorInvalidValue;
    }
}

// The first n_one tasks (of at most one_gc Gaussians) are reduced in one stage, the others in two.
// masks: the items' record masks (or NULL: every record is written), rec: floats per record.
// max_gc: the largest chunk of any task (a whole scene for the ray-lane backward); max_nval: the
// largest first-stage record of any group.
hipError_t launch_fin(int n_tasks, int n_one, int one_gc, int n_groups, int max_gc, int max_nval, hipStream_t st, const Params &P,
                      const FinTask *tasks, const FinGroup *groups, const float *partial, const float *bpart,
                      const unsigned long long *masks, int rec, double *stage, double *stage_beta, float *g_means, float *g_prec, float *g_weights,
                      float *g_colors, float *g_betas)
{
    if (max_gc < 1 || max_nval < 1) return hipErrorInvalidValue;
    if (n_one > 0) {
        const int per = fin_one_gauss(rec);
        if ((one_gc + per - 1) / per > kGridYMax) return hipErrorInvalidValue;
        hipLaunchKernelGGL(fin_one_kernel, dim3(n_one, (one_gc + per - 1) / per), dim3(1024), 0, st, P, tasks, partial, bpart,
                           g_means, g_prec, g_weights, g_colors, g_betas);
    }
    if (n_tasks > n_one) {
        const int slices = (max_nval + 255) / 256 < kGridYMax ? (max_nval + 255) / 256 : kGridYMax;
        const int gslices = (max_gc + kFinSlice - 1) / kFinSlice;
        if (gslices > kGridYMax) return hipErrorInvalidValue;
        if (masks)
            hipLaunchKernelGGL((fin1s_kernel<256>), dim3(n_groups, (max_gc + 255) / 256 < kGridYMax ? (max_gc + 255) / 256 : kGridYMax),
                               dim3(256), 0, st, groups, partial, bpart, masks, rec, stage, stage_beta);
        else
            hipLaunchKernelGGL((fin1_kernel<256>), dim3(n_groups, slices), dim3(256), 0, st, groups, partial, bpart, stage,
                               stage_beta);
        hipLaunchKernelGGL((fin2_kernel<256>), dim3(n_tasks - n_one, gslices), dim3(256), 0, st, P, tasks + n_one, groups, stage,
                           stage_beta, g_means, g_prec, g_weights, g_colors, g_betas);
    }
    return hipGetLastError();
}

hipError_t launch_stat(int n_items, int n_tasks, int max_gc, hipStream_t st, const Params &P, const float *loss,
                       const float *stash, const BwdItem *items, const StatTask *tasks, float *partial,
                       const int64_t *rays_per_scene, float *lbar)
{
    if (n_items > 0)
        hipLaunchKernelGGL((statt_kernel<512, kStatTiles, 64>), dim3(n_items), dim3(512), 0, st, P, loss, stash, items,
                           partial);
    if (n_tasks > 0)
        hipLaunchKernelGGL(stat_fin_kernel, dim3(n_tasks, max_gc), dim3(256), 0, st, P, tasks, items, partial,
                           rays_per_scene, lbar);
    return hipGetLastError();
}

hipError_t launch_fill(int *p, int n, int value, hipStream_t st)
{
    hipLaunchKernelGGL(fill_int_kernel, dim3((n + 255) / 256), dim3(256), 0, st, p, n, value);
    return hipGetLastError();
}

hipError_t launch_validate(const Params &P, int n_total, int n_scenes, int *flags, hipStream_t st)
{
    const int n = n_total > n_scenes ? n_total : n_scenes;
    hipLaunchKernelGGL(validate_kernel, dim3((n + 255) / 256), dim3(256), 0, st, P, n_total, n_scenes, flags);
    return hipGetLastError();
}

}  // namespace fmb
