// gfx950 kernels of the span wavefront (Sec. 5, Algorithm 1, re-designed for the GPU).
//
// One step per span length g.  A team owns one layer pair (p, q = p + g) and therefore every
// cell (a, b) with a in layer p and b in layer q: a workgroup of 4, 8 or 16 wavefronts, one wavefront of a
// workgroup whose waves work on pairs of their own, or 2 to 16 of them.  It is the only writer of
// the candidate segments C_b of its right endpoints in this step (the endpoint-ownership rule of
// Sec. 5), so appends need no atomics and land in start-state order.  Its waves share out the closed
// values of the inner boundary pairs, the candidate scans of eq. (7) and the tables later spans read; after one
// barrier the cells are completed.  One extra team fills the external column one layer behind.
// Generic lattices (a forbidden-motif matcher intersected with the codon automaton) have their
// own span kernel in a section of its own below.
//
// Two-loop closure (stack / bulge / interior, l1 + l2 <= 30).  For a generic interior loop the
// energy is init(l1+l2) + asymmetry + mm[t][x_{i+1}][x_{j-1}] + mm[t'][x_{l+1}][x_{k-1}]: the
// outer mismatch couples only the two bases next to the closing pair and the inner mismatch only
// the two bases next to the inner pair.  When each unpaired segment crosses a codon boundary the
// trie's minimum segment cost splits the same way (first edge + rest of its codon, whole codons,
// last edge), so the whole term separates into
//     OUT(a1, b1, t)  [closing-pair side]  +  IN(c, d)  [inner-pair side]  +  layer constants.
// IN depends on the inner cell only, so its minimum over the states of a layer pair, LM, is
// stored once per layer pair (ring over the last 64 spans) when that pair is finished; a later
// cell then needs one lookup per (l1, l2) instead of an enumeration, and one per loop when only one
// segment separates.  The short segments that do not cross a codon boundary are enumerated.
#include <hip/hip_runtime.h>

#include <stddef.h>
#include <string.h>

#include <algorithm>

#include "sd_devutil.h"
#include "sd_internal.h"

namespace sd {

// Pair types as bit fields: 5' base, 3' base, and the type of the reversed pair.
__device__ __forceinline__ constexpr int type_x(int t) { return (0xFA4 >> (2 * t)) & 3; }
__device__ __forceinline__ constexpr int type_y(int t) { return (0x8DB >> (2 * t)) & 3; }
__device__ __forceinline__ constexpr int type_rev(int t) { return t == 0 ? 4 : t == 1 ? 2 : t == 2 ? 1 : t == 3 ? 5 : t == 4 ? 0 : 3; }

// ---- hairpin closure ------------------------------------------------------------------------
template <class IT>
__device__ int64_t hairpin_lane(const IT& I, const SmallE& S, const int32_t* __restrict__ spec,
                                int b, int t, int a1, int64_t Ua, int g, int lane) {
    const int m = g - 2, s = I.shift;
    const int x = kTX[t], y = kTY[t];
    int64_t best = kINF;
    if (m == 3 || m == 4 || m == 6) {
        // each lane walks the paths whose bases at positions 1..3 spell its lane id in base 4
        const int l1 = (lane >> 4) & 3, l2 = (lane >> 2) & 3, l3 = lane & 3;
        int st = a1, key = x;
        int64_t cost = Ua;
        const int labs[3] = {l1, l2, l3};
        for (int i = 0; i < 3; i++) {
            const int e = st * 4 + labs[i], d = I.out_dst()[e];
            if (d < 0) return kINF;
            cost += I.out_U()[e];
            key = key * 4 + labs[i];
            st = d;
        }
        const int nfree = g - 5;  // 0, 1 or 3 free positions before the final base y
        const int combos = 1 << (2 * nfree);
        for (int k = 0; k < combos; k++) {
            int st2 = st, key2 = key, ok = 1, last = l3;
            int64_t c2 = cost;
            for (int i = nfree - 1; i >= 0; i--) {
                const int lab = (k >> (2 * i)) & 3, e = st2 * 4 + lab, d = I.out_dst()[e];
                if (d < 0) {  // no path spells these labels: on to the next label here
                    ok = 0;
                    k |= (1 << (2 * i)) - 1;
                    break;
                }
                c2 += I.out_U()[e];
                key2 = key2 * 4 + lab;
                st2 = d;
                last = lab;
            }
            if (!ok) continue;
            const int e = st2 * 4 + y;
            if (I.out_dst()[e] != b) continue;
            c2 += I.out_U()[e];
            key2 = key2 * 4 + y;
            const int off = m == 3 ? kSpecOff5 : m == 4 ? kSpecOff6 : kSpecOff8;
            int32_t en = spec[off + key2];
            if (en == kNoSpecial) en = I.hp_init()[m] + (m == 3 ? au_pen(S, t) : S.mmH[t][l1][last]);
            best = mn(best, c2 + fx(en, s));
        }
        return best;
    }
    return best;
}

// ---- separable loop segments ---------------------------------------------------------------------
// An unpaired segment of l bases is separable when its first and last edges lie in different codons:
// its cheapest path with given end labels then costs first edge + rest of the first edge's codon
// + whole codons + last edge, with no coupling between the two labels.  The left segment of a loop
// closed by (p, q) runs from layer p + 1 to p + 1 + l1, the right one from q - 1 - l2 to q - 1.
// With alpha(d, x) = U(first edge) + tail and beta(c, x) = U(last edge) the whole codons are
// P[(p + l1) / 3] - P[(p + 2) / 3 + 1] on the left and P[(q - 2) / 3] - P[(q - l2) / 3 + 1] on the right;
// a segment that starts with a third base takes all further bases from the next codon, whose
// minimum is in alpha's tail and is taken off again by the prefix difference (the weight cost sits on
// third edges).  Shortest separable lengths: left 3, 2, 4 for p mod 3 = 0, 1, 2; right 2, 3, 4 for
// (q - 2) mod 3 = 0, 1, 2; every longer one is separable too.
// per-state rings [state][class][label][span mod 64]: a consumer walks consecutive spans
__device__ __forceinline__ int64_t ring_idx(int state, int span, int X, int lab) {
    return (((int64_t)state * 3 + X) * 4 + lab) * kLMRing + (span & (kLMRing - 1));
}
// per-layer-pair ring [left layer][class][span mod 64]
__device__ __forceinline__ int64_t lm_idx(int layer, int span, int X) {
    return ((int64_t)layer * 2 + X) * kLMRing + (span & (kLMRing - 1));
}
// ring of prepared both-separable minima [layer p][span mod 64][class]
__device__ __forceinline__ int64_t mini_idx(int p, int span, int X) {
    return ((int64_t)p * kLMRing + (span & (kLMRing - 1))) * 2 + X;
}
// one-sided tables [state][span mod 64][explicit length - 1][label]
__device__ __forceinline__ int64_t rs_idx(int state, int span, int l, int lab) {
    return ((int64_t)state * kLMRing + (span & (kLMRing - 1))) * 16 + (l - 1) * 4 + lab;
}
// The slot records, read-only while a kernel runs: through the constant address space, so that
// uniform reads go to scalar registers.
typedef const __attribute__((address_space(4))) SlotRec* SlotPtr;
__device__ __forceinline__ SlotPtr slot_ptr(const Inst& I) { return (SlotPtr)(uintptr_t)I.recs(); }

// A value every lane of the wave holds, moved to a scalar register so that the addresses and loop
// bounds derived from it stay scalar.
__device__ __forceinline__ int uni(int x) { return __builtin_amdgcn_readfirstlane(x); }
__device__ __forceinline__ int64_t uni(int64_t x) {
    const int hi = __builtin_amdgcn_readfirstlane((int)(x >> 32)), lo = __builtin_amdgcn_readfirstlane((int)x);
    return (int64_t)(((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo);
}
// Orders LDS accesses of the lanes of one wave (they execute in order; the compiler must not move them).
__device__ __forceinline__ void wave_lds_order() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
__device__ __forceinline__ void lds_min(int64_t* p, int64_t v) {
    __hip_atomic_fetch_min(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Hairpins of 3, 4 or 6 unpaired bases (listed special loops) over the paths a1 ~> b1, closed by type t:
// each lane walks the paths whose first three bases spell its lane id in base 4.
template <class IT>
__device__ __forceinline__ int64_t special_hairpin(const IT& I, const SmallE& S, const int32_t* __restrict__ spec, int a1,
                                   int b1, int t, int g, int lane) {
    const int m = g - 2, nfree = m - 3;  // 0, 1 or 3 bases after the first three
    int st = a1, key = type_x(t);
    int64_t cost = 0, best = kINF;
    for (int i = 2; i >= 0; i--) {
        const int lab = (lane >> (2 * i)) & 3, e = st * 4 + lab, d = I.out_dst()[e];
        if (d < 0) return kINF;
        cost += I.out_U()[e];
        key = key * 4 + lab;
        st = d;
    }
    for (int k = 0; k < 1 << (2 * nfree); k++) {
        int st2 = st, key2 = key, last = lane & 3;
        int64_t c2 = cost;
        bool ok = true;
        for (int i = nfree - 1; i >= 0 && ok; i--) {
            const int lab = (k >> (2 * i)) & 3, e = st2 * 4 + lab, d = I.out_dst()[e];
            ok = d >= 0;
            if (!ok) {  // no path spells these labels: on to the next label here
                k |= (1 << (2 * i)) - 1;
                break;
            }
            c2 += I.out_U()[e];
            key2 = key2 * 4 + lab;
            st2 = d;
            last = lab;
        }
        if (!ok || st2 != b1) continue;
        key2 = key2 * 4 + type_y(t);
        int32_t en = spec[(m == 3 ? kSpecOff5 : m == 4 ? kSpecOff6 : kSpecOff8) + key2];
        if (en == kNoSpecial) en = I.hp_init()[m] + (m == 3 ? au_pen(S, t) : S.mmH[t][(lane >> 4) & 3][last]);
        best = mn(best, c2 + fx(en, I.shift));
    }
    return best;
}

// ---- closed values of one inner boundary pair -----------------------------------------------------
// The loop closed by a pair (a -x-> a1 .. b1 -y-> b) of type t = (x, y) depends on a and b only through
// the two edge costs, so its minimum W_t(a1, b1) over hairpins, two-loops and the multiloop is found
// once per (a1, b1), for every type some edge pair can close, by one wave:
//   T[K][xi][xj]  (64 lanes) everything whose type dependence is a boundary table of class K (hairpin,
//                 generic interior, 1xn, 2x3) at the two bases next to the closing pair:
//                 hairpins, interior loops with a separable segment (A / B: minima of the other,
//                 explicit segment by its outer label; RS / LS hold them minimised over the separable
//                 segment's length, MINI over both), and explicit generic loops (LDS minima);
//   TA            everything whose type dependence is the AU/GU penalty: bulges of >= 2 bases and
//                 the multiloop;
//   special loops (stack, 1-base bulge, 1x1, 1x2, 2x1, 2x2), whose tables couple both pairs: per type.
// The step is bound by chains of dependent loads, so what counts is how many chains there are: one
// per (a1, b1) here, where one per (a, b, t) and per loop class walked the same inner cells again for
// each type (a span's slowest pairs close six types), and few short paths, since a segment counts
// as separable from its first codon boundary on.  300 aa fill 28.3 -> 19.5 ms, 1,976 aa 535 -> 391 ms, 64
// proteins of 50-1,000 aa in one launch 1.29 -> 0.71 s.
// The explicit loops are the combinations of the short label paths out of a1 and into b1 (the empty
// path included), flattened over the lanes; each reads its inner cell's six typed values once.
struct PairScratch {
    int64_t T[64];        // [class][xi][xj] minima of explicit generic loops
    int64_t AB[2][3][4];  // [left / right explicit][generic, 1xn, 2x3][outer label]
    // the pair's label paths: the empty one, then the states' lists
    int64_t fcost[kFwdPaths + 1], fcrow[kFwdPaths + 1], bcost[kBwdPaths + 1];
    int fmeta[kFwdPaths + 1], bmeta[kBwdPaths + 1];
};
constexpr int64_t kBarred = ((int64_t)1 << 61) + ((int64_t)1 << 60) + ((int64_t)1 << 59);  // infeasible, and adding kINF stays in range

__device__ __forceinline__ void closed_pair(const Inst& I, const SmallE& S, const int32_t* __restrict__ spec, int p, int q,
                            SlotPtr ra, SlotPtr rb, int tm, int parts, int lane, PairScratch& X, int64_t* wout) {
    // ra / rb: the records of a1 and b1.  parts: 1 the loops read through rings (hairpins, separable
    // segments, long bulges, multiloop), 2 the explicit loops, 3 both; two waves of a team share them
    const bool rings = parts & 1, paths = parts & 2;
    const int g = q - p, s = I.shift, m = g - 2;
    const int cap = min(g - 7, kMaxLoop);
    const int pl = p % 3, pr = (q - 2) % 3;
    const bool lsep2 = pl == 1, rsep2 = pr == 0;  // a 2-base segment is separable
    const SlotPtr rp = slot_ptr(I) + 2 * p, rq = slot_ptr(I) + 2 * q;
    const int a1 = ra->state, b1 = rb->state;
    const int f1 = ra->nf[0], f2 = ra->nf[1], r1 = rb->nb[0], r2 = rb->nb[1];  // list ends by length
    const int nf = ra->nf[2], nb = rb->nb[2];
    // path lists: lanes 0-11 left, 16-33 right
    const bool lleft = lane < kFwdPaths;
    const int le = lleft ? lane : min(max(lane - 16, 0), kBwdPaths - 1);
    const int64_t lcost = *(lleft ? &ra->fcost[le] : &rb->bcost[le]);
    const int lmeta = *(lleft ? &ra->fmeta[le] : &rb->bmeta[le]);
    const int64_t lcrow = ra->fcrow[min(lane, kFwdPaths - 1)];
    // hairpin and both-separable interior loops: lane = 16 K + 4 xi + xj
    const int K = lane >> 4, xi4 = (lane >> 2) & 3, xj4 = lane & 3;
    const int64_t al = ra->alpha[xi4], be = rb->beta[xj4];
    int64_t mini = I.MINI()[mini_idx(p, g, K >> 1)];  // (written from span 12 on)
    // bulges of >= 3 bases (lanes 0-27 right side unpaired, 32-59 left side) and the multiloop (lane 63)
    const bool bright = lane < 32;
    const int bl = 3 + (lane & 31);
    const int64_t* bsrc = (bright ? I.BI() + (int64_t)a1 * kLMRing : I.BJ() + (int64_t)b1 * kLMRing) + ((m - bl) & (kLMRing - 1));
    const int64_t bring = *(lane == 63 ? I.S2() + ra->rowbase + b1 : bsrc);
    X.T[lane] = kINF;
    if (lane < 24) (&X.AB[0][0][0])[lane] = kINF;
    if (lane < 6) wout[lane] = kINF;
    if (lleft) {
        X.fcost[lane + 1] = lcost;
        X.fmeta[lane + 1] = lmeta;
        X.fcrow[lane + 1] = lcrow;
    } else if (lane >= 16 && lane < 16 + kBwdPaths) {
        X.bcost[lane - 15] = lcost;
        X.bmeta[lane - 15] = lmeta;
    } else if (lane == 63) {
        X.fcost[0] = X.bcost[0] = 0;
        X.fcrow[0] = ra->rowbase;
        X.fmeta[0] = a1 << 4;
        X.bmeta[0] = b1 << 4;
    }
    wave_lds_order();
    // explicit loops, 64 path combinations a round (nearly always one round); the inner cells of a
    // round are read before the one-sided tables are waited for
    const int nl = 1 + nf, nr = 1 + nb;
    const int tot = paths ? nl * nr : 0, rcp = (65536 + nr - 1) / nr;
    int l1, l2, xi, xk, xl, xj;
    int64_t vin[6], bs;
    auto read_cells = [&](int idx) {
        const bool in_list = idx < tot;
        const int i = in_list ? (int)(((unsigned)idx * (unsigned)rcp) >> 16) : 0, j = in_list ? idx - i * nr : 0;
        l1 = (i > 0) + (i > f1) + (i > f2);
        l2 = (j > 0) + (j > r1) + (j > r2);
        const bool ok = in_list && l1 + l2 <= max(cap, 0) &&
                        ((l1 <= 2 && l2 <= 2) || (l1 > 0 && l2 > 0 && !(l1 == 2 && lsep2) && !(l2 == 2 && rsep2)));
        const int fm = X.fmeta[i], bm = X.bmeta[j];
        bs = ok ? X.fcost[i] + X.bcost[j] : kBarred;
        xi = (fm >> 2) & 3, xk = fm & 3, xl = (bm >> 2) & 3, xj = bm & 3;
        const longlong2* vp = reinterpret_cast<const longlong2*>(I.V() + (ok ? X.fcrow[i] + (bm >> 4) : ra->rowbase + b1) * 6);
        const longlong2 v01 = vp[0], v23 = vp[1], v45 = vp[2];
        vin[0] = v01.x, vin[1] = v01.y, vin[2] = v23.x, vin[3] = v23.y, vin[4] = v45.x, vin[5] = v45.y;
    };
    if (paths) read_cells(lane);
    int64_t ta = kINF;
    if (rings) {
        // one-sided: explicit paths of length l (not separable; at most 30 of them) against RS / LS, and
        // the 2x3 / 3x2 loops, whose mismatch class differs from the rest of their row, against IDL / JDL
        const int ne = lsep2 ? f1 : nf, nt = ne + (rsep2 ? r1 : nb);
        const bool left = lane < ne;
        const int e = lane < nt ? (left ? lane : lane - ne) : 0;
        const int l = left ? 1 + (e >= f1) + (e >= f2) : 1 + (e >= r1) + (e >= r2);
        const int meta = lane < nt ? (left ? X.fmeta[e + 1] : X.bmeta[e + 1]) : X.bmeta[0];
        const int64_t cost = left ? X.fcost[e + 1] : X.bcost[e + 1];
        const int st = meta >> 4;
        // label next to the inner pair, label next to the closing pair
        const int in = left ? meta & 3 : (meta >> 2) & 3, out = left ? (meta >> 2) & 3 : meta & 3;
        const int64_t v = (left ? I.RS() : I.LS())[rs_idx(st, m - l, l, in)];
        const int64_t w = (left ? I.IDL() : I.JDL())[ring_idx(st, m - 5, 1, in)];
        const bool x23 = left ? (l == 2 && pr != 2) || (l == 3 && rsep2) : (l == 2 && pl != 2) || (l == 3 && lsep2);
        ta = bring + (lane == 63 ? fx(S.ml_closing + S.ml_intern, s)
                                 : (bright ? rq->pb1 : ra->tail - rp->pa1) + fx(S.bulge[min(bl, kMaxLoop)], s));
        if (lane != 63 && bl > cap) ta = kINF;
        int64_t* ab = &X.AB[left ? 0 : 1][0][0];
        if (lane < nt && v < kHalfINF) lds_min(ab + (l == 1 ? 4 : 0) + out, cost + v);
        if (lane < nt && x23 && w < kHalfINF)
            lds_min(ab + 8 + out, cost + w + fx(interior_base(S, 2, 3), s) + (left ? rq->pb2 : -rp->pa2));
    }
    int B0, St, Sr, sl = 0, sr = 0, live = 0;
    bool spl;
    // this lane's special loop closed by type t, biased: the word at byte B0 + t St + rev(t') Sr, whose entry
    // (4 bytes, or for 1x2, 2x1, 2x2 one of its halves, the same for every t and t') two shifts cut
    // out; vin then holds the inner cell's values + path costs + bias
    auto special = [&](int t) {
        int64_t v = kINF + kBias;
#pragma unroll
        for (int tp = 0; tp < 6; tp++) {
            if (!((live >> tp) & 1)) continue;
            const int w = *reinterpret_cast<const int*>(reinterpret_cast<const char*>(&S) + (B0 + type_rev(tp) * Sr + t * St));
            v = min_positive(v, vin[tp] + fx((int)((unsigned)w << sl) >> sr, s));
        }
        return v;
    };
    if (paths)
        for (int idx = lane;;) {
            // type dependence of the loop: a special table (l1, l2 <= 2 except the 2-base bulge) or a
            // boundary class (1 generic, 2 1xn, 3 2x3, 4 AU penalty only)
            const bool small = l1 <= 2 && l2 <= 2;
            spl = small && (l1 + l2 != 2 || l1 == 1);
            const int KK = small ? 4 : (l1 == 1 || l2 == 1) ? 2 : l1 + l2 == 5 ? 3 : 1;
            const int32_t cst = !small ? interior_base(S, l1, l2) : l1 + l2 == 1 ? S.bulge[1] : spl ? 0 : S.bulge[2];
            bs += fx(cst, s);
            // inner minimum over the inner pair's types for the boundary classes
            {
                const int32_t* tab = &S.mmH[0][0][0] + KK * 96 + xl * 4 + xk;
                int64_t in = kINF + kBias;
                live = 0;
#pragma unroll
                for (int tp = 0; tp < 6; tp++) {
                    vin[tp] += kBias;
                    in = min_positive(in, vin[tp] + fx(tab[type_rev(tp) * 16], s));
                    const bool fin = spl && vin[tp] < kINF + kBias;
                    live |= __ballot(fin) ? 1 << tp : 0;
                    vin[tp] = fin ? vin[tp] + bs : kINF + kBias;
                }
                in += bs - kBias;
                if (!spl) {
                    if (KK == 4) ta = mn(ta, in);
                    else if (in < kHalfINF) lds_min(&X.T[KK * 16 + xi * 4 + xj], in);
                }
            }
            sl = sr = l1 + l2 > 2 ? 16 : 0;
            if (l1 + l2 <= 1) {
                B0 = offsetof(SmallE, stack), St = 24, Sr = 4;
            } else if (l1 + l2 == 2) {
                B0 = (int)offsetof(SmallE, int11) + (xi * 4 + xj) * 4, St = 384, Sr = 64;
            } else if (l1 + l2 == 4) {
                B0 = (int)offsetof(SmallE, int22) + (xi * 64 + xk * 16 + xl * 4 + xj) * 2, St = 3072, Sr = 512;
            } else if (l1 == 1) {
                B0 = (int)offsetof(SmallE, int21) + (xi * 16 + xl * 4 + xj) * 2, St = 768, Sr = 128;
            } else {
                B0 = (int)offsetof(SmallE, int21) + (xl * 16 + xi * 4 + xk) * 2, St = 128, Sr = 768;
            }
            if (!spl) B0 = 0, St = 0, Sr = 0, sl = sr = 16;  // any valid entry: added to an infinite value
            if (B0 & 2) sl = 0;
            B0 &= ~3;
            idx += 64;
            if (idx - lane >= tot) break;
#pragma unroll 1
            for (int t = 0; t < 6; t++) {
                if (!((tm >> t) & 1)) continue;
                const int64_t v = wave_min_biased(special(t)) - kBias;
                if (lane == 0) wout[t] = mn(wout[t], v);
            }
            read_cells(idx);
        }
    wave_lds_order();
    // T: explicit generic minima, hairpin / both-separable, one-sided
    int64_t T = X.T[lane];
    if (rings) {
        // (MINI holds its pair's whole-codon terms)
        const int64_t hp = m >= 5 && m != 6 ? fx(I.hp_init()[m], s) + rq->pb2 - rp->pa2 : kINF;
        const int64_t x = K == 0 ? hp : (K & 1) && g >= 12 ? mini : kINF;
        if (al < kINF && be < kINF && x < kINF) T = mn(T, al + be + x);
        if (K > 0) {
            const int64_t A = X.AB[0][K - 1][xi4], B = X.AB[1][K - 1][xj4];
            if (A < kINF && be < kINF) T = mn(T, A + be);
            if (al < kINF && B < kINF) T = mn(T, al + B);
        }
    }
    ta = wave_min(ta);
    T += kBias;
    const int32_t* tab = &S.mmH[0][0][0] + K * 96 + (lane & 15);
#pragma unroll 1
    for (int t = 0; t < 6; t++) {
        if (!((tm >> t) & 1)) continue;
        const int64_t x = T + fx(tab[t * 16], s);
        const int64_t v = mn(wave_min_biased(paths ? min_positive(special(t), x) : x) - kBias, ta + fx(au_pen(S, t), s));
        if (lane == 0) wout[t] = norm_inf(mn(wout[t], v));
    }
    if (rings && (m == 3 || m == 4 || m == 6)) {
#pragma unroll 1
        for (int t = 0; t < 6; t++) {
            if (!((tm >> t) & 1)) continue;
            const int64_t v = wave_min(special_hairpin(I, S, spec, a1, b1, t, g, lane));
            if (lane == 0) wout[t] = mn(wout[t], v);
        }
    }
}

// ---- the work of one layer pair (p, q) in span step g: one workgroup of several waves ----------
// The threads that work on one layer pair: the whole workgroup (ordered by workgroup barriers),
// or a single wavefront of a workgroup whose waves each work on their own pair (ordered within the
// wave; a workgroup barrier there would pair up unrelated points of different waves).
// The lane index produced per call: teams run inside loops over their items, and lane predicates
// derived from threadIdx would be hoisted to the kernel entry and held throughout, where they crowd
// the scalar registers and are spilled to vector lanes.
__device__ __forceinline__ int lane_id() {
    int l;
    asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(l));
    return l;
}
template <int NT>
struct BlockTeam {
    __device__ int wave() const { return __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); }
    __device__ int lane() const { return lane_id(); }
    __device__ static constexpr int waves() { return NT / 64; }
    __device__ void sync() { __syncthreads(); }
};
// `n` consecutive waves of a workgroup, ordered by an LDS arrival counter (zero when the team is
// formed; every wave of the workgroup is resident, so the wait ends).  One wave needs no counter.
struct WaveTeam {
    unsigned* ctr = nullptr;
    int w = 0, n = 1;
    unsigned epoch = 0;
    __device__ int wave() const { return w; }
    __device__ int lane() const { return lane_id(); }
    __device__ int waves() const { return n; }
    __device__ void sync() {
        if (n == 1) {
            wave_lds_order();
            return;
        }
        epoch += n;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        if (lane() == 0) __hip_atomic_fetch_add(ctr, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        while (__hip_atomic_load(ctr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) < epoch) __builtin_amdgcn_s_sleep(1);
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    }
};

// A wave by itself.
struct SoloTeam {
    __device__ static constexpr int wave() { return 0; }
    __device__ int lane() const { return lane_id(); }
    __device__ static constexpr int waves() { return 1; }
    __device__ void sync() { wave_lds_order(); }
};

// LDS of one team; a wave's own scratch lies in the element of its own index, so that an array of
// as many elements as waves serves teams of any size.
constexpr int kTrieCells = kTrieWidth * kTrieWidth;
struct GroupShared {
    int64_t w[2][kTrieCells][6];      // W_t(a1, b1) of the pair's inner boundary pairs, in two parts
    union {
        PairScratch scratch;          // phase 1
        int64_t vbuf[kTrieCells][6];  // phase 2: typed closed values of the pair's cells
    };
    int64_t s2[kTrieCells];           // S2 of the cells
    int64_t ps[kTrieCells];           // P_S of the cells; once they are completed, B
    // the pair's records, as phase 2 needs them, read beside phase 1
    int64_t aU[kTrieWidth][4], bU[kTrieWidth][4];        // edge costs out of the left states and of layer q - 1
    int64_t abeta[kTrieWidth][4], balpha[kTrieWidth][4]; // beta of the left states, alpha of the right ones
    int64_t btail[kTrieWidth], boff[kTrieWidth];         // right states: tail, candidate segment,
    int bcnt[kTrieWidth], bcap[kTrieWidth];              //   committed count and capacity
    int task;                         // next task of phase 1 (zero between items)
    int8_t adst[kTrieWidth][4], bdst[kTrieWidth][4];     // the edges' targets by slot (-1 none)
    int8_t keep[kTrieCells];          // 0 none, 1 strict, 2 retained non-strict
};

// One-sided tables of state st of the pair for span g (left states c of layer p: RS, right states d of
// layer q: LS), by one wave: the minimum over the separable side's length of IDL / JDL of spans
// <= g - 3 + loop energy + whole codons, per explicit length 1..3 and inner label.  They read nothing
// this span writes.
__device__ __forceinline__ void produce_one_sided(const Inst& I, const SmallE& S, int p, int q, bool left, int st, int lane) {
    const int s = I.shift, g = q - p;
    // the consumer closes (.., q + 1) around c, or (p - 1, ..) around d
    if (left ? q == I.n : p == 0) return;
    const int64_t cod = left ? slot_ptr(I)[2 * (q + 1)].pb2 : -slot_ptr(I)[2 * (p - 1)].pa2;
    const int l0 = left ? (q - 1) % 3 + 2 : (p + 2) % 3 == 0 ? 3 : (p + 2) % 3 == 1 ? 2 : 4;  // shortest separable length
    // lane = 4 * grp + lab covers separable lengths 3 + grp and 19 + grp
    const int lab = lane & 3, grp = lane >> 2;
    const int64_t* T = left ? I.IDL() : I.JDL();
    int64_t in0[2], in2[2];
#pragma unroll
    for (int h = 0; h < 2; h++) {
        const int ls = 3 + grp + 16 * h;
        const bool ok = ls <= 29 && g - ls >= 5 && ls >= l0;
        const int gr = ok ? g - ls : 0;
        in0[h] = T[ring_idx(st, gr, 0, lab)];
        in2[h] = T[ring_idx(st, gr, 2, lab)];
        if (!ok) in0[h] = in2[h] = kINF;
        in0[h] += kBias;
        in2[h] += kBias;
    }
    int64_t o[3] = {kINF + kBias, kINF + kBias, kINF + kBias};
#pragma unroll
    for (int h = 0; h < 2; h++) {
        const int ls = 3 + grp + 16 * h;
#pragma unroll
        for (int le = 1; le <= 3; le++) {
            if (le + ls > kMaxLoop || (le == 2 && ls == 3)) continue;
            // the energy depends on |l1 - l2| and l1 + l2 only
            o[le - 1] = min_positive(o[le - 1], (le == 1 ? in2[h] : in0[h]) + fx(interior_base(S, le, ls), s));
        }
    }
#pragma unroll
    for (int j = 0; j < 3; j++) {
        // over the lanes that share lane & 3: rotations by 4 and 8 within each row, then rows
        o[j] = min_xor32(min_xor16(min_dpp<kDppRor8>(min_dpp<kDppRor4>(o[j]))));
    }
    if (grp < 3)
        (left ? I.RS() : I.LS())[rs_idx(st, g, grp + 1, lab)] = norm_inf((grp == 0 ? o[0] : grp == 1 ? o[1] : o[2]) + (cod - kBias));
}

// Inner minima of the pair's left or right states for span g, by one wave: IDL and BI (left states, and
// LM) or JDL and BJ (right states).  v: lane 6 * cell + type holds the typed value; only the feasible
// ones (about one per pair) are visited.
__device__ __forceinline__ void produce_inner(const Inst& I, const SmallE& S, const GroupShared& G, int p, int q,
                              bool left, int64_t v, int wa, int wb, int lane) {
    const int s = I.shift, g = q - p;
    const SlotPtr rp = slot_ptr(I) + 2 * p, rq = slot_ptr(I) + 2 * q;
    // lane = 16 * X + 4 * xx + z (48 lanes), minimised over z; left: vary x_{l+1} = z with alpha(d),
    // right: vary x_{k-1} = z with beta(c)
    const int X = lane >> 4, xx = (lane >> 2) & 3, z = lane & 3;
    const int cls = X == 0 ? 1 : X == 1 ? 3 : 2;  // boundary class of X (row 3 repeats 1xn and is not stored)
    const int32_t* tab = &S.mmH[0][0][0] + cls * 96 + (left ? z * 4 + xx : xx * 4 + z);
    const int64_t w0 = left ? G.balpha[0][z] : G.abeta[0][z], w1 = left ? G.balpha[1][z] : G.abeta[1][z];
    int64_t acc0 = kINF, acc1 = kINF, bu0 = kINF, bu1 = kINF;  // the two states' minima, and their bulge rings'
    for (unsigned long long m = __ballot(lane < wa * wb * 6 && v < kINF); m; m &= m - 1) {
        const int k = __builtin_ctzll(m), ci = k / 6, t = k - 6 * ci, ia = ci / wb, ib = ci - wb * ia;
        const int i = left ? ia : ib, o = left ? ib : ia;
        const int64_t vin = readlane64(v, k), w = o ? w1 : w0;
        const int64_t x = w < kINF ? vin + w + fx(tab[((0x305124 >> (4 * t)) & 7) * 16], s) : kINF;
        const int64_t u = vin + (left ? G.btail[o] : 0) + fx(au_pen(S, t), s);
        if (i) acc1 = mn(acc1, x), bu1 = mn(bu1, u);
        else acc0 = mn(acc0, x), bu0 = mn(bu0, u);
    }
    int64_t lm = kINF;
    for (int i = 0; i < (left ? wa : wb); i++) {
        int64_t acc = i ? acc1 : acc0;
        acc = mn(acc, dpp64<kDppXor1>(acc));
        acc = mn(acc, dpp64<kDppXor2>(acc));
        acc = norm_inf(acc + (left ? -rq->in2 : rp->ip1));
        const int st = left ? rp[i].state : rq[i].state;
        if (X < 3 && z == 0) (left ? I.IDL() : I.JDL())[ring_idx(st, g, X, xx)] = acc;
        const int64_t bu = norm_inf((i ? bu1 : bu0) + (left ? -rq->in1 : rp->ip0));
        if (lane == 63) (left ? I.BI() : I.BJ())[(int64_t)st * kLMRing + (g & (kLMRing - 1))] = bu;
        if (left) {
            const int64_t be = G.abeta[i][xx];
            if (acc < kINF && be < kINF) lm = mn(lm, acc + be);
        }
    }
    if (left) {
        // LM: layer-pair minimum of the both-separable form, over the row of class X (0 generic, 1 2x3)
        lm = mn(lm, dpp64<kDppRor4>(lm));
        lm = mn(lm, dpp64<kDppRor8>(lm));
        if (X < 2 && (lane & 15) == 0) I.LM()[lm_idx(p, g, X)] = norm_inf(lm + rp->ip1);
    }
}

// Both-separable interior minima of layer pair (p, q), q - p >= 12, into the ring MINI, by one wave:
// LM of the inner layer pairs (spans <= q - p - 8) + loop energy + whole codons.  The lengths
// (l1 >= L0, l2 >= R0, l1 + l2 <= cap) form a triangle of M rows (row a, l1 = L0 + a, holds M - a);
// rows r and M - r hold M together, so four lanes take each such pair of rows in at most seven rounds.
__device__ __forceinline__ void prepare_mini(const Inst& I, const SmallE& S, int p, int q, int lane) {
    const int s = I.shift, g = q - p, cap = min(g - 7, kMaxLoop);
    const int pl = p % 3, L0 = pl == 0 ? 3 : pl == 1 ? 2 : 4, R0 = (q - 2) % 3 + 2;  // shortest separable lengths
    const int M = cap - L0 - R0 + 1;
    const int64_t cod = slot_ptr(I)[2 * q].pb2 - slot_ptr(I)[2 * p].pa2;
    const int r = lane >> 2;
    int64_t m0 = kINF, m1 = kINF;
#pragma unroll 1
    for (int it = 0; it < 7; it++) {
        const int j = (lane & 3) + 4 * it;
        const bool first = j < M - r;
        const int a = first ? r : M - r, l1 = L0 + a, l2 = R0 + (first ? j : j - (M - r));
        // 2x2 loops read their full table and are always enumerated
        if (j >= M || 2 * r > M || (!first && 2 * r == M) || l1 + l2 == 4) continue;
        const int X = pair_class(l1, l2);
        const int64_t lm = I.LM()[lm_idx(p + 1 + l1, g - 2 - l1 - l2, X)];
        const int64_t v = lm + fx(interior_base(S, l1, l2), s);
        if (X) m1 = mn(m1, v);
        else m0 = mn(m0, v);
    }
    m0 = wave_min(m0);
    m1 = wave_min(m1);
    if (lane < 2) I.MINI()[mini_idx(p, g, lane)] = norm_inf((lane ? m1 : m0) + cod);
}

struct GroupCounters {
    unsigned long long visits, feasible;
};

// The committed prefix of C_b with the gathered S1(a, c) (eq. 7), the lanes' minima.  Every entry was
// committed by an earlier span, so its start state lies in a layer after a's.
__device__ __forceinline__ int64_t scan_candidates(const int* __restrict__ cc, const int64_t* __restrict__ cB,
                                                   const int64_t* __restrict__ S1r, int committed, int lane) {
    int64_t s2 = kINF;
    // four entries per lane and round, their loads issued together: the gathers of S1(a, c)
    // depend on the start states, so one entry at a time would serialise two load latencies
    // per 64 entries
    int k = lane;
    for (; k + 192 < committed; k += 256) {
        const int c0 = cc[k] & 0x7fffffff, c1 = cc[k + 64] & 0x7fffffff;
        const int c2 = cc[k + 128] & 0x7fffffff, c3 = cc[k + 192] & 0x7fffffff;
        const int64_t b0 = cB[k], b1 = cB[k + 64], b2 = cB[k + 128], b3 = cB[k + 192];
        const int64_t s0 = S1r[c0], s1v = S1r[c1], s2v = S1r[c2], s3 = S1r[c3];
        s2 = mn(s2, mn(mn(s0 + b0, s1v + b1), mn(s2v + b2, s3 + b3)));
    }
    for (; k < committed; k += 64) s2 = mn(s2, S1r[cc[k] & 0x7fffffff] + cB[k]);
    return s2;
}

// The split part of one cell (a, b) of layer pair (p, q) on a lattice without slot records: S2 (eq. 7: in-edge
// extensions, then the committed prefix of C_b) and P_S; neither depends on the cell's direct cost.  Sixteen lanes per
// cell: a wave takes four at once.
__device__ __forceinline__ void gen_scan(const Inst& I, int p, int q, int a, int b, bool valid, int lane, int64_t* s2_out, int64_t* ps_out,
                                         int* committed_out) {
    const int l16 = lane & 15;
    int64_t s2 = kINF, ps = kINF;
    int committed = 0;
    if (valid) {
        const int64_t arow = I.rowbase()[a], cbase = I.coff()[b];
        const int64_t* S1r = I.S1() + arow;
        const int64_t* S2r = I.S2() + arow;
        committed = I.ccnt()[b];
        if (q - p >= 2) {
            const int j1 = I.in_start()[b + 1];
            for (int j = I.in_start()[b] + l16; j < j1; j += 16) {
                const int c = I.in_src()[j];
                const int64_t u = I.in_U()[j] + I.mlbase_fx;
                s2 = mn(s2, S2r[c] + u);
                ps = mn(ps, S1r[c] + u);
            }
            if (l16 < 4) {
                const int ap = I.out_dst()[a * 4 + l16];
                if (ap >= 0) ps = mn(ps, I.S1()[I.rowbase()[ap] + b] + I.out_U()[a * 4 + l16] + I.mlbase_fx);
            }
        }
        const int* cc = I.cc() + cbase;
        const int64_t* cB = I.cB() + cbase;
#pragma unroll 4
        for (int k = l16; k < committed; k += 16) s2 = mn(s2, S1r[cc[k] & 0x7fffffff] + cB[k]);
    }
    s2 = norm_inf(row_min(s2));
    ps = norm_inf(mn(s2, row_min(ps)));
    if (valid && l16 == 0) {
        *s2_out = s2;
        *ps_out = ps;
        *committed_out = committed;
    }
}

// The same on the codon trie, by one wave, from the slot records: ia / ib the slots of a and b in their layers.
__device__ __forceinline__ void trie_scan(const Inst& I, int p, int q, int ia, int ib, int lane, int64_t* s2_out, int64_t* ps_out) {
    const SlotPtr rp = slot_ptr(I) + 2 * p, rq = slot_ptr(I) + 2 * q;
    const int b = rq[ib].state;
    const int64_t arow = rp[ia].rowbase, cbase = rq[ib].coff;
    const int committed = uni(I.ccnt()[b]);
    const int64_t* __restrict__ S1r = I.S1() + arow;
    const int64_t* __restrict__ S2r = I.S2() + arow;
    int64_t s2 = kINF, ps = kINF;
    if (q - p >= 2) {
        // lanes 0-7 the edges of layer q - 1 (slot, label), lanes 8-11 a's out-edges by label
        const int x = lane & 3;
        const SlotPtr rb = rq - 2 + ((lane >> 2) & 1);
        const bool in = lane < 8 && rb->state >= 0 && rb->dst[x] == ib;
        const int d = lane >= 8 && lane < 12 ? rp[ia].dst[x] : -1;
        const int64_t u = (in ? rb->outU[x] : rp[ia].outU[x]) + I.mlbase_fx;
        if (in) {
            s2 = S2r[rb->state] + u;
            ps = S1r[rb->state] + u;
        } else if (d >= 0) {
            ps = I.S1()[rp[2 + d].rowbase + b] + u;
        }
    }
    s2 = norm_inf(wave_min(mn(s2, scan_candidates(I.cc() + cbase, I.cB() + cbase, S1r, committed, lane))));
    *s2_out = s2;
    *ps_out = norm_inf(mn(s2, wave_min(ps)));
}

// Appends the retained entries (a, B(a, b)) of layer pair (p, q) to the segments C_b in
// start-state order, one lane per right endpoint: the caller's workgroup owns these segments in
// step g (endpoint ownership), so no atomics are needed and the layout is deterministic.  An
// append beyond a segment's capacity records the earliest overflowing span instead.
template <class IT>
__device__ void append_candidates(const IT& I, int a_lo, int wa, int b_lo, int wb, const int8_t* keep,
                                  const int64_t* cellB, int g, int lane, int committed, int cap,
                                  int64_t base) {
    // committed / cap / base: lane < wb's segment C_(b_lo + lane), count, capacity and offset
    int added = 0;
    if (lane < wb) {
        for (int ia = 0; ia < wa; ia++) {
            const int ci = ia * wb + lane;
            if (!keep[ci]) continue;
            const int slot = committed + added;
            if (slot < cap) {
                I.cc()[base + slot] = (a_lo + ia) | (keep[ci] == 1 ? 0 : (int)0x80000000);
                I.cB()[base + slot] = cellB[ci];
            } else {
                atomicMin(&I.stats()[2], (unsigned long long)g);
            }
            added++;
        }
        if (added) I.ccnt()[b_lo + lane] = min(committed + added, cap);
    }
}

// The same with the segments' counts, capacities and offsets read from the instance.
template <class IT>
__device__ void append_candidates(const IT& I, int a_lo, int wa, int b_lo, int wb, const int8_t* keep,
                                  const int64_t* cellB, int g, int lane) {
    const bool mine = lane < wb;
    append_candidates(I, a_lo, wa, b_lo, wb, keep, cellB, g, lane, mine ? I.ccnt()[b_lo + lane] : 0,
                      mine ? I.ccap()[b_lo + lane] : 0, mine ? I.coff()[b_lo + lane] : 0);
}

// Phase 2 of a layer pair, by one wave: the typed values of its cells, and with `cells` their
// completion (branch value, S1, retention, appends), with `left` / `right` the inner minima of its
// left / right states.  Several waves may share the work; each completes the same typed values.
__device__ __forceinline__ void complete_cells(const Inst& I, const SmallE& S, int p, int q, int wa, int wb, int wb1, int split, bool cells,
                               bool left_role, bool right_role, int lane, GroupShared& G, GroupCounters& ctr) {
    const int g = q - p, s = I.shift, ncell = wa * wb;
    const SlotPtr rp = slot_ptr(I) + 2 * p, rq = slot_ptr(I) + 2 * q;
    int64_t v = kINF;
    if (lane < ncell * 6) {
        const int ci = lane / 6, t = lane - 6 * ci, ia = ci / wb, ib = ci - wb * ia;
        if (g >= 5) {
            const int a1 = G.adst[ia][type_x(t)];
            if (a1 >= 0)
                for (int j = 0; j < wb1; j++)
                    if (G.bdst[j][type_y(t)] == ib) {
                        int64_t w = G.w[0][a1 * kTrieWidth + j][t];
                        if (split == 2) w = mn(w, G.w[1][a1 * kTrieWidth + j][t]);
                        v = mn(v, G.aU[ia][type_x(t)] + G.bU[j][type_y(t)] + w);
                    }
        }
        v = norm_inf(v);
        if (cells) {
            G.vbuf[ci][t] = v;
            I.V()[(rp[ia].rowbase + rq[ib].state) * 6 + t] = v;
        }
    }
    if (cells) {
        wave_lds_order();
        // branch value (eq. 2), S1 and the retention test (eq. 6), one lane per cell
        bool feasible = false;
        if (lane < ncell) {
            const int ia = lane / wb, ib = lane - wb * ia;
            int64_t Bv = kINF;
#pragma unroll
            for (int t = 0; t < 6; t++) Bv = mn(Bv, G.vbuf[lane][t] + fx(S.ml_intern + au_pen(S, t), s));
            Bv = norm_inf(Bv);
            const int64_t cell = rp[ia].rowbase + rq[ib].state, ps = G.ps[lane];
            I.Bt()[cell] = Bv;
            I.S2()[cell] = G.s2[lane];
            I.S1()[cell] = mn(Bv, ps);
            const bool strict = Bv < ps;
            G.keep[lane] = I.retain_all ? (Bv < kINF ? (strict ? 1 : 2) : 0) : (strict ? 1 : 0);
            G.ps[lane] = Bv;
            feasible = Bv < kINF;
        }
        ctr.feasible = __popcll(__ballot(feasible));
        ctr.visits = (unsigned long long)(G.bcnt[0] + (wb > 1 ? G.bcnt[1] : 0)) * wa;
        wave_lds_order();
        // appends in start-state order, one lane per right endpoint (this team owns C_b in this step)
        const bool mine = lane < wb;
        append_candidates(I, rp[0].state, wa, rq[0].state, wb, G.keep, G.ps, g, lane, mine ? G.bcnt[lane] : 0,
                          mine ? G.bcap[lane] : 0, mine ? G.boff[lane] : (int64_t)0);
    }
    if (left_role) produce_inner(I, S, G, p, q, true, v, wa, wb, lane);
    if (right_role) produce_inner(I, S, G, p, q, false, v, wa, wb, lane);
}

// One layer pair of span step g on the codon trie.  Phase 1 is a list of tasks that read only earlier
// spans and are dealt to the team's waves (everything they need of the pair's states is one level of
// loads away, in the slot records): the closed values W(a1, b1) of each inner boundary pair,
// the split part of each cell, the one-sided tables of each state, and the next span's
// both-separable minima.  After one barrier, the cells are completed (typed values, branch value, S1,
// retention, appends) by one wave while others derive the inner minima for later two-loops.
template <class Team>
__device__ __forceinline__ GroupCounters span_group(const Inst& I, const SmallE& S, const int32_t* __restrict__ spec, int p, int q,
                                    GroupShared* Gs, Team& T) {
    // Gs: the team's elements, one per wave; the first holds the pair's shared state
    const int g = q - p;
    const int wave = T.wave(), lane = T.lane(), nw = T.waves();
    GroupShared& G = Gs[0];
    GroupCounters ctr{0, 0};
    const SlotPtr rp1 = slot_ptr(I) + 2 * p, rq1 = slot_ptr(I) + 2 * q;
    const int wa = 1 + (rp1[1].state >= 0), wb = 1 + (rq1[1].state >= 0), ncell = wa * wb;
    const int wa1 = 1 + (rp1[3].state >= 0), wb1 = 1 + (rq1[-1].state >= 0);
    if (wave == nw - 1) {
        const SlotPtr rp = rp1, rq = rq1;
        // lanes 0-7 the left states' out-edges (slot, label) and beta, 8-15 the edges out of layer q - 1,
        // 16-23 the right states' alpha, 24-25 their candidate segments
        const int i = (lane >> 2) & 1, x = lane & 3;
        if (lane < 8) {
            G.adst[i][x] = rp[i].dst[x];
            G.aU[i][x] = rp[i].outU[x];
            G.abeta[i][x] = rp[i].beta[x];
        } else if (lane < 16) {
            G.bdst[i][x] = rq[i - 2].state >= 0 ? rq[i - 2].dst[x] : -1;
            G.bU[i][x] = rq[i - 2].outU[x];
        } else if (lane < 24) {
            G.balpha[i][x] = rq[i].alpha[x];
        } else if (lane < 24 + wb) {
            G.btail[x] = rq[x].tail;
            G.boff[x] = rq[x].coff;
            G.bcap[x] = rq[x].ccap;
            G.bcnt[x] = I.ccnt()[rq[x].state];
        }
    }
    // teams of eight waves or more give the two parts of a closed value to different waves
    const int split = nw >= 8 ? 2 : 1, nclosed = g >= 5 ? wa1 * wb1 * split : 0, nstate = g >= 5 ? wa + wb : 0;
    const int nmini = g + 1 >= 12 && q + 1 <= I.n ? 1 : 0, ntask = nclosed + ncell + nmini + nstate;
    // With more tasks than waves, every wave draws its next one (they differ threefold: closed values and
    // splits first): 1,976 aa fill 271 -> 252 ms, 925 aa 74.8 -> 70.0, 300 aa 14.7 -> 14.3; with fewer
    // (sixteen waves: 17 tasks at most) there is nothing to draw, and the counter's latency cost 2.5 % at 50 aa.
    const bool draw = nw > 1 && nw < 16 && ntask > nw;
    auto next_task = [&](int k0) {
        if (!draw) return k0 + nw;
        int d = 0;
        if (lane == 0) d = __hip_atomic_fetch_add(&G.task, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        return nw + uni(d);
    };
    for (int k0 = wave; k0 < ntask; k0 = next_task(k0)) {
        int k = k0;
        const Inst J = rebased(I);
        if (k < nclosed) {
            const int kk = k / split, part = k - kk * split, ia1 = kk / wb1, ib1 = kk - wb1 * ia1;
            const SlotPtr ra = slot_ptr(J) + 2 * (p + 1) + ia1, rb = slot_ptr(J) + 2 * (q - 1) + ib1;
            // types some edge pair around (a1, b1) has: first base entering a1, last base leaving b1
            const int im = ra->inmask, om = rb->outmask;
            int tm = 0;
#pragma unroll
            for (int t = 0; t < 6; t++) tm |= ((im >> type_x(t)) & (om >> type_y(t)) & 1) << t;
            if (tm)
                closed_pair(J, S, spec, p, q, ra, rb, tm, split == 2 ? 1 + part : 3, lane, Gs[wave].scratch,
                            G.w[part][ia1 * kTrieWidth + ib1]);
            continue;
        }
        k -= nclosed;
        if (k < ncell) {
            int64_t s2, ps;
            trie_scan(J, p, q, k / wb, k - wb * (k / wb), lane, &s2, &ps);
            if (lane == 0) {
                G.s2[k] = s2;
                G.ps[k] = ps;
            }
            continue;
        }
        k -= ncell;
        if (k < nmini) {
            prepare_mini(J, S, p, q + 1, lane);
            continue;
        }
        k -= nmini;
        const bool left = k < wa;
        produce_one_sided(J, S, p, q, left, left ? slot_ptr(J)[2 * p + k].state : slot_ptr(J)[2 * q + k - wa].state, lane);
    }
    T.sync();
    if (draw && wave == 0 && lane == 0) G.task = 0;
    const bool left_role = g >= 5 && (1 % nw) == wave, right_role = g >= 5 && (2 % nw) == wave;
    if (wave != 0 && !left_role && !right_role) return ctr;
    complete_cells(rebased(I), S, p, q, wa, wb, wb1, split, wave == 0, left_role, right_role, lane, G, ctr);
    return ctr;
}

// ---- external column: X(a) for every a of layer L (one team) ------------------------------------
// X(a) = min(U + X of the out-edges, AU + V_t(a, b) + X(b) over closing pairs).  The branch value holds
// min over t of V_t + ML_intern + AU, so the scan reads it (8 contiguous bytes per b) and takes
// ML_intern off.
template <class IT, class Team>
__device__ __forceinline__ void ext_column(const IT& I, const SmallE& S, int L, GroupShared* Gs, Team& T) {
    const int tid = T.wave() * 64 + T.lane(), nt = T.waves() * 64;
    const int64_t mi = fx(S.ml_intern, I.shift);
    for (int a = I.off()[L]; a < I.off()[L + 1]; a++) {
        int64_t v = kINF;
        if (tid < 4) {
            const int d = I.out_dst()[a * 4 + tid];
            if (d >= 0) v = I.out_U()[a * 4 + tid] + I.X()[d];
        }
        if (L + 5 <= I.n) {
            const int64_t* Br = I.Bt() + I.rowoff()[a] - I.off()[L + 1];
#pragma unroll 4
            for (int bb = I.off()[L + 5] + tid; bb < I.N; bb += nt) v = mn(v, Br[bb] + (I.X()[bb] - mi));
        }
        v = wave_min(v);
        if (T.waves() > 1) {
            if (T.lane() == 0) Gs[T.wave()].s2[0] = v;
            T.sync();
            for (int w = 0; w < T.waves(); w++) v = mn(v, Gs[w].s2[0]);
        }
        if (tid == 0) I.X()[a] = norm_inf(v);
        T.sync();
    }
}

template <class IT>
__device__ __forceinline__ void flush_counters(const IT& I, const GroupCounters& c, int p, int lane) {
    if (lane != 0) return;
    if (c.visits) atomicAdd(&I.visits()[p], c.visits);
    if (c.feasible) atomicAdd(&I.feasible()[p], c.feasible);
}

// Workgroups are dispatched round-robin over the 8 XCDs (workgroup i on XCD i mod 8), each with
// its own L2.  Neighbouring layer pairs read each other's rows and rings, so every XCD gets one
// contiguous band of layer pairs: a bijection of [0, nb) that sends the workgroups of residue x
// to the x-th band.
__device__ __forceinline__ int xcd_band(int i, int nb) {
    const int x = i & 7, k = i >> 3;
    int base = 0;
    for (int r = 0; r < x; r++) base += (nb - r + 7) >> 3;
    return base + k;
}

// Brings the records of a pair's four layers to this XCD's L2 while the tables are staged: one word of
// each of their lines, by the first wave.
__device__ __forceinline__ void prefetch_records(const Inst& I, int p, int g) {
    if (threadIdx.x >= 64) return;
    constexpr int kLines = 4 * sizeof(SlotRec) / 128;  // two layers
    const int lane = threadIdx.x;
    const char* base = reinterpret_cast<const char*>(I.recs() + (lane < kLines ? 2 * p : 2 * (p + g - 1)));
    const int w = *reinterpret_cast<const int*>(base + (lane < kLines ? lane : min(lane - kLines, kLines - 1)) * 128);
    asm volatile("" ::"v"(w));
}

// ---- the span step (plain mode) ----------------------------------------------------------------
// Items are the span's layer pairs (item x is pair xcd_band(x)), then the external column.  A span
// with more items than the chip holds workgroups runs as many workgroups as it holds, each taking
// every gridDim.x-th item with one staging of the energy tables.  Held to 128 VGPRs: four workgroups of 256
// threads fit a CU, two of 512.  (k_span<512> spills two VGPRs, the others none; about 230 scalar registers
// go to vector lanes.)  With 148 VGPRs (three) the 1,976-aa fill took 384 ms
// instead of 324; one staging per resident workgroup, direct copies to LDS and the records brought
// to L2 beside them made it 279 ms (300 aa 17.7 -> 16.7 ms).
template <int NT>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(NT == 64 ? 1 : 4)))
void k_span(Inst I, const EnergyTables* __restrict__ E, const int32_t* __restrict__ spec, int g,
            int ext_layer, int npairs) {
    __shared__ SmallE S;
    __shared__ GroupShared G[NT / 64];
    stage_begin(S, E);
    if (threadIdx.x == 0) G[0].task = 0;
    if ((int)blockIdx.x < npairs) prefetch_records(I, xcd_band(blockIdx.x, npairs), g);
    stage_wait();
    BlockTeam<NT> T;
    const int items = npairs + (ext_layer >= 0 ? 1 : 0);
    for (int i = blockIdx.x; i < items; i += gridDim.x) {
        if (i < npairs) {
            const int p = xcd_band(i, npairs);
            const Inst J = rebased(I);
            flush_counters(J, span_group(J, S, spec, p, p + g, G, T), p, T.lane());
        } else {
            ext_column(I, S, ext_layer, G, T);
        }
        __syncthreads();  // the team's shared state is free for its next item
    }
}

// The span step with every wave on its own layer pair, sixteen pairs per workgroup and one staging of
// the energy tables: the waves' items are independent and no workgroup barrier follows the staging.
template <int NT>
__global__ __launch_bounds__(NT) void k_span_waves(
    Inst I, const EnergyTables* __restrict__ E, const int32_t* __restrict__ spec, int g, int ext_layer, int npairs) {
    constexpr int NWV = NT / 64;
    __shared__ SmallE S;
    __shared__ GroupShared G[NWV];
    stage_tables(S, E);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int items = npairs + (ext_layer >= 0 ? 1 : 0), nblk = (items + NWV - 1) / NWV;
    WaveTeam T;
    for (int i = blockIdx.x; i < nblk; i += gridDim.x) {
        const int item = xcd_band(i, nblk) * NWV + wave;
        const Inst J = rebased(I);
        if (item < npairs) flush_counters(J, span_group(J, S, spec, item, item + g, &G[wave], T), item, T.lane());
        else if (item < items) ext_column(J, S, ext_layer, &G[wave], T);
    }
}

__global__ __launch_bounds__(256) void k_ext(Inst I, const EnergyTables* __restrict__ E, int L) {
    __shared__ SmallE S;
    __shared__ GroupShared G[4];
    stage_tables(S, E);
    BlockTeam<256> T;
    ext_column(I, S, L, G, T);
}

__global__ void k_init(Inst I) {
    const int tid = blockIdx.x * blockDim.x + threadIdx.x, nt = gridDim.x * blockDim.x;
    for (int i = tid; i < I.N; i += nt) {
        I.ccnt()[i] = 0;
        I.X()[i] = I.layer()[i] == I.n ? 0 : kINF;  // every state of the last layer is a sink
    }
    if (I.gwin) {  // no rings on a generic lattice
        if (tid < 4) I.stats()[tid] = tid == 2 ? ~0ull : 0ull;
        for (int i = tid; i <= I.n; i += nt) I.visits()[i] = I.feasible()[i] = 0;
        return;
    }
    for (size_t i = tid; i < (size_t)(I.n + 1) * 2 * kLMRing; i += nt) I.LM()[i] = kINF;
    for (size_t i = tid; i < (size_t)I.N * kLMRing * 12; i += nt) {
        I.IDL()[i] = kINF;
        I.JDL()[i] = kINF;
    }
    for (size_t i = tid; i < (size_t)I.N * kLMRing; i += nt) {
        I.BI()[i] = kINF;
        I.BJ()[i] = kINF;
    }
    for (size_t i = tid; i < (size_t)I.N * kLMRing * 16; i += nt) {
        I.RS()[i] = kINF;
        I.LS()[i] = kINF;
    }
    if (tid < 4) I.stats()[tid] = tid == 2 ? ~0ull : 0ull;
    for (int i = tid; i <= I.n; i += nt) {
        I.visits()[i] = 0;
        I.feasible()[i] = 0;
    }
}

// ---- the multiloop recurrences alone on an abstract layered DAG (test hook) -----------------------
// Direct branch costs B are given per cell (row layout, in the V array of the instance) instead of
// coming from loop energies; the unpaired-edge costs are the automaton's edge costs (ML_base 0).
// One wave per layer pair of span g runs the generic span step's own gen_scan and
// append_candidates: the exact-integer abstract test of Sec. 7.1 on the GPU code path.
__global__ __launch_bounds__(64) void k_ml_abstract(Inst I, int g) {
    constexpr int kCells = kMaxWidth * kMaxWidth;
    __shared__ int8_t keep[kCells];
    __shared__ int64_t s2[kCells], ps[kCells], cellB[kCells];
    __shared__ int committed[kCells];
    const int p = blockIdx.x, q = p + g, lane = threadIdx.x;
    const int a_lo = I.off()[p], wa = I.off()[p + 1] - a_lo, b_lo = I.off()[q], wb = I.off()[q + 1] - b_lo, ncell = wa * wb;
    GroupCounters ctr{0, 0};
    for (int c0 = 0; c0 < ncell; c0 += 4) {
        const int ci = c0 + (lane >> 4), cv = min(ci, ncell - 1);
        gen_scan(I, p, q, a_lo + cv / wb, b_lo + cv % wb, ci < ncell, lane, s2 + cv, ps + cv, committed + cv);
    }
    __syncthreads();
    if (lane < ncell) {
        const int64_t cell = I.rowbase()[a_lo + lane / wb] + b_lo + lane % wb, Bv = I.V()[cell];
        I.Bt()[cell] = Bv;
        I.S2()[cell] = s2[lane];
        I.S1()[cell] = mn(Bv, ps[lane]);
        const bool strict = Bv < ps[lane];
        keep[lane] = I.retain_all ? (Bv < kINF ? (strict ? 1 : 2) : 0) : (strict ? 1 : 0);
        cellB[lane] = Bv;
    }
    __syncthreads();
    append_candidates(I, a_lo, wa, b_lo, wb, keep, cellB, g, lane);
    for (int ci = 0; ci < ncell; ci++) {
        ctr.visits += (unsigned long long)committed[ci];
        ctr.feasible += cellB[ci] < kINF;
    }
    flush_counters(I, ctr, p, lane);
}

// ---- span checksums (debug mode) -----------------------------------------------------------------
// An order-independent digest (wrapping sum of mixed (tag, index, value) words) of what a span
// step writes: the cells of span g (V, B, S1, S2), the committed candidate counts and entries,
// the visit and feasibility counters, the external column and the ring slots of span g.  With
// g = 0 it covers every cell and no ring slot (the whole tables of a finished design).  Two runs
// of a step that read the same inputs must give the same digest whatever their schedule.
__device__ __forceinline__ unsigned long long mix64(unsigned long long x) {
    x ^= x >> 30;
    x *= 0xbf58476d1ce4e5b9ull;
    x ^= x >> 27;
    x *= 0x94d049bb133111ebull;
    return x ^ (x >> 31);
}
__device__ __forceinline__ unsigned long long dword(int tag, int64_t idx, int64_t v) {
    return mix64((unsigned long long)v ^ mix64(((unsigned long long)idx << 4) | (unsigned)tag));
}

__global__ void k_checksum(Inst I, int g, unsigned long long* out) {
    const int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, nt = (int64_t)gridDim.x * blockDim.x;
    unsigned long long h = 0;
    // cells: of span g (p = 0 .. n - g), or every cell
    const int plo = 0, phi = g > 0 ? I.n - g : I.n;
    for (int p = plo; p <= phi; p++) {
        const int q0 = g > 0 ? p + g : p + 1, q1 = g > 0 ? p + g : I.n;
        if (q0 > I.n) break;
        const int a0 = I.off()[p], a1 = I.off()[p + 1], b0 = I.off()[q0], b1 = I.off()[q1 + 1];
        const int64_t wb = b1 - b0, tot = (int64_t)(a1 - a0) * wb;
        for (int64_t k = tid; k < tot; k += nt) {
            const int a = a0 + (int)(k / wb), b = b0 + (int)(k % wb);
            const int64_t c = I.rowoff()[a] + (b - I.off()[p + 1]);
            for (int t = 0; t < 6; t++) h += dword(1 + t, c, I.V()[c * 6 + t]);
            h += dword(7, c, I.Bt()[c]) + dword(8, c, I.S1()[c]) + dword(9, c, I.S2()[c]);
        }
    }
    for (int64_t b = tid; b < I.N; b += nt) {
        const int cnt = I.ccnt()[b];
        h += dword(10, b, cnt) + dword(11, b, I.X()[b]);
        const int64_t base = I.coff()[b];
        for (int k = 0; k < cnt; k++) h += dword(12, base + k, I.cc()[base + k]) + dword(13, base + k, I.cB()[base + k]);
    }
    for (int64_t l = tid; l <= I.n; l += nt) h += dword(14, l, (int64_t)I.visits()[l]) + dword(15, l, (int64_t)I.feasible()[l]);
    if (g > 0) {
        const int r = g & (kLMRing - 1), r1 = (g + 1) & (kLMRing - 1);
        for (int64_t st = tid; st < I.N; st += nt) {
            for (int k = 0; k < 12; k++) {
                h += dword(16, st * 12 + k, I.IDL()[(st * 12 + k) * kLMRing + r]);
                h += dword(17, st * 12 + k, I.JDL()[(st * 12 + k) * kLMRing + r]);
            }
            for (int k = 0; k < 16; k++) {
                h += dword(18, st * 16 + k, I.RS()[(st * kLMRing + r) * 16 + k]);
                h += dword(19, st * 16 + k, I.LS()[(st * kLMRing + r) * 16 + k]);
            }
            h += dword(20, st, I.BI()[st * kLMRing + r]) + dword(21, st, I.BJ()[st * kLMRing + r]);
        }
        for (int64_t l = tid; l <= I.n; l += nt)
            for (int X = 0; X < 2; X++) {
                h += dword(22, l * 2 + X, I.LM()[(l * 2 + X) * kLMRing + r]);
                h += dword(23, l * 2 + X, I.MINI()[(l * kLMRing + r1) * 2 + X]);
            }
    }
    // wave sum, then one atomic per wave (wrapping, so the total is order independent)
    for (int o = 32; o > 0; o >>= 1) h += __shfl_xor(h, o, 64);
    if ((threadIdx.x & 63) == 0) atomicAdd(out, h);
}

// ---- generic lattice: the codon automaton intersected with a forbidden-motif matcher --------------
// Nothing below relies on the codon trie.  With e = (a, x) an out-edge (state and label), i = (v, y) a
// row (state and the label of an in-edge), the span step fills for its own cells and later spans read
//   G(a, b)    minimum path cost a -> b (cell layout);
//   LG(e, i)   minimum cost of a path that starts with edge e and ends in v through an edge labelled
//              y, for layer distances 1..30: the unpaired segments of a two-loop;
//   IN_X(i, f) for row i = (c, xk) and out-edge f = (d, xl): min over types t' of V_t'(c, d) + mm_X[t'
//              reversed][xl][xk], the inner part of an interior loop of mismatch class X.
// An interior loop couples its segments only through the four bases next to its pairs, so the closed
// value of an inner boundary pair (a1, b1) of layers p1, q1 is the minimum over e out of a1 and rows j
// of b1 of T_X(e, j) + mm_X[t][x(e)][y(j)], with
//   Q(e, f) = min over l1 and rows i of layer p1 + l1 of LG(e, i) + IN(i, f) + size(l1, l2)
//   T(e, j) = min over l2 and out-edges f of layer q1 - l2 of Q(e, f) + LG(f, j)
// two min-plus products that serve every closing type and every pair of states of the two layers: per
// layer pair about 465 * rows * edges * edges sums, where one evaluation per (a, b, type) took states^3 *
// edges * 160.  Loops with a side of one base (class 1xn) need only one of the products and 2x3 loops are
// a handful of rows; stacks, bulges of one base and the tabulated 1x1, 1x2, 2x2 loops enumerate the
// label walks of up to two edges on both sides.
// One workgroup of sixteen waves per layer pair (one per CU: 143 KB of LDS).  What bounds a span is the chain
// of loads and barriers of its widest pair, and more than 256 pairs take a second round.  105 residues under
// 16 motifs (3.1 states per layer, up to 10): a launch takes 58 us on average with 166 to 285 pairs, 37 with 66
// to 115, 23 with five or fewer; over all spans 45 us, against 110 with these products on eight waves and 600
// with a (cell, type) per wave and job tickets.  31 residues under 5 motifs: 205 -> 30 us.
// Infinite operands: LG is kINF, IN and the accumulators kHalfINF, finite values lie within 2^60, so a
// sum of all three neither overflows nor falls below kGenBig.
constexpr int64_t kGenBig = kHalfINF >> 1;
constexpr int kGenGroup = 8;   // left edges per task
constexpr int kGenRows = 16;   // rows per unit
constexpr int kGenTasks = 16;  // (eight left edges, 64 right edges) per round

typedef const __attribute__((address_space(4))) int* IntPtr;
typedef const __attribute__((address_space(4))) int64_t* LongPtr;

// The states of an inner layer and the row base of its first state; every state's row has len cells.
struct GenLayer {
    int first, cnt;
    int64_t row, len;
};
struct GenShared {
    int64_t w[kGenMaxWidth * kGenMaxWidth * 6];  // W_t(a1, b1)
    int64_t v[kGenMaxWidth * kGenMaxWidth * 6];  // hairpins of 3, 4, 6 bases, then V of the cells
    int64_t s2[kGenMaxWidth * kGenMaxWidth], ps[kGenMaxWidth * kGenMaxWidth], cellB[kGenMaxWidth * kGenMaxWidth];
    int committed[kGenMaxWidth * kGenMaxWidth];
    int8_t keep[kGenMaxWidth * kGenMaxWidth];
    GenLayer left[kGenLoopWin + 1], right[kGenLoopWin + 1];  // layers p1 + l, q1 - l
    int64_t size[kGenLoopWin][32];               // size(l1, l2) + kBias in fixed point
    int64_t q[kGenTasks][64][kGenGroup + 1];     // Q + kBias of one round
};

// minimum into a shared word; values that hold an infinite operand are left out
__device__ __forceinline__ void gen_min(int64_t* w, int64_t v) {
    if (v < kGenBig) __hip_atomic_fetch_min(w, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// The sums of one layer pair that a two-loop of layers p1 = p + 1, q1 = q - 1 needs.
struct GenPair {
    int p, q, p1, q1, g, a1lo, wa1, b1lo, wb1;
    int e0, ne, j0, nj;  // out-edges of layer p1, rows of layer q1
};

// Bulges of two bases and more around every (a1, b1): one thread per (a1, b1, share of the sizes).  The branch
// value of the inner pair holds the minimum over its types; the rows of a layer's states are equally long.
__device__ __forceinline__ void gen_bulges(const Inst& I, const SmallE& S, const GenPair& P, GenShared& G, int tid, int nt) {
    const int s = I.shift, outs = P.wa1 * P.wb1, parts = max(1, min(kGenLoopWin - 1, nt / outs));
    const int lmax = min(kGenLoopWin, P.g - 7);
    const int64_t* Gt = I.Gt();
    const int64_t* Bt = I.Bt();
    for (int k = tid; k < outs * parts; k += nt) {
        const int ib = k % P.wb1, r = k / P.wb1, ia = r % P.wa1, part = r / P.wa1;
        const int a1 = P.a1lo + ia, b1 = P.b1lo + ib;
        const int64_t arow = I.rowbase()[a1];
        int64_t v = kHalfINF;
        for (int l = 2 + part; l <= lmax; l += parts) {
            const GenLayer Lc = G.left[l], Ld = G.right[l];
            int64_t w = kHalfINF;
#pragma unroll 2
            for (int i = 0; i < Lc.cnt; i++)
                w = mn(w, mn(Gt[arow + Lc.first + i], kHalfINF) + Bt[Lc.row + (int64_t)i * Lc.len + b1]);
#pragma unroll 2
            for (int i = 0; i < Ld.cnt; i++)
                w = mn(w, mn(Gt[Ld.row + (int64_t)i * Ld.len + b1], kHalfINF) + Bt[arow + Ld.first + i]);
            v = mn(v, w + fx(S.bulge[l] - S.ml_intern, s));
        }
        if (v < kGenBig)
#pragma unroll
            for (int t = 0; t < 6; t++) gen_min(G.w + (ia * P.wb1 + ib) * 6 + t, v + fx(au_pen(S, t), s));
    }
}

// Hairpins of listless sizes, one thread per (edge out of a1, edge into b1), and multiloops, one thread per
// (a1, b1, type).
__device__ __forceinline__ void gen_hairpins(const Inst& I, const SmallE& S, const GenPair& P, int64_t* w, int tid, int nt) {
    const IntPtr eo = (IntPtr)(uintptr_t)I.geoff();
    const int s = I.shift, m = P.g - 2;
    if (m == 5 || m >= 7) {
        const int f0 = eo[P.q1 - 1], nf = eo[P.q1] - f0;
        const int64_t init = fx(I.hp_init()[m], s);
        for (int k = tid; k < P.ne * nf; k += nt) {
            const GenEdge& e = I.gedges()[P.e0 + k / nf];
            const GenEdge& f = I.gedges()[f0 + k % nf];
            const int64_t gg = I.Gt()[I.rowbase()[e.dst] + f.src];
            if (gg >= kINF) continue;
            const int64_t h = e.U + gg + f.U + init;
            int64_t* w6 = w + ((e.src - P.a1lo) * P.wb1 + (f.dst - P.b1lo)) * 6;
#pragma unroll
            for (int t = 0; t < 6; t++) gen_min(w6 + t, h + fx(S.mmH[t][e.lab][f.lab], s));
        }
    }
    if (m >= 10)  // from the next wave on
        for (int k = (tid - 64) & (nt - 1); k < P.wa1 * P.wb1 * 6; k += nt) {
            const int t = k % 6, r = k / 6, ia = r / P.wb1, ib = r - ia * P.wb1;
            gen_min(w + k, I.S2()[I.rowbase()[P.a1lo + ia] + P.b1lo + ib] + fx(S.ml_closing + S.ml_intern + au_pen(S, t), s));
        }
}

// Stacks, bulges of one base and the loops of the 1x1, 1x2, 2x2 tables: one (left walk, right walk,
// closing type) per thread.  Walks of 0, 1, 2 edges: states, out-edges, entries of the walk list.
__device__ __forceinline__ void gen_small(const Inst& I, const SmallE& S, const GenPair& P, int64_t* w, int tid, int nt) {
    const IntPtr eo = (IntPtr)(uintptr_t)I.geoff(), wo = (IntPtr)(uintptr_t)I.gwoff();
    const int s = I.shift, g1 = P.g - 2;
    int nl[3], nr[3], cum[7], total = 0;
    nl[0] = P.wa1;
    nl[1] = P.ne;
    const int lw = wo[P.p1];
    nl[2] = wo[P.p1 + 1] - lw;
    nr[0] = P.wb1;
    const int rf = eo[P.q1 - 1];
    nr[1] = eo[P.q1] - rf;
    const int rw = wo[P.q1 - 2];
    nr[2] = wo[P.q1 - 1] - rw;
#pragma unroll
    for (int k = 0; k < 7; k++) {
        constexpr int L1[7] = {0, 0, 1, 1, 1, 2, 2}, L2[7] = {0, 1, 0, 1, 2, 1, 2};
        cum[k] = total;
        if (g1 - L1[k] - L2[k] >= 5) total += nl[L1[k]] * nr[L2[k]];
    }
    for (int it = tid; it < 6 * total; it += nt) {
        const int t = it % 6, k = it / 6;
        int cls = 0, base = 0;
#pragma unroll
        for (int c = 1; c < 7; c++)
            if (k >= cum[c]) {
                cls = c;
                base = cum[c];
            }
        const int l1 = cls < 2 ? 0 : cls < 5 ? 1 : 2, l2 = cls == 0 || cls == 2 ? 0 : cls == 1 || cls == 3 || cls == 5 ? 1 : 2;
        const int n2 = l2 == 0 ? nr[0] : l2 == 1 ? nr[1] : nr[2], kl = (k - base) / n2, kr = (k - base) - kl * n2;
        int a1 = P.a1lo + kl, c = a1, xi = 0, xk = 0, d = P.b1lo + kr, b1 = d, xl = 0, xj = 0;
        int64_t U = 0;
        if (l1 > 0) {
            const GenEdge& e = l1 == 1 ? I.gedges()[P.e0 + kl] : I.gwalks()[lw + kl];
            a1 = e.src;
            c = e.dst;
            xi = e.lab & 3;
            xk = e.lab >> 2;
            U = e.U;
            if (l1 == 1) xk = xi;
        }
        if (l2 > 0) {
            const GenEdge& e = l2 == 1 ? I.gedges()[rf + kr] : I.gwalks()[rw + kr];
            d = e.src;
            b1 = e.dst;
            xl = e.lab & 3;
            xj = e.lab >> 2;
            U += e.U;
            if (l2 == 1) xj = xl;
        }
        const int64_t* vv = I.V() + (I.rowbase()[c] + d) * 6;
        int64_t best = kINF;
#pragma unroll
        for (int tp = 0; tp < 6; tp++) {
            const int tr = type_rev(tp);
            const int32_t e2 = l1 + l2 == 0 ? S.stack[t][tr]
                               : l1 * l2 == 0 ? bulge_e(S, t, tr, 1) : interior_e(S, nullptr, t, tr, l1, l2, xi, xk, xl, xj);
            best = mn(best, vv[tp] + fx(e2, s));
        }
        gen_min(w + ((a1 - P.a1lo) * P.wb1 + (b1 - P.b1lo)) * 6 + t, best + U);
    }
}

// Interior loops other than the tabulated ones: both products.  A task is eight left edges x 64 right edges
// of one part, generic loops and those with l2 = 1 (part 0), 2x3 loops (1), loops with l1 = 1 (2);
// its rows are cut into units of kGenRows, dealt to the waves.  The second product has one thread per (left
// edge, row of layer q1, share of the right edges).  `rest` is the other work of the step, done by each wave
// between its units of the first round and the barrier.
template <int NT, class F>
__device__ __forceinline__ void gen_products(const Inst& I, const SmallE& S, const GenPair& P, GenShared& G, int wave, int lane, F rest) {
    constexpr int NW = NT / 64;
    const IntPtr eo = (IntPtr)(uintptr_t)I.geoff();
    const LongPtr LG4 = (LongPtr)(uintptr_t)I.LG();
    const int s = I.shift, g1 = P.g - 2, win = I.win, smax = min(kGenLoopWin, g1 - 5);
    // right edges of the parts (inner span >= 5), blocks of 64 of each
    int fa[3] = {0, 0, 0}, fb[3] = {0, 0, 0};
    if (g1 >= 9) {
        fa[0] = eo[max(P.q1 - 28, P.p1 + 7)];
        fb[0] = eo[P.q1];
        fa[2] = eo[max(P.q1 - 29, P.p1 + 6)];
        fb[2] = eo[P.q1 - 2];
    }
    if (g1 >= 10) {
        fa[1] = eo[P.q1 - 3];
        fb[1] = eo[P.q1 - 1];
    }
    const int n0 = (fb[0] - fa[0] + 63) / 64, n1 = (fb[1] - fa[1] + 63) / 64, nbt = n0 + n1 + (fb[2] - fa[2] + 63) / 64;
    const int ntask = nbt * ((P.ne + kGenGroup - 1) / kGenGroup);
    for (int t0 = 0; t0 < ntask || t0 == 0; t0 += kGenTasks) {
        if (t0) {
            for (int k = wave * 64 + lane; k < kGenTasks * 64 * (kGenGroup + 1); k += NT) (&G.q[0][0][0])[k] = kHalfINF + kBias;
            __syncthreads();
        }
        // lane t describes task t0 + t of the round
        const int nt = min(kGenTasks, ntask - t0);
        int part = 0, tf = 0, te = 0, ti0 = 0, ti1 = 0, te0 = 0;
        if (lane < nt) {
            const int grp = (t0 + lane) / nbt, r = (t0 + lane) - grp * nbt;
            part = r < n0 ? 0 : r < n0 + n1 ? 1 : 2;
            tf = (part == 0 ? fa[0] + r * 64 : part == 1 ? fa[1] + (r - n0) * 64 : fa[2] + (r - n0 - n1) * 64);
            te = min(tf + 64, part == 0 ? fb[0] : part == 1 ? fb[1] : fb[2]);
            te0 = P.e0 + grp * kGenGroup;
            const int l1a = part == 2 ? 1 : 2, l1b = part == 0 ? smax - (P.q1 - I.gedges()[te - 1].layer) : part == 1 ? 3 : 1;
            ti0 = I.groff()[P.p1 + l1a];
            ti1 = l1b >= l1a ? I.groff()[P.p1 + l1b + 1] : ti0;
        }
        int units = (ti1 - ti0 + kGenRows - 1) / kGenRows, cum = units;  // inclusive prefix over the tasks
#pragma unroll
        for (int o = 1; o < kGenTasks; o <<= 1) {
            const int w = __shfl_up(cum, o, 64);
            if (lane >= o) cum += w;
        }
        const int total = nt > 0 ? uni(__shfl(cum, nt - 1, 64)) : 0;
        for (int u = wave; u < total; u += NW) {
            const int task = __popcll(__ballot(lane < nt && cum <= u));
            const int X = __builtin_amdgcn_readlane(part, task), f0 = __builtin_amdgcn_readlane(tf, task),
                      f1 = __builtin_amdgcn_readlane(te, task), e = __builtin_amdgcn_readlane(te0, task);
            const int first = __builtin_amdgcn_readlane(ti0, task) +
                              (u - __builtin_amdgcn_readlane(cum - units, task)) * kGenRows;
            const int last = min(first + kGenRows, __builtin_amdgcn_readlane(ti1, task));
            const int f = min(f0 + lane, f1 - 1), l2 = P.q1 - I.gedges()[f].layer;
            // class of the lane's loops and the left sizes it takes
            const int cls = X == 0 ? (l2 == 1 ? 2 : 0) : X;
            const int lo = X == 0 ? (l2 == 1 ? 3 : l2 < 4 ? 6 - l2 : 2) : X == 1 ? 5 - l2 : 1;
            const int hi = X == 0 ? smax - l2 : X == 1 ? 5 - l2 : 1;
            const int64_t* INf = I.IN() + (int64_t)cls * I.nil * win + f % win;
            int64_t acc[kGenGroup];
#pragma unroll
            for (int y = 0; y < kGenGroup; y++) acc[y] = kHalfINF + kBias;
            // the unit's rows are read at once (rows past its end repeat the last one)
            const GenRow& mine = I.grows()[min(first + (lane & (kGenRows - 1)), last - 1)];
            const int ml1 = mine.layer - P.p1;
            const int64_t mlg = mine.lgbase;
            int64_t in[kGenRows];
#pragma unroll
            for (int k = 0; k < kGenRows; k++) in[k] = INf[(int64_t)min(first + k, last - 1) * win];
#pragma unroll
            for (int k = 0; k < kGenRows; k++) {
                const int l1 = __builtin_amdgcn_readlane(ml1, k);
                const LongPtr lg = LG4 + (readlane64(mlg, k) + e);
                const int64_t x = l1 >= lo && l1 <= hi ? in[k] + G.size[l1][l2] : kHalfINF + kBias;
#pragma unroll
                for (int y = 0; y < kGenGroup; y++) acc[y] = min_positive(acc[y], lg[y] + x);
            }
#pragma unroll
            for (int y = 0; y < kGenGroup; y++)
                if (acc[y] < kGenBig + kBias)
                    __hip_atomic_fetch_min(&G.q[task][lane][y], acc[y], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
        if (t0 == 0) rest();
        __syncthreads();
        if (nt > 0) {
            const int ga = t0 / nbt, gb = (t0 + nt - 1) / nbt;  // edge groups of the round
            const int ea = P.e0 + ga * kGenGroup, en = min(P.e0 + P.ne, P.e0 + (gb + 1) * kGenGroup) - ea, outs = en * P.nj;
            const int parts = max(1, min(32, NT / outs));
            for (int k = wave * 64 + lane; k < outs * parts; k += NT) {
                const int e = ea + k % en, r = k / en, j = P.j0 + r % P.nj, share = r / P.nj;
                const int grp = (e - P.e0) / kGenGroup, y = (e - P.e0) % kGenGroup;
                const GenRow& row = I.grows()[j];
                const int64_t* LGj = I.LG() + row.lgbase;
                int64_t c[3];
                c[0] = c[1] = c[2] = kHalfINF + kBias;
                const int fl1 = eo[P.q1 - 1];  // right edges from here on have l2 = 1
                for (int t = max(0, grp * nbt - t0); t < min(nt, (grp + 1) * nbt - t0); t++) {
                    const int b = t0 + t - grp * nbt, X = b < n0 ? 0 : b < n0 + n1 ? 1 : 2;
                    const int f0 = X == 0 ? fa[0] + b * 64 : X == 1 ? fa[1] + (b - n0) * 64 : fa[2] + (b - n0 - n1) * 64;
                    const int cnt = min(64, (X == 0 ? fb[0] : X == 1 ? fb[1] : fb[2]) - f0);
                    int64_t v = kHalfINF + kBias, v1 = v;  // v1: l2 = 1
#pragma unroll 4
                    for (int m = share; m < cnt; m += parts) {
                        const int64_t x = G.q[t][m][y] + LGj[f0 + m];
                        if (f0 + m >= fl1) v1 = min_positive(v1, x);
                        else v = min_positive(v, x);
                    }
                    if (X == 0) {
                        c[0] = min_positive(c[0], v);
                        c[2] = min_positive(c[2], v1);
                    } else if (X == 1) {
                        c[1] = min_positive(c[1], v);
                    } else {
                        c[2] = min_positive(c[2], v);
                    }
                }
                const GenEdge& ed = I.gedges()[e];
                int64_t* w6 = G.w + ((ed.src - P.a1lo) * P.wb1 + (row.state - P.b1lo)) * 6;
                if (mn(mn(c[0], c[1]), c[2]) >= kGenBig + kBias) continue;
#pragma unroll
                for (int t = 0; t < 6; t++)
                    gen_min(w6 + t, mn(mn(c[0] + fx(S.mmI[t][ed.lab][row.lab], s), c[1] + fx(S.mm23[t][ed.lab][row.lab], s)),
                                       c[2] + fx(S.mm1n[t][ed.lab][row.lab], s)) - kBias);
            }
        }
        __syncthreads();
    }
}

// One layer pair of span step g by one workgroup.  Between the first barriers every wave takes its share
// of the tasks that read only earlier spans; then typed values, cells and the tables of the span.
template <int NT>
__device__ __forceinline__ void gen_span_group(const Inst& I, const SmallE& S, const int32_t* __restrict__ spec, int p, int q,
                                               GenShared& G) {
    const int g = q - p, s = I.shift, tid = threadIdx.x, lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    constexpr int NW = NT / 64;
    const IntPtr off = (IntPtr)(uintptr_t)I.off(), eo = (IntPtr)(uintptr_t)I.geoff(), io = (IntPtr)(uintptr_t)I.groff(),
                 re = (IntPtr)(uintptr_t)I.growedge();
    const int a_lo = off[p], wa = off[p + 1] - a_lo, b_lo = off[q], wb = off[q + 1] - b_lo, ncell = wa * wb;
    GenPair P;
    P.p = p;
    P.q = q;
    P.p1 = p + 1;
    P.q1 = q - 1;
    P.g = g;
    P.a1lo = off[p + 1];
    P.wa1 = off[p + 2] - P.a1lo;  // off has n + 2 entries and p + 1 <= n
    P.b1lo = off[q - 1];
    P.wb1 = off[q] - P.b1lo;
    P.e0 = eo[p + 1];
    P.ne = eo[p + 2] - P.e0;
    P.j0 = io[q - 1];
    P.nj = io[q] - P.j0;
    for (int k = tid; k < kGenMaxWidth * kGenMaxWidth * 6; k += NT) {
        G.w[k] = kHalfINF;
        G.v[k] = kINF;
    }
    if (tid < 2 * (kGenLoopWin + 1)) {
        const int l = tid >> 1, y = tid & 1 ? P.q1 - l : P.p1 + l;
        GenLayer L{0, 0, 0, 0};
        if (y >= 0 && y <= I.n) {
            L.first = I.off()[y];
            L.cnt = I.off()[y + 1] - L.first;
            L.row = I.rowbase()[L.first];
            L.len = I.N - I.off()[y + 1];
        }
        (tid & 1 ? G.right : G.left)[l] = L;
    }
    for (int k = tid; k < kGenTasks * 64 * (kGenGroup + 1); k += NT) (&G.q[0][0][0])[k] = kHalfINF + kBias;
    for (int k = tid; k < kGenLoopWin * 32; k += NT) {
        const int l1 = k >> 5, l2 = k & 31;
        G.size[l1][l2] = l1 > 0 && l2 > 0 && l1 + l2 <= kGenLoopWin ? fx(interior_base(S, l1, l2), s) + kBias : kBias;
    }
    GroupCounters ctr{0, 0};
    __syncthreads();
    // the loops beside the products: each starts at a wave of its own, since most fill only a few waves and one
    // wave would otherwise run all of their load chains one after another
    auto from = [&](int w) { return (tid - 64 * w) & (NT - 1); };
    auto rest = [&]() {
        for (int c0 = wave * 4; c0 < ncell; c0 += NW * 4) {
            const int ci = c0 + (lane >> 4), cv = min(ci, ncell - 1);
            gen_scan(I, p, q, a_lo + cv / wb, b_lo + cv % wb, ci < ncell, lane, G.s2 + ci, G.ps + ci, G.committed + ci);
        }
        if (g >= 9) gen_bulges(I, S, P, G, from(4), NT);
        if (g >= 5) gen_hairpins(I, S, P, G.w, from(10), NT);
        const int nspec = g == 5 || g == 6 || g == 8 ? ncell * 6 : 0;
        for (int k = wave; k < nspec; k += NW) {
            // hairpins of 3, 4 and 6 bases, whose listed loops depend on the whole label path
            const int t = k % 6, ci = k / 6, a = a_lo + ci / wb, b = b_lo + ci % wb, a1 = I.out_dst()[a * 4 + type_x(t)];
            if (a1 < 0) continue;
            const int64_t v = wave_min(hairpin_lane(I, S, spec, b, t, a1, I.out_U()[a * 4 + type_x(t)], g, lane));
            if (lane == 0) G.v[k] = v;
        }
        if (g >= 7) gen_small(I, S, P, G.w, from(3), NT);
        // gap table of this span's cells and labelled gaps (later spans read them)
        for (int ci = from(12); ci < ncell; ci += NT) {
            const int a = a_lo + ci / wb, b = b_lo + ci % wb;
            int64_t gv = kINF;
            for (int eb = I.in_start()[b]; eb < I.in_start()[b + 1]; eb++) {
                const int bp = I.in_src()[eb];
                const int64_t gp = g == 1 ? (bp == a ? 0 : kINF) : I.Gt()[I.rowoff()[a] + (bp - off[p + 1])];
                if (gp < kINF) gv = mn(gv, gp + I.in_U()[eb]);
            }
            I.Gt()[I.rowoff()[a] + (b - off[p + 1])] = gv;
        }
        if (g <= kGenLoopWin) {
            const int f0 = eo[p], nf = eo[p + 1] - f0, i0 = io[q], ni = io[q + 1] - i0;
            for (int k = from(13); k < nf * ni; k += NT) {
                const int f = f0 + k % nf, i = i0 + k / nf;
                const GenEdge& e = I.gedges()[f];
                const GenRow& row = I.grows()[i];
                int64_t lv = kINF;
                if (g == 1) {
                    if (e.row == i) lv = e.U;
                } else {
                    for (int m = 0; m < row.cnt; m++) {
                        const GenEdge& l = I.gedges()[re[row.first + m]];
                        const int64_t gg = g == 2 ? (e.dst == l.src ? 0 : kINF) : I.Gt()[I.rowoff()[e.dst] + (l.src - off[p + 2])];
                        if (gg < kINF) lv = mn(lv, e.U + gg + l.U);
                    }
                }
                I.LG()[row.lgbase + f] = lv;
            }
        }
    };
    gen_products<NT>(I, S, P, G, wave, lane, rest);
    // typed values, branch value, S1 and the retention test: eight lanes per cell, one per type
    for (int k = tid; k < ncell * 8; k += NT) {
        const int ci = k >> 3, t = k & 7, a = a_lo + ci / wb, b = b_lo + ci % wb;
        const int64_t cell = I.rowoff()[a] + (b - off[p + 1]);
        int64_t v = kINF, Bv = kINF;
        if (t < 6) {
            const int x = type_x(t), y = type_y(t), a1 = g >= 5 ? I.out_dst()[a * 4 + x] : -1;
            if (a1 >= 0) {
                for (int eb = I.in_start()[b]; eb < I.in_start()[b + 1]; eb++)
                    if (I.in_lab()[eb] == y)
                        v = mn(v, G.w[((a1 - P.a1lo) * P.wb1 + (I.in_src()[eb] - P.b1lo)) * 6 + t] + I.in_U()[eb]);
                v = mn(v + I.out_U()[a * 4 + x], G.v[ci * 6 + t]);
                if (v >= kGenBig) v = kINF;
            }
            I.V()[cell * 6 + t] = v;
            if (v < kINF) Bv = v + fx(S.ml_intern + au_pen(S, t), s);
        }
        Bv = mn(Bv, shfl_xor64(Bv, 1));
        Bv = mn(Bv, shfl_xor64(Bv, 2));
        Bv = mn(Bv, shfl_xor64(Bv, 4));
        if (t < 6) G.v[ci * 6 + t] = v;
        if (t == 0) {
            const int64_t ps = G.ps[ci];
            I.Bt()[cell] = Bv;
            I.S2()[cell] = G.s2[ci];
            I.S1()[cell] = mn(Bv, ps);
            const bool strict = Bv < ps;
            G.keep[ci] = I.retain_all ? (Bv < kINF ? (strict ? 1 : 2) : 0) : (strict ? 1 : 0);
            G.cellB[ci] = Bv;
        }
    }
    __syncthreads();
    if (wave == 0) {
        // appends in start-state order, one lane per right endpoint; candidates visited, feasible cells
        append_candidates(I, a_lo, wa, b_lo, wb, G.keep, G.cellB, g, lane);
        for (int ci = lane; ci < ncell; ci += 64) {
            ctr.visits += (unsigned long long)G.committed[ci];
            ctr.feasible += G.cellB[ci] < kINF;
        }
        if (ctr.visits) atomicAdd(&I.visits()[p], ctr.visits);
        if (ctr.feasible) atomicAdd(&I.feasible()[p], ctr.feasible);
    }
    if (g >= 5) {
        // the inner parts of interior loops around this span's cells, per class, row of a, out-edge of b
        const int f0 = eo[q], nf = eo[q + 1] - f0, i0 = io[p], ni = io[p + 1] - i0, tot = nf * ni;
        for (int k = tid; k < 3 * tot; k += NT) {
            const int X = k / tot, r = k - X * tot, f = f0 + r % nf, i = i0 + r / nf;
            const GenEdge& e = I.gedges()[f];
            const GenRow& row = I.grows()[i];
            const int64_t* vv = G.v + ((row.state - a_lo) * wb + (e.src - b_lo)) * 6;
            int64_t v = kINF;
#pragma unroll
            for (int tp = 0; tp < 6; tp++) v = mn(v, vv[tp] + fx(mmx(S, X, type_rev(tp), e.lab, row.lab), s));
            I.IN()[((int64_t)X * I.nil + i) * I.win + f % I.win] = v >= kGenBig ? kHalfINF : v;
        }
    }
}

// span step on a generic lattice: layer pair xcd_band(x) for block x < layer pairs, then the
// external column one layer behind
template <int NT>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(4))) void k_span_gen(
    Inst I, const EnergyTables* __restrict__ E, const int32_t* __restrict__ spec, int g, int ext_layer, int npairs) {
    __shared__ SmallE S;
    __shared__ union {
        GenShared g;
        GroupShared x[NT / 64];
    } G;
    stage_tables(S, E);
    if ((int)blockIdx.x >= npairs) {
        BlockTeam<NT> T;
        if (ext_layer >= 0) ext_column(I, S, ext_layer, G.x, T);
        return;
    }
    const int p = xcd_band(blockIdx.x, npairs);
    gen_span_group<NT>(rebased(I), S, spec, p, p + g, G.g);
}

// ---- batched persistent kernel ------------------------------------------------------------------
// All instances advance one global span per grid barrier.  At step g the work items are the layer
// pairs of span g of every instance with n >= g, followed (per instance) by the external column
// of layer n - g + 1 (one layer behind).  The items of a step are cut into 8 contiguous bands, one
// per workgroup group (XCD).
//
// Grid barrier.  The cell values and candidate appends are stored by many waves, and a workgroup
// barrier alone does not wait for their stores (no vmcnt wait before s_barrier).  So every wave
// first waits until its own stores are acknowledged by its XCD's L2 (vmcnt 0); after the workgroup
// barrier the workgroup arrives at the counter of its XCD (read from the hardware register, not
// assumed from the block index).  The last arrival of an XCD writes that L2 back once for all of
// them, waits for the other XCDs, and invalidates; only then are the XCD's workgroups released,
// each invalidating its own CU's cache.  A write-back and an invalidation per workgroup, on both
// sides of the barrier, queue up at the L2: with 1,024 workgroups of 256 threads a bare barrier
// took 31.2 us that way, 11.5 us with one write-back per XCD, and 4.8 us with one workgroup of
// 1,024 threads per CU; early arrivals also invalidated the caches of workgroups still working.
// Waits are polled with relaxed loads (an acquire per poll would invalidate likewise).
__device__ __forceinline__ void wait_own_stores() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");  // keeps the compiler from sinking stores
    __builtin_amdgcn_s_waitcnt(0x0F70);                      // vmcnt(0), expcnt and lgkmcnt untouched
}
__device__ __forceinline__ unsigned ctl_load(const CtlWord& w) {
    return __hip_atomic_load(&w.v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void ctl_store(CtlWord& w, unsigned v) {
    __hip_atomic_store(&w.v, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned ctl_add(CtlWord& w) {
    return __hip_atomic_fetch_add(&w.v, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1u;
}
// The XCD this workgroup runs on (hardware register XCC_ID, 4 bits).
__device__ __forceinline__ unsigned xcd_id() { return __builtin_amdgcn_s_getreg(20 | (3 << 11)) & (kMaxXcd - 1); }

// Thread 0's share of the barrier state.
struct BarrierTeam {
    unsigned xcd, members, xcds, gen;
};

// Waits until `w` no longer holds `old`; false when the wait exceeds its cap or another workgroup has
// given up.  The pause between polls grows to about 0.4 us.
__device__ __forceinline__ bool ctl_wait(BatchCtl* ctl, const CtlWord& w, unsigned old, unsigned spin_cap) {
    int pause = 1;
    for (unsigned spins = 0; ctl_load(w) == old; spins++) {
        if (spins > spin_cap || ctl_load(ctl->err)) {
            ctl_store(ctl->err, 1u);
            return false;
        }
        for (int k = 0; k < pause; k++) __builtin_amdgcn_s_sleep(2);
        if (pause < 8) pause <<= 1;
    }
    return true;
}

// Counts this workgroup at its XCD (thread 0, once, at kernel start).
__device__ __forceinline__ void barrier_join(BatchCtl* ctl, BarrierTeam& B) {
    B.xcd = xcd_id();
    ctl_add(ctl->count[B.xcd]);
    __builtin_amdgcn_s_waitcnt(0x0F70);
    ctl_add(ctl->joined);
}

// `meanwhile` is run by another wave while thread 0 waits (by the only wave, before it arrives).
template <int NT, class F>
__device__ bool grid_barrier(BatchCtl* ctl, BarrierTeam& B, unsigned spin_cap, int* s_flag, F meanwhile) {
    wait_own_stores();
    __syncthreads();
    if (NT == 64 || (threadIdx.x >> 6) == 1) meanwhile();
    if (threadIdx.x == 0) {
        bool ok = true;
        if (!B.members) {  // the first barrier: every workgroup has to be counted first
            int pause = 1;
            for (unsigned spins = 0; ok && ctl_load(ctl->joined) < gridDim.x; spins++) {
                if (spins > spin_cap || ctl_load(ctl->err)) {
                    ctl_store(ctl->err, 1u);
                    ok = false;
                }
                for (int k = 0; k < pause; k++) __builtin_amdgcn_s_sleep(2);
                if (pause < 8) pause <<= 1;
            }
            B.members = ctl_load(ctl->count[B.xcd]);
            for (int x = 0; x < kMaxXcd; x++) B.xcds += ctl_load(ctl->count[x]) != 0;
        }
        if (ok && ctl_add(ctl->arrive[B.xcd]) == B.members) {
            ctl_store(ctl->arrive[B.xcd], 0u);  // before any of its workgroups is released
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");  // writes this XCD's L2 back
            if (ctl_add(ctl->top) == B.xcds) {
                ctl_store(ctl->top, 0u);
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
                ctl_store(ctl->gen, B.gen + 1u);
            } else {
                ok = ctl_wait(ctl, ctl->gen, B.gen, spin_cap);
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
            ctl_store(ctl->release[B.xcd], B.gen + 1u);
        } else if (ok) {
            ok = ctl_wait(ctl, ctl->release[B.xcd], B.gen, spin_cap);
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        }
        B.gen++;
        *s_flag = !ok;
    }
    __syncthreads();
    return *s_flag == 0;
}

// Work items per instance at its span g = g0 + step: the layer pairs of span g, then one external
// column (layer n - g + 1, one layer behind).  pref[i] is the exclusive prefix over instances and
// pref[ninst] the step's total; by one wave, each lane a contiguous run of instances.
__device__ void step_prefix(const Inst* __restrict__ insts, int ninst, int step, int* pref, int lane) {
    const int per = (ninst + 63) / 64, lo = min(lane * per, ninst), hi = min(lo + per, ninst);
    auto items = [&](int i) {
        const int n = insts[i].n, g = insts[i].g0 + step;
        return (g <= n ? n - g + 1 : 0) + ((g >= 2 && g <= n + 1) ? 1 : 0);
    };
    int sum = 0;
    for (int i = lo; i < hi; i++) sum += items(i);
    int incl = sum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int v = __shfl_up(incl, o, 64);
        if (lane >= o) incl += v;
    }
    int acc = incl - sum;
    for (int i = lo; i < hi; i++) {
        pref[i] = acc;
        acc += items(i);
    }
    if (lane == 63) pref[ninst] = incl;
}

// the last instance whose prefix is <= item
__device__ __forceinline__ int item_instance(const int* pref, int ninst, int item) {
    int lo = 0, hi = ninst - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (pref[mid] <= item) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// Persistent launch.  The workgroup's waves share the staged energy tables and the step's prefix and
// work in teams of consecutive waves, one work item per team at a time.  A step with more items than
// the launch has waves gives every workgroup of a band each grp_blocks-th item, drawn by its waves from a
// counter in LDS (the items' costs differ; neighbouring items cost alike, so the workgroups' shares do not);
// with fewer items the teams grow (to the whole workgroup when there is at most one item per
// workgroup), since a step then takes its longest item's time, and each team's items follow from its index.
// Tickets of a band drawn by every wave from one word in memory cost 455 ms instead of 430 for 64 proteins
// of 50-1,000 aa and 70.4 instead of 63.4 for 24 of 50-400; runs of 2, 4, 8 neighbouring items per workgroup
// 434, 438, 444.  Waves by themselves have a code path of their own (no team size to carry: 431 -> 414 ms), and
// the barrier's state lies in LDS (409; 24 proteins 59.7 ms, 7 of 50-150 aa 10.6 -> 10.4).  At 128 VGPRs, eight of
// them spilled (36 B of scratch per lane) and 450 scalar registers in vector lanes.  min_team is the schedule's waves
// per item (1, or all of a 256- or 512-thread workgroup's).
template <int NT>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(4))) void k_persistent(
    const Inst* __restrict__ insts, int ninst, int nsteps, const EnergyTables* __restrict__ E,
    const int32_t* __restrict__ spec, BatchCtl* ctl, int min_team, unsigned spin_cap) {
    constexpr int NWV = NT / 64;
    __shared__ SmallE S;
    __shared__ GroupShared G[NWV];
    __shared__ int pref[kMaxBatch + 1];
    __shared__ unsigned team_ctr[NWV];
    __shared__ int s_flag;
    __shared__ unsigned s_next;
    __shared__ BarrierTeam B;  // thread 0's (in LDS: as registers it would be held by every lane)
    if (threadIdx.x == 0) {
        B = BarrierTeam();
        barrier_join(ctl, B);
    }
    stage_tables(S, E);
    const unsigned grp = blockIdx.x & 7, ngrp = gridDim.x < 8 ? gridDim.x : 8;
    const unsigned grp_blocks = (gridDim.x - grp + 7) >> 3;  // workgroups of this group
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // one wave's preparation of a step: the prefix over the instances, counters at zero.  From the second step
    // on it runs while the grid barrier is waited for: by the whole workgroup at the step's start it cost two
    // barriers and a first touch of the descriptors (and registers: 84 B of scratch per lane against 36).  64
    // proteins of 50-1,000 aa 409 -> 393 ms, 24 of 50-400 59.8 -> 55.7, 7 of 50-150 10.4 -> 9.6.
    auto prepare = [&](int step) {
        const int lane = lane_id();
        if (lane < NWV) {
            team_ctr[lane] = 0;
            G[lane].task = 0;
        }
        if (lane == 0) s_next = 0;
        step_prefix(insts, ninst, step, pref, lane);
    };
    if (wave == 0) prepare(0);
    __syncthreads();
    for (int step = 0; step < nsteps; step++) {
        const unsigned total = (unsigned)__builtin_amdgcn_readfirstlane(pref[ninst]);
        const unsigned lo_item = (unsigned)((uint64_t)total * grp / ngrp);
        const unsigned band = (unsigned)((uint64_t)total * (grp + 1) / ngrp) - lo_item;
        // the largest team that still gives every item a team at once, at least the schedule's
        int tw = min_team;
        while (tw < NWV && (uint64_t)total * (2 * tw) <= (uint64_t)gridDim.x * NWV) tw *= 2;
        WaveTeam T;
        T.n = tw;
        T.w = wave & (tw - 1);
        T.ctr = &team_ctr[wave - T.w];
        GroupShared* Gs = &G[wave - T.w];
        // team 1: the workgroup's items, drawn by its waves; larger teams: every grp_blocks * NWV / tw -th item
        const unsigned stride = grp_blocks * (unsigned)(NWV / tw);
        unsigned next = (blockIdx.x >> 3) * (unsigned)(NWV / tw) + (unsigned)(wave / tw);
        auto work = [&](unsigned k, auto& team) {
            const int item = (int)(lo_item + k);
            const int inst = __builtin_amdgcn_readfirstlane(item_instance(pref, ninst, item));
            const Inst I = load_inst(insts + inst);  // a few scalar registers: bases and sizes
            const int local = __builtin_amdgcn_readfirstlane(item - pref[inst]), g = I.g0 + step;
            const int n = I.n, ncell_items = g <= n ? n - g + 1 : 0;
            if (local < ncell_items) flush_counters(I, span_group(I, S, spec, local, local + g, Gs, team), local, team.lane());
            else ext_column(I, S, n - g + 1, Gs, team);
        };
        if (tw == 1) {
            SoloTeam solo;
            for (;;) {
                unsigned j = 0;
                if (solo.lane() == 0) j = __hip_atomic_fetch_add(&s_next, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                const unsigned k = __builtin_amdgcn_readfirstlane(j) * grp_blocks + (blockIdx.x >> 3);
                if (k >= band) break;
                work(k, solo);
            }
        } else {
            for (; next < band; next += stride) {
                work(next, T);
                T.sync();  // the team's shared state is free for its next item
            }
        }
        if (!grid_barrier<NT>(ctl, B, spin_cap, &s_flag, [&]() { prepare(step + 1); })) return;
        if (blockIdx.x == 0 && threadIdx.x == 0) ctl->steps_done.v = step + 1;
    }
}

// The schedules of full residency need four 256-thread workgroups of 160 KB of LDS per CU: launch_persistent
// runs 4 (or 2) per CU as one workgroup, and three would stay 768 workgroups that all arrive at the
// grid barrier (31 us per step against 4.8).  64 bytes for what the alignment of the arrays takes.
static_assert(4 * (sizeof(SmallE) + 4 * (sizeof(GroupShared) + sizeof(unsigned)) + (kMaxBatch + 1) * sizeof(int) + sizeof(int) +
                   sizeof(unsigned) + sizeof(BarrierTeam) + 64) <= 160 << 10,
              "four 256-thread workgroups of k_persistent fit a CU's LDS");

// Resets the barrier state and initialises every instance whose g0 is 1 (new instances): gridDim.y
// workgroups per instance.  The rings are 31 KB per state, so one workgroup per instance took 1.3 ms for 64
// proteins of 50-1,000 aa and 0.18 ms for 7 of 50-150.
__global__ void k_batch_init(const Inst* __restrict__ insts, BatchCtl* ctl) {
    const Inst I = load_inst(insts + blockIdx.x);
    const int tid = blockIdx.y * blockDim.x + threadIdx.x, nt = gridDim.y * blockDim.x;
    if (blockIdx.x == 0 && tid < kMaxXcd) {
        ctl->arrive[tid].v = 0;
        ctl->release[tid].v = 0;
        ctl->count[tid].v = 0;
        if (tid == 0) {
            ctl->joined.v = 0;
            ctl->top.v = 0;
            ctl->gen.v = 0;
            ctl->err.v = 0;
            ctl->steps_done.v = 0;
        }
    }
    if (I.g0 != 1) return;
    for (int i = tid; i < I.N; i += nt) {
        I.ccnt()[i] = 0;
        I.X()[i] = I.layer()[i] == I.n ? 0 : kINF;  // every state of the last layer is a sink
    }
    for (size_t i = tid; i < (size_t)(I.n + 1) * 2 * kLMRing; i += nt) I.LM()[i] = kINF;
    for (size_t i = tid; i < (size_t)I.N * kLMRing * 12; i += nt) {
        I.IDL()[i] = kINF;
        I.JDL()[i] = kINF;
    }
    for (size_t i = tid; i < (size_t)I.N * kLMRing; i += nt) {
        I.BI()[i] = kINF;
        I.BJ()[i] = kINF;
    }
    for (size_t i = tid; i < (size_t)I.N * kLMRing * 16; i += nt) {
        I.RS()[i] = kINF;
        I.LS()[i] = kINF;
    }
    if (tid < 4) I.stats()[tid] = tid == 2 ? ~0ull : 0ull;
    for (int i = tid; i <= I.n; i += nt) {
        I.visits()[i] = 0;
        I.feasible()[i] = 0;
    }
}

}  // namespace sd

// ---- host launch wrappers ----------------------------------------------------------------------
namespace sd {

hipError_t launch_init(const Inst& I, hipStream_t st) {
    hipLaunchKernelGGL(k_init, dim3(64), dim3(256), 0, st, I);
    return hipGetLastError();
}

// one span step: cells of span g plus the external column of layer ext_layer (or -1)
hipError_t launch_span(const Inst& I, const EnergyTables* E, const int32_t* spec, int g,
                       int ext_layer, int threads, int item_waves, int num_cu, hipStream_t st) {
    const int layers = I.n - g + 1;
    const int nblk = layers > 0 ? layers : 0;
    const int total = nblk + (ext_layer >= 0 ? 1 : 0);
    if (total == 0) return hipSuccess;
    if (item_waves == 1 && threads == 256) {  // every wave on its own pair, sixteen per workgroup
        hipLaunchKernelGGL(k_span_waves<1024>, dim3(std::min((total + 15) / 16, num_cu)), dim3(1024), 0, st, I, E, spec, g,
                           ext_layer, nblk);
        return hipGetLastError();
    }
    if (item_waves != threads / 64) return hipErrorInvalidValue;
#define SD_LAUNCH(NT, PER_CU)                                                                                      \
    hipLaunchKernelGGL(k_span<NT>, dim3(std::min(total, (PER_CU) * num_cu)), dim3(NT), 0, st, I, E, spec, g, ext_layer, nblk)
    switch (threads) {
    case 64: SD_LAUNCH(64, 4); break;
    case 256: SD_LAUNCH(256, 4); break;
    case 512: SD_LAUNCH(512, 2); break;
    case 1024: SD_LAUNCH(1024, 1); break;
    default: return hipErrorInvalidValue;
    }
#undef SD_LAUNCH
    return hipGetLastError();
}

// one span step on a generic lattice: a workgroup per layer pair, and one for the external column
hipError_t launch_span_gen(const Inst& I, const EnergyTables* E, const int32_t* spec, int g,
                           int ext_layer, hipStream_t st) {
    const int layers = I.n - g + 1;
    const int nblk = layers > 0 ? layers : 0;
    const int total = nblk + (ext_layer >= 0 ? 1 : 0);
    if (total == 0) return hipSuccess;
    hipLaunchKernelGGL(k_span_gen<1024>, dim3(total), dim3(1024), 0, st, I, E, spec, g, ext_layer, nblk);
    return hipGetLastError();
}

hipError_t launch_batch_init(const Inst* insts_dev, int ninst, BatchCtl* ctl, hipStream_t st) {
    if (ninst <= 0) return hipSuccess;
    const int parts = std::max(1, 1024 / ninst);
    hipLaunchKernelGGL(k_batch_init, dim3(ninst, parts), dim3(256), 0, st, insts_dev, ctl);
    return hipGetLastError();
}

// Schedule of the persistent launch: threads per workgroup and waves per work item.  64 threads:
// one wave per item; 256 or 512 threads with item_waves = threads / 64: the waves share each
// item; 256 threads with item_waves = 1: every wave on its own items.
bool persistent_schedule_valid(int threads, int item_waves) {
    return (threads == 64 && item_waves == 1) || (threads == 256 && (item_waves == 4 || item_waves == 1)) ||
           (threads == 512 && item_waves == 8);
}

hipError_t persistent_occupancy(int threads, int item_waves, int* blocks_per_cu) {
    if (!persistent_schedule_valid(threads, item_waves)) return hipErrorInvalidValue;
    if (threads == 64) return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, k_persistent<64>, 64, 0);
    if (threads == 512) return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, k_persistent<512>, 512, 0);
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, k_persistent<256>, 256, 0);
}

// A schedule of 2 or 4 workgroups of 256 threads on every CU runs as one workgroup of 512 or 1,024
// threads per CU: the same waves, one staging of the energy tables and one barrier arrival per CU.
hipError_t launch_persistent(const Inst* insts_dev, int ninst, int nsteps, const EnergyTables* E,
                             const int32_t* spec, BatchCtl* ctl, int grid, int threads, int item_waves, int num_cu,
                             unsigned spin_cap, hipStream_t st) {
    if (!persistent_schedule_valid(threads, item_waves)) return hipErrorInvalidValue;
    if (threads == 256 && (grid == 2 * num_cu || grid == 4 * num_cu)) {
        threads *= grid / num_cu;
        grid = num_cu;
    }
#define SD_LAUNCH(NT)                                                                                              \
    hipLaunchKernelGGL(k_persistent<NT>, dim3(grid), dim3(NT), 0, st, insts_dev, ninst, nsteps, E, spec, ctl, item_waves, \
                       spin_cap)
    if (threads == 64) SD_LAUNCH(64);
    else if (threads == 256) SD_LAUNCH(256);
    else if (threads == 512) SD_LAUNCH(512);
    else SD_LAUNCH(1024);
#undef SD_LAUNCH
    return hipGetLastError();
}

hipError_t launch_ml_abstract(const Inst& I, int g, hipStream_t st) {
    if (I.n - g + 1 <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_ml_abstract, dim3(I.n - g + 1), dim3(64), 0, st, I, g);
    return hipGetLastError();
}

hipError_t launch_checksum(const Inst& I, int g, unsigned long long* out, hipStream_t st) {
    hipError_t e = hipMemsetAsync(out, 0, sizeof(unsigned long long), st);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_checksum, dim3(256), dim3(256), 0, st, I, g, out);
    return hipGetLastError();
}

hipError_t launch_ext(const Inst& I, const EnergyTables* E, int L, hipStream_t st) {
    hipLaunchKernelGGL(k_ext, dim3(1), dim3(256), 0, st, I, E, L);
    return hipGetLastError();
}

}  // namespace sd
