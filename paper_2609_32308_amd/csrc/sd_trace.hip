// Canonical first-match traceback on the device (Sec. 5: the traceback is deferred until the
// fill is complete and reconstructs every decision from the stored costs; Sec. 7: optima are
// often tied, so one fixed order of alternatives makes the emitted design reproducible).
//
// A workgroup of eight wavefronts per design replays the decisions from X(s).  A decision either
// continues in the same wave or also defers an independent sub-interval (the rest of the external
// loop beside a closed pair, the left part of a multiloop split), which a free wave takes from a
// shared stack.  At each decision the alternatives are enumerated in a fixed order and the first
// whose value equals the stored value exactly is taken, so the design does not depend on which
// wave replays which interval:
//   X(a):   unpaired out-edges by label; then branches (b by state index, pair type in the order
//           AU, CG, GC, GU, UA, UG)
//   V_t:    hairpin (sizes 3, 4, 6: paths in lexicographic base order; other sizes: x_{i+1} by
//           base, the closing in-edge of b, the in-edge of b1), then two-loops (l1 ascending,
//           l2 ascending, closing in-edge of b, inner c by index, d by index, inner type, left
//           segment, right segment), then the multiloop (closing in-edge of b)
//   S1:     direct branch, S2, left unpaired edge (by label), right unpaired edge (in-edge order)
//   S2:     right unpaired edge (in-edge order), then candidates c of C_b by state index (eq. 7)
//   branch: pair type order
//   gaps:   the minimum-cost path that takes the smallest base staying on a minimum path
// The lanes of a wave evaluate alternatives side by side and the first match is the lowest set
// lane of a ballot (or the wave minimum of the matching indices), which is what a sequential
// replay in this order picks.  Two-loop alternatives are grouped by (l1, l2, closing edge, c, d); a group
// is enumerated only if an exact lower bound (segment costs at their minima, the gap costs;
// the loop energy at the minimum of its table over boundary bases and inner types) does not
// already exceed the stored value.  The decisions only read the completed tables, so the design
// does not depend on how the fill was scheduled.
//
// Only O(n) results leave the device: the base at every position, the partner of every paired
// position, the energy, the path cost, a status and X(s).
#include <hip/hip_runtime.h>

#include <limits.h>

#include "sd_devutil.h"
#include "sd_internal.h"
#include "sd_trace_status.h"

namespace sd {
namespace {

enum : int { kFX = 0, kFV = 1, kFS1 = 2, kFS2 = 3, kFBR = 4 };

__device__ __forceinline__ int64_t sadd(int64_t a, int64_t b) { return (a >= kINF || b >= kINF) ? kINF : a + b; }
__device__ __forceinline__ int first_lane(unsigned long long m) { return __ffsll((unsigned long long)m) - 1; }
__device__ __forceinline__ int bcast(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ int wmin_int(int v) { return (int)wave_min((int64_t)v); }

// minimum path cost u -> v (INF if unreachable): the trie's closed form, or the device gap table
// of a generic lattice
__device__ __forceinline__ int64_t tgap(const Inst& I, int u, int v) {
    const int lu = I.layer()[u], lv = I.layer()[v];
    if (lu == lv) return u == v ? 0 : kINF;
    if (lu > lv) return kINF;
    if (I.gwin) return I.Gt()[I.rowoff()[u] + (v - I.off()[lu + 1])];
    const int ku = lu / 3, kv = lv / 3;
    if (ku == kv) {
        if (lu % 3 == 0) return 0;
        return (I.pfx()[v] >> 2) == I.pfx()[u] ? 0 : kINF;
    }
    return I.tail()[u] + I.P()[kv] - I.P()[ku + 1];
}
__device__ __forceinline__ int64_t tcell(const Inst& I, int a, int b) {
    if (I.gwin) return I.rowbase()[a] + b;
    return I.rowoff()[a] + (b - I.off()[I.layer()[a] + 1]);
}
__device__ __forceinline__ bool fwd(const Inst& I, int a, int b) { return I.layer()[a] < I.layer()[b]; }
__device__ __forceinline__ int64_t tV(const Inst& I, int t, int a, int b) { return fwd(I, a, b) ? I.V()[tcell(I, a, b) * 6 + t] : kINF; }
__device__ __forceinline__ int64_t tB(const Inst& I, int a, int b) { return fwd(I, a, b) ? I.Bt()[tcell(I, a, b)] : kINF; }
__device__ __forceinline__ int64_t tS1(const Inst& I, int a, int b) { return fwd(I, a, b) ? I.S1()[tcell(I, a, b)] : kINF; }
__device__ __forceinline__ int64_t tS2(const Inst& I, int a, int b) { return fwd(I, a, b) ? I.S2()[tcell(I, a, b)] : kINF; }

// loop energy of a two-loop (stack, bulge, interior) closed by t around the reversed inner type tr
__device__ __forceinline__ int32_t two_loop_e(const SmallE& S, int t, int tr, int l1, int l2, int xi, int xk, int xl,
                                              int xj) {
    if (l1 == 0 && l2 == 0) return S.stack[t][tr];
    if (l1 == 0 || l2 == 0) return bulge_e(S, t, tr, l1 + l2);
    return interior_e(S, nullptr, t, tr, l1, l2, xi, xk, xl, xj);
}

// lower bound of two_loop_e(t, *, l1, l2, *) over inner types and boundary bases
__device__ __forceinline__ int32_t two_loop_lb(const SmallE& S, int t, int l1, int l2) {
    const LoopMin& M = S.lmin;
    if (l1 == 0 && l2 == 0) return M.stack[t];
    if (l1 == 0 || l2 == 0) {
        const int l = l1 + l2;
        return l == 1 ? S.bulge[1] + M.stack[t] : S.bulge[l] + au_pen(S, t) + M.au_min;
    }
    if (l1 == 1 && l2 == 1) return M.int11[t];
    if (l1 == 1 && l2 == 2) return M.int12[t];
    if (l1 == 2 && l2 == 1) return M.int21[t];
    if (l1 == 2 && l2 == 2) return M.int22[t];
    const int X = mm_class(l1, l2);
    return interior_base(S, l1, l2) + M.mm_out[X][t] + M.mm_in[X];
}

struct Seg {
    int e1, e2, gfrom, gto, xa, xb;  // out-edge id of the first base, in-edge index of the last
    int64_t cost;
};

// The idx-th segment of l bases from u to v in canonical order (first base, then the in-edge of
// v in CSR order); false if there are fewer.  With idx < 0 the count is returned in *count.
__device__ bool seg_at(const Inst& I, int u, int v, int l, int idx, Seg& s, int* count = nullptr) {
    int k = 0;
    if (l == 0) {
        if (u == v) {
            if (k == idx) {
                s = Seg{-1, -1, -1, -1, 0, 0, 0};
                return true;
            }
            k++;
        }
    } else if (l == 1) {
        for (int x = 0; x < 4; x++) {
            const int e = u * 4 + x;
            if (I.out_dst()[e] != v) continue;
            if (k == idx) {
                s = Seg{e, -1, -1, -1, x, x, I.out_U()[e]};
                return true;
            }
            k++;
        }
    } else {
        const int j0 = I.in_start()[v], j1 = I.in_start()[v + 1];
        for (int x = 0; x < 4; x++) {
            const int e = u * 4 + x, u2 = I.out_dst()[e];
            if (u2 < 0) continue;
            for (int j = j0; j < j1; j++) {
                const int64_t gg = tgap(I, u2, I.in_src()[j]);
                if (gg >= kINF) continue;
                if (k == idx) {
                    s = Seg{e, j, u2, I.in_src()[j], x, I.in_lab()[j], I.out_U()[e] + gg + I.in_U()[j]};
                    return true;
                }
                k++;
            }
        }
    }
    if (count) *count = k;
    return false;
}

// The segments of l bases from u to v, one at a time, in seg_at's order.
struct SegIter {
    int u, v, l, x, j, j0, j1;
    bool done;
    __device__ SegIter(const Inst& I, int u_, int v_, int l_) : u(u_), v(v_), l(l_), x(0), done(false) {
        j0 = l >= 2 ? I.in_start()[v] : 0;
        j1 = l >= 2 ? I.in_start()[v + 1] : 0;
        j = j0;
    }
    __device__ bool next(const Inst& I, Seg& s) {
        if (l == 0) {
            if (done || u != v) return false;
            done = true;
            s = Seg{-1, -1, -1, -1, 0, 0, 0};
            return true;
        }
        if (l == 1) {
            while (x < 4) {
                const int e = u * 4 + x++;
                if (I.out_dst()[e] == v) {
                    s = Seg{e, -1, -1, -1, e & 3, e & 3, I.out_U()[e]};
                    return true;
                }
            }
            return false;
        }
        while (x < 4) {
            const int e = u * 4 + x, u2 = I.out_dst()[e];
            if (u2 >= 0)
                while (j < j1) {
                    const int jj = j++;
                    const int64_t gg = tgap(I, u2, I.in_src()[jj]);
                    if (gg < kINF) {
                        s = Seg{e, jj, u2, I.in_src()[jj], x, I.in_lab()[jj], I.out_U()[e] + gg + I.in_U()[jj]};
                        return true;
                    }
                }
            x++;
            j = j0;
        }
        return false;
    }
};

// Waves per design: deferred decisions of independent sub-intervals (the rest of the external
// loop beside a closed pair; the left part of a multiloop split beside its last branch) are taken
// by whichever wave is free.
constexpr int kTraceWaves = 8;
constexpr unsigned kTraceSpinCap = 1u << 24;  // polls before a wait is declared failed

constexpr int kHelix = 16;  // stacks replayed per look-up of their cells

// one wave's scratch for the decision it is working on
struct TraceScratch {
    int pre[kNumPairs + 1];  // tuples of the two-loop pairs before pair k
    int jl[64];              // in-edges of b labelled y (closing edge of a pair)
    int hpre[65];            // generic hairpins: prefix of in-degrees of the b1 of jl
    // codon trie: the inner states at every distance l from the closing pair, index 2 l + slot
    int64_t gl[64], row[64];  // gap a1 ~> c (infinite: no such state or path), row base of c
    int64_t gr[2][64];        // gap d ~> b1 for each slot of b1
    int st[64];               // state of d
    // helices: values of the cells (layer p + k + 1, layer q - k - 1) at index 4 k + 2 slot + slot, costs and
    // targets (a byte per label) of the edges out of layers p + k and q - 1 - k at index 2 k + slot
    int64_t hv[4 * kHelix][6], lu[2 * kHelix + 2][4], ru[2 * kHelix + 2][4];
    int ldst[2 * kHelix + 2], rdst[2 * kHelix + 2];
};

struct TraceLds {
    SmallE S;
    unsigned char pl1[kNumPairs], pl2[kNumPairs];
    TraceScratch w[kTraceWaves];
    // the shared stack of deferred frames (frames in region A, its top here), guarded by `lock`
    int lock, sp, busy, failed, emitted;
    unsigned long long E, U;  // sums over the waves (two's complement)
};

// A wavefront's replay state; every lane holds the same values.
struct Tracer {
    const Inst& I;
    TraceLds& L;
    TraceScratch& W;
    const int32_t* spec;
    int lane;
    int64_t E = 0, U = 0;
    bool fail = false;
    int emitted = 0;   // bases this wave emitted (over all waves n, or one was emitted twice)
    TFrame next;
    bool have_next = false;
    // what is known of the next closed value beside its frame (codon trie): layers, slots, value
    bool known = false;
    int kp = 0, kq = 0, kia = 0, kib = 0;
    int64_t kv = 0;
    bool no_stack = false;     // the next closed value is known not to be a stack
    int64_t El = 0, Ul = 0;    // this lane's shares of E and U beside the wave's

    __device__ Tracer(const Inst& I_, TraceLds& L_, TraceScratch& W_, const int32_t* sp_, int ln)
        : I(I_), L(L_), W(W_), spec(sp_), lane(ln) {}

    __device__ int64_t fxe(int64_t e) const { return e * ((int64_t)1 << I.shift); }

    // the stack's lock: lane 0 spins, the whole wave then orders its accesses after it
    __device__ bool lock() {
        int ok = 1;
        if (lane == 0) {
            unsigned spins = 0;
            while (atomicCAS(&L.lock, 0, 1) != 0) {
                if (++spins > kTraceSpinCap) {
                    ok = 0;
                    break;
                }
                __builtin_amdgcn_s_sleep(1);
            }
        }
        ok = bcast(ok);
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
        if (!ok) fail_all(kTrWait);
        return ok;
    }
    // A workgroup-scope release waits only for LDS operations, so the frame a push stored, or the
    // frame a take is still loading from a slot a later push may reuse, is waited for explicitly
    // (vmcnt 0) before the lock is given up.  All waves of the design share this CU's L2.
    __device__ void unlock() {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0), expcnt and lgkmcnt untouched
        __builtin_amdgcn_wave_barrier();
        if (lane == 0) atomicExch(&L.lock, 0);
    }
    // ends every wave's replay; the first reason recorded is the one reported
    __device__ void fail_all(int reason) {
        fail = true;
        if (lane == 0) atomicCAS(&L.failed, 0, reason);
    }
    // Frames move between waves through region A.  Stack slots are reused, so they are written
    // and read with agent-scope atomic accesses (to L2, past this CU's L1 copy of the slot); the
    // lock's release and acquire order them.
    __device__ static void store_frame(TFrame* p, const TFrame& f) {
        __hip_atomic_store(&p->kind, f.kind, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&p->a, f.a, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&p->b, f.b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&p->t, f.t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __device__ static TFrame load_frame(TFrame* p) {
        return TFrame{__hip_atomic_load(&p->kind, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT),
                      __hip_atomic_load(&p->a, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT),
                      __hip_atomic_load(&p->b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT),
                      __hip_atomic_load(&p->t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)};
    }
    // defers a decision to the shared stack (at most n + 2 frames: each covers a disjoint interval)
    __device__ void push(int kind, int a, int b, int t) {
        if (!lock()) return;
        int over = 0;
        if (lane == 0) {
            const int slot = L.sp;
            if (slot >= I.n + 2) {
                over = 1;
            } else {
                store_frame(I.tr_stack() + slot, TFrame{kind, a, b, t});
                L.sp = slot + 1;
            }
        }
        unlock();
        if (bcast(over)) fail_all(kTrStack);
    }
    // The next deferred frame once this wave's chain has ended (a wave counted busy stops being
    // busy first): true with a frame (the wave is busy again), false when no wave is busy and the
    // stack is empty, or on failure.  Waiting waves poll the stack's state with plain loads and
    // take the lock only to pop a frame or to confirm the end, so that they do not keep the lock
    // from the busy waves' pushes.
    __device__ bool take(TFrame& f, bool was_busy) {
        if (was_busy) {
            if (!lock()) return false;
            if (lane == 0) L.busy--;
            unlock();
        }
        for (unsigned spins = 0;; spins++) {
            int look = 0;  // 1: a frame to pop or a possible end, 2: failed
            if (lane == 0) {
                const int fl = __hip_atomic_load(&L.failed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                const int sp = __hip_atomic_load(&L.sp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                const int bz = __hip_atomic_load(&L.busy, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                look = fl ? 2 : (sp > 0 || bz == 0) ? 1 : 0;
            }
            look = bcast(look);
            if (look == 2) return false;
            if (look == 1) {
                if (!lock()) return false;
                int st = 0;  // 0: wait, 1: frame, 2: done
                TFrame h{0, 0, 0, 0};
                if (lane == 0) {
                    if (L.failed) {
                        st = 2;
                    } else if (L.sp > 0) {
                        h = load_frame(I.tr_stack() + --L.sp);
                        L.busy++;
                        st = 1;
                    } else if (L.busy == 0) {
                        st = 2;
                    }
                }
                unlock();
                st = bcast(st);
                if (st == 1) {
                    f = TFrame{bcast(h.kind), bcast(h.a), bcast(h.b), bcast(h.t)};
                    // a frame names states of this design (a corrupted one would index out of range)
                    if (f.kind < kFX || f.kind > kFBR || f.a < 0 || f.a >= I.N || f.b < -1 || f.b >= I.N ||
                        f.t < -1 || f.t >= 6) {
                        fail_all(kTrFrame);
                        return false;
                    }
                    return true;
                }
                if (st == 2) return false;
            }
            if (spins > kTraceSpinCap) {
                fail_all(kTrWait);
                return false;
            }
            __builtin_amdgcn_s_sleep(4);
        }
    }
    __device__ void go(int kind, int a, int b, int t) {
        next = TFrame{kind, a, b, t};
        have_next = true;
        known = no_stack = false;
    }
    __device__ void emit_at(int pos, int lab, int64_t cost) {
        if (lane == 0) I.tr_seq()[pos] = lab;
        emitted++;
        U += cost;
    }
    __device__ void emit_out(int e) { emit_at(I.layer()[e >> 2], e & 3, I.out_U()[e]); }
    __device__ void emit_in(int j) { emit_at(I.layer()[I.in_src()[j]], I.in_lab()[j], I.in_U()[j]); }
    // the minimum-cost path u -> v, smallest base first at every step (lanes 0..3 try the bases)
    __device__ void emit_gap(int u, int v) {
        while (u != v && !fail) {
            const int64_t g = tgap(I, u, v);
            bool ok = false;
            int d = -1;
            if (lane < 4) {
                const int e = u * 4 + lane;
                d = I.out_dst()[e];
                ok = d >= 0 && sadd(I.out_U()[e], tgap(I, d, v)) == g;
            }
            const unsigned long long m = __ballot(ok);
            if (!m) {
                fail = true;
                return;
            }
            const int x = first_lane(m);
            emit_out(u * 4 + x);
            u = I.out_dst()[u * 4 + x];
        }
    }
    __device__ void emit_seg(const Seg& s) {
        if (s.e1 >= 0) emit_out(s.e1);
        if (s.e2 >= 0) {
            emit_gap(s.gfrom, s.gto);
            emit_in(s.e2);
        }
    }

    __device__ void ext(int a);
    __device__ void closed(int a, int b, int t);
    __device__ bool hairpin(int a, int b, int t, int64_t v, int ea, int a1);
    __device__ bool twoloop(int a, int b, int t, int64_t v, int ea, int a1);
    __device__ void closed_trie(int a, int b, int t, int p, int q, int ia, int ib, int64_t v);
    __device__ bool helix(int t, int p, int q, int ia, int ib, int64_t v);
    __device__ void s1(int a, int b);
    __device__ void s2(int a, int b);
    __device__ void branch(int a, int b);
};

__device__ void Tracer::ext(int a) {
    if (I.layer()[a] == I.n) return;
    const int64_t x = I.X()[a];
    bool ok = false;
    if (lane < 4) {
        const int d = I.out_dst()[a * 4 + lane];
        ok = d >= 0 && sadd(I.out_U()[a * 4 + lane], I.X()[d]) == x;
    }
    unsigned long long m = __ballot(ok);
    if (m) {
        const int y = first_lane(m), e = a * 4 + y;
        emit_out(e);
        go(kFX, I.out_dst()[e], -1, -1);
        return;
    }
    // branches b (state order), pair types in order; one state per lane
    const int la = I.layer()[a];
    const int b0 = la + 5 <= I.n ? I.off()[la + 5] : I.N;
    const int64_t* Br = I.Bt() + I.rowoff()[a] - I.off()[la + 1];
    for (int base = b0; base < I.N; base += 64) {
        const int bb = base + lane;
        // the branch value holds min over t of V_t + ML_intern + AU, and no branch lies below X(a): a
        // state matches exactly if its branch value does
        const bool hit = bb < I.N && sadd(sadd(Br[bb], -fxe(L.S.ml_intern)), I.X()[bb]) == x;
        const unsigned long long hm = __ballot(hit);
        if (hm) {
            const int b = base + first_lane(hm);
            const int64_t xb = I.X()[b];
            bool th = false;
            if (lane < 6) th = sadd(sadd(tV(I, lane, a, b), fxe(au_pen(L.S, lane))), xb) == x;
            const unsigned long long tmk = __ballot(th);
            if (!tmk) break;
            const int t = first_lane(tmk);
            E += au_pen(L.S, t);
            push(kFX, b, -1, -1);
            go(kFV, a, b, t);
            return;
        }
    }
    fail = true;
}

__device__ bool Tracer::hairpin(int a, int b, int t, int64_t v, int ea, int a1) {
    const int g = I.layer()[b] - I.layer()[a], m = g - 2;
    if (m < 3) return false;
    if (m == 3 || m == 4 || m == 6) {
        // every label path of g edges from a whose first base is x and last base y, in
        // lexicographic order: the middle g - 2 bases are the digits of the lane's combination
        const int mid = g - 2, combos = 1 << (2 * mid);
        const int off = m == 3 ? kSpecOff5 : m == 4 ? kSpecOff6 : kSpecOff8;
        // the bases before the last three are the whole wave's: they are walked once, and a missing label
        // skips every combination that begins alike (of the 64 beginnings of a 6-base loop a few exist; trying
        // them all took 78 us)
        const int np = mid - 2;  // edges walked together: the closing one and mid - 3
        for (int base = 0; base < combos; base += 64) {
            int st0 = a, key0 = 0, first = 0, miss = -1;
            int64_t cost0 = 0;
            for (int i = 0; i < np && miss < 0; i++) {
                const int lab = i == 0 ? kTX[t] : (base >> (2 * (mid - i))) & 3;
                const int e = st0 * 4 + lab, d = bcast(I.out_dst()[e]);
                if (i == 1) first = lab;
                cost0 += I.out_U()[e];
                key0 = key0 * 4 + lab;
                if (d < 0) miss = i;
                st0 = d;
            }
            if (miss == 0) return false;
            if (miss > 0) {
                base |= (64 << (2 * (np - 1 - miss))) - 64;
                continue;
            }
            const int cmb = base + lane;
            bool ok = false;
            int32_t en = 0;
            if (cmb < combos) {
                int st = st0, key = key0, l1 = first, lm = 0;
                int64_t cost = cost0;
                ok = true;
                for (int i = np; i < g && ok; i++) {
                    const int lab = i == 0 ? kTX[t] : i == g - 1 ? kTY[t] : (cmb >> (2 * (mid - i))) & 3;
                    if (i == 1) l1 = lab;
                    if (i == g - 2) lm = lab;
                    const int e = st * 4 + lab, d = I.out_dst()[e];
                    if (d < 0) ok = false;
                    else {
                        cost += I.out_U()[e];
                        key = key * 4 + lab;
                        st = d;
                    }
                }
                if (ok && st == b) {
                    en = spec[off + key];
                    if (en == kNoSpecial) en = I.hp_init()[m] + (m == 3 ? au_pen(L.S, t) : L.S.mmH[t][l1][lm]);
                    ok = cost + fxe(en) == v;
                } else {
                    ok = false;
                }
            }
            const unsigned long long msk = __ballot(ok);
            if (msk) {
                const int win = base + first_lane(msk);
                int st = a, key = 0, l1 = 0, lm = 0;
                for (int i = 0; i < g; i++) {
                    const int lab = i == 0 ? kTX[t] : i == g - 1 ? kTY[t] : (win >> (2 * (mid - i))) & 3;
                    if (i == 1) l1 = lab;
                    if (i == g - 2) lm = lab;
                    emit_out(st * 4 + lab);
                    key = key * 4 + lab;
                    st = I.out_dst()[st * 4 + lab];
                }
                int32_t e2 = spec[off + key];
                if (e2 == kNoSpecial) e2 = I.hp_init()[m] + (m == 3 ? au_pen(L.S, t) : L.S.mmH[t][l1][lm]);
                E += e2;
                return true;
            }
        }
        return false;
    }
    // generic size: a -x-> a1 -x2-> a2 ~~> b2 -z-> b1 -y-> b, alternatives (x2, closing in-edge of
    // b, in-edge of b1) in order, flattened over the lanes with the prefix of the b1 in-degrees
    const int y = kTY[t];
    const int ib0 = I.in_start()[b], ib1 = I.in_start()[b + 1];
    int nj = 0;
    for (int j0 = ib0; j0 < ib1; j0 += 64) {
        const int j = j0 + lane;
        const bool lab = j < ib1 && I.in_lab()[j] == y;
        const unsigned long long msk = __ballot(lab);
        const int at = nj + __popcll(msk & ((1ull << lane) - 1));
        if (lab && at < 64) W.jl[at] = j;
        nj += __popcll(msk);
    }
    if (nj > 64) nj = 64;  // a state has at most 64 in-edges (4 labels x 16 sources)
    __builtin_amdgcn_wave_barrier();
    int deg = 0;
    if (lane < nj) {
        const int b1 = I.in_src()[W.jl[lane]];
        deg = I.in_start()[b1 + 1] - I.in_start()[b1];
    }
    int incl = deg;
    for (int o = 1; o < 64; o <<= 1) {
        const int w = __shfl_up(incl, o, 64);
        if (lane >= o) incl += w;
    }
    if (lane < nj) W.hpre[lane + 1] = incl;
    if (lane == 0) W.hpre[0] = 0;
    __builtin_amdgcn_wave_barrier();
    const int per = bcast(__shfl(incl, 63, 64));
    const int total = 4 * per;
    const int64_t Ua = I.out_U()[ea];
    for (int base = 0; base < total; base += 64) {
        const int idx = base + lane;
        bool ok = false;
        if (idx < total) {
            const int x2 = idx / per, r = idx - x2 * per;
            int jj = 0;
            while (jj + 1 < nj && W.hpre[jj + 1] <= r) jj++;
            const int j = W.jl[jj], b1 = I.in_src()[j];
            const int j2 = I.in_start()[b1] + (r - W.hpre[jj]);
            const int e1 = a1 * 4 + x2, a2 = I.out_dst()[e1];
            if (a2 >= 0) {
                const int64_t gg = tgap(I, a2, I.in_src()[j2]);
                if (gg < kINF) {
                    const int32_t en = I.hp_init()[m] + L.S.mmH[t][x2][I.in_lab()[j2]];
                    ok = Ua + I.out_U()[e1] + gg + I.in_U()[j2] + I.in_U()[j] + fxe(en) == v;
                }
            }
        }
        const unsigned long long msk = __ballot(ok);
        if (msk) {
            const int win = base + first_lane(msk);
            const int x2 = win / per, r = win - x2 * per;
            int jj = 0;
            while (jj + 1 < nj && W.hpre[jj + 1] <= r) jj++;
            const int j = W.jl[jj], b1 = I.in_src()[j];
            const int j2 = I.in_start()[b1] + (r - W.hpre[jj]);
            const int e1 = a1 * 4 + x2;
            emit_out(ea);
            emit_out(e1);
            emit_gap(I.out_dst()[e1], I.in_src()[j2]);
            emit_in(j2);
            emit_in(j);
            E += I.hp_init()[m] + L.S.mmH[t][x2][I.in_lab()[j2]];
            return true;
        }
    }
    return false;
}

__device__ bool Tracer::twoloop(int a, int b, int t, int64_t v, int ea, int a1) {
    const int la = I.layer()[a], lb = I.layer()[b], g = lb - la;
    if (g < 7) return false;
    const int y = kTY[t];
    // closing in-edges of b labelled y, in CSR order
    const int ib0 = I.in_start()[b], ib1 = I.in_start()[b + 1];
    int nj = 0;
    for (int j0 = ib0; j0 < ib1; j0 += 64) {
        const int j = j0 + lane;
        const bool lab = j < ib1 && I.in_lab()[j] == y;
        const unsigned long long msk = __ballot(lab);
        const int at = nj + __popcll(msk & ((1ull << lane) - 1));
        if (lab && at < 64) W.jl[at] = j;
        nj += __popcll(msk);
    }
    if (nj > 64) nj = 64;
    if (nj == 0) return false;
    __builtin_amdgcn_wave_barrier();
    // stacks come first in the order and match most often: (closing edge, inner type) over the lanes,
    // without the list of all pairs (generic lattices; 105 residues, fill to result: 3.5 -> 2.8 ms)
    for (int base = 0; base < nj * 6; base += 64) {
        const int idx = base + lane, jj = min(idx / 6, nj - 1), tp = idx % 6, j = W.jl[jj];
        const int64_t vin = tV(I, tp, a1, I.in_src()[j]);
        const bool ok = idx < nj * 6 && vin < kINF && I.out_U()[ea] + vin + I.in_U()[j] + fxe(L.S.stack[t][kRev[tp]]) == v;
        const unsigned long long msk = __ballot(ok);
        if (msk) {
            const int win = base + first_lane(msk), jw = W.jl[win / 6], tw = win % 6;
            emit_out(ea);
            emit_in(jw);
            E += L.S.stack[t][kRev[tw]];
            go(kFV, a1, I.in_src()[jw], tw);
            return true;
        }
    }
    // tuples (pair k, closing edge, c, d) per pair: nj * width(cl) * width(dl) when the pair fits
    // (l1 + l2 <= g - 7); prefix over the pairs in canonical order, eight pairs per lane
    {
        int cnt[8], sum = 0;
        for (int i = 0; i < 8; i++) {
            const int k = lane * 8 + i;
            int c = 0;
            if (k < kNumPairs) {
                const int l1 = L.pl1[k], l2 = L.pl2[k];
                if (l1 + l2 <= g - 7) {
                    const int cl = la + 1 + l1, dl = lb - 1 - l2;
                    c = nj * (I.off()[cl + 1] - I.off()[cl]) * (I.off()[dl + 1] - I.off()[dl]);
                }
            }
            cnt[i] = c;
            sum += c;
        }
        int incl = sum;
        for (int o = 1; o < 64; o <<= 1) {
            const int w = __shfl_up(incl, o, 64);
            if (lane >= o) incl += w;
        }
        int acc = incl - sum;
        for (int i = 0; i < 8; i++) {
            const int k = lane * 8 + i;
            if (k <= kNumPairs) W.pre[k] = acc;
            acc += cnt[i];
        }
        __builtin_amdgcn_wave_barrier();
    }
    const int total = W.pre[kNumPairs];
    const int64_t Ua = I.out_U()[ea];
    // four groups per lane and round (group T = base + lane + 64 k): their independent loads are
    // issued together, then each group's lower bound is tested and, rarely, its alternatives
    // enumerated; the lane's first match is its smallest matching group
    constexpr int kPer = 4;
    for (int base = 0; base < total; base += 64 * kPer) {
        int code = INT_MAX;  // the lane's first matching group and its (tp, p, q)
        int wtp = 0, wp = 0, wq = 0;
        int tl1[kPer], tl2[kPer], tc[kPer], td[kPer], tj[kPer], tb1[kPer];
        int64_t tU[kPer], tgl[kPer], tgr[kPer];
        const int64_t* tvr[kPer];
#pragma unroll
        for (int k = 0; k < kPer; k++) {
            const int T = base + lane + 64 * k;
            tl1[k] = -1;
            if (T >= total) continue;
            int lo = 0, hi = kNumPairs - 1;  // last pair whose prefix <= T
            while (lo < hi) {
                const int mid = (lo + hi + 1) >> 1;
                if (W.pre[mid] <= T) lo = mid;
                else hi = mid - 1;
            }
            const int l1 = L.pl1[lo], l2 = L.pl2[lo];
            const int cl = la + 1 + l1, dl = lb - 1 - l2;
            const int c0 = I.off()[cl], d0 = I.off()[dl];
            const int wc = I.off()[cl + 1] - c0, wd = I.off()[dl + 1] - d0;
            const int r = T - W.pre[lo], jj = r / (wc * wd), ci = (r / wd) % wc, di = r % wd;
            tl1[k] = l1;
            tl2[k] = l2;
            tc[k] = c0 + ci;
            td[k] = d0 + di;
            tj[k] = W.jl[jj];
        }
#pragma unroll
        for (int k = 0; k < kPer; k++) {
            if (tl1[k] < 0) continue;
            tb1[k] = I.in_src()[tj[k]];
            tU[k] = I.in_U()[tj[k]];
            tvr[k] = I.V() + tcell(I, tc[k], td[k]) * 6;
        }
#pragma unroll
        for (int k = 0; k < kPer; k++) {
            if (tl1[k] < 0) continue;
            tgl[k] = tl1[k] == 0 ? (a1 == tc[k] ? 0 : kINF) : tgap(I, a1, tc[k]);
            tgr[k] = tl2[k] == 0 ? (td[k] == tb1[k] ? 0 : kINF) : tgap(I, td[k], tb1[k]);
        }
        for (int k = 0; k < kPer && code == INT_MAX; k++) {
            if (tl1[k] < 0 || tgl[k] >= kINF || tgr[k] >= kINF) continue;
            const int l1 = tl1[k], l2 = tl2[k], c = tc[k], d = td[k], b1 = tb1[k];
            const int64_t* vr = tvr[k];
            int64_t vmin = kINF;
            for (int tp = 0; tp < 6; tp++) vmin = mn(vmin, vr[tp]);
            // exact lower bound of every alternative of the group
            const int64_t lb0 = Ua + tgl[k] + tgr[k] + tU[k] + fxe(two_loop_lb(L.S, t, l1, l2));
            if (vmin >= kINF || lb0 + vmin > v) continue;
            // enumerate (inner type, left segment, right segment) in order
            for (int tp = 0; tp < 6 && code == INT_MAX; tp++) {
                const int64_t vin = vr[tp];
                if (vin >= kINF || lb0 + vin > v) continue;
                const int tr = kRev[tp];
                Seg sl, sr;
                SegIter li(I, a1, c, l1);
                for (int p = 0; code == INT_MAX && li.next(I, sl); p++) {
                    SegIter ri(I, d, b1, l2);
                    for (int q = 0; code == INT_MAX && ri.next(I, sr); q++) {
                        const int32_t e2 = two_loop_e(L.S, t, tr, l1, l2, sl.xa, sl.xb, sr.xa, sr.xb);
                        if (Ua + sl.cost + vin + sr.cost + tU[k] + fxe(e2) == v) {
                            code = base + lane + 64 * k;
                            wtp = tp;
                            wp = p;
                            wq = q;
                        }
                    }
                }
            }
        }
        const int best = wmin_int(code);
        if (best == INT_MAX) continue;
        const int wl = first_lane(__ballot(code == best));
        const int tp = __shfl(wtp, wl, 64), p = __shfl(wp, wl, 64), q = __shfl(wq, wl, 64);
        // decode the winning tuple (uniform)
        int lo = 0, hi = kNumPairs - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (W.pre[mid] <= best) lo = mid;
            else hi = mid - 1;
        }
        const int k = lo, l1 = L.pl1[k], l2 = L.pl2[k];
        const int cl = la + 1 + l1, dl = lb - 1 - l2;
        const int wc = I.off()[cl + 1] - I.off()[cl], wd = I.off()[dl + 1] - I.off()[dl];
        const int r = best - W.pre[k], jj = r / (wc * wd), ci = (r / wd) % wc, di = r % wd;
        const int j = W.jl[jj], b1 = I.in_src()[j], c = I.off()[cl] + ci, d = I.off()[dl] + di;
        Seg sl, sr;
        seg_at(I, a1, c, l1, p, sl);
        seg_at(I, d, b1, l2, q, sr);
        const int32_t e2 = two_loop_e(L.S, t, kRev[tp], l1, l2, sl.xa, sl.xb, sr.xa, sr.xb);
        emit_out(ea);
        emit_seg(sl);
        emit_seg(sr);
        emit_in(j);
        E += e2;
        go(kFV, c, d, tp);
        return true;
    }
    return false;
}

// The stacks a closed value on the codon trie continues with, up to kHelix at once: the cells of every pair
// of slots along the diagonal are read in two levels of loads, then each stack is one comparison of the
// twelve (closing edge, inner type) candidates in LDS.  A stack is the first two-loop of the order, so only a
// hairpin can come before it: the hairpin minima of all pairs found are compared side by side
// afterwards, and the first that matches ends the helix.  Spans below 9 (listed hairpin sizes) are left to
// the caller.  False if no stack was taken.
// A stack costs 0.3 us this way plus 3 us per helix, 8 us as a decision of its own.
__device__ bool Tracer::helix(int t, int p, int q, int ia, int ib, int64_t v) {
    const int g = q - p, kmax = min(kHelix, (g - 9) / 2 + 1);
    if (g < 9) return false;
    const SlotRec* R = I.recs();
    // records of layers p + k and q - 1 - k, k = 0..kmax, two lanes each
    const int rk = min(lane >> 1, kmax), rs = lane & 1;
    const SlotRec& rl = R[2 * (p + rk) + rs];
    const SlotRec& rr = R[2 * (q - 1 - rk) + rs];
    const int lstate = rl.state, rstate = rr.state;
    const int64_t lrow = rl.rowbase;
    if (lane < 2 * kHelix + 2) {
        W.ldst[lane] = *reinterpret_cast<const int*>(rl.dst);
        W.rdst[lane] = *reinterpret_cast<const int*>(rr.dst);
#pragma unroll
        for (int x = 0; x < 4; x++) {
            W.lu[lane][x] = rl.outU[x];
            W.ru[lane][x] = rr.outU[x];
        }
    }
    {
        const int k = lane >> 2, sl = (lane >> 1) & 1, sr = lane & 1;
        const int cs = __shfl(lstate, 2 * k + 2 + sl, 64), ds = __shfl(rstate, 2 * k + sr, 64);
        const int64_t row = ((int64_t)__shfl((int)(lrow >> 32), 2 * k + 2 + sl, 64) << 32) |
                            (uint32_t)__shfl((int)lrow, 2 * k + 2 + sl, 64);
        const bool ok = k < kmax && cs >= 0 && ds >= 0;
        if (ok) {
            const longlong2* vp = reinterpret_cast<const longlong2*>(I.V() + (row + ds) * 6);
            const longlong2 v0 = vp[0], v1 = vp[1], v2 = vp[2];
            int64_t* h = W.hv[lane];
            h[0] = v0.x, h[1] = v0.y, h[2] = v1.x, h[3] = v1.y, h[4] = v2.x, h[5] = v2.y;
        } else {
#pragma unroll
            for (int tp = 0; tp < 6; tp++) W.hv[lane][tp] = kINF;
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    // lane k keeps level k: the pair's slots, type, value, source slot and inner type of its stack
    int mia = 0, mib = 0, mt = 0, ms = 0, mtp = 0;
    int64_t mv = 0;
    const int ls = lane < 6 ? 0 : 1, ltp = lane < 6 ? lane : min(lane - 6, 5);
    int n = 0;
    for (; n < kmax; n++) {
        const int x = kTX[t], y = kTY[t], ia1 = bcast((int)(int8_t)(W.ldst[2 * n + ia] >> (8 * x)));
        if (ia1 < 0) break;
        const int64_t val = W.hv[4 * n + 2 * ia1 + ls][ltp];
        const bool ok = lane < 12 && (int)(int8_t)(W.rdst[2 * n + ls] >> (8 * y)) == ib && val < kINF &&
                        W.lu[2 * n + ia][x] + W.ru[2 * n + ls][y] + val + fxe(L.S.stack[t][kRev[ltp]]) == v;
        const unsigned long long hit = __ballot(ok);
        if (!hit) break;
        const int w = first_lane(hit), tp = w < 6 ? w : w - 6;
        if (lane == n) {
            mia = ia, mib = ib, mt = t, mv = v;
            ms = w >= 6, mtp = tp;
        }
        v = readlane64(val, w);
        ia = ia1;
        ib = w >= 6;
        t = tp;
    }
    if (n == 0) return false;
    // hairpins before a stack: lanes 4 k + x2
    {
        const int k = lane >> 2, x2 = lane & 3;
        const int ht = __shfl(mt, k, 64), hia = __shfl(mia, k, 64), hib = __shfl(mib, k, 64);
        const int64_t hvv = ((int64_t)__shfl((int)(mv >> 32), k, 64) << 32) | (uint32_t)__shfl((int)mv, k, 64);
        bool bad = false;
        if (k < n) {
            const int x = kTX[ht], y = kTY[ht], m = g - 2 * k - 2, ia1 = (int8_t)(W.ldst[2 * k + hia] >> (8 * x));
            const int64_t al = R[2 * (p + k + 1) + ia1].alpha[x2];
            const int64_t base = W.lu[2 * k + hia][x] + al + R[2 * (q - k)].pb2 - R[2 * (p + k)].pa2;
            const int init = I.hp_init()[m];
#pragma unroll
            for (int sr = 0; sr < 2; sr++) {
                if ((int)(int8_t)(W.rdst[2 * k + sr] >> (8 * y)) != hib) continue;
#pragma unroll
                for (int z = 0; z < 4; z++) {
                    const int64_t be = R[2 * (q - 1 - k) + sr].beta[z];
                    bad = bad || (al < kINF && be < kINF &&
                                  base + W.ru[2 * k + sr][y] + be + fxe(init + L.S.mmH[ht][x2][z]) == hvv);
                }
            }
        }
        const unsigned long long bm = __ballot(bad);
        if (bm) {
            n = first_lane(bm) >> 2;
            if (n == 0) return false;
            ia = bcast(__shfl(mia, n, 64));
            ib = bcast(__shfl(mib, n, 64));
            t = bcast(__shfl(mt, n, 64));
            v = readlane64(mv, n);
        }
    }
    if (lane < n) {
        const int x = kTX[mt], y = kTY[mt], i = p + lane, j = q - 1 - lane;
        I.tr_seq()[i] = x;
        I.tr_seq()[j] = y;
        I.tr_pair()[i] = j;
        I.tr_pair()[j] = i;
        Ul += W.lu[2 * lane + mia][x] + W.ru[2 * lane + ms][y];
        El += L.S.stack[mt][kRev[mtp]];
    }
    emitted += 2 * n;
    go(kFV, bcast(__shfl(lstate, 2 * n + ia, 64)), bcast(__shfl(rstate, 2 * n - 2 + ib, 64)), t);
    known = true;
    no_stack = n < kmax;
    kp = p + n;
    kq = q - n;
    kia = ia;
    kib = ib;
    kv = v;
    return true;
}

// A closed value on the codon trie, inner span >= 5.  A replay is one chain of decisions, so what bounds
// it is the dependent loads of each: the general functions look states, layers, edges and gaps up one
// after another (two-loop decision 17 us, hairpin test 3 us at 300 residues).  Here one level of loads
// brings the slot records of every layer a two-loop can reach, the next one the inner cells, and a helix
// carries layers, slots and the closed value from pair to pair.  The hairpin is enumerated only if its
// separable minimum equals v: the value is the minimum over all loops, so nothing else can match.
// 17 -> 8 us per decision; with the helices above, between the fill and the result: 50 residues 0.95 -> 0.35 ms,
// 300 residues 4.7 -> 1.6, 1,976 residues 20 -> 8.6 (there the cells come from beyond the caches).  The
// compiler spills 310 VGPRs of the traceback kernels (1,216 B of scratch per lane).
__device__ void Tracer::closed_trie(int a, int b, int t, int p, int q, int ia, int ib, int64_t v) {
    const int g = q - p, m = g - 2, x = kTX[t], y = kTY[t];
    const SlotRec* R = I.recs();
    if (lane == 0) {
        I.tr_pair()[p] = q - 1;
        I.tr_pair()[q - 1] = p;
    }
    // closing edges: a -x-> a1, and b1 -y-> b from either slot of layer q - 1 (in CSR order)
    const int ia1 = bcast(R[2 * p + ia].dst[x]);
    if (ia1 < 0 || v >= kINF) {
        fail = true;
        return;
    }
    const int64_t Ua = R[2 * p + ia].outU[x];
    const SlotRec &r1 = R[2 * (p + 1) + ia1], &rb0 = R[2 * (q - 1)], &rb1 = R[2 * (q - 1) + 1];
    const int a1 = bcast(r1.state);
    const bool e0 = rb0.dst[y] == ib, e1 = rb1.state >= 0 && rb1.dst[y] == ib;
    const int nj = (int)e0 + (int)e1, s0 = e0 ? 0 : 1;  // slots of the nj sources: s0 (then 1)
    if (nj == 0) {
        fail = true;
        return;
    }
    const int64_t U0 = R[2 * (q - 1) + s0].outU[y], U1 = rb1.outU[y];
    // the states at every distance: lane 2 l + slot, left c of layer p + 1 + l, right d of layer q - 1 - l
    {
        const int l = lane >> 1, sl = lane & 1, maxl = min(g - 7, kMaxLoop);
        const bool in = l <= maxl;
        const SlotRec& rc = R[2 * (p + 1 + (in ? l : 0)) + sl];
        const SlotRec& rd = R[2 * (q - 1 - (in ? l : 0)) + sl];
        const int cs = rc.state, ds = rd.state;
        int64_t gl = kINF, g0 = kINF, g1 = kINF;
        if (in && cs >= 0) {
            const int cl = p + 1 + l;
            if (l == 0) gl = sl == ia1 ? 0 : kINF;
            else if (cl / 3 != (p + 1) / 3) gl = r1.tail + rc.ip0 - R[2 * p].pa1;
            else if ((p + 1) % 3 == 0) gl = 0;
            else gl = r1.dst[0] == sl || r1.dst[1] == sl || r1.dst[2] == sl || r1.dst[3] == sl ? 0 : kINF;
        }
        if (in && ds >= 0) {
            const int dl = q - 1 - l;
            if (l == 0) {
                g0 = sl == 0 ? 0 : kINF;
                g1 = sl == 1 ? 0 : kINF;
            } else if (dl / 3 != (q - 1) / 3) {
                g0 = g1 = rd.tail + R[2 * q].pb1 - rd.in1;
            } else if (dl % 3 == 0) {
                g0 = g1 = 0;
            } else {
                g0 = rd.dst[0] == 0 || rd.dst[1] == 0 || rd.dst[2] == 0 || rd.dst[3] == 0 ? 0 : kINF;
                g1 = rd.dst[0] == 1 || rd.dst[1] == 1 || rd.dst[2] == 1 || rd.dst[3] == 1 ? 0 : kINF;
            }
        }
        W.gl[lane] = gl;
        W.row[lane] = rc.rowbase;
        W.st[lane] = ds;
        W.gr[0][lane] = g0;
        W.gr[1][lane] = g1;
    }
    // hairpin: sizes 3, 4 and 6 (listed loops) are enumerated, the others only if their minimum is v
    {
        bool hit = m == 3 || m == 4 || m == 6;
        if (!hit) {
            const int k = lane >> 4, x2 = (lane >> 2) & 3, z = lane & 3;
            const int64_t al = r1.alpha[x2], be = (k && e1 ? rb1 : R[2 * (q - 1) + s0]).beta[z];
            const int64_t w = al >= kINF || be >= kINF ? kINF
                              : Ua + (k && e1 ? U1 : U0) + al + be + R[2 * q].pb2 - R[2 * p].pa2 +
                                    fxe(I.hp_init()[m] + L.S.mmH[t][x2][z]);
            hit = __ballot(lane < 32 && w == v) != 0;
        }
        if (hit && hairpin(a, b, t, v, a * 4 + x, a1)) return;
    }
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    // two-loops: tuple = pair (l1, l2), source of the closing edge, slot of c, slot of d, in canonical
    // order; two tuples per lane and round
    const int sh = nj == 2 ? 3 : 2, total = kNumPairs << sh;
    constexpr int kPer = 2;
    for (int base = 0; base < total; base += 64 * kPer) {
        int code = INT_MAX, wtp = 0, wp = 0, wq = 0;
        int64_t wv = 0;
        int tl1[kPer], tl2[kPer], tjj[kPer];
        int64_t tg[kPer];
        longlong2 tv[kPer][3];
        bool ok[kPer];
#pragma unroll
        for (int k = 0; k < kPer; k++) {
            const int T = base + lane + 64 * k, pk = min(T >> sh, kNumPairs - 1);
            tl1[k] = L.pl1[pk];
            tl2[k] = L.pl2[pk];
            tjj[k] = nj == 2 ? (T >> 2) & 1 : s0;
            const int il = 2 * tl1[k] + ((T >> 1) & 1), ir = 2 * tl2[k] + (T & 1);
            const int64_t gl = W.gl[il], gr = W.gr[tjj[k]][ir];
            ok[k] = T < total && tl1[k] + tl2[k] <= g - 7 && gl < kINF && gr < kINF;
            tg[k] = gl + gr;
            const longlong2* vp = reinterpret_cast<const longlong2*>(I.V() + (ok[k] ? W.row[il] + W.st[ir] : r1.rowbase + rb0.state) * 6);
            tv[k][0] = vp[0];
            tv[k][1] = vp[1];
            tv[k][2] = vp[2];
        }
#pragma unroll
        for (int k = 0; k < kPer; k++) {
            if (!ok[k] || code != INT_MAX) continue;
            const int l1 = tl1[k], l2 = tl2[k];
            const int64_t vin[6] = {tv[k][0].x, tv[k][0].y, tv[k][1].x, tv[k][1].y, tv[k][2].x, tv[k][2].y};
            const int64_t Uj = nj == 2 && tjj[k] ? U1 : U0;
            const int64_t lb0 = Ua + tg[k] + Uj + fxe(two_loop_lb(L.S, t, l1, l2));
            int64_t vmin = kINF;
#pragma unroll
            for (int tp = 0; tp < 6; tp++) vmin = mn(vmin, vin[tp]);
            if (vmin >= kINF || lb0 + vmin > v) continue;
            const int T = base + lane + 64 * k;
#pragma unroll
            for (int tp = 0; tp < 6; tp++) {
                if (code != INT_MAX || vin[tp] >= kINF || lb0 + vin[tp] > v) continue;
                const int tr = kRev[tp];
                if (l1 == 0 || l2 == 0) {
                    // no boundary base enters the energy: the segment's minimum decides
                    const int32_t e2 = l1 + l2 == 0 ? L.S.stack[t][tr] : bulge_e(L.S, t, tr, l1 + l2);
                    if (Ua + tg[k] + vin[tp] + Uj + fxe(e2) == v) {
                        code = T;
                        wtp = tp;
                        wp = wq = -1;
                        wv = vin[tp];
                    }
                    continue;
                }
                const int c = R[2 * (p + 1 + l1) + ((T >> 1) & 1)].state, d = W.st[2 * l2 + (T & 1)];
                const int b1 = R[2 * (q - 1) + tjj[k]].state;
                Seg sl, sr;
                SegIter li(I, a1, c, l1);
                for (int pp = 0; code == INT_MAX && li.next(I, sl); pp++) {
                    SegIter ri(I, d, b1, l2);
                    for (int qq = 0; code == INT_MAX && ri.next(I, sr); qq++) {
                        const int32_t e2 = interior_e(L.S, nullptr, t, tr, l1, l2, sl.xa, sl.xb, sr.xa, sr.xb);
                        if (Ua + sl.cost + vin[tp] + sr.cost + Uj + fxe(e2) == v) {
                            code = T;
                            wtp = tp;
                            wp = pp;
                            wq = qq;
                            wv = vin[tp];
                        }
                    }
                }
            }
        }
        const int best = wmin_int(code);
        if (best == INT_MAX) {
            if (L.pl1[min((base + 64 * kPer) >> sh, kNumPairs - 1)] > g - 7) break;  // no further pair fits
            continue;
        }
        const int wl = first_lane(__ballot(code == best));
        const int tp = bcast(__shfl(wtp, wl, 64)), pp = bcast(__shfl(wp, wl, 64)), qq = bcast(__shfl(wq, wl, 64));
        const int64_t vn = readlane64(wv, wl);
        const int l1 = L.pl1[best >> sh], l2 = L.pl2[best >> sh], ci = (best >> 1) & 1, di = best & 1;
        const int jj = nj == 2 ? (best >> 2) & 1 : s0;
        const int c = R[2 * (p + 1 + l1) + ci].state, d = R[2 * (q - 1 - l2) + di].state, b1 = R[2 * (q - 1) + jj].state;
        emit_at(p, x, Ua);
        if (pp < 0) {  // stack or bulge: the first path at the segment's minimum, if there is a segment
            E += l1 + l2 == 0 ? L.S.stack[t][kRev[tp]] : bulge_e(L.S, t, kRev[tp], l1 + l2);
            Seg s;
            for (int side = 0; side < 2; side++) {
                const int l = side ? l2 : l1, u = side ? d : a1, w = side ? b1 : c;
                const int64_t want = side ? W.gr[jj][2 * l2 + di] : W.gl[2 * l1 + ci];
                if (l == 0) continue;
                int k = 0;
                bool got;
                while ((got = seg_at(I, u, w, l, k, s)) && s.cost != want) k++;
                if (!got) {
                    fail = true;
                    return;
                }
                emit_seg(s);
            }
        } else {
            Seg sl, sr;
            seg_at(I, a1, c, l1, pp, sl);
            seg_at(I, d, b1, l2, qq, sr);
            E += interior_e(L.S, nullptr, t, kRev[tp], l1, l2, sl.xa, sl.xb, sr.xa, sr.xb);
            emit_seg(sl);
            emit_seg(sr);
        }
        emit_at(q - 1, y, nj == 2 && jj ? U1 : U0);
        go(kFV, c, d, tp);
        known = true;
        kp = p + 1 + l1;
        kq = q - 1 - l2;
        kia = ci;
        kib = di;
        kv = vn;
        return;
    }
    // multiloop: closing in-edge of b labelled y, in CSR order
    const int32_t mlc = L.S.ml_closing + L.S.ml_intern + au_pen(L.S, t);
    for (int k = 0; k < nj; k++) {
        const int sl = k ? 1 : s0, b1 = R[2 * (q - 1) + sl].state;
        const int64_t Uj = k ? U1 : U0;
        if (g >= 12 && sadd(Ua + Uj + fxe(mlc), I.S2()[r1.rowbase + b1]) == v) {
            emit_at(p, x, Ua);
            emit_at(q - 1, y, Uj);
            E += mlc;
            go(kFS2, a1, b1, -1);
            return;
        }
    }
    fail = true;
}

__device__ void Tracer::closed(int a, int b, int t) {
    if (!I.gwin) {
        int p = kp, q = kq, ia = kia, ib = kib;
        int64_t v = kv;
        if (!known) {
            p = bcast(I.layer()[a]);
            q = bcast(I.layer()[b]);
            ia = a - bcast(I.off()[p]);
            ib = b - bcast(I.off()[q]);
            v = tV(I, t, a, b);
        }
        const bool stack = !no_stack;
        known = no_stack = false;
        if (q - p >= 7) {
            if (stack && v < kINF && helix(t, p, q, ia, ib, v)) return;
            closed_trie(a, b, t, p, q, ia, ib, v);
            return;
        }
    }
    const int64_t v = tV(I, t, a, b);
    const int i = I.layer()[a], j = I.layer()[b] - 1;
    if (lane == 0) {
        I.tr_pair()[i] = j;
        I.tr_pair()[j] = i;
    }
    const int ea = a * 4 + kTX[t], a1 = I.out_dst()[ea];
    if (a1 < 0 || v >= kINF) {
        fail = true;
        return;
    }
    if (hairpin(a, b, t, v, ea, a1)) return;
    if (twoloop(a, b, t, v, ea, a1)) return;
    // multiloop: closing in-edge of b labelled y, in CSR order
    if (I.layer()[b] - I.layer()[a] >= 12) {
        const int y = kTY[t];
        const int32_t mlc = L.S.ml_closing + L.S.ml_intern + au_pen(L.S, t);
        const int64_t Ua = I.out_U()[ea];
        const int ib0 = I.in_start()[b], ib1 = I.in_start()[b + 1];
        for (int j0 = ib0; j0 < ib1; j0 += 64) {
            const int jj = j0 + lane;
            bool ok = false;
            if (jj < ib1 && I.in_lab()[jj] == y) {
                const int b1 = I.in_src()[jj];
                ok = I.layer()[b1] - I.layer()[a1] >= 10 && sadd(Ua + I.in_U()[jj] + fxe(mlc), tS2(I, a1, b1)) == v;
            }
            const unsigned long long msk = __ballot(ok);
            if (msk) {
                const int jw = j0 + first_lane(msk);
                emit_out(ea);
                emit_in(jw);
                E += mlc;
                go(kFS2, a1, I.in_src()[jw], -1);
                return;
            }
        }
    }
    fail = true;
}

__device__ void Tracer::branch(int a, int b) {
    const int64_t v = tB(I, a, b);
    bool ok = false;
    if (lane < 6) ok = sadd(tV(I, lane, a, b), fxe(L.S.ml_intern + au_pen(L.S, lane))) == v;
    const unsigned long long m = __ballot(ok);
    if (!m) {
        fail = true;
        return;
    }
    const int t = first_lane(m);
    E += L.S.ml_intern + au_pen(L.S, t);
    go(kFV, a, b, t);
}

__device__ void Tracer::s1(int a, int b) {
    const int64_t v = tS1(I, a, b);
    // items: 0 direct branch, 1 S2, 2..5 left unpaired edge by label, 6.. right unpaired in-edge
    const int ib0 = I.in_start()[b], ib1 = I.in_start()[b + 1], total = 6 + (ib1 - ib0);
    const int la = I.layer()[a], lb = I.layer()[b];
    for (int base = 0; base < total; base += 64) {
        const int it = base + lane;
        bool ok = false;
        if (it == 0) ok = tB(I, a, b) == v;
        else if (it == 1) ok = tS2(I, a, b) == v;
        else if (it < 6) {
            const int e = a * 4 + it - 2, ap = I.out_dst()[e];
            ok = ap >= 0 && I.layer()[ap] < lb && sadd(I.out_U()[e] + I.mlbase_fx, tS1(I, ap, b)) == v;
        } else if (it < total) {
            const int j = ib0 + it - 6, bp = I.in_src()[j];
            ok = I.layer()[bp] > la && sadd(tS1(I, a, bp), I.in_U()[j] + I.mlbase_fx) == v;
        }
        const unsigned long long m = __ballot(ok);
        if (!m) continue;
        const int w = base + first_lane(m);
        if (w == 0) go(kFBR, a, b, -1);
        else if (w == 1) go(kFS2, a, b, -1);
        else if (w < 6) {
            const int e = a * 4 + w - 2;
            emit_out(e);
            E += L.S.ml_base;
            go(kFS1, I.out_dst()[e], b, -1);
        } else {
            const int j = ib0 + w - 6;
            emit_in(j);
            E += L.S.ml_base;
            go(kFS1, a, I.in_src()[j], -1);
        }
        return;
    }
    fail = true;
}

__device__ void Tracer::s2(int a, int b) {
    const int64_t v = tS2(I, a, b);
    const int ib0 = I.in_start()[b], ib1 = I.in_start()[b + 1];
    const int la = I.layer()[a];
    for (int j0 = ib0; j0 < ib1; j0 += 64) {
        const int j = j0 + lane;
        bool ok = false;
        if (j < ib1) {
            const int bp = I.in_src()[j];
            ok = I.layer()[bp] > la && sadd(tS2(I, a, bp), I.in_U()[j] + I.mlbase_fx) == v;
        }
        const unsigned long long m = __ballot(ok);
        if (m) {
            const int jw = j0 + first_lane(m);
            emit_in(jw);
            E += L.S.ml_base;
            go(kFS2, a, I.in_src()[jw], -1);
            return;
        }
    }
    // strict candidates c of C_b with layer(c) > layer(a): the smallest matching state index
    const int64_t cbase = I.coff()[b];
    const int cnt = I.ccnt()[b];
    int best = INT_MAX;
    for (int k = lane; k < cnt; k += 64) {
        const int raw = I.cc()[cbase + k];
        if (raw < 0 || raw >= best || I.layer()[raw] <= la) continue;  // non-strict entries have bit 31 set
        if (sadd(tS1(I, a, raw), tB(I, raw, b)) == v) best = raw;
    }
    best = wmin_int(best);
    if (best == INT_MAX) {
        fail = true;
        return;
    }
    push(kFS1, a, best, -1);
    go(kFBR, best, b, -1);
}

__device__ void trace_instance(const Inst& I, const EnergyTables* __restrict__ E, const int32_t* __restrict__ spec,
                               TraceLds& L) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    stage_tables(L.S, E);
    for (int k = tid; k < kNumPairs; k += blockDim.x) {  // (l1, l2) in canonical order
        int l1 = 0, r = k;
        while (r >= 31 - l1) {
            r -= 31 - l1;
            l1++;
        }
        L.pl1[k] = (unsigned char)l1;
        L.pl2[k] = (unsigned char)r;
    }
    for (int p = tid; p < I.n; p += blockDim.x) {
        I.tr_seq()[p] = -1;
        I.tr_pair()[p] = -1;
    }
    if (tid == 0) {
        L.lock = 0;
        L.sp = 0;
        L.busy = 1;  // wave 0 starts busy with X(s)
        L.failed = 0;
        L.emitted = 0;
        L.E = 0;
        L.U = 0;
    }
    __syncthreads();  // every wave's share of the energy tables is staged
    // A position is initialised by one wave and later written by whichever wave emits it: every
    // wave waits for its initialising stores before the barrier (which by itself waits only for
    // LDS operations), so that no -1 can land after an emitted value.
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
    __syncthreads();
    Tracer tr(I, L, L.w[wave], spec, lane);
    const int64_t xs = I.X()[0];
    if (wave == 0) {
        if (xs >= kINF) tr.fail_all(kTrUnreachable);
        tr.go(kFX, 0, -1, -1);
    }
    bool busy = wave == 0;
    for (;;) {
        if (tr.fail) {
            tr.fail_all(kTrNoMatch);  // a no-match decision (other reasons were recorded already)
            break;
        }
        TFrame f;
        if (tr.have_next) {
            f = tr.next;
            tr.have_next = false;
        } else {
            // this wave's chain has ended (or it never had one): a deferred frame, or the end
            const bool got = tr.take(f, busy);
            busy = got;
            if (!got) break;
        }
        switch (f.kind) {
            case kFX: tr.ext(f.a); break;
            case kFV: tr.closed(f.a, f.b, f.t); break;
            case kFS1: tr.s1(f.a, f.b); break;
            case kFS2: tr.s2(f.a, f.b); break;
            default: tr.branch(f.a, f.b); break;
        }
    }
    if (tr.El || tr.Ul || lane == 0) {
        atomicAdd(&L.E, (unsigned long long)(tr.El + (lane == 0 ? tr.E : 0)));
        atomicAdd(&L.U, (unsigned long long)(tr.Ul + (lane == 0 ? tr.U : 0)));
        if (lane == 0) atomicAdd(&L.emitted, tr.emitted);
    }
    __syncthreads();
    if (tid == 0) {
        I.tr_res()[0] = (long long)L.E;
        I.tr_res()[1] = (long long)L.U;
        I.tr_res()[2] = L.failed ? L.failed : L.emitted > I.n ? kTrDup : kTrOk;
        I.tr_res()[3] = xs;
    }
}

__global__ __launch_bounds__(64 * kTraceWaves) void k_trace(Inst I, const EnergyTables* __restrict__ E,
                                                            const int32_t* __restrict__ spec) {
    __shared__ TraceLds L;
    trace_instance(I, E, spec, L);
}

__global__ __launch_bounds__(64 * kTraceWaves) void k_trace_many(const Inst* __restrict__ insts,
                                                                 const EnergyTables* __restrict__ E,
                                                                 const int32_t* __restrict__ spec) {
    __shared__ TraceLds L;
    const Inst I = load_inst(insts + blockIdx.x);
    trace_instance(I, E, spec, L);
}

// strict candidates per right endpoint (retain-all control: non-strict entries carry bit 31)
__global__ void k_strict_count(Inst I) {
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= I.N) return;
    const int64_t base = I.coff()[b];
    int c = 0;
    for (int k = 0; k < I.ccnt()[b]; k++) c += I.cc()[base + k] >= 0;
    I.cstrict()[b] = c;
}

}  // namespace

hipError_t launch_trace(const Inst& I, const EnergyTables* E, const int32_t* spec, hipStream_t st) {
    hipLaunchKernelGGL(k_trace, dim3(1), dim3(64 * kTraceWaves), 0, st, I, E, spec);
    return hipGetLastError();
}

hipError_t launch_trace_many(const Inst* insts_dev, int n, const EnergyTables* E, const int32_t* spec,
                             hipStream_t st) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_trace_many, dim3(n), dim3(64 * kTraceWaves), 0, st, insts_dev, E, spec);
    return hipGetLastError();
}

hipError_t launch_strict_count(const Inst& I, hipStream_t st) {
    hipLaunchKernelGGL(k_strict_count, dim3((I.N + 255) / 256), dim3(256), 0, st, I);
    return hipGetLastError();
}

}  // namespace sd
