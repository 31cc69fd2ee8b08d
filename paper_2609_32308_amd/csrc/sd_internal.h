// Internal layout shared by the host side of the library and its gfx950 kernels.
//
// Device data of one design instance (all int64 values are fixed point: energy * 2^s plus
// rounded codon costs; kINF = 2^62 marks infeasible):
//   automaton   layer[N], off[n+2] (first state of each layer), out_dst/out_U[N*4] (edge by
//               label, DFA so at most one per label), in-edge CSR sorted by (source, label).
//   gap         closed form for the codon trie: G(a,b) = tail(a) + P[k(b)] - P[k(a)+1] across
//               codons, 0 / unreachable inside one codon (prefix test on pfx).
//   cells       row layout over state pairs: cell(a,b) = rowoff[a] + b - off[layer(a)+1], i.e.
//               row a holds every b of a later layer, contiguous in state order.  Per cell:
//               V[6] (typed closed values), B (branch), S1, S2 (multiloop fragments).
//   candidates  per right endpoint b a packed segment [coff[b], coff[b]+ccap[b]) of
//               (cc = start state, cB = B(c,b)); ccnt[b] entries committed so far, appended in
//               span order (each span's entries in start-state order).
#pragma once
#include <stdint.h>

namespace sd {

constexpr int64_t kINF = int64_t(1) << 62;
constexpr int64_t kHalfINF = int64_t(1) << 61;  // anything above is infeasible
constexpr int kMaxLoop = 30;                    // bulge / interior unpaired cap (Sec. 3)
constexpr int kNumPairs = 496;                  // (l1,l2) with l1 + l2 <= 30

// Lower bounds of two-loop energies per closing type over boundary bases and inner types (traceback).
struct LoopMin {
    int32_t stack[6], int11[6], int12[6], int21[6], int22[6];
    int32_t mm_out[3][6];  // min over (x_{i+1}, x_{j-1}) of mm_X[t], X = 0 generic, 1 2x3, 2 1xn
    int32_t mm_in[3];      // min over inner types and boundary bases of mm_X
    int32_t au_min;
};

// Loop tables as the kernels stage them in LDS, a multiple of 1 KiB (the 1x2 and 2x2 full-loop tables as
// 16-bit copies; the parser requires entries in [-32768, 32767]).
struct SmallE {
    alignas(16) int16_t int21[6][6][4][4][4];    // 1x2 loops
    alignas(16) int16_t int22[6][6][4][4][4][4]; // 2x2 loops
    int32_t stack[6][6];
    // boundary tables by class, addressed as one array [class][type][16]: hairpin, generic interior,
    // 1xn, 2x3, and the terminal AU/GU penalty of the type (the same for all 16 label pairs)
    int32_t mmH[6][4][4], mmI[6][4][4], mm1n[6][4][4], mm23[6][4][4], mmA[6][4][4];
    int32_t int11[6][6][4][4];
    int32_t hairpin[31], bulge[31], interior[31];
    int32_t ml_closing, ml_intern, ml_base, terminal_au, ninio, ninio_max;
    LoopMin lmin;
    int32_t pad[165];
};
static_assert(sizeof(SmallE) % 1024 == 0, "staged in pieces of 1 KiB");

// Energy tables in 0.01 kcal/mol; two-loop tables index the inner pair from inside the loop.
struct EnergyTables {
    int32_t stack[6][6];
    int32_t mmH[6][4][4], mmI[6][4][4], mm1n[6][4][4], mm23[6][4][4];
    int32_t int11[6][6][4][4];
    int32_t int21[6][6][4][4][4];
    int32_t int22[6][6][4][4][4][4];
    int32_t hairpin[31], bulge[31], interior[31];
    int32_t ml_closing, ml_intern, ml_base, terminal_au, ninio, ninio_max;
    int32_t pad[2];
    alignas(16) SmallE small;  // what the kernels stage
};

// Special hairpin lookup: key = base-4 number of the loop sequence (closing pair included),
// value = listed total energy or kNoSpecial.
constexpr int32_t kNoSpecial = 0x7fffffff;
constexpr int kSpecOff5 = 0, kSpecOff6 = 1024, kSpecOff8 = 1024 + 4096, kSpecSize = 1024 + 4096 + 65536;

// A pending decision of the traceback: kind (external column, closed value, S1, S2, branch),
// the cell (a, b) and, for closed values, the pair type.
struct TFrame {
    int kind, a, b, t;
};

// Instance descriptor.  All arrays of one design live in two device regions whose layout is a
// function of a few sizes, so the descriptor holds two base pointers plus sizes and every array
// address is recomputed arithmetically where it is used (cheap scalar ALU, few live registers,
// also when the descriptor is read from memory by the batched kernel).
//
// Region A (inputs and small mutable state) is cut into units of U bytes, U >= 8 * (N + 2),
// >= 8 * (n + 2) and >= 8 * (A + 1), a multiple of 256; unit k starts at ra + k * U:
//   0 layer[N]  1 off[n+2]  2 in_start[N+1]  3 tail[N]  4 pfx[N]  5 P[A+1]  6 hp_init[n+1]
//   7 rowoff[N]  8 coff[N]  9 ccap[N]  10 inmask[N]  11 X[N]  12-13 out_dst[4N]  14-17 out_U[4N]
//   18 stats[4], trace results [8..11]
//   19 visits[n+1]  20 feasible[n+1]  21 ccnt[N]  22 tr_seq[n]  23 tr_pair[n]
//   24-25 tr_stack[n+2] (16-byte frames)  26 cstrict[N]
//   27.. in_src[nE], in_lab[nE], in_U[nE] (each start 8-byte aligned), then for the codon trie
//        recs[nrec] (64-byte aligned, SlotRec)
// Region B (DP tables) is cut into ring units of R = 512 * N bytes (N states x 64 spans x 8 B):
//   0-1 LM  2-13 IDL  14-25 JDL  26 BI  27 BJ  28-43 RS  44-59 LS  60-61 MINI, then from 62 R:
//   V[cells][6], Bt[cells], S1[cells], S2[cells], cc[slots], cB[slots], and for generic lattices
//   G[cells] (minimum path cost a -> b), LG[row][wl] and IN[class 3][row][win] (see GenRow).
// Meaning of the arrays:
//   layer/off: layer of a state, first state of a layer; out_dst/out_U: out-edge by label
//   (-1 / cost); in_start/in_src/in_lab/in_U: in-edges (CSR, sorted by source and label);
//   inmask: bit y set if the state has an in-edge labelled y, bit 4 + x if it has an out-edge
//   labelled x; tail: cheapest completion of the
//   current codon from a state; pfx: 2-base prefix code of a
//   phase-2 state (4x+y), base x of phase 1; P: prefix sums of per-codon minimum cost;
//   hp_init: hairpin initiation per size (extrapolated above 30); rowoff: cell row offsets,
//   cell(a,b) = rowoff[a] + b - off[layer(a)+1]; V/Bt/S1/S2: typed closed values, branch value,
//   multiloop prefixes; coff/ccap/ccnt/cc/cB: candidate segment per right endpoint (offset,
//   capacity, committed count, start states with the non-strict flag in bit 31, B values);
//   X: external column; stats: [2] earliest overflow span, [8..11] traceback results (energy,
//   path cost, status, X(s)); tr_seq / tr_pair: the traceback's base label per position and
//   pairing partner per position (-1 unpaired); tr_stack: its pending decisions; cstrict:
//   strict candidates per right endpoint (retain-all control only); visits / feasible:
//   candidate visits and cells with finite B, summed per left layer (one adder per layer pair
//   and step, so the counters see no contention).
//   LM[layer][class 2][span]: layer-pair minima of the both-separable interior form.  The rings of a
//   separable side (LM, IDL, JDL, BI, BJ) already hold the whole-codon prefix term of their own
//   layers; a consumer adds the one of its closing pair.
//   MINI[layer p][span][class 2]: both-separable interior minimum of layer pair (p, p + span),
//   prepared one step ahead.
//   IDL/JDL[state][class 3][label 4][span]: inner minima per left / right inner state.
//   BI[c][span] = min over d, t' of V_t'(c,d) + tail(d) + AU(t');  BJ[d][span] likewise without
//   the tail.  RS[c][span][l-1][label], LS[d][span][l-1][label]: one-sided loops minimised over
//   the separable side's length (explicit side of l <= 3 bases).
// Everything the span step needs of one state of the codon trie in one record, two records per layer
// (a layer of the trie holds one or two states), so that it is found from the layer alone with one
// level of loads.
constexpr int kTrieWidth = 2, kFwdPaths = 12, kBwdPaths = 18;
struct alignas(64) SlotRec {
    int32_t state;            // state index (-1: the layer has no second state)
    uint8_t inmask, outmask;  // labels of the in- and out-edges
    uint8_t nf[3], nb[3];     // forward / backward paths of 1, up to 2, up to 3 edges
    int8_t dst[4];            // out-edge by label: slot in the next layer (-1: none)
    int64_t rowbase;          // cell(state, b) = rowbase + b
    int64_t tail, coff;       // cheapest completion of the codon; candidate segment
    int32_t ccap, pad;
    // whole-codon prefix terms of the layer l as the closing layer of a pair (P at (l + 1) / 3 + 1,
    // (l + 2) / 3 + 1, (l - 1) / 3, (l - 2) / 3) and as an inner layer (P at l / 3 + 1 and
    // (l + 1) / 3 + 1 to take off, l / 3 and (l - 1) / 3 to add)
    int64_t pa1, pa2, pb1, pb2, in1, in2, ip0, ip1;
    int64_t outU[4];          // out-edge costs by label
    int64_t alpha[4];         // U of the out-edge labelled x + tail of its target
    int64_t beta[4];          // min U over the in-edges labelled x
    // label paths of 1..3 edges out of / into the state, by length (3 from / into codon boundaries
    // only): meta = other end << 4 | first label << 2 | last label, cost, row base of the end state
    int64_t fcost[kFwdPaths], fcrow[kFwdPaths], bcost[kBwdPaths];
    int32_t fmeta[kFwdPaths], bmeta[kBwdPaths];
};

// Generic lattices.  Out-edges in order of state and label, walks of two edges in order of their edges,
// and rows: one per state and label of its in-edges, in order of state and label.
struct GenEdge {
    int32_t src, dst, lab, layer;  // of a walk: lab = first label | last label << 2; layer of src
    int64_t U;
    int32_t row, pad;              // row of (dst, lab)
};
// LG(e, row) lies at lgbase + e, e an out-edge of the 30 layers before the row's; IN_X(row, f) in column
// f mod win, a ring over the out-edges of 33 layers.
struct GenRow {
    int32_t state, lab, layer, cnt;  // cnt edges enter the state with the label:
    int32_t first, pad;              // growedge()[first..]
    int64_t lgbase;
};

struct Inst {
    char *ra, *rb;         // region bases
    int64_t U;             // region-A unit in bytes
    int64_t nE, nrec;      // in-edges, slot records (0 for generic lattices)
    int64_t cells, slots;  // DP cells, candidate slots
    int64_t mlbase_fx;     // ML_base * 2^s
    int64_t nwalk, lgsize;  // generic lattices: walks of two edges, words of LG
    int n, N, A, shift;
    int retain_all;
    int g0;  // persistent launches: first span this launch processes for the instance
    int gwin;  // 1 for generic lattices (0 for the codon trie)
    int nil, win;  // generic lattices: rows, ring width of IN
    int wmax;  // widest layer

    __host__ __device__ static int64_t al8(int64_t x) { return (x + 7) & ~(int64_t)7; }
    __host__ __device__ char* ua(int k) const { return ra + (int64_t)k * U; }
    __host__ __device__ int64_t R() const { return (int64_t)512 * N; }
    __host__ __device__ char* ub(int k) const { return rb + (int64_t)k * R(); }

    __host__ __device__ const int* layer() const { return (const int*)ua(0); }
    __host__ __device__ const int* off() const { return (const int*)ua(1); }
    __host__ __device__ const int* in_start() const { return (const int*)ua(2); }
    __host__ __device__ const int64_t* tail() const { return (const int64_t*)ua(3); }
    // generic lattices (which have no tail): cell(a, b) = rowbase[a] + b
    __host__ __device__ const int64_t* rowbase() const { return tail(); }
    __host__ __device__ const int* pfx() const { return (const int*)ua(4); }
    __host__ __device__ const int64_t* P() const { return (const int64_t*)ua(5); }
    __host__ __device__ const int* hp_init() const { return (const int*)ua(6); }
    __host__ __device__ const int64_t* rowoff() const { return (const int64_t*)ua(7); }
    __host__ __device__ const int64_t* coff() const { return (const int64_t*)ua(8); }
    __host__ __device__ const int* ccap() const { return (const int*)ua(9); }
    __host__ __device__ int* ccnt() const { return (int*)ua(21); }
    __host__ __device__ int64_t* X() const { return (int64_t*)ua(11); }
    __host__ __device__ const int* out_dst() const { return (const int*)ua(12); }
    __host__ __device__ const int64_t* out_U() const { return (const int64_t*)ua(14); }
    __host__ __device__ unsigned long long* stats() const { return (unsigned long long*)ua(18); }
    __host__ __device__ unsigned long long* visits() const { return (unsigned long long*)ua(19); }
    __host__ __device__ unsigned long long* feasible() const { return (unsigned long long*)ua(20); }
    __host__ __device__ const int* inmask() const { return (const int*)ua(10); }
    __host__ __device__ int* tr_seq() const { return (int*)ua(22); }
    __host__ __device__ int* tr_pair() const { return (int*)ua(23); }
    __host__ __device__ TFrame* tr_stack() const { return (TFrame*)ua(24); }
    // everything a finished design returns lies in one range: units 18..23
    __host__ __device__ const char* results() const { return ua(18); }
    __host__ __device__ size_t stats_bytes() const { return (size_t)(2 * U + 8 * ((int64_t)n + 1)); }
    __host__ __device__ size_t results_bytes() const { return (size_t)(5 * U + 4 * (int64_t)n); }
    __host__ __device__ int* cstrict() const { return (int*)ua(26); }
    __host__ __device__ long long* tr_res() const { return (long long*)ua(18) + 8; }
    __host__ __device__ const int* in_src() const { return (const int*)ua(27); }
    __host__ __device__ const int* in_lab() const { return (const int*)(ua(27) + al8(4 * nE)); }
    __host__ __device__ const int64_t* in_U() const { return (const int64_t*)(ua(27) + 2 * al8(4 * nE)); }
    __host__ __device__ const SlotRec* recs() const {
        return (const SlotRec*)(ra + ((ua(27) + 2 * al8(4 * nE) + 8 * nE - ra + 63) & ~(int64_t)63));
    }
    // generic lattices: edges, rows, walks, the edges of each row, and the first edge, row and walk of
    // every layer
    __host__ __device__ const GenEdge* gedges() const { return (const GenEdge*)(recs() + nrec); }
    __host__ __device__ const GenEdge* gwalks() const { return gedges() + (gwin ? nE : 0); }
    __host__ __device__ const GenRow* grows() const { return (const GenRow*)(gwalks() + nwalk); }
    __host__ __device__ const int* growedge() const { return (const int*)(grows() + nil); }
    __host__ __device__ const int* geoff() const { return growedge() + (gwin ? nE : 0); }
    __host__ __device__ const int* groff() const { return geoff() + n + 2; }
    __host__ __device__ const int* gwoff() const { return groff() + n + 2; }
    __host__ __device__ int64_t a_bytes() const {
        return (int64_t)((char*)geoff() - ra) + (gwin ? 12 * ((int64_t)n + 2) : 0);
    }

    __host__ __device__ int64_t* LM() const { return (int64_t*)ub(0); }
    __host__ __device__ int64_t* IDL() const { return (int64_t*)ub(2); }
    __host__ __device__ int64_t* JDL() const { return (int64_t*)ub(14); }
    __host__ __device__ int64_t* BI() const { return (int64_t*)ub(26); }
    __host__ __device__ int64_t* BJ() const { return (int64_t*)ub(27); }
    __host__ __device__ int64_t* RS() const { return (int64_t*)ub(28); }
    __host__ __device__ int64_t* LS() const { return (int64_t*)ub(44); }
    __host__ __device__ int64_t* MINI() const { return (int64_t*)ub(60); }
    __host__ __device__ int64_t* V() const { return (int64_t*)ub(62); }
    __host__ __device__ int64_t* Bt() const { return (int64_t*)(ub(62) + 48 * cells); }
    __host__ __device__ int64_t* S1() const { return (int64_t*)(ub(62) + 56 * cells); }
    __host__ __device__ int64_t* S2() const { return (int64_t*)(ub(62) + 64 * cells); }
    __host__ __device__ int* cc() const { return (int*)(ub(62) + 72 * cells); }
    __host__ __device__ int64_t* cB() const { return (int64_t*)(ub(62) + 72 * cells + al8(4 * slots)); }
    // generic lattices only: gap table G[cells], labelled gaps LG and inner loop parts IN
    __host__ __device__ int64_t* Gt() const { return (int64_t*)(ub(62) + 72 * cells + al8(4 * slots) + 8 * slots); }
    __host__ __device__ int64_t* LG() const { return Gt() + cells; }
    __host__ __device__ int64_t* IN() const { return LG() + lgsize; }
    __host__ __device__ int64_t b_bytes() const {
        return 62 * R() + 72 * cells + al8(4 * slots) + 8 * slots +
               (gwin ? 8 * (cells + lgsize + 3 * (int64_t)nil * win) : 0);
    }
};

constexpr int kLMRing = 64;
constexpr int kMaxWidth = 4;  // states per layer of an abstract DAG (the multiloop test hook)
constexpr int kGenMaxWidth = 16;  // states per layer of a generic (motif-constrained) lattice
constexpr int kGenLoopWin = 30;   // layer distances covered by the labelled gap table
static_assert(sizeof(Inst) % 8 == 0, "instance descriptors are copied as 8-byte words");

// Batched persistent launch: barrier state shared by all workgroups.  Every contended word sits on its
// own 128-byte line.  Barrier words are per XCD (the one a workgroup runs on); the work bands are per
// group, block index mod 8.
struct alignas(128) CtlWord {
    unsigned int v;
    unsigned int pad[31];
};
constexpr int kMaxXcd = 16;
struct BatchCtl {
    CtlWord count[kMaxXcd];    // workgroups of each XCD
    CtlWord joined;            // workgroups counted
    CtlWord arrive[kMaxXcd];   // arrivals of each XCD at the current barrier
    CtlWord top;               // XCDs complete at the current barrier
    CtlWord gen;               // barrier generation
    CtlWord release[kMaxXcd];  // generation each XCD's workgroups are released to
    CtlWord err;        // set when a barrier wait exceeds its spin limit (every group then exits)
    CtlWord steps_done; // spans completed (diagnostics)
};
constexpr int kMaxBatch = 1024;  // instances per persistent launch

}  // namespace sd
