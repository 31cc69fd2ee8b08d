// Device helpers shared by the span-step kernels and the traceback kernel: pair types, the loop
// tables staged in LDS, fixed-point and INF arithmetic, wavefront reductions over DPP moves, cell
// addressing, and the loop energies of the
// nearest-neighbour model (Sec. 3).
#pragma once
#include <hip/hip_runtime.h>

#include <stddef.h>
#include <stdint.h>

#include "sd_internal.h"

namespace sd {

static __constant__ int kTX[6] = {0, 1, 2, 2, 3, 3};  // 5' base of AU CG GC GU UA UG
static __constant__ int kTY[6] = {3, 2, 1, 3, 0, 2};  // 3' base
static __constant__ int kRev[6] = {4, 2, 1, 5, 0, 3}; // type of the reversed pair

// Copies the loop tables to LDS, straight from memory (no registers in between): one KiB per wave and
// instruction.  stage_wait ends the copy for the whole workgroup; loads that do not need the tables
// can be issued in between.
__device__ __forceinline__ void stage_begin(SmallE& S, const EnergyTables* __restrict__ E) {
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, nw = blockDim.x >> 6;
    const char* src = reinterpret_cast<const char*>(&E->small);
    char* dst = reinterpret_cast<char*>(&S);
    for (int c = wave; c < (int)(sizeof(SmallE) / 1024); c += nw)
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src + c * 1024 + lane * 16),
                                         (__attribute__((address_space(3))) void*)(dst + c * 1024), 16, 0, 0);
}
__device__ __forceinline__ void stage_wait() {
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): this wave's share has landed
    __syncthreads();
}
__device__ __forceinline__ void stage_tables(SmallE& S, const EnergyTables* __restrict__ E) {
    stage_begin(S, E);
    stage_wait();
}

// The region bases of an instance as global pointers the compiler knows nothing else about.  A
// descriptor read from memory holds generic pointers, whose accesses would be flat instructions
// (which also wait on the LDS counter); and array addresses derived from a laundered base are not
// hoisted out of the loop that launders it, where they would crowd the scalar registers.
__device__ __forceinline__ char* global_base(char* p) {
    uint64_t x = (uint64_t)p;
    asm volatile("" : "+s"(x));
    return (char*)(__attribute__((address_space(1))) char*)x;
}
__device__ __forceinline__ Inst rebased(Inst I) {
    I.ra = global_base(I.ra);
    I.rb = global_base(I.rb);
    return I;
}

// A descriptor from memory that no kernel writes: scalar loads.
__device__ __forceinline__ Inst load_inst(const Inst* p) {
    const __attribute__((address_space(4))) uint64_t* w = (const __attribute__((address_space(4))) uint64_t*)(uintptr_t)p;
    Inst I;
    uint64_t* d = reinterpret_cast<uint64_t*>(&I);
#pragma unroll
    for (int k = 0; k < (int)(sizeof(Inst) / 8); k++) d[k] = w[k];
    return rebased(I);
}

__device__ __forceinline__ int32_t au_pen(const SmallE& S, int t) {
    return (t == 1 || t == 2) ? 0 : S.terminal_au;
}
__device__ __forceinline__ int64_t mn(int64_t a, int64_t b) { return a < b ? a : b; }
__device__ __forceinline__ int64_t fx(int32_t e, int s) { return (int64_t)e * ((int64_t)1 << s); }
__device__ __forceinline__ int64_t norm_inf(int64_t v) { return v >= kHalfINF ? kINF : v; }

__device__ __forceinline__ int64_t shfl_xor64(int64_t v, int m) {
    int lo = __shfl_xor((int)(uint32_t)(uint64_t)v, m, 64);
    int hi = __shfl_xor((int)(uint32_t)((uint64_t)v >> 32), m, 64);
    return (int64_t)(((uint64_t)(uint32_t)hi << 32) | (uint64_t)(uint32_t)lo);
}
// DPP moves of a 64-bit value within rows of 16 lanes (no LDS traffic).  Callers run with every
// lane of the wave active.
template <int CTRL>
__device__ __forceinline__ int64_t dpp64(int64_t v) {
    const int lo = (int)(uint32_t)(uint64_t)v, hi = (int)(uint32_t)((uint64_t)v >> 32);
    const int l2 = __builtin_amdgcn_update_dpp(lo, lo, CTRL, 0xF, 0xF, false);
    const int h2 = __builtin_amdgcn_update_dpp(hi, hi, CTRL, 0xF, 0xF, false);
    return (int64_t)(((uint64_t)(uint32_t)h2 << 32) | (uint64_t)(uint32_t)l2);
}
constexpr int kDppXor1 = 0xB1, kDppXor2 = 0x4E;               // quad_perm [1,0,3,2], [2,3,0,1]
constexpr int kDppHalfMirror = 0x141, kDppMirror = 0x140;     // lane i <-> 7-i, 15-i of its row
constexpr int kDppRor4 = 0x124, kDppRor8 = 0x128;             // rotate the row by 4, 8 lanes
__device__ __forceinline__ int64_t readlane64(int64_t v, int l) {
    const int lo = __builtin_amdgcn_readlane((int)(uint32_t)(uint64_t)v, l);
    const int hi = __builtin_amdgcn_readlane((int)(uint32_t)((uint64_t)v >> 32), l);
    return (int64_t)(((uint64_t)(uint32_t)hi << 32) | (uint64_t)(uint32_t)lo);
}
// Minimum of two int64 in [0, 2^63 - 2^52): positive patterns of finite doubles order as the integers do,
// so one instruction replaces a compare and two selects.  kBias brings every value of the tables and
// their sums into that range: finite ones, sums of unfinished loops included, lie strictly between -2^60 and
// 2^60 (see energy_bound; patterns below 2^52 are denormal doubles, which the FP64 mode of every kernel
// keeps), infinite ones reach 2^62 and a little.
constexpr int64_t kBias = (int64_t)1 << 60;
__device__ __forceinline__ int64_t min_positive(int64_t a, int64_t b) {
    int64_t r;
    asm("v_min_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
template <int CTRL>
__device__ __forceinline__ int64_t min_dpp(int64_t v) { return min_positive(v, dpp64<CTRL>(v)); }
// the minimum with the value 16 or 32 lanes away (lane xor 16 / 32): one swap per half of the value
__device__ __forceinline__ int64_t min_xor16(int64_t v) {
    const auto l = __builtin_amdgcn_permlane16_swap((unsigned)v, (unsigned)v, false, false);
    const auto h = __builtin_amdgcn_permlane16_swap((unsigned)((uint64_t)v >> 32), (unsigned)((uint64_t)v >> 32), false, false);
    return min_positive((int64_t)((uint64_t)h[0] << 32 | l[0]), (int64_t)((uint64_t)h[1] << 32 | l[1]));
}
__device__ __forceinline__ int64_t min_xor32(int64_t v) {
    const auto l = __builtin_amdgcn_permlane32_swap((unsigned)v, (unsigned)v, false, false);
    const auto h = __builtin_amdgcn_permlane32_swap((unsigned)((uint64_t)v >> 32), (unsigned)((uint64_t)v >> 32), false, false);
    return min_positive((int64_t)((uint64_t)h[0] << 32 | l[0]), (int64_t)((uint64_t)h[1] << 32 | l[1]));
}
// minimum over each row of 16 lanes (every lane of the wave active) of biased values
__device__ __forceinline__ int64_t row_min_biased(int64_t v) {
    return min_dpp<kDppMirror>(min_dpp<kDppHalfMirror>(min_dpp<kDppXor2>(min_dpp<kDppXor1>(v))));
}
__device__ __forceinline__ int64_t row_min(int64_t v) { return row_min_biased(v + kBias) - kBias; }
// minimum over the whole wave (every lane active) of biased values, in every lane's scalar copy
__device__ __forceinline__ int64_t wave_min_biased(int64_t v) {
    v = min_xor32(min_xor16(row_min_biased(v)));
    const int lo = __builtin_amdgcn_readfirstlane((int)v), hi = __builtin_amdgcn_readfirstlane((int)((uint64_t)v >> 32));
    return (int64_t)((uint64_t)(uint32_t)hi << 32 | (uint32_t)lo);
}
// minimum over the whole wave (every lane active): about half the instructions of 64-bit compares and selects
__device__ __forceinline__ int64_t wave_min(int64_t v) { return wave_min_biased(v + kBias) - kBias; }

__device__ __forceinline__ int32_t bulge_e(const SmallE& S, int t, int tr, int l) {
    return l == 1 ? S.bulge[1] + S.stack[t][tr] : S.bulge[l] + au_pen(S, t) + au_pen(S, tr);
}

__device__ __forceinline__ int32_t interior_base(const SmallE& S, int l1, int l2) {
    int d = l1 > l2 ? l1 - l2 : l2 - l1;
    int32_t asym = S.ninio * d;
    return S.interior[l1 + l2] + (asym < S.ninio_max ? asym : S.ninio_max);
}

// interior loop with l1, l2 >= 1
__device__ inline int32_t interior_e(const SmallE& S, const EnergyTables* __restrict__ E, int t, int tr,
                              int l1, int l2, int xi1, int xk1, int xl1, int xj1) {
    if (l1 == 1 && l2 == 1) return S.int11[t][tr][xi1][xj1];
    if (l1 == 1 && l2 == 2) return S.int21[t][tr][xi1][xl1][xj1];
    if (l1 == 2 && l2 == 1) return S.int21[tr][t][xl1][xi1][xk1];
    if (l1 == 2 && l2 == 2) return S.int22[t][tr][xi1][xk1][xl1][xj1];
    int32_t e = interior_base(S, l1, l2);
    if (l1 == 1 || l2 == 1) return e + S.mm1n[t][xi1][xj1] + S.mm1n[tr][xl1][xk1];
    if (l1 + l2 == 5 && (l1 == 2 || l1 == 3)) return e + S.mm23[t][xi1][xj1] + S.mm23[tr][xl1][xk1];
    return e + S.mmI[t][xi1][xj1] + S.mmI[tr][xl1][xk1];
}

__device__ __forceinline__ int pair_class(int l1, int l2) {  // 1: 2x3 mismatch table, 0: generic
    return (l1 + l2 == 5 && (l1 == 2 || l1 == 3)) ? 1 : 0;
}
// mismatch class of an interior loop: 0 generic, 1 2x3, 2 1xn
__device__ __forceinline__ int mm_class(int l1, int l2) {
    return (l1 == 1 || l2 == 1) ? 2 : pair_class(l1, l2);
}
__device__ __forceinline__ int32_t mmx(const SmallE& S, int X, int t, int i, int j) {
    return X == 0 ? S.mmI[t][i][j] : X == 1 ? S.mm23[t][i][j] : S.mm1n[t][i][j];
}

}  // namespace sd
