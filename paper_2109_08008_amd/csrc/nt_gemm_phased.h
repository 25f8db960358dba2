// The projections' large tiles: the same product as nt_gemm.hip, bit for bit, on workgroups
// whose k-loop runs in phases.
//
// What bounds nt_gemm.hip's tiles at a few hundred workgroups and more is the chain inside a
// k-step -- wait for the tile, barrier, issue the next tile's loads, read fragments, wait,
// multiply -- with loads that have one k-step at most to land.  Here a wave forms
// 2*FMH x 2*FNH MFMA blocks (16x16), and a k-step (128 bytes of K) is four phases of FMH x FNH
// blocks each:
//   (A0,B0) (A1,B0) (A1,B1) (A0,B1)
// so that every phase needs one new half of one operand; the other is already in registers.
// A phase is one asm block: its MFMAs, and between them the fragment reads of the next phase
// and the loads that refill LDS, then the wait for the reads (and for the oldest refill) and
// the barrier.  Reads in flight never outlive their block, and the matrix core works through
// them.  LDS holds two k-steps as eight half-operand regions.  A region is read in exactly
// one phase, the one before its half is multiplied, and refilled in the next: the direct
// global->LDS loads have six phases (1.5 k-steps) to land.
//
// No k-step is peeled: past the last one the refills read one line and land in regions that
// nobody reads.  Blocks are formed transposed (the weights as the MFMA's first operand), so a
// lane holds four consecutive columns of a row: bias, column sums and scales are vector
// loads, two neighbouring blocks trade halves between lane groups (v_permlane16_swap) to make
// 16-byte residual loads and stores of 16-bit results, and whole tiles stage nothing through
// LDS.
//
// The sum over k of an element runs through the same MFMAs in the same order as in
// nt_gemm.hip, so the choice of kernel never changes a result.
//
// Measured on MI355X (us, nt_gemm.hip's tile / this): 16384x1024x4096 with residual 154 / 113
// (1.22 PFLOP/s; a large library product reaches 1.29 on the card), 16384x4096x1024 194 / 127,
// 8192x1536x512 25.8 / 19.2, 2160x4096x1024 with a folded LayerNorm 43 / 33, 1114x1024x4096
// 38 / 24.5, the output projection's records at 1300x32000x512 78 / 52.  At K = 512 a 256x256
// tile spends 0.8 us on arguments and addresses, 0.9 filling LDS, 9-11 in the k-loop and 4-6
// on bias, residual and stores; two workgroups a CU (128x128: 64 KB of LDS, 160 VGPRs) or
// three (64x128: 48 KB) cover each other's ends, which is why the largest tile pays only where
// its k-loop is the whole of the launch.
#pragma once
#include <limits.h>

#include "nt_gemm_common.h"

namespace nt {
namespace {

// Fragments of an LDS region (both halves of the k-step), complete on return: the reads and
// their wait are one asm block, so no register of a read in flight is ever the compiler's to
// reuse.  For the prologue.
template <int OFF>
__device__ __forceinline__ void lds_frags(u32x4 (&f)[1][2], unsigned p0, unsigned p1) {
  asm volatile(
      "ds_read_b128 %0, %2 offset:%4\n\t"
      "ds_read_b128 %1, %3 offset:%4\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(f[0][0]), "=&v"(f[0][1])
      : "v"(p0), "v"(p1), "i"(OFF)
      : "memory");
}
template <int OFF>
__device__ __forceinline__ void lds_frags(u32x4 (&f)[2][2], unsigned p0, unsigned p1) {
  asm volatile(
      "ds_read_b128 %0, %4 offset:%6\n\t"
      "ds_read_b128 %1, %4 offset:%7\n\t"
      "ds_read_b128 %2, %5 offset:%6\n\t"
      "ds_read_b128 %3, %5 offset:%7\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(f[0][0]), "=&v"(f[1][0]), "=&v"(f[0][1]), "=&v"(f[1][1])
      : "v"(p0), "v"(p1), "i"(OFF), "i"(OFF + 16 * ROWB)
      : "memory");
}
template <int OFF>
__device__ __forceinline__ void lds_frags(u32x4 (&f)[4][2], unsigned p0, unsigned p1) {
  asm volatile(
      "ds_read_b128 %0, %8 offset:%10\n\t"
      "ds_read_b128 %1, %8 offset:%11\n\t"
      "ds_read_b128 %2, %8 offset:%12\n\t"
      "ds_read_b128 %3, %8 offset:%13\n\t"
      "ds_read_b128 %4, %9 offset:%10\n\t"
      "ds_read_b128 %5, %9 offset:%11\n\t"
      "ds_read_b128 %6, %9 offset:%12\n\t"
      "ds_read_b128 %7, %9 offset:%13\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(f[0][0]), "=&v"(f[1][0]), "=&v"(f[2][0]), "=&v"(f[3][0]), "=&v"(f[0][1]), "=&v"(f[1][1]),
        "=&v"(f[2][1]), "=&v"(f[3][1])
      : "v"(p0), "v"(p1), "i"(OFF), "i"(OFF + 16 * ROWB), "i"(OFF + 32 * ROWB), "i"(OFF + 48 * ROWB)
      : "memory");
}
// FP8 rows: one 16-byte read per fragment carries both halves of the k-step.
template <int OFF>
__device__ __forceinline__ void lds_frags8(u32x4 (&f)[2], unsigned p) {
  asm volatile(
      "ds_read_b128 %0, %2 offset:%3\n\t"
      "ds_read_b128 %1, %2 offset:%4\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(f[0]), "=&v"(f[1])
      : "v"(p), "i"(OFF), "i"(OFF + 16 * ROWB8)
      : "memory");
}
template <int OFF>
__device__ __forceinline__ void lds_frags8(u32x4 (&f)[4], unsigned p) {
  asm volatile(
      "ds_read_b128 %0, %4 offset:%5\n\t"
      "ds_read_b128 %1, %4 offset:%6\n\t"
      "ds_read_b128 %2, %4 offset:%7\n\t"
      "ds_read_b128 %3, %4 offset:%8\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(f[0]), "=&v"(f[1]), "=&v"(f[2]), "=&v"(f[3])
      : "v"(p), "i"(OFF), "i"(OFF + 16 * ROWB8), "i"(OFF + 32 * ROWB8), "i"(OFF + 48 * ROWB8)
      : "memory");
}

// ---- one phase: FMH x FNH blocks, both halves of the k-step; next-phase reads; refill ----
// Operands: c<i><j> accumulators, a<i><k> and b<j><k> fragments; n* the next fragments, from
// lane addresses p0 / p1 (the k-halves) at offsets o0..; vo*, sb the refill's lane offsets and
// base, m its LDS address.  The compiler does not look into an asm block for the wait states that
// gfx9 leaves to software, so the block keeps them: an MFMA stands between each write of M0 and
// the load that takes its LDS address from it (one is due).  An accumulator comes back two
// (1 x 2 blocks) to eight MFMAs later, always as the same registers of the same kind of MFMA,
// which are forwarded (none is due), and nothing else touches it before the nops behind the loop.
// tests/test_device_waits.py holds the built code to all of them, across the blocks' edges too.
#define NT_MM(c, b, a) "v_mfma_f32_16x16x32_" NT_MFMA_T " %[" c "], %[" b "], %[" a "], %[" c "]\n\t"
#define NT_DS(n, p, o) "ds_read_b128 %[" n "], %[" p "] offset:%[" o "]\n\t"
#define NT_M0 "s_mov_b32 m0, %[m]\n\t"
#define NT_M1 "s_add_u32 m0, %[m], 0x400\n\t"
#define NT_LD0 "global_load_lds_dwordx4 %[vo0], %[sb]\n\t"
#define NT_LD1 "global_load_lds_dwordx4 %[vo1], %[sb]\n\t"
#define NT_END "s_waitcnt vmcnt(%[vm]) lgkmcnt(0)\n\ts_barrier"
// MFMAs of one k-half (suffix K), with something before each
#define NT_H24(K, r0, r1, r2, r3, r4, r5, r6, r7)                                                   \
  r0 NT_MM("c00", "b0" K, "a0" K) r1 NT_MM("c01", "b1" K, "a0" K) r2 NT_MM("c02", "b2" K, "a0" K)   \
  r3 NT_MM("c03", "b3" K, "a0" K) r4 NT_MM("c10", "b0" K, "a1" K) r5 NT_MM("c11", "b1" K, "a1" K)   \
  r6 NT_MM("c12", "b2" K, "a1" K) r7 NT_MM("c13", "b3" K, "a1" K)
#define NT_H22(K, r0, r1, r2, r3, r4, r5, r6, r7)                                                   \
  r0 r1 NT_MM("c00", "b0" K, "a0" K) r2 r3 NT_MM("c01", "b1" K, "a0" K)                             \
  r4 r5 NT_MM("c10", "b0" K, "a1" K) r6 r7 NT_MM("c11", "b1" K, "a1" K)
#define NT_H14(K, r0, r1, r2, r3, r4, r5, r6, r7)                                                   \
  r0 r1 NT_MM("c00", "b0" K, "a0" K) r2 r3 NT_MM("c01", "b1" K, "a0" K)                             \
  r4 r5 NT_MM("c02", "b2" K, "a0" K) r6 r7 NT_MM("c03", "b3" K, "a0" K)
#define NT_H12(K, r0, r1, r2, r3, r4, r5, r6, r7)                                                   \
  r0 r1 NT_MM("c00", "b0" K, "a0" K) r2 r3 NT_MM("c01", "b1" K, "a0" K) r4 r5 r6 r7
#define NT_READS2(H) H("0", NT_DS("n0", "p0", "o0"), NT_DS("n1", "p1", "o0"), "", "", "", "", "", "")
#define NT_READS4(H)                                                                                \
  H("0", NT_DS("n0", "p0", "o0"), NT_DS("n1", "p0", "o1"), NT_DS("n2", "p1", "o0"),                 \
    NT_DS("n3", "p1", "o1"), "", "", "", "")
#define NT_READS8(H)                                                                                \
  H("0", NT_DS("n0", "p0", "o0"), NT_DS("n1", "p0", "o1"), NT_DS("n2", "p0", "o2"),                 \
    NT_DS("n3", "p0", "o3"), NT_DS("n4", "p1", "o0"), NT_DS("n5", "p1", "o1"),                      \
    NT_DS("n6", "p1", "o2"), NT_DS("n7", "p1", "o3"))
#define NT_READSQ2(H) H("0", NT_DS("n0", "p0", "o0"), NT_DS("n1", "p0", "o1"), "", "", "", "", "", "")
#define NT_READSQ4(H)                                                                               \
  H("0", NT_DS("n0", "p0", "o0"), NT_DS("n1", "p0", "o1"), NT_DS("n2", "p0", "o2"),                 \
    NT_DS("n3", "p0", "o3"), "", "", "", "")
#define NT_C1(i) [c##i##0] "+v"(c[I0 + i][J0]), [c##i##1] "+v"(c[I0 + i][J0 + 1])
#define NT_C2(i) [c##i##2] "+v"(c[I0 + i][J0 + 2]), [c##i##3] "+v"(c[I0 + i][J0 + 3])
#define NT_ACC24 NT_C1(0), NT_C2(0), NT_C1(1), NT_C2(1)
#define NT_ACC22 NT_C1(0), NT_C1(1)
#define NT_ACC14 NT_C1(0), NT_C2(0)
#define NT_ACC12 NT_C1(0)
#define NT_FRAG(x, i) [x##i##0] "v"(x[i][0]), [x##i##1] "v"(x[i][1])
#define NT_AB24 NT_FRAG(a, 0), NT_FRAG(a, 1), NT_FRAG(b, 0), NT_FRAG(b, 1), NT_FRAG(b, 2), NT_FRAG(b, 3)
#define NT_AB22 NT_FRAG(a, 0), NT_FRAG(a, 1), NT_FRAG(b, 0), NT_FRAG(b, 1)
#define NT_AB14 NT_FRAG(a, 0), NT_FRAG(b, 0), NT_FRAG(b, 1), NT_FRAG(b, 2), NT_FRAG(b, 3)
#define NT_AB12 NT_FRAG(a, 0), NT_FRAG(b, 0), NT_FRAG(b, 1)
#define NT_OUT2 [n0] "=&v"(n[0][0]), [n1] "=&v"(n[0][1])
#define NT_OUT4 [n0] "=&v"(n[0][0]), [n1] "=&v"(n[1][0]), [n2] "=&v"(n[0][1]), [n3] "=&v"(n[1][1])
#define NT_OUT8                                                                                     \
  [n0] "=&v"(n[0][0]), [n1] "=&v"(n[1][0]), [n2] "=&v"(n[2][0]), [n3] "=&v"(n[3][0]),               \
      [n4] "=&v"(n[0][1]), [n5] "=&v"(n[1][1]), [n6] "=&v"(n[2][1]), [n7] "=&v"(n[3][1])
#define NT_OUTQ2 [n0] "=&v"(n[0]), [n1] "=&v"(n[1])
#define NT_OUTQ4 NT_OUTQ2, [n2] "=&v"(n[2]), [n3] "=&v"(n[3])
#define NT_IN2 [p0] "v"(p0), [p1] "v"(p1), [o0] "i"(OFF)
#define NT_IN4 NT_IN2, [o1] "i"(OFF + 16 * ROWB)
#define NT_IN8 NT_IN4, [o2] "i"(OFF + 32 * ROWB), [o3] "i"(OFF + 48 * ROWB)
#define NT_INQ2 [p0] "v"(p0), [o0] "i"(OFF), [o1] "i"(OFF + 16 * ROWB8)
#define NT_INQ4 NT_INQ2, [o2] "i"(OFF + 32 * ROWB8), [o3] "i"(OFF + 48 * ROWB8)
#define NT_LOAD1 [vo0] "v"(vo[0]), [sb] "s"(sb), [m] "s"(m)
#define NT_LOAD2 NT_LOAD1, [vo1] "v"(vo[1])
// LOADS: refill loads of this wave in the phase (1 or 2); S: FMH and FNH; R: reads
#define NT_PHASE_ASM(S, R)                                                                          \
  if constexpr (LOADS == 2)                                                                         \
    asm volatile(NT_READS##R(NT_H##S) NT_H##S("1", "", NT_M0, NT_LD0, NT_M1, NT_LD1, "", "", "") NT_END \
                 : NT_ACC##S, NT_OUT##R                                                             \
                 : NT_AB##S, NT_IN##R, NT_LOAD2, [vm] "i"(VM) : "memory", "m0", "scc");             \
  else                                                                                              \
    asm volatile(NT_READS##R(NT_H##S) NT_H##S("1", "", NT_M0, NT_LD0, "", "", "", "", "") NT_END    \
                 : NT_ACC##S, NT_OUT##R                                                             \
                 : NT_AB##S, NT_IN##R, NT_LOAD1, [vm] "i"(VM) : "memory", "m0", "scc");
#define NT_PHASE_FN(NAME, S, FMH, FNH, R, NTYPE)                                                    \
    template <int I0, int J0, int OFF, int LOADS, int VM>                                           \
    static __device__ __forceinline__ void NAME(floatx4 (&c)[2 * FMH][2 * FNH],                     \
                                                const u32x4 (&a)[FMH][2],                           \
                                                const u32x4 (&b)[FNH][2], u32x4 (&n)NTYPE,          \
                                                unsigned p0, unsigned p1, const unsigned* vo,       \
                                                const char* sb, unsigned m) {                       \
      NT_PHASE_ASM(S, R)                                                                            \
    }
// the phases that read the next A half, B half, or FP8 B half (one read carries both k-halves)
template <typename T, int FMH, int FNH> struct Phase;
#define NT_PHASE_STRUCT(TYPE)                                                                       \
  template <> struct Phase<TYPE, 2, 4> {                                                            \
    NT_PHASE_FN(read_a, 24, 2, 4, 4, [2][2])                                                        \
    NT_PHASE_FN(read_b, 24, 2, 4, 8, [4][2])                                                        \
    NT_PHASE_FN(read_q, 24, 2, 4, Q4, [4])                                                          \
  };                                                                                                \
  template <> struct Phase<TYPE, 2, 2> {                                                            \
    NT_PHASE_FN(read_a, 22, 2, 2, 4, [2][2])                                                        \
    NT_PHASE_FN(read_b, 22, 2, 2, 4, [2][2])                                                        \
    NT_PHASE_FN(read_q, 22, 2, 2, Q2, [2])                                                          \
  };                                                                                                \
  template <> struct Phase<TYPE, 1, 2> {                                                            \
    NT_PHASE_FN(read_a, 12, 1, 2, 2, [1][2])                                                        \
    NT_PHASE_FN(read_b, 12, 1, 2, 4, [2][2])                                                        \
    NT_PHASE_FN(read_q, 12, 1, 2, Q2, [2])                                                          \
  };                                                                                                \
  template <> struct Phase<TYPE, 1, 4> {                                                            \
    NT_PHASE_FN(read_a, 14, 1, 4, 2, [1][2])                                                        \
    NT_PHASE_FN(read_b, 14, 1, 4, 8, [4][2])                                                        \
    NT_PHASE_FN(read_q, 14, 1, 4, Q4, [4])                                                          \
  };
#define NT_MFMA_T "f16"
NT_PHASE_STRUCT(f16)
#undef NT_MFMA_T
#define NT_MFMA_T "bf16"
NT_PHASE_STRUCT(bf16)
#undef NT_MFMA_T

__device__ __forceinline__ void dma16(const char* src, unsigned char* dst) {
  __builtin_amdgcn_global_load_lds(src, NT_LDS(dst), 16, 0, 0);
}
__device__ __forceinline__ unsigned uniform(unsigned v) { return __builtin_amdgcn_readfirstlane(v); }
template <int N>
__device__ __forceinline__ void wait_vm() { asm volatile("s_waitcnt vmcnt(%0)" ::"i"(N) : "memory"); }
// The MFMAs of an asm block may still be writing their results when it ends.  The compiler does
// not know, so no use of c may come before the nops: to it, c is written again behind them.
template <int FM, int FN>
__device__ __forceinline__ void mfma_drain(floatx4 (&c)[FM][FN]) {
  asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) asm volatile("" : "+v"(c[i][j]));
}

// The first element of a word.
template <typename T>
__device__ __forceinline__ T first_value(unsigned w) {
  if constexpr (sizeof(T) == 2) return __builtin_bit_cast(T, (unsigned short)(w & 0xffffu));
  else return __builtin_bit_cast(T, w);
}
// Orders a wave's LDS writes before its own reads of what other lanes wrote.
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
}

// Exchanges the odd 16-lane rows of a with the even ones of b: of two neighbouring blocks'
// words, a lane then holds words of eight consecutive columns of one block.
__device__ __forceinline__ void row_swap(unsigned& a, unsigned& b) {
  const auto r = __builtin_amdgcn_permlane16_swap(a, b, false, false);
  a = r[0];
  b = r[1];
}
template <typename T>
__device__ __forceinline__ unsigned pack2(float x, float y) {
  const T t[2] = {from_f32<T>(x), from_f32<T>(y)};
  return __builtin_bit_cast(unsigned, t);
}
template <typename T>
__device__ __forceinline__ float2 unpack2(unsigned w) {
  struct P { T a, b; };
  const P p = __builtin_bit_cast(P, w);
  return make_float2(to_f32(p.a), to_f32(p.b));
}

// The epilogue's mode as a constant: the modes that a role's launches use.
template <int ROLE, typename F>
__device__ __forceinline__ void mode_switch(int mode, F& f) {
  using std::integral_constant;
  switch (mode) {
    case EPI_RELU:
      if constexpr (ROLE != 2) f(integral_constant<int, EPI_RELU>{});
      break;
    case EPI_RESID:
      if constexpr (ROLE != 2) f(integral_constant<int, EPI_RESID>{});
      break;
    case EPI_SELF_QKV:
      if constexpr (ROLE == 1) f(integral_constant<int, EPI_SELF_QKV>{});
      break;
    case EPI_CROSS_KV:
      if constexpr (ROLE == 0) f(integral_constant<int, EPI_CROSS_KV>{});
      break;
    default: f(integral_constant<int, EPI_STORE>{}); break;
  }
}

// A word that no block of this launch writes, through the scalar cache.
__device__ __forceinline__ int scalar_int(const int* p) {
  return *reinterpret_cast<const __attribute__((address_space(4))) int*>(reinterpret_cast<uintptr_t>(p));
}

// What the epilogue of a whole, aligned tile of one block row adds, read before the k-loop: at
// the few k-steps of a small product these loads, one after another behind the last MFMA, are
// a fifth of its time.
template <int FN>
struct EpiAhead {
  float4 bias[FN];
  floatx4 colsum[FN];
  uint4 resid[FN];      // 16-bit: [FN / 2] used
  int sent = 0;
  bool on = false;
};
template <typename T, int FN, int ROLE, bool LNF>
__device__ __forceinline__ void epi_ahead(EpiAhead<FN>& e, const GemmEpi& epi, int M, int mw, int nw, int fr, int fc) {
  const int m = min(mw + fr, M - 1);
  if constexpr (LNF) {
#pragma unroll
    for (int j = 0; j < FN; ++j) e.colsum[j] = *reinterpret_cast<const floatx4*>(epi.lnf_colsum + nw + j * 16 + 4 * fc);
  }
  if (epi.bias) {
#pragma unroll
    for (int j = 0; j < FN; ++j) e.bias[j] = *reinterpret_cast<const float4*>(epi.bias + nw + j * 16 + 4 * fc);
  }
  if (epi.mode == EPI_RESID) {
    const T* r = static_cast<const T*>(epi.resid) + (size_t)m * epi.ldc + nw;
    if constexpr (sizeof(T) == 2) {
#pragma unroll
      for (int jp = 0; jp < FN / 2; ++jp)
        e.resid[jp] = *reinterpret_cast<const uint4*>(r + jp * 32 + (fc & 1) * 16 + (fc >> 1) * 8);
    } else {
#pragma unroll
      for (int j = 0; j < FN; ++j) e.resid[j] = *reinterpret_cast<const uint4*>(r + j * 16 + 4 * fc);
    }
  }
  if constexpr (ROLE == 1) {
    if (epi.mode == EPI_SELF_QKV) e.sent = epi.sent_list[m / epi.beam];
  }
}
template <typename T, bool F8, bool LNF>
__device__ __forceinline__ bool epi_whole(const GemmEpi& epi, int nw, int cols, int N) {
  const bool f32_out = epi.mode <= EPI_STORE || epi.mode == EPI_TOPK ? epi.out_f32 : 0;
  uintptr_t al = reinterpret_cast<uintptr_t>(epi.bias);
  if (epi.mode != EPI_CROSS_KV) al |= reinterpret_cast<uintptr_t>(epi.out) | ((uintptr_t)epi.ldc * (f32_out ? 4 : sizeof(T)));
  if (epi.mode == EPI_RESID) al |= reinterpret_cast<uintptr_t>(epi.resid);
  if (F8) al |= reinterpret_cast<uintptr_t>(epi.wscale);
  if (LNF) al |= reinterpret_cast<uintptr_t>(epi.lnf_colsum);
  return nw + cols <= N && (al & 15) == 0;
}

// The epilogue of a wave's FM x FN blocks: lane (fr, fc) holds columns nw + 16 j + 4 fc .. + 3 of
// the rows mw + 16 i + fr.  mu, rs: the rows' statistics (folded LayerNorm); cs: LDS of the
// wave's own for half its rows in fp32, ln_mu / ln_rs the statistics of all its rows in LDS.
template <typename T, int FM, int FN, int ROLE, bool F8, bool LNF>
__device__ __forceinline__ void phased_epilogue(floatx4 (&c)[FM][FN], const GemmEpi& epi, int M, int N, int mw, int nw,
                                                int t_slot, int fr, int fc, const float (&mu)[FM],
                                                const float (&rs)[FM], float* cs, const float* ln_mu,
                                                const float* ln_rs, const EpiAhead<FN>& ahead) {
  using std::integral_constant;

  if constexpr (ROLE == 2) {
    static_assert(FN * 16 == 128, "a wave's columns are one selection tile");
    // selection records, as topk_tile_rows forms them: a lane's columns in increasing order,
    // then the four lanes of the row
    if (epi.mode == EPI_TOPK) {
      if (nw + 128 > N) {
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
          for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r)
              if (nw + j * 16 + 4 * fc + r >= N) c[i][j][r] = -INFINITY;
      }
#pragma unroll
      for (int i = 0; i < FM; ++i) {
        float mx = -INFINITY;
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
          for (int r = 0; r < 4; ++r) mx = fmaxf(mx, c[i][j][r]);
        int bi = INT_MAX;   // the lowest of the lane's columns holding its maximum
        if (mx != -INFINITY) {
#pragma unroll
          for (int j = FN - 1; j >= 0; --j)
#pragma unroll
            for (int r = 3; r >= 0; --r)
              if (c[i][j][r] == mx) bi = nw + j * 16 + 4 * fc + r;
        }
#pragma unroll
        for (int o = 32; o > 8; o >>= 1) {
          const float om = __shfl_xor(mx, o, kWave);
          const int oi = __shfl_xor(bi, o, kWave);
          if (om > mx || (om == mx && oi < bi)) { mx = om; bi = oi; }
        }
        float sum = 0.f;
        if (mx != -INFINITY) {
#pragma unroll
          for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) sum += __expf(c[i][j][r] - mx);
        }
        sum += __shfl_xor(sum, 32, kWave);
        sum += __shfl_xor(sum, 16, kWave);
        const int m = mw + i * 16 + fr;
        if (fc == 0 && m < M && nw < N)
          *reinterpret_cast<float4*>(epi.part + ((size_t)m * epi.n_tiles + nw / 128) * topk_record(1)) =
              make_float4(mx, sum, mx, __int_as_float(bi));
      }
      if (!epi.out) return;   // the records are all the selection needs; else the logits too
    }
  }

  if (FM == 1 ? !ahead.on : !epi_whole<T, F8, LNF>(epi, nw, FN * 16, N)) {
    if constexpr (FM == 1) {   // a ragged or unaligned tile, four columns at a time
      auto finish = [&](auto mode_c) {
        constexpr int MODE = decltype(mode_c)::value;
        const int m = mw + fr;
#pragma unroll
        for (int j = 0; j < FN; ++j) {
          const int n = nw + j * 16 + 4 * fc;
          if (m >= M || n >= N) continue;
          float v[4];
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int cc = min(n + r, N - 1);
            v[r] = c[0][j][r];
            if constexpr (F8) v[r] *= epi.wscale[cc];
            if constexpr (LNF) v[r] = (v[r] - mu[0] * epi.lnf_colsum[cc]) * rs[0];
            if constexpr (F8 || LNF) asm("" : "+v"(v[r]));   // rounded before the bias is added, as where staged
          }
          epilogue4<T, MODE, true>(epi, m, n, N, make_float4(v[0], v[1], v[2], v[3]), t_slot);
        }
      };
      mode_switch<ROLE>(epi.mode, finish);
    } else {
      // A ragged or unaligned tile: its halves through LDS (the wave's own part), then four columns
      // at a time.  A lane's columns are the same in every row it takes, so what the columns add is
      // read once, and four rows' residuals together: one after another these loads were most of the
      // tile's time (fp16, one after another / now: 2160x1000x512 with a residual 20.2 / 10.9 us,
      // 16384x4092x512 with a bias 147 / 88, 2160x1000x256 with a folded LayerNorm 11.5 / 8.3).
      constexpr int HROWS = FM * 8, CS = FN * 16 + 4, FH = FM / 2;
      constexpr int GC = FN * 4, RP = kWave / GC, U = 4;   // groups of four columns; rows a pass; passes together
      static_assert(HROWS % (RP * U) == 0, "a half's rows are whole batches of passes");
      const int lane = fc * 16 + fr, c4 = lane % GC * 4, n = nw + c4;
      float bias[4], colsum[4], scale[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int cc = min(n + r, N - 1);
        bias[r] = epi.bias ? epi.bias[cc] : 0.f;
        colsum[r] = LNF ? epi.lnf_colsum[cc] : 0.f;
        scale[r] = F8 ? epi.wscale[cc] : 1.f;
      }
#pragma unroll 1
      for (int h = 0; h < 2; ++h) {
#pragma unroll
        for (int i = 0; i < FM; ++i)
          if (i / FH == h) {
#pragma unroll
            for (int j = 0; j < FN; ++j)
              *reinterpret_cast<floatx4*>(&cs[(i % FH * 16 + fr) * CS + j * 16 + 4 * fc]) = c[i][j];
          }
        wave_lds_fence();
        auto finish = [&](auto mode_c) {
          constexpr int MODE = decltype(mode_c)::value;
          if (n >= N) return;
#pragma unroll 1
          for (int p = 0; p < HROWS / RP; p += U) {
            const int row0 = p * RP + lane / GC;
            T q[MODE == EPI_RESID ? U : 1][4];
            if constexpr (MODE == EPI_RESID) {
#pragma unroll
              for (int u = 0; u < U; ++u) {
                const int m = min(mw + h * HROWS + row0 + u * RP, M - 1);
                const T* x = static_cast<const T*>(epi.resid) + (size_t)m * epi.ldc + n;
#pragma unroll
                for (int r = 0; r < 4; ++r) q[u][r] = x[min(r, N - 1 - n)];
              }
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
              const int row = row0 + u * RP, m = mw + h * HROWS + row;
              float v[4];
#pragma unroll
              for (int r = 0; r < 4; ++r) {
                v[r] = cs[row * CS + c4 + r];
                if constexpr (F8) v[r] *= scale[r];
                if constexpr (LNF) v[r] = (v[r] - ln_mu[h * HROWS + row] * colsum[r]) * ln_rs[h * HROWS + row];
                if constexpr (F8 || LNF) asm("" : "+v"(v[r]));   // rounded before the bias is added, as where staged
                if (epi.bias) v[r] += bias[r];
                if constexpr (MODE == EPI_RESID) v[r] += to_f32(q[u][r]);
              }
              if (m < M) epilogue4<T, MODE, false>(epi, m, n, N, make_float4(v[0], v[1], v[2], v[3]), t_slot);
            }
          }
        };
        mode_switch<ROLE>(epi.mode, finish);
        wave_lds_fence();
      }
    }
    return;
  }

  // Whole columns: 16-bit results leave as eight columns a lane -- after the swap lane group
  // fc holds columns 8 (fc / 2) .. + 7 of block j + fc % 2 -- and addresses are a row's, formed
  // once, plus constants.
  const int n8 = (fc & 1) * 16 + (fc >> 1) * 8;
  if constexpr (F8 || LNF) {   // scales and the folded LayerNorm, in the order of the staged tiles
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      const int n = nw + j * 16 + 4 * fc;
      floatx4 c4{}, w4{};
      if constexpr (LNF && FM == 1) c4 = ahead.colsum[j];
      else if constexpr (LNF) c4 = *reinterpret_cast<const floatx4*>(epi.lnf_colsum + n);
      if constexpr (F8) w4 = *reinterpret_cast<const floatx4*>(epi.wscale + n);
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          float x = c[i][j][r];
          if constexpr (F8) x *= w4[r];
          if constexpr (LNF) x = (x - mu[i] * c4[r]) * rs[i];
          asm("" : "+v"(x));   // rounded before the bias is added
          c[i][j][r] = x;
        }
    }
  }
  auto direct = [&](auto mode_c) {
    constexpr int MODE = decltype(mode_c)::value;
    float4 b4[FN];
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      if constexpr (FM == 1) b4[j] = ahead.bias[j];
      else b4[j] = epi.bias ? *reinterpret_cast<const float4*>(epi.bias + nw + j * 16 + 4 * fc) : make_float4(0.f, 0.f, 0.f, 0.f);
    }
    constexpr bool RES = MODE == EPI_RESID && sizeof(T) == 2;
    uint4 res[RES ? FM : 1][RES ? FN / 2 : 1];
    if constexpr (RES) {   // every residual before the first store (the output may alias it)
#pragma unroll
      for (int i = 0; i < FM; ++i) {
        const T* r = static_cast<const T*>(epi.resid) + (size_t)min(mw + i * 16 + fr, M - 1) * epi.ldc + nw + n8;
#pragma unroll
        for (int jp = 0; jp < FN / 2; ++jp) {
          if constexpr (FM == 1) res[i][jp] = ahead.resid[jp];
          else res[i][jp] = *reinterpret_cast<const uint4*>(r + jp * 32);
        }
      }
    }
#pragma unroll
    for (int i = 0; i < FM; ++i) {
      const int m = mw + i * 16 + fr;
      // the row's place; column blocks of 32 lie within one head
      size_t row = (size_t)m * epi.ldc, cell = 0;
      if constexpr (MODE == EPI_STORE) {
        if (epi.out_map && m < M) row = (size_t)(epi.sent_list[m / epi.beam] * epi.beam + m % epi.beam) * epi.ldc;
      }
      if constexpr (MODE == EPI_SELF_QKV) {
        const int mc = min(m, M - 1);
        const int p = (FM == 1 ? ahead.sent : epi.sent_list[mc / epi.beam]) * epi.beam + mc % epi.beam;
        cell = ((size_t)p * epi.H * epi.Tcap + t_slot) * epi.dh;
      }
      if constexpr (MODE == EPI_CROSS_KV) {
        const int b = m / epi.S;
        cell = ((size_t)b * epi.H * epi.S + (m - b * epi.S)) * epi.dh;
      }
      if (m >= M) continue;
      auto cache_of = [&](auto elem, int n) {   // column n >= d of the row, in the step's cache slot
        int cd = n - epi.d;
        const int kv = cd >= epi.d;
        cd -= kv * epi.d;
        const int hd = cd / epi.dh, x = cd - hd * epi.dh;
        return static_cast<decltype(elem)*>(kv ? epi.vcache : epi.kcache) + cell + (size_t)hd * epi.Tcap * epi.dh + x;
      };
      auto cell_of = [&](int n) -> T* {         // column n of the row
        if constexpr (MODE == EPI_SELF_QKV) {
          if (n >= epi.d) return cache_of(T{}, n);
        }
        if constexpr (MODE == EPI_CROSS_KV) {
          const int jl = n / (2 * epi.d);
          int cd = n - jl * 2 * epi.d;
          const int kv = cd >= epi.d;
          cd -= kv * epi.d;
          const int hd = cd / epi.dh, x = cd - hd * epi.dh;
          return static_cast<T*>(epi.cross) + (((size_t)jl * 2 + kv) * epi.B * epi.H + hd) * (size_t)epi.S * epi.dh + x + cell;
        }
        return static_cast<T*>(epi.out) + row + n;
      };
#pragma unroll
      for (int jp = 0; jp < FN / 2; ++jp) {
        float v[2][4];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const int j = 2 * jp + u;
          const float bb[4] = {b4[j].x, b4[j].y, b4[j].z, b4[j].w};
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            float x = c[i][j][r];
            if (epi.bias) x += bb[r];
            if constexpr (MODE == EPI_RELU) x = fmaxf(x, 0.f);
            v[u][r] = x;
          }
        }
        const int n = nw + jp * 32;   // the same in every lane
        if constexpr (MODE == EPI_STORE) {
          if (epi.out_f32) {
            float* o = static_cast<float*>(epi.out) + row + n + 4 * fc;
#pragma unroll
            for (int u = 0; u < 2; ++u)
              *reinterpret_cast<float4*>(o + u * 16) = make_float4(v[u][0], v[u][1], v[u][2], v[u][3]);
            continue;
          }
        }
        if constexpr (sizeof(T) == 4) {   // four columns a lane are 16 bytes already
#pragma unroll
          for (int u = 0; u < 2; ++u) {
            const int nu = n + u * 16 + 4 * fc;
            if constexpr (MODE == EPI_RESID) {
              static_assert(FM == 1, "fp32 tiles are one block row");
              const floatx4 q = __builtin_bit_cast(floatx4, ahead.resid[2 * jp + u]);
#pragma unroll
              for (int r = 0; r < 4; ++r) v[u][r] += q[r];
            }
            *reinterpret_cast<float4*>(cell_of(n) + u * 16 + 4 * fc) = make_float4(v[u][0], v[u][1], v[u][2], v[u][3]);
          }
        } else {
          if constexpr (RES) {   // the residual's words back into the blocks' layout
            uint4 q = res[i][jp];
            row_swap(q.x, q.z);
            row_swap(q.y, q.w);
            const unsigned w[4] = {q.x, q.y, q.z, q.w};
  #pragma unroll
            for (int r = 0; r < 4; ++r) {
              const float2 f = unpack2<T>(w[r]);
              v[r / 2][r % 2 * 2] += f.x;
              v[r / 2][r % 2 * 2 + 1] += f.y;
            }
          }
          if constexpr (MODE == EPI_SELF_QKV && std::is_same<T, f16>::value) {
            if (epi.kv_f8 && n >= epi.d) {   // E4M3 cache
              uint8_t* o8 = cache_of(uint8_t{}, n);
  #pragma unroll
              for (int u = 0; u < 2; ++u)
                *reinterpret_cast<uint32_t*>(o8 + u * 16 + 4 * fc) =
                    (uint32_t)e4m3_rne(v[u][0]) | ((uint32_t)e4m3_rne(v[u][1]) << 8) |
                    ((uint32_t)e4m3_rne(v[u][2]) << 16) | ((uint32_t)e4m3_rne(v[u][3]) << 24);
              continue;
            }
          }
          uint4 q;
          q.x = pack2<T>(v[0][0], v[0][1]);
          q.y = pack2<T>(v[0][2], v[0][3]);
          q.z = pack2<T>(v[1][0], v[1][1]);
          q.w = pack2<T>(v[1][2], v[1][3]);
          row_swap(q.x, q.z);
          row_swap(q.y, q.w);
          *reinterpret_cast<uint4*>(cell_of(n) + n8) = q;
        }
      }
    }
  };
  mode_switch<ROLE>(epi.mode, direct);
}

// Direct loads of a wave that may be outstanding when phase q of a k-step ends: those of the
// six halves behind the one the phase after the next multiplies.
constexpr int phase_vm(int la, int lb) { return 3 * la + 3 * lb; }

// Workgroup shapes: waves in M and N, blocks per half of a wave's rows and columns.
struct Tile256 { static constexpr int WGM = 4, WGN = 2, FMH = 2, FNH = 4; };   // 256x256, eight waves
struct Tile128 { static constexpr int WGM = 2, WGN = 2, FMH = 2, FNH = 2; };   // 128x128, four waves
struct Tile64 { static constexpr int WGM = 2, WGN = 2, FMH = 1, FNH = 2; };    // 64x128, four waves
struct TileSel { static constexpr int WGM = 4, WGN = 1, FMH = 1, FNH = 4; };   // 128x128, a wave 128 columns

template <typename T, typename W, int ROLE, bool F8, bool LNF>
__global__ __launch_bounds__(W::WGM * W::WGN * kWave, 2) void gemm_phased_kernel(
    const T* __restrict__ A, int lda, const void* __restrict__ Bt, int M, int N, int K, GemmEpi epi, int tiles_m,
    int tiles_n) {
  constexpr int WGM = W::WGM, WGN = W::WGN, NW = WGM * WGN, FMH = W::FMH, FNH = W::FNH;
  constexpr int FM = 2 * FMH, FN = 2 * FNH;               // blocks per wave
  static_assert(!F8 || std::is_same<T, f16>::value, "FP8 weights pair with fp16 activations");
  constexpr int BM = WGM * FM * 16, BN = WGN * FN * 16;
  using Ph = Phase<T, FMH, FNH>;
  constexpr int ROWB_B = F8 ? ROWB8 : ROWB;
  constexpr int HAB = WGM * FMH * 16 * ROWB, HBB = WGN * FNH * 16 * ROWB_B;   // bytes of a half region
  constexpr int LPA = HAB / 1024 / NW, LPB = HBB / 1024 / NW;                 // direct loads per wave and half
  static_assert(LPA * 1024 * NW == HAB && LPB * 1024 * NW == HBB, "halves split evenly over the waves");
  constexpr int SLOT = 2 * (HAB + HBB);
  constexpr int OB0 = 0, OB1 = HBB, OA0 = 2 * HBB, OA1 = 2 * HBB + HAB;
  static_assert(OA1 + HAB <= 65536, "region offsets fit the ds_read immediate");
  // the epilogue's staging reuses the k-loop's LDS: per wave, half its rows in fp32
  constexpr int HROWS = FMH * 16, CS = FN * 16 + 4, CSB = NW * HROWS * CS * 4;
  constexpr int EPIB = CSB + (LNF ? 2 * BM * 4 : 0);
  __shared__ __attribute__((aligned(1024))) unsigned char lds[2 * SLOT > EPIB ? 2 * SLOT : EPIB];

  asm volatile("" ::"s"(epi.ctl), "s"(epi.bias), "s"(epi.out), "s"(epi.ldc), "s"(epi.wscale), "s"(epi.part),
               "s"(tiles_n), "s"(M), "s"(Bt));
  if (epi.ctl) {
    M = min(M, epi.ctl[CTL_NLIVE] * epi.ctl_rows);
    tiles_m = (M + BM - 1) / BM;
  }
  // tile assignment: XCD-contiguous, then grouped by 8 tile-rows
  const int ntiles = tiles_m * tiles_n;
  int pid = blockIdx.x;
  if (pid >= ntiles) return;
  {
    const int q = ntiles / 8, r = ntiles % 8, xcd = pid % 8, idx = pid / 8;
    pid = xcd < r ? xcd * (q + 1) + idx : r * (q + 1) + (xcd - r) * q + idx;
  }
  constexpr int GROUP = 8;
  const int per_group = GROUP * tiles_n;
  const int first_m = (pid / per_group) * GROUP;
  const int gsize = min(tiles_m - first_m, GROUP);
  const int tm = first_m + (pid % per_group) % gsize, tn = (pid % per_group) / gsize;
  const int m0 = tm * BM, n0 = tn * BN;
  const int t_slot = epi.ctl ? epi.ctl[CTL_T] : epi.t;

  int lane = threadIdx.x % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int wm = wave / WGN, wn = wave % WGN;
  int fr = lane & 15, fc = lane >> 4;

  // Direct loads: one instruction fills 1 KB of a half region, 8 rows of 128 bytes (16 of
  // 64 for FP8 weights); region row r of half h is tile row (r / rows) * 2 * rows + h *
  // rows + r % rows, rows being a wave's rows of the half.  A lane's rows of one operand
  // share their 16-byte chunk, so each is the lane's first one plus a uniform offset, and
  // rows past the edge re-read the last one (never stored) by a minimum on the offset.
  const unsigned lda_b = (unsigned)lda * sizeof(T), ldb_b = (unsigned)K * (F8 ? 1 : sizeof(T));
  const int ga = wave * LPA * 8, gb = wave * LPB * (F8 ? 16 : 8);   // first region rows of the wave
  const unsigned cha = ((lane & 7) ^ (lane >> 3)) << 4;
  const unsigned chb = F8 ? ((lane & 3) ^ (lane >> 4)) << 4 : cha;
  const unsigned a_last = (unsigned)(M - 1) * lda_b + cha, b_last = (unsigned)(N - 1) * ldb_b + chb;
  unsigned a_first = (unsigned)(m0 + ga / (FMH * 16) * (FM * 16) + ga % (FMH * 16) + (lane >> 3)) * lda_b + cha;
  unsigned b_first =
      (unsigned)(n0 + gb / (FNH * 16) * (FN * 16) + gb % (FNH * 16) + (F8 ? lane >> 2 : lane >> 3)) * ldb_b + chb;
  const char* Ab = reinterpret_cast<const char*>(A);
  const char* Bb = static_cast<const char*>(Bt);
  auto off_a = [&](int h, unsigned cap, unsigned (&vo)[2]) {
#pragma unroll
    for (int i = 0; i < LPA; ++i) vo[i] = min(min(a_first + (h * (FMH * 16) + i * 8) * lda_b, a_last), cap);
  };
  auto off_b = [&](int h, unsigned cap, unsigned (&vo)[2]) {
#pragma unroll
    for (int i = 0; i < LPB; ++i) vo[i] = min(min(b_first + (h * (FNH * 16) + i * 8) * ldb_b, b_last), cap);
  };
  const unsigned lb = (unsigned)(uintptr_t)NT_LDS(lds);
  const unsigned ma = lb + wave * LPA * 1024, mb_ = lb + wave * LPB * 1024;   // the wave's part of a region
  auto load_a = [&](int h, int kt, int slot) {
    unsigned vo[2];
    off_a(h, ~0u, vo);
#pragma unroll
    for (int i = 0; i < LPA; ++i)
      dma16(Ab + (size_t)kt * ROWB + vo[i], lds + slot * SLOT + (h ? OA1 : OA0) + (wave * LPA + i) * 1024);
  };
  auto load_b = [&](int h, int kt, int slot) {
    unsigned vo[2];
    off_b(h, ~0u, vo);
#pragma unroll
    for (int i = 0; i < LPB; ++i)
      dma16(Bb + (size_t)kt * ROWB_B + vo[i], lds + slot * SLOT + (h ? OB1 : OB0) + (wave * LPB + i) * 1024);
  };

  floatx4 acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};

  // lane addresses of the fragments in slot 0: first half of the k-step; the second half's
  // chunks (FP8: the k-values of both operands pair up 16 by 16) differ in one address bit
  unsigned pa = lb + (wm * FMH * 16 + fr) * ROWB + (((F8 ? 2 * fc : fc) ^ (fr & 7)) << 4);
  unsigned pb = F8 ? lb + (wn * FNH * 16 + fr) * ROWB8 + ((fc ^ ((fr >> 2) & 3)) << 4)
                         : lb + (wn * FNH * 16 + fr) * ROWB + ((fc ^ (fr & 7)) << 4);
  constexpr unsigned XA = F8 ? 16 : 64, XB = 64;
  u32x4 ax[FMH][2], ay[FMH][2], az[FMH][2], b0[FNH][2], b1[FNH][2], bq[FNH];

  // folded LayerNorm: the row statistics of the wave's rows, A half wn of them in this wave
  // (both waves of a row hold the same fragments)
  static_assert(!LNF || WGN == 2, "two waves share a row's statistics");
  float lsum[LNF ? FMH : 1], lsq[LNF ? FMH : 1];
  T lsh[LNF ? FMH : 1];
#pragma unroll
  for (int i = 0; i < (LNF ? FMH : 1); ++i) lsum[i] = lsq[i] = 0.f;
  auto stats = [&](u32x4 (&a)[FMH][2], int h) {
    if constexpr (LNF) {
      if (wn == h) {
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
          for (int i = 0; i < FMH; ++i) frag_stats<T>(a[i][k], lsh[i], lsum[i], lsq[i]);
      }
    }
  };
  auto widen = [&](u32x4 (&b)[FNH][2]) {
    if constexpr (F8) {
#pragma unroll
      for (int j = 0; j < FNH; ++j) {
        b[j][0] = f8_to_f16x8(bq[j].x, bq[j].y);
        b[j][1] = f8_to_f16x8(bq[j].z, bq[j].w);
      }
    }
  };

  const int nk = (int)((size_t)K * sizeof(T) / ROWB);   // even (checked by the launcher)
  // prologue: both slots, in the order the phases read them; A0 and B0 of the first k-step
  // (with a folded LayerNorm also A1, whose rows' first values are the statistics' shifts)
  load_a(0, 0, 0);
  load_b(0, 0, 0);
  load_a(1, 0, 0);
  load_b(1, 0, 0);
  load_a(0, 1, 1);
  load_b(0, 1, 1);
  load_a(1, 1, 1);
  load_b(1, 1, 1);
  wait_vm<2 * LPA + 3 * LPB>();   // A0, B0 and A1 of the first k-step have landed
  __builtin_amdgcn_s_barrier();
  lds_frags<OA0>(ax, pa, pa ^ XA);
  if constexpr (F8) lds_frags8<OB0>(bq, pb);
  else lds_frags<OB0>(b0, pb, pb ^ XB);
  if constexpr (LNF) {
    lds_frags<OA1>(ay, pa, pa ^ XA);
#pragma unroll
    for (int i = 0; i < FMH; ++i) {
      // chunk 0 of the row is in lane group 0 of the first half of the k-step
      const unsigned w = __shfl(wn ? ay[i][0].x : ax[i][0].x, fr, kWave);
      lsh[i] = first_value<T>(w);
    }
  }
  __builtin_amdgcn_s_barrier();
  load_a(0, min(2, nk - 1), 0);
  widen(b0);

  // One k-step in slot S.  A0 is in a0 and B0 in b0 on entry, the next k-step's in a2 and b0 on
  // return.  Refills past the last k-step read the operand's first line only.
  constexpr int VM = phase_vm(LPA, LPB);
  auto kstep = [&](auto slot_c, int kt, u32x4 (&a0)[FMH][2], u32x4 (&a1)[FMH][2], u32x4 (&a2)[FMH][2]) {
    constexpr int S = decltype(slot_c)::value;
    constexpr int SO = S * SLOT, SN = (1 - S) * SLOT;
    const bool in2 = kt + 2 < nk, in3 = kt + 3 < nk;
    const unsigned cap2 = in2 ? ~0u : 0u, cap3 = in3 ? ~0u : 0u;
    const char* A2 = in2 ? Ab + (size_t)(kt + 2) * ROWB : Ab;
    const char* A3 = in3 ? Ab + (size_t)(kt + 3) * ROWB : Ab;
    const char* B2 = in2 ? Bb + (size_t)(kt + 2) * ROWB_B : Bb;
    // opaque here, so that what derives from them is formed where it is used and not kept in
    // registers through the loop (the four phases hold 224 of 256)
    asm volatile("" : "+v"(pa), "+v"(pb), "+v"(a_first), "+v"(b_first));
    unsigned vo[2] = {0, 0};
    // (A0, B0); reads A1, refills B0
    {
      off_b(0, cap2, vo);
      const unsigned p = pa + SO;
      Ph::template read_a<0, 0, OA1, LPB, VM>(acc, a0, b0, a1, p, p ^ XA, vo, B2, mb_ + SO + OB0);
    }
    stats(a0, 0);
    // (A1, B0); reads B1, refills A1
    {
      off_a(1, cap2, vo);
      const unsigned p = pb + SO;
      if constexpr (F8) Ph::template read_q<FMH, 0, OB1, LPA, VM>(acc, a1, b0, bq, p, p, vo, A2, ma + SO + OA1);
      else Ph::template read_b<FMH, 0, OB1, LPA, VM>(acc, a1, b0, b1, p, p ^ XB, vo, A2, ma + SO + OA1);
    }
    stats(a1, 1);
    widen(b1);
    // (A1, B1); reads the next A0, refills B1
    {
      off_b(1, cap2, vo);
      const unsigned p = pa + SN;
      Ph::template read_a<FMH, FNH, OA0, LPB, VM>(acc, a1, b1, a2, p, p ^ XA, vo, B2, mb_ + SO + OB1);
    }
    // (A0, B1); reads the next B0, refills the next k-step's A0
    {
      off_a(0, cap3, vo);
      const unsigned p = pb + SN;
      if constexpr (F8) Ph::template read_q<0, FNH, OB0, LPA, VM>(acc, a0, b1, bq, p, p, vo, A3, ma + SN + OA0);
      else Ph::template read_b<0, FNH, OB0, LPA, VM>(acc, a0, b1, b0, p, p ^ XB, vo, A3, ma + SN + OA0);
    }
    widen(b0);
  };
  using std::integral_constant;
  for (int kt = 0; kt < nk; kt += 2) {
    kstep(integral_constant<int, 0>{}, kt, ax, ay, az);
    kstep(integral_constant<int, 1>{}, kt + 1, az, ay, ax);
  }
  lane = __lane_id();             // formed again: nothing of the lane's is kept through the loop
  asm volatile("" : "+v"(lane));
  fr = lane & 15;
  fc = lane >> 4;
  mfma_drain(acc);
  wait_vm<0>();                   // the refills past the end have landed
  __builtin_amdgcn_s_barrier();   // in every wave: LDS is free

  // folded LayerNorm: mean and 1/sqrt(biased variance + eps) per tile row, as in nt_gemm.hip
  float* ln_mu = reinterpret_cast<float*>(lds + CSB);
  float* ln_rs = ln_mu + BM;
  if constexpr (LNF) {
    const float inv_k = 1.0f / (float)K;
#pragma unroll
    for (int i = 0; i < FMH; ++i) {
      float s = lsum[i], q = lsq[i];
      s += __shfl_xor(s, 16, kWave);
      q += __shfl_xor(q, 16, kWave);
      s += __shfl_xor(s, 32, kWave);
      q += __shfl_xor(q, 32, kWave);
      if (fc == 0) {
        const float ms = s * inv_k;
        const float var = fmaxf(q * inv_k - ms * ms, 0.f);
        const int row = wm * (FM * 16) + wn * (FMH * 16) + i * 16 + fr;
        ln_mu[row] = to_f32(lsh[i]) + ms;
        ln_rs[row] = 1.0f / sqrtf(var + epi.lnf_eps);
      }
    }
    __syncthreads();
  }

  float mu[FM], rs[FM];
#pragma unroll
  for (int i = 0; i < FM; ++i) {
    mu[i] = LNF ? ln_mu[wm * (FM * 16) + i * 16 + fr] : 0.f;
    rs[i] = LNF ? ln_rs[wm * (FM * 16) + i * 16 + fr] : 1.f;
  }
  phased_epilogue<T, FM, FN, ROLE, F8, LNF>(acc, epi, M, N, m0 + wm * (FM * 16), n0 + wn * (FN * 16), t_slot, fr, fc, mu,
                                            rs, reinterpret_cast<float*>(lds) + wave * (HROWS * CS),
                                            ln_mu + wm * (FM * 16), ln_rs + wm * (FM * 16), EpiAhead<FN>{});
}

// ---- few tiles: 64x32, one phase a k-step ----------------------------------------------------
// Where a product has few tiles for the GPU's CUs, a tile's own chain bounds the launch: four
// phases a k-step cost four LDS round trips and barriers.  Here a k-step is one phase: a wave
// (16 rows, two blocks of columns) multiplies while it reads the next k-step's fragments, and
// NS k-steps in LDS give the direct loads NS - 2 phases to land.  A k-step takes 0.13 us
// against 0.28 on the three- and four-stage 64x32 tiles of nt_gemm.hip and 0.4 on the 64x128
// phased tile with one workgroup a CU.  Measured (us, nt_gemm.hip's tile / this): a step's
// projections at 128 rows, 1536x512 with a folded LayerNorm 6.4 / 5.1, 512x512 4.6 / 4.1,
// 512x2048 9.9 / 7.4, 1024x4096 17.1 / 11.9.  Six k-steps (72 KB, two workgroups a CU): eight and
// ten are no faster alone and slower from 256 tiles on (300x3072x1024 9.2, 12.5, 12.9), where
// the second workgroup has to wait.
#define NT_S2(RB0, RB1, RB2, RB3, LD)                                                               \
  "ds_read_b128 %[na0], %[pa0]\n\tds_read_b128 %[na1], %[pa1]\n\t"                                 \
  NT_MM("c0", "b00", "a0") RB0 RB1 NT_MM("c1", "b10", "a0") RB2 RB3                                 \
  LD NT_MM("c0", "b01", "a1") NT_MM("c1", "b11", "a1")
#define NT_S_LD3                                                                                    \
  "s_mov_b32 m0, %[ma]\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %[xa0], %[sa]\n\t"                    \
  "s_add_u32 m0, %[ma], 0x400\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %[xa1], %[sa]\n\t"             \
  "s_mov_b32 m0, %[mb]\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %[xb], %[sb]\n\t"
template <typename T, int FN> struct SlimPhase;
#define NT_SLIM_STRUCT(TYPE)                                                                        \
  template <> struct SlimPhase<TYPE, 2> {                                                             \
    template <int OB, int VM>                                                                       \
    static __device__ __forceinline__ void step(floatx4 (&c)[1][2], const u32x4 (&a)[2],            \
                                                const u32x4 (&b)[2][2], u32x4 (&na)[2],             \
                                                u32x4 (&nb)[2][2], unsigned pa0, unsigned pa1,      \
                                                unsigned pb0, unsigned pb1, const unsigned* xa,     \
                                                const char* sa, unsigned ma, const unsigned* xb,    \
                                                const char* sb, unsigned mb) {                      \
      asm volatile(NT_S2("ds_read_b128 %[nb00], %[pb0] offset:%[o0]\n\t",                           \
                         "ds_read_b128 %[nb01], %[pb1] offset:%[o0]\n\t",                           \
                         "ds_read_b128 %[nb10], %[pb0] offset:%[o1]\n\t",                           \
                         "ds_read_b128 %[nb11], %[pb1] offset:%[o1]\n\t", NT_S_LD3) NT_END          \
                   : [c0] "+v"(c[0][0]), [c1] "+v"(c[0][1]), [na0] "=&v"(na[0]), [na1] "=&v"(na[1]), \
                     [nb00] "=&v"(nb[0][0]), [nb01] "=&v"(nb[0][1]), [nb10] "=&v"(nb[1][0]),        \
                     [nb11] "=&v"(nb[1][1])                                                         \
                   : [a0] "v"(a[0]), [a1] "v"(a[1]), [b00] "v"(b[0][0]), [b01] "v"(b[0][1]),        \
                     [b10] "v"(b[1][0]), [b11] "v"(b[1][1]), [pa0] "v"(pa0), [pa1] "v"(pa1),        \
                     [pb0] "v"(pb0), [pb1] "v"(pb1), [o0] "i"(OB), [o1] "i"(OB + 16 * ROWB),        \
                     [xa0] "v"(xa[0]), [xa1] "v"(xa[1]), [sa] "s"(sa), [ma] "s"(ma), [xb] "v"(xb[0]), \
                     [sb] "s"(sb), [mb] "s"(mb), [vm] "i"(VM)                                       \
                   : "memory", "m0", "scc");                                                        \
    }                                                                                               \
  };
#define NT_MFMA_T "f16"
NT_SLIM_STRUCT(f16)
#undef NT_MFMA_T
#define NT_MFMA_T "bf16"
NT_SLIM_STRUCT(bf16)
#undef NT_MFMA_T

// fp32: a 16-byte chunk is four MFMAs a block, its words named one by one; they go round the two
// blocks, so that an MFMA does not wait for the one before it.
#define NT_FM(c, b, a) "v_mfma_f32_16x16x4_f32 %[" c "], %[" b "], %[" a "], %[" c "]\n\t"
#define NT_F2(h, w) NT_FM("c0", "p" h w, "a" h w) NT_FM("c1", "q" h w, "a" h w)
#define NT_WORDS(n, v) [n##0] "v"(v.x), [n##1] "v"(v.y), [n##2] "v"(v.z), [n##3] "v"(v.w)
template <> struct SlimPhase<float, 2> {
  template <int OB, int VM>
  static __device__ __forceinline__ void step(floatx4 (&c)[1][2], const u32x4 (&a)[2], const u32x4 (&b)[2][2],
                                              u32x4 (&na)[2], u32x4 (&nb)[2][2], unsigned pa0, unsigned pa1,
                                              unsigned pb0, unsigned pb1, const unsigned* xa, const char* sa,
                                              unsigned ma, const unsigned* xb, const char* sb, unsigned mb) {
    asm volatile("ds_read_b128 %[na0], %[r0]\n\tds_read_b128 %[na1], %[r1]\n\t"
                 NT_F2("0", "0") "ds_read_b128 %[nb00], %[t0] offset:%[o0]\n\t"
                 "ds_read_b128 %[nb01], %[t1] offset:%[o0]\n\t"
                 NT_F2("0", "1") "ds_read_b128 %[nb10], %[t0] offset:%[o1]\n\t"
                 "ds_read_b128 %[nb11], %[t1] offset:%[o1]\n\t"
                 NT_F2("0", "2") NT_S_LD3 NT_F2("0", "3")
                 NT_F2("1", "0") NT_F2("1", "1") NT_F2("1", "2") NT_F2("1", "3") NT_END
                 : [c0] "+v"(c[0][0]), [c1] "+v"(c[0][1]), [na0] "=&v"(na[0]), [na1] "=&v"(na[1]),
                   [nb00] "=&v"(nb[0][0]), [nb01] "=&v"(nb[0][1]), [nb10] "=&v"(nb[1][0]), [nb11] "=&v"(nb[1][1])
                 : NT_WORDS(a0, a[0]), NT_WORDS(a1, a[1]), NT_WORDS(p0, b[0][0]), NT_WORDS(p1, b[0][1]),
                   NT_WORDS(q0, b[1][0]), NT_WORDS(q1, b[1][1]), [r0] "v"(pa0), [r1] "v"(pa1), [t0] "v"(pb0),
                   [t1] "v"(pb1), [o0] "i"(OB), [o1] "i"(OB + 16 * ROWB), [xa0] "v"(xa[0]), [xa1] "v"(xa[1]),
                   [sa] "s"(sa), [ma] "s"(ma), [xb] "v"(xb[0]), [sb] "s"(sb), [mb] "s"(mb), [vm] "i"(VM)
                 : "memory", "m0", "scc");
  }
};
// The same on four blocks of columns.
#define NT_F4(h, w)                                                                                 \
  NT_FM("c0", "p" h w, "a" h w) NT_FM("c1", "q" h w, "a" h w)                                       \
  NT_FM("c2", "u" h w, "a" h w) NT_FM("c3", "w" h w, "a" h w)
template <> struct SlimPhase<float, 4> {
  template <int OB, int VM>
  static __device__ __forceinline__ void step(floatx4 (&c)[1][4], const u32x4 (&a)[2], const u32x4 (&b)[4][2],
                                              u32x4 (&na)[2], u32x4 (&nb)[4][2], unsigned pa0, unsigned pa1,
                                              unsigned pb0, unsigned pb1, const unsigned* xa, const char* sa,
                                              unsigned ma, const unsigned* xb, const char* sb, unsigned mb) {
    asm volatile("ds_read_b128 %[na0], %[r0]\n\tds_read_b128 %[na1], %[r1]\n\t"
                 NT_F4("0", "0") "ds_read_b128 %[nb00], %[t0] offset:%[o0]\n\t"
                 "ds_read_b128 %[nb01], %[t1] offset:%[o0]\n\t"
                 NT_F4("0", "1") "ds_read_b128 %[nb10], %[t0] offset:%[o1]\n\t"
                 "ds_read_b128 %[nb11], %[t1] offset:%[o1]\n\t"
                 NT_F4("0", "2") "ds_read_b128 %[nb20], %[t0] offset:%[o2]\n\t"
                 "ds_read_b128 %[nb21], %[t1] offset:%[o2]\n\t"
                 NT_F4("0", "3") "ds_read_b128 %[nb30], %[t0] offset:%[o3]\n\t"
                 "ds_read_b128 %[nb31], %[t1] offset:%[o3]\n\t"
                 NT_F4("1", "0") NT_S_LD3 "s_add_u32 m0, %[mb], 0x400\n\ts_nop 0\n\t"
                 "global_load_lds_dwordx4 %[xb1], %[sb]\n\t"
                 NT_F4("1", "1") NT_F4("1", "2") NT_F4("1", "3") NT_END
                 : [c0] "+v"(c[0][0]), [c1] "+v"(c[0][1]), [c2] "+v"(c[0][2]), [c3] "+v"(c[0][3]),
                   [na0] "=&v"(na[0]), [na1] "=&v"(na[1]), [nb00] "=&v"(nb[0][0]), [nb01] "=&v"(nb[0][1]),
                   [nb10] "=&v"(nb[1][0]), [nb11] "=&v"(nb[1][1]), [nb20] "=&v"(nb[2][0]), [nb21] "=&v"(nb[2][1]),
                   [nb30] "=&v"(nb[3][0]), [nb31] "=&v"(nb[3][1])
                 : NT_WORDS(a0, a[0]), NT_WORDS(a1, a[1]), NT_WORDS(p0, b[0][0]), NT_WORDS(p1, b[0][1]),
                   NT_WORDS(q0, b[1][0]), NT_WORDS(q1, b[1][1]), NT_WORDS(u0, b[2][0]), NT_WORDS(u1, b[2][1]),
                   NT_WORDS(w0, b[3][0]), NT_WORDS(w1, b[3][1]), [r0] "v"(pa0), [r1] "v"(pa1), [t0] "v"(pb0),
                   [t1] "v"(pb1), [o0] "i"(OB), [o1] "i"(OB + 16 * ROWB), [o2] "i"(OB + 32 * ROWB),
                   [o3] "i"(OB + 48 * ROWB), [xa0] "v"(xa[0]), [xa1] "v"(xa[1]), [sa] "s"(sa), [ma] "s"(ma),
                   [xb] "v"(xb[0]), [xb1] "v"(xb[1]), [sb] "s"(sb), [mb] "s"(mb), [vm] "i"(VM)
                 : "memory", "m0", "scc");
  }
};


template <typename T, int FN, int NS, int ROLE, bool LNF>
__global__ __launch_bounds__(256) void gemm_slim_kernel(const T* __restrict__ A, int lda, const void* __restrict__ Bt,
                                                        int M, int N, int K, GemmEpi epi, int tiles_m, int tiles_n) {
  constexpr int BM = 64, BN = 16 * FN, LB = BN / 32;   // LB: direct loads of B per wave and k-step
  constexpr int AB = BM * ROWB, BB = BN * ROWB, SLOT = AB + BB;
  __shared__ __attribute__((aligned(1024))) unsigned char lds[NS * SLOT];

  // every argument the k-loop needs in one round of scalar loads
  asm volatile("" ::"s"(epi.ctl), "s"(epi.bias), "s"(epi.out), "s"(epi.ldc), "s"(epi.mode), "s"(epi.resid),
               "s"(epi.lnf_colsum), "s"(epi.sent_list), "s"(epi.beam), "s"(epi.ctl_rows), "s"(A), "s"(lda), "s"(K),
               "s"(N), "s"(M), "s"(Bt), "s"(tiles_n));
  // A decoder step's tiles do not depend on how many rows are live (the grid's y is the tile row),
  // so their first loads are under way before the count is known; rows past the live ones are rows
  // of the same buffers.  An XCD owns a panel of columns where they divide evenly among the eight.
  // Otherwise tiles go round the XCDs as they come: panels of ceil(tiles_n / 8) would leave some
  // idle (with a folded LayerNorm, times those of nt_gemm.hip's 64x32 tile: 2160x384x128, on six
  // XCDs, 1.24 with panels and 0.89 without, 3500x128x128, on four, 1.09 and 0.86, 800x1152x384
  // 1.10 and 0.83).
  int tm, tn, n_live = 0, t_slot = 0;
  if constexpr (ROLE == 1) {
    const int* ctl = epi.ctl ? epi.ctl : reinterpret_cast<const int*>(A);   // (no branch to wait in)
    n_live = scalar_int(ctl + CTL_NLIVE);
    t_slot = scalar_int(ctl + CTL_T);
    tm = blockIdx.y;
    tn = tiles_n % 8 ? blockIdx.x : blockIdx.x % 8 * (tiles_n / 8) + blockIdx.x / 8;
  } else {
    // XCD-contiguous, then grouped by 8 tile-rows
    const int ntiles = tiles_m * tiles_n;
    int pid = blockIdx.x;
    const int q = ntiles / 8, r = ntiles % 8, xcd = pid % 8, idx = pid / 8;
    pid = xcd < r ? xcd * (q + 1) + idx : r * (q + 1) + (xcd - r) * q + idx;
    constexpr int GROUP = 8;
    const int per_group = GROUP * tiles_n;
    const int first_m = (pid / per_group) * GROUP;
    const int gsize = min(tiles_m - first_m, GROUP);
    tm = first_m + (pid % per_group) % gsize;
    tn = (pid % per_group) / gsize;
  }
  const int m0 = tm * BM, n0 = tn * BN;

  const int lane = threadIdx.x % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int fr = lane & 15, fc = lane >> 4;

  // direct loads: 8 rows of 128 bytes each
  const unsigned lda_b = (unsigned)lda * sizeof(T), ldb_b = (unsigned)K * sizeof(T);
  const unsigned ch = ((lane & 7) ^ (lane >> 3)) << 4;
  unsigned xa[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) xa[i] = (unsigned)min(m0 + (wave * 2 + i) * 8 + (lane >> 3), M - 1) * lda_b + ch;
  unsigned xb[LB];
#pragma unroll
  for (int i = 0; i < LB; ++i) xb[i] = (unsigned)min(n0 + (wave * LB + i) * 8 + (lane >> 3), N - 1) * ldb_b + ch;
  const char* Ab = reinterpret_cast<const char*>(A);
  const char* Bb = static_cast<const char*>(Bt);
  const unsigned lb = (unsigned)(uintptr_t)NT_LDS(lds);
  const unsigned ma = lb + wave * 2048, mb = lb + AB + wave * (LB * 1024);
  // lane addresses of the fragments in slot 0; the halves of a k-step differ in one bit
  const unsigned pa = lb + (wave * 16 + fr) * ROWB + ((fc ^ (fr & 7)) << 4);
  const unsigned pb = lb + AB + fr * ROWB + ((fc ^ (fr & 7)) << 4);

  const int nk = (int)((size_t)K * sizeof(T) / ROWB);
  auto fill = [&](int kt) {   // past the last k-step: its bytes again, never read
    const size_t at = (size_t)min(kt, nk - 1) * ROWB;
#pragma unroll
    for (int i = 0; i < 2; ++i) dma16(Ab + at + xa[i], lds + kt * SLOT + wave * 2048 + i * 1024);
#pragma unroll
    for (int i = 0; i < LB; ++i) dma16(Bb + at + xb[i], lds + kt * SLOT + AB + (wave * LB + i) * 1024);
  };
  fill(0);
  fill(1);
  int live = M;
  if constexpr (ROLE == 1) {
    asm volatile("" : "+s"(n_live), "+s"(t_slot));
    if (epi.ctl) live = min(M, n_live * epi.ctl_rows);
    else t_slot = epi.t;
    if (m0 >= live) {   // no load into LDS outlives the workgroup
      wait_vm<0>();
      return;
    }
  }
  EpiAhead<FN> ahead{};
  ahead.on = epi_whole<T, false, LNF>(epi, n0, BN, N);
  // (64x64 tiles have a second workgroup's k-loop to cover the epilogue's loads: 4096x512x512 in
  // fp32 takes 21.6 us with them here, 21.3 behind the loop)
  if (FN == 2 && ahead.on) epi_ahead<T, FN, ROLE, LNF>(ahead, epi, M, m0 + wave * 16, n0, fr, fc);
#pragma unroll
  for (int kt = 2; kt < NS; ++kt) fill(kt);
  floatx4 acc[1][FN];
#pragma unroll
  for (int j = 0; j < FN; ++j) acc[0][j] = floatx4{0.f, 0.f, 0.f, 0.f};
  constexpr int VM = (NS - 2) * (2 + LB);   // the loads behind the k-step after the next
  wait_vm<VM>();
  __builtin_amdgcn_s_barrier();
  u32x4 a0[2], a1[2], b0[FN][2], b1[FN][2];
  {
    u32x4 t[1][2];
    lds_frags<0>(t, pa, pa ^ 64);
    a0[0] = t[0][0];
    a0[1] = t[0][1];
    lds_frags<0>(b0, pb, pb ^ 64);
  }
  __builtin_amdgcn_s_barrier();
  float ls = 0.f, lq = 0.f;
  T sh{};
  if constexpr (LNF) sh = first_value<T>(__shfl(a0[0].x, fr, kWave));

  unsigned s0 = 0, s1 = SLOT;   // slots of this k-step and the next
  auto kstep = [&](int kt, u32x4 (&a)[2], u32x4 (&b)[FN][2], u32x4 (&na)[2], u32x4 (&nb)[FN][2]) {
    const size_t at = (size_t)min(kt + NS, nk - 1) * ROWB;
    const unsigned qa = pa + s1, qb = pb + s1;
    SlimPhase<T, FN>::template step<0, VM>(acc, a, b, na, nb, qa, qa ^ 64, qb, qb ^ 64, xa, Ab + at, uniform(ma + s0), xb,
                                       Bb + at, uniform(mb + s0));
    if constexpr (LNF) {
      frag_stats<T>(a[0], sh, ls, lq);
      frag_stats<T>(a[1], sh, ls, lq);
    }
    s0 = s1;
    s1 = s1 == (NS - 1) * SLOT ? 0 : s1 + SLOT;
  };
  for (int kt = 0;;) {
    kstep(kt, a0, b0, a1, b1);
    if (++kt >= nk) break;
    kstep(kt, a1, b1, a0, b0);
    if (++kt >= nk) break;
  }
  mfma_drain(acc);
  if (FN != 2 && ahead.on) epi_ahead<T, FN, ROLE, LNF>(ahead, epi, M, m0 + wave * 16, n0, fr, fc);
  float mu[1] = {0.f}, rs[1] = {1.f};
  if constexpr (LNF) {   // every lane of a row ends with its sums
    const float inv_k = 1.0f / (float)K;
    ls += __shfl_xor(ls, 16, kWave);
    lq += __shfl_xor(lq, 16, kWave);
    ls += __shfl_xor(ls, 32, kWave);
    lq += __shfl_xor(lq, 32, kWave);
    const float ms = ls * inv_k;
    const float var = fmaxf(lq * inv_k - ms * ms, 0.f);
    mu[0] = to_f32(sh) + ms;
    rs[0] = 1.0f / sqrtf(var + epi.lnf_eps);
  }
  phased_epilogue<T, 1, FN, ROLE, false, LNF>(acc, epi, live, N, m0 + wave * 16, n0, t_slot, fr, fc, mu, rs, nullptr,
                                              nullptr, nullptr, ahead);
  wait_vm<0>();   // no load into LDS outlives the workgroup
}

template <typename T, int FN, int NS, int ROLE, bool LNF>
hipError_t launch_slim(const void* A, int lda, const void* Bt, int M, int N, int K, const GemmEpi& epi, hipStream_t s) {
  const int tm = (M + 63) / 64, tn = (N + 16 * FN - 1) / (16 * FN);
  const dim3 grid = ROLE == 1 ? dim3(tn, tm) : dim3(tm * tn);
  NT_LAUNCH((gemm_slim_kernel<T, FN, NS, ROLE, LNF>), grid, dim3(256), 0, s, static_cast<const T*>(A), lda, Bt, M, N,
            K, epi, tm, tn);
  return hipGetLastError();
}

template <typename T, typename W, int ROLE, bool F8, bool LNF>
hipError_t launch_phased(const void* A, int lda, const void* Bt, int M, int N, int K, const GemmEpi& epi,
                         hipStream_t s) {
  constexpr int BM = W::WGM * W::FMH * 32, BN = W::WGN * W::FNH * 32;
  const int tm = (M + BM - 1) / BM, tn = (N + BN - 1) / BN;
  NT_LAUNCH((gemm_phased_kernel<T, W, ROLE, F8, LNF>), dim3(tm * tn), dim3(W::WGM * W::WGN * kWave), 0, s,
            static_cast<const T*>(A), lda, Bt, M, N, K, epi, tm, tn);
  return hipGetLastError();
}

template <typename T, int ROLE, bool LNF>
hipError_t launch_tile(const void* A, int lda, const void* Bt, int M, int N, int K, const GemmEpi& epi, hipStream_t s,
                       int bm) {
  if constexpr (ROLE == 2) {
    return launch_phased<T, TileSel, 2, false, false>(A, lda, Bt, M, N, K, epi, s);
  } else {
    if constexpr (std::is_same<T, f16>::value)
      if (epi.wscale) return launch_phased<T, Tile128, ROLE, true, LNF>(A, lda, Bt, M, N, K, epi, s);
    if (bm == 32) return launch_slim<T, 2, 6, ROLE, LNF>(A, lda, Bt, M, N, K, epi, s);
    if (bm == 64) return launch_phased<T, Tile64, ROLE, false, LNF>(A, lda, Bt, M, N, K, epi, s);
    if constexpr (ROLE == 0)
      if (bm == 256) return launch_phased<T, Tile256, ROLE, false, false>(A, lda, Bt, M, N, K, epi, s);
    return launch_phased<T, Tile128, ROLE, false, LNF>(A, lda, Bt, M, N, K, epi, s);
  }
}

template <typename T>
hipError_t launch_roles(const void* A, int lda, const void* Bt, int M, int N, int K, const GemmEpi& epi,
                        hipStream_t s, int role, int bm) {
  if (epi.lnf_colsum) return role == 1 ? launch_tile<T, 1, true>(A, lda, Bt, M, N, K, epi, s, bm) : hipErrorInvalidValue;
  switch (role) {
    case 1: return launch_tile<T, 1, false>(A, lda, Bt, M, N, K, epi, s, bm);
    case 2: return epi.wscale ? hipErrorInvalidValue : launch_tile<T, 2, false>(A, lda, Bt, M, N, K, epi, s, bm);
    default: return launch_tile<T, 0, false>(A, lda, Bt, M, N, K, epi, s, bm);
  }
}

}  // namespace
}  // namespace nt
