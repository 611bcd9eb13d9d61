// Device helpers shared by the kernel files (spear_kernels.hip, spear_gemm.hip,
// spear_mid.hip):
// MFMA wrappers, code unpacking, bounds-checked buffer accesses, coherent
// cross-workgroup reads.
//
// MFMA operand convention (v_mfma_f32_16x16x32_{f16,bf16}, wave64): lane l
// supplies row (l % 16) of the A operand and column (l % 16) of the B operand,
// each as 8 consecutive K positions of K-block (l / 16); the 16x16 fp32 result
// gives lane l the column (l % 16) and rows 4*(l/16) .. 4*(l/16)+3. Any
// permutation of the K positions is harmless as long as both operands use it.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <type_traits>

#include "spear_internal.h"

// A kernel file is compiled once per weight-code width (SPEAR_WB: 4 or 3) and
// activation dtype (SPEAR_BF16_UNIT: fp16 or bf16); its launchers carry both in
// their names (launch_gemv_w4_f16, ...). Kernels that do not read the codes
// are compiled with the 4-bit unit only and carry the dtype (launch_ec_f16).
#ifndef SPEAR_WB
#define SPEAR_WB 4
#endif
#ifndef SPEAR_BF16_UNIT
#define SPEAR_BF16_UNIT 0
#endif
#if SPEAR_BF16_UNIT
#define SPEAR_DT_SUFFIX _bf16
#else
#define SPEAR_DT_SUFFIX _f16
#endif
#define SPEAR_CAT2(a, b) a##b
#define SPEAR_CAT(a, b) SPEAR_CAT2(a, b)
#define SPEAR_D(name) SPEAR_CAT(name, SPEAR_DT_SUFFIX)
#define SPEAR_W(name) SPEAR_D(SPEAR_CAT(name, SPEAR_CAT(_w, SPEAR_WB)))

namespace spear {

// this unit's activation dtype
constexpr int DTC = SPEAR_BF16_UNIT ? DT_BF16 : DT_F16;

typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x3 __attribute__((ext_vector_type(3)));

// ---------------------------------------------------------------------------
// small helpers
// ---------------------------------------------------------------------------

template <int DT>
__device__ __forceinline__ f32x4 mfma16(u32x4 a, u32x4 b, f32x4 c) {
  if constexpr (DT == DT_F16)
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a),
                                                  __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
  else
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a),
                                                   __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// 32 x 32 x 16 MFMA: lane l holds A row l % 32 and B column l % 32, each at
// K 8 (l / 32) .. +8; result element i of lane l is D[8 (i / 4) + 4 (l / 32)
// + i % 4][l % 32]
typedef float f32x16 __attribute__((ext_vector_type(16)));
template <int DT>
__device__ __forceinline__ f32x16 mfma32(u32x4 a, u32x4 b, f32x16 c) {
  if constexpr (DT == DT_F16)
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a),
                                                  __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
  else
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a),
                                                   __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

template <int DT>
__device__ __forceinline__ float act2f(uint32_t bits16) {
  if constexpr (DT == DT_F16)
    return (float)__builtin_bit_cast(_Float16, (uint16_t)bits16);
  else
    return __uint_as_float(bits16 << 16);
}

// Round-to-nearest-even conversion to the activation dtype.
template <int DT>
__device__ __forceinline__ uint16_t f2act(float f) {
  if constexpr (DT == DT_F16)
    return __builtin_bit_cast(uint16_t, (_Float16)f);
  else
    return __builtin_bit_cast(uint16_t, (__bf16)f);
}

// two fp32 values, rounded to nearest even, as a bf16 pair (one instruction)
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{a, b}, bf16x2));
}

__device__ __forceinline__ float h2f(uint16_t b) { return (float)__builtin_bit_cast(_Float16, b); }

// Codes of one packed word as biased act-dtype values, paired (q0,q4),
// (q1,q5), (q2,q6), (q3,q7). OR-ing a 4-bit code into the mantissa of
// 1024.0 (fp16 0x6400) or 128.0 (bf16 0x4300) gives exactly 1024+q / 128+q.
template <int DT>
__device__ __forceinline__ u32x4 unpack_biased(uint32_t w) {
  constexpr uint32_t kMag = DT == DT_F16 ? 0x64006400u : 0x43004300u;
  u32x4 r;
  r[0] = (w & 0x000F000Fu) | kMag;
  r[1] = ((w >> 4) & 0x000F000Fu) | kMag;
  r[2] = ((w >> 8) & 0x000F000Fu) | kMag;
  r[3] = ((w >> 12) & 0x000F000Fu) | kMag;
  return r;
}
// Same, with the mask and the magic number in registers (`km` = 0x000F000F,
// `kg` = the magic pair): each code pair is then one v_and_or_b32 (plus a
// shift), which the literal-constant form above does not compile to.
__device__ __forceinline__ u32x4 unpack_biased_r(uint32_t w, uint32_t km, uint32_t kg) {
  u32x4 r;
  r[0] = (w & km) | kg;
  r[1] = ((w >> 4) & km) | kg;
  r[2] = ((w >> 8) & km) | kg;
  r[3] = ((w >> 12) & km) | kg;
  return r;
}
// 3-bit codes: a block of 32 codes c_0..c_31 in three words (w[0], w[1]:
// two-bit low fields, c_{2i} in bits 2i..2i+1 and c_{2i+1} in bits
// 16+2i..17+2i of w[0] for i < 8, of w[1] for i >= 8; w[2]: the high bits,
// c_{2i} at bit i and c_{2i+1} at bit 16+i). Pair p = (c_{2p}, c_{2p+1}),
// in natural K order, as two 16-bit lanes; `kg` = 0 gives the codes
// themselves, the magic pair (above) the biased act-dtype values.
__device__ __forceinline__ uint32_t w3_pair(const u32x4& w, int p, uint32_t kg) {
  const uint32_t lo = p < 8 ? w[0] : w[1];
  const uint32_t l = (lo >> (2 * (p & 7))) & 0x00030003u;
  const uint32_t h = (p >= 2 ? (w[2] >> (p - 2)) : (w[2] << (2 - p))) & 0x00040004u;
  return l | h | kg;
}
// MFMA operand jj (codes 8 jj .. 8 jj + 7 of the block, natural order) as
// biased act-dtype values
__device__ __forceinline__ u32x4 unpack3_biased(const u32x4& w, int jj, uint32_t kg) {
  return u32x4{w3_pair(w, 4 * jj, kg), w3_pair(w, 4 * jj + 1, kg), w3_pair(w, 4 * jj + 2, kg),
               w3_pair(w, 4 * jj + 3, kg)};
}
// Bytes of one row of packed codes.
template <int WB>
__host__ __device__ __forceinline__ uint32_t row_code_bytes(int K) {
  return WB == 4 ? (uint32_t)K / 2 : (uint32_t)K / 8 * 3;
}

// Opaque copy of a constant in a VGPR (the compiler cannot fold it back into
// an instruction literal).
__device__ __forceinline__ uint32_t opaque_v(uint32_t c) {
  asm volatile("" : "+v"(c));
  return c;
}
template <int DT>
__device__ __forceinline__ constexpr float code_bias() { return DT == DT_F16 ? 1024.f : 128.f; }

// Reorder 8 consecutive activations (x0..x7) into the pairing above.
__device__ __forceinline__ u32x4 pair_like_codes(u32x4 x) {
  u32x4 r;
  r[0] = (x[0] & 0xFFFFu) | (x[2] << 16);
  r[1] = (x[0] >> 16) | (x[2] & 0xFFFF0000u);
  r[2] = (x[1] & 0xFFFFu) | (x[3] << 16);
  r[3] = (x[1] >> 16) | (x[3] & 0xFFFF0000u);
  return r;
}

template <int DT>
__device__ __forceinline__ u32x4 ones8() {
  constexpr uint32_t o = DT == DT_F16 ? 0x3C003C00u : 0x3F803F80u;
  return u32x4{o, o, o, o};
}

__device__ __forceinline__ u32x4 ldg16(const void* p) { return *(const u32x4*)p; }

// INT8 per-channel symmetric codes (the EC factors' deployment format):
// code q of channel c stands for sa[c] * q. Where a code feeds an MFMA it is
// dequantised to the activation dtype like the 4-bit weights, one rounding
// of the fp32 product s * q (exact for |q| <= 127). Bytes 2p and 2p + 1 of w.
template <int DT>
__device__ __forceinline__ uint32_t i8pair_to_act(uint32_t w, int p, float s) {
  const int b0 = (int)(w << (24 - 16 * p)) >> 24;
  const int b1 = (int)(w << (16 - 16 * p)) >> 24;
  return (uint32_t)f2act<DT>((float)b0 * s) | ((uint32_t)f2act<DT>((float)b1 * s) << 16);
}
// eight codes (two dwords, K order) -> an 8-element MFMA operand
template <int DT>
__device__ __forceinline__ u32x4 i8x8_to_act(uint32_t w0, uint32_t w1, float s) {
  return u32x4{i8pair_to_act<DT>(w0, 0, s), i8pair_to_act<DT>(w0, 1, s),
               i8pair_to_act<DT>(w1, 0, s), i8pair_to_act<DT>(w1, 1, s)};
}
template <int DT>
__device__ __forceinline__ uint16_t i8_to_act(int8_t q, float s) {
  return f2act<DT>((float)q * s);
}
// Eight INT8 codes as exact activation-dtype integers (|q| <= 127 is exact
// in both), for kernels that apply the scale to the fp32 result instead.
// fp16: the byte q + 128 is placed under the exponent of 1024 (0x64 high
// byte gives 1024 + b exactly) and 1152 is subtracted; bf16: through fp32.
template <int DT>
__device__ __forceinline__ u32x4 i8x8_exact(uint32_t w0, uint32_t w1) {
  if constexpr (DT == DT_F16) {
    const uint32_t b0 = w0 ^ 0x80808080u, b1 = w1 ^ 0x80808080u;
    const f16x2 off = f16x2{(_Float16)-1152.f, (_Float16)-1152.f};
    auto pr = [&](uint32_t b, uint32_t sel) {
      return __builtin_bit_cast(uint32_t,
                                __builtin_bit_cast(f16x2, __builtin_amdgcn_perm(0x64646464u, b, sel)) + off);
    };
    return u32x4{pr(b0, 0x04010400u), pr(b0, 0x04030402u), pr(b1, 0x04010400u), pr(b1, 0x04030402u)};
  } else {
    auto pr = [&](uint32_t w, int p) {
      const float a0 = (float)((int)(w << (24 - 16 * p)) >> 24);
      const float a1 = (float)((int)(w << (16 - 16 * p)) >> 24);
      return (__float_as_uint(a0) >> 16) | (__float_as_uint(a1) & 0xFFFF0000u);
    };
    return u32x4{pr(w0, 0), pr(w0, 1), pr(w1, 0), pr(w1, 1)};
  }
}

// Raw buffer loads through a bounds-checked resource (gfx9 descriptor word 3
// = 0x00020000): a byte offset at or past `bytes` reads as zero. Masked
// elements are given the offset kOOB, so every load is issued without a
// branch and a wave's loads all stay in flight together.
typedef __amdgpu_buffer_rsrc_t rsrc_t;
constexpr uint32_t kOOB = 0x80000000u;
__device__ __forceinline__ rsrc_t make_rsrc(const void* p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, (int)bytes, 0x00020000);
}
__device__ __forceinline__ u32x4 bld128(rsrc_t r, uint32_t off) {
  return __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0);
}
// 16 bytes per lane from `r` at byte offset `off` straight into LDS: lane l
// of the wave writes lds + 16 l (lds wave-uniform, 1 KB per instruction);
// completion is counted by vmcnt
__device__ __forceinline__ void bld128_lds(rsrc_t r, void* lds, uint32_t off) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void*)lds, 16, off, 0, 0, 0);
}
// voffset (per lane, carries the mask) + soffset (wave-uniform)
__device__ __forceinline__ u32x4 bld128s(rsrc_t r, uint32_t voff, uint32_t soff) {
  return __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, 0);
}
// 12 bytes (one block of 3-bit codes) into the first three lanes of a u32x4
__device__ __forceinline__ u32x4 bld96s(rsrc_t r, uint32_t voff, uint32_t soff) {
  const u32x3 v = __builtin_amdgcn_raw_buffer_load_b96(r, voff, soff, 0);
  return u32x4{v[0], v[1], v[2], 0u};
}
__device__ __forceinline__ uint32_t bld16s(rsrc_t r, uint32_t voff, uint32_t soff) {
  return __builtin_amdgcn_raw_buffer_load_b16(r, voff, soff, 0);
}
__device__ __forceinline__ uint32_t bld8s(rsrc_t r, uint32_t voff, uint32_t soff) {
  return __builtin_amdgcn_raw_buffer_load_b8(r, voff, soff, 0);
}
__device__ __forceinline__ uint32_t bld16(rsrc_t r, uint32_t off) {
  return __builtin_amdgcn_raw_buffer_load_b16(r, off, 0, 0);
}
__device__ __forceinline__ uint32_t bld8(rsrc_t r, uint32_t off) {
  return __builtin_amdgcn_raw_buffer_load_b8(r, off, 0, 0);
}

__device__ __forceinline__ void bst16(rsrc_t r, uint32_t off, uint16_t v) {
  __builtin_amdgcn_raw_buffer_store_b16((short)v, r, off, 0, 0);
}

// The GEMMs' final store: CNT fp32 results of a lane at byte offsets off(i) of
// y (kOOB: not stored), the residual added before the rounding. The residual
// elements are all requested before the first is used, and neither loads nor
// stores branch: with a branch and a wait per element 8192 x 8192 at 4096 tokens
// took 578 us with a residual (fp16), 507 without; this way 526.
template <int DT, int CNT, class Off, class Val>
__device__ __forceinline__ void store_results(rsrc_t ry, rsrc_t rres, bool has_res, Off off, Val val) {
  if (has_res) {  // uniform
    uint32_t rv[CNT];
#pragma unroll
    for (int i = 0; i < CNT; ++i) rv[i] = bld16(rres, off(i));
#pragma unroll
    for (int i = 0; i < CNT; ++i) bst16(ry, off(i), f2act<DT>(val(i) + act2f<DT>(rv[i])));
  } else {
#pragma unroll
    for (int i = 0; i < CNT; ++i) bst16(ry, off(i), f2act<DT>(val(i)));
  }
}

// Cross-workgroup data (partial sums, the EC coordinates, flags, counters)
// moves only through relaxed agent-scope atomic accesses: on gfx950 these are
// plain loads/stores with the sc1 bit, coherent across the eight XCDs' L2s on
// every access, so no cache-wide writeback or invalidate is ever issued.
// Ordering comes from waiting for the stores to complete (s_waitcnt) before
// the barrier that precedes the publishing atomic.
__device__ __forceinline__ void st_agent(float* p, float v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float ld_agent(const float* p) {
  return __hip_atomic_load(const_cast<float*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint32_t ld_agent_u32(const uint32_t* p) {
  return __hip_atomic_load(const_cast<uint32_t*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// All of this thread's memory operations have completed; then the block meets.
// 16-byte agent-scope (sc1) buffer store and load
__device__ __forceinline__ void bst128c(rsrc_t r, uint32_t off, f32x4 v) {
  __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), r, off, 0, 0x10);
}
__device__ __forceinline__ f32x4 bld128cf(rsrc_t r, uint32_t off) {
  return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0x10));
}
__device__ __forceinline__ void complete_and_sync() {
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
}

// Last-arriver detection: one relaxed agent-scope fetch-add per arrival (no
// compare-and-swap retries, which serialise at one memory round trip each).
// The arrival that completes `total` resets the counter to zero, so every
// launch (also a replayed graph) starts from zero; the workspace holding the
// counters is zero-filled once before first use. Callers publish their data
// with st_agent and complete_and_sync() before arriving, and the last arriver
// reads it back with ld_agent.
__device__ __forceinline__ bool arrive_last(uint32_t* ctr, uint32_t total) {
  const uint32_t old = __hip_atomic_fetch_add(ctr, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (old + 1u != total) return false;
  __hip_atomic_store(ctr, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return true;
}

// ---------------------------------------------------------------------------
// Coherent reads of data other workgroups published in this launch: buffer
// loads with the sc1 bit (what a relaxed agent-scope atomic load is on
// gfx950), bounds-checked so that every load of a batch is issued without a
// branch. A thread's loads go out four at a time, all in flight together.
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint32_t bld32c(rsrc_t r, uint32_t off) {
  return __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0x10);
}
__device__ __forceinline__ u32x2 bld64(rsrc_t r, uint32_t off) {
  return __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0);
}
__device__ __forceinline__ u32x2 bld64c(rsrc_t r, uint32_t off) {
  return __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0x10);
}

// dst[i] = fp32 part of the tagged word (tag << 32 | fp32 bits) at off(i), i in
// [0, n); returns 1 if any word this thread read carries another tag.
template <class Off>
__device__ __forceinline__ int gather_tagged(rsrc_t r, int n, Off off, uint32_t tag, float* dst) {
  const int nthr = blockDim.x;
  int stale = 0;
  for (int i0 = threadIdx.x; i0 < n; i0 += 4 * nthr) {
    const int i1 = i0 + nthr, i2 = i1 + nthr, i3 = i2 + nthr;
    const u32x2 w0 = bld64c(r, off(i0));
    const u32x2 w1 = bld64c(r, i1 < n ? off(i1) : kOOB);
    const u32x2 w2 = bld64c(r, i2 < n ? off(i2) : kOOB);
    const u32x2 w3 = bld64c(r, i3 < n ? off(i3) : kOOB);
    stale |= w0[1] != tag;
    dst[i0] = __uint_as_float(w0[0]);
    if (i1 < n) { stale |= w1[1] != tag; dst[i1] = __uint_as_float(w1[0]); }
    if (i2 < n) { stale |= w2[1] != tag; dst[i2] = __uint_as_float(w2[0]); }
    if (i3 < n) { stale |= w3[1] != tag; dst[i3] = __uint_as_float(w3[0]); }
  }
  return stale;
}

// out(i, sum over q < P of the word at off(q, i)), i in [0, n), summed in
// slice order. The slices lie at the device coherence point, a memory round
// trip away, so each thread sums two elements at a time with U slices of
// both in flight and nothing goes through LDS (a staged copy of bounded size
// took six dependent round trips for a 16-token tile of rank 64 in eight
// slices: 1024 x 8192 at 16 tokens, producer-fused, 22.3 us against 19.3).
// U: eight where the slices are many (the EC projection's); four for the
// GEMV's few K-slices, where eight issued mostly loads past the last one (local
// variant, rank 16, bf16: 1024 x 4096 at two tokens staged 11.8 us, eight 12.0,
// four 11.3; 2048 x 8192 at 16 tokens 15.1, 14.5, 13.6).
// Every thread of the block calls it; it ends with a barrier.
template <int U = 8, class Off, class Out>
__device__ __forceinline__ void sum_slices(rsrc_t r, int P, int n, Off off, Out out) {
  const int nthr = blockDim.x;
  for (int i0 = threadIdx.x; i0 < n; i0 += 2 * nthr) {
    const int i1 = i0 + nthr;
    float a = 0.f, b = 0.f;
    for (int q0 = 0; q0 < P; q0 += U) {
      uint32_t wa[U], wb[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const bool ok = q0 + u < P;
        wa[u] = bld32c(r, ok ? off(q0 + u, i0) : kOOB);
        wb[u] = bld32c(r, ok && i1 < n ? off(q0 + u, i1) : kOOB);
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (q0 + u < P) {
          a += __uint_as_float(wa[u]);
          b += __uint_as_float(wb[u]);
        }
    }
    out(i0, a);
    if (i1 < n) out(i1, b);
  }
  __syncthreads();
}

// One layer of the rank-space gate's MLP, fp32: out(t, i, bias[i] + sum_j
// W[i][j] in[t][j]) for rows i and cnt tokens, by nthr threads (this one is
// tid). Latency bound: a few KB of parameters, a few thousand multiplies per
// token. So one thread takes one row for up to four tokens, reads the row
// with 16-byte loads (rows of a multiple of eight, 16-byte aligned), and the
// tokens' inputs, the same for every lane of a token group, come from LDS as
// broadcasts; each sum keeps its order over j. (One thread per row and token
// at a time, two bytes per load, one token after another, took the EC
// pre-kernel of the 8B layers, rank 32, h 128, at eight tokens to 105 us; this
// takes it to 15.)
template <int DT, class Out>
__device__ __forceinline__ void mlp_layer(int tid, int nthr, const uint16_t* W, const uint16_t* bias,
                                          int rows, int cols, const float* in, int is, int cnt, Out out) {
  const int tgs = (cnt + 3) >> 2;
  for (int idx = tid; idx < rows * tgs; idx += nthr) {
    const int tg = idx / rows, i = idx - tg * rows;
    const uint16_t* wr = W + (size_t)i * cols;
    const float b = act2f<DT>(bias[i]);
    const float *p0 = in + 4 * tg * is, *p1 = in + min(4 * tg + 1, cnt - 1) * is,
                *p2 = in + min(4 * tg + 2, cnt - 1) * is, *p3 = in + min(4 * tg + 3, cnt - 1) * is;
    f32x4 a = f32x4{b, b, b, b};
    int j = 0;
    if ((cols & 7) == 0) {
#pragma unroll 4
      for (; j < cols; j += 8) {
        const u32x4 w = *(const u32x4*)(wr + j);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float wf = act2f<DT>((w[e >> 1] >> (16 * (e & 1))) & 0xFFFFu);
          a[0] += wf * p0[j + e];
          a[1] += wf * p1[j + e];
          a[2] += wf * p2[j + e];
          a[3] += wf * p3[j + e];
        }
      }
    }
    for (; j < cols; ++j) {
      const float wf = act2f<DT>(wr[j]);
      a[0] += wf * p0[j];
      a[1] += wf * p1[j];
      a[2] += wf * p2[j];
      a[3] += wf * p3[j];
    }
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (4 * tg + q < cnt) out(4 * tg + q, i, a[q]);
  }
}

// The paper's rank-space gate for cnt tokens at once, by the whole block:
// hid = ReLU(W1 u + b1) for every token, then v = alpha (1 + tanh(W2 hid +
// b2)) (.) u, in fp32, cap tokens per pass (hid holds cap x h floats). u
// rows are us floats apart, v rows vs. Ends with a barrier.
template <int DT>
__device__ __forceinline__ void tanh_gate_tokens(int cnt, int r, int h, const float* u, int us,
                                 const uint16_t* W1, const uint16_t* b1, const uint16_t* W2,
                                 const uint16_t* b2, float alpha, float* hid, int cap, float* v,
                                 int vs) {
  const int tid = threadIdx.x, nthr = blockDim.x;
  for (int t0 = 0; t0 < cnt; t0 += cap) {
    const int c = min(cap, cnt - t0);
    const float* ut = u + t0 * us;
    mlp_layer<DT>(tid, nthr, W1, b1, h, r, ut, us, c,
                  [&](int t, int i, float a) { hid[t * h + i] = a > 0.f ? a : 0.f; });
    __syncthreads();
    mlp_layer<DT>(tid, nthr, W2, b2, r, h, hid, h, c, [&](int t, int j, float a) {
      v[(t0 + t) * vs + j] = alpha * (1.f + tanhf(a)) * ut[t * us + j];
    });
    __syncthreads();
  }
}

// NP pairs of raw codes (natural K order, one code per 16-bit lane) to
// dequantised act-dtype pairs: (q - z) exact, then one rounding of its
// product with s (fp16: the biased code minus 1024 + z, an exact integer, in
// packed half math; bf16: in fp32, then rounded).
template <int DT, int NP>
__device__ __forceinline__ void dequant_pairs(const uint32_t (&p)[NP], float s, int z,
                                              uint32_t (&out)[NP]) {
  if constexpr (DT == DT_F16) {
    const _Float16 zb = (_Float16)(1024 + z);
    const f16x2 nz = f16x2{-zb, -zb};
    const f16x2 s2 = f16x2{(_Float16)s, (_Float16)s};
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      const f16x2 q = __builtin_bit_cast(f16x2, p[i] | 0x64006400u);
      out[i] = __builtin_bit_cast(uint32_t, (q + nz) * s2);
    }
  } else {
    const float c = -(float)z * s;  // exact, and so is the fused multiply-add
#pragma unroll
    for (int i = 0; i < NP; ++i)
      out[i] = pack_bf16(__builtin_fmaf((float)(p[i] & 0xFFFFu), s, c), __builtin_fmaf((float)(p[i] >> 16), s, c));
  }
}

// One packed word of 4-bit codes as exact fp16 integers q - z in natural order:
// pairs (q0,q1), (q2,q3), (q4,q5), (q6,q7). Each byte, copied to both halves
// of a register, gives 1024 + q_even and 1024 + 16 q_odd by one mask-and-or
// (km 0x00F0000F, kg 0x64006400, in registers so that it is one
// instruction), and one fused multiply-add with (1, 1/16) and `cz` =
// exact_cz(z), exact, the integers: 12 instructions per word.
__device__ __forceinline__ uint32_t exact_cz(uint32_t z) {
  return 0xD400E400u + z * 0x00100001u;  // fp16 -(1024 + z) | -(64 + z) << 16
}
__device__ __forceinline__ u32x4 exact_word(uint32_t w, uint32_t km, uint32_t kg, uint32_t cz) {
  const f16x2 m = f16x2{(_Float16)1.f, (_Float16)0.0625f}, c = __builtin_bit_cast(f16x2, cz);
  u32x4 r;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const uint32_t t = (__builtin_amdgcn_perm(0u, w, 0x0C000C00u | (uint32_t)i * 0x00010001u) & km) | kg;
    r[i] = __builtin_bit_cast(uint32_t, __builtin_elementwise_fma(__builtin_bit_cast(f16x2, t), m, c));
  }
  return r;
}

// The same word as biased values (fp16 1024 + q, bf16 128 + q) in natural
// order, nine instructions (km 0x000F000F, kg the magic pair, in registers).
__device__ __forceinline__ u32x4 biased_word_nat(uint32_t w, uint32_t km, uint32_t kg) {
  const uint32_t hi = w >> 4;
  return u32x4{(__builtin_amdgcn_perm(hi, w, 0x0C040C00u) & km) | kg, (__builtin_amdgcn_perm(hi, w, 0x0C050C01u) & km) | kg,
               (__builtin_amdgcn_perm(hi, w, 0x0C060C02u) & km) | kg, (__builtin_amdgcn_perm(hi, w, 0x0C070C03u) & km) | kg};
}

// One packed word of 4-bit codes, dequantised in natural order: (q - z) exact,
// then one rounding of its product with s. fp16: 1024 + q, less 1024 + z, times
// s in packed half math: 19 instructions, and still the faster form beside the
// MFMAs of the large GEMMs, whose clock the power limit sets (with the exact
// integers by fused multiply-add, 16 instructions, 70B gate at 4096 tokens
// took 1716 us against 1660). bf16: q s - z s in one fp32 fused multiply-add
// (z s and the result are exact: at most 16 significant bits), then rounded.
template <int DT>
__device__ __forceinline__ void dequant_word_pairs(uint32_t w, float s, int z, uint32_t (&out)[4]) {
  const uint32_t lo = w & 0x0F0F0F0Fu, hi = (w >> 4) & 0x0F0F0F0Fu;  // q0 q2 q4 q6, q1 q3 q5 q7
  if constexpr (DT == DT_F16) {
    const uint32_t p[4] = {__builtin_amdgcn_perm(hi, lo, 0x0C040C00u), __builtin_amdgcn_perm(hi, lo, 0x0C050C01u),
                           __builtin_amdgcn_perm(hi, lo, 0x0C060C02u), __builtin_amdgcn_perm(hi, lo, 0x0C070C03u)};
    dequant_pairs<DT, 4>(p, s, z, out);
  } else {
    const float c = -(float)z * s;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float a0 = __builtin_fmaf((float)((lo >> (8 * i)) & 0xFFu), s, c);
      const float a1 = __builtin_fmaf((float)((hi >> (8 * i)) & 0xFFu), s, c);
      out[i] = pack_bf16(a0, a1);
    }
  }
}

// Pairs P0 .. P0 + NP - 1 of a block of 3-bit codes (three words in w),
// dequantised in natural order.
template <int DT, int P0, int NP>
__device__ __forceinline__ void dequant_block3_pairs(const u32x4& w, float s, int z,
                                                     uint32_t (&out)[NP]) {
  uint32_t p[NP];
#pragma unroll
  for (int i = 0; i < NP; ++i) p[i] = w3_pair(w, P0 + i, 0u);
  dequant_pairs<DT, NP>(p, s, z, out);
}

// Raise a kernel's dynamic-LDS limit when a launch needs more than 64 KB.
template <typename F>
static hipError_t allow_lds(F* fn, size_t lds) {
  if (lds <= 65536) return hipSuccess;
  return hipFuncSetAttribute((const void*)fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
}

}  // namespace spear
