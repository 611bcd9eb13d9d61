// gfx950 (MI355X) prefill kernels of the W4+EC linear layer (operand and layout
// conventions: spear_device.h):
//   k_dequant  bit-exact dequantisation diagnostic
//   k_gemm     LDS-tiled 4-bit GEMM (dequantised tiles, double buffered), MFMA
//              epilogue adding B v from the EC pre-kernel, or with the EC
//              projected by its own waves
//   k_gemm_ws  the same product with loading and multiplying waves
#include "spear_device.h"

namespace spear {

// ---------------------------------------------------------------------------
// Prefill GEMM: 128x128 output tile per block (tokens x rows), K staged 64 at
// a time through double-buffered LDS; the packed codes are dequantised once
// per block into the LDS tile, (q - z) exact then times s with one rounding
// (fp16) or via fp32 (bf16). Four waves, 2x2, each 64x64 = 4x4 MFMA tiles.
// ---------------------------------------------------------------------------
// ---------------------------------------------------------------------------
// Dequantisation diagnostic, by the code the prefill GEMM dequantises its
// weight tiles with ((q - z) exact, then one rounding of its product with s):
// one thread per packed word of 4-bit codes (eight outputs), or per block of
// 3-bit codes (three words, 32 outputs).
// ---------------------------------------------------------------------------
template <int DT, int WB>
__global__ __launch_bounds__(256) void k_dequant(const uint32_t* __restrict__ qw,
                                                 const uint16_t* __restrict__ sc,
                                                 const uint8_t* __restrict__ zr,
                                                 uint16_t* __restrict__ out, int N, int K, int G) {
  constexpr int CPU = WB == 4 ? 8 : 32;  // codes per unit (word or block)
  const int kw = K / CPU;
  const long long nunits = (long long)N * kw;
  const long long wi = (long long)blockIdx.x * 256 + threadIdx.x;
  if (wi >= nunits) return;
  const int n = (int)(wi / kw);
  const int k = (int)(wi % kw) * CPU;
  const int ng = K / G;
  const int g = k / G;
  const float s = h2f(sc[(long long)n * ng + g]);
  const int z = zr[(long long)n * ng + g];
  if constexpr (WB == 4) {
    uint32_t o[4];
    dequant_word_pairs<DT>(qw[wi], s, z, o);
    *(u32x4*)(out + (long long)n * K + k) = u32x4{o[0], o[1], o[2], o[3]};
  } else {
    const uint32_t* b = qw + 3 * wi;
    const u32x4 w = u32x4{b[0], b[1], b[2], 0u};
    uint32_t o[16];
    dequant_block3_pairs<DT, 0, 16>(w, s, z, o);
#pragma unroll
    for (int c = 0; c < 4; ++c)
      *(u32x4*)(out + (long long)n * K + k + 8 * c) = u32x4{o[4 * c], o[4 * c + 1], o[4 * c + 2], o[4 * c + 3]};
  }
}

// Split-K tile reduction of the GEMM: a thread's 16 f32x4 of the tile from
// each of the S slices, summed in slice order (slice 0 first, so the result
// does not depend on which slice arrives last). The slices' loads are issued
// in rounds of 32 (S/2 rounds), each round's loads all in flight together:
// the partials sit at the device coherence point, a memory round trip away,
// and one round per slice would pay that latency S times.
// base: byte offset of the thread's first f32x4 in slice 0; slice: bytes
// between slices; entry (i, j) is 1024 * (4i + j) bytes further.
template <int S>
__device__ __forceinline__ void gemm_sum_slices(rsrc_t rp, uint32_t base, uint32_t slice,
                                                f32x4 (&acc)[4][4]) {
  constexpr int E = 32 / S;  // entries per round
#pragma unroll
  for (int rd = 0; rd < S / 2; ++rd) {
    f32x4 pv[S][E];
#pragma unroll
    for (int q = 0; q < S; ++q)
#pragma unroll
      for (int e = 0; e < E; ++e) pv[q][e] = bld128cf(rp, base + q * slice + (rd * E + e) * 1024);
#pragma unroll
    for (int e = 0; e < E; ++e) {
      f32x4 t = pv[0][e];
#pragma unroll
      for (int q = 1; q < S; ++q) t += pv[q][e];
      acc[(rd * E + e) >> 2][(rd * E + e) & 3] = t;
    }
  }
}

// The same for the fully fused variant's EC accumulators: 4 f32x4 per
// thread per slice, all slices' loads in one round (S <= 8: 32 loads).
template <int S>
__device__ __forceinline__ void gemm_sum_ec_slices(rsrc_t rp, uint32_t base, uint32_t slice,
                                                   f32x4 (&eacc)[4]) {
  f32x4 pv[S][4];
#pragma unroll
  for (int q = 0; q < S; ++q)
#pragma unroll
    for (int i = 0; i < 4; ++i) pv[q][i] = bld128cf(rp, base + q * slice + i * 1024);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    f32x4 t = pv[0][i];
#pragma unroll
    for (int q = 1; q < S; ++q) t += pv[q][i];
    eacc[i] = t;
  }
}

// TMW: waves along the tokens. TMW = 2: 128-token tiles, 4 waves, two
// workgroups per CU; TMW = 4: 256-token tiles, 8 waves, one workgroup per
// CU. Both keep 64 x 64 per wave and two waves per SIMD; the 256-token tile
// reuses each dequantised weight tile for twice the MFMAs, halving the
// dequantisation's VALU work per MFMA.
template <int DT, int EPI, int TMW, int WB>
__global__ __launch_bounds__(128 * TMW, TMW == 2 ? 2 : 1) void k_gemm(GemmParams a) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  constexpr bool kLoc = EPI == EPI_LOCAL || EPI == EPI_LOCAL_I8;
  constexpr bool kI8 = EPI == EPI_LOCAL_I8;  // INT8 A and B
  constexpr int TM = 64 * TMW;         // tokens per tile
  constexpr int NT = 128 * TMW;        // threads
  constexpr int WPT = TMW == 2 ? 4 : 2;  // packed words of codes per thread and step
  constexpr int WPR = 8 / WPT;         // threads per row of codes
  constexpr int LR = kGemmLdsRow;
  constexpr int TILEX = TM * LR;       // halves per LDS activation tile
  constexpr int TILEW = kGemmTN * LR;  // halves per LDS weight tile
  constexpr int ETILE = kGemmEcRows * LR;
  uint16_t* Xs = (uint16_t*)smem;             // [2][TM][LR]
  uint16_t* Ws = Xs + 2 * TILEX;              // [2][128][LR]
  uint16_t* Es = Ws + 2 * TILEW;              // EPI_LOCAL: [2][17][LR] A rows, w_g
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int lr = lane & 15, lg = lane >> 4;
  const int wm = wave >> 1, wn = wave & 1;
  const int M = a.M, N = a.N, K = a.K;
  const int tiles_m = (M + TM - 1) / TM, tiles_n = (N + kGemmTN - 1) / kGemmTN;
  // Workgroups are dealt to the eight XCDs in turn (b % 8), and each XCD has
  // its own L2: give XCD x a contiguous band of token tiles (or, failing
  // that, of row tiles) so that the tiles its workgroups share are fetched
  // into its L2 once, instead of every activation tile once per XCD.
  // split-K: workgroup b of slice s is blockIdx.x = s * tiles + b
  const int T = tiles_m * tiles_n;
  const int ks = (int)blockIdx.x / T, tb = (int)blockIdx.x - ks * T;
  int mt_i, nt_i;
  {
    const int b = tb, x = b & 7, j = b >> 3;
    if ((tiles_m & 7) == 0) {
      const int pm = tiles_m >> 3;
      mt_i = x * pm + j % pm;
      nt_i = j / pm;
    } else if ((tiles_n & 7) == 0) {
      const int pn = tiles_n >> 3;
      nt_i = x * pn + j % pn;
      mt_i = j / pn;
    } else {
      mt_i = b / tiles_n;
      nt_i = b - mt_i * tiles_n;
    }
  }
  const int m0 = mt_i * TM;
  const int n0 = nt_i * kGemmTN;
  const int KT = K / kGemmTK / a.S;  // steps of this slice (an even count)
  const int kbase = ks * KT;

  // per-thread global load assignments (bounds-checked buffer loads)
  const rsrc_t rx = make_rsrc(a.x, (uint32_t)M * K * 2);
  const rsrc_t rq = make_rsrc(a.qw, (uint32_t)N * row_code_bytes<WB>(K));
  const rsrc_t rsc = make_rsrc(a.sc, (uint32_t)N * a.ngroups * 2);
  const rsrc_t rz = make_rsrc(a.zr, (uint32_t)N * a.ngroups);
  int xr[4], xc[4];
  uint32_t xoff[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int c = tid + NT * i;
    xr[i] = c >> 3;
    xc[i] = (c & 7) * 8;
    xoff[i] = m0 + xr[i] < M ? ((uint32_t)(m0 + xr[i]) * K + xc[i]) * 2 : kOOB;
  }
  // codes: row wr, K [8 WPT wp, +8 WPT) of the row's 64-wide step: 4-bit
  // words [wp WPT, +WPT); 3-bit: block wp (WPT = 4) or half wp % 2 of block
  // wp / 2 (WPT = 2), whose three words are loaded whole
  const int wr = tid / WPR, wp = tid % WPR;
  const int wn_row = n0 + wr;
  const bool wok = wn_row < N;
  const uint32_t woff = !wok      ? kOOB
                        : WB == 4 ? (uint32_t)wn_row * (K / 2) + 4 * WPT * wp
                                  : (uint32_t)wn_row * row_code_bytes<WB>(K) + 12 * (WPT == 4 ? wp : wp >> 1);
  // EPI_LOCAL: thread t < 136 stages 16 bytes of the EC tile per step: row
  // t / 8 (A's row while below r, zero up to 15; w_g as row 16), chunk t % 8
  const int er = tid >> 3, ec8 = tid & 7;
  // INT8 A: the chunk's eight codes (8 bytes), dequantised with row er's
  // scale when stored
  const rsrc_t ra = kI8 ? make_rsrc(a.A8, (uint32_t)a.r * K)
                        : make_rsrc(kLoc ? a.A : nullptr, kLoc ? (uint32_t)a.r * K * 2 : 0u);
  const rsrc_t rgw = make_rsrc(kLoc ? a.wg : nullptr,
                               kLoc && a.gate == GATE_SIGMOID ? (uint32_t)K * 2 : 0u);
  const uint32_t eoff = er < 16 && er < a.r ? ((uint32_t)er * K + 8 * ec8) * 2 : kOOB;
  float sa_er = 0.f;
  if constexpr (kI8) {
    const rsrc_t rsa = make_rsrc(a.sa, (uint32_t)a.r * 4);
    sa_er = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(
        rsa, er < 16 && er < a.r ? (uint32_t)er * 4 : kOOB, 0, 0));
  }
  const uint32_t goff = er == 16 ? 16u * ec8 : kOOB;

  // two register sets of global loads, so that the loads of step kt+2 are
  // in flight while step kt is computed. The scale and zero point stay raw
  // until the stage is stored: converting them at load time would make the
  // wave wait for every load issued before them (the vector-memory counter
  // retires in order).
  struct Stage {
    u32x4 x[4];
    u32x4 w;
    uint32_t s, z;
    u32x4 e, g;  // EPI_LOCAL: A / w_g chunk, combined when stored
  };
  Stage g0, g1;
  auto gload = [&](Stage& st, int kt) {
    const uint32_t k0 = (uint32_t)(kbase + kt) * kGemmTK;
#pragma unroll
    for (int i = 0; i < 4; ++i) st.x[i] = bld128(rx, xoff[i] + k0 * 2);
    if constexpr (WB == 3) {
      st.w = bld96s(rq, woff, k0 / 8 * 3);
    } else if constexpr (WPT == 4) {
      st.w = bld128(rq, woff + k0 / 2);
    } else {
      const u32x2 q = bld64(rq, woff + k0 / 2);
      st.w = u32x4{q[0], q[1], 0u, 0u};
    }
    const uint32_t g = k0 / a.G;
    st.s = bld16(rsc, wok ? ((uint32_t)wn_row * a.ngroups + g) * 2 : kOOB);
    st.z = bld8(rz, wok ? (uint32_t)wn_row * a.ngroups + g : kOOB);
    if constexpr (kI8) {
      const u32x2 q = bld64(ra, eoff == kOOB ? kOOB : eoff / 2 + k0);
      st.e = u32x4{q[0], q[1], 0u, 0u};
      st.g = bld128(rgw, goff == kOOB ? kOOB : goff + k0 * 2);
    } else if constexpr (kLoc) {
      st.e = bld128(ra, eoff == kOOB ? kOOB : eoff + k0 * 2);
      st.g = bld128(rgw, goff == kOOB ? kOOB : goff + k0 * 2);
    }
  };
  auto lstore = [&](const Stage& st, int buf) {
    const u32x4 (&xreg)[4] = st.x;
    const u32x4 wreg = st.w;
    const float sreg = h2f((uint16_t)st.s);
    const int zreg = (int)st.z;
    uint16_t* xs = Xs + buf * TILEX;
    uint16_t* ws = Ws + buf * TILEW;
#pragma unroll
    for (int i = 0; i < 4; ++i) *(u32x4*)(xs + xr[i] * LR + xc[i]) = xreg[i];
    if constexpr (WB == 4) {
#pragma unroll
      for (int c = 0; c < WPT; ++c) {
        uint32_t o[4];
        dequant_word_pairs<DT>(wreg[c], sreg, zreg, o);
        *(u32x4*)(ws + wr * LR + 8 * (WPT * wp + c)) = u32x4{o[0], o[1], o[2], o[3]};
      }
    } else {
      uint32_t o[4 * WPT];
      if constexpr (WPT == 4) {
        dequant_block3_pairs<DT, 0, 16>(wreg, sreg, zreg, o);
      } else {
        // half 1 of the block: its low fields are word 1, its high bits the
        // upper byte of each half of word 2 (moved down: no branch per lane)
        const bool h1 = (wp & 1) != 0;
        const u32x4 wh = u32x4{h1 ? wreg[1] : wreg[0], 0u, h1 ? wreg[2] >> 8 : wreg[2], 0u};
        dequant_block3_pairs<DT, 0, 8>(wh, sreg, zreg, o);
      }
#pragma unroll
      for (int c = 0; c < WPT; ++c)
        *(u32x4*)(ws + wr * LR + 8 * (WPT * wp + c)) = u32x4{o[4 * c], o[4 * c + 1], o[4 * c + 2], o[4 * c + 3]};
    }
    if constexpr (kLoc) {
      u32x4 ev = st.e;
      if constexpr (kI8) ev = i8x8_to_act<DT>(ev[0], ev[1], sa_er);
      if (tid < kGemmEcRows * 8) *(u32x4*)(Es + buf * ETILE + er * LR + 8 * ec8) = ev | st.g;
    }
  };

  f32x4 acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  // EPI_LOCAL: u = x A^T (waves of row half 0) and the gate logit x w_g
  // (row half 1, w_g in every column) for the wave's 64 tokens
  f32x4 eacc[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) eacc[i] = f32x4{0.f, 0.f, 0.f, 0.f};

  auto compute = [&](int buf) {
    const uint16_t* xs = Xs + buf * TILEX;
    const uint16_t* ws = Ws + buf * TILEW;
#pragma unroll
    for (int kk = 0; kk < kGemmTK; kk += 32) {
      u32x4 af[4], bf[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) af[i] = *(const u32x4*)(xs + (wm * 64 + 16 * i + lr) * LR + kk + 8 * lg);
#pragma unroll
      for (int j = 0; j < 4; ++j) bf[j] = *(const u32x4*)(ws + (wn * 64 + 16 * j + lr) * LR + kk + 8 * lg);
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = mfma16<DT>(af[i], bf[j], acc[i][j]);
      if constexpr (kLoc) {
        const u32x4 ef = *(const u32x4*)(Es + buf * ETILE + (wn == 0 ? lr : 16) * LR + kk + 8 * lg);
#pragma unroll
        for (int i = 0; i < 4; ++i) eacc[i] = mfma16<DT>(af[i], ef, eacc[i]);
      }
    }
  };

  // Step kt computes LDS buffer kt & 1. Its loads were issued two steps
  // earlier into register set kt & 1, and it is stored at the start of its
  // step while the next step's loads are still in flight. K is a multiple of
  // 128, so the steps come in pairs and the loop has a single exit; loads
  // past the last step re-read it (never stored), so that every load is
  // unconditional. Both ways into the loop head thus leave the same loads in
  // flight, and the wait before a store covers only the stage being stored.
  // One barrier per step: a buffer is rewritten only after every wave has
  // passed the barrier that follows its last read.
  const int kl = KT - 1;
  gload(g0, 0);
  __builtin_amdgcn_sched_barrier(0);
  gload(g1, 1);
  __builtin_amdgcn_sched_barrier(0);
  for (int kt = 0; kt < KT; kt += 2) {
    lstore(g0, 0);
    __syncthreads();
    gload(g0, min(kt + 2, kl));
    __builtin_amdgcn_sched_barrier(0);
    compute(0);
    __builtin_amdgcn_sched_barrier(0);
    lstore(g1, 1);
    __syncthreads();
    gload(g1, min(kt + 3, kl));
    __builtin_amdgcn_sched_barrier(0);
    compute(1);
    __builtin_amdgcn_sched_barrier(0);
  }

  // split-K: every slice publishes its tile (lane-major f32x4), and with
  // EPI_LOCAL its EC accumulators; the last to arrive sums the slices in
  // slice order (reading its own back like the others) and runs the epilogue
  if (a.S > 1) {
    __shared__ int s_last;
    const uint32_t tbytes = TM * kGemmTN * 4;
    const rsrc_t rp = make_rsrc(a.ypart, (uint32_t)a.S * T * tbytes);
    const uint32_t ybase = (uint32_t)tb * tbytes + (uint32_t)(wave * 16 * 64 + lane) * 16;
    const uint32_t yslice = (uint32_t)T * tbytes;
    constexpr uint32_t ebytes = 2 * TMW * 4 * 64 * 16;  // EC accumulators of a tile
    const rsrc_t rep = make_rsrc(kLoc ? a.epart : nullptr, kLoc ? (uint32_t)a.S * T * ebytes : 0u);
    const uint32_t ebase = (uint32_t)tb * ebytes + (uint32_t)(wave * 4 * 64 + lane) * 16;
    const uint32_t eslice = (uint32_t)T * ebytes;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) bst128c(rp, ybase + ks * yslice + (i * 4 + j) * 1024, acc[i][j]);
    if constexpr (kLoc) {
#pragma unroll
      for (int i = 0; i < 4; ++i) bst128c(rep, ebase + ks * eslice + i * 1024, eacc[i]);
    }
    complete_and_sync();
    if (tid == 0) s_last = arrive_last(a.ctr + tb, (uint32_t)a.S) ? 1 : 0;
    __syncthreads();
    if (!s_last) return;
    if (a.S == 2) {
      gemm_sum_slices<2>(rp, ybase, yslice, acc);
      if constexpr (kLoc) gemm_sum_ec_slices<2>(rep, ebase, eslice, eacc);
    } else if (a.S == 4) {
      gemm_sum_slices<4>(rp, ybase, yslice, acc);
      if constexpr (kLoc) gemm_sum_ec_slices<4>(rep, ebase, eslice, eacc);
    } else {
      gemm_sum_slices<8>(rp, ybase, yslice, acc);
      if constexpr (kLoc) gemm_sum_ec_slices<8>(rep, ebase, eslice, eacc);
    }
  }

  // EPI_LOCAL: v = alpha g(x) (.) u for the block's TM tokens, as act-dtype
  // high and low parts [TM][32] in LDS (the stage buffers are free once
  // every wave is past its last step)
  constexpr int kVS = 32;
  float* u_sh = (float*)smem;                                  // [TM][17]
  uint16_t* vh_sh = (uint16_t*)(smem + TM * 17 * 4);           // [TM][kVS]
  uint16_t* vl_sh = vh_sh + TM * kVS;
  if constexpr (kLoc) {
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int e2 = 0; e2 < 4; ++e2) {
        const int t = wm * 64 + 16 * i + 4 * lg + e2;
        if (wn == 0 && lr < a.r) u_sh[t * 17 + lr] = eacc[i][e2];
        if (wn == 1 && lr == 0) u_sh[t * 17 + 16] = eacc[i][e2];
      }
    __syncthreads();
    // the tanh-MLP gate: v [TM][16] in fp32 first, its hidden layer in the
    // rest of the (free) stage buffers
    float* v_sh = (float*)(smem + TM * 17 * 4 + 2 * TM * kVS * 2);
    const bool tanh_g = a.gate == GATE_TANH;  // uniform
    if (tanh_g) {
      // after v: the hidden layer
      constexpr int kLds = 2 * (TM + kGemmTN) * LR * 2 + 2 * kGemmEcRows * LR * 2;
      float* hid = v_sh + TM * 16;
      const int hid_floats = (kLds - (int)((char*)hid - smem)) / 4;
      const int cap = max(1, min(TM, hid_floats / max(1, a.h)));
      tanh_gate_tokens<DT>(TM, a.r, a.h, u_sh, 17, a.W1, a.b1, a.W2, a.b2, a.alpha, hid, cap,
                           v_sh, 16);
    }
    for (int idx = tid; idx < TM * kVS; idx += NT) {
      const int t = idx / kVS, j = idx - t * kVS;
      float val = 0.f;
      if (j < a.r && tanh_g) {
        val = v_sh[t * 16 + j];
      } else if (j < a.r) {
        float g = 1.f;
        if (a.gate == GATE_SIGMOID) {
          const float z = u_sh[t * 17 + 16] + a.b_g;
          g = z >= 0.f ? 1.f / (1.f + __expf(-z)) : __expf(z) / (1.f + __expf(z));
        }
        val = a.alpha * g * u_sh[t * 17 + j];
      }
      const uint16_t hi = f2act<DT>(val);
      vh_sh[idx] = hi;
      vl_sh[idx] = f2act<DT>(val - act2f<DT>(hi));
    }
    __syncthreads();
  }

  if constexpr (EPI == EPI_READY || kLoc) {
    // y += v_hi B^T + v_lo B^T over the rank (zero-padded to vstride); INT8
    // B rows are dequantised with their scale
    const int r = a.r;
    const bool bvec = (r & 7) == 0;
    const bool b8 = kI8 || (EPI == EPI_READY && a.B8 != nullptr);  // uniform
    const int vstride = kLoc ? kVS : a.vstride;
    for (int kr = 0; kr < vstride; kr += 32) {
      const int kk = kr + 8 * lg;
      u32x4 vhf[4], vlf[4], bfr[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int t = wm * 64 + 16 * i + lr, m = m0 + t;
        const bool ok = m < M;
        if constexpr (kLoc) {
          vhf[i] = *(const u32x4*)(vh_sh + t * kVS + kk);
          vlf[i] = *(const u32x4*)(vl_sh + t * kVS + kk);
        } else {
          vhf[i] = ok ? ldg16(a.vh + (size_t)m * a.vstride + kk) : u32x4{0, 0, 0, 0};
          vlf[i] = ok ? ldg16(a.vl + (size_t)m * a.vstride + kk) : u32x4{0, 0, 0, 0};
        }
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int n = n0 + wn * 64 + 16 * j + lr;
        u32x4 f = u32x4{0, 0, 0, 0};
        if (n < N && b8) {
          const int8_t* br = a.B8 + (size_t)n * r;
          const float sb = a.sb[n];
          if (bvec) {
            if (kk < r) {
              const u32x2 q = *(const u32x2*)(br + kk);
              f = i8x8_to_act<DT>(q[0], q[1], sb);
            }
          } else {
            uint32_t h[8];
#pragma unroll
            for (int e2 = 0; e2 < 8; ++e2) h[e2] = (kk + e2 < r) ? i8_to_act<DT>(br[kk + e2], sb) : 0u;
            f = u32x4{h[0] | (h[1] << 16), h[2] | (h[3] << 16), h[4] | (h[5] << 16), h[6] | (h[7] << 16)};
          }
        } else if (n < N) {
          const uint16_t* br = a.B + (size_t)n * r;
          if (bvec) {
            if (kk < r) f = ldg16(br + kk);
          } else {
            uint32_t h[8];
#pragma unroll
            for (int e2 = 0; e2 < 8; ++e2) h[e2] = (kk + e2 < r) ? br[kk + e2] : 0u;
            f = u32x4{h[0] | (h[1] << 16), h[2] | (h[3] << 16), h[4] | (h[5] << 16), h[6] | (h[7] << 16)};
          }
        }
        bfr[j] = f;
      }
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          acc[i][j] = mfma16<DT>(vhf[i], bfr[j], acc[i][j]);
          acc[i][j] = mfma16<DT>(vlf[i], bfr[j], acc[i][j]);
        }
    }
  }

  const rsrc_t ry = make_rsrc(a.y, (uint32_t)M * N * 2), rres = make_rsrc(a.res, (uint32_t)M * N * 2);
#pragma unroll
  for (int i = 0; i < 4; ++i)
    store_results<DT, 16>(
        ry, rres, a.res != nullptr,
        [&](int q) {  // q = 4 j + e2
          const int n = n0 + wn * 64 + 16 * (q >> 2) + lr, m = m0 + wm * 64 + 16 * i + 4 * lg + (q & 3);
          return n < N && m < M ? ((uint32_t)m * N + n) * 2 : kOOB;
        },
        [&](int q) { return acc[i][q >> 2][q & 3]; });
}

// ---------------------------------------------------------------------------
// Prefill GEMM with loading and multiplying waves (4-bit codes, 256 x 128
// tiles, one K-slice; the plain and the semi-fused epilogue). In k_gemm every
// wave dequantises its share of the next step and then multiplies, and the
// step's barrier lines the waves up, so a SIMD runs the dequantisation's
// VALU work and the MFMAs one after the other. Here waves 0-3 only multiply
// (each owns 128 tokens x 64 rows: 8 x 4 MFMA tiles) and waves 4-7 only load:
// they dequantise and store step kt+1's tiles into the free LDS buffer while
// the multiplying waves read step kt's, and issue the loads of step kt+3.
// Each SIMD holds one loading wave beside its multiplying ones, so the two
// streams overlap; one barrier per step. A wave also reads 12 fragments per
// 32 MFMAs here, not 16.
// TNB = 1: 256 x 128 tiles, four multiplying waves (one per SIMD);
// TNB = 2: 256 x 256 tiles, eight multiplying waves (two per SIMD, 144 KB
// of LDS), twelve waves in all, at most 168 registers each.
// WB: code width (4, or 3: three words per 32 codes).
// PLAIN: the epilogue of 256 x 256 tiles without a residual stores under the
// row and token bounds; a call with one, and 256 x 128 tiles, take the
// branch-free buffer stores (fp16, PLAIN against those: 8192 x 2048 at 2048
// tokens 70.4 us against 75.3, at 4096 136 against 149, but with a residual 94
// against 77; 4096 x 4096 at 2048 tokens on 256 x 128 tiles 81 against 79).
// ---------------------------------------------------------------------------
template <int DT, int EPI, int TNB, int WB, bool PLAIN>
__global__ __launch_bounds__(256 * (1 + TNB), 1) void k_gemm_ws(GemmParams a) {
  static_assert(EPI == EPI_NONE || EPI == EPI_READY, "plain and semi-fused epilogues");
  extern __shared__ __attribute__((aligned(16))) char smem[];
  constexpr int TM = 256, TN = kGemmTN * TNB, LR = kGemmLdsRow;
  constexpr int TILEX = TM * kGemmTK, TILEW = TN * LR;
  constexpr int NCW = 4 * TNB;   // multiplying waves: 2 along the tokens, 2 TNB along the rows
  constexpr int WPT = 4 * TNB;   // code words per loading thread and step
  // activations: [2][TM][64] unpadded, the 16-byte chunk c of row t at
  // chunk c ^ (t % 8) (conflict-free fragment reads without padding, which
  // the 1 KB runs of the direct loads below cannot skip)
  uint16_t* Xs = (uint16_t*)smem;
  uint16_t* Ws = Xs + 2 * TILEX;   // [2][TN][LR]
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int M = a.M, N = a.N, K = a.K;
  const int tiles_m = (M + TM - 1) / TM, tiles_n = (N + TN - 1) / TN;
  // XCD banding as in k_gemm
  int mt_i, nt_i;
  {
    const int b = (int)blockIdx.x, x = b & 7, j = b >> 3;
    if ((tiles_m & 7) == 0) {
      const int pm = tiles_m >> 3;
      mt_i = x * pm + j % pm;
      nt_i = j / pm;
    } else if ((tiles_n & 7) == 0) {
      const int pn = tiles_n >> 3;
      nt_i = x * pn + j % pn;
      mt_i = j / pn;
    } else {
      mt_i = b / tiles_n;
      nt_i = b - mt_i * tiles_n;
    }
  }
  const int m0 = mt_i * TM, n0 = nt_i * TN;
  const int KT = K / kGemmTK;  // steps (K is a multiple of 128: an even count)

  // EPI_READY: v_hi, v_lo [TM][64] and B [TN][64] (act dtype, zero past the
  // rank, INT8 rows dequantised with their scale) for rank columns
  // kr0 .. kr0 + 63, staged into LDS (free after the K loop) by all waves
  constexpr int ER = 72;  // padded LDS row (halves)
  uint16_t* vhs = (uint16_t*)smem;  // [TM][ER]
  uint16_t* vls = vhs + TM * ER;    // [TM][ER]
  uint16_t* bss = vls + TM * ER;    // [TN][ER]
  auto ec_stage = [&](int kr0) {
    const int r = a.r;
    for (int c = tid; c < 2 * TM * 8; c += 256 * (1 + TNB)) {
      const int lo = c >= TM * 8, cc = lo ? c - TM * 8 : c;
      const int t = cc >> 3, col = kr0 + (cc & 7) * 8, m = m0 + t;
      u32x4 v = u32x4{0, 0, 0, 0};
      if (m < M && col < a.vstride) v = ldg16((lo ? a.vl : a.vh) + (size_t)m * a.vstride + col);
      *(u32x4*)((lo ? vls : vhs) + t * ER + (cc & 7) * 8) = v;
    }
    for (int c = tid; c < TN * 8; c += 256 * (1 + TNB)) {
      const int row = c >> 3, col = kr0 + (c & 7) * 8, n = n0 + row;
      u32x4 f = u32x4{0, 0, 0, 0};
      if (n < N && col < r) {
        if (a.B8) {
          const int8_t* br = a.B8 + (size_t)n * r;
          const float sb = a.sb[n];
          if ((r & 7) == 0) {
            const u32x2 q = *(const u32x2*)(br + col);
            f = i8x8_to_act<DT>(q[0], q[1], sb);
          } else {
            uint32_t h[8];
#pragma unroll
            for (int e2 = 0; e2 < 8; ++e2) h[e2] = col + e2 < r ? i8_to_act<DT>(br[col + e2], sb) : 0u;
            f = u32x4{h[0] | (h[1] << 16), h[2] | (h[3] << 16), h[4] | (h[5] << 16), h[6] | (h[7] << 16)};
          }
        } else {
          const uint16_t* br = a.B + (size_t)n * r;
          if ((r & 7) == 0) {
            f = ldg16(br + col);
          } else {
            uint32_t h[8];
#pragma unroll
            for (int e2 = 0; e2 < 8; ++e2) h[e2] = col + e2 < r ? br[col + e2] : 0u;
            f = u32x4{h[0] | (h[1] << 16), h[2] | (h[3] << 16), h[4] | (h[5] << 16), h[6] | (h[7] << 16)};
          }
        }
      }
      *(u32x4*)(bss + row * ER + (c & 7) * 8) = f;
    }
  };

  if (wave >= NCW) {
    // ---- loading waves: thread pt stages, of each 64-wide step, the codes
    // of K half pt % 2 of row pt / 2 (TNB = 1) or both halves of row pt
    // (TNB = 2): per half four words, or one 3-bit block of three
    const int pt = tid - 64 * NCW;
    const rsrc_t rq = make_rsrc(a.qw, (uint32_t)N * row_code_bytes<WB>(K));
    const rsrc_t rsc = make_rsrc(a.sc, (uint32_t)N * a.ngroups * 2);
    const rsrc_t rz = make_rsrc(a.zr, (uint32_t)N * a.ngroups);
    const int wr = TNB == 2 ? pt : pt >> 1, wp = TNB == 2 ? 0 : pt & 1;
    const int wn_row = n0 + wr;
    const bool wok = wn_row < N;
    const uint32_t woff = !wok ? kOOB : (uint32_t)wn_row * row_code_bytes<WB>(K) + (WB == 4 ? 16 : 12) * wp;
    struct Stage {
      u32x4 w[TNB];
      uint32_t s, z;
    };
    Stage g0, g1;
    auto gload = [&](Stage& st, int kt) {
      const uint32_t k0 = (uint32_t)kt * kGemmTK;
#pragma unroll
      for (int h = 0; h < TNB; ++h) {
        if constexpr (WB == 4) st.w[h] = bld128(rq, wok ? woff + k0 / 2 + 16 * h : kOOB);
        else st.w[h] = bld96s(rq, woff, k0 / 8 * 3 + 12 * h);
      }
      const uint32_t g = k0 / a.G;
      st.s = bld16(rsc, wok ? ((uint32_t)wn_row * a.ngroups + g) * 2 : kOOB);
      st.z = bld8(rz, wok ? (uint32_t)wn_row * a.ngroups + g : kOOB);
    };
    auto lstore = [&](const Stage& st, int buf) {
      uint16_t* ws = Ws + buf * TILEW;
      const float sreg = h2f((uint16_t)st.s);
      const int zreg = (int)st.z;
      if constexpr (WB == 4) {
#pragma unroll
        for (int c = 0; c < WPT; ++c) {
          uint32_t o[4];
          dequant_word_pairs<DT>(st.w[c >> 2][c & 3], sreg, zreg, o);
          *(u32x4*)(ws + wr * LR + 8 * (4 * wp + c)) = u32x4{o[0], o[1], o[2], o[3]};
        }
      } else {
#pragma unroll
        for (int h = 0; h < TNB; ++h) {
          uint32_t o[16];
          dequant_block3_pairs<DT, 0, 16>(st.w[h], sreg, zreg, o);
#pragma unroll
          for (int c = 0; c < 4; ++c)
            *(u32x4*)(ws + wr * LR + 8 * (4 * (wp + h) + c)) =
                u32x4{o[4 * c], o[4 * c + 1], o[4 * c + 2], o[4 * c + 3]};
        }
      }
    };
    // step kt stores step kt + 1 (loaded two steps earlier) and then loads
    // step kt + 3 into the same registers; loads past the end re-read the
    // last step (never stored), so that every load is unconditional
    const int kl = KT - 1;
    gload(g0, 0);
    __builtin_amdgcn_sched_barrier(0);
    gload(g1, min(1, kl));
    __builtin_amdgcn_sched_barrier(0);
    lstore(g0, 0);
    gload(g0, min(2, kl));
    __syncthreads();
    for (int kt = 0; kt < KT; kt += 2) {
      lstore(g1, 1);
      gload(g1, min(kt + 3, kl));
      __syncthreads();
      if (kt + 2 < KT) {
        lstore(g0, 0);
        gload(g0, min(kt + 4, kl));
      }
      __syncthreads();
    }
    if constexpr (EPI == EPI_READY) {
      for (int kr0 = 0; kr0 < a.vstride; kr0 += 64) {
        ec_stage(kr0);
        __syncthreads();
        __syncthreads();
      }
    }
    return;
  }

  // ---- multiplying waves: wave c owns tokens 128 (c / (2 TNB)) .., rows
  // 64 (c % (2 TNB)) .., as 4 x 2 tiles of the 32 x 32 x 16 MFMA (half the
  // MFMA instructions of 16 x 16 x 32 tiles for the same LDS reads: measured
  // alone with the stage stores, 60% of the peak against 51%). They issue
  // ahead of the loading wave of their SIMD when both are ready: the loading
  // waves have a step of slack, the MFMA pipe none.
  __builtin_amdgcn_s_setprio(1);
  const int l32 = lane & 31, lh = lane >> 5;
  const int wm = wave / (2 * TNB), wn = wave % (2 * TNB);
  constexpr int FM32 = 4, FN32 = 2;
  // The activation tile goes straight from memory into LDS (16-byte buffer
  // loads to LDS): the multiplying waves issue it, one step ahead into the
  // free buffer, and wait for it only at the step's barrier, behind their
  // own MFMAs; they have no other memory loads, so the wait covers nothing
  // else. Wave w writes the 1 KB runs w IPW .. +IPW of the tile (eight rows
  // each); lane l of a run lands at 16 l: row 8 run + l / 8, stored chunk
  // l % 8, which holds the row's chunk (l % 8) ^ (row % 8).
  constexpr int IPW = 32 / NCW;  // 1 KB runs per multiplying wave and step
  const rsrc_t rx = make_rsrc(a.x, (uint32_t)M * K * 2);
  uint32_t xoff[IPW];
#pragma unroll
  for (int u = 0; u < IPW; ++u) {
    const int row = (wave * IPW + u) * 8 + (lane >> 3);
    const int c = (lane & 7) ^ (row & 7);
    xoff[u] = m0 + row < M ? ((uint32_t)(m0 + row) * K + 8 * c) * 2 : kOOB;
  }
  auto xdma = [&](int kt, int buf) {
    const uint32_t kb = (uint32_t)kt * kGemmTK * 2;
#pragma unroll
    for (int u = 0; u < IPW; ++u)
      bld128_lds(rx, Xs + buf * TILEX + (wave * IPW + u) * 512, xoff[u] == kOOB ? kOOB : xoff[u] + kb);
  };
  f32x16 acc[FM32][FN32];
#pragma unroll
  for (int i = 0; i < FM32; ++i)
#pragma unroll
    for (int j = 0; j < FN32; ++j) acc[i][j] = f32x16{};
  // 16-K slices: the slice's six fragments, then its eight MFMAs; SW: the
  // token operand is the swizzled activation tile (rows of 64 halves). The
  // scheduling groups keep the reads ahead: the weight fragments and the
  // first two token fragments go out before the first MFMA, then each pair
  // of MFMAs is followed by the next token fragment's read.
  auto mma = [&](const uint16_t* xs, const uint16_t* ws, int xr0, int wr0, int ld, int kk, bool sw) {
    u32x4 bf[FN32], af[FM32];
#pragma unroll
    for (int j = 0; j < FN32; ++j) bf[j] = *(const u32x4*)(ws + (wr0 + 32 * j + l32) * ld + kk + 8 * lh);
#pragma unroll
    for (int i = 0; i < FM32; ++i) {
      const int t = xr0 + 32 * i + l32;
      af[i] = sw ? *(const u32x4*)(xs + t * kGemmTK + 8 * (((kk >> 3) + lh) ^ (t & 7)))
                 : *(const u32x4*)(xs + t * ld + kk + 8 * lh);
    }
#pragma unroll
    for (int i = 0; i < FM32; ++i)
#pragma unroll
      for (int j = 0; j < FN32; ++j) acc[i][j] = mfma32<DT>(af[i], bf[j], acc[i][j]);
    __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);  // 4 LDS reads
    __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);  // 2 MFMAs
    __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
    __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    __builtin_amdgcn_sched_group_barrier(0x008, 4, 0);
  };
  xdma(0, 0);
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  // one copy of the step's MFMAs in the loop (two copies, one per buffer,
  // make the register allocator shuffle accumulators between them)
  for (int kt = 0; kt < KT; ++kt) {
    if (kt + 1 < KT) xdma(kt + 1, (kt + 1) & 1);
    const uint16_t* xs = Xs + (kt & 1) * TILEX;
    const uint16_t* ws = Ws + (kt & 1) * TILEW;
#pragma unroll
    for (int kk = 0; kk < kGemmTK; kk += 16) mma(xs, ws, wm * 128, wn * 64, LR, kk, true);
    __builtin_amdgcn_s_waitcnt(0);  // this wave's share of the next tile is in LDS
    __syncthreads();
  }

  if constexpr (EPI == EPI_READY) {
    // y += v_hi B^T + v_lo B^T over the rank (zero-padded to vstride), 64
    // rank columns at a time from LDS, as 32 x 32 x 16 MFMAs like the K loop
    for (int kr0 = 0; kr0 < a.vstride; kr0 += 64) {
      ec_stage(kr0);
      __syncthreads();
#pragma unroll
      for (int kk = 0; kk < 64; kk += 16) {
        if (kr0 + kk < a.vstride) {
          mma(vhs, bss, wm * 128, wn * 64, ER, kk, false);
          mma(vls, bss, wm * 128, wn * 64, ER, kk, false);
        }
      }
      __syncthreads();
    }
  }

  if constexpr (PLAIN) {
#pragma unroll
    for (int i = 0; i < FM32; ++i)
#pragma unroll
      for (int j = 0; j < FN32; ++j) {
        const int n = n0 + wn * 64 + 32 * j + l32;
        if (n >= N) continue;
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int m = m0 + wm * 128 + 32 * i + 8 * (e >> 2) + 4 * lh + (e & 3);
          if (m < M) a.y[(size_t)m * N + n] = f2act<DT>(acc[i][j][e]);
        }
      }
  } else {
    const rsrc_t ry = make_rsrc(a.y, (uint32_t)M * N * 2), rres = make_rsrc(a.res, (uint32_t)M * N * 2);
#pragma unroll
    for (int i = 0; i < FM32; ++i)
#pragma unroll
      for (int j = 0; j < FN32; ++j)
        store_results<DT, 16>(
            ry, rres, a.res != nullptr,
            [&](int e) {
              const int n = n0 + wn * 64 + 32 * j + l32;
              const int m = m0 + wm * 128 + 32 * i + 8 * (e >> 2) + 4 * lh + (e & 3);
              return n < N && m < M ? ((uint32_t)m * N + n) * 2 : kOOB;
            },
            [&](int e) { return acc[i][j][e]; });
  }
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
hipError_t SPEAR_W(launch_dequant)(const uint32_t* qw, const uint16_t* sc, const uint8_t* zr,
                                   uint16_t* out, int N, int K, int G, hipStream_t st) {
  const long long nunits = (long long)N * (K / (SPEAR_WB == 4 ? 8 : 32));
  const unsigned grid = (unsigned)((nunits + 255) / 256);
  if (grid == 0) return hipSuccess;
  hipLaunchKernelGGL((k_dequant<DTC, SPEAR_WB>), dim3(grid), dim3(256), 0, st,
                                         qw, sc, zr, out, N, K, G);
  return hipGetLastError();
}

hipError_t SPEAR_W(launch_gemm)(int epi, const GemmParams& p, hipStream_t st) {
  // split-K needs its partial tiles and tile counters (workspace); the
  // 256-token tile takes the plain and the semi-fused epilogue only
  const bool loc = epi == EPI_LOCAL || epi == EPI_LOCAL_I8;
  if (p.S < 1 || (p.S > 1 && (!p.ypart || !p.ctr || (loc && !p.epart))) ||
      (p.S != 1 && p.S != 2 && p.S != 4 && p.S != 8) ||
      (epi == EPI_LOCAL_I8 && (!p.A8 || !p.sa || !p.B8 || !p.sb)) ||
      (p.tmw != 2 && p.tmw != 4) || (p.tmw == 4 && loc))
    return hipErrorInvalidValue;
  const int TM = 64 * p.tmw;
  const int tm = (p.M + TM - 1) / TM, tn = (p.N + kGemmTN - 1) / kGemmTN;
  const unsigned grid = (unsigned)(tm * tn * p.S);
  if (grid == 0) return hipSuccess;
  size_t lds = (size_t)2 * (TM + kGemmTN) * kGemmLdsRow * 2;
  if (loc) lds += (size_t)2 * kGemmEcRows * kGemmLdsRow * 2;
#define SPEAR_GEMM_GO(E, W)                                                            \
  do {                                                                                 \
    hipError_t err = allow_lds(k_gemm<DTC, E, W, SPEAR_WB>, lds);                      \
    if (err != hipSuccess) return err;                                                 \
    hipLaunchKernelGGL((k_gemm<DTC, E, W, SPEAR_WB>), dim3(grid), dim3(128 * W), lds, st, p); \
  } while (0)
  if (p.roles == 2 || p.roles == 3) {
    // loading and multiplying waves: 256 x 128 (roles 2) or 256 x 256
    // (roles 3) tiles, one K-slice
    if (p.tmw != 4 || p.S != 1 || (epi != EPI_NONE && epi != EPI_READY)) return hipErrorInvalidValue;
    const int tnb = p.roles == 3 ? 2 : 1;
    const unsigned gws = (unsigned)(tm * ((p.N + 128 * tnb - 1) / (128 * tnb)));
    // unpadded activation stages, padded weight stages; the EC epilogue
    // reuses the space for v_hi, v_lo [256][72] and B [rows][72]
    const size_t lws = std::max((size_t)2 * TM * kGemmTK * 2 + (size_t)2 * 128 * tnb * kGemmLdsRow * 2,
                                (size_t)(2 * TM + 128 * tnb) * kGemmLdsRow * 2);
    const auto go = [&](auto kern) {
      hipError_t err = allow_lds(kern, lws);
      if (err != hipSuccess) return err;
      hipLaunchKernelGGL(kern, dim3(gws), dim3(256 * (1 + tnb)), lws, st, p);
      return hipGetLastError();
    };
    if (tnb == 1)
      return epi == EPI_NONE ? go(k_gemm_ws<DTC, EPI_NONE, 1, SPEAR_WB, false>)
                             : go(k_gemm_ws<DTC, EPI_READY, 1, SPEAR_WB, false>);
    if (p.res)
      return epi == EPI_NONE ? go(k_gemm_ws<DTC, EPI_NONE, 2, SPEAR_WB, false>)
                             : go(k_gemm_ws<DTC, EPI_READY, 2, SPEAR_WB, false>);
    return epi == EPI_NONE ? go(k_gemm_ws<DTC, EPI_NONE, 2, SPEAR_WB, true>)
                           : go(k_gemm_ws<DTC, EPI_READY, 2, SPEAR_WB, true>);
  }
  if (p.tmw == 4) {
    if (epi == EPI_NONE) SPEAR_GEMM_GO(EPI_NONE, 4);
    else SPEAR_GEMM_GO(EPI_READY, 4);
  } else if (epi == EPI_NONE) {
    SPEAR_GEMM_GO(EPI_NONE, 2);
  } else if (epi == EPI_LOCAL) {
    SPEAR_GEMM_GO(EPI_LOCAL, 2);
  } else if (epi == EPI_LOCAL_I8) {
    SPEAR_GEMM_GO(EPI_LOCAL_I8, 2);
  } else {
    SPEAR_GEMM_GO(EPI_READY, 2);
  }
#undef SPEAR_GEMM_GO
  return hipGetLastError();
}

}  // namespace spear
