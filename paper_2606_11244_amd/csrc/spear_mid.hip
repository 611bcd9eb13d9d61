// gfx950 (MI355X) GEMM of the W4+EC linear layer for decode batches and prefill
// chunks, from 17 tokens up (operand and layout conventions: spear_device.h).
//
// At these sizes every code is used by few tokens, so the product is bound by
// streaming the codes and by the VALU work of dequantising them, not by the
// MFMAs. The codes therefore go from memory straight into the registers of
// the one wave that multiplies by them (no LDS round trip, no store, and no
// barrier between their arrival and their use), a ring of ST iterations ahead,
// while the activation tile, which all waves share, comes into LDS by direct
// 16-byte loads as many iterations ahead.
#include "spear_device.h"

namespace spear {

// Waits until at most `n` of this wave's vector-memory operations are
// outstanding (they complete in order); LDS and export counters untouched.
template <int n>
__device__ __forceinline__ void wait_vm() {
  static_assert(n < 64, "6-bit counter");
  __builtin_amdgcn_s_waitcnt((n & 15) | (7 << 4) | (15 << 8) | ((n >> 4) << 14));
}

// Workgroup barrier with no wait for outstanding loads to LDS (a __syncthreads()
// waits for all of them): the caller has waited for what it publishes.
__device__ __forceinline__ void bare_barrier() {
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

// acc[i] = sum over S slices, in slice order, of entry i (1024 bytes apart) of
// the thread's partials at `base`; the loads of up to 32 entries are in
// flight together.
template <int S, int NE>
__device__ __forceinline__ void sum_tile_slices(rsrc_t rp, uint32_t base, uint32_t slice, f32x4 (&acc)[NE]) {
  constexpr int E = NE < 32 / S ? NE : 32 / S;
#pragma unroll
  for (int r0 = 0; r0 < NE; r0 += E) {
    f32x4 pv[S][E];
#pragma unroll
    for (int q = 0; q < S; ++q)
#pragma unroll
      for (int e = 0; e < E; ++e)
        if (r0 + e < NE) pv[q][e] = bld128cf(rp, base + q * slice + (r0 + e) * 1024);
#pragma unroll
    for (int e = 0; e < E; ++e)
      if (r0 + e < NE) {
        f32x4 t = pv[0][e];
#pragma unroll
        for (int q = 1; q < S; ++q) t += pv[q][e];
        acc[r0 + e] = t;
      }
  }
}

// A workgroup owns 16 MT tokens x 128 rows and a K-slice of 128-wide
// iterations; wave w of its four owns rows 32 w .. +32 as two 16-row tiles.
// A wave multiplies iteration it while it unpacks the codes of it + 1 in the
// shadow of the MFMAs. FOLD (up to 64 tokens): the codes become exact
// integers (fp16: q - z; bf16: 128 + q, with sum_k x from MFMAs against ones,
// as in k_gemv) and each 128-wide group's sum is folded with its scale (and
// zero point) in fp32: fewer VALU instructions than a multiplication per code
// while few token tiles share it, and no rounding of the weights. Otherwise
// the codes are dequantised with one rounding, as in k_gemm, and the
// accumulators run over all of K.
template <int DT, int MT, int WB, bool FOLD>
__device__ __forceinline__ void gemm_r_body(const GemmParams& a, int bid, char* smem) {
  constexpr int RT = 2, TM = 16 * MT, ST = mid_stages(MT);
  constexpr int DW = 6;  // code stages (even: the unpacked sets alternate)
  static_assert(DW >= ST + 1, "the codes of it + 1 land with the activations of it");
  constexpr bool kEx = FOLD && DT == DT_F16, kBi = FOLD && DT == DT_BF16;
  constexpr int XST = TM * kIterK;  // halves per activation stage
  uint16_t* Xs = (uint16_t*)smem;   // [ST][TM][128], chunk c of row t at c ^ (t % 16)
  uint32_t* szs = (uint32_t*)(smem + (size_t)ST * XST * 2);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane & 15, lg = lane >> 4;
  const int M = a.M, N = a.N, K = a.K;
  const int tiles_m = (M + TM - 1) / TM, tiles_n = (N + kMidTN - 1) / kMidTN;
  // consecutive workgroups go to the eight XCDs in turn: the token tiles of
  // one row tile, which read the same codes, follow each other on one XCD
  const int T = tiles_m * tiles_n;
  const int ks = bid / T, tb = bid - ks * T;
  int mt_i, nt_i;
  if ((tiles_n & 7) == 0) {
    const int x = tb & 7, j = tb >> 3;
    mt_i = j % tiles_m;
    nt_i = (j / tiles_m) * 8 + x;
  } else {
    mt_i = tb % tiles_m;
    nt_i = tb / tiles_m;
  }
  const int m0 = mt_i * TM, n0 = nt_i * kMidTN;
  const int IT = K / kIterK;
  const int it_beg = ks * a.ips, it_end = min(IT, it_beg + a.ips), last = it_end - 1;
  // The slice's iterations are walked from a start that differs between the
  // row tiles of one XCD: the rows of x and of the codes are a multiple of
  // 4 KB apart, so all rows of one K position lie in the same L2 channel, and
  // workgroups that walk K in step would queue at one channel at a time.
  const int nit = it_end - it_beg, rot = (nt_i >> 3) % nit;
  auto at = [&](int j) {  // the j-th iteration of the walk; past the end, the last
    const int i = min(j, nit - 1) + rot;
    return it_beg + (i >= nit ? i - nit : i);
  };

  const rsrc_t rx = make_rsrc(a.x, (uint32_t)M * K * 2);
  const rsrc_t rq = make_rsrc(a.qw, (uint32_t)N * row_code_bytes<WB>(K));
  const rsrc_t rsc = make_rsrc(a.sc, (uint32_t)N * a.ngroups * 2);
  const rsrc_t rz = make_rsrc(a.zr, (uint32_t)N * a.ngroups);

  // scales and zero points of the workgroup's rows over its groups, staged
  // once ([row][group] as s | z << 16, odd row stride); eight groups per load
  // when the group range is aligned
  const int ipg = a.G / kIterK;
  const int g_lo = it_beg / ipg, ngb = last / ipg + 1 - g_lo, ngs = ngb | 1;
  const bool sz8 = (a.ngroups & 7) == 0 && (g_lo & 7) == 0 && (ngb & 7) == 0;
  const int c8 = sz8 ? ngb >> 3 : 1, nsz = sz8 ? kMidTN * c8 : kMidTN * ngb;
  constexpr int SZU = 4;
  auto sz_load = [&](int i, u32x4& s, u32x2& z) {
    if (sz8) {
      const int row = i / c8, q = i - row * c8;
      const uint32_t eo = (uint32_t)(n0 + row) * a.ngroups + g_lo + 8 * q;
      const bool ok = i < nsz && n0 + row < N;
      s = bld128(rsc, ok ? eo * 2 : kOOB);
      z = bld64(rz, ok ? eo : kOOB);
    } else {
      const int row = i / ngb, g = i - row * ngb;
      const uint32_t eo = (uint32_t)(n0 + row) * a.ngroups + g_lo + g;
      const bool ok = i < nsz && n0 + row < N;
      s[0] = bld16(rsc, ok ? eo * 2 : kOOB);
      z[0] = bld8(rz, ok ? eo : kOOB);
    }
  };
  auto sz_store = [&](int i, const u32x4& s, const u32x2& z) {
    if (i >= nsz) return;
    if (sz8) {
      const int row = i / c8, q = i - row * c8;
#pragma unroll
      for (int e = 0; e < 8; ++e)
        szs[row * ngs + 8 * q + e] =
            ((s[e >> 1] >> (16 * (e & 1))) & 0xFFFFu) | (((z[e >> 2] >> (8 * (e & 3))) & 0xFFu) << 16);
    } else {
      const int row = i / ngb, g = i - row * ngb;
      szs[row * ngs + g] = s[0] | (z[0] << 16);
    }
  };
  u32x4 s_st[SZU];
  u32x2 z_st[SZU];
#pragma unroll
  for (int u = 0; u < SZU; ++u) sz_load(tid + 256 * u, s_st[u], z_st[u]);

  // activation tile: wave w brings the 1 KB runs w MT .. +MT (four rows each);
  // lane l of a run lands at 16 l: row 4 run + l / 16, stored chunk l % 16
  uint32_t xoff[MT];
#pragma unroll
  for (int u = 0; u < MT; ++u) {
    const int row = (wave * MT + u) * 4 + (lane >> 4), c = (lane & 15) ^ (row & 15);
    xoff[u] = m0 + row < M ? ((uint32_t)(m0 + row) * K + 8 * c) * 2 : kOOB;
  }
  // codes: lane group lg holds K [32 lg, +32) of its row's iteration
  uint32_t vw[RT];
#pragma unroll
  for (int t = 0; t < RT; ++t) {
    const int n = n0 + wave * 32 + 16 * t + lr;
    vw[t] = n < N ? (uint32_t)n * row_code_bytes<WB>(K) + (WB == 4 ? 16 : 12) * lg : kOOB;
  }
  u32x4 w[DW][RT];
  // iterations past the last re-read it (never multiplied), so that the
  // number of operations in flight is fixed
  auto issue_x = [&](int j) {
    const uint32_t kb = (uint32_t)at(j) * (kIterK * 2);
    uint16_t* xs = Xs + (j % ST) * XST + wave * MT * 512;
#pragma unroll
    for (int u = 0; u < MT; ++u) bld128_lds(rx, xs + u * 512, xoff[u] == kOOB ? kOOB : xoff[u] + kb);
  };
  auto issue_w = [&](u32x4 (&wq)[RT], int j) {
    const int i = at(j);
#pragma unroll
    for (int t = 0; t < RT; ++t)
      wq[t] = WB == 4 ? bld128s(rq, vw[t], (uint32_t)i * (kIterK / 2))
                      : bld96s(rq, vw[t], (uint32_t)i * (kIterK / 8 * 3));
  };
  // in the order of the loop below: the code stages ahead of its first
  // group, then one group of MT + RT operations per iteration
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int q = 0; q < DW - ST + 1; ++q) issue_w(w[q], q);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int q = 0; q < ST - 1; ++q) {
    issue_x(q);
    issue_w(w[q + DW - ST + 1], q + DW - ST + 1);
    __builtin_amdgcn_sched_barrier(0);
  }
#pragma unroll
  for (int u = 0; u < SZU; ++u) sz_store(tid + 256 * u, s_st[u], z_st[u]);
  if (nsz > 256 * SZU) {  // uniform
    for (int i = tid + 256 * SZU; i < nsz; i += 256) {
      u32x4 s;
      u32x2 z;
      sz_load(i, s, z);
      sz_store(i, s, z);
    }
  }

  f32x4 acc[RT * MT];
#pragma unroll
  for (int i = 0; i < RT * MT; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  uint32_t xrd[4];  // this lane's fragment of token row lr (halves): K 32 lg + 8 jj
#pragma unroll
  for (int jj = 0; jj < 4; ++jj) xrd[jj] = lr * kIterK + 8 * ((4 * lg + jj) ^ lr);
  const uint32_t* szl = szs + (wave * 32 + lr) * ngs;
  const uint32_t km = opaque_v(DT == DT_F16 ? 0x00F0000Fu : 0x000F000Fu);
  const uint32_t kg = opaque_v(DT == DT_F16 ? 0x64006400u : 0x43004300u);
  // unpacked codes of one iteration, with the scale and bias of its fold
  struct Unpacked {
    u32x4 c[RT][4];
    float sf[RT], cf[RT];
  };
  Unpacked ua, ub;
  // code word jj of a row, dequantised with one rounding (natural order)
  auto dequant = [&](const u32x4& wq, int jj, uint32_t sz) {
    const uint32_t z = sz >> 16;
    uint32_t r[4];
    if constexpr (WB == 4 && DT == DT_F16) {
      const _Float16 s1 = __builtin_bit_cast(_Float16, (uint16_t)(sz & 0xFFFFu));
      const u32x4 q = exact_word(wq[jj], km, kg, exact_cz(z));
#pragma unroll
      for (int e = 0; e < 4; ++e)
        r[e] = __builtin_bit_cast(uint32_t, __builtin_bit_cast(f16x2, (uint32_t)q[e]) * f16x2{s1, s1});
    } else if constexpr (WB == 4) {
      dequant_word_pairs<DT>(wq[jj], h2f((uint16_t)(sz & 0xFFFFu)), (int)z, r);
    } else {
      const u32x4 bq = unpack3_biased(wq, jj, 0u);
      const uint32_t pq[4] = {bq[0], bq[1], bq[2], bq[3]};
      dequant_pairs<DT, 4>(pq, h2f((uint16_t)(sz & 0xFFFFu)), (int)z, r);
    }
    return u32x4{r[0], r[1], r[2], r[3]};
  };
  // words 4 t + jj in [w0, w1) of an iteration's codes
  auto unpack = [&](Unpacked& o, const u32x4 (&wq)[RT], const uint32_t (&sz)[RT], int w0, int w1) {
#pragma unroll
    for (int i = 0; i < 4 * RT; ++i) {
      if (i < w0 || i >= w1) continue;
      const int t = i >> 2, jj = i & 3;
      const uint32_t z = sz[t] >> 16;
      if (jj == 0) {
        o.sf[t] = h2f((uint16_t)(sz[t] & 0xFFFFu));
        o.cf[t] = code_bias<DT>() + (float)z;
      }
      if constexpr (kEx && WB == 4) {
        o.c[t][jj] = exact_word(wq[t][jj], km, kg, exact_cz(z));
      } else if constexpr (kEx) {
        const _Float16 zb = (_Float16)(1024 + (int)z);
        const u32x4 bq = unpack3_biased(wq[t], jj, kg);
#pragma unroll
        for (int e = 0; e < 4; ++e)
          o.c[t][jj][e] = __builtin_bit_cast(uint32_t, __builtin_bit_cast(f16x2, (uint32_t)bq[e]) + f16x2{-zb, -zb});
      } else if constexpr (kBi) {
        o.c[t][jj] = WB == 4 ? biased_word_nat(wq[t][jj], km, kg) : unpack3_biased(wq[t], jj, kg);
      } else {
        o.c[t][jj] = dequant(wq[t], jj, sz[t]);
      }
    }
  };
  auto read_sz = [&](uint32_t (&sz)[RT], int j) {
    const int gg = at(j) / ipg - g_lo;
#pragma unroll
    for (int t = 0; t < RT; ++t) sz[t] = szl[16 * t * ngs + gg];
  };
  // multiplies iteration it by `u`, and unpacks `wn`, the codes of it + 1,
  // into `un`; the fragments of a token tile are read while the tile before
  // it multiplies, and (FOLD) a tile's sums are folded while the next does
  auto compute = [&](const Unpacked& u, Unpacked& un, const u32x4 (&wn)[RT], int j) {
    const uint16_t* xs = Xs + (j % ST) * XST;
    uint32_t sz[RT];
    read_sz(sz, j + 1);
    u32x4 xf[2][4];
    auto xread = [&](int mt) {
#pragma unroll
      for (int jj = 0; jj < 4; ++jj) xf[mt & 1][jj] = *(const u32x4*)(xs + mt * 16 * kIterK + xrd[jj]);
    };
    xread(0);
    f32x4 p[2][RT], xb[2];
    auto fold = [&](int mt) {
#pragma unroll
      for (int t = 0; t < RT; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          acc[t * MT + mt][i] += kEx ? u.sf[t] * p[mt & 1][t][i]
                                     : u.sf[t] * (p[mt & 1][t][i] - u.cf[t] * xb[mt & 1][i]);
    };
    constexpr int NW = 4 * RT;  // code words per iteration, spread over the token tiles
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      if (mt + 1 < MT) xread(mt + 1);
      const u32x4 (&x4)[4] = xf[mt & 1];
      if constexpr (FOLD) {
        if (kBi) xb[mt & 1] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int t = 0; t < RT; ++t) p[mt & 1][t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) {
          if (kBi) xb[mt & 1] = mfma16<DT>(x4[jj], ones8<DT>(), xb[mt & 1]);
#pragma unroll
          for (int t = 0; t < RT; ++t) p[mt & 1][t] = mfma16<DT>(x4[jj], u.c[t][jj], p[mt & 1][t]);
        }
        if (mt > 0) fold(mt - 1);
      } else {
#pragma unroll
        for (int jj = 0; jj < 4; ++jj)
#pragma unroll
          for (int t = 0; t < RT; ++t) acc[t * MT + mt] = mfma16<DT>(x4[jj], u.c[t][jj], acc[t * MT + mt]);
      }
      unpack(un, wn, sz, NW * mt / MT, NW * (mt + 1) / MT);
    }
    if constexpr (FOLD) fold(MT - 1);
  };

  // Iteration it: its activations, issued ST - 1 iterations earlier, and the
  // codes of it + 1, issued no later, have landed (the ST - 2 later groups may
  // still be in flight). The barrier shows every wave's share of the stage,
  // and that every wave is done with the stage of it - 1, which the loads of
  // it + ST - 1 then fill. The rounds of DW iterations have no branch inside:
  // with one, the waits for the codes would cover every load in flight.
  auto step = [&](int q, int j) {
    wait_vm<(ST - 2) * (MT + RT)>();
    bare_barrier();
    issue_x(j + ST - 1);
    issue_w(w[q], j + DW);
    __builtin_amdgcn_sched_barrier(0);
    if ((q & 1) == 0) compute(ua, ub, w[(q + 1) % DW], j);
    else compute(ub, ua, w[(q + 1) % DW], j);
    __builtin_amdgcn_sched_barrier(0);
  };
  __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): this wave's scales are in LDS
  bare_barrier();
  {
    uint32_t sz[RT];
    read_sz(sz, 0);
    unpack(ua, w[0], sz, 0, 4 * RT);
  }
  int j = 0;
  for (; j + DW <= nit; j += DW) {
#pragma unroll
    for (int q = 0; q < DW; ++q) step(q, j + q);
  }
#pragma unroll
  for (int q = 0; q < DW - 1; ++q)
    if (j + q < nit) step(q, j + q);  // uniform over the workgroup
  wait_vm<0>();  // the last groups' loads to LDS, before the workgroup's LDS is given up

  // The biased codes of kBi (128 + q, less 128 + z afterwards) turn an infinite
  // activation into infinity less infinity, and overflow from about 2^120 on.
  // A wave that holds a sum that is not finite forms its tile again from the
  // dequantised weights, which keep infinities and large values as they are.
  if constexpr (kBi) {
    bool lost = false;
#pragma unroll
    for (int i = 0; i < RT * MT; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) lost |= !(__builtin_fabsf(acc[i][e]) < __builtin_inff());
    if (__ballot(lost) != 0) {
#pragma unroll
      for (int i = 0; i < RT * MT; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
      for (int q = 0; q < nit; ++q) {
        u32x4 wq[RT];
        uint32_t sz[RT];
        issue_w(wq, q);
        read_sz(sz, q);
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) {
          u32x4 c[RT];
#pragma unroll
          for (int t = 0; t < RT; ++t) c[t] = dequant(wq[t], jj, sz[t]);
#pragma unroll
          for (int mt = 0; mt < MT; ++mt) {
            const int m = m0 + 16 * mt + lr;
            const u32x4 xq = bld128(rx, m < M ? ((uint32_t)m * K + at(q) * kIterK + 32 * lg + 8 * jj) * 2 : kOOB);
#pragma unroll
            for (int t = 0; t < RT; ++t) acc[t * MT + mt] = mfma16<DT>(xq, c[t], acc[t * MT + mt]);
          }
        }
      }
    }
  }

  // v_hi and v_lo of the tile's tokens for the epilogue, [2][TM][vstride + 8]
  // in LDS (the stages are free once every wave is here); requested before
  // the slices' partial tiles, so that the two round trips overlap
  const int vch = a.vh ? a.vstride >> 3 : 0, nv = 2 * TM * vch, vrow = a.vstride + 8;
  uint16_t* vs = (uint16_t*)smem;
  u32x4 v_st[4];
  auto v_load = [&](int i) {
    const int row = i / vch, c = i - row * vch, t = row < TM ? row : row - TM;
    return i < nv && m0 + t < M ? ldg16((row < TM ? a.vh : a.vl) + (size_t)(m0 + t) * a.vstride + 8 * c)
                                : u32x4{0, 0, 0, 0};
  };
  auto v_store = [&](int i, const u32x4& v) {
    const int row = i / vch, c = i - row * vch;
    if (i < nv) *(u32x4*)(vs + row * vrow + 8 * c) = v;
  };
  // split-K: every slice publishes its tile (lane-major); the last to arrive
  // sums the slices in slice order and runs the epilogue
  if (a.S > 1) {
    __shared__ int s_last;
    constexpr uint32_t tbytes = TM * kMidTN * 4;
    const rsrc_t rp = make_rsrc(a.ypart, (uint32_t)a.S * T * tbytes);
    const uint32_t ybase = (uint32_t)tb * tbytes + (uint32_t)(wave * RT * MT * 64 + lane) * 16;
    const uint32_t yslice = (uint32_t)T * tbytes;
#pragma unroll
    for (int i = 0; i < RT * MT; ++i) bst128c(rp, ybase + ks * yslice + i * 1024, acc[i]);
    complete_and_sync();
    if (tid == 0) s_last = arrive_last(a.ctr + tb, (uint32_t)a.S) ? 1 : 0;
    __syncthreads();
    if (!s_last) return;
    if (a.vh) {
#pragma unroll
      for (int u = 0; u < 4; ++u) v_st[u] = v_load(tid + 256 * u);
    }
    if (a.S == 2) sum_tile_slices<2>(rp, ybase, yslice, acc);
    else if (a.S == 4) sum_tile_slices<4>(rp, ybase, yslice, acc);
    else sum_tile_slices<8>(rp, ybase, yslice, acc);
  }

  if (a.vh) {  // uniform
    // y += v_hi B^T + v_lo B^T over the rank (zero-padded to vstride); INT8 B
    // rows are dequantised with their scale
    const int r = a.r;
    const bool bvec = (r & 7) == 0;
    if (a.S == 1) {
#pragma unroll
      for (int u = 0; u < 4; ++u) v_st[u] = v_load(tid + 256 * u);
      __syncthreads();  // every wave is past its last stage
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) v_store(tid + 256 * u, v_st[u]);
    for (int i = tid + 1024; i < nv; i += 1024) {
#pragma unroll
      for (int u = 0; u < 4; ++u) v_st[u] = v_load(i + 256 * u);
#pragma unroll
      for (int u = 0; u < 4; ++u) v_store(i + 256 * u, v_st[u]);
    }
    __syncthreads();
    for (int kr = 0; kr < a.vstride; kr += 32) {
      const int kk = kr + 8 * lg;
      u32x4 bfr[RT];
#pragma unroll
      for (int t = 0; t < RT; ++t) {
        const int n = n0 + wave * 32 + 16 * t + lr;
        u32x4 f = u32x4{0, 0, 0, 0};
        if (n < N && kk < r) {
          if (bvec) {
            if (a.B8) {
              const u32x2 q = *(const u32x2*)(a.B8 + (size_t)n * r + kk);
              f = i8x8_to_act<DT>(q[0], q[1], a.sb[n]);
            } else {
              f = ldg16(a.B + (size_t)n * r + kk);
            }
          } else {
            uint32_t h[8];
#pragma unroll
            for (int e = 0; e < 8; ++e)
              h[e] = kk + e >= r ? 0u
                     : a.B8      ? (uint32_t)i8_to_act<DT>(a.B8[(size_t)n * r + kk + e], a.sb[n])
                                 : (uint32_t)a.B[(size_t)n * r + kk + e];
            f = u32x4{h[0] | (h[1] << 16), h[2] | (h[3] << 16), h[4] | (h[5] << 16), h[6] | (h[7] << 16)};
          }
        }
        bfr[t] = f;
      }
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        const u32x4 vh = *(const u32x4*)(vs + (16 * mt + lr) * vrow + kk);
        const u32x4 vl = *(const u32x4*)(vs + (TM + 16 * mt + lr) * vrow + kk);
#pragma unroll
        for (int t = 0; t < RT; ++t) {
          acc[t * MT + mt] = mfma16<DT>(vh, bfr[t], acc[t * MT + mt]);
          acc[t * MT + mt] = mfma16<DT>(vl, bfr[t], acc[t * MT + mt]);
        }
      }
    }
  }

  const rsrc_t ry = make_rsrc(a.y, (uint32_t)M * N * 2), rres = make_rsrc(a.res, (uint32_t)M * N * 2);
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
    store_results<DT, 4 * RT>(
        ry, rres, a.res != nullptr,
        [&](int q) {  // q = 4 t + i
          const int n = n0 + wave * 32 + 16 * (q >> 2) + lr, m = m0 + 16 * mt + 4 * lg + (q & 3);
          return n < N && m < M ? ((uint32_t)m * N + n) * 2 : kOOB;
        },
        [&](int q) { return acc[(q >> 2) * MT + mt][q & 3]; });
}

// Up to kGroupMax independent layer calls in one launch (one for a single
// call): member i owns workgroups [start[i], start[i+1]) and runs exactly the
// workgroups its own launch would run. The member index is uniform.
template <int DT, int MT, int WB, bool FOLD>
__global__ __launch_bounds__(256, MT <= 4 ? 2 : 1) void k_gemm_r(GemmGroup g) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int b = blockIdx.x;
  int i = 0;
#pragma unroll
  for (int j = 1; j < kGroupMax; ++j)
    if (j < g.n && b >= g.start[j]) i = j;
  gemm_r_body<DT, MT, WB, FOLD>(g.p[i], b - g.start[i], smem);
}

// ---------------------------------------------------------------------------
// launcher
// ---------------------------------------------------------------------------
template <int MT>
static hipError_t mid_launch(const GemmGroup& g, hipStream_t st) {
  constexpr bool FOLD = MT <= 4;
  size_t lds = 0;
  for (int i = 0; i < g.n; ++i) {
    const int ipg = g.p[i].G / kIterK;
    lds = std::max(lds, mid_lds(MT, std::min(g.p[i].ngroups, (g.p[i].ips + ipg - 1) / ipg + 1)));
    if (g.p[i].vh) lds = std::max(lds, (size_t)4 * 16 * MT * (g.p[i].vstride + 8));
  }
  hipError_t err = allow_lds(k_gemm_r<DTC, MT, SPEAR_WB, FOLD>, lds);
  if (err != hipSuccess) return err;
  hipLaunchKernelGGL((k_gemm_r<DTC, MT, SPEAR_WB, FOLD>), dim3(g.start[g.n]), dim3(256), lds, st, g);
  return hipGetLastError();
}

hipError_t SPEAR_W(launch_mid)(int MT, const GemmGroup& g, hipStream_t st) {
  if (g.n < 1 || g.n > kGroupMax || g.start[0] != 0) return hipErrorInvalidValue;
  for (int i = 0; i < g.n; ++i) {
    // every slice holds an iteration, the slices cover K, and the grid is
    // the tiles times the slices
    const GemmParams& p = g.p[i];
    const int IT = p.K / kIterK;
    if ((p.S != 1 && p.S != 2 && p.S != 4 && p.S != 8) || (p.S > 1 && (!p.ypart || !p.ctr)) || p.ips < 1 ||
        (p.S - 1) * p.ips >= IT || p.S * p.ips < IT ||
        g.start[i + 1] - g.start[i] != mid_tiles(MT, p.M, p.N) * p.S)
      return hipErrorInvalidValue;
  }
  if (g.start[g.n] == 0) return hipSuccess;
  switch (MT) {
    case 2: return mid_launch<2>(g, st);
    case 3: return mid_launch<3>(g, st);
    case 4: return mid_launch<4>(g, st);
    case 6: return mid_launch<6>(g, st);
    case 8: return mid_launch<8>(g, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace spear
