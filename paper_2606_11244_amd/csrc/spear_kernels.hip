// gfx950 (MI355X) decode kernels of the W4+EC linear layer, its EC pre-kernel
// and the post-EC tail (the prefill GEMMs are in spear_gemm.hip).
//
// Y = X . What^T + alpha * (gate (.) (X . A^T)) . B^T      (SPEAR, section 3.1, Eq. 3)
// What[n][k] = (q[n][k] - z[n][k/G]) * s[n][k/G]          (sections 2.1, 5.1)
//
// Kernels:
//   k_ec       EC projection u = [A; w_g] x over a K-slice, last-arriver
//              reduction across slices, gate, v = alpha * gate (.) u
//   k_gemv     decode: 4-bit product with MFMA on one 16-row tile per block,
//              per-128 dequant correction, cross-wave (and, for long K,
//              cross-block) reduction, epilogue adding B v; in the fused
//              variant the grid's first blocks run k_ec's work and publish v
//              as tagged words that the other blocks poll
//   k_gate, k_ec_up_acc   the naive split chain's separate gate and
//              reprojection+accumulate launches
//   k_rmsnorm  post-EC tail
#include "spear_device.h"

namespace spear {

// ---------------------------------------------------------------------------
// EC projection of one token tile over iterations [it_beg, it_end) and row
// tiles [t_beg, t_end) of R = [A; w_g] (R1 rows; the gate row w_g is row r):
// u_lds[t][j] = sum_k x[16*tb + t][k] * R[j][k] for the rows of those tiles.
// Each wave takes IPP iterations per pass with all of their loads issued
// first; the waves' partial tiles are summed in LDS in a fixed order (wave 0
// first), so the result does not depend on timing.
// ---------------------------------------------------------------------------
template <int DT, int IPP>
__device__ __forceinline__ void ec_project(const EcParams& e, int tb, int it_beg, int it_end, int t_beg, int t_end,
                           float* u_lds, float* red) {
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int NW = blockDim.x >> 6;
  const int lr = lane & 15, lg = lane >> 4;
  // token rows past M read row M-1: their results are never used
  const int m = min(tb * kTokTile + lr, e.M - 1);
  const rsrc_t rx = make_rsrc(e.x, (uint32_t)e.M * e.K * 2);
  const bool i8 = e.A8 != nullptr;  // uniform
  const rsrc_t ra = i8 ? make_rsrc(e.A8, (uint32_t)e.r * e.K) : make_rsrc(e.A, (uint32_t)e.r * e.K * 2);
  const rsrc_t rg = make_rsrc(e.wg, e.gate == GATE_SIGMOID ? (uint32_t)e.K * 2 : 0u);
  // K order within an iteration: MFMA jj, lane group lg takes K
  // [8 lg + 32 jj, +8) for both operands, so that each load reads 64
  // contiguous bytes per row (the MFMA lane layout would otherwise spread a
  // load over twice as many cache lines)
  const uint32_t xoff = (uint32_t)m * e.K * 2 + 16 * lg;
  for (int tg0 = t_beg; tg0 < t_end; tg0 += kEcTiles) {
    const int nt = min(kEcTiles, t_end - tg0);
    f32x4 acc[kEcTiles];
    uint32_t aoff[kEcTiles], goff[kEcTiles];
    bool has_g[kEcTiles];
#pragma unroll
    for (int t = 0; t < kEcTiles; ++t) {
      acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
      const int j = (tg0 + t) * 16 + lr;
      aoff[t] = (t < nt && j < e.r) ? (uint32_t)j * e.K * 2 + 16 * lg : kOOB;
      goff[t] = (t < nt && j == e.r && e.gate == GATE_SIGMOID) ? 16u * lg : kOOB;
      // uniform: does this row tile hold the gate row?
      has_g[t] = t < nt && e.gate == GATE_SIGMOID && e.r >= (tg0 + t) * 16 &&
                 e.r < (tg0 + t + 1) * 16;
    }
    // the gate row's tile (uniform), or -1; w_g goes to registers of its own
    // and joins that tile's operand only at the MFMA (a value combined right
    // after its load would make the wave wait for every earlier load)
    int gt = -1;
#pragma unroll
    for (int t = 0; t < kEcTiles; ++t)
      if (has_g[t]) gt = t;
    uint32_t goff_g = kOOB;
#pragma unroll
    for (int t = 0; t < kEcTiles; ++t)
      if (t == gt) goff_g = goff[t];
    // the iterations, for act-dtype A (16-byte loads) or INT8 A (8-byte
    // loads of the same eight K, dequantised with the row's scale at the MFMA)
    auto iterate = [&](auto i8c) {
      constexpr bool kI8 = decltype(i8c)::value;
      float sa[kEcTiles];
#pragma unroll
      for (int t = 0; t < kEcTiles; ++t) {
        const int j = (tg0 + t) * 16 + lr;
        sa[t] = kI8 && t < nt && j < e.r ? e.sa[j] : 0.f;
      }
      for (int it0 = it_beg + wave * IPP; it0 < it_end; it0 += NW * IPP) {
        u32x4 xv[IPP][4], av[IPP][kEcTiles][4], gv[IPP][4];
#pragma unroll
        for (int h = 0; h < IPP; ++h) {
          const bool ok = it0 + h < it_end;  // uniform
          const uint32_t kb = (uint32_t)(it0 + h) * (kIterK * 2);
#pragma unroll
          for (int jj = 0; jj < 4; ++jj) xv[h][jj] = bld128(rx, ok ? xoff + kb + 64 * jj : kOOB);
#pragma unroll
          for (int t = 0; t < kEcTiles; ++t)
#pragma unroll
            for (int jj = 0; jj < 4; ++jj) {
              if constexpr (kI8) {
                // aoff[t] and kb count 2-byte elements twice: halve them
                const u32x2 q = bld64(ra, ok && aoff[t] != kOOB ? (aoff[t] + kb) / 2 + 32 * jj : kOOB);
                av[h][t][jj] = u32x4{q[0], q[1], 0u, 0u};
              } else {
                av[h][t][jj] = bld128(ra, ok && aoff[t] != kOOB ? aoff[t] + kb + 64 * jj : kOOB);
              }
            }
#pragma unroll
          for (int jj = 0; jj < 4; ++jj)
            gv[h][jj] = bld128(rg, ok && goff_g != kOOB ? goff_g + kb + 64 * jj : kOOB);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int h = 0; h < IPP; ++h)
#pragma unroll
          for (int t = 0; t < kEcTiles; ++t)
#pragma unroll
            for (int jj = 0; jj < 4; ++jj) {
              u32x4 af = av[h][t][jj];
              if constexpr (kI8) af = i8x8_to_act<DT>(af[0], af[1], sa[t]);
              acc[t] = mfma16<DT>(t == gt ? (af | gv[h][jj]) : af, xv[h][jj], acc[t]);
            }
      }
    };
    if (i8) iterate(std::true_type{});
    else iterate(std::false_type{});
    // lane l holds token l % 16 and rows 4 * (l / 16) .. + 3 of each tile
#pragma unroll
    for (int t = 0; t < kEcTiles; ++t)
      *(f32x4*)(red + ((wave * kEcTiles + t) * 64 + lane) * 4) = acc[t];
    __syncthreads();
    for (int idx = tid; idx < nt * 256; idx += blockDim.x) {
      const int t = idx >> 8, rem = idx & 255, ln = rem >> 2, i = rem & 3;
      float s = 0.f;
      for (int w = 0; w < NW; ++w) s += red[((w * kEcTiles + t) * 64 + ln) * 4 + i];
      const int j = (tg0 + t) * 16 + 4 * (ln >> 4) + i;
      if (j < e.R1) u_lds[(ln & 15) * e.R1p + j] = s;
    }
    __syncthreads();
  }
}

// Gate of one token tile: from u (LDS, [16][R1p]) to v_tile (LDS, [16][r]):
// v = alpha * g * u (sigmoid-linear), alpha * (1 + tanh(W2 ReLU(W1 u + b1) + b2)) (.) u
// (tanh-MLP), or alpha * u (gate one). Ends with a barrier.
template <int DT>
__device__ __forceinline__ void ec_gate_tile(const EcParams& e, int cnt, const float* u_lds, float* hid,
                             float* v_tile) {
  const int tid = threadIdx.x, nthr = blockDim.x;
  const int r = e.r;
  if (e.gate == GATE_TANH) {
    tanh_gate_tokens<DT>(cnt, r, e.h, u_lds, e.R1p, e.W1, e.b1, e.W2, e.b2, e.alpha, hid,
                         ec_hid_tokens(e.h), v_tile, r);
  } else {
    for (int idx = tid; idx < cnt * r; idx += nthr) {
      const int t = idx / r, j = idx - t * r;
      float g = 1.f;
      if (e.gate == GATE_SIGMOID) {
        const float z = u_lds[t * e.R1p + r] + e.b_g;
        g = z >= 0.f ? 1.f / (1.f + __expf(-z)) : __expf(z) / (1.f + __expf(z));
      }
      v_tile[idx] = e.alpha * g * u_lds[t * e.R1p + j];
    }
    __syncthreads();
  }
}

// One EC producer workgroup b: token tile, K-slice and row-tile group from b.
// It projects its share; then (EC_GATHER) publishes its tagged partial sums
// for the consumers to add up, or joins the last-arriver reduction of its
// token tile, whose last workgroup sums the slices in order, applies the gate
// and publishes v: as fp32 (read by a later kernel), as act-dtype hi/lo parts
// (the prefill GEMM epilogue) and/or as tagged words in one copy per XCD (the
// fused kernel's consumers).
template <int DT, int IPP, bool PRE>
__device__ __forceinline__ void ec_producer(const EcParams& e, int b, uint32_t gen, char* smem) {
  __shared__ int s_last;
  const int tid = threadIdx.x, nthr = blockDim.x;
  const int NW = nthr >> 6;
  const int IT = e.K / kIterK;
  const int per_tb = e.P * e.PG;
  const int tb = b / per_tb, rem = b - tb * per_tb;
  const int pk = rem / e.PG, pg = rem - pk * e.PG;
  const int it_beg = pk * e.ips, it_end = min(IT, it_beg + e.ips);
  const int RTe = (e.R1 + 15) >> 4;
  const int t_beg = pg * e.tpg, t_end = min(RTe, t_beg + e.tpg);
  float* red = (float*)smem;
  char* es = smem + ec_red_bytes(NW);
  float* u_lds = (float*)(es + ec_lds_u_off());
  float* hid = (float*)(es + ec_lds_hid_off(e.R1p));
  float* v_tile = (float*)(es + ec_lds_v_off(e.R1p, ec_hid_floats(e.h)));
  const int m0 = tb * kTokTile;
  const int cnt = min(kTokTile, e.M - m0);
  const int j_beg = 16 * t_beg, nj = min(e.R1, 16 * t_end) - j_beg;

  // the tanh-MLP gate's parameters, which only the token tile's last workgroup
  // reads, after everything else: requested here (up to 16 KB of each matrix)
  // so that its reads find them in this XCD's L2 instead of in memory. (Not
  // among the fused GEMV's producers, whose registers it costs: 4096 x 14336 at
  // four tokens 26.9 us without it, 27.9 with it.)
  if (PRE && e.gate == GATE_TANH) {
    const rsrc_t r1 = make_rsrc(e.W1, (uint32_t)e.h * e.r * 2), r2 = make_rsrc(e.W2, (uint32_t)e.h * e.r * 2);
    u32x4 t[4];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      t[u] = bld128(r1, 16u * (tid + u * nthr));
      t[2 + u] = bld128(r2, 16u * (tid + u * nthr));
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) asm volatile("" ::"v"(t[u]));
  }
  ec_project<DT, IPP>(e, tb, it_beg, it_end, t_beg, t_end, u_lds, red);

  if (e.mode == EC_GATHER) {
    const uint32_t tag = ec_tag(gen);
    const size_t per_copy = (size_t)e.P * e.M * e.R1;
    for (int idx = tid; idx < kVCopies * cnt * nj; idx += nthr) {
      const int c = idx / (cnt * nj), o = idx - c * (cnt * nj);
      const int t = o / nj, j = j_beg + (o - t * nj);
      const unsigned long long w =
          ((unsigned long long)tag << 32) | __float_as_uint(u_lds[t * e.R1p + j]);
      __hip_atomic_store(e.vtag + c * per_copy + ((size_t)pk * e.M + m0 + t) * e.R1 + j, w,
                         __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    // the data is complete before the ready counters count it
    complete_and_sync();
    if (tid < kVCopies)
      __hip_atomic_fetch_add(e.ready + tid * (kReadyStride / 8), (unsigned long long)publisher_increment(b, e.npub),
                             __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return;
  }

  if (per_tb > 1) {
    float* part = e.upart + ((size_t)tb * e.P + pk) * kTokTile * e.R1;
    for (int idx = tid; idx < cnt * nj; idx += nthr) {
      const int t = idx / nj, j = j_beg + (idx - t * nj);
      st_agent(part + t * e.R1 + j, u_lds[t * e.R1p + j]);
    }
    complete_and_sync();
    if (tid == 0) s_last = arrive_last(e.ctr + tb, (uint32_t)per_tb) ? 1 : 0;
    __syncthreads();
    if (!s_last) return;
    // the slices' partial tiles [P][cnt][R1], summed in slice order
    const rsrc_t rp = make_rsrc(e.upart + (size_t)tb * e.P * kTokTile * e.R1,
                                (uint32_t)e.P * kTokTile * e.R1 * 4);
    sum_slices(rp, e.P, cnt * e.R1,
               [&](int q, int i) { return (uint32_t)(q * kTokTile * e.R1 + i) * 4u; },
               [&](int i, float v) {
                 const int t = i / e.R1, j = i - t * e.R1;
                 u_lds[t * e.R1p + j] = v;
               });
  }

  if (e.mode == EC_RAW) {
    for (int idx = tid; idx < cnt * e.R1; idx += nthr) {
      const int t = idx / e.R1, j = idx - t * e.R1;
      e.u_out[(size_t)(m0 + t) * e.R1 + j] = u_lds[t * e.R1p + j];
    }
    return;
  }

  ec_gate_tile<DT>(e, cnt, u_lds, hid, v_tile);
  if (e.v)
    for (int idx = tid; idx < cnt * e.r; idx += nthr) e.v[(size_t)m0 * e.r + idx] = v_tile[idx];
  if (e.vh) {
    for (int idx = tid; idx < cnt * e.vstride; idx += nthr) {
      const int t = idx / e.vstride, j = idx - t * e.vstride;
      const float val = j < e.r ? v_tile[t * e.r + j] : 0.f;
      const uint16_t hi = f2act<DT>(val);
      const uint16_t lo = f2act<DT>(val - act2f<DT>(hi));
      e.vh[(size_t)(m0 + t) * e.vstride + j] = hi;
      e.vl[(size_t)(m0 + t) * e.vstride + j] = lo;
    }
  }
  if (e.vtag) {
    const uint32_t tag = ec_tag(gen);
    const size_t per_copy = (size_t)e.M * e.r;
    for (int idx = tid; idx < cnt * e.r * kVCopies; idx += nthr) {
      const int c = idx / (cnt * e.r), o = idx - c * (cnt * e.r);
      const unsigned long long w =
          ((unsigned long long)tag << 32) | __float_as_uint(v_tile[o]);
      __hip_atomic_store(e.vtag + c * per_copy + (size_t)m0 * e.r + o, w, __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_AGENT);
    }
    complete_and_sync();
    if (tid < kVCopies)
      __hip_atomic_fetch_add(e.ready + tid * (kReadyStride / 8), (unsigned long long)publisher_increment(tb, e.npub),
                             __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// EC pre-kernel (semi-fused and chain paths): one producer per workgroup. The
// call of one layer passes that layer's parameters alone: with the group's
// member table, four times as long, the 3000 x 2944 layer of rank 8 took 14.8
// us at three tokens against 14.0, 14336 x 4096 of rank 32 at four 22.3 against
// 21.4.
template <int DT, int IPP>
__global__ __launch_bounds__(512) void k_ec(EcParams e) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  ec_producer<DT, IPP, true>(e, blockIdx.x, 0u, smem);
}

// The same of up to kGroupMax layers in one launch (the layers of a group share
// no data, and a launch of a few workgroups costs as much as one of a few
// hundred).
template <int DT, int IPP>
__global__ __launch_bounds__(512) void k_ec_group(EcGroup g) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int b = blockIdx.x;
  int i = 0;
#pragma unroll
  for (int j = 1; j < kGroupMax; ++j)
    if (j < g.n && b >= g.start[j]) i = j;
  ec_producer<DT, IPP, true>(g.p[i], b - g.start[i], 0u, smem);
}

// Naive chain, gate launch: reads u [M][R1] and writes v [M][r].
template <int DT>
__global__ __launch_bounds__(256) void k_gate(EcParams e) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  float* u_lds = (float*)(smem + ec_lds_u_off());
  float* hid = (float*)(smem + ec_lds_hid_off(e.R1p));
  float* v_tile = (float*)(smem + ec_lds_v_off(e.R1p, ec_hid_floats(e.h)));
  const int m0 = blockIdx.x * kTokTile;
  const int cnt = min(kTokTile, e.M - m0);
  for (int idx = threadIdx.x; idx < cnt * e.R1; idx += blockDim.x) {
    const int t = idx / e.R1, j = idx - t * e.R1;
    u_lds[t * e.R1p + j] = e.u_out[(size_t)(m0 + t) * e.R1 + j];
  }
  __syncthreads();
  ec_gate_tile<DT>(e, cnt, u_lds, hid, v_tile);
  for (int idx = threadIdx.x; idx < cnt * e.r; idx += blockDim.x) e.v[(size_t)m0 * e.r + idx] = v_tile[idx];
}

// Naive chain, reprojection + accumulate: y[m][n] += sum_j v[m][j] B[n][j]
// (INT8 B: sb[n] * sum_j v[m][j] q[n][j], in fp32).
template <int DT>
__global__ __launch_bounds__(256) void k_ec_up_acc(const float* __restrict__ v,
                                                   const uint16_t* __restrict__ B,
                                                   const int8_t* __restrict__ B8,
                                                   const float* __restrict__ sb,
                                                   uint16_t* __restrict__ y, int M, int N, int r) {
  const long long idx = (long long)blockIdx.x * 256 + threadIdx.x;
  if (idx >= (long long)M * N) return;
  const int m = (int)(idx / N), n = (int)(idx % N);
  float a = act2f<DT>(y[idx]);
  if (B8) {
    float t = 0.f;
    for (int j = 0; j < r; ++j) t += v[(size_t)m * r + j] * (float)B8[(size_t)n * r + j];
    a += sb[n] * t;
  } else {
    for (int j = 0; j < r; ++j) a += v[(size_t)m * r + j] * act2f<DT>(B[(size_t)n * r + j]);
  }
  y[idx] = f2act<DT>(a);
}

// Post-EC tail, next-layer RMSNorm: y_norm[m][n] = y[m][n] * rsqrt(mean_n y[m][n]^2
// + eps) * w[n] over the stored (rounded) row, in fp32, one rounding. One
// workgroup per token row; the sum of squares is reduced in a fixed order.
//
// Rows of a multiple of eight elements: at decode the kernel is one memory
// round trip and a reduction, at prefill a copy. Each thread takes C 16-byte
// chunks of the row (chunk c * threads + tid), all loaded together with the
// norm weights and kept in registers for the second pass, and the reduction
// is a butterfly per wave and one exchange of the wave sums, one barrier.
// (Two-byte loads in a strided loop, one round trip per element and a
// barrier per tree level took 16.0 us for an 8192-wide row at one token and
// 47 at 4096 tokens; this takes 4.3 us, of which about 3 are the launch and
// the first byte, and about 20.)
template <int DT, int C>
__global__ __launch_bounds__(1024) void k_rmsnorm_v(const uint16_t* __restrict__ y,
                                                    const uint16_t* __restrict__ w, float eps,
                                                    uint16_t* __restrict__ y_norm, int N) {
  __shared__ float red[16];
  const int tid = threadIdx.x, nthr = blockDim.x, n8 = N >> 3;
  const uint16_t* yr = y + (size_t)blockIdx.x * N;
  u32x4 v[C], wv[C];
#pragma unroll
  for (int c = 0; c < C; ++c) {
    const int i = c * nthr + tid;
    v[c] = i < n8 ? ldg16(yr + 8 * i) : u32x4{0, 0, 0, 0};
  }
#pragma unroll
  for (int c = 0; c < C; ++c) {
    const int i = c * nthr + tid;
    wv[c] = i < n8 ? ldg16(w + 8 * i) : u32x4{0, 0, 0, 0};
  }
  float ss = 0.f;
#pragma unroll
  for (int c = 0; c < C; ++c)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float lo = act2f<DT>(v[c][q] & 0xFFFFu), hi = act2f<DT>(v[c][q] >> 16);
      ss += lo * lo;
      ss += hi * hi;
    }
#pragma unroll
  for (int h = 32; h > 0; h >>= 1) ss += __shfl_xor(ss, h);
  if ((tid & 63) == 0) red[tid >> 6] = ss;
  __syncthreads();
  ss = 0.f;
  for (int i = 0; i < nthr >> 6; ++i) ss += red[i];
  const float scale = 1.f / sqrtf(ss / (float)N + eps);
  uint16_t* out = y_norm + (size_t)blockIdx.x * N;
#pragma unroll
  for (int c = 0; c < C; ++c) {
    const int i = c * nthr + tid;
    u32x4 o;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float lo = act2f<DT>(v[c][q] & 0xFFFFu) * scale * act2f<DT>(wv[c][q] & 0xFFFFu);
      const float hi = act2f<DT>(v[c][q] >> 16) * scale * act2f<DT>(wv[c][q] >> 16);
      o[q] = (uint32_t)f2act<DT>(lo) | ((uint32_t)f2act<DT>(hi) << 16);
    }
    if (i < n8) *(u32x4*)(out + 8 * i) = o;
  }
}

// Any other row length: 256 threads, element by element (per-thread strided
// sums, then a tree in LDS).
template <int DT>
__global__ __launch_bounds__(256) void k_rmsnorm(const uint16_t* __restrict__ y,
                                                 const uint16_t* __restrict__ w, float eps,
                                                 uint16_t* __restrict__ y_norm, int N) {
  __shared__ float red[256];
  const int m = blockIdx.x, tid = threadIdx.x;
  const uint16_t* yr = y + (size_t)m * N;
  float ss = 0.f;
  for (int n = tid; n < N; n += 256) {
    const float v = act2f<DT>(yr[n]);
    ss += v * v;
  }
  red[tid] = ss;
  __syncthreads();
  for (int h = 128; h > 0; h >>= 1) {
    if (tid < h) red[tid] += red[tid + h];
    __syncthreads();
  }
  const float scale = 1.f / sqrtf(red[0] / (float)N + eps);
  uint16_t* out = y_norm + (size_t)m * N;
  for (int n = tid; n < N; n += 256) out[n] = f2act<DT>(act2f<DT>(yr[n]) * scale * act2f<DT>(w[n]));
}

// Every workgroup of the fused grid advances its class's launch counter once
// as it ends (see gen_increment): relaxed adds that nothing waits for.
__device__ __forceinline__ unsigned long long* gen_counter(const GemvParams& a, int block) {
  return a.ec.gen + (size_t)(block % kGenClasses) * (kGenStride / 8);
}
__device__ __forceinline__ void fused_exit(const GemvParams& a) {
  const int b = blockIdx.x;
  if (threadIdx.x == 0)
    __hip_atomic_fetch_add(gen_counter(a, b), (unsigned long long)gen_increment(b, a.grid_total),
                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  // classes without a member in a small grid advance with workgroup 0
  if (b == 0 && (int)threadIdx.x >= a.grid_total && (int)threadIdx.x < kGenClasses)
    __hip_atomic_fetch_add(gen_counter(a, threadIdx.x), 1ull << 32, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
}

// ---------------------------------------------------------------------------
// The GEMV's EC wave. In the EC variants every workgroup carries one wave
// beyond its GEMV waves; on the first K-slice it obtains v for each token
// tile and computes v B^T for the workgroup's rows while the GEMV waves
// stream the codes, so its waits (for the producers, for cold caches) stay
// off the critical path. Everything below is single-wave: lanes exchange data
// through LDS in program order, with no workgroup barrier.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void wave_sync() { __builtin_amdgcn_wave_barrier(); }

// dst[i] = fp32 part of the tagged word at off(i), i in [0, n), over the
// wave's 64 lanes; returns 1 (in every lane) if any word carries another tag.
// COH: coherent (sc1) loads, else loads through this XCD's L2, which are
// cheaper but may return a line cached before the data was published (its
// tag then tells). Nine loads per lane go out together (576 words), so that
// the EC data of a token tile at rank 64 (520 words in eight partials) costs
// one round trip, not three; more would push the fused GEMV past its
// 128-VGPR budget into scratch.
template <bool COH, class Off>
__device__ __forceinline__ bool gather_tagged_w(rsrc_t r, int n, Off off, uint32_t tag, float* dst) {
  const int lane = threadIdx.x & 63;
  constexpr int aux = COH ? 0x10 : 0;
  constexpr int U = 9;
  int stale = 0;
  for (int i0 = lane; i0 < n; i0 += 64 * U) {
    u32x2 w[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = i0 + 64 * u;
      w[u] = __builtin_amdgcn_raw_buffer_load_b64(r, i < n ? off(i) : kOOB, 0, aux);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = i0 + 64 * u;
      if (i < n) {
        stale |= w[u][1] != tag;
        dst[i] = __uint_as_float(w[u][0]);
      }
    }
  }
  wave_sync();
  return __any(stale);
}

// u_lds[t][j] = sum_k x[16 tb + t][k] R[j][k] for all R1 rows and all of K,
// by one wave (the EC wave's fallback when the producers' data never came).
template <int DT>
__device__ void ec_project_wave(const EcParams& e, int tb, float* u_lds) {
  const int lane = threadIdx.x & 63, lr = lane & 15, lg = lane >> 4;
  const int IT = e.K / kIterK, RTe = (e.R1 + 15) >> 4;
  const int m = min(tb * kTokTile + lr, e.M - 1);
  const rsrc_t rx = make_rsrc(e.x, (uint32_t)e.M * e.K * 2);
  const bool i8 = e.A8 != nullptr;  // uniform
  const rsrc_t ra = i8 ? make_rsrc(e.A8, (uint32_t)e.r * e.K) : make_rsrc(e.A, (uint32_t)e.r * e.K * 2);
  const rsrc_t rg = make_rsrc(e.wg, e.gate == GATE_SIGMOID ? (uint32_t)e.K * 2 : 0u);
  // K order within an iteration: MFMA jj, lane group lg takes K
  // [8 lg + 32 jj, +8), so that each load reads 64 contiguous bytes per row
  const uint32_t xoff = (uint32_t)m * e.K * 2 + 16 * lg;
  for (int t = 0; t < RTe; ++t) {
    const int j = t * 16 + lr;
    const uint32_t aoff = j < e.r ? (uint32_t)j * e.K * 2 + 16 * lg : kOOB;
    const uint32_t goff = (j == e.r && e.gate == GATE_SIGMOID) ? 16u * lg : kOOB;
    const float saj = i8 && j < e.r ? e.sa[j] : 0.f;
    f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int it = 0; it < IT; ++it) {
      const uint32_t kb = (uint32_t)it * (kIterK * 2);
#pragma unroll
      for (int jj = 0; jj < 4; ++jj) {
        const u32x4 xv = bld128(rx, xoff + kb + 64 * jj);
        u32x4 av;
        if (i8) {
          const u32x2 q = bld64(ra, aoff != kOOB ? (aoff + kb) / 2 + 32 * jj : kOOB);
          av = i8x8_to_act<DT>(q[0], q[1], saj);
        } else {
          av = bld128(ra, aoff != kOOB ? aoff + kb + 64 * jj : kOOB);
        }
        av |= bld128(rg, goff != kOOB ? goff + kb + 64 * jj : kOOB);
        acc = mfma16<DT>(av, xv, acc);
      }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int jr = t * 16 + 4 * lg + i;
      if (jr < e.R1) u_lds[lr * e.R1p + jr] = acc[i];
    }
  }
  wave_sync();
}

// The gate of one token tile by one wave: u_lds [16][R1p] -> v_tile [16][r].
template <int DT>
__device__ void ec_gate_wave(const EcParams& e, int cnt, const float* u_lds, float* hid,
                             float* v_tile) {
  const int lane = threadIdx.x & 63;
  const int r = e.r;
  if (e.gate == GATE_TANH) {
    for (int t = 0; t < cnt; ++t) {
      const float* u = u_lds + t * e.R1p;
      for (int i = lane; i < e.h; i += 64) {
        float a = act2f<DT>(e.b1[i]);
        const uint16_t* w1 = e.W1 + (size_t)i * r;
        for (int j = 0; j < r; ++j) a += act2f<DT>(w1[j]) * u[j];
        hid[i] = a > 0.f ? a : 0.f;
      }
      wave_sync();
      for (int j = lane; j < r; j += 64) {
        float a = act2f<DT>(e.b2[j]);
        const uint16_t* w2 = e.W2 + (size_t)j * e.h;
        for (int i = 0; i < e.h; ++i) a += act2f<DT>(w2[i]) * hid[i];
        v_tile[t * r + j] = e.alpha * (1.f + tanhf(a)) * u[j];
      }
      wave_sync();
    }
  } else {
    for (int idx = lane; idx < cnt * r; idx += 64) {
      const int t = idx / r, j = idx - t * r;
      float g = 1.f;
      if (e.gate == GATE_SIGMOID) {
        const float z = u_lds[t * e.R1p + r] + e.b_g;
        g = z >= 0.f ? 1.f / (1.f + __expf(-z)) : __expf(z) / (1.f + __expf(z));
      }
      v_tile[idx] = e.alpha * g * u_lds[t * e.R1p + j];
    }
    wave_sync();
  }
}

// The EC wave's work for the workgroup's rows n0 .. n0 + 16 RT: for every
// token tile, v (from the previous kernel, or from this grid's producers once
// their ready flags carry this launch's tag, or computed here on time-out),
// then ev = v B^T as two MFMAs per 32 ranks (v split into act-dtype high and
// low parts), stored per (row tile, token tile) in the layout of a GEMV
// wave's accumulators.
template <int DT, int MT, int RT, int EPI>
__device__ void ec_wave(const GemvParams& a, uint32_t gen, char* smem, int n0, bool bpre) {
  const EcParams& e = a.ec;
  const int lane = threadIdx.x & 63, lr = lane & 15, lg = lane >> 4;
  const int M = a.M, N = a.N, r = a.r;
  char* es = smem + a.lds_e;
  float* u_lds = (float*)(es + ec_lds_u_off());
  float* hid = (float*)(es + ec_lds_hid_off(e.R1p));
  float* v_tile = (float*)(es + ec_lds_v_off(e.R1p, e.h));
  const uint16_t* bs = (const uint16_t*)(smem + a.lds_b);
  float* gsc = (float*)(smem + a.lds_g);
  float* evs = (float*)(smem + a.lds_ev);
  const rsrc_t rb = make_rsrc(a.B, (uint32_t)N * r * 2);
  const uint32_t tag = ec_tag(gen);
  const int copy = blockIdx.x % kVCopies;
  const int nkk = (r + 31) / 32;
  // ev = v B^T for token tile mt from v_tile, into the result tiles
  auto up_project = [&](int mt, int cnt) {
    f32x4 ev[RT];
#pragma unroll
    for (int t = 0; t < RT; ++t) ev[t] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int kk = 0; kk < nkk; ++kk) {
      const int j0 = 32 * kk + 8 * lg;
      u32x4 ah, al;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int j = j0 + 2 * q;
        const float f0 = (lr < cnt && j < r) ? v_tile[lr * r + j] : 0.f;
        const float f1 = (lr < cnt && j + 1 < r) ? v_tile[lr * r + j + 1] : 0.f;
        const uint32_t h0 = f2act<DT>(f0), h1 = f2act<DT>(f1);
        ah[q] = h0 | (h1 << 16);
        al[q] = (uint32_t)f2act<DT>(f0 - act2f<DT>(h0)) |
                ((uint32_t)f2act<DT>(f1 - act2f<DT>(h1)) << 16);
      }
#pragma unroll
      for (int t = 0; t < RT; ++t) {
        const int row = 16 * t + lr, n = n0 + row;
        u32x4 bf;
        if (bpre && (r & 7) == 0 && j0 < r) {
          bf = *(const u32x4*)(bs + row * r + j0);
        } else {
          auto bval = [&](int j) -> uint32_t {
            if (n >= N || j >= r) return 0u;
            if (a.B8) return i8_to_act<DT>(a.B8[(size_t)n * r + j], a.sb[n]);
            return bpre ? (uint32_t)bs[row * r + j] : bld16(rb, (uint32_t)(n * r + j) * 2);
          };
#pragma unroll
          for (int q = 0; q < 4; ++q) bf[q] = bval(j0 + 2 * q) | (bval(j0 + 2 * q + 1) << 16);
        }
        ev[t] = mfma16<DT>(ah, bf, ev[t]);
        ev[t] = mfma16<DT>(al, bf, ev[t]);
      }
    }
#pragma unroll
    for (int t = 0; t < RT; ++t) *(f32x4*)(evs + ((t * MT + mt) * 64 + lane) * 4) = ev[t];
    wave_sync();
  };

  if constexpr (EPI == EPI_READY) {
    for (int mt = 0; mt < MT; ++mt) {
      const int m0 = 16 * mt, cnt = min(16, M - m0);
      for (int idx = lane; idx < cnt * r; idx += 64) v_tile[idx] = e.v[(size_t)m0 * r + idx];
      wave_sync();
      up_project(mt, cnt);
    }
    return;
  }

  // Fused: one attempt reads the published data of token tile mt (tagged
  // words), completes v and its product, and tells whether every word was
  // current; a stale attempt still runs the whole path, which warms this
  // wave's caches while the producers finish. `dry` reads nothing.
  auto attempt = [&](int mt, int cnt, bool coh, bool dry) -> bool {
    const int m0 = 16 * mt;
    bool stale;
    if (e.mode == EC_GATHER) {
      const int per = cnt * e.R1;
      const size_t per_copy = (size_t)e.P * e.M * e.R1;
      const rsrc_t rv = make_rsrc(e.vtag + copy * per_copy, (uint32_t)(per_copy * 8));
      auto off = [&](int i) {
        const int q = i / per, o = i - q * per;
        return (uint32_t)(((size_t)q * e.M + m0) * e.R1 + o) * 8u;
      };
      const int n = dry ? 0 : e.P * per;
      stale = dry || (coh ? gather_tagged_w<true>(rv, n, off, tag, gsc)
                          : gather_tagged_w<false>(rv, n, off, tag, gsc));
      for (int idx = lane; idx < per; idx += 64) {
        float sum = 0.f;
        for (int q = 0; q < e.P; ++q) sum += gsc[q * per + idx];
        const int t = idx / e.R1, j = idx - t * e.R1;
        u_lds[t * e.R1p + j] = sum;
      }
      wave_sync();
      ec_gate_wave<DT>(e, cnt, u_lds, hid, v_tile);
    } else {
      const size_t per_copy = (size_t)e.M * r;
      const rsrc_t rv = make_rsrc(e.vtag + copy * per_copy, (uint32_t)(per_copy * 8));
      auto off = [&](int i) { return (uint32_t)((size_t)m0 * r + i) * 8u; };
      const int n = dry ? 0 : cnt * r;
      stale = dry || (coh ? gather_tagged_w<true>(rv, n, off, tag, v_tile)
                          : gather_tagged_w<false>(rv, n, off, tag, v_tile));
    }
    up_project(mt, cnt);
    return !stale;
  };

  // warm-up pass, then wait: small problems poll the tagged data itself;
  // the others wait (bounded) for this copy's ready counter to show every
  // publisher of this launch and then read the data once through the L2,
  // re-reading it coherently if a cached line was stale. (Coherent reads
  // from every EC wave at once were measured: hundreds of waves reading the
  // same few lines at the memory side delay the producers' own stores, 70B
  // q 44.7 us against 18.7 us.)
  bool ok = true;
  if (!e.direct) {
    attempt(0, min(16, M), false, true);
    const unsigned long long* rc = e.ready + copy * (kReadyStride / 8);
    const rsrc_t rr = make_rsrc(rc, 8);
    const unsigned long long goal = ((unsigned long long)gen + 1ull) << 32;
    for (int poll = 0;; ++poll) {
      const u32x2 c = bld64c(rr, 0u);
      const unsigned long long cv = ((unsigned long long)c[1] << 32) | c[0];
      // counts of this launch lie in [goal - 2^32, goal]; the difference is
      // taken modulo 2^64 so that wrap-around is harmless
      if ((long long)(cv - goal) >= 0) break;
      if (poll >= a.wait_polls) { ok = false; break; }
      __builtin_amdgcn_s_sleep(16);
    }
  }
  for (int mt = 0; mt < MT; ++mt) {
    const int cnt = min(16, M - 16 * mt);
    bool have = false;
    if (e.direct) {
      for (int k = 0; k <= a.wait_polls && !have; ++k) {
        have = attempt(mt, cnt, true, false);
        if (!have) __builtin_amdgcn_s_sleep(4);
      }
    } else if (ok) {
      have = attempt(mt, cnt, false, false) || attempt(mt, cnt, true, false);
    }
    if (!have) {
      ec_project_wave<DT>(e, mt, u_lds);
      ec_gate_wave<DT>(e, cnt, u_lds, hid, v_tile);
      up_project(mt, cnt);
    }
  }
}

// ---------------------------------------------------------------------------
// Decode GEMV. A block owns RT row tiles (16 rows each) and a K-slice of
// iterations (128 K each); each of its NW waves walks a contiguous chunk of
// that slice as a software pipeline: the codes of iteration it+1 are in
// flight while iteration it is computed. The block's slice of x is staged in
// LDS once when it fits (else read through the cache per iteration), and so
// are the scales and zero points of its rows. The MFMA multiplies
// activations (A operand, 16 token rows) by the biased codes (B operand, 16
// weight rows as columns), so each lane owns one weight row per tile and
// needs one scale and one zero point per iteration:
//   sum_k x (q - z) s = s * ( sum_k x (bias + q) - (bias + z) * sum_k x ),
// with sum_k x from an MFMA against ones, shared by the RT tiles.
// In the EC variants the block has one more wave, the EC wave (above), whose
// v B^T tiles join the waves' partial tiles in the fixed-order reduction of
// the first K-slice. K-slices are reduced through partial sums and a last
// arriver.
//
// Fused variant: the first n_prod blocks of the grid are EC producers; the
// others' EC waves wait for what they publish.
//
// SPLIT: with the split-K reduction. Calls of one token tile in one K-slice run
// a build without it: its code, though never reached there, changed the
// registers and the schedule of the whole kernel (local variant 2048 x 2048, rank
// 16, bf16, one token: 8.4 us with it, 7.4 without; 4-bit product 8192 x 8192 at
// one token 12.0 and 11.5; producer-fused 8192 x 8192, rank 32, 18.0 and 17.3).
// ---------------------------------------------------------------------------
template <int DT, int MT, int RT, int EPI, int WB, int NST, bool SPLIT>
__device__ __forceinline__ void gemv_body(const GemvParams& a, int bid, uint32_t gen, char* smem) {
  __shared__ int s_flag;
  constexpr bool kEC = EPI == EPI_READY || EPI == EPI_FUSED;  // with an EC wave
  constexpr bool kLoc = EPI == EPI_LOCAL || EPI == EPI_LOCAL_I8;
  constexpr bool kI8 = EPI == EPI_LOCAL_I8;  // INT8 A and B
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform
  const int NW = (blockDim.x >> 6) - (kEC ? 1 : 0);           // GEMV waves
  const bool gw = wave < NW;
  const int lr = lane & 15, lg = lane >> 4;
  constexpr int RB = 16 * RT;
  const int M = a.M, N = a.N, K = a.K, G = a.G;
  const int IT = K / kIterK;
  const int S = SPLIT ? a.S : 1;
  const int rg = bid / S, s = bid - rg * S;
  const int n0 = rg * RB;
  const int it_blk = s * a.ips;
  const int it_end = min(IT, it_blk + a.ips);
  const int iw_beg = gw ? it_blk + wave * a.iw : 0;
  const int iw_end = gw ? min(it_end, iw_beg + a.iw) : 0;
  const int r = a.r;

  const rsrc_t rq = make_rsrc(a.qw, (uint32_t)N * row_code_bytes<WB>(K));
  const rsrc_t rsc = make_rsrc(a.sc, (uint32_t)N * a.ngroups * 2);
  const rsrc_t rz = make_rsrc(a.zr, (uint32_t)N * a.ngroups);
  const rsrc_t rx = make_rsrc(a.x, (uint32_t)M * K * 2);
  const rsrc_t rb = kI8 ? make_rsrc(a.B8, (uint32_t)N * r) : make_rsrc(a.B, (uint32_t)N * r * 2);

  // The residual of the post-EC tail: when the block's outputs are at most
  // one per thread (decode), each thread's element is fetched here with the
  // other prologue loads instead of right before its store. The load is
  // issued unconditionally (out of range, it reads nothing): a branch around
  // it would make the wait before the first compute cover every prologue load.
  const bool res_pre = a.res != nullptr && RB * M <= (int)blockDim.x;
  uint32_t resv;
  {
    const int m = tid / RB, row = tid - (tid / RB) * RB;
    const rsrc_t rres = make_rsrc(a.res, a.res ? (uint32_t)M * N * 2 : 0u);
    resv = bld16(rres, res_pre && tid < RB * M && n0 + row < N
                           ? ((uint32_t)m * N + n0 + row) * 2 : kOOB);
  }
  // the rows of B ([RB][r], contiguous) of the block that adds v B^T (the
  // first K-slice's with an EC wave; any slice's in EPI_LOCAL, whose last
  // arriver adds it) are fetched up front into LDS when two 16-byte chunks
  // per thread cover them
  // (INT8 B: the codes, 16 per chunk, and then the rows' fp32 scales)
  constexpr int BCH = 2;
  const bool bpre = ((kEC && s == 0) || kLoc) && a.bpre;
  const int bchunks = kI8 ? RB * r / 16 : RB * r / 8;
  u32x4 bst[BCH];
  uint32_t sbst = 0;
  if (bpre) {
#pragma unroll
    for (int c = 0; c < BCH; ++c) {
      const int ci = tid + c * (int)blockDim.x;
      bst[c] = bld128(rb, ci < bchunks ? (uint32_t)n0 * r * (kI8 ? 1 : 2) + 16u * ci : kOOB);
    }
    if constexpr (kI8) {
      const rsrc_t rsb = make_rsrc(a.sb, (uint32_t)N * 4);
      sbst = __builtin_amdgcn_raw_buffer_load_b32(rsb, tid < RB ? (uint32_t)(n0 + tid) * 4 : kOOB, 0, 0);
    }
  }

  // per-lane parts of the load offsets (row, token, lane group; kOOB for
  // rows >= N); the iteration enters as a wave-uniform soffset. Token rows
  // past M read row M-1: their MFMA rows only feed outputs that are never
  // stored, and in-bounds duplicates cost the address unit far less than
  // masked lanes.
  uint32_t vw[RT], vx[MT];
#pragma unroll
  for (int t = 0; t < RT; ++t) {
    const int n = n0 + 16 * t + lr;
    // lane group lg: the codes of K [32 lg, 32 lg + 32) of each iteration
    // (4-bit: 16 bytes, 3-bit: one block of 12)
    vw[t] = n < N ? (uint32_t)n * row_code_bytes<WB>(K) + (WB == 4 ? 16 : 12) * lg : kOOB;
  }
  const bool xl = a.xlds;
  const char* xs = smem;
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    const int m = min(16 * mt + lr, M - 1);
    vx[mt] = xl ? (uint32_t)m * a.xstride + 64 * lg : ((uint32_t)m * K + 32 * lg) * 2;
  }
  auto load_w = [&](u32x4 (&w)[RT], int it) {
#pragma unroll
    for (int t = 0; t < RT; ++t)
      w[t] = WB == 4 ? bld128s(rq, vw[t], (uint32_t)it * (kIterK / 2))
                     : bld96s(rq, vw[t], (uint32_t)it * (kIterK / 8 * 3));
  };
  // EPI_LOCAL: the block's K-slice of A (16 rows, rows >= r zero) and of
  // w_g (row 16) is staged in LDS with coalesced 16-byte chunks: read in the
  // MFMA lane layout straight from memory, every load would touch 32 cache
  // lines. The MFMAs then take A's rows (lane lr: row lr) and w_g in every
  // column as two further B operands.
  // INT8 A: eight codes (8 bytes) per chunk, staged as exact integers; the
  // rows' scales multiply the fp32 projection sums instead. The thread that
  // reduces column c of the projection tiles always has c = (lane / 4) % 16
  // (the block is a whole number of waves), so it holds that row's scale.
  const rsrc_t ra = kI8 ? make_rsrc(a.ec.A8, (uint32_t)r * K)
                        : make_rsrc(kLoc ? a.ec.A : nullptr, kLoc ? (uint32_t)r * K * 2 : 0u);
  const rsrc_t rgw = make_rsrc(kLoc ? a.ec.wg : nullptr,
                               kLoc && a.ec.gate == GATE_SIGMOID ? (uint32_t)K * 2 : 0u);
  // (a buffer load: a flat load would also hold the LDS counter the
  // prologue's barriers wait on)
  float sa_c = 1.f;
  if constexpr (kI8) {
    const rsrc_t rsa = make_rsrc(a.ec.sa, (uint32_t)r * 4);
    sa_c = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(
        rsa, ((lane >> 2) & 15) < r ? (uint32_t)((lane >> 2) & 15) * 4 : kOOB, 0, 0));
  }
  const int acpr = (it_end - it_blk) * (kIterK / 8);  // 16-byte chunks per row
  const int astride = acpr * 8 + 8;                   // LDS row stride (halves)
  uint16_t* als = (uint16_t*)(smem + a.lds_a);        // [17][astride]
  auto a_issue = [&](int base, u32x4 (&c4)[4]) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int ci = base + u * (int)blockDim.x;
      const int row = ci / acpr, kc = ci - row * acpr;
      const bool ok = ci < 16 * acpr && row < r;
      if constexpr (kI8) {
        const u32x2 q = bld64(ra, ok ? (uint32_t)row * K + it_blk * kIterK + 8 * kc : kOOB);
        c4[u] = u32x4{q[0], q[1], 0u, 0u};
      } else {
        c4[u] = bld128(ra, ok ? ((uint32_t)row * K + it_blk * kIterK + 8 * kc) * 2 : kOOB);
      }
    }
  };
  auto a_store = [&](int base, const u32x4 (&c4)[4]) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int ci = base + u * (int)blockDim.x;
      const int row = ci / acpr, kc = ci - row * acpr;
      u32x4 v = c4[u];
      if constexpr (kI8) v = i8x8_exact<DT>(v[0], v[1]);
      if (ci < 16 * acpr) *(u32x4*)(als + row * astride + 8 * kc) = v;
    }
  };
  auto load_x = [&](u32x4 (&xv)[MT][4], int it) {
    if (xl) {
      const uint32_t kb = (uint32_t)(it - it_blk) * (kIterK * 2);
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) xv[mt][jj] = *(const u32x4*)(xs + vx[mt] + kb + 16 * jj);
    } else {
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int jj = 0; jj < 4; ++jj)
          xv[mt][jj] = bld128s(rx, vx[mt] + 16 * jj, (uint32_t)it * (kIterK * 2));
    }
  };

  // Every global load of the prologue is issued before the first wait: the
  // rows of B, the block's slice of x, the scales and zero points, then the
  // first two pipeline stages of codes. Small layers give a wave one or two
  // iterations, so the prologue's round trips are most of the kernel.
  // NST stages of codes in flight per wave: two alternating register sets,
  // or (NST > 2, for long K-slices on wide layers) a ring of NST sets with
  // the activations read right before each iteration (from LDS when staged)
  u32x4 wA[RT], wB[RT];
  u32x4 xA[MT][4], xB[MT][4];
  u32x4 wR[NST > 2 ? NST : 1][RT];
  const int last = iw_end - 1;
  // the block's slice of x into LDS ([M][slice] with a padded row stride),
  // four 16-byte chunks per thread per round
  const int cpr = (it_end - it_blk) * (kIterK / 8);  // 16-byte chunks per row
  const int nch = xl ? M * cpr : 0;
  auto x_issue = [&](int base, u32x4 (&c4)[4]) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int ci = base + u * (int)blockDim.x;
      const int m = ci / cpr, kc = ci - m * cpr;
      c4[u] = bld128(rx, ci < nch ? ((uint32_t)m * K + it_blk * kIterK + 8 * kc) * 2 : kOOB);
    }
  };
  auto x_store = [&](int base, const u32x4 (&c4)[4]) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int ci = base + u * (int)blockDim.x;
      const int m = ci / cpr, kc = ci - m * cpr;
      if (ci < nch) *(u32x4*)(smem + (size_t)m * a.xstride + 16 * kc) = c4[u];
    }
  };
  // scales and zero points of the block's rows and groups, staged once in
  // LDS with coalesced loads ([row][group] as s | z << 16): per-iteration
  // scattered 2- and 1-byte loads would cost a cache-line request per row
  const int ipg = G / kIterK;  // iterations per quantisation group
  const int g_lo = it_blk / ipg;
  const int ngb = (it_end - 1) / ipg + 1 - g_lo;
  const int ngs = ngb | 1;  // odd LDS row stride: rows fall on distinct banks
  uint32_t* szs = (uint32_t*)(smem + a.lds_sz);
  const int nsz = RB * ngb;
  auto sz_issue = [&](int i0, uint32_t (&sv)[4], uint32_t (&zv)[4]) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int idx = i0 + u * (int)blockDim.x;
      const int row = idx / ngb, gg = idx - row * ngb;
      const uint32_t eo = (uint32_t)(n0 + row) * a.ngroups + g_lo + gg;
      const bool ok = idx < nsz && n0 + row < N;
      sv[u] = bld16(rsc, ok ? eo * 2 : kOOB);
      zv[u] = bld8(rz, ok ? eo : kOOB);
    }
  };
  auto sz_store = [&](int i0, const uint32_t (&sv)[4], const uint32_t (&zv)[4]) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int idx = i0 + u * (int)blockDim.x;
      if (idx < nsz) {
        const int row = idx / ngb, gg = idx - row * ngb;
        szs[row * ngs + gg] = sv[u] | (zv[u] << 16);
      }
    }
  };
  // eight groups per 16-byte scale load and 8-byte zero load when the
  // block's group range is 8-aligned (2- and 1-byte loads per entry would be
  // a third of the block's load instructions for a few percent of its bytes)
  const bool sz8 = (a.ngroups & 7) == 0 && (g_lo & 7) == 0 && (ngb & 7) == 0;
  const int c8 = ngb >> 3, nsz8 = RB * c8;
  auto sz8_issue = [&](int i, u32x4& s8, u32x2& z8) {
    const int row = i / c8, q = i - row * c8;
    const bool ok = i < nsz8 && n0 + row < N;
    const uint32_t eo = (uint32_t)(n0 + row) * a.ngroups + g_lo + 8 * q;
    s8 = bld128(rsc, ok ? eo * 2 : kOOB);
    z8 = bld64(rz, ok ? eo : kOOB);
  };
  auto sz8_store = [&](int i, const u32x4& s8, const u32x2& z8) {
    if (i < nsz8) {
      const int row = i / c8, q = i - row * c8;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const uint32_t sv = (s8[e >> 1] >> (16 * (e & 1))) & 0xFFFFu;
        const uint32_t zv = (z8[e >> 2] >> (8 * (e & 3))) & 0xFFu;
        szs[row * ngs + 8 * q + e] = sv | (zv << 16);
      }
    }
  };
  {
    const int step = 4 * (int)blockDim.x;
    u32x4 c4[4];
    uint32_t sv[4], zv[4];
    u32x4 s8;
    u32x2 z8;
    // EPI_LOCAL: the first round of A and w_g goes out with the first round
    // of x, scales and zero points, so that the staging costs one round
    // trip. The second round of x and of the 8-group scales goes out with
    // the first too (a deep slice, 28672 wide, needs two), except in the
    // producer-fused variant, whose 22 more VGPRs there would cost it the
    // second workgroup per CU.
    constexpr bool kTwo = EPI != EPI_FUSED;
    u32x4 a0[4], a1[4], gv0;
    u32x4 c4b[4], s8b;
    u32x2 z8b;
    x_issue(tid, c4);
    if constexpr (kTwo) x_issue(tid + step, c4b);
    if (sz8) {
      sz8_issue(tid, s8, z8);
      if constexpr (kTwo) sz8_issue(tid + (int)blockDim.x, s8b, z8b);
    } else {
      sz_issue(tid, sv, zv);
    }
    if constexpr (kLoc) {
      a_issue(tid, a0);
      a_issue(tid + step, a1);
      gv0 = bld128(rgw, tid < acpr ? ((uint32_t)it_blk * kIterK + 8 * tid) * 2 : kOOB);
    }
    // the first code stages go out after the staging loads: the counter
    // retires in order, so the LDS stores below wait only for x, the scales
    // and A (L2-resident after the first workgroups), not for the codes
    // coming from HBM (70B q, k, v as one launch: 17.7 -> 16.9 us)
    if (iw_beg < iw_end) {
      if constexpr (NST > 2) {
#pragma unroll
        for (int q = 0; q < NST; ++q) load_w(wR[q], min(iw_beg + q, last));
      } else {
        load_w(wA, iw_beg);
        if (!xl) load_x(xA, iw_beg);
        load_w(wB, min(iw_beg + 1, last));
        if (!xl) load_x(xB, min(iw_beg + 1, last));
      }
    }
    x_store(tid, c4);
    if constexpr (kTwo) x_store(tid + step, c4b);
    if (sz8) {
      sz8_store(tid, s8, z8);
      if constexpr (kTwo) sz8_store(tid + (int)blockDim.x, s8b, z8b);
    } else {
      sz_store(tid, sv, zv);
    }
    if constexpr (kLoc) {
      a_store(tid, a0);
      a_store(tid + step, a1);
      if (tid < acpr) *(u32x4*)(als + 16 * astride + 8 * tid) = gv0;
    }
    for (int base = tid + (kTwo ? 2 : 1) * step; base < nch; base += step) {
      x_issue(base, c4);
      x_store(base, c4);
    }
    if (sz8) {
      for (int i = tid + (kTwo ? 2 : 1) * (int)blockDim.x; i < nsz8; i += blockDim.x) {
        sz8_issue(i, s8, z8);
        sz8_store(i, s8, z8);
      }
    } else {
      for (int i0 = tid + step; i0 < nsz; i0 += step) {
        sz_issue(i0, sv, zv);
        sz_store(i0, sv, zv);
      }
    }
    if constexpr (kLoc) {
      // the rest of A: two rounds of four chunks per thread in flight; of
      // w_g: one chunk
      for (int base = tid + 2 * step; base < 16 * acpr; base += 2 * step) {
        a_issue(base, a0);
        a_issue(base + step, a1);
        a_store(base, a0);
        a_store(base + step, a1);
      }
      for (int kc = tid + (int)blockDim.x; kc < acpr; kc += blockDim.x) {
        const u32x4 gv = bld128(rgw, ((uint32_t)it_blk * kIterK + 8 * kc) * 2);
        *(u32x4*)(als + 16 * astride + 8 * kc) = gv;
      }
    }
  }
  uint16_t* bs = (uint16_t*)(smem + a.lds_b);
  if (bpre) {
#pragma unroll
    for (int c = 0; c < BCH; ++c) {
      const int ci = tid + c * (int)blockDim.x;
      if (ci < bchunks) *(u32x4*)(bs + 8 * ci) = bst[c];
    }
    if constexpr (kI8) {
      if (tid < RB) ((uint32_t*)((char*)bs + RB * r))[tid] = sbst;
    }
  }
  __syncthreads();
  if (NST == 2 && xl && iw_beg < iw_end) {
    load_x(xA, iw_beg);
    load_x(xB, min(iw_beg + 1, last));
  }

  constexpr float kBias = code_bias<DT>();
  f32x4 acc[RT][MT];
#pragma unroll
  for (int t = 0; t < RT; ++t)
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) acc[t][mt] = f32x4{0.f, 0.f, 0.f, 0.f};
  const uint32_t km = opaque_v(0x000F000Fu);
  const uint32_t kg = opaque_v(DT == DT_F16 ? 0x64006400u : 0x43004300u);
  f32x4 eacc[kLocalTiles][MT];
#pragma unroll
  for (int t = 0; t < kLocalTiles; ++t)
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) eacc[t][mt] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto compute = [&](const u32x4 (&w)[RT], const u32x4 (&xv)[MT][4], int it) {
    if constexpr (kLoc) {
      // A x and w_g x: activations (A operand, token rows) times the rows of
      // A / copies of w_g (B operand, one per column) from LDS, accumulated
      // over the wave's chunk
      const int kb = (it - it_blk) * kIterK + 32 * lg;
#pragma unroll
      for (int jj = 0; jj < 4; ++jj) {
        const u32x4 af = *(const u32x4*)(als + lr * astride + kb + 8 * jj);
        const u32x4 gf = *(const u32x4*)(als + 16 * astride + kb + 8 * jj);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
          eacc[0][mt] = mfma16<DT>(xv[mt][jj], af, eacc[0][mt]);
          eacc[1][mt] = mfma16<DT>(xv[mt][jj], gf, eacc[1][mt]);
        }
      }
    }
    f32x4 xb[MT];
    u32x4 xp[MT][4];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      xb[mt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int jj = 0; jj < 4; ++jj) {
        xb[mt] = mfma16<DT>(xv[mt][jj], ones8<DT>(), xb[mt]);
        // 4-bit codes pair (q_i, q_{i+4}) within a word: the activations
        // follow; 3-bit pairs are in natural order
        xp[mt][jj] = WB == 4 ? pair_like_codes(xv[mt][jj]) : xv[mt][jj];
      }
    }
    const int gg = it / ipg - g_lo;
#pragma unroll
    for (int t = 0; t < RT; ++t) {
      u32x4 wd[4];
#pragma unroll
      for (int jj = 0; jj < 4; ++jj)
        wd[jj] = WB == 4 ? unpack_biased_r(w[t][jj], km, kg) : unpack3_biased(w[t], jj, kg);
      const uint32_t sz = szs[(16 * t + lr) * ngs + gg];
      const float sf = h2f((uint16_t)(sz & 0xFFFF));
      const float cf = kBias + (float)(sz >> 16);
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        f32x4 pacc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) pacc = mfma16<DT>(xp[mt][jj], wd[jj], pacc);
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[t][mt][i] += sf * (pacc[i] - cf * xb[mt][i]);
      }
    }
  };

  // software pipeline over this wave's iterations: batch it+1 is in flight
  // while batch it is computed (two register sets, alternating, both filled
  // by the prologue). Loads past the wave's last iteration re-read that
  // iteration (never computed), so every load is unconditional.
  if (NST > 2 && iw_beg < iw_end) {
    for (int it = iw_beg; it < iw_end; it += NST) {
#pragma unroll
      for (int q = 0; q < NST; ++q) {
        if (it + q < iw_end) {  // uniform
          u32x4 xv[MT][4];
          load_x(xv, it + q);
          compute(wR[q], xv, it + q);
          load_w(wR[q], min(it + q + NST, last));
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
  } else if (iw_beg < iw_end) {
    for (int it = iw_beg; it < iw_end; it += 2) {
      compute(wA, xA, it);
      if (it + 1 >= iw_end) break;
      load_w(wA, min(it + 2, last));
      load_x(xA, min(it + 2, last));
      __builtin_amdgcn_sched_barrier(0);
      compute(wB, xB, it + 1);
      load_w(wB, min(it + 3, last));
      load_x(xB, min(it + 3, last));
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  if constexpr (kEC) {
    if (!gw && s == 0) ec_wave<DT, MT, RT, EPI>(a, gen, smem, n0, bpre);
  }
  if (xl) __syncthreads();  // the x region is reused below

  // ---- cross-wave reduction (fixed order) into yacc[token][row]; the EC
  // wave's tiles come last
  float* red = (float*)smem;
  float* ered = red + NW * RT * MT * 256;  // EPI_LOCAL: [NW][kLocalTiles][MT] tiles
  if (gw) {
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
        *(f32x4*)(red + (((wave * RT + t) * MT + mt) * 64 + lane) * 4) = acc[t][mt];
    if constexpr (kLoc) {
#pragma unroll
      for (int t = 0; t < kLocalTiles; ++t)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
          *(f32x4*)(ered + (((wave * kLocalTiles + t) * MT + mt) * 64 + lane) * 4) = eacc[t][mt];
    }
  }
  __syncthreads();
  // EPI_LOCAL: this block's [A; w_g] x (its K-slice), u [token][R1p] in LDS
  float* u_loc = (float*)(smem + a.lds_e);
  const int R1 = a.ec.R1, R1p = a.ec.R1p;
  // Without split-K the sums are complete here: each thread that owns u_j of
  // a token also sums that token's gate logit and writes v_j directly
  // (EPI_LOCAL, below), saving a pass and a barrier.
  float* v_loc = u_loc + 16 * MT * R1p;
  const bool v_direct = S == 1 && a.ec.gate != GATE_TANH;
  if constexpr (kLoc) {
    // tile 0: column j < r is u_j; tile 1: column 0 is the gate logit w_g x
    for (int e = tid; e < 256 * kLocalTiles * MT; e += blockDim.x) {
      const int tm = e >> 8, rem = e & 255, ln = rem >> 2, i = rem & 3;
      const int t = tm / MT, mt = tm - t * MT;
      const int tok = 16 * mt + 4 * (ln >> 4) + i, c = ln & 15;
      const int j = t == 0 ? (c < r ? c : -1) : (c == 0 && R1 > r ? r : -1);
      if (j < 0 || (v_direct && t != 0)) continue;
      float v = 0.f;
      for (int w = 0; w < NW; ++w) v += ered[(((w * kLocalTiles + t) * MT + mt) * 64 + ln) * 4 + i];
      if constexpr (kI8) {
        if (t == 0) v *= sa_c;  // c == (lane / 4) % 16 here
      }
      if (v_direct) {
        float g = 1.f;
        if (a.ec.gate == GATE_SIGMOID) {
          float zl = 0.f;  // the logit: tile 1, column 0, same token
          for (int w = 0; w < NW; ++w)
            zl += ered[(((w * kLocalTiles + 1) * MT + mt) * 64 + (ln & 48)) * 4 + i];
          const float z = zl + a.ec.b_g;
          g = z >= 0.f ? 1.f / (1.f + __expf(-z)) : __expf(z) / (1.f + __expf(z));
        }
        v_loc[tok * r + j] = a.ec.alpha * g * v;
      } else {
        u_loc[tok * R1p + j] = v;
      }
    }
  }
  float* yacc = (float*)(smem + a.lds_y);
  const float* evs = (const float*)(smem + a.lds_ev);
  const bool add_ev = kEC && s == 0;
  constexpr int YS = RB;  // yacc row stride: [token][RB rows]
  for (int e = tid; e < 256 * RT * MT; e += blockDim.x) {
    const int tm = e >> 8, rem = e & 255, ln = rem >> 2, i = rem & 3;
    const int t = tm / MT, mt = tm - t * MT;
    float v = 0.f;
    for (int w = 0; w < NW; ++w) v += red[(((w * RT + t) * MT + mt) * 64 + ln) * 4 + i];
    if (add_ev) v += evs[((t * MT + mt) * 64 + ln) * 4 + i];
    const int tok = 16 * mt + 4 * (ln >> 4) + i, row = 16 * t + (ln & 15);
    yacc[tok * YS + row] = v;
  }
  __syncthreads();

  // ---- cross-block split-K reduction: the last arriver sums the slices in order
  // (the local variant is faster with it out of the straight line, 2048 x 8192,
  // rank 16, at 16 tokens in several slices 14.5 us against 14.7)
  if (kLoc ? __builtin_expect(S > 1, 0) : S > 1) {
    for (int e = tid; e < RB * M; e += blockDim.x) {
      const int m = e / RB, row = e - m * RB;
      if (n0 + row < N) st_agent(a.ypart + ((size_t)s * M + m) * N + n0 + row, yacc[m * YS + row]);
    }
    if constexpr (kLoc) {
      // the slice's partial [A; w_g] x, for the last arriver of this row
      // group (which waits for this row group's slices only)
      for (int e = tid; e < M * R1; e += blockDim.x) {
        const int m = e / R1, j = e - m * R1;
        st_agent(a.eupart + ((size_t)(rg * a.S + s) * M + m) * R1 + j, u_loc[m * R1p + j]);
      }
    }
    complete_and_sync();
    if (tid == 0) s_flag = arrive_last(a.rb_ctr + rg, (uint32_t)a.S) ? 1 : 0;
    __syncthreads();
    if (!s_flag) {
      if constexpr (EPI == EPI_FUSED) fused_exit(a);
      return;
    }
    // every slice's [M][RB] partial, summed in slice order
    const rsrc_t rp = make_rsrc(a.ypart, (uint32_t)a.S * M * N * 4);
    sum_slices<4>(rp, a.S, M * RB, [&](int q, int i) {
      const int m = i / RB, row = i - m * RB;
      return n0 + row < N ? (uint32_t)(((size_t)q * M + m) * N + n0 + row) * 4u : kOOB;
    }, [&](int i, float v) {
      const int m = i / RB, row = i - m * RB;
      yacc[m * YS + row] = v;
    });
    if constexpr (kLoc) {
      // this row group's slices' [A; w_g] x, summed in slice order
      const rsrc_t re = make_rsrc(a.eupart, (uint32_t)((size_t)a.N / RB + 1) * a.S * M * R1 * 4);
      sum_slices<4>(re, a.S, M * R1, [&](int q, int i) {
        return (uint32_t)(((size_t)(rg * a.S + q) * M) * R1 + i) * 4u;
      }, [&](int i, float v) {
        const int m = i / R1, j = i - m * R1;
        u_loc[m * R1p + j] = v;
      });
    }
  }

  // EPI_LOCAL: v = alpha g(x) (.) A x for every token (g the sigmoid of the
  // gate row's sum plus b_g, or one; or the tanh-MLP gate of u, whose hidden
  // layer takes the LDS after v), then y += v B^T in fp32 below
  if (kLoc && !v_direct &&
      (SPLIT ? __builtin_expect(a.ec.gate == GATE_TANH, 0) : a.ec.gate == GATE_TANH)) {
    // LDS after v: the hidden layer (cap x h floats)
    tanh_gate_tokens<DT>(M, r, a.ec.h, u_loc, R1p, a.ec.W1, a.ec.b1, a.ec.W2, a.ec.b2, a.ec.alpha,
                         v_loc + 16 * MT * r, local_tanh_cap(M, a.ec.h), v_loc, r);
  } else if (kLoc && !v_direct) {
    for (int idx = tid; idx < M * r; idx += blockDim.x) {
      const int m = idx / r, j = idx - m * r;
      float g = 1.f;
      if (a.ec.gate == GATE_SIGMOID) {
        const float z = u_loc[m * R1p + r] + a.ec.b_g;
        g = z >= 0.f ? 1.f / (1.f + __expf(-z)) : __expf(z) / (1.f + __expf(z));
      }
      v_loc[idx] = a.ec.alpha * g * u_loc[m * R1p + j];
    }
    __syncthreads();
  }
  const uint16_t* bsl = (const uint16_t*)(smem + a.lds_b);

  for (int e = tid; e < RB * M; e += blockDim.x) {
    const int m = e / RB, row = e - m * RB;
    if (n0 + row < N) {
      float v = yacc[m * YS + row];
      if constexpr (kLoc) {
        // v B^T for this row: eight ranks per 16-byte chunk of the staged row
        // of B (r is a multiple of 8 when B is staged), independent loads
        const float* vm = v_loc + m * r;
        float ev = 0.f;
        if (bpre && kI8) {
          // INT8 B staged: the codes and the row's scale exactly, in fp32
          const int8_t* b8row = (const int8_t*)bsl + row * r;
          for (int j0 = 0; j0 < r; j0 += 8) {
            const u32x2 q = *(const u32x2*)(b8row + j0);
            const f32x4 v0 = *(const f32x4*)(vm + j0), v1 = *(const f32x4*)(vm + j0 + 4);
#pragma unroll
            for (int e2 = 0; e2 < 4; ++e2) {
              ev += v0[e2] * (float)((int)(q[0] << (24 - 8 * e2)) >> 24);
              ev += v1[e2] * (float)((int)(q[1] << (24 - 8 * e2)) >> 24);
            }
          }
          ev *= ((const float*)((const char*)bsl + RB * r))[row];
        } else if (bpre) {
          for (int j0 = 0; j0 < r; j0 += 8) {
            const u32x4 b8 = *(const u32x4*)(bsl + row * r + j0);
            const f32x4 v0 = *(const f32x4*)(vm + j0), v1 = *(const f32x4*)(vm + j0 + 4);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              const float vlo = q < 2 ? v0[2 * q] : v1[2 * q - 4];
              const float vhi = q < 2 ? v0[2 * q + 1] : v1[2 * q - 3];
              ev += vlo * act2f<DT>((uint16_t)(b8[q] & 0xFFFFu)) + vhi * act2f<DT>((uint16_t)(b8[q] >> 16));
            }
          }
        } else if constexpr (kI8) {
          // INT8 B: the codes and the row's scale exactly, in fp32
          const int8_t* br = a.B8 + (size_t)(n0 + row) * r;
          for (int j = 0; j < r; ++j) ev += vm[j] * (float)br[j];
          ev *= a.sb[n0 + row];
        } else {
          const uint16_t* br = a.B + (size_t)(n0 + row) * r;
          for (int j = 0; j < r; ++j) ev += vm[j] * act2f<DT>(br[j]);
        }
        v += ev;
      }
      if (a.res) v += act2f<DT>(res_pre ? resv : a.res[(size_t)m * N + n0 + row]);
      a.y[(size_t)m * N + n0 + row] = f2act<DT>(v);
    }
  }
  if constexpr (EPI == EPI_FUSED) fused_exit(a);
}

// Minimum waves per SIMD the compiler must leave room for (the second
// launch bound). One token tile on up to 32 rows without the local EC asks
// for 4, two workgroups of eight waves per CU (at most 128 VGPRs): wide
// layers run several rounds of blocks, and one block per CU leaves half the
// latency hiding unused (70B gate, fused: 60.8 us at 156 VGPRs, 42.6 us at
// 125).
constexpr int gemv_min_waves(int MT, int RT, int EPI) {
  return MT == 1 && RT <= 2 && EPI <= EPI_FUSED ? 4 : 1;
}

template <int DT, int MT, int RT, int EPI, int WB, int NST, bool SPLIT>
__global__ __launch_bounds__(kGemvMaxThreads, gemv_min_waves(MT, RT, EPI)) void k_gemv(GemvParams a) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  int bid = blockIdx.x;
  uint32_t gen = 0;
  if constexpr (EPI == EPI_FUSED) {
    // the first n_prod workgroups are the EC producers
    gen = (uint32_t)(__hip_atomic_load(gen_counter(a, bid), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >> 32);
    if (bid < a.n_prod) {
      ec_producer<DT, 1, false>(a.ec, bid, gen, smem);
      fused_exit(a);
      return;
    }
    bid -= a.n_prod;
  }
  gemv_body<DT, MT, RT, EPI, WB, NST, SPLIT>(a, bid, gen, smem);
}

// Several independent layer calls of one GEMV variant in one launch: member i
// owns the workgroups [start[i], start[i+1]) and runs exactly the blocks its
// own launch would run, so each member's output is the one its single call
// writes. The member index is uniform over the workgroup.
template <int DT, int MT, int RT, int EPI, int WB, bool SPLIT>
__global__ __launch_bounds__(kGemvMaxThreads, gemv_min_waves(MT, RT, EPI)) void k_gemv_group(GemvGroup g) {
  static_assert(EPI != EPI_FUSED, "grouped launches take the variants without cross-launch state");
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int b = blockIdx.x;
  int i = 0;
#pragma unroll
  for (int j = 1; j < kGroupMax; ++j)
    if (j < g.n && b >= g.start[j]) i = j;
  gemv_body<DT, MT, RT, EPI, WB, 2, SPLIT>(g.p[i], b - g.start[i], 0u, smem);
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
#if SPEAR_WB == 4

hipError_t SPEAR_D(launch_ec)(const EcGroup& g, int block, int ipp, size_t lds, hipStream_t st) {
  if (g.n < 1 || g.n > kGroupMax || g.start[0] != 0) return hipErrorInvalidValue;
  const int grid = g.start[g.n];
  if (grid == 0) return hipSuccess;
  const auto go = [&](auto kern, const auto& p) {
    hipError_t err = allow_lds(kern, lds);
    if (err != hipSuccess) return err;
    hipLaunchKernelGGL(kern, dim3(grid), dim3(block), lds, st, p);
    return hipGetLastError();
  };
  if (g.n == 1) return ipp == 1 ? go(k_ec<DTC, 1>, g.p[0]) : go(k_ec<DTC, 2>, g.p[0]);
  return ipp == 1 ? go(k_ec_group<DTC, 1>, g) : go(k_ec_group<DTC, 2>, g);
}

hipError_t SPEAR_D(launch_gate)(const EcParams& e, int ntb, size_t lds, hipStream_t st) {
  if (ntb == 0) return hipSuccess;
  hipError_t err = allow_lds(k_gate<DTC>, lds);
  if (err != hipSuccess) return err;
  hipLaunchKernelGGL(k_gate<DTC>, dim3(ntb), dim3(256), lds, st, e);
  return hipGetLastError();
}

hipError_t SPEAR_D(launch_rmsnorm)(const uint16_t* y, const uint16_t* w, float eps, uint16_t* y_norm,
                          int M, int N, hipStream_t st) {
  if (M == 0 || N == 0) return hipSuccess;
  // rows of whole 16-byte chunks (the buffers are 16-byte aligned): the
  // fewest threads, at least 256, that cover the row in four chunks each
  const int n8 = N / 8;
  if (N % 8 != 0 || n8 > 4096) {
    hipLaunchKernelGGL(k_rmsnorm<DTC>, dim3(M), dim3(256), 0, st, y, w, eps, y_norm, N);
  } else if (n8 <= 256) {
    hipLaunchKernelGGL((k_rmsnorm_v<DTC, 1>), dim3(M), dim3(256), 0, st, y, w, eps, y_norm, N);
  } else if (n8 <= 512) {
    hipLaunchKernelGGL((k_rmsnorm_v<DTC, 2>), dim3(M), dim3(256), 0, st, y, w, eps, y_norm, N);
  } else {
    const int thr = n8 <= 1024 ? 256 : n8 <= 2048 ? 512 : 1024;
    hipLaunchKernelGGL((k_rmsnorm_v<DTC, 4>), dim3(M), dim3(thr), 0, st, y, w, eps, y_norm, N);
  }
  return hipGetLastError();
}

hipError_t SPEAR_D(launch_ec_up_acc)(const float* v, const uint16_t* B, const int8_t* B8,
                            const float* sb, uint16_t* y, int M, int N, int r, hipStream_t st) {
  const long long total = (long long)M * N;
  const unsigned grid = (unsigned)((total + 255) / 256);
  if (grid == 0) return hipSuccess;
  hipLaunchKernelGGL(k_ec_up_acc<DTC>, dim3(grid), dim3(256), 0, st, v, B, B8,
                                         sb, y, M, N, r);
  return hipGetLastError();
}

#endif  // SPEAR_WB == 4

template <int DT, int MT, int RT, int EPI, int NST>
static hipError_t gemv_launch_one(const GemvParams& p, int grid, int block, size_t lds,
                                  hipStream_t st) {
  const auto go = [&](auto kern) {
    hipError_t err = allow_lds(kern, lds);
    if (err != hipSuccess) return err;
    hipLaunchKernelGGL(kern, dim3(grid), dim3(block), lds, st, p);
    return hipGetLastError();
  };
  if constexpr (MT == 1 && NST == 2)
    if (p.S == 1) return go(k_gemv<DT, MT, RT, EPI, SPEAR_WB, NST, false>);
  return go(k_gemv<DT, MT, RT, EPI, SPEAR_WB, NST, true>);
}

// Pipeline depths compiled in: 2 everywhere; 4 for one token tile on the
// variants wide layers take at decode (4-bit only, fused, semi-fused).
template <int DT, int MT, int RT, int EPI>
static hipError_t gemv_launch_nst(int nst, const GemvParams& p, int grid, int block, size_t lds,
                                  hipStream_t st) {
  if constexpr (MT == 1 && (EPI == EPI_NONE || EPI == EPI_READY || EPI == EPI_FUSED)) {
    if (nst == 4) return gemv_launch_one<DT, MT, RT, EPI, 4>(p, grid, block, lds, st);
  }
  if (nst != 2) return hipErrorInvalidValue;
  return gemv_launch_one<DT, MT, RT, EPI, 2>(p, grid, block, lds, st);
}

template <int DT, int MT, int RT>
static hipError_t gemv_launch(int epi, int nst, const GemvParams& p, int grid, int block,
                              size_t lds, hipStream_t st) {
  switch (epi) {
    case EPI_NONE: return gemv_launch_nst<DT, MT, RT, EPI_NONE>(nst, p, grid, block, lds, st);
    case EPI_READY: return gemv_launch_nst<DT, MT, RT, EPI_READY>(nst, p, grid, block, lds, st);
    case EPI_FUSED: return gemv_launch_nst<DT, MT, RT, EPI_FUSED>(nst, p, grid, block, lds, st);
    case EPI_LOCAL: return gemv_launch_nst<DT, MT, RT, EPI_LOCAL>(nst, p, grid, block, lds, st);
    default: return gemv_launch_nst<DT, MT, RT, EPI_LOCAL_I8>(nst, p, grid, block, lds, st);
  }
}

// The GEMV shapes compiled in: (token tiles MT, row tiles RT).
// gemv_shape_supported() mirrors this list for the planner.
#define SPEAR_GEMV_SHAPES(X) \
  X(1, 1) X(1, 2) X(1, 4) X(2, 1) X(2, 2) X(2, 4) X(3, 1) X(3, 2) X(4, 1)

#if SPEAR_WB == 4 && !SPEAR_BF16_UNIT
bool gemv_shape_supported(int MT, int RT) {
#define SPEAR_GEMV_MATCH(mt, rt) if (MT == mt && RT == rt) return true;
  SPEAR_GEMV_SHAPES(SPEAR_GEMV_MATCH)
#undef SPEAR_GEMV_MATCH
  return false;
}
#endif

hipError_t SPEAR_W(launch_gemv)(int MT, int RT, int epi, int nst, const GemvParams& p,
                                int grid, int block, size_t lds, hipStream_t st) {
  // split-K needs its partial sums and row-group counters (workspace)
  const bool loc = epi == EPI_LOCAL || epi == EPI_LOCAL_I8;
  if (p.S < 1 || (p.S > 1 && (!p.ypart || !p.rb_ctr || (loc && !p.eupart))) ||
      (epi == EPI_LOCAL_I8 && (!p.ec.A8 || !p.ec.sa || !p.B8 || !p.sb)))
    return hipErrorInvalidValue;
  if (grid == 0) return hipSuccess;
#define SPEAR_GEMV_CASE(mt, rt) \
  if (MT == mt && RT == rt)  \
    return gemv_launch<DTC, mt, rt>(epi, nst, p, grid, block, lds, st);
  SPEAR_GEMV_SHAPES(SPEAR_GEMV_CASE)
#undef SPEAR_GEMV_CASE
  return hipErrorInvalidValue;
}

template <int DT, int MT, int RT>
static hipError_t gemv_group_launch(int epi, const GemvGroup& g, int block, size_t lds,
                                    hipStream_t st) {
  constexpr int WB = SPEAR_WB;
  const int grid = g.start[g.n];
  bool split = MT > 1;  // a member in several K-slices
  for (int i = 0; i < g.n; ++i) split |= g.p[i].S > 1;
  const auto go = [&](auto kern) {
    hipError_t err = allow_lds(kern, lds);
    if (err != hipSuccess) return err;
    hipLaunchKernelGGL(kern, dim3(grid), dim3(block), lds, st, g);
    return hipGetLastError();
  };
#define SPEAR_GEMV_GROUP_GO(E) \
  case E: return split ? go(k_gemv_group<DT, MT, RT, E, WB, true>) : go(k_gemv_group<DT, MT, RT, E, WB, MT != 1>);
  switch (epi) {
    SPEAR_GEMV_GROUP_GO(EPI_NONE)
    SPEAR_GEMV_GROUP_GO(EPI_READY)
    SPEAR_GEMV_GROUP_GO(EPI_LOCAL)
    SPEAR_GEMV_GROUP_GO(EPI_LOCAL_I8)
    default: return hipErrorInvalidValue;
  }
#undef SPEAR_GEMV_GROUP_GO
}

hipError_t SPEAR_W(launch_gemv_group)(int MT, int RT, int epi, const GemvGroup& g,
                                      int block, size_t lds, hipStream_t st) {
  if (g.n < 1 || g.n > kGroupMax || g.start[0] != 0) return hipErrorInvalidValue;
  const bool loc = epi == EPI_LOCAL || epi == EPI_LOCAL_I8;
  for (int i = 0; i < g.n; ++i) {
    const GemvParams& p = g.p[i];
    if (g.start[i + 1] < g.start[i] || p.S < 1 ||
        (p.S > 1 && (!p.ypart || !p.rb_ctr || (loc && !p.eupart))) ||
        (epi == EPI_LOCAL_I8 && (!p.ec.A8 || !p.ec.sa || !p.B8 || !p.sb)))
      return hipErrorInvalidValue;
  }
  if (g.start[g.n] == 0) return hipSuccess;
#define SPEAR_GEMV_GROUP_CASE(mt, rt) \
  if (MT == mt && RT == rt)  \
    return gemv_group_launch<DTC, mt, rt>(epi, g, block, lds, st);
  SPEAR_GEMV_SHAPES(SPEAR_GEMV_GROUP_CASE)
#undef SPEAR_GEMV_GROUP_CASE
  return hipErrorInvalidValue;
}

}  // namespace spear
