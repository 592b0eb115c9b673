// Row-streaming GEMV for the draft layer's projections and its widened head: bf16 steps of up to four rows (chain
// drafting of a few sequences) and fp32 ones.  out[m][n] = sum_k a[m][k] w[n][k].
//
// With so few activation rows the matrix cores buy nothing: the kernel is a pure weight
// stream.  A wave takes two weight rows at a time and reads each along K with 16-byte loads,
// 1 KB per instruction and three instructions per row in flight (four, five, eight and ten measured: no faster), multiplies with the
// fp32 activations held in LDS and reduces across its lanes.  There is no split over K, so
// nothing is left for a later kernel (or a last-arriving workgroup) to add up: the epilogue
// runs in the wave that owns the rows, lane m for activation row m.  The two rows of a pair are chosen by the epilogue:
//   0 rows   (2p, 2p+1): residual add, fp32 / stored outputs, pieces of the rows' sums of
//            squares for the RMSNorm the consumer applies;
//   1 rotary (head*d + c, head*d + c + d/2) of the concatenated q|k|v projection: the pair
//            is rotated and stored as a query element or a cache entry (Sec. 3.1 draft layer);
//   2 gate   (p, I + p) of the concatenated gate|up projection: silu(gate) * up;
//   3 head   (2p, 2p+1) of the widened head (Eq. 1): rows below V enter a running argmax (lowest
//            index on ties) kept per wave and merged per workgroup, the signal rows V.. are
//            written out; a later launch merges the workgroups' candidates;
//   4 rows   (2p, 2p+1) of the fp32 head, written out for the ranking kernels.
//
// What bounds it: for the head the stream (V = 151936, D = 2560: 778 MB in 114.7 us, 6.8 TB/s), for the projections (0.5 to 100
// MB) that a launch is a chain: arguments, activations, weights, sum, epilogue.  So the lines of the arguments are
// requested together, the first weights behind the activations and the pieces of the sums of squares (loads return in the order of
// their requests: with most pieces asked for behind the weights the barrier came 1.9 to 2.6 us later, as time stamps in the kernels showed; a
// step of 1 / 8 rows, fp32, D = 512: 43 / 66 -> 41 / 61 us; a round of six steps, D = 2560, V = 151936: 1221 -> 1205; a barrier that keeps
// every wave's weights behind all waves' activations: slower) and before anything waits (under
// a norm x gain is staged, 1 / rms enters after the product), the residual, the rotation and the cache entry of a pair
// while its weights are on their way, and a pair's first loads before the pair in front of it is summed.  Measured against the form
// that did these one after the other (and fp32 models on one kernel per operation, fifteen launches a step instead of nine):
//   bf16  a draft step of 1 / 2 rows, D = 2560, V = 151936: 189 / 216 -> 177 / 190 us; D = 5120: 457 / - -> 430; D = 1536, V =
//         100000: 103 / 122 -> 89 / 100
//   fp32  a draft step of D = 512 (V = 4096), 1 / 8 rows: 54 / 101 -> 39 / 67 us; D = 1024 (V = 20000), 8 rows 166 -> 108;
//         a level of 16 rows 205 -> 146
#include "common.hpp"
#include "kernels.hpp"

#include <limits.h>

#include <algorithm>

namespace sx {

namespace {

typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

// The head's 778 MB are read once per launch and must not displace anything: non-temporal
// loads.  The layer's projections come round again one draft step later; when they fit the 256 MB
// last-level cache (228 MB at the metric's workload) ordinary loads let it keep part of them
// (measured: 764 -> 775 rounds/s; with ordinary loads in the head as well, 696).  A layer that
// does not fit is streamed like the head (ordinary loads cost 2 % there, measured on the
// matrix-core projections of the 8B- and 32B-like shapes).
template <bool STREAM>
__device__ __forceinline__ uint4 load_weights16(const char* p) {
  if constexpr (STREAM) {
    const u32x4_t t = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(p));
    return make_uint4(t.x, t.y, t.z, t.w);
  } else {
    return *reinterpret_cast<const uint4*>(p);
  }
}

// First byte of weight row n.  (Sums of conditional distances: an indexed pointer is another load of an argument.)
template <typename T>
__device__ __forceinline__ const char* weight_row(const GemvArgs& g, int n) {
  const char* w = static_cast<const char*>(g.w[0]);
  int row = n;
  if (g.nseg > 1 && n >= g.seg_end[0]) { w = static_cast<const char*>(g.w[1]); row = n - g.seg_end[0]; }
  if (g.nseg > 2 && n >= g.seg_end[1]) { w = static_cast<const char*>(g.w[2]); row = n - g.seg_end[1]; }
  return w + static_cast<size_t>(row) * g.K * sizeof(T);
}

// Where head hh of the concatenated q|k|v rows goes for activation row m: its query row or cache entry (null: outside the cache)
__device__ __forceinline__ void* rope_entry(const RopeArgs& ra, int m, int hh, int elem) {
  if (hh < ra.Hq) return static_cast<char*>(ra.q_out) + (static_cast<size_t>(m) * ra.Hq + hh) * ra.d * elem;
  const int b = m / ra.W;
  const int slot = ra.pos[b] + (ra.node ? ra.node[m % ra.W] : 0);
  if (slot < 0 || slot >= ra.l_max) return nullptr;
  const bool is_k = hh < ra.Hq + ra.Hkv;
  const int h = is_k ? hh - ra.Hq : hh - ra.Hq - ra.Hkv;
  size_t off;
  if (ra.paged) {
    const int page = ra.page_table[static_cast<size_t>(b) * ra.max_pages + slot / ra.page_size];
    if (!page_in_pool(page, ra.n_pages, ra.status)) return nullptr;
    off = ((static_cast<size_t>(page) * ra.Hkv + h) * ra.page_size + slot % ra.page_size) * ra.d;
  } else {
    off = ((static_cast<size_t>(b) * ra.Hkv + h) * ra.l_max + slot) * ra.d;
  }
  return static_cast<char*>(is_k ? ra.kc : ra.vc) + off * elem;
}

// The values of 16 bytes of storage
__device__ __forceinline__ void widen(const uint4& v, float (&f)[8]) { unpack16(v, f); }
__device__ __forceinline__ void widen(const uint4& v, float (&f)[4]) {
  f[0] = __uint_as_float(v.x); f[1] = __uint_as_float(v.y); f[2] = __uint_as_float(v.z); f[3] = __uint_as_float(v.w);
}

// N consecutive elements of storage (bf16 rows are 16-byte aligned, fp32 ones need not be)
__device__ __forceinline__ void load_row(const bf16_t* p, float (&f)[8]) { unpack16(*reinterpret_cast<const uint4*>(p), f); }
__device__ __forceinline__ void load_row(const float* p, float (&f)[4]) {
#pragma unroll
  for (int e = 0; e < 4; ++e) f[e] = p[e];
}

// MR activation rows per workgroup (fp32: blockIdx.y tells which), SIF 16-byte loads per weight row in flight.
template <typename T, int MR, int SIF, int AMODE, int EPI, bool STREAM>
__global__ __launch_bounds__(512) void k_gemv(const GemvArgs g) {
  constexpr int EP = 16 / sizeof(T);           // elements per load
  constexpr int NE = EP / 4;                   // float4 of activations beside it
  extern __shared__ float lds[];
  __shared__ float ssq_sh[8][MR], rs_sh[MR];
  __shared__ float bv_sh[8][MR];
  __shared__ int bi_sh[8][MR];
  arguments_at_once<sizeof(GemvArgs)>();
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nwaves = g.waves, nt = nwaves << 6;
  const int K = g.K;
  const int steps = K / (64 * EP);             // K is a multiple of that
  const int m0 = sizeof(T) == 4 ? blockIdx.y * MR : 0;   // rows past the last one repeat it and are dropped later
  const int mine = m0 + lane;                  // the row that this lane finishes
  const bool owner = lane < MR && mine < g.M;

  // ---- stage the activations, without waiting for the rows' sums of squares: under a norm, x gain is staged and 1 / rms enters
  // behind the dot product.  Four units of a thread are requested together.
  // The pieces of the sums are requested in front of the weights, since loads return in the order of their requests; a wave has one row
  // (further rows, which few shapes have, are added up before the weights are asked for).  A lane adds its pieces in their
  // order: those beyond the first NP are fetched behind the weights.
  // (Up to 512 pieces of bf16 models: D = 5120 has that many, a round of three steps 1522 -> 1504 us; fp32 models have 256 at most up to
  // D = 4096, and 1 % more to do with eight.  A piece is a workgroup's, of which D <= 8192 gives 512 on 256 compute units: the loop behind
  // the weights runs for fp32 models of more than 4096.)
  constexpr int NP = sizeof(T) == 2 ? 8 : 4;
  const float* const pieces = AMODE == 3 ? g.a_ssq + min(m0 + min(wv, MR - 1), g.M - 1) * g.a_nssq : nullptr;
  float sq[NP];
  auto root = [&](int m, float t) {
    const float rs = 1.0f / sqrtf(wave_sum_dpp(t) / static_cast<float>(K) + g.a_eps);
    if (lane == 0) rs_sh[m] = rs;
  };
  if constexpr (AMODE == 3) {
#pragma unroll
    for (int u = 0; u < NP; ++u) sq[u] = pieces[min(lane + 64 * u, g.a_nssq - 1)];
  }
  const int per_row = K / EP, units = MR * per_row;
  constexpr int U = 4;
  float f[U][EP], gn[U][EP];
  auto stage_load = [&](int base) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int idx = min(base + u * nt + static_cast<int>(threadIdx.x), units - 1);
      const int r = MR == 1 ? 0 : idx / per_row, k = (idx - r * per_row) * EP;
      const int m = min(m0 + r, g.M - 1);
      if constexpr (AMODE == 0 || AMODE == 3) {
        const float4* src = reinterpret_cast<const float4*>(static_cast<const float*>(g.a_src) + static_cast<size_t>(m) * K + k);
#pragma unroll
        for (int h = 0; h < NE; ++h) {
          const float4 x = src[h];
          f[u][4 * h] = x.x; f[u][4 * h + 1] = x.y; f[u][4 * h + 2] = x.z; f[u][4 * h + 3] = x.w;
        }
        if constexpr (AMODE == 3) load_row(static_cast<const T*>(g.a_gain) + k, gn[u]);
      } else if constexpr (AMODE == 1) {
        load_row(static_cast<const T*>(g.a_src) + static_cast<size_t>(m) * K + k, f[u]);
      } else {
        const int half = K >> 1;
        load_row(k < half ? static_cast<const T*>(g.a_embed) + static_cast<size_t>(checked_token(g.a_tok[m], g.a_vocab, g.status)) * half + k
                          : static_cast<const T*>(g.a_src) + static_cast<size_t>(m) * half + (k - half), f[u]);
      }
    }
  };
  auto stage_store = [&](int base) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int idx = base + u * nt + static_cast<int>(threadIdx.x);
      const int r = MR == 1 ? 0 : idx / per_row, i = idx - r * per_row;
      if (idx < units) {
        // step i / 64 holds lane i % 64's values as NE float4: conflict-free reads
#pragma unroll
        for (int h = 0; h < NE; ++h) {
          float x[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) x[e] = AMODE == 3 ? f[u][4 * h + e] * gn[u][4 * h + e] : f[u][4 * h + e];
          *reinterpret_cast<float4*>(lds + ((((i >> 6) * MR + r) * NE + h) * 64 + (i & 63)) * 4) = make_float4(x[0], x[1], x[2], x[3]);
        }
      }
    }
  };
  int base = 0;
  for (; base + U * nt < units; base += U * nt) {
    stage_load(base);
    stage_store(base);
  }
  stage_load(base);
  if constexpr (AMODE == 3) {
    for (int m = wv + nwaves; m < MR; m += nwaves) {
      float t = 0.f;
      for (int j = lane; j < g.a_nssq; j += 64) t += g.a_ssq[min(m0 + m, g.M - 1) * g.a_nssq + j];
      root(m, t);
    }
  }

  // ---- pairs of rows, dealt round-robin over all waves of the launch: at any time the waves read
  // one moving window of neighbouring rows (measured 0.9 % on the round against a contiguous
  // range of pairs per workgroup), and no wave gets more than one pair above the others.  A pair's first loads are under way
  // while the pair before it is summed and finished, those of the first one while the activations are staged.
  const int P = (g.N + 1) >> 1;          // only the head's row count can be odd: its last pair is half empty
  const char *r1, *r2;
  int n1, n2;
  auto pair_rows = [&](int p) {
    if constexpr (EPI == 1) {
      const int half = g.rope.d >> 1;
      const int head = p / half;
      n1 = head * g.rope.d + (p - head * half);
      n2 = n1 + half;
    } else if constexpr (EPI == 2) {
      n1 = p;
      n2 = P + p;
    } else {
      n1 = 2 * p;
      n2 = n1 + 1;
    }
    r1 = weight_row<T>(g, n1) + lane * 16;
    r2 = weight_row<T>(g, min(n2, g.N - 1)) + lane * 16;   // a row past the end repeats the last one, unused
  };
  uint4 w1[SIF], w2[SIF];
  auto request = [&](int j0) {           // (behind the last step the last one again, unused)
#pragma unroll
    for (int u = 0; u < SIF; ++u) {
      const size_t at = static_cast<size_t>(min(j0 + u, steps - 1)) << 10;
      w1[u] = load_weights16<STREAM>(r1 + at);
      w2[u] = load_weights16<STREAM>(r2 + at);
    }
  };
  int p = blockIdx.x * nwaves + wv;
  pair_rows(min(p, P - 1));
  request(0);
  __builtin_amdgcn_sched_barrier(0);
  stage_store(base);
  if constexpr (AMODE == 3) {
    float t = 0.f;
#pragma unroll
    for (int u = 0; u < NP; ++u) t += lane + 64 * u < g.a_nssq ? sq[u] : 0.f;
    if (__builtin_expect(g.a_nssq > 64 * NP, 0)) {      // (uniform; lane by lane a round of two fp32 rows, D = 1024, 324 us, 321.5 this way)
      for (int j = lane + 64 * NP; j < g.a_nssq; j += 64) t += pieces[j];
    }
    if (wv < MR) root(wv, t);
  }
  __syncthreads();
  float rs[MR];
#pragma unroll
  for (int m = 0; m < MR; ++m) rs[m] = AMODE == 3 ? rs_sh[m] : 1.f;

  float ssq = 0.f, bestv = -INFINITY;    // lane m: of row m0 + m
  int besti = INT_MAX;
  float acc1[MR], acc2[MR];
#pragma unroll
  for (int m = 0; m < MR; ++m) { acc1[m] = 0.f; acc2[m] = 0.f; }
  float cs = 1.f, sn = 0.f;
  float2 res = make_float2(0.f, 0.f);
  T* dst = nullptr;
  for (int j0 = 0; p < P;) {
    // what finishing the pair needs, while its weights are on their way
    if constexpr (EPI == 0) {
      if (j0 == 0 && g.residual && owner) res = *reinterpret_cast<const float2*>(g.residual + static_cast<size_t>(mine) * g.N + n1);
    }
    if constexpr (EPI == 1) {
      if (j0 == 0 && owner) dst = static_cast<T*>(rope_entry(g.rope, mine, n1 / g.rope.d, sizeof(T)));
      // angle in double, so that long positions keep their phase
      if (j0 == 0 && n1 < (g.rope.Hq + g.rope.Hkv) * g.rope.d) {
        const double ang = static_cast<double>(g.rope.pos[min(mine, g.M - 1) / g.rope.W] + g.rope.level) * g.rope.inv_freq[n1 % g.rope.d];
        if constexpr (sizeof(T) == 4) {
          double s, c;
          sincos(ang, &s, &c);
          sn = static_cast<float>(s);
          cs = static_cast<float>(c);
        } else {
          // reduced to [-pi, pi] in double, sine and cosine of the remainder in float
          const double turns = rint(ang * 0.15915494309189535);
          const float red = static_cast<float>(fma(-turns, 6.283185307179586, ang));
          cs = cosf(red);
          sn = sinf(red);
        }
      }
    }
#pragma unroll
    for (int u = 0; u < SIF; ++u) {
      const int j = j0 + u;
      if (j < steps) {
        float f1[EP], f2[EP];
        widen(w1[u], f1);
        widen(w2[u], f2);
#pragma unroll
        for (int m = 0; m < MR; ++m)
#pragma unroll
          for (int h = 0; h < NE; ++h) {
            const float4 a = *reinterpret_cast<const float4*>(lds + (((j * MR + m) * NE + h) * 64 + lane) * 4);
            acc1[m] = fmaf(a.x, f1[4 * h], acc1[m]); acc1[m] = fmaf(a.y, f1[4 * h + 1], acc1[m]);
            acc1[m] = fmaf(a.z, f1[4 * h + 2], acc1[m]); acc1[m] = fmaf(a.w, f1[4 * h + 3], acc1[m]);
            acc2[m] = fmaf(a.x, f2[4 * h], acc2[m]); acc2[m] = fmaf(a.y, f2[4 * h + 1], acc2[m]);
            acc2[m] = fmaf(a.z, f2[4 * h + 2], acc2[m]); acc2[m] = fmaf(a.w, f2[4 * h + 3], acc2[m]);
          }
      }
    }
    j0 += SIF;
    if (j0 < steps) {
      request(j0);
      continue;
    }
    j0 = 0;
    const int done = p, d1 = n1, d2 = n2;      // the finished pair
    p += g.grid * nwaves;
    if (p < P) {
      pair_rows(p);
      request(0);
    }
    __builtin_amdgcn_sched_barrier(0);
    float x1 = 0.f, x2 = 0.f;                  // lane m: row m0 + m
#pragma unroll
    for (int m = 0; m < MR; ++m) {
      const float v1 = wave_sum_dpp(acc1[m]) * rs[m], v2 = wave_sum_dpp(acc2[m]) * rs[m];
      if (lane == m) { x1 = v1; x2 = v2; }
      acc1[m] = 0.f;
      acc2[m] = 0.f;
    }
    if (!owner) continue;
    if constexpr (EPI == 0) {
      const size_t at = static_cast<size_t>(mine) * g.N + d1;
      x1 += res.x;
      x2 += res.y;
      *reinterpret_cast<float2*>(g.out_x + at) = make_float2(x1, x2);
      if (g.out_store) {
        if constexpr (sizeof(T) == 2) {
          *reinterpret_cast<uint32_t*>(static_cast<bf16_t*>(g.out_store) + at) = pack_bf16x2(x1, x2);
        } else {
          static_cast<float*>(g.out_store)[at] = x1;
          static_cast<float*>(g.out_store)[at + 1] = x2;
        }
      }
      ssq += x1 * x1 + x2 * x2;
    } else if constexpr (EPI == 1) {
      if (dst) {
        const int c = d1 % g.rope.d;
        const bool turn = d1 < (g.rope.Hq + g.rope.Hkv) * g.rope.d;
        Elem<T>::store(dst + c, turn ? x1 * cs - x2 * sn : x1);
        Elem<T>::store(dst + c + (g.rope.d >> 1), turn ? x2 * cs + x1 * sn : x2);
      }
    } else if constexpr (EPI == 2) {
      g.out_x[static_cast<size_t>(mine) * P + done] = x1 * sigmoidf_(x1) * x2;
    } else if constexpr (EPI == 3) {
      if (d1 < g.V) { if (better(x1, d1, bestv, besti)) { bestv = x1; besti = d1; } }
      else if (g.extra_out) g.extra_out[mine * g.n_extra + (d1 - g.V)] = x1;
      if (d2 < g.N) {
        if (d2 < g.V) { if (better(x2, d2, bestv, besti)) { bestv = x2; besti = d2; } }
        else if (g.extra_out) g.extra_out[mine * g.n_extra + (d2 - g.V)] = x2;
      }
    } else {
      const size_t at = static_cast<size_t>(mine) * g.N;
      g.out_x[at + d1] = x1;
      if (d2 < g.N) g.out_x[at + d2] = x2;
    }
  }

  // ---- the workgroup's pieces of the rows' sums of squares, its best (value, index) per row (waves in a fixed order)
  if constexpr (EPI == 0 || EPI == 3) {
    if (lane < MR) {
      ssq_sh[wv][lane] = ssq;
      bv_sh[wv][lane] = bestv;
      bi_sh[wv][lane] = besti;
    }
    __syncthreads();
    if (wv == 0 && owner) {
      const size_t at = static_cast<size_t>(mine) * g.grid + blockIdx.x;
      if constexpr (EPI == 0) {
        float t = 0.f;
        for (int w = 0; w < nwaves; ++w) t += ssq_sh[w][lane];
        if (g.out_ssq) g.out_ssq[at] = t;
      } else {
        float bv = bv_sh[0][lane];
        int bi = bi_sh[0][lane];
        for (int w = 1; w < nwaves; ++w)
          if (better(bv_sh[w][lane], bi_sh[w][lane], bv, bi)) { bv = bv_sh[w][lane]; bi = bi_sh[w][lane]; }
        g.part_val[at] = bv;
        g.part_idx[at] = bi;
      }
    }
  }
}

constexpr int kLdsMax = 158 * 1024, kLdsMore = 144 * 1024;    // (of one and two rows, of three and four)
constexpr int kMaxWaves = 8;             // per workgroup

template <typename T, int MR, int SIF, int AMODE, int EPI, bool STREAM>
hipError_t launch_as(const GemvArgs& g, hipStream_t s) {
  // set once per process; a function-local static is initialised under the language's own lock,
  // so first calls from several host threads are safe
  static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_gemv<T, MR, SIF, AMODE, EPI, STREAM>),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, kLdsMax);
  if (attr != hipSuccess) return attr;
  hipLaunchKernelGGL((k_gemv<T, MR, SIF, AMODE, EPI, STREAM>), dim3(g.grid, (g.M + MR - 1) / MR), dim3(64 * g.waves),
                     static_cast<size_t>(g.K) * MR * sizeof(float), s, g);
  return hipGetLastError();
}

constexpr int kHeadSteps = 2, kSteps = 3;    // 16-byte loads per weight row in flight

template <typename T, int MR, bool STREAM>
hipError_t launch_projection(const GemvArgs& g, hipStream_t s) {
  switch (g.epi * 4 + g.a_mode) {
    case 0: return launch_as<T, MR, kSteps, 0, 0, STREAM>(g, s);
    case 1:
      if constexpr (sizeof(T) == 2) return launch_as<T, MR, kSteps, 1, 0, STREAM>(g, s);
      return hipErrorInvalidValue;
    case 2: return launch_as<T, MR, kSteps, 2, 0, STREAM>(g, s);
    case 4 + 3:
      if constexpr (MR <= 4) return launch_as<T, MR, kSteps, 3, 1, STREAM>(g, s);
      return hipErrorInvalidValue;
    case 8 + 3: return launch_as<T, MR, kSteps, 3, 2, STREAM>(g, s);
    default: return hipErrorInvalidValue;
  }
}

template <int MR>
hipError_t launch_bf16(const GemvArgs& g, hipStream_t s) {
  if (g.epi == 3 && g.a_mode == 3) return launch_as<bf16_t, MR, kHeadSteps, 3, 3, true>(g, s);
  return g.stream ? launch_projection<bf16_t, MR, true>(g, s) : launch_projection<bf16_t, MR, false>(g, s);
}

template <int MR>
hipError_t launch_f32(const GemvArgs& g, hipStream_t s) {
  if (g.epi == 3 && g.a_mode == 3) return launch_as<float, MR, kSteps, 3, 3, false>(g, s);
  if (g.epi == 4 && g.a_mode == 3) return launch_as<float, MR, kSteps, 3, 4, false>(g, s);
  return launch_projection<float, MR, false>(g, s);
}

}  // namespace

// bf16 weights: up to four rows whose activations fit the LDS (three and four rows: 144 KB of it).  From three rows on the
// matrix-core kernels are faster (a draft step of 2 / 3 / 4 rows here and there, D = 1536 100 / 120 / 149 us and 117 / 117 / 117; 2048
// 152 / 174 / 210 and 152 / 151 / 152; 2560 191 / 233 / - and 210 / 210 / 211; 4096 300 / 346 / - and 305 / 306 / 308), but they take the
// rows in two bf16 parts, where here everything stays in 32 bits: the signals of known rows, D = 2048, are off by 1e-7 here
// and by 2.5e-6 there.
// fp32: against the kernels of gemm.hip, whose activation rows come from the caches, a step of 24 rows, D = 1024, 181 us here
// and 232 there, of 48 rows 302 and 323; of 48 rows with D = 2048, I = 4096 761 and 650, of 16 296 and 359.
constexpr int kBf16Rows = 4, kF32Rows = 24, kF32RowsLongK = 3072;

bool gemv_supported(bool f32, int M, int N, int K) {
  if (M < 1 || N < 2 || K < 1) return false;
  if (f32) return K % 256 == 0 && (M <= kF32Rows || K <= kF32RowsLongK) && K <= kLdsMax / (M <= 4 ? 16 : 32);    // four or eight rows in LDS
  return M <= kBf16Rows && K % 512 == 0 && static_cast<size_t>(K) * M * 4 <= (M <= 2 ? kLdsMax : kLdsMore);
}

// One pair per wave at a time.  The waves of a compute unit share its pairs evenly, with at most 8 per_cu of them: a launch
// whose workgroups do not divide by the compute units waits for those that have one more (eight waves a workgroup
// whatever the shape: 160 workgroups for the 1280 pairs of D = 2560).  More waves, up to kMaxWaves, where the step's rows are many values to
// stage: eight units a thread, counted over all rows, although an fp32 workgroup stages four or eight of them (counted over
// these alone, levels of 16 / 24 / 48 fp32 rows, D = 1024, take 130 / 197 / 316 us instead of 126 / 188 / 300).
void gemv_plan(GemvArgs& g, int num_cus, int per_cu) {
  const int P = (g.N + 1) / 2;
  const int each = (P + num_cus - 1) / num_cus;                 // pairs of a compute unit
  const int rounds = (each + per_cu * kMaxWaves - 1) / (per_cu * kMaxWaves);
  const int waves = (each + rounds - 1) / rounds;               // of a compute unit
  const int groups = (waves + kMaxWaves - 1) / kMaxWaves;
  const int stage = g.M * g.K / (g.f32 ? 4 : 8) / (64 * 8);
  g.waves = std::min(kMaxWaves, std::max((waves + groups - 1) / groups, stage));
  g.grid = std::min(groups * num_cus, (P + g.waves - 1) / g.waves);
}

hipError_t launch_gemv(const GemvArgs& g, hipStream_t s) {
  if (!gemv_supported(g.f32, g.M, g.N, g.K)) return hipErrorInvalidValue;
  if (g.f32) {
    if (g.M == 1) return launch_f32<1>(g, s);
    if (g.M == 2) return launch_f32<2>(g, s);
    // (eight rows beside the rotation in double leave values in scratch memory)
    return g.M <= 4 || g.epi == 1 ? launch_f32<4>(g, s) : launch_f32<8>(g, s);
  }
  switch (g.M) {
    case 1: return launch_bf16<1>(g, s);
    case 2: return launch_bf16<2>(g, s);
    case 3: return launch_bf16<3>(g, s);
    default: return launch_bf16<4>(g, s);
  }
}

}  // namespace sx
