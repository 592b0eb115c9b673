// Verification attention (Alg. 1, the target's verification forward over the draft block): the
// block's n_q queries of every head attend to the whole cached context plus the block
// entries their ancestor mask allows.  The KV cache is read once: all G * n_q query rows
// that share a KV head are processed together, the keys of all sequences are dealt to the
// workgroups in equal shares (attn_sched.hpp; each segment keeps an online softmax), and a
// second kernel merges the segments' (max, sum, output) triples exactly.
#include "attn_sched.hpp"
#include "common.hpp"
#include "kernels.hpp"

#include <algorithm>

namespace sx {

namespace {

// Entry p of a unit: its row in the pools.
__device__ __forceinline__ size_t kv_entry(const AttnArgs& a, int b, int g, int p) {
  if (a.paged) {
    const int in_seq = static_cast<int>(static_cast<uint32_t>(p) / static_cast<uint32_t>(a.page_size));
    const int page = checked_page(a.page_table[static_cast<size_t>(b) * a.max_pages + in_seq], a.n_pages, a.status);
    return (static_cast<size_t>(page) * a.Hkv + g) * a.page_size + (p - in_seq * a.page_size);
  }
  return (static_cast<size_t>(b) * a.Hkv + g) * a.l_max + p;
}

// Plain-ALU kernel, any storage type: fp32 caches, and bf16 ones whose page size is no power of two.
// A tile is a granule of 64 keys: a wave has a row's scores in its 64 lanes, so that the softmax needs no LDS round trip and a
// tile two barriers.  The entries of the next tile are requested into registers before the current one is worked on, and those
// of the first together with the queries: short launches are a chain of latencies (one granule per workgroup up to 256 of
// them), long ones wait for memory otherwise.  Rows that are few leave threads over in P V: these take the keys in
// groups, whose sums meet at the segment's end.  Whole calls, before (tiles of 32 keys, five barriers each, the softmax by a thread per row) / now:
// fp32, 1 sequence of 256-512 entries, 8 queries of 8 heads, 64 wide 21.1 / 15.5 us; 2 of 1000-2000, 10 of 16, 64 wide 29.3 / 22.7; 4 of
// 500-1000, 17 of 16, 64 wide 37.2 / 29.6; 8 of 1000-2000, 5 of 8, 128 wide, paged 48.0 / 46.5; the split kernel of 1 x 256
// entries, 1 query 11.7 / 7.5.
constexpr int kTK = kAttnGran;
constexpr int kTP = kTK + 4;              // floats per row of probabilities (padded: several rows of it are read at once)
constexpr size_t kValuLds = 150 * 1024;
__host__ __device__ constexpr size_t valu_lds_bytes(int R, int d, int B) {
  return sizeof(float) * (static_cast<size_t>(R) * (d + kTP + 3) + kTK * (d + 4) + kTK * d + attn_sched_words(B));
}
// Most rows that the kernel is built for: its accumulators are sized for them (with those of 128 rows for all, 128-wide heads
// of 16 / 32 rows took 24 / 35 us where they take 19 / 28 now, 4 sequences of 900 entries, 16 heads over 4).  128-wide heads of more rows
// go to the kernel below.
__host__ __device__ constexpr int valu_rows_few(int d) { return d == 128 ? 32 : 64; }
__host__ __device__ constexpr int valu_rows_most(int d) { return d == 128 ? 64 : 128; }
static_assert(valu_lds_bytes(valu_rows_most(64), 64, kAttnMaxSeqs) <= kValuLds && valu_lds_bytes(valu_rows_most(128), 128, kAttnMaxSeqs) <= kValuLds, "K and V tiles fit beside the rows");

template <typename T, int D, int ROWS>
__global__ __launch_bounds__(256) void k_attn_split_valu(const AttnArgs a) {
  extern __shared__ float smem[];
  const int G = a.G;
  const int R = G * a.n_q;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  constexpr int DP = D + 4;
  float* Qs = smem;                       // [R][D]
  float* Ks = Qs + R * D;                 // [kTK][DP]
  float* Vs = Ks + kTK * DP;              // [kTK][D]
  float* Ss = Vs + kTK * D;               // [R][kTP] probabilities
  float* Ms = Ss + R * kTP;               // [R] running max
  float* Ls = Ms + R;                     // [R] running sum
  float* As = Ls + R;                     // [R] rescale of this tile
  int* sched_lds = reinterpret_cast<int*>(As + R);
  const AttnTable table = attn_sched_build(a, sched_lds);
  const AttnLine line = attn_sched_line(a, table);
  if (static_cast<int>(blockIdx.x) >= line.W) return;
  // P V: thread (c4, r0) has columns 4 c4 .. + 3 of rows r0, r0 + RSTEP, ..; with at most half of RSTEP rows, KG groups of
  // RP row slots take kTK / KG keys each
  constexpr int C4 = D / 4;               // float4 columns
  constexpr int RSTEP = 256 / C4;         // rows covered per pass
  constexpr int MAXU = ROWS / RSTEP;
  const int c4 = tid % C4;
  int KG = 1;
  while (2 * KG * R <= RSTEP) KG *= 2;
  const int RP = RSTEP / KG;
  const int r0 = (tid / C4) % RP, kgrp = (tid / C4) / RP;
  const int jlo = kgrp * (kTK / KG), jhi = jlo + kTK / KG;
  constexpr int EPV = Elem<T>::kPer16B;
  constexpr int VPR = D / EPV;            // 16-byte pieces of a cache row
  constexpr int NL = kTK * VPR / 256;     // pieces of a K or V tile per thread
  constexpr int JSTEP = 256 / VPR;        // keys between them
  const int lj = tid / VPR, lc = tid % VPR;

  const int x_hi = attn_sched_lo(line, blockIdx.x + 1);
  AttnSeg seg = attn_sched_next(a, table, true, line.pad, attn_sched_lo(line, blockIdx.x), x_hi);
  if (seg.next < x_hi) attn_sched_keep(a, table);
  for (; seg.s1 > seg.s0; seg = attn_sched_next(a, table, false, line.pad, seg.next, x_hi)) {
  attn_sched_publish(a, seg);
  const int g = seg.g, b = seg.b, L = seg.L, s0 = seg.s0, s1 = seg.s1;

  uint4 kr[NL], vr[NL];
  auto fetch = [&](int t0) {              // (keys past the range repeat the last one; they are masked, their V is zeroed)
#pragma unroll
    for (int u = 0; u < NL; ++u) {
      const size_t at = kv_entry(a, b, g, min(t0 + lj + u * JSTEP, s1 - 1)) * VPR + lc;
      kr[u] = static_cast<const uint4*>(a.k)[at];
      vr[u] = static_cast<const uint4*>(a.v)[at];
    }
  };
  auto put = [&](float* dst, int stride, const uint4& raw, int j) {
    float f[8];
    if constexpr (EPV == 8) {
      unpack16(raw, f);
      *reinterpret_cast<float4*>(dst + j * stride + lc * 8 + 4) = make_float4(f[4], f[5], f[6], f[7]);
    } else {
      f[0] = __uint_as_float(raw.x); f[1] = __uint_as_float(raw.y); f[2] = __uint_as_float(raw.z); f[3] = __uint_as_float(raw.w);
    }
    *reinterpret_cast<float4*>(dst + j * stride + lc * EPV) = make_float4(f[0], f[1], f[2], f[3]);
  };
  auto put_v = [&](int t0) {
#pragma unroll
    for (int u = 0; u < NL; ++u) put(Vs, D, t0 + lj + u * JSTEP < s1 ? vr[u] : make_uint4(0u, 0u, 0u, 0u), lj + u * JSTEP);
  };
  fetch(s0);
  for (int idx = tid; idx < R * D; idx += 256) {
    const int r = idx / D, c = idx % D;
    const int i = (r * a.g_inv) >> 16, hh = r - i * G;         // r / G
    const T* qp = static_cast<const T*>(a.q) + ((static_cast<size_t>(b) * a.n_q + i) * a.Hq + g * G + hh) * D;
    Qs[idx] = Elem<T>::load(qp + c);
  }
  for (int r = tid; r < R; r += 256) { Ms[r] = -INFINITY; Ls[r] = 0.f; }
  float4 o[MAXU];
#pragma unroll
  for (int u = 0; u < MAXU; ++u) o[u] = make_float4(0.f, 0.f, 0.f, 0.f);

  for (int t0 = s0; t0 < s1; t0 += kTK) {
    const bool more = t0 + kTK < s1;
    if (t0 > s0) __syncthreads();         // the tile before is done with
#pragma unroll
    for (int u = 0; u < NL; ++u) put(Ks, DP, kr[u], lj + u * JSTEP);
    put_v(t0);
    if (more) fetch(t0 + kTK);
    __syncthreads();
    // scores and softmax: lane = key, wave w has rows w, w + 4, .., four at a time
    const int p = t0 + lane;
    const float4* kv = reinterpret_cast<const float4*>(Ks + lane * DP);
    for (int rb = wv; rb < R; rb += 16) {
      float acc[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
      for (int c = 0; c < C4; ++c) {
        const float4 y = kv[c];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float4 x = *reinterpret_cast<const float4*>(Qs + min(rb + 4 * e, R - 1) * D + 4 * c);
          acc[e] = fmaf(x.x, y.x, acc[e]); acc[e] = fmaf(x.y, y.y, acc[e]);
          acc[e] = fmaf(x.z, y.z, acc[e]); acc[e] = fmaf(x.w, y.w, acc[e]);
        }
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int r = rb + 4 * e;
        if (r >= R) break;                // uniform
        bool vis = p < s1;
        if (vis && p >= L) {
          const int i = (r * a.g_inv) >> 16;
          const uint64_t row = a.mask ? a.mask[static_cast<size_t>(b) * a.mask_stride + i] : ((2ull << i) - 1ull);
          vis = (row >> (p - L)) & 1ull;
        }
        const float x = vis ? acc[e] * a.scale : -INFINITY;
        const float m_old = Ms[r];
        const float m_new = fmaxf(m_old, wave_max_dpp(x));
        float alpha = 1.f, pr = 0.f;
        if (m_new != -INFINITY) {
          alpha = m_old == -INFINITY ? 0.f : expf(m_old - m_new);
          pr = expf(x - m_new);           // exp(-inf) = 0 for masked keys
        }
        const float sum = wave_sum_dpp(pr);
        Ss[r * kTP + lane] = pr;
        if (lane == 0) {
          Ms[r] = m_new;
          Ls[r] = Ls[r] * alpha + sum;
          As[r] = alpha;
        }
      }
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < MAXU; ++u) {
      const int r = r0 + u * RSTEP;
      if (r < R) {
        const float al = As[r];
        float4 acc = make_float4(o[u].x * al, o[u].y * al, o[u].z * al, o[u].w * al);
#pragma unroll 2
        for (int j = jlo; j < jhi; j += 4) {
          const float4 pj = *reinterpret_cast<const float4*>(Ss + r * kTP + j);
          const float w[4] = {pj.x, pj.y, pj.z, pj.w};
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float4 vv = *reinterpret_cast<const float4*>(Vs + (j + e) * D + c4 * 4);
            acc.x = fmaf(w[e], vv.x, acc.x); acc.y = fmaf(w[e], vv.y, acc.y);
            acc.z = fmaf(w[e], vv.z, acc.z); acc.w = fmaf(w[e], vv.w, acc.w);
          }
        }
        o[u] = acc;
      }
    }
  }
  const size_t unit = static_cast<size_t>(blockIdx.x) + static_cast<size_t>(b) * a.Hkv + g;   // partial slot of segment (w, u)
  if (KG > 1) {                           // uniform: at most RSTEP / 2 rows, one slot each
    float4* meet = reinterpret_cast<float4*>(Ks);
    __syncthreads();
    meet[tid] = o[0];
    __syncthreads();
    if (kgrp == 0) {
      for (int k = 1; k < KG; ++k) {
        const float4 v = meet[tid + k * RP * C4];
        o[0].x += v.x; o[0].y += v.y; o[0].z += v.z; o[0].w += v.w;
      }
    }
  }
  if (kgrp == 0) {
#pragma unroll
    for (int u = 0; u < MAXU; ++u) {
      const int r = r0 + u * RSTEP;
      if (r < R && (u == 0 || KG == 1)) *reinterpret_cast<float4*>(a.part_o + (unit * R + r) * D + c4 * 4) = o[u];
    }
  }
  for (int r = tid; r < R; r += 256) {
    a.part_ml[(unit * R + r) * 2 + 0] = Ms[r];
    a.part_ml[(unit * R + r) * 2 + 1] = Ls[r];
  }
  __syncthreads();   // a further segment restarts the running maxima and sums
  }
}

// The same for 128-wide heads with many rows, where P V is what takes the time: tiles of 32 keys, a thread per row for the softmax.
// 48 / 64 / 68 / 96 rows per KV head, calls of 16 heads over 4, this one / the one above built for as many rows: fp32, 4 sequences of
// 900 entries 41.1 / 37.6, 50.2 / 46.7, 53.5 / 63.0, 67.7 / 80.4 us; 8 of 500-2500 101 / 84, 144 / 120, 154 / 181, 197 / 235; bf16, pages of
// 48, 4 of 900 40.4 / 36.2, 49.2 / 44.9, 52.7 / 49.2, 67.0 / 62.0 (there the line could lie higher).
constexpr int kTKMany = 32;
__host__ __device__ constexpr size_t many_lds_bytes(int R, int d, int B) {
  return sizeof(float) * (static_cast<size_t>(R) * (d + kTKMany + 3) + 2 * kTKMany * (d + 4) + attn_sched_words(B));
}
static_assert(many_lds_bytes(128, 128, kAttnMaxSeqs) <= kValuLds, "a tile fits beside the rows");

template <typename T, int D>
__global__ __launch_bounds__(256) void k_attn_split_rows(const AttnArgs a) {
  extern __shared__ float smem[];
  const int G = a.G;
  const int R = G * a.n_q;
  const int tid = threadIdx.x;
  constexpr int DP = D + 4;
  float* Qs = smem;                 // [R][D]
  float* Ks = Qs + R * D;           // [kTKMany][DP]
  float* Vs = Ks + kTKMany * DP;        // [kTKMany][DP]
  float* Ss = Vs + kTKMany * DP;        // [R][kTKMany]
  float* Ms = Ss + R * kTKMany;         // [R] running max
  float* Ls = Ms + R;               // [R] running sum
  float* As = Ls + R;               // [R] rescale of this tile
  int* sched_lds = reinterpret_cast<int*>(As + R);
  const AttnTable table = attn_sched_build(a, sched_lds);
  const AttnLine line = attn_sched_line(a, table);
  if (static_cast<int>(blockIdx.x) >= line.W) return;
  const int x_hi = attn_sched_lo(line, blockIdx.x + 1);
  AttnSeg seg = attn_sched_next(a, table, true, line.pad, attn_sched_lo(line, blockIdx.x), x_hi);
  if (seg.next < x_hi) attn_sched_keep(a, table);
  for (; seg.s1 > seg.s0; seg = attn_sched_next(a, table, false, line.pad, seg.next, x_hi)) {
  attn_sched_publish(a, seg);
  const int g = seg.g, b = seg.b, L = seg.L, s0 = seg.s0, s1 = seg.s1;

  for (int idx = tid; idx < R * D; idx += 256) {
    const int r = idx / D, c = idx % D;
    const int i = (r * a.g_inv) >> 16, hh = r - i * G;         // r / G
    const T* qp = static_cast<const T*>(a.q) + ((static_cast<size_t>(b) * a.n_q + i) * a.Hq + g * G + hh) * D;
    Qs[idx] = Elem<T>::load(qp + c);
  }
  for (int r = tid; r < R; r += 256) { Ms[r] = -INFINITY; Ls[r] = 0.f; }

  constexpr int C4 = D / 4;               // float4 columns
  constexpr int RSTEP = 256 / C4;         // rows covered per pass
  constexpr int MAXU = (128 + RSTEP - 1) / RSTEP;
  const int c4 = tid % C4, r0 = tid / C4;
  float4 o[MAXU];
#pragma unroll
  for (int u = 0; u < MAXU; ++u) o[u] = make_float4(0.f, 0.f, 0.f, 0.f);
  __syncthreads();

  for (int t0 = s0; t0 < s1; t0 += kTKMany) {
    // stage K and V rows of this tile as fp32
    for (int idx = tid; idx < kTKMany * (D / Elem<T>::kPer16B); idx += 256) {
      constexpr int VPR = D / Elem<T>::kPer16B;
      const int j = idx / VPR, vc = idx % VPR;
      const int p = t0 + j;
      float kf[8], vf[8];
      if (p < s1) {
        const size_t at = kv_entry(a, b, g, p) * VPR + vc;
        const uint4 kraw = static_cast<const uint4*>(a.k)[at];
        const uint4 vraw = static_cast<const uint4*>(a.v)[at];
        if (Elem<T>::kPer16B == 8) {
          unpack16(kraw, kf);
          unpack16(vraw, vf);
        } else {
          kf[0] = __uint_as_float(kraw.x); kf[1] = __uint_as_float(kraw.y);
          kf[2] = __uint_as_float(kraw.z); kf[3] = __uint_as_float(kraw.w);
          vf[0] = __uint_as_float(vraw.x); vf[1] = __uint_as_float(vraw.y);
          vf[2] = __uint_as_float(vraw.z); vf[3] = __uint_as_float(vraw.w);
        }
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) { kf[e] = 0.f; vf[e] = 0.f; }
      }
#pragma unroll
      for (int e = 0; e < Elem<T>::kPer16B; ++e) {
        Ks[j * DP + vc * Elem<T>::kPer16B + e] = kf[e];
        Vs[j * DP + vc * Elem<T>::kPer16B + e] = vf[e];
      }
    }
    __syncthreads();
    // scores with the block mask applied
    for (int idx = tid; idx < R * kTKMany; idx += 256) {
      const int r = idx / kTKMany, j = idx % kTKMany;
      const int p = t0 + j;
      bool vis = p < s1;
      if (vis && p >= L) {
        const int i = (r * a.g_inv) >> 16;
        const uint64_t row = a.mask ? a.mask[static_cast<size_t>(b) * a.mask_stride + i] : ((2ull << i) - 1ull);
        vis = (row >> (p - L)) & 1ull;
      }
      float acc = 0.f;
      if (vis) {
        const float4* qv = reinterpret_cast<const float4*>(Qs + r * D);
        const float4* kv = reinterpret_cast<const float4*>(Ks + j * DP);
#pragma unroll 8
        for (int c = 0; c < C4; ++c) {
          const float4 x = qv[c], y = kv[c];
          acc = fmaf(x.x, y.x, acc); acc = fmaf(x.y, y.y, acc);
          acc = fmaf(x.z, y.z, acc); acc = fmaf(x.w, y.w, acc);
        }
      }
      Ss[idx] = vis ? acc * a.scale : -INFINITY;
    }
    __syncthreads();
    // online softmax bookkeeping, one thread per row
    for (int r = tid; r < R; r += 256) {
      float tmax = -INFINITY;
      for (int j = 0; j < kTKMany; ++j) tmax = fmaxf(tmax, Ss[r * kTKMany + j]);
      const float m_old = Ms[r];
      const float m_new = fmaxf(m_old, tmax);
      float alpha = 1.f, sum = 0.f;
      if (m_new == -INFINITY) {
        for (int j = 0; j < kTKMany; ++j) Ss[r * kTKMany + j] = 0.f;
      } else {
        alpha = (m_old == -INFINITY) ? 0.f : expf(m_old - m_new);
        for (int j = 0; j < kTKMany; ++j) {
          const float pj = expf(Ss[r * kTKMany + j] - m_new);  // exp(-inf) = 0 for masked keys
          Ss[r * kTKMany + j] = pj;
          sum += pj;
        }
      }
      Ms[r] = m_new;
      Ls[r] = Ls[r] * alpha + sum;
      As[r] = alpha;
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < MAXU; ++u) {
      const int r = r0 + u * RSTEP;
      if (r < R) {
        const float al = As[r];
        float4 acc = make_float4(o[u].x * al, o[u].y * al, o[u].z * al, o[u].w * al);
        for (int j = 0; j < kTKMany; ++j) {
          const float pj = Ss[r * kTKMany + j];
          const float4 vv = *reinterpret_cast<const float4*>(Vs + j * DP + c4 * 4);
          acc.x = fmaf(pj, vv.x, acc.x); acc.y = fmaf(pj, vv.y, acc.y);
          acc.z = fmaf(pj, vv.z, acc.z); acc.w = fmaf(pj, vv.w, acc.w);
        }
        o[u] = acc;
      }
    }
    __syncthreads();
  }
  const size_t unit = static_cast<size_t>(blockIdx.x) + static_cast<size_t>(b) * a.Hkv + g;   // partial slot of segment (w, u)
#pragma unroll
  for (int u = 0; u < MAXU; ++u) {
    const int r = r0 + u * RSTEP;
    if (r < R) *reinterpret_cast<float4*>(a.part_o + (unit * R + r) * D + c4 * 4) = o[u];
  }
  for (int r = tid; r < R; r += 256) {
    a.part_ml[(unit * R + r) * 2 + 0] = Ms[r];
    a.part_ml[(unit * R + r) * 2 + 1] = Ls[r];
  }
  __syncthreads();   // a further segment restarts the running maxima and sums
  }
}

// One output row of a launch with two-part probabilities again, by one wave, with fp32 ones.  The matrix-core kernel
// multiplies V with a probability in two parts, of which the second is 0 or negative as often as not: an infinite V
// entry then becomes inf - inf or 0 inf, although its probability is positive.  So the merging kernels hand every row
// that is not finite to this function: infinities come out as the one product p v gives them, and NaN where the
// inputs ask for it (a NaN among them, infinities of both signs, an infinite entry that the mask hides: 0 inf).
// A lane takes eight columns of a key, eight or four keys go together, and the running maximum moves with them.  A launch without
// such rows pays for the test only (verify_attn, 8 sequences of 1000-8000 entries, 16 queries: 35.0 -> 35.7 us; 64 of
// 500, 8 queries: 27 us either way); one in which every row is infinite takes 1.2 ms at the first of these sizes.
template <int D>
__device__ __forceinline__ void attn_row_again(const AttnArgs& a, int b, int i, int h) {
  constexpr int LPK = D / 8, KPW = 64 / LPK;     // lanes of a key, keys of a wave
  const int lane = threadIdx.x & 63;
  const int kq = lane / LPK, c = lane % LPK;
  const int G = a.Hq / a.Hkv, g = h / G;
  const int L = attn_ctx_len(a, b), n = L + a.n_blk;
  const size_t row = ((static_cast<size_t>(b) * a.n_q + i) * a.Hq + h) * D;
  const uint64_t seen = a.mask ? a.mask[static_cast<size_t>(b) * a.mask_stride + i] : ((2ull << i) - 1ull);
  float q[8], acc[8], m = -INFINITY, sum = 0.f;
  unpack16(*reinterpret_cast<const uint4*>(static_cast<const bf16_t*>(a.q) + row + 8 * c), q);
#pragma unroll
  for (int e = 0; e < 8; ++e) acc[e] = 0.f;
#pragma unroll 1
  for (int p0 = 0; p0 < n; p0 += KPW) {
    const int p = p0 + kq;
    const bool in = p < n;
    const size_t at = kv_entry(a, b, g, min(p, n - 1)) * LPK + c;
    const uint4 kr = static_cast<const uint4*>(a.k)[at], vr = static_cast<const uint4*>(a.v)[at];
    float kf[8], vf[8], x = 0.f;
    unpack16(kr, kf);
    unpack16(vr, vf);
#pragma unroll
    for (int e = 0; e < 8; ++e) x = fmaf(q[e], kf[e], x);
#pragma unroll
    for (int o = 1; o < LPK; o <<= 1) x += __shfl_xor(x, o, 64);
    const bool vis = in && (p < L || (seen >> (p - L) & 1ull));
    x = vis ? x * a.scale : -INFINITY;
    float mt = x;
#pragma unroll
    for (int o = LPK; o < 64; o <<= 1) mt = fmaxf(mt, __shfl_xor(mt, o, 64));
    const float m_new = fmaxf(m, mt);
    float al = 1.f, pr = 0.f;
    if (m_new != -INFINITY) {
      al = m == -INFINITY ? 0.f : expf(m - m_new);
      pr = expf(x - m_new);
    }
    if (x != x) pr = x;                       // (also where no score has been a number yet)
    m = m_new;
    sum = fmaf(sum, al, pr);
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] = fmaf(pr, in ? vf[e] : 0.f, acc[e] * al);
  }
#pragma unroll
  for (int o = LPK; o < 64; o <<= 1) {
    sum += __shfl_xor(sum, o, 64);
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] += __shfl_xor(acc[e], o, 64);
  }
  __threadfence();                  // the first result has been stored
  if (kq == 0) {
    bf16_t* dst = static_cast<bf16_t*>(a.out) + row + 8 * c;
#pragma unroll
    for (int e = 0; e < 8; ++e) Elem<bf16_t>::store(dst + e, acc[e] / sum);
  }
}
// (uniform over the wave: one of its lanes holds a value that is no number or infinite)
__device__ __forceinline__ bool any_not_finite(float v) { return __builtin_amdgcn_ballot_w64(!(fabsf(v) < INFINITY)) != 0ull; }

// The segments of an output row: consecutive slots, one per workgroup whose share holds keys of its unit.
struct RowSegs {
  const float *ml, *po;   // segment s: (max, sum) at ml[s * ml_step], partial output at po[s * po_step]
  size_t ml_step, po_step;
  int n;
};
template <int D>
__device__ __forceinline__ RowSegs row_segments(const AttnArgs& a, int b, int i, int h) {
  const int G = a.G, R = G * a.n_q, g = h / G, r = i * G + h - g * G;
  typedef const __attribute__((address_space(4))) int* words_t;           // (scalar loads: nothing writes these words meanwhile)
  const int u = b * a.Hkv + g;
  const words_t ends = (words_t)a.sched + 2 * u;
  const int w_first = ends[0], w_last = ends[1];
  const size_t slot = static_cast<size_t>(w_first) + u;
  RowSegs q;
  q.n = w_last - w_first + 1;
  q.ml = a.part_ml + (slot * R + r) * 2;
  q.po = a.part_o + (slot * R + r) * D;
  q.ml_step = 2 * static_cast<size_t>(R);
  q.po_step = static_cast<size_t>(R) * D;
  return q;
}
__device__ __forceinline__ float seg_exp(const AttnArgs& a, float x) { return a.use_mfma ? exp2f(x) : expf(x); }

// A segment's part of the sum.  NaN counts whatever the weight: a maximum passes NaN over, so that a segment whose scores are NaN
// can be left with the lowest one.
__device__ __forceinline__ float seg_sum(float w, float l) { return w != 0.f || l != l ? w * l : 0.f; }

// Merge the segments of one (sequence, query, head): exact log-sum-exp combination.  One workgroup per output row; groups
// of lanes take every NG-th segment of one float4 column and are added in a fixed order.
// Latency is all there is (a row reads 17 KB at 33 segments): the two words with the unit's workgroups, one round to memory, a
// meeting of the groups.  The first kEarly partial outputs of every group are requested together with the (max, sum) pairs,
// every wave works out all weights for itself (lane s holds those of segments s, s + 64, ..), and the maximum and the sum over
// the lanes are taken without LDS: no barrier before the one at which the groups meet.  Segments beyond 64 in rounds.
constexpr int kCombThreads = 256;
constexpr int kEarly = 6;

template <typename T, int D>
__global__ __launch_bounds__(kCombThreads) void k_attn_combine(const AttnArgs a) {
  constexpr int C4 = D / 4;                 // float4 columns of a row
  constexpr int NG = kCombThreads / C4;     // groups
  __shared__ float4 gs[NG][C4];
  arguments_at_once<sizeof(AttnArgs)>();
  const int h = blockIdx.x, i = blockIdx.y, b = blockIdx.z;
  const int lane = threadIdx.x & 63;
  const RowSegs q = row_segments<D>(a, b, i, h);
  const int sg = threadIdx.x / C4, c4 = threadIdx.x % C4;
  const float* po = q.po + c4 * 4;
  float2 ml = *reinterpret_cast<const float2*>(q.ml + min(lane, q.n - 1) * q.ml_step);
  float4 o[kEarly];
#pragma unroll
  for (int u = 0; u < kEarly; ++u) o[u] = *reinterpret_cast<const float4*>(po + min(sg + u * NG, q.n - 1) * q.po_step);
  float mmax = ml.x;
  for (int s = 64 + lane; s < q.n; s += 64) mmax = fmaxf(mmax, q.ml[s * q.ml_step]);
  mmax = wave_max_dpp(mmax);
  float den = 0.f;
  float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int s0 = 0; s0 < q.n; s0 += 64) {
    if (s0 > 0) ml = *reinterpret_cast<const float2*>(q.ml + min(s0 + lane, q.n - 1) * q.ml_step);
    const float w = s0 + lane < q.n && ml.x != -INFINITY ? seg_exp(a, ml.x - mmax) : 0.f;
    den += seg_sum(w, ml.y);                // (lane by lane, summed behind the loop)
    const int n = min(64, q.n - s0);
    for (int sb = 0; sb < n; sb += kEarly * NG) {     // (uniform: a shuffle reads lanes that take part only)
      const int s = sb + sg;
      if (s0 + sb > 0) {
#pragma unroll
        for (int u = 0; u < kEarly; ++u) o[u] = *reinterpret_cast<const float4*>(po + (s0 + min(s + u * NG, n - 1)) * q.po_step);
      }
#pragma unroll
      for (int u = 0; u < kEarly; ++u) {
        float wu = __shfl(w, min(s + u * NG, n - 1), 64);
        if (s + u * NG >= n) wu = 0.f;
        if (wu != 0.f) {
          acc.x = fmaf(wu, o[u].x, acc.x); acc.y = fmaf(wu, o[u].y, acc.y);
          acc.z = fmaf(wu, o[u].z, acc.z); acc.w = fmaf(wu, o[u].w, acc.w);
        }
      }
    }
  }
  gs[sg][c4] = acc;
  den = wave_sum_dpp(den);
  __syncthreads();
  float4 sum = make_float4(0.f, 0.f, 0.f, 0.f);
  if (sg == 0) {
    float4 v[NG];
#pragma unroll
    for (int u = 0; u < NG; ++u) v[u] = gs[u][c4];
    sum = v[0];
#pragma unroll
    for (int u = 1; u < NG; ++u) { sum.x += v[u].x; sum.y += v[u].y; sum.z += v[u].z; sum.w += v[u].w; }
    if constexpr (sizeof(T) == 2) {
      const float inv = 1.0f / den;            // (rounded to bf16 below; four divisions are 0.5 % slower, and no digit of the error against 64 bits moves)
      sum.x *= inv; sum.y *= inv; sum.z *= inv; sum.w *= inv;
    } else {
      sum.x /= den; sum.y /= den; sum.z /= den; sum.w /= den;
    }
  }
  if (sg == 0) {
    T* dst = static_cast<T*>(a.out) + ((static_cast<size_t>(b) * a.n_q + i) * a.Hq + h) * D + c4 * 4;
    // (as bytes: the caller's buffer may begin at any element, which these stores take in one instruction all the same)
    if constexpr (sizeof(T) == 2) {
      const uint2 v = make_uint2(pack_bf16x2(sum.x, sum.y), pack_bf16x2(sum.z, sum.w));
      __builtin_memcpy(dst, &v, sizeof(v));
    } else {
      __builtin_memcpy(dst, &sum, sizeof(sum));
    }
  }
  if constexpr (sizeof(T) == 2) {             // (behind the store, off the way of it)
    if (__builtin_expect(a.use_mfma == kTwoPart && threadIdx.x < 64 && any_not_finite((sum.x + sum.y) + (sum.z + sum.w)), 0)) attn_row_again<D>(a, b, i, h);
  }
}

// The same with one wave per output row: for many rows, where a workgroup each spends its time starting.  The first
// segments' partial outputs are requested with the (max, sum) pairs, and sixteen together from there on, so that a unit of many
// segments in a batch of short ones costs a few memory round trips (four at a time: one context of 32768 among 15 of 300, 2
// queries, 41.7 us; 38.6 this way).
constexpr int kRowEarly = 4;

template <typename T, int D>
__global__ __launch_bounds__(256) void k_attn_combine_rows(const AttnArgs a) {
  constexpr int EPL = D / 64;               // columns per lane
  arguments_at_once<sizeof(AttnArgs)>();
  const int lane = threadIdx.x & 63;
  const int row = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + (threadIdx.x >> 6));
  if (row >= a.B * a.n_q * a.Hq) return;
  const int b = row / (a.n_q * a.Hq), ih = row - b * (a.n_q * a.Hq), i = ih / a.Hq, h = ih - i * a.Hq;
  const RowSegs q = row_segments<D>(a, b, i, h);
  const float* po = q.po + lane * EPL;
  float2 ml = *reinterpret_cast<const float2*>(q.ml + min(lane, q.n - 1) * q.ml_step);
  float first[kRowEarly][EPL];
#pragma unroll
  for (int u = 0; u < kRowEarly; ++u)
#pragma unroll
    for (int e = 0; e < EPL; ++e) first[u][e] = po[min(u, q.n - 1) * q.po_step + e];
  float mmax = ml.x;
  for (int s = 64 + lane; s < q.n; s += 64) mmax = fmaxf(mmax, q.ml[s * q.ml_step]);
  mmax = wave_max_dpp(mmax);
  float den = 0.f, acc[EPL];
#pragma unroll
  for (int e = 0; e < EPL; ++e) acc[e] = 0.f;
  auto add = [&](float w, const float (&o)[EPL]) {
    if (w != 0.f) {
#pragma unroll
      for (int e = 0; e < EPL; ++e) acc[e] = fmaf(w, o[e], acc[e]);
    }
  };
  for (int s0 = 0; s0 < q.n; s0 += 64) {
    if (s0 > 0) ml = *reinterpret_cast<const float2*>(q.ml + min(s0 + lane, q.n - 1) * q.ml_step);
    const float w = s0 + lane < q.n && ml.x != -INFINITY ? seg_exp(a, ml.x - mmax) : 0.f;
    den += seg_sum(w, ml.y);                // (lane by lane, summed behind the loop)
    auto weight = [&](int j) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(w), j)); };
    const int n = min(64, q.n - s0);
    int j = 0;
    if (s0 == 0) {
#pragma unroll
      for (int u = 0; u < kRowEarly; ++u)
        if (u < n) add(weight(u), first[u]);
      j = kRowEarly;
    }
    for (; j < n; j += 16) {
      float o[16][EPL];
#pragma unroll
      for (int u = 0; u < 16; ++u)
#pragma unroll
        for (int e = 0; e < EPL; ++e) o[u][e] = po[(s0 + min(j + u, n - 1)) * q.po_step + e];
#pragma unroll
      for (int u = 0; u < 16; ++u)
        if (j + u < n) add(weight(j + u), o[u]);
    }
  }
  den = wave_sum_dpp(den);
  T* dst = static_cast<T*>(a.out) + static_cast<size_t>(row) * D + lane * EPL;
#pragma unroll
  for (int e = 0; e < EPL; ++e) Elem<T>::store(dst + e, acc[e] / den);
  if constexpr (sizeof(T) == 2) {
    if (__builtin_expect(a.use_mfma == kTwoPart && any_not_finite((D == 64 ? acc[0] : acc[0] + acc[EPL - 1]) / den), 0)) attn_row_again<D>(a, b, i, h);
  }
}

template <typename T, int D>
hipError_t launch_combine(const AttnArgs& a, hipStream_t s) {
  // A workgroup per row costs about 1 us per 1000 rows, a wave per row about 0.05 us per segment of the unit.  Whole
  // calls, workgroup / wave, 32768 entries in all, 32 query heads over 8 KV heads:
  //   segments per unit    64          32          16          8           4           2           1
  //   1 query              29.9 / 32.6 29.4 / 30.7 29.2 / 29.8 29.4 / 29.8 30.2 / 29.8 30.7 / 30.0 31.4 / 30.6
  //   5 queries            30.3 / 32.8 30.1 / 30.9 30.2 / 30.3 31.2 / 30.3 34.2 / 31.4 37.6 / 32.5 44.1 / 34.0
  //   12 queries           44.3 / 47.4 44.3 / 44.4 44.1 / 43.7 47.0 / 43.8 51.0 / 45.2 59.3 / 48.9 75.7 / 55.0
  // The lengths are not known here, and one long sequence among short ones has more segments than the average: 32768
  // among n - 1 of 300, n = 16 / 32 / 64, 2 queries 36.4 / 38.6, 39.6 / 40.4, 61.5 / 59.0, 8 queries 45.2 / 43.2, 54.2 / 48.2,
  // 86 / 72.  So the wave's side starts at 256 rows per segment of an average unit, where it leads with room to spare.
  const int64_t units = static_cast<int64_t>(a.B) * a.Hkv;
  const int64_t rows = static_cast<int64_t>(a.B) * a.n_q * a.Hq;
  if (rows * units > 256 * static_cast<int64_t>(a.wgrid)) {
    hipLaunchKernelGGL((k_attn_combine_rows<T, D>), dim3(static_cast<unsigned>((rows + 3) / 4)), dim3(256), 0, s, a);
  } else {
    hipLaunchKernelGGL((k_attn_combine<T, D>), dim3(a.Hq, a.n_q, a.B), dim3(kCombThreads), 0, s, a);
  }
  return hipGetLastError();
}

template <typename T, int D, int ROWS>
hipError_t launch_valu_as(const AttnArgs& a, int R, hipStream_t s) {
  // set once per process; a function-local static is initialised under the language's own lock,
  // so first calls from several host threads are safe
  static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_attn_split_valu<T, D, ROWS>),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, kValuLds);
  if (attr != hipSuccess) return attr;
  hipLaunchKernelGGL((k_attn_split_valu<T, D, ROWS>), dim3(a.wgrid), dim3(256), valu_lds_bytes(R, D, a.B), s, a);
  return hipGetLastError();
}

template <typename T, int D>
hipError_t launch_valu(const AttnArgs& a, hipStream_t s) {
  const int R = a.G * a.n_q;
  if constexpr (D == 128) {
    if (R > valu_rows_most(D)) {
      static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_attn_split_rows<T, D>),
                                                         hipFuncAttributeMaxDynamicSharedMemorySize, kValuLds);
      if (attr != hipSuccess) return attr;
      hipLaunchKernelGGL((k_attn_split_rows<T, D>), dim3(a.wgrid), dim3(256), many_lds_bytes(R, D, a.B), s, a);
      return hipGetLastError();
    }
  }
  return R <= valu_rows_few(D) ? launch_valu_as<T, D, valu_rows_few(D)>(a, R, s) : launch_valu_as<T, D, valu_rows_most(D)>(a, R, s);
}

}  // namespace

// Padding of the units (attn_sched.hpp), in granules: what starting a segment costs.  Per layer, 0 / 1 / 2 / 3 granules, 8 KV heads, mean
// context 300 .. 900, G = 4: 64 sequences x 1 query 26.0 / 24.1 / 24.3 / 24.7 us, x 11 42.9 / 42.6 / 42.4 / 42.0; 16 x 11 (900)
// 30.8 / 29.9 / 28.9 / 29.0; 64-wide heads, 64 x 8 (600) 34.3 / 32.8 / 32.2 / 32.1.  With one sequence, whose units are few, it
// does not matter.
static int unit_pad(const AttnArgs& a) { return a.d == 64 ? 3 : 2; }

// Granules from which two workgroups per compute unit are worth their partial results, of which each writes R rows that are read
// again.  Per layer, 256 / 512 workgroups, T granules: R = 4 rows: 1 sequence, T = 1800 19.4 / 18.8 us, 3200 26.6 / 24.8;
// 20 rows: 1 sequence, 1800 20.0 / 20.8, 2400 23.4 / 23.5, 3200 27.5 / 26.6; 4 sequences, 1800 20.9 / 19.7; 44 rows: 1 sequence,
// 2400 25.9 / 28.1, 4800 37.9 / 38.4; 16 sequences, 2400 28.1 / 28.9, 3200 32.8 / 33.2.  With more units than compute units
// every workgroup writes several of them anyway, and the second one is at work while the first starts a unit: 64
// sequences, 44 rows, 1200 34.0 / 33.0, 4800 54.7 / 50.1.  64-wide heads, granules of half the bytes, 32 rows: 1 sequence, 1200
// 12.6 / 14.2, 2400 15.7 / 17.8, 4800 22.2 / 22.1; 64 sequences, 2400 28.9 / 26.0; 64 rows: 8 sequences, 4500 27.7 / 26.6 (there the
// second workgroup's waves are wanted for the arithmetic as well).
// (The figures of 4 rows are a draft step's.)  Verifications of up to 16 rows of 128-wide heads have one workgroup per compute unit at
// any length: from the line on all 256 take part, below it the fewest with the same largest share, whose number suits units of one
// length.  The fewest instead of 256, 3 to 12 sequences of equal and of unequal lengths, 8 KV heads, 8 rows: T = 1630-1850 -1 %, 2300
// -1 %, 2400 +0.6 %, 3000 -0.4 %, 4300 +0.8 %, 6800 -0.2 %; 6 of 3000 entries (T = 2256) 19.9 -> 19.0 us, 16 rows, paged, 23.1 -> 20.8.
constexpr int kAllFrom = 2400;
static int wide_from(const AttnArgs& a) {
  if (!a.use_mfma || static_cast<int64_t>(a.B) * a.Hkv >= kAttnSpread) return 0;
  if (a.rings > 2 && attn_mfma_per_cu(a) == 1) return kAllFrom;
  return 1000 + std::min(a.G * a.n_q * (a.d == 64 ? 80 : 50), 2600);
}

static bool plan_as(AttnArgs& a, int num_cus, int use_mfma, int pad) {
  // The host knows only the upper bound l_max of the lengths; the kernels deal the keys that
  // are really there to the workgroups in equal shares.  Here only the number of workgroups is
  // set: as many as are resident at once (one or two of the matrix-core kernel per compute unit),
  // fewer when even the longest possible caches would leave them too few granules
  // (attn_sched_line), more when a share could otherwise exceed what one segment can hold.
  a.use_mfma = use_mfma ? (attn_mfma_two_part(a) ? kTwoPart : kOnePart) : 0;
  a.G = a.Hq / a.Hkv;
  a.g_inv = (65536 + a.G - 1) / a.G;
  a.pad = pad;
  if (a.B > kAttnMaxSeqs || a.l_max < a.n_blk) return false;
  const int64_t units = static_cast<int64_t>(a.B) * a.Hkv;
  const int64_t gmax = (a.l_max + kAttnGran - 1) / kAttnGran;      // granules of the longest possible unit
  if (units * (gmax + pad) >= (1ll << 30)) return false;
  a.rings = a.use_mfma ? attn_mfma_rings(a) : 0;
  a.wide_from = wide_from(a);
  a.stages = a.use_mfma ? attn_mfma_stages(a) : 0;
  const int64_t resident = static_cast<int64_t>(num_cus) * (a.use_mfma ? attn_mfma_per_cu(a) : 1);
  const AttnLine line = attn_sched_line(static_cast<int>(a.B * gmax), a.B, a.Hkv, pad, a.wide_from, a.use_mfma == kOnePart, static_cast<int>(resident));
  int64_t w = line.W;
  if (line.T > kAttnSpread && w < kAttnSpread) w = std::min<int64_t>(kAttnSpread, resident);   // (fewer granules may take more workgroups)
  if (a.use_mfma) {
    const int64_t seg_gran = attn_mfma_max_chunk(a) / kAttnGran;   // granules one segment may span
    const int64_t need = (line.T + seg_gran - 1) / seg_gran;
    if (w < need) w = need;
  }
  if (w > kAttnMaxGrid) return false;
  a.wgrid = static_cast<int>(w);
  return true;
}

bool attn_plan(AttnArgs& a, int num_cus) {
  if (!attn_mfma_supported(a)) return plan_as(a, num_cus, 0, 0);
  // The matrix-core kernel keeps the page ids of a segment in LDS, which bounds a segment and so asks for
  // many workgroups where the page tables could hold hundreds of millions of entries.  Where that is
  // more than a launch has, 64-wide heads go to the ALU kernel, whose segments are unbounded.
  return plan_as(a, num_cus, 1, unit_pad(a)) || plan_as(a, num_cus, 1, 0) || (a.d == 64 && plan_as(a, num_cus, 0, 0));
}

int attn_slots(const AttnArgs& a) { return a.wgrid + a.B * a.Hkv; }

size_t attn_workspace_bytes(const AttnArgs& a) {
  const size_t R = static_cast<size_t>(a.Hq / a.Hkv) * a.n_q;
  const size_t slots = static_cast<size_t>(attn_slots(a));
  size_t o = slots * R * a.d * sizeof(float);
  o = (o + 255) & ~static_cast<size_t>(255);
  size_t ml = slots * R * 2 * sizeof(float);
  ml = (ml + 255) & ~static_cast<size_t>(255);
  size_t sc = static_cast<size_t>(a.B) * a.Hkv * 2 * sizeof(int);
  sc = (sc + 255) & ~static_cast<size_t>(255);
  return o + ml + sc;
}

void attn_carve(AttnArgs& a, void* workspace) {
  const size_t R = static_cast<size_t>(a.Hq / a.Hkv) * a.n_q;
  const size_t slots = static_cast<size_t>(attn_slots(a));
  char* p = static_cast<char*>(workspace);
  a.part_o = reinterpret_cast<float*>(p);
  p += (slots * R * a.d * sizeof(float) + 255) & ~static_cast<size_t>(255);
  a.part_ml = reinterpret_cast<float*>(p);
  p += (slots * R * 2 * sizeof(float) + 255) & ~static_cast<size_t>(255);
  a.sched = reinterpret_cast<int*>(p);
}

hipError_t launch_attn(const AttnArgs& a, hipStream_t s, KernelHook hook, int hook_id) {
  hipError_t e;
  if (hook) hook(hook_id, 0, s);
  if (a.use_mfma) {
    e = launch_attn_mfma(a, s);
  } else if (a.dtype == 1) {
    e = a.d == 128 ? launch_valu<bf16_t, 128>(a, s) : launch_valu<bf16_t, 64>(a, s);
  } else {
    e = a.d == 128 ? launch_valu<float, 128>(a, s) : launch_valu<float, 64>(a, s);
  }
  if (hook) hook(hook_id, 1, s);
  if (e != hipSuccess) return e;
  if (a.dtype == 1) return a.d == 128 ? launch_combine<bf16_t, 128>(a, s) : launch_combine<bf16_t, 64>(a, s);
  return a.d == 128 ? launch_combine<float, 128>(a, s) : launch_combine<float, 64>(a, s);
}

}  // namespace sx
