// Plain fp32 ALU GEMM  out[m][n] = sum_k act[m][k] * w[n][k]  (the fp32 LM head, and any shape the row-streaming and
// matrix-core kernels reject; HBM-bound, 16-byte loads coalesced along K), and the small kernels behind the heads: merging of
// argmax / ranked candidates, signal activations.
#include "common.hpp"
#include "kernels.hpp"

#include <limits.h>

namespace sx {

namespace {

struct SegRef {
  const char* base;  // first row of the segment
  int row0;          // its first logical row
  int rows;          // rows in the segment
};

__device__ __forceinline__ SegRef find_segment(const GemmArgs& g, int n) {
  SegRef r;
  int start = 0;
  int s = 0;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    if (s + 1 < g.nseg && n >= g.seg_end[s]) {
      start = g.seg_end[s];
      ++s;
    }
  }
  r.base = static_cast<const char*>(g.w[s]);
  r.row0 = start;
  r.rows = g.seg_end[s] - start;
  return r;
}

// ------------------------------------------------------------------------- VALU path
// A wave takes NR weight rows and up to eight activation rows (blockIdx.y: which eight).  With several activation
// rows their reads are the bound (every weight row reads all of them from L1 / L2), so four weight rows share them;
// with one or two, one weight row per wave gives the most waves.
template <typename WT, int NR>
__global__ __launch_bounds__(256) void k_gemv_valu(const GemmArgs g) {
  constexpr int EPV = Elem<WT>::kPer16B;
  const int lane = threadIdx.x & 63;
  const int n = (blockIdx.x * 4 + (threadIdx.x >> 6)) * NR;
  if (n >= g.N) return;
  const SegRef sg = find_segment(g, n);        // (segment ends are multiples of 4: the rows lie in one)
  const uint4* wrow[NR];
#pragma unroll
  for (int r = 0; r < NR; ++r)
    wrow[r] = reinterpret_cast<const uint4*>(sg.base + static_cast<size_t>(min(n - sg.row0 + r, sg.rows - 1)) * g.K * sizeof(WT));
  const int nvec = g.K / EPV;
  const int m0 = blockIdx.y * 8;
  const int mc = min(8, g.M - m0);
  float acc[8][NR];
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int r = 0; r < NR; ++r) acc[i][r] = 0.f;
  for (int c = lane; c < nvec; c += 64) {
    float wf[NR][8];
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      const uint4 wv = wrow[r][c];
      if (EPV == 8) {
        unpack16(wv, wf[r]);
      } else {
        wf[r][0] = __uint_as_float(wv.x); wf[r][1] = __uint_as_float(wv.y);
        wf[r][2] = __uint_as_float(wv.z); wf[r][3] = __uint_as_float(wv.w);
      }
    }
#pragma unroll
    for (int mm = 0; mm < 8; ++mm) {
      if (mm < mc) {
        const float* a = g.act + static_cast<size_t>(m0 + mm) * g.K + static_cast<size_t>(c) * EPV;
#pragma unroll
        for (int e = 0; e < EPV; e += 4) {
          const float4 av = *reinterpret_cast<const float4*>(a + e);
#pragma unroll
          for (int r = 0; r < NR; ++r) {
            acc[mm][r] = fmaf(av.x, wf[r][e + 0], acc[mm][r]);
            acc[mm][r] = fmaf(av.y, wf[r][e + 1], acc[mm][r]);
            acc[mm][r] = fmaf(av.z, wf[r][e + 2], acc[mm][r]);
            acc[mm][r] = fmaf(av.w, wf[r][e + 3], acc[mm][r]);
          }
        }
      }
    }
  }
#pragma unroll
  for (int mm = 0; mm < 8; ++mm) {
    if (mm < mc) {
#pragma unroll
      for (int r = 0; r < NR; ++r) {
        const float v = wave_sum(acc[mm][r]);
        if (lane == 0 && n + r < g.N) g.partial[static_cast<size_t>(m0 + mm) * g.N + n + r] = v;
      }
    }
  }
}

constexpr int kFinalThreads = 1024;

// Signal logits -> signals: confidence and progress pass through a sigmoid (Eqs. 3-4); the remaining-length head
// regresses log(1 + r) (Eq. 5), so r = expm1(z), floored at zero (or the activation the descriptor names)
__device__ __forceinline__ void write_signals(const float* z, int rem_activation, float* sig_raw, float* sig) {
  const float zc = z[0], zp = z[1], zr = z[2];
  sig_raw[0] = zc; sig_raw[1] = zp; sig_raw[2] = zr;
  sig[0] = sigmoidf_(zc);
  sig[1] = sigmoidf_(zp);
  sig[2] = rem_activation == 0 ? fmaxf(0.f, expm1f(zr)) : (rem_activation == 1 ? sigmoidf_(zr) : zr);
}

// One block per activation row: reduce the (max, index) candidates; for the draft head
// the same block also turns the three signal logits into signals (Eqs. 3-5).
__global__ __launch_bounds__(kFinalThreads) void k_argmax_finalize(const float* __restrict__ part_val,
                                                                   const int* __restrict__ part_idx, int ntiles,
                                                                   int32_t* __restrict__ argmax,
                                                                   float* __restrict__ max_logit,
                                                                   const float* __restrict__ extra,
                                                                   int rem_activation, float* __restrict__ sig_raw,
                                                                   float* __restrict__ sig) {
  __shared__ float sv[kFinalThreads / 64];
  __shared__ int si[kFinalThreads / 64];
  const int m = blockIdx.x;
  float bv = -INFINITY;
  int bi = INT_MAX;
  constexpr int U = 2;   // candidates per thread requested at once (256 workgroups x up to 4 slots, or 512 of the row stream: 1)
  for (int t0 = threadIdx.x; t0 < ntiles; t0 += U * kFinalThreads) {
    float v[U];
    int i[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int t = t0 + u * kFinalThreads;
      const bool ok = t < ntiles;
      v[u] = ok ? part_val[static_cast<size_t>(m) * ntiles + t] : -INFINITY;
      i[u] = ok ? part_idx[static_cast<size_t>(m) * ntiles + t] : INT_MAX;
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (better(v[u], i[u], bv, bi)) { bv = v[u]; bi = i[u]; }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const float ov = __shfl_xor(bv, o, 64);
    const int oi = __shfl_xor(bi, o, 64);
    if (better(ov, oi, bv, bi)) { bv = ov; bi = oi; }
  }
  if ((threadIdx.x & 63) == 0) { sv[threadIdx.x >> 6] = bv; si[threadIdx.x >> 6] = bi; }
  __syncthreads();
  if (threadIdx.x < 64) {
    // the 16 waves' results, one per lane, merged by a butterfly
    const bool have = threadIdx.x < kFinalThreads / 64;
    bv = have ? sv[threadIdx.x] : -INFINITY;
    bi = have ? si[threadIdx.x] : INT_MAX;
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) {
      const float ov = __shfl_xor(bv, o, 64);
      const int oi = __shfl_xor(bi, o, 64);
      if (better(ov, oi, bv, bi)) { bv = ov; bi = oi; }
    }
    if (threadIdx.x == 0) {
      argmax[m] = bi;
      if (max_logit) max_logit[m] = bv;
    }
  }
  if (sig && threadIdx.x == 64) write_signals(extra + m * 3, rem_activation, sig_raw + m * 3, sig + m * 3);
}

// The top_b best of each row, best first (value descending, lower index first among equals),
// from candidate lists (part_idx != nullptr: C pairs per row, INT_MAX marks an
// empty slot) or from a full logits row (part_idx == nullptr: candidate c is (row[c], c)).
// Pass r takes the best candidate that comes after pass r-1's pick in that order.
__global__ __launch_bounds__(kFinalThreads) void k_topb_finalize(const float* __restrict__ vals,
                                                                 const int* __restrict__ idxs, int C, int stride,
                                                                 int top_b, int32_t* __restrict__ cand_tok,
                                                                 float* __restrict__ cand_logit,
                                                                 const float* __restrict__ extra, int rem_activation,
                                                                 float* __restrict__ sig_raw, float* __restrict__ sig) {
  __shared__ float sv[kFinalThreads / 64];
  __shared__ int si[kFinalThreads / 64];
  __shared__ float pick_v;
  __shared__ int pick_i;
  const int m = blockIdx.x;
  const float* rv = vals + static_cast<size_t>(m) * stride;
  const int* ri = idxs ? idxs + static_cast<size_t>(m) * stride : nullptr;
  float prev_v = INFINITY;
  int prev_i = -1;
  // candidate lists (up to 256 workgroups x 4 slots x 4) are read once, all requests at once, and the passes
  // run from registers; a full logits row is streamed in every pass.  Kept short on purpose: this kernel runs
  // once on a cold instruction cache.
  constexpr int U = 4;
  const bool held = ri != nullptr && C <= U * kFinalThreads;
  float hv[U];
  int hi[U];
  if (held) {
    // slot groups past the end are skipped as a whole (a uniform branch); inside the last group
    // the last candidate is read again and marked empty
#pragma unroll
    for (int u = 0; u < U; ++u) {
      hv[u] = -INFINITY;
      hi[u] = INT_MAX;
      if (u * kFinalThreads < C) {
        const int c = threadIdx.x + u * kFinalThreads;
        const int cc = min(c, C - 1);
        const float v = rv[cc];
        const int i = ri[cc];
        hv[u] = v;
        hi[u] = c < C ? i : INT_MAX;
      }
    }
  }
  for (int r = 0; r < top_b; ++r) {
    float bv = -INFINITY;
    int bi = INT_MAX;
    if (held) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (u * kFinalThreads < C) {
          const bool after = (hv[u] < prev_v) | ((hv[u] == prev_v) & (hi[u] > prev_i));
          const bool take = (hi[u] != INT_MAX) & after & better(hv[u], hi[u], bv, bi);
          bv = take ? hv[u] : bv;
          bi = take ? hi[u] : bi;
        }
      }
    } else {
      for (int c = threadIdx.x; c < C; c += kFinalThreads) {
        const float v = rv[c];
        const int i = ri ? ri[c] : c;
        const bool after = v < prev_v || (v == prev_v && i > prev_i);
        if (i != INT_MAX && after && better(v, i, bv, bi)) { bv = v; bi = i; }
      }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      const float ov = __shfl_xor(bv, o, 64);
      const int oi = __shfl_xor(bi, o, 64);
      if (better(ov, oi, bv, bi)) { bv = ov; bi = oi; }
    }
    if ((threadIdx.x & 63) == 0) { sv[threadIdx.x >> 6] = bv; si[threadIdx.x >> 6] = bi; }
    __syncthreads();
    if (threadIdx.x < 64) {
      const bool have = threadIdx.x < kFinalThreads / 64;
      bv = have ? sv[threadIdx.x] : -INFINITY;
      bi = have ? si[threadIdx.x] : INT_MAX;
#pragma unroll
      for (int o = 8; o > 0; o >>= 1) {
        const float ov = __shfl_xor(bv, o, 64);
        const int oi = __shfl_xor(bi, o, 64);
        if (better(ov, oi, bv, bi)) { bv = ov; bi = oi; }
      }
      if (threadIdx.x == 0) {
        cand_tok[m * top_b + r] = bi == INT_MAX ? -1 : bi;
        if (cand_logit) cand_logit[m * top_b + r] = bv;
        pick_v = bv;
        pick_i = bi;
      }
    }
    __syncthreads();
    prev_v = pick_v;
    prev_i = pick_i;
  }
  if (sig && threadIdx.x == 64) write_signals(extra + m * 3, rem_activation, sig_raw + m * 3, sig + m * 3);
}

// One block per row of fp32 logits: argmax over the rows n < V, copy of the signal rows and (debug) of the logits;
// for the draft head also the signals (Eqs. 3-5).  Latency-bound: 1024 threads with four values each under way
// (4096 logits: 7.4 us with 256 threads and one value at a time, plus 2 us for the signals in a launch of their own).
__global__ __launch_bounds__(kFinalThreads) void k_argmax_rows(const float* __restrict__ logits, int N, int V,
                                                     int n_extra, int32_t* __restrict__ argmax,
                                                     float* __restrict__ max_logit,
                                                     float* __restrict__ extra_out,
                                                     float* __restrict__ logits_dbg, int rem_activation,
                                                     float* __restrict__ sig_raw, float* __restrict__ sig) {
  __shared__ float sv[kFinalThreads / 64];
  __shared__ int si[kFinalThreads / 64];
  const int m = blockIdx.x;
  const float* row = logits + static_cast<size_t>(m) * N;
  float bv = -INFINITY;
  int bi = INT_MAX;
  constexpr int U = 4;
  for (int n0 = threadIdx.x; n0 < V; n0 += U * kFinalThreads) {
    float v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = row[min(n0 + u * kFinalThreads, V - 1)];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int n = n0 + u * kFinalThreads;
      if (n < V) {
        if (logits_dbg) logits_dbg[static_cast<size_t>(m) * V + n] = v[u];
        if (better(v[u], n, bv, bi)) { bv = v[u]; bi = n; }
      }
    }
  }
  if (extra_out && static_cast<int>(threadIdx.x) < n_extra) extra_out[m * n_extra + threadIdx.x] = row[V + threadIdx.x];
  if (sig && threadIdx.x == 64) write_signals(row + V, rem_activation, sig_raw + m * 3, sig + m * 3);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const float ov = __shfl_xor(bv, o, 64);
    const int oi = __shfl_xor(bi, o, 64);
    if (better(ov, oi, bv, bi)) { bv = ov; bi = oi; }
  }
  if ((threadIdx.x & 63) == 0) { sv[threadIdx.x >> 6] = bv; si[threadIdx.x >> 6] = bi; }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < kFinalThreads / 64; ++w)
      if (better(sv[w], si[w], bv, bi)) { bv = sv[w]; bi = si[w]; }
    argmax[m] = bi;
    if (max_logit) max_logit[m] = bv;
  }
}

template <typename T>
__global__ __launch_bounds__(256) void k_unpack_rows(const T* __restrict__ src, int K, float* __restrict__ act) {
  const int m = blockIdx.x;
  for (int k = threadIdx.x; k < K; k += 256)
    act[static_cast<size_t>(m) * K + k] = Elem<T>::load(src + static_cast<size_t>(m) * K + k);
}

}  // namespace

__global__ void k_zero_i32(int* p, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0;
}

hipError_t launch_zero_i32(int* p, int n, hipStream_t s) {
  hipLaunchKernelGGL(k_zero_i32, dim3((n + 255) / 256), dim3(256), 0, s, p, n);
  return hipGetLastError();
}

hipError_t launch_gemm_valu(const GemmArgs& g, bool bf16, hipStream_t s) {
  // (fp32, K = 1024: N = 20000 with 4 / 24 rows 31 -> 27.5 / 111 -> 79 us, N = 4096 with 24 rows 26 -> 22.6; with 12 rows,
  // 2048 waves, four weight rows would take 21.7 us against 16.5)
  const int64_t waves4 = static_cast<int64_t>((g.N + 3) / 4) * ((g.M + 7) / 8);
  const int nr = g.M >= 4 && waves4 >= 3000 ? 4 : 1;
  const dim3 grid((g.N + 4 * nr - 1) / (4 * nr), (g.M + 7) / 8);
  if (bf16) {
    if (nr == 4) hipLaunchKernelGGL((k_gemv_valu<bf16_t, 4>), grid, dim3(256), 0, s, g);
    else hipLaunchKernelGGL((k_gemv_valu<bf16_t, 1>), grid, dim3(256), 0, s, g);
  } else {
    if (nr == 4) hipLaunchKernelGGL((k_gemv_valu<float, 4>), grid, dim3(256), 0, s, g);
    else hipLaunchKernelGGL((k_gemv_valu<float, 1>), grid, dim3(256), 0, s, g);
  }
  return hipGetLastError();
}

hipError_t launch_argmax_finalize(const float* part_val, const int* part_idx, int ntiles, int M,
                                  int32_t* argmax, float* max_logit, hipStream_t s, const float* extra,
                                  int rem_activation, float* sig_raw, float* sig) {
  hipLaunchKernelGGL(k_argmax_finalize, dim3(M), dim3(kFinalThreads), 0, s, part_val, part_idx, ntiles, argmax,
                     max_logit, extra, rem_activation, sig_raw, sig);
  return hipGetLastError();
}

hipError_t launch_topb_finalize(const float* vals, const int* idxs, int C, int stride, int top_b, int M,
                                int32_t* cand_tok, float* cand_logit, hipStream_t s, const float* extra,
                                int rem_activation, float* sig_raw, float* sig) {
  hipLaunchKernelGGL(k_topb_finalize, dim3(M), dim3(kFinalThreads), 0, s, vals, idxs, C, stride, top_b, cand_tok,
                     cand_logit, extra, rem_activation, sig_raw, sig);
  return hipGetLastError();
}

hipError_t launch_argmax_rows(const float* logits, int M, int N, int V, int n_extra, int32_t* argmax, float* max_logit, float* extra_out,
                              float* logits_dbg, hipStream_t s, int rem_activation, float* sig_raw, float* sig) {
  hipLaunchKernelGGL(k_argmax_rows, dim3(M), dim3(kFinalThreads), 0, s, logits, N, V, n_extra, argmax, max_logit, extra_out, logits_dbg,
                     rem_activation, sig_raw, sig);
  return hipGetLastError();
}

hipError_t launch_unpack_rows(const void* src, bool bf16, int M, int K, float* act, hipStream_t s) {
  if (bf16)
    hipLaunchKernelGGL(k_unpack_rows<bf16_t>, dim3(M), dim3(256), 0, s, static_cast<const bf16_t*>(src), K, act);
  else
    hipLaunchKernelGGL(k_unpack_rows<float>, dim3(M), dim3(256), 0, s, static_cast<const float*>(src), K, act);
  return hipGetLastError();
}

}  // namespace sx
