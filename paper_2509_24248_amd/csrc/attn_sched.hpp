// Work split of the split-KV attention kernels.
//
// The context lengths live on the device, so the host cannot cut the caches into equal pieces.
// The kernels do it themselves: the keys of every (sequence, KV head) unit are counted in
// granules of 64, the units are laid end to end on one line of T granules (unit u = b * Hkv + g
// starts at Hkv * S[b] + g * n_b, S = prefix sums of the sequences' granule counts n_b), and
// workgroup w of W takes the granules [w T / W, (w + 1) T / W).  Every workgroup therefore has
// the same amount of cache to read whatever the mix of lengths, all of them are resident at
// once, and nobody waits for a long sequence's last chunk.  A workgroup whose range crosses a
// unit boundary finishes one unit's partial result and starts the next (a "segment" per unit).
// Segment (w, u) writes partial slot w + u: both grow along the line, so the slots of one unit
// are consecutive and no two segments share one; W + units slots are enough.
//
// Starting a segment costs as much as several granules (queries and first tiles from memory, nothing in flight
// meanwhile), and with equal shares the workgroups that cross a unit's end are the last to finish: 8 sequences of 2k to 16k
// entries, 8 KV heads, one query each, 512 workgroups: half of them done 44.7 us after the start, the last one 51.3.  So every
// unit has `pad` granules of nothing in front of its keys: a workgroup that starts a unit has that much less to read, and
// one whose share ends within them does not start it at all.
#pragma once
#include "common.hpp"
#include "kernels.hpp"

namespace sx {

constexpr int kAttnGran = 64;        // keys per granule
constexpr int kAttnMaxSeqs = 1024;   // sequences per launch (prefix table in LDS)

// A context length as the kernels use it: forced into 0 .. l_max - n_blk so that no access can
// leave the cache whatever the array holds.
__device__ __forceinline__ int attn_ctx_len(const AttnArgs& a, int b) {
  const int raw = a.ctx_len[b];
  const int hi = static_cast<int>(a.l_max) - a.n_blk;
  const int L = min(max(raw, 0), hi);
  if (L != raw) report_status(a.status, kStatusBadLength);
  return L;
}

// LDS words of the table below.
__host__ __device__ constexpr int attn_sched_words(int B) { return (B + 1 + (B + 3) / 4 + 3) & ~3; }

// Prefix sums S[0 .. B] of the sequences' granule counts in LDS and, behind them, a byte per sequence: how far its entries fall
// short of full granules, which with the count gives its length back.  (Whole lengths take four times that, and with
// more than 930 sequences a second workgroup of a paged launch then finds no room in the compute unit's LDS: B = 1000,
// 4 queries of 8 heads, contexts 200-500: 141 us; 111 this way, and 114 -> 80 with 64-wide heads.)
// Up to 64 sequences every wave has them in its lanes, for a workgroup's first segment: no barrier, and a lane read where the
// table is an LDS round trip (with the words for the merging kernel below, 36 calls of 1 sequence x 4096 entries, 28 rows: 449 -> 435
// us; 2 units of 600 entries, 28 rows, 12 calls 107 -> 102).  The table is written for workgroups with further segments: lanes
// that are wanted behind a segment are registers through all of it, and three waves a ring have none to spare (40 rows, paged: 45 -> 53 us).
struct AttnTable {
  int* S;
  int upto, len;             // up to 64 sequences, lane b: S[b + 1] and the entries of sequence b
};
__device__ __forceinline__ unsigned char* attn_sched_short(const AttnArgs& a, int* S) { return reinterpret_cast<unsigned char*>(S + a.B + 1); }

// Every thread of the workgroup calls this.
__device__ __forceinline__ AttnTable attn_sched_build(const AttnArgs& a, int* S) {
  const int lane = threadIdx.x & 63;
  AttnTable t;
  t.S = S;
  t.len = t.upto = 0;
  if (a.B <= 64) {
    if (lane < a.B) t.len = attn_ctx_len(a, lane) + a.n_blk;
    t.upto = wave_scan((t.len + kAttnGran - 1) / kAttnGran);
    return t;
  }
  if (threadIdx.x < 64) {
    int run = 0;
    for (int c = 0; c < a.B; c += 64) {
      const int b = c + lane;
      int x = 0;
      if (b < a.B) {
        const int n = attn_ctx_len(a, b) + a.n_blk;
        x = (n + kAttnGran - 1) / kAttnGran;
        attn_sched_short(a, S)[b] = static_cast<unsigned char>(x * kAttnGran - n);
      }
      x = wave_scan(x);
      if (b < a.B) S[b + 1] = run + x;
      run += __builtin_amdgcn_readlane(x, 63);
    }
    if (lane == 0) S[0] = 0;
  }
  __syncthreads();
  return t;
}

// For the further segments: the table of up to 64 sequences from the lanes to LDS, there behind the workgroup's next barrier.
__device__ __forceinline__ void attn_sched_keep(const AttnArgs& a, const AttnTable& t) {
  const int lane = threadIdx.x & 63;
  if (a.B > 64 || threadIdx.x >= 64) return;
  if (lane < a.B) {
    t.S[lane + 1] = t.upto;
    attn_sched_short(a, t.S)[lane] = static_cast<unsigned char>((t.len + kAttnGran - 1) / kAttnGran * kAttnGran - t.len);
  }
  if (lane == 0) t.S[0] = 0;
}

// The line of a launch whose sequences have `gran` granules in all.  Workgroups that take part: one per granule while the launch
// has a compute unit for each (no workgroup crosses a unit's end then: no padding); up to `wide_from` granules as few as
// keep the largest share at T / 256, rounded up, since that sets the time and every partial result is read again (1 sequence x 5610
// entries, 4 KV heads, 9 queries of 12 heads: 12.5 us a layer with 256 workgroups, 11.2 with 180); from there on as many as
// are resident, with at least two granules each.
// In the middle range that is a whole number of workgroups per unit where 256 allow it: sequences of one length, whose units
// are equal, then have no workgroup that crosses a unit's end.  (8 sequences x 2048 entries, 8 KV heads, 16 queries of 32 heads: 24.0
// us a layer; 28.1 with 249 workgroups of nine granules each, whose every other one starts a second segment.)  `spread` launches
// take 256 all the same: their probabilities have 8 bits, the largest of a segment none to lose, so fewer segments are less exact (4
// sequences x 600, 68 rows: error against 64 bits 2.059e-3 with the fewest workgroups, 2.044e-3 with 256, 2.039e-3 without
// padding, where unequal lengths take 5 to 20 % longer; time within 5 % of one another either way).
constexpr int kAttnSpread = 256;
constexpr int kAttnMaxGrid = 14336;       // workgroups; more are refused
struct AttnLine {
  int T, W, pad;   // granules with the padding, workgroups, padding per unit
  int q, r;        // T / W and its remainder
};
__host__ __device__ __forceinline__ float attn_sched_rcp(int x) {
#ifdef __HIP_DEVICE_COMPILE__
  return __builtin_amdgcn_rcpf(static_cast<float>(x));
#else
  return 1.0f / static_cast<float>(x);
#endif
}
// a / b, rounded down, for 0 <= a < 2^21, b >= 1: (a + 1/2) / b is at least 1 / 2b away from an integer, and the product with the
// reciprocal is off by at most 2^-22 of itself.
__host__ __device__ __forceinline__ int attn_sched_div(int a, int b) {
  return static_cast<int>((static_cast<float>(a) + 0.5f) * attn_sched_rcp(b));
}
__host__ __device__ __forceinline__ AttnLine attn_sched_line(int gran, int B, int Hkv, int pad, int wide_from, int spread, int wgrid) {
  AttnLine l;
  l.T = gran * Hkv;
  l.pad = l.T <= kAttnSpread ? 0 : pad;
  int want = l.T;
  if (l.T > kAttnSpread) {
    const bool wide = l.T >= wide_from;
    const int units = B * Hkv;
    l.T += units * pad;
    want = (l.T + 1) >> 1;
    if (!wide || want < kAttnSpread) {                                    // (T < 2^21)
      const int most = (l.T + kAttnSpread - 1) / kAttnSpread;             // the largest share
      want = spread ? kAttnSpread : units * attn_sched_div(l.T + units * most - 1, units * most);
      if (want > kAttnSpread) want = attn_sched_div(l.T + most - 1, most);
    }
  }
  l.W = want < 1 ? 1 : want < wgrid ? want : wgrid;
  l.q = l.T < 1 << 21 ? attn_sched_div(l.T, l.W) : static_cast<int>(static_cast<uint32_t>(l.T) / static_cast<uint32_t>(l.W));
  l.r = l.T - l.q * l.W;                                                  // (q is at least 1: W <= T)
  return l;
}

// First granule of workgroup w, w T / W rounded down.  (An even deal: with the first T % W workgroups one granule larger, 4 of which
// fit a unit of 67 granules evenly would have 68.  The products of the formula need 64 bits, whose division is 150 dependent
// instructions, fetched for a single use; w r is less than kAttnMaxGrid squared, the quotient from floats off by one at most before the comparisons.)
__host__ __device__ __forceinline__ int attn_sched_lo(const AttnLine& l, int w) {
  const int x = w * l.r;
  int k = attn_sched_div(x, l.W);
  if (k * l.W > x) --k;
  if ((k + 1) * l.W <= x) ++k;
  return w * l.q + k;
}

// The line of a launch on the device.
__device__ __forceinline__ AttnLine attn_sched_line(const AttnArgs& a, const AttnTable& t) {
  const int gran = a.B <= 64 ? __builtin_amdgcn_readlane(t.upto, 63) : __builtin_amdgcn_readfirstlane(t.S[a.B]);
  return attn_sched_line(gran, a.B, a.Hkv, a.pad, a.wide_from, a.use_mfma == kOnePart, a.wgrid);
}

struct AttnSeg {
  int b, g;      // unit
  int s0, s1;    // keys [s0, s1) of the unit, none if s1 <= s0
  int L;         // context length of the sequence (block entries follow)
  int next;      // granule on the line where the next segment starts
};

__host__ __device__ __forceinline__ int attn_sched_uniform(int x) {
#ifdef __HIP_DEVICE_COMPILE__
  return __builtin_amdgcn_readfirstlane(x);
#else
  return x;
#endif
}

// The segment that starts at granule x of the line, which is one of sequence b's (`first` granules in front of the sequence, n of it
// in each of its Hkv units, L entries in front of n_blk of the block), and ends at the unit's end or at `hi`; no keys where that is
// still padding.
__host__ __device__ __forceinline__ AttnSeg attn_sched_cut(int Hkv, int n_blk, int pad, int b, int first, int n, int L, int x, int hi) {
  AttnSeg s;
  s.b = b;
  s.L = L;
  const int rel = x - Hkv * (first + pad * b);
  const int g = rel < 1 << 21 ? attn_sched_div(rel, n + pad) : static_cast<int>(static_cast<uint32_t>(rel) / static_cast<uint32_t>(n + pad));
  s.g = min(attn_sched_uniform(g), Hkv - 1);
  const int at = min(rel - s.g * (n + pad), n + pad - 1);   // granule of the unit, padding first
  const int end = min(at + (hi - x), n + pad);
  s.s0 = max(at - pad, 0) * kAttnGran;
  s.s1 = min(L + n_blk, (end - pad) * kAttnGran);
  s.next = x + max(end - at, 1);                // (the minima above cannot bind while the table is that of these lengths)
  return s;
}

// The segment from granule x on, on the device.  Uniform over the workgroup.  `lanes`: the table in the lanes will do (see AttnTable).
__device__ __forceinline__ AttnSeg attn_sched_segment(const AttnArgs& a, const AttnTable& t, bool lanes, int pad, int x, int hi) {
  const int lane = threadIdx.x & 63;
  int b = 0, first, n, L;
  if (lanes && a.B <= 64) {
    b = min(static_cast<int>(__popcll(__builtin_amdgcn_ballot_w64(lane < a.B && a.Hkv * (t.upto + pad * (lane + 1)) <= x))), a.B - 1);
    first = b > 0 ? __builtin_amdgcn_readlane(t.upto, b - 1) : 0;
    n = __builtin_amdgcn_readlane(t.upto, b) - first;
    L = __builtin_amdgcn_readlane(t.len, b) - a.n_blk;
  } else {
    for (int c = 0; c < a.B; c += 64) {
      const int i = c + lane;
      const bool before = i < a.B && a.Hkv * (t.S[i + 1] + pad * (i + 1)) <= x;
      b += static_cast<int>(__popcll(__builtin_amdgcn_ballot_w64(before)));
    }
    b = __builtin_amdgcn_readfirstlane(min(b, a.B - 1));
    first = __builtin_amdgcn_readfirstlane(t.S[b]);
    n = __builtin_amdgcn_readfirstlane(t.S[b + 1]) - first;
    L = __builtin_amdgcn_readfirstlane(n * kAttnGran - attn_sched_short(a, t.S)[b] - a.n_blk);
  }
  return attn_sched_cut(a.Hkv, a.n_blk, pad, b, first, n, L, x, hi);
}

// The first segment with keys from granule x of a workgroup's share on; s1 <= s0 if there is none.
__device__ __forceinline__ AttnSeg attn_sched_next(const AttnArgs& a, const AttnTable& t, bool lanes, int pad, int x, int hi) {
  AttnSeg s;
  s.s0 = s.s1 = 0;
  while (x < hi) {
    s = attn_sched_segment(a, t, lanes, pad, x, hi);
    if (s.s1 > s.s0) break;
    x = s.next;
  }
  return s;
}

// The workgroups that have a unit's first and last keys, for the merging kernel: [unit][2].  (From prefix sums and the line that kernel
// worked the two out again, a chain of divisions in front of its first request: 36 calls as above 442 us, 435 this way.)
__device__ __forceinline__ void attn_sched_publish(const AttnArgs& a, const AttnSeg& s) {
  if (threadIdx.x == 0) {
    int* p = a.sched + 2 * (s.b * a.Hkv + s.g);
    if (s.s0 == 0) p[0] = blockIdx.x;
    if (s.s1 == s.L + a.n_blk) p[1] = blockIdx.x;
  }
}

}  // namespace sx
