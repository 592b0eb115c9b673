// Projections of the draft layer for the steps that the row-streaming kernel does not take (bf16 weights, up to 64 activation rows):
// out[m][n] = sum_k act[m][k] * w[n][k], as partial sums over K ranges.
//
// HBM-bound (each weight byte is used for at most 128 products) and short, 10 to 90 us, so what counts is that
// every compute unit streams from start to end.  The weights are 128-row groups x 128-k blocks of
// 32 KB; all blocks of a projection lie on one line, group after group, and workgroup w of W (one per compute
// unit) takes the blocks [w T / W, (w + 1) T / W): equal shares whatever the shape.  A share that
// crosses a group's end finishes that group's partial sums and starts the next ("segment" (w, g), partial slot
// w + g: both grow along the line, so W + groups slots are enough and a group's slots are consecutive).
// The small kernel that follows each projection anyway (norm, rotary embedding, SiLU gate) adds the slots of a
// group in their order: no atomics, no last-arriving workgroup that would add up 64 rows alone.
// Inside a workgroup as in gemm_wide.hip: two producer waves bring blocks into an LDS ring three ahead,
// consumer waves hold the activation operands of a block in registers (loaded one block ahead).
// Every workgroup takes the blocks of a segment from another starting point: rows are often a multiple of 4 KB
// apart, and in step the workgroups would all read the same L2 channels.
// Measured, the projections and the kernels behind them of one draft step, against the kernel this replaced, which
// staged the activations of every K range in LDS for each 128 rows and let the last workgroup of a group add
// up the ranges: 8B-like layer (452 MB), 8 rows 129 -> 121 us, 64 rows 355 -> 177 us; 32B-like (1080 MB), 16
// rows 247 -> 220 us.  The large ones reach 6 TB/s (gate/up of the 32B-like layer: 524 MB in 86 us); the rest is
// what starting and draining ten short kernels costs (of the five that add up 1.6 to 3.5 us each and 1.7 us to the next kernel; a
// projection about 3 us beside its stream).
#include "kernels.hpp"
#include "stream.hpp"

#include <algorithm>

namespace sx {

namespace {

constexpr int kTG = 8, kStages = 4;            // 16-row tiles per block, ring slots
constexpr int kStageBytes = kTG * 4096;

// The blocks of a workgroup's share in the order they are taken.
struct LineCursor {
  int KB, left;          // k blocks per group; blocks of the share from this segment's start on
  int g, k0, len, j, kb; // segment: group, first k block, blocks; blocks of it done; now at k block kb
  __device__ __forceinline__ LineCursor(int lo, int n, int KB_) : KB(KB_), left(n), g(lo / KB_), k0(lo % KB_) { enter(); }
  __device__ __forceinline__ void enter() {
    len = min(KB - k0, left);
    j = 0;
    kb = k0 + (static_cast<int>(blockIdx.x) >> 3) % max(len, 1);
  }
  __device__ __forceinline__ bool last_of_segment() const { return j + 1 == len; }
  __device__ __forceinline__ void next() {
    if (++j < len) {
      kb = kb + 1 == k0 + len ? k0 : kb + 1;
      return;
    }
    left -= len;
    ++g;
    k0 = 0;
    if (left > 0) enter();
  }
};

// RG groups of RT row tiles, the four k steps of a block split over KS waves; PL = 2: tiles 2 o and 2 o + 1 hold value
// and rest of the same 16 rows, whose products are added before they are stored.  The split is over k and not
// over the block's columns so that no activation piece is fetched by two waves: at 16 rows the pieces of a block
// are 8 KB, and four waves that each fetch all of them double what the compute unit takes from its L2
// (gate/up of the 32B-like layer, 16 rows: 125 us, 104 to 117 with the split over k).
template <int RG, int RT, int KS, int PL>
__global__ __launch_bounds__(64 * (RG * KS + kProducers)) void k_proj(const ProjArgs g) {
  constexpr int NC = RG * KS, JN = kTG, RO = RT / PL, S = kStages, SPW = 4 / KS;
  extern __shared__ uint4 lds4[];
  char* lds = reinterpret_cast<char*>(lds4);
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int KB = g.K >> 7;
  const int64_t T = static_cast<int64_t>(proj_groups(g.N)) * KB;
  const int lo = static_cast<int>(blockIdx.x * T / g.W);
  const int total = static_cast<int>((blockIdx.x + 1) * T / g.W) - lo;     // at least one: W <= T
  const size_t row_bytes = static_cast<size_t>(g.K) * 2;
  LineCursor cur(lo, total, KB);

  if (wv >= NC) {
    // ------------------------------------------------------------------ producer
    // piece p of a block = rows 4 (p % 4) .. + 3 of tile p / 4; lane l fetches row 4 (p % 4) + l / 16, 16-byte
    // piece (l % 16) ^ row and lands at piece base + 16 l, so that tile entry [row][pos] holds piece
    // pos ^ row: the consumers' per-row operand reads then touch 16 distinct slots
    constexpr int PP = 4 * kTG / kProducers;
    static_assert((S - 2) * PP < 64, "the load counter has six bits");
    const int pw = wv - NC;
    const char* w0 = static_cast<const char*>(g.w[0]);
    const int64_t d1 = reinterpret_cast<int64_t>(g.w[1]) - reinterpret_cast<int64_t>(g.w[0]);
    const int64_t d2 = reinterpret_cast<int64_t>(g.w[2]) - reinterpret_cast<int64_t>(g.w[1]);
    const int end0 = g.nseg > 1 ? g.seg_end[0] : g.N, end1 = g.nseg > 2 ? g.seg_end[1] : g.N;
    // the lane's offset in a tile: rows 4 (p % 4) .. of this producer's pieces, which alternate between two values
    const int r0 = 4 * pw + (lane >> 4), r1 = r0 + 8;
    const uint32_t lane_off0 = r0 * static_cast<uint32_t>(row_bytes) + (((lane & 15) ^ r0) << 4);
    const uint32_t lane_off1 = r1 * static_cast<uint32_t>(row_bytes) + (((lane & 15) ^ r1) << 4);
    static_assert(kProducers == 2, "");
    // The tiles' first rows, worked out once per group: a request is then one addition.  (Worked out per request
    // it is 40 scalar instructions, 16 times per block, which takes this wave longer than the memory takes to
    // deliver the block: gate/up of the 32B-like layer 117 us, 86 this way.)
    uint64_t tile_base[kTG];
    int have = -1;
    auto issue = [&](int slot) {
      char* stage = lds + slot * kStageBytes;
      if (cur.g != have) {
        have = cur.g;
#pragma unroll
        for (int t = 0; t < kTG; ++t) {
          const int n0 = (cur.g * kTG + t) * 16;
          // weight block of the tile (block ends are multiples of 16); sums of conditional distances, because a choice
          // between pointers makes the compiler keep them in scratch memory
          const int64_t dist = (n0 >= end0 ? d1 : 0) + (n0 >= end1 ? d2 : 0);
          const int row = n0 - (n0 >= end0 ? end0 : 0) - (n0 >= end1 ? end1 - end0 : 0);
          tile_base[t] = reinterpret_cast<uint64_t>(w0) + dist + static_cast<size_t>(row) * row_bytes;
        }
      }
      const uint64_t kb_off = static_cast<uint64_t>(cur.kb) << 8;
#pragma unroll
      for (int u = 0; u < PP; ++u) {
        const int p = pw + u * kProducers;
        load_to_lds16(reinterpret_cast<const char*>(tile_base[u / 2] + kb_off), u & 1 ? lane_off1 : lane_off0, stage + p * 1024);
      }
      cur.next();
    };
    LineCursor use = cur;                        // the block the consumers are at
    auto segment_barriers = [&]() {              // the consumers of a row group meet over a finished segment
      if (KS > 1 && use.last_of_segment()) {
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_s_barrier();
      }
    };
    int issued = 0;
    for (; issued < S - 1 && issued < total; ++issued) issue(issued % S);
    for (int i = 0; i < total; ++i) {
      // this wave's pieces of block i have landed once at most the pieces of the S-2 blocks issued
      // after it are outstanding (loads return in order); near the end simply wait for all
      if (i + S - 1 < total) __builtin_amdgcn_s_waitcnt(vmcnt_imm((S - 2) * PP));
      else __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_s_barrier();              // block i is complete; the slot of block i-1 is free
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      if (issued < total) {
        issue(issued % S);
        ++issued;
      }
      if (i > 0) {
        segment_barriers();
        use.next();
      }
    }
    segment_barriers();
    return;
  }

  // -------------------------------------------------------------------- consumer
  const int rt0 = (wv / KS) * RT, ks = wv % KS;
  const int fr = lane & 15, fq = lane >> 4;
  // operand pieces of row tile t at k block kb, k step s: two planes packed [k block][row tile][k step][lane], one in
  // place from bf16 rows [K] (with a_embed: k blocks of the first half of K from the row's embedding; rows from M on
  // repeat the last one, dropped later)
  const char* p0[RT];
  int64_t to_second[RT];          // from there to the row of the second half of K, less the first half's blocks
  constexpr int s_stride = PL == 2 ? 1024 : 64;
  constexpr size_t kb_stride = PL == 2 ? static_cast<size_t>(RG * RT) * 4096 : 256;
  const int kb_half = PL == 1 && g.a_embed ? KB >> 1 : KB;
#pragma unroll
  for (int t = 0; t < RT; ++t) {
    to_second[t] = 0;
    if constexpr (PL == 2) {
      p0[t] = static_cast<const char*>(g.a_packed) + (static_cast<size_t>(rt0 + t) * 256 + lane) * 16;
    } else {
      const int m = min(16 * (rt0 + t) + fr, g.M - 1);
      const size_t width = g.a_embed ? g.K : 2 * g.K;             // bytes of a row of a_src
      p0[t] = static_cast<const char*>(g.a_src) + m * width + fq * 16;
      if (g.a_embed) {
        const char* e = static_cast<const char*>(g.a_embed) + checked_token(g.a_tok[m], g.a_vocab, g.status) * width + fq * 16;
        to_second[t] = reinterpret_cast<int64_t>(p0[t]) - reinterpret_cast<int64_t>(e) - static_cast<int64_t>(width);
        p0[t] = e;
      }
    }
  }
  uint4 b[RT][SPW], bn[RT][SPW];
  auto fetch = [&](uint4 (&dst)[RT][SPW], int kb) {
    const bool second = PL == 1 && kb >= kb_half;                 // uniform
    const size_t off = static_cast<size_t>(kb) * kb_stride;
#pragma unroll
    for (int t = 0; t < RT; ++t) {
      const char* p = p0[t] + (second ? to_second[t] : 0) + off;
#pragma unroll
      for (int s = 0; s < SPW; ++s) dst[t][s] = *reinterpret_cast<const uint4*>(p + (ks * SPW + s) * s_stride);
    }
  };
  LineCursor nxt = cur;
  fetch(b, cur.kb);

  f32x4_t acc[RT][JN];
#pragma unroll
  for (int t = 0; t < RT; ++t)
#pragma unroll
    for (int j = 0; j < JN; ++j) acc[t][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  // read groups of CH tiles, the operand reads one group ahead of the matrix instructions; the barrier that
  // hands over the next block sits before the last group's (see gemm_wide.hip)
  constexpr int CH = JN < 4 ? JN : 4;
  constexpr int GPS = JN / CH;
  constexpr int NCH = SPW * GPS;
  uint4 wf[2][CH];
  int stage_no = 0;
  auto wait_stage = [&]() -> const uint4* {
    __builtin_amdgcn_s_waitcnt(0xC07F);            // lgkmcnt(0): this wave is done reading the block it leaves
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const uint4* stage = reinterpret_cast<const uint4*>(lds + (stage_no % S) * kStageBytes) + fr * 16;
    ++stage_no;
    return stage;
  };
  auto read_group = [&](uint4 (&dst)[CH], const uint4* stage, int c) {
    const int s = ks * SPW + c / GPS, j0 = CH * (c % GPS);
#pragma unroll
    for (int jj = 0; jj < CH; ++jj) dst[jj] = stage[(j0 + jj) * 256 + ((4 * s + fq) ^ fr)];
  };
  const uint4* stage = wait_stage();
  read_group(wf[0], stage, 0);
#pragma unroll 1
  for (int i = 0; i < total; ++i) {
    const bool more = i + 1 < total;
    // (behind the last block its own pieces once more: a request under a branch would make every wait for the
    // current pieces wait for these as well)
    if (more) nxt.next();
    fetch(bn, nxt.kb);
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      const int s = c / GPS, j0 = CH * (c % GPS);
      if (c + 1 < NCH) {
        read_group(wf[(c + 1) & 1], stage, c + 1);
      } else if (more) {
        stage = wait_stage();
        read_group(wf[0], stage, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int jj = 0; jj < CH; ++jj)
#pragma unroll
        for (int t = 0; t < RT; ++t)
          acc[t][j0 + jj] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, wf[c & 1][jj]),
                                                                    __builtin_bit_cast(bf16x8_t, b[t][s]), acc[t][j0 + jj], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
    if (cur.last_of_segment()) {
      // lane (c = lane % 16, q = lane / 16) holds weight rows 16 j + 4 q .. + 3 of the group, activation row
      // 16 (rt0 / PL + o) + c; the first wave of a row group adds the others' sums to its own, in their order
      float4* meet = reinterpret_cast<float4*>(lds + S * kStageBytes) + (wv / KS) * ((KS - 1) * RO * JN * 64) + lane;
      if constexpr (PL == 2) {
#pragma unroll
        for (int o = 0; o < RO; ++o)
#pragma unroll
          for (int j = 0; j < JN; ++j) acc[o][j] = acc[2 * o][j] + acc[2 * o + 1][j];
      }
      if constexpr (KS > 1) {
        if (ks > 0) {
#pragma unroll
          for (int o = 0; o < RO; ++o)
#pragma unroll
            for (int j = 0; j < JN; ++j) {
              const f32x4_t v = acc[o][j];
              meet[((ks - 1) * RO * JN + o * JN + j) * 64] = make_float4(v[0], v[1], v[2], v[3]);
            }
        }
        __builtin_amdgcn_s_waitcnt(0xC07F);          // lgkmcnt(0)
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        if (ks == 0) {
#pragma unroll
          for (int o = 0; o < RO; ++o)
#pragma unroll
            for (int j = 0; j < JN; ++j)
#pragma unroll
              for (int w = 0; w < KS - 1; ++w) {
                const float4 v = meet[(w * RO * JN + o * JN + j) * 64];
                acc[o][j] += f32x4_t{v.x, v.y, v.z, v.w};
              }
        }
        __builtin_amdgcn_s_waitcnt(0xC07F);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_s_barrier();                // the meeting place is free again
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      }
      if (ks == 0) {
        float* slot = g.partial + (static_cast<size_t>(blockIdx.x) + cur.g) * (static_cast<size_t>(g.M) * 128);
#pragma unroll
        for (int o = 0; o < RO; ++o) {
          const int m = 16 * (rt0 / PL + o) + fr;
          if (m < g.M) {
#pragma unroll
            for (int j = 0; j < JN; ++j) {
              const f32x4_t v = acc[o][j];
              *reinterpret_cast<float4*>(slot + m * 128 + 16 * j + 4 * fq) = make_float4(v[0], v[1], v[2], v[3]);
            }
          }
        }
      }
#pragma unroll
      for (int t = 0; t < RT; ++t)
#pragma unroll
        for (int j = 0; j < JN; ++j) acc[t][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    }
    cur = nxt;
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
      for (int s = 0; s < SPW; ++s) b[t][s] = bn[t][s];
  }
}

// ---- the kernels behind a projection

// Where the partial sums of columns n .. of row m begin, and how many slots they lie in.
struct ProjSlots {
  const float* src;
  uint32_t step;          // from one slot to the next, in floats
  int n;
};

__device__ __forceinline__ ProjSlots proj_slots(const ProjSum& p, int m, int n) {
  const int g = n >> 7, x0 = g * p.KB;
  const int w0 = proj_owner(p.T, p.inv_T, p.W, x0);
  ProjSlots r;
  r.step = static_cast<uint32_t>(p.M) * 128;
  r.src = p.partial + static_cast<size_t>(w0 + g) * r.step + m * 128 + (n & 127);
  r.n = proj_owner(p.T, p.inv_T, p.W, x0 + p.KB - 1) - w0 + 1;
  return r;
}

// Sum of the slots, in their order, of VEC columns.  The first kSlotsEarly are requested by `request` (the last one again where there are
// fewer), so that a caller has those of several sums on their way at once; more are fetched when they are added.  (One sum's eight after the
// other's, and the owners from fp64, traced / this way: D = 4096, I = 12288, 8 rows, the three norms 5.5-5.8 / 5.2 us, 64 rows 7.2-7.3 /
// 6.2-6.6 and the gate 8.2 / 7.3; D = 5120, 16 rows 6.2-6.6 / 5.1-5.7.  Kernels for two and four slots where a shape has no
// more: 353.0 us a step of 8 rows, 353.2 with one form; 64 rows 447 and 448.)
constexpr int kSlotsEarly = 8;
template <typename VEC>
struct ProjTerms {
  VEC v[kSlotsEarly];
  __device__ __forceinline__ void request(const ProjSlots& s, int off = 0) {
#pragma unroll
    for (int u = 0; u < kSlotsEarly; ++u) v[u] = *reinterpret_cast<const VEC*>(s.src + off + static_cast<size_t>(min(u, s.n - 1)) * s.step);
  }
  static __device__ __forceinline__ void add(float4& a, const float4& b) { a.x += b.x; a.y += b.y; a.z += b.z; a.w += b.w; }
  static __device__ __forceinline__ void add(float& a, const float& b) { a += b; }
  __device__ __forceinline__ VEC sum(const ProjSlots& s, int off = 0) const {
    VEC t = v[0];
#pragma unroll
    for (int u = 1; u < kSlotsEarly; ++u)
      if (u < s.n) add(t, v[u]);
    for (int i = kSlotsEarly; i < s.n; ++i) add(t, *reinterpret_cast<const VEC*>(s.src + off + static_cast<size_t>(i) * s.step));
    return t;
  }
};

// Four values of row m, columns k .. k + 3, into the packed operand order as value and rest (two planes)
__device__ __forceinline__ void pack4(char* dst, int NT, int m, int k, const float (&f)[4]) {
  uint2 hi, lo;
  hi.x = pack_bf16x2(f[0], f[1]);
  hi.y = pack_bf16x2(f[2], f[3]);
  lo.x = pack_bf16x2(f[0] - __uint_as_float(hi.x << 16), f[1] - __uint_as_float(hi.x & 0xFFFF0000u));
  lo.y = pack_bf16x2(f[2] - __uint_as_float(hi.y << 16), f[3] - __uint_as_float(hi.y & 0xFFFF0000u));
  char* p = dst + packed_byte(NT, 2 * (m >> 4), m, k);
  *reinterpret_cast<uint2*>(p) = hi;
  *reinterpret_cast<uint2*>(p + 4096) = lo;      // the next row tile
}

constexpr int kRowThreads = 1024;
constexpr int kRowIters = 2;        // float4 per thread: rows up to 8192 wide

// One workgroup per row: sums (+ residual) -> x (fp32), optionally the storage type, and the RMSNorm of the
// row as the next projection's operand.
__global__ __launch_bounds__(kRowThreads) void k_proj_norm(const ProjSum ps, int N, const float* __restrict__ residual, const bf16_t* __restrict__ gain,
                                                           float eps, float* __restrict__ out_x, bf16_t* __restrict__ out_store,
                                                           char* __restrict__ packed, int NT) {
  constexpr int NW = kRowThreads / 64;
  __shared__ float4 sh[NW / 4];
  const int m = blockIdx.x;
  float4 v[kRowIters], r[kRowIters];
  uint2 gn[kRowIters];
  ProjSlots slots[kRowIters];
  ProjTerms<float4> terms[kRowIters];
#pragma unroll
  for (int it = 0; it < kRowIters; ++it) {
    const int n = (threadIdx.x + it * kRowThreads) * 4;
    if (n < N) {
      slots[it] = proj_slots(ps, m, n);
      terms[it].request(slots[it]);
      gn[it] = *reinterpret_cast<const uint2*>(gain + n);
      r[it] = residual ? *reinterpret_cast<const float4*>(residual + static_cast<size_t>(m) * N + n) : make_float4(0.f, 0.f, 0.f, 0.f);
    }
  }
  float ssq = 0.f;
#pragma unroll
  for (int it = 0; it < kRowIters; ++it) {
    const int n = (threadIdx.x + it * kRowThreads) * 4;
    if (n < N) {
      float4 s = terms[it].sum(slots[it]);
      s.x += r[it].x; s.y += r[it].y; s.z += r[it].z; s.w += r[it].w;
      v[it] = s;
      ssq += s.x * s.x + s.y * s.y + s.z * s.z + s.w * s.w;
    }
  }
  ssq = wave_sum_halves(ssq);
  if ((threadIdx.x & 63) == 0) reinterpret_cast<float*>(sh)[threadIdx.x >> 6] = ssq;
  __syncthreads();
  float tot = 0.f;
#pragma unroll
  for (int w = 0; w < NW / 4; ++w) {
    const float4 t = sh[w];
    tot += t.x; tot += t.y; tot += t.z; tot += t.w;
  }
  const float rs = 1.0f / sqrtf(tot / static_cast<float>(N) + eps);
#pragma unroll
  for (int it = 0; it < kRowIters; ++it) {
    const int n = (threadIdx.x + it * kRowThreads) * 4;
    if (n < N) {
      const float4 s = v[it];
      const float f[4] = {s.x * rs * __uint_as_float(gn[it].x << 16), s.y * rs * __uint_as_float(gn[it].x & 0xFFFF0000u),
                          s.z * rs * __uint_as_float(gn[it].y << 16), s.w * rs * __uint_as_float(gn[it].y & 0xFFFF0000u)};
      pack4(packed, NT, m, n, f);
      if (out_x) *reinterpret_cast<float4*>(out_x + static_cast<size_t>(m) * N + n) = s;
      if (out_store)
        *reinterpret_cast<uint2*>(out_store + static_cast<size_t>(m) * N + n) = make_uint2(pack_bf16x2(s.x, s.y), pack_bf16x2(s.z, s.w));
    }
  }
}

// silu(gate) * up of the concatenated gate|up projection -> operand of the down projection
__global__ __launch_bounds__(256) void k_proj_silu(const ProjSum ps, int I, char* __restrict__ packed, int NT) {
  const int m = blockIdx.y, k = (blockIdx.x * 256 + threadIdx.x) * 4;
  if (k >= I) return;
  const ProjSlots sg = proj_slots(ps, m, k), su = proj_slots(ps, m, I + k);
  ProjTerms<float4> tg, tu;
  tg.request(sg);
  tu.request(su);
  const float4 gt = tg.sum(sg), up = tu.sum(su);
  const float f[4] = {gt.x * sigmoidf_(gt.x) * up.x, gt.y * sigmoidf_(gt.y) * up.y, gt.z * sigmoidf_(gt.z) * up.z, gt.w * sigmoidf_(gt.w) * up.w};
  pack4(packed, NT, m, k, f);
}

// q | k | v heads: rotary embedding (pairs c, c + d/2; v as it is), q rows and cache entries.  A thread takes one pair.
__global__ __launch_bounds__(256) void k_proj_rope(const ProjSum ps, const RopeArgs ra) {
  const int half = ra.d >> 1;
  const int idx = blockIdx.x * 256 + threadIdx.x;
  const int m = blockIdx.y;
  const int hh = idx / half, c = idx - hh * half;
  if (hh >= ra.Hq + 2 * ra.Hkv) return;
  // (a head of at most 128 columns lies in one group)
  const ProjSlots sl = proj_slots(ps, m, hh * ra.d + c);
  ProjTerms<float> t1, t2;
  t1.request(sl);
  t2.request(sl, half);
  const int b = m / ra.W;
  const int pos = ra.pos[b];
  const int slot = pos + (ra.node ? ra.node[m % ra.W] : 0);
  const bool turn = hh < ra.Hq + ra.Hkv;
  float cs = 1.f, sn = 0.f;
  if (turn) {
    // angle in double (long positions keep their phase), reduced to [-pi, pi] in double,
    // sine and cosine of the remainder in float
    const double ang = static_cast<double>(pos + ra.level) * ra.inv_freq[c];
    const double turns = rint(ang * 0.15915494309189535);
    const float red_ang = static_cast<float>(fma(-turns, 6.283185307179586, ang));
    sincosf(red_ang, &sn, &cs);
  }
  float x1 = t1.sum(sl), x2 = t2.sum(sl, half);
  if (turn) {
    // (written out: which of the two products a compiler fuses into the sum depends on the code around it)
    const float r1 = fmaf(x1, cs, -(x2 * sn));
    x2 = fmaf(x2, cs, x1 * sn);
    x1 = r1;
  }
  bf16_t* dst;
  if (hh < ra.Hq) {
    dst = static_cast<bf16_t*>(ra.q_out) + (static_cast<size_t>(m) * ra.Hq + hh) * ra.d;
  } else {
    if (slot < 0 || slot >= ra.l_max) return;             // an entry outside the cache is not written
    const bool is_k = hh < ra.Hq + ra.Hkv;
    const int h = is_k ? hh - ra.Hq : hh - ra.Hq - ra.Hkv;
    size_t off;
    if (ra.paged) {
      const int page = ra.page_table[static_cast<size_t>(b) * ra.max_pages + slot / ra.page_size];
      if (!page_in_pool(page, ra.n_pages, ra.status)) return;
      off = ((static_cast<size_t>(page) * ra.Hkv + h) * ra.page_size + slot % ra.page_size) * ra.d;
    } else {
      off = ((static_cast<size_t>(b) * ra.Hkv + h) * ra.l_max + slot) * ra.d;
    }
    dst = static_cast<bf16_t*>(is_k ? ra.kc : ra.vc) + off;
  }
  dst[c] = f32_to_bf16(x1);
  dst[c + half] = f32_to_bf16(x2);
}

template <int RG, int RT, int KS, int PL>
hipError_t launch_as(const ProjArgs& g, hipStream_t s) {
  // set once per process; a function-local static is initialised under the language's own lock
  static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_proj<RG, RT, KS, PL>),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
  if (attr != hipSuccess) return attr;
  hipLaunchKernelGGL((k_proj<RG, RT, KS, PL>), dim3(g.W), dim3(64 * (RG * KS + kProducers)), static_cast<size_t>(kStages) * kStageBytes + RG * (KS - 1) * (RT / PL) * kTG * 1024, s, g);
  return hipGetLastError();
}

ProjSum sum_of(const ProjArgs& g) {
  ProjSum p;
  p.partial = g.partial;
  p.KB = g.K >> 7;
  p.T = proj_groups(g.N) * p.KB;
  p.inv_T = proj_inverse(p.T);
  p.W = g.W;
  p.M = g.M;
  return p;
}

}  // namespace

bool proj_supported(int M, int N, int K) { return M >= 1 && M <= 64 && N % 128 == 0 && N >= 128 && K % 128 == 0 && K >= 128; }

// One workgroup per compute unit, each with at least two blocks while there are that many.
void proj_plan(ProjArgs& g, int num_cus) {
  const int64_t T = static_cast<int64_t>(proj_groups(g.N)) * (g.K >> 7);
  g.W = static_cast<int>(std::max<int64_t>(1, std::min<int64_t>(num_cus, T / 2)));
}

size_t proj_partial_bytes(const ProjArgs& g) { return static_cast<size_t>(g.W + proj_groups(g.N)) * g.M * 128 * sizeof(float); }

hipError_t launch_proj(const ProjArgs& g, hipStream_t s) {
  if (!proj_supported(g.M, g.N, g.K) || g.W < 1) return hipErrorInvalidValue;
  const int tiles = (g.M + 15) / 16;
  if (g.planes == 2 ? !g.a_packed : !g.a_src) return hipErrorInvalidValue;
  if (g.planes == 2) {
    switch (tiles) {
      case 1: return launch_as<1, 2, 4, 2>(g, s);
      case 2: return launch_as<2, 2, 2, 2>(g, s);
      case 3: return launch_as<3, 2, 2, 2>(g, s);
      default: return launch_as<4, 2, 1, 2>(g, s);
    }
  }
  switch (tiles) {
    case 1: return launch_as<1, 1, 4, 1>(g, s);
    case 2: return launch_as<2, 1, 2, 1>(g, s);
    default: return launch_as<4, 1, 1, 1>(g, s);
  }
}

hipError_t launch_proj_norm(const ProjArgs& g, const float* residual, const void* gain, float eps, float* out_x, void* out_store, void* packed,
                            hipStream_t s) {
  if (g.N > kRowThreads * kRowIters * 4) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_proj_norm, dim3(g.M), dim3(kRowThreads), 0, s, sum_of(g), g.N, residual, static_cast<const bf16_t*>(gain), eps, out_x,
                     static_cast<bf16_t*>(out_store), static_cast<char*>(packed), packed_tiles(g.M, 2));
  return hipGetLastError();
}

hipError_t launch_proj_silu(const ProjArgs& g, void* packed, hipStream_t s) {
  const int I = g.N / 2;
  hipLaunchKernelGGL(k_proj_silu, dim3((I / 4 + 255) / 256, g.M), dim3(256), 0, s, sum_of(g), I, static_cast<char*>(packed), packed_tiles(g.M, 2));
  return hipGetLastError();
}

hipError_t launch_proj_rope(const ProjArgs& g, const RopeArgs& ra, hipStream_t s) {
  const int items = (ra.Hq + 2 * ra.Hkv) * (ra.d >> 1);
  hipLaunchKernelGGL(k_proj_rope, dim3((items + 255) / 256, g.M), dim3(256), 0, s, sum_of(g), ra);
  return hipGetLastError();
}

}  // namespace sx
