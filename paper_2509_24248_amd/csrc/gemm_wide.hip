// The two heads in bf16: widened head of the draft (Eq. 1; fp32 rows under an RMSNorm as two bf16 planes) and LM
// head over the verification block (Alg. 1), GEMM + argmax or ranked candidates, logits never stored.
//
// A pure weight stream with up to 160 activation rows beside it:
//   - one workgroup per compute unit walks an equal share of the weight tiles (16 rows each),
//     whatever the vocabulary size: no rounds of workgroups, no refill of the pipeline between them;
//   - the WEIGHTS pass through an LDS ring of S stages, one 128-k block of TG tiles per stage.  Two
//     producer waves do nothing but bring stages in with direct global->LDS loads (16 bytes per
//     lane, streaming), S-1 stages ahead; their load counters hold nothing else, so three stages
//     stay in flight across the barriers;
//   - the ACTIVATIONS stay in registers: a consumer wave owns RT 16-row tiles of the rows and
//     loads their operand pieces of the next k block (L2 hits) while it works on this one, from a
//     copy of the activations in operand order (k_pack_act, k_pack_norm) so that a load covers whole cache
//     lines; up to 32 plain bf16 rows are read in place;
//   - a pass takes 2 to 5 times TG tiles through all k blocks, the "halves" of a k block one after the other,
//     so the activation pieces of a k block are fetched once for 256 to 640 weight rows; one LDS read (the
//     transposed weight operand) feeds RT matrix instructions.
// One workgroup barrier per stage hands a landed stage to the consumers and the stage read
// before it back to the producers.  Every lane keeps the best of the logits it has seen; they become one
// candidate per workgroup and row (and column split) at the end.
// What bounds it: the weight stream.  V = 151936, D = 4096, whole call: 8 / 24 / 56 / 144 rows 188 / 196 / 207 /
// 230 us = 6.6 / 6.4 / 6.0 / 5.4 TB/s (one call after the other; 2 % less with single calls), where a kernel that staged
// the activations in LDS for every eight weight tiles took 230 / 233 us for the first two and the same form with one wave
// per 32 rows 225 us for the third.  Draft head with 8 / 64 fp32 rows, same size: 230 -> 183 and 503 -> 216 us (that kernel
// read all 128 virtual rows from LDS for every tile: the LDS was the bound); 64 rows 210 us with value and rest in one accumulator.  Many rows are slower: by leaving parts out
// at 144 rows (D = 5120), the producers alone stream at 7 TB/s (230 us), the consumers alone take 225 us, of
// that the LDS reads and barriers 45 us, the matrix instructions 45 us, the activation loads 25 us (80 us
// before they covered whole cache lines: straight from the row-major matrix a load is 16 rows x 64 bytes,
// and those half-line requests, not their bytes, were the cost).
#include "../../include/specexit.h"
#include "kernels.hpp"
#include "stream.hpp"

#include <limits.h>

#include <algorithm>

namespace sx {

namespace {

// The order in which a workgroup takes the k blocks of a pass.  The workgroups run in step, and where the
// weight rows are a multiple of 4 KB apart the reads of one k block by all of them fall on one of the
// sixteen 256-byte-interleaved channels of each L2 (8 rows, D = 2048: V = 128259 in 112 us, 83 us with four
// starting points, 81 with eight; D = 4096: V = 32000 in 58, 44, 44 us, V = 151936 in 193, 190, 199).  So K is cut into 2^LV chunks, and workgroup w takes them in the
// order i ^ s, s from w.  Identical weight rows must give identical bits in whichever workgroup they are (ties
// go to the lowest index): every chunk is summed on its own, and the chunks are added as a balanced binary
// tree, in which the order i ^ s only exchanges the two operands of an addition.
template <int LV>
struct KOrder {
  static constexpr int P = 1 << LV;
  int KB, s, lv, ci, kb, hi;    // ci: position in the order; chunk ci ^ s = k blocks .. hi - 1, now at kb
  __device__ __forceinline__ explicit KOrder(int KB_) : KB(KB_) {
    lv = KB >= P ? LV : 0;      // (fewer k blocks than chunks: one chunk)
    s = lv ? (static_cast<int>(blockIdx.x) >> 3) & (P - 1) : 0;    // neighbours on one XCD are eight apart
    ci = 0;
    enter();
  }
  __device__ __forceinline__ void enter() {
    kb = ((ci ^ s) * KB) >> lv;
    hi = (((ci ^ s) + 1) * KB) >> lv;
  }
  __device__ __forceinline__ bool last_of_chunk() const { return kb + 1 == hi; }
  // after the last k block of a pass comes the first of the next one
  __device__ __forceinline__ void next() {
    if (++kb < hi) return;
    ci = ci + 1 == (1 << lv) ? 0 : ci + 1;
    enter();
  }
};

// The workgroup's tiles [t_lo, t_hi) in equal "halves" of at most TG tiles (equal: 17 tiles as 8 + 8 + 1 would
// take the last one through all k blocks at one tile per stage, too little in flight to fill the latency).
struct Halves {
  int t_lo, n, count, most;     // tiles, halves, tiles of the largest half
  __device__ __forceinline__ Halves(int lo, int hi, int TG) : t_lo(lo), n(hi - lo), count((hi - lo + TG - 1) / TG) {
    most = (n + count - 1) / count;
  }
  __device__ __forceinline__ int first(int h) const { return t_lo + n * h / count; }
};

// A pass takes up to MAXH halves through all k blocks; the passes of a workgroup are as equal as they can be, the first ones
// larger.  Number of halves of the pass that starts with half0 still to take `left` of them.
template <int MAXH>
__device__ __forceinline__ int pass_halves(int left) {
  const int passes = (left + MAXH - 1) / MAXH;
  return passes > 0 ? (left + passes - 1) / passes : 0;
}

// The stages of a workgroup in the order they pass through the ring: the halves of a k block one after the other, so that
// the consumers fetch their activation pieces of a k block once for all halves of the pass.
template <int MAXH, int LV>
struct StageCursor {
  int half0, nh, h, n;   // first half and number of halves of the current pass; half within the pass; k blocks done
  KOrder<LV> k;
  __device__ __forceinline__ StageCursor(int nhalf, int KB) : half0(0), nh(pass_halves<MAXH>(nhalf)), h(0), n(0), k(KB) {}
  __device__ __forceinline__ void advance(int nhalf, int KB) {
    if (++h < nh) return;
    h = 0;
    k.next();
    if (++n < KB) return;
    n = 0;
    half0 += nh;
    nh = pass_halves<MAXH>(nhalf - half0);
  }
};

// The TB best (value, index) pairs a lane has seen, best first.  Values arrive with growing indices, so
// a strict comparison keeps the lowest index among equals in front; a value that is not above
// the initial -inf is never taken (index INT_MAX: empty).
template <int TB>
struct Best {
  float v[TB];
  int i[TB];
  __device__ __forceinline__ void clear() {
#pragma unroll
    for (int r = 0; r < TB; ++r) { v[r] = -INFINITY; i[r] = INT_MAX; }
  }
  __device__ __forceinline__ void add(float x, int n) {
#pragma unroll
    for (int r = TB - 1; r >= 0; --r) {
      const bool here = x > v[r];
      if (r > 0) {
        const bool above = x > v[r - 1];
        v[r] = here ? (above ? v[r - 1] : x) : v[r];
        i[r] = here ? (above ? i[r - 1] : n) : i[r];
      } else {
        v[0] = here ? x : v[0];
        i[0] = here ? n : i[0];
      }
    }
  }
  // first entry out
  __device__ __forceinline__ void pop() {
#pragma unroll
    for (int r = 0; r + 1 < TB; ++r) { v[r] = v[r + 1]; i[r] = i[r + 1]; }
    v[TB - 1] = -INFINITY;
    i[TB - 1] = INT_MAX;
  }
};

// The consumer side of k_head_wide for a wave that owns RT row tiles of the operand (from tile rt0 on) and, of
// every half, the JN weight tiles from jc0 on: one barrier per stage, a candidate update per pass.
// PL = 2: tiles 2 o and 2 o + 1 are the bf16 value and the bf16 rounding of the rest of the same 16
// activation rows.  Their products are added at the end where both have accumulators for the whole pass (up to 16 rows:
// LV = 2); with more rows they add up in one, a k block at a time (kBlockSums).  Every lane keeps the TB best of what it has seen;
// they are merged over the four lanes of a row when the workgroup's share is done.
// A row has `slots` candidate slots per workgroup, one per column split; a wave that covers the whole half
// (JN = TG) where others split it fills the remaining one with nothing.
template <int RT, int JN, int TG, int S, int PL, int TB, int MAXH, int LV>
struct Consumer {
  static constexpr int kStage = TG * 4096;
  static constexpr int RO = RT / PL;        // 16-row tiles of results
  // Value and rest of a draft row in one accumulator leave registers for passes of more halves, but in a sum over all of K every
  // product of the rest is then rounded at the size of the value's sum, 256 roundings instead of 128 at D = 4096.  So the products of a k
  // block are summed by themselves and added to the pass's accumulators: 32 roundings at that size.  Error of the ranked logits, D =
  // 4096, 17 / 40 / 64 rows, against 64-bit sums of the same parts: 3.8e-7 / 3.8e-7 / 3.9e-7 with an accumulator each,
  // 5.0e-7 / 5.2e-7 / 5.0e-7 with one, 2.1e-7 / 2.2e-7 / 2.3e-7 this way, in the same time (draft steps of 20 / 48 / 64 rows,
  // V = 151936: 326 / 354 / 382 us with one accumulator, 326 / 355 / 380 this way).
  static constexpr bool kBlockSums = PL == 2 && LV < 2;
  static constexpr int RA = kBlockSums ? RO : RT;
  const GemmArgs& g;
  char* lds;
  int rt0, jc0, fr, fq, KB;
  Halves halves;
  KOrder<LV> k;             // at the k block whose pieces `b` holds
  const uint4* apack[RT];   // this lane's piece of row tile t, k block 0, k step 0
  size_t kb_stride;         // uint4 entries from one k block to the next
  int s_stride;             // and from one k step to the next
  uint4 bn[RT][2];  // pieces 0 and 1 of the next k block, on their way
  uint4 b[RT][4];   // activation operand pieces of the current k block: row 16 tile + fr, k = 32 s + 8 fq .. + 7
  int stage_no;     // stages consumed so far: stage i lives in ring slot i % S
  Best<TB> best[RO];

  __device__ __forceinline__ Consumer(const GemmArgs& g_, char* lds_, int rt0_, int jc0_, int NT, int lane, const Halves& halves_, int KB_)
      : g(g_), lds(lds_), rt0(rt0_), jc0(jc0_), fr(lane & 15), fq(lane >> 4), KB(KB_), halves(halves_), k(KB_), stage_no(0) {
    if (g.a_packed) {
      // packed activations: [k block][row tile][k step][lane] 16-byte pieces (NT row tiles), so that one
      // load instruction of a wave reads 1 KB of consecutive bytes
      kb_stride = static_cast<size_t>(NT) * 256;
      s_stride = 64;
#pragma unroll
      for (int t = 0; t < RT; ++t) apack[t] = static_cast<const uint4*>(g.a_packed) + static_cast<size_t>(rt0 + t) * 256 + lane;
    } else {
      // straight from the row-major bf16 matrix (few rows); rows from M on repeat the last one, dropped later
      kb_stride = 16;
      s_stride = 4;
#pragma unroll
      for (int t = 0; t < RT; ++t)
        apack[t] = static_cast<const uint4*>(g.a_src) + static_cast<size_t>(min(16 * (rt0 + t) + fr, g.M - 1)) * (g.K >> 3) + fq;
    }
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
      for (int s = 0; s < 4; ++s) b[t][s] = apack[t][k.kb * kb_stride + s * s_stride];
#pragma unroll
    for (int o = 0; o < RO; ++o) best[o].clear();
  }

  // one pass: NH halves starting at half `half0`
  template <int NH>
  __device__ __forceinline__ void pass(int half0) {
    f32x4_t acc[RA][NH * JN];
#pragma unroll
    for (int o = 0; o < RA; ++o)
#pragma unroll
      for (int j = 0; j < NH * JN; ++j) acc[o][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};

    f32x4_t left[LV > 0 ? LV : 1][RA][NH * JN];     // finished left siblings of the chunk tree, per level

    // The waves go through a stage's four k steps in read groups of CH tiles, the operand reads one
    // group ahead of the matrix instructions (k steps outermost: between two matrix instructions on the
    // same accumulator lie those of all other tiles; with block sums the tiles of a group outermost, so that one group's
    // sums are under way at a time; the scheduler is kept from sinking the reads back
    // to their uses).  The barrier that hands over the next stage sits before the last group's matrix
    // instructions, whose operands are in registers by then: the first reads of the next stage are in
    // flight while those instructions run, so neither the LDS nor the matrix cores idle around a barrier.
    constexpr int CH = JN < 4 ? JN : 4;   // tiles per read group
    constexpr int GPS = JN / CH;          // read groups per k step
    constexpr int NCH = 4 * GPS;          // read groups per stage
    const auto step_of = [](int c) { return kBlockSums ? c & 3 : c / GPS; };             // k step and first tile of group c
    const auto tile_of = [](int c) { return CH * (kBlockSums ? c >> 2 : c % GPS); };
    uint4 wf[2][CH];
    f32x4_t blk[RO][CH];
    auto wait_stage = [&]() -> const uint4* {
      __builtin_amdgcn_s_waitcnt(0xC07F);            // lgkmcnt(0): this wave is done reading the stage it leaves
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_s_barrier();                  // the next stage has landed; the one just read is free
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      const uint4* stage = reinterpret_cast<const uint4*>(lds + (stage_no % S) * kStage) + fr * 16;
      ++stage_no;
      return stage;
    };
    auto read_group = [&](uint4 (&dst)[CH], const uint4* stage, int c) {
      const int s = step_of(c), j0 = tile_of(c);
#pragma unroll
      for (int jj = 0; jj < CH; ++jj) dst[jj] = stage[(jc0 + j0 + jj) * 256 + ((4 * s + fq) ^ fr)];
    };
    const uint4* stage = wait_stage();
    read_group(wf[0], stage, 0);
#pragma unroll 1
    for (int kb = 0; kb < KB; ++kb) {
      // the pieces of the next k block (after the last one that is where the next pass starts)
      const int ci = k.ci;
      const bool chunk_end = LV > 0 && k.lv > 0 && k.last_of_chunk();
      k.next();
      const size_t noff = static_cast<size_t>(k.kb) * kb_stride;
#pragma unroll
      for (int h = 0; h < NH; ++h) {
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
          const int s = step_of(c), j0 = tile_of(c);
          if (c + 1 < NCH) {
            read_group(wf[(c + 1) & 1], stage, c + 1);
          } else if (h < NH - 1 || kb + 1 < KB) {
            stage = wait_stage();
            read_group(wf[0], stage, 0);
          }
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int i = 0; i < RT * CH; ++i) {
            // (block sums: the instructions on one accumulator lie CH apart)
            const int t = kBlockSums ? i / CH : i % RT, jj = kBlockSums ? i % CH : i / RT;
            f32x4_t& to = kBlockSums ? blk[t / PL][jj] : acc[t][h * JN + j0 + jj];
            const f32x4_t from = kBlockSums && s == 0 && t % PL == 0 ? f32x4_t{0.f, 0.f, 0.f, 0.f} : to;
            to = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, wf[c & 1][jj]), __builtin_bit_cast(bf16x8_t, b[t][s]), from, 0, 0, 0);
          }
          // The next k block's activation pieces (1 KB of consecutive bytes per instruction, L2 hits that
          // take more than a microsecond under the weight stream).  Pieces 0 and 1, which the next block
          // needs first, are requested into spare registers at the start of this block and moved over when
          // the last half is done with the old ones; pieces 2 and 3 are requested into their own place as
          // soon as the last half is done with them.
          if (h == 0 && c == 0) {
#pragma unroll
            for (int t = 0; t < RT; ++t) {
              bn[t][0] = apack[t][noff];
              bn[t][1] = apack[t][noff + s_stride];
            }
          }
          if constexpr (kBlockSums) {
            if (s == 3) {
#pragma unroll
              for (int o = 0; o < RO; ++o)
#pragma unroll
                for (int jj = 0; jj < CH; ++jj) {
                  f32x4_t& sum = acc[o][h * JN + j0 + jj];
                  sum += blk[o][jj];
                  asm volatile("" : "+v"(sum));    // (here: put off to the k block's end, the sums of all halves are live)
                }
            }
          }
          if (h == NH - 1 && (kBlockSums ? c >= NCH - 4 : (c + 1) % GPS == 0)) {
#pragma unroll
            for (int t = 0; t < RT; ++t) {
              if (s < 2) b[t][s] = bn[t][s];
              else b[t][s] = apack[t][noff + s * s_stride];
            }
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      // a chunk is summed: up the tree as far as its right siblings go
      if constexpr (LV > 0) {
        if (chunk_end) {
          bool up = true;
#pragma unroll
          for (int l = 0; l < LV; ++l) {
            if (!up) continue;
            if (ci >> l & 1) {
#pragma unroll
              for (int o = 0; o < RA; ++o)
#pragma unroll
                for (int j = 0; j < NH * JN; ++j) acc[o][j] += left[l][o][j];
            } else {
              up = false;
#pragma unroll
              for (int o = 0; o < RA; ++o)
#pragma unroll
                for (int j = 0; j < NH * JN; ++j) { left[l][o][j] = acc[o][j]; acc[o][j] = f32x4_t{0.f, 0.f, 0.f, 0.f}; }
            }
          }
        }
      }
    }

    // ---- epilogue: lane (c = lane % 16, q = lane / 16) holds weight rows 16 (tile0 + j) + 4 q + i of
    // activation row 16 (rt0 / PL + o) + c; rows below V enter the lane's best, the rows V.. are the
    // widened head's extra rows.
    if constexpr (RA > RO) {
      static_assert(RO == 1 || RA == RO, "value and rest of one row tile");
#pragma unroll
      for (int j = 0; j < NH * JN; ++j) acc[0][j] += acc[1][j];
    }
    int fr_e = fr, fq_e = fq;     // (what follows from them is worked out here and not held through the loop above)
    asm volatile("" : "+v"(fr_e), "+v"(fq_e));
#pragma unroll
    for (int h = 0; h < NH; ++h) {
      const int tile0 = halves.first(half0 + h) + jc0;      // this wave's first tile of the half
      const int tile1 = halves.first(half0 + h + 1);        // (the stage repeats the half's last tile from here on)
#pragma unroll
      for (int o = 0; o < RO; ++o) {
        const int m = 16 * (rt0 / PL + o) + fr_e;
        const bool owner = m < g.M;
        // tiles that lie wholly below the signal rows (all but the last of a launch) need no checks per
        // element: the consumers stand still during the epilogue while the ring fills up, so its length counts
        const bool plain = !g.logits_dbg && (tile0 + JN) * 16 <= g.V;    // uniform
        const int nb = tile0 * 16 + 4 * fq_e;
        if constexpr (TB > 1) {
          // ranked candidates: the values pass through a corner of the LDS (this lane's own 16 bytes per tile), so
          // that the insertion exists once, in a loop.  Unrolled over the accumulators it is several KB of code
          // that arrives line by line behind the weight stream (16 rows, V = 151936, D = 4096: 213 us; 187 without
          // ranked candidates).
          float4* mine = reinterpret_cast<float4*>(lds + S * kStage) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) * (JN * 64) + 16 * fq_e + fr_e;
#pragma unroll
          for (int j = 0; j < JN; ++j) {
            const f32x4_t v = acc[o][h * JN + j];
            mine[j * 64] = make_float4(v[0], v[1], v[2], v[3]);
          }
          const int left_j = min(JN, tile1 - tile0);
#pragma unroll 1
          for (int x = 0; x < 4 * left_j; ++x) {
            const float val = reinterpret_cast<const float*>(mine + (x >> 2) * 64)[x & 3];
            const int n = nb + 16 * (x >> 2) + (x & 3);
            if (n < g.V) best[o].add(val, n);
            else if (owner && n < g.N && g.extra_out) g.extra_out[m * g.n_extra + (n - g.V)] = val;
          }
        } else if (plain) {
#pragma unroll
          for (int j = 0; j < JN; ++j) {
            const bool inside = tile0 + j < tile1;           // uniform
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const float val = acc[o][h * JN + j][i];
              best[o].add(inside ? val : -INFINITY, nb + 16 * j + i);    // n grows with h, j and i
            }
          }
        } else {
#pragma unroll
          for (int j = 0; j < JN; ++j) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const int n = nb + 16 * j + i;
              const float val = acc[o][h * JN + j][i];
              if (owner && tile0 + j < tile1 && n < g.N) {
                if (n < g.V) {
                  if (g.logits_dbg) g.logits_dbg[static_cast<size_t>(m) * g.V + n] = val;
                  best[o].add(val, n);
                } else if (g.extra_out) {
                  g.extra_out[m * g.n_extra + (n - g.V)] = val;
                }
              }
            }
          }
        }
      }
    }
  }

  __device__ __forceinline__ void run() {
#pragma unroll 1
    for (int half0 = 0; half0 < halves.count;) {
      const int nh = pass_halves<MAXH>(halves.count - half0);
      if (MAXH >= 5 && nh == 5) pass<MAXH >= 5 ? 5 : 1>(half0);
      else if (MAXH >= 4 && nh == 4) pass<MAXH >= 4 ? 4 : 1>(half0);
      else if (MAXH >= 3 && nh == 3) pass<MAXH >= 3 ? 3 : 1>(half0);
      else if (nh == 2) pass<2>(half0);
      else pass<1>(half0);
      half0 += nh;
    }
    // the row's best over its four lanes, one candidate (list) per workgroup and column split
    const int slots = g.wide_slots;
    const int top_b = TB > 1 ? g.top_b : 1;
    int fr_e = fr;                // (likewise)
    asm volatile("" : "+v"(fr_e));
#pragma unroll
    for (int o = 0; o < RO; ++o) {
      const int m = 16 * (rt0 / PL + o) + fr_e;
      const size_t at = (static_cast<size_t>(m) * gridDim.x + blockIdx.x) * slots * top_b;
      const int mine = jc0 / JN;
#pragma unroll 1
      for (int r = 0; r < top_b; ++r) {
        float bv = best[o].v[0];
        int bi = best[o].i[0];
#pragma unroll
        for (int x = 16; x < 64; x <<= 1) {
          const float ov = __shfl_xor(bv, x, 64);
          const int oi = __shfl_xor(bi, x, 64);
          if (better(ov, oi, bv, bi)) { bv = ov; bi = oi; }
        }
        if (best[o].i[0] == bi) best[o].pop();               // (an index belongs to one lane; popping an empty list changes nothing)
        if (m < g.M && fq == 0) {
          g.part_val[at + mine * top_b + r] = bv;
          g.part_idx[at + mine * top_b + r] = bi;
          if (JN == TG && slots == 2) {
            g.part_val[at + top_b + r] = -INFINITY;
            g.part_idx[at + top_b + r] = INT_MAX;
          }
        }
      }
    }
  }
};

// Activations [M, K] bf16 -> operand pieces [k block][row tile][k step][lane]: lane (c = lane % 16,
// q = lane / 16) of piece (kb, tile, s) holds row 16 tile + c, k = 128 kb + 32 s + 8 q .. + 7; rows
// from M on are zero.  The consumers of k_head_wide then fetch a k block's pieces with loads that
// cover whole cache lines: read straight from the row-major matrix, the same pieces are 16 rows x
// 64 bytes per instruction, and those half-line requests, not their bytes, were what the
// activations cost (144 rows: 80 us of 395 with them, 29 us with full-line loads of the same bytes).
__global__ __launch_bounds__(256) void k_pack_act(const bf16_t* __restrict__ src, uint4* __restrict__ dst, int M, int K, int NT) {
  const int lane = threadIdx.x & 63;
  const int unit = blockIdx.x * 4 + (threadIdx.x >> 6);     // (kb, tile)
  const int KB = K >> 7;
  if (unit >= KB * NT) return;
  const int kb = unit / NT, tile = unit - kb * NT;
  const int m = 16 * tile + (lane & 15);
  const bf16_t* row = src + static_cast<size_t>(m < M ? m : 0) * K + 128 * kb + 8 * (lane >> 4);
  uint4 v[4];
#pragma unroll
  for (int s = 0; s < 4; ++s) v[s] = *reinterpret_cast<const uint4*>(row + 32 * s);
#pragma unroll
  for (int s = 0; s < 4; ++s) dst[(static_cast<size_t>(unit) * 4 + s) * 64 + lane] = m < M ? v[s] : uint4{0u, 0u, 0u, 0u};
}

// The same for fp32 rows under an RMSNorm, x rsqrt(mean x^2 + eps) gain, split into two bf16 planes: row tile
// 2 o holds the bf16 rounding of rows 16 o .. + 15, row tile 2 o + 1 the bf16 rounding of what that lost.
__global__ __launch_bounds__(256) void k_pack_norm(const float* __restrict__ src, const float* __restrict__ ssq, int nssq,
                                                   const bf16_t* __restrict__ gain, float eps, uint4* __restrict__ dst, int M, int K, int NO) {
  const int lane = threadIdx.x & 63;
  const int unit = blockIdx.x * 4 + (threadIdx.x >> 6);     // (kb, rows 16 o ..)
  const int KB = K >> 7;
  if (unit >= KB * NO) return;
  const int kb = unit / NO, o = unit - kb * NO;
  const int m = 16 * o + (lane & 15), q = lane >> 4;
  const int row = m < M ? m : 0;
  const float* p = src + static_cast<size_t>(row) * K + 128 * kb + 8 * q;
  const bf16_t* gp = gain + 128 * kb + 8 * q;
  float4 x[4][2];
  uint4 gn[4];
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    x[s][0] = *reinterpret_cast<const float4*>(p + 32 * s);
    x[s][1] = *reinterpret_cast<const float4*>(p + 32 * s + 4);
    gn[s] = *reinterpret_cast<const uint4*>(gp + 32 * s);
  }
  float t = 0.f;
  for (int j = q; j < nssq; j += 4) t += ssq[row * nssq + j];
  t += __shfl_xor(t, 16, 64);
  t += __shfl_xor(t, 32, 64);
  const float rs = 1.0f / sqrtf(t / static_cast<float>(K) + eps);
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    float f[8] = {x[s][0].x, x[s][0].y, x[s][0].z, x[s][0].w, x[s][1].x, x[s][1].y, x[s][1].z, x[s][1].w}, gf[8], hf[8];
    unpack16(gn[s], gf);
#pragma unroll
    for (int e = 0; e < 8; ++e) f[e] = m < M ? f[e] * rs * gf[e] : 0.f;
    const uint4 hi = make_uint4(pack_bf16x2(f[0], f[1]), pack_bf16x2(f[2], f[3]), pack_bf16x2(f[4], f[5]), pack_bf16x2(f[6], f[7]));
    unpack16(hi, hf);
    const uint4 lo = make_uint4(pack_bf16x2(f[0] - hf[0], f[1] - hf[1]), pack_bf16x2(f[2] - hf[2], f[3] - hf[3]),
                                pack_bf16x2(f[4] - hf[4], f[5] - hf[5]), pack_bf16x2(f[6] - hf[6], f[7] - hf[7]));
    uint4* d = dst + static_cast<size_t>(kb * 2 * NO + 2 * o) * 256 + s * 64 + lane;
    d[0] = hi;
    d[256] = lo;
  }
}

// s_waitcnt vmcnt(PER * n) for n = 1 .. N (the count is part of the instruction)
template <int N, int PER>
__device__ __forceinline__ void wait_tiles(int n) {
  if constexpr (N > 1) {
    if (n < N) { wait_tiles<N - 1, PER>(n); return; }
  }
  __builtin_amdgcn_s_waitcnt(vmcnt_imm(PER * N));
}

// Halves per pass: as many as the accumulators have registers for, because every pass fetches all activations again, through the
// same path as the weights (V = 151936, D = 5120, 64 rows: 242 us, 227 with the fetches left out; 144 rows 281 and 241).  A
// workgroup has five halves of that vocabulary.  Draft step, D = 4096, with two halves / three / five: 20 rows 337 / 330 / 326 us, 48
// rows 366 / 359 / 353 (two row tiles of value and rest, half of the columns each); 64 rows 379 / 372 / - (all columns); LM
// head of 64 rows, D = 4096 / 5120: 198 / 243 -> 192 / 237.  More than 64 rows: three row tiles per wave, with three
// consumer waves of 512 registers and passes of 20 tiles, are slower (144 rows 281 -> 310).
constexpr int max_halves(int RT, int CS, int PL, int LV) {
  if (LV > 0 || RT != 2) return 2;
  return PL == 2 ? (CS == 2 ? 5 : 3) : CS == 2 ? 3 : 2;
}

// RG groups of RT row tiles, each group's columns split over CS waves; then the producers.  SPLIT (CS = 1): the
// last group's second row tile does not exist (an odd number of row tiles), and its one tile is shared with
// a further wave after the producers, each taking half of the columns: no SIMD then carries three row
// tiles' worth of matrix instructions.
template <int RG, int RT, int CS, int PL, int TB, int TG, int S, bool SPLIT, int LV>
__global__ __launch_bounds__(64 * (RG * CS + kProducers + (SPLIT ? 1 : 0))) void k_head_wide(const GemmArgs g) {
  constexpr int NC = RG * CS, MAXH = max_halves(RT, CS, PL, LV);
  static_assert((4 * TG) % kProducers == 0, "the pieces of a stage are dealt evenly to the producers");
  constexpr int PP = 4 * TG / kProducers;       // 1 KB pieces (4 weight rows x 256 bytes) per producer and stage
  static_assert((S - 2) * PP < 64, "the load counter has six bits");
  constexpr int kStage = TG * 4096;             // bytes of a stage: TG tiles of 16 rows x 128 k
  extern __shared__ uint4 lds4[];
  char* lds = reinterpret_cast<char*>(lds4);
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int ntiles = (g.N + 15) >> 4;
  // this workgroup's share of the weight tiles: equal shares whatever the vocabulary size
  const int t_lo = static_cast<int>(static_cast<int64_t>(blockIdx.x) * ntiles / gridDim.x);
  const int t_hi = static_cast<int>(static_cast<int64_t>(blockIdx.x + 1) * ntiles / gridDim.x);
  const Halves halves(t_lo, t_hi, TG);
  const int nhalf = halves.count;
  const int KB = g.K >> 7;
  const int total = nhalf * KB;                 // stages of this workgroup
  const size_t row_bytes = static_cast<size_t>(g.K) * 2;

  if (wv >= NC && wv < NC + kProducers) {
    // ------------------------------------------------------------------ producer
    // piece j of a stage = rows 4 (j % 4) .. + 3 of tile j / 4; lane l fetches row 4 (j % 4) + l / 16,
    // 16-byte piece (l % 16) ^ row and lands at piece base + 16 l, so that tile entry [row][pos]
    // holds piece pos ^ row: the consumers' per-row operand reads then touch 16 distinct slots.
    // Every stage is as many tiles as the largest half has: a half of one tile less fetches its last one
    // again (an L2 hit), so that every stage counts the same number of loads.
    const int pw = wv - NC;
    static_assert(PP == 2 * TG, "each producer brings in half of every tile");
    const int per_stage = 2 * halves.most;
    StageCursor<MAXH, LV> cur(nhalf, KB);
    // the lane's offset in a tile: rows 4 (j % 4) .. of this producer's pieces, which alternate between two values
    const int r0 = 4 * pw + (lane >> 4), r1 = r0 + 8;
    const uint32_t lane_off0 = r0 * static_cast<uint32_t>(row_bytes) + (((lane & 15) ^ r0) << 4);
    const uint32_t lane_off1 = r1 * static_cast<uint32_t>(row_bytes) + (((lane & 15) ^ r1) << 4);
    static_assert(kProducers == 2, "two producers: each has rows 0-3 and 8-11 or 4-7 and 12-15 of a tile");
    // the same in the launch's last tile: rows past the end repeat the last one, masked later.  (Worked out per request
    // in a loop, the ragged tile's half takes the last workgroup half a microsecond per stage longer, and the launch waits
    // for it: D = 4096, 24 rows, V = 500 / 50257 49.5 / 69.3 us; 32.4 / 68.4 this way.)
    const int rag = (g.N - 1) & 15;              // its last row
    const uint32_t rag_off0 = min(r0, rag) * static_cast<uint32_t>(row_bytes) + (((lane & 15) ^ r0) << 4);
    const uint32_t rag_off1 = min(r1, rag) * static_cast<uint32_t>(row_bytes) + (((lane & 15) ^ r1) << 4);
    auto issue = [&](int slot) {
      char* stage = lds + slot * kStage;
      const int tile0 = halves.first(cur.half0 + cur.h), tile1 = halves.first(cur.half0 + cur.h + 1);
      const uint64_t stride = 16 * row_bytes;
      uint64_t base = reinterpret_cast<uint64_t>(g.w[0]) + static_cast<uint64_t>(tile0) * stride + (static_cast<uint64_t>(cur.k.kb) << 8);
      // (one addition per tile: what a request costs this wave in instructions has to stay below what it costs the memory)
      const auto bring = [&](uint32_t last0, uint32_t last1) {     // the lane's offsets in the half's last tile
#pragma unroll
        for (int u = 0; u < PP; ++u) {
          if (u >= per_stage) break;             // uniform
          if ((u & 1) == 0 && u > 0 && tile0 + u / 2 < tile1) base += stride;
          const bool last = tile0 + u / 2 >= tile1 - 1;      // uniform
          load_to_lds16(reinterpret_cast<const char*>(base), u & 1 ? (last ? last1 : lane_off1) : (last ? last0 : lane_off0),
                        stage + (pw + u * kProducers) * 1024);
        }
      };
      if (tile1 * 16 <= g.N) bring(lane_off0, lane_off1);
      else bring(rag_off0, rag_off1);            // the half with the launch's last, ragged tile
      cur.advance(nhalf, KB);
    };
    int issued = 0;
    for (; issued < S - 1 && issued < total; ++issued) issue(issued % S);
    for (int i = 0; i < total; ++i) {
      // this wave's pieces of stage i have landed once at most the pieces of the S-2 stages issued
      // after it are outstanding (loads return in order); near the end simply wait for all
      if (i + S - 1 < total) wait_tiles<TG, (S - 2) * 2>(halves.most);
      else __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_s_barrier();              // stage i is complete; the slot of stage i-1 is free
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      if (issued < total) {
        issue(issued % S);
        ++issued;
      }
    }
    return;
  }

  // -------------------------------------------------------------------- consumer
  constexpr int NT = RG * RT;      // row tiles of the packed activations
  if constexpr (SPLIT) {
    static_assert(RT == 2 && CS == 1 && PL == 1, "a split last tile is the first of a pair");
    if (wv == NC - 1) Consumer<1, TG / 2, TG, S, PL, TB, MAXH, LV>(g, lds, (NC - 1) * RT, 0, NT, lane, halves, KB).run();
    else if (wv > NC) Consumer<1, TG / 2, TG, S, PL, TB, MAXH, LV>(g, lds, (NC - 1) * RT, TG / 2, NT, lane, halves, KB).run();
    else Consumer<RT, TG, TG, S, PL, TB, MAXH, LV>(g, lds, wv * RT, 0, NT, lane, halves, KB).run();
  } else {
    constexpr int JN = TG / CS;
    Consumer<RT, JN, TG, S, PL, TB, MAXH, LV>(g, lds, (wv / CS) * RT, (wv % CS) * JN, NT, lane, halves, KB).run();
  }
}

// Eight tiles (128 weight rows, 32 KB) per stage and four stages: 96 KB in flight per compute unit.
// Measured at 144 rows, V = 151936, D = 5120: three and five stages the same; three consumer waves of
// three row tiles with one half per pass no faster (fewer LDS reads, more activation loads); the ninth
// row tile shared by two waves instead of one wave next to a full consumer on its SIMD: 1.5 % faster.
constexpr int kWideTiles = 8, kWideStages = 4;

// How the rows are dealt to consumer waves.  One plane: pairs of row tiles per wave from 33 rows on (one LDS read
// then feeds two matrix instructions); fewer rows leave one or two row tiles, whose columns are split
// over four waves, one per SIMD.  Two planes: the pair is value and rest of the same 16 rows.
// Four row tiles: two waves per pair, half of the columns each, so that all four SIMDs work (64 rows, D = 2560 / 5120:
// V = 57000 52 / 98 us, 57 / 106 with one wave per pair; V = 151936 133 / 257 and 139 / 264).  With three, five or six
// an odd last tile is shared by two waves instead, or all SIMDs are busy anyway.
//
// lv: levels of the chunk tree.  Two where the accumulators of a pass take at most 32 registers (one row tile per
// wave, or the draft head's first).  Otherwise the finished siblings do not fit beside them: one level leaves 16 to 20
// bytes a lane of the LM head's kernels in scratch memory and costs 5 to 12 % (V = 40000, 64 rows, D = 2560 / 5120 46.8 / 84 us, 41 / 73 without it;
// the draft step of D = 4096, 40 rows 383, 375).  It pays all the same where rows are 4 KB apart, and every workgroup on
// the same k block keeps one memory channel busy: D = 2048, V = 151936, 40 / 64 / 80 rows 114 / 115 / 124 us, 133 / 141 / 138
// without it; the draft step of 40 rows 188, 185 to 205.  (Half of an 8 KB row is where the same channel comes round
// again: at D = 4096 one level changes nothing.  Rows of 2 KB and less spread over the channels by themselves: D = 1024, 40 /
// 56 / 80 rows, V = 65536 40 / 40 / 43, 30 / 29 / 31 without it, V = 151936 63 / 63 / 69, 57 / 55 / 59.)
struct WideShape { int rg, rt, cs, split, lv; };
WideShape wide_shape(const GemmArgs& g) {
  const int tiles = (g.M + 15) / 16;
  const bool aligned = g.K == 2048;
  if (g.planes == 2) return {tiles, 2, tiles == 1 ? 4 : tiles <= 3 ? 2 : 1, 0, tiles == 1 ? 2 : aligned && tiles <= 3 && g.top_b <= 1 ? 1 : 0};
  if (tiles <= 2) return {tiles, 1, tiles == 1 ? 4 : 2, 0, 2};
  if (aligned && tiles <= 6) return {(tiles + 1) / 2, 2, 2, 0, 1};
  if (tiles == 4) return {2, 2, 2, 0, 0};
  return {(tiles + 1) / 2, 2, 1, tiles & 1, 0};
}

template <int RG, int RT, int CS, int PL, int TB, bool SPLIT, int LV>
hipError_t launch_wide_as(const GemmArgs& g, hipStream_t s) {
  constexpr int TG = kWideTiles, S = kWideStages;
  // set once per process; a function-local static is initialised under the language's own lock
  static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_head_wide<RG, RT, CS, PL, TB, TG, S, SPLIT, LV>),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
  if (attr != hipSuccess) return attr;
  hipLaunchKernelGGL((k_head_wide<RG, RT, CS, PL, TB, TG, S, SPLIT, LV>), dim3(g.wide_w), dim3(64 * (RG * CS + kProducers + (SPLIT ? 1 : 0))),
                     static_cast<size_t>(S) * TG * 4096 + (TB > 1 ? RG * TG * 1024 : 0), s, g);
  return hipGetLastError();
}

// two planes (the draft's widened head): argmax or ranked candidates (those without the one-level tree)
template <int RG, int CS, int LV>
hipError_t launch_wide2(const GemmArgs& g, hipStream_t s) {
  if (g.top_b > 1) return launch_wide_as<RG, 2, CS, 2, SPECEXIT_MAX_TOP_B, false, LV == 2 ? 2 : 0>(g, s);
  return launch_wide_as<RG, 2, CS, 2, 1, false, LV>(g, s);
}

// one plane, pairs of row tiles
template <int RG>
hipError_t launch_wide1(const GemmArgs& g, const WideShape& sh, hipStream_t s) {
  if constexpr (RG <= 3)
    if (sh.lv == 1) return launch_wide_as<RG, 2, 2, 1, 1, false, 1>(g, s);
  if (sh.split) return launch_wide_as<RG, 2, 1, 1, 1, true, 0>(g, s);
  return launch_wide_as<RG, 2, RG == 2 ? 2 : 1, 1, 1, false, 0>(g, s);
}

}  // namespace

bool head_wide_supported(const GemmArgs& g) {
  if (g.V < 0 || g.K % 128 != 0 || g.nseg != 1 || g.M < 1) return false;
  return g.planes == 2 ? g.M <= 64 && g.top_b <= SPECEXIT_MAX_TOP_B : g.top_b <= 1 && g.M <= 160;
}

// One workgroup per compute unit, each walking an equal share of the weight tiles, one candidate slot per workgroup and
// column split.  Vocabularies of less than a stage per compute unit: workgroups of at most one stage's tiles.  (Of at
// least one stage's, the share of 2001 tiles among 250 workgroups is nine, two halves where one would do, and twice the
// stages: V = 32003, D = 5120, 1 / 8 rows 59.5 / 58.5 -> 54 us; V = 4001, D = 4096, 1 / 56 rows 36 / 48 -> 26 / 37.)
void head_wide_plan(GemmArgs& g, int num_cus) {
  if (!head_wide_supported(g)) return;
  const int ntiles = gemm_ntiles(g.N);
  const WideShape sh = wide_shape(g);
  g.wide_w = std::min(num_cus, (ntiles + kWideTiles - 1) / kWideTiles);
  g.wide_slots = sh.split ? 2 : sh.cs;
}

int head_wide_groups(const GemmArgs& g) { return g.wide_w * g.wide_slots; }

// bytes of the packed activations: the row tiles the consumer waves cover x K (none: read in place)
size_t head_wide_pack_bytes(const GemmArgs& g) {
  if (g.wide_w < 1) return 0;
  const WideShape sh = wide_shape(g);
  if (g.planes == 1 && sh.rt == 1) return 0;
  return static_cast<size_t>(sh.rg) * sh.rt * 16 * g.K * 2;
}

hipError_t launch_head_wide(const GemmArgs& ga, hipStream_t s) {
  if (!head_wide_supported(ga) || ga.wide_w < 1) return hipErrorInvalidValue;
  const WideShape sh = wide_shape(ga);
  GemmArgs g = ga;
  const int KB = g.K >> 7;
  if (g.planes == 2) {
    if ((g.a_mode != 3 && g.a_mode != 4) || !g.a_packed) return hipErrorInvalidValue;
    if (g.a_mode == 3)
      hipLaunchKernelGGL(k_pack_norm, dim3((KB * sh.rg + 3) / 4), dim3(256), 0, s, static_cast<const float*>(g.a_src), g.a_ssq, g.a_nssq,
                         static_cast<const bf16_t*>(g.a_gain), g.a_eps, static_cast<uint4*>(g.a_packed), g.M, g.K, sh.rg);
    switch (sh.rg) {
      case 1: return launch_wide2<1, 4, 2>(g, s);                                              //  1 .. 16 rows
      case 2: return sh.lv ? launch_wide2<2, 2, 1>(g, s) : launch_wide2<2, 2, 0>(g, s);        // 17 .. 32
      case 3: return sh.lv ? launch_wide2<3, 2, 1>(g, s) : launch_wide2<3, 2, 0>(g, s);        // 33 .. 48
      case 4: return launch_wide2<4, 1, 0>(g, s);                                              // 49 .. 64
      default: return hipErrorInvalidValue;
    }
  }
  if (g.a_mode != 1) return hipErrorInvalidValue;
  if (sh.rt == 1) {
    g.a_packed = nullptr;
    return sh.rg == 1 ? launch_wide_as<1, 1, 4, 1, 1, false, 2>(g, s) : launch_wide_as<2, 1, 2, 1, 1, false, 2>(g, s);
  }
  if (!g.a_packed) return hipErrorInvalidValue;
  const int units = KB * sh.rg * sh.rt;
  hipLaunchKernelGGL(k_pack_act, dim3((units + 3) / 4), dim3(256), 0, s, static_cast<const bf16_t*>(g.a_src),
                     static_cast<uint4*>(g.a_packed), g.M, g.K, sh.rg * sh.rt);
  switch (sh.rg) {
    case 2: return launch_wide1<2>(g, sh, s);      // 33 ..  64 rows
    case 3: return launch_wide1<3>(g, sh, s);      // 65 ..  96
    case 4: return launch_wide1<4>(g, sh, s);      // 97 .. 128
    case 5: return launch_wide1<5>(g, sh, s);      // 129 .. 160
    default: return hipErrorInvalidValue;
  }
}

}  // namespace sx
