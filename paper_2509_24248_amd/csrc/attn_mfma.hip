// bf16 attention on the matrix cores (head_dim 128 or 64), HBM-bound by design.
//
// A workgroup takes an equal share of all keys of the launch (attn_sched.hpp): one or more
// segments, each a key range of one (sequence, KV head) unit, processed against all
// R = G * n_q query rows that share that head, so the cache is read once.
//
// Inside a workgroup there are two independent tile rings (key groups), four in verifications of few query rows; ring kg
// takes the 32-key tiles kg, kg+2 (kg+4), ... of the chunk.  A ring is S slots in LDS (K tile + V tile: 16 KB
// with 128-wide heads, 8 KB with 64-wide ones).  Tiles are brought in by direct global->LDS loads (16 bytes per lane, streaming),
// issued S-1 tiles ahead by the ring's waves in turn, so most of the LDS holds bytes in
// flight.  Each of the ring's NR waves owns one or two 16-row tiles of the queries and computes them
// against every tile of the ring:
//   S^T = K Q^T : A operand = K rows (row = key, 8 consecutive d per lane) read from the
//                 XOR-swizzled K tile; B operand = Q^T pieces held in registers;
//   softmax     : online, per wave, in log2 units; lane (row, q) owns 8 keys of its row;
//   O^T += V^T P^T : A operand = V^T read from the row-major V tile with the LDS transpose
//                 load (ds_read_b64_tr_b16), B operand = P^T straight from the softmax
//                 registers.
// One workgroup barrier per tile step hands a landed tile to the waves and frees the slot
// consumed one step earlier (rings of one wave need none).  The rings merge at the end in a fixed order.
//
// Short calls are a chain: lengths, split, queries and tiles, one or two tiles of arithmetic, merge.  So queries and tiles are
// requested together, addresses that only later code needs are worked out behind the requests, and code that runs once is
// kept short (it is fetched for that).  Calls of many rows are bound by the vector instructions of the softmax: one fused
// multiply-add and one exponential per score, no maximum over the lanes unless a row's grew.  Whole calls, before / after this
// form (with the work split that pads units, and the merge in one round of requests): 36 calls of 1 sequence x 4096 entries, 7
// queries of 32 heads, 15.1 / 13.1 us each; 8 of 1000-8000, 64 rows of 64-wide heads, paged 29.6 / 26.2; 16 of 8192-32768, 72
// rows, paged 251 / 238 (4.9 TB/s of cache entries); 16 of 250-750, 5 queries of 32 heads 20.2 / 17.0.
#include "attn_sched.hpp"
#include "common.hpp"
#include "kernels.hpp"
#include "stream.hpp"

#include <float.h>

namespace sx {

namespace {

// Tile rings (key groups) per workgroup, NK: two of several waves each, or, in verifications of up to 16 query rows per KV head, four of one
// wave, which then wait for nobody: the wave that brings a tile in is the one that reads it, and one workgroup per compute unit has in
// flight what two of two rings had, with half the partial results.  Layers of 8 KV heads, 2 rings / 4: 3 sequences of 1000-3000 entries,
// 12 rows, contiguous / paged 13.0 -> 12.2 / 13.7 -> 13.2 us, 8 rows 12.7 -> 11.6; 1 of 5000, 12 rows 11.8 -> 11.3; 64-wide heads, 16 of
// 500-2500, 16 rows 14.8 -> 14.1, 8 of 4000-8000, 12 rows 21.0 -> 19.7 (two workgroups of two-slot rings; one of four slots 20.6).
// Draft steps and tree levels (AttnArgs::draft) keep two rings whatever the rows: four add the keys in another order, and a call that
// ranks its own logits then names other tokens where two of them are closer than that rounding (2 of 48 candidates of a level of 4 x 4
// nodes, V = 151936).  That costs a round of six steps, D = 2560, 0.3 % of its time (1199 -> 1203 us).
constexpr int kFewRings = 4;
constexpr int slot_bytes(int hd) { return 128 * hd; }   // one ring slot: 32 K rows then 32 V rows of hd bf16 values
// From big_from waves per ring (128-wide heads: more than 48 query rows per KV head) one workgroup is resident per
// compute unit (its eight to sixteen waves need more than the 96-128 registers per lane that two
// workgroups would leave them) and its two rings take four slots; below that, two workgroups of two
// two-slot rings (or one of four such rings, see above).  Measured at 64 / 72 rows per KV head (8B-like tree block / 32B-like chain block):
// two resident workgroups with spills 41.6 us against 31.3 us with one; two, three and four slots
// within 3 % of each other at 72 rows.
// With 64-wide heads the output accumulators and the slots are half as large: two workgroups fit up to
// four waves per ring, and the rings take twice the slots in the same LDS.  Measured at 64 rows per KV
// head, contexts 1000-8000 of 8 sequences (74 MB), whole call: 26 us; on the ALU kernel 365 us.
constexpr int big_from(int hd) { return hd == 64 ? 5 : 4; }
constexpr bool two_part(int hd, int nr) { return hd == 64 || nr <= 3; }     // (see kSplitP)
// Four rings take two slots each.
constexpr int stages_of(int hd, int nr, int nk) { return nk == kFewRings ? 2 : (nr >= big_from(hd) ? 4 : 2) * (hd == 64 ? 2 : 1); }
constexpr int wgs_per_cu(int hd, int nr, int nk) { return nr >= big_from(hd) || (nk == kFewRings && hd == 128) ? 1 : 2; }
// K operand reads / V operand read pairs issued ahead of the matrix instructions that use them: as
// many as the registers allow (one resident workgroup: all eight K reads, four V pairs; 64-wide heads
// have four of each)
constexpr int k_ahead(int hd, int nr) { return hd == 128 && nr >= big_from(hd) ? 8 : 4; }
constexpr int v_ahead(int hd, int nr) { return hd == 64 || nr >= big_from(hd) ? 4 : 3; }
// From kPairFrom row tiles on (97 and more query rows per KV head, 128-wide heads) a wave takes two row tiles: four
// waves per ring with 256 registers a lane, which read every K and V operand once for 32 rows.  One tile per
// wave leaves the seven or eight waves of a ring 128 registers, of which 8 to 150 bytes a lane go to scratch memory.
// Whole calls, contiguous / paged: 16 sequences of 4000-16000 entries, 64 query heads, 104 rows 182 / 192 -> 152 / 161 us,
// 128 rows 164 / 175 -> 166 / 174; 32 query heads, 8 sequences of 2000-8000, 128 rows 64 / 69 -> 58 / 60; 1 of 20000, 100
// rows 43.5 / 44 -> 35.5 / 36; a 16-node tree over 4 sequences of 300-900, 128 rows 35.5 -> 31.8.  With fewer rows nothing
// spills and one tile per wave is faster (measured at 72 rows).
constexpr int kPairFrom = 7;
constexpr int tiles_per_wave(int hd, int tiles) { return hd == 128 && tiles >= kPairFrom ? 2 : 1; }
constexpr int kMaxChunkPages = 2048;   // page ids of one chunk kept in LDS (8 KB)

constexpr int ml_rows(int nk, int rp) { return nk == kFewRings ? nk * rp : rp; }   // (max, sum) pairs that the merge of the rings passes through LDS

typedef short s16x4_t __attribute__((ext_vector_type(4)));

// Maxima that hand a NaN on: the instruction needs no quieting of its inputs, of which there would be one each.
__device__ __forceinline__ float max_nan(float a, float b) { return __builtin_elementwise_maximum(a, b); }
__device__ __forceinline__ float max3_nan(float a, float b, float c) { return max_nan(max_nan(a, b), c); }

// XOR swizzle of the 16-byte chunks of a tile row.  K rows are read one row per lane (16 rows
// at once): chunk ^ (key % 16) spreads them over all banks.  V rows are read by the transpose
// load, 4 rows x 2 adjacent chunks at once: chunk ^ (2 (key % 8)) keeps those eight apart.
// A 64-wide row is 8 chunks, two rows to the 256 bytes of all banks: the row's parity already picks
// one half of them, the other bits of the key spread the chunks of that half.
template <int HD> __device__ __forceinline__ int swz_k(int key) { return HD == 128 ? key & 15 : (key >> 1) & 7; }
template <int HD> __device__ __forceinline__ int swz_v(int key) { return HD == 128 ? (key & 7) << 1 : ((key >> 1) & 3) << 1; }

// waves per SIMD the register allocation has to leave room for: the resident workgroups' waves on
// four SIMDs
// (One wave a ring has room for any number, and the compiler then keeps the accumulators where every rescaling has to fetch them: 3
// sequences of 1000-3000 entries, 12 rows, 13.5 -> 13.0 us a call with 256 registers.)
constexpr int min_waves_per_simd(int hd, int nr, int nk) { return nr == 1 ? 2 : (wgs_per_cu(hd, nr, nk) * nk * nr + 3) / 4; }

// NR waves per ring, each owning RTW 16-row tiles of the queries (rows 16 (rr RTW + t) ..).
// RTW = 2 halves the LDS reads per query row (K and V operands are fetched once per wave and
// used for both row tiles) at the price of fewer, fatter waves (see kPairFrom).
template <int HD, int NR, int RTW, int S, int NK, bool PAGED>
__global__ __launch_bounds__(64 * NK * NR, min_waves_per_simd(HD, NR, NK)) void k_attn_ring(const AttnArgs a) {
  constexpr int RP = 16 * NR * RTW;             // query rows covered (padded)
  constexpr int kKAhead = k_ahead(HD, NR), kVAhead = v_ahead(HD, NR);
  constexpr int kSlot = slot_bytes(HD);
  constexpr int kRowB = 2 * HD;                 // bytes of a cache row
  constexpr int kChunks = HD / 8;               // 16-byte chunks of a cache row
  constexpr int kKeysPP = 1024 / kRowB;         // keys of a 1 KB piece
  constexpr int kTileP = 32 / kKeysPP;          // pieces of a K (or V) tile
  // Probabilities as a bf16 value plus the bf16 rounding of the rest, 16 to 17 bits.  64-wide heads: the ALU
  // kernel that served them multiplied with fp32 probabilities.  What is lost (2^-17 relative per probability) is far below
  // the bf16 rounding of the output: error against 64 bits over eight inputs each, that kernel / this one, 8 contexts of
  // 300-3000 x 16 queries 1.658633e-3 / 1.658634e-3, 4 of 64-200 x 5 1.661877e-3 / 1.661878e-3, 1 of 9000 x 7 1.660461e-3 /
  // 1.660462e-3.  128-wide heads of up to 48 rows: the matrix cores have the time (36 layers of 1 sequence x 4096 entries, 28 rows: 445
  // us with one part, 449 with two; 8 of 4000-8000, 40 rows, paged 53 and 46, because two parts need no sum by matrix instructions
  // and leave nothing in scratch memory), and with one part the error grows where the work split makes segments larger
  // (2.055e-3 with the segments of an unpadded split, 2.077e-3 with today's; 1.657e-3 with two parts).  More rows: two parts
  // cost 3 to 9 % (16 sequences of 8192-32768, 72 rows: 237 and 259 us), so the probabilities keep one.
  // An infinite V entry is not what the two parts can multiply with: the merging kernels compute rows that are not finite
  // again.
  constexpr bool kSplitP = two_part(HD, NR);
  // Slack of the softmax reference in log2 units: with probabilities of 16 bits it does not matter how far above 1 they
  // reach (8 sequences of 1000-8000 entries, 64 rows per KV head: 27.8 -> 26.8 us, the same error).  bf16 ones are nearest where the
  // largest are 1 or just below: a slack of 8 is 3 % faster at 72 rows per KV head and costs 6 % of the error against 64 bits
  // (2.05e-3 -> 2.19e-3, 4096 entries), so they have none.
  constexpr float kSlack = kSplitP ? 8.f : 0.f;
  constexpr int kKS = HD / 32, kDT = HD / 16;   // k steps of K Q^T, 16-wide column tiles of the output
  // LDS: the rings' slots, S each (for the merge of two rings free ones hold ring 1's sums, for that of four each ring's its own), (max, sum)
  // per row, of ring 1 or of each of the four, the schedule's prefix table, the page ids of the segment
  constexpr int kFront = NK * S * kSlot;
  extern __shared__ uint4 smem4[];
  char* smem = reinterpret_cast<char*>(smem4);
  float* ml_lds = reinterpret_cast<float*>(smem + kFront);
  int* sched_lds = reinterpret_cast<int*>(smem + kFront + ml_rows(NK, RP) * 2 * sizeof(float));
  int* pg_lds = sched_lds + attn_sched_words(a.B);
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int kg = wv / NR, rr = wv % NR;
  const int G = a.G;
  const int R = G * a.n_q;
  const int fr = lane & 15, fq = lane >> 4;
  const AttnTable table = attn_sched_build(a, sched_lds);
  const AttnLine line = attn_sched_line(a, table);
  if (static_cast<int>(blockIdx.x) >= line.W) return;  // the whole workgroup leaves together
  const int x_hi = attn_sched_lo(line, blockIdx.x + 1);
  bool again = false;                           // a segment before this one used the rings
  AttnSeg seg = attn_sched_next(a, table, true, line.pad, attn_sched_lo(line, blockIdx.x), x_hi);
  if (seg.next < x_hi) attn_sched_keep(a, table);
  for (; seg.s1 > seg.s0; seg = attn_sched_next(a, table, false, line.pad, seg.next, x_hi)) {
  attn_sched_publish(a, seg);
  const int g = seg.g, b = seg.b;
  const int L = __builtin_amdgcn_readfirstlane(seg.L);
  const int s0 = seg.s0, s1 = __builtin_amdgcn_readfirstlane(seg.s1);
  const int ntl = (s1 - s0 + 31) >> 5;          // 32-key tiles in this segment
  const int nit = (ntl + NK - 1) / NK;          // tile steps (the same for all rings)
  char* ring = smem + kg * (S * kSlot);

  // ---- Q^T operand pieces and the mask words of this wave's rows (rows past the last one repeat it and are not stored)
  uint4 qf[kKS][RTW];
  uint64_t rowmask[RTW];
  int rho[RTW];
#pragma unroll
  for (int t = 0; t < RTW; ++t) {
    rho[t] = 16 * (rr * RTW + t) + fr;
    const int r = min(rho[t], R - 1);
    const int i = (r * a.g_inv) >> 16;          // r / G
    const bf16_t* qp = static_cast<const bf16_t*>(a.q) + ((static_cast<size_t>(b) * a.n_q + i) * a.Hq + g * G + (r - i * G)) * HD + fq * 8;
#pragma unroll
    for (int ks = 0; ks < kKS; ++ks) qf[ks][t] = *reinterpret_cast<const uint4*>(qp + ks * 32);
    rowmask[t] = a.mask ? a.mask[static_cast<size_t>(b) * a.mask_stride + i] : ((2ull << i) - 1ull);
  }

  // ---- page ids of the segment, copied to LDS once: loads from there do not count against
  // the vector-memory counter that paces the tile loads
  const int ps_shift = 31 - __builtin_clz(a.page_size);
  const int pg0 = s0 >> ps_shift;               // first page index of the segment
  if (PAGED) {
    const int npg = ((s1 - 1) >> ps_shift) - pg0 + 1;
    const int32_t* ptab = a.page_table + static_cast<size_t>(b) * a.max_pages + pg0;
    for (int i = threadIdx.x; i < npg; i += 64 * NK * NR) {
      pg_lds[i] = checked_page(ptab[i], a.n_pages, a.status);   // never leave the pool
    }
  }
  if (PAGED || again) __syncthreads();          // the page ids are there, and the rings are free of the segment before
  again = true;

  // ---- tile loads: the ring's waves take the one-KB pieces of a tile (K, then V: kTileP each) in
  // turn.  Piece j holds the kKeysPP keys from kKeysPP (j % kTileP) on; lane l fetches key
  // l / kChunks of them, 16-byte chunk (l % kChunks) ^ swizzle(key), and lands at piece base + 16 l, so
  // that LDS entry [key][pos] holds chunk pos ^ swizzle(key).  The swizzle is the exclusive or of a lane's part and a piece's
  // part, so a piece costs one instruction per lane and no registers between tiles.
  constexpr int kPieces = (2 * kTileP + NR - 1) / NR;   // pieces a wave issues per tile, at most
  // (where they divide evenly a wave has kPieces in a row, whose swizzles are then constants, since the first key is a multiple of
  // 16: 0.5 to 1 % of a short call, whose first requests wait for this arithmetic)
  constexpr bool kInRow = 2 * kTileP % NR == 0 && kPieces * kKeysPP % 16 == 0;
  const int piece0 = kInRow ? rr * kPieces : rr;
  constexpr int kPieceStep = kInRow ? 1 : NR;
  const int key0 = kKeysPP * (piece0 & (kTileP - 1));
  const bool only_v = NR > 1 && piece0 >= kTileP;        // (kInRow, several waves: a wave has K pieces or V pieces)
  const char* const pool = static_cast<const char*>(only_v ? a.v : a.k);
  const int lkey = lane / kChunks, lpos = lane % kChunks;
  const uint32_t lane_k = static_cast<uint32_t>(lkey) * kRowB + ((lpos ^ swz_k<HD>(lkey)) << 4);
  const uint32_t lane_v = static_cast<uint32_t>(lkey) * kRowB + ((lpos ^ swz_v<HD>(lkey)) << 4);
  // Byte offsets in the pool of a whole tile's first and second 16 keys (pages of 16 * 2^n tokens: a 32-aligned tile
  // touches at most the page of key 0 and the page of key 16), uniform.
  const int64_t seq_off = PAGED ? 0 : (static_cast<int64_t>(b) * a.Hkv + g) * a.l_max * kRowB;
  int64_t off_a, off_b;
  auto locate = [&](int it) {
    const int t0 = s0 + 32 * (it * NK + kg);
    if (t0 >= s1) return;                        // uniform per wave
    if (PAGED) {
      const int p1 = min(t0 + 16, s1 - 1);
      const int pg_a = __builtin_amdgcn_readfirstlane(pg_lds[(t0 >> ps_shift) - pg0]), pg_b = __builtin_amdgcn_readfirstlane(pg_lds[(p1 >> ps_shift) - pg0]);
      off_a = (static_cast<int64_t>(pg_a) * a.Hkv + g) * a.page_size * kRowB;
      off_b = (static_cast<int64_t>(pg_b) * a.Hkv + g) * a.page_size * kRowB;
    } else {
      off_a = off_b = seq_off;
    }
  };
  auto issue = [&](int it) {                     // (after locate of the same tile)
    const int t0 = s0 + 32 * (it * NK + kg);
    if (t0 >= s1) return;
    char* slot = ring + (it % S) * kSlot;
    if (t0 + 32 <= s1) {
      // whole tile inside the range: uniform base per piece + the lane's constant offset
      const int64_t in_page = static_cast<int64_t>(PAGED ? t0 & (a.page_size - 1) : t0) * kRowB;
      if constexpr (kInRow) {
#pragma unroll
        for (int u = 0; u < kPieces; ++u) {
          const int rel = kKeysPP * (u & (kTileP - 1));                           // keys behind key0
          const bool is_v = NR > 1 ? only_v : u >= kTileP;
          const int row = PAGED ? (key0 + rel) & (a.page_size - 1) : key0 + rel;
          const char* base = (NR > 1 ? pool : static_cast<const char*>(is_v ? a.v : a.k)) +
                             ((PAGED && a.page_size == 16 && key0 + rel >= 16 ? off_b : off_a) + in_page + row * kRowB);
          const uint32_t lane_off = is_v ? lane_v ^ (swz_v<HD>(rel) << 4) : lane_k ^ (swz_k<HD>(rel) << 4);
          load_to_lds16(base, lane_off, slot + (piece0 + u) * 1024);
        }
        return;
      }
#pragma unroll
      for (int u = 0; u < kPieces; ++u) {
        const int j = piece0 + u * kPieceStep;
        if (j < 2 * kTileP) {
          const bool second = PAGED && a.page_size == 16 && (j & (kTileP / 2));   // keys 16..31 sit in the next page
          const int key = kKeysPP * (j & (kTileP - 1));                           // the piece's first key
          const int row = PAGED ? key & (a.page_size - 1) : key;
          const char* base = static_cast<const char*>(j < kTileP ? a.k : a.v) + ((second ? off_b : off_a) + in_page + row * kRowB);
          load_to_lds16(base, j < kTileP ? lane_k ^ (swz_k<HD>(key) << 4) : lane_v ^ (swz_v<HD>(key) << 4), slot + j * 1024);
        }
      }
      return;
    }
    const int page0 = t0 >> ps_shift;
    int lk = lkey;                               // (worked out here, once per segment at most)
    asm volatile("" : "+v"(lk));
#pragma unroll
    for (int u = 0; u < kPieces; ++u) {
      const int j = piece0 + u * kPieceStep;
      if (j < 2 * kTileP) {
        const int key = kKeysPP * (j & (kTileP - 1)) + lk;
        const int p = min(t0 + key, s1 - 1);   // keys past the range are masked in the softmax
        int64_t off;
        if (PAGED) off = ((p >> ps_shift) == page0 ? off_a : off_b) + (p & (a.page_size - 1)) * kRowB;
        else off = off_a + static_cast<int64_t>(p) * kRowB;
        load_to_lds16(static_cast<const char*>(j < kTileP ? a.k : a.v) + off + ((lpos ^ (j < kTileP ? swz_k<HD>(key) : swz_v<HD>(key))) << 4), slot + j * 1024);
      }
    }
  };
  constexpr int kPiecesMin = 2 * kTileP / NR;  // pieces every wave of a ring issues per tile, at least

  f32x4_t oacc[kDT][RTW], lacc[RTW];
  float m_run[RTW], l_run[RTW];
#pragma unroll
  for (int t = 0; t < RTW; ++t) {
    m_run[t] = -FLT_MAX;
    l_run[t] = 0.f;
    lacc[t] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int dt = 0; dt < kDT; ++dt) oacc[dt][t] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  }
  const float sl2 = a.scale * 1.44269504088896340736f;  // scores are kept in log2 units

  // Every slot is free here: a short segment has all its tiles in flight at once, behind the queries and at the same time.  In the
  // deep rings of a longer one that is up to 128 KB in front of the first matrix instruction, and nothing is requested
  // meanwhile: there the wait is for the queries and the first tile (a paged launch has the queries with the page ids), and the other
  // tiles follow it.  8 sequences x 4096 entries, 64 rows, contiguous 35.2 -> 33.6 us, paged 38.5 -> 36.6 (two-slot
  // rings gain nothing from it).
  const int together = S == 2 ? S : PAGED ? 0 : nit < S ? S : 1;
#pragma unroll 1
  for (int it = 0; it < together; ++it) {
    locate(it);
    issue(it);
  }
  // (the lane's part of the operand addresses is worked out here, while the loads are on their way, and not in front of them)
  int fr_t = fr, fq_t = fq;
  asm volatile("" : "+v"(fr_t), "+v"(fq_t));
  __builtin_amdgcn_sched_barrier(0);
  // Of the reads' addresses a lane keeps one for K and one for V: a read is the exclusive or with its number and the slot's base,
  // one instruction (held in registers they are 24, and the paged kernel of three waves a ring spills).
  const int ve = fr_t >> 2, vc = fr_t & 3;
  int k_at = fr_t * kRowB + ((fq_t ^ swz_k<HD>(fr_t)) << 4);
  int v_at = (4 * fq_t + ve) * kRowB + (((vc >> 1) ^ swz_v<HD>(4 * fq_t + ve)) << 4) + ((vc & 1) << 3);

  __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));    // from here on vmcnt counts tile loads only
  if constexpr (S > 2) {
#pragma unroll 1
    for (int it = together; it < S; ++it) {
      locate(it);
      issue(it);
    }
  }

#pragma unroll 1                              // (no first round of its own: code that is run once is fetched for that)
  for (int it = 0; it < nit; ++it) {
    if (it > 0) locate(it + S - 1);
    // this wave's pieces of tile `it` have landed once at most the pieces of the S-2 tiles (S-1 before the first, if this ring
    // has that many) issued after it are outstanding (loads return in order); near the end simply wait for all
    if (S == 2 || it + S - 1 >= nit) __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
    else if (it == 0 && (S - 1) * NK + kg < ntl) __builtin_amdgcn_s_waitcnt(vmcnt_imm((S - 1) * kPiecesMin));
    else __builtin_amdgcn_s_waitcnt(vmcnt_imm((S - 2) * kPiecesMin));
    // plain barrier (no memory fence: a fence would wait for the loads still in flight); the
    // wave-scope fences only keep the compiler from moving LDS accesses across it
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    if constexpr (NR > 1) __builtin_amdgcn_s_barrier();   // tile `it` complete; slot of tile it-1 free
    else __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0): (of one wave, tile it-1 is read)
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    if (it > 0) issue(it + S - 1);
    const int ti = it * NK + kg;
    if (ti >= ntl) continue;
    const int t0 = s0 + 32 * ti;
    const char* k_lds = ring + (it % S) * kSlot;
    const char* v_lds = k_lds + kSlot / 2;
    asm volatile("" : "+v"(k_at), "+v"(v_at));

    // ---- S^T = K Q^T for the two 16-key halves.  The K operand reads run kKAhead reads ahead of the
    // matrix instructions that use them, and the first V operand reads are issued here as well (they do
    // not depend on the softmax).  The scheduler is kept from sinking the reads back to their uses: left
    // alone it aims at the fewest registers and leaves one LDS round trip per matrix instruction exposed.
    f32x4_t sacc[2][RTW];
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int t = 0; t < RTW; ++t) sacc[j][t] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    auto kread = [&](int i) {       // read i: k step i / 2, key half i % 2
      return *reinterpret_cast<const uint4*>(k_lds + (k_at ^ ((i >> 1) << 6)) + (i & 1) * 16 * kRowB);
    };
    // Transpose load of V: within 16 lanes, lane i = 4 e + c points at key e's four values
    // d0 + 4c .. d0 + 4c + 3 and lane j receives column d0 + j of keys e = 0..3.  Two loads give the
    // 8 keys of the operand in the order P^T uses: 4q..4q+3 of the first half, then of the second half.
    s16x4_t vlo[kDT], vhi[kDT];
    auto vread = [&](int dt) {
      const char* p = v_lds + (v_at ^ (dt << 5));
      vlo[dt] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4_t*)(lds_ptr_t)p);
      vhi[dt] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4_t*)(lds_ptr_t)(p + 16 * kRowB));
    };
    constexpr int kReads = 2 * kKS;
    uint4 kf[kReads];
#pragma unroll
    for (int i = 0; i < kKAhead; ++i) kf[i] = kread(i);
#pragma unroll
    for (int i = 0; i < kReads; ++i) {
      if (i + kKAhead < kReads) kf[i + kKAhead] = kread(i + kKAhead);
      if (i >= kReads - kVAhead) vread(i - (kReads - kVAhead));      // the last K steps also start the V reads
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int t = 0; t < RTW; ++t)
        sacc[i & 1][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, kf[i]),
                                                                __builtin_bit_cast(bf16x8_t, qf[i >> 1][t]), sacc[i & 1][t], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }

    // ---- online softmax; lane (row, q) owns keys t0 + 16 j + 4 q + e of its row.  The reference the exponents are taken
    // against moves only when one of the wave's scores exceeds its row's by more than kSlack: tiles in which none does need
    // neither the maximum over the row's lanes nor the rescaling.
    const bool plain = t0 + 32 <= min(L, s1) && sl2 > 0.f;
    uint4 pf[RTW], pl[RTW];
#pragma unroll
    for (int t = 0; t < RTW; ++t) {
      float x[8];
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) x[4 * j + e] = sacc[j][t][e];
      float unit = sl2;
      if (!plain) {
        unit = 1.f;
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int p = t0 + 16 * j + 4 * fq_t + e;
            bool vis = p < s1;
            if (vis && p >= L) vis = (rowmask[t] >> (p - L)) & 1ull;
            x[4 * j + e] = vis ? x[4 * j + e] * sl2 : -INFINITY;
          }
      }
      float mt = max3_nan(max3_nan(x[0], x[1], x[2]), max3_nan(x[3], x[4], x[5]), max_nan(x[6], x[7])) * unit;
      if (__builtin_amdgcn_ballot_w64(mt > m_run[t] + kSlack) != 0ull) {
        const float m_new = fmaxf(m_run[t], quad_row_max(mt));
        const float al = __builtin_amdgcn_exp2f(m_run[t] - m_new);
        m_run[t] = m_new;
        if constexpr (kSplitP) l_run[t] *= al;
        else lacc[t][0] *= al;
#pragma unroll
        for (int dt = 0; dt < kDT; ++dt) {
          oacc[dt][t][0] *= al; oacc[dt][t][1] *= al;
          oacc[dt][t][2] *= al; oacc[dt][t][3] *= al;
        }
      }
      float pr[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) pr[e] = __builtin_amdgcn_exp2f(fmaf(x[e], unit, -m_run[t]));
      pf[t] = make_uint4(pack_bf16x2(pr[0], pr[1]), pack_bf16x2(pr[2], pr[3]), pack_bf16x2(pr[4], pr[5]),
                         pack_bf16x2(pr[6], pr[7]));
      if constexpr (kSplitP) {
        float hi[8];
        unpack16(pf[t], hi);
        pl[t] = make_uint4(pack_bf16x2(pr[0] - hi[0], pr[1] - hi[1]), pack_bf16x2(pr[2] - hi[2], pr[3] - hi[3]),
                           pack_bf16x2(pr[4] - hi[4], pr[5] - hi[5]), pack_bf16x2(pr[6] - hi[6], pr[7] - hi[7]));
        l_run[t] += ((pr[0] + pr[1]) + (pr[2] + pr[3])) + ((pr[4] + pr[5]) + (pr[6] + pr[7]));
      } else {
        // the probabilities as V is multiplied with them, summed in fp32 by a product with a column of ones: weights that are
        // normalised with their own sum leave less of their rounding in the output than with the sum of the unrounded ones
        const uint32_t one = 0x3F803F80u;
        lacc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, make_uint4(one, one, one, one)),
                                                          __builtin_bit_cast(bf16x8_t, pf[t]), lacc[t], 0, 0, 0);
      }
    }

    // ---- O^T += V^T P^T, the V operand reads kVAhead matrix instructions ahead
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int dt = 0; dt < kDT; ++dt) {
      if (dt + kVAhead < kDT) vread(dt + kVAhead);
      __builtin_amdgcn_sched_barrier(0);
      const uint2 l2 = __builtin_bit_cast(uint2, vlo[dt]), h2 = __builtin_bit_cast(uint2, vhi[dt]);
      const bf16x8_t va = __builtin_bit_cast(bf16x8_t, make_uint4(l2.x, l2.y, h2.x, h2.y));
#pragma unroll
      for (int t = 0; t < RTW; ++t) {
        oacc[dt][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(va, __builtin_bit_cast(bf16x8_t, pf[t]), oacc[dt][t], 0, 0, 0);
        if constexpr (kSplitP)
          oacc[dt][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(va, __builtin_bit_cast(bf16x8_t, pl[t]), oacc[dt][t], 0, 0, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  }

  constexpr int kOBytes = 64 * HD;               // 16 rows
  if constexpr (NK == 2) {
  // ---- merge the two rings of each row: ring 1 leaves its sums in LDS, ring 0 adds them to its own (always in this order) and
  // stores the segment's partial result.  Slots other than the last tile's are free since the last barrier: wave rr of ring 1
  // takes piece rr of them, ring 1's first.  Within a row the 16-byte pieces are swizzled like the tiles.
  constexpr int kPerSlot = kSlot / kOBytes;
  static_assert(kSlot == 2 * kOBytes && NR * RTW <= 2 * kPerSlot * (S - 1), "the free slots hold ring 1's sums");
  int fr_o = fr, fq_o = fq;                      // (addresses worked out here, see above)
  asm volatile("" : "+v"(fr_o), "+v"(fq_o));
  auto o_lds = [&](int t) {
    const int n = rr * RTW + t, in = n % (kPerSlot * (S - 1));
    return smem + (n < kPerSlot * (S - 1) ? S * kSlot : 0) + ((nit + in / kPerSlot) % S) * kSlot + in % kPerSlot * kOBytes + fr_o * (4 * HD);
  };
#pragma unroll
  for (int t = 0; t < RTW; ++t) {
    l_run[t] = kSplitP ? quad_row_sum(l_run[t]) : lacc[t][0];
    if (kg == 1) {
      if (fq == 0) *reinterpret_cast<float2*>(ml_lds + 2 * rho[t]) = make_float2(m_run[t], l_run[t]);
      char* dst = o_lds(t);
#pragma unroll
      for (int dt = 0; dt < kDT; ++dt)
        *reinterpret_cast<float4*>(dst + (((4 * dt + fq_o) ^ fr_o) << 4)) = make_float4(oacc[dt][t][0], oacc[dt][t][1], oacc[dt][t][2], oacc[dt][t][3]);
    }
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
  if (kg == 1) continue;
  const size_t unit = static_cast<size_t>(blockIdx.x) + static_cast<size_t>(b) * a.Hkv + g;   // partial slot of segment (w, u)
#pragma unroll
  for (int t = 0; t < RTW; ++t) {
    if (rho[t] >= R) continue;
    const float2 ml = *reinterpret_cast<const float2*>(ml_lds + 2 * rho[t]);
    const float mm = fmaxf(m_run[t], ml.x);
    const float f0 = __builtin_amdgcn_exp2f(m_run[t] - mm), f1 = __builtin_amdgcn_exp2f(ml.x - mm);
    if (fq == 0) *reinterpret_cast<float2*>(a.part_ml + (unit * R + rho[t]) * 2) = make_float2(mm, fmaf(f1, ml.y, f0 * l_run[t]));
    float* dst = a.part_o + (unit * R + rho[t]) * HD + 4 * fq_o;
    const char* src = o_lds(t);
#pragma unroll
    for (int dt = 0; dt < kDT; ++dt) {
      const float4 o = *reinterpret_cast<const float4*>(src + (((4 * dt + fq_o) ^ fr_o) << 4));
      *reinterpret_cast<float4*>(dst + 16 * dt) = make_float4(fmaf(o.x, f1, oacc[dt][t][0] * f0), fmaf(o.y, f1, oacc[dt][t][1] * f0),
                                                              fmaf(o.z, f1, oacc[dt][t][2] * f0), fmaf(o.w, f1, oacc[dt][t][3] * f0));
    }
  }
  } else {
    // ---- merge the four rings: each leaves its sums in its own slots, the 16-byte pieces of a row swizzled like the tiles, and every
    // wave adds some rows, in the order of the rings
    static_assert(NR == 1 && RTW == 1 && kOBytes <= S * kSlot, "a ring's slots hold its sums");
    constexpr int C4 = HD / 4, RPW = 64 / C4;     // 16-byte pieces of a row, rows that a wave adds at a time
    const float l = kSplitP ? quad_row_sum(l_run[0]) : lacc[0][0];
    int fr_o = fr, fq_o = fq;                     // (addresses worked out here, see above)
    asm volatile("" : "+v"(fr_o), "+v"(fq_o));
    if (fq == 0) *reinterpret_cast<float2*>(ml_lds + 2 * (kg * RP + fr_o)) = make_float2(m_run[0], l);
#pragma unroll
    for (int dt = 0; dt < kDT; ++dt)
      *reinterpret_cast<float4*>(ring + fr_o * (4 * HD) + (((4 * dt + fq_o) ^ fr_o) << 4)) = make_float4(oacc[dt][0][0], oacc[dt][0][1], oacc[dt][0][2], oacc[dt][0][3]);
    __syncthreads();
    const size_t unit = static_cast<size_t>(blockIdx.x) + static_cast<size_t>(b) * a.Hkv + g;   // partial slot of segment (w, u)
    const int c4 = lane % C4;
#pragma unroll 1
    for (int r = RPW * wv + lane / C4; r < R; r += RPW * NK) {
      float2 ml[NK];
      float4 o[NK];
#pragma unroll
      for (int k = 0; k < NK; ++k) {
        ml[k] = *reinterpret_cast<const float2*>(ml_lds + 2 * (k * RP + r));
        o[k] = *reinterpret_cast<const float4*>(smem + k * (S * kSlot) + r * (4 * HD) + ((c4 ^ r) << 4));
      }
      float mm = ml[0].x;
#pragma unroll
      for (int k = 1; k < NK; ++k) mm = fmaxf(mm, ml[k].x);
      float sum = 0.f;
      float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
      for (int k = 0; k < NK; ++k) {
        const float f = __builtin_amdgcn_exp2f(ml[k].x - mm);
        sum = fmaf(f, ml[k].y, sum);
        v.x = fmaf(f, o[k].x, v.x); v.y = fmaf(f, o[k].y, v.y);
        v.z = fmaf(f, o[k].z, v.z); v.w = fmaf(f, o[k].w, v.w);
      }
      *reinterpret_cast<float4*>(a.part_o + (unit * R + r) * HD + 4 * c4) = v;
      if (c4 == 0) *reinterpret_cast<float2*>(a.part_ml + (unit * R + r) * 2) = make_float2(mm, sum);
    }
  }
  }
}

constexpr size_t lds_bytes(int hd, int nk, int rp, int stages, int B, bool paged) {
  return static_cast<size_t>(nk) * stages * slot_bytes(hd) + static_cast<size_t>(ml_rows(nk, rp)) * 2 * sizeof(float) +
         static_cast<size_t>(attn_sched_words(B)) * sizeof(int) + (paged ? static_cast<size_t>(kMaxChunkPages + 1) * sizeof(int) : 0);
}

template <int HD, int NR, int RTW, int S, int NK, bool PAGED>
hipError_t launch_one(const AttnArgs& a, hipStream_t s) {
  // as many workgroups as attn_mfma_per_cu counts on fit the 160 KB of a compute unit, at any number of sequences
  static_assert(lds_bytes(HD, NK, 16 * NR * RTW, S, kAttnMaxSeqs, PAGED) * wgs_per_cu(HD, NR, NK) <= 160 * 1024, "the LDS of a compute unit");
  static_assert(NR * RTW <= 8, "at most 128 query rows");
  // set once per process; a function-local static is initialised under the language's own lock,
  // so first calls from several host threads are safe
  static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_attn_ring<HD, NR, RTW, S, NK, PAGED>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
  if (attr != hipSuccess) return attr;
  hipLaunchKernelGGL((k_attn_ring<HD, NR, RTW, S, NK, PAGED>), dim3(a.wgrid), dim3(64 * NK * NR), attn_mfma_lds_bytes(a), s, a);
  return hipGetLastError();
}

template <int HD, int NR, int RTW, int NK>
hipError_t launch_rings(const AttnArgs& a, hipStream_t s) {
  constexpr int S = stages_of(HD, NR, NK);
  return a.paged ? launch_one<HD, NR, RTW, S, NK, true>(a, s) : launch_one<HD, NR, RTW, S, NK, false>(a, s);
}

template <int HD, int TILES>
hipError_t launch_tiles(const AttnArgs& a, hipStream_t s) {
  constexpr int RTW = tiles_per_wave(HD, TILES), NR = (TILES + RTW - 1) / RTW;
  if constexpr (NR == 1) {
    if (a.rings == kFewRings) return launch_rings<HD, NR, RTW, kFewRings>(a, s);
  }
  return launch_rings<HD, NR, RTW, 2>(a, s);
}

template <int HD>
hipError_t launch_hd(const AttnArgs& a, hipStream_t s) {
  const int R = (a.Hq / a.Hkv) * a.n_q;
  switch ((R + 15) / 16) {
    case 1: return launch_tiles<HD, 1>(a, s);
    case 2: return launch_tiles<HD, 2>(a, s);
    case 3: return launch_tiles<HD, 3>(a, s);
    case 4: return launch_tiles<HD, 4>(a, s);
    case 5: return launch_tiles<HD, 5>(a, s);
    case 6: return launch_tiles<HD, 6>(a, s);
    case 7: return launch_tiles<HD, 7>(a, s);
    case 8: return launch_tiles<HD, 8>(a, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

bool attn_mfma_supported(const AttnArgs& a) {
  const int R = (a.Hq / a.Hkv) * a.n_q;
  const bool pow2 = (a.page_size & (a.page_size - 1)) == 0;
  return a.dtype == 1 && (a.d == 128 || a.d == 64) && R <= 128 && (!a.paged || (pow2 && a.page_size >= 16));
}

// Rings, workgroups per compute unit and ring depth (see kFewRings and big_from).
static int row_tiles(const AttnArgs& a) { return ((a.Hq / a.Hkv) * a.n_q + 15) / 16; }
static int waves_per_ring(const AttnArgs& a) {
  const int per = tiles_per_wave(a.d, row_tiles(a));
  return (row_tiles(a) + per - 1) / per;
}
int attn_mfma_rings(const AttnArgs& a) { return waves_per_ring(a) == 1 && !a.draft ? kFewRings : 2; }
int attn_mfma_per_cu(const AttnArgs& a) { return wgs_per_cu(a.d, waves_per_ring(a), a.rings); }
bool attn_mfma_two_part(const AttnArgs& a) { return two_part(a.d, waves_per_ring(a)); }
int attn_mfma_stages(const AttnArgs& a) { return stages_of(a.d, waves_per_ring(a), a.rings); }

size_t attn_mfma_lds_bytes(const AttnArgs& a) {
  const int rp = 16 * waves_per_ring(a) * tiles_per_wave(a.d, row_tiles(a));
  return lds_bytes(a.d, a.rings, rp, a.stages, a.B, a.paged);
}

int attn_mfma_max_chunk(const AttnArgs& a) { return a.paged ? kMaxChunkPages * a.page_size : (1 << 30); }

hipError_t launch_attn_mfma(const AttnArgs& a, hipStream_t s) { return a.d == 64 ? launch_hd<64>(a, s) : launch_hd<128>(a, s); }

}  // namespace sx
