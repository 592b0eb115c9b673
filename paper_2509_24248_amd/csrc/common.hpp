// Shared device helpers for the SpecExit kernels (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace sx {

typedef uint16_t bf16_t;  // raw bfloat16 bits

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(4))) float f32x4_t;

constexpr int kWave = 64;

__device__ __forceinline__ float bf16_to_f32(bf16_t b) {
  return __uint_as_float(static_cast<uint32_t>(b) << 16);
}

// round to nearest even; inputs here are finite
__device__ __forceinline__ bf16_t f32_to_bf16(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return static_cast<bf16_t>(u >> 16);
}

// two floats -> packed bf16 pair (a in the low half), round to nearest even in hardware
__device__ __forceinline__ uint32_t pack_bf16x2(float a, float b) {
  typedef __attribute__((ext_vector_type(2))) float f32x2_t;
  typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_t;
  const f32x2_t v = {a, b};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_t));
}

// Requests every 64-byte line of the kernel's arguments (`BYTES` of them) at once and waits.  They lie in memory that no cache
// holds yet, and the compiler loads each where it is first needed: a chain of misses in a kernel that takes 4 us.
template <int BYTES>
__device__ __forceinline__ void arguments_at_once() {
  typedef const __attribute__((address_space(4))) int* kernarg_t;
  const kernarg_t p = (kernarg_t)__builtin_amdgcn_kernarg_segment_ptr();
  constexpr int N = (BYTES + 63) / 64;
  static_assert(N <= 16, "");
  int v[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) v[i] = p[(i < N ? i : 0) * 16];
  asm volatile("" ::"s"(v[0]), "s"(v[1]), "s"(v[2]), "s"(v[3]), "s"(v[4]), "s"(v[5]), "s"(v[6]), "s"(v[7]), "s"(v[8]), "s"(v[9]), "s"(v[10]),
               "s"(v[11]), "s"(v[12]), "s"(v[13]), "s"(v[14]), "s"(v[15]));
}

template <typename T> struct Elem;
template <> struct Elem<float> {
  static constexpr int kPer16B = 4;
  __device__ static __forceinline__ float load(const float* p) { return *p; }
  __device__ static __forceinline__ void store(float* p, float v) { *p = v; }
};
template <> struct Elem<bf16_t> {
  static constexpr int kPer16B = 8;
  __device__ static __forceinline__ float load(const bf16_t* p) { return bf16_to_f32(*p); }
  __device__ static __forceinline__ void store(bf16_t* p, float v) { *p = f32_to_bf16(v); }
};

// 16-byte vector of storage elements -> floats
__device__ __forceinline__ void unpack16(const uint4& v, float (&f)[8]) {
  f[0] = __uint_as_float(v.x << 16); f[1] = __uint_as_float(v.x & 0xFFFF0000u);
  f[2] = __uint_as_float(v.y << 16); f[3] = __uint_as_float(v.y & 0xFFFF0000u);
  f[4] = __uint_as_float(v.z << 16); f[5] = __uint_as_float(v.z & 0xFFFF0000u);
  f[6] = __uint_as_float(v.w << 16); f[7] = __uint_as_float(v.w & 0xFFFF0000u);
}

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// Maximum over the four lanes l, l ^ 16, l ^ 32, l ^ 48 (the four k groups of a matrix-core
// accumulator column) without an LDS round trip: the swap instructions hand every lane both halves
// of the exchange with its partner row (with both operands equal, the first result holds rows
// 0, 0, 2, 2 and the second rows 1, 1, 3, 3 of 16 lanes; the 32-lane form likewise).
__device__ __forceinline__ float quad_row_max(float v) {
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}

// Sum over the same four lanes.
__device__ __forceinline__ float quad_row_sum(float v) {
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = __uint_as_float(a[0]) + __uint_as_float(a[1]);
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

// Maximum and sum over a wave by rotations within the rows of 16 lanes and the swaps above: some 40 cycles where six shuffles
// through LDS take 400.
template <int CTRL> __device__ __forceinline__ float row_lane(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, false));
}
__device__ __forceinline__ float wave_max_dpp(float v) {
  v = fmaxf(v, row_lane<0x128>(v)); v = fmaxf(v, row_lane<0x124>(v));
  v = fmaxf(v, row_lane<0x122>(v)); v = fmaxf(v, row_lane<0x121>(v));
  return quad_row_max(v);
}
__device__ __forceinline__ float wave_sum_dpp(float v) {
  v += row_lane<0x128>(v); v += row_lane<0x124>(v);
  v += row_lane<0x122>(v); v += row_lane<0x121>(v);
  return quad_row_sum(v);
}

// The sum in the order of wave_sum, lanes 32 apart first: the same bits.  (Once lanes 8 apart hold equal values, those that a rotation
// by 4 brings are the ones 4 apart, and so on.)
__device__ __forceinline__ float wave_sum_halves(float v) {
  const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = __uint_as_float(a[0]) + __uint_as_float(a[1]);
  const auto b = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = __uint_as_float(b[0]) + __uint_as_float(b[1]);
  v += row_lane<0x128>(v); v += row_lane<0x124>(v);
  v += row_lane<0x122>(v); v += row_lane<0x121>(v);
  return v;
}

// Inclusive prefix sum over a wave, by lanes as well: shifts within the rows of 16 lanes, then the last lane of a row to the next one
// (rows 1 and 3) and of the first two rows to the last two.
__device__ __forceinline__ int wave_scan(int x) {
  x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);
  x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);
  x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);
  x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);
  x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);
  x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);
  return x;
}

// (value, index) pair ordered by larger value, then lower index
__device__ __forceinline__ bool better(float v, int i, float bv, int bi) {
  return v > bv || (v == bv && i < bi);
}

__device__ __forceinline__ float sigmoidf_(float x) { return 1.0f / (1.0f + expf(-x)); }

// Values read from device arrays never reach an address unchecked: they are forced into range
// (a bad value then gives a wrong result for its row, never a fault), and the first one seen is
// reported in the caller's device status word when one was given.
constexpr int kStatusBadLength = 1;  // ctx_len / pos < 0 or beyond the cache capacity
constexpr int kStatusBadPage = 2;    // page id outside 0 .. n_pages-1
constexpr int kStatusBadToken = 3;   // token id outside 0 .. V-1
constexpr int kStatusBadNode = 4;    // node id, path entry or row index outside its block

__device__ __forceinline__ void report_status(int* status, int code) {
  if (status) atomicCAS(status, 0, code);
}

__device__ __forceinline__ int checked_page(int page, int64_t n_pages, int* status) {
  if (static_cast<uint32_t>(page) < static_cast<uint32_t>(n_pages)) return page;
  report_status(status, kStatusBadPage);
  return 0;
}

// for writes: a cache entry whose page id is out of range is not written at all
__device__ __forceinline__ bool page_in_pool(int page, int64_t n_pages, int* status) {
  if (static_cast<uint32_t>(page) < static_cast<uint32_t>(n_pages)) return true;
  report_status(status, kStatusBadPage);
  return false;
}

__device__ __forceinline__ int checked_token(int tok, int vocab, int* status) {
  if (static_cast<uint32_t>(tok) < static_cast<uint32_t>(vocab)) return tok;
  report_status(status, kStatusBadToken);
  return 0;
}

}  // namespace sx
