// Device helpers shared by the kernel files: bf16 high / low splits, fragment and cache offsets, reductions, the
// hand-off primitives and the arithmetic of the epilogues.
#pragma once
#include "stairs_kernels.h"

namespace stairs {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;

// ---------------------------------------------------------------------------------------
// helpers
// ---------------------------------------------------------------------------------------
__device__ __forceinline__ float bf16_bits_to_float(uint32_t b) { return __uint_as_float(b << 16); }
// Two floats -> a packed pair of bf16 (a in the low half), round to nearest even, by the conversion instruction of
// gfx950 (one instruction for the pair), and the split
// of the pair into that high part and the bf16 of the remainders.
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t bf16_pack2_rne(float a, float b) {
  const f32x2_t v = {a, b};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_t));
}
// (contraction off here and in split_half8: the remainder must not be fused with a product in front of it in one
// instantiation and left alone in another, or a row's bits would depend on how many rows its kernel was built for)
__device__ __forceinline__ void bf16_split2(float a, float b, uint32_t& hi, uint32_t& lo) {
#pragma clang fp contract(off)
  hi = bf16_pack2_rne(a, b);
  lo = bf16_pack2_rne(a - __uint_as_float(hi << 16), b - __uint_as_float(hi & 0xFFFF0000u));
}

// Activation fragments: the MFMA B operand of a forward with more than 4 rows is formed ONCE by whoever produces the
// activation (embedding gather, attention, the previous projection's epilogue) and kept beside the fp32 values as
// [k-step of 32][column tile of 16 rows (2)][high, low][lane] x 16 bytes: lane r + 16 g of k-step kt holds
// x[16 ct + r][32 kt + 8 g .. + 8] * gain as bf16 (high part) and the bf16 of the remainders (low part), the very
// values split_bf16x8 gives.  A consumer wave loads a fragment as one coalesced 1 KiB read.
// Rows 32..63 (forwards of several sequences) have a second block of the same layout kFragHalfU4 uint4 further on.
__device__ __forceinline__ size_t frag_off(int m, int k) {        // in units of 8 bytes: 4 consecutive k of row m, high part
  return (size_t)(m >> 5) * (kFragHalfU4 * 2) +
         ((((size_t)(k >> 5) * 2 + ((m >> 4) & 1)) * 2) * 64 + (size_t)(k >> 9) * kFragChunkPad + (m & 15) + 16 * ((k & 31) >> 3)) * 2 +
         ((k & 7) >> 2);
}
// row m, columns k .. k+3 (k a multiple of 4); g = the gain of those columns or nullptr
__device__ __forceinline__ void store_frag4(uint4* frag, int m, int k, float4 v, const float* gain) {
  if (gain) {
    const float4 g = *reinterpret_cast<const float4*>(gain + k);
    v.x = v.x * g.x; v.y = v.y * g.y; v.z = v.z * g.z; v.w = v.w * g.w;
  }
  uint2 hi, lo;
  bf16_split2(v.x, v.y, hi.x, lo.x);
  bf16_split2(v.z, v.w, hi.y, lo.y);
  uint2* dst = reinterpret_cast<uint2*>(frag) + frag_off(m, k);
  dst[0] = hi;
  dst[128] = lo;                                               // the low fragment follows 64 lanes x 16 bytes later
}
// base + a byte offset of 32 bits: one address register beside a scalar base
template <typename T>
__device__ __forceinline__ T ld_at(const void* base, uint32_t bytes) {
  return *reinterpret_cast<const T*>(static_cast<const char*>(base) + bytes);
}
// A kernel argument wanted in a register now: all of a kernel's arguments then come in one round trip at its start instead
// of one in front of each part that uses some of them.
template <typename T>
__device__ __forceinline__ void want(const T& v) {
  asm volatile("" ::"s"(v));
}
__device__ __forceinline__ float load_elem(const float* p) { return *p; }
__device__ __forceinline__ float load_elem(const uint16_t* p) { return bf16_bits_to_float(*p); }
// keys/values of bf16 models are cached as IEEE half: same bytes as bf16, 8x smaller rounding step
// (bf16 storage alone moves 1B-class logits by 1.7e-2); saturates at the half range
__device__ __forceinline__ void store_kv(_Float16* p, float v) { *p = (_Float16)fminf(fmaxf(v, -65504.f), 65504.f); }

// four adjacent halves of a key tile (one 8-byte store)
__device__ __forceinline__ void store_kv4(_Float16* p, float4 v) {
  _Float16 h[4];
  store_kv(h, v.x); store_kv(h + 1, v.y); store_kv(h + 2, v.z); store_kv(h + 3, v.w);
  *reinterpret_cast<uint2*>(p) = *reinterpret_cast<const uint2*>(h);
}

// Fragments of a row block (stairs_block.hip): row r, columns k .. k+3 (k a multiple of 4) of a buffer of RT column tiles
__device__ __forceinline__ void blk_store_frag4(uint4* frag, int RT, int r, int k, float4 v) {
  uint2 hi, lo;
  bf16_split2(v.x, v.y, hi.x, lo.x);
  bf16_split2(v.z, v.w, hi.y, lo.y);
  const size_t u4 = (((size_t)(k >> 5) * RT + (r >> 4)) * 2) * 64 + (r & 15) + 16 * ((k & 31) >> 3);
  uint2* dst = reinterpret_cast<uint2*>(frag) + u4 * 2 + ((k & 7) >> 2);
  dst[0] = hi;
  dst[128] = lo;
}

// Butterfly sums without the LDS unit (a ds_bpermute of __shfl_xor is a round trip of 100 cycles and more, a swap or a
// rotation one instruction): x + x of the lane at distance 16, 8, 4, 2, 1, in that order, the additions and the bits of the
// __shfl_xor form.  (A rotation by 8 in a row of 16 is the exchange of its halves; after it the row repeats every 8
// lanes, so a rotation by 4 is the next exchange, and so on.)
template <int CTRL>
__device__ __forceinline__ float dpp(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, true));
}
constexpr int kDppRor8 = 0x128, kDppRor4 = 0x124, kDppXor2 = 0x4E, kDppXor1 = 0xB1;   // (quad_perm [2,3,0,1], [1,0,3,2])
constexpr int kDppHalfMirror = 0x141;                            // lane ^ 7: the other quad of eight lanes
constexpr int kDppQuad0 = 0x00, kDppQuad1 = 0x55, kDppQuad2 = 0xAA, kDppQuad3 = 0xFF;   // a lane of the quad in all four
__device__ __forceinline__ float half_wave_sum(float v) {      // over lanes 0 .. 31 and 32 .. 63
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  v += dpp<kDppRor8>(v);
  v += dpp<kDppRor4>(v);
  v += dpp<kDppXor2>(v);
  return v + dpp<kDppXor1>(v);
}

__device__ __forceinline__ float wave_sum(float v) {           // (distance 32 first)
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return half_wave_sum(__uint_as_float(r[0]) + __uint_as_float(r[1]));
}
// Four of them together, a's in lanes 0 .. 15, b's in 16 .. 31, c's in 32 .. 47, d's in 48 .. 63: a swap with another value in
// place of the value itself leaves the halves of two sums in one register.  The bits of wave_sum.
__device__ __forceinline__ float wave_sums4(float a, float b, float c, float d) {
  const auto ac = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(c), false, false);
  const auto bd = __builtin_amdgcn_permlane32_swap(__float_as_uint(b), __float_as_uint(d), false, false);
  const float x = __uint_as_float(ac[0]) + __uint_as_float(ac[1]), y = __uint_as_float(bd[0]) + __uint_as_float(bd[1]);
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(y), false, false);
  float v = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  v += dpp<kDppRor8>(v);
  v += dpp<kDppRor4>(v);
  v += dpp<kDppXor2>(v);
  return v + dpp<kDppXor1>(v);
}
__device__ __forceinline__ float wave_max(float v) {
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
  r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
  v = fmaxf(v, dpp<kDppRor8>(v));
  v = fmaxf(v, dpp<kDppRor4>(v));
  v = fmaxf(v, dpp<kDppXor2>(v));
  return fmaxf(v, dpp<kDppXor1>(v));
}

// Data handed from one work-group to another inside a kernel (split-K partial sums, attention chunk
// partials) is written and read with relaxed device-scope atomic accesses: they write through to / read
// from the level all XCDs share, so the hand-off needs no cache-wide write-back or invalidate; the
// writer only waits for its own stores (s_waitcnt) before it takes its ticket.
__device__ __forceinline__ void st_dev2(float* p, float a, float b) {
  const unsigned long long v = (unsigned long long)__float_as_uint(a) | ((unsigned long long)__float_as_uint(b) << 32);
  __hip_atomic_store(reinterpret_cast<unsigned long long*>(p), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_dev(float* p, float a) {
  __hip_atomic_store(p, a, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float ld_dev(const float* p) {
  return __hip_atomic_load(const_cast<float*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float2 ld_dev2(const float* p) {
  const unsigned long long v = __hip_atomic_load(reinterpret_cast<unsigned long long*>(const_cast<float*>(p)),
                                                 __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return make_float2(__uint_as_float((unsigned)v), __uint_as_float((unsigned)(v >> 32)));
}
// all of this work-group's stores have completed; then one thread takes the ticket.  Returns true in
// every thread of the work-group that arrived last of `expected`.
__device__ __forceinline__ bool last_arrival(int* counter, int expected, int* s_flag) {
  // The hand-off rests on two things the memory model does not promise for relaxed accesses: (1) a device-scope
  // write-through store is acknowledged only once it sits at the level all XCDs share, so "vmcnt == 0" means the
  // partial results are visible there; (2) the last arrival's loads of the others' results are issued after its
  // ticket.  (1) is the hardware's behaviour for sc1 stores; for (2) the signal fences keep the compiler from moving
  // memory accesses across the ticket in either direction (they emit no instruction).  Should either stop holding,
  // the fix is a release fence before and an acquire fence after the ticket (__atomic_thread_fence at agent scope):
  // correct by the model, at the price of an L2 write-back / invalidate per work-group.
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  if (threadIdx.x == 0)
    *s_flag = (__hip_atomic_fetch_add(counter, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == expected - 1) ? 1 : 0;
  __syncthreads();
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
  return *s_flag != 0;
}

// Row order of the re-laid-out matrix.  Output column n' of the GEMM is source row perm(n'):
//   kPermNone  : identity
//   kPermGateUp: W = [f gate rows; f up rows]; tile t holds gate rows 8t..8t+7 then up rows 8t..8t+7, so a SwiGLU
//                pair sits at columns (j, j+8) of one 16-column tile
//   kPermQKV   : W = [q; k; v] of d rows each, heads of hd rows; inside a q or k head tile t holds dims 8t..8t+7 then
//                hd/2+8t..hd/2+8t+7, so a rotation pair (e, e+hd/2) sits at columns (j, j+8) of one tile; v unchanged
__device__ __forceinline__ size_t perm_row(int nprime, int perm, int p0, int p1) {
  const int r = nprime & 15;
  if (perm == kPermGateUp) return (size_t)((r >> 3) ? p0 : 0) + (size_t)(nprime >> 4) * 8 + (r & 7);
  if (perm == kPermQKV) {
    const int d = p0, hd = p1;
    const int part = nprime / d, c = nprime - part * d;
    if (part == 2) return (size_t)nprime;
    const int h = c / hd, w = c - h * hd;
    return (size_t)part * d + (size_t)h * hd + (w >> 4) * 8 + (r & 7) + (r >> 3) * (hd >> 1);
  }
  return (size_t)nprime;
}

__device__ __forceinline__ size_t k_cache_off(int pos, int e, int hd) {   // element offset inside one head
  return ((size_t)((pos >> 4) * (hd >> 5) + (e >> 5)) * 64 + (pos & 15) + 16 * ((e & 31) >> 3)) * 8 + (e & 7);
}
__device__ __forceinline__ size_t v_cache_off(int pos, int e, int hd) {
  const int p32 = pos & 31, k16 = p32 & 15;
  return ((size_t)((pos >> 5) * (hd >> 4) + (e >> 4)) * 64 + (e & 15) + 16 * (k16 >> 2)) * 8 + (k16 & 3) + 4 * (p32 >> 4);
}

// The arithmetic of the epilogues lives in these helpers so that every GEMM variant produces the same bits.
__device__ __forceinline__ float swiglu(float g, float u) {
#pragma clang fp contract(off)
  return g / (1.0f + expf(-g)) * u;
}
// sum of squares of 4 adjacent residual values; a 16-column tile's partial is ((s0 + s1) + (s2 + s3)) of these
__device__ __forceinline__ float sumsq4(float x, float y, float z, float w) {
#pragma clang fp contract(off)
  return (x * x + y * y) + (z * z + w * w);
}
// the same partial with the 16 values in 16 adjacent lanes, one each
__device__ __forceinline__ float tile_sumsq(float x) {
#pragma clang fp contract(off)
  float s = x * x;
  s = s + dpp<kDppXor1>(s);
  s = s + dpp<kDppXor2>(s);                                      // sumsq4 of a quad's values in each of its lanes
  s = s + dpp<kDppHalfMirror>(s);
  return s + dpp<kDppRor8>(s);
}
__device__ __forceinline__ float2 rope_rotate(float a, float b, float2 cs) {
#pragma clang fp contract(off)
  return make_float2(a * cs.x - b * cs.y, b * cs.x + a * cs.y);
}
typedef __attribute__((ext_vector_type(8))) _Float16 f16x8;

__device__ __forceinline__ void split_half8(const float* v, f16x8& hi, f16x8& lo) {
#pragma clang fp contract(off)
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    float x = v[e];
    asm("" : "+v"(x));       // a product in front must be rounded to float first: its conversion would else become one
    const _Float16 h = (_Float16)x;   // instruction with a single rounding in some instantiations and not in others
    hi[e] = h;
    lo[e] = (_Float16)(x - (float)h);
  }
}

// e^x for the attention softmax of the half-cache kernels: the hardware's exp2 on x * log2(e) (two instructions, about
// 1 ulp; the library expf costs ten times that and a wave evaluates 16 per key block).  Arguments are <= 0 here.
__device__ __forceinline__ float exp_fast(float x) { return __builtin_amdgcn_exp2f(x * 1.44269504088896340736f); }

}  // namespace stairs
