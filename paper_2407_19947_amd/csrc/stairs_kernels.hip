// gfx950 kernels of the stairs library.  Written for wave64 / MFMA / LDS of CDNA4 only.
//
// Numerics contract shared by all kernels: activations, residual stream, logits and every
// accumulation are fp32; bf16 appears only as stored weights, stored keys/values and as the
// MFMA activation operand, which is fed as a bf16 high part plus a bf16 low part (two MFMAs
// per weight tile) so that the activation keeps ~16 mantissa bits.  Every reduction runs in
// an order that does not depend on the number of rows M of the launch, so a row of a stair
// batch gets bit-identical results to the same position computed alone (the property that
// makes the stair batch return what plain greedy decoding returns, paper abstract / Sec. 3.3).
#include "stairs_device.h"
#include <hip/hip_ext.h>

#include <math.h>
#include <stdio.h>
#include <stdlib.h>

#include <algorithm>
#include <mutex>
#include <vector>

namespace stairs {

// ---------------------------------------------------------------------------------------
// weight re-layout
// ---------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_swizzle_bf16(const uint16_t* __restrict__ W, uint4* __restrict__ Wsw,
                                                      int KT, int NTILES, size_t total, int K, int perm, int p0, int p1) {
  size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= total) return;
  // destination order: [k-slice][row tile][k-step inside the slice][lane]
  const int lane = (int)(idx & 63);
  const size_t tile_idx = idx >> 6;
  constexpr int SK = kSliceUnits * 8;                    // k-steps of a full slice
  const size_t full = (size_t)NTILES * SK;               // tiles per full slice
  const int s = (int)(tile_idx / full);
  const size_t rem = tile_idx - (size_t)s * full;
  const int ks = min(SK, KT - s * SK);                   // k-steps of this slice (the last one may be short)
  const int nt = (int)(rem / ks), kk = (int)(rem - (size_t)nt * ks);
  const int kt = s * SK + kk;
  const int r = lane & 15, g = lane >> 4;
  const size_t row = perm_row(nt * 16 + r, perm, p0, p1);
  Wsw[idx] = *reinterpret_cast<const uint4*>(W + row * K + kt * 32 + g * 8);
}

void launch_swizzle_bf16(const uint16_t* W, uint4* Wsw, int N, int K, int perm, int p0, int p1, hipStream_t st) {
  int KT = K / 32;
  size_t total = (size_t)(N / 16) * KT * 64;
  unsigned blocks = (unsigned)((total + 255) / 256);
  hipLaunchKernelGGL(k_swizzle_bf16, dim3(blocks), dim3(256), 0, st, W, Wsw, KT, N / 16, total, K, perm, p0, p1);
}

// ---------------------------------------------------------------------------------------
// skinny GEMM, bf16 weights, MFMA 16x16x32, with the projection's epilogue fused in
//   work-group = 4 waves; all four work on the same 512-wide k-slice (the X slice is staged once
//   in LDS as MFMA B fragments, high and low halves) and on 4*NT consecutive 16-row weight tiles.
//   The weight tile is the MFMA A operand and is loaded straight from HBM in operand order
//   (1 KiB per wave-load, fully coalesced); the X rows are the B operand.
//   Split-K: every work-group writes its partial sums; the one that arrives last at the column
//   group's counter adds the slices up in slice order (so the result does not depend on which
//   one that is) and applies the epilogue of the projection (ROLE).
//   What bounds it is a chain of round trips: activations, weights, partial sums, ticket, sums.  So all activations (of both
//   chunks) are requested at the start behind the first weight unit, two units stay requested at every time, and no weight
//   unit is requested under a condition.  That takes registers, and with two chunks a grid may have two to three work-groups
//   per CU (4096 x 12288: 768), which must all be resident: 3 waves per SIMD, held to 168 registers by fetching the second
//   chunk's gains when the first's are used up (residual projections have none).  Launches one after the other over several
//   layers' weights, us: one unit and one chunk's activations at a time (3 waves) / all at once (174 registers, 2 waves) / now:
//     2048 x 8192   9 / 16 rows  15.7 / 12.9 / 12.8    16.3 / 13.6 / 13.4      4096 x 11008  9 / 16  20.1 / 21.4 / 20.0    21.8 / 22.5 / 21.6
//     1024 x 16384  9 / 16 rows  14.3 / 12.3 / 12.0    14.9 / 13.0 / 12.6      4096 x 12288  9 / 16  21.1 / 24.0 / 21.2    22.6 / 25.9 / 22.7
//     3072 x 8192   9 / 16 rows  15.4 / 14.5 / 14.4    16.6 / 15.8 / 15.4      5120 x 13824  9 / 16  30.2 / 29.5 / 29.9    32.6 / 31.5 / 32.6
//   One chunk per work-group, before / now: 1024 x 16384 at 1 / 4 / 8 rows 12.2 / 11.3, 13.0 / 12.1, 14.3 / 13.5; 2048 x 8192 at 5 / 8
//   12.3 / 11.4, 12.7 / 11.8; 4096 x 9216 at 5 rows 18.1 / 18.5, where it is 2 % behind; 17..32 rows (two work-groups per CU by
//   their LDS) 1024 x 8192 12.5 / 11.5 .. 14.0 / 13.1.
// ---------------------------------------------------------------------------------------
// Sum of the split-K partial sums of one element (or 4 adjacent ones).  The order is fixed for every GEMM variant:
// the 512-wide k chunks are added in pairs, (c0 + c1), (c2 + c3), ..., and the pair sums one after the other.
// PAIRS = true: the S partials are single chunks (the pairs are formed here); false: they already are pair sums.
// The loads of up to 8 (slice_sum4: 16) partials are issued together (they are full round trips to the memory side).
template <bool PAIRS>
__device__ __forceinline__ float slice_sum(const float* partial, int S, size_t stride, size_t off) {
  float a = 0.f;
  for (int s0 = 0; s0 < S; s0 += 8) {
    float v[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = ld_dev(partial + (size_t)min(s0 + i, S - 1) * stride + off);
    if (PAIRS) {
#pragma unroll
      for (int i = 0; i < 8; i += 2)
        if (s0 + i < S) a += (s0 + i + 1 < S) ? (v[i] + v[i + 1]) : v[i];
    } else {
#pragma unroll
      for (int i = 0; i < 8; ++i) a += (s0 + i < S) ? v[i] : 0.f;
    }
  }
  return a;
}
template <bool PAIRS>
__device__ __forceinline__ float4 slice_sum4(const float* partial, int S, size_t stride, size_t off) {
  float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int s0 = 0; s0 < S; s0 += 16) {
    float2 p[16], q[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const float* src = partial + (size_t)min(s0 + i, S - 1) * stride + off;
      p[i] = ld_dev2(src);
      q[i] = ld_dev2(src + 2);
    }
    if (PAIRS) {
#pragma unroll
      for (int i = 0; i < 16; i += 2) {
        if (s0 + i < S) {
          const bool two = s0 + i + 1 < S;
          a.x += two ? (p[i].x + p[i + 1].x) : p[i].x; a.y += two ? (p[i].y + p[i + 1].y) : p[i].y;
          a.z += two ? (q[i].x + q[i + 1].x) : q[i].x; a.w += two ? (q[i].y + q[i + 1].y) : q[i].y;
        }
      }
    } else {
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const bool ok = s0 + i < S;
        a.x += ok ? p[i].x : 0.f; a.y += ok ? p[i].y : 0.f; a.z += ok ? q[i].x : 0.f; a.w += ok ? q[i].y : 0.f;
      }
    }
  }
  return a;
}

// Row m, columns col and col+8 of the permuted QKV output (col & 15 < 8): a rotation pair of q or k, or two
// plain values of v.  pos0 = position of row 0.
// index of the rotation entry of columns (col, col + 8) of row m (q and k parts; for the v part some valid index)
__device__ __forceinline__ int qkv_rope_index(int m, int col, int d, int hd) {
  const int c = col % d, w = c % hd;
  return m * 64 + (w >> 4) * 8 + (w & 7);
}
// p: the row's position (pos_of), cs: its rotation entry (epi.rope_cs[qkv_rope_index]); a caller may have loaded both early
__device__ __forceinline__ void qkv_pair_at(float a, float b, int m, int col, int d, const GemmEpi& epi, int p, float2 cs) {
  if (p < 0) return;
  const size_t slot_off = (size_t)slot_of(epi.pos, m) * epi.kv_slot_stride;
  const int hd = epi.hd, half = hd >> 1;
  const int part = col / d, c = col - part * d;
  const int h = c / hd, w = c - h * hd;
  if (part == 2) {
    _Float16* dst = epi.Vc + slot_off + (size_t)h * epi.cap * hd;
    store_kv(dst + v_cache_off(p, w, hd), a);
    store_kv(dst + v_cache_off(p, w + 8, hd), b);
    return;
  }
  const int e = (w >> 4) * 8 + (w & 7);
  const float2 r = rope_rotate(a, b, cs);
  if (part == 0) {
    epi.out[(size_t)m * d + h * hd + e] = r.x;
    epi.out[(size_t)m * d + h * hd + e + half] = r.y;
  } else {
    _Float16* dst = epi.Kc + slot_off + (size_t)h * epi.cap * hd;
    store_kv(dst + k_cache_off(p, e, hd), r.x);
    store_kv(dst + k_cache_off(p, e + half, hd), r.y);
  }
}
__device__ __forceinline__ void qkv_pair(float a, float b, int m, int col, int d, const GemmEpi& epi) {
  const int p = pos_of(epi.pos, m);
  if (p < 0) return;
  qkv_pair_at(a, b, m, col, d, epi, p, epi.rope_cs[qkv_rope_index(m, col, d, epi.hd)]);
}

// Epilogue of one column group [c0, c0+W) for all M rows, run by the 256 threads of one work-group.
// rs: the rows' 1/rms in LDS when the GEMM's input is normalised (the X fragments carry x * gain only), else null.
template <int ROLE, int W, bool PAIRS>
__device__ __forceinline__ void gemm_epilogue(const float* partial, int S, int M, int N, int c0, const GemmEpi& epi,
                                              const float* rs) {
  const int tid = threadIdx.x;
  const size_t stride = (size_t)M * N;
  if (ROLE == kRoleHead) {
    constexpr int PR = W / 4;
    for (int idx = tid; idx < M * PR; idx += 256) {
      const int m = idx / PR, col = c0 + (idx - m * PR) * 4;
      if (col < N) {
        float4 a = slice_sum4<PAIRS>(partial, S, stride, (size_t)m * N + col);
        if (rs) { const float r = rs[m]; a.x *= r; a.y *= r; a.z *= r; a.w *= r; }
        if (epi.act == kActRelu) a = make_float4(fmaxf(a.x, 0.f), fmaxf(a.y, 0.f), fmaxf(a.z, 0.f), fmaxf(a.w, 0.f));
        *reinterpret_cast<float4*>(epi.out + (size_t)m * N + col) = a;
        if (epi.frag_out) store_frag4(epi.frag_out, m, col, a, epi.frag_gain);
      }
    }
  } else if (ROLE == kRoleWo || ROLE == kRoleDown) {
    constexpr int PR = W / 4;                       // threads per row; 4 adjacent threads = one 16-column tile
    const int total = M * PR;
    for (int idx0 = 0; idx0 < total; idx0 += 256) {
      const int idx = idx0 + tid;
      const int m = idx / PR, col = c0 + (idx - m * PR) * 4;
      float ss = 0.f;
      if (idx < total && col < N) {
        float4* xp = reinterpret_cast<float4*>(epi.out + (size_t)m * N + col);
        const float4 r = *xp;                           // requested ahead of the partial sums
        __builtin_amdgcn_sched_barrier(0);
        float4 a = slice_sum4<PAIRS>(partial, S, stride, (size_t)m * N + col);
        if (rs) { const float q = rs[m]; a.x *= q; a.y *= q; a.z *= q; a.w *= q; }
        a.x += r.x; a.y += r.y; a.z += r.z; a.w += r.w;
        *xp = a;
        ss = sumsq4(a.x, a.y, a.z, a.w);
        if (epi.frag_out) store_frag4(epi.frag_out, m, col, a, epi.frag_gain);
      }
      ss += __shfl_xor(ss, 1);
      ss += __shfl_xor(ss, 2);
      if (idx < total && col < N && (idx & 3) == 0) epi.ssq_out[m * (N >> 4) + (col >> 4)] = ss;
    }
  } else if (ROLE == kRoleGateUp) {
    // tile t = 8 gate columns then the 8 up columns of features 8t..8t+7; a thread takes 4 features
    constexpr int PR = W / 8;
    const int f = N / 2;
    for (int idx = tid; idx < M * PR; idx += 256) {
      const int m = idx / PR, r = idx - m * PR;
      const int gcol = c0 + 16 * (r >> 1) + 4 * (r & 1);
      if (gcol < N) {
        float4 g = slice_sum4<PAIRS>(partial, S, stride, (size_t)m * N + gcol);
        float4 u = slice_sum4<PAIRS>(partial, S, stride, (size_t)m * N + gcol + 8);
        if (rs) {
          const float q = rs[m];
          g.x *= q; g.y *= q; g.z *= q; g.w *= q;
          u.x *= q; u.y *= q; u.z *= q; u.w *= q;
        }
        const float4 o = make_float4(swiglu(g.x, u.x), swiglu(g.y, u.y), swiglu(g.z, u.z), swiglu(g.w, u.w));
        *reinterpret_cast<float4*>(epi.out + (size_t)m * f + (gcol >> 4) * 8 + (gcol & 7)) = o;
        if (epi.frag_out) store_frag4(epi.frag_out, m, (gcol >> 4) * 8 + (gcol & 7), o, nullptr);
      }
    }
  } else {   // kRoleQKV: rotate q and k, append k and v to the cache
    constexpr int PR = W / 2;
    for (int idx = tid; idx < M * PR; idx += 256) {
      const int m = idx / PR, r = idx - m * PR;
      const int col = c0 + 16 * (r >> 3) + (r & 7);
      if (col < N) {
        float a = slice_sum<PAIRS>(partial, S, stride, (size_t)m * N + col);
        float b = slice_sum<PAIRS>(partial, S, stride, (size_t)m * N + col + 8);
        if (rs) { a *= rs[m]; b *= rs[m]; }
        qkv_pair(a, b, m, col, N / 3, epi);
      }
    }
  }
}

// 1/rms of the rows from the sum-of-squares partials: half a wave (32 lanes) per row; a lane adds partials
// p = lane, lane + 32, ... in that order, then the 32 lanes are combined by a butterfly.  Wave w takes the row
// pairs w, w+4, ... (PASSES of them: 8 * PASSES >= M).  The first 256 partials of every pass are requested before any
// of them is used, so a work-group pays one round trip for all its rows.
template <int PASSES>
__device__ __forceinline__ void rows_rstd(const RowNorm& nrm, int M, int K, float* s_rstd) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int half = lane >> 5, pl = lane & 31;
  float v[PASSES][8];
#pragma unroll
  for (int ps = 0; ps < PASSES; ++ps) {
    const int m = min(2 * wave + 8 * ps + half, M - 1);
    const float* sp = nrm.ssq_part + (size_t)m * nrm.ssq_n;
#pragma unroll
    for (int i = 0; i < 8; ++i) v[ps][i] = sp[min(pl + 32 * i, nrm.ssq_n - 1)];
  }
#pragma unroll
  for (int ps = 0; ps < PASSES; ++ps) {
    const int m = 2 * wave + 8 * ps + half;
    float ss = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) ss += (pl + 32 * i < nrm.ssq_n) ? v[ps][i] : 0.f;
    if (m < M) {
      for (int p0 = pl + 256; p0 < nrm.ssq_n; p0 += 256) {   // rows wider than 4096: the rest, 8 loads at a time
        float u[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) u[i] = (p0 + 32 * i < nrm.ssq_n) ? nrm.ssq_part[m * nrm.ssq_n + p0 + 32 * i] : 0.f;
#pragma unroll
        for (int i = 0; i < 8; ++i) ss += u[i];
      }
    }
#pragma unroll
    for (int off = 16; off >= 1; off >>= 1) ss += __shfl_xor(ss, off);
    if (pl == 0 && m < M) s_rstd[m] = 1.0f / sqrtf(ss / (float)K + nrm.eps);
  }
}

// 8 consecutive x of one row -> (x * gain) -> bf16 high part and the bf16 of the remainder
__device__ __forceinline__ void split_bf16x8(const float4& xa, const float4& xb, const float4& g0, const float4& g1,
                                             bool scale, uint4& hi, uint4& lo) {
  // the row's 1/rms is not applied here: it is a scalar per row and multiplies the finished sums in the epilogue, so
  // the conversion does not wait for the row statistics
  float v[8] = {xa.x, xa.y, xa.z, xa.w, xb.x, xb.y, xb.z, xb.w};
  if (scale) {
    v[0] = v[0] * g0.x; v[1] = v[1] * g0.y; v[2] = v[2] * g0.z; v[3] = v[3] * g0.w;
    v[4] = v[4] * g1.x; v[5] = v[5] * g1.y; v[6] = v[6] * g1.z; v[7] = v[7] * g1.w;
  }
  bf16_split2(v[0], v[1], hi.x, lo.x);
  bf16_split2(v[2], v[3], hi.y, lo.y);
  bf16_split2(v[4], v[5], hi.z, lo.z);
  bf16_split2(v[6], v[7], hi.w, lo.w);
}

typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));
// streaming load: the line is not kept in the caches on its way
__device__ __forceinline__ uint4 ld_nt(const uint4* p) {
  const u32x4_t v = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(p));
  return make_uint4(v.x, v.y, v.z, v.w);
}
// One 8 KiB weight unit of a wave (8 loads of 1 KiB) from a base that is the same in all lanes: lane l reads base + off + i * STEP *
// 16 bytes; what lies outside [base, base + span) is not fetched and reads as zeros.  STREAM (a template argument: a run-time
// choice between the two load forms cost the whole gain in the kernels' prologues): weights of a model far larger than the
// 256 MB memory-side cache are read once per forward and gain from the streaming hint (a bare 2 GB read: 6.2 -> 7.05
// TB/s); a model that about fits that cache is served from it forward after forward and must keep plain loads.
template <bool STREAM, int STEP>
__device__ __forceinline__ void load_unit_in(const uint4* base, uint32_t off, uint32_t span, uint4 (&wb)[8]) {
  const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint4*>(base), 0, span, 0x00027000);
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const u32x4_t v = __builtin_amdgcn_raw_buffer_load_b128(r, off + i * (STEP * 16), 0, STREAM ? 2 : 0);
    wb[i] = make_uint4(v.x, v.y, v.z, v.w);
  }
}

template <int CT, int NT, int ROLE, int SPW, bool STREAM>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(SPW == 2 ? 3 : 1, 8))) void k_gemm_bf16(const uint4* __restrict__ Wsw, const float* __restrict__ X,
                                                  const float* __restrict__ gain, float* partial, int K, int N, int ldx, int M,
                                                  const float* ssq_part, int ssq_n, float eps, GemmEpi epi) {
  constexpr bool NORMED = ROLE != kRoleWo && ROLE != kRoleDown;      // (the residual-writing projections' inputs are not)
  const RowNorm nrm{gain, ssq_part, ssq_n, eps};
  const bool scaled = NORMED && gain != nullptr;
  const int NTILES = N >> 4;
  // SPW = k chunks (512 wide) a work-group takes, one after the other through the same LDS buffer: 1, or 2 (then
  // it writes the sum of its two chunk sums, which halves the partial sums in memory; used for many rows)
  extern __shared__ uint4 lds[];   // [16 k-steps][CT][hi,lo][64 lanes]
  __shared__ int s_last;
  __shared__ float s_rstd[kMaxRows];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int sp = blockIdx.y, SG = gridDim.y;               // this work-group's partial slice, number of them
  const int units_total = K / kUnitK;
  // weights are stored slice-major: [k chunk][row tile][k-step][lane]; the four waves take adjacent tiles, so
  // the work-group reads contiguous runs of 64*NT KiB
  const int tile0 = blockIdx.x * 4 * NT + wave;          // this wave's tiles: tile0 + 4 t
  auto chunk_units = [&](int j) { return max(0, min(kSliceUnits, units_total - (sp * SPW + j) * kSliceUnits)); };
  // unit u of this wave's sequence: chunk j = u / (2 NT), tile t = (u / 2) % NT, unit ku = u % 2 of the chunk
  auto unit_ok = [&](int u) {
    const int j = u / (kSliceUnits * NT), t = (u / kSliceUnits) % NT, ku = u % kSliceUnits;
    return ku < chunk_units(j) && (tile0 + 4 * t) < NTILES;
  };
  // requested whatever the condition says (a request inside a condition would make every wait behind it one for all
  // requests); a unit that is not there is not fetched
  uint4 wb[2][8];
  auto request = [&](int u) {
    const int j = u / (kSliceUnits * NT), t = (u / kSliceUnits) % NT, ku = u % kSliceUnits;
    const uint4* p = Wsw + (size_t)(sp * SPW + j) * NTILES * (kSliceUnits * 8) * 64 + ((size_t)(tile0 + 4 * t) * chunk_units(j) + ku) * 8 * 64;
    load_unit_in<STREAM, 64>(p, lane * 16, unit_ok(u) ? 8 * 64 * 16 : 0, wb[u & 1]);
  };
  // first weight unit goes out before anything else: it depends on nothing
  request(0);

  // the X chunks: this thread's items are (row m, 8 consecutive k)
  constexpr int ITEMS = 4 * CT;          // 16*CT rows x 64 groups / 256 threads (a full chunk)
  float4 xa[SPW][ITEMS], xb[SPW][ITEMS];
#pragma unroll
  for (int j = 0; j < SPW; ++j) {
    const int units = chunk_units(j), kgs = max(units, 1) * 32, k0 = (sp * SPW + j) * kSliceUnits * kUnitK;
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
      const int w = tid + 256 * it;
      const int m = w / kgs, kg = w - m * kgs;
      xa[j][it] = make_float4(0.f, 0.f, 0.f, 0.f);
      xb[j][it] = xa[j][it];
      if (units > 0 && w < 16 * CT * kgs && m < M) {
        const float4* xp = reinterpret_cast<const float4*>(X + (size_t)m * ldx + k0 + kg * 8);
        xa[j][it] = xp[0];
        xb[j][it] = xp[1];
      }
    }
  }
  // the norm gain of this thread's k group (every item of a thread has kg = lane modulo the 64 or 32 groups of the chunk)
  float4 g0, g1;
  auto request_gain = [&](int j) {
    const int units = chunk_units(j), kgs = max(units, 1) * 32;
    if (scaled && units > 0) {
      const float4* gp = reinterpret_cast<const float4*>(gain + (sp * SPW + j) * kSliceUnits * kUnitK + (lane & (kgs - 1)) * 8);
      g0 = gp[0];
      g1 = gp[1];
    }
  };
  g0 = g1 = make_float4(1.f, 1.f, 1.f, 1.f);
  request_gain(0);
  __builtin_amdgcn_sched_barrier(0);
  request(1);
  __builtin_amdgcn_sched_barrier(0);

  f32x4 sum[NT][CT];
#pragma unroll
  for (int j = 0; j < SPW; ++j) {
    const int units = chunk_units(j), kgs = max(units, 1) * 32;    // groups of 8 k per row
    if (j > 0) __syncthreads();            // the previous chunk's fragments have been read
    // fp32 -> (x * gain) -> bf16 hi + lo, stored in B-fragment order
    if (units > 0) {
#pragma unroll
      for (int it = 0; it < ITEMS; ++it) {
        const int w = tid + 256 * it;                       // w < 16*CT*kgs is uniform per wave
        const int m = min(w / kgs, 16 * CT - 1), kg = w - (w / kgs) * kgs;
        if (w < 16 * CT * kgs) {
          const bool scale = scaled && m < M;
          uint4 hi, lo;
          split_bf16x8(xa[j][it], xb[j][it], g0, g1, scale, hi, lo);
          const int kt = kg >> 2, g = kg & 3, ct = m >> 4, jj = m & 15;
          const int base = ((kt * CT + ct) * 2) * 64 + g * 16 + jj;
          lds[base] = hi;
          lds[base + 64] = lo;
        }
      }
    }
    if (j + 1 < SPW) request_gain(j + 1);
    __syncthreads();

#pragma unroll
    for (int t = 0; t < NT; ++t) {
      f32x4 acc[CT];
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) acc[ct] = f32x4{0.f, 0.f, 0.f, 0.f};
      const bool tile_ok = (tile0 + 4 * t) < NTILES;
#pragma unroll
      for (int ku = 0; ku < kSliceUnits; ++ku) {
        const int u = (j * NT + t) * kSliceUnits + ku;
        if (ku < units && tile_ok) {
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            const bf16x8 a = __builtin_bit_cast(bf16x8, wb[u & 1][i]);
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) {
              const int base = (((ku * 8 + i) * CT + ct) * 2) * 64 + lane;
              const bf16x8 bh = __builtin_bit_cast(bf16x8, lds[base]);
              const bf16x8 bl = __builtin_bit_cast(bf16x8, lds[base + 64]);
              acc[ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, bh, acc[ct], 0, 0, 0);
              acc[ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, bl, acc[ct], 0, 0, 0);
            }
          }
        }
        // the unit after the next (it may belong to the next chunk) into this one's registers
        if (u + 2 < SPW * NT * kSliceUnits) {
          request(u + 2);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      // chunk sums of a pair are added once, first + second
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) {
        if (j == 0) {
          sum[t][ct] = acc[ct];
        } else if (units > 0) {
          sum[t][ct][0] += acc[ct][0]; sum[t][ct][1] += acc[ct][1];
          sum[t][ct][2] += acc[ct][2]; sum[t][ct][3] += acc[ct][3];
        }
      }
    }
  }

#pragma unroll
  for (int t = 0; t < NT; ++t) {
    if ((tile0 + 4 * t) < NTILES) {
      const int n = (tile0 + 4 * t) * 16 + 4 * (lane >> 4);
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) {
        const int m = ct * 16 + (lane & 15);
        if (m < M) {
          float* dst = partial + ((size_t)sp * M + m) * N + n;
          st_dev2(dst, sum[t][ct][0], sum[t][ct][1]);
          st_dev2(dst + 2, sum[t][ct][2], sum[t][ct][3]);
        }
      }
    }
  }

  // split-K hand-off: the partial sums are out, take a ticket; the last arrival finishes the group
  if (!last_arrival(&epi.counters[blockIdx.x], SG, &s_last)) return;
  // the rows' 1/rms is needed here only: the work-group that finishes a column group forms it
  const bool normed = scaled && ssq_part;
  if (normed) {
    rows_rstd<2 * CT>(nrm, M, K, s_rstd);
    __syncthreads();
  }
  gemm_epilogue<ROLE, 64 * NT, SPW == 1>(partial, SG, M, N, blockIdx.x * 64 * NT, epi, normed ? s_rstd : nullptr);
  if (tid == 0) epi.counters[blockIdx.x] = 0;   // ready for the next launch on this stream
}

// ---------------------------------------------------------------------------------------
// The same GEMM for R <= 7 rows when the whole X block fits in LDS (K * R * 4 bytes): one work-group owns ONE
// 16-row weight tile over the whole k range, its waves split the 512-wide k chunks between them, the chunk
// sums meet in LDS and the epilogue follows in the same work-group.  No partial sums in memory and no hand-off
// between work-groups, so the tail of one work-group overlaps the streaming of the others.  Chunk boundaries,
// the MFMA order inside a chunk and the order in which the chunk sums are added are those of the split-K
// kernel: both give the same bits for a row.
//   What bounds it: large matrices, the weights' way from memory; small ones the chain launch (1.6 us for an empty kernel
//   in a graph, 1.9 with a load and a store) - arguments - x and weights - conversion - arithmetic - epilogue, i.e. round
//   trips and the number of instructions one wave runs one after the other (4 cycles each).  So what the first
//   loads need comes in registers (the arguments in front of the structure: KERNEL_ARGS_IN_REGISTERS in binding.py; unembedding of one
//   row and small layers 0.2 .. 0.3 us a launch), the rest in one round trip (want), a thread stages no more of x than there is for it (GP, Q), waves without a k chunk fetch no weights,
//   the row statistics are summed beside the arithmetic by the waves with the least of it, everything that depends on the
//   tile alone is scalar, and sums over lanes stay out of the LDS unit.  Layers of five launches in a graph, 200 keys,
//   before / now, us: d 768 (ffn 3072) 1 / 3 / 5 rows 23.4 / 26.0 / 27.3 -> 21.7 / 22.6 / 24.5, d 1024 (ffn 4096) 23.9 /
//   26.5 / 28.3 -> 22.0 / 22.9 / 24.7, d 2048 (ffn 8192) 1 / 3 rows 40.5 / 43.8 -> 39.9 / 42.2; unembedding of 32000 x 768
//   10.9 / 14.1 / 11.7 -> 9.6 / 9.7 / 10.1; d 4096 as before.
//   LDS: X high parts [K/8][R] uint4, X low parts [K/8][R] uint4, chunk sums float [chunks][R][16]
// ---------------------------------------------------------------------------------------
// Sum of one element's chunk sums held in LDS (stride floats apart), in the order of slice_sum<true>: pairs first.
// 8 chunks are read before any is used.
__device__ __forceinline__ float lds_chunk_sum(const float* base, int stride, int nchunks) {
  float a = 0.f;
  for (int c0 = 0; c0 < nchunks; c0 += 8) {
    float v[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = base[min(c0 + i, nchunks - 1) * stride];
#pragma unroll
    for (int i = 0; i < 8; i += 2)
      if (c0 + i < nchunks) a += (c0 + i + 1 < nchunks) ? (v[i] + v[i + 1]) : v[i];
  }
  return a;
}

// (value, index) pairs: the larger value, of equal ones the lower index
__device__ __forceinline__ void argmax_take(float& best, int& bi, float ov, int oi) {
  if (ov > best || (ov == best && oi < bi)) { best = ov; bi = oi; }
}
template <int CTRL>
__device__ __forceinline__ void argmax_dpp(float& best, int& bi) {
  argmax_take(best, bi, dpp<CTRL>(best), __builtin_amdgcn_update_dpp(0, bi, CTRL, 0xF, 0xF, true));
}
__device__ __forceinline__ void argmax_swap(float& best, int& bi, bool far) {      // lanes at distance 32 or 16
  const uint32_t b = __float_as_uint(best), i = (uint32_t)bi;
  const auto rb = far ? __builtin_amdgcn_permlane32_swap(b, b, false, false) : __builtin_amdgcn_permlane16_swap(b, b, false, false);
  const auto ri = far ? __builtin_amdgcn_permlane32_swap(i, i, false, false) : __builtin_amdgcn_permlane16_swap(i, i, false, false);
  const bool second = threadIdx.x & (far ? 32 : 16);     // (this lane's own value is in the other half of the pair)
  argmax_take(best, bi, __uint_as_float(second ? rb[0] : rb[1]), (int)(second ? ri[0] : ri[1]));
}

// what a launch of k_gemm_bf16_rows takes behind its leading arguments (one structure: every argument more costs the host 0.1 us a launch)
struct RowsEpi : GemmEpi {
  float2* cand;
};
// ROWMAJOR: W as the caller has it, [N, K] row-major: lane r + 16 g reads row 16 tile + r, k 32 kt + 8 g .. + 8, the very
// operand the tile layout holds in one piece (a wave's load is then 16 runs of 64 bytes; for a matrix used once that is
// far less than laying it out first).
// GP, Q: k groups (of 8 k) a thread stages in its first pass, threads that share the rows of a k group (covers
// K <= 8 * 64 * NW * GP / Q: rows_kernel).  WALK: a work-group takes several tiles; else its only one is blockIdx.x.
template <int R, int ROLE, int NW, int GP, int Q, bool WALK, bool STREAM, bool ROWMAJOR = false>
__global__ __launch_bounds__(64 * NW) void k_gemm_bf16_rows(const uint4* __restrict__ Wsw, const float* __restrict__ X,
                                                            const float* __restrict__ gain, const float* __restrict__ ssq_part,
                                                            int K, int N, int ldx, int ssq_n, float* out, float eps, RowsEpi epi) {
  constexpr int NTH = 64 * NW, NG = NTH / Q, RP = (R + Q - 1) / Q;
  constexpr bool NORMED = ROLE != kRoleWo && ROLE != kRoleDown;      // (the residual-writing projections' inputs are not)
  extern __shared__ uint4 lds[];
  __shared__ float s_rstd[8];
  const int NTILES = N >> 4;
  if (ROLE == kRoleQKV) { want(epi.rope_cs); want(epi.pos.base); want(epi.pos.offset); want(epi.pos.rps); want(epi.Kc); want(epi.Vc); want(epi.cap); want(epi.hd); }
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // a work-group takes the tiles blockIdx.x, blockIdx.x + gridDim.x, ...: the X block is staged once for all of them
  int cur_tile = blockIdx.x;
  const int KG = K >> 3;                                   // groups of 8 k per row
  const int units_total = (unsigned)K / kUnitK;
  const int nchunks = (unsigned)(units_total + kSliceUnits - 1) / kSliceUnits;
  const int cpw = (unsigned)(nchunks + NW - 1) / NW;       // chunks per wave
  const int c_begin = min(wave * cpw, nchunks), c_end = min(nchunks, c_begin + cpw);
  const int nu = min(units_total, c_end * kSliceUnits) - c_begin * kSliceUnits;   // this wave's units (<= 0: none)

  // address of unit u of this wave: chunk c_begin + u/2 (= split-K slice), unit u%2 inside it (the same in all lanes)
  auto unit_ptr = [&](int u) {
    const int c = c_begin + (u >> 1);
    if (ROWMAJOR) return Wsw + (size_t)cur_tile * 16 * (K >> 3) + (c * kSliceUnits + (u & 1)) * 32;
    const int units_c = min(kSliceUnits, units_total - c * kSliceUnits);
    return Wsw + (size_t)c * NTILES * (kSliceUnits * 8) * 64 + ((size_t)cur_tile * units_c + (u & 1)) * 8 * 64;
  };
  const uint32_t lane_off = ROWMAJOR ? (uint32_t)((lane & 15) * (K >> 3) + (lane >> 4)) * 16u : (uint32_t)lane * 16u;
  // bytes a unit spans from its first lane's on; 0 for a unit this wave does not have: its loads then fetch nothing
  const uint32_t unit_span = ROWMAJOR ? (uint32_t)(15 * (K >> 3) + 32) * 16u : 8u * 1024u;

  // first pass over the X block: a thread takes RP rows of k group kg (the gain is per k, so it is fetched once).  These
  // loads (x, gain, row statistics) go out before the weights, so they are not queued behind them.
  const bool scale = NORMED && gain != nullptr;
  float4 xa[GP][RP], xb[GP][RP], ga[GP], gb[GP];
  const int kg0 = tid & (NG - 1), m0 = tid / NG;           // this thread's first k group and first row (rows m0, m0 + Q, ...)
#pragma unroll
  for (int j = 0; j < GP; ++j) {
    ga[j] = make_float4(1.f, 1.f, 1.f, 1.f);
    gb[j] = ga[j];
    // no condition around the loads (a k group past the end re-reads the last one and is dropped later): the
    // compiler can then count them exactly and later waits do not have to cover the weight loads as well
    const uint32_t k4 = (uint32_t)min(kg0 + NG * j, KG - 1) * 32u;
    if (scale) {
      ga[j] = ld_at<float4>(gain, k4);
      gb[j] = ld_at<float4>(gain, k4 + 16u);
    }
#pragma unroll
    for (int i = 0; i < RP; ++i) {
      const uint32_t off = (uint32_t)min(m0 + Q * i, R - 1) * (uint32_t)ldx * 4u + k4;
      xa[j][i] = ld_at<float4>(X, off);
      xb[j][i] = ld_at<float4>(X, off + 16u);
    }
  }
  // row statistics: half a wave per row, the last waves first (with a short k those have no weights to multiply).  The
  // first 256 partials of the row are requested here (indices clamped, values masked later); they are added up beside the
  // arithmetic, in the order rows_rstd uses: the 1/rms multiplies the finished sums in the epilogue.
  const bool has_stats = scale && ssq_part;
  const int st_row = 2 * NW - 1 - (tid >> 5), st_pl = lane & 31;
  float sv[8];
  if (has_stats) {
    const uint32_t row = (uint32_t)min(st_row, R - 1) * ssq_n;
#pragma unroll
    for (int i = 0; i < 2; ++i) sv[i] = ld_at<float>(ssq_part, (row + min(st_pl + 32 * i, ssq_n - 1)) * 4u);
    if (ssq_n > 64) {
#pragma unroll
      for (int i = 2; i < 8; ++i) sv[i] = ld_at<float>(ssq_part, (row + min(st_pl + 32 * i, ssq_n - 1)) * 4u);
    }
  }

  // what the epilogue reads -- old x (residual-writing roles), the row's position, the rotation entry: requested ahead of the
  // arithmetic (behind it they were a round trip of their own at the end of every launch), by all threads (a condition
  // around a load would make the waits for what was requested before it cover the weights as well)
  const int half = epi.hd >> 1, hd_log = 31 - __builtin_clz(epi.hd), part_tiles = (unsigned)NTILES / 3u;
  float x_old = 0.f;
  int q_pos = 0;
  float2 q_cs = make_float2(1.f, 0.f);
  auto request_operands = [&](int tile) {
    if (!NORMED) x_old = ld_at<float>(out, ((uint32_t)min(tid >> 4, R - 1) * N + tile * 16 + (tid & 15)) * 4u);
    if (ROLE == kRoleQKV) {                                // (v tiles: some valid entry)
      const int c = (tile - (tile >= part_tiles ? part_tiles : 0) - (tile >= 2 * part_tiles ? part_tiles : 0)) * 16;
      q_cs = ld_at<float2>(epi.rope_cs, (uint32_t)(min(tid >> 3, R - 1) * 64 + ((c & (epi.hd - 1)) >> 4) * 8 + (tid & 7)) * 8u);
    }
  };
  if (ROLE == kRoleQKV) q_pos = pos_of(epi.pos, min(tid >> 3, R - 1));
  if (!WALK) request_operands(cur_tile);
  // the wave's first two weight units, again without conditions: a unit the wave does not have (short K) is requested with
  // an empty range, which fetches nothing (as repeated reads of a valid unit they were most of a short-K launch's traffic:
  // 6 of 8 waves at K = 768)
  uint4 wb0[8], wb1[8];
  // (a macro, not a lambda: register arrays a lambda captures by reference end up in scratch memory)
#define STAIRS_FIRST_UNITS()                                                                                              \
  do {                                                                                                                    \
    load_unit_in<STREAM, ROWMAJOR ? 4 : 64>(nu > 0 ? unit_ptr(0) : Wsw, lane_off, nu > 0 ? unit_span : 0u, wb0);          \
    load_unit_in<STREAM, ROWMAJOR ? 4 : 64>(nu > 1 ? unit_ptr(1) : Wsw, lane_off, nu > 1 ? unit_span : 0u, wb1);          \
  } while (0)
  STAIRS_FIRST_UNITS();
  uint4* xhi = lds;
  uint4* xlo = lds + KG * R;
  float* csum = reinterpret_cast<float*>(lds + 2 * KG * R); // [chunk][R][16]
#pragma unroll
  for (int j = 0; j < GP; ++j) {
    const int kg = kg0 + NG * j;
    if (kg < KG) {
#pragma unroll
      for (int i = 0; i < RP; ++i) {
        const int m = m0 + Q * i;
        if (R % Q && m >= R) continue;
        uint4 hi, lo;
        split_bf16x8(xa[j][i], xb[j][i], ga[j], gb[j], scale, hi, lo);
        xhi[kg * R + m] = hi;
        xlo[kg * R + m] = lo;
      }
    }
  }
  // further passes (longer K): same thing, loads and conversion back to back
  if (Q == 1 && (GP > 1 || NW > 4))
    for (int kg = NTH * GP + tid; kg < KG; kg += NTH) {
      float4 g0 = make_float4(1.f, 1.f, 1.f, 1.f), g1 = g0;
      if (scale) {
        g0 = ld_at<float4>(gain, kg * 32u);
        g1 = ld_at<float4>(gain, kg * 32u + 16u);
      }
#pragma unroll
      for (int m = 0; m < R; ++m) {
        const uint32_t off = (uint32_t)m * (uint32_t)ldx * 4u + kg * 32u;
        uint4 hi, lo;
        split_bf16x8(ld_at<float4>(X, off), ld_at<float4>(X, off + 16u), g0, g1, scale, hi, lo);
        xhi[kg * R + m] = hi;
        xlo[kg * R + m] = lo;
      }
    }
  auto row_stats = [&]() {
    if (has_stats && wave >= NW - (R + 1) / 2) {           // (whole waves)
      float ss = 0.f;
#pragma unroll
      for (int i = 0; i < 2; ++i) ss += (st_pl + 32 * i < ssq_n) ? sv[i] : 0.f;
      if (ssq_n > 64) {
#pragma unroll
        for (int i = 2; i < 8; ++i) ss += (st_pl + 32 * i < ssq_n) ? sv[i] : 0.f;
        if (ssq_n > 256 && st_row < R) {
          for (int p0 = st_pl + 256; p0 < ssq_n; p0 += 256) {
            float v[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] = (p0 + 32 * i < ssq_n) ? ssq_part[st_row * ssq_n + p0 + 32 * i] : 0.f;
#pragma unroll
            for (int i = 0; i < 8; ++i) ss += v[i];
          }
        }
      }
      ss = half_wave_sum(ss);
      if (st_pl == 0 && st_row < R) s_rstd[st_row] = 1.0f / sqrtf(ss / (float)K + eps);
    }
  };
  // (long k: in front of the barrier, every wave has weights to multiply behind it)
  constexpr bool kStatsFirst = GP > 1;
  if (kStatsFirst) row_stats();
  __syncthreads();
  if (!kStatsFirst) row_stats();

  // B fragment of lane l at k-step kt: row (l & 15) of X (lanes of rows >= R take row 0; their columns of the
  // result are never read), k group kt*4 + (l >> 4)
  const int bofs = (lane >> 4) * R + (((lane & 15) < R) ? (lane & 15) : 0);
  auto mfma_unit = [&](const uint4 (&wb)[8], int u, f32x4& acc) {
    const int kt0 = ((c_begin + (u >> 1)) * kSliceUnits + (u & 1)) * 8;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const bf16x8 a = __builtin_bit_cast(bf16x8, wb[i]);
      const int idx = (kt0 + i) * 4 * R + bofs;
      const bf16x8 bh = __builtin_bit_cast(bf16x8, xhi[idx]);
      const bf16x8 bl = __builtin_bit_cast(bf16x8, xlo[idx]);
      acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, bh, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, bl, acc, 0, 0, 0);
    }
  };
  // sum of one element's chunk sums (lds_chunk_sum; one or two chunks without its loop)
  auto chunk_sum = [&](int m, int n) {
    const float* src = csum + (m << 4) + n;
    if (nchunks == 1) return 0.f + src[0];
    if (nchunks == 2) return 0.f + (src[0] + src[R * 16]);
    return lds_chunk_sum(src, R * 16, nchunks);
  };
  for (;;) {
  const int tile = cur_tile;
  if (WALK) request_operands(tile);
  for (int u = 0; u < nu; u += 2) {                        // one chunk per pass
    f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
    mfma_unit(wb0, u, acc);
    if (u + 2 < nu) load_unit_in<STREAM, ROWMAJOR ? 4 : 64>(unit_ptr(u + 2), lane_off, unit_span, wb0);
    if (u + 1 < nu) {
      mfma_unit(wb1, u + 1, acc);
      if (u + 3 < nu) load_unit_in<STREAM, ROWMAJOR ? 4 : 64>(unit_ptr(u + 3), lane_off, unit_span, wb1);
    }
    const int m = lane & 15;
    if (m < R) {
      float* dst = csum + (((c_begin + (u >> 1)) * R + m) << 4) + 4 * (lane >> 4);
      dst[0] = acc[0]; dst[1] = acc[1]; dst[2] = acc[2]; dst[3] = acc[3];
    }
  }
  __builtin_amdgcn_sched_barrier(0);
  // the next tile's first units are requested ahead of the epilogue, which loads nothing from memory
  const int next_tile = tile + (int)gridDim.x;
  if (WALK && next_tile < NTILES) {
    cur_tile = next_tile;
    STAIRS_FIRST_UNITS();
  }
  __syncthreads();

  if (ROLE == kRoleWo || ROLE == kRoleDown) {
    // a thread takes one element of the tile; the 16 squares of a row, in 16 adjacent lanes, are added up in the order of
    // the split-K kernel's epilogue
    if (tid < R * 16) {
      const int m = tid >> 4, n = tid & 15;
      const float a = chunk_sum(m, n) + x_old;
      out[(size_t)m * N + tile * 16 + n] = a;
      const float sq = tile_sumsq(a);
      if (n == 0) epi.ssq_out[m * (N >> 4) + tile] = sq;
      // more than 4 rows: the next projection may take the kernel that reads activation fragments
      if (R > 4 && epi.frag_out) {
        const float4 v = make_float4(dpp<kDppQuad0>(a), dpp<kDppQuad1>(a), dpp<kDppQuad2>(a), dpp<kDppQuad3>(a));
        if ((n & 3) == 0) store_frag4(epi.frag_out, m, tile * 16 + n, v, epi.frag_gain);
      }
    }
  } else if (tid < R * 8) {                                // a thread takes row m, columns j and j+8 of the tile
    const int m = tid >> 3, j = tid & 7;
    float a = chunk_sum(m, j);
    float b = chunk_sum(m, j + 8);
    if (has_stats) {
      a *= s_rstd[m];
      b *= s_rstd[m];
    }
    const int col = tile * 16 + j;
    // (more than 4 rows: also the result's activation fragments -- the four threads of columns 4q .. 4q+3 are a quad of
    // wave 0, which holds all R * 8 <= 64 threads of this branch)
    if (ROLE == kRoleHead) {
      const bool relu = epi.act == kActRelu;
      if (relu) {
        a = fmaxf(a, 0.f);
        b = fmaxf(b, 0.f);
      }
      out[(size_t)m * N + col] = a;
      out[(size_t)m * N + col + 8] = b;
      if (!ROWMAJOR && epi.cand) {                         // the tile's largest value, for k_decide (a NaN is none)
        float v = fmaxf(a, -INFINITY);
        int ix = col;
        if (b > v) { v = b; ix = col + 8; }
        argmax_dpp<kDppXor1>(v, ix);
        argmax_dpp<kDppXor2>(v, ix);
        argmax_dpp<kDppHalfMirror>(v, ix);
        if (j == 0) epi.cand[(size_t)m * NTILES + tile] = make_float2(v, __int_as_float(ix));
      }
      if (R > 4 && epi.frag_out) {
        const float4 va = make_float4(dpp<kDppQuad0>(a), dpp<kDppQuad1>(a), dpp<kDppQuad2>(a), dpp<kDppQuad3>(a));
        const float4 vb = make_float4(dpp<kDppQuad0>(b), dpp<kDppQuad1>(b), dpp<kDppQuad2>(b), dpp<kDppQuad3>(b));
        if ((j & 3) == 0) {
          store_frag4(epi.frag_out, m, col, va, epi.frag_gain);
          store_frag4(epi.frag_out, m, col + 8, vb, epi.frag_gain);
        }
      }
    } else if (ROLE == kRoleGateUp) {
      const float o = swiglu(a, b);
      out[(size_t)m * (N >> 1) + tile * 8 + j] = o;
      if (R > 4 && epi.frag_out) {
        const float4 vo = make_float4(dpp<kDppQuad0>(o), dpp<kDppQuad1>(o), dpp<kDppQuad2>(o), dpp<kDppQuad3>(o));
        if ((j & 3) == 0) store_frag4(epi.frag_out, m, tile * 8 + j, vo, nullptr);
      }
    } else if (q_pos >= 0) {
      // qkv_pair_at with everything that depends on the tile alone in scalar registers
      const int part = (tile >= part_tiles) + (tile >= 2 * part_tiles), c = (tile - part * part_tiles) * 16;
      const int h = c >> hd_log, w = c & (epi.hd - 1);
      const size_t head = (size_t)slot_of(epi.pos, m) * epi.kv_slot_stride + (size_t)h * epi.cap * epi.hd;
      if (part == 2) {
        store_kv(epi.Vc + head + v_cache_off(q_pos, w + j, epi.hd), a);
        store_kv(epi.Vc + head + v_cache_off(q_pos, w + j + 8, epi.hd), b);
      } else {
        const int e = (w >> 4) * 8 + j;
        const float2 r = rope_rotate(a, b, q_cs);
        if (part == 0) {
          float* dst = out + (size_t)m * (part_tiles * 16) + h * epi.hd + e;
          dst[0] = r.x;
          dst[half] = r.y;
        } else {
          store_kv(epi.Kc + head + k_cache_off(q_pos, e, epi.hd), r.x);
          store_kv(epi.Kc + head + k_cache_off(q_pos, e + half, epi.hd), r.y);
        }
      }
    }
  }
  if (!WALK || next_tile >= NTILES) break;
  __syncthreads();                                         // the chunk sums are free for the next tile
  }
#undef STAIRS_FIRST_UNITS
}

// ---------------------------------------------------------------------------------------
// The hand-off-free GEMM for more than 4 rows (M <= 32): a work-group owns NT adjacent 16-row weight tiles over the
// WHOLE k range, its waves split the 512-wide k chunks between them, and a wave feeds every k-step's weight tiles
// with the activation fragments their producer left in memory (see frag_off): per k-step NT coalesced 1 KiB reads of
// weights (HBM) and 2 CT of fragments (L2), no conversion, nothing staged in LDS, no barrier before the first MFMA.
// A fragment is shared by the wave's NT tiles.  The chunk sums meet in LDS as in k_gemm_bf16_rows and the epilogue
// runs in the same work-group: no partial sums in memory, no ticket.  Chunk boundaries, the MFMA order inside a chunk
// and the order of the chunk sums are those of the other two kernels: all three give the same bits for a row.
//   CT = 16-row column tiles (rows of x) per MFMA pass: 1 (M <= 16) or 2; DEPTH = k-steps whose loads are in flight
//   LDS: chunk sums float [chunks][M][NT * 16]
// The epilogue can leave the fragments of ITS result for the next projection (epi.frag_out, with epi.frag_gain
// folded in): residual stream and SwiGLU output.
// ---------------------------------------------------------------------------------------
// 1/rms of the rows for a work-group of any size: half a wave per row, the additions in the order of rows_rstd
__device__ __forceinline__ void rows_rstd_any(const RowNorm& nrm, int M, int K, float* s_rstd) {
  // (the last waves first: with a short k the first ones have the k chunks and the others nothing to wait for)
  const int pl = threadIdx.x & 31, nhw = blockDim.x >> 5, hw = nhw - 1 - (threadIdx.x >> 5);
  for (int m = hw; m < M; m += nhw) {
    const float* sp = nrm.ssq_part + (size_t)m * nrm.ssq_n;
    float v[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = sp[min(pl + 32 * i, nrm.ssq_n - 1)];
    float ss = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) ss += (pl + 32 * i < nrm.ssq_n) ? v[i] : 0.f;
    for (int p0 = pl + 256; p0 < nrm.ssq_n; p0 += 256) {
      float u[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) u[i] = (p0 + 32 * i < nrm.ssq_n) ? sp[p0 + 32 * i] : 0.f;
#pragma unroll
      for (int i = 0; i < 8; ++i) ss += u[i];
    }
#pragma unroll
    for (int off = 16; off >= 1; off >>= 1) ss += __shfl_xor(ss, off);
    if (pl == 0) s_rstd[m] = 1.0f / sqrtf(ss / (float)K + nrm.eps);
  }
}

// The epilogue of gemm_epilogue with the chunk sums in LDS ([chunk][M][W] floats) instead of partial sums in memory;
// run by all threads of the work-group.  The additions are those of slice_sum<true>: chunk pairs first.
template <int ROLE, int W>
__device__ __forceinline__ void gemm_epilogue_lds(const float* csum, int nchunks, int M, int N, int c0, const GemmEpi& epi,
                                                  const float* rs, float4 x_first, int p_first, float2 cs_first) {
  const int tid = threadIdx.x, nth = blockDim.x;
  const int cstride = M * W;
  auto sum4 = [&](int m, int lc) {
    const float* src = csum + m * W + lc;
    float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int c = 0; c < nchunks; c += 2) {
      const float4 p = *reinterpret_cast<const float4*>(src + c * cstride);
      if (c + 1 < nchunks) {
        const float4 q = *reinterpret_cast<const float4*>(src + (c + 1) * cstride);
        a.x += p.x + q.x; a.y += p.y + q.y; a.z += p.z + q.z; a.w += p.w + q.w;
      } else {
        a.x += p.x; a.y += p.y; a.z += p.z; a.w += p.w;
      }
    }
    return a;
  };
  auto sum1 = [&](int m, int lc) {
    const float* src = csum + m * W + lc;
    float a = 0.f;
    for (int c = 0; c < nchunks; c += 2) a += (c + 1 < nchunks) ? (src[c * cstride] + src[(c + 1) * cstride]) : src[c * cstride];
    return a;
  };
  if (ROLE == kRoleHead) {
    constexpr int PR = W / 4;
    for (int idx = tid; idx < M * PR; idx += nth) {
      const int m = idx / PR, lc = (idx - m * PR) * 4, col = c0 + lc;
      if (col < N) {
        float4 a = sum4(m, lc);
        if (rs) { const float r = rs[m]; a.x *= r; a.y *= r; a.z *= r; a.w *= r; }
        if (epi.act == kActRelu) a = make_float4(fmaxf(a.x, 0.f), fmaxf(a.y, 0.f), fmaxf(a.z, 0.f), fmaxf(a.w, 0.f));
        *reinterpret_cast<float4*>(epi.out + (size_t)m * N + col) = a;
        if (epi.frag_out) store_frag4(epi.frag_out, m, col, a, epi.frag_gain);
      }
    }
  } else if (ROLE == kRoleWo || ROLE == kRoleDown) {
    constexpr int PR = W / 4;                       // 4 adjacent threads = one 16-column tile
    const int total = M * PR;
    for (int idx0 = 0; idx0 < total; idx0 += nth) {
      const int idx = idx0 + tid;
      const int m = idx / PR, lc = (idx - m * PR) * 4, col = c0 + lc;
      float ss = 0.f;
      if (idx < total && col < N) {
        float4 a = sum4(m, lc);
        if (rs) { const float q = rs[m]; a.x *= q; a.y *= q; a.z *= q; a.w *= q; }
        float4* xp = reinterpret_cast<float4*>(epi.out + (size_t)m * N + col);
        const float4 r = idx0 == 0 ? x_first : *xp;   // (the first pass' were requested ahead of the k loop)
        a.x += r.x; a.y += r.y; a.z += r.z; a.w += r.w;
        *xp = a;
        ss = sumsq4(a.x, a.y, a.z, a.w);
        if (epi.frag_out) store_frag4(epi.frag_out, m, col, a, epi.frag_gain);
      }
      ss += __shfl_xor(ss, 1);
      ss += __shfl_xor(ss, 2);
      if (idx < total && col < N && (idx & 3) == 0) epi.ssq_out[m * (N >> 4) + (col >> 4)] = ss;
    }
  } else if (ROLE == kRoleGateUp) {
    constexpr int PR = W / 8;
    const int f = N / 2;
    for (int idx = tid; idx < M * PR; idx += nth) {
      const int m = idx / PR, r = idx - m * PR;
      const int lc = 16 * (r >> 1) + 4 * (r & 1), gcol = c0 + lc;
      if (gcol < N) {
        float4 g = sum4(m, lc);
        float4 u = sum4(m, lc + 8);
        if (rs) {
          const float q = rs[m];
          g.x *= q; g.y *= q; g.z *= q; g.w *= q;
          u.x *= q; u.y *= q; u.z *= q; u.w *= q;
        }
        const float4 o = make_float4(swiglu(g.x, u.x), swiglu(g.y, u.y), swiglu(g.z, u.z), swiglu(g.w, u.w));
        *reinterpret_cast<float4*>(epi.out + (size_t)m * f + (gcol >> 4) * 8 + (gcol & 7)) = o;
        if (epi.frag_out) store_frag4(epi.frag_out, m, (gcol >> 4) * 8 + (gcol & 7), o, nullptr);
      }
    }
  } else {   // kRoleQKV
    constexpr int PR = W / 2;
    for (int idx = tid; idx < M * PR; idx += nth) {
      const int m = idx / PR, r = idx - m * PR;
      const int lc = 16 * (r >> 3) + (r & 7), col = c0 + lc;
      if (col < N) {
        float a = sum1(m, lc);
        float b = sum1(m, lc + 8);
        if (rs) { a *= rs[m]; b *= rs[m]; }
        if (idx < nth) qkv_pair_at(a, b, m, col, N / 3, epi, p_first, cs_first);   // (requested ahead of the k loop)
        else qkv_pair(a, b, m, col, N / 3, epi);
      }
    }
  }
}

template <int CT, int NT, int DEPTH, bool STREAM, bool ROWMAJOR = false>     // (ROWMAJOR as above)
__global__ __launch_bounds__(512) void k_gemm_bf16_wide(const uint4* __restrict__ Wsw, const uint4* __restrict__ XF,
                                                        const float* __restrict__ gain, const float* __restrict__ ssq_part, int K, int N,
                                                        int M, int role, int ssq_n, float eps, GemmEpi epi) {
  const RowNorm nrm{gain, ssq_part, ssq_n, eps};
  const int NTILES = N >> 4;
  constexpr int RING = DEPTH < kWideDepthChunk ? DEPTH + 1 : DEPTH;
  constexpr int W = NT * 16;
  extern __shared__ float csum[];                          // [chunk][M][W]
  __shared__ float s_rstd[kMaxFwdRows];
  const int tid = threadIdx.x, lane = tid & 63, NW = blockDim.x >> 6;
  // (the wave index as a scalar: everything derived from it -- chunk, k-step, addresses -- is then scalar arithmetic)
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int j = lane & 15, g = lane >> 4;
  const int tile0 = blockIdx.x * NT;
  const int units_total = K / kUnitK;
  const int nchunks = (units_total + kSliceUnits - 1) / kSliceUnits;
  const int cpw = (nchunks + NW - 1) / NW;                 // chunks per wave
  const int c_begin = min(wave * cpw, nchunks), c_end = min(nchunks, c_begin + cpw);
  const int s_begin = c_begin * 16, s_end = min(K >> 5, c_end * 16);   // this wave's k-steps (32 k each)
  const bool has_stats = nrm.gain && nrm.ssq_part;

  struct Stage {
    uint4 a[NT], bh[CT], bl[CT];
  };
  // what a k-step needs, requested without conditions (tiles past the end re-read the last one and are dropped
  // later), so that the outstanding loads can be counted exactly
  int tile_c[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) tile_c[t] = min(tile0 + t, NTILES - 1);
  auto load_stage = [&](Stage& st, int s) {
    const int c = s >> 4, kk = s & 15;
    const int ksteps_c = min(kSliceUnits, units_total - c * kSliceUnits) * 8;
    const uint4* wbase = Wsw + (size_t)c * NTILES * (kSliceUnits * 8) * 64 + (size_t)kk * 64 + lane;
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const uint4* p = ROWMAJOR ? Wsw + (size_t)(tile_c[t] * 16 + (lane & 15)) * (K >> 3) + s * 4 + (lane >> 4)
                                : wbase + (size_t)tile_c[t] * ksteps_c * 64;
      st.a[t] = STREAM ? ld_nt(p) : *p;
    }
    const uint4* xb = XF + (size_t)s * 4 * 64 + (size_t)c * kFragChunkPad + lane;
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {                      // column tiles 2, 3: the second fragment block
      const uint4* xc = xb + (size_t)(ct >> 1) * kFragHalfU4 + ((ct & 1) * 2) * 64;
      st.bh[ct] = xc[0];
      st.bl[ct] = xc[64];
    }
  };

  f32x4 acc[NT][CT];
  auto compute_stage = [&](const Stage& st, int s) {
    if ((s & 15) == 0) {
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) acc[t][ct] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const bf16x8 a = __builtin_bit_cast(bf16x8, st.a[t]);
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) {
        acc[t][ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, __builtin_bit_cast(bf16x8, st.bh[ct]), acc[t][ct], 0, 0, 0);
        acc[t][ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, __builtin_bit_cast(bf16x8, st.bl[ct]), acc[t][ct], 0, 0, 0);
      }
    }
    if ((s & 15) == 15 || s == s_end - 1) {                // the chunk is complete (the last one may be short)
      float* dst = csum + (size_t)(s >> 4) * M * W;
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) {
        const int m = ct * 16 + j;
        if (m < M) {
#pragma unroll
          for (int t = 0; t < NT; ++t)
            *reinterpret_cast<float4*>(dst + m * W + t * 16 + 4 * g) =
                make_float4(acc[t][ct][0], acc[t][ct][1], acc[t][ct][2], acc[t][ct][3]);
        }
      }
    }
  };

  Stage st[RING];
  const bool work = s_begin < s_end;                       // (a wave without k chunks only helps in the epilogue)
  if (work) {
#pragma unroll
    for (int i = 0; i < DEPTH; ++i) load_stage(st[i], min(s_begin + i, s_end - 1));
  }
  // needed by the epilogue only, requested behind the first weights: the old x (first pass of the epilogue's threads) and
  // the rows' 1/rms
  float4 x_first = make_float4(0.f, 0.f, 0.f, 0.f);
  if (role == kRoleWo || role == kRoleDown) {
    const int m = tid / (W / 4), col = tile0 * 16 + (tid - m * (W / 4)) * 4;
    if (m < M && col < N) x_first = *reinterpret_cast<const float4*>(epi.out + (size_t)m * N + col);
  }
  int p_first = 0;                                         // QKV: the row's position and rotation entry
  float2 cs_first = make_float2(1.f, 0.f);
  if (role == kRoleQKV) {
    const int m = tid / (W / 2), r = tid - m * (W / 2), col = tile0 * 16 + 16 * (r >> 3) + (r & 7);
    if (m < M && col < N) {
      p_first = pos_of(epi.pos, m);
      cs_first = epi.rope_cs[qkv_rope_index(m, col, N / 3, epi.hd)];
    }
  }
  if (has_stats) rows_rstd_any(nrm, M, K, s_rstd);
  if (work) {
    // whole turns of the ring without a condition around a request (a branch would make the compiler assume the
    // fewest outstanding loads at every join and wait for nearly all of them); the last DEPTH or fewer k-steps have
    // been requested by then
    int s = s_begin;
    if constexpr (DEPTH < kWideDepthChunk)             // (else the wave's only chunk has been requested as a whole)
    for (; s + RING <= s_end; s += RING) {
#pragma unroll
      for (int i = 0; i < RING; ++i) {
        load_stage(st[(i + DEPTH) % RING], min(s + i + DEPTH, s_end - 1));
        __builtin_amdgcn_sched_barrier(0);         // the requests stay in front of the arithmetic they overlap with
        compute_stage(st[i], s + i);
      }
    }
#pragma unroll
    for (int i = 0; i < DEPTH; ++i)
      if (s + i < s_end) compute_stage(st[i], s + i);
  }
  __syncthreads();

  const float* rs = has_stats ? s_rstd : nullptr;
  const int c0 = tile0 * 16;
  switch (role) {
    case kRoleQKV: gemm_epilogue_lds<kRoleQKV, W>(csum, nchunks, M, N, c0, epi, rs, x_first, p_first, cs_first); break;
    case kRoleWo:
    case kRoleDown: gemm_epilogue_lds<kRoleWo, W>(csum, nchunks, M, N, c0, epi, rs, x_first, p_first, cs_first); break;
    case kRoleGateUp: gemm_epilogue_lds<kRoleGateUp, W>(csum, nchunks, M, N, c0, epi, rs, x_first, p_first, cs_first); break;
    default: gemm_epilogue_lds<kRoleHead, W>(csum, nchunks, M, N, c0, epi, rs, x_first, p_first, cs_first); break;
  }
}

// x [M, K] (row stride ldx) -> its fragments, gain folded in (nullptr: none): for activations whose producer does not
// leave them itself.  One thread per (row, 4 consecutive k).
__global__ __launch_bounds__(256) void k_split_frag(const float* __restrict__ X, int ldx, int M, int K,
                                                    const float* __restrict__ gain, uint4* __restrict__ frag) {
  const int idx = blockIdx.x * 256 + threadIdx.x;
  const int k4 = K >> 2;
  if (idx >= M * k4) return;
  const int m = idx / k4, k = (idx - m * k4) * 4;
  store_frag4(frag, m, k, *reinterpret_cast<const float4*>(X + (size_t)m * ldx + k), gain);
}
void launch_split_frag(const float* X, int ldx, int M, int K, const float* gain, uint4* frag, hipStream_t st) {
  hipLaunchKernelGGL(k_split_frag, dim3((M * (K / 4) + 255) / 256), dim3(256), 0, st, X, ldx, M, K, gain, frag);
}

// LDS bytes of k_gemm_bf16_rows, or 0 if this shape does not take that path.  The residual-writing projections
// have few weight tiles (N = d_model): they run one 8-wave work-group per CU and only when the tiles about
// cover the chip.
size_t rows_path_lds(int role, int M, int N, int K) {
  static const int max_rows = [] { const char* e = getenv("STAIRS_ROWS_MAX"); return e ? atoi(e) : 7; }();   // tuning aid
  if (M > 7 || M > max_rows) return 0;
  const size_t bytes = (size_t)K * M * 4 + (size_t)(gemm_slices(K, 1) + 1) * M * 16 * 4;
  // 5..7 rows (at 8 the fragment-reading kernel is as fast), three cases:
  // k below 2048, a work-group per tile: up to as many as CUs 4.5 .. 5.2 us a launch at 125M and at the large encoder-decoder
  // shape, where the fragment-reading kernel takes 5.1 .. 5.4; more at 5 / 7 rows: 384 tiles, k = 768 5.6 / 5.9 us of a layer
  // against 7.2 / 7.8, 2000 tiles, k = 1024 12.8 / 13.4 against 14.7 / 15.6 (with work-groups that walk through the tiles it
  // was the slower one).
  if (M > 4 && role != kRoleDown && K < 2048) return bytes <= kRowsPathMaxLds ? bytes : 0;
  // feed-forward outputs with k up to 4096 (one staging pass) and few tiles: 5.0 .. 5.5 against 7.0 us at 125M
  if (M > 4 && role == kRoleDown) return K <= 4096 && N / 16 <= 128 && bytes <= kRowsPathMaxLdsWide ? bytes : 0;
  // k of 2048 and more, a chunk for each wave: the block takes more than half a CU's LDS, so one work-group per CU walks
  // through the tiles
  if (M > 4) return bytes <= kRowsPathMaxLdsWide && N / 16 >= 192 ? std::max(bytes, (size_t)81 * 1024) : 0;
  if (role == kRoleWo || role == kRoleDown) {
    // few tiles: only matrices so small that the launch is latency-bound anyway (no partial sums, no hand-off)
    if (N / 16 < 192) {
      if ((size_t)N * K * 2 <= kRowsPathSmallMatrix) return bytes <= kRowsPathMaxLdsWide ? bytes : 0;
      // a larger matrix with few tiles but a long k range (down projection of a 1B-class model: 128 tiles x 16
      // chunks): 16 waves per work-group, a k chunk each -- half the CUs stream it faster than split-K work-groups
      // on all of them with their hand-off (measured: 12.4 -> 9.7 us per launch)
      return (role == kRoleDown && gemm_slices(K, 1) >= 12 && gemm_slices(K, 1) <= 16 && bytes <= kRowsPathMaxLdsWide)
                 ? std::max(bytes, (size_t)81 * 1024) : 0;
    }
    return bytes <= kRowsPathMaxLdsWide ? std::max(bytes, (size_t)81 * 1024) : 0;   // > half a CU's LDS: one per CU
  }
  return bytes <= kRowsPathMaxLds ? bytes : 0;
}

// Launch shape of k_gemm_bf16_wide: NT weight tiles per wave and NW waves that split the k chunks; nt == 0: the
// split-K kernel instead.  Measured on 7B-class projections (isolated launches, 8 / 17 rows, microseconds; split-K
// in brackets): gate/up 1376 tiles 8/4 33 / 36 (37 / 48), unembedding 2000 tiles 8/4 41 / 43 (48 / 63), QKV 768 tiles
// 4/4 21 / 25 (23 / 33), attention-out 256 tiles 1/8 10.4 / 13.4 (11.4 / 15.4), down 256 tiles and 22 chunks 1/4 23 /
// 32 (21 / 34).  More tiles per wave means fewer fragment reads and fewer, longer-lived waves per weight byte; with
// few tiles (N = d_model) that leaves too few work-groups, and for a long k at up to 16 rows split-K's extra
// parallelism still wins.
constexpr int wide_depth2(int depth1) { return depth1 <= 2 ? 1 : depth1 <= 3 ? 2 : depth1 <= 5 ? 3 : 5; }   // ring depth at two column tiles
constexpr int wide_depth3(int depth1) { return depth1 <= 3 ? 1 : depth1 <= 5 ? 2 : 3; }                      // at three (33..48 rows)
constexpr int wide_depth4(int depth1) { return depth1 <= 3 ? 1 : 2; }                                        // at four (49..64 rows; 3 spills at one tile)
// STAIRS_WIDE_CFG="nt/nw,nt/nw,nt/nw,nt/nw,nt/nw" (QKV, out, gate-up, down, head; nt = 0: split-K) sends the role's projections
// of more than 4 rows to this kernel with that shape: tuning aid.  nullptr: not set, or not a shape there is.
static const WideCfg* wide_forced(int role) {
  static const std::vector<WideCfg> forced = [] {
    std::vector<WideCfg> v;
    if (const char* e = getenv("STAIRS_WIDE_CFG")) {
      int nt = 0, nw = 0, n = 0;
      while (sscanf(e, "%d/%d%n", &nt, &nw, &n) == 2) {
        v.push_back({nt, nw});
        e += n;
        if (*e == ',') ++e;
      }
    }
    return v;
  }();
  if ((int)forced.size() != 5) return nullptr;
  const WideCfg& f = forced[role];
  const bool ok = (f.nt == 0 || f.nt == 1 || f.nt == 2 || f.nt == 3 || f.nt == 4 || f.nt == 6 || f.nt == 8) && f.nw >= 1 && f.nw <= 8;
  return ok ? &f : nullptr;
}
bool wide_cfg_is_forced(int role) { return wide_forced(role) != nullptr; }

WideCfg wide_cfg(int role, int M, int NTILES, int K) {
  const int nchunks = gemm_slices(K, 1);
  // Measured on the 125M, 1B and 7B workloads (5..32 rows): about one work-group per CU, i.e. the smallest number of
  // tiles per wave (1, 2, 3, 4, 6, 8) that covers the matrix with at most 256 work-groups, as long as about 170 remain
  // (7B: gate/up 1376 tiles -> 6, 230 work-groups: 29.6 us at 9 rows against 32.4 us for 172 work-groups of 8; QKV
  // 768 -> 3, 256 work-groups: 19.6 against 22.0 us for 192 of 4; unembedding 2000 -> 8); with one tile per wave up
  // to 8 waves share the k chunks, else 4 (8 and 2 measured slower).  Few tiles with a long k range (down projections:
  // 128 x 8192 at 1B, 256 x 11008 at 7B) stream better through the split-K kernel, whose grid also cuts k; from 17
  // rows on the 7B shape is the exception.  Small matrices are latency-bound either way and the missing hand-off is
  // what counts (125M at 16 rows: 595 -> 470 us per forward).
  WideCfg c{0, 0};
  if (nchunks > 8 && NTILES < 512) {
    if (NTILES >= 192 && M > 16) c = {1, 4};
  } else {
    static const int kNts[] = {1, 2, 3, 4, 6, 8};
    int i = 0;
    while (i < 5 && kNts[i] * 256 < NTILES) ++i;
    while (i > 0 && NTILES / kNts[i] < 170) --i;
    const int nt = kNts[i];
    c = {nt, std::min(nt == 1 ? 8 : 4, nchunks)};
  }
  const WideCfg* const f = wide_forced(role);
  if (f) c = *f;
  if (M > 2 * 16) {                      // 33..64 rows: never split-K, which stops at two column tiles; up to 48 rows one or two tiles per wave, then one
    // 8 waves, two a SIMD, cover each other's waits for the fragments, which outweigh the weights here
    if (!f || f->nt == 0) c.nw = std::min(8, nchunks);
    c.nt = M <= 3 * 16 && c.nt >= 2 ? 2 : 1;
  }
  return c;
}

// The form of k_gemm_bf16_rows for a k range, and for work-groups of one tile or several.
template <int R, int ROLE, int NW, int GP, bool STREAM, bool ROWMAJOR = false>
static auto rows_kernel(int K, bool walk) {
  constexpr int reach = 8 * 64 * NW;       // k a work-group's threads cover with one k group each
  constexpr bool walks = ROLE != kRoleDown && !ROWMAJOR;    // (down projections of 5..7 rows: at most 128 tiles)
  if (walks && walk) return &k_gemm_bf16_rows<R, ROLE, NW, GP, 1, walks, STREAM, ROWMAJOR>;
  if (R > 2 && K <= reach / 4) return &k_gemm_bf16_rows<R, ROLE, NW, 1, (R > 2 ? 4 : 1), false, STREAM, ROWMAJOR>;
  if (R > 1 && K <= reach / 2) return &k_gemm_bf16_rows<R, ROLE, NW, 1, (R > 1 ? 2 : 1), false, STREAM, ROWMAJOR>;
  if (GP > 1 && K <= reach) return &k_gemm_bf16_rows<R, ROLE, NW, 1, 1, false, STREAM, ROWMAJOR>;
  return &k_gemm_bf16_rows<R, ROLE, NW, GP, 1, false, STREAM, ROWMAJOR>;
}

// Y [M, N] = X . W^T with W [N, K] as the caller has it (bf16, row-major); frag: scratch for M > 4.  Returns false,
// launching nothing, for shapes that need the split-K kernel (few tiles with a long k; LDS).
bool launch_gemm_rowmajor(const uint16_t* W, int N, int K, const float* X, int M, float* Y, uint4* frag, hipStream_t st) {
  const int NTILES = N / 16, nchunks = gemm_slices(K, 1);
  const RowNorm none{nullptr, nullptr, 0, 0.f};
  GemmEpi e{};
  e.out = Y;
  e.hd = 64;
  const uint4* Wr = reinterpret_cast<const uint4*>(W);
  const size_t rl = rows_path_lds(kRoleHead, M, N, K);
  if (rl && M <= 4) {
#define STAIRS_ROWM(r) \
  hipLaunchKernelGGL((rows_kernel<r, kRoleHead, 4, 2, false, true>(K, false)), dim3(NTILES), dim3(256), rl, st, Wr, X, none.gain, none.ssq_part, K, N, K, none.ssq_n, e.out, none.eps, RowsEpi{e, nullptr})
    if (M == 1) STAIRS_ROWM(1);
    else if (M == 2) STAIRS_ROWM(2);
    else if (M == 3) STAIRS_ROWM(3);
    else STAIRS_ROWM(4);
#undef STAIRS_ROWM
    return true;
  }
  const WideCfg wc = wide_cfg(kRoleHead, M, NTILES, K);
  const int nt = NTILES <= 256 ? 1 : 2, nw = std::min(8, nchunks);
  const size_t lds = (size_t)nchunks * M * nt * 16 * sizeof(float);
  if (M <= 4 || wc.nt == 0 || lds > kWideMaxLds) return false;
  launch_split_frag(X, K, M, K, nullptr, frag, st);
  const dim3 grid((NTILES + nt - 1) / nt), block(64 * nw);
#define STAIRS_WIDEM(ct, nt, dp) \
  hipLaunchKernelGGL((k_gemm_bf16_wide<ct, nt, dp, false, true>), grid, block, lds, st, Wr, frag, none.gain, none.ssq_part, K, N, M, (int)kRoleHead, none.ssq_n, none.eps, e)
  if (M <= 16) {
    if (nt == 1) STAIRS_WIDEM(1, 1, kWideDepth1);
    else STAIRS_WIDEM(1, 2, kWideDepth2);
  } else {
    if (nt == 1) STAIRS_WIDEM(2, 1, wide_depth2(kWideDepth1));
    else STAIRS_WIDEM(2, 2, wide_depth2(kWideDepth2));
  }
#undef STAIRS_WIDEM
  return true;
}

// fp32 weights, row-major: a wave takes the two output features an epilogue combines (rotation pairs, gate and up, else
// neighbours) for all rows, lanes stride over k, and runs the epilogue itself.  The sum of squares of a normalised input
// is gathered on the way (every wave reads the whole row anyway).  What bounds it: the launch and one round trip to
// memory (models of this type are tiny).  With the epilogues in kernels of their own, the attention's merge in another
// and a branch around every row's loads a layer was 10 launches, now 5 (d 256, 4 layers + 2 of draft, 32 + 64 tokens:
// 12.6 -> 7.4 ms; residual-writing projection at 1 / 5 rows: 3.35 + 2.4 / 6.9 + 2.4 -> 2.4 / 4.9 us).
constexpr int kRoleLogits = 5;           // kRoleHead with a normalised input
// The sums over the wave of rows q .. q + 3, row q + m's in lanes 16 m .. 16 m + 15 (one row: in all lanes).  Four rows share
// the exchanges: 12 instructions a row and sum become 4, and a norm's square root and division are done once for four rows.
// From 6 rows on the kernel asks for two waves a SIMD, no more: with the short reduction the compiler otherwise aims at more
// waves and puts the loop's loads one after the other (54 .. 154 registers; 32 rows, 1000 x 2044 34.5 us).  Host call on device
// buffers, row by row through the LDS unit -> now, us: 1000 x 2044 at 6 / 16 / 32 rows 7.6 / 16.9 / 21.5 -> 7.0 / 12.2 / 12.9,
// 1024 x 1024 at 16 / 32 rows 10.7 / 14.0 -> 7.6 / 9.4, 256 x 256 at 32 rows 9.7 -> 6.7; the tiny pair 7.1 -> 6.2 ms.
template <int MR>
__device__ __forceinline__ float rows_sum4(const float (&v)[MR], int q) {
  if constexpr (MR == 1) return wave_sum(v[0]);
  return wave_sums4(v[q], q + 1 < MR ? v[min(q + 1, MR - 1)] : 0.f, q + 2 < MR ? v[min(q + 2, MR - 1)] : 0.f, q + 3 < MR ? v[min(q + 3, MR - 1)] : 0.f);
}
template <int MR, int ROLE>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(MR >= 6 ? 2 : 4, MR >= 6 ? 2 : 8))) void k_gemm_f32(const float* __restrict__ W, const float* __restrict__ X,
                                                  const float* __restrict__ gain, float* out, int N, int K, int ldx, int M, const int* pos_base,
                                                  float eps, GemmEpi epi) {
  constexpr bool NORMED = ROLE == kRoleQKV || ROLE == kRoleGateUp || ROLE == kRoleLogits;
  const int lane = threadIdx.x & 63;
  const int pr = blockIdx.x * 4 + (threadIdx.x >> 6);                 // feature pair
  if (pr >= N / 2) return;
  const int d = N / 3, half = epi.hd >> 1;
  int n0, n1, part = 0, h = 0, e = 0;
  if (ROLE == kRoleQKV) {                                              // (e, e + hd/2) of one head of q, k or v
    part = pr / (d >> 1);
    const int c = pr - part * (d >> 1);
    h = c / half;
    e = c - h * half;
    n0 = part * d + h * epi.hd + e;
    n1 = n0 + half;
  } else if (ROLE == kRoleGateUp) {
    n0 = pr;
    n1 = pr + N / 2;
  } else {
    n0 = 2 * pr;
    n1 = n0 + 1;
  }
  // a row is finished by the lane where wave_sums4 leaves its sums: what it needs beside them is requested first
  const int row = (lane & 15) * 4 + (lane >> 4);
  const bool mine = row < M && row < MR;
  float2 old = make_float2(0.f, 0.f), cs = make_float2(1.f, 0.f);
  int pos = 0;
  if (mine) {
    if (ROLE == kRoleWo || ROLE == kRoleDown) old = *reinterpret_cast<const float2*>(out + (size_t)row * N + n0);
    if (ROLE == kRoleQKV) {
      pos = *pos_base + epi.pos.offset + row;
      if (part < 2) cs = epi.rope_cs[row * 64 + e];
    }
  }
  float a0[MR], a1[MR], ss[MR];
#pragma unroll
  for (int i = 0; i < MR; ++i) a0[i] = a1[i] = ss[i] = 0.f;
  // rows past the last are read as the last one and dropped: a branch per row would put one round trip after another
  const float* xr[MR];
#pragma unroll
  for (int i = 0; i < MR; ++i) xr[i] = X + (size_t)min(i, M - 1) * ldx;
  constexpr int UNROLL = MR > 16 ? 1 : 2;
#pragma unroll UNROLL
  for (int k = lane * 4; k < K; k += 256) {
    const float4 w0 = *reinterpret_cast<const float4*>(W + (size_t)n0 * K + k), w1 = *reinterpret_cast<const float4*>(W + (size_t)n1 * K + k);
    float4 g = make_float4(1.f, 1.f, 1.f, 1.f), x[MR];
    if (NORMED && gain) g = *reinterpret_cast<const float4*>(gain + k);
#pragma unroll
    for (int i = 0; i < MR; ++i) x[i] = *reinterpret_cast<const float4*>(xr[i] + k);
#pragma unroll
    for (int i = 0; i < MR; ++i) {
      float4 y = x[i];
      if (NORMED) {
        ss[i] = fmaf(y.w, y.w, fmaf(y.z, y.z, fmaf(y.y, y.y, fmaf(y.x, y.x, ss[i]))));
        y = make_float4(__fmul_rn(y.x, g.x), __fmul_rn(y.y, g.y), __fmul_rn(y.z, g.z), __fmul_rn(y.w, g.w));
      }
      a0[i] = fmaf(w0.w, y.w, fmaf(w0.z, y.z, fmaf(w0.y, y.y, fmaf(w0.x, y.x, a0[i]))));
      a1[i] = fmaf(w1.w, y.w, fmaf(w1.z, y.z, fmaf(w1.y, y.y, fmaf(w1.x, y.x, a1[i]))));
    }
  }
  // (1/rms goes onto the lanes' sums, not onto the finished one: 64 roundings that average out instead of one that stays)
  if (NORMED && gain) {
#pragma unroll
    for (int q = 0; q < MR; q += 4) {
      const float r4 = 1.0f / sqrtf(rows_sum4<MR>(ss, q) / (float)K + eps);
#pragma unroll
      for (int i = q; i < MR && i < q + 4; ++i) {
        const float r = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(r4), (i - q) * 16));
        a0[i] = __fmul_rn(a0[i], r);
        a1[i] = __fmul_rn(a1[i], r);
      }
    }
  }
  float v0 = 0.f, v1 = 0.f;
#pragma unroll
  for (int q = 0; q < MR; q += 4) {
    const float s0 = rows_sum4<MR>(a0, q), s1 = rows_sum4<MR>(a1, q);
    v0 = (lane & 15) * 4 == q ? s0 : v0;
    v1 = (lane & 15) * 4 == q ? s1 : v1;
  }
  if (!mine) return;
  if (ROLE == kRoleWo || ROLE == kRoleDown) {
    *reinterpret_cast<float2*>(out + (size_t)row * N + n0) = make_float2(__fadd_rn(old.x, v0), __fadd_rn(old.y, v1));
  } else if (ROLE == kRoleGateUp) {
    out[(size_t)row * (N / 2) + pr] = swiglu(v0, v1);
  } else if (ROLE == kRoleHead || ROLE == kRoleLogits) {
    *reinterpret_cast<float2*>(out + (size_t)row * N + n0) = make_float2(v0, v1);
  } else if (pos >= 0) {
    if (part < 2) {
      const float2 r = rope_rotate(v0, v1, cs);
      v0 = r.x;
      v1 = r.y;
    }
    float* dst = part == 0 ? out + (size_t)row * d + h * epi.hd + e
                           : (part == 1 ? epi.Kc32 : epi.Vc32) + ((size_t)h * epi.cap + pos) * epi.hd + e;
    dst[0] = v0;
    dst[half] = v1;
  }
}

// weight tiles per wave (1 or 2) of the split-K kernel: two when that still leaves enough work-groups to cover
// the chip a few times over (more tiles per work-group = fewer activation slices staged per weight byte)
static int pick_nt(int NTILES, int SG, int want_wgs) {
  return ((size_t)((NTILES + 7) / 8) * SG >= (size_t)want_wgs) ? 2 : 1;
}

// Events the next GEMM launch records at the kernel's own start and end (set_gemm_launch_events): lets a measurement
// take one kernel's duration inside a running forward without event records around it in the stream.
// (per thread: a context is used by one thread at a time)
static thread_local hipEvent_t g_gemm_ev_start = nullptr, g_gemm_ev_stop = nullptr;
void set_gemm_launch_events(hipEvent_t start, hipEvent_t stop) {
  g_gemm_ev_start = start;
  g_gemm_ev_stop = stop;
}
template <typename F, typename... Args>
static void launch_gemm_kernel(F kernel, dim3 grid, dim3 block, size_t lds, hipStream_t st, Args... args) {
  if (g_gemm_ev_start && g_gemm_ev_stop) {
    hipExtLaunchKernelGGL(kernel, grid, block, (std::uint32_t)lds, st, g_gemm_ev_start, g_gemm_ev_stop, 0, args...);
    g_gemm_ev_start = g_gemm_ev_stop = nullptr;
  } else {
    hipLaunchKernelGGL(kernel, grid, block, lds, st, args...);
  }
}

bool gemm_takes_rows(int M, int K) {
  return M <= kMaxFwdRows && (size_t)gemm_slices(K, 1) * M * 16 * sizeof(float) <= kWideMaxLds;
}

static void gemm(int role, int dtype_bf16, const void* W, int N, int K, const float* X, int ldx, int M, RowNorm nrm,
                 float* partial, const GemmEpi& epi, hipStream_t st, const uint4* xfrag, float2* cand) {
  if (!dtype_bf16) {
    const dim3 grid((N / 2 + 3) / 4), block(256);
    const float* Wf = static_cast<const float*>(W);
#define STAIRS_F32(mr, role) launch_gemm_kernel(k_gemm_f32<mr, role>, grid, block, (size_t)0, st, Wf, X, nrm.gain, epi.out, N, K, ldx, M, epi.pos.base, nrm.eps, epi)
#define STAIRS_F32_ROLE(role)               \
  do {                                      \
    if (M <= 1) STAIRS_F32(1, role);        \
    else if (M <= 2) STAIRS_F32(2, role);   \
    else if (M <= 3) STAIRS_F32(3, role);   \
    else if (M <= 4) STAIRS_F32(4, role);   \
    else if (M <= 6) STAIRS_F32(6, role);   \
    else if (M <= 8) STAIRS_F32(8, role);   \
    else if (M <= 16) STAIRS_F32(16, role); \
    else STAIRS_F32(32, role);              \
  } while (0)
    switch (role) {
      case kRoleQKV: STAIRS_F32_ROLE(kRoleQKV); break;
      case kRoleWo:
      case kRoleDown: STAIRS_F32_ROLE(kRoleWo); break;
      case kRoleGateUp: STAIRS_F32_ROLE(kRoleGateUp); break;
      default:
        if (nrm.gain) STAIRS_F32_ROLE(kRoleLogits);
        else STAIRS_F32_ROLE(kRoleHead);
        break;
    }
#undef STAIRS_F32_ROLE
#undef STAIRS_F32
    return;
  }
  const int S = gemm_slices(K, 1);
  const int NTILES = N / 16;
  const uint4* Wsw = static_cast<const uint4*>(W);
  if (const size_t rl = rows_path_lds(role, M, N, K)) {
    // gate/up has several times more tiles than the chip has CUs: one work-group per CU that walks through its
    // share of the tiles (X block staged once, the next tile's first units requested before the epilogue, all
    // work-groups resident from the start and done together) streams better than a work-group per tile (7B, 1376
    // tiles, isolated: 30.1 -> 28.5 us at 3 rows with 230 work-groups of 6 tiles; 459 x 3: 29.1, 344 x 4: 32.5 -- two
    // work-groups on some CUs and one on others is the worst case; the unembedding's 2000 tiles and, with its
    // epilogue's loads requested early, QKV's 768 gain nothing)
    int tpw = 1;
    if ((role == kRoleGateUp && NTILES >= 4 * 256) || (M > 4 && NTILES > 256 && K >= 2048)) tpw = (NTILES + 255) / 256;
    {
      static const int forced = [] { const char* e = getenv("STAIRS_ROWS_TPW"); return e ? atoi(e) : 0; }();
      if (forced > 0 && (role == kRoleGateUp || role == kRoleHead)) tpw = forced;    // tuning aid
    }
    const dim3 rgrid((NTILES + tpw - 1) / tpw);
    // (walking work-groups ask for more than half a CU's LDS, so that no CU gets two of them while another has none)
    const size_t rl_launch = tpw > 1 ? std::max(rl, (size_t)81 * 1024) : rl;
#define STAIRS_ROWS(r, role, nw, gp)                                                                                    \
  launch_gemm_kernel(epi.stream_weights ? rows_kernel<r, role, nw, gp, true>(K, tpw > 1) : rows_kernel<r, role, nw, gp, false>(K, tpw > 1), rgrid, \
                     dim3(64 * nw), rl_launch, st, Wsw, X, nrm.gain, nrm.ssq_part, K, N, ldx, nrm.ssq_n, epi.out, nrm.eps, RowsEpi{epi, cand})
#define STAIRS_ROWS_ROLE4(role, nw, gp)          \
  if (M <= 1) STAIRS_ROWS(1, role, nw, gp);      \
  else if (M == 2) STAIRS_ROWS(2, role, nw, gp); \
  else if (M == 3) STAIRS_ROWS(3, role, nw, gp); \
  else STAIRS_ROWS(4, role, nw, gp)
#define STAIRS_ROWS_ROLE(role, nw, gp)                \
  if (M <= 4) { STAIRS_ROWS_ROLE4(role, nw, gp); }    \
  else if (M == 5) STAIRS_ROWS(5, role, nw, gp);      \
  else if (M == 6) STAIRS_ROWS(6, role, nw, gp);      \
  else STAIRS_ROWS(7, role, nw, gp)
    if (role == kRoleQKV) { STAIRS_ROWS_ROLE(kRoleQKV, 4, 2); }
    else if (role == kRoleGateUp) { STAIRS_ROWS_ROLE(kRoleGateUp, 4, 2); }
    else if (role == kRoleHead) { STAIRS_ROWS_ROLE(kRoleHead, 4, 2); }
    else if (role == kRoleWo) { STAIRS_ROWS_ROLE(kRoleWo, 8, 1); }
    else if (M <= 4 && NTILES < 192 && (size_t)N * K * 2 > kRowsPathSmallMatrix) { STAIRS_ROWS_ROLE4(kRoleDown, 16, 1); }
    else if (M == 5) STAIRS_ROWS(5, kRoleDown, 8, 1);
    else if (M == 6) STAIRS_ROWS(6, kRoleDown, 8, 1);
    else if (M == 7) STAIRS_ROWS(7, kRoleDown, 8, 1);
    else { STAIRS_ROWS_ROLE4(kRoleDown, 8, 3); }
#undef STAIRS_ROWS_ROLE
#undef STAIRS_ROWS_ROLE4
#undef STAIRS_ROWS
    return;
  }
  // more than 16 rows with the activation fragments at hand: where it is faster, the kernel that shares them through LDS
  if (M > 16 && xfrag && launch_gemm_shared(role, W, N, K, xfrag, M, nrm, partial, epi, st)) return;
  // more than 4 rows with the activation fragments at hand: the hand-off-free kernel
  WideCfg wc = wide_cfg(role, M, NTILES, K);
  const int nchunks = gemm_slices(K, 1);
  auto wide_lds = [&](int nt) { return (size_t)nchunks * M * nt * 16 * sizeof(float); };
  while (wc.nt > 1 && wide_lds(wc.nt) > kWideMaxLds) wc.nt = wc.nt == 6 ? 4 : wc.nt == 3 ? 2 : wc.nt / 2;   // very long k: fewer tiles per work-group
  if (xfrag && wc.nt > 0 && wide_lds(wc.nt) <= kWideMaxLds) {
    const int CT = (M + 15) / 16;
    dim3 grid((NTILES + wc.nt - 1) / wc.nt), block(64 * wc.nw);
    const size_t lds = wide_lds(wc.nt);
#define STAIRS_WIDE(ct, nt, dp)                                                                                          \
  do {                                                                                                                   \
    if (epi.stream_weights)                                                                                              \
      launch_gemm_kernel(k_gemm_bf16_wide<ct, nt, dp, true>, grid, block, lds, st, Wsw, xfrag, nrm.gain, nrm.ssq_part,   \
                         K, N, M, role, nrm.ssq_n, nrm.eps, epi);                                                                                     \
    else                                                                                                                 \
      launch_gemm_kernel(k_gemm_bf16_wide<ct, nt, dp, false>, grid, block, lds, st, Wsw, xfrag, nrm.gain, nrm.ssq_part,  \
                         K, N, M, role, nrm.ssq_n, nrm.eps, epi);                                                                                     \
  } while (0)
  // (two column tiles hold one k-step less in flight: a deeper ring would not fit the 256 registers of a wave)
  // (three and four column tiles, one more: see shared_takes)
#define STAIRS_WIDE_CT2(nt, dp)        \
  if (CT == 1) STAIRS_WIDE(1, nt, dp); \
  else STAIRS_WIDE(2, nt, wide_depth2(dp))
#define STAIRS_WIDE_CT(nt, dp)                          \
  if (CT <= 2) { STAIRS_WIDE_CT2(nt, dp); }             \
  else if (CT == 3) STAIRS_WIDE(3, nt, wide_depth3(dp)); \
  else STAIRS_WIDE(4, nt, wide_depth4(dp))
    if (wc.nt == 8) { STAIRS_WIDE_CT2(8, kWideDepth8); }
    else if (wc.nt == 6) { STAIRS_WIDE_CT2(6, kWideDepth6); }
    else if (wc.nt == 3) { STAIRS_WIDE_CT2(3, kWideDepth3); }
    else if (wc.nt == 4) { STAIRS_WIDE_CT2(4, kWideDepth4); }
    else if (wc.nt == 2 && CT == 3) { STAIRS_WIDE(3, 2, wide_depth3(kWideDepth2)); }
    else if (wc.nt == 2) { STAIRS_WIDE_CT2(2, kWideDepth2); }
    else if (wide_whole_chunk(M, nchunks, wc.nw)) STAIRS_WIDE(1, 1, kWideDepthChunk);
    else { STAIRS_WIDE_CT(1, kWideDepth1); }
#undef STAIRS_WIDE_CT
#undef STAIRS_WIDE_CT2
#undef STAIRS_WIDE
    return;
  }
  // 9..16 rows: a work-group takes two k chunks and writes the sum of the pair (half the partial sums in memory;
  // measured -7 % on a 7B layer at 16 rows).  With two column tiles (17..32 rows) the halved work-group count
  // or, with one weight tile per wave, the doubled activation staging cost more than the partial sums saved.
  const int CT = (M <= 16) ? 1 : 2;
  const int SPW = (M >= kSpwRows && CT == 1 && S >= 2) ? 2 : 1;
  const int SG = (S + SPW - 1) / SPW;
  int NT;
  if (SPW == 1) NT = (role == kRoleWo || role == kRoleDown) ? 2 : pick_nt(NTILES, SG, 1024);
  else NT = pick_nt(NTILES, SG, 640);
  dim3 grid((NTILES + 4 * NT - 1) / (4 * NT), SG), block(256);
  const size_t lds = (size_t)16 * CT * 2 * 64 * sizeof(uint4);
#define STAIRS_GEMM(ct, nt, role, spw) \
  do {                                                                                                                \
    if (epi.stream_weights)                                                                                           \
      launch_gemm_kernel(k_gemm_bf16<ct, nt, role, spw, true>, grid, block, lds, st, Wsw, X, nrm.gain, partial, K, N,    \
                         ldx, M, nrm.ssq_part, nrm.ssq_n, nrm.eps, epi);                                                                            \
    else                                                                                                              \
      launch_gemm_kernel(k_gemm_bf16<ct, nt, role, spw, false>, grid, block, lds, st, Wsw, X, nrm.gain, partial, K, N,   \
                         ldx, M, nrm.ssq_part, nrm.ssq_n, nrm.eps, epi);                                                                         \
  } while (0)
#define STAIRS_GEMM_NT(ct, role, spw)             \
  if (NT == 1) STAIRS_GEMM(ct, 1, role, spw);     \
  else STAIRS_GEMM(ct, 2, role, spw)
#define STAIRS_GEMM_ROLE(role)                                  \
  if (CT == 1 && SPW == 1) { STAIRS_GEMM_NT(1, role, 1); }      \
  else if (CT == 1) { STAIRS_GEMM_NT(1, role, 2); }             \
  else { STAIRS_GEMM_NT(2, role, 1); }
  switch (role) {
    case kRoleQKV: STAIRS_GEMM_ROLE(kRoleQKV); break;
    case kRoleWo: STAIRS_GEMM_ROLE(kRoleWo); break;
    case kRoleGateUp: STAIRS_GEMM_ROLE(kRoleGateUp); break;
    case kRoleDown: STAIRS_GEMM_ROLE(kRoleDown); break;
    default: STAIRS_GEMM_ROLE(kRoleHead); break;
  }
#undef STAIRS_GEMM_NT
#undef STAIRS_GEMM_ROLE
#undef STAIRS_GEMM
}
void launch_gemm(int role, int dtype_bf16, const void* W, int N, int K, const float* X, int ldx, int M, RowNorm nrm,
                 float* partial, const GemmEpi& epi, hipStream_t st, const uint4* xfrag) {
  gemm(role, dtype_bf16, W, N, K, X, ldx, M, nrm, partial, epi, st, xfrag, nullptr);
}
void launch_unembed(int dtype_bf16, const void* W, int N, int K, const float* X, int M, RowNorm nrm, float* partial, const GemmEpi& epi,
                    hipStream_t st, const uint4* xfrag, float2* cand) {
  gemm(kRoleHead, dtype_bf16, W, N, K, X, K, M, nrm, partial, epi, st, xfrag, cand);
}

// ---------------------------------------------------------------------------------------
// embedding gather, rope table
// ---------------------------------------------------------------------------------------
// bf16 models: a sum-of-squares partial per 16 residual columns (the fp32 GEMM gathers its own)
// The block column after the last embedding column copies the rotation entries of the row's position from the model's
// table instead (identity without one, and outside it).
// A row whose position lies outside [0, tok_cap) or whose token id lies outside [0, vocab) becomes a row of zeros:
// the gather never leaves the token array or the embedding table, whatever the array holds.
// columns c .. c+3 (c < d, a multiple of 4; all lanes of a quad come along) of the row of token id
template <typename E>
__device__ __forceinline__ void embed_cols(const E* emb, int id, int vocab, int d, int c, float* x, float* ssq_part, uint4* frag, int m,
                                           const float* frag_gain) {
  float ss = 0.f;
  if (c < d) {
    float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
    if (id >= 0 && id < vocab) {
      const E* row = emb + (size_t)id * d + c;
      v.x = load_elem(row); v.y = load_elem(row + 1); v.z = load_elem(row + 2); v.w = load_elem(row + 3);
    }
    *reinterpret_cast<float4*>(x + c) = v;
    ss = (v.x * v.x + v.y * v.y) + (v.z * v.z + v.w * v.w);   // (squares of bf16 values are exact: contracted or not, the same)
    if (frag) store_frag4(frag, m, c, v, frag_gain);
  }
  if (sizeof(E) == 2) {
    ss += dpp<kDppXor1>(ss);
    ss += dpp<kDppXor2>(ss);
    if ((c & 12) == 0 && c < d) ssq_part[c / 16] = ss;
  }
}
// Row `row` of the embeddings the next forward starts from, by a work-group of nth threads that all know the token: position p,
// token id (kernel that decided them: no launch of its own, no round trip through the token array).
__device__ __forceinline__ void next_embed(const NextEmbed& n, int p, int id, int nth, int row = 0) {
  const int tid = threadIdx.x;
  float2* const cs = n.cs + row * 64;
  float* const x = n.x + (size_t)row * n.d;
  float* const ssq = n.ssq_part + row * ((n.d + kSsqGroup - 1) / kSsqGroup);
  if (p < 0 || p >= n.tok_cap) id = -1;
  if (tid < n.hd / 2) cs[tid] = n.tab && p >= 0 && p < n.tab_len ? n.tab[(size_t)p * 64 + tid] : make_float2(1.f, 0.f);
  for (int c = tid * 4; c - tid * 4 < n.d; c += nth * 4) {
    if (n.bf16) embed_cols(static_cast<const uint16_t*>(n.emb), id, n.vocab, n.d, c, x, ssq, nullptr, 0, nullptr);
    else embed_cols(static_cast<const float*>(n.emb), id, n.vocab, n.d, c, x, ssq, nullptr, 0, nullptr);
  }
}
template <typename E>
__global__ __launch_bounds__(256) void k_embed(const E* __restrict__ emb, const int* __restrict__ tokens, const int* __restrict__ pos_base,
                                               int pos_offset, int pos_rps, int tok_slot_stride, int tok_cap, int vocab, int d, int ssq_n,
                                               float* __restrict__ x, float* __restrict__ ssq_part, int hd, const float2* __restrict__ tab,
                                               int tab_len, float2* __restrict__ cs, uint4* frag, const float* __restrict__ frag_gain) {
  const PosRef pos{pos_base, pos_offset, pos_rps};
  const int m = blockIdx.y;
  const int p = pos_of(pos, m);
  tokens += (size_t)slot_of(pos, m) * tok_slot_stride;
  if (blockIdx.x == gridDim.x - 1) {
    const int i = threadIdx.x;
    if (i < hd / 2) cs[m * 64 + i] = tab && p >= 0 && p < tab_len ? tab[(size_t)p * 64 + i] : make_float2(1.f, 0.f);
    return;
  }
  embed_cols(emb, p >= 0 && p < tok_cap ? tokens[p] : -1, vocab, d, (blockIdx.x * 256 + threadIdx.x) * 4, x + (size_t)m * d,
             ssq_part + (size_t)m * ssq_n, frag, m, frag_gain);
}

void launch_embed(const void* emb, int emb_bf16, const int* tokens, int tok_slot_stride, int tok_cap, int vocab, PosRef pos,
                  int M, int d, float* x, float* ssq_part, int hd, const float2* tab, int tab_len, float2* cs, hipStream_t st, uint4* frag,
                  const float* frag_gain) {
  dim3 grid((d + 1023) / 1024 + 1, M), block(256);
  const int sn = ssq_groups(d);
  if (emb_bf16)
    hipLaunchKernelGGL((k_embed<uint16_t>), grid, block, 0, st, static_cast<const uint16_t*>(emb), tokens,
                       pos.base, pos.offset, pos.rps, tok_slot_stride, tok_cap, vocab, d, sn, x, ssq_part, hd, tab, tab_len, cs, frag, frag_gain);
  else
    hipLaunchKernelGGL((k_embed<float>), grid, block, 0, st, static_cast<const float*>(emb), tokens,
                       pos.base, pos.offset, pos.rps, tok_slot_stride, tok_cap, vocab, d, sn, x, ssq_part, hd, tab, tab_len, cs, nullptr, nullptr);
}

// tab[p][i] = (cos, sin)(p * theta^(-2i/hd)), angle in double, once per model: formed in front of every forward the
// double-precision power, sine and cosine were most of the embedding kernel's 4.3 us
__global__ void k_rope_table(int hd, double theta, float2* __restrict__ tab) {
  const int p = blockIdx.x, i = threadIdx.x;
  if (i >= hd / 2) return;
  const double ang = (double)p * pow(theta, -2.0 * (double)i / (double)hd);
  tab[(size_t)p * 64 + i] = make_float2((float)cos(ang), (float)sin(ang));
}
void launch_rope_table(int len, int hd, float theta, float2* tab, hipStream_t st) {
  hipLaunchKernelGGL(k_rope_table, dim3(len), dim3(64), 0, st, hd, (double)theta, tab);
}
__global__ void k_rope_rows(PosRef pos, int hd, const float2* __restrict__ tab, int tab_len, float2* __restrict__ cs) {
  const int m = blockIdx.x, i = threadIdx.x, p = pos_of(pos, m);
  if (i < hd / 2) cs[m * 64 + i] = p >= 0 && p < tab_len ? tab[(size_t)p * 64 + i] : make_float2(1.f, 0.f);
}
void launch_rope_rows(PosRef pos, int M, int hd, const float2* tab, int tab_len, float2* cs, hipStream_t st) {
  hipLaunchKernelGGL(k_rope_rows, dim3(M), dim3(64), 0, st, pos, hd, tab, tab_len, cs);
}

// ---------------------------------------------------------------------------------------
// fp32 caches: work-group = (128-key chunk, head, MR query rows: attn_f32_rows).
// The chunk's keys, then its values, are staged in LDS; every load of a chunk is in flight at once (with a loop over the
// staged pieces a chunk was 8 round trips to memory in a row), the values while the scores are formed.
// Chunk boundaries are absolute key positions and chunks are combined in index order; a launch of one chunk writes
// the result itself, with the bits the merge of one chunk has.  Neither MR nor the launch changes a row's bits.
// (4 heads of 64, contexts up to 96, 1 / 5 rows: 6.7 / 12.3 us and 3.3 us of merge -> 4.7 us)
// ---------------------------------------------------------------------------------------
template <int HD, int MR, bool DIRECT>
__global__ __launch_bounds__(256) void k_attn(const float* __restrict__ q, const float* __restrict__ Kc,
                                              const float* __restrict__ Vc, const int* __restrict__ pos_base, int pos_offset, int cap, int d, int M,
                                              float* __restrict__ out, float scale, int H, int nchunk_cap, float* __restrict__ part_o,
                                              float* __restrict__ part_ml) {
  constexpr int ROW = HD + 4;              // padded LDS row
  constexpr int VPR = HD / 4;              // 16-byte vectors per key
  constexpr int VPT = VPR / 2;             // vectors per thread of a chunk
  constexpr int PARTS = 256 / HD;          // the keys of a chunk are summed in that many runs, added in order
  extern __shared__ uint4 smem_u4[];
  float* s_kv = reinterpret_cast<float*>(smem_u4);                             // [128][ROW]
  float* s_q = s_kv + 128 * ROW;                                               // [MR][HD]
  float* s_p = s_q + MR * HD;                                                  // [MR][128]
  float* s_ml = s_p + MR * 128;                                                // [MR][2]
  float* s_o = s_ml + MR * 2 + 2 * (MR & 1);                                   // [MR][256]

  const int c = blockIdx.x, h = blockIdx.y, row0 = blockIdx.z * MR;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int pos0 = *pos_base + pos_offset;
  const int rows = min(MR, M - row0);      // valid query rows of this group
  const int kv_len = MR == 1 ? pos0 + row0 + 1 : pos0 + M;
  const int key0 = c * kAttnChunk;
  if (key0 >= kv_len) {
    if (DIRECT && tid < HD)                // no position of these rows exists
      for (int i = 0; i < rows; ++i) out[(size_t)(row0 + i) * d + h * HD + tid] = 0.f;
    return;
  }
  const int nkeys = min(kAttnChunk, kv_len - key0);

  float4 kr[VPT], vr[VPT];
  const float4* ksrc = reinterpret_cast<const float4*>(Kc + ((size_t)h * cap + key0) * HD);
  const float4* vsrc = reinterpret_cast<const float4*>(Vc + ((size_t)h * cap + key0) * HD);
  const int nvec = nkeys * VPR;            // (vectors past the last key are read as the last vector)
#pragma unroll
  for (int u = 0; u < VPT; ++u) kr[u] = ksrc[min(u * 256 + tid, nvec - 1)];
#pragma unroll
  for (int u = 0; u < VPT; ++u) vr[u] = vsrc[min(u * 256 + tid, nvec - 1)];
  for (int idx = tid; idx < MR * HD; idx += 256) {
    const int i = idx / HD, e = idx - i * HD;
    s_q[idx] = (i < rows) ? q[(size_t)(row0 + i) * d + h * HD + e] : 0.f;
  }
#pragma unroll
  for (int u = 0; u < VPT; ++u) {
    const int idx = u * 256 + tid, r = idx / VPR, cc = idx - r * VPR;
    *reinterpret_cast<float4*>(s_kv + r * ROW + cc * 4) = kr[u];
  }
  __syncthreads();

  {                                        // two neighbouring lanes per key, alternate quadruples of the dimensions
    const int key = tid >> 1, part = tid & 1;
    float sacc[MR];
#pragma unroll
    for (int i = 0; i < MR; ++i) sacc[i] = 0.f;
    const float* krow = s_kv + key * ROW + part * 4;
#pragma unroll 4
    for (int e0 = 0; e0 < HD; e0 += 8) {
      const float4 kf = *reinterpret_cast<const float4*>(krow + e0);
#pragma unroll
      for (int i = 0; i < MR; ++i) {
        const float4 qf = *reinterpret_cast<const float4*>(s_q + i * HD + part * 4 + e0);
        sacc[i] = fmaf(qf.w, kf.w, fmaf(qf.z, kf.z, fmaf(qf.y, kf.y, fmaf(qf.x, kf.x, sacc[i]))));
      }
    }
#pragma unroll
    for (int i = 0; i < MR; ++i) {
      const float sum = __fadd_rn(sacc[i], __shfl_xor(sacc[i], 1));
      const bool ok = (key < nkeys) && (i < rows) && (key0 + key <= pos0 + row0 + i);
      if (part == 0) s_p[i * 128 + key] = ok ? sum * scale : -INFINITY;
    }
  }
  __syncthreads();   // everybody is done with the keys; scores are in LDS

#pragma unroll
  for (int u = 0; u < VPT; ++u) {
    const int idx = u * 256 + tid, r = idx / VPR, cc = idx - r * VPR;
    *reinterpret_cast<float4*>(s_kv + r * ROW + cc * 4) = idx < nvec ? vr[u] : make_float4(0.f, 0.f, 0.f, 0.f);
  }
  for (int i = wave; i < MR; i += 4) {
    const float a = s_p[i * 128 + lane], b = s_p[i * 128 + lane + 64];
    const float mx = wave_max(fmaxf(a, b));
    float pa = 0.f, pb = 0.f;
    if (mx != -INFINITY) {
      pa = expf(a - mx);
      pb = expf(b - mx);
    }
    const float l = wave_sum(pa + pb);
    s_p[i * 128 + lane] = pa;
    s_p[i * 128 + lane + 64] = pb;
    if (lane == 0) {
      s_ml[i * 2] = mx;
      s_ml[i * 2 + 1] = l;
    }
  }
  __syncthreads();

  {
    const int e = tid % HD, t0 = tid / HD * (128 / PARTS);
    float o[MR];
#pragma unroll
    for (int i = 0; i < MR; ++i) o[i] = 0.f;
#pragma unroll 2
    for (int t = t0; t < t0 + 128 / PARTS; t += 8) {   // (keys past the last one: probability 0, values 0)
      float v[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = s_kv[(t + j) * ROW + e];
#pragma unroll
      for (int i = 0; i < MR; ++i) {
        const float4 p0 = *reinterpret_cast<const float4*>(s_p + i * 128 + t), p1 = *reinterpret_cast<const float4*>(s_p + i * 128 + t + 4);
        o[i] = fmaf(p0.w, v[3], fmaf(p0.z, v[2], fmaf(p0.y, v[1], fmaf(p0.x, v[0], o[i]))));
        o[i] = fmaf(p1.w, v[7], fmaf(p1.z, v[6], fmaf(p1.y, v[5], fmaf(p1.x, v[4], o[i]))));
      }
    }
#pragma unroll
    for (int i = 0; i < MR; ++i) s_o[i * 256 + tid] = o[i];
  }
  __syncthreads();
  if (tid < HD)
    for (int i = 0; i < rows; ++i) {
      float o = s_o[i * 256 + tid];
#pragma unroll
      for (int part = 1; part < PARTS; ++part) o = __fadd_rn(o, s_o[i * 256 + part * HD + tid]);
      if (DIRECT) out[(size_t)(row0 + i) * d + h * HD + tid] = pos0 + row0 + i < 0 ? 0.f : o / s_ml[i * 2 + 1];
      else part_o[(((size_t)(row0 + i) * H + h) * nchunk_cap + c) * HD + tid] = o;
    }
  if (!DIRECT && tid < rows) {
    float* ml = part_ml + (((size_t)(row0 + tid) * H + h) * nchunk_cap + c) * 2;
    ml[0] = s_ml[tid * 2];
    ml[1] = s_ml[tid * 2 + 1];
  }
}

template <int HD>
__global__ void k_attn_combine(const float* __restrict__ part_o, const float* __restrict__ part_ml, int H, PosRef pos,
                               int nchunk_cap, float* __restrict__ out, int d) {
  const int h = blockIdx.x, m = blockIdx.y, e = threadIdx.x;
  const int p = *pos.base + pos.offset + m;
  float* dst = out + (size_t)m * d + h * HD + e;
  if (p < 0) {
    *dst = 0.f;
    return;
  }
  const int nch = p / kAttnChunk + 1;
  const size_t base = ((size_t)m * H + h) * nchunk_cap;
  float gmax = -INFINITY;
  for (int c = 0; c < nch; ++c) gmax = fmaxf(gmax, part_ml[(base + c) * 2]);
  float num = 0.f, den = 0.f;
  for (int c = 0; c < nch; ++c) {
    const float mc = part_ml[(base + c) * 2];
    if (mc == -INFINITY) continue;
    const float w = expf(mc - gmax);
    num = fmaf(w, part_o[(base + c) * HD + e], num);
    den = fmaf(w, part_ml[(base + c) * 2 + 1], den);
  }
  *dst = num / den;
}

// ---------------------------------------------------------------------------------------
// KV-cache attention for half-precision caches, MFMA 16x16x32 f16.
//   Cache layout (per layer, per head): keys in 16-position blocks stored as MFMA A tiles
//   [16 keys x 32 dims] (k_cache_off), values in 32-position blocks stored as A tiles of V^T
//   [16 dims x 32 key slots] whose slot order is the one the score tiles come out in (v_cache_off),
//   so neither K, V nor the probabilities ever pass through LDS for a transpose.
//   Work-group = (128-key chunk at an absolute position, head); wave w owns keys 32w..32w+31 of the
//   chunk: scores^T = K . q^T (q as half hi+lo), masked softmax over its 32 keys, out^T = V^T . p^T
//   (p as half hi+lo).  The four waves are merged in LDS in wave order, the chunks of a head by the
//   work-group that arrives last at the head's counter, in chunk order.
// ---------------------------------------------------------------------------------------
// the attention output's fragments, in the layout the next projection reads (AttnMode::frag_rt)
__device__ __forceinline__ void store_attn_frag4(uint4* frag, int frag_rt, int m, int k, float4 v) {
  if (frag_rt > 0) blk_store_frag4(frag, frag_rt, m, k, v);
  else store_frag4(frag, m, k, v, nullptr);
}

// Merge of the chunk partials of one head (one slot): out[m] = sum_c w_c o_c / sum_c w_c l_c with w_c = exp(max_c - max).
// Step A: all (max, sum) pairs of all rows go to LDS in one round trip, then the row maxima and, in place of the chunk
// maxima, the weights w_c (one exp per row and chunk; formed per thread they made up most of the merge's time).
// Step B, up to kMergeCB chunks: one thread per (row, 4 adjacent dims) adds its chunks up in chunk order, all loads in
// flight together.
// More chunks: groups of kMergeCB chunks are summed by different threads in parallel (each as above, from zero) and the
// group sums added in group order; the grouping depends only on the row's own position.  Dynamic LDS:
// [M][nch_lds][2] pairs (weight, sum), [kMaxRows] unused, [M][HD/4][groups][5] group sums (see launch_attention).
constexpr int kMergeCB = 20;
// Step A of the merge: the (weight, sum) table of all rows and chunks in LDS (see attn_merge)
__device__ __forceinline__ void attn_merge_table(const float* part_ml, int H, int h, int M, int pos0, int step, int nch_max,
                                                 int nchunk_cap, int nch_lds, float* s_ml) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  for (int idx = tid; idx < M * nch_max; idx += 256) {
    const int m = idx / nch_max, cc = idx - m * nch_max;
    const float2 ml = ld_dev2(&part_ml[(((size_t)m * H + h) * nchunk_cap + cc) * 2]);
    s_ml[((size_t)m * nch_lds + cc) * 2] = ml.x;
    s_ml[((size_t)m * nch_lds + cc) * 2 + 1] = ml.y;
  }
  __syncthreads();
  if (nch_max <= 16) {
    // few chunks: 16 lanes per row, four rows per wave at a time (max is exact in any order)
    const int cc = lane & 15;
    for (int m = wave * 4 + (lane >> 4); m < M; m += 16) {
      const int p = pos0 + m * step;
      const int nch = p >= 0 ? p / kAttnChunkH + 1 : 0;
      const float mc = cc < nch ? s_ml[((size_t)m * nch_lds + cc) * 2] : -INFINITY;
      float g = mc;
#pragma unroll
      for (int off = 8; off >= 1; off >>= 1) g = fmaxf(g, __shfl_xor(g, off));
      if (cc < nch) s_ml[((size_t)m * nch_lds + cc) * 2] = (mc == -INFINITY) ? 0.f : exp_fast(mc - g);
    }
    __syncthreads();
    return;
  }
  for (int m = wave; m < M; m += 4) {                 // row maxima (max is exact in any order)
    const int p = pos0 + m * step;
    const int nch = p >= 0 ? p / kAttnChunkH + 1 : 0;
    float g = -INFINITY;
    for (int cc = lane; cc < nch; cc += 64) g = fmaxf(g, s_ml[((size_t)m * nch_lds + cc) * 2]);
    g = wave_max(g);
    // the chunk weights, once per (row, chunk) instead of once per thread that uses them: each replaces its chunk's
    // maximum in the table (the lane that read the slot writes it)
    for (int cc = lane; cc < nch; cc += 64) {
      const float mc = s_ml[((size_t)m * nch_lds + cc) * 2];
      s_ml[((size_t)m * nch_lds + cc) * 2] = (mc == -INFINITY) ? 0.f : exp_fast(mc - g);
    }
  }
  __syncthreads();
}

// The merge for at most CB chunks: a thread takes IPT items (row, 4 adjacent dims) per pass and requests all their
// chunks' outputs before the table is built -- they do not depend on it, so the merge's two round trips to memory
// become one -- then adds them up in chunk order, from zero (the order of attn_merge's step B).
template <int HD, int CB, int IPT>
__device__ __forceinline__ void attn_merge_direct(const float* part_o, const float* part_ml, int H, int h, int M, int pos0,
                                                  int step, int nch_max, int nchunk_cap, int nch_lds, float* out, int d,
                                                  float* s_ml, uint4* frag, int frag_rt, int frag_row0) {
  constexpr int QPR = HD / 4;                         // threads per row
  const int tid = threadIdx.x, items = M * QPR;
  float2 va[IPT][CB], vb[IPT][CB];
  // (a chunk past the row's last re-reads its last: no condition inside an item's requests)
#define STAIRS_MERGE_LOADS(base)                                                         \
  _Pragma("unroll") for (int ip = 0; ip < IPT; ++ip) {                                   \
    const int idx = (base) + ip * 256 + tid;                                             \
    if (idx < items) {                                                                   \
      const int m = idx / QPR, e = (idx - m * QPR) * 4;                                  \
      const int p = pos0 + m * step;                                                     \
      const int last = p >= 0 ? p / kAttnChunkH : 0;                                     \
      const float* src = part_o + ((size_t)m * H + h) * nchunk_cap * HD + e;             \
      _Pragma("unroll") for (int i = 0; i < CB; ++i) {                                   \
        const float* q = src + (size_t)min(i, last) * HD;                                \
        va[ip][i] = ld_dev2(q);                                                          \
        vb[ip][i] = ld_dev2(q + 2);                                                      \
      }                                                                                  \
    }                                                                                    \
  }
  STAIRS_MERGE_LOADS(0);
  attn_merge_table(part_ml, H, h, M, pos0, step, nch_max, nchunk_cap, nch_lds, s_ml);
  for (int base = 0; base < items; base += 256 * IPT) {
    if (base > 0) { STAIRS_MERGE_LOADS(base); }
#pragma unroll
    for (int ip = 0; ip < IPT; ++ip) {
      const int idx = base + ip * 256 + tid;
      if (idx < items) {
        const int m = idx / QPR, e = (idx - m * QPR) * 4;
        const int p = pos0 + m * step;
        float4 res = make_float4(0.f, 0.f, 0.f, 0.f);
        if (p >= 0) {
          const int nch = p / kAttnChunkH + 1;
          const float* mlr = s_ml + (size_t)m * nch_lds * 2;
          float4 num = make_float4(0.f, 0.f, 0.f, 0.f);
          float den = 0.f;
#pragma unroll
          for (int i = 0; i < CB; ++i) {
            if (i < nch) {
              const float w = mlr[i * 2];
              num.x = fmaf(w, va[ip][i].x, num.x); num.y = fmaf(w, va[ip][i].y, num.y);
              num.z = fmaf(w, vb[ip][i].x, num.z); num.w = fmaf(w, vb[ip][i].y, num.w);
              den = fmaf(w, mlr[i * 2 + 1], den);
            }
          }
          res = make_float4(num.x / den, num.y / den, num.z / den, num.w / den);
        }
        *reinterpret_cast<float4*>(out + (size_t)m * d + h * HD + e) = res;
        if (frag) store_attn_frag4(frag, frag_rt, frag_row0 + m, h * HD + e, res);
      }
    }
  }
#undef STAIRS_MERGE_LOADS
}

template <int HD>
__device__ __forceinline__ void attn_merge(const float* part_o, const float* part_ml, int H, int h, int M, int pos0, int step,
                                           int kv_len, int nchunk_cap, int nch_lds, float* out, int d, float* s_ml,
                                           uint4* frag, int frag_rt, int frag_row0) {
  const int tid = threadIdx.x;
  const int nch_max = (kv_len > 0) ? (kv_len - 1) / kAttnChunkH + 1 : 0;
  if (nch_max <= kMergeCB / 2)                        // (no chunk at all: every row gets zeros)
    return attn_merge_direct<HD, kMergeCB / 2, 2>(part_o, part_ml, H, h, M, pos0, step, nch_max, nchunk_cap, nch_lds, out, d,
                                                  s_ml, frag, frag_rt, frag_row0);
  if (nch_max <= kMergeCB)
    return attn_merge_direct<HD, kMergeCB, 1>(part_o, part_ml, H, h, M, pos0, step, nch_max, nchunk_cap, nch_lds, out, d,
                                              s_ml, frag, frag_rt, frag_row0);
  // more chunks: groups of kMergeCB chunks summed in parallel, the group sums added in group order
  float* grp = s_ml + (size_t)M * nch_lds * 2 + kMaxRows;   // (kMaxRows floats after the table stay unused)
  attn_merge_table(part_ml, H, h, M, pos0, step, nch_max, nchunk_cap, nch_lds, s_ml);
  constexpr int QPR = HD / 4;                         // threads per row
  constexpr int CB = kMergeCB;
  const int G = (nch_max + CB - 1) / CB;
  // sum of the chunks [c0, c1) of row m, dims e..e+3, weighted; all loads of the (at most CB) chunks together
  auto group_sum = [&](int m, int e, int c0, int c1, float4& num, float& den) {
    const float* mlr = s_ml + (size_t)m * nch_lds * 2;
    const float* src = part_o + ((size_t)m * H + h) * nchunk_cap * HD + e;
    float2 va[CB], vb[CB];
#pragma unroll
    for (int i = 0; i < CB; ++i) {
      const float* q = src + (size_t)min(c0 + i, c1 - 1) * HD;
      va[i] = ld_dev2(q);
      vb[i] = ld_dev2(q + 2);
    }
#pragma unroll
    for (int i = 0; i < CB; ++i) {
      if (c0 + i < c1) {
        const float w = mlr[(c0 + i) * 2];
        num.x = fmaf(w, va[i].x, num.x); num.y = fmaf(w, va[i].y, num.y);
        num.z = fmaf(w, vb[i].x, num.z); num.w = fmaf(w, vb[i].y, num.w);
        den = fmaf(w, mlr[(c0 + i) * 2 + 1], den);
      }
    }
  };
  for (int idx = tid; idx < M * QPR * G; idx += 256) {
    const int g = idx % G, rq = idx / G;
    const int m = rq / QPR, e = (rq - m * QPR) * 4;
    const int p = pos0 + m * step;
    float4 num = make_float4(0.f, 0.f, 0.f, 0.f);
    float den = 0.f;
    if (p >= 0) {
      const int nch = p / kAttnChunkH + 1;
      if (g * CB < nch) group_sum(m, e, g * CB, min(nch, (g + 1) * CB), num, den);
    }
    float* o = grp + (size_t)idx * 5;
    o[0] = num.x; o[1] = num.y; o[2] = num.z; o[3] = num.w; o[4] = den;
  }
  __syncthreads();
  for (int idx = tid; idx < M * QPR; idx += 256) {
    const int m = idx / QPR, e = (idx - m * QPR) * 4;
    const int p = pos0 + m * step;
    float4 res = make_float4(0.f, 0.f, 0.f, 0.f);
    if (p >= 0) {
      const int ng = (p / kAttnChunkH + 1 + CB - 1) / CB;
      float4 num = make_float4(0.f, 0.f, 0.f, 0.f);
      float den = 0.f;
      for (int g = 0; g < ng; ++g) {
        const float* o = grp + ((size_t)idx * G + g) * 5;
        num.x += o[0]; num.y += o[1]; num.z += o[2]; num.w += o[3]; den += o[4];
      }
      res = make_float4(num.x / den, num.y / den, num.z / den, num.w / den);
    }
    *reinterpret_cast<float4*>(out + (size_t)m * d + h * HD + e) = res;
    if (frag) store_attn_frag4(frag, frag_rt, frag_row0 + m, h * HD + e, res);
  }
}

// (two work-groups per CU: the register budget that keeps both resident)
template <int HD, int CT, bool FUSED>
__global__ __launch_bounds__(256, 2) void k_attn_f16(const float* __restrict__ q, const _Float16* __restrict__ Kc,
                                                  const _Float16* __restrict__ Vc, const int* __restrict__ pos_base, int pos_offset, int pos_rps,
                                                  int cap, int d, int M, int early_keys, size_t kv_slot_stride, float scale, int H, AttnMode am,
                                                  int nchunk_cap, float* part_o, float* part_ml, int* counters,
                                                  float* __restrict__ out) {
  const PosRef pos{pos_base, pos_offset, pos_rps};
  const int kv_fixed = max(0, -early_keys);
  constexpr int KK = HD / 32;   // k-steps of the score MFMA
  constexpr int ET = HD / 16;   // output-dim tiles of the value MFMA
  __shared__ float s_o[4][16][HD + 4];               // (+4: the 16 rows a wave writes at once fall into different banks)
  __shared__ float s_m[4][16], s_l[4][16];
  __shared__ int s_last;
  const int c = blockIdx.x, h = blockIdx.y;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int j = lane & 15, g = lane >> 4;
  // several sequences: blockIdx.z is the slot; its M = pos.rps rows, caches, partial results and counters follow
  // those of the slots before it, and everything below sees only this slot
  const int row0 = blockIdx.z * M;
  q += (size_t)row0 * d;
  out += (size_t)row0 * d;
  part_o += (size_t)row0 * H * nchunk_cap * HD;
  part_ml += (size_t)row0 * H * nchunk_cap * 2;
  counters += blockIdx.z * H;
  if (blockIdx.z > 0) {                              // (one slot: no wait for the stride)
    Kc += blockIdx.z * kv_slot_stride;
    Vc += blockIdx.z * kv_slot_stride;
  }
  // a wave owns 64 keys of the chunk as two blocks of 32 (the tiles of the cache layout)
  const int kb = c * kAttnChunkH + wave * 64;         // first key of this wave
  // The first query tile's rows are requested before the keys and values (they come from L2 and are converted while the
  // cache tiles are still on their way), and the wave's whole share of the chunk at once (keys and values of both
  // blocks: 16 KiB at head_dim 128).  Keys below early_keys (attn_early_keys) are requested before the rows' position has
  // come back from memory, a round trip less in front of every head; positions of a block past the last key hold finite
  // numbers and meet probability 0.
  float4 qa0[KK], qb0[KK];
  uint4 kreg[2][2][KK], vreg[2][ET];
  auto request = [&](bool first, bool second) {
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      qa0[kk] = make_float4(0.f, 0.f, 0.f, 0.f);
      qb0[kk] = qa0[kk];
      if (first && j < M) {
        const float4* qp = reinterpret_cast<const float4*>(q + (size_t)j * d + h * HD + kk * 32 + g * 8);
        qa0[kk] = qp[0];
        qb0[kk] = qp[1];
      }
    }
    const uint4* Kh = reinterpret_cast<const uint4*>(Kc + (size_t)h * cap * HD);
    const uint4* Vh = reinterpret_cast<const uint4*>(Vc + (size_t)h * cap * HD);
#pragma unroll
    for (int sb = 0; sb < 2; ++sb) {
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) kreg[sb][t][kk] = make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
      for (int et = 0; et < ET; ++et) vreg[sb][et] = make_uint4(0u, 0u, 0u, 0u);
      if (sb ? second : first) {
        const int kbs = kb + 32 * sb;
        // (the two-kernel form runs at long contexts only, where a layer's keys and values exceed what the memory-side
        // cache could keep until the next forward: streaming loads there, as for the weights of a large model)
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
          for (int kk = 0; kk < KK; ++kk) {
            const uint4* p = &Kh[((size_t)((kbs >> 4) + t) * KK + kk) * 64 + lane];
            kreg[sb][t][kk] = FUSED ? *p : ld_nt(p);
          }
#pragma unroll
        for (int et = 0; et < ET; ++et) {
          const uint4* p = &Vh[((size_t)(kbs >> 5) * ET + et) * 64 + lane];
          vreg[sb][et] = FUSED ? *p : ld_nt(p);
        }
      }
    }
  };
  // (one request site: with a second one for the other chunks the registers of both spill)
  const int len0 = kv_fixed > 0 ? kv_fixed : kb + 32 < early_keys ? early_keys : pos_of(pos, row0) + M;
  request(kb < len0, kb + 32 < len0);
  // causal: row i sees the keys 0 .. qpos0 + i; fixed key set (kv_fixed > 0): every row sees the keys 0 .. kv_fixed-1
  const int qpos0 = pos_of(pos, row0);
  const bool fixed = kv_fixed > 0;   // (then also for rows that sit nowhere: their result is unused)
  const int pos0 = fixed ? kv_fixed - 1 : qpos0;   // last key row 0 sees
  const int step = fixed ? 0 : 1;
  const int kv_len = pos0 + (fixed ? 1 : M);
  const float* brow = am.bias ? am.bias + (size_t)h * am.bias_ld + am.bias_zero : nullptr;
  const bool have_keys = kb < kv_len;
  // all keys in the first chunk: its work-group writes the result itself (what the merge would give for one chunk:
  // weight exp(0) = 1), the others have nothing to do; no partial results, no ticket
  const bool single = FUSED && kv_len <= kAttnChunkH;
  if (single && c > 0) return;

#pragma unroll
  for (int ct = 0; ct < CT; ++ct) {
    const int qi = ct * 16 + j;                      // this lane's query row
    f32x4 oacc[ET];
#pragma unroll
    for (int et = 0; et < ET; ++et) oacc[et] = f32x4{0.f, 0.f, 0.f, 0.f};
    float mw = -INFINITY, lw = 0.f;
    if (have_keys) {
      f16x8 qh[KK], ql[KK];
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) {
        const float4 a = qa0[kk], b = qb0[kk];
        const float v[8] = {a.x * scale, a.y * scale, a.z * scale, a.w * scale,
                            b.x * scale, b.y * scale, b.z * scale, b.w * scale};
        split_half8(v, qh[kk], ql[kk]);
      }
      // the next query tile's rows are requested now, into the registers just converted: they arrive while this
      // tile's scores and outputs are computed
      if (ct + 1 < CT) {
        const int qn = (ct + 1) * 16 + j;
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) {
          qa0[kk] = make_float4(0.f, 0.f, 0.f, 0.f);
          qb0[kk] = qa0[kk];
          if (qn < M) {
            const float4* qp = reinterpret_cast<const float4*>(q + (size_t)qn * d + h * HD + kk * 32 + g * 8);
            qa0[kk] = qp[0];
            qb0[kk] = qp[1];
          }
        }
      }
      // scores of the wave's 64 keys, their joint maximum, the exponentials, then the two value products
      float sc[2][8];
#pragma unroll
      for (int sb = 0; sb < 2; ++sb) {
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          f32x4 sacc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int kk = 0; kk < KK; ++kk) {
            const f16x8 a = __builtin_bit_cast(f16x8, kreg[sb][t][kk]);
            sacc = __builtin_amdgcn_mfma_f32_16x16x32_f16(a, qh[kk], sacc, 0, 0, 0);
            sacc = __builtin_amdgcn_mfma_f32_16x16x32_f16(a, ql[kk], sacc, 0, 0, 0);
          }
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const int key = kb + sb * 32 + t * 16 + g * 4 + v;
            const bool seen = qi < M && key <= pos0 + qi * step;
            const float bv = (brow && seen) ? brow[key - (qpos0 + qi)] : 0.f;   // bias by key position - query position
            sc[sb][t * 4 + v] = seen ? sacc[v] + bv : -INFINITY;
          }
        }
      }
      float mx = sc[0][0];
#pragma unroll
      for (int i = 1; i < 8; ++i) mx = fmaxf(mx, sc[0][i]);
#pragma unroll
      for (int i = 0; i < 8; ++i) mx = fmaxf(mx, sc[1][i]);
      mx = fmaxf(mx, __shfl_xor(mx, 16));
      mx = fmaxf(mx, __shfl_xor(mx, 32));
      float sum = 0.f;
      f16x8 ph[2], pl[2];
#pragma unroll
      for (int sb = 0; sb < 2; ++sb) {
        float pv[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          pv[i] = (mx == -INFINITY) ? 0.f : exp_fast(sc[sb][i] - mx);
          sum += pv[i];
        }
        split_half8(pv, ph[sb], pl[sb]);
      }
      sum += __shfl_xor(sum, 16);
      sum += __shfl_xor(sum, 32);
      mw = mx;
      lw = sum;
#pragma unroll
      for (int sb = 0; sb < 2; ++sb)
#pragma unroll
        for (int et = 0; et < ET; ++et) {
          const f16x8 a = __builtin_bit_cast(f16x8, vreg[sb][et]);
          oacc[et] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a, ph[sb], oacc[et], 0, 0, 0);
          oacc[et] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a, pl[sb], oacc[et], 0, 0, 0);
        }
    }
    // merge the four waves (wave order): every wave leaves its maximum, its sum and its output rows as they are; the
    // threads that add the four outputs up scale them by exp(max_w - max) on the way (product rounded, then added)
    if (ct > 0) __syncthreads();                     // LDS of the previous query tile has been read
    if (g == 0) {
      s_m[wave][j] = mw;
      s_l[wave][j] = lw;
    }
    if (qi < M) {                                    // rows past the last one are never read back
#pragma unroll
      for (int et = 0; et < ET; ++et)
        *reinterpret_cast<float4*>(&s_o[wave][j][et * 16 + g * 4]) =
            make_float4(oacc[et][0], oacc[et][1], oacc[et][2], oacc[et][3]);
    }
    __syncthreads();
    const int rows_here = min(16, M - ct * 16);      // (<= 0 for a second tile no row falls into)
    // (a thread takes 4 adjacent dims of a row: 16 rows are two passes of the 256 threads)
    for (int idx = tid; idx < rows_here * (HD / 4); idx += 256) {
      const int jj = idx / (HD / 4), e = (idx - jj * (HD / 4)) * 4;
      const int m = ct * 16 + jj;
      if (m < M) {
        const float m0 = s_m[0][jj], m1 = s_m[1][jj], m2 = s_m[2][jj], m3 = s_m[3][jj];
        const float mcc = fmaxf(fmaxf(m0, m1), fmaxf(m2, m3));
        const float f0 = (m0 == -INFINITY) ? 0.f : exp_fast(m0 - mcc), f1 = (m1 == -INFINITY) ? 0.f : exp_fast(m1 - mcc);
        const float f2 = (m2 == -INFINITY) ? 0.f : exp_fast(m2 - mcc), f3 = (m3 == -INFINITY) ? 0.f : exp_fast(m3 - mcc);
        const float4 a0 = *reinterpret_cast<const float4*>(&s_o[0][jj][e]), a1 = *reinterpret_cast<const float4*>(&s_o[1][jj][e]);
        const float4 a2 = *reinterpret_cast<const float4*>(&s_o[2][jj][e]), a3 = *reinterpret_cast<const float4*>(&s_o[3][jj][e]);
        const float o0 = __fadd_rn(__fadd_rn(__fadd_rn(__fmul_rn(a0.x, f0), __fmul_rn(a1.x, f1)), __fmul_rn(a2.x, f2)), __fmul_rn(a3.x, f3));
        const float o1 = __fadd_rn(__fadd_rn(__fadd_rn(__fmul_rn(a0.y, f0), __fmul_rn(a1.y, f1)), __fmul_rn(a2.y, f2)), __fmul_rn(a3.y, f3));
        const float o2 = __fadd_rn(__fadd_rn(__fadd_rn(__fmul_rn(a0.z, f0), __fmul_rn(a1.z, f1)), __fmul_rn(a2.z, f2)), __fmul_rn(a3.z, f3));
        const float o3 = __fadd_rn(__fadd_rn(__fadd_rn(__fmul_rn(a0.w, f0), __fmul_rn(a1.w, f1)), __fmul_rn(a2.w, f2)), __fmul_rn(a3.w, f3));
        // the chunk's sum of exponentials (a wave without keys has weight 0 and sum 0: it adds nothing); no branch
        // around the LDS reads
        const float l0 = s_l[0][jj], l1 = s_l[1][jj], l2 = s_l[2][jj], l3 = s_l[3][jj];
        const float lc = __fadd_rn(__fadd_rn(__fadd_rn(__fmul_rn(f0, l0), __fmul_rn(f1, l1)), __fmul_rn(f2, l2)), __fmul_rn(f3, l3));
        if (single) {
          float4 res = make_float4(0.f, 0.f, 0.f, 0.f);
          if (pos0 + m * step >= 0) res = make_float4(o0 / lc, o1 / lc, o2 / lc, o3 / lc);
          *reinterpret_cast<float4*>(out + (size_t)m * d + h * HD + e) = res;
          if (am.frag_out) store_attn_frag4(am.frag_out, am.frag_rt, row0 + m, h * HD + e, res);
        } else {
          float* po = &part_o[(((size_t)m * H + h) * nchunk_cap + c) * HD + e];
          st_dev2(po, o0, o1);
          st_dev2(po + 2, o2, o3);
          // the thread with the row's first dims also leaves the chunk's (max, sum) pair
          if (e == 0) st_dev2(part_ml + (((size_t)m * H + h) * nchunk_cap + c) * 2, mcc, lc);
        }
      }
    }
  }

  // FUSED: the work-group that arrives last at the head's counter merges the chunks; otherwise a second kernel does
  if (!FUSED || single) return;
  if (!last_arrival(&counters[h], (int)gridDim.x, &s_last)) return;
  extern __shared__ float s_ml[];
  attn_merge<HD>(part_o, part_ml, H, h, M, pos0, step, kv_len, nchunk_cap, (int)gridDim.x, out, d, s_ml,
                 am.frag_out, am.frag_rt, row0);
  if (tid == 0) counters[h] = 0;
}

// the merge alone (long contexts: the attention work-groups then leave without waiting for their stores), a work-group per head and
// row (a head's rows one after the other in one: 32 heads of 128, 33 chunks, 5 rows 8.1 -> 4.9 us)
template <int HD>
__global__ __launch_bounds__(256) void k_attn_merge(const float* part_o, const float* part_ml, const int* __restrict__ pos_base, int pos_offset,
                                                    int pos_rps, int d, int H, int M, int kv_fixed, int nchunk_cap, int nch_lds,
                                                    float* __restrict__ out, uint4* frag, int frag_rt) {
  const PosRef pos{pos_base, pos_offset, pos_rps};
  extern __shared__ float s_ml[];
  const int h = blockIdx.x, row = blockIdx.y * M + blockIdx.z;
  const int last = kv_fixed > 0 ? kv_fixed - 1 : pos_of(pos, row);     // last key the row sees
  attn_merge<HD>(part_o + (size_t)row * H * nchunk_cap * HD, part_ml + (size_t)row * H * nchunk_cap * 2, H, h, 1, last, 0, last + 1,
                 nchunk_cap, nch_lds, out + (size_t)row * d, d, s_ml, frag, frag_rt, row);
}

// Query rows a work-group of the fp32 attention takes.  Up to 8 rows: one, as long as that makes fewer than 1024 groups (four
// per CU): the loads of a chunk are what a group waits for.  With more of them the chunk is read once per row, and 4 rows
// share it (32 heads of 64, 8 rows at 1024 / 2048 / 4096 / 8192 keys: 18.9 / 37.2 / 97.4 / 185 us by single rows, 14.5 /
// 26.8 / 48.5 / 86.1 by four; 16 heads, 5 rows, 512 keys: 8.7 against 9.9).
int attn_f32_rows(int units, int H, int M) { return M > 8 ? 16 : M > 1 && units > 1 && units * H * M >= 1024 ? 4 : 1; }

template <int HD>
static void attn_dispatch(const float* q, const float* K, const float* V, int cap, int d, int H, int M, PosRef pos,
                          int nchunk_launch, int nchunk_cap, float* part_o, float* part_ml, float* out, hipStream_t st) {
  const float scale = 1.0f / sqrtf((float)HD);
  const int mr = attn_f32_rows(nchunk_launch, H, M);
  const dim3 grid(nchunk_launch, H, (M + mr - 1) / mr), block(256);
  const size_t lds = (size_t)(128 * (HD + 4) + mr * (HD + 128 + 2 + 256) + 2) * sizeof(float);
#define STAIRS_ATTN(mrv, direct)                                                                                          \
  hipLaunchKernelGGL((k_attn<HD, mrv, direct>), grid, block, lds, st, q, K, V, pos.base, pos.offset, cap, d, M, out, scale, H, \
                     nchunk_cap, part_o, part_ml)
  if (nchunk_launch == 1) {
    if (mr == 1) STAIRS_ATTN(1, true);
    else STAIRS_ATTN(16, true);
    return;
  }
  if (mr == 1) STAIRS_ATTN(1, false);
  else if (mr == 4) STAIRS_ATTN(4, false);
  else STAIRS_ATTN(16, false);
#undef STAIRS_ATTN
  hipLaunchKernelGGL(k_attn_combine<HD>, dim3(H, M), dim3(HD), 0, st, part_o, part_ml, H, pos, nchunk_cap, out, d);
}

// Callers round the 128-key units of a launch up to a multiple of 4 at most, so the longest rows it is sized for see more than
// (units - 4) of them: what lies below that is requested before the length is known, nothing else.  Rows may see fewer, by up to
// k - 1 keys in the early steps of a proposal, whose launches are sized for its last, and by up to k more in an iteration
// launched while the one before it runs, which is sized for all of that one's tokens: those keys lie inside the cache all the
// same, hold finite numbers and meet probability 0.  (The first chunk whole at any length: 3 rows
// at contexts of 16 / 64 / 130 / 256 keys, 16 heads of 128: 5.2 / 5.1 / 5.2 / 5.2 us, now 4.7 / 4.7 / 4.8 / 5.2; 12 heads of
// 64: 4.3 / 4.4 / 4.2 / 4.3, now 4.0 / 4.2 / 4.2 / 4.3; a head's chunk is 128 and 64 KiB.)  Several sequences: their lengths
// differ, so each work-group looks its own up (64 slots of 16 heads, 3 rows, contexts of 16..210 keys: 27.3 -> 17.9 us; 16
// of 32, 4 rows, 40..350 keys: 19.7 -> 15.8 us against requesting the first chunk whole).
int attn_early_keys(int units, int nslots) { return nslots > 1 ? 0 : std::max(0, (units - 4) * kAttnChunk + 1); }

void launch_attention(const float* q_rot, const void* Kc, const void* Vc, int kv_half, int cap, int d, int H, int M,
                      PosRef pos, int nslots, size_t kv_slot_stride, int nchunk_launch, int nchunk_cap, float* part_o,
                      float* part_ml, int* counters, float* out, hipStream_t st, const AttnMode& am) {
  const int hd = d / H;
  if (kv_half) {
    const float scale = am.scale > 0.f ? am.scale : 1.0f / sqrtf((float)hd);
    const _Float16* K = static_cast<const _Float16*>(Kc);
    const _Float16* V = static_cast<const _Float16*>(Vc);
    // the half-cache kernels take 256-key chunks: half as many work-groups as the 128-key units the callers count in
    const int units = nchunk_launch;
    nchunk_launch = (nchunk_launch * kAttnChunk + kAttnChunkH - 1) / kAttnChunkH;
    dim3 grid(nchunk_launch, H, nslots), block(256);
    const int early = am.kv_fixed > 0 ? -am.kv_fixed : attn_early_keys(units, nslots);   // (k_attn_f16: one argument for both)
    // long contexts: attention work-groups only store their partials, a second kernel merges (no wait, no ticket)
    const bool fused = nchunk_launch <= kAttnFusedMaxChunks;
    // LDS of a merge of so many rows: their (max, sum) table and, for more than kMergeCB chunks, their group sums.  Fused: at most
    // 47 KiB (32 rows, 24 chunks); by itself, a row a work-group: 17 KiB at 60000 keys.
    const int G = (nchunk_launch + kMergeCB - 1) / kMergeCB;
    auto merge_lds = [&](int rows) {
      return ((size_t)rows * (nchunk_launch * 2 + (G > 1 ? hd / 4 * G * 5 : 0)) + kMaxRows) * sizeof(float);
    };
#define STAIRS_ATTN16(hdv, ct)                                                                                              \
  if (fused)                                                                                                                \
    hipLaunchKernelGGL((k_attn_f16<hdv, ct, true>), grid, block, merge_lds(M), st, q_rot, K, V, pos.base, pos.offset, pos.rps, cap, d, M, early, \
                       kv_slot_stride, scale, H, am, nchunk_cap, part_o, part_ml, counters, out);                                              \
  else {                                                                                                                    \
    hipLaunchKernelGGL((k_attn_f16<hdv, ct, false>), grid, block, 0, st, q_rot, K, V, pos.base, pos.offset, pos.rps, cap, d, M, early, \
                       kv_slot_stride, scale, H, am, nchunk_cap, part_o, part_ml, counters, out);                                              \
    hipLaunchKernelGGL((k_attn_merge<hdv>), dim3(H, nslots, M), dim3(256), merge_lds(1), st, part_o, part_ml, pos.base, pos.offset, \
                       pos.rps, d, H, M, am.kv_fixed, nchunk_cap, nchunk_launch, out, am.frag_out, am.frag_rt);              \
  }
    if (hd == 128) {
      if (M <= 16) STAIRS_ATTN16(128, 1) else STAIRS_ATTN16(128, 2)
    } else {
      if (M <= 16) STAIRS_ATTN16(64, 1) else STAIRS_ATTN16(64, 2)
    }
#undef STAIRS_ATTN16
    return;
  }
  const float *K = static_cast<const float*>(Kc), *V = static_cast<const float*>(Vc);
  if (hd == 128) attn_dispatch<128>(q_rot, K, V, cap, d, H, M, pos, nchunk_launch, nchunk_cap, part_o, part_ml, out, st);
  else attn_dispatch<64>(q_rot, K, V, cap, d, H, M, pos, nchunk_launch, nchunk_cap, part_o, part_ml, out, st);
}

// ---------------------------------------------------------------------------------------
// per-row vocabulary argmax (ties -> lowest index) and stairs validation
// ---------------------------------------------------------------------------------------
// One work-group per row, bound by its chain: the row through one CU, compares, lane exchanges, the waves' results, the store.
// The position is requested first, the exchanges stay out of the LDS unit and the last thread reads the waves' results at once
// (32000 logits, launches of 1 and 5 rows inside a 125M call: 5.4 -> 4.8 us).  NEXT: the same work-group goes on with the token's
// embedding (5.4 us and a launch of 4.6 become 6.4 per draft token).
template <bool NEXT>
__global__ __launch_bounds__(1024) void k_argmax(const float* __restrict__ logits, int* __restrict__ out, const int* __restrict__ pos_base,
                                                 int pos_offset, int pos_rps, int ld, int V, int row0, int row_stride, int out_slot_stride,
                                                 NextEmbed next) {
  const PosRef out_pos{pos_base, pos_offset, pos_rps};
  __shared__ __align__(16) float sv[16];
  __shared__ __align__(16) int si[16];
  __shared__ int s_id;
  const int r = blockIdx.x, tid = threadIdx.x;
  const float* row = logits + (size_t)(row0 + r * row_stride) * ld;
  // (several sequences: the slot's own token array, only while it is active)
  const int o = out_pos.rps ? pos_of(out_pos, r) : (out_pos.base ? *out_pos.base : 0) + out_pos.offset + r;
  float best = -INFINITY;
  int bi = 0x7fffffff;
  // a thread walks its candidates in ascending index order, 8 loads in flight at a time
  for (int v0 = tid * 4; v0 < V; v0 += 8 * 4096) {
    float4 x[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int v = v0 + 4096 * i;
      x[i] = (v < V) ? *reinterpret_cast<const float4*>(row + v) : make_float4(0.f, 0.f, 0.f, 0.f);
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int v = v0 + 4096 * i;
      if (v < V) {
        if (x[i].x > best || bi == 0x7fffffff) { best = x[i].x; bi = v; }
        if (x[i].y > best) { best = x[i].y; bi = v + 1; }
        if (x[i].z > best) { best = x[i].z; bi = v + 2; }
        if (x[i].w > best) { best = x[i].w; bi = v + 3; }
      }
    }
  }
  argmax_swap(best, bi, true);
  argmax_swap(best, bi, false);
  argmax_dpp<kDppRor8>(best, bi);
  argmax_dpp<kDppRor4>(best, bi);
  argmax_dpp<kDppXor2>(best, bi);
  argmax_dpp<kDppXor1>(best, bi);
  if ((tid & 63) == 0) { sv[tid >> 6] = best; si[tid >> 6] = bi; }
  __syncthreads();
  if (tid == 0) {
    float4 v[4];
    int4 i4[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      v[q] = reinterpret_cast<const float4*>(sv)[q];
      i4[q] = reinterpret_cast<const int4*>(si)[q];
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (q > 0) argmax_take(best, bi, v[q].x, i4[q].x);
      argmax_take(best, bi, v[q].y, i4[q].y);
      argmax_take(best, bi, v[q].z, i4[q].z);
      argmax_take(best, bi, v[q].w, i4[q].w);
    }
    if (out_pos.rps) {
      if (o >= 0) out[(size_t)slot_of(out_pos, r) * out_slot_stride + o] = bi;
    } else {
      out[o] = bi;
    }
    s_id = bi;
  }
  if constexpr (NEXT) {
    __syncthreads();
    next_embed(next, o, s_id, 1024);
  }
}

void launch_argmax(const float* logits, int ld, int V, int nrows, int row0, int row_stride, int* out, PosRef out_pos,
                   int out_slot_stride, hipStream_t st, const NextEmbed& next) {
  hipLaunchKernelGGL(next.emb ? k_argmax<true> : k_argmax<false>, dim3(nrows), dim3(1024), 0, st, logits, out, out_pos.base,
                     out_pos.offset, out_pos.rps, ld, V, row0, row_stride, out_slot_stride, next);
}

// {L, n} of an iteration to the host, in turn to two places: no copy behind the iteration, which was a launch of 3 us
__device__ __forceinline__ void host_result(const HostResult& h, int turn, int L, int n) {
  if (!h.at) return;
  int* const at = h.at + 2 * (turn & 1);
  __hip_atomic_store(at, L, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  __hip_atomic_store(at + 1, n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  *h.turn = turn + 1;
}

// The greedy choice of M <= 8 rows of one sequence and what follows from it, by one work-group whose waves share the rows:
//   ACCEPT: validation of the stair batch (k_accept) and the embeddings the next iteration starts from;
//   else  : a draft token (M = 1) and the embedding of the step it leads to.
// CAND: src holds a (value, index) pair per row and 16 columns, left by the unembedding's work-groups (launch_unembed); else the
// rows of logits themselves, where they are short (decide_takes, decide_accept_takes).  A row of 32000 logits through one CU took longer than all its
// candidates, and the validation and the first embedding of a proposal were launches of their own (125M, k = 4, us: a draft token
// 5.9 -> 4.7; choice of five rows, validation and embedding 4.6 + 2.1 + 2.2 -> 6.3; tiny fp32 pair 3.3 -> 3.2 and 2.7 + 1.3 + 2.2
// -> 3.9).  What bounds it: the chain of three round trips (candidates, the token's embedding, its store).
template <bool CAND, bool ACCEPT>
__global__ __launch_bounds__(1024) void k_decide(const float* __restrict__ src, int* __restrict__ tokens, const int* pos_base,
                                                 int pos_offset, int n, int M, int next_rows, int* __restrict__ tgt, int* state,
                                                 HostResult host, NextEmbed next) {
  __shared__ float s_v[16];
  __shared__ int s_i[16], s_id[kMaxNextRows], s_pos;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int base = *pos_base;                              // ACCEPT: L, state[0] itself, written below
  const int wpr = 16 / (unsigned)M, m = wave / (unsigned)wpr, seg = wave - m * wpr;
  int mine = 0, prev = 0, active = 0, turn = 0;
  if (ACCEPT && wave == 0) {                               // lane i: draft token i
    mine = tokens[base + min(lane, M - 1)];
    prev = tokens[max(base - 1, 0)];
    active = state[3];
    if (host.at) turn = *host.turn;
  }
  float best = -INFINITY;
  int bi = 0x7fffffff;
  if (m < M) {
    const float* row = src + (size_t)m * n * (CAND ? 2 : 1);
    constexpr int NL = ACCEPT ? 16 : 2;                    // (2000 pairs a row: one round trip up to 7 rows)
    for (int e0 = seg * 64 + lane; e0 < n; e0 += wpr * 64 * NL) {
      float2 x[NL];
#pragma unroll
      for (int i = 0; i < NL; ++i) {
        const int e = min(e0 + i * wpr * 64, n - 1);
        x[i] = CAND ? reinterpret_cast<const float2*>(row)[e] : make_float2(fmaxf(row[e], -INFINITY), __int_as_float(e));
      }
#pragma unroll
      for (int i = 0; i < NL; ++i)
        if (e0 + i * wpr * 64 < n && (x[i].x > best || bi == 0x7fffffff)) { best = x[i].x; bi = __float_as_int(x[i].y); }
    }
  }
  argmax_swap(best, bi, true);
  argmax_swap(best, bi, false);
  argmax_dpp<kDppRor8>(best, bi);
  argmax_dpp<kDppRor4>(best, bi);
  argmax_dpp<kDppXor2>(best, bi);
  argmax_dpp<kDppXor1>(best, bi);
  if (lane == 0) { s_v[wave] = best; s_i[wave] = bi; }
  __syncthreads();
  if (wave == 0) {
    // 16 lanes put a row's shares together, then lane i takes row i's
    auto row_choice = [&](int first) {
      const int r = first + (lane >> 4), q = lane & 15;
      const bool has = r < M && q < wpr;
      float v = has ? s_v[r * wpr + q] : -INFINITY;
      int ix = has ? s_i[r * wpr + q] : 0x7fffffff;
      argmax_dpp<kDppRor8>(v, ix);
      argmax_dpp<kDppRor4>(v, ix);
      argmax_dpp<kDppXor2>(v, ix);
      argmax_dpp<kDppXor1>(v, ix);
      return ix;
    };
    bi = row_choice(0);
    if (ACCEPT) {
      const int k = M - 1;
      bi = __shfl(bi, (lane & 3) * 16);
      if (M > 4) {
        const int hi = __shfl(row_choice(4), (lane & 3) * 16);
        if (lane & 4) bi = hi;
      }
      if (lane < M) tgt[lane] = bi;
      const unsigned long long differ = __ballot(lane < k && mine != bi);
      const int acc = differ ? __builtin_ctzll(differ) : k;
      const int before = __shfl(bi, max(acc - 1, 0));
      if (lane == acc) {
        if (active) {
          tokens[base + acc] = bi;
          state[0] = base + acc + 1;
          state[1] = acc;
          host_result(host, turn, base + acc + 1, acc);
        }
        s_id[0] = acc > 0 ? before : prev;
        s_id[1] = bi;
        s_pos = base + acc;
      }
    } else if (lane == 0) {
      tokens[base + pos_offset] = bi;
      s_id[1] = bi;
      s_pos = base + pos_offset;
    }
  }
  if (!next.emb) return;
  __syncthreads();
  for (int i = 0; i < next_rows; ++i) next_embed(next, s_pos - (next_rows - 1 - i), s_id[kMaxNextRows - next_rows + i], 1024, i);
}
// Rows of logits themselves are read by one CU, so joined launches pay while they are short.  Launches before / joined, generation of
// a pair of 2 + 1 fp32 layers (d 256): a draft token (its step) at 1024 / 4096 / 8192 / 16384 logits 23.8 / 23.7, 24.2 / 24.2, 24.8 /
// 25.1, 25.8 / 27.3 us; a verification of 1 row at 16384 / 32768 51.4 / 49.1, 57.4 / 55.1, of 2 at 8192 / 16384 54.4 / 51.9, 55.5 /
// 54.2, of 8 at 2048 / 4096 / 8192 58.9 / 57.3, 59.9 / 59.1, 61.7 / 63.4 (bf16, 8 rows: 78.2 / 76.6, 78.8 / 77.9, 78.7 / 80.5).
// Candidates are ahead at every size: 32000 logits, a draft token 30.2 / 29.2, 1 / 4 / 7 rows 55.8 / 53.6, 60.2 / 58.1, 65.5 / 63.5;
// 130944, 48.5 / 45.3, 74.3 / 67.9, 80.9 / 77.1, 87.2 / 85.4.
bool decide_takes(bool cand, int V) { return cand || V <= 4096; }
bool decide_accept_takes(bool cand, int M, int V) { return M <= 8 && (cand || M * V <= 16384); }
void launch_decide(const float* src, bool cand, int V, int M, int* tokens, PosRef out_pos, hipStream_t st, const NextEmbed& next) {
  hipLaunchKernelGGL((cand ? k_decide<true, false> : k_decide<false, false>), dim3(1), dim3(1024), 0, st, src, tokens, out_pos.base, out_pos.offset,
                     cand ? V / 16 : V, M, 1, nullptr, nullptr, HostResult{}, next);
}
void launch_decide_accept(const float* src, bool cand, int V, int k, int* tokens, int* tgt, int* state, hipStream_t st, const NextEmbed& next,
                          int next_rows, const HostResult& host) {
  hipLaunchKernelGGL((cand ? k_decide<true, true> : k_decide<false, true>), dim3(1), dim3(1024), 0, st, src, tokens, state, 0, cand ? V / 16 : V, k + 1,
                     next_rows, tgt, state, host, next);
}

// (a lane per draft token: one round trip behind the state's, whatever k)
__global__ __launch_bounds__(64) void k_accept(int* __restrict__ tokens, const int* __restrict__ tgt, int k, int* __restrict__ state,
                                               int tok_slot_stride, const int* __restrict__ limits) {
  const int s = blockIdx.x, i = threadIdx.x;   // slot
  state += s * kSlotState;
  tokens += (size_t)s * tok_slot_stride;
  const int t = tgt[s * (k + 1) + min(i, k)];
  const int L = state[0], limit = limits ? limits[s] : 0x7fffffff;
  if (!state[3]) return;                    // the slot is not generating (any more)
  const unsigned long long differ = __ballot(i < k && tokens[L + min(i, k)] != t);
  const int n = differ ? __builtin_ctzll(differ) : k;
  if (i == n) {
    tokens[L + n] = t;
    state[0] = L + n + 1;
    state[1] = n;
    if (L + n + 1 >= limit) state[3] = 0;
  }
}
static_assert(kMaxRows <= 64, "k_accept, k_accept_sampled: a lane per stair row");

void launch_accept(int* tokens, const int* tgt, int k, int* state, int nslots, int tok_slot_stride, const int* limits, hipStream_t st) {
  hipLaunchKernelGGL(k_accept, dim3(nslots), dim3(64), 0, st, tokens, tgt, k, state, tok_slot_stride, limits);
}

// ---------------------------------------------------------------------------------------
// sampling variant: counter-based random numbers, Gumbel-max draws, keep / replace walk
// ---------------------------------------------------------------------------------------
// "squares" counter-based generator (Widynski 2020): four rounds of squaring, 32-bit output
__device__ __forceinline__ uint32_t squares32(uint64_t ctr, uint64_t key) {
  uint64_t x = ctr * key;
  const uint64_t y = x, z = y + key;
  x = x * x + y; x = (x >> 32) | (x << 32);
  x = x * x + z; x = (x >> 32) | (x << 32);
  x = x * x + y; x = (x >> 32) | (x << 32);
  return (uint32_t)((x * x + z) >> 32);
}
// the draw of (position of the token being decided, stream, vocabulary index) as a uniform in (0, 1)
__device__ __forceinline__ double sample_uniform(int pos, int stream, int v, uint64_t key) {
  const uint64_t ctr = ((uint64_t)pos << 34) | ((uint64_t)stream << 32) | (uint32_t)v;
  return ((double)squares32(ctr, key) + 0.5) * (1.0 / 4294967296.0);
}
__device__ __forceinline__ double sample_gumbel(int pos, int stream, int v, uint64_t key) {
  return -log(-log(sample_uniform(pos, stream, v, key)));
}

// (max, index) over a 256-thread block, ties -> lowest index; result valid in thread 0
__device__ __forceinline__ void block_argmax_256(double& best, int& bi, double* sv, int* si) {
  const int tid = threadIdx.x;
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    const double ov = __shfl_xor(best, off);
    const int oi = __shfl_xor(bi, off);
    if (ov > best || (ov == best && oi < bi)) { best = ov; bi = oi; }
  }
  if ((tid & 63) == 0) { sv[tid >> 6] = best; si[tid >> 6] = bi; }
  __syncthreads();
  if (tid == 0)
    for (int w = 1; w < 4; ++w)
      if (sv[w] > best || (sv[w] == best && si[w] < bi)) { best = sv[w]; bi = si[w]; }
  __syncthreads();
}

// A draw over the whole vocabulary spread over the blocks of a launch: every block reduces its candidates to one
// (score, index), stores it, and the block that arrives last at the ticket reduces those.  Returns true (in every
// thread of that last block) with the winner in best / bi of thread 0; the ticket is zero again afterwards.
__device__ __forceinline__ bool grid_argmax(double& best, int& bi, SampleWs* ws, double* sv, int* si, int* s_flag) {
  block_argmax_256(best, bi, sv, si);
  if (threadIdx.x == 0) {
    __hip_atomic_store(&ws->score[blockIdx.x], (unsigned long long)__double_as_longlong(best), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(&ws->idx[blockIdx.x], bi, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  if (!last_arrival(&ws->ticket, (int)gridDim.x, s_flag)) return false;
  best = -INFINITY;
  bi = 0x7fffffff;
  for (int i = threadIdx.x; i < (int)gridDim.x; i += 256) {
    const double ov = __longlong_as_double((long long)__hip_atomic_load(&ws->score[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    const int oi = __hip_atomic_load(&ws->idx[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (ov > best || (ov == best && oi < bi)) { best = ov; bi = oi; }
  }
  block_argmax_256(best, bi, sv, si);
  if (threadIdx.x == 0) __hip_atomic_store(&ws->ticket, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return true;
}

// (maximum, sum of exponentials) of a share of a row times inv_temp: kLseParts blocks per row, rows 0..n_a-1 from a, the rest
// from b; whoever needs a row's log-sum-exp puts its parts together (row_lse).  A block holds its values in registers, 16 loads a
// thread in flight (one block per row, two loops of one load a turn over 32000 values: 20 us; now 5).
__global__ __launch_bounds__(256) void k_row_lse(const float* __restrict__ a, const float* __restrict__ b, const SampleParams* __restrict__ sp,
                                                 float* __restrict__ lse, int n_a, int ld, int V) {
  __shared__ float red[8];
  const int r = blockIdx.x, tid = threadIdx.x;
  const float* row = r < n_a ? a + (size_t)r * ld : b + (size_t)(r - n_a) * ld;
  const int share = (V + kLseParts - 1) / kLseParts, v0 = blockIdx.y * share, v1 = min(V, v0 + share);
  const float it = sp->inv_temp;
  float mx = -INFINITY, sum = 0.f;
  for (int base = v0; base < v1; base += 16 * 256) {     // (one turn up to 32768 values a row)
    float x[16], m = -INFINITY;
#pragma unroll
    for (int i = 0; i < 16; ++i) x[i] = row[min(base + i * 256 + tid, v1 - 1)];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      x[i] = base + i * 256 + tid < v1 ? x[i] * it : -INFINITY;
      m = fmaxf(m, x[i]);
    }
    m = wave_max(m);
    if ((tid & 63) == 0) red[tid >> 6] = m;
    __syncthreads();
    const float mn = fmaxf(mx, fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3])));
    sum *= mx == -INFINITY ? 0.f : expf(mx - mn);
    mx = mn;
    if (mx != -INFINITY)
#pragma unroll
      for (int i = 0; i < 16; ++i) sum += expf(x[i] - mx);
    __syncthreads();
  }
  sum = wave_sum(sum);
  if ((tid & 63) == 0) red[4 + (tid >> 6)] = sum;
  __syncthreads();
  if (tid == 0)
    reinterpret_cast<float2*>(lse)[r * kLseParts + blockIdx.y] = make_float2(mx, ((red[4] + red[5]) + red[6]) + red[7]);
}
__device__ __forceinline__ float row_lse(const float* lse, int r) {
  float2 p[kLseParts];
#pragma unroll
  for (int i = 0; i < kLseParts; ++i) p[i] = reinterpret_cast<const float2*>(lse)[r * kLseParts + i];
  float mx = p[0].x, sum = 0.f;
#pragma unroll
  for (int i = 1; i < kLseParts; ++i) mx = fmaxf(mx, p[i].x);
#pragma unroll
  for (int i = 0; i < kLseParts; ++i) sum += p[i].x == -INFINITY ? 0.f : p[i].y * expf(p[i].x - mx);
  return mx + logf(sum);
}

// tokens[o] = argmax_v(logits[v] / T + gumbel(o, stream, v)) with o = the position out_pos gives: one categorical
// draw, one candidate per thread (grid-stride for very large vocabularies)
__global__ __launch_bounds__(256) void k_sample(const float* __restrict__ logits, const SampleParams* __restrict__ sp, const int* __restrict__ pos_base,
                                                int pos_offset, int V, int stream, int* __restrict__ tokens, SampleWs* ws, NextEmbed next) {
  __shared__ int s_id;
  __shared__ double sv[4];
  __shared__ int si[4];
  __shared__ int s_flag;
  const int o = *pos_base + pos_offset;
  const float it = sp->inv_temp;
  const uint64_t key = sp->key;
  double best = -INFINITY;
  int bi = 0x7fffffff;
  for (int v = blockIdx.x * 256 + threadIdx.x; v < V; v += gridDim.x * 256) {
    const double sc = (double)(logits[v] * it) + sample_gumbel(o, stream, v, key);
    if (sc > best || bi == 0x7fffffff) { best = sc; bi = v; }
  }
  if (!grid_argmax(best, bi, ws, sv, si, &s_flag)) return;
  if (threadIdx.x == 0) {
    tokens[o] = bi;
    s_id = bi;
  }
  if (next.emb) {                                        // (the block that decided the token, as in k_argmax)
    __syncthreads();
    next_embed(next, o, s_id, 256);
  }
}

// Validation of a sampled stair batch (one sequence).  tokens[L .. L+k) hold the assistant's draws d_1..d_k, dl[j-1]
// the logits d_j was drawn from, tl[i] the main model's logits of stair row i, lse[0..k] / lse[k+1..2k] their
// log-sum-exps at the temperature.  d_i is kept while u_i * q_i(d_i) < p_{i-1}(d_i); at the first one that is not,
// tokens[L+n] is drawn from the positive part of p_n - q_{n+1}; with all kept, tokens[L+k] from p_k.
// state = {L + n + 1, n}; emitted[0..n] = the n + 1 tokens of this iteration.  Every block repeats the (cheap) decisions
// and scores its share of the vocabulary; the block that arrives last picks the winner and writes the results.
__global__ __launch_bounds__(256) void k_accept_sampled(int* __restrict__ tokens, int* __restrict__ state, const float* __restrict__ lse,
                                                        const SampleParams* __restrict__ sp, const float* __restrict__ tl,
                                                        const float* __restrict__ dl, int ld, int V, int k, int* __restrict__ emitted,
                                                        SampleWs* ws, HostResult host, NextEmbed next, int next_rows) {
  __shared__ double sv[4];
  __shared__ int si[4];
  __shared__ int s_n, s_flag, s_empty, s_id[kMaxNextRows];
  __shared__ float s_lse[2 * kMaxRows];
  const int tid = threadIdx.x;
  const int L = state[0];
  const float it = sp->inv_temp;
  const uint64_t key = sp->key;
  if (tid <= 2 * k) s_lse[tid] = row_lse(lse, tid);
  // a lane per draft token, all of them in the round trips of one (one after the other they were two each)
  float lp = 0.f, lq1 = 0.f;
  if (tid < k) {
    const int d = tokens[L + tid];
    lp = tl[(size_t)tid * ld + d];
    lq1 = dl[(size_t)tid * ld + d];
  }
  __syncthreads();
  if (tid < 64) {
    bool kept = true;
    if (tid < k) {
      const float logp = lp * it - s_lse[tid];
      const float logq = lq1 * it - s_lse[k + 1 + tid];
      kept = sample_uniform(L + tid, 1, 0, key) < (double)expf(logp - logq);
    }
    const unsigned long long out = __ballot(!kept);
    if (tid == 0) s_n = out ? __builtin_ctzll(out) : k;
  }
  __syncthreads();
  const int n = s_n;
  const int pos = L + n;
  const float* trow = tl + (size_t)n * ld;
  const float* drow = dl + (size_t)n * ld;     // only read when n < k
  const float lt = s_lse[n], lq = n < k ? s_lse[k + 1 + n] : 0.f;
  double best = -INFINITY;
  int bi = 0x7fffffff;
  for (int v = blockIdx.x * 256 + tid; v < V; v += gridDim.x * 256) {
    double sc;
    if (n < k) {                               // the positive part of p - q (a token was not kept)
      const float diff = expf(trow[v] * it - lt) - expf(drow[v] * it - lq);
      sc = diff > 0.f ? (double)logf(diff) + sample_gumbel(pos, 2, v, key) : -INFINITY;
    } else {                                   // all kept: p itself
      sc = (double)(trow[v] * it) + sample_gumbel(pos, 2, v, key);
    }
    if (sc > best || bi == 0x7fffffff) { best = sc; bi = v; }
  }
  if (!grid_argmax(best, bi, ws, sv, si, &s_flag)) return;
  if (tid == 0) s_empty = best == -INFINITY;
  __syncthreads();
  if (s_empty) {
    // possible only in rounding (p and q agree to the last bit and a token was still not kept): draw from p, by
    // this block alone
    best = -INFINITY;
    bi = 0x7fffffff;
    for (int v = tid; v < V; v += 256) {
      const double sc = (double)(trow[v] * it) + sample_gumbel(pos, 2, v, key);
      if (sc > best || bi == 0x7fffffff) { best = sc; bi = v; }
    }
    block_argmax_256(best, bi, sv, si);
  }
  if (tid < n) emitted[tid] = tokens[L + tid];
  if (tid == 0) {
    emitted[n] = bi;
    s_id[0] = tokens[max(pos - 1, 0)];
    s_id[1] = bi;
    tokens[pos] = bi;
    state[0] = L + n + 1;
    state[1] = n;
    if (host.at) host_result(host, *host.turn, L + n + 1, n);
  }
  if (!next.emb) return;                                 // (the block that decided the last token, as in k_decide)
  __syncthreads();
  for (int i = 0; i < next_rows; ++i) next_embed(next, pos - (next_rows - 1 - i), s_id[kMaxNextRows - next_rows + i], 256, i);
}

void launch_row_lse(const float* a, int n_a, const float* b, int n_b, int ld, int V, const SampleParams* sp, float* lse,
                    hipStream_t st) {
  hipLaunchKernelGGL(k_row_lse, dim3(n_a + n_b, kLseParts), dim3(256), 0, st, a, b, sp, lse, n_a, ld, V);
}
static int sample_blocks(int V) { return std::min(kSampleBlocksMax, (V + 255) / 256); }
void launch_sample(const float* logits, int V, const SampleParams* sp, int stream, int* tokens, PosRef out_pos,
                   SampleWs* ws, hipStream_t st, const NextEmbed& next) {
  hipLaunchKernelGGL(k_sample, dim3(sample_blocks(V)), dim3(256), 0, st, logits, sp, out_pos.base, out_pos.offset, V, stream, tokens, ws,
                     next);
}
void launch_accept_sampled(int* tokens, const float* tl, const float* dl, int ld, int V, int k, const float* lse,
                           const SampleParams* sp, int* state, int* emitted, SampleWs* ws, hipStream_t st, const NextEmbed& next, int next_rows,
                           const HostResult& host) {
  hipLaunchKernelGGL(k_accept_sampled, dim3(sample_blocks(V)), dim3(256), 0, st, tokens, state, lse, sp, tl, dl, ld, V, k,
                     emitted, ws, host, next, next_rows);
}

// plain streaming copy, the calibration kernel for HBM traffic counters
__global__ __launch_bounds__(256) void k_copy_probe(const uint4* __restrict__ src, uint4* __restrict__ dst, size_t n) {
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) dst[i] = src[i];
}

void launch_copy_probe(const void* src, void* dst, size_t bytes, hipStream_t st) {
  const size_t n = bytes / 16;
  hipLaunchKernelGGL(k_copy_probe, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st,
                     static_cast<const uint4*>(src), static_cast<uint4*>(dst), n);
}

// Once per device: a function's attributes belong to the device, and some 200 calls of 40 us were part of every
// stairs_init (tens of ms for a small model's).
hipError_t configure_kernels() {
  static std::mutex mu;
  static bool done[64] = {};
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  const bool counted = dev >= 0 && dev < 64;
  const std::lock_guard<std::mutex> lock(mu);
  if (counted && done[dev]) return hipSuccess;
  std::vector<const void*> seen;             // (one kernel serves several k)
  auto optin = [&](const void* fn, size_t bytes) {
    if (std::find(seen.begin(), seen.end(), fn) != seen.end()) return;
    seen.push_back(fn);
    const hipError_t r = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
    if (r != hipSuccess) e = r;
  };
  // (forms for k up to 2048 only where the launch asks for more than the block needs, i.e. for more than half a CU's LDS)
#define STAIRS_OPTIN1(r, role, nw, gp, st, lds, ...) \
  for (int K : {__VA_ARGS__}) optin((const void*)rows_kernel<r, role, nw, gp, st>(K, false), lds)
#define STAIRS_OPTIN2(r, st, lds)                                                                           \
  STAIRS_OPTIN1(r, kRoleQKV, 4, 2, st, lds, (r > 4 ? 2048 : 1 << 20), 1 << 20);                             \
  STAIRS_OPTIN1(r, kRoleGateUp, 4, 2, st, kRowsPathMaxLdsWide, (r > 4 ? 2048 : 1 << 20), 1 << 20);          \
  STAIRS_OPTIN1(r, kRoleHead, 4, 2, st, lds, (r > 4 ? 2048 : 1 << 20), 1 << 20);                            \
  STAIRS_OPTIN1(r, kRoleWo, 8, 1, st, kRowsPathMaxLdsWide, 1024, 2048, 1 << 20);                            \
  STAIRS_OPTIN1(r, kRoleDown, 8, (r > 4 ? 1 : 3), st, kRowsPathMaxLdsWide, 1024, 2048, 4096, 1 << 20);      \
  STAIRS_OPTIN1((r > 4 ? 4 : r), kRoleDown, 16, 1, st, kRowsPathMaxLdsWide, 1 << 20);                       \
  optin((const void*)rows_kernel<r, kRoleQKV, 4, 2, st>(1 << 20, true), kRowsPathMaxLdsWide);               \
  optin((const void*)rows_kernel<r, kRoleGateUp, 4, 2, st>(1 << 20, true), kRowsPathMaxLdsWide);            \
  optin((const void*)rows_kernel<r, kRoleHead, 4, 2, st>(1 << 20, true), kRowsPathMaxLdsWide);              \
  optin((const void*)rows_kernel<r, kRoleWo, 8, 1, st>(1 << 20, true), kRowsPathMaxLdsWide)
#define STAIRS_OPTIN(r, lds)    \
  STAIRS_OPTIN2(r, true, lds);  \
  STAIRS_OPTIN2(r, false, lds)
  STAIRS_OPTIN(1, kRowsPathMaxLds);
  STAIRS_OPTIN(2, kRowsPathMaxLds);
  STAIRS_OPTIN(3, kRowsPathMaxLds);
  STAIRS_OPTIN(4, kRowsPathMaxLds);
  STAIRS_OPTIN(5, kRowsPathMaxLdsWide);
  STAIRS_OPTIN(6, kRowsPathMaxLdsWide);
  STAIRS_OPTIN(7, kRowsPathMaxLdsWide);
#undef STAIRS_OPTIN1
#undef STAIRS_OPTIN2
#undef STAIRS_OPTIN
#define STAIRS_OPTIN_WIDE(ct, nt, dp0)                                                                   \
  constexpr int dp_##ct##_##nt = (ct) == 1 ? (dp0) : (ct) == 2 ? wide_depth2(dp0) : (ct) == 3 ? wide_depth3(dp0) : wide_depth4(dp0);   \
  STAIRS_OPTIN_WIDE_(ct, nt, dp_##ct##_##nt)
#define STAIRS_OPTIN_WIDE_(ct, nt, dp)                                           \
  optin((const void*)k_gemm_bf16_wide<ct, nt, dp, true>, kWideMaxLds);            \
  optin((const void*)k_gemm_bf16_wide<ct, nt, dp, false>, kWideMaxLds)
  STAIRS_OPTIN_WIDE(1, 8, kWideDepth8); STAIRS_OPTIN_WIDE(2, 8, kWideDepth8);
  STAIRS_OPTIN_WIDE(1, 6, kWideDepth6); STAIRS_OPTIN_WIDE(2, 6, kWideDepth6);
  STAIRS_OPTIN_WIDE(1, 3, kWideDepth3); STAIRS_OPTIN_WIDE(2, 3, kWideDepth3);
  STAIRS_OPTIN_WIDE(1, 4, kWideDepth4); STAIRS_OPTIN_WIDE(2, 4, kWideDepth4);
  STAIRS_OPTIN_WIDE(1, 2, kWideDepth2); STAIRS_OPTIN_WIDE(2, 2, kWideDepth2);
  STAIRS_OPTIN_WIDE(1, 1, kWideDepth1); STAIRS_OPTIN_WIDE(2, 1, kWideDepth1);
  STAIRS_OPTIN_WIDE_(1, 1, kWideDepthChunk);
  optin((const void*)rows_kernel<1, kRoleHead, 4, 2, false, true>(1 << 20, false), kRowsPathMaxLds);
  optin((const void*)rows_kernel<2, kRoleHead, 4, 2, false, true>(1 << 20, false), kRowsPathMaxLds);
  optin((const void*)rows_kernel<3, kRoleHead, 4, 2, false, true>(1 << 20, false), kRowsPathMaxLds);
  optin((const void*)rows_kernel<4, kRoleHead, 4, 2, false, true>(1 << 20, false), kRowsPathMaxLds);
  optin((const void*)k_gemm_bf16_wide<1, 1, kWideDepth1, false, true>, kWideMaxLds);
  optin((const void*)k_gemm_bf16_wide<1, 2, kWideDepth2, false, true>, kWideMaxLds);
  optin((const void*)k_gemm_bf16_wide<2, 1, wide_depth2(kWideDepth1), false, true>, kWideMaxLds);
  optin((const void*)k_gemm_bf16_wide<2, 2, wide_depth2(kWideDepth2), false, true>, kWideMaxLds);
  STAIRS_OPTIN_WIDE(3, 2, kWideDepth2);
  STAIRS_OPTIN_WIDE(3, 1, kWideDepth1); STAIRS_OPTIN_WIDE(4, 1, kWideDepth1);
#undef STAIRS_OPTIN_WIDE
#undef STAIRS_OPTIN_WIDE_
  if (configure_block_kernels() != hipSuccess) e = hipErrorInvalidValue;
  optin((const void*)k_attn<128, 1, true>, 128 * 1024);
  optin((const void*)k_attn<128, 1, false>, 128 * 1024);
  optin((const void*)k_attn<128, 4, false>, 128 * 1024);
  optin((const void*)k_attn<128, 16, true>, 128 * 1024);
  optin((const void*)k_attn<128, 16, false>, 128 * 1024);
  if (counted && e == hipSuccess) done[dev] = true;
  return e;
}

}  // namespace stairs
