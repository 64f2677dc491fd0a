// gfx950 kernels of the prompt ingestion in large row blocks and of forwards of many rows: the MFMA-bound block GEMM,
// the attention of a prompt block and the element-wise work around them.  Numerics contract as in stairs_kernels.hip.
#include "stairs_device.h"

#include <math.h>

#include <algorithm>

namespace stairs {

// Attention of a prefill block (R consecutive rows at positions p0 .. p0+R-1 of one sequence) without partial
// results: a wave owns 16 query rows (a work-group 64) of one head and
// walks over the keys 0 .. its last row's position, 32 at a time, keeping the running maximum, the running sum and the
// running output of its rows in registers (rescaled whenever the maximum grows).  Same operands and splits as
// k_attn_f16 (scores^T = K q^T with q as half high + low, out^T = V^T p^T with p as half high + low); the order of
// the additions differs from the decode kernels, which only ever see their own results.
template <int HD>
__global__ __launch_bounds__(256, 2) void k_attn_flash(const float* __restrict__ q, const _Float16* __restrict__ Kc,
                                                    const _Float16* __restrict__ Vc, int cap, int d, int H, int R, int p0,
                                                    float scale, float* __restrict__ out) {
  constexpr int KK = HD / 32, ET = HD / 16;
  const int h = blockIdx.x;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int j = lane & 15, g = lane >> 4;
  const int r0 = blockIdx.y * 64 + wave * 16;         // first row of this wave's tile
  if (r0 >= R) return;                                // no barriers in this kernel: waves are independent
  const int row = r0 + j;
  const bool row_ok = row < R;
  const int p_row = p0 + row;
  const int tile_last = p0 + min(r0 + 15, R - 1);     // last position of the tile = last key any of its rows sees
  f16x8 qh[KK], ql[KK];
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) {
    float4 a = make_float4(0.f, 0.f, 0.f, 0.f), b = a;
    if (row_ok) {
      const float4* qp = reinterpret_cast<const float4*>(q + (size_t)row * d + h * HD + kk * 32 + g * 8);
      a = qp[0];
      b = qp[1];
    }
    const float v[8] = {a.x * scale, a.y * scale, a.z * scale, a.w * scale, b.x * scale, b.y * scale, b.z * scale, b.w * scale};
    split_half8(v, qh[kk], ql[kk]);
  }
  const uint4* Kh = reinterpret_cast<const uint4*>(Kc + (size_t)h * cap * HD) + lane;
  const uint4* Vh = reinterpret_cast<const uint4*>(Vc + (size_t)h * cap * HD) + lane;
  f32x4 oacc[ET];
#pragma unroll
  for (int et = 0; et < ET; ++et) oacc[et] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m_run = -INFINITY, l_run = 0.f;
  // two register sets: the keys and values of the next step are requested before this step's arithmetic
  uint4 kA[2][KK], vA[ET], kB[2][KK], vB[ET];
  auto load_kv = [&](int kb, uint4 (&kreg)[2][KK], uint4 (&vreg)[ET]) {
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) kreg[t][kk] = Kh[((size_t)((kb >> 4) + t) * KK + kk) * 64];
#pragma unroll
    for (int et = 0; et < ET; ++et) vreg[et] = Vh[((size_t)(kb >> 5) * ET + et) * 64];
  };
  auto step = [&](int kb, const uint4 (&kreg)[2][KK], const uint4 (&vreg)[ET]) {
    float sc[8];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      f32x4 sacc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) {
        const f16x8 a = __builtin_bit_cast(f16x8, kreg[t][kk]);
        sacc = __builtin_amdgcn_mfma_f32_16x16x32_f16(a, qh[kk], sacc, 0, 0, 0);
        sacc = __builtin_amdgcn_mfma_f32_16x16x32_f16(a, ql[kk], sacc, 0, 0, 0);
      }
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int key = kb + t * 16 + g * 4 + v;
        sc[t * 4 + v] = (row_ok && key <= p_row) ? sacc[v] : -INFINITY;
      }
    }
    float mx = sc[0];
#pragma unroll
    for (int i = 1; i < 8; ++i) mx = fmaxf(mx, sc[i]);
    mx = fmaxf(mx, __shfl_xor(mx, 16));
    mx = fmaxf(mx, __shfl_xor(mx, 32));
    const float m_new = fmaxf(m_run, mx);
    const float alpha = (m_run == -INFINITY) ? 0.f : exp_fast(m_run - m_new);   // m_new >= m_run > -inf there
    float pv[8], sum = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      pv[i] = (m_new == -INFINITY) ? 0.f : exp_fast(sc[i] - m_new);
      sum += pv[i];
    }
    sum += __shfl_xor(sum, 16);
    sum += __shfl_xor(sum, 32);
    l_run = l_run * alpha + sum;
    m_run = m_new;
    f16x8 ph, pl;
    split_half8(pv, ph, pl);
#pragma unroll
    for (int et = 0; et < ET; ++et) {
      oacc[et][0] *= alpha; oacc[et][1] *= alpha; oacc[et][2] *= alpha; oacc[et][3] *= alpha;
      const f16x8 a = __builtin_bit_cast(f16x8, vreg[et]);
      oacc[et] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a, ph, oacc[et], 0, 0, 0);
      oacc[et] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a, pl, oacc[et], 0, 0, 0);
    }
  };
  load_kv(0, kA, vA);
#pragma nounroll
  for (int kb = 0; kb <= tile_last; kb += 64) {
    if (kb + 32 <= tile_last) load_kv(kb + 32, kB, vB);
    step(kb, kA, vA);
    if (kb + 32 > tile_last) break;
    if (kb + 64 <= tile_last) load_kv(kb + 64, kA, vA);
    step(kb + 32, kB, vB);
  }
  if (row_ok) {
    const float inv = 1.0f / l_run;
#pragma unroll
    for (int et = 0; et < ET; ++et)
      *reinterpret_cast<float4*>(out + (size_t)row * d + h * HD + et * 16 + g * 4) =
          make_float4(oacc[et][0] * inv, oacc[et][1] * inv, oacc[et][2] * inv, oacc[et][3] * inv);
  }
}

void launch_attention_flash(const float* q, const void* Kc, const void* Vc, int cap, int d, int H, int R, int p0, float* out,
                            hipStream_t st) {
  const int hd = d / H;
  const float scale = 1.0f / sqrtf((float)hd);
  const _Float16* K = static_cast<const _Float16*>(Kc);
  const _Float16* V = static_cast<const _Float16*>(Vc);
  dim3 grid(H, (R + 63) / 64);
  if (hd == 128)
    hipLaunchKernelGGL((k_attn_flash<128>), grid, dim3(256), 0, st, q, K, V, cap, d, H, R, p0, scale, out);
  else
    hipLaunchKernelGGL((k_attn_flash<64>), grid, dim3(256), 0, st, q, K, V, cap, d, H, R, p0, scale, out);
}

// ---------------------------------------------------------------------------------------
// prompt ingestion in large row blocks: an MFMA-bound GEMM and the element-wise work around it
// ---------------------------------------------------------------------------------------
// Activations of a row block as MFMA B-operand fragments, written once by their producer: [k-step of 32][column tile
// of 16 rows][high, low][lane] x 16 bytes (lane r + 16 g: x[16 ct + r][32 kt + 8 g .. + 8] as bf16 high part / bf16 of
// the remainders).  RT = column tiles the buffer is laid out for (rows rounded up to a multiple of kBlkRows).
__device__ __forceinline__ void pf_store_frag4(uint4* frag, int RT, int r, int k, const float (&v)[4]) {
  uint2 hi, lo;
  bf16_split2(v[0], v[1], hi.x, lo.x);
  bf16_split2(v[2], v[3], hi.y, lo.y);
  const size_t u4 = (((size_t)(k >> 5) * RT + (r >> 4)) * 2) * 64 + (r & 15) + 16 * ((k & 31) >> 3);
  uint2* dst = reinterpret_cast<uint2*>(frag) + u4 * 2 + ((k & 7) >> 2);
  dst[0] = hi;
  dst[128] = lo;
}

// Y[R, N] (+)= X[R, K] . W[N, K]^T for row blocks of up to thousands of rows: the MFMA-bound regime.
//   W: the operand-tile layout of the decode kernels (read as the MFMA A operand straight from memory, 1 KiB per load);
//   X: block fragments (above), staged through LDS one k-step at a time, double-buffered, shared by the 8 waves.
//   Work-group = 256 output features (16 weight tiles) x 128 rows (8 column tiles) on 8 waves, each 4 weight tiles x
//   4 column tiles: a wave's k-step is 4 KiB of weights from memory, 8 KiB of fragments from LDS and 32 MFMAs (high and
//   low part of x), fp32 accumulators [4][4] tiles.  Output columns are stored in natural order (the row permutation of the weight layout is undone:
//   4 consecutive permuted rows are 4 consecutive features).  accumulate: Y += (the residual connections).
//   One order of additions per output (k ascending, high before low): results do not depend on R or on the grid.
constexpr int kBlkKs = 2;                              // k-steps per stage (the unit the k splits are counted in)
constexpr int kBlkStageU4 = (kBlkRows / 16) * 2 * 64;  // uint4 per LDS buffer (one k-step): 1024 (16 KiB)
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_gemm_bf16_block(const uint4* __restrict__ Wsw, int NTILES, int K,
                                                         const uint4* __restrict__ XF, int RT, int R,
                                                         float* __restrict__ Y, int ldy, int perm, int p0, int p1,
                                                         int accumulate, int stages_per_split, size_t split_stride) {
  // 8 waves: wave = (row half rh, feature group fw); a wave owns 4 weight tiles x 4 column tiles (64 x 64 outputs)
  // blockIdx.z = k split: with few rows and few features there are too few (feature, row) blocks to fill the chip, so
  // the k range is cut into gridDim.z pieces whose results go to Y + z * split_stride and are added up, in split
  // order, by k_block_reduce
  constexpr int NT = 4, CT = kBlkRows / 32, CTW = kBlkRows / 16;
  extern __shared__ uint4 lds[];                       // [2][kBlkStageU4]
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int fw = wave & 3, rh = wave >> 2;
  const int j = lane & 15, g = lane >> 4;
  const int tile0 = (blockIdx.x * 4 + fw) * NT;
  const int ct0 = blockIdx.y * CTW;                    // first column tile of the work-group
  const int units_total = K / kUnitK;
  const int nstages_all = (K >> 5) / kBlkKs;           // K is a multiple of 256: whole stages
  const int stage0 = blockIdx.z * stages_per_split;
  const int nstages = min(nstages_all, stage0 + stages_per_split);     // this split's stages: [stage0, nstages)
  Y += blockIdx.z * split_stride;
  int tile_c[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) tile_c[t] = min(tile0 + t, NTILES - 1);

  // this split's k-steps: [ks0, ks_end), a multiple of 4 (K is a multiple of 256 and a split an even number of stages)
  const int ks0 = stage0 * kBlkKs, ks_end = nstages * kBlkKs, ks_last = ks_end - 1;
  // weights of k-step s (past the split's end the last one is read again): 4 tiles x 1 KiB
  auto load_a = [&](uint4 (&a)[NT], int s_) {
    const int s = min(s_, ks_last), c = s >> 4, kk = s & 15;
    const int ksteps_c = min(kSliceUnits, units_total - c * kSliceUnits) * 8;
    const uint4* wbase = Wsw + (size_t)c * NTILES * (kSliceUnits * 8) * 64 + (size_t)kk * 64 + lane;
#pragma unroll
    for (int t = 0; t < NT; ++t) a[t] = wbase[(size_t)tile_c[t] * ksteps_c * 64];
  };
  f32x4 acc[NT][CT];
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) acc[t][ct] = f32x4{0.f, 0.f, 0.f, 0.f};

  // one k-step: the work-group's 8 column tiles x (high, low) are 1024 consecutive uint4 of LDS buffer buf
  auto compute = [&](const uint4 (&a)[NT], int buf) {
    const uint4* src = lds + buf * kBlkStageU4 + (rh * CT * 2) * 64 + lane;
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
      const bf16x8 vh = __builtin_bit_cast(bf16x8, src[(ct * 2) * 64]);
      const bf16x8 vl = __builtin_bit_cast(bf16x8, src[(ct * 2 + 1) * 64]);
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const bf16x8 av = __builtin_bit_cast(bf16x8, a[t]);
        acc[t][ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, vh, acc[t][ct], 0, 0, 0);
      }
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const bf16x8 av = __builtin_bit_cast(bf16x8, a[t]);
        acc[t][ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, vl, acc[t][ct], 0, 0, 0);
      }
    }
  };
  // Rings of four k-steps in registers, for the weights (4 x 16) and for the fragments on their way to LDS (4 x 8):
  // before the arithmetic of k-step s, weights and fragments of k-step s + 3 are requested, so a request has three
  // k-steps' arithmetic to come back in (with one stage of two k-steps the waves spent nearly half their cycles waiting for memory, also at
  // thousands of rows); after the arithmetic the fragments of k-step s + 1 go to the other LDS buffer.  Four k-steps
  // per turn of the loop name the rings' registers statically; a split's k-steps are a multiple of four, so no turn
  // ends early.  All requests are unconditional.  Two waves per SIMD fill each other's waits for LDS and memory.
  uint4 a0[NT], a1[NT], a2[NT], a3[NT];
  uint4 b0_0, b0_1, b1_0, b1_1, b2_0, b2_1, b3_0, b3_1;    // (plain variables: small arrays ended up in scratch memory)
#define STAIRS_LOAD_B(b, s_)                                                                      \
  do {                                                                                            \
    const uint4* src_ = XF + ((size_t)min((s_), ks_last) * RT + ct0) * 2 * 64 + tid;              \
    b##_0 = src_[0];                                                                              \
    b##_1 = src_[512];                                                                            \
  } while (0)
#define STAIRS_STORE_B(buf, b)                               \
  do {                                                       \
    uint4* dst_ = lds + (buf) * kBlkStageU4 + tid;           \
    dst_[0] = b##_0;                                         \
    dst_[512] = b##_1;                                       \
  } while (0)
  // k-step s in LDS buffer buf: ac = its weights, an / bn = the ring slots for k-step s + 3, bs = the fragments of s + 1
#define STAIRS_BLOCK_STEP(ac, an, bn, bs, s, buf)            \
  do {                                                       \
    STAIRS_LOAD_B(bn, (s) + 3);                              \
    load_a(an, (s) + 3);                                     \
    __builtin_amdgcn_sched_barrier(0);                       \
    compute(ac, buf);                                        \
    STAIRS_STORE_B((buf) ^ 1, bs);                           \
    __syncthreads();                                         \
  } while (0)
  STAIRS_LOAD_B(b0, ks0);
  load_a(a0, ks0);
  STAIRS_LOAD_B(b1, ks0 + 1);
  load_a(a1, ks0 + 1);
  STAIRS_LOAD_B(b2, ks0 + 2);
  load_a(a2, ks0 + 2);
  STAIRS_STORE_B(0, b0);
  __syncthreads();
  for (int ks = ks0; ks < ks_end; ks += 4) {
    STAIRS_BLOCK_STEP(a0, a3, b3, b1, ks, 0);
    STAIRS_BLOCK_STEP(a1, a0, b0, b2, ks + 1, 1);
    STAIRS_BLOCK_STEP(a2, a1, b1, b3, ks + 2, 0);
    STAIRS_BLOCK_STEP(a3, a2, b2, b0, ks + 3, 1);
  }
#undef STAIRS_BLOCK_STEP
#undef STAIRS_LOAD_B
#undef STAIRS_STORE_B

#pragma unroll
  for (int t = 0; t < NT; ++t) {
    if (tile0 + t < NTILES) {
      const size_t col = perm_row((tile0 + t) * 16 + 4 * g, perm, p0, p1);
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) {
        const int row = (ct0 + rh * CT + ct) * 16 + j;
        if (row < R) {
          float4* dst = reinterpret_cast<float4*>(Y + (size_t)row * ldy + col);
          float4 v = make_float4(acc[t][ct][0], acc[t][ct][1], acc[t][ct][2], acc[t][ct][3]);
          if (accumulate) {
            const float4 o = *dst;
            v.x = v.x + o.x; v.y = v.y + o.y; v.z = v.z + o.z; v.w = v.w + o.w;
          }
          *dst = v;
        }
      }
    }
  }
}

// Y = (accumulate ? Y : 0) + part[0] + part[1] + ... (in that order): the k splits of a block GEMM with few rows
__global__ __launch_bounds__(256) void k_block_reduce(const float* __restrict__ part, int nsplit, size_t split_stride, int R, int N,
                                                      float* __restrict__ Y, int ldy, int accumulate) {
  const int r = blockIdx.y, c = (blockIdx.x * 256 + threadIdx.x) * 4;
  if (c >= N) return;
  float4* dst = reinterpret_cast<float4*>(Y + (size_t)r * ldy + c);
  float4 a = accumulate ? *dst : make_float4(0.f, 0.f, 0.f, 0.f);
  for (int z = 0; z < nsplit; ++z) {
    const float4 v = *reinterpret_cast<const float4*>(part + z * split_stride + (size_t)r * N + c);
    a.x = a.x + v.x; a.y = a.y + v.y; a.z = a.z + v.z; a.w = a.w + v.w;
  }
  *dst = a;
}

void launch_gemm_block(const void* W, int N, int K, const uint4* xfrag, int R, float* Y, int ldy, int perm, int p0, int p1,
                       int accumulate, hipStream_t st, float* part, size_t part_floats) {
  const int NTILES = N / 16;
  const int FB = (NTILES + 15) / 16, RB = (R + kBlkRows - 1) / kBlkRows;
  const int nstages = (K / 32) / kBlkKs;
  // few (feature, row) blocks: cut k into pieces until about every CU has a work-group (each piece at least 8 stages
  // and an even number of them), as far as the scratch for the pieces' results reaches
  int nsplit = 1;
  if (part && FB * RB < 160) {
    nsplit = std::min({(256 + FB * RB - 1) / (FB * RB), nstages / 8, (int)(part_floats / ((size_t)R * N))});
    nsplit = std::max(nsplit, 1);
  }
  int per = (nstages + nsplit - 1) / nsplit;
  per += per & 1;
  nsplit = (nstages + per - 1) / per;
  dim3 grid(FB, RB, nsplit), block(512);
  const size_t lds = 2 * kBlkStageU4 * sizeof(uint4);
  if (nsplit == 1) {
    hipLaunchKernelGGL(k_gemm_bf16_block, grid, block, lds, st, static_cast<const uint4*>(W), NTILES, K, xfrag, pf_col_tiles(R), R, Y,
                       ldy, perm, p0, p1, accumulate, per, (size_t)0);
    return;
  }
  const size_t stride = (size_t)R * N;
  hipLaunchKernelGGL(k_gemm_bf16_block, grid, block, lds, st, static_cast<const uint4*>(W), NTILES, K, xfrag, pf_col_tiles(R), R, part,
                     N, perm, p0, p1, 0, per, stride);
  hipLaunchKernelGGL(k_block_reduce, dim3((N / 4 + 255) / 256, R), dim3(256), 0, st, part, nsplit, stride, R, N, Y, ldy, accumulate);
}

__global__ __launch_bounds__(256) void k_pf_embed(const uint16_t* __restrict__ emb, const int* __restrict__ tokens, int p0,
                                                  int tok_cap, int vocab, int d, float* __restrict__ x) {
  const int r = blockIdx.y, c = (blockIdx.x * 256 + threadIdx.x) * 4;
  if (c >= d) return;
  const int p = p0 + r;
  const int id = (p >= 0 && p < tok_cap) ? tokens[p] : -1;     // as k_embed: never outside the array or the table
  float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
  if (id >= 0 && id < vocab) {
    const uint16_t* row = emb + (size_t)id * d + c;
    v = make_float4(load_kv(row), load_kv(row + 1), load_kv(row + 2), load_kv(row + 3));
  }
  *reinterpret_cast<float4*>(x + (size_t)r * d + c) = v;
}
void launch_pf_embed(const uint16_t* emb, const int* tokens, int p0, int tok_cap, int vocab, int R, int d, float* x,
                     hipStream_t st) {
  hipLaunchKernelGGL(k_pf_embed, dim3((d + 1023) / 1024, R), dim3(256), 0, st, emb, tokens, p0, tok_cap, vocab, d, x);
}

__global__ __launch_bounds__(256) void k_pf_norm_split(const float* __restrict__ x, const float* __restrict__ gain, float eps,
                                                       int d, uint4* __restrict__ frag, int RT) {
  __shared__ float sm[4];
  const int r = blockIdx.x, tid = threadIdx.x;
  const float* row = x + (size_t)r * d;
  float rstd = 1.0f;
  if (gain) {
    float ss = 0.f;
    for (int c = tid * 4; c < d; c += 1024) {
      const float4 v = *reinterpret_cast<const float4*>(row + c);
      ss += sumsq4(v.x, v.y, v.z, v.w);
    }
    ss = block_sum_256(ss, sm);
    rstd = 1.0f / sqrtf(ss / (float)d + eps);
  }
  for (int c = tid * 4; c < d; c += 1024) {
    const float4 v = *reinterpret_cast<const float4*>(row + c);
    float e[4] = {v.x, v.y, v.z, v.w};
    if (gain) {
      const float4 g = *reinterpret_cast<const float4*>(gain + c);
      e[0] = e[0] * rstd * g.x; e[1] = e[1] * rstd * g.y; e[2] = e[2] * rstd * g.z; e[3] = e[3] * rstd * g.w;
    }
    pf_store_frag4(frag, RT, r, c, e);
  }
}
void launch_pf_norm_split(const float* x, const float* gain, float eps, int R, int d, uint4* frag, hipStream_t st) {
  hipLaunchKernelGGL(k_pf_norm_split, dim3(R), dim3(256), 0, st, x, gain, eps, d, frag, pf_col_tiles(R));
}

__global__ void k_pf_rope_table(int p0, int hd, double theta, float2* __restrict__ cs) {
  const int r = blockIdx.x, i = threadIdx.x;
  if (i >= hd / 2) return;
  const double ang = (double)(p0 + r) * pow(theta, -2.0 * (double)i / (double)hd);
  cs[r * 64 + i] = make_float2((float)cos(ang), (float)sin(ang));
}
void launch_pf_rope_table(int p0, int R, int hd, float theta, float2* cs, hipStream_t st) {
  hipLaunchKernelGGL(k_pf_rope_table, dim3(R), dim3(64), 0, st, p0, hd, (double)theta, cs);
}

__global__ __launch_bounds__(256) void k_pf_rope_kv(const float* __restrict__ y, int d, int H, int hd, int p0,
                                                    const float2* __restrict__ cs, float* __restrict__ q_rot,
                                                    _Float16* __restrict__ Kc, _Float16* __restrict__ Vc, int cap) {
  // thread = (row r, head h, pair e < hd/2)
  const int r = blockIdx.y, half = hd >> 1;
  const int idx = blockIdx.x * 256 + threadIdx.x;
  if (idx >= H * half) return;
  const int h = idx / half, e = idx - h * half;
  const int p = p0 + r;
  const float* yr = y + (size_t)r * 3 * d + h * hd;
  const float2 c = cs[r * 64 + e];
  const float2 q = rope_rotate(yr[e], yr[e + half], c);
  q_rot[(size_t)r * d + h * hd + e] = q.x;
  q_rot[(size_t)r * d + h * hd + e + half] = q.y;
  const float2 k = rope_rotate(yr[d + e], yr[d + e + half], c);
  _Float16* kd = Kc + (size_t)h * cap * hd;
  store_kv(kd + k_cache_off(p, e, hd), k.x);
  store_kv(kd + k_cache_off(p, e + half, hd), k.y);
  _Float16* vd = Vc + (size_t)h * cap * hd;
  store_kv(vd + v_cache_off(p, e, hd), yr[2 * d + e]);
  store_kv(vd + v_cache_off(p, e + half, hd), yr[2 * d + e + half]);
}
// The same for rows that sit wherever `pos` puts them (several sequences: row r belongs to slot slot_of(pos, r), whose
// caches start kv_slot_stride elements after the previous slot's); a row without a position writes nothing.
__global__ __launch_bounds__(256) void k_pf_rope_kv_rows(const float* __restrict__ y, int d, int H, int hd, PosRef pos,
                                                         size_t kv_slot_stride, const float2* __restrict__ cs,
                                                         float* __restrict__ q_rot, _Float16* __restrict__ Kc,
                                                         _Float16* __restrict__ Vc, int cap) {
  const int r = blockIdx.y, half = hd >> 1;
  const int idx = blockIdx.x * 256 + threadIdx.x;
  if (idx >= H * half) return;
  const int h = idx / half, e = idx - h * half;
  const int p = pos_of(pos, r);
  const float* yr = y + (size_t)r * 3 * d + h * hd;
  const float2 c = cs[r * 64 + e];
  const float2 q = rope_rotate(yr[e], yr[e + half], c);
  q_rot[(size_t)r * d + h * hd + e] = q.x;
  q_rot[(size_t)r * d + h * hd + e + half] = q.y;
  if (p < 0 || p >= cap) return;
  const size_t off = (size_t)slot_of(pos, r) * kv_slot_stride + (size_t)h * cap * hd;
  const float2 k = rope_rotate(yr[d + e], yr[d + e + half], c);
  store_kv(Kc + off + k_cache_off(p, e, hd), k.x);
  store_kv(Kc + off + k_cache_off(p, e + half, hd), k.y);
  store_kv(Vc + off + v_cache_off(p, e, hd), yr[2 * d + e]);
  store_kv(Vc + off + v_cache_off(p, e + half, hd), yr[2 * d + e + half]);
}
void launch_pf_rope_kv_rows(const float* y, int R, int d, int H, PosRef pos, size_t kv_slot_stride, const float2* cs,
                            float* q_rot, _Float16* Kc, _Float16* Vc, int cap, hipStream_t st) {
  const int hd = d / H;
  hipLaunchKernelGGL(k_pf_rope_kv_rows, dim3((H * hd / 2 + 255) / 256, R), dim3(256), 0, st, y, d, H, hd, pos, kv_slot_stride, cs,
                     q_rot, Kc, Vc, cap);
}

void launch_pf_rope_kv(const float* y, int R, int d, int H, int p0, const float2* cs, float* q_rot, _Float16* Kc,
                       _Float16* Vc, int cap, hipStream_t st) {
  const int hd = d / H;
  hipLaunchKernelGGL(k_pf_rope_kv, dim3((H * hd / 2 + 255) / 256, R), dim3(256), 0, st, y, d, H, hd, p0, cs, q_rot, Kc, Vc, cap);
}

__global__ __launch_bounds__(256) void k_pf_swiglu_split(const float* __restrict__ y, int f, uint4* __restrict__ frag, int RT) {
  const int r = blockIdx.y, c = (blockIdx.x * 256 + threadIdx.x) * 4;
  if (c >= f) return;
  const float4 g = *reinterpret_cast<const float4*>(y + (size_t)r * 2 * f + c);
  const float4 u = *reinterpret_cast<const float4*>(y + (size_t)r * 2 * f + f + c);
  const float e[4] = {swiglu(g.x, u.x), swiglu(g.y, u.y), swiglu(g.z, u.z), swiglu(g.w, u.w)};
  pf_store_frag4(frag, RT, r, c, e);
}
void launch_pf_swiglu_split(const float* y, int R, int f, uint4* frag, hipStream_t st) {
  hipLaunchKernelGGL(k_pf_swiglu_split, dim3((f + 1023) / 1024, R), dim3(256), 0, st, y, f, frag, pf_col_tiles(R));
}

hipError_t configure_block_kernels() {
  hipError_t e = hipSuccess;
  auto optin = [&](const void* fn, size_t bytes) {
    const hipError_t r = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
    if (r != hipSuccess) e = r;
  };
  optin((const void*)k_gemm_bf16_block, 2 * kBlkStageU4 * sizeof(uint4));
  return e;
}

}  // namespace stairs
