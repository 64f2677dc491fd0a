// gfx950 kernels of the prompt ingestion in large row blocks and of forwards of many rows: the MFMA-bound block GEMM,
// the attention of a prompt block and the element-wise work around them.  Numerics contract as in stairs_kernels.hip.
#include "stairs_device.h"

#include <math.h>

#include <algorithm>
#include <type_traits>

namespace stairs {

// ---------------------------------------------------------------------------------------
// rows of a block: where they sit, their rotation entries, their embeddings
// ---------------------------------------------------------------------------------------
// rows[r] = (slot, position) of row r, position < 0: a padding row; cs[r] = the rotation table's entries of the position
// (tab == nullptr: the identity rotation)
__device__ __forceinline__ void blk_row_entry(int r, int slot, int p, int hd, const float2* tab, int tab_len, int2* rows, float2* cs) {
  const int i = threadIdx.x;
  if (i == 0) rows[r] = make_int2(slot, p);
  if (i < hd / 2) cs[r * 64 + i] = tab && p >= 0 && p < tab_len ? tab[(size_t)p * 64 + i] : make_float2(1.f, 0.f);
}
__global__ __launch_bounds__(64) void k_blk_rows(BlkSegs segs, int hd, const float2* __restrict__ tab, int tab_len, int2* __restrict__ rows,
                                                 float2* __restrict__ cs) {
  const int r = blockIdx.x;
  int s = 0;
  while (s + 1 < segs.n && r >= segs.row0[s + 1]) ++s;
  const int i = r - segs.row0[s];
  blk_row_entry(r, segs.slot[s], i < segs.len[s] ? segs.pos0[s] + i : -1, hd, tab, tab_len, rows, cs);
}
__global__ __launch_bounds__(64) void k_blk_rows_pos(PosRef pos, int hd, const float2* __restrict__ tab, int tab_len, int2* __restrict__ rows,
                                                     float2* __restrict__ cs) {
  const int r = blockIdx.x;
  blk_row_entry(r, slot_of(pos, r), pos_of(pos, r), hd, tab, tab_len, rows, cs);
}
void launch_blk_rows(const BlkSegs& segs, int R, int hd, const float2* tab, int tab_len, int2* rows, float2* cs, hipStream_t st) {
  hipLaunchKernelGGL(k_blk_rows, dim3(R), dim3(64), 0, st, segs, hd, tab, tab_len, rows, cs);
}
void launch_blk_rows_pos(PosRef pos, int R, int hd, const float2* tab, int tab_len, int2* rows, float2* cs, hipStream_t st) {
  hipLaunchKernelGGL(k_blk_rows_pos, dim3(R), dim3(64), 0, st, pos, hd, tab, tab_len, rows, cs);
}

// Activations of a row block as MFMA B-operand fragments, written once by their producer: [k-step of 32][column tile
// of 16 rows][high, low][lane] x 16 bytes (lane r + 16 g: x[16 ct + r][32 kt + 8 g .. + 8] as bf16 high part / bf16 of
// the remainders).  RT = column tiles the buffer is laid out for (rows rounded up to a multiple of kBlkRows).
// (blk_store_frag4 in stairs_device.h)

// x[r][:] = the row's embedding (zeros for a padding row, a position outside [0, tok_cap) or an id outside [0, vocab)),
// frag = the fragments of x * gain, ssq[r][g] = sum of squares of columns 32 g .. 32 g + 31.  A wave takes 16 rows x 32
// columns, i.e. one high and one low fragment, which it writes as two whole KiB (a row per work-group left 16-byte pieces
// of a line to eight XCDs: 36 us for 2048 rows of 4096 columns, 14 this way).
__global__ __launch_bounds__(256) void k_blk_embed(const uint16_t* __restrict__ emb, const int* __restrict__ tokens, int tok_stride,
                                                   int tok_cap, int vocab, const int2* __restrict__ rows, int R, int d, float* __restrict__ x,
                                                   const float* __restrict__ gain, uint4* __restrict__ frag, int RT, float* __restrict__ ssq) {
  const int lane = threadIdx.x & 63, kt = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int r = blockIdx.y * 16 + (lane & 15), c = kt * 32 + (lane >> 4) * 8;
  if (kt * 32 >= d) return;                          // (whole waves)
  const int2 w = r < R ? rows[r] : make_int2(0, -1);
  const int id = (w.y >= 0 && w.y < tok_cap) ? tokens[(size_t)w.x * tok_stride + w.y] : -1;
  uint4 b = make_uint4(0u, 0u, 0u, 0u);
  if (id >= 0 && id < vocab) b = *reinterpret_cast<const uint4*>(emb + (size_t)id * d + c);
  const uint32_t u[4] = {b.x, b.y, b.z, b.w};
  float v[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) v[i] = bf16_bits_to_float((u[i >> 1] >> (16 * (i & 1))) & 0xFFFFu);
  const float4 g0 = *reinterpret_cast<const float4*>(gain + c), g1 = *reinterpret_cast<const float4*>(gain + c + 4);
  uint4 hi, lo;
  bf16_split2(v[0] * g0.x, v[1] * g0.y, hi.x, lo.x);
  bf16_split2(v[2] * g0.z, v[3] * g0.w, hi.y, lo.y);
  bf16_split2(v[4] * g1.x, v[5] * g1.y, hi.z, lo.z);
  bf16_split2(v[6] * g1.z, v[7] * g1.w, hi.w, lo.w);
  uint4* dst = frag + ((size_t)kt * RT + blockIdx.y) * 128 + lane;
  dst[0] = hi;
  dst[64] = lo;
  float ss = sumsq4(v[0], v[1], v[2], v[3]) + sumsq4(v[4], v[5], v[6], v[7]);
  ss += __shfl_xor(ss, 16);
  ss += __shfl_xor(ss, 32);
  if (r >= R) return;
  float4* xr = reinterpret_cast<float4*>(x + (size_t)r * d + c);
  xr[0] = make_float4(v[0], v[1], v[2], v[3]);
  xr[1] = make_float4(v[4], v[5], v[6], v[7]);
  if (lane < 16) ssq[(size_t)r * (d / kBlkSsqCols) + kt] = ss;
}
void launch_blk_embed(const uint16_t* emb, const int* tokens, int tok_stride, int tok_cap, int vocab, const int2* rows, int R, int d,
                      float* x, const float* gain, uint4* frag, float* ssq, hipStream_t st) {
  hipLaunchKernelGGL(k_blk_embed, dim3((d + 127) / 128, (R + 15) / 16), dim3(256), 0, st, emb, tokens, tok_stride, tok_cap, vocab, rows, R, d,
                     x, gain, frag, pf_col_tiles(R), ssq);
}

// ---------------------------------------------------------------------------------------
// block GEMM
// ---------------------------------------------------------------------------------------
// 1 / rms of row `row` of the input, by 4 lanes (q = 0 .. 3; `near` and `far` are their two lane distances)
__device__ __forceinline__ float blk_row_rstd(const BlkGemm& p, int row, int q, int near, int far) {
  const float* src = p.ssq + (size_t)row * p.ssq_n;
  float ss = 0.f;
  for (int i = q * 4; i < p.ssq_n; i += 16) {          // (ssq_n is a multiple of 8)
    const float4 v = *reinterpret_cast<const float4*>(src + i);
    ss += (v.x + v.y) + (v.z + v.w);
  }
  ss += __shfl_xor(ss, near);
  ss += __shfl_xor(ss, far);
  return 1.0f / sqrtf(ss / (float)p.K + p.eps);
}

// What a launch does with its sums (BlkGemm::kind): a wave holds NT weight tiles x CT column tiles as the MFMA leaves
// them, lane = 16 g + j: outputs 16 (tile0 + t) + 4 g .. + 3 of row row0 + 16 ct (row0 includes j).  Both the GEMM and
// the kernel that adds up k pieces end here, so the bits do not depend on which of the two a launch takes.  What has to
// be read (old x, rotation entries, positions) is requested ahead of the stores of a whole column tile: the compiler
// may not move loads over stores, and one after the other they cost a work-group as much as its k loop.
template <int NT, int CT>
__device__ __forceinline__ void blk_epilogue(const BlkGemm& p, const f32x4 (&sums)[NT][CT], int tile0, int row0, int g, const float (&rs)[CT]) {
  // (rs is 1 where nothing is normalised; single floats from here on: exchanged as parts of the MFMAs' register
  // quadruples the accumulators of the larger tiles spill)
  float acc[NT][CT][4];
#pragma unroll
  for (int ct = 0; ct < CT; ++ct)
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int i = 0; i < 4; ++i) acc[t][ct][i] = sums[t][ct][i] * rs[ct];
  if constexpr (CT % 2 == 0) if (p.kind == kBlkSwiglu || p.kind == kBlkQKV) {
    // Columns 0..7 and 8..15 of a tile belong together (gate / up, the halves of rotation pairs).  The lower half of the
    // wave holds the first eight, the upper half the second: after exchanging the upper half of column tile ct with the
    // lower half of ct + 1, acc[t][ct] is the first and acc[t][ct + 1] the second member of every lane's pairs; the
    // lower half works on column tile ct, the upper half on ct + 1.
    const bool up = g >= 2;
    g &= 1;
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int ct = 0; ct < CT; ct += 2)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(acc[t][ct][i]), __float_as_uint(acc[t][ct + 1][i]), false, false);
          acc[t][ct][i] = __uint_as_float(r[0]);
          acc[t][ct + 1][i] = __uint_as_float(r[1]);
        }
    if (p.kind == kBlkSwiglu) {
#pragma unroll
      for (int ct = 0; ct < CT; ct += 2) {
        const int row = row0 + (ct + (up ? 1 : 0)) * 16;
        if (row < p.R)
#pragma unroll
          for (int t = 0; t < NT; ++t) {
            const float (&a)[4] = acc[t][ct], (&b)[4] = acc[t][ct + 1];
            if (tile0 + t < p.NTILES)
              blk_store_frag4(p.frag_out, p.RT, row, (tile0 + t) * 8 + 4 * g,
                              make_float4(swiglu(a[0], b[0]), swiglu(a[1], b[1]), swiglu(a[2], b[2]), swiglu(a[3], b[3])));
            __builtin_amdgcn_sched_barrier(0);         // (here and below: else the tiles' work is interleaved until it spills)
          }
      }
      return;
    }
    const int hd = p.hd, half = hd >> 1;
    constexpr int G = NT;                          // tiles whose rotation entries are requested together
    int2 at[CT / 2];
#pragma unroll
    for (int c2 = 0; c2 < CT / 2; ++c2) at[c2] = p.rows[min(row0 + (2 * c2 + (up ? 1 : 0)) * 16, p.R - 1)];
#pragma unroll
    for (int c2 = 0; c2 < CT / 2; ++c2) {
      const int row = row0 + (2 * c2 + (up ? 1 : 0)) * 16;
      const bool cached = row < p.R && at[c2].y >= 0 && at[c2].y < p.cap;
#pragma unroll
      for (int t0 = 0; t0 < NT; t0 += G) {
      float4 cs[G][2];
#pragma unroll
      for (int q = 0; q < G; ++q) {
        const int n = min(tile0 + t0 + q, p.NTILES - 1) * 16, w = n % p.da % hd;
        const float4* src = reinterpret_cast<const float4*>(p.cs + min(row, p.R - 1) * 64 + (w >> 4) * 8 + 4 * g);
        cs[q][0] = src[0];
        cs[q][1] = src[1];
      }
#pragma unroll
      for (int q = 0; q < G; ++q) {
        const int t = t0 + q;
        if (tile0 + t >= p.NTILES) continue;
        const float (&a)[4] = acc[t][2 * c2], (&b)[4] = acc[t][2 * c2 + 1];
        const int n = (tile0 + t) * 16, part = n / p.da, c = n - part * p.da, h = c / hd, w = c - h * hd;
        const size_t off = (size_t)at[c2].x * p.slot_stride + (size_t)h * p.cap * hd;
        if (part == 2) {
          if (cached)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              store_kv(p.Vc + off + v_cache_off(at[c2].y, w + 4 * g + i, hd), a[i]);
              store_kv(p.Vc + off + v_cache_off(at[c2].y, w + 8 + 4 * g + i, hd), b[i]);
            }
          continue;
        }
        const int e = (w >> 4) * 8 + 4 * g;
        const float2 r0 = rope_rotate(a[0], b[0], make_float2(cs[q][0].x, cs[q][0].y)), r1 = rope_rotate(a[1], b[1], make_float2(cs[q][0].z, cs[q][0].w));
        const float2 r2 = rope_rotate(a[2], b[2], make_float2(cs[q][1].x, cs[q][1].y)), r3 = rope_rotate(a[3], b[3], make_float2(cs[q][1].z, cs[q][1].w));
        if (part == 0) {
          if (row < p.R) {
            float* dst = p.out + (size_t)row * p.da + h * hd + e;
            *reinterpret_cast<float4*>(dst) = make_float4(r0.x, r1.x, r2.x, r3.x);
            *reinterpret_cast<float4*>(dst + half) = make_float4(r0.y, r1.y, r2.y, r3.y);
          }
        } else if (cached) {
          store_kv4(p.Kc + off + k_cache_off(at[c2].y, e, hd), make_float4(r0.x, r1.x, r2.x, r3.x));
          store_kv4(p.Kc + off + k_cache_off(at[c2].y, e + half, hd), make_float4(r0.y, r1.y, r2.y, r3.y));
        }
      }
      __builtin_amdgcn_sched_barrier(0);
      }
    }
    return;
  }
  if constexpr (NT % 2 == 0) if (p.kind == kBlkResid) {
    constexpr int G = NT;                          // tiles whose old values are requested together
#pragma unroll
    for (int t0 = 0; t0 < NT; t0 += G) {
      float4 gain[G];
      if (p.frag_out)
#pragma unroll
        for (int q = 0; q < G; ++q) gain[q] = *reinterpret_cast<const float4*>(p.gain + min(tile0 + t0 + q, p.NTILES - 1) * 16 + 4 * g);
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) {
        const int row = row0 + ct * 16;
        float* xr = p.out + (size_t)min(row, p.R - 1) * p.ldo + 4 * g;
        float4 old[G];
#pragma unroll
        for (int q = 0; q < G; ++q) old[q] = *reinterpret_cast<const float4*>(xr + min(tile0 + t0 + q, p.NTILES - 1) * 16);
#pragma unroll
        for (int q2 = 0; q2 < G; q2 += 2) {
          const int tile = tile0 + t0 + q2;
          const bool ok = row < p.R && tile < p.NTILES;  // (N is a multiple of 256: tiles come in pairs)
          float ss = 0.f;
#pragma unroll
          for (int q = q2; q < q2 + 2; ++q) {
            const float (&a)[4] = acc[t0 + q][ct];
            const float4 o = old[q], v = make_float4(o.x + a[0], o.y + a[1], o.z + a[2], o.w + a[3]);
            if (ok) {
              const int n = (tile0 + t0 + q) * 16;
              *reinterpret_cast<float4*>(xr + n) = v;
              if (p.frag_out)
                blk_store_frag4(p.frag_out, p.RT, row, n + 4 * g, make_float4(v.x * gain[q].x, v.y * gain[q].y, v.z * gain[q].z, v.w * gain[q].w));
            }
            ss += sumsq4(v.x, v.y, v.z, v.w);
          }
          if (p.ssq_out) {
            ss += __shfl_xor(ss, 16);
            ss += __shfl_xor(ss, 32);
            if (g == 0 && ok) p.ssq_out[(size_t)row * (p.ldo / kBlkSsqCols) + tile / 2] = ss;
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    return;
  }
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
      const int row = row0 + ct * 16, n = (tile0 + t) * 16 + 4 * g;
      const float (&v)[4] = acc[t][ct];
      if (row >= p.R || tile0 + t >= p.NTILES) continue;
      if (p.kind == kBlkRelu)
        blk_store_frag4(p.frag_out, p.RT, row, n, make_float4(fmaxf(v[0], 0.f), fmaxf(v[1], 0.f), fmaxf(v[2], 0.f), fmaxf(v[3], 0.f)));
      else
        *reinterpret_cast<float4*>(p.out + (size_t)row * p.ldo + n) = make_float4(v[0], v[1], v[2], v[3]);
      __builtin_amdgcn_sched_barrier(0);
    }
}

// Sums[R, N] = X[R, K] . W[N, K]^T for row blocks of up to thousands of rows: the MFMA-bound regime.
//   W: the operand-tile layout of the decode kernels (1 KiB MFMA A operands); X: block fragments (above, 1 KiB B operands).
//   Work-group = WF x WR waves, each 4 weight tiles x CT column tiles of fp32 accumulators; a k-step of 32 is
//   WF*4 + 2*WR*CT KiB-sized operands, copied from memory straight into LDS (buffer_load ... lds, 16 bytes per lane: no
//   staging registers, and every operand enters the CU once), ST k-steps deep, and read from there as they lie
//   (ds_read_b128, no bank conflicts: the layouts are lane order).
//   Where each wave has weight tiles of its own (WR = 1), only the fragments go through LDS: a weight tile is loaded into the
//   wave's registers two k-steps ahead, into those of the tile whose MFMAs were just issued.  LDS then takes 8 instead of 24
//   KiB a k-step in and 32 instead of 48 out (busy 16 % of the cycles, 24 before), and a k-step's reads are 8, not 12.
//   256 x 64 tiles, traced: 2048 rows, 7B QKV and gate/up 434 -> 408 us, 333 rows, pieces 101 -> 96 us; calls: 2048-token prompt
//   1.01x, 333 1.02x.
//   One barrier per k-step: the wave waits for its own copies of k-step s + 1 (those of the following ones stay in
//   flight: the waits count instructions), the barrier makes everybody's visible and says that everybody holds k-step s
//   in registers, so its buffer takes the copies of s + ST.
//   k pieces: the k range is cut into p.pieces parts that are summed separately (k ascending, high before low) and added
//   up in order: by different work-groups and k_blk_reduce (gridDim.z = pieces), or one after the other by the same
//   work-group with a second set of accumulators (PIECED).  The bits depend on p.pieces alone, not on R, the tile shape
//   or the grid.
//   What bounds it: at thousands of rows the issue of MFMAs, 1.23 .. 1.30 PFLOP/s with plain stores in launches by
//   themselves (2047 rows, 7B projections; a library product of two 8192-wide matrices: 1.49 on the same card) and 1.07 over
//   a profiled 2048-token prompt with its epilogues (matrix cores busy in 0.69 of the cycles, at 1.74 GHz: the card lowers its
//   clock under this load, so fewer idle cycles gain less than they save); at a few hundred the rounds of work-groups and, with one work-group on a
//   CU, the pace of a single wave per SIMD (kBlkShapes); at <= 64 rows the weights' way from memory.
//   Plain stores, against the kernel before (weights through registers, 256 x 128 tiles only), 7B projections, us:
//   2047 rows: QKV 384 -> 323, out 115 -> 107, gate/up 712 -> 600, down 297 -> 284; 333 rows: 111 -> 83, 45 -> 35,
//   198 -> 140, 96 -> 75; 60 (now 64) rows: 45 -> 28, 23 -> 17, 78 -> 40, 38 -> 28.  The SwiGLU epilogue costs less than plain
//   stores.  (A first form of this loop read k-step s from LDS in front of its MFMAs: 0.52 us per k-step with
//   one work-group on a CU, whatever the depth of the ring.)
template <int N> __device__ __forceinline__ void wait_copies_and_sync() {
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}
// lane l: lds_base[l] = base[offset / 16 + l] (buffer form: its waits do not hold up the LDS reads in flight, as those
// of the flat-encoded form do, and the address arithmetic is scalar)
__device__ __forceinline__ void copy_to_lds_16(const uint4* base, uint32_t offset, uint4* lds_base, uint32_t lane_bytes) {
  const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint4*>(base), 0, 0xFFFFFFFFu, 0x00027000);
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void*)(static_cast<uint32_t>(reinterpret_cast<uintptr_t>(lds_base))), 16,
                                           lane_bytes, offset, 0, 0);
}
constexpr int kBlkNT = 4;                              // weight tiles of a wave
constexpr int blk_lds_bytes(int WF, int WR, int CT, int ST) {
  return ST * ((WR == 1 ? 0 : WF * kBlkNT) + 2 * WR * CT) * 1024 + WR * CT * 64;
}

//   CT: column tiles of a wave, ST: k-steps in LDS.  4 and 3 for many rows (24 KiB a k-step); 2 and 4 (16 KiB) where half the
//   rows a work-group make the rounds come out or all CUs have work: see kBlkShapes.
template <int WF, int WR, int CT, int ST, bool PIECED>
__global__ __launch_bounds__(64 * WF * WR) __attribute__((amdgpu_waves_per_eu(2, 2)))
void k_gemm_bf16_block(BlkGemm p, float* part, int RB, int per_xcd, int nblocks) {
  constexpr int NT = kBlkNT;
  constexpr bool DIRECT = WR == 1;                     // each wave loads its weight tiles itself, two k-steps ahead
  constexpr int NW = WF * WR, AT = WF * NT, LT = DIRECT ? 0 : AT, BT = 2 * WR * CT, STAGE = (LT + BT) * 64;   // uint4 per LDS stage
  constexpr int PER = (LT + BT) / NW;                                                   // copies per wave and k-step
  static_assert(LT % NW == 0 && BT % NW == 0 && (ST - 1) * PER < 48, "whole copies per wave, countable by vmcnt");
  static_assert(!DIRECT || (ST == 3 && CT == NT), "the order of requests the waits count");
  extern __shared__ uint4 lds[];                       // [ST][weight tiles AT | fragments BT][64], then the rows' 1/rms
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int fw = wave % WF, rw = wave / WF;
  const int j = lane & 15, g = lane >> 4;
  // Work-groups go round-robin to the 8 XCDs: each XCD takes a contiguous run of (feature block, row block) pairs, row
  // blocks fastest, so that the row blocks that share weight tiles meet in one L2.
  const int lin = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if (lin >= nblocks) return;                          // (whole work-groups, before any barrier)
  const int fb = lin / RB, rb = lin - fb * RB;
  const int ksteps = p.K >> 5, P = p.pieces;
  // (pieces begin at even k-steps, differ by at most two of them and have at least 8: launch_blk_gemm)
  auto piece_begin = [&](int i) { return ksteps * i / P & ~1; };
  const int piece0 = PIECED ? 0 : (int)blockIdx.z;
  const bool split = gridDim.z > 1;
  const int ks0 = split ? piece_begin(piece0) : 0, ks_end = split && piece0 + 1 < P ? piece_begin(piece0 + 1) : ksteps;

  // copies of the next k-step into LDS buffer buf: every NW-th operand of the stage is this wave's (tiles past the matrix
  // and column tiles past the fragment buffer repeat the last one, their results are dropped)
  const int full_chunks = ksteps >> 4;                 // (the last chunk may be half as long)
  uint32_t off[PER];                                   // bytes from the chunk's (weights) or the k-step's (fragments) start
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    const int i = wave + q * NW;
    off[q] = q < LT / NW ? (uint32_t)min(p.tile_first + fb * AT + i, p.NTILES - 1) * (kSliceUnits * 8 * 1024u)
                         : (uint32_t)min(rb * BT + i - LT, 2 * p.RT - 1) * 1024u;
  }
  uint32_t aoff[DIRECT ? NT : 1];
  if constexpr (DIRECT)
#pragma unroll
    for (int t = 0; t < NT; ++t) aoff[t] = (uint32_t)min(p.tile_first + fb * AT + fw * NT + t, p.NTILES - 1) * (kSliceUnits * 8 * 1024u);
  int rs_ = ks0;                                       // the next k-step (DIRECT: of the weights)
  const uint4* wp = p.W + ((size_t)(ks0 >> 4) * p.NTILES * (kSliceUnits * 8) + (ks0 & 15)) * 64;
  const uint4* xp = p.XF + (size_t)ks0 * p.RT * 128;
  const size_t wskip = (size_t)(p.NTILES - 1) * (kSliceUnits * 8) * 64, xstep = (size_t)p.RT * 128;
  auto next_weights = [&]() {
    ++rs_;
    wp += 64;
    if ((rs_ & 15) == 0) wp += wskip;
  };
  auto request = [&](int buf) {
    const int half = __builtin_amdgcn_readfirstlane((rs_ >> 4) >= full_chunks ? 1 : 0);
    uint4* dst = lds + buf * STAGE + wave * 64;
#pragma unroll
    for (int q = 0; q < PER; ++q) copy_to_lds_16(q < LT / NW ? wp : xp, q < LT / NW ? off[q] >> half : off[q], dst + q * NW * 64, lane * 16);
    if constexpr (!DIRECT) next_weights();
    xp += xstep;
  };
  f32x4 acc[NT][CT], tot[PIECED ? NT : 1][PIECED ? CT : 1];
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) acc[t][ct] = f32x4{0.f, 0.f, 0.f, 0.f};
  struct Frags {
    bf16x8 a[NT], h[CT], l[CT];
  };
  auto read = [&](Frags& f, int buf) {
    const uint4* sa = lds + buf * STAGE + fw * NT * 64 + lane;
    const uint4* sb = lds + buf * STAGE + (LT + rw * CT * 2) * 64 + lane;
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
      f.h[ct] = __builtin_bit_cast(bf16x8, sb[(ct * 2) * 64]);
      f.l[ct] = __builtin_bit_cast(bf16x8, sb[(ct * 2 + 1) * 64]);
    }
    if constexpr (!DIRECT)
#pragma unroll
      for (int t = 0; t < NT; ++t) f.a[t] = __builtin_bit_cast(bf16x8, sa[t * 64]);
  };
  auto multiply_tile = [&](const Frags& f, int t) {
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) acc[t][ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f.a[t], f.h[ct], acc[t][ct], 0, 0, 0);
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) acc[t][ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f.a[t], f.l[ct], acc[t][ct], 0, 0, 0);
  };
  auto multiply = [&](const Frags& f) {
#pragma unroll
    for (int t = 0; t < NT; ++t) multiply_tile(f, t);
  };
  // DIRECT: weight tile t of the next k-step not yet requested
  auto load_weights = [&](Frags& f, int t) {
    const int half = __builtin_amdgcn_readfirstlane((rs_ >> 4) >= full_chunks ? 1 : 0);
    const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint4*>(wp), 0, 0xFFFFFFFFu, 0x00027000);
    f.a[t] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(r, lane * 16, aoff[t] >> half, 0));
  };
  // the rows' 1/rms, while the first copies are on their way (its loads go first, so the counted waits cover them)
  float* s_rstd = reinterpret_cast<float*>(lds + ST * STAGE);
  if (p.ssq && part == nullptr)
    for (int r = tid >> 2; r < WR * CT * 16; r += 16 * NW) {
      const float v = blk_row_rstd(p, min(rb * WR * CT * 16 + r, p.R - 1), tid & 3, 1, 2);
      if ((tid & 3) == 0) s_rstd[r] = v;
    }
  int piece = 0, bound = PIECED ? piece_begin(1) : 0;
  auto fold = [&](int ks) {                            // PIECED: a piece ends in front of k-step ks
    if constexpr (PIECED) {
      if (ks == bound) {
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
          for (int ct = 0; ct < CT; ++ct) {
            tot[t][ct] = piece == 0 ? acc[t][ct] : tot[t][ct] + acc[t][ct];
            acc[t][ct] = f32x4{0.f, 0.f, 0.f, 0.f};
          }
        ++piece;
        bound = piece_begin(piece + 1);
      }
    }
  };
  // The fragments of k-step s + 1 are read from LDS while the MFMAs of k-step s run (two register sets), so buffer
  // s % ST is free again at the barrier in front of k-step s and takes the copies of s + ST.  With one or two waves on a
  // SIMD everything that is not an MFMA has to be issued in their shadow: requests and LDS reads are dealt out between
  // them (all in front of them, a lone work-group took 0.52 us per k-step of 32 MFMAs a wave whatever the depth of the
  // ring; see kBlkShapes).
  Frags f0, f1;
  // (a piece has at least 8 k-steps; DIRECT: in the order in which the loop requests them, the copies of k-step s + 3 and then
  // the weights of s + 2)
  constexpr int AHEAD = DIRECT ? 2 * NT : 0;           // weight loads younger than the copies a wait is for
#pragma unroll
  for (int i = 0; i < ST; ++i) {
    request(i);
    if constexpr (DIRECT) {
      __builtin_amdgcn_sched_barrier(0);
      if (i >= ST - 2) {
#pragma unroll
        for (int t = 0; t < NT; ++t) load_weights(i == ST - 2 ? f0 : f1, t);
        next_weights();
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
  wait_copies_and_sync<(ST - 1) * PER + AHEAD>();
  read(f0, 0);
  int s = ks0, rbuf = 1, wbuf = 0;                     // buffers of k-steps s + 1 and s + ST
  auto advance = [&]() {
    rbuf = rbuf + 1 == ST ? 0 : rbuf + 1;
    wbuf = wbuf + 1 == ST ? 0 : wbuf + 1;
    ++s;
  };
  constexpr int MFMAS = 2 * NT * CT, READS = (DIRECT ? 0 : NT) + 2 * CT, GAP = (MFMAS - PER) / READS;
  static_assert(GAP >= 1, "an MFMA in front of every request and read");
  // DIRECT: k-step s tile by tile; the registers of a weight tile take the tile of s + 2 as soon as its MFMAs are issued
  auto step_direct = [&](Frags& cur, Frags& next, bool copies) {
    const uint4* sb = lds + rbuf * STAGE + lane;
    if (copies) request(wbuf);
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      if (t > 0) load_weights(cur, t - 1);
      if constexpr (DIRECT) {
        next.h[t] = __builtin_bit_cast(bf16x8, sb[(t * 2) * 64]);
        next.l[t] = __builtin_bit_cast(bf16x8, sb[(t * 2 + 1) * 64]);
      }
      multiply_tile(cur, t);
#pragma unroll
      for (int i = 0; i < (t > 0 ? 1 : copies ? PER : 0); ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
      }
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      }
      __builtin_amdgcn_sched_group_barrier(0x008, 2 * CT, 0);
      __builtin_amdgcn_sched_barrier(0);               // (the waits count on the order of the requests)
    }
    load_weights(cur, NT - 1);
    next_weights();
    __builtin_amdgcn_sched_barrier(0);
    advance();
  };
  auto step = [&](Frags& cur, Frags& next) {           // any k-step but the last ST
    wait_copies_and_sync<(ST - 2) * PER + AHEAD>();
    if constexpr (DIRECT) {
      step_direct(cur, next, true);
      return;
    }
    request(wbuf);
    read(next, rbuf);
    multiply(cur);
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
    }
#pragma unroll
    for (int i = 0; i < READS; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, GAP, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    }
    __builtin_amdgcn_sched_group_barrier(0x008, MFMAS - PER - READS * GAP, 0);
    advance();
  };
  while (s + 1 + ST < ks_end) {
    fold(s);                                           // (pieces begin at even k-steps, and none among the last 8)
    step(f0, f1);
    step(f1, f0);
  }
  // The number of k-steps is even (pieces begin at even ones, K is whole units of 8), so ST of them are left where ST is even,
  // else ST + 1; nothing more to request for the last ST, so the waits count down
  auto last = [&](auto self, auto I, Frags& x, Frags& y) -> void {
    constexpr int i = decltype(I)::value;
    if constexpr (i < ST - 1) wait_copies_and_sync<(ST - 2 - i) * PER + AHEAD>();
    if constexpr (DIRECT && i == 0) {
      step_direct(x, y, false);
      self(self, std::integral_constant<int, i + 1>{}, y, x);
      return;
    }
    if constexpr (i < ST - 1) read(y, rbuf);
    multiply(x);
    if constexpr (i < ST - 1 && CT == 2) {             // (with 4 column tiles it spills)
#pragma unroll
      for (int q = 0; q < READS; ++q) {
        __builtin_amdgcn_sched_group_barrier(0x008, MFMAS / READS, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      }
      __builtin_amdgcn_sched_group_barrier(0x008, MFMAS % READS, 0);
    }
    advance();
    if constexpr (i < ST - 1) self(self, std::integral_constant<int, i + 1>{}, y, x);
  };
  fold(s);
  if constexpr (ST % 2 == 1) {
    step(f0, f1);
    last(last, std::integral_constant<int, 0>{}, f1, f0);
  } else {
    last(last, std::integral_constant<int, 0>{}, f0, f1);
  }
  if constexpr (PIECED) {
    if (piece > 0) {
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) acc[t][ct] = tot[t][ct] + acc[t][ct];
    }
  }

  const int tile0 = p.tile_first + fb * AT + fw * NT, row0 = (rb * WR + rw) * CT * 16 + j;   // column tile ct: row0 + 16 ct
  if (part) {                                          // one piece: its sums as they lie, [piece][tile][column tile][lane]
    const int ntiles = p.NTILES - p.tile_first, cts = (p.R + 15) >> 4;
    float4* dst = reinterpret_cast<float4*>(part) + ((size_t)piece0 * ntiles + (tile0 - p.tile_first)) * cts * 64 + lane;
    const int ct0 = (rb * WR + rw) * CT;
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int ct = 0; ct < CT; ++ct)
        if (tile0 + t < p.NTILES && ct0 + ct < cts)
          dst[((size_t)t * cts + ct0 + ct) * 64] = make_float4(acc[t][ct][0], acc[t][ct][1], acc[t][ct][2], acc[t][ct][3]);
    return;
  }
#pragma unroll
  for (int ct = 0; ct < CT; ct += 2) {                 // (two column tiles at a time: more at once spill)
    f32x4 part2[NT][2];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      part2[t][0] = acc[t][ct];
      part2[t][1] = acc[t][ct + 1];
    }
    const float* sr = s_rstd + (rw * CT + ct) * 16 + j;
    const float rs[2] = {p.ssq ? sr[0] : 1.f, p.ssq ? sr[16] : 1.f};
    blk_epilogue<NT, 2>(p, part2, tile0, row0 + ct * 16, g, rs);
    __builtin_amdgcn_sched_barrier(0);
  }
}

// The k pieces of a launch with few rows added up in order, then the launch's epilogue: a wave takes two weight tiles x two
// column tiles or, where that leaves SIMDs without a wave, the two its epilogue combines; up to four pieces are requested
// together.  Bound by round trips (192 rows, 128 tiles, 4 / 8 pieces with the product: 17.4 -> 16.3 / 29.6 -> 28.5 us; 48 tiles
// of 768: 10.9 -> 10.4).
template <int NT, int CT>
__global__ __launch_bounds__(256) void k_blk_reduce(BlkGemm p, const float* __restrict__ part) {
  const int lane = threadIdx.x & 63, g = lane >> 4, j = lane & 15;
  const int ntiles = p.NTILES - p.tile_first, cts = (p.R + 15) >> 4;
  const int t0 = (blockIdx.x * 4 + (threadIdx.x >> 6)) * NT, ct0 = blockIdx.y * CT;
  if (t0 >= ntiles) return;                            // (whole waves; no barriers)
  const float4* src = reinterpret_cast<const float4*>(part) + lane;
  f32x4 acc[NT][CT];
  for (int z0 = 0; z0 < p.pieces; z0 += 4) {
    float4 v[4][NT][CT];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int ct = 0; ct < CT; ++ct)
          v[i][t][ct] = src[(((size_t)min(z0 + i, p.pieces - 1) * ntiles + min(t0 + t, ntiles - 1)) * cts + min(ct0 + ct, cts - 1)) * 64];
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (z0 + i < p.pieces)
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
          for (int ct = 0; ct < CT; ++ct) {
            const f32x4 u = {v[i][t][ct].x, v[i][t][ct].y, v[i][t][ct].z, v[i][t][ct].w};
            acc[t][ct] = z0 + i == 0 ? u : acc[t][ct] + u;
          }
  }
  float rs[CT];
  const int row0 = ct0 * 16 + j;
#pragma unroll
  for (int ct = 0; ct < CT; ++ct) rs[ct] = p.ssq ? blk_row_rstd(p, min(row0 + ct * 16, p.R - 1), g, 16, 32) : 1.f;
  blk_epilogue<NT, CT>(p, acc, p.tile_first + t0, row0, g, rs);
}

// Tile shapes: features x rows of a work-group (two fit a CU), and the microseconds of a k-step with one work-group on the CU
// and with two: fitted to 17 projections of the 125M, 1B, 7B and wide encoder widths at 12 row counts from 40 to 2047, every
// shape and way of summing timed, while the 256 x 64 shape still copied its weights into LDS.  Whole launches of 100 to 256
// work-groups, k of 2048 and more, take 0.39 .. 0.57 (0.34 .. 0.57 since 256 x 64 loads its weights itself) and, the third
// shape, 0.25 .. 0.42 us a k-step with their start and end.  The third shape does half the work a step of the others in a little
// more than half the time: it wins wherever it puts work on more CUs or the rounds come out better (us, the best of the other two in
// brackets: 192 rows, 6144 x 2048 21.1 (24.9); 128 rows, 16384 x 2048 22.7 (31.0), 16384 x 1024 14.8 (19.8), 12288 x 4096 37.7
// (40.1); 64 rows, 32000 x 2048 26.8 (35.2); 333 rows, 6144 x 768 14.8 (15.2)).  Shapes with larger
// wave tiles (256 x 256 on 8 waves, 256 x 128 and 192 x 128 on 4) were no faster at 2047 rows (7B gate/up 588, 633 and 617 us
// against 602).  Two k-steps for each barrier (rings of two to four pairs) were slower in every shape (64 rows, 2048 x 8192
// in one piece: 64 -> 77..83 us), deeper rings no faster.
struct BlkShape { int feat, rows; float one, two; };
// (numbers: bit 0 the orientation, bit 1 half the size; the half of 128 x 128 is not built)
constexpr int kBlkShapeCount = 4;
constexpr BlkShape kBlkShapes[kBlkShapeCount] = {{128, 128, 0.435f, 0.84f}, {256, 64, 0.434f, 0.839f}, {0, 0, 0.f, 0.f}, {128, 64, 0.273f, 0.477f}};

// floats the pieces of a split launch take
static size_t blk_part_floats(const BlkGemm& p) { return (size_t)p.pieces * ((p.R + 15) / 16 * 16) * ((p.NTILES - p.tile_first) * 16); }

// The kernel's prologue requests the first ST (3 or 4) k-steps of its piece unasked and its loop ends on the last ST + 1: a
// piece shorter than that would copy k-steps that are not its own, at the end of the range operands past the matrix (the
// copies carry no bounds).  K is whole units of the weight layout (256 k); pieces end at ksteps * i / pieces rounded down
// to even, which moves an end by less than two: all of them have 8 k-steps exactly if 8 * pieces <= ksteps.
bool blk_pieces_fit(int K, int pieces) { return K >= 256 && K % 256 == 0 && pieces >= 1 && pieces <= K / 256; }

hipError_t launch_blk_gemm_as(int shape, bool split, const BlkGemm& p, hipStream_t st, float* part, size_t part_floats) {
  if (shape < 0 || shape >= kBlkShapeCount || !kBlkShapes[shape].feat || p.R < 1 || p.RT * 16 < p.R || p.tile_first < 0 || p.tile_first >= p.NTILES ||
      !blk_pieces_fit(p.K, p.pieces))
    return hipErrorInvalidValue;
  const BlkShape& b = kBlkShapes[shape];
  const int N = (p.NTILES - p.tile_first) * 16;
  if (split && (p.pieces == 1 || !part || blk_part_floats(p) > part_floats)) return hipErrorInvalidValue;
  const int FB = (N + b.feat - 1) / b.feat, RB = (p.R + b.rows - 1) / b.rows;
  const int blocks = FB * RB, per_xcd = (blocks + 7) / 8;
  const dim3 grid(per_xcd * 8, 1, split ? p.pieces : 1), block(256);
  float* dst = split ? part : nullptr;
#define STAIRS_BLK(WF, WR, CT, ST)                                                                                        \
  hipLaunchKernelGGL((pieced ? k_gemm_bf16_block<WF, WR, CT, ST, true> : k_gemm_bf16_block<WF, WR, CT, ST, false>), grid, block, \
                     blk_lds_bytes(WF, WR, CT, ST), st, p, dst, RB, per_xcd, blocks)
  const bool pieced = p.pieces > 1 && !split;
  if (shape == 0) STAIRS_BLK(2, 2, 4, 3);
  else if (shape == 1) STAIRS_BLK(4, 1, 4, 3);
  else STAIRS_BLK(2, 2, 2, 4);
#undef STAIRS_BLK
  if (split) {
    // (two by two tiles where that leaves every SIMD a wave: 333 rows, 768 tiles 92 against 100 us by halves)
    const int cts = (p.R + 15) / 16;
    if (N / 16 * cts >= 4096) hipLaunchKernelGGL((k_blk_reduce<2, 2>), dim3((N / 16 + 7) / 8, (p.R + 31) / 32), dim3(256), 0, st, p, part);
    else if (p.kind == kBlkResid) hipLaunchKernelGGL((k_blk_reduce<2, 1>), dim3((N / 16 + 7) / 8, cts), dim3(256), 0, st, p, part);
    else hipLaunchKernelGGL((k_blk_reduce<1, 2>), dim3((N / 16 + 3) / 4, (p.R + 31) / 32), dim3(256), 0, st, p, part);
  }
  return hipSuccess;
}

// Pieces of a k range for blocks of rows that belong to sequences of at most kBlkPiecedRows rows each: a function of K
// alone, so that a row's bits are the same in whatever block it is computed.  K / 256 below 1024 (1..3), 4 from there to
// 5119, then K / 1024 (8 for 8192, 10 for 11008).  No count is best at all row counts.  Rule against the best of 1 .. 17 at 60
// / 128 / 333 rows, us (N x K): 6144 x 2048 14.1 / 16.1 / 29.9 against 14.1 / 16.1 / 27.9 (4, 5, 3 pieces), 4096 x 4096 19.5
// / 21.2 / 35.0 against 16.5 / 19.3 / 33.9 (9, 7, 5), 12288 x 4096 26.9 / 39.3 / 86.7 against 26.9 / 36.4 / 83.9 (4, 2, 3),
// 2048 x 8192 23.5 / 26.6 / 37.5 against 19.4 / 21.4 / 32.0 (11, 11, 5), 4096 x 11008 28.0 / 40.5 / 77.0 against 27.5 / 32.3
// / 66.1 (9, 8, 5).  Beyond 1024 rows no launch gains from cutting k.
int blk_pieces(int K) {
  const int ksteps = K / 32;
  return std::min(ksteps / 8, std::max(4, ksteps / 32));
}

// The tile shape and the way the pieces are summed, by a model of the launch's time: rounds of work-groups over the 256
// CUs, each k-step at the rate of the shape's occupancy (a CU with two work-groups sets the pace as soon as there is one; a last
// round of few is partly hidden behind the one before), the matrix at the rate memory delivers it, and for a split launch the
// pieces' way through memory and the second kernel.  Over 247 launches (19 projections, 40 to 2047 rows, timed with the kernels as
// they are) the choice costs 0.8 % against the best of all, 18 % at most (768 x 3072, 777 rows: 20.6 against 17.4 us; 12288 x
// 4096, 160 rows: 59.0 against 51.9); two shapes and the model before cost 12 %.
hipError_t launch_blk_gemm(BlkGemm p, bool pieced, hipStream_t st, float* part, size_t part_floats) {
  p.pieces = pieced ? blk_pieces(p.K) : 1;
  const int N = (p.NTILES - p.tile_first) * 16, ksteps = p.K / 32;
  int best = 0;
  bool best_split = false;
  float best_us = 1e30f;
  for (int s = 0; s < kBlkShapeCount; ++s) {
    const BlkShape& b = kBlkShapes[s];
    if (!b.feat) continue;
    const int blocks = ((N + b.feat - 1) / b.feat) * ((p.R + b.rows - 1) / b.rows);
    for (int split = 0; split < 2; ++split) {
      if (split && (p.pieces == 1 || !part || blk_part_floats(p) > part_floats)) continue;
      const int wgs = split ? blocks * p.pieces : blocks, full = wgs / 512, rem = wgs - full * 512;
      float rounds = full * b.two;
      if (rem > 256) rounds += b.one + (b.two - b.one) * (0.55f + 0.45f * (rem - 256) / 256);
      else if (rem > 0) rounds += full > 0 ? 0.74f * b.one : b.one;
      float us = rounds * (split ? (float)ksteps / p.pieces : (float)ksteps);
      us = std::max(us, (float)N * p.K * 2 / 5.9e6f);
      if (split) us += 1.f + (2.f * p.pieces + 1.f) * p.R * N * 4 / 4.5e6f;
      us += 0.001f * blocks;                // (equal rounds: fewer blocks read fewer operands)
      // (next to equal to the model; one piece, 2047 rows, as squares / the other way, us: 4096 x 4096 107 / 110, 2048 x 8192 112 /
      // 114, but 4096 x 11008 284 / 280, 2048 x 2048 31.9 / 29.5.  From before the second shape loaded its weights itself: 122 / 125
      // and 298 / 303 in the two 4096-feature ones.  By now about even: prompts of 1026 to 2048 tokens, ten widths from 768 to
      // 4096, take 0.7 % less without this line on average, 4.1 % less at the most (4096 wide, 1600 tokens), 3.3 % more at the
      // least (2560 wide, 1200))
      if (s == 0 && N <= 4096 && p.pieces == 1) us *= 0.98f;
      if (us < best_us) {
        best_us = us;
        best = s;
        best_split = split != 0;
      }
    }
  }
  return launch_blk_gemm_as(best, best_split, p, st, part, part_floats);
}

// ---------------------------------------------------------------------------------------
// 33..64 rows of several sequences, in the decode kernels' order of additions
// ---------------------------------------------------------------------------------------
// The contract of k_gemm_bf16_wide (decode fragments in, decode epilogue out, the same bits) with the loop of the block
// GEMM: 128 features x 64 rows a work-group, weights and fragments copied into LDS once and read from there by the two waves
// that need them.  In k_gemm_bf16_wide a wave that owns few tiles pulls 8 KiB of fragments through the CU's vector memory path
// for 1..4 KiB of weights, and wider tiles do not fit the chunk sums into LDS; here the sums of a 512-wide chunk, of the chunk
// in front of it and of the pairs so far are three sets of accumulators.  A launch of few tiles gives each pair of chunks to a
// work-group of its own (SPLIT) and a second kernel adds the pairs up.
// us at 64 rows, k_gemm_bf16_wide in brackets, in a layer: 7B QKV 32.6 (39), out 16.7 (20.8), gate/up 45 (66), down 30.6 (48.5),
// unembedding 55 (80); 1B 16.7 (21.6), 12 (13.2), 22.4 (26.1), 18.8 (35.3), 31 (41).  A whole layer: 7B 191 -> 140, 1B 107 -> 84,
// 125M 67 -> 56.  What bounds it: the weights' way from memory in the large projections (gate/up: 180 MB), else the pace of one
// wave per SIMD (0.25 us a k-step) and, in split launches, the second kernel.
// A wave's NT weight tiles x CT column tiles as the MFMA leaves them (see blk_epilogue), rs: the rows' 1/rms.
template <int NT, int CT>
__device__ __forceinline__ void shared_epilogue(int role, const GemmEpi& epi, int M, int N, const f32x4 (&sums)[NT][CT], int tile0, int row0,
                                                int g, const float (&rs)[CT]) {
  const int NTILES = N >> 4;
  float acc[NT][CT][4];
#pragma unroll
  for (int ct = 0; ct < CT; ++ct)
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int i = 0; i < 4; ++i) acc[t][ct][i] = sums[t][ct][i] * rs[ct];
  if constexpr (CT % 2 == 0) {
    if (role == kRoleGateUp || role == kRoleQKV) {       // pairs at columns (j, j + 8): exchanged as in blk_epilogue
      const bool up = g >= 2;
      g &= 1;
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int ct = 0; ct < CT; ct += 2)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(acc[t][ct][i]), __float_as_uint(acc[t][ct + 1][i]), false, false);
            acc[t][ct][i] = __uint_as_float(r[0]);
            acc[t][ct + 1][i] = __uint_as_float(r[1]);
          }
      const int d = N / 3, hd = epi.hd, half = hd >> 1, hd_log = 31 - __builtin_clz(hd), part_tiles = NTILES / 3;
#pragma unroll
      for (int ct = 0; ct < CT; ct += 2) {
        const int row = row0 + (ct + (up ? 1 : 0)) * 16;
        if (row >= M) continue;
        if (role == kRoleGateUp) {
#pragma unroll
          for (int t = 0; t < NT; ++t) {
            const float (&a)[4] = acc[t][ct], (&b)[4] = acc[t][ct + 1];
            const int col = (tile0 + t) * 8 + 4 * g;
            if (tile0 + t < NTILES) {
              const float4 o = make_float4(swiglu(a[0], b[0]), swiglu(a[1], b[1]), swiglu(a[2], b[2]), swiglu(a[3], b[3]));
              *reinterpret_cast<float4*>(epi.out + (size_t)row * (N >> 1) + col) = o;
              if (epi.frag_out) store_frag4(epi.frag_out, row, col, o, nullptr);
            }
          }
          continue;
        }
        const int pos = pos_of(epi.pos, row);
        const size_t slot = (size_t)slot_of(epi.pos, row) * epi.kv_slot_stride;
        float4 cs[NT][2];
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          const int w = min(tile0 + t, NTILES - 1) * 16 % d & (hd - 1);
          const float4* src = reinterpret_cast<const float4*>(epi.rope_cs + row * 64 + (w >> 4) * 8 + 4 * g);
          cs[t][0] = src[0];
          cs[t][1] = src[1];
        }
        if (pos < 0) continue;
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          const int tile = tile0 + t;
          if (tile >= NTILES) continue;
          const float (&a)[4] = acc[t][ct], (&b)[4] = acc[t][ct + 1];
          const int part = (tile >= part_tiles) + (tile >= 2 * part_tiles), c = (tile - part * part_tiles) * 16;
          const int h = c >> hd_log, w = c & (hd - 1);
          const size_t head = slot + (size_t)h * epi.cap * hd;
          if (part == 2) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              store_kv(epi.Vc + head + v_cache_off(pos, w + 4 * g + i, hd), a[i]);
              store_kv(epi.Vc + head + v_cache_off(pos, w + 8 + 4 * g + i, hd), b[i]);
            }
            continue;
          }
          const int e = (w >> 4) * 8 + 4 * g;
          const float2 r0 = rope_rotate(a[0], b[0], make_float2(cs[t][0].x, cs[t][0].y)), r1 = rope_rotate(a[1], b[1], make_float2(cs[t][0].z, cs[t][0].w));
          const float2 r2 = rope_rotate(a[2], b[2], make_float2(cs[t][1].x, cs[t][1].y)), r3 = rope_rotate(a[3], b[3], make_float2(cs[t][1].z, cs[t][1].w));
          if (part == 0) {
            float* dst = epi.out + (size_t)row * d + h * hd + e;
            *reinterpret_cast<float4*>(dst) = make_float4(r0.x, r1.x, r2.x, r3.x);
            *reinterpret_cast<float4*>(dst + half) = make_float4(r0.y, r1.y, r2.y, r3.y);
          } else {
            store_kv4(epi.Kc + head + k_cache_off(pos, e, hd), make_float4(r0.x, r1.x, r2.x, r3.x));
            store_kv4(epi.Kc + head + k_cache_off(pos, e + half, hd), make_float4(r0.y, r1.y, r2.y, r3.y));
          }
        }
      }
      return;
    }
  }
  if (role == kRoleHead) {
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) {
        const int row = row0 + ct * 16, col = (tile0 + t) * 16 + 4 * g;
        const float (&a)[4] = acc[t][ct];
        if (row >= M || tile0 + t >= NTILES) continue;
        const bool relu = epi.act == kActRelu;
        const float4 v = relu ? make_float4(fmaxf(a[0], 0.f), fmaxf(a[1], 0.f), fmaxf(a[2], 0.f), fmaxf(a[3], 0.f)) : make_float4(a[0], a[1], a[2], a[3]);
        *reinterpret_cast<float4*>(epi.out + (size_t)row * N + col) = v;
        if (epi.frag_out) store_frag4(epi.frag_out, row, col, v, epi.frag_gain);
      }
    return;
  }
  float4 old[NT][CT];                                    // residual-writing roles
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int ct = 0; ct < CT; ++ct)
      old[t][ct] = *reinterpret_cast<const float4*>(epi.out + (size_t)min(row0 + ct * 16, M - 1) * N + min(tile0 + t, NTILES - 1) * 16 + 4 * g);
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
      const int row = row0 + ct * 16, col = (tile0 + t) * 16 + 4 * g;
      const float (&a)[4] = acc[t][ct];
      const float4 o = old[t][ct], v = make_float4(o.x + a[0], o.y + a[1], o.z + a[2], o.w + a[3]);
      const bool ok = row < M && tile0 + t < NTILES;
      if (ok) {
        *reinterpret_cast<float4*>(epi.out + (size_t)row * N + col) = v;
        if (epi.frag_out) store_frag4(epi.frag_out, row, col, v, epi.frag_gain);
      }
      float ss = sumsq4(v.x, v.y, v.z, v.w);
      ss += __shfl_xor(ss, 16);
      ss += __shfl_xor(ss, 32);
      if (ok && g == 0) epi.ssq_out[(size_t)row * NTILES + tile0 + t] = ss;
    }
}

// s_rstd[i] = 1/rms of row row0 + i, i < rows, by 4 waves: half a wave per row as in rows_rstd, the partials of four rows
// requested together
__device__ __forceinline__ void shared_rstd(RowNorm nrm, int row0, int rows, int K, float* s_rstd) {
  const int pl = threadIdx.x & 31, hw = threadIdx.x >> 5, M = rows;
  nrm.ssq_part += (size_t)row0 * nrm.ssq_n;
#pragma unroll 1
  for (int m0 = hw; m0 < M; m0 += 32) {
    float v[4][8];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float* sp = nrm.ssq_part + (size_t)min(m0 + 8 * r, M - 1) * nrm.ssq_n;
#pragma unroll
      for (int i = 0; i < 8; ++i) v[r][i] = sp[min(pl + 32 * i, nrm.ssq_n - 1)];
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int m = m0 + 8 * r;
      const float* sp = nrm.ssq_part + (size_t)min(m, M - 1) * nrm.ssq_n;
      float ss = 0.f;
#pragma unroll
      for (int i = 0; i < 8; ++i) ss += (pl + 32 * i < nrm.ssq_n) ? v[r][i] : 0.f;
      for (int p0 = pl + 256; p0 < nrm.ssq_n; p0 += 256) {
        float u[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) u[i] = (p0 + 32 * i < nrm.ssq_n) ? sp[p0 + 32 * i] : 0.f;
#pragma unroll
        for (int i = 0; i < 8; ++i) ss += u[i];
      }
      ss = half_wave_sum(ss);
      if (pl == 0 && m < M) s_rstd[m] = 1.0f / sqrtf(ss / (float)K + nrm.eps);
    }
  }
}

constexpr int kShST = 4, kShLds = kShST * 16 * 1024;
template <bool STREAM>
__device__ __forceinline__ void copy_weights_to_lds(const uint4* base, uint32_t offset, uint4* lds_base, uint32_t lane_bytes) {
  const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint4*>(base), 0, 0xFFFFFFFFu, 0x00027000);
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void*)(static_cast<uint32_t>(reinterpret_cast<uintptr_t>(lds_base))), 16,
                                           lane_bytes, offset, 0, STREAM ? 2 : 0);
}
template <bool SPLIT, bool STREAM>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2)))
void k_gemm_bf16_shared(const uint4* __restrict__ W, const uint4* __restrict__ XF, float* part, const float* __restrict__ gain, int K, int N,
                        int M, int role, const float* __restrict__ ssq_part, int ssq_n, float eps, GemmEpi epi) {
  const RowNorm nrm{gain, ssq_part, ssq_n, eps};
  const int NTILES = N >> 4;
  constexpr int NT = 4, CT = 2, ST = kShST, AT = 8, STAGE = 16 * 64, PER = 4;   // (a stage: 8 weight tiles, 2 x 4 fragments)
  extern __shared__ uint4 lds[];
  __shared__ float s_rstd[64];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int fw = wave & 1, rw = wave >> 1, j = lane & 15, g = lane >> 4;
  const int fb = blockIdx.x, ksteps = K >> 5;
  const int ks0 = SPLIT ? (int)blockIdx.z * 32 : 0, ks_end = SPLIT ? min(ksteps, ks0 + 32) : ksteps;   // (32 k-steps: a pair of chunks)
  const int full_chunks = ksteps >> 4;                   // (the last chunk may be half as long)
  uint32_t off[PER];                                     // bytes from the chunk's (weights) or the k-step's (fragments) start
#pragma unroll
  for (int q = 0; q < 2; ++q) off[q] = (uint32_t)min(fb * AT + wave + q * 4, NTILES - 1) * (kSliceUnits * 8 * 1024u);
  off[2] = wave * 1024u;
  off[3] = (uint32_t)(kFragHalfU4 * 16) + wave * 1024u;
  int rs_ = ks0;                                         // the next k-step
  const uint4* wp = W + (size_t)(ks0 >> 4) * NTILES * (kSliceUnits * 8) * 64;
  const uint4* xp = XF + (size_t)ks0 * 256 + (size_t)(ks0 >> 4) * kFragChunkPad;
  const size_t wskip = (size_t)(NTILES - 1) * (kSliceUnits * 8) * 64;
  auto request = [&](int buf) {
    const int half = __builtin_amdgcn_readfirstlane((rs_ >> 4) >= full_chunks ? 1 : 0);
    uint4* dst = lds + buf * STAGE + wave * 64;
#pragma unroll
    for (int q = 0; q < 2; ++q) copy_weights_to_lds<STREAM>(wp, off[q] >> half, dst + q * 256, lane * 16);
#pragma unroll
    for (int q = 2; q < PER; ++q) copy_to_lds_16(xp, off[q], dst + q * 256, lane * 16);
    ++rs_;
    wp += 64;
    xp += 256;
    if ((rs_ & 15) == 0) {
      wp += wskip;
      xp += kFragChunkPad;
    }
  };
  f32x4 acc[NT][CT], first[NT][CT], tot[NT][CT];
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) acc[t][ct] = tot[t][ct] = f32x4{0.f, 0.f, 0.f, 0.f};
  struct Frags {
    bf16x8 a[NT], h[CT], l[CT];
  };
  auto read = [&](Frags& f, int buf) {
    const uint4* sa = lds + buf * STAGE + fw * NT * 64 + lane;
    const uint4* sb = lds + buf * STAGE + (AT + rw * CT * 2) * 64 + lane;
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
      f.h[ct] = __builtin_bit_cast(bf16x8, sb[(ct * 2) * 64]);
      f.l[ct] = __builtin_bit_cast(bf16x8, sb[(ct * 2 + 1) * 64]);
    }
#pragma unroll
    for (int t = 0; t < NT; ++t) f.a[t] = __builtin_bit_cast(bf16x8, sa[t * 64]);
  };
  auto multiply = [&](const Frags& f) {
#pragma unroll
    for (int t = 0; t < NT; ++t) {
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) acc[t][ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f.a[t], f.h[ct], acc[t][ct], 0, 0, 0);
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) acc[t][ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f.a[t], f.l[ct], acc[t][ct], 0, 0, 0);
    }
  };
  // in front of k-step ks, where a chunk ends: the first of a pair is put aside, the second closes the pair
  auto fold = [&](int ks) {
    if ((ks & 15) || ks == ks0) return;
    const bool second = (ks & 16) == 0;
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) {
        if (second) tot[t][ct] += first[t][ct] + acc[t][ct];
        else first[t][ct] = acc[t][ct];
        acc[t][ct] = f32x4{0.f, 0.f, 0.f, 0.f};
      }
  };
  Frags f0, f1;
#pragma unroll
  for (int i = 0; i < ST; ++i) request(i);               // (a range has at least 8 k-steps)
  const bool normed = !SPLIT && nrm.gain && nrm.ssq_part;
  if (normed) shared_rstd(nrm, 0, M, K, s_rstd);            // (while the first copies are on their way; read behind barriers)
  wait_copies_and_sync<(ST - 1) * PER>();
  read(f0, 0);
  int s = ks0, rbuf = 1, wbuf = 0;                       // the loop of k_gemm_bf16_block
  auto advance = [&]() {
    rbuf = rbuf + 1 == ST ? 0 : rbuf + 1;
    wbuf = wbuf + 1 == ST ? 0 : wbuf + 1;
    ++s;
  };
  constexpr int MFMAS = 2 * NT * CT, READS = NT + 2 * CT;
  auto step = [&](const Frags& cur, Frags& next) {
    wait_copies_and_sync<(ST - 2) * PER>();
    request(wbuf);
    read(next, rbuf);
    multiply(cur);
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
    }
#pragma unroll
    for (int i = 0; i < READS; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    }
    __builtin_amdgcn_sched_group_barrier(0x008, MFMAS - PER - READS, 0);
    advance();
  };
  while (s + ST < ks_end) {                              // (an even number of k-steps, ST even: ST are left)
    fold(s);                                             // (chunks begin at even k-steps, and none among the last 7)
    step(f0, f1);
    step(f1, f0);
  }
  auto last = [&](auto self, auto I, Frags& x, Frags& y) -> void {
    constexpr int i = decltype(I)::value;
    if constexpr (i < ST - 1) {
      wait_copies_and_sync<(ST - 2 - i) * PER>();
      read(y, rbuf);
    }
    multiply(x);
    if constexpr (i < ST - 1) {
#pragma unroll
      for (int q = 0; q < READS; ++q) {
        __builtin_amdgcn_sched_group_barrier(0x008, MFMAS / READS, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      }
    }
    advance();
    if constexpr (i < ST - 1) self(self, std::integral_constant<int, i + 1>{}, y, x);
  };
  last(last, std::integral_constant<int, 0>{}, f0, f1);
  const bool paired = ((ks_end - 1) >> 4) & 1;           // the last chunk is the second of a pair
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
      if (paired) acc[t][ct] = first[t][ct] + acc[t][ct];
      tot[t][ct] += acc[t][ct];
    }
  const int tile0 = fb * AT + fw * NT;
  if constexpr (SPLIT) {                                 // the pair's sums as they lie, [pair][tile][column tile][lane]
    const int cts = (M + 15) >> 4;
    float4* dst = reinterpret_cast<float4*>(part) + ((size_t)blockIdx.z * NTILES + tile0) * cts * 64 + lane;
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int ct = 0; ct < CT; ++ct)
        if (tile0 + t < NTILES && rw * CT + ct < cts)
          dst[((size_t)t * cts + rw * CT + ct) * 64] = make_float4(acc[t][ct][0], acc[t][ct][1], acc[t][ct][2], acc[t][ct][3]);
    return;
  }
  float rs[CT];
#pragma unroll
  for (int ct = 0; ct < CT; ++ct) rs[ct] = normed ? s_rstd[min((rw * CT + ct) * 16 + j, 63)] : 1.f;
  shared_epilogue<NT, CT>(role, epi, M, N, tot, tile0, rw * CT * 16 + j, g, rs);
}

// the pairs of a SPLIT launch added up in order, then its epilogue: a wave takes CT column tiles (two where the epilogue
// exchanges between them) of a weight tile, the work-group's four waves those of adjacent tiles
template <int CT>
__global__ __launch_bounds__(256) void k_shared_reduce(const float* __restrict__ part, int pairs, int M, RowNorm nrm, int K, int N, int role,
                                                       GemmEpi epi) {
  __shared__ float s_rstd[16 * CT];
  const int lane = threadIdx.x & 63, NTILES = N >> 4, cts = (M + 15) >> 4;
  const int tile = min((int)(blockIdx.x * 4 + (threadIdx.x >> 6)), NTILES), ct0 = blockIdx.y * CT;
  const float4* src = reinterpret_cast<const float4*>(part) + (size_t)min(tile, NTILES - 1) * cts * 64 + lane;
  const size_t stride = (size_t)NTILES * cts * 64;
  f32x4 sum[1][CT];
#pragma unroll
  for (int ct = 0; ct < CT; ++ct) sum[0][ct] = f32x4{0.f, 0.f, 0.f, 0.f};
  const bool normed = nrm.gain && nrm.ssq_part;
  if (normed) shared_rstd(nrm, ct0 * 16, min(16 * CT, M - ct0 * 16), K, s_rstd);
  for (int z0 = 0; z0 < pairs; z0 += 8) {
    float4 v[8][CT];
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) v[i][ct] = src[min(z0 + i, pairs - 1) * stride + min(ct0 + ct, cts - 1) * 64];
#pragma unroll
    for (int i = 0; i < 8; ++i)
      if (z0 + i < pairs)
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) sum[0][ct] += f32x4{v[i][ct].x, v[i][ct].y, v[i][ct].z, v[i][ct].w};
  }
  __syncthreads();
  float rs[CT];
#pragma unroll
  for (int ct = 0; ct < CT; ++ct) rs[ct] = normed ? s_rstd[ct * 16 + (lane & 15)] : 1.f;
  shared_epilogue<1, CT>(role, epi, M, N, sum, tile, ct0 * 16 + (lane & 15), lane >> 4, rs);   // (tile NTILES: nothing is stored)
}

// 17..32 rows, where half of the column tiles are empty: only residual-writing projections with 16 chunks and more (17 / 32
// rows: 128 tiles x 8192 20.7 / 24.9 -> 16.8 / 17.2, 256 x 11008 32.4 / 32.7 -> 27.0 / 27.2; the other 7B projections 1..6 us
// slower).
// 33..64 rows: a launch costs about the pace of one wave per SIMD over its k range, or over one pair of chunks and then the
// second kernel, so where there are few tiles or the k is short the fragment-reading kernel is ahead.  That one fetches the
// fragments, fresh from the launch before it, once per work-group: it loses with more rows, and 1.2 .. 1.8 us more inside a
// forward than in launches by themselves, so the lines are from forwards (decoder models 512 to 2560 wide; us a layer with the
// fragment-reading kernel instead of this one, at 33 / 48 / 64 rows):
//   residual-writing, 32 x 512 -2.2 / -2.2 / -1.2, 64 x 1024 -6.6 / -6.3 / -6.2, 128 x 2048 -3.3 / -3.5 / -2.2, 48 x 2304 -3.0 / -3.0 / -1.9, 144 x
//     2304 -2.4 / -2.5 / -2.0; 48 x 3072 -0.6 / -0.4 / +1.2, 96 x 3072 -0.4 / -0.5 / +1.0, 160 x 2560 -1.5 / -1.5 / -0.3; 80 x 3584 +1.4 / +1.6 /
//     +3.2, 64 x 4096 +2.7 / +2.7 / +4.4, 128 x 4096 +2.4 / +2.4 / +4.2;
//   QKV, 96 x 512 +8.9 / +12.7 / +18.9 (one chunk: a wave has the whole k), 144 x 768 +0.2 / +1.9 / +5.2, 192 x 1024 -0.7 / +0.3 / +3.3 (39 rows
//     -0.2), 240 x 1280 -3.4 / -2.3 / +0.6, 288 x 1536 +0.9 / +2.0 / +5.7;
//   gate and up, 384 x 768 +0.9 / +3.0 / +6.0, 256 x 1024 -1.7 / -0.4 / +2.7, 352 x 1024 -0.3 / +1.2 / +4.2, 512 x 1024 -0.5 / +1.6 / +4.0, 448 x 1280
//     -3.5 / -3.1 / -0.3, 512 x 1536 -2.8 / -1.1 / +1.6, 512 x 2048 -1.9 / -0.8 / +1.7, 640 x 1280 -0.6 / +0.8 / +4.3, 704 x 2048 +3.4 / +4.2 / +7.3;
//     unembeddings of few tiles go with them (launches by themselves: 256 x 1280 9.3 / 10.2 / 12.4 us, this kernel 13.6 / 13.7 / 13.9);
//   unembedding of 32000 x 768 +5.3 / +8.2 / +12.6, x 2560 +29 / +33 / +44.
bool shared_takes(int role, int M, int NTILES, int K) {
  if (wide_cfg_is_forced(role)) return false;
  const bool resid = role == kRoleWo || role == kRoleDown, three = M <= 48;
  if (M <= 32) return M > 16 && resid && K > 15 * 512;
  if (resid) return !(NTILES <= 160 && K <= (three ? 3072 : 2304));
  if (role == kRoleQKV) return !(NTILES <= 256 && K > 768 && M <= (K <= 1024 ? 40 : 48));
  return !(three && K >= 1024 && K <= 2048 && (NTILES <= 256 || (K >= 1280 && NTILES <= 512)));
}

// whether the pairs of chunks go to different work-groups: the cheaper of the two by the model of launch_blk_gemm
bool shared_splits(int M, int NTILES, int K) {
  const int blocks = (NTILES + 7) / 8, ksteps = K / 32, pairs = (gemm_slices(K, 1) + 1) / 2;
  if (pairs == 1) return false;
  auto steps_us = [](int wgs, float ks) {
    const BlkShape& b = kBlkShapes[3];
    const int full = wgs / 512, rem = wgs % 512;
    return ks * (full * b.two + (rem > 256 ? b.one + (b.two - b.one) * (0.55f + 0.45f * (rem - 256) / 256) : rem == 0 ? 0.f : full ? 0.74f * b.one : b.one));
  };
  return steps_us(blocks * pairs, 32.f) + 1.f + (2.f * pairs + 1.f) * M * (NTILES * 16) * 4 / 4.5e6f < steps_us(blocks, (float)ksteps);
}

bool launch_gemm_shared(int role, const void* W, int N, int K, const uint4* xfrag, int M, RowNorm nrm, float* partial, const GemmEpi& epi,
                        hipStream_t st) {
  const int NTILES = N / 16, blocks = (NTILES + 7) / 8, pairs = (gemm_slices(K, 1) + 1) / 2;
  const bool paired_ct = role == kRoleQKV || role == kRoleGateUp;
  if (M > kMaxFwdRows || !shared_takes(role, M, NTILES, K)) return false;
  const uint4* Wsw = static_cast<const uint4*>(W);
#define STAIRS_SHARED(split, stream, z)                                                                                            \
  hipLaunchKernelGGL((k_gemm_bf16_shared<split, stream>), dim3(blocks, 1, z), dim3(256), kShLds, st, Wsw, xfrag, partial, nrm.gain, K, N, \
                     M, role, nrm.ssq_part, nrm.ssq_n, nrm.eps, epi)
  if (shared_splits(M, NTILES, K)) {
    if (epi.stream_weights) STAIRS_SHARED(true, true, pairs); else STAIRS_SHARED(true, false, pairs);
    const dim3 grid((NTILES + 3) / 4, paired_ct ? (M + 31) / 32 : (M + 15) / 16);
    hipLaunchKernelGGL(paired_ct ? k_shared_reduce<2> : k_shared_reduce<1>, grid, dim3(256), 0, st, partial, pairs, M, nrm, K, N, role, epi);
  } else {
    if (epi.stream_weights) STAIRS_SHARED(false, true, 1); else STAIRS_SHARED(false, false, 1);
  }
#undef STAIRS_SHARED
  return true;
}

// Attention of a row block without partial results (the rows of a 16-row tile belong to one sequence, see BlkSegs): a
// wave owns QT tiles of 16 query rows of one head and walks over the keys 0 .. its last row's position (kv_fixed > 0: over the
// keys 0 .. kv_fixed - 1 whatever the row, encoder), 64 at a time, keeping the running maximum, each lane's share of the
// running sum and the running output of its rows in registers (rescaled where the maximum grows).  Same operands and splits
// as k_attn_f16 (scores^T = K q^T with q as half high + low, out^T = V^T p^T with p as half high + low); the order of the
// additions differs from the decode kernels, which only ever see their own results, and depends on the row alone.  The output
// is left as the block fragments the output projection reads.
//   The 4 waves share the keys and values: 64 of them (32 KiB at head_dim 128) are copied into one of two LDS buffers while the
//   other is worked on.  A wave of 16 rows that loads 16 KiB for every 32 MFMAs itself asks for twice what the CU's path to
//   L2 gives, and per 32 keys the masks, lane exchanges and rescaling of every step were more vector instructions than the
//   MFMAs leave room for: now masks only at the diagonal, sums over the lanes at the end, rescaling where a maximum grew.
//   Tiles of several sequences in one work-group: the runs of tiles of one sequence one after the other.
//   Launches by themselves, before -> now, us: 32 heads of 128, 2048 rows behind nothing / behind 6144 keys 110 -> 83 / 597 -> 400
//   (1.2 PFLOP/s issued), 333 rows 13.4 -> 11.8, 777 rows of an encoder 54.3 -> 46.3; 16 heads of 64, 2048 rows behind 6144 keys
//   199 -> 135.  What bounds it then: MFMAs and the softmax's vector instructions on a SIMD, which overlap only in part.
//   Where log2 e goes: on the queries it makes them overflow their half from 45400 on instead of 65504.  Without a bias, where
//   scores of half queries and keys stay far inside a float, the exponent is one s * log2 e - m with m in units of log 2; with one,
//   whose lowest float must not become infinite, the difference from the maximum is multiplied as in the decode kernel.
//   QT = 2 where that leaves two work-groups per CU, else 1.  Row blocks come longest first; where all work-groups are
//   resident at once, the second half shortest first, so that a long one shares its CU with a short one.
template <int HD, bool BIAS, int QT>
__global__ __launch_bounds__(256, 2) void k_attn_flash(const float* __restrict__ q, const _Float16* __restrict__ Kc,
                                                    const _Float16* __restrict__ Vc, int cap, int d, size_t slot_stride,
                                                    const int2* __restrict__ rows, int R, float scale, AttnMode am,
                                                    uint4* __restrict__ frag, int RT) {
  constexpr int KK = HD / 32, ET = HD / 16, TILES = 4 * QT;
  constexpr int KP = 4 * KK, VP = 2 * ET, STAGE = (KP + VP) * 64;      // KiB pieces of 64 keys and of their values
  static_assert(KP % 4 == 0 && VP % 4 == 0, "whole pieces per wave");
  __shared__ uint4 lds[2 * STAGE];
  const int h = blockIdx.x;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int j = lane & 15, g = lane >> 4;
  int yb = gridDim.y - 1 - blockIdx.y;
  if (gridDim.x * gridDim.y <= 512 && blockIdx.y >= (gridDim.y + 1) / 2) yb = blockIdx.y - (gridDim.y + 1) / 2;
  const int r00 = yb * TILES * 16;                    // first row of the work-group
  // every tile's sequence and the last key any of its rows sees (-1: none)
  int tslot[TILES], tlast[TILES];
#pragma unroll
  for (int t4 = 0; t4 < QT; ++t4) {
    const int r = r00 + t4 * 64 + lane;
    const int2 at = r < R ? rows[r] : make_int2(-1, -1);
    int last = at.y < 0 ? -1 : am.kv_fixed > 0 ? am.kv_fixed - 1 : at.y;
#pragma unroll
    for (int off = 1; off < 16; off <<= 1) last = max(last, __shfl_xor(last, off));
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      tslot[t4 * 4 + i] = __builtin_amdgcn_readlane(at.x, i * 16);
      tlast[t4 * 4 + i] = __builtin_amdgcn_readlane(last, i * 16);
    }
  }
  int pos[QT], seen[QT], all_see[QT];                 // the lane's row; keys up to all_see are seen by the tile's 16 rows
  f16x8 qh[QT][KK], ql[QT][KK];
#pragma unroll
  for (int t = 0; t < QT; ++t) {
    const int row = r00 + (wave * QT + t) * 16 + j;
    pos[t] = row < R ? rows[row].y : -1;
    const bool ok = pos[t] >= 0;
    seen[t] = !ok ? -1 : am.kv_fixed > 0 ? am.kv_fixed - 1 : pos[t];
    int m = seen[t];
#pragma unroll
    for (int off = 1; off < 16; off <<= 1) m = min(m, __shfl_xor(m, off));
    all_see[t] = __builtin_amdgcn_readfirstlane(m);
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      float4 a = make_float4(0.f, 0.f, 0.f, 0.f), b = a;
      if (ok) {
        const float4* qp = reinterpret_cast<const float4*>(q + (size_t)row * d + h * HD + kk * 32 + g * 8);
        a = qp[0];
        b = qp[1];
      }
      const float v[8] = {a.x * scale, a.y * scale, a.z * scale, a.w * scale, b.x * scale, b.y * scale, b.z * scale, b.w * scale};
      split_half8(v, qh[t][kk], ql[t][kk]);
    }
  }
  f32x4 oacc[QT][ET];
  constexpr float kLog2e = 1.44269504088896340736f;
  float m_run[QT], l_run[QT];                         // (the maximum times log2 e but with a bias, see above)
#pragma unroll
  for (int t = 0; t < QT; ++t) {
#pragma unroll
    for (int et = 0; et < ET; ++et) oacc[t][et] = f32x4{0.f, 0.f, 0.f, 0.f};
    m_run[t] = -INFINITY;
    l_run[t] = 0.f;
  }
  const float* brow = BIAS ? am.bias + (size_t)h * am.bias_ld + am.bias_zero : nullptr;   // bias by key position - query position

  // 64 keys from LDS; tiles that see none of them (sees[t] < kb) add exactly nothing
  auto step = [&](int kb, const uint4* buf, const int (&sees)[QT], const int (&all)[QT]) {
    f32x4 sacc[QT][4];
#pragma unroll
    for (int t = 0; t < QT; ++t)
#pragma unroll
      for (int i = 0; i < 4; ++i) sacc[t][i] = f32x4{0.f, 0.f, 0.f, 0.f};
    // (reads run ahead of the MFMAs that need them: a k-step of keys, four pieces of values)
    f16x8 a[2][4], va[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) a[0][i] = __builtin_bit_cast(f16x8, buf[i * KK * 64 + lane]);
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (kk + 1 < KK) a[(kk + 1) & 1][i] = __builtin_bit_cast(f16x8, buf[(i * KK + kk + 1) * 64 + lane]);
        else va[i] = __builtin_bit_cast(f16x8, buf[(KP + i) * 64 + lane]);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int t = 0; t < QT; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) sacc[t][i] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[kk & 1][i], qh[t][kk], sacc[t][i], 0, 0, 0);
#pragma unroll
      for (int t = 0; t < QT; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) sacc[t][i] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[kk & 1][i], ql[t][kk], sacc[t][i], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
    f16x8 ph[QT][2], pl[QT][2];
#pragma unroll
    for (int t = 0; t < QT; ++t) {
      if (BIAS) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const int key = kb + i * 16 + g * 4 + v;
            if (key <= sees[t]) sacc[t][i][v] += brow[key - pos[t]];
          }
      }
      if (all[t] < kb + 63) {                          // (uniform: some row does not see some key)
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int v = 0; v < 4; ++v) sacc[t][i][v] = kb + i * 16 + g * 4 + v <= sees[t] ? sacc[t][i][v] : -INFINITY;
      }
      float mx = fmaxf(fmaxf(sacc[t][0][0], sacc[t][0][1]), fmaxf(sacc[t][0][2], sacc[t][0][3]));
#pragma unroll
      for (int i = 1; i < 4; ++i) mx = fmaxf(mx, fmaxf(fmaxf(sacc[t][i][0], sacc[t][i][1]), fmaxf(sacc[t][i][2], sacc[t][i][3])));
      auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
      mx = fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
      sw = __builtin_amdgcn_permlane16_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
      mx = fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
      if (!BIAS) mx *= kLog2e;
      if (__any(mx > m_run[t])) {
        const float m_new = fmaxf(m_run[t], mx);
        const float alpha = m_run[t] == -INFINITY ? 0.f : BIAS ? exp_fast(m_run[t] - m_new) : __builtin_amdgcn_exp2f(m_run[t] - m_new);
        l_run[t] *= alpha;
#pragma unroll
        for (int et = 0; et < ET; ++et) {
          oacc[t][et][0] *= alpha; oacc[t][et][1] *= alpha; oacc[t][et][2] *= alpha; oacc[t][et][3] *= alpha;
        }
        m_run[t] = m_new;
      }
      const float m = m_run[t] == -INFINITY ? 0.f : m_run[t];
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        float pv[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const float s = sacc[t][2 * b + (i >> 2)][i & 3];
          pv[i] = BIAS ? exp_fast(s - m) : __builtin_amdgcn_exp2f(fmaf(s, kLog2e, -m));
        }
        l_run[t] += ((pv[0] + pv[1]) + (pv[2] + pv[3])) + ((pv[4] + pv[5]) + (pv[6] + pv[7]));
        split_half8(pv, ph[t][b], pl[t][b]);
      }
    }
#pragma unroll
    for (int p0 = 0; p0 < VP; p0 += 2) {               // (two pieces: no product waits for the one in front of it)
#pragma unroll
      for (int t = 0; t < QT; ++t)
#pragma unroll
        for (int p = p0; p < p0 + 2; ++p)
          oacc[t][p % ET] = __builtin_amdgcn_mfma_f32_16x16x32_f16(va[p & 3], ph[t][p / ET], oacc[t][p % ET], 0, 0, 0);
#pragma unroll
      for (int t = 0; t < QT; ++t)
#pragma unroll
        for (int p = p0; p < p0 + 2; ++p)
          oacc[t][p % ET] = __builtin_amdgcn_mfma_f32_16x16x32_f16(va[p & 3], pl[t][p / ET], oacc[t][p % ET], 0, 0, 0);
      if (p0 + 4 < VP) {
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int p = p0 + 4; p < p0 + 6; ++p) va[p & 3] = __builtin_bit_cast(f16x8, buf[(KP + p) * 64 + lane]);
      }
    }
  };

  for (int t0 = 0; t0 < TILES;) {                     // runs of tiles of one sequence
    const int slot = tslot[t0];
    int t1 = t0, last = -1;
#pragma unroll
    for (int t = 0; t < TILES; ++t)
      if (t == t1 && tslot[t] == slot) {
        last = max(last, tlast[t]);
        ++t1;
      }
    if (last >= 0) {                                  // (rows past the block's last and sequences of padding see nothing)
      const uint4* Kh = reinterpret_cast<const uint4*>(Kc + slot * slot_stride + (size_t)h * cap * HD);
      const uint4* Vh = reinterpret_cast<const uint4*>(Vc + slot * slot_stride + (size_t)h * cap * HD);
      // (cap is whole blocks of 32 keys: where the second half of 64 lies past it, the first half comes twice, unseen)
      auto request = [&](int kb, uint4* buf) {
        const int past = __builtin_amdgcn_readfirstlane(kb + 32 >= cap ? 1 : 0);
#pragma unroll
        for (int i = 0; i < KP / 4; ++i) {
          const int p = wave + 4 * i, src = past && p >= KP / 2 ? p - KP / 2 : p;
          copy_to_lds_16(Kh, (uint32_t)((kb >> 4) * KK + src) * 1024u, buf + p * 64, lane * 16);
        }
#pragma unroll
        for (int i = 0; i < VP / 4; ++i) {
          const int p = wave + 4 * i, src = past && p >= VP / 2 ? p - VP / 2 : p;
          copy_to_lds_16(Vh, (uint32_t)((kb >> 5) * ET + src) * 1024u, buf + (KP + p) * 64, lane * 16);
        }
      };
      int sees[QT], all[QT], mine = -1;
#pragma unroll
      for (int t = 0; t < QT; ++t) {
        const bool in = wave * QT + t >= t0 && wave * QT + t < t1;
        sees[t] = in ? seen[t] : -1;
        all[t] = in ? all_see[t] : -1;
#pragma unroll
        for (int u = 0; u < TILES; ++u)
          if (u == wave * QT + t && in) mine = max(mine, tlast[u]);
      }
      __syncthreads();                                // (the run before this one has been read)
      request(0, lds);
      int cur = 0;
      for (int kb = 0; kb <= last; kb += 64, cur ^= 1) {
        wait_copies_and_sync<0>();                    // these 64 keys are there, the 64 before them have been read
        if (kb + 64 <= last) request(kb + 64, lds + (cur ^ 1) * STAGE);
        if (kb <= mine) step(kb, lds + cur * STAGE, sees, all);
      }
    }
    t0 = t1;
  }
#pragma unroll
  for (int t = 0; t < QT; ++t) {
    const int row = r00 + (wave * QT + t) * 16 + j;
    float l = l_run[t];
    l += __shfl_xor(l, 16);
    l += __shfl_xor(l, 32);
    if (row < R) {
      const float inv = pos[t] >= 0 ? 1.0f / l : 0.f;  // (a padding row sees no key: zeros)
#pragma unroll
      for (int et = 0; et < ET; ++et)
        blk_store_frag4(frag, RT, row, h * HD + et * 16 + g * 4,
                        make_float4(oacc[t][et][0] * inv, oacc[t][et][1] * inv, oacc[t][et][2] * inv, oacc[t][et][3] * inv));
    }
  }
}

void launch_attention_flash(const float* q, const void* Kc, const void* Vc, int cap, int d, int H, size_t slot_stride, const int2* rows,
                            int R, uint4* frag, hipStream_t st, const AttnMode& am) {
  const int hd = d / H;
  const float scale = am.scale > 0.f ? am.scale : 1.0f / sqrtf((float)hd);
  const _Float16* K = static_cast<const _Float16*>(Kc);
  const _Float16* V = static_cast<const _Float16*>(Vc);
  const int qt = H * ((R + 127) / 128) >= 512 ? 2 : 1;
  dim3 grid(H, (R + 64 * qt - 1) / (64 * qt));
#define STAIRS_FLASH(hdv, bias)                                                                                                    \
  hipLaunchKernelGGL((qt == 2 ? k_attn_flash<hdv, bias, 2> : k_attn_flash<hdv, bias, 1>), grid, dim3(256), 0, st, q, K, V, cap, d, \
                     slot_stride, rows, R, scale, am, frag, pf_col_tiles(R))
  if (hd == 128) {
    if (am.bias) STAIRS_FLASH(128, true); else STAIRS_FLASH(128, false);
  } else {
    if (am.bias) STAIRS_FLASH(64, true); else STAIRS_FLASH(64, false);
  }
#undef STAIRS_FLASH
}

hipError_t configure_block_kernels() {
  hipError_t e = hipSuccess;
  auto optin = [&](const void* fn, size_t bytes) {
    const hipError_t r = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
    if (r != hipSuccess) e = r;
  };
#define STAIRS_OPTIN_BLK(WF, WR, CT, ST)                                                        \
  optin((const void*)k_gemm_bf16_block<WF, WR, CT, ST, true>, blk_lds_bytes(WF, WR, CT, ST));   \
  optin((const void*)k_gemm_bf16_block<WF, WR, CT, ST, false>, blk_lds_bytes(WF, WR, CT, ST))
  STAIRS_OPTIN_BLK(2, 2, 4, 3);
  STAIRS_OPTIN_BLK(4, 1, 4, 3);
  STAIRS_OPTIN_BLK(2, 2, 2, 4);
#undef STAIRS_OPTIN_BLK
  optin((const void*)k_gemm_bf16_shared<true, true>, kShLds);
  optin((const void*)k_gemm_bf16_shared<true, false>, kShLds);
  optin((const void*)k_gemm_bf16_shared<false, true>, kShLds);
  optin((const void*)k_gemm_bf16_shared<false, false>, kShLds);
  return e;
}

}  // namespace stairs
