// Launch wrappers of the gfx950 kernels behind the stairs C ABI (see include/stairs.h).
// Host code only sees these functions; every pointer is a device pointer unless named h_*.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>

namespace stairs {

constexpr int kMaxRows = 32;        // rows (new tokens) of ONE sequence a forward of the decode kernels can take
constexpr int kMaxFwdRows = 64;     // rows of all sequences together a forward of the decode kernels can take (bf16)
constexpr int kMaxBlockRows = 256;  // rows one forward of several sequences can take on the block kernels (beyond kMaxRows)
constexpr int kAttnChunk = 128;     // keys per attention work-group of the fp32-cache kernels and the unit callers count chunks in; boundaries are absolute positions
constexpr int kAttnChunkH = 256;    // keys per attention work-group of the half-cache kernels (a wave owns 64)
constexpr int kAttnFusedMaxChunks = 24;   // more chunks per head than this: the chunk merge runs as a second kernel
constexpr int kSsqGroup = 16;       // residual columns per sum-of-squares partial, bf16 models (= one weight tile of the residual-writing GEMMs)
constexpr int kUnitK = 256;         // k extent of one weight "unit" (8 MFMA k-steps of 32)
constexpr int kSliceUnits = 2;      // units per split-K slice (512 k)
constexpr int kSpwRows = 9;         // 9..16 rows: a split-K work-group takes two k chunks (see launch_gemm)
// most LDS the small-M GEMM (whole X block in LDS) may take per work-group: projections with many weight tiles keep
// two work-groups per CU, the residual-writing ones (one work-group per CU) take most of the CU's LDS
constexpr size_t kRowsPathMaxLds = 68 * 1024;
constexpr size_t kRowsPathMaxLdsWide = 150 * 1024;
constexpr size_t kWideMaxLds = 150 * 1024;      // chunk sums of k_gemm_bf16_wide: chunks * rows * 16 NT * 4 bytes
// one column tile, one weight tile and one k chunk per wave (small models at 5..16 rows): the whole chunk in flight, one
// round trip to memory instead of two or three (7.2 -> 6.8 us a launch at 125M and at the large encoder-decoder shape).
// Up to 4 chunks: with more the weights' way from memory is the bound, and 16 k-steps in flight a wave only take registers
// (8 chunks x 256 tiles, 8 / 16 rows: 10.9 us, with 8 in flight 10.1 / 10.2; 6 x 48: 6.8 / 6.9 and 6.6).
constexpr int kWideDepthChunk = 16, kWideWholeChunkMax = 4;
inline bool wide_whole_chunk(int M, int nchunks, int nw) { return M <= 16 && nchunks <= nw && nchunks <= kWideWholeChunkMax; }
constexpr int kWideDepth8 = 2, kWideDepth6 = 2, kWideDepth4 = 3, kWideDepth3 = 4, kWideDepth2 = 5, kWideDepth1 = 8;   // k-steps in flight per wave at 4 / 2 / 1 tiles per wave
constexpr size_t kRowsPathSmallMatrix = 16u << 20;   // residual-writing projections with fewer tiles than CUs: up to this many bytes

// Where the rows of a forward sit.  One sequence (rps == 0): row r is at position *base + offset + r (base lives
// in device memory so that the same launch sequence can be replayed without the host knowing the sequence length).
// Several sequences ("slots", rps > 0): the forward holds rps consecutive rows per slot; slot s = r / rps keeps its
// state in base[s * kSlotState + ...] = {L, n of the last iteration, 0, active}; row r is at position
// L_s + offset + r % rps, or nowhere (negative) when the slot is not active.
constexpr int kSlotState = 4;
struct PosRef {
  const int* base;
  int offset;
  int rps;
};
#ifdef __HIPCC__
__device__ __forceinline__ int slot_of(const PosRef& p, int r) { return p.rps ? r / p.rps : 0; }
__device__ __forceinline__ int pos_of(const PosRef& p, int r) {
  if (!p.rps) return *p.base + p.offset + r;
  const int s = r / p.rps;
  const int* st = p.base + s * kSlotState;
  return st[3] ? st[0] + p.offset + (r - s * p.rps) : -(1 << 24);
}
#endif

// Row normalisation folded into a GEMM: the input is x[m][k] * gain[k] * rstd[m] with
// rstd[m] = 1/sqrt(sum_p ssq_part[m*ssq_n + p] / K + eps).  gain == nullptr: no scaling at all.
// (bf16 kernels: the gain goes into the activation fragments, rstd[m] multiplies the row's finished sums; the
// split-K kernel forms it in the work-group that finishes a column group, the small-M kernel in every work-group.)
struct RowNorm {
  const float* gain;
  const float* ssq_part;
  int ssq_n;
  float eps;
};

inline int ssq_groups(int d) { return (d + kSsqGroup - 1) / kSsqGroup; }
inline int gemm_slices(int K, int dtype_bf16) {
  if (!dtype_bf16) return 1;
  int units = K / kUnitK;
  return (units + kSliceUnits - 1) / kSliceUnits;
}

// ---- weights --------------------------------------------------------------------------
// bf16 [N, K] row-major -> MFMA-operand tiles: tile (nt, kt) covers rows nt*16.., k kt*32.., is 1 KiB;
// inside it lane l = r + 16*g holds W[nt*16+r][kt*32+g*8..+8].  Tiles are stored slice-major:
// [split-K slice of 16 k-steps][nt][k-step inside the slice], so that one work-group of the GEMM
// (one slice, 4*NT adjacent row tiles) reads one contiguous run.
// perm: order of the rows (= output columns of the GEMM): kPermGateUp (p0 = f) puts the gate and up rows of 8
// features into one tile, kPermQKV (p0 = d, p1 = head_dim) the two halves of 8 rotation pairs; the epilogues undo it.
enum { kPermNone = 0, kPermGateUp = 1, kPermQKV = 2 };
void launch_swizzle_bf16(const uint16_t* W, uint4* Wsw, int N, int K, int perm, int p0, int p1, hipStream_t st);

enum { kRoleQKV = 0, kRoleWo = 1, kRoleGateUp = 2, kRoleDown = 3, kRoleHead = 4 };   // which projection a GEMM launch is

// What the GEMM does with its result (by role):
//   QKV    : columns [0,d) q, [d,2d) k, [2d,3d) v: rotate q and k by the row's position, out = q as
//            float [M, d], append k and v to the layer's cache at that position
//   Wo/Down: out = x [M, N] += result; ssq_out[m][g] = sum over column group g of x^2
//   GateUp : out = h [M, N/2] = silu(gate) * up
//   Head   : out = logits [M, N]; with act == kActRelu out = max(result, 0) (the first matrix of an ungated
//            feed-forward block)
enum { kActNone = 0, kActRelu = 1 };
struct GemmEpi {
  int* counters;            // bf16 path: one int per column group, zero between launches
  float* out;
  float* ssq_out;
  const float2* rope_cs;    // [M][64] (cos, sin)
  PosRef pos;
  _Float16* Kc;             // bf16 models: half caches of this layer, tiled layout
  _Float16* Vc;
  float* Kc32;              // fp32 models: float caches of this layer, [H][cap][hd]
  float* Vc32;
  int cap, H, hd;
  size_t kv_slot_stride;    // elements between the caches of consecutive slots (several sequences), else unused
  // k_gemm_bf16_wide, residual-writing and gate/up roles: where the fragments of the result go for the next
  // projection (see frag_bytes), with frag_gain[k] folded in; nullptr: none
  uint4* frag_out;
  const float* frag_gain;
  int act;                  // Head role only: kActNone / kActRelu
  int stream_weights;       // bf16: read the weights with the streaming hint (models far larger than the memory-side cache)
};

// ---- skinny GEMM + epilogue ---------------------------------------------------------------
// bf16: W is swizzled, split-K slices of 512 k, epilogue fused; fp32: W row-major,
// epilogue fused, the row norm gathered from X itself (nrm.ssq_part unused).  partial (bf16): scratch of gemm_slices() * M * N
// floats (M > 16: see launch_gemm_shared as well).
// xfrag (bf16, M > 4): the fragments of X with nrm.gain folded in, left by X's producer or by launch_split_frag; with
// them the launch takes the hand-off-free kernel k_gemm_bf16_wide (no partial sums), without them the split-K kernel.
void launch_gemm(int role, int dtype_bf16, const void* W, int N, int K, const float* X, int ldx, int M,
                 RowNorm nrm, float* partial, const GemmEpi& epi, hipStream_t st, const uint4* xfrag = nullptr);
// The Head role, which where rows_path_lds takes it also leaves cand (nullptr: not): [M][N / 16] (largest value, its column) of
// the outputs of each 16 columns; a NaN counts as the lowest.
void launch_unembed(int dtype_bf16, const void* W, int N, int K, const float* X, int M, RowNorm nrm, float* partial, const GemmEpi& epi,
                    hipStream_t st, const uint4* xfrag, float2* cand);

// dynamic LDS of the kernel that keeps the whole activation block of up to 7 rows in LDS; 0: the projection does not take it
size_t rows_path_lds(int role, int M, int N, int K);

// launch shape of the GEMM that reads fragments (5..64 rows): weight tiles per wave, waves; nt == 0: the split-K kernel
struct WideCfg { int nt, nw; };
WideCfg wide_cfg(int role, int M, int NTILES, int K);
bool wide_cfg_is_forced(int role);            // by STAIRS_WIDE_CFG

// launch_gemm for 17..64 rows on the kernel that shares the activation fragments of a work-group through LDS; false: another
// kernel is faster for the shape, nothing launched.  partial: room for (gemm_slices(K, 1) + 1) / 2 times M rounded up to 16
// times N floats.  shared_takes: the rule; shared_splits: whether it is two kernels with partial sums in between.
bool shared_takes(int role, int M, int NTILES, int K);
bool shared_splits(int M, int NTILES, int K);
bool launch_gemm_shared(int role, const void* W, int N, int K, const uint4* xfrag, int M, RowNorm nrm, float* partial, const GemmEpi& epi,
                        hipStream_t st);

// Y [M <= 32, N] = X [M, K] . W^T with W [N, K] row-major bf16 read as it is, one kernel (M > 4: two), the bits launch_gemm
// gives for the laid-out matrix; frag: frag_bytes(K) of scratch.  false: the shape takes the split-K kernel, nothing done.
bool launch_gemm_rowmajor(const uint16_t* W, int N, int K, const float* X, int M, float* Y, uint4* frag, hipStream_t st);

// Activation fragments of a [M <= 32, K] block: K / 32 k-steps x 2 column tiles x (high, low) x 1 KiB
// (+ kFragChunkPad uint4 after every 16 k-steps: the k chunks the waves of a work-group read at the same time then do
// not sit a power of two apart)
constexpr int kFragChunkPad = 272;
// rows 32..63 of a forward have a second fragment block of the same layout kFragHalfU4 uint4 after the first
constexpr size_t kFragHalfU4 = (4u << 20) / 16;
inline size_t frag_bytes(int K) { return ((size_t)(K / 32) * 256 + (size_t)(K / 512 + 1) * kFragChunkPad) * 16; }   // one block of 32 rows
inline size_t frag_alloc_bytes(int K) { return kFragHalfU4 * 16 + frag_bytes(K); }                                      // both blocks
// frag = fragments of x [M, K] (row stride ldx) times gain (nullptr: none)
// whether launch_gemm takes M > kMaxRows rows of a bf16 projection with k = K (the chunk sums of all rows fit the LDS of
// k_gemm_bf16_wide)
bool gemm_takes_rows(int M, int K);
void launch_split_frag(const float* X, int ldx, int M, int K, const float* gain, uint4* frag, hipStream_t st);

// The next bf16 launch_gemm records `start` at the beginning and `stop` at the end of its kernel (the events of the
// launch itself, not records around it in the stream); one launch only.  Measurement aid.
void set_gemm_launch_events(hipEvent_t start, hipEvent_t stop);

// ---- small kernels ----------------------------------------------------------------------
// x[m][:] = emb[tokens[pos+m]][:] (row of zeros if pos+m lies outside [0, tok_cap) or the id found there outside
// [0, vocab)), plus sum-of-squares partials; the same launch copies the M positions' rotation entries from tab (tab_len
// positions; nullptr: the identity rotation (1, 0)) to cs.  tok_cap = ints one sequence's token array holds.
void launch_embed(const void* emb, int emb_bf16, const int* tokens, int tok_slot_stride, int tok_cap, int vocab, PosRef pos,
                  int M, int d, float* x, float* ssq_part, int hd, const float2* tab, int tab_len, float2* cs, hipStream_t st,
                  uint4* frag = nullptr, const float* frag_gain = nullptr);   // bf16: also the fragments of x * frag_gain
// Where the next forward of one sequence finds its embeddings (launch_embed's outputs, without fragments): a launch that decides
// a token can leave them itself, the token's row alone or behind that of the token in front of it.  emb == nullptr: it does not.
constexpr int kMaxNextRows = 2;
struct NextEmbed {
  const void* emb;
  int bf16, tok_cap, vocab, d, hd;
  float* x;
  float* ssq_part;
  const float2* tab;
  int tab_len;
  float2* cs;
};
// tab[p][i] = (cos, sin)(p * theta^(-2i/hd)), p < len, angle formed in double: [len][64], once per model
void launch_rope_table(int len, int hd, float theta, float2* tab, hipStream_t st);
// cs[m] = tab's entries of the positions of rows 0 .. M-1
void launch_rope_rows(PosRef pos, int M, int hd, const float2* tab, int tab_len, float2* cs, hipStream_t st);
// split-KV attention of M query rows at positions pos..pos+M-1 against keys 0..pos+M-1
// (kv_half: half caches in the tiled layout; else float caches [H][cap][hd]); counters: one int per (slot, head).
// Several sequences (pos.rps > 0, half caches only): M = pos.rps rows per slot, nslots slots, caches kv_slot_stride
// elements apart.
// am (half caches only): score scale, additive bias by relative position, fixed key set (see AttnMode).
struct AttnMode {
  float scale;        // multiplies q; <= 0: 1/sqrt(head_dim)
  const float* bias;  // nullptr, or [H][bias_ld]: score += bias[h][key position - query position + bias_zero]
  int bias_ld, bias_zero;
  int kv_fixed;       // > 0: no causal mask, every row sees the keys 0 .. kv_fixed-1 (nchunk_launch must cover them)
  uint4* frag_out;    // half caches: also leave the output's activation fragments here (nullptr: none)
  int frag_rt;        // 0: fragments in the decode kernels' layout; > 0: block fragments of that many column tiles
};
void launch_attention(const float* q_rot, const void* Kc, const void* Vc, int kv_half, int cap, int d, int H, int M,
                      PosRef pos, int nslots, size_t kv_slot_stride, int nchunk_launch, int nchunk_cap, float* part_o,
                      float* part_ml, int* counters, float* out, hipStream_t st,
                      const AttnMode& am = AttnMode{0.f, nullptr, 0, 0, 0, nullptr, 0});
// keys of a launch over `units` 128-key units that its work-groups request before they know the rows' position (half
// caches, causal; a fixed key set is known to the launch)
int attn_early_keys(int units, int nslots);
// query rows per work-group of a launch over `units` 128-key chunks (fp32 caches)
int attn_f32_rows(int units, int H, int M);
// out[o(r)] = argmax_v logits[row0 + r * row_stride][v], ties -> lowest v, r < nrows.  One sequence:
// o(r) = *out_pos.base + out_pos.offset + r (base == nullptr: r).  Several: o(r) = s * out_slot_stride + position of
// out_pos for row r, nothing written for a slot that is not active.  next (one sequence, one row): also the embedding of the
// forward whose only row is that token at that position.
void launch_argmax(const float* logits, int ld, int V, int nrows, int row0, int row_stride, int* out, PosRef out_pos,
                   int out_slot_stride, hipStream_t st, const NextEmbed& next = NextEmbed{});
// The same and what follows it in one launch, for M <= 8 rows of one sequence (where ..._takes).  src: the unembedding's candidates
// (cand: launch_unembed's, V / 16 pairs a row), else the rows of V logits themselves.
//   launch_decide       : M = 1, tokens[out_pos] = the choice; next: its embedding
//   launch_decide_accept: the choices of k + 1 stair rows (to tgt as well), launch_accept, and the embeddings of the last
//                         next_rows (1 .. kMaxNextRows) tokens then, as rows 0 .. of a forward
// host (at nullptr: none): {L, n} also go to at[0 .. 1] or at[2 .. 3], memory of the host, as *turn, which counts up, is even or odd
struct HostResult {
  int* at;
  int* turn;
};
bool decide_takes(bool cand, int V);
bool decide_accept_takes(bool cand, int M, int V);
void launch_decide(const float* src, bool cand, int V, int M, int* tokens, PosRef out_pos, hipStream_t st, const NextEmbed& next);
void launch_decide_accept(const float* src, bool cand, int V, int k, int* tokens, int* tgt, int* state, hipStream_t st, const NextEmbed& next,
                          int next_rows, const HostResult& host);
// stairs validation on device, one block per slot s (one sequence: nslots = 1, strides unused): state = {L, n, 0,
// active}.  n = longest run with tokens[L+i] == tgt[i]; tokens[L+n] = tgt[n]; state[0] = L+n+1; state[1] = n.
// tokens of slot s start at s * tok_slot_stride, its tgt at s * (k+1), its state at s * kSlotState.  limits (nullptr: none): the
// slot stops being active where its sequence reaches limits[s] tokens.
void launch_accept(int* tokens, const int* tgt, int k, int* state, int nslots, int tok_slot_stride, const int* limits, hipStream_t st);

// ---- sampling variant -------------------------------------------------------------------------------------
// Device-resident parameters of a sampled generation (so that captured launches stay valid across seeds)
struct SampleParams {
  float inv_temp;      // 1 / temperature
  uint64_t key;        // key of the counter-based generator (from the seed)
};
// Scratch of a draw spread over several blocks: one (score, index) per block and the ticket of the last arrival
// (zero at allocation, zero again after every launch)
constexpr int kSampleBlocksMax = 512;
struct SampleWs {
  int ticket;
  int pad;
  unsigned long long score[kSampleBlocksMax];
  int idx[kSampleBlocksMax];
};
// lse[r][part] = (maximum, sum of exponentials relative to it) of a share of row_r * inv_temp, for the n_a rows of a followed by
// the n_b rows of b (row stride ld)
constexpr int kLseParts = 8;
void launch_row_lse(const float* a, int n_a, const float* b, int n_b, int ld, int V, const SampleParams* sp, float* lse,
                    hipStream_t st);
// tokens[o] = one draw from softmax(logits / T) by Gumbel-max with the random numbers of (o, stream), o = out_pos; next: as for
// launch_argmax
void launch_sample(const float* logits, int V, const SampleParams* sp, int stream, int* tokens, PosRef out_pos,
                   SampleWs* ws, hipStream_t st, const NextEmbed& next = NextEmbed{});
// keep / replace walk over a sampled stair batch of one sequence (see k_accept_sampled); lse = launch_row_lse over
// the k+1 rows of tl followed by the k rows of dl
void launch_accept_sampled(int* tokens, const float* tl, const float* dl, int ld, int V, int k, const float* lse,
                           const SampleParams* sp, int* state, int* emitted, SampleWs* ws, hipStream_t st, const NextEmbed& next = NextEmbed{},
                           int next_rows = 1, const HostResult& host = HostResult{});

// ---- row blocks (bf16 models): prompts, forwards of many sequences, encoders -------------------------------------
// The projections of a block of up to kPfRows rows run on the MFMA-bound kernel k_gemm_bf16_block: the weights in the
// decode kernels' layout, the activations as fragments (bf16 high + low parts in operand order).  Every producer of an
// activation writes the next projection's fragments itself, with the gain of the norm in between folded in; the rows'
// 1/rms multiplies the finished sums (partial sums of squares travel beside x).
constexpr int kPfRows = 2048;
constexpr int kBlkRows = 128;       // fragment buffers are laid out for whole groups of this many rows
constexpr int kBlkSegRows = 16;     // a sequence's rows start at a multiple of this (one attention tile, one column tile)
constexpr int kBlkSsqCols = 32;     // columns of x per sum-of-squares partial
constexpr int kBlkPiecedRows = 1024;   // rows of sequences up to this long are summed in k pieces (launch_blk_gemm)
inline int pf_col_tiles(int R) { return (R + kBlkRows - 1) / kBlkRows * (kBlkRows / 16); }
// bytes of the fragments of a [R, K] activation block
inline size_t pf_frag_bytes(int R, int K) { return (size_t)(K / 32) * pf_col_tiles(R) * 2 * 1024; }

// Where a block's rows sit: segment s is len[s] consecutive positions from pos0[s] on of sequence slot slot[s], at rows
// row0[s] .. (row0[0] = 0, row0 ascending multiples of kBlkSegRows); rows behind a segment's last are padding.
constexpr int kBlkMaxSegs = 128;
struct BlkSegs {
  int n;
  int row0[kBlkMaxSegs], len[kBlkMaxSegs], slot[kBlkMaxSegs], pos0[kBlkMaxSegs];
};
// rows[r] = (slot, position; < 0 for padding), cs[r] = tab's entries of the position (tab as for launch_embed)
void launch_blk_rows(const BlkSegs& segs, int R, int hd, const float2* tab, int tab_len, int2* rows, float2* cs, hipStream_t st);
void launch_blk_rows_pos(PosRef pos, int R, int hd, const float2* tab, int tab_len, int2* rows, float2* cs, hipStream_t st);
// x = the rows' embeddings, frag = fragments of x * gain, ssq [R][d / kBlkSsqCols]
void launch_blk_embed(const uint16_t* emb, const int* tokens, int tok_stride, int tok_cap, int vocab, const int2* rows, int R, int d,
                      float* x, const float* gain, uint4* frag, float* ssq, hipStream_t st);

// What a block projection does with its sums (after the rows' 1/rms, when ssq is given):
//   Plain : out[row][n] = sum (W without row permutation)
//   Resid : out = x [R, ldo] += sum; frag_out (optional) = fragments of x * gain; ssq_out (optional) = its partials
//   Swiglu: W = gate/up tiles; frag_out = fragments of silu(gate) * up
//   QKV   : W = q | k | v tiles of da columns each; out = rotated q [R, da]; k, v -> the tiled half caches at rows[r]
//   Relu  : frag_out = fragments of max(sum, 0)
enum { kBlkPlain = 0, kBlkResid, kBlkSwiglu, kBlkQKV, kBlkRelu };
struct BlkGemm {
  const uint4* W;              // operand tiles of [N, K]
  int NTILES, tile_first, K;   // N / 16; output tiles before tile_first are left out
  const uint4* XF;             // fragments of the input [R, K]
  int RT, R;                   // column tiles the fragment buffers (XF, frag_out) are laid out for; rows
  int kind;
  float* out;
  int ldo;
  const float* ssq;            // partials of the input's rows [R][ssq_n], or nullptr: no normalisation
  int ssq_n;
  float eps;
  uint4* frag_out;
  const float* gain;
  float* ssq_out;
  const int2* rows;
  const float2* cs;
  _Float16 *Kc, *Vc;
  size_t slot_stride;          // elements between the caches of consecutive slots
  int cap, hd, da;
  int pieces;                  // set by launch_blk_gemm
};
// pieced: the k range is summed in a number of pieces that depends on K alone (rows of sequences of at most
// kBlkPiecedRows rows: their results are the same bits in whatever block they are computed), else in one.
// part (part_floats floats): scratch that lets different work-groups take the pieces.
// hipErrorInvalidValue, nothing launched: a shape the kernel does not take (launch_blk_gemm_as).
hipError_t launch_blk_gemm(BlkGemm p, bool pieced, hipStream_t st, float* part, size_t part_floats);
// The same with the tile shape (0: 128 features x 128 rows, 1: 256 x 64, 3: 128 x 64) and the way the p.pieces are summed (split:
// different work-groups, through part) given by the caller; results do not depend on either.
hipError_t launch_blk_gemm_as(int shape, bool split, const BlkGemm& p, hipStream_t st, float* part, size_t part_floats);
int blk_pieces(int K);                          // pieces of a pieced launch
bool blk_pieces_fit(int K, int pieces);         // whether every one is long enough for the kernel
// attention of the block's rows against their sequences' half caches (slot_stride elements apart), output as block
// fragments; am: scale, bias, kv_fixed as for launch_attention
void launch_attention_flash(const float* q, const void* Kc, const void* Vc, int cap, int d, int H, size_t slot_stride, const int2* rows,
                            int R, uint4* frag, hipStream_t st, const AttnMode& am = AttnMode{0.f, nullptr, 0, 0, 0, nullptr, 0});

// dst[0..bytes) = src[0..bytes), bytes a multiple of 16: reads `bytes` and writes `bytes` of HBM
void launch_copy_probe(const void* src, void* dst, size_t bytes, hipStream_t st);

// opt in to large dynamic LDS for the kernels that need it (the first call on a device does it)
hipError_t configure_kernels();
hipError_t configure_block_kernels();   // (called by configure_kernels)

}  // namespace stairs
