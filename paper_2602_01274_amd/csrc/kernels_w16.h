// Fused kernels of the bf16-weight path (gfx950, wave64, v_mfma_f32_16x16x32_f16).
//
// One decoder layer is five launches:
//   QKV GEMM   (epilogue: row scale of the RMSNorm, RoPE, Q -> f16 attention operand, K/V -> cache)
//   attention  (MFMA scores and weighted values, 8 waves per key range merged through LDS, output = the
//               f16 operand of the O projection; few heads or long contexts: several key ranges per
//               head, combined by the block that finishes last)
//   O GEMM     (epilogue: residual add, next norm's operand x*g as f16, row sum of squares)
//   gate/up GEMM (epilogue: row scale, SwiGLU, f16 operand of the down projection)
//   down GEMM  (epilogue: residual add, next norm's operand, row sum of squares)
//
// RMSNorm never runs as a kernel: x*g is what the consuming GEMM multiplies, and the per-row factor
// 1/sqrt(mean x^2 + eps) commutes with the matrix product, so it is applied to the accumulators.  The
// row sums of squares are accumulated by the producing GEMM's blocks with integer (fixed point,
// 2^-26) atomics: integer addition is associative, so the result does not depend on block order.
//
// Weight tiles hold the bf16 values converted to f16 (see kernels.h).  Tile layouts (written by pack_weight_kind_kernel):
//   PLAIN   tile nt, row i  <- matrix row 16*nt + i
//   QKV     Q and K parts: a tile holds 8 rotation pairs of one head: row i<8 <- dim 8t+i, row i+8 <-
//           dim 8t+i+hd/2 (t = tile within the head); V part plain.  RoPE then stays inside a tile.
//   GATEUP  tile nt: rows 0..7 <- gate rows 8nt..8nt+7, rows 8..15 <- up rows 8nt..8nt+7.
// KV cache of a bf16 model, per (sequence, layer): K then V, both f16, both stored per head in the
// order the attention MFMAs read them, so that every operand load of a wave is one contiguous 1 KiB:
//   K  [head][position/16][feature/32][lane][8]   lane = 16*((feature%32)/8) + position%16
//   V  [head][position/32][feature/16][lane][8]   lane = 16*((position%16)/4) + feature%16,
//                                                 element = position%4 + 4*((position%32)/16)
// (A row-major [position][d] cache makes a wave's 16 rows of one load sit a power of two apart, which
// serialises them on one memory channel: measured 4x slower at 550 keys.)
#pragma once
#include "kernels.h"

#define PACK_PLAIN 0
#define PACK_QKV 1
#define PACK_GATEUP 2

#define EPI_STORE 0
#define EPI_RESID 1
#define EPI_QKV 2
#define EPI_SWIGLU 3

#define SSQ_SCALE 67108864.0f            // 2^26
#define SSQ_INV_SCALE 1.4901161193847656e-08f

typedef unsigned long long u64;

// A slot of row sums is SSQ_SUB interleaved accumulators [sub][stride] (blocks spread their atomics
// over them to cut contention); the sum of the parts is an integer sum, so still order independent.
#define SSQ_SUB 8
__device__ __forceinline__ float row_scale(const u64* ssq, int stride, int m, float inv_dim, float eps) {
  u64 t = 0;
#pragma unroll
  for (int i = 0; i < SSQ_SUB; ++i) t += ssq[(size_t)i * stride + m];
  return 1.0f / sqrtf((float)t * SSQ_INV_SCALE * inv_dim + eps);
}
// row r's accumulators of every slot: slot 0 part 0 = v, everything else 0
__device__ __forceinline__ void ssq_init_row(u64* ssq, int n_slots, int stride, int r, float ss) {
  for (int i = threadIdx.x; i < n_slots * SSQ_SUB; i += blockDim.x) ssq[(size_t)i * stride + r] = (i == 0) ? (u64)(ss * SSQ_SCALE + 0.5f) : 0ull;
}

// bad (may be null): incremented once per weight whose half-float value is not finite (|w| > 65504, inf, NaN)
__global__ void pack_weight_kind_kernel(uint4* __restrict__ dst, const uint16_t* __restrict__ src, int N, int K, int kind, int param,
                                        int* __restrict__ bad) {
  const int KT = K >> 5;
  const size_t total = (size_t)(N >> 4) * KT * 64;
  for (size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x; idx < total; idx += (size_t)gridDim.x * blockDim.x) {
    const int lane = (int)(idx & 63);
    const size_t tile = idx >> 6;
    const int kt = (int)(tile % KT);
    const int nt = (int)(tile / KT);
    const int i = lane & 15;
    int row = nt * 16 + i;
    if (kind == PACK_QKV) {
      const int hd = param, d = N / 3;
      if (row < 2 * d) {
        const int part = (nt * 16) / d;                 // 0 = Q, 1 = K
        const int tq = nt - part * (d / 16);            // tile within the part
        const int tph = hd / 16;                        // tiles per head
        const int h = tq / tph, t = tq % tph;
        row = part * d + h * hd + 8 * t + (i & 7) + (i >> 3) * (hd / 2);
      }
    } else if (kind == PACK_GATEUP) {
      const int F = N / 2;
      row = (i < 8) ? (8 * nt + i) : (F + 8 * nt + (i - 8));
    }
    const uint16_t* p = src + (size_t)row * K + kt * 32 + (lane >> 4) * 8;
    const u32x4 h = bf16x8_to_f16x8(*reinterpret_cast<const u32x4*>(p));
    dst[idx] = make_uint4(h[0], h[1], h[2], h[3]);
    if (bad) {
      int nb = 0;
#pragma unroll
      for (int e = 0; e < 4; ++e) nb += ((h[e] & 0x7c00u) == 0x7c00u) + ((h[e] & 0x7c000000u) == 0x7c000000u);   // exponent all ones
      if (nb) atomicAdd(bad, nb);
    }
  }
}

// ------------------------------------------------------------------ producers of layer-0 input
// The f16 operand of a GEMM is stored as two tiles per (k tile, row tile): hi = f16(v) and
// lo = f16(v - hi).  hi alone carries 11 significant bits; 32 layers of a 4096-wide model turn that
// rounding into 1.5e-2 of the logit RMS (measured against the float64 oracle and reproduced by rounding
// the oracle's activations), so the target model's GEMMs multiply both tiles into the same accumulator.
// Layout: [k tile][row tile][hi|lo][row in tile][32 features]: inside a 1 KiB tile a row is 64
// contiguous bytes, and MFMA lane 16*g + j reads bytes 64*j + 16*g..+15 of it.  (Storing the tile in
// lane order instead makes a launch with 9..16 rows touch all eight 128-byte lines of every tile and
// measured 5 to 10 % slower GEMMs; this way the lines touched follow the row count.)
// where feature k0 of row m starts (hi part; lo is 512 elements further); 4 or 2 consecutive features there
__device__ __forceinline__ _Float16* packed_at(_Float16* xp, int MT_total, int m, int k0) {
  return xp + ((size_t)((k0 >> 5) * MT_total + (m >> 4)) * 128 + ((m & 15) * 4 + ((k0 & 31) >> 3))) * 8 + (k0 & 7);
}
__device__ __forceinline__ void store_packed4(_Float16* p, float a, float b, float c, float d) {
  typedef _Float16 half4 __attribute__((ext_vector_type(4)));
  const half4 h = {(_Float16)a, (_Float16)b, (_Float16)c, (_Float16)d};
  const half4 l = {(_Float16)(a - (float)h[0]), (_Float16)(b - (float)h[1]), (_Float16)(c - (float)h[2]), (_Float16)(d - (float)h[3])};
  *reinterpret_cast<half4*>(p) = h;
  *reinterpret_cast<half4*>(p + 512) = l;
}
__device__ __forceinline__ void store_packed2(_Float16* p, float a, float b) {
  const half2v h = {(_Float16)a, (_Float16)b}, l = {(_Float16)(a - (float)h[0]), (_Float16)(b - (float)h[1])};
  *reinterpret_cast<half2v*>(p) = h;
  *reinterpret_cast<half2v*>(p + 512) = l;
}

// x = E[token]; operand = f16(x * g); ssq slot 0 = sum x^2; the row's accumulators of the other slots are cleared.
// cos/sin of every absolute position for a model's rotation frequencies, evaluated in double and rounded once:
// tab[pos][j] = (cos, sin)(pos * theta^(-2j/hd)).  Filled when the workspace is bound; the QKV epilogue reads the
// row of a token's position.  grid = max_seq, block = hd/2
__global__ void rope_positions_kernel(float* __restrict__ tab, int hd, float theta) {
  const int pos = blockIdx.x, j = threadIdx.x, half = hd >> 1;
  if (j >= half) return;
  const double inv = pow((double)theta, -2.0 * (double)j / (double)hd);
  double sn, cs;
  sincos((double)pos * inv, &sn, &cs);
  tab[((size_t)pos * half + j) * 2] = (float)cs;
  tab[((size_t)pos * half + j) * 2 + 1] = (float)sn;
}

// Row r of a forward's input from embedding row e: x, the first norm's operand f16(x * g) and the row's sums of
// squares (slot 0 = sum x^2; the other slots and parts cleared unless somebody else does).  Called by all threads of a block;
// `meanwhile` runs while the row and the gains are on their way.
struct EmbedOut {
  float* x;              // residual stream rows [.][ldx]
  int ldx;
  const float* g;        // gain of the first layer's attention norm
  _Float16* xp;          // operand of the first GEMM
  int MT_total;
  u64* ssq;
  int n_slots, slot_stride;
};
template <typename F>
__device__ __forceinline__ void embed_row_w16(const uint16_t* __restrict__ e, int d, int r, const EmbedOut& o, float* red, bool clear_others, F meanwhile) {
  constexpr int CH = 4;                                  // 8-byte chunks per thread requested together: 4096 features of 256 threads
  float ss = 0.f;
  for (int k0 = threadIdx.x * 4; k0 - (int)threadIdx.x * 4 < d; k0 += CH * 256 * 4) {
    uint2 w[CH];
    float4 g[CH];
#pragma unroll
    for (int u = 0; u < CH; ++u) {
      const int k = min(k0 + u * 1024, d - 4);           // a chunk past the end repeats the last one and is dropped
      w[u] = *reinterpret_cast<const uint2*>(e + k);
      g[u] = *reinterpret_cast<const float4*>(o.g + k);
    }
    if (k0 == (int)threadIdx.x * 4) meanwhile();
#pragma unroll
    for (int u = 0; u < CH; ++u) {
      const int k = k0 + u * 1024;
      if (k >= d) break;
      const float v0 = __uint_as_float(w[u].x << 16), v1 = __uint_as_float(w[u].x & 0xffff0000u);
      const float v2 = __uint_as_float(w[u].y << 16), v3 = __uint_as_float(w[u].y & 0xffff0000u);
      *reinterpret_cast<float4*>(o.x + (size_t)r * o.ldx + k) = make_float4(v0, v1, v2, v3);
      store_packed4(packed_at(o.xp, o.MT_total, r, k), v0 * g[u].x, v1 * g[u].y, v2 * g[u].z, v3 * g[u].w);
      ss += v0 * v0 + v1 * v1 + v2 * v2 + v3 * v3;
    }
  }
  ss = block_sum(ss, red);
  if (clear_others) ssq_init_row(o.ssq, o.n_slots, o.slot_stride, r, ss);
  else if (threadIdx.x == 0) o.ssq[r] = (u64)(ss * SSQ_SCALE + 0.5f);
}
// Clears the accumulators of rows 0..R-1 but for slot 0 part 0: wave w of block z takes accumulator 4z + w.  (Each row's block
// clearing its own scatters 8-byte stores over all of them: 520 a row for a 32-layer model, in lines that 16 rows share.  512
// rows of d 4096 took 10.1 us, 17 rows 8.0; now 8.4 and 4.5.)
__device__ __forceinline__ void ssq_clear_rows(u64* ssq, int n_slots, int stride, int R, int z) {
  const int i = z * 4 + (threadIdx.x >> 6);
  if (i == 0 || i >= n_slots * SSQ_SUB) return;
  for (int r = threadIdx.x & 63; r < R; r += 64) ssq[(size_t)i * stride + r] = 0ull;
}
__host__ __device__ constexpr int ssq_clear_blocks(int n_slots) { return (n_slots * SSQ_SUB + 3) / 4; }

// grid R + ssq_clear_blocks, 256 threads
__global__ __launch_bounds__(256) void embed_w16_kernel(const uint16_t* __restrict__ E, const int* __restrict__ tokens, const int* __restrict__ draft_tok,
                                 int R, int max_seq, int G1, int d, SeqRows sr, EmbedOut out) {
  __shared__ float red[16];
  const int r = blockIdx.x;
  if (r >= R) return ssq_clear_rows(out.ssq, out.n_slots, out.slot_stride, R, r - R);
  const SeqOf q = seq_of_row(sr, r);
  const int s = q.seq, p = q.pos0 + (r - q.row0);
  const int tok = p < q.len ? tokens[(size_t)s * max_seq + p] : draft_tok[s * G1 + (p - q.len)];
  embed_row_w16(E + (size_t)tok * d, d, r, out, red, false, [] {});
}

// input rows of the pre-verification layer: x = hidden + PosEmb[e]; operand and ssq as above
// grid R + ssq_clear_blocks, 256 threads
__global__ __launch_bounds__(256) void mb_input_w16_kernel(const float* __restrict__ src, int lds, const float* __restrict__ posemb, int R,
                                    int d, float* __restrict__ x, int ldx, const float* __restrict__ g, _Float16* __restrict__ xp,
                                    int MT_total, u64* __restrict__ ssq, int n_slots, int slot_stride, SeqRows sr, MbRows mr) {
  __shared__ float red[16];
  const int r = blockIdx.x;
  if (r >= R) return ssq_clear_rows(ssq, n_slots, slot_stride, R, r - R);
  const SeqOf q = seq_of_row(sr, r);
  const int si = q.si, rr = r - q.row0;
  const float* h = src + (size_t)(mr.src_row0[si] + rr) * lds;
  const float* e = posemb + (size_t)(mr.e0[si] < 0 ? 0 : mr.e0[si] + rr) * d;
  float4 a0 = {0.f, 0.f, 0.f, 0.f}, b0 = a0;
  if ((int)threadIdx.x * 4 < d) { a0 = *reinterpret_cast<const float4*>(h + threadIdx.x * 4); b0 = *reinterpret_cast<const float4*>(e + threadIdx.x * 4); }
  float ss = 0.f;
  for (int k = threadIdx.x * 4; k < d; k += blockDim.x * 4) {
    const bool first = k == (int)threadIdx.x * 4;
    const float4 a = first ? a0 : *reinterpret_cast<const float4*>(h + k), b = first ? b0 : *reinterpret_cast<const float4*>(e + k);
    const float v0 = a.x + b.x, v1 = a.y + b.y, v2 = a.z + b.z, v3 = a.w + b.w;
    *reinterpret_cast<float4*>(x + (size_t)r * ldx + k) = make_float4(v0, v1, v2, v3);
    store_packed4(packed_at(xp, MT_total, r, k), v0 * g[k], v1 * g[k + 1], v2 * g[k + 2], v3 * g[k + 3]);
    ss += v0 * v0 + v1 * v1 + v2 * v2 + v3 * v3;
  }
  ss = block_sum(ss, red);
  if (threadIdx.x == 0) ssq[r] = (u64)(ss * SSQ_SCALE + 0.5f);
}

// hidden = x * g * row_scale for R rows (prompt ingestion: feeds M_B's prefix rows)
__global__ void hidden_rows_kernel(const float* __restrict__ x, int ldx, const float* __restrict__ g, const u64* __restrict__ ssq,
                                   int ssq_stride, float inv_dim, float eps, int d, float* __restrict__ out, int ldo) {
  const int r = blockIdx.x;
  const float rs = row_scale(ssq, ssq_stride, r, inv_dim, eps);
  for (int k = threadIdx.x; k < d; k += blockDim.x) out[(size_t)r * ldo + k] = x[(size_t)r * ldx + k] * g[k] * rs;
}

// ------------------------------------------------------------------ weight-streaming small-M GEMM, fused epilogues
// element offsets inside one (sequence, layer) K or V block of the f16 cache (layout in the file header)
__device__ __forceinline__ size_t kcache_index(int h, int hd, int max_seq, int pos, int f) {
  return (((size_t)h * (max_seq >> 4) + (pos >> 4)) * (hd >> 5) + (f >> 5)) * 512 + ((((f & 31) >> 3) << 4) + (pos & 15)) * 8 + (f & 7);
}
__device__ __forceinline__ size_t vcache_index(int h, int hd, int max_seq, int pos, int f) {
  const int p = pos & 31;
  return (((size_t)h * (max_seq >> 5) + (pos >> 5)) * (hd >> 4) + (f >> 4)) * 512 + ((((p & 15) >> 2) << 4) + (f & 15)) * 8 + (p & 3) + ((p >> 4) << 2);
}

struct GemmArgs {
  const u32x4* W;        // packed weights
  const u32x4* X;        // packed f16 operand [kt][mt_total][lane]
  int KT, R, mt0, mt_total, nt_begin;
  int nt_end;            // one past the last output tile (streaming kernel: blocks may overhang it)
  const u64* ssq_in;     // row sums of squares of the operand's source rows (null: no row scale)
  int ssq_stride;
  float inv_dim, eps;
  float* out;            // STORE: [rows][ldo] ; RESID: the residual stream x (read, add, write)
  int ldo, rowmap, G1;
  _Float16* xp_out;      // RESID: next operand f16(x*g_next) ; SWIGLU: f16(act)
  int mt_total_out;
  const float* g_next;
  u64* ssq_out;
  _Float16* qp;          // QKV: attention operand [slot][head][kt][2][lane][8]
  _Float16* kv;          // QKV: cache base of the model
  const float* rope;     // QKV: the model's table [max_seq][hd/2][2] cos, sin by absolute position
  int d, hd, layer, n_layers, max_seq, H;
  // STORE of draft logits: per (row, output tile) candidate of the token choice
  float* pick_val;       // [rows][pick_tiles] best logit (+ Gumbel noise when sampling); null: off
  int* pick_idx;
  int pick_tiles, pick_mode;
  uint64_t pick_seed;
  uint32_t pick_step;
  SeqRows sr;
  u64 row_slot;          // launches of up to 16 rows: sequence slot of row m in bits 4m..4m+3
  // K split across blocks: per-block partial sums (streaming kernel, KSB > 1: [group][KSB][NT*MT][64] f32x4) and one
  // arrival counter per group of output tiles (zero between launches)
  float* sk_part;
  unsigned* sk_cnt;
};

// What an epilogue needs to know about an activation row, looked up once per row and used for all its output tiles.
struct RowCtx {
  bool live;
  float rs;              // row scale of the operand's RMSNorm (1 without one)
  int si, rl, pos;       // QKV: sequence slot, row within the sequence, absolute position
  _Float16* Kc;          // QKV: the (sequence, layer)'s K block; V follows
  float* out;            // STORE: the row's logits
  int seq, draft;        // STORE with token choice: sequence id, 1-based draft index
};
// everything but the row scale, which waits for memory
// FEW: at most 16 rows, whose slots the launch lists (walking the table of 16 sequences takes a wave 110 instructions)
template <int EPI, bool FEW = false>
__device__ __forceinline__ RowCtx row_place(const GemmArgs& ga, int m) {
  RowCtx rc{};
  rc.live = m < ga.R;
  rc.rs = 1.f;
  auto seq_of = [&]() {
    if (!FEW || ga.sr.n_seqs == 1) return seq_of_row(ga.sr, m);
    const int si = (int)(ga.row_slot >> (4 * m)) & 15;
    return SeqOf{si, ga.sr.seq[si], ga.sr.row_off[si], ga.sr.pos0[si], ga.sr.len[si]};
  };
  if (EPI == EPI_QKV && rc.live) {
    const SeqOf q = seq_of();
    rc.si = q.si;
    rc.rl = m - q.row0;
    rc.pos = q.pos0 + rc.rl;
    rc.Kc = ga.kv + (((size_t)q.seq * ga.n_layers + ga.layer) * 2) * (size_t)ga.max_seq * ga.d;
  }
  if (EPI == EPI_STORE && rc.live) {
    const SeqOf q = seq_of();
    const int rl = m - q.row0;
    rc.seq = q.seq;
    rc.draft = q.pos0 + rl - (q.len - 1) + 1;
    const int row = ga.rowmap == ROWMAP_LIST ? q.si * ga.G1 + rl : ga.rowmap == ROWMAP_RING ? q.seq * ga.G1 + rc.draft - 1 : m;
    rc.out = ga.out + (size_t)row * ga.ldo;
  }
  return rc;
}
template <int EPI>
__device__ __forceinline__ RowCtx row_ctx(const GemmArgs& ga, int m) {
  RowCtx rc = row_place<EPI>(ga, m);
  if (EPI != EPI_RESID && rc.live) rc.rs = row_scale(ga.ssq_in, ga.ssq_stride, m, ga.inv_dim, ga.eps);
  return rc;
}
// What an epilogue reads for one (tile, row), and where its results go: the old residual values and the next norm's gains
// (RESID), cos and sin of the tile's rotation pairs (QKV), or the token choice's Gumbel noise (STORE: computed, not read).
// Kernels with several tiles per wave look it up for all tiles before the first result is stored: a load after a store that
// may alias it waits for its own memory round trip.  nt is uniform over the wave and tile counts per head are powers of two,
// so which matrix, head and tile nt falls into is scalar arithmetic and shifts.
struct EpiAux { f32x4 a, b; char* p; };
template <int EPI>
__device__ __forceinline__ EpiAux epi_aux(const GemmArgs& ga, const RowCtx& rc, int nt, int m, int l) {
  EpiAux x{};
  if (!rc.live) return x;
  const int g4 = l >> 4;
  if (EPI == EPI_RESID) {
    const int n = nt * 16 + g4 * 4;
    x.p = reinterpret_cast<char*>(ga.out + (size_t)m * ga.ldo + n);
    x.a = *reinterpret_cast<const f32x4*>(x.p);
    x.b = *reinterpret_cast<const f32x4*>(ga.g_next + n);
  } else if (EPI == EPI_QKV) {
    const int tiles_d = ga.d >> 4, half = ga.hd >> 1, tsh = ga.hd == 128 ? 3 : 2;      // 8 or 4 tiles per head
    if (nt < 2 * tiles_d) {
      const int tq = nt >= tiles_d ? nt - tiles_d : nt;
      // rotation pairs (dim, dim + hd/2) and (dim + 1, dim + 1 + hd/2), see gemm_epilogue
      const int h = tq >> tsh, dim = 8 * (tq & ((1 << tsh) - 1)) + 4 * (g4 & 1) + (g4 >= 2 ? 2 : 0);
      x.a = *reinterpret_cast<const f32x4*>(ga.rope + ((size_t)rc.pos * half + dim) * 2);
      if (nt < tiles_d)
        // attention operand: [slot][head][kt][2 row tiles][hi|lo][lane][8], lane = 16*(dim%32/8) + row%16
        x.p = reinterpret_cast<char*>(ga.qp + ((((size_t)rc.si * ga.H + h) * (ga.hd >> 5) + (dim >> 5)) * 2 + (rc.rl >> 4)) * 1024 + (((dim & 31) >> 3) * 16 + (rc.rl & 15)) * 8 + (dim & 7));
      else
        x.p = reinterpret_cast<char*>(rc.Kc + kcache_index(h, ga.hd, ga.max_seq, rc.pos, dim));
    } else {
      const int tv = nt - 2 * tiles_d, h = tv >> tsh, f0 = (tv & ((1 << tsh) - 1)) * 16 + g4 * 4;
      x.p = reinterpret_cast<char*>(rc.Kc + (size_t)ga.max_seq * ga.d + vcache_index(h, ga.hd, ga.max_seq, rc.pos, f0));
    }
  } else if (EPI == EPI_STORE) {
    x.p = reinterpret_cast<char*>(rc.out + nt * 16 + g4 * 4);
    if (ga.pick_val && ga.pick_mode) {
      const uint4 bits = vocab_bits(ga.pick_seed, rc.seq, ga.pick_step, (uint32_t)rc.draft, PURPOSE_DRAFT, (uint32_t)(nt * 4 + g4));
      x.a = f32x4{gumbel(u01(bits.x)), gumbel(u01(bits.y)), gumbel(u01(bits.z)), gumbel(u01(bits.w))};
    }
  } else {
    // each of lanes l and l ^ 32 takes two of the four features whose gate and up they hold, see gemm_epilogue
    x.p = reinterpret_cast<char*>(packed_at(ga.xp_out, ga.mt_total_out, m, nt * 8 + (g4 & 1) * 4 + (g4 >= 2 ? 2 : 0)));
  }
  return x;
}
// A row's squares over one tile's 16 outputs as a fixed-point number (all 64 lanes call it; sq: this lane's part), and the
// addition to the row's accumulator.  Each half of a tile (8 outputs) is a whole number, and kernels with several tiles per
// wave add whole numbers before the one atomic: the accumulator ends up with the same bits however tiles and half tiles are
// dealt to waves and blocks.
__device__ __forceinline__ u64 tile_ssq(float sq) {
  const unsigned u = __float_as_uint(sq);
  const auto a = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  const u64 half = (u64)((__uint_as_float(a[0]) + __uint_as_float(a[1])) * SSQ_SCALE + 0.5f);
  const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)half, (unsigned)half, false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)(half >> 32), (unsigned)(half >> 32), false, false);
  return ((u64)hi[0] << 32 | lo[0]) + ((u64)hi[1] << 32 | lo[1]);
}
__device__ __forceinline__ void add_row_ssq(const GemmArgs& ga, const RowCtx& rc, int m, int l, u64 fixed) {
  if (rc.live && (l >> 4) == 0) atomicAdd(ga.ssq_out + (size_t)(blockIdx.x % SSQ_SUB) * ga.ssq_stride + m, fixed);
}
// the hardware's 2^x (1 ulp; results below 2^-126 are zero)
__device__ __forceinline__ float exp2_hw(float x) { return __builtin_amdgcn_exp2f(x); }
// 4 x 4 transpose of v among the four lanes of a quad: lane i gets v[i] of lanes 0..3
template <int O>
__device__ __forceinline__ void quad_step(float (&v)[4], int l) {
  const bool up = l & O;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    if (i & O) continue;
    const float got = dpp_f32<O == 1 ? 0xB1 : 0x4E>(up ? v[i] : v[i + O]);       // of lane l ^ O
    v[i] = up ? got : v[i];
    v[i + O] = up ? v[i + O] : got;
  }
}
__device__ __forceinline__ void quad_transpose(float (&v)[4], int l) {
  quad_step<1>(v, l);
  quad_step<2>(v, l);
}
// x: lanes 0..31 keep theirs and give y's; lanes 32..63 get x's upper partner (one exchange for two values)
__device__ __forceinline__ void swap_halves(float& x, float& y) {
  const auto p = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false);
  x = __uint_as_float(p[0]);
  y = __uint_as_float(p[1]);
}
// g / (1 + exp(-g)) * u.  exp(-g) = 2^n 2^f with n + f = -g log2(e), f small and with the product's rounding put back; the
// quotient by a refined reciprocal.  The divisor lies in [1, 2^126], so neither needs the range handling of expf and of a
// division, a third of this epilogue's instructions; the error is theirs (2.3 ulp over g in [-85, 100]).
__device__ __forceinline__ float silu_times(float g, float u) {
  const float p = -g * 1.44269504f;                                    // log2(e) = 1.44269504 + 1.925963e-8
  const float lost = fmaf(-g, 1.92596303e-8f, fmaf(-g, 1.44269504f, -p));
  const float pc = fminf(p, 126.f), n = __builtin_rintf(pc);
  const float d = 1.0f + __builtin_amdgcn_ldexpf(exp2_hw((pc - n) + lost), (int)n);
  float r = __builtin_amdgcn_rcpf(d);
  r = fmaf(fmaf(-d, r, 1.0f), r, r);
  float q = g * r;
  q = fmaf(fmaf(-d, q, g), r, q);
  return q * u;
}

// Epilogue of one accumulator lane, shared by the GEMM kernels.  Lane l of a 16x16 result tile holds tile rows (outputs)
// 4*(l/16)..+3 of activation row m.  All 64 lanes of the tile call this together: in the paired weight layouts (rotation pairs
// of QKV, gate/up of SwiGLU) lane l ^ 32 holds the partners i+8 resp. i-8 of this lane's outputs, and the two exchange so that
// each has both members of two of the four pairs.
// (Exchanges as vector swaps; through LDS, with expf and divisions: 512 rows QKV 90.9 -> 89.4 us, 160 rows 71.9 -> 70.5, 1 row of
// d 768 QKV 3.5 -> 3.4, gate/up 4.1 -> 4.0.)
// RESID returns the lane's part of the row's sum of squares over this tile, for tile_ssq.
// XP: RESID's operand goes to xp, which the caller has worked out ahead.
// VT: rows of a tile may be 16 consecutive positions (prompt rows): V is stored 4 positions at a time where they are.
template <int EPI, bool VT = false, bool XP = false>
__device__ __forceinline__ float gemm_epilogue(const GemmArgs& ga, const RowCtx& rc, const EpiAux& ax, int nt, int m, int l, f32x4 s, _Float16* xp = nullptr) {
  typedef _Float16 half4 __attribute__((ext_vector_type(4)));
  const int g4 = l >> 4;
  const bool live = rc.live;
  const float rs = rc.rs;
  float sq = 0.f;
  if (EPI == EPI_STORE) {
    const int n = nt * 16 + g4 * 4;
    const f32x4 lg = s * rs;
    if (live) {
      *reinterpret_cast<f32x4*>(ax.p) = lg;
    }
    if (ga.pick_val) {
      // token choice, first stage: best of this tile's 16 vocabulary entries for row m
      // (argmax of the logits, or of logits + Gumbel noise; lowest id wins ties)
      float best = -INFINITY;
      int bi = 0x7fffffff;
      if (live) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float v = lg[r] + ax.a[r];
          if (v > best) { best = v; bi = n + r; }
        }
      }
#pragma unroll
      for (int o = 16; o <= 32; o <<= 1) {
        const float ov = __shfl_xor(best, o, 64);
        const int oi = __shfl_xor(bi, o, 64);
        if (ov > best || (ov == best && oi < bi)) { best = ov; bi = oi; }
      }
      if (live && g4 == 0) {
        ga.pick_val[(size_t)m * ga.pick_tiles + nt] = best;
        ga.pick_idx[(size_t)m * ga.pick_tiles + nt] = bi;
      }
    }
  } else if (EPI == EPI_RESID) {
    if (live) {
      const f32x4 xn = ax.a + s, gn = ax.b;
      *reinterpret_cast<f32x4*>(ax.p) = xn;
      store_packed4(XP ? xp : packed_at(ga.xp_out, ga.mt_total_out, m, nt * 16 + g4 * 4), xn[0] * gn[0], xn[1] * gn[1], xn[2] * gn[2], xn[3] * gn[3]);
      sq = xn[0] * xn[0] + xn[1] * xn[1] + xn[2] * xn[2] + xn[3] * xn[3];
    }
  } else if (EPI == EPI_SWIGLU) {
    float g0 = s[0], u0 = s[2], g1 = s[1], u1 = s[3];
    swap_halves(g0, u0);
    swap_halves(g1, u1);
    if (live) store_packed2(reinterpret_cast<_Float16*>(ax.p), silu_times(g0 * rs, u0 * rs), silu_times(g1 * rs, u1 * rs));
  } else {  // EPI_QKV
    _Float16* p = reinterpret_cast<_Float16*>(ax.p);
    const int tiles_d = ga.d >> 4;
    if (nt < 2 * tiles_d) {
      float a0 = s[0], b0 = s[2], a1 = s[1], b1 = s[3];
      swap_halves(a0, b0);
      swap_halves(a1, b1);
      if (live) {
        a0 *= rs; b0 *= rs; a1 *= rs; b1 *= rs;
        const float v[4] = {a0 * ax.a[0] - b0 * ax.a[1], a1 * ax.a[2] - b1 * ax.a[3],              // dims dim, dim + 1
                            b0 * ax.a[0] + a0 * ax.a[1], b1 * ax.a[2] + a1 * ax.a[3]};             // and hd/2 further
        const half2v h0 = {(_Float16)v[0], (_Float16)v[1]}, h1 = {(_Float16)v[2], (_Float16)v[3]};
        const int far = (ga.hd >> 6) * 512;              // half a head in both layouts: blocks of 32 dims, 512 elements each (Q: 2048)
        if (nt < tiles_d) {
          const half2v l0 = {(_Float16)(v[0] - (float)h0[0]), (_Float16)(v[1] - (float)h0[1])}, l1 = {(_Float16)(v[2] - (float)h1[0]), (_Float16)(v[3] - (float)h1[1])};
          *reinterpret_cast<half2v*>(p) = h0;
          *reinterpret_cast<half2v*>(p + 512) = l0;
          *reinterpret_cast<half2v*>(p + 4 * far) = h1;
          *reinterpret_cast<half2v*>(p + 4 * far + 512) = l1;
        } else {
          *reinterpret_cast<half2v*>(p) = h0;
          *reinterpret_cast<half2v*>(p + far) = h1;
        }
      }
    } else {
      float v[4] = {s[0] * rs, s[1] * rs, s[2] * rs, s[3] * rs};
      bool quad = false;
      if (VT) {
        // the quad's rows are four live positions 4i..4i+3 of one sequence (rows ascend, so the last one decides)
        const int last = l | 3;
        const bool same = __shfl((int)live, last, 64) && __shfl(rc.si, last, 64) == rc.si && __shfl(rc.si, l & ~3, 64) == rc.si;
        quad = same && (rc.pos & 3) == (l & 3);
        float t[4] = {v[0], v[1], v[2], v[3]};
        quad_transpose(t, l);
        if (quad) {
          const half4 hv = {(_Float16)t[0], (_Float16)t[1], (_Float16)t[2], (_Float16)t[3]};
          // feature l & 3 of the four, at the quad's first position (of one such quad position is the fastest index)
          *reinterpret_cast<half4*>(p - (rc.pos & 3) + (l & 3) * 8) = hv;
        }
      }
      if (live && !quad) {
#pragma unroll
        for (int r = 0; r < 4; ++r) p[r * 8] = (_Float16)v[r];   // features are 8 elements apart
      }
    }
  }
  return sq;
}

// X17 = 1 (with MT = 2): the launch covers exactly 17 rows (a full draft window plus the committed
// token).  Only row 16 of the second row tile exists, so its hi and lo parts share ONE extra MFMA: operand
// column 0 = hi of row 16, column 1 = lo of row 16, the other columns zero in registers, and the epilogue
// adds accumulator columns 0 and 1.  That is three MFMAs and 17 fetched operand rows per K step instead
// of four and 32.
// 8-wave blocks are held to 128 VGPRs (4 waves per SIMD) so that two blocks fit a CU.
// HL = operand parts multiplied: 2 = hi and lo tiles (the target model's QKV, gate/up and down GEMMs),
// 1 = hi only (draft and pre-verification layer: two layers deep, their logits stay at 4e-3 of the RMS).
// KSB > 1: K is also split across KSB blocks (block id = group * KSB + slice; a group is NT output tiles).
// Every block of the launch needs the operand rows of its K range, so a matrix with about as many tiles as
// there are CUs (O and down projections) fetches the operand once per tile; with KSB slices of NT = KSB
// tiles each the block count stays and each block fetches 1/KSB of it.  The slices' sums meet in memory
// without a device-scope fence (which writes back and invalidates a whole L2 and costs far more than it
// saves here): each block writes its partial tiles with agent-scope relaxed atomic stores (write-through
// to memory: `sc1`), waits until they have completed (vmcnt 0), and then bumps the group's counter with
// an agent-scope atomic add; the block that sees the other KSB-1 arrivals reads all partials back with
// agent-scope atomic loads (which do not hit in its XCD's L2), adds them in slice order (so the result
// does not depend on which block came last), resets the counter and runs the epilogue.  Nobody waits
// for anybody: a block that is not the last one simply ends.
template <int EPI, int MT, int NT, int WAVES, int U, int TAG, int X17 = 0, int HL = 1, int KSB = 1>
__global__ __launch_bounds__(WAVES * 64, (WAVES == 8 ? (NT >= 5 ? 2 : 4) : 1)) void gemm_w16_kernel(const GemmArgs ga) {
  static_assert(!X17 || MT == 2, "the 17-row form uses two row tiles");
  // partial sums of the waves; more than 64 KB of them are handed over in two halves
  constexpr int RW = (WAVES * NT * MT > 64) ? WAVES / 2 : WAVES;
  static_assert(RW * NT * MT <= 64, "the reduction buffer must fit the 64 KB of static LDS");
  static_assert(KSB <= RW, "the partial sums of the K slices are gathered in the reduction buffer");
  constexpr int NRED = KSB > 1 ? KSB : RW;            // summands per accumulator lane in the epilogue
  __shared__ f32x4 red[RW][NT * MT][64];
  __shared__ unsigned sk_arrived;
  const int grp = blockIdx.x / KSB, ks = blockIdx.x % KSB;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;   // wave id as a scalar
  const int nt0 = ga.nt_begin + grp * NT;
  const int KT = ga.KT;
  const int kbeg = (int)((long)ks * KT / KSB), kend = (int)((long)(ks + 1) * KT / KSB);   // this block's K steps
  // K steps are dealt to the block's waves round-robin (wave w takes w, w+WAVES, ...): at any moment
  // the waves of a block, and the blocks sharing a CU, read neighbouring operand tiles, which keeps the
  // operand in the CU's L1 instead of fetching it once per wave from L2
  // steps of this wave: index i -> kt = kbeg + i*WAVES + wave
  const int ke = (kend - kbeg - wave + WAVES - 1) / WAVES;
  f32x4 acc[NT][MT];
#pragma unroll
  for (int a = 0; a < NT; ++a)
#pragma unroll
    for (int b = 0; b < MT; ++b) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
  const u32x4* wp[NT];
#pragma unroll
  for (int a = 0; a < NT; ++a) wp[a] = ga.W + (size_t)min(nt0 + a, ga.nt_end - 1) * KT * 64 + lane;   // a tile past the end repeats the last one, unused
  // Operand pointers, one per row tile.  Lanes whose row does not exist read the tile's last live row instead
  // (the same cache lines the live lanes fetch, and their accumulator columns are discarded): the operand
  // traffic scales with the number of rows, not with whole 16-row tiles, and no load is conditional.
  const u32x4* xpb[MT];
#pragma unroll
  for (int b = 0; b < MT; ++b) {
    const int live = min(16, max(1, ga.R - (ga.mt0 + b) * 16));
    xpb[b] = ga.X + (size_t)(ga.mt0 + b) * 128 + min(lane & 15, live - 1) * 4 + (lane >> 4);
  }
  // row 0 of row tile mt0+1: its hi part for even operand columns, its lo part for odd ones
  const u32x4* xp17 = ga.X + (size_t)(ga.mt0 + 1) * 128 + (lane >> 4) + (HL == 2 ? (lane & 1) * 64 : 0);
  const bool x17_live = (lane & 15) < HL;
  const int mtt = ga.mt_total;

  constexpr int BW = X17 ? HL + 1 : MT * HL;           // operand tiles per K step: [row tile][part]
  u32x4 A0[U][NT], A1[U][NT], B0[U][BW], B1[U][BW];
  const u32x4 zero = {0u, 0u, 0u, 0u};
  // The K loop has no branches: a branch around a load makes the compiler wait for every outstanding load
  // where the paths join (the load counter completes in order, and the number of newer loads then differs
  // by path), which would serialise each wave on memory latency.  K steps past the wave's last one re-read
  // its last tile (an L1 hit) and their weights are replaced by zeros before use.
  auto load = [&](u32x4(&A)[U][NT], u32x4(&B)[U][BW], int k0) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const size_t kt = (size_t)min(kbeg + (k0 + u) * WAVES + wave, kend - 1);
#pragma unroll
      for (int a = 0; a < NT; ++a) A[u][a] = __builtin_nontemporal_load(wp[a] + kt * 64);
      if (X17) {
#pragma unroll
        for (int h = 0; h < HL; ++h) B[u][h] = xpb[0][(kt * mtt * 2 + h) * 64];
        B[u][HL] = xp17[kt * mtt * 2 * 64];
      } else {
#pragma unroll
        for (int b = 0; b < MT; ++b)
#pragma unroll
          for (int h = 0; h < HL; ++h) B[u][b * HL + h] = xpb[b][(kt * mtt * 2 + h) * 64];
      }
    }
  };
  auto compute = [&](u32x4(&A)[U][NT], u32x4(&B)[U][BW], int k0) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const bool valid = k0 + u < ke;                  // wave-uniform
      half8 bh[BW];
#pragma unroll
      for (int b = 0; b < BW; ++b) bh[b] = __builtin_bit_cast(half8, (X17 && b == HL && !x17_live) ? zero : B[u][b]);
#pragma unroll
      for (int a = 0; a < NT; ++a) {
        const half8 ah = __builtin_bit_cast(half8, valid ? A[u][a] : zero);
#pragma unroll
        for (int b = 0; b < MT; ++b)
#pragma unroll
          for (int h = 0; h < HL; ++h) {
            if (X17 && b == 1 && h > 0) continue;
            acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ah, bh[(X17 && b == 1) ? HL : b * HL + h], acc[a][b], 0, 0, 0);
          }
      }
    }
  };
  // Two register sets, both requested before the loop; each is refilled right after its products were issued, in the same
  // order on every path into the loop, and the scheduler may not move loads across the phase boundaries: the wait before a
  // phase's products then leaves the other set's loads in flight.  The last two sets are not refilled.
  // The weights are requested before anything else, since theirs is the longest of the memory round trips that a launch is a
  // chain of.  What the epilogue needs is looked up while they travel: sums of squares, places, residuals and gains, rotations
  // or noise, and with them the kernel arguments, each line of which is a round trip of its own where it is first read.
  // Doing all that at the end, kernel durations before and now: 7B at 9 rows QKV 19.3 -> 18.4 us, O 8.9 -> 8.5, LM head 43.3 ->
  // 41.2; 13 rows of d 768 QKV 5.1 -> 4.3, O 4.4 -> 4.0; 1 row of d 768 QKV 4.2 -> 3.6, LM head with sampling 12.6 -> 10.3.
  constexpr int EIT = (NT * MT + WAVES - 1) / WAVES;   // epilogue items ([tile][row tile], a wave each) per wave
  // where the registers hold two sets and the epilogue's inputs
  constexpr bool AHEAD = (2 * U * (NT + BW) + NT * MT) * 4 <= (WAVES == 8 && NT < 5 ? 72 : 160);
  u64 ssq_pre[EIT][SSQ_SUB];
  RowCtx rcs[EIT];
  EpiAux axs[EIT];
  __builtin_amdgcn_sched_barrier(0);
  load(A0, B0, 0);
  __builtin_amdgcn_sched_barrier(0);
  if (EPI != EPI_RESID) {
#pragma unroll
    for (int it = 0; it < EIT; ++it) {
      const int ab = wave + it * WAVES;
      if (ab < NT * MT) {
        const u64* sp = ga.ssq_in + min((ga.mt0 + ab % MT) * 16 + (lane & 15), ga.R - 1);
#pragma unroll
        for (int i = 0; i < SSQ_SUB; ++i) ssq_pre[it][i] = sp[(size_t)i * ga.ssq_stride];
      }
    }
  }
  if (EPI == EPI_RESID) asm volatile("" ::"s"(ga.out), "s"(ga.xp_out), "s"(ga.g_next), "s"(ga.ssq_out), "s"(ga.ldo), "s"(ga.mt_total_out), "s"(ga.ssq_stride));
  if (EPI == EPI_SWIGLU) asm volatile("" ::"s"(ga.xp_out), "s"(ga.mt_total_out));
  if (EPI == EPI_QKV) asm volatile("" ::"s"(ga.qp), "s"(ga.kv), "s"(ga.rope), "s"(ga.max_seq), "s"(ga.H), "s"(ga.hd), "s"(ga.d));
  if (EPI == EPI_STORE) asm volatile("" ::"s"(ga.out), "s"(ga.pick_val), "s"(ga.pick_idx), "s"(ga.pick_tiles));
  __builtin_amdgcn_sched_barrier(0);
  load(A1, B1, U);
  __builtin_amdgcn_sched_barrier(0);
  auto look_up = [&](int it) {
    const int ab = wave + it * WAVES, m = (ga.mt0 + ab % MT) * 16 + (lane & 15);
    rcs[it] = row_place<EPI>(ga, m);
    axs[it] = epi_aux<EPI>(ga, rcs[it], min(nt0 + ab / MT, ga.nt_end - 1), m, lane);
  };
  if (AHEAD) {
#pragma unroll
    for (int it = 0; it < EIT; ++it)
      if (wave + it * WAVES < NT * MT) look_up(it);
    __builtin_amdgcn_sched_barrier(0);
  }
  int k0 = 0;
  for (; k0 + 2 * U < ke; k0 += 2 * U) {
    compute(A0, B0, k0);
    __builtin_amdgcn_sched_barrier(0);
    load(A0, B0, k0 + 2 * U);
    __builtin_amdgcn_sched_barrier(0);
    compute(A1, B1, k0 + U);
    __builtin_amdgcn_sched_barrier(0);
    load(A1, B1, k0 + 3 * U);
    __builtin_amdgcn_sched_barrier(0);
  }
  compute(A0, B0, k0);
  compute(A1, B1, k0 + U);
  if (RW < WAVES) {
    if (wave >= RW) {
#pragma unroll
      for (int a = 0; a < NT; ++a)
#pragma unroll
        for (int b = 0; b < MT; ++b) red[wave - RW][a * MT + b][lane] = acc[a][b];
    }
    __syncthreads();
    if (wave < RW) {
#pragma unroll
      for (int a = 0; a < NT; ++a)
#pragma unroll
        for (int b = 0; b < MT; ++b) acc[a][b] += red[wave][a * MT + b][lane];
    }
    __syncthreads();
  }
  if (wave < RW) {
#pragma unroll
    for (int a = 0; a < NT; ++a)
#pragma unroll
      for (int b = 0; b < MT; ++b) red[wave][a * MT + b][lane] = acc[a][b];
  }
  __syncthreads();
  if (KSB > 1) {
    u64* part = reinterpret_cast<u64*>(ga.sk_part);
#pragma unroll
    for (int it = 0; it < EIT; ++it) {
      const int t = threadIdx.x + it * WAVES * 64;
      if (t < NT * MT * 64) {
        f32x4 p = red[0][t >> 6][t & 63];
#pragma unroll
        for (int w = 1; w < RW; ++w) p += red[w][t >> 6][t & 63];
        u64* dst = part + ((size_t)(grp * KSB + ks) * NT * MT * 64 + t) * 2;
        const float2 lo = {p[0], p[1]}, hi = {p[2], p[3]};
        __hip_atomic_store(dst, __builtin_bit_cast(u64, lo), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(dst + 1, __builtin_bit_cast(u64, hi), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
    }
    PACER_WAIT_VMCNT0();   // this wave's write-through stores have completed
    __syncthreads();
    if (threadIdx.x == 0) sk_arrived = __hip_atomic_fetch_add(ga.sk_cnt + grp, 1u, PACER_HO_ORDER, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    if (sk_arrived != KSB - 1) return;
    if (threadIdx.x == 0) __hip_atomic_store(ga.sk_cnt + grp, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
    for (int it = 0; it < EIT; ++it) {
      const int t = threadIdx.x + it * WAVES * 64;
      if (t < NT * MT * 64) {
#pragma unroll
        for (int k = 0; k < KSB; ++k) {
          const u64* src = part + ((size_t)(grp * KSB + k) * NT * MT * 64 + t) * 2;
          const float2 lo = __builtin_bit_cast(float2, __hip_atomic_load(src, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
          const float2 hi = __builtin_bit_cast(float2, __hip_atomic_load(src + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
          red[k][t >> 6][t & 63] = f32x4{lo.x, lo.y, hi.x, hi.y};
        }
      }
    }
    __syncthreads();
  }

  // Epilogue.  One wave per (tile a, row tile b); lane l owns the accumulator lane l: activation row m = 16*(mt0+b) + l%16,
  // tile rows 4*(l/16)..+3.
#pragma unroll
  for (int it = 0; it < EIT; ++it) {
    const int ab = wave + it * WAVES;
    if (ab >= NT * MT) break;
    const int a = ab / MT, b = ab % MT, l = lane;
    const int m = (ga.mt0 + b) * 16 + (l & 15);
    const int nt = nt0 + a;
    if (nt >= ga.nt_end) continue;
    f32x4 s = red[0][ab][l];
#pragma unroll
    for (int w = 1; w < NRED; ++w) s += red[w][ab][l];
    if (X17 && HL == 2 && b == 1 && (l & 15) == 0) {   // row 16: hi product in column 0, lo product in column 1
#pragma unroll
      for (int w = 0; w < NRED; ++w) s += red[w][ab][l + 1];
    }
    if (!AHEAD) look_up(it);
    RowCtx rc = rcs[it];
    if (EPI != EPI_RESID) {
      u64 ssq = 0;
#pragma unroll
      for (int i = 0; i < SSQ_SUB; ++i) ssq += ssq_pre[it][i];
      rc.rs = 1.0f / sqrtf((float)ssq * SSQ_INV_SCALE * ga.inv_dim + ga.eps);
    }
    const float sq = gemm_epilogue<EPI>(ga, rc, axs[it], nt, m, l, s);
    if (EPI == EPI_RESID) add_row_ssq(ga, rc, m, l, tile_ssq(sq));
  }
}

// ------------------------------------------------------------------ GEMM of a few rows over a short K
// Up to 16 rows and a K that a block's waves hold in registers: the draft and pre-verification layers, narrow targets.
//   block   one output tile, or half of one (HALF); WAVES waves take the K tiles round-robin, U steps each
// Such a launch takes 3 to 5 us of which the bytes take a fraction; what bounds it is one wave's way through the kernel:
// each memory round trip (0.2 to 1 us), and 2.4 to 3.7 ns for every instruction of a wave that is alone on its SIMD, so 300
// instructions are one more us.  Hence: everything is requested at once, without a loop; loads go through buffer
// descriptors whose range ends with the tile's last K step (a step past it reads zeros: no clamps, no selects) and whose
// lane offsets are the same for all steps; the arguments that the loads need come first and in registers (kernarg preload);
// what the epilogue needs is worked out while the weights travel, down to the addresses it stores to.
// Kernel durations, gemm_w16_kernel -> this: 1 row of d 768 O 3.7 -> 3.2 us, down 5.3 -> 4.4, gate/up 4.8 -> 4.2; 13 rows hi+lo
// QKV 4.3 -> 4.2, gate/up 4.9 -> 4.5, down 6.0 -> 5.5; 1 row of d 2048 O and down together 13.4 -> 11.5, QKV 7.1 -> 6.5.
// HALF: a matrix of at most 128 tiles leaves CUs idle.  A weight load takes 8 outputs of two K tiles: lanes of tile rows 0..7
// bring K tile 2s, the others 2s + 1.  Both K tiles' products run with the whole register; of the first the lanes of result
// rows 0..7 count, of the second the others, and the epilogue adds the two.
// v of lane l ^ 32
__device__ __forceinline__ float other_half(float v, int lane) {
  const unsigned u = __float_as_uint(v);
  const auto p = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return __uint_as_float(lane < 32 ? p[1] : p[0]);
}
template <int EPI, int TAG, int HL, int WAVES, int U, int HALF>
__global__ __launch_bounds__(WAVES * 64) void gemm_row_kernel(const u32x4* W, const u32x4* X, int KT, int R, int nt_begin, const GemmArgs ga) {
  static_assert(!HALF || (EPI != EPI_QKV && EPI != EPI_SWIGLU), "half tiles have no pairs");
  constexpr int KP = HALF ? 2 : 1;                     // K tiles per step
  constexpr int NT_LOAD = 2;                           // cache policy: non-temporal
  __shared__ f32x4 red[WAVES - 1][64];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int half = HALF ? blockIdx.x & 1 : 0, nt = nt_begin + (HALF ? blockIdx.x >> 1 : blockIdx.x);
  const auto wr = buffer_of(W + (size_t)nt * KT * 64, KT * 1024), xr = buffer_of(X, KT * 2048);
  const int wv = HALF ? (lane & 48) * 16 + half * 128 + (lane & 7) * 16 + ((lane >> 3) & 1) * 1024 : lane * 16;
  const int xv = min(lane & 15, R - 1) * 64 + (lane >> 4) * 16;      // lanes of rows that do not exist repeat the last one's
  u32x4 A[U], B[U][KP * HL];
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int s = (wave + u * WAVES) * KP;
    A[u] = __builtin_amdgcn_raw_buffer_load_b128(wr, wv, s * 1024, NT_LOAD);
#pragma unroll
    for (int j = 0; j < KP; ++j)
#pragma unroll
      for (int h = 0; h < HL; ++h) B[u][j * HL + h] = __builtin_amdgcn_raw_buffer_load_b128(xr, xv + j * 2048 + h * 1024, s * 2048, 0);
  }
  __builtin_amdgcn_sched_barrier(0);
  const int m = lane & 15, l = HALF ? (lane & 31) + 32 * half : lane;  // l: the lane whose outputs this one finishes
  RowCtx rc{};
  EpiAux ax{};
  _Float16* xp = nullptr;
  u64* ssq_to = nullptr;
  // the arguments of the epilogue in one round trip
  if (EPI == EPI_RESID) asm volatile("" ::"s"(ga.R), "s"(ga.out), "s"(ga.xp_out), "s"(ga.g_next), "s"(ga.ssq_out), "s"(ga.ldo), "s"(ga.mt_total_out), "s"(ga.ssq_stride));
  else asm volatile("" ::"s"(ga.R), "s"(ga.ssq_in), "s"(ga.ssq_stride), "s"(ga.inv_dim), "s"(ga.eps));
  if (EPI == EPI_SWIGLU) asm volatile("" ::"s"(ga.xp_out), "s"(ga.mt_total_out));
  if (EPI == EPI_QKV) asm volatile("" ::"s"(ga.qp), "s"(ga.kv), "s"(ga.rope), "s"(ga.max_seq), "s"(ga.H), "s"(ga.hd), "s"(ga.d), "s"(ga.layer), "s"(ga.n_layers), "s"(ga.sr.n_seqs), "s"(ga.sr.seq[0]), "s"(ga.sr.row_off[0]), "s"(ga.sr.pos0[0]));
  if (EPI == EPI_STORE) asm volatile("" ::"s"(ga.out), "s"(ga.pick_val), "s"(ga.pick_idx), "s"(ga.pick_tiles), "s"(ga.pick_mode), "s"(ga.pick_seed), "s"(ga.pick_step), "s"(ga.sr.n_seqs), "s"(ga.sr.seq[0]), "s"(ga.sr.row_off[0]), "s"(ga.sr.pos0[0]), "s"(ga.sr.len[0]));
  if (wave == 0) {
    u64 ssq = 0;
    if (EPI != EPI_RESID) {
      const u64* sp = ga.ssq_in + (size_t)((lane >> 4) * 2) * ga.ssq_stride + min(m, R - 1);
      ssq = sp[0] + sp[ga.ssq_stride];
    }
    rc = row_place<EPI, true>(ga, m);
    ax = epi_aux<EPI>(ga, rc, nt, m, l);
    if (EPI == EPI_RESID) {
      xp = packed_at(ga.xp_out, ga.mt_total_out, m, nt * 16 + (l >> 4) * 4);
      ssq_to = ga.ssq_out + (size_t)(blockIdx.x % SSQ_SUB) * ga.ssq_stride + m;
    } else {
      ssq += __shfl_xor((unsigned long long)ssq, 16, 64);
      ssq += __shfl_xor((unsigned long long)ssq, 32, 64);
      rc.rs = 1.0f / sqrtf((float)ssq * SSQ_INV_SCALE * ga.inv_dim + ga.eps);
    }
  }
  __builtin_amdgcn_sched_barrier(0);
  f32x4 acc[KP];
#pragma unroll
  for (int j = 0; j < KP; ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int u = 0; u < U; ++u)
#pragma unroll
    for (int j = 0; j < KP; ++j)
#pragma unroll
      for (int h = 0; h < HL; ++h)
        acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8, A[u]), __builtin_bit_cast(half8, B[u][j * HL + h]), acc[j], 0, 0, 0);
  f32x4 s = acc[0];
  if (HALF) {
    const bool first = lane < 32;
#pragma unroll
    for (int r = 0; r < 4; ++r) s[r] = first ? acc[0][r] : acc[KP - 1][r];
  }
  if (wave) red[wave - 1][lane] = s;
  __syncthreads();
  if (wave) return;
#pragma unroll
  for (int w = 0; w < WAVES - 1; ++w) s += red[w][lane];
  if (HALF) {
#pragma unroll
    for (int r = 0; r < 4; ++r) s[r] += other_half(s[r], lane);
    if (lane >= 32) rc.live = false;                   // lane - 32 finishes these outputs
  }
  const float sq = gemm_epilogue<EPI, false, true>(ga, rc, ax, nt, m, l, s, xp);
  if (EPI == EPI_RESID) {
    const u64 fixed = tile_ssq(sq);
    if (rc.live && lane < 16) atomicAdd(ssq_to, fixed);
  }
}

// ------------------------------------------------------------------ MFMA attention over the f16 KV cache
// grid (key splits, heads, sequences), NW waves per block.  A block owns `kps` keys of one head; its
// waves take the 32-key groups of that range round-robin, each running an online softmax in registers:
//   scores  S^T[key][row] = K[key][:] . Q[row][:]   (A = K tile straight from the cache, B = Q operand)
//   values  O^T[dim][row] += V^T[dim][keys] P^T[keys][row]; the probabilities leave the first MFMA in
//           exactly the lane layout the second one wants for B (contraction index = the 8 keys a lane
//           holds), and V^T rows are contiguous along keys.
// The NW wave states meet in LDS (dynamic, NW x live rows x (HD + 4) floats) and are combined in one pass.
// With one split the block writes the f16 operand of the O projection directly; with several, each block
// writes a partial (un-normalised values, running max, running sum per row) and the block of a (head,
// sequence, row tile) that arrives last combines them, in split order.  The hand-over needs no device-scope
// fence (see gemm_w16_kernel): write-through stores, a wait for their completion, an agent-scope counter,
// and loads that bypass the reader's L2.  `cnt` holds one counter per (sequence slot, head, row-tile half),
// zero between launches.
// QL = 2: the query operand is used as hi + lo (target model), 1: hi only.  NW waves per block.
// seqs: the launch's sequences in grid order (longest first), one 32-byte entry per block to read.
// What bounds it: with few pairs a chain of memory and dependency latencies, with many the vector units' softmax beside the
// cache stream.  Scores are kept in units of log2, so a probability is one v_exp_f32 (with expf: 16 instructions): 12 heads,
// 530 keys 6.5 -> 5.4 us; 512 prompt rows, 32 heads 50 -> 43 us.  A second row tile without rows is skipped.
// A wave that is alone on its SIMD takes 2.4 to 3.7 ns per instruction, hence: arguments in registers and one table entry to
// read, masks only in groups that need them, the scale inside the exponent's fma, exchanges between the 16-lane groups as
// vector instructions, sums of a row kept per lane until the end, no rescaling while no maximum moves: 12 heads, 530 keys
// 5.4 -> 4.4 us, 13 rows 200 keys 4.6 -> 3.9, 512 prompt rows of 12 heads over up to 4000 keys 15.7 -> 12.8.
struct AttnSeq { int seq, slot, row0, n_rows, pos0, pad[3]; };
struct AttnSeqs { AttnSeq s[PK_MAXB]; };
template <int HD, int MT, int QL, int NW>
__global__ __launch_bounds__(NW * 64, NW == 16 ? 4 : HD == 128 ? (MT == 2 ? 2 : 3) : (MT == 2 ? 3 : 4)) void attn_mfma_kernel(
    const _Float16* __restrict__ qp, const _Float16* __restrict__ kv, int layer, int n_layers, int max_seq, int d, int kps, int H, int rt_split, int S,
    _Float16* __restrict__ xp_out, int MT_total_out, float* __restrict__ part, unsigned* __restrict__ cnt, const AttnSeqs seqs) {
  constexpr int KTS = HD / 32, DTS = HD / 16;
  __shared__ unsigned arrived;
  extern __shared__ __align__(16) float att_state[];   // [NW waves][live rows][HD + 4]: values, running max, running sum
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, g = lane >> 4, j = lane & 15;
  // rt_split (MT == 1 launches only): two blocks per key range, one per 16-row tile of the sequence
  const int rt = rt_split ? (int)(blockIdx.x & 1) : 0;
  const int split = rt_split ? (int)(blockIdx.x >> 1) : (int)blockIdx.x, h = blockIdx.y;
  const AttnSeq sq = seqs.s[blockIdx.z];
  const int si = sq.slot, r0 = sq.row0 + rt * 16, pos0 = sq.pos0;
  const int n_keys = pos0 + sq.n_rows;
  const int Rs = sq.n_rows - rt * 16;                    // rows from this block's first one to the sequence's last
  const int n_split = S == 1 ? 1 : (n_keys + kps - 1) / kps;
  const int ks_begin = split * kps, ks_end = min(n_keys, ks_begin + kps);
  if (ks_begin >= n_keys || Rs <= 0) return;
  const _Float16* Kc = kv + (((size_t)sq.seq * n_layers + layer) * 2) * (size_t)max_seq * d + (size_t)h * HD * max_seq;
  const _Float16* Vt = Kc + (size_t)max_seq * d;
  // scores in units of log2: the softmax then takes the hardware's 2^x as it is
  const float scale = 1.4426950408889634f / sqrtf((float)HD);
  const int mts = MT == 2 && Rs > 16 ? 2 : 1;          // row tiles that have rows (uniform)

  half8 q[KTS][MT][QL];
#pragma unroll
  for (int kt = 0; kt < KTS; ++kt)
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int pq = 0; pq < QL; ++pq)
        q[kt][mt][pq] = *reinterpret_cast<const half8*>(qp + (((((size_t)si * H + h) * KTS + kt) * 2 + rt + mt) * 2 + pq) * 512 + lane * 8);
  f32x4 acc[DTS][MT];
  float mrun[MT], lrun[MT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    mrun[mt] = -INFINITY;
    lrun[mt] = 0.f;
#pragma unroll
    for (int dt = 0; dt < DTS; ++dt) acc[dt][mt] = f32x4{0.f, 0.f, 0.f, 0.f};
  }

  // One 32-key group = two 16-key K tiles x KTS feature groups, and DTS fragments of V^T.  K and V each have
  // one register set; a set is refilled for the wave's next group as soon as its last product was issued
  // (K after the scores, V after the values), so each load has half a step of this wave's arithmetic, and
  // the other waves, to hide behind.  The loop has no branches and the loads keep their program order
  // (sched_barrier): a wait for K then leaves the V loads in flight and vice versa.  The step after the
  // wave's last one re-reads the last group (cache hits, unused).
  // Cache slots of positions not written yet hold zeros or old finite values (the cache is cleared when it is
  // bound), so their zero probabilities contribute nothing.
  auto load_k = [&](int kk, half8(&ka)[2][KTS]) {
    const _Float16* kt0 = Kc + (size_t)(kk >> 4) * (KTS * 512) + lane * 8;
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int kt = 0; kt < KTS; ++kt) ka[t][kt] = *reinterpret_cast<const half8*>(kt0 + (t * KTS + kt) * 512);
  };
  auto load_v = [&](int kk, half8(&va)[DTS]) {
    const _Float16* vg = Vt + (size_t)(kk >> 5) * (DTS * 512) + lane * 8;
#pragma unroll
    for (int dt = 0; dt < DTS; ++dt) va[dt] = *reinterpret_cast<const half8*>(vg + dt * 512);
  };
  // scores of one group for row tile mt -> probabilities (f16, in the lane layout the value product wants
  // for B) and the rescale factor of the running state.  mrun holds the maximum of the products themselves (the scale is
  // positive and goes into the exponent's fma); lrun is this lane's part of the row's sum, added up over the groups at the end.
  auto scores = [&](int kk, int mt, half8(&ka)[2][KTS], half8& pb, float& corr) {
    f32x4 st[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      f32x4 sacc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int kt = 0; kt < KTS; ++kt)
#pragma unroll
        for (int pq = 0; pq < QL; ++pq) sacc = __builtin_amdgcn_mfma_f32_16x16x32_f16(ka[t][kt], q[kt][mt][pq], sacc, 0, 0, 0);
      st[t] = sacc;
    }
    if (kk + 31 > pos0) {                                // uniform: keys that some row of the sequence does not see
      const int lk = min(pos0 + (rt + mt) * 16 + j, n_keys - 1) - kk - 4 * g;   // the last one that this lane's row sees
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) st[t][r] = 16 * t + r <= lk ? st[t][r] : -INFINITY;
    }
    float mx = fmaxf(fmaxf(fmaxf(st[0][0], st[0][1]), fmaxf(st[0][2], st[0][3])), fmaxf(fmaxf(st[1][0], st[1][1]), fmaxf(st[1][2], st[1][3])));
    const float mn = fmaxf(mrun[mt], group_max(mx));
    const float ms = mn == -INFINITY ? 0.f : mn * scale;   // nothing seen yet: every exponent below is -inf
    float ps = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float pe = exp2_hw(fmaf(st[e >> 2][e & 3], scale, -ms));
      ps += pe;
      pb[e] = (_Float16)pe;
    }
    corr = exp2_hw(fmaf(mrun[mt], scale, -ms));
    lrun[mt] = lrun[mt] * corr + ps;
    mrun[mt] = mn;
  };
  {
    const int first = ks_begin + 32 * wave;
    const int G = first < ks_end ? (ks_end - first + 32 * NW - 1) / (32 * NW) : 0;
    auto values = [&](half8(&va)[DTS], half8(&pb)[MT], float(&corr)[MT]) {
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
        if (mt < mts) {
          if (__any(corr[mt] != 1.f)) {                  // a row's maximum has moved
#pragma unroll
            for (int dt = 0; dt < DTS; ++dt) acc[dt][mt] *= corr[mt];
          }
#pragma unroll
          for (int dt = 0; dt < DTS; ++dt) acc[dt][mt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(va[dt], pb[mt], acc[dt][mt], 0, 0, 0);
        }
    };
    auto key_of = [&](int gi) { return first + min(gi, G - 1) * (32 * NW); };
    if (G > 0) {
      half8 ka[2][KTS], va[DTS];
      __builtin_amdgcn_sched_barrier(0);
      load_k(first, ka);
      __builtin_amdgcn_sched_barrier(0);
      load_v(first, va);
      __builtin_amdgcn_sched_barrier(0);
      for (int gi = 0; gi < G; ++gi) {
        const int kk = key_of(gi), kn = key_of(gi + 1);
        half8 pb[MT];
        float corr[MT];
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
          if (mt < mts) scores(kk, mt, ka, pb[mt], corr[mt]);
        __builtin_amdgcn_sched_barrier(0);
        load_k(kn, ka);
        __builtin_amdgcn_sched_barrier(0);
        values(va, pb, corr);
        __builtin_amdgcn_sched_barrier(0);
        load_v(kn, va);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    mrun[mt] *= scale;
    lrun[mt] = group_sum(lrun[mt]);
  }

  // Merge of the wave states: every wave writes its live rows (values, running max, running sum) to LDS
  // once, then each thread combines the states of one (row, 4 dims) group and writes the result.  One
  // barrier (a pairwise tree over the MFMA tiles took six per row tile and 1.4 to 4 us).
  const int rcap = min(Rs, MT * 16);
  float* st = att_state;
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    const int rl = mt * 16 + j;
    if (rl < rcap) {
      float* o = st + (size_t)(wave * rcap + rl) * (HD + 4);
#pragma unroll
      for (int dt = 0; dt < DTS; ++dt) *reinterpret_cast<f32x4*>(o + dt * 16 + 4 * g) = acc[dt][mt];
      if (g == 0) { o[HD] = mrun[mt]; o[HD + 1] = lrun[mt]; }
    }
  }
  __syncthreads();
  for (int o4 = threadIdx.x; o4 < rcap * (HD / 4); o4 += NW * 64) {
    const int rl = o4 / (HD / 4), d4 = (o4 % (HD / 4)) * 4;
    const float* p = st + (size_t)rl * (HD + 4);
    float M = -INFINITY;
#pragma unroll
    for (int w = 0; w < NW; ++w) M = fmaxf(M, p[(size_t)w * rcap * (HD + 4) + HD]);
    float L = 0.f;
    f32x4 a = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const float* pw = p + (size_t)w * rcap * (HD + 4);
      const float m = pw[HD];
      const float wt = (m == -INFINITY) ? 0.f : exp2_hw(m - M);
      L += pw[HD + 1] * wt;
      a += *reinterpret_cast<const f32x4*>(pw + d4) * wt;
    }
    if (n_split == 1) {
      const float inv = 1.0f / L;
      store_packed4(packed_at(xp_out, MT_total_out, r0 + rl, h * HD + d4), a[0] * inv, a[1] * inv, a[2] * inv, a[3] * inv);
    } else {
      // several splits: un-normalised partial (values, running max, running sum), written through to memory
      u64* o = reinterpret_cast<u64*>(part + (((size_t)(r0 + rl) * H + h) * S + split) * (HD + 2));
      const float2 a01 = {a[0], a[1]}, a23 = {a[2], a[3]}, ml = {M, L};
      __hip_atomic_store(o + d4 / 2, __builtin_bit_cast(u64, a01), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(o + d4 / 2 + 1, __builtin_bit_cast(u64, a23), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (d4 == 0) __hip_atomic_store(o + HD / 2, __builtin_bit_cast(u64, ml), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
  if (n_split == 1) return;
  PACER_WAIT_VMCNT0();   // this wave's write-through stores have completed
  __syncthreads();
  unsigned* my_cnt = cnt + ((size_t)si * H + h) * 2 + rt;
  if (threadIdx.x == 0) arrived = __hip_atomic_fetch_add(my_cnt, 1u, PACER_HO_ORDER, __HIP_MEMORY_SCOPE_AGENT);
  __syncthreads();
  if (arrived != (unsigned)(n_split - 1)) return;
  if (threadIdx.x == 0) __hip_atomic_store(my_cnt, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  // last block of this (sequence, head, row tile): combine the splits, eight at a time (all loads of a
  // batch are issued before the first is used; a split past the last repeats it and is skipped)
  for (int o4 = threadIdx.x; o4 < rcap * (HD / 4); o4 += NW * 64) {
    const int rl = o4 / (HD / 4), d4 = (o4 % (HD / 4)) * 4;
    const u64* p = reinterpret_cast<const u64*>(part + ((size_t)(r0 + rl) * H + h) * S * (HD + 2));
    float M = -INFINITY, L = 0.f;
    f32x4 a = {0.f, 0.f, 0.f, 0.f};
    for (int c0 = 0; c0 < n_split; c0 += 8) {
      u64 ml[8], v01[8], v23[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const u64* pc = p + (size_t)min(c0 + i, n_split - 1) * (HD / 2 + 1);
        ml[i] = __hip_atomic_load(pc + HD / 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        v01[i] = __hip_atomic_load(pc + d4 / 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        v23[i] = __hip_atomic_load(pc + d4 / 2 + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
      float Mb = M;
#pragma unroll
      for (int i = 0; i < 8; ++i)
        if (c0 + i < n_split) Mb = fmaxf(Mb, __builtin_bit_cast(float2, ml[i]).x);
      const float keep = (M == -INFINITY) ? 0.f : exp2_hw(M - Mb);
      L *= keep;
      a *= keep;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const float2 mli = __builtin_bit_cast(float2, ml[i]);
        const float w = (c0 + i < n_split && mli.x != -INFINITY) ? exp2_hw(mli.x - Mb) : 0.f;
        const float2 x01 = __builtin_bit_cast(float2, v01[i]), x23 = __builtin_bit_cast(float2, v23[i]);
        L += mli.y * w;
        a[0] += x01.x * w; a[1] += x01.y * w; a[2] += x23.x * w; a[3] += x23.y * w;
      }
      M = Mb;
    }
    const float inv = 1.0f / L;
    store_packed4(packed_at(xp_out, MT_total_out, r0 + rl, h * HD + d4), a[0] * inv, a[1] * inv, a[2] * inv, a[3] * inv);
  }
}

// ------------------------------------------------------------------ tail of a draft forward
// one block per listed sequence: hidden state h = x * g_final * row_scale into the ring, and the token
// = best of the per-tile candidates the LM-head GEMM left.  The block goes on to what the next draft
// step would start with, the embedding of the token it has just chosen (row si of next.x, operand, sums of
// squares): a launch less per draft step.  The host skips its embedding launch only if that step really comes next.
__global__ __launch_bounds__(256) void draft_tail_kernel(const float* x, int ldx, const float* __restrict__ g, const u64* ssq,
                                  int ssq_stride, float inv_dim, float eps, int d, float* __restrict__ hidden, const float* __restrict__ pick_val,
                                  const int* __restrict__ pick_idx, int pick_tiles, int* __restrict__ draft_tok, PickArgs pa, int G1,
                                  const uint16_t* __restrict__ E, EmbedOut next, int V, int* host_bad) {
  __shared__ float redv[16];
  __shared__ int redi[16];
  __shared__ float red[16];
  const int si = blockIdx.x, s = pa.seq[si], j = pa.j[si];
  // every input is requested before anything is used: the kernel is a chain of memory round trips otherwise
  constexpr int XMAX = 8, CMAX = 16;                   // d <= 2048 and <= 4096 candidate tiles stay in registers
  float xv[XMAX], gv[XMAX], cv[CMAX];
  int ci[CMAX];
  const bool in_regs = d <= XMAX * (int)blockDim.x && pick_tiles <= CMAX * (int)blockDim.x;
  if (in_regs) {
#pragma unroll
    for (int u = 0; u < CMAX; ++u) {
      const int t = threadIdx.x + u * blockDim.x;
      cv[u] = t < pick_tiles ? pick_val[(size_t)si * pick_tiles + t] : -INFINITY;
      ci[u] = t < pick_tiles ? pick_idx[(size_t)si * pick_tiles + t] : 0x7fffffff;
    }
#pragma unroll
    for (int u = 0; u < XMAX; ++u) {
      const int k = threadIdx.x + u * blockDim.x;
      xv[u] = k < d ? x[(size_t)si * ldx + k] : 0.f;
      gv[u] = k < d ? g[k] : 0.f;
    }
  }
  const float rs = row_scale(ssq, ssq_stride, si, inv_dim, eps);
  float* ho = hidden + (size_t)(s * G1 + j) * d;
  float best = -INFINITY;
  int bi = 0x7fffffff;
  auto hidden_from_regs = [&] {
#pragma unroll
    for (int u = 0; u < XMAX; ++u) {
      const int k = threadIdx.x + u * blockDim.x;
      if (k < d) ho[k] = xv[u] * gv[u] * rs;
    }
  };
  if (in_regs) {
#pragma unroll
    for (int u = 0; u < CMAX; ++u)
      if (cv[u] > best || (cv[u] == best && ci[u] < bi)) { best = cv[u]; bi = ci[u]; }
  } else {
    for (int k = threadIdx.x; k < d; k += blockDim.x) ho[k] = x[(size_t)si * ldx + k] * g[k] * rs;
    for (int t = threadIdx.x; t < pick_tiles; t += blockDim.x) {
      const float v = pick_val[(size_t)si * pick_tiles + t];
      const int i = pick_idx[(size_t)si * pick_tiles + t];
      if (v > best || (v == best && i < bi)) { best = v; bi = i; }
    }
  }
  block_argmax(best, bi, redv, redi);       // (its barriers also separate the reads of x and ssq above from the writes below)
  bi = checked_token(bi, V, threadIdx.x == 0 ? host_bad : nullptr, s);   // candidates without a finite value leave the sentinel
  if (threadIdx.x == 0) draft_tok[s * G1 + j] = bi;
  // the hidden state while the chosen token's embedding is on its way
  embed_row_w16(E + (size_t)bi * d, d, si, next, red, true, [&] { if (in_regs) hidden_from_regs(); });
}

// pre-verification head on the un-normalised residual rows: z = (x*g*rs) . cls
// One wave per row of the block; every input of the wave (the row, the gain, both head rows, the row's sums of
// squares) is requested with 16-byte loads before the first is used: the kernel is one memory round trip, not a chain.
__global__ void mb_head_w16_kernel(const float* x, int ldx, const float* __restrict__ g, const u64* ssq,
                                   int ssq_stride, float inv_dim, float eps, const float* __restrict__ cls, int d, int b, HaltArgs ha,
                                   float* __restrict__ alpha, int* __restrict__ stop, int* __restrict__ host_stop,
                                   const uint16_t* __restrict__ E, const int* __restrict__ next_tok, EmbedOut next) {
  __shared__ float al[32];
  __shared__ float red[16];
  const int si = blockIdx.x, lane = threadIdx.x & 63, wv = threadIdx.x >> 6, nw = blockDim.x >> 6;
  constexpr int CH = 4;                                 // 16-byte chunks per lane held in registers: d <= 1024
  const int n4 = d >> 2;
  for (int jj = wv; jj < b; jj += nw) {
    const int r = si * b + jj;
    const float4* xr = reinterpret_cast<const float4*>(x + (size_t)r * ldx);
    const float4* g4 = reinterpret_cast<const float4*>(g);
    const float4* c0 = reinterpret_cast<const float4*>(cls);
    const float4* c1 = reinterpret_cast<const float4*>(cls + d);
    float z0 = 0.f, z1 = 0.f;
    u64 sq[SSQ_SUB];
#pragma unroll
    for (int i = 0; i < SSQ_SUB; ++i) sq[i] = ssq[(size_t)i * ssq_stride + r];
    if (n4 <= CH * 64) {
      float4 xv[CH], gv[CH], a0[CH], a1[CH];
#pragma unroll
      for (int u = 0; u < CH; ++u) {
        const int k = min(lane + 64 * u, n4 - 1);        // a chunk past the end repeats the last one and is not added
        xv[u] = xr[k]; gv[u] = g4[k]; a0[u] = c0[k]; a1[u] = c1[k];
      }
#pragma unroll
      for (int u = 0; u < CH; ++u) {
        if (lane + 64 * u < n4) {
          const float v0 = xv[u].x * gv[u].x, v1 = xv[u].y * gv[u].y, v2 = xv[u].z * gv[u].z, v3 = xv[u].w * gv[u].w;
          z0 += v0 * a0[u].x + v1 * a0[u].y + v2 * a0[u].z + v3 * a0[u].w;
          z1 += v0 * a1[u].x + v1 * a1[u].y + v2 * a1[u].z + v3 * a1[u].w;
        }
      }
    } else {
      for (int k = lane; k < n4; k += 64) {
        const float4 xv = xr[k], gv = g4[k], a0 = c0[k], a1 = c1[k];
        const float v0 = xv.x * gv.x, v1 = xv.y * gv.y, v2 = xv.z * gv.z, v3 = xv.w * gv.w;
        z0 += v0 * a0.x + v1 * a0.y + v2 * a0.z + v3 * a0.w;
        z1 += v0 * a1.x + v1 * a1.y + v2 * a1.z + v3 * a1.w;
      }
    }
    u64 t = 0;
#pragma unroll
    for (int i = 0; i < SSQ_SUB; ++i) t += sq[i];
    const float rs = 1.0f / sqrtf((float)t * SSQ_INV_SCALE * inv_dim + eps);
    z0 = wave_total(z0) * rs;
    z1 = wave_total(z1) * rs;
    if (lane == 0) al[jj] = 1.0f / (1.0f + expf(z0 - z1));
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int jj = 0; jj < b; ++jj) alpha[si * b + jj] = al[jj];
    const int st = ha.force[si] >= 0 ? ha.force[si] : halt_decision(al, b, ha.t[si], ha.rule);
    stop[si] = st;
    host_stop[ha.seq[si]] = ha.ticket[si] * 2 + st;
  }
  // E != null (single-sequence launches only: row 0 of next.x is one of the rows this block has just read): the
  // embedding of the newest draft token, which the next round's first draft step would start with if drafting goes on
  if (E) embed_row_w16(E + (size_t)next_tok[0] * d, d, 0, next, red, true, [] {});
}
