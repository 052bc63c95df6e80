// Device kernels of the Pacer hot path for gfx950 (CDNA4, wave64).
//
// Data layout conventions used by every kernel in this file
//   activations ........ f32 [rows][width], row major
//   packed activations . (bf16 models) f16 operand tiles for the MFMA GEMM: tile (kt, mt) holds rows
//                        mt*16..+15 and features kt*32..+31 as 16 columns of 64 bytes: row j's 32
//                        features are contiguous, MFMA lane 16*g + j reads bytes 64*j + 16*g..+15.
//                        Rows are what a launch has few of, so a GEMM wave fetches only the 64-byte
//                        columns of live rows: operand traffic is proportional to the row count.
//   packed weights ..... the model's bf16 values stored as IEEE f16 (same bytes; the matrix units take
//                        f16 pairs with f16 activations, and converting while packing instead of in
//                        every GEMM frees three vector instructions per weight pair; bf16 -> f16 is
//                        exact down to 2^-17): tile (nt, kt) holds outputs nt*16..+15 and inputs kt*32..+31 in MFMA
//                        lane order (lane 16*g + i = output i, inputs 8*g..+7), tiles ordered
//                        [nt][kt], so a wave that walks along K for one output tile reads one
//                        contiguous stream with one 1 KiB load per step.
//   KV cache ........... f32 models: [seq][layer][K|V][position][d_model].  bf16 models: IEEE f16
//                        (same bytes as bf16, 3 more mantissa bits: K after RoPE and V are O(1)
//                        quantities, so range is no concern and rounding is what matters), in the
//                        per-head tile order given in kernels_w16.h
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half2v __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// The cross-block hand-overs rest on gfx950 behaviour (see "KSB" at gemm_w16_kernel) and on the encoding of
// s_waitcnt for that target: refuse to build device code for anything else.
#if defined(__HIP_DEVICE_COMPILE__) && !defined(__gfx950__)
#error "these kernels are written for gfx950 (MI355X): the fence-free hand-over and the s_waitcnt immediates are specific to it"
#endif
// Memory order of the arrival-counter increment of those hand-overs.  Relaxed by default: ordering comes from the
// write-through stores having completed (vmcnt 0) before the block's barrier, and from loads that do not hit in L2.
// Building with -DPACER_FENCED_HANDOVER makes the increment an agent-scope acquire-release (L2 write-back before it,
// invalidation after it, 4 to 15 us per launch): the variant to compare with if results ever differ between runs.
#ifdef PACER_FENCED_HANDOVER
#define PACER_HO_ORDER __ATOMIC_ACQ_REL
#else
#define PACER_HO_ORDER __ATOMIC_RELAXED
#endif
#define PACER_WAIT_VMCNT0() __builtin_amdgcn_s_waitcnt(0x0F70)   // gfx9 encoding: vmcnt = 0, expcnt and lgkmcnt at their maxima (no wait)

#define PK_MAXB 16

// Rows of a launch: sequence si (slot in the call's list) owns rows row_off[si]..row_off[si+1]-1
// at consecutive absolute positions starting at pos0[si]; len[si] = committed tokens.
struct SeqRows {
  int n_seqs;
  int seq[PK_MAXB];
  int row_off[PK_MAXB + 1];
  int pos0[PK_MAXB];
  int len[PK_MAXB];
};

__device__ __forceinline__ int find_seq(const SeqRows& sr, int r) {
  int s = 0;
  while (s + 1 < sr.n_seqs && sr.row_off[s + 1] <= r) ++s;
  return s;
}

// The sequence of row r with what the launch says about it.  Every table read has the same index in all lanes (scalar
// loads that do not wait for each other), where find_seq followed by look-ups is a chain of vector loads per lane.  A launch
// of one sequence reads only the first entries (all sixteen cost the streamed QKV launches 0.3 us each).
struct SeqOf { int si, seq, row0, pos0, len; };
__device__ __forceinline__ SeqOf seq_of_row(const SeqRows& sr, int r) {
  SeqOf o{0, sr.seq[0], sr.row_off[0], sr.pos0[0], sr.len[0]};
  if (sr.n_seqs > 1) {
#pragma unroll
    for (int s = 1; s < PK_MAXB; ++s) {
      const bool in = s < sr.n_seqs && sr.row_off[s] <= r;
      o.si = in ? s : o.si;
      o.seq = in ? sr.seq[s] : o.seq;
      o.row0 = in ? sr.row_off[s] : o.row0;
      o.pos0 = in ? sr.pos0[s] : o.pos0;
      o.len = in ? sr.len[s] : o.len;
    }
  }
  return o;
}

__device__ __forceinline__ float bf16_to_f32(uint16_t h) { return __uint_as_float(((uint32_t)h) << 16); }

template <typename T> __device__ __forceinline__ float ld_f32(const T* p);
template <> __device__ __forceinline__ float ld_f32<float>(const float* p) { return *p; }
template <> __device__ __forceinline__ float ld_f32<uint16_t>(const uint16_t* p) { return bf16_to_f32(*p); }
// A wave's exchange without a trip to LDS: v of another lane of the same 16 (DPP), and the two swaps between 16-lane groups.
template <int CTRL> __device__ __forceinline__ float dpp_f32(float v) {
  return __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(v), CTRL, 0xf, 0xf, true));
}
// over the four 16-lane groups of a wave, same lane of each
__device__ __forceinline__ float group_max(float v) {
  const unsigned u = __float_as_uint(v);
  const auto a = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  const unsigned w = __float_as_uint(fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1])));
  const auto b = __builtin_amdgcn_permlane32_swap(w, w, false, false);
  return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ __forceinline__ float group_sum(float v) {
  const unsigned u = __float_as_uint(v);
  const auto a = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  const unsigned w = __float_as_uint(__uint_as_float(a[0]) + __uint_as_float(a[1]));
  const auto b = __builtin_amdgcn_permlane32_swap(w, w, false, false);
  return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}
// over 16 lanes: quad_perm [1,0,3,2] and [2,3,0,1], row_half_mirror, row_mirror
__device__ __forceinline__ float row16_sum(float v) {
  v += dpp_f32<0xB1>(v);
  v += dpp_f32<0x4E>(v);
  v += dpp_f32<0x141>(v);
  v += dpp_f32<0x140>(v);
  return v;
}
__device__ __forceinline__ float wave_total(float v) { return group_sum(row16_sum(v)); }
__device__ __forceinline__ float wave_largest(float v) {
  v = fmaxf(v, dpp_f32<0xB1>(v));
  v = fmaxf(v, dpp_f32<0x4E>(v));
  v = fmaxf(v, dpp_f32<0x141>(v));
  v = fmaxf(v, dpp_f32<0x140>(v));
  return group_max(v);
}
template <int CTRL> __device__ __forceinline__ unsigned min_dpp(unsigned v) {
  return min(v, (unsigned)__builtin_amdgcn_update_dpp(0, v, CTRL, 0xf, 0xf, true));
}
__device__ __forceinline__ unsigned wave_least(unsigned v) {
  v = min_dpp<0x140>(min_dpp<0x141>(min_dpp<0x4E>(min_dpp<0xB1>(v))));
  const auto a = __builtin_amdgcn_permlane16_swap(v, v, false, false);
  v = min(a[0], a[1]);
  const auto b = __builtin_amdgcn_permlane32_swap(v, v, false, false);
  return min(b[0], b[1]);
}
// best candidate of a wave: the largest value, the lowest id (not negative) among equal ones
__device__ __forceinline__ void wave_best(float& v, int& id) {
  const float m = wave_largest(v);
  id = (int)wave_least(v == m ? (unsigned)id : 0x7fffffffu);
  v = m;
}
// Block-wide sum in a fixed order (deterministic).  red: LDS scratch of >= 16 floats.
__device__ __forceinline__ float block_sum(float v, float* red) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
  v = wave_total(v);
  __syncthreads();
  if (lane == 0) red[w] = v;
  __syncthreads();
  float t = 0.f;
  for (int i = 0; i < nw; ++i) t += red[i];
  return t;
}
// Block-wide argmax; the lowest index wins among equal values.  Result valid in all threads.
__device__ __forceinline__ void block_argmax(float& v, int& idx, float* redv, int* redi) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
  wave_best(v, idx);
  __syncthreads();
  if (lane == 0) { redv[w] = v; redi[w] = idx; }
  __syncthreads();
  v = redv[0]; idx = redi[0];
  for (int i = 1; i < nw; ++i)
    if (redv[i] > v || (redv[i] == v && redi[i] < idx)) { v = redv[i]; idx = redi[i]; }
}

// ------------------------------------------------------------------ Philox-4x32-10
// Salmon et al., "Parallel random numbers: as easy as 1, 2, 3" (SC'11).
__device__ __forceinline__ uint4 philox4x32_10(uint4 c, uint32_t k0, uint32_t k1) {
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    const uint32_t hi0 = __umulhi(0xD2511F53u, c.x), lo0 = 0xD2511F53u * c.x;
    const uint32_t hi1 = __umulhi(0xCD9E8D57u, c.z), lo1 = 0xCD9E8D57u * c.z;
    c = make_uint4(hi1 ^ c.y ^ k0, lo1, hi0 ^ c.w ^ k1, lo0);
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
  }
  return c;
}
// uniform in (0,1), exactly representable in f32: ((bits >> 9) + 0.5) * 2^-23
__device__ __forceinline__ float u01(uint32_t bits) { return ((float)(bits >> 9) + 0.5f) * 1.1920928955078125e-07f; }
__device__ __forceinline__ float gumbel(float u) { return -logf(-logf(u)); }
#define PURPOSE_DRAFT 0u
#define PURPOSE_ACCEPT 1u
#define PURPOSE_NEXT 2u
// four uniforms for vocabulary ids 4*blk..4*blk+3
__device__ __forceinline__ uint4 vocab_bits(uint64_t seed, int seq, uint32_t step, uint32_t row, uint32_t purpose, uint32_t blk) {
  return philox4x32_10(make_uint4(blk, row, step, purpose | ((uint32_t)seq << 8)), (uint32_t)seed, (uint32_t)(seed >> 32));
}

// ------------------------------------------------------------------ token ids as table indices
// A token id that is about to be stored, or used as an index, is checked against the vocabulary first.  An argmax
// over logits that held no finite value leaves the sentinel 0x7fffffff, and a caller may hand in anything: such an
// id is replaced by the nearest valid one, so that no later load leaves its table, and the sequence's word in
// pinned host memory (host_bad, may be null) is set, which the host turns into an error at its next read-back.
__device__ __forceinline__ int checked_token(int tok, int V, int* host_bad, int seq) {
  if ((unsigned)tok < (unsigned)V) return tok;
  if (host_bad) {
    host_bad[seq] = 1;
    __threadfence_system();
  }
  return tok < 0 ? 0 : V - 1;
}
// prompt tokens into the sequence's token buffer
__global__ void copy_tokens_kernel(int* __restrict__ dst, const int* __restrict__ src, int n, int V, int* host_bad, int seq) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) dst[i] = checked_token(src[i], V, host_bad, seq);
}

// ------------------------------------------------------------------ embedding gather
// token of (sequence, position): committed token below len, else the draft made at that position
template <typename T>
__global__ void embed_rows_kernel(const T* __restrict__ E, const int* __restrict__ tokens, const int* __restrict__ draft_tok,
                                  SeqRows sr, int max_seq, int G1, int d, float* __restrict__ x, int ldx) {
  const int r = blockIdx.x;
  const int si = find_seq(sr, r);
  const int s = sr.seq[si];
  const int p = sr.pos0[si] + (r - sr.row_off[si]);
  const int tok = p < sr.len[si] ? tokens[(size_t)s * max_seq + p] : draft_tok[s * G1 + (p - sr.len[si])];
  const T* e = E + (size_t)tok * d;
  for (int k = threadIdx.x; k < d; k += blockDim.x) x[(size_t)r * ldx + k] = ld_f32<T>(e + k);
}

// input rows of the pre-verification layer: hidden + PosEmb[e] (e = 0 for prefix rows)
struct MbRows { int src_row0[PK_MAXB]; int e0[PK_MAXB]; };
__global__ void mb_input_kernel(const float* __restrict__ src, int lds, const float* __restrict__ posemb, SeqRows sr, MbRows mr,
                                int d, float* __restrict__ x, int ldx) {
  const int r = blockIdx.x;
  const int si = find_seq(sr, r);
  const int rr = r - sr.row_off[si];
  const float* h = src + (size_t)(mr.src_row0[si] + rr) * lds;
  const float* e = posemb + (size_t)(mr.e0[si] < 0 ? 0 : mr.e0[si] + rr) * d;
  for (int k = threadIdx.x; k < d; k += blockDim.x) x[(size_t)r * ldx + k] = h[k] + e[k];
}

// ------------------------------------------------------------------ f32 path: norm and activation
// RMSNorm of rows (one block each): the draft's hidden states of a prompt, which M_B's prefix rows start from
__global__ void rmsnorm_rows_kernel(const float* __restrict__ x, int ldx, const float* __restrict__ g, float eps, int d, float* __restrict__ out, int ldo) {
  __shared__ float red[16];
  const float* xr = x + (size_t)blockIdx.x * ldx;
  float ss = 0.f;
  for (int k = threadIdx.x; k < d; k += blockDim.x) { const float v = xr[k]; ss += v * v; }
  ss = block_sum(ss, red);
  const float inv = 1.0f / sqrtf(ss / (float)d + eps);
  for (int k = threadIdx.x; k < d; k += blockDim.x) out[(size_t)blockIdx.x * ldo + k] = xr[k] * inv * g[k];
}

// ------------------------------------------------------------------ output row mapping of a GEMM
#define ROWMAP_ID 0      // out row = r
#define ROWMAP_RING 1    // out row = seq*G1 + draft index      (draft logits ring)
#define ROWMAP_LIST 2    // out row = slot*G1 + row within seq  (verify logits)
// bf16 -> f16 of 8 weights (exact for |w| >= 2^-17; smaller ones round to the nearest f16 subnormal,
// absolute error <= 2^-25).  Done once, when a matrix is packed.
__device__ __forceinline__ u32x4 bf16x8_to_f16x8(u32x4 w) {
  half8 h;
  const uint32_t u[4] = {w[0], w[1], w[2], w[3]};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float lo = __uint_as_float(u[i] << 16), hi = __uint_as_float(u[i] & 0xffff0000u);
    h[2 * i] = (_Float16)lo;
    h[2 * i + 1] = (_Float16)hi;
  }
  return __builtin_bit_cast(u32x4, h);
}

// ------------------------------------------------------------------ f32 models: GEMMs with fused norm and epilogue
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_of(const void* p, int bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, bytes, 0x00020000);
}

#define F32_QKV 0      // norm; rotation, q rows out, K and V rows into the cache
#define F32_RESID 1    // out += the product
#define F32_SWIGLU 2   // norm; silu(gate) * up
#define F32_LOGITS 3   // norm; logits, and the normalised rows for the hidden-state ring
struct F32Args {
  float eps;
  int rowmap, G1;
  const float* rope;                     // [max_seq][32][2] cos, sin by absolute position
  float* kv;
  int layer, n_layers, max_seq, d;
  float* hid_out;                        // LOGITS: may be null; one block per row behind the output's blocks
  SeqRows sr;
};
// One wave per output, or per pair of outputs that the epilogue needs together (a rotation pair, gate and up, two logits), for
// RG rows at a time; 4 waves per block.  The launch is a chain of latencies over a few hundred KiB, and what counts is what is
// not in it: the norm costs no launch of its own (a wave that reads a row adds its squares up on the way), nor do rotation,
// cache append and SwiGLU.  16-byte loads through descriptors that end with the row: a K that is not a multiple of 256 reads
// zeros.  The arguments that the first loads need come first, in registers; the others are read in one go while those travel.
// n_waves: waves with work.  extra: 1 = K and V only (QKV); the number of outputs (LOGITS).  Tiny pair (d 256,
// FFN 688, 4 layers), two draft steps, their pre-verification and verification: 88 launches and 285 us of kernels with norm,
// rotation and SwiGLU as kernels of their own, now 45 and 141.
template <int RG, int U, int EPI>
__global__ __launch_bounds__(256) void gemm_f32_kernel(const float* W, const float* X, int K, int ldx, int R, int ldo, float* out, const float* gain,
                                                       int n_waves, int extra, const F32Args a) {
  constexpr bool NORM = EPI != F32_RESID, PAIR = EPI != F32_RESID;
  const int lane = threadIdx.x & 63;
  const int out_blocks = (n_waves + 3) >> 2;
  if (EPI == F32_LOGITS && (int)blockIdx.x >= out_blocks) {            // hidden state of one row
    __shared__ float red[16];
    const int r = blockIdx.x - out_blocks, si = find_seq(a.sr, r);
    const float* xr = X + (size_t)r * ldx;
    float ss = 0.f;
    for (int k = threadIdx.x; k < K; k += 256) ss += xr[k] * xr[k];
    const float inv = 1.0f / sqrtf(block_sum(ss, red) / (float)K + a.eps);
    const int j = a.sr.pos0[si] + (r - a.sr.row_off[si]) - (a.sr.len[si] - 1);
    float* ho = a.hid_out + (size_t)(a.sr.seq[si] * a.G1 + j) * K;
    for (int k = threadIdx.x; k < K; k += 256) ho[k] = xr[k] * inv * gain[k];
    return;
  }
  const int n = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + (threadIdx.x >> 6));
  const int part = EPI == F32_QKV ? extra + (int)blockIdx.y : 0;       // Q, K, V: K rows of W each (d outputs of d inputs)
  if (n >= n_waves) return;
  // the wave's two rows of W: dims j and j + 32 of a head (QKV), gate and up, two neighbours
  const int ca = EPI == F32_QKV ? (n >> 5) * 64 + (n & 31) : EPI == F32_LOGITS ? 2 * n : n;
  const int cb = EPI == F32_QKV ? ca + 32 : EPI == F32_LOGITS ? min(ca + 1, extra - 1) : n_waves + n;
  const auto wa = buffer_of(W + (size_t)(part * K + ca) * K, K * 4), wb = buffer_of(W + (size_t)(part * K + (PAIR ? cb : ca)) * K, K * 4);
  const auto gr = buffer_of(gain, K * 4);
  for (int r0 = 0; r0 < R; r0 += RG) {
    float sa[RG], sb[RG], ss[RG];
#pragma unroll
    for (int i = 0; i < RG; ++i) sa[i] = sb[i] = ss[i] = 0.f;
    // what lane i needs for row r0 + i, requested beside the first products
    const int r = r0 + lane;
    const bool mine = lane < RG && r < R;
    float old = 0.f, cs = 1.f, sn = 0.f;
    float* dst = nullptr;
    for (int k0 = 0; k0 < K; k0 += 256 * U) {
      float4 va[U], vb[U], vg[U], vx[U][RG];
      auto ld = [](__amdgpu_buffer_rsrc_t b, int off) { return __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(b, off, 0, 0)); };
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int off = (k0 + u * 256) * 4 + lane * 16;
        va[u] = ld(wa, off);
        if (PAIR) vb[u] = ld(wb, off);
        if (NORM) vg[u] = ld(gr, off);
#pragma unroll
        for (int i = 0; i < RG; ++i) vx[u][i] = ld(buffer_of(X + (size_t)min(r0 + i, R - 1) * ldx, K * 4), off);   // a row past the last repeats it
      }
      if (k0 == 0) {
        if (EPI == F32_QKV || EPI == F32_LOGITS) asm volatile("" ::"s"(a.sr.n_seqs), "s"(a.sr.seq[0]), "s"(a.sr.row_off[0]), "s"(a.sr.pos0[0]));
        if (EPI == F32_QKV) asm volatile("" ::"s"(a.rope), "s"(a.kv), "s"(a.layer), "s"(a.n_layers), "s"(a.max_seq), "s"(a.d), "s"(a.eps));
        if (EPI == F32_LOGITS) asm volatile("" ::"s"(a.rowmap), "s"(a.G1), "s"(a.sr.len[0]), "s"(a.eps));
      }
      if (k0 == 0 && mine) {
        if (EPI == F32_RESID) {
          dst = out + (size_t)r * ldo + ca;
          old = *dst;
        } else if (EPI == F32_SWIGLU) {
          dst = out + (size_t)r * ldo + ca;
        } else {
          const SeqOf q = seq_of_row(a.sr, r);
          const int pos = q.pos0 + r - q.row0;
          if (EPI == F32_QKV) {
            const int j = n & 31;
            if (part < 2) {
              cs = a.rope[((size_t)pos * 32 + j) * 2];
              sn = a.rope[((size_t)pos * 32 + j) * 2 + 1];
            }
            dst = part == 0 ? out + (size_t)r * ldo + ca
                            : a.kv + ((((size_t)q.seq * a.n_layers + a.layer) * 2 + (part - 1)) * (size_t)a.max_seq + pos) * a.d + ca;
          } else {
            const int row = a.rowmap == ROWMAP_LIST ? q.si * a.G1 + (r - q.row0) : q.seq * a.G1 + (pos - (q.len - 1));
            dst = out + (size_t)row * ldo + ca;
          }
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int i = 0; i < RG; ++i) {
          const float4 x = vx[u][i];
          float4 t = x;
          if (NORM) {
            t = make_float4(x.x * vg[u].x, x.y * vg[u].y, x.z * vg[u].z, x.w * vg[u].w);
            ss[i] += x.x * x.x + x.y * x.y + x.z * x.z + x.w * x.w;
          }
          sa[i] += va[u].x * t.x + va[u].y * t.y + va[u].z * t.z + va[u].w * t.w;
          if (PAIR) sb[i] += vb[u].x * t.x + vb[u].y * t.y + vb[u].z * t.z + vb[u].w * t.w;
        }
    }
    // lane i takes row r0 + i
    float va = 0.f, vb = 0.f, vs = 0.f;
#pragma unroll
    for (int i = 0; i < RG; ++i) {
      const float ta = wave_total(sa[i]), tb = PAIR ? wave_total(sb[i]) : 0.f, ts = NORM ? wave_total(ss[i]) : 0.f;
      va = lane == i ? ta : va;
      vb = lane == i ? tb : vb;
      vs = lane == i ? ts : vs;
    }
    if (!mine) continue;
    const float inv = NORM ? 1.0f / sqrtf(vs / (float)K + a.eps) : 1.f;
    va *= inv;
    vb *= inv;
    if (EPI == F32_RESID) {
      *dst = old + va;
    } else if (EPI == F32_SWIGLU) {
      *dst = va / (1.0f + expf(-va)) * vb;
    } else if (EPI == F32_QKV) {
      dst[0] = va * cs - vb * sn;
      dst[32] = vb * cs + va * sn;
    } else {
      dst[0] = va;
      if (cb != ca) dst[1] = vb;
    }
  }
}

// ------------------------------------------------------------------ f32 models: attention over the KV cache
// grid (rows, heads); a block's NW waves take 32 keys each in turn, and their states meet in LDS (one barrier).  16 lanes hold
// a key's 64 dims, 4 each, so a load instruction covers 4 whole keys and a score is 4 products and 4 adds across the lanes;
// scores, probabilities and values stay in registers.  Latency bound: 3 rows and 35 keys took 4.9 us with keys and scores in
// LDS plus 2.8 us for a launch that combined key ranges, now 3.5.
struct F32Seqs { int n_seqs; int seq[PK_MAXB], row_off[PK_MAXB + 1], pos0[PK_MAXB]; };
__global__ __launch_bounds__(1024) void attn_f32_kernel(const float* q, const float* kv, int ldq, int layer, int n_layers, int max_seq, int d, int NW,
                                                        int ldo, float* out, const F32Seqs sq) {
  __shared__ float st[16][64 + 2];
  const int r = blockIdx.x, h = blockIdx.y, lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int g = lane >> 4, c = (lane & 15) * 4;
  int si = 0;
  while (si + 1 < sq.n_seqs && sq.row_off[si + 1] <= r) ++si;
  const int pos = sq.pos0[si] + r - sq.row_off[si];                   // the row sees keys 0..pos
  const float* K0 = kv + (((size_t)sq.seq[si] * n_layers + layer) * 2) * (size_t)max_seq * d + h * 64;
  const float4 q4 = *reinterpret_cast<const float4*>(q + (size_t)r * ldq + h * 64 + c);
  const float scale = 0.125f;                                         // 1 / sqrt(64)
  const float4 qs = make_float4(q4.x * scale, q4.y * scale, q4.z * scale, q4.w * scale);
  const int voff = (g * d + c) * 4;
  float m = -INFINITY, l = 0.f;
  float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int kk = wave * 32; kk <= pos; kk += NW * 32) {
    // these 32 keys; one past the row's last reads zeros
    const int bytes = (min(pos - kk, 31) * d + 64) * 4;
    const auto kb = buffer_of(K0 + (size_t)kk * d, bytes), vb = buffer_of(K0 + ((size_t)max_seq + kk) * d, bytes);
    float4 k4[8], v4[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) k4[e] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(kb, voff, 4 * e * d * 4, 0));
#pragma unroll
    for (int e = 0; e < 8; ++e) v4[e] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(vb, voff, 4 * e * d * 4, 0));
    float s[8], mx = -INFINITY;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float t = row16_sum(qs.x * k4[e].x + qs.y * k4[e].y + qs.z * k4[e].z + qs.w * k4[e].w);
      s[e] = kk + 4 * e + g <= pos ? t : -INFINITY;
      mx = fmaxf(mx, s[e]);
    }
    const float mn = fmaxf(m, group_max(mx));
    const float ms = mn == -INFINITY ? 0.f : mn;
    const float corr = expf(m - ms);
    float ps = 0.f;
    acc.x *= corr; acc.y *= corr; acc.z *= corr; acc.w *= corr;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float p = expf(s[e] - ms);
      ps += p;
      acc.x += p * v4[e].x; acc.y += p * v4[e].y; acc.z += p * v4[e].z; acc.w += p * v4[e].w;
    }
    l = l * corr + ps;
    m = mn;
  }
  l = group_sum(l);
  acc.x = group_sum(acc.x); acc.y = group_sum(acc.y); acc.z = group_sum(acc.z); acc.w = group_sum(acc.w);
  if (lane < 16) {
    st[wave][c] = acc.x; st[wave][c + 1] = acc.y; st[wave][c + 2] = acc.z; st[wave][c + 3] = acc.w;
    if (lane == 0) { st[wave][64] = m; st[wave][65] = l; }
  }
  __syncthreads();
  if (wave) return;
  float M = -INFINITY, L = 0.f, o = 0.f;                              // lane = dim
  for (int w = 0; w < NW; ++w) M = fmaxf(M, st[w][64]);
  for (int w = 0; w < NW; ++w) {
    const float f = st[w][64] == -INFINITY ? 0.f : expf(st[w][64] - M);
    L += st[w][65] * f;
    o += st[w][lane] * f;
  }
  out[(size_t)r * ldo + h * 64 + lane] = o / L;
}

// ------------------------------------------------------------------ token choice of the draft model
// one block per listed sequence: y = argmax(logits) or Gumbel-max sample; row j of the ring
struct PickArgs { int n_seqs; int seq[PK_MAXB]; int j[PK_MAXB]; };
__global__ __launch_bounds__(1024) void pick_token_kernel(const float* __restrict__ ring, int* __restrict__ draft_tok, PickArgs pa,
                                                          int G1, int V, int mode, uint64_t seed, uint32_t step, int* host_bad) {
  __shared__ float redv[16];
  __shared__ int redi[16];
  const int si = blockIdx.x, s = pa.seq[si], j = pa.j[si];
  const float* lg = ring + (size_t)(s * G1 + j) * V;
  float best = -INFINITY;
  int bi = 0x7fffffff;
  for (int blk = threadIdx.x; blk * 4 < V; blk += blockDim.x) {
    float g4[4] = {0.f, 0.f, 0.f, 0.f};
    if (mode) {
      const uint4 b = vocab_bits(seed, s, step, (uint32_t)(j + 1), PURPOSE_DRAFT, (uint32_t)blk);
      g4[0] = gumbel(u01(b.x)); g4[1] = gumbel(u01(b.y)); g4[2] = gumbel(u01(b.z)); g4[3] = gumbel(u01(b.w));
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int v = blk * 4 + e;
      if (v < V) {
        const float val = lg[v] + g4[e];
        if (val > best) { best = val; bi = v; }
      }
    }
  }
  block_argmax(best, bi, redv, redi);
  if (threadIdx.x == 0) draft_tok[s * G1 + j] = checked_token(bi, V, host_bad, s);
}

// ------------------------------------------------------------------ pre-verification head + halting test
// x: M_B's last residual rows, grouped per sequence (b rows each); their final norm is taken here.  alpha_j = softmax(z)[1]
// = 1/(1+exp(z0-z1)); stop = (mean alpha <= t) with the mean summed in index order in f32.
// rule: 0 mean, 1 any, 2 last.  seq/ticket: the stop flag also goes to pinned host memory as
// host_stop[seq] = ticket*2 + stop, which the host polls instead of synchronising the stream.
// force: -1 = decide by the rule; 0 / 1 = the flag is forced (test tap: sweeps over stop patterns), the kernel still
// computes and writes alpha
struct HaltArgs { int n_seqs; int rule; float t[PK_MAXB]; int seq[PK_MAXB]; int ticket[PK_MAXB]; int force[PK_MAXB]; };
// the halting test of one block, decided in f32 (al: the block's alpha values in index order)
__device__ __forceinline__ int halt_decision(const float* al, int b, float t, int rule) {
  if (rule == 1) {
    int any = 0;
    for (int j = 0; j < b; ++j) any |= (al[j] <= t) ? 1 : 0;
    return any;
  }
  if (rule == 2) return (al[b - 1] <= t) ? 1 : 0;
  float s = 0.f;
  for (int j = 0; j < b; ++j) s += al[j];
  return (s / (float)b <= t) ? 1 : 0;
}
__global__ void mb_head_kernel(const float* __restrict__ x, int ldx, const float* __restrict__ gain, float eps, const float* __restrict__ cls, int d,
                               int b, HaltArgs ha, float* __restrict__ alpha, int* __restrict__ stop, int* __restrict__ host_stop) {
  __shared__ float al[32];
  const int si = blockIdx.x, lane = threadIdx.x & 63, wv = threadIdx.x >> 6, nw = blockDim.x >> 6;
  for (int j = wv; j < b; j += nw) {
    const float* xr = x + (size_t)(si * b + j) * ldx;
    float z0 = 0.f, z1 = 0.f, ss = 0.f;
    for (int k = lane; k < d; k += 64) {
      const float v = xr[k], t = v * gain[k];
      ss += v * v;
      z0 += t * cls[k];
      z1 += t * cls[d + k];
    }
    const float inv = 1.0f / sqrtf(wave_total(ss) / (float)d + eps);
    z0 = wave_total(z0) * inv; z1 = wave_total(z1) * inv;
    if (lane == 0) al[j] = 1.0f / (1.0f + expf(z0 - z1));
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int j = 0; j < b; ++j) alpha[si * b + j] = al[j];
    const int st = ha.force[si] >= 0 ? ha.force[si] : halt_decision(al, b, ha.t[si], ha.rule);
    stop[si] = st;
    host_stop[ha.seq[si]] = ha.ticket[si] * 2 + st;
  }
}

// ------------------------------------------------------------------ acceptance (Eq. 5)
// slot: the sequence's index in the verify call that wrote the logits (row slot*G1 + i of tl, entry slot of the
// caller's n / z arrays).  The kernels run over the rows i < gamma (ACC_PHASE_DRAFTS: everything a step needs unless
// every draft is accepted), the bonus row i = gamma of the sequences that accepted all drafts (ACC_PHASE_BONUS), or all rows
// at once, the bonus row whether it is needed or not (ACC_PHASE_ALL: the caller already holds its draft logits).
// qslot: the sequence's block of G1 rows in the draft logits and draft token buffers (the sequence id for a context's
// rings); seq itself keys the random streams and indexes the committed tokens and the host words.
struct AccArgs { int n_seqs; int seq[PK_MAXB]; int slot[PK_MAXB]; int qslot[PK_MAXB]; int gamma[PK_MAXB]; int len[PK_MAXB]; float beta[PK_MAXB]; };

// One row of logits is split into ACC_CHUNKS vocabulary ranges, one block each (a single block per row
// spent 53 us walking 32000 entries three times).  Two launches:
//   sampling  accept_stats_kernel   per (row, chunk): running max and sum of exp of the effective target logits and
//                                   of the draft logits over the chunk
//             accept_pick_kernel    ACC_PICKERS blocks per sequence: every block takes the log-sum-exps and accept tests of all rows
//                                   from the statistics (a few KB), so that it knows the row where drafting is cut, and looks
//                                   for the best candidates of that row only, in its part of the vocabulary; whoever comes last finishes the sequence
//   greedy    accept_rows_kernel    per (row, chunk): best effective logit
//             accept_finalize_kernel per sequence: best over the chunks of each row, first rejection, tokens
// In a context rows i < gamma come first; the bonus row i = gamma (whose draft logits cost one more draft forward) only for
// the sequences that turn out to have accepted every draft.  pacer_accept_noalloc, whose caller holds them, evaluates it beside.
#define ACC_CHUNKS 16
#define ACC_PART 8      // floats per (row, chunk): [0..3] = mp, sp, mq, sq ; [4..7] = best, bi, bestp, bip
#define ACC_PICKERS 64  // blocks of a sequence that look for its candidates
#define ACC_MAXROWS 32  // rows of a sequence: the pick kernel takes them four per wave in one go

__device__ __forceinline__ void acc_chunk_range(int V, int chunk, int& v0, int& v1) {
  const int per = ((V + ACC_CHUNKS - 1) / ACC_CHUNKS + 3) & ~3;   // multiple of 4: a Philox block never straddles chunks
  v0 = min(V, chunk * per);
  v1 = min(V, v0 + per);
}

// (best, id) of a candidate and another one: the larger value, the lower id among equal values
__device__ __forceinline__ void take_better(float& v, int& id, float ov, int oid) {
  if (ov > v || (ov == v && oid < id)) { v = ov; id = oid; }
}

// Rows of a launch by phase: 0 rows i < gamma; 1 the bonus row i = gamma; 2 all of them (both logits buffers already hold
// the bonus row: one set of launches instead of two).  False: this block has no row.
#define ACC_PHASE_DRAFTS 0
#define ACC_PHASE_BONUS 1
#define ACC_PHASE_ALL 2
__device__ __forceinline__ bool acc_row(int phase, int gamma, int bx, int& i) {
  i = phase == ACC_PHASE_BONUS ? gamma : bx;
  return i < gamma || (i == gamma && phase != ACC_PHASE_DRAFTS);
}

// grid (rows, n_seqs, ACC_CHUNKS), 512 threads.  One pass: a thread keeps the running maximum of what it has seen and the sum
// of exp relative to it, four entries requested at a time (17 rows of 32000: two passes of dependent loads 8.3 us; 256 threads
// of eight entries and reductions through LDS 5.4; now 4.9).
__global__ __launch_bounds__(512) void accept_stats_kernel(const float* tl, const float* ring, float* part, int* arrivals, int G1, int V, int phase,
                                                           AccArgs aa) {
  constexpr int NWV = 8, U = 4;
  __shared__ float red[NWV][4];
  const int si = blockIdx.y, ch = blockIdx.z, sl = aa.slot[si];
  if (blockIdx.x == 0 && ch == 0 && threadIdx.x == 0) arrivals[sl * G1] = 0;   // of the pick kernel's blocks, the next launch
  int i;
  if (!acc_row(phase, aa.gamma[si], blockIdx.x, i)) return;
  const float beta = aa.beta[si];
  const float* t = tl + (size_t)(sl * G1 + i) * V;
  const float* q = ring + (size_t)(aa.qslot[si] * G1 + i) * V;
  int v0, v1;
  acc_chunk_range(V, ch, v0, v1);
  float m[2] = {-INFINITY, -INFINITY}, s[2] = {0.f, 0.f};              // [0] effective target, [1] draft
  // an entry of -inf adds nothing; a NaN makes the sum NaN (fmaxf ignores it)
  auto rel = [](float e, float mx) { return e == -INFINITY ? 0.f : expf(e - mx); };
  for (int base = v0 + threadIdx.x; base < v1; base += U * 512) {
    float e[2][U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int v = base + u * 512;
      e[0][u] = v < v1 ? t[v] : -INFINITY;
      e[1][u] = v < v1 ? q[v] : -INFINITY;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) e[0][u] = base + u * 512 < v1 ? e[0][u] + beta * e[1][u] : -INFINITY;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      float mn = m[k];
#pragma unroll
      for (int u = 0; u < U; ++u) mn = fmaxf(mn, e[k][u]);
      s[k] *= rel(m[k], mn);
#pragma unroll
      for (int u = 0; u < U; ++u) s[k] += rel(e[k][u], mn);
      m[k] = mn;
    }
  }
  // wave, then block (in wave order)
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const float mw = wave_largest(m[k]);
    s[k] = wave_total(s[k] * (m[k] == -INFINITY ? 1.f : expf(m[k] - mw)));   // nothing seen: s is 0, or NaN
    m[k] = mw;
  }
  if ((threadIdx.x & 63) == 0) {
    float* r = red[threadIdx.x >> 6];
    r[0] = m[0]; r[1] = s[0]; r[2] = m[1]; r[3] = s[1];
  }
  __syncthreads();
  if (threadIdx.x < 16) {                                // 8 lanes per statistic, one wave's each
    static_assert(NWV == 8, "");
    const int k = (threadIdx.x >> 3) * 2;
    const float mw = red[threadIdx.x & 7][k], sw = red[threadIdx.x & 7][k + 1];
    float mb = mw;
    mb = fmaxf(mb, dpp_f32<0xB1>(mb));
    mb = fmaxf(mb, dpp_f32<0x4E>(mb));
    mb = fmaxf(mb, dpp_f32<0x141>(mb));
    float sb = sw * (mw == -INFINITY ? 1.f : expf(mw - mb));
    sb += dpp_f32<0xB1>(sb);
    sb += dpp_f32<0x4E>(sb);
    sb += dpp_f32<0x141>(sb);
    if ((threadIdx.x & 7) == 0) {
      float* o = part + ((size_t)(sl * G1 + i) * ACC_CHUNKS + ch) * ACC_PART;
      o[k] = mb; o[k + 1] = sb;
    }
  }
}

// Four consecutive entries v..v+3 of both rows (one Philox block); 16-byte loads where the rows start on 16 bytes
__device__ __forceinline__ void acc_load4(const float* t, const float* q, bool wide, int v, int v1, float (&tv)[4], float (&qv)[4]) {
  if (wide && v + 4 <= v1) {
    const float4 a = *reinterpret_cast<const float4*>(t + v), b = *reinterpret_cast<const float4*>(q + v);
    tv[0] = a.x; tv[1] = a.y; tv[2] = a.z; tv[3] = a.w;
    qv[0] = b.x; qv[1] = b.y; qv[2] = b.z; qv[3] = b.w;
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      tv[e] = v + e < v1 ? t[v + e] : -INFINITY;
      qv[e] = v + e < v1 ? q[v + e] : -INFINITY;
    }
  }
}

// greedy: grid (rows, n_seqs, ACC_CHUNKS), 512 threads: best effective logit of row i over chunk ch
__global__ __launch_bounds__(512) void accept_rows_kernel(const float* __restrict__ tl, const float* __restrict__ ring, AccArgs aa, int G1, int V,
                                                          int phase, float* __restrict__ part) {
  __shared__ float redv[16];
  __shared__ int redi[16];
  const int si = blockIdx.y, ch = blockIdx.z, sl = aa.slot[si];
  int i;
  if (!acc_row(phase, aa.gamma[si], blockIdx.x, i)) return;
  const float beta = aa.beta[si];
  const float* t = tl + (size_t)(sl * G1 + i) * V;
  const float* q = ring + (size_t)(aa.qslot[si] * G1 + i) * V;
  float* o = part + ((size_t)(sl * G1 + i) * ACC_CHUNKS + ch) * ACC_PART;
  int v0, v1;
  acc_chunk_range(V, ch, v0, v1);
  const bool wide = ((reinterpret_cast<uintptr_t>(t) | reinterpret_cast<uintptr_t>(q)) & 15) == 0;
  float best = -INFINITY;
  int bi = 0x7fffffff;
  for (int v = v0 + threadIdx.x * 4; v < v1; v += 512 * 4) {
    float tv[4], qv[4];
    acc_load4(t, q, wide, v, v1, tv, qv);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float x = tv[e] + beta * qv[e];
      if (v + e < v1 && x > best) { best = x; bi = v + e; }
    }
  }
  block_argmax(best, bi, redv, redi);
  if (threadIdx.x == 0) {
    o[6] = best; o[7] = __int_as_float(bi);
  }
}

// Results of one sequence (one thread calls it; the accepted drafts' tokens are the caller's): the emitted token, (n, z) to the
// caller's arrays and to pinned host memory.  The ticket is written last; the host polls for it.
__device__ __forceinline__ void acc_emit(const AccArgs& aa, int si, int n, int z, int* tk, int* out_n, int* out_z, int* host_res, int* host_tick, int ticket,
                                         int V, int* host_bad) {
  const int s = aa.seq[si], sl = aa.slot[si];
  if (z >= 0 && tk) tk[n] = checked_token(z, V, host_bad, s);   // out_z keeps the raw value: 0x7fffffff = no finite logit decided
  out_n[sl] = n;
  out_z[sl] = z;
  if (host_res) {
    host_res[2 * s] = n;
    host_res[2 * s + 1] = z;
    __threadfence_system();            // the results first, then the ticket the host polls for
    host_tick[s] = ticket;
  }
}

// sampling, after accept_stats_kernel: grid (ACC_PICKERS, n_seqs), 512 threads of one entry each at a time.  Bound by a chain
// of round trips and by the instructions between them (a Philox block, logarithms and exponentials: 0.5 us for one entry, 1.5
// for the four that a Philox block serves, hence one per thread).  Candidates of the one row that is cut at, instead of all
// rows' in a launch between the statistics and a third one that found that row, take a window of 16 from 15.7 us a call to 10.4.
// A row's log-sum-exps combine the chunks in the order of their butterfly over 16 lanes, the same in every block.
// cand: per slot [ACC_PICKERS][2] (value, id) of the residual and of p.
__global__ __launch_bounds__(512) void accept_pick_kernel(const float* tl, const float* ring, const int* draft_tok, const float* part, int* arrivals, int G1,
                                                          int V, uint64_t seed, uint32_t step, int phase, uint64_t* cand, int max_seq, int* tokens,
                                                          int* out_n, int* out_z, int* host_res, int* host_tick, int ticket, int* host_bad, AccArgs aa) {
  static_assert(ACC_CHUNKS == 16 && ACC_MAXROWS == 32, "16 lanes per row, four rows per wave, eight waves");
  __shared__ float lse[ACC_MAXROWS][2];
  __shared__ int rej[ACC_MAXROWS];
  __shared__ float redv[2][8];
  __shared__ int redi[2][8];
  __shared__ int last;
  const int blk = blockIdx.x, si = blockIdx.y, lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int s = aa.seq[si], sl = aa.slot[si], qs = aa.qslot[si], gamma = aa.gamma[si];
  const float beta = aa.beta[si];
  const int rows = phase == ACC_PHASE_DRAFTS ? gamma : gamma + 1, first = phase == ACC_PHASE_BONUS ? gamma : 0;   // rows with statistics
  {
    const int i = wave * 4 + (lane >> 4);                // row of this group of 16 lanes, one chunk per lane
    const int ic = max(first, min(i, rows - 1));
    int rj = 0;
    if (rows > first) {
      const float4 pc = *reinterpret_cast<const float4*>(part + ((size_t)(sl * G1 + ic) * ACC_CHUNKS + (lane & 15)) * ACC_PART);
      const int y = ic < gamma ? draft_tok[qs * G1 + ic] : 0;
      const int yc = min(max(y, 0), V - 1);              // a caller-held draft id outside the vocabulary must not index past the row
      const float ty = tl[(size_t)(sl * G1 + ic) * V + yc], qy = ring[(size_t)(qs * G1 + ic) * V + yc];
      const uint4 b = vocab_bits(seed, s, step, (uint32_t)(ic + 1), PURPOSE_ACCEPT, 0u);
      float mp = pc.x, mq = pc.z;
      mp = fmaxf(mp, dpp_f32<0x128>(mp)); mq = fmaxf(mq, dpp_f32<0x128>(mq));      // row_ror 8, 4, 2, 1
      mp = fmaxf(mp, dpp_f32<0x124>(mp)); mq = fmaxf(mq, dpp_f32<0x124>(mq));
      mp = fmaxf(mp, dpp_f32<0x122>(mp)); mq = fmaxf(mq, dpp_f32<0x122>(mq));
      mp = fmaxf(mp, dpp_f32<0x121>(mp)); mq = fmaxf(mq, dpp_f32<0x121>(mq));
      float sp = pc.x > -INFINITY ? pc.y * expf(pc.x - mp) : 0.f, sq = pc.z > -INFINITY ? pc.w * expf(pc.z - mq) : 0.f;
      sp += dpp_f32<0x128>(sp); sq += dpp_f32<0x128>(sq);
      sp += dpp_f32<0x124>(sp); sq += dpp_f32<0x124>(sq);
      sp += dpp_f32<0x122>(sp); sq += dpp_f32<0x122>(sq);
      sp += dpp_f32<0x121>(sp); sq += dpp_f32<0x121>(sq);
      const float lsp = mp + logf(sp), lsq = mq + logf(sq);
      const float ratio = expf((ty + beta * qy - lsp) - (qy - lsq));
      rj = u01(b.x) > ratio ? 1 : 0;
      if ((lane & 15) == 0) { lse[i][0] = lsp; lse[i][1] = lsq; }
    }
    if ((lane & 15) == 0) rej[i] = i < gamma && phase != ACC_PHASE_BONUS ? rj : 0;
  }
  __syncthreads();
  const unsigned long long bad = __ballot(lane < ACC_MAXROWS && rej[lane & 31]);
  const int n = bad ? __ffsll(bad) - 1 : gamma;          // first rejected row, or every draft accepted
  int z = -1;
  if (n < gamma || phase != ACC_PHASE_DRAFTS) {
    // candidate tokens of row n: Gumbel-max over log max(0, p - q) (rows < gamma) or log p (bonus row);
    // if no residual mass exists the row falls back to log p with the same noise
    const float* t = tl + (size_t)(sl * G1 + n) * V;
    const float* q = ring + (size_t)(qs * G1 + n) * V;
    const float lsp = lse[n][0], lsq = lse[n][1];
    float best[2] = {-INFINITY, -INFINITY};              // [0] residual, [1] p
    int bi[2] = {0x7fffffff, 0x7fffffff};
    for (int v = blk * 512 + threadIdx.x; v < V; v += ACC_PICKERS * 512) {
      const float tv = t[v], qv = q[v];
      const uint4 b = vocab_bits(seed, s, step, (uint32_t)(n + 1), PURPOSE_NEXT, (uint32_t)v >> 2);
      const float g = gumbel(u01((v & 2) ? ((v & 1) ? b.w : b.z) : ((v & 1) ? b.y : b.x)));
      const float lp = tv + beta * qv - lsp;
      const float kp = lp + g;
      if (kp > best[1]) { best[1] = kp; bi[1] = v; }
      if (n < gamma) {
        const float w = expf(lp) - expf(qv - lsq);
        if (w > 0.f) {
          const float kr = logf(w) + g;
          if (kr > best[0]) { best[0] = kr; bi[0] = v; }
        }
      }
    }
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      wave_best(best[k], bi[k]);
      if (lane == 0) { redv[k][wave] = best[k]; redi[k][wave] = bi[k]; }
    }
    __syncthreads();
    // the block's candidates, written through to memory; the last block to arrive reads all of them (hand-over without a
    // device-scope fence: see gemm_w16_kernel)
    if (wave == 0) {
      uint64_t* o = cand + (size_t)sl * ACC_PICKERS * 2;
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        float v = redv[k][lane & 7];
        int id = redi[k][lane & 7];
        wave_best(v, id);
        if (lane == 0)
          __hip_atomic_store(o + blk * 2 + k, (uint64_t)__float_as_uint(v) | (uint64_t)(uint32_t)id << 32, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
      // one wave stores, waits and counts, so there is no barrier that would keep the compiler from moving the counter up
      asm volatile("" ::: "memory");
      PACER_WAIT_VMCNT0();                               // the write-through stores have completed
      asm volatile("" ::: "memory");
      int got = 0;
      if (lane == 0) got = __hip_atomic_fetch_add(arrivals + sl * G1, 1, PACER_HO_ORDER, __HIP_MEMORY_SCOPE_AGENT);
      got = __builtin_amdgcn_readfirstlane(got);
      if (got == ACC_PICKERS - 1) {
        static_assert(ACC_PICKERS == 64, "a lane per block");
        float cv[2];
        int ci[2];
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          const uint64_t w = __hip_atomic_load(o + lane * 2 + k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          cv[k] = __uint_as_float((uint32_t)w);
          ci[k] = (int)(w >> 32);
        }
#pragma unroll
        for (int k = 0; k < 2; ++k) wave_best(cv[k], ci[k]);
        z = n < gamma && cv[0] > -INFINITY ? ci[0] : ci[1];
      }
      if (lane == 0) last = got == ACC_PICKERS - 1;
    }
    __syncthreads();
    if (!last) return;
  } else if (blk) {
    return;                                              // nothing to look for: one block reports
  }
  int* tk = tokens ? tokens + (size_t)s * max_seq + aa.len[si] : nullptr;
  if (phase != ACC_PHASE_BONUS && tk && (int)threadIdx.x < n) tk[threadIdx.x] = draft_tok[qs * G1 + threadIdx.x];
  if (threadIdx.x == 0) acc_emit(aa, si, n, z, tk, out_n, out_z, host_res, host_tick, ticket, V, host_bad);
}

// greedy: n = first rejected row (or gamma).  n < gamma: next token = row n's best, tokens appended.  n = gamma: the bonus
// row's best if it has been evaluated (phases BONUS and ALL); in phase DRAFTS its draft logits still need one more draft
// forward: the drafts are appended and (gamma, -1) says that phase BONUS is still to come.
// tokens and the host words may be null (acceptance on caller-held logits without a context).
// One wave per sequence: 16 lanes look at a row's 16 chunks, so that the rows' candidates are a few rounds of loads (a
// serial walk over rows and chunks took 50 us for 16 greedy windows).
__global__ __launch_bounds__(64) void accept_finalize_kernel(const float* __restrict__ part, const int* __restrict__ draft_tok,
                                       AccArgs aa, int G1, int phase, int max_seq, int* __restrict__ tokens,
                                       int* __restrict__ out_n, int* __restrict__ out_z, int* __restrict__ host_res,
                                       int* __restrict__ host_tick, int ticket, int V, int* host_bad) {
  static_assert(ACC_CHUNKS == 16, "one lane per chunk, four rows at a time");
  const int si = blockIdx.x, s = aa.seq[si], sl = aa.slot[si], qs = aa.qslot[si];
  const int gamma = aa.gamma[si], lane = threadIdx.x, ch = lane & 15;
  // best candidate over the chunks of a row (the 16 lanes of a group call it with their chunk's; all get the result)
  auto over_chunks = [](float& v, int& id) {
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) take_better(v, id, __shfl_xor(v, o, 64), __shfl_xor(id, o, 64));
  };
  int n = gamma;
  if (phase != ACC_PHASE_BONUS) {
    // row i's draft is rejected when it differs from the row's argmax
    for (int i0 = 0; i0 < gamma && n == gamma; i0 += 4) {
      const int i = i0 + (lane >> 4), ic = min(i, gamma - 1);
      const float* pr = part + ((size_t)(sl * G1 + ic) * ACC_CHUNKS + ch) * ACC_PART;
      float best = pr[6];
      int bi = __float_as_int(pr[7]);
      // a chunk without a finite value leaves (-inf, sentinel), as does a row of them
      over_chunks(best, bi);
      const unsigned long long bad = __ballot(i < gamma && bi != draft_tok[qs * G1 + ic]);
      if (bad) n = i0 + (__ffsll(bad) - 1) / 16;
    }
  }
  int z = -1;
  if (phase != ACC_PHASE_DRAFTS || n < gamma) {
    const float* pr = part + ((size_t)(sl * G1 + n) * ACC_CHUNKS + ch) * ACC_PART;
    float best = pr[6];
    z = __float_as_int(pr[7]);
    over_chunks(best, z);
  }
  int* tk = tokens ? tokens + (size_t)s * max_seq + aa.len[si] : nullptr;
  if (phase != ACC_PHASE_BONUS && tk)
    for (int k = threadIdx.x; k < n; k += blockDim.x) tk[k] = draft_tok[qs * G1 + k];
  if (threadIdx.x == 0) acc_emit(aa, si, n, z, tk, out_n, out_z, host_res, host_tick, ticket, V, host_bad);
}

// ------------------------------------------------------------------ streaming-read probe (benchmarks)
// Reads n16 16-byte words once (grid-stride, eight loads in flight per lane) and folds them into one word per
// block: what a kernel that only streams from HBM through the L1s reaches on this GPU, the practical ceiling the
// weight-streaming GEMMs are measured against.  Launched as 256 blocks of 4 waves (one wave per SIMD): of the
// shapes tried (256..8192 blocks, 4..16 loads in flight, per-wave contiguous ranges or grid-stride) that one read
// fastest, 7.0 to 7.2 TB/s on 2 GiB.
__global__ __launch_bounds__(256) void stream_probe_kernel(const u32x4* __restrict__ src, size_t n16, uint32_t* __restrict__ sink) {
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  u32x4 acc = {0u, 0u, 0u, 0u};
  for (; i + 7 * stride < n16; i += 8 * stride) {
    u32x4 v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = __builtin_nontemporal_load(src + i + u * stride);
#pragma unroll
    for (int u = 0; u < 8; ++u) acc ^= v[u];
  }
  for (; i < n16; i += stride) acc ^= src[i];
  uint32_t x = acc[0] ^ acc[1] ^ acc[2] ^ acc[3];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) x ^= __shfl_xor(x, o, 64);
  if ((threadIdx.x & 63) == 0) sink[(blockIdx.x * 4 + (threadIdx.x >> 6)) & 63] = x;   // keeps the loads alive; the value is not used
}
