// Tiled GEMM of the bf16-weight path for many rows (gfx950): operand and weights staged in LDS by direct loads.
#pragma once
#include "kernels_w16.h"
#include <type_traits>

// One wave's 1 KiB load from global memory straight into LDS: lane l's 16 bytes at base + voff go to LDS byte m0 + 16 l.
// Written as asm because the compiler, which cannot tell the stages apart, waits for every outstanding load of this kind
// before any LDS read; there is no output register, and the kernel counts the loads itself (s_waitcnt vmcnt).  m0 is an
// operand of the asm: the compiler writes the address there itself and so knows what the register holds (as a reserved
// register it could not be declared as clobbered; saving and restoring it around each load cost 0.3 to 0.6 % of a pass).
// ONCE: bytes that no other block reads; they pass L2 without displacing what the next kernels find there.
template <bool ONCE>
__device__ __forceinline__ void load_to_lds(const void* base, unsigned voff, unsigned lds_byte) {
  if constexpr (ONCE) asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 nt" ::"{m0}"(lds_byte), "v"(voff), "s"(base) : "memory");
  else asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"{m0}"(lds_byte), "v"(voff), "s"(base) : "memory");
}
template <int N> __device__ __forceinline__ void wait_vm_lds() {   // vmcnt <= N and all LDS reads of this wave back
  static_assert(N < 64, "6-bit counter");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (0 << 8));
}

// Where lane l of a staging load takes its 16 bytes of a 1 KiB operand tile ([row][64 bytes]), and where MFMA lane l finds
// its own in the staged copy (units of 16 bytes).  A load's 16-lane quarter covers 4 whole rows = 256 contiguous bytes
// (two cache lines); taking the tile in MFMA lane order instead makes every quarter touch all eight lines of the tile,
// four times the work of the CU's memory pipeline.  Chunk c of row r sits in slot 4r + (c ^ (r/2 % 4)), so that the
// lanes that one LDS read cycle serves fall on different banks (SQ_LDS_BANK_CONFLICT is 0 in verify and prompt passes).
__device__ __forceinline__ int stage_src(int l) { return (l & ~3) + ((l & 3) ^ ((l >> 3) & 3)); }
__device__ __forceinline__ int stage_slot(int l) { return (l & 15) * 4 + ((l >> 4) ^ ((l >> 1) & 3)); }

// More than 32 rows (batched verification, prompt passes, and some launches from 18 rows on).
//   block   RT row tiles x CT output tiles, WR x WC waves of RT/WR x CT/WC tiles each
//   K loop  one step of 32 inputs per barrier.  Operand (RT * HL KiB per step) and weights (CT KiB) go straight from global
//           memory into two LDS rings: NX operand steps, NW batches of WB weight steps.  A wave reads the fragments of step
//           k+1 from LDS between the products of step k, and issues its share of the loads of step k + NX there too.
// Why this form (7B QKV GEMM at 512 rows unless said otherwise):
//   - LDS reads that a wave issues in one go after the barrier keep all waves from their products until the LDS has served
//     all of them: 91 us in a microbenchmark, 83 with the reads spread between the products.
//   - A CU's loads return in order, so an operand load that hits in L2 waits behind a weight load from HBM: what counts is the
//     bytes a CU pulls per product, hence blocks as large as the rows and registers allow (up to 176 tile pairs), and that the
//     weights of several steps are under way together, hence their own ring with batches (80 us).
//   - In a prompt pass it takes 91 us; register staging of the operand with per-wave register streams of the weights, the
//     form this replaces, took 118, and the library's GEMM with the same number of products (512 x 12288 x 8192, f16) 92.
// K slices across blocks (ksb > 1) hand their sums over as in gemm_w16_kernel.  Blocks that share weights (same output
// tiles, other rows) get consecutive slots on one XCD (block id mod 8), so that the later ones find them in that L2.
// Tiles and row tiles that do not exist are replaced by the nearest one that does; their products are never stored.
template <int EPI, int RT, int CT, int WR, int WC, int HL, int NX, int WB, int NW>
__global__ __launch_bounds__(WR * WC * 64, 1) void gemm_tile_kernel(const GemmArgs ga, int n_tiles, int n_groups, int row_groups, int ksb) {
  constexpr int WV = WR * WC, MR = RT / WR, NC = CT / WC, XT = RT * HL, WT = WB * CT;
  constexpr int LX = (XT + WV - 1) / WV, LW = (WT + WV - 1) / WV;      // loads per wave: operand of a step, weights of a batch
  constexpr bool SPLIT = CT <= 8;      // wider blocks always take all of K
  constexpr bool ONCE = RT == 2;       // up to 32 rows are one row group: each weight byte is one block's
  static_assert(RT % WR == 0 && CT % WC == 0, "the waves cover the block tile");
  static_assert(NX >= 3 && NW >= 2 && (WB == 1 || WB % 2 == 0) && (NW > 2 || WB > 1), "");
  extern __shared__ __align__(16) u32x4 tile_stage[];       // [NX][XT][64] operand, then [NW][WB][CT][64] weights
  __shared__ unsigned arrived;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int wr = wave % WR, wc = wave / WR;
  const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
  const int rg = slot % row_groups, ksl = (slot / row_groups) % ksb, ng = (slot / (row_groups * ksb)) * 8 + xcd;
  if (ng >= n_groups) return;
  const int mtt = ga.mt_total;
  const int mt_lo = mtt * rg / row_groups;
  const int mtb = mtt * (rg + 1) / row_groups - mt_lo;       // row tiles of this block, 1..RT
  const int nt0 = ga.nt_begin + ng * CT;
  const int nt_end = ga.nt_begin + n_tiles;
  const int kb = ksl * ga.KT / ksb, nk = (ksl + 1) * ga.KT / ksb - kb;   // this block's K steps (at least WB)

  // this wave's share of the loads: parts wave, wave + WV, ... (one past the last repeats it: same bytes, same place)
  const char* xk = reinterpret_cast<const char*>(ga.X + ((size_t)mt_lo * 2 + (size_t)kb * mtt * 2) * 64);   // next step to load
  const char* w0 = reinterpret_cast<const char*>(ga.W + ((size_t)nt0 * ga.KT + kb) * 64);
  unsigned xv[LX], wv[LW], xdst[LX], wdst[LW];
  const unsigned lds0 = (unsigned)(size_t)(__attribute__((address_space(3))) void*)tile_stage;
#pragma unroll
  for (int i = 0; i < LX; ++i) {
    const int t = min(wave + WV * i, XT - 1);
    xv[i] = stage_src(lane) * 16 + (min(t / HL, mtb - 1) * 2 + t % HL) * 1024;
    xdst[i] = lds0 + t * 1024;
  }
#pragma unroll
  for (int i = 0; i < LW; ++i) {
    const int t = min(wave + WV * i, WT - 1), c = t / WB, j = t % WB;    // waves next to each other read K steps next to each other
    wv[i] = lane * 16 + (min(c, nt_end - 1 - nt0) * ga.KT + j) * 1024;
    wdst[i] = lds0 + (NX * XT + j * CT + c) * 1024;
  }
  auto issue_x = [&](int i, int slot_x) {
    load_to_lds<false>(xk, xv[i], xdst[i] + slot_x * (XT * 1024));
    if (i == LX - 1) xk += (unsigned)mtt * 2048;
  };
  auto issue_w = [&](int i, int k0, int slot_w) {                        // k0: the batch's first step; a short last batch starts earlier
    load_to_lds<ONCE>(w0 + ((size_t)min(k0, nk - WB) << 10), wv[i], wdst[i] + slot_w * (WT * 1024));
  };
  f32x4 acc[NC][MR];
#pragma unroll
  for (int a = 0; a < NC; ++a)
#pragma unroll
    for (int b = 0; b < MR; ++b) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int slot_rd = stage_slot(lane);
  typedef half8 Frag[NC + MR * HL];
  constexpr int NF = NC + MR * HL, NM = NC * MR * HL;
  // fragment i of a step whose operand is at xb and whose weights are at wb
  auto fetch1 = [&](Frag& f, int i, const u32x4* xb, const u32x4* wb) {
    f[i] = __builtin_bit_cast(half8, i < NC ? wb[(wc * NC + i) * 64 + lane] : xb[(wr * MR * HL + i - NC) * 64 + slot_rd]);
  };
  auto mul1 = [&](Frag& f, int m) {
    const int t = m / NC, a = m % NC;
    acc[a][t / HL] = __builtin_amdgcn_mfma_f32_16x16x32_f16(f[a], f[NC + t], acc[a][t / HL], 0, 0, 0);
  };
  auto xbase = [&](int sx) { return tile_stage + (size_t)sx * XT * 64; };
  auto wbase = [&](int sw, int j) { return tile_stage + ((size_t)NX * XT + (size_t)sw * WT + j * CT) * 64; };

  // Order of the loads: step s issues (W batch s/WB + NW-1 if s is a multiple of WB) and then (X of step s + NX).
  // The prologue issues those of the steps before 0 in the same order.
  constexpr int PRE = NX > (NW - 1) * WB ? NX : (NW - 1) * WB;
#pragma unroll
  for (int s = -PRE; s < 0; ++s) {
    if (s % WB == 0 && s / WB + NW - 1 >= 0) {
      const int b = s / WB + NW - 1;
      if (b * WB < nk) {
#pragma unroll
        for (int i = 0; i < LW; ++i) issue_w(i, b * WB, b);
      }
    }
    if (s + NX >= 0 && s + NX < nk) {
#pragma unroll
      for (int i = 0; i < LX; ++i) issue_x(i, s + NX);
    }
  }
  wait_vm_lds<0>();
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  Frag f0, f1;
#pragma unroll
  for (int i = 0; i < NF; ++i) fetch1(f0, i, xbase(0), wbase(0, 0));
  int sx = 0, sw = 0, k = 0;                        // operand slot of step k, weight slot of its batch
  // Step k, phase ph = k % WB: multiplies the fragments of step k (read during step k-1) while it reads those of step
  // k+1; at its start every wave has the fragments of step k in registers, so its operand slot is free.
  auto body = [&](auto ph_c, Frag& cur, Frag& nxt) {
    constexpr int PH = decltype(ph_c)::value;
    constexpr int NEED_X = (NX - 2) * LX + ((PH - 1 + WB * 64) / WB - (PH + 1 - NX + WB * 64) / WB) * LW;   // issued after X(k+1)
    constexpr int NEED_W = ((NW - 2) * WB + WB - 1) * LX + ((NW - 2) * WB + WB - 2) / WB * LW;               // issued after the next batch
    constexpr int N = PH == WB - 1 ? (NEED_X < NEED_W ? NEED_X : NEED_W) : NEED_X;
    wait_vm_lds<N>();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    const int sxn = sx + 1 == NX ? 0 : sx + 1, swn = PH == WB - 1 ? (sw + 1 == NW ? 0 : sw + 1) : sw;
    const u32x4 *xb = xbase(sxn), *wb = wbase(swn, PH == WB - 1 ? 0 : PH + 1);
    const int swp = sw == 0 ? NW - 1 : sw - 1;      // the slot of the batch before: takes batch p + NW - 1
    constexpr int LL = LX + (PH == 0 ? LW : 0);
#pragma unroll
    for (int m = 0; m < NM; ++m) {
#pragma unroll
      for (int i = 0; i < NF; ++i)
        if (i * NM / NF == m) fetch1(nxt, i, xb, wb);
#pragma unroll
      for (int i = 0; i < LL; ++i)
        if (i * NM / LL == m) {
          if (i < LL - LX) issue_w(i, k + (NW - 1) * WB, swp);
          else issue_x(i - (LL - LX), sx);
        }
      __builtin_amdgcn_sched_barrier(0);
      mul1(cur, m);
      __builtin_amdgcn_sched_barrier(0);
    }
    sx = sxn;
    sw = swn;
    ++k;
  };
  // main part: every load that a step issues exists
  constexpr int U = WB == 1 ? 2 : WB;
  const int n_main = nk - PRE - U;
  while (k <= n_main) {
    if constexpr (WB == 1) {
      body(std::integral_constant<int, 0>{}, f0, f1);
      body(std::integral_constant<int, 0>{}, f1, f0);
    } else if constexpr (WB == 2) {
      body(std::integral_constant<int, 0>{}, f0, f1);
      body(std::integral_constant<int, 1>{}, f1, f0);
    } else {
      body(std::integral_constant<int, 0>{}, f0, f1);
      body(std::integral_constant<int, 1>{}, f1, f0);
      body(std::integral_constant<int, 2>{}, f0, f1);
      body(std::integral_constant<int, 3>{}, f1, f0);
    }
  }
  // the last steps: k is a multiple of WB here
  for (int ph = 0; k < nk; ++k) {
    wait_vm_lds<0>();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    if (ph == 0 && k + (NW - 1) * WB < nk) {
#pragma unroll
      for (int i = 0; i < LW; ++i) issue_w(i, k + (NW - 1) * WB, sw == 0 ? NW - 1 : sw - 1);
    }
    if (k + NX < nk) {
#pragma unroll
      for (int i = 0; i < LX; ++i) issue_x(i, sx);
    }
    sx = sx + 1 == NX ? 0 : sx + 1;
    if (++ph == WB) { ph = 0; sw = sw + 1 == NW ? 0 : sw + 1; }
    const int k0 = k + 1 - ph;                                          // first step of the batch of step k + 1
    if (k + 1 < nk) {
#pragma unroll
      for (int i = 0; i < NF; ++i) fetch1(f1, i, xbase(sx), wbase(sw, k + 1 - min(k0, nk - WB)));
    }
#pragma unroll
    for (int m = 0; m < NM; ++m) mul1(f0, m);
#pragma unroll
    for (int i = 0; i < NF; ++i) f0[i] = f1[i];
  }
  if (SPLIT && ksb > 1) {
    // partial tiles of this K slice, written through to memory; whoever arrives last adds all slices in slice order
    // (hand-over without a device-scope fence: see gemm_w16_kernel).  A store covers 512 contiguous bytes.
    u64* part = reinterpret_cast<u64*>(ga.sk_part);
    constexpr size_t per_block = (size_t)WV * NC * MR * 128;           // 8-byte words
    const size_t gidx = (size_t)ng * row_groups + rg;
    u64* mine = part + (gidx * ksb + ksl) * per_block + (size_t)wave * NC * MR * 128 + lane;
#pragma unroll
    for (int a = 0; a < NC; ++a)
#pragma unroll
      for (int b = 0; b < MR; ++b) {
        const float2 lo = {acc[a][b][0], acc[a][b][1]}, hi = {acc[a][b][2], acc[a][b][3]};
        u64* d = mine + (size_t)(a * MR + b) * 128;
        __hip_atomic_store(d, __builtin_bit_cast(u64, lo), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(d + 64, __builtin_bit_cast(u64, hi), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
    PACER_WAIT_VMCNT0();   // this wave's write-through stores have completed
    __syncthreads();
    if (threadIdx.x == 0) arrived = __hip_atomic_fetch_add(ga.sk_cnt + gidx, 1u, PACER_HO_ORDER, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    if (arrived != (unsigned)(ksb - 1)) return;
    if (threadIdx.x == 0) __hip_atomic_store(ga.sk_cnt + gidx, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    f32x4 own[NC][MR];
#pragma unroll
    for (int a = 0; a < NC; ++a)
#pragma unroll
      for (int b = 0; b < MR; ++b) { own[a][b] = acc[a][b]; acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f}; }
    for (int s = 0; s < ksb; ++s) {
      if (s == ksl) {
#pragma unroll
        for (int a = 0; a < NC; ++a)
#pragma unroll
          for (int b = 0; b < MR; ++b) acc[a][b] += own[a][b];
        continue;
      }
      const u64* srcp = part + (gidx * ksb + s) * per_block + (size_t)wave * NC * MR * 128 + lane;
#pragma unroll
      for (int a = 0; a < NC; ++a) {
        u64 v0[MR], v1[MR];
#pragma unroll
        for (int b = 0; b < MR; ++b) {
          v0[b] = __hip_atomic_load(srcp + (size_t)(a * MR + b) * 128, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          v1[b] = __hip_atomic_load(srcp + (size_t)(a * MR + b) * 128 + 64, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
#pragma unroll
        for (int b = 0; b < MR; ++b) {
          const float2 lo = __builtin_bit_cast(float2, v0[b]), hi = __builtin_bit_cast(float2, v1[b]);
          acc[a][b] += f32x4{lo.x, lo.y, hi.x, hi.y};
        }
      }
    }
  }
  constexpr int BCH = EPI == EPI_RESID || EPI == EPI_QKV ? (12 / NC > 0 ? (12 / NC < MR ? 12 / NC : MR) : 1) : 1;   // rows whose inputs are in flight together
  RowCtx rc[MR];
#pragma unroll
  for (int b = 0; b < MR; ++b) rc[b] = row_ctx<EPI>(ga, wr * MR + b < mtb ? (mt_lo + wr * MR + b) * 16 + (lane & 15) : ga.R);   // a row tile past the block's last is dead
#pragma unroll
  for (int b0 = 0; b0 < MR; b0 += BCH) {
    EpiAux ax[BCH][NC];
#pragma unroll
    for (int b = b0; b < b0 + BCH && b < MR; ++b)
#pragma unroll
      for (int a = 0; a < NC; ++a) ax[b - b0][a] = epi_aux<EPI>(ga, rc[b], min(nt0 + wc * NC + a, nt_end - 1), (mt_lo + wr * MR + b) * 16 + (lane & 15), lane);
#pragma unroll
    for (int b = b0; b < b0 + BCH && b < MR; ++b) {
      if (wr * MR + b >= mtb) continue;
      const int m = (mt_lo + wr * MR + b) * 16 + (lane & 15);
      u64 ssq = 0;
#pragma unroll
      for (int a = 0; a < NC; ++a) {
        const int nt = nt0 + wc * NC + a;
        if (nt >= nt_end) continue;
        const float sq = gemm_epilogue<EPI, true>(ga, rc[b], ax[b - b0][a], nt, m, lane, acc[a][b]);
        if (EPI == EPI_RESID) ssq += tile_ssq(sq);
      }
      if (EPI == EPI_RESID) add_row_ssq(ga, rc[b], m, lane, ssq);
    }
  }
}
