// GEMM on fragment-order operands in tiles of 160 columns: the staged blocks' projections and FFN where 160 divides the
// columns and 64 the contraction.
//
// The ring kernel's wavefronts (k_conv.h) pass through "wait, barrier, issue loads, read LDS, MFMAs" once per 32 channels, one
// phase after the other, and hide them behind a second workgroup where there is one.  Here a stage is 64 channels; its
// fragments are read three steps ahead of their MFMAs and the loads of a later stage are issued one per step between them,
// so that a lone workgroup keeps its matrix cores busy.  Every result is the sum in the ring kernel's order: the same bits.
//   WC = 2, TM = 2: 256 tokens x 320 columns, 8 wavefronts of 64 x 160, 7 KiB of LDS reads per 10 MFMAs (ff1)
//   WC = 1, TM = 1: 128 tokens x 160 columns, 4 wavefronts of 32 x 160
// In the kernel, cycles: 669 per 16 channels of the first form (its MFMAs are 660) + 4.3 k prologue + 10.7 k epilogue (the GELU's
// vector instructions); ff1 at 1280 channels on 2048 tokens 61 -> 47 us (1.15 PFLOP/s; dense bf16 MFMAs on such data reach 1.8 at the
// clock they leave).  Second form: 215 per 16 channels (165), 334 with two slots, which L2's latency then bounds.
// Blocks, all of their GEMMs on the ring kernel -> this one where it takes them: 640 channels, 14 frames x 500 positions per window 1282 -> 1141 us; 640 spatial, one frame per window
// 1405 -> 1341; 1280 spatial 1077 -> 1029, temporal 888 -> 839; 320 spatial with heads of 40 9257 -> 8990.
#pragma once
#include "k_conv.h"

namespace si {

// a.act, a.wf, a.M, a.C (contraction length, a multiple of 64), a.O as in ring_mma_kernel, the weights packed in column tiles of
// 160; a.ncol: column tiles of this kernel; a.ntiles, a.col_major likewise.
template <int WC, int TM, int NSLOT, bool F16, class Epi>
__global__ __launch_bounds__(256 * WC, WC == 2 ? 2 : 1) void gemm_160_kernel(ConvArgs a, Epi epi) {
  constexpr int TN = 5, NW = 4 * WC;          // 32-column blocks of a wavefront, wavefronts
  constexpr int TOK = 128 * TM;               // tokens of a workgroup
  constexpr int AFR = 16 * TM, WFR = 20 * WC;  // fragments of a stage: token blocks x 4 k-steps, column tiles x 2 k-tiles x 10
  constexpr int SLOT = (AFR + WFR) * 1024;
  constexpr int NL = (AFR + WFR) / NW;        // loads per wavefront and stage
  static_assert(AFR % NW == 0 && WFR % NW == 0 && NL <= 17, "every wavefront loads as much of either operand");
  __shared__ __attribute__((aligned(1024))) char lds[NSLOT * SLOT];

  const int chunk = (a.ntiles + 7) / 8;  // XCD-aware order, as in ring_mma_kernel
  const int tile = (blockIdx.x % 8) * chunk + blockIdx.x / 8;
  if (tile >= a.ntiles) return;
  const int nrow = a.ntiles / a.ncol;
  const int col = __builtin_amdgcn_readfirstlane(a.col_major ? tile / nrow : tile % a.ncol);
  const int64_t m0 = (int64_t)__builtin_amdgcn_readfirstlane(a.col_major ? tile % nrow : tile / a.ncol) * TOK;

  const int tid = threadIdx.x, lane = tid % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int wrow = wave / WC, wcol = wave % WC;
  const int nst = a.C / 64;

  // ---- number wave + NW l of a stage's loads is this wavefront's l-th.  Token blocks past the last one repeat it.
  const unsigned lds0 = (unsigned)(size_t)(__attribute__((address_space(3))) void*)lds;
  const char* actp = a.act + kActZeroBytes;  // running: the stage being loaded
  const char* wfp = a.wf + (int64_t)(WC * col) * (a.C / 32) * (2 * TN * 1024);
  const int last_block = (int)((a.M + 31) / 32) - 1;
  unsigned off[NL];
#pragma unroll
  for (int l = 0; l < NL; ++l) {
    const int id = wave + NW * l;
    if (l < AFR / NW) {
      const int tb = (int)(m0 / 32) + id / 4;
      off[l] = ((unsigned)(tb < last_block ? tb : last_block) * (unsigned)(a.C / 16) + (unsigned)(id % 4)) * 1024u;
    } else {
      off[l] = ((unsigned)((id - AFR) / 20) * (unsigned)(a.C / 32) * (2 * TN) + (unsigned)((id - AFR) % 20)) * 1024u;
    }
  }
  auto load = [&](int l, int slot) {
    const char* src = (l < AFR / NW ? actp : wfp) + off[l];
    asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dwordx4 %0, %1"
                 :
                 : "v"((unsigned)(lane * 16)), "s"(src), "s"(lds0 + (unsigned)(slot * SLOT + (wave + NW * l) * 1024))
                 : "memory");
  };
  auto advance = [&](int st) {  // to stage st; past the end the last one is fetched once more, into a slot nobody reads
    if (st < nst) {
      actp += 4 * 1024;
      wfp += 20 * 1024;
    }
  };

  f32x16_t acc[TN][TM];
#pragma unroll
  for (int i = 0; i < TN; ++i)
#pragma unroll
    for (int j = 0; j < TM; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

  // a weight fragment serves the TM MFMAs of one step; it is read three steps ahead, the next k-step's activations two or three
  u32x4_t wf[TN], af[2][TM];
  const char* mine = lds + lane * 16;
  auto read_a = [&](int slot, int q, int j) {
    return *reinterpret_cast<const u32x4_t*>(mine + slot * SLOT + ((wrow * TM + j) * 4 + q) * 1024);
  };
  auto read_w = [&](int slot, int q, int i) {
    return *reinterpret_cast<const u32x4_t*>(mine + slot * SLOT + (AFR + wcol * 20 + q * TN + i) * 1024);
  };
  auto mma = [&](const u32x4_t& w, const u32x4_t& x, f32x16_t& c) {
    if constexpr (F16) c = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8_t, w), __builtin_bit_cast(f16x8_t, x), c, 0, 0, 0);
    else c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, w), __builtin_bit_cast(bf16x8_t, x), c, 0, 0, 0);
  };
  // this wavefront's loads of the next stage have landed (those of NSLOT - 2 younger stages may be under way) and its LDS reads
  // returned; then everybody's
  auto stage_barrier = [&]() {
    constexpr int n = (NSLOT - 2) * NL;
    static_assert(n <= 63, "vmcnt range");
    __builtin_amdgcn_s_waitcnt(0x0070 | (n & 15) | (n >> 4) << 14);
    __syncthreads();
  };

#pragma unroll
  for (int s = 0; s < NSLOT - 1; ++s) {
    if (s > 0) advance(s);
#pragma unroll
    for (int l = 0; l < NL; ++l) load(l, s);
  }
  stage_barrier();
  advance(NSLOT - 1);
#pragma unroll
  for (int l = 0; l < 3; ++l) load(l, NSLOT - 1);
#pragma unroll
  for (int j = 0; j < TM; ++j) af[0][j] = read_a(0, 0, j);
#pragma unroll
  for (int i = 0; i < 3; ++i) wf[i] = read_w(0, 0, i);
  int slot = 0, prev = NSLOT - 1;  // of this stage and the one before
  for (int st = 0; st < nst; ++st) {
    const int next = slot + 1 == NSLOT ? 0 : slot + 1;
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int i = 0; i < TN; ++i) {
        const int nq = (q + 1) % 4, nslot = q == 3 ? next : slot;  // the k-step behind this one
        // nobody reads this stage any more (its last fragments are in registers), and the next one has landed
        if (q == 3 && i == 2) {
          stage_barrier();
          advance(st + NSLOT);
        }
        if (i < 2) wf[i + 3] = read_w(slot, q, i + 3);
        else wf[i - 2] = read_w(nslot, nq, i - 2);
        if (i >= 2 && i < 2 + TM) af[nq & 1][i - 2] = read_a(nslot, nq, i - 2);
#pragma unroll
        for (int j = 0; j < TM; ++j) mma(wf[i], af[q & 1][j], acc[i][j]);
        // the stage NSLOT further on, into the slot left behind: a load per step from the barrier on
        const int since = q == 3 ? i - 2 : q * TN + i + 3;
        __builtin_amdgcn_sched_barrier(0);
        if (q == 3 && since >= 0) load(since, slot);
        else if (q < 3 && since < NL) load(since, prev);
        __builtin_amdgcn_sched_barrier(0);
      }
    prev = slot;
    slot = next;
  }

  const int trow = lane % 32, half = lane / 32;
  auto column = [&](int i) { return ((WC * col + wcol) * TN + i) * 32; };
  if constexpr (epi_block32<Epi>::value) {
    typename Epi::Ahead ahead[TN];
#pragma unroll
    for (int i = 0; i < TN; ++i) epi.request(ahead[i], column(i), half);
    __builtin_amdgcn_s_waitcnt(0x0070 | 0xF00);  // vmcnt(0)
#pragma unroll
    for (int j = 0; j < TM; ++j) {
      const int64_t m = m0 + (wrow * TM + j) * 32 + trow;
#pragma unroll
      for (int i = 0; i < TN; ++i) epi.block32(m, m < a.M, column(i), acc[i][j], half, ahead[i]);
    }
  } else if constexpr (epi_slice_out<Epi>::value) {
    static_assert(WC == 1 && 2 * 32 * (TOK + 4) * 4 <= NSLOT * SLOT, "one column tile, buffers fit");
    __builtin_amdgcn_s_waitcnt(0x0070 | 0xF00);  // vmcnt(0): the padding loads of the last stages
    __syncthreads();
    slice_out_rows<TN, TOK, 256>(lds, epi, m0, a.M, column(0), a.O, [&](int i, float* patch) {
#pragma unroll
      for (int j = 0; j < TM; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) patch[(e / 4 * 8 + half * 4 + e % 4) * (TOK + 4) + (wrow * TM + j) * 32 + trow] = acc[i][j][e];
    });
  } else if constexpr (epi_residual<Epi>::value) {
    // Rows of the fp32 residual stream through the idle slots: a result lane holds four columns of one token, and going to
    // memory like that, 32 rows per instruction, took 16.5 k cycles of a tile (as much as its contraction over 1280 channels),
    // whole rows take 12 k.  Unit u, 16 bytes: row t = u / G, the row's columns 4 ((u % G) ^ (t % 8)) .. + 3, so that the lanes of a
    // wavefront, one row each, use different banks.
    static_assert(WC == 1 && TOK * 32 * TN * 4 <= NSLOT * SLOT, "one column tile, within the slots");
    constexpr int G = 8 * TN, ITER = TOK * G / 256;
    const int n0 = column(0);
    float* base = epi.h + m0 * epi.ld + n0;
    const int rows = a.M - m0 < TOK ? (int)(a.M - m0) : TOK;
    auto offset = [&](int u) {
      const int t = u / G;
      return (unsigned)t * (unsigned)epi.ld + 4u * (unsigned)((u - t * G) ^ (t & 7));
    };
    uint2 bias[4 * TN];  // requested together
    if (epi.bias) {
#pragma unroll
      for (int k = 0; k < 4 * TN; ++k) bias[k] = *reinterpret_cast<const uint2*>(epi.bias + n0 + 8 * k + 4 * half);
    } else {
#pragma unroll
      for (int k = 0; k < 4 * TN; ++k) bias[k] = make_uint2(0u, 0u);
    }
    __builtin_amdgcn_s_waitcnt(0x0070 | 0xF00);  // vmcnt(0): the padding loads of the last stages
    __syncthreads();
    if (epi.accumulate) {
#pragma unroll 2
      for (int k = 0; k < ITER; ++k) {
        const int u = k * 256 + tid;
        const unsigned at = u / G < rows ? 4 * offset(u) : 0u;
        asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dwordx4 %0, %1"
                     :
                     : "v"(at), "s"(base), "s"(lds0 + (unsigned)(k * 256 + wave * kWave) * 16)
                     : "memory");
      }
    }
    __builtin_amdgcn_s_waitcnt(0x0070 | 0xF00);
    __syncthreads();
#pragma unroll
    for (int j = 0; j < TM; ++j) {
      const int t = (wrow * TM + j) * 32 + trow;
#pragma unroll
      for (int k = 0; k < 4 * TN; ++k) {
        float4* p = reinterpret_cast<float4*>(lds) + t * G + ((2 * k + half) ^ (t & 7));
        float4 o = epi.accumulate ? *p : make_float4(0.f, 0.f, 0.f, 0.f);
        o.x += acc[k / 4][j][k % 4 * 4 + 0] + __uint_as_float(bias[k].x << 16);
        o.y += acc[k / 4][j][k % 4 * 4 + 1] + __uint_as_float(bias[k].x & 0xffff0000u);
        o.z += acc[k / 4][j][k % 4 * 4 + 2] + __uint_as_float(bias[k].y << 16);
        o.w += acc[k / 4][j][k % 4 * 4 + 3] + __uint_as_float(bias[k].y & 0xffff0000u);
        *p = o;
        if (epi.copy && t < rows) epi.store_copy(m0 + t, n0 + 8 * k + 4 * half, o);
      }
    }
    __syncthreads();
#pragma unroll 2
    for (int k = 0; k < ITER; ++k) {
      const int u = k * 256 + tid;
      if (u / G < rows) *reinterpret_cast<float4*>(base + offset(u)) = reinterpret_cast<const float4*>(lds)[u];
    }
  } else {
    static_assert(!Epi::kRows8, "no such epilogue");
    __builtin_amdgcn_s_waitcnt(0x0070 | 0xF00);
#pragma unroll
    for (int j = 0; j < TM; ++j) {
      const int64_t m = m0 + (wrow * TM + j) * 32 + trow;
      if (m >= a.M) continue;
#pragma unroll
      for (int i = 0; i < TN; ++i)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const float v[4] = {acc[i][j][q * 4 + 0], acc[i][j][q * 4 + 1], acc[i][j][q * 4 + 2], acc[i][j][q * 4 + 3]};
          epi(m, column(i) + q * 8 + half * 4, v);
        }
    }
  }
}

}  // namespace si
