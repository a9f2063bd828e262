// Matrix-core attention for long sequences (spatial self-attention over H*W positions, cross-
// attention over the context tokens): bf16, any head dimension up to 128, any sequence length,
// online softmax in fp32.
//
// One workgroup = 4 x 32 queries of one (sequence, head), its 4 wavefronts sharing the key / value
// stages; one wavefront = 32 queries, which stay the
// *column* operand of every MFMA (v_mfma_f32_32x32x16_bf16: lane l supplies column l%32, k-slots
// 8*(l/32) .. +7; a result lane holds column l%32 and, in register 4q + j, row 8q + 4*(l/32) + j):
//   S^T[key, query] = K Q^T      row operand: 32 keys x 16 head channels
//   O^T[chan, query] += V^T P^T  row operand: 32 head channels x 16 keys; column operand: the softmax
//                                result registers of the lane, converted to bf16 -- no data movement.
// Every operand arrives as 1 KiB MFMA fragments (64 lanes x 16 bytes), written in this order by whoever
// produces it (the projections' epilogues, spatial_pre_kernel, pack_ctx_frag_kernel), so that every
// load of a wavefront is one contiguous KiB, whatever the head dimension: head dimensions that are no
// multiple of 16 are padded with zero channels in q and k only (d = 40: 48 of q and k, 64 of V^T), and
// the products' cost follows from the padded widths.
//   q: [(sequence, head)][32-query tile][KS k-steps]         lane (query r, half g): channels 16 ks + 8 g + e
//   k, v: [(key sequence, head)][32-key tile][KS + 2 DB]     KS fragments of K (lane (key r, g), same
//      channels), then V^T (block b, 16-key step t: fragment KS + 2 b + t, lane (channel r, g), keys
//      16 t + frak_k(g, e)): the result registers of S^T, packed pairwise, are in that k-order
// The channel order inside a k-step is free as long as q and k agree (spatial_pre_kernel's is frag_k's).
// Row-major q / k rows and a transposed copy of v (32 to 64 cache lines per wavefront load, head dimension
// 64 only) took 247 us instead of 223 per frame of 9216 keys (5 heads, 2 sequences) and 18.0 instead of 16.6 at
// 1024 keys x 10 heads x 2; heads of 40 went from the vector-ALU kernel to this one (4096 keys, 8 heads,
// 2 sequences: 4390 -> 66.7 us per frame, 43 GFLOP; its context attention 104 -> 10.5 us).
// Bound by the exponentials and the MFMAs, which do not overlap on a SIMD (per 64-key stage 32 v_exp_f32 at
// quarter rate = 512 cycles beside 16 MFMAs = 512 at 64 channels, 14 = 448 at 40).
// Keys past the end of the last tile may hold anything: their scores are overwritten with -inf and
// their values are cleared in registers.
#pragma once
#include "k_fused.h"

namespace si {

struct AttnMfmaArgs {
  const bf16* q;   // fragments; pre-scaled by softmax scale * log2(e), so that q k^T is the exponent in base 2
  const bf16* kv;  // fragments of key sequence s / kv_div
  bf16* o;         // token i of sequence s: row s*Nq + i
  int64_t ldo;
  int Nq, Nk, heads, d, kv_div;
  int o_frag;        // 0: o rows of ldo elements; else o is a fragment-order buffer of that many channels per token
  int nqt, ntiles;   // 128-query tiles per (sequence, head) pair; nqt * heads * sequences * ksplit (the grid is 8 * ceil(ntiles / 8))
  // FUSED only.  ksplit == 2: a workgroup takes one half of the keys; half kh leaves its output,
  // normalised by its own row sum, in o (kh = 0) / o2 (kh = 1) and, per lane, (reference maximum,
  // row sum) in ml[(kh * tiles + tile) * 64 + lane] -- whoever reads o merges the halves.
  int ksplit;
  bf16* o2;
  float2* ml;
  int64_t tiles32;   // 32-query tiles of all sequences
};

constexpr int kAttnStages = 3;
__host__ __device__ constexpr int attn_ksteps(int d) { return (d + 15) / 16; }
__host__ __device__ constexpr int attn_blocks(int d) { return (d + 31) / 32; }
// fragments of one 32-key tile of one head, and bytes of a query / key-value fragment buffer
__host__ __device__ constexpr int attn_tile_frags(int d) { return attn_ksteps(d) + 2 * attn_blocks(d); }
inline size_t attn_q_bytes(int64_t seqs, int heads, int64_t N, int d) { return (size_t)(seqs * heads * ((N + 31) / 32) * attn_ksteps(d)) * 1024; }
inline size_t attn_kv_bytes(int64_t seqs, int heads, int64_t N, int d) { return (size_t)(seqs * heads * ((N + 31) / 32) * attn_tile_frags(d)) * 1024; }

// Where the projections' epilogues put channel c (of heads * d) of token (s, i), as 16-bit elements.
struct AttnFragMap {
  int heads, d, tiles;  // tiles: 32-token tiles of a sequence
  // granule of the 8 channels that start at c8 * 8; *last: they end the head and the k-step's other half is padding
  __device__ __forceinline__ int64_t q_elem(int s, int i, int c8, bool* last) const {
    const int d8 = d >> 3, h = c8 / d8, g8 = c8 - h * d8;
    *last = (d8 & 1) && g8 == d8 - 1;
    return ((((int64_t)(s * heads + h) * tiles + (i >> 5)) * attn_ksteps(d) + (g8 >> 1)) * 64 + (g8 & 1) * 32 + (i & 31)) * 8;
  }
  __device__ __forceinline__ int64_t k_elem(int s, int i, int c8, bool* last) const {
    const int d8 = d >> 3, h = c8 / d8, g8 = c8 - h * d8;
    *last = (d8 & 1) && g8 == d8 - 1;
    return ((((int64_t)(s * heads + h) * tiles + (i >> 5)) * attn_tile_frags(d) + (g8 >> 1)) * 64 + (g8 & 1) * 32 + (i & 31)) * 8;
  }
  // V^T granule of channel c and the 8 keys 16 t + frag_k(g, .) of tile i32
  __device__ __forceinline__ int64_t v_elem(int s, int i32, int t, int g, int c) const {
    const int h = c / d, ch = c - h * d;
    return ((((int64_t)(s * heads + h) * tiles + i32) * attn_tile_frags(d) + attn_ksteps(d) + 2 * (ch >> 5) + t) * 64 + g * 32 + (ch & 31)) * 8;
  }
};

// Context keys / values, rows [B*Mc, 2D] (keys, then values), as the fragments above; padding keys and
// channels are zero.  One thread per 16-byte granule.
__global__ __launch_bounds__(256) void pack_ctx_frag_kernel(const bf16* __restrict__ kv, u32x4_t* __restrict__ dst, int B, int Mc,
                                                            int heads, int d) {
  const int KS = attn_ksteps(d), T = attn_tile_frags(d), tiles = (Mc + 31) / 32, D = heads * d;
  const int64_t id = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (id >= (int64_t)B * heads * tiles * T * 64) return;
  const int lane = (int)(id % 64), r = lane % 32, g = lane / 32;
  int64_t rest = id / 64;
  const int fr = (int)(rest % T);
  rest /= T;
  const int tile = (int)(rest % tiles), pair = (int)(rest / tiles), h = pair % heads, b = pair / heads;
  u32x4_t out = u32x4_t{0, 0, 0, 0};
  if (fr < KS) {
    const int key = tile * 32 + r, c = 16 * fr + 8 * g;
    if (key < Mc && c < d) out = *reinterpret_cast<const u32x4_t*>(kv + ((int64_t)b * Mc + key) * 2 * D + h * d + c);
  } else {
    const int c = 32 * ((fr - KS) / 2) + r, t = (fr - KS) % 2;
    unsigned short v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int key = tile * 32 + 16 * t + frag_k(g, e);
      v[e] = key < Mc && c < d ? kv[((int64_t)b * Mc + key) * 2 * D + D + h * d + c].v : (unsigned short)0;
    }
    out = u32x4_t{v[0] | ((unsigned)v[1] << 16), v[2] | ((unsigned)v[3] << 16), v[4] | ((unsigned)v[5] << 16), v[6] | ((unsigned)v[7] << 16)};
  }
  dst[id] = out;
}

// Online softmax, per 32-key tile of this wavefront's 32 queries.  The queries arrive pre-scaled by
// softmax scale * log2(e) (the projection's epilogue does it before its one rounding), so S^T is in
// base-2 exponent units.  `minit` holds -m (the lane's reference maximum) in all 16 registers and is
// the accumulator input of the first score MFMA of a tile: the result registers are s - m and go
// straight into v_exp_f32.  m is a *lazy* maximum: it is raised (and the output rescaled) only when
// some lane's partial row sum says that an exponent went beyond kLazyTrigger, so the steady state
// per tile is 16 exponentials, 8 conversions to bf16 pairs and 8 packed dot products for the row
// sum -- no maximum, no subtraction, no cross-lane traffic.  lsum is the lane's own half of the row
// sum (16 of a tile's 32 keys); the two halves meet once, after the last tile.
constexpr float kLazyTrigger = 256.f;  // 2^8: an exponential this large, or 16 of them each above 2^4

__device__ __forceinline__ float dot2_ones(unsigned packed_bf16x2, float acc) {
  return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, packed_bf16x2), __builtin_bit_cast(bf16x2_t, 0x3f803f80u), acc,
                                         false);
}

template <int DB>
struct AttnState {
  f32x16_t oacc[DB];  // O^T, 32-channel blocks
  f32x16_t minit;    // -m in every register
  float lsum;
};

// keys >= Nk of the tile that starts at key0 get a score of -inf
__device__ __forceinline__ void attn_mask_tile(f32x16_t& sc, int key0, int Nk, int g) {
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    if (key0 + 8 * (e / 4) + 4 * g + (e % 4) >= Nk) sc[e] = -INFINITY;
  }
}

__device__ __forceinline__ void attn_exp_pack(const f32x16_t& sc, float delta, u32x4_t (&pk)[2], float& rs) {
  unsigned w[8];
#pragma unroll
  for (int e = 0; e < 16; e += 2) w[e / 2] = pack_bf16x2(__builtin_amdgcn_exp2f(sc[e] - delta), __builtin_amdgcn_exp2f(sc[e + 1] - delta));
  rs = 0.f;
#pragma unroll
  for (int i = 0; i < 8; ++i) rs = dot2_ones(w[i], rs);
  pk[0] = u32x4_t{w[0], w[1], w[2], w[3]};
  pk[1] = u32x4_t{w[4], w[5], w[6], w[7]};
}

// Probabilities of one tile (scores sc = s - m) as the bf16 column operand pk of O^T += V^T P^T.
// Rare path: the reference maximum rises by delta -- the output so far and the row sum shrink by
// 2^-delta, and score tiles that were already taken against the old reference (l0, l1, l2; NULL =
// none) move by -delta.
template <int DB>
__device__ __forceinline__ void attn_softmax_tile(f32x16_t& sc, u32x4_t (&pk)[2], AttnState<DB>& st, f32x16_t* l0, f32x16_t* l1,
                                                  f32x16_t* l2) {
  float rs;
  attn_exp_pack(sc, 0.f, pk, rs);
  if (__builtin_amdgcn_ballot_w64(rs > kLazyTrigger) != 0) {
    float mx = sc[0];
#pragma unroll
    for (int e = 1; e < 16; ++e) mx = fmaxf(mx, sc[e]);
    mx = fmaxf(mx, __shfl_xor(mx, 32, kWave));  // both halves of the row agree on the new reference
    const float delta = fmaxf(mx, 0.f);
    const float alpha = __builtin_amdgcn_exp2f(-delta);
    st.lsum *= alpha;
#pragma unroll
    for (int b = 0; b < DB; ++b)
#pragma unroll
      for (int e = 0; e < 16; ++e) st.oacc[b][e] *= alpha;
#pragma unroll
    for (int e = 0; e < 16; ++e) st.minit[e] -= delta;
    attn_exp_pack(sc, delta, pk, rs);
    f32x16_t* later[3] = {l0, l1, l2};
#pragma unroll
    for (int i = 0; i < 3; ++i)
      if (later[i]) {
#pragma unroll
        for (int e = 0; e < 16; ++e) (*later[i])[e] -= delta;
      }
  }
  st.lsum += rs;
}

// values of keys >= Nk of the tile that starts at key0 become zero; vf: the tile's V^T fragments
template <int DB>
__device__ __forceinline__ void attn_mask_values(u32x4_t (&vf)[2 * DB], int key0, int Nk, int g) {
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const int key = key0 + 16 * t + frag_k(g, 2 * w);  // keys of a register: this one and the next
      const unsigned keep = key + 1 < Nk ? 0xffffffffu : key < Nk ? 0xffffu : 0u;
#pragma unroll
      for (int b = 0; b < DB; ++b) vf[2 * b + t][w] &= keep;
    }
}

// S^T of the stage's two tiles against minit; kf[u]: the K fragments of tile u.  The two chains are
// interleaved so that no MFMA waits for the one issued just before it.
template <int KS>
__device__ __forceinline__ void attn_scores(const u32x4_t (&kf)[2][KS], const bf16x8_t (&qop)[KS], const f32x16_t& minit, f32x16_t (&sc)[2]) {
#pragma unroll
  for (int ks = 0; ks < KS; ++ks)
#pragma unroll
    for (int u = 0; u < 2; ++u)
      sc[u] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, kf[u][ks]), qop[ks], ks == 0 ? minit : sc[u], 0, 0, 0);
}

// O^T += V^T P^T for one tile; vf: its V^T fragments (channel block b, k-step t: vf[2b + t])
template <int DB>
__device__ __forceinline__ void attn_pv(const u32x4_t (&vf)[2 * DB], const u32x4_t (&pk)[2], f32x16_t (&oacc)[DB]) {
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int b = 0; b < DB; ++b)
      oacc[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, vf[2 * b + t]), __builtin_bit_cast(bf16x8_t, pk[t]),
                                                        oacc[b], 0, 0, 0);
}

// KS: 16-channel k-steps of a head; DB: its 32-channel blocks.  FUSED: the three-kernel window (heads of
// 64, Nq % 128 == 0, Nk % (64 ksplit) == 0, kv_div == 1): the output leaves as the column operand of the
// next contraction, [32-token tile][k-step 0 .. 4 heads - 1 over the block width], optionally in two key
// halves.  Up to 64 channels the stages are software-pipelined; wider heads (whose operands and
// accumulators would not fit 256 registers that way) take a stage's products one after the other.
template <int KS, int DB, bool FUSED = false>
__global__ __launch_bounds__(256, KS <= 6 ? 2 : 1) void attn_mfma_kernel(AttnMfmaArgs a) {
  constexpr int NS = kAttnStages, T = KS + 2 * DB, FR = 2 * T;  // fragments per 32-key tile / 64-key stage
  constexpr int PER = (FR + 3) / 4;                             // stage loads per wavefront
  constexpr bool PIPE = KS <= 4;
  static_assert(!FUSED || (KS == 4 && DB == 2), "fused windows have heads of 64");
  __shared__ u32x4_t ring[NS][FR * kWave];
  const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
  const int wave_s = __builtin_amdgcn_readfirstlane(wave);
  const int r = lane % 32, g = lane / 32;
  // XCD-aware order: workgroups go to the 8 XCDs round-robin, and every XCD has an L2 of its own.
  // The work list (query tiles of one (sequence, head) pair after the other) is cut into 8
  // contiguous chunks, one per XCD, so that the keys and values of a pair are fetched into one L2
  // (two for a pair that straddles a chunk boundary) instead of into all eight.
  const int chunk = (a.ntiles + 7) / 8;
  const int work = (int)(blockIdx.x % 8) * chunk + (int)(blockIdx.x / 8);
  if (work >= a.ntiles) return;
  const int ksplit = FUSED ? a.ksplit : 1;
  // work list: the query tiles of one (pair, key half) after the other
  const int qtile = work % a.nqt, kh = (work / a.nqt) % ksplit, pair = work / (a.nqt * ksplit);
  const int h = pair % a.heads, s = pair / a.heads, ks = s / a.kv_div;
  const int qtiles = (a.Nq + 31) / 32;  // 32-query tiles of a sequence
  const int qt = qtile * 4 + wave, qi = qt * 32 + r;
  const bool qvalid = qi < a.Nq;
  const int ktiles = (a.Nk + 31) / 32;
  const int nst = (ktiles + 1) / 2 / ksplit;             // stages of this workgroup
  const bool ragged = !FUSED && (a.Nk % 64) != 0;        // the last stage has missing keys
  const bool half_stage = !FUSED && (ktiles & 1) != 0;   // ... or even no second tile

  // ---- stage loads: fragment ids wave + 4*i, i < PER (ids past the stage's end repeat the wavefront's
  // first one: same source, same destination).  Stages are issued in order, so every fragment's source
  // is a running scalar pointer and the ring slot a running scalar too: a stage's loads cost a few
  // scalar additions.  A missing second tile is filled from the first (its keys are masked).
  const unsigned voff = (unsigned)(lane * 16);
  const char* fb = reinterpret_cast<const char*>(a.kv) +
                   (FUSED ? (int64_t)((ks * a.heads + h) * ksplit + kh) * nst * FR : (int64_t)(ks * a.heads + h) * ktiles * T) * 1024;
  const char* cur[PER];
  unsigned loff[PER];
  bool second[PER];
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int id = wave_s + 4 * i < FR ? wave_s + 4 * i : wave_s;
    cur[i] = fb + id * 1024;
    loff[i] = (unsigned)(id * kWave * 16);
    second[i] = id >= T;
  }
  const unsigned ring_lds = (unsigned)(size_t)(__attribute__((address_space(3))) void*)(&ring[0][0]);
  constexpr unsigned kSlotBytes = FR * kWave * 16;
  unsigned islot = ring_lds;  // LDS address of the slot the next issued stage lands in
  auto issue = [&](int st) {
    if (st >= nst) return;
    const bool part = half_stage && st == nst - 1;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const char* src = part && second[i] ? cur[i] - T * 1024 : cur[i];
      // assembly for the same reason as in WeightPipe::issue: completion is awaited explicitly
      asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dwordx4 %0, %1" : : "v"(voff), "s"(src), "s"(islot + loff[i]) : "memory");
      cur[i] += FR * 1024;
    }
    islot = islot + kSlotBytes == ring_lds + NS * kSlotBytes ? ring_lds : islot + kSlotBytes;
  };
#pragma unroll
  for (int st = 0; st < NS - 1; ++st) issue(st);

  // ---- this lane's query as column operand; queries past the end are zero (their lanes take part in
  // the wavefront's decisions, so that must not depend on what the buffer holds)
  bf16x8_t qop[KS];
  {
    const u32x4_t* qf = reinterpret_cast<const u32x4_t*>(a.q) +
                        ((int64_t)(s * a.heads + h) * qtiles + (qt < qtiles ? qt : qtiles - 1)) * KS * kWave + lane;
#pragma unroll
    for (int k4 = 0; k4 < KS; ++k4) {
      const u32x4_t v = qf[k4 * kWave];
      qop[k4] = __builtin_bit_cast(bf16x8_t, FUSED || qvalid ? v : u32x4_t{0, 0, 0, 0});
    }
  }
  __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): the query loads; nothing the compiler tracks stays pending in the loop

  AttnState<DB> as;
#pragma unroll
  for (int b = 0; b < DB; ++b)
#pragma unroll
    for (int e = 0; e < 16; ++e) as.oacc[b][e] = 0.f;
#pragma unroll
  for (int e = 0; e < 16; ++e) as.minit[e] = 0.f;
  as.lsum = 0.f;

  // own loads of stage st have landed (at most the batches of the next NS - 2 stages stay in flight),
  // then the barrier: stage st is visible to all and everybody has left stage st - 1, whose slot the
  // load issued next overwrites
  auto open_stage = [&](int st) {
    if (nst - 1 - st >= 1) __builtin_amdgcn_s_waitcnt(WeightPipe<4>::wait_imm(PER));
    else __builtin_amdgcn_s_waitcnt(WeightPipe<4>::wait_imm(0));
    __syncthreads();
    issue(st + NS - 1);
  };
  const u32x4_t* slot = ring[0];  // slot of the stage whose scores are being formed
  auto next_ring = [&]() { slot = slot + FR * kWave == &ring[0][0] + NS * FR * kWave ? &ring[0][0] : slot + FR * kWave; };
  // the first tile sets the reference maximum (key 0 always exists, so it is finite)
  auto first_max = [&](f32x16_t(&sc)[2]) {
    float mx = sc[0][0];
#pragma unroll
    for (int e = 1; e < 16; ++e) mx = fmaxf(mx, sc[0][e]);
    mx = fmaxf(mx, __shfl_xor(mx, 32, kWave));
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      as.minit[e] = -mx;
      sc[0][e] -= mx;
      sc[1][e] -= mx;
    }
  };
  auto mask_scores = [&](f32x16_t(&sc)[2]) {
    attn_mask_tile(sc[0], 64 * (nst - 1), a.Nk, g);
    attn_mask_tile(sc[1], 64 * (nst - 1) + 32, a.Nk, g);
  };

  u32x4_t kf[2][KS], vf[2][2 * DB];
  auto read_k = [&]() {
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int i = 0; i < KS; ++i) kf[u][i] = slot[(u * T + i) * kWave + lane];
  };
  auto read_v = [&]() {
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int i = 0; i < 2 * DB; ++i) vf[u][i] = slot[(u * T + KS + i) * kWave + lane];
  };
  auto mask_values = [&]() {
    attn_mask_values<DB>(vf[0], 64 * (nst - 1), a.Nk, g);
    attn_mask_values<DB>(vf[1], 64 * (nst - 1) + 32, a.Nk, g);
  };
  if constexpr (PIPE) {
    // Software pipeline over stages: while the matrix cores form the scores of stage st, the vector
    // ALUs exponentiate the first tile of stage st - 1; O^T += V^T P^T of that tile then runs under the
    // exponentials of the second one.  The V^T fragments of a stage are taken out of LDS before the
    // next barrier, because that barrier frees their slot.
    f32x16_t scA[2], scB[2];  // scores of the previous / the new stage, roles alternating
    open_stage(0);
    read_k();
    read_v();
    attn_scores<KS>(kf, qop, as.minit, scA);
    if (ragged && nst == 1) mask_scores(scA);
    first_max(scA);
    // one stage: scores of stage st into scn while scp (stage st - 1) is exponentiated and multiplied into O^T
    auto stage_body = [&](int st, f32x16_t(&scp)[2], f32x16_t(&scn)[2]) {
      open_stage(st);
      next_ring();
      read_k();
      u32x4_t pk[2];
      attn_scores<KS>(kf, qop, as.minit, scn);
      attn_softmax_tile<DB>(scp[0], pk, as, &scp[1], &scn[0], &scn[1]);
      attn_pv<DB>(vf[0], pk, as.oacc);
      attn_softmax_tile<DB>(scp[1], pk, as, &scn[0], &scn[1], nullptr);
      attn_pv<DB>(vf[1], pk, as.oacc);
      read_v();
    };
    // drain: the last stage's tiles (the only ones that can hold keys past the end)
    auto drain = [&](f32x16_t(&scp)[2]) {
      if (ragged) {
        if (nst > 1) mask_scores(scp);
        mask_values();
      }
      u32x4_t pk[2];
      attn_softmax_tile<DB>(scp[0], pk, as, &scp[1], nullptr, nullptr);
      attn_pv<DB>(vf[0], pk, as.oacc);
      attn_softmax_tile<DB>(scp[1], pk, as, nullptr, nullptr, nullptr);
      attn_pv<DB>(vf[1], pk, as.oacc);
    };
    int st = 1;
    for (; st + 1 < nst; st += 2) {
      stage_body(st, scA, scB);
      stage_body(st + 1, scB, scA);
    }
    if (st < nst) {
      stage_body(st, scA, scB);
      drain(scB);
    } else {
      drain(scA);
    }
  } else {
    for (int st = 0; st < nst; ++st) {
      open_stage(st);
      if (st > 0) next_ring();
      f32x16_t sc[2];
      u32x4_t pk[2];
      read_k();
      attn_scores<KS>(kf, qop, as.minit, sc);
      read_v();
      if (ragged && st == nst - 1) {
        mask_scores(sc);
        mask_values();
      }
      if (st == 0) first_max(sc);
      attn_softmax_tile<DB>(sc[0], pk, as, &sc[1], nullptr, nullptr);
      attn_pv<DB>(vf[0], pk, as.oacc);
      attn_softmax_tile<DB>(sc[1], pk, as, nullptr, nullptr, nullptr);
      attn_pv<DB>(vf[1], pk, as.oacc);
    }
  }
  const float lsum = as.lsum + __shfl_xor(as.lsum, 32, kWave);  // the two halves of the row
  const float inv = 1.0f / lsum;
  f32x16_t(&oacc)[DB] = as.oacc;

  // ---- O^T / l: register 4q + j of block b is head channel 32b + 8q + 4g + j of this lane's query
  if constexpr (FUSED) {
    const int64_t tile = (int64_t)s * qtiles + qt;
    u32x4_t* of = reinterpret_cast<u32x4_t*>(kh ? a.o2 : a.o) + (tile * (a.heads * 4) + 4 * h) * kWave + lane;
    if (ksplit > 1) a.ml[(((int64_t)kh * a.heads + h) * a.tiles32 + tile) * kWave + lane] = make_float2(-as.minit[0], lsum);
#pragma unroll
    for (int b = 0; b < DB; ++b)
#pragma unroll
      for (int hf = 0; hf < 2; ++hf) {
        u32x4_t v;
        v.x = pack_bf16x2(oacc[b][8 * hf + 0] * inv, oacc[b][8 * hf + 1] * inv);
        v.y = pack_bf16x2(oacc[b][8 * hf + 2] * inv, oacc[b][8 * hf + 3] * inv);
        v.z = pack_bf16x2(oacc[b][8 * hf + 4] * inv, oacc[b][8 * hf + 5] * inv);
        v.w = pack_bf16x2(oacc[b][8 * hf + 6] * inv, oacc[b][8 * hf + 7] * inv);
        of[(2 * b + hf) * kWave] = v;
      }
  } else {
    // one lane^32 exchange per two register quads leaves each lane with the 8 consecutive channels of a
    // 16-byte granule: lane half g takes channels 32b + 16hf + 8g .. +7
    const int64_t m = (int64_t)s * a.Nq + qi;
#pragma unroll
    for (int b = 0; b < DB; ++b)
#pragma unroll
      for (int hf = 0; hf < 2; ++hf) {
        unsigned w[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) w[i] = pack_bf16x2(oacc[b][8 * hf + 2 * i] * inv, oacc[b][8 * hf + 2 * i + 1] * inv);
        // lanes 32..63 of the first operand change places with lanes 0..31 of the second
        const auto x = __builtin_amdgcn_permlane32_swap(w[0], w[2], false, false);
        const auto y = __builtin_amdgcn_permlane32_swap(w[1], w[3], false, false);
        const int c = 32 * b + 16 * hf + 8 * g;
        if (qvalid && c < a.d) {
          u32x4_t v;
          v.x = x[0]; v.y = y[0]; v.z = x[1]; v.w = y[1];
          bf16* dst = a.o_frag ? a.o + act_offset(m, h * a.d + c, a.o_frag) : a.o + m * a.ldo + h * a.d + c;
          *reinterpret_cast<u32x4_t*>(dst) = v;
        }
      }
  }
}

// ----------------------------------------------------------------------------- projections that feed it

// q/k/v projection (columns [0, D) queries, [D, 2D) keys, [2D, 3D) values): queries times qscale
// (softmax scale * log2(e)) in fp32 before their one rounding.  A lane holds four consecutive columns of
// one token, i.e. half a granule of q or k.  Values: column tiles at or behind swap_from are computed
// with the operands swapped (activations as the MFMA row operand), which leaves the lane with 16 tokens
// of one channel -- two V^T granules as they stand (vblock32; needs sequences of whole 32-token blocks);
// otherwise they are scattered as 2-byte stores.
struct EpiQKVFrag {
  static constexpr bool kRows8 = false;
  static constexpr bool kSwapCols = true;
  bf16 *q, *kv;
  AttnFragMap map;
  int D, Pw;
  float qscale;
  int swap_from;
  __device__ __forceinline__ void operator()(int64_t m, int n0, const float (&v)[4]) const {
    const int c8 = __builtin_amdgcn_readfirstlane(n0 >> 3);  // the two halves of a wavefront hold one granule
    const int mi = (int)m, s = mi / Pw, i = mi - s * Pw;     // window tokens fit 31 bits
    if (8 * c8 < 2 * D) {
      const bool isq = 8 * c8 < D;
      const float sc = isq ? qscale : 1.f;
      bool last;
      bf16* dst = isq ? q + map.q_elem(s, i, c8, &last) : kv + map.k_elem(s, i, c8 - D / 8, &last);
      uint2 pk;
      pk.x = (unsigned)float_to_bf16_bits(v[0] * sc) | ((unsigned)float_to_bf16_bits(v[1] * sc) << 16);
      pk.y = (unsigned)float_to_bf16_bits(v[2] * sc) | ((unsigned)float_to_bf16_bits(v[3] * sc) << 16);
      *reinterpret_cast<uint2*>(dst + (n0 & 7)) = pk;
      if (last) *reinterpret_cast<uint2*>(dst + 32 * 8 + (n0 & 7)) = make_uint2(0, 0);  // the k-step's padding half
    } else {
      const int j = i & 15;
      bf16* dst = kv + map.v_elem(s, i >> 5, (i >> 4) & 1, (j >> 2) & 1, n0 - 2 * D) + (j & 3) + 4 * (j >> 3);
#pragma unroll
      for (int e = 0; e < 4; ++e) dst[e * 8] = from_float<bf16>(v[e]);  // four channels of one block: adjacent granules
    }
  }
  // One 32-column result block of the ring kernel (D % 32 == 0: all queries, all keys or all values): one
  // lane^32 exchange per two register quads makes every q / k store a whole granule.
  static constexpr bool kBlock32 = true;
  __device__ __forceinline__ void block32(int64_t m, bool mvalid, int n0, const f32x16_t& acc, int half) const {
    const int mi = (int)m, s = mi / Pw, i = mi - s * Pw;
    if (n0 < 2 * D) {
      const bool isq = n0 < D;
      const float sc = isq ? qscale : 1.f;
#pragma unroll
      for (int hf = 0; hf < 2; ++hf) {
        unsigned w[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) w[e] = pack_bf16x2(acc[8 * hf + 2 * e] * sc, acc[8 * hf + 2 * e + 1] * sc);
        const auto x = __builtin_amdgcn_permlane32_swap(w[0], w[2], false, false);
        const auto y = __builtin_amdgcn_permlane32_swap(w[1], w[3], false, false);
        if (mvalid) {
          bool last;
          const int c8 = (isq ? n0 : n0 - D) / 8 + 2 * hf + half;
          u32x4_t* dst = reinterpret_cast<u32x4_t*>(isq ? q + map.q_elem(s, i, c8, &last) : kv + map.k_elem(s, i, c8, &last));
          *dst = u32x4_t{x[0], y[0], x[1], y[1]};
          if (last) dst[32] = u32x4_t{0, 0, 0, 0};  // the k-step's padding half
        }
      }
    } else if (mvalid) {
      const int j = i & 15;
#pragma unroll
      for (int qd = 0; qd < 4; ++qd) {
        bf16* dst = kv + map.v_elem(s, i >> 5, (i >> 4) & 1, (j >> 2) & 1, n0 - 2 * D + 8 * qd + 4 * half) + (j & 3) + 4 * (j >> 3);
#pragma unroll
        for (int e = 0; e < 4; ++e) dst[e * 8] = from_float<bf16>(acc[4 * qd + e]);
      }
    }
  }
  __device__ __forceinline__ void vblock32(int64_t m0, int n, const f32x16_t& acc, int half) const {
    const int mi = (int)m0, s = mi / Pw, i32 = (mi - s * Pw) >> 5;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      unsigned w[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) w[i] = pack_bf16x2(acc[8 * t + 2 * i], acc[8 * t + 2 * i + 1]);
      *reinterpret_cast<u32x4_t*>(kv + map.v_elem(s, i32, t, half, n - 2 * D)) = u32x4_t{w[0], w[1], w[2], w[3]};
    }
  }
};

// Query projection of the attention over the context.
struct EpiQFrag {
  static constexpr bool kRows8 = false;
  bf16* q;
  AttnFragMap map;
  int Pw;
  float qscale;
  static constexpr bool kBlock32 = true;
  __device__ __forceinline__ void block32(int64_t m, bool mvalid, int n0, const f32x16_t& acc, int half) const {
    EpiQKVFrag{q, nullptr, map, 1 << 28, Pw, qscale, 0}.block32(m, mvalid, n0, acc, half);
  }
  __device__ __forceinline__ void operator()(int64_t m, int n0, const float (&v)[4]) const {
    const int c8 = __builtin_amdgcn_readfirstlane(n0 >> 3);
    const int mi = (int)m, s = mi / Pw, i = mi - s * Pw;
    bool last;
    bf16* dst = q + map.q_elem(s, i, c8, &last) + (n0 & 7);
    uint2 pk;
    pk.x = (unsigned)float_to_bf16_bits(v[0] * qscale) | ((unsigned)float_to_bf16_bits(v[1] * qscale) << 16);
    pk.y = (unsigned)float_to_bf16_bits(v[2] * qscale) | ((unsigned)float_to_bf16_bits(v[3] * qscale) << 16);
    *reinterpret_cast<uint2*>(dst) = pk;
    if (last) *reinterpret_cast<uint2*>(dst + 32 * 8) = make_uint2(0, 0);
  }
};

}  // namespace si
