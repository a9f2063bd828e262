// 3x3 convolution (same map, or after nearest doubling) whose activations reach LDS once per 32 channels
// instead of once per tap.
//
// What bounds the tap-by-tap ring kernel (k_conv.h) is the global->LDS delivery, 18 KiB for every 10 MFMAs of a
// wavefront, and phases that follow one another because a CU holds one workgroup.  Here a workgroup of 8 wavefronts
// owns 256 tokens x 160 output channels, and a channel chunk's patch -- the source tokens that any tap of the 256
// outputs reads, consecutive in memory -- is fetched once and read at nine shifts.
// Wavefront (pair, ks) contracts the pair's 64 tokens over channels 16 ks .. +15 of every chunk: 7 KiB of
// LDS reads for 10 MFMAs, where 32-token wavefronts would need 6 KiB for 5.  The two halves of a sum meet in LDS once,
// after the last stage.  A stage is one kernel row (three taps) of a chunk: 42 KiB of weights and patch arrive one load
// per wavefront and every other step, because a load blocks its wavefront while the address unit takes it: all at once
// behind the barrier they made the first of the calls below 2262 us instead of 2152, and with 4 wavefronts of 96 x 160,
// where they stop the only wavefront of a SIMD, it took 2697.
// In the kernel, cycles, one frame of 72 x 128 x 2, 320 channels (144 workgroups): 700 per tap, 660 of them the MFMAs of a SIMD's two
// wavefronts, x 90; prologue 5.4 k, exchange 4 k, epilogue 12 k (conv1) and 10.5 k (conv2, whose slice-out waited for x once per
// channel block before: 52.6 -> 50.3 us per launch).  At 1.8 GHz, which MFMAs on such data leave, that is the 50 us.
// Measured (ring kernel -> this one): ResBlock of 320 channels on 72 x 128, 25 frames one at a time, 2450 -> 2240 us; 640
// channels on 36 x 64, 16 frames two at a time, 1490 -> 1267 us; 640 channels doubled to 72 x 128, 12 frames, 1630 ->
// 1394 us (1.0 -> 1.17 PFLOP/s).
#pragma once
#include "k_conv.h"

namespace si {

constexpr int kHaloTokens = 256, kHaloTN = 5;  // output tokens and 32-channel blocks of a workgroup

// 64-token blocks of source tokens that the taps of kHaloTokens consecutive output tokens reach
inline int64_t halo_blocks(int W, int Wi, int mode) {
  if (mode == kConvSame) return (kHaloTokens + 2 * (int64_t)W + 2 + 63) / 64;
  const int64_t rows = (kHaloTokens - 1 + (int64_t)W - 1) / W + 1;  // output rows that a tile touches, at most
  return (((rows + 1) / 2 + 2) * Wi + 63) / 64;
}

// N64: 64-token blocks per patch that LDS holds.  a.H, a.W: output map; a.Hi, a.Wi: source map; nblk = halo_blocks().
// UP: source pixel of output (y, x), tap (dy, dx) is ((y + dy) / 2, (x + dx) / 2) of the half-size map.
template <int N64, bool F16, bool UP, class Epi>
__global__ __launch_bounds__(512, 2) void conv_halo_kernel(ConvArgs a, int nblk, Epi epi) {
  constexpr int TM = 2, TN = kHaloTN;               // 32-token row tiles, 32-channel blocks of a wavefront
  constexpr int WFR = 2 * TN;                       // weight fragments of one tap's k-tile
  constexpr int WST = 3 * WFR * 1024;               // weights of a stage
  constexpr int PLANE = N64 * 1024;                 // a patch: 4 planes [8-channel granule][token], 16 bytes each
  constexpr int AST = 4 * PLANE;
  constexpr int ZERO = 2 * WST + 2 * AST;           // 16 zero bytes: what a tap outside the image reads
  __shared__ __attribute__((aligned(1024))) char lds[ZERO + 64];

  const int chunk_tiles = (a.ntiles + 7) / 8;  // consecutive tiles stay on one XCD, as in ring_mma_kernel
  const int tile = (blockIdx.x % 8) * chunk_tiles + blockIdx.x / 8;
  if (tile >= a.ntiles) return;
  const int col = tile % a.ncol;
  const int m0 = (tile / a.ncol) * kHaloTokens;  // window tokens fit 31 bits

  const int tid = threadIdx.x, lane = tid % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int pair = wave >> 1, ks = wave & 1;
  const int trow = lane % 32, half = lane / 32;
  const int M = (int)a.M, W = a.W, H = a.H, Wi = UP ? a.Wi : a.W;
  const int nch = a.C / 32;
  if (tid < 4) *reinterpret_cast<unsigned*>(lds + ZERO + 4 * tid) = 0u;

  // first source token of the patch, last valid source token
  int s0, slast;
  if constexpr (UP) {  // H is even: (image row + dy) / 2 is also the row in the stack of all images
    const int Y0 = m0 / W;
    s0 = (Y0 > 0 ? (Y0 - 1) >> 1 : 0) * Wi;
    slast = (M / (W * H)) * (a.Hi * Wi) - 1;
  } else {
    s0 = m0 - W - 1;
    slast = M - 1;
  }

  // per row tile: LDS offset of the lane's source granule at the centre tap; bit t: tap t lies inside the image,
  // bits 9 and 10: odd row, odd column (UP).  Two registers, re-derived per tap: nine offsets would not fit.
  int base[TM], mask[TM];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int tok = m0 + pair * 64 + j * 32 + trow;
    const int Y = tok / W, x = tok - Y * W, y = Y % H;
    const int src = UP ? (Y >> 1) * Wi + (x >> 1) : tok;
    base[j] = 2 * WST + (2 * ks + half) * PLANE + 16 * (src - s0);
    mask[j] = (Y & 1) << 9 | (x & 1) << 10;
#pragma unroll
    for (int t = 0; t < 9; ++t) {
      const int dy = t / 3 - 1, dx = t % 3 - 1;
      if (tok < M && (unsigned)(y + dy) < (unsigned)H && (unsigned)(x + dx) < (unsigned)W) mask[j] |= 1 << t;
    }
  }

  const unsigned lds0 = (unsigned)(size_t)(__attribute__((address_space(3))) void*)lds;
  const char* wtile = a.wf + (int64_t)col * (9 * nch) * (WFR * 1024);
  auto load = [&](unsigned voff, const char* sbase, unsigned dst) {
    asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dwordx4 %0, %1" : : "v"(voff), "s"(sbase), "s"(lds0 + dst) : "memory");
  };
  // A stage's loads, numbered per wavefront: first the weights of kernel row r, chunk cc (fragments past the stage repeat
  // the last one: same source, same destination), then part p (of three) of plane wave % 4 of a patch: its
  // 64-token blocks 2 (p + 3 i) + wave / 4 (blocks past the patch repeat the last); tokens outside the window repeat
  // its first or last one (no tap inside the image reads them).
  constexpr int NLW = (3 * WFR + 7) / 8, NLA = ((N64 + 1) / 2 + 2) / 3, NL = NLW + NLA;
  auto load_w = [&](int cc, int r, int i, int buf) {
    const int id = wave + 8 * i < 3 * WFR ? wave + 8 * i : 3 * WFR - 1;
    const int t = id / WFR, f = id - t * WFR;
    load((unsigned)(lane * 16), wtile + ((int64_t)((3 * r + t) * nch + cc) * WFR + f) * 1024, (unsigned)(buf * WST + id * 1024));
  };
  auto load_a = [&](int cc, int p, int i, int buf) {
    const int plane = wave & 3, b0 = 2 * (p + 3 * i) + (wave >> 2), blk = b0 < nblk ? b0 : nblk - 1;
    int src = s0 + blk * 64 + lane;
    src = src < 0 ? 0 : src > slast ? slast : src;
    const unsigned voff =
        (unsigned)kActZeroBytes + 16u * ((unsigned)((src >> 5) * (a.C / 16) + 2 * cc + (plane >> 1)) * 64u + (plane & 1) * 32u + (src & 31));
    load(voff, a.act, (unsigned)(2 * WST + buf * AST + plane * PLANE + blk * 1024));
  };
  // i-th load of what takes the place of stage (cc, r) when everybody has left it: weights of the stage after the next,
  // a third of the next patch.  Past the last chunk the last one is fetched once more, into slots nobody reads.
  auto refill = [&](int cc, int r, int i) {
    const int wc = r == 0 ? cc : cc + 1, an = r == 2 ? cc + 2 : cc + 1;
    if (i < NLW) load_w(wc < nch ? wc : nch - 1, r == 0 ? 2 : r - 1, i, (cc + r) & 1);
    else load_a(an < nch ? an : nch - 1, r == 2 ? 0 : r + 1, i - NLW, an & 1);
  };

  f32x16_t acc[TN][2];
#pragma unroll
  for (int i = 0; i < TN; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

  // Fragments: a weight fragment serves the TM MFMAs of one step and is read three steps ahead, the next tap's activations two
  // or three.
  u32x4_t wf[TN], af[2][TM];
  auto read_w = [&](int cc, int r, int t, int i) {
    return *reinterpret_cast<const u32x4_t*>(lds + ((cc + r) & 1) * WST + (t * WFR + ks * TN + i) * 1024 + lane * 16);
  };
  auto read_a = [&](int cc, int r, int t, int j) {
    int in = base[j];
    if constexpr (UP) {  // (y + dy) / 2 - y / 2 is -1 for dy = -1 on even rows, +1 for dy = 1 on odd ones
      if (r == 0) in -= mask[j] & 512 ? 0 : 16 * Wi;
      if (r == 2) in += mask[j] & 512 ? 16 * Wi : 0;
      if (t == 0) in -= mask[j] & 1024 ? 0 : 16;
      if (t == 2) in += mask[j] & 1024 ? 16 : 0;
    } else {
      in += 16 * ((r - 1) * W + t - 1);
    }
    const int off = mask[j] & (1 << (3 * r + t)) ? in + (cc & 1) * AST : ZERO;
    return *reinterpret_cast<const u32x4_t*>(lds + off);
  };
  auto mma = [&](const u32x4_t& w, const u32x4_t& x, f32x16_t& c) {
    if constexpr (F16) c = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8_t, w), __builtin_bit_cast(f16x8_t, x), c, 0, 0, 0);
    else c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, w), __builtin_bit_cast(bf16x8_t, x), c, 0, 0, 0);
  };
  // all but this wavefront's last `flying` loads have landed and its LDS reads have returned; then everybody's
  auto stage_barrier = [&](auto flying) {
    __builtin_amdgcn_s_waitcnt(0x0070 | decltype(flying)::value);  // vmcnt(flying) lgkmcnt(0)
    __syncthreads();
  };
  using All = std::integral_constant<int, 0>;
  using NotPatch = std::integral_constant<int, NLA>;

#pragma unroll
  for (int i = 0; i < NLW; ++i) load_w(0, 0, i, 0);
#pragma unroll
  for (int p = 0; p < 3; ++p)
#pragma unroll
    for (int i = 0; i < NLA; ++i) load_a(0, p, i, 0);
  stage_barrier(All());
  refill(-1, 2, 0);
  refill(-1, 2, 1);
#pragma unroll
  for (int j = 0; j < TM; ++j) af[0][j] = read_a(0, 0, 0, j);
#pragma unroll
  for (int i = 0; i < TN - 2; ++i) wf[i] = read_w(0, 0, 0, i);
  static_assert(TN == 5 && TM == 2, "step order");
  for (int cc = 0; cc < nch; ++cc) {
    // opaque: the taps' offsets and masks are not to be kept in registers across chunks
#pragma unroll
    for (int j = 0; j < TM; ++j) asm volatile("" : "+v"(base[j]), "+v"(mask[j]));
#pragma unroll
    for (int tap = 0; tap < 9; ++tap) {
      const int r = tap / 3, t = tap % 3;
      // the tap behind this one (past the last chunk the reads go on, into registers nobody uses: no branch)
      const int ntap = (tap + 1) % 9, ncc = tap == 8 ? cc + 1 : cc;
#pragma unroll
      for (int i = 0; i < TN; ++i) {
        // Nobody reads this stage any more (its last fragments are in registers) and the next one's data has had time
        // to land; the part of a patch that came with it is not needed before the next chunk.
        if (t == 2 && i == 2) {
          if (r == 2) stage_barrier(All());
          else stage_barrier(NotPatch());
        }
        if (i < 2) wf[i + 3] = read_w(cc, r, t, i + 3);
        else wf[i - 2] = read_w(ncc, ntap / 3, ntap % 3, i - 2);
        if (i == 2 || i == 3) af[(tap + 1) & 1][i - 2] = read_a(ncc, ntap / 3, ntap % 3, i - 2);
#pragma unroll
        for (int j = 0; j < TM; ++j) mma(wf[i], af[tap & 1][j], acc[i][j]);
        // the loads of a refill, one every other step from the barrier on
        const int since = t == 2 ? i - 2 : t * TN + i + 3;  // steps behind the barrier
        __builtin_amdgcn_sched_barrier(0);
        if (t == 2 && since >= 0 && since % 2 == 0) refill(cc, r, since / 2);
        else if (t < 2 && since % 2 == 0 && since / 2 < NL) refill(r == 0 ? cc - 1 : cc, r == 0 ? 2 : r - 1, since / 2);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
#pragma unroll
    for (int j = 0; j < TM; ++j) af[0][j] = af[1][j];
  }
  stage_barrier(All());

  // the wavefronts of a pair exchange a row tile each: ks keeps tile ks, whose sum over all channels it then holds
  if (ks) {
#pragma unroll
    for (int i = 0; i < TN; ++i) {
      const f32x16_t s = acc[i][0];
      acc[i][0] = acc[i][1];
      acc[i][1] = s;
    }
  }
  constexpr int XB = 3;  // channel blocks per exchange
  static_assert(8 * XB * 4096 <= ZERO, "exchange fits");
#pragma unroll
  for (int i0 = 0; i0 < TN; i0 += XB) {
    __syncthreads();
#pragma unroll
    for (int i = i0; i < TN && i < i0 + XB; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        *reinterpret_cast<float4*>(lds + (((i - i0) * 8 + wave) * 4 + q) * 1024 + lane * 16) =
            make_float4(acc[i][1][4 * q], acc[i][1][4 * q + 1], acc[i][1][4 * q + 2], acc[i][1][4 * q + 3]);
    __syncthreads();
#pragma unroll
    for (int i = i0; i < TN && i < i0 + XB; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float4 o = *reinterpret_cast<const float4*>(lds + (((i - i0) * 8 + (wave ^ 1)) * 4 + q) * 1024 + lane * 16);
        acc[i][0][4 * q] += o.x;
        acc[i][0][4 * q + 1] += o.y;
        acc[i][0][4 * q + 2] += o.z;
        acc[i][0][4 * q + 3] += o.w;
      }
  }

  const int trel = pair * 64 + ks * 32 + trow;  // the lane's token of the tile
  if constexpr (epi_slice_out<Epi>::value) {
    static_assert(2 * 32 * (kHaloTokens + 4) * 4 <= ZERO, "buffers fit");
    __syncthreads();  // the exchange has been read
    slice_out_rows<TN, kHaloTokens, 512>(lds, epi, m0, M, col * TN * 32, a.O, [&](int i, float* patch) {
#pragma unroll
      for (int e = 0; e < 16; ++e) patch[(e / 4 * 8 + half * 4 + e % 4) * (kHaloTokens + 4) + trel] = acc[i][0][e];
    });
  } else if constexpr (Epi::kRows8) {  // 8 consecutive tokens of one channel at a time, transposed through LDS
    constexpr int TOK = 256, LDP = TOK + 4;
    static_assert(32 * LDP * 4 <= ZERO, "patch fits");
    float* patch = reinterpret_cast<float*>(lds);
#pragma unroll
    for (int i = 0; i < TN; ++i) {
      __syncthreads();
#pragma unroll
      for (int e = 0; e < 16; ++e) patch[(e / 4 * 8 + half * 4 + e % 4) * LDP + trel] = acc[i][0][e];
      __syncthreads();
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int id = tid + u * 512, ch = id / (TOK / 8), t8 = (id % (TOK / 8)) * 8;
        const int n = (col * TN + i) * 32 + ch;
        if (n < a.O && m0 + t8 < M) {
          const float4 lo = *reinterpret_cast<const float4*>(patch + ch * LDP + t8);
          const float4 hi = *reinterpret_cast<const float4*>(patch + ch * LDP + t8 + 4);
          const float v[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
          epi.rows8(m0 + t8, n, v, a.M);
        }
      }
    }
  } else {
    if (m0 + trel >= M) return;
#pragma unroll
    for (int i = 0; i < TN; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int n = (col * TN + i) * 32 + q * 8 + half * 4;
        if (n < a.O) {
          const float v[4] = {acc[i][0][4 * q], acc[i][0][4 * q + 1], acc[i][0][4 * q + 2], acc[i][0][4 * q + 3]};
          epi(m0 + trel, n, v);
        }
      }
  }
}

}  // namespace si
