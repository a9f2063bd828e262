// DownSample: 3x3 convolution of stride 2 that reads the feature as it lies in memory -- [image][channel][position], bf16 --
// and therefore takes every window of a call in one launch: no operand buffer, no slice-in pass.  Calls of many windows or
// of many full tiles run on it (down_pays, si_resblock_api.h), the others on the ring kernel, summing in the same order.
//
// What bounded the ring kernel (k_conv.h) here was delivery, every source token once per tap, and launches of 180
// workgroups with a copy pass of 12 us before each.  A workgroup of 8 wavefronts owns 256 consecutive output positions of
// one image x 320 output channels; wavefront (pair, chalf) the pair's 64 positions x the 160 channels of its half: per 16
// input channels and tap 7 KiB of LDS reads for 10 MFMAs.  A chunk of 16 input channels passes through LDS as a patch -- the
// source positions that any tap of the 256 outputs reads are consecutive in memory -- and is read at nine shifts.  Patch
// values travel memory -> registers -> (transposed) LDS one chunk ahead; weights memory -> LDS directly, three taps
// (30 KiB) at a time.  Even and odd source positions lie in separate halves of the patch, so that the outputs of a
// wavefront read consecutive granules; which half a tap reads and how far it is shifted is the same for all lanes.
// 320 channels, 72 x 128 -> 36 x 64, 50 frames (212 GFLOP), whole call: ring kernel 575 us, this one 211 us; 1280 channels,
// 18 x 32, 32 frames 887 -> 311 us.  In the kernel (cycles per tap, 660 of them MFMAs of a SIMD's two wavefronts): 836 as it
// is, 682 with the patch left alone; 916 when both wavefronts of a SIMD converted at the same time.  Per workgroup 150 k
// cycles are taps, 30 k prologue and epilogue; 450 workgroups make 1.8 rounds.
#pragma once
#include "k_conv.h"

namespace si {

constexpr int kDownTokens = 256, kDownTN = 10;  // output positions and 32-channel blocks of a workgroup

struct ConvDownArgs {
  const bf16* src;   // element (image, c, p) at (image / F * C + c) * F * P + image % F * P + p
  bf16* out;         // the same of O channels, Po positions
  const bf16* bias;  // may be NULL
  const char* wf;    // fragment-ordered kernel, column tiles of 320 channels (pack_conv_kernel, CHUNKS)
  int C, O, F;       // input / output channels, frames per batch entry
  int W, H, P;       // source map
  int Wo, Po;        // output map
  int ntile, ncol;   // 256-position tiles per image, 320-channel tiles
  int nwg;           // images * ntile * ncol
};

// First source position (a multiple of 4) and position count of the patch of output positions [m0, m1] of an image
__host__ __device__ inline void down_patch(int m0, int m1, int W, int Wo, int* s0, int* n) {
  *s0 = ((2 * (m0 / Wo) - 1) * W + 2 * (m0 % Wo) - 1) & ~3;
  *n = (2 * (m1 / Wo) + 1) * W + 2 * (m1 % Wo) + 2 - *s0;
}

constexpr int kDownGroups = 352;  // groups of four source positions that a patch has room for

// Granule v of a plane lies at 16 * swizzle(v): the positions that a wavefront writes at once, four or two apart, spread
// over the banks (sixteen-fold conflicts otherwise), those it reads stay a permutation of 64 consecutive bytes.
__device__ __forceinline__ int swizzle(int v) { return v ^ ((v >> 4) & 3); }

__global__ __launch_bounds__(512, 2) void conv_down_kernel(ConvDownArgs a) {
  constexpr int TM = 2, TN = 5;              // 32-position row tiles, 32-channel blocks of a wavefront
  constexpr int WFR = kDownTN;             // weight fragments of a tap
  constexpr int WST = 3 * WFR * 1024;        // weights of a stage
  constexpr int PLANE = kDownGroups * 4 * 16;  // a patch: 2 planes [8-channel granule][position], 16 bytes each
  constexpr int AST = 2 * PLANE;
  constexpr int ZERO = 2 * WST + 2 * AST;    // 16 zero bytes: what a tap outside the image reads
  constexpr int U = (kDownGroups + 127) / 128;  // patch units (4 positions x 4 channels) per thread
  __shared__ __attribute__((aligned(1024))) char lds[ZERO + 64];

  const int share = (a.nwg + 7) / 8;  // consecutive tiles stay on one XCD
  const int wg = (blockIdx.x % 8) * share + blockIdx.x / 8;
  if (wg >= a.nwg) return;
  const int col = wg % a.ncol, tile = wg / a.ncol % a.ntile, img = wg / (a.ncol * a.ntile);
  const int64_t fP = (int64_t)a.F * a.P, fPo = (int64_t)a.F * a.Po;  // channel strides
  const int b = img / a.F, f = img - b * a.F;
  const int m0 = tile * kDownTokens;

  const int tid = threadIdx.x, lane = tid % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int pair = wave >> 1, chalf = wave & 1;
  const int trow = lane % 32, half = lane / 32;
  const int nch = a.C / 16;

  int s0, npos;
  down_patch(m0, (m0 + kDownTokens < a.Po ? m0 + kDownTokens : a.Po) - 1, a.W, a.Wo, &s0, &npos);
  const int ngrp = (npos + 3) / 4;

  // ---- weights: load i of this wavefront fetches fragment id = wave + 8 i of a stage's 30 (ids past them repeat the last)
  const unsigned lds0 = (unsigned)(size_t)(__attribute__((address_space(3))) void*)lds;
  constexpr int NLW = (3 * WFR + 7) / 8;
  const char* wchunk = a.wf + (int64_t)col * nch * (3 * WST);  // the current chunk's three stages
  unsigned wsrc[NLW];
#pragma unroll
  for (int i = 0; i < NLW; ++i) wsrc[i] = (unsigned)(wave + 8 * i < 3 * WFR ? wave + 8 * i : 3 * WFR - 1) * 1024;
  auto load_w = [&](const char* row, int i, int buf) {
    asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dwordx4 %0, %1"
                 :
                 : "v"((unsigned)(lane * 16)), "s"(row + wsrc[i]), "s"(lds0 + wsrc[i] + (unsigned)(buf * WST))
                 : "memory");
  };
  // i-th load of what takes the place of stage (cc, r) when everybody has left it: the stage after the next.  Past the
  // last chunk the last one is fetched once more, into slots nobody reads.  wchunk is chunk wc's.
  auto refill = [&](int cc, int wc, int r, int i) {
    const int ahead = (r == 0 ? cc : cc + 1) - wc;
    load_w(wchunk + (ahead && wc + 1 < nch ? 3 * WST : 0) + (r == 0 ? 2 : r - 1) * WST, i, (cc + r) & 1);
  };

  // ---- patch: unit u of a thread is the chunk's channels 4 * quad .. + 3 at the positions of one group.
  // Groups that hold no position of the image read its first positions; the last group of an image whose size is no
  // multiple of 4 is read from its last four positions and shifted into place.
  const int quad = wave & 3;
  const bf16* simg = a.src + (int64_t)b * a.C * fP + (int64_t)f * a.P;
  int group0 = (wave >> 2) * 64 + lane;
  uint2 pv[U][4];
  auto load_patch = [&](int cc, int u) {
    int p = s0 + 4 * (group0 + 128 * u);
    if (p < 0 || p >= a.P) p = 0;
    if (p > a.P - 4) p = a.P - 4;
    const bf16* cb = simg + (int64_t)((cc < nch ? cc : nch - 1) * 16 + 4 * quad) * fP;
#pragma unroll
    for (int k = 0; k < 4; ++k) __builtin_memcpy(&pv[u][k], cb + k * fP + p, 8);
  };
  // positions 2 h, 2 h + 1 of unit u, chunk cc, into their patch
  auto store_patch = [&](int cc, int u, int h) {
    const int g = group0 + 128 * u;
    if ((wave >> 2) * 64 + 128 * u >= ngrp) return;  // nobody in this wavefront has a group
    unsigned w[4];  // the two positions of the four channels
#pragma unroll
    for (int k = 0; k < 4; ++k) w[k] = h ? pv[u][k].y : pv[u][k].x;
    if (a.P & 3) {
      const int p = s0 + 4 * g, late = p < a.P && p > a.P - 4 ? 16 * (p - (a.P - 4)) : 0;
#pragma unroll
      for (int k = 0; k < 4; ++k) w[k] = (unsigned)((((uint64_t)pv[u][k].y << 32) | pv[u][k].x) >> late >> (32 * h));
    }
    if (g < ngrp) {
      char* d = lds + 2 * WST + (cc & 1) * AST + (quad >> 1) * PLANE + 8 * (quad & 1) + 16 * swizzle(2 * g + h);
      *reinterpret_cast<uint2*>(d) = make_uint2(__builtin_amdgcn_perm(w[1], w[0], 0x05040100u), __builtin_amdgcn_perm(w[3], w[2], 0x05040100u));
      *reinterpret_cast<uint2*>(d + PLANE / 2) =
          make_uint2(__builtin_amdgcn_perm(w[1], w[0], 0x07060302u), __builtin_amdgcn_perm(w[3], w[2], 0x07060302u));
    }
  };

#pragma unroll
  for (int u = 0; u < U; ++u) load_patch(0, u);
#pragma unroll
  for (int i = 0; i < NLW; ++i) load_w(wchunk, i, 0);
#pragma unroll
  for (int i = 0; i < 1; ++i) load_w(wchunk + WST, i, 1);
  if (tid < 4) *reinterpret_cast<unsigned*>(lds + ZERO + 4 * tid) = 0u;
  // per row tile: the lane's source granule at the centre tap; bit t of the mask: tap t lies inside the image
  int base[TM], mask[TM];
#pragma unroll
  for (int j = 0; j < TM; ++j) {
    const int tok = m0 + pair * 64 + j * 32 + trow;
    const int y = tok / a.Wo, x = tok - y * a.Wo;
    base[j] = (2 * y * a.W + 2 * x - s0) >> 1;  // s0 is even
    mask[j] = 0;
#pragma unroll
    for (int t = 0; t < 9; ++t)
      if (tok < a.Po && (unsigned)(2 * y + t / 3 - 1) < (unsigned)a.H && (unsigned)(2 * x + t % 3 - 1) < (unsigned)a.W) mask[j] |= 1 << t;
  }
#pragma unroll
  for (int u = 0; u < U; ++u) {
    store_patch(0, u, 0);
    store_patch(0, u, 1);
  }

  f32x16_t acc[TN][TM];
#pragma unroll
  for (int i = 0; i < TN; ++i)
#pragma unroll
    for (int j = 0; j < TM; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

  // Fragments: a weight fragment serves the TM MFMAs of one step and is read two steps ahead, the next tap's
  // activations two or three.
  u32x4_t wf[TN], af[2][TM];
  auto read_w = [&](int cc, int r, int t, int i) {
    return *reinterpret_cast<const u32x4_t*>(lds + ((cc + r) & 1) * WST + (t * WFR + chalf * TN + i) * 1024 + lane * 16);
  };
  auto read_a = [&](int cc, int r, int t, int j) {
    const int d = (r - 1) * a.W + t - 1;  // odd shifts read the odd half
    const int plane = 2 * WST + (cc & 1) * AST + (d & 1 ? PLANE / 2 : 0);
    const int at = half * PLANE + plane + 16 * swizzle(base[j] + (d >> 1));
    return *reinterpret_cast<const u32x4_t*>(lds + (mask[j] & (1 << (3 * r + t)) ? at : ZERO));
  };
  auto mma = [&](const u32x4_t& w, const u32x4_t& x, f32x16_t& c) {
    c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, w), __builtin_bit_cast(bf16x8_t, x), c, 0, 0, 0);
  };
  // all but this wavefront's last `flying` loads have landed and its LDS accesses are done; then everybody's
  auto stage_barrier = [&](auto flying) {
    constexpr int n = decltype(flying)::value;
    __builtin_amdgcn_s_waitcnt(0x0070 | (n & 15) | (n >> 4) << 14);  // vmcnt(n) lgkmcnt(0)
    __syncthreads();
  };
  using All = std::integral_constant<int, 0>;

  stage_barrier(All());
#pragma unroll
  for (int u = 0; u < U; ++u) load_patch(1, u);
#pragma unroll
  for (int j = 0; j < TM; ++j) af[0][j] = read_a(0, 0, 0, j);
#pragma unroll
  for (int i = 0; i < TN - 3; ++i) wf[i] = read_w(0, 0, 0, i);
  static_assert(TN == 5 && TM == 2, "step order");
  // The next chunk's patch goes into LDS while this one is contracted, half a unit at a time.  The two wavefronts of a SIMD
  // (w and w + 4) take turns: while one converts, with priority, the other's MFMAs run, and the stage ends for both at
  // once; a wavefront that converted behind the other's back would hold everybody up at the barrier.  Units 0 and 1:
  // wavefronts 0-3 in stage 1, 4-7 in stage 2; unit 2 (few patches are that large) in stage 0.  A unit is requested again
  // behind its conversion.
  auto contract = [&](auto later) {
    constexpr int L = decltype(later)::value;  // 1: wavefronts 4-7
    static_assert(U == 3, "units");
    constexpr auto jobs = [](int r) { return r == 0 ? 2 : r == 1 + L ? 4 : 0; };               // conversions of stage r
    constexpr auto job = [](int r, int k) { return r == 0 ? 4 + k : k; };                      // the k-th: 2 unit + half
    constexpr auto asks = [](int r) { return r == 0 ? 1 : r == 1 + L ? 2 : 0; };               // requests of stage r
    constexpr auto ask = [](int r, int k) { return r == 0 ? 2 : k; };                          // the k-th: unit
    auto end_stage = [&](auto row) {
      constexpr int r = decltype(row)::value;
      // the requests are the youngest loads of their stage
      stage_barrier(std::integral_constant<int, 4 * asks(r)>());
      __builtin_amdgcn_s_setprio(jobs((r + 1) % 3) > 0 ? 2 : 0);
    };
    for (int cc = 0; cc < nch; ++cc) {
      // opaque: addresses that follow from these are not to be kept in registers across chunks
#pragma unroll
      for (int j = 0; j < TM; ++j) asm volatile("" : "+v"(base[j]), "+v"(mask[j]));
      asm volatile("" : "+v"(group0));
#pragma unroll
      for (int tap = 0; tap < 9; ++tap) {
        const int r = tap / 3, t = tap % 3;
        // the tap behind this one (past the last chunk the reads go on, into registers nobody uses: no branch)
        const int ntap = (tap + 1) % 9, ncc = tap == 8 ? cc + 1 : cc;
#pragma unroll
        for (int i = 0; i < TN; ++i) {
          // Nobody reads this stage any more (its last fragments are in registers); the next one's weights have had a
          // stage to land, and so have patch loads of the stage before.
          if (t == 2 && i == 3) {
            if (r == 0) end_stage(std::integral_constant<int, 0>());
            else if (r == 1) end_stage(std::integral_constant<int, 1>());
            else end_stage(std::integral_constant<int, 2>());
          }
          if (i < 3) wf[i + 2] = read_w(cc, r, t, i + 2);
          else wf[i - 3] = read_w(ncc, ntap / 3, ntap % 3, i - 3);
          if (tap == 8 ? i >= 3 : i == 2 || i == 3) af[(tap + 1) & 1][tap == 8 ? i - 3 : i - 2] = read_a(ncc, ntap / 3, ntap % 3, tap == 8 ? i - 3 : i - 2);
          const int at = t * TN + i;  // step of the stage
#pragma unroll
          for (int j = 0; j < TM; ++j) mma(wf[i], af[tap & 1][j], acc[i][j]);
          // the loads of a refill, one every other step from the barrier on
          const int since = t == 2 ? i - 3 : at + 2;  // steps behind the barrier
          __builtin_amdgcn_sched_barrier(0);
          if (t == 2 && since >= 0 && since % 2 == 0) refill(cc, cc, r, since / 2);
          else if (t < 2 && since % 2 == 0 && since / 2 < NLW) refill(r == 0 ? cc - 1 : cc, cc, r == 0 ? 2 : r - 1, since / 2);
          __builtin_amdgcn_sched_barrier(0);
          const int first = jobs(r) < 5 ? 5 : jobs(r);  // behind the last load of the refill
          if (at < jobs(r)) store_patch(cc + 1, job(r, at) / 2, job(r, at) % 2);
          else if (at >= first && at < first + asks(r)) load_patch(cc + 2, ask(r, at - first));
        }
      }
#pragma unroll
      for (int j = 0; j < TM; ++j) af[0][j] = af[1][j];
      if (cc + 1 < nch) wchunk += 3 * WST;
    }
    __builtin_amdgcn_s_setprio(0);
  };
  if (wave < 4) contract(std::integral_constant<int, 0>());
  else contract(std::integral_constant<int, 1>());
  stage_barrier(All());

  // ---- 8 consecutive positions of one channel at a time, transposed through LDS: 16 channels of block i of either half
  // per step, in two buffers, so that a step's reads and stores run beside the next one's writes
  constexpr int LDP = kDownTokens + 8, BUF = 32 * LDP * 4;  // the halves of a wavefront write 32 banks apart
  static_assert(2 * BUF <= ZERO, "exchange fits");
  const int t8 = (tid % 32) * 8, p8 = m0 + t8;
  auto chan = [&](int k, int u) { return (col * kDownTN + u * TN + k / 2) * 32 + (k % 2) * 16 + tid / 32; };
  const bool whole = a.Po % 8 == 0;  // every row of the output is 16-byte aligned
  bf16* oimg = a.out + (int64_t)b * a.O * fPo + (int64_t)f * a.Po + p8;
  float bias[2][2];
  auto request = [&](int k) {
#pragma unroll
    for (int u = 0; u < 2; ++u) bias[k & 1][u] = param_or(a.bias, chan(k, u), 0.f);
  };
  request(0);
#pragma unroll
  for (int k = 0; k < 2 * TN; ++k) {
    float* patch = reinterpret_cast<float*>(lds + (k & 1) * BUF);
    if (k + 1 < 2 * TN) request(k + 1);
#pragma unroll
    for (int j = 0; j < TM; ++j)
#pragma unroll
      for (int e = 0; e < 8; ++e)
        patch[(chalf * 16 + e / 4 * 8 + half * 4 + e % 4) * LDP + pair * 64 + j * 32 + trow] = acc[k / 2][j][(k % 2) * 8 + e];
    __syncthreads();
    if (p8 < a.Po) {
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const float* row = patch + (u * 16 + tid / 32) * LDP + t8;
        const float4 lo = *reinterpret_cast<const float4*>(row);
        const float4 hi = *reinterpret_cast<const float4*>(row + 4);
        const float v[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w}, bn = bias[k & 1][u];
        bf16* o = oimg + chan(k, u) * fPo;
        if (whole) {
          u32x4_t w;
#pragma unroll
          for (int q = 0; q < 4; ++q)
            w[q] = (unsigned)float_to_bf16_bits(v[2 * q] + bn) | ((unsigned)float_to_bf16_bits(v[2 * q + 1] + bn) << 16);
          *reinterpret_cast<u32x4_t*>(o) = w;
        } else {
#pragma unroll
          for (int q = 0; q < 8; ++q)
            if (p8 + q < a.Po) o[q] = from_float<bf16>(v[q] + bn);
        }
      }
    }
  }
}

}  // namespace si
