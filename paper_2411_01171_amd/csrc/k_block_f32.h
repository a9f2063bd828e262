// The whole temporal block in single precision, one launch: slice-in, proj_in, LN1 (+ frame embedding), q/k/v,
// attention, out-projection, LN3, GEGLU FFN, proj_out, residual and slice-out, for every window of the call.
//
// A workgroup takes as many whole sequences (positions) as fill 16 TT token columns and keeps everything of
// them in LDS, channel-major ([channel][token]), so a window has no intermediates in memory and nothing needs
// to be ordered between windows: a grid covers them all.  The contractions run on v_mfma_f32_16x16x4_f32 (fp32
// operands, fp32 accumulation in k order): the weight is the row operand, read from the caller's [K, N] matrix
// as it is (a lane's element (k, n): four 64-byte pieces per load), the tokens are the column operand, one
// LDS read of 64 consecutive floats (TT = 1; with TT = 2 four pieces of 16, two of which share their banks).  The next 64 k-values of weight are loaded before the MFMAs
// of the current ones, the first ones of the next contraction before the barriers in between.
//
// The results are those of the staged fp32 kernels bit for bit, so that a call's windows may take either: the matrix
// instruction is a chain of fused multiply-adds in k order, as gemm_f32_kernel's and attn_valu_kernel's loops are, and
// the sums of LayerNorm and softmax are added in layer_norm_kernel's and attn_valu_kernel's order.
//
// Whole calls, staged kernels (one launch per operator and window, 49 in the first row) -> this kernel:
//   D 64, 8 frames of 8x8, B 1                  454 -> 26 us
//   D 64, 16 frames of 20x20, B 2, 4 windows    494 -> 72 us
//   D 128, 16 frames of 20x20, B 2, 4 windows   836 -> 175 us
//   D 320, 16 frames of 20x20, B 2, 4 windows  1974 -> 960 us
// Bound: small calls by the chain of some fifteen barriers and weight round trips (L2), large ones by the fp32
// matrix rate (256 flop per clock and CU) and the weight stream, 64 D^2 + 8 C D bytes per 16 TT tokens.
#pragma once
#include "k_norm.h"
#include "si_common.h"

namespace si {

// Two instantiations per TT.  64 KiB of LDS and 8 wavefronts, so that two workgroups share a CU; else 16 wavefronts,
// which is what one workgroup needs to keep weight loads in flight (the kernel alone on 12800 tokens: D = 64 63 us with 8,
// 87 us with 16; D = 320 1128 us with 8, 945 us with 16; twice as many k-steps in flight per wavefront gain 0 .. 6 % at D >= 128
// and lose 25 % on a call of 512 tokens).
constexpr int kF32SmallFloats = 16384, kF32SmallThreads = 512;
constexpr int kF32LdsFloats = 40960 - 512, kF32Threads = 1024;  // 160 KiB less the reduction scratch

struct BlockF32Args {
  const float* x;
  float* out;
  const float* stats;
  const float *gn_g, *gn_b, *w_in, *b_in, *ln1_g, *ln1_b, *wq, *wk, *wv, *wo, *bo, *ln3_g, *ln3_b, *w1, *b1, *w2, *b2, *w_out, *b_out;
  const float* pe;  // [F, D] or NULL
  int B, C, F, G, heads, d, D, nseq;  // sequences per workgroup
  int64_t P, groups, first;            // groups of nseq sequences of this launch, sequence that it starts at
  float ln_eps, scale;
};

// LDS rows (of 16 TT floats): residual stream, operand, and q/k/v + scores or the FFN's inner values
static inline int64_t block_f32_rows(int C, int D, int heads, int F) {
  const int64_t qkv = 3 * (int64_t)D + (int64_t)heads * (F + 1), ff = 4 * (int64_t)D;
  return D + (C > D ? C : D) + (qkv > ff ? qkv : ff);
}

// 32 token columns: at most 128 registers, so that two workgroups of the small form share a CU (20 frames at 64 channels,
// 6400 tokens: 77 us without the bound, 59 with it); 16 columns need 81 without a bound and lose 3 % with it.
template <int TT, int CAP, int NT>
__global__ __launch_bounds__(NT, TT == 1 ? 1 : 4) void temporal_block_f32_kernel(BlockF32Args a) {
  constexpr int TK = 16 * TT, NWV = NT / kWave;
  __shared__ float lds[CAP];
  __shared__ float red[NWV * TK];
  const int tid = threadIdx.x, lane = tid % kWave, wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int C = a.C, D = a.D, F = a.F;
  // consecutive groups on one XCD: they share the cache lines of their features
  const int64_t chunk = (a.groups + 7) / 8;
  const int64_t grp = (int64_t)(blockIdx.x % 8) * chunk + blockIdx.x / 8;
  if (grp >= a.groups) return;
  float* const hs = lds;
  float* const as = hs + D * TK;
  float* const bs = as + (C > D ? C : D) * TK;

  // token column t = (sequence i) * F + f
  const int64_t s0 = a.first + grp * a.nseq, S = (int64_t)a.B * a.P;
  const int nseq = (int)(s0 + a.nseq <= S ? a.nseq : S - s0), ntok = nseq * F;
  auto locate = [&](int t, int& b, int& f, int64_t& p) {
    const int i = t / F;
    f = t - i * F;
    const int64_t s = s0 + i;
    b = (int)(s / a.P);
    p = s - b * a.P;
  };

  // acc = sum_k W[k, n] act[k, t] for the wavefront's 16-column tiles; NS = 2: columns n and n + off together
  constexpr int KC = 16;  // k-steps of 4 in flight
  const int kl = lane / 16, nl = lane % 16;
  auto load_w = [&](auto ns_tag, float (&w)[KC], const float* W, int N, int K, int tiles, int it, int nchunk, int off) {
    constexpr int NS = decltype(ns_tag)::value, per = KC / NS;
    const int tile = wave + (it / nchunk) * NWV, k0 = (it % nchunk) * per * 4;
    if (tile >= tiles) return;
    const float* base = W + (int64_t)(k0 + kl) * N + tile * 16 + nl;
    if (k0 + per * 4 <= K) {  // a whole chunk: no branch between the loads
#pragma unroll
      for (int i = 0; i < KC; ++i) w[i] = base[(int64_t)(i / NS) * 4 * N + (i % NS) * off];
    } else {
#pragma unroll
      for (int i = 0; i < KC; ++i)
        if (k0 + i / NS * 4 < K) w[i] = base[(int64_t)(i / NS) * 4 * N + (i % NS) * off];
    }
  };
  // w0: the first chunk, loaded by the caller (load_w with it = 0)
  auto gemm = [&](auto ns_tag, float (&w0)[KC], const float* W, int N, int K, int cols, int off, const float* act, auto epi) {
    constexpr int NS = decltype(ns_tag)::value;
    constexpr int per = KC / NS;
    const int tiles = cols / 16, nchunk = (K + per * 4 - 1) / (per * 4);
    const int mine = wave < tiles ? (tiles - wave + NWV - 1) / NWV : 0;
    f32x4_t acc[NS][TT];
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
      for (int t = 0; t < TT; ++t) acc[s][t] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    for (int it = 0; it < mine * nchunk; ++it) {
      float w1[KC];
#pragma unroll
      for (int i = 0; i < KC; ++i) w1[i] = 0.f;
      if (it + 1 < mine * nchunk) load_w(ns_tag, w1, W, N, K, tiles, it + 1, nchunk, off);
      const int k0 = (it % nchunk) * per * 4;
      auto contract = [&](int ks) {
#pragma unroll
        for (int t = 0; t < TT; ++t) {
          const float v = act[(k0 + ks * 4 + kl) * TK + t * 16 + nl];
#pragma unroll
          for (int s = 0; s < NS; ++s) acc[s][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(w0[ks * NS + s], v, acc[s][t], 0, 0, 0);
        }
      };
      if (k0 + per * 4 <= K) {
#pragma unroll
        for (int ks = 0; ks < per; ++ks) contract(ks);
      } else {
#pragma unroll
        for (int ks = 0; ks < per; ++ks)
          if (k0 + ks * 4 < K) contract(ks);
      }
      if (it % nchunk == nchunk - 1) {
        const int n0 = (wave + (it / nchunk) * NWV) * 16 + kl * 4;
#pragma unroll
        for (int t = 0; t < TT; ++t)
#pragma unroll
          for (int r = 0; r < 4; ++r) epi(n0 + r, t * 16 + nl, acc[0][t][r], acc[NS - 1][t][r]);
#pragma unroll
        for (int s = 0; s < NS; ++s)
#pragma unroll
          for (int t = 0; t < TT; ++t) acc[s][t] = f32x4_t{0.f, 0.f, 0.f, 0.f};
      }
#pragma unroll
      for (int i = 0; i < KC; ++i) w0[i] = w1[i];
    }
  };
  auto first = [&](auto ns_tag, float (&w0)[KC], const float* W, int N, int K, int cols, int off) {
    constexpr int per = KC / decltype(ns_tag)::value;
#pragma unroll
    for (int i = 0; i < KC; ++i) w0[i] = 0.f;
    load_w(ns_tag, w0, W, N, K, cols / 16, 0, (K + per * 4 - 1) / (per * 4), off);
  };
  const std::integral_constant<int, 1> one;
  const std::integral_constant<int, 2> two;
  auto bias = [](const float* p, int n) { return p ? p[n] : 0.f; };

  // LayerNorm of the residual columns into `as`.  Sums in layer_norm_kernel's order: 64 partial sums, number L over the
  // rows 4 L .. + 3 of every 256, added by halves.  A thread forms RL of them (the top bits of L); the lanes of a wavefront
  // hold the next bits, the wavefronts the lowest.
  auto layer_norm = [&](const float* g, const float* bt, const float* pe) {
    constexpr int NP = NT / TK, RL = kWave / NP, PW = kWave / TK;
    const int t = tid % TK, part = tid / TK, pin = lane / TK;
    auto total = [&](auto quad) {
      float v[RL];
#pragma unroll
      for (int k = 0; k < RL; ++k) {
        v[k] = 0.f;
        for (int n = 4 * ((k * PW + pin) * NWV + wave); n < D; n += 4 * kWave) v[k] += quad(hs + n * TK + t);
      }
#pragma unroll
      for (int h = RL / 2; h > 0; h >>= 1)
#pragma unroll
        for (int k = 0; k < h; ++k) v[k] += v[k + h];
#pragma unroll
      for (int o = kWave / 2; o >= TK; o >>= 1) v[0] += __shfl_xor(v[0], o, kWave);
      __syncthreads();  // the previous use of red
      if (lane < TK) red[wave * TK + lane] = v[0];
      __syncthreads();
      float s[NWV];
#pragma unroll
      for (int w = 0; w < NWV; ++w) s[w] = red[w * TK + t];
#pragma unroll
      for (int h = NWV / 2; h > 0; h >>= 1)
#pragma unroll
        for (int w = 0; w < h; ++w) s[w] += s[w + h];
      return s[0];
    };
    const float mean = total([&](const float* x) { return (x[0] + x[TK]) + (x[2 * TK] + x[3 * TK]); }) / (float)D;
    const float rstd = rsqrtf(total([&](const float* x) {
                                const float dx = x[0] - mean, dy = x[TK] - mean, dz = x[2 * TK] - mean, dw = x[3 * TK] - mean;
                                return (dx * dx + dy * dy) + (dz * dz + dw * dw);
                              }) / (float)D + a.ln_eps);
    const float* perow = pe ? pe + (int64_t)(t % F) * D : nullptr;  // columns start at whole sequences
    for (int n = part; n < D; n += NP) {
      float y = (hs[n * TK + t] - mean) * rstd * (g ? g[n] : 1.f) + (bt ? bt[n] : 0.f);
      if (perow) y += perow[n];
      as[n * TK + t] = y;
    }
  };

  float w0[KC];
  first(one, w0, a.w_in, D, C, D, 0);
  {  // slice-in: normalised features; columns without a token hold zeros
    const int t = tid % TK, ng = C / a.G;
    int b = 0, f = 0;
    int64_t p = 0;
    if (t < ntok) locate(t, b, f, p);
    const float* st = a.stats + ((int64_t)b * F + f) * a.G * 2;
    const float* xp = a.x + ((int64_t)b * C * F + f) * a.P + p;
#pragma unroll 4
    for (int c = tid / TK; c < C; c += NT / TK) {
      float v = 0.f;
      if (t < ntok) {
        const int g = c / ng;
        v = (xp[(int64_t)c * F * a.P] - st[g * 2]) * st[g * 2 + 1] * (a.gn_g ? a.gn_g[c] : 1.f) + bias(a.gn_b, c);
      }
      as[c * TK + t] = v;
    }
  }
  __syncthreads();
  gemm(one, w0, a.w_in, D, C, D, 0, as, [&](int n, int t, float v, float) { hs[n * TK + t] = v + bias(a.b_in, n); });
  first(one, w0, a.wq, D, D, D, 0);
  __syncthreads();
  layer_norm(a.ln1_g, a.ln1_b, a.pe);
  __syncthreads();
  gemm(one, w0, a.wq, D, D, D, 0, as, [&](int n, int t, float v, float) { bs[n * TK + t] = v * a.scale; });
  first(one, w0, a.wk, D, D, D, 0);
  gemm(one, w0, a.wk, D, D, D, 0, as, [&](int n, int t, float v, float) { bs[(D + n) * TK + t] = v; });
  first(one, w0, a.wv, D, D, D, 0);
  gemm(one, w0, a.wv, D, D, D, 0, as, [&](int n, int t, float v, float) { bs[(2 * D + n) * TK + t] = v; });
  first(one, w0, a.wo, D, D, D, 0);
  __syncthreads();
  float* const sc = bs + 3 * D * TK;  // scores, then weights: row head * F + key; then the heads' 1 / row sum
  for (int e = tid; e < a.heads * F * TK; e += NT) {
    const int t = e % TK, hj = e / TK, h = hj / F, j = hj - h * F;
    if (t >= ntok) continue;
    const float* qp = bs + h * a.d * TK + t;
    const float* kp = bs + (D + h * a.d) * TK + t / F * F + j;
    float s = 0.f;
#pragma unroll 8
    for (int c = 0; c < a.d; ++c) s = fmaf(qp[c * TK], kp[c * TK], s);
    sc[e] = s;
  }
  __syncthreads();
  for (int e = tid; e < a.heads * TK; e += NT) {
    const int t = e % TK, h = e / TK;
    if (t >= ntok) continue;
    float* row = sc + h * F * TK + t;
    float m = -INFINITY, w[TK];  // F <= TK
#pragma unroll
    for (int j = 0; j < TK; ++j) {
      w[j] = row[(j < F ? j : 0) * TK];
      m = fmaxf(m, w[j]);
    }
#pragma unroll
    for (int j = 0; j < TK; ++j) {
      if (j < F) row[j * TK] = w[j] = expf(w[j] - m);
      else w[j] = 0.f;
    }
#pragma unroll
    for (int o = TK / 2; o > 0; o >>= 1)  // the row sum by halves, as attn_valu_kernel's lanes add theirs
#pragma unroll
      for (int j = 0; j < o; ++j) w[j] += w[j + o];
    sc[(a.heads * F + h) * TK + t] = 1.f / w[0];
  }
  __syncthreads();
  for (int e = tid; e < D * TK; e += NT) {
    const int t = e % TK, c = e / TK, h = c / a.d;
    float o = 0.f;
    if (t < ntok) {
      const float* wrow = sc + h * F * TK + t;
      const float* vp = bs + (2 * D + c) * TK + t / F * F;
      for (int j = 0; j < F; ++j) o = fmaf(wrow[j * TK], vp[j], o);
      o *= sc[(a.heads * F + h) * TK + t];
    }
    as[e] = o;
  }
  __syncthreads();
  gemm(one, w0, a.wo, D, D, D, 0, as, [&](int n, int t, float v, float) { hs[n * TK + t] += v + bias(a.bo, n); });
  first(two, w0, a.w1, 8 * D, D, 4 * D, 4 * D);
  __syncthreads();
  layer_norm(a.ln3_g, a.ln3_b, nullptr);
  __syncthreads();
  gemm(two, w0, a.w1, 8 * D, D, 4 * D, 4 * D, as, [&](int n, int t, float v, float g) {
    bs[n * TK + t] = (v + bias(a.b1, n)) * gelu_erf(g + bias(a.b1, 4 * D + n));
  });
  first(one, w0, a.w2, D, 4 * D, D, 0);
  __syncthreads();
  gemm(one, w0, a.w2, D, 4 * D, D, 0, bs, [&](int n, int t, float v, float) { hs[n * TK + t] += v + bias(a.b2, n); });
  first(one, w0, a.w_out, C, D, C, 0);
  __syncthreads();
  int ob[TT], of[TT];
  int64_t op[TT];
#pragma unroll
  for (int t = 0; t < TT; ++t) {
    ob[t] = of[t] = 0;
    op[t] = 0;
    if (t * 16 + nl < ntok) locate(t * 16 + nl, ob[t], of[t], op[t]);
  }
  gemm(one, w0, a.w_out, C, D, C, 0, hs, [&](int n, int t, float v, float) {
    if (t < ntok) {
      const int u = t / 16;  // a constant after unrolling
      const int64_t off = (((int64_t)ob[u] * C + n) * F + of[u]) * a.P + op[u];
      a.out[off] = a.x[off] + (v + bias(a.b_out, n));
    }
  });
}

}  // namespace si
