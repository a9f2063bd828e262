// Attention kernels.
//
// Sequences are described by strides so that one kernel serves the three uses:
//   temporal self-attention  sequence (b, p): rows b*Fw*Pw + p + i*Pw, i < F
//   spatial self-attention   sequence (b, f): rows (b*Fw + f)*Pw + i,  i < P
//   cross-attention          queries as spatial; keys/values = context rows of b
// Row r of sequence s:  base(s) + i*row_stride,  base(s) = (s / inner)*outer_stride
// + (s % inner)*inner_stride, separately for the query side and the key side.
#pragma once
#include "si_common.h"
#include "k_norm.h"

namespace si {

struct SeqMap {
  int inner;
  int64_t outer_stride, inner_stride, row_stride;
  __device__ __forceinline__ int64_t row(int s, int i) const {
    return (int64_t)(s / inner) * outer_stride + (int64_t)(s % inner) * inner_stride + (int64_t)i * row_stride;
  }
};

struct AttnArgs {
  const void *q, *k, *v;  // element type T; head h occupies columns [h*d, (h+1)*d)
  void* o;
  int64_t ldq, ldk, ldv, ldo;
  SeqMap qmap, kmap;
  int S, heads, d, Nq, Nk;
  float scale;
};

// Plain vector-ALU attention with an online (running max / running sum) softmax.
// One wavefront serves QB queries of one (sequence, head): in the score phase
// each lane owns one key of a 64-key chunk and forms QB dot products; in the
// value phase each lane owns channels lane and lane+64 (d <= 128).  Exact expf,
// fp32 throughout: this is the path of the staged fp32 block (16-bit storage takes
// attn_short_kernel and attn_f32mma_kernel, the same arithmetic on fp32 matrix
// instructions).
template <typename T, int QB>
__global__ __launch_bounds__(256) void attn_valu_kernel(AttnArgs a) {
  __shared__ float qs[4][QB][128];
  __shared__ float ps[4][QB][kWave];
  const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
  const int s = blockIdx.z, head = blockIdx.y;
  const int q0 = (blockIdx.x * 4 + wave) * QB;
  if (q0 >= a.Nq) return;  // whole wavefront leaves; no block-wide barrier is used below
  const T* Q = static_cast<const T*>(a.q);
  const T* Kp = static_cast<const T*>(a.k);
  const T* Vp = static_cast<const T*>(a.v);
  T* O = static_cast<T*>(a.o);
  const int d = a.d, hc = head * d;

  for (int i = lane; i < QB * d; i += kWave) {
    const int qi = i / d, c = i % d;
    float v = 0.f;
    if (q0 + qi < a.Nq) v = to_float(Q[a.qmap.row(s, q0 + qi) * a.ldq + hc + c]) * a.scale;
    qs[wave][qi][c] = v;
  }
  __builtin_amdgcn_wave_barrier();  // LDS operations of one wavefront complete in program order

  float mrun[QB], lrun[QB], o0[QB], o1[QB];
#pragma unroll
  for (int qi = 0; qi < QB; ++qi) {
    mrun[qi] = -INFINITY;
    lrun[qi] = 0.f;
    o0[qi] = 0.f;
    o1[qi] = 0.f;
  }
  const int c0 = lane, c1 = lane + kWave;
  for (int kc = 0; kc < a.Nk; kc += kWave) {
    const int kj = kc + lane;
    const bool valid = kj < a.Nk;
    float sc[QB];
#pragma unroll
    for (int qi = 0; qi < QB; ++qi) sc[qi] = 0.f;
    if (valid) {
      const T* krow = Kp + a.kmap.row(s, kj) * a.ldk + hc;
      for (int c = 0; c < d; ++c) {
        const float kv = to_float(krow[c]);
#pragma unroll
        for (int qi = 0; qi < QB; ++qi) sc[qi] = fmaf(qs[wave][qi][c], kv, sc[qi]);
      }
    }
    float alpha[QB];
#pragma unroll
    for (int qi = 0; qi < QB; ++qi) {
      const float cm = wave_max(valid ? sc[qi] : -INFINITY);
      const float mn = fmaxf(mrun[qi], cm);
      const float p = valid ? expf(sc[qi] - mn) : 0.f;
      alpha[qi] = expf(mrun[qi] - mn);  // first chunk: exp(-inf) = 0
      lrun[qi] = lrun[qi] * alpha[qi] + wave_sum(p);
      mrun[qi] = mn;
      ps[wave][qi][lane] = p;
      o0[qi] *= alpha[qi];
      o1[qi] *= alpha[qi];
    }
    __builtin_amdgcn_wave_barrier();
    const int nvalid = min(kWave, a.Nk - kc);
    for (int j = 0; j < nvalid; ++j) {
      const T* vrow = Vp + a.kmap.row(s, kc + j) * a.ldv + hc;
      const float v0 = c0 < d ? to_float(vrow[c0]) : 0.f;
      const float v1 = c1 < d ? to_float(vrow[c1]) : 0.f;
#pragma unroll
      for (int qi = 0; qi < QB; ++qi) {
        const float p = ps[wave][qi][j];
        o0[qi] = fmaf(p, v0, o0[qi]);
        o1[qi] = fmaf(p, v1, o1[qi]);
      }
    }
    __builtin_amdgcn_wave_barrier();
  }
#pragma unroll
  for (int qi = 0; qi < QB; ++qi) {
    if (q0 + qi >= a.Nq) continue;
    T* orow = O + a.qmap.row(s, q0 + qi) * a.ldo + hc;
    const float inv = 1.f / lrun[qi];
    if (c0 < d) orow[c0] = from_float<T>(o0[qi] * inv);
    if (c1 < d) orow[c1] = from_float<T>(o1[qi] * inv);
  }
}

// Short sequences in 16-bit storage (at most 32 tokens per sequence: temporal blocks on the staged path, small maps),
// head dimension d = 8 D8, on the fp32 matrix instructions: one wavefront per (sequence, head), no LDS.  Scores,
// probabilities and sums are fp32 with exact expf; v_mfma_f32_16x16x4_f32 is a chain of fused multiply-adds in k order,
// so the results are those of the vector ALUs that worked channel by channel and key by key.
// FT: 16-token tiles.  Operands as in attn_f32mma_kernel: S^T = K Q^T with key 4 j + g of a tile in register j of lane
// group g, whose probabilities are then the column operand of O^T += V^T P^T.  A lane loads 16-byte pieces of its q and
// k rows (group g of every four); two lane-half exchanges hand it the channels 4 s + g that the products want.
// Row sums: heads of 64 add even and odd keys in sequence, the halves last; others add by halving, as a reduction over
// 64 lanes does.  Both orders are what results of these calls have always had.
// Bound by the gather of q/k/v rows, which lie Pw rows apart: a workgroup takes one head of 4 consecutive sequences
// (adjacent token rows on either side), the heads of those sequences follow each other, and every XCD gets a
// contiguous share of that list, so that an L2 sees whole lines.  500 sequences of 14 frames, 8 heads of 80: 54.7 us
// (attn_valu_kernel) -> 12.6; 128 of 16 frames, 20 heads of 64: 21.3 us (one lane per query) -> 10.5.
// o_frag: 0, or o is a fragment-order buffer of that many channels per token.
template <int D8, int FT>
__global__ __launch_bounds__(256) void attn_short_kernel(AttnArgs a, int o_frag) {
  constexpr int NS = 2 * D8, NB = (D8 + 3) / 4, DB = (D8 + 1) / 2;  // steps of 4 channels, 32-channel loads, 16-channel blocks
  const int lane = threadIdx.x % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int r = lane % 16, g = lane / 16;
  const unsigned short* Q = static_cast<const unsigned short*>(a.q);
  const unsigned short* Kp = static_cast<const unsigned short*>(a.k);
  const unsigned short* Vp = static_cast<const unsigned short*>(a.v);
  unsigned short* O = static_cast<unsigned short*>(a.o);
  const int F = a.Nk;
  const int64_t ntiles = (int64_t)((a.S + 3) / 4) * a.heads, chunk = (ntiles + 7) / 8;
  for (int64_t it = blockIdx.x / 8; it < chunk; it += gridDim.x / 8) {
    const int64_t work = (int64_t)(blockIdx.x % 8) * chunk + it;
    if (work >= ntiles) return;
    const int s = (int)(work / a.heads) * 4 + wave, hc = (int)(work % a.heads) * a.d;
    if (s >= a.S) continue;  // no barrier below

    // rows past the sequence repeat its last one, pieces past the head its last one: their scores are overwritten,
    // their values cleared, their columns and channels not stored
    u32x4_t qr[FT][NB], kr[FT][NB];
    float vf[FT][4][DB];
#pragma unroll
    for (int t = 0; t < FT; ++t) {
      const int qi = 16 * t + r, ki = 16 * t + 4 * (r % 4) + r / 4;
      const unsigned short* qrow = Q + a.qmap.row(s, qi < F ? qi : F - 1) * a.ldq + hc;
      const unsigned short* krow = Kp + a.kmap.row(s, ki < F ? ki : F - 1) * a.ldk + hc;
#pragma unroll
      for (int n = 0; n < NB; ++n) {
        const int c8 = 4 * n + g < D8 ? 4 * n + g : D8 - 1;
        qr[t][n] = *reinterpret_cast<const u32x4_t*>(qrow + 8 * c8);
        kr[t][n] = *reinterpret_cast<const u32x4_t*>(krow + 8 * c8);
      }
    }
#pragma unroll
    for (int t = 0; t < FT; ++t)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int vi = 16 * t + 4 * j + g;
        const unsigned short* vrow = Vp + a.kmap.row(s, vi < F ? vi : F - 1) * a.ldv + hc;
#pragma unroll
        for (int b = 0; b < DB; ++b) {
          const float v = bf16_bits_to_float(vrow[16 * b + r < 8 * D8 ? 16 * b + r : r % 8]);
          vf[t][j][b] = vi < F ? v : 0.f;
        }
      }
    // step st of a row whose pieces 4 n + g the lane groups hold: channel 4 st + g
    auto steps = [&](const u32x4_t(&raw)[NB], float(&out)[NS]) {
#pragma unroll
      for (int n = 0; n < NB; ++n) {
        unsigned v[8];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          v[2 * e] = raw[n][e] << 16;
          v[2 * e + 1] = raw[n][e] & 0xffff0000u;
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) {  // channels 4 h .. + 3 of the piece: group bits and channel bits change places
          const auto x0 = __builtin_amdgcn_permlane32_swap(v[4 * h], v[4 * h + 2], false, false);
          const auto x1 = __builtin_amdgcn_permlane32_swap(v[4 * h + 1], v[4 * h + 3], false, false);
          const auto y0 = __builtin_amdgcn_permlane16_swap(x0[0], x1[0], false, false);  // pieces 0, 1
          const auto y1 = __builtin_amdgcn_permlane16_swap(x0[1], x1[1], false, false);  // pieces 2, 3
          const unsigned p[4] = {y0[0], y0[1], y1[0], y1[1]};
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (8 * n + 2 * i + h < NS) out[8 * n + 2 * i + h] = __uint_as_float(p[i]);
        }
      }
    };
    const f32x4_t zero = f32x4_t{0.f, 0.f, 0.f, 0.f};
    f32x4_t sc[FT][FT];  // [query tile][key tile]
    {
      float kf[FT][NS];
#pragma unroll
      for (int t = 0; t < FT; ++t) steps(kr[t], kf[t]);
#pragma unroll
      for (int u = 0; u < FT; ++u) {
        float qf[NS];
        steps(qr[u], qf);
#pragma unroll
        for (int t = 0; t < FT; ++t) sc[u][t] = zero;
#pragma unroll
        for (int i = 0; i < NS; ++i)
#pragma unroll
          for (int t = 0; t < FT; ++t) sc[u][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[t][i], qf[i] * a.scale, sc[u][t], 0, 0, 0);
      }
    }
#pragma unroll
    for (int u = 0; u < FT; ++u) {
      float m = -INFINITY;
#pragma unroll
      for (int t = 0; t < FT; ++t)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          if (16 * t + 4 * j + g >= F) sc[u][t][j] = -INFINITY;
          m = fmaxf(m, sc[u][t][j]);
        }
      m = fmaxf(m, __shfl_xor(m, 32, kWave));
      m = fmaxf(m, __shfl_xor(m, 16, kWave));
#pragma unroll
      for (int t = 0; t < FT; ++t)
#pragma unroll
        for (int j = 0; j < 4; ++j) sc[u][t][j] = expf(sc[u][t][j] - m);  // a key beyond the sequence: exp(-inf) = 0
      float l;
      if constexpr (D8 == 8) {  // even keys are in groups 0 and 2, odd ones in 1 and 3
        l = 0.f;
#pragma unroll
        for (int t = 0; t < FT; ++t)
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const float own = sc[u][t][j], other = __shfl_xor(own, 32, kWave);
            l += g & 2 ? other : own;
            l += g & 2 ? own : other;
          }
      } else {
        float p[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) p[j] = FT == 2 ? sc[u][0][j] + sc[u][FT - 1][j] : sc[u][0][j];
        l = (p[0] + p[2]) + (p[1] + p[3]);
        l += __shfl_xor(l, 32, kWave);
      }
      l += __shfl_xor(l, 16, kWave);
      const float inv = 1.f / l;
      f32x4_t o[DB];
#pragma unroll
      for (int b = 0; b < DB; ++b) o[b] = zero;
#pragma unroll
      for (int t = 0; t < FT; ++t)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
          for (int b = 0; b < DB; ++b) o[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[t][j][b], sc[u][t][j], o[b], 0, 0, 0);
      // register j of block b: channel 16 b + 4 g + j.  Of two blocks, one exchange between neighbouring groups leaves
      // even groups with a whole 16-byte piece of the first, odd ones with one of the second
      const int qi = 16 * u + r;
      const int64_t row = a.qmap.row(s, qi < F ? qi : 0);
      auto word = [&](int b, int i) {
        return (unsigned)float_to_bf16_bits(o[b][2 * i] * inv) | ((unsigned)float_to_bf16_bits(o[b][2 * i + 1] * inv) << 16);
      };
      auto dst = [&](int c) { return O + (o_frag ? act_offset(row, hc + c, o_frag) : row * a.ldo + hc + c); };
#pragma unroll
      for (int b = 0; b + 1 < DB; b += 2) {
        const auto x = __builtin_amdgcn_permlane16_swap(word(b, 0), word(b + 1, 0), false, false);
        const auto y = __builtin_amdgcn_permlane16_swap(word(b, 1), word(b + 1, 1), false, false);
        const int c = 16 * (b + g % 2) + 8 * (g / 2);
        if (qi < F && c < 8 * D8) *reinterpret_cast<u32x4_t*>(dst(c)) = u32x4_t{x[0], y[0], x[1], y[1]};
      }
      if constexpr (DB % 2 == 1) {
        const int c = 16 * (DB - 1) + 4 * g;
        if (qi < F && c < 8 * D8) *reinterpret_cast<uint2*>(dst(c)) = make_uint2(word(DB - 1, 0), word(DB - 1, 1));
      }
    }
  }
}

}  // namespace si
