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
// fp32 throughout: this is the path of the fp32 block (16-bit storage takes
// attn_f32mma_kernel, the same arithmetic on fp32 matrix instructions).
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

// Short sequences in 16-bit storage (temporal blocks on the staged path: at most 32 tokens per
// sequence, any head dimension d = 8 .. 128, d % 8 == 0) on the matrix cores: one wavefront per
// (sequence, head), no LDS.  A lane's 16-byte pieces of the q, k and v rows are MFMA operands as they
// stand (lane (token r, half g): channels 16 ks + 8 g + e), so S^T[key, query] = K Q^T takes both
// straight from memory, and the softmax result registers are the column operand of O^T += V^T P^T.
// V^T comes from V by a product with the identity (V as row operand, 16-channel slices of I as column
// operand: exact, and the result registers are keys in the order P^T has them).  P enters as the sum of
// two bf16 values (p and what its rounding leaves), so the probabilities keep 16 significand bits.
// Bound by the gather of q/k/v rows, which lie Pw rows apart: a workgroup takes one head of 4 consecutive
// sequences (adjacent token rows on either side), the heads of those sequences follow each other, and
// every XCD gets a contiguous share of that list, so that an L2 sees whole lines.
// 500 sequences of 14 frames, 8 heads of 80: 54.7 us (vector-ALU online softmax) -> 13.4; 128 of 16
// frames, 20 heads of 64: 21.3 us (one lane per query, fp32 dot products) -> 12.7, and the out-projection
// behind it reads fragments instead of rows (24.1 -> 20.7 us).
// o_frag: o is a fragment-order buffer of that many channels per token instead of rows.
template <int KS, int DB>
__global__ __launch_bounds__(256, KS <= 5 ? 4 : 2) void attn_short_kernel(AttnArgs a, int o_frag) {
  const int lane = threadIdx.x % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int r = lane % 32, g = lane / 32;
  const int groups = (a.S + 3) / 4, ntiles = groups * a.heads, chunk = (ntiles + 7) / 8;
  const int work = (int)(blockIdx.x % 8) * chunk + (int)(blockIdx.x / 8);
  if (work >= ntiles || (int)(blockIdx.x / 8) >= chunk) return;
  const int s = (work / a.heads) * 4 + wave, hc = (work % a.heads) * a.d;
  if (s >= a.S) return;  // whole wavefront leaves; no block-wide barrier below
  const int F = a.Nk;
  const int rr = r < F ? r : F - 1;  // rows past the sequence repeat the last one: masked as keys, not stored as queries
  const unsigned short* qrow = static_cast<const unsigned short*>(a.q) + a.qmap.row(s, rr) * a.ldq + hc + 8 * g;
  const unsigned short* krow = static_cast<const unsigned short*>(a.k) + a.kmap.row(s, rr) * a.ldk + hc + 8 * g;
  const unsigned short* vrow = static_cast<const unsigned short*>(a.v) + a.kmap.row(s, rr) * a.ldv + hc + 8 * g;
  u32x4_t qf[KS], kf[KS], vf[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
    const bool in = 16 * ks + 8 * g < a.d;  // only the last k-step of an odd number of 8-channel pieces is half empty
    qf[ks] = kf[ks] = vf[ks] = u32x4_t{0, 0, 0, 0};
    if (in) {
      qf[ks] = *reinterpret_cast<const u32x4_t*>(qrow + 16 * ks);
      kf[ks] = *reinterpret_cast<const u32x4_t*>(krow + 16 * ks);
      vf[ks] = *reinterpret_cast<const u32x4_t*>(vrow + 16 * ks);
    }
  }
  auto mfma = [](u32x4_t row, u32x4_t col, f32x16_t acc) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, row), __builtin_bit_cast(bf16x8_t, col), acc, 0, 0, 0);
  };
  f32x16_t zero;
#pragma unroll
  for (int e = 0; e < 16; ++e) zero[e] = 0.f;
  f32x16_t sc = zero;
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) sc = mfma(kf[ks], qf[ks], sc);

  // softmax over the keys: this lane holds keys 8 (e / 4) + 4 g + e % 4 of query r, lane ^ 32 the others
  const float scale2 = a.scale * 1.4426950408889634f;
  float m = -INFINITY;
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    sc[e] = 8 * (e / 4) + 4 * g + (e % 4) < F ? sc[e] * scale2 : -INFINITY;
    m = fmaxf(m, sc[e]);
  }
  m = fmaxf(m, __shfl_xor(m, 32, kWave));
  unsigned hi[8], lo[8];
  float l = 0.f;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const float p0 = __builtin_amdgcn_exp2f(sc[2 * i] - m), p1 = __builtin_amdgcn_exp2f(sc[2 * i + 1] - m);
    l += p0 + p1;
    hi[i] = (unsigned)float_to_bf16_bits(p0) | ((unsigned)float_to_bf16_bits(p1) << 16);
    lo[i] = (unsigned)float_to_bf16_bits(p0 - __uint_as_float(hi[i] << 16)) |
            ((unsigned)float_to_bf16_bits(p1 - __uint_as_float(hi[i] & 0xffff0000u)) << 16);
  }
  l += __shfl_xor(l, 32, kWave);
  const float inv = 1.f / l;

  // slices of the identity: k-step s2 of a 32-channel block, lane (column r, half g): element e is 1 where 16 s2 + 8 g + e == r
  u32x4_t eye[2];
#pragma unroll
  for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const int at = r - (16 * s2 + 8 * g + 2 * w);
      eye[s2][w] = at == 0 ? 0x3f80u : at == 1 ? 0x3f800000u : 0u;
    }
  const int64_t orow = a.qmap.row(s, rr);
  unsigned short* O = static_cast<unsigned short*>(a.o);
#pragma unroll
  for (int b = 0; b < DB; ++b) {
    f32x16_t vt = mfma(vf[2 * b], eye[0], zero);
    if (2 * b + 1 < KS) vt = mfma(vf[2 * b + 1 < KS ? 2 * b + 1 : 0], eye[1], vt);
    f32x16_t o = zero;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      u32x4_t vrow4;
#pragma unroll
      for (int i = 0; i < 4; ++i)
        vrow4[i] = (unsigned)float_to_bf16_bits(vt[8 * t + 2 * i]) | ((unsigned)float_to_bf16_bits(vt[8 * t + 2 * i + 1]) << 16);
      o = mfma(vrow4, u32x4_t{hi[4 * t], hi[4 * t + 1], hi[4 * t + 2], hi[4 * t + 3]}, o);
      o = mfma(vrow4, u32x4_t{lo[4 * t], lo[4 * t + 1], lo[4 * t + 2], lo[4 * t + 3]}, o);
    }
    // registers 8 hf .. + 7: channels 32b + 16hf + {4g .. +3, 8 + 4g .. +3}; one lane^32 exchange per register
    // pair hands each lane the 8 consecutive channels 32b + 16hf + 8g .. +7
#pragma unroll
    for (int hf = 0; hf < 2; ++hf) {
      unsigned w[4];
#pragma unroll
      for (int i = 0; i < 4; ++i)
        w[i] = (unsigned)float_to_bf16_bits(o[8 * hf + 2 * i] * inv) | ((unsigned)float_to_bf16_bits(o[8 * hf + 2 * i + 1] * inv) << 16);
      const auto x = __builtin_amdgcn_permlane32_swap(w[0], w[2], false, false);
      const auto y = __builtin_amdgcn_permlane32_swap(w[1], w[3], false, false);
      const int c = 32 * b + 16 * hf + 8 * g;
      if (r < F && c < a.d)
        *reinterpret_cast<u32x4_t*>(O + (o_frag ? act_offset(orow, hc + c, o_frag) : orow * a.ldo + hc + c)) = u32x4_t{x[0], y[0], x[1], y[1]};
    }
  }
}

}  // namespace si
