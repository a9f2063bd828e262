// Attention in 16-bit storage with everything between the operands and the result in fp32, for the shapes that the
// bf16 matrix-core kernel does not take: spatial self- and cross-attention with heads other than 64 channels or H*W
// no multiple of 8, and temporal sequences of more than 32 frames.
//
// Scores, probabilities, row sums and the output are attn_valu_kernel's (k_attn.h), bit for bit: queries times the
// softmax scale in fp32, exact expf against the running maximum of 64-key chunks, row sums over the same tree,
// products accumulated key by key.  Both contractions run on v_mfma_f32_16x16x4_f32, which is a chain of four fused
// multiply-adds in k order (bf16 values as fp32 are exact), so the matrix cores change the speed and nothing else.
//   S^T[key, query] = K Q^T      row operand: 16 keys x 4 channels; a lane (row f, group g) supplies channel 4 s + g
//   O^T[chan, query] += V^T P^T  row operand: 16 channels x 4 keys; column operand: the lane's own probabilities
// A result lane holds column (query) lane % 16 and rows 4 g + j, g = lane / 16.  Row f = 4 g + j of a key tile is key
// 4 j + g, so that register j of group g is the column operand of the j-th step of four keys as it stands.
//
// One workgroup = 4 wavefronts x 32 queries (two column tiles, so that a key / value operand serves two MFMAs) of one
// (sequence, head).  Chunks of 64 keys pass through LDS as fp32 operands, [operand][lane][4 steps]: one 16-byte read
// of consecutive lanes per four steps; the values' channels lie exclusive-ored with the key group, so that a store of
// one channel of many keys spreads over half of the banks instead of an eighth.  The next chunk's rows are loaded while
// the current one is contracted.
//
// Bound by the fp32 matrix rate, 256 flop per clock and CU, and the exponentials, which overlap with it in part only:
// at 40 channels 176 MFMAs of 32 cycles (channels padded to 48 in the second product) and 34 expf of some 14
// instructions per 64 keys x 32 queries.  Three wavefronts per SIMD up to 40 channels, as many as the registers allow.
// Self-attention of one 64 x 64 frame, 8 heads of 40, two sequences (43 GFLOP): attn_valu_kernel 4390 us, this kernel 542
// with the values in channel order, 498 as it is; 16 such frames, whole call, 66.7 -> 9.28 ms.
#pragma once
#include "k_attn.h"

namespace si {

constexpr int kF32MmaChunk = 64;  // keys per softmax step: attn_valu_kernel's

// D8: head channels / 8.  o_frag: 0, or o is a fragment-order buffer of that many channels per token.
template <int D8>
__global__ __launch_bounds__(256, D8 <= 5 ? 3 : D8 <= 10 ? 2 : 1) void attn_f32mma_kernel(AttnArgs a, int o_frag) {
  constexpr int NS = 2 * D8, KQ = (NS + 3) / 4, DB = (D8 + 1) / 2;  // k-steps of 4 channels, quads of them, 16-channel blocks
  constexpr int NG = kF32MmaChunk * D8, PT = (NG + 255) / 256;      // 16-byte pieces of a chunk's keys, per thread
  __shared__ float4 kl[4 * KQ * kWave];
  __shared__ float4 vl[4 * DB * kWave];
  const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
  const int r = lane % 16, g = lane / 16;
  const unsigned short* Q = static_cast<const unsigned short*>(a.q);
  const unsigned short* Kp = static_cast<const unsigned short*>(a.k);
  const unsigned short* Vp = static_cast<const unsigned short*>(a.v);
  const int nqt = (a.Nq + 127) / 128;
  // query tiles of one (sequence, head) follow each other, and every XCD takes a contiguous share of the list
  const int64_t ntiles = (int64_t)nqt * a.heads * a.S, chunk = (ntiles + 7) / 8;
  for (int64_t it = blockIdx.x / 8; it < chunk; it += gridDim.x / 8) {
    const int64_t work = (int64_t)(blockIdx.x % 8) * chunk + it;
    if (work >= ntiles) return;
    const int s = (int)(work / nqt / a.heads), hc = (int)(work / nqt % a.heads) * a.d;
    const int q0 = (int)(work % nqt) * 128 + wave * 32;
    auto half = [](unsigned w, int hi) { return __uint_as_float(hi ? w & 0xffff0000u : w << 16); };

    u32x4_t kr[PT], vr[PT];
    auto load = [&](int kc) {
#pragma unroll
      for (int i = 0; i < PT; ++i) {
        const int id = tid + i * 256, key = id / D8, c8 = id % D8;
        kr[i] = vr[i] = u32x4_t{0, 0, 0, 0};
        if (id < NG && kc + key < a.Nk) {
          const int64_t row = a.kmap.row(s, kc + key);
          kr[i] = *reinterpret_cast<const u32x4_t*>(Kp + row * a.ldk + hc + 8 * c8);
          vr[i] = *reinterpret_cast<const u32x4_t*>(Vp + row * a.ldv + hc + 8 * c8);
        }
      }
    };
    auto store = [&]() {
#pragma unroll
      for (int i = 0; i < PT; ++i) {
        const int id = tid + i * 256, key = id / D8, c8 = id % D8;
        if (id >= NG) continue;
        const int t = key / 16, j = key % 16 / 4, kg = key % 4;
        float* kd = reinterpret_cast<float*>(kl + (t * KQ + c8 / 2) * kWave + 4 * kg + j) + 2 * (c8 % 2);
        float* vd = reinterpret_cast<float*>(vl + (t * DB + c8 / 2) * kWave + 16 * kg) + j;
#pragma unroll
        for (int e = 0; e < 4; ++e)
          *reinterpret_cast<float2*>(kd + 16 * 4 * e) = make_float2(half(kr[i][e / 2], e & 1), half(kr[i][2 + e / 2], e & 1));
#pragma unroll
        for (int e = 0; e < 8; ++e) vd[4 * ((8 * (c8 % 2) + e) ^ 2 * kg)] = half(vr[i][e / 2], e & 1);
      }
    };
    load(0);

    // queries past the end are zero
    float qf[2][NS];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int qi = q0 + 16 * u + r;
      const unsigned short* qrow = Q + a.qmap.row(s, qi < a.Nq ? qi : 0) * a.ldq + hc;
#pragma unroll
      for (int c8 = 0; c8 < D8; ++c8) {
        u32x4_t v = u32x4_t{0, 0, 0, 0};
        if (qi < a.Nq) v = *reinterpret_cast<const u32x4_t*>(qrow + 8 * c8);
        qf[u][2 * c8] = half(g & 2 ? v.y : v.x, g & 1) * a.scale;
        qf[u][2 * c8 + 1] = half(g & 2 ? v.w : v.z, g & 1) * a.scale;
      }
    }

    const f32x4_t zero = f32x4_t{0.f, 0.f, 0.f, 0.f};
    f32x4_t o[2][DB];
    float mrun[2], lrun[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      mrun[u] = -INFINITY;
      lrun[u] = 0.f;
#pragma unroll
      for (int b = 0; b < DB; ++b) o[u][b] = zero;
    }
    for (int kc = 0; kc < a.Nk; kc += kF32MmaChunk) {
      __syncthreads();  // everybody has left the previous chunk
      store();
      __syncthreads();
      if (kc + kF32MmaChunk < a.Nk) load(kc + kF32MmaChunk);
      f32x4_t sc[2][4];
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        sc[0][t] = sc[1][t] = zero;
        if (kc + 16 * t < a.Nk) {
#pragma unroll
          for (int q4 = 0; q4 < KQ; ++q4) {
            const f32x4_t kq = *reinterpret_cast<const f32x4_t*>(kl + (t * KQ + q4) * kWave + lane);
#pragma unroll
            for (int i = 0; i < 4; ++i)
              if (4 * q4 + i < NS) {
                sc[0][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(kq[i], qf[0][4 * q4 + i], sc[0][t], 0, 0, 0);
                sc[1][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(kq[i], qf[1][4 * q4 + i], sc[1][t], 0, 0, 0);
              }
          }
        }
      }
      if (kc + kF32MmaChunk > a.Nk) {
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
          for (int j = 0; j < 4; ++j)
            if (kc + 16 * t + 4 * j + g >= a.Nk) sc[0][t][j] = sc[1][t][j] = -INFINITY;
      }
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        float cm = sc[u][0][0];
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
          for (int j = 0; j < 4; ++j) cm = fmaxf(cm, sc[u][t][j]);
        cm = fmaxf(cm, __shfl_xor(cm, 32, kWave));
        cm = fmaxf(cm, __shfl_xor(cm, 16, kWave));
        const float mn = fmaxf(mrun[u], cm);
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
          for (int j = 0; j < 4; ++j) sc[u][t][j] = expf(sc[u][t][j] - mn);
        const float alpha = expf(mrun[u] - mn);  // first chunk: exp(-inf) = 0
        // the tree of a sum over 64 lanes by halves: key bits 5 .. 2 lie in registers, 1 and 0 in lane bits 5 and 4
        float p[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) p[j] = (sc[u][0][j] + sc[u][2][j]) + (sc[u][1][j] + sc[u][3][j]);
        float l = (p[0] + p[2]) + (p[1] + p[3]);
        l += __shfl_xor(l, 32, kWave);
        l += __shfl_xor(l, 16, kWave);
        lrun[u] = lrun[u] * alpha + l;
        mrun[u] = mn;
#pragma unroll
        for (int b = 0; b < DB; ++b) o[u][b] *= alpha;
      }
#pragma unroll
      for (int t = 0; t < 4; ++t)
        if (kc + 16 * t < a.Nk) {
          f32x4_t vq[DB];
#pragma unroll
          for (int b = 0; b < DB; ++b) vq[b] = *reinterpret_cast<const f32x4_t*>(vl + (t * DB + b) * kWave + (lane ^ 2 * g));
#pragma unroll
          for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int b = 0; b < DB; ++b)
#pragma unroll
              for (int u = 0; u < 2; ++u) o[u][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(vq[b][j], sc[u][t][j], o[u][b], 0, 0, 0);
        }
    }

    unsigned short* O = static_cast<unsigned short*>(a.o);
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int qi = q0 + 16 * u + r;
      if (qi >= a.Nq) continue;
      const float inv = 1.f / lrun[u];
      const int64_t row = a.qmap.row(s, qi);
#pragma unroll
      for (int b = 0; b < DB; ++b) {
        const int c = 16 * b + 4 * g;  // register j: channel c + j
        if (c >= a.d) continue;
        uint2 v;
        v.x = (unsigned)float_to_bf16_bits(o[u][b][0] * inv) | ((unsigned)float_to_bf16_bits(o[u][b][1] * inv) << 16);
        v.y = (unsigned)float_to_bf16_bits(o[u][b][2] * inv) | ((unsigned)float_to_bf16_bits(o[u][b][3] * inv) << 16);
        *reinterpret_cast<uint2*>(O + (o_frag ? act_offset(row, hc + c, o_frag) : row * a.ldo + hc + c)) = v;
      }
    }
  }
}

}  // namespace si
