// Single-token decode step on the persistent int8 state: the chunked method with a chunk of one
// token (Sec. 4.2 quantization; Eq. 7-8 chunk state, Eq. 9 state passing, Eq. 10 correction),
// for every (batch, head) at once.  With one token the chunk quantities reduce to
//   cs = dA = dt A,  LUT_state = dt,  q_d = rne(exp(dA) 2^k)
//   X_q[p]    = Q(fl32(dt x[p]) / a_X[p])                          (Eq. 7)
//   S_q[p,n]  = requant(X_q[p] B_q[n], m_S[p])                       (Eq. 8)
//   state'    = sat(S_q + ((q_d state + r) >> k))                    (Eq. 9)
//   y[p]      = (sum_n C_q[n] state[p,n]) a_C exp(dA) a_S[p]         (ChunkScan1, entering state)
//             + fp16(CB_q a_CB dt) fp16(x[p])                        (ChunkScan2, i = j)
//             + D x[p] + corr[p]
// with CB_q = requant(C_q . B_q, m_CB).  Every integer quantity and every fp32 rounding before
// an integer decision is formed exactly as in the chunked kernels (ChunkState, ChunkBMM, state
// passing), so a decode step equals the layer run over that token with chunk size 1.
//
// One workgroup per head and run of nb batch elements, 256 threads: thread t owns state row p =
// t / 4 and the 32 state entries n in [16 (t % 4), +16) and [64 + 16 (t % 4), +16): two 16-byte
// reads and writes of the row-major state per element, in place.
//
// What bounds it: at large batches the state's bytes, once the vector work is below them.  C.state
// and C.B are four-element dot instructions, Eq. 9 runs on packed 16-bit pairs (S_q comes out of its
// rounding as an int16), the fp64 chain of a (b, h) runs once, in one lane, instead of in all 256
// threads, and the per-channel steps serve the whole run of batch elements.  128 x 80 heads: 60 ->
// 36 us (168 MB).  At small batches (one element per workgroup) it is the latency of the loads and
// of that chain: nothing waits for a barrier there (8 x 24 heads: 5.5 -> 4.4 us).
#include <type_traits>

#include "common.hpp"
#include "launch.hpp"

namespace ssdi8 {

namespace {

// The quantities of one (b, h): dt and dA, Q(Decay), LUT_state.
struct TokenScalars {
  float dtv, dA, lut;
  int qd;
};
__device__ __forceinline__ TokenScalars token_scalars(float dt, int dt_softplus, float A,
                                                      int shift) {
  TokenScalars s;
  s.dtv = dt_softplus ? softplus_f32(dt) : dt;
  s.dA = s.dtv * A;
  const double cs = (double)s.dA;
  s.qd = (int)rint(exp(cs) * (double)(1 << shift));
  // exp(cs_last - cs) of the only token: 1, or NaN where dA is not finite
  s.lut = s.dtv * ((s.dA - s.dA) + 1.0f);
  return s;
}

// kMulti: several batch elements per workgroup (their scalars through LDS); else one.
constexpr int kMaxRun = 8;

template <typename XT, typename YT, bool kMulti>
__global__ __launch_bounds__(256) void decode_kernel(
    const XT* __restrict__ x, const float* __restrict__ dt, int dt_softplus,
    const float* __restrict__ A, const int8_t* __restrict__ Bq, const int8_t* __restrict__ Cq,
    const float* __restrict__ B_scale, const float* __restrict__ C_scale, int c_per_token,
    const float* __restrict__ Dv, const float* __restrict__ corr,
    const float* __restrict__ xs_scale, int xs_per_head, const float* __restrict__ state_scale,
    const float* __restrict__ cb_scale, int shift, int radd, int8_t* __restrict__ state,
    YT* __restrict__ y, float* __restrict__ state_f32, int B, int H, int G, int nb) {
  __shared__ TokenScalars s_tok[kMaxRun];
  const int t = threadIdx.x;
  const int p = t >> 2, n0 = 16 * (t & 3);
  const int h = blockIdx.x % H;
  const int b0 = kMulti ? (int)(blockIdx.x / H) * nb : (int)(blockIdx.x / H);
  const int b1 = kMulti ? (b0 + nb < B ? b0 + nb : B) : b0 + 1;
  const int g = h / (H / G);

  struct Item {
    uint4 bv[2], cv[2], sv[2];
    float xval;
  };
  auto load = [&](int b, Item& it) {
    const size_t bg = (size_t)b * G + g, bh = (size_t)b * H + h;
    const int8_t* brow = Bq + bg * kN + n0;
    const int8_t* crow = Cq + bg * kN + n0;
    const int8_t* srow = state + (bh * kP + p) * kN + n0;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      it.bv[i] = *reinterpret_cast<const uint4*>(brow + 64 * i);
      it.cv[i] = *reinterpret_cast<const uint4*>(crow + 64 * i);
      it.sv[i] = *reinterpret_cast<const uint4*>(srow + 64 * i);
    }
    it.xval = (float)x[bh * kP + p];
  };

  // ---- every load first (none depends on another), then the dependent fp64 chain
  Item cur;
  load(b0, cur);
  const float Ah = A[h];
  const float axs = xs_per_head ? xs_scale[h] : xs_scale[h * kP + p];
  const float aS = state_scale[h * kP + p];
  const float aB = B_scale[g], aCB = cb_scale[g];
  const float Dh = Dv ? Dv[h] : 0.0f;
  const float cr = corr ? corr[h * kP + p] : 0.0f;
  TokenScalars tok;
  if constexpr (kMulti) {
    if (t < b1 - b0) s_tok[t] = token_scalars(dt[(size_t)(b0 + t) * H + h], dt_softplus, Ah, shift);
  } else {
    tok = token_scalars(dt[(size_t)b0 * H + h], dt_softplus, Ah, shift);
  }
  // X_q's inverse step of channel p and its state multiplier (Eq. 7-8)
  const float inv = 1.0f / axs;
  const float ms = (float)(((double)axs * (double)aB) / (double)aS);
  if constexpr (kMulti) __syncthreads();

  for (int b = b0; b < b1; ++b) {
    Item nxt;
    if constexpr (kMulti) {
      if (b + 1 < b1) load(b + 1, nxt);
      tok = s_tok[b - b0];
    }
    const int qd = __builtin_amdgcn_readfirstlane(tok.qd);   // one value per workgroup
    const size_t bg = (size_t)b * G + g, bh = (size_t)b * H + h;
    const float xq = (float)quant_i8(tok.lut * cur.xval, inv);
    // the packed step is exact for these (common.hpp); others, e.g. a decay above 1 from inputs
    // outside the method's domain, take the 32-bit one
    const bool packed = shift <= 8 && qd >= 0 && qd <= (1 << shift);
    int y1 = 0, cb = 0;
    uint4 nv[2];
    auto row = [&](auto pk) {
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const uint32_t bw[4] = {cur.bv[i].x, cur.bv[i].y, cur.bv[i].z, cur.bv[i].w};
        const uint32_t cw[4] = {cur.cv[i].x, cur.cv[i].y, cur.cv[i].z, cur.cv[i].w};
        const uint32_t sw[4] = {cur.sv[i].x, cur.sv[i].y, cur.sv[i].z, cur.sv[i].w};
        uint32_t ow[4];
#pragma unroll
        for (int d = 0; d < 4; ++d) {
          y1 = __builtin_amdgcn_sdot4((int)cw[d], (int)sw[d], y1, false);   // entering state
          cb = __builtin_amdgcn_sdot4((int)cw[d], (int)bw[d], cb, false);   // token with itself
          // S_q = requant(X_q B_q): the product of two int8 codes is exact in fp32
          uint32_t q[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) q[e] = quant_bits(xq * (float)sext8(bw[d], e), ms);
          if constexpr (decltype(pk)::value) {
            ow[d] = pass_step4_pk16_q(sw[d], q, qd, radd, shift);
          } else {
            int o[4];
#pragma unroll
            for (int e = 0; e < 4; ++e)
              o[e] = pass_step(sext8(sw[d], e), (int)q[e] - 0x4B400000, qd, shift, radd);
            ow[d] = pack4_i8(o[0], o[1], o[2], o[3]);
          }
        }
        nv[i] = make_uint4(ow[0], ow[1], ow[2], ow[3]);
      }
    };
    if (packed) row(std::true_type{});
    else row(std::false_type{});
    // the 4 threads of row p are adjacent lanes
    y1 += __shfl_xor(y1, 1, 64);
    y1 += __shfl_xor(y1, 2, 64);
    cb += __shfl_xor(cb, 1, 64);
    cb += __shfl_xor(cb, 2, 64);
    int8_t* srow = state + (bh * kP + p) * kN + n0;
#pragma unroll
    for (int i = 0; i < 2; ++i) *reinterpret_cast<uint4*>(srow + 64 * i) = nv[i];
    if (state_f32) {
      float* fo = state_f32 + (bh * kP + p) * kN + n0;
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const uint32_t w[4] = {nv[i].x, nv[i].y, nv[i].z, nv[i].w};
#pragma unroll
        for (int d = 0; d < 4; ++d)
          *reinterpret_cast<float4*>(fo + 64 * i + 4 * d) =
              make_float4((float)sext8(w[d], 0) * aS, (float)sext8(w[d], 1) * aS,
                          (float)sext8(w[d], 2) * aS, (float)sext8(w[d], 3) * aS);
      }
    }
    if ((t & 3) == 0) {
      const float ac = c_per_token ? C_scale[bg] : C_scale[g];
      const float mcb = (float)(((double)ac * (double)aB) / (double)aCB);
      const int cbq = requant_i8(cb, mcb);
      const float dtcb = aCB * tok.dtv;
      const _Float16 w = (_Float16)((float)cbq * dtcb);        // W of the diagonal, exp(0) = 1
      float yd = __builtin_fmaf(Dh, cur.xval, cr);
      yd += (float)w * (float)(_Float16)cur.xval;
      const float eo = ac * __expf(tok.dA);
      const float out = __builtin_fmaf((float)y1 * eo, aS, yd);
      y[bh * kP + p] = (YT)out;
    }
    if constexpr (kMulti) cur = nxt;
  }
}

}  // namespace

hipError_t launch_decode(int64_t batch, int64_t nheads, int64_t ngroups, const void* x,
                         int x_dtype, const float* dt, int dt_softplus, const float* A,
                         const int8_t* Bq, const int8_t* Cq, const float* B_scale,
                         const float* C_scale, int c_per_token, const float* D,
                         const float* corr, const float* xs_scale, int xs_per_head,
                         const float* state_scale, const float* cb_scale, int shift,
                         int shift_round, int8_t* state, void* y, int y_dtype, float* state_f32,
                         hipStream_t st) {
  const int64_t items = batch * nheads;
  if (items == 0) return hipSuccess;
  const int radd = shift_round ? (1 << (shift - 1)) : 0;
  // Batch elements per workgroup.  A run amortises the fp64 chain and the per-channel steps, but
  // its elements are serial: measured (us, runs of 1 / 2 / 4 / 8) 1536 items 9.7 / 9.7 / 11.7 /
  // 13.2, 2560 items 13.9 / 14.0 / 14.9 / 18.7, 3200 items 17.0 / 16.6 / 17.4 / 19.2, 5120 items
  // 24.2 / 22.8 / 22.4 / 24.6, 10240 items 44.0 / 38.3 / 37.3 / 36.1.
  int64_t nb = items >= 8192 ? 8 : items >= 4096 ? 4 : items >= 3072 ? 2 : 1;
  if (nb > batch) nb = batch;
  const bool multi = nb >= 2;
  const int64_t nwg = multi ? (batch + nb - 1) / nb * nheads : items;
#define SSDI8_DECODE_LAUNCH(XT, YT, M)                                                         \
  hipLaunchKernelGGL((decode_kernel<XT, YT, M>), dim3((unsigned)nwg), dim3(256), 0, st,        \
                     static_cast<const XT*>(x), dt, dt_softplus, A, Bq, Cq, B_scale, C_scale, \
                     c_per_token, D, corr, xs_scale, xs_per_head, state_scale, cb_scale,      \
                     shift, radd, state, static_cast<YT*>(y), state_f32, (int)batch,          \
                     (int)nheads, (int)ngroups, (int)nb)
#define SSDI8_DECODE_TYPES(XT, YT)                \
  do {                                            \
    if (multi) SSDI8_DECODE_LAUNCH(XT, YT, true); \
    else SSDI8_DECODE_LAUNCH(XT, YT, false);      \
  } while (0)
  if (x_dtype == 1 && y_dtype == 1) SSDI8_DECODE_TYPES(_Float16, _Float16);
  else if (x_dtype == 1) SSDI8_DECODE_TYPES(_Float16, float);
  else if (y_dtype == 1) SSDI8_DECODE_TYPES(float, _Float16);
  else SSDI8_DECODE_TYPES(float, float);
#undef SSDI8_DECODE_TYPES
#undef SSDI8_DECODE_LAUNCH
  return hipGetLastError();
}

}  // namespace ssdi8
