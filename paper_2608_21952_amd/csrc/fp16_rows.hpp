// Device code shared by the FP16 layer's scan kernels: the raw x pairs, ChunkScan's decay tables
// and one row block (32 tokens) of ChunkScan2 on top of a ChunkScan1 product.
#pragma once

#include "common.hpp"
#include "frag.hpp"

namespace ssdi8 {
namespace fp16 {

constexpr int kXTS = kQ * 2 + 16;     // bytes per channel row of x^T (fp16)
// A diagonal block whose decay span stays below this bound splits its decay without overflow.
constexpr float kDiagSpan = 64.0f;

typedef float f2_t __attribute__((ext_vector_type(2)));
typedef _Float16 h2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pack_h2(float a, float b) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector((f2_t){a, b}, h2_t));
}
// Two tokens' X~ = LUT x of one channel as packed fp16: the exact product rounded once, to fp16
// (left to the compiler it is rounded once or, through fp32, twice, depending on how the result is
// packed: 4.7e-6 of the final state).  fp16 x: channel `half` of the tokens' pairs w0, w1.
template <int half>
__device__ __forceinline__ uint32_t lut_x2(float l0, uint32_t w0, float l1, uint32_t w1) {
  uint32_t d;
  if constexpr (half == 0)
    asm("v_fma_mixlo_f16 %0, %1, %2, 0 op_sel_hi:[0,1,0]\n\t"
        "v_fma_mixhi_f16 %0, %3, %4, 0 op_sel_hi:[0,1,0]"
        : "=&v"(d) : "v"(l0), "v"(w0), "v"(l1), "v"(w1));
  else
    asm("v_fma_mixlo_f16 %0, %1, %2, 0 op_sel:[0,1,0] op_sel_hi:[0,1,0]\n\t"
        "v_fma_mixhi_f16 %0, %3, %4, 0 op_sel:[0,1,0] op_sel_hi:[0,1,0]"
        : "=&v"(d) : "v"(l0), "v"(w0), "v"(l1), "v"(w1));
  return d;
}
__device__ __forceinline__ uint32_t lut_x2(float l0, float x0, float l1, float x1) {
  uint32_t d;
  asm("v_fma_mixlo_f16 %0, %1, %2, 0\n\tv_fma_mixhi_f16 %0, %3, %4, 0"
      : "=&v"(d) : "v"(l0), "v"(x0), "v"(l1), "v"(x1));
  return d;
}

// Two adjacent channels of one token row, loaded raw.
template <typename XT> struct Pair;
template <> struct Pair<_Float16> {
  typedef uint32_t raw;
  template <int kPol = 0>
  static __device__ __forceinline__ raw load(__amdgpu_buffer_rsrc_t r, uint32_t vo, uint32_t so) {
    return buf_load4<kPol>(r, vo, so);
  }
  static __device__ __forceinline__ uint16_t lo(raw v) { return (uint16_t)(v & 0xffffu); }
  static __device__ __forceinline__ uint16_t hi(raw v) { return (uint16_t)(v >> 16); }
  static __device__ __forceinline__ float lof(raw v) {
    return (float)__builtin_bit_cast(_Float16, lo(v));
  }
  static __device__ __forceinline__ float hif(raw v) {
    return (float)__builtin_bit_cast(_Float16, hi(v));
  }
  // X~ of tokens 0 and 1: channel lo, channel hi
  static __device__ __forceinline__ uint32_t lut_lo(float l0, raw v0, float l1, raw v1) {
    return lut_x2<0>(l0, v0, l1, v1);
  }
  static __device__ __forceinline__ uint32_t lut_hi(float l0, raw v0, float l1, raw v1) {
    return lut_x2<1>(l0, v0, l1, v1);
  }
};
template <> struct Pair<float> {
  typedef float2 raw;
  template <int kPol = 0>
  static __device__ __forceinline__ raw load(__amdgpu_buffer_rsrc_t r, uint32_t vo, uint32_t so) {
    const uint2 v = buf_load8<kPol>(r, vo, so);
    return make_float2(__uint_as_float(v.x), __uint_as_float(v.y));
  }
  static __device__ __forceinline__ uint16_t lo(raw v) {
    return __builtin_bit_cast(uint16_t, (_Float16)v.x);
  }
  static __device__ __forceinline__ uint16_t hi(raw v) {
    return __builtin_bit_cast(uint16_t, (_Float16)v.y);
  }
  static __device__ __forceinline__ float lof(raw v) { return v.x; }
  static __device__ __forceinline__ float hif(raw v) { return v.y; }
  static __device__ __forceinline__ uint32_t lut_lo(float l0, raw v0, float l1, raw v1) {
    return lut_x2(l0, v0.x, l1, v1.x);
  }
  static __device__ __forceinline__ uint32_t lut_hi(float l0, raw v0, float l1, raw v1) {
    return lut_x2(l0, v0.y, l1, v1.y);
  }
};

// ChunkScan's decay tables of a chunk (r_t = cs at the last token of 32-token block t, r_{-1} = 0).
struct Tables {
  float u[kQ];         // dt_i exp(r_I - cs_i)                          (off-diagonal blocks)
  float dg[kQ];        // dt_i exp(r_{I-1} - cs_i) if block I has a small span, else dt_i
  float csr[kQ];       // cs_i - r_{I-1}
  float R[8][8];       // exp(r_a - r_b), b <= a
  float umax[8];       // max |u_i| over block I (inf if one is NaN or an x is not finite)
  double r[8];
};

// The tables' entries of token t (threads 0 .. 255); r is complete.
__device__ __forceinline__ void build_tables(Tables& T, int t, float dtv, double cs) {
  const int blk = t >> 5;
  const double rprev = blk ? T.r[blk - 1] : 0.0;
  const float u = dtv * expf((float)(T.r[blk] - cs));
  T.u[t] = u;
  float um = u == u ? __builtin_fabsf(u) : __builtin_inff();
#pragma unroll
  for (int o = 1; o < 32; o <<= 1) um = __builtin_fmaxf(um, __shfl_xor(um, o));
  if ((t & 31) == 0) T.umax[blk] = um;
  const float csr = (float)(cs - rprev);
  T.csr[t] = csr;
  const bool small_span = (float)(T.r[blk] - rprev) >= -kDiagSpan;
  T.dg[t] = small_span ? dtv * expf(__builtin_fminf(-csr, kDiagSpan)) : dtv;
  if (t < 64) {
    const int ra = t >> 3, rb = t & 7;
    T.R[ra][rb] = (rb <= ra) ? expf((float)(T.r[ra] - T.r[rb])) : 0.0f;
  }
}

// The maximum this lane contributes to row block jt's skip test (lane & 7 = block), for row_block:
// its sign bit says that the block holds a NaN.
__device__ __forceinline__ float block_max(const float* cb_max_cg, int jt, int lane) {
  const int k = lane & 7;
  return cb_max_cg[frag::cb_block(jt, 0) + (k < jt ? k : 0)];
}

// Row block jt on its ChunkScan1 product: y = Y1 exp(cs_j) + D x, then Scan2 over the causal
// blocks on top.  Lane l: token row j = 32 jt + l % 32; register r of y0 / y1 holds channel p = 32
// pt + 8 (r / 4) + 4 (l / 32) + r % 4.  cbrs: the chunk-group's fp32 CB blocks; cbm: block_max;
// xg: fp32 x of the chunk and head (the D skip of an fp32 x is not rounded), token stride HP.
template <typename XT>
__device__ __forceinline__ void row_block(int jt, int lane, const Tables& T, const uint8_t* xT,
                                          __amdgpu_buffer_rsrc_t cbrs, float cbm, const XT* xg,
                                          size_t HP, float Dh, v16f& y0, v16f& y1) {
  asm volatile("" : "+s"(jt) :: "memory");
  const int pc = lane & 31, half = lane >> 5;
  const uint32_t lane16 = lane * 16;
  const int jrow = jt * 32 + pc;
  const float csrj = T.csr[jrow];
  const float ej = __expf(csrj);
  // exp(cs_j) = exp(cs_j - r_{J-1}) exp(r_{J-1})
  const float eo = ej * (jt ? __expf((float)T.r[jt - 1]) : 1.0f);
#pragma unroll
  for (int pt = 0; pt < 2; ++pt) {
#pragma unroll
    for (int g4 = 0; g4 < 4; ++g4) {
      const int pb = pt * 32 + 8 * g4 + 4 * half;
      float xv[4];
      if constexpr (sizeof(XT) == 2) {
#pragma unroll
        for (int q = 0; q < 4; ++q)
          xv[q] = (float)*reinterpret_cast<const _Float16*>(xT + (pb + q) * kXTS + jrow * 2);
      } else {
        const float4 xf = *reinterpret_cast<const float4*>(xg + (size_t)jrow * HP + pb);
        xv[0] = xf.x; xv[1] = xf.y; xv[2] = xf.z; xv[3] = xf.w;
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int r = 4 * g4 + q;
        if (pt) y1[r] = __builtin_fmaf(y1[r], eo, Dh * xv[q]);
        else y0[r] = __builtin_fmaf(y0[r], eo, Dh * xv[q]);
      }
    }
  }
  // Leading off-diagonal blocks whose every weight rounds to an fp16 zero are skipped: |W| <=
  // max |CB| max |u| R e_j, and below 2^-26 (half the smallest fp16 subnormal is 2^-25) it is zero.
  // e_j <= 1 where no row of the block lies above cs at the block's start; a block in which one
  // does (or is NaN; dt or A outside the method's signs) skips nothing.
  const uint32_t cbrow = frag::cb_block(jt, 0) * 4096;
  const bool diag_fast =
      __builtin_amdgcn_readfirstlane((int)(T.csr[jt * 32 + 31] >= -kDiagSpan)) != 0;
  int it0 = jt;
  {
    const int k = lane & 7;
    const bool rises = __ballot(!(csrj <= 0.0f)) != 0;
    const bool live =
        k < jt && (rises || (int)__float_as_uint(cbm) < 0 ||
                   !(cbm * T.umax[k] * T.R[jt ? jt - 1 : 0][k] < 0x1p-26f));
    const uint32_t lv = (uint32_t)__ballot(live) & 0xffu;
    if (lv) it0 = (int)__builtin_ctz(lv);
    it0 = __builtin_amdgcn_readfirstlane(it0);
  }
  auto mfma_block = [&](const float (&wv)[8], int i0) {
    v8h wf;
#pragma unroll
    for (int e = 0; e < 8; e += 2) {
      const h2_t hh = __builtin_convertvector((f2_t){wv[e], wv[e + 1]}, h2_t);
      wf[e] = hh.x;
      wf[e + 1] = hh.y;
    }
    const v8h xa0 = *reinterpret_cast<const v8h*>(xT + pc * kXTS + i0 * 2);
    const v8h xa1 = *reinterpret_cast<const v8h*>(xT + (32 + pc) * kXTS + i0 * 2);
    y0 = __builtin_amdgcn_mfma_f32_32x32x16_f16(xa0, wf, y0, 0, 0, 0);
    y1 = __builtin_amdgcn_mfma_f32_32x32x16_f16(xa1, wf, y1, 0, 0, 0);
  };
  auto load_block = [&](uint32_t off, uint4 (&v)[4]) {   // four planes of 1 KB (fp16_bmm.hip)
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = buf_load16(cbrs, lane16, off + 1024 * u);
  };
  auto cbv = [](const uint4 (&v)[4], int k) {   // float k of this lane's 16
    const uint4 q = v[k >> 2];
    const uint32_t e = (k & 3) == 0 ? q.x : (k & 3) == 1 ? q.y : (k & 3) == 2 ? q.z : q.w;
    return __uint_as_float(e);
  };
  uint4 cur[4];
  load_block(cbrow + it0 * 4096, cur);
  for (int it = it0; it < jt; ++it) {
    uint4 nx[4];
    load_block(cbrow + (it + 1) * 4096, nx);
    __builtin_amdgcn_sched_barrier(0);
    const float vj = ej * T.R[jt - 1][it];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      const int i0 = it * 32 + ks * 16 + 8 * half;
      float wv[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) wv[e] = (cbv(cur, 8 * ks + e) * T.u[i0 + e]) * vj;
      mfma_block(wv, i0);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) cur[u] = nx[u];
  }
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) {
    const int i0 = jt * 32 + ks * 16 + 8 * half;
    float wv[8];
    if (diag_fast) {
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float v = (cbv(cur, 8 * ks + e) * T.dg[i0 + e]) * ej;
        wv[e] = (i0 + e <= jrow) ? v : 0.0f;
      }
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float ex = __expf(__builtin_fminf(csrj - T.csr[i0 + e], 0.0f));
        const float v = (cbv(cur, 8 * ks + e) * T.dg[i0 + e]) * ex;
        wv[e] = (i0 + e <= jrow) ? v : 0.0f;
      }
    }
    mfma_block(wv, i0);
  }
}

// A row block's fp16 output in the stage of 256 rows of 128 bytes: row j at 128 j, its 16-byte
// chunk k at slot k ^ (j & 7) (conflict-free writes by token and reads by row).
__device__ __forceinline__ void stage_rows_f16(uint8_t* s_y, int jt, int lane, const v16f& y0,
                                               const v16f& y1) {
  const uint32_t pc = lane & 31;
  uint8_t* row = s_y + (jt * 32 + pc) * 128 + 8 * (lane >> 5);
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const int r = 4 * (k & 3);
    const v16f& v = k < 4 ? y0 : y1;
    *reinterpret_cast<uint2*>(row + (k ^ (pc & 7)) * 16) =
        make_uint2(pack_h2(v[r], v[r + 1]), pack_h2(v[r + 2], v[r + 3]));
  }
}
// The same for fp32 output, 128 rows of 256 bytes (blocks 0..3 or 4..7; jt4 = block % 4): 16-byte
// chunk k at slot k ^ (j & 15).
__device__ __forceinline__ void stage_rows_f32(uint8_t* s_y, int jt4, int lane, const v16f& y0,
                                               const v16f& y1) {
  const uint32_t pc = lane & 31, half = lane >> 5;
  uint8_t* row = s_y + (jt4 * 32 + pc) * 256;
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const int r = 4 * (k & 3);
    const v16f& v = k < 4 ? y0 : y1;
    *reinterpret_cast<float4*>(row + ((2 * k + half) ^ (pc & 15)) * 16) =
        make_float4(v[r], v[r + 1], v[r + 2], v[r + 3]);
  }
}
// Rows [row0, row0 + rows) of the chunk leave the stage as whole rows (kRB bytes each: 128 or
// 256), by kThreads threads; yrs: y of the chunk and head, token stride HP elements.
template <int kRB, int kThreads>
__device__ __forceinline__ void rows_out(const uint8_t* s_y, __amdgpu_buffer_rsrc_t yrs, int t,
                                         size_t HP, int row0, int stream) {
  constexpr int kC = kRB / 16;              // 16-byte chunks per row
  constexpr int kRows = kThreads / kC;      // rows per step
  constexpr int kSteps = (kQ * kP * 2) / (16 * kThreads);   // the stage holds 32 KB
  const int row = t / kC, col = t % kC;
  const uint8_t* src = s_y + row * kRB + ((col ^ (row & (kC - 1))) * 16);
  const uint32_t es = kRB / kP;             // bytes per element
  const uint32_t yo = (uint32_t)(row * HP * es + col * 16);
#pragma unroll
  for (int k = 0; k < kSteps; ++k) {
    const uint4 v = *reinterpret_cast<const uint4*>(src + k * kRows * kRB);
    const uint32_t so = (uint32_t)((row0 + kRows * k) * HP * es);
    if (stream) buf_store16<kPolicyNT>(v, yrs, yo, so);
    else buf_store16(v, yrs, yo, so);
  }
}
// The 32 fp32 rows from row0 on that one wave has staged, by that wave alone: four rows per store.
__device__ __forceinline__ void rows_out_f32_wave(const uint8_t* s_y, __amdgpu_buffer_rsrc_t yrs,
                                                  int lane, size_t HP, int row0, int stream) {
  const int row = lane >> 4, col = lane & 15;
  const uint32_t yo = (uint32_t)(row * HP * 4 + col * 16);
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const int r = 4 * k + row;
    const uint4 v = *reinterpret_cast<const uint4*>(s_y + r * 256 + ((col ^ (r & 15)) * 16));
    const uint32_t so = (uint32_t)((row0 + 4 * k) * HP * 4);
    if (stream) buf_store16<kPolicyNT>(v, yrs, yo, so);
    else buf_store16(v, yrs, yo, so);
  }
}
static_assert(kP * kXTS >= kQ * kP * 2, "the output stages reuse the x^T bytes");

// v of lane l ^ kXor, kXor < 32: a swizzle, which needs no lane address in a register.
template <int kXor> __device__ __forceinline__ double swizzle_xor_f64(double v) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_ds_swizzle((int)(uint32_t)u, (kXor << 10) | 0x1f);
  const uint32_t hi =
      (uint32_t)__builtin_amdgcn_ds_swizzle((int)(uint32_t)(u >> 32), (kXor << 10) | 0x1f);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
// One exchange of a reduce-scatter: of values 0 .. 2 kO - 1 the lanes with bit kO keep the upper half.
template <int kO> __device__ __forceinline__ void exchange_half(double (&v)[16], int lane) {
  const bool up = (lane & kO) != 0;
#pragma unroll
  for (int i = 0; i < kO; ++i) {
    const double keep = up ? v[i + kO] : v[i], send = up ? v[i] : v[i + kO];
    v[i] = keep + swizzle_xor_f64<kO>(send);
  }
}

// Instead of its rows: the fp64 sums over the chunk's 256 tokens of every channel of y, in a fixed
// order, to out[0 .. 63] (calibration needs only the mean of y; as rows it would be written and
// read back in fp32).  A lane adds its two rows, then the 32 lanes of a half-wave reduce and
// scatter in five exchanges, after which lane l % 32 holds register l % 32 of (y0, y1); the four
// waves add up through LDS (s_sum: 2 KB that nothing else uses any more).  By shuffles, whose lane
// address the compiler formed at the kernel's start and held across it, the FP16 layer's scan
// spilled two registers.
__device__ __forceinline__ void channel_sums(double* s_sum, int wv, int lane, const v16f& ya0,
                                             const v16f& ya1, const v16f& yb0, const v16f& yb1,
                                             double* out) {
  double v[16];
  const bool upper = (lane & 16) != 0;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const double s0 = (double)ya0[r] + (double)yb0[r], s1 = (double)ya1[r] + (double)yb1[r];
    v[r] = (upper ? s1 : s0) + swizzle_xor_f64<16>(upper ? s0 : s1);
  }
  exchange_half<8>(v, lane);
  exchange_half<4>(v, lane);
  exchange_half<2>(v, lane);
  exchange_half<1>(v, lane);
  const int r = lane & 31;
  const int p = 32 * (r >> 4) + 8 * ((r & 15) >> 2) + 4 * (lane >> 5) + (r & 3);
  s_sum[wv * kP + p] = v[0];
  __syncthreads();
  const int t = threadIdx.x;
  if (t < kP)
    out[t] = (s_sum[t] + s_sum[kP + t]) + (s_sum[2 * kP + t] + s_sum[3 * kP + t]);
}

}  // namespace fp16
}  // namespace ssdi8
