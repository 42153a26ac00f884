// FP16 layer, ChunkState and StatePassing as one kernel that walks the sequences: one workgroup of
// 8 waves per (batch, head) takes the chunks in order with the fp32 state in registers, so the
// chunk states never go through memory.
//   per chunk  P_in[c] = fp16(P) out, ChunkScan1's operand (frag::pk16_offset)
//              dt, cs, LUT as in ChunkState; X~^T = fp16(LUT x)^T in LDS
//              P <- fma(exp(cs_last), P, S), S = B^T X~ summed from zero
// with the bits of ChunkState and StatePassing: a sequence's result does not depend on how many
// others share the call.
// A sequence's chunks are serial here, so it takes enough sequences to fill the GPU, and a chunk
// must take no longer than its bytes.  Vector loads complete in order, so the two streams are
// split over the waves: waves 0 .. 3 load x two chunks ahead and prepare X~ of chunk c + 1 (one
// token per thread for its ChunkCumsum) while waves 4 .. 7, each one 32-wide n-tile of the state
// for all channels, multiply chunk c with B^T fragments requested 12 K-steps ahead.
// Registers: state 32, S 32, fragments 48 of the 128 that two workgroups per CU leave (14 K-steps
// ahead spill).  S is rounded into P after the next scan barrier, off the chain: whole layer of
// 128, 256, 257 and 320 sequences of 16 chunks 88.8, 156, 171 and 208 us, against 87.2, 156, 172
// and 207 with the products added straight into P (other roundings).
//
// 2.7B-shaped layer, 320 sequences of 16 chunks: 100 us for the 80 + 41 us of ChunkState and
// StatePassing (252 instead of 588 MB), and ChunkScan after it 109 instead of 130 us (x is still
// in the Infinity Cache).  What bounds it: the chain of a chunk (softplus, scan, LUT, X~, with two
// barriers; a third one for X~ cost 6 to 20 %: 128, 192, 256 and 320 sequences of 16 chunks 53.6,
// 55.6, 62.0 and 107 us, now 42.6, 48.0, 55.6 and 99.8), beside a second workgroup on the same CU:
// the walk of 257 sequences takes what that of 512 does (101 us).  32 four-byte loads per thread and chunk stalled on
// the 63 a wave can have counted, so x comes in 16-byte runs.
#include "common.hpp"
#include "fp16_rows.hpp"
#include "frag.hpp"
#include "launch.hpp"

namespace ssdi8 {

namespace {

using namespace fp16;

constexpr int kThreads = 512;

// Byte offset of the 16-byte run of tokens [8 k, 8 k + 8) of channel p in a [64][256] fp16 tile.
// The run index is XOR-ed with four bits of p chosen so that both accesses are free of bank
// conflicts: 16 consecutive channels at one k (the MFMA operand; bijective in p3 p2 p1 p0) and
// channels p, p + 8, .. p + 56 at k, k + 1 (the producer's writes; its upper three bits bijective
// in p5 p4 p3).
__device__ __forceinline__ int xs_offset(int p, int k) {
  const int g = ((((p >> 5) ^ (p >> 2)) & 1) << 3) | ((((p >> 4) ^ (p >> 1)) & 1) << 2) |
                (((p >> 3) & 1) << 1) | (p & 1);
  return p * (kQ * 2) + ((k ^ g) << 4);
}

template <typename XT>
__global__ __launch_bounds__(kThreads, 4) void fp16_walk_kernel(
    const XT* __restrict__ x, const float* __restrict__ dt, const float* __restrict__ A,
    const _Float16* __restrict__ bT_frag, int dt_softplus, const float* __restrict__ init,
    _Float16* __restrict__ pin, float* __restrict__ final_state, int L, int H, int G, int nc) {
  struct __attribute__((aligned(16))) Smem {
    float lut[kQ];       // dt_j exp(cs_last - cs_j)
    float stage[kQ];     // the terms of an inexact scan
    double scan[kScanScratch];
    float decay[2];      // exp(cs_last) of chunks of either parity
    alignas(16) uint8_t xs[2][kP * kQ * 2];   // X~^T of chunks of either parity
  };
  __shared__ Smem sm;

  const int t = threadIdx.x, lane = t & 63;
  const int wv = __builtin_amdgcn_readfirstlane(t >> 6);
  const int bh = xcd_remap(blockIdx.x, gridDim.x);
  // wave-uniform (the divisions run on the vector unit)
  const int b = __builtin_amdgcn_readfirstlane(bh / H);
  const int h = __builtin_amdgcn_readfirstlane(bh - b * H);
  const int g = __builtin_amdgcn_readfirstlane(h / (H / G));
  uint32_t* sr = reinterpret_cast<uint32_t*>(sm.scan + 4);

  // Both roles pass the same barriers: two per chunk (scan totals, LUT), a third when the scan is
  // inexact (the test reads the same words in every wave).  X~ and the decay of chunk c are there
  // for the consumers after the scan barrier of chunk c + 1, and its buffers are written again
  // after the one of chunk c + 2, which the consumers reach when they have read them.
  if (wv < 4) {
    // ---- x -> X~, one chunk ahead of the products
    // this thread: channels [8 ch, 8 ch + 8) of tokens [8 tg, 8 tg + 8), one 16-byte (fp32: two)
    // load per token: few enough loads that two chunks stay within the 63 a wave can have counted
    const size_t HP = (size_t)H * kP;
    const int ch = t & 7, tg = t >> 3;
    const float Ah = A[h];
    constexpr int kAhead = sizeof(XT) == 2 ? 2 : 1;   // chunks of x in flight (register sets)
    constexpr int kV = sizeof(XT) / 2;                // 16-byte loads per token
    uint4 xr[kAhead][8 * kV];
    float dtr[kAhead];
    // dt and x of chunk cc (nothing is read past the last chunk: an empty buffer returns zeros)
    auto load = [&](int cc, uint4 (&xv)[8 * kV], float& dv) {
      const bool in = cc < nc;
      const size_t tok = (size_t)b * L + (size_t)(in ? cc : 0) * kQ;
      // 2^32 - 1 or 0 by scalar arithmetic (a select runs on the vector unit, and every access
      // with that resource in a loop)
      int past = cc - nc;
      asm("" : "+s"(past));
      const uint32_t n = (uint32_t)(past >> 31);
      const __amdgpu_buffer_rsrc_t drs = uniform_rsrc(dt + tok * H + h, n);
      dv = __uint_as_float(buf_load4(drs, (uint32_t)(t * H * 4), 0));
      const __amdgpu_buffer_rsrc_t xrs = uniform_rsrc(x + tok * HP + (size_t)h * kP, n);
      const uint32_t xo = (uint32_t)((tg * 8 * HP + ch * 8) * sizeof(XT));
#pragma unroll
      for (int r = 0; r < 8; ++r)
#pragma unroll
        for (int i = 0; i < kV; ++i)
          xv[r * kV + i] = buf_load16(xrs, xo + 16 * i, (uint32_t)(r * HP * sizeof(XT)));
    };
    // X~ of channel i of tokens r and r + 1
    auto lut_x = [](const uint4 (&xv)[8 * kV], int r, int i, float l0, float l1) {
      auto word = [&](int row, int k) {
        const uint4 v = xv[row];
        return k == 0 ? v.x : k == 1 ? v.y : k == 2 ? v.z : v.w;
      };
      if constexpr (kV == 1) {
        const uint32_t w0 = word(r, i >> 1), w1 = word(r + 1, i >> 1);
        return (i & 1) ? lut_x2<1>(l0, w0, l1, w1) : lut_x2<0>(l0, w0, l1, w1);
      } else {
        const int k = i & 3, q = i >> 2;
        return lut_x2(l0, __uint_as_float(word(2 * r + q, k)), l1,
                      __uint_as_float(word(2 * r + 2 + q, k)));
      }
    };
    // chunk cc: its register set becomes X~ in LDS, then takes chunk cc + kAhead
    auto produce = [&](int cc, uint4 (&xv)[8 * kV], float& dv) {
      const float dtv = dt_softplus ? softplus_f32(dv) : dv;
      const float dA = dtv * Ah;
      double v;
      uint32_t er;
      wave_scan_f64(dA, v, er);
      if (lane == 63) {
        sm.scan[wv] = v;
        sr[wv] = er;
      }
      __syncthreads();
      double cs, last;
      if (scan_is_exact(sr)) {
        double pre = 0.0;
        for (int i = 0; i < wv; ++i) pre += sm.scan[i];
        cs = v + pre;
        // exact sums: the total may be added in any order
        last = (sm.scan[0] + sm.scan[1]) + (sm.scan[2] + sm.scan[3]);
      } else {
        sm.stage[t] = dA;
        __syncthreads();
        cs = exact_sum_f32_outlined(sm.stage, t + 1);
        last = exact_sum_f32_outlined(sm.stage, kQ);
      }
      sm.lut[t] = dtv * (float)exp(last - cs);
      if (t == 0) sm.decay[cc & 1] = (float)exp(last);
      __syncthreads();
      uint8_t* xs = sm.xs[cc & 1];
      float lut[8];
#pragma unroll
      for (int r = 0; r < 8; ++r) lut[r] = sm.lut[tg * 8 + r];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        uint32_t w[4];
#pragma unroll
        for (int u = 0; u < 4; ++u)
          w[u] = lut_x(xv, 2 * u, i, lut[2 * u], lut[2 * u + 1]);
        *reinterpret_cast<uint4*>(xs + xs_offset(8 * ch + i, tg)) =
            make_uint4(w[0], w[1], w[2], w[3]);
      }
      load(cc + kAhead, xv, dv);
    };
    load(0, xr[0], dtr[0]);
    if constexpr (kAhead == 2) load(1, xr[1], dtr[1]);
    for (int c = 0; c <= nc; c += 2) {
      produce(c, xr[0], dtr[0]);
      if (c + 1 <= nc) produce(c + 1, xr[kAhead - 1], dtr[kAhead - 1]);
    }
  } else {
    // ---- P_in out, P <- exp(cs_last) P + B^T X~ (rows n, columns p)
    const int nt = wv - 4;
    const uint32_t lane16 = lane * 16;
    // P[mt]: lane -> channel p = 32 mt + lane % 32, register 4 q + i -> n = 32 nt + 8 q + 4 half + i
    v16f P0 = {}, P1 = {};
    // (formed where it is used: held across the loop it would spill)
    auto state_row = [&](int l) {
      return ((size_t)bh * kP + (l & 31)) * kN + 32 * nt + 4 * (l >> 5);
    };
    if (init) {
      const size_t srow = state_row(lane);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float4 f0 = *reinterpret_cast<const float4*>(init + srow + 8 * q);
        const float4 f1 = *reinterpret_cast<const float4*>(init + srow + 32 * kN + 8 * q);
        P0[4 * q] = f0.x; P0[4 * q + 1] = f0.y; P0[4 * q + 2] = f0.z; P0[4 * q + 3] = f0.w;
        P1[4 * q] = f1.x; P1[4 * q + 1] = f1.y; P1[4 * q + 2] = f1.z; P1[4 * q + 3] = f1.w;
      }
    }
    constexpr int kS = kQ / 16, kF = 12;  // K-steps of a chunk; B^T fragments in flight
    auto b_rsrc = [&](int cc) {   // the last chunk's again past the end
      const size_t bc = (size_t)b * nc + (cc < nc ? cc : nc - 1);
      return uniform_rsrc(bT_frag + (bc * G + g) * (size_t)kN * kQ + (size_t)nt * kS * 512);
    };
    uint4 f[kF];
    {
      const __amdgpu_buffer_rsrc_t brs = b_rsrc(0);
#pragma unroll
      for (int ks = 0; ks < kF; ++ks) f[ks] = buf_load16(brs, lane16, 1024 * ks);
    }
    auto pass_scan = [&]() {
      __syncthreads();
      if (!scan_is_exact(sr)) __syncthreads();
    };
    pass_scan();          // chunk 0
    __syncthreads();
    if (nc > 0) pass_scan();   // chunk 1: X~ of chunk 0 is there
    for (int c = 0; c < nc; ++c) {
      _Float16* dst = pin + (((size_t)b * nc + c) * H + h) * (size_t)kP * kN +
                      (size_t)(2 * nt) * 512 + lane * 8;
      auto put = [&](const v16f& P, _Float16* o) {
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
          *reinterpret_cast<uint4*>(o + kb * 512) = make_uint4(
              pack_h2(P[8 * kb], P[8 * kb + 1]), pack_h2(P[8 * kb + 2], P[8 * kb + 3]),
              pack_h2(P[8 * kb + 4], P[8 * kb + 5]), pack_h2(P[8 * kb + 6], P[8 * kb + 7]));
      };
      put(P0, dst);
      put(P1, dst + (kN / 16) * 512);
      __syncthreads();   // LUT of chunk c + 1
      const __amdgpu_buffer_rsrc_t bcur = b_rsrc(c), brs = b_rsrc(c + 1);
      const uint8_t* xs = sm.xs[c & 1];
      // opaque per chunk: its addresses are formed here and not held across the loop
      int l = lane;
      asm volatile("" : "+v"(l));
      const int pc = l & 31, half = l >> 5;
      // S on its own from zero, then one rounding into P, as ChunkState and StatePassing form them
      // (bit-equal to those)
      v16f S0, S1;
#pragma unroll
      for (int ks = 0; ks < kS; ++ks) {
        const v8h bf = __builtin_bit_cast(v8h, f[ks < kF ? ks : ks - kF]);
        const v8h a0 = *reinterpret_cast<const v8h*>(xs + xs_offset(pc, 2 * ks + half));
        const v8h a1 = *reinterpret_cast<const v8h*>(xs + xs_offset(32 + pc, 2 * ks + half));
        S0 = __builtin_amdgcn_mfma_f32_32x32x16_f16(bf, a0, ks ? S0 : (v16f){}, 0, 0, 0);
        S1 = __builtin_amdgcn_mfma_f32_32x32x16_f16(bf, a1, ks ? S1 : (v16f){}, 0, 0, 0);
        // the slot's next fragment: of this chunk's end, or of the next chunk
        if (ks < kS - kF) f[ks] = buf_load16(bcur, lane16, 1024 * (ks + kF));
        else f[ks < kF ? ks : ks - kF] = buf_load16(brs, lane16, 1024 * (ks < kF ? ks : ks - kF));
      }
      // (one value per workgroup; read here, as the producers may write it after the next barrier)
      const float d = __uint_as_float(
          __builtin_amdgcn_readfirstlane((int)__float_as_uint(sm.decay[c & 1])));
      if (c + 1 < nc) pass_scan();   // chunk c + 2: X~ of chunk c + 1 is there
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        P0[r] = __builtin_fmaf(d, P0[r], S0[r]);
        P1[r] = __builtin_fmaf(d, P1[r], S1[r]);
      }
    }
    if (final_state) {
      int l = threadIdx.x & 63;
      asm volatile("" : "+v"(l));
      const size_t srow = state_row(l);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        *reinterpret_cast<float4*>(final_state + srow + 8 * q) =
            make_float4(P0[4 * q], P0[4 * q + 1], P0[4 * q + 2], P0[4 * q + 3]);
        *reinterpret_cast<float4*>(final_state + srow + 32 * kN + 8 * q) =
            make_float4(P1[4 * q], P1[4 * q + 1], P1[4 * q + 2], P1[4 * q + 3]);
      }
    }
  }
}

}  // namespace

hipError_t launch_fp16_walk(const LayerDims& d, const void* x, int x_dtype, const float* dt,
                            int dt_softplus, const float* A, const _Float16* bT_frag,
                            const float* init, _Float16* pin, float* final_state,
                            hipStream_t st) {
  const int64_t nwork = (int64_t)d.batch * d.nheads;
  if (nwork == 0) return hipSuccess;
#define SSDI8_WALK_LAUNCH(XT)                                                                  \
  hipLaunchKernelGGL(fp16_walk_kernel<XT>, dim3((unsigned)nwork), dim3(kThreads), 0, st,        \
                     static_cast<const XT*>(x), dt, A, bT_frag, dt_softplus, init, pin,        \
                     final_state, d.seqlen, d.nheads, d.ngroups, d.nchunks)
  if (x_dtype == 1) SSDI8_WALK_LAUNCH(_Float16);
  else SSDI8_WALK_LAUNCH(float);
#undef SSDI8_WALK_LAUNCH
  return hipGetLastError();
}

}  // namespace ssdi8
