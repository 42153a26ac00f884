// FP16 baseline, ChunkScan1 + ChunkScan2 + output (Alg. 2 modules 5-6 without quantization):
//   Scan1  Y1[j, p] = sum_n C[j, n] fp16(P_in[p, n])      fp16 MFMA, fp32 accumulation
//   Scan2  W[j, i]  = fp16(CB[j, i] dt_i exp(cs_j - cs_i)), i <= j;  y_diag = W . x
//   y = Y1 exp(cs_j) + y_diag + D x
// The structure is the INT8 ChunkScan's (one workgroup per (b, c, h), transposed products so a
// lane owns a token row, x^T staged once in LDS, block-factorised decay, output staged
// through LDS), with fp32 CB blocks in place of the int8 ones.  P_in arrives as the fp16 operand
// itself: StatePassing rounds its fp32 running state once, where it writes it.
//
// What bounds it: operand bytes through L1/L2 (CB 147 KB, C 64 KB, P_in per workgroup) beside the
// x / y stream.  So each wave runs Scan1 of both of its row blocks from one load of P_in (64 KB
// per workgroup; per row block, in fp32, it was 256 KB), its result seeds the Scan2 accumulators,
// and CB blocks that decay makes zero weights of are not loaded.  At most 127 VGPRs and 37 KB of LDS
// keep four workgroups per CU (three before).  2.7B-shaped layer, slow heads included: 209 -> 99.5 us;
// 130M-shaped: 51.5 -> 33.8 us.
#include "common.hpp"
#include "fp16_rows.hpp"
#include "frag.hpp"
#include "launch.hpp"

namespace ssdi8 {

namespace {

using namespace fp16;

template <typename XT, typename YT>
__global__ __launch_bounds__(256, 4) void fp16_scan_kernel(
    const XT* __restrict__ x, const float* __restrict__ dt, const float* __restrict__ A,
    const _Float16* __restrict__ c_frag, const _Float16* __restrict__ pin,
    const float* __restrict__ cb, const float* __restrict__ cb_max,
    const float* __restrict__ Dv, int dt_softplus, YT* __restrict__ y, int L, int H, int G, int nc,
    int stream) {
  struct __attribute__((aligned(16))) Smem {
    Tables tab;
    double scan[kScanScratch];
    alignas(16) uint8_t xT[kP * kXTS];   // 128-bit accesses: 16-byte aligned explicitly
  };
  __shared__ Smem sm;
  uint8_t* s_xT = sm.xT;

  const int t = threadIdx.x, lane = t & 63;
  const int wv = __builtin_amdgcn_readfirstlane(t >> 6);
  const int w = xcd_remap(blockIdx.x, gridDim.x);
  const int h = w % H;
  const int bc = w / H;
  const int c = bc % nc;
  const int b = bc / nc;
  const int g = h / (H / G);
  const size_t tok0 = (size_t)b * L + (size_t)c * kQ;
  const size_t HP = (size_t)H * kP;

  const int pp = t & 31, jb = t >> 5, p0 = 2 * pp;
  typename Pair<XT>::raw xr[32];
  {
    const __amdgpu_buffer_rsrc_t xrs = uniform_rsrc(x + tok0 * HP + (size_t)h * kP);
    const uint32_t xo = (uint32_t)((jb * 32 * HP + p0) * sizeof(XT));
    // x and y streamed when they exceed the Infinity Cache, as in the INT8 layer's scan
    if (stream) {
#pragma unroll
      for (int r = 0; r < 32; ++r)
        xr[r] = Pair<XT>::template load<kPolicyNT>(xrs, xo, (uint32_t)(r * HP * sizeof(XT)));
    } else {
#pragma unroll
      for (int r = 0; r < 32; ++r) xr[r] = Pair<XT>::load(xrs, xo, (uint32_t)(r * HP * sizeof(XT)));
    }
  }

  float dtv = dt[(tok0 + t) * H + h];
  if (dt_softplus) dtv = softplus_f32(dtv);   // the dt of this layer's ChunkState
  const float dA = dtv * A[h];
  const double cs = block_scan_f64_256(dA, sm.scan, sm.tab.u);
  if ((t & 31) == 31) sm.tab.r[t >> 5] = cs;
  __syncthreads();
  build_tables(sm.tab, t, dtv, cs);
  {
    uint8_t* r0 = s_xT + p0 * kXTS + jb * 64;
    uint8_t* r1 = r0 + kXTS;
    h2_t fin = {};   // 0, NaN where one of the values is not finite
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      uint32_t a[4], bb[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int r = 8 * q + 2 * u;
        a[u] = (uint32_t)Pair<XT>::lo(xr[r]) | ((uint32_t)Pair<XT>::lo(xr[r + 1]) << 16);
        bb[u] = (uint32_t)Pair<XT>::hi(xr[r]) | ((uint32_t)Pair<XT>::hi(xr[r + 1]) << 16);
        fin = __builtin_elementwise_fma(__builtin_bit_cast(h2_t, a[u]), (h2_t){}, fin);
        fin = __builtin_elementwise_fma(__builtin_bit_cast(h2_t, bb[u]), (h2_t){}, fin);
      }
      *reinterpret_cast<uint4*>(r0 + 16 * q) = make_uint4(a[0], a[1], a[2], a[3]);
      *reinterpret_cast<uint4*>(r1 + 16 * q) = make_uint4(bb[0], bb[1], bb[2], bb[3]);
    }
    // A zero weight times an infinite or NaN x is NaN, so the blocks of these 32 tokens are not
    // skipped then (this wave wrote umax[jb] in build_tables; one instruction per pair of x)
    if (!(fin.x == fin.x && fin.y == fin.y)) sm.tab.umax[jb] = __builtin_inff();
  }
  __syncthreads();

  const size_t cg = ((size_t)b * nc + c) * G + g;
  const __amdgpu_buffer_rsrc_t prs =
      uniform_rsrc(pin + (((size_t)b * nc + c) * H + h) * (size_t)kP * kN);
  const __amdgpu_buffer_rsrc_t cbrs = uniform_rsrc(cb + cg * (size_t)frag::kCbBlocks * 1024);
  const __amdgpu_buffer_rsrc_t cqrs = uniform_rsrc(c_frag + cg * (size_t)kQ * kN);
  const uint32_t lane16 = lane * 16;
  const float Dh = Dv ? Dv[h] : 0.0f;
  const int jta = wv, jtb = 7 - wv;   // this wave's row blocks
  const float cma = block_max(cb_max + cg * frag::kCbBlocks, jta, lane);
  float cmb = 0.0f;   // fp32 x has no register for it during Scan1
  if constexpr (sizeof(XT) == 2) cmb = block_max(cb_max + cg * frag::kCbBlocks, jtb, lane);

  // -- Scan1 of both row blocks: Y1^T = fp16(P_in) . C^T over n (8 K-steps of 16).  The P_in
  //    fragments (fp16, as StatePassing leaves them) serve both blocks from one load.
  v16f ya0 = {}, ya1 = {}, yb0 = {}, yb1 = {};
  {
    const uint32_t ca = jta * (kN / 16) * 1024, cbo = jtb * (kN / 16) * 1024;
#pragma unroll
    for (int ks = 0; ks < kN / 16; ++ks) {
      const v8h p0f = __builtin_bit_cast(v8h, buf_load16(prs, lane16, ks * 1024));
      const v8h p1f = __builtin_bit_cast(v8h, buf_load16(prs, lane16, (kN / 16 + ks) * 1024));
      const v8h fa = __builtin_bit_cast(v8h, buf_load16(cqrs, lane16, ca + 1024 * ks));
      const v8h fb = __builtin_bit_cast(v8h, buf_load16(cqrs, lane16, cbo + 1024 * ks));
      ya0 = __builtin_amdgcn_mfma_f32_32x32x16_f16(p0f, fa, ya0, 0, 0, 0);
      ya1 = __builtin_amdgcn_mfma_f32_32x32x16_f16(p1f, fa, ya1, 0, 0, 0);
      yb0 = __builtin_amdgcn_mfma_f32_32x32x16_f16(p0f, fb, yb0, 0, 0, 0);
      yb1 = __builtin_amdgcn_mfma_f32_32x32x16_f16(p1f, fb, yb1, 0, 0, 0);
    }
  }

  const XT* xg = x + tok0 * HP + (size_t)h * kP;
  row_block<XT>(jta, lane, sm.tab, s_xT, cbrs, cma, xg, HP, Dh, ya0, ya1);
  if constexpr (sizeof(XT) == 4) cmb = block_max(cb_max + cg * frag::kCbBlocks, jtb, lane);
  row_block<XT>(jtb, lane, sm.tab, s_xT, cbrs, cmb, xg, HP, Dh, yb0, yb1);

  // -- output: the two row blocks leave through the x^T bytes as whole token rows
  __syncthreads();
  if constexpr (sizeof(YT) == 8) {
    channel_sums(reinterpret_cast<double*>(s_xT), wv, lane, ya0, ya1, yb0, yb1,
                 y + ((size_t)b * nc + c) * HP + (size_t)h * kP);
    return;
  }
  const __amdgpu_buffer_rsrc_t yrs = uniform_rsrc(y + tok0 * HP + (size_t)h * kP);
  if constexpr (sizeof(YT) == 2) {
    stage_rows_f16(s_xT, jta, lane, ya0, ya1);
    stage_rows_f16(s_xT, jtb, lane, yb0, yb1);
    __syncthreads();
    rows_out<128, 256>(s_xT, yrs, t, HP, 0, stream);
  } else if constexpr (sizeof(YT) == 4) {
    stage_rows_f32(s_xT, jta, lane, ya0, ya1);
    __syncthreads();
    rows_out<256, 256>(s_xT, yrs, t, HP, 0, stream);
    __syncthreads();
    stage_rows_f32(s_xT, jtb - 4, lane, yb0, yb1);
    __syncthreads();
    rows_out<256, 256>(s_xT, yrs, t, HP, 128, stream);
  }
}

}  // namespace

hipError_t launch_fp16_scan(const LayerDims& d, const void* x, int x_dtype, const float* dt,
                            int dt_softplus, const float* A, const _Float16* c_frag,
                            const _Float16* pin, const float* cb, const float* cb_max,
                            const float* D, void* y, int y_dtype, hipStream_t st) {
  const int64_t nwork = (int64_t)d.batch * d.nchunks * d.nheads;
  if (nwork == 0) return hipSuccess;
  const int stream = stream_xy(d, x_dtype == 1 ? 2 : 4, y_dtype == kYSums ? 0 : y_dtype == 1 ? 2 : 4);
#define SSDI8_F16SCAN_LAUNCH(XT, YT)                                                           \
  hipLaunchKernelGGL((fp16_scan_kernel<XT, YT>), dim3((unsigned)nwork), dim3(256), 0, st,       \
                     static_cast<const XT*>(x), dt, A, c_frag, pin, cb, cb_max, D, dt_softplus, \
                     static_cast<YT*>(y), d.seqlen, d.nheads, d.ngroups, d.nchunks, stream)
  if (x_dtype == 1 && y_dtype == kYSums) SSDI8_F16SCAN_LAUNCH(_Float16, double);
  else if (y_dtype == kYSums) SSDI8_F16SCAN_LAUNCH(float, double);
  else if (x_dtype == 1 && y_dtype == 1) SSDI8_F16SCAN_LAUNCH(_Float16, _Float16);
  else if (x_dtype == 1) SSDI8_F16SCAN_LAUNCH(_Float16, float);
  else if (y_dtype == 1) SSDI8_F16SCAN_LAUNCH(float, _Float16);
  else SSDI8_F16SCAN_LAUNCH(float, float);
#undef SSDI8_F16SCAN_LAUNCH
  return hipGetLastError();
}

}  // namespace ssdi8
