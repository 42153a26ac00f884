// Static-step calibration and the single-layer mean correction on the device (Sec. 5 setup:
// symmetric static steps from a calibration draw; Eq. 10 / Alg. 1 restricted to one layer).
//   alpha_B, alpha_C   absmax / 127 per group            (the dynamic quantizer, Eq. 1)
//   alpha_Xs           absmax of X_scaled = LUT_state x per (h, p) or per h   (Eq. 7)
//   alpha_S            absmax over (b, c, n) of the chunk-local and the passed fp states,
//                      per (h, p) (Eq. 8: the int8 states must rarely saturate)
//   alpha_CB           absmax of the causal entries of C B^T per group
//   corr[h, p]         eta * mean over (b, l) of (Y_fp - Y_q), Y_q the INT8 layer with corr = 0
// X_scaled is formed with exactly the fp32 operations of ChunkState, so alpha_Xs is exact.  The fp
// states are accumulated from x~ = fl32(LUT x) split into two fp16 parts (hi = fp16(x~),
// lo = fp16(x~ - hi)), about 22 significant bits, times fp16 B, in fp32; C B^T of fp16 C, B is
// exact per product and summed in fp32.  Y_fp is the FP16 layer.
#include <type_traits>

#include "common.hpp"
#include "fp16_rows.hpp"
#include "frag.hpp"
#include "launch.hpp"

namespace ssdi8 {

namespace {

constexpr int kXS = kQ * 2 + 16;

// ---- per (b, c, h): the absmax over the chunk's tokens of |x~| per channel, x~ = fl32(LUT x) (alpha_Xs),
//      and the fp states of the chunk from the split x~ (two fp16 MFMA products), in the plane
//      order of the FP16 path's S, plus the chunk decay exp(cs_last) in fp64.  x is read once for
//      both, its loads under way during the ChunkCumsum; the product is formed transposed (rows n),
//      so the states go to memory from the accumulators.  26 + 66 us as two kernels that loaded x
//      inside their loops and staged the states in LDS -> 43 us (2.7B-shaped, 8192 tokens).
template <typename XT>
__global__ __launch_bounds__(256) void calib_state_kernel(
    const XT* __restrict__ x, const float* __restrict__ dt, const float* __restrict__ A,
    const _Float16* __restrict__ bT_frag, int dt_softplus, uint32_t* __restrict__ xs_amax,
    float* __restrict__ S, double* __restrict__ dec64, int L, int H, int G, int nc) {
  __shared__ __attribute__((aligned(16))) uint8_t s_x[kP * kXS];
  __shared__ float s_lut[kQ];
  __shared__ double s_scan[kScanScratch];
  __shared__ double s_last;
  __shared__ float s_m[8][kP];
  const int t = threadIdx.x, lane = t & 63;
  const int wv = __builtin_amdgcn_readfirstlane(t >> 6);
  const int w = xcd_remap(blockIdx.x, gridDim.x);
  const int h = w % H, bc = w / H, c = bc % nc, b = bc / nc;
  const int g = h / (H / G);
  const size_t tok0 = (size_t)b * L + (size_t)c * kQ;
  const size_t HP = (size_t)H * kP;
  const int pp = t & 31, jb = t >> 5, p0 = 2 * pp;
  typename fp16::Pair<XT>::raw xr[32];
  {
    const __amdgpu_buffer_rsrc_t xrs = uniform_rsrc(x + tok0 * HP + (size_t)h * kP);
    const uint32_t xo = (uint32_t)((jb * 32 * HP + p0) * sizeof(XT));
#pragma unroll
    for (int r = 0; r < 32; ++r)
      xr[r] = fp16::Pair<XT>::load(xrs, xo, (uint32_t)(r * HP * sizeof(XT)));
  }
  // ChunkCumsum as in ChunkState
  float dtv = dt[(tok0 + t) * H + h];
  if (dt_softplus) dtv = softplus_f32(dtv);
  const float dA = dtv * A[h];
  const double cs = block_scan_f64_256<true>(dA, s_scan, s_lut);
  if (t == kQ - 1) s_last = cs;
  __syncthreads();
  const double last = s_last;
  s_lut[t] = dtv * (float)exp(last - cs);
  if (t == 0) dec64[((size_t)b * H + h) * nc + c] = exp(last);
  __syncthreads();
  // x~ = hi + lo (+ a remainder below 2^-22 |x~|), both parts as fp16, transposed ([p][j], tokens
  // contiguous); the hi parts go through the LDS first, then the lo parts, formed again from x
  float m0 = 0.0f, m1 = 0.0f;
  auto stage = [&](auto low) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      uint32_t wa[4], wb[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        _Float16 va[2], vb[2];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          const int r = 8 * q + 2 * u + e;
          const float lut = s_lut[jb * 32 + r];
          const float xa = lut * fp16::Pair<XT>::lof(xr[r]), xb = lut * fp16::Pair<XT>::hif(xr[r]);
          va[e] = (_Float16)xa;
          vb[e] = (_Float16)xb;
          if constexpr (decltype(low)::value) {
            va[e] = (_Float16)(xa - (float)va[e]);
            vb[e] = (_Float16)(xb - (float)vb[e]);
          } else {
            m0 = __builtin_fmaxf(m0, __builtin_fabsf(xa));
            m1 = __builtin_fmaxf(m1, __builtin_fabsf(xb));
          }
        }
        wa[u] = __builtin_bit_cast(uint16_t, va[0]) |
                ((uint32_t)__builtin_bit_cast(uint16_t, va[1]) << 16);
        wb[u] = __builtin_bit_cast(uint16_t, vb[0]) |
                ((uint32_t)__builtin_bit_cast(uint16_t, vb[1]) << 16);
      }
      uint8_t* o = s_x + p0 * kXS + jb * 64 + 16 * q;
      *reinterpret_cast<uint4*>(o) = make_uint4(wa[0], wa[1], wa[2], wa[3]);
      *reinterpret_cast<uint4*>(o + kXS) = make_uint4(wb[0], wb[1], wb[2], wb[3]);
    }
  };
  // S^T = B^T x~ (rows n, columns p): wave -> n-tile wv and both p-tiles
  const int half = lane >> 5;
  const __amdgpu_buffer_rsrc_t brs =
      uniform_rsrc(bT_frag + (((size_t)b * nc + c) * G + g) * (size_t)kN * kQ +
                   (size_t)wv * (kQ / 16) * 512);
  const uint8_t* arow = s_x + (lane & 31) * kXS + 16 * half;
  v16f acc0 = {}, acc1 = {};
  auto product = [&]() {
#pragma unroll 8
    for (int ks = 0; ks < kQ / 16; ++ks) {
      const v8h bf = __builtin_bit_cast(v8h, buf_load16(brs, lane * 16, 1024 * ks));
      const v8h a0 = *reinterpret_cast<const v8h*>(arow + ks * 32);
      const v8h a1 = *reinterpret_cast<const v8h*>(arow + 32 * kXS + ks * 32);
      acc0 = __builtin_amdgcn_mfma_f32_32x32x16_f16(bf, a0, acc0, 0, 0, 0);
      acc1 = __builtin_amdgcn_mfma_f32_32x32x16_f16(bf, a1, acc1, 0, 0, 0);
    }
  };
  stage(std::false_type{});
  s_m[jb][p0] = m0;
  s_m[jb][p0 + 1] = m1;
  __syncthreads();
  if (t < kP) {
    float m = 0.0f;
#pragma unroll
    for (int k = 0; k < 8; ++k) m = __builtin_fmaxf(m, s_m[k][t]);
    atomicMax(xs_amax + h * kP + t, __float_as_uint(m));
  }
  product();
  __syncthreads();
  stage(std::true_type{});
  __syncthreads();
  product();
  float* dst = S + (((size_t)b * nc + c) * H + h) * (size_t)kP * kN + (size_t)wv * 1024 + lane * 4;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    *reinterpret_cast<float4*>(dst + 256 * q) =
        make_float4(acc0[4 * q], acc0[4 * q + 1], acc0[4 * q + 2], acc0[4 * q + 3]);
    *reinterpret_cast<float4*>(dst + (kN / 32) * 1024 + 256 * q) =
        make_float4(acc1[4 * q], acc1[4 * q + 1], acc1[4 * q + 2], acc1[4 * q + 3]);
  }
}

// ---- absmax of the chunk-local states and of the states after each chunk (fp64 passing, as
//      the calibration reference) per (h, p); 4 elements (one p) per thread
__global__ __launch_bounds__(256) void calib_pass_kernel(const float* __restrict__ S,
                                                         const double* __restrict__ dec64,
                                                         uint32_t* __restrict__ s_amax, int nc,
                                                         int H, int64_t nthreads) {
  constexpr int64_t kE = (int64_t)kP * kN;
  const int64_t gt = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (gt >= nthreads) return;
  const int64_t e = gt * 4;
  const int64_t bh = e / kE;
  const int64_t off = e - bh * kE;
  const int64_t b = bh / H, h = bh - b * H;
  // plane order: 256 floats of a run of four n, four per lane; 16 planes per channel tile
  const int p = (int)(off >> 12 << 5) | (int)((off >> 2) & 31);
  double run[4] = {0.0, 0.0, 0.0, 0.0};
  float m = 0.0f;
  const size_t cstride = (size_t)H * kE;
  const size_t base = ((size_t)b * nc * H + h) * kE + off;
  for (int c = 0; c < nc; ++c) {
    const float4 s = *reinterpret_cast<const float4*>(S + base + (size_t)c * cstride);
    const double d = dec64[bh * nc + c];
    const float sv[4] = {s.x, s.y, s.z, s.w};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      run[q] = (double)sv[q] + d * run[q];
      m = __builtin_fmaxf(m, __builtin_fmaxf(__builtin_fabsf(sv[q]),
                                             (float)__builtin_fabs(run[q])));
    }
  }
  // lanes l and l ^ 32 hold the same p; every workgroup is whole (the thread count is a multiple
  // of 256), so the shuffle is safe
  m = __builtin_fmaxf(m, __shfl_xor(m, 32, 64));
  if ((threadIdx.x & 32) == 0) atomicMax(s_amax + h * kP + p, __float_as_uint(m));
}

// ---- steps from the absolute maxima: block b < nsteps the x and state steps of 256 channels, the
//      others the C.B^T step of one group each, from the maxima of its 36 blocks per chunk
//      (cb_max [ncg, 36], chunk-groups of a group G apart, the sign bit for NaNs left out; one
//      atomic per block on one word per group took ChunkBMM from 7 to 19 us)
__global__ __launch_bounds__(256) void calib_steps_kernel(
    const uint32_t* __restrict__ xs_amax, const uint32_t* __restrict__ s_amax,
    const float* __restrict__ cb_max, float* __restrict__ aXs, float* __restrict__ aS,
    float* __restrict__ aCB, int H, int G, int xs_per_head, int nsteps, int nchunks) {
  if ((int)blockIdx.x >= nsteps) {
    __shared__ float wmax[4];
    const int g = blockIdx.x - nsteps;
    const int n = nchunks * frag::kCbBlocks;
    float m = 0.0f;
    for (int i = threadIdx.x; i < n; i += 256) {
      const int c = i / frag::kCbBlocks, k = i - c * frag::kCbBlocks;
      m = __builtin_fmaxf(m, __builtin_fabsf(cb_max[((size_t)c * G + g) * frag::kCbBlocks + k]));
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) m = __builtin_fmaxf(m, __shfl_xor(m, o, 64));
    if ((threadIdx.x & 63) == 0) wmax[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
      m = __builtin_fmaxf(__builtin_fmaxf(wmax[0], wmax[1]), __builtin_fmaxf(wmax[2], wmax[3]));
      const float a = (float)((double)m / 127.0);
      aCB[g] = a == 0.0f ? 1.0f : a;
    }
    return;
  }
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t < H * kP) {
    const float sm = __uint_as_float(s_amax[t]);
    const float a = (float)((double)sm / 127.0);
    aS[t] = a == 0.0f ? 1.0f : a;
    if (!xs_per_head) {
      const float x = __uint_as_float(xs_amax[t]) / 127.0f;
      aXs[t] = x == 0.0f ? 1.0f : x;
    }
  }
  if (xs_per_head && t < H) {
    float m = 0.0f;
    for (int p = 0; p < kP; ++p) m = __builtin_fmaxf(m, __uint_as_float(xs_amax[t * kP + p]));
    const float x = m / 127.0f;
    aXs[t] = x == 0.0f ? 1.0f : x;
  }
}

// ---- corr[h, p] = eta * mean over (b, l) of (y_fp - y_q), in fp64 and in a fixed order, from the
//      channel sums both layers' scan kernels leave per chunk ([rows, H P], rows = batch chunks):
//      64 channels per workgroup, four row ranges
__global__ __launch_bounds__(256) void calib_corr_kernel(const double* __restrict__ s_fp,
                                                         const double* __restrict__ s_q,
                                                         float* __restrict__ corr, int rows, int HP,
                                                         double scale) {
  __shared__ double s_sum[4][kP];
  const int p = threadIdx.x & 63, q = threadIdx.x >> 6;
  const int i = blockIdx.x * kP + p;
  double s = 0.0;
#pragma unroll 8
  for (int r = (int)((int64_t)rows * q / 4); r < (int)((int64_t)rows * (q + 1) / 4); ++r)
    s += s_fp[(size_t)r * HP + i] - s_q[(size_t)r * HP + i];
  s_sum[q][p] = s;
  __syncthreads();
  if (threadIdx.x < kP)
    corr[i] = (float)(scale * ((s_sum[0][p] + s_sum[1][p]) + (s_sum[2][p] + s_sum[3][p])));
}

__global__ void zero_u32(uint32_t* p, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0u;
}

}  // namespace

hipError_t launch_calib_zero(uint32_t* p, int n, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(zero_u32, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, p, n);
  return hipGetLastError();
}

hipError_t launch_calib_states(const LayerDims& d, const void* x, int x_dtype, const float* dt,
                               int dt_softplus, const float* A, const _Float16* bT_frag,
                               uint32_t* xs_amax, float* S, double* dec64, uint32_t* s_amax,
                               hipStream_t st) {
  const int64_t nwork = (int64_t)d.batch * d.nchunks * d.nheads;
  if (nwork == 0) return hipSuccess;
  if (x_dtype == 1)
    hipLaunchKernelGGL(calib_state_kernel<_Float16>, dim3((unsigned)nwork), dim3(256), 0, st,
                       static_cast<const _Float16*>(x), dt, A, bT_frag, dt_softplus, xs_amax, S,
                       dec64, d.seqlen, d.nheads, d.ngroups, d.nchunks);
  else
    hipLaunchKernelGGL(calib_state_kernel<float>, dim3((unsigned)nwork), dim3(256), 0, st,
                       static_cast<const float*>(x), dt, A, bT_frag, dt_softplus, xs_amax, S,
                       dec64, d.seqlen, d.nheads, d.ngroups, d.nchunks);
  const int64_t nthreads = (int64_t)d.batch * d.nheads * kP * kN / 4;
  hipLaunchKernelGGL(calib_pass_kernel, dim3((unsigned)((nthreads + 255) / 256)), dim3(256), 0,
                     st, S, dec64, s_amax, d.nchunks, d.nheads, nthreads);
  return hipGetLastError();
}

hipError_t launch_calib_steps(const LayerDims& d, const uint32_t* xs_amax, const uint32_t* s_amax,
                              const float* cb_max, float* aXs, float* aS, float* aCB,
                              int xs_per_head, hipStream_t st) {
  const int nsteps = (d.nheads * kP + 255) / 256;
  hipLaunchKernelGGL(calib_steps_kernel, dim3((unsigned)(nsteps + d.ngroups)), dim3(256), 0, st,
                     xs_amax, s_amax, cb_max, aXs, aS, aCB, d.nheads, d.ngroups, xs_per_head,
                     nsteps, d.batch * d.nchunks);
  return hipGetLastError();
}

hipError_t launch_calib_corr(const LayerDims& d, const double* s_fp, const double* s_q,
                             float* corr, float eta, hipStream_t st) {
  const double T = (double)d.batch * (double)d.seqlen;
  hipLaunchKernelGGL(calib_corr_kernel, dim3((unsigned)d.nheads), dim3(256), 0, st, s_fp, s_q,
                     corr, d.batch * d.nchunks, d.nheads * kP, (double)eta / T);
  return hipGetLastError();
}

}  // namespace ssdi8
