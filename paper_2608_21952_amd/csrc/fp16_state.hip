// FP16 baseline, ChunkCumsum + ChunkState and StatePassing (Alg. 2 modules 1-3 without
// quantization):
//   dt, dA, cs, LUT_state    as in the INT8 ChunkState (fp64 softplus and in-chunk sum)
//   X~       = fp16(LUT_j x_jp), the exact product rounded once
//   S[p, n]  = sum_j X~[j, p] B[j, n]       fp16 MFMA 32x32x16 over tokens, fp32 accumulation
//   d        = fl32(exp(cs_last))
//   P_in[c+1] = fl32(d P_in[c] + S[c])      one fma per element, fp32 states
// fp16(P_in), ChunkScan1's operand, is kept in that operand's fragment order (frag::pk16_offset
// with rows p, K = n); S in the same order split into planes of four elements per lane (the order
// in which the accumulators hold it, so that every store covers a contiguous 1 KB); the initial
// and final states are row-major [p][n].
#include "common.hpp"
#include "fp16_rows.hpp"
#include "frag.hpp"
#include "launch.hpp"

namespace ssdi8 {

namespace {

constexpr int kXS = kQ * 2 + 16;   // LDS bytes per channel row of X~^T (fp16)

typedef _Float16 h8 __attribute__((ext_vector_type(8)));

template <typename XT>
__global__ __launch_bounds__(256) void fp16_state_kernel(
    const XT* __restrict__ x, const float* __restrict__ dt, const float* __restrict__ A,
    const _Float16* __restrict__ bT_frag, int dt_softplus, float* __restrict__ S,
    float* __restrict__ dec, int L, int H, int G, int nc) {
  __shared__ __attribute__((aligned(16))) uint8_t s_x[kP * kXS];
  __shared__ float s_lut[kQ];
  __shared__ double s_scan[kScanScratch];
  __shared__ double s_last;

  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const int w = xcd_remap(blockIdx.x, gridDim.x);
  const int h = w % H;
  const int bc = w / H;
  const int c = bc % nc;
  const int b = bc / nc;
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

  float dtv = dt[(tok0 + t) * H + h];
  if (dt_softplus) dtv = softplus_f32(dtv);
  const float dA = dtv * A[h];
  const double cs = block_scan_f64_256(dA, s_scan, s_lut);
  if (t == kQ - 1) s_last = cs;
  __syncthreads();
  const double last = s_last;
  s_lut[t] = dtv * (float)exp(last - cs);
  if (t == 0) dec[((size_t)b * H + h) * nc + c] = (float)exp(last);
  __syncthreads();

  // ---- X~ = fp16(LUT x), written transposed to LDS ([p][j], tokens contiguous)
  {
    uint32_t w0[16], w1[16];
#pragma unroll
    for (int r2 = 0; r2 < 16; ++r2) {
      const int r = 2 * r2;
      const float l0 = s_lut[jb * 32 + r], l1 = s_lut[jb * 32 + r + 1];
      w0[r2] = fp16::Pair<XT>::lut_lo(l0, xr[r], l1, xr[r + 1]);
      w1[r2] = fp16::Pair<XT>::lut_hi(l0, xr[r], l1, xr[r + 1]);
    }
    uint8_t* r0 = s_x + p0 * kXS + jb * 64;
    uint8_t* r1 = r0 + kXS;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      *reinterpret_cast<uint4*>(r0 + 16 * q) =
          make_uint4(w0[4 * q], w0[4 * q + 1], w0[4 * q + 2], w0[4 * q + 3]);
      *reinterpret_cast<uint4*>(r1 + 16 * q) =
          make_uint4(w1[4 * q], w1[4 * q + 1], w1[4 * q + 2], w1[4 * q + 3]);
    }
  }
  __syncthreads();

  // ---- S^T = B^T X~ (rows n, columns p): wave -> n-tile wv and both p-tiles, so that each B^T
  //      fragment (64 KB per chunk, from L2) is loaded by one wave.  The result leaves every
  //      lane with the fp32 elements of its fragment slices, so S goes to memory straight from
  //      the accumulators.
  const int half = lane >> 5;
  v16f acc0 = {}, acc1 = {};
  {
    const uint8_t* arow = s_x + (lane & 31) * kXS + 16 * half;
    const _Float16* bf = bT_frag + (((size_t)b * nc + c) * G + g) * (size_t)kN * kQ +
                         (size_t)wv * (kQ / 16) * 512 + lane * 8;
#pragma unroll
    for (int ks = 0; ks < kQ / 16; ++ks) {
      const h8 b0 = *reinterpret_cast<const h8*>(bf + ks * 512);
      const h8 a0 = *reinterpret_cast<const h8*>(arow + ks * 32);
      const h8 a1 = *reinterpret_cast<const h8*>(arow + 32 * kXS + ks * 32);
      acc0 = __builtin_amdgcn_mfma_f32_32x32x16_f16(b0, a0, acc0, 0, 0, 0);
      acc1 = __builtin_amdgcn_mfma_f32_32x32x16_f16(b0, a1, acc1, 0, 0, 0);
    }
  }
  // run q (four rows n) of every lane of a tile is one 1 KB plane
  float* dst = S + (((size_t)b * nc + c) * H + h) * (size_t)kP * kN + (size_t)wv * 1024 + lane * 4;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    *reinterpret_cast<float4*>(dst + 256 * q) =
        make_float4(acc0[4 * q], acc0[4 * q + 1], acc0[4 * q + 2], acc0[4 * q + 3]);
    *reinterpret_cast<float4*>(dst + (kN / 32) * 1024 + 256 * q) =
        make_float4(acc1[4 * q], acc1[4 * q + 1], acc1[4 * q + 2], acc1[4 * q + 3]);
  }
}

// P_in[c+1] = fl32(d[c] P_in[c] + S[c]) over [b, c, h, P*N] fp32 in fragment order, kE elements
// per thread, kDepth chunks of loads in flight.  The running state stays fp32 in registers; what
// is written is ChunkScan1's operand, fp16(P_in[c]) (6 instead of 8 bytes per element of HBM
// traffic, which bounds it: 54 -> 41 us on the 2.7B-shaped layer).
template <int kV>   // float4 per thread
__global__ __launch_bounds__(256) void fp16_pass_kernel(
    const float* __restrict__ S, const float* __restrict__ dec, const float* __restrict__ init,
    _Float16* __restrict__ pin, float* __restrict__ final_state, int nc, int H,
    int64_t nthreads) {
  constexpr int kDepth = 8;
  constexpr int kE = 4 * kV;
  constexpr int64_t kSlab = (int64_t)kP * kN;
  const int64_t gt = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (gt >= nthreads) return;
  const int64_t e = gt * kE;
  const int64_t bh = e / kSlab;
  const int slot = (int)(e - bh * kSlab) / kE;   // lane slices (kV = 2) or their halves (kV = 1)
  const int64_t b = bh / H, h = bh - b * H;
  // plane order of S: 256 floats per run of four k, 4 per lane; pin: 8 elements per lane slice
  const int lane = slot & 63;
  const int plane = (slot >> 6) * kV;
  const int soff = plane * 256 + lane * 4;
  const int off = (plane >> 1) * 512 + lane * 8 + 4 * (plane & 1);
  int row, k;
  frag::pk16_coords((size_t)off, kN, &row, &k);
  // row-major offset of the same elements: runs of four, 8 apart
  const int64_t roff = (int64_t)row * kN + k;
  float st[kE];
#pragma unroll
  for (int i = 0; i < kE; ++i) st[i] = 0.0f;
  if (init) {
#pragma unroll
    for (int i = 0; i < kV; ++i) {
      const float4 f = *reinterpret_cast<const float4*>(init + bh * kSlab + roff + 8 * i);
      st[4 * i] = f.x; st[4 * i + 1] = f.y; st[4 * i + 2] = f.z; st[4 * i + 3] = f.w;
    }
  }
  const size_t cstride = (size_t)H * kSlab;
  const size_t base = ((size_t)b * nc * H + h) * kSlab;
  const float* drow = dec + bh * nc;
  for (int c0 = 0; c0 < nc; c0 += kDepth) {
    float4 v[kDepth][kV];
    float d[kDepth];
#pragma unroll
    for (int q = 0; q < kDepth; ++q) {
      if (c0 + q < nc) {
#pragma unroll
        for (int i = 0; i < kV; ++i)
          v[q][i] = *reinterpret_cast<const float4*>(S + base + soff + 256 * i +
                                                     (size_t)(c0 + q) * cstride);
        d[q] = drow[c0 + q];
      }
    }
#pragma unroll
    for (int q = 0; q < kDepth; ++q) {
      if (c0 + q < nc) {
        uint32_t o[2 * kV];
#pragma unroll
        for (int i = 0; i < 2 * kV; ++i) o[i] = fp16::pack_h2(st[2 * i], st[2 * i + 1]);
        _Float16* dst = pin + base + off + (size_t)(c0 + q) * cstride;
        if constexpr (kV == 2)
          *reinterpret_cast<uint4*>(dst) = make_uint4(o[0], o[1], o[2], o[3]);
        else
          *reinterpret_cast<uint2*>(dst) = make_uint2(o[0], o[1]);
#pragma unroll
        for (int i = 0; i < kV; ++i) {
          st[4 * i] = __builtin_fmaf(d[q], st[4 * i], v[q][i].x);
          st[4 * i + 1] = __builtin_fmaf(d[q], st[4 * i + 1], v[q][i].y);
          st[4 * i + 2] = __builtin_fmaf(d[q], st[4 * i + 2], v[q][i].z);
          st[4 * i + 3] = __builtin_fmaf(d[q], st[4 * i + 3], v[q][i].w);
        }
      }
    }
  }
  if (final_state) {
#pragma unroll
    for (int i = 0; i < kV; ++i)
      *reinterpret_cast<float4*>(final_state + bh * kSlab + roff + 8 * i) =
          make_float4(st[4 * i], st[4 * i + 1], st[4 * i + 2], st[4 * i + 3]);
  }
}

}  // namespace

hipError_t launch_fp16_state(const LayerDims& d, const void* x, int x_dtype, const float* dt,
                             int dt_softplus, const float* A, const _Float16* bT_frag, float* S,
                             float* dec, hipStream_t st) {
  const int64_t nwork = (int64_t)d.batch * d.nchunks * d.nheads;
  if (nwork == 0) return hipSuccess;
  if (x_dtype == 1)
    hipLaunchKernelGGL(fp16_state_kernel<_Float16>, dim3((unsigned)nwork), dim3(256), 0, st,
                       static_cast<const _Float16*>(x), dt, A, bT_frag, dt_softplus, S, dec,
                       d.seqlen, d.nheads, d.ngroups, d.nchunks);
  else
    hipLaunchKernelGGL(fp16_state_kernel<float>, dim3((unsigned)nwork), dim3(256), 0, st,
                       static_cast<const float*>(x), dt, A, bT_frag, dt_softplus, S, dec,
                       d.seqlen, d.nheads, d.ngroups, d.nchunks);
  return hipGetLastError();
}

hipError_t launch_fp16_pass(const LayerDims& d, const float* S, const float* dec,
                            const float* init, _Float16* pin, float* final_state,
                            hipStream_t st) {
  const int64_t elems = (int64_t)d.batch * d.nheads * kP * kN;
  if (elems == 0) return hipSuccess;
  // 8 elements per thread (one 16-byte store each) while that leaves two waves per SIMD
  const bool wide = elems / 8 >= 131072;
  const int64_t nthreads = elems / (wide ? 8 : 4);
  const dim3 grid((unsigned)((nthreads + 255) / 256)), block(256);
  if (wide)
    hipLaunchKernelGGL(fp16_pass_kernel<2>, grid, block, 0, st, S, dec, init, pin, final_state,
                       d.nchunks, d.nheads, nthreads);
  else
    hipLaunchKernelGGL(fp16_pass_kernel<1>, grid, block, 0, st, S, dec, init, pin, final_state,
                       d.nchunks, d.nheads, nthreads);
  return hipGetLastError();
}

}  // namespace ssdi8
