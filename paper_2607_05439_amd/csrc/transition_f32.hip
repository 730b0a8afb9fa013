// Pair transition in fp32 (Appendix "Manual SwiGLU decomposition"):
//   N = LayerNorm(z),  z <- z + W3 (SiLU(W1 N) * W2 N),
// on the fp32 matrix cores, or on the vector units for the shapes and
// alignments their 16-byte operand loads do not take.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "cdna4.h"
#include "dcp_internal.h"

namespace dcp {
namespace {

// v_mfma_f32_16x16x4_f32: A holds row n, B column n, both at k-slot g; the
// accumulator holds rows 4g..4g+3 of column n. Products and sums are fp32.
__device__ __forceinline__ f32x4 mfma4(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// The transition of P tiles of 16 pairs per workgroup in fp32 on the matrix
// cores (c_z <= 16 CT, a multiple of 4; hidden a multiple of 16; 16-byte
// aligned weights). Channel 16j + 4g + i of pair n sits in lane (n, g), register
// (j, i): what one 16-byte load of z brings. As the k-slot numbering is free,
// that is the B operand of step (j, i) of N W1^T, with the 16-byte load of row
// n of W1 as its A operand; the hidden units come out as rows 4g + i of column
// n, which is in turn the B operand of the product with W3; and its accumulator
// has z's own layout again, so LayerNorm, SiLU and the residual are lane-local.
// The four waves share the pairs and take every fourth tile of 16 hidden units,
// each streaming its own weight tiles from L2 one tile ahead; their partial sums
// meet in LDS and are added in wave order. Splitting the hidden units rather
// than the pairs keeps four waves busy on each 16 pairs. What bounds it: 36864
// pairs of 128 channels take 165 us with two tiles per workgroup and 233 with
// one, where the products alone need 95 at the rate of a large fp32 matrix
// product; without the weight loads in the loop (a timing probe) 149 and 134. So
// one tile is limited by the latency of the weights, two by the uneven last round
// of workgroups (1152 of them, two per CU, are 2.25 rounds). gamma and beta are
// read once for both tiles: a tile at a time they and the addresses did not fit
// the registers (24 spilled, 185 us).
template <int CT, int P>
__global__ void __launch_bounds__(256, CT > 8 ? 1 : 2) trans_f32_kernel(TransGenArgs a) {
  __shared__ f32x4 red[4][P][CT][64];
  const int lane = threadIdx.x & 63, n = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t pair0 = (int64_t)blockIdx.x * (16 * P);
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
  auto chunk = [](const float* p) { return *reinterpret_cast<const f32x4*>(p); };
  // Channels past c_z (c_z < 16 CT): z is 0 there, and loads repeat the row's
  // last chunk, so no load is conditional (a branch around one would make the
  // compiler wait for those in flight)
  auto inside = [&](int j) { return 16 * j + 4 * g < a.c_z; };
  int ch[CT];
#pragma unroll
  for (int j = 0; j < CT; ++j) ch[j] = min(16 * j + 4 * g, a.c_z - 4);

  f32x4 nz[P][CT];
#pragma unroll
  for (int p = 0; p < P; ++p) {
    const int64_t pr = min(pair0 + 16 * p + n, a.n_pairs - 1);
    const float* z = a.z_in + pr * a.c_z;
#pragma unroll
    for (int j = 0; j < CT; ++j) nz[p][j] = chunk(z + ch[j]);
  }
  float rstd[P];
#pragma unroll
  for (int p = 0; p < P; ++p) {
    float s = 0.0f, v = 0.0f;
#pragma unroll
    for (int j = 0; j < CT; ++j)
#pragma unroll
      for (int i = 0; i < 4; ++i) s += inside(j) ? nz[p][j][i] : 0.0f;
    const float mu = sum4(s) / (float)a.c_z;
#pragma unroll
    for (int j = 0; j < CT; ++j)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        nz[p][j][i] = inside(j) ? nz[p][j][i] - mu : 0.0f;
        v = fmaf(nz[p][j][i], nz[p][j][i], v);
      }
    rstd[p] = 1.0f / sqrtf(sum4(v) / (float)a.c_z + a.eps);
  }
#pragma unroll
  for (int j = 0; j < CT; ++j) {
    const f32x4 ga = a.gamma ? chunk(a.gamma + ch[j]) : f32x4{1.f, 1.f, 1.f, 1.f};
    const f32x4 be = a.beta ? chunk(a.beta + ch[j]) : zero;
#pragma unroll
    for (int p = 0; p < P; ++p)
#pragma unroll
      for (int i = 0; i < 4; ++i) nz[p][j][i] = inside(j) ? ga[i] * (nz[p][j][i] * rstd[p]) + be[i] : 0.0f;
  }

  f32x4 out[P][CT];
#pragma unroll
  for (int p = 0; p < P; ++p)
#pragma unroll
    for (int j = 0; j < CT; ++j) out[p][j] = zero;
  const int n_ht = a.hidden / 16;
  // Weight tiles arrive in two halves of CT / 2 chunks, each requested half a
  // product phase before its use: at most two phases' worth is in flight, which
  // is what the registers hold at two waves per SIMD.
  constexpr int kHalf = CT / 2;
  f32x4 w1[CT], w2[CT], w3[CT];
  // Channels past c_z of W1 and W2 are read out of range, zeros: z is 0 there, and 0
  // times the row's last chunk would make a NaN of an infinite weight.
  const __amdgpu_buffer_rsrc_t res1 =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(a.w1), 0, a.hidden * a.c_z * 4, kRawBufferFlags);
  const __amdgpu_buffer_rsrc_t res2 =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(a.w2), 0, a.hidden * a.c_z * 4, kRawBufferFlags);
  auto load12 = [&](int ht, int j0) {
    const int row = 16 * ht * a.c_z * 4;
#pragma unroll
    for (int j = j0; j < j0 + kHalf; ++j) {
      const int off = inside(j) ? (n * a.c_z + 16 * j + 4 * g) * 4 : kOutOfRange;
      w1[j] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(res1, off, row, 0));
      w2[j] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(res2, off, row, 0));
    }
  };
  auto load3 = [&](int ht, int j0) {
#pragma unroll
    for (int j = j0; j < j0 + kHalf; ++j)
      w3[j] = chunk(a.w3 + (int64_t)min(16 * j + n, a.c_z - 1) * a.hidden + 16 * ht + 4 * g);
  };
  f32x4 x[P], y[P];
  auto products12 = [&](int j0) {
#pragma unroll
    for (int j = j0; j < j0 + kHalf; ++j)
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int p = 0; p < P; ++p) {
          x[p] = mfma4(w1[j][i], nz[p][j][i], x[p]);
          y[p] = mfma4(w2[j][i], nz[p][j][i], y[p]);
        }
    __builtin_amdgcn_sched_barrier(0);
  };
  auto products3 = [&](int j0) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = j0; j < j0 + kHalf; ++j)
#pragma unroll
        for (int p = 0; p < P; ++p) out[p][j] = mfma4(w3[j][i], x[p][i], out[p][j]);
    __builtin_amdgcn_sched_barrier(0);
  };
  if (wave < n_ht) {
    load12(wave, 0);
    load12(wave, kHalf);
  }
  for (int ht = wave; ht < n_ht; ht += 4) {
    const int next = min(ht + 4, n_ht - 1);
#pragma unroll
    for (int p = 0; p < P; ++p) x[p] = y[p] = zero;
    products12(0);
    load3(ht, 0);
    products12(kHalf);
    load3(ht, kHalf);
    load12(next, 0);
#pragma unroll
    for (int p = 0; p < P; ++p)
#pragma unroll
      for (int i = 0; i < 4; ++i) x[p][i] = x[p][i] / (1.0f + expf(-x[p][i])) * y[p][i];
    products3(0);
    load12(next, kHalf);
    products3(kHalf);
  }
#pragma unroll
  for (int p = 0; p < P; ++p)
#pragma unroll
    for (int j = 0; j < CT; ++j) red[wave][p][j][lane] = out[p][j];
  __syncthreads();
  for (int t = wave; t < P * CT; t += 4) {
    const int p = t / CT, j = t % CT;
    const int64_t pr = pair0 + 16 * p + n;
    if (pr >= a.n_pairs || 16 * j + 4 * g >= a.c_z) continue;
    const f32x4 sum = ((red[0][p][j][lane] + red[1][p][j][lane]) + red[2][p][j][lane]) + red[3][p][j][lane];
    const int64_t e = pr * a.c_z + 16 * j + 4 * g;
    *reinterpret_cast<f32x4*>(a.z_out + e) = chunk(a.z_in + e) + sum;
  }
}

// Two tiles of 16 pairs per workgroup halve the weight traffic (and the stalls
// on it) but also the workgroups: while one tile per workgroup leaves a CU no
// second workgroup, one is faster (4096 pairs of 128 channels: 28.4 us against
// 34.0; 64 channels 9.2 against 12.0), and two beyond (4097 pairs: 33.7 against
// 49.8, 9000 71.5 against 78.5; 64 channels 12.1 against 15.1; 100 channels lose
// 1 % between 9000 and 12288).
constexpr int64_t kTransF32SmallPairs = 256 * 16;

template <int CT, int P>
hipError_t launch_trans_f32(const TransGenArgs& a, hipStream_t st) {
  hipLaunchKernelGGL((trans_f32_kernel<CT, P>), dim3((unsigned)((a.n_pairs + 16 * P - 1) / (16 * P))), dim3(256), 0,
                     st, a);
  return hipGetLastError();
}

// One wave per pair: LayerNorm, then 8+ hidden units per lane, h in LDS, then
// the output channels per lane; fp32 throughout.
__global__ void __launch_bounds__(256) trans_gen_kernel(TransGenArgs a) {
  __shared__ float s_n[4][kGenMaxCz];
  __shared__ float s_h[4][kTransGenMaxHidden];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t p = (int64_t)blockIdx.x * 4 + wave;
  if (p >= a.n_pairs) return;
  const float* z = a.z_in + p * a.c_z;
  float s = 0.0f;
  for (int c = lane; c < a.c_z; c += 64) s += z[c];
  for (int m = 32; m > 0; m >>= 1) s += __shfl_xor(s, m);
  const float mu = s / (float)a.c_z;
  float v = 0.0f;
  for (int c = lane; c < a.c_z; c += 64) v = fmaf(z[c] - mu, z[c] - mu, v);
  for (int m = 32; m > 0; m >>= 1) v += __shfl_xor(v, m);
  const float rstd = 1.0f / sqrtf(v / (float)a.c_z + a.eps);
  float* nn = s_n[wave];
  for (int c = lane; c < a.c_z; c += 64)
    nn[c] = (a.gamma ? a.gamma[c] : 1.0f) * ((z[c] - mu) * rstd) + (a.beta ? a.beta[c] : 0.0f);
  __builtin_amdgcn_wave_barrier();
  float* hh = s_h[wave];
  for (int u = lane; u < a.hidden; u += 64) {
    float x = 0.0f, y = 0.0f;
    for (int c = 0; c < a.c_z; ++c) {
      x = fmaf(a.w1[(int64_t)u * a.c_z + c], nn[c], x);
      y = fmaf(a.w2[(int64_t)u * a.c_z + c], nn[c], y);
    }
    hh[u] = x / (1.0f + expf(-x)) * y;
  }
  __builtin_amdgcn_wave_barrier();
  for (int c = lane; c < a.c_z; c += 64) {
    float t = 0.0f;
    for (int u = 0; u < a.hidden; ++u) t = fmaf(a.w3[(int64_t)c * a.hidden + u], hh[u], t);
    a.z_out[p * a.c_z + c] = z[c] + t;
  }
}

}  // namespace

hipError_t launch_transition_gen(const TransGenArgs& a, hipStream_t st) {
  // The matrix-core kernel wherever its 16-byte loads fit; the vector kernel
  // takes any other width or alignment (192 x 192 pairs of 128 channels: 3450 us
  // on the vector units, 165 us here).
  const auto at16 = [](const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; };
  if (a.c_z % 4 == 0 && a.hidden % 16 == 0 && at16(a.w1) && at16(a.w2) && at16(a.w3) && at16(a.gamma) && at16(a.beta)) {
    if (a.c_z > 128) return launch_trans_f32<16, 1>(a, st);
    if (a.n_pairs <= kTransF32SmallPairs)
      return a.c_z > 64 ? launch_trans_f32<8, 1>(a, st)
             : a.c_z > 32 ? launch_trans_f32<4, 1>(a, st)
                          : launch_trans_f32<2, 1>(a, st);
    return a.c_z > 64 ? launch_trans_f32<8, 2>(a, st)
           : a.c_z > 32 ? launch_trans_f32<4, 2>(a, st)
                        : launch_trans_f32<2, 2>(a, st);
  }
  hipLaunchKernelGGL(trans_gen_kernel, dim3((unsigned)((a.n_pairs + 3) / 4)), dim3(256), 0, st, a);
  return hipGetLastError();
}

}  // namespace dcp
