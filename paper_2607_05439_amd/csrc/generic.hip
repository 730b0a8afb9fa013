// General fp32 path: any c_z <= 256, H <= 16, d <= 64, H*d <= 128, with s and
// z in fp32 or bf16, for the shapes the fused bf16 kernels do not cover. fp32
// arithmetic throughout (two-pass LayerNorm, expf); the projections and the pair
// bias run on the fp32 matrix cores. Partial states use natural-log units.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "cdna4.h"
#include "dcp_internal.h"

namespace dcp {
namespace {

__device__ __forceinline__ float load_act(const void* p, int bf16, int64_t idx) {
  if (bf16) return __uint_as_float((uint32_t)static_cast<const uint16_t*>(p)[idx] << 16);
  return static_cast<const float*>(p)[idx];
}

// v_mfma_f32_16x16x4_f32: A holds row n, B column n (n = lane % 16), both at
// k-slot g = lane / 16; the accumulator holds rows 4g..4g+3 of column n.
__device__ __forceinline__ f32x4 mfma4(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// Four consecutive elements at p + i0 as loaded (fp32: 16 bytes, bf16: 8), or
// one by one, indices past the last repeating it, where the row length is not a
// multiple of four. Kept apart from the conversion so that loads can be
// issued ahead of their use.
__device__ __forceinline__ u32x4 load_raw4(const void* p, int bf16, int vec, int64_t base, int i0, int len) {
  u32x4 r;
  if (vec) {
    if (bf16) {
      const u32x2 t = *reinterpret_cast<const u32x2*>(static_cast<const uint16_t*>(p) + base + i0);
      r[0] = t[0], r[1] = t[1], r[2] = 0u, r[3] = 0u;
    } else {
      r = *reinterpret_cast<const u32x4*>(static_cast<const float*>(p) + base + i0);
    }
  } else {
    uint32_t e[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int64_t x = base + min(i0 + i, len - 1);
      e[i] = bf16 ? (uint32_t)static_cast<const uint16_t*>(p)[x] : static_cast<const uint32_t*>(p)[x];
    }
    if (bf16)
      r[0] = e[0] | (e[1] << 16), r[1] = e[2] | (e[3] << 16), r[2] = 0u, r[3] = 0u;
    else
      r[0] = e[0], r[1] = e[1], r[2] = e[2], r[3] = e[3];
  }
  return r;
}
__device__ __forceinline__ f32x4 raw4_to_f32(const u32x4& r, int bf16) {
  f32x4 v;
  if (bf16) {
    v[0] = __uint_as_float(r[0] << 16), v[1] = __uint_as_float(r[0] & 0xFFFF0000u);
    v[2] = __uint_as_float(r[1] << 16), v[3] = __uint_as_float(r[1] & 0xFFFF0000u);
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = __uint_as_float(r[i]);
  }
  return v;
}

// k and v for the tiled attention: per 16 keys [heads by fours][4-channel
// piece][head of the four][key][4], so that lane (n, g)'s piece c of head g lies
// 16 bytes after its neighbour's: the memory path takes four consecutive lanes'
// 64 bytes at a time, and pieces in any other order (row-major, or key before
// head) cost it a lookup per lane. The last keys and heads are packed without
// padding: n_tok * H * d floats in all. Offset of piece 0 of head h of a key, and
// the step from piece to piece. (The tiled attention runs where both fit 31-bit
// byte offsets.)
__device__ __forceinline__ int kv_tile_offset(int key, int n_tok, int h, int H, int d, int* step) {
  const int t = key >> 4, keys = min(16, n_tok - 16 * t), heads = min(4, H - (h & ~3));
  *step = 4 * keys * heads;
  return t * 16 * H * d + (h & ~3) * d * keys + ((h & 3) * keys + (key & 15)) * 4;
}

// The four projections on the fp32 matrix cores: each wave forms T x T tiles of
// 16 outputs (rows of W, the A operand) by 16 tokens (the B operand); channel
// 16j + 4g + i is k-slot g of step (j, i), so both operands are plain 16-byte
// loads of a row, eight of each in flight. Blocks: 4 waves of consecutive output
// tiles over the same tokens; the side (k and v over all tokens, q and g over
// the query rows) comes from the block index. With one thread per output,
// reading its row of W alone, 128 tokens took 20 us.
template <int T>
__global__ void __launch_bounds__(256) gen_proj_kernel(GenProjArgs a) {
  const int lane = threadIdx.x & 63, n = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n_ot = (a.hd + 16 * T - 1) / (16 * T);  // output tiles of one projection
  const int ot = (int)(blockIdx.y * 4 + wave);       // tiles of the side's two projections
  if (ot >= 2 * n_ot) return;
  const int64_t kv_tiles = (a.n_tok + 16 * T - 1) / (16 * T);
  const bool q_side = blockIdx.x >= kv_tiles;
  const int64_t row0 = ((int64_t)blockIdx.x - (q_side ? kv_tiles : 0)) * (16 * T);
  const int64_t rows = q_side ? a.n_q : a.n_tok;
  const bool second = ot >= n_ot;
  const int o0 = (second ? ot - n_ot : ot) * (16 * T);
  const float* w = q_side ? (second ? a.w_g : a.w_q) : (second ? a.w_v : a.w_k);
  float* dst = q_side ? (second ? a.g : a.q) : (second ? a.v : a.k);
  if (!dst) return;
  const bool w_vec = a.s_vec && (reinterpret_cast<uintptr_t>(w) & 15) == 0;
  int64_t s_base[T], w_base[T];
#pragma unroll
  for (int t = 0; t < T; ++t) {
    s_base[t] = ((q_side ? a.q_row0 : 0) + min(row0 + 16 * t + n, rows - 1)) * a.c_s;
    w_base[t] = (int64_t)min(o0 + 16 * t + n, a.hd - 1) * a.c_s;
  }
  f32x4 acc[T][T];
#pragma unroll
  for (int x = 0; x < T; ++x)
#pragma unroll
    for (int y = 0; y < T; ++y) acc[x][y] = f32x4{0.f, 0.f, 0.f, 0.f};
  constexpr int kC = 8 / T;  // chunks of 16 channels per step
  for (int c0 = 0; c0 < a.c_s; c0 += 16 * kC) {
    u32x4 sr[T][kC], wr[T][kC];
#pragma unroll
    for (int j = 0; j < kC; ++j) {
      const int ch = c0 + 16 * j + 4 * g;
      const int at = a.s_vec ? min(ch, a.c_s - 4) : ch;  // past the row: any element of it, times 0
#pragma unroll
      for (int t = 0; t < T; ++t) {
        sr[t][j] = load_raw4(a.s, a.s_bf16, a.s_vec, s_base[t], at, a.c_s);
        wr[t][j] = load_raw4(w, 0, w_vec, w_base[t], at, a.c_s);
      }
    }
#pragma unroll
    for (int j = 0; j < kC; ++j) {
      f32x4 sv[T], wv[T];
#pragma unroll
      for (int t = 0; t < T; ++t) {
        sv[t] = raw4_to_f32(sr[t][j], a.s_bf16);
        wv[t] = raw4_to_f32(wr[t][j], 0);
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const bool in = c0 + 16 * j + 4 * g + i < a.c_s;
#pragma unroll
        for (int t = 0; t < T; ++t) {
          sv[t][i] = in ? sv[t][i] : 0.0f;
          wv[t][i] = in ? wv[t][i] : 0.0f;
        }
#pragma unroll
        for (int x = 0; x < T; ++x)
#pragma unroll
          for (int y = 0; y < T; ++y) acc[x][y] = mfma4(wv[x][i], sv[y][i], acc[x][y]);
      }
    }
  }
#pragma unroll
  for (int y = 0; y < T; ++y) {
    const int64_t row = row0 + 16 * y + n;
    if (row >= rows) continue;
#pragma unroll
    for (int x = 0; x < T; ++x) {
      const int o = o0 + 16 * x + 4 * g;
      f32x4 v = acc[x][y];
      if (q_side && second)
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = 1.0f / (1.0f + expf(-v[i]));
      // a masked key's v: 0, as its weight is (0 times a NaN would be one)
      if (!q_side && second && a.mask && a.mask[row] == 0) v = f32x4{0.f, 0.f, 0.f, 0.f};
      if (a.kv_head_dim && !q_side) {
        if (o < a.hd) {
          const int h = o / a.kv_head_dim, c = (o - h * a.kv_head_dim) >> 2;
          int step;
          const int at = kv_tile_offset((int)row, (int)a.n_tok, h, a.hd / a.kv_head_dim, a.kv_head_dim, &step);
          *reinterpret_cast<f32x4*>(dst + at + c * step) = v;
        }
      } else if (a.hd % 4 == 0) {
        if (o < a.hd) *reinterpret_cast<f32x4*>(dst + row * a.hd + o) = v;
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (o + i < a.hd) dst[row * a.hd + o + i] = v[i];
      }
    }
  }
}

// LayerNorm statistics of one pair in fp32, two passes.
__device__ __forceinline__ void ln_stats(const void* z, int bf16, int64_t off, int c_z, float eps, float& mu,
                                         float& rstd) {
  float s = 0.0f;
  for (int c = 0; c < c_z; ++c) s += load_act(z, bf16, off + c);
  mu = s / (float)c_z;
  float v = 0.0f;
  for (int c = 0; c < c_z; ++c) {
    const float t = load_act(z, bf16, off + c) - mu;
    v = fmaf(t, t, v);
  }
  rstd = 1.0f / sqrtf(v / (float)c_z + eps);
}

// The shapes the tiled kernel below does not take: grid (n_q rows, n_parts
// parts), one wave. Each lane owns keys start+lane,
// start+lane+64, ... with its own online-softmax state in LDS; the 64 states
// are then merged in lane order.
__global__ void __launch_bounds__(64) gen_attn_any_kernel(GenAttnArgs a) {
  __shared__ float wg[kGenMaxH * kGenMaxCz];  // W_b * gamma
  __shared__ float st_m[64][kGenMaxH];
  __shared__ float st_l[64][kGenMaxH];
  __shared__ float st_acc[64][kGenMaxHD];
  const int lane = threadIdx.x;
  const int64_t row = blockIdx.x;
  const int part = blockIdx.y;
  const int H = a.n_heads, d = a.head_dim, hd = H * d, c_z = a.c_z;
  for (int x = lane; x < H * c_z; x += 64) wg[x] = a.w_b[x] * (a.gamma ? a.gamma[x % c_z] : 1.0f);
  for (int h = 0; h < H; ++h) {
    st_m[lane][h] = -INFINITY;
    st_l[lane][h] = 0.0f;
  }
  for (int x = 0; x < hd; ++x) st_acc[lane][x] = 0.0f;
  __syncthreads();

  int64_t size, start;
  chunk_of(a.k_len, a.n_parts, part, &size, &start);
  start += a.k_lo;
  const float scale = 1.0f / sqrtf((float)d);
  const float* qr = a.q + row * hd;
  for (int64_t j = start + lane; j < start + size; j += 64) {
    if (a.mask && a.mask[j] == 0) continue;
    const int64_t off = (row * a.n_tok + j) * c_z;
    float mu, rstd;
    ln_stats(a.z, a.z_bf16, off, c_z, a.eps, mu, rstd);
    for (int h = 0; h < H; ++h) {
      float b = 0.0f;
      for (int c = 0; c < c_z; ++c) b = fmaf(wg[h * c_z + c], (load_act(a.z, a.z_bf16, off + c) - mu) * rstd, b);
      float dot = 0.0f;
      for (int e = 0; e < d; ++e) dot = fmaf(qr[h * d + e], a.k[j * hd + h * d + e], dot);
      const float lg = dot * scale + b;
      const float mo = st_m[lane][h];
      const float mn = fmaxf(mo, lg);
      const float al = expf(mo - mn);  // 0 when mo = -inf
      const float p = expf(lg - mn);
      st_l[lane][h] = st_l[lane][h] * al + p;
      for (int e = 0; e < d; ++e)
        st_acc[lane][h * d + e] = fmaf(p, a.v[j * hd + h * d + e], st_acc[lane][h * d + e] * al);
      st_m[lane][h] = mn;
    }
  }
  __syncthreads();
  for (int x = lane; x < hd; x += 64) {
    const int h = x / d;
    float mx = -INFINITY;
    for (int t = 0; t < 64; ++t) mx = fmaxf(mx, st_m[t][h]);
    float l = 0.0f, acc = 0.0f;
    for (int t = 0; t < 64; ++t) {
      if (st_m[t][h] == -INFINITY && st_l[t][h] == 0.0f) continue;
      const float sc = expf(st_m[t][h] - mx);
      l = fmaf(sc, st_l[t][h], l);
      acc = fmaf(sc, st_acc[t][x], acc);
    }
    a.acc_parts[((int64_t)part * a.n_q + row) * hd + x] = acc;
    if (x % d == 0) {
      a.m_parts[((int64_t)part * H + h) * a.n_q + row] = mx;
      a.l_parts[((int64_t)part * H + h) * a.n_q + row] = l;
    }
  }
}

// Four consecutive elements of z as loaded (byte offset off), and as fp32.
template <bool BF16>
struct RawZ;
template <>
struct RawZ<false> {
  typedef u32x4 type;
  static __device__ __forceinline__ type load(__amdgpu_buffer_rsrc_t r, int off, int soff) {
    return __builtin_amdgcn_raw_buffer_load_b128(r, off, soff, 0);
  }
  static __device__ __forceinline__ f32x4 to_f32(const type& r) { return __builtin_bit_cast(f32x4, r); }
};
template <>
struct RawZ<true> {
  typedef u32x2 type;
  static __device__ __forceinline__ type load(__amdgpu_buffer_rsrc_t r, int off, int soff) {
    return __builtin_amdgcn_raw_buffer_load_b64(r, off, soff, 0);
  }
  static __device__ __forceinline__ f32x4 to_f32(const type& r) {
    return f32x4{__uint_as_float(r[0] << 16), __uint_as_float(r[0] & 0xFFFF0000u), __uint_as_float(r[1] << 16),
                 __uint_as_float(r[1] & 0xFFFF0000u)};
  }
};

constexpr int kGenWaves = 4;  // 8 were slower: 79 against 61 us (601 tokens, 128 channels, no mask), 66 against 54 (900, 32)

// grid (rows / R, parts), 4 waves that share R query rows and take every fourth
// tile of 16 keys of the part. Lane (n, g) holds key n of the tile.
//  - z: the tile's 16 pair vectors are consecutive in memory; the lane loads
//    channels 16j + 4g .. +3 of its key (one tile ahead) and the four lanes of a
//    key form its two-pass LayerNorm statistics.
//  - bias on the fp32 matrix cores: A = W_b gamma with head 4 (n % 4) + n / 4 in
//    row n, B = z - mean as loaded; accumulator register i of lane (n, g) is then
//    head 4i + g of key n, so each lane owns NH = ceil(H / 4) heads of one key,
//  - and the logits, an online softmax of the lane's own keys and the weighted
//    sum of v run in the lane, with k and v read straight from L2 (laid out for
//    it by the projection) and no exchange between lanes until the row's end.
// The 16 lanes' and 4 waves' states meet in LDS, in a fixed order.
// DP: the head size padded to a multiple of 4; c_z <= 16 CT.
// What bounds it: the memory path's lookups. 601 tokens of 128 channels (183 MB of
// z) take 62 us here and 77 a call with masked keys, the same rows at the rate of a
// large read 27; timing probes without the bias products, or with z or k and v always
// from the same addresses, gained 1 to 5 us each, but k and v in an order that
// puts four lanes' pieces on one line gained 8, and a z load's four
// consecutive lanes still lie in four rows. With k and v row-major a call took 106;
// with a lane per key, its state in LDS and z read three times in 4-byte pieces,
// 1810.
template <int NH, int DP, int CT, bool BF16, int R>
__global__ void __launch_bounds__(64 * kGenWaves, 2) gen_attn_kernel(GenAttnArgs a) {
  constexpr int kHd = 4 * NH * DP;  // padded channels of all lanes' heads
  constexpr int kQs = DP + 4;       // q row stride: the four heads read at once fall in different banks
  __shared__ __align__(16) float s_q[R][4 * NH * kQs];
  __shared__ __align__(16) float s_w[16 * 16 * CT];  // [j][lane][4]: A operands
  __shared__ __align__(16) float s_o[kGenWaves][16][kHd];
  __shared__ float s_l[kGenWaves][16][4 * NH];
  __shared__ float s_m[kGenWaves][4 * NH];
  const int tid = threadIdx.x, lane = tid & 63, n = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t row0 = (int64_t)blockIdx.x * R;
  const int part = blockIdx.y;
  const int H = a.n_heads, d = a.head_dim, hd = H * d, c_z = a.c_z;
  int64_t size, first;
  chunk_of(a.k_len, a.n_parts, part, &size, &first);
  const int start = (int)(a.k_lo + first), end = start + (int)size;
  const int n_tiles = ((int)size + 15) / 16;

  // Chunks past c_z or d repeat the last one: no load is conditional. fm is 0
  // there (and so are the weights and q), else 1.
  typedef typename RawZ<BF16>::type raw_t;
  raw_t zr[CT];
  float fm[CT];
#pragma unroll
  for (int j = 0; j < CT; ++j) fm[j] = 16 * j < c_z ? 1.0f : 0.0f;
  constexpr int kEb = BF16 ? 2 : 4;
  const int row_bytes = (int)a.n_tok * c_z * kEb;
  __amdgpu_buffer_rsrc_t zres[R];
#pragma unroll
  for (int r = 0; r < R; ++r)
    zres[r] = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<char*>(static_cast<const char*>(a.z)) + min(row0 + r, a.n_q - 1) * row_bytes, 0, row_bytes,
        kRawBufferFlags);
  const __amdgpu_buffer_rsrc_t kres =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(a.k), 0, (int)a.n_tok * hd * 4, kRawBufferFlags);
  const __amdgpu_buffer_rsrc_t vres =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(a.v), 0, (int)a.n_tok * hd * 4, kRawBufferFlags);
  auto load_z = [&](int t, int r) {
    const int off = (min(start + 16 * t + n, end - 1) * c_z + 4 * g) * kEb;
#pragma unroll
    for (int j = 0; j < CT; ++j) zr[j] = RawZ<BF16>::load(zres[r], off, min(16 * j, c_z - 16) * kEb);
  };
  if (wave < n_tiles) load_z(wave, 0);

  // q and the bias weights into LDS; every load unconditional (past the end: any
  // element, times 0), so that they are in flight together
  constexpr int kQn = (R * 4 * NH * kQs + 64 * kGenWaves - 1) / (64 * kGenWaves);
  constexpr int kWn = 16 * 16 * CT / (64 * kGenWaves);
  float qv[kQn], wv[kWn], gv[kWn];
#pragma unroll
  for (int u = 0; u < kQn; ++u) {
    const int x = min(tid + 64 * kGenWaves * u, R * 4 * NH * kQs - 1), r = x / (4 * NH * kQs);
    const int h = (x - r * (4 * NH * kQs)) / kQs, e = x % kQs;
    qv[u] = a.q[min(row0 + r, a.n_q - 1) * hd + min(h, H - 1) * d + min(e, d - 1)];
    if (h >= H || e >= d) qv[u] = 0.0f;
  }
#pragma unroll
  for (int u = 0; u < kWn; ++u) {
    const int x = tid + 64 * kGenWaves * u, l = (x >> 2) & 63, c = 16 * (x >> 8) + 4 * (l >> 4) + (x & 3);
    const int h = 4 * (l & 3) + ((l & 15) >> 2);
    wv[u] = a.w_b[min(h, H - 1) * c_z + min(c, c_z - 1)];
    gv[u] = a.gamma ? a.gamma[min(c, c_z - 1)] : 1.0f;
    if (h >= H || c >= c_z) wv[u] = gv[u] = 0.0f;
  }
#pragma unroll
  for (int u = 0; u < kQn; ++u) {
    const int x = tid + 64 * kGenWaves * u;
    if (x < R * 4 * NH * kQs) (&s_q[0][0])[x] = qv[u];
  }
#pragma unroll
  for (int u = 0; u < kWn; ++u) s_w[tid + 64 * kGenWaves * u] = wv[u] * gv[u];
  __syncthreads();

  const float scale = 1.0f / sqrtf((float)d), inv_cz = 1.0f / (float)c_z;
  float m[R][NH], l[R][NH];
  f32x4 o[R][NH][DP / 4];
  int head[NH];  // the lane's heads (past the last: the last)
#pragma unroll
  for (int i = 0; i < NH; ++i) {
    head[i] = min(4 * i + g, H - 1);
#pragma unroll
    for (int r = 0; r < R; ++r) {
      m[r][i] = -INFINITY;
      l[r][i] = 0.0f;
#pragma unroll
      for (int c = 0; c < DP / 4; ++c) o[r][i][c] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
  }

  for (int t = wave; t < n_tiles; t += kGenWaves) {
    const int key = start + 16 * t + n;
    const int kk = min(key, end - 1);
    const bool valid = key < end && (!a.mask || a.mask[kk] != 0);
    // lanes past the part's end read k and v out of range, zeros: the last key's own,
    // times a weight of 0, would turn an infinite v into a NaN
    uint32_t at[NH];  // byte offset of piece 0
    int step[NH];
#pragma unroll
    for (int i = 0; i < NH; ++i) {
      const int x = kv_tile_offset(kk, (int)a.n_tok, head[i], H, d, &step[i]);
      at[i] = key < end ? 4u * (uint32_t)x : (uint32_t)kOutOfRange;
    }
    // k and v of this tile before the next tile's z: loads complete in order, so
    // waiting for v must not mean waiting for z from HBM
    f32x4 kr[NH][DP / 4], vr[NH][DP / 4];
#pragma unroll
    for (int i = 0; i < NH; ++i)
#pragma unroll
      for (int c = 0; c < DP / 4; ++c) kr[i][c] = __builtin_bit_cast(
          f32x4, __builtin_amdgcn_raw_buffer_load_b128(kres, (int)(at[i] + 4u * (uint32_t)(min(c, d / 4 - 1) * step[i])), 0, 0));
#pragma unroll
    for (int i = 0; i < NH; ++i)
#pragma unroll
      for (int c = 0; c < DP / 4; ++c)
        vr[i][c] = __builtin_bit_cast(
            f32x4,
            __builtin_amdgcn_raw_buffer_load_b128(vres, (int)(at[i] + 4u * (uint32_t)(min(c, d / 4 - 1) * step[i])), 0, 0));
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int r = 0; r < R; ++r) {
      f32x4 z[CT];
#pragma unroll
      for (int j = 0; j < CT; ++j) z[j] = RawZ<BF16>::to_f32(zr[j]);
      if (r + 1 < R)
        load_z(t, r + 1);
      else
        load_z(min(t + kGenWaves, n_tiles - 1), 0);
      f32x4 w[CT];
#pragma unroll
      for (int j = 0; j < CT; ++j) w[j] = *reinterpret_cast<const f32x4*>(&s_w[(j * 64 + lane) * 4]);
      __builtin_amdgcn_sched_barrier(0);  // (in flight during the statistics)
      // four chains each: one wave per SIMD has nothing else to fill a chain's latency with
      f32x4 s = {0.f, 0.f, 0.f, 0.f}, v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int j = 0; j < CT; ++j)
#pragma unroll
        for (int i = 0; i < 4; ++i) s[i] = fmaf(z[j][i], fm[j], s[i]);
      const float mu = sum4((s[0] + s[1]) + (s[2] + s[3])) * inv_cz;
#pragma unroll
      for (int j = 0; j < CT; ++j)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          z[j][i] = fmaf(z[j][i], fm[j], -mu * fm[j]);
          v[i] = fmaf(z[j][i], z[j][i], v[i]);
        }
      const float rstd = 1.0f / sqrtf(fmaf(sum4((v[0] + v[1]) + (v[2] + v[3])), inv_cz, a.eps));
      f32x4 b = {0.f, 0.f, 0.f, 0.f}, b1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int j = 0; j < CT; j += 2)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          b = mfma4(w[j][i], z[j][i], b);
          b1 = mfma4(w[j + 1][i], z[j + 1][i], b1);
        }
      b += b1;
#pragma unroll
      for (int i = 0; i < NH; ++i) {
        f32x4 dots = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int c = 0; c < DP / 4; ++c) {
          const f32x4 q = *reinterpret_cast<const f32x4*>(&s_q[r][(4 * i + g) * kQs + 4 * c]);
#pragma unroll
          for (int e = 0; e < 4; ++e) dots[e] = fmaf(q[e], kr[i][c][e], dots[e]);
        }
        const float dot = (dots[0] + dots[1]) + (dots[2] + dots[3]);
        const float lg = valid ? fmaf(b[i], rstd, dot * scale) : -INFINITY;
        const float mn = fmaxf(m[r][i], lg);
        const float base = mn == -INFINITY ? 0.0f : mn;
        const float al = expf(m[r][i] - base);  // 0 when m = -inf
        const float p = expf(lg - base);     // 0 for a masked key, whose v the projection zeroed
        l[r][i] = fmaf(l[r][i], al, p);
#pragma unroll
        for (int c = 0; c < DP / 4; ++c)
#pragma unroll
          for (int e = 0; e < 4; ++e) o[r][i][c][e] = fmaf(p, vr[i][c][e], o[r][i][c][e] * al);
        m[r][i] = mn;
      }
    }
  }

  // the lane's state relative to the wave's maximum, then all of them by channel
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int64_t row = row0 + r;
    if (row >= a.n_q) break;
    if (r > 0) __syncthreads();
#pragma unroll
    for (int i = 0; i < NH; ++i) {
      float mx = m[r][i];
#pragma unroll
      for (int x = 8; x >= 1; x >>= 1) mx = fmaxf(mx, __shfl_xor(mx, x, 16));
      const float f = expf(m[r][i] - (mx == -INFINITY ? 0.0f : mx));
      s_l[wave][n][4 * i + g] = l[r][i] * f;
      if (n == 0) s_m[wave][4 * i + g] = mx;
#pragma unroll
      for (int c = 0; c < DP / 4; ++c)
        *reinterpret_cast<f32x4*>(&s_o[wave][n][(4 * i + g) * DP + 4 * c]) = o[r][i][c] * f;
    }
    __syncthreads();
    for (int x = tid; x < hd; x += 64 * kGenWaves) {
      const int h = x / d, e = x - h * d;
      float mx = -INFINITY;
#pragma unroll
      for (int w = 0; w < kGenWaves; ++w) mx = fmaxf(mx, s_m[w][h]);
      float ls = 0.0f, acc = 0.0f;
#pragma unroll
      for (int w = 0; w < kGenWaves; ++w) {
        const float f = expf(s_m[w][h] - (mx == -INFINITY ? 0.0f : mx));
        float lw = 0.0f, ow = 0.0f;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          lw += s_l[w][i][h];
          ow += s_o[w][i][h * DP + e];
        }
        ls = fmaf(f, lw, ls);
        acc = fmaf(f, ow, acc);
      }
      const int64_t at = row * hd + x;
      if (a.out) {  // one part: gate and normalise here
        const float r = ls == 0.0f ? 0.0f : a.g[at] * (acc / ls);
        if (a.out_bf16)
          static_cast<__bf16*>(a.out)[at] = (__bf16)r;
        else
          static_cast<float*>(a.out)[at] = r;
      } else {
        a.acc_parts[(int64_t)part * a.n_q * hd + at] = acc;
        if (e == 0) {
          a.m_parts[((int64_t)part * H + h) * a.n_q + row] = mx;
          a.l_parts[((int64_t)part * H + h) * a.n_q + row] = ls;
        }
      }
    }
  }
}

// Two rows per workgroup share each k and v load: faster where z is small beside
// them and there are rows for it (32 channels, no mask: 900 tokens 54 against 61 us,
// though 700, where one row each takes little more than a round, 45 against 42), but
// the second row's state does not fit the registers beside 64 or 128 channels
// (601 tokens of 128: 75 against 61 us, of 64: 50 against 46).
template <int NH, int DP, bool BF16>
void gen_attn_launch(const GenAttnArgs& a, hipStream_t st) {
  const dim3 grid((unsigned)a.n_q, (unsigned)a.n_parts), block(64 * kGenWaves);
  if (a.c_z <= 32 && a.n_q * a.n_parts >= 512)
    hipLaunchKernelGGL((gen_attn_kernel<NH, DP, 2, BF16, 2>), dim3((grid.x + 1) / 2, grid.y), block, 0, st, a);
  else if (a.c_z <= 32)
    hipLaunchKernelGGL((gen_attn_kernel<NH, DP, 2, BF16, 1>), grid, block, 0, st, a);
  else if (a.c_z <= 64)
    hipLaunchKernelGGL((gen_attn_kernel<NH, DP, 4, BF16, 1>), grid, block, 0, st, a);
  else
    hipLaunchKernelGGL((gen_attn_kernel<NH, DP, 8, BF16, 1>), grid, block, 0, st, a);
}
template <int NH, int DP>
void gen_attn_launch(const GenAttnArgs& a, hipStream_t st) {
  if (a.z_bf16)
    gen_attn_launch<NH, DP, true>(a, st);
  else
    gen_attn_launch<NH, DP, false>(a, st);
}

// One thread per pair: the full bias with the LayerNorm affine and b_b.
__global__ void __launch_bounds__(256) gen_bias_kernel(GenBiasArgs a) {
  const int64_t total = a.n_rows * a.n_cols;
  for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < total; t += (int64_t)gridDim.x * blockDim.x) {
    const int64_t r = t / a.n_cols, c = t - r * a.n_cols;
    const int64_t off = r * a.row_stride + c * a.c_z;
    float mu, rstd;
    ln_stats(a.z, a.z_bf16, off, a.c_z, a.eps, mu, rstd);
    for (int h = 0; h < a.n_heads; ++h) {
      float b = a.b_b ? a.b_b[h] : 0.0f;
      for (int k = 0; k < a.c_z; ++k) {
        const float ln = (load_act(a.z, a.z_bf16, off + k) - mu) * rstd * (a.gamma ? a.gamma[k] : 1.0f) +
                         (a.beta ? a.beta[k] : 0.0f);
        b = fmaf(a.w_b[(int64_t)h * a.c_z + k], ln, b);
      }
      a.out[t * a.n_heads + h] = b;
    }
  }
}

int grid_for(int64_t items) {
  int64_t g = (items + 255) / 256;
  if (g > 8192) g = 8192;
  return (int)(g < 1 ? 1 : g);
}

}  // namespace

hipError_t launch_gen_proj(const GenProjArgs& a, hipStream_t st) {
  GenProjArgs b = a;
  b.s_vec = a.c_s % 4 == 0;  // s itself is 16-byte aligned
  // One 16 x 16 tile per wave while that leaves the chip short of waves (2048 =
  // two per SIMD), 2 x 2 beyond: each loaded operand then serves two products.
  const int64_t tiles = ((a.n_tok + 15) / 16 + (a.n_q + 15) / 16) * 2 * ((a.hd + 15) / 16);
  const int t = tiles <= 2048 ? 1 : 2;
  const int n_ot = (a.hd + 16 * t - 1) / (16 * t);
  const int64_t blocks = (a.n_tok + 16 * t - 1) / (16 * t) + (a.n_q + 16 * t - 1) / (16 * t);
  const dim3 grid((unsigned)blocks, (unsigned)((2 * n_ot + 3) / 4));
  if (t == 1)
    hipLaunchKernelGGL(gen_proj_kernel<1>, grid, dim3(256), 0, st, b);
  else
    hipLaunchKernelGGL(gen_proj_kernel<2>, grid, dim3(256), 0, st, b);
  return hipGetLastError();
}

// The tiled kernel takes pair widths of whole 16-channel chunks up to 128 and
// the head shapes whose k, v and accumulators (heads per lane times head size)
// fit its registers: up to 4 heads of 32, 8 of 16 or 16 of 8.
// Its 31-bit offsets reach 2 GiB of k or v and of one row of z.
bool gen_attn_tiled(int64_t n_tok, int32_t c_z, int32_t n_heads, int32_t head_dim) {
  const int per_lane = (n_heads + 3) / 4;
  return n_tok <= (1 << 22) - 16 && c_z % 16 == 0 && c_z <= 128 && head_dim % 4 == 0 &&
         head_dim <= (per_lane == 1 ? 32 : per_lane == 2 ? 16 : 8);
}

hipError_t launch_gen_attn(const GenAttnArgs& a, hipStream_t st) {
  if (!gen_attn_tiled(a.n_tok, a.c_z, a.n_heads, a.head_dim))
    hipLaunchKernelGGL(gen_attn_any_kernel, dim3((unsigned)a.n_q, (unsigned)a.n_parts), dim3(64), 0, st, a);
  else if (a.n_heads > 8)
    gen_attn_launch<4, 8>(a, st);
  else if (a.n_heads > 4)
    gen_attn_launch<2, 16>(a, st);
  else if (a.head_dim > 16)
    gen_attn_launch<1, 32>(a, st);
  else
    gen_attn_launch<1, 16>(a, st);
  return hipGetLastError();
}

hipError_t launch_gen_bias(const GenBiasArgs& a, hipStream_t st) {
  hipLaunchKernelGGL(gen_bias_kernel, dim3(grid_for(a.n_rows * a.n_cols)), dim3(256), 0, st, a);
  return hipGetLastError();
}

}  // namespace dcp
