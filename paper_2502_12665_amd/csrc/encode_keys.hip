// Prefill / append-side key encoder: query-aware quantisation function f' of section 4.2
// (f of section 2.2 when H = I), per subspace:
//     code = argmin_c (k_m - C[m,c]) H_m (k_m - C[m,c])^T ,  lowest c on exact ties.
//
// Following the Cholesky reformulation of section 4.2 (H = L L^T, z = k L, c^z = c L), keys and
// centroids are first mapped to the space where the distortion is the plain squared distance;
// sqrt(h) takes the place of L for per-dimension weights.  The 256 distances of a subvector are then
// formed on the matrix cores, where 1/2 |z - c|^2 = 1/2 |z|^2 + 1/2 |c|^2 - z . c fits one or two
// products: the inner dimension of a 32 x 32 x 16 product holds the 4 or 8 dimensions of a subspace
// twice, as the two f16 halves of the operands, and the two norms in the slots left over.  What
// remains for the vector ALU is ranking the results.
//
// A subvector whose two smallest distances are closer than that arithmetic can tell apart is decided
// again: its 256 distortions are evaluated in float64 straight from the definition by a whole wave.
// So the emitted code is the float64 argmin.
#include "common.hpp"
#include "internal.hpp"
#include "encode_few.hpp"

namespace a2ats {

size_t encode_ws_bytes(const a2ats_dims& d) {
  const size_t blocks = (size_t)d.n_kv_heads * d.n_sub;
  return blocks * d.sub_dim * d.sub_dim * sizeof(float) +
         blocks * kCentroids * d.sub_dim * sizeof(float);
}

// One workgroup per (KV head, subspace): transform matrix T (z = k T) and transformed centroids.
template <int DS>
__global__ __launch_bounds__(kCentroids) void encode_prepare_kernel(
    const float* __restrict__ codebook, const float* __restrict__ weights, int mode, int M,
    float* __restrict__ tmat, float* __restrict__ cz) {
  __shared__ double s_T[DS][DS];
  const int blk = blockIdx.x;          // kv * M + m
  const int kv = blk / M, m = blk % M;
  if (threadIdx.x == 0) {
    for (int r = 0; r < DS; ++r)
      for (int c = 0; c < DS; ++c) s_T[r][c] = 0.0;
    if (mode == A2ATS_W_DIAG) {
      for (int t = 0; t < DS; ++t) s_T[t][t] = sqrt((double)weights[(size_t)kv * M * DS + m * DS + t]);
    } else {   // lower Cholesky factor of the ds x ds block
      const float* H = weights + (size_t)blk * DS * DS;
      for (int r = 0; r < DS; ++r)
        for (int c = 0; c <= r; ++c) {
          double s = (double)H[r * DS + c];
          for (int t = 0; t < c; ++t) s -= s_T[r][t] * s_T[c][t];
          s_T[r][c] = (r == c) ? sqrt(s > 0.0 ? s : 0.0) : (s_T[c][c] > 0.0 ? s / s_T[c][c] : 0.0);
        }
    }
    for (int r = 0; r < DS; ++r)
      for (int c = 0; c < DS; ++c) tmat[(size_t)blk * DS * DS + r * DS + c] = (float)s_T[r][c];
  }
  __syncthreads();
  const int c = threadIdx.x;
  const float* cw = codebook + ((size_t)blk * kCentroids + c) * DS;
#pragma unroll
  for (int t = 0; t < DS; ++t) {
    double s = 0.0;
#pragma unroll
    for (int r = 0; r < DS; ++r) s += (double)cw[r] * s_T[r][t];
    cz[((size_t)blk * kCentroids + c) * DS + t] = (float)s;
  }
}

typedef __attribute__((ext_vector_type(8))) _Float16 f16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;

// Three f16 terms of x >= 0, x <= 65504, to 2^-33 x or 2^-25.
__device__ __forceinline__ void f16_limbs(float x, _Float16 (&o)[3]) {
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    o[i] = (_Float16)x;
    x -= (float)o[i];
  }
}

// a = {a of lanes 0..31, b of lanes 0..31}, b = {a of lanes 32..63, b of lanes 32..63}
__device__ __forceinline__ void swap_halves(uint32_t& a, uint32_t& b) {
  const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
  a = r[0];
  b = r[1];
}
__device__ __forceinline__ void swap_halves(f16x8& a, f16x8& b) {
  typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
  u32x4 x = __builtin_bit_cast(u32x4, a), y = __builtin_bit_cast(u32x4, b);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    uint32_t xi = x[i], yi = y[i];
    swap_halves(xi, yi);
    x[i] = xi;
    y[i] = yi;
  }
  a = __builtin_bit_cast(f16x8, x);
  b = __builtin_bit_cast(f16x8, y);
}

// The float64 decision of one subvector by a wave: every lane evaluates four centroids, the nearest wins
// (the lower index on ties; centroid 0 where no distortion is a finite number).
template <int DS, int MODE>
__device__ __forceinline__ int encode_exact_wave(const float* __restrict__ kp, const float* __restrict__ cw,
                                                 const float* __restrict__ w, int lane) {
  // cw: the subspace's centroids; w: its DS weights (per-dimension mode) or its DS x DS matrix
  double best = INFINITY;
  int arg = kCentroids;
#pragma unroll 1
  for (int c = lane; c < kCentroids; c += 64) {
    double dv[DS], dist = 0.0;
#pragma unroll
    for (int t = 0; t < DS; ++t) dv[t] = (double)kp[t] - (double)cw[(size_t)c * DS + t];
    if (MODE == A2ATS_W_NONE) {
#pragma unroll
      for (int t = 0; t < DS; ++t) dist += dv[t] * dv[t];
    } else if (MODE == A2ATS_W_DIAG) {
#pragma unroll
      for (int t = 0; t < DS; ++t) dist += dv[t] * (double)w[t] * dv[t];
    } else {
#pragma unroll
      for (int r = 0; r < DS; ++r)
#pragma unroll
        for (int cc = 0; cc < DS; ++cc) dist += dv[r] * (double)w[r * DS + cc] * dv[cc];
      asm volatile("" : "+s"(w));   // (the matrix is read again for the next centroid: it does not fit the registers)
    }
    if (dist < best) {
      best = dist;
      arg = c;
    }
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    const double od = __shfl_xor(best, off);
    const int oi = __shfl_xor(arg, off);
    if (od < best || (od == best && oi < arg)) {
      best = od;
      arg = oi;
    }
  }
  return arg & (kCentroids - 1);   // (nothing finite: kCentroids -> 0)
}

// A wave owns one subspace and walks over the keys 64 at a time, a lane per key; the 8 waves of a workgroup
// take 8 consecutive subspaces of the same keys, so that together they read 128 or 256 consecutive bytes of a
// key row and write 8 consecutive code bytes.  The subspace's 256 centroids stay in registers as A operands
// (8 blocks of 32); 32 keys at a time are the B operand, lane = key (lane % 32) in both lane halves
// g = lane / 32:
//
//   ds = 8, two products:  g = 0: z_hi . -c_hi  +  z_hi . -c_lo
//                          g = 1: z_lo . -c_hi  +  1/2|c|^2 . 1 + 1 . 1/2|z|^2  (three f16 terms each)
//   ds = 4, one product:   g = 0: z_hi . -c_hi + z_lo . -c_hi
//                          g = 1: z_hi . -c_lo + 1/2|c|^2 . 1 + 1 . 1/2|z|^2    (two f16 terms each)
//
// Ranking is by quads (the four centroids of four consecutive result registers of a lane): the smallest
// distance of each quad goes on with the quad's number in its low 6 mantissa bits, and the two smallest quads
// are kept.  The four centroids of the nearest quad are then compared by their direct float32 distances.
//
// Operands are scaled by the power of two that brings the subspace's largest centroid norm into [4, 8):
// f16 then holds keys of up to 45 times that norm, and its smallest step (2^-25 rounding) is 2^-27 of the norm.
// Error of a product, with S = (|z| + |c|)^2 / 2: operand rounding and the dropped z_lo . c_lo 5 * 2^-22 S,
// float32 accumulation over at most 32 terms about 2^-21 S, f16 steps 2^-25 * 2.9 (|z| + |c|) + 2^-24.  A
// centroid near the key has |c| <= |z| + sqrt(d), so S <= 4 |z|^2 + d; the margin between the two nearest
// quads covers two such errors and the 6 mantissa bits (2^-17) that give way to the quad's number.
// With a matrix, z = k L itself is off by e = (ds + 1) 2^-24 |k| |L|, which is no small part of a short z where the key lies
// along a direction that the block hardly weighs.  It moves |z - a|^2 - |z - b|^2 by 2 e |a - b|, and |a - b| is at most
// the sum of the two distances: 4 e sqrt(d) of a difference, half of it between halves.
//
// What bounds it: the vector ALU, of which the ranking is 17 instructions of a lane per 16 distances; these (min,
// med3, and_or) issue at half the rate of an add, 4 cycles a wave.  50001 keys x 32 heads x 16 subspaces,
// per-dimension weights: 2157 -> 545 us (one thread per subvector with 19 vector instructions per distance
// before; 698 us with the two smallest of all distances tracked, 9 cycles each).
constexpr int kEncThreads = 512;
constexpr int kEncWaves = kEncThreads / 64;   // subspaces of a workgroup
constexpr int kEncSteps = 16;                 // most steps of 64 keys of a workgroup

// 16-byte piece `p` of a quad of centroids in LDS: the position within the quad varies with the quad, so that
// lanes with different quads meet on different banks.
template <int DS>
__device__ __forceinline__ int quad_piece(int quad, int p) {
  return DS == 8 ? quad * 8 + (p ^ (quad & 7)) : quad * 4 + (p ^ ((quad >> 2) & 3));
}

template <int DS, int MODE>
__global__ __launch_bounds__(kEncThreads) __attribute__((amdgpu_waves_per_eu(4, 4))) void encode_kernel(
    const float* __restrict__ keys, const float* __restrict__ codebook,
    const float* __restrict__ weights, const float* __restrict__ tmat, const float* __restrict__ cz,
    uint8_t* __restrict__ codes, int Hkv, int M, int n_new, int pos0, int64_t ctx_stride, int n_steps) {
  constexpr int D = 128, kBlk = kCentroids / 32;
  __shared__ float4 s_cz[kEncWaves][kCentroids * DS / 4];   // scaled centroids, see quad_piece
  __shared__ __align__(16) uint8_t s_code[kEncSteps * 64][kEncWaves];
  __shared__ uint64_t s_near[kEncWaves][kEncSteps];   // keys of a step that float64 has to decide
  const int tid = threadIdx.x, lane = tid & 63, col = lane & 31, g = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int m = blockIdx.x * kEncWaves + wave, bkv = blockIdx.z, kv = bkv % Hkv, blk = kv * M + m;
  const int first = blockIdx.y * n_steps * 64;   // (host: first < n_new)
  const int n_mine = min(n_new - first, n_steps * 64);
  const float* my_keys = keys + ((size_t)bkv * n_new + first) * D + m * DS;

  // Centroid operands.  Lane `col` of block b holds centroid 32 b + col.
  f16x8 a1[kBlk], a2[DS == 8 ? kBlk : 1];
  float scale = 1.f;
  bool all_near = false;   // a subspace whose centroids are not finite or too far from 1 is left to float64
  {
    const float* cp = (MODE == A2ATS_W_NONE ? codebook : cz) + (size_t)blk * kCentroids * DS;
    float most = 0.f;
    bool finite = true;
#pragma unroll
    for (int b = 0; b < kBlk; ++b) {
      float n2 = 0.f;
#pragma unroll
      for (int t = 0; t < DS; ++t) {
        const float c = cp[(32 * b + col) * DS + t];
        n2 += c * c;
      }
      finite &= n2 < INFINITY;
      most = fmaxf(most, n2);
    }
#pragma unroll
    for (int off = 16; off >= 1; off >>= 1) most = fmaxf(most, __shfl_xor(most, off));
    all_near = __builtin_amdgcn_ballot_w64(!finite) != 0;
    const int e = (int)(__float_as_uint(sqrtf(most)) >> 23) - 127;   // |c| in [2^e, 2^(e+1))
    if (!(e > -60 && e < 60)) all_near = true;
    else scale = __uint_as_float((uint32_t)(127 + 2 - e) << 23);
#pragma unroll
    for (int b = 0; b < kBlk; ++b) {
      _Float16 hi[DS], lo[DS], nn[3];
      float c[DS], n2 = 0.f;
      const int row = 32 * b + col;
#pragma unroll
      for (int t = 0; t < DS; ++t) {
        c[t] = scale * cp[row * DS + t];
        n2 += c[t] * c[t];
        hi[t] = (_Float16)-c[t];
        lo[t] = (_Float16)(-c[t] - (float)hi[t]);
      }
      {   // (a lane half writes half of an 8-dimension centroid, both write the same of a 4-dimension one)
        const float4 f = *(const float4*)(cp + row * DS + (DS == 8 ? 4 * g : 0));
        s_cz[wave][quad_piece<DS>(row >> 2, DS == 8 ? (row & 3) * 2 + g : row & 3)] =
            make_float4(scale * f.x, scale * f.y, scale * f.z, scale * f.w);
      }
      f16_limbs(0.5f * n2, nn);
      const _Float16 one = (_Float16)1.f, zero = (_Float16)0.f;
      if constexpr (DS == 8) {
        const _Float16 tail[8] = {nn[0], nn[1], nn[2], one, one, one, zero, zero};
#pragma unroll
        for (int t = 0; t < 8; ++t) {
          a1[b][t] = hi[t];
          a2[b][t] = g ? tail[t] : lo[t];
        }
      } else {
        const _Float16 tail[4] = {nn[0], nn[1], one, one};
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          a1[b][t] = g ? lo[t] : hi[t];
          a1[b][4 + t] = g ? tail[t] : hi[t];
        }
      }
    }
  }

  const float* T = MODE == A2ATS_W_NONE ? nullptr : tmat + (size_t)blk * DS * DS;
  float t_err2 = 0.f;   // e^2 of a key of length 1
  if (MODE == A2ATS_W_BLOCK) {
#pragma unroll
    for (int r = 0; r < DS; ++r)
#pragma unroll
      for (int t = 0; t <= r; ++t) t_err2 += T[r * DS + t] * T[r * DS + t];
    t_err2 *= (DS + 1) * 6e-8f * scale * ((DS + 1) * 6e-8f * scale);
  }
  const int steps = (n_mine + 63) / 64;
  const uint32_t keep = ~63u;
#pragma unroll 1
  for (int step = 0; step < steps; ++step) {
    float z[DS], zz = 0.f, kk = 0.f;
    {
      const float* kp = my_keys + (size_t)min(step * 64 + lane, n_mine - 1) * D;
      float ks[DS];
#pragma unroll
      for (int t = 0; t < DS; t += 4) {
        const float4 f = *(const float4*)(kp + t);
        ks[t] = f.x; ks[t + 1] = f.y; ks[t + 2] = f.z; ks[t + 3] = f.w;
      }
#pragma unroll
      for (int t = 0; t < DS; ++t) {
        if (MODE == A2ATS_W_NONE) {
          z[t] = ks[t];
        } else if (MODE == A2ATS_W_DIAG) {
          z[t] = ks[t] * T[t * DS + t];
        } else {
          z[t] = 0.f;
#pragma unroll
          for (int r = t; r < DS; ++r) z[t] += ks[r] * T[r * DS + t];   // T is lower triangular
        }
        z[t] *= scale;
        zz += z[t] * z[t];
        if (MODE == A2ATS_W_BLOCK) kk += ks[t] * ks[t];
      }
    }
    // Operands of the lane's key, then of keys 0 .. 31 (b1a, b2a) and 32 .. 63 (b1b, b2b) in both halves.
    f16x8 b1a, b2a, b1b, b2b;
    {
      _Float16 hi[DS], lo[DS], qq[3];
#pragma unroll
      for (int t = 0; t < DS; ++t) {
        hi[t] = (_Float16)z[t];
        lo[t] = (_Float16)(z[t] - (float)hi[t]);
      }
      f16_limbs(0.5f * zz, qq);
      const _Float16 one = (_Float16)1.f, zero = (_Float16)0.f;
      if constexpr (DS == 8) {
        b1a = b2a = f16x8{hi[0], hi[1], hi[2], hi[3], hi[4], hi[5], hi[6], hi[7]};
        b1b = f16x8{lo[0], lo[1], lo[2], lo[3], lo[4], lo[5], lo[6], lo[7]};
        b2b = f16x8{one, one, one, qq[0], qq[1], qq[2], zero, zero};
        swap_halves(b1a, b1b);
        swap_halves(b2a, b2b);
      } else {
        b1a = f16x8{hi[0], hi[1], hi[2], hi[3], lo[0], lo[1], lo[2], lo[3]};
        b1b = f16x8{hi[0], hi[1], hi[2], hi[3], one, one, qq[0], qq[1]};
        swap_halves(b1a, b1b);
      }
    }

    // Register v of block b: centroid 32 b + 8 (v / 4) + 4 g + v % 4, quad 2 (4 b + v / 4) + g.  Results are
    // >= 0 up to their error, so their bit patterns order like the values as signed integers; two below zero
    // are within the margin of each other whatever their order.
    auto rank = [&](const f16x8& b1, const f16x8& b2, int32_t& k1, int32_t& k2) {
      k1 = k2 = 0x7fffffff;
#pragma unroll
      for (int b = 0; b < kBlk; ++b) {
        f32x16 acc;   // (three other waves of the SIMD rank meanwhile)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[v] = 0.f;
        acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(a1[b], b1, acc, 0, 0, 0);
        if constexpr (DS == 8) acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(a2[b], b2, acc, 0, 0, 0);
        int32_t key[4], m0, m1;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int32_t x0 = (int32_t)__float_as_uint(acc[4 * u]), x1 = (int32_t)__float_as_uint(acc[4 * u + 1]),
                        x2 = (int32_t)__float_as_uint(acc[4 * u + 2]), x3 = (int32_t)__float_as_uint(acc[4 * u + 3]);
          const int32_t least = min(min(min(x0, x1), x2), x3);
          key[u] = (int32_t)(((uint32_t)least & keep) | (uint32_t)(2 * (4 * b + u)));
        }
        // two at a time: the median of (smallest so far, two new) is the only candidate they add for second place
        asm("v_med3_i32 %0, %1, %2, %3" : "=v"(m0) : "v"(k1), "v"(key[0]), "v"(key[1]));
        asm("v_min3_i32 %0, %1, %2, %3" : "=v"(k1) : "v"(k1), "v"(key[0]), "v"(key[1]));
        asm("v_med3_i32 %0, %1, %2, %3" : "=v"(m1) : "v"(k1), "v"(key[2]), "v"(key[3]));
        asm("v_min3_i32 %0, %1, %2, %3" : "=v"(k1) : "v"(k1), "v"(key[2]), "v"(key[3]));
        asm("v_min3_i32 %0, %1, %2, %3" : "=v"(k2) : "v"(k2), "v"(m0), "v"(m1));
        __builtin_amdgcn_sched_barrier(0);   // one result tile at a time: two and the operands do not fit 128 registers
      }
      k1 |= g;
      k2 |= g;
    };
    int32_t k1, k2;
    {
      int32_t p1, p2, q1, q2;
      rank(b1a, b2a, p1, p2);
      rank(b1b, b2b, q1, q2);
      uint32_t u0 = (uint32_t)p1, u1 = (uint32_t)q1, w0 = (uint32_t)p2, w1 = (uint32_t)q2;
      swap_halves(u0, u1);   // now lane = key: both lane halves' smallest two
      swap_halves(w0, w1);
      k1 = min((int32_t)u0, (int32_t)u1);
      k2 = min(max((int32_t)u0, (int32_t)u1), min((int32_t)w0, (int32_t)w1));
    }
    const float q1 = __uint_as_float((uint32_t)k1 & keep), q2 = __uint_as_float((uint32_t)k2 & keep);
    const int quad = k1 & 63;
    int32_t c1 = 0x7fffffff, c2 = 0x7fffffff;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float d = 0.f;
#pragma unroll
      for (int t = 0; t < DS; t += 4) {
        const float4 c = s_cz[wave][quad_piece<DS>(quad, (i * DS + t) / 4)];
        const float e0 = z[t] - c.x, e1 = z[t + 1] - c.y, e2 = z[t + 2] - c.z, e3 = z[t + 3] - c.w;
        d += e0 * e0;
        d += e1 * e1;
        d += e2 * e2;
        d += e3 * e3;
      }
      const int32_t key = (int32_t)((__float_as_uint(d) & ~3u) | (uint32_t)i);
      c2 = min(c2, max(c1, key));
      c1 = min(c1, key);
    }
    const float d1 = __uint_as_float((uint32_t)c1 & ~3u), d2 = __uint_as_float((uint32_t)c2 & ~3u);
    float between = 3.5e-5f * q2 + 2e-5f * zz + 1e-6f, within = 1e-5f * d2 + 4e-6f * zz + 1e-30f;
    if (MODE == A2ATS_W_BLOCK) {
      const float e2 = t_err2 * kk;   // (the bare instruction is good to an ulp; the library's root takes as long as half a tile)
      between += __builtin_amdgcn_sqrtf(8.f * e2 * fmaxf(q2, 0.f));
      within += __builtin_amdgcn_sqrtf(16.f * e2 * d2);
    }
    // (NaN anywhere: not decided)
    const bool decided = q2 - q1 > between && d2 - d1 > within && zz <= 1.2e5f && !all_near;
    const uint64_t near = __builtin_amdgcn_ballot_w64(!decided);
    s_code[step * 64 + lane][wave] = (uint8_t)(4 * quad + (c1 & 3));
    if (lane == 0) s_near[wave][step] = near;
  }
#pragma unroll 1
  for (int step = 0; step < steps; ++step) {
    uint64_t near = s_near[wave][step];
    near = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)near) |
           (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(near >> 32)) << 32;
    while (near) {
      const int at = step * 64 + __builtin_ctzll(near);
      near &= near - 1;
      if (at >= n_mine) break;
      const float* w = MODE == A2ATS_W_NONE   ? nullptr
                       : MODE == A2ATS_W_DIAG ? weights + (size_t)kv * D + m * DS
                                              : weights + (size_t)blk * DS * DS;
      const int arg = encode_exact_wave<DS, MODE>(my_keys + (size_t)at * D, codebook + (size_t)blk * kCentroids * DS, w, lane);
      if (lane == 0) s_code[at][wave] = (uint8_t)arg;
    }
  }
  __syncthreads();
  uint8_t* out = codes + ((size_t)bkv * ctx_stride + pos0 + first) * M + blockIdx.x * kEncWaves;
  if (((uintptr_t)codes & 7) == 0) {   // (M is a multiple of 8)
    for (int i = tid; i < n_mine; i += kEncThreads) *(uint2*)(out + (size_t)i * M) = *(const uint2*)s_code[i];
  } else {
    for (int i = tid; i < n_mine * kEncWaves; i += kEncThreads)
      out[(size_t)(i / kEncWaves) * M + i % kEncWaves] = s_code[i / kEncWaves][i % kEncWaves];
  }
}

// Append-time shape (a few new keys per sequence, e.g. one per decode step): a workgroup of 256 threads takes one (key,
// subspace) pair, a thread per centroid, in float64 from the definition (see encode_few.hpp), so nothing is prepared and the
// weighted modes too are one launch; the matrix-core kernel has 64 rows of keys in a step whatever the number of keys, and the
// weighted modes a launch before it.  Bound by float64 arithmetic, a time that grows with the pairs: M = 16, weights per
// dimension, a whole call: 8 us up to 4096 pairs (one key of 32 sequences x 8 KV heads), 126 at 131072 (32 keys of them),
// where the other kernel takes 19 (33 keys; 8 KV heads of one sequence: 8 here, 13 there).  The line at 32 keys is
// a2ats_decode_prologue's, which takes as many and has no workspace; by time alone it would lie near 8192 pairs.
template <int DS>
__global__ __launch_bounds__(kCentroids) void encode_few_kernel(
    const float* __restrict__ keys, const float* __restrict__ codebook,
    const float* __restrict__ weights, int mode, uint8_t* __restrict__ codes, int Hkv, int M,
    int n_new, int pos0, int64_t ctx_stride) {
  __shared__ double s_d[4];
  __shared__ int s_i[4];
  encode_few_pair<DS>(keys, codebook, weights, mode, codes, Hkv, M, n_new, pos0, ctx_stride, blockIdx.x,
                      blockIdx.y, blockIdx.z, threadIdx.x, 0, true, s_d, s_i);
}

template <int DS>
static hipError_t launch_encode_ds(const a2ats_dims& d, const float* keys, int n_new, int pos0,
                                   const float* codebook, const float* weights, int mode, uint8_t* codes,
                                   void* ws, hipStream_t stream) {
  const int M = d.n_sub, Hkv = d.n_kv_heads;
  if (n_new <= kFewKeys) {
    hipLaunchKernelGGL((encode_few_kernel<DS>), dim3(M, n_new, d.batch * Hkv), dim3(kCentroids), 0, stream,
                       keys, codebook, weights, mode, codes, Hkv, M, n_new, pos0, d.ctx_stride);
    return hipGetLastError();
  }
  float* tmat = (float*)ws;
  float* cz = tmat ? tmat + (size_t)Hkv * M * DS * DS : nullptr;
  if (mode != A2ATS_W_NONE) {
    hipLaunchKernelGGL((encode_prepare_kernel<DS>), dim3(Hkv * M), dim3(kCentroids), 0, stream, codebook,
                       weights, mode, M, tmat, cz);
    hipError_t err = hipGetLastError();
    if (err != hipSuccess) return err;
  }
  // Steps of 64 keys per workgroup: preparing the centroid operands costs a workgroup about as much as one step
  // (6 us each with all 512 workgroups resident), so the number that needs the fewest such units over all rounds.
  // 2 x 8000 keys, 8 heads, M = 16: 53 us; with a step per workgroup 97 us.
  const long steps = ((long)n_new + 63) / 64, groups = (long)d.batch * Hkv * (M / kEncWaves);
  int per = 1;
  long least = -1;
  for (int p = 1; p <= kEncSteps; ++p) {
    const long units = ((steps + p - 1) / p * groups + 511) / 512 * (p + 1);
    if (least < 0 || units < least) {
      least = units;
      per = p;
    }
  }
  const dim3 grid(M / kEncWaves, (unsigned)((steps + per - 1) / per), d.batch * Hkv), block(kEncThreads);
#define A2ATS_LAUNCH_ENC(MODE)                                                                      \
  hipLaunchKernelGGL((encode_kernel<DS, MODE>), grid, block, 0, stream, keys, codebook, weights, tmat, \
                     cz, codes, Hkv, M, n_new, pos0, d.ctx_stride, per)
  if (mode == A2ATS_W_NONE) A2ATS_LAUNCH_ENC(A2ATS_W_NONE);
  else if (mode == A2ATS_W_DIAG) A2ATS_LAUNCH_ENC(A2ATS_W_DIAG);
  else A2ATS_LAUNCH_ENC(A2ATS_W_BLOCK);
#undef A2ATS_LAUNCH_ENC
  return hipGetLastError();
}

hipError_t launch_encode(const a2ats_dims& d, const float* keys, int n_new, int pos0, const float* codebook,
                         const float* weights, int mode, uint8_t* codes, void* ws, hipStream_t stream) {
  if (n_new == 0 || d.batch == 0) return hipSuccess;
  if (d.sub_dim == 8)
    return launch_encode_ds<8>(d, keys, n_new, pos0, codebook, weights, mode, codes, ws, stream);
  return launch_encode_ds<4>(d, keys, n_new, pos0, codebook, weights, mode, codes, ws, stream);
}

}  // namespace a2ats
