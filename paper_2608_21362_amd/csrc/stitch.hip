// Stitch: dequantise cached KIVI chunks and rotate their keys from the cached
// position to the new one (Sec. 4.3 assembly, Sec. 3.2 R^Delta, Sec. 4.5).
//
// One workgroup per (chunk, layer, kv head): 128 tokens x d channels of K and
// of V (small launches split the tokens, below).  HBM-bound: per workgroup it
// reads the K and V code blocks (C*d*b/8 bytes each) and their float
// statistics, and writes 2*C*d output elements.
//
// Keys: one thread takes 4 consecutive tokens (one statistic group, Gk % 4 == 0),
// or one in small launches, and 8 channel pairs (j, j + d/2).
// Values: one thread takes one token and 8 consecutive channels (one statistic group,
// Gv % 8 == 0; the API asks Gv % 16) at a time, so 16 (d = 128) or 8 (d = 64)
// lanes store a whole row and a wave's stores are contiguous.
// stitch_kernel requests every input before its key work starts, the head's key
// statistics and the rotation row first: they are staged in LDS and read two
// channel pairs at a time, widened to double once for the thread's four tokens.
// (Held in registers for all 8 pairs they took 182 registers instead of 120, two
// waves per SIMD instead of four: 32 int8 chunks x 36 layers 51.0 -> 48.9 us, 4.7
// TB/s from cold caches, where a streaming copy reaches 5.2.)
// stitch_deviation_kernel, which also holds the fresh keys, reads the staged
// statistics for every token and loads its value inputs after the key work:
// neither is then held in registers while a key job's loads are in flight (158
// registers, three waves per SIMD, 5.4 TB/s; the order of stitch_kernel took 224
// registers, or 166 with the steps kept apart, and 424.5 instead of 422.0 us for
// 256 chunks x 36 layers).
//
// Arithmetic is double with contraction off: x = fma(code, scale, zero) is
// exact in the product (8-bit code times 24-bit scale), so it equals the
// product-then-sum form; the rotation is mul, mul, sub / add.  The double is
// rounded to float, and for bfloat16 output the float is rounded again.
//
// Fused deviation: one workgroup per (chunk, layer) walks the kv heads;
// every key job also reads the fresh key pieces of its tokens and accumulates
// dot and both squared norms in double over the bf16 values it stores (Alg. 2
// step 2 on the stitched rows, K only, per layer).  The eight (d = 128) or four
// (d = 64) lanes of a job combine their sums with xor-shuffles, every
// lane forms the head's cosine and adds it to the token's running sum, and after
// the last head one lane per job writes delta for its tokens.  Summing
// dot and both norms in one order keeps identical rows at delta = 0 exactly.
#include <math.h>

#include <type_traits>

#include "kvb_device.h"
#include "kvb_internal.h"

namespace kvb {
namespace {

constexpr int kC = 128;

// sum of x over the TPT adjacent lanes of a job (TPT a power of two)
template <int TPT>
__device__ __forceinline__ double quad_lanes_sum(double x) {
#pragma unroll
  for (int m = 1; m < TPT; m <<= 1) x += __shfl_xor(x, m, 64);
  return x;
}

// N consecutive floats at p (N * 4-byte aligned)
template <int N>
__device__ __forceinline__ void load_stat(const float* p, float (&x)[N]) {
  typedef __attribute__((ext_vector_type(N < 4 ? N : 4))) float V;
  constexpr int E = N < 4 ? N : 4;
#pragma unroll
  for (int i = 0; i < N / E; ++i) {
    const V v = reinterpret_cast<const V*>(p)[i];
#pragma unroll
    for (int e = 0; e < E; ++e) x[i * E + e] = v[e];
  }
}

template <int BITS, int D, bool BF16, int TOK>
__global__ void __launch_bounds__(256)
stitch_kernel(int32_t L, int32_t Hkv, int32_t Gk, int32_t Gv, int32_t n_pool,
              const uint8_t* __restrict__ k_codes, const float* __restrict__ k_scale,
              const float* __restrict__ k_zero, const uint8_t* __restrict__ v_codes,
              const float* __restrict__ v_scale, const float* __restrict__ v_zero,
              const kvb_chunk* __restrict__ chunks, const float* __restrict__ rope_cos,
              const float* __restrict__ rope_sin, int64_t t_total, void* __restrict__ k_out,
              void* __restrict__ v_out) {
  constexpr int H = D / 2;
  constexpr int CB = D * BITS / 8;       // code bytes per token row
  constexpr int TPT = H / 8;             // key threads per token
  constexpr int WT = TOK == 4 ? kC : 256 / TPT;  // tokens of a workgroup
  constexpr int KJOBS = (WT / TOK) * TPT;  // 256, or 128 (d = 64, four tokens a thread)
  static_assert(KJOBS <= 256, "one key job per thread");
  const int c = blockIdx.x;
  const kvb_chunk ch = chunks[c];
  if (ch.pool_idx < 0 || ch.pool_idx >= n_pool || ch.dst_row < 0 ||
      (int64_t)ch.dst_row + kC > t_total)
    return;
  const int ngk = kC / Gk, ngv = D / Gv;
  const int u_base = TOK == 4 ? 0 : (int)blockIdx.z * WT;
  const int tid = threadIdx.x;
  const int l = (int)blockIdx.y / Hkv, h = (int)blockIdx.y % Hkv;
  const int64_t slab = ((int64_t)ch.pool_idx * L + l) * Hkv + h;  // (p, l, h)
  const int64_t out_row0 = ((int64_t)l * Hkv + h) * t_total + ch.dst_row;

  // whole chunks: the head's key statistics (scale, then zero; at most WT/4
  // groups) and the rotation row (cos, then sin) go through LDS; requested first,
  // they are waited for first
  constexpr bool STAGED = TOK == 4;
  __shared__ float4 st_k4[STAGED ? 2 * (WT / 4) * D / 4 : 1];
  __shared__ float4 st_r4[STAGED ? D / 4 : 1];
  const int n4 = ngk * D / 4;
  const float4* ks4 = reinterpret_cast<const float4*>(k_scale + slab * ngk * D);
  const float4* kz4 = reinterpret_cast<const float4*>(k_zero + slab * ngk * D);
  float4 a_sc = {}, a_zr = {}, a_rot = {};
  if constexpr (STAGED) {
    if (tid < n4) {
      a_sc = ks4[tid];
      a_zr = kz4[tid];
    }
    if (tid < D / 4)
      a_rot = reinterpret_cast<const float4*>((tid < H / 4 ? rope_cos : rope_sin) +
                                              (int64_t)c * H)[tid % (H / 4)];
  }
  // key codes: TOK tokens from u0, channel pairs [j0, j0 + 8)
  const bool keys = KJOBS == 256 || tid < KJOBS;
  const int u0 = u_base + TOK * (tid / TPT), j0 = 8 * (tid % TPT), g = u0 / Gk;
  uint32_t cwl[TOK][2], cwh[TOK][2];
  if (keys) {
#pragma unroll
    for (int i = 0; i < TOK; ++i) {
      const uint8_t* row = k_codes + (slab * kC + u0 + i) * CB;
      if constexpr (BITS == 8) {
        const uint2 a = *reinterpret_cast<const uint2*>(row + j0);
        const uint2 b = *reinterpret_cast<const uint2*>(row + H + j0);
        cwl[i][0] = a.x; cwl[i][1] = a.y; cwh[i][0] = b.x; cwh[i][1] = b.y;
      } else {
        cwl[i][0] = *reinterpret_cast<const uint32_t*>(row + j0 / 2);
        cwh[i][0] = *reinterpret_cast<const uint32_t*>(row + (H + j0) / 2);
        cwl[i][1] = cwh[i][1] = 0;
      }
    }
  }
  // value inputs of this thread's pieces (token u, channels [v0, v0 + 8))
  constexpr int VP = D / 8;              // pieces per token row
  constexpr int VPT = WT * VP / 256;     // pieces per thread
  uint32_t vw[VPT][2];
  float vsc[VPT], vzr[VPT];
#pragma unroll
  for (int k = 0; k < VPT; ++k) {
    const int vj = tid + 256 * k;
    const int u = u_base + vj / VP, v0 = (vj % VP) * 8;
    const int64_t srow = slab * kC + u;
    vsc[k] = v_scale[srow * ngv + v0 / Gv];
    vzr[k] = v_zero[srow * ngv + v0 / Gv];
    const uint8_t* row = v_codes + srow * CB;
    if constexpr (BITS == 8) {
      const uint2 a = *reinterpret_cast<const uint2*>(row + v0);
      vw[k][0] = a.x;
      vw[k][1] = a.y;
    } else {
      vw[k][0] = *reinterpret_cast<const uint32_t*>(row + v0 / 2);
      vw[k][1] = 0;
    }
  }
  if constexpr (STAGED) {
    if (tid < n4) {
      st_k4[tid] = a_sc;
      st_k4[n4 + tid] = a_zr;
    }
    if (tid < D / 4) st_r4[tid] = a_rot;
    for (int i = tid + 256; i < n4; i += 256) {  // groups of 4 or 8 tokens
      st_k4[i] = ks4[i];
      st_k4[n4 + i] = kz4[i];
    }
    __syncthreads();
  }

  if (keys) {
    // ---- keys: a step's statistics are widened once for the thread's tokens
    const float* sc = STAGED ? reinterpret_cast<const float*>(st_k4) + g * D
                             : k_scale + (slab * ngk + g) * D;
    const float* zr = STAGED ? reinterpret_cast<const float*>(st_k4) + (ngk + g) * D
                             : k_zero + (slab * ngk + g) * D;
    const float* rc = STAGED ? reinterpret_cast<const float*>(st_r4) : rope_cos + (int64_t)c * H;
    const float* rs = STAGED ? reinterpret_cast<const float*>(st_r4) + H : rope_sin + (int64_t)c * H;
    constexpr int KS = STAGED ? 2 : 8;  // channel pairs per step
    // a token's results: bf16 pairs, or floats
    typedef typename std::conditional<BF16, uint32_t, float>::type Out;
    constexpr int NO = BF16 ? 4 : 8;
    Out lo[TOK][NO], hi[TOK][NO];
#pragma unroll
    for (int k0 = 0; k0 < 8; k0 += KS) {
      if (STAGED && k0 > 0) asm volatile("" ::: "memory");  // each step's statistics in its turn
      float s_lo[KS], s_hi[KS], z_lo[KS], z_hi[KS], cs[KS], sn[KS];
      load_stat<KS>(sc + j0 + k0, s_lo);
      load_stat<KS>(sc + H + j0 + k0, s_hi);
      load_stat<KS>(zr + j0 + k0, z_lo);
      load_stat<KS>(zr + H + j0 + k0, z_hi);
      load_stat<KS>(rc + j0 + k0, cs);
      load_stat<KS>(rs + j0 + k0, sn);
#pragma unroll
      for (int e = 0; e < KS; e += 2)
#pragma unroll
        for (int i = 0; i < TOK; ++i) {
          float ylo[2], yhi[2];
#pragma unroll
          for (int m = 0; m < 2; ++m) {
            const int k = k0 + e + m;
            const double xl = __builtin_fma((double)code_at<BITS>(cwl[i], k),
                                            (double)s_lo[e + m], (double)z_lo[e + m]);
            const double xh = __builtin_fma((double)code_at<BITS>(cwh[i], k),
                                            (double)s_hi[e + m], (double)z_hi[e + m]);
            const double a = xl * (double)cs[e + m];
            const double b = xh * (double)sn[e + m];
            const double f = xh * (double)cs[e + m];
            const double w = xl * (double)sn[e + m];
            ylo[m] = (float)(a - b);
            yhi[m] = (float)(f + w);
          }
          if constexpr (BF16) {
            lo[i][(k0 + e) / 2] = pack_bf16x2(ylo[0], ylo[1]);
            hi[i][(k0 + e) / 2] = pack_bf16x2(yhi[0], yhi[1]);
          } else {
#pragma unroll
            for (int m = 0; m < 2; ++m) {
              lo[i][k0 + e + m] = ylo[m];
              hi[i][k0 + e + m] = yhi[m];
            }
          }
        }
    }
#pragma unroll
    for (int i = 0; i < TOK; ++i) {
      const int64_t o = (out_row0 + u0 + i) * D;
      if constexpr (BF16) {
        uint16_t* ko = reinterpret_cast<uint16_t*>(k_out) + o;
        *reinterpret_cast<uint4*>(ko + j0) = make_uint4(lo[i][0], lo[i][1], lo[i][2], lo[i][3]);
        *reinterpret_cast<uint4*>(ko + H + j0) = make_uint4(hi[i][0], hi[i][1], hi[i][2], hi[i][3]);
      } else {
        float* ko = reinterpret_cast<float*>(k_out) + o;
#pragma unroll
        for (int k = 0; k < 8; k += 4) {
          *reinterpret_cast<float4*>(ko + j0 + k) =
              make_float4(lo[i][k], lo[i][k + 1], lo[i][k + 2], lo[i][k + 3]);
          *reinterpret_cast<float4*>(ko + H + j0 + k) =
              make_float4(hi[i][k], hi[i][k + 1], hi[i][k + 2], hi[i][k + 3]);
        }
      }
    }
  }

  // ---- values
#pragma unroll
  for (int k = 0; k < VPT; ++k) {
    const int vj = tid + 256 * k;
    const int u = u_base + vj / VP, v0 = (vj % VP) * 8;
    const double sc = vsc[k], zr = vzr[k];
    float y[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) y[e] = (float)__builtin_fma((double)code_at<BITS>(vw[k], e), sc, zr);
    const int64_t o = (out_row0 + u) * D + v0;
    if constexpr (BF16) {
      *reinterpret_cast<uint4*>(reinterpret_cast<uint16_t*>(v_out) + o) =
          make_uint4(pack_bf16x2(y[0], y[1]), pack_bf16x2(y[2], y[3]), pack_bf16x2(y[4], y[5]),
                     pack_bf16x2(y[6], y[7]));
    } else {
      float* vo = reinterpret_cast<float*>(v_out) + o;
      *reinterpret_cast<float4*>(vo) = make_float4(y[0], y[1], y[2], y[3]);
      *reinterpret_cast<float4*>(vo + 4) = make_float4(y[4], y[5], y[6], y[7]);
    }
  }
}

template <int BITS, int D, int TOK>
__global__ void __launch_bounds__(256)
stitch_deviation_kernel(int32_t L, int32_t Hkv, int32_t Gk, int32_t Gv, int32_t n_pool,
              const uint8_t* __restrict__ k_codes, const float* __restrict__ k_scale,
              const float* __restrict__ k_zero, const uint8_t* __restrict__ v_codes,
              const float* __restrict__ v_scale, const float* __restrict__ v_zero,
              const kvb_chunk* __restrict__ chunks, const float* __restrict__ rope_cos,
              const float* __restrict__ rope_sin, int64_t t_total, uint16_t* __restrict__ k_out,
              uint16_t* __restrict__ v_out, const uint16_t* __restrict__ k_fresh,
              float* __restrict__ delta) {
  constexpr int H = D / 2;
  constexpr int CB = D * BITS / 8;       // code bytes per token row
  constexpr int TPT = H / 8;             // key threads per token
  constexpr int WT = TOK == 4 ? kC : 256 / TPT;  // tokens of a workgroup
  constexpr int KJOBS = (WT / TOK) * TPT;  // 256, or 128 (d = 64, four tokens a thread)
  static_assert(KJOBS <= 256, "one key job per thread");
  const int c = blockIdx.x;
  const kvb_chunk ch = chunks[c];
  if (ch.pool_idx < 0 || ch.pool_idx >= n_pool || ch.dst_row < 0 ||
      (int64_t)ch.dst_row + kC > t_total)
    return;
  const int ngk = kC / Gk, ngv = D / Gv;
  const int u_base = TOK == 4 ? 0 : (int)blockIdx.z * WT;
  // fused deviation: running cosine sum over heads of this thread's tokens
  double cos_sum[TOK] = {};
  // fused: the head's key statistics of the workgroup's groups (scale, then
  // zero; at most WT/4 groups) and the chunk's rotation row (cos, then sin)
  // staged in LDS, read per token
  const int g_base = u_base / Gk, n_gs = Gk < WT ? WT / Gk : 1;
  __shared__ float4 st_k4[2 * (WT / 4) * D / 4];
  __shared__ float4 st_r4[D / 4];
  const int l = blockIdx.y;
  for (int h = 0; h < Hkv; ++h) {
    const int64_t slab = ((int64_t)ch.pool_idx * L + l) * Hkv + h;  // (p, l, h)
    const int64_t out_row0 = ((int64_t)l * Hkv + h) * t_total + ch.dst_row;
    // the previous head's key jobs are done with the staged statistics
    __syncthreads();
    const int n4 = n_gs * D / 4;
    const float4* ks4 = reinterpret_cast<const float4*>(k_scale + (slab * ngk + g_base) * D);
    const float4* kz4 = reinterpret_cast<const float4*>(k_zero + (slab * ngk + g_base) * D);
    for (int i = threadIdx.x; i < n4; i += blockDim.x) {
      st_k4[i] = ks4[i];
      st_k4[n4 + i] = kz4[i];
    }
    if (threadIdx.x < H / 4) {
      st_r4[threadIdx.x] = reinterpret_cast<const float4*>(rope_cos + (int64_t)c * H)[threadIdx.x];
      st_r4[H / 4 + threadIdx.x] =
          reinterpret_cast<const float4*>(rope_sin + (int64_t)c * H)[threadIdx.x];
    }
    __syncthreads();

    // value inputs of this thread's pieces (token u, channels [j0, j0 + 8)); with
    // four tokens a thread requested after the key work (fewer live registers
    // during the key jobs)
    constexpr int VP = D / 8;              // pieces per token row
    constexpr int VPT = WT * VP / 256;     // pieces per thread
    uint32_t vw[VPT][2];
    float vsc[VPT], vzr[VPT];
    auto load_values = [&]() {
#pragma unroll
      for (int k = 0; k < VPT; ++k) {
        const int vj = threadIdx.x + 256 * k;
        const int u = u_base + vj / VP, j0 = (vj % VP) * 8;
        const int64_t srow = slab * kC + u;
        vsc[k] = v_scale[srow * ngv + j0 / Gv];
        vzr[k] = v_zero[srow * ngv + j0 / Gv];
        const uint8_t* row = v_codes + srow * CB;
        if constexpr (BITS == 8) {
          const uint2 a = *reinterpret_cast<const uint2*>(row + j0);
          vw[k][0] = a.x;
          vw[k][1] = a.y;
        } else {
          vw[k][0] = *reinterpret_cast<const uint32_t*>(row + j0 / 2);
          vw[k][1] = 0;
        }
      }
    };
    if constexpr (TOK == 1) load_values();

    for (int job = threadIdx.x; job < KJOBS; job += blockDim.x) {
      {
        // ---- keys: TOK tokens from u0, channel pairs [8cg, 8cg + 8)
        const int q = job / TPT, cg = job % TPT;
        const int u0 = u_base + TOK * q, j0 = 8 * cg;
        const int g = u0 / Gk;
        // statistics and rotation row of the job's channels, kept as float
        // (half the registers of double) and widened exactly at use: read from
        // LDS for every token (so they are not live while the loads are in flight)
        float s_lo[8], s_hi[8], z_lo[8], z_hi[8], cs[8], sn[8];
        auto load_stats = [&]() {
          const float* sc = reinterpret_cast<const float*>(st_k4) + (g - g_base) * D;
          const float* zr = reinterpret_cast<const float*>(st_k4) + (n_gs + g - g_base) * D;
          const float* rc = reinterpret_cast<const float*>(st_r4);
          const float* rs = reinterpret_cast<const float*>(st_r4) + H;
#pragma unroll
          for (int k = 0; k < 8; k += 4) {
            const float4 a = *reinterpret_cast<const float4*>(sc + j0 + k);
            const float4 b = *reinterpret_cast<const float4*>(sc + H + j0 + k);
            const float4 e = *reinterpret_cast<const float4*>(zr + j0 + k);
            const float4 f = *reinterpret_cast<const float4*>(zr + H + j0 + k);
            const float4 cc = *reinterpret_cast<const float4*>(rc + j0 + k);
            const float4 ss = *reinterpret_cast<const float4*>(rs + j0 + k);
            s_lo[k] = a.x; s_lo[k + 1] = a.y; s_lo[k + 2] = a.z; s_lo[k + 3] = a.w;
            s_hi[k] = b.x; s_hi[k + 1] = b.y; s_hi[k + 2] = b.z; s_hi[k + 3] = b.w;
            z_lo[k] = e.x; z_lo[k + 1] = e.y; z_lo[k + 2] = e.z; z_lo[k + 3] = e.w;
            z_hi[k] = f.x; z_hi[k + 1] = f.y; z_hi[k + 2] = f.z; z_hi[k + 3] = f.w;
            cs[k] = cc.x; cs[k + 1] = cc.y; cs[k + 2] = cc.z; cs[k + 3] = cc.w;
            sn[k] = ss.x; sn[k + 1] = ss.y; sn[k + 2] = ss.z; sn[k + 3] = ss.w;
          }
        };
        // the codes of the job's tokens and their fresh key pieces are all requested
        // before any is used: one memory round trip per job
        uint32_t cwl[TOK][2], cwh[TOK][2];
        uint4 fra[TOK], frb[TOK];
#pragma unroll
        for (int i = 0; i < TOK; ++i) {
          const uint8_t* row = k_codes + (slab * kC + u0 + i) * CB;
          if constexpr (BITS == 8) {
            const uint2 a = *reinterpret_cast<const uint2*>(row + j0);
            const uint2 b = *reinterpret_cast<const uint2*>(row + H + j0);
            cwl[i][0] = a.x; cwl[i][1] = a.y; cwh[i][0] = b.x; cwh[i][1] = b.y;
          } else {
            cwl[i][0] = *reinterpret_cast<const uint32_t*>(row + j0 / 2);
            cwh[i][0] = *reinterpret_cast<const uint32_t*>(row + (H + j0) / 2);
            cwl[i][1] = cwh[i][1] = 0;
          }
          const uint16_t* fr = k_fresh + (out_row0 + u0 + i) * D;
          fra[i] = *reinterpret_cast<const uint4*>(fr + j0);
          frb[i] = *reinterpret_cast<const uint4*>(fr + H + j0);
        }
#pragma unroll
        for (int i = 0; i < TOK; ++i) {
          const int u = u0 + i;
          asm volatile("" ::: "memory");  // re-read the staged values for every token
          load_stats();
          const uint32_t wl[2] = {cwl[i][0], cwl[i][1]}, wh[2] = {cwh[i][0], cwh[i][1]};
          float ylo[8], yhi[8];
#pragma unroll
          for (int k = 0; k < 8; ++k) {
            const double xl = __builtin_fma((double)code_at<BITS>(wl, k), (double)s_lo[k], (double)z_lo[k]);
            const double xh = __builtin_fma((double)code_at<BITS>(wh, k), (double)s_hi[k], (double)z_hi[k]);
            const double a = xl * (double)cs[k];
            const double b = xh * (double)sn[k];
            const double e = xh * (double)cs[k];
            const double f = xl * (double)sn[k];
            ylo[k] = (float)(a - b);
            yhi[k] = (float)(e + f);
          }
          const int64_t o = (out_row0 + u) * D;
          uint16_t* ko = k_out + o;
          uint4 A, B;
          A.x = pack_bf16x2(ylo[0], ylo[1]); A.y = pack_bf16x2(ylo[2], ylo[3]);
          A.z = pack_bf16x2(ylo[4], ylo[5]); A.w = pack_bf16x2(ylo[6], ylo[7]);
          B.x = pack_bf16x2(yhi[0], yhi[1]); B.y = pack_bf16x2(yhi[2], yhi[3]);
          B.z = pack_bf16x2(yhi[4], yhi[5]); B.w = pack_bf16x2(yhi[6], yhi[7]);
          *reinterpret_cast<uint4*>(ko + j0) = A;
          *reinterpret_cast<uint4*>(ko + H + j0) = B;
          const uint4 FA = fra[i], FB = frb[i];
          const uint32_t cw[8] = {A.x, A.y, A.z, A.w, B.x, B.y, B.z, B.w};
          const uint32_t fw[8] = {FA.x, FA.y, FA.z, FA.w, FB.x, FB.y, FB.z, FB.w};
          double dot = 0.0, na = 0.0, nb = 0.0;
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const double a0 = bf16_lo(cw[e]), a1 = bf16_hi(cw[e]);
            const double b0 = bf16_lo(fw[e]), b1 = bf16_hi(fw[e]);
            dot = __builtin_fma(a0, b0, dot);
            dot = __builtin_fma(a1, b1, dot);
            na = __builtin_fma(a0, a0, na);
            na = __builtin_fma(a1, a1, na);
            nb = __builtin_fma(b0, b0, nb);
            nb = __builtin_fma(b1, b1, nb);
          }
          dot = quad_lanes_sum<TPT>(dot);
          na = quad_lanes_sum<TPT>(na);
          nb = quad_lanes_sum<TPT>(nb);
          const double den = na * nb;
          cos_sum[i] += (den == 0.0) ? ((na == 0.0 && nb == 0.0) ? 1.0 : 0.0) : dot / sqrt(den);
        }
      }
    }

    // ---- values
    if constexpr (TOK != 1) load_values();
#pragma unroll
    for (int k = 0; k < VPT; ++k) {
      const int vj = threadIdx.x + 256 * k;
      const int u = u_base + vj / VP, j0 = (vj % VP) * 8;
      const double sc = vsc[k], zr = vzr[k];
      float y[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) y[e] = (float)__builtin_fma((double)code_at<BITS>(vw[k], e), sc, zr);
      const int64_t o = (out_row0 + u) * D + j0;
      *reinterpret_cast<uint4*>(v_out + o) =
          make_uint4(pack_bf16x2(y[0], y[1]), pack_bf16x2(y[2], y[3]), pack_bf16x2(y[4], y[5]),
                     pack_bf16x2(y[6], y[7]));
    }
  }  // heads
  // one lane per job: delta[l][dst_row + u0 ..], for four tokens one 16-byte
  // store when they are 16-byte aligned (dst_row and t_total multiples of 4),
  // else 4-byte stores (e.g. after one to three sink rows)
  const int job = threadIdx.x;
  if (job < KJOBS && job % TPT == 0) {
    const int u0 = u_base + TOK * (job / TPT);
    const double n = (double)Hkv;
    const int64_t first = (int64_t)blockIdx.y * t_total + ch.dst_row;
    float* dp = delta + first + u0;
    float dv[TOK];
#pragma unroll
    for (int i = 0; i < TOK; ++i) dv[i] = (float)(1.0 - cos_sum[i] / n);
    if (TOK == 4 && (first & 3) == 0) {
      *reinterpret_cast<float4*>(dp) = make_float4(dv[0], dv[TOK / 4], dv[TOK / 2], dv[TOK - 1]);
    } else {
#pragma unroll
      for (int i = 0; i < TOK; ++i) dp[i] = dv[i];
    }
  }
}

// A workgroup takes a whole chunk (four tokens a thread, the statistics loaded
// once for them) when the grid has enough of them; otherwise a thread takes one
// token and the chunk is split over 4 (d = 128) or 2 workgroups: a launch of a
// few chunks is bound by one workgroup's chain of loads and double arithmetic,
// which is then a quarter as long.  Measured, one token against four a thread:
// fused, 36 chunk-layers 6.2 against 13.0 us, 252 14.8 / 17.7, 1152 61.8 / 65.1,
// 2304 119 / 116; plain, 2 chunk-heads 3.2 / 4.6 us, 96 4.7 / 5.5, 240 8.0 / 7.5,
// 2304 56 / 47 (its statistics are loaded per token then).
constexpr int64_t kSplitFused = 1536, kSplitPlain = 128;
unsigned token_splits(int head_dim) { return head_dim == 128 ? 4 : 2; }

}  // namespace

hipError_t launch_stitch(const kvb_pool_layout& p, int32_t n_pool, const uint8_t* k_codes,
                         const float* k_scale, const float* k_zero, const uint8_t* v_codes,
                         const float* v_scale, const float* v_zero, const kvb_chunk* chunks,
                         int32_t n_chunks, const float* rope_cos, const float* rope_sin,
                         int64_t t_total, kvb_dtype out_dtype, void* k_cache, void* v_cache,
                         hipStream_t s) {
  const bool split = (int64_t)n_chunks * p.n_layers * p.n_kv_heads < kSplitPlain;
  const dim3 grid(n_chunks, p.n_layers * p.n_kv_heads, split ? token_splits(p.head_dim) : 1);
  const dim3 block(256);
  const bool bf = out_dtype == KVB_BF16;
#define KVB_STITCH_T(B, D, F, T)                                                                  \
  hipLaunchKernelGGL((stitch_kernel<B, D, F, T>), grid, block, 0, s, p.n_layers,          \
                     p.n_kv_heads, p.k_group, p.v_group, n_pool, k_codes, k_scale, k_zero,       \
                     v_codes, v_scale, v_zero, chunks, rope_cos, rope_sin, t_total, k_cache,     \
                     v_cache)
#define KVB_STITCH(B, D, F)      \
  do {                           \
    if (split)                   \
      KVB_STITCH_T(B, D, F, 1);  \
    else                         \
      KVB_STITCH_T(B, D, F, 4);  \
  } while (0)
  if (p.bits == 8) {
    if (p.head_dim == 128) { if (bf) KVB_STITCH(8, 128, true); else KVB_STITCH(8, 128, false); }
    else { if (bf) KVB_STITCH(8, 64, true); else KVB_STITCH(8, 64, false); }
  } else {
    if (p.head_dim == 128) { if (bf) KVB_STITCH(4, 128, true); else KVB_STITCH(4, 128, false); }
    else { if (bf) KVB_STITCH(4, 64, true); else KVB_STITCH(4, 64, false); }
  }
#undef KVB_STITCH
#undef KVB_STITCH_T
  return hipGetLastError();
}

hipError_t launch_stitch_deviation(const kvb_pool_layout& p, int32_t n_pool,
                                   const uint8_t* k_codes, const float* k_scale,
                                   const float* k_zero, const uint8_t* v_codes,
                                   const float* v_scale, const float* v_zero,
                                   const kvb_chunk* chunks, int32_t n_chunks,
                                   const float* rope_cos, const float* rope_sin, int64_t t_total,
                                   void* k_cache, void* v_cache, const uint16_t* k_fresh,
                                   float* delta, hipStream_t s) {
  const bool split = (int64_t)n_chunks * p.n_layers < kSplitFused;
  const dim3 grid(n_chunks, p.n_layers, split ? token_splits(p.head_dim) : 1), block(256);
#define KVB_STITCH_DEV_T(B, D, T)                                                                 \
  hipLaunchKernelGGL((stitch_deviation_kernel<B, D, T>), grid, block, 0, s, p.n_layers,        \
                     p.n_kv_heads, p.k_group, p.v_group, n_pool, k_codes, k_scale, k_zero,       \
                     v_codes, v_scale, v_zero, chunks, rope_cos, rope_sin, t_total,              \
                     (uint16_t*)k_cache, (uint16_t*)v_cache, k_fresh, delta)
#define KVB_STITCH_DEV(B, D)      \
  do {                            \
    if (split)                    \
      KVB_STITCH_DEV_T(B, D, 1);  \
    else                          \
      KVB_STITCH_DEV_T(B, D, 4);  \
  } while (0)
  if (p.bits == 8) {
    if (p.head_dim == 128) KVB_STITCH_DEV(8, 128); else KVB_STITCH_DEV(8, 64);
  } else {
    if (p.head_dim == 128) KVB_STITCH_DEV(4, 128); else KVB_STITCH_DEV(4, 64);
  }
#undef KVB_STITCH_DEV
#undef KVB_STITCH_DEV_T
  return hipGetLastError();
}

}  // namespace kvb
