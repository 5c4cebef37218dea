// Cache population kernels: RoPE at absolute positions (Eq. 3), KIVI
// quantisation of cached chunks (Sec. 4.5, Eq. 7) and the chunks' importance
// for the eviction order (Sec. 4.4).  These prepare the chunk pool and the
// probe-pass tensors: every chunk a request did not find goes through them.
#include <math.h>

#include "kvb_device.h"
#include "kvb_internal.h"

namespace kvb {
namespace {

// One thread per (vector, group of 4 channel pairs).  Double arithmetic:
// y_lo = x_lo*c - x_hi*s, y_hi = x_hi*c + x_lo*s (contraction is off for this
// file, so each product and sum rounds once).
template <int D, int OUT>
__global__ void __launch_bounds__(256)
rope_rows_kernel(int64_t n_outer, int64_t n_rows, int64_t n_inner, const float* __restrict__ x,
                 const int32_t* __restrict__ row_pos, const int32_t* __restrict__ outer_pos,
                 const float* __restrict__ tcos, const float* __restrict__ tsin, int32_t table_len,
                 void* __restrict__ out) {
  constexpr int H = D / 2;
  constexpr int G = H / 4;  // threads per vector
  const int64_t n_vec = n_outer * n_rows * n_inner;
  for (int64_t w = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; w < n_vec * G;
       w += (int64_t)gridDim.x * blockDim.x) {
    const int64_t v = w / G;
    const int i0 = (int)(w % G) * 4;
    const int64_t r = (v / n_inner) % n_rows;
    const int64_t o = v / (n_inner * n_rows);
    const float4 lo = *reinterpret_cast<const float4*>(x + v * D + i0);
    const float4 hi = *reinterpret_cast<const float4*>(x + v * D + H + i0);
    double xl[4] = {lo.x, lo.y, lo.z, lo.w};
    double xh[4] = {hi.x, hi.y, hi.z, hi.w};
    double yl[4], yh[4];
    if (tcos != nullptr) {
      const int64_t p = (int64_t)row_pos[r] + (outer_pos ? (int64_t)outer_pos[o] : 0);
      if (p < 0 || p >= table_len) {
        for (int k = 0; k < 4; ++k) yl[k] = yh[k] = __builtin_nan("");
      } else {
        const float4 c4 = *reinterpret_cast<const float4*>(tcos + p * H + i0);
        const float4 s4 = *reinterpret_cast<const float4*>(tsin + p * H + i0);
        const double c[4] = {c4.x, c4.y, c4.z, c4.w};
        const double s[4] = {s4.x, s4.y, s4.z, s4.w};
        for (int k = 0; k < 4; ++k) {
          yl[k] = xl[k] * c[k] - xh[k] * s[k];
          yh[k] = xh[k] * c[k] + xl[k] * s[k];
        }
      }
    } else {
      for (int k = 0; k < 4; ++k) { yl[k] = xl[k]; yh[k] = xh[k]; }
    }
    if constexpr (OUT == KVB_F64) {
      double* o64 = reinterpret_cast<double*>(out) + v * D;
      *reinterpret_cast<double2*>(o64 + i0) = make_double2(yl[0], yl[1]);
      *reinterpret_cast<double2*>(o64 + i0 + 2) = make_double2(yl[2], yl[3]);
      *reinterpret_cast<double2*>(o64 + H + i0) = make_double2(yh[0], yh[1]);
      *reinterpret_cast<double2*>(o64 + H + i0 + 2) = make_double2(yh[2], yh[3]);
    } else if constexpr (OUT == KVB_F32) {
      float* o32 = reinterpret_cast<float*>(out) + v * D;
      *reinterpret_cast<float4*>(o32 + i0) =
          make_float4((float)yl[0], (float)yl[1], (float)yl[2], (float)yl[3]);
      *reinterpret_cast<float4*>(o32 + H + i0) =
          make_float4((float)yh[0], (float)yh[1], (float)yh[2], (float)yh[3]);
    } else {
      uint16_t* o16 = reinterpret_cast<uint16_t*>(out) + v * D;
      uint2 a, b;
      a.x = pack_bf16x2((float)yl[0], (float)yl[1]);
      a.y = pack_bf16x2((float)yl[2], (float)yl[3]);
      b.x = pack_bf16x2((float)yh[0], (float)yh[1]);
      b.y = pack_bf16x2((float)yh[2], (float)yh[3]);
      *reinterpret_cast<uint2*>(o16 + i0) = a;
      *reinterpret_cast<uint2*>(o16 + H + i0) = b;
    }
  }
}

// Code of x in a group with minimum mn and range r:
//   c = clamp(rint(((x - mn) / r) * levels), 0, levels), 0 for a constant group.
// The double division is replaced by a product with k = (1 / r) * levels wherever
// that cannot change c: both forms carry at most three roundings of a value of at
// most `levels` (255), so they differ by less than 1e-12, and rint can only tell
// them apart within that distance of a half.  A value closer than 1e-9 to a half,
// or not a number, is `unsure` and takes the division (slow_code); so does a range
// whose reciprocal leaves the normal numbers (k = NaN: every value is unsure).
// Adding 1.5 * 2^52 rounds to the nearest integer, ties to even, as rint does, and
// leaves it in the low word; a sure value lies in [0, levels] as it is.
__device__ __forceinline__ uint32_t sure_code(double x, double mn, double k, bool& unsure) {
  constexpr double shift = 6755399441055744.0;
  const double t = (x - mn) * k, u = t + shift;
  unsure |= !(fabs(t - (u - shift)) < 0.5 - 1e-9);
  return (uint32_t)__builtin_bit_cast(uint64_t, u);
}
__device__ __forceinline__ uint32_t slow_code(double x, double mn, double r, double levels) {
  const double t = r != 0.0 ? ((x - mn) / r) * levels : 0.0;
  return (uint32_t)fmin(fmax(rint(t), 0.0), levels);
}
// k of a range (1 / 0 and the like included: NaN)
__device__ __forceinline__ double code_factor(double r, double levels) {
  return r > 1e-290 && r < 1e290 ? (1.0 / r) * levels : __builtin_nan("");
}

// N consecutive elements at p (16-byte aligned for N * sizeof(T) >= 16)
template <typename T, int N>
__device__ __forceinline__ void load_n(const T* p, T (&x)[N]) {
  typedef __attribute__((ext_vector_type(N * sizeof(T) >= 16 ? 16 / (int)sizeof(T) : N))) T V;
  constexpr int E = sizeof(V) / sizeof(T);
#pragma unroll
  for (int i = 0; i < N / E; ++i) {
    const V v = reinterpret_cast<const V*>(p)[i];
#pragma unroll
    for (int e = 0; e < E; ++e) x[i * E + e] = v[e];
  }
}

// Keys: one workgroup of 2 D threads per (slot, layer, head) slab; a thread
// owns one channel pair of 32 consecutive tokens, so a row is read by adjacent
// lanes, and holds them in registers: the input is read once, every load in
// flight together.  HBM-bound on the input.  Groups of 64 or 128 tokens meet
// through LDS; smaller ones (SMALL) are found among the thread's own quads.
// (One thread per group and channel pair, reading the group twice, divided
// every value: 12 int4 chunks x 36 layers of fp64 keys, 113 MB, took 45 us; this
// takes 21 us, 5.3 TB/s of input, 23 while each code was clamped, converted and
// branched on by itself.)
template <typename T, int D, int BITS, bool SMALL>
__global__ void __launch_bounds__(2 * D)
quant_keys_kernel(int64_t n_slabs, int32_t L, int32_t first_layer, int32_t n_in, int32_t Hkv,
                  int32_t Gk, const T* __restrict__ in, uint8_t* __restrict__ codes,
                  float* __restrict__ scale, float* __restrict__ zero) {
  constexpr int C = 128, TT = 32, NQ = TT / 4;  // tokens per chunk and thread, quads per thread
  constexpr int CB = D * BITS / 8;
  constexpr double levels = (double)((1 << BITS) - 1);
  __shared__ double2 part[SMALL ? 1 : C / TT][SMALL ? 1 : 2][SMALL ? 1 : D / 2];
  const int pr = threadIdx.x % (D / 2), tg = threadIdx.x / (D / 2);
  const int j0 = 2 * pr, u0 = tg * TT;
  const int n_groups = C / Gk;
  for (int64_t s = blockIdx.x; s < n_slabs; s += gridDim.x) {  // (p, layer of the input, h)
    const int64_t pl = s / Hkv;
    const int64_t slab =
        ((pl / n_in) * L + first_layer + pl % n_in) * Hkv + s % Hkv;  // (p, pool layer, h)
    const T* src = in + (s * C + u0) * D + j0;
    T x[TT][2];
#pragma unroll
    for (int u = 0; u < TT; ++u) load_n<T, 2>(src + u * D, x[u]);
    double mn[SMALL ? NQ : 1][2], mx[SMALL ? NQ : 1][2];
#pragma unroll
    for (int q = 0; q < (SMALL ? NQ : 1); ++q)
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        double lo = INFINITY, hi = -INFINITY;
#pragma unroll
        for (int u = 0; u < (SMALL ? 4 : TT); ++u) {
          lo = fmin(lo, (double)x[4 * q + u][e]);
          hi = fmax(hi, (double)x[4 * q + u][e]);
        }
        mn[q][e] = lo;
        mx[q][e] = hi;
      }
    if constexpr (SMALL) {  // groups of 4, 8 or 16 tokens: merge the quads of a group
#pragma unroll
      for (int w = 1; w < NQ / 2; w <<= 1) {
        if (Gk >= 8 * w) {
#pragma unroll
          for (int q = 0; q < NQ; q += 2 * w)
#pragma unroll
            for (int e = 0; e < 2; ++e) {
              const double lo = fmin(mn[q][e], mn[q + w][e]), hi = fmax(mx[q][e], mx[q + w][e]);
#pragma unroll
              for (int k = 0; k < 2 * w; ++k) {
                mn[q + k][e] = lo;
                mx[q + k][e] = hi;
              }
            }
        }
      }
    } else if (Gk > TT) {
      __syncthreads();  // the previous slab's reads are done
      part[tg][0][pr] = make_double2(mn[0][0], mn[0][1]);
      part[tg][1][pr] = make_double2(mx[0][0], mx[0][1]);
      __syncthreads();
      const int n = Gk / TT, first = tg / n * n;
      for (int k = first; k < first + n; ++k) {
        const double2 lo = part[k][0][pr], hi = part[k][1][pr];
        mn[0][0] = fmin(mn[0][0], lo.x);
        mn[0][1] = fmin(mn[0][1], lo.y);
        mx[0][0] = fmax(mx[0][0], hi.x);
        mx[0][1] = fmax(mx[0][1], hi.y);
      }
    }
    double k[2], r[2];
#pragma unroll
    for (int u = 0; u < TT; ++u) {
      const int q = SMALL ? u / 4 : 0;
      if (u % (SMALL ? 4 : TT) == 0) {
        const bool first = (u0 + u) % Gk == 0;  // this thread starts the group
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          r[e] = mx[q][e] - mn[q][e];
          k[e] = code_factor(r[e], levels);
        }
        if (first) {
          const int64_t st = (slab * n_groups + (u0 + u) / Gk) * D + j0;
          *reinterpret_cast<float2*>(scale + st) =
              make_float2(r[0] == 0.0 ? 0.0f : (float)(r[0] / levels),
                          r[1] == 0.0 ? 0.0f : (float)(r[1] / levels));
          *reinterpret_cast<float2*>(zero + st) = make_float2((float)mn[q][0], (float)mn[q][1]);
        }
      }
      bool unsure = false;
      uint32_t c0 = sure_code((double)x[u][0], mn[q][0], k[0], unsure);
      uint32_t c1 = sure_code((double)x[u][1], mn[q][1], k[1], unsure);
      if (__builtin_expect(unsure, 0)) {
        c0 = slow_code((double)x[u][0], mn[q][0], r[0], levels);
        c1 = slow_code((double)x[u][1], mn[q][1], r[1], levels);
      }
      uint8_t* row = codes + (slab * C + u0 + u) * CB;
      if constexpr (BITS == 8)
        *reinterpret_cast<uint16_t*>(row + j0) = (uint16_t)(c0 | (c1 << 8));
      else
        row[j0 / 2] = (uint8_t)(c0 | (c1 << 4));
    }
  }
}

// Values: a thread owns 8 consecutive channels of one token (one code word),
// so the D / 8 lanes of a token read whole rows; the Gv / 8 lanes of a group
// (a power of two: Gv is 16, 32, 64 or 128) meet with xor-shuffles.  HBM-bound
// on the input.  (One thread per group, reading its Gv values one by one and
// twice with its neighbours Gv elements away, took 379 us for 12 int4 chunks x
// 36 layers of fp64 values, 113 MB; this takes 23 us, 4.9 TB/s of input.)
template <typename T, int D, int BITS>
__global__ void __launch_bounds__(256)
quant_values_kernel(int64_t n_slabs, int32_t L, int32_t first_layer, int32_t n_in, int32_t Hkv,
                    int32_t Gv, const T* __restrict__ in, uint8_t* __restrict__ codes,
                    float* __restrict__ scale, float* __restrict__ zero) {
  constexpr int C = 128, LPT = D / 8;  // lanes per token
  constexpr int CB = D * BITS / 8;
  constexpr double levels = (double)((1 << BITS) - 1);
  const int n_groups = D / Gv;
  const int j0 = (threadIdx.x % LPT) * 8;
  // a workgroup steps over whole token groups of one slab: every lane of a
  // token's group is active, and the slab's indices are found once for all of them
  constexpr int TW = 256 / LPT, PER = C / TW;  // tokens per workgroup, steps per slab
  for (int64_t step = blockIdx.x; step < n_slabs * PER; step += gridDim.x) {
    const int64_t s = step / PER;  // (p, layer of the input, h)
    const int64_t pl = s / Hkv;
    const int u = (int)(step % PER) * TW + (int)threadIdx.x / LPT;
    const int64_t row = s * C + u;
    const int64_t out_row =
        (((pl / n_in) * L + first_layer + pl % n_in) * Hkv + s % Hkv) * C + u;
    T x[8];
    load_n<T, 8>(in + row * D + j0, x);
    double mn = INFINITY, mx = -INFINITY;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      mn = fmin(mn, (double)x[e]);
      mx = fmax(mx, (double)x[e]);
    }
    for (int m = 1; m < Gv / 8; m <<= 1) {
      mn = fmin(mn, __shfl_xor(mn, m, 64));
      mx = fmax(mx, __shfl_xor(mx, m, 64));
    }
    const double r = mx - mn, k = code_factor(r, levels);
    uint32_t c[8];
    bool unsure = false;
#pragma unroll
    for (int e = 0; e < 8; ++e) c[e] = sure_code((double)x[e], mn, k, unsure);
    if (__builtin_expect(unsure, 0)) {
#pragma unroll
      for (int e = 0; e < 8; ++e) c[e] = slow_code((double)x[e], mn, r, levels);
    }
    uint32_t w[BITS == 8 ? 2 : 1] = {};
#pragma unroll
    for (int e = 0; e < 8; ++e) w[e * BITS / 32] |= c[e] << (e * BITS % 32);
    uint8_t* dst = codes + out_row * CB + j0 * BITS / 8;
    if constexpr (BITS == 8)
      *reinterpret_cast<uint2*>(dst) = make_uint2(w[0], w[1]);
    else
      *reinterpret_cast<uint32_t*>(dst) = w[0];
    if (j0 % Gv == 0) {
      const int64_t st = out_row * n_groups + j0 / Gv;
      scale[st] = r == 0.0 ? 0.0f : (float)(r / levels);
      zero[st] = (float)mn;
    }
  }
}

int grid_for(int64_t work) {
  int64_t b = (work + 255) / 256;
  if (b > 65536) b = 65536;
  return (int)(b < 1 ? 1 : b);
}

}  // namespace

hipError_t launch_rope_rows(int head_dim, int64_t n_outer, int64_t n_rows, int64_t n_inner,
                            const float* x, const int32_t* row_pos, const int32_t* outer_pos,
                            const float* tcos, const float* tsin, int32_t table_len,
                            kvb_dtype out_dtype, void* out, hipStream_t s) {
  const int64_t work = n_outer * n_rows * n_inner * (head_dim / 8);
  const dim3 grid(grid_for(work)), block(256);
#define KVB_ROPE(D, O)                                                                     \
  hipLaunchKernelGGL((rope_rows_kernel<D, O>), grid, block, 0, s, n_outer, n_rows, n_inner, \
                     x, row_pos, outer_pos, tcos, tsin, table_len, out)
  if (head_dim == 64) {
    if (out_dtype == KVB_F64) KVB_ROPE(64, KVB_F64);
    else if (out_dtype == KVB_F32) KVB_ROPE(64, KVB_F32);
    else KVB_ROPE(64, KVB_BF16);
  } else {
    if (out_dtype == KVB_F64) KVB_ROPE(128, KVB_F64);
    else if (out_dtype == KVB_F32) KVB_ROPE(128, KVB_F32);
    else KVB_ROPE(128, KVB_BF16);
  }
#undef KVB_ROPE
  return hipGetLastError();
}

// Chunk importance (Sec. 4.4): workgroups of 1024 lanes, each over a slice of a
// chunk's vectors; a chunk is dealt to up to kImpSplit of them (imp_split), and the
// last one to finish adds the slices' sums (imp_finish).  12 chunks x 36 layers of
// fp64 keys (113 MB): one workgroup a chunk 96 us, eight 24.  Each key
// vector is read by 8 adjacent lanes: 16-byte piece i of the vector goes to
// lane i % 8, so every load instruction of a wave reads 8 whole 128-byte
// segments (8 vectors).  All of a lane's pieces are requested before any is
// summed; a lane sums its squares in piece order (double), the 8 lanes combine
// theirs with a fixed xor tree (every level adds two values, so all 8 end with
// the same bits), and one of them, another for each vector, adds the norm to its
// running sum: the square root and the addition run once for eight vectors of a
// group.  From there on every sum keeps its rounding errors (SumDD) and the chunk's
// is rounded once at the end, so that it is the same however the chunk was dealt
// (but for a sum within some 2^-40 of a last place of the middle of two doubles).
constexpr int kImpLanes = 8;  // lanes per key vector

// Meeting place of a chunk's workgroups.  The call has no workspace, so it is a
// static device array, safe for any streams and threads: a slot belongs to one
// dispatch (its packet's address, which a queue uses again only after a round of
// its whole ring) from its chunk's first finished workgroup to its last, which
// clears it.  Every workgroup of the dispatch arrives exactly once, so no call,
// whatever it overlaps with or adds to, leaves a slot taken or finds one of
// another's.  A chunk's workgroups look only at the 64 slots of its index in the launch (one a
// lane), so slots run out only if 64 dispatches hold one at once; an arrival then
// waits for one of them to end.  That wait ends: all of them but those that are
// still being dispatched (at most one per hardware queue, of which a process has
// at most 32) have every workgroup on the chip, and none of these waits.
constexpr int kImpSplit = 16;    // most workgroups per chunk
constexpr int kImpMaxWg = 256;   // most workgroups of a launch that splits chunks
constexpr int kImpMaxChunks = kImpMaxWg / 2;  // most chunks that it has
struct ImpSlot {
  unsigned long long key;  // address of the dispatch packet, 0 = free
  unsigned int arrived;    // finished workgroups
  unsigned int pad;
  double part[kImpSplit][2];  // a slice's sum and its rounding errors
};
static __device__ ImpSlot imp_slots[kImpMaxChunks][64];
static __device__ unsigned int imp_locks[kImpMaxChunks];

#define KVB_AGENT __HIP_MEMORY_SCOPE_AGENT

// Slot of `key` among the 64 of chunk index p, taken if there is none yet.  Wave
// uniform.  A slot found belongs to the caller's chunk until the caller has
// arrived.  Slots are taken under the index's lock, so that a key is never given
// two; its holder waits for nothing, so every wait on it ends.
__device__ __forceinline__ ImpSlot* imp_slot(int p, unsigned long long key) {
  ImpSlot* const row = imp_slots[p];
  const int lane = threadIdx.x & 63;
  auto look = [&](unsigned long long what) {
    return __builtin_amdgcn_ballot_w64(
        __hip_atomic_load(&row[lane].key, __ATOMIC_ACQUIRE, KVB_AGENT) == what);
  };
  uint64_t hit = look(key);
  while (hit == 0) {
    unsigned int held = 1;
    if (lane == 0) held = __hip_atomic_exchange(&imp_locks[p], 1u, __ATOMIC_ACQUIRE, KVB_AGENT);
    if (__builtin_amdgcn_readfirstlane(held) == 0) {
      hit = look(key);
      if (hit == 0 && (hit = look(0ull)) != 0 && lane == __ffsll((unsigned long long)hit) - 1)
        __hip_atomic_store(&row[lane].key, key, __ATOMIC_RELAXED, KVB_AGENT);
      if (lane == 0) __hip_atomic_store(&imp_locks[p], 0u, __ATOMIC_RELEASE, KVB_AGENT);
    } else {
      __builtin_amdgcn_s_sleep(2);
      hit = look(key);
    }
  }
  return row + (__ffsll((unsigned long long)hit) - 1);
}

// x of the lane that a DPP control names (a vector move, no LDS round trip)
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double x) {
  const uint64_t w = __builtin_bit_cast(uint64_t, x);
  const uint32_t lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)w, CTRL, 0xF, 0xF, false);
  const uint32_t hi = __builtin_amdgcn_update_dpp(0, (int)(w >> 32), CTRL, 0xF, 0xF, false);
  return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}

// Sum of doubles that keeps the rounding errors of its additions (two-sum): about
// 2^-104 relative, whatever the order.
struct SumDD {
  double s = 0.0, c = 0.0;
  __device__ __forceinline__ void add(double x, double xc = 0.0) {
    const double t = s + x, y = t - s;
    c = (c + xc) + ((s - (t - y)) + (x - y));
    s = t;
  }
  // sum over N adjacent lanes (16 or 64) by a fixed tree; each ends with the same
  // bits.  Every lane must call.
  template <int N>
  __device__ __forceinline__ void add_lanes() {
    add(dpp_f64<0xB1>(s), dpp_f64<0xB1>(c));    // quad_perm [1, 0, 3, 2]
    add(dpp_f64<0x4E>(s), dpp_f64<0x4E>(c));    // quad_perm [2, 3, 0, 1]
    add(dpp_f64<0x141>(s), dpp_f64<0x141>(c));  // row_half_mirror: the other quad of 8 lanes
    add(dpp_f64<0x140>(s), dpp_f64<0x140>(c));  // row_mirror: the other 8 of 16
#pragma unroll
    for (int m = 16; m < N; m <<= 1) {
      const double x = __shfl_xor(s, m, 64), xc = __shfl_xor(c, m, 64);
      add(x, xc);
    }
  }
  // an infinite or NaN sum has no error term
  __device__ __forceinline__ double value() const { return isfinite(c) ? s + c : s; }
};

// Leaves this slice's sum in its chunk's slot.  True, with the chunk's sum, for the
// chunk's last workgroup (both in the first kImpSplit lanes).  Called by one whole wave.
__device__ __forceinline__ bool imp_finish(int p, int slice, int n_slices, SumDD* sum) {
  const int lane = threadIdx.x & 63;
  ImpSlot* const slot =
      imp_slot(p, (unsigned long long)(uintptr_t)__builtin_amdgcn_dispatch_ptr());
  unsigned int before = 0;
  if (lane == 0) {
    __hip_atomic_store(&slot->part[slice][0], sum->s, __ATOMIC_RELAXED, KVB_AGENT);
    __hip_atomic_store(&slot->part[slice][1], sum->c, __ATOMIC_RELAXED, KVB_AGENT);
    before = __hip_atomic_fetch_add(&slot->arrived, 1u, __ATOMIC_ACQ_REL, KVB_AGENT);
  }
  if (__builtin_amdgcn_readfirstlane(before) + 1 < (unsigned)n_slices) return false;
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
  *sum = SumDD();
  if (lane < n_slices)
    sum->add(__hip_atomic_load(&slot->part[lane][0], __ATOMIC_RELAXED, KVB_AGENT),
             __hip_atomic_load(&slot->part[lane][1], __ATOMIC_RELAXED, KVB_AGENT));
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");  // every lane's loads before the slot is free
  __builtin_amdgcn_wave_barrier();
  if (lane == 0) {
    __hip_atomic_store(&slot->arrived, 0u, __ATOMIC_RELAXED, KVB_AGENT);
    __hip_atomic_store(&slot->key, 0ull, __ATOMIC_RELEASE, KVB_AGENT);
  }
  sum->add_lanes<kImpSplit>();
  return true;
}

template <typename T>
__device__ __forceinline__ double sum_sq_piece(const T* p) {  // one 16-byte piece
  if constexpr (sizeof(T) == 8) {
    const double2 a = *reinterpret_cast<const double2*>(p);
    return __builtin_fma(a.y, a.y, a.x * a.x);
  } else {
    const float4 a = *reinterpret_cast<const float4*>(p);
    const double x0 = a.x, x1 = a.y, x2 = a.z, x3 = a.w;
    return __builtin_fma(x3, x3, __builtin_fma(x2, x2, __builtin_fma(x1, x1, x0 * x0)));
  }
}

template <typename T, int D>
__global__ void __launch_bounds__(1024)
importance_kernel(int32_t n_vectors, double count, const void* __restrict__ in,
                  double* __restrict__ importance) {
  constexpr int PER = 16 / (int)sizeof(T);    // elements per piece
  constexpr int NP = D / PER;                 // pieces per vector
  constexpr int LP = NP / kImpLanes;          // pieces per lane
  static_assert(LP >= 1 && NP % kImpLanes == 0, "a vector spans whole pieces of every lane");
  __shared__ double wave_sum[16][2];
  const int p = blockIdx.x;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int sub = threadIdx.x % kImpLanes;
  const T* base = reinterpret_cast<const T*>(in) + (int64_t)p * n_vectors * D;
  // this workgroup's slice: whole rounds of 128 vectors
  constexpr int kRound = 1024 / kImpLanes;
  const int n_slices = gridDim.y, slice = blockIdx.y;
  const int rounds = (n_vectors + kRound - 1) / kRound;
  const int v_lo = (int)((int64_t)rounds * slice / n_slices) * kRound;
  const int v_hi = min((int)((int64_t)rounds * (slice + 1) / n_slices) * kRound, n_vectors);
  SumDD acc;
  double mine = 0.0;  // squared norm of one of this group's last eight vectors
  int i = 0;
  for (int v = v_lo + threadIdx.x / kImpLanes; v < v_hi; v += kRound) {
    const T* row = base + (int64_t)v * D + sub * PER;
    double part[LP];
#pragma unroll
    for (int j = 0; j < LP; ++j) part[j] = sum_sq_piece<T>(row + j * kImpLanes * PER);
    double ss = 0.0;
#pragma unroll
    for (int j = 0; j < LP; ++j) ss += part[j];
#pragma unroll
    for (int m = 1; m < kImpLanes; m <<= 1) ss += __shfl_xor(ss, m, 64);
    if (sub == (i & (kImpLanes - 1))) mine = ss;
    if ((++i & (kImpLanes - 1)) == 0) {
      acc.add(sqrt(mine));
      mine = 0.0;
    }
  }
  acc.add(sqrt(mine));
  acc.add_lanes<64>();
  if (lane == 0) {
    wave_sum[wave][0] = acc.s;
    wave_sum[wave][1] = acc.c;
  }
  __syncthreads();
  if (wave != 0) return;
  SumDD total;
  if (lane < 16) total.add(wave_sum[lane][0], wave_sum[lane][1]);
  total.add_lanes<16>();
  if (n_slices > 1 && !imp_finish(p, slice, n_slices, &total)) return;
  if (lane == 0) importance[p] += total.value() / count;
}

hipError_t launch_kivi_quantize(const kvb_pool_layout& p, int32_t n_pool, int32_t first_layer,
                                int32_t n_in, kvb_dtype in_dtype, const void* k_in,
                                const void* v_in, uint8_t* k_codes, float* k_scale, float* k_zero,
                                uint8_t* v_codes, float* v_scale, float* v_zero, hipStream_t s) {
  const int64_t n_slabs = (int64_t)n_pool * n_in * p.n_kv_heads;
  const dim3 kgrid((unsigned)(n_slabs < 65536 ? n_slabs : 65536));
  const dim3 vgrid(grid_for(n_slabs * p.chunk_len * (p.head_dim / 8)));
#define KVB_QUANT(T, D, B)                                                                       \
  do {                                                                                           \
    const T* k = reinterpret_cast<const T*>(k_in);                                               \
    if (p.k_group < 32)                                                                          \
      hipLaunchKernelGGL((quant_keys_kernel<T, D, B, true>), kgrid, dim3(2 * D), 0, s, n_slabs,  \
                         p.n_layers, first_layer, n_in, p.n_kv_heads, p.k_group, k, k_codes,     \
                         k_scale, k_zero);                                                       \
    else                                                                                         \
      hipLaunchKernelGGL((quant_keys_kernel<T, D, B, false>), kgrid, dim3(2 * D), 0, s, n_slabs, \
                         p.n_layers, first_layer, n_in, p.n_kv_heads, p.k_group, k, k_codes,     \
                         k_scale, k_zero);                                                       \
    hipLaunchKernelGGL((quant_values_kernel<T, D, B>), vgrid, dim3(256), 0, s, n_slabs,          \
                       p.n_layers, first_layer, n_in, p.n_kv_heads, p.v_group,                   \
                       reinterpret_cast<const T*>(v_in), v_codes, v_scale, v_zero);              \
  } while (0)
#define KVB_QUANT_D(T, D)  \
  do {                     \
    if (p.bits == 8)       \
      KVB_QUANT(T, D, 8);  \
    else                   \
      KVB_QUANT(T, D, 4);  \
  } while (0)
  if (in_dtype == KVB_F64) {
    if (p.head_dim == 128) KVB_QUANT_D(double, 128); else KVB_QUANT_D(double, 64);
  } else {
    if (p.head_dim == 128) KVB_QUANT_D(float, 128); else KVB_QUANT_D(float, 64);
  }
#undef KVB_QUANT_D
#undef KVB_QUANT
  return hipGetLastError();
}

// Workgroups per chunk: at most one per CU, and what an estimate says ends first,
// in us.  A CU reads about 80 GB/s of keys that the last-level cache holds and 50
// from HBM whatever its loads in flight, the chip 6 TB/s (the longer of the two,
// and a little more where they are alike); a workgroup's arrival at the meeting
// place (cache write-back and atomics, one after another on an XCD) holds the
// launch up by 0.05 us, and the last one's by 2, so that many chunks, or small
// ones, are better left whole.  One workgroup a chunk, this rule and up to 512 workgroups a launch: 36 layers
// of fp64 keys, d = 128, 12 chunks 96 / 24 / 27 us, 40 175 / 73 / 85, 100 202 / 168 /
// 187, 256 400 / 399 / 427; 12 layers of fp32, d = 64, 64 17 / 17 / 27, 170 21 / 21 /
// 47.  A slice has four rounds of 128 vectors or more, a chunk that is split 16
// (8 chunks of 8 rounds, fp32, d = 64: 7.0 us whole, 8.6 in two).
static int imp_split(int32_t n_pool, int32_t n_vectors, size_t vector_bytes) {
  const double chunk = (double)n_vectors * vector_bytes, total = chunk * n_pool;
  const double alone = chunk / (total < 250e6 ? 80e3 : 50e3), all = total / 6e6;
  int split = 1;
  double best = INFINITY;
  for (int k = 1; k <= kImpSplit; ++k) {
    if (k > 1 && (n_vectors < 2048 || k > n_vectors / 512 || (int64_t)n_pool * k > kImpMaxWg)) break;
    const double r = alone / k;
    const double t = sqrt(sqrt(all * all * all * all + r * r * r * r)) + (k > 1 ? 2.0 + 0.05 * n_pool * k : 0.0);
    if (t < best) {
      best = t;
      split = k;
    }
  }
  return split;
}

hipError_t launch_chunk_importance(const kvb_pool_layout& p, int32_t n_pool, int32_t n_in,
                                   kvb_dtype in_dtype, const void* k_in, double* importance,
                                   hipStream_t s) {
  const int32_t n_vectors = n_in * p.n_kv_heads * p.chunk_len;
  const double count = (double)p.n_layers * p.n_kv_heads * p.chunk_len;
  const int split = imp_split(n_pool, n_vectors, (size_t)p.head_dim * (in_dtype == KVB_F64 ? 8 : 4));
#define KVB_IMPORTANCE(T, D)                                                                    \
  hipLaunchKernelGGL((importance_kernel<T, D>), dim3(n_pool, split), dim3(1024), 0, s, n_vectors, \
                     count, k_in, importance)
  if (in_dtype == KVB_F64) {
    if (p.head_dim == 128) KVB_IMPORTANCE(double, 128); else KVB_IMPORTANCE(double, 64);
  } else {
    if (p.head_dim == 128) KVB_IMPORTANCE(float, 128); else KVB_IMPORTANCE(float, 64);
  }
#undef KVB_IMPORTANCE
  return hipGetLastError();
}

}  // namespace kvb
