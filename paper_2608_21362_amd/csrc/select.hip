// Row selection (Alg. 2 step 3, Alg. 1 seam windows, live rows).
//
// One 1024-thread workgroup per (set, prompt) segment.  Deviations are mapped
// to order-preserving uint32 keys (NaN lowest, -0 equal to +0); a 4-pass
// 8-bit radix select over the segment's candidate rows finds the k-th largest
// key tau and how many rows equal to tau are still needed.  One ordered pass
// over the rows then takes: forced rows, candidates with key > tau, and the
// first `need_eq` candidates with key == tau in row order (the lower row wins
// a tie).  Positions come from wave ballots and a block-wide prefix, so the
// output is ascending without a sort and no atomic decides an order.  LDS
// atomics only count histogram bins.
//
// Batches of up to 64K rows in all (a host value; the prompts' own lengths are on
// the device) use select_reg_kernel: the prompt's rows are split
// into 16 equal runs, one per wave, and lane i of a wave holds the keys and
// flags of rows i, i + 64, .. of its run in registers (coalesced loads, read
// once), so the histogram passes touch no memory but LDS and a row's rank is
// its wave's base plus ballots on the scalar unit.  A launch has one workgroup
// per prompt and set, so it is bound by one CU's instruction issue (about 65
// vector instructions per slot and wave: 0.5 us per slot).  Hence three digits
// (12, 12 and 8 bits) instead of four of 8 bits, keys and flags folded into one
// word per row, and an end as soon as the k-th key's bin is selected whole
// (typically after 24 bits).  Four copies of the histogram (lane % 4) keep equal
// keys of a wave from queueing at one word.  36 sets of 8192 rows take 9 us (22
// with four 8-bit digits, one histogram and per-slot ranks through LDS), of
// 32772 rows 22 us (65).  Adds to a spare word instead of a branch around rows
// that do not count, and 16 copies of an 8-bit histogram, measured the same.
// Larger batches use select_kernel, which re-reads the keys on every pass.
//
// Several prompts per set: rows go to a staging area at the prompt's own row
// offset and a second small kernel packs them and writes cu_rows.
#include "kvb_device.h"
#include "kvb_internal.h"

#include <mutex>

namespace kvb {
namespace {

constexpr int kThreads = 1024;
constexpr int kWaves = kThreads / 64;

__device__ __forceinline__ uint32_t order_key(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7FFFFFFFu) > 0x7F800000u) return 0u;  // NaN: below everything
  if (u == 0x80000000u) u = 0u;                     // -0 -> +0
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

struct ScanLds {
  uint32_t wave_tot[kWaves];
};

// Block-wide exclusive prefix of a 0/1 flag (every thread must call).
__device__ __forceinline__ uint32_t block_excl(bool bit, ScanLds& s, uint32_t* total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint64_t m = __ballot(bit);
  const uint32_t below = (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
  if (lane == 0) s.wave_tot[wave] = (uint32_t)__popcll(m);
  __syncthreads();
  uint32_t before = 0, tot = 0;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    const uint32_t c = s.wave_tot[w];
    before += (w < wave) ? c : 0u;
    tot += c;
  }
  __syncthreads();
  *total = tot;
  return before + below;
}

__global__ void __launch_bounds__(kThreads)
select_kernel(int64_t t_total, const int32_t* __restrict__ cu_seqlens, int32_t n_seqs,
              const float* __restrict__ delta, const uint8_t* __restrict__ flags,
              const int32_t* __restrict__ k_per_seq, int32_t* __restrict__ rows_out,
              int32_t* __restrict__ cu_rows, int32_t* __restrict__ staging,
              int32_t* __restrict__ counts) {
  __shared__ uint32_t hist[256];
  __shared__ ScanLds scan;
  __shared__ uint32_t sh_prefix, sh_remaining;
  const int b = blockIdx.x;
  const int64_t set = blockIdx.y;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t lo = cu_seqlens[b], hi = cu_seqlens[b + 1];
  const float* dl = delta + set * t_total;

  // candidates in the segment
  uint32_t n_cand = 0;
  for (int64_t base = lo; base < hi; base += kThreads) {
    const int64_t r = base + tid;
    const bool c = r < hi && (flags[r] & KVB_ROW_CANDIDATE);
    uint32_t tot;
    block_excl(c, scan, &tot);
    n_cand += tot;
  }
  int64_t k = k_per_seq[set * n_seqs + b];
  if (k < 0) k = 0;
  const bool take_all = k >= (int64_t)n_cand;
  const bool take_none = k == 0;

  uint32_t tau = 0, need_eq = 0;
  if (!take_all && !take_none) {
    uint32_t prefix = 0, remaining = (uint32_t)k;
    for (int digit = 3; digit >= 0; --digit) {
      for (int i = tid; i < 256; i += kThreads) hist[i] = 0;
      __syncthreads();
      const uint32_t hi_mask = digit == 3 ? 0u : (0xFFFFFFFFu << (8 * (digit + 1)));
      int run_bin = -1;
      uint32_t run_n = 0;
      for (int64_t r = lo + tid; r < hi; r += kThreads) {
        if (!(flags[r] & KVB_ROW_CANDIDATE)) continue;
        const uint32_t key = order_key(dl[r]);
        if ((key & hi_mask) != (prefix & hi_mask)) continue;
        const int bin = (key >> (8 * digit)) & 0xFF;
        if (bin == run_bin) {
          ++run_n;
        } else {
          if (run_n) atomicAdd(&hist[run_bin], run_n);
          run_bin = bin;
          run_n = 1;
        }
      }
      if (run_n) atomicAdd(&hist[run_bin], run_n);
      __syncthreads();
      if (wave == 0) {
        // lane i owns bins 255-4i .. 252-4i (walking from the top)
        uint32_t hb[4], s = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          hb[j] = hist[255 - 4 * lane - j];
          s += hb[j];
        }
        uint32_t incl = s;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
          const uint32_t v = __shfl_up(incl, off, 64);
          if (lane >= off) incl += v;
        }
        const uint64_t hit = __ballot(incl >= remaining);
        const int first = __ffsll((unsigned long long)hit) - 1;
        if (lane == first) {
          uint32_t cum = incl - s;
          for (int j = 0; j < 4; ++j) {
            if (cum + hb[j] >= remaining) {
              sh_prefix = prefix | ((uint32_t)(255 - 4 * lane - j) << (8 * digit));
              sh_remaining = remaining - cum;
              break;
            }
            cum += hb[j];
          }
        }
      }
      __syncthreads();
      prefix = sh_prefix;
      remaining = sh_remaining;
    }
    tau = prefix;
    need_eq = remaining;
  }

  // ordered compaction
  uint32_t run_sel = 0, run_eq = 0;
  int32_t* dst = (n_seqs == 1) ? rows_out + set * t_total : staging + set * t_total + lo;
  for (int64_t base = lo; base < hi; base += kThreads) {
    const int64_t r = base + tid;
    const bool valid = r < hi;
    const uint32_t f = valid ? flags[r] : 0u;
    const bool cand = f & KVB_ROW_CANDIDATE;
    const bool forced = f & KVB_ROW_FORCED;
    bool gt = false, eq = false;
    if (cand) {
      if (take_all) {
        gt = true;
      } else if (!take_none) {
        const uint32_t key = order_key(dl[r]);
        gt = key > tau;
        eq = key == tau;
      }
    }
    uint32_t eq_tot;
    const uint32_t eq_rank = run_eq + block_excl(eq, scan, &eq_tot);
    const bool sel = forced || gt || (eq && eq_rank < need_eq);
    uint32_t sel_tot;
    const uint32_t idx = run_sel + block_excl(sel, scan, &sel_tot);
    if (sel) dst[idx] = (int32_t)r;
    run_sel += sel_tot;
    run_eq += eq_tot;
  }
  if (tid == 0) {
    if (n_seqs == 1) {
      cu_rows[set * 2] = 0;
      cu_rows[set * 2 + 1] = (int32_t)run_sel;
    } else {
      counts[set * n_seqs + b] = (int32_t)run_sel;
    }
  }
  (void)lane;
}


// Inclusive prefix sum over the 64 lanes of a wave, on the vector unit (DPP
// row shifts, then the two row broadcasts), no LDS round trips.
__device__ __forceinline__ uint32_t wave_incl(uint32_t x) {
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xF, 0xF, false);  // row_shr:1
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xF, 0xF, false);  // row_shr:2
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xF, 0xF, false);  // row_shr:4
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xF, 0xF, false);  // row_shr:8
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xA, 0xF, false);  // row_bcast:15
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xC, 0xF, false);  // row_bcast:31
  return x;
}

// Set lanes of a wave's ballot below this lane.
__device__ __forceinline__ uint32_t lanes_below(uint64_t ball) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(ball >> 32),
                                   __builtin_amdgcn_mbcnt_lo((uint32_t)ball, 0u));
}

constexpr int kBins = 4096;           // bins of a digit of up to 12 bits
constexpr int kCopies = 4;            // copies of every histogram (lane % 4)
constexpr int kCopyWords = kBins + 16;  // a bin's copies lie in different banks

// order_key for the register kernel, where 0 stands for a row that is no
// candidate: NaN is 1, below every number (the lowest, -inf, is 0x007FFFFF).
__device__ __forceinline__ uint32_t order_key_from1(float f) {
  const uint32_t u = __float_as_uint(f + 0.0f);  // -0 -> +0
  const uint32_t key = u ^ ((uint32_t)((int32_t)u >> 31) | 0x80000000u);
  return f != f ? 1u : key;
}

// Runs body(j) for the register slots of this thread, kBatch of them behind one
// uniform branch; slots from nslots on hold no rows.
template <int KPT, int kBatch, typename F>
__device__ __forceinline__ void for_slots(int nslots, F body) {
#pragma unroll
  for (int j0 = 0; j0 < KPT; j0 += kBatch)
    if (j0 < nslots) {
#pragma unroll
      for (int j = j0; j < j0 + kBatch; ++j) body(j);
    }
}

template <int KPT>
__global__ void __launch_bounds__(kThreads)
select_reg_kernel(int64_t t_total, const int32_t* __restrict__ cu_seqlens, int32_t n_seqs,
                  const float* __restrict__ delta, const uint8_t* __restrict__ flags,
                  const int32_t* __restrict__ k_per_seq, int32_t* __restrict__ rows_out,
                  int32_t* __restrict__ cu_rows, int32_t* __restrict__ staging,
                  int32_t* __restrict__ counts) {
  __shared__ uint4 hist4[kCopies * kCopyWords / 4];
  __shared__ uint32_t wave_tot[kWaves], eq_tot[kWaves], sel_tot[kWaves];
  __shared__ uint32_t sh_bin, sh_in_bin, sh_left;
  uint32_t* const hist = reinterpret_cast<uint32_t*>(hist4);
  constexpr int kBatch = KPT < 32 ? 4 : 8;
  const int b = blockIdx.x;
  const int64_t set = blockIdx.y;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t lo = cu_seqlens[b];
  const int n = (int)(cu_seqlens[b + 1] - lo);
  const int32_t k = k_per_seq[set * n_seqs + b];
  const int nslots = (n + kThreads - 1) / kThreads;  // <= KPT by the launch
  const float* dl = delta + set * t_total + lo;
  const uint8_t* fl = flags + lo;
  const int first = wave * 64 * nslots + lane;  // slot j: row lo + first + 64 j

  for (int i = tid; i < (int)(sizeof(hist4) / sizeof(uint4)); i += kThreads)
    hist4[i] = make_uint4(0, 0, 0, 0);

  // this thread's keys (0: no candidate) and forced bits, loaded once.  Loads
  // are unconditional (past the segment its last row is read again, and a row
  // that is no candidate has a deviation in range that is never used), and all
  // of them (half of them from 48 slots on, for the registers) go out before any is used.
  constexpr int kStage = KPT > 32 ? KPT / 2 : KPT;
  uint32_t key[KPT] = {}, forced[(KPT + 31) / 32] = {};
#pragma unroll
  for (int s0 = 0; s0 < KPT; s0 += kStage) {
    uint32_t f[kStage];
    for_slots<kStage, kBatch>(nslots - s0, [&](int i) {
      const uint32_t r = (uint32_t)min(first + 64 * (s0 + i), n - 1);
      f[i] = fl[r];
      key[s0 + i] = __float_as_uint(dl[r]);
    });
    for_slots<kStage, kBatch>(nslots - s0, [&](int i) {
      const int j = s0 + i;
      const uint32_t fj = j < nslots && first + 64 * j < n ? f[i] : 0u;
      key[j] = (fj & KVB_ROW_CANDIDATE) ? order_key_from1(__uint_as_float(key[j])) : 0u;
      forced[j / 32] |= ((fj & KVB_ROW_FORCED) ? 1u : 0u) << (j % 32);
    });
  }
  __syncthreads();

  // candidates with (key & mask) >= prefix are selected, except those equal to
  // it past the first `remaining` of n_eq
  uint32_t prefix = 0, mask = 0, n_eq = 0;
  uint32_t remaining = k > 0 ? (uint32_t)k : 0u;
  if (remaining == 0) {
    prefix = mask = 0xFFFFFFFFu;  // above every key
  } else {
    // digits of 12, 12 and 8 bits
#pragma unroll 1
    for (int shift = 20; shift > -12; shift -= 12) {
      const int sh = shift < 0 ? 0 : shift;
      const uint32_t digit_mask = shift < 0 ? 0xFFu : 0xFFFu;
      const uint32_t copy = (uint32_t)(lane % kCopies) * kCopyWords;
      for_slots<KPT, kBatch>(nslots, [&](int j) {
        if ((key[j] & mask) == prefix && key[j] != 0)
          atomicAdd(&hist[copy + ((key[j] >> sh) & digit_mask)], 1u);
      });
      __syncthreads();
      // thread t owns bins 4095-4t .. 4092-4t (walking from the top): adds their
      // copies and clears them for the next digit
      uint4 q = make_uint4(0, 0, 0, 0);
#pragma unroll
      for (int c = 0; c < kCopies; ++c) {
        uint4* p = hist4 + c * (kCopyWords / 4) + (kThreads - 1 - tid);
        const uint4 x = *p;
        *p = make_uint4(0, 0, 0, 0);
        q.x += x.x;
        q.y += x.y;
        q.z += x.z;
        q.w += x.w;
      }
      const uint32_t hb[4] = {q.w, q.z, q.y, q.x};
      const uint32_t sum = q.x + q.y + q.z + q.w;
      const uint32_t incl = wave_incl(sum);
      if (lane == 63) wave_tot[wave] = incl;
      __syncthreads();
      uint32_t before = 0, total = 0;
#pragma unroll
      for (int w = 0; w < kWaves; ++w) {
        const uint32_t c = wave_tot[w];
        before += w < wave ? c : 0u;
        total += c;
      }
      if (shift == 20 && remaining >= total) {
        prefix = 1;  // k reaches every candidate
        mask = 0xFFFFFFFFu;
        n_eq = remaining;
        break;
      }
      uint32_t cum = before + incl - sum;
      if (cum < remaining && cum + sum >= remaining) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          if (cum < remaining && cum + hb[j] >= remaining) {
            sh_bin = (uint32_t)(kBins - 1 - 4 * tid - j);
            sh_in_bin = hb[j];
            sh_left = remaining - cum;
          }
          cum += hb[j];
        }
      }
      __syncthreads();
      prefix |= sh_bin << sh;
      mask |= digit_mask << sh;
      n_eq = sh_in_bin;
      remaining = sh_left;
      if (remaining == n_eq) break;  // the whole bin is selected: no finer digit matters
    }
    if (prefix == 0) {  // a bin of NaN keys alone: keep rows that are no candidates out
      prefix = 1;
      mask = 0xFFFFFFFFu;
    }
    if (remaining < n_eq) {
      // of the keys equal to the k-th only the first `remaining` in row order
      // (the lower row wins a tie): the others leave the candidates
      uint32_t mine = 0;
      for_slots<KPT, kBatch>(nslots, [&](int j) {
        mine += (uint32_t)__popcll(__builtin_amdgcn_ballot_w64(key[j] == prefix));
      });
      if (lane == 0) eq_tot[wave] = mine;
      __syncthreads();
      uint32_t run = 0;
      for (int w = 0; w < wave; ++w) run += eq_tot[w];
      for_slots<KPT, kBatch>(nslots, [&](int j) {
        const bool eq = key[j] == prefix;
        const uint64_t ball = __builtin_amdgcn_ballot_w64(eq);
        if (eq && run + lanes_below(ball) >= remaining) key[j] = 0;
        run += (uint32_t)__popcll(ball);
      });
    }
  }

  // ascending rows: waves in order, slots in order, lanes in order
  const auto selected = [&](int j) {
    return (key[j] & mask) >= prefix || ((forced[j / 32] >> (j % 32)) & 1u);
  };
  uint32_t mine = 0;
  for_slots<KPT, kBatch>(nslots, [&](int j) {
    mine += (uint32_t)__popcll(__builtin_amdgcn_ballot_w64(selected(j)));
  });
  if (lane == 0) sel_tot[wave] = mine;
  __syncthreads();
  uint32_t run = 0, n_sel = 0;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    const uint32_t c = sel_tot[w];
    run += w < wave ? c : 0u;
    n_sel += c;
  }
  int32_t* dst = (n_seqs == 1) ? rows_out + set * t_total : staging + set * t_total + lo;
  for_slots<KPT, kBatch>(nslots, [&](int j) {
    const bool sel = selected(j);
    const uint64_t ball = __builtin_amdgcn_ballot_w64(sel);
    if (sel) dst[run + lanes_below(ball)] = (int32_t)lo + first + 64 * j;
    run += (uint32_t)__popcll(ball);
  });
  if (tid == 0) {
    if (n_seqs == 1) {
      cu_rows[set * 2] = 0;
      cu_rows[set * 2 + 1] = (int32_t)n_sel;
    } else {
      counts[set * n_seqs + b] = (int32_t)n_sel;
    }
  }
}

// Packs the prompts' rows of a set and writes its offsets.  Bound by its chain of
// loads: the prompts' counts are read 64 at a time and summed across lanes, and
// the first rows of the staging area are requested beside them (deviation and
// selection of 8 prompts of 1.0K to 2.1K rows 65.1 us; 67.2 with the counts added
// one by one and the rows read after them).
__global__ void __launch_bounds__(256)
pack_kernel(int64_t t_total, const int32_t* __restrict__ cu_seqlens, int32_t n_seqs,
            const int32_t* __restrict__ staging, const int32_t* __restrict__ counts,
            int32_t* __restrict__ rows_out, int32_t* __restrict__ cu_rows) {
  const int b = blockIdx.x;
  const int64_t set = blockIdx.y;
  const int tid = threadIdx.x, lane = tid & 63;
  const int32_t* cnt = counts + set * n_seqs;
  int32_t* cu = cu_rows + set * (n_seqs + 1);
  const int64_t lo = cu_seqlens[b];
  const int len = (int)(cu_seqlens[b + 1] - lo);
  const int32_t n = cnt[b];
  const int32_t* src = staging + set * t_total + lo;
  // the first rows, whether or not the prompt has that many (read within its
  // part of the staging area)
  constexpr int U = 4;
  int32_t head[U];
#pragma unroll
  for (int u = 0; u < U; ++u) head[u] = len > 0 ? src[min(tid + 256 * u, len - 1)] : 0;
  int64_t off = 0;
  int32_t acc = 0;  // rows of the prompts before base
  if (b == 0 && tid == 0) cu[0] = 0;
  for (int base = 0; base < n_seqs && (b == 0 || base < b); base += 64) {
    const int i = base + lane;
    const int32_t c = i < n_seqs ? cnt[i] : 0;
    const uint32_t incl = wave_incl((uint32_t)c);
    if (b == 0 && tid < 64 && i < n_seqs) cu[i + 1] = acc + (int32_t)incl;
    const int before = min(b - base, 64);  // prompts of these 64 before b
    if (before > 0) off += (uint32_t)__builtin_amdgcn_readlane((int)incl, before - 1);
    acc += __builtin_amdgcn_readlane((int)incl, 63);
  }
  int32_t* dst = rows_out + set * t_total + off;
#pragma unroll
  for (int u = 0; u < U; ++u)
    if (tid + 256 * u < n) dst[tid + 256 * u] = head[u];
  for (int i = tid + 256 * U; i < n; i += 256) dst[i] = src[i];
}

}  // namespace

size_t select_workspace_bytes(int32_t n_sets, int64_t t_total, int32_t n_seqs) {
  if (n_seqs <= 1) return 0;
  const size_t staging = (size_t)n_sets * (size_t)t_total * sizeof(int32_t);
  const size_t counts = (size_t)n_sets * (size_t)n_seqs * sizeof(int32_t);
  return ((staging + 255) / 256) * 256 + counts;
}

hipError_t launch_select(int32_t n_sets, int64_t t_total, const int32_t* cu_seqlens,
                         int32_t n_seqs, const float* delta, const uint8_t* row_flags,
                         const int32_t* k_per_seq, int32_t* rows, int32_t* cu_rows,
                         void* workspace, hipStream_t s) {
  int32_t* staging = nullptr;
  int32_t* counts = nullptr;
  if (n_seqs > 1) {
    staging = reinterpret_cast<int32_t*>(workspace);
    const size_t st = (size_t)n_sets * (size_t)t_total * sizeof(int32_t);
    counts = reinterpret_cast<int32_t*>(reinterpret_cast<char*>(workspace) + ((st + 255) / 256) * 256);
  }
  // the longest prompt is at most t_total rows: pick the register-slot count from
  // it (at most 64 keys a thread: with 16 waves a workgroup a thread has 128
  // registers)
  const dim3 grid(n_seqs, n_sets);
#define KVB_SELECT_REG(K)                                                                       \
  hipLaunchKernelGGL(select_reg_kernel<K>, grid, dim3(kThreads), 0, s, t_total, cu_seqlens,     \
                     n_seqs, delta, row_flags, k_per_seq, rows, cu_rows, staging, counts)
  if (t_total <= 8 * kThreads)
    KVB_SELECT_REG(8);
  else if (t_total <= 16 * kThreads)
    KVB_SELECT_REG(16);
  else if (t_total <= 32 * kThreads)
    KVB_SELECT_REG(32);
  else if (t_total <= 48 * kThreads)
    KVB_SELECT_REG(48);
  else if (t_total <= 64 * kThreads)
    KVB_SELECT_REG(64);
  else
    hipLaunchKernelGGL(select_kernel, grid, dim3(kThreads), 0, s, t_total, cu_seqlens, n_seqs,
                       delta, row_flags, k_per_seq, rows, cu_rows, staging, counts);
#undef KVB_SELECT_REG
  if (n_seqs > 1)
    hipLaunchKernelGGL(pack_kernel, dim3(n_seqs, n_sets), dim3(256), 0, s, t_total, cu_seqlens,
                       n_seqs, staging, counts, rows, cu_rows);
  return hipGetLastError();
}

// Scratch of the allocation-free selection (kvb_select_noalloc): the staging
// rows and per-prompt counts that kvb_select keeps in the caller's workspace.
// Every device the library runs on holds one copy for the life of the process.
// In host code `scratch` names a host-side stand-in, not device memory: host
// code reaches the array only through the address select_scratch returns.
static __device__ __align__(256) unsigned char scratch[kSelectScratchBytes];

// Device address of this device's copy of `scratch`, looked up once per device
// (with that device current) and kept.
hipError_t select_scratch(void** ptr) {
  static std::mutex mu;
  static void* addr[kMaxDevices] = {};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (addr[dev] == nullptr) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    addr[dev] = p;
  }
  *ptr = addr[dev];
  return hipSuccess;
}

hipError_t launch_select_noalloc(int32_t n_sets, int64_t t_total, const int32_t* cu_seqlens,
                                 int32_t n_seqs, const float* delta, const uint8_t* row_flags,
                                 const int32_t* k_per_seq, int32_t* rows, int32_t* cu_rows,
                                 hipStream_t s) {
  void* ws = nullptr;
  if (n_seqs > 1) {
    hipError_t e = select_scratch(&ws);
    if (e != hipSuccess) return e;
  }
  return launch_select(n_sets, t_total, cu_seqlens, n_seqs, delta, row_flags, k_per_seq, rows,
                       cu_rows, ws, s);
}

}  // namespace kvb
