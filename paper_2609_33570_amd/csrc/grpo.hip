// GRPO update quantities on gfx950: group-relative advantages, importance
// ratios, clip flags and the per-token loss coefficients omega_t = dL/ds_t.
//
//   A_j     = (R_j - mean_group) / (population std_group + adv_eps)
//             (Sec. 3.1; App. D.1.1, "GRPO and optimization")
//   r_t     = exp(s_t - s_t^old)                               (Sec. 3.1)
//   chi_t   = [(A >= 0 and r <= 1+eps) or (A < 0 and r >= 1-eps)]
//                                             (Sec. 3.2, Eq. update-coefficient)
//   omega_t = (m_t / N) (-chi_t r_t A - beta expm1(s_ref - s_t))
//             (Eq. update-coefficient with the K3 KL derivative of the proof of
//             Prop. 1)
//
// Each workgroup of grpo_kernel owns a run of 1024 consecutive token slots
// (4 per thread, 128-bit loads), from 2^20 slots on two runs (the group
// statistics, the count and the launch ramp are then paid half as often; four
// runs leave too few loads in flight) unless the operands are far larger than the
// caches (see launch_grpo).  At 2^22 masked slots with K3 and N
// counted, in a graph: 28.3 us with one run, 64-bit indices, a division per slot
// and expm1f throughout (then bound by its vector instructions), 19.4 us now, 23.0
// with four runs; 92 MB at the copy rate take 15.  It first forms, with wave
// butterflies, the advantages of every group its slots touch (a group of G <= 64
// rewards sits in the lanes of one wave; the group sums are the pairwise tree over
// the next power of two >= G, which the xor butterfly produces exactly) and keeps
// them in LDS; then every thread processes its 4 slots elementwise.
// When N has to be counted (no N given, a mask present), calls of at most
// kGrpoCountInKernelSlots slots let every workgroup count the whole mask
// itself (bytes summed four at a time with a dot product): one launch, no
// scratch, and the mask (at most 64 KB) stays in L2.  Larger calls first run
// count_kernel, whose workgroups each count one contiguous range of the mask
// into the caller's workspace (one 32-bit count each, at most kGrpoCounts),
// and every workgroup of grpo_kernel then adds those counts (exact integer
// sums): the mask is read once more in total instead of once per workgroup.
// Every load a thread makes is issued before the first arithmetic (the mask
// words or counts for N in batches of 8 per thread), so a launch waits on
// memory about once instead of once per phase.
#include "device_common.hpp"
#include "hilore_internal.hpp"

// Every rounding step is the one written: no implicit fused multiply-add
// (the exact sequences above depend on it; wanted FMAs are explicit fmaf).
#pragma clang fp contract(off)

namespace hilore {
namespace {

constexpr int kThreads = 256;
constexpr int kSlotsPerThread = 4;
constexpr int kSlotsPerBlock = kThreads * kSlotsPerThread;
constexpr int kCountThreads = 1024;  // pre-pass: 2^16 slots are four mask words per thread
constexpr int kCountBatch = 4;
constexpr int64_t kTwoRunSlots = int64_t(1) << 20;  // from here on two runs per workgroup,
constexpr int64_t kOneRunBytes = int64_t(576) << 20;  // and one again from these operands on
constexpr int kMaskBatch = 8;  // 16-byte mask words per thread in flight while counting
static_assert(kGrpoCounts <= kThreads, "one pre-pass count per thread");

// Pairwise-tree sum over the first P2 lanes (P2 a power of two <= 64) by an
// xor butterfly; lanes >= P2 must not be mixed in, so the loop stops at P2/2.
__device__ __forceinline__ float group_sum(float v, int p2) {
  for (int off = 1; off < p2; off <<= 1) v += __shfl_xor(v, off, kWave);
  return v;
}

__device__ __forceinline__ uint32_t nonzero_bytes(uint32_t w) {
  w |= w >> 4;
  w |= w >> 2;
  w |= w >> 1;
  return __builtin_amdgcn_udot4(w & 0x01010101u, 0x01010101u, 0u, false);
}

// Count of the nonzero bytes of mask words [w0, w1) plus, in the last
// workgroup, of the bytes past the last whole word; one 32-bit count per
// workgroup.
__global__ __launch_bounds__(kCountThreads) void count_kernel(const uint8_t *mask, int64_t n_slots,
                                                         int64_t words_per_wg, uint32_t *counts) {
  __shared__ uint32_t red[kCountThreads / kWave];
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
  const int64_t n_words = n_slots / 16;
  const int64_t w0 = (int64_t)blockIdx.x * words_per_wg;
  const int64_t w1 = w0 + words_per_wg < n_words ? w0 + words_per_wg : n_words;
  const uint4 *m4 = reinterpret_cast<const uint4 *>(mask);
  uint32_t cnt = 0;
  for (int64_t base = w0; base < w1; base += kCountBatch * kCountThreads) {
    uint4 mw[kCountBatch];
#pragma unroll
    for (int u = 0; u < kCountBatch; ++u) {
      const int64_t i = base + (int64_t)u * kCountThreads + tid;
      mw[u] = i < w1 ? m4[i] : make_uint4(0u, 0u, 0u, 0u);
    }
#pragma unroll
    for (int u = 0; u < kCountBatch; ++u)
      cnt += nonzero_bytes(mw[u].x) + nonzero_bytes(mw[u].y) + nonzero_bytes(mw[u].z) +
             nonzero_bytes(mw[u].w);
  }
  if (blockIdx.x == gridDim.x - 1)
    for (int64_t i = n_words * 16 + tid; i < n_slots; i += kCountThreads) cnt += mask[i] != 0;
  for (int off = 1; off < kWave; off <<= 1) cnt += __shfl_xor(cnt, off, kWave);
  if (lane == 0) red[wave] = cnt;
  __syncthreads();
  if (tid == 0) {
    uint32_t n = 0;
#pragma unroll
    for (int w = 0; w < kCountThreads / kWave; ++w) n += red[w];
    counts[blockIdx.x] = n;
  }
}

// expm1 for |x| <= 1/2: the Taylor polynomial to x^8 (its remainder is below
// 2^-26 of x there) closed by one rounding of x + x^2 P(x); 9 instructions
// against about 35 of expm1f, and closer to fp64 (4e6 points of the range: 0.85
// ulp at worst and 2.6e-8 rms, expm1f 1.37 and 2.9e-8).
__device__ __forceinline__ float expm1_near0(float x) {
  float p = 1.0f / 40320.0f;
  p = fmaf(p, x, 1.0f / 5040.0f);
  p = fmaf(p, x, 1.0f / 720.0f);
  p = fmaf(p, x, 1.0f / 120.0f);
  p = fmaf(p, x, 1.0f / 24.0f);
  p = fmaf(p, x, 1.0f / 6.0f);
  p = fmaf(p, x, 0.5f);
  return fmaf(x * x, p, x);
}

// Outputs of large calls (NT) stream past the caches, which leaves more of them to
// the inputs: 2^22 slots with K3, mask and ratio 21.3 -> 19.3 us, 2^24 75 -> 61.
typedef float f32x4 __attribute__((ext_vector_type(4)));
template <bool NT, typename T, typename V>
__device__ __forceinline__ void store(T *p, V v) {
  if constexpr (NT) __builtin_nontemporal_store(v, reinterpret_cast<V *>(p));
  else *reinterpret_cast<V *>(p) = v;
}

// One workgroup owns U runs of kSlotsPerBlock slots.  Indices fit 32 bits
// (fewer than 2^31 slots; unsigned sums of a run stay below 2^32).
template <int U, bool NT>
__global__ __launch_bounds__(kThreads) void grpo_kernel(const GrpoArgs a, int p2) {
  constexpr uint32_t kRun = U * kSlotsPerBlock;
  __shared__ float adv_lds[kRun + 2];  // responses overlapping the runs (T >= 1)
  __shared__ uint32_t red[kThreads / kWave];

  const int tid = threadIdx.x;
  const int lane = tid & (kWave - 1);
  const int wave = tid / kWave;
  const uint32_t R = (uint32_t)a.P * (uint32_t)a.G;
  const bool no_tokens = a.T == 0;
  const uint32_t T = no_tokens ? 1u : (uint32_t)a.T;  // with T == 0 a run covers responses
  const uint32_t n_slots = R * T;
  const uint32_t c0 = blockIdx.x * kRun;
  const uint32_t c1 = c0 + kRun < n_slots ? c0 + kRun : n_slots;
  const uint32_t j_lo = c0 / T;
  const uint32_t j_hi = (c1 - 1) / T;  // inclusive
  const uint32_t g_lo = j_lo / (uint32_t)a.G;
  const uint32_t g_hi = j_hi / (uint32_t)a.G;

  // ---- loads first ----
  // Nothing below changes what a thread reads, so its token slots and the
  // first batch of mask words for the count are requested before any
  // arithmetic: the whole prologue then waits on memory about once.
  float sn[U][4], so[U][4], sref[U][4];
  uint32_t mk[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const uint32_t i0 = c0 + (uint32_t)(u * kSlotsPerBlock + tid * kSlotsPerThread);
    mk[u] = 0x01010101u;
#pragma unroll
    for (int k = 0; k < 4; ++k) sn[u][k] = so[u][k] = sref[u][k] = 0.f;
    if (no_tokens || i0 >= c1) continue;
    if (i0 + kSlotsPerThread <= c1) {
      const float4 n4 = *reinterpret_cast<const float4 *>(a.logp_new + i0);
      const float4 o4 = *reinterpret_cast<const float4 *>(a.logp_old + i0);
      sn[u][0] = n4.x; sn[u][1] = n4.y; sn[u][2] = n4.z; sn[u][3] = n4.w;
      so[u][0] = o4.x; so[u][1] = o4.y; so[u][2] = o4.z; so[u][3] = o4.w;
      if (a.beta != 0.0f) {
        const float4 r4 = *reinterpret_cast<const float4 *>(a.logp_ref + i0);
        sref[u][0] = r4.x; sref[u][1] = r4.y; sref[u][2] = r4.z; sref[u][3] = r4.w;
      }
      if (a.mask) mk[u] = *reinterpret_cast<const uint32_t *>(a.mask + i0);
    } else {
      mk[u] = 0;
#pragma unroll
      for (int k = 0; k < kSlotsPerThread; ++k) {
        const uint32_t i = i0 + k;
        const bool in = i < c1;
        sn[u][k] = in ? a.logp_new[i] : 0.0f;
        so[u][k] = in ? a.logp_old[i] : 0.0f;
        if (a.beta != 0.0f) sref[u][k] = in ? a.logp_ref[i] : 0.0f;
        const uint32_t m = in ? (a.mask ? a.mask[i] : 1u) : 0u;
        mk[u] |= m << (8 * k);
      }
    }
  }
  // counts of a count_kernel pre-pass (one per thread at most), else the mask itself
  uint32_t pre = 0;
  if (!no_tokens && a.count_mask && a.counts && tid < a.n_counts) pre = a.counts[tid];
  const bool count_words = !no_tokens && a.count_mask && a.mask && !a.counts;
  const uint32_t n_words = count_words ? n_slots / 16 : 0;
  const uint4 *m4 = reinterpret_cast<const uint4 *>(a.mask);
  uint4 mw[kMaskBatch];
  if constexpr (U == 1) {  // larger calls count in a pre-pass
#pragma unroll
    for (int u = 0; u < kMaskBatch; ++u) {
      const uint32_t i = (uint32_t)(u * kThreads + tid);
      mw[u] = i < n_words ? m4[i] : make_uint4(0u, 0u, 0u, 0u);
    }
  }

  // ---- advantages of the groups this run touches ----
  for (uint32_t grp = g_lo + wave; grp <= g_hi; grp += kThreads / kWave) {
    const uint32_t j = grp * (uint32_t)a.G + lane;
    const bool in = lane < a.G;
    const float rew = in ? a.rewards[j] : 0.0f;
    const float mu = group_sum(rew, p2) / (float)a.G;
    const float dv = in ? rew - mu : 0.0f;
    const float sigma = sqrtf(group_sum(dv * dv, p2) / (float)a.G);
    const float adv = dv / (sigma + a.adv_eps);
    if (in) {
      if (j >= j_lo && j <= j_hi) adv_lds[j - j_lo] = adv;
      if (j * T >= c0 && j * T < c1) a.adv[j] = adv;  // owner of the response's first slot
    }
  }

  if (no_tokens) return;  // advantages only

  // ---- normaliser ----
  float inv_n = a.inv_n;
  if (a.count_mask) {
    uint32_t cnt = 0;
    if (a.counts) {
      cnt = pre;
    } else if (a.mask) {
      if constexpr (U == 1) {
        for (uint32_t base = 0; base < n_words; base += kMaskBatch * kThreads) {
          if (base > 0) {  // later batches: all loads of a batch in flight at once
#pragma unroll
            for (int u = 0; u < kMaskBatch; ++u) {
              const uint32_t i = base + (uint32_t)(u * kThreads + tid);
              mw[u] = i < n_words ? m4[i] : make_uint4(0u, 0u, 0u, 0u);
            }
          }
#pragma unroll
          for (int u = 0; u < kMaskBatch; ++u)
            cnt += nonzero_bytes(mw[u].x) + nonzero_bytes(mw[u].y) + nonzero_bytes(mw[u].z) +
                   nonzero_bytes(mw[u].w);
        }
        for (uint32_t i = n_words * 16 + tid; i < n_slots; i += kThreads) cnt += a.mask[i] != 0;
      }
    } else {
      cnt = tid == 0 ? n_slots : 0u;
    }
    for (int off = 1; off < kWave; off <<= 1) cnt += __shfl_xor(cnt, off, kWave);
    if (lane == 0) red[wave] = cnt;
    __syncthreads();
    const uint32_t n = red[0] + red[1] + red[2] + red[3];
    inv_n = n > 0 ? 1.0f / (float)n : 0.0f;
  } else {
    __syncthreads();
  }

  // ---- per-token quantities ----
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const uint32_t i0 = c0 + (uint32_t)(u * kSlotsPerBlock + tid * kSlotsPerThread);
    if (i0 >= c1) continue;
    float kl[4] = {0.f, 0.f, 0.f, 0.f};
    if (a.beta != 0.0f) {
      float d[4], e[4];
      bool near0 = true;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        d[k] = sref[u][k] - sn[u][k];
        e[k] = expm1_near0(d[k]);
        near0 = near0 && fabsf(d[k]) <= 0.5f;
      }
      if (!__all(near0)) {  // a slot's value depends on its own difference alone
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const float far = expm1f(d[k]);
          e[k] = fabsf(d[k]) <= 0.5f ? e[k] : far;
        }
      }
#pragma unroll
      for (int k = 0; k < 4; ++k) kl[k] = a.beta * e[k];
    }
    float rat[4], om[4];
    uint32_t fl = 0;
    uint32_t j = i0 / T, next = (j + 1) * T;  // response of slot i0, first slot of the next one
#pragma unroll
    for (int k = 0; k < kSlotsPerThread; ++k) {
      if (i0 + k == next) {
        ++j;
        next += T;
      }
      const float A = adv_lds[(j < j_hi ? j : j_hi) - j_lo];
      const bool m = ((mk[u] >> (8 * k)) & 0xFFu) != 0;
      const float delta = sn[u][k] - so[u][k];
      const bool chi = A >= 0.0f ? delta <= a.hi : delta >= a.lo;
      const float r = expf(delta);
      const float pol = chi ? r * A : 0.0f;
      rat[k] = r;
      om[k] = m ? (-pol - kl[k]) * inv_n : 0.0f;
      const uint32_t f = (m && chi ? 1u : 0u) | (m && A != 0.0f && !chi ? 2u : 0u);
      fl |= f << (8 * k);
    }
    if (i0 + kSlotsPerThread <= c1) {
      store<NT>(a.coeff + i0, f32x4{om[0], om[1], om[2], om[3]});
      if (a.ratio) store<NT>(a.ratio + i0, f32x4{rat[0], rat[1], rat[2], rat[3]});
      store<NT>(a.flags + i0, fl);
    } else {
#pragma unroll
      for (int k = 0; k < kSlotsPerThread; ++k) {
        const uint32_t i = i0 + k;
        if (i < c1) {
          a.coeff[i] = om[k];
          if (a.ratio) a.ratio[i] = rat[k];
          a.flags[i] = (uint8_t)(fl >> (8 * k));
        }
      }
    }
  }
}

}  // namespace

int grpo_count_blocks(int64_t slots) {
  if (slots <= kGrpoCountInKernelSlots) return 0;
  const int64_t n = (slots + kGrpoSlotsPerCount - 1) / kGrpoSlotsPerCount;
  return (int)(n < kGrpoCounts ? n : kGrpoCounts);
}

hipError_t launch_grpo(const GrpoArgs &a, uint32_t *counts, hipStream_t s) {
  const int64_t R = (int64_t)a.P * a.G;
  const int64_t slots = a.T == 0 ? R : R * a.T;
  if (slots == 0) return hipSuccess;
  int p2 = 1;
  while (p2 < a.G) p2 <<= 1;
  GrpoArgs b = a;
  b.counts = nullptr;
  b.n_counts = 0;
  if (a.T > 0 && a.count_mask && a.mask && counts) {
    const int nb = grpo_count_blocks(slots);
    if (nb > 0) {  // counted by a pre-pass into the workspace
      const int64_t n_words = slots / 16;
      const int64_t per = (n_words + nb - 1) / nb;
      hipLaunchKernelGGL(count_kernel, dim3((unsigned)nb), dim3(kCountThreads), 0, s, a.mask, slots,
                         per, counts);
      const hipError_t e = hipGetLastError();
      if (e != hipSuccess) return e;
      b.counts = counts;
      b.n_counts = nb;
    }
  }
  // Two runs per workgroup need the pre-pass (or no count), and the chip full with
  // half the workgroups: at 2^20 slots 512 of them.  Once the operands are more than
  // twice the 256 MB cache, calls with logp_ref or ratio run slower in pairs: 2^26
  // masked slots, N given, 248 us with one run and 264 with two (K3 and ratio), 198 and
  // 212 (K3), 199 and 214 (ratio); 2^25 131 / 134, 104 / 107, 102 / 107; 2^24 55 / 56,
  // 47.5 / 46.5, 48 / 46.  The line lies at 18 bytes for 2^25 slots: 17 bytes (ratio
  // without a mask) still take 89 / 85.  Without both operands pairs stay ahead or
  // close (2^26 unmasked slots 163 / 151, masked 179 / 169 counted, 155 / 163 given).
  const bool large = slots >= kTwoRunSlots;
  const int64_t bytes = 13 + (a.mask ? 1 : 0) + (a.logp_ref ? 4 : 0) + (a.ratio ? 4 : 0);
  const bool single = (a.logp_ref || a.ratio) && slots * bytes >= kOneRunBytes;
  const bool two = large && !single && (b.counts || !a.mask || !a.count_mask);
  const int64_t run = kSlotsPerBlock * (two ? 2 : 1);
  const dim3 grid((unsigned)((slots + run - 1) / run));
  if (two) hipLaunchKernelGGL((grpo_kernel<2, true>), grid, dim3(kThreads), 0, s, b, p2);
  else if (large) hipLaunchKernelGGL((grpo_kernel<1, true>), grid, dim3(kThreads), 0, s, b, p2);
  else hipLaunchKernelGGL((grpo_kernel<1, false>), grid, dim3(kThreads), 0, s, b, p2);
  return hipGetLastError();
}

}  // namespace hilore
