// Joint H/L/R recovery allocation on gfx950 (Sec. 3.4 Eq. joint-allocation,
// solved as in App. B.2 Eqs. allocation-grid, allocation-integer-costs and
// allocation-dp, with the available actions of App. B.3 Eq.
// available-recovery-actions).
//
// Each unit u takes one action in {R, H, L}: R (recompute) is the baseline
// with zero utility, memory and risk; H keeps the activation (utility tau_h,
// memory dm_h, risk 0); L keeps its low-precision codes (tau_l, dm_l, risk
// psi_u).  Memory and risk costs are rounded up to integer steps of the
// budgets (N_B and N_delta intervals), and the dynamic programme
//   F_i(j, k) = max over available a of F_{i-1}(j - b_i(a), k - r_i(a)) + tau_i(a)
// runs over the (N_B + 1) x (N_delta + 1) grid of exact integer costs.
//
// Mapping.  One launch (setup_kernel) forms the integer costs, the memory cost
// reach after each unit and the initial tables.  Then one launch per pair of
// units updates the whole grid, one thread per cell (rows k of risk cost,
// columns j of memory cost, a row padded to a multiple of 64 cells so that a wave
// covers 64 consecutive cells of one row; each XCD takes one contiguous band of
// cells: 100 us less of a call with 196 units).  Each cell forms the first unit's
// value at itself and at the two cells the second unit's actions shift it to,
// from up to nine cells of the table before the pair (fp64, all in the 256 MB
// infinity cache for grids up to a few thousand squared), and writes the value
// after the pair; the chosen actions come out of the comparisons as lane masks
// and are stored as two 64-bit words per unit and 64 cells, so the backtracking
// record of a 1025 x 1025 grid is 279 KB per unit.  A reduction kernel then finds
// the best terminal cell, and one wave backtracks through the records (four units
// per round trip) and sums the chosen costs in unit order.
//
// Every value is produced by the same fp64 operations in the same order as
// a plain sequential implementation (one addition per unit along a path,
// comparisons with the fixed tie rules), so actions and totals are exact.
#include <math.h>

#include "device_common.hpp"
#include "hilore_internal.hpp"

#pragma clang fp contract(off)

namespace hilore {
namespace {

constexpr int kActR = 0, kActH = 1, kActL = 2;
typedef uint64_t u64x2 __attribute__((ext_vector_type(2)));
constexpr int kDpThreads = 256;
constexpr int kPartials = 1024;  // workgroups of the terminal reduction
constexpr int kFinalThreads = 1024;
constexpr int kDpGroup = 2;  // units per DP launch

constexpr int kNever = 1 << 20;  // risk cost of an unavailable action: no state can pay it

// Availability of a non-R action (App. B.3 Eq. available-recovery-actions;
// non-R actions with non-positive utility are excluded, App. B.2): verified,
// allowed by the retained representation q (H keeps everything, L excludes
// H, R allows only R), and finite non-negative costs.
__device__ bool action_ok(int act, uint8_t q, uint8_t verified, double tau, double dm,
                          double risk) {
  if (((verified >> act) & 1u) == 0) return false;
  if (q == kActL && act == kActH) return false;
  if (q != kActH && q != kActL) return false;
  if (!(tau > 0.0) || !isfinite(tau)) return false;
  if (!(dm >= 0.0) || !isfinite(dm)) return false;
  if (!(risk >= 0.0) || !isfinite(risk)) return false;
  return true;
}

// Integer cost on a grid of n intervals over `budget` (Eq.
// allocation-integer-costs): ceil(cost / h) with h = budget / n, or n + 1
// (does not fit) beyond n; with a zero budget only a zero cost fits.
__device__ int64_t grid_cost(double cost, double budget, int n) {
  if (!(budget > 0.0)) return cost == 0.0 ? 0 : (int64_t)n + 1;
  const double h = budget / (double)n;
  const double c = ceil(cost / h);
  return c > (double)n ? (int64_t)n + 1 : (int64_t)c;
}

__device__ AllocUnitCost unit_cost(const AllocArgs &a, int u) {
  const uint8_t q = a.q[u], v = a.verified[u];
  const double tau_h = a.tau_h[u], tau_l = a.tau_l[u], dm_h = a.dm_h[u], dm_l = a.dm_l[u];
  const double psi = a.psi[u];
  int ok_h = action_ok(kActH, q, v, tau_h, dm_h, 0.0);
  int ok_l = action_ok(kActL, q, v, tau_l, dm_l, psi) && a.delta_b > 0.0;
  const int64_t b_h = ok_h ? grid_cost(dm_h, a.m_res, a.n_b) : 0;
  const int64_t b_l = ok_l ? grid_cost(dm_l, a.m_res, a.n_b) : 0;
  const int64_t r_l = ok_l ? grid_cost(psi, a.delta_b, a.n_d) : 0;
  if (b_h > a.n_b) ok_h = 0;
  if (b_l > a.n_b || r_l > a.n_d) ok_l = 0;
  AllocUnitCost c;
  c.b_h = ok_h ? (int32_t)b_h : 0;
  c.r_h = ok_h ? 0 : kNever;
  c.b_l = ok_l ? (int32_t)b_l : 0;
  c.r_l = ok_l ? (int32_t)r_l : kNever;
  c.reach = 0;
  c.tau_h = tau_h;
  c.tau_l = tau_l;
  return c;
}

// Before the DP, in one launch.  Workgroup 0: the integer costs of every unit
// and the memory cost reach after it, i.e. the running sum, in unit order, of
// the largest memory cost of each unit's available actions, capped at KB - 1
// (a scan per chunk of 1024 units plus a carry): no state after unit i has a
// memory cost above uc[i].reach.  The other workgroups: F_0, which is 0 at
// (0, 0) and -inf elsewhere (padding cells included), and the second table all
// -inf (a DP launch skips the waves whose cells lie beyond the reach, which must
// then read as unreachable in either table); the guard cell holds -inf.
constexpr int kSetupThreads = 1024;
constexpr int kSetupCells = 4 * kSetupThreads;  // cells of each table per workgroup
__global__ __launch_bounds__(kSetupThreads) void setup_kernel(const AllocArgs a, AllocUnitCost *uc,
                                                              int KB, double *f0, double *f1,
                                                              int64_t cells, double *guard) {
  __shared__ int part[kSetupThreads];
  const int tid = (int)threadIdx.x;
  if (blockIdx.x > 0) {
    const int64_t c0 = (int64_t)(blockIdx.x - 1) * kSetupCells + tid;
#pragma unroll
    for (int i = 0; i < kSetupCells / kSetupThreads; ++i) {
      const int64_t cell = c0 + i * kSetupThreads;
      if (cell < cells) {
        f0[cell] = cell == 0 ? 0.0 : -INFINITY;
        f1[cell] = -INFINITY;
      }
    }
    return;
  }
  if (tid == 0) *guard = -INFINITY;
  int carry = 0;
  for (int base = 0; base < a.U; base += kSetupThreads) {
    const int i = base + tid;
    AllocUnitCost c{};
    if (i < a.U) c = unit_cost(a, i);
    const int v = max(c.b_h, c.b_l);  // 0 for an action that is not available, each at most KB
    part[tid] = v;
    __syncthreads();
    for (int off = 1; off < kSetupThreads; off <<= 1) {
      const int t = tid >= off ? part[tid - off] : 0;
      __syncthreads();
      part[tid] += t;  // at most 1024 * KB: no overflow for KB <= 4097
      __syncthreads();
    }
    c.reach = min(KB - 1, carry + part[tid]);
    if (i < a.U) uc[i] = c;
    carry = min(KB, carry + part[kSetupThreads - 1]);
    __syncthreads();
  }
}

// The larger of two values; a NaN (-inf plus the tau of an unavailable action,
// which may be anything) loses.  No value here is a signalling NaN or -0.
__device__ __forceinline__ double max_f64(double a, double b) {
  double r;
  asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}

constexpr int ipow3(int n) { return n == 0 ? 1 : 3 * ipow3(n - 1); }

// F after the N consecutive units uc[0 .. N-1] from the table before them, and
// the records of all N: bit for bit what N single-unit launches would write
// (every value is formed by the same fp64 additions and comparisons in the same
// order: actions R, H, L, each replacing the incumbent only when strictly
// larger); the tables in between are never stored.  One thread per cell; a cell
// combines up to 3^N cells of the table before, one per choice of actions
// ("source"), each the same shift for the whole wave, so a source that no action
// or no row can provide costs a scalar branch.  All loads are requested before
// any is used.
// What bounds a launch is the round trip of the table through the memory behind
// the L2s (17.8 MB, cold in every launch) on top of the launch itself: 6.3 us a
// pair of units on the 1025 x 1025 grid, of which 2.8 are left on a grid a
// sixteenth of it.  With a 64-bit division, a branch and a wait per source the
// chain of dependent loads came on top (7.2 us).  A call with 196 units takes 653
// us.  Measured and not better, in us more of that call: 3 units a launch (27
// sources: 75; better only on small grids), one unit (320), 2, 3 or 6 chunks a
// wave (200 to 530: longer code, fetched cold by every launch), workgroups of 128
// and 1024 threads.
template <int N>
__global__ __launch_bounds__(kDpThreads) void dpn_kernel(
    const double *__restrict__ prev, double *__restrict__ cur, uint64_t *__restrict__ pred,
    const AllocUnitCost *__restrict__ uc, uint32_t pred_words_per_unit, uint32_t chunks,
    uint32_t chunk_recip, uint32_t n, int KB, int KD, uint32_t guard) {
  const uint32_t x = blockIdx.x & 7u, q = n >> 3, rem = n & 7u;
  const uint32_t bid = x * q + (x < rem ? x : rem) + (blockIdx.x >> 3);
  const int lane = (int)threadIdx.x & (kWave - 1);
  // this wave's 64-cell chunk, its row k and first column j0
  const uint32_t w = bid * (kDpThreads / kWave) +
                     (uint32_t)__builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
  const int k = (int)(chunks == 1 ? w : __umulhi(w, chunk_recip));
  const int j0 = (int)(w - (uint32_t)k * chunks) * kWave;
  AllocUnitCost c[N];
#pragma unroll
  for (int m = 0; m < N; ++m) {
    c[m] = uc[m];
    // all of it now, not behind the branches below
    asm volatile("" ::"s"(c[m].b_h), "s"(c[m].r_h), "s"(c[m].b_l), "s"(c[m].r_l),
                 "s"(c[m].reach), "s"(c[m].tau_h), "s"(c[m].tau_l));
  }
  if (k >= KD) return;
  // A wave (64 consecutive cells of one row) wholly beyond the memory cost
  // reach after the group holds only unreachable states: they stay -inf in
  // both tables, and no path the backtrack follows passes through them, so
  // neither their values nor their records are written.
  if (j0 > c[N - 1].reach) return;
  const int j = j0 + lane < KB ? j0 + lane : -1;  // padding cells: nothing leads here
  const uint32_t cell8 = (w * kWave + (uint32_t)lane) * 8u;  // byte offset of this cell

  // source s: unit m takes action (s / 3^m) % 3; a lane without it reads the
  // guard cell, which holds -inf
  constexpr int kSrc = ipow3(N);
  const __amdgpu_buffer_rsrc_t table = __builtin_amdgcn_make_buffer_rsrc(
      (void *)prev, 0, (int)(guard + 8u), 0x00020000);
  double none = -INFINITY;
  asm("" : "+s"(none));
  double f[kSrc];
#pragma unroll
  for (int s = 0; s < kSrc; ++s) {
    int db = 0, dk = 0;
#pragma unroll
    for (int m = 0; m < N; ++m) {
      const int act = s / ipow3(m) % 3;
      if (act == kActH) db += c[m].b_h, dk += c[m].r_h;
      if (act == kActL) db += c[m].b_l, dk += c[m].r_l;
    }
    f[s] = none;
    if (s == 0 || dk <= k) {  // the same for the whole wave
      const uint32_t from = cell8 - ((uint32_t)dk * chunks * kWave + (uint32_t)db) * 8u;
      f[s] = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(
                                            table, (int)(j >= db ? from : guard), 0, 0));
    }
  }
  uint64_t lo[N], hi[N];  // records: bit 0 and 1 of the action, one bit per lane
#pragma unroll
  for (int m = 0; m < N; ++m)
#pragma unroll
    for (int t = 0; t < ipow3(N - 1 - m); ++t) {
      const double r = f[3 * t];
      const double vh = f[3 * t + 1] + c[m].tau_h, vl = f[3 * t + 2] + c[m].tau_l;
      const double rh = max_f64(r, vh);
      if (t == 0) {  // the record of the cell itself
        hi[m] = __ballot(vl > rh);
        lo[m] = __ballot(vh > r) & ~hi[m];
      }
      f[t] = max_f64(rh, vl);
    }
  // Written through at device scope: a table left dirty in the L2s is flushed at
  // the launch's end, with every CU idle (52 us more of a call with 196 units).
  __hip_atomic_store(reinterpret_cast<double *>(reinterpret_cast<char *>(cur) + cell8), f[0],
                     __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (lane == 0) {
#pragma unroll
    for (int m = 0; m < N; ++m)
      *reinterpret_cast<u64x2 *>(pred + (m * pred_words_per_unit + 2u * w)) = u64x2{lo[m], hi[m]};
  }
}

// The better of two terminal candidates: larger value, then the earlier cell
// in (risk cost, memory cost) order, which is lower risk, then lower memory.
__device__ __forceinline__ bool better(double v, int64_t i, double bv, int64_t bi) {
  return v > bv || (v == bv && i < bi);
}

struct Best {
  double v;
  int64_t i;
};

template <int THREADS>
__device__ Best block_best(Best b) {
  __shared__ double sv[THREADS];
  __shared__ int64_t si[THREADS];
  sv[threadIdx.x] = b.v;
  si[threadIdx.x] = b.i;
  __syncthreads();
  for (int off = THREADS / 2; off > 0; off >>= 1) {
    if ((int)threadIdx.x < off && better(sv[threadIdx.x + off], si[threadIdx.x + off],
                                         sv[threadIdx.x], si[threadIdx.x])) {
      sv[threadIdx.x] = sv[threadIdx.x + off];
      si[threadIdx.x] = si[threadIdx.x + off];
    }
    __syncthreads();
  }
  return Best{sv[0], si[0]};
}

__global__ __launch_bounds__(kDpThreads) void terminal_partial_kernel(const double *f,
                                                                       int64_t cells,
                                                                       Best *partial) {
  Best b{-INFINITY, INT64_MAX};
  for (int64_t i = (int64_t)blockIdx.x * kDpThreads + threadIdx.x; i < cells;
       i += (int64_t)gridDim.x * kDpThreads) {
    const double v = f[i];
    if (better(v, i, b.v, b.i)) b = Best{v, i};
  }
  b = block_best<kDpThreads>(b);
  if (threadIdx.x == 0) partial[blockIdx.x] = b;
}

// Action of unit `unit` recorded at cell (j, k).
__device__ __forceinline__ int record(const uint64_t *pred, int64_t unit, int64_t k, int64_t j,
                                      int KD, int64_t chunks) {
  const int64_t w = (unit * KD + k) * chunks + j / kWave;
  const int bit = (int)(j % kWave);
  return (int)((pred[2 * w] >> bit) & 1u) | ((int)((pred[2 * w + 1] >> bit) & 1u) << 1);
}

__device__ __forceinline__ int lane_int(int v, int lane) {
  return __builtin_amdgcn_readlane(v, lane);
}

__device__ __forceinline__ double lane_f64(double v, int lane) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)u, lane);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), lane);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// Memory and risk of the chosen actions, summed in unit order (one wave:
// the inputs of 64 units are loaded at once, one chunk ahead, and the
// additions stay sequential).  A unit whose action adds nothing adds +0.0,
// which leaves the sums unchanged: they start at +0.0 and every chosen cost
// is finite and non-negative, so neither sum is ever -0.0.
struct UnitTotals {
  double mem, risk;
};

__device__ __forceinline__ UnitTotals unit_costs(const AllocArgs &a, int u) {
  UnitTotals c{0.0, 0.0};
  if (u < a.U) {
    const int act = a.action[u];
    if (act == kActH) c.mem = a.dm_h[u];
    if (act == kActL) {
      c.mem = a.dm_l[u];
      c.risk = a.psi[u];
    }
  }
  return c;
}

__device__ __forceinline__ void sum_chosen(const AllocArgs &a, int lane) {
  double mem = 0.0, risk = 0.0;
  UnitTotals c = unit_costs(a, lane);
  for (int base = 0; base < a.U; base += kWave) {
    const UnitTotals next = unit_costs(a, base + kWave + lane);
    // all 64 lanes, unrolled (constant lane indices): lanes past the last
    // unit hold +0.0, which leaves the sums unchanged
#pragma unroll
    for (int t = 0; t < kWave; ++t) {
      mem += lane_f64(c.mem, t);
      risk += lane_f64(c.risk, t);
    }
    c = next;
  }
  if (lane == 0) {
    a.totals[1] = mem;
    a.totals[2] = risk;
  }
}

// Backtracking, one wave.  The record of unit i at the current cell decides
// where the record of unit i - 1 is read, so a walk of one unit per step is
// a chain of dependent loads.  Each round trip instead loads the records of
// units i .. i - 3 at every cell the path can reach from the current one
// (1 + 3 + 9 + 27 = 40 cells, one lane each; lane 1 + 3 + ... + 3^(d-1) + p
// holds the record of unit i - d after the actions whose base-3 digits,
// unit i first, spell p; actions R, H, L are 0, 1, 2) and resolves the four
// actions from registers.  Lanes 0..3 carry the costs of units i .. i - 3
// and fetch those of the next four units during the same round trip.
constexpr int kLookUnits = 4;
constexpr int kLookLanes = 40;

__global__ __launch_bounds__(kFinalThreads) void terminal_backtrack_kernel(
    const AllocArgs a, const Best *partial, int n_partial, const uint64_t *pred,
    const AllocUnitCost *uc, int S, int KD) {
  Best b{-INFINITY, INT64_MAX};
  for (int p = threadIdx.x; p < n_partial; p += kFinalThreads)
    if (better(partial[p].v, partial[p].i, b.v, b.i)) b = partial[p];
  b = block_best<kFinalThreads>(b);
  if (threadIdx.x >= kWave) return;
  const int lane = (int)threadIdx.x;
  int64_t k = b.i / S, j = b.i % S;
  if (lane == 0) {
    a.jk[0] = j;
    a.jk[1] = k;
    a.totals[0] = b.v;
  }
  const int64_t chunks = S / kWave;
  // this lane's depth d and path p, and the base-3 digits of p (unit i's
  // action first)
  const int d = lane == 0 ? 0 : lane < 4 ? 1 : lane < 13 ? 2 : 3;
  const int p = lane - (d == 0 ? 0 : d == 1 ? 1 : d == 2 ? 4 : 13);
  int digit[3];
  {
    int rest = p, pw = d == 3 ? 9 : d == 2 ? 3 : 1;
#pragma unroll
    for (int m = 0; m < 3; ++m) {
      digit[m] = m < d ? rest / pw : kActR;
      if (m < d) {
        rest -= digit[m] * pw;
        pw /= 3;
      }
    }
  }
  // Every load below is issued unconditionally (a lane with nothing to load
  // reads a valid dummy address and discards the value), so that no branch
  // forces a wait: the costs of the next four units are waited for only in
  // the next round trip, and the record load is the one latency per trip.
  const bool cost_lane = lane < kLookUnits;
  auto load_costs = [&](int unit, int &bh, int &bl, int &rl) {
    const bool ok = cost_lane && unit - lane >= 0;
    const AllocUnitCost &c = uc[ok ? unit - lane : 0];
    const int h = c.b_h, l = c.b_l, r = c.r_l;
    bh = ok ? h : 0;
    bl = ok ? l : 0;
    rl = ok ? r : 0;
  };
  int bh, bl, rl;
  load_costs(a.U - 1, bh, bl, rl);
  for (int i = a.U - 1; i >= 0; i -= kLookUnits) {
    int nbh, nbl, nrl;
    load_costs(i - kLookUnits, nbh, nbl, nrl);
    // the cell of this lane's record: the current cell minus the costs of
    // the actions its path takes at units i .. i - d + 1
    int64_t jj = j, kk = k;
#pragma unroll
    for (int m = 0; m < 3; ++m) {
      const int ubh = lane_int(bh, m), ubl = lane_int(bl, m), url = lane_int(rl, m);
      if (digit[m] == kActH) jj -= ubh;
      if (digit[m] == kActL) {
        jj -= ubl;
        kk -= url;
      }
    }
    const bool rec = lane < kLookLanes && i - d >= 0 && jj >= 0 && kk >= 0;
    const int r = record(pred, rec ? i - d : 0, rec ? kk : 0, rec ? jj : 0, KD, chunks);
    const int act = rec ? r : kActR;
    const int a0 = lane_int(act, 0);
    const int a1 = lane_int(act, 1 + a0);
    const int a2 = lane_int(act, 4 + 3 * a0 + a1);
    const int a3 = lane_int(act, 13 + 9 * a0 + 3 * a1 + a2);
    const int mine = lane == 0 ? a0 : lane == 1 ? a1 : lane == 2 ? a2 : a3;
    if (lane < kLookUnits && i - lane >= 0) a.action[i - lane] = (uint8_t)mine;
    const int acts[4] = {a0, a1, a2, a3};
#pragma unroll
    for (int m = 0; m < kLookUnits; ++m) {
      const int ubh = lane_int(bh, m), ubl = lane_int(bl, m), url = lane_int(rl, m);
      if (i - m >= 0) {
        if (acts[m] == kActH) j -= ubh;
        if (acts[m] == kActL) {
          j -= ubl;
          k -= url;
        }
      }
    }
    bh = nbh;
    bl = nbl;
    rl = nrl;
  }
  __threadfence_block();  // the actions are read back by other lanes
  sum_chosen(a, lane);
}

}  // namespace

AllocLayout alloc_layout(int U, int KB, int KD) {
  auto up = [](size_t x) { return (x + 255) & ~size_t(255); };
  AllocLayout l{};
  l.S = (KB + kWave - 1) / kWave * kWave;
  l.cells = (int64_t)l.S * KD;
  l.off_costs = 0;
  l.off_f0 = up(sizeof(AllocUnitCost) * (size_t)(U > 0 ? U : 1));
  l.off_f1 = l.off_f0 + up(sizeof(double) * (size_t)l.cells);
  l.off_partial = l.off_f1 + up(sizeof(double) * (size_t)l.cells);
  l.off_pred = l.off_partial + up(sizeof(Best) * kPartials);
  l.pred_bytes_per_unit = (size_t)(l.cells / kWave) * 16;
  l.bytes = l.off_pred + up(l.pred_bytes_per_unit * (size_t)U);
  return l;
}

hipError_t launch_allocate(const AllocArgs &a, int KB, int KD, void *workspace, hipStream_t s) {
  const AllocLayout l = alloc_layout(a.U, KB, KD);
  char *ws = static_cast<char *>(workspace);
  AllocUnitCost *uc = reinterpret_cast<AllocUnitCost *>(ws + l.off_costs);
  double *f[2] = {reinterpret_cast<double *>(ws + l.off_f0),
                  reinterpret_cast<double *>(ws + l.off_f1)};
  Best *partial = reinterpret_cast<Best *>(ws + l.off_partial);
  uint64_t *pred = reinterpret_cast<uint64_t *>(ws + l.off_pred);

  const int setup_grid = 1 + (int)((l.cells + kSetupCells - 1) / kSetupCells);
  hipLaunchKernelGGL(setup_kernel, dim3(setup_grid), dim3(kSetupThreads), 0, s, a, uc, KB, f[0],
                     f[1], l.cells, reinterpret_cast<double *>(partial));
  const int grid = (int)((l.cells + kDpThreads - 1) / kDpThreads);
  auto pred_of = [&](int i) {
    return reinterpret_cast<uint64_t *>(reinterpret_cast<char *>(pred) +
                                        l.pred_bytes_per_unit * (size_t)i);
  };
  // units in groups of kDpGroup (one launch each), the rest in a smaller
  // group; the table after launch t lives in f[t & 1]
  const uint32_t words = (uint32_t)(l.pred_bytes_per_unit / sizeof(uint64_t));
  // w / chunks = mulhi(w, recip) for every chunk w of a table (at most 2^19 of
  // them and 65 a row, so w < 2^32 / chunks)
  const uint32_t chunks = (uint32_t)(l.S / kWave);
  const uint32_t recip = (uint32_t)((uint64_t(1) << 32) / chunks + 1);
  int t = 0;
  for (int i = 0; i < a.U; i += kDpGroup, ++t) {
    const int g = a.U - i < kDpGroup ? a.U - i : kDpGroup;
    const dim3 gd(grid), bd(kDpThreads);
    const uint32_t guard = (uint32_t)(l.off_partial - (t & 1 ? l.off_f1 : l.off_f0));
    double *src = f[t & 1], *dst = f[(t + 1) & 1];
    uint64_t *pr = pred_of(i);
    auto launch = [&](auto kernel) {
      hipLaunchKernelGGL(kernel, gd, bd, 0, s, src, dst, pr, uc + i, words, chunks, recip,
                         (uint32_t)grid, KB, KD, guard);
    };
    static_assert(kDpGroup == 2);
    if (g == 2) launch(dpn_kernel<2>);
    else launch(dpn_kernel<1>);
  }
  const int n_partial = grid < kPartials ? grid : kPartials;
  hipLaunchKernelGGL(terminal_partial_kernel, dim3(n_partial), dim3(kDpThreads), 0, s,
                     f[t & 1], l.cells, partial);
  hipLaunchKernelGGL(terminal_backtrack_kernel, dim3(1), dim3(kFinalThreads), 0, s, a, partial,
                     n_partial, pred, uc, l.S, KD);
  return hipGetLastError();
}

}  // namespace hilore
