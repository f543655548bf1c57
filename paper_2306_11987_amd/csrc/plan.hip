// Leverage-score sampling of the bit-split gradient rows and the GEMM operands it
// selects (gfx950).
//
// lss_plan (one workgroup per problem: 1024 threads, 256 for N <= 4096).  Its inputs are
// the integer leverage scores of the 2N stacked rows, formed by the bit-split kernel
// (Sec. 4.2: with the common factor
// s_dn s_x dropped, c^2 = w^2 sum q^2 x_sumsq, w = 14 for the upper row of a token and 1
// for the lower one, c = isqrt(c^2 2^16)), and that kernel's per-workgroup totals:
//   1. inclusion probabilities by the clamp-and-rescale loop of App. A.2 with sum p = B,
//      in exact integers.  Thresholds S/R only fall from one round to the next, so the
//      rows clamped after a round are exactly {c > 0 : R c >= S} for that round's (R, S):
//      a round needs that set's count and sum, one pass over the scores, and no per-row
//      state.  If no more than B rows have c > 0, every such row has p = 1 (the
//      "keep rows with norm > 0" rule of the paper's implementation, App. A.6);
//   2. upper rows are kept iff non-zero; a lower row with p* < 1 gets p~ = 2^-e >= p*, the
//      smallest power of two (e <= 4, e <= 2 if the token's upper row is non-zero), and is
//      kept iff u16 < 2^(16-e) (Philox stream 1), weight m/p~ = 2^e;
//   3. kept tokens (w_up + w_dn > 0) are compacted in ascending order: each thread owns 8
//      consecutive tokens per round of 8192 (vector loads and stores, one Philox block),
//      and a block-wide scan of the per-thread counts places them.
//
// build_operands materialises, for the kept tokens only, the weighted integer
// rows A_t = 14 w_up q_up[t] + w_dn q_dn[t] (|A| <= 126, one int8 operand that carries the
// bit split and the 1/p factors together; the dX GEMM reads it K-contiguous, the dW GEMM
// k-major through transposing LDS reads) and the gathered X^ rows, transposed to the
// K-contiguous layout the dW GEMM reads.  The int8 operand uses the "K-interleaved" byte
// order of the GEMM: inside every group of 8 consecutive k the bytes hold
// k = 0,2,4,6,1,3,5,7, the order in which a packed INT4 word unpacks for free.
#include "common.h"
#include "launch.h"

namespace hqlss {

namespace {

// Workgroup sizes of the sampler: 1024 threads, or 256 for short sequences (N <= 4096),
// where four samplers then share a CU (a batched call runs one per batch).  The result
// does not depend on the size: counters are per 8 tokens and every sum is exact.
constexpr int kPlanThreads = 1024;
constexpr int kPlanThreadsSmall = 256;

// Sum of a 32-bit value over the wave (every lane gets it): DPP adds inside each row of
// 16 lanes (swap neighbours, swap pairs, mirror halves, mirror the row), then the four row
// sums read as scalars.  Needs every lane of the wave active.
__device__ __forceinline__ uint32_t wave_sum_u32_dpp(uint32_t v) {
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, true);   // quad_perm 1,0,3,2
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, true);   // quad_perm 2,3,0,1
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xF, 0xF, true);  // row_half_mirror
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x140, 0xF, 0xF, true);  // row_mirror
  return (uint32_t)__builtin_amdgcn_readlane((int)v, 0) + (uint32_t)__builtin_amdgcn_readlane((int)v, 16) +
         (uint32_t)__builtin_amdgcn_readlane((int)v, 32) + (uint32_t)__builtin_amdgcn_readlane((int)v, 48);
}

// The same over the first 16 lanes only.
__device__ __forceinline__ uint32_t row16_sum_u32_dpp(uint32_t v) {
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, true);
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, true);
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xF, 0xF, true);
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x140, 0xF, 0xF, true);
  return (uint32_t)__builtin_amdgcn_readlane((int)v, 0);
}

// 64-bit wave sum as three 21-bit limbs (64 limbs of at most 22 bits stay below 2^28, so
// each limb sum is exact in 32 bits), recombined modulo 2^64.
__device__ __forceinline__ uint64_t wave_sum_u64_dpp(uint64_t v) {
  constexpr uint64_t kM21 = (1ull << 21) - 1;
  const uint32_t s0 = wave_sum_u32_dpp((uint32_t)(v & kM21));
  const uint32_t s1 = wave_sum_u32_dpp((uint32_t)((v >> 21) & kM21));
  const uint32_t s2 = wave_sum_u32_dpp((uint32_t)(v >> 42));
  return (uint64_t)s0 + ((uint64_t)s1 << 21) + ((uint64_t)s2 << 42);
}

__device__ __forceinline__ uint64_t row16_sum_u64_dpp(uint64_t v) {
  constexpr uint64_t kM21 = (1ull << 21) - 1;
  const uint32_t s0 = row16_sum_u32_dpp((uint32_t)(v & kM21));
  const uint32_t s1 = row16_sum_u32_dpp((uint32_t)((v >> 21) & kM21));
  const uint32_t s2 = row16_sum_u32_dpp((uint32_t)(v >> 42));
  return (uint64_t)s0 + ((uint64_t)s1 << 21) + ((uint64_t)s2 << 42);
}

// Inclusive prefix sum over the wave by DPP (shifts inside each row of 16 lanes, then the
// rows' last lanes broadcast to the rows after them).  Needs every lane of the wave active.
__device__ __forceinline__ uint32_t wave_scan_u32_dpp(uint32_t v) {
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xF, 0xF, true);  // row_shr 1
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xF, 0xF, true);  // row_shr 2
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xF, 0xF, true);  // row_shr 4
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xF, 0xF, true);  // row_shr 8
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xA, 0xF, false);  // row_bcast 15, rows 1 and 3
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xC, 0xF, false);  // row_bcast 31, rows 2 and 3
  return v;
}

// floor(S / R) for 0 < R < 2^18 and S < 2^50, and the remainder: the quotient from a
// reciprocal refined to double precision is off by at most one, which the exact remainder
// corrects (a dozen instructions in a row instead of the 64-bit division's hundred and fifty).
__device__ __forceinline__ uint64_t quotient(uint64_t S, uint32_t R, uint64_t& rem) {
  const double d = (double)R;
  double r = __builtin_amdgcn_rcp(d);
  r = __builtin_fma(__builtin_fma(-d, r, 1.0), r, r);
  r = __builtin_fma(__builtin_fma(-d, r, 1.0), r, r);
  uint64_t q = (uint64_t)((double)S * r);
  int64_t m = (int64_t)(S - q * R);
  if (m < 0) { --q; m += R; }
  if (m >= (int64_t)R) { ++q; m -= R; }
  rem = (uint64_t)m;
  return q;
}

// 8 consecutive words from p + t0 (n8 of them valid, the rest 0).
__device__ __forceinline__ void load8u(const uint32_t* p, int t0, int n8, uint32_t v[8]) {
  if (n8 == 8) {
    const uint4 a = *reinterpret_cast<const uint4*>(p + t0), b = *reinterpret_cast<const uint4*>(p + t0 + 4);
    v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
    v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
  } else {
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = j < n8 ? p[t0 + j] : 0u;
  }
}

// What bounds it is latency: one workgroup (per problem) and a chain of dependent loads,
// rounds and barriers on one CU.  So:
//   - the loads of a problem of up to 16 tokens per thread are issued before the first is
//     used (8 consecutive tokens per thread and group, as 16-byte pieces);
//   - a clamp-and-rescale round is one pass over registers that counts by scalar popcounts
//     of the comparison masks; what is the same for all (the sums over the waves, the
//     quotient S / R) is formed by the first wave alone, the others waiting: in every wave
//     it cost four times its instructions, 16 waves sharing four SIMDs;
//   - R c >= S and R c 2^e <= S are comparisons of c with quotients formed once;
//   - the kept list is compacted in LDS and leaves in whole lines (8 scattered words a thread
//     before).
// N = 128 (five rounds): 11.3 -> 8.6 us; N = 16384, lognormal rows, budget N (no round), event
// times: 11.5 -> 9.0 us; Pareto rows (eight rounds): 37.9 -> 23.7 us.
template <int THREADS>
__global__ __launch_bounds__(THREADS) void lss_plan_kernel(
    const int32_t* __restrict__ sumsq_up, const uint32_t* __restrict__ scores, int64_t pitch,
    const uint4* __restrict__ parts, int nparts, int N, int64_t B, uint64_t seed,
    uint64_t offset, uint8_t* __restrict__ w_up, uint8_t* __restrict__ w_dn,
    int32_t* __restrict__ kept, int32_t* __restrict__ n_kept, uint64_t offset_stride) {
  constexpr int WAVES = THREADS / kWave;
  static_assert(WAVES <= 16, "the waves' sums are combined by one row of 16 lanes");
  struct Ctl {
    uint64_t T, F;  // ceil(S / R) and floor(S / R) of the round, saturated where R = 0
    int done, all;
  };
  struct WaveSum {
    uint32_t n;
    uint64_t sum;
  };
  __shared__ Ctl ctl;
  __shared__ WaveSum red[WAVES];
  __shared__ uint32_t wtot[WAVES];    // kept tokens of each wave, two groups packed
  __shared__ int32_t kept_s[16 * THREADS];
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  {  // workgroup b samples batch b of a batched call (its own inputs, outputs and counters)
    const int64_t bt = blockIdx.x;
    sumsq_up += bt * N;
    scores += bt * 2 * pitch;
    parts += bt * nparts;
    w_up += bt * N;
    w_dn += bt * N;
    kept += bt * N;
    n_kept += bt;
    offset += (uint64_t)bt * offset_stride;
  }
  const uint32_t* cup = scores;
  const uint32_t* cdn = scores + pitch;
  const uint32_t* sup = reinterpret_cast<const uint32_t*>(sumsq_up);

  // up to 16 tokens per thread (two groups of 8 consecutive ones) stay in registers
  const bool in_regs = N <= 16 * THREADS;
  int t0[2] = {0, 0}, n8[2] = {0, 0};
  uint32_t su[2][8], cu[2][8], cd[2][8];
  if (in_regs) {
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      t0[r] = r * 8 * THREADS + 8 * tid;
      n8[r] = t0[r] < N ? (N - t0[r] < 8 ? N - t0[r] : 8) : 0;
      load8u(cdn, t0[r], n8[r], cd[r]);
      load8u(sup, t0[r], n8[r], su[r]);
      load8u(cup, t0[r], n8[r], cu[r]);
    }
  }

  // App. A.2 clamp-and-rescale: k rows clamped so far, R = B - k and S the sum of the
  // others' scores.  R c >= S  <=>  c >= ceil(S / R) for integers and R > 0; S = 0 admits
  // every non-zero score, R = 0 with S > 0 none.  The first wave holds the state.
  uint64_t S_all = 0, S = 0;
  int64_t k = 0;
  uint64_t rT = 1, rF = 0;  // ceil(S / R) and floor(S / R)
  // Both are formed before either is assigned, once each and by selection: assigned in three
  // branches, through the captured references, the state lived in private memory.
  auto set_round = [&]() {
    const int64_t R = B - k;
    uint64_t rem;
    const uint64_t F = quotient(S, R > 0 ? (uint32_t)R : 1u, rem), T = F + (rem ? 1 : 0);
    const bool none = R <= 0;
    rT = S == 0 ? 1 : none ? ~uint64_t(0) : T;
    rF = S == 0 ? 0 : none ? ~uint64_t(0) : F;
  };
  if (wid == 0) {  // totals of the bit-split workgroups: non-zero rows and the score sum
    uint32_t nz = 0;
    uint64_t st = 0;
    // four loads in flight (one after the other, as the remainder of an unrolled loop, 256
    // partials took 1 us more)
    for (int i = lane; i < nparts; i += 4 * 64) {
      uint4 p[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) p[q] = parts[i + 64 * q < nparts ? i + 64 * q : i];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const bool in = i + 64 * q < nparts;
        nz += in ? p[q].x : 0u;
        st += in ? ((uint64_t)p[q].z << 32) | p[q].y : 0ull;
      }
    }
    nz = wave_sum_u32_dpp(nz);
    S = S_all = wave_sum_u64_dpp(st);
    const bool all = (int64_t)nz <= B;  // T = 1 clamps every non-zero row
    if (!all) set_round();
    if (lane == 0) ctl = {rT, rF, 0, all};
  }
  __syncthreads();
  const bool all_nonzero_kept = ctl.all;
  if (!all_nonzero_kept) {
    const int64_t n2 = 2 * (int64_t)N;
    // upper scores of each group of tokens not counted for good yet: their number in the
    // wave; thresholds only fall, so once all of them are clamped they stay so, and the
    // count and sum carry over (most upper rows are zero, the others large)
    uint32_t up[2] = {0u, 0u}, n_up = 0;
    uint64_t s_up = 0;
    if (in_regs) {
#pragma unroll
      for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int j = 0; j < 8; ++j) up[r] += (uint32_t)__builtin_popcountll(__ballot(cu[r][j] != 0));
    }
    auto pass = [&](uint64_t T, uint32_t& n, uint64_t& sum) {  // n: of the wave, sum: of the thread
      // T >= 1, so c >= T implies c > 0; a threshold past the 32-bit scores admits none
      const uint32_t T32 = (uint32_t)T;
      n = n_up;
      sum = s_up;
      if (T > 0xFFFFFFFFull) return;  // uniform; no upper row has been clamped then
      auto take = [&](uint32_t c, uint32_t& m, uint64_t& v) {
        const bool in = c >= T32;
        m += (uint32_t)__builtin_popcountll(__ballot(in));
        v += in ? c : 0u;
      };
      if (in_regs) {
#pragma unroll
        for (int r = 0; r < 2; ++r) {
          if (r == 1 && N <= 8 * THREADS) break;  // uniform: no second group
#pragma unroll
          for (int j = 0; j < 8; ++j) take(cd[r][j], n, sum);
          if (up[r]) {
            uint32_t m = 0;
            uint64_t v = 0;
#pragma unroll
            for (int j = 0; j < 8; ++j) take(cu[r][j], m, v);
            n += m;
            sum += v;
            if (m == up[r]) {
              up[r] = 0;
              n_up += m;
              s_up += v;
            }
          }
        }
      } else {  // eight loads in flight per thread
        for (int64_t i0 = wid * 64; i0 < n2; i0 += 8 * (int64_t)THREADS) {  // uniform
          uint32_t c8[8];
#pragma unroll
          for (int u = 0; u < 8; ++u) {
            const int64_t i = i0 + lane + (int64_t)u * THREADS;
            c8[u] = i < n2 ? scores[i < N ? i : pitch + (i - N)] : 0u;
          }
#pragma unroll
          for (int u = 0; u < 8; ++u) take(c8[u], n, sum);
        }
      }
    };
    auto advance = [&](int64_t cnt, uint64_t sum) -> bool {  // first wave: the round's totals
      if (cnt == k) return true;  // nothing newly clamped
      S = S_all - sum;
      k = cnt;
      set_round();
      return false;
    };
    if (N <= 8 * kWave) {  // the first wave holds every token: no barrier
      if (wid == 0) {
        for (;;) {
          uint32_t n;
          uint64_t sum;
          pass(rT, n, sum);
          if (advance(n, wave_sum_u64_dpp(sum))) break;
        }
        if (lane == 0) ctl = {rT, rF, 1, 0};
      }
      __syncthreads();
    } else {
      for (;;) {
        uint32_t n;
        uint64_t sum;
        pass(ctl.T, n, sum);
        sum = wave_sum_u64_dpp(sum);
        if (lane == 0) red[wid] = {n, sum};
        __syncthreads();
        if (wid == 0) {
          const WaveSum p = lane < WAVES ? red[lane] : WaveSum{0u, 0u};
          const bool done = advance(row16_sum_u32_dpp(p.n), row16_sum_u64_dpp(p.sum));
          if (lane == 0) ctl = {rT, rF, done, 0};
        }
        __syncthreads();
        if (ctl.done) break;  // read before the barrier that precedes its next write
      }
    }
  }
  // a lower row is clamped (p = 1) for c >= T; else R c 2^i <= S  <=>  c <= floor(F / 2^i)
  const uint64_t T = ctl.T, F = ctl.F;
  const uint32_t T32 = T > 0xFFFFFFFFull ? 0xFFFFFFFFu : (uint32_t)T;
  const bool none = T > 0xFFFFFFFFull;  // no 32-bit score reaches T
  uint32_t Fi[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) Fi[i] = (F >> (i + 1)) > 0xFFFFFFFFull ? 0xFFFFFFFFu : (uint32_t)(F >> (i + 1));

  // weights and masks of 8 consecutive tokens; returns the mask of the kept ones
  auto weigh = [&](int t, int n, const uint32_t* su8, const uint32_t* cd8) -> uint32_t {
    // Bernoulli draws only when some row has p < 1 (uniform over the workgroup)
    const U4 rnd = all_nonzero_kept ? U4{0u, 0u, 0u, 0u}
                                    : philox_block(seed, offset, 1u, (uint64_t)t);
    uint32_t wu8[2] = {0u, 0u}, wd8[2] = {0u, 0u};
    uint32_t keepmask = 0;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const uint32_t c = cd8[j], wu = su8[j] ? 1u : 0u;
      uint32_t wd = 0;
      if (!none && c >= T32) {  // T >= 1: c > 0
        wd = 1;
      } else if (c) {
        uint32_t e = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) e += c <= Fi[i] ? 1u : 0u;
        const uint32_t cap = wu ? 2u : 4u;
        e = e < cap ? e : cap;
        wd = (u16_of(rnd, j) < (1u << (16 - e))) ? (1u << e) : 0u;
      }
      wu8[j >> 2] |= wu << (8 * (j & 3));
      wd8[j >> 2] |= wd << (8 * (j & 3));
      if (wu + wd) keepmask |= 1u << j;
    }
    if (n == 8) {
      *reinterpret_cast<uint2*>(w_up + t) = make_uint2(wu8[0], wu8[1]);
      *reinterpret_cast<uint2*>(w_dn + t) = make_uint2(wd8[0], wd8[1]);
    } else {
      for (int j = 0; j < n; ++j) {
        w_up[t + j] = (uint8_t)(wu8[j >> 2] >> (8 * (j & 3)));
        w_dn[t + j] = (uint8_t)(wd8[j >> 2] >> (8 * (j & 3)));
      }
    }
    return keepmask;
  };
  // The kept tokens of one or two groups, in order, into kept[base ...]: the counts of both
  // packed in one scan (at most 8 THREADS = 8192 each), the tokens placed in LDS.
  int base = 0;
  auto compact = [&](int ta, uint32_t ka, int tb, uint32_t kb) {
    const uint32_t mine = __builtin_popcount(ka) | (__builtin_popcount(kb) << 16);
    const uint32_t incl = wave_scan_u32_dpp(mine);
    if (lane == 63) wtot[wid] = incl;
    __syncthreads();
    const uint32_t w = lane < WAVES ? wtot[lane] : 0u;
    const uint32_t before = wave_sum_u32_dpp(lane < wid ? w : 0u), total = wave_sum_u32_dpp(w);
    const uint32_t excl = before + incl - mine;
    const int na = (int)(total & 0xFFFFu), nb = (int)(total >> 16);
    int pa = (int)(excl & 0xFFFFu), pb = na + (int)(excl >> 16);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      if ((ka >> j) & 1) kept_s[pa++] = ta + j;
      if ((kb >> j) & 1) kept_s[pb++] = tb + j;
    }
    __syncthreads();
    for (int i = tid; i < na + nb; i += THREADS) kept[base + i] = kept_s[i];
    base += na + nb;
  };
  if (in_regs) {
    const uint32_t ka = weigh(t0[0], n8[0], su[0], cd[0]);
    const uint32_t kb = N > 8 * THREADS ? weigh(t0[1], n8[1], su[1], cd[1]) : 0u;
    compact(t0[0], ka, t0[1], kb);
  } else {
    for (int r0 = 0; r0 < N; r0 += 8 * THREADS) {
      const int t = r0 + 8 * tid;
      const int n = t < N ? (N - t < 8 ? N - t : 8) : 0;
      uint32_t su8[8], cd8[8];
      load8u(sup, t, n, su8);
      load8u(cdn, t, n, cd8);
      const uint32_t ka = weigh(t, n, su8, cd8);
      compact(t, ka, 0, 0u);
      __syncthreads();  // the LDS copy is read before the next group fills it
    }
  }
  if (tid == 0) *n_kept = base;
}

__device__ __forceinline__ int sext4(uint32_t n) { return (int)(n ^ 8u) - 8; }

// 8 weighted values (k = 0..7) -> K-interleaved bytes: low word k = 0,2,4,6; high 1,3,5,7.
__device__ __forceinline__ uint2 interleave8(const int a[8]) {
  uint32_t lo = 0, hi = 0;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    lo |= ((uint32_t)a[2 * j] & 0xFFu) << (8 * j);
    hi |= ((uint32_t)a[2 * j + 1] & 0xFFu) << (8 * j);
  }
  return make_uint2(lo, hi);
}

__device__ __forceinline__ void weighted8(uint32_t up, uint32_t dn, int wu, int wd, int a[8]) {
#pragma unroll
  for (int j = 0; j < 8; ++j)
    a[j] = kBsRatio * wu * sext4((up >> (4 * j)) & 15u) + wd * sext4((dn >> (4 * j)) & 15u);
}

// One pass over the kept tokens builds every GEMM operand the sample selects: workgroup
// (x, y) takes kept indices [128 x, 128 x + 128) and one block of up to 128 columns (the
// last block of C or D may hold 64).  Blocks of the C columns read q_up, q_dn and the
// weights, form A_t and write it row-major into Ag (the operand of both gradient GEMMs);
// blocks of the D columns gather X^ rows and write them, through an LDS transpose,
// column-major into XtT.  Every row piece written is 128 bytes (64 for XtT), two full
// cache lines.  The last block row zeroes the rows of dX that belong to dropped tokens.
// Rows of Ag and columns of XtT between n_kept and the next multiple of 128 are written as
// zeros (the GEMMs read whole K steps).
constexpr int kBK = 128;  // kept indices per workgroup
constexpr int kBC = 128;  // columns per workgroup
template <int DT>
__global__ __launch_bounds__(256) void build_operands_kernel(
    const uint8_t* __restrict__ qup, const uint8_t* __restrict__ qdn,
    const uint8_t* __restrict__ w_up, const uint8_t* __restrict__ w_dn,
    const int32_t* __restrict__ kept, const int32_t* __restrict__ n_kept,
    const uint8_t* __restrict__ xq, int64_t N, int64_t C, int64_t D, int8_t* __restrict__ Ag,
    uint8_t* __restrict__ XtT, void* __restrict__ dX) {
  __shared__ __attribute__((aligned(16))) int8_t tile[kBK][kBC + 4];  // [kept index][column]
  const int tid = threadIdx.x;
  const int64_t cb = (C + kBC - 1) / kBC, db = (D + kBC - 1) / kBC;
  {  // grid z: batch b of a batched call, every operand one block per batch
    const int64_t bt = blockIdx.z, kpad = (N + 127) / 128 * 128;
    qup += bt * N * (C / 2);
    qdn += bt * N * (C / 2);
    w_up += bt * N;
    w_dn += bt * N;
    kept += bt * N;
    n_kept += bt;
    xq += bt * N * (D / 2);
    if (Ag) Ag += bt * kpad * C;
    if (XtT) XtT += bt * D * (kpad / 2);
    if (dX) dX = static_cast<char*>(dX) + bt * N * D * Elem<DT>::bytes;
  }
  if ((int64_t)blockIdx.y == cb + db) {  // zero the dX rows of dropped tokens
    if (!dX) return;
    const int64_t bytes = D * Elem<DT>::bytes;
    const int64_t t0 = (int64_t)blockIdx.x * kBK, t1 = t0 + kBK < N ? t0 + kBK : N;
    for (int64_t t = t0 + (tid >> 6); t < t1; t += 4) {
      if (w_up[t] + w_dn[t]) continue;
      char* row = static_cast<char*>(dX) + t * bytes;
      for (int64_t o = (tid & 63) * 16; o < bytes; o += 64 * 16)
        st_stream<HQ_NT_B_ST>(row + o, make_uint4(0u, 0u, 0u, 0u));
    }
    return;
  }
  const int64_t nk = *n_kept;
  const int64_t kp = (nk + 127) / 128 * 128;
  const int64_t i0 = (int64_t)blockIdx.x * kBK;
  if (i0 >= kp) return;
  const int64_t pitch = (N + 127) / 128 * 128;  // K pitch of XtT (in codes)
  const bool isA = (int64_t)blockIdx.y < cb;
  if (isA ? !Ag : !XtT) return;
  const int64_t col0 = isA ? (int64_t)blockIdx.y * kBC : ((int64_t)blockIdx.y - cb) * kBC;
  const int64_t ncol = isA ? C : D;
  // 128 kept rows x 4 chunks of 32 columns, two per thread: 16-byte loads of the code rows
  if (isA) {  // uniform: A_t is written row-major straight from registers
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const int item = tid + 256 * k, r = item >> 2, q = (item & 3) * 32;
      const int64_t i = i0 + r;
      if (col0 + q >= ncol) continue;  // the last block of a 64-multiple width
      int v[32];
#pragma unroll
      for (int j = 0; j < 32; ++j) v[j] = 0;
      if (i < nk) {  // rows past the kept count are the zero padding up to 128
        const int64_t t = kept[i];
        const int wu = w_up[t], wd = w_dn[t];
        const uint4 up = ld_stream<HQ_NT_B_LD>(qup + t * (C / 2) + (col0 + q) / 2);
        const uint4 dn = ld_stream<HQ_NT_B_LD>(qdn + t * (C / 2) + (col0 + q) / 2);
        weighted8(up.x, dn.x, wu, wd, v);
        weighted8(up.y, dn.y, wu, wd, v + 8);
        weighted8(up.z, dn.z, wu, wd, v + 16);
        weighted8(up.w, dn.w, wu, wd, v + 24);
      }
      const uint2 a0 = interleave8(v), a1 = interleave8(v + 8), a2 = interleave8(v + 16),
                  a3 = interleave8(v + 24);
      st_stream<HQ_NT_B_ST>(Ag + i * C + col0 + q, make_uint4(a0.x, a0.y, a1.x, a1.y));
      st_stream<HQ_NT_B_ST>(Ag + i * C + col0 + q + 16, make_uint4(a2.x, a2.y, a3.x, a3.y));
    }
    return;
  }
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const int item = tid + 256 * k, r = item >> 2, q = (item & 3) * 32;
    const int64_t i = i0 + r;
    uint4 x = make_uint4(0u, 0u, 0u, 0u);
    if (i < nk && col0 + q < ncol) x = ld_stream<HQ_NT_B_LD>(xq + kept[i] * (D / 2) + (col0 + q) / 2);
    // word w of row r sits at word w ^ ((r / 16) % 8) of the row: the transpose below reads
    // one column of 8 row blocks at once, which would otherwise fall on 4 banks
    uint32_t* tp = reinterpret_cast<uint32_t*>(&tile[r][0]);  // 4-byte aligned: pitch 132
    const int sw = (r >> 4) & 7;
    const uint32_t xw[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
    for (int w = 0; w < 8; ++w) {  // bytes 4 w .. 4 w + 3 of the chunk: one code each
      const uint32_t c4 = xw[w >> 1] >> (16 * (w & 1));
      uint32_t b = 0;
#pragma unroll
      for (int j = 0; j < 4; ++j) b |= ((uint32_t)sext4((c4 >> (4 * j)) & 15u) & 0xFFu) << (8 * j);
      tp[(q / 4 + w) ^ sw] = b;
    }
  }
  __syncthreads();
  // 128 columns x 8 chunks of 16 kept indices, four per thread
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int item = tid + 256 * k, c = item >> 3, q = (item & 7) * 16;
    if (col0 + c >= ncol) continue;
    const int cs = (((c >> 2) ^ ((q >> 4) & 7)) << 2) | (c & 3);  // column c's byte in rows q..q+15
    uint32_t w0 = 0, w1 = 0;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const uint32_t byte = ((uint32_t)tile[q + 2 * j][cs] & 15u) |
                            (((uint32_t)tile[q + 2 * j + 1][cs] & 15u) << 4);
      if (j < 4) w0 |= byte << (8 * j);
      else w1 |= byte << (8 * (j - 4));
    }
    st_stream2<HQ_NT_B_ST>(XtT + (col0 + c) * (pitch / 2) + (i0 + q) / 2, make_uint2(w0, w1));
  }
}

// Orders of the kept rows for the FP6 MFMA route (gemm6.hip), one workgroup per 1024 tokens.
// Categories of a token t: upper (w_up = 1), kept lower-only (w_up = 0, w_dn > 0), and the
// lower weight class e = log2 w_dn (0..4).
//   order6: the kept tokens, upper tokens first, each part ascending (the dX row order:
//           tiles holding upper tokens run a second K pass over the upper codes);
//   ent:    the dW K entries (2 t + 1: the upper row of t, 2 t: its lower row) grouped by
//           weight, classes 2^4 .. 2^0, each class padded with -1 to a multiple of 128 (one
//           GEMM stage).  The upper weight 14 = 8 + 4 + 2 puts each upper row into classes
//           3, 2 and 1 (after that class's lower rows);
//   cls:    the first entries of classes 3, 2, 1, 0 and the padded total.
// Every workgroup counts the categories over all tokens and over those before its own, from
// the weight bytes (16 tokens a thread, by popcounts; 32 KB for N = 16384, read from L2), and
// so knows its places without waiting for another; its own tokens, one per thread, are ranked
// by ballots.  One workgroup for all tokens: 36.4 us at N = 16384, 5.6 us so.
constexpr int kCat = 7;  // upper, lower-only, lower classes 0..4
__global__ __launch_bounds__(1024) void fp6_plan_kernel(
    const uint8_t* __restrict__ w_up, const uint8_t* __restrict__ w_dn, int N,
    int32_t* __restrict__ order6, int32_t* __restrict__ n_up_out, int32_t* __restrict__ ent,
    int32_t* __restrict__ cls) {
  __shared__ uint32_t s_sum[16][8];  // per wave: categories in pairs of halves, all tokens then before
  __shared__ int s_tot[8], s_bef[8];
  __shared__ int s_wave[16][kCat];   // kept tokens of each wave, then those of the waves before
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int T0 = (int)blockIdx.x * 1024, t = T0 + tid;
  const int up = t < N ? w_up[t] : 0, dn = t < N ? w_dn[t] : 0;
  uint32_t sum[8] = {0u, 0u, 0u, 0u, 0u, 0u, 0u, 0u};
  for (int q = 16 * tid; q < N; q += 16 * 1024) {  // at most 64 tokens a thread: halves of a wave sum fit
    uint32_t u[4] = {0u, 0u, 0u, 0u}, d[4] = {0u, 0u, 0u, 0u};
    if (q + 16 <= N) {
      const uint4 a = *reinterpret_cast<const uint4*>(w_up + q), b = *reinterpret_cast<const uint4*>(w_dn + q);
      u[0] = a.x; u[1] = a.y; u[2] = a.z; u[3] = a.w;
      d[0] = b.x; d[1] = b.y; d[2] = b.z; d[3] = b.w;
    } else {
#pragma unroll
      for (int j = 0; j < 16; ++j)
        if (q + j < N) {
          u[j >> 2] |= (uint32_t)w_up[q + j] << (8 * (j & 3));
          d[j >> 2] |= (uint32_t)w_dn[q + j] << (8 * (j & 3));
        }
    }
    constexpr uint32_t kOnes = 0x01010101u;
    uint32_t c[4] = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const uint32_t any = (d[w] | (d[w] >> 1) | (d[w] >> 2) | (d[w] >> 3) | (d[w] >> 4)) & kOnes;
      c[0] += __builtin_popcount(u[w] & kOnes) | (__builtin_popcount(any & ~u[w]) << 16);
      c[1] += __builtin_popcount(d[w] & kOnes) | (__builtin_popcount((d[w] >> 1) & kOnes) << 16);
      c[2] += __builtin_popcount((d[w] >> 2) & kOnes) | (__builtin_popcount((d[w] >> 3) & kOnes) << 16);
      c[3] += __builtin_popcount((d[w] >> 4) & kOnes);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      sum[i] += c[i];
      if (q < T0) sum[4 + i] += c[i];
    }
  }
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    sum[i] = wave_sum_u32_dpp(sum[i]);
    if (lane == 0) s_sum[wv][i] = sum[i];
  }
  // this thread's token: its category's rank among the wave's
  const int e = dn ? 31 - __clz(dn) : -1;
  int rank_ord = 0, rank_cls = 0;
#pragma unroll
  for (int k = 0; k < kCat; ++k) {
    const bool in = k == 0 ? up != 0 : k == 1 ? (!up && dn) : e == k - 2;
    const uint64_t b = __ballot(in);
    const int r = __builtin_amdgcn_mbcnt_hi((uint32_t)(b >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)b, 0u));
    if (in) (k < 2 ? rank_ord : rank_cls) = r;
    if (lane == 0) s_wave[wv][k] = (int)__builtin_popcountll(b);
  }
  __syncthreads();
  if (tid < 8 && tid < kCat) {  // category tid: word tid / 2, half tid % 2
    int all = 0, before = 0, run = 0;
#pragma unroll
    for (int w = 0; w < 16; ++w) {
      all += (int)((s_sum[w][tid >> 1] >> (16 * (tid & 1))) & 0xFFFFu);
      before += (int)((s_sum[w][4 + (tid >> 1)] >> (16 * (tid & 1))) & 0xFFFFu);
      const int n = s_wave[w][tid];
      s_wave[w][tid] = run;
      run += n;
    }
    s_tot[tid] = all;
    s_bef[tid] = before;
  }
  __syncthreads();
  const int n_up = s_tot[0], n_d0 = s_tot[2], n_d1 = s_tot[3], n_d2 = s_tot[4], n_d3 = s_tot[5],
            n_d4 = s_tot[6];
  auto r128 = [](int x) { return (x + 127) & ~127; };
  const int b3 = r128(n_d4), b2 = b3 + r128(n_d3 + n_up), b1 = b2 + r128(n_d2 + n_up),
            b0 = b1 + r128(n_d1 + n_up), ke = b0 + r128(n_d0);
  const int base[5] = {b0, b1, b2, b3, 0};  // first entry of lower class e
  if (up) {
    const int p = s_bef[0] + s_wave[wv][0] + rank_ord;
    order6[p] = t;
    ent[b3 + n_d3 + p] = 2 * t + 1;
    ent[b2 + n_d2 + p] = 2 * t + 1;
    ent[b1 + n_d1 + p] = 2 * t + 1;
  } else if (dn) {
    order6[n_up + s_bef[1] + s_wave[wv][1] + rank_ord] = t;
  }
  if (dn) ent[base[e] + s_bef[2 + e] + s_wave[wv][2 + e] + rank_cls] = 2 * t;
  if (blockIdx.x) return;
  // padding of every class to its 128-entry boundary
  const int pad_lo[5] = {n_d4, b3 + n_d3 + n_up, b2 + n_d2 + n_up, b1 + n_d1 + n_up, b0 + n_d0};
  const int pad_hi[5] = {b3, b2, b1, b0, ke};
#pragma unroll
  for (int q = 0; q < 5; ++q)
    for (int i = pad_lo[q] + tid; i < pad_hi[q]; i += 1024) ent[i] = -1;
  if (tid == 0) {
    *n_up_out = n_up;
    cls[0] = b3; cls[1] = b2; cls[2] = b1; cls[3] = b0; cls[4] = ke;
  }
}

}  // namespace

hipError_t launch_lss_plan(hipStream_t s, const int32_t* sumsq_up, const uint32_t* scores,
                           int64_t score_pitch, const uint4* parts, int nparts, int64_t N,
                           int64_t budget, uint64_t seed, uint64_t offset, uint8_t* w_up,
                           uint8_t* w_dn, int32_t* kept, int32_t* n_kept, int64_t batch,
                           uint64_t offset_stride) {
  timing_begin(s);
  if (N <= 16 * kPlanThreadsSmall)
    lss_plan_kernel<kPlanThreadsSmall><<<(unsigned)batch, kPlanThreadsSmall, 0, s>>>(
        sumsq_up, scores, score_pitch, parts, nparts, (int)N, budget, seed, offset, w_up, w_dn,
        kept, n_kept, offset_stride);
  else
    lss_plan_kernel<kPlanThreads><<<(unsigned)batch, kPlanThreads, 0, s>>>(
        sumsq_up, scores, score_pitch, parts, nparts, (int)N, budget, seed, offset, w_up, w_dn,
        kept, n_kept, offset_stride);
  timing_end(s, kKPlan);
  return hipGetLastError();
}

hipError_t launch_build_operands(hipStream_t s, int dt, const uint8_t* qup, const uint8_t* qdn,
                                 const uint8_t* w_up, const uint8_t* w_dn, const int32_t* kept,
                                 const int32_t* n_kept, const uint8_t* xq, int64_t N, int64_t C,
                                 int64_t D, int8_t* Ag, uint8_t* XtT, void* dX, int64_t batch) {
  const int64_t pitch = (N + 127) / 128 * 128;
  dim3 grid((unsigned)(pitch / kBK), (unsigned)((C + kBC - 1) / kBC + (D + kBC - 1) / kBC + 1),
            (unsigned)batch);
  timing_begin(s);
  switch (dt) {
    case kF32:
      build_operands_kernel<kF32><<<grid, 256, 0, s>>>(qup, qdn, w_up, w_dn, kept, n_kept, xq, N, C, D, Ag, XtT, dX);
      break;
    case kF16:
      build_operands_kernel<kF16><<<grid, 256, 0, s>>>(qup, qdn, w_up, w_dn, kept, n_kept, xq, N, C, D, Ag, XtT, dX);
      break;
    case kBF16:
      build_operands_kernel<kBF16><<<grid, 256, 0, s>>>(qup, qdn, w_up, w_dn, kept, n_kept, xq, N, C, D, Ag, XtT, dX);
      break;
    default:
      return hipErrorInvalidValue;
  }
  timing_end(s, kKBuild);
  return hipGetLastError();
}

hipError_t launch_fp6_plan(hipStream_t s, const uint8_t* w_up, const uint8_t* w_dn, int64_t N,
                           int32_t* order6, int32_t* n_up, int32_t* ent, int32_t* cls) {
  timing_begin(s);
  fp6_plan_kernel<<<(unsigned)((N + 1023) / 1024), 1024, 0, s>>>(w_up, w_dn, (int)N, order6, n_up, ent, cls);
  timing_end(s, kKFp6Plan);
  return hipGetLastError();
}

}  // namespace hqlss
