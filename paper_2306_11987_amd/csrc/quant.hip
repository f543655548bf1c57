// Quantisers of HQ-MM and LSS-MM (gfx950).
//
//  * fwht_absmax / fwht_quant: the Hadamard quantiser HQ (Sec. 3.3): block-diagonal
//    unnormalised Hadamard transform of each row (radix-2 butterflies, strides ascending,
//    fp32), then per-tensor absmax and INT4 codes clamp(rint(v * fl(7/a)), -7, 7)
//    (Sec. 3.1, Eq. 2), packed two per byte (App. A.6) with per-row sums of squares
//    (the ||X_i|| factor of the leverage score, Sec. 4.2).  One launch serves X and W:
//    X by rows, W by tiles, each tile workgroup writing its codes row-major and also
//    transposed through LDS (the K-contiguous operand of the dX GEMM), so W is read once.
//    On request the codes of X and W are also written as FP6 (e2m3, the padded layout of
//    fp6.hip) for a product on the FP6 MFMA, through the hardware conversion.
//  * fwht_lsq: the same transform quantised at a caller-given (learned) step in one pass,
//    with the fp16 deltas q - I r that the learned-step backward needs (Eq. 2, App. A.3);
//    the second tensor by tiles as above.
//  * bit_split: bit splitting of the output gradient (Sec. 4.2, Eq. 4): upper codes by
//    round-to-nearest at s_up = a/7, lower codes by stochastic rounding of 14 x the exact
//    residual (s_dn = s_up / 14), Philox stream 0.  It also forms the integer leverage
//    scores of both stacked rows of every token and per-workgroup totals of them, which
//    is all the sampler needs.  At a row's end the group reduces the two row sums (one
//    packed reduction for rows of at most 640 columns) and two of its lanes form the two
//    scores, each with one integer square root.
//
// Work decomposition: a row belongs to a group of G lanes (choose_group: the largest power
// of two <= 64 dividing cols/16, or wider, up to the whole workgroup, where that saves time),
// so a wave holds 64/G rows or a part of one, and every per-row result (sum of squares,
// scores) is one plain store: no atomics, nothing to pre-zero.  Each lane loads 16
// consecutive elements per step (fwht_absmax of the 16-bit types 32, for blocks of 32 columns
// and more) and has two steps' loads in flight, bit_split and fwht_lsq one's.  A Hadamard block
// of b = 2^k <= 128 columns lives in b/16 consecutive lanes of one group (b/16 <= G for
// every admitted shape), so strides 1..8 run in registers and strides 16..64 are lane
// exchanges folded into the butterfly add (DPP) or a swizzle.  Per-tensor maxima leave
// each workgroup as one plain store of a partial; consumers reduce the partials.
// A batched job (the attention BMM) holds many equal tensors; its workgroups are split
// evenly over the batches and every per-tensor output is one block per batch.
//
// These kernels are bound by vector-ALU issue as much as by HBM, so the per-element work
// is kept to a handful of instructions: codes come from the magic-number form of
// round-half-even (x + 1.5 * 2^23 leaves rint(x) in the low mantissa bits, exact for
// |x| < 2^22), packing uses byte permutes, and the sums of squares of the codes are dot
// products of the packed INT4 words with themselves.
#include "common.h"
#include "launch.h"

#include <mutex>
#include <type_traits>
#include <unordered_map>

namespace hqlss {

namespace {

constexpr int kQThreads = 512;
constexpr int kQWaves = kQThreads / kWave;
constexpr int kVE = 16;  // elements per lane per step
constexpr float kRne = 12582912.0f;  // 1.5 * 2^23

template <int DT, bool NT>
__device__ __forceinline__ void load16(const char* p, float v[16]) {
  load8<DT, NT>(p, v);
  load8<DT, NT>(p + 8 * Elem<DT>::bytes, v + 8);
}

// The same in two parts, so that a load can be issued well before its values are widened (a
// widening in the load's own basic block would wait for it there).
template <int DT>
struct Raw16 {
  uint4 q[Elem<DT>::bytes];
  template <bool NT>
  __device__ __forceinline__ void load(const char* p) {
#pragma unroll
    for (int i = 0; i < Elem<DT>::bytes; ++i) q[i] = ld_stream<NT>(p + 16 * i);
  }
  __device__ __forceinline__ void widen(float v[16]) const {
#pragma unroll
    for (int i = 0; i < Elem<DT>::bytes; ++i) widen_piece<DT>(q[i], v + i * (16 / Elem<DT>::bytes));
  }
};

// Value of lane (lane ^ M), M in {1, 2, 4}, added to x: DPP quad permutations (folded into
// the add) or a ds_swizzle swap of 4-lane groups.
template <int M>
__device__ __forceinline__ float add_xor_lane(float v, float x) {
  const int i = __float_as_int(v);
  if constexpr (M == 1) return __int_as_float(__builtin_amdgcn_update_dpp(0, i, 0xB1, 0xF, 0xF, true)) + x;
  else if constexpr (M == 2) return __int_as_float(__builtin_amdgcn_update_dpp(0, i, 0x4E, 0xF, 0xF, true)) + x;
  else return __int_as_float(__builtin_amdgcn_ds_swizzle(i, (4 << 10) | 0x1F)) + x;
}

// In-place unnormalised FWHT of blocks of 2^LOG2B consecutive elements; the lane holds 16
// consecutive elements, the lanes of one block are consecutive.  Pairs (a, c) at stride h
// become (a + c, a - c), strides ascending.  Across lanes the lower lane adds its
// partner's value and the upper lane adds its own negated value to the partner's (a - c
// = a + (-c) exactly), so both take one DPP add.
template <int LOG2B>
__device__ __forceinline__ void fwht16(float v[16], int lane) {
  constexpr int b = 1 << LOG2B;
#pragma unroll
  for (int h = 1; h < 16 && h < b; h <<= 1) {
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      if ((j & h) == 0) {
        const float a = v[j], c = v[j + h];
        v[j] = a + c;
        v[j + h] = a - c;
      }
    }
  }
#define HQLSS_XSTAGE(M)                                                       \
  if constexpr (16 * (M) < b) {                                               \
    const uint32_t sgn = (lane & (M)) ? 0x80000000u : 0u;                     \
    _Pragma("unroll") for (int j = 0; j < 16; ++j) {                          \
      const float own = __uint_as_float(__float_as_uint(v[j]) ^ sgn);         \
      v[j] = add_xor_lane<M>(v[j], own);                                      \
    }                                                                         \
  }
  HQLSS_XSTAGE(1)
  HQLSS_XSTAGE(2)
  HQLSS_XSTAGE(4)
#undef HQLSS_XSTAGE
}

// The same with 32 consecutive elements in a lane.
template <int LOG2B>
__device__ __forceinline__ void fwht32(float v[32], int lane) {
  constexpr int b = 1 << LOG2B;
#pragma unroll
  for (int h = 1; h < 32 && h < b; h <<= 1) {
#pragma unroll
    for (int j = 0; j < 32; ++j) {
      if ((j & h) == 0) {
        const float a = v[j], c = v[j + h];
        v[j] = a + c;
        v[j + h] = a - c;
      }
    }
  }
#define HQLSS_XSTAGE32(M)                                                     \
  if constexpr (32 * (M) < b) {                                               \
    const uint32_t sgn = (lane & (M)) ? 0x80000000u : 0u;                     \
    _Pragma("unroll") for (int j = 0; j < 32; ++j) {                          \
      const float own = __uint_as_float(__float_as_uint(v[j]) ^ sgn);         \
      v[j] = add_xor_lane<M>(v[j], own);                                      \
    }                                                                         \
  }
  HQLSS_XSTAGE32(1)
  HQLSS_XSTAGE32(2)
#undef HQLSS_XSTAGE32
}

// Bits of fl(x + 1.5 * 2^23): rint(x) (half-to-even) sits in the low mantissa bits.
__device__ __forceinline__ uint32_t rne_bits(float x) { return __float_as_uint(x + kRne); }

// 16 consecutive codes (as rne_bits) -> their 12 bytes of FP6 (e2m3) fields, field i at bits
// 6i..6i+5: half of a 32-code group of the padded FP6 layout.  The hardware conversion of
// two 16-float operands interleaves them (field 2k from the first, 2k + 1 from the second),
// so even and odd codes go in separately; the upper 16 fields come out zero.  Exact: the
// codes are integers |q| <= 7, all e2m3 values, and the scale is 1.  The instruction is
// issued through inline assembly with an early-clobber result: the compiler builtin let
// the result registers overlap the source registers, and the instruction then read some
// sources after writing over them (wrong fields at one fixed position of the chunk).
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef int i32x6 __attribute__((ext_vector_type(6)));
__device__ __forceinline__ uint3 fp6_half16(const uint32_t y[16]) {
  f32x16 ev, od;
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    ev[k] = __uint_as_float(y[2 * k]) - kRne;
    od[k] = __uint_as_float(y[2 * k + 1]) - kRne;
    ev[8 + k] = 0.f;
    od[8 + k] = 0.f;
  }
  i32x6 w;
  asm volatile("v_cvt_scalef32_2xpk16_fp6_f32 %0, %1, %2, 1.0" : "=&v"(w) : "v"(ev), "v"(od));
  return make_uint3((uint32_t)w[0], (uint32_t)w[1], (uint32_t)w[2]);
}

// The 16 bytes lane pair (2g, 2g + 1) stores of 32-code group g of a row in the padded FP6
// layout: the even chunk's fields fill bytes 0..11, the odd one's bytes 12..23, then 8 zero
// bytes.  The even lane takes bytes 0..15 (the first word of its partner's fields comes
// over), the odd lane bytes 16..31, so both store one aligned 16-byte piece.  Lanes 2g and
// 2g + 1 must hold chunks 2g and 2g + 1 and both be active.
__device__ __forceinline__ uint4 fp6_chunk16(const uint32_t y[16], bool odd) {
  const uint3 f = fp6_half16(y);
  const uint32_t partner = (uint32_t)__shfl_xor((int)f.x, 1);
  return odd ? make_uint4(f.y, f.z, 0u, 0u) : make_uint4(f.x, f.y, f.z, partner);
}
__device__ __forceinline__ void store_fp6_chunk(uint8_t* row6, int64_t c, const uint4& v) {
  *reinterpret_cast<uint4*>(row6 + (c >> 1) * 32 + (c & 1) * 16) = v;
}

// Pack 8 codes given as rne_bits (low nibbles) into one word, element j at bits 4j.
__device__ __forceinline__ uint32_t pack8_bits(const uint32_t y[8]) {
  uint32_t b[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) b[i] = (y[2 * i + 1] << 4) | (y[2 * i] & 15u);  // valid low byte
  const uint32_t lo = __builtin_amdgcn_perm(b[1], b[0], 0x0C0C0400u);  // [b0, b1, 0, 0]
  const uint32_t hi = __builtin_amdgcn_perm(b[3], b[2], 0x0C0C0400u);  // [b2, b3, 0, 0]
  return __builtin_amdgcn_perm(hi, lo, 0x05040100u);                  // [b0, b1, b2, b3]
}

// Sum of squares of the eight signed nibbles of a packed word, accumulated into acc.
__device__ __forceinline__ int sumsq8(uint32_t w, int acc) {
  return __builtin_amdgcn_sdot8((int)w, (int)w, acc, false);
}

// Sum over the 2^log2g threads of a row group, for every thread of it.  Groups inside a wave
// add by DPP (swap neighbours, swap pairs, mirror halves, mirror the row of 16), one lane
// exchange for 32 and the four row sums as scalars for 64; wider groups add their waves'
// sums through LDS, `red` holding two buffers of kQWaves words used in turn (a buffer is
// written again only after the barrier of the call in between).  Every thread of the
// workgroup calls it where log2g > 6, every lane of the wave otherwise.
__device__ __forceinline__ int group_sum(int v, int log2g, int* red, int& par) {
  v += __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xF, 0xF, true);  // log2g >= 2 always
  v += __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xF, 0xF, true);
  if (log2g == 2) return v;
  v += __builtin_amdgcn_update_dpp(0, v, 0x141, 0xF, 0xF, true);
  if (log2g == 3) return v;
  v += __builtin_amdgcn_update_dpp(0, v, 0x140, 0xF, 0xF, true);
  if (log2g == 4) return v;
  if (log2g == 5) return v + __shfl_xor(v, 16);
  v = __builtin_amdgcn_readlane(v, 0) + __builtin_amdgcn_readlane(v, 16) +
      __builtin_amdgcn_readlane(v, 32) + __builtin_amdgcn_readlane(v, 48);
  if (log2g == 6) return v;
  const int w = threadIdx.x >> 6, n = 1 << (log2g - 6);
  if ((threadIdx.x & 63) == 0) red[par * kQWaves + w] = v;
  __syncthreads();
  v = 0;
  for (int i = 0; i < n; ++i) v += red[par * kQWaves + (w & ~(n - 1)) + i];
  par ^= 1;
  return v;
}

// Lanes without a chunk of their own load chunk (lane & mask) of a row instead.  They must
// form whole Hadamard blocks, or their transform could exceed the tensor's maximum: blocks
// of 128 columns (8 lanes) need rows of whole 8 chunks, shorter blocks fit 4.
__device__ __forceinline__ int spare_mask(int row_chunks) { return row_chunks % 8 == 0 ? 7 : 3; }

// Row-group geometry of one job (one tensor).  The wave walks a uniform sequence of steps
// (row k of its groups, 16-column chunk it), kept several steps ahead in loads whatever
// the row boundaries; group rows past the end re-read the last row and store nothing, and
// so do the lanes past a row's last chunk where G does not divide the row (they load one of
// its first chunks).  Groups wider than a wave (log2g > 6) take the same number of steps in
// every wave of the workgroup.
struct Geo {
  int lane, sub, G, iters, chunks, spare;
  bool ragged;
  int64_t first_row, row_step, rows, steps;
  __device__ Geo(const QJob& j, int wg) {
    lane = threadIdx.x & 63;
    G = 1 << j.log2g;
    sub = threadIdx.x & (G - 1);
    chunks = (int)(j.cols / kVE);
    iters = (chunks + G - 1) >> j.log2g;
    ragged = iters * G != chunks;
    spare = spare_mask(chunks);
    const int rw = kQThreads >> j.log2g;  // rows of a workgroup at a time
    const int64_t wg_row0 = (int64_t)wg * rw;
    first_row = wg_row0 + (threadIdx.x >> j.log2g);
    row_step = (int64_t)j.wg * rw;
    rows = j.rows;
    const int64_t row0 = j.log2g <= 6 ? wg_row0 + ((threadIdx.x & ~63u) >> j.log2g) : wg_row0;
    steps = row0 < rows ? (rows - row0 + row_step - 1) / row_step * iters : 0;
  }
  // row of step (k, it) for this lane's group, clamped into the tensor
  __device__ int64_t row_of(int64_t k) const {
    const int64_t r = first_row + k * row_step;
    return r < rows ? r : rows - 1;
  }
  __device__ bool valid(int64_t k) const { return first_row + k * row_step < rows; }
  // 16-column chunk of step (k, it), whether the row has it, and the first of its columns, or
  // where it has not, that of the chunk this lane loads instead (the ragged test is uniform)
  __device__ int chunk(int it) const { return it * G + sub; }
  __device__ bool live(int it) const { return !ragged || chunk(it) < chunks; }
  __device__ int load_col(int it) const {
    int c = it * (G * kVE) + sub * kVE;
    if (ragged && chunk(it) >= chunks) c = (sub & spare) * kVE;
    return c;
  }
};

// The row groups of Geo with 32 elements a lane: half the steps a row where Geo takes an even
// number of whole ones, else half the lanes.  The second half of the workgroup's threads then
// takes the rows of the next round, so that a row stays on the workgroup (and XCD) that Geo
// gives it.  (Half the lanes throughout left half of the threads idle wherever there is no next
// round: 8192 x 4096 beside a small weight, fp16, b = 32: 19.1 us, 16.4 with 16 elements a lane.)
struct Geo32 {
  int lane, sub, G, iters, chunks, spare;
  int64_t first_row, row_step, rows, steps;
  __device__ Geo32(const QJob& j, int wg) {
    const int64_t c16 = j.cols / kVE;
    const bool whole = c16 % (int64_t(2) << j.log2g) == 0;
    const int l = whole ? j.log2g : j.log2g - 1;  // lanes per row; log2g >= 2, and >= 3 where a block has 128 columns
    lane = threadIdx.x & 63;
    G = 1 << l;
    sub = threadIdx.x & (G - 1);
    chunks = (int)(j.cols / 32);
    iters = (chunks + G - 1) >> l;
    spare = chunks % 4 == 0 ? 3 : 1;  // whole blocks, as spare_mask()
    const int rw = kQThreads >> j.log2g;  // Geo's rows of a workgroup at a time
    const int64_t round = (int64_t)j.wg * rw;
    auto row = [&](int t) { return (int64_t)wg * rw + (t >> l) % rw + (t >> l) / rw * round; };
    first_row = row(threadIdx.x);
    row_step = whole ? round : 2 * round;
    rows = j.rows;
    const int64_t row0 = row(threadIdx.x & ~63u);  // the wave's first
    steps = row0 < rows ? (rows - row0 + row_step - 1) / row_step * iters : 0;
  }
  __device__ int64_t row_of(int64_t k) const {
    const int64_t r = first_row + k * row_step;
    return r < rows ? r : rows - 1;
  }
  __device__ int load_col(int it) const {
    const int c = it * G + sub;
    return (c < chunks ? c : (sub & spare)) * 32;
  }
};

// Geometry of the block-size search, which has no per-row results: the tensor is one run of
// 16-element chunks, 64 to a wave and step, whatever its rows: a row is a multiple of 64
// elements and of the Hadamard block, so blocks never straddle a row and stay aligned.
// Lanes past the end load one of the first chunks, a whole block of lanes at a time.
struct Flat {
  int lane, spare;
  int64_t wave, waves, chunks, steps;
  __device__ Flat(const QJob& j, int wg) {
    lane = threadIdx.x & 63;
    wave = (int64_t)wg * kQWaves + (threadIdx.x >> 6);
    waves = (int64_t)j.wg * kQWaves;
    chunks = j.rows * (j.cols / kVE);
    spare = spare_mask((int)(j.cols / kVE));
    const int64_t all = (chunks + 63) / 64;
    steps = wave < all ? (all - wave + waves - 1) / waves : 0;
  }
  __device__ int64_t chunk(int64_t s) const { return (wave + s * waves) * 64 + lane; }
  __device__ bool valid(int64_t s) const { return chunk(s) < chunks; }
  __device__ int64_t load_chunk(int64_t s) const { return valid(s) ? chunk(s) : (lane & spare); }
};

// max over the first n partial maxima (every thread of the workgroup gets it).
__device__ __forceinline__ float reduce_parts(const float* __restrict__ part, int n) {
  __shared__ float red[kQWaves];
  float m = 0.f;
  for (int i = threadIdx.x; i < n; i += 2 * kQThreads) {  // both loads in flight at once
    const float p0 = part[i], p1 = part[i + kQThreads < n ? i + kQThreads : i];
    m = fmaxf(m, fmaxf(p0, p1));
  }
  m = wave_max(m);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
  __syncthreads();
  m = red[0];
#pragma unroll
  for (int i = 1; i < kQWaves; ++i) m = fmaxf(m, red[i]);
  return m;
}

// Position of this workgroup in a launch over two (possibly batched) jobs: which job, the
// batch b inside it, and the workgroup index within that batch.
struct QPos {
  bool second;
  int b, wg;
};
__device__ __forceinline__ QPos qpos(const QJob& j0, const QJob& j1) {
  const int n0 = j0.wg * j0.batch;
  const bool second = (int)blockIdx.x >= n0;
  const int idx = second ? (int)blockIdx.x - n0 : (int)blockIdx.x;
  const int per = second ? j1.wg : j0.wg;
  return {second, idx / per, idx % per};
}

// Plain 16-byte copy: the reference kernel against which hardware traffic counters are
// calibrated (its bytes read and written are known exactly).
__global__ __launch_bounds__(256) void copy_kernel(const uint4* __restrict__ src,
                                                   uint4* __restrict__ dst, int64_t n) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride)
    dst[i] = src[i];
}

// Workgroups [0, j0.wg) serve job 0 and [j0.wg, j0.wg + j1.wg) job 1; each writes the
// maximum |FWHT| of its rows to part[its index within the job].
template <int DT, int LOG2B>
__global__ __launch_bounds__(kQThreads) void fwht_absmax_kernel(QJob j0, QJob j1,
                                                                float* __restrict__ part0,
                                                                float* __restrict__ part1) {
  // steps in flight: 2 measured faster than 4 (fewer registers, more waves per SIMD;
  // -5 % per FFN step's maximum passes, -9 % on the 4096..11008-wide sweep) and than 8
  constexpr int U = 2;
  // blocks of 32 columns and more: the two steps are one of 32 elements in a row, one lane
  // exchange less an element (at b = 128 the one that goes through LDS); vector instructions
  // bound this pass there (event times, 16384 x 4096 and 4096 x 4096 fp16, b = 128: 40.9 -> 37.2
  // us; 16384 x 768 and 3072 x 768, b = 32: 10.1 -> 9.0).  Not for fp32, whose lanes would
  // load 128 bytes each (1003 x 832: 4.6 -> 5.2)
  constexpr bool WIDE = LOG2B >= 5 && DT != kF32;
  __shared__ float red[kQWaves];
  const QPos q = qpos(j0, j1);
  const QJob& j = q.second ? j1 : j0;
  const int wg = q.wg;
  using G_ = std::conditional_t<WIDE, Geo32, Geo>;
  const G_ g(j, wg);
  constexpr int EB = Elem<DT>::bytes;
  float m = 0.f;
  const char* base = static_cast<const char*>(j.src) + (int64_t)q.b * j.bstride * EB;
  int64_t k = 0;
  int it = 0;
  if constexpr (WIDE) {
    for (int64_t s0 = 0; s0 < g.steps; ++s0) {
      float v[32];
      const char* p = base + (g.row_of(k) * j.cols + g.load_col(it)) * EB;
      load16<DT, HQ_NT_ABS_LD>(p, v);
      load16<DT, HQ_NT_ABS_LD>(p + 16 * EB, v + 16);
      if (++it == g.iters) { it = 0; ++k; }
      fwht32<LOG2B>(v, g.lane);  // rows and chunks loaded twice leave the maximum unchanged
#pragma unroll
      for (int e = 0; e < 32; e += 2) m = fmaxf(m, fmaxf(fabsf(v[e]), fabsf(v[e + 1])));
    }
  } else
  for (int64_t s0 = 0; s0 < g.steps; s0 += U) {
    float v[U][kVE];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (s0 + u < g.steps) {
        load16<DT, HQ_NT_ABS_LD>(base + (g.row_of(k) * j.cols + g.load_col(it)) * EB, v[u]);
        if (++it == g.iters) { it = 0; ++k; }
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (s0 + u < g.steps) {  // rows and chunks loaded twice leave the maximum unchanged
        fwht16<LOG2B>(v[u], g.lane);
#pragma unroll
        for (int e = 0; e < kVE; e += 2) m = fmaxf(m, fmaxf(fabsf(v[u][e]), fabsf(v[u][e + 1])));
      }
    }
  }
  m = wave_max(m);
  if (g.lane == 0) red[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
#pragma unroll
    for (int i = 1; i < kQWaves; ++i) m = fmaxf(m, red[i]);
    m = fmaxf(m, red[0]);
    (q.second ? part1 : part0)[q.b * j.wg + wg] = m;
  }
}

// One tile of the second job (W), quantised by one workgroup: TW columns (whole Hadamard
// blocks) x R rows, 16 elements per lane as in the row kernels, so the transform and the
// rounding are the same operations on the same values.  The workgroup writes the tile's
// codes both ways: row-major from registers (as the row kernels do, with the fp16 deltas
// of the learned-step mode) and transposed through LDS (thread (d, q) packs rows
// 16 q .. 16 q + 15 of column d).  The tiles thus read W once and replace the row
// workgroups of that job.  Rows past the end are loaded from the last row and not stored.
template <int LOG2B> struct TileT {
  static constexpr int TW = (1 << LOG2B) > 64 ? 128 : 64;
  static constexpr int LPR = TW / kVE;         // lanes per row
  static constexpr int R = kQThreads / LPR;    // rows per tile
  __host__ __device__ static int64_t tiles(int64_t rows, int64_t cols) { return (rows + R - 1) / R * (cols / TW); }
};

// LSQ selects the learned-step quantiser: code clamp(rint(v inv), -7, 7) (the clamp first)
// and delta as in fwht_lsq_kernel; else the code rint(v inv) of fwht_quant_kernel.
// inv_of() gives the scale; it is called after the tile's loads were issued.
template <int DT, int LOG2B, bool LSQ, class F>
__device__ void quant_tile(const void* src, int64_t rows, int64_t cols, F&& inv_of, int t,
                           uint8_t* __restrict__ packed, uint16_t* __restrict__ delta,
                           uint8_t* __restrict__ packed_t, uint8_t* __restrict__ fp6 = nullptr) {
  using T = TileT<LOG2B>;
  constexpr int TW = T::TW, LPR = T::LPR, R = T::R, PITCH = TW + 4;
  __shared__ uint8_t tile[R * PITCH];
  constexpr int EB = Elem<DT>::bytes;
  const int64_t ntc = cols / TW;
  const int64_t r0 = (int64_t)(t / ntc) * R, c0 = (int64_t)(t % ntc) * TW;
  const int tid = threadIdx.x, rr = tid / LPR, sub = tid % LPR;
  {
    const bool ok = r0 + rr < rows;
    const int64_t r = ok ? r0 + rr : rows - 1;
    float v[kVE];
    load16<DT, HQ_NT_Q_LD>(static_cast<const char*>(src) + (r * cols + c0 + sub * kVE) * EB, v);
    const float inv = inv_of();
    fwht16<LOG2B>(v, tid & 63);
    uint32_t y[kVE], dh[kVE / 2];
#pragma unroll
    for (int e = 0; e < kVE; e += 2) {
      uint32_t h[2];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const float x = v[e + u] * inv;
        if constexpr (LSQ) {
          const float rc = __builtin_amdgcn_fmed3f(x, -7.0f, 7.0f);
          const float m = rc + kRne;
          y[e + u] = __float_as_uint(m);
          const float q = m - kRne;
          const float d = (rc == x) ? q - x : q;
          h[u] = (uint32_t)__builtin_bit_cast(uint16_t, (_Float16)d);
        } else {
          y[e + u] = rne_bits(x);
          h[u] = 0u;
        }
      }
      dh[e / 2] = h[0] | (h[1] << 16);
    }
    const int64_t c = (c0 + sub * kVE) / kVE;  // 16-column chunk of the row
    const uint4 f6 = fp6 ? fp6_chunk16(y, (c & 1) != 0) : make_uint4(0u, 0u, 0u, 0u);  // all lanes
    if (ok) {
      st_stream2<HQ_NT_Q_ST>(reinterpret_cast<uint2*>(packed + r * (cols / 2)) + c,
                             make_uint2(pack8_bits(y), pack8_bits(y + 8)));
      if (fp6) store_fp6_chunk(fp6 + r * cols, c, f6);
      if constexpr (LSQ) {
        uint4* dp = reinterpret_cast<uint4*>(delta + r * cols) + 2 * c;
        st_stream<HQ_NT_Q_ST>(dp, make_uint4(dh[0], dh[1], dh[2], dh[3]));
        st_stream<HQ_NT_Q_ST>(dp + 1, make_uint4(dh[4], dh[5], dh[6], dh[7]));
      }
    }
    uint32_t* row = reinterpret_cast<uint32_t*>(tile + rr * PITCH + sub * kVE);
#pragma unroll
    for (int w = 0; w < 4; ++w)
      row[w] = (y[4 * w] & 15u) | ((y[4 * w + 1] & 15u) << 8) | ((y[4 * w + 2] & 15u) << 16) |
               ((y[4 * w + 3] & 15u) << 24);
  }
  __syncthreads();
  const int d = tid / (R / 16), q = tid % (R / 16);
  if (r0 + 16 * q < rows) {
    uint32_t w2[2] = {0u, 0u};
#pragma unroll
    for (int i = 0; i < 16; ++i) w2[i >> 3] |= (uint32_t)tile[(16 * q + i) * PITCH + d] << (4 * (i & 7));
    *reinterpret_cast<uint2*>(packed_t + (c0 + d) * (rows / 2) + r0 / 2 + 8 * q) = make_uint2(w2[0], w2[1]);
  }
}

// Codes of FWHT(rows) at the reduced maximum a; the first workgroup of each job also
// stores a.  When o1.packed_t is set, job 1 has no row workgroups (j1.wg = 0): workgroups
// past job 0's quantise it by tiles (quant_tile), writing its codes and their transpose.
// Row sums of squares are plain stores by the group's first lane.  The clamp to +-7 of the
// definition never engages here: |v| <= a gives |v * fl(7/a)| <= 7 (1 + 2^-24), which
// rounds to at most 7.
template <int DT, int LOG2B>
__global__ __launch_bounds__(kQThreads) void fwht_quant_kernel(QJob j0, QJob j1, QOut o0, QOut o1) {
  constexpr int U = 2;  // steps in flight (2 measured faster than 4, as for the maximum)
  if ((int)blockIdx.x >= j0.wg + j1.wg) {  // uniform per workgroup
    const int t = (int)blockIdx.x - j0.wg - j1.wg;
    auto inv_of = [&]() {
      const float a = reduce_parts(o1.part, o1.nparts);
      if (t == 0 && threadIdx.x == 0) *o1.amax_out = a;
      return a > 0.f ? 7.0f / a : 0.f;
    };
    quant_tile<DT, LOG2B, false>(j1.src, j1.rows, j1.cols, inv_of, t, o1.packed, nullptr,
                                 o1.packed_t, o1.fp6);
    return;
  }
  const bool second = (int)blockIdx.x >= j0.wg;
  const QJob& j = second ? j1 : j0;
  const QOut& o = second ? o1 : o0;
  const int wg = second ? (int)blockIdx.x - j0.wg : (int)blockIdx.x;
  const Geo g(j, wg);
  constexpr int EB = Elem<DT>::bytes;
  const char* base = static_cast<const char*>(j.src);
  __shared__ int rsum[2 * kQWaves];
  int par = 0;
  int64_t k = 0, kp = 0;  // load and process positions
  int it = 0, ip = 0;
  int ss = 0;
  // Each pass loads its own two steps.  With the next pass's loads beside them the 16-bit types
  // held 91 registers and two workgroups a CU, without 77 and three (16384 x 4096 and 4096 x
  // 4096 fp16: 49 and 44 to 46 us; 200 x 4096 and 11008 x 4096: 40.5 and 34.7).  The first loads
  // go out before the maximum is formed for fp32 alone (16384 x 4096 and 4096 x 4096: 84 us, 88
  // after it); fp16 takes 48.7 us so instead of 43.7.
  constexpr bool EARLY = DT == kF32;
  Raw16<DT> raw[U];
  auto load = [&](int64_t s0) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (s0 + u < g.steps) {
        raw[u].template load<HQ_NT_Q_LD>(base + (g.row_of(k) * j.cols + g.load_col(it)) * EB);
        if (++it == g.iters) { it = 0; ++k; }
      }
    }
  };
  if constexpr (EARLY) load(0);
  const float a = reduce_parts(o.part, o.nparts);
  if (wg == 0 && threadIdx.x == 0) *o.amax_out = a;
  const float inv = a > 0.f ? 7.0f / a : 0.f;
  for (int64_t s0 = 0; s0 < g.steps; s0 += U) {
    if (!EARLY || s0) load(s0);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (s0 + u < g.steps) {
        float v[kVE];
        raw[u].widen(v);
        fwht16<LOG2B>(v, g.lane);
        uint32_t y[kVE];
#pragma unroll
        for (int e = 0; e < kVE; ++e) y[e] = rne_bits(v[e] * inv);
        const uint32_t w0 = pack8_bits(y), w1 = pack8_bits(y + 8);
        const int c = g.chunk(ip);
        const bool live = g.live(ip);
        ss = live ? sumsq8(w1, sumsq8(w0, ss)) : ss;
        const bool in_row = g.valid(kp), ok = live && in_row;
        const int64_t r = g.row_of(kp);
        if (ok) st_stream2<HQ_NT_Q_ST>(reinterpret_cast<uint2*>(o.packed + r * (j.cols / 2)) + c, make_uint2(w0, w1));
        if (o.fp6) {  // the pair exchange runs in every lane, the store only in valid rows
          const uint4 f6 = fp6_chunk16(y, (c & 1) != 0);
          if (ok) store_fp6_chunk(o.fp6 + r * j.cols, c, f6);
        }
        if (++ip == g.iters) {  // end of the group's row
          if (o.row_sumsq) {
            ss = group_sum(ss, j.log2g, rsum, par);
            if (in_row && g.sub == 0) o.row_sumsq[r] = ss;
          }
          ss = 0;
          ip = 0;
          ++kp;
        }
      }
    }
  }
}

// Learned-step-size codes (Eq. 2 at a caller-given step, after the transform of Sec. 3.3):
// r = fl(v * fl(1/s)), q = clamp(rint(r), -7, 7) and delta = q - [-7 <= r <= 7] r, the
// term that the step-size gradient weights (App. A.3).  One pass: no maximum is needed.
// The clamp comes first (med3), so the magic-number rounding only sees |x| <= 7, and
// rint(clamp(r)) = clamp(rint(r)) as the bounds are integers.  q - r is exact in fp32 (q
// and r lie within a factor of two of each other, or q = 0), then rounded to fp16 (to
// nearest even); |delta| <= 1/2 holds exactly for the entries inside the range and
// |delta| > 1/2 for the clipped ones, so the gradient kernels recover the clip indicator
// from delta alone.
template <int DT, int LOG2B>
__global__ __launch_bounds__(kQThreads) void fwht_lsq_kernel(QJob j0, QJob j1, LsqOut o0, LsqOut o1) {
  // one step in flight: 70-73 registers instead of 96, three workgroups per CU instead of
  // two (the BMM's quantiser 31.3 -> 28.9 us; the FFN's unchanged)
  constexpr int U = 1;
  {  // o1.packed_t set: job 1 by tiles (j1.wg = 0), one tile per workgroup past job 0's
    const int nrow = j0.wg * j0.batch + j1.wg * j1.batch;
    if ((int)blockIdx.x >= nrow) {  // uniform per workgroup
      const int nt = (int)TileT<LOG2B>::tiles(j1.rows, j1.cols);
      const int tt = (int)blockIdx.x - nrow, b = tt / nt;
      const int64_t rc = j1.rows * j1.cols;  // elements of one batch
      quant_tile<DT, LOG2B, true>(static_cast<const char*>(j1.src) + (int64_t)b * j1.bstride * Elem<DT>::bytes,
                                  j1.rows, j1.cols, [&]() { return 1.0f / o1.step[b]; }, tt % nt,
                                  o1.packed + b * (rc / 2), o1.delta + b * rc, o1.packed_t + b * (rc / 2));
      return;
    }
  }
  const QPos qp = qpos(j0, j1);
  const QJob& j = qp.second ? j1 : j0;
  const LsqOut& o = qp.second ? o1 : o0;
  const int wg = qp.wg;
  const float inv = 1.0f / o.step[qp.b];
  const Geo g(j, wg);
  constexpr int EB = Elem<DT>::bytes;
  const char* base = static_cast<const char*>(j.src) + (int64_t)qp.b * j.bstride * EB;
  __shared__ int rsum[2 * kQWaves];
  int par = 0;
  // this batch's outputs
  uint8_t* const packed = o.packed + (int64_t)qp.b * j.rows * (j.cols / 2);
  uint16_t* const delta = o.delta + (int64_t)qp.b * j.rows * j.cols;
  int32_t* const row_sumsq = o.row_sumsq ? o.row_sumsq + (int64_t)qp.b * j.rows : nullptr;
  int64_t k = 0, kp = 0;
  int it = 0, ip = 0;
  int ss = 0;
  for (int64_t s0 = 0; s0 < g.steps; s0 += U) {
    float v[U][kVE];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (s0 + u < g.steps) {
        load16<DT, HQ_NT_Q_LD>(base + (g.row_of(k) * j.cols + g.load_col(it)) * EB, v[u]);
        if (++it == g.iters) { it = 0; ++k; }
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (s0 + u < g.steps) {
        fwht16<LOG2B>(v[u], g.lane);
        uint32_t y[kVE], dh[kVE / 2];
#pragma unroll
        for (int e = 0; e < kVE; e += 2) {
          uint32_t h[2];
#pragma unroll
          for (int t = 0; t < 2; ++t) {
            const float r = v[u][e + t] * inv;
            const float rc = __builtin_amdgcn_fmed3f(r, -7.0f, 7.0f);
            const float m = rc + kRne;
            y[e + t] = __float_as_uint(m);
            const float q = m - kRne;
            const float d = (rc == r) ? q - r : q;
            h[t] = (uint32_t)__builtin_bit_cast(uint16_t, (_Float16)d);
          }
          dh[e / 2] = h[0] | (h[1] << 16);
        }
        const uint32_t w0 = pack8_bits(y), w1 = pack8_bits(y + 8);
        const int c = g.chunk(ip);  // 16-column chunk
        const bool live = g.live(ip);
        ss = live ? sumsq8(w1, sumsq8(w0, ss)) : ss;
        const bool in_row = g.valid(kp), ok = live && in_row;
        const int64_t r = g.row_of(kp);
        if (ok) {
          st_stream2<HQ_NT_Q_ST>(reinterpret_cast<uint2*>(packed + r * (j.cols / 2)) + c, make_uint2(w0, w1));
          uint4* dp = reinterpret_cast<uint4*>(delta + r * j.cols) + 2 * c;
          st_stream<HQ_NT_Q_ST>(dp, make_uint4(dh[0], dh[1], dh[2], dh[3]));
          st_stream<HQ_NT_Q_ST>(dp + 1, make_uint4(dh[4], dh[5], dh[6], dh[7]));
        }
        if (++ip == g.iters) {
          if (row_sumsq) {
            ss = group_sum(ss, j.log2g, rsum, par);
            if (in_row && g.sub == 0) row_sumsq[r] = ss;
          }
          ss = 0;
          ip = 0;
          ++kp;
        }
      }
    }
  }
}

// Bit split of dY [N][C] (no transform: the gradient is split as it is, Sec. 4.2) and the
// integer leverage scores of the two stacked rows of every token:
//   c_up = isqrt(14^2 sum q_up^2 * x_sumsq * 2^16),  c_dn = isqrt(sum q_dn^2 * x_sumsq * 2^16)
// (the common factor s_dn s_x dropped).  Each workgroup stores the count of non-zero scores
// and their sum (u64) of its rows as one partial.
template <int DT>
__global__ __launch_bounds__(kQThreads) void bit_split_kernel(QJob j, const float* __restrict__ part,
                                                              int nparts, BsOut o, uint64_t seed,
                                                              uint64_t offset) {
  // one 16-element step per loop pass: the Philox state and the two code planes already
  // hold many registers, and one step (more waves per SIMD) measured 9 % faster than two
  constexpr int U = 1;
  __shared__ uint64_t red_s[kQWaves];
  __shared__ uint32_t red_n[kQWaves];
  // batch b of a batched job: its own maximum, outputs and Philox counter range
  const int b = (int)blockIdx.x / j.wg, wg = (int)blockIdx.x % j.wg;
  // -0.0f, from an argument so that the fma below is not folded into a multiply
  const float nzero = __uint_as_float(0x80000000u | (uint32_t)((uint64_t)j.cols >> 63));
  const Geo g(j, wg);
  const int64_t C = j.cols;
  constexpr int EB = Elem<DT>::bytes;
  uint32_t nnz = 0;
  uint64_t ssum = 0;
  const char* base = static_cast<const char*>(j.src) + (int64_t)b * j.bstride * EB;
  __shared__ int rsum[2 * kQWaves];
  int par = 0;
  offset += (uint64_t)b * o.offset_stride;
  const int64_t rb = (int64_t)b * j.rows;  // first row of this batch in the row-indexed outputs
  uint8_t* const qup = o.qup + rb * (C / 2);
  uint8_t* const qdn = o.qdn + rb * (C / 2);
  uint32_t* const scores = o.scores + (int64_t)b * 2 * o.score_pitch;
  // a row's sums of squared codes are at most 49 C (codes within +-7); below 2^15 both fit
  // one int in 16-bit halves without reaching its sign bit
  const bool packed_sums = 49 * C < 32768;
  int64_t k = 0, kp = 0;
  int it = 0, ip = 0;
  int su = 0, sd = 0;
  // The first loads go out before the maximum is formed; not for fp32, whose 16 registers of
  // raw data then cost a third of the workgroups a CU holds (85 registers, with 71 three).
  constexpr bool EARLY = DT != kF32;
  Raw16<DT> raw[U];
  auto load = [&](int64_t s0) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (s0 + u < g.steps) {
        raw[u].template load<HQ_NT_BS_LD>(base + (g.row_of(k) * C + g.load_col(it)) * EB);
        if (++it == g.iters) { it = 0; ++k; }
      }
    }
  };
  if constexpr (EARLY) load(0);
  const float a = reduce_parts(part + (int64_t)b * nparts, nparts);
  if (wg == 0 && threadIdx.x == 0) o.amax_out[b] = a;
  const float inv = a > 0.f ? 7.0f / a : 0.f;
  for (int64_t s0 = 0; s0 < g.steps; s0 += U) {
    if (!EARLY || s0) load(s0);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (s0 + u < g.steps) {
        const int c = g.chunk(ip);
        const bool live = g.live(ip), in_row = g.valid(kp);
        const int64_t r = g.row_of(kp);
        const int64_t col = (int64_t)c * kVE;
        uint32_t yu[kVE], yd[kVE];
        float v[kVE];
        raw[u].widen(v);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const U4 rnd = philox_block(seed, offset, 0u, (uint64_t)(r * C + col + 8 * h));
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            // fl(v inv): one rounding, so the fma with a -0 addend equals the product
            // (an fp16 operand widens inside the instruction)
            const float x = __builtin_fmaf(v[8 * h + e], inv, nzero);
            const uint32_t bu = rne_bits(x);                  // |x| <= 7 (1 + 2^-23)
            // -14 rint(x) exactly from the bits 1.5 * 2^23 + rint(x); then
            // fl(14 x - 14 rint(x)) = fl(14 (x - rint(x))), the residual being exact
            const float m14 = __builtin_fmaf(__uint_as_float(bu), -14.0f, 14.0f * kRne);
            const float w = __builtin_fmaf(x, 14.0f, m14);   // |w| <= 7
            const float fl = floorf(w);
            const float thr = (w - fl) * 65536.0f;
            const uint32_t bd = __float_as_uint(fl + kRne);   // floor(w) in the low bits
            yu[8 * h + e] = bu;
            yd[8 * h + e] = bd + (((float)u16_of(rnd, e) < thr) ? 1u : 0u);
          }
        }
        const uint32_t u0 = pack8_bits(yu), u1 = pack8_bits(yu + 8);
        const uint32_t d0 = pack8_bits(yd), d1 = pack8_bits(yd + 8);
        su = live ? sumsq8(u1, sumsq8(u0, su)) : su;
        sd = live ? sumsq8(d1, sumsq8(d0, sd)) : sd;
        if (live && in_row) {
          const int64_t o8 = r * (C / 16) + c;  // uint2 index
          st_stream2<HQ_NT_BS_ST>(reinterpret_cast<uint2*>(qup) + o8, make_uint2(u0, u1));
          st_stream2<HQ_NT_BS_ST>(reinterpret_cast<uint2*>(qdn) + o8, make_uint2(d0, d1));
        }
        if (++ip == g.iters) {  // end of the group's row
          if (packed_sums) {  // one reduction of the two halves
            const int p = group_sum(su | (sd << 16), j.log2g, rsum, par);
            su = p & 0xFFFF;
            sd = (int)((uint32_t)p >> 16);
          } else {
            su = group_sum(su, j.log2g, rsum, par);
            sd = group_sum(sd, j.log2g, rsum, par);
          }
          // the group's lane 0 forms the upper row's score and lane 1 the lower row's
          // (G >= 4), so a wave runs one square root per row end, not two in sequence
          if (in_row && g.sub < 2) {
            const uint64_t sx = (uint32_t)o.x_sumsq[rb + r];
            const bool upper = g.sub == 0;
            const uint64_t k2 = upper ? (uint64_t)(kBsRatio * kBsRatio) * (uint32_t)su : (uint64_t)(uint32_t)sd;
            const uint32_t c = isqrt64((k2 * sx) << 16);
            if (upper) {
              o.sumsq_up[rb + r] = su;
              o.sumsq_dn[rb + r] = sd;
            }
            scores[(upper ? 0 : o.score_pitch) + r] = c;
            nnz += c > 0;
            ssum += c;
          }
          su = sd = 0;
          ip = 0;
          ++kp;
        }
      }
    }
  }
  nnz = (uint32_t)wave_sum((int)nnz);
  ssum = wave_sum_u64(ssum);
  if (g.lane == 0) {
    red_n[threadIdx.x >> 6] = nnz;
    red_s[threadIdx.x >> 6] = ssum;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t n = 0;
    uint64_t t = 0;
#pragma unroll
    for (int i = 0; i < kQWaves; ++i) {
      n += red_n[i];
      t += red_s[i];
    }
    o.parts[(int64_t)b * j.wg + wg] = make_uint4(n, (uint32_t)t, (uint32_t)(t >> 32), 0u);
  }
}

// ---------------------------------------------------------------- block-size search
// Choice of the Hadamard block 2^k (App. A.5): k minimising MSE(X_bar, X) MSE(W_bar, W),
// V_bar = s int_s(V H) H^T.  The transform with strides ascending is nested: after the
// stages of strides 1 .. 2^(k-1) every 2^k block holds its own FWHT, so one pass over the
// data yields the transforms of all k = 0..7 in turn.  The error is taken in the transform
// domain, ||V_bar - V||^2 = ||s q - V H_u||^2 / 2^k (H_u / 2^(k/2) is orthogonal), so it
// needs no inverse transform.  For D not a multiple of 128 the deepest stages mix blocks
// that are no candidates; their values are computed and never used.
constexpr int kLevels = 8;  // k = 0 .. 7

// One butterfly stage at stride H (in-lane for H < 16, else across lanes H / 16 apart).
template <int H>
__device__ __forceinline__ void fwht_stage(float v[16], int lane) {
  if constexpr (H < 16) {
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      if ((j & H) == 0) {
        const float a = v[j], c = v[j + H];
        v[j] = a + c;
        v[j + H] = a - c;
      }
    }
  } else {
    constexpr int M = H / 16;
    const uint32_t sgn = (lane & M) ? 0x80000000u : 0u;
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      const float own = __uint_as_float(__float_as_uint(v[j]) ^ sgn);
      v[j] = add_xor_lane<M>(v[j], own);
    }
  }
}

// Calls f(level, v) for level 0 (the input) and after each of the 7 stages.
template <class F>
__device__ __forceinline__ void fwht_nested(float v[16], int lane, F&& f) {
  f(0, v);
  fwht_stage<1>(v, lane);  f(1, v);
  fwht_stage<2>(v, lane);  f(2, v);
  fwht_stage<4>(v, lane);  f(3, v);
  fwht_stage<8>(v, lane);  f(4, v);
  fwht_stage<16>(v, lane); f(5, v);
  fwht_stage<32>(v, lane); f(6, v);
  fwht_stage<64>(v, lane); f(7, v);
}

// Pass 1: per-workgroup maxima of |FWHT_k(rows)| for every k, part[wg * 8 + k].
template <int DT>
__global__ __launch_bounds__(kQThreads) void hsize_max_kernel(QJob j0, QJob j1,
                                                              float* __restrict__ part0,
                                                              float* __restrict__ part1) {
  constexpr int U = 2;
  __shared__ float red[kQWaves][kLevels];
  const bool second = (int)blockIdx.x >= j0.wg;
  const QJob& j = second ? j1 : j0;
  const int wg = second ? (int)blockIdx.x - j0.wg : (int)blockIdx.x;
  const Flat g(j, wg);
  constexpr int EB = Elem<DT>::bytes;
  float m[kLevels];
#pragma unroll
  for (int l = 0; l < kLevels; ++l) m[l] = 0.f;
  const char* base = static_cast<const char*>(j.src);
  for (int64_t s0 = 0; s0 < g.steps; s0 += U) {
    float v[U][kVE];
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (s0 + u < g.steps) load16<DT, HQ_NT_ABS_LD>(base + g.load_chunk(s0 + u) * (kVE * EB), v[u]);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (s0 + u < g.steps) {  // chunks loaded twice leave the maxima unchanged
        fwht_nested(v[u], g.lane, [&](int l, const float* x) {
#pragma unroll
          for (int e = 0; e < kVE; e += 2) m[l] = fmaxf(m[l], fmaxf(fabsf(x[e]), fabsf(x[e + 1])));
        });
      }
    }
  }
#pragma unroll
  for (int l = 0; l < kLevels; ++l) {
    const float w = wave_max(m[l]);
    if (g.lane == 0) red[threadIdx.x >> 6][l] = w;
  }
  __syncthreads();
  if (threadIdx.x < kLevels) {
    float r = red[0][threadIdx.x];
#pragma unroll
    for (int i = 1; i < kQWaves; ++i) r = fmaxf(r, red[i][threadIdx.x]);
    (second ? part1 : part0)[wg * kLevels + threadIdx.x] = r;
  }
}

// Pass 2: per-workgroup sums over valid rows of (s_k q - v)^2 for every k, with
// s_k = fl(a_k / 7) and q = rint(v fl(7 / a_k)) the forward quantiser's codes (no clamp
// needed, as there).  Each 16-element chunk is summed in fp32 (one fused multiply-add
// per element on the correctly rounded difference), chunks in fp64; err[wg * 8 + k].
// Bound by vector-ALU issue (some 45 instructions an element).  8192 x 1024 and 4096 x 1024
// fp16: 26.2 -> 24.5 us with the maxima's partials read four at a time by all threads,
// the first data loads issued before them (12 dependent loads a lane before).
template <int DT>
__global__ __launch_bounds__(kQThreads) void hsize_err_kernel(QJob j0, QJob j1,
                                                              const float* __restrict__ mx0, int n0,
                                                              const float* __restrict__ mx1, int n1,
                                                              double* __restrict__ err0,
                                                              double* __restrict__ err1) {
  constexpr int U = 2;
  __shared__ float amax[kQWaves][kLevels];
  __shared__ double red[kQWaves][kLevels];
  const bool second = (int)blockIdx.x >= j0.wg;
  const QJob& j = second ? j1 : j0;
  const int wg = second ? (int)blockIdx.x - j0.wg : (int)blockIdx.x;
  const Flat g(j, wg);
  constexpr int EB = Elem<DT>::bytes;
  double acc[kLevels];
#pragma unroll
  for (int l = 0; l < kLevels; ++l) acc[l] = 0.0;
  const char* base = static_cast<const char*>(j.src);
  Raw16<DT> raw[U];
  auto load = [&](int64_t s0) {
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (s0 + u < g.steps) raw[u].template load<HQ_NT_ABS_LD>(base + g.load_chunk(s0 + u) * (kVE * EB));
  };
  load(0);  // in flight while the maxima are formed
  float inv[kLevels], st[kLevels];
  {  // a_k = max over the pass-1 partials of this tensor: thread t takes level t % 8 of
     // partials t / 8, t / 8 + 64, ..., four of them in flight
    const float* mx = second ? mx1 : mx0;
    const int n = second ? n1 : n0, l = threadIdx.x & 7;
    constexpr int kSlots = kQThreads / kLevels;
    float r = 0.f;
    for (int i = threadIdx.x >> 3; i < n; i += 4 * kSlots) {
      float p[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) p[q] = mx[(i + q * kSlots < n ? i + q * kSlots : i) * kLevels + l];
      r = fmaxf(r, fmaxf(fmaxf(p[0], p[1]), fmaxf(p[2], p[3])));
    }
#pragma unroll
    for (int o = 8; o < 64; o <<= 1) r = fmaxf(r, __shfl_xor(r, o));
    if (g.lane < kLevels) amax[threadIdx.x >> 6][l] = r;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kLevels; ++k) {
      float a = amax[0][k];
#pragma unroll
      for (int w = 1; w < kQWaves; ++w) a = fmaxf(a, amax[w][k]);
      inv[k] = a > 0.f ? 7.0f / a : 0.f;
      st[k] = a / 7.0f;
    }
  }
  for (int64_t s0 = 0; s0 < g.steps; s0 += U) {
    if (s0) load(s0);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (s0 + u < g.steps) {
        const bool ok = g.valid(s0 + u);
        float v[kVE];
        raw[u].widen(v);
        fwht_nested(v, g.lane, [&](int l, const float* x) {
          float e2 = 0.f;
#pragma unroll
          for (int e = 0; e < kVE; ++e) {
            const float q = __builtin_rintf(x[e] * inv[l]);
            const float d = __builtin_fmaf(st[l], q, -x[e]);
            e2 = __builtin_fmaf(d, d, e2);
          }
          acc[l] += ok ? (double)e2 : 0.0;
        });
      }
    }
  }
#pragma unroll
  for (int l = 0; l < kLevels; ++l) {
    double w = acc[l];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) w += __shfl_xor(w, o);
    if (g.lane == 0) red[threadIdx.x >> 6][l] = w;
  }
  __syncthreads();
  if (threadIdx.x < kLevels) {
    double r = red[0][threadIdx.x];
#pragma unroll
    for (int i = 1; i < kQWaves; ++i) r += red[i][threadIdx.x];
    (second ? err1 : err0)[wg * kLevels + threadIdx.x] = r;
  }
}

// Pass 3 (one workgroup of 1024): MSE_k = sum / (2^k numel) per tensor, the candidates
// k <= kmax with cols % 2^k == 0, and the argmin of MSE_X MSE_W (ties to the smaller k).
// mse_out[k] = MSE_X(k), mse_out[8 + k] = MSE_W(k), NaN for k not a candidate.  Latency is
// all it costs: 128 threads share a level's partials, so that few loads and additions stand
// in a row (10.4 us with 32 threads a level and one thread adding up their sums, 4.6 us so).
constexpr int kPickThreads = 1024;
__global__ __launch_bounds__(kPickThreads) void hsize_pick_kernel(const double* __restrict__ err0, int n0,
                                                         const double* __restrict__ err1, int n1,
                                                         double numel0, double numel1, int64_t cols,
                                                         int kmax, int32_t* __restrict__ k_out,
                                                         double* __restrict__ mse_out) {
  __shared__ double red[2][kPickThreads / 64][kLevels];
  __shared__ double tot[2][kLevels];
  const int l = threadIdx.x & 7, slot = threadIdx.x >> 3;  // 128 slots per level
  constexpr int kSlots = kPickThreads / kLevels;
  double a = 0.0, b = 0.0;
  for (int i = slot; i < (n0 > n1 ? n0 : n1); i += kSlots) {
    if (i < n0) a += err0[i * kLevels + l];
    if (i < n1) b += err1[i * kLevels + l];
  }
#pragma unroll
  for (int o = 8; o < 64; o <<= 1) {  // lanes of one level are 8 apart
    a += __shfl_xor(a, o);
    b += __shfl_xor(b, o);
  }
  if ((threadIdx.x & 63) < kLevels) {
    red[0][threadIdx.x >> 6][l] = a;
    red[1][threadIdx.x >> 6][l] = b;
  }
  __syncthreads();
  if (threadIdx.x < 2 * kLevels) {
    double t = 0.0;
#pragma unroll
    for (int i = 0; i < kPickThreads / 64; ++i) t += red[threadIdx.x >> 3][i][l];
    tot[threadIdx.x >> 3][l] = t;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    int best = 0;
    double best_obj = 0.0;
    bool any = false;
    for (int k = 0; k < kLevels; ++k) {
      const double sx = tot[0][k], sw = tot[1][k];
      const double scale = (double)(1 << k);
      const double mx = numel0 > 0 ? sx / (scale * numel0) : 0.0;
      const double mw = numel1 > 0 ? sw / (scale * numel1) : 0.0;
      const bool cand = k <= kmax && cols % (int64_t(1) << k) == 0;
      const double nan = __longlong_as_double(0x7FF8000000000000LL);
      mse_out[k] = cand ? mx : nan;
      mse_out[kLevels + k] = cand ? mw : nan;
      if (cand) {
        const double obj = mx * mw;
        if (!any || obj < best_obj) {
          best = k;
          best_obj = obj;
          any = true;
        }
      }
    }
    *k_out = best;
  }
}

template <template <int, int> class F, int DT, typename... Args>
hipError_t dispatch_block(int log2b, Args... args) {
  switch (log2b) {
    case 0: return F<DT, 0>::run(args...);
    case 1: return F<DT, 1>::run(args...);
    case 2: return F<DT, 2>::run(args...);
    case 3: return F<DT, 3>::run(args...);
    case 4: return F<DT, 4>::run(args...);
    case 5: return F<DT, 5>::run(args...);
    case 6: return F<DT, 6>::run(args...);
    case 7: return F<DT, 7>::run(args...);
  }
  return hipErrorInvalidValue;
}

// Workgroups of kernel f that fit on the device at once (cached per kernel).
int resident_wgs(const void* f) {
  static std::mutex mu;
  static std::unordered_map<const void*, int> cache;
  std::lock_guard<std::mutex> lock(mu);
  auto it = cache.find(f);
  if (it != cache.end()) return it->second;
  int dev = 0, cus = 0, per = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
      hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, f, kQThreads, 0) != hipSuccess)
    return 256;
  int n = (per > 0 ? per : 1) * (cus > 0 ? cus : 1);
  if (n > kQMaxWg) n = kQMaxWg;
  cache.emplace(f, n);
  return n;
}

// Lanes per row (as a logarithm).  The default, the largest power of two up to 64 that divides
// the row's chunks, leaves no lane idle; wider groups, up to the workgroup, take fewer steps a
// row and idle in its last one.  Estimated time: the steps a wave takes of a row, and 0.4 of
// one for its end (0.9 where a group spans waves and ends in a barrier), times the waves each
// of the 1024 SIMDs runs one after the other or side by side, below three of which latency and
// not throughput counts.  A wider group is taken where it saves a fifth by this estimate, and
// inside a wave the widest of about equal ones, for its longer runs of memory.  Measured over
// 8 to 512 lanes a row at 140 shapes:
//   few rows, odd factors: 1003 x 832 and 1344 x 832 fp32 with 4 lanes and with 64: maximum 12.7
//   and 6.0 us, quantiser 17.1 and 8.3; bit split of 300 x 2752 with 4 lanes 57 us, with 256 8.5;
//   rows that fill the device: bit split of 81920 x 192 with 4 lanes 19.2 us, with 16 (a quarter
//   of them idle) 25.4; of 8192 x 768 with 16 lanes 12.0, with 64 13.8; quantiser of 8192 x 768
//   and 2112 x 768 10.9 and 12.7.
// The choice does not depend on the kernel, and an unbatched grid of more than one round gives
// each tensor a multiple of 8 workgroups (where it does not run out of rows), so every kernel
// that walks a tensor reads a row on the same XCD and finds what fits its L2 there (the
// quantiser of 16384 x 768 fp16 after a maximum pass that walked the tensor in another order:
// 13.9 us, in this one 12.4 us).
void choose_group(QJob& j) {
  if (j.rows <= 0) return;
  const int64_t chunks = j.cols / kVE, rows = j.rows * j.batch;
  auto cost = [&](int l) {
    const int64_t steps = ((chunks - 1) >> l) + 1, threads = rows << l;
    constexpr int64_t three = 3 * 1024 * 64;  // threads of three waves on each SIMD
    return (double)(10 * steps + (l > 6 ? 9 : 4)) * (double)(threads > three ? threads : three);
  };
  int best = j.log2g;
  double c = 0.8 * cost(best);
  for (int l = j.log2g + 1; (1 << l) <= kQThreads && (chunks >> (l - 1)) > 0; ++l) {
    const double x = cost(l);
    if (x < c || (best != j.log2g && l <= 6 && x <= 1.05 * c)) best = l;
    if (x < c) c = x;
  }
  j.log2g = best;
}

// Workgroups that leave each thread one step (flat kernels) or each group one row.
int64_t wgs_needed(const QJob& j, bool flat) {
  if (j.rows <= 0) return 0;
  if (flat) return (j.rows * (j.cols / kVE) + kQThreads - 1) / kQThreads;
  const int64_t per = kQThreads >> j.log2g;
  return (j.rows + per - 1) / per;
}

// Share one resident grid between two jobs: all they need if it fits, else in proportion
// to their sizes.
// flat: a kernel that takes the tensors as runs of chunks; else the row groups are chosen here.
void fit_grid(QJob& a, QJob& b, int cap, bool flat = false) {
  if (!flat) {
    choose_group(a);
    choose_group(b);
  }
  const int64_t na = wgs_needed(a, flat), nb = wgs_needed(b, flat);  // per batch
  if (na * a.batch + nb * b.batch <= cap) {
    a.wg = (int)na;
    b.wg = (int)nb;
    return;
  }
  if (a.batch > 1 || b.batch > 1) {
    // batched: about two resident rounds shared by size, then per batch (many small
    // batches would otherwise get one workgroup each and leave the CUs half occupied);
    // at most kBatchWgSlack + batch workgroups per job in all (the partials bound)
    const double sa = (double)a.rows * a.cols * a.batch, sb = (double)b.rows * b.cols * b.batch;
    const int64_t c2 = 2 * (int64_t)cap;
    const int64_t ca = nb ? (int64_t)(c2 * sa / (sa + sb)) : c2, cb = c2 - ca;
    auto per = [](int64_t c, int64_t n, int64_t batch) {
      int64_t w = (c + batch - 1) / batch;
      if (w > n) w = n;
      return (int)(w < 1 ? 1 : w);
    };
    a.wg = na ? per(ca, na, a.batch) : 0;
    b.wg = nb ? per(cb, nb, b.batch) : 0;
    return;
  }
  // Whole rounds of the 8 XCDs: job 1's share is rounded up where that leaves job 0 at least
  // 7/8 of its own share, else down; each job with rows gets 8 where it needs them.  (Rounded up
  // always, a short batch beside a wide weight was left one workgroup of the grid: 64 x 4096 and
  // 11008 x 4096 fp16, maximum 36.2 us, so 25.7, block search 139.8 and 89.3.)
  const double ba = (double)a.rows * a.cols, bb = (double)b.rows * b.cols;
  int64_t wb = 0;
  if (nb) {
    wb = (int64_t)(cap * bb / (ba + bb) + 0.5);
    const int64_t up = (wb + 7) / 8 * 8;
    wb = 8 * (cap - up) >= 7 * (cap - wb) ? up : wb / 8 * 8;
    if (na && wb > cap - 8) wb = cap - 8;
    if (wb < 8) wb = 8;
    if (wb > nb) wb = nb;
  }
  int64_t wa = (cap - wb) / 8 * 8;
  if (wa > na) wa = na;
  a.wg = (int)wa;
  b.wg = (int)wb;
}

template <int DT, int LOG2B> struct AbsmaxF {
  static hipError_t run(hipStream_t s, QJob& j0, QJob& j1, float* p0, float* p1) {
    const void* f = reinterpret_cast<const void*>(&fwht_absmax_kernel<DT, LOG2B>);
    fit_grid(j0, j1, resident_wgs(f));
    timing_begin(s);
    fwht_absmax_kernel<DT, LOG2B><<<j0.wg * j0.batch + j1.wg * j1.batch, kQThreads, 0, s>>>(j0, j1, p0, p1);
    timing_end(s, kKAbsmax);
    return hipGetLastError();
  }
};
template <int DT, int LOG2B> struct QuantF {
  static hipError_t run(hipStream_t s, QJob j0, QJob j1, QOut o0, QOut o1) {
    const void* f = reinterpret_cast<const void*>(&fwht_quant_kernel<DT, LOG2B>);
    int64_t nt = 0;
    if (o1.packed_t) {  // job 1 by tiles only
      QJob none = make_job(nullptr, 0, j1.cols);
      fit_grid(j0, none, resident_wgs(f));
      j1.wg = 0;
      nt = TileT<LOG2B>::tiles(j1.rows, j1.cols);
    } else {
      fit_grid(j0, j1, resident_wgs(f));
    }
    timing_begin(s);
    fwht_quant_kernel<DT, LOG2B><<<(unsigned)(j0.wg + j1.wg + nt), kQThreads, 0, s>>>(j0, j1, o0, o1);
    timing_end(s, kKQuant);
    return hipGetLastError();
  }
};

template <int DT, int LOG2B> struct LsqF {
  static hipError_t run(hipStream_t s, QJob j0, QJob j1, LsqOut o0, LsqOut o1) {
    const void* f = reinterpret_cast<const void*>(&fwht_lsq_kernel<DT, LOG2B>);
    int64_t nt = 0;
    if (o1.packed_t) {  // job 1 by tiles only
      QJob none = make_job(nullptr, 0, j1.cols);
      fit_grid(j0, none, resident_wgs(f));
      j1.wg = 0;
      nt = TileT<LOG2B>::tiles(j1.rows, j1.cols) * j1.batch;
    } else {
      fit_grid(j0, j1, resident_wgs(f));
    }
    timing_begin(s);
    fwht_lsq_kernel<DT, LOG2B><<<(unsigned)(j0.wg * j0.batch + j1.wg * j1.batch + nt), kQThreads, 0, s>>>(
        j0, j1, o0, o1);
    timing_end(s, kKLsqQuant);
    return hipGetLastError();
  }
};

int log2_group(int64_t cols) {
  const int64_t v = cols / kVE;
  int l = 0;
  while (l < 6 && v % (int64_t(2) << l) == 0) ++l;
  return l;
}

}  // namespace

QJob make_job(const void* src, int64_t rows, int64_t cols) {
  QJob j{src, rows > 0 ? rows : 0, cols, log2_group(cols), 0, 1, (rows > 0 ? rows : 0) * cols};
  return j;
}

QJob make_job_batched(const void* src, int64_t batch, int64_t rows, int64_t cols) {
  QJob j = make_job(src, rows, cols);
  j.batch = (int)batch;
  return j;
}

hipError_t launch_copy(hipStream_t s, const void* src, void* dst, int64_t bytes) {
  const int64_t n = bytes / 16;
  int64_t wg = (n + 255) / 256;
  if (wg > 4096) wg = 4096;
  if (wg < 1) wg = 1;
  timing_begin(s);
  copy_kernel<<<(int)wg, 256, 0, s>>>(static_cast<const uint4*>(src), static_cast<uint4*>(dst), n);
  timing_end(s, kKCopy);
  return hipGetLastError();
}

hipError_t launch_fwht_absmax(hipStream_t s, int dt, int log2b, QJob& j0, float* part0,
                              QJob& j1, float* part1) {
  switch (dt) {
    case kF32: return dispatch_block<AbsmaxF, kF32, hipStream_t, QJob&, QJob&, float*, float*>(log2b, s, j0, j1, part0, part1);
    case kF16: return dispatch_block<AbsmaxF, kF16, hipStream_t, QJob&, QJob&, float*, float*>(log2b, s, j0, j1, part0, part1);
    case kBF16: return dispatch_block<AbsmaxF, kBF16, hipStream_t, QJob&, QJob&, float*, float*>(log2b, s, j0, j1, part0, part1);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_fwht_quant(hipStream_t s, int dt, int log2b, const QJob& j0, const QOut& o0,
                             const QJob& j1, const QOut& o1) {
  switch (dt) {
    case kF32: return dispatch_block<QuantF, kF32>(log2b, s, j0, j1, o0, o1);
    case kF16: return dispatch_block<QuantF, kF16>(log2b, s, j0, j1, o0, o1);
    case kBF16: return dispatch_block<QuantF, kBF16>(log2b, s, j0, j1, o0, o1);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_fwht_lsq(hipStream_t s, int dt, int log2b, const QJob& j0, const LsqOut& o0,
                           const QJob& j1, const LsqOut& o1) {
  switch (dt) {
    case kF32: return dispatch_block<LsqF, kF32>(log2b, s, j0, j1, o0, o1);
    case kF16: return dispatch_block<LsqF, kF16>(log2b, s, j0, j1, o0, o1);
    case kBF16: return dispatch_block<LsqF, kBF16>(log2b, s, j0, j1, o0, o1);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_bit_split(hipStream_t s, int dt, QJob& j, const float* part, int nparts,
                            const BsOut& o, uint64_t seed, uint64_t offset) {
  const void* f = dt == kF32 ? reinterpret_cast<const void*>(&bit_split_kernel<kF32>)
                  : dt == kF16 ? reinterpret_cast<const void*>(&bit_split_kernel<kF16>)
                               : reinterpret_cast<const void*>(&bit_split_kernel<kBF16>);
  QJob none = make_job(nullptr, 0, j.cols);
  fit_grid(j, none, resident_wgs(f));
  timing_begin(s);
  switch (dt) {
    case kF32:
      bit_split_kernel<kF32><<<j.wg * j.batch, kQThreads, 0, s>>>(j, part, nparts, o, seed, offset);
      break;
    case kF16:
      bit_split_kernel<kF16><<<j.wg * j.batch, kQThreads, 0, s>>>(j, part, nparts, o, seed, offset);
      break;
    case kBF16:
      bit_split_kernel<kBF16><<<j.wg * j.batch, kQThreads, 0, s>>>(j, part, nparts, o, seed, offset);
      break;
    default:
      return hipErrorInvalidValue;
  }
  timing_end(s, kKBitSplit);
  return hipGetLastError();
}


void row_grid(QJob& j0, QJob& j1, int cap, bool flat) { fit_grid(j0, j1, cap, flat); }

hipError_t launch_hsize_search(hipStream_t s, int dt, QJob& j0, QJob& j1, float* mx0, float* mx1,
                               double* err0, double* err1, int kmax, int32_t* k_out,
                               double* mse_out) {
  const void* fm = dt == kF32 ? reinterpret_cast<const void*>(&hsize_max_kernel<kF32>)
                   : dt == kF16 ? reinterpret_cast<const void*>(&hsize_max_kernel<kF16>)
                                : reinterpret_cast<const void*>(&hsize_max_kernel<kBF16>);
  const void* fe = dt == kF32 ? reinterpret_cast<const void*>(&hsize_err_kernel<kF32>)
                   : dt == kF16 ? reinterpret_cast<const void*>(&hsize_err_kernel<kF16>)
                                : reinterpret_cast<const void*>(&hsize_err_kernel<kBF16>);
  if (dt != kF32 && dt != kF16 && dt != kBF16) return hipErrorInvalidValue;
  QJob a0 = j0, a1 = j1;
  fit_grid(a0, a1, resident_wgs(fm), true);
  timing_begin(s);
  if (dt == kF32) hsize_max_kernel<kF32><<<a0.wg + a1.wg, kQThreads, 0, s>>>(a0, a1, mx0, mx1);
  else if (dt == kF16) hsize_max_kernel<kF16><<<a0.wg + a1.wg, kQThreads, 0, s>>>(a0, a1, mx0, mx1);
  else hsize_max_kernel<kBF16><<<a0.wg + a1.wg, kQThreads, 0, s>>>(a0, a1, mx0, mx1);
  timing_end(s, kKHsizeMax);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  QJob b0 = j0, b1 = j1;
  fit_grid(b0, b1, resident_wgs(fe), true);
  timing_begin(s);
  if (dt == kF32)
    hsize_err_kernel<kF32><<<b0.wg + b1.wg, kQThreads, 0, s>>>(b0, b1, mx0, a0.wg, mx1, a1.wg, err0, err1);
  else if (dt == kF16)
    hsize_err_kernel<kF16><<<b0.wg + b1.wg, kQThreads, 0, s>>>(b0, b1, mx0, a0.wg, mx1, a1.wg, err0, err1);
  else
    hsize_err_kernel<kBF16><<<b0.wg + b1.wg, kQThreads, 0, s>>>(b0, b1, mx0, a0.wg, mx1, a1.wg, err0, err1);
  timing_end(s, kKHsizeErr);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  timing_begin(s);
  hsize_pick_kernel<<<1, kPickThreads, 0, s>>>(err0, b0.wg, err1, b1.wg, (double)j0.rows * (double)j0.cols,
                                      (double)j1.rows * (double)j1.cols, j0.cols, kmax, k_out,
                                      mse_out);
  timing_end(s, kKHsizePick);
  j0.wg = b0.wg;
  j1.wg = b1.wg;
  return hipGetLastError();
}

}  // namespace hqlss
