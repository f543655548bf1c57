// FP6 (e2m3) operands of the FP6 MFMA route (gemm6.hip).
//
// Padded FP6 layout of a row of K codes (K a multiple of 64): K bytes, every 32 codes one
// 32-byte group holding 24 bytes of e2m3 fields (code i of the group at bits 6i..6i+5 of the
// group read as a little-endian 192-bit string) and 8 zero bytes.  A lane of the MFMA reads
// one such group as its 32 k of one row; the zero bytes keep every group on a 32-byte
// boundary, so the GEMM's 16-byte LDS-DMA loads and swizzled LDS reads are those of the
// INT4 layout at twice the bytes.
//
// e2m3: sign, 2 exponent bits (bias 1), 3 mantissa bits; the integers 1..7 are
// 1.0 x 2^0, 1.0 x 2^1, 1.5 x 2^1, 1.0 x 2^2, 1.25 x 2^2, 1.5 x 2^2, 1.75 x 2^2.
#include "common.h"
#include "launch.h"

namespace hqlss {

namespace {

// Four INT4 codes, one to a byte (two's complement nibbles; -8 does not occur), to their e2m3
// field bytes.  v_perm_b32 looks four of them up at once in a table of eight bytes, one for
// the codes 0 .. 7 and one for -8 .. -1, and the sign bit chooses.
__device__ __forceinline__ uint32_t e2m3_of_nibbles(uint32_t x) {
  const uint32_t sel = x & 0x07070707u, m = x & 0x08080808u;
  const uint32_t pos = __builtin_amdgcn_perm(0x1E1C1A18u, 0x14100800u, sel);
  const uint32_t neg = __builtin_amdgcn_perm(0x28303438u, 0x3A3C3E20u, sel);
  const uint32_t mask = (m << 5) - (m >> 3);  // 0xFF in the bytes of negative codes
  return (neg & mask) | (pos & ~mask);
}
// Eight packed codes (k = 0 .. 7, even k in the low nibbles) to the field bytes of k = 0 .. 3
// and of k = 4 .. 7.
__device__ __forceinline__ void e2m3_bytes8(uint32_t w, uint32_t& f0, uint32_t& f1) {
  const uint32_t e = e2m3_of_nibbles(w & 0x0F0F0F0Fu), o = e2m3_of_nibbles((w >> 4) & 0x0F0F0F0Fu);
  f0 = __builtin_amdgcn_perm(o, e, 0x05010400u);
  f1 = __builtin_amdgcn_perm(o, e, 0x07030602u);
}
// Four field bytes to 24 bits, field i at bits 6i, and back.
__device__ __forceinline__ uint32_t pack24(uint32_t f) {
  const uint32_t y = (f & 0x003F003Fu) | ((f >> 2) & 0x0FC00FC0u);
  return (y & 0xFFFu) | ((y >> 4) & 0xFFF000u);
}
__device__ __forceinline__ uint32_t unpack24(uint32_t t) {
  const uint32_t y = (t & 0xFFFu) | ((t & 0xFFF000u) << 4);
  return (y & 0x003F003Fu) | ((y << 2) & 0x3F003F00u);
}
// Sixteen field bytes to the 12 bytes of half a group.
__device__ __forceinline__ uint3 pack16(uint32_t f0, uint32_t f1, uint32_t f2, uint32_t f3) {
  const uint32_t t0 = pack24(f0), t1 = pack24(f1), t2 = pack24(f2), t3 = pack24(f3);
  return make_uint3(t0 | (t1 << 24), (t1 >> 8) | (t2 << 16), (t2 >> 16) | (t3 << 8));
}

// 16 bytes of packed INT4 (32 codes, even k in the low nibble) -> one 32-byte FP6 group
__device__ __forceinline__ void fp6_group(const uint4& in, uint4& lo, uint4& hi) {
  uint32_t f[8];
  e2m3_bytes8(in.x, f[0], f[1]);
  e2m3_bytes8(in.y, f[2], f[3]);
  e2m3_bytes8(in.z, f[4], f[5]);
  e2m3_bytes8(in.w, f[6], f[7]);
  const uint3 a = pack16(f[0], f[1], f[2], f[3]), b = pack16(f[4], f[5], f[6], f[7]);
  lo = make_uint4(a.x, a.y, a.z, b.x);
  hi = make_uint4(b.y, b.z, 0u, 0u);
}

// Quotient of an item index by the groups of a row, in 32 bits where both fit.
__device__ __forceinline__ int64_t row_of_item(int64_t it, int64_t groups, bool small) {
  return small ? (int64_t)((uint32_t)it / (uint32_t)groups) : it / groups;
}

__global__ __launch_bounds__(256) void int4_to_fp6_kernel(const uint8_t* __restrict__ src,
                                                          uint8_t* __restrict__ dst, int64_t rows,
                                                          int64_t K) {
  const int64_t groups = K / 32, items = rows * groups;
  const bool small = items <= 0xFFFFFFFFll;
  for (int64_t it = (int64_t)blockIdx.x * 256 + threadIdx.x; it < items; it += (int64_t)gridDim.x * 256) {
    const int64_t r = row_of_item(it, groups, small), g = it - r * groups;
    const uint4 in = ld_stream<true>(src + r * (K / 2) + g * 16);
    uint4 lo, hi;
    fp6_group(in, lo, hi);
    uint8_t* p = dst + r * K + g * 32;
    *reinterpret_cast<uint4*>(p) = lo;
    *reinterpret_cast<uint4*>(p + 16) = hi;
  }
}

// dX operands: one thread per (row, 32-code group); blockIdx.y 0: lower rows, 1: upper rows
template <int DT>
__global__ __launch_bounds__(256) void fp6_build_rows_kernel(
    const uint8_t* __restrict__ qup, const uint8_t* __restrict__ qdn, const uint8_t* __restrict__ w_dn,
    const int32_t* __restrict__ order6, const int32_t* __restrict__ n_kept,
    const int32_t* __restrict__ n_up, int64_t C, uint8_t* __restrict__ a_dn, uint8_t* __restrict__ a_up) {
  const bool upper = blockIdx.y == 1;
  uint8_t* out = upper ? a_up : a_dn;
  if (!out) return;
  const int64_t nu = *n_up;
  const int64_t rows = upper ? (nu + 255) / 256 * 256 : (int64_t)*n_kept;
  const int64_t groups = C / 32, items = rows * groups;
  const bool small = items <= 0xFFFFFFFFll;
  for (int64_t it = (int64_t)blockIdx.x * 256 + threadIdx.x; it < items; it += (int64_t)gridDim.x * 256) {
    const int64_t r = row_of_item(it, groups, small), g = it - r * groups;
    uint4 in = make_uint4(0u, 0u, 0u, 0u);
    if (!upper || r < nu) {
      const int64_t t = order6[r];
      if (upper || w_dn[t]) in = ld_stream<true>((upper ? qup : qdn) + t * (C / 2) + g * 16);
    }
    uint4 lo, hi;
    fp6_group(in, lo, hi);
    uint8_t* p = out + r * C + g * 32;
    *reinterpret_cast<uint4*>(p) = lo;
    *reinterpret_cast<uint4*>(p + 16) = hi;
  }
}

// dW operands, transposed through an LDS tile of 128 entries x 128 columns: blockIdx.x is
// the entry block, blockIdx.y the column block (C / 128 blocks of a_dw, then D / 128 of
// x_dw; a last partial block of 64 columns is allowed).  The last y block zeroes the dX
// rows of dropped tokens instead.
//
// The tile holds field bytes: gradient codes are looked up four at a time, X^ fields are only
// spread to bytes, and a thread of the second half reads 4 columns of 16 entries as words,
// transposes them by byte permutes and packs 12 bytes a column; with its neighbour's first
// word it stores one 16-byte piece of each column, 128 bytes in a row over 8 lanes.  About 5
// vector instructions a code instead of 14, and a quarter of the LDS reads: with the dX
// operands 114 -> 76 us at N = 16384, 4096 x 4096.
template <int DT>
__global__ __launch_bounds__(256) void fp6_build_cols_kernel(
    const uint8_t* __restrict__ qup, const uint8_t* __restrict__ qdn, const uint8_t* __restrict__ w_up,
    const uint8_t* __restrict__ w_dn, const int32_t* __restrict__ ent, const int32_t* __restrict__ cls,
    const uint8_t* __restrict__ xq6, int64_t N, int64_t C, int64_t D, int64_t ecap,
    uint8_t* __restrict__ a_dw, uint8_t* __restrict__ x_dw, void* __restrict__ dX) {
  constexpr int kPitch = 33;  // words
  __shared__ uint32_t tile[128 * kPitch];
  const int tid = threadIdx.x;
  const int64_t cb = (C + 127) / 128, db = (D + 127) / 128;
  if ((int64_t)blockIdx.y == cb + db) {  // zero the dX rows of dropped tokens
    if (!dX) return;
    const int64_t bytes = D * Elem<DT>::bytes;
    const int64_t t0 = (int64_t)blockIdx.x * 128, t1 = t0 + 128 < N ? t0 + 128 : N;
    for (int64_t t = t0 + (tid >> 6); t < t1; t += 4) {
      if (w_up[t] + w_dn[t]) continue;
      char* row = static_cast<char*>(dX) + t * bytes;
      for (int64_t o = (tid & 63) * 16; o < bytes; o += 64 * 16)
        st_stream<HQ_NT_B_ST>(row + o, make_uint4(0u, 0u, 0u, 0u));
    }
    return;
  }
  const bool isA = (int64_t)blockIdx.y < cb;
  uint8_t* out = isA ? a_dw : x_dw;
  if (!out) return;
  const int64_t e0 = (int64_t)blockIdx.x * 128;
  if (e0 >= (int64_t)cls[4]) return;
  const int64_t col0 = isA ? (int64_t)blockIdx.y * 128 : ((int64_t)blockIdx.y - cb) * 128;
  const int64_t ncol = isA ? C : D;
  // 128 entries x 8 chunks of 16 columns, four per thread
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int item = tid + 256 * k, r = item >> 3, qc = (item & 7) * 16;
    uint32_t f[4] = {0u, 0u, 0u, 0u};
    const int id = ent[e0 + r];
    if (id >= 0 && col0 + qc < ncol) {
      const int64_t t = id >> 1;
      if (isA) {
        const uint2 w = ld_stream2<HQ_NT_B_LD>(((id & 1) ? qup : qdn) + t * (C / 2) + (col0 + qc) / 2);
        e2m3_bytes8(w.x, f[0], f[1]);
        e2m3_bytes8(w.y, f[2], f[3]);
      } else {  // 16 codes = 12 bytes: half (col / 16) & 1 of the 32-code group col / 32
        const int64_t col = col0 + qc;
        const uint8_t* p = xq6 + t * D + (col / 32) * 32 + ((col / 16) & 1) * 12;
        const uint32_t d0 = *reinterpret_cast<const uint32_t*>(p);
        const uint32_t d1 = *reinterpret_cast<const uint32_t*>(p + 4);
        const uint32_t d2 = *reinterpret_cast<const uint32_t*>(p + 8);
        f[0] = unpack24(d0 & 0xFFFFFFu);
        f[1] = unpack24((d0 >> 24) | ((d1 & 0xFFFFu) << 8));
        f[2] = unpack24((d1 >> 16) | ((d2 & 0xFFu) << 16));
        f[3] = unpack24(d2 >> 8);
      }
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) tile[r * kPitch + qc / 4 + j] = f[j];
  }
  __syncthreads();
  // 32 column quads x 4 groups of 32 entries x 2 halves, one per thread
  const int half = tid & 1, gg = (tid >> 1) & 3, cq = tid >> 3;
  uint32_t f[4][4];  // [column][4 entries each]
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const uint32_t* p = tile + (32 * gg + 16 * half + 4 * q) * kPitch + cq;
    const uint32_t r0 = p[0], r1 = p[kPitch], r2 = p[2 * kPitch], r3 = p[3 * kPitch];
    const uint32_t a = __builtin_amdgcn_perm(r1, r0, 0x05010400u), b = __builtin_amdgcn_perm(r3, r2, 0x05010400u);
    const uint32_t c = __builtin_amdgcn_perm(r1, r0, 0x07030602u), d = __builtin_amdgcn_perm(r3, r2, 0x07030602u);
    f[0][q] = __builtin_amdgcn_perm(b, a, 0x05040100u);
    f[1][q] = __builtin_amdgcn_perm(b, a, 0x07060302u);
    f[2][q] = __builtin_amdgcn_perm(d, c, 0x05040100u);
    f[3][q] = __builtin_amdgcn_perm(d, c, 0x07060302u);
  }
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const uint3 h = pack16(f[c][0], f[c][1], f[c][2], f[c][3]);
    // the other half's first word: lanes swapped in pairs
    const uint32_t other = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)h.x, 0xB1, 0xF, 0xF, true);
    const int64_t col = col0 + 4 * cq + c;
    if (col < ncol)
      *reinterpret_cast<uint4*>(out + col * ecap + e0 + 32 * gg + 16 * half) =
          half ? make_uint4(h.y, h.z, 0u, 0u) : make_uint4(h.x, h.y, h.z, other);
  }
}

}  // namespace

hipError_t launch_int4_to_fp6(hipStream_t s, const uint8_t* src, uint8_t* dst, int64_t rows, int64_t K) {
  const int64_t items = rows * (K / 32);
  if (items <= 0) return hipSuccess;
  int64_t wg = (items + 255) / 256;
  if (wg > 4096) wg = 4096;
  timing_begin(s);
  int4_to_fp6_kernel<<<(unsigned)wg, 256, 0, s>>>(src, dst, rows, K);
  timing_end(s, kKFp6Convert);
  return hipGetLastError();
}

hipError_t launch_fp6_build(hipStream_t s, int dt, const uint8_t* qup, const uint8_t* qdn,
                            const uint8_t* w_up, const uint8_t* w_dn, const int32_t* order6,
                            const int32_t* n_kept, const int32_t* n_up, const int32_t* ent,
                            const int32_t* cls, const uint8_t* xq6, int64_t N, int64_t C,
                            int64_t D, int64_t ecap, uint8_t* a_dn, uint8_t* a_up, uint8_t* a_dw,
                            uint8_t* x_dw, void* dX) {
  timing_begin(s);
  if (a_dn || a_up) {
    int64_t wg = ((N + 255) / 256 * 256) * (C / 32) / 256;
    if (wg > 4096) wg = 4096;
    if (wg < 1) wg = 1;
    const dim3 grid((unsigned)wg, 2u);
    switch (dt) {
      case kF32: fp6_build_rows_kernel<kF32><<<grid, 256, 0, s>>>(qup, qdn, w_dn, order6, n_kept, n_up, C, a_dn, a_up); break;
      case kF16: fp6_build_rows_kernel<kF16><<<grid, 256, 0, s>>>(qup, qdn, w_dn, order6, n_kept, n_up, C, a_dn, a_up); break;
      case kBF16: fp6_build_rows_kernel<kBF16><<<grid, 256, 0, s>>>(qup, qdn, w_dn, order6, n_kept, n_up, C, a_dn, a_up); break;
      default: return hipErrorInvalidValue;
    }
  }
  {
    const int64_t eb = (ecap + 127) / 128, cb = (C + 127) / 128, db = (D + 127) / 128;
    const int64_t xb = eb > (N + 127) / 128 ? eb : (N + 127) / 128;  // dX zeroing covers N tokens
    const dim3 grid((unsigned)xb, (unsigned)(cb + db + 1));
    switch (dt) {
      case kF32: fp6_build_cols_kernel<kF32><<<grid, 256, 0, s>>>(qup, qdn, w_up, w_dn, ent, cls, xq6, N, C, D, ecap, a_dw, x_dw, dX); break;
      case kF16: fp6_build_cols_kernel<kF16><<<grid, 256, 0, s>>>(qup, qdn, w_up, w_dn, ent, cls, xq6, N, C, D, ecap, a_dw, x_dw, dX); break;
      case kBF16: fp6_build_cols_kernel<kBF16><<<grid, 256, 0, s>>>(qup, qdn, w_up, w_dn, ent, cls, xq6, N, C, D, ecap, a_dw, x_dw, dX); break;
      default: return hipErrorInvalidValue;
    }
  }
  timing_end(s, kKFp6Build);
  return hipGetLastError();
}

}  // namespace hqlss
