// General matrix-core contraction (gfx950): sum-of-products blocks whose sizes, layouts or element types none of the
// specialised families take -- fp32 products, odd or unaligned extents, A stored [k][m], three input channels,
// transposed convolutions.
//
// The planner splits the block's indexes by the operands that use them (Section 3.2: every access is affine): indexes of
// A and the output form the rows m, indexes of B and the output the columns n, reduction indexes k, indexes of all three
// a batch.  An index of a shared output element (O[2y + i]: y of A, i of B) is rewritten first: with i = 2*i1 + i0 and
// y' = y + i1 the output is O[2y' + i0], one owner per element, and i1 is a reduction index; 0 <= y' - i1 < Y and
// 2*i1 + i0 < R become range tests.  What the atomic form did in 117 us (stride-2 transposed 3x3, 8 x 28 x 28 x 32) then
// is a product like any other.
//
// Operands are fetched through buffer loads: a point outside the
// polyhedron or the tile's remainder gets an offset beyond the buffer's range and the load returns zero, so no select
// follows.  The range is the operand's declared buffer: a constraint is tested for one operand (that suffices for the
// sum, one factor is zero), so the other one may be fetched at a removed point, where its address is not the block's to
// read.  It is then fetched element by element, and an element outside the buffer loads as zero.  Ways to fetch, chosen per operand
// by the planner: 16 or 8 bytes along k; vectors along the row index; or element by element with neighbouring lanes on
// neighbouring k.  Tiles go registers -> LDS, k-contiguous operands as rows of k, the others as they lie in memory, lines of
// rows that the transposing LDS reads turn (Stager, KMajor); a 16-byte fragment is one
// 16x16x32 bf16 / 16x16x64 int8 instruction or four 16x16x4 fp32 ones; sums are fp32 / int32 throughout.
// Two kernels: many tiles are shared by four wavefronts each (contract_kernel), few tiles by eight or sixteen that share the
// reduction out (contract_waves_kernel); tile_us() has what each tile takes.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <type_traits>
#include <vector>

#include "contract.hpp"
#include "kernels.hpp"

namespace stripe {
namespace {

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef int32_t i32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));

constexpr int kFar = -0x40000000;          // a range-test value no other part can bring back into range
[[maybe_unused]] constexpr uint32_t kTop = 0x3fffffffu;     // "no upper end"
constexpr int kNoStore = 0x3fffffff;       // a part of an output bound that no bound reaches, alone or twice
constexpr uint32_t kOutside = 0x80000000u; // byte offset beyond every buffer's range: the load returns zero
[[maybe_unused]] constexpr uint32_t kRecords = 0x7fffffffu; // largest range of a buffer

__device__ __forceinline__ uint32_t fast_div(uint32_t v, uint32_t mul, int shift) { return __umulhi(v, mul) >> shift; }

// calls f(index number, value) for the indexes of a flat position; unused slots (range, mul 0) get 0.  Without branches, so
// that the parameters stay in scalar registers.
template <typename F>
__device__ __forceinline__ void decode(const CtIndex& ix, uint32_t v, F f) {
#pragma unroll
  for (int j = 0; j < kCtIdx; ++j) {
    const uint32_t q = fast_div(v, ix.mul[j], ix.shift[j]);
    f(j, (int)(v - q * ix.range[j]));
    v = q;
  }
}

// The launch parameters, read again: what only the end of the kernel needs is not kept in scalar registers through the main
// loop (the float kernels spilled up to 170 of them there; int8's spill few, and the reads would cost them 10 % where a workgroup
// has one K tile).
struct KernelArgs {
  ContractParams p;
  const void *a, *b;
  void* o;
  const float* bias;
};
__device__ __forceinline__ const KernelArgs& reread() {
  auto at = __builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(at));
  return *(const KernelArgs*)at;
}

struct KPart {
  int off, t0, t1;
  int run;        // elements from here to the end of the innermost index's real range
};

// `side_a` may differ between lanes
__device__ __forceinline__ KPart k_part(const ContractParams& p, uint32_t k, bool side_a) {
  KPart r = {0, 0, 0, 0};
  auto add = [&](int j, int v) {
    if (j == 0) r.run = p.k_run - v;
    r.off += (side_a ? p.k_a[j] : p.k_b[j]) * v;
    r.t0 += (side_a ? p.ka_t[0][j] : p.kb_t[0][j]) * v;
    r.t1 += (side_a ? p.ka_t[1][j] : p.kb_t[1][j]) * v;
  };
  if (p.k.n == 1) add(0, (int)k);
  else decode(p.k, k, add);
  if (k >= p.K || r.run <= 0) r.t0 = kFar;
  return r;
}

template <typename T>
struct Ct;
template <>
struct Ct<uint16_t> {
  using Acc = f32x4;
  using S = float;
  [[maybe_unused]] static constexpr int KP = 2, V = 8;      // elements per dword; rows per vector of the row-wise fetch
  static __device__ __forceinline__ Acc mma(u32x4 a, u32x4 b, Acc c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
  }
  // a 64-byte step's products, summed from zero
  static __device__ __forceinline__ Acc step(u32x4 a, u32x4 b) { return mma(a, b, (Acc){0.f, 0.f, 0.f, 0.f}); }
  static __device__ __forceinline__ S widen(uint16_t v) { return __uint_as_float((uint32_t)v << 16); }
  static __device__ __forceinline__ bool finite(uint32_t w) { return ((w & 0x7f80u) != 0x7f80u) & ((w & 0x7f800000u) != 0x7f800000u); }
};
template <>
struct Ct<int8_t> {
  using Acc = i32x4;
  using S = int32_t;
  [[maybe_unused]] static constexpr int KP = 4, V = 8;
  static __device__ __forceinline__ Acc mma(u32x4 a, u32x4 b, Acc c) {
    return __builtin_amdgcn_mfma_i32_16x16x64_i8(__builtin_bit_cast(i32x4, a), __builtin_bit_cast(i32x4, b), c, 0, 0, 0);
  }
  static __device__ __forceinline__ S widen(int8_t v) { return v; }
  static __device__ __forceinline__ bool finite(uint32_t) { return true; }
};
template <>
struct Ct<float> {
  using Acc = f32x4;
  using S = float;
  [[maybe_unused]] static constexpr int KP = 1, V = 4;
  static __device__ __forceinline__ Acc mma(u32x4 a, u32x4 b, Acc c) {
    const f32x4 x = __builtin_bit_cast(f32x4, a), y = __builtin_bit_cast(f32x4, b);
#pragma unroll
    for (int i = 0; i < 4; ++i) c = __builtin_amdgcn_mfma_f32_16x16x4f32(x[i], y[i], c, 0, 0, 0);
    return c;
  }
  static __device__ __forceinline__ Acc step(u32x4 a, u32x4 b) {     // as two chains of eight products
    const f32x4 x = __builtin_bit_cast(f32x4, a), y = __builtin_bit_cast(f32x4, b);
    Acc t[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) t[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[2 * i], y[2 * i], (Acc){0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
#pragma unroll
    for (int i = 0; i < 2; ++i) t[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[2 * i + 1], y[2 * i + 1], t[i], 0, 0, 0);
    return t[0] + t[1];
  }
  static __device__ __forceinline__ S widen(float v) { return v; }
  static __device__ __forceinline__ bool finite(uint32_t w) { return (w & 0x7f800000u) != 0x7f800000u; }
};

template <typename T>
__device__ __forceinline__ uint32_t load_elem(__amdgpu_buffer_rsrc_t r, uint32_t off) {
  if constexpr (sizeof(T) == 4) return __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0);
  else if constexpr (sizeof(T) == 2) return __builtin_amdgcn_raw_buffer_load_b16(r, off, 0, 0);
  else return __builtin_amdgcn_raw_buffer_load_b8(r, off, 0, 0);
}

template <int E>
struct Bits {
  using type = typename std::conditional<E == 4, uint32_t, typename std::conditional<E == 2, uint16_t, uint8_t>::type>::type;
};

// How a tile lies in LDS.  Row-major operands: rows of BKB bytes of k whose 16-byte chunks are swizzled with the row, so that the
// 16 rows of a fragment read cover all banks.
template <int BKB>
__device__ __forceinline__ constexpr uint32_t row_key(uint32_t row) {      // 16 chunks are one sweep over the banks
  return BKB >= 256 ? row & 15 : BKB == 128 ? (row >> 1) & 7 : (row >> 2) & 3;
}
template <int BKB>
__device__ __forceinline__ constexpr uint32_t row_at(uint32_t row, uint32_t chunk) {
  return row * BKB + ((chunk ^ row_key<BKB>(row)) << 4);
}
// Operands fetched along their row index stay as they lie in memory, a line of ROWS elements per k; fragments are read with
// the transposing LDS reads (fp32: element by element).  A half wavefront of such a read meets 8 (bf16), 4 (fp32) or 16 (int8)
// values of k whose lines must fall on different banks: they differ in the bits of k listed here.  As many of them as a line
// has groups of 16 rows are exclusive-ored onto the group, the others become the lowest bits of the line's number.
template <typename T, int ROWS>
struct KMajor {
  static constexpr int E = sizeof(T), BITS = E == 2 ? 3 : E == 4 ? 2 : 4, STEP_BITS = E == 2 ? 5 : E == 4 ? 4 : 6;
  static constexpr int LINE = ROWS * E, GROUPS = ROWS / 16, LG = GROUPS >= 8 ? 3 : GROUPS >= 4 ? 2 : GROUPS >= 2 ? 1 : 0;
  static constexpr int LOW = BITS > LG ? BITS - LG : 0;
  static __device__ __forceinline__ constexpr int bit(int t) { return E == 2 ? (t == 2 ? 3 : t) : E == 4 ? t + 2 : (t == 3 ? 4 : t); }
  static __device__ __forceinline__ constexpr bool low(int b) {
    for (int t = 0; t < LOW; ++t)
      if (bit(t) == b) return true;
    return false;
  }
  static __device__ __forceinline__ constexpr uint32_t line(uint32_t k) {       // k -> number of its line
    uint32_t out = k >> STEP_BITS << STEP_BITS;
    int pos = 0;
    for (int t = 0; t < LOW; ++t) out |= (k >> bit(t) & 1) << pos++;
    for (int b = 0; b < STEP_BITS; ++b)
      if (!low(b)) out |= (k >> b & 1) << pos++;
    return out;
  }
  static __device__ __forceinline__ constexpr uint32_t k_of(uint32_t line) {
    uint32_t out = line >> STEP_BITS << STEP_BITS;
    int pos = 0;
    for (int t = 0; t < LOW; ++t) out |= (line >> pos++ & 1) << bit(t);
    for (int b = 0; b < STEP_BITS; ++b)
      if (!low(b)) out |= (line >> pos++ & 1) << b;
    return out;
  }
  static __device__ __forceinline__ constexpr uint32_t key(uint32_t k) {
    uint32_t out = 0;
    for (int t = LOW; t < BITS; ++t) out |= (k >> bit(t) & 1) << (t - LOW);
    return out;
  }
  static __device__ __forceinline__ constexpr uint32_t at(uint32_t k, uint32_t row) {
    return line(k) * LINE + ((row / 16) ^ key(k)) * (16 * E) + row % 16 * E;
  }
};

// One operand's share of a K tile: ROWS x BKB bytes over NT lanes, DW dwords each.  MODE: how it is fetched (see
// ContractParams::mode_a); a template parameter, so that the loads of a K tile are straight-line code: with the forms
// behind branches the compiler waits for each load at the join.
template <typename T, int NT, int ROWS, int BKB, bool SIDE_A, int MODE>
struct Stager {
  static constexpr int E = sizeof(T), KP = Ct<T>::KP, V = Ct<T>::V;
  static constexpr int DW = ROWS * BKB / 4 / NT;
  static constexpr int CH = BKB / 16, STEP1 = NT / CH, VE = 16 / E;          // mode 1: vectors of VE along k
  static constexpr int KD = BKB / 4, STEP0 = NT / KD;                        // mode 0: dwords of KP along k
  static constexpr int G = ROWS / V, STEP2 = NT / G, UD = V * E / 4;         // mode 2: groups of V rows, UD dwords each, neighbouring groups on neighbouring lanes
  static constexpr int CH3 = BKB / 8, STEP3 = NT / CH3, VE3 = 8 / E;          // mode 3: vectors of 8 bytes along k
  static_assert(DW % 4 == 0, "whole vectors per lane");
  using L = KMajor<T, ROWS>;
  static constexpr int SPAN = MODE == 1 ? VE : MODE == 3 ? VE3 : 1, ENTRIES = BKB / E / SPAN;   // k per table entry, entries of a K tile
  static constexpr int NR = MODE == 1 ? DW / 4 : MODE == 3 ? DW / 2 : MODE == 2 ? 1 : 0;      // rows whose entries a lane keeps
  uint32_t r[DW];
  uint32_t back[MODE == 3 ? DW / 2 : 1];     // mode 3: bits a vector was fetched early (it would end behind the operand)
  uint64_t mask = 0;                         // mode 3: the vector's elements inside the innermost index's range

  // the row entries a lane's loads need in every K tile
  static __device__ __forceinline__ void keep(const i32x4* rows, i32x4* row, int tid) {
#pragma unroll
    for (int i = 0; i < NR; ++i) row[i] = rows[MODE == 1 ? tid / CH + i * STEP1 : MODE == 3 ? tid / CH3 + i * STEP3 : tid % G * V];
  }

  static __device__ __forceinline__ uint32_t place(const ContractParams& p, const i32x4 row, const i32x4 k) {
    const bool ok = ((uint32_t)(row[1] + k[1]) <= (SIDE_A ? p.top_a[0] : p.top_b[0])) & ((uint32_t)(row[2] + k[2]) <= (SIDE_A ? p.top_a[1] : p.top_b[1]));
    return ok ? (uint32_t)(row[0] + k[0]) * E : kOutside;
  }

  __device__ __forceinline__ void load(const ContractParams& p, __amdgpu_buffer_rsrc_t buf, const i32x4* rows, const i32x4* row, const i32x4* ks, uint32_t k0, int tid) {
    if constexpr (MODE == 1) {
      const uint32_t k = k0 + (tid % CH) * VE;
      i32x4 kp = ks[tid % CH];
      if (k < p.K && k + VE > p.K) kp[0] -= (int)(k + VE - p.K);    // a row's last, partial vector is fetched from earlier on; store() shifts it down
#pragma unroll
      for (int i = 0; i < DW / 4; ++i) {
        const u32x4 x = __builtin_amdgcn_raw_buffer_load_b128(buf, place(p, row[i], kp), 0, 0);
#pragma unroll
        for (int e = 0; e < 4; ++e) r[4 * i + e] = x[e];
      }
    } else if constexpr (MODE == 3) {
      const i32x4 kp = ks[tid % CH3];
      const uint32_t last = (SIDE_A ? p.bytes_a : p.bytes_b) - 8;
      mask = kp[3] >= VE3 ? ~0ull : kp[3] <= 0 ? 0ull : (1ull << (8 * E * kp[3])) - 1;
#pragma unroll
      for (int i = 0; i < DW / 2; ++i) {
        const uint32_t off = place(p, row[i], kp);
        const bool late = off > last && off != kOutside;
        back[i] = late ? (off - last) * 8 : 0;
        const u32x2 x = __builtin_amdgcn_raw_buffer_load_b64(buf, late ? last : off, 0, 0);
        r[2 * i] = x[0];
        r[2 * i + 1] = x[1];
      }
    } else if constexpr (MODE == 2) {
#pragma unroll
      for (int i = 0; i < DW / UD; ++i) {
        const uint32_t off = place(p, row[0], ks[L::k_of(tid / G + i * STEP2)]);
        if constexpr (UD == 4) {
          const u32x4 x = __builtin_amdgcn_raw_buffer_load_b128(buf, off, 0, 0);
#pragma unroll
          for (int e = 0; e < 4; ++e) r[4 * i + e] = x[e];
        } else {
          const u32x2 x = __builtin_amdgcn_raw_buffer_load_b64(buf, off, 0, 0);
          r[2 * i] = x[0];
          r[2 * i + 1] = x[1];
        }
      }
    } else {
      i32x4 kp[KP];
#pragma unroll
      for (int q = 0; q < KP; ++q) kp[q] = ks[(tid % KD) * KP + q];
#pragma unroll
      for (int i = 0; i < DW; ++i) {
        const i32x4 ri = rows[tid / KD + i * STEP0];
        uint32_t w = 0;
#pragma unroll
        for (int q = 0; q < KP; ++q) w |= load_elem<T>(buf, place(p, ri, kp[q])) << (8 * E * q % 32);
        r[i] = w;
      }
    }
  }

  // The same for an operand with one row index, one reduction index and no tests (a plain product): row[i] holds the row's
  // byte offset (beyond every buffer for a row past the end), step is the reduction index's stride in bytes.
  __device__ __forceinline__ void load_plain(const ContractParams& p, __amdgpu_buffer_rsrc_t buf, const uint32_t* row, uint32_t step, uint32_t k0, int tid) {
    static_assert(MODE == 1 || MODE == 2, "vectors along k or along the rows");
    if constexpr (MODE == 1) {
      const uint32_t k = k0 + (tid % CH) * VE, at = k + VE <= p.K ? k : p.K - VE;
#pragma unroll
      for (int i = 0; i < DW / 4; ++i) {
        const u32x4 x = __builtin_amdgcn_raw_buffer_load_b128(buf, k < p.K ? row[i] + at * E : kOutside, 0, 0);
#pragma unroll
        for (int e = 0; e < 4; ++e) r[4 * i + e] = x[e];
      }
    } else {
#pragma unroll
      for (int i = 0; i < DW / UD; ++i) {
        const uint32_t k = k0 + L::k_of(tid / G + i * STEP2), off = k < p.K ? row[0] + k * step : kOutside;
        if constexpr (UD == 4) {
          const u32x4 x = __builtin_amdgcn_raw_buffer_load_b128(buf, off, 0, 0);
#pragma unroll
          for (int e = 0; e < 4; ++e) r[4 * i + e] = x[e];
        } else {
          const u32x2 x = __builtin_amdgcn_raw_buffer_load_b64(buf, off, 0, 0);
          r[2 * i] = x[0];
          r[2 * i + 1] = x[1];
        }
      }
    }
  }

  // -> LDS; returns whether every value is finite
  __device__ __forceinline__ bool store(const ContractParams& p, unsigned char* lds, uint32_t k0, bool look, int tid) {
    bool fin = true;
    if constexpr (MODE == 3) {
#pragma unroll
      for (int i = 0; i < DW / 2; ++i) {
        const uint64_t x = ((r[2 * i] | (uint64_t)r[2 * i + 1] << 32) >> back[i]) & mask;
        r[2 * i] = (uint32_t)x;
        r[2 * i + 1] = (uint32_t)(x >> 32);
      }
    }
    if (look) {
#pragma unroll
      for (int i = 0; i < DW; ++i) fin &= Ct<T>::finite(r[i]);
    }
    if constexpr (MODE == 1) {
      if (p.K % VE && k0 + CH * VE > p.K) {      // uniform: the last K tile
        const uint32_t k = k0 + (tid % CH) * VE;
        const uint32_t drop = k < p.K && k + VE > p.K ? (k + VE - p.K) * E : 0;   // bytes that belong to the vector before
#pragma unroll
        for (int i = 0; i < DW / 4; ++i) {
          uint64_t lo = r[4 * i] | (uint64_t)r[4 * i + 1] << 32, hi = r[4 * i + 2] | (uint64_t)r[4 * i + 3] << 32;
          if (drop & 8) { lo = hi; hi = 0; }
          const uint32_t bits = (drop & 7) * 8;
          if (bits) { lo = lo >> bits | hi << (64 - bits); hi >>= bits; }
          r[4 * i] = (uint32_t)lo; r[4 * i + 1] = (uint32_t)(lo >> 32);
          r[4 * i + 2] = (uint32_t)hi; r[4 * i + 3] = (uint32_t)(hi >> 32);
        }
      }
#pragma unroll
      for (int i = 0; i < DW / 4; ++i)
        *(u32x4*)(lds + row_at<BKB>(tid / CH + i * STEP1, tid % CH)) = (u32x4){r[4 * i], r[4 * i + 1], r[4 * i + 2], r[4 * i + 3]};
    } else if constexpr (MODE == 3) {
#pragma unroll
      for (int i = 0; i < DW / 2; ++i) *(u32x2*)(lds + row_at<BKB>(tid / CH3 + i * STEP3, tid % CH3 / 2) + tid % 2 * 8) = (u32x2){r[2 * i], r[2 * i + 1]};
    } else if constexpr (MODE == 2) {
#pragma unroll
      for (int i = 0; i < DW / UD; ++i) {
        unsigned char* at = lds + L::at(L::k_of(tid / G + i * STEP2), tid % G * V);
        if constexpr (UD == 4) *(u32x4*)at = (u32x4){r[4 * i], r[4 * i + 1], r[4 * i + 2], r[4 * i + 3]};
        else *(u32x2*)at = (u32x2){r[2 * i], r[2 * i + 1]};
      }
    } else {
#pragma unroll
      for (int i = 0; i < DW; ++i) *(uint32_t*)(lds + row_at<BKB>(tid / KD + i * STEP0, tid % KD / 4) + tid % 4 * 4) = r[i];
    }
    return fin;
  }

  // Fragment reads.  first(): a lane's address for the fragment of 16 rows from `row` on in step 0; fragment(): its 16 bytes of
  // k in a 64-byte step.
  static __device__ __forceinline__ uint32_t first(uint32_t row, int lane) {
    if constexpr (MODE != 2) return row_at<BKB>(row + lane % 16, lane / 16);
    else if constexpr (E == 4) return L::at(lane / 16 * 4, row + lane % 16);
    else if constexpr (E == 2) return L::at(lane / 16 * 8 + lane % 16 / 4, row + lane % 4 * 4);
    else return L::at(lane / 16 * 16 + lane % 16 / 2, row + lane % 2 * 8);
  }
  static __device__ __forceinline__ u32x4 fragment(const unsigned char* lds, uint32_t first, int step) {
    if constexpr (MODE != 2) {
      return *(const u32x4*)(lds + (first ^ (uint32_t)(step << 6)));
    } else {
      const unsigned char* at = lds + first + step * (64 / E * L::LINE);
      if constexpr (E == 4) {
        u32x4 v;
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = *(const uint32_t*)(at + L::line(i) * L::LINE);
        return v;
      } else {
        const u32x2 lo = transposed(at), hi = transposed(at + L::line(E == 2 ? 4 : 8) * L::LINE);
        return (u32x4){lo[0], lo[1], hi[0], hi[1]};
      }
    }
  }
  // 16 lanes receive 16 columns of 4 (2-byte elements) or 8 (1-byte) lines: lane p gives the address of 8 bytes of line p / 4 (p / 2)
  static __device__ __forceinline__ u32x2 transposed(const unsigned char* at) {
    if constexpr (E == 2) {
      typedef short s4 __attribute__((ext_vector_type(4)));
      return __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s4*)at));
    } else {
      typedef int i2 __attribute__((ext_vector_type(2)));
      return __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr8_b64_v2i32((__attribute__((address_space(3))) i2*)at));
    }
  }
  // 16 bytes of one row's k from k = 16 / E * chunk on
  static __device__ __forceinline__ u32x4 piece(const unsigned char* lds, uint32_t row, uint32_t chunk) {
    if constexpr (MODE != 2) {
      return *(const u32x4*)(lds + row_at<BKB>(row, chunk));
    } else {
      u32x4 v = {0, 0, 0, 0};
#pragma unroll
      for (int e = 0; e < VE; ++e) v[e * E / 4] |= (uint32_t)(*(const typename Bits<E>::type*)(lds + L::at(chunk * VE + e, row))) << (8 * E * e % 32);
      return v;
    }
  }
};

// one output element, through the launch's epilogue
template <typename S>
__device__ __forceinline__ void put(const ContractParams& p, void* O, const float* bias, int off, uint32_t n, S v) {
  if constexpr (std::is_same<S, float>::value) {
    if (p.epilogue >= 2) v = v + bias[n] > 0.f ? v + bias[n] : 0.f;
    if (p.epilogue & 1) {
      ((__bf16*)O)[off] = (__bf16)v;
      return;
    }
  }
  ((S*)O)[off] = v;
}

// LDS of a workgroup in bytes, as the two kernels below declare it: staging buffers, row tables, k tables.
constexpr int k_entries(int esize, int bkb, int mode) { return bkb / (mode == 1 ? 16 : mode == 3 ? 8 : esize); }
constexpr int shared_lds_bytes(int esize, int bm, int bn, int bkb, int mode_a, int mode_b) {
  const int entries = k_entries(esize, bkb, mode_a) + k_entries(esize, bkb, mode_b), batch = 8 * entries <= 256 ? 8 : 4 * entries <= 256 ? 4 : 2 * entries <= 256 ? 2 : 1;
  return (bm + bn) * (2 * bkb + 24) + 2 * batch * entries * 16;
}
constexpr int waves_lds_bytes(int esize, int waves, int bm, int bn, int bkb, int mode_a, int mode_b, bool precise, bool plain) {
  const int stage = waves * (bm + bn) * bkb, part = (waves - 1) * bm * bn * (precise ? 8 : 4), bkb_again = 16 * 64 * waves / bm;
  const int again = plain || esize == 1 ? 0 : (bm + bn) * bkb_again + 2 * bkb_again / esize * 16, most = stage > part ? stage : part;
  const int entries = k_entries(esize, bkb, mode_a) + k_entries(esize, bkb, mode_b), tables = 4 * entries <= 64 ? 4 : 2 * entries <= 64 ? 2 : 1;
  return (most > again ? most : again) + (bm + bn) * 24 + (plain ? 0 : waves * tables * entries * 16);
}

// What every kernel below does first: the row tables of its tile.
struct TileRows {
  i32x4 *a, *b;      // {input offset, range-test values, output offset}
  int2 *ob_m, *ob_n;
};
template <typename T, int NT, int BM, int BN, int MA, int MB>
__device__ __forceinline__ void fill_rows(const ContractParams& p, uint32_t m0, uint32_t n0, int a_base, int b_base, const TileRows& rows) {
  for (int i = threadIdx.x; i < BM + BN; i += NT) {
    const bool am = i < BM;
    uint32_t at = am ? m0 + i : n0 + i - BM;
    // Vectors along the row index: the operand's last, partial group of V rows starts V rows before its end instead.  The
    // rows it shares with the group before are computed twice.  Where that group is another workgroup's, only that one
    // stores them (the two may differ in rounding: one of them may have summed its tile again, see below).
    constexpr uint32_t V = Ct<T>::V;
    const uint32_t end = am ? p.M : p.N;
    if ((am ? MA : MB) == 2 && at / V * V < end && at / V * V + V > end) at = end - V + at % V;
    i32x4 e = {am ? a_base : b_base, am ? p.c_a[0] : p.c_b[0], am ? p.c_a[1] : p.c_b[1], 0};
    int2 ob = {at < (am ? m0 : n0) ? kNoStore : 0, 0};
    if (am) {
      decode(p.m, at, [&](int j, int v) {
        e[0] += p.m_in[j] * v; e[1] += p.m_t[0][j] * v; e[2] += p.m_t[1][j] * v; e[3] += p.m_out[j] * v;
        ob.x += p.m_ob[0][j] * v; ob.y += p.m_ob[1][j] * v;
      });
      if (at >= p.M) e[1] = kFar;
      rows.a[i] = e;
      rows.ob_m[i] = ob;
    } else {
      decode(p.n, at, [&](int j, int v) {
        e[0] += p.n_in[j] * v; e[1] += p.n_t[0][j] * v; e[2] += p.n_t[1][j] * v; e[3] += p.n_out[j] * v;
        ob.x += p.n_ob[0][j] * v; ob.y += p.n_ob[1][j] * v;
      });
      if (at >= p.N) e[1] = kFar;
      rows.b[i - BM] = e;
      rows.ob_n[i - BM] = ob;
    }
  }
}

// Stores fragments (i, j) of the tile whose number is MINE modulo WK; m_at, n_at: the wavefront's place in the tile.
template <typename T, int FM, int FN, int WK, typename Total>
__device__ __forceinline__ void store_fragments(const ContractParams& q, void* out, const float* bias_n, int o_base, const TileRows& rows, int m_at, int n_at,
                                                int wk, int lane, const Total (&acc)[FM][FN]) {
  using S = typename Ct<T>::S;
  const int frag_row = lane & 15, frag_k = lane >> 4;
#pragma unroll
  for (int j = 0; j < FN; ++j) {
    const int ni = n_at + j * 16 + frag_k * 4;
    int n_off[4];
    bool n_in[4];
    int2 on[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const i32x4 rn = rows.b[ni + e];
      n_off[e] = rn[3];
      n_in[e] = rn[1] != kFar;
      on[e] = rows.ob_n[ni + e];
    }
    float bs[4] = {0.f, 0.f, 0.f, 0.f};
    if (q.epilogue >= 2) {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (n_in[e]) bs[e] = bias_n[n_off[e]];      // one column index of unit output stride
    }
#pragma unroll
    for (int i = 0; i < FM; ++i) {
      if ((i * FN + j) % WK != wk) continue;
      const int mi = m_at + i * 16 + frag_row;
      const i32x4 rm = rows.a[mi];
      if (rm[1] == kFar) continue;
      const int off = o_base + rm[3];
      const int2 om = rows.ob_m[mi];
      S v[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        v[e] = (S)acc[i][j][e];
        if constexpr (std::is_same<S, float>::value) {
          if (q.epilogue >= 2) v[e] = v[e] + bs[e] > 0.f ? v[e] + bs[e] : 0.f;
        }
      }
      const bool half = std::is_same<S, float>::value && (q.epilogue & 1);
      // the planner: four columns from a multiple of four are neighbours and share the bound
      if (q.vec_out && n_in[0]) {
        if (om.x + on[0].x <= q.ob[0] && om.y + on[0].y <= q.ob[1]) {
          typedef S s4 __attribute__((ext_vector_type(4)));
          if (half) *(bf16x4*)((uint16_t*)out + off + n_off[0]) = __builtin_convertvector((f32x4){(float)v[0], (float)v[1], (float)v[2], (float)v[3]}, bf16x4);
          else *(s4*)((S*)out + off + n_off[0]) = (s4){v[0], v[1], v[2], v[3]};
        }
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (n_in[e] && om.x + on[e].x <= q.ob[0] && om.y + on[e].y <= q.ob[1]) {
            if (half) ((__bf16*)out)[off + n_off[e]] = (__bf16)(float)v[e];
            else ((S*)out)[off + n_off[e]] = v[e];
          }
      }
    }
  }
}

// The block's batch indexes, from the grid's second dimension.
__device__ __forceinline__ void batch_bases(const ContractParams& p, int* a_base, int* b_base, int* o_base) {
  *a_base = p.a_base;
  *b_base = p.b_base;
  *o_base = p.o_base;
  uint32_t t = blockIdx.y;     // unused batch indexes: range 1
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int v = (int)(t % p.batch_range[j]);
    t /= p.batch_range[j];
    *a_base += p.batch_a[j] * v;
    *b_base += p.batch_b[j] * v;
    *o_base += p.batch_o[j] * v;
  }
}

// A removed point contributes 0 * x, which is not 0 where x is an infinity or NaN: a tile that met one is summed again
// (Definition 2: a removed point contributes nothing).  The operands are staged as before, in parts of at most 64 x 32 outputs;
// 16 bytes of k at a time are summed, and only where such a sum is NaN are its points looked at one by one.  (Point by point from
// memory, one infinity in the images of the 3 -> 64-channel 7x7 convolution at 8 x 224 x 224 made the call take 2456 us, with
// this 122; its literal kernel takes 215.)  All lanes of the workgroup; lds: (BM + BN) * BKB bytes and 16 bytes for each table entry.
template <typename T, int NT, int BM, int BN, int BKB, int MA, int MB>
__device__ __forceinline__ void sum_again(const KernelArgs& args, const TileRows& rows, int o_base, unsigned char* lds) {
  using S = typename Ct<T>::S;
  using SA = Stager<T, NT, BM, BKB, true, MA>;
  using SB = Stager<T, NT, BN, BKB, false, MB>;
  constexpr uint32_t BK = BKB / sizeof(T);
  const ContractParams& q = args.p;
  const int tid = threadIdx.x;
  i32x4 *const ks_a = (i32x4*)(lds + (BM + BN) * BKB), *const ks_b = ks_a + SA::ENTRIES;
  // lanes: 16 x 16 for a part, as many parts at a time as there are such sets of lanes
  constexpr int SM = BM < 64 ? BM : 64, SN = BN < 32 ? BN : 32, RM = SM / 16, RN = SN / 16, VE = 16 / sizeof(T);
  constexpr int PARTS = BM / SM * (BN / SN), AT_ONCE = NT / 256;
  const int lm = tid / 16 % 16, ln = tid % 16;
  auto element = [](u32x4 v, int e) {
    if constexpr (sizeof(T) == 2) return __uint_as_float(e % 2 ? v[e / 2] & 0xffff0000u : v[e / 2] << 16);
    else return __uint_as_float(v[e]);
  };
  const uint32_t n_kt = (q.K + BK - 1) / BK;
  for (int part0 = 0; part0 < PARTS; part0 += AT_ONCE) {
    const int part = part0 + tid / 256 < PARTS ? part0 + tid / 256 : PARTS - 1;      // a set without a part of its own repeats the last one
    const int pm = part / (BN / SN) * SM + lm, pn = part % (BN / SN) * SN + ln;
    double total[RM][RN];
#pragma unroll
    for (int i = 0; i < RM; ++i)
#pragma unroll
      for (int j = 0; j < RN; ++j) total[i][j] = 0;
    for (uint32_t kt = 0; kt < n_kt; ++kt) {
      __syncthreads();
      for (int x = tid; x < SA::ENTRIES + SB::ENTRIES; x += NT) {
        const bool a = x < SA::ENTRIES;
        const KPart k = k_part(q, kt * BK + (a ? x * SA::SPAN : (x - SA::ENTRIES) * SB::SPAN), a);
        ks_a[x] = (i32x4){k.off, k.t0, k.t1, k.run};
      }
      __syncthreads();
      SA one_a;
      SB one_b;
      i32x4 row_a[SA::NR + 1], row_b[SB::NR + 1];
      SA::keep(rows.a, row_a, tid);
      SB::keep(rows.b, row_b, tid);
      one_a.load(q, __builtin_amdgcn_make_buffer_rsrc((void*)args.a, 0, (int)q.bytes_a, 0x00020000), rows.a, row_a, ks_a, kt * BK, tid);
      one_b.load(q, __builtin_amdgcn_make_buffer_rsrc((void*)args.b, 0, (int)q.bytes_b, 0x00020000), rows.b, row_b, ks_b, kt * BK, tid);
      one_a.store(q, lds, kt * BK, false, tid);
      one_b.store(q, lds + BM * BKB, kt * BK, false, tid);
      __syncthreads();
#pragma unroll 1
      for (int c = 0; c < BKB / 16; ++c) {
        u32x4 av[RM], bv[RN];
#pragma unroll
        for (int i = 0; i < RM; ++i) av[i] = SA::piece(lds, pm + 16 * i, c);
#pragma unroll
        for (int j = 0; j < RN; ++j) bv[j] = SB::piece(lds + BM * BKB, pn + 16 * j, c);
#pragma unroll
        for (int i = 0; i < RM; ++i)
#pragma unroll
          for (int j = 0; j < RN; ++j) {
            float s = 0.f;
#pragma unroll
            for (int e = 0; e < VE; ++e) s = __builtin_fmaf(element(av[i], e), element(bv[j], e), s);
            if (s != s) {
              const i32x4 rm = rows.a[pm + 16 * i], rn = rows.b[pn + 16 * j];
              s = 0.f;
              for (int e = 0; e < VE; ++e) {
                const i32x4 ka = ks_a[(c * VE + e) / SA::SPAN], kb = ks_b[(c * VE + e) / SB::SPAN];
                const bool in = ((uint32_t)(rm[1] + ka[1]) <= q.top_a[0]) & ((uint32_t)(rm[2] + ka[2]) <= q.top_a[1]) &
                                ((uint32_t)(rn[1] + kb[1]) <= q.top_b[0]) & ((uint32_t)(rn[2] + kb[2]) <= q.top_b[1]);
                if (in) s += element(av[i], e) * element(bv[j], e);
              }
            }
            total[i][j] += s;
          }
      }
    }
#pragma unroll
    for (int i = 0; i < RM; ++i)
#pragma unroll
      for (int j = 0; j < RN; ++j) {
        const int mi = pm + 16 * i, ni = pn + 16 * j;
        const i32x4 rm = rows.a[mi], rn = rows.b[ni];
        if (rm[1] == kFar || rn[1] == kFar || rows.ob_m[mi].x + rows.ob_n[ni].x > q.ob[0] || rows.ob_m[mi].y + rows.ob_n[ni].y > q.ob[1]) continue;
        put<S>(q, args.o, args.bias, o_base + rm[3] + rn[3], rn[3], (S)total[i][j]);
      }
  }
}

// The sums of NW wavefronts that share a tile's reduction out: fragment f is stored by wavefront f % NW, the others' sums reach it
// through LDS and are added in pairs (one after the other: 1.2 times the error at 5 x 88 x 1520 bf16).
template <int NW, int FM, int FN, typename Total>
__device__ __forceinline__ void meet(Total (&acc)[FM][FN], unsigned char* lds, int wave, int lane) {
  constexpr int NF = FM * FN;
  Total* part = (Total*)lds + lane;
#pragma unroll
  for (int f = 0; f < NF; ++f) {
    const int owner = f % NW;
    if (wave != owner) part[((wave < owner ? wave : wave - 1) * NF + f) * 64] = acc[f / FN][f % FN];
  }
  __syncthreads();
#pragma unroll
  for (int f = 0; f < NF; ++f)
    if (wave == f % NW) {
      Total sums[NW];
#pragma unroll
      for (int w = 0; w < NW - 1; ++w) sums[w] = part[(w * NF + f) * 64];
      sums[NW - 1] = acc[f / FN][f % FN];
#pragma unroll
      for (int h = NW / 2; h > 0; h /= 2)
#pragma unroll
        for (int w = 0; w < h; ++w) sums[w] += sums[w + h];
      acc[f / FN][f % FN] = sums[0];
    }
}

// Many tiles: BM x BN tile shared by four wavefronts, K tiles of BKB bytes per row staged for all of them; WM x WN wavefronts
// over the tile, or (32 x 32) all four over the tile and every fourth 64-byte step of a K tile, their sums meeting at the end.
// PRECISE (float types): the products of one 64-byte step are summed from zero and join a total in double precision.  For blocks
// whose literal kernel holds several sums per output (see wants_double): against it, fp32 totals had 1.1 to 1.5 times the error
// in 64 bits (K of 64 to 33000), totals in double 0.7 to 0.99 times.  They cost up to 15 % (250 x 250 x 1001 nt fp32 20.1 -> 23.3
// us, 1000 x 1000 x 3000 [k][m] bf16 50 -> 55), so other blocks, already more exact than before (1000^3 fp32: 5.6e-7 literal,
// 1.5e-7 here), keep fp32 totals.
template <typename T, int BM, int BN, int BKB, int WM, int WN, int MA, int MB, bool PRECISE>
__global__ __launch_bounds__(256, sizeof(T) == 1 ? 1 : BM == 128 && BN == 128 || PRECISE ? 2 : 3) void contract_kernel(
    const ContractParams p, const T* __restrict__ A, const T* __restrict__ B, void* __restrict__ O, const float* __restrict__ bias) {
  using Acc = typename Ct<T>::Acc;
  using S = typename Ct<T>::S;
  using SA = Stager<T, 256, BM, BKB, true, MA>;
  using SB = Stager<T, 256, BN, BKB, false, MB>;
  constexpr int WK = 4 / (WM * WN), STEPS = BKB / 64 / WK, FM = BM / WM / 16, FN = BN / WN / 16;
  constexpr int BUF = (BM + BN) * BKB;
  using Total = typename std::conditional<PRECISE, f64x4, Acc>::type;
  __shared__ __align__(16) unsigned char lds[2 * BUF];
  __shared__ i32x4 rows_a[BM], rows_b[BN];
  __shared__ int2 ob_m[BM], ob_n[BN];
  const TileRows rows = {rows_a, rows_b, ob_m, ob_n};
  constexpr uint32_t BK = BKB / sizeof(T);
  // k's share of the addresses and range tests, for both operands, one entry per vector of k: worked out for BATCH K tiles at a
  // time on as many lanes, at least one iteration before the first of their loads, in a ring of two batches (decoded at each load,
  // they are most of the kernel's time; a K tile's entries in each iteration a fifth of it)
  constexpr uint32_t ENTRIES = SA::ENTRIES + SB::ENTRIES;
  constexpr uint32_t BATCH = 8 * ENTRIES <= 256 ? 8 : 4 * ENTRIES <= 256 ? 4 : 2 * ENTRIES <= 256 ? 2 : 1;
  __shared__ i32x4 ks_a[2 * BATCH][SA::ENTRIES], ks_b[2 * BATCH][SB::ENTRIES];
  static_assert(2 * BUF >= BUF + (int)ENTRIES * 16, "room for the tables of sum_again");
  static_assert(sizeof lds + sizeof rows_a + sizeof rows_b + sizeof ob_m + sizeof ob_n + sizeof ks_a + sizeof ks_b == shared_lds_bytes(sizeof(T), BM, BN, BKB, MA, MB), "LDS");

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const uint32_t m0 = blockIdx.x / (uint32_t)p.tiles_n * BM, n0 = blockIdx.x % (uint32_t)p.tiles_n * BN;
  int a_base, b_base, o_base;
  batch_bases(p, &a_base, &b_base, &o_base);
  auto fill_ks = [&](uint32_t t) {       // K tiles t .. t + BATCH - 1, t a multiple of BATCH
#pragma unroll
    for (uint32_t x0 = 0; x0 < BATCH * ENTRIES; x0 += 256) {
      const uint32_t x = x0 + tid;
      if (x < BATCH * SA::ENTRIES) {
        const uint32_t tile = t + x / SA::ENTRIES, e = x % SA::ENTRIES;
        const KPart a = k_part(p, tile * BK + e * SA::SPAN, true);
        ks_a[tile % (2 * BATCH)][e] = (i32x4){a.off, a.t0, a.t1, a.run};
      } else if (x < BATCH * ENTRIES) {
        const uint32_t y = x - BATCH * SA::ENTRIES, tile = t + y / SB::ENTRIES, e = y % SB::ENTRIES;
        const KPart b = k_part(p, tile * BK + e * SB::SPAN, false);
        ks_b[tile % (2 * BATCH)][e] = (i32x4){b.off, b.t0, b.t1, b.run};
      }
    }
  };
  fill_ks(0);
  if (BATCH == 1) fill_ks(1);
  fill_rows<T, 256, BM, BN, MA, MB>(p, m0, n0, a_base, b_base, rows);
  __syncthreads();

  const __amdgpu_buffer_rsrc_t buf_a = __builtin_amdgcn_make_buffer_rsrc((void*)A, 0, (int)p.bytes_a, 0x00020000);
  const __amdgpu_buffer_rsrc_t buf_b = __builtin_amdgcn_make_buffer_rsrc((void*)B, 0, (int)p.bytes_b, 0x00020000);
  SA sa[2];      // K tiles t and t + 1 on their way
  SB sb[2];
  i32x4 row_a[SA::NR + 1], row_b[SB::NR + 1];
  SA::keep(rows_a, row_a, tid);
  SB::keep(rows_b, row_b, tid);
  const uint32_t n_kt = (p.K + BK - 1) / BK;
  const bool look = p.tested && std::is_same<S, float>::value;
  bool fin = true;

  static_assert(WM * WN * WK == 4 && (WK == 1 || WK == 4) && STEPS * WK * 64 == BKB, "four wavefronts, over the tile or over a K tile");
  const int wk = WK == 1 ? 0 : wave, wm = WK == 1 ? wave / WN : 0, wn = WK == 1 ? wave % WN : 0;
  // Where the wavefronts share a K tile, one total for the even ones and one for the odd ones: chains of totals half as long, as short
  // as with eight wavefronts that stage for themselves (4 x 32 x 32, 128 -> 192, 3x3, fp32: 1.05e-7 off with one, 9.4e-8 there).
  constexpr int TOTALS = WK > 1 && !PRECISE && sizeof(T) > 1 ? 2 : 1;
  Total totals[TOTALS][FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) totals[0][i][j] = totals[TOTALS - 1][i][j] = (Total){0, 0, 0, 0};
  Total(&acc)[FM][FN] = totals[0];

  // bf16 / fp32: partial sums over FLUSH K tiles start from zero and are added to the total, short chains of roundings
  // instead of one long one (not on the largest tile, whose registers hold one set of sums at two wavefronts per SIMD)
  // On the 64 x 64 tile a sum for the even steps and one for the odd ones, 16 (fp32) or 32 (bf16) products each (fp32, one sum: 1.2 times the error of
  // 32 x 32 tiles at 29 x 29, 64 -> 64, transposed 2x2, 0.8 times now, for 2 % of the time).  Where the fetch by elements holds the registers, one:
  // 6 x 49 x 49, 11 -> 72, 5x5 took 36 us instead of 27.  So do two bf16 operands along their rows: 1501 x 832 x 598 [k][m] 14.9 us instead of 13.0.
  constexpr int SUMS = sizeof(T) > 1 && STEPS > 1 && BM * BN <= 4096 && MA != 3 && MB != 3 && !(sizeof(T) == 2 && MA == 2 && MB == 2) ? 2 : 1;
  constexpr uint32_t FLUSH = BM * BN > 8192 ? 0xffffffffu : std::is_same<T, float>::value || TOTALS == 2 ? 1 : std::is_same<T, uint16_t>::value ? 4 : 0xffffffffu;
  Acc sum[SUMS][FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) sum[0][i][j] = sum[SUMS - 1][i][j] = (Acc){0, 0, 0, 0};
  auto flush = [&](Total (&to)[FM][FN]) {
    if constexpr (!PRECISE) {
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) {
          if constexpr (SUMS == 1) to[i][j] += sum[0][i][j];
          else to[i][j] += sum[0][i][j] + sum[1][i][j];
          sum[0][i][j] = sum[SUMS - 1][i][j] = (Acc){0, 0, 0, 0};
        }
    }
  };
  uint32_t at_a[FM], at_b[FN];
#pragma unroll
  for (int i = 0; i < FM; ++i) at_a[i] = SA::first(wm * (BM / WM) + i * 16, lane);
#pragma unroll
  for (int j = 0; j < FN; ++j) at_b[j] = SB::first(wn * (BN / WN) + j * 16, lane);

  // Two K tiles are in flight in registers (set t & 1 holds tile t): with one, few workgroups and long reductions spent an
  // iteration waiting for memory.  The loop's loads are unconditional (a tile past the last one loads zeros); the last two tiles
  // are peeled off without loads.
  sa[0].load(p, buf_a, rows_a, row_a, ks_a[0], 0, tid);
  sb[0].load(p, buf_b, rows_b, row_b, ks_b[0], 0, tid);
  if (n_kt > 1) {
    sa[1].load(p, buf_a, rows_a, row_a, ks_a[1], BK, tid);
    sb[1].load(p, buf_b, rows_b, row_b, ks_b[1], BK, tid);
  }
  if (n_kt > 2 && BATCH <= 2) {
    if (BATCH == 1) __syncthreads();      // over the entries of tile 0
    fill_ks(2);
  }
  fin &= sa[0].store(p, lds, 0, look, tid);
  fin &= sb[0].store(p, lds + BM * BKB, 0, look, tid);
  auto step = [&](uint32_t t, auto set, auto loads, auto stores) {
    constexpr int S0 = decltype(set)::value;
    __syncthreads();
    if constexpr (decltype(loads)::value) {
      const uint32_t slot = (t + 2) % (2 * BATCH);
      sa[S0].load(p, buf_a, rows_a, row_a, ks_a[slot], (t + 2) * BK, tid);
      sb[S0].load(p, buf_b, rows_b, row_b, ks_b[slot], (t + 2) * BK, tid);
      if ((t + 3) % BATCH == 0) fill_ks(t + 3);        // over the batch before tile t + 2's
    }
    const unsigned char *base_a = lds + S0 * BUF, *base_b = base_a + BM * BKB;
#pragma unroll
    for (int s = 0; s < STEPS; ++s) {
      u32x4 fa[FM], fb[FN];
#pragma unroll
      for (int i = 0; i < FM; ++i) fa[i] = SA::fragment(base_a, at_a[i], s * WK + wk);
#pragma unroll
      for (int j = 0; j < FN; ++j) fb[j] = SB::fragment(base_b, at_b[j], s * WK + wk);
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) {   // rows of the result: n
          if constexpr (PRECISE) acc[i][j] += __builtin_convertvector(Ct<T>::step(fb[j], fa[i]), f64x4);
          else sum[s % SUMS][i][j] = Ct<T>::mma(fb[j], fa[i], sum[s % SUMS][i][j]);
        }
    }
    if ((t + 1) % FLUSH == 0) flush(totals[TOTALS == 2 ? S0 : 0]);
    if constexpr (decltype(stores)::value) {
      unsigned char* next = lds + (1 - S0) * BUF;
      fin &= sa[1 - S0].store(p, next, (t + 1) * BK, look, tid);
      fin &= sb[1 - S0].store(p, next + BM * BKB, (t + 1) * BK, look, tid);
    }
  };
  constexpr std::integral_constant<int, 0> even;
  constexpr std::integral_constant<int, 1> odd;
  constexpr std::true_type yes;
  constexpr std::false_type no;
  uint32_t t = 0;
  for (; t + 2 < n_kt; t += 2) {
    step(t, even, yes, yes);
    step(t + 1, odd, yes, yes);
  }
  if (t + 1 < n_kt) {
    step(t, even, no, yes);
    step(t + 1, odd, no, no);
  } else {
    step(t, even, no, no);
  }
  flush(acc);
  if constexpr (TOTALS == 2) {
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j) acc[i][j] += totals[1][i][j];
  }

  constexpr bool again = sizeof(T) > 1;
  const KernelArgs& args = reread();
  if constexpr (again) {
    if (look && __syncthreads_or(!fin)) {
      sum_again<T, 256, BM, BN, BKB, MA, MB>(args, rows, o_base, lds);
      return;
    }
  }
  if constexpr (WK > 1) {
    static_assert((WK - 1) * FM * FN * 64 * (int)sizeof(Total) <= 2 * BUF, "partial sums fit the staging buffers");
    __syncthreads();
    meet<WK>(acc, lds, wave, lane);
  }
  store_fragments<T, FM, FN, WK>(again ? args.p : p, again ? args.o : O, again ? args.bias : bias, o_base, rows, wm * (BM / WM), wn * (BN / WN), wk, lane, acc);
}

// Order of a wavefront's memory accesses, for the compiler: no instruction.
__device__ __forceinline__ void wave_order() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Few tiles: the tile's NW wavefronts share its reduction out.  Each stages its own K tiles, every NW-th, through its own part of
// LDS and multiplies them into its own BM x BN sums, which meet at the end: no barrier inside the reduction, so that loads, LDS and
// matrix instructions of different wavefronts overlap.  (Four wavefronts that stage K tiles for each other were bound by that
// chain, barrier to barrier: without its loads or its matrix instructions their loop took the same time.)  A wavefront's LDS
// instructions execute in order, so a K tile may be written over the one before without a wait; wave_order() keeps the compiler,
// which looks at one lane at a time, from moving a lane's reads and writes across each other.
// PLAIN: a product with one index per side and no tests, whose addresses need no tables.
// Measured, us (before: four wavefronts per tile): 56 x 64 x 4080 nt bf16 9.3 -> 5.4 (16 x 16), 400 x 500 x 3000 nt bf16 11.5 -> 8.3
// and [k][m] 14.2 -> 10.9 (32 x 32), 1000 x 1000 x 3000 [k][m] bf16 48.5 -> 20, 1000^3 fp32 39 -> 25 (64 x 64).
template <typename T, int NW, int BM, int BN, int BKB, int MA, int MB, bool PRECISE, bool PLAIN>
__global__ __launch_bounds__(NW * 64, NW / 4) void contract_waves_kernel(const ContractParams p, const T* __restrict__ A, const T* __restrict__ B,
                                                                        void* __restrict__ O, const float* __restrict__ bias) {
  using Acc = typename Ct<T>::Acc;
  using S = typename Ct<T>::S;
  using SA = Stager<T, 64, BM, BKB, true, MA>;
  using SB = Stager<T, 64, BN, BKB, false, MB>;
  constexpr int NT = NW * 64, STEPS = BKB / 64, FM = BM / 16, FN = BN / 16, NF = FM * FN, STAGE = (BM + BN) * BKB;
  constexpr uint32_t BK = BKB / sizeof(T);
  using Total = typename std::conditional<PRECISE, f64x4, Acc>::type;
  constexpr int PART = (NW - 1) * NF * 64 * (int)sizeof(Total);
  // tables of a wavefront's next TABLES K tiles, one entry per vector of k
  constexpr int ENTRIES = SA::ENTRIES + SB::ENTRIES, TABLES = 4 * ENTRIES <= 64 ? 4 : 2 * ENTRIES <= 64 ? 2 : 1;
  constexpr int BKB_AGAIN = 16 * NT / BM, AGAIN = PLAIN || sizeof(T) == 1 ? 0 : (BM + BN) * BKB_AGAIN + 2 * BKB_AGAIN / (int)sizeof(T) * 16;
  constexpr int NEED = NW * STAGE > PART ? NW * STAGE : PART, LDS = NEED > AGAIN ? NEED : AGAIN;
  __shared__ __align__(16) unsigned char lds[LDS];
  __shared__ i32x4 rows_a[BM], rows_b[BN];
  __shared__ int2 ob_m[BM], ob_n[BN];
  __shared__ i32x4 tables[PLAIN ? 1 : NW][PLAIN ? 1 : TABLES * ENTRIES];
  static_assert(LDS + sizeof rows_a + sizeof rows_b + sizeof ob_m + sizeof ob_n + (PLAIN ? 0 : sizeof tables) == waves_lds_bytes(sizeof(T), NW, BM, BN, BKB, MA, MB, PRECISE, PLAIN), "LDS");
  const TileRows rows = {rows_a, rows_b, ob_m, ob_n};
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t m0 = blockIdx.x / (uint32_t)p.tiles_n * BM, n0 = blockIdx.x % (uint32_t)p.tiles_n * BN;
  int a_base, b_base, o_base;
  batch_bases(p, &a_base, &b_base, &o_base);
  SA sa;
  SB sb;
  unsigned char *const mine_a = lds + wave * STAGE, *const mine_b = mine_a + BM * BKB;
  const uint32_t n_kt = (p.K + BK - 1) / BK;
  const bool look = !PLAIN && p.tested && std::is_same<S, float>::value;
  bool fin = true;
  uint32_t off_a[PLAIN ? SA::NR : 1], off_b[PLAIN ? SB::NR : 1], step_a = 0, step_b = 0;
  i32x4 row_a[PLAIN ? 1 : SA::NR + 1], row_b[PLAIN ? 1 : SB::NR + 1];
  auto load = [&](uint32_t t) {
    // behind the last K tile nothing is fetched: the buffers are empty (a branch around the loads lets the compiler sink them)
    const bool live = t < n_kt;
    const __amdgpu_buffer_rsrc_t buf_a = __builtin_amdgcn_make_buffer_rsrc((void*)A, 0, live ? (int)p.bytes_a : 0, 0x00020000);
    const __amdgpu_buffer_rsrc_t buf_b = __builtin_amdgcn_make_buffer_rsrc((void*)B, 0, live ? (int)p.bytes_b : 0, 0x00020000);
    if constexpr (PLAIN) {
      sa.load_plain(p, buf_a, off_a, step_a, t * BK, lane);
      sb.load_plain(p, buf_b, off_b, step_b, t * BK, lane);
    } else {
      const uint32_t it = t / NW % TABLES;
      if (it == 0 && live) {
#pragma unroll
        for (int x0 = 0; x0 < TABLES * ENTRIES; x0 += 64) {
          const int x = x0 + lane, y = x % ENTRIES;
          const bool a = y < SA::ENTRIES;
          const KPart k = k_part(p, (t + x / ENTRIES * NW) * BK + (a ? y * SA::SPAN : (y - SA::ENTRIES) * SB::SPAN), a);
          if (x < TABLES * ENTRIES) tables[wave][x] = (i32x4){k.off, k.t0, k.t1, k.run};
        }
        wave_order();
      }
      const i32x4* ks = &tables[wave][it * ENTRIES];
      sa.load(p, buf_a, rows_a, row_a, ks, t * BK, lane);
      sb.load(p, buf_b, rows_b, row_b, ks + SA::ENTRIES, t * BK, lane);
    }
  };
  if constexpr (PLAIN) {
    auto offset = [](uint32_t at, uint32_t end, int stride, int base, int mode) {
      constexpr uint32_t V = Ct<T>::V;
      if (mode == 2 && at < end && at + V > end) at = end - V;
      return at < end ? (uint32_t)(base + (int)at * stride) * (uint32_t)sizeof(T) : kOutside;
    };
#pragma unroll
    for (int i = 0; i < SA::NR; ++i) off_a[i] = offset(m0 + (MA == 1 ? lane / SA::CH + i * SA::STEP1 : lane % SA::G * SA::V), p.M, p.m_in[0], a_base, MA);
#pragma unroll
    for (int i = 0; i < SB::NR; ++i) off_b[i] = offset(n0 + (MB == 1 ? lane / SB::CH + i * SB::STEP1 : lane % SB::G * SB::V), p.N, p.n_in[0], b_base, MB);
    step_a = (uint32_t)p.k_a[0] * (uint32_t)sizeof(T);
    step_b = (uint32_t)p.k_b[0] * (uint32_t)sizeof(T);
    load(wave);
  }
  fill_rows<T, NT, BM, BN, MA, MB>(p, m0, n0, a_base, b_base, rows);      // PLAIN: read behind the barrier after the reduction
  if constexpr (!PLAIN) {
    __syncthreads();
    SA::keep(rows_a, row_a, lane);
    SB::keep(rows_b, row_b, lane);
    load(wave);
  }

  Total acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) acc[i][j] = (Total){0, 0, 0, 0};
  uint32_t at_a[FM], at_b[FN];
#pragma unroll
  for (int i = 0; i < FM; ++i) at_a[i] = SA::first(i * 16, lane);
#pragma unroll
  for (int j = 0; j < FN; ++j) at_b[j] = SB::first(j * 16, lane);
  for (uint32_t t = wave; t < n_kt; t += NW) {
    wave_order();      // the fragments of the K tile before are read
    fin &= sa.store(p, mine_a, t * BK, look, lane);
    fin &= sb.store(p, mine_b, t * BK, look, lane);
    load(t + NW);
    wave_order();
    __builtin_amdgcn_sched_barrier(0);
    u32x4 fa[STEPS][FM], fb[STEPS][FN];
#pragma unroll
    for (int s = 0; s < STEPS; ++s) {
#pragma unroll
      for (int i = 0; i < FM; ++i) fa[s][i] = SA::fragment(mine_a, at_a[i], s);
#pragma unroll
      for (int j = 0; j < FN; ++j) fb[s][j] = SB::fragment(mine_b, at_b[j], s);
    }
    // float types: sums that start from zero join the total, of 16 products (fp32) or of 32, the K tile's one to four in pairs (bf16)
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j) {   // rows of the result: n
        if constexpr (std::is_same<T, int8_t>::value) {
#pragma unroll
          for (int s = 0; s < STEPS; ++s) acc[i][j] = Ct<T>::mma(fb[s][j], fa[s][i], acc[i][j]);
        } else if constexpr (PRECISE) {
#pragma unroll
          for (int s = 0; s < STEPS; ++s) acc[i][j] += __builtin_convertvector(Ct<T>::step(fb[s][j], fa[s][i]), f64x4);
        } else if constexpr (std::is_same<T, float>::value) {
#pragma unroll
          for (int s = 0; s < STEPS; ++s) acc[i][j] += Ct<T>::mma(fb[s][j], fa[s][i], (Acc){0, 0, 0, 0});
        } else {
          Acc sum[STEPS];
#pragma unroll
          for (int s = 0; s < STEPS; ++s) sum[s] = Ct<T>::mma(fb[s][j], fa[s][i], (Acc){0, 0, 0, 0});
#pragma unroll
          for (int h = STEPS / 2; h > 0; h /= 2)
#pragma unroll
            for (int s = 0; s < h; ++s) sum[s] += sum[s + h];
          acc[i][j] += sum[0];
        }
      }
  }

  const KernelArgs& args = reread();
  if (__syncthreads_or(look && !fin)) {      // also: the staging buffers are free from here on
    if constexpr (!PLAIN && sizeof(T) > 1) sum_again<T, NT, BM, BN, BKB_AGAIN, MA, MB>(args, rows, o_base, lds);
    return;
  }
  meet<NW>(acc, lds, wave, lane);
  store_fragments<T, FM, FN, NW>(args.p, args.o, args.bias, o_base, rows, 0, 0, wave, lane, acc);
}

}  // namespace

// one translation unit per element type compiles the kernels (CONTRACT_T); the planner is compiled with the last of them
hipError_t launch_contract_f32(const ContractLaunch&, const ContractParams&, const void*, const void*, void*, const float*, hipStream_t);
hipError_t launch_contract_bf16(const ContractLaunch&, const ContractParams&, const void*, const void*, void*, const float*, hipStream_t);
hipError_t launch_contract_i8(const ContractLaunch&, const ContractParams&, const void*, const void*, void*, const float*, hipStream_t);

namespace {

template <typename T, int MA, int MB>
hipError_t launch_modes(const ContractLaunch& l, const ContractParams& p, const void* a, const void* b, void* o, const float* bias, hipStream_t s) {
  const dim3 g((unsigned)l.grid, (unsigned)l.batch);
  auto go = [&](auto kernel, int lanes) {
    hipLaunchKernelGGL(kernel, g, dim3((unsigned)lanes), 0, s, p, (const T*)a, (const T*)b, o, bias);
    return hipGetLastError();
  };
  constexpr bool real = sizeof(T) > 1, vectors = (MA == 1 || MA == 2) && (MB == 1 || MB == 2);
  switch (l.tile) {
    case 0: return go(contract_kernel<T, 128, 128, 64, 2, 2, MA, MB, false>, 256);
    case 1:
      if constexpr (real) if (l.precise) return go(contract_kernel<T, 64, 64, 128, 2, 2, MA, MB, true>, 256);
      return go(contract_kernel<T, 64, 64, 128, 2, 2, MA, MB, false>, 256);
    case 3:
      if constexpr (MB == 2 && sizeof(T) < 4) return hipErrorInvalidValue;   // the planner takes tile 1
      else return go(contract_kernel<T, 128, 64, 64, 2, 2, MA, MB, false>, 256);
    case 4:
      if constexpr (vectors) {
        if (l.plain) {
          if constexpr (real) if (l.precise) return go(contract_waves_kernel<T, 16, 16, 16, 256, MA, MB, true, true>, 1024);
          return go(contract_waves_kernel<T, 16, 16, 16, 256, MA, MB, false, true>, 1024);
        }
      }
      if constexpr (real) if (l.precise) return go(contract_waves_kernel<T, 16, 16, 16, 128, MA, MB, true, false>, 1024);
      return go(contract_waves_kernel<T, 16, 16, 16, 128, MA, MB, false, false>, 1024);
    case 5:
      if constexpr (vectors) return go(contract_waves_kernel<T, 8, 64, 64, 64, MA, MB, false, true>, 512);
      else return hipErrorInvalidValue;
    case 6:
      if constexpr (real) if (l.precise) return go(contract_kernel<T, 32, 32, 256, 1, 1, MA, MB, true>, 256);
      return go(contract_kernel<T, 32, 32, 256, 1, 1, MA, MB, false>, 256);
    default:
      if constexpr (vectors) {
        if (l.plain) {
          if constexpr (real) if (l.precise) return go(contract_waves_kernel<T, 8, 32, 32, 128, MA, MB, true, true>, 512);
          return go(contract_waves_kernel<T, 8, 32, 32, 128, MA, MB, false, true>, 512);
        }
      }
      if constexpr (real) if (l.precise) return go(contract_waves_kernel<T, 8, 32, 32, 128, MA, MB, true, false>, 512);
      return go(contract_waves_kernel<T, 8, 32, 32, 128, MA, MB, false, false>, 512);
  }
}

template <typename T>
hipError_t launch_t(const ContractLaunch& l, const ContractParams& p, const void* a, const void* b, void* o, const float* bias, hipStream_t s) {
  switch (p.mode_a * 4 + p.mode_b) {
    case 0: return launch_modes<T, 0, 0>(l, p, a, b, o, bias, s);
    case 1: return launch_modes<T, 0, 1>(l, p, a, b, o, bias, s);
    case 2: return launch_modes<T, 0, 2>(l, p, a, b, o, bias, s);
    case 3: return launch_modes<T, 0, 3>(l, p, a, b, o, bias, s);
    case 4: return launch_modes<T, 1, 0>(l, p, a, b, o, bias, s);
    case 5: return launch_modes<T, 1, 1>(l, p, a, b, o, bias, s);
    case 6: return launch_modes<T, 1, 2>(l, p, a, b, o, bias, s);
    case 8: return launch_modes<T, 2, 0>(l, p, a, b, o, bias, s);
    case 9: return launch_modes<T, 2, 1>(l, p, a, b, o, bias, s);
    case 10: return launch_modes<T, 2, 2>(l, p, a, b, o, bias, s);
    case 11: return launch_modes<T, 2, 3>(l, p, a, b, o, bias, s);
    case 12: return launch_modes<T, 3, 0>(l, p, a, b, o, bias, s);
    case 14: return launch_modes<T, 3, 2>(l, p, a, b, o, bias, s);
    case 15: return launch_modes<T, 3, 3>(l, p, a, b, o, bias, s);
    default: return hipErrorInvalidValue;     // modes 1 and 3 exclude each other: both follow from the innermost reduction index's range
  }
}

}  // namespace


#if CONTRACT_T == 4
hipError_t launch_contract_f32(const ContractLaunch& l, const ContractParams& p, const void* a, const void* b, void* o, const float* bias, hipStream_t s) {
  return launch_t<float>(l, p, a, b, o, bias, s);
}
#elif CONTRACT_T == 2
hipError_t launch_contract_bf16(const ContractLaunch& l, const ContractParams& p, const void* a, const void* b, void* o, const float* bias, hipStream_t s) {
  return launch_t<uint16_t>(l, p, a, b, o, bias, s);
}
#else
hipError_t launch_contract_i8(const ContractLaunch& l, const ContractParams& p, const void* a, const void* b, void* o, const float* bias, hipStream_t s) {
  return launch_t<int8_t>(l, p, a, b, o, bias, s);
}

namespace {

typedef __int128 i128;

// 0, 1, 3, 6: staged for four wavefronts; 2, 4, 5: the wavefronts share the reduction out and stage for themselves
struct Tile {
  int bm, bn, bkb, lanes;
};
constexpr Tile kTiles[] = {{128, 128, 64, 256}, {64, 64, 128, 256}, {32, 32, 128, 512}, {128, 64, 64, 256}, {16, 16, 256, 1024}, {64, 64, 64, 512}, {32, 32, 256, 256}};

struct Ix {                      // one index: range, address coefficients, constraint coefficients, output-bound coefficients
  int64_t range = 1, a = 0, b = 0, o = 0;
  std::vector<int64_t> con;
  int64_t ob[kCtTests] = {0, 0};
};

bool fill_side(const std::vector<Ix>& v, CtIndex* c) {
  if ((int)v.size() > kCtIdx) return false;
  c->n = (int)v.size();
  for (int j = 0; j < kCtIdx; ++j) {
    c->range[j] = 0;
    c->mul[j] = 0;
    c->shift[j] = 0;
  }
  for (size_t j = 0; j < v.size(); ++j) {
    const uint64_t d = (uint64_t)v[j].range;
    if (d < 2 || d > 0x3fffffff) return false;
    int s = 0;
    while (((uint64_t)1 << s) < d) ++s;
    // floor(v * mul / 2^(31+s)) = v / d for v < 2^31: mul exceeds 2^(31+s)/d by at most 1, and 2^s >= d
    c->range[j] = (uint32_t)d;
    c->mul[j] = (uint32_t)((((uint64_t)1 << (31 + s)) / d) + 1);
    c->shift[j] = s - 1;
  }
  return true;
}

}  // namespace

// Whether totals in double precision are needed for an error no larger than the literal kernel's.  It is not larger anyway
// where that kernel sums an output's points in one chain (here chains of at most 32 fp32 products, 17 on the 32 x 32 tiles, and
// fp32 totals), also where such chains meet in atomic additions, if they are as long as this kernel's (transposed 3x3, 32
// channels, fp32: 1.08e-7 both; 8 channels: 6.6e-8 and 1.0e-7).  bf16 sums run through chains of up to 256 products.
// few: fewer than 96 tiles of 64 x 64.  There fp32 reductions of 9 to 16, one step of 16 products, run as the two chains of eight of
// the form with totals in double on every tile, as on the 32 x 32 ones: half the roundings in a row for no time (a launch is most of it).
static bool wants_double(int dtype, int tile, bool few, const LiteralSums& lit) {
  if (dtype == STRIPE_I8) return false;
  if (lit.lanes == 64) return true;
  if (dtype == STRIPE_BF16) return lit.atomic;
  if (lit.atomic) return tile == 0 || tile == 3 || lit.chain < (tile == 1 ? 32 : 17);
  return (tile == 2 || tile == 6 || few) && lit.chain > 8 && lit.chain < 17;
}

// Time of a block on tile t: a launch, per round of workgroups a fixed part and one for each K tile in a row -- all of them where
// four wavefronts share a tile, every 8th or 16th where they share the reduction out -- and a part for what all workgroups' K tiles
// take from memory together.  us, fitted to 344 products, convolutions and transposed convolutions of 1 to 4096 rows, 7 to 12544
// points of reduction, each on every tile: the tile chosen by it takes 1.02 times as long as the best one (geometric mean).
// single_rows: rows of a tile that are fetched element by element, 0.05 us for the loads of 64 elements (2 x 49 x 49, 64 channels,
// transposed 3 x 3 to 15, bf16: 12.8 on 64 x 64, 17.7 on 32 x 32 where each wavefront stages for itself, 11.0 where four share a K tile).
// The last, tile 6 (no products: plain ones are never the fastest there): chosen to lose least on 330 convolutions and transposed
// ones, half of them on tiles 1, 2, 4 and 6 (0.5 % over the fastest, 5 % with tiles 0 to 4 alone: 3x3, 64 -> 115 at 2 x 55 x 55, fp32 25.7 -> 19.6).
// Its operands fetched along their rows cost it more than the others.
static double tile_us(int dtype, int t, bool plain, int single_rows, int along_rows, double tiles, double k_bytes) {
  struct Cost {
    double fixed, k_tile, all;      // per round, per K tile and round, per K tile of 256 workgroups
    double at_once;                 // workgroups of a round
  };
  static const Cost other[3][7] = {      // fp32, bf16, int8
      {{5.3, 1.51, 0.92, 384}, {1.9, 1.20, 0.15, 384}, {2.2, 2.01, 0.76, 256}, {3.3, 1.01, 0.57, 384}, {1.6, 1.42, 1.59, 384}, {}, {1.7, 1.07, 0.00, 384}},
      {{5.6, 0.93, 0.00, 256}, {2.8, 0.95, 0.03, 512}, {3.7, 1.48, 0.07, 256}, {4.1, 0.81, 0.03, 384}, {2.4, 1.20, 0.52, 256}, {}, {3.7, 0.59, 0.17, 512}},
      {{4.2, 0.56, 0.57, 512}, {1.9, 0.38, 0.42, 768}, {3.2, 0.41, 0.56, 256}, {2.4, 0.43, 0.31, 384}, {3.2, 0.01, 1.34, 384}, {}, {2.6, 0.57, 0.13, 512}}};
  static const Cost plain_product[3][6] = {
      {{2.9, 1.32, 0.55, 256}, {1.4, 0.94, 0.25, 384}, {1.2, 1.37, 0.35, 256}, {2.2, 0.82, 0.49, 512}, {0.1, 2.04, 1.08, 256}, {1.9, 2.38, 0.88, 256}},
      {{5.1, 0.50, 0.19, 256}, {2.2, 0.55, 0.16, 512}, {1.7, 0.57, 0.64, 384}, {3.0, 0.49, 0.11, 256}, {0.7, 1.46, 1.18, 256}, {3.1, 0.78, 0.96, 256}},
      {{2.9, 0.71, 0.00, 256}, {1.6, 0.67, 0.06, 768}, {0.1, 1.45, 1.41, 768}, {1.7, 0.34, 0.17, 512}, {1.1, 0.80, 1.19, 256}, {2.0, 0.90, 1.04, 256}}};
  const int d = dtype == STRIPE_F32 ? 0 : dtype == STRIPE_BF16 ? 1 : 2;
  Cost c = plain ? plain_product[d][t] : other[d][t];
  double single_us = 0.05;
  if (t == 6) {
    static const double along_rows_us[3] = {1.55, 0.4, 0.3}, singles_us[3] = {0.045, 0.03, 0.025};
    c.fixed += along_rows * along_rows_us[d];
    single_us = singles_us[d];
  }
  double k_tiles = std::ceil(k_bytes / (t == 4 && !plain ? 128 : kTiles[t].bkb));
  if (t == 2 || t == 4 || t == 5) k_tiles = std::ceil(k_tiles * 64 / kTiles[t].lanes);
  // int8 products of one K tile on many 64 x 64 tiles, an operand along its rows: start and end of every workgroup (4096 x 4096 x 64 nn 25.7 us
  // there, 16.8 on 128 x 128; 1500 x 2500 x 100 10.9 and 9.2; below 512 tiles and with two K tiles 64 x 64 is the faster one).
  const double one_k_tile = plain && d == 2 && t == 1 && along_rows && k_tiles == 1 && tiles > 512 ? 0.75 * (tiles - 512) / 256 : 0.0;
  const double singles = single_rows * k_bytes / (dtype == STRIPE_F32 ? 4 : dtype == STRIPE_BF16 ? 2 : 1) / 64;
  return 4.0 + std::max(1.0, tiles / c.at_once) * (c.fixed + c.k_tile * k_tiles) + tiles / 256 * (c.all * k_tiles + single_us * singles) + one_k_tile;
}

// Blocks that stay on their literal kernel; here_us: what they take on this file's kernels.  Measured on 1,060 blocks of 65536 to
// 3e9 points in fp32, bf16 and int8: the faster kernel is chosen, or one within 6 %, for all but 20 (the worst 30 %).
static bool literal_is_faster(int dtype, const ContractParams& p, const LiteralSums& lit, bool simple, bool fused, __int128 points, double here_us) {
  if (points < (simple && !fused ? 1024 : 65536)) return true;        // there a launch is all the time there is
  if (fused) return false;               // a launch and a temporary more: 33 x 33 x 1001 bf16 with bias and relu 12.0 us against 13.3
  if (lit.atomic && points >= 65536) return false;          // two launches and atomic additions: 118 us against 10 for a transposed convolution
  if (lit.tiled) {
    // Short reductions into few columns: 100000 x 3 x 5 fp32 7 us against 12 (20000 x 200 x 8 18 against 14).  Large images with few
    // output channels fill a fraction of a tile's columns: 3x3, 3 -> 8 channels at 27 x 184 x 184 fp32 68 us against 164, 3 -> 4
    // bf16 40 against 71.  Products with a few columns whose first operand is contiguous along the rows: 300000 x 5 x 30 fp32 23 us against 31.
    const uint32_t few = std::min(p.M, p.N);
    if (lit.chain <= 8 && few <= 40) return true;
    if (p.tested && lit.chain <= 32 && few <= (dtype == STRIPE_F32 ? 24u : 4u) && points >= ((__int128)1 << 26)) return true;
    return dtype == STRIPE_F32 && p.mode_a == 2 && p.N <= 8 && lit.chain <= 64 && points >= ((__int128)1 << 23);
  }
  // A wavefront per output: 64 points a step, 0.36 us (0.6 with several reduction indexes to divide up), or what all outputs' steps
  // take together (250 x 250 x 1001 122 us, here 10).  Few steps of few outputs, whose wavefronts each have a CU's loads to
  // themselves, stay there, unless one 32 x 32 tile walking the whole reduction would be as fast.
  if (lit.lanes == 64) {
    const double many = lit.n_red > 1 ? 2.0 : 1.0;
    const double literal = 5.0 + 4e-4 * (double)lit.outputs + (double)((lit.chain + 63) / 64) * std::max(lit.n_red > 1 ? 0.6 : 0.36, 1.2e-4 * many * (double)lit.outputs);
    const double k_bytes = (double)p.K * (dtype == STRIPE_F32 ? 4 : dtype == STRIPE_BF16 ? 2 : 1);
    const double one_tile = (p.tested && dtype != STRIPE_I8 ? 7.5 : 6.0) + std::ceil(k_bytes / 256) * (dtype == STRIPE_F32 ? 0.78 : dtype == STRIPE_BF16 ? 0.62 : 0.8);
    if (literal < one_tile && ((literal < 12 && lit.outputs <= 4096) || lit.outputs <= 512)) return true;
    return literal < here_us;
  }
  // A lane per output: 0.21 us a point (1 x 349 x 3328 int8 784 us).  Reductions of a K tile or two take 1.5 us less here than their
  // estimate says (transposed 2x2, 12 -> 11 at 4 x 36 x 36, bf16: 8.6 us there).
  if (lit.outputs >= 100000) here_us -= 1.5;
  return (5.0 + 0.21 * (double)lit.chain * std::max(1.0, (double)lit.outputs / 5e5)) * (lit.atomic ? 2 : 1) < here_us;
}

bool contract_select(const FlatBlock& fb, const LiteralSums& lit, bool fused, ContractLaunch* l, stripe_block_info_t* info) {
  l->use = false;
  if (!tune_int("contract", 1)) return false;
  if (fb.empty || fb.n_refs != 3 || fb.intrinsic != STRIPE_INTR_MUL || fb.agg != STRIPE_AGG_ADD) return false;
  const int dt = fb.ref[0].dtype;
  if (fb.ref[1].dtype != dt || (dt != STRIPE_F32 && dt != STRIPE_BF16 && dt != STRIPE_I8)) return false;
  const int esize = dt == STRIPE_F32 ? 4 : dt == STRIPE_BF16 ? 2 : 1;

  // the block's indexes and constraints
  std::vector<Ix> ix;
  std::vector<int64_t> con_k;
  size_t n_con = fb.cons.size();
  for (const Affine& q : fb.cons) con_k.push_back(q.k);
  for (int j = 0; j < fb.n_idx; ++j) {
    Ix x;
    x.range = fb.range[j];
    x.a = fb.ref[0].addr.c[j];
    x.b = fb.ref[1].addr.c[j];
    x.o = fb.ref[2].addr.c[j];
    for (const Affine& q : fb.cons) x.con.push_back(q.c[j]);
    ix.push_back(x);
  }
  // all values the kernel forms stay far inside 32 bits (bytes for the operands)
  auto small = [&](int64_t k, auto coef, i128 lim) {
    i128 m = k < 0 ? -(i128)k : (i128)k;
    for (const Ix& x : ix) {
      const int64_t c = coef(x);
      m += (c < 0 ? -(i128)c : (i128)c) * (x.range + 1);
    }
    return m < lim;
  };

  // Every output element one owner: pairs p (of A), i (of B) with o_p = s * o_i and overlapping spans are rewritten as in
  // the file's head comment.
  const size_t first_new = n_con;      // constraints from here on come from the rewriting
  int n_ob = 0;
  int64_t ob[kCtTests] = {0, 0};
  std::vector<std::pair<int64_t, int64_t>> combined;    // (output stride, extent) of the rewritten pairs
  std::vector<char> in_pair(ix.size(), 0);
  for (size_t pi = 0; pi < in_pair.size(); ++pi)
    for (size_t ii = 0; ii < in_pair.size(); ++ii) {
      if (pi == ii || in_pair[pi] || in_pair[ii]) continue;
      const Ix p = ix[pi], i = ix[ii];
      if (!p.a || p.b || !i.b || i.a || p.o <= 0 || i.o <= 0 || p.o % i.o) continue;
      const int64_t s = p.o / i.o;
      if (i.range <= s) continue;                        // no overlap
      bool free = n_ob < kCtTests;
      for (size_t q = 0; q < n_con && free; ++q) free = !p.con[q] && !i.con[q];
      if (!free) return false;
      const int64_t i1n = (i.range + s - 1) / s;
      Ix pp = p, i1, i0 = i;
      pp.range = p.range + i1n - 1;
      i1.range = i1n; i1.a = -p.a; i1.b = s * i.b; i1.o = 0;
      i0.range = s;
      pp.ob[n_ob] = s;
      i0.ob[n_ob] = 1;
      ob[n_ob] = s * (p.range - 1) + i.range - 1;
      combined.push_back({i.o, ob[n_ob] + 1});
      ++n_ob;
      i1.con.assign(con_k.size(), 0);
      ix[pi] = pp;
      ix[ii] = i0;
      ix.push_back(i1);
      in_pair[pi] = in_pair[ii] = 1;
      auto add_con = [&](int64_t k, int64_t cp, int64_t c1, int64_t c0) {
        con_k.push_back(k);
        for (Ix& x : ix) x.con.push_back(0);
        ix[pi].con.back() = cp;
        ix[ii].con.back() = c0;
        ix.back().con.back() = c1;
      };
      add_con(0, 1, -1, 0);                              // p' - i1 >= 0
      add_con(p.range - 1, -1, 1, 0);                    // p' - i1 <= P - 1
      if (i.range % s) add_con(i.range - 1, 0, -s, -1);  // s*i1 + i0 <= R - 1
    }
  n_con = con_k.size();
  // one owner per element now?  strides by magnitude, each beyond the span of the smaller ones
  {
    std::vector<std::pair<int64_t, int64_t>> t = combined;
    for (const Ix& x : ix)
      if (x.o && !x.ob[0] && !x.ob[1]) t.push_back({x.o < 0 ? -x.o : x.o, x.range});
    std::sort(t.begin(), t.end());
    i128 span = 0;
    for (const auto& e : t) {
      if ((i128)e.first <= span) return false;
      span += (i128)e.first * (e.second - 1);
    }
    if (n_ob && fb.out_bf16) return false;
  }
  // ranges of 1 (a stride-1 transposed convolution's i0) carry nothing
  for (size_t j = 0; j < ix.size();) {
    if (ix[j].range == 1) ix.erase(ix.begin() + j);
    else ++j;
  }
  const i128 lim = 0x3fffffff;
  if (!small(fb.ref[0].addr.k, [](const Ix& x) { return x.a; }, lim / esize) || !small(fb.ref[1].addr.k, [](const Ix& x) { return x.b; }, lim / esize) ||
      !small(fb.ref[2].addr.k, [](const Ix& x) { return x.o; }, lim))
    return false;
  for (size_t q = 0; q < n_con; ++q)
    if (!small(con_k[q], [q](const Ix& x) { return x.con[q]; }, lim / 4)) return false;

  // Every owner has a point (constraints that share no index are independent): else an element would have to stay
  // unwritten.  The rewritten pairs' own constraints are covered by the output bounds.
  {
    std::vector<char> done(first_new, 0);
    for (size_t q0 = 0; q0 < first_new; ++q0) {
      if (done[q0]) continue;
      std::vector<size_t> group{q0};
      done[q0] = 1;
      std::vector<char> uses(ix.size(), 0);
      for (bool grown = true; grown;) {
        grown = false;
        for (size_t g : group)
          for (size_t j = 0; j < ix.size(); ++j)
            if (ix[j].con[g]) uses[j] = 1;
        for (size_t q = 0; q < first_new; ++q) {
          bool shares = false;
          for (size_t j = 0; j < ix.size(); ++j) shares = shares || (uses[j] && ix[j].con[q]);
          if (!done[q] && shares) {
            done[q] = 1;
            group.push_back(q);
            grown = true;
          }
        }
      }
      std::vector<size_t> outs, reds;
      i128 pts = 1;
      for (size_t j = 0; j < ix.size(); ++j)
        if (uses[j]) {
          pts *= ix[j].range;
          (ix[j].o ? outs : reds).push_back(j);
        }
      if (pts > ((i128)1 << 20)) return false;
      i128 n_outs = 1, n_reds = 1;
      for (size_t j : outs) n_outs *= ix[j].range;
      for (size_t j : reds) n_reds *= ix[j].range;
      for (int64_t o = 0; o < (int64_t)n_outs; ++o) {
        bool any = false;
        for (int64_t r = 0; r < (int64_t)n_reds && !any; ++r) {
          bool ok = true;
          for (size_t g : group) {
            int64_t v = con_k[g], to = o, tr = r;
            for (size_t j : outs) { v += ix[j].con[g] * (to % ix[j].range); to /= ix[j].range; }
            for (size_t j : reds) { v += ix[j].con[g] * (tr % ix[j].range); tr /= ix[j].range; }
            ok = ok && v >= 0;
          }
          any = ok;
        }
        if (!any) return false;
      }
    }
  }

  // the second operand plays A where it owns the output's unit stride (columns are stored four at a time)
  l->swap = false;
  for (const Ix& x : ix)
    if (x.o == 1 && x.a && !x.b) l->swap = true;
  if (l->swap)
    for (Ix& x : ix) std::swap(x.a, x.b);
  const int64_t base_a = fb.ref[l->swap ? 1 : 0].addr.k, base_b = fb.ref[l->swap ? 0 : 1].addr.k;

  std::vector<Ix> m, n, k, bat;
  for (const Ix& x : ix) {
    if (!x.o) k.push_back(x);
    else if (x.a && x.b) bat.push_back(x);
    else if (x.b) n.push_back(x);
    else m.push_back(x);
  }
  if (n.empty() || k.empty() || bat.size() > 2) return false;      // no row index: one row (a matrix-vector product)
  auto mag = [](int64_t v) { return v < 0 ? -v : v; };
  // rows: the index A holds contiguously first (vector fetches), else by output stride
  std::sort(m.begin(), m.end(), [&](const Ix& x, const Ix& y) { return (x.a == 1) != (y.a == 1) ? x.a == 1 : mag(x.o) < mag(y.o); });
  std::sort(n.begin(), n.end(), [&](const Ix& x, const Ix& y) {
    const int rx = x.o == 1 ? 0 : x.b == 1 ? 1 : 2, ry = y.o == 1 ? 0 : y.b == 1 ? 1 : 2;
    return rx != ry ? rx < ry : mag(x.o) < mag(y.o);
  });
  // reduction: the index that is contiguous in most operands first
  std::sort(k.begin(), k.end(), [&](const Ix& x, const Ix& y) {
    const int rx = (x.a == 1) + (x.b == 1), ry = (y.a == 1) + (y.b == 1);
    return rx != ry ? rx > ry : mag(x.a) + mag(x.b) < mag(y.a) + mag(y.b);
  });

  ContractParams& p = l->p;
  std::memset(&p, 0, sizeof p);
  // The range of each operand's fetches: its declared buffer, or the hull's last address if that comes first.
  int64_t first[2];
  for (int side = 0; side < 2; ++side) {
    const FlatRef& r = fb.ref[(side == 0) != l->swap ? 0 : 1];
    i128 origin = r.addr.k, end = 0, hull = r.addr.k;
    for (int d = 0; d < r.ndim; ++d) {
      origin -= (i128)r.coord[d].k * r.strides[d];
      end += (i128)(r.sizes[d] - 1) * r.strides[d];
    }
    for (int j = 0; j < fb.n_idx; ++j)
      if (r.addr.c[j] > 0) hull += (i128)r.addr.c[j] * (fb.range[j] - 1);
    end = std::min(end, hull - origin) + 1;
    if (origin < 0 || origin > lim / esize || end < 1) return false;
    first[side] = (int64_t)origin;
    (side == 0 ? p.bytes_a : p.bytes_b) = (uint32_t)std::min(end * esize, (i128)kRecords);
  }
  l->first_a = first[0];
  l->first_b = first[1];
  if (!fill_side(m, &p.m) || !fill_side(n, &p.n) || !fill_side(k, &p.k)) return false;
  i128 M = 1, N = 1, K = 1;
  for (const Ix& x : m) M *= x.range;
  for (const Ix& x : n) N *= x.range;
  for (const Ix& x : k) K *= x.range;
  if (M > lim || N > lim || K > lim) return false;
  p.M = (uint32_t)M; p.N = (uint32_t)N; p.K = (uint32_t)K;
  for (size_t j = 0; j < m.size(); ++j) {
    p.m_in[j] = (int32_t)m[j].a;
    p.m_out[j] = (int32_t)m[j].o;
    for (int t = 0; t < kCtTests; ++t) p.m_ob[t][j] = (int32_t)m[j].ob[t];
  }
  for (size_t j = 0; j < n.size(); ++j) {
    p.n_in[j] = (int32_t)n[j].b;
    p.n_out[j] = (int32_t)n[j].o;
    for (int t = 0; t < kCtTests; ++t) p.n_ob[t][j] = (int32_t)n[j].ob[t];
  }
  for (size_t j = 0; j < k.size(); ++j) {
    p.k_a[j] = (int32_t)k[j].a;
    p.k_b[j] = (int32_t)k[j].b;
  }
  p.a_base = (int32_t)(base_a - first[0]); p.b_base = (int32_t)(base_b - first[1]); p.o_base = (int32_t)fb.ref[2].addr.k;
  p.batch_range[0] = p.batch_range[1] = 1;
  l->batch = 1;
  for (size_t j = 0; j < bat.size(); ++j) {
    p.batch_range[j] = (uint32_t)bat[j].range;
    p.batch_a[j] = (int32_t)bat[j].a; p.batch_b[j] = (int32_t)bat[j].b; p.batch_o[j] = (int32_t)bat[j].o;
    l->batch *= bat[j].range;
    if (l->batch > 65535) return false;
  }
  p.n_ob_used = n_ob;     // unused bounds: 0 <= 0
  for (int t = 0; t < kCtTests; ++t) p.ob[t] = (int32_t)ob[t];

  // constraints -> range tests; a pair f + c >= 0, -f + d >= 0 is one test.  A test with a column index goes to B, any
  // other to A; one over reduction indexes alone can guard both.
  for (int t = 0; t < kCtTests; ++t) p.top_a[t] = p.top_b[t] = kTop;
  int used_a = 0, used_b = 0;
  std::vector<char> done(n_con, 0);
  std::vector<Affine> guards_a, guards_b;                   // the block's own constraints that an operand is tested for
  struct KTest {
    size_t q;
    int64_t top;
    std::vector<size_t> members;
  };
  std::vector<KTest> k_only;
  auto add_a = [&](size_t q, int64_t top) {
    if (used_a >= kCtTests) return false;
    p.c_a[used_a] = (int32_t)con_k[q];
    p.top_a[used_a] = (uint32_t)top;
    for (size_t j = 0; j < m.size(); ++j) p.m_t[used_a][j] = (int32_t)m[j].con[q];
    for (size_t j = 0; j < k.size(); ++j) p.ka_t[used_a][j] = (int32_t)k[j].con[q];
    ++used_a;
    return true;
  };
  auto add_b = [&](size_t q, int64_t top) {
    if (used_b >= kCtTests) return false;
    p.c_b[used_b] = (int32_t)con_k[q];
    p.top_b[used_b] = (uint32_t)top;
    for (size_t j = 0; j < n.size(); ++j) p.n_t[used_b][j] = (int32_t)n[j].con[q];
    for (size_t j = 0; j < k.size(); ++j) p.kb_t[used_b][j] = (int32_t)k[j].con[q];
    ++used_b;
    return true;
  };
  for (size_t q = 0; q < n_con; ++q) {
    if (done[q]) continue;
    bool in_m = false, in_n = false;
    for (const Ix& x : m) in_m = in_m || x.con[q];
    for (const Ix& x : n) in_n = in_n || x.con[q];
    for (const Ix& x : bat)
      if (x.con[q]) return false;
    if (in_m && in_n) return false;
    int64_t top = kTop;
    std::vector<size_t> members{q};
    for (size_t r = q + 1; r < n_con; ++r) {
      bool opposite = !done[r];
      for (const Ix& x : ix) opposite = opposite && x.con[r] == -x.con[q];
      if (opposite) {
        done[r] = 1;
        top = std::min(top, con_k[q] + con_k[r]);
        members.push_back(r);
      }
    }
    if (top < 0) return false;
    if (!(in_n ? add_b(q, top) : add_a(q, top))) return false;
    for (size_t r : members)
      if (r < first_new) (in_n ? guards_b : guards_a).push_back(fb.cons[r]);
    if (!in_m && !in_n) k_only.push_back({q, top, members});
  }
  // Does an operand stay inside its buffer under its own tests?  (The rewritten pairs' tests restore the block's own ranges.)
  const int ref_a = l->swap ? 1 : 0, ref_b = 1 - ref_a;
  const bool inside_a = access_inside(fb, ref_a, guards_a);
  bool inside_b = access_inside(fb, ref_b, guards_b);
  for (size_t t = 0; t < k_only.size() && !inside_b; ++t) {
    if (!add_b(k_only[t].q, k_only[t].top)) break;
    for (size_t r : k_only[t].members)
      if (r < first_new) guards_b.push_back(fb.cons[r]);
    inside_b = access_inside(fb, ref_b, guards_b);
  }
  p.tested = used_a + used_b > 0;

  // How each operand is fetched.  An operand that may leave its buffer at a removed point is fetched element by element
  // (an element is inside the buffer's range or it is not; a vector could straddle its end).  A vector needs its elements neighbours and under the same tests, and stays inside one
  // run of its innermost index: the run is a multiple of the vector, or the side has one index only of at least a vector,
  // whose end is fetched as an overlapping vector.  (Buffer loads take any element alignment.)  Where no 16-byte vector fits
  // the innermost reduction index (three or 24 channels), 8-byte vectors do, with that index's range padded to whole
  // vectors: the padding is zero in both operands.  For three bf16 channels that is one load and one set of range tests for
  // four elements of k.
  const int ve = 16 / esize, ve3 = 8 / esize, vr = dt == STRIPE_F32 ? 4 : 8;
  auto fetch = [&](bool a) {
    if (!(a ? inside_a : inside_b)) return 0;
    const Ix& k0 = k[0];
    const std::vector<Ix>& row = a ? m : n;
    bool k_tests = false, row_tests = false;
    for (int t = 0; t < kCtTests; ++t) {
      k_tests = k_tests || (a ? p.ka_t[t][0] : p.kb_t[t][0]) != 0;
      row_tests = row_tests || (a ? p.m_t[t][0] : p.n_t[t][0]) != 0;
    }
    const bool k_unit = (a ? k0.a : k0.b) == 1 && !k_tests;
    if (k_unit && ((k.size() == 1 && k0.range >= ve) || k0.range % ve == 0)) return 1;
    if (!row.empty() && (a ? row[0].a : row[0].b) == 1 && !row_tests && ((row.size() == 1 && row[0].range >= vr) || row[0].range % vr == 0)) return 2;
    if (k_unit && (a ? p.bytes_a : p.bytes_b) >= 8 && k0.range > 1) return 3;
    return 0;
  };
  p.mode_a = fetch(true);
  p.mode_b = fetch(false);
  p.k_run = (int32_t)k[0].range;
  if ((p.mode_a == 3 || p.mode_b == 3) && k[0].range % ve3) {
    const int64_t padded = (k[0].range + ve3 - 1) / ve3 * ve3;
    const i128 padded_K = K / k[0].range * padded;
    if (padded_K > lim / 4) return false;
    k[0].range = padded;
    if (!fill_side(k, &p.k)) return false;
    p.K = (uint32_t)padded_K;
  }
  bool vec = n[0].o == 1 && n[0].range % 4 == 0 && p.o_base % 4 == 0 && !n[0].ob[0] && !n[0].ob[1];
  for (size_t j = 1; j < n.size(); ++j) vec = vec && n[j].o % 4 == 0;
  for (const Ix& x : m) vec = vec && x.o % 4 == 0;
  for (const Ix& x : bat) vec = vec && x.o % 4 == 0;
  p.vec_out = vec;
  p.epilogue = fb.out_bf16 ? 1 : 0;

  i128 points = 1;
  for (int j = 0; j < fb.n_idx; ++j) points *= fb.range[j];
  const int least = tune_int("contract_min", 0);     // STRIPE_TUNE contract_min = n: every block of at least n points; 0: the rule
  if (least > 0 && points < least) return false;
  auto tiles = [&](int t) { return ((M + kTiles[t].bm - 1) / kTiles[t].bm) * ((N + kTiles[t].bn - 1) / kTiles[t].bn) * l->batch; };
  const bool simple = m.size() <= 1 && n.size() == 1 && k.size() == 1 && !p.tested;      // a product
  l->plain = simple && (p.mode_a == 1 || p.mode_a == 2) && (p.mode_b == 1 || p.mode_b == 2);
  // A bf16 output's own rounding hides the sums'.
  auto precise_on = [&](int t) { return !fb.out_bf16 && wants_double(dt, t, tiles(1) < 96, lit); };
  auto runs = [&](int t) {
    if (t == 3 && p.mode_b == 2 && esize < 4) return false;
    if (t == 5 && !l->plain) return false;
    if (t == 6 && l->plain) return false;
    return !(precise_on(t) && (t == 0 || t == 3 || t == 5));
  };
  int tile = -1;
  for (int t = 0; t < 7; ++t) {
    if (!runs(t)) continue;
    const int singles = (p.mode_a == 0 ? kTiles[t].bm : 0) + (p.mode_b == 0 ? kTiles[t].bn : 0);
    const double us = tile_us(dt, t, l->plain, singles, (p.mode_a == 2) + (p.mode_b == 2), (double)tiles(t), (double)p.K * esize);
    if (tile < 0 || us < l->us) {
      tile = t;
      l->us = us;
    }
  }
  const int forced = tune_int("contract_tile", -1);
  if (forced >= 0 && forced <= 6) tile = forced;
  if (tile == 3 && p.mode_b == 2 && esize < 4) tile = 1;
  if (tile == 5 && (!l->plain || precise_on(5))) tile = 1;
  l->precise = precise_on(tile);
  l->tile = tile;
  const int bkb = tile == 4 && !l->plain ? 128 : kTiles[tile].bkb;
  const i128 grid = tiles(tile) / l->batch;
  if (grid > 0x7fffffff) return false;
  if (least == 0 && literal_is_faster(dt, p, lit, simple, fused, points, l->us)) return false;
  p.tiles_n = (int32_t)((N + kTiles[tile].bn - 1) / kTiles[tile].bn);
  l->grid = (int64_t)grid;
  l->use = true;
  info->path = STRIPE_PATH_GENERIC;
  info->tile_m = kTiles[tile].bm; info->tile_n = kTiles[tile].bn; info->tile_k = bkb / esize;
  info->frag_m = info->frag_n = 16;
  info->frag_k = dt == STRIPE_F32 ? 4 : 64 / esize;
  const Tile& kt = kTiles[tile];
  info->lds_bytes = kt.lanes > 256 ? waves_lds_bytes(esize, kt.lanes / 64, kt.bm, kt.bn, bkb, p.mode_a, p.mode_b, l->precise, l->plain)
                                   : shared_lds_bytes(esize, kt.bm, kt.bn, bkb, p.mode_a, p.mode_b);
  info->workgroup_size = kTiles[tile].lanes;
  info->grid = l->grid * l->batch;
  std::snprintf(info->kernel, sizeof info->kernel, "contract_%s_%dx%dx%d_fetch%d%d%s", dt == STRIPE_F32 ? "f32" : dt == STRIPE_BF16 ? "bf16" : "i8",
                kTiles[tile].bm, kTiles[tile].bn, (int)info->tile_k, p.mode_a, p.mode_b, l->precise ? "_f64" : "");
  return true;
}

hipError_t launch_contract(const ContractLaunch& l, int in_dtype, const void* in0, const void* in1, void* out, const float* bias, bool out_bf16,
                           hipStream_t stream) {
  if (!l.use || l.grid <= 0) return hipErrorInvalidValue;
  ContractParams p = l.p;
  if (bias) p.epilogue = out_bf16 ? 3 : 2;
  if ((uintptr_t)out % ((p.epilogue & 1) ? 8 : 16)) p.vec_out = 0;
  const int64_t esize = in_dtype == STRIPE_F32 ? 4 : in_dtype == STRIPE_BF16 ? 2 : 1;
  const void *a = (const char*)(l.swap ? in1 : in0) + l.first_a * esize, *b = (const char*)(l.swap ? in0 : in1) + l.first_b * esize;
  switch (in_dtype) {
    case STRIPE_I8: return launch_contract_i8(l, p, a, b, out, bias, stream);
    case STRIPE_BF16: return launch_contract_bf16(l, p, a, b, out, bias, stream);
    default: return launch_contract_f32(l, p, a, b, out, bias, stream);
  }
}
#endif

}  // namespace stripe
