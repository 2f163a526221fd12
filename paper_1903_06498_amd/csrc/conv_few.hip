// Convolutions with at most four input channels on the matrix cores (gfx950): the first layer of an image network,
//   O[n,y,x,k] = sum over taps (i,j) and channels c of I[n, sy*y+i-py, sx*x+j-px, c] * F[i,j,k,c],
// bf16, fp32 or int8, any filter, stride and padding, any number of output channels.
//
// The contraction of three channels at a time fetched every input element once for each of its taps, 8 bytes a load with two
// range tests each (7x7 stride 2, 3 -> 64, bf16, 8 x 224 x 224: 34 us on the general contraction for 14 MB).  Here a workgroup puts
// the image rows of TY output rows into LDS once, every pixel padded to four channels and the rows to the taps outside the image
// (zeros), so the taps j, j+1, .. of one filter row are consecutive bytes: a lane's 16 bytes of k are 2 (bf16), 1 (fp32) or 4 (int8)
// taps of its output pixel, read where they lie, whatever the stride.  A K step is four such chunks -- 16x16x32 bf16, 16x16x64 int8 or
// four 16x16x4 fp32 instructions -- and the filter's fragments stay in registers.  Filter rows end with zero weights where the
// taps do not fill a chunk (7 taps of bf16: 8), a fourth channel is zero in both operands.
// The filter's rows are laid out so that a lane ends up with 4 * FN consecutive output channels of its pixel, which leave
// in stores of four of them (fp32, int32: 16 bytes, bf16: 8) without a pass through LDS; ordinary ones, since a line of the output
// is written by several of them, which meet in L2 (past it, 24 x 94 x 94, 3 -> 64, 3x3, int8 took 68.1 us instead of 25.4).
// What bounds it at that size (34.7 us before, 12.2 here; 13.6 to 18.2, by where the output lay in memory, with stores past L2): the rows' arrival, then the
// write of the output (12.8 MB in bf16, 2.3 us), one after the other in the one workgroup that a CU has (up to 200 registers of filter
// and sums).  The same layer in int8 at 13 x 61 x 61, 7x7 to 32 channels: 11.7 and 5.8; in fp32 at 3 x 75 x 75, 7x7 to 64: 21.6 and 12.0.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdio>
#include <type_traits>

#include "kernels.hpp"

namespace stripe {
namespace {

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4_at4 __attribute__((ext_vector_type(4), aligned(4)));
typedef int32_t i32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));

constexpr int kWaves = 8, kLanes = 64 * kWaves;
constexpr uint32_t kOutside = 0x80000000u;
constexpr int kMaxLds = 144 * 1024;      // the vote of __syncthreads_or takes a little more

struct FewParams {
  int32_t Ho, Wo, H, W, Co, Ci, R, S, sy, sx, py, px;
  int32_t ty, strips;               // output rows of a workgroup, workgroups per image
  int32_t chunks_per_row;           // 16-byte chunks of taps per filter row
  int32_t rows, cols, groups;       // image rows and columns in LDS, groups of 16 output pixels per row
  int32_t row_bytes, filter_bytes;  // LDS: a row, the filter in front of the rows
  uint32_t chunks_mul, groups_mul;  // ceil(2^32 / chunks_per_row), ceil(2^32 / groups); 0 where that is 1
  int32_t co_tiles, co_split;       // tiles of output channels, workgroups they are shared out to
  int32_t i_n, i_y, i_x, f_r, f_s, f_k;      // bytes
  int32_t i_base, f_base;                    // bytes
  uint32_t i_bytes, f_bytes;        // the operands' ends
  int64_t o_n, o_y, o_x, o_base;    // elements
  int32_t epilogue;                 // 0: sums; 2: relu(sum + bias[k]) in fp32; 3: the same in bf16
  int32_t vec;                      // four channels are one store
};

template <typename T>
struct Few;
template <>
struct Few<uint16_t> {
  using Acc = f32x4;
  template <bool>
  static __device__ __forceinline__ void add(u32x4 a, u32x4 b, Acc& c) {
    c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
  }
  static __device__ __forceinline__ float widen(const unsigned char* p) { return __uint_as_float((uint32_t)*(const uint16_t*)p << 16); }
  static __device__ __forceinline__ bool finite(uint32_t w) { return ((w & 0x7f80u) != 0x7f80u) & ((w & 0x7f800000u) != 0x7f800000u); }
};
template <>
struct Few<float> {
  using Acc = f32x4;
  // 16 products in one chain that starts from zero; the few of a short filter as two chains of eight
  template <bool SHORT>
  static __device__ __forceinline__ void add(u32x4 a, u32x4 b, Acc& c) {
    const f32x4 x = __builtin_bit_cast(f32x4, a), y = __builtin_bit_cast(f32x4, b);
    Acc s[2] = {(Acc){0, 0, 0, 0}, (Acc){0, 0, 0, 0}};
#pragma unroll
    for (int i = 0; i < 4; ++i) s[SHORT ? i / 2 : 0] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[i], y[i], s[SHORT ? i / 2 : 0], 0, 0, 0);
    c += SHORT ? s[0] + s[1] : s[0];
  }
  static __device__ __forceinline__ float widen(const unsigned char* p) { return *(const float*)p; }
  static __device__ __forceinline__ bool finite(uint32_t w) { return (w & 0x7f800000u) != 0x7f800000u; }
};
template <>
struct Few<int8_t> {
  using Acc = i32x4;
  template <bool>
  static __device__ __forceinline__ void add(u32x4 a, u32x4 b, Acc& c) {
    c = __builtin_amdgcn_mfma_i32_16x16x64_i8(__builtin_bit_cast(i32x4, a), __builtin_bit_cast(i32x4, b), c, 0, 0, 0);
  }
  static __device__ __forceinline__ float widen(const unsigned char* p) { return (float)*(const int8_t*)p; }
  static __device__ __forceinline__ bool finite(uint32_t) { return true; }
};

// Four channels of a pixel (or of a filter tap and output channel): the first `ci` elements at byte `off`, zeros behind them.  A load
// that would end behind the operand is made from its last bytes and shifted down.  end: the operand's bytes, at least one load.
template <typename T>
struct Pixel {
  static constexpr int N = sizeof(T);      // dwords
  uint32_t w[N];
  __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t buf, uint32_t off, uint32_t end, int ci) {
    const uint32_t last = end - 4 * N;
    const bool late = off > last && off != kOutside;
    const uint32_t at = late ? last : off, back = late ? off - last : 0;      // bytes to shift down
    if constexpr (N == 1) {
      w[0] = __builtin_amdgcn_raw_buffer_load_b32(buf, at, 0, 0) >> (8 * back);
      w[0] &= ci >= 4 ? 0xffffffffu : (1u << (8 * ci)) - 1;
    } else if constexpr (N == 2) {
      const u32x2 x = __builtin_amdgcn_raw_buffer_load_b64(buf, at, 0, 0);
      uint64_t v = (x[0] | (uint64_t)x[1] << 32) >> (8 * back);
      v &= ci >= 4 ? ~0ull : (1ull << (16 * ci)) - 1;
      w[0] = (uint32_t)v;
      w[1] = (uint32_t)(v >> 32);
    } else {
      const u32x4 x = __builtin_amdgcn_raw_buffer_load_b128(buf, at, 0, 0);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        uint32_t v = x[e];
#pragma unroll
        for (int s = 1; s < 4; ++s)
          if (back == 4u * s) v = e + s < 4 ? x[e + s < 4 ? e + s : 0] : 0;
        w[e] = e < ci ? v : 0;
      }
    }
  }
  __device__ __forceinline__ bool finite() const {
    bool f = true;
#pragma unroll
    for (int e = 0; e < N; ++e) f &= Few<T>::finite(w[e]);
    return f;
  }
  __device__ __forceinline__ void store(unsigned char* at) const {
    if constexpr (N == 1) *(uint32_t*)at = w[0];
    else if constexpr (N == 2) *(u32x2*)at = (u32x2){w[0], w[1]};
    else *(u32x4*)at = (u32x4){w[0], w[1], w[2], w[3]};
  }
};

// STEPS: K steps of four chunks (at least the filter's); FN: fragments of 16 output channels
template <typename T, int STEPS, int FN>
__global__ __launch_bounds__(kLanes, 2) void conv_few_kernel(const FewParams p, const unsigned char* __restrict__ I, const unsigned char* __restrict__ F,
                                                          void* __restrict__ O, const float* __restrict__ bias) {
  using Acc = typename Few<T>::Acc;
  using S = typename std::conditional<sizeof(T) == 1, int32_t, float>::type;
  constexpr int PX = 4 * sizeof(T), TAPS = 16 / PX, CO = 16 * FN, BATCH = 4;
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  unsigned char* const img = lds + p.filter_bytes;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = (int)blockIdx.x / p.strips, y0 = ((int)blockIdx.x - n * p.strips) * p.ty;
  const __amdgpu_buffer_rsrc_t buf_i = __builtin_amdgcn_make_buffer_rsrc((void*)I, 0, (int)p.i_bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t buf_f = __builtin_amdgcn_make_buffer_rsrc((void*)F, 0, (int)p.f_bytes, 0x00020000);
  bool fin = true;
  auto divide = [](uint32_t v, uint32_t mul) { return mul ? __umulhi(v, mul) : v; };      // v < 2^16

  // ---- the filter of CO output channels: [slot][row of the fragments][16 bytes]; channel 4*FN*q + 4*j + e of the tile is row
  // 4*q + e of fragment j.  All loads of a lane are in flight together (one after the other they were a third of the call's time).
  constexpr int FILTER = (STEPS * 4 * TAPS * CO + kLanes - 1) / kLanes;
  const int slots = p.R * p.chunks_per_row;
  Pixel<T> fv[FILTER];
  auto load_filter = [&](int ct) {
#pragma unroll
    for (int f = 0; f < FILTER; ++f) {
      const int x = tid + f * kLanes, ko = x % CO, tap = x / CO, slot = tap / TAPS, i = (int)divide((uint32_t)slot, p.chunks_mul);
      const int j = (slot - i * p.chunks_per_row) * TAPS + tap % TAPS, k = ct * CO + ko;
      fv[f].load(buf_f, slot < slots && j < p.S && k < p.Co ? (uint32_t)(p.f_base + i * p.f_r + j * p.f_s + k * p.f_k) : kOutside, p.f_bytes, p.Ci);
    }
  };
  auto store_filter = [&]() {
#pragma unroll
    for (int f = 0; f < FILTER; ++f) {
      const int x = tid + f * kLanes, ko = x % CO, tap = x / CO, slot = tap / TAPS, row = (ko % (4 * FN) / 4) * 16 + ko / (4 * FN) * 4 + ko % 4;
      fin &= fv[f].finite();
      if (x < STEPS * 4 * TAPS * CO) fv[f].store(lds + (slot * CO + row) * 16 + tap % TAPS * PX);
    }
  };
  load_filter((int)blockIdx.y);

  // ---- the rows: a wavefront takes every 8th, BATCH loads of a lane in flight
  for (int r = wave; r < p.rows; r += kWaves) {
    const int y = y0 * p.sy - p.py + r;
    const bool row_in = y >= 0 && y < p.H;
    const int base = row_in ? p.i_base + n * p.i_n + y * p.i_y : 0;
    for (int c0 = 0; c0 < p.cols; c0 += 64 * BATCH) {
      Pixel<T> v[BATCH];
#pragma unroll
      for (int b = 0; b < BATCH; ++b) {
        const int c = c0 + 64 * b + lane, x = c - p.px;
        v[b].load(buf_i, row_in && x >= 0 && x < p.W && c < p.cols ? (uint32_t)(base + x * p.i_x) : kOutside, p.i_bytes, p.Ci);
      }
#pragma unroll
      for (int b = 0; b < BATCH; ++b) {
        const int c = c0 + 64 * b + lane;
        fin &= v[b].finite();
        if (c < p.cols) v[b].store(img + r * p.row_bytes + c * PX);
      }
    }
  }

  const int q = lane >> 4, pixel = lane & 15;
  uint32_t slot_at[STEPS];      // a lane's chunk in each step, from its pixel's first tap
#pragma unroll
  for (int t = 0; t < STEPS; ++t) {
    const int slot = 4 * t + q, i = (int)divide((uint32_t)slot, p.chunks_mul);
    slot_at[t] = slot < slots ? (uint32_t)(i * p.row_bytes + (slot - i * p.chunks_per_row) * 16) : 0;
  }
  const int rows_here = p.Ho - y0 < p.ty ? p.Ho - y0 : p.ty;

  for (int ct = blockIdx.y; ct < p.co_tiles; ct += p.co_split) {
    if (ct != (int)blockIdx.y) {
      load_filter(ct);
      __syncthreads();      // the tile before is done with its own
    }
    store_filter();
    const bool bad = __syncthreads_or(!fin);
    u32x4 fb[STEPS][FN];
#pragma unroll
    for (int t = 0; t < STEPS; ++t)
#pragma unroll
      for (int j = 0; j < FN; ++j) fb[t][j] = *(const u32x4*)(lds + ((4 * t + q) * CO + j * 16 + pixel) * 16);
    const int k0 = ct * CO + q * (4 * FN);
    float bs[FN][4];
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) bs[j][e] = p.epilogue && k0 + 4 * j + e < p.Co ? bias[k0 + 4 * j + e] : 0.f;

    for (int u = wave; u < rows_here * p.groups; u += kWaves) {
      const int row = (int)divide((uint32_t)u, p.groups_mul), x = (u - row * p.groups) * 16 + pixel;
      const unsigned char* at = img + row * p.sy * p.row_bytes + x * p.sx * PX;
      S sum[FN][4];
      if constexpr (sizeof(T) > 1) {
        if (bad) {
          // A zero weight or a tap outside the image contributes 0 * x, which is not 0 where x is an infinity or NaN: such a
          // workgroup sums its points one by one (Definition 2: a removed point contributes nothing).
          const int ylo = (y0 + row) * p.sy - p.py, xlo = x * p.sx - p.px;
#pragma unroll 1
          for (int v = 0; v < 4 * FN; ++v) {
            double total = 0;
#pragma unroll 1
            for (int i = 0; i < p.R; ++i)
#pragma unroll 1
              for (int j = 0; j < p.S; ++j) {
                if (ylo + i < 0 || ylo + i >= p.H || xlo + j < 0 || xlo + j >= p.W) continue;
                const unsigned char* a = at + i * p.row_bytes + j * PX;
                const unsigned char* b = lds + ((i * p.chunks_per_row + j / TAPS) * CO + v / 4 * 16 + q * 4 + v % 4) * 16 + j % TAPS * PX;
                for (int c = 0; c < p.Ci; ++c) total += (double)(Few<T>::widen(a + c * sizeof(T)) * Few<T>::widen(b + c * sizeof(T)));
              }
#pragma unroll
            for (int w = 0; w < 4 * FN; ++w)
              if (w == v) sum[w / 4][w % 4] = (S)total;
          }
        }
      }
      if (sizeof(T) == 1 || !bad) {
        u32x4 fa[STEPS];
#pragma unroll
        for (int t = 0; t < STEPS; ++t) fa[t] = *(const u32x4_at4*)(at + slot_at[t]);
#pragma unroll
        for (int j = 0; j < FN; ++j) {      // rows of the result: output channels; floats: K step t joins sum t % SUMS
          constexpr int SUMS = sizeof(T) == 1 ? 1 : STEPS >= 7 ? 4 : 2;
          Acc acc[4] = {(Acc){0, 0, 0, 0}, (Acc){0, 0, 0, 0}, (Acc){0, 0, 0, 0}, (Acc){0, 0, 0, 0}};
#pragma unroll
          for (int t = 0; t < STEPS; ++t) Few<T>::template add<STEPS == 2>(fb[t][j], fa[t], acc[t % SUMS]);
          if (SUMS == 4) acc[0] += acc[2], acc[1] += acc[3];
          if (SUMS >= 2) acc[0] += acc[1];
#pragma unroll
          for (int e = 0; e < 4; ++e) sum[j][e] = acc[0][e];
        }
      }
      if (x >= p.Wo) continue;
      const int64_t off = p.o_base + n * p.o_n + (int64_t)(y0 + row) * p.o_y + (int64_t)x * p.o_x + k0;
#pragma unroll
      for (int j = 0; j < FN; ++j) {
        if constexpr (std::is_same<S, float>::value) {
          if (p.epilogue) {
#pragma unroll
            for (int e = 0; e < 4; ++e) sum[j][e] = sum[j][e] + bs[j][e] > 0.f ? sum[j][e] + bs[j][e] : 0.f;
          }
        }
      }
#pragma unroll
      for (int j = 0; j < FN; ++j) {
        typedef S s4 __attribute__((ext_vector_type(4)));
        const s4 v = {sum[j][0], sum[j][1], sum[j][2], sum[j][3]};
        const int k = k0 + 4 * j;
        if (p.vec && k + 4 <= p.Co) {
          if (std::is_same<S, float>::value && p.epilogue == 3)
            *(bf16x4*)((uint16_t*)O + off + 4 * j) = __builtin_convertvector((f32x4){(float)v[0], (float)v[1], (float)v[2], (float)v[3]}, bf16x4);
          else *(s4*)((S*)O + off + 4 * j) = v;
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (k + e < p.Co) {
              if (std::is_same<S, float>::value && p.epilogue == 3) ((__bf16*)O)[off + 4 * j + e] = (__bf16)(float)v[e];
              else ((S*)O)[off + 4 * j + e] = v[e];
            }
        }
      }
    }
  }
}

int chunks_of(const Conv2dShape& c, int esize) { return (int)((c.S * 4 * esize + 15) / 16); }

// What lies in LDS, in 64 bits: strides of up to 2^20 make rows that no 32-bit product of them holds.
struct FewLds {
  int64_t rows, cols, groups, row_bytes, filter_bytes;
  int64_t bytes() const { return filter_bytes + rows * row_bytes; }
};
FewLds few_lds(const Conv2dShape& c, int esize, const FewLaunch& l) {
  FewLds f;
  f.rows = (l.ty - 1) * c.stride_y + c.R;
  f.groups = (c.Wo + 15) / 16;
  f.cols = (f.groups * 16 - 1) * c.stride_x + chunks_of(c, esize) * (4 / esize);      // the taps of the last pixel's last chunk included
  f.row_bytes = (f.cols * 4 * esize + 15) / 16 * 16;
  f.filter_bytes = (int64_t)l.steps * 4 * 16 * l.fn * 16;
  return f;
}

// (for shapes that conv_few_select took: everything fits)
FewParams make_params(const Conv2dShape& c, int esize, const FewLaunch& l) {
  FewParams p = {};
  const FewLds lds = few_lds(c, esize, l);
  p.Ho = (int)c.Ho; p.Wo = (int)c.Wo; p.H = (int)c.H; p.W = (int)c.W; p.Co = (int)c.Co; p.Ci = (int)c.Ci;
  p.R = (int)c.R; p.S = (int)c.S; p.sy = (int)c.stride_y; p.sx = (int)c.stride_x; p.py = (int)c.pad_y; p.px = (int)c.pad_x;
  p.ty = l.ty;
  p.strips = (int)((c.Ho + l.ty - 1) / l.ty);
  p.chunks_per_row = chunks_of(c, esize);
  p.rows = (int)lds.rows;
  p.groups = (int)lds.groups;
  p.cols = (int)lds.cols;
  auto magic = [](int d) { return d == 1 ? 0u : (uint32_t)((((uint64_t)1 << 32) + d - 1) / d); };
  p.chunks_mul = magic(p.chunks_per_row);
  p.groups_mul = magic(p.groups);
  p.row_bytes = (int)lds.row_bytes;
  p.filter_bytes = (int)lds.filter_bytes;
  p.co_tiles = (int)((c.Co + 16 * l.fn - 1) / (16 * l.fn));
  p.co_split = l.co_split;
  p.i_n = (int)(c.i_n * esize); p.i_y = (int)(c.i_y * esize); p.i_x = (int)(c.i_x * esize);
  p.f_r = (int)(c.f_r * esize); p.f_s = (int)(c.f_s * esize); p.f_k = (int)(c.f_k * esize);
  p.i_base = (int)(c.i_base * esize); p.f_base = (int)(c.f_base * esize);
  p.i_bytes = (uint32_t)((c.i_base + (c.N - 1) * c.i_n + (c.H - 1) * c.i_y + (c.W - 1) * c.i_x + c.Ci) * esize);
  p.f_bytes = (uint32_t)((c.f_base + (c.R - 1) * c.f_r + (c.S - 1) * c.f_s + (c.Co - 1) * c.f_k + c.Ci) * esize);
  p.o_n = c.o_n; p.o_y = c.o_y; p.o_x = c.o_x; p.o_base = c.o_base;
  return p;
}

}  // namespace

// us, fitted to 316 blocks of one to four channels, 1 to 1008 output channels, 2x2 to 7x7 (standard deviation 11 %).  Per round of
// workgroups: the tiles of output channels that one takes in turn, each with its filter and the image fragments of a wavefront's groups
// of pixels read again; then the write of the output, slower where its channels are no multiple of four and leave one by one, 4 * FN apart.
static double few_us(const Conv2dShape& c, int esize, const FewLaunch& l, int out_size) {
  const double rounds = std::max(1.0, (double)(l.grid * l.co_split) / 256), tiles = std::ceil((double)((c.Co + 16 * l.fn - 1) / (16 * l.fn)) / l.co_split);
  const double units = std::ceil((double)(std::min<int64_t>(l.ty, c.Ho) * ((c.Wo + 15) / 16)) / kWaves);
  const double out_mb = (double)c.N * (double)c.Ho * (double)c.Wo * (double)c.Co * out_size / 1e6;
  return 4.0 + rounds * tiles * (0.32 + units * l.fn * (0.0655 * l.steps * (esize == 4 ? 2 : 1) + 0.02)) + out_mb * (c.Co % 4 == 0 ? 0.245 : l.fn == 4 ? 1.21 : 0.54);
}

bool conv_few_select(const Conv2dShape& c, int in_dtype, int out_size, double other_us, FewLaunch* l, stripe_block_info_t* info) {
  l->use = false;
  if (!tune_int("conv_few", !tune_sets("conv_") && !tune_sets("contract_"))) return false;
  const int esize = in_dtype == STRIPE_F32 ? 4 : in_dtype == STRIPE_BF16 ? 2 : in_dtype == STRIPE_I8 ? 1 : 0;
  if (!esize || c.Ci < 1 || c.Ci > 4 || c.i_c != 1 || c.f_c != 1 || c.o_k != 1 || c.R * c.S < 2) return false;
  if (c.dil_x != 1 || c.dil_y != 1 || c.stride_x < 1 || c.stride_y < 1 || c.pad_x < 0 || c.pad_y < 0) return false;
  // a filter whose fragments fit the registers
  const int64_t chunks = c.R * (int64_t)chunks_of(c, esize), steps = (chunks + 3) / 4;
  if (c.R > 64 || c.S > 64 || steps > (esize == 4 ? 13 : 7)) return false;
  l->steps = steps <= 2 ? 2 : steps <= 4 ? 4 : steps <= 7 ? 7 : 13;
  l->fn = l->steps == 13 ? 2 : c.Co <= 16 ? 1 : c.Co <= 32 ? 2 : 4;
  // offsets in 31 bits; strides forward
  for (int64_t v : {c.i_n, c.i_y, c.i_x, c.f_r, c.f_s, c.f_k, c.i_base, c.f_base, c.o_n, c.o_y, c.o_x, c.o_base})
    if (v < 0) return false;
  for (int64_t v : {c.N, c.Ho, c.Wo, c.H, c.W, c.Co, c.stride_y, c.stride_x, c.pad_y, c.pad_x})
    if (v > (1 << 20)) return false;
  const __int128 i_end = ((__int128)c.i_base + (__int128)(c.N - 1) * c.i_n + (__int128)(c.H - 1) * c.i_y + (__int128)(c.W - 1) * c.i_x + c.Ci) * esize;
  const __int128 f_end = ((__int128)c.f_base + (__int128)(c.R - 1) * c.f_r + (__int128)(c.S - 1) * c.f_s + (__int128)(c.Co - 1) * c.f_k + c.Ci) * esize;
  if (i_end > 0x3fffffff || f_end > 0x3fffffff || i_end < 4 * esize || f_end < 4 * esize) return false;
  // every output element is written: each row and column of outputs has a tap inside the image
  auto all_have_tap = [](int64_t outs, int64_t stride, int64_t pad, int64_t taps, int64_t extent) {
    return pad < taps && (outs - 1) * stride - pad < extent;      // the first and the last one do, so all do (taps are consecutive)
  };
  if (!all_have_tap(c.Ho, c.stride_y, c.pad_y, c.R, c.H) || !all_have_tap(c.Wo, c.stride_x, c.pad_x, c.S, c.W)) return false;
  // Rows per workgroup: the fewest with which every CU has at most one workgroup, up to 8 and half of LDS.  A workgroup's own cost
  // (the filter, the first row's arrival) is paid once per round of workgroups: 8 x 224 x 224 x 3 -> 64, 7x7 stride 2, bf16, takes
  // 28.5 us with one row (896 workgroups), 18.3 with two, 13.7 with four (224), 15.0 with six (152); 9 x 34 x 34 x 3 -> 96, 3x3,
  // fp32, 16.4 with one, 12.8 with two, 9.2 with three (108 x 2), 11.4 with six.
  const int co_tiles = (int)((c.Co + 16 * l->fn - 1) / (16 * l->fn));
  l->co_split = 1;
  l->ty = 1;
  while (l->ty < 8 && l->ty < c.Ho && c.N * ((c.Ho + l->ty - 1) / l->ty) * std::min(co_tiles, 2) > 256) {
    ++l->ty;
    if (few_lds(c, esize, *l).bytes() > 80 * 1024) {
      --l->ty;
      break;
    }
  }
  const int forced = tune_int("conv_few_ty", 0);
  if (forced > 0 && forced <= 64) l->ty = forced;
  const FewLds lds = few_lds(c, esize, *l);
  if (lds.bytes() > kMaxLds || l->ty * lds.groups > 65535) return false;
  const int64_t strips = c.N * ((c.Ho + l->ty - 1) / l->ty);
  while (l->co_split < co_tiles && strips * (l->co_split + 1) <= 256) ++l->co_split;
  if (strips > 0x7fffffff) return false;
  l->grid = strips;
  // Where the general contraction is the faster one, it stays: many tiles of output channels (10 x 50 x 50, 2 -> 1008, 3x3 stride 3,
  // fp32 29.6 us here and 10.9 there), large outputs in single elements (7 x 127 x 127, 3 -> 103, 2x2, fp32 61.8 and 36.8).  The tenth is
  // for both estimates' errors.  Of 316 blocks on both, 5 are taken that lose more than 5 %, and 15 are left that would gain as much.
  if (tune_int("conv_few", 1) != 2 && few_us(c, esize, *l, out_size) > 0.9 * other_us) return false;
  l->lds = (int)lds.bytes();
  l->use = true;
  info->tile_m = (int)(l->ty * 16 * lds.groups); info->tile_n = 16 * l->fn; info->tile_k = 64 / esize;
  info->frag_m = info->frag_n = 16;
  info->frag_k = esize == 4 ? 4 : 64 / esize;
  info->lds_bytes = l->lds;
  info->workgroup_size = kLanes;
  info->grid = strips * l->co_split;
  std::snprintf(info->kernel, sizeof info->kernel, "conv_few_%s_c%dk%d_rows%d", in_dtype == STRIPE_F32 ? "f32" : in_dtype == STRIPE_BF16 ? "bf16" : "i8", (int)c.Ci,
                16 * l->fn, l->ty);
  return true;
}

namespace {

template <typename T>
hipError_t launch_few(const FewParams& p, const FewLaunch& l, const void* in, const void* flt, void* out, const float* bias, hipStream_t st) {
  auto go = [&](auto kernel) {
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev != l.lds_enabled_on) {   // more than 64 KB of dynamic LDS has to be enabled once per device
      e = hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, kMaxLds);
      if (e != hipSuccess) return e;
      l.lds_enabled_on = dev;
    }
    hipLaunchKernelGGL(kernel, dim3((unsigned)l.grid, (unsigned)l.co_split), dim3(kLanes), l.lds, st, p, (const unsigned char*)in, (const unsigned char*)flt, out, bias);
    return hipGetLastError();
  };
  switch (l.steps * 8 + l.fn) {
    case 2 * 8 + 1: return go(conv_few_kernel<T, 2, 1>);
    case 2 * 8 + 2: return go(conv_few_kernel<T, 2, 2>);
    case 2 * 8 + 4: return go(conv_few_kernel<T, 2, 4>);
    case 4 * 8 + 1: return go(conv_few_kernel<T, 4, 1>);
    case 4 * 8 + 2: return go(conv_few_kernel<T, 4, 2>);
    case 4 * 8 + 4: return go(conv_few_kernel<T, 4, 4>);
    case 7 * 8 + 1: return go(conv_few_kernel<T, 7, 1>);
    case 7 * 8 + 2: return go(conv_few_kernel<T, 7, 2>);
    case 7 * 8 + 4: return go(conv_few_kernel<T, 7, 4>);
    case 13 * 8 + 2:
      if constexpr (sizeof(T) == 4) return go(conv_few_kernel<T, 13, 2>);
      return hipErrorInvalidValue;
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

hipError_t launch_conv_few(const Conv2dShape& c, const FewLaunch& l, int in_dtype, const void* in, const void* flt, void* out, const float* bias, bool out_bf16,
                           hipStream_t st) {
  if (!l.use) return hipErrorInvalidValue;
  const int esize = in_dtype == STRIPE_F32 ? 4 : in_dtype == STRIPE_BF16 ? 2 : 1;
  FewParams p = make_params(c, esize, l);
  p.epilogue = bias ? (out_bf16 ? 3 : 2) : 0;
  p.vec = c.o_x % 4 == 0 && c.o_y % 4 == 0 && c.o_n % 4 == 0 && c.o_base % 4 == 0 && (uintptr_t)out % (p.epilogue == 3 ? 8 : 16) == 0;
  switch (in_dtype) {
    case STRIPE_I8: return launch_few<int8_t>(p, l, in, flt, out, bias, st);
    case STRIPE_BF16: return launch_few<uint16_t>(p, l, in, flt, out, bias, st);
    default: return launch_few<float>(p, l, in, flt, out, bias, st);
  }
}

}  // namespace stripe
