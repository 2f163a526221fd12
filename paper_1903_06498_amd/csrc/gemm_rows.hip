// Products with few rows (gfx950): C[m, n] = sum over k of A[m, k] * B[n, k] with at most 32 rows, both operands
// k-contiguous -- a Linear layer at a small batch.  What bounds it is reading B once; a 256-wide tile leaves most CUs
// idle (4096 x 4096 weights: 16 workgroups) and computes padding rows.
//
// A workgroup owns 16 columns; its eight wavefronts share the reduction out in 128-byte pieces (together 1 KB of every
// row per step) and add their sums through LDS, so 4096 columns are 256 workgroups with up to 16 16-byte loads of B per lane
// in flight.  Nothing is staged: a lane's 16 bytes along k are a matrix instruction's fragment as they are, for
// both operands; A (a few rows) comes from L2.  Rows, columns and k beyond the operand load zeros (buffer range).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdio>
#include <type_traits>

#include "kernels.hpp"

namespace stripe {
namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef int32_t i32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));

constexpr uint32_t kOutside = 0x80000000u, kRecords = 0x7fffffffu;
constexpr int kWaves = 8, kCols = 16, kMaxRows = 32;

template <typename T>
__device__ __forceinline__ f32x4 mma(u32x4 a, u32x4 b, f32x4 c) {
  if constexpr (sizeof(T) == 2) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
  } else {
    const f32x4 x = __builtin_bit_cast(f32x4, a), y = __builtin_bit_cast(f32x4, b);
#pragma unroll
    for (int i = 0; i < 4; ++i) c = __builtin_amdgcn_mfma_f32_16x16x4f32(x[i], y[i], c, 0, 0, 0);
    return c;
  }
}
template <typename T>
__device__ __forceinline__ i32x4 mma(u32x4 a, u32x4 b, i32x4 c) {
  return __builtin_amdgcn_mfma_i32_16x16x64_i8(__builtin_bit_cast(i32x4, a), __builtin_bit_cast(i32x4, b), c, 0, 0, 0);
}

// epilogue: 0 sums; 2 relu(sum + bias[n]) in fp32; 3 the same in bf16
template <typename T, int FM, int UNROLL>
__global__ __launch_bounds__(64 * kWaves) void rows_kernel(const T* __restrict__ A, const T* __restrict__ B, void* __restrict__ C, const float* __restrict__ bias,
                                                           uint32_t M, uint32_t N, uint32_t k_bytes, uint32_t a_row, uint32_t b_row, int64_t c_row,
                                                           int epilogue, int vec_out) {
  using Acc = typename std::conditional<sizeof(T) == 1, i32x4, f32x4>::type;
  using S = typename std::conditional<sizeof(T) == 1, int32_t, float>::type;
  // float types: sums of 16 (fp32) or 64 (bf16) products start from zero and join a total in double precision.  With one fp32
  // accumulator over all of a wavefront's k, a chain of K / 8 roundings, the error against 64 bits was 2.6 times (fp32) and
  // 1.3 times (bf16, median) that of the kernels these products ran on before, now at most the same and half of it (fp32,
  // median); 8 x 4096 x 4096 bf16 takes the same time, 16 x 4096 x 2048 fp32 10.6 instead of 10.0 us.
  constexpr int FLUSH = sizeof(T) == 4 ? 1 : 2;
  using Total = typename std::conditional<sizeof(T) == 1, i32x4, f64x4>::type;
  __shared__ Total part[kWaves][FM][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, row = lane & 15;
  const uint32_t n0 = blockIdx.x * kCols;
  const __amdgpu_buffer_rsrc_t buf_a = __builtin_amdgcn_make_buffer_rsrc((void*)A, 0, kRecords, 0x00020000);
  const __amdgpu_buffer_rsrc_t buf_b = __builtin_amdgcn_make_buffer_rsrc((void*)B, 0, kRecords, 0x00020000);
  const bool b_in = n0 + row < N;
  const uint32_t b_off = (n0 + row) * b_row;
  uint32_t a_off[FM];
  bool a_in[FM];
#pragma unroll
  for (int i = 0; i < FM; ++i) {
    a_in[i] = (uint32_t)(i * 16 + row) < M;
    a_off[i] = (i * 16 + row) * a_row;
  }
  Total total[FM];
#pragma unroll
  for (int i = 0; i < FM; ++i) total[i] = (Total){0, 0, 0, 0};
  // the bias of the columns this lane stores, asked for before the reduction
  const uint32_t n = n0 + (lane >> 4) * 4;
  float bs[4] = {0.f, 0.f, 0.f, 0.f};
  if (epilogue && wave < FM) {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (n + e < N) bs[e] = bias[n + e];
  }
  uint32_t at = wave * 128 + (lane >> 4) * 16;
  const uint32_t steps = (k_bytes + kWaves * 128 - 1) / (kWaves * 128);
  for (uint32_t s = 0; s < steps; s += UNROLL) {
    u32x4 b[2 * UNROLL], a[2 * UNROLL][FM];
#pragma unroll
    for (int u = 0; u < 2 * UNROLL; ++u) {      // piece u / 2 of the unrolled steps, its lower or upper 64 bytes
      const uint32_t k = at + u / 2 * (kWaves * 128) + u % 2 * 64;
      b[u] = __builtin_amdgcn_raw_buffer_load_b128(buf_b, b_in && k < k_bytes ? b_off + k : kOutside, 0, 0);
    }
#pragma unroll
    for (int u = 0; u < 2 * UNROLL; ++u) {
      const uint32_t k = at + u / 2 * (kWaves * 128) + u % 2 * 64;
#pragma unroll
      for (int i = 0; i < FM; ++i) a[u][i] = __builtin_amdgcn_raw_buffer_load_b128(buf_a, a_in[i] && k < k_bytes ? a_off[i] + k : kOutside, 0, 0);
    }
    __builtin_amdgcn_sched_barrier(0);          // all loads of the unrolled steps are issued before the first is waited for
    Acc acc[FM];
#pragma unroll
    for (int u = 0; u < 2 * UNROLL; ++u)
#pragma unroll
      for (int i = 0; i < FM; ++i) {            // rows of the result: n
        if constexpr (sizeof(T) == 1) {
          total[i] = mma<T>(b[u], a[u][i], total[i]);
        } else {
          acc[i] = mma<T>(b[u], a[u][i], u % FLUSH ? acc[i] : (Acc){0, 0, 0, 0});
          if (u % FLUSH == FLUSH - 1) total[i] += __builtin_convertvector(acc[i], f64x4);
        }
      }
    at += UNROLL * kWaves * 128;
  }
#pragma unroll
  for (int i = 0; i < FM; ++i) part[wave][i][lane] = total[i];
  __syncthreads();
  if (wave >= FM) return;
  Total sum = part[0][wave][lane];
#pragma unroll
  for (int w = 1; w < kWaves; ++w) sum += part[w][wave][lane];
  const uint32_t m = wave * 16 + row;
  if (m >= M) return;
  S v[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    v[e] = (S)sum[e];
    if constexpr (std::is_same<S, float>::value) {
      if (epilogue) {
        const float y = v[e] + bs[e];
        v[e] = y > 0.f ? y : 0.f;
      }
    }
  }
  const int64_t off = (int64_t)m * c_row + n;
  if (vec_out && n + 4 <= N) {
    typedef S s4 __attribute__((ext_vector_type(4)));
    if (epilogue == 3) *(bf16x4*)((uint16_t*)C + off) = __builtin_convertvector((f32x4){(float)v[0], (float)v[1], (float)v[2], (float)v[3]}, bf16x4);
    else *(s4*)((S*)C + off) = (s4){v[0], v[1], v[2], v[3]};
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (n + e < N) {
        if (epilogue == 3) ((__bf16*)C)[off + e] = (__bf16)(float)v[e];
        else ((S*)C)[off + e] = v[e];
      }
  }
}

template <typename T>
hipError_t launch_t(const GemmShape& g, const void* a, const void* b, void* c, const float* bias, int epi, int64_t c_row, int vec, hipStream_t s) {
  const dim3 grid((unsigned)((g.N + kCols - 1) / kCols)), wg(64 * kWaves);
  const T *pa = (const T*)a + g.a_base, *pb = (const T*)b + g.b_base;
  const uint32_t e = sizeof(T);
  // a step beyond the reduction costs its loads and matrix instructions all the same: no more steps at once than there are
  // (2 x 120000 x 512 bf16, one step: 80 us with eight at once, 27 us with two)
  const uint32_t steps = ((uint32_t)g.K * e + kWaves * 128 - 1) / (kWaves * 128);
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, grid, wg, 0, s, pa, pb, c, bias, (uint32_t)g.M, (uint32_t)g.N, (uint32_t)g.K * e, (uint32_t)g.a_m * e,
                       (uint32_t)g.b_n * e, c_row, epi, vec);
  };
  if (g.M <= 16) {
    if (steps <= 2) go(rows_kernel<T, 1, 2>);
    else if (steps <= 4) go(rows_kernel<T, 1, 4>);
    else go(rows_kernel<T, 1, 8>);
  } else {
    if (steps <= 2) go(rows_kernel<T, 2, 2>);
    else go(rows_kernel<T, 2, 4>);
  }
  return hipGetLastError();
}

}  // namespace

// What this kernel takes: every workgroup walks the whole reduction in steps of 1 KB per row, whose time grows with the rows of
// A fetched beside B (2 rows 0.52, 8 0.66, 16 0.80, 32 1.19 us), 256 workgroups at a time, and the operands come from memory
// once.  Few columns and long reductions are the split product's (8 x 256 x 32768 bf16: 47 us here, 16 split; 32 x 1024 x 16384:
// 44 and 23), ten thousands of columns the 256-wide tiles' with more than 16 rows (32 x 120000 x 2048: 164 and 147).
static double rows_us(const GemmShape& g, int64_t e) {
  const double steps = (double)((g.K * e + kWaves * 128 - 1) / (kWaves * 128)), rounds = std::max(1.0, (double)((g.N + kCols - 1) / kCols) / 256);
  return 4.0 + steps * rounds * (0.5 + 0.0186 * (double)g.M + (g.M > 16 ? 0.09 : 0.0)) + (double)g.N * (double)g.K * (double)e * 0.02e-6;
}

bool gemm_rows_select(const GemmShape& g, int in_dtype, double other_us, RowsLaunch* l, stripe_block_info_t* info) {
  l->use = false;
  if (!tune_int("gemm_rows", 1)) return false;
  if (in_dtype != STRIPE_BF16 && in_dtype != STRIPE_I8 && in_dtype != STRIPE_F32) return false;
  const int64_t e = in_dtype == STRIPE_F32 ? 4 : in_dtype == STRIPE_BF16 ? 2 : 1;
  // both operands k-contiguous, whole 16-byte pieces of k (rows at any element: buffer loads need no more), one product
  if (g.a_k != 1 || g.b_k != 1 || g.c_n != 1 || g.batch != 1 || g.M > kMaxRows || g.K * e % 16) return false;
  // at least one piece for each wavefront; operands within a buffer's range
  if (g.K * e < 1024 || g.N > 0x3fffffff || g.a_m > (1 << 24) || g.b_n > (1 << 26)) return false;
  const __int128 a_end = ((__int128)(g.M - 1) * g.a_m + g.K) * e, b_end = ((__int128)(g.N - 1) * g.b_n + g.K) * e;
  if (a_end > 0x7fffff00 || b_end > 0x7fffff00) return false;
  if (rows_us(g, e) > other_us && tune_int("gemm_rows", 1) != 2) return false;    // STRIPE_TUNE gemm_rows = 2: wherever it can
  l->use = true;
  info->tile_m = g.M <= 16 ? 16 : 32; info->tile_n = kCols; info->tile_k = (int)(kWaves * 128 / e);
  info->frag_m = info->frag_n = 16; info->frag_k = in_dtype == STRIPE_F32 ? 4 : (int)(64 / e);
  info->lds_bytes = kWaves * (g.M <= 16 ? 1 : 2) * (in_dtype == STRIPE_I8 ? 1024 : 2048);
  info->workgroup_size = 64 * kWaves;
  info->grid = (g.N + kCols - 1) / kCols;
  std::snprintf(info->kernel, sizeof info->kernel, "gemm_rows_%s_%dx16_w8", in_dtype == STRIPE_F32 ? "f32" : in_dtype == STRIPE_BF16 ? "bf16" : "i8",
                g.M <= 16 ? 16 : 32);
  return true;
}

hipError_t launch_gemm_rows(const GemmShape& g, int in_dtype, const void* a, const void* b, void* c, int64_t c_row, int64_t c_base, const float* bias,
                            bool out_bf16, hipStream_t stream) {
  const int epi = bias ? (out_bf16 ? 3 : 2) : 0;
  void* out = (char*)c + c_base * (out_bf16 ? 2 : 4);
  const int vec = c_row % 4 == 0 && (uintptr_t)out % (out_bf16 ? 8 : 16) == 0;
  switch (in_dtype) {
    case STRIPE_I8: return launch_t<int8_t>(g, a, b, out, bias, epi, c_row, vec, stream);
    case STRIPE_BF16: return launch_t<uint16_t>(g, a, b, out, bias, epi, c_row, vec, stream);
    default: return launch_t<float>(g, a, b, out, bias, epi, c_row, vec, stream);
  }
}

}  // namespace stripe
