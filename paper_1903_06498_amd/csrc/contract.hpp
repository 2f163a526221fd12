// Launch record of the general matrix-core contraction (contract.hip): a sum-of-products block as a product
//   O[m, n] = sum over k of A[m, k] * B[k, n]
// whose three sides m, n, k are tuples of the block's indexes.
#pragma once

#include <hip/hip_runtime.h>

#include "plan.hpp"

namespace stripe {

constexpr int kCtIdx = 4;       // indexes per side
constexpr int kCtTests = 2;     // range tests 0 <= f <= top per operand

struct CtIndex {                // one side's flat position -> its indexes, innermost first (division by multiplication)
  int32_t n;
  uint32_t range[kCtIdx], mul[kCtIdx];
  int32_t shift[kCtIdx];
};

struct ContractParams {
  CtIndex m, n, k;
  int32_t m_in[kCtIdx], m_out[kCtIdx], n_in[kCtIdx], n_out[kCtIdx], k_a[kCtIdx], k_b[kCtIdx];   // address coefficients (elements)
  // points outside the polyhedron: 0 <= ca + (m part) + (k part) <= top_a, and the same for B with n
  int32_t m_t[kCtTests][kCtIdx], ka_t[kCtTests][kCtIdx], n_t[kCtTests][kCtIdx], kb_t[kCtTests][kCtIdx];
  int32_t c_a[kCtTests], c_b[kCtTests];
  uint32_t top_a[kCtTests], top_b[kCtTests];
  // output elements nobody writes (transposed convolutions): stored only where (m part) + (n part) <= bound
  int32_t m_ob[kCtTests][kCtIdx], n_ob[kCtTests][kCtIdx], ob[kCtTests];
  int32_t n_ob_used, tested;
  uint32_t M, N, K;
  int32_t a_base, b_base, o_base;
  int32_t mode_a, mode_b;       // how an operand is fetched: 0 element by element, 1 16 bytes along k, 2 vectors along its row index,
                                // 3 8 bytes along k, the innermost reduction index padded to whole vectors
  int32_t k_run;                // the innermost reduction index's range without that padding
  uint32_t bytes_a, bytes_b;    // an operand's declared buffer (from its origin) in bytes: no fetch goes beyond it
  int32_t vec_out;              // 1: four neighbouring outputs of a lane are one 16-byte (8-byte) store
  uint32_t batch_range[2];
  int32_t batch_a[2], batch_b[2], batch_o[2];
  int32_t tiles_n;
  int32_t epilogue;             // 0: fp32 / int32; 1: bf16; 2: relu(sum + bias[n]) in fp32; 3: the same in bf16
};

struct ContractLaunch {
  bool use = false;
  bool swap = false;            // the block's second operand plays A
  int tile = 0;                 // index into the kernel's tile table
  bool precise = false;         // totals in double precision (not on the largest tiles)
  double us = 0;                // the block's estimated time
  bool plain = false;           // one index per side, no tests, both operands fetched in vectors
  int64_t grid = 0, batch = 1;
  int64_t first_a = 0, first_b = 0;   // an operand's buffer origin, in elements from the caller's pointer (a_base, b_base count from it)
  ContractParams p;
};

// The literal kernel the block would run on: lanes that share an output, points one lane sums in a row, reduction indexes, outputs,
// whether sums meet in atomic additions, whether a lane computes a patch of 4 x 4 outputs.
struct LiteralSums {
  int lanes;
  int64_t chain;
  int n_red;
  int64_t outputs;
  bool atomic, tiled;
};
// Fills l if the kernel covers the block and is expected to be the faster one (fused: with a following statement in its store, so
// that the literal kernel would need a launch more); info: kernel name, tile, grid.
bool contract_select(const FlatBlock& fb, const LiteralSums& lit, bool fused, ContractLaunch* l, stripe_block_info_t* info);
// bias != nullptr: fused with a following O = relu(T + bias[n]) of the same output map (out_bf16: its element type)
hipError_t launch_contract(const ContractLaunch& l, int in_dtype, const void* in0, const void* in1, void* out, const float* bias, bool out_bf16,
                           hipStream_t stream);

}  // namespace stripe
