// Gradients of the masked second-order HLA for bf16 inputs (MFMA).  See hla2_backward.hip.
#pragma once
#include "common.h"

namespace hla {
struct Bwd {
  const void* q; const void* k; const void* v;   // bf16 [BH][n][d]
  const float* g;                                 // upstream gradient, fp32 [BH][n][dv]
  void* dq; void* dk; void* dv;                   // grad_dtype [BH][n][d] (dv: [BH][n][dv])
  int BH, n, d, dvd, dtype;                      // dvd: value width
  int grad_dtype;                                // of dq, dk, dv: 0 fp32, 1 bf16 (the fp32 sums rounded once)
};
bool backward_supported(int n, int d, int dv, int dtype);
size_t backward_workspace_bytes(int BH, int n, int d, int grad_dtype);
hipError_t launch_backward(const Bwd& b, void* workspace, hipStream_t s);
}  // namespace hla
