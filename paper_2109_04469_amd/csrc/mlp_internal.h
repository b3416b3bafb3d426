// Internal declarations of the warm-start network's kernels (k_mlp.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace pic {

// epilogues of the matrix-core product
enum GemmEpilogue { EP_STORE = 0, EP_BIAS_GELU = 1, EP_BIAS = 2, EP_GELU_GRAD = 3 };

// C[m][n] = sum_k A(m, k) B(k, n), A(m, k) = A[m sam + k sak] (FP32),
// B(k, n) = B[k sbk + n sbn] (FP32 or BF16 bits); operands rounded to BF16,
// FP32 accumulation; epilogue as GemmEpilogue (bias, Z: see k_mlp.hip).
hipError_t launch_gemm_f32(int ep, const float* A, int64_t sam, int64_t sak, const float* B,
                           int64_t sbk, int64_t sbn, float* C, int64_t ldc, const float* bias,
                           float* Z, int M, int N, int K, hipStream_t s);
hipError_t launch_gemm_bf16(int ep, const float* A, int64_t sam, int64_t sak, const uint16_t* B,
                            int64_t sbk, int64_t sbn, float* C, int64_t ldc, const float* bias,
                            float* Z, int M, int N, int K, hipStream_t s);
hipError_t launch_colsum(const float* dZ, int M, int N, float* db, hipStream_t s);
hipError_t launch_mse(const float* Y, const float* T, int64_t count, float* dY, float* loss,
                      hipStream_t s);
struct AdamArgs {
  float* w;
  float* m;
  float* v;
  float lr, b1, b2, eps, wd, bc1, bc2;
};
hipError_t launch_adam(const AdamArgs& a, const float* g, int64_t n, hipStream_t s);
hipError_t launch_to_bf16(const float* src, uint16_t* dst, int64_t n, hipStream_t s);

// ---- networks whose rows fit the LDS (k_mlp_fused.hip) ----------------------

struct MlpDims {
  int n_in, width, depth, n_out;
};

__host__ __device__ inline int pad32(int v) { return (v + 31) & ~31; }

// Layer l of 0 .. depth: input and output features, the offset of its weights
// in the parameter vector (the biases follow them), and the offset of its
// packed BF16 weights.
struct MlpLayer {
  int di, dn;
  int64_t w, packed;
};
__host__ __device__ inline MlpLayer mlp_layer(const MlpDims& d, int l) {
  MlpLayer r;
  r.di = l == 0 ? d.n_in : d.width;
  r.dn = l == d.depth ? d.n_out : d.width;
  r.w = 0;
  r.packed = 0;
  if (l > 0) {
    const int64_t pw = pad32(d.width);
    r.w = (int64_t)(d.n_in + 1) * d.width + (int64_t)(l - 1) * (d.width + 1) * d.width;
    r.packed = pad32(d.n_in) * pw + (int64_t)(l - 1) * pw * pw;
  }
  return r;
}
__host__ __device__ inline int64_t mlp_packed(const MlpDims& d) {
  const MlpLayer r = mlp_layer(d, d.depth);
  return r.packed + (int64_t)pad32(r.di) * pad32(r.dn);
}

// features of the widest row a pass keeps in LDS, and whether two of them fit
constexpr int kMlpMaxRow = 1024;
__host__ __device__ inline int mlp_row(const MlpDims& d, bool train) {
  int v = d.n_in;
  if (d.depth > 0 && d.width > v) v = d.width;
  if (train && d.n_out > v) v = d.n_out;
  return pad32(v);
}

// Buffers of a pass. `rows` is the batch rounded up to 32. Fragment order (of
// the packed weights and of xf and dzf) is that of an operand of the
// 32x32x16 product: blocks of 32 features x 16 k, lane-major, 8 k per lane.
struct MlpArgs {
  MlpDims d;
  const float* par;
  const uint16_t* wf;   // weights for the forward pass: features n, k = inputs
  const uint16_t* wt;   // for the backward pass: features = inputs, k = n
  const float* x;
  float* y;             // [batch][n_out]
  // training only
  const float* target;
  float* gg;            // gelu'(z) of the hidden layers, in accumulator order
  uint16_t* xf;         // layer inputs, features x rows, fragment order
  uint16_t* dzf;        // deltas, the same
  float* dz;            // deltas, [rows][pad32(dn)] per layer
  float* grad;
  float* loss;
  int batch;
  int rows;
};
size_t mlp_xf_elems(const MlpDims& d, int rows);
size_t mlp_dz_elems(const MlpDims& d, int rows);
size_t mlp_gg_elems(const MlpDims& d, int rows);

// packed weights from the parameter vector, wt only if not null
hipError_t launch_mlp_pack(const MlpDims& d, const float* par, uint16_t* wf, uint16_t* wt,
                           hipStream_t s);
hipError_t launch_mlp_forward(const MlpArgs& a, hipStream_t s);
// forward and backward pass up to the deltas of every layer
hipError_t launch_mlp_deltas(const MlpArgs& a, hipStream_t s);
// gradients and loss from the deltas; with `adam` the parameters and packed
// weights (wf, wt) are stepped in the same launch
hipError_t launch_mlp_update(const MlpArgs& a, const AdamArgs* adam, uint16_t* wf, uint16_t* wt,
                             hipStream_t s);

}  // namespace pic
