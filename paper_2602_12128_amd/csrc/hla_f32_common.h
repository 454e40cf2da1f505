// Pieces shared by the fp32 matrix-core kernels of the generic path (hla_f32.hip, hla_f32_phi.hip).
#ifndef HLA_F32_COMMON_H_
#define HLA_F32_COMMON_H_

#include "hla_handle.h"
#include "hla_mfma_common.h"

namespace hla {
namespace f32 {

using mf::f32x16;
using mf::f32x4;

// D[32x32] += A[32x2] B[2x32]: lane l holds A[l % 32][l / 32] and B[l / 32][l % 32]; D as in the bf16
// 32x32 shapes (column l % 32, register i is row d_row(i, l / 32)).  The two products are added one
// after the other, each rounded: k runs in the order the steps are issued.
__device__ __forceinline__ f32x16 mfma32(float a, float b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}
// D[16x16] += A[16x4] B[4x16]: lane l holds A[l % 16][l / 16] and B[l / 16][l % 16]; D: column l % 16,
// register i is row 4 (l / 16) + i
__device__ __forceinline__ f32x4 mfma16(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f32x16 zero16() {
  f32x16 z;
#pragma unroll
  for (int i = 0; i < 16; ++i) z[i] = 0.0f;
  return z;
}

// Rows [t0, t0 + nt) of a caller's tensor into LDS as fp32, row stride LD floats; rows from nt on are
// zero.  16-byte loads where the view's pointer and strides allow it (16-byte writes if LD keeps rows
// aligned), all of a thread's in flight together.
template <int D, int TOK, int THREADS, int LD>
__device__ __forceinline__ void stage_rows(const View& X, int b, int h, int t0, int nt, bool bf16, bool vec,
                                           float* dst) {
  if (vec && !bf16) {
    constexpr int P = D / 4, IT = TOK * P / THREADS;  // float4 pieces per row, of a thread
    f32x4 v[IT];
#pragma unroll
    for (int i = 0; i < IT; ++i) {
      const int idx = threadIdx.x + i * THREADS, t = idx / P, p = idx % P;
      v[i] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
      if (t < nt) v[i] = *reinterpret_cast<const f32x4*>(X.row<const float>(b, h, t0 + t) + 4 * p);
    }
#pragma unroll
    for (int i = 0; i < IT; ++i) {
      const int idx = threadIdx.x + i * THREADS, t = idx / P, p = idx % P;
      if constexpr (LD % 4 == 0) {
        *reinterpret_cast<f32x4*>(dst + t * LD + 4 * p) = v[i];
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) dst[t * LD + 4 * p + e] = v[i][e];
      }
    }
    return;
  }
#pragma unroll 8
  for (int i = 0; i < TOK * D / THREADS; ++i) {
    const int idx = threadIdx.x + i * THREADS, t = idx / D, c = idx % D;
    float v = 0.0f;
    if (t < nt) v = bf16 ? to_float(X.row<const bf16_t>(b, h, t0 + t)[c]) : X.row<const float>(b, h, t0 + t)[c];
    dst[t * LD + c] = v;
  }
}

// 16-byte accesses need the pointer and every stride of the view on 16 bytes
inline bool rows_vec(const View& v, size_t elem) {
  return ((reinterpret_cast<uintptr_t>(v.ptr) | (v.sb * elem) | (v.sh * elem) | (v.sn * elem)) & 15) == 0;
}

}  // namespace f32
}  // namespace hla

#endif  // HLA_F32_COMMON_H_
