// Non-causal operator of the generic path (fp32 features and state, any supported (F, d_phi), fp32 or
// bf16 I/O): state, query contraction and both halves of the backward on the fp32 matrix cores
// (v_mfma_f32_32x32x2_f32: fp32 operands, fp32 accumulation).
//
// Like the bf16 path, everything runs over the monomials of the symmetric form (Qm[m] = product of
// q over the monomial, S[m] = sum over its distinct orderings of the key products,
// C[m] = sum_j S_j[m] (x) v_j): C(d_phi + F - 1, F) rows instead of d_phi^F, exact algebra.
//
// A workgroup serves a run of tokens of one (sequence, head), TOK tokens at a time.  A tile's
// features and rows are staged in LDS; lane = token evaluates monomials and chain rule, the waves
// taking a share of the monomials each; the four products per token (C += S^T V, O = Qm C,
// X = dO C^T, ..) are 32x32 MFMA tiles dealt out to the waves, both operands from LDS.  An fp32
// MFMA holds the matrix pipe 64 cycles for 512 bytes of operands, a sixteenth of what LDS delivers in
// that time (a quarter with all four SIMDs at it), so plain LDS operands keep the pipe fed without
// register blocking.
#include <algorithm>

#include "hla_f32_common.h"
#include "hla_runs.h"

namespace hla {
namespace {

using namespace f32;
using mf::static_for;

// four floats on a 4-byte address: a state is nm (d + 1) floats, and they follow each other without gaps
typedef float f32x4_dw __attribute__((ext_vector_type(4), aligned(4)));

// ---- forms --------------------------------------------------------------------------------------
// The paper's two forms with everything about their monomials known at compile time, and the
// run-time form (tables below) for every other (F, d_phi).
template <int F_, int DP_>
struct Form {
  static constexpr bool kRt = false;
  static constexpr int F = F_, DP = DP_;
  static constexpr int NM = F == 3 ? mf::sym3_num_mono(DP) : mf::sym2_num_mono(DP);
  static constexpr int MPB = (NM + 31) / 32;
  static constexpr int TOK = 64;
};
struct FormRt {
  static constexpr bool kRt = true;
  static constexpr int F = 0, DP = 0, NM = 0;
  static constexpr int MPB = 8;    // most row blocks (d_phi^F <= 256); a call uses ceil(nm / 32)
  static constexpr int TOK = 32;   // two [256][TOK] monomial tiles have to fit LDS
};

// Run-time description of the monomials; entry Di of the outer product has digits in bytes 0..F-1
// of dig[Di] (slot 0 slowest) and belongs to monomial cls[Di]; list holds the entries sorted by
// monomial, monomial m's from start[m] to start[m + 1].
struct MonoTable {
  uint32_t dig[256];
  uint32_t cls[256];
  uint32_t list[256];
  uint32_t start[260];
};

struct F32Geom {
  int64_t stride;   // floats of one state: [nm][d] rows, then z [nm]
  int nm, mpb;      // monomials, row blocks
  int F, dphi, D;   // D = d_phi^F
  int io_bf16;      // caller's tensors are bf16 (else fp32)
  int vec;          // bit i: rows of view i can be read and written 16 bytes at a time
  const MonoTable* tab;
};

// columns [off, off + n) of the feature rows of TOK consecutive token-heads, LDS row stride ld
template <int TOK, int THREADS>
__device__ __forceinline__ void stage_features(const float* __restrict__ feat, int64_t th0, int nfeat, int off,
                                               int n, int nt, int ld, float* fs) {
  for (int idx = threadIdx.x; idx < TOK * n; idx += THREADS) {
    const int t = idx / n, a = idx % n;
    fs[t * ld + a] = t < nt ? feat[(th0 + t) * nfeat + off + a] : 0.0f;
  }
}

// compile-time split of the monomials over W waves: f(integral_constant<part>) on the wave's own part
template <int W, class Fn>
__device__ __forceinline__ void on_part(int wave, Fn&& f) {
  static_for<0, W>([&](auto I) {
    if (wave == decltype(I)::value) f(I);
  });
}
template <class FM, int W>
struct Part {
  static constexpr int MQ = (FM::NM + W - 1) / W;
};

template <class FM, int M>
__device__ __forceinline__ float query_mono(const float (&q)[FM::DP]) {
  if constexpr (FM::F == 3) {
    constexpr mf::Tri t = mf::sym3_mono(FM::DP, M);
    return (q[t.x] * q[t.y]) * q[t.z];
  } else {
    constexpr mf::Duo t = mf::sym2_mono(FM::DP, M);
    return q[t.x] * q[t.y];
  }
}
template <class FM, int M>
__device__ __forceinline__ void query_mono_grad(const float (&q)[FM::DP], float dm, float (&dq)[FM::DP]) {
  if constexpr (FM::F == 3) {
    constexpr mf::Tri t = mf::sym3_mono(FM::DP, M);
    dq[t.x] += dm * (q[t.y] * q[t.z]);
    dq[t.y] += dm * (q[t.x] * q[t.z]);
    dq[t.z] += dm * (q[t.x] * q[t.y]);
  } else {
    constexpr mf::Duo t = mf::sym2_mono(FM::DP, M);
    dq[t.x] += dm * q[t.y];
    dq[t.y] += dm * q[t.x];
  }
}
template <class FM, int M>
__device__ __forceinline__ float key_mono(const float (&k)[FM::F][FM::DP]) {
  if constexpr (FM::F == 3) {
    constexpr mf::Tri t = mf::sym3_mono(FM::DP, M);
    return mf::key_monomial<FM::DP, t.x, t.y, t.z>(k[0], k[1], k[2]);
  } else {
    constexpr mf::Duo t = mf::sym2_mono(FM::DP, M);
    if constexpr (t.x == t.y) return k[0][t.x] * k[1][t.x];
    return k[0][t.x] * k[1][t.y] + k[0][t.y] * k[1][t.x];
  }
}
template <class FM, int M>
__device__ __forceinline__ void key_mono_grad(const float (&k)[FM::F][FM::DP], float ds,
                                              float (&dk)[FM::F][FM::DP]) {
  if constexpr (FM::F == 3) {
    constexpr mf::Tri t = mf::sym3_mono(FM::DP, M);
    constexpr mf::Perm3 p = mf::sym3_perms(t);
    static_for<0, p.n>([&](auto E) {
      constexpr int e = decltype(E)::value;
      dk[0][p.a[e]] += ds * (k[1][p.b[e]] * k[2][p.c[e]]);
      dk[1][p.b[e]] += ds * (k[0][p.a[e]] * k[2][p.c[e]]);
      dk[2][p.c[e]] += ds * (k[0][p.a[e]] * k[1][p.b[e]]);
    });
  } else {
    constexpr mf::Duo t = mf::sym2_mono(FM::DP, M);
    dk[0][t.x] += ds * k[1][t.y];
    dk[1][t.y] += ds * k[0][t.x];
    if constexpr (t.x != t.y) {
      dk[0][t.y] += ds * k[1][t.x];
      dk[1][t.x] += ds * k[0][t.y];
    }
  }
}

// Monomials of a tile into mt[m][LT] (lane = token), times a per-token factor for the query side.
// QUERY: fs holds phi_q rows; else phi_k1 .. phi_kF one after the other.
template <class FM, bool QUERY, int W, int LT>
__device__ __forceinline__ void tile_monomials(const F32Geom& x, const float* fs, int ld, int wave, int lane,
                                               float scale, float* mt) {
  if constexpr (!FM::kRt) {
    constexpr int MQ = Part<FM, W>::MQ, NM = FM::NM;
    if constexpr (QUERY) {
      float q[FM::DP];
#pragma unroll
      for (int a = 0; a < FM::DP; ++a) q[a] = fs[lane * ld + a];
      on_part<W>(wave, [&](auto I) {
        constexpr int p = decltype(I)::value;
        static_for<p * MQ, (p * MQ + MQ < NM ? p * MQ + MQ : NM)>([&](auto M) {
          constexpr int m = decltype(M)::value;
          mt[m * LT + lane] = query_mono<FM, m>(q) * scale;
        });
      });
    } else {
      float k[FM::F][FM::DP];
#pragma unroll
      for (int f = 0; f < FM::F; ++f)
#pragma unroll
        for (int a = 0; a < FM::DP; ++a) k[f][a] = fs[lane * ld + f * FM::DP + a];
      on_part<W>(wave, [&](auto I) {
        constexpr int p = decltype(I)::value;
        static_for<p * MQ, (p * MQ + MQ < NM ? p * MQ + MQ : NM)>([&](auto M) {
          constexpr int m = decltype(M)::value;
          mt[m * LT + lane] = key_mono<FM, m>(k);
        });
      });
    }
  } else {
    const int t = lane % 32, part = wave * 2 + lane / 32;
    for (int m = part; m < x.nm; m += 2 * W) {
      float v = 0.0f;
      const int e0 = x.tab->start[m], e1 = QUERY ? e0 + 1 : static_cast<int>(x.tab->start[m + 1]);
      for (int e = e0; e < e1; ++e) {
        uint32_t dg = x.tab->dig[x.tab->list[e]];
        float p = 1.0f;
        for (int s = 0; s < x.F; ++s, dg >>= 8) p *= fs[t * ld + (QUERY ? 0 : s * x.dphi) + (dg & 255u)];
        v += p;
      }
      mt[m * LT + t] = v * scale;
    }
  }
}

// acc[i] += A^T B over a tile's tokens for the wave's (32 monomial, 32 channel) tiles: A = mt[m][token],
// B = rows[token][c].  Tile number = cb * mpb + mb, dealt out round robin.
template <class FM, int D, int W, int LT, int TPW>
__device__ __forceinline__ void accumulate_state(int mpb, const float* mt, const float* rows, int wave, int lane,
                                                 f32x16 (&acc)[TPW]) {
  constexpr int LD = D + 4, TOK = FM::TOK;
  const int r = lane % 32, hf = lane / 32;
#pragma unroll
  for (int i = 0; i < TPW; ++i) {
    const int tile = wave + W * i;
    if (tile < mpb * (D / 32)) {
      const int mb = tile % mpb, cb = tile / mpb;
      const float* ap = mt + (32 * mb + r) * LT + (TOK / 2) * hf;
      const float* bp = rows + (TOK / 2) * hf * LD + 32 * cb + r;
#pragma unroll
      for (int k4 = 0; k4 < TOK / 8; ++k4) {  // tokens (TOK / 2) hf + 4 k4 + 0..3
        const f32x4 a = *reinterpret_cast<const f32x4*>(ap + 4 * k4);
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i] = mfma32(a[j], bp[(4 * k4 + j) * LD], acc[i]);
      }
    }
  }
}

// out[m][t] = sum_c C[m][c] rows[t][c] into xt[m][LT] (rows of C from LDS or, run-time form, from memory:
// the last one stands in for those past it, whose products nobody reads)
template <class FM, int D, int W, int LT>
__device__ __forceinline__ void rows_times_state(int nm, int mpb, const float* C, const float* rows, int wave, int lane,
                                                 float* xt) {
  constexpr int LD = D + 4, TB = FM::TOK / 32, LC = FM::kRt ? D : LD;
  constexpr int TPW = (FM::MPB * TB + W - 1) / W;
  const int r = lane % 32, hf = lane / 32;
#pragma unroll
  for (int i = 0; i < TPW; ++i) {
    const int tile = wave + W * i;
    if (tile < mpb * TB) {
      const int mb = tile % mpb, tb = tile / mpb;
      const int row = FM::kRt ? min(32 * mb + r, nm - 1) : 32 * mb + r;
      const float* ap = C + static_cast<int64_t>(row) * LC + (D / 2) * hf;
      const float* bp = rows + (32 * tb + r) * LD + (D / 2) * hf;
      f32x16 acc = zero16();
#pragma unroll
      for (int k4 = 0; k4 < D / 8; ++k4) {
        const f32x4 a = *reinterpret_cast<const std::conditional_t<FM::kRt, f32x4_dw, f32x4>*>(ap + 4 * k4);
        const f32x4 b = *reinterpret_cast<const f32x4*>(bp + 4 * k4);
#pragma unroll
        for (int j = 0; j < 4; ++j) acc = mfma32(a[j], b[j], acc);
      }
#pragma unroll
      for (int j = 0; j < 16; ++j) xt[(32 * mb + mf::d_row(j, hf)) * LT + 32 * tb + r] = acc[j];
    }
  }
}

// rows of out[t][c] = sum_m mt[m][t] C[m][c], divided by dn[t] when dn != nullptr, to the caller's view
template <class FM, int D, int W, int LT>
__device__ __forceinline__ void monomials_times_state(const F32Geom& x, const float* C, const float* mt,
                                                      const float* dn, int wave, int lane, const View& Out, int b,
                                                      int h, int t0, int nt) {
  constexpr int LD = D + 4, TB = FM::TOK / 32, NT = TB * (D / 32), LC = FM::kRt ? D : LD;
  constexpr int TPW = (NT + W - 1) / W;
  const int r = lane % 32, hf = lane / 32;
#pragma unroll
  for (int i = 0; i < TPW; ++i) {
    const int tile = wave + W * i;
    if (tile < NT) {
      const int tb = tile % TB, cb = tile / TB;
      const float* ap = mt + hf * LT + 32 * tb + r;
      const float* bp = C + hf * LC + 32 * cb + r;
      f32x16 acc = zero16();
      if constexpr (!FM::kRt) {
        static_assert(FM::NM % 2 == 0, "whole k-steps");
#pragma unroll 8
        for (int s = 0; s < FM::NM / 2; ++s) acc = mfma32(ap[2 * s * LT], bp[2 * s * LC], acc);
      } else {
        const int steps = (x.nm + 1) / 2;  // row nm of an odd form: zero in mt, masked in C
        for (int s = 0; s < steps; ++s) {
          const float bv = 2 * s + hf < x.nm ? bp[static_cast<int64_t>(2 * s) * LC] : 0.0f;
          acc = mfma32(ap[2 * s * LT], bv, acc);
        }
      }
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        const int t = 32 * tb + mf::d_row(j, hf);
        if (t < nt) {
          const float v = dn != nullptr ? acc[j] / dn[t] : acc[j];
          if (x.io_bf16)
            Out.row<bf16_t>(b, h, t0 + t)[32 * cb + r] = from_float<bf16_t>(v);
          else
            Out.row<float>(b, h, t0 + t)[32 * cb + r] = v;
        }
      }
    }
  }
}

// a state's rows into LDS (row stride D + 4); the run-time form reads them from memory instead
template <class FM, int D, int THREADS>
__device__ __forceinline__ void stage_state(const float* __restrict__ st, float* cs) {
  constexpr int P = D / 4;
  for (int i = threadIdx.x; i < FM::NM * P; i += THREADS)
    *reinterpret_cast<f32x4*>(cs + (i / P) * (D + 4) + 4 * (i % P)) = *reinterpret_cast<const f32x4_dw*>(st + 4 * i);
}

template <class FM, int D>
struct Cfg {
  static constexpr int TOK = FM::TOK;
  // the tiles of the three-factor form at d = 128 fill LDS with one workgroup: eight waves there
  static constexpr int W = !FM::kRt && FM::F == 3 && D == 128 ? 8 : 4;
  static constexpr int THREADS = W * 64;
  static constexpr int LD = D + 4, LT = TOK + 4;
  static constexpr int TPW = (FM::MPB * (D / 32) + W - 1) / W;  // state tiles per wave
  static constexpr int NZ = (FM::MPB * 32 + 63) / 64;            // z entries per thread
};

// z entries: thread (m % 64, part of the tile's tokens), summed over the W parts at the end
template <class FM, int D>
__device__ __forceinline__ void accumulate_z(int rows, const float* mt, const float* weight, float (&z)[Cfg<FM, D>::NZ]) {
  using CF = Cfg<FM, D>;
  constexpr int per = CF::TOK / CF::W;
  const int t0 = (threadIdx.x / 64) * per;
#pragma unroll
  for (int i = 0; i < CF::NZ; ++i) {
    const int m = threadIdx.x % 64 + 64 * i;
    if (m < rows) {
#pragma unroll
      for (int t = 0; t < per; t += 4) {
        const f32x4 v = *reinterpret_cast<const f32x4*>(mt + m * CF::LT + t0 + t);
#pragma unroll
        for (int j = 0; j < 4; ++j) z[i] += weight != nullptr ? v[j] * weight[t0 + t + j] : v[j];
      }
    }
  }
}
// accumulators and z to one partial state ([nm][D], then z [nm]); red: W * 64 * NZ floats of LDS
template <class FM, int D>
__device__ __forceinline__ void store_partial(int nm, int mpb, const f32x16 (&acc)[Cfg<FM, D>::TPW],
                                              const float (&z)[Cfg<FM, D>::NZ], float* red, float* __restrict__ out) {
  using CF = Cfg<FM, D>;
  const int lane = threadIdx.x % 64, wave = mf::wave_index();
  const int r = lane % 32, hf = lane / 32;
#pragma unroll
  for (int i = 0; i < CF::TPW; ++i) {
    const int tile = wave + CF::W * i;
    if (tile < mpb * (D / 32)) {
      const int mb = tile % mpb, cb = tile / mpb;
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        const int m = 32 * mb + mf::d_row(j, hf);
        if (m < nm) out[m * D + 32 * cb + r] = acc[i][j];
      }
    }
  }
#pragma unroll
  for (int i = 0; i < CF::NZ; ++i) red[(wave * CF::NZ + i) * 64 + lane] = z[i];
  __syncthreads();
  for (int m = threadIdx.x; m < nm; m += CF::THREADS) {
    float s = 0.0f;
#pragma unroll
    for (int w = 0; w < CF::W; ++w) s += red[(w * CF::NZ + m / 64) * 64 + m % 64];
    out[nm * D + m] = s;
  }
}

// ---- LDS layouts (floats) -------------------------------------------------------------------------
template <class FM, int D>
struct Lds {
  using CF = Cfg<FM, D>;
  static constexpr int kRows = CF::TOK * CF::LD;
  __host__ __device__ static int mono(int mpb) { return 32 * mpb * CF::LT; }
  __host__ __device__ static int feats(int n) { return (CF::TOK * (n | 1) + 3) / 4 * 4; }
  static constexpr int kState = FM::kRt ? 0 : FM::NM * CF::LD;
  // rows of C past the last monomial are read as padding rows of an operand: keep them inside LDS
  static constexpr int kStatePad = FM::kRt ? 0 : 32 * FM::MPB * CF::LD;
  // partial feature gradients of the waves (compile-time forms): may overlay the X tile
  __host__ __device__ static int parts(int nout) { return FM::kRt ? 0 : CF::W * nout * (CF::TOK + 1); }
  __host__ __device__ static int xreg(int mpb, int nout) { return mono(mpb) > parts(nout) ? mono(mpb) : (parts(nout) + 3) / 4 * 4; }
  static constexpr int kRed = CF::W * 64 * (CF::NZ > 1 ? CF::NZ : 1);
  __host__ static size_t state_bytes(const F32Geom& x) {
    return 4u * (kRows + mono(x.mpb) + feats(x.F * x.dphi) + kRed);
  }
  __host__ static size_t query_bytes(const F32Geom& x) {
    return 4u * (kState + mono(x.mpb) + feats(x.dphi) + 2 * CF::THREADS + CF::TOK);
  }
  __host__ static size_t bwd_query_bytes(const F32Geom& x) {
    return 4u * (kStatePad + kRows + mono(x.mpb) + xreg(x.mpb, x.dphi) + feats(x.dphi) + 2 * CF::THREADS +
                 2 * CF::TOK + kRed);
  }
  __host__ static size_t bwd_key_bytes(const F32Geom& x) {
    return 4u * (kStatePad + kRows + mono(x.mpb) + xreg(x.mpb, x.F * x.dphi) + feats(x.F * x.dphi));
  }
};

// ---- key-side state: partial C, z of a run of tokens -----------------------------------------------
// grid (runs, H).
template <class FM, int D>
__global__ __launch_bounds__((Cfg<FM, D>::THREADS)) void k_f32_state(Geom g, F32Geom x, const BlockEnt* __restrict__ runs,
                                                                  const float* __restrict__ feat, View V,
                                                                  float* __restrict__ partial) {
  using CF = Cfg<FM, D>;
  using L = Lds<FM, D>;
  extern __shared__ __align__(16) float sm[];
  const int nm = FM::kRt ? x.nm : FM::NM, mpb = FM::kRt ? x.mpb : FM::MPB;
  const int nk = FM::kRt ? x.F * x.dphi : FM::F * FM::DP, dp = FM::kRt ? x.dphi : FM::DP;
  float* vs = sm;
  float* mt = vs + L::kRows;
  float* fs = mt + L::mono(mpb);
  float* red = fs + L::feats(nk);
  const BlockEnt e = runs[blockIdx.x];
  const int h = blockIdx.y, lane = threadIdx.x % 64, wave = mf::wave_index();
  f32x16 acc[CF::TPW];
  float z[CF::NZ];
#pragma unroll
  for (int i = 0; i < CF::TPW; ++i) acc[i] = zero16();
#pragma unroll
  for (int i = 0; i < CF::NZ; ++i) z[i] = 0.0f;
  for (int t0 = e.t0; t0 < e.t1; t0 += CF::TOK) {
    const int nt = min(CF::TOK, e.t1 - t0);
    stage_rows<D, CF::TOK, CF::THREADS, CF::LD>(V, e.b, h, t0, nt, x.io_bf16, x.vec & 1, vs);
    stage_features<CF::TOK, CF::THREADS>(feat, g.th(e.b, h, t0), g.nfeat, dp, nk, nt, nk | 1, fs);
    __syncthreads();
    tile_monomials<FM, false, CF::W, CF::LT>(x, fs, nk | 1, wave, lane, 1.0f, mt);
    __syncthreads();
    accumulate_state<FM, D, CF::W, CF::LT, CF::TPW>(mpb, mt, vs, wave, lane, acc);
    accumulate_z<FM, D>(nm, mt, nullptr, z);
    __syncthreads();
  }
  store_partial<FM, D>(nm, mpb, acc, z, red,
                       partial + (static_cast<int64_t>(blockIdx.x) * g.H + h) * x.stride);
}

// ---- sum of the partial states of each (sequence, head), in a fixed order ------------------------------
// grid (num_seqs, H, ceil(stride / 64)), block 256: four slices of the runs per element, sixteen loads in
// flight each (a run's load next to its addition would cost a memory round trip per run).
__global__ __launch_bounds__(256) void k_f32_reduce(int H, const int32_t* __restrict__ seq_off,
                                                    const float* __restrict__ partial, float* __restrict__ state,
                                                    int64_t stride) {
  const int s = blockIdx.x, h = blockIdx.y;
  const int c0 = seq_off[s], c1 = seq_off[s + 1];
  const int64_t step = H * stride;
  const float* src = partial + (static_cast<int64_t>(c0) * H + h) * stride;
  float* out = state + (static_cast<int64_t>(s) * H + h) * stride;
  __shared__ float slices[4][64];
  const int slice = threadIdx.x / 64;
  const int64_t i = static_cast<int64_t>(blockIdx.z) * 64 + threadIdx.x % 64, at = min(i, stride - 1);
  const int per = (c1 - c0 + 3) / 4, r0 = slice * per, r1 = min(r0 + per, c1 - c0);
  float a = 0.0f;
  for (int c = r0; c < r1; c += 16) {
    float v[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) v[u] = src[min(c + u, r1 - 1) * step + at];
#pragma unroll
    for (int u = 0; u < 16; ++u)
      if (c + u < r1) a += v[u];
  }
  slices[slice][threadIdx.x % 64] = a;
  __syncthreads();
  if (slice == 0 && i < stride) out[i] = ((a + slices[1][threadIdx.x]) + slices[2][threadIdx.x]) + slices[3][threadIdx.x];
}

// ---- query side: O = Qm C / (Qm z + eps) ------------------------------------------------------------
template <class FM, int D>
__global__ __launch_bounds__((Cfg<FM, D>::THREADS)) void k_f32_query(Geom g, F32Geom x, const BlockEnt* __restrict__ runs,
                                                                  const float* __restrict__ feat,
                                                                  const float* __restrict__ state, View O,
                                                                  float* __restrict__ den) {
  using CF = Cfg<FM, D>;
  using L = Lds<FM, D>;
  extern __shared__ __align__(16) float sm[];
  const int nm = FM::kRt ? x.nm : FM::NM, mpb = FM::kRt ? x.mpb : FM::MPB, dp = FM::kRt ? x.dphi : FM::DP;
  float* cs = sm;
  float* mt = cs + L::kState;
  float* fs = mt + L::mono(mpb);
  float* eparts = fs + L::feats(dp);           // [parts][TOK]
  float* dn = eparts + 2 * CF::THREADS;        // [TOK]
  const BlockEnt e = runs[blockIdx.x];
  const int h = blockIdx.y, lane = threadIdx.x % 64, wave = mf::wave_index();
  const float* st = state + (static_cast<int64_t>(e.seq) * g.H + h) * x.stride;
  const float* zv = st + nm * D;
  if constexpr (!FM::kRt) stage_state<FM, D, CF::THREADS>(st, cs);
  if (FM::kRt && (nm & 1)) {
    if (threadIdx.x < CF::TOK) mt[nm * CF::LT + threadIdx.x] = 0.0f;
  }
  for (int t0 = e.t0; t0 < e.t1; t0 += CF::TOK) {
    const int nt = min(CF::TOK, e.t1 - t0);
    const int64_t th0 = g.th(e.b, h, t0);
    stage_features<CF::TOK, CF::THREADS>(feat, th0, g.nfeat, 0, dp, nt, dp | 1, fs);
    __syncthreads();
    tile_monomials<FM, true, CF::W, CF::LT>(x, fs, dp | 1, wave, lane, 1.0f, mt);
    __syncthreads();
    {  // eta: thread (token, part) over the monomials m = part, part + parts, ..
      constexpr int parts = CF::THREADS / CF::TOK;
      const int t = threadIdx.x % CF::TOK, part = threadIdx.x / CF::TOK;
      float s = 0.0f;
      for (int m = part; m < nm; m += parts) s += mt[m * CF::LT + t] * zv[m];
      eparts[part * CF::TOK + t] = s;
      __syncthreads();
      if (threadIdx.x < CF::TOK) {
        float eta = 0.0f;
#pragma unroll
        for (int p = 0; p < parts; ++p) eta += eparts[p * CF::TOK + t];
        dn[t] = eta + g.eps;
        if (t < nt) den[th0 + t] = eta + g.eps;
      }
    }
    __syncthreads();
    monomials_times_state<FM, D, CF::W, CF::LT>(x, FM::kRt ? st : cs, mt, dn, wave, lane, O, e.b, h, t0, nt);
    __syncthreads();
  }
}

// ---- backward, query side ---------------------------------------------------------------------------
// With inv = 1 / den, Wm = inv Qm, X = C dO:  s = -<dO, o> / den = -inv sum_m Wm X_m (taken from the
// product that feeds dM, so that the component of dM along Qm cancels to rounding),
// dM = inv X + s z, chain rule to d(phi_q); partial dC += Wm (x) dO, dz += Wm (s / inv).
template <class FM, int D>
__global__ __launch_bounds__((Cfg<FM, D>::THREADS)) void k_f32_bwd_query(
    Geom g, F32Geom x, const BlockEnt* __restrict__ runs, const float* __restrict__ feat,
    const float* __restrict__ state, const float* __restrict__ den, View dO, float* __restrict__ dfeat,
    float* __restrict__ partial) {
  using CF = Cfg<FM, D>;
  using L = Lds<FM, D>;
  extern __shared__ __align__(16) float sm[];
  const int nm = FM::kRt ? x.nm : FM::NM, mpb = FM::kRt ? x.mpb : FM::MPB, dp = FM::kRt ? x.dphi : FM::DP;
  constexpr int parts = CF::THREADS / CF::TOK;
  float* cs = sm;
  float* gs = cs + L::kStatePad;               // dO rows
  float* mt = gs + L::kRows;                   // Wm
  float* xt = mt + L::mono(mpb);               // X, then the waves' partial feature gradients
  float* fs = xt + L::xreg(mpb, dp);
  float* sparts = fs + L::feats(dp);           // [parts][TOK]
  float* us = sparts + 2 * CF::THREADS;        // [TOK] s / inv
  float* invs = us + CF::TOK;                  // [TOK]
  float* red = invs + CF::TOK;
  const BlockEnt e = runs[blockIdx.x];
  const int h = blockIdx.y, lane = threadIdx.x % 64, wave = mf::wave_index();
  const float* st = state + (static_cast<int64_t>(e.seq) * g.H + h) * x.stride;
  const float* zv = st + nm * D;
  if constexpr (!FM::kRt) stage_state<FM, D, CF::THREADS>(st, cs);
  f32x16 acc[CF::TPW];
  float z[CF::NZ];
#pragma unroll
  for (int i = 0; i < CF::TPW; ++i) acc[i] = zero16();
#pragma unroll
  for (int i = 0; i < CF::NZ; ++i) z[i] = 0.0f;
  for (int t0 = e.t0; t0 < e.t1; t0 += CF::TOK) {
    const int nt = min(CF::TOK, e.t1 - t0);
    const int64_t th0 = g.th(e.b, h, t0);
    stage_rows<D, CF::TOK, CF::THREADS, CF::LD>(dO, e.b, h, t0, nt, x.io_bf16, x.vec & 1, gs);
    stage_features<CF::TOK, CF::THREADS>(feat, th0, g.nfeat, 0, dp, nt, dp | 1, fs);
    if (threadIdx.x < CF::TOK) invs[threadIdx.x] = static_cast<int>(threadIdx.x) < nt ? 1.0f / den[th0 + threadIdx.x] : 0.0f;
    __syncthreads();
    const float inv = invs[lane % CF::TOK];
    tile_monomials<FM, true, CF::W, CF::LT>(x, fs, dp | 1, wave, lane, inv, mt);
    rows_times_state<FM, D, CF::W, CF::LT>(nm, mpb, FM::kRt ? st : cs, gs, wave, lane, xt);
    __syncthreads();
    {
      const int t = threadIdx.x % CF::TOK, part = threadIdx.x / CF::TOK;
      float s = 0.0f;
      for (int m = part; m < nm; m += parts) s += mt[m * CF::LT + t] * xt[m * CF::LT + t];
      sparts[part * CF::TOK + t] = s;
    }
    __syncthreads();
    float u = 0.0f;
#pragma unroll
    for (int p = 0; p < parts; ++p) u -= sparts[p * CF::TOK + lane % CF::TOK];
    if (threadIdx.x < CF::TOK) us[threadIdx.x] = u;
    const float s = u * inv;
    if constexpr (!FM::kRt) {
      constexpr int MQ = Part<FM, CF::W>::MQ, NM = FM::NM, DP = FM::DP;
      float q[DP], dq[DP];
#pragma unroll
      for (int a = 0; a < DP; ++a) {
        q[a] = fs[lane * (DP | 1) + a];
        dq[a] = 0.0f;
      }
      on_part<CF::W>(wave, [&](auto I) {
        constexpr int p = decltype(I)::value;
        static_for<p * MQ, (p * MQ + MQ < NM ? p * MQ + MQ : NM)>([&](auto M) {
          constexpr int m = decltype(M)::value;
          query_mono_grad<FM, m>(q, inv * xt[m * CF::LT + lane] + s * zv[m], dq);
        });
      });
      __syncthreads();  // X has been read: its place takes the partial gradients; us is visible
#pragma unroll
      for (int a = 0; a < DP; ++a) xt[(wave * DP + a) * (CF::TOK + 1) + lane] = dq[a];
    } else {
      // dM over the orderings of its monomial, in place; then one output per (token, part) at a time
      const int t = threadIdx.x % CF::TOK, part = threadIdx.x / CF::TOK;
      for (int m = part; m < nm; m += parts)
        xt[m * CF::LT + t] = (inv * xt[m * CF::LT + t] + s * zv[m]) / static_cast<float>(x.tab->start[m + 1] - x.tab->start[m]);
      __syncthreads();
      const int lo_n = x.D / dp;
      for (int a = part; a < dp; a += parts) {
        float gsum = 0.0f;
        for (int lo = 0; lo < lo_n; ++lo) {
          const int Di = a * lo_n + lo;
          uint32_t dg = x.tab->dig[Di] >> 8;
          float p = xt[x.tab->cls[Di] * CF::LT + t];
          for (int sl = 1; sl < x.F; ++sl, dg >>= 8) p *= fs[t * (dp | 1) + (dg & 255u)];
          gsum += p;
        }
        if (t < nt) dfeat[(th0 + t) * g.nfeat + a] = static_cast<float>(x.F) * gsum;
      }
    }
    accumulate_state<FM, D, CF::W, CF::LT, CF::TPW>(mpb, mt, gs, wave, lane, acc);
    accumulate_z<FM, D>(nm, mt, us, z);
    __syncthreads();
    if constexpr (!FM::kRt) {
      constexpr int DP = FM::DP;
      for (int i = threadIdx.x; i < CF::TOK * DP; i += CF::THREADS) {
        const int t = i / DP, a = i % DP;
        float v = 0.0f;
#pragma unroll
        for (int p = 0; p < CF::W; ++p) v += xt[(p * DP + a) * (CF::TOK + 1) + t];
        if (t < nt) dfeat[(th0 + t) * g.nfeat + a] = v;
      }
      __syncthreads();
    }
  }
  store_partial<FM, D>(nm, mpb, acc, z, red,
                       partial + (static_cast<int64_t>(blockIdx.x) * g.H + h) * x.stride);
}

// ---- backward, key side: dS = dC v + dz, dV = dC^T S, chain rule to d(phi_kf) -----------------------
template <class FM, int D>
__global__ __launch_bounds__((Cfg<FM, D>::THREADS)) void k_f32_bwd_key(Geom g, F32Geom x, const BlockEnt* __restrict__ runs,
                                                                    const float* __restrict__ feat,
                                                                    const float* __restrict__ dstate, View V,
                                                                    View dV, float* __restrict__ dfeat) {
  using CF = Cfg<FM, D>;
  using L = Lds<FM, D>;
  extern __shared__ __align__(16) float sm[];
  const int nm = FM::kRt ? x.nm : FM::NM, mpb = FM::kRt ? x.mpb : FM::MPB, dp = FM::kRt ? x.dphi : FM::DP;
  const int nk = FM::kRt ? x.F * x.dphi : FM::F * FM::DP;
  float* cs = sm;
  float* vs = cs + L::kStatePad;
  float* mt = vs + L::kRows;
  float* xt = mt + L::mono(mpb);
  float* fs = xt + L::xreg(mpb, nk);
  const BlockEnt e = runs[blockIdx.x];
  const int h = blockIdx.y, lane = threadIdx.x % 64, wave = mf::wave_index();
  const float* st = dstate + (static_cast<int64_t>(e.seq) * g.H + h) * x.stride;
  const float* zv = st + nm * D;
  if constexpr (!FM::kRt) stage_state<FM, D, CF::THREADS>(st, cs);
  if (FM::kRt && (nm & 1)) {
    if (threadIdx.x < CF::TOK) mt[nm * CF::LT + threadIdx.x] = 0.0f;
  }
  for (int t0 = e.t0; t0 < e.t1; t0 += CF::TOK) {
    const int nt = min(CF::TOK, e.t1 - t0);
    const int64_t th0 = g.th(e.b, h, t0);
    stage_rows<D, CF::TOK, CF::THREADS, CF::LD>(V, e.b, h, t0, nt, x.io_bf16, x.vec & 1, vs);
    stage_features<CF::TOK, CF::THREADS>(feat, th0, g.nfeat, dp, nk, nt, nk | 1, fs);
    __syncthreads();
    tile_monomials<FM, false, CF::W, CF::LT>(x, fs, nk | 1, wave, lane, 1.0f, mt);
    rows_times_state<FM, D, CF::W, CF::LT>(nm, mpb, FM::kRt ? st : cs, vs, wave, lane, xt);
    __syncthreads();
    if constexpr (!FM::kRt) {
      constexpr int MQ = Part<FM, CF::W>::MQ, NM = FM::NM, DP = FM::DP, F = FM::F;
      float k[F][DP], dk[F][DP];
#pragma unroll
      for (int f = 0; f < F; ++f)
#pragma unroll
        for (int a = 0; a < DP; ++a) {
          k[f][a] = fs[lane * ((F * DP) | 1) + f * DP + a];
          dk[f][a] = 0.0f;
        }
      on_part<CF::W>(wave, [&](auto I) {
        constexpr int p = decltype(I)::value;
        static_for<p * MQ, (p * MQ + MQ < NM ? p * MQ + MQ : NM)>([&](auto M) {
          constexpr int m = decltype(M)::value;
          key_mono_grad<FM, m>(k, xt[m * CF::LT + lane] + zv[m], dk);
        });
      });
      __syncthreads();
#pragma unroll
      for (int f = 0; f < F; ++f)
#pragma unroll
        for (int a = 0; a < DP; ++a) xt[(wave * F * DP + f * DP + a) * (CF::TOK + 1) + lane] = dk[f][a];
    } else {
      constexpr int parts = CF::THREADS / CF::TOK;
      const int t = threadIdx.x % CF::TOK, part = threadIdx.x / CF::TOK;
      for (int m = part; m < nm; m += parts) xt[m * CF::LT + t] += zv[m];
      __syncthreads();
      for (int o = part; o < nk; o += parts) {
        const int f = o / dp, a = o % dp;
        int lo_n = 1;
        for (int s = f + 1; s < x.F; ++s) lo_n *= dp;
        const int hi_n = x.D / (dp * lo_n);
        float gsum = 0.0f;
        for (int hi = 0; hi < hi_n; ++hi)
          for (int lo = 0; lo < lo_n; ++lo) {
            const int Di = (hi * dp + a) * lo_n + lo;
            const uint32_t dg = x.tab->dig[Di];
            float p = xt[x.tab->cls[Di] * CF::LT + t];
            for (int sl = 0; sl < x.F; ++sl)
              if (sl != f) p *= fs[t * (nk | 1) + sl * dp + ((dg >> (8 * sl)) & 255u)];
            gsum += p;
          }
        if (t < nt) dfeat[(th0 + t) * g.nfeat + dp + o] = gsum;
      }
    }
    monomials_times_state<FM, D, CF::W, CF::LT>(x, FM::kRt ? st : cs, mt, nullptr, wave, lane, dV, e.b, h, t0, nt);
    __syncthreads();
    if constexpr (!FM::kRt) {
      constexpr int NK = FM::F * FM::DP;
      for (int i = threadIdx.x; i < CF::TOK * NK; i += CF::THREADS) {
        const int t = i / NK, a = i % NK;
        float v = 0.0f;
#pragma unroll
        for (int p = 0; p < CF::W; ++p) v += xt[(p * NK + a) * (CF::TOK + 1) + t];
        if (t < nt) dfeat[(th0 + t) * g.nfeat + FM::DP + a] = v;
      }
      __syncthreads();
    }
  }
}

// ---- host ---------------------------------------------------------------------------------------------
int64_t binomial(int n, int k) {
  int64_t r = 1;
  for (int i = 1; i <= k; ++i) r = r * (n - k + i) / i;
  return r;
}

F32Geom f32_geom(const hla_handle* hd) {
  F32Geom x{};
  x.F = hd->g.F;
  x.dphi = hd->g.dphi;
  x.D = hd->g.D;
  x.nm = static_cast<int>(binomial(x.dphi + x.F - 1, x.F));
  x.mpb = (x.nm + 31) / 32;
  x.stride = static_cast<int64_t>(x.nm) * (hd->g.d + 1);
  x.io_bf16 = hd->cfg.io_dtype == HLA_BF16;
  x.tab = static_cast<const MonoTable*>(hd->path_ws);
  return x;
}

bool is_form(const hla_handle* hd, int F, int dphi) { return hd->g.F == F && hd->g.dphi == dphi; }
bool is_rt(const hla_handle* hd) { return !is_form(hd, 3, 6) && !is_form(hd, 2, 12); }
int tok_of(const hla_handle* hd) { return is_rt(hd) ? FormRt::TOK : 64; }

// Runs of tokens per (sequence, head): enough workgroups for two per compute unit, never more
// partial states than the workspace holds (but at least one run per sequence).
int64_t max_partials(const hla_handle* hd) {
  // 504 workgroups for the three-factor form at d = 64, 254 (of eight waves) at d = 128: 8 MiB of partial
  // states with their rows counted in whole tiles; more would only add to what the reduction reads
  const int64_t fit = (8ll << 20) / (static_cast<int64_t>(128) * f32_geom(hd).mpb * (hd->g.d + 1));
  return std::min<int64_t>(512, std::max<int64_t>(fit, 16));
}

template <class FM, int D>
hla_status allow_lds(const F32Geom& x) {
  using L = Lds<FM, D>;
  struct {
    const void* k;
    size_t bytes;
  } ks[4] = {{reinterpret_cast<const void*>(&k_f32_state<FM, D>), L::state_bytes(x)},
             {reinterpret_cast<const void*>(&k_f32_query<FM, D>), L::query_bytes(x)},
             {reinterpret_cast<const void*>(&k_f32_bwd_query<FM, D>), L::bwd_query_bytes(x)},
             {reinterpret_cast<const void*>(&k_f32_bwd_key<FM, D>), L::bwd_key_bytes(x)}};
  for (const auto& k : ks) {
    if (k.bytes > 160 * 1024) return HLA_ERR_UNSUPPORTED;
    if (k.bytes > 64 * 1024 &&
        hipFuncSetAttribute(k.k, hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(k.bytes)) != hipSuccess)
      return HLA_ERR_HIP;
  }
  return HLA_OK;
}

hla_status runs_table(hla_handle* hd, const hla_call_args& a, hla_token_table** out) {
  // the same sequences and heads as the last call's (its backward, the next step): the same runs
  if (hd->tables[0].valid && hd->runs_heads == a.H) return get_table(hd, 0, hd->tables[0].block_tokens, a.stream, out);
  const int tok = tok_of(hd);
  const int64_t cap = max_partials(hd);
  const int nseq = a.num_seqs;
  auto count = [&](int64_t per) {  // runs per head with `per` tiles each
    const int64_t blk = per * tok;
    if (!a.packed) return static_cast<int64_t>(a.B) * ((a.N + blk - 1) / blk);
    int64_t c = 0;
    for (int s = 0; s < nseq; ++s) c += (hd->cu_host[s + 1] - hd->cu_host[s] + blk - 1) / blk;
    return c;
  };
  const int64_t per = tiles_per_run(a.H, nseq, cap, count);
  HLA_TRY(get_table(hd, 0, static_cast<int32_t>(per * tok), a.stream, out));
  hd->runs_heads = a.H;
  return HLA_OK;
}

hla_status reduce_partials(hla_handle* hd, const hla_call_args& a, const F32Geom& x, const hla_token_table* runs,
                           const char* name, float* out) {
  const unsigned slices = static_cast<unsigned>((x.stride + 63) / 64);
  return launch(hd, name, k_f32_reduce, dim3(a.num_seqs, a.H, slices), dim3(256), 0, a.stream, a.H,
                runs->seq_off_dev, static_cast<const float*>(hd->partial), out, x.stride);
}

template <class FM, int D>
hla_status forward_fd(hla_handle* hd, const hla_call_args& a) {
  using CF = Cfg<FM, D>;
  using L = Lds<FM, D>;
  const Geom& g = hd->g;
  F32Geom x = f32_geom(hd);
  hla_token_table* runs = nullptr;
  HLA_TRY(runs_table(hd, a, &runs));
  const dim3 grid(runs->count, a.H);
  x.vec = rows_vec(a.V, x.io_bf16 ? 2 : 4);
  HLA_TRY(launch(hd, "generic_state", &k_f32_state<FM, D>, grid, dim3(CF::THREADS), L::state_bytes(x), a.stream, g, x,
                 runs->dev, static_cast<const float*>(hd->feat), a.V, hd->partial));
  HLA_TRY(reduce_partials(hd, a, x, runs, "generic_state_reduce", hd->state));
  return launch(hd, "generic_query", &k_f32_query<FM, D>, grid, dim3(CF::THREADS), L::query_bytes(x), a.stream, g, x,
                runs->dev, static_cast<const float*>(hd->feat), static_cast<const float*>(hd->state), a.O, hd->den);
}

template <class FM, int D>
hla_status backward_fd(hla_handle* hd, const hla_call_args& a) {
  using CF = Cfg<FM, D>;
  using L = Lds<FM, D>;
  const Geom& g = hd->g;
  F32Geom x = f32_geom(hd);
  hla_token_table* runs = nullptr;
  HLA_TRY(runs_table(hd, a, &runs));
  const dim3 grid(runs->count, a.H);
  const size_t elem = x.io_bf16 ? 2 : 4;
  x.vec = rows_vec(a.dO, elem);
  HLA_TRY(launch(hd, "generic_bwd_query", &k_f32_bwd_query<FM, D>, grid, dim3(CF::THREADS), L::bwd_query_bytes(x),
                 a.stream, g, x, runs->dev, static_cast<const float*>(hd->feat), static_cast<const float*>(hd->state),
                 static_cast<const float*>(hd->den), a.dO, hd->dfeat, hd->partial));
  HLA_TRY(reduce_partials(hd, a, x, runs, "generic_dstate_reduce", hd->dstate));
  x.vec = rows_vec(a.V, elem);
  return launch(hd, "generic_bwd_key", &k_f32_bwd_key<FM, D>, grid, dim3(CF::THREADS), L::bwd_key_bytes(x), a.stream, g,
                x, runs->dev, static_cast<const float*>(hd->feat), static_cast<const float*>(hd->dstate), a.V, a.dV,
                hd->dfeat);
}

// run fn<FM, D> for the handle's form and head dim
#define HLA_F32_DISPATCH(fn, ...)                                            \
  do {                                                                       \
    if (is_form(hd, 3, 6)) {                                                 \
      switch (hd->g.d) {                                                     \
        case 32: return fn<Form<3, 6>, 32>(__VA_ARGS__);                     \
        case 64: return fn<Form<3, 6>, 64>(__VA_ARGS__);                     \
        case 128: return fn<Form<3, 6>, 128>(__VA_ARGS__);                   \
      }                                                                      \
    } else if (is_form(hd, 2, 12)) {                                         \
      switch (hd->g.d) {                                                     \
        case 32: return fn<Form<2, 12>, 32>(__VA_ARGS__);                    \
        case 64: return fn<Form<2, 12>, 64>(__VA_ARGS__);                    \
        case 128: return fn<Form<2, 12>, 128>(__VA_ARGS__);                  \
      }                                                                      \
    } else {                                                                 \
      switch (hd->g.d) {                                                     \
        case 32: return fn<FormRt, 32>(__VA_ARGS__);                         \
        case 64: return fn<FormRt, 64>(__VA_ARGS__);                         \
        case 128: return fn<FormRt, 128>(__VA_ARGS__);                       \
      }                                                                      \
    }                                                                        \
    return HLA_ERR_UNSUPPORTED;                                              \
  } while (0)

// the run-time form's tables, built on the device: one workgroup of 256 threads
__global__ __launch_bounds__(256) void k_mono_table(int F, int dphi, int D, MonoTable* __restrict__ tab) {
  __shared__ uint32_t key[256];   // digits sorted: equal for the orderings of one monomial
  __shared__ uint32_t first[256]; // smallest entry with the same key
  const int i = threadIdx.x;
  uint32_t dig = 0, k = 0;
  if (i < D) {
    int v[4], rem = i;
    for (int s = F - 1; s >= 0; --s) {
      v[s] = rem % dphi;
      rem /= dphi;
    }
    for (int s = 0; s < F; ++s) dig |= static_cast<uint32_t>(v[s]) << (8 * s);
    for (int s = 1; s < F; ++s)
      for (int u = s; u > 0 && v[u - 1] > v[u]; --u) {
        const int w = v[u];
        v[u] = v[u - 1];
        v[u - 1] = w;
      }
    for (int s = 0; s < F; ++s) k |= static_cast<uint32_t>(v[s]) << (8 * s);
    key[i] = k;
  }
  __syncthreads();
  if (i < D) {
    int f = 0;
    while (key[f] != k) ++f;
    first[i] = f;
  }
  __syncthreads();
  if (i < D) {
    int cls = 0, pos = 0;
    for (int j = 0; j < D; ++j) {
      const int fj = first[j], fi = first[i];
      if (j < fi && fj == j) ++cls;                        // monomials in front of this one
      if (fj < fi || (fj == fi && j < i)) ++pos;            // entries in front of this one, sorted by monomial
    }
    tab->dig[i] = dig;
    tab->cls[i] = cls;
    tab->list[pos] = i;
    if (static_cast<int>(first[i]) == i) tab->start[cls] = pos;
    if (i == 0) {
      int n = 0;
      for (int j = 0; j < D; ++j) n += static_cast<int>(first[j]) == j;
      tab->start[n] = D;
    }
  }
}

}  // namespace

hla_status f32_workspace_plan(hla_handle* hd) {
  const F32Geom x = f32_geom(hd);
  hd->state_stride = x.stride;
  const int tok = tok_of(hd);
  const hla_config& c = hd->cfg;
  // as many partial states as a call can ask for
  const int64_t most = std::min<int64_t>((c.max_tokens + tok - 1) / tok + c.max_seqs,
                                         std::max<int64_t>((max_partials(hd) + c.max_heads - 1) / c.max_heads, c.max_seqs));
  hd->max_chunks = most;
  hd->tables[0].min_block = tok;
  if (is_rt(hd)) hd->path_ws_bytes = sizeof(MonoTable);
  return HLA_OK;
}

hla_status f32_prepare_kernels(const hla_handle* hd, hipStream_t s) {
  const F32Geom x = f32_geom(hd);
  if (is_rt(hd)) {
    k_mono_table<<<dim3(1), dim3(256), 0, s>>>(x.F, x.dphi, x.D, static_cast<MonoTable*>(hd->path_ws));
    if (hipGetLastError() != hipSuccess) return HLA_ERR_HIP;
  }
  HLA_F32_DISPATCH(allow_lds, x);
}

hla_status f32_forward(hla_handle* hd, const hla_call_args& a) { HLA_F32_DISPATCH(forward_fd, hd, a); }
hla_status f32_backward(hla_handle* hd, const hla_call_args& a) { HLA_F32_DISPATCH(backward_fd, hd, a); }

}  // namespace hla
