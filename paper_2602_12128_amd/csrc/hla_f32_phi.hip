// Feature maps of the generic path (App. A.1: Linear d->d, exact GELU, Linear d->d_phi, ReLU), their
// input gradients and the gradients of their weights on the fp32 matrix cores, fp32 or bf16 I/O.
//
// A workgroup serves 64 tokens of one (batch row, head).  The tile's rows are staged in LDS as fp32;
// hidden^T is never formed: tokens are MFMA rows, hidden units columns, the weights stream from L2 in
// B-operand order (32 consecutive floats per half wave) with the next steps' loads in flight.
//
// At 12 heads x 4095 tokens x 64 channels, three factors, fp32 (us; before: a thread per hidden unit on
// the vector ALU, an LDS read per multiply-add): forward 36 (147), backward with the weight gradients
// 94 (197 + 491 for a second pass that recomputed the hidden layer), of which 11 and 27 are
// matrix-pipe time; the rest is the phases' barriers, GELU and the weights' way from L2.  With erff and
// the weights loaded where they are used, 43 and 100.
#include <algorithm>
#include <cmath>

#include "hla_f32_common.h"

namespace hla {
namespace {

using namespace f32;

constexpr int kTok = 64;
constexpr int kMaxGridX = 1 << 22;  // a grid takes fewer than 2^32 threads in one direction

// Phi(h) of the exact GELU, h Phi(h).  Below |h| = 1 it is 0.5 + h P(h^2), where an error of P shrinks with
// h; beyond, Phi(-t) = 2^-(1 + P(t)) with a degree-8 minimax fit of P(t) = -log2(erfc(t / sqrt 2)) up to 5.9,
// after which P keeps growing and Phi(-t) runs to zero as it should.  Without branches: erff takes
// its two ranges one after the other when the lanes of a wave need both.  Errors against 64 bits on the
// card, h normal with a spread of 0.02, 0.2, 1 and 4 (2-norm, 1e-8; in brackets 0.5 (1 + erff), expf): GELU 3.7,
// 3.7, 3.4, 2.1 (3.7, 3.9, 3.9, 2.3), GELU' 4.1, 3.8, 3.7, 3.6 (4.1, 3.8, 4.0, 3.8); Phi at most 6.9 (7.6).
// The second fit alone, without the first: GELU 5.8, 5.2, 3.5, 2.1, GELU' 5.5, 5.3, 4.2, 3.7.
__device__ __forceinline__ float normal_cdf(float h) {
  constexpr float n[6] = {0.3989423f, -0.06649058f, 0.00997454f, -0.0011890578f, 0.000116174444f, -8.620451e-06f};
  constexpr float c[9] = {1.0f,           1.1511064f,      0.45919567f,     0.052539267f, -0.0071317810f,
                          0.00019325814f, 0.00016142147f, -3.3898614e-05f, 2.3575092e-06f};
  const float t = fabsf(h), s = h * h;
  float near = n[5], p = c[8];
#pragma unroll
  for (int k = 4; k >= 0; --k) near = __builtin_fmaf(near, s, n[k]);
#pragma unroll
  for (int k = 7; k >= 0; --k) p = __builtin_fmaf(p, t, c[k]);
  const float e = __builtin_amdgcn_exp2f(-p);
  const float far = h > 0.0f ? 1.0f - e : e;
  return t < 1.0f ? __builtin_fmaf(h, near, 0.5f) : far;
}

template <int D>
struct PhiCfg {
  static constexpr int NCB = D / 32;                      // column blocks
  static constexpr int NT = 2 * NCB;                      // 32x32 tiles of a [64][D] matrix
  // W waves: tile number wave + W i; row block tile / NCB .. so that a wave of four keeps its column
  // block (and its weight operands) for both row blocks at d = 128
  template <int W>
  static constexpr int tpw() { return (NT + W - 1) / W; }
};
// tile -> (row block, column block): tiles of one column block are NCB apart
template <int D>
__device__ __forceinline__ void tile_pos(int tile, int& rb, int& cb) {
  rb = tile / PhiCfg<D>::NCB;
  cb = tile % PhiCfg<D>::NCB;
}

// use(s, v) for the batches s = 0, NB, .. < STEPS of weight operands that load(s, v) fetches, each batch in
// flight while the one before is used.  Two sets take turns (a copy from one to the other would wait for
// the loads), and the compiler must not move the loads down to where they are used, which it otherwise
// does: d = 128, 4 heads x 3000 tokens with weight gradients, 208 us a step that way, 161 like this.
template <int NB, int STEPS, class Load, class Use>
__device__ __forceinline__ void weight_steps(float (&first)[NB], Load&& load, Use&& use) {
  static_assert(STEPS % (2 * NB) == 0, "pairs of batches");
  float second[NB];
#pragma unroll 1
  for (int s = 0; s < STEPS; s += 2 * NB) {
    load(s + NB, second);
    asm volatile("" ::: "memory");
    use(s, first);
    load(s + 2 * NB < STEPS ? s + 2 * NB : s, first);
    asm volatile("" ::: "memory");
    use(s + NB, second);
  }
}

struct PhiCall {
  Geom g;
  PhiF32 w;
  int bf16, vec_q, vec_k;
  int tpr;    // 64-token tiles per (batch row, head)
  int tiles;  // tiles of a workgroup's list: all (batch row, head) rows, or one head's with per-head weights
};
// tile of the list -> batch row, head, first token
__device__ __forceinline__ void tile_coords(const PhiCall& c, int tile, int head, int& b, int& h, int& t0) {
  const int row = tile / c.tpr;
  t0 = (tile % c.tpr) * kTok;
  b = c.w.heads_w == 1 ? row / c.g.H : row;
  h = c.w.heads_w == 1 ? row % c.g.H : head;
}

// ---- forward ------------------------------------------------------------------------------------
// grid (tiles, 1 or H, 1 + F), block 256; with shared weights and more than kMaxGridX tiles, rows of that
// many workgroups in y.  The sums run in the order of the input channels and of the
// hidden units, one rounding per term: features near zero land on the same side of the ReLU as in
// any other fp32 evaluation in that order.
template <int D>
__global__ __launch_bounds__(256) void k_f32_phi_fwd(PhiCall c, View Q, View K, float* __restrict__ feat) {
  constexpr int W = 4, LD = D + 1, NCB = PhiCfg<D>::NCB, NT = PhiCfg<D>::NT, TPW = PhiCfg<D>::template tpw<W>();
  constexpr int NB = 8;  // k-steps whose weight operands are in flight
  extern __shared__ __align__(16) float sm[];  // [64][LD]: input rows, then GELU(hidden)
  const int lane = threadIdx.x % 64, wave = mf::wave_index();
  const int r = lane % 32, hf = lane / 32;
  const Geom& g = c.g;
  const int m = blockIdx.z, hw = c.w.heads_w == 1 ? 0 : blockIdx.y;
  const int tile = c.w.heads_w == 1 ? blockIdx.y * gridDim.x + blockIdx.x : blockIdx.x;
  if (tile >= c.tiles) return;
  int b, h, t0;
  tile_coords(c, tile, blockIdx.y, b, h, t0);
  const int nt = min(kTok, g.N - t0);
  const int64_t mh = static_cast<int64_t>(m) * c.w.heads_w + hw;
  const float* W1 = c.w.W1 + mh * D * D;
  const float* W2 = c.w.W2 + mh * D * g.dphi;
  int rb0, cb;
  tile_pos<D>(wave, rb0, cb);  // W is a multiple of NCB: a wave's tiles share their column block
  static_assert(W % NCB == 0, "one column block per wave");
  const bool busy = wave < NT;
  // the first weights and the second layer's, up to sixteen features, travel with the tile's rows: a
  // workgroup is one chain of memory round trips, and this makes it one shorter per kind
  const int l16 = lane % 16, q = lane / 16;
  const float* bp = W1 + hf * D + 32 * cb + r;
  float bv[NB], w2v[D / 4];
#pragma unroll
  for (int s = 0; s < NB; ++s) bv[s] = busy ? bp[2 * s * D] : 0.0f;
#pragma unroll
  for (int s = 0; s < D / 4; ++s) w2v[s] = W2[(4 * s + q) * g.dphi + (l16 < g.dphi ? l16 : 0)];
  const float bias = busy ? c.w.b1[mh * D + 32 * cb + r] : 0.0f;
  const float b2v = c.w.b2[mh * g.dphi + (l16 < g.dphi ? l16 : 0)];
  stage_rows<D, kTok, 256, LD>(m == 0 ? Q : K, b, h, t0, nt, c.bf16, m == 0 ? c.vec_q : c.vec_k, sm);
  f32x16 acc[TPW];
#pragma unroll
  for (int i = 0; i < TPW; ++i) acc[i] = zero16();
  __syncthreads();
  if (busy) {
    weight_steps<NB, D / 2>(bv, [&](int s, float (&v)[NB]) {
#pragma unroll
      for (int t = 0; t < NB; ++t) v[t] = bp[2 * (s + t) * D];
    }, [&](int s, const float (&v)[NB]) {
#pragma unroll
      for (int t = 0; t < NB; ++t)
#pragma unroll
        for (int i = 0; i < TPW; ++i)
          acc[i] = mfma32(sm[(32 * (rb0 + i * W / NCB) + r) * LD + 2 * (s + t) + hf], v[t], acc[i]);
    });
  }
  __syncthreads();
  if (busy) {
#pragma unroll
    for (int i = 0; i < TPW; ++i)
#pragma unroll
      for (int j = 0; j < 16; ++j) {
          const float hv = acc[i][j] + bias;
          sm[(32 * (rb0 + i * W / NCB) + mf::d_row(j, hf)) * LD + 32 * cb + r] = hv * normal_cdf(hv);
        }
  }
  __syncthreads();
  // second layer: wave w serves tokens 16 w .. 16 w + 15, sixteen features per pass
  const float* ap = sm + (16 * wave + l16) * LD + q;
  auto put = [&](int a, const f32x4& u) {
    if (a >= g.dphi) return;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int t = 16 * wave + 4 * q + i;
      if (t < nt) feat[g.th(b, h, t0 + t) * g.nfeat + m * g.dphi + a] = fmaxf(u[i], 0.0f);
    }
  };
  f32x4 u = {b2v, b2v, b2v, b2v};
#pragma unroll
  for (int s = 0; s < D / 4; ++s) u = mfma16(ap[4 * s], l16 < g.dphi ? w2v[s] : 0.0f, u);
  put(l16, u);
  for (int c0 = 16; c0 < g.dphi; c0 += 16) {
    const int a = c0 + l16;
    const bool live = a < g.dphi;
    const float b2 = live ? c.w.b2[mh * g.dphi + a] : 0.0f;
    u = f32x4{b2, b2, b2, b2};
    const float* wp = W2 + q * g.dphi + (live ? a : 0);
#pragma unroll 8
    for (int s = 0; s < D / 4; ++s) {
      const float wv = wp[4 * s * g.dphi];
      u = mfma16(ap[4 * s], live ? wv : 0.0f, u);
    }
    put(a, u);
  }
}

// ---- backward -----------------------------------------------------------------------------------
// With du = d(feature) where the ReLU was open: dg = du W2^T, dh = dg GELU'(h) (h recomputed),
// dX = sum over the maps of dh W1^T.  NM > 0: also the weight gradients of the NM maps,
// dW1 = X^T dh, db1 = sum dh, dW2 = GELU(h)^T du, db2 = sum du, accumulated in registers over the
// workgroup's tiles and written as one partial per workgroup and map:
// partial[((map * heads + head) * gridDim.x + block)][D*D | D | D*dphi | dphi].
template <int D, int NM>
struct BwdCfg {
  // the accumulators of three maps at d = 128 need eight waves
  static constexpr int W = NM > 0 && D == 128 ? 8 : 4;
  static constexpr int THREADS = W * 64;
  static constexpr int LD = D + 4;
  static constexpr int NTW = (D / 32) * (D / 32);              // dW1 tiles
  static constexpr int TW = (NTW + W - 1) / W;                 // per wave
  static constexpr int NT2 = D / 16, T2 = (NT2 + W - 1) / W;   // 16-row tiles of dW2
  static constexpr int kRows = kTok * LD;
  __host__ __device__ static int ldu(int dphi) { return NM > 0 ? 17 : dphi | 1; }  // weight gradients: d_phi <= 16
  __host__ static size_t bytes(int dphi) {
    return 4u * ((NM > 0 ? 3 : 2) * kRows + (kTok * ldu(dphi) + 3) / 4 * 4 + (NM > 0 ? 2 * THREADS : 0));
  }
};

template <int D, int NM, int MAPS>
__device__ __forceinline__ void phi_bwd_body(const PhiCall& c, const View& X, bool vec, int map0, int nmaps,
                                             const float* __restrict__ feat, const float* __restrict__ dfeat,
                                             const View& dX, float* __restrict__ partial, float* sm) {
  using CF = BwdCfg<D, NM>;
  constexpr int W = CF::W, LD = CF::LD, NCB = PhiCfg<D>::NCB, NT = PhiCfg<D>::NT, TPW = PhiCfg<D>::template tpw<W>();
  constexpr int THREADS = CF::THREADS;
  static_assert(W % NCB == 0, "one column block per wave");
  const Geom& g = c.g;
  const int dphi = g.dphi, ldu = CF::ldu(dphi);
  float* xs = sm;
  float* dhs = xs + CF::kRows;
  float* gs = dhs + CF::kRows;                       // weight gradients only
  float* dus = NM > 0 ? gs + CF::kRows : gs;
  float* red = dus + (kTok * ldu + 3) / 4 * 4;       // weight gradients only
  const int lane = threadIdx.x % 64, wave = mf::wave_index();
  const int r = lane % 32, hf = lane / 32, l16 = lane % 16, q = lane / 16;
  const int head = blockIdx.y, hw = c.w.heads_w == 1 ? 0 : head;
  int rb0, cb;
  tile_pos<D>(wave, rb0, cb);
  const bool busy = wave < NT;
  constexpr int NA = NM > 0 ? MAPS : 1;
  f32x16 aw1[NA][CF::TW];
  f32x4 aw2[NA][CF::T2];
  float ab1[NA], ab2[NA];
#pragma unroll
  for (int m = 0; m < NA; ++m) {
#pragma unroll
    for (int i = 0; i < CF::TW; ++i) aw1[m][i] = zero16();
#pragma unroll
    for (int i = 0; i < CF::T2; ++i) aw2[m][i] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    ab1[m] = ab2[m] = 0.0f;
  }
  if (NM > 0)  // columns d_phi .. 15 of the du tile stay zero
    for (int i = threadIdx.x; i < kTok * 17; i += THREADS) dus[i] = 0.0f;
  for (int tile = blockIdx.x; tile < c.tiles; tile += gridDim.x) {
    int b, h, t0;
    tile_coords(c, tile, head, b, h, t0);
    const int nt = min(kTok, g.N - t0);
    const int64_t th0 = g.th(b, h, t0);
    __syncthreads();  // the previous tile's readers of xs, dhs, gs, dus are done
    stage_rows<D, kTok, THREADS, LD>(X, b, h, t0, nt, c.bf16, vec, xs);
    f32x16 dx[TPW];
#pragma unroll
    for (int i = 0; i < TPW; ++i) dx[i] = zero16();
    auto one_map = [&](int m, auto slot_tag) {
      constexpr int SLOT = decltype(slot_tag)::value;  // the map's accumulators
      const int64_t mh = static_cast<int64_t>(map0 + m) * c.w.heads_w + hw;
      const float* W1 = c.w.W1 + mh * D * D;
      const float* W1T = c.w.W1T + mh * D * D;
      const float* W2 = c.w.W2 + mh * D * dphi;
      for (int idx = threadIdx.x; idx < kTok * dphi; idx += THREADS) {
        const int t = idx / dphi, a = idx % dphi;
        float du = 0.0f;
        if (t < nt) {
          const int64_t o = (th0 + t) * g.nfeat + (map0 + m) * dphi + a;
          const float f = feat[o], d = dfeat[o];
          du = f > 0.0f ? d : 0.0f;  // ReLU passes gradient only where it was open
        }
        dus[t * ldu + a] = du;
      }
      __syncthreads();
      if (busy) {
        const float bias = c.w.b1[mh * D + 32 * cb + r];
        f32x16 hid[TPW], dg[TPW];
#pragma unroll
        for (int i = 0; i < TPW; ++i) hid[i] = dg[i] = zero16();
        // k-slot (step 4 k4 + j, half hf) is input channel (D / 2) hf + 4 k4 + j
        const float* bp = W1 + (D / 2) * hf * D + 32 * cb + r;
        float bv[8];
        auto load = [&](int s, float (&v)[8]) {
#pragma unroll
          for (int t = 0; t < 8; ++t) v[t] = bp[(s + t) * D];
        };
        load(0, bv);
        weight_steps<8, D / 2>(bv, load, [&](int s, const float (&v)[8]) {
#pragma unroll
          for (int s4 = 0; s4 < 8; s4 += 4)
#pragma unroll
            for (int i = 0; i < TPW; ++i) {
              const f32x4 a = *reinterpret_cast<const f32x4*>(xs + (32 * (rb0 + i * W / NCB) + r) * LD + (D / 2) * hf + s + s4);
#pragma unroll
              for (int j = 0; j < 4; ++j) hid[i] = mfma32(a[j], v[s4 + j], hid[i]);
            }
        });
        for (int s = 0; s < (dphi + 1) / 2; ++s) {
          const int a = 2 * s + hf;
          const float w2 = a < dphi ? W2[(32 * cb + r) * dphi + a] : 0.0f;
#pragma unroll
          for (int i = 0; i < TPW; ++i)
            dg[i] = mfma32(a < dphi ? dus[(32 * (rb0 + i * W / NCB) + r) * ldu + a] : 0.0f, w2, dg[i]);
        }
#pragma unroll
        for (int i = 0; i < TPW; ++i)
#pragma unroll
          for (int j = 0; j < 16; ++j) {
            const float hv = hid[i][j] + bias;
            const float cdf = normal_cdf(hv);
            const float pdf = 0.39894228040143267794f * expf(-0.5f * hv * hv);
            const float dh = dg[i][j] * (cdf + hv * pdf);
            const int at = (32 * (rb0 + i * W / NCB) + mf::d_row(j, hf)) * LD + 32 * cb + r;
            dhs[at] = dh;
            if constexpr (NM > 0) {
              gs[at] = hv * cdf;
              ab1[SLOT] += dh;
            }
          }
      }
      __syncthreads();
      if (busy) {
        const float* bp = W1T + (D / 2) * hf * D + 32 * cb + r;
        float bv[8];
        auto load = [&](int s, float (&v)[8]) {
#pragma unroll
          for (int t = 0; t < 8; ++t) v[t] = bp[(s + t) * D];
        };
        load(0, bv);
        weight_steps<8, D / 2>(bv, load, [&](int s, const float (&v)[8]) {
#pragma unroll
          for (int s4 = 0; s4 < 8; s4 += 4)
#pragma unroll
            for (int i = 0; i < TPW; ++i) {
              const f32x4 a = *reinterpret_cast<const f32x4*>(dhs + (32 * (rb0 + i * W / NCB) + r) * LD + (D / 2) * hf + s + s4);
#pragma unroll
              for (int j = 0; j < 4; ++j) dx[i] = mfma32(a[j], v[s4 + j], dx[i]);
            }
        });
      }
      if constexpr (NM > 0) {
#pragma unroll
        for (int i = 0; i < CF::TW; ++i) {
          const int tw = wave + W * i;
          if (tw < CF::NTW) {
            const float* ap = xs + 32 * hf * LD + 32 * (tw / NCB) + r;
            const float* bp = dhs + 32 * hf * LD + 32 * (tw % NCB) + r;
#pragma unroll 8
            for (int s = 0; s < 32; ++s) aw1[SLOT][i] = mfma32(ap[s * LD], bp[s * LD], aw1[SLOT][i]);
          }
        }
#pragma unroll
        for (int i = 0; i < CF::T2; ++i) {
          const int tw = wave + W * i;
          if (tw < CF::NT2) {
            const float* ap = gs + q * LD + 16 * tw + l16;
            const float* bp = dus + q * 17 + l16;
#pragma unroll 8
            for (int s = 0; s < 16; ++s) aw2[SLOT][i] = mfma16(ap[4 * s * LD], bp[4 * s * 17], aw2[SLOT][i]);
          }
        }
        constexpr int per = kTok * 16 / THREADS;  // thread (feature, group of tokens)
#pragma unroll
        for (int t = 0; t < per; ++t) ab2[SLOT] += dus[((threadIdx.x / 16) * per + t) * 17 + threadIdx.x % 16];
      }
      __syncthreads();  // dhs, gs, dus are free for the next map
    };
    if constexpr (NM > 0) {
      mf::static_for<0, MAPS>([&](auto M) { one_map(decltype(M)::value, M); });
    } else {
      for (int m = 0; m < nmaps; ++m) one_map(m, std::integral_constant<int, 0>{});
    }
    if (busy) {
#pragma unroll
      for (int i = 0; i < TPW; ++i)
#pragma unroll
        for (int j = 0; j < 16; ++j) {
          const int t = 32 * (rb0 + i * W / NCB) + mf::d_row(j, hf);
          if (t < nt) {
            if (c.bf16)
              dX.row<bf16_t>(b, h, t0 + t)[32 * cb + r] = from_float<bf16_t>(dx[i][j]);
            else
              dX.row<float>(b, h, t0 + t)[32 * cb + r] = dx[i][j];
          }
        }
    }
  }
  if constexpr (NM > 0) {
    const int64_t floats = static_cast<int64_t>(D) * D + D + D * dphi + dphi;
    mf::static_for<0, MAPS>([&](auto M) {
      constexpr int m = decltype(M)::value;
      float* out = partial + ((static_cast<int64_t>(map0 + m) * gridDim.y + head) * gridDim.x + blockIdx.x) * floats;
#pragma unroll
      for (int i = 0; i < CF::TW; ++i) {
        const int tw = wave + W * i;
        if (tw < CF::NTW) {
#pragma unroll
          for (int j = 0; j < 16; ++j)
            out[(32 * (tw / NCB) + mf::d_row(j, hf)) * D + 32 * (tw % NCB) + r] = aw1[m][i][j];
        }
      }
#pragma unroll
      for (int i = 0; i < CF::T2; ++i) {
        const int tw = wave + W * i;
        if (tw < CF::NT2 && l16 < dphi) {
#pragma unroll
          for (int j = 0; j < 4; ++j) out[D * D + D + (16 * tw + 4 * q + j) * dphi + l16] = aw2[m][i][j];
        }
      }
      __syncthreads();
      red[threadIdx.x] = busy ? ab1[m] : 0.0f;
      red[THREADS + threadIdx.x] = ab2[m];
      __syncthreads();
      for (int j = threadIdx.x; j < D; j += THREADS) {  // waves of column block j / 32, both lane halves
        float s = 0.0f;
        for (int w = j / 32; w < W; w += NCB) s += red[w * 64 + j % 32] + red[w * 64 + 32 + j % 32];
        out[D * D + j] = s;
      }
      for (int a = threadIdx.x; a < dphi; a += THREADS) {
        float s = 0.0f;
        for (int p = 0; p < THREADS / 16; ++p) s += red[THREADS + p * 16 + a];
        out[D * D + D + D * dphi + a] = s;
      }
    });
  }
}

// grid (workgroups per tile list, 1 or H, 2), block W * 64; z = 0: the key maps, z = 1: the query map.
// Two waves per SIMD: with 260 registers instead of 256 the d = 64 form took 171 us instead of 86 (at 12 heads x
// 4095 tokens, weight gradients included).
template <int D, int NM>
__global__ __launch_bounds__((BwdCfg<D, NM>::THREADS), 2) void k_f32_phi_bwd(PhiCall c, View Q, View K,
                                                                         const float* __restrict__ feat,
                                                                         const float* __restrict__ dfeat, View dQ,
                                                                         View dK, float* __restrict__ partial) {
  extern __shared__ __align__(16) float sm[];
  if (blockIdx.z == 0)
    phi_bwd_body<D, NM, NM>(c, K, c.vec_k, 1, c.g.F, feat, dfeat, dK, partial, sm);
  else
    phi_bwd_body<D, NM, 1>(c, Q, c.vec_q, 0, 1, feat, dfeat, dQ, partial, sm);
}

// W1T of every (map, head): out[j][i] = W1[i][j].  grid (d / 32, d / 32, maps * heads), block 32 x 8.
__global__ void k_transpose_w1(int d, const float* __restrict__ in, float* __restrict__ out) {
  __shared__ float tile[32][33];
  const int64_t base = static_cast<int64_t>(blockIdx.z) * d * d;
  const int r0 = blockIdx.y * 32, c0 = blockIdx.x * 32;
  for (int i = threadIdx.y; i < 32; i += 8) tile[i][threadIdx.x] = in[base + (r0 + i) * d + c0 + threadIdx.x];
  __syncthreads();
  for (int i = threadIdx.y; i < 32; i += 8) out[base + (c0 + i) * d + r0 + threadIdx.x] = tile[threadIdx.x][i];
}

// ---- host ---------------------------------------------------------------------------------------
PhiCall phi_call(const hla_handle* hd, const hla_call_args& a) {
  PhiCall c{};
  c.g = hd->g;
  c.w = hd->phi;
  c.bf16 = hd->cfg.io_dtype == HLA_BF16;
  const size_t elem = c.bf16 ? 2 : 4;
  c.vec_q = rows_vec(a.Q, elem);
  c.vec_k = rows_vec(a.K, elem);
  c.tpr = (a.N + kTok - 1) / kTok;
  c.tiles = c.tpr * (c.w.heads_w == 1 ? a.B * a.H : a.B);
  return c;
}

template <int D>
hla_status fwd_d(hla_handle* hd, const hla_call_args& a) {
  const PhiCall c = phi_call(hd, a);
  const bool shared = c.w.heads_w == 1;
  const int gx = shared ? std::min(c.tiles, kMaxGridX) : c.tiles;
  return launch(hd, "generic_phi_forward", &k_f32_phi_fwd<D>, dim3(gx, shared ? (c.tiles + gx - 1) / gx : a.H, 1 + c.g.F),
                dim3(256), kTok * (D + 1) * sizeof(float), a.stream, c, a.Q, a.K, hd->feat);
}

template <int D, int NM>
hla_status bwd_dn(hla_handle* hd, const hla_call_args& a) {
  using CF = BwdCfg<D, NM>;
  const PhiCall c = phi_call(hd, a);
  const int heads = c.w.heads_w == 1 ? 1 : a.H;
  // without weight gradients a workgroup per tile; with them at most f32_phi_parts workgroups per list,
  // each of equally many tiles, as every one leaves a partial to be added up
  int parts = std::min(c.tiles, kMaxGridX);
  if (NM > 0) {
    const int most = std::max(1, f32_phi_parts(D) / heads);
    const int per = static_cast<int>((c.tiles + most - 1) / most);
    parts = (c.tiles + per - 1) / per;
  }
  HLA_TRY(launch(hd, "generic_phi_backward", &k_f32_phi_bwd<D, NM>, dim3(parts, heads, 2), dim3(CF::THREADS),
                 CF::bytes(c.g.dphi), a.stream, c, a.Q, a.K, static_cast<const float*>(hd->feat),
                 static_cast<const float*>(hd->dfeat), a.dQ, a.dK, hd->wg_partial));
  if (NM == 0) return HLA_OK;
  return weight_grads_reduce(hd, parts, heads, 1.0f, 1.0f, 1.0f, 1.0f, a.stream);
}

template <int D>
hla_status bwd_d(hla_handle* hd, const hla_call_args& a) {
  if (!hd->wg_on) return bwd_dn<D, 0>(hd, a);
  switch (hd->g.F) {
    case 1: return bwd_dn<D, 1>(hd, a);
    case 2: return bwd_dn<D, 2>(hd, a);
    case 3: return bwd_dn<D, 3>(hd, a);
    case 4: return bwd_dn<D, 4>(hd, a);
  }
  return HLA_ERR_UNSUPPORTED;
}

template <int D, int NM>
hla_status allow_lds(int dphi) {
  const size_t bytes = BwdCfg<D, NM>::bytes(dphi);
  if (bytes > 160 * 1024) return HLA_ERR_UNSUPPORTED;
  return bytes <= 64 * 1024 || hipFuncSetAttribute(reinterpret_cast<const void*>(&k_f32_phi_bwd<D, NM>),
                                                   hipFuncAttributeMaxDynamicSharedMemorySize,
                                                   static_cast<int>(bytes)) == hipSuccess
             ? HLA_OK
             : HLA_ERR_HIP;
}
template <int D>
hla_status allow_lds_d(const Geom& g) {
  HLA_TRY((allow_lds<D, 0>(g.dphi)));
  if (g.dphi > 16) return HLA_OK;  // no weight gradients there
  switch (g.F) {
    case 1: return allow_lds<D, 1>(g.dphi);
    case 2: return allow_lds<D, 2>(g.dphi);
    case 3: return allow_lds<D, 3>(g.dphi);
    case 4: return allow_lds<D, 4>(g.dphi);
  }
  return HLA_ERR_UNSUPPORTED;
}

}  // namespace

hla_status f32_phi_prepare_kernels(const hla_handle* hd) {
  switch (hd->g.d) {
    case 32: return allow_lds_d<32>(hd->g);
    case 64: return allow_lds_d<64>(hd->g);
    case 128: return allow_lds_d<128>(hd->g);
  }
  return HLA_ERR_UNSUPPORTED;
}
hla_status f32_phi_set_weights(hla_handle* hd, hipStream_t s) {
  const int d = hd->g.d;
  return launch(hd, "transpose_weights", &k_transpose_w1, dim3(d / 32, d / 32, (1 + hd->g.F) * hd->phi.heads_w),
                dim3(32, 8), 0, s, d, hd->phi.W1, hd->w_f32_t);
}
hla_status f32_phi_forward(hla_handle* hd, const hla_call_args& a) {
  switch (hd->g.d) {
    case 32: return fwd_d<32>(hd, a);
    case 64: return fwd_d<64>(hd, a);
    case 128: return fwd_d<128>(hd, a);
  }
  return HLA_ERR_UNSUPPORTED;
}
// input gradients and, when their arrays are registered, the weight gradients
hla_status f32_phi_backward(hla_handle* hd, const hla_call_args& a) {
  switch (hd->g.d) {
    case 32: return bwd_d<32>(hd, a);
    case 64: return bwd_d<64>(hd, a);
    case 128: return bwd_d<128>(hd, a);
  }
  return HLA_ERR_UNSUPPORTED;
}

}  // namespace hla
