// Generic path, common parts: feature import / export, conversion of the feature-map weights, the sum
// of their gradients' partials, and the causal variant as a token-by-token scan over the literal d_phi^F feature
// tensor (a cross-check of the matrix-core path; throughput is not a goal there).  The non-causal
// operator of this path is hla_f32.hip, its feature maps hla_f32_phi.hip.
//
// The scan uses the augmented state  Chat = [C | z]  ([D, d+1]) and augmented per-token rows
// vhat_j = [v_j | 1], ghat_i = [dO_i/den_i | -<dO_i,o_i>/den_i].
#include <cmath>

#include "hla_handle.h"

namespace hla {
namespace {

constexpr int kThreads = 256;
constexpr int kChunk = 1024;      // tokens per table entry of the causal scan
constexpr int kMaxF = 4;

// Slot offsets into a feature row: query tensors use phi_q in every slot, key tensors use map f.
__device__ __forceinline__ int slot_offset(bool query, int slot, int dphi) {
  return query ? 0 : (1 + slot) * dphi;
}

// Entry `Di` of the outer product of one token's features (first slot slowest).
__device__ __forceinline__ float outer_entry(const float* frow, bool query, int Di, int F,
                                             int dphi) {
  float p = 1.0f;
  for (int s = F - 1; s >= 0; --s) {
    const int a = Di % dphi;
    Di /= dphi;
    p *= frow[slot_offset(query, s, dphi) + a];
  }
  return p;
}

// ---- weights / features I/O -------------------------------------------------------------------
template <typename T>
__global__ void k_convert_weights(const T* __restrict__ src, int64_t head_stride, float* dst,
                                  int count, int heads_w) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  const int hw = blockIdx.y;
  if (i < count && hw < heads_w) dst[static_cast<int64_t>(hw) * count + i] = to_float(src[hw * head_stride + i]);
}

// PHI_NONE: copy caller-provided features into the fp32 feature workspace.  One thread per
// token-head: its two feature rows are contiguous in the caller's tensors, and in the tiled
// workspace of the MFMA path 32 consecutive threads write 32 consecutive floats per feature.
template <typename T>
__global__ void k_feat_import(Geom g, View Q, View K, float* __restrict__ feat) {
  const uint32_t th = blockIdx.x * blockDim.x + threadIdx.x;
  if (th >= static_cast<uint32_t>(g.B) * g.H * g.N) return;  // < 2^31 by the create-time check
  const int n = static_cast<int>(th % g.N);
  const uint32_t bh = th / g.N;
  const int h = static_cast<int>(bh % g.H), b = static_cast<int>(bh / g.H);
  const T* q = Q.row<const T>(b, h, n);
  const T* k = K.row<const T>(b, h, n);
  if constexpr (sizeof(T) == 2) {
    // a pair of bf16 features per load and an 8-byte store per pair where the rows allow it: a
    // pair is adjacent in both layouts of the workspace (see fidx), pair p + 1 sits `step` floats on
    const bool pairs = g.dphi % 2 == 0 && ((reinterpret_cast<uintptr_t>(q) | reinterpret_cast<uintptr_t>(k)) & 3) == 0;
    if (pairs) {
      const uint32_t* q2 = reinterpret_cast<const uint32_t*>(q);
      const uint32_t* k2 = reinterpret_cast<const uint32_t*>(k);
      float* dst = feat + g.fidx(th, 0);
      const int step = g.feat_tiled ? 64 : 2, nq = g.dphi / 2, np = g.nfeat / 2;
      // eight pairs' loads in flight before the first store (a load next to the store that needs
      // it would cost a memory round trip per pair)
      for (int p0 = 0; p0 < np; p0 += 8) {
        uint32_t w[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const int p = p0 + i < np ? p0 + i : np - 1;
          w[i] = p < nq ? q2[p] : k2[p - nq];
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) asm volatile("" : "+v"(w[i]));  // all eight are loaded here: the compiler may not sink a load to its store
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          if (p0 + i >= np) break;
          float2 v;
          v.x = __uint_as_float(w[i] << 16);
          v.y = __uint_as_float(w[i] & 0xffff0000u);
          *reinterpret_cast<float2*>(dst + static_cast<int64_t>(p0 + i) * step) = v;
        }
      }
      return;
    }
  }
  for (int j = 0; j < g.dphi; ++j) feat[g.fidx(th, j)] = to_float(q[j]);
  for (int j = g.dphi; j < g.nfeat; ++j) feat[g.fidx(th, j)] = to_float(k[j - g.dphi]);
}

// PHI_NONE: feature gradients are the answer; store them in the I/O dtype.
template <typename T>
__global__ void k_dfeat_export(Geom g, const float* __restrict__ dfeat, View dQ, View dK) {
  const uint32_t th = blockIdx.x * blockDim.x + threadIdx.x;
  if (th >= static_cast<uint32_t>(g.B) * g.H * g.N) return;
  const int n = static_cast<int>(th % g.N);
  const uint32_t bh = th / g.N;
  const int h = static_cast<int>(bh % g.H), b = static_cast<int>(bh / g.H);
  T* q = dQ.row<T>(b, h, n);
  T* k = dK.row<T>(b, h, n);
  if constexpr (sizeof(T) == 2) {
    // two bf16 values per store where the rows allow it
    const bool pairs = g.dphi % 2 == 0 && ((reinterpret_cast<uintptr_t>(q) | reinterpret_cast<uintptr_t>(k)) & 3) == 0;
    if (pairs) {
      uint32_t* q2 = reinterpret_cast<uint32_t*>(q);
      uint32_t* k2 = reinterpret_cast<uint32_t*>(k);
      const float* src = dfeat + g.fidx(th, 0);  // pair p: 8 bytes at src + p * step (see fidx)
      const int step = g.feat_tiled ? 64 : 2, nq = g.dphi / 2, np = g.nfeat / 2;
      for (int p0 = 0; p0 < np; p0 += 8) {  // eight pairs' loads in flight before the first store
        float2 v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i)
          v[i] = *reinterpret_cast<const float2*>(src + static_cast<int64_t>(p0 + i < np ? p0 + i : np - 1) * step);
#pragma unroll
        for (int i = 0; i < 8; ++i) asm volatile("" : "+v"(v[i].x), "+v"(v[i].y));  // as in k_feat_import
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          if (p0 + i >= np) break;
          const uint32_t w = static_cast<uint32_t>(f32_to_bf16_bits(v[i].x)) |
                             (static_cast<uint32_t>(f32_to_bf16_bits(v[i].y)) << 16);
          if (p0 + i < nq) q2[p0 + i] = w; else k2[p0 + i - nq] = w;
        }
      }
      return;
    }
  }
  for (int j = 0; j < g.dphi; ++j) q[j] = from_float<T>(dfeat[g.fidx(th, j)]);
  for (int j = g.dphi; j < g.nfeat; ++j) k[j - g.dphi] = from_float<T>(dfeat[g.fidx(th, j)]);
}

// ---- weight gradients of the feature maps: sum of the partials --------------------------------
// Sum of the partial weight gradients of one (map, head) in a fixed order, times the scale of its
// section, into the caller's arrays.  grid (ceil(floats SL / 256), 1+F, heads), block 256: SL slices of
// the partials per element, sixteen loads in flight each.  A workgroup is a chain of memory round trips, which
// slices shorten; where the elements fill the card by themselves, they only add to what is in its way.
struct WgradOut {
  float* dW1[kMaxF + 1];
  float* db1[kMaxF + 1];
  float* dW2[kMaxF + 1];
  float* db2[kMaxF + 1];
};
template <int SL>
__global__ __launch_bounds__(256) void k_wgrad_reduce(int d, int dphi, int nparts,
                               const float* __restrict__ partial, WgradOut out, float sW1, float sb1,
                               float sW2, float sb2) {
  const int nW1 = d * d, nb1 = d, nW2 = d * dphi, nb2 = dphi;
  const int floats = nW1 + nb1 + nW2 + nb2;
  constexpr int EL = 256 / SL;
  __shared__ float slices[SL][EL];
  const int slice = threadIdx.x / EL, e = blockIdx.x * EL + threadIdx.x % EL;
  const int m = blockIdx.y, hw = blockIdx.z;
  const float* p = partial + (static_cast<int64_t>(m) * gridDim.z + hw) * nparts * floats + (e < floats ? e : floats - 1);
  const int per = (nparts + SL - 1) / SL, k0 = slice * per, k1 = min(k0 + per, nparts);
  float sum = 0.0f;
  for (int k = k0; k < k1; k += 16) {
    float v[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) v[u] = p[static_cast<int64_t>(min(k + u, k1 - 1)) * floats];
#pragma unroll
    for (int u = 0; u < 16; ++u)
      if (k + u < k1) sum += v[u];
  }
  if (SL > 1) {
    slices[slice][threadIdx.x % EL] = sum;
    __syncthreads();
  }
  if (slice != 0 || e >= floats) return;
#pragma unroll
  for (int u = 1; u < SL; ++u) sum += slices[u][threadIdx.x];
  if (e < nW1) {
    out.dW1[m][static_cast<int64_t>(hw) * nW1 + e] = sW1 * sum;
  } else if (e < nW1 + nb1) {
    out.db1[m][static_cast<int64_t>(hw) * nb1 + (e - nW1)] = sb1 * sum;
  } else if (e < nW1 + nb1 + nW2) {
    out.dW2[m][static_cast<int64_t>(hw) * nW2 + (e - nW1 - nb1)] = sW2 * sum;
  } else {
    out.db2[m][static_cast<int64_t>(hw) * nb2 + (e - nW1 - nb1 - nW2)] = sb2 * sum;
  }
}

// ghat_i = [dO_i / den_i | -<dO_i, o_i> / den_i]   (one block row of d threads per token)
// grid (ceil(N/R), H, B), block 256.
template <typename T>
__global__ void k_backward_prep(Geom g, View dO, View O, const float* __restrict__ den,
                                float* __restrict__ yhat) {
  __shared__ float red[kThreads];
  const int d = g.d;
  const int R = kThreads / d;
  const int c = threadIdx.x % d, r = threadIdx.x / d;
  const int n = blockIdx.x * R + r, h = blockIdx.y, b = blockIdx.z;
  const bool live = n < g.N;
  float go = 0.0f, dn = 1.0f, dot = 0.0f;
  if (live) {
    dn = den[g.th(b, h, n)];
    go = to_float(dO.row<const T>(b, h, n)[c]);
    dot = go * to_float(O.row<const T>(b, h, n)[c]);
  }
  red[threadIdx.x] = dot;
  __syncthreads();
  for (int s = d / 2; s > 0; s >>= 1) {
    if (c < s) red[threadIdx.x] += red[threadIdx.x + s];
    __syncthreads();
  }
  if (live) {
    float* y = yhat + g.th(b, h, n) * (d + 1);
    y[c] = go / dn;
    if (c == 0) y[d] = -red[r * d] / dn;
  }
}

// Chain rule from dT [tile][D] (LDS) through the outer product to the feature gradients of the
// tile's tokens: the gradient of slot s, coordinate a, token t is the sum over the entries whose
// digit s equals a of dT[entry] times the product of the other slots' features.  QUERY: all F
// slots hold phi_q and their gradients are summed into dfeat[.., 0:dphi]; otherwise slot f goes
// to dfeat[.., (1+f)*dphi : ..].  Called by all threads of the block; fs = features [tile][nfeat].
template <bool QUERY>
__device__ __forceinline__ void slot_gradients(const Geom& g, const float* fs, const float* dts,
                                               int tile, int nt, int b, int h, int t0,
                                               float* __restrict__ dfeat) {
  const int D = g.D, dphi = g.dphi, F = g.F;
  const int nout = QUERY ? tile * dphi : tile * F * dphi;
  for (int idx = threadIdx.x; idx < nout; idx += blockDim.x) {
    int t, s_lo, s_hi, a;
    if (QUERY) {
      t = idx / dphi;
      a = idx % dphi;
      s_lo = 0;
      s_hi = F;
    } else {
      t = idx / (F * dphi);
      s_lo = (idx / dphi) % F;
      s_hi = s_lo + 1;
      a = idx % dphi;
    }
    if (t >= nt) continue;
    const float* frow = fs + t * g.nfeat;
    float grad = 0.0f;
    for (int s = s_lo; s < s_hi; ++s) {
      for (int Di = 0; Di < D; ++Di) {
        int rem = Di;
        float p = 1.0f;
        bool hit = false;
        for (int sl = F - 1; sl >= 0; --sl) {
          const int dig = rem % dphi;
          rem /= dphi;
          if (sl == s)
            hit = dig == a;
          else
            p *= frow[slot_offset(QUERY, sl, dphi) + dig];
        }
        if (hit) grad += dts[t * D + Di] * p;
      }
    }
    const int col = QUERY ? a : (1 + s_lo) * dphi + a;
    dfeat[g.fidx(g.th(b, h, t0 + t), col)] = grad;
  }
}

// ---- causal variant (Sec. 4.4): one scan over the tokens of a (sequence, head) ------------------
// The sequential state update  Chat^i = decay Chat^{i-1} + T_k,i (x) vhat_i  (and, for the gradient
// of the key side, its mirror image from the back,  dChat^j = decay dChat^{j+1} + T_q,j (x) ghat_j)
// carried through the sequence by ONE workgroup, TT tokens at a time, with the running state in
// LDS.  With a = the tensor that builds the state and ya its augmented rows, b = the tensor that
// reads it and yb its rows, m_tj = decay^|t-j| on the visible side of the mask (j <= t going
// forward, j >= t going back) and c_t the decay of the carried state C as seen from token t:
//   out_t = c_t b_t . C  + sum_j m_tj <b_t, a_j> ya_j          (contract)
//   db_t  = c_t C yb_t   + sum_j m_tj <yb_t, ya_j> a_j         (dtensor, then the chain rule)
//   C    <- decay^TT C   + sum_j u_j a_j (x) ya_j              (u_j: decay from token j to the carry's reference)
// MODE 0: a = T_k, ya = vhat, b = T_q:            O = out[0:d] / (out[d] + eps), den
// MODE 1: same state, yb = ghat:                  d(phi_q) from db
// MODE 2: a = T_q, ya = ghat, b = T_k, yb = vhat, from the back:  dV = out[0:d], d(phi_k) from db
// grid (num_seqs, H), block 256.  Throughput is not a goal: this is the fp32 cross-check of the scan.
template <int TT>
__host__ __device__ constexpr size_t causal_scan_floats(int D, int d, int nfeat) {
  return static_cast<size_t>(D) * (d + 1) + 3 * static_cast<size_t>(TT) * D + 2 * static_cast<size_t>(TT) * (d + 1) +
         static_cast<size_t>(TT) * nfeat + 2 * TT * TT + 3 * TT;
}

template <typename T, int MODE, int TT>
__global__ __launch_bounds__(kThreads) void k_causal_scan(
    Geom g, const BlockEnt* __restrict__ chunks, const int32_t* __restrict__ seq_chunk_off,
    const float* __restrict__ feat, View V, const float* __restrict__ ghat, float decay, View Out,
    float* __restrict__ den, float* __restrict__ dfeat) {
  extern __shared__ float smem[];
  constexpr bool BACK = MODE == 2;
  const int d = g.d, D = g.D, d1 = g.d + 1;
  const int R = kThreads / d;
  float* C = smem;                 // [D][d+1] carried state
  float* A = C + D * d1;           // [TT][D]  state-building tensor
  float* Bt = A + TT * D;          // [TT][D]  reading tensor
  float* dts = Bt + TT * D;        // [TT][D]  db
  float* ya = dts + TT * D;        // [TT][d+1]
  float* yb = ya + TT * d1;        // [TT][d+1]
  float* fs = yb + TT * d1;        // [TT][nfeat]
  float* mp = fs + TT * g.nfeat;   // [TT][TT] m_tj <b_t, a_j>
  float* mw = mp + TT * TT;        // [TT][TT] m_tj <yb_t, ya_j>
  float* cf = mw + TT * TT;        // [TT] c_t
  float* uf = cf + TT;             // [TT] u_j
  float* etas = uf + TT;           // [TT]
  const int s = blockIdx.x, h = blockIdx.y;
  const int tid = threadIdx.x;
  const int c0 = seq_chunk_off[s], c1 = seq_chunk_off[s + 1];
  if (c0 == c1) return;  // empty sequence (uniform over the block)
  const int b = chunks[c0].b, lo = chunks[c0].t0, hi = chunks[c1 - 1].t1;
  const int ntiles = (hi - lo + TT - 1) / TT;
  for (int idx = tid; idx < D * d1; idx += kThreads) C[idx] = 0.0f;
  if (tid < TT) {
    // forward: C is the state at the last token before the tile; back: at the first token behind it
    cf[tid] = powf(decay, static_cast<float>(BACK ? TT - tid : tid + 1));
    uf[tid] = powf(decay, static_cast<float>(BACK ? tid : TT - 1 - tid));
  }
  const float tile_decay = powf(decay, static_cast<float>(TT));
  for (int ti = 0; ti < ntiles; ++ti) {
    const int t0 = lo + (BACK ? ntiles - 1 - ti : ti) * TT;
    const int nt = min(TT, hi - t0);
    __syncthreads();  // the previous tile's readers of fs, A, ya, dts are done; C is up to date
    for (int idx = tid; idx < TT * g.nfeat; idx += kThreads) {
      const int t = idx / g.nfeat;
      fs[idx] = t < nt ? feat[g.fidx(g.th(b, h, t0 + t), idx % g.nfeat)] : 0.0f;
    }
    for (int idx = tid; idx < TT * d1; idx += kThreads) {
      const int t = idx / d1, cc = idx % d1;
      float v = 0.0f, gh = 0.0f;  // rows of tokens beyond the sequence are zero, the 1 included
      if (t < nt) {
        v = cc < d ? to_float(V.row<const T>(b, h, t0 + t)[cc]) : 1.0f;
        if (MODE != 0) gh = ghat[g.th(b, h, t0 + t) * d1 + cc];
      }
      (BACK ? yb : ya)[idx] = v;
      if (MODE != 0) (BACK ? ya : yb)[idx] = gh;
    }
    __syncthreads();
    for (int idx = tid; idx < TT * D; idx += kThreads) {
      const int t = idx / D, Di = idx % D;
      const float tq = outer_entry(fs + t * g.nfeat, true, Di, g.F, g.dphi);
      const float tk = outer_entry(fs + t * g.nfeat, false, Di, g.F, g.dphi);
      A[idx] = BACK ? tq : tk;
      Bt[idx] = BACK ? tk : tq;
    }
    __syncthreads();
    for (int idx = tid; idx < (MODE == 0 ? 1 : 2) * TT * TT; idx += kThreads) {
      const int w = idx / (TT * TT), t = (idx / TT) % TT, j = idx % TT;
      const bool visible = BACK ? j >= t : j <= t;
      float acc = 0.0f;
      if (visible) {
        if (w == 0) {
          for (int Di = 0; Di < D; ++Di) acc += Bt[t * D + Di] * A[j * D + Di];
        } else {
          for (int cc = 0; cc < d1; ++cc) acc += yb[t * d1 + cc] * ya[j * d1 + cc];
        }
        acc *= powf(decay, static_cast<float>(BACK ? j - t : t - j));
      }
      (w == 0 ? mp : mw)[t * TT + j] = acc;
    }
    __syncthreads();
    // contract: thread (r, c) owns column c of tokens r, r + R, ..
    float out[TT];
    if (MODE != 1) {
      const int c = tid % d, r = tid / d;
#pragma unroll
      for (int k = 0; k < TT; ++k) {
        const int t = r + k * R;
        float acc = 0.0f;
        if (t < TT) {
          for (int Di = 0; Di < D; ++Di) acc += Bt[t * D + Di] * C[Di * d1 + c];
          acc *= cf[t];
          for (int j = 0; j < TT; ++j) acc += mp[t * TT + j] * ya[j * d1 + c];
        }
        out[k] = acc;
      }
      if (MODE == 0 && tid < TT) {
        float eta = 0.0f;
        for (int Di = 0; Di < D; ++Di) eta += Bt[tid * D + Di] * C[Di * d1 + d];
        eta *= cf[tid];
        for (int j = 0; j < TT; ++j) eta += mp[tid * TT + j] * ya[j * d1 + d];
        etas[tid] = eta + g.eps;
        if (tid < nt) den[g.th(b, h, t0 + tid)] = eta + g.eps;
      }
    }
    // dtensor: thread Di owns row Di of the state
    if (MODE != 0 && tid < D) {
      float dt[TT];
#pragma unroll
      for (int t = 0; t < TT; ++t) dt[t] = 0.0f;
      for (int cc = 0; cc < d1; ++cc) {
        const float cv = C[tid * d1 + cc];
#pragma unroll
        for (int t = 0; t < TT; ++t) dt[t] += cv * yb[t * d1 + cc];
      }
#pragma unroll
      for (int t = 0; t < TT; ++t) {
        float acc = dt[t] * cf[t];
        for (int j = 0; j < TT; ++j) acc += mw[t * TT + j] * A[j * D + tid];
        dts[t * D + tid] = acc;
      }
    }
    __syncthreads();  // every read of C is done; etas and dts are visible
    if (MODE != 1) {
      const int c = tid % d, r = tid / d;
#pragma unroll
      for (int k = 0; k < TT; ++k) {
        const int t = r + k * R;
        if (t < nt) Out.row<T>(b, h, t0 + t)[c] = from_float<T>(MODE == 0 ? out[k] / etas[t] : out[k]);
      }
    }
    if (MODE == 1) slot_gradients<true>(g, fs, dts, TT, nt, b, h, t0, dfeat);
    if (MODE == 2) slot_gradients<false>(g, fs, dts, TT, nt, b, h, t0, dfeat);
    for (int idx = tid; idx < D * d1; idx += kThreads) {
      const int Di = idx / d1, cc = idx % d1;
      float acc = C[idx] * tile_decay;
      for (int j = 0; j < TT; ++j) acc += uf[j] * A[j * D + Di] * ya[j * d1 + cc];
      C[idx] = acc;
    }
  }
}

template <typename T>
hla_status features_import_t(hla_handle* hd, const hla_call_args& a) {
  const int64_t total = static_cast<int64_t>(hd->g.B) * hd->g.H * hd->g.N;
  return launch(hd, "generic_feat_import", k_feat_import<T>, dim3((total + 255) / 256), dim3(256), 0, a.stream, hd->g,
                a.Q, a.K, hd->feat);
}
template <typename T>
hla_status features_export_t(hla_handle* hd, const hla_call_args& a) {
  const int64_t total = static_cast<int64_t>(hd->g.B) * hd->g.H * hd->g.N;
  return launch(hd, "generic_dfeat_export", k_dfeat_export<T>, dim3((total + 255) / 256), dim3(256), 0, a.stream,
                hd->g, hd->dfeat, a.dQ, a.dK);
}

// The causal scan in one of its three modes; TT = 8 tokens per step where the LDS allows, else 4.
constexpr size_t kLdsLimit = 160 * 1024;
inline int causal_scan_tile(const Geom& g) {
  if (causal_scan_floats<8>(g.D, g.d, g.nfeat) * sizeof(float) <= kLdsLimit) return 8;
  if (causal_scan_floats<4>(g.D, g.d, g.nfeat) * sizeof(float) <= kLdsLimit) return 4;
  return 0;
}

template <typename T, int MODE, int TT>
hla_status causal_scan_launch(hla_handle* hd, const hla_call_args& a, const char* name, View out) {
  const Geom& g = hd->g;
  hla_token_table* chunks = nullptr;
  HLA_TRY(get_table(hd, 0, kChunk, a.stream, &chunks));
  const size_t sh = causal_scan_floats<TT>(g.D, g.d, g.nfeat) * sizeof(float);
  auto kernel = &k_causal_scan<T, MODE, TT>;
  const float dec = hd->cfg.decay > 0.0f && hd->cfg.decay < 1.0f ? hd->cfg.decay : 1.0f;
  return launch(hd, name, kernel, dim3(a.num_seqs, g.H), dim3(kThreads), sh, a.stream, g, chunks->dev,
                chunks->seq_off_dev, static_cast<const float*>(hd->feat), a.V,
                static_cast<const float*>(hd->yhat), dec, out, hd->den, hd->dfeat);
}

// The scan's LDS exceeds the 64 KB a kernel gets without asking: the three modes of a handle's
// dtype and tile are given their size once, when the handle is planned.
template <typename T, int TT>
hla_status causal_scan_allow_lds(const Geom& g) {
  const int sh = static_cast<int>(causal_scan_floats<TT>(g.D, g.d, g.nfeat) * sizeof(float));
  const void* kernels[3] = {reinterpret_cast<const void*>(&k_causal_scan<T, 0, TT>),
                            reinterpret_cast<const void*>(&k_causal_scan<T, 1, TT>),
                            reinterpret_cast<const void*>(&k_causal_scan<T, 2, TT>)};
  for (const void* k : kernels)
    if (hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, sh) != hipSuccess) return HLA_ERR_HIP;
  return HLA_OK;
}

template <typename T, int MODE>
hla_status causal_scan(hla_handle* hd, const hla_call_args& a, const char* name, View out) {
  switch (causal_scan_tile(hd->g)) {
    case 8: return causal_scan_launch<T, MODE, 8>(hd, a, name, out);
    case 4: return causal_scan_launch<T, MODE, 4>(hd, a, name, out);
    default: return HLA_ERR_UNSUPPORTED;
  }
}

template <typename T>
hla_status causal_backward_t(hla_handle* hd, const hla_call_args& a) {
  const Geom& g = hd->g;
  const int R = kThreads / g.d;
  HLA_TRY(launch(hd, "generic_backward_prep", k_backward_prep<T>, dim3((g.N + R - 1) / R, g.H, g.B),
                 dim3(kThreads), 0, a.stream, g, a.dO, a.O, hd->den, hd->yhat));
  // the same state recurrence once more for d(phi_q), its mirror image from the back for
  // d(phi_k) and dV
  HLA_TRY((causal_scan<T, 1>(hd, a, "generic_causal_dquery", a.dV)));
  return causal_scan<T, 2>(hd, a, "generic_causal_dkey", a.dV);
}

}  // namespace

hla_status generic_workspace_plan(hla_handle* hd) {
  const Geom& g = hd->g;
  if (g.F > kMaxF || g.D > kThreads) return HLA_ERR_UNSUPPORTED;
  if (!hd->cfg.causal) return f32_workspace_plan(hd);
  // the scan keeps its state in LDS: token table and the augmented gradient rows only
  if (causal_scan_tile(g) == 0) return HLA_ERR_UNSUPPORTED;
  hd->state_stride = 1;
  hd->max_chunks = 1;
  hd->yhat_floats = hd->max_th * (g.d + 1);
  hd->tables[0].min_block = kChunk;
  return HLA_OK;
}

// What a handle on this path needs once: kernel attributes and, where the form has none at compile
// time, the monomial tables (written on `s`).
hla_status generic_prepare_kernels(const hla_handle* hd, hipStream_t s) {
  if (hd->cfg.phi_mode == HLA_PHI_MLP) HLA_TRY(f32_phi_prepare_kernels(hd));
  if (!hd->cfg.causal) return f32_prepare_kernels(hd, s);
  const Geom& g = hd->g;
  const bool f32 = hd->cfg.io_dtype == HLA_F32;
  switch (causal_scan_tile(g)) {
    case 8: return f32 ? causal_scan_allow_lds<float, 8>(g) : causal_scan_allow_lds<bf16_t, 8>(g);
    case 4: return f32 ? causal_scan_allow_lds<float, 4>(g) : causal_scan_allow_lds<bf16_t, 4>(g);
    default: return HLA_ERR_UNSUPPORTED;
  }
}

hla_status convert_weights_to_f32(hla_handle* hd, const hla_phi_weights* maps, hipStream_t s) {
  const Geom& g = hd->g;
  const int nm = 1 + g.F;
  bool shared = true;
  for (int m = 0; m < nm; ++m)
    shared = shared && maps[m].head_stride_W1 == 0 && maps[m].head_stride_b1 == 0 &&
             maps[m].head_stride_W2 == 0 && maps[m].head_stride_b2 == 0;
  const int hw = shared ? 1 : hd->cfg.max_heads;
  const int64_t nW1 = static_cast<int64_t>(g.d) * g.d, nb1 = g.d, nW2 = static_cast<int64_t>(g.d) * g.dphi,
                nb2 = g.dphi;
  float* W1 = hd->w_f32;
  float* b1 = W1 + nm * hw * nW1;
  float* W2 = b1 + nm * hw * nb1;
  float* b2 = W2 + nm * hw * nW2;
  hd->phi = PhiF32{W1, b1, W2, b2, hd->w_f32_t, hw};
  for (int m = 0; m < nm; ++m) {
    struct Item {
      const void* src;
      int64_t stride;
      float* dst;
      int64_t count;
    } items[4] = {{maps[m].W1, maps[m].head_stride_W1, W1 + m * hw * nW1, nW1},
                  {maps[m].b1, maps[m].head_stride_b1, b1 + m * hw * nb1, nb1},
                  {maps[m].W2, maps[m].head_stride_W2, W2 + m * hw * nW2, nW2},
                  {maps[m].b2, maps[m].head_stride_b2, b2 + m * hw * nb2, nb2}};
    for (const Item& it : items) {
      dim3 grid(static_cast<unsigned>((it.count + 255) / 256), hw);
      if (hd->cfg.io_dtype == HLA_F32)
        HLA_TRY(launch(hd, "convert_weights", k_convert_weights<float>, grid, dim3(256), 0, s,
                       static_cast<const float*>(it.src), it.stride, it.dst, static_cast<int>(it.count), hw));
      else
        HLA_TRY(launch(hd, "convert_weights", k_convert_weights<bf16_t>, grid, dim3(256), 0, s,
                       static_cast<const bf16_t*>(it.src), it.stride, it.dst, static_cast<int>(it.count), hw));
    }
  }
  return HLA_OK;
}

hla_status generic_set_weights(hla_handle* hd, hipStream_t s) { return f32_phi_set_weights(hd, s); }

hla_status weight_grads_reduce(hla_handle* hd, int nparts, int heads, float sW1, float sb1, float sW2,
                               float sb2, hipStream_t s) {
  const int nm = 1 + hd->g.F;
  WgradOut out{};
  for (int m = 0; m < nm; ++m) {
    out.dW1[m] = hd->wg_out[m].dW1;
    out.db1[m] = hd->wg_out[m].db1;
    out.dW2[m] = hd->wg_out[m].dW2;
    out.db2[m] = hd->wg_out[m].db2;
  }
  const int floats = static_cast<int>(hd->wg_part_floats);
  // Four slices where one would leave compute units without a workgroup.  us with one / four slices, workgroups of
  // one slice in brackets: 256 partials of 64 channels and 4 maps (76) 11.8 / 6.6, of 128 channels and 2
  // maps (138) 12.3 / 10.2, 3 maps (213) 13.0 / 13.8, 4 maps (272) 13.9 / 16.5; 128 partials of 64 channels,
  // 4 maps and 4 heads (304) 8.5 / 9.6.  With 64 partials and fewer either is within 0.7 of the other.
  const int64_t groups = static_cast<int64_t>((floats + 255) / 256) * nm * heads;
  const int sl = groups < 200 ? 4 : 1;
  return launch(hd, "phi_weight_grads_reduce", sl == 4 ? &k_wgrad_reduce<4> : &k_wgrad_reduce<1>,
                dim3((floats * sl + 255) / 256, nm, heads), dim3(256), 0, s, hd->g.d, hd->g.dphi, nparts, static_cast<const float*>(hd->wg_partial), out,
                sW1, sb1, sW2, sb2);
}

hla_status phi_weight_grads(hla_handle* hd, const hla_call_args& a) {
  // the generic path's backward through the maps forms them along with the input gradients
  return hd->path == HLA_PATH_MFMA ? mfma_phi_weight_grads(hd, a) : HLA_OK;
}

// Features in (feature maps, or import of caller-provided features) and feature gradients out
// (through the maps, or exported as they are).  Import and export are shared with the MFMA path.
hla_status generic_features_in(hla_handle* hd, const hla_call_args& a) {
  if (hd->cfg.phi_mode == HLA_PHI_MLP) return f32_phi_forward(hd, a);
  return hd->cfg.io_dtype == HLA_F32 ? features_import_t<float>(hd, a) : features_import_t<bf16_t>(hd, a);
}
hla_status generic_features_out(hla_handle* hd, const hla_call_args& a) {
  if (hd->cfg.phi_mode == HLA_PHI_MLP) return f32_phi_backward(hd, a);
  return hd->cfg.io_dtype == HLA_F32 ? features_export_t<float>(hd, a) : features_export_t<bf16_t>(hd, a);
}

hla_status generic_forward(hla_handle* hd, const hla_call_args& a) {
  HLA_TRY(generic_features_in(hd, a));
  if (!hd->cfg.causal) return f32_forward(hd, a);
  return hd->cfg.io_dtype == HLA_F32 ? causal_scan<float, 0>(hd, a, "generic_causal_forward", a.O)
                                     : causal_scan<bf16_t, 0>(hd, a, "generic_causal_forward", a.O);
}

hla_status generic_backward(hla_handle* hd, const hla_call_args& a) {
  if (!hd->cfg.causal)
    HLA_TRY(f32_backward(hd, a));
  else
    HLA_TRY(hd->cfg.io_dtype == HLA_F32 ? causal_backward_t<float>(hd, a) : causal_backward_t<bf16_t>(hd, a));
  return generic_features_out(hd, a);
}

}  // namespace hla
