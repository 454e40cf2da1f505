// Value modulation (paper Sec. 4.5) on the matrix cores, bf16 I/O, head dim 64 or 128:
//   O = T + phi_v1(T) * phi_v2(V),   phi_v (App. A.1) = Linear d->d, GELU, Linear d->d, LayerNorm,
// forward and the backward to (dT, dV).
//
// A token is an MFMA column (lane (r, gl): token r of a 32-token tile, half gl), as in the feature
// maps.  Every product takes its A operand from the LDS copy of a weight matrix with lane r
// addressing matrix row swap23(r) (bits 2 and 3 of the row exchanged) instead of row r.  With that
// the accumulator register i of row block b on lane (r, gl) holds row
//        32 b + 16 (i / 8) + 8 gl + i % 8
// of the product: eight CONSECUTIVE rows per lane half, which is at once
//   - the order in which a lane loads its token's input channels (one 16-byte piece per k-step),
//   - the k-slot order of the B operand of the next product (packed straight from the registers,
//     its A operand again a plain 16-byte LDS read at natural columns),
//   - the order of a token row in memory (outputs leave as 16-byte pieces, no lane exchange).
// Forward per map:   y^T = (W1^T/4) X^T + b1/4,  g = GELU(4y)/4 (packed fp16),  u^T = (4 W2^T) g^T + b2,
// LayerNorm over the 128 channels of a token = over 64 registers of a lane and its partner lane.
// Backward per map:  dg^T = W2 du^T,  dh = dg * GELU'(4y),  dx^T = W1 dh^T, with the A operands
// read from the same LDS copies by transpose reads.  du is handed to the matrix cores in fp16
// scaled per token to unit Euclidean norm (the scale goes back on dx, which is linear in du), so
// its range does not depend on the size of the upstream gradient or of 1/std.
// The forward keeps the weights of both maps resident in LDS (one workgroup of four waves per
// compute unit); the backward runs one map per launch (two workgroups per unit).  Each wave streams
// its own 32-token tiles.
#include "hla_handle.h"
#include "hla_mfma_common.h"
#include "hla_mfma_gelu.h"

namespace hla {
namespace {

using namespace mf;

// Workgroups of four waves.  The forward keeps both maps' weights in LDS, so one workgroup fits a
// compute unit and a wave has its SIMD, and all 512 registers, to itself: that is what lets it
// hold a tile's intermediate values and the next tile's inputs at once.  The backward runs one
// map per launch, two workgroups per unit, 256 registers per wave.
constexpr int kWavesV = 4;
constexpr int kRowsOut = 16;  // token rows of a wave's output tile in LDS (a tile leaves in 32/16 passes)

// packed weights of one map in global memory
template <int D>
struct VPacked {
  static constexpr int kW1T = 0;                  // bf16 [D][D]: row = hidden unit, col = input channel; times 1/4
  static constexpr int kW2T = kW1T + D * D * 2;   // fp16 [D][D]: row = output channel, col = hidden unit; times 4
  static constexpr int kB1 = kW2T + D * D * 2;    // fp32 [D]; times 1/4
  static constexpr int kB2 = kB1 + D * 4;         // fp32 [D]
  static constexpr int kGamma = kB2 + D * 4;      // fp32 [D]
  static constexpr int kBeta = kGamma + D * 4;    // fp32 [D]
  static constexpr int kW2 = kBeta + D * 4;       // fp16 [D][D]: row = hidden unit, col = output channel; times 4
  static constexpr int kBytes = kW2 + D * D * 2;
};

template <typename T>
__global__ void k_vmod_pack_mfma(const T* W1, const T* b1, const T* W2, const T* b2, const T* gamma,
                                 const T* beta, int d, unsigned char* __restrict__ out) {
  // W1, W2 are [in][out] row-major
  uint16_t* w1t = reinterpret_cast<uint16_t*>(out);
  uint16_t* w2t = w1t + d * d;
  float* vec = reinterpret_cast<float*>(w2t + d * d);
  uint16_t* w2 = reinterpret_cast<uint16_t*>(vec + 4 * d);
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < d * d; i += gridDim.x * blockDim.x) {
    const int row = i / d, col = i % d;  // row = output of the layer, col = its input
    w1t[i] = f32_to_bf16_bits(kHiddenScale * to_float(W1[col * d + row]));
    w2t[i] = __builtin_bit_cast(uint16_t, static_cast<_Float16>(to_float(W2[col * d + row]) / kHiddenScale));
    w2[i] = __builtin_bit_cast(uint16_t, static_cast<_Float16>(to_float(W2[i]) / kHiddenScale));
    if (i < d) {
      vec[i] = kHiddenScale * to_float(b1[i]);
      vec[d + i] = to_float(b2[i]);
      vec[2 * d + i] = to_float(gamma[i]);
      vec[3 * d + i] = to_float(beta[i]);
    }
  }
}

// LDS: per map the two matrices row-major with swizzled 16-byte chunks (tile_off), then the four
// vectors; after the maps one output tile per wave.
template <int D>
struct VSmem {
  static constexpr int kRowB = D * 2;
  static constexpr int kW1 = 0;
  static constexpr int kW2 = D * D * 2;
  static constexpr int kVec = 2 * D * D * 2;   // b1/4, b2, gamma, beta
  static constexpr int kMap = kVec + 4 * D * 4;
  static constexpr int total(int waves) { return 2 * kMap + waves * RowTile<D, kRowsOut>::kBytes; }
};

__host__ __device__ __forceinline__ int swap23(int r) { return (r & ~12) | ((r & 4) << 1) | ((r & 8) >> 1); }

template <int D, int THREADS>
__device__ __forceinline__ void load_map(unsigned char* dst, const unsigned char* src) {
  using SM = VSmem<D>;
  constexpr int CH = D / 8;           // 16-byte chunks per matrix row
  constexpr int NM = 2 * D * CH;      // chunks of both matrices
  constexpr int IT = (NM + THREADS - 1) / THREADS;
  static_assert(NM % THREADS == 0 && D * 4 * 4 / 16 <= THREADS, "copy loops assume whole rounds");
  const int t = threadIdx.x;
  u32x4 v[IT];
#pragma unroll
  for (int k = 0; k < IT; ++k) v[k] = *reinterpret_cast<const u32x4*>(src + (t + k * THREADS) * 16);
  u32x4 vv;
  if (t < D) vv = *reinterpret_cast<const u32x4*>(src + VPacked<D>::kB1 + t * 16);
#pragma unroll
  for (int k = 0; k < IT; ++k) {
    const int i = t + k * THREADS;
    const int mat = i / (D * CH), row = (i / CH) % D, chunk = i % CH;
    *reinterpret_cast<u32x4*>(dst + mat * SM::kW2 + tile_off<SM::kRowB>(row, chunk)) = v[k];
  }
  if (t < D) *reinterpret_cast<u32x4*>(dst + SM::kVec + t * 16) = vv;
}

// the lane's share of a token row as B operands / in accumulator order: one 16-byte piece per
// k-step, channels 16 ks + 8 gl .. + 7.  Rows at or beyond N read the last row.
template <int D>
__device__ __forceinline__ void load_row(const View& X, int b, int h, int n, int N, int gl,
                                         u32x4 (&x)[D / 16]) {
  const bf16_t* row = X.row<const bf16_t>(b, h, n < N ? n : N - 1);
#pragma unroll
  for (int ks = 0; ks < D / 16; ++ks) x[ks] = *reinterpret_cast<const u32x4*>(row + 16 * ks + 8 * gl);
}

// 16 entries of an fp32 vector in LDS in accumulator order of row block rb
__device__ __forceinline__ f32x16 vec_block(const float* v, int rb, int gl) {
  f32x16 z;
#pragma unroll
  for (int hf = 0; hf < 2; ++hf)
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const f32x4 t = *reinterpret_cast<const f32x4*>(v + 32 * rb + 16 * hf + 8 * gl + 4 * q);
      z[8 * hf + 4 * q] = t[0];
      z[8 * hf + 4 * q + 1] = t[1];
      z[8 * hf + 4 * q + 2] = t[2];
      z[8 * hf + 4 * q + 3] = t[3];
    }
  return z;
}

// entry i of a token row held as packed bf16 pieces (register i of block rb <-> piece 2 rb + i / 8)
template <int D>
__device__ __forceinline__ float row_entry(const u32x4 (&x)[D / 16], int rb, int i) {
  const uint32_t p = x[2 * rb + i / 8][(i % 8) / 2];
  return i % 2 ? bf16_hi(p) : bf16_lo(p);
}

// entry i of a vector held as packed fp16 pieces in the same order
template <int D>
__device__ __forceinline__ float half_entry(const u32x4 (&x)[D / 16], int rb, int i) {
  const uint32_t w = x[2 * rb + i / 8][(i % 8) / 2];  // (a bit_cast applied to the element expression itself reads element 0)
  const f16x2 p = __builtin_bit_cast(f16x2, w);
  return static_cast<float>(p[i % 2]);
}

// 16-byte load through a pointer known to be global memory (after a pointer has been passed
// through an asm statement the compiler no longer knows, and would use the slower generic form)
__device__ __forceinline__ u32x4 load_global16(const void* p) {
  typedef const u32x4 __attribute__((address_space(1))) * gptr;
  return *(gptr)(p);
}

// What the forward keeps of a 32-token tile for the backward: the normalised outputs u-hat of the
// two maps in fp16, [map][piece][lane] 16 bytes (lane-private pieces: the backward's lane reads
// what the forward's lane wrote), then the two 1/std per token, [map][lane] fp32.
template <int D>
struct SavedTile {
  static constexpr int kUhat = 2 * (D / 16) * 1024;
  static constexpr int kBytes = kUhat + 2 * 256;
};

// What the backward kernel leaves of map m for the maps' weight gradients when they are asked for: the
// gradient w.r.t. the second layer's output as the matrix cores see it (fp16 [token-heads][D], a token's
// row scaled to norm kRowNorm) and the scale of each token.  The LayerNorm's dgamma = sum over tokens of
// dm * u-hat and dbeta = sum of dm (dm: gradient w.r.t. the map's output) need no array: the kernel adds
// them up per lane as it goes and leaves one partial per workgroup in gb_part
// ([workgroup][dgamma | dbeta][D] floats).
struct VmodFactors {
  uint16_t* t[2];
  float* scale[2];
  float* gb_part;
};

struct TileWalk {
  int tiles_per_row, total, H;
  __device__ __forceinline__ void decode(int t, int& b, int& h, int& n0) const {
    const int row = t / tiles_per_row;
    b = row / H;
    h = row % H;
    n0 = (t % tiles_per_row) * 32;
  }
};

// First layer of one map for hidden block rb: y = h/4 of the 16 hidden units the lane holds.
// All LDS operands are read before the first MFMA is issued (one exposed LDS round trip per
// block instead of one per MFMA).
template <int D>
__device__ __forceinline__ f32x16 first_layer_block(const unsigned char* wm, const int (&a_off)[D / 16], int gl,
                                                    const u32x4 (&x)[D / 16], int rb) {
  using SM = VSmem<D>;
  constexpr int NKS = D / 16;
  u32x4 a[NKS];
#pragma unroll
  for (int ks = 0; ks < NKS; ++ks)
    a[ks] = *reinterpret_cast<const u32x4*>(wm + SM::kW1 + rb * 32 * SM::kRowB + a_off[ks]);
  f32x16 hb = vec_block(reinterpret_cast<const float*>(wm + SM::kVec), rb, gl);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int ks = 0; ks < NKS; ++ks) hb = mfma32(a[ks], x[ks], hb);
  return hb;
}

// One map applied to the token rows in x: on return u holds u-hat (the LayerNorm's normalised
// value, before gamma and beta) in accumulator order, rstd the token's 1/std and, if KEEP, yk the
// first layer's y = h/4 as packed fp16 pairs (pair p of block rb = registers 2p, 2p+1).
// The two layers run as a software pipeline over the 32-row blocks of the hidden layer: in stage
// s the vector ALU evaluates GELU on block s while the matrix cores compute the first layer of
// block s + 1 and the second layer's share of block s - 1.  A wave issues in order and has its
// SIMD to itself, so the overlap needs the two kinds of instructions to alternate in program
// order: a stage is cut into four slices (scheduling barriers in between) of four MFMAs, the LDS
// reads of the next slice's operands and a quarter of the block's GELU.
template <int D, bool KEEP>
__device__ __forceinline__ void map_forward(const unsigned char* wm, const int (&a_off)[D / 16], int gl,
                                            const u32x4 (&x)[D / 16], float ln_eps,
                                            f32x16 (&u)[D / 32], f16x2 (&yk)[KEEP ? D / 32 : 1][8],
                                            float& rstd) {
  using SM = VSmem<D>;
  constexpr int NRB = D / 32, NKS = D / 16;
  constexpr int P1 = NKS / 4;       // first-layer MFMAs per slice
  constexpr int P2 = 2 * NRB / 4;   // second-layer MFMAs per slice
  static_assert(NKS % 4 == 0 && (2 * NRB) % 4 == 0, "four slices per stage");
  const float* vec = reinterpret_cast<const float*>(wm + SM::kVec);
#pragma unroll
  for (int ob = 0; ob < NRB; ++ob) u[ob] = vec_block(vec + D, ob, gl);
  // operand of first-layer MFMA i of slice (s, j): block s + 1, k-step P1 j + i
  auto a1 = [&](int s, int j, int i) {
    return *reinterpret_cast<const u32x4*>(wm + SM::kW1 + (s + 1) * 32 * SM::kRowB + a_off[P1 * j + i]);
  };
  // second-layer MFMA i of slice (s, j) is number n = P2 j + i of block s - 1's 2 NRB products:
  // k-step half n / NRB, output block n % NRB
  auto a2 = [&](int s, int j, int i) {
    const int n = P2 * j + i;
    return *reinterpret_cast<const u32x4*>(wm + SM::kW2 + (n % NRB) * 32 * SM::kRowB + a_off[2 * (s - 1) + n / NRB]);
  };
  f32x16 hb[2];
  hb[0] = first_layer_block<D>(wm, a_off, gl, x, 0);
  u32x4 gprev[2], gcur[2], an1[P1], an2[P2];
#pragma unroll
  for (int i = 0; i < P1; ++i) an1[i] = a1(0, 0, i);
#pragma unroll
  for (int s = 0; s <= NRB; ++s) {
    if (s + 1 < NRB) hb[(s + 1) % 2] = vec_block(vec, s + 1, gl);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      __builtin_amdgcn_sched_barrier(0);
      if (s + 1 < NRB) {
#pragma unroll
        for (int i = 0; i < P1; ++i) hb[(s + 1) % 2] = mfma32(an1[i], x[P1 * j + i], hb[(s + 1) % 2]);
      }
      if (s >= 1) {
#pragma unroll
        for (int i = 0; i < P2; ++i) {
          const int n = P2 * j + i;
          u[n % NRB] = mfma32_f16(an2[i], gprev[n / NRB], u[n % NRB]);
        }
      }
      // operands of the next slice
      const int sn = j < 3 ? s : s + 1, jn = j < 3 ? j + 1 : 0;
      if (sn + 1 < NRB) {
#pragma unroll
        for (int i = 0; i < P1; ++i) an1[i] = a1(sn, jn, i);
      }
      if (sn >= 1 && sn <= NRB) {
#pragma unroll
        for (int i = 0; i < P2; ++i) an2[i] = a2(sn, jn, i);
      }
      if (s < NRB) {  // GELU of entries 4j .. 4j+3 of block s -> two dwords of the B operand
        f16x2 y[2];
        y[0] = to_f16x2(hb[s % 2][4 * j], hb[s % 2][4 * j + 1]);
        y[1] = to_f16x2(hb[s % 2][4 * j + 2], hb[s % 2][4 * j + 3]);
        if (KEEP) {
          yk[s][2 * j] = y[0];
          yk[s][2 * j + 1] = y[1];
        }
        uint32_t gp[2];
        gelu_y16<2>(y, gp);
        gcur[j / 2][2 * (j % 2)] = gp[0];
        gcur[j / 2][2 * (j % 2) + 1] = gp[1];
      }
    }
    gprev[0] = gcur[0];
    gprev[1] = gcur[1];
  }
  __builtin_amdgcn_sched_barrier(0);
  // LayerNorm statistics of the token: this lane's D/2 channels and the partner lane's
  float s = 0.0f;
#pragma unroll
  for (int ob = 0; ob < NRB; ++ob)
#pragma unroll
    for (int i = 0; i < 16; ++i) s += u[ob][i];
  s += partner32(s);
  const float mean = s * (1.0f / D);
  float v = 0.0f;
#pragma unroll
  for (int ob = 0; ob < NRB; ++ob)
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      u[ob][i] -= mean;
      v = __builtin_fmaf(u[ob][i], u[ob][i], v);
    }
  v += partner32(v);
  rstd = 1.0f / sqrtf(v * (1.0f / D) + ln_eps);
#pragma unroll
  for (int ob = 0; ob < NRB; ++ob)
#pragma unroll
    for (int i = 0; i < 16; ++i) u[ob][i] *= rstd;
}

// 16 accumulator entries -> the two 16-byte bf16 pieces of the token row they stand for
__device__ __forceinline__ void pack_block(const f32x16& a, u32x4 (&w)[2]) {
#pragma unroll
  for (int hf = 0; hf < 2; ++hf)
#pragma unroll
    for (int p = 0; p < 4; ++p) w[hf][p] = pack_bf16(a[8 * hf + 2 * p], a[8 * hf + 2 * p + 1]);
}

template <int D, class RowPtr>
__device__ __forceinline__ void store_tile(const u32x4 (&w)[D / 32][2], int lane, unsigned char* lds,
                                           RowPtr&& row_ptr) {
#pragma unroll
  for (int pass = 0; pass < 32 / kRowsOut; ++pass) {
    put_rows<D, kRowsOut>(w, pass, lane, lds);
    flush_rows<D, kRowsOut>(pass, lane, lds, row_ptr);
  }
}

template <int D>
__device__ __forceinline__ void first_layer_offsets(int lane, int (&a_off)[D / 16]) {
  const int r = lane % 32, gl = lane / 32;
#pragma unroll
  for (int ks = 0; ks < D / 16; ++ks) a_off[ks] = tile_off<D * 2>(swap23(r), 2 * ks + gl);
}

// grid: one workgroup per compute unit, block WAVES*64.  Tin holds T; O receives T + phi_v1(T) * phi_v2(V).
template <int D, int WAVES>
__global__ __launch_bounds__(WAVES * 64) void k_vmod_fwd_mfma(Geom g, const unsigned char* __restrict__ wpk,
                                                              float ln_eps, View Tin, View V, View O,
                                                              unsigned char* __restrict__ saved) {
  using SM = VSmem<D>;
  constexpr int NRB = D / 32, NKS = D / 16;
  extern __shared__ __align__(16) unsigned char smem[];
  const int lane = threadIdx.x % kWave, wave = wave_index();
  const int r = lane % 32, gl = lane / 32;
  load_map<D, WAVES * 64>(smem, wpk);
  load_map<D, WAVES * 64>(smem + SM::kMap, wpk + VPacked<D>::kBytes);
  __syncthreads();
  unsigned char* otile = smem + 2 * SM::kMap + wave * RowTile<D, kRowsOut>::kBytes;
  int a_off[NKS];
  first_layer_offsets<D>(lane, a_off);
  TileWalk tw;
  tw.tiles_per_row = (g.N + 31) / 32;
  tw.total = tw.tiles_per_row * g.B * g.H;
  tw.H = g.H;
  const int stride = gridDim.x * WAVES;
  // u-hat and 1/std of map m for the backward (see SavedTile)
  auto save = [&](int tile_index, int m, const f32x16 (&u)[NRB], float rstd) {
    unsigned char* slot = saved + static_cast<int64_t>(tile_index) * SavedTile<D>::kBytes;
#pragma unroll
    for (int ob = 0; ob < NRB; ++ob)
#pragma unroll
      for (int hf = 0; hf < 2; ++hf) {
        u32x4 v;
#pragma unroll
        for (int p = 0; p < 4; ++p)
          v[p] = __builtin_bit_cast(uint32_t, to_f16x2(u[ob][8 * hf + 2 * p], u[ob][8 * hf + 2 * p + 1]));
        __builtin_nontemporal_store(v, reinterpret_cast<u32x4*>(slot + (m * NKS + 2 * ob + hf) * 1024 + lane * 16));
      }
    *reinterpret_cast<float*>(slot + SavedTile<D>::kUhat + m * 256 + lane * 4) = rstd;
  };
  // The value map runs first: its input rows were requested during the previous tile, the rows
  // of T are requested at the top of the tile and needed only after it, and the next tile's V
  // rows are requested once the value map is done with the registers -- no wait of the tile
  // loop sits right behind its load, and the tile's stores have a whole map to complete before
  // the next wait on the memory counter.
  int tile = blockIdx.x * WAVES + wave;
  int b = 0, h = 0, n0 = 0;
  u32x4 xv[NKS];
  if (tile < tw.total) {
    tw.decode(tile, b, h, n0);
    load_row<D>(V, b, h, n0 + r, g.N, gl, xv);
  }
  for (; tile < tw.total; tile += stride) {
    u32x4 xt[NKS];
    load_row<D>(Tin, b, h, n0 + r, g.N, gl, xt);
    const int ob_ = b, oh_ = h, on0 = n0;
    f16x2 none[1][8];
    u32x4 m2p[NKS];  // phi_v2(V), packed bf16 in token-row order
    {
      f32x16 m2[NRB];
      float rstd;
      map_forward<D, false>(smem + SM::kMap, a_off, gl, xv, ln_eps, m2, none, rstd);
      save(tile, 1, m2, rstd);
      const float* vec = reinterpret_cast<const float*>(smem + SM::kMap + SM::kVec);
#pragma unroll
      for (int ob = 0; ob < NRB; ++ob) {
        const f32x16 ga = vec_block(vec + 2 * D, ob, gl), be = vec_block(vec + 3 * D, ob, gl);
        f32x16 o;
#pragma unroll
        for (int i = 0; i < 16; ++i) o[i] = __builtin_fmaf(m2[ob][i], ga[i], be[i]);
        u32x4 pk[2];
        pack_block(o, pk);
        m2p[2 * ob] = pk[0];
        m2p[2 * ob + 1] = pk[1];
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    if (tile + stride < tw.total) {
      tw.decode(tile + stride, b, h, n0);
      load_row<D>(V, b, h, n0 + r, g.N, gl, xv);
    }
    f32x16 m1[NRB];
    float rstd;
    map_forward<D, false>(smem, a_off, gl, xt, ln_eps, m1, none, rstd);
    save(tile, 0, m1, rstd);
    __builtin_amdgcn_sched_barrier(0);
    u32x4 w[NRB][2];
    {
      const float* vec = reinterpret_cast<const float*>(smem + SM::kVec);
#pragma unroll
      for (int ob = 0; ob < NRB; ++ob) {
        const f32x16 ga = vec_block(vec + 2 * D, ob, gl), be = vec_block(vec + 3 * D, ob, gl);
        f32x16 o;
#pragma unroll
        for (int i = 0; i < 16; ++i)
          o[i] = __builtin_fmaf(__builtin_fmaf(m1[ob][i], ga[i], be[i]), row_entry<D>(m2p, ob, i), row_entry<D>(xt, ob, i));
        pack_block(o, w[ob]);
      }
    }
    store_tile<D>(w, lane, otile, [&](int t) -> bf16_t* {
      return on0 + t < g.N ? O.row<bf16_t>(ob_, oh_, on0 + t) : nullptr;
    });
  }
}

// LayerNorm backward of one map for the lane's token, ready for the matrix cores.  With
// gg = dO * m_other * gamma (m_other = the other map's output) and means over the channels,
//   du = rstd (gg - mean(gg) - u-hat mean(gg u-hat)).
// Returns t = kRowNorm (gg - mean(gg) - u-hat mean(gg u-hat)) / |gg|_2 as packed fp16 B operands (k-slot =
// channel) and the factor rstd |gg|_2 / kRowNorm that dx must be multiplied with: scaled to one
// Euclidean norm per token, the operand's range does not depend on the size of dO or of 1/std.  The norm is
// 1024, so that channels down to 2^-24 of a row's norm are normal fp16 numbers.
constexpr float kRowNorm = 1024.0f;
// The row is streamed twice, 16-byte piece by piece (first for the three sums, then for the
// result), through `load(which, ks, pass)`: piece ks of dO (which = 0, packed bf16), of this map's
// u-hat (1) and of the other map's (2, both packed fp16).  Only the result stays in registers; the
// second pass must really load again (its loader is handed pass = 1 so that it can use an address
// the compiler cannot match with the first pass's).
// fT: this lane's token row of that factor array (see VmodFactors; + 8 gl already applied), or
// nullptr.  ag / ab (D / 2 entries; 1 entry: no sums wanted): the lane's running sums of dm * u-hat and of dm over its
// tokens, entry 8 ks + j for channel 16 ks + 8 gl + j; `live` is 1 for a token of the sequence
// and 0 for the padding of a ragged tile, whose rows must not be counted.
template <int D, int NA, class Load>
__device__ __forceinline__ float norm_backward(const unsigned char* wm_self, const unsigned char* wm_other,
                                               int gl, Load&& load, float rstd, u32x4 (&dub)[D / 16],
                                               uint16_t* fT, float (&ag)[NA], float (&ab)[NA], float live) {
  static_assert(NA == D / 2 || NA == 1, "the lane's 64 channels, or no sums wanted");
  using SM = VSmem<D>;
  constexpr int NKS = D / 16;
  // a pass requests all its pieces before it looks at the first one: one memory round trip per
  // pass instead of one per piece
  u32x4 dd[NKS], ss[NKS], oo[NKS];
  auto request = [&](int pass) {
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) {
      dd[ks] = load(0, ks, pass);
      ss[ks] = load(1, ks, pass);
      oo[ks] = load(2, ks, pass);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  auto piece = [&](int ks, int pass, int opaque, float (&gg)[8], float (&uh)[8], float (&dmv)[8]) {
    const u32x4 d = dd[ks], s = ss[ks], o = oo[ks];
    const float* vs = reinterpret_cast<const float*>(wm_self + SM::kVec) + opaque + 16 * ks + 8 * gl;
    const float* vo = reinterpret_cast<const float*>(wm_other + SM::kVec) + opaque + 16 * ks + 8 * gl;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const f32x4 gs = *reinterpret_cast<const f32x4*>(vs + 2 * D + 4 * q);
      const f32x4 go = *reinterpret_cast<const f32x4*>(vo + 2 * D + 4 * q);
      const f32x4 bo = *reinterpret_cast<const f32x4*>(vo + 3 * D + 4 * q);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int j = 4 * q + e;
        const uint32_t dw = d[j / 2], sw = s[j / 2], ow = o[j / 2];
        const f16x2 sp = __builtin_bit_cast(f16x2, sw), op = __builtin_bit_cast(f16x2, ow);
        const float mo = __builtin_fmaf(static_cast<float>(op[j % 2]), go[e], bo[e]);
        dmv[j] = (j % 2 ? bf16_hi(dw) : bf16_lo(dw)) * mo;
        gg[j] = dmv[j] * gs[e];
        uh[j] = static_cast<float>(sp[j % 2]);
      }
    }
  };
  float sa = 0.0f, sb = 0.0f, sc = 0.0f;
  int z1 = 0, z2 = 0;  // zeros the compiler cannot see through: the LDS vectors are read again, too
  asm volatile("" : "+s"(z1));
  request(0);
#pragma unroll
  for (int ks = 0; ks < NKS; ++ks) {
    float gg[8], uh[8], dmv[8];
    piece(ks, 0, z1, gg, uh, dmv);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      sa += gg[j];
      sb = __builtin_fmaf(gg[j], uh[j], sb);
      sc = __builtin_fmaf(gg[j], gg[j], sc);
    }
  }
  sa += partner32(sa);
  sb += partner32(sb);
  sc += partner32(sc);
  const float nrm = sqrtf(sc);
  const float inv = nrm > 0.0f ? kRowNorm / nrm : 0.0f;
  const float a = sa * (1.0f / D) * inv, bq = sb * (1.0f / D) * inv;
  asm volatile("" : "+s"(z2));
  __builtin_amdgcn_sched_barrier(0);
  request(1);
#pragma unroll
  for (int ks = 0; ks < NKS; ++ks) {
    float gg[8], uh[8], dmv[8], tv[8];
    piece(ks, 1, z2, gg, uh, dmv);
#pragma unroll
    for (int j = 0; j < 8; ++j) tv[j] = __builtin_fmaf(gg[j], inv, -a) - uh[j] * bq;
#pragma unroll
    for (int p = 0; p < 4; ++p) dub[ks][p] = __builtin_bit_cast(uint32_t, to_f16x2(tv[2 * p], tv[2 * p + 1]));
    if (fT != nullptr) *reinterpret_cast<u32x4*>(fT + 16 * ks) = dub[ks];
    if constexpr (NA == D / 2) {
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const float dl = dmv[j] * live;
        ab[8 * ks + j] += dl;
        ag[8 * ks + j] = __builtin_fmaf(dl, uh[j], ag[8 * ks + j]);
      }
    }
  }
  return rstd * nrm * (1.0f / kRowNorm);
}

// dx^T = W1 (GELU'(4y) * (W2 du^T)) for one map: dub = du as fp16 B operands, x = the map's input
// rows (the first layer is computed again, block by block).
// Per 32-row block of the hidden layer: y and dg (NKS MFMAs each, the operands of dg by transpose
// reads, all requested up front), GELU' and the product on the vector ALU, then the block's share
// of dx.
template <int D>
__device__ __forceinline__ void map_backward(const unsigned char* wm, const int (&a_off)[D / 16],
                                             const int (&t_off)[2][D / 32], int gl,
                                             const u32x4 (&x)[D / 16], const u32x4 (&dub)[D / 16],
                                             f32x16 (&dx)[D / 32]) {
  using SM = VSmem<D>;
  constexpr int NRB = D / 32, NKS = D / 16;
  auto tr_operand = [&](const unsigned char* mat, int blk, int ks) {
    const u32x2 lo = lds_read_tr16(mat + ks * 16 * SM::kRowB + t_off[0][blk]);
    const u32x2 hi = lds_read_tr16(mat + ks * 16 * SM::kRowB + t_off[1][blk]);
    u32x4 a;
    a[0] = lo[0];
    a[1] = lo[1];
    a[2] = hi[0];
    a[3] = hi[1];
    return a;
  };
#pragma unroll
  for (int ib = 0; ib < NRB; ++ib)
#pragma unroll
    for (int i = 0; i < 16; ++i) dx[ib][i] = 0.0f;
  u32x4 ag[NKS];
#pragma unroll
  for (int ks = 0; ks < NKS; ++ks) ag[ks] = tr_operand(wm + SM::kW2, 0, ks);
#pragma unroll
  for (int hb = 0; hb < NRB; ++hb) {
    __builtin_amdgcn_sched_barrier(0);
    // y (first layer again) and dg are two chains of NKS dependent MFMAs each: issued alternately,
    // one fills the other's latency
    u32x4 a1[NKS];
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks)
      a1[ks] = *reinterpret_cast<const u32x4*>(wm + SM::kW1 + hb * 32 * SM::kRowB + a_off[ks]);
    f32x16 yb = vec_block(reinterpret_cast<const float*>(wm + SM::kVec), hb, gl);
    f32x16 dg;
#pragma unroll
    for (int i = 0; i < 16; ++i) dg[i] = 0.0f;
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) {
      yb = mfma32(a1[ks], x[ks], yb);
      dg = mfma32_f16(ag[ks], dub[ks], dg);
    }
    u32x4 ax[2][NRB];
#pragma unroll
    for (int hf = 0; hf < 2; ++hf)
#pragma unroll
      for (int ib = 0; ib < NRB; ++ib) ax[hf][ib] = tr_operand(wm + SM::kW1, ib, 2 * hb + hf);
    __builtin_amdgcn_sched_barrier(0);
    f16x2 y[8], gp[8];
#pragma unroll
    for (int p = 0; p < 8; ++p) y[p] = to_f16x2(yb[2 * p], yb[2 * p + 1]);
    gelu_grad_y16<8>(y, gp);  // eight independent chains in lockstep: no issue slot waits for its predecessor
    u32x4 dhb[2];
#pragma unroll
    for (int p = 0; p < 8; ++p)
      dhb[p / 4][p % 4] = pack_bf16(static_cast<float>(gp[p][0]) * dg[2 * p], static_cast<float>(gp[p][1]) * dg[2 * p + 1]);
    if (hb + 1 < NRB) {
#pragma unroll
      for (int ks = 0; ks < NKS; ++ks) ag[ks] = tr_operand(wm + SM::kW2, hb + 1, ks);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int hf = 0; hf < 2; ++hf)
#pragma unroll
      for (int ib = 0; ib < NRB; ++ib) dx[ib] = mfma32(ax[hf][ib], dhb[hf], dx[ib]);
  }
  __builtin_amdgcn_sched_barrier(0);
}

// The backward of ONE map per launch (MAP 0: dT = dO + phi_v1'(T)^T (dO * phi_v2(V)), written to dT;
// MAP 1: dV += phi_v2'(V)^T (dO * phi_v1(T)), added to the rows the operator's backward has written).
// Only that map's matrices are in LDS (plus the other map's gamma, beta), so two workgroups share
// a compute unit and one wave's memory and matrix-pipe waits are filled by another's arithmetic.
constexpr int kRowsOutB = 8;
template <int D>
struct VSmemB {
  static constexpr int kOtherVec = VSmem<D>::kMap;            // the other map's four vectors
  static constexpr int kTiles = kOtherVec + 4 * D * 4;
  static constexpr int total(int waves) { return kTiles + waves * RowTile<D, kRowsOutB>::kBytes; }
  // the factor-writing form ends with the sums of dgamma and dbeta over lanes and waves: a
  // [D][33] float tile per wave and 2 x D floats per wave (one workgroup per compute unit)
  static constexpr int kSumTile = D * 33;
  static constexpr int total_factors(int waves) {
    const int sums = (waves * kSumTile + 2 * waves * D) * 4;
    return sums > total(waves) ? sums : total(waves);
  }
};
template <int D, int WAVES, bool FACTORS, int MAP>
__global__ __launch_bounds__(WAVES * 64, FACTORS ? 1 : 2) void k_vmod_bwd_map(Geom g, const unsigned char* __restrict__ wpk,
                                                             View Tin, View V, View dO, View out,
                                                             const unsigned char* __restrict__ saved,
                                                             VmodFactors fac) {
  using SM = VSmem<D>;
  using SB = VSmemB<D>;
  constexpr int NRB = D / 32, NKS = D / 16;
  extern __shared__ __align__(16) unsigned char smem[];
  const int lane = threadIdx.x % kWave, wave = wave_index();
  const int r = lane % 32, gl = lane / 32;
  const int L = lane % 16, q = lane / 16;
  load_map<D, WAVES * 64>(smem, wpk + MAP * VPacked<D>::kBytes);
  if (threadIdx.x < D)
    *reinterpret_cast<u32x4*>(smem + SB::kOtherVec + threadIdx.x * 16) =
        *reinterpret_cast<const u32x4*>(wpk + (1 - MAP) * VPacked<D>::kBytes + VPacked<D>::kB1 + threadIdx.x * 16);
  __syncthreads();
  const unsigned char* wm_other = smem + SB::kOtherVec - SM::kVec;  // only its vectors are there
  unsigned char* otile = smem + SB::kTiles + wave * RowTile<D, kRowsOutB>::kBytes;
  int a_off[NKS];
  first_layer_offsets<D>(lane, a_off);
  // Transpose reads of a [k][m] matrix copy (row = contraction index, 16 per k-step: slot (gl, j)
  // is row 8 gl + j) for the lane's A operand row: lanes 4j'..4j'+3 of a 16-lane group supply row
  // j' of a 4 x 16 block, and lane L receives its column L, which is to be matrix column
  // 32 blk + 16 (q % 2) + swap23(L): the lane that supplies block columns 4c..4c+3 therefore
  // addresses the matrix columns of group c with its two bits exchanged.
  int t_off[2][NRB];
#pragma unroll
  for (int hi = 0; hi < 2; ++hi)
#pragma unroll
    for (int blk = 0; blk < NRB; ++blk) {
      const int c = L % 4, cs = ((c & 1) << 1) | (c >> 1);
      const int row = 8 * gl + 4 * hi + L / 4;
      const int col = 32 * blk + 16 * (q % 2) + 4 * cs;
      t_off[hi][blk] = tile_off<SM::kRowB>(row, col >> 3) + ((col & 7) << 1);
    }
  TileWalk tw;
  tw.tiles_per_row = (g.N + 31) / 32;
  tw.total = tw.tiles_per_row * g.B * g.H;
  tw.H = g.H;
  const int stride = gridDim.x * WAVES;
  const int lane16 = lane * 16;
  const View& X = MAP == 0 ? Tin : V;
  // FACTORS: the lane's sums of dm * u-hat and of dm over its tokens (see norm_backward)
  float ag[FACTORS ? D / 2 : 1], ab[FACTORS ? D / 2 : 1];
#pragma unroll
  for (int i = 0; i < (FACTORS ? D / 2 : 1); ++i) ag[i] = ab[i] = 0.0f;
  for (int tile = blockIdx.x * WAVES + wave; tile < tw.total; tile += stride) {
    int b, h, n0;
    tw.decode(tile, b, h, n0);
    const unsigned char* slot_rd[2] = {saved + static_cast<int64_t>(tile) * SavedTile<D>::kBytes, nullptr};
    slot_rd[1] = slot_rd[0];
    asm volatile("" : "+s"(slot_rd[1]));
    const float rstd = *reinterpret_cast<const float*>(slot_rd[0] + SavedTile<D>::kUhat + MAP * 256 + lane * 4);
    const bf16_t* drow[2] = {dO.row<const bf16_t>(b, h, n0 + r < g.N ? n0 + r : g.N - 1) + 8 * gl, nullptr};
    drow[1] = drow[0];
    asm volatile("" : "+v"(drow[1]));
    auto loader = [&](int which, int ks, int pass) -> u32x4 {
      if (which == 0) return load_global16(drow[pass] + 16 * ks);
      const int m = which == 1 ? MAP : 1 - MAP;
      return load_global16(slot_rd[pass] + (m * NKS + ks) * 1024 + lane16);
    };
    const int64_t frow = FACTORS && n0 + r < g.N ? g.th(b, h, n0 + r) : -1;
    u32x4 x[NKS];  // the map's input rows, for the first layer's recomputation
    load_row<D>(X, b, h, n0 + r, g.N, gl, x);
    u32x4 du[NKS];
    const float sc = norm_backward<D>(smem, wm_other, gl, loader, rstd, du,
                                      FACTORS && frow >= 0 ? fac.t[MAP] + frow * D + 8 * gl : nullptr, ag, ab,
                                      frow >= 0 ? 1.0f : 0.0f);
    if (FACTORS && frow >= 0 && gl == 0) fac.scale[MAP][frow] = sc;
    __builtin_amdgcn_sched_barrier(0);
    f32x16 dx[NRB];
    map_backward<D>(smem, a_off, t_off, gl, x, du, dx);
    __builtin_amdgcn_sched_barrier(0);
    // what the result is added to: dO (MAP 0) or the operator's own dV (MAP 1), this lane's row
    load_row<D>(MAP == 0 ? dO : out, b, h, n0 + r, g.N, gl, x);
    u32x4 w[NRB][2];
#pragma unroll
    for (int ib = 0; ib < NRB; ++ib) {
      f32x16 o;
#pragma unroll
      for (int i = 0; i < 16; ++i) o[i] = __builtin_fmaf(dx[ib][i], sc, row_entry<D>(x, ib, i));
      pack_block(o, w[ib]);
    }
#pragma unroll
    for (int pass = 0; pass < 32 / kRowsOutB; ++pass) {
      put_rows<D, kRowsOutB>(w, pass, lane, otile);
      flush_rows<D, kRowsOutB>(pass, lane, otile, [&](int t) -> bf16_t* {
        return n0 + t < g.N ? out.row<bf16_t>(b, h, n0 + t) : nullptr;
      });
    }
  }
  if constexpr (FACTORS) {
    // The workgroup's share of dgamma and dbeta: per wave the 32 token lanes of a channel are added
    // in lane order through a [channel][33] LDS tile (the weights are done with), then the four
    // waves in wave order; one partial per workgroup.
    constexpr int kTile = SB::kSumTile;
    __syncthreads();
    float* red = reinterpret_cast<float*>(smem) + wave * kTile;
    float* wsum = reinterpret_cast<float*>(smem) + WAVES * kTile;  // [2][WAVES][D]
    auto wave_sum = [&](const float (&src)[FACTORS ? D / 2 : 1], int which) {
#pragma unroll
      for (int i = 0; i < D / 2; ++i) red[(16 * (i / 8) + 8 * gl + i % 8) * 33 + r] = src[i];
      wave_lds_sync();
      for (int c = lane; c < D; c += kWave) {
        float sum = 0.0f;
#pragma unroll
        for (int k = 0; k < 32; ++k) sum += red[c * 33 + k];
        wsum[(which * WAVES + wave) * D + c] = sum;
      }
      wave_lds_sync();
    };
    wave_sum(ag, 0);
    wave_sum(ab, 1);
    __syncthreads();
    for (int i = threadIdx.x; i < 2 * D; i += WAVES * 64) {
      const int which = i / D, c = i % D;
      float sum = wsum[(which * WAVES) * D + c];
#pragma unroll
      for (int w = 1; w < WAVES; ++w) sum += wsum[(which * WAVES + w) * D + c];
      fac.gb_part[(static_cast<int64_t>(blockIdx.x) * 2 + which) * D + c] = sum;
    }
  }
}

// Adds the `nparts` per-workgroup partials of dgamma and dbeta (see VmodFactors) in order: eight
// slices of the partials per output, each with sixteen loads in flight, then the slices in order.
// grid (2 D / 32), block 256.
__global__ __launch_bounds__(256) void k_vmod_gb_reduce(const float* __restrict__ part, int nparts, int D,
                                                        float* __restrict__ dgamma, float* __restrict__ dbeta) {
  __shared__ float sh[8][32];
  const int o = blockIdx.x * 32 + threadIdx.x % 32, slice = threadIdx.x / 32;  // o = which * D + c
  const int per = (nparts + 7) / 8;
  const int p0 = slice * per, p1 = p0 + per < nparts ? p0 + per : nparts;
  float sum = 0.0f;
  for (int p = p0; p < p1; p += 16) {
    float ld[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) ld[k] = p + k < p1 ? part[static_cast<int64_t>(p + k) * 2 * D + o] : 0.0f;
#pragma unroll
    for (int k = 0; k < 16; ++k) sum += ld[k];
  }
  sh[slice][threadIdx.x % 32] = sum;
  __syncthreads();
  if (slice == 0) {
    float t = sh[0][threadIdx.x];
#pragma unroll
    for (int k = 1; k < 8; ++k) t += sh[k][threadIdx.x];
    (o < D ? dgamma : dbeta)[o % D] = t;
  }
}

// ---- weight gradients of the two layers ---------------------------------------------------------------
// With y the first layer's output / 4, t and s what the backward kernel left of a token (see VmodFactors):
//   dU = s t,  dH = GELU'(4y) * s (t W2^T),  G = GELU(4y):
//   dW1 = X^T dH, db1 = sum dH, dW2 = (s G)^T t, db2 = sum dU       (sums over all tokens)
// t is contracted as it stands: forming dU in 16 bits would round it a second time.  s G goes into fp16 in
// units of 2^e, e the exponent of the largest scale a wave has met: the sums are rescaled where a larger one
// turns up, and a token is rounded to nothing only 2^-24 below it.
// for map blockIdx.y.  A token is an MFMA row here (as in the feature maps' weight gradients): the
// hidden layer leaves its unit in a lane and its tokens in the accumulator registers, which is the
// operand the contractions over tokens want, so dH and G never leave the registers.
// Waves w and w + 4 share a SIMD and a block of 32 hidden units whose weights they keep in registers;
// the first forms dH and dW1, the second G and dW2 (both compute the block's first layer).  The 64-token
// tiles of X and t are shared by the waves of a group in LDS, two buffers, loaded through
// registers a tile ahead; one barrier per tile.  A group (512 threads at D = 128, 256 at D = 64) ends
// with one partial: [dW1 (in, hidden) | dW2 transposed (out, hidden) | db1 | db2] floats.
// With the backward writing dU, dH and G and a kernel that contracted them from memory (each array read
// twice), a map cost 242 us in the backward, and the contractions and their sums 214 + 22 us, at 12 heads
// x 32760 tokens x 128 channels; now 193 a map, 188 + 7.  No unit is busy more than half of the time: a
// wave's LDS reads, matrix chain, GELU and second chain follow each other, and two waves share a SIMD.
// Bringing the tiles in by the waves of one role only (the other then has registers to spare): 206.
template <int D>
struct VWgSmem {
  static constexpr int kTok = 64;
  static constexpr int kRows = kTok * D * 2;                   // one tile of one array
  static constexpr int kScale = 2 * kRows;                     // X, t, then the tokens' scales
  static constexpr int kBuf = kScale + kTok * 4;
  static constexpr int kGroups = 128 / D;
  static constexpr int kTotal = kGroups * 2 * kBuf;
  static constexpr int kPart = 2 * D * D + 2 * D;              // floats of a partial
};
constexpr int kWgBlocks = 128;  // workgroups per map; with two maps one per compute unit of the card's 256

template <int D>
__global__ __launch_bounds__(512, 2) void k_vmod_wgrad(Geom g, const unsigned char* __restrict__ wpk, View Tin, View V,
                                                       VmodFactors fac, float* __restrict__ part) {
  using SM = VWgSmem<D>;
  using PK = VPacked<D>;
  constexpr int NRB = D / 32, NKS = D / 16, kPieces = D / 8, kThreads = 2 * NRB * 64;  // of a group
  static_assert(SM::kTok * kPieces == 2 * kThreads, "two 16-byte pieces of a tile per thread");
  extern __shared__ __align__(256) unsigned char smem[];
  const int lane = threadIdx.x % kWave, wave = wave_index();
  const int r = lane % 32, gl = lane / 32;
  const int L = lane % 16, q = lane / 16;
  const int role = wave / 4, grp = wave % 4 / NRB, hb = wave % NRB;
  const int m = blockIdx.y;
  unsigned char* bufs = smem + grp * 2 * SM::kBuf;
  const unsigned char* wm = wpk + m * PK::kBytes;
  const View& X = m == 0 ? Tin : V;
  const uint16_t* __restrict__ tarr = fac.t[m];
  const float* __restrict__ sarr = fac.scale[m];
  // rows 32 hb + r of W1^T or W2, k-slot (ks, gl, j) = column 16 ks + 8 gl + j
  auto weight_rows = [&](int mat, u32x4 (&w)[NKS]) {
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks)
      w[ks] = *reinterpret_cast<const u32x4*>(wm + mat + ((32 * hb + r) * D + 16 * ks + 8 * gl) * 2);
  };
  u32x4 w1b[NKS];
  weight_rows(PK::kW1T, w1b);
  const float bias = *reinterpret_cast<const float*>(wm + PK::kB1 + (32 * hb + r) * 4);
  // this thread's share of a tile: 16-byte piece `piece` of tokens tok and tok + 32
  const int tid = (role * NRB + hb) * 64 + lane, piece = tid % kPieces, tok = tid / kPieces;
  const int tpr = (g.N + SM::kTok - 1) / SM::kTok;
  const int total = tpr * g.B * g.H;
  u32x4 xr[2], tr[2];
  float sr[2];
  float db2[8];  // of channels 8 piece .. + 7, over this thread's tokens
#pragma unroll
  for (int e = 0; e < 8; ++e) db2[e] = 0.0f;
  auto fetch = [&](int tile) {  // every address is valid; what must not count has scale and t zero
    const int tc = tile < total ? tile : total - 1;
    const int row = tc / tpr, n0 = (tc % tpr) * SM::kTok, b = row / g.H, h = row % g.H;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const int n = n0 + tok + 32 * k, nc = n < g.N ? n : g.N - 1;
      const int64_t th = g.th(b, h, nc);
      xr[k] = *reinterpret_cast<const u32x4*>(X.row<const bf16_t>(b, h, nc) + 8 * piece);
      tr[k] = *reinterpret_cast<const u32x4*>(tarr + th * D + 8 * piece);
      sr[k] = sarr[th];
    }
  };
  auto put = [&](int tile, unsigned char* buf) {
    const int n0 = (tile % tpr) * SM::kTok;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const int t = tok + 32 * k, at = tile_off<D * 2>(t, piece);
      const bool live = tile < total && n0 + t < g.N;
      u32x4 tv = tr[k];
      const float sv = live ? sr[k] : 0.0f;
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        if (!live) tv[p] = 0u;
        const uint32_t w = tv[p];
        const f16x2 t2 = __builtin_bit_cast(f16x2, w);
        db2[2 * p] += static_cast<float>(t2[0]) * sv;
        db2[2 * p + 1] += static_cast<float>(t2[1]) * sv;
      }
      *reinterpret_cast<u32x4*>(buf + at) = xr[k];
      *reinterpret_cast<u32x4*>(buf + SM::kRows + at) = tv;
      if (piece == 0) *reinterpret_cast<float*>(buf + SM::kScale + t * 4) = sv;
    }
  };
  // LDS addresses: row r, chunk 2 ks + gl of the layers' operands; transpose reads whose k-slot (gl, j) of
  // step ks is token 16 ks + 8 (j / 4) + 4 gl + j % 4, the order the accumulators hold
  int a_off[NKS], t_off[2][NRB];
#pragma unroll
  for (int ks = 0; ks < NKS; ++ks) a_off[ks] = tile_off<D * 2>(r, 2 * ks + gl);
#pragma unroll
  for (int hi = 0; hi < 2; ++hi)
#pragma unroll
    for (int ib = 0; ib < NRB; ++ib) {
      const int row = 4 * gl + 8 * hi + L / 4, col = 32 * ib + 16 * (q % 2) + 4 * (L % 4);
      t_off[hi][ib] = tile_off<D * 2>(row, col >> 3) + ((col & 7) << 1);
    }
  f32x16 acc[NRB];  // role 0: dW1 rows 32 ib + d_row(i, gl), role 1: dW2^T rows, column 32 hb + r
  float db1 = 0.0f;
#pragma unroll
  for (int ib = 0; ib < NRB; ++ib)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[ib][i] = 0.0f;
  int e2 = -1000;  // role 1: the sums are in units of 2^e2
  // acc += (rows of `tile` transposed) * v over the 32 tokens of a sub-tile, bf16 (X, dH) or fp16 (t, s G)
  auto contract = [&](auto BF16, const unsigned char* tile, const u32x4 (&v)[2]) {
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      u32x4 a[NRB];
      __builtin_amdgcn_sched_barrier(0);  // no operand read early: registers are short
#pragma unroll
      for (int ib = 0; ib < NRB; ++ib) {
        const u32x2 lo = lds_read_tr16(tile + 16 * ks * D * 2 + t_off[0][ib]), hi = lds_read_tr16(tile + 16 * ks * D * 2 + t_off[1][ib]);
        a[ib][0] = lo[0];
        a[ib][1] = lo[1];
        a[ib][2] = hi[0];
        a[ib][3] = hi[1];
      }
#pragma unroll
      for (int ib = 0; ib < NRB; ++ib)
        acc[ib] = BF16.value ? mfma32(a[ib], v[ks], acc[ib]) : mfma32_f16(a[ib], v[ks], acc[ib]);
    }
  };
  auto first_layer = [&](const unsigned char* xs) {
    f32x16 y;
    float bv = bias;
    asm volatile("" : "+v"(bv));  // else the sixteen copies are kept in registers across the loop
#pragma unroll
    for (int i = 0; i < 16; ++i) y[i] = bv;
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) y = mfma32(*reinterpret_cast<const u32x4*>(xs + a_off[ks]), w1b[ks], y);
    return y;
  };
  const int step = gridDim.x * SM::kGroups, first = blockIdx.x * SM::kGroups;
  const int iters = (total - first + step - 1) / step;  // of group 0, which has the most
  // the loop over tiles of one role: code of its own for each, so that a role pays for its own registers only
  auto run = [&](auto DH) {
    int tile = first + grp;
    u32x4 w2b[NKS];
    if constexpr (DH.value) weight_rows(PK::kW2, w2b);
    fetch(tile);
    put(tile, bufs);
    fetch(tile + step);
    __syncthreads();
    for (int it = 0; it < iters; ++it, tile += step) {
      const unsigned char* buf = bufs + (it % 2) * SM::kBuf;
#pragma unroll 1
      for (int sub = 0; sub < 2; ++sub) {
        const unsigned char* xs = buf + sub * 32 * D * 2;
        const unsigned char* ts = xs + SM::kRows;
        f32x4 sc[4];  // of tokens 8 i + 4 gl + 0 .. 3
        auto scales = [&]() {
#pragma unroll
          for (int i = 0; i < 4; ++i) sc[i] = *reinterpret_cast<const f32x4*>(buf + SM::kScale + (32 * sub + 8 * i + 4 * gl) * 4);
        };
        u32x4 v[2];
        if constexpr (DH.value) {
          f32x16 dg;
#pragma unroll
          for (int i = 0; i < 16; ++i) dg[i] = 0.0f;
#pragma unroll
          for (int ks = 0; ks < NKS; ++ks) dg = mfma32_f16(*reinterpret_cast<const u32x4*>(ts + a_off[ks]), w2b[ks], dg);
          asm volatile("" : "+v"(dg) : : "memory");  // the first layer's operands are read after this: registers are short
          const f32x16 y = first_layer(xs);
          __builtin_amdgcn_sched_barrier(0);
          scales();
          f16x2 yh[8], gp[8];
#pragma unroll
          for (int p = 0; p < 8; ++p) yh[p] = to_f16x2(y[2 * p], y[2 * p + 1]);
          gelu_grad_y16<8>(yh, gp);
#pragma unroll
          for (int p = 0; p < 8; ++p) {
            const float d0 = static_cast<float>(gp[p][0]) * (dg[2 * p] * sc[p / 2][2 * (p % 2)]);
            const float d1 = static_cast<float>(gp[p][1]) * (dg[2 * p + 1] * sc[p / 2][2 * (p % 2) + 1]);
            db1 += d0 + d1;
            v[p / 4][p % 4] = pack_bf16(d0, d1);
          }
          contract(DH, xs, v);
        } else {
          const f32x16 y = first_layer(xs);
          f16x2 yh[8];
          uint32_t gq[8];
#pragma unroll
          for (int p = 0; p < 8; ++p) yh[p] = to_f16x2(y[2 * p], y[2 * p + 1]);
          gelu_y16<8>(yh, gq);
          scales();
          float top = 0.0f;
#pragma unroll
          for (int i = 0; i < 16; ++i) top = fmaxf(top, sc[i / 4][i % 4]);
          top = fmaxf(top, partner32(top));
          const int et = __builtin_amdgcn_readfirstlane(top > 0.0f ? __builtin_amdgcn_frexp_expf(top) : e2);
          if (et > e2) {
#pragma unroll
            for (int ib = 0; ib < NRB; ++ib)
#pragma unroll
              for (int i = 0; i < 16; ++i) acc[ib][i] = __builtin_amdgcn_ldexpf(acc[ib][i], e2 - et);
            e2 = et;
          }
#pragma unroll
          for (int p = 0; p < 8; ++p) {
            const f16x2 g2 = __builtin_bit_cast(f16x2, gq[p]);
            const float s0 = __builtin_amdgcn_ldexpf(sc[p / 2][2 * (p % 2)], -e2);
            const float s1 = __builtin_amdgcn_ldexpf(sc[p / 2][2 * (p % 2) + 1], -e2);
            v[p / 4][p % 4] = __builtin_bit_cast(uint32_t, to_f16x2(static_cast<float>(g2[0]) * s0, static_cast<float>(g2[1]) * s1));
          }
          contract(DH, ts, v);
        }
      }
      // the buffer of the tile before this one, which every wave left before the last barrier
      put(tile + step, bufs + ((it + 1) % 2) * SM::kBuf);
      fetch(tile + 2 * step);
      __syncthreads();
    }
  };
  if (role == 0)
    run(std::true_type{});
  else
    run(std::false_type{});
  float* out = part + (static_cast<int64_t>(m) * gridDim.x * SM::kGroups + blockIdx.x * SM::kGroups + grp) * SM::kPart;
#pragma unroll
  for (int ib = 0; ib < NRB; ++ib)
#pragma unroll
    for (int i = 0; i < 16; ++i)
      out[role * D * D + (32 * ib + d_row(i, gl)) * D + 32 * hb + r] = role == 0 ? acc[ib][i] : __builtin_amdgcn_ldexpf(acc[ib][i], e2);
  db1 += partner32(db1);
  if (role == 0 && gl == 0) out[2 * D * D + 32 * hb + r] = db1;
  // db2 over the 32 threads of a piece (the tiles are done with)
  float* red = reinterpret_cast<float*>(bufs);
#pragma unroll
  for (int e = 0; e < 8; ++e) red[tok * (D + 1) + 8 * piece + e] = db2[e];
  __syncthreads();
  if (tid < D) {
    float sum = 0.0f;
    for (int k = 0; k < 32; ++k) sum += red[k * (D + 1) + tid];
    out[2 * D * D + D + tid] = sum;
  }
}

// Adds the `nparts` partials of k_vmod_wgrad in a fixed order, undoes the packing factors (the first layer
// and with it GELU are a quarter of their scale, t W2^T four times it) and puts dW2 the right way round.
// Four slices of the partials per output, sixteen loads in flight each.  grid (kPart / 64, 2 maps), block 256.
template <int D>
__global__ __launch_bounds__(256) void k_vmod_wgrad_reduce(const float* __restrict__ part, int nparts,
                                                           hla_vmod_weight_grads o0, hla_vmod_weight_grads o1) {
  constexpr int64_t PW = VWgSmem<D>::kPart;
  __shared__ float sh[4][64];
  const int c = threadIdx.x % 64, slice = threadIdx.x / 64, idx = blockIdx.x * 64 + c;
  const hla_vmod_weight_grads& o = blockIdx.y == 0 ? o0 : o1;
  const float* base = part + static_cast<int64_t>(blockIdx.y) * nparts * PW + idx;
  const int per = (nparts + 3) / 4, p0 = slice * per, p1 = p0 + per < nparts ? p0 + per : nparts;
  float sum = 0.0f;
  for (int p = p0; p < p1; p += 16) {
    float ld[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) ld[k] = p + k < p1 ? base[(p + k) * PW] : 0.0f;
#pragma unroll
    for (int k = 0; k < 16; ++k) sum += ld[k];
  }
  sh[slice][c] = sum;
  __syncthreads();
  if (slice != 0) return;
  sum = ((sh[0][c] + sh[1][c]) + sh[2][c]) + sh[3][c];
  if (idx < D * D)
    o.dW1[idx] = sum * kHiddenScale;
  else if (idx < 2 * D * D)
    o.dW2[(idx % D) * D + (idx - D * D) / D] = sum * (1.0f / kHiddenScale);
  else if (idx < 2 * D * D + D)
    o.db1[idx - 2 * D * D] = sum * kHiddenScale;
  else
    o.db2[idx - 2 * D * D - D] = sum;
}

template <int D>
hla_status prepare_t() {
  HLA_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(k_vmod_fwd_mfma<D, kWavesV>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, VSmem<D>::total(kWavesV)));
  HLA_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(k_vmod_bwd_map<D, kWavesV, false, 0>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, VSmemB<D>::total(kWavesV)));
  HLA_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(k_vmod_bwd_map<D, kWavesV, false, 1>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, VSmemB<D>::total(kWavesV)));
  HLA_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(k_vmod_bwd_map<D, kWavesV, true, 0>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, VSmemB<D>::total_factors(kWavesV)));
  HLA_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(k_vmod_bwd_map<D, kWavesV, true, 1>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, VSmemB<D>::total_factors(kWavesV)));
  HLA_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(k_vmod_wgrad<D>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, VWgSmem<D>::kTotal));
  return HLA_OK;
}

int compute_units() {
  int dev = 0, n = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 256;
  if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) return 256;
  return n;
}

template <int D>
hla_status forward_t(hla_handle* hd, const hla_call_args& a) {
  const Geom& g = hd->g;
  const int64_t tiles = static_cast<int64_t>((g.N + 31) / 32) * g.B * g.H;
  const int grid = static_cast<int>(std::min<int64_t>(compute_units(), (tiles + kWavesV - 1) / kWavesV));
  return launch(hd, "vmod_forward", k_vmod_fwd_mfma<D, kWavesV>, dim3(grid), dim3(kWavesV * 64),
                VSmem<D>::total(kWavesV), a.stream, g, static_cast<const unsigned char*>(hd->vmod_wpk),
                hd->vmod_ln_eps, vmod_view(hd->vmod_T, g), a.V, a.O, hd->vmod_wpk + vmod_mfma_packed_bytes(hd));
}

// the factor arrays inside hd->vmod_wg_rows; the workgroups' partial sums of dgamma and dbeta go to the
// head of the contractions' partial buffer, which is free while the backward kernels run
VmodFactors factor_arrays(const hla_handle* hd) {
  VmodFactors f;
  const int64_t per = hd->max_th * hd->g.d;
  for (int m = 0; m < 2; ++m) {
    f.t[m] = reinterpret_cast<uint16_t*>(hd->vmod_wg_rows) + m * per;
    f.scale[m] = hd->vmod_wg_rows + per + m * hd->max_th;  // behind two 16-bit arrays
  }
  f.gb_part = hd->vmod_wg_partial;
  return f;
}

// the backward of map MAP: MAP 0 writes dT (before the operator's backward), MAP 1 adds the
// modulation's share to the dV the operator's backward has written
template <int D, int MAP>
hla_status backward_map_t(hla_handle* hd, const hla_call_args& a, View out) {
  const Geom& g = hd->g;
  const int64_t tiles = static_cast<int64_t>((g.N + 31) / 32) * g.B * g.H;
  // two workgroups share a compute unit, but not of the form that also adds up dgamma and dbeta: one round
  // of those (two rounds start and sum twice: 203 us a map at 12 heads x 32760 tokens x 128 channels, now 193)
  const int grid = static_cast<int>(std::min<int64_t>((hd->vmod_wg_on ? 1 : 2) * compute_units(), (tiles + kWavesV - 1) / kWavesV));
  const unsigned char* saved = hd->vmod_wpk + vmod_mfma_packed_bytes(hd);
  const char* name = MAP == 0 ? "vmod_backward" : "vmod_backward_value";
  if (hd->vmod_wg_on) {
    HLA_TRY(launch(hd, name, k_vmod_bwd_map<D, kWavesV, true, MAP>, dim3(grid), dim3(kWavesV * 64),
                   VSmemB<D>::total_factors(kWavesV), a.stream, g, static_cast<const unsigned char*>(hd->vmod_wpk),
                   vmod_view(hd->vmod_T, g), a.V, a.dO, out, saved, factor_arrays(hd)));
    const hla_vmod_weight_grads& o = hd->vmod_wg_out[MAP];
    return launch(hd, "vmod_weight_grads_norm", k_vmod_gb_reduce, dim3(2 * D / 32), dim3(256), 0, a.stream,
                  static_cast<const float*>(hd->vmod_wg_partial), grid, D, o.dgamma, o.dbeta);
  }
  return launch(hd, name, k_vmod_bwd_map<D, kWavesV, false, MAP>, dim3(grid), dim3(kWavesV * 64),
                VSmemB<D>::total(kWavesV), a.stream, g, static_cast<const unsigned char*>(hd->vmod_wpk),
                vmod_view(hd->vmod_T, g), a.V, a.dO, out, saved, VmodFactors{});
}
template <int D>
hla_status backward_t(hla_handle* hd, const hla_call_args& a) {
  return backward_map_t<D, 0>(hd, a, vmod_view(hd->vmod_dT, hd->g));
}

template <int D>
hla_status weight_grads_t(hla_handle* hd, const hla_call_args& a) {
  using SM = VWgSmem<D>;
  const Geom& g = hd->g;
  const int64_t tiles = static_cast<int64_t>((g.N + SM::kTok - 1) / SM::kTok) * g.B * g.H;
  const int blocks = static_cast<int>(std::min<int64_t>(kWgBlocks, (tiles + SM::kGroups - 1) / SM::kGroups));
  HLA_TRY(launch(hd, "vmod_weight_grads_gemm", k_vmod_wgrad<D>, dim3(blocks, 2), dim3(512), SM::kTotal, a.stream, g,
                 static_cast<const unsigned char*>(hd->vmod_wpk), vmod_view(hd->vmod_T, g), a.V, factor_arrays(hd),
                 hd->vmod_wg_partial));
  return launch(hd, "vmod_weight_grads_reduce", k_vmod_wgrad_reduce<D>, dim3((2 * D * D + 2 * D) / 64, 2), dim3(256), 0, a.stream,
                static_cast<const float*>(hd->vmod_wg_partial), blocks * SM::kGroups, hd->vmod_wg_out[0], hd->vmod_wg_out[1]);
}

template <int D>
hla_status add_t(hla_handle* hd, const hla_call_args& a) {
  return backward_map_t<D, 1>(hd, a, a.dV);
}

}  // namespace

bool vmod_mfma_supported(const hla_handle* hd) {
  return hd->path == HLA_PATH_MFMA && hd->cfg.io_dtype == HLA_BF16 && (hd->g.d == 64 || hd->g.d == 128);
}
size_t vmod_mfma_packed_bytes(const hla_handle* hd) {
  return 2 * static_cast<size_t>(hd->g.d == 64 ? VPacked<64>::kBytes : VPacked<128>::kBytes);
}
// packed weights, then what the forward keeps for the backward: one SavedTile per 32-token tile
size_t vmod_mfma_workspace_bytes(const hla_handle* hd) {
  const int64_t tiles = hd->max_th / 32 + static_cast<int64_t>(hd->cfg.max_heads) * hd->cfg.max_seqs + 1;
  const size_t per = hd->g.d == 64 ? SavedTile<64>::kBytes : SavedTile<128>::kBytes;
  return vmod_mfma_packed_bytes(hd) + static_cast<size_t>(tiles) * per;
}
hla_status vmod_mfma_prepare_kernels(const hla_handle* hd) {
  return hd->g.d == 64 ? prepare_t<64>() : prepare_t<128>();
}
hla_status vmod_mfma_set_weights(hla_handle* hd, const hla_vmod_weights* maps, hipStream_t s) {
  const int d = hd->g.d;
  const size_t per = vmod_mfma_packed_bytes(hd) / 2;
  for (int m = 0; m < 2; ++m)
    HLA_TRY(launch(hd, "vmod_pack", k_vmod_pack_mfma<bf16_t>, dim3(64), dim3(256), 0, s,
                   static_cast<const bf16_t*>(maps[m].W1), static_cast<const bf16_t*>(maps[m].b1),
                   static_cast<const bf16_t*>(maps[m].W2), static_cast<const bf16_t*>(maps[m].b2),
                   static_cast<const bf16_t*>(maps[m].gamma), static_cast<const bf16_t*>(maps[m].beta), d,
                   hd->vmod_wpk + m * per));
  return HLA_OK;
}
hla_status vmod_mfma_forward(hla_handle* hd, const hla_call_args& a) {
  return hd->g.d == 64 ? forward_t<64>(hd, a) : forward_t<128>(hd, a);
}
hla_status vmod_mfma_backward(hla_handle* hd, const hla_call_args& a) {
  return hd->g.d == 64 ? backward_t<64>(hd, a) : backward_t<128>(hd, a);
}
// the modulation's weight gradients from the factors the backward kernel left (it must have run
// with hd->vmod_wg_on)
hla_status vmod_mfma_weight_grads(hla_handle* hd, const hla_call_args& a) {
  return hd->g.d == 64 ? weight_grads_t<64>(hd, a) : weight_grads_t<128>(hd, a);
}
// floats the factor arrays and the partials of the contractions need
int64_t vmod_mfma_factor_floats(const hla_handle* hd) { return hd->max_th * (hd->g.d + 2); }
int64_t vmod_mfma_partial_floats(const hla_handle* hd) {
  const int64_t groups = hd->g.d == 64 ? VWgSmem<64>::kGroups : VWgSmem<128>::kGroups;
  return 2 * kWgBlocks * groups * (2 * hd->g.d * hd->g.d + 2 * hd->g.d);
}
hla_status vmod_mfma_add_value_grads(hla_handle* hd, const hla_call_args& a) {
  return hd->g.d == 64 ? add_t<64>(hd, a) : add_t<128>(hd, a);
}

}  // namespace hla
