// Feature maps phi_q, phi_k1..3 (App. A.1: Linear d->d, GELU, Linear d->d_phi, ReLU) and their
// input gradients on the matrix cores.
//
// A token is an MFMA *column* (lane (r, gl): token r of a 32-token tile, half gl), so the two
// layers chain without any layout change:
//   hidden^T[d x 32] = W1^T X^T      A = rows of W1^T read from LDS with plain 16-byte reads;
//                                    B = the token's own input channels, loaded from global
//                                    memory in operand order
//   u^T[d_phi x 32]  = W2^T g^T      B = GELU(hidden) packed straight from the accumulators
// and backward   dg^T = W2 du^T,  dh = dg * GELU'(hidden),  dx^T = W1 dh^T  (A = the same LDS copy
// of W1^T, transpose reads).  The weights of all maps (of one map where tiles are few, see forward_t)
// stay resident in LDS while the workgroup works through its tiles, the key tiles first; each wave
// takes 32-token tiles from the workgroup's list, and two (backward) or three (forward) waves
// share a SIMD so that one wave's GELU arithmetic overlaps the others' matrix and LDS work.
#include "hla_handle.h"
#include "hla_mfma_common.h"
#include "hla_mfma_gelu.h"

namespace hla {
namespace {

using namespace mf;

using TrueTag = std::true_type;
using FalseTag = std::false_type;


// ---- packed weights of one (map, head) in global memory ---------------------------------------
template <int D>
struct Packed {
  static constexpr int kW1T = 0;                      // bf16 [D][D]: row = hidden unit, col = input channel; times 1/4
  static constexpr int kW2A = kW1T + D * D * 2;       // fp16 [D/16][32][8]: A operand of u^T = W2^T g^T (16 rows); times 4
  static constexpr int kW2B = kW2A + D * 16 * 2;      // bf16 [D/32][64][8]: A operand of dg^T = W2 du^T; times 4
  static constexpr int kB1 = kW2B + D * 16 * 2;       // fp32 [D]; times 1/4
  static constexpr int kB2 = kB1 + D * 4;             // fp32 [16]
  static constexpr int kBytes = kB2 + 64;
};

// hidden unit that k-slot (ks2, gl, j) of the second-layer contraction stands for: the slots
// follow the accumulator layout of the first layer (register i = 8*half + j of row block rb).
__host__ __device__ inline int hidden_of_slot(int ks2, int gl, int j) {
  const int rb = ks2 / 2, half = ks2 % 2;
  return 32 * rb + 16 * half + 8 * (j / 4) + 4 * gl + j % 4;
}

template <int D>
__global__ void k_pack_phi(PhiF32 w, int dphi, unsigned char* __restrict__ out) {
  const int64_t mh = blockIdx.x;  // map * heads_w + head
  unsigned char* base = out + mh * Packed<D>::kBytes;
  const float* W1 = w.W1 + mh * D * D;
  const float* W2 = w.W2 + mh * D * dphi;
  uint16_t* w1t = reinterpret_cast<uint16_t*>(base + Packed<D>::kW1T);
  uint16_t* w2a = reinterpret_cast<uint16_t*>(base + Packed<D>::kW2A);
  uint16_t* w2b = reinterpret_cast<uint16_t*>(base + Packed<D>::kW2B);
  float* b1 = reinterpret_cast<float*>(base + Packed<D>::kB1);
  float* b2 = reinterpret_cast<float*>(base + Packed<D>::kB2);
  for (int i = threadIdx.x; i < D * D; i += blockDim.x) {
    const int hid = i / D, in = i % D;
    w1t[i] = f32_to_bf16_bits(kHiddenScale * W1[in * D + hid]);
  }
  for (int i = threadIdx.x; i < (D / 16) * 256; i += blockDim.x) {
    const int ks2 = i / 256, gl = (i / 128) % 2, r = (i / 8) % 16, j = i % 8;
    const int n = hidden_of_slot(ks2, gl, j);
    w2a[i] = r < dphi ? __builtin_bit_cast(uint16_t, static_cast<_Float16>(W2[n * dphi + r] / kHiddenScale)) : 0;
  }
  for (int i = threadIdx.x; i < (D / 32) * 512; i += blockDim.x) {
    const int rb = i / 512, lane = (i / 8) % 64, j = i % 8;
    const int r = lane % 32, gl = lane / 32;
    const int a = 8 * gl + j;
    w2b[i] = a < dphi ? f32_to_bf16_bits(W2[(32 * rb + r) * dphi + a] / kHiddenScale) : 0;
  }
  for (int i = threadIdx.x; i < D; i += blockDim.x) b1[i] = kHiddenScale * w.b1[mh * D + i];
  for (int i = threadIdx.x; i < 16; i += blockDim.x) b2[i] = i < dphi ? w.b2[mh * dphi + i] : 0.0f;
}

// ---- LDS layout ---------------------------------------------------------------------------------
// W1^T is kept row-major (row = hidden unit) with the 16-byte chunks of a row XOR-swizzled by a
// function of the row chosen so that both access patterns spread over all banks without padding:
//   plain 16-byte reads of 16 consecutive rows at one chunk (first-layer A operand), and
//   transpose reads of 4 consecutive rows x 4 consecutive chunks (A operand of dx^T = W1 dh^T).
// SLOTS (backward): slots of the contraction over features that are kept, 8 where d_phi <= 8 (lane half 1
// holds the upper eight, whose feature gradients are zero: it reads half 0's).
template <int D, bool BACKWARD = false, int SLOTS = 16>
struct PhiSmem {
  static constexpr int kChunks = D / 8;               // 16-byte chunks per row
  static constexpr int kRow = D * 2;                  // bytes per row
  static constexpr int kW1 = D * D * 2;
  static constexpr int kW2 = D * SLOTS * 2;           // W2B (backward) or W2A (forward)
  static constexpr int kMap = kW1 + kW2 + D * 4 + 64;  // then b1 [D] and b2 [16] in fp32
  // the maps, the counter of the list of tiles and, backward, a transpose tile per wave for whole-row stores of dX
  static constexpr int kRowsOut = 8;
  static constexpr int total(int nmaps, int waves) {
    return nmaps * kMap + 16 + (BACKWARD ? waves * RowTile<D, kRowsOut>::kBytes : 0);
  }
  __host__ __device__ static __forceinline__ int swz(int row) {
    return D == 128 ? (((row & 3) << 2) | ((row >> 2) & 3)) : ((((row >> 1) & 1) << 2) | ((row >> 2) & 3));
  }
  __device__ static __forceinline__ int off(int row, int chunk) {
    return row * kRow + (((chunk ^ swz(row)) & (kChunks - 1)) << 4);
  }
};

// Copy the packed weights of NMAPS maps (blocks `step` bytes apart in memory, kMap apart in LDS) into
// LDS, all THREADS threads of the workgroup.  All global loads are issued before the first LDS store
// so that they are in flight together: the copy costs one memory round trip, not one per map or piece.
template <int D, bool BACKWARD, int THREADS, int NMAPS = 1, int SLOTS = 16>
__device__ __forceinline__ void load_weights(unsigned char* dst, const unsigned char* src, int64_t step = 0) {
  using SM = PhiSmem<D, BACKWARD, SLOTS>;
  using PK = Packed<D>;
  constexpr int N1 = D * SM::kChunks;              // 16-byte chunks of W1^T
  constexpr int N2 = SM::kW2 / 16;                 // 16-byte chunks of the W2 image
  constexpr int NB = D + 16;                       // floats of b1 and b2
  constexpr int I1 = (N1 + THREADS - 1) / THREADS, I2 = (N2 + THREADS - 1) / THREADS;
  const int t = threadIdx.x;
  u32x4 v1[NMAPS][I1], v2[NMAPS][I2];
  float vb[NMAPS];
#pragma unroll
  for (int m = 0; m < NMAPS; ++m) {
    const unsigned char* s = src + m * step;
    const unsigned char* w2 = s + (BACKWARD ? PK::kW2B : PK::kW2A);
#pragma unroll
    for (int k = 0; k < I1; ++k)
      if (N1 % THREADS == 0 || t + k * THREADS < N1) v1[m][k] = *reinterpret_cast<const u32x4*>(s + PK::kW1T + (t + k * THREADS) * 16);
#pragma unroll
    for (int k = 0; k < I2; ++k)
      if (N2 % THREADS == 0 || t + k * THREADS < N2) {
        const int i = t + k * THREADS;
        v2[m][k] = *reinterpret_cast<const u32x4*>(w2 + (SLOTS == 8 ? (i / 32) * 64 + i % 32 : i) * 16);
      }
    vb[m] = t < NB ? *reinterpret_cast<const float*>(s + PK::kB1 + t * 4) : 0.0f;
  }
#pragma unroll
  for (int m = 0; m < NMAPS; ++m) {
    unsigned char* d = dst + m * SM::kMap;
#pragma unroll
    for (int k = 0; k < I1; ++k) {
      const int i = t + k * THREADS;
      if (N1 % THREADS == 0 || i < N1) *reinterpret_cast<u32x4*>(d + SM::off(i / SM::kChunks, i % SM::kChunks)) = v1[m][k];
    }
#pragma unroll
    for (int k = 0; k < I2; ++k) {
      const int i = t + k * THREADS;
      if (N2 % THREADS == 0 || i < N2) *reinterpret_cast<u32x4*>(d + SM::kW1 + i * 16) = v2[m][k];
    }
    if (t < NB) *reinterpret_cast<float*>(d + SM::kW1 + SM::kW2 + t * 4) = vb[m];
  }
}

// The lane's share of its token's input vector as B operands: k-slot (ks, gl, j) is channel
// 16 ks + 8 gl + j, i.e. one 16-byte piece per k-step.  Tokens at or beyond N read the last row
// (a token is an MFMA column, so what such a lane computes never reaches another token and is
// not stored).  The loads are unconditional: the same number of loads is in flight on every
// path, which lets the wait counters keep a prefetch in flight across the loop back-edge.
template <int D>
__device__ __forceinline__ void load_x(const View& X, int b, int h, int n, int N, int gl,
                                       u32x4 (&x)[D / 16]) {
  const bf16_t* row = X.row<const bf16_t>(b, h, n < N ? n : N - 1);
#pragma unroll
  for (int ks = 0; ks < D / 16; ++ks) x[ks] = *reinterpret_cast<const u32x4*>(row + 16 * ks + 8 * gl);
}

// Per-lane byte offsets (inside a map's W1^T block, row block 0) of the first-layer A operand of
// each k-step: row r, chunk 2 ks + gl.  Row blocks add the compile-time constant 32 rows.
template <int D>
__device__ __forceinline__ void first_layer_offsets(int lane, int (&a_off)[D / 16]) {
  using SM = PhiSmem<D>;
  const int r = lane % 32, gl = lane / 32;
#pragma unroll
  for (int ks = 0; ks < D / 16; ++ks) a_off[ks] = SM::off(r, 2 * ks + gl);
}

// Which (batch row, head, first token) a 32-token tile index stands for.  With weights shared by
// all heads the tiles of every (batch row, head) form one flat list that is dealt out evenly to
// all waves of the grid; with per-head weights a workgroup stays on the head of blockIdx.y/z.
struct TileMap {
  int tiles_per_row;  // ceil(N / 32)
  int total;          // tiles this workgroup's list holds
  int H;
  bool flat;
  __device__ __forceinline__ void decode(int t, int& b, int& h, int& n0) const {
    if (flat) {
      const int row = t / tiles_per_row;
      b = row / H;
      h = row % H;
      n0 = (t % tiles_per_row) * 32;
    } else {
      b = blockIdx.z;
      h = blockIdx.y;
      n0 = t * 32;
    }
  }
};
__device__ __forceinline__ TileMap make_tile_map(const Geom& g, int heads_w) {
  TileMap tm;
  tm.tiles_per_row = (g.N + 31) / 32;
  tm.flat = heads_w == 1;
  tm.total = tm.flat ? tm.tiles_per_row * g.B * g.H : tm.tiles_per_row;
  tm.H = g.H;
  return tm;
}

// ---- forward ------------------------------------------------------------------------------------
// block WAVES*64, three waves per SIMD.  The query map is applied to Q, the F key maps to K; the
// features go to the fp32 feature workspace.  Workgroup x owns the 32-token tiles x, x + gridDim.x, ..
// of both tensors, the key tiles first; its waves take them one at a time from a counter in LDS: of
// three waves that share a SIMD the oldest is served first, so waves with equal shares of the tiles
// finish far apart and the SIMD runs its last tiles one wave at a time.  A wave loads its next tile's
// inputs while it computes the current one.
// `split` (shared weights only): workgroup (x, y) applies map y alone.  The other form keeps all maps
// in LDS and reads K once; with few tiles that leaves most waves without any, see forward_t.
// Bound: the card's power.  The clock falls to 1.8 GHz under this mix (a loop of 8 MFMAs and 96 packed
// FMAs per wave runs at 2.4 GHz on constant operands, at 1.8 on random ones), where the vector ALU
// issues in 69 % of a wave's life and the matrix pipe is busy 48 %.  Fixed shares of the tiles, with
// the query map's weights swapped for the key maps' half way: 84 us at 12 heads x 32760 tokens x 128
// channels, 622 us at 40 x 75600, 20.7 us at 12 x 1560; now 75, 578 and 10.4 us.
template <int D, int F, int WAVES, int DPH>
__global__ __launch_bounds__(WAVES * 64) void k_phi_fwd(Geom g, View Q, View K,
                                                        const unsigned char* __restrict__ wpk,
                                                        int heads_w, int split, float* __restrict__ feat) {
  using SM = PhiSmem<D>;
  constexpr int NRB = D / 32, NKS = D / 16;
  extern __shared__ __align__(16) unsigned char smem[];
  const int lane = threadIdx.x % kWave, wave = wave_index();
  const int r = lane % 32, gl = lane / 32;
  TileMap tm = make_tile_map(g, heads_w);
  const int hw = heads_w == 1 ? 0 : blockIdx.y;
  const int64_t step = static_cast<int64_t>(heads_w) * Packed<D>::kBytes;  // packed blocks are ordered [map][head]
  const int mbase = split ? blockIdx.y : 0;  // the map at the start of LDS
  int* counter = reinterpret_cast<int*>(smem + (split ? 1 : 1 + F) * SM::kMap);
  if (threadIdx.x == 0) *counter = WAVES;
  // the list: entries 0 .. nk-1 are this workgroup's key tiles, nk .. nk+nq-1 its query tiles
  const int own = (tm.total - static_cast<int>(blockIdx.x) + static_cast<int>(gridDim.x) - 1) / static_cast<int>(gridDim.x);
  const int nk = split && mbase == 0 ? 0 : own;
  const int entries = nk + (split && mbase != 0 ? 0 : own);
  int entry = wave;  // this wave's current one, then its next one
  int b = 0, h = 0, n0 = 0;
  // The tile's inputs live in xb only: the next tile's loads are issued into xb as soon as the
  // last first-layer MFMA of the current tile has read it (one and a half stages before the end).
  // The kernel is kept lean in registers (168) so that three waves share a SIMD.
  u32x4 xb[NKS];
  auto fetch = [&]() {
    const bool is_k = entry < nk;
    tm.decode(blockIdx.x + (is_k ? entry : entry - nk) * gridDim.x, b, h, n0);
    load_x<D>(is_k ? K : Q, b, h, n0 + r, g.N, gl, xb);
  };
  if (entry < entries) fetch();
  if (split)
    load_weights<D, false, WAVES * 64>(smem, wpk + mbase * step);
  else
    load_weights<D, false, WAVES * 64, 1 + F>(smem, wpk + static_cast<int64_t>(hw) * Packed<D>::kBytes, step);
  __syncthreads();
  int a_off[NKS];
  first_layer_offsets<D>(lane, a_off);
  // features of the last finished map, not yet stored: accumulator register i of the second layer
  // is feature d_row(i, gl) = 8 (i/4) + 4 gl + i%4; the registers with a feature below d_phi on
  // either lane half are kept
  constexpr int NU = DPH > 8 ? 8 : 4;
  static_assert(DPH <= 16, "one 16-row group of second-layer outputs");
  float pend[NU];
#pragma unroll
  for (int i = 0; i < NU; ++i) pend[i] = 0.0f;
  float* pend_ptr = nullptr;  // feature 4 gl of the token
  auto flush = [&]() {  // a pair of features of 32 consecutive tokens is one contiguous 256-byte run
    if (pend_ptr != nullptr) {
      f32x2* pp = reinterpret_cast<f32x2*>(pend_ptr);
#pragma unroll
      for (int i = 0; i < NU; i += 2) {
        const int a0 = 8 * (i / 4) + i % 4;  // even feature held by lane half 0; half 1 holds a0 + 4
        f32x2 v;
        v[0] = pend[i];
        v[1] = pend[i + 1];
        if (a0 + 4 < DPH) {
          pp[32 * (a0 / 2)] = v;
        } else if (a0 < DPH) {
          if (gl == 0) pp[32 * (a0 / 2)] = v;
        }
      }
    }
    pend_ptr = nullptr;
  };
  // rows 16 .. 31 of the second layer's product are not used: their lanes read row 15, which is zero
  const int w2_lane = (gl * 16 + (r < 16 ? r : 15)) * 16;
  // the first layer accumulates on top of its bias: the lane's 16 entries of a 32-row block
  auto bias_acc = [&](const unsigned char* wmap, int rb) {
    f32x16 z;
    const float* b1 = reinterpret_cast<const float*>(wmap + SM::kW1 + SM::kW2) + 32 * rb + 4 * gl;
#pragma unroll
    for (int i = 0; i < 4; ++i) {  // registers 4i..4i+3 are hidden units 32 rb + 8 i + 4 gl + 0..3
      const f32x4 v = *reinterpret_cast<const f32x4*>(b1 + 8 * i);
      z[4 * i] = v[0];
      z[4 * i + 1] = v[1];
      z[4 * i + 2] = v[2];
      z[4 * i + 3] = v[3];
    }
    return z;
  };
  while (entry < entries) {
    const int n = n0 + r;
    const bool live = n < g.N;
    const int64_t th = g.th(b, h, live ? n : 0);
    const int m0 = split ? mbase : (entry < nk ? 1 : 0), m1 = split ? mbase + 1 : (entry < nk ? 1 + F : 1);
    int ticket = 0;
    if (lane == 0) ticket = atomicAdd(counter, 1);  // read where the next tile's loads start
    // Software pipeline over 32-row blocks of the hidden layer (block t = m * NRB + rb): while the
    // vector ALU evaluates GELU on block t, the matrix pipe works on block t + 1, two MFMAs
    // between quarters of the vector work, their LDS operands read one quarter ahead.  Blocks
    // past the last map alias the last map's LDS: their results are never used.
    // hidden blocks alternate between two accumulator sets (NRB is even, so block 0 of every map
    // lands in set 0): no copy from "next" to "current" at the end of a stage
    static_assert(NRB % 2 == 0, "two alternating accumulator sets");
    f32x16 hb[2];
    constexpr int kPer = NKS / 4;  // first-layer MFMAs per slice
    u32x4 an[kPer];                // their A operands, read one slice ahead
    f32x16 bias_nx;                // and what they accumulate onto, read a stage ahead
    const unsigned char* w0 = smem + (m0 - mbase) * SM::kMap;
    {
      u32x4 a0[NKS];
#pragma unroll
      for (int ks = 0; ks < NKS; ++ks) a0[ks] = *reinterpret_cast<const u32x4*>(w0 + a_off[ks]);
      hb[0] = bias_acc(w0, 0);
      bias_nx = bias_acc(w0, 1 % NRB);
      __builtin_amdgcn_sched_barrier(0);  // all reads in flight before the first product waits for its own
#pragma unroll
      for (int ks = 0; ks < NKS; ++ks) hb[0] = mfma32(a0[ks], xb[ks], hb[0]);
#pragma unroll
      for (int t = 0; t < kPer; ++t)
        an[t] = *reinterpret_cast<const u32x4*>(w0 + (1 % NRB) * 32 * SM::kRow + a_off[t]);
    }
    // The last map of a tile is code of its own: only there the next tile's loads start, and in the
    // other maps the compiler would have to wait for them (and for every store issued since).
    auto run_map = [&](int m, auto LAST) {
      constexpr bool last_map = decltype(LAST)::value;
      const unsigned char* wm = smem + (m - mbase) * SM::kMap;
      f32x16 u;
#pragma unroll
      for (int i = 0; i < 16; ++i) u[i] = 0.0f;
      float b2v[NU];
#pragma unroll
      for (int rb = 0; rb < NRB; ++rb) {
        // block t+1 (first layer, this stage) and block t+2 (whose first operands the last slice reads)
        const unsigned char* w1 = rb + 1 < NRB ? wm : (last_map ? wm : wm + SM::kMap);
        const unsigned char* w2 = rb + 2 < NRB ? wm : (last_map ? wm : wm + SM::kMap);
        const unsigned char* a1_base = w1 + ((rb + 1) % NRB) * 32 * SM::kRow;
        const unsigned char* a2_base = w2 + ((rb + 2) % NRB) * 32 * SM::kRow;
        f32x16& cur = hb[rb % 2];
        f32x16& nxt = hb[(rb + 1) % 2];
        const u32x4 a20 = *reinterpret_cast<const u32x4*>(wm + SM::kW1 + (2 * rb) * 512 + w2_lane);
        const u32x4 a21 = *reinterpret_cast<const u32x4*>(wm + SM::kW1 + (2 * rb + 1) * 512 + w2_lane);
        u32x4 gb[2];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          // the empty asm statements pin the order MFMAs -> GELU slice -> next MFMAs: they are
          // volatile (kept in program order) and the values flow through them
          if (j > 0) asm volatile("" : "+v"(nxt));
          // first layer of block t+1 (there is none after the last block, and xb already belongs
          // to the next tile's loads by then)
          if (rb + 1 < NRB || !last_map) {
#pragma unroll
            for (int t = 0; t < kPer; ++t) {
              nxt = mfma32(an[t], xb[j * kPer + t], j == 0 && t == 0 ? bias_nx : nxt);
              an[t] = j < 3 ? *reinterpret_cast<const u32x4*>(a1_base + a_off[(j + 1) * kPer + t])
                            : *reinterpret_cast<const u32x4*>(a2_base + a_off[t]);
            }
          }
          // The previous map's features leave here: stores count in the same wait counter as loads, and
          // these are old when the next tile's inputs, requested after them, are waited for.
          if (rb == 0 && j == 1) flush();
          if (rb == NRB - 1 && j == 2) {
            const float* b2 = reinterpret_cast<const float*>(wm + SM::kW1 + SM::kW2 + D * 4) + 4 * gl;
#pragma unroll
            for (int i = 0; i < NU; ++i) b2v[i] = b2[8 * (i / 4) + i % 4];
          }
          if (j == 2) bias_nx = bias_acc(w2, (rb + 2) % NRB);
          if (j == 3) u = mfma32_f16(a20, gb[0], u);
          // the next tile's inputs: xb is free once the last first-layer MFMA has been issued
          if constexpr (last_map) if (rb == NRB - 2 && j == 3) {
            entry = __builtin_amdgcn_readfirstlane(ticket);
            if (entry < entries) fetch();
          }
          const float in[4] = {cur[4 * j], cur[4 * j + 1], cur[4 * j + 2], cur[4 * j + 3]};
          __builtin_amdgcn_sched_barrier(0);
          uint32_t out[2];
          gelu_f16<2>(in, out);
          asm volatile("" : "+v"(out[0]), "+v"(out[1]));
          gb[j / 2][2 * (j % 2)] = out[0];
          gb[j / 2][2 * (j % 2) + 1] = out[1];
          __builtin_amdgcn_sched_barrier(0);
        }
        u = mfma32_f16(a21, gb[1], u);
      }
#pragma unroll
      for (int i = 0; i < NU; ++i) pend[i] = fmaxf(u[i] + b2v[i], 0.0f);
      pend_ptr = live ? feat + g.fidx(th, m * DPH + 4 * gl) : nullptr;
    };
#pragma unroll 1
    for (int m = m0; m + 1 < m1; ++m) run_map(m, FalseTag{});
    run_map(m1 - 1, TrueTag{});
  }
  flush();
}

// ---- backward -----------------------------------------------------------------------------------
// block WAVES*64, two waves per SIMD.  dQ through the query map, dK through the F key maps:
// dX = sum over the maps of W1 (GELU'(h) * (W2 du)), with du = d(feature) where the ReLU was open (the
// form in which the feature-gradient workspace arrives).  Hidden activations are recomputed.  All
// maps stay in LDS; the waves of a workgroup take its 32-token tiles from a counter as in the forward.
// Bound: the clock falls as in the forward, but vector ALU and matrix pipe together are busy only
// 77 % of the cycles (forward 89 %), 38 % of the matrix time has vector work beside it (57 %), and a wave
// waits to issue 37 % and sits in s_waitcnt 21 % of its life: two waves per SIMD do not cover each other's
// LDS transpose reads and chains, with 470 MB of traffic beside it.  With fixed shares and the
// weights swapped half way: 150 us at 12 heads x 32760 tokens x 128 channels, 70 at 12600 (a third
// round of tiles for some waves only), 129 in the two-factor form at 32760; now 138, 60 and 113 us.
template <int D, int F, int WAVES, int DPH>
__global__ __launch_bounds__(WAVES * 64) void k_phi_bwd(Geom g, View Q, View K,
                                                        const unsigned char* __restrict__ wpk, int heads_w,
                                                        const float* __restrict__ dfeat, View dQ, View dK) {
  constexpr int SLOTS = DPH <= 8 ? 8 : 16;
  using SM = PhiSmem<D, true, SLOTS>;
  constexpr int NRB = D / 32, NKS = D / 16;
  extern __shared__ __align__(16) unsigned char smem[];
  const int lane = threadIdx.x % kWave, wave = wave_index();
  const int r = lane % 32, gl = lane / 32;
  const int L = lane % 16, q = lane / 16;
  const TileMap tm = make_tile_map(g, heads_w);
  const int hw = heads_w == 1 ? 0 : blockIdx.y;
  int* counter = reinterpret_cast<int*>(smem + (1 + F) * SM::kMap);
  unsigned char* const rows = smem + (1 + F) * SM::kMap + 16 + wave * RowTile<D, SM::kRowsOut>::kBytes;  // dX transpose tile
  if (threadIdx.x == 0) *counter = WAVES;
  // the list: entries 0 .. own-1 are this workgroup's key tiles, own .. 2 own-1 its query tiles
  const int own = (tm.total - static_cast<int>(blockIdx.x) + static_cast<int>(gridDim.x) - 1) / static_cast<int>(gridDim.x);
  int entry = wave;
  bool is_k = entry < own;
  int b = 0, h = 0, n0 = 0;
  auto locate = [&]() { tm.decode(blockIdx.x + (is_k ? entry : entry - own) * gridDim.x, b, h, n0); };
  // The tile's inputs live in xb only: the next tile's loads are issued into xb as soon as the
  // last first-layer MFMA of the current tile has read it (one and a half stages before the end).
  u32x4 xb[NKS];
  if (entry < 2 * own) {
    locate();
    load_x<D>(is_k ? K : Q, b, h, n0 + r, g.N, gl, xb);
  }
  load_weights<D, true, WAVES * 64, 1 + F, SLOTS>(smem, wpk + static_cast<int64_t>(hw) * Packed<D>::kBytes,
                                           static_cast<int64_t>(heads_w) * Packed<D>::kBytes);
  __syncthreads();
  int a_off[NKS];
  first_layer_offsets<D>(lane, a_off);
  // Transpose reads for dx^T[in x tok] += W1[in x hidden] dh^T: k-slots (ks2, gl, j) stand for
  // hidden units 16 ks2 + 4 gl + {0..3} (j < 4) and + 8 (j >= 4); a lane of a 16-lane group
  // addresses hidden row k0 + L/4 and four input channels.  The channel groups are addressed with
  // their two bits exchanged, so that accumulator register i of block rb holds channel
  // 32 rb + 16 (i / 8) + 8 gl + i % 8: eight consecutive ones, and dX leaves as 16-byte pieces.
  // swz() ignores the row's bits 4 and up, so the k-step only adds a constant to the address.
  int t_off[2][NRB];
#pragma unroll
  for (int hi = 0; hi < 2; ++hi)
#pragma unroll
    for (int rb = 0; rb < NRB; ++rb) {
      const int row = 4 * gl + 8 * hi + L / 4;
      const int c = L % 4, col = 32 * rb + 16 * (q % 2) + 4 * (((c & 1) << 1) | (c >> 1));
      t_off[hi][rb] = SM::off(row, col >> 3) + ((col & 7) << 1);
    }
  // du^T of one map as B operand of a single 16-slot step: slot (gl, j) is feature 8gl + j (with
  // d_phi <= 8 only gl = 0 is used).  The feature gradients arrive already zeroed where the ReLU
  // was closed (the core backward kernels, which hold the features anyway, write them that way), so
  // this is a plain load.  In two halves: issue_du puts the loads in flight (unconditional, from
  // addresses valid for every lane), finish_du packs them a whole map later.  Anything that looks
  // at the loaded values next to the loads makes the wave sit out the memory round trip there.
  static_assert(DPH % 2 == 0 && DPH <= 16, "features are packed in pairs into one k-step");
  constexpr int NJ = DPH <= 8 ? DPH : 8;  // features per lane half
  auto issue_du = [&](int64_t th, int m, float (&dv)[NJ]) {
    // lane half 1 holds the features from the ninth on (none when d_phi <= 8: it re-reads half 0's);
    // surplus slots re-read the half's first feature
    const int first = DPH <= 8 ? 0 : 8 * gl;
    const int have = DPH <= 8 ? DPH : (gl ? DPH - 8 : 8);
    const f32x2* dp = reinterpret_cast<const f32x2*>(dfeat + g.fidx(th, m * DPH + first));
#pragma unroll
    for (int p = 0; p < NJ / 2; ++p) {
      const f32x2 v = dp[32 * (2 * p < have ? p : 0)];
      dv[2 * p] = v[0];
      dv[2 * p + 1] = v[1];
    }
  };
  auto finish_du = [&](const float (&dv)[NJ]) -> u32x4 {
    const int have = DPH <= 8 ? (gl ? 0 : DPH) : (gl ? DPH - 8 : 8);
    u32x4 d;
    d[0] = d[1] = d[2] = d[3] = 0u;
#pragma unroll
    for (int p = 0; p < NJ / 2; ++p)
      d[p] = pack_bf16(2 * p < have ? dv[2 * p] : 0.0f, 2 * p + 1 < have ? dv[2 * p + 1] : 0.0f);
    return d;
  };
  auto zero_acc = []() {  // a constant: becomes the inline 0 of the MFMA's C operand
    f32x16 z;
#pragma unroll
    for (int i = 0; i < 16; ++i) z[i] = 0.0f;
    return z;
  };
  // the first layer accumulates on top of its bias: the lane's 16 entries of a 32-row block
  auto bias_acc = [&](const unsigned char* wmap, int rb) {
    f32x16 z;
    const float* b1 = reinterpret_cast<const float*>(wmap + SM::kW1 + SM::kW2) + 32 * rb + 4 * gl;
#pragma unroll
    for (int i = 0; i < 4; ++i) {  // registers 4i..4i+3 are hidden units 32 rb + 8 i + 4 gl + 0..3
      const f32x4 v = *reinterpret_cast<const f32x4*>(b1 + 8 * i);
      z[4 * i] = v[0];
      z[4 * i + 1] = v[1];
      z[4 * i + 2] = v[2];
      z[4 * i + 3] = v[3];
    }
    return z;
  };
  // du of the coming tile's first map: loaded during the last map of the tile before, like the
  // later maps' du is loaded a map ahead
  // Lanes past the end of a sequence do what the lane of its last token does, stores included: with
  // no lane idle the number of stores in flight is known where the next tile's inputs are waited for.
  auto token = [&]() { return g.th(b, h, n0 + r < g.N ? n0 + r : g.N - 1); };
  u32x4 dub_first;
  if (entry < 2 * own) {
    float dv0[NJ];
    issue_du(token(), is_k ? 1 : 0, dv0);
    dub_first = finish_du(dv0);
  }
  while (entry < 2 * own) {
    const int64_t th = token();
    const int m0 = is_k ? 1 : 0, m1 = is_k ? 1 + F : 1;
    const View& dX = is_k ? dK : dQ;
    const int ob = b, oh = h, on0 = n0;
    int ticket = 0;
    if (lane == 0) ticket = atomicAdd(counter, 1);  // read at the start of the tile's last map
    f32x16 dx[NRB];  // first written by the second stage of the first map (accumulating onto zero)
    // Software pipeline over 32-row blocks of the hidden layer, block t = m * NRB + rb.  Stage t:
    //   vector ALU : dh(t) = dg(t) * GELU'(hidden(t) + b1), packed as the B operand of dx
    //   matrix pipe: hidden(t+1) = W1^T X^T block (A: 16-byte LDS reads), dg(t) = W2 du^T block,
    //                dx += W1 dh(t-1)^T (A: transpose reads of the same LDS copy),
    // the MFMAs two or three at a time between quarters of the vector-ALU work, their LDS
    // operands read one step ahead.  Blocks before the first / after the last alias valid LDS
    // and meet zero operands or are dropped.
    static_assert(NRB % 2 == 0, "two alternating accumulator sets");
    f32x16 hb[2];  // hidden blocks alternate between two accumulator sets (as in the forward)
    constexpr int kPer = NKS / 4;  // first-layer MFMAs per slice
    u32x4 an[kPer];                // their A operands, read one slice ahead
    const unsigned char* w0 = smem + m0 * SM::kMap;
    {
      u32x4 a0[NKS];
#pragma unroll
      for (int ks = 0; ks < NKS; ++ks) a0[ks] = *reinterpret_cast<const u32x4*>(w0 + a_off[ks]);
      hb[0] = bias_acc(w0, 0);
      __builtin_amdgcn_sched_barrier(0);  // all reads in flight before the first product waits for its own
#pragma unroll
      for (int ks = 0; ks < NKS; ++ks) hb[0] = mfma32(a0[ks], xb[ks], hb[0]);
#pragma unroll
      for (int t = 0; t < kPer; ++t)
        an[t] = *reinterpret_cast<const u32x4*>(w0 + (1 % NRB) * 32 * SM::kRow + a_off[t]);
    }
    u32x4 dub = dub_first;
    u32x4 dhp[2];  // dh of the previous block (two 16-slot steps)
    // The first map is peeled off the loop over maps: its first stage has no previous block (no dx
    // step at all) and its second stage starts the dx accumulators from the constant zero, which
    // spares clearing them and carrying them into the loop as copies.
    // last_map: a tag (the last map is code of its own, as in the forward) or, where that spills, a bool
    auto run_map = [&](int m, auto first_tag, auto last_map) {
      constexpr bool FIRST = decltype(first_tag)::value;
      const unsigned char* wm = smem + m * SM::kMap;
      float dvn[NJ];  // the next map's du, or the coming tile's first
      if (last_map) {
        entry = __builtin_amdgcn_readfirstlane(ticket);
        if (entry < 2 * own) {  // is_k, b, h, n0 now name the next tile (no next tile: this one again)
          is_k = entry < own;
          locate();
        }
        issue_du(token(), is_k ? 1 : 0, dvn);
      } else {
        issue_du(th, m + 1, dvn);
      }
#pragma unroll
      for (int rb = 0; rb < NRB; ++rb) {
        // block t+1 (first layer, this stage) and block t+2 (whose first operands the last slice reads)
        const unsigned char* a1_base = (rb + 1 < NRB ? wm : (last_map ? wm : wm + SM::kMap)) + ((rb + 1) % NRB) * 32 * SM::kRow;
        const unsigned char* a2_base = (rb + 2 < NRB ? wm : (last_map ? wm : wm + SM::kMap)) + ((rb + 2) % NRB) * 32 * SM::kRow;
        const unsigned char* wp = rb > 0 || FIRST ? wm : wm - SM::kMap;
        const int ks2p = 2 * ((rb + NRB - 1) % NRB);  // first of the two 16-slot steps of block t-1
        const u32x4 a2 = *reinterpret_cast<const u32x4*>(wm + SM::kW1 + (SLOTS == 8 ? rb * 32 + r : rb * 64 + lane) * 16);
        const f32x16 dg = mfma32(a2, dub, zero_acc());
        f32x16& cur = hb[rb % 2];
        f32x16& nxt = hb[(rb + 1) % 2];
        nxt = bias_acc(rb + 1 < NRB ? wm : (last_map ? wm : wm + SM::kMap), (rb + 1) % NRB);
        u32x4 dhc[2];
        // transpose-read operands of the first dx step of this stage
        u32x2 tlo[NRB / 2], thi[NRB / 2];
        const bool has_prev = !(FIRST && rb == 0);  // compile-time after unrolling
        if (has_prev) {
#pragma unroll
          for (int x = 0; x < NRB / 2; ++x) {
            tlo[x] = lds_read_tr16(wp + ks2p * 16 * SM::kRow + t_off[0][x]);
            thi[x] = lds_read_tr16(wp + ks2p * 16 * SM::kRow + t_off[1][x]);
          }
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          asm volatile("" : "+v"(nxt));
          // first layer of block t+1 (there is none after the last block, and xb already belongs
          // to the next tile's loads by then)
          if (rb + 1 < NRB || !last_map) {
#pragma unroll
            for (int t = 0; t < kPer; ++t) {
              nxt = mfma32(an[t], xb[j * kPer + t], nxt);
              an[t] = j < 3 ? *reinterpret_cast<const u32x4*>(a1_base + a_off[(j + 1) * kPer + t])
                            : *reinterpret_cast<const u32x4*>(a2_base + a_off[t]);
            }
          }
          // dx += W1[row blocks of this slice, hidden of block t-1] dh(t-1)^T
#pragma unroll
          for (int x = 0; x < NRB / 2; ++x) {
            if (!has_prev) break;
            const int rbx = (j % 2) * (NRB / 2) + x;
            u32x4 a;
            a[0] = tlo[x][0];
            a[1] = tlo[x][1];
            a[2] = thi[x][0];
            a[3] = thi[x][1];
            // each accumulator is touched twice per stage; its very first touch starts from zero
            dx[rbx] = FIRST && rb == 1 && j < 2 ? mfma32(a, dhp[j / 2], zero_acc())
                                                : mfma32(a, dhp[j / 2], dx[rbx]);
            // operands of the next slice's dx step (the last slice reads ahead into valid LDS)
            const int jn = j + 1 < 4 ? j + 1 : 3;
            const int rbn = (jn % 2) * (NRB / 2) + x;
            tlo[x] = lds_read_tr16(wp + (ks2p + jn / 2) * 16 * SM::kRow + t_off[0][rbn]);
            thi[x] = lds_read_tr16(wp + (ks2p + jn / 2) * 16 * SM::kRow + t_off[1][rbn]);
          }
          // the next tile's inputs: xb is free once the last first-layer MFMA has been issued
          if (last_map && rb == NRB - 2 && j == 3) load_x<D>(is_k ? K : Q, b, h, n0 + r, g.N, gl, xb);
          const float in[4] = {cur[4 * j], cur[4 * j + 1], cur[4 * j + 2], cur[4 * j + 3]};
          __builtin_amdgcn_sched_barrier(0);
          f16x2 gp[2];
          gelu_grad_f16<2>(in, gp);
          // dg * GELU' in fp32 with the fp16 factor read in place (mixed-precision FMA)
          uint32_t o0 = pack_bf16(__builtin_fmaf(static_cast<float>(gp[0][0]), dg[4 * j], 0.0f),
                                  __builtin_fmaf(static_cast<float>(gp[0][1]), dg[4 * j + 1], 0.0f));
          uint32_t o1 = pack_bf16(__builtin_fmaf(static_cast<float>(gp[1][0]), dg[4 * j + 2], 0.0f),
                                  __builtin_fmaf(static_cast<float>(gp[1][1]), dg[4 * j + 3], 0.0f));
          asm volatile("" : "+v"(o0), "+v"(o1));
          dhc[j / 2][2 * (j % 2)] = o0;
          dhc[j / 2][2 * (j % 2) + 1] = o1;
          __builtin_amdgcn_sched_barrier(0);
        }
        dhp[0] = dhc[0];
        dhp[1] = dhc[1];
      }
      dub = finish_du(dvn);  // after the last map: the coming tile's
    };
    if constexpr (D > 64) {  // code of its own: 393 us a step at 12 x 32760 x 128, 384 without
      run_map(m0, TrueTag{}, m0 + 1 == m1);
#pragma unroll 1
      for (int m = m0 + 1; m < m1; ++m) run_map(m, FalseTag{}, m + 1 == m1);
    } else if (m0 == 0) {
      run_map(0, TrueTag{}, TrueTag{});
    } else {
      run_map(1, TrueTag{}, FalseTag{});
#pragma unroll 1
      for (int m = 2; m < F; ++m) run_map(m, FalseTag{}, FalseTag{});
      run_map(F, FalseTag{}, TrueTag{});
    }
    dub_first = dub;
    // dx of the last block
    {
      const unsigned char* wp = smem + (m1 - 1) * SM::kMap;
      constexpr int ks2p = 2 * (NRB - 1);
#pragma unroll
      for (int hf = 0; hf < 2; ++hf)
#pragma unroll
        for (int rbx = 0; rbx < NRB; ++rbx) {
          const u32x2 lo = lds_read_tr16(wp + (ks2p + hf) * 16 * SM::kRow + t_off[0][rbx]);
          const u32x2 hi = lds_read_tr16(wp + (ks2p + hf) * 16 * SM::kRow + t_off[1][rbx]);
          u32x4 a;
          a[0] = lo[0];
          a[1] = lo[1];
          a[2] = hi[0];
          a[3] = hi[1];
          dx[rbx] = mfma32(a, dhp[hf], dx[rbx]);
        }
    }
    u32x4 w[NRB][2];
#pragma unroll
    for (int rb = 0; rb < NRB; ++rb)
#pragma unroll
      for (int hf = 0; hf < 2; ++hf)
#pragma unroll
        for (int p = 0; p < 4; ++p) w[rb][hf][p] = pack_bf16(dx[rb][8 * hf + 2 * p], dx[rb][8 * hf + 2 * p + 1]);
    // whole rows per store instruction: 32-byte pieces cost 5 us of 140 (76 if nontemporal)
#pragma unroll
    for (int pass = 0; pass < 32 / SM::kRowsOut; ++pass) {
      put_rows<D, SM::kRowsOut>(w, pass, lane, rows);
      flush_rows<D, SM::kRowsOut>(pass, lane, rows, [&](int t) -> bf16_t* {
        return dX.row<bf16_t>(ob, oh, on0 + t < g.N ? on0 + t : g.N - 1);
      });
    }
  }
}

// ---- weight gradients ---------------------------------------------------------------------------
// dW1 = X^T dh, db1 = sum dh, dW2 = GELU(h)^T du, db2 = sum du over tokens, for one map per
// workgroup (blockIdx.y) and, with per-head weights, one head (blockIdx.z).  Both products contract
// over TOKENS, so here, unlike in the other kernels, a token is an MFMA *row* of the hidden layer:
// hidden[tok x hid] = X W1 (A = X rows, B = rows of W1^T: the same operand images) leaves a hidden
// unit in a lane with its tokens in the accumulator registers, which is what the contractions want
// as operand: GELU(h) and dh go from the accumulators into the MFMAs without touching LDS.
// Wave w of the workgroup owns hidden block hb = w % (D/32) (its first-layer weights stay in
// registers) and serves the 64-token tiles of group w / (D/32).  The waves of a group share the
// tile in LDS: X in rows (first-layer operand by 16-byte reads, X^T by transpose reads), loaded from
// memory straight to LDS a tile ahead, and du in bf16; three buffers, one barrier per tile.  Workgroups
// of four waves, two per compute unit, so that the waves of a SIMD do not meet at the same barrier.
// A group's sums end as partial number blockIdx.x * T + group of this (map, head):
//   [dW1 D*D | db1 D | dW2 D*d_phi | db2 d_phi] floats, scaled by the packing factors
// (dW1, db1 four times too large, dW2 four times too small); a second kernel adds the partials.
// At 12 heads x 128 channels, three factors (us, same box): 76 at 12600 tokens, 175 at 32760; a form
// that kept tokens in columns and took X, dh and GELU(h) of every wave through LDS and back needed
// 105 and 247.  The vector ALU (GELU and GELU', 250 instructions per 32 tokens and hidden block) is
// busy 53 % of the time, the matrix pipe 33 %, the two at once 12 %; finer interleaving changes nothing.
template <int D>
struct WgSmem {
  static constexpr int kTok = 64;
  static constexpr int kX = kTok * D * 2;             // [token][channels], chunks swizzled (tile_off)
  static constexpr int kDu = kTok * 32;               // [token][16] bf16
  static constexpr int kBuf = kX + kDu;               // one buffer of one group
  static constexpr int kBufs = 3;
};

template <int D, int WAVES, int DPH>
__global__ __launch_bounds__(WAVES * 64, 2) void k_phi_wgrad(Geom g, View Q, View K,
                                                             const unsigned char* __restrict__ wpk,
                                                             int heads_w,
                                                             const float* __restrict__ dfeat,
                                                             float* __restrict__ partial) {
  using SM = WgSmem<D>;
  using PK = Packed<D>;
  constexpr int NRB = D / 32, NKS = D / 16, TH = WAVES / NRB;
  static_assert(WAVES % NRB == 0, "whole groups of hidden blocks");
  constexpr int kPieces = D / 8;                        // 16-byte pieces per row
  constexpr int kLoads = SM::kTok * kPieces / (NRB * 64);  // of a lane, per tile
  constexpr int kPairs = DPH / 2, kDuLoads = (kPairs + NRB - 1) / NRB;
  extern __shared__ __align__(256) unsigned char smem[];
  const int lane = threadIdx.x % kWave, wave = wave_index();
  const int r = lane % 32, gl = lane / 32;
  const int L = lane % 16, q = lane / 16;
  const int hb = wave % NRB, grp = wave / NRB;
  const int m = blockIdx.y, hw = blockIdx.z;
  unsigned char* bufs = smem + grp * SM::kBufs * SM::kBuf;
  const unsigned char* wm = wpk + (static_cast<int64_t>(m) * heads_w + hw) * PK::kBytes;
  const View& X = m == 0 ? Q : K;
  // this wave's first-layer operands: rows 32 hb + r of W1^T, k-slot (ks, gl, j) = channel 16ks + 8gl + j
  u32x4 w1b[NKS];
#pragma unroll
  for (int ks = 0; ks < NKS; ++ks)
    w1b[ks] = *reinterpret_cast<const u32x4*>(wm + PK::kW1T + ((32 * hb + r) * D + 16 * ks + 8 * gl) * 2);
  const u32x4 w2b = *reinterpret_cast<const u32x4*>(wm + PK::kW2B + (hb * 64 + lane) * 16);
  f32x16 bias;  // of hidden unit 32 hb + r, for every token
  {
    const float bv = *reinterpret_cast<const float*>(wm + PK::kB1 + (32 * hb + r) * 4);
#pragma unroll
    for (int i = 0; i < 16; ++i) bias[i] = bv;
  }
  // token tiles: one list over all (batch row, head) pairs when the weights are shared
  const bool shared = heads_w == 1;
  const int tpr = (g.N + SM::kTok - 1) / SM::kTok;
  const int total = (shared ? g.B * g.H : g.B) * tpr;
  f32x16 zero;
#pragma unroll
  for (int i = 0; i < 16; ++i) zero[i] = 0.0f;
  f32x16 acc[NRB];   // dW1 rows 32 ib + d_row(i, gl), column 32 hb + r
  f32x16 acc2 = zero;  // dW2^T rows = features d_row(i, gl), column 32 hb + r
  float db1 = 0.0f;  // of hidden unit 32 hb + r, over the lane half's tokens
  float db2[2 * kDuLoads];  // of the features this wave loads, over the lane's tokens
#pragma unroll
  for (int ib = 0; ib < NRB; ++ib) acc[ib] = zero;
#pragma unroll
  for (int a = 0; a < 2 * kDuLoads; ++a) db2[a] = 0.0f;
  // columns d_phi .. 15 of the du tiles stay zero
  for (int i = threadIdx.x; i < TH * SM::kBufs * SM::kDu / 16; i += WAVES * 64) {
    u32x4 z4;
    z4[0] = z4[1] = z4[2] = z4[3] = 0u;
    const int b = i / (SM::kDu / 16);
    *reinterpret_cast<u32x4*>(smem + b * SM::kBuf + SM::kX + (i % (SM::kDu / 16)) * 16) = z4;
  }
  __syncthreads();
  f32x2 dr[kDuLoads];
  bool du_live = false;
  // Start the loads of one tile: this wave's share of the X rows straight to LDS (16 bytes per lane to
  // consecutive places, so the lane fetches the piece that the swizzle puts there), its share of du to
  // registers.  Every address is valid (tiles past the list re-read the last, rows past the sequence
  // its last row); what must not count is zeroed in du.
  auto fetch = [&](int tile, unsigned char* buf) {
    const int tc = tile < total ? tile : total - 1;
    const int row = tc / tpr, n0 = (tc % tpr) * SM::kTok;
    const int b = shared ? row / g.H : row, h = shared ? row % g.H : hw;
#pragma unroll
    for (int i = 0; i < kLoads; ++i) {
      const int pos = (hb * kLoads + i) * 64 + lane, t = pos / kPieces;
      const int piece = (pos % kPieces) ^ (tile_swz<D * 2>(t) & (kPieces - 1));
      const int n = n0 + t;
      load_to_lds16(X.row<const bf16_t>(b, h, n < g.N ? n : g.N - 1) + 8 * piece, buf + (hb * kLoads + i) * 1024);
    }
    const int n = n0 + lane;
    du_live = tile < total && n < g.N;
    const f32x2* dp = reinterpret_cast<const f32x2*>(dfeat + g.fidx(g.th(b, h, n < g.N ? n : g.N - 1), m * DPH));
#pragma unroll
    for (int i = 0; i < kDuLoads; ++i) {
      const int p = hb * kDuLoads + i;
      dr[i] = dp[32 * (p < kPairs ? p : 0)];
    }
  };
  auto put_du = [&](unsigned char* buf) {
#pragma unroll
    for (int i = 0; i < kDuLoads; ++i) {
      const int p = hb * kDuLoads + i;
      if (p < kPairs) {
        const float d0 = du_live ? dr[i][0] : 0.0f, d1 = du_live ? dr[i][1] : 0.0f;
        db2[2 * i] += d0;
        db2[2 * i + 1] += d1;
        *reinterpret_cast<uint32_t*>(buf + SM::kX + lane * 32 + p * 4) = pack_bf16(d0, d1);
      }
    }
  };
  // LDS addresses.  First layer: row r, chunk 2 ks + gl.  Transpose reads of X^T: k-slot (gl, j) of
  // step ks is token 16 ks + 8 (j / 4) + 4 gl + j % 4, the order the accumulators hold.  Swizzling
  // ignores the row's bits 4 and up: sub-tiles and steps add constants.
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
  const int du_a = SM::kX + r * 32 + gl * 16;                          // operand of dg: token r, features 8 gl ..
  const int du_t = SM::kX + (4 * gl + L / 4) * 32 + 8 * (L % 4);  // of dW2^T; rows past the sixteenth feature repeat: never stored
  // A operand number x of the contraction over tokens 16 ks .. + 15 of a sub-tile: X^T block x, or du^T
  auto tn_operand = [&](const unsigned char* buf, int sub, int ks, int x) {
    const unsigned char* lo_p = x < NRB ? buf + (32 * sub + 16 * ks) * D * 2 + t_off[0][x < NRB ? x : 0]
                                        : buf + (32 * sub + 16 * ks) * 32 + du_t;
    const unsigned char* hi_p = x < NRB ? buf + (32 * sub + 16 * ks) * D * 2 + t_off[1][x < NRB ? x : 0]
                                        : buf + (32 * sub + 16 * ks + 8) * 32 + du_t;
    const u32x2 lo = lds_read_tr16(lo_p), hi = lds_read_tr16(hi_p);
    u32x4 a;
    a[0] = lo[0];
    a[1] = lo[1];
    a[2] = hi[0];
    a[3] = hi[1];
    return a;
  };
  constexpr int kPer = NKS / 4;       // first-layer MFMAs per slice
  constexpr int NX = NRB + 1;         // operands of a contraction step
  constexpr int kSplit = (NX + 1) / 2;  // of them in its first slice
  u32x4 an[kPer], ct[kSplit], dua;
  u32x4 dhp, gvp;                     // dh, GELU of the previous sub-tile's second step
  f32x16 hb2[2];                      // hidden blocks of this and the next sub-tile
  // One 32-token sub-tile: GELU and GELU' on the vector ALU in four slices; between them the matrix
  // pipe does the next sub-tile's first layer, the previous one's second contraction step (slices 0,
  // 1) and this one's first (slices 2, 3), operands read a slice ahead.
  auto sub_tile = [&](auto PAR, const unsigned char* cur_b, int sub, const unsigned char* nxt_b, int nsub,
                      const unsigned char* prv_b, int psub) {
    constexpr int par = decltype(PAR)::value;
    f32x16& cur = hb2[par];
    f32x16& nxt = hb2[1 - par];
    const f32x16 dg = mfma32(dua, w2b, zero);
    u32x4 dh[2], gv[2];
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
#pragma unroll
      for (int t = 0; t < kPer; ++t) {
        nxt = mfma32(an[t], w1b[j * kPer + t], j == 0 && t == 0 ? bias : nxt);
        an[t] = j < 3 ? *reinterpret_cast<const u32x4*>(nxt_b + nsub * 32 * D * 2 + a_off[((j + 1) % 4) * kPer + t]) : an[t];
      }
      if (j == 3) dua = *reinterpret_cast<const u32x4*>(nxt_b + nsub * 32 * 32 + du_a);
      {
        constexpr int half[2] = {0, kSplit};
        const int x0 = half[j % 2], x1 = j % 2 == 0 ? kSplit : NX;
        const u32x4 bd = j < 2 ? dhp : dh[0], bg = j < 2 ? gvp : gv[0];
#pragma unroll
        for (int x = x0; x < x1; ++x) {
          if (x < NRB)
            acc[x < NRB ? x : 0] = mfma32(ct[x - x0], bd, acc[x < NRB ? x : 0]);
          else
            acc2 = mfma32(ct[x - x0], bg, acc2);
        }
        // the next slice's operands: second half of the same step, or the next step's first half
        const int y0 = half[(j + 1) % 2], y1 = (j + 1) % 2 == 0 ? kSplit : NX;
#pragma unroll
        for (int y = y0; y < y1; ++y)
          ct[y - y0] = j == 0 ? tn_operand(prv_b, psub, 1, y) : (j < 3 ? tn_operand(cur_b, sub, 0, y) : tn_operand(cur_b, sub, 1, y));
      }
      __builtin_amdgcn_sched_barrier(0);
      {
        const int ks = j / 2, jj = j % 2, i0 = 4 * j;  // accumulator registers of tokens 16 ks + 8 jj + 4 gl + 0..3
        const float in[4] = {cur[i0], cur[i0 + 1], cur[i0 + 2], cur[i0 + 3]};
        f16x2 gg[2], gp[2];
        gelu_both_f16<2>(in, gg, gp);
        const float d0 = __builtin_fmaf(static_cast<float>(gp[0][0]), dg[i0], 0.0f);
        const float d1 = __builtin_fmaf(static_cast<float>(gp[0][1]), dg[i0 + 1], 0.0f);
        const float d2 = __builtin_fmaf(static_cast<float>(gp[1][0]), dg[i0 + 2], 0.0f);
        const float d3 = __builtin_fmaf(static_cast<float>(gp[1][1]), dg[i0 + 3], 0.0f);
        db1 += (d0 + d1) + (d2 + d3);
        asm volatile("" : "+v"(db1));  // summed here, not with the terms kept until the next tile
        dh[ks][2 * jj] = pack_bf16(d0, d1);
        dh[ks][2 * jj + 1] = pack_bf16(d2, d3);
        gv[ks][2 * jj] = pack_bf16(static_cast<float>(gg[0][0]), static_cast<float>(gg[0][1]));
        gv[ks][2 * jj + 1] = pack_bf16(static_cast<float>(gg[1][0]), static_cast<float>(gg[1][1]));
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    dhp = dh[1];
    gvp = gv[1];
    // the coming sub-tile's next one: its first-layer operands are read by the caller's next call
  };
  const int step = gridDim.x * TH;
  const int first = blockIdx.x * TH;
  const int iters = (total - first + step - 1) / step;  // of group 0, which has the most
  fetch(first + grp, bufs);
  put_du(bufs);
  fetch(first + step + grp, bufs + SM::kBuf);
  wait_lds_loads();
  __syncthreads();
  // hidden block of the first sub-tile, and what its first slice needs
#pragma unroll
  for (int ks = 0; ks < NKS; ++ks)
    hb2[0] = mfma32(*reinterpret_cast<const u32x4*>(bufs + a_off[ks]), w1b[ks], ks == 0 ? bias : hb2[0]);
  dua = *reinterpret_cast<const u32x4*>(bufs + du_a);
  dhp[0] = dhp[1] = dhp[2] = dhp[3] = 0u;  // nothing before the first sub-tile
  gvp = dhp;
#pragma unroll
  for (int x = 0; x < kSplit; ++x) ct[x] = tn_operand(bufs, 0, 1, x);
#pragma unroll
  for (int t = 0; t < kPer; ++t) an[t] = *reinterpret_cast<const u32x4*>(bufs + 32 * D * 2 + a_off[t]);
  // Tile `it` sits in buffer it % 3.  Its second sub-tile already needs the next tile: the barrier in
  // front of it comes after every wave's loads of that tile have landed, and says that the tile
  // before this one is done with, whose buffer takes the loads of the tile after next.
  auto tile_step = [&](auto B, int it) {
    constexpr int b = decltype(B)::value;
    unsigned char* cb = bufs + b * SM::kBuf;
    unsigned char* nb = bufs + ((b + 1) % 3) * SM::kBuf;
    unsigned char* pb = bufs + ((b + 2) % 3) * SM::kBuf;
    sub_tile(std::integral_constant<int, 0>{}, cb, 0, cb, 1, it == 0 ? cb : pb, it == 0 ? 0 : 1);
    put_du(nb);
    wait_lds_loads();
    __syncthreads();
    fetch(first + (it + 2) * step + grp, pb);
#pragma unroll
    for (int t = 0; t < kPer; ++t) an[t] = *reinterpret_cast<const u32x4*>(nb + a_off[t]);
    sub_tile(std::integral_constant<int, 1>{}, cb, 1, nb, 0, cb, 0);
#pragma unroll
    for (int t = 0; t < kPer; ++t) an[t] = *reinterpret_cast<const u32x4*>(nb + 32 * D * 2 + a_off[t]);
  };
  for (int it = 0; it < iters; it += 3) {
    tile_step(std::integral_constant<int, 0>{}, it);
    if (it + 1 < iters) tile_step(std::integral_constant<int, 1>{}, it + 1);
    if (it + 2 < iters) tile_step(std::integral_constant<int, 2>{}, it + 2);
  }
  // the last sub-tile's second contraction step: its operands are in ct (first half) and LDS
  {
    const unsigned char* lb = bufs + ((iters - 1) % 3) * SM::kBuf;
#pragma unroll
    for (int x = 0; x < NX; ++x) {
      const u32x4 a = x < kSplit ? ct[x] : tn_operand(lb, 1, 1, x);
      if (x < NRB)
        acc[x < NRB ? x : 0] = mfma32(a, dhp, acc[x < NRB ? x : 0]);
      else
        acc2 = mfma32(a, gvp, acc2);
    }
  }
  // ---- this wave's share of the partial (fetches past the list counted as zero)
  const int nparts = gridDim.x * TH;
  const int64_t floats = static_cast<int64_t>(D) * D + D + D * DPH + DPH;
  float* out = partial + ((static_cast<int64_t>(m) * gridDim.z + hw) * nparts + blockIdx.x * TH + grp) * floats;
#pragma unroll
  for (int ib = 0; ib < NRB; ++ib)
#pragma unroll
    for (int i = 0; i < 16; ++i) out[(32 * ib + d_row(i, gl)) * D + 32 * hb + r] = acc[ib][i];
#pragma unroll
  for (int i = 0; i < (DPH > 8 ? 8 : 4); ++i) {
    const int a = d_row(i, gl);
    if (a < DPH) out[D * D + D + (32 * hb + r) * DPH + a] = acc2[i];
  }
  {
    const float v = db1 + partner32(db1);
    if (gl == 0) out[D * D + 32 * hb + r] = v;
  }
#pragma unroll
  for (int i = 0; i < kDuLoads; ++i) {
    const int p = hb * kDuLoads + i;
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      float v = db2[2 * i + e];
#pragma unroll
      for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
      if (lane == 0 && p < kPairs) out[D * D + D + D * DPH + 2 * p + e] = v;
    }
  }
}

template <typename K>
hla_status allow_lds(K kernel, int bytes) {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                             hipFuncAttributeMaxDynamicSharedMemorySize, bytes) == hipSuccess
             ? HLA_OK
             : HLA_ERR_HIP;
}

constexpr int kUnits = 256;  // compute units of the card

// One workgroup per compute unit in total.  Shared weights: a flat grid over all tiles; per-head
// weights: (x, H, B) with x workgroups per (batch row, head).
dim3 phi_grid(const hla_handle* hd, int waves) {
  const Geom& g = hd->g;
  const int tiles = (g.N + 31) / 32;
  if (hd->phi.heads_w == 1) {
    const int64_t total = static_cast<int64_t>(tiles) * g.B * g.H;
    const int64_t want = (total + waves - 1) / waves;
    return dim3(static_cast<unsigned>(want < kUnits ? (want < 1 ? 1 : want) : kUnits), 1, 1);
  }
  const int units = g.B * g.H;
  int gx = kUnits / units;  // rounding down keeps the whole grid resident in one round
  const int need = (tiles + waves - 1) / waves;
  if (gx > need) gx = need;
  return dim3(gx < 1 ? 1 : gx, g.H, g.B);
}

// waves per workgroup: three per SIMD in the forward kernel (it stays within 168 registers), two
// in the backward one
constexpr int kWavesF = 12, kWavesB = 8;

// F key maps of DPH features each, after the query map.  With shared weights and fewer than
// kSplitTiles tiles a workgroup applies one map only (the 1 + F maps' workgroups side by side, K read
// F times): otherwise a tile of K is three maps in a row on one wave while most of the waves have none.
// From kSplitTiles on every wave of 256 workgroups has a tile of K.  Forward calls in us, 12 heads x
// 128 channels, split / whole: 26 / 36 at 1024 tokens, 33 / 40 at 4096, 48.8 / 49.4 at 8192 (3072
// tiles), 65.0 / 65.7 at 12600; two-factor form 44 / 48 at 4096, 60.9 / 60.3 at 8192.
constexpr int kSplitTiles = 3072;

template <int D, int F, int DPH>
hla_status forward_t(hla_handle* hd, const hla_call_args& a) {
  using SM = PhiSmem<D>;
  Geom g = hd->g;
  const unsigned char* wpk = static_cast<const unsigned char*>(hd->path_ws) + hd->w_packed_off;
  const int64_t tiles = static_cast<int64_t>((g.N + 31) / 32) * g.B * g.H;
  const int split = hd->phi.heads_w == 1 && tiles < kSplitTiles;
  dim3 grid = phi_grid(hd, kWavesF);
  if (split) grid = dim3(static_cast<unsigned>(std::min<int64_t>(kUnits / (1 + F), tiles)), 1 + F, 1);
  return launch(hd, "mfma_phi_forward", k_phi_fwd<D, F, kWavesF, DPH>, grid, dim3(kWavesF * 64),
                SM::total(split ? 1 : 1 + F, kWavesF), a.stream, g, a.Q, a.K, wpk, hd->phi.heads_w, split, hd->feat);
}

template <int D, int F, int DPH>
hla_status backward_t(hla_handle* hd, const hla_call_args& a) {
  using SM = PhiSmem<D, true, (DPH <= 8 ? 8 : 16)>;
  Geom g = hd->g;
  const unsigned char* wpk = static_cast<const unsigned char*>(hd->path_ws) + hd->w_packed_off;
  const dim3 grid = phi_grid(hd, kWavesB);
  HLA_TRY(launch(hd, "mfma_phi_backward", k_phi_bwd<D, F, kWavesB, DPH>, grid, dim3(kWavesB * 64),
                 SM::total(1 + F, kWavesB), a.stream, g, a.Q, a.K, wpk, hd->phi.heads_w, hd->dfeat, a.dQ, a.dK));
  return HLA_OK;
}

// two workgroups per compute unit: their barriers leave each other alone
constexpr int kWavesW = 4, kGridW = 2 * kUnits;
constexpr int wgrad_groups(int d) { return kWavesW / (d / 32); }  // wave groups of a workgroup, a partial sum each

template <int D, int DPH>
hla_status weight_grads_t(hla_handle* hd, const hla_call_args& a) {
  using SM = WgSmem<D>;
  constexpr int TH = wgrad_groups(D);
  constexpr int lds = TH * SM::kBufs * SM::kBuf;
  Geom g = hd->g;
  const unsigned char* wpk = static_cast<const unsigned char*>(hd->path_ws) + hd->w_packed_off;
  const int nm = 1 + g.F;
  const bool shared = hd->phi.heads_w == 1;
  const int heads = shared ? 1 : g.H;
  const int64_t tiles = static_cast<int64_t>(shared ? g.B * g.H : g.B) * ((g.N + SM::kTok - 1) / SM::kTok);
  // at most kGridW workgroups in total (but one per map and head), each with at least one tile per wave group
  int64_t nblk = kGridW / (static_cast<int64_t>(nm) * heads);
  if (nblk > (tiles + TH - 1) / TH) nblk = (tiles + TH - 1) / TH;
  if (nblk < 1) nblk = 1;
  const int64_t nparts = nblk * TH;
  if (nm * heads * nparts > hd->wg_parts_cap) return HLA_ERR_STATE;
  HLA_TRY(launch(hd, "mfma_phi_weight_grads", k_phi_wgrad<D, kWavesW, DPH>,
                 dim3(static_cast<unsigned>(nblk), nm, heads), dim3(kWavesW * 64), lds, a.stream, g, a.Q, a.K,
                 wpk, hd->phi.heads_w, static_cast<const float*>(hd->dfeat), hd->wg_partial));
  // undo the packing factors: dh and dg carry 1/kHiddenScale, GELU(h) carries kHiddenScale
  return weight_grads_reduce(hd, static_cast<int>(nparts), heads, kHiddenScale, kHiddenScale,
                             1.0f / kHiddenScale, 1.0f, a.stream);
}

template <int D, int F, int DPH>
hla_status prepare_t() {
  HLA_TRY(allow_lds(&k_phi_fwd<D, F, kWavesF, DPH>, PhiSmem<D>::total(1 + F, kWavesF)));
  HLA_TRY(allow_lds(&k_phi_bwd<D, F, kWavesB, DPH>, PhiSmem<D, true, (DPH <= 8 ? 8 : 16)>::total(1 + F, kWavesB)));
  return allow_lds(&k_phi_wgrad<D, kWavesW, DPH>, wgrad_groups(D) * WgSmem<D>::kBufs * WgSmem<D>::kBuf);
}

}  // namespace

hla_status mfma_phi_prepare_kernels(const hla_handle* hd) {
  if (hd->g.F == 3) return hd->g.d == 128 ? prepare_t<128, 3, 6>() : prepare_t<64, 3, 6>();
  return hd->g.d == 128 ? prepare_t<128, 2, 12>() : prepare_t<64, 2, 12>();
}

// the two forms the matrix-core path serves: (F, d_phi) = (3, 6) and (2, 12)
bool mfma_phi_supported(const hla_handle* hd) {
  return (hd->g.F == 3 && hd->g.dphi == 6) || (hd->g.F == 2 && hd->g.dphi == 12);
}

hla_status mfma_phi_weight_grads(hla_handle* hd, const hla_call_args& a) {
  if (!mfma_phi_supported(hd)) return HLA_ERR_UNSUPPORTED;
  if (hd->g.F == 3) return hd->g.d == 128 ? weight_grads_t<128, 6>(hd, a) : weight_grads_t<64, 6>(hd, a);
  return hd->g.d == 128 ? weight_grads_t<128, 12>(hd, a) : weight_grads_t<64, 12>(hd, a);
}

// most partial weight gradients of a call, all maps and heads together
int64_t mfma_phi_wgrad_parts(const hla_handle* hd) {
  return wgrad_groups(hd->g.d) * std::max<int64_t>(kGridW, static_cast<int64_t>(1 + hd->g.F) * hd->cfg.max_heads);
}

size_t mfma_phi_packed_bytes(const hla_handle* hd) {
  const size_t per = hd->g.d == 128 ? Packed<128>::kBytes : Packed<64>::kBytes;
  return per * (1 + hd->g.F) * hd->cfg.max_heads;
}

hla_status mfma_phi_set_weights(hla_handle* hd, hipStream_t s) {
  unsigned char* wpk = static_cast<unsigned char*>(hd->path_ws) + hd->w_packed_off;
  const int blocks = (1 + hd->g.F) * hd->phi.heads_w;
  if (hd->g.d == 128)
    return launch(hd, "mfma_pack_phi", k_pack_phi<128>, dim3(blocks), dim3(256), 0, s, hd->phi, hd->g.dphi, wpk);
  return launch(hd, "mfma_pack_phi", k_pack_phi<64>, dim3(blocks), dim3(256), 0, s, hd->phi, hd->g.dphi, wpk);
}

hla_status mfma_phi_forward(hla_handle* hd, const hla_call_args& a) {
  if (!mfma_phi_supported(hd)) return HLA_ERR_UNSUPPORTED;
  if (hd->g.F == 3) return hd->g.d == 128 ? forward_t<128, 3, 6>(hd, a) : forward_t<64, 3, 6>(hd, a);
  return hd->g.d == 128 ? forward_t<128, 2, 12>(hd, a) : forward_t<64, 2, 12>(hd, a);
}

hla_status mfma_phi_backward(hla_handle* hd, const hla_call_args& a) {
  if (!mfma_phi_supported(hd)) return HLA_ERR_UNSUPPORTED;
  if (hd->g.F == 3) return hd->g.d == 128 ? backward_t<128, 3, 6>(hd, a) : backward_t<64, 3, 6>(hd, a);
  return hd->g.d == 128 ? backward_t<128, 2, 12>(hd, a) : backward_t<64, 2, 12>(hd, a);
}

}  // namespace hla

