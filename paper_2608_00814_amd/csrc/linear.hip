// Projections of the target decoder around the verification path: the
// q/k/v, output and MLP projections of every layer (Section 4.5: the target
// scores the tree in one forward pass; Section 5: Qwen3 targets).  With the
// trie's N <= 256 rows these are skinny GEMMs, Y[N][O] = X[N][K] W[O][K]^T,
// bound by streaming W from HBM once.
//
// Design (the LM head's streaming scheme, made shape-independent):
//  * W is packed once into 16 KiB blocks of 128 rows x 64 columns (the LM
//    head's layout, ooo_linear_pack); the work is the sequence of (128-row
//    tile, 64-column chunk) blocks in tile-major order.
//  * Stream-K: a persistent grid (one block per CU) where block b takes a
//    contiguous run of chunks, C / B of them or one more (Runs).  Every block
//    streams the same bytes whatever O and K are; a run covers the end of
//    one tile and the start of the next.
//  * Inside a block, the LM head's streaming core (stream_core.h) with
//    128-row tiles: four loader waves copy one 32-row W slot each and a
//    quarter of the X rows there are into an LDS ring; four compute waves
//    run mfma_f32_32x32x16_bf16 (32 W rows x the nodes each).  Taller tiles
//    move fewer X bytes but twice the partial sums: 256-row tiles measured
//    214.6 against 202.4 us for two Qwen3-8B layers at one node, 262.6
//    against 238.2 at 64.
//  * At the end of each tile segment a block stores its partial sums (of the
//    nodes there are) in the workspace as fp16 ([node][128 rows]) times a
//    power of two per compute wave (its 32 rows), chosen so that the wave's
//    largest magnitude lies in [2^14, 2^15): half the bytes of fp32, with
//    the range of fp32.  A reduce kernel adds a tile's partials in float32
//    in block order (deterministic, no atomics) and applies the epilogue:
//    store fp32 or bf16, add into an fp32 output (the residual rows), or
//    silu(gate) * up of a fused gate/up projection.  Where the partials lie
//    follows from the cut's closed form in registers (a list built in LDS by
//    one thread per tile cost each of these kernels about 1.5 us).
//  * The gate/up projection usually has enough rows for every block to own
//    whole output columns: then it runs without partial sums
//    (linear_swiglu_kernel).
// Two layers at the Qwen3-8B shape (graph replay), with 128-row tiles of
// seven waves, padded X and partial rows, slot lists in LDS and SwiGLU
// through stream-K against this: 243.3 -> 196.9 us at one node, 282.9 ->
// 231.4 at 64; one layer at H 5120, I 27648, 128 nodes 314.9 -> 259.2.
#include <math.h>

#include "device_common.h"
#include "ooo_internal.h"
#include "rope.h"
#include "runs.h"
#include "stream_core.h"

namespace ooo {
namespace {

// Stream-K partial sums in the workspace: slot k (block b, segment j: k =
// b * seg + j) holds v[k][node][128 rows] in fp16 and sc[k][4], the factor
// that turns the fp16 values of rows 32 w .. 32 w + 31 back into the sums.
struct Partials {
  uint16_t* v;
  float* sc;
};

template <int NB, bool PACKED>
__global__ __launch_bounds__(kTallThreads) void linear_bf16_kernel(const uint16_t* __restrict__ X,
                                                                   const uint16_t* __restrict__ Wt, int N, int K,
                                                                   int O, Runs runs, Ring ring, Partials part) {
  constexpr int NPAD = 32 * NB;
  __shared__ __attribute__((aligned(1024))) uint8_t lds[kRingBytes];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int KC = K / 64;
  const int groups = (O + 31) / 32;
  const int b = (int)blockIdx.x;
  const int lo = runs.lo(b);
  const int total = runs.lo(b + 1) - lo;  // chunks of this block (>= 1: B <= C)
  const int first_tile = (int)((unsigned)lo / (unsigned)KC), kc0 = lo - first_tile * KC;
  const auto tile = [&](int t) { return GroupRange{4 * t, min(4 * t + 4, groups)}; };

  if (wave >= 4) {
    const int ld = wave - 4;
    XShare<NB> xs(X, N, K, ld, lane);
    GroupSlots<1, PACKED> slots(Wt, KC, O, K, lane);
    tall_load<NB, 1>(first_tile, kc0, total, KC, (groups - 1) % 4 + 1, ld, tile, slots, xs, ring, lds);
    return;
  }

  // ------------------------------------------------------------------ compute
  const int c = lane & 31, u = lane >> 5;
  uint32_t off[4];
  frag_offsets(lane, off);
  int stage = 0, left = total, kc = kc0;
  wg_barrier();  // the first chunk has landed
  for (int t = first_tile; left > 0; ++t) {
    const int n = min(left, KC - kc), ng = tile(t).hi - tile(t).lo;
    left -= n;
    kc = 0;
    f32x16 acc[1][NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) acc[0][nb] = f32x16{};
    tall_tile<NB, 1>(n, left == 0, ng, wave, lds, ring, off, stage, acc);
    if (wave >= ng) continue;
    // segment done: acc[0][nb][j] = partial of tile row 32 wave + 8(j/4) + 4u + j%4, node 32nb + c.
    // Scale: the wave's largest finite magnitude a < 2^ex (over the nodes
    // there are) goes to [2^14, 2^15) (fp16 holds up to 65504); exact powers
    // of two both ways.  Inf and NaN stay what they are and do not set it:
    // fmax passes NaN over, and where an infinity shows up the maximum is
    // taken once more without.  (With both tests on every value a call of 256
    // rows took 1.5 to 3 us longer: K 4096, O 6144 28.7 against 25.8 us.)
    const size_t slot = (size_t)b * runs.seg + (t - first_tile);
    float amax = 0.f;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      float m = 0.f;
#pragma unroll
      for (int j = 0; j < 16; ++j) m = __builtin_fmaxf(m, __builtin_fabsf(acc[0][nb][j]));
      amax = __builtin_fmaxf(amax, 32 * nb + c < N ? m : 0.f);
    }
    if (__any(!(amax < INFINITY))) {
      amax = 0.f;
#pragma unroll
      for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int j = 0; j < 16; ++j) {
          const float m = __builtin_fabsf(acc[0][nb][j]);
          amax = __builtin_fmaxf(amax, 32 * nb + c < N && m < INFINITY ? m : 0.f);
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) amax = __builtin_fmaxf(amax, shfl_xor_f(amax, o));
    const int ex = min(max(__builtin_amdgcn_frexp_expf(amax), -100), 100);
    const float mul = __builtin_amdgcn_ldexpf(1.f, 15 - ex);
    uint16_t* dst = part.v + slot * NPAD * kStreamRows + 32 * wave;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
      if (32 * nb + c < N)
#pragma unroll
        for (int jq = 0; jq < 4; ++jq)
          *reinterpret_cast<u32x2*>(dst + (size_t)(32 * nb + c) * kStreamRows + 8 * jq + 4 * u) =
              u32x2{pack_f16x2(acc[0][nb][4 * jq] * mul, acc[0][nb][4 * jq + 1] * mul),
                    pack_f16x2(acc[0][nb][4 * jq + 2] * mul, acc[0][nb][4 * jq + 3] * mul)};
    if (lane == 0) part.sc[slot * 4 + wave] = __builtin_amdgcn_ldexpf(1.f, ex - 15);
  }
}

// W sources of the kernel below: unit g's 16 gate rows, then its 16 up rows
// (row 16 + r of the slot swizzles as row r).
template <int RG, bool PACKED>
struct PairSlots {
  const uint16_t* W;
  int KC, K, inter, lane;
  const uint16_t* p[RG][2];
  __device__ __forceinline__ PairSlots(const uint16_t* w, int kc, int k, int i, int ln)
      : W(w), KC(kc), K(k), inter(i), lane(ln) {}
  __device__ __forceinline__ void set(int r, int g, int kc) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int row0 = 16 * g + h * inter;
      p[r][h] = PACKED ? W + ((size_t)(row0 / 128) * KC + kc) * (kStreamRows * 64) + (row0 % 128) * 64
                       : W + (size_t)row0 * K + kc * 64;
    }
  }
  __device__ __forceinline__ void dma(int r, uint8_t* dst) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
      for (int jj = 0; jj < 2; ++jj) {
        const int row = 8 * jj + lane / 8;
        const uint16_t* src = PACKED ? p[r][h] + jj * 512 + lane * 8
                                     : p[r][h] + (size_t)row * K + ((lane % 8) ^ piece_swz(row)) * 8;
        __builtin_amdgcn_global_load_lds(OOO_GLB(src), OOO_LDS(dst + h * 2048 + jj * 1024), 16, 0, kStreamOnce);
      }
      p[r][h] += PACKED ? kStreamRows * 64 : 64;
    }
  }
};

// silu(gate) * up without partial sums: a block owns whole output columns.
// A unit is 16 gate rows and the 16 up rows of the same columns; they share
// a 32-row slot (gate rows in its first half), so a lane's accumulators j
// and j + 8 are the gate and the up value of one output.  The units are
// dealt out evenly over the blocks, each block streams the whole K of its
// units, and the activation is applied to the float32 sums in registers:
// no workspace traffic, no second kernel, no fp16 rounding.
template <int NB, int RG, bool PACKED>
__global__ __launch_bounds__(kTallThreads) void linear_swiglu_kernel(const uint16_t* __restrict__ X,
                                                                     const uint16_t* __restrict__ Wt, int N, int K,
                                                                     int inter, Deal deal, Ring ring,
                                                                     uint16_t* __restrict__ out) {
  __shared__ __attribute__((aligned(1024))) uint8_t lds[kRingBytes];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int KC = K / 64;
  const int grid = (int)gridDim.x, b = (int)blockIdx.x;
  const int T = deal.T;
  const auto tile = [&](int t) { return GroupRange{deal.first(b + t * grid), deal.first(b + t * grid + 1)}; };

  if (wave >= 4) {
    const int ld = wave - 4;
    XShare<NB> xs(X, N, K, ld, lane);
    PairSlots<RG, PACKED> slots(Wt, KC, K, inter, lane);
    tall_load<NB, RG>(0, 0, T * KC, KC, deal.per, ld, tile, slots, xs, ring, lds);
    return;
  }

  const int c = lane & 31, u = lane >> 5;
  uint32_t off[4];
  frag_offsets(lane, off);
  int stage = 0;
  wg_barrier();  // the first chunk has landed
  for (int t = 0; t < T; ++t) {
    const int u0 = tile(t).lo, ng = tile(t).hi - u0;
    f32x16 acc[RG][NB];
#pragma unroll
    for (int r = 0; r < RG; ++r)
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) acc[r][nb] = f32x16{};
    tall_tile<NB, RG>(KC, t + 1 == T, ng, wave, lds, ring, off, stage, acc);
    // acc[r][nb][j], j < 8: gate of column 16 unit + 8(j/4) + 4u + j%4, node 32nb + c; [j + 8]: its up value
#pragma unroll
    for (int r = 0; r < RG; ++r) {
      if (wave + 4 * r >= ng) break;
      uint16_t* o = out + 16 * (u0 + wave + 4 * r) + 4 * u;
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        const int n = 32 * nb + c;
        if (n >= N) continue;
#pragma unroll
        for (int jq = 0; jq < 2; ++jq) {
          float y[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float gt = acc[r][nb][4 * jq + e];
            y[e] = gt / (1.f + expf(-gt)) * acc[r][nb][8 + 4 * jq + e];
          }
          *reinterpret_cast<u32x2*>(o + (size_t)n * inter + 8 * jq) =
              u32x2{pack_bf16x2(y[0], y[1]), pack_bf16x2(y[2], y[3])};
        }
      }
    }
  }
}

enum Epi { kStoreF32 = 0, kStoreBF16 = 1, kAddF32 = 2, kSwiGLU = 3 };

// Where a tile's partials are: in block order, first the slot `s0` (the run
// that holds the tile's first chunk, which may have begun in an earlier
// tile), then segment 0 of each of the next n - 1 runs.
struct TileSlots {
  int s0, next, seg, n;
  __device__ __forceinline__ int at(int i) const { return i == 0 ? s0 : next + i * seg; }
};
__device__ __forceinline__ TileSlots tile_slots(const Runs& runs, int KC, int t) {
  const int b0 = runs.of(t * KC), b1 = runs.of(t * KC + KC - 1);
  const int first = (int)((unsigned)runs.lo(b0) / (unsigned)KC);
  return TileSlots{b0 * runs.seg + (t - first), b0 * runs.seg, runs.seg, b1 - b0 + 1};
}

// Sum of the partials at (node n, tile row r): element e = n * 128 + r, in block
// order whichever kernel adds them (the same rounding).  The loads of a batch of S slots (S = 4, 8 or 16, the smallest
// that holds the list; longer lists take several batches) are all issued
// before the first add, so a sum costs one round trip to memory; slots past
// the end of the list re-read the last one and are not added.
typedef float f32x8 __attribute__((ext_vector_type(8)));
// fp16 partial values: 8 (f32x8), 4 (f32x4) or 1 (float)
__device__ __forceinline__ void load_part(const uint16_t* p, f32x8& x) {
  const u32x4 h = *reinterpret_cast<const u32x4*>(p);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const f32x2_t v = unpack_f16x2(h[i]);
    x[2 * i] = v[0];
    x[2 * i + 1] = v[1];
  }
}
__device__ __forceinline__ void load_part(const uint16_t* p, f32x4& x) {
  const u32x2 h = *reinterpret_cast<const u32x2*>(p);
  const f32x2_t lo = unpack_f16x2(h[0]), hi = unpack_f16x2(h[1]);
  x = f32x4{lo[0], lo[1], hi[0], hi[1]};
}
__device__ __forceinline__ void load_part(const uint16_t* p, float& x) { x = unpack_f16x2(*p)[0]; }
template <typename T, int S>
__device__ __forceinline__ T slot_batches(const Partials& part, const TileSlots& ts, int npad, int n, int r) {
  T s{};
  const size_t stride = (size_t)npad * kStreamRows, e = (size_t)n * kStreamRows + r;
  for (int i0 = 0; i0 < ts.n; i0 += S) {
    T x[S];
    float sc[S];
#pragma unroll
    for (int i = 0; i < S; ++i) {
      const int k = ts.at(min(i0 + i, ts.n - 1));
      load_part(part.v + k * stride + e, x[i]);
      sc[i] = part.sc[k * 4 + r / 32];
    }
#pragma unroll
    for (int i = 0; i < S; ++i)
      if (i0 + i < ts.n) s += x[i] * sc[i];
  }
  return s;
}
// The same at rows r0 and r1 of one tile, both rows' loads in flight together.
template <int S>
__device__ __forceinline__ f32x2_t slot_pair_batches(const Partials& part, const TileSlots& ts, int npad, int n, int r0,
                                                     int r1) {
  f32x2_t s{};
  const size_t stride = (size_t)npad * kStreamRows, e = (size_t)n * kStreamRows;
  for (int i0 = 0; i0 < ts.n; i0 += S) {
    float x[2][S], sc[2][S];
#pragma unroll
    for (int i = 0; i < S; ++i) {
      const int k = ts.at(min(i0 + i, ts.n - 1));
      load_part(part.v + k * stride + e + r0, x[0][i]);
      load_part(part.v + k * stride + e + r1, x[1][i]);
      sc[0][i] = part.sc[k * 4 + r0 / 32];
      sc[1][i] = part.sc[k * 4 + r1 / 32];
    }
#pragma unroll
    for (int i = 0; i < S; ++i)
      if (i0 + i < ts.n) {
        s[0] += x[0][i] * sc[0][i];
        s[1] += x[1][i] * sc[1][i];
      }
  }
  return s;
}
__device__ __forceinline__ f32x2_t slot_pair_of(const Partials& part, const TileSlots& ts, int npad, int n, int r0,
                                                int r1) {
  if (ts.n <= 4) return slot_pair_batches<4>(part, ts, npad, n, r0, r1);
  if (ts.n <= 8) return slot_pair_batches<8>(part, ts, npad, n, r0, r1);
  return slot_pair_batches<16>(part, ts, npad, n, r0, r1);
}
template <typename T>
__device__ __forceinline__ T slot_sum_of(const Partials& part, const TileSlots& ts, int npad, int n, int r) {
  if (ts.n <= 4) return slot_batches<T, 4>(part, ts, npad, n, r);
  if (ts.n <= 8) return slot_batches<T, 8>(part, ts, npad, n, r);
  return slot_batches<T, 16>(part, ts, npad, n, r);
}

// Four blocks per 128 output rows (per 128 gate rows for kSwiGLU): block q
// takes rows 64 (q % 2) .. +63 of the nodes n = q / 2 (mod 2); thread item
// (n, 8 consecutive rows), so every partial read is 16 bytes and eight
// lanes read one node's whole 128-byte line.
__global__ __launch_bounds__(256) void linear_reduce_kernel(Partials part, int npad, Runs runs, int N, int K, int O,
                                                            int epi, void* __restrict__ out, int inter) {
  const int row0 = (int)(blockIdx.x >> 2) * 128 + (int)(blockIdx.x & 1) * 64, par = (blockIdx.x >> 1) & 1;
  const int KC = K / 64;
  const int t0 = row0 / kStreamRows, t1 = (row0 + inter) / kStreamRows;
  const TileSlots ts0 = tile_slots(runs, KC, t0);
  const TileSlots ts1 = epi == kSwiGLU ? tile_slots(runs, KC, t1) : ts0;
  for (int item = threadIdx.x; item < (N - par + 1) / 2 * 8; item += 256) {
    const int n = 2 * (item >> 3) + par, col = row0 + 8 * (item & 7);
    const f32x8 sv = slot_sum_of<f32x8>(part, ts0, npad, n, col - t0 * kStreamRows);
    if (epi == kSwiGLU) {
      const f32x8 uv = slot_sum_of<f32x8>(part, ts1, npad, n, col + inter - t1 * kStreamRows);
      uint16_t* o = reinterpret_cast<uint16_t*>(out) + (size_t)n * inter + col;
#pragma unroll
      for (int j = 0; j < 8; ++j)
        if (col + j < inter) o[j] = (uint16_t)(pack_bf16x2(sv[j] / (1.f + expf(-sv[j])) * uv[j], 0.f) & 0xFFFFu);
      continue;
    }
    const size_t o = (size_t)n * O + col;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      if (col + j >= O) break;
      if (epi == kStoreF32) reinterpret_cast<float*>(out)[o + j] = sv[j];
      else if (epi == kAddF32) reinterpret_cast<float*>(out)[o + j] += sv[j];
      else reinterpret_cast<uint16_t*>(out)[o + j] = (uint16_t)(pack_bf16x2(sv[j], 0.f) & 0xFFFFu);
    }
  }
}

// Projection epilogue fused with the next RMSNorm: for row n,
// h[n] += the projection (its partial sums), then out[n] = bf16(h[n] /
// sqrt(mean(h[n]^2) + eps) * w).  One block per row, one float4 column group
// per thread and item (out_dim <= 8192: up to two items of 1024 threads), so
// that a row's loads are all in flight at once.
constexpr int kAddNormItems = 2;
__global__ __launch_bounds__(1024) void linear_add_rmsnorm_kernel(Partials part, int npad, Runs runs, int K, int O,
                                                                  float* __restrict__ resid,
                                                                  const uint16_t* __restrict__ w, float eps,
                                                                  uint16_t* __restrict__ out) {
  __shared__ float red[16];
  const int n = blockIdx.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nt = blockDim.x;
  const int KC = K / 64;
  float* hrow = resid + (size_t)n * O;
  f32x4 hv[kAddNormItems];
  u32x2 wv[kAddNormItems];
  float ss = 0.f;
#pragma unroll
  for (int i = 0; i < kAddNormItems; ++i) {
    const int c = 4 * (threadIdx.x + nt * i);
    hv[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    wv[i] = u32x2{0u, 0u};
    if (c < O) {
      hv[i] = *reinterpret_cast<const f32x4*>(hrow + c);
      wv[i] = *reinterpret_cast<const u32x2*>(w + c);
    }
  }
#pragma unroll
  for (int i = 0; i < kAddNormItems; ++i) {
    const int c = 4 * (threadIdx.x + nt * i);
    if (c < O) {
      const int t = c / kStreamRows;
      hv[i] += slot_sum_of<f32x4>(part, tile_slots(runs, KC, t), npad, n, c - t * kStreamRows);
      *reinterpret_cast<f32x4*>(hrow + c) = hv[i];
    }
  }
#pragma unroll
  for (int i = 0; i < kAddNormItems; ++i)
#pragma unroll
    for (int e = 0; e < 4; ++e) ss = __builtin_fmaf(hv[i][e], hv[i][e], ss);
  for (int off = 32; off > 0; off >>= 1) ss += shfl_xor_f(ss, off);
  if (lane == 0) red[wave] = ss;
  __syncthreads();
  float tot = 0.f;
  for (int k = 0; k < nt / 64; ++k) tot += red[k];
  const float r = 1.f / sqrtf(tot / (float)O + eps);
#pragma unroll
  for (int i = 0; i < kAddNormItems; ++i) {
    const int c = 4 * (threadIdx.x + nt * i);
    if (c < O) {
      u32x2 o;
      o[0] = pack_bf16x2(hv[i][0] * r * __uint_as_float(wv[i][0] << 16),
                         hv[i][1] * r * __uint_as_float(wv[i][0] & 0xFFFF0000u));
      o[1] = pack_bf16x2(hv[i][2] * r * __uint_as_float(wv[i][1] << 16),
                         hv[i][3] * r * __uint_as_float(wv[i][1] & 0xFFFF0000u));
      *reinterpret_cast<u32x2*>(out + (size_t)n * O + c) = o;
    }
  }
}

// Projection epilogue fused with the q/k norms and the rotation: block
// (node n, 16 heads), one wave per head of the fused q/k/v projection.  Lane
// j < D/2 sums the partials of its pair (j, j + D/2) in float32 and then
// proceeds as the rotation kernel: per-head RMSNorm of q and k, rotation at
// position P + depth[n], q to q_out, k and v (rounded to bf16) to cache row
// P + n.
template <int D>
__global__ __launch_bounds__(1024) void linear_qk_norm_rope_kernel(
    Partials part, int npad, Runs runs, int K, const uint16_t* __restrict__ q_norm,
    const uint16_t* __restrict__ k_norm, float eps, const int32_t* __restrict__ depth, int P,
    const int32_t* __restrict__ P_dev, RopeFreq fr, int Hq, int Hkv, uint16_t* __restrict__ q_out,
    uint16_t* __restrict__ k_cache, uint16_t* __restrict__ v_cache, long long cap) {
  constexpr int HALF = D / 2;
  static_assert(kStreamRows % D == 0, "a head lies in one tile");
  if (P_dev) P = min(max(*P_dev, 0), P);
  const int n = blockIdx.x, lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nh = Hq + 2 * Hkv;
  const int hh = blockIdx.y * 16 + wave;
  if (hh >= nh) return;
  const int t = hh * D / kStreamRows, r0 = hh * D - t * kStreamRows;
  const TileSlots ts = tile_slots(runs, K / 64, t);
  const long long row = (long long)P + n;
  const bool act = lane < HALF, is_q = hh < Hq, is_v = hh >= Hq + Hkv;
  // Every load is issued before the partial sums are waited for (the pair's
  // partials together, the weights and the depth ahead of them): with one
  // round trip instead of four, two Qwen3-8B layers 240.8 -> 240.1 us at 64
  // nodes, one layer at H 5120, 128 nodes 278.8 -> 277.1.
  const int dp = depth[n];
  const double freq = fr.f[lane % HALF];
  const uint16_t* nw = is_v ? nullptr : is_q ? q_norm : k_norm;
  float wa = 1.f, wb = 1.f;
  if (nw && act) {
    wa = bf16_bits_to_f32(nw[lane]);
    wb = bf16_bits_to_f32(nw[lane + HALF]);
  }
  float a = 0.f, b = 0.f;
  if (act) {
    const f32x2_t ab = slot_pair_of(part, ts, npad, n, r0 + lane, r0 + lane + HALF);
    a = ab[0];
    b = ab[1];
  }
  if (is_v) {
    uint16_t* dst = v_cache + ((size_t)(hh - Hq - Hkv) * cap + row) * D;
    if (act) {
      dst[lane] = f32_to_bf16_bits(a);
      dst[lane + HALF] = f32_to_bf16_bits(b);
    }
    return;
  }
  float cs = 1.f, sn = 0.f;
  if (act) rope_sincos(P + dp, freq, sn, cs);
  norm_rotate(a, b, nw != nullptr, wa, wb, eps, D, cs, sn);
  uint16_t* dst = is_q ? q_out + ((size_t)n * Hq + hh) * D : k_cache + ((size_t)(hh - Hq) * cap + row) * D;
  if (act) {
    dst[lane] = f32_to_bf16_bits(a);
    dst[lane + HALF] = f32_to_bf16_bits(b);
  }
}

struct LinPlan {
  int nb;
  long long chunks;  // (128-row tile, 64-column chunk) blocks of the weight
  Runs runs;
  size_t val_bytes;  // fp16 partial values (the factors follow)
  size_t ws_bytes;
};

Partials partials_in(void* workspace, const LinPlan& p) {
  return Partials{(uint16_t*)workspace, (float*)((uint8_t*)workspace + p.val_bytes)};
}

LinPlan lin_plan(int N, int K, int O) {
  LinPlan p{};
  p.nb = N <= 32 ? 1 : N <= 64 ? 2 : N <= 128 ? 4 : 8;
  const int KC = K / 64;
  p.chunks = (O + (long long)kStreamRows - 1) / kStreamRows * KC;
  p.runs = cut_runs(p.chunks, p.chunks < device_cus() ? (int)p.chunks : device_cus(), KC,
                    (long long)N * K * 2 > (4 << 20));
  const size_t slots = (size_t)p.runs.B * p.runs.seg;
  p.val_bytes = (slots * (32 * p.nb) * kStreamRows * sizeof(uint16_t) + 255) / 256 * 256;
  p.ws_bytes = p.val_bytes + slots * 4 * sizeof(float);
  return p;
}

}  // namespace
}  // namespace ooo

using namespace ooo;

extern "C" size_t ooo_linear_packed_bytes(int32_t out_dim, int32_t in_dim) {
  return ooo_lmhead_packed_bytes(out_dim, in_dim, OOO_BF16);
}

extern "C" int ooo_linear_pack(const void* weight, int32_t out_dim, int32_t in_dim, void* packed, size_t packed_bytes,
                               void* stream) {
  return ooo_lmhead_pack(weight, out_dim, in_dim, OOO_BF16, packed, packed_bytes, stream);
}

extern "C" size_t ooo_linear_workspace(int32_t n_rows, int32_t in_dim, int32_t out_dim) {
  if (n_rows < 1 || n_rows > 256 || in_dim < 64 || in_dim % 64 || out_dim < 1) return 0;
  return lin_plan(n_rows, in_dim, out_dim).ws_bytes;
}

// The fused epilogues refuse shapes whose chunks, cut at C b / B on at most
// 256 blocks, put more than 64 runs on one 128-row tile (very few tiles under
// a long K: 256 columns under K 8192).  Only the entry points' contract asks
// for it: earlier epilogues kept a tile's runs in lists of 64, these take any
// number in batches of 16, and the count is of that cut, whichever the kernels
// use, so that the same shapes are refused as ever.
constexpr int kMaxTileRuns = 64;
static bool too_many_runs(int n_rows, int in_dim, int out_dim) {
  if (n_rows < 1 || in_dim < 64 || in_dim % 64 || n_rows > 256 || out_dim < 1) return false;  // refused elsewhere
  const long long KC = in_dim / 64, tiles = (out_dim + 127LL) / 128, C = tiles * KC;
  const long long cus = device_cus() < 256 ? device_cus() : 256, B = C < cus ? C : cus;
  if (B / tiles + 2 <= kMaxTileRuns) return false;
  for (long long t = 0; t < tiles; ++t) {
    int n = 0;
    for (long long b = 0; b < B; ++b) n += C * b / B < (t + 1) * KC && C * (b + 1) / B > t * KC;
    if (n > kMaxTileRuns) return true;
  }
  return false;
}

// Validation shared by the entry points; on success *plan is set.
static int lin_check(const char* who, const void* x, const void* weight, int32_t n_rows, int32_t in_dim,
                     int32_t out_dim, int32_t weight_layout, const void* workspace, size_t ws_bytes, LinPlan* plan) {
  OOO_REQUIRE(x && weight, OOO_ERR_INVALID, "%s: null pointer", who);
  OOO_REQUIRE(n_rows >= 1 && in_dim >= 1 && out_dim >= 1, OOO_ERR_INVALID, "%s: sizes must be positive", who);
  OOO_REQUIRE(weight_layout == OOO_W_ROWS || weight_layout == OOO_W_PACKED, OOO_ERR_INVALID,
              "%s: unknown weight layout %d", who, weight_layout);
  OOO_REQUIRE(in_dim % 64 == 0, OOO_ERR_UNSUPPORTED, "%s: in_dim %% 64 != 0", who);
  OOO_REQUIRE(n_rows <= 256, OOO_ERR_UNSUPPORTED, "%s: at most 256 rows", who);
  const LinPlan p = lin_plan(n_rows, in_dim, out_dim);
  OOO_REQUIRE(workspace && ws_bytes >= p.ws_bytes, OOO_ERR_CAPACITY, "%s: workspace of %zu bytes needed (got %zu)",
              who, p.ws_bytes, ws_bytes);
  // the kernels count chunks in 32 bits; 2^31 of them are 32 TiB of weight
  OOO_REQUIRE(p.chunks <= INT32_MAX, OOO_ERR_UNSUPPORTED, "%s: weight of %lld 16 KiB blocks", who, p.chunks);
  *plan = p;
  return OOO_OK;
}

// The streaming kernel shared by the entry points: leaves the partial sums
// in the workspace.
static int stream_k(const char* who, const void* x, const void* weight, int32_t n_rows, int32_t in_dim,
                    int32_t out_dim, int32_t weight_layout, void* workspace, size_t ws_bytes, hipStream_t st,
                    LinPlan* plan) {
  LinPlan p{};
  const int rc = lin_check(who, x, weight, n_rows, in_dim, out_dim, weight_layout, workspace, ws_bytes, &p);
  if (rc != OOO_OK) return rc;
  const uint16_t* X = (const uint16_t*)x;
  const uint16_t* W = (const uint16_t*)weight;
  const Partials part = partials_in(workspace, p);
  const bool pk = weight_layout == OOO_W_PACKED;
  const int groups = (out_dim + 31) / 32;
  const Ring ring = make_ring(groups < 4 ? groups : 4, n_rows, p.nb);
#define OOO_LIN_LAUNCH(NBV)                                                                                            \
  do {                                                                                                                \
    if (pk)                                                                                                           \
      linear_bf16_kernel<NBV, true><<<p.runs.B, kTallThreads, 0, st>>>(X, W, n_rows, in_dim, out_dim, p.runs, ring,    \
                                                                       part);                                         \
    else                                                                                                              \
      linear_bf16_kernel<NBV, false><<<p.runs.B, kTallThreads, 0, st>>>(X, W, n_rows, in_dim, out_dim, p.runs, ring,   \
                                                                        part);                                        \
  } while (0)
  if (p.nb == 1) OOO_LIN_LAUNCH(1);
  else if (p.nb == 2) OOO_LIN_LAUNCH(2);
  else if (p.nb == 4) OOO_LIN_LAUNCH(4);
  else OOO_LIN_LAUNCH(8);
#undef OOO_LIN_LAUNCH
  *plan = p;
  return OOO_OK;
}

// Whether the SwiGLU projection owns whole columns per block or goes through
// stream-K.  With u units per CU a block of the direct kernel takes about
// KC max(flat, slope u), where below one or two units a CU the chunk
// pipeline's own period binds (flat) and not the bytes, and stream-K with its
// second kernel KC slope u + ahead: so stream-K is ahead for few units under a
// long K.  The prices (0.01 us) are fitted to both kernels at 14 shapes (K 1024
// to 8192, I 2176 to 27648; weights read from HBM each call) and 7 row counts;
// the choice is the better one, within 1 %, at each.  Direct / stream-K us at
// 1, 64, 128 and 256 rows: K 4096, I 4352 (u 1.06) 19.1 / 18.8, 22.5 / 22.1,
// 34.7 / 30.0, 51.8 / 43.9; I 6016 (1.47) 20.4 / 22.9, 26.5 / 26.9, 37.1 /
// 35.7, 52.7 / 51.1; I 12416 (3.03) 37.0 / 39.3, 39.2 / 45.3, 48.6 / 59.0,
// 75.2 / 79.8; K 8192, I 4352 36.1 / 29.2, 45.1 / 33.7, 65.9 / 44.5, 97.0 /
// 62.2; I 7168 (1.75) 48.9 / 42.9, 50.6 / 48.8, 67.9 / 60.4, 102.1 / 84.9; K
// 1024, I 3072 (0.75) 6.8 / 9.6, 7.7 / 12.8, 10.6 / 18.0, 16.5 / 29.8.
// The direct kernel stores four outputs (8 bytes) at a time; an output that
// is not aligned for it goes through stream-K, whose epilogue stores each.
static bool swiglu_direct(int n_rows, int in_dim, int inter, const void* out) {
  if (reinterpret_cast<uintptr_t>(out) % 8) return false;
  struct Price {
    int flat, slope, ahead;
  };
  const Price p = n_rows <= 64 ? Price{30, 13, 800} : n_rows <= 128 ? Price{49, 22, 1000} : Price{78, 29, 2000};
  const long long KC = in_dim / 64, units = inter / 16, cus = device_cus();
  return KC * (p.flat * cus - p.slope * units) < p.ahead * cus;
}

static void launch_swiglu(int nb, bool pk, const uint16_t* X, const uint16_t* W, int N, int K, int inter, uint16_t* out,
                          hipStream_t st) {
  const int units = inter / 16;
  const int blocks = units < device_cus() ? units : device_cus();
  const bool tall = (units + blocks - 1) / blocks > 4;
  const Deal deal = make_deal(units, blocks, tall && nb < 8 ? 2 : 1);
  const Ring ring = make_ring(deal.slots(), N, nb);
#define OOO_SW_LAUNCH(NBV, RGV)                                                                                  \
  do {                                                                                                          \
    if (pk) linear_swiglu_kernel<NBV, RGV, true><<<blocks, kTallThreads, 0, st>>>(X, W, N, K, inter, deal, ring, out); \
    else linear_swiglu_kernel<NBV, RGV, false><<<blocks, kTallThreads, 0, st>>>(X, W, N, K, inter, deal, ring, out);   \
  } while (0)
  if (nb == 1 && tall) OOO_SW_LAUNCH(1, 2);
  else if (nb == 1) OOO_SW_LAUNCH(1, 1);
  else if (nb == 2 && tall) OOO_SW_LAUNCH(2, 2);
  else if (nb == 2) OOO_SW_LAUNCH(2, 1);
  else if (nb == 4 && tall) OOO_SW_LAUNCH(4, 2);
  else if (nb == 4) OOO_SW_LAUNCH(4, 1);
  else OOO_SW_LAUNCH(8, 1);
#undef OOO_SW_LAUNCH
}

extern "C" int ooo_linear(const void* x, const void* weight, int32_t n_rows, int32_t in_dim, int32_t out_dim,
                          int32_t weight_layout, ooo_epilogue epilogue, void* out, void* workspace, size_t ws_bytes,
                          void* stream) {
  OOO_REQUIRE(out, OOO_ERR_INVALID, "ooo_linear: null pointer");
  OOO_REQUIRE(epilogue >= OOO_EPI_STORE_F32 && epilogue <= OOO_EPI_SWIGLU_BF16, OOO_ERR_INVALID,
              "ooo_linear: unknown epilogue %d", (int)epilogue);
  OOO_REQUIRE(epilogue != OOO_EPI_SWIGLU_BF16 || out_dim % 256 == 0, OOO_ERR_UNSUPPORTED,
              "ooo_linear: the SwiGLU epilogue needs out_dim %% 256 == 0 (gate and up halves of whole tiles)");
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  LinPlan p{};
  if (epilogue == OOO_EPI_SWIGLU_BF16 && swiglu_direct(n_rows, in_dim, out_dim / 2, out)) {
    const int rc = lin_check("ooo_linear", x, weight, n_rows, in_dim, out_dim, weight_layout, workspace, ws_bytes, &p);
    if (rc != OOO_OK) return rc;
    launch_swiglu(p.nb, weight_layout == OOO_W_PACKED, (const uint16_t*)x, (const uint16_t*)weight, n_rows, in_dim,
                  out_dim / 2, (uint16_t*)out, st);
    const hipError_t e = hipGetLastError();
    OOO_REQUIRE(e == hipSuccess, OOO_ERR_HIP, "ooo_linear: launch failed: %s", hipGetErrorString(e));
    return ooo::ok();
  }
  const int rc = stream_k("ooo_linear", x, weight, n_rows, in_dim, out_dim, weight_layout, workspace, ws_bytes, st, &p);
  if (rc != OOO_OK) return rc;
  const Partials part = partials_in(workspace, p);
  const int rows = epilogue == OOO_EPI_SWIGLU_BF16 ? out_dim / 2 : out_dim;
  linear_reduce_kernel<<<4 * ((rows + 127) / 128), 256, 0, st>>>(part, 32 * p.nb, p.runs, n_rows, in_dim, out_dim,
                                                                 (int)epilogue, out, out_dim / 2);
  const hipError_t e = hipGetLastError();
  OOO_REQUIRE(e == hipSuccess, OOO_ERR_HIP, "ooo_linear: launch failed: %s", hipGetErrorString(e));
  return ooo::ok();
}

extern "C" int ooo_linear_add_rmsnorm(const void* x, const void* weight, int32_t n_rows, int32_t in_dim,
                                      int32_t out_dim, int32_t weight_layout, float* residual,
                                      const void* norm_weight, float eps, void* normed_out, void* workspace,
                                      size_t ws_bytes, void* stream) {
  OOO_REQUIRE(residual && norm_weight && normed_out, OOO_ERR_INVALID, "ooo_linear_add_rmsnorm: null pointer");
  OOO_REQUIRE(eps >= 0.f, OOO_ERR_INVALID, "ooo_linear_add_rmsnorm: eps must be >= 0");
  OOO_REQUIRE(out_dim % 4 == 0 && out_dim <= 1024 * 4 * kAddNormItems, OOO_ERR_UNSUPPORTED,
              "ooo_linear_add_rmsnorm: out_dim %d must be a multiple of 4 and at most %d", out_dim,
              1024 * 4 * kAddNormItems);
  OOO_REQUIRE(!too_many_runs(n_rows, in_dim, out_dim), OOO_ERR_UNSUPPORTED,
              "ooo_linear_add_rmsnorm: more than %d partial slots per tile at this shape", kMaxTileRuns);
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  LinPlan p{};
  const int rc = stream_k("ooo_linear_add_rmsnorm", x, weight, n_rows, in_dim, out_dim, weight_layout, workspace,
                          ws_bytes, st, &p);
  if (rc != OOO_OK) return rc;
  const int threads = out_dim / 4 >= 1024 ? 1024 : (out_dim / 4 + 63) / 64 * 64;
  linear_add_rmsnorm_kernel<<<n_rows, threads, 0, st>>>(partials_in(workspace, p), 32 * p.nb, p.runs, in_dim, out_dim,
                                                        residual, (const uint16_t*)norm_weight, eps,
                                                        (uint16_t*)normed_out);
  const hipError_t e = hipGetLastError();
  OOO_REQUIRE(e == hipSuccess, OOO_ERR_HIP, "ooo_linear_add_rmsnorm: launch failed: %s", hipGetErrorString(e));
  return ooo::ok();
}

extern "C" int ooo_linear_qk_norm_rope(const void* x, const void* weight, int32_t n_rows, int32_t in_dim,
                                       int32_t weight_layout, const void* q_norm, const void* k_norm, float eps,
                                       const int32_t* depth, int32_t prefix_len, const int32_t* prefix_len_dev,
                                       double rope_theta, int32_t n_q_heads, int32_t n_kv_heads, int32_t head_dim,
                                       void* q_out, void* k_cache, void* v_cache, int64_t cap, void* workspace,
                                       size_t ws_bytes, void* stream) {
  OOO_REQUIRE(depth && q_out && k_cache && v_cache, OOO_ERR_INVALID, "ooo_linear_qk_norm_rope: null pointer");
  OOO_REQUIRE(n_q_heads >= 1 && n_kv_heads >= 1 && prefix_len >= 0, OOO_ERR_INVALID,
              "ooo_linear_qk_norm_rope: sizes must be positive");
  OOO_REQUIRE((int64_t)prefix_len + n_rows <= cap, OOO_ERR_INVALID,
              "ooo_linear_qk_norm_rope: prefix_len + n_rows (%lld) exceeds cap (%lld)", (long long)prefix_len + n_rows,
              (long long)cap);
  OOO_REQUIRE(rope_theta > 0.0 && eps >= 0.f, OOO_ERR_INVALID, "ooo_linear_qk_norm_rope: rope_theta must be > 0");
  OOO_REQUIRE(head_dim == 64 || head_dim == 128, OOO_ERR_UNSUPPORTED,
              "ooo_linear_qk_norm_rope: head_dim %d not supported (64 or 128)", head_dim);
  const int nh = n_q_heads + 2 * n_kv_heads;
  OOO_REQUIRE((int64_t)nh * head_dim % kStreamRows == 0, OOO_ERR_UNSUPPORTED,
              "ooo_linear_qk_norm_rope: (n_q_heads + 2 n_kv_heads) * head_dim must be a multiple of %d", kStreamRows);
  OOO_REQUIRE(!too_many_runs(n_rows, in_dim, nh * head_dim), OOO_ERR_UNSUPPORTED,
              "ooo_linear_qk_norm_rope: more than %d partial slots per tile at this shape", kMaxTileRuns);
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  LinPlan p{};
  const int rc = stream_k("ooo_linear_qk_norm_rope", x, weight, n_rows, in_dim, nh * head_dim, weight_layout,
                          workspace, ws_bytes, st, &p);
  if (rc != OOO_OK) return rc;
  const RopeFreq fr = rope_freq(rope_theta, head_dim);
  const dim3 grid(n_rows, (nh + 15) / 16);
  const Partials part = partials_in(workspace, p);
  if (head_dim == 128)
    linear_qk_norm_rope_kernel<128><<<grid, 1024, 0, st>>>(part, 32 * p.nb, p.runs, in_dim,
                                                            (const uint16_t*)q_norm, (const uint16_t*)k_norm, eps, depth,
                                                            prefix_len, prefix_len_dev, fr, n_q_heads, n_kv_heads,
                                                            (uint16_t*)q_out, (uint16_t*)k_cache, (uint16_t*)v_cache,
                                                            cap);
  else
    linear_qk_norm_rope_kernel<64><<<grid, 1024, 0, st>>>(part, 32 * p.nb, p.runs, in_dim,
                                                           (const uint16_t*)q_norm, (const uint16_t*)k_norm, eps, depth,
                                                           prefix_len, prefix_len_dev, fr, n_q_heads, n_kv_heads,
                                                           (uint16_t*)q_out, (uint16_t*)k_cache, (uint16_t*)v_cache,
                                                           cap);
  const hipError_t e = hipGetLastError();
  OOO_REQUIRE(e == hipSuccess, OOO_ERR_HIP, "ooo_linear_qk_norm_rope: launch failed: %s", hipGetErrorString(e));
  return ooo::ok();
}
