// LM head and greedy token of every trie node (Eq. 1: the next committed
// token is the target's most likely one; ties go to the lowest index).
//
// bf16 path: the product is W[V][H] x X[N][H]^T, a skinny GEMM that streams
// W from HBM once.  Up to 64 nodes HBM binds it; from 128 on the power cap
// does: the matrix cores' work and every byte moved into LDS lower the clock
// (2.4 GHz at 32 nodes, 1.6-1.7 at 128 and 256; with zero hidden rows the
// same kernel runs 128 nodes at 2.3 GHz and at the HBM rate).  So the design
// keeps whole lines in flight and moves few X bytes per W byte:
//  * A persistent grid, one block per CU, that walks tiles of up to 8
//    32-row groups (256 rows; 4 at 129-256 nodes, where the accumulators of
//    two groups a wave do not fit) round-robin: every tile re-reads all of X
//    from L2, so taller tiles move half the X bytes of 128-row ones.  The
//    tiles of a call are nearly equal (V 151936 on 256 blocks: three tiles
//    each of 6 or 7 groups), so no round runs with most slots empty.  A
//    contiguous range per block streams as fast but makes the first pass
//    over a new weight 50 us longer (275 against 225 us).
//    Per call, 128-row tiles of seven waves against this: 307.6 -> 280.4 us
//    at 128 nodes, H 5120, V 152064; 326.9 -> 310.4 at 256 nodes, H 4096, V
//    128256 (there the fragment reads a k-step ahead, below); 186.8 -> 185.7
//    at 64 nodes, H 4096, V 151936 (HBM-bound at 6.7 TB/s).
//  * The streaming core (stream_core.h): four loader waves copy each W
//    chunk (a group's 32 rows x 128 B per slot) and the X chunk (all nodes x
//    128 B) straight into an LDS ring with global_load_lds; four compute
//    waves own up to two groups each and run the MFMAs from LDS, never
//    issuing global loads in the loop, with the fragments of the next k-step
//    read under the MFMAs of this one.
//  * Each lane ends a tile with 16 logits per group of one node; the per-node
//    argmax is kept in registers across tiles, merged across the block's
//    waves in LDS and across blocks by a small finalize kernel (value, then
//    lowest index).
#include <math.h>

#include "device_common.h"
#include "ooo_internal.h"
#include "stream_core.h"

namespace ooo {
namespace {

struct Cand {
  float v;
  int i;
};

constexpr int kLmRows = kStreamRows;  // vocabulary rows per tile (4 waves x 32)

template <int NB, int RG, bool PACKED>
__global__ __launch_bounds__(kTallThreads) void lmhead_bf16_kernel(const uint16_t* __restrict__ X,
                                                                   const uint16_t* __restrict__ Wt, int N, int H,
                                                                   int V, Deal deal, Ring ring,
                                                                   Cand* __restrict__ partial,
                                                                   float* __restrict__ logits) {
  __shared__ __attribute__((aligned(1024))) uint8_t lds[kRingBytes];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int chunks = H / 64;
  const int b = (int)blockIdx.x, grid = (int)gridDim.x;
  const int T = deal.T;
  const auto tile = [&](int t) { return GroupRange{deal.first(b + t * grid), deal.first(b + t * grid + 1)}; };

  if (wave >= 4) {
    const int ld = wave - 4;
    XShare<NB> xs(X, N, H, ld, lane);
    GroupSlots<RG, PACKED> slots(Wt, chunks, V, H, lane);
    tall_load<NB, RG>(0, 0, T * chunks, chunks, deal.per, ld, tile, slots, xs, ring, lds);
    __syncthreads();  // matches the compute waves' barriers around the final reduction
    __syncthreads();
    return;
  }

  // ------------------------------------------------------------------ compute
  const int c = lane & 31, u = lane >> 5;
  uint32_t off[4];
  frag_offsets(lane, off);
  float bestv[NB];
  int besti[NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    bestv[nb] = -INFINITY;
    besti[nb] = 0x7FFFFFFF;
  }
  int stage = 0;
  wg_barrier();  // the first chunk has landed
  for (int t = 0; t < T; ++t) {
    const int g0 = tile(t).lo, ng = tile(t).hi - g0;
    f32x16 acc[RG][NB];
#pragma unroll
    for (int r = 0; r < RG; ++r)
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) acc[r][nb] = f32x16{};
    tall_tile<NB, RG>(chunks, t + 1 == T, ng, wave, lds, ring, off, stage, acc);
    // acc[r][nb][j] = logit of vocabulary row 32 g + 8(j/4) + 4u + j%4, g = g0 + wave + 4r, node 32nb + c
#pragma unroll
    for (int r = 0; r < RG; ++r) {
      if (wave + 4 * r >= ng) break;
      const int v0 = 32 * (g0 + wave + 4 * r);
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        float bv = -INFINITY;
        int bi = 0x7FFFFFFF;
#pragma unroll
        for (int j = 0; j < 16; ++j) {
          const int row = v0 + 8 * (j / 4) + 4 * u + (j % 4);
          if (row < V && acc[r][nb][j] > bv) {
            bv = acc[r][nb][j];
            bi = row;
          }
        }
        const float ov = shfl_xor_f(bv, 32);
        const int oi = shfl_xor_i(bi, 32);
        if (better(ov, oi, bv, bi)) {
          bv = ov;
          bi = oi;
        }
        if (better(bv, bi, bestv[nb], besti[nb])) {
          bestv[nb] = bv;
          besti[nb] = bi;
        }
        if (logits) {
          const int n = 32 * nb + c;
          if (n < N)
#pragma unroll
            for (int j = 0; j < 16; ++j) {
              const int row = v0 + 8 * (j / 4) + 4 * u + (j % 4);
              if (row < V) logits[(size_t)n * V + row] = acc[r][nb][j];
            }
        }
      }
    }
  }
  Cand* red = reinterpret_cast<Cand*>(lds);
  __syncthreads();  // every wave is past its last read of the ring
  if (u == 0)
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) red[wave * 32 * NB + 32 * nb + c] = Cand{bestv[nb], besti[nb]};
  __syncthreads();
  for (int n = threadIdx.x; n < N; n += 256) {
    Cand best = red[n];
    for (int w2 = 1; w2 < 4; ++w2) {
      const Cand o = red[w2 * 32 * NB + n];
      if (better(o.v, o.i, best.v, best.i)) best = o;
    }
    partial[(size_t)blockIdx.x * N + n] = best;
  }
}

// Packed weight layout: for tile t (128 rows) and chunk kc (64 columns), the
// 16 KiB block at ((t * chunks + kc) * 128 + r) * 64 elements holds row
// t*128 + r; its physical 16-byte piece p holds columns
// kc*64 + 8*(p ^ (r/2)%8) .. +8, the swizzle the kernel's LDS reads expect.
// Rows >= V are zero.
__global__ __launch_bounds__(256) void lmhead_pack_kernel(const uint16_t* __restrict__ W, int V, int H,
                                                          uint16_t* __restrict__ out, long long pieces) {
  const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
  if (i >= pieces) return;
  const int chunks = H / 64;
  const int p = (int)(i % 8);
  const int r = (int)((i / 8) % kLmRows);
  const long long tk = i / (8 * kLmRows);  // t * chunks + kc
  const int kc = (int)(tk % chunks);
  const long long t = tk / chunks;
  const long long row = t * kLmRows + r;
  u32x4 v = {0, 0, 0, 0};
  if (row < V) v = ld16(W + row * H + kc * 64 + ((p ^ piece_swz(r)) * 8));
  st16(out + i * 8, v);
}

// float32 path, on the f32 matrix instruction (16x16x4): a block takes tiles
// of 16 vocabulary rows against 16*NB nodes, its four waves a quarter of H
// each; the waves' partial products meet in LDS and wave nb turns those of
// node block nb into logits and running winners.  Operands go straight from
// memory to registers, 16 bytes per lane (four lanes cover 64 bytes of a
// row), 64 columns ahead of their use; lane (c, q) of step s holds columns
// 16 s + 4 q .. +3; the order of the columns inside a step is the same for
// both operands.  Bound by latency at small sizes and by reads of X from the
// L2 at large ones.  One thread per vocabulary row and a block column per
// node, the earlier form, read W once per node: per call 64 nodes x H 1024 x V
// 8000 took 325 us and now take 33, 100 x 1024 x 32000 12.9 ms and 177 us, 25 x
// 256 x 1024 13.2 and 7.6 us, 40 x 64 x 500 7.5 and 7.4.
template <int NB>
__global__ __launch_bounds__(256) void lmhead_f32_kernel(const float* __restrict__ X, const float* __restrict__ Wt,
                                                         int N, int H, int V, Cand* __restrict__ partial,
                                                         float* __restrict__ logits) {
  constexpr int U = 4;  // 16-column steps per round of loads
  __shared__ f32x4 red[4][NB][64];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int c = lane & 15, qd = lane >> 4;
  const int n0 = blockIdx.y * 16 * NB;
  const int kq = (H + 63) / 64 * 16;  // columns per wave
  const int k_begin = min(wave * kq, H), k_end = min(k_begin + kq, H);
  const int tiles = (V + 15) / 16;
  const float* xr[NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) xr[nb] = X + (size_t)min(n0 + 16 * nb + c, N - 1) * H;
  const int n = n0 + 16 * wave + c;  // the node of the lane's logits
  const bool vec = V % 4 == 0 && (reinterpret_cast<uintptr_t>(logits) & 15) == 0;
  Cand best{-INFINITY, 0x7FFFFFFF};
  const float* wr = Wt + (size_t)min(16 * (int)blockIdx.x + c, V - 1) * H;
  f32x4 wv[2][U], xv[2][NB][U], acc[NB][2];
  auto load = [&](int b, int k0) {  // steps past the wave's range are loaded from the row's end and not used
#pragma unroll
    for (int s = 0; s < U; ++s) {
      const int kk = min(k0 + 16 * s + 4 * qd, H - 4);
      wv[b][s] = *reinterpret_cast<const f32x4*>(wr + kk);
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) xv[b][nb][s] = *reinterpret_cast<const f32x4*>(xr[nb] + kk);
    }
  };
  auto mul_step = [&](int b, int s) {
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int nb = 0; nb < NB; ++nb)
        acc[nb][s & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(wv[b][s][j], xv[b][nb][s][j], acc[nb][s & 1], 0, 0, 0);
  };
  auto mul_full = [&](int b) {
#pragma unroll
    for (int s = 0; s < U; ++s) mul_step(b, s);
  };
  auto mul_tail = [&](int b, int k0) {
#pragma unroll
    for (int s = 0; s < U; ++s) {
      const int kk = k0 + 16 * s;
      if (kk >= k_end) break;
      if (kk + 16 > H && kk + 4 * qd >= H) {  // H no multiple of 16: zeros on both sides
        wv[b][s] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) xv[b][nb][s] = f32x4{0.f, 0.f, 0.f, 0.f};
      }
      mul_step(b, s);
    }
  };
  load(0, k_begin);
  for (int t = blockIdx.x; t < tiles; t += gridDim.x) {
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) acc[nb][0] = acc[nb][1] = f32x4{0.f, 0.f, 0.f, 0.f};
    // The loop's loads are unconditional: under a branch the wait for one
    // round would be a wait for all that are in flight.
    int k0 = k_begin;
    for (; k0 + 32 * U <= k_end; k0 += 32 * U) {
      load(1, k0 + 16 * U);
      mul_full(0);
      load(0, k0 + 32 * U);
      mul_full(1);
    }
    if (k0 < k_end) {
      if (k0 + 16 * U < k_end) load(1, k0 + 16 * U);
      mul_tail(0, k0);
      mul_tail(1, k0 + 16 * U);
    }
    wr = Wt + (size_t)min(16 * (t + (int)gridDim.x) + c, V - 1) * H;  // the next tile's first columns
    load(0, k_begin);
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) red[wave][nb][lane] = acc[nb][0] + acc[nb][1];
    __syncthreads();
    if (wave < NB && n < N) {
      const f32x4 l = (red[0][wave][lane] + red[1][wave][lane]) + (red[2][wave][lane] + red[3][wave][lane]);
      const int r0 = 16 * t + 4 * qd;
      if (logits && vec && r0 < V) {
        *reinterpret_cast<f32x4*>(logits + (size_t)n * V + r0) = l;
      } else if (logits) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (r0 + r < V) logits[(size_t)n * V + r0 + r] = l[r];
      }
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (r0 + r < V && better(l[r], r0 + r, best.v, best.i)) best = Cand{l[r], r0 + r};
    }
    __syncthreads();  // before the next tile's partials
  }
#pragma unroll
  for (int off = 16; off < 64; off *= 2) {
    const Cand o{shfl_xor_f(best.v, off), shfl_xor_i(best.i, off)};
    if (better(o.v, o.i, best.v, best.i)) best = o;
  }
  if (wave < NB && qd == 0 && n < N) partial[(size_t)blockIdx.x * N + n] = best;
}

// One block per node: best of the per-block winners, by shuffles in a wave and
// one barrier (a tree through LDS takes eight).
__global__ __launch_bounds__(256) void lmhead_finalize_kernel(const Cand* __restrict__ partial, int blocks, int N,
                                                              int32_t* __restrict__ ids, float* __restrict__ maxv) {
  __shared__ Cand red[4];
  const int n = blockIdx.x;
  Cand b{-INFINITY, 0x7FFFFFFF};
  for (int i = threadIdx.x; i < blocks; i += 256) {
    const Cand o = partial[(size_t)i * N + n];
    if (better(o.v, o.i, b.v, b.i)) b = o;
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    const Cand o{shfl_xor_f(b.v, off), shfl_xor_i(b.i, off)};
    if (better(o.v, o.i, b.v, b.i)) b = o;
  }
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = b;
  __syncthreads();
  if (threadIdx.x == 0) {
#pragma unroll
    for (int w = 1; w < 4; ++w)
      if (better(red[w].v, red[w].i, b.v, b.i)) b = red[w];
    ids[n] = b.i;
    maxv[n] = b.v;
  }
}

struct LmPlan {
  int nb, blocks;
  size_t ws_bytes;
};

LmPlan lm_plan(int N, int H, int V, ooo_dtype dt) {
  LmPlan p{};
  if (dt == OOO_BF16) {
    p.nb = N <= 32 ? 1 : N <= 64 ? 2 : N <= 128 ? 4 : 8;
    const int groups = (V + 31) / 32;
    p.blocks = groups < device_cus() ? groups : device_cus();  // persistent grid: one block per CU
  } else {
    p.nb = N <= 16 ? 1 : N <= 32 ? 2 : 4;
    const int tiles = (V + 15) / 16;
    p.blocks = tiles < 4 * device_cus() ? tiles : 4 * device_cus();  // four blocks of four waves per CU
  }
  p.ws_bytes = (size_t)p.blocks * N * sizeof(Cand);
  return p;
}

}  // namespace
}  // namespace ooo

using namespace ooo;

extern "C" size_t ooo_lmhead_workspace(int32_t n_nodes, int32_t hidden_dim, int32_t vocab, ooo_dtype dt) {
  if (n_nodes < 1 || hidden_dim < 1 || vocab < 1) return 0;
  return lm_plan(n_nodes, hidden_dim, vocab, dt).ws_bytes;
}

extern "C" size_t ooo_lmhead_packed_bytes(int32_t vocab, int32_t hidden_dim, ooo_dtype dt) {
  if (vocab < 1 || hidden_dim < 1 || hidden_dim % 64 || dt != OOO_BF16) return 0;
  const size_t tiles = (vocab + kLmRows - 1) / kLmRows;
  return tiles * kLmRows * (size_t)hidden_dim * 2;
}

extern "C" int ooo_lmhead_pack(const void* weight, int32_t vocab, int32_t hidden_dim, ooo_dtype dt, void* packed,
                               size_t packed_bytes, void* stream) {
  OOO_REQUIRE(weight && packed, OOO_ERR_INVALID, "ooo_lmhead_pack: null pointer");
  OOO_REQUIRE(vocab >= 1 && hidden_dim >= 1, OOO_ERR_INVALID, "ooo_lmhead_pack: sizes must be positive");
  OOO_REQUIRE(dt == OOO_BF16, OOO_ERR_UNSUPPORTED, "ooo_lmhead_pack: only OOO_BF16 weights are packed");
  OOO_REQUIRE(hidden_dim % 64 == 0, OOO_ERR_UNSUPPORTED, "ooo_lmhead_pack: hidden_dim %% 64 != 0");
  const size_t need = ooo_lmhead_packed_bytes(vocab, hidden_dim, dt);
  OOO_REQUIRE(packed_bytes >= need, OOO_ERR_CAPACITY, "ooo_lmhead_pack: %zu bytes needed (got %zu)", need,
              packed_bytes);
  const long long pieces = (long long)(need / 16);
  lmhead_pack_kernel<<<(unsigned)((pieces + 255) / 256), 256, 0, reinterpret_cast<hipStream_t>(stream)>>>(
      (const uint16_t*)weight, vocab, hidden_dim, (uint16_t*)packed, pieces);
  const hipError_t e = hipGetLastError();
  OOO_REQUIRE(e == hipSuccess, OOO_ERR_HIP, "ooo_lmhead_pack: launch failed: %s", hipGetErrorString(e));
  return ooo::ok();
}

extern "C" int ooo_lmhead_argmax(const void* hidden, const void* weight, int32_t n_nodes, int32_t hidden_dim,
                                 int32_t vocab, ooo_dtype dt, int32_t weight_layout, int32_t* argmax_ids,
                                 float* max_logit, float* logits, void* workspace, size_t ws_bytes, void* stream) {
  OOO_REQUIRE(hidden && weight && argmax_ids && max_logit, OOO_ERR_INVALID, "ooo_lmhead_argmax: null pointer");
  OOO_REQUIRE(n_nodes >= 1 && hidden_dim >= 1 && vocab >= 1, OOO_ERR_INVALID,
              "ooo_lmhead_argmax: sizes must be positive (n_nodes=%d hidden_dim=%d vocab=%d)", n_nodes,
              hidden_dim, vocab);
  OOO_REQUIRE(dt == OOO_F32 || dt == OOO_BF16, OOO_ERR_INVALID, "ooo_lmhead_argmax: unknown dtype %d", (int)dt);
  OOO_REQUIRE(weight_layout == OOO_W_ROWS || weight_layout == OOO_W_PACKED, OOO_ERR_INVALID,
              "ooo_lmhead_argmax: unknown weight layout %d", weight_layout);
  if (dt == OOO_BF16) {
    OOO_REQUIRE(hidden_dim % 64 == 0, OOO_ERR_UNSUPPORTED, "ooo_lmhead_argmax: bf16 needs hidden_dim %% 64 == 0");
    OOO_REQUIRE(n_nodes <= 256, OOO_ERR_UNSUPPORTED, "ooo_lmhead_argmax: bf16 supports up to 256 nodes");
  } else {
    OOO_REQUIRE(hidden_dim % 4 == 0, OOO_ERR_UNSUPPORTED, "ooo_lmhead_argmax: f32 needs hidden_dim %% 4 == 0");
    OOO_REQUIRE(n_nodes <= 65535, OOO_ERR_UNSUPPORTED, "ooo_lmhead_argmax: too many nodes");
    OOO_REQUIRE(weight_layout == OOO_W_ROWS, OOO_ERR_UNSUPPORTED, "ooo_lmhead_argmax: f32 weights are row-major only");
  }
  const LmPlan p = lm_plan(n_nodes, hidden_dim, vocab, dt);
  OOO_REQUIRE(workspace && ws_bytes >= p.ws_bytes, OOO_ERR_CAPACITY,
              "ooo_lmhead_argmax: workspace of %zu bytes needed (got %zu)", p.ws_bytes, ws_bytes);
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  Cand* part = reinterpret_cast<Cand*>(workspace);
  if (dt == OOO_BF16) {
    const uint16_t* X = (const uint16_t*)hidden;
    const uint16_t* W = (const uint16_t*)weight;
    const bool pk = weight_layout == OOO_W_PACKED;
    const int rg = p.nb == 8 ? 1 : 2;
    const Deal deal = make_deal((vocab + 31) / 32, p.blocks, rg);
    const Ring ring = make_ring(deal.slots(), n_nodes, p.nb);
#define OOO_LM_LAUNCH(NBV, RGV)                                                                                       \
  do {                                                                                                               \
    if (pk)                                                                                                          \
      lmhead_bf16_kernel<NBV, RGV, true><<<p.blocks, kTallThreads, 0, st>>>(X, W, n_nodes, hidden_dim, vocab, deal,   \
                                                                            ring, part, logits);                     \
    else                                                                                                             \
      lmhead_bf16_kernel<NBV, RGV, false><<<p.blocks, kTallThreads, 0, st>>>(X, W, n_nodes, hidden_dim, vocab, deal,  \
                                                                             ring, part, logits);                    \
  } while (0)
    if (p.nb == 1) OOO_LM_LAUNCH(1, 2);
    else if (p.nb == 2) OOO_LM_LAUNCH(2, 2);
    else if (p.nb == 4) OOO_LM_LAUNCH(4, 2);
    else OOO_LM_LAUNCH(8, 1);
#undef OOO_LM_LAUNCH
  } else {
    const dim3 grid(p.blocks, (n_nodes + 16 * p.nb - 1) / (16 * p.nb));
    const float* X = (const float*)hidden;
    const float* W = (const float*)weight;
    if (p.nb == 1) lmhead_f32_kernel<1><<<grid, 256, 0, st>>>(X, W, n_nodes, hidden_dim, vocab, part, logits);
    else if (p.nb == 2) lmhead_f32_kernel<2><<<grid, 256, 0, st>>>(X, W, n_nodes, hidden_dim, vocab, part, logits);
    else lmhead_f32_kernel<4><<<grid, 256, 0, st>>>(X, W, n_nodes, hidden_dim, vocab, part, logits);
  }
  lmhead_finalize_kernel<<<n_nodes, 256, 0, st>>>(part, p.blocks, n_nodes, argmax_ids, max_logit);
  const hipError_t e = hipGetLastError();
  OOO_REQUIRE(e == hipSuccess, OOO_ERR_HIP, "ooo_lmhead_argmax: launch failed: %s", hipGetErrorString(e));
  return ooo::ok();
}
