// Weight-streaming cores of the LM head (lmhead.hip; tall tiles, below) and
// the decoder projections (linear.hip): products W X^T of a weight W that is streamed
// once from HBM with a few node rows X (N <= 256) that every block re-reads
// from L2.
//  * W is cut into 128-row tiles and 64-column chunks; a chunk is 16 KiB,
//    four 32-row slots of 4 KiB.  In the packed layout (ooo_lmhead_pack)
//    chunk (t, kc) is one contiguous 16 KiB block, already swizzled; in the
//    row layout (nn.Linear) a slot is gathered row by row.
//  * In LDS the 16-byte piece p of row r sits at piece p ^ ((r / 2) % 8).
//    A 128-byte row covers half of gfx950's 64 LDS banks, so even and odd
//    rows fall in opposite halves, and a 16-byte read serves 16 lanes (16
//    rows, one piece) at a time: with the XOR by (r / 2) % 8 the eight rows
//    in each half read eight different pieces, all 64 banks once.  (An XOR
//    by r % 8 gave rows r and r + 8 the same banks: a 2-way conflict on
//    every fragment read.)
//  * Eight waves per block: four compute waves own the 32-row slots (one or
//    two each); four loader waves copy a share of the W slots and of the X
//    rows each into a ring whose depth follows from the bytes of a stage
//    (make_ring), all but one stage requested ahead of the one consumed.
//  * The contraction index inside a chunk follows the pieces: MFMA k-step s,
//    lane half u, element e is k = 8 (2s + u) + e for both operands.
#pragma once

#include "device_common.h"

namespace ooo {

constexpr int kStreamRows = 128;  // W rows per tile (4 compute waves x 32)

// physical piece of logical piece p in LDS row r (and in the packed layout)
__device__ __forceinline__ int piece_swz(int r) { return (r >> 1) & 7; }

// One 32-row W slot (4 KiB at dst).  Packed: src is the slot's 4 KiB run
// plus lane * 8 elements.
__device__ __forceinline__ void dma_w_slot_packed(const uint16_t* src, uint8_t* dst) {
#pragma unroll
  for (int jj = 0; jj < 4; ++jj)
    __builtin_amdgcn_global_load_lds(OOO_GLB(src + jj * 512), OOO_LDS(dst + jj * 1024), 16, 0, kStreamOnce);
}
// Row layout: rows row0 .. row0 + 31 of W[rows][ld] (clamped to the last
// row), columns 64 kc .. 64 kc + 63; lane = (row within an instruction,
// physical piece).
__device__ __forceinline__ void dma_w_slot_rows(const uint16_t* W, long long ld, int row0, int rows, int kc,
                                                uint8_t* dst, int lane) {
#pragma unroll
  for (int jj = 0; jj < 4; ++jj) {
    const int r = 8 * jj + lane / 8;
    const int pc = (lane % 8) ^ piece_swz(r);
    const int row = min(row0 + r, rows - 1);
    __builtin_amdgcn_global_load_lds(OOO_GLB(W + (size_t)row * ld + kc * 64 + pc * 8), OOO_LDS(dst + jj * 1024),
                                     16, 0, kStreamOnce);
  }
}

// LDS byte offsets of compute lane (c, u)'s fragments in a W or X stage:
// piece 2s + u of row c (swizzled), for the k-steps s of a chunk.
__device__ __forceinline__ void frag_offsets(int lane, uint32_t (&off)[4]) {
  const int c = lane & 31, u = lane >> 5;
#pragma unroll
  for (int s4 = 0; s4 < 4; ++s4) off[s4] = c * 128 + (((2 * s4 + u) ^ piece_swz(c)) << 4);
}

// ------------------------------------------------------------- tall tiles
// The same stream with tiles of up to 128 RG rows: RG 32-row slots per
// compute wave, so that one X chunk serves RG times the W bytes.  Four
// compute and four loader waves; loader i copies the W slots i, i + 4, ...
// and a quarter of the X chunk.  A tile holds n <= 4 RG groups (32 rows);
// slot s is empty from n on, costs no DMA and no arithmetic.
constexpr int kTallThreads = 512;

// Workgroup barrier after this wave's LDS reads have returned.
__device__ __forceinline__ void lds_read_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

constexpr int kRingBytes = 160 * 1024;  // the whole LDS: one block per CU

// Bytes a block requests ahead.  Enough for the HBM latency at its share of
// the rate; more makes the first chunks of all blocks land later and gains
// nothing after (2 x 12288 gate/up rows of 4096 columns, one node: 37.9 us
// with 144 KiB ahead, 37.2 with 48; 2 x 4352 rows: 24.0 and 23.1; two
// Qwen3-8B layers at one node 212.8 and 204.8, at 64 nodes 245.1 and 243.1).
constexpr int kRingAhead = 48 * 1024;

// Ring of the chunks of tiles of up to `slots` groups: a stage holds the W
// slots, then the X rows there are (in eights).  Fewer slots or nodes give
// more stages, so a block with little work per chunk still has many bytes in
// flight.  Fragment reads of node rows past the ones copied run into what
// follows (the next stage, or room kept behind the last).  Made on the host,
// as the deal below: each integer division ahead of a block's first request
// is about 0.1 us of the call (bf16 LM heads of 500 to 152064 rows, 140
// shapes: 1.8 %; 64 nodes, H 256, V 1000: 8.7 -> 8.3 us).
struct Ring {
  int xoff, bytes, ns;
};
inline Ring make_ring(int slots, int N, int NB) {
  const int x = (N + 7) / 8 * 1024, xoff = slots * 4096, bytes = xoff + x;
  const int most = (kRingBytes - (NB * 4096 - x)) / bytes, ahead = 1 + (kRingAhead + bytes - 1) / bytes;
  const int ns = ahead > 3 ? ahead : 3;
  return Ring{xoff, bytes, ns < most ? ns : most};
}

// Units (32-row groups, or the pairs of the SwiGLU kernel) dealt out in T
// tiles for each of `grid` blocks, `more` of them of per + 1 units and the
// rest of `per`, at most 4 RG: block b takes the tiles b, b + grid, ...
struct Deal {
  int T, per, more;
  __host__ __device__ __forceinline__ int first(int i) const { return per * i + (i < more ? i : more); }  // of tile i
  int slots() const { return per + (more > 0); }
};
inline Deal make_deal(int units, int grid, int RG) {
  const int T = (units + 4 * RG * grid - 1) / (4 * RG * grid);
  return Deal{T, units / (T * grid), units % (T * grid)};
}

// s_waitcnt vmcnt(n) for a count known at run time only (wave-uniform): a
// jump into a table of waits, because what follows the wait is on every
// chunk's critical path (compare-and-branch code for the same choice made
// the LM head at 128 nodes 3.5% slower: 286.5 against 276.9 us).  Counts past
// 56 wait for 56; waiting for fewer is always right.
__device__ __forceinline__ void wait_vmcnt_at(int n) {
  const int to = __builtin_amdgcn_readfirstlane(12 + 8 * min(max(n, 0), 56));
  // s_getpc gives the address of the s_add; three instructions of 4 bytes,
  // then entries of two
  asm volatile(
      "s_getpc_b64 s[90:91]\n\t"
      "s_add_u32 s90, s90, %0\n\t"
      "s_addc_u32 s91, s91, 0\n\t"
      "s_setpc_b64 s[90:91]\n\t"
      ".set .Lcount%=, 0\n\t"
      ".rept 57\n\t"
      "s_waitcnt vmcnt(.Lcount%=)\n\t"
      "s_branch .Lwaited%=\n\t"
      ".set .Lcount%=, .Lcount%=+1\n\t"
      ".endr\n"
      ".Lwaited%=:"
      :
      : "s"(to)
      : "s90", "s91", "scc", "memory");
}

// Loader i's share of the X chunks: rows 8 (i NB + j) + lane / 8, j < n.
// Rows are copied in eights up to the last one that N needs (rows past N in
// the last eight repeat row N - 1); stage rows past those are never written,
// and whatever they hold only reaches accumulator columns past N.
template <int NB>
struct XShare {
  const uint16_t* p[NB];
  int n;
  __device__ __forceinline__ XShare(const uint16_t* X, int N, long long ld, int i, int lane) {
    n = __builtin_amdgcn_readfirstlane(min(NB, max(0, (N + 7) / 8 - i * NB)));
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      const int r = 8 * (i * NB + j) + lane / 8;
      p[j] = X + (size_t)min(r, N - 1) * ld + ((lane % 8) ^ piece_swz(r)) * 8;
    }
  }
  int col = 0;
  __device__ __forceinline__ void set(int kc) { col = kc * 64; }
  // copies the chunk it points at and moves on to the next
  __device__ __forceinline__ void dma(int i, uint8_t* dst) {
#pragma unroll
    for (int j = 0; j < NB; ++j)
      if (j < n)
        __builtin_amdgcn_global_load_lds(OOO_GLB(p[j] + col), OOO_LDS(dst + (i * NB + j) * 1024), 16, 0, 0);
    col += 64;
  }
};

struct GroupRange {
  int lo, hi;
};

// Slots of a tile of ng groups that belong to loader (or compute wave) i.
template <int RG>
__device__ __forceinline__ int slots_of(int ng, int i) {
  return __builtin_amdgcn_readfirstlane(max(0, min(RG, (ng - i + 3) / 4)));
}

// Loader wave i over `total` chunks from chunk kc0 of tile t0 on; a tile has
// `chunks` chunks and is the groups tile(t).  slots: the W
// sources; slots.set(r, g, kc) points source r at chunk kc of group g,
// slots.dma(r, dst) copies the chunk it points at (4 instructions) and moves
// on to the next.  The wait for a chunk counts the instructions of the
// chunks requested behind it; around a tile boundary where this loader's
// slots change it takes the smaller count (waits for a little more).
// ng_least: the fewest groups of any tile (tiles shorter than the ring,
// where a wait can span several).
template <int NB, int RG, class Tile, class Slots>
__device__ __forceinline__ void tall_load(int t0, int kc0, int total, int chunks, int ng_least, int i, Tile&& tile,
                                          Slots&& slots, XShare<NB>& xs, const Ring& ring, uint8_t* lds) {
  int it = t0, in = 0, ikc = 0, left = total;  // tile and chunk of the next request
  const auto enter = [&](int t, int kc) {
    const int g0 = tile(t).lo;
    in = slots_of<RG>(tile(t).hi - g0, i);
    ikc = kc;
    xs.set(kc);
#pragma unroll
    for (int r = 0; r < RG; ++r)
      if (r < in) slots.set(r, g0 + i + 4 * r, kc);
  };
  uint8_t* dst = lds;
  uint8_t* const end = lds + ring.ns * ring.bytes;
  const auto issue = [&]() {
    xs.dma(i, dst + ring.xoff);
#pragma unroll
    for (int r = 0; r < RG; ++r)
      if (r < in) slots.dma(r, dst + (i + 4 * r) * 4096);
    dst += ring.bytes;
    if (dst == end) dst = lds;
    if (--left > 0 && ++ikc == chunks) enter(++it, 0);
  };
  enter(t0, kc0);
  int ckc = kc0, ct = t0, cn = in;  // chunk being waited for
  for (int q = 0; q < ring.ns - 1 && left > 0; ++q) issue();
  const int least = slots_of<RG>(ng_least, i);
  const bool long_tiles = chunks >= ring.ns;
  for (int q = 0; q < total; ++q) {
    const int ahead = min(ring.ns - 2, total - 1 - q);
    wait_vmcnt_at(ahead * (xs.n + 4 * (long_tiles ? min(cn, in) : least)));
    wg_barrier();
    if (left > 0) issue();
    if (++ckc == chunks && q + 1 < total) {
      ckc = 0;
      ++ct;
      cn = slots_of<RG>(tile(ct).hi - tile(ct).lo, i);
    }
  }
}

// W sources of a loader: 32-row groups of the packed or the row layout.
template <int RG, bool PACKED>
struct GroupSlots {
  const uint16_t* W;
  int chunks, rows, lane;
  long long ld;
  const uint16_t* p[RG];
  int g[RG], kc[RG];
  __device__ __forceinline__ GroupSlots(const uint16_t* w, int c, int nrows, long long l, int ln)
      : W(w), chunks(c), rows(nrows), lane(ln), ld(l) {}
  __device__ __forceinline__ void set(int r, int grp, int k) {
    if (PACKED) {
      p[r] = W + ((size_t)(grp / 4) * chunks + k) * (kStreamRows * 64) + 32 * 64 * (grp % 4);
    } else {
      g[r] = grp;
      kc[r] = k;
    }
  }
  __device__ __forceinline__ void dma(int r, uint8_t* dst) {
    if (PACKED) {
      dma_w_slot_packed(p[r] + lane * 8, dst);
      p[r] += kStreamRows * 64;
    } else {
      dma_w_slot_rows(W, ld, 32 * g[r], rows, kc[r]++, dst, lane);
    }
  }
};

// `chunks` chunks of compute wave w's slots w + 4 r, r < RA: acc[r][nb] +=
// slot times node block nb.  Fragments are read one k-step (16 columns)
// ahead of the MFMAs that use them, over chunk boundaries too: the barrier
// that frees a chunk's stage and publishes the next chunk stands before the
// chunk's last k-step, whose fragments are in registers by then, and the
// next chunk's first fragments are read under that k-step's MFMAs.  The
// stage of the first chunk (of the block's first tile) is waited for by the
// caller; `last` leaves out the barrier after the last chunk.
template <int NB, int RG, int RA>
__device__ __forceinline__ void tall_run(int chunks, bool last, int w, const uint8_t* lds, const Ring& ring,
                                         const uint32_t (&off)[4], int& stage, f32x16 (&acc)[RG][NB]) {
  bf16x8 af[2][RA], bf[2][NB];
  const uint8_t* st = lds + stage * ring.bytes;
  const auto read = [&](int s4, int buf) {
#pragma unroll
    for (int r = 0; r < RA; ++r)
      af[buf][r] = as_bf16x8(*reinterpret_cast<const u32x4*>(st + (w + 4 * r) * 4096 + off[s4]));
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
      bf[buf][nb] = as_bf16x8(*reinterpret_cast<const u32x4*>(st + ring.xoff + nb * 4096 + off[s4]));
  };
  const auto mma = [&](int buf) {
#pragma unroll
    for (int r = 0; r < RA; ++r)
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) acc[r][nb] = mfma32(af[buf][r], bf[buf][nb], acc[r][nb]);
  };
  read(0, 0);
  for (int kc = 0; kc < chunks; ++kc) {
#pragma unroll
    for (int s4 = 0; s4 < 3; ++s4) {
      read(s4 + 1, (s4 + 1) & 1);
      mma(s4 & 1);
      __builtin_amdgcn_sched_barrier(0);
    }
    if (++stage == ring.ns) stage = 0;
    st = lds + stage * ring.bytes;
    const bool more = kc + 1 < chunks;
    if (more || !last) lds_read_barrier();
    if (more) read(0, 0);
    mma(1);
    __builtin_amdgcn_sched_barrier(0);
  }
}

// One tile of ng groups for compute wave w.
template <int NB, int RG>
__device__ __forceinline__ void tall_tile(int chunks, bool last, int ng, int w, const uint8_t* lds,
                                          const Ring& ring, const uint32_t (&off)[4], int& stage,
                                          f32x16 (&acc)[RG][NB]) {
  if (w >= ng) {  // no slot of this tile: barriers only
    for (int kc = 0; kc < chunks; ++kc) {
      if (++stage == ring.ns) stage = 0;
      if (kc + 1 < chunks || !last) lds_read_barrier();
    }
  } else if (RG == 1 || w + 4 >= ng) {
    tall_run<NB, RG, 1>(chunks, last, w, lds, ring, off, stage, acc);
  } else {
    tall_run<NB, RG, RG>(chunks, last, w, lds, ring, off, stage, acc);
  }
}

}  // namespace ooo
