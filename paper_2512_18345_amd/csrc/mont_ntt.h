// Device-side building blocks of the key-switching transforms (keyswitch.hip):
// the two NTT passes in wave-sized pieces, in Montgomery arithmetic.
//
// A limb of N = N1 * 256 words is N1 rows ("blocks") of 256 columns.  The
// column pass runs the first log2(N1) Cooley-Tukey stages down the columns,
// the block pass the last 8 stages inside each row.  Both are cut into pieces
// that one wave (four rows) or half a wave (the column pass, 512 words)
// transforms alone, 16 words per lane, as two register phases with one
// exchange through its own LDS words between them: no barrier in a transform.
//
// Twiddles are single words w 2^32 mod q.  A product is three full-rate
// instructions, as the Shoup form needs, but with half the table: a lane's 15
// twiddles of a phase fit in 15 registers, so no phase reads them from LDS.
//
// Between the two passes a limb lies in the row-group layout: word (row, col)
// at (row >> 4) * 4096 + col * 16 + (row & 15).  The 16 rows of a block-pass
// work-group are one contiguous 16 KB run in it, and a column tile of C
// columns is a run of 64 C bytes (128 bytes at N = 2^16) in every row group, so
// either pass reads and writes whole lines and the column tile can be as
// narrow as two columns.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>

#include "arith.h"
#include "ctx.h"

namespace ckks {

// Orders a wave's LDS writes before its later LDS reads of other lanes' words
// (the LDS serves one wave's accesses in order; this keeps the compiler to it).
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// A prime and qn = -q^-1 mod 2^32.
struct MontQ {
  uint32_t q, q2, qn;
};
__device__ __forceinline__ MontQ mont_q(const ModC& m) { return MontQ{m.q, 2 * m.q, m.qn}; }

// The same through vector loads, for a prime that differs between lanes.
__device__ __forceinline__ MontQ mont_q_load(const ModC* p) {
  const uint32_t* w = reinterpret_cast<const uint32_t*>(p);
  const uint32_t q = ld1(w + offsetof(ModC, q) / 4);
  return MontQ{q, 2 * q, ld1(w + offsetof(ModC, qn) / 4)};
}

// y w 2^-32 mod q in [0, 2q) for any y < 2^32 and w < q: both addends of the
// sum are below 2^32 q, and the sum is a multiple of 2^32.
__device__ __forceinline__ uint32_t mont_mul(uint32_t y, uint32_t w, const MontQ& m) {
  const uint64_t t = (uint64_t)y * w;
  const uint32_t u = (uint32_t)t * m.qn;
  return (uint32_t)((t + (uint64_t)u * m.q) >> 32);
}

// Stages [S0, S1) of a 16-point Cooley-Tukey network on v (stage s pairs
// words 2^(3-s) apart), twiddle of group g of stage s at tw[2^s + g].
// Harvey's lazy form: words in [0, 4q).
template <int S0, int S1>
__device__ __forceinline__ void ct_stages(uint32_t v[16], const uint32_t tw[16], const MontQ& m) {
#pragma unroll
  for (int s = S0; s < S1; ++s) {
    const int d = 8 >> s;
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      if (j & d) continue;
      const uint32_t x = csub(v[j], m.q2);
      const uint32_t t = mont_mul(v[j + d], tw[(1 << s) + j / (2 * d)], m);
      v[j] = x + t;
      v[j + d] = x + m.q2 - t;
    }
  }
}
// The inverse network's stages S1 - 1 down to S0 (Gentleman-Sande, words in [0, 2q)).
template <int S0, int S1>
__device__ __forceinline__ void gs_stages(uint32_t v[16], const uint32_t tw[16], const MontQ& m) {
#pragma unroll
  for (int s = S1 - 1; s >= S0; --s) {
    const int d = 8 >> s;
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      if (j & d) continue;
      const uint32_t x = v[j], y = v[j + d];
      v[j] = csub(x + y, m.q2);
      v[j + d] = mont_mul(x + m.q2 - y, tw[(1 << s) + j / (2 * d)], m);
    }
  }
}

// A lane's 15 twiddles of the low phase: node h of the level with n nodes in
// a bit-reversed table, and its descendants: tw[1] = tab[n + h], tw[2..3] =
// tab[2n + 2h ..], tw[4..7] = tab[4n + 4h ..], tw[8..15] = tab[8n + 8h ..].
__device__ __forceinline__ void load_node_tw(uint32_t tw[16], const uint32_t* tab, int n, int h) {
  tw[0] = 0;
  tw[1] = ld1(tab + n + h);
  const uint2 b = ld2(tab + 2 * (n + h));
  tw[2] = b.x;
  tw[3] = b.y;
  const uint4 c = ld4(tab + 4 * (n + h));
  tw[4] = c.x;
  tw[5] = c.y;
  tw[6] = c.z;
  tw[7] = c.w;
  const uint4 d = ld4(tab + 8 * (n + h)), e = ld4(tab + 8 * (n + h) + 4);
  tw[8] = d.x;
  tw[9] = d.y;
  tw[10] = d.z;
  tw[11] = d.w;
  tw[12] = e.x;
  tw[13] = e.y;
  tw[14] = e.z;
  tw[15] = e.w;
}
// 16 words read at once, the same for every lane.
struct Words16 {
  uint32_t w[16];
};
// The first 16 words of a table.
__device__ __forceinline__ void load_top_tw(uint32_t tw[16], const uint32_t* tab) {
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const uint4 q = ld4(tab + 4 * k);
    tw[4 * k] = q.x;
    tw[4 * k + 1] = q.y;
    tw[4 * k + 2] = q.z;
    tw[4 * k + 3] = q.w;
  }
}

// ----- column pass: 16 LANES words (all N1 rows of C columns) per LANES lanes --
// LANES = 64: a wave holds C columns of one limb.  LANES = 32 (ColHalf): the
// halves of a wave hold the same columns of two limbs, so twiddles and moduli
// are per lane; n is the lane's number in its half.
// Low layout: lane n = h C + c holds rows 16 h + j, j < 16, of column c.
// High layout: lane n = r C + c holds rows 16 kh + (kl << E) + r as word
// k = kh 2^(4-E) + kl, so the row bits above the low four are register bits.
template <int LOGN1, int LANES>
struct ColPart {
  static constexpr int E = LOGN1 - 4;     // row bits above the low nibble
  static constexpr int C = LANES >> E;    // columns of a tile
  static constexpr int XCH = 17 * LANES;  // exchange words (one word of pad per 16 rows)

  __device__ static __forceinline__ int high_at(int k) {
    return 17 * C * (k >> (4 - E)) + C * ((k & ((16 >> E) - 1)) << E);
  }
  __device__ static __forceinline__ void low_to_high(uint32_t v[16], uint32_t* x, int n) {
    if constexpr (E == 0) return;
    uint32_t* p = x + 17 * C * (n / C) + n % C;
#pragma unroll
    for (int j = 0; j < 16; ++j) p[C * j] = v[j];
    wave_sync();
#pragma unroll
    for (int k = 0; k < 16; ++k) v[k] = x[high_at(k) + n];
    wave_sync();
  }
  __device__ static __forceinline__ void high_to_low(uint32_t v[16], uint32_t* x, int n) {
    if constexpr (E == 0) return;
    const uint32_t* p = x + 17 * C * (n / C) + n % C;
#pragma unroll
    for (int k = 0; k < 16; ++k) x[high_at(k) + n] = v[k];
    wave_sync();
#pragma unroll
    for (int j = 0; j < 16; ++j) v[j] = p[C * j];
    wave_sync();
  }
  // A lane's twiddles: its low-phase node and the table's top for the high phase.
  struct Tw {
    uint32_t lo[16], hi[16];
    __device__ __forceinline__ void load(const uint32_t* tab, int n) {
      load_node_tw(lo, tab, 1 << E, n / C);
      if constexpr (E > 0) load_top_tw(hi, tab);
    }
  };
  // Inverse: low layout in, high layout out, words in [0, 2q).
  __device__ static __forceinline__ void inverse(uint32_t v[16], uint32_t* x, const Tw& tw, const MontQ& m, int n) {
    gs_stages<0, 4>(v, tw.lo, m);
    low_to_high(v, x, n);
    gs_stages<0, E>(v, tw.hi, m);
  }
  // Forward: high layout in, low layout out, words in [0, 4q).
  __device__ static __forceinline__ void forward(uint32_t v[16], uint32_t* x, const Tw& tw, const MontQ& m, int n) {
    ct_stages<0, E>(v, tw.hi, m);
    high_to_low(v, x, n);
    ct_stages<0, 4>(v, tw.lo, m);
  }
  // First word of a lane's 16 in the row-group layout, column tile t.
  __device__ static __forceinline__ uint32_t lane_word(int t, int n) {
    return (uint32_t)(n / C) * 4096 + (t * C + n % C) * 16;
  }
  __device__ static __forceinline__ void load(uint32_t v[16], const uint32_t* row, int t, int n) {
    const uint32_t* p = row + lane_word(t, n);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const uint4 q = ld4(p + 4 * k);
      v[4 * k] = q.x;
      v[4 * k + 1] = q.y;
      v[4 * k + 2] = q.z;
      v[4 * k + 3] = q.w;
    }
  }
  // Stores a low-layout piece so that four consecutive lanes write 64
  // consecutive bytes per instruction: a lane writing its own 64 bytes in four
  // instructions would send four times the write requests to L2.  The quads
  // change lanes through the half's exchange words, rotated by n / 4 so that 16
  // lanes meet no bank twice.
  __device__ static __forceinline__ void store(const uint32_t v[16], uint32_t* x, const OutRow& out, uint32_t row,
                                               int t, int n, bool on) {
#pragma unroll
    for (int k = 0; k < 4; ++k)
      *reinterpret_cast<uint4*>(x + 16 * n + 4 * ((k + (n >> 2)) & 3)) =
          make_uint4(v[4 * k], v[4 * k + 1], v[4 * k + 2], v[4 * k + 3]);
    wave_sync();
    uint4 q[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) q[k] = *reinterpret_cast<const uint4*>(x + 4 * (LANES * k + n));
    wave_sync();
    if (!on) return;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int owner = LANES / 4 * k + (n >> 2);
      out.st4(row + lane_word(t, owner) + 4 * (((n & 3) - (owner >> 2)) & 3), q[k]);
    }
  }
};

template <int LOGN1>
using ColHalf = ColPart<LOGN1, 32>;

// ----- block pass: four rows of 256 words per wave ----------------------------
// LDS tile of 16 rows (or four): word pos of line at line kBlkS + pos + pos / 16.
// The stride makes lines four apart fall 16 banks apart: a wave's four lines
// (w, w + 4, w + 8, w + 12) and the four-row columns of the row-group layout
// both reach 64 different banks.
constexpr int kBlkS = 276;
constexpr int kBlkTile = 16 * kBlkS;

__device__ __forceinline__ int blk_at(int line, int pos) { return line * kBlkS + pos + (pos >> 4); }

// Which lines a wave of a tile transforms: LINES = 16 (four waves) or 4 (one).
template <int LINES>
__device__ __forceinline__ int blk_line(int lane, int w) {
  return LINES == 16 ? 4 * (lane >> 4) + w : lane >> 4;
}

// A lane's twiddles: node (of its row: the first four stages) and its factor
// rho_b^(+-n) (n = lane & 15, see ctx.h), and of the last four stages.
struct BlkTw {
  uint32_t node[16], lo, tail[16];
  __device__ __forceinline__ void load(const uint32_t* row_tab, const uint32_t* tab, int lane) {
    const int n = lane & 15;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const uint4 q = ld4(row_tab + 4 * k);
      node[4 * k] = q.x;
      node[4 * k + 1] = q.y;
      node[4 * k + 2] = q.z;
      node[4 * k + 3] = q.w;
    }
    lo = ld1(row_tab + 16 + n);
    load_node_tw(tail, tab, 16, n);
  }
};

// Forward block pass of the lane's line in two halves (a caller with several
// tiles runs the halves over all of them): first the four stages across the
// line's sixteenths with the row's own twiddles and the factor rho_b^n common
// to the lane's words, then the four stages inside each sixteenth.
__device__ __forceinline__ void blk_fwd_a(uint32_t* s, int line, int lane, const BlkTw& tw, const MontQ& m) {
  uint32_t* p = s + line * kBlkS + (lane & 15);
  uint32_t v[16];
#pragma unroll
  for (int j = 0; j < 16; ++j) v[j] = p[17 * j];
  ct_stages<0, 4>(v, tw.node, m);
#pragma unroll
  for (int j = 0; j < 16; ++j) p[17 * j] = mont_mul(v[j], tw.lo, m);
}
__device__ __forceinline__ void blk_fwd_b(uint32_t* s, int line, int lane, const BlkTw& tw, const MontQ& m) {
  uint32_t* p = s + line * kBlkS + 17 * (lane & 15);
  uint32_t v[16];
#pragma unroll
  for (int j = 0; j < 16; ++j) v[j] = p[j];
  ct_stages<0, 4>(v, tw.tail, m);
#pragma unroll
  for (int j = 0; j < 16; ++j) p[j] = v[j];
}
// The inverse halves, in the opposite order.
__device__ __forceinline__ void blk_inv_a(uint32_t* s, int line, int lane, const BlkTw& tw, const MontQ& m) {
  uint32_t* p = s + line * kBlkS + 17 * (lane & 15);
  uint32_t v[16];
#pragma unroll
  for (int j = 0; j < 16; ++j) v[j] = p[j];
  gs_stages<0, 4>(v, tw.tail, m);
#pragma unroll
  for (int j = 0; j < 16; ++j) p[j] = v[j];
}
__device__ __forceinline__ void blk_inv_b(uint32_t* s, int line, int lane, const BlkTw& tw, const MontQ& m) {
  uint32_t* p = s + line * kBlkS + (lane & 15);
  uint32_t v[16];
#pragma unroll
  for (int j = 0; j < 16; ++j) v[j] = mont_mul(p[17 * j], tw.lo, m);
  gs_stages<0, 4>(v, tw.node, m);
#pragma unroll
  for (int j = 0; j < 16; ++j) p[17 * j] = v[j];
}

// Quad k (of four) of a lane in row order: words 4 (n + 16 k) .. + 3 of its line.
__device__ __forceinline__ uint4 blk_quad(const uint32_t* s, int line, int pos) {
  const uint32_t* p = s + blk_at(line, pos);
  return make_uint4(p[0], p[1], p[2], p[3]);
}
__device__ __forceinline__ void blk_quad_store(uint32_t* s, int line, int pos, uint4 v) {
  uint32_t* p = s + blk_at(line, pos);
  p[0] = v.x;
  p[1] = v.y;
  p[2] = v.z;
  p[3] = v.w;
}

// A row-group tile's quads: quad k of thread t covers rows 4a .. 4a + 3 of one
// column.  LINES = 16: the whole group, quads in memory order.  LINES = 4: the
// rows 4a .. 4a + 3 alone (one quad of 16 bytes from every column's 64).
template <int LINES>
struct RowGroup {
  // word of the quad inside the group, its column, and its first line in the LDS tile
  __device__ static __forceinline__ int word(int t, int k, int a) {
    return LINES == 16 ? 4 * (t + 256 * k) : 16 * (t + 64 * k) + 4 * a;
  }
  __device__ static __forceinline__ int col(int t, int k) { return LINES == 16 ? (t + 256 * k) >> 2 : t + 64 * k; }
  __device__ static __forceinline__ int line(int t) { return LINES == 16 ? 4 * (t & 3) : 0; }

  __device__ static __forceinline__ void to_lds(uint32_t* s, int t, int k, uint4 v) {
    uint32_t* p = s + blk_at(line(t), col(t, k));
    p[0] = v.x;
    p[kBlkS] = v.y;
    p[2 * kBlkS] = v.z;
    p[3 * kBlkS] = v.w;
  }
  __device__ static __forceinline__ uint4 from_lds(const uint32_t* s, int t, int k) {
    const uint32_t* p = s + blk_at(line(t), col(t, k));
    return make_uint4(p[0], p[kBlkS], p[2 * kBlkS], p[3 * kBlkS]);
  }
};

}  // namespace ckks
