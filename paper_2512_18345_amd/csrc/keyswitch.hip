// Fused key-switching pipeline over a job table (see keyswitch.h).
//
// Key-switching has three stages (Fig. keysw): ModUp of every digit, the
// inner product with the evaluation key, ModDown of both components, here in
// five kernels:
//
//  K1  INTT block pass of the input (loader forms d: d, c1*c1', or sigma(c1)) -> y
//  KC  (up) INTT column pass of each digit's limbs, N^-1 (D_j/q_i)^-1, ModUp
//      BConv, NTT column pass of the new rows                        -> z
//  K5  (P rows) NTT block pass fused with the inner product over the digits
//      (hoisted jobs gather sigma(M) instead of transforming), then the first
//      INTT pass of ModDown                                          -> acc
//  KC  (down) INTT column pass of the P rows, N^-1 (P/p_m)^-1, ModDown BConv,
//      NTT column pass, both components                              -> w
//  K5  (Q rows) the same inner product (digit rows come straight from the
//      loader), the NTT block pass of w, (acc - w) P^-1 plus the epilogue term
//      (d0 / d1 of HMult, sigma(c0) of HRot)                         -> out
//
// The Q rows' inner product waits for w so that it never leaves registers:
// written and read back by a kernel of its own it cost 2L rows each way.
//
// The NTT's block pass is row-parallel; its column pass works down the columns
// as BConv does, which is why the three column stages are one kernel.
//
// Every launch covers all jobs (grid.z) and all rows of a stage, which is
// what gives small levels enough work-groups (the batching argument of
// Sec. IV-A).  Rescale has its own three kernels (R1, R2, R4).
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "arith.h"
#include "ctx.h"
#include "keyswitch.h"
#include "mont_ntt.h"

namespace ckks {

namespace {

struct KsConst {
  DevTab T;
  int k, alpha, beta_max;
  const uint32_t* modup_T_off;
  const uint2* pinv;
  const uint2* rescale_inv;
  MontTab M;
};

KsConst make_const(const Ctx& c) {
  return KsConst{c.tab(), c.k, c.alpha, c.beta_max(), c.d_modup_T_off, c.d_pinv, c.d_rescale_inv, c.mont};
}

// Scratch layout of one job (rows of N words): acc [2][R] (its P rows alone are
// used), [2][k] that the pipeline leaves alone, w [2][L], then, for jobs that run
// ModUp, y [L], z [beta][R] and de [L] (the eval-domain polynomial being switched,
// kept by K1 for the digit rows of K5); R = L + k.  The whole-limb kernels lay
// [groups][2][R] over the same rows, groups = min(beta, kSrGroups) at most: a
// layout with fewer rows would have to keep 2 groups R of them.
struct KsView {
  uint32_t *y, *z, *de, *acc, *w;
  const uint32_t* p;  // the P rows after their INTT block pass (row-group layout), component c at p + c ps N
  int ps;
  int L, R, beta;
};

__device__ __forceinline__ KsView ks_view(const KsJob& J, const KsConst& K, size_t N) {
  KsView v;
  v.L = J.L;
  v.R = J.L + K.k;
  v.beta = (J.L + K.alpha - 1) / K.alpha;
  if (J.kind == KS_MODUP) {  // ModUp alone: y in the scratch, z is the output M
    v.y = J.ws;
    v.z = J.out;
    v.acc = v.w = v.de = nullptr;
    v.p = nullptr;
    v.ps = 0;
    return v;
  }
  if (J.kind == KS_MODDOWN) {  // ModDown alone: P rows, then w, in the scratch
    v.y = J.ws;
    v.w = J.ws + (size_t)K.k * N;
    v.p = J.ws;
    v.ps = K.k;
    v.z = v.acc = v.de = nullptr;
    return v;
  }
  v.acc = J.ws;
  v.p = v.acc + (size_t)v.L * N;
  v.ps = v.R;
  v.w = v.acc + ((size_t)2 * v.R + 2 * K.k) * N;
  v.y = v.w + (size_t)2 * v.L * N;
  v.z = v.y + (size_t)v.L * N;
  v.de = v.z + (size_t)v.beta * v.R * N;
  return v;
}

__device__ __forceinline__ int ks_pidx(int r, int L, int L_max) { return r < L ? r : L_max + (r - L); }

// Source index of the eval-domain automorphism: out[j] = in[auto_src(j)].
__device__ __forceinline__ uint32_t auto_src(uint32_t j, uint32_t g, int logN) {
  const uint32_t bj = __builtin_bitreverse32(j) >> (32 - logN);
  const uint32_t e = (g * (2u * bj + 1u)) & ((2u << logN) - 1u);
  return __builtin_bitreverse32((e - 1u) >> 1) >> (32 - logN);
}

// sigma on an aligned quad.  auto_src takes an aligned group of 2^m indexes to
// an aligned group (g is odd: the low bits of the index are the high bits of
// brv), and g = 5^r is 1 mod 4, so four words are four words of one source
// quad, rotated in bit-reversed order (x, z, y, w): one 16-byte load and eight
// selects instead of four index chains and four 4-byte loads.
struct AutoQuad {
  uint32_t src;  // first word of the source quad
  bool r1, r2;   // rotate by one, by two
};
__device__ __forceinline__ AutoQuad auto_quad(uint32_t n, uint32_t g, int logN) {
  const uint32_t s = auto_src(n, g, logN);
  return AutoQuad{s & ~3u, (s & 2) != 0, (s & 1) != 0};
}
__device__ __forceinline__ uint4 auto_turn(uint4 v, const AutoQuad& a) {
  const uint4 u = a.r1 ? make_uint4(v.z, v.w, v.y, v.x) : v;
  return a.r2 ? make_uint4(u.y, u.x, u.w, u.z) : u;
}

__device__ __forceinline__ uint32_t mulmod(uint32_t a, uint32_t b, const ModC& m) {
  return reduce64((uint64_t)a * b, m.q, m.mu_hi, m.mu_lo);
}

// The four quads (words n0 + 64 kk .. + 3) of row r of the polynomial a job
// key-switches: d (PLAIN), c1 c1' (HMULT), sigma(c1) (HROT).  Every load is
// issued before any of them is used.
__device__ __forceinline__ void load_d16(const KsJob& J, int r, uint32_t n0, size_t N, int logN,
                                         const ModC& m, uint4 d[4]) {
  if (J.kind == KS_PLAIN || J.kind == KS_MODUP || J.kind == KS_MODDOWN) {
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) d[kk] = ld4(J.a + (size_t)r * N + n0 + 64 * kk);
    return;
  }
  const size_t row1 = (size_t)(J.L + r) * N;
  if (J.kind == KS_HMULT) {
    uint4 x[4], y[4];
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      x[kk] = ld4(J.a + row1 + n0 + 64 * kk);
      y[kk] = ld4(J.b + row1 + n0 + 64 * kk);
    }
#pragma unroll
    for (int kk = 0; kk < 4; ++kk)
      d[kk] = make_uint4(mulmod(x[kk].x, y[kk].x, m), mulmod(x[kk].y, y[kk].y, m),
                         mulmod(x[kk].z, y[kk].z, m), mulmod(x[kk].w, y[kk].w, m));
    return;
  }
  const uint32_t* src = J.a + row1;
  AutoQuad aq[4];
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) {
    const uint32_t n = n0 + 64 * kk;
    aq[kk] = auto_quad(n, J.gal, logN);
    d[kk] = ld4(src + aq[kk].src);
  }
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) d[kk] = auto_turn(d[kk], aq[kk]);
}

// ============================================================================
// Stage 1: ModUp
// ============================================================================

// One work-group per 16-row group of a limb (four waves, four rows each).
// Bound: the loads' and stores' latency of one round of work-groups; the
// transform is in-wave, so the only barrier is the one before the row-group
// store, whose quads cross the waves' rows.
__global__ __launch_bounds__(kWG) void k1_intt_blks(KsConst K, JobArg<KsJob> JA) {
  const KsJob J = JA.get(blockIdx.z);
  const int r = blockIdx.y;
  const bool down = J.kind == KS_MODDOWN;  // the P rows of its input, else every row
  if (J.kind == KS_HOIST || r >= (down ? K.k : J.L)) return;
  __shared__ __align__(16) uint32_t s[kBlkTile];
  const int logN = K.T.logN;
  const size_t N = (size_t)1 << logN;
  const int pi = down ? K.T.L_max + r : r;
  const ModC mc = ldc(K.T.mod + pi);
  const MontQ m = mont_q(mc);
  const uint32_t base = blockIdx.x * kTile;
  const KsView V = ks_view(J, K, N);
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int line = blk_line<16>(lane, w);
  const uint32_t n0 = base + line * 256 + 4 * (lane & 15);
  // the switched polynomial in the evaluation domain, kept for K5's digit
  // rows (a ModUp-only job keeps it as the digit row of its output M)
  const OutRow de(J.kind == KS_MODUP ? V.z + ((size_t)(r / K.alpha) * V.R + r) * N : V.de + (size_t)r * N);
  // all loads first: a store to de could alias the next quad's source
  BlkTw tw;
  uint4 d[4];
  load_d16(J, down ? J.L + r : r, n0, N, logN, mc, d);
  tw.load(K.M.row_itw(K.T, pi, blockIdx.x * 16 + line), K.M.blk_itw(pi), lane);
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) {
    blk_quad_store(s, line, 4 * (lane & 15) + 64 * kk, d[kk]);
    if (J.kind != KS_PLAIN && !down) de.st4(n0 + 64 * kk, d[kk]);  // HMULT, HROT, MODUP
  }
  wave_sync();
  blk_inv_a(s, line, lane, tw, m);
  wave_sync();
  blk_inv_b(s, line, lane, tw, m);
  __syncthreads();
  const OutRow y(V.y + (size_t)r * N + base);
#pragma unroll
  for (int kk = 0; kk < 4; ++kk)
    y.st4(RowGroup<16>::word(threadIdx.x, kk, 0), RowGroup<16>::from_lds(s, threadIdx.x, kk));
}

// Column stages of a base conversion, one work-group per (column tile, group
// of output rows): every input limb's INTT column pass, its scaling, the
// conversion to each output row and that row's NTT column pass.  All three
// work down the columns, so a tile of 512 words per limb needs nothing from
// outside it: between the two transforms nothing goes through memory (three
// kernels wrote and read the scaled inputs and the converted rows before).
//   CONV_UP:   digit blockIdx.y / groups of y -> its ModUp rows z
//   CONV_DOWN: component blockIdx.y / groups: the P rows of acc -> w
// A wave takes two limbs at a time, one per half.  The waves first share out
// the input limbs, whose scaled columns stay in LDS, then draw the output rows
// from a counter, so that an odd number of rows or waves per SIMD does not
// leave one idle.  Each group of output rows repeats the input transforms, so
// a launch uses one group unless its work-groups would not fill the chip
// (conv_groups).
// The conversion of more than four limbs runs on the matrix cores, in whole
// numbers: inputs and table as four signed bytes each, the table's already
// times 2^(8 d) mod q for the input's byte d (modup_bytes), so that one product
// of 16 x 64 by 64 x 16 bytes gives the four byte sums of up to 16 limbs for 64
// words, and the word's sum mod q is these times 1, 2^8, 2^16 and 2^24: eight
// vector instructions a word instead of a multiply-add per limb and four.  At
// four limbs or fewer the multiply-adds are no more than that.
// Bound: in batches vector arithmetic, 570 instructions a wave for a pair of rows
// (half a transform a word is 450 of them) and 650 for a pair of inputs; with the
// 384 and 256 work-groups of a single key-switch at L = 36, one or two a CU, also
// the chain of load, input transforms and rows (46 and 48% of the issue rate).
// N = 2^16, L = 36, 12 + 12 limbs: ModUp 43.5 us in three kernels -> 28.4 with
// multiply-adds -> 26.3, ModDown 32.1 -> 18.0 -> 16.9; HMult and rescale
// together 234.8 -> 226.9 us by the matrix cores, 16 rotations 633 -> 620.  Two
// limbs a wave instead of one (tiles of 1024 words, half the work-groups, so
// twice the groups): 34.8 -> 28.4 and 24.1 -> 19.9.
using i32x4 = int __attribute__((ext_vector_type(4)));
enum ConvMode : int { CONV_UP = 0, CONV_DOWN = 1 };
constexpr int kConvWaves = 8;

template <int LOGN1, int MODE, int NY>
__global__ __launch_bounds__(64 * kConvWaves, 4) void kc_conv(KsConst K, JobArg<KsJob> JA, int groups,
                                                              const uint32_t* bytes) {
  using CH = ColHalf<LOGN1>;
  static_assert(NY % 4 == 0 && NY <= 16, "base conversion in steps of four limbs");
  constexpr bool BYTES = NY > 4;  // the conversion on the matrix cores
  const KsJob J = JA.get(blockIdx.z);
  const size_t N = (size_t)1 << K.T.logN;
  const KsView V = ks_view(J, K, N);
  const int tile = blockIdx.x;
  const int jd = blockIdx.y / groups, g = blockIdx.y % groups;
  int lo = 0, nin, nout;  // first input limb, inputs, output rows
  if (MODE == CONV_UP) {
    if (J.kind == KS_HOIST || jd >= V.beta) return;
    lo = jd * K.alpha;
    nin = min(K.alpha, V.L - lo);
    nout = V.R - nin;
  } else {
    nin = K.k;
    nout = V.L;
  }
  const int per = (nout + groups - 1) / groups;
  const int o0 = g * per, o1 = min(o0 + per, nout);
  if (o0 >= o1) return;
  __shared__ __align__(16) uint32_t y[NY * 512];
  __shared__ __align__(16) uint32_t xch[kConvWaves * 2 * CH::XCH];
  __shared__ __align__(16) uint32_t Ts[BYTES ? 4 : kMaxPrimes * NY];  // the group's rows of the table, zero past nin
  __shared__ int next;
  const int lane = threadIdx.x & 63, n = lane & 31, half = lane >> 5;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  uint32_t* x = xch + (2 * w + half) * CH::XCH;
  auto row_of = [&](int o) { return MODE == CONV_UP && o >= lo ? o + nin : o; };

  const int stride = MODE == CONV_UP ? K.alpha : K.k, pad = (stride + 3) & ~3;
  // the digit's place in its table, in words or (BYTES) rows
  const size_t T0 =
      MODE == CONV_UP ? ldc(K.modup_T_off + (size_t)(V.L + (BYTES ? K.T.L_max + 1 : 0)) * K.beta_max + jd) : 0;
  // The A operands of a pair of output rows: lane l holds row l & 15 (bit 3: which
  // output, bit 2: for which of two blocks, bits 1..0: byte e of the table), limbs
  // 4 (l >> 4) and up.
  auto load_a = [&](int u) {
    const size_t row = T0 + row_of(min(o0 + u + (lane >> 3 & 1), o1 - 1));
    return 4 * (lane >> 4) < pad ? ld4(bytes + (row * 4 + (lane & 3)) * pad + 4 * (lane >> 4))
                                 : make_uint4(0, 0, 0, 0);
  };
  uint4 ta;
  if constexpr (BYTES) {
    ta = load_a(min(2 * w, o1 - o0 - 1));
  } else {
    const uint32_t* T = (MODE == CONV_UP ? K.M.modup_T : K.M.moddown_T) + T0;
    for (int e = threadIdx.x; e < (o1 - o0) * NY; e += 64 * kConvWaves) {
      const int o = e / NY, i = e % NY;
      Ts[e] = i < nin ? ld1(T + (size_t)row_of(o0 + o) * stride + i) : 0;
    }
  }
  if (threadIdx.x == 0) next = 2 * kConvWaves;
  for (int i0 = 2 * w; i0 < nin; i0 += 2 * kConvWaves) {
    const int i = min(i0 + half, nin - 1);  // an odd last limb: both halves, the same words
    const int pi = MODE == CONV_UP ? lo + i : K.T.L_max + i;
    const uint32_t* src = MODE == CONV_UP ? V.y + (size_t)(lo + i) * N
                                          : V.p + ((size_t)jd * V.ps + i) * N;
    uint32_t v[16];
    typename CH::Tw tw;
    CH::load(v, src, tile, n);
    tw.load(K.M.col_itw(K.T, pi), n);
    const MontQ m = mont_q_load(K.T.mod + pi);
    const uint32_t sc = ld1(MODE == CONV_UP ? K.M.modup_scale + (size_t)V.L * K.T.L_max + pi
                                            : K.M.moddown_scale + i);
    CH::inverse(v, x, tw, m, n);
#pragma unroll
    for (int k = 0; k < 16; ++k) v[k] = csub(mont_mul(v[k], sc, m), m.q);
    if constexpr (BYTES) {
      // word k of lane n: column n & 15 of block 2 k + (n >> 4); a block's columns
      // of four limbs lie together, the limb innermost
      uint32_t* yi = y + ((n >> 4) * (NY / 4) + (i >> 2)) * 64 + (n & 15) * 4 + (i & 3);
#pragma unroll
      for (int k = 0; k < 16; ++k) yi[k * 2 * (NY / 4) * 64] = signed_bytes(v[k]);
    } else {
#pragma unroll
      for (int k = 0; k < 4; ++k)
        *reinterpret_cast<uint4*>(y + i * 512 + k * 128 + n * 4) =
            make_uint4(v[4 * k], v[4 * k + 1], v[4 * k + 2], v[4 * k + 3]);
    }
  }
  __syncthreads();

  const OutRow out(MODE == CONV_UP ? V.z + (size_t)jd * V.R * N : V.w + (size_t)jd * V.L * N);
  for (int u = 2 * w; u < o1 - o0;) {
    const int o = min(o0 + u + half, o1 - 1);
    const int r = row_of(o);
    const int pi = MODE == CONV_UP ? ks_pidx(r, V.L, K.T.L_max) : r;
    typename CH::Tw tw;
    tw.load(K.M.col_tw(K.T, pi), n);
    const MontQ m = mont_q_load(K.T.mod + pi);
    int un = 0;
    if (lane == 0) un = atomicAdd(&next, 2);
    uint32_t v[16];
    if constexpr (BYTES) {
      // Two products of 16 x 64 by 64 x 16 bytes a word: the first fills the
      // rows of lanes with bit 4 clear (block 2 k), the second the others
      // (block 2 k + 1), so that a lane ends up with the four byte sums of its own
      // word of its own half's output.
      const bool odd = lane & 4;
      const i32x4 a0 = {odd ? 0 : (int)ta.x, odd ? 0 : (int)ta.y, odd ? 0 : (int)ta.z, odd ? 0 : (int)ta.w};
      const i32x4 a1 = {odd ? (int)ta.x : 0, odd ? (int)ta.y : 0, odd ? (int)ta.z : 0, odd ? (int)ta.w : 0};
      // (opaque to the compiler: a shift of 64 bits and a negation a word otherwise)
      int k16 = 1 << 16;
      uint32_t qi = 0u - m.qn;
      asm("" : "+s"(k16));
      asm("" : "+v"(qi));
      const uint32_t* yb = y + min(lane >> 4, NY / 4 - 1) * 64 + (lane & 15) * 4;
#pragma unroll
      for (int k = 0; k < 16; ++k) {
        const i32x4 b0 = *reinterpret_cast<const i32x4*>(yb + 2 * k * (NY / 4) * 64);
        const i32x4 b1 = *reinterpret_cast<const i32x4*>(yb + (2 * k + 1) * (NY / 4) * 64);
        i32x4 s = {0, 0, 0, 0};
        s = __builtin_amdgcn_mfma_i32_16x16x64_i8(a0, b0, s, 0, 0, 0);
        s = __builtin_amdgcn_mfma_i32_16x16x64_i8(a1, b1, s, 0, 0, 0);
        // |s_e| <= 64 2^14, so the sum's high word is within 2^12 + 2^4 of zero,
        // less than any prime (q > 2 N): the reduced word lies in (0, 4q)
        const int64_t sum = (int64_t)(s[2] + (s[3] << 8)) * k16 + (s[0] + (s[1] << 8));
        v[k] = (uint32_t)(sum >> 32) + m.q2 - __umulhi((uint32_t)sum * qi, m.q);
        if (k % 4 == 3) {  // four words in flight (left alone, the compiler keeps 16 and spills)
          asm volatile("" : "+v"(v[k - 3]), "+v"(v[k - 2]), "+v"(v[k - 1]), "+v"(v[k]));
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    } else {
      const uint32_t* t = Ts + (o - o0) * NY;
      uint64_t a[16];
#pragma unroll
      for (int k = 0; k < 16; ++k) a[k] = 0;
      const uint4 t4 = *reinterpret_cast<const uint4*>(t);
      const uint32_t ts[4] = {t4.x, t4.y, t4.z, t4.w};
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const uint4 c = *reinterpret_cast<const uint4*>(y + i * 512 + k * 128 + n * 4);
          a[4 * k] += (uint64_t)c.x * ts[i];
          a[4 * k + 1] += (uint64_t)c.y * ts[i];
          a[4 * k + 2] += (uint64_t)c.z * ts[i];
          a[4 * k + 3] += (uint64_t)c.w * ts[i];
        }
      // Montgomery reduction of the sum (the table carries 2^32): with T < q and
      // inputs below 2^30 its high word is below q, so the result is in (0, 4q).
#pragma unroll
      for (int k = 0; k < 16; ++k)
        v[k] = (uint32_t)(a[k] >> 32) + m.q - __umulhi((uint32_t)a[k] * (0u - m.qn), m.q);
    }
    const bool pair = half == 0 || u + 1 < o1 - o0;
    u = __builtin_amdgcn_readfirstlane(un);
    if constexpr (BYTES) ta = load_a(min(u, o1 - o0 - 1));
    CH::forward(v, x, tw, m, n);
    CH::store(v, x, out, (uint32_t)r << K.T.logN, tile, n, pair);
  }
}

// ModUp-only jobs: the block pass of the new rows of M (left after the column
// pass, in the row-group layout), canonical output in row order in place (a
// work-group's rows are the same 16 KiB in both layouts), so that M is wholly in
// the evaluation domain for the hoisted rotations' gathers.
__global__ __launch_bounds__(kWG) void km_ntt_blks(KsConst K, JobArg<KsJob> JA) {
  const KsJob J = JA.get(blockIdx.z);
  if (J.kind != KS_MODUP) return;
  const size_t N = (size_t)1 << K.T.logN;
  const KsView V = ks_view(J, K, N);
  const int gr = blockIdx.y;
  const int j = gr / V.R, r = gr % V.R;
  if (j >= V.beta) return;
  const int lo = j * K.alpha, hi = min(lo + K.alpha, V.L);
  if (r >= lo && r < hi) return;
  __shared__ __align__(16) uint32_t s[kBlkTile];
  const int pi = ks_pidx(r, V.L, K.T.L_max);
  const MontQ m = mont_q(ldc(K.T.mod + pi));
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int line = blk_line<16>(lane, w);
  uint32_t* row = V.z + (size_t)gr * N + blockIdx.x * kTile;
  BlkTw tw;
  const OutRow out(row);
  uint4 raw[4];
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) raw[kk] = ld4(row + RowGroup<16>::word(threadIdx.x, kk, 0));
  tw.load(K.M.row_tw(K.T, pi, blockIdx.x * 16 + line), K.M.blk_tw(pi), lane);
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) RowGroup<16>::to_lds(s, threadIdx.x, kk, raw[kk]);
  __syncthreads();
  blk_fwd_a(s, line, lane, tw, m);
  wave_sync();
  blk_fwd_b(s, line, lane, tw, m);
  wave_sync();
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) {
    const int pos = 4 * (lane & 15) + 64 * kk;
    out.st4(line * 256 + pos, canon4(blk_quad(s, line, pos), m.q, m.q2));
  }
}

// ============================================================================
// Stage 2: NTT block pass + inner product (+ first INTT pass of ModDown on P rows)
// ============================================================================

// P rows of the inner product: the INTT block pass that ModDown starts with,
// on both components (res0, res1: the lane's four quads of its line) under the
// inverse twiddles tw, requested before the inner product, in LDS
// tiles s and s + kBlkTile that other waves may still be reading; stored in the
// row-group layout for the column kernel.
__device__ __forceinline__ void p_rows_intt(uint32_t* s, const KsConst& K, int pi, const MontQ& m,
                                            const BlkTw& tw, const uint4 res0[4], const uint4 res1[4],
                                            uint32_t* acc0, uint32_t* acc1) {
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int line = blk_line<16>(lane, w);
  __syncthreads();
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) {
    const int pos = 4 * (lane & 15) + 64 * kk;
    blk_quad_store(s, line, pos, res0[kk]);
    blk_quad_store(s + kBlkTile, line, pos, res1[kk]);
  }
  wave_sync();
  blk_inv_a(s, line, lane, tw, m);
  blk_inv_a(s + kBlkTile, line, lane, tw, m);
  wave_sync();
  blk_inv_b(s, line, lane, tw, m);
  blk_inv_b(s + kBlkTile, line, lane, tw, m);
  const OutRow o0(acc0), o1(acc1);
  __syncthreads();
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) {
    const int at = RowGroup<16>::word(threadIdx.x, kk, 0);
    o0.st4(at, RowGroup<16>::from_lds(s, threadIdx.x, kk));
    o1.st4(at, RowGroup<16>::from_lds(s + kBlkTile, threadIdx.x, kk));
  }
}

// Has the quad's words computed here: no instruction, an order for the scheduler.
__device__ __forceinline__ void pin4(uint4& v) {
  asm volatile("" : "+v"(v.x), "+v"(v.y), "+v"(v.z), "+v"(v.w));
  __builtin_amdgcn_sched_barrier(0);
}

// Reduction of four 64-bit sums.
__device__ __forceinline__ uint4 reduce4(const uint64_t a[4], const ModC& m) {
  return make_uint4(reduce64(a[0], m.q, m.mu_hi, m.mu_lo), reduce64(a[1], m.q, m.mu_hi, m.mu_lo),
                    reduce64(a[2], m.q, m.mu_hi, m.mu_lo), reduce64(a[3], m.q, m.mu_hi, m.mu_lo));
}
__device__ __forceinline__ void mac4(uint64_t a[4], uint4 v, uint4 e) {
  a[0] += (uint64_t)v.x * e.x;
  a[1] += (uint64_t)v.y * e.y;
  a[2] += (uint64_t)v.z * e.z;
  a[3] += (uint64_t)v.w * e.w;
}

// The w row of component c and Q row r (column pass done, row-group layout), loaded ahead.
__device__ __forceinline__ void load_w(const KsView& V, int c, int r, uint32_t base, size_t N, uint4 w[8]) {
#pragma unroll
  for (int kk = 0; kk < 4; ++kk)
    w[4 * c + kk] = ld4(V.w + ((size_t)c * V.L + r) * N + base + RowGroup<16>::word(threadIdx.x, kk, 0));
}

// What a job adds to a quad of row i of the two components of
//   out[c] = (acc[c] - w[c]) P^-1 + e[c]:
// e = (c0 c0', c0 c1' + c1 c0') for HMULT, (sigma(c0), 0) for rotations, else
// 0.  Loaded ahead without a branch (the kind selects addresses; a load in a
// branch whose value merges after it makes the compiler wait for it there).
struct TermQuad {
  uint4 a, b, c, d;  // HMULT: c0, c0', c1, c1'; rotations: a holds the source quad of sigma(c0)
  AutoQuad aq;
};
template <bool HOIST = false>
__device__ __forceinline__ TermQuad term_load(const KsJob& J, int L, int i, uint32_t n, size_t N, int logN) {
  const bool hm = J.kind == KS_HMULT, rot = HOIST || J.kind == KS_HROT || J.kind == KS_HOIST;
  const size_t row = (size_t)i * N, LN = (size_t)L * N;
  TermQuad t;
  t.aq = rot ? auto_quad(n, J.gal, logN) : AutoQuad{n, false, false};
  t.a = ld4(J.a + row + t.aq.src);
  if (HOIST) return t;
  t.b = ld4((hm ? J.b : J.a) + row + t.aq.src);
  t.c = ld4(J.a + row + (hm ? LN : 0) + t.aq.src);
  t.d = ld4((hm ? J.b + LN : J.a) + row + t.aq.src);
  return t;
}
// Component c of the result for a quad.  w comes in [0, 4q); x = acc + 2q - w < 3q
// < 2^32 after a correction.  HMULT reduces x P^-1 and its products in one sum,
// at most 5 q^2 < 2^63.
template <bool HOIST = false>
__device__ __forceinline__ uint4 combine_comp(const KsConst& K, const KsJob& J, int c, int i, const ModC& mc,
                                              const TermQuad& t, uint4 a, uint4 w) {
  const MontQ m = mont_q(mc);
  w = csub4(w, m.q2);
  const uint4 x = make_uint4(a.x + m.q2 - w.x, a.y + m.q2 - w.y, a.z + m.q2 - w.z, a.w + m.q2 - w.w);
  if (!HOIST && J.kind == KS_HMULT) {
    const uint32_t pv = ldc(K.pinv + i).x;
    uint64_t s[4] = {(uint64_t)x.x * pv, (uint64_t)x.y * pv, (uint64_t)x.z * pv, (uint64_t)x.w * pv};
    if (c == 0) {
      mac4(s, t.a, t.b);
    } else {
      mac4(s, t.a, t.d);
      mac4(s, t.c, t.b);
    }
    return reduce4(s, mc);
  }
  const uint32_t pv = ldc(K.M.pinv + i);
  const uint4 o = make_uint4(csub(mont_mul(x.x, pv, m), m.q), csub(mont_mul(x.y, pv, m), m.q),
                             csub(mont_mul(x.z, pv, m), m.q), csub(mont_mul(x.w, pv, m), m.q));
  if (c || (!HOIST && J.kind == KS_PLAIN)) return o;
  const uint4 e = auto_turn(t.a, t.aq);
  return make_uint4(csub(o.x + e.x, m.q), csub(o.y + e.y, m.q), csub(o.z + e.z, m.q), csub(o.w + e.w, m.q));
}
template <bool HOIST = false>
__device__ __forceinline__ void combine_quad(const KsConst& K, const KsJob& J, int L, int i, uint32_t n, size_t N,
                                             const ModC& mc, const TermQuad& t, uint4 a0, uint4 a1, uint4 w0,
                                             uint4 w1) {
  const OutRow out0(J.out + (size_t)i * N), out1(J.out + ((size_t)L + i) * N);
  const uint4 o0 = combine_comp<HOIST>(K, J, 0, i, mc, t, a0, w0);
  const uint4 o1 = combine_comp<HOIST>(K, J, 1, i, mc, t, a1, w1);
  out0.st4(n, o0);
  out1.st4(n, o1);
}

// Q rows: ModDown's combine on the inner product where it stands, in the
// lane's registers (res0, res1): the block pass of both w rows in tiles s and
// s + kBlkTile, which other waves may still be reading, under the twiddles the
// digits used (same prime, same rows), then the job's term and the output.
template <bool HOIST>
__device__ __forceinline__ void q_rows_combine(uint32_t* s, const KsConst& K, const KsJob& J, const KsView& V,
                                               int r, const ModC& mc, const BlkTw& tw, const uint4 wraw[8],
                                               const uint4 res0[4], const uint4 res1[4]) {
  const MontQ m = mont_q(mc);
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int line = blk_line<16>(lane, w);
  const size_t N = (size_t)1 << K.T.logN;
  __syncthreads();
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) {
    RowGroup<16>::to_lds(s, threadIdx.x, kk, wraw[kk]);
    RowGroup<16>::to_lds(s + kBlkTile, threadIdx.x, kk, wraw[4 + kk]);
  }
  const uint32_t n0 = blockIdx.x * kTile + line * 256 + 4 * (lane & 15);
  // the job's terms: two quads now, to land during the transforms, two after
  // them (all four would cost a resident work-group in registers)
  TermQuad term[4];
#pragma unroll
  for (int kk = 0; kk < 2; ++kk) term[kk] = term_load<HOIST>(J, V.L, r, n0 + 64 * kk, N, K.T.logN);
  __syncthreads();
  blk_fwd_a(s, line, lane, tw, m);
  blk_fwd_a(s + kBlkTile, line, lane, tw, m);
  wave_sync();
  blk_fwd_b(s, line, lane, tw, m);
  blk_fwd_b(s + kBlkTile, line, lane, tw, m);
  wave_sync();
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) {
    if (kk < 2) term[kk + 2] = term_load<HOIST>(J, V.L, r, n0 + 64 * (kk + 2), N, K.T.logN);
    const int pos = 4 * (lane & 15) + 64 * kk;
    combine_quad<HOIST>(K, J, V.L, r, n0 + 64 * kk, N, mc, term[kk], res0[kk], res1[kk], blk_quad(s, line, pos),
                 blk_quad(s + kBlkTile, line, pos));
  }
}

// Any digit count: the digits in turn through one tile, accumulators in
// registers.  HOIST selects the variant for hoisted-rotation jobs (gather of
// sigma(M), no transform; each rotation brings its own key, streamed with the
// non-temporal hint); the other variant serves every other job kind.
// Bound: the chain of digits, which the P rows and the Q rows each walk.  Asking
// for a digit's words only when its turn came made that two latencies a digit:
// HMult of 24 one-limb digits at N = 2^14 174 us, 148 with them requested ahead
// (N = 2^13 166 -> 142; ten two-limb digits at N = 2^14 93 -> 83; eight jobs of 24
// digits at N = 2^14 409 -> 367).
template <bool HOIST, bool Q>
__global__ __launch_bounds__(kWG) void k5_ntt_blks_ip(KsConst K, JobArg<KsJob> JA) {
  const KsJob J = JA.get(blockIdx.z);
  const int logN = K.T.logN;
  const size_t N = (size_t)1 << logN;
  const KsView V = ks_view(J, K, N);
  const int r = Q ? blockIdx.y : V.L + blockIdx.y;
  if ((Q && r >= V.L) || (J.kind == KS_HOIST) != HOIST) return;
  __shared__ __align__(16) uint32_t s[2 * kBlkTile];
  const int pi = ks_pidx(r, V.L, K.T.L_max);
  const ModC mc = ldc(K.T.mod + pi);
  const MontQ m = mont_q(mc);
  const uint32_t base = blockIdx.x * kTile;
  const size_t KR = (size_t)K.T.L_max + K.k;  // key rows
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int line = blk_line<16>(lane, w);
  const uint32_t n0 = base + line * 256 + 4 * (lane & 15);  // the lane's quads: n0 + 64 kk
  BlkTw tw;
  if (!HOIST) tw.load(K.M.row_tw(K.T, pi, blockIdx.x * 16 + line), K.M.blk_tw(pi), lane);
  uint64_t a0[4][4], a1[4][4];
#pragma unroll
  for (int kk = 0; kk < 4; ++kk)
#pragma unroll
    for (int i = 0; i < 4; ++i) a0[kk][i] = a1[kk][i] = 0;

  // hoisted rotation: sigma_g applied to the shared ModUp rows (a gather).  A
  // digit's words are requested a digit ahead, its key words with them: nothing
  // else would cover their latency (20 digits at N = 2^12, eight rotations: P
  // rows 57 -> 25 us, Q rows 52 -> 34).
  AutoQuad aq[4];
  uint4 nv[4], ne0[4], ne1[4];
  auto hoist_load = [&](int j) {
    const uint32_t* Mrow = J.b + ((size_t)j * V.R + r) * N;
    const uint32_t* k0 = J.key + ((size_t)j * 2 * KR + pi) * N + n0;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      nv[kk] = ld4(Mrow + aq[kk].src);
      ne0[kk] = ld4nt(k0 + 64 * kk);
      ne1[kk] = ld4nt(k0 + KR * N + 64 * kk);
    }
  };
  if (HOIST) {
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) aq[kk] = auto_quad(n0 + 64 * kk, J.gal, logN);
    hoist_load(0);
  }
  // Any other job: a digit's words -- the digit row itself in row order (kept by K1
  // unless it is the input) or its ModUp row in the row-group layout -- are
  // requested a digit ahead, its key words before its transform.
  auto owns = [&](int j) { return r >= j * K.alpha && r < min((j + 1) * K.alpha, V.L); };
  auto digit_load = [&](int j) {
    const bool own = owns(j);
    const uint32_t* src = own ? (J.kind == KS_PLAIN ? J.a : V.de) + (size_t)r * N
                              : V.z + ((size_t)j * V.R + r) * N + base;
    const uint32_t at = own ? n0 : (uint32_t)RowGroup<16>::word(threadIdx.x, 0, 0);
    const uint32_t step = own ? 64 : 1024;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) nv[kk] = ld4(src + at + step * kk);
  };
  if (!HOIST) digit_load(0);
  uint32_t* tile = s;  // two in turn: one barrier a transform
  for (int j = 0; j < V.beta; ++j) {
    uint4 v[4], e0[4], e1[4];
    if (HOIST) {
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) {
        v[kk] = nv[kk];
        e0[kk] = ne0[kk];
        e1[kk] = ne1[kk];
      }
      hoist_load(min(j + 1, V.beta - 1));
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) v[kk] = auto_turn(v[kk], aq[kk]);
    } else {
      const uint32_t* k0 = J.key + ((size_t)j * 2 * KR + pi) * N + n0;
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) {
        e0[kk] = ld4(k0 + 64 * kk);
        e1[kk] = ld4(k0 + KR * N + 64 * kk);
      }
      const bool own = owns(j);
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) {
        v[kk] = nv[kk];
        if (!own) RowGroup<16>::to_lds(tile, threadIdx.x, kk, v[kk]);
      }
      digit_load(min(j + 1, V.beta - 1));
      if (!own) {
        __syncthreads();
        blk_fwd_a(tile, line, lane, tw, m);
        wave_sync();
        blk_fwd_b(tile, line, lane, tw, m);
        wave_sync();
#pragma unroll
        for (int kk = 0; kk < 4; ++kk)
          v[kk] = canon4(blk_quad(tile, line, 4 * (lane & 15) + 64 * kk), m.q, m.q2);
        tile = tile == s ? s + kBlkTile : s;
      }
    }
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      mac4(a0[kk], v[kk], e0[kk]);
      mac4(a1[kk], v[kk], e1[kk]);
    }
    // Each product of canonical words is below q^2 < 2^60, so 16 of them fit
    // a 64-bit sum; chains of more digits (digit size 1 allows up to 63) fold
    // the sums back below q after every eighth digit.
    if ((j & 7) == 7) {
#pragma unroll
      for (int kk = 0; kk < 4; ++kk)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          a0[kk][i] = reduce64(a0[kk][i], mc.q, mc.mu_hi, mc.mu_lo);
          a1[kk][i] = reduce64(a1[kk][i], mc.q, mc.mu_hi, mc.mu_lo);
        }
    }
  }

  // one reduction per output (the overflow-free accumulation of Sec. III-C2)
  uint4 r0[4], r1[4], wraw[8];
  BlkTw itw;
  if constexpr (Q) {
    load_w(V, 0, r, base, N, wraw);
    load_w(V, 1, r, base, N, wraw);
  } else
    itw.load(K.M.row_itw(K.T, pi, blockIdx.x * 16 + line), K.M.blk_itw(pi), lane);
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) {
    r0[kk] = reduce4(a0[kk], mc);
    r1[kk] = reduce4(a1[kk], mc);
  }
  if constexpr (Q) {
    if (HOIST) tw.load(K.M.row_tw(K.T, pi, blockIdx.x * 16 + line), K.M.blk_tw(pi), lane);
    q_rows_combine<HOIST>(s, K, J, V, r, mc, tw, wraw, r0, r1);
  } else {
    uint32_t* acc0 = V.acc + (size_t)r * N;
    uint32_t* acc1 = V.acc + ((size_t)V.R + r) * N;
    p_rows_intt(s, K, pi, m, itw, r0, r1, acc0 + base, acc1 + base);
  }
}

// Variant of K5 for contexts with at most NB digits: every digit's tile is
// staged and transformed in its own LDS slot first (all loads in flight at
// once), then the inner product runs one 16-byte quad at a time, so the
// 64-bit accumulators never hold more than four elements per component.
// Bound: Q rows, memory (HMult at N = 2^16, L = 36: 160 MB in 33 us, 4.8 TB/s;
// with a combine kernel of its own, all rows 29.6 + 19.1 us); P rows, the
// chain of one round of work-groups (17 us for a quarter of the rows).  16
// hoisted rotations: 316 + 183 us in two kernels -> 86 + 311.  Up to three digits
// at most 168 registers, so that three work-groups share a CU: at 191 the Q rows
// took 37.9.  (Four digits: two, by their 69 KiB of LDS as by the Q rows' 189.)
// NT: the key words are read with the non-temporal hint (a launch of one
// job reads its key once; batches whose jobs share a key keep it cached).
template <int NB, bool NT, bool Q>
__global__ __launch_bounds__(kWG) void k5s_ntt_blks_ip(KsConst K, JobArg<KsJob> JA) {
  const KsJob J = JA.get(blockIdx.z);
  const int logN = K.T.logN;
  const size_t N = (size_t)1 << logN;
  const KsView V = ks_view(J, K, N);
  const int r = Q ? blockIdx.y : V.L + blockIdx.y;
  if ((Q && r >= V.L) || J.kind == KS_HOIST) return;
  __shared__ __align__(16) uint32_t s[NB * kBlkTile];
  const int pi = ks_pidx(r, V.L, K.T.L_max);
  const ModC mc = ldc(K.T.mod + pi);
  const MontQ m = mont_q(mc);
  const uint32_t base = blockIdx.x * kTile;
  const size_t KR = (size_t)K.T.L_max + K.k;  // key rows
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int line = blk_line<16>(lane, w);
  const uint32_t n0 = base + line * 256 + 4 * (lane & 15);  // the lane's quads: n0 + 64 kk

  // Every load of the staging is issued before any of them is used, in
  // straight-line code (a branch between them would make the compiler wait
  // for the earlier ones): each digit's tile -- the digit row itself, in row
  // order, for the digit that holds r, else its ModUp row in the row-group
  // layout; digits past beta re-read the last digit's rows, unused -- the
  // twiddles, and the key words of the first KPF quads, whose latency overlaps
  // the transforms.
  uint4 raw[NB][4];
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    const int jj = min(j, V.beta - 1);
    const int lo = jj * K.alpha, hi = min(lo + K.alpha, V.L);
    const bool own = r >= lo && r < hi;
    const uint32_t* src = own ? (J.kind == KS_PLAIN ? J.a : V.de) + (size_t)r * N
                              : V.z + ((size_t)jj * V.R + r) * N + base;
    const uint32_t at = own ? n0 : (uint32_t)RowGroup<16>::word(threadIdx.x, 0, 0);
    const uint32_t step = own ? 64 : 1024;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) raw[j][kk] = ld4(src + at + step * kk);
  }
  BlkTw tw;
  tw.load(K.M.row_tw(K.T, pi, blockIdx.x * 16 + line), K.M.blk_tw(pi), lane);
  constexpr int KPF = NB <= 2 ? 4 : 2;
  uint4 kpre0[4][NB], kpre1[4][NB];
  auto key_quad = [&](int kk) {
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      const uint32_t* k0 = J.key + ((size_t)min(j, V.beta - 1) * 2 * KR + pi) * N + n0 + 64 * kk;
      kpre0[kk][j] = NT ? ld4nt(k0) : ld4(k0);
      kpre1[kk][j] = NT ? ld4nt(k0 + KR * N) : ld4(k0 + KR * N);
    }
  };
#pragma unroll
  for (int kk = 0; kk < KPF; ++kk) key_quad(kk);
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    if (j >= V.beta) break;
    const int lo = j * K.alpha, hi = min(lo + K.alpha, V.L);
    uint32_t* slot = s + j * kBlkTile;
    if (r >= lo && r < hi) {
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) blk_quad_store(slot, line, 4 * (lane & 15) + 64 * kk, raw[j][kk]);
    } else {
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) RowGroup<16>::to_lds(slot, threadIdx.x, kk, raw[j][kk]);
    }
  }
  __syncthreads();
  // The block pass of all digit tiles, half by half; from here every wave
  // works on its own four lines alone.
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    const int lo = j * K.alpha, hi = min(lo + K.alpha, V.L);
    if (j < V.beta && !(r >= lo && r < hi)) blk_fwd_a(s + j * kBlkTile, line, lane, tw, m);
  }
  wave_sync();
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    const int lo = j * K.alpha, hi = min(lo + K.alpha, V.L);
    if (j < V.beta && !(r >= lo && r < hi)) blk_fwd_b(s + j * kBlkTile, line, lane, tw, m);
  }
  wave_sync();

  // inner product, one quad at a time (one reduction per output, Sec. III-C2).
  // No branch on the digit count: tiles past beta (never staged) are masked
  // to zero, so the prefetched key words are consumed in straight-line code.
  // The transformed words enter uncorrected: each lies in [0, 4q) and each
  // key word below q < 2^30, so a product is below 2^62 and the sum of at
  // most four (NB <= 4) stays below 2^64 for the single exact reduction.
  static_assert(NB >= 2 && NB <= 4, "64-bit sum of lazy products; two slots for the P rows");
  uint4 res0[4], res1[4], wraw[8];
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) {
    uint64_t a0[4] = {0, 0, 0, 0}, a1[4] = {0, 0, 0, 0};
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      const uint32_t msk = j < V.beta ? ~0u : 0u;
      uint4 v = blk_quad(s + j * kBlkTile, line, 4 * (lane & 15) + 64 * kk);
      v.x &= msk;
      v.y &= msk;
      v.z &= msk;
      v.w &= msk;
      mac4(a0, v, kpre0[kk][j]);
      mac4(a1, v, kpre1[kk][j]);
    }
    res0[kk] = reduce4(a0, mc);
    res1[kk] = reduce4(a1, mc);
    // the next loads in the registers this quad leaves, no earlier (raising
    // them all costs a resident work-group)
    pin4(res0[kk]);
    pin4(res1[kk]);
    if (kk + KPF < 4) key_quad(kk + KPF);
    if (Q && kk == 3) {
      load_w(V, 0, r, base, N, wraw);
      load_w(V, 1, r, base, N, wraw);
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  if constexpr (Q) {
    q_rows_combine<false>(s, K, J, V, r, mc, tw, wraw, res0, res1);
  } else {
    uint32_t* acc0 = V.acc + (size_t)r * N;
    uint32_t* acc1 = V.acc + ((size_t)V.R + r) * N;
    BlkTw itw;
    itw.load(K.M.row_itw(K.T, pi, blockIdx.x * 16 + line), K.M.blk_itw(pi), lane);
    p_rows_intt(s, K, pi, m, itw, res0, res1, acc0 + base, acc1 + base);
  }
}

// K5 for hoisted rotations of at most NB digits.  sigma_g maps each aligned
// 4096-word tile of an evaluation-domain row onto one aligned source tile (g
// is odd, so only the low 12 bits of the bit-reversed index are permuted), so
// every digit's source tile of M is loaded whole and contiguously into its
// own LDS slot and the permutation is a read from LDS, a rotated quad at a
// time (auto_quad).  The key words of the
// first KPF quads are requested with the tiles; the inner product and the
// P-row INTT block pass follow as in k5s, on canonical words (M is fully
// transformed).
template <int NB, bool Q>
__global__ __launch_bounds__(kWG) void k5h_gather_ip(KsConst K, JobArg<KsJob> JA) {
  static_assert(NB >= 2 && NB <= 4, "slots for two to four digits");
  const KsJob J = JA.get(blockIdx.z);
  const int logN = K.T.logN;
  const size_t N = (size_t)1 << logN;
  const KsView V = ks_view(J, K, N);
  const int r = Q ? blockIdx.y : V.L + blockIdx.y;
  if ((Q && r >= V.L) || J.kind != KS_HOIST) return;
  constexpr int WORDS = NB * kTile > 2 * kBlkTile ? NB * kTile : 2 * kBlkTile;
  __shared__ __align__(16) uint32_t s[WORDS];
  const int pi = ks_pidx(r, V.L, K.T.L_max);
  const ModC mc = ldc(K.T.mod + pi);
  const uint32_t base = blockIdx.x * kTile;
  const size_t KR = (size_t)K.T.L_max + K.k;  // key rows
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int line = blk_line<16>(lane, w);
  const uint32_t n0 = base + line * 256 + 4 * (lane & 15);  // the lane's quads: n0 + 64 kk
  const uint32_t src0 = auto_src(base, J.gal, logN) & ~(uint32_t)(kTile - 1);
  // every digit's source tile (digits past beta re-read the last one, unused)
  uint4 raw[NB][4];
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    const int jj = min(j, V.beta - 1);
    const uint32_t* Mrow = J.b + ((size_t)jj * V.R + r) * N + src0;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) raw[j][kk] = ld4(Mrow + 4 * (threadIdx.x + kk * kWG));
  }
  constexpr int KPF = NB <= 2 ? 4 : 2;
  uint4 kpre0[4][NB], kpre1[4][NB];
  auto key_quad = [&](int kk) {
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      const uint32_t* k0 = J.key + ((size_t)min(j, V.beta - 1) * 2 * KR + pi) * N + n0 + 64 * kk;
      kpre0[kk][j] = ld4nt(k0);
      kpre1[kk][j] = ld4nt(k0 + KR * N);
    }
  };
#pragma unroll
  for (int kk = 0; kk < KPF; ++kk) key_quad(kk);
#pragma unroll
  for (int j = 0; j < NB; ++j)
#pragma unroll
    for (int kk = 0; kk < 4; ++kk)
      *reinterpret_cast<uint4*>(s + j * kTile + 4 * (threadIdx.x + kk * kWG)) = raw[j][kk];
  __syncthreads();

  // inner product of sigma(M) quad by quad (canonical words: products below
  // 2^60, at most four summed, one reduction per output)
  uint4 res0[4], res1[4], wraw[8];
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) {
    const uint32_t n = n0 + 64 * kk;
    const AutoQuad aq = auto_quad(n, J.gal, logN);
    uint64_t a0[4] = {0, 0, 0, 0}, a1[4] = {0, 0, 0, 0};
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      const uint32_t msk = j < V.beta ? ~0u : 0u;
      uint4 v = auto_turn(*reinterpret_cast<const uint4*>(s + j * kTile + (aq.src & (kTile - 1))), aq);
      v.x &= msk;
      v.y &= msk;
      v.z &= msk;
      v.w &= msk;
      mac4(a0, v, kpre0[kk][j]);
      mac4(a1, v, kpre1[kk][j]);
    }
    res0[kk] = reduce4(a0, mc);
    res1[kk] = reduce4(a1, mc);
    // the next loads in the registers this quad leaves, no earlier (raising
    // them all costs a resident work-group)
    pin4(res0[kk]);
    pin4(res1[kk]);
    if (kk + KPF < 4) key_quad(kk + KPF);
    if (Q && kk == 3) {
      load_w(V, 0, r, base, N, wraw);
      load_w(V, 1, r, base, N, wraw);
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  if constexpr (Q) {
    BlkTw tw;
    tw.load(K.M.row_tw(K.T, pi, blockIdx.x * 16 + line), K.M.blk_tw(pi), lane);
    q_rows_combine<true>(s, K, J, V, r, mc, tw, wraw, res0, res1);
  } else {
    uint32_t* acc0 = V.acc + (size_t)r * N;
    uint32_t* acc1 = V.acc + ((size_t)V.R + r) * N;
    BlkTw itw;
    itw.load(K.M.row_itw(K.T, pi, blockIdx.x * 16 + line), K.M.blk_itw(pi), lane);
    p_rows_intt(s, K, pi, mont_q(mc), itw, res0, res1, acc0 + base, acc1 + base);
  }
}

// K5 for small grids (few tiles x rows): one work-group per four rows of a
// limb, one wave per digit, so the digits' transforms run side by side; then
// the threads share out the inner product's 256 quads, and for P rows waves 0
// and 1 take a component each.  Four times the work-groups of k5s and a third
// of its chain per wave.  Every barrier below is reached by all threads.
// The line of 128 work-groups (the schedule's small_grid): below it, with half of
// the CUs idle under k5s, HMult at N = 2^14, L = 13 (48 and 52 work-groups) takes
// 35.3 us against 43.9 by k5s and HRot at N = 2^15, L = 25 (96) 55.9 against 59.7;
// above it the side-by-side waves load a CU more than they shorten its chain: at
// 192 HRot at N = 2^16, L = 7 takes 41.7 us against 40.3, a step at L = 36 229.5
// against 227.4 (at 200, three digits, 55.4 against 56.0).
template <int NB, bool Q>
__global__ __launch_bounds__(64 * NB) void k5p_ntt_blks_ip(KsConst K, JobArg<KsJob> JA) {
  static_assert(NB >= 2 && NB <= 4, "one wave per digit");
  constexpr int T = 64 * NB;
  constexpr int QPT = (256 + T - 1) / T;  // quads per thread of the inner product, at most
  constexpr int TILE4 = 4 * kBlkS;
  const KsJob J = JA.get(blockIdx.z);
  const int logN = K.T.logN;
  const size_t N = (size_t)1 << logN;
  const KsView V = ks_view(J, K, N);
  const int r = Q ? blockIdx.y : V.L + blockIdx.y;
  if ((Q && r >= V.L) || J.kind == KS_HOIST) return;
  __shared__ __align__(16) uint32_t s[NB * TILE4];
  const int pi = ks_pidx(r, V.L, K.T.L_max);
  const ModC mc = ldc(K.T.mod + pi);
  const MontQ m = mont_q(mc);
  // which four rows of which group of 16: the work-groups of one group, which
  // share its lines, a multiple of N / 4096 apart, so on one XCD from N = 2^15 on
  const int tiles = gridDim.x >> 2;
  const int a4 = blockIdx.x / tiles, row4 = 4 * (blockIdx.x % tiles) + a4;
  const uint32_t group = (blockIdx.x % tiles) * kTile;  // the group's first word
  const uint32_t base = row4 * 1024;                    // the four rows' first word in row order
  const size_t KR = (size_t)K.T.L_max + K.k;            // key rows
  const int j = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int line = blk_line<4>(lane, 0);
  const int lo = j * K.alpha, hi = min(lo + K.alpha, V.L);
  const bool own = r >= lo && r < hi;
  uint32_t* slot = s + j * TILE4;
  BlkTw tw;
  tw.load(K.M.row_tw(K.T, pi, row4 * 4 + line), K.M.blk_tw(pi), lane);
  if (j < V.beta) {
    uint4 v[4];
    if (own) {
      const uint32_t* drow = (J.kind == KS_PLAIN ? J.a : V.de) + (size_t)r * N + base + line * 256 + 4 * (lane & 15);
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) v[kk] = ld4(drow + 64 * kk);
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) blk_quad_store(slot, line, 4 * (lane & 15) + 64 * kk, v[kk]);
    } else {
      const uint32_t* zrow = V.z + ((size_t)j * V.R + r) * N + group;
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) v[kk] = ld4(zrow + RowGroup<4>::word(lane, kk, a4));
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) RowGroup<4>::to_lds(slot, lane, kk, v[kk]);
    }
  }
  // key words of this thread's quads, requested before the transforms (past
  // the last quad or digit they repeat earlier ones, unused)
  uint4 k0v[QPT][NB], k1v[QPT][NB];
#pragma unroll
  for (int i = 0; i < QPT; ++i) {
    const uint32_t e = 4 * min((int)threadIdx.x + i * T, 255);
#pragma unroll
    for (int jj = 0; jj < NB; ++jj) {
      const uint32_t* k0 = J.key + ((size_t)min(jj, V.beta - 1) * 2 * KR + pi) * N + base + e;
      k0v[i][jj] = ld4(k0);
      k1v[i][jj] = ld4(k0 + KR * N);
    }
  }
  uint4 wv[4];
  BlkTw itw;
  if (!Q) itw.load(K.M.row_itw(K.T, pi, row4 * 4 + line), K.M.blk_itw(pi), lane);
  if (Q && j < 2) {
    const uint32_t* wrow = V.w + ((size_t)j * V.L + r) * N + group;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) wv[kk] = ld4(wrow + RowGroup<4>::word(lane, kk, a4));
  }
  if (j < V.beta && !own) {
    wave_sync();
    blk_fwd_a(slot, line, lane, tw, m);
    wave_sync();
    blk_fwd_b(slot, line, lane, tw, m);
  }
  __syncthreads();

  // inner product (one reduction per output); the lazy words in [0, 4q) enter
  // uncorrected, as in k5s (NB <= 4 products of at most 2^62 each)
  uint4 res0[QPT], res1[QPT];
#pragma unroll
  for (int i = 0; i < QPT; ++i) {
    const int e = 4 * min((int)threadIdx.x + i * T, 255);
    uint64_t a0[4] = {0, 0, 0, 0}, a1[4] = {0, 0, 0, 0};
#pragma unroll
    for (int jj = 0; jj < NB; ++jj) {
      const uint32_t msk = jj < V.beta ? ~0u : 0u;
      uint4 v = blk_quad(s + jj * TILE4, e >> 8, e & 255);
      v.x &= msk;
      v.y &= msk;
      v.z &= msk;
      v.w &= msk;
      mac4(a0, v, k0v[i][jj]);
      mac4(a1, v, k1v[i][jj]);
    }
    res0[i] = reduce4(a0, mc);
    res1[i] = reduce4(a1, mc);
  }
  if constexpr (Q) {
    // ModDown's combine: waves 0 and 1 transform a w row each, then every
    // thread finishes its quads
    __syncthreads();  // the inner product has read the tiles
    if (j < 2) {
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) RowGroup<4>::to_lds(slot, lane, kk, wv[kk]);
      wave_sync();
      blk_fwd_a(slot, line, lane, tw, m);
      wave_sync();
      blk_fwd_b(slot, line, lane, tw, m);
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < QPT; ++i) {
      const int e = 4 * (threadIdx.x + i * T);
      if (e < 1024)
        combine_quad(K, J, V.L, r, base + e, N, mc, term_load(J, V.L, r, base + e, N, logN), res0[i], res1[i], blk_quad(s, e >> 8, e & 255),
                     blk_quad(s + TILE4, e >> 8, e & 255));
    }
    return;
  }
  uint32_t* acc0 = V.acc + (size_t)r * N;
  uint32_t* acc1 = V.acc + ((size_t)V.R + r) * N;
  __syncthreads();  // the inner product has read the tiles
#pragma unroll
  for (int i = 0; i < QPT; ++i) {
    const int e = 4 * (threadIdx.x + i * T);
    if (e < 1024) {
      blk_quad_store(s, e >> 8, e & 255, res0[i]);
      blk_quad_store(s + TILE4, e >> 8, e & 255, res1[i]);
    }
  }
  __syncthreads();
  if (j < 2) {
    blk_inv_a(slot, line, lane, itw, m);
    wave_sync();
    blk_inv_b(slot, line, lane, itw, m);
    wave_sync();
    const OutRow dst((j ? acc1 : acc0) + group);
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) dst.st4(RowGroup<4>::word(lane, kk, a4), RowGroup<4>::from_lds(slot, lane, kk));
  }
}

// ============================================================================
// Rescale: t = INTT_{q_{L-1}}(a_{L-1}); out_i = (a_i - NTT_{q_i}(t mod q_i)) q_{L-1}^-1
// Scratch, in the row-group layout: t [2][N] after the block pass, u [2][L-1][N]
// after the column pass.
// ============================================================================
__global__ __launch_bounds__(kWG) void r1_intt_blks(KsConst K, JobArg<RsJob> JA) {
  const RsJob J = JA.get(blockIdx.z);
  const int c = blockIdx.y, pi = J.L - 1;
  __shared__ __align__(16) uint32_t s[kBlkTile];
  const size_t N = (size_t)1 << K.T.logN;
  const MontQ m = mont_q(ldc(K.T.mod + pi));
  const uint32_t base = blockIdx.x * kTile;
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int line = blk_line<16>(lane, w);
  const uint32_t* in = J.a + ((size_t)c * J.L + pi) * N + base + line * 256 + 4 * (lane & 15);
  uint4 x[4];
  BlkTw tw;
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) x[kk] = ld4(in + 64 * kk);
  tw.load(K.M.row_itw(K.T, pi, blockIdx.x * 16 + line), K.M.blk_itw(pi), lane);
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) blk_quad_store(s, line, 4 * (lane & 15) + 64 * kk, x[kk]);
  wave_sync();
  blk_inv_a(s, line, lane, tw, m);
  wave_sync();
  blk_inv_b(s, line, lane, tw, m);
  __syncthreads();
  const OutRow t(J.ws + (size_t)c * N + base);
#pragma unroll
  for (int kk = 0; kk < 4; ++kk)
    t.st4(RowGroup<16>::word(threadIdx.x, kk, 0), RowGroup<16>::from_lds(s, threadIdx.x, kk));
}

// The column stages of a component, as in kc_conv with one input limb: its INTT
// column pass and N^-1 by the first wave, then t mod q_i and its NTT column pass
// for the group's rows, a pair of rows a wave at a time.  One launch for what
// were two (4.9 + 14.2 -> 12.8 us at N = 2^16, L = 36).
template <int LOGN1>
__global__ __launch_bounds__(64 * kConvWaves, 4) void r2_cols(KsConst K, JobArg<RsJob> JA, int groups) {
  using CH = ColHalf<LOGN1>;
  const RsJob J = JA.get(blockIdx.z);
  const size_t N = (size_t)1 << K.T.logN;
  const int tile = blockIdx.x, L1 = J.L - 1;
  const int c = blockIdx.y / groups, g = blockIdx.y % groups;
  const int per = (L1 + groups - 1) / groups;
  const int o0 = g * per, o1 = min(o0 + per, L1);
  if (o0 >= o1) return;
  __shared__ __align__(16) uint32_t y[512];
  __shared__ __align__(16) uint32_t xch[kConvWaves * 2 * CH::XCH];
  __shared__ int next;
  const int lane = threadIdx.x & 63, n = lane & 31, half = lane >> 5;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  uint32_t* x = xch + (2 * w + half) * CH::XCH;
  if (w == 0) {  // both halves, the same words
    if (lane == 0) next = 2 * kConvWaves;
    uint32_t v[16];
    typename CH::Tw tw;
    CH::load(v, J.ws + (size_t)c * N, tile, n);
    tw.load(K.M.col_itw(K.T, L1), n);
    const ModC mc = ldc(K.T.mod + L1);
    const MontQ m = mont_q(mc);
    CH::inverse(v, x, tw, m, n);
#pragma unroll
    for (int k = 0; k < 16; ++k) v[k] = csub(mul_shoup(v[k], mc.ninv, mc.ninv_s, m.q), m.q);
#pragma unroll
    for (int k = 0; k < 4; ++k)
      *reinterpret_cast<uint4*>(y + k * 128 + n * 4) = make_uint4(v[4 * k], v[4 * k + 1], v[4 * k + 2], v[4 * k + 3]);
  }
  __syncthreads();
  const OutRow out(J.ws + (size_t)(2 + c * L1) * N);
  for (int u = 2 * w; u < o1 - o0;) {
    const int i = min(o0 + u + half, o1 - 1);
    typename CH::Tw tw;
    tw.load(K.M.col_tw(K.T, i), n);
    const MontQ m = mont_q_load(K.T.mod + i);
    const uint32_t mu32 = ld1(reinterpret_cast<const uint32_t*>(K.T.mod + i) + offsetof(ModC, mu32) / 4);
    int un = 0;
    if (lane == 0) un = atomicAdd(&next, 2);
    uint32_t v[16];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const uint4 q = *reinterpret_cast<const uint4*>(y + k * 128 + n * 4);
      v[4 * k] = reduce32(q.x, m.q, mu32);
      v[4 * k + 1] = reduce32(q.y, m.q, mu32);
      v[4 * k + 2] = reduce32(q.z, m.q, mu32);
      v[4 * k + 3] = reduce32(q.w, m.q, mu32);
    }
    CH::forward(v, x, tw, m, n);
    CH::store(v, x, out, (uint32_t)i << K.T.logN, tile, n, half == 0 || u + 1 < o1 - o0);
    u = __builtin_amdgcn_readfirstlane(un);
  }
}

// One row group of out = (a - NTT(u)) f mod q of prime i: the block pass of u
// (column pass done, row-group layout), a and out in row order; f with its
// Shoup companion.
__device__ __forceinline__ void sub_scale_rows(const KsConst& K, int i, const uint32_t* u, const uint32_t* a,
                                               uint32_t* dst, uint2 f) {
  __shared__ __align__(16) uint32_t s[kBlkTile];
  const MontQ m = mont_q(ldc(K.T.mod + i));
  const uint32_t base = blockIdx.x * kTile;
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int line = blk_line<16>(lane, w);
  const uint32_t n0 = base + line * 256 + 4 * (lane & 15);
  uint4 raw[4], xs[4];
  BlkTw tw;
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) raw[kk] = ld4(u + base + RowGroup<16>::word(threadIdx.x, kk, 0));
  tw.load(K.M.row_tw(K.T, i, blockIdx.x * 16 + line), K.M.blk_tw(i), lane);
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) xs[kk] = ld4(a + n0 + 64 * kk);
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) RowGroup<16>::to_lds(s, threadIdx.x, kk, raw[kk]);
  __syncthreads();
  blk_fwd_a(s, line, lane, tw, m);
  wave_sync();
  blk_fwd_b(s, line, lane, tw, m);
  wave_sync();
  const OutRow out(dst);
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) {
    const uint4 v = csub4(blk_quad(s, line, 4 * (lane & 15) + 64 * kk), m.q2);  // [0, 2q): x + 2q - v < 3q
    const uint4 x = xs[kk];
    out.st4(n0 + 64 * kk, make_uint4(csub(mul_shoup(x.x + m.q2 - v.x, f.x, f.y, m.q), m.q),
                                     csub(mul_shoup(x.y + m.q2 - v.y, f.x, f.y, m.q), m.q),
                                     csub(mul_shoup(x.z + m.q2 - v.z, f.x, f.y, m.q), m.q),
                                     csub(mul_shoup(x.w + m.q2 - v.w, f.x, f.y, m.q), m.q)));
  }
}

// Bound: memory (a, u in, out: 55 MB at N = 2^16, L = 36, both components).
__global__ __launch_bounds__(kWG) void r4_ntt_blks_combine(KsConst K, JobArg<RsJob> JA) {
  const RsJob J = JA.get(blockIdx.z);
  const int L1 = J.L - 1;
  const int gr = blockIdx.y;
  if (gr >= 2 * L1) return;
  const int c = gr / L1, i = gr % L1;
  const size_t N = (size_t)1 << K.T.logN;
  sub_scale_rows(K, i, J.ws + (size_t)(2 + gr) * N, J.a + ((size_t)c * J.L + i) * N,
                 J.out + ((size_t)c * L1 + i) * N, ldc(K.rescale_inv + (size_t)J.L * K.T.L_max + i));
}

// ModDown alone (one component): the combine.
__global__ __launch_bounds__(kWG) void kd_ntt_blks_combine(KsConst K, JobArg<KsJob> JA) {
  const KsJob J = JA.get(blockIdx.z);
  const int i = blockIdx.y;
  if (i >= J.L) return;
  const size_t N = (size_t)1 << K.T.logN;
  const KsView V = ks_view(J, K, N);
  sub_scale_rows(K, i, V.w + (size_t)i * N, J.a + (size_t)i * N, J.out + (size_t)i * N, ldc(K.pinv + i));
}

// ============================================================================
// Small rings (N = 2^kSrLog = 4096): a whole limb fits one work-group, so the
// column pass needs no kernel of its own -- and neither does the five-kernel
// pipeline.  A key-switch runs as two kernels of 256 threads, 16 words each:
//   S1  per (ModUp row t, group of digits): each non-digit limb of a digit
//       transformed back whole, scaled, converted to row t (BConv), the sum
//       transformed forward, times the key rows; the products summed over the
//       group's digits -> one partial accumulator per group;
//   S2  per (Q row i, component): the partials summed; ModDown -- the P rows'
//       INTT, their conversion to q_i, its NTT -- combined with the
//       accumulator, plus the job's epilogue term.
// The arithmetic is that of the five kernels (exact: the same residues).
// Scratch of a job: the partials [groups][2][L + k][N] (at most kSrGroups = 4).
// Bound: the chain of one work-group, four transforms of about 800 instructions
// a wave with one barrier each.  With 1024 threads in radix-4 phases, six
// barriers a transform and both 32 KiB twiddle tables staged in LDS, HMult at
// L = 4 took 12.0 + 14.6 us, and 16 of them 23.4 + 14.8; now 9.3 + 9.9 and
// 15.4 + 10.9.
// ============================================================================
constexpr int kSrN = 1 << kSrLog;
static_assert(kSrN == kTile, "one 16-row group per limb");

__device__ __forceinline__ int sr_per(int beta) { return (beta + kSrGroups - 1) / kSrGroups; }  // digits per group
__device__ __forceinline__ int sr_groups(int beta) { return (beta + sr_per(beta) - 1) / sr_per(beta); }

// The column pass of a whole limb is one 16-point network: thread c (of 256)
// holds rows 0..15 of column c.
struct SrTw {
  BlkTw blk;
  Words16 col;  // uniform
  __device__ __forceinline__ void load(const KsConst& K, int pi, int line, int lane) {
    blk.load(K.M.row_tw(K.T, pi, line), K.M.blk_tw(pi), lane);
    col = ldc(reinterpret_cast<const Words16*>(K.M.col_tw(K.T, pi)));
  }
  __device__ __forceinline__ void load_inv(const KsConst& K, int pi, int line, int lane) {
    blk.load(K.M.row_itw(K.T, pi, line), K.M.blk_itw(pi), lane);
    col = ldc(reinterpret_cast<const Words16*>(K.M.col_itw(K.T, pi)));
  }
};

// The lane's four quads of its line (evaluations) -> the thread's column of
// coefficients, times sc 2^-32, canonical.  s: a tile no wave still reads.
__device__ __forceinline__ void sr_inverse(uint32_t v[16], uint32_t* s, const uint4 x[4], const SrTw& tw,
                                           uint32_t sc, const MontQ& m, int line, int lane) {
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) blk_quad_store(s, line, 4 * (lane & 15) + 64 * kk, x[kk]);
  wave_sync();
  blk_inv_a(s, line, lane, tw.blk, m);
  wave_sync();
  blk_inv_b(s, line, lane, tw.blk, m);
  __syncthreads();
#pragma unroll
  for (int j = 0; j < 16; ++j) v[j] = s[blk_at(j, threadIdx.x)];
  gs_stages<0, 4>(v, tw.col.w, m);
#pragma unroll
  for (int j = 0; j < 16; ++j) v[j] = csub(mont_mul(v[j], sc, m), m.q);
}
// The thread's column of coefficients (below 4q) -> the lane's quads of
// evaluations, in [0, 4q).
__device__ __forceinline__ void sr_forward(uint4 x[4], uint32_t* s, uint32_t v[16], const SrTw& tw, const MontQ& m,
                                           int line, int lane) {
  ct_stages<0, 4>(v, tw.col.w, m);
#pragma unroll
  for (int j = 0; j < 16; ++j) s[blk_at(j, threadIdx.x)] = v[j];
  __syncthreads();
  blk_fwd_a(s, line, lane, tw.blk, m);
  wave_sync();
  blk_fwd_b(s, line, lane, tw.blk, m);
  wave_sync();
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) x[kk] = blk_quad(s, line, 4 * (lane & 15) + 64 * kk);
}

// The lane's quads (words n0 + 64 kk) of row r of the polynomial a job
// key-switches (evaluation domain): d, c1 c1' or sigma(c1).  Loaded raw (both
// factors of the product) so that a prefetch does not wait for its data; the
// product is taken by finish where the quads are used.  Branch-free (the kind
// selects addresses, every load is issued): a load in a branch whose value
// merges after it makes the compiler wait for it there.
struct SrRaw {
  uint4 x[4], y[4];
  AutoQuad aq[4];
  __device__ __forceinline__ void load(const KsJob& J, int r, uint32_t n0) {
    const size_t N = kSrN;
    const bool rot = J.kind == KS_HROT;
    const uint32_t* src = J.a + (size_t)(J.kind == KS_PLAIN ? r : J.L + r) * N;
    const uint32_t* src2 = J.kind == KS_HMULT ? J.b + (size_t)(J.L + r) * N : src;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      const uint32_t n = n0 + 64 * kk;
      aq[kk] = rot ? auto_quad(n, J.gal, kSrLog) : AutoQuad{n, false, false};
      x[kk] = ld4(src + aq[kk].src);
      y[kk] = ld4(src2 + n);
    }
  }
  __device__ __forceinline__ void finish(const KsJob& J, const ModC& m, uint4 d[4]) const {
#pragma unroll
    for (int kk = 0; kk < 4; ++kk)
      d[kk] = J.kind != KS_HMULT
                  ? auto_turn(x[kk], aq[kk])
                  : make_uint4(mulmod(x[kk].x, y[kk].x, m), mulmod(x[kk].y, y[kk].y, m),
                               mulmod(x[kk].z, y[kk].z, m), mulmod(x[kk].w, y[kk].w, m));
  }
};

// S1.  The work-group's items are its digits' limbs in order (a digit row of
// the switched polynomial is one item without transforms).  Two tiles in turn,
// so that one barrier a transform is enough.
// ONE: a single digit per group, so no accumulators.  With several the sums and the
// transform's words fill a wave's registers (one work-group a CU): 41 us for HMult
// at L = 24 with one-limb digits, a group's six one after another.
template <bool ONE>
__global__ __launch_bounds__(kWG, ONE ? 2 : 1) void s1_modup_ip(KsConst K, JobArg<KsJob> JA) {
  const KsJob J = JA.get(blockIdx.z);
  const int L = J.L, R = L + K.k, beta = (L + K.alpha - 1) / K.alpha;
  const int t = blockIdx.x, per = ONE ? 1 : sr_per(beta), gi = blockIdx.y;
  const int j0 = gi * per, j1 = min(beta, j0 + per);
  if (t >= R || j0 >= beta || J.kind > KS_HROT) return;
  __shared__ __align__(16) uint32_t s[2 * kBlkTile];
  const size_t N = kSrN;
  const size_t KR = (size_t)K.T.L_max + K.k;
  const int pt = ks_pidx(t, L, K.T.L_max);
  const ModC mct = ldc(K.T.mod + pt);
  const MontQ mt = mont_q(mct);
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int line = blk_line<16>(lane, w);
  const uint32_t n0 = line * 256 + 4 * (lane & 15);
  uint32_t* cur = s;
  uint32_t* other = s + kBlkTile;
  uint64_t a0[4][4], a1[4][4];
#pragma unroll
  for (int kk = 0; kk < 4; ++kk)
#pragma unroll
    for (int e = 0; e < 4; ++e) a0[kk][e] = a1[kk][e] = 0;
  for (int j = j0; j < j1; ++j) {
    const int lo = j * K.alpha, hi = min(lo + K.alpha, L);
    const bool own = t >= lo && t < hi;
    const uint32_t* k0 = J.key + ((size_t)j * 2 * KR + pt) * N + n0;
    const uint32_t* k1 = k0 + KR * N;
    SrRaw x;
    SrTw it, ft;
    uint4 d[4], e0[4], e1[4];
    const int first = own ? t : lo;
    x.load(J, first, n0);
    it.load_inv(K, first, line, lane);
    ft.load(K, pt, line, lane);
    auto keys = [&]() {
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) {
        e0[kk] = ld4(k0 + 64 * kk);
        e1[kk] = ld4(k1 + 64 * kk);
      }
    };
    if (own) {
      keys();
      x.finish(J, mct, d);
    } else {
      uint64_t z[16];
#pragma unroll
      for (int c = 0; c < 16; ++c) z[c] = 0;
      const uint32_t* T = K.M.modup_T + ldc(K.modup_T_off + (size_t)L * K.beta_max + j) + (size_t)t * K.alpha;
      for (int i = lo; i < hi; ++i) {
        const ModC mci = ldc(K.T.mod + i);
        const uint32_t sc = ldc(K.M.modup_scale + (size_t)L * K.T.L_max + i), Ti = ldc(T + (i - lo));
        if (i > lo) {
          x.load(J, i, n0);
          it.load_inv(K, i, line, lane);
        }
        x.finish(J, mci, d);
        uint32_t v[16];
        sr_inverse(v, cur, d, it, sc, mont_q(mci), line, lane);
        uint32_t* sw = cur;
        cur = other;
        other = sw;
#pragma unroll
        for (int c = 0; c < 16; ++c) z[c] += (uint64_t)v[c] * Ti;
      }
      // the key words land during the forward transform (no earlier: the
      // registers would not hold them beside the inverse one's)
      __builtin_amdgcn_sched_barrier(0);
      keys();
      uint32_t v[16];
#pragma unroll
      for (int c = 0; c < 16; ++c)  // REDC (the table carries 2^32): below 4q, see kc_conv
        v[c] = csub((uint32_t)(z[c] >> 32), mt.q2) + mt.q - __umulhi((uint32_t)z[c] * (0u - mt.qn), mt.q);
      sr_forward(d, cur, v, ft, mt, line, lane);
      uint32_t* sw = cur;
      cur = other;
      other = sw;
      if (!ONE) {
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) d[kk] = canon4(d[kk], mt.q, mt.q2);
      }
    }
    // (ONE: a word below 4q times a key word, reduced at once)
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      mac4(a0[kk], d[kk], e0[kk]);
      mac4(a1[kk], d[kk], e1[kk]);
    }
    if (ONE) break;
    if (((j - j0) & 7) == 7) {  // canonical products < 2^60: fold every eighth digit
#pragma unroll
      for (int kk = 0; kk < 4; ++kk)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          a0[kk][e] = reduce64(a0[kk][e], mct.q, mct.mu_hi, mct.mu_lo);
          a1[kk][e] = reduce64(a1[kk][e], mct.q, mct.mu_hi, mct.mu_lo);
        }
    }
  }
  const OutRow p0(J.ws + ((size_t)(2 * gi) * R + t) * N), p1(J.ws + ((size_t)(2 * gi + 1) * R + t) * N);
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) {
    p0.st4(n0 + 64 * kk, reduce4(a0[kk], mct));
    p1.st4(n0 + 64 * kk, reduce4(a1[kk], mct));
  }
}

// The groups' partials (at most four) at the lane's quads of row r, summed: a
// sum of four canonical words stays below 4q < 2^32.  Group indices past
// `groups` repeat the last group and are dropped.
struct SrPartials {
  uint4 v[4][4];
  __device__ __forceinline__ void load(const uint32_t* ws, int groups, int c, int R, int r, uint32_t n0) {
    const size_t N = kSrN;
#pragma unroll
    for (int g = 0; g < 4; ++g)
#pragma unroll
      for (int kk = 0; kk < 4; ++kk)
        v[g][kk] = ld4(ws + ((size_t)(2 * min(g, groups - 1) + c) * R + r) * N + n0 + 64 * kk);
  }
  __device__ __forceinline__ uint4 sum(int kk, int groups, uint32_t q) const {
    uint4 a = v[0][kk];
#pragma unroll
    for (int g = 1; g < 4; ++g) {
      const uint32_t on = g < groups ? 0xffffffffu : 0u;
      a.x += v[g][kk].x & on;
      a.y += v[g][kk].y & on;
      a.z += v[g][kk].z & on;
      a.w += v[g][kk].w & on;
    }
    return canon4(a, q, 2 * q);
  }
};

__global__ __launch_bounds__(kWG, 2) void s2_moddown(KsConst K, JobArg<KsJob> JA) {
  const KsJob J = JA.get(blockIdx.z);
  const int L = J.L, R = L + K.k, beta = (L + K.alpha - 1) / K.alpha;
  const int i = blockIdx.x, c = blockIdx.y, groups = sr_groups(beta);
  if (i >= L || J.kind > KS_HROT) return;
  __shared__ __align__(16) uint32_t s[2 * kBlkTile];
  const size_t N = kSrN;
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int line = blk_line<16>(lane, w);
  const uint32_t n0 = line * 256 + 4 * (lane & 15);
  const ModC mc = ldc(K.T.mod + i);
  const MontQ m = mont_q(mc);
  uint32_t* cur = s;
  uint32_t* other = s + kBlkTile;
  // ModDown: w = sum_m x_m [P / p_m]_{q_i}, x_m = INTT(acc P row m) N^-1 (P / p_m)^-1
  uint64_t z[16];
#pragma unroll
  for (int e = 0; e < 16; ++e) z[e] = 0;
  uint4 x[4];
  for (int mm = 0; mm < K.k; ++mm) {
    const int pm = K.T.L_max + mm;
    const ModC mcp = ldc(K.T.mod + pm);
    const uint32_t sc = ldc(K.M.moddown_scale + mm), T = ldc(K.M.moddown_T + (size_t)i * K.k + mm);
    SrPartials px;
    px.load(J.ws, groups, c, R, L + mm, n0);
    SrTw it;
    it.load_inv(K, pm, line, lane);
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) x[kk] = px.sum(kk, groups, mcp.q);
    uint32_t v[16];
    sr_inverse(v, cur, x, it, sc, mont_q(mcp), line, lane);
    uint32_t* sw = cur;
    cur = other;
    other = sw;
#pragma unroll
    for (int e = 0; e < 16; ++e) z[e] += (uint64_t)v[e] * T;
  }
  // what the end needs, to land during the forward transform (no earlier: the
  // registers would not hold it beside the inverse ones)
  __builtin_amdgcn_sched_barrier(0);
  SrTw ft;
  SrPartials pa;
  TermQuad term[4];
  ft.load(K, i, line, lane);
  pa.load(J.ws, groups, c, R, i, n0);
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) term[kk] = term_load(J, L, i, n0 + 64 * kk, N, kSrLog);
  uint32_t v[16];
#pragma unroll
  for (int e = 0; e < 16; ++e)
    v[e] = csub((uint32_t)(z[e] >> 32), m.q2) + m.q - __umulhi((uint32_t)z[e] * (0u - m.qn), m.q);
  sr_forward(x, cur, v, ft, m, line, lane);
  const OutRow out(J.out + ((size_t)c * L + i) * N);
#pragma unroll
  for (int kk = 0; kk < 4; ++kk)
    out.st4(n0 + 64 * kk, combine_comp(K, J, c, i, mc, term[kk], pa.sum(kk, groups, m.q), x[kk]));
}
}  // namespace

size_t ks_ws_words(const Ctx& c, int L) {
  const size_t R = (size_t)L + c.k;
  return ks_hoist_ws_words(c, L) + (2 * (size_t)L + (size_t)c.beta(L) * R) * c.N;
}

size_t ks_hoist_ws_words(const Ctx& c, int L) {
  return (2 * ((size_t)L + c.k) + 2 * (size_t)c.k + 2 * (size_t)L) * c.N;
}

size_t rs_ws_words(const Ctx& c, int L) { return (2 + 2 * (size_t)L) * c.N; }

namespace {
// Launch of a pipeline kernel; when its stage is traced, the trace events
// are attached to the dispatch itself.
template <typename F, typename... A>
void klaunch_b(const Ctx& c, int stage, F kern, dim3 g, int block, hipStream_t st, A... args) {
  hipEvent_t t0, t1;
  c.trace_take(stage, &t0, &t1);
  hipExtLaunchKernelGGL(kern, g, dim3(block), 0, st, t0, t1, 0, args...);
}
template <typename F, typename... A>
void klaunch(const Ctx& c, int stage, F kern, dim3 g, hipStream_t st, A... args) {
  klaunch_b(c, stage, kern, g, kWG, st, args...);
}

// Groups of output rows of a column-conversion launch whose work-groups number
// `base` at one group each (column tiles x digits or components x jobs), with
// at most `rows` output rows: enough to have a work-group per CU (a group more
// repeats the input transforms, a quarter of the work at 12 inputs and 36 rows,
// and a second work-group on a CU only shares its vector units), none with
// less than a pair of rows, and at most 8 `cap` rows in a group, `cap` being
// the schedule's BConv rows.
int conv_groups(long base, int rows, int cap) {
  constexpr long kFill = 256;
  const long fill = std::min<long>((kFill + base - 1) / base, (rows + 1) / 2);
  const long need = (rows + 8 * cap - 1) / (8 * cap);
  return (int)std::max({1l, fill, need});
}

int up_groups(const Ctx& c, const Ctx::Sched& sc, int njobs, int Lmax) {
  return conv_groups((long)(c.N / 512) * c.beta(Lmax) * njobs, Lmax + c.k - 1, sc.up_rows);
}
// comps: components, two of a key-switch
int down_groups(const Ctx& c, const Ctx::Sched& sc, int njobs, int Lmax, int comps) {
  return conv_groups((long)(c.N / 512) * comps * njobs, Lmax, sc.down_rows);
}
// The inner product of `rows` rows a job takes the kernel for small grids: too few
// work-groups to fill the CUs (k5p_ntt_blks_ip has the line's reasons).
bool small_ip(const Ctx& c, const Ctx::Sched& sc, int njobs, int Lmax, int rows) {
  return c.beta(Lmax) <= 4 && c.N / kTile * rows * njobs <= sc.small_grid;
}

template <int L1, int MODE>
hipError_t conv_launch(const Ctx& c, int stage, int nin, dim3 g, hipStream_t st, const KsConst& K,
                       const JobArg<KsJob>& jobs, int groups) {
  const uint32_t* bytes = MODE == CONV_UP ? c.modup_bytes : c.moddown_bytes;
  auto go = [&](auto kern) { klaunch_b(c, stage, kern, g, 64 * kConvWaves, st, K, jobs, groups, bytes); };
  if (nin <= 4)
    go(kc_conv<L1, MODE, 4>);
  else if (nin <= 12)
    go(kc_conv<L1, MODE, 12>);
  else
    go(kc_conv<L1, MODE, 16>);
  return hipGetLastError();
}

// Stage 1 (ModUp): the block pass and the column kernel.
template <int L1>
hipError_t modup_stage_t(const Ctx& c, const Ctx::Sched& sc, const KsConst& K, const JobArg<KsJob>& jobs,
                         int njobs, int Lmax, hipStream_t st) {
  const int beta = c.beta(Lmax), tiles = c.N / 512;
  const int groups = up_groups(c, sc, njobs, Lmax);
  klaunch(c, CKKS_STAGE_INTT_BLOCKS, k1_intt_blks, dim3(c.N / kTile, Lmax, njobs), st, K, jobs);
  return conv_launch<L1, CONV_UP>(c, CKKS_STAGE_INTT_COLS, c.alpha, dim3(tiles, beta * groups, njobs), st, K, jobs,
                                  groups);
}

template <int L1>
hipError_t ks_modup_launch_t(const Ctx& c, const Ctx::Sched& sc, const KsConst& K, const JobArg<KsJob>& jobs,
                             int njobs, int Lmax, hipStream_t st) {
  const hipError_t e = modup_stage_t<L1>(c, sc, K, jobs, njobs, Lmax, st);
  if (e != hipSuccess) return e;
  klaunch(c, -1, km_ntt_blks, dim3(c.N / kTile, c.beta(Lmax) * (Lmax + c.k), njobs), st, K, jobs);
  return hipGetLastError();
}

// ModDown alone: block pass of the P rows, the column kernel, the combine
// (N = 2^16, L = 36: 57 us in six stand-alone kernels -> 28).
template <int L1>
hipError_t ks_moddown_launch_t(const Ctx& c, const Ctx::Sched& sc, const KsConst& K, const JobArg<KsJob>& jobs,
                               int njobs, int Lmax, hipStream_t st) {
  klaunch(c, -1, k1_intt_blks, dim3(c.N / kTile, c.k, njobs), st, K, jobs);
  const int groups = down_groups(c, sc, njobs, Lmax, 1);
  const hipError_t e =
      conv_launch<L1, CONV_DOWN>(c, -1, c.k, dim3(c.N / 512, groups, njobs), st, K, jobs, groups);
  if (e != hipSuccess) return e;
  klaunch(c, -1, kd_ntt_blks_combine, dim3(c.N / kTile, Lmax, njobs), st, K, jobs);
  return hipGetLastError();
}

bool takes_whole_limbs(const Ctx& c, const Ctx::Sched& sc, bool whole_limb) {
  return whole_limb && (sc.ntt_shape & kShapeWholeLimb) && ks_whole_limb_ring(c);
}

template <int L1>
hipError_t ks_launch_t(const Ctx& c, const Ctx::Sched& sc, const KsConst& K, const JobArg<KsJob>& jobs,
                       int njobs, int Lmax, bool with_modup, bool with_hoist, hipStream_t st,
                       bool whole_limb) {
  const int tiles = c.N / kTile;
  hipError_t e;
  if constexpr (L1 + kBlockLog == kSrLog) {
    // small ring: two kernels on whole limbs (plain, HMult and HRot jobs), for
    // digits of at most kSrDigit limbs
    if (with_modup && !with_hoist && takes_whole_limbs(c, sc, whole_limb)) {
      // every job splits its own digits into sr_groups(beta) <= min(beta, kSrGroups)
      // groups, so the grid covers min(bmax, kSrGroups) (not the largest job's count)
      const int groups = std::min(c.beta(Lmax), kSrGroups);
      const dim3 g1(Lmax + c.k, groups, njobs);
      if (c.beta(Lmax) <= kSrGroups)
        klaunch(c, CKKS_STAGE_NTT_IP, s1_modup_ip<true>, g1, st, K, jobs);
      else
        klaunch(c, CKKS_STAGE_NTT_IP, s1_modup_ip<false>, g1, st, K, jobs);
      klaunch_b(c, CKKS_STAGE_NTT_COMBINE, s2_moddown, dim3(Lmax, 2, njobs), kWG, st, K, jobs);
      return hipGetLastError();
    }
  }
  if (with_modup && (e = modup_stage_t<L1>(c, sc, K, jobs, njobs, Lmax, st)) != hipSuccess) return e;
  // Stage 2 on the P rows, ModDown's column stages, stage 2 on the Q rows with
  // the combine.
  auto k5 = [&](auto q, int stage, int rows) {
    constexpr bool Q = decltype(q)::value;
    const dim3 g5(tiles, rows, njobs), g4(4 * tiles, rows, njobs);
    const int nb = std::max(c.beta(Lmax), 2);  // slots for the launch's own largest digit count
    // a single job streams its key (measured: K5 39.8 -> 35.6 us at N = 2^16,
    // L = 36, alternating keys); jobs of a batch may share one
    const bool nt = njobs == 1;
    auto of = [&](auto n) {
      constexpr int NB = decltype(n)::value;
      if (small_ip(c, sc, njobs, Lmax, rows))
        klaunch_b(c, stage, k5p_ntt_blks_ip<NB, Q>, g4, 64 * NB, st, K, jobs);
      else if (nt)
        klaunch(c, stage, k5s_ntt_blks_ip<NB, true, Q>, g5, st, K, jobs);
      else
        klaunch(c, stage, k5s_ntt_blks_ip<NB, false, Q>, g5, st, K, jobs);
    };
    switch (nb) {
      case 2: of(std::integral_constant<int, 2>()); break;
      case 3: of(std::integral_constant<int, 3>()); break;
      case 4: of(std::integral_constant<int, 4>()); break;
      default: klaunch(c, stage, k5_ntt_blks_ip<false, Q>, g5, st, K, jobs); break;
    }
  };
  auto k5h = [&](auto q, int stage, int rows) {
    constexpr bool Q = decltype(q)::value;
    const dim3 gh(tiles, rows, njobs);
    switch (std::max(c.beta(Lmax), 2)) {  // slots for the launch's own largest digit count
      case 2: klaunch(c, stage, k5h_gather_ip<2, Q>, gh, st, K, jobs); break;
      case 3: klaunch(c, stage, k5h_gather_ip<3, Q>, gh, st, K, jobs); break;
      case 4: klaunch(c, stage, k5h_gather_ip<4, Q>, gh, st, K, jobs); break;
      default: klaunch(c, stage, k5_ntt_blks_ip<true, Q>, gh, st, K, jobs); break;
    }
  };
  if (with_modup) k5(std::false_type(), CKKS_STAGE_NTT_IP_P, c.k);
  if (with_hoist) k5h(std::false_type(), CKKS_STAGE_NTT_IP_P, c.k);
  const int groups = down_groups(c, sc, njobs, Lmax, 2);
  e = conv_launch<L1, CONV_DOWN>(c, CKKS_STAGE_INTT_COLS_P, c.k, dim3(c.N / 512, 2 * groups, njobs), st, K, jobs,
                                 groups);
  if (e != hipSuccess) return e;
  // one kernel under two names
  const int stage_q = c.trace.stage == CKKS_STAGE_NTT_COMBINE ? CKKS_STAGE_NTT_COMBINE : CKKS_STAGE_NTT_IP;
  if (with_modup) k5(std::true_type(), stage_q, Lmax);
  if (with_hoist) k5h(std::true_type(), stage_q, Lmax);
  return hipGetLastError();
}

template <int L1>
hipError_t rs_launch_t(const Ctx& c, const KsConst& K, const JobArg<RsJob>& jobs, int njobs,
                       int Lmax, hipStream_t st) {
  const int tiles = c.N / kTile;
  klaunch(c, -1, r1_intt_blks, dim3(tiles, 2, njobs), st, K, jobs);
  const int groups = conv_groups((long)(c.N / 512) * 2 * njobs, Lmax - 1, kMaxPrimes);
  klaunch_b(c, -1, r2_cols<L1>, dim3(c.N / 512, 2 * groups, njobs), 64 * kConvWaves, st, K, jobs, groups);
  klaunch(c, CKKS_STAGE_RESCALE_NTT, r4_ntt_blks_combine, dim3(tiles, 2 * (Lmax - 1), njobs), st, K, jobs);
  return hipGetLastError();
}
}  // namespace

KsGrids ks_grids(const Ctx& c, const Ctx::Sched& sc, int njobs, int Lmax, bool whole_limb) {
  if (takes_whole_limbs(c, sc, whole_limb)) return KsGrids{true, 0, 0, false, false};
  return KsGrids{false, up_groups(c, sc, njobs, Lmax), down_groups(c, sc, njobs, Lmax, 2),
                 small_ip(c, sc, njobs, Lmax, c.k), small_ip(c, sc, njobs, Lmax, Lmax)};
}

hipError_t ks_launch(const Ctx& c, const Ctx::Sched& sc, const JobArg<KsJob>& jobs, int njobs, int Lmax,
                     bool with_modup, bool with_hoist, hipStream_t st, bool whole_limb) {
  if (njobs <= 0) return hipSuccess;
  const KsConst K = make_const(c);
  switch (c.logN - kBlockLog) {
    case 4: return ks_launch_t<4>(c, sc, K, jobs, njobs, Lmax, with_modup, with_hoist, st, whole_limb);
    case 5: return ks_launch_t<5>(c, sc, K, jobs, njobs, Lmax, with_modup, with_hoist, st, whole_limb);
    case 6: return ks_launch_t<6>(c, sc, K, jobs, njobs, Lmax, with_modup, with_hoist, st, whole_limb);
    case 7: return ks_launch_t<7>(c, sc, K, jobs, njobs, Lmax, with_modup, with_hoist, st, whole_limb);
    case 8: return ks_launch_t<8>(c, sc, K, jobs, njobs, Lmax, with_modup, with_hoist, st, whole_limb);
    default: return hipErrorInvalidValue;
  }
}

hipError_t ks_modup_launch(const Ctx& c, const Ctx::Sched& sc, const JobArg<KsJob>& jobs, int njobs, int Lmax,
                           hipStream_t st) {
  if (njobs <= 0) return hipSuccess;
  const KsConst K = make_const(c);
  switch (c.logN - kBlockLog) {
    case 4: return ks_modup_launch_t<4>(c, sc, K, jobs, njobs, Lmax, st);
    case 5: return ks_modup_launch_t<5>(c, sc, K, jobs, njobs, Lmax, st);
    case 6: return ks_modup_launch_t<6>(c, sc, K, jobs, njobs, Lmax, st);
    case 7: return ks_modup_launch_t<7>(c, sc, K, jobs, njobs, Lmax, st);
    case 8: return ks_modup_launch_t<8>(c, sc, K, jobs, njobs, Lmax, st);
    default: return hipErrorInvalidValue;
  }
}

hipError_t ks_moddown_launch(const Ctx& c, const Ctx::Sched& sc, const JobArg<KsJob>& jobs, int njobs, int Lmax,
                             hipStream_t st) {
  if (njobs <= 0) return hipSuccess;
  const KsConst K = make_const(c);
  switch (c.logN - kBlockLog) {
    case 4: return ks_moddown_launch_t<4>(c, sc, K, jobs, njobs, Lmax, st);
    case 5: return ks_moddown_launch_t<5>(c, sc, K, jobs, njobs, Lmax, st);
    case 6: return ks_moddown_launch_t<6>(c, sc, K, jobs, njobs, Lmax, st);
    case 7: return ks_moddown_launch_t<7>(c, sc, K, jobs, njobs, Lmax, st);
    case 8: return ks_moddown_launch_t<8>(c, sc, K, jobs, njobs, Lmax, st);
    default: return hipErrorInvalidValue;
  }
}

hipError_t rs_launch(const Ctx& c, const JobArg<RsJob>& jobs, int njobs, int Lmax, hipStream_t st) {
  if (njobs <= 0 || Lmax < 2) return hipSuccess;
  const KsConst K = make_const(c);
  switch (c.logN - kBlockLog) {
    case 4: return rs_launch_t<4>(c, K, jobs, njobs, Lmax, st);
    case 5: return rs_launch_t<5>(c, K, jobs, njobs, Lmax, st);
    case 6: return rs_launch_t<6>(c, K, jobs, njobs, Lmax, st);
    case 7: return rs_launch_t<7>(c, K, jobs, njobs, Lmax, st);
    case 8: return rs_launch_t<8>(c, K, jobs, njobs, Lmax, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace ckks
