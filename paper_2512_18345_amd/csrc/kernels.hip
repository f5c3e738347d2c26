// gfx950 kernels for the stand-alone entry points: NTT / INTT (two passes,
// see mont_ntt.h), inner product, tensor, automorphism, plaintext sums.  The
// key-switching pipeline, ModUp and ModDown live in keyswitch.hip.
#include <hip/hip_runtime.h>

#include "arith.h"
#include "ctx.h"
#include "kernels.h"
#include "mont_ntt.h"

namespace ckks {

// ============================================================================
// NTT kernels: in place and in row order throughout (a transform has no
// workspace), so the column pass takes tiles of at least 32 columns, whole
// 128-byte lines of every row, through LDS.  A wave owns C of the columns and
// transforms them in the LDS tile as mont_ntt.h does, without a barrier; the
// block pass needs none at all.  Bound: the loads, transform and stores of one
// round of work-groups follow one another.  N = 2^16, 48 rows: forward 12.3 +
// 13.0 -> 8.6 + 7.4 us, inverse 10.6 + 15.5 -> 7.0 + 9.1 (radix-16 tiles of 256
// threads with barriers and twiddles in LDS before).  Few rows: a call of up to 16
// rows (36 at N = 2^15) takes the 10.4 us of its two launches back to back, before
// as now, but for N = 2^16 (11.1 .. 14.4).
// ============================================================================
template <int LOGN1>
struct ColTile {
  using CH = ColPart<LOGN1, 64>;
  static constexpr int N1 = 1 << LOGN1, C = CH::C;
  static constexpr int W = C >= 8 ? 4 : 8;   // waves
  static constexpr int COLS = W * C;         // 32 .. 256
  static constexpr int T = 64 * W;
  static constexpr int QUADS = N1 * COLS / (4 * T);  // per thread: 4
  // word (row, col) of the tile: both layouts of a wave's columns meet 64
  // different banks (rows of one 16 C + COLS words apart, groups of 16 rows C more)
  __device__ static __forceinline__ int at(int row, int col) { return row * (COLS + C) + (row >> 4) * C + col; }
  static constexpr int LDS = N1 * (COLS + C) + (N1 >> 4) * C;
};

template <int LOGN1, bool INV>
__global__ __launch_bounds__(ColTile<LOGN1>::T) void k_ntt_cols(DevTab T, MontTab M, RowMap rm, uint32_t* a) {
  using CT = ColTile<LOGN1>;
  using CH = typename CT::CH;
  __shared__ __align__(16) uint32_t s[CT::LDS];
  const int r = blockIdx.y, pi = rm.pidx(r);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  uint32_t* row = a + ((size_t)r << T.logN) + blockIdx.x * CT::COLS;
  uint4 raw[CT::QUADS];
#pragma unroll
  for (int k = 0; k < CT::QUADS; ++k) {
    const int lin = 4 * (threadIdx.x + k * CT::T);
    raw[k] = ld4(row + (lin / CT::COLS) * 256 + lin % CT::COLS);
  }
  typename CH::Tw tw;
  tw.load(INV ? M.col_itw(T, pi) : M.col_tw(T, pi), lane);
  const ModC mc = ldc(T.mod + pi);
  const MontQ m = mont_q(mc);
#pragma unroll
  for (int k = 0; k < CT::QUADS; ++k) {
    const int lin = 4 * (threadIdx.x + k * CT::T);
    *reinterpret_cast<uint4*>(s + CT::at(lin / CT::COLS, lin % CT::COLS)) = raw[k];
  }
  __syncthreads();
  const int c0 = w * CT::C + lane % CT::C, node = lane / CT::C;  // node: 16-row group (low layout), r (high)
  constexpr int E = CH::E;
  uint32_t v[16];
  auto high_row = [&](int k) { return 16 * (k >> (4 - E)) + ((k & ((16 >> E) - 1)) << E) + node; };
  auto get_high = [&]() {
#pragma unroll
    for (int k = 0; k < 16; ++k) v[k] = s[CT::at(high_row(k), c0)];
  };
  auto put_high = [&]() {
#pragma unroll
    for (int k = 0; k < 16; ++k) s[CT::at(high_row(k), c0)] = v[k];
  };
  auto get_low = [&]() {
#pragma unroll
    for (int j = 0; j < 16; ++j) v[j] = s[CT::at(16 * node + j, c0)];
  };
  auto put_low = [&]() {
#pragma unroll
    for (int j = 0; j < 16; ++j) s[CT::at(16 * node + j, c0)] = v[j];
  };
  if constexpr (!INV) {
    if constexpr (E > 0) {
      get_high();
      ct_stages<0, E>(v, tw.hi, m);
      put_high();
      wave_sync();
    }
    get_low();
    ct_stages<0, 4>(v, tw.lo, m);
    put_low();
  } else {
    get_low();
    gs_stages<0, 4>(v, tw.lo, m);
    if constexpr (E > 0) {
      put_low();
      wave_sync();
      get_high();
      gs_stages<0, E>(v, tw.hi, m);
    }
#pragma unroll
    for (int k = 0; k < 16; ++k) v[k] = csub(mul_shoup(v[k], mc.ninv, mc.ninv_s, m.q), m.q);
    if constexpr (E > 0)
      put_high();
    else
      put_low();
  }
  __syncthreads();
  const OutRow out(row);
#pragma unroll
  for (int k = 0; k < CT::QUADS; ++k) {
    const int lin = 4 * (threadIdx.x + k * CT::T);
    out.st4((lin / CT::COLS) * 256 + lin % CT::COLS,
            *reinterpret_cast<const uint4*>(s + CT::at(lin / CT::COLS, lin % CT::COLS)));
  }
}

template <bool INV>
__global__ __launch_bounds__(kWG) void k_ntt_blks(DevTab T, MontTab M, RowMap rm, uint32_t* a) {
  __shared__ __align__(16) uint32_t s[kBlkTile];
  const int r = blockIdx.y, pi = rm.pidx(r);
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int line = blk_line<16>(lane, w);
  uint32_t* row = a + ((size_t)r << T.logN) + blockIdx.x * kTile;
  const int n0 = line * 256 + 4 * (lane & 15);
  uint4 x[4];
  BlkTw tw;
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) x[kk] = ld4(row + n0 + 64 * kk);
  tw.load(INV ? M.row_itw(T, pi, blockIdx.x * 16 + line) : M.row_tw(T, pi, blockIdx.x * 16 + line),
          INV ? M.blk_itw(pi) : M.blk_tw(pi), lane);
  const MontQ m = mont_q(ldc(T.mod + pi));
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) blk_quad_store(s, line, 4 * (lane & 15) + 64 * kk, x[kk]);
  wave_sync();
  if constexpr (INV)
    blk_inv_a(s, line, lane, tw, m);
  else
    blk_fwd_a(s, line, lane, tw, m);
  wave_sync();
  if constexpr (INV)
    blk_inv_b(s, line, lane, tw, m);
  else
    blk_fwd_b(s, line, lane, tw, m);
  wave_sync();
  const OutRow out(row);
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) {
    const uint4 v = blk_quad(s, line, 4 * (lane & 15) + 64 * kk);
    out.st4(n0 + 64 * kk, INV ? v : canon4(v, m.q, m.q2));
  }
}

// ============================================================================
// Element-wise kernels (Sec. II-B3)
// ============================================================================

// acc[c][r] = sum_j M[j][r] * evk[j][c][krow(r)] (Sec. IV-B stage 2).
__global__ __launch_bounds__(kWG) void k_inner_product(DevTab T, RowMap rm, const uint32_t* M,
                                                       int beta, int nrows, const uint32_t* evk,
                                                       uint32_t* acc) {
  const size_t N = (size_t)1 << T.logN;
  const size_t n = (size_t)blockIdx.x * kWG + threadIdx.x;
  const int r = blockIdx.y;
  const int pi = rm.pidx(r);
  const ModC mc = T.mod[pi];
  const size_t krows = (size_t)(T.L_max + (nrows - rm.L));
  uint64_t a0 = 0, a1 = 0;
  for (int j = 0; j < beta; ++j) {
    const uint32_t m = M[((size_t)j * nrows + r) * N + n];
    const uint32_t* e = evk + (size_t)j * 2 * krows * N + (size_t)pi * N + n;
    a0 += (uint64_t)m * e[0];
    a1 += (uint64_t)m * e[krows * N];
    if ((j & 7) == 7) {  // products below 2^60: fold before 16 of them add up
      a0 = reduce64(a0, mc.q, mc.mu_hi, mc.mu_lo);
      a1 = reduce64(a1, mc.q, mc.mu_hi, mc.mu_lo);
    }
  }
  acc[(size_t)r * N + n] = reduce64(a0, mc.q, mc.mu_hi, mc.mu_lo);
  acc[((size_t)nrows + r) * N + n] = reduce64(a1, mc.q, mc.mu_hi, mc.mu_lo);
}

// d0 = c0 c0', d1 = c0 c1' + c1 c0', d2 = c1 c1' over [L][N].
__global__ __launch_bounds__(kWG) void k_tensor(DevTab T, const uint32_t* ct1, const uint32_t* ct2,
                                                int L, uint32_t* out) {
  const size_t N = (size_t)1 << T.logN;
  const size_t n = (size_t)blockIdx.x * kWG + threadIdx.x;
  const int r = blockIdx.y;
  const ModC mc = T.mod[r];
  const size_t e = (size_t)r * N + n, P = (size_t)L * N;
  const uint32_t a0 = ct1[e], a1 = ct1[P + e], b0 = ct2[e], b1 = ct2[P + e];
  out[e] = reduce64((uint64_t)a0 * b0, mc.q, mc.mu_hi, mc.mu_lo);
  out[P + e] = reduce64((uint64_t)a0 * b1 + (uint64_t)a1 * b0, mc.q, mc.mu_hi, mc.mu_lo);
  out[2 * P + e] = reduce64((uint64_t)a1 * b1, mc.q, mc.mu_hi, mc.mu_lo);
}

// Eval-domain automorphism: out[r][j] = in[r][j'], 2 brv(j') + 1 = g (2 brv(j) + 1) mod 2N.
__global__ __launch_bounds__(kWG) void k_automorph(int logN, const uint32_t* in, uint32_t* out,
                                                   int rows, uint32_t g, int rows_per_block) {
  const size_t N = (size_t)1 << logN;
  const uint32_t j = blockIdx.x * kWG + threadIdx.x;
  const uint32_t mask2n = (uint32_t)(2 * N - 1);
  const uint32_t bj = __builtin_bitreverse32(j) >> (32 - logN);
  const uint32_t e = (g * (2 * bj + 1)) & mask2n;
  const uint32_t src = __builtin_bitreverse32((e - 1) >> 1) >> (32 - logN);
  const int r0 = blockIdx.y * rows_per_block;
  const int r1 = min(r0 + rows_per_block, rows);
  for (int r = r0; r < r1; ++r) out[(size_t)r * N + j] = in[(size_t)r * N + src];
}

// Plaintext products summed (the baby-step inner products of a BSGS linear
// transform): out[c][i] = sum_b ct_b[c][i] * pt_b[i] mod q_i, b < nb <= 16.
// Sixteen products of canonical residues stay below 2^64: one reduction.
struct PtrList16 {
  const uint32_t* p[16];
};
__global__ __launch_bounds__(kWG) void k_pmult_sum(DevTab T, PtrList16 cts, PtrList16 pts, int nb, int L,
                                                   uint32_t* out) {
  const size_t N = (size_t)1 << T.logN;
  const size_t n = ((size_t)blockIdx.x * kWG + threadIdx.x) * 4;  // four coefficients per thread
  const int i = blockIdx.y;
  const ModC m = ldc(T.mod + i);
  uint64_t a0[4] = {0, 0, 0, 0}, a1[4] = {0, 0, 0, 0};
  for (int b = 0; b < nb; ++b) {
    const uint4 pt = ld4(pts.p[b] + (size_t)i * N + n);
    const uint4 x = ld4(cts.p[b] + (size_t)i * N + n);
    const uint4 y = ld4(cts.p[b] + ((size_t)L + i) * N + n);
    a0[0] += (uint64_t)x.x * pt.x;
    a0[1] += (uint64_t)x.y * pt.y;
    a0[2] += (uint64_t)x.z * pt.z;
    a0[3] += (uint64_t)x.w * pt.w;
    a1[0] += (uint64_t)y.x * pt.x;
    a1[1] += (uint64_t)y.y * pt.y;
    a1[2] += (uint64_t)y.z * pt.z;
    a1[3] += (uint64_t)y.w * pt.w;
  }
  st4(out + (size_t)i * N + n, make_uint4(reduce64(a0[0], m.q, m.mu_hi, m.mu_lo), reduce64(a0[1], m.q, m.mu_hi, m.mu_lo),
                                          reduce64(a0[2], m.q, m.mu_hi, m.mu_lo), reduce64(a0[3], m.q, m.mu_hi, m.mu_lo)));
  st4(out + ((size_t)L + i) * N + n,
      make_uint4(reduce64(a1[0], m.q, m.mu_hi, m.mu_lo), reduce64(a1[1], m.q, m.mu_hi, m.mu_lo),
                 reduce64(a1[2], m.q, m.mu_hi, m.mu_lo), reduce64(a1[3], m.q, m.mu_hi, m.mu_lo)));
}

// Several inner sums over the same ciphertexts (the giant steps of one BSGS
// level): out_g[c][i] = sum_b ct_b[c][i] * pt_{g,b}[i] mod q_i for g < NG.
// Each ciphertext word is read once for all NG sums.
struct PtrList128 {
  const uint32_t* p[128];
};
struct OutList8 {
  uint32_t* p[8];
};
template <int NG>
__global__ __launch_bounds__(kWG) void k_pmult_sums(DevTab T, PtrList16 cts, PtrList128 pts, OutList8 outs,
                                                    int nb, int L) {
  const size_t N = (size_t)1 << T.logN;
  const size_t n = ((size_t)blockIdx.x * kWG + threadIdx.x) * 4;  // four coefficients per thread
  const int i = blockIdx.y;
  const ModC m = ldc(T.mod + i);
  uint64_t a0[NG][4], a1[NG][4];
#pragma unroll
  for (int g = 0; g < NG; ++g)
#pragma unroll
    for (int e = 0; e < 4; ++e) a0[g][e] = a1[g][e] = 0;
  for (int b = 0; b < nb; ++b) {
    const uint4 x = ld4(cts.p[b] + (size_t)i * N + n);
    const uint4 y = ld4(cts.p[b] + ((size_t)L + i) * N + n);
#pragma unroll
    for (int g = 0; g < NG; ++g) {
      const uint4 pt = ld4(pts.p[g * 16 + b] + (size_t)i * N + n);
      a0[g][0] += (uint64_t)x.x * pt.x;
      a0[g][1] += (uint64_t)x.y * pt.y;
      a0[g][2] += (uint64_t)x.z * pt.z;
      a0[g][3] += (uint64_t)x.w * pt.w;
      a1[g][0] += (uint64_t)y.x * pt.x;
      a1[g][1] += (uint64_t)y.y * pt.y;
      a1[g][2] += (uint64_t)y.z * pt.z;
      a1[g][3] += (uint64_t)y.w * pt.w;
    }
  }
#pragma unroll
  for (int g = 0; g < NG; ++g) {
    st4(outs.p[g] + (size_t)i * N + n,
        make_uint4(reduce64(a0[g][0], m.q, m.mu_hi, m.mu_lo), reduce64(a0[g][1], m.q, m.mu_hi, m.mu_lo),
                   reduce64(a0[g][2], m.q, m.mu_hi, m.mu_lo), reduce64(a0[g][3], m.q, m.mu_hi, m.mu_lo)));
    st4(outs.p[g] + ((size_t)L + i) * N + n,
        make_uint4(reduce64(a1[g][0], m.q, m.mu_hi, m.mu_lo), reduce64(a1[g][1], m.q, m.mu_hi, m.mu_lo),
                   reduce64(a1[g][2], m.q, m.mu_hi, m.mu_lo), reduce64(a1[g][3], m.q, m.mu_hi, m.mu_lo)));
  }
}

// Ciphertext sum: out = a + b over [2][L][N].
__global__ __launch_bounds__(kWG) void k_ct_add(DevTab T, const uint32_t* a, const uint32_t* b, int L,
                                                uint32_t* out) {
  const size_t N = (size_t)1 << T.logN;
  const int r = blockIdx.y;  // 0 .. 2L-1
  const uint32_t q = ldc(T.mod + (r % L)).q;
  const size_t e = (size_t)r * N + ((size_t)blockIdx.x * kWG + threadIdx.x) * 4;
  const uint4 x = ld4(a + e), y = ld4(b + e);
  st4(out + e, make_uint4(csub(x.x + y.x, q), csub(x.y + y.y, q), csub(x.z + y.z, q), csub(x.w + y.w, q)));
}

// ============================================================================
// Launchers
// ============================================================================
#define CKKS_DISPATCH_LOGN1(logN1, CALL) \
  switch (logN1) {                       \
    case 4: CALL(4); break;              \
    case 5: CALL(5); break;              \
    case 6: CALL(6); break;              \
    case 7: CALL(7); break;              \
    case 8: CALL(8); break;              \
    default: return hipErrorInvalidValue; \
  }

hipError_t launch_ntt(const Ctx& c, uint32_t* a, int rows, RowMap rm, bool inverse, hipStream_t st) {
  if (rows <= 0) return hipSuccess;
  const dim3 blks(c.N / kTile, rows);
#define CALL(L1)                                                                       \
  {                                                                                    \
    const dim3 cols(256 / ColTile<L1>::COLS, rows);                                    \
    if (inverse) {                                                                     \
      k_ntt_blks<true><<<blks, kWG, 0, st>>>(c.tab(), c.mont, rm, a);                  \
      k_ntt_cols<L1, true><<<cols, ColTile<L1>::T, 0, st>>>(c.tab(), c.mont, rm, a);   \
    } else {                                                                           \
      k_ntt_cols<L1, false><<<cols, ColTile<L1>::T, 0, st>>>(c.tab(), c.mont, rm, a);  \
      k_ntt_blks<false><<<blks, kWG, 0, st>>>(c.tab(), c.mont, rm, a);                 \
    }                                                                                  \
  }
  CKKS_DISPATCH_LOGN1(c.logN - kBlockLog, CALL)
#undef CALL
  return hipGetLastError();
}

hipError_t launch_inner_product(const Ctx& c, RowMap rm, const uint32_t* M, int beta, int nrows,
                                const uint32_t* evk, uint32_t* acc, hipStream_t st) {
  k_inner_product<<<dim3(c.N / kWG, nrows), kWG, 0, st>>>(c.tab(), rm, M, beta, nrows, evk, acc);
  return hipGetLastError();
}

hipError_t launch_tensor(const Ctx& c, const uint32_t* ct1, const uint32_t* ct2, int L,
                         uint32_t* out, hipStream_t st) {
  k_tensor<<<dim3(c.N / kWG, L), kWG, 0, st>>>(c.tab(), ct1, ct2, L, out);
  return hipGetLastError();
}

hipError_t launch_automorph(const Ctx& c, const uint32_t* in, uint32_t* out, int rows, uint32_t g,
                            hipStream_t st) {
  const int rpb = 4;
  k_automorph<<<dim3(c.N / kWG, (rows + rpb - 1) / rpb), kWG, 0, st>>>(c.logN, in, out, rows, g, rpb);
  return hipGetLastError();
}

hipError_t launch_pmult_sum(const Ctx& c, const uint32_t* const* cts, const uint32_t* const* pts, int nb,
                            int L, uint32_t* out, hipStream_t st) {
  if (nb < 1 || nb > 16) return hipErrorInvalidValue;
  PtrList16 a{}, b{};
  for (int i = 0; i < nb; ++i) {
    a.p[i] = cts[i];
    b.p[i] = pts[i];
  }
  k_pmult_sum<<<dim3(c.N / (4 * kWG), L), kWG, 0, st>>>(c.tab(), a, b, nb, L, out);
  return hipGetLastError();
}

hipError_t launch_pmult_sums(const Ctx& c, const uint32_t* const* cts, int nb, const uint32_t* const* pts,
                             int ng, int L, uint32_t* const* outs, hipStream_t st) {
  if (nb < 1 || nb > 16 || ng < 1 || ng > 8) return hipErrorInvalidValue;
  PtrList16 a{};
  PtrList128 b{};
  OutList8 o{};
  for (int j = 0; j < nb; ++j) a.p[j] = cts[j];
  for (int g = 0; g < ng; ++g) {
    o.p[g] = outs[g];
    for (int j = 0; j < nb; ++j) b.p[g * 16 + j] = pts[g * nb + j];
  }
  const dim3 grid(c.N / (4 * kWG), L);
  switch (ng) {
    case 1: k_pmult_sums<1><<<grid, kWG, 0, st>>>(c.tab(), a, b, o, nb, L); break;
    case 2: k_pmult_sums<2><<<grid, kWG, 0, st>>>(c.tab(), a, b, o, nb, L); break;
    case 3: k_pmult_sums<3><<<grid, kWG, 0, st>>>(c.tab(), a, b, o, nb, L); break;
    case 4: k_pmult_sums<4><<<grid, kWG, 0, st>>>(c.tab(), a, b, o, nb, L); break;
    case 5: k_pmult_sums<5><<<grid, kWG, 0, st>>>(c.tab(), a, b, o, nb, L); break;
    case 6: k_pmult_sums<6><<<grid, kWG, 0, st>>>(c.tab(), a, b, o, nb, L); break;
    case 7: k_pmult_sums<7><<<grid, kWG, 0, st>>>(c.tab(), a, b, o, nb, L); break;
    default: k_pmult_sums<8><<<grid, kWG, 0, st>>>(c.tab(), a, b, o, nb, L); break;
  }
  return hipGetLastError();
}

hipError_t launch_ct_add(const Ctx& c, const uint32_t* a, const uint32_t* b, int L, uint32_t* out,
                         hipStream_t st) {
  k_ct_add<<<dim3(c.N / (4 * kWG), 2 * L), kWG, 0, st>>>(c.tab(), a, b, L, out);
  return hipGetLastError();
}

}  // namespace ckks
