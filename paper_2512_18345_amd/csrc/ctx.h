// Context (per ring degree N): device-resident tables and the launchers'
// view of them.  Internal to the library; the public surface is ckks.h.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <string>
#include <vector>

#include "../../include/ckks.h"

namespace ckks {

constexpr int kTileLog = 12;            // words of a block-pass work-group (16 rows)
constexpr int kTile = 1 << kTileLog;
constexpr int kBlockLog = 8;            // pass-2 line length (N = N1 * 256)
constexpr int kWG = 256;                // threads per work-group
constexpr int kMinLogN = 12, kMaxLogN = 16;
constexpr int kMaxPrimes = 64;
constexpr int kMaxAlpha = 16;           // digit size / special-prime count

// Per-prime constants (device).
struct ModC {
  uint32_t q;
  uint32_t mu32;        // floor(2^32 / q)
  uint32_t mu_hi, mu_lo;  // floor(2^64 / q)
  uint32_t ninv, ninv_s;  // N^-1 mod q and its Shoup companion
  uint32_t qn;            // -q^-1 mod 2^32 (Montgomery)
  uint32_t pad;
};

// Per-prime constants and the ring.
constexpr int kSrLog = 12;  // rings of this degree: whole-limb key-switch kernels
struct DevTab {
  const ModC* mod;   // [nprimes]
  int logN;
  int L_max;
  __host__ __device__ int logN1() const { return logN - 8; }
};

// Tables of the two-pass transforms (mont_ntt.h) and of the base conversions,
// one word w 2^32 mod q per entry:
//  * column pass: col / icol [nprimes][N1], index m + i < N1 -> psi^(+-brv_logN(m + i));
//  * block pass, first four stages: row / irow [nprimes][N1][32] with row b's own
//    twiddles, entry 2^s + g < 16 -> psi^(+-brv_logN((N1 + b) 2^s + g)), and at
//    entry 16 + j the factor rho_b^(+-j), rho_b = psi^(2 brv_logN1(b) + 1);
//  * block pass, last four stages: blk / iblk [nprimes][256], shared by every row
//    once its words carry that factor: index 2^s + g -> psi^(+-(N / 2^s) brv_s(g));
//  * the base-conversion pre-multipliers and tables.
struct MontTab {
  const uint32_t *col, *icol, *blk, *iblk, *row, *irow;
  const uint32_t *modup_scale, *modup_T, *moddown_scale, *moddown_T, *pinv;
  __device__ const uint32_t* col_tw(const DevTab& T, int pi) const { return col + ((size_t)pi << T.logN1()); }
  __device__ const uint32_t* col_itw(const DevTab& T, int pi) const { return icol + ((size_t)pi << T.logN1()); }
  __device__ const uint32_t* blk_tw(int pi) const { return blk + ((size_t)pi << 8); }
  __device__ const uint32_t* blk_itw(int pi) const { return iblk + ((size_t)pi << 8); }
  __device__ const uint32_t* row_tw(const DevTab& T, int pi, int b) const {
    return row + ((((size_t)pi << T.logN1()) + b) << 5);
  }
  __device__ const uint32_t* row_itw(const DevTab& T, int pi, int b) const {
    return irow + ((((size_t)pi << T.logN1()) + b) << 5);
  }
};

// A word below 2^31 - 2^23 as four signed bytes, sum b_d 2^(8 d).
__host__ __device__ inline uint32_t signed_bytes(uint32_t v) { return (v + 0x808080u) ^ 0x808080u; }

// Rows of a launch: row r of the data is prime index pidx(r).
struct RowMap {
  int L;       // rows [0, L) are q_0..q_{L-1}
  int L_max;   // rows >= L are p_{r - L}, prime index L_max + (r - L)
  __host__ __device__ int pidx(int r) const { return r < L ? r : L_max + (r - L); }
};

struct Ctx {
  int device;
  int logN, N;
  int L_max, k, dnum, alpha;
  std::vector<uint32_t> primes;  // q_0..q_{L_max-1}, p_0..p_{k-1}

  // device tables
  ModC* d_mod = nullptr;
  // Base conversions: the constants times 2^32 are in `mont`.  ModUp at level L
  // (1-based): pre-multipliers N^-1 (D_j/q_i)^-1 at [L][i], tables T[r][i] =
  // (D_j / q_{j alpha + i}) mod prime(r) over the L + k ModUp rows at offset
  // modup_T_off of (L, j).  ModDown: N^-1 (P/p_m)^-1, T[i][m] = (P/p_m) mod q_i.
  std::vector<size_t> modup_T_off;    // index (L * beta_max + j)
  uint32_t* d_modup_T_off = nullptr;  // modup_T_off in words, then again in table rows
  // P^-1 mod q_i with Shoup.
  uint2* d_pinv = nullptr;            // [L_max]
  // Rescale at level L: q_{L-1}^-1 mod q_i (Shoup), i < L - 1.
  uint2* d_rescale_inv = nullptr;     // [L_max + 1][L_max]

  MontTab mont{};
  uint32_t* d_mont = nullptr;         // every table of `mont`, one allocation
  // In it too, for conversions of more than four limbs: the tables in signed
  // bytes, four words an entry.  Word [row][e][i], a row's limbs padded to a
  // multiple of four, holds byte e of T[row][i] 2^(32 + 8 d) mod q in its byte d.
  const uint32_t *modup_bytes = nullptr, *moddown_bytes = nullptr;

  // kernel tracing (ckks_trace_begin / ckks_trace_end)
  struct Trace {
    int stage = 0;
    std::vector<hipEvent_t> starts, stops;
    int count = 0;
  };
  mutable Trace trace;

  // Kernel schedule of the key-switching pipeline (ckks_ctx_set_schedule /
  // ckks_ctx_tune): a work-group of ModUp's or ModDown's column kernel takes at
  // most eight times this many output rows (2, 4, 6 or 12; conv_groups), and the
  // largest inner-product grid that uses one thread group per digit (0: never).
  // Launch shapes only: results are bitwise the same under every schedule.
  // ntt_shape bits: kShapeWholeLimb (keyswitch.h).
  struct Sched {
    int up_rows = 12, down_rows = 6, small_grid = 128, ntt_shape = 0;
  };
  Sched sched;
  // The start / stop events for the next launch of a traced stage (both null
  // when the stage is not traced or the capacity is used up).  Launchers pass
  // them to hipExtLaunchKernel, which records them at the dispatch's own
  // start and end.
  void trace_take(int stage, hipEvent_t* t0, hipEvent_t* t1) const {
    *t0 = *t1 = nullptr;
    if (trace.stage == stage && trace.count < (int)trace.starts.size()) {
      *t0 = trace.starts[trace.count];
      *t1 = trace.stops[trace.count++];
    }
  }

  DevTab tab() const {
    return DevTab{d_mod, logN, L_max};
  }
  RowMap rows(int L) const { return RowMap{L, L_max}; }
  int beta(int L) const { return (L + alpha - 1) / alpha; }
  int beta_max() const { return beta(L_max); }
};

// Host-side table construction (params.cpp).  Returns "" or an error message.
std::string build_tables(Ctx& c, const uint32_t* q, const uint32_t* p, int* code);
void free_tables(Ctx& c);

}  // namespace ckks

struct ckks_ctx {
  ckks::Ctx c;
};
