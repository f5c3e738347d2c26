// Host launchers of the gfx950 kernels (kernels.hip).  All are asynchronous
// on `st` and return the launch status.
#pragma once
#include <hip/hip_runtime.h>

#include "ctx.h"

namespace ckks {

// Forward / inverse NTT of rows [0, rows) in place, canonical result.
hipError_t launch_ntt(const Ctx& c, uint32_t* a, int rows, RowMap rm, bool inverse, hipStream_t st);
hipError_t launch_inner_product(const Ctx& c, RowMap rm, const uint32_t* M, int beta, int nrows,
                                const uint32_t* evk, uint32_t* acc, hipStream_t st);
hipError_t launch_tensor(const Ctx& c, const uint32_t* ct1, const uint32_t* ct2, int L,
                         uint32_t* out, hipStream_t st);
hipError_t launch_automorph(const Ctx& c, const uint32_t* in, uint32_t* out, int rows, uint32_t g,
                            hipStream_t st);
hipError_t launch_pmult_sum(const Ctx& c, const uint32_t* const* cts, const uint32_t* const* pts, int nb,
                            int L, uint32_t* out, hipStream_t st);
hipError_t launch_pmult_sums(const Ctx& c, const uint32_t* const* cts, int nb, const uint32_t* const* pts,
                             int ng, int L, uint32_t* const* outs, hipStream_t st);
hipError_t launch_ct_add(const Ctx& c, const uint32_t* a, const uint32_t* b, int L, uint32_t* out,
                         hipStream_t st);

}  // namespace ckks
