// sdq_nt_fast.hip -- the sweeps with the norm-sorted blocked QR
// (sdq_block.hpp) for one tile count SDQ_NT (compiled once per NT = 1..8,
// apart from sdq_nt.hip so that the sources compile in parallel).
#include "sdq_device.hpp"

#ifndef SDQ_NT
#error "define SDQ_NT"
#endif

#define SDQ_CAT2(a, b) a##b
#define SDQ_CAT(a, b) SDQ_CAT2(a, b)

namespace sdq {

namespace {
constexpr int NT = SDQ_NT;
constexpr bool TG = fast_sweep_tg(NT);
constexpr bool kLdsB = NT <= 5;              // a dense slice beside them
template <class KF>
hipError_t launch(KF kern, const Inst* inst, const SweepItem* items, int count, Queue* q, int grid, double* tscr,
                  hipStream_t s) {
  if (!tscr) return hipErrorInvalidValue;
  hipLaunchKernelGGL(kern, dim3(grid), dim3(64 * NT), 0, s, inst, items, count, q, tscr);
  return hipGetLastError();
}
template <class F>
hipError_t with_kernel(int variant, F f) {
  if (variant == kFastPlain) return f(k_sweep<NT, NT, false, false, false, TG, false, true>, false);
  if (variant == kFastDense) return f(k_sweep<NT, NT, kLdsB, false, true, TG, false, true>, kLdsB);
  if constexpr (NT >= kProdMinNT)
    if (variant == kFastProd) return f(k_sweep<NT, NT, false, false, true, true, true, true>, false);
  return hipErrorInvalidValue;
}
}  // namespace

hipError_t SDQ_CAT(launch_fast_sweep_nt, SDQ_NT)(int variant, const Inst* inst, const SweepItem* items, int count,
                                                Queue* q, int grid, double* tscr, hipStream_t s) {
  return with_kernel(variant, [&](auto kern, bool) { return launch(kern, inst, items, count, q, grid, tscr, s); });
}
hipError_t SDQ_CAT(fast_sweep_info_nt, SDQ_NT)(int variant, KernelInfo* out) {
  return with_kernel(variant, [&](auto kern, bool lds) {
    int nb = 0;
    hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, kern, 64 * NT, 0);
    out->threads = 64 * NT;
    out->lds_bytes = lds ? (int)sizeof(Smem<NT, NT, true>) : (int)sizeof(Smem<NT, NT, false>);
    out->blocks_per_cu = nb;
    return e;
  });
}

}  // namespace sdq
