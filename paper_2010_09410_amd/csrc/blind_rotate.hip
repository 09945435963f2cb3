// Launches of the one-wave form of the blind rotation, in a source of its own because its kernel gains from
// an instruction order that the others lose by (build.py).
#include "blind_rotate.h"

namespace vsp {

hipError_t init_blind_rotate_waves() {
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_blind_rotate<8, true>),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)br_lds_bytes(8, true));
  if (e == hipSuccess)
    e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_blind_rotate<8, false>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)br_lds_bytes(8, false));
  return e;
}

hipError_t blind_rotate_waves_per_cu(int* workgroups) {
  return hipOccupancyMaxActiveBlocksPerMultiprocessor(workgroups, reinterpret_cast<const void*>(&k_blind_rotate<8, true>), 512,
                                                      br_lds_bytes(8, true));
}

// One key for all gates: a workgroup shares it; per-gate keys: each wave reads its own.
hipError_t launch_blind_rotate_waves(const vsp_context* ctx, const c64* bkf, const uint8_t* ops, const uint32_t* abar,
                                     uint32_t* tlwe1, uint32_t* trlwe, uint64_t B, const c64* const* keytab,
                                     const uint16_t* kid, hipStream_t st) {
  auto* kern = keytab ? &k_blind_rotate<8, false> : &k_blind_rotate<8, true>;
  hipLaunchKernelGGL(kern, dim3((unsigned)((B + 7) / 8)), dim3(512), br_lds_bytes(8, keytab == nullptr), st, bkf, ctx->ftab,
                     ops, abar, tlwe1, trlwe, B, keytab, kid);
  return hipGetLastError();
}

}  // namespace vsp
