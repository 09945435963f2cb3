// Blind-rotation kernel (device code only; its launcher lives with the other launchers).
// Kept in a file of its own so that its source fingerprint names exactly the code a
// profile of it measured.
#pragma once
#include "fft.h"
#include "vsp_internal.h"

namespace vsp {

// One wave per gate. The accumulator lives in LDS (its a polynomial for lanes 0-31, b for
// lanes 32-63; coefficient l + 32 t belongs to lane l). ACC starts as (0, X^{-bbar} tv) with
// tv = mu everywhere; step i adds BK_i (ext) (X^{abar_i} ACC - ACC) (a CMUX between ACC and
// its rotation selected by the key bit s0_i); a step with abar_i = 0 has a zero difference,
// hence a zero product, and is skipped. LDS per workgroup: the lane tables, then per wave
// the accumulator (2 x 1024 u32) and the two exchange regions.
constexpr int BR_WAVE_U32 = 2 * RING_N + 2 * FFT_WAVE_F64;

constexpr size_t br_lds_bytes(int waves, bool shared) {
  return FFT_TAB_C64 * 16 + (shared ? 2 * FFT_PIECE_C64 * 16 : 0) + (size_t)waves * BR_WAVE_U32 * 4;
}

// What bounds it is VALU issue, 75% busy: 3,944 instructions a wave and step, 2,784 of them float64, with
// the two waves a SIMD that 256 registers and 17 KiB of LDS per gate allow; LDS is 42% busy, barriers and
// key stream cost 6%. 2,048 gates, one round, take 12.2 ms (12.5 with LDS atomics into ACC and its
// words read again in the next step); the transform modulo a 64-bit prime took 54, the int8 matrix
// products 41.
// SHARED: every gate uses the key bkf, which the workgroup streams through LDS; its waves meet at
// every piece, so a wave without a gate takes part as well (on a zero accumulator). A workgroup none of
// whose gates bootstraps ends before its first barrier (2,048 NOT gates 0.19 ms with their other launches,
// 12.1 with a pass over the key), by the instruction itself: a return there changed the order of the
// instructions of the steps for the worse (2,048 gates 12.21 ms instead of 12.14). Otherwise gate g reads
// the key keytab[kid[g]] by itself (clients with their own keys in one launch), or bkf with keytab NULL,
// and steps whose difference is zero are skipped.
template <int WAVES, bool SHARED>
__global__ __launch_bounds__(WAVES * 64) void k_blind_rotate(const c64* __restrict__ bkf, const c64* __restrict__ tab,
                                                             const uint8_t* __restrict__ ops,
                                                             const u32* __restrict__ abar, u32* __restrict__ tlwe1,
                                                             u32* __restrict__ trlwe, uint64_t B,
                                                             const c64* const* __restrict__ keytab,
                                                             const uint16_t* __restrict__ kid) {
  extern __shared__ c64 lds[];
  c64* tabs = lds;
  c64* ring = lds + FFT_TAB_C64;
  for (int i = threadIdx.x; i < FFT_TAB_C64; i += WAVES * 64) tabs[i] = tab[i];
  SharedKey<WAVES, false> shared;
  if (SHARED) shared.start((gkey)bkf, ring, LWE_N * FFT_PIECES);
  if (SHARED && ops) {  // the same answer in every wave, so no barrier is met by some only
    const uint64_t i = (uint64_t)blockIdx.x * WAVES + threadIdx.x % WAVES;
    if (__ballot(op_bootstraps(ops[i < B ? i : B - 1])) == 0) __builtin_amdgcn_endpgm();
  }
  __syncthreads();
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint64_t g = (uint64_t)blockIdx.x * WAVES + wave;
  const bool live = g < B && (!ops || op_bootstraps(ops[g]));
  if (!SHARED && !live) return;
  if (!SHARED && keytab) bkf = keytab[__builtin_amdgcn_readfirstlane(kid[g])];
  const int lane = threadIdx.x & 63, l = lane & 31, h = lane >> 5;
  u32* wbase = reinterpret_cast<u32*>(ring + (SHARED ? 2 * FFT_PIECE_C64 : 0)) + wave * BR_WAVE_U32;
  const u32* ab = abar + (live ? g : 0) * TLWE0;
  {
    const int k0 = (2 * RING_N - (int)ab[LWE_N]) & (2 * RING_N - 1);
    u32* accs = wbase + h * RING_N;
#pragma unroll
    for (int t = 0; t < 32; t++) accs[l + 32 * t] = (h && live) ? rotated_testvector(l + 32 * t, k0) : 0u;
  }
  wave_lds_sync();
  u32 own[32];  // the lane's coefficients of ACC, from the end of a step to the start of the next
#pragma unroll
  for (int t = 0; t < 32; t++) own[t] = wbase[h * RING_N + l + 32 * t];
  for (int i = 0; i < LWE_N; i++) {
    const int a = (int)__builtin_amdgcn_readfirstlane(ab[i]);
    if (!SHARED && a == 0) continue;
    const int ln = opaque_lane(lane);
    const int li = ln & 31, hi = ln >> 5;
    u32* accs = wbase + hi * RING_N;
    double* reg = reinterpret_cast<double*>(wbase + 2 * RING_N) + hi * FFT_REGION;
    const int bt = 4 * (li - a);
    auto word = [&](int t) { return rotated_word(accs, bt + 128 * t, own[t]); };
    u32 z[32];
    if constexpr (SHARED) {
      fft_external_product(word, shared, tabs, reg, ln, z);
    } else {
      GlobalKey key;
      key.base = (gkey)bkf + (size_t)i * TRGSW_FFT_C64 + ln;
      fft_external_product(word, key, tabs, reg, ln, z);
    }
#pragma unroll
    for (int t = 0; t < 32; t++) own[t] = accs[li + 32 * t];
#pragma unroll
    for (int t = 0; t < 32; t++) accs[li + 32 * t] = own[t] += z[t];
    wave_lds_sync();
  }
  if (!live) return;
  const u32* accs = wbase + h * RING_N;
  if (trlwe) {
    u32* o = trlwe + g * 2 * RING_N + h * RING_N;
#pragma unroll
    for (int t = 0; t < 32; t++) o[l + 32 * t] = accs[l + 32 * t];
  }
  if (tlwe1) {
    // SampleExtract at 0: a'_0 = A_0, a'_j = -A_{N-j}; b' = B_0.
    u32* o = tlwe1 + g * TLWE1;
    if (h == 0) {
#pragma unroll
      for (int t = 0; t < 32; t++) {
        const int j = l + 32 * t;
        const u32 v = accs[j];
        o[(RING_N - j) & (RING_N - 1)] = (j == 0) ? v : 0u - v;
      }
    } else if (l == 0) {
      o[RING_N] = accs[0];
    }
  }
}

}  // namespace vsp
