// Latency form of the blind rotation: one gate per workgroup of three waves, wave k computing
// round k of every external product (gadget digit k+1 of both halves of X^a ACC - ACC, its
// forward transform and its key products). The partial sums meet in LDS: wave 0 inverts those of the
// K_hi products and wave 1 the packed ones, and both add into the accumulator. A step's critical path
// is one forward and one inverse transform and the exchange, instead of three and two.
// Results are bit-identical to the one-wave form (exact integer arithmetic).
#pragma once
#include "blind_rotate.h"

namespace vsp {

constexpr int BRW_WAVES = GADGET_L;  // one wave per gadget level
// LDS per gate: the accumulator (2N u32) and blocks of one product's sums (8 slot pairs x 64
// lanes): 0 the packed product of wave 0, 1-2 the K_hi products of wave 1, 3-5 all of wave 2. The
// waves' exchange regions lie in the same area.
constexpr int BRW_SUM_C64 = 8 * 64;
static_assert(BRW_WAVES * FFT_WAVE_F64 * 8 <= 6 * BRW_SUM_C64 * 16, "the exchange regions fit in the sum blocks");

constexpr size_t brw_lds_bytes() { return FFT_TAB_C64 * 16 + 2 * RING_N * 4 + 6 * BRW_SUM_C64 * 16; }

__device__ __forceinline__ void brw_put(const FftSum& sum, int q, c64* dst, int lane) {
#pragma unroll
  for (int p = 0; p < 8; p++) dst[p * 64 + lane] = make_double2(sum.r[q][p], sum.i[q][p]);
}
__device__ __forceinline__ void brw_add(FftSum& sum, int q, const c64* s0, const c64* s1, int lane) {
#pragma unroll
  for (int p = 0; p < 8; p++) {
    const c64 x = s0[p * 64 + lane], y = s1[p * 64 + lane];
    sum.r[q][p] += x.x + y.x;
    sum.i[q][p] += x.y + y.y;
  }
}

__global__ __launch_bounds__(BRW_WAVES * 64, 2) void k_blind_rotate_wide(const c64* __restrict__ bkf,
                                                                      const c64* __restrict__ tab,
                                                                      const uint8_t* __restrict__ ops,
                                                                      const u32* __restrict__ abar,
                                                                      u32* __restrict__ tlwe1, u32* __restrict__ trlwe,
                                                                      uint64_t B, const c64* const* __restrict__ keytab,
                                                                      const uint16_t* __restrict__ kid) {
  extern __shared__ c64 lds[];
  c64* tabs = lds;
  for (int i = threadIdx.x; i < FFT_TAB_C64; i += BRW_WAVES * 64) tabs[i] = tab[i];
  const uint64_t g = blockIdx.x;  // the grid has exactly B workgroups
  if (ops && !op_bootstraps(ops[g])) return;  // uniform over the workgroup: no barrier is skipped by half
  if (keytab) bkf = keytab[kid[g]];           // per-gate key (same value in every wave)
  const int k = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // this wave's digit level
  const int lane = threadIdx.x & 63, l = lane & 31, h = lane >> 5;
  c64* blocks = lds + FFT_TAB_C64;
  u32* acc = reinterpret_cast<u32*>(blocks + 6 * BRW_SUM_C64);
  double* reg = reinterpret_cast<double*>(blocks) + k * FFT_WAVE_F64 + h * FFT_REGION;
  u32* accs = acc + h * RING_N;
  const u32* ab = abar + g * TLWE0;
  if (k == 0) {
    const int bbar = (int)ab[LWE_N];
    const int k0 = (2 * RING_N - bbar) & (2 * RING_N - 1);
#pragma unroll
    for (int t = 0; t < 32; t++) accs[l + 32 * t] = h ? rotated_testvector(l + 32 * t, k0) : 0u;
  }
  __syncthreads();
  for (int i = 0; i < LWE_N; i++) {
    const int a = (int)__builtin_amdgcn_readfirstlane(ab[i]);
    if (a == 0) continue;  // same value in every wave of the workgroup
    double re[16], im[16];
    FftSum sum;
    sum.clear();
    const int lo = opaque_lane(l), bt = 4 * (lo - a);
#pragma unroll
    for (int t = 0; t < 16; t++) {
      re[t] = (double)((int)(rotated_word(accs, bt + 128 * t, accs[lo + 32 * t]) << (BG_BIT * k)) >> 26);
      im[t] = (double)((int)(rotated_word(accs, bt + 128 * t + 2048, accs[lo + 32 * t + 512]) << (BG_BIT * k)) >> 26);
    }
    fft_forward(re, im, tabs, reg, l);
    GlobalKey key;
    key.base = (gkey)bkf + (size_t)i * TRGSW_FFT_C64 + lane;
    fft_key_round(re, im, sum, k, key);
    __syncthreads();  // every wave is done with its exchange region and with ACC
    if (k == 0) {
      brw_put(sum, 2, blocks, lane);
    } else if (k == 1) {
      brw_put(sum, 0, blocks + BRW_SUM_C64, lane);
      brw_put(sum, 1, blocks + 2 * BRW_SUM_C64, lane);
    } else {
#pragma unroll
      for (int q = 0; q < FFT_PRODUCTS; q++) brw_put(sum, q, blocks + (3 + q) * BRW_SUM_C64, lane);
    }
    __syncthreads();
    if (k == 0) {
      brw_add(sum, 0, blocks + BRW_SUM_C64, blocks + 3 * BRW_SUM_C64, lane);
      brw_add(sum, 1, blocks + 2 * BRW_SUM_C64, blocks + 4 * BRW_SUM_C64, lane);
      fft_take_hi(sum, re, im);
    } else if (k == 1) {
      brw_add(sum, 2, blocks, blocks + 5 * BRW_SUM_C64, lane);
      fft_take_lo(sum, re, im);
    }
    __syncthreads();  // the sums are read: the area holds exchange regions again
    if (k < 2) {
      fft_inverse(re, im, tabs, reg, l);
#pragma unroll
      for (int t = 0; t < 32; t++) {
        const double v = t < 16 ? re[t & 15] : im[t & 15];
        const u32 z = k == 0 ? fft_round_u32(v) << FFT_LO_BITS : fft_combine(0u, v);
        __hip_atomic_fetch_add(&accs[l + 32 * t], z, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      }
    }
    __syncthreads();  // the updated ACC is visible to the next step's digits
  }
  if (k != 0) return;
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
