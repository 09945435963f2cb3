// Latency forms of the blind rotation: one gate per workgroup of eight waves. Per step, waves 0-5 form
// and transform one TRGSW row's digits each (row r: gadget level r mod 3 + 1 of ACC polynomial r / 3);
// then wave w takes slot w of the transform, 64 values, and adds the six rows' products with the
// three key polynomials; then waves 0-2 invert the three sums and add into the accumulator. A
// step's critical path is one digit row, one forward and one inverse transform over whole waves and
// three barriers; what bounds it is the latency of that chain (LDS exchanges, dependent
// multiply-adds). Two variants:
//  - one gate per compute unit (PER_SIMD 2): the wave's share of the next step's key (18 KiB) is loaded
//    whole while the step goes on (AHEAD 6): 256 gates 3.6 ms;
//  - two gates per compute unit (PER_SIMD 4, 128 registers): one row of the key ahead (AHEAD 1), the two
//    workgroups fill each other's waits: 512 gates 4.9 ms, against 7.0 ms in two rounds of the first.
// Each key entry is read once per gate. Results are bit-identical to the one-wave form (exact integer
// arithmetic).
#pragma once
#include "blind_rotate.h"

namespace vsp {

constexpr int BRW_WAVES = 8;
constexpr int BRW_ROWS = 2 * GADGET_L;
// LDS: a region per row (its exchanges, then its transform [slot][lane]; the inverse exchanges reuse
// the first three), the three sums [product][slot][lane], the accumulator.
constexpr size_t brw_lds_bytes() {
  return (size_t)(BRW_ROWS + FFT_PRODUCTS) * FFT8_REGION_C64 * 16 + 2 * RING_N * 4;
}

template <int AHEAD, int PER_SIMD>
__global__ __launch_bounds__(BRW_WAVES * 64, PER_SIMD) void k_blind_rotate_wide(const c64* __restrict__ bkf,
                                                                      const c64* __restrict__ tab8,
                                                                      const uint8_t* __restrict__ ops,
                                                                      const u32* __restrict__ abar,
                                                                      u32* __restrict__ tlwe1, u32* __restrict__ trlwe,
                                                                      uint64_t B, const c64* const* __restrict__ keytab,
                                                                      const uint16_t* __restrict__ kid) {
  extern __shared__ c64 lds[];
  const uint64_t g = blockIdx.x;  // the grid has exactly B workgroups
  if (ops && !op_bootstraps(ops[g])) return;  // uniform over the workgroup: no barrier is skipped by half
  if (keytab) bkf = keytab[kid[g]];           // per-gate key (same value in every wave)
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane0 = tid & 63;
  c64* sums = lds + BRW_ROWS * FFT8_REGION_C64;
  u32* acc = reinterpret_cast<u32*>(sums + FFT_PRODUCTS * FFT8_REGION_C64);
  c64* reg = lds + (wave < BRW_ROWS ? wave : 0) * FFT8_REGION_C64;
  const u32* ab = abar + g * TLWE0;
  Fft8Lane tab;
  tab.load(tab8, lane0);
  // wait for the table here: a wait left to its first use, inside the loop, would count the key
  // loads issued since and so wait for those in every step
  __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
  // this wave's slot of the key, row r = k + 3 e, product q: [k][slot][e][q][entry]. For the products
  // lane m takes entry m (contiguous loads); lane L of a transform owns entry fft_half_lane(L). Values
  // pass between the two by LDS places that spread both over all banks.
  const gkey key0 = (gkey)bkf + wave * FFT_PIECE_C64 + lane0;
  auto place = [](int m) { return m ^ ((m >> 1) & 8) ^ ((m >> 3) & 4); };
  c64 key[AHEAD][FFT_PRODUCTS];
  auto load_rows = [&](int i, int r0, c64(&kv)[AHEAD][FFT_PRODUCTS]) {
    const gkey ks = key0 + (size_t)i * TRGSW_FFT_C64;
#pragma unroll
    for (int j = 0; j < AHEAD; j++)
#pragma unroll
      for (int q = 0; q < FFT_PRODUCTS; q++) {
        const int r = r0 + j;
        kv[j][q] = gkey_load(ks + (r % GADGET_L) * 8 * FFT_PIECE_C64 + (r / GADGET_L) * FFT_HALF_C64 + q * 64);
      }
  };
  load_rows(0, 0, key);
  {
    const int k0 = (2 * RING_N - (int)ab[LWE_N]) & (2 * RING_N - 1);
    for (int j = tid; j < 2 * RING_N; j += BRW_WAVES * 64) acc[j] = j < RING_N ? 0u : rotated_testvector(j - RING_N, k0);
  }
  int a_next = (int)__builtin_amdgcn_readfirstlane(ab[0]);
  __syncthreads();
  for (int i = 0; i < LWE_N; i++) {
    const int a = a_next;
    a_next = (int)__builtin_amdgcn_readfirstlane(ab[i + 1]);  // (the last one is b)
    double re[8], im[8];
    // with two workgroups on a compute unit (PER_SIMD 4, 128 registers) the lane's LDS addresses are
    // formed anew in every step instead of being kept
    const int lane = PER_SIMD > 2 ? opaque_lane(lane0) : lane0;
    const int pm = place(lane), pl = place(fft_half_lane(lane));
    if (wave < BRW_ROWS) {
      const u32* accs = acc + (wave / GADGET_L) * RING_N;
      const int up = BG_BIT * (wave % GADGET_L);
#pragma unroll
      for (int t = 0; t < 8; t++) {
        const int j = lane + 64 * t;
        re[t] = (double)((int)(rotated_word(accs, 4 * (j - a), accs[j]) << up) >> 26);
        im[t] = (double)((int)(rotated_word(accs, 4 * (j - a) + 2 * RING_N, accs[j + RING_N / 2]) << up) >> 26);
      }
      fft8_forward(re, im, tab, reg, lane);
#pragma unroll
      for (int s = 0; s < 8; s++) reg[s * 64 + pl] = make_double2(re[s], im[s]);
    }
    __syncthreads();
    {
      double sr[FFT_PRODUCTS] = {}, si[FFT_PRODUCTS] = {};
#pragma unroll
      for (int r0 = 0; r0 < BRW_ROWS; r0 += AHEAD) {
#pragma unroll
        for (int j = 0; j < AHEAD; j++) {
          const c64 x = lds[(r0 + j) * FFT8_REGION_C64 + wave * 64 + pm];
#pragma unroll
          for (int q = 0; q < FFT_PRODUCTS; q++) fft_cmac(sr[q], si[q], x.x, x.y, key[j][q]);
        }
        if (r0 + AHEAD < BRW_ROWS)
          load_rows(i, r0 + AHEAD, key);
        else
          load_rows(i + 1 < LWE_N ? i + 1 : i, 0, key);
      }
#pragma unroll
      for (int q = 0; q < FFT_PRODUCTS; q++)
        sums[q * FFT8_REGION_C64 + wave * 64 + pm] = make_double2(sr[q], si[q]);
    }
    __syncthreads();
    if (wave < FFT_PRODUCTS) {
#pragma unroll
      for (int s = 0; s < 8; s++) {
        const c64 x = sums[wave * FFT8_REGION_C64 + s * 64 + pl];
        re[s] = x.x;
        im[s] = x.y;
      }
      fft8_inverse(re, im, tab, reg, lane);
#pragma unroll
      for (int t = 0; t < 16; t++) {
        const double v = t < 8 ? re[t & 7] : im[t & 7];
        u32* p = acc + lane + 64 * t;
        if (wave < 2) {
          __hip_atomic_fetch_add(p + wave * RING_N, fft_round_u32(v) << FFT_LO_BITS, __ATOMIC_RELAXED,
                                 __HIP_MEMORY_SCOPE_WORKGROUP);
        } else {
          u32 x, y;
          fft_unpack(v, x, y);
          __hip_atomic_fetch_add(p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
          __hip_atomic_fetch_add(p + RING_N, y, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
      }
    }
    __syncthreads();
  }
  if (trlwe) {
    for (int j = tid; j < 2 * RING_N; j += BRW_WAVES * 64) trlwe[g * 2 * RING_N + j] = acc[j];
  }
  if (tlwe1) {  // SampleExtract at 0: a'_0 = A_0, a'_j = -A_{N-j}; b' = B_0
    u32* o = tlwe1 + g * TLWE1;
    for (int j = tid; j < RING_N; j += BRW_WAVES * 64) o[j] = j == 0 ? acc[0] : 0u - acc[RING_N - j];
    if (tid == 0) o[RING_N] = acc[RING_N];
  }
}

}  // namespace vsp
