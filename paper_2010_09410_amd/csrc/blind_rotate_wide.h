// Latency forms: a chain of external products on one workgroup of eight waves, and the blind rotation
// of one gate by it. A step, ACC <- ACC + C_i (ext) D_i with D_i formed from ACC, is four phases between
// barriers:
//  1. all waves add the last step's small products into their four coefficients per thread of ACC and
//     form the digit words of D_i (the new ACC is stored in phase 2, when all have read it);
//  2. wave r < 6 transforms TRGSW row r's digits (gadget level r mod 3 + 1 of ACC polynomial r / 3);
//  3. wave w takes slot w of the transform, 64 values, and adds the six rows' products with the three
//     key polynomials;
//  4. waves 0-2 invert one of the three sums each; waves 0 and 1 add their K_hi product into ACC, wave 2
//     leaves the small products in LDS. No LDS atomics: 64 lanes of one take about 34 cycles.
// What bounds a step is the latency of that chain, about 9,600 cycles: 800, 3,300 (three LDS writes of
// 8 KiB by each of six waves, at 39 B/clk per pair of SIMDs, are 1,900 of it), 1,200 and 4,000. Each key
// entry is read once per gate, its load issued where it delays no one: in phase 4, by waves 3-7 while
// waves 0-2 invert and by those after they have stored their results (a wave's 18 KiB take 290 cycles
// to issue; among the products they delayed the sums, in the inverse transform the transform). Two
// variants:
//  - one gate per compute unit (PER_SIMD 2): a wave's whole share of the next step's key ahead (AHEAD 6);
//  - two gates per compute unit (PER_SIMD 4, 128 registers): one row of the key ahead (AHEAD 1), the two
//    workgroups fill each other's waits.
// Measured, 256 gates one per unit 2.62 ms, 512 gates two per unit 4.82; with three phases, each forward
// wave forming its own digit words, LDS atomics into ACC and the loads among the products 3.72 and 5.25.
// Results are bit-identical to the one-wave form (exact integer arithmetic).
#pragma once
#include "blind_rotate.h"

namespace vsp {

constexpr int BRW_WAVES = 8;
constexpr int BRW_ROWS = 2 * GADGET_L;
// LDS: a region per row (its exchanges, then its transform [slot][lane]; the inverse exchanges reuse
// the first three), the three sums [product][slot][lane] (before they are written, the digit words in
// the first one's place; after they are read, the small products in the last one's), the accumulator.
constexpr size_t brw_lds_bytes() {
  return (size_t)(BRW_ROWS + FFT_PRODUCTS) * FFT8_REGION_C64 * 16 + 2 * RING_N * 4;
}

// The chain, on ACC that the caller has put in LDS at brw_acc(lds) and reads there afterwards. `chain` says what a step is: chain.begin(i) stands at its start,
// chain.key(i) is TRGSW C_i, and chain.words(acc, small, p, j, own, word) takes coefficient j of
// polynomial p (at index p N + j of acc and of the small products still to be added) and gives the
// accumulator that stays (own) and the digit word of D_i.
__device__ __forceinline__ u32* brw_acc(c64* lds) {
  return reinterpret_cast<u32*>(lds + (BRW_ROWS + FFT_PRODUCTS) * FFT8_REGION_C64);
}
template <int AHEAD, int PER_SIMD, class Chain>
__device__ __forceinline__ void brw_chain(c64* lds, const c64* __restrict__ tab8, int steps, Chain& chain) {
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane0 = tid & 63;
  c64* sums = lds + BRW_ROWS * FFT8_REGION_C64;
  u32* acc = brw_acc(lds);
  u32* words = reinterpret_cast<u32*>(sums);                       // [2][N], in the first sum's place
  u32* small = reinterpret_cast<u32*>(sums + 2 * FFT8_REGION_C64);  // [2][N], in the packed sum's place
  c64* reg = lds + (wave < BRW_ROWS ? wave : 0) * FFT8_REGION_C64;
  Fft8Lane tab;
  tab.load(tab8, lane0);
  // wait for the table here: a wait left to its first use, inside the loop, would count the key
  // loads issued since and so wait for those in every step
  __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
  // this wave's slot of the key, row r = k + 3 e, product q: [k][slot][e][q][entry]. For the products
  // lane m takes entry m (contiguous loads); lane L of a transform owns entry fft_half_lane(L). Values
  // pass between the two by LDS places that spread both over all banks.
  auto place = [](int m) { return m ^ ((m >> 1) & 8) ^ ((m >> 3) & 4); };
  c64 key[AHEAD][FFT_PRODUCTS];
  auto load_rows = [&](int i, int r0, c64(&kv)[AHEAD][FFT_PRODUCTS]) {
    const gkey ks = chain.key(i) + wave * FFT_PIECE_C64 + lane0;
#pragma unroll
    for (int j = 0; j < AHEAD; j++)
#pragma unroll
      for (int q = 0; q < FFT_PRODUCTS; q++) {
        const int r = r0 + j;
        kv[j][q] = gkey_load(ks + (r % GADGET_L) * 8 * FFT_PIECE_C64 + (r / GADGET_L) * FFT_HALF_C64 + q * 64);
      }
  };
  load_rows(0, 0, key);
  for (int j = tid; j < 2 * RING_N; j += BRW_WAVES * 64) small[j] = 0u;
  __syncthreads();
  for (int i = 0; i < steps; i++) {
    chain.begin(i);
    double re[8], im[8];
    // with 128 registers the lane's LDS addresses are formed anew in every step instead of being kept
    const int lane = PER_SIMD > 2 ? opaque_lane(lane0) : lane0;
    const int pm = place(lane), pl = place(fft_half_lane(lane));
    u32 own[4];  // coefficients 512 q + tid of (a, b), polynomial q / 2: ACC with the last step's small products
#pragma unroll
    for (int q = 0; q < 4; q++) {
      const int p = (q >> 1) * RING_N, j = (q & 1) * (RING_N / 2) + wave * 64 + lane;
      chain.words(acc, small, p, j, own[q], words[p + j]);
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 4; q++) acc[q * (RING_N / 2) + wave * 64 + lane] = own[q];
    if (wave < BRW_ROWS) {
      const u32* w = words + (wave / GADGET_L) * RING_N + lane;
      const int up = BG_BIT * (wave % GADGET_L);
#pragma unroll
      for (int t = 0; t < 8; t++) {
        re[t] = (double)((int)(w[64 * t] << up) >> 26);
        im[t] = (double)((int)(w[64 * t + RING_N / 2] << up) >> 26);
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
        if (r0 + AHEAD < BRW_ROWS) load_rows(i, r0 + AHEAD, key);
      }
#pragma unroll
      for (int q = 0; q < FFT_PRODUCTS; q++)
        sums[q * FFT8_REGION_C64 + wave * 64 + pm] = make_double2(sr[q], si[q]);
    }
    __syncthreads();
    const int next = i + 1 < steps ? i + 1 : i;
    if (wave < FFT_PRODUCTS) {
      __builtin_amdgcn_s_setprio(3);  // the chain, against the other waves' loads
#pragma unroll
      for (int s = 0; s < 8; s++) {
        const c64 x = sums[wave * FFT8_REGION_C64 + s * 64 + pl];
        re[s] = x.x;
        im[s] = x.y;
      }
      fft8_inverse(re, im, tab, reg, lane);
      auto value = [&](int t) { return t < 8 ? re[t & 7] : im[t & 7]; };
      if (wave < 2) {
        u32* p = acc + wave * RING_N + lane;
        u32 old[16];
#pragma unroll
        for (int t = 0; t < 16; t++) old[t] = p[64 * t];
#pragma unroll
        for (int t = 0; t < 16; t++) p[64 * t] = old[t] + (fft_round_u32(value(t)) << FFT_LO_BITS);
      } else {
#pragma unroll
        for (int t = 0; t < 16; t++) {
          u32 x, y;
          fft_unpack(value(t), x, y);
          small[lane + 64 * t] = x;
          small[RING_N + lane + 64 * t] = y;
        }
      }
      __builtin_amdgcn_sched_barrier(0);
      if (AHEAD > 1) load_rows(next, 0, key);
    } else if (AHEAD > 1) {
      load_rows(next, 0, key);
    }
    __builtin_amdgcn_s_setprio(0);
    if (AHEAD == 1) load_rows(next, 0, key);
    __syncthreads();
  }
  for (int j = tid; j < 2 * RING_N; j += BRW_WAVES * 64) acc[j] += small[j];
  __syncthreads();
}

// D = X^a ACC - ACC: a step of a blind rotation.
__device__ __forceinline__ void brw_rotated(const u32* acc, const u32* small, int p, int j, int a, u32& own, u32& word) {
  own = acc[p + j] + small[p + j];
  const int r = j - a, at = p + (r & (RING_N - 1));
  const u32 v = acc[at] + small[at];
  word = digit_word((r & RING_N ? 0u - v : v) - own);
}

struct BlindChain {
  const u32* ab;
  gkey keys;
  int a, next;
  __device__ __forceinline__ void start() { next = (int)__builtin_amdgcn_readfirstlane(ab[0]); }
  __device__ __forceinline__ void begin(int i) {
    a = next;
    next = (int)__builtin_amdgcn_readfirstlane(ab[i + 1]);  // (the last one is b)
  }
  __device__ __forceinline__ gkey key(int i) const { return keys + (size_t)i * TRGSW_FFT_C64; }
  __device__ __forceinline__ void words(const u32* acc, const u32* small, int p, int j, u32& own, u32& word) const {
    brw_rotated(acc, small, p, j, a, own, word);
  }
};

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
  const int tid = threadIdx.x;
  u32* acc = brw_acc(lds);
  BlindChain chain;
  chain.ab = abar + g * TLWE0;
  chain.keys = (gkey)bkf;
  chain.start();
  {
    const int k0 = (2 * RING_N - (int)chain.ab[LWE_N]) & (2 * RING_N - 1);
    for (int j = tid; j < 2 * RING_N; j += BRW_WAVES * 64) acc[j] = j < RING_N ? 0u : rotated_testvector(j - RING_N, k0);
  }
  brw_chain<AHEAD, PER_SIMD>(lds, tab8, LWE_N, chain);
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
