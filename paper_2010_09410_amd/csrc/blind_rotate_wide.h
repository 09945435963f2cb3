// Latency forms: chains of external products on a workgroup of eight waves, one or two (G) chains with the
// same TRGSWs at a time, and the blind rotation of one or two gates by it. A step,
// ACC <- ACC + C_i (ext) D_i with D_i formed from ACC, is four phases between barriers:
//  1. all waves add the last step's small products into their four coefficients per thread of ACC and
//     form the digit words of D_i (the new ACC is stored in phase 2, when all have read it);
//  2. wave r < 6 transforms TRGSW row r's digits (gadget level r mod 3 + 1 of ACC polynomial r / 3); with
//     two chains, wave r rows r and r + 8 of the twelve;
//  3. wave w takes slot w of the transform, 64 values, and adds the six rows' products with the three
//     key polynomials;
//  4. a wave per sum inverts it; those of the K_hi products add it into ACC, the others leave the small
//     products in LDS. No LDS atomics: 64 lanes of one take about 34 cycles.
// What bounds a step is the latency of that chain, for one gate about 9,000 cycles: phases of 800, 3,300
// (three LDS writes of 8 KiB by each of six waves, at 39 B/clk per pair of SIMDs, are 1,900 of it), 1,200 and
// 4,000, a little more with the clock reads that told them apart; VALU issue is 41% busy, LDS 44%. For two
// gates 15,200 cycles, 58% and 44%. A wave's whole share of the next step's key is loaded where that delays no one: in
// phase 4, by the waves without a sum while the others invert, and by those after they have stored their
// results (its 18 KiB take 290 cycles to issue; among the products they delayed the sums, in the inverse
// transform the transform). With two gates LDS is the bound of phase 2 and the first exchange of the
// forward transforms goes through the VALU (512 gates 4.04 ms instead of 4.34); with one gate that
// is the longer way (256 gates 2.47 instead of 2.38).
// Measured: 256 gates one per unit 2.38 ms; with three phases, each forward wave forming its own digit
// words, LDS atomics into ACC and the loads among the products 3.72. 512 gates two per workgroup 4.04; as
// two workgroups of one gate per unit, with 128 registers and a row of the key ahead, 4.64.
// Results are bit-identical to the one-wave form (exact integer arithmetic).
#pragma once
#include "blind_rotate.h"

namespace vsp {

constexpr int BRW_WAVES = 8;
constexpr int BRW_ROWS = 2 * GADGET_L;
// LDS per chain: a region per row (its exchanges, then its transform [slot][lane]; the inverse exchanges
// reuse those of the first rows), the three sums [product][slot][lane] (before they are written, the
// digit words in the first one's place; after they are read, the small products in the last one's), the
// accumulator: 80 KiB.
constexpr size_t brw_lds_bytes(int gates) {
  return gates * ((size_t)(BRW_ROWS + FFT_PRODUCTS) * FFT8_REGION_C64 * 16 + 2 * RING_N * 4);
}

// The chains, on the G accumulators that the caller has put in LDS at brw_acc(lds, g) and reads there
// afterwards. `chain` says what a step is: chain.begin(i) stands at its start, chain.key(i) is TRGSW C_i,
// and chain.words(g, acc, small, p, j, own, word) takes coefficient j of polynomial p of chain g (at
// index p + j, p = 0 or N, of acc and of the small products still to be added) and gives the
// accumulator that stays (own) and the digit word of D_i.
template <int G>
__device__ __forceinline__ u32* brw_acc(c64* lds, int g) {
  return reinterpret_cast<u32*>(lds + G * (BRW_ROWS + FFT_PRODUCTS) * FFT8_REGION_C64) + g * 2 * RING_N;
}
template <int G, class Chain>
__device__ __forceinline__ void brw_chain(c64* lds, const c64* __restrict__ tab8, int steps, Chain& chain) {
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  c64* sums = lds + G * BRW_ROWS * FFT8_REGION_C64;              // [gate][product]
  auto acc = [&](int g) { return brw_acc<G>(lds, g); };
  auto words = [&](int g) { return reinterpret_cast<u32*>(sums + g * FFT_PRODUCTS * FFT8_REGION_C64); };
  auto small = [&](int g) { return reinterpret_cast<u32*>(sums + (g * FFT_PRODUCTS + 2) * FFT8_REGION_C64); };
  Fft8Lane tab;
  tab.load(tab8, lane);
  // wait for the table here: a wait left to its first use, inside the loop, would count the key
  // loads issued since and so wait for those in every step
  __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
  // this wave's slot of the key, row r = k + 3 e, product q: [k][slot][e][q][entry]. For the products
  // lane m takes entry m (contiguous loads); lane L of a transform owns entry fft_half_lane(L). Values
  // pass between the two by LDS places that spread both over all banks.
  auto place = [](int m) { return m ^ ((m >> 1) & 8) ^ ((m >> 3) & 4); };
  c64 key[BRW_ROWS][FFT_PRODUCTS];
  auto load_key = [&](int i) {
    const gkey ks = chain.key(i) + wave * FFT_PIECE_C64 + lane;
#pragma unroll
    for (int r = 0; r < BRW_ROWS; r++)
#pragma unroll
      for (int q = 0; q < FFT_PRODUCTS; q++)
        key[r][q] = gkey_load(ks + (r % GADGET_L) * 8 * FFT_PIECE_C64 + (r / GADGET_L) * FFT_HALF_C64 + q * 64);
  };
  load_key(0);
#pragma unroll
  for (int g = 0; g < G; g++)
    for (int j = tid; j < 2 * RING_N; j += BRW_WAVES * 64) small(g)[j] = 0u;
  __syncthreads();
  const int pm = place(lane), pl = place(fft_half_lane(lane));
  for (int i = 0; i < steps; i++) {
    chain.begin(i);
    double re[8], im[8];
    u32 own[G][4];  // coefficients 512 q + tid of (a, b), polynomial q / 2: ACC with the last step's small products
#pragma unroll
    for (int g = 0; g < G; g++)
#pragma unroll
      for (int q = 0; q < 4; q++) {
        const int p = (q >> 1) * RING_N, j = (q & 1) * (RING_N / 2) + tid;
        chain.words(g, acc(g), small(g), p, j, own[g][q], words(g)[p + j]);
      }
    __syncthreads();
#pragma unroll
    for (int g = 0; g < G; g++)
#pragma unroll
      for (int q = 0; q < 4; q++) acc(g)[q * (RING_N / 2) + tid] = own[g][q];
#pragma unroll 1
    for (int r = wave; r < G * BRW_ROWS; r += BRW_WAVES) {
      const int g = r / BRW_ROWS, row = r % BRW_ROWS;
      const u32* w = words(g) + (row / GADGET_L) * RING_N + lane;
      const int up = BG_BIT * (row % GADGET_L);
      c64* reg = lds + r * FFT8_REGION_C64;
#pragma unroll
      for (int t = 0; t < 8; t++) {
        re[t] = (double)((int)(w[64 * t] << up) >> 26);
        im[t] = (double)((int)(w[64 * t + RING_N / 2] << up) >> 26);
      }
      fft8_forward<G == 1>(re, im, tab, reg, lane);
#pragma unroll
      for (int s = 0; s < 8; s++) reg[s * 64 + pl] = make_double2(re[s], im[s]);
    }
    __syncthreads();
#pragma unroll
    for (int g = 0; g < G; g++) {
      double sr[FFT_PRODUCTS] = {}, si[FFT_PRODUCTS] = {};
#pragma unroll
      for (int r = 0; r < BRW_ROWS; r++) {
        const c64 x = lds[(g * BRW_ROWS + r) * FFT8_REGION_C64 + wave * 64 + pm];
#pragma unroll
        for (int q = 0; q < FFT_PRODUCTS; q++) fft_cmac(sr[q], si[q], x.x, x.y, key[r][q]);
      }
#pragma unroll
      for (int q = 0; q < FFT_PRODUCTS; q++)
        sums[(g * FFT_PRODUCTS + q) * FFT8_REGION_C64 + wave * 64 + pm] = make_double2(sr[q], si[q]);
    }
    __syncthreads();
    if (wave < G * FFT_PRODUCTS) {
      __builtin_amdgcn_s_setprio(3);  // the chain, against the other waves' loads
      const int g = wave / FFT_PRODUCTS, q = wave % FFT_PRODUCTS;
#pragma unroll
      for (int s = 0; s < 8; s++) {
        const c64 x = sums[wave * FFT8_REGION_C64 + s * 64 + pl];
        re[s] = x.x;
        im[s] = x.y;
      }
      fft8_inverse(re, im, tab, lds + wave * FFT8_REGION_C64, lane);
      auto value = [&](int t) { return t < 8 ? re[t & 7] : im[t & 7]; };
      if (q < 2) {
        u32* p = acc(g) + q * RING_N + lane;
        u32 old[16];
#pragma unroll
        for (int t = 0; t < 16; t++) old[t] = p[64 * t];
#pragma unroll
        for (int t = 0; t < 16; t++) p[64 * t] = old[t] + (fft_round_u32(value(t)) << FFT_LO_BITS);
      } else {
        u32* p = small(g) + lane;
#pragma unroll
        for (int t = 0; t < 16; t++) {
          u32 x, y;
          fft_unpack(value(t), x, y);
          p[64 * t] = x;
          p[RING_N + 64 * t] = y;
        }
      }
      __builtin_amdgcn_sched_barrier(0);
      load_key(i + 1 < steps ? i + 1 : i);
      __builtin_amdgcn_s_setprio(0);
    } else {
      load_key(i + 1 < steps ? i + 1 : i);
    }
    __syncthreads();
  }
#pragma unroll
  for (int g = 0; g < G; g++)
    for (int j = tid; j < 2 * RING_N; j += BRW_WAVES * 64) acc(g)[j] += small(g)[j];
  __syncthreads();
}

// D = X^a ACC - ACC: a step of a blind rotation.
__device__ __forceinline__ void brw_rotated(const u32* acc, const u32* small, int p, int j, int a, u32& own, u32& word) {
  own = acc[p + j] + small[p + j];
  const int r = j - a, at = p + (r & (RING_N - 1));
  const u32 v = acc[at] + small[at];
  word = digit_word((r & RING_N ? 0u - v : v) - own);
}

template <int G>
struct BlindChain {
  const u32* ab[G];
  gkey keys;
  int a[G], next[G];
  __device__ __forceinline__ void start() {
#pragma unroll
    for (int g = 0; g < G; g++) next[g] = (int)__builtin_amdgcn_readfirstlane(ab[g][0]);
  }
  __device__ __forceinline__ void begin(int i) {
#pragma unroll
    for (int g = 0; g < G; g++) {
      a[g] = next[g];
      next[g] = (int)__builtin_amdgcn_readfirstlane(ab[g][i + 1]);  // (the last one is b)
    }
  }
  __device__ __forceinline__ gkey key(int i) const { return keys + (size_t)i * TRGSW_FFT_C64; }
  __device__ __forceinline__ void words(int g, const u32* acc, const u32* small, int p, int j, u32& own, u32& word) const {
    brw_rotated(acc, small, p, j, a[g], own, word);
  }
};

// Workgroup x rotates the gates G x .. G x + G - 1 (one past the batch repeats the last one, unused). Per-gate
// keys (keytab) take G = 1.
template <int G>
__global__ __launch_bounds__(BRW_WAVES * 64, 2) void k_blind_rotate_wide(const c64* __restrict__ bkf, const c64* __restrict__ tab8,
                                                                 const uint8_t* __restrict__ ops,
                                                                 const u32* __restrict__ abar, u32* __restrict__ tlwe1,
                                                                 u32* __restrict__ trlwe, uint64_t B,
                                                                 const c64* const* __restrict__ keytab,
                                                                 const uint16_t* __restrict__ kid) {
  extern __shared__ c64 lds[];
  const uint64_t g0 = (uint64_t)blockIdx.x * G;
  bool live[G], any = false;  // uniform over the workgroup: no barrier is skipped by half
#pragma unroll
  for (int g = 0; g < G; g++) {
    live[g] = g0 + g < B && (!ops || op_bootstraps(ops[g0 + g]));
    any = any || live[g];
  }
  if (!any) return;
  if (G == 1 && keytab) bkf = keytab[kid[g0]];  // per-gate key (same value in every wave)
  const int tid = threadIdx.x;
  BlindChain<G> chain;
  chain.keys = (gkey)bkf;
#pragma unroll
  for (int g = 0; g < G; g++) {
    chain.ab[g] = abar + (g0 + g < B ? g0 + g : B - 1) * TLWE0;
    const int k0 = (2 * RING_N - (int)chain.ab[g][LWE_N]) & (2 * RING_N - 1);
    u32* acc = brw_acc<G>(lds, g);
    for (int j = tid; j < 2 * RING_N; j += BRW_WAVES * 64) acc[j] = j < RING_N ? 0u : rotated_testvector(j - RING_N, k0);
  }
  chain.start();
  brw_chain<G>(lds, tab8, LWE_N, chain);
#pragma unroll
  for (int g = 0; g < G; g++) {
    if (!live[g]) continue;
    const u32* acc = brw_acc<G>(lds, g);
    if (trlwe) {
      for (int j = tid; j < 2 * RING_N; j += BRW_WAVES * 64) trlwe[(g0 + g) * 2 * RING_N + j] = acc[j];
    }
    if (tlwe1) {  // SampleExtract at 0: a'_0 = A_0, a'_j = -A_{N-j}; b' = B_0
      u32* o = tlwe1 + (g0 + g) * TLWE1;
      for (int j = tid; j < RING_N; j += BRW_WAVES * 64) o[j] = j == 0 ? acc[0] : 0u - acc[RING_N - j];
      if (tid == 0) o[RING_N] = acc[RING_N];
    }
  }
}

}  // namespace vsp
