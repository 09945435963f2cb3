// Circuit bootstrapping on the GPU (Sec. 2.1.2 "Circuit Bootstrapping"; the CMUX memory needs
// it for its address bits, Sec. 8.2, and the paper's GPU library lacked it because its moduli
// exceed 64 bits, Sec. 6.2(a)). A level-0 TLWE of a bit becomes a level-1 TRGSW (l x 2^6
// gadget): for each gadget level j = 1..l, a level-2 blind rotation over the 2^64 torus
// (degree N2 = 2048, gadget l2 = 4 x 2^9) with the test vector 1/(2 Bg^j), SampleExtract at 0
// plus 1/(2 Bg^j), then two private functional key switches to level-1 TRLWE (x -> -s1 x and
// x -> x) that give TRGSW rows j-1 and l+j-1.
//
// Level-2 products. A product d(X) K(X) in Z[X]/(X^2048 + 1) with gadget digits |d| <= 2^8 and 64-bit
// torus key words runs through the complex transform of fft.h, folded to C[X]/(X^1024 - i): the key
// is split into three signed limbs, K = K_0 + 2^22 K_1 + 2^44 K_2 (mod 2^64, |K_b| <= 2^21), and every
// limb's product is rounded to the nearest integer. Ten splittings leave a transform within 46 u of
// its norm (u = 2^-53; 52 u with the turned constants below), for the digits and for the key. The products
// of a slot, 16 fused operations per part, add 16 sqrt(2) = 22.6 u of the sum of their magnitudes, and the ten
// joinings 43 u. So the error of a coefficient is at most 170 u x 8 rows x 2^8 sqrt(2048) x 2^21 sqrt(2048) = 0.17
// before rounding: the integers are exact (below 2^43) and the torus words the schoolbook ones.
#include <algorithm>
#include <vector>

#include "onehot_mfma.h"

namespace vsp {

constexpr int CB_N2 = 2048;
constexpr int CB_L2 = 4;
constexpr int CB_BG2 = 9;
constexpr int CB_ROWS = 2 * CB_L2;       // level-2 TRGSW rows
constexpr int CB_T = 12;                 // private key-switch digits
constexpr int CB_BB = 2;                 // private key-switch base bits
constexpr int CB_TLWE2 = CB_N2 + 1;
constexpr int CB_LIMBS = 3;
constexpr int CB_LIMB_BITS = 22;
constexpr int CB_PRODUCTS = 2 * CB_LIMBS;  // output o, limb b: product 3 o + b
constexpr int CB_WAVES = 8;                // waves per job
// Transformed key in complex numbers, in the order the waves read it: [step][wave w][row][product]
// [slot 2 w, 2 w + 1][lane].
constexpr size_t CB_KEY_ROW = (size_t)CB_PRODUCTS * 2 * 64;
constexpr size_t CB_KEY_STEP = (size_t)CB_WAVES * CB_ROWS * CB_KEY_ROW;
// Private key-switching keys: [u][k <= N2][p < t][v - 1 < 3][2][N] u32.
constexpr size_t CB_PKS_ROW = (size_t)2 * RING_N;
constexpr size_t CB_PKS_U = (size_t)CB_TLWE2 * CB_T * 3 * CB_PKS_ROW;
// Rounding offset of the level-2 gadget decomposition: sum_r (Bg2/2) 2^(64 - 9r) + 2^(64 - 36 - 1).
constexpr u64 cb_decomp_offset() {
  u64 o = 0;
  for (int r = 1; r <= CB_L2; r++) o += (u64)(1u << (CB_BG2 - 1)) << (64 - CB_BG2 * r);
  return o + (1ull << (64 - CB_BG2 * CB_L2 - 1));
}
constexpr u64 CB_DECOMP_OFFSET = cb_decomp_offset();
constexpr u64 CB_DIGIT_FLIP = (1ull << 63) | (1ull << 54) | (1ull << 45) | (1ull << 36);
static_assert(CB_BG2 == 9 && CB_L2 == 4, "digit fields at bits 63, 54, 45 and 36");

// ------------------------------------------------------------------ transform of degree 2048
// One polynomial per wave: lane L holds the complex coefficients L + 64 t (t = 0..15). With Z = X^64 four
// splittings of Z^16 - i (the constants of fft.h), with Y = X^4 four of Y^16 - z_u, then two of X^4 - z_{u,u'}.
// The exchanges give lane 4 u + v the coefficients v + 4 s of residue u, then lane 4 u + v the four residues
// (u, 4 v + k), four coefficients each, through 16 KiB of LDS in words of one complex number, placed
// so that the sixteen lanes of an access phase hit all banks.
constexpr int CB_TAB = 8;                  // lane table, see CbTab
constexpr int CB_REGION_C64 = 1024;

// A lane's constants. Those of pass 2 at the angles a/2, a/4, a/8, a/16 (a the angle of z_u); the others
// of its eight are the last two turned by 1/8 (and 1/16) of a turn. The residues 4 v + k of pass 3,
// k = 2 b + c, have the angles n/4 + b/4 + c/2 for the angle n of their common node, and so use
// n/8 + b/8 (+ c/4, a factor i) and n/16 + b/16 + c/8: entries 4 + b and 6 + b, the latter turned for
// c = 1. Turning costs four operations where it is used and keeps 32 registers free for the key.
struct CbTab {
  c64 w[CB_TAB];
};
template <int K>  // K 64ths of a turn
__device__ __forceinline__ c64 cb_turn(const c64& w) {
  constexpr double c = cos64(K), s = sin64(K);
  return make_double2(__builtin_fma(c, w.x, -(s * w.y)), __builtin_fma(c, w.y, s * w.x));
}
struct CbPass2 {
  const c64* w;
  __device__ __forceinline__ c64 operator()(int e) const {
    switch (e) {
      case 0: return w[0];
      case 1: return w[1];
      case 2: return w[2];
      case 3: return cb_turn<8>(w[2]);
      case 4: return w[3];
      case 5: return cb_turn<8>(w[3]);
      case 6: return cb_turn<4>(w[3]);
      default: return cb_turn<12>(w[3]);
    }
  }
};
struct CbPass3 {  // residue k = 2 b + c
  const c64* w;
  int k;
  __device__ __forceinline__ c64 operator()(int e) const {
    if (e == 0) {
      const c64 x = w[4 + (k >> 1)];
      return (k & 1) ? make_double2(-x.y, x.x) : x;
    }
    return (k & 1) ? cb_turn<8>(w[6 + (k >> 1)]) : w[6 + (k >> 1)];
  }
};

__device__ __forceinline__ int cb_place1(int u, int j) { return u * 64 + (j ^ (4 * (u & 3))); }
__device__ __forceinline__ int cb_place2(int u, int up, int v) { return u * 64 + ((4 * up + (v ^ (up >> 2))) ^ (4 * (u & 3))); }

__device__ __forceinline__ void cb_pass3(double (&re)[16], double (&im)[16], const CbTab& tab, bool inverse) {
#pragma unroll
  for (int k = 0; k < 4; k++) {
    double r[4], i[4];
#pragma unroll
    for (int q = 0; q < 4; q++) {
      r[q] = re[4 * k + q];
      i[q] = im[4 * k + q];
    }
    if (inverse)
      fft_pass_inverse(r, i, CbPass3{tab.w, k});
    else
      fft_pass(r, i, CbPass3{tab.w, k});
#pragma unroll
    for (int q = 0; q < 4; q++) {
      re[4 * k + q] = r[q];
      im[4 * k + q] = i[q];
    }
  }
}
// The exchanges form their LDS places anew from an opaque copy of the lane index, so that none of
// them stays live across a pass.
__device__ __forceinline__ void cb_put1(const double (&re)[16], const double (&im)[16], c64* reg, int lane, bool rows) {
  const int L = opaque_lane(lane), u = L >> 2, v = L & 3;
#pragma unroll
  for (int t = 0; t < 16; t++) reg[rows ? cb_place1(u, v + 4 * t) : cb_place1(t, L)] = make_double2(re[t], im[t]);
  wave_lds_sync();
}
__device__ __forceinline__ void cb_get1(double (&re)[16], double (&im)[16], const c64* reg, int lane, bool rows) {
  const int L = opaque_lane(lane), u = L >> 2, v = L & 3;
#pragma unroll
  for (int t = 0; t < 16; t++) {
    const c64 x = reg[rows ? cb_place1(u, v + 4 * t) : cb_place1(t, L)];
    re[t] = x.x;
    im[t] = x.y;
  }
  wave_lds_sync();
}
// Second exchange: by residue u' of the lane's v (rows), or coefficient s mod 4 of residue 4 v + s / 4.
__device__ __forceinline__ void cb_put2(const double (&re)[16], const double (&im)[16], c64* reg, int lane, bool rows) {
  const int L = opaque_lane(lane), u = L >> 2, v = L & 3;
#pragma unroll
  for (int s = 0; s < 16; s++)
    reg[rows ? cb_place2(u, s, v) : cb_place2(u, 4 * v + (s >> 2), s & 3)] = make_double2(re[s], im[s]);
  wave_lds_sync();
}
__device__ __forceinline__ void cb_get2(double (&re)[16], double (&im)[16], const c64* reg, int lane, bool rows) {
  const int L = opaque_lane(lane), u = L >> 2, v = L & 3;
#pragma unroll
  for (int s = 0; s < 16; s++) {
    const c64 x = reg[rows ? cb_place2(u, s, v) : cb_place2(u, 4 * v + (s >> 2), s & 3)];
    re[s] = x.x;
    im[s] = x.y;
  }
  wave_lds_sync();
}
__device__ __forceinline__ void cb_forward(double (&re)[16], double (&im)[16], const CbTab& tab, c64* reg, int lane) {
  fft_pass(re, im, FftConst{});
  cb_put1(re, im, reg, lane, false);
  cb_get1(re, im, reg, lane, true);
  fft_pass(re, im, CbPass2{tab.w});
  cb_put2(re, im, reg, lane, true);
  cb_get2(re, im, reg, lane, false);
  cb_pass3(re, im, tab, false);
}
// Inverse transform, times 1024.
__device__ __forceinline__ void cb_inverse(double (&re)[16], double (&im)[16], const CbTab& tab, c64* reg, int lane) {
  cb_pass3(re, im, tab, true);
  cb_put2(re, im, reg, lane, false);
  cb_get2(re, im, reg, lane, true);
  fft_pass_inverse(re, im, CbPass2{tab.w});
  cb_put1(re, im, reg, lane, true);
  cb_get1(re, im, reg, lane, false);
  fft_pass_inverse(re, im, FftConst{});
}

// Limb b of a key word as a signed integer.
__device__ __forceinline__ int cb_limb(u64 k, int b) {
  const int l0 = (int)((u32)k << (32 - CB_LIMB_BITS)) >> (32 - CB_LIMB_BITS);
  if (b == 0) return l0;
  const int64_t k1 = (int64_t)(k - (u64)(int64_t)l0) >> CB_LIMB_BITS;
  const int l1 = (int)((u32)k1 << (32 - CB_LIMB_BITS)) >> (32 - CB_LIMB_BITS);
  return b == 1 ? l1 : (int)((k1 - l1) >> CB_LIMB_BITS);
}

// Key conversion: one wave per (step i, row, product).
__global__ __launch_bounds__(256) void k_cb_key(const u64* __restrict__ bk2, c64* __restrict__ dst,
                                                const c64* __restrict__ tab, uint64_t jobs) {
  __shared__ c64 lds[4 * CB_REGION_C64];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const uint64_t job = (uint64_t)blockIdx.x * 4 + wave;
  if (job >= jobs) return;
  const uint64_t row = job / CB_PRODUCTS;  // i * 8 + row
  const int q = (int)(job % CB_PRODUCTS);
  const u64* K = bk2 + (row * 2 + q / CB_LIMBS) * CB_N2;
  CbTab t;
#pragma unroll
  for (int e = 0; e < CB_TAB; e++) t.w[e] = tab[e * 64 + lane];
  double re[16], im[16];
#pragma unroll
  for (int s = 0; s < 16; s++) {
    re[s] = (double)cb_limb(K[lane + 64 * s], q % CB_LIMBS);
    im[s] = (double)cb_limb(K[lane + 64 * s + CB_N2 / 2], q % CB_LIMBS);
  }
  cb_forward(re, im, t, lds + wave * CB_REGION_C64, lane);
  c64* out = dst + (row / CB_ROWS) * CB_KEY_STEP + (row % CB_ROWS) * CB_KEY_ROW + q * 2 * 64 + lane;
#pragma unroll
  for (int s = 0; s < 16; s++)  // the inverse's factor 1024 is taken off here (exactly)
    out[(size_t)(s >> 1) * CB_ROWS * CB_KEY_ROW + (s & 1) * 64] = make_double2(re[s] * 0x1p-10, im[s] * 0x1p-10);
}

// Level-2 blind rotation, one workgroup of eight waves per job (circuit bootstrap c = job / l, gadget
// level j = job % l + 1), one per compute unit. Per step: all waves form the digit words of
// X^abar ACC - ACC; wave r transforms gadget digit r mod 4 + 1 of polynomial r / 4 into its own 16 KiB of
// LDS; wave w adds the eight rows' products with the six key polynomials at slots 2 w and 2 w + 1; once
// every row has been read, the sums take the rows' place, waves 0-5 invert one each and leave its
// integers, shifted by their limb, in its region, and all waves add the three of each output to ACC.
// The rows and the accumulator fill the 160 KiB of LDS. The key, 786 KB a step, is read once per job,
// two rows' entries (12 each per lane) ahead of use. A step of 255 jobs takes 17.0 us (of 24 jobs 17.8, of
// three 19.7: fewer jobs share what comes from memory), 12.3 without the key loads (transforms and LDS in
// turn: VALU issue is 40% busy, LDS 28%), the rest is the key's stream, 50 to 64 bytes a clock, past the
// two rows that the registers hold. Those two are loaded beside the inverse transform; asked for among
// the last products, where the stream is the bound, a step took 1 us more. The result is
// SampleExtract_0 + 1/(2 Bg^j) as a TLWE2.
constexpr size_t CB_LDS = (size_t)CB_ROWS * CB_REGION_C64 * 16 + 2 * CB_N2 * 8;
static_assert(CB_ROWS == CB_WAVES && CB_PRODUCTS <= CB_WAVES, "one wave per row and per sum");

__global__ __launch_bounds__(CB_WAVES * 64) void k_cb_rotate(const c64* __restrict__ key, const c64* __restrict__ tab,
                                                            const u32* __restrict__ in, u64* __restrict__ out,
                                                            int gadget_l, int bgbit) {
  extern __shared__ c64 cb_lds[];
  u64* acc = reinterpret_cast<u64*>(cb_lds + CB_ROWS * CB_REGION_C64);  // [2][N2]
  const uint64_t job = blockIdx.x;
  const int j = (int)(job % (uint64_t)gadget_l) + 1;
  const u32* c = in + (job / (uint64_t)gadget_l) * TLWE0;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane0 = tid & 63;
  c64* reg = cb_lds + wave * CB_REGION_C64;
  const u64 tvv = 1ull << (63 - bgbit * j);                    // 1/(2 Bg^j)
  CbTab t;
#pragma unroll
  for (int e = 0; e < CB_TAB; e++) t.w[e] = tab[e * 64 + lane0];
  // wait for the table here: a wait left to its first use, inside the loop, would count the key
  // loads issued since and so wait for those in every step
  __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
  const gkey kbase = (gkey)key + (size_t)wave * CB_ROWS * CB_KEY_ROW + lane0;
  c64 kr[2][CB_PRODUCTS * 2];
  auto load_row = [&](int i, int row, c64(&k)[CB_PRODUCTS * 2]) {
    const gkey p = kbase + (size_t)i * CB_KEY_STEP + row * CB_KEY_ROW;
#pragma unroll
    for (int e = 0; e < CB_PRODUCTS * 2; e++) k[e] = gkey_load(p + e * 64);
  };
  load_row(0, 0, kr[0]);
  load_row(0, 1, kr[1]);
  {
    const u32 bbar = ((c[LWE_N] + (1u << 19)) >> 20) & (2 * CB_N2 - 1);
    const int k = (int)((2 * CB_N2 - bbar) & (2 * CB_N2 - 1));
    for (int m = tid; m < CB_N2; m += CB_WAVES * 64) {
      const bool neg = (m < (k & (CB_N2 - 1))) != (k >= CB_N2);
      acc[m] = 0;
      acc[CB_N2 + m] = neg ? (0ull - tvv) : tvv;
    }
  }
  u32 c_next = __builtin_amdgcn_readfirstlane(c[0]);
  __syncthreads();
  u64 own[2 * CB_N2 / (CB_WAVES * 64)];  // this thread's words of ACC, from the end of a step to the next one's start
#pragma unroll
  for (int q = 0; q < 2 * CB_N2 / (CB_WAVES * 64); q++) own[q] = acc[tid + CB_WAVES * 64 * q];
  for (int i = 0; i < LWE_N; i++) {
    const int abar = (int)(((c_next + (1u << 19)) >> 20) & (2 * CB_N2 - 1));
    c_next = __builtin_amdgcn_readfirstlane(c[i + 1]);  // (the last one is b)
    const int lane = opaque_lane(lane0);                // addresses are formed anew in every step
    double re[16], im[16];
    // The digit words of X^abar ACC_h - ACC_h (d + the rounding offset, the top bit of each digit field
    // flipped so that it is a signed field), once for the four rows of a polynomial, in regions 0 and 1.
    u64* words = reinterpret_cast<u64*>(cb_lds);
#pragma unroll
    for (int q = 0; q < 2 * CB_N2 / (CB_WAVES * 64); q++) {
      const int m = (opaque_lane(tid) + CB_WAVES * 64 * q) & (CB_N2 - 1);
      const u64* P = acc + (q / (CB_N2 / (CB_WAVES * 64))) * CB_N2;
      const int src = m - abar;
      const u64 raw = P[src & (CB_N2 - 1)], neg = (u64)((int64_t)((int)((u32)src << 20) >> 31));
      words[tid + CB_WAVES * 64 * q] = ((raw ^ neg) + (CB_DECOMP_OFFSET - own[q] - neg)) ^ CB_DIGIT_FLIP;
    }
    __syncthreads();
    {
      const u64* W = words + (wave / CB_L2) * CB_N2 + lane;
      const int up = CB_BG2 * (wave % CB_L2);
#pragma unroll
      for (int s = 0; s < 16; s++) {
        re[s] = (double)((int)(u32)((W[64 * s] << up) >> 32) >> (32 - CB_BG2));
        im[s] = (double)((int)(u32)((W[64 * s + CB_N2 / 2] << up) >> 32) >> (32 - CB_BG2));
      }
    }
    __syncthreads();
    cb_forward(re, im, t, reg, lane);
#pragma unroll
    for (int s = 0; s < 16; s++) reg[s * 64 + lane] = make_double2(re[s], im[s]);
    __syncthreads();
    {
      double sr[CB_PRODUCTS][2], si[CB_PRODUCTS][2];
#pragma unroll
      for (int q = 0; q < CB_PRODUCTS; q++) sr[q][0] = sr[q][1] = si[q][0] = si[q][1] = 0.0;
#pragma unroll
      for (int row = 0; row < CB_ROWS; row++) {
        const c64 x0 = cb_lds[row * CB_REGION_C64 + (2 * wave) * 64 + lane];
        const c64 x1 = cb_lds[row * CB_REGION_C64 + (2 * wave + 1) * 64 + lane];
#pragma unroll
        for (int q = 0; q < CB_PRODUCTS; q++) {
          fft_cmac(sr[q][0], si[q][0], x0.x, x0.y, kr[row & 1][2 * q]);
          fft_cmac(sr[q][1], si[q][1], x1.x, x1.y, kr[row & 1][2 * q + 1]);
        }
        if (row + 2 < CB_ROWS) load_row(i, row + 2, kr[row & 1]);
        __builtin_amdgcn_sched_barrier(0);
      }
      __syncthreads();  // every row has been read
#pragma unroll
      for (int q = 0; q < CB_PRODUCTS; q++)
#pragma unroll
        for (int e = 0; e < 2; e++)
          cb_lds[q * CB_REGION_C64 + (2 * wave + e) * 64 + lane] = make_double2(sr[q][e], si[q][e]);
    }
    __syncthreads();
    if (wave < CB_PRODUCTS) {
#pragma unroll
      for (int s = 0; s < 16; s++) {
        const c64 x = reg[s * 64 + lane];
        re[s] = x.x;
        im[s] = x.y;
      }
      wave_lds_sync();
      cb_inverse(re, im, t, reg, lane);
      // the integers, shifted by their limb, in the wave's own region
      u64* z = reinterpret_cast<u64*>(reg) + lane;
      const int up = CB_LIMB_BITS * (wave % CB_LIMBS);
#pragma unroll
      for (int s = 0; s < 32; s++) {
        const double v = s < 16 ? re[s & 15] : im[s & 15];
        z[64 * s] = (__builtin_bit_cast(u64, v + 0x1.8p+52) - __builtin_bit_cast(u64, 0x1.8p+52)) << up;
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    load_row(i + 1 < LWE_N ? i + 1 : i, 0, kr[0]);
    load_row(i + 1 < LWE_N ? i + 1 : i, 1, kr[1]);
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 2 * CB_N2 / (CB_WAVES * 64); q++) {  // ACC += the three limbs' words
      constexpr int PER = CB_N2 / (CB_WAVES * 64), REGION = CB_REGION_C64 * 2;
      const int m = opaque_lane(tid) + CB_WAVES * 64 * (q % PER);
      const u64* z = reinterpret_cast<const u64*>(cb_lds) + (q / PER) * CB_LIMBS * REGION + m;
      own[q] = acc[(q / PER) * CB_N2 + m] + (z[0] + z[REGION] + z[2 * REGION]);
      acc[(q / PER) * CB_N2 + m] = own[q];
    }
    __syncthreads();
  }
  u64* dst = out + job * CB_TLWE2;
  for (int m = tid; m < CB_N2; m += CB_WAVES * 64) dst[m] = (m == 0) ? acc[0] : (0ull - acc[CB_N2 - m]);
  if (tid == 0) dst[CB_N2] = acc[CB_N2] + tvv;
}

// Private functional key switch: out = sum_{k <= N2, p < t2} PKSK[u][k][p][v_{k,p} - 1] over the
// nonzero base-4 digits v_{k,p} (most significant first) of c_k rounded to 24 bits. Row u = 0
// is TRGSW row j - 1, u = 1 row l + j - 1. Runs on the matrix cores (onehot_mfma.h): a coefficient
// has three digit bytes.
constexpr int CB_DIGIT_BYTES = CB_TLWE2 * CB_T / 4;
constexpr int CB_QUADS = (CB_DIGIT_BYTES + 15) / 16;                        // of four blocks of four digit bytes
constexpr int CB_COL_TILES = (int)(CB_PKS_ROW / 16);
constexpr size_t CB_PKS_TILE = (size_t)CB_QUADS * 4 * OH_BLOCK;             // 16-byte entries of a column tile
constexpr uint64_t CB_PKS_CHUNK = 8192;                                     // jobs whose digits are held at once

// Key planes of one u, one digit (a word per plane) per thread.
__global__ __launch_bounds__(256) void k_cb_pkskey(const u32* __restrict__ pksk, u32* __restrict__ dst) {
  const uint64_t id = (uint64_t)blockIdx.x * 256 + threadIdx.x;
  const int w = (int)(id & 3), lane = (int)((id >> 2) & 63);
  const uint64_t rest = id >> 8;
  const int block = (int)(rest % (CB_QUADS * 4)), ct = (int)(rest / (CB_QUADS * 4));
  if (ct >= CB_COL_TILES) return;
  const int i = 4 * block + (lane >> 4);
  u32 x[3] = {0u, 0u, 0u}, p[OH_PLANES];
  if (i < CB_DIGIT_BYTES)
#pragma unroll
    for (int v = 0; v < 3; v++)
      x[v] = pksk[((size_t)(i * 4 + w) * 3 + v) * CB_PKS_ROW + 16 * ct + (lane & 15)];
  oh_planes(x[0], x[1], x[2], p);
#pragma unroll
  for (int b = 0; b < OH_PLANES; b++) dst[((rest * OH_PLANES + b) * 64 + lane) * 4 + w] = p[b];
}

// Digits of `jobs` TLWE2s, one word per thread; elements past them select nothing.
__global__ __launch_bounds__(256) void k_cb_digits(const u64* __restrict__ tl2, u32* __restrict__ dst, uint64_t jobs,
                                                   uint64_t words) {
  const uint64_t id = (uint64_t)blockIdx.x * 256 + threadIdx.x;
  if (id >= words) return;
  const int lane = (int)(id & 63);
  const uint64_t rest = id >> 6;
  const uint64_t job = rest / CB_QUADS * 16 + (lane & 15);
  constexpr int TB = CB_T * CB_BB;
  u32 d = 0;
#pragma unroll
  for (int t = 0; t < 4; t++) {
    const int i = (int)(rest % CB_QUADS) * 16 + 4 * t + (lane >> 4);
    if (job >= jobs || i >= CB_DIGIT_BYTES) continue;
    const u32 c = (u32)((tl2[job * CB_TLWE2 + i / 3] + (1ull << (64 - TB - 1))) >> (64 - TB));
    d |= ((c >> (16 - 8 * (i % 3))) & 255u) << (8 * t);
  }
  dst[id] = ~d;
}

// A wave's digits: every eighth quad, the next one's words loaded a step ahead.
template <int T>
struct CbDigits {
  oh_digits at;
  int wave;
  u32 next[T];
  __device__ __forceinline__ int quad(int n) const { return wave + OH_WAVES * n; }
  __device__ __forceinline__ void load(int n) {
#pragma unroll
    for (int i = 0; i < T; i++) next[i] = at[((size_t)i * CB_QUADS + quad(n)) * 64];
  }
  __device__ __forceinline__ void start() { load(0); }
  __device__ __forceinline__ void get(int, u32 (&d)[T]) {
#pragma unroll
    for (int i = 0; i < T; i++) d[i] = next[i];
  }
  __device__ __forceinline__ void issue(int n) { load(quad(n + 1) < CB_QUADS ? n + 1 : n); }
  __device__ __forceinline__ void finish(int) {}
};

// One workgroup of eight waves per (16 T jobs, u, 16 columns), each wave an eighth of the digits. The
// workgroups of a column tile follow each other on one XCD (of eight, dealt out in turn), so that its
// key, 6.3 MB, is read from memory once for all jobs. Measured: 24 jobs 0.26 ms, the key's 1.6 GB at
// 6.2 TB/s; 864 jobs 0.89 ms, 1.4 x 10^12 multiply-adds at 1.6 x 10^15/s, where the matrix cores and the
// one-hot construction on the VALU share the issue slots. Selecting rows through LDS, a word per
// thread, took 2.1 and 12.6 ms. Wider tiles of jobs build each operand for the same key loads, so the
// widest that the batch fills is taken.
template <int T>
__global__ __launch_bounds__(OH_WAVES * 64, 2) void k_cb_privks(const oh_v4i* __restrict__ key, const u32* __restrict__ digits,
                                                     u32* __restrict__ out, int gadget_l, uint64_t job0, uint64_t jobs,
                                                     u32 job_tiles) {
  __shared__ u32 red[OH_WAVES][T * 4][64];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const u32 seq = blockIdx.x / 8, jt = seq % job_tiles;
  const int uc = (int)(seq / job_tiles * 8 + blockIdx.x % 8), u = uc / CB_COL_TILES, ct = uc % CB_COL_TILES;
  u32 sum[T][4];
  CbDigits<T> source;
  source.at = (oh_digits)digits + (size_t)jt * T * CB_QUADS * 64 + lane;
  source.wave = wave;
  oh_products<T>((oh_key)key + (size_t)uc * CB_PKS_TILE + lane, source, (CB_QUADS - wave + OH_WAVES - 1) / OH_WAVES, sum);
  oh_reduce<T, OH_WAVES>(sum, red, wave, lane, [&](int i, int x, u32 v) {
    const uint64_t g = ((uint64_t)jt * T + i) * 16 + 4 * (lane >> 4) + x;
    if (g >= jobs) return;
    const uint64_t job = job0 + g;
    const int row = u * gadget_l + (int)(job % (uint64_t)gadget_l);
    out[((job / (uint64_t)gadget_l) * 2 * gadget_l + row) * CB_PKS_ROW + 16 * ct + (lane & 15)] = v;
  });
}
static_assert(2 * CB_COL_TILES % 8 == 0, "column tiles are dealt out to eight XCDs");

template <int T>
static void launch_privks(const oh_v4i* key, const u32* digits, u32* out, uint64_t job0, uint64_t jobs, hipStream_t st) {
  const uint64_t tiles = (jobs + 16 * T - 1) / (16 * T);
  hipLaunchKernelGGL(k_cb_privks<T>, dim3((unsigned)(tiles * 2 * CB_COL_TILES)), dim3(OH_WAVES * 64), 0, st, key, digits, out,
                     GADGET_L, job0, jobs, (u32)tiles);
}
static uint64_t digit_words(uint64_t jobs) { return (jobs + 127) / 128 * 128 / 16 * CB_QUADS * 64; }

hipError_t init_cb_kernel_attributes() {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(&k_cb_rotate), hipFuncAttributeMaxDynamicSharedMemorySize,
                             (int)CB_LDS);
}

// Lane table (CbTab): lane 4 u + v has the root z_u in pass 2, the residues 4 v + k in pass 3.
static std::vector<c64> make_cb_table() {
  std::vector<c64> t(CB_TAB * 64);
  for (int L = 0; L < 64; L++) {
    const long double zu = fft_leaf(0.25L, 4, L >> 2), n = fft_leaf(zu, 2, L & 3);
    const long double a[CB_TAB] = {zu / 2, zu / 4, zu / 8, zu / 16, n / 8, n / 8 + 1 / 8.0L, n / 16, n / 16 + 1 / 16.0L};
    for (int e = 0; e < CB_TAB; e++) t[e * 64 + L] = fft_unit(a[e]);
  }
  return t;
}

}  // namespace vsp

using namespace vsp;

struct vsp_cbkey {
  vsp_context* ctx = nullptr;
  c64* key = nullptr;   // transformed level-2 bootstrapping key
  c64* tab = nullptr;   // lane table of its transform
  oh_v4i* pksk = nullptr;  // byte planes of the private key-switching keys
  Scratch tl2;          // TLWE2 outputs of the blind rotations, then digits of the key switch
};

extern "C" {

vsp_status vsp_cbkey_create(vsp_context* ctx, const uint64_t* bk2_host, const uint32_t* pksk_host, vsp_cbkey** out) {
  if (out == nullptr) return fail(VSP_E_ARG, "out is NULL");
  *out = nullptr;
  if (ctx == nullptr) return fail(VSP_E_ARG, "context is NULL");
  if (bk2_host == nullptr || pksk_host == nullptr) return fail(VSP_E_ARG, "bk2_host and pksk_host must not be NULL");
  VSP_HIP(hipSetDevice(ctx->device));
  VSP_HIP(init_cb_kernel_attributes());
  auto* k = new vsp_cbkey();
  k->ctx = ctx;
  u64* tmp = nullptr;
  auto bail = [&](vsp_status st) {
    if (tmp) (void)hipFree(tmp);
    vsp_cbkey_destroy(k);
    return st;
  };
  const size_t bk2_bytes = (size_t)LWE_N * CB_ROWS * 2 * CB_N2 * 8;
  hipError_t e;
  if ((e = hipMalloc(&tmp, bk2_bytes)) != hipSuccess) return bail(hip_fail(e, "hipMalloc(level-2 key)"));
  if ((e = hipMalloc(&k->key, (size_t)LWE_N * CB_KEY_STEP * sizeof(c64))) != hipSuccess)
    return bail(hip_fail(e, "hipMalloc(level-2 key, transformed)"));
  if ((e = hipMalloc(&k->pksk, 2 * CB_COL_TILES * CB_PKS_TILE * sizeof(oh_v4i))) != hipSuccess)
    return bail(hip_fail(e, "hipMalloc(private key-switching keys)"));
  if ((e = hipMemcpy(tmp, bk2_host, bk2_bytes, hipMemcpyHostToDevice)) != hipSuccess) return bail(hip_fail(e, "upload"));
  const std::vector<c64> tab = make_cb_table();
  if ((e = hipMalloc(&k->tab, tab.size() * sizeof(c64))) != hipSuccess) return bail(hip_fail(e, "hipMalloc(table)"));
  if ((e = hipMemcpy(k->tab, tab.data(), tab.size() * sizeof(c64), hipMemcpyHostToDevice)) != hipSuccess)
    return bail(hip_fail(e, "upload table"));
  const uint64_t jobs = (uint64_t)LWE_N * CB_ROWS * CB_PRODUCTS;
  hipLaunchKernelGGL(k_cb_key, dim3((unsigned)((jobs + 3) / 4)), dim3(256), 0, nullptr, tmp, k->key, k->tab, jobs);
  if ((e = hipGetLastError()) != hipSuccess) return bail(hip_fail(e, "level-2 key conversion"));
  if ((e = hipDeviceSynchronize()) != hipSuccess) return bail(hip_fail(e, "level-2 key conversion"));
  (void)hipFree(tmp);
  tmp = nullptr;
  if ((e = hipMalloc(&tmp, CB_PKS_U * 4)) != hipSuccess) return bail(hip_fail(e, "hipMalloc(private key-switching keys, staging)"));
  for (int u = 0; u < 2; u++) {
    if ((e = hipMemcpy(tmp, pksk_host + (size_t)u * CB_PKS_U, CB_PKS_U * 4, hipMemcpyHostToDevice)) != hipSuccess)
      return bail(hip_fail(e, "upload"));
    hipLaunchKernelGGL(k_cb_pkskey, dim3((unsigned)(CB_COL_TILES * CB_QUADS * 4)), dim3(256), 0, nullptr,
                       reinterpret_cast<const u32*>(tmp), reinterpret_cast<u32*>(k->pksk + (size_t)u * CB_COL_TILES * CB_PKS_TILE));
    if ((e = hipGetLastError()) != hipSuccess) return bail(hip_fail(e, "private key-switching key conversion"));
    if ((e = hipDeviceSynchronize()) != hipSuccess) return bail(hip_fail(e, "private key-switching key conversion"));
  }
  (void)hipFree(tmp);
  tmp = nullptr;
  *out = k;
  return VSP_OK;
}

vsp_status vsp_cbkey_destroy(vsp_cbkey* k) {
  if (k == nullptr) return VSP_OK;
  (void)hipSetDevice(k->ctx->device);
  (void)hipDeviceSynchronize();
  for (void* p : {(void*)k->key, (void*)k->tab, (void*)k->pksk, k->tl2.ptr})
    if (p) (void)hipFree(p);
  delete k;
  return VSP_OK;
}

vsp_status vsp_cbkey_set_form(vsp_cbkey* key, int form) {
  if (key == nullptr) return fail(VSP_E_ARG, "key is NULL");
  if (form < 0 || form > 2) return fail(VSP_E_ARG, "form must be 0, 1 or 2");
  return VSP_OK;  // one form serves every batch size
}

vsp_status vsp_circuit_bootstrap(vsp_context* ctx, vsp_cbkey* key, const uint32_t* d_in, uint32_t* d_out, uint64_t R,
                                 void* stream) {
  if (ctx == nullptr) return fail(VSP_E_ARG, "context is NULL");
  vsp_status s = VSP_OK;
  if (key == nullptr || key->ctx != ctx) return fail(VSP_E_ARG, "key is NULL or belongs to another context");
  if (R == 0) return VSP_OK;
  if (R > (1ull << 20)) return fail(VSP_E_ARG, "R too large");
  VSP_HIP(hipSetDevice(ctx->device));
  const size_t ib = (size_t)R * TLWE0 * 4, ob = (size_t)R * 2 * GADGET_L * 2 * RING_N * 4;
  if ((s = check_device_range(ctx, d_in, ib, "d_in"))) return s;
  if ((s = check_device_range(ctx, d_out, ob, "d_out"))) return s;
  if ((s = check_no_overlap(d_out, ob, d_in, ib, "d_out and d_in"))) return s;
  const uint64_t jobs = R * GADGET_L;
  const size_t tl2_bytes = (jobs * CB_TLWE2 * 8 + 255) / 256 * 256;
  if ((s = scratch_reserve(ctx, key->tl2, tl2_bytes + digit_words(std::min(jobs, CB_PKS_CHUNK)) * 4))) return s;
  hipStream_t st = static_cast<hipStream_t>(stream);
  u64* tl2 = static_cast<u64*>(key->tl2.ptr);
  u32* digits = reinterpret_cast<u32*>(static_cast<char*>(key->tl2.ptr) + tl2_bytes);
  hipLaunchKernelGGL(k_cb_rotate, dim3((unsigned)jobs), dim3(CB_WAVES * 64), CB_LDS, st, key->key, key->tab, d_in, tl2,
                     GADGET_L, BG_BIT);
  for (uint64_t j0 = 0; j0 < jobs; j0 += CB_PKS_CHUNK) {
    const uint64_t n = std::min(jobs - j0, CB_PKS_CHUNK), words = digit_words(n);
    hipLaunchKernelGGL(k_cb_digits, dim3((unsigned)((words + 255) / 256)), dim3(256), 0, st, tl2 + j0 * CB_TLWE2, digits, n,
                       words);
    if (n <= 16)
      launch_privks<1>(key->pksk, digits, d_out, j0, n, st);
    else if (n <= 32)
      launch_privks<2>(key->pksk, digits, d_out, j0, n, st);
    else if (n <= 64)
      launch_privks<4>(key->pksk, digits, d_out, j0, n, st);
    else
      launch_privks<8>(key->pksk, digits, d_out, j0, n, st);
  }
  VSP_HIP(hipGetLastError());
  return VSP_OK;
}

}  // extern "C"
