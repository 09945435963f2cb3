// Identity key switch on the matrix cores (Sec. 2.1.2, Sample Extraction and Identity Key
// Switching): out = (0, b') - sum_{j < N, p < t} KSK[j][p][v_{j,p}], v_{j,p} the p-th base-4
// digit of a'_j rounded to 16 bits, as a product of one-hot digits with the key's byte planes
// (onehot_mfma.h). A coefficient has two digit bytes, a quad of blocks eight coefficients.
#include "onehot_mfma.h"

namespace vsp {

constexpr int KM_CT = (TLWE0 + 15) / 16;          // 40 column tiles of 16 (631 columns)
constexpr int KM_QUADS = RING_N * KS_T / 64;      // 128
constexpr size_t KM_TILE = (size_t)KM_QUADS * 4 * OH_BLOCK;  // 16-byte entries of a column tile
constexpr size_t KM_KEY_BYTES = KM_CT * KM_TILE * 16;
constexpr int KM_ROW = 68;                        // words of a staged quad: 64 lanes, padded to spread the banks

// Key planes, one digit (a word per plane) per thread.
__global__ __launch_bounds__(256) void k_ks_mfkey(const u32* __restrict__ ksk, u32* __restrict__ dst) {
  const uint64_t id = (uint64_t)blockIdx.x * 256 + threadIdx.x;
  const int w = (int)(id & 3), lane = (int)((id >> 2) & 63);
  const uint64_t rest = id >> 8;
  const int block = (int)(rest % (KM_QUADS * 4)), ct = (int)(rest / (KM_QUADS * 4));
  if (ct >= KM_CT) return;
  const int i = 4 * block + (lane >> 4), c = 16 * ct + (lane & 15);  // digit byte, column
  u32 x[3] = {0u, 0u, 0u}, p[OH_PLANES];
  if (c < TLWE0)
#pragma unroll
    for (int v = 0; v < 3; v++) x[v] = ksk[((size_t)(i * 4 + w) * 4 + v + 1) * TLWE0 + c];
  oh_planes(x[0], x[1], x[2], p);
#pragma unroll
  for (int b = 0; b < OH_PLANES; b++) dst[((rest * OH_PLANES + b) * 64 + lane) * 4 + w] = p[b];
}

// The digit words of a workgroup's 16 T gates, formed from a' in LDS a chunk of quads at a time and
// shared by its waves. A thread's unit of that work is one gate, quad and half h: the coefficients
// 8 Q + 2 t + h (t = 0..3) give the words of the lanes (gate, 2 h) and (gate, 2 h + 1). The next
// chunk is formed during the steps of this one, in the other buffer, its loads issued before a
// step's products. A gate past the batch selects nothing.
template <int T, int SPLIT>
struct KsDigits {
  static constexpr int CHUNK = T >= 2 ? 256 / T : KM_QUADS;              // quads
  static constexpr int CHUNKS = KM_QUADS / CHUNK;
  static constexpr int STEPS = CHUNK / SPLIT;                            // a wave's steps per chunk
  static constexpr int UNITS = 16 * T * CHUNK * 2 / (OH_WAVES * 64);     // per thread and chunk
  static constexpr int PER_STEP = CHUNKS > 1 ? UNITS / STEPS : 1;
  static constexpr int WORDS = T * CHUNK * KM_ROW;                       // of a buffer
  static_assert(CHUNK <= KM_QUADS && CHUNKS * CHUNK == KM_QUADS && STEPS * SPLIT == CHUNK, "whole chunks and steps");
  static_assert(CHUNKS == 1 || PER_STEP * STEPS == UNITS, "a chunk is formed in the steps of another");
  const u32* __restrict__ tlwe1;
  uint64_t g0, B;
  u32* lds;   // [CHUNKS > 1 ? 2 : 1][WORDS]
  int split, lane;
  u32 x[PER_STEP][4];
  // unit u of this thread: a wave covers 8 quads x 2 halves (64 consecutive coefficients) of four gates
  __device__ __forceinline__ void place(int u, int& g, int& Q, int& h) const {
    const int id = u * OH_WAVES * 64 + (int)threadIdx.x;
    h = id & 1;
    const int ql = (id >> 1) & 7, gl = (id >> 4) & 3, rest = id >> 6;
    Q = rest % (CHUNK / 8) * 8 + ql;
    g = rest / (CHUNK / 8) * 4 + gl;
  }
  __device__ __forceinline__ void fetch(int chunk, int u, u32 (&v)[4]) const {
    int g, Q, h;
    place(u, g, Q, h);
    const u32* p = tlwe1 + (g0 + g < B ? g0 + g : 0) * TLWE1 + (chunk * CHUNK + Q) * 8 + h;
#pragma unroll
    for (int t = 0; t < 4; t++) v[t] = p[2 * t];
  }
  __device__ __forceinline__ void put(int chunk, int u, const u32 (&v)[4]) const {
    int g, Q, h;
    place(u, g, Q, h);
    u32 hi = 0, lo = 0;
#pragma unroll
    for (int t = 0; t < 4; t++) {
      const u32 r = v[t] + (1u << 15);
      hi |= (r >> 24) << (8 * t);
      lo |= ((r >> 16) & 255u) << (8 * t);
    }
    const bool live = g0 + g < B;
    u32* w = lds + (chunk & 1) * WORDS + ((g >> 4) * CHUNK + Q) * KM_ROW + (g & 15) + 32 * h;
    w[0] = live ? ~hi : ~0u;
    w[16] = live ? ~lo : ~0u;
  }
  __device__ __forceinline__ int quad(int n) const { return n / STEPS * CHUNK + split * STEPS + n % STEPS; }
  __device__ __forceinline__ void start() {
#pragma unroll 1
    for (int u = 0; u < UNITS; u += 4) {
      u32 v[4][4];
#pragma unroll
      for (int k = 0; k < 4; k++) fetch(0, u + k, v[k]);
#pragma unroll
      for (int k = 0; k < 4; k++) put(0, u + k, v[k]);
    }
  }
  __device__ __forceinline__ void get(int n, u32 (&d)[T]) const {
    if (n % STEPS == 0) __syncthreads();  // the chunk is formed, and no wave reads the one before it any more
    const u32* w = lds + (n / STEPS & 1) * WORDS + (split * STEPS + n % STEPS) * KM_ROW + lane;
#pragma unroll
    for (int i = 0; i < T; i++) d[i] = w[i * CHUNK * KM_ROW];
  }
  __device__ __forceinline__ void issue(int n) {
    if (CHUNKS == 1 || n / STEPS + 1 == CHUNKS) return;
#pragma unroll
    for (int k = 0; k < PER_STEP; k++) fetch(n / STEPS + 1, n % STEPS * PER_STEP + k, x[k]);
  }
  __device__ __forceinline__ void finish(int n) {
    if (CHUNKS == 1 || n / STEPS + 1 == CHUNKS) return;
#pragma unroll
    for (int k = 0; k < PER_STEP; k++) put(n / STEPS + 1, n % STEPS * PER_STEP + k, x[k]);
  }
};

template <int T, int SPLIT>
constexpr size_t km_lds_bytes() {
  using D = KsDigits<T, SPLIT>;
  const size_t stage = (size_t)(D::CHUNKS > 1 ? 2 : 1) * D::WORDS * 4, red = (size_t)OH_WAVES * T * 4 * 64 * 4;
  return stage > red ? stage : red;
}

// One workgroup of eight waves per 16 T gates and 8 / SPLIT column tiles, SPLIT waves sharing a column
// tile's quads. Workgroups are dealt out to eight XCDs in turn: each XCD takes an eighth of the list
// ordered by column group, so that the key of a group is read from memory once for all gates.
template <int T, int SPLIT>
__global__ __launch_bounds__(OH_WAVES * 64, 2) void k_ks_mfma(const oh_v4i* __restrict__ key, const uint8_t* __restrict__ ops,
                                                   const u32* __restrict__ tlwe1, const u32* __restrict__ idxo,
                                                   u32* __restrict__ out, uint64_t B, u32 gate_tiles) {
  constexpr u32 COLS = OH_WAVES / SPLIT;
  extern __shared__ u32 km_lds[];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const u32 item = blockIdx.x % 8 * (gridDim.x / 8) + blockIdx.x / 8;
  if (item >= KM_CT / COLS * gate_tiles) return;  // the whole workgroup: no barrier is skipped by half
  const int ct = (int)(item / gate_tiles * COLS) + wave / SPLIT;
  KsDigits<T, SPLIT> source;
  source.tlwe1 = tlwe1;
  source.g0 = (uint64_t)(item % gate_tiles) * 16 * T;
  source.B = B;
  source.lds = km_lds;
  source.split = wave % SPLIT;
  source.lane = lane;
  u32 sum[T][4];
  oh_products<T>((oh_key)key + (size_t)ct * KM_TILE + lane, source, KM_QUADS / SPLIT, sum);
  __syncthreads();  // the digits are read; the partial sums take their place
  oh_reduce<T, SPLIT>(sum, reinterpret_cast<u32(*)[T * 4][64]>(km_lds) + wave / SPLIT * SPLIT, wave % SPLIT, lane,
                      [&](int i, int x, u32 v) {
    const uint64_t g = source.g0 + 16 * i + 4 * (lane >> 4) + x;
    const int c = 16 * ct + (lane & 15);
    if (g >= B || c >= TLWE0 || (ops && !op_bootstraps(ops[g]))) return;
    out[(uint64_t)(idxo ? idxo[g] : (u32)g) * TLWE0 + c] = (c == LWE_N ? tlwe1[g * TLWE1 + RING_N] : 0u) - v;
  });
}

size_t ks_mf_key_bytes() { return KM_KEY_BYTES; }

hipError_t launch_ks_mfkey(const uint32_t* ksk, int8_t* KB, hipStream_t st) {
  hipLaunchKernelGGL(k_ks_mfkey, dim3((unsigned)(KM_CT * KM_QUADS * 4)), dim3(256), 0, st, ksk, reinterpret_cast<u32*>(KB));
  return hipGetLastError();
}

template <int T, int SPLIT>
static hipError_t launch_km(const int8_t* KB, const uint8_t* ops, const uint32_t* tlwe1, const uint32_t* idxo, uint32_t* out,
                            uint64_t B, hipStream_t st) {
  static_assert(KM_CT % (OH_WAVES / SPLIT) == 0, "whole column groups");
  const uint64_t tiles = (B + 16 * T - 1) / (16 * T);
  const unsigned grid = (unsigned)((tiles * (KM_CT * SPLIT / OH_WAVES) + 7) / 8 * 8);
  const size_t lds = km_lds_bytes<T, SPLIT>();
  hipLaunchKernelGGL((k_ks_mfma<T, SPLIT>), dim3(grid), dim3(OH_WAVES * 64), lds, st,
                     reinterpret_cast<const oh_v4i*>(KB), ops, tlwe1, idxo, out, B, (u32)tiles);
  return hipGetLastError();
}

template <int T, int SPLIT>
static hipError_t km_attribute() {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(&k_ks_mfma<T, SPLIT>), hipFuncAttributeMaxDynamicSharedMemorySize,
                             (int)km_lds_bytes<T, SPLIT>());
}
hipError_t init_keyswitch_mfma_attributes() {
  hipError_t e = km_attribute<1, 8>();
  if (e == hipSuccess) e = km_attribute<2, 8>();
  if (e == hipSuccess) e = km_attribute<4, 8>();
  if (e == hipSuccess) e = km_attribute<8, 8>();
  if (e == hipSuccess) e = km_attribute<8, 4>();
  return e;
}

// Which tile: the fewest gates per workgroup that still give at most one workgroup per compute unit
// (the key streams through each workgroup at a fixed rate: the narrower its tile, the sooner it is
// done), up to 128 gates. From there on every compute unit is busy, and two column tiles per
// workgroup form the digits half as often (a round of workgroups takes 90 us instead of 60 for twice the
// work), so that variant is taken unless its last round wastes more. Measured on 256 compute units, us:
//   gates    16 per workgroup    32     64    128    128 x 2 columns
//      1                 26      30     36     59      88
//     64                 24      29     36     59      88
//    128                 43      29     36     59      89
//    256                 61      52     36     59      90
//    700                145     103     73     62      91
//  1,024                205     128    106    120      91
//  4,096                833     512    356    307     276
// Rows selected through LDS took 157 us for 1 gate, 215 for 256; a 32 x 32 product with the planes one
// after the other 297 us for 700, 430 for 4,096.
hipError_t launch_keyswitch_mfma(const int8_t* KB, const uint8_t* ops, const uint32_t* tlwe1, const uint32_t* idxo,
                                 uint32_t* out, uint64_t B, int cus, hipStream_t st) {
  if (B == 0) return hipSuccess;
  const uint64_t n = cus > 0 ? (uint64_t)cus : 256;
  auto groups = [&](uint64_t gates) { return (B + gates - 1) / gates * KM_CT; };
  auto rounds = [&](uint64_t workgroups) { return (workgroups + n - 1) / n; };
  if (groups(16) <= n) return launch_km<1, 8>(KB, ops, tlwe1, idxo, out, B, st);
  if (groups(32) <= n) return launch_km<2, 8>(KB, ops, tlwe1, idxo, out, B, st);
  if (groups(64) <= n) return launch_km<4, 8>(KB, ops, tlwe1, idxo, out, B, st);
  if (2 * rounds(groups(128)) <= 3 * rounds(groups(128) / 2)) return launch_km<8, 8>(KB, ops, tlwe1, idxo, out, B, st);
  return launch_km<8, 4>(KB, ops, tlwe1, idxo, out, B, st);
}

}  // namespace vsp
