// Matrix-core GEMM for the stage's linear layers (forward, input gradient and
// weight gradient with fused fp32 accumulation), gfx950.
//
// bf16: the ring kernel (gemm_pipe_kernel, 64 x 64 to 256 x 128 tiles) and the
// ping-pong kernel (gemm_pp_kernel, 256 x 256 and 256 x 128), both with
// direct-to-LDS loads. fp32 (gemm_kernel): one 256-thread workgroup (4
// wavefronts, 2 x 2) per 128 x 128, 64 x 64 or 32 x 32 output tile of 16 x 16
// MFMA tiles; the contracted dimension advances in 32-element slices,
// double-buffered in LDS, the global loads of slice k+1 in flight while slice k
// is multiplied. Operands stored contracted-major (K-major) are copied as
// 16-byte vectors and read as one 16-byte fragment; operands stored the other
// way (MN-major: the weight in dX = dY W, both activations in dW = dY^T X) are
// transposed in registers (4 x 4 blocks).
//
// Tile order is XCD-aware: workgroup w runs on XCD w % 8, so each XCD gets a
// contiguous range of tiles, walked in groups of 8 tile-rows to keep A and B
// panels in that XCD's L2.
#include "device_common.hpp"
#include <algorithm>
#include <cmath>

#include "kernels.hpp"

namespace paci {

int cu_count() {
  static int cus = 0;
  if (cus == 0) {
    int dev = 0, n = 0;
    if (hipGetDevice(&dev) == hipSuccess && hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) ==
                                                hipSuccess && n > 0)
      cus = n;
    else
      cus = 256;
  }
  return cus;
}

// fp32 products: the largest tile edge that still gives two workgroups per CU,
// else the smallest. A 256 x 128 product over 512 runs two 128 x 128 tiles on
// the whole chip, or 32 of 32 x 32: 33 -> 8.4 us a launch over its calls with
// K 128 and 512 (matrix work is 2.4, 0.7 and 0.45 us per 32-deep k-tile at 128,
// 64 and 32, the last two bound by the latency of the loads). us on 128 / 64 / 32
// at K 512, forward and input gradient, by tiles of 128 x 128: 384 of them 78 / 67 /
// 75 and 80 / 73 / 90; 512 79 / 86 / 97 and 80 / 97 / 118; weight gradients 2048 x
// 512 over 8192 rows 241 / 204 / 261. A single whole round of 128 x 128 tiles is 2
// to 9% faster than 64 x 64 (256 tiles: 49 / 53 / 52, 48 / 54 / 64) but not taken:
// with one chain of sums for four a block's output is further from 64 bits (512 wide,
// 2048 tokens: 1.5e-7 against 1.1e-7; 1024 wide, 4096 tokens: 5.9e-7 against 4.0e-7).
int gemm_f32_tile(int M, int N, int splits) {
  for (int e = 128; e > 32; e /= 2)
    if ((int64_t)((M + e - 1) / e) * ((N + e - 1) / e) * splits >= 2 * cu_count()) return e;
  return 32;
}

// Products with both operands K-major, by the rounds their tiles take on the CUs.
// Grids that leave CUs idle: the largest tiles that still fit one round. A
// k-tile takes about 0.2 us on 64 x 64 tiles, 0.24 on 128 x 64, 0.36 on
// 128 x 128 and 0.6-0.8 on 256 x 128, so below one round of tiles the
// smaller ones win (128 x 768 x 3072: 34.1 us on 256 x 128, 12.8 on 64 x
// 64; 2048 x 768 x 3072: 36.9, 21.9 on 384 of 64 x 64, 18.3 on 192 of 128
// x 64; 4096 x 1024 x 4096: 48.8, 54.4, 49.1, 38.5 on 256 of 128 x 128),
// above it the larger ones, which re-read the operands less.
// 256 x 256 ping-pong tiles where they take fewer rounds than 256 x 128 ring
// tiles, a round of them costing 1.8 of the others (whole rounds at 8192 x 4096
// x 1024, in the stage: FFN1 forward 106 -> 88.9 us, FFN2 input gradient 110 ->
// 82.2; at 8192 x 2048, mean of K 2048 and 8192: residual 163 -> 131, plain 157
// -> 131; qkv 8192 x 6144 x 2048: 209 -> 170).
// Columns of whole 256 x 256 rounds, the others in a launch of their own: 8192 x
// 3072 as 2048 + 1024, at K 1024 qkv 67 -> 36.9 + 23.4 us; at K 768 FFN1 forward
// 68.6 -> 39.3 + 24.4, FFN2 input gradient 65 -> 36.4 + 25.0; qkv 8192 x 2304 x
// 768 (2048 + 256) 54.5 -> 29.9 + 9.5.
// The rest: 256 x 128 ring tiles, which re-read the weights half as often as
// 128 x 128 ones.
KmajorPlan gemm_kmajor_plan(int M, int N) {
  const int64_t cus = cu_count(), tm = (M + 255) / 256;
  auto tiles = [&](int bm, int bn) { return (int64_t)((M + bm - 1) / bm) * ((N + bn - 1) / bn); };
  if (tiles(64, 64) <= cus) return {KT_64x64, 0};
  if (tiles(128, 64) <= cus) return {KT_128x64, 0};
  if (tiles(128, 128) <= cus) return {KT_128x128, 0};
  auto rounds = [&](int64_t n, int bn) { return (double)((tm * ((n + bn - 1) / bn) + cus - 1) / cus); };
  const double wide = 1.8 * rounds(N, 256), narrow = rounds(N, 128);
  const int64_t per = cus % tm == 0 ? cus / tm * 256 : 0, n1 = per > 0 ? N / per * per : 0;
  if (n1 > 0 && n1 < N && 1.8 * rounds(n1, 256) + rounds(N - n1, 128) + 0.1 < std::min(wide, narrow))
    return {KT_PP_256x256, (int)n1};
  return {wide < narrow ? KT_PP_256x256 : KT_256x128, 0};
}

// Tiles and split-K count of a window weight gradient: long contractions over
// few output tiles, so K is split until one round of workgroups (the CUs) is
// full, each split at least 512 rows, and of the two tile widths the one with
// the least work per CU is taken, a 256 x 256 tile costing 1.8 of 256 x 128.
// Atomic adds grow with the splits, at most 32. At 768-wide blocks over 32768
// rows: 3072 x 768 in 207 us with the three-stage ring on 256 x 128 tiles (two
// rounds), 196 ping-pong, 172 on 252 of 256 x 256; 2304 x 768 170, 160, 138; 768
// x 768 114, 112, 93. About 60 us of each are the atomic adds, which cross the
// XCDs in memory. All four products of a block of other widths, the ring's rule
// (about 512 workgroups) and this one: 1024 946 and 791 us, 1280 1580 and 1123,
// 1536 2197 and 1697, 1600 2495 and 1856, 1792 3032 and 2137; 512 over 16384 rows
// 305 and 308.
WindowPlan gemm_window_plan(int M, int N, int64_t K) {
  WindowPlan best{128, 1};
  double best_t = 1e30;
  const int cus = cu_count();
  for (int bn : {256, 128}) {
    const int64_t tiles = (int64_t)((M + 255) / 256) * ((N + bn - 1) / bn), kt = (K + 63) / 64;
    const int64_t most = std::max<int64_t>(1, std::min<int64_t>(32, K / 512));
    const int sp = (int)std::max<int64_t>(1, std::min(most, cus / tiles));
    const double t = (double)((tiles * sp + cus - 1) / cus) * (double)((kt + sp - 1) / sp) * (bn == 256 ? 1.8 : 1.0);
    if (t < best_t) {
      best_t = t;
      best = {bn, sp};
    }
  }
  return best;
}

namespace {

constexpr int KVN = 8, GROUP_M = 8;

// Tile configuration: a BM x BN output tile per workgroup, WM x WN per wavefront.
// CH partial sums per output (an MFMA adds to every CH-th): the k-ranges of the
// small fp32 tiles are split over fewer workgroups than those of 128 x 128 ones,
// and in one chain their weight gradients were 13-30% further from a 64-bit
// product than on split 128 x 128 tiles (256-wide block, 600 tokens: 4.0e-7 with
// the splits, 4.5e-7 in one chain, 2.5e-7 in four; the block's output 8.1e-8,
// 8.1e-8, 5.2e-8). The MFMAs issue at the same rate either way.
template <int BM_, int BN_, int WM_, int WN_, int CH_ = 1>
struct Tile {
  static constexpr int CH = CH_;
  static constexpr int BM = BM_, BN = BN_, WM = WM_, WN = WN_;
  static constexpr int WAVES = (BM / WM) * (BN / WN);
  static constexpr int NT = 64 * WAVES;
};

// Register-staged tile loader (global -> registers -> LDS), fp32. K-major
// operands are copied as 16-byte vectors, MN-major ones loaded as 4 x 4 blocks
// and transposed in registers.
template <int ROWS, bool KMAJ, int NT>
struct TileLoader {
  static constexpr int V = Vec<float>::V;
  static constexpr int ITEMS = KMAJ ? ROWS * KVN : (ROWS / V) * KVN;
  static constexpr int PT = (ITEMS + NT - 1) / NT;
  static constexpr int NV = KMAJ ? 1 : V;
  u32x4 r[PT][NV];

  // rows [row0, row0+ROWS) of `rows_total`; contracted [k0, k0 + 8V) of k_end.
  __device__ __forceinline__ void load(const float* src, int64_t ld, int row0, int rows_total, int k0,
                                       int k_end, int tid) {
#pragma unroll
    for (int p = 0; p < PT; ++p) {
      const int it = tid + p * NT;
      if ((ITEMS % NT) != 0 && it >= ITEMS) continue;
      if (KMAJ) {
        const int kv = it % KVN, rr = it / KVN;
        const int row = row0 + rr, k = k0 + kv * V;
        u32x4 v = {0, 0, 0, 0};
        if (row < rows_total && k < k_end) {
          v = ld16(src + (int64_t)row * ld + k);
          if (k + V > k_end) v = vmask_tail<float>(v, k_end - k);
        }
        r[p][0] = v;
      } else {
        const int kv = it % KVN, rr = it / KVN;
        const int rb = row0 + rr * V;
#pragma unroll
        for (int j = 0; j < V; ++j) {
          const int k = k0 + kv * V + j;
          u32x4 v = {0, 0, 0, 0};
          if (k < k_end && rb < rows_total) {
            v = ld16(src + (int64_t)k * ld + rb);
            if (rb + V > rows_total) v = vmask_tail<float>(v, rows_total - rb);
          }
          r[p][j] = v;
        }
      }
    }
  }

  __device__ __forceinline__ void store(u32x4* tile, int tid) const {
#pragma unroll
    for (int p = 0; p < PT; ++p) {
      const int it = tid + p * NT;
      if ((ITEMS % NT) != 0 && it >= ITEMS) continue;
      if (KMAJ) {
        const int kv = it % KVN, rr = it / KVN;
        tile[lds_slot<ROWS>(kv, rr)] = r[p][0];
      } else {
        const int kv = it % KVN, rr = it / KVN;
        u32x4 out[V];
        transpose_block<float>(r[p], out);
#pragma unroll
        for (int i = 0; i < V; ++i) tile[lds_slot<ROWS>(kv, rr * V + i)] = out[i];
      }
    }
  }

  // operand fragment of MFMA step s for the 16 rows starting at row0
  __device__ __forceinline__ static u32x4 frag(const u32x4* tile, int s, int row0) {
    return lds_frag<ROWS>(tile, s, row0);
  }
};

// GELU, tanh form: gelu(u) = u (1 + tanh z) / 2 with z = c (u + a u^3). Since
// (1 + tanh z) / 2 is the logistic function of 2z, s = 1 / (1 + 2^(-2 z log2 e)),
// it is u s, and its derivative s + 2 c u s (1 - s) (1 + 3 a u^2). One hardware
// exp2 and one reciprocal (about 1 ulp each); s saturates to 0 or 1.
__device__ __forceinline__ float gelu_sig(float u, float u2) {
  const float k = -2.0f * 1.4426950408889634f * 0.7978845608028654f;   // -2 c log2 e
  return __builtin_amdgcn_rcpf(1.0f + fast_exp2(k * u * fmaf(0.044715f, u2, 1.0f)));
}
// The derivative from u, u^2 and s: s + s (1 - s) u (2c + 6ac u^2).
__device__ __forceinline__ float gelu_grad_s(float u, float u2, float sg) {
  constexpr float c2 = 2.0f * 0.7978845608028654f, c6a = 6.0f * 0.044715f * 0.7978845608028654f;
  return fmaf(fmaf(-sg, sg, sg), u * fmaf(c6a, u2, c2), sg);
}
// The FFN up-projection's epilogue keeps gelu'(u) for the backward instead of
// u, the only use of u there: both values then share one exponential and one
// reciprocal, and the down-projection's input gradient only multiplies.
__device__ __forceinline__ void gelu_and_grad(float u, float& g, float& dg) {
  const float u2 = u * u, sg = gelu_sig(u, u2);
  g = u * sg;
  dg = gelu_grad_s(u, u2, sg);
}

// Write four consecutive outputs C[m][n .. n+3].
__device__ __forceinline__ void store4(float* C, int64_t idx, const float* v, int nvalid) {
  if (nvalid >= 4)
    st16(C + idx, u32x4{__builtin_bit_cast(uint32_t, v[0]), __builtin_bit_cast(uint32_t, v[1]),
                        __builtin_bit_cast(uint32_t, v[2]), __builtin_bit_cast(uint32_t, v[3])});
  else
    for (int j = 0; j < nvalid; ++j) C[idx + j] = v[j];
}

template <int EPI>
__device__ __forceinline__ void epilogue(const GemmArgs& a, int m, int n, const floatx4& acc) {
  if (m >= a.M || n >= a.N) return;
  const int nv = min(4, a.N - n);
  float* C = reinterpret_cast<float*>(a.C);
  const int64_t at = (int64_t)m * a.ldc + n;
  if (EPI == EPI_ATOMIC) {
    for (int j = 0; j < nv; ++j) atomicAdd(C + at + j, acc[j]);
    return;
  }
  if (EPI == EPI_ACC) {
    if (nv == 4) {
      const u32x4 old = ld16(C + at);
      float o[4];
      for (int j = 0; j < 4; ++j) o[j] = vget<float>(old, j) + acc[j];
      store4(C, at, o, 4);
    } else {
      for (int j = 0; j < nv; ++j) C[at + j] += acc[j];
    }
    return;
  }
  float o[4], bias[4] = {0.f, 0.f, 0.f, 0.f}, aux[4] = {0.f, 0.f, 0.f, 0.f};
  constexpr bool HAS_BIAS = EPI == EPI_BIAS || EPI == EPI_BIAS_RES || EPI == EPI_BIAS_GELU;
  constexpr bool HAS_AUX = EPI == EPI_BIAS_RES || EPI == EPI_GELU_GRAD;
  const float* ap = reinterpret_cast<const float*>(a.aux) + (int64_t)m * a.ld_aux + n;
  if (nv == 4) {
    if (HAS_BIAS) {
      const u32x4 b = ld16(a.bias + n);
#pragma unroll
      for (int j = 0; j < 4; ++j) bias[j] = vget<float>(b, j);
    }
    if (HAS_AUX) {
      const u32x4 x = ld16(ap);
#pragma unroll
      for (int j = 0; j < 4; ++j) aux[j] = vget<float>(x, j);
    }
  } else {
    for (int j = 0; j < nv; ++j) {
      if (HAS_BIAS) bias[j] = a.bias[n + j];
      if (HAS_AUX) aux[j] = ap[j];
    }
  }
  float g[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    float x = acc[j] + bias[j];
    if (EPI == EPI_BIAS_RES) x += aux[j];
    if (EPI == EPI_GELU_GRAD) x *= aux[j];
    if (EPI == EPI_BIAS_GELU) gelu_and_grad(x, g[j], x);
    o[j] = x;
  }
  store4(C, at, o, nv);
  if (EPI == EPI_BIAS_GELU) store4(reinterpret_cast<float*>(a.C2), at, g, nv);
}

__device__ __forceinline__ void tile_coords(int pid, int tiles_m, int tiles_n, int& tm, int& tn) {
  const int ntiles = tiles_m * tiles_n;
  int logical = pid;
  if ((ntiles & 7) == 0) logical = (pid & 7) * (ntiles >> 3) + (pid >> 3);
  const int group_size = GROUP_M * tiles_n;
  const int first_m = (logical / group_size) * GROUP_M;
  const int gm = min(tiles_m - first_m, GROUP_M);
  const int in_group = logical % group_size;
  tm = first_m + in_group % gm;
  tn = in_group / gm;
}

template <bool AK, bool BK, int EPI, class CF>
__global__ void __launch_bounds__(CF::NT, 1) gemm_kernel(GemmArgs a, int k_per_split) {
  constexpr int BM = CF::BM, BN = CF::BN, WM = CF::WM, WN = CF::WN, NT = CF::NT;
  constexpr int WAVES_N = BN / WN;
  constexpr int V = Vec<float>::V;
  constexpr int BKE = KVN * V;
  __shared__ u32x4 smem[2][(BM + BN) * KVN];
  const int tid = threadIdx.x, l = lane_id(), w = tid >> 6;
  const int tiles_m = (a.M + BM - 1) / BM, tiles_n = (a.N + BN - 1) / BN;
  int tm, tn;
  tile_coords(blockIdx.x, tiles_m, tiles_n, tm, tn);
  const int m0 = tm * BM, n0 = tn * BN;
  const int k_begin = blockIdx.y * k_per_split;
  const int k_end = min(a.K, k_begin + k_per_split);
  const int nk = (k_end - k_begin + BKE - 1) / BKE;
  const int wm0 = (w / WAVES_N) * WM, wn0 = (w % WAVES_N) * WN;

  const float* A = reinterpret_cast<const float*>(a.A);
  const float* B = reinterpret_cast<const float*>(a.B);
  TileLoader<BM, AK, NT> la;
  TileLoader<BN, BK, NT> lb;
  // MN-major operands load V x V blocks on part of the threads; spread A and B apart
  const int tid_b = (!AK && !BK) ? ((tid + NT / 2) % NT) : tid;

  constexpr int CH = CF::CH;
  floatx4 acc[CH][WM / 16][WN / 16];
#pragma unroll
  for (int c = 0; c < CH; ++c)
#pragma unroll
    for (int i = 0; i < WM / 16; ++i)
#pragma unroll
      for (int j = 0; j < WN / 16; ++j) acc[c][i][j] = floatx4{0.f, 0.f, 0.f, 0.f};

  if (nk > 0) {
    la.load(A, a.lda, m0, a.M, k_begin, k_end, tid);
    lb.load(B, a.ldb, n0, a.N, k_begin, k_end, tid_b);
    la.store(smem[0], tid);
    lb.store(smem[0] + BM * KVN, tid_b);
  }
  __syncthreads();
  for (int kt = 0; kt < nk; ++kt) {
    const int cur = kt & 1;
    if (kt + 1 < nk) {
      const int kn = k_begin + (kt + 1) * BKE;
      la.load(A, a.lda, m0, a.M, kn, k_end, tid);
      lb.load(B, a.ldb, n0, a.N, kn, k_end, tid_b);
    }
    const u32x4* sa = smem[cur];
    const u32x4* sb = smem[cur] + BM * KVN;
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      u32x4 yf[WM / 16], xf[WN / 16];
#pragma unroll
      for (int i = 0; i < WM / 16; ++i) yf[i] = TileLoader<BM, AK, NT>::frag(sa, s, wm0 + i * 16);
#pragma unroll
      for (int j = 0; j < WN / 16; ++j) xf[j] = TileLoader<BN, BK, NT>::frag(sb, s, wn0 + j * 16);
#pragma unroll
      for (int i = 0; i < WM / 16; ++i)
#pragma unroll
        for (int j = 0; j < WN / 16; ++j)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const uint32_t xw = xf[j][q], yw = yf[i][q];
            floatx4& c = acc[q % CH][i][j];
            c = __builtin_amdgcn_mfma_f32_16x16x4f32(as_float(xw), as_float(yw), c, 0, 0, 0);
          }
    }
    if (kt + 1 < nk) {
      la.store(smem[cur ^ 1], tid);
      lb.store(smem[cur ^ 1] + BM * KVN, tid_b);
    }
    __syncthreads();
  }
  // lane holds C[m][n .. n+3] with m = row (l % 16) of an A tile, n = 4 (l / 16) of a B tile
#pragma unroll
  for (int i = 0; i < WM / 16; ++i)
#pragma unroll
    for (int j = 0; j < WN / 16; ++j) {
#pragma unroll
      for (int h = CH / 2; h > 0; h /= 2)
#pragma unroll
        for (int c = 0; c < h; ++c) acc[c][i][j] += acc[c + h][i][j];
      epilogue<EPI>(a, m0 + wm0 + i * 16 + (l & 15), n0 + wn0 + j * 16 + 4 * (l >> 4), acc[0][i][j]);
    }
}

// ============================================================================================
// bf16 pipelined kernel: direct-to-LDS loads into an NS-stage ring.
//
// Each 16-byte slot of a tile is filled by global_load_lds_dwordx4. A wave
// instruction fills 64 consecutive slots, so the LDS layouts are chosen to be
// wave-contiguous:
//   K-major   [row][8 vectors of k], vector kv stored at kv ^ ((row >> 1) & 7);
//             8 lanes fetch one 128-byte row segment, and a 16-row fragment
//             read touches 16 distinct bank groups;
//   MN-major  [k][rows] with 16-byte chunk c of line k at c ^ trt_swz(k),
//             read by ds_read_b64_tr_b16 (see lds_frag_tr_at).
// Slots outside the operand (rows past M or N, k past K) are filled from a
// zero page, so the ring never holds stale data and the k tail sums exactly.
// The loads of tile kt + NS are issued right after the barrier that publishes
// tile kt + 1, into the stage of tile kt, which every wave has read by then.
// ============================================================================================
template <int BM_, int BN_, int WM_, int WN_, int NS_, int OCC_ = 1>
struct PipeTile {
  static constexpr int BM = BM_, BN = BN_, WM = WM_, WN = WN_, NS = NS_;
  static constexpr int OCC = OCC_;   // wavefronts per SIMD the register budget must allow
  static constexpr int WAVES = (BM / WM) * (BN / WN);
  static constexpr int NT = 64 * WAVES;
  static constexpr int SLOTS_A = BM * 8, SLOTS_B = BN * 8;       // 16-byte slots per tile
  static constexpr int LA = SLOTS_A / NT, LB = SLOTS_B / NT;     // loads per thread per tile
  static constexpr int STAGE_SLOTS = SLOTS_A + SLOTS_B;
  static_assert(SLOTS_A % NT == 0 && SLOTS_B % NT == 0, "tile slots must split evenly over the threads");
  // epilogue staging: PR rows of BN + 4 floats at a time, in the same LDS
  static constexpr int LDC = BN + 4;
  static constexpr int PR = (BM * LDC <= NS * STAGE_SLOTS * 4) ? BM : (BM > 128 ? 128 : BM);
  static constexpr int SMEM_SLOTS = (NS * STAGE_SLOTS > PR * LDC / 4) ? NS * STAGE_SLOTS : PR * LDC / 4;
  static_assert(BM % PR == 0 && PR % WM == 0 && (PR * LDC) % 4 == 0, "epilogue panels must align with wave rows");
};

__device__ __forceinline__ int kmaj_slot(int row, int kv) { return row * 8 + (kv ^ ((row >> 1) & 7)); }

template <int ROWS> __device__ __forceinline__ u32x4 pipe_frag_k(const u32x4* tile, int s, int row0) {
  const int l = lane_id();
  const int row = row0 + (l & 15), kv = s * 4 + (l >> 4);
  return tile[kmaj_slot(row, kv)];
}


// Issue load p (of ROWS * 8 / NT) of this thread's loads of one operand tile
// (ROWS rows x 64 contracted). `tile` is the LDS byte address of the operand's
// part of the stage, `w` the wave index (wave-uniform).
template <int ROWS, bool KMAJ, int NT>
__device__ __forceinline__ void pipe_fill_one(int p, const bf16* src, int64_t ld, int row0, int rows_total, int k0,
                                              int k_end, uint32_t tile, const void* zeros, int w, int l) {
  {
    const int blk = p * (NT / 64) + w;        // wave-uniform block of 64 slots
    const int slot = blk * 64 + l;
    const void* g;
    bool ok;
    if (KMAJ) {
      const int row = slot >> 3;
      const int kv = (slot & 7) ^ ((row >> 1) & 7);
      const int k = k0 + kv * 8;
      ok = (row0 + row < rows_total) && (k < k_end);
      g = src + (int64_t)(row0 + row) * ld + k;
    } else {
      constexpr int CPL = ROWS / 8;
      const int line = slot / CPL;
      const int c = (slot % CPL) ^ trt_swz<ROWS>(line);
      const int k = k0 + line, rb = row0 + c * 8;
      ok = (k < k_end) && (rb < rows_total);
      g = src + (int64_t)k * ld + rb;
    }
    dma16(ok ? g : zeros, tile + (uint32_t)(blk * 64 * 16));
  }
}

// The address of load p of this thread for contracted offset 0 (add k0 for a
// K-major operand, k0 rows for an MN-major one), with its row (K-major) or
// column group (MN-major) clamped into the operand: a clamped row only feeds
// outputs past M or N, which are never stored. Whole k-steps inside K then
// need one address add per load; the last, partial one takes pipe_fill_one,
// which reads the zero page for every slot outside the operand.
template <int ROWS, bool KMAJ, int NT>
__device__ __forceinline__ const bf16* pipe_fill_base(int p, const bf16* src, int64_t ld, int row0, int rows_total,
                                                      int w, int l) {
  const int blk = p * (NT / 64) + w;
  const int slot = blk * 64 + l;
  if (KMAJ) {
    const int row = slot >> 3;
    const int kv = (slot & 7) ^ ((row >> 1) & 7);
    return src + (int64_t)min(row0 + row, rows_total - 1) * ld + kv * 8;
  } else {
    constexpr int CPL = ROWS / 8;
    const int line = slot / CPL;
    const int c = (slot % CPL) ^ trt_swz<ROWS>(line);
    return src + (int64_t)line * ld + min(row0 + c * 8, (rows_total - 1) & ~7);
  }
}

// Output pass of the staged epilogue (every mode but the atomic one). A unit
// is one 16-byte store: 8 bf16 or 4 fp32 columns. Each thread keeps the same
// unit column for all its rows, so the bias is loaded once; the aux rows of
// all passes are loaded before any store, so their latencies overlap.
template <typename TO, int BN, int PR, int NT> struct EpiGeom {
  static constexpr int U = 16 / sizeof(TO), UPR = BN / U, RPI = NT / UPR, P = PR / RPI;
};
// The bf16 aux rows (residual or u) of a one-panel epilogue, loaded before the
// main loop so that their latency hides behind it: the same units staged_out
// gives this thread, one 16-byte load per row; zeros where staged_out will not
// use them (it then loads for itself).
template <typename TO, int BN, int PR, int NT>
__device__ __forceinline__ void prefetch_aux(const GemmArgs& a, int m0, int n0, int tid,
                                             u32x4 (&pre)[EpiGeom<TO, BN, PR, NT>::P]) {
  using G = EpiGeom<TO, BN, PR, NT>;
  static_assert(G::U == 8, "bf16 output units");
  const int n = n0 + (tid % G::UPR) * G::U, r0 = tid / G::UPR;
  const bf16* ap = reinterpret_cast<const bf16*>(a.aux);
  const bool ok = n + G::U <= a.N && a.ld_aux % 8 == 0 && (reinterpret_cast<uintptr_t>(ap) & 15) == 0;
#pragma unroll
  for (int p = 0; p < G::P; ++p) {
    const int m = m0 + r0 + p * G::RPI;
    pre[p] = (ok && m < a.M) ? ld16g(ap + (int64_t)m * a.ld_aux + n) : u32x4{0, 0, 0, 0};
  }
}

// The bias of this thread's output unit, loaded before the main loop as well.
template <typename TO, int BN, int PR, int NT>
__device__ __forceinline__ void prefetch_bias(const GemmArgs& a, int n0, int tid, float (&pb)[16 / sizeof(TO)]) {
  using G = EpiGeom<TO, BN, PR, NT>;
  const int n = n0 + (tid % G::UPR) * G::U;
#pragma unroll
  for (int j = 0; j < G::U; ++j) pb[j] = n + j < a.N ? a.bias[n + j] : 0.f;
}

template <typename TO, int EPI, int BN, int PR, int NT, bool PRE>
__device__ __forceinline__ void staged_out(const GemmArgs& a, const float* cl, int mb, int n0, int tid,
                                           float (&csum)[16 / sizeof(TO)],
                                           const u32x4 (&pre)[EpiGeom<TO, BN, PR, NT>::P],
                                           const float (&pb)[16 / sizeof(TO)]) {
  constexpr int U = 16 / sizeof(TO), UPR = BN / U, RPI = NT / UPR, P = PR / RPI;
  static_assert(NT % UPR == 0 && PR % RPI == 0, "units must tile the panel");
  constexpr int LDC = BN + 4;
  constexpr bool HAS_BIAS = EPI == EPI_BIAS || EPI == EPI_BIAS_RES || EPI == EPI_BIAS_GELU;
  constexpr bool HAS_AUX = EPI == EPI_BIAS_RES || EPI == EPI_GELU_GRAD;   // aux holds bf16 here
  const int cu = tid % UPR, r0 = tid / UPR;
  const int n = n0 + cu * U;
  if (n >= a.N) return;
  const int nv = min(U, a.N - n);
  auto al16 = [](const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; };
  const bool vec = nv == U && a.ldc % U == 0 && al16(a.C) && (EPI != EPI_BIAS_GELU || al16(a.C2)) &&
                   (!HAS_AUX || (a.ld_aux % 8 == 0 && al16(a.aux))) && (!HAS_BIAS || al16(a.bias));
  float bias[U];   // prefetched at kernel start (zero past the last column)
#pragma unroll
  for (int j = 0; j < U; ++j) bias[j] = HAS_BIAS ? pb[j] : 0.f;
  // EPI_ACC: every old value of this thread's units is loaded before the
  // first store, so the loads overlap (the compiler cannot order a load past
  // an earlier store to C, which might alias it)
  u32x4 acc_old[EPI == EPI_ACC ? P : 1];
  if constexpr (EPI == EPI_ACC) {
    const float* Cc = reinterpret_cast<const float*>(a.C);
#pragma unroll
    for (int p = 0; p < P; ++p) {
      const int m = mb + r0 + p * RPI;
      acc_old[p] = (vec && m < a.M) ? ld16g(Cc + (int64_t)m * a.ldc + n) : u32x4{0, 0, 0, 0};
    }
  }
  float aux[P][U];
  if constexpr (HAS_AUX) {
    const bf16* ap = reinterpret_cast<const bf16*>(a.aux);
#pragma unroll
    for (int p = 0; p < P; ++p) {
      const int m = mb + r0 + p * RPI;
      if (m < a.M) {
        const int64_t off = (int64_t)m * a.ld_aux + n;
        if (PRE && vec) {
#pragma unroll
          for (int j = 0; j < U; ++j) aux[p][j] = vget<bf16>(pre[p], j);
        } else if (vec) {
#pragma unroll
          for (int h = 0; h < U / 8 + (U < 8 ? 1 : 0); ++h) {
            if constexpr (U >= 8) {
              const u32x4 w = ld16g(ap + off + 8 * h);
#pragma unroll
              for (int j = 0; j < 8; ++j) aux[p][8 * h + j] = vget<bf16>(w, j);
            } else {
              const u32x2 w = *reinterpret_cast<const u32x2*>(ap + off);
#pragma unroll
              for (int j = 0; j < U; ++j) {
                const uint32_t word = w[j >> 1];
                aux[p][j] = as_float((j & 1) ? (word & 0xffff0000u) : (word << 16));
              }
            }
          }
        } else {
#pragma unroll
          for (int j = 0; j < U; ++j) aux[p][j] = j < nv ? (float)ap[off + j] : 0.f;
        }
      }
    }
  }
#pragma unroll
  for (int p = 0; p < P; ++p) {
    const int r = r0 + p * RPI, m = mb + r;
    if (m >= a.M) continue;
    float o[U], g2[EPI == EPI_BIAS_GELU ? U : 1];
#pragma unroll
    for (int q = 0; q < U / 4; ++q) {
      const floatx4 v = *reinterpret_cast<const floatx4*>(cl + r * LDC + cu * U + 4 * q);
#pragma unroll
      for (int j = 0; j < 4; ++j) o[4 * q + j] = v[j];
    }
    const int64_t off = (int64_t)m * a.ldc + n;
    if constexpr (EPI == EPI_ACC) {
      float* C = reinterpret_cast<float*>(a.C);
      if (vec) {
#pragma unroll
        for (int j = 0; j < 4; ++j) o[j] += as_float(acc_old[p][j]);
      } else {
#pragma unroll
        for (int j = 0; j < U; ++j)
          if (j < nv) o[j] += C[off + j];
      }
    } else if constexpr (EPI == EPI_CE_GRAD) {
      const float l = a.row_lse[m];
      const int y = a.row_tgt[m] - n;
#pragma unroll
      for (int j = 0; j < U; ++j) o[j] = a.alpha * (expf(o[j] - l) - (j == y ? 1.f : 0.f));
    } else {
#pragma unroll
      for (int j = 0; j < U; ++j) {
        float x = o[j] + bias[j];
        if constexpr (EPI == EPI_BIAS_RES) x += aux[p][j];
        if constexpr (EPI == EPI_GELU_GRAD) x *= aux[p][j];
        if constexpr (EPI == EPI_BIAS_GELU) gelu_and_grad(x, g2[j], x);
        o[j] = x;
      }
    }
    if (a.colsum != nullptr) {
#pragma unroll
      for (int j = 0; j < U; ++j)
        if (j < nv) csum[j] += o[j];
    }
    if constexpr (sizeof(TO) == 4 && (EPI == EPI_ACC || EPI == EPI_STORE)) {
      if (a.nonfinite != nullptr) {   // uniform
        bool bad = false;
#pragma unroll
        for (int j = 0; j < U; ++j) bad |= (j < nv) && !__builtin_isfinite(o[j]);
        if (bad) *a.nonfinite = 1;
      }
    }
    TO* C = reinterpret_cast<TO*>(a.C);
    if (vec) {
      if constexpr (sizeof(TO) == 2) {
        st16g(C + off, u32x4{pack_bf16x2(o[0], o[1]), pack_bf16x2(o[2], o[3]), pack_bf16x2(o[4], o[5]),
                            pack_bf16x2(o[6], o[7])});
      } else {
        st16g(C + off, u32x4{__builtin_bit_cast(uint32_t, o[0]), __builtin_bit_cast(uint32_t, o[1]),
                            __builtin_bit_cast(uint32_t, o[2]), __builtin_bit_cast(uint32_t, o[3])});
      }
    } else {
#pragma unroll
      for (int j = 0; j < U; ++j)
        if (j < nv) C[off + j] = from_f32<TO>(o[j]);
    }
    if constexpr (EPI == EPI_BIAS_GELU) {
      TO* C2 = reinterpret_cast<TO*>(a.C2);
#pragma unroll
      for (int j = 0; j < U; ++j) o[j] = g2[j];
      if (vec) {
        if constexpr (sizeof(TO) == 2)
          st16g(C2 + off, u32x4{pack_bf16x2(o[0], o[1]), pack_bf16x2(o[2], o[3]), pack_bf16x2(o[4], o[5]),
                               pack_bf16x2(o[6], o[7])});
        else
          st16g(C2 + off, u32x4{__builtin_bit_cast(uint32_t, o[0]), __builtin_bit_cast(uint32_t, o[1]),
                               __builtin_bit_cast(uint32_t, o[2]), __builtin_bit_cast(uint32_t, o[3])});
      } else {
#pragma unroll
        for (int j = 0; j < U; ++j)
          if (j < nv) C2[off + j] = from_f32<TO>(o[j]);
      }
    }
  }
}

// Cross-entropy row statistics of a staged panel (EPI_CE_STATS): per row and
// 64-column group, the maximum and the sum of exp(x - max) over the valid
// columns, and the target's logit when the group holds it. Consecutive lanes
// take consecutive rows; at row stride BN + 4 floats the 16-byte reads of 16
// lanes cover the 64 banks once.
template <int BN, int PR, int NT>
__device__ __forceinline__ void ce_stats_panel(const GemmArgs& a, const float* cl, int mb, int n0, int tid) {
  constexpr int LDC = BN + 4, G = BN / 64;
  static_assert(BN % 64 == 0, "64-column groups must tile the block");
  for (int idx = tid; idx < PR * G; idx += NT) {
    const int r = idx % PR, g = idx / PR;
    const int m = mb + r, nb = n0 + 64 * g;
    if (m >= a.M || nb >= a.N) continue;
    const int nv = min(64, a.N - nb);
    const float* row = cl + r * LDC + 64 * g;
    float mx = -INFINITY, sum = 0.f;
    // The sum is of exp(x - ref): a group of nothing but -inf has no finite maximum
    // to subtract, and sums to 0. (A NaN still makes the sum NaN.)
    auto ref_of = [](float m) { return m == -INFINITY ? 0.f : m; };
    if (nv == 64) {
      floatx4 v[16];
#pragma unroll
      for (int c = 0; c < 16; ++c) {
        v[c] = *reinterpret_cast<const floatx4*>(row + 4 * c);
        mx = fmaxf(fmaxf(mx, fmaxf(v[c][0], v[c][1])), fmaxf(v[c][2], v[c][3]));
      }
      const float ref = ref_of(mx);
#pragma unroll
      for (int c = 0; c < 16; ++c)
#pragma unroll
        for (int j = 0; j < 4; ++j) sum += expf(v[c][j] - ref);
    } else {
      for (int c = 0; c < nv; ++c) mx = fmaxf(mx, row[c]);
      const float ref = ref_of(mx);
      for (int c = 0; c < nv; ++c) sum += expf(row[c] - ref);
    }
    const int64_t q = (int64_t)m * a.ld_part + nb / 64;
    *reinterpret_cast<float2*>(a.ce_part + 2 * q) = make_float2(mx, sum);
    const int y = a.row_tgt[m] - nb;
    if (y >= 0 && y < nv) a.ce_zt[m] = row[y];
  }
}

// Epilogue through LDS. The accumulator tile goes to LDS as fp32 (row stride
// BN + 4 floats, so the 16 rows a wave writes at once fall in distinct banks)
// and is read back with consecutive lanes on consecutive columns: a wave then
// covers whole 256-byte row segments with each store, and each atomic add
// covers 64 consecutive floats. Tiles larger than the ring are done in row
// panels of PR rows.
// CF gives BM, BN, NT, PR and LDC; put(p) writes this wave's accumulators of
// panel p (rows p * PR ..) into the panel, row stride LDC.
template <typename TO, int EPI, class CF, bool PRE, class Put>
__device__ __forceinline__ void staged_epilogue(const GemmArgs& a, float* cl, int m0, int n0, Put&& put,
                                                const u32x4 (&pre)[EpiGeom<TO, CF::BN, CF::PR, CF::NT>::P],
                                                const float (&pb)[16 / sizeof(TO)]) {
  constexpr int BM = CF::BM, BN = CF::BN, NT = CF::NT, LDC = CF::LDC, PR = CF::PR;
  constexpr int U = 16 / sizeof(TO), UPR = BN / U;
  const int tid = threadIdx.x, l = lane_id();
  float csum[U];
#pragma unroll
  for (int j = 0; j < U; ++j) csum[j] = 0.f;
  // bf16 aux rows of a multi-panel epilogue: each panel's are loaded before its
  // staging, so their latency overlaps the staging and its barriers
  constexpr bool PANEL_AUX = (EPI == EPI_BIAS_RES || EPI == EPI_GELU_GRAD) && sizeof(TO) == 2 && !PRE;
#pragma unroll
  for (int p = 0; p < BM / PR; ++p) {
    u32x4 pre_p[PANEL_AUX ? EpiGeom<TO, BN, PR, NT>::P : 1];
    if constexpr (PANEL_AUX) prefetch_aux<TO, BN, PR, NT>(a, m0 + p * PR, n0, tid, pre_p);
    __syncthreads();   // every wave is done with the ring (or with the previous panel)
    put(p);
    __syncthreads();
    const int mb = m0 + p * PR;
    if constexpr (EPI == EPI_CE_STATS) {
      ce_stats_panel<BN, PR, NT>(a, cl, mb, n0, tid);
    } else if constexpr (EPI == EPI_ATOMIC) {
      float* C = reinterpret_cast<float*>(a.C);
      for (int idx = tid; idx < PR * BN; idx += NT) {
        const int r = idx / BN, c = idx % BN;
        const int m = mb + r, n = n0 + c;
        if (m < a.M && n < a.N) atomicAdd(C + (int64_t)m * a.ldc + n, cl[r * LDC + c]);
      }
    } else {
      if constexpr (EPI == EPI_STORE_CE) ce_stats_panel<BN, PR, NT>(a, cl, mb, n0, tid);
      if constexpr (PANEL_AUX) staged_out<TO, EPI, BN, PR, NT, true>(a, cl, mb, n0, tid, csum, pre_p, pb);
      else staged_out<TO, EPI, BN, PR, NT, PRE>(a, cl, mb, n0, tid, csum, pre, pb);
    }
  }
  if constexpr (EPI != EPI_ATOMIC && EPI != EPI_CE_STATS && UPR <= 64 && 64 % UPR == 0) {
    if (a.colsum != nullptr) {   // uniform: column sums of the tile's output into a.colsum
      // threads with equal tid % UPR hold the same columns: lanes l, l ^ UPR, ... within a
      // wavefront, then the wavefronts through LDS, then one atomic per column
#pragma unroll
      for (int j = 0; j < U; ++j)
#pragma unroll
        for (int off = UPR; off < 64; off *= 2) csum[j] += __shfl_xor(csum[j], off, 64);
      __syncthreads();   // every thread is done reading the staged tile
      const int w = tid >> 6;
      if (l < UPR) {
#pragma unroll
        for (int j = 0; j < U; ++j) cl[w * BN + l * U + j] = csum[j];
      }
      __syncthreads();
      for (int c = tid; c < BN; c += NT) {
        float sum = 0.f;
#pragma unroll
        for (int v = 0; v < NT / 64; ++v) sum += cl[v * BN + c];
        if (n0 + c < a.N) atomicAdd(a.colsum + n0 + c, sum);
      }
    }
  }
}

__device__ __forceinline__ const void* uniform_ptr(const void* p) {
  const uint64_t v = reinterpret_cast<uint64_t>(p);
  const uint32_t lo = __builtin_amdgcn_readfirstlane((int)(uint32_t)v), hi = __builtin_amdgcn_readfirstlane((int)(v >> 32));
  return reinterpret_cast<const void*>((uint64_t)hi << 32 | lo);
}
// This workgroup's output tile. Grouped weight gradients (GRP): its problem is
// found with wave-uniform scalar loads and put into `a`; false for the padding
// workgroups past a problem's tiles.
template <int BM, int BN, bool GRP>
__device__ __forceinline__ bool locate_tile(GemmArgs& a, int& m0, int& n0) {
  int pid = blockIdx.x;
  int xcd_m = 0;   // grouped weight gradients: XCD blocks of the tile grid (0: generic order)
  if constexpr (GRP) {
    int p = 0;
    while (p + 1 < a.group_n && pid >= a.group[p + 1].tile0) ++p;
    const WgradProblem& pr = a.group[p];
    pid -= __builtin_amdgcn_readfirstlane(pr.tile0);
    xcd_m = __builtin_amdgcn_readfirstlane(pr.xcd_m);
    a.A = uniform_ptr(pr.A);   // in scalar registers, whichever way they were loaded
    a.B = uniform_ptr(pr.B);
    a.C = pr.C;
    a.M = __builtin_amdgcn_readfirstlane(pr.M);
    a.N = __builtin_amdgcn_readfirstlane(pr.N);
    a.lda = a.M;
    a.ldb = a.N;
    a.ldc = a.N;
    if (pid >= ((a.M + BM - 1) / BM) * ((a.N + BN - 1) / BN)) return false;   // padding to a multiple of 8
  }
  const int tiles_m = (a.M + BM - 1) / BM, tiles_n = (a.N + BN - 1) / BN;
  int tm, tn;
  if (xcd_m > 0) {
    // XCD x = pid % 8 takes block (x % xcd_m, x / xcd_m) of bm x bn tiles, column by column
    const int x = pid & 7, k = pid >> 3;
    const int bm = tiles_m / xcd_m, bn = tiles_n / (8 / xcd_m);
    tm = (x % xcd_m) * bm + k % bm;
    tn = (x / xcd_m) * bn + k / bm;
  } else {
    tile_coords(pid, tiles_m, tiles_n, tm, tn);
  }
  m0 = tm * BM;
  n0 = tn * BN;
  return true;
}

// Scheduling pattern for one MFMA step: NREAD LDS reads (of the next step)
// spread evenly between NMFMA independent MFMAs (of this step).
template <int NREAD, int NMFMA>
__device__ __forceinline__ void interleave_reads() {
  constexpr int PER = NMFMA / NREAD > 0 ? NMFMA / NREAD : 1;
#pragma unroll
  for (int i = 0; i < NREAD; ++i) {
    __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);   // one DS read
    __builtin_amdgcn_sched_group_barrier(0x008, PER, 0); // PER MFMAs
  }
}

template <typename TO, bool AK, bool BK, int EPI, class CF, bool GRP = false>
__global__ void __launch_bounds__(CF::NT, CF::OCC) gemm_pipe_kernel(GemmArgs a, int k_per_split) {
  constexpr int BM = CF::BM, BN = CF::BN, WM = CF::WM, WN = CF::WN, NT = CF::NT, NS = CF::NS;
  constexpr int WAVES_N = BN / WN;
  constexpr int BKE = 64;
  constexpr int L = CF::LA + CF::LB;
  __shared__ u32x4 smem[CF::SMEM_SLOTS];
  const int tid = threadIdx.x, l = lane_id(), w = tid >> 6;
  int m0, n0;
  if (!locate_tile<BM, BN, GRP>(a, m0, n0)) return;
  const int k_begin = blockIdx.y * k_per_split;
  const int k_end = min(a.K, k_begin + k_per_split);
  const int nk = (k_end - k_begin + BKE - 1) / BKE;
  const int wm0 = (w / WAVES_N) * WM, wn0 = (w % WAVES_N) * WN;
  const bf16* A = reinterpret_cast<const bf16*>(a.A);
  const bf16* B = reinterpret_cast<const bf16*>(a.B);

  const uint32_t smem_lds = (uint32_t)(uintptr_t)((__attribute__((address_space(3))) u32x4*)smem);
  const int wu = __builtin_amdgcn_readfirstlane(w);
  // Per-thread load addresses at contracted offset 0. When every k-step lies
  // wholly inside K, a load is one address add (kf: true); fills past the last
  // k-step then repeat the last one's addresses, into stages that are never read.
  // Otherwise each load masks itself against K and the operand (pipe_fill_one).
  const bool kfull = k_end - k_begin >= BKE && (k_end - k_begin) % BKE == 0;   // uniform
  const bf16* fa[CF::LA];
  const bf16* fb[CF::LB];
#pragma unroll
  for (int p = 0; p < CF::LA; ++p) fa[p] = pipe_fill_base<BM, AK, NT>(p, A, a.lda, m0, a.M, wu, l);
#pragma unroll
  for (int p = 0; p < CF::LB; ++p) fb[p] = pipe_fill_base<BN, BK, NT>(p, B, a.ldb, n0, a.N, wu, l);
  // load p of the L loads of tile kt (the A operand's first, then B's)
  auto fill_one = [&](auto kf, int kt, int stage, int p) {   // stage = kt % NS
    const uint32_t st = smem_lds + (uint32_t)(stage * CF::STAGE_SLOTS * 16);
    const int k0 = k_begin + kt * BKE;
    if constexpr (decltype(kf)::value) {
      const int kc = min(k0, k_end - BKE);
      if (p < CF::LA) {
        const int blk = p * (NT / 64) + wu;
        dma16(fa[p] + (AK ? (int64_t)kc : (int64_t)kc * a.lda), st + (uint32_t)(blk * 64 * 16));
      } else {
        const int q = p - CF::LA, blk = q * (NT / 64) + wu;
        dma16(fb[q] + (BK ? (int64_t)kc : (int64_t)kc * a.ldb), st + CF::SLOTS_A * 16 + (uint32_t)(blk * 64 * 16));
      }
    } else if (p < CF::LA) {
      pipe_fill_one<BM, AK, NT>(p, A, a.lda, m0, a.M, k0, k_end, st, a.zeros, wu, l);
    } else {
      pipe_fill_one<BN, BK, NT>(p - CF::LA, B, a.ldb, n0, a.N, k0, k_end, st + CF::SLOTS_A * 16, a.zeros, wu, l);
    }
  };
  auto fill = [&](auto kf, int kt, int stage) {
#pragma unroll
    for (int p = 0; p < L; ++p) fill_one(kf, kt, stage, p);
  };

  floatx4 acc[WM / 16][WN / 16];
#pragma unroll
  for (int i = 0; i < WM / 16; ++i)
#pragma unroll
    for (int j = 0; j < WN / 16; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
  // bf16 residual or u rows of a one-panel epilogue: loaded now, used after the loop
  constexpr bool PRE = (EPI == EPI_BIAS_RES || EPI == EPI_GELU_GRAD) && sizeof(TO) == 2 && CF::PR == BM;
  u32x4 pre[EpiGeom<TO, BN, CF::PR, NT>::P];
  if constexpr (PRE) prefetch_aux<TO, BN, CF::PR, NT>(a, m0, n0, tid, pre);
  float pb[16 / sizeof(TO)];
  constexpr bool HAS_BIAS = EPI == EPI_BIAS || EPI == EPI_BIAS_RES || EPI == EPI_BIAS_GELU;
  if constexpr (HAS_BIAS) prefetch_bias<TO, BN, CF::PR, NT>(a, n0, tid, pb);

  // Fragments are double-buffered in registers: the LDS reads of the next
  // MFMA step are issued before the MFMAs of the current one. The barrier that
  // publishes tile kt + 1 sits between the two steps of tile kt; each wave
  // first waits for its own reads of tile kt, so after the barrier the stage of
  // tile kt is free and is refilled at once with tile kt + NS. Loads of a tile
  // are thus issued NS - 1 tiles of MFMA work before they are needed.
  u32x4 ya[WM / 16], xa[WN / 16], yb[WM / 16], xb[WN / 16];
  // MN-major operands: each fragment's transpose-read offset within its tile,
  // computed once (the swizzle makes it a non-affine function of the fragment)
  uint32_t tro_a[WM / 16], tro_b[WN / 16];
#pragma unroll
  for (int i = 0; i < WM / 16; ++i) tro_a[i] = AK ? 0u : lds_frag_tr_off<BM>(wm0 + i * 16);
#pragma unroll
  for (int j = 0; j < WN / 16; ++j) tro_b[j] = BK ? 0u : lds_frag_tr_off<BN>(wn0 + j * 16);
  // stage st (0 .. NS - 1) of the ring; the loop keeps st of k-steps kt and kt + 1
  auto read_step = [&](int st, int s, u32x4* yf, u32x4* xf) {
    const u32x4* sa = smem + st * CF::STAGE_SLOTS;
    const u32x4* sb = sa + CF::SLOTS_A;
    const uint32_t la = smem_lds + (uint32_t)(st * CF::STAGE_SLOTS * 16), lb = la + CF::SLOTS_A * 16;
#pragma unroll
    for (int i = 0; i < WM / 16; ++i)
      yf[i] = AK ? pipe_frag_k<BM>(sa, s, wm0 + i * 16) : lds_frag_tr_at<BM>(la + tro_a[i], s);
#pragma unroll
    for (int j = 0; j < WN / 16; ++j)
      xf[j] = BK ? pipe_frag_k<BN>(sb, s, wn0 + j * 16) : lds_frag_tr_at<BN>(lb + tro_b[j], s);
  };
  auto mma_all = [&](const u32x4* yf, const u32x4* xf) {
#pragma unroll
    for (int i = 0; i < WM / 16; ++i)
#pragma unroll
      for (int j = 0; j < WN / 16; ++j) mma_step<bf16>(acc[i][j], xf[j], yf[i]);
  };
  // fragment f of step s (A's fragments first, then B's), and MFMA q of a step
  auto read_frag = [&](int st, int s, int f, u32x4* yf, u32x4* xf) {
    const u32x4* sa = smem + st * CF::STAGE_SLOTS;
    const u32x4* sb = sa + CF::SLOTS_A;
    const uint32_t la = smem_lds + (uint32_t)(st * CF::STAGE_SLOTS * 16), lb = la + CF::SLOTS_A * 16;
    if (f < WM / 16) yf[f] = AK ? pipe_frag_k<BM>(sa, s, wm0 + f * 16) : lds_frag_tr_at<BM>(la + tro_a[f], s);
    else {
      const int j = f - WM / 16;
      xf[j] = BK ? pipe_frag_k<BN>(sb, s, wn0 + j * 16) : lds_frag_tr_at<BN>(lb + tro_b[j], s);
    }
  };
  auto mma_one = [&](int q, const u32x4* yf, const u32x4* xf) {
    const int i = q / (WN / 16), j = q % (WN / 16);
    mma_step<bf16>(acc[i][j], xf[j], yf[i]);
  };

  // The loop body has no branches: fills past the last tile read the zero page
  // and the reads after the last tile are discarded. Within each MFMA step the
  // scheduler spreads the LDS reads of the next step between the MFMAs.
  constexpr int NRI = (AK ? 1 : 2) * (WM / 16) + (BK ? 1 : 2) * (WN / 16);   // LDS read instructions per step
  constexpr int NM = (WM / 16) * (WN / 16);                                 // MFMAs per step
  constexpr int NF = WM / 16 + WN / 16;                                      // fragments per step
  // weight gradients (both operands MN-major, two workgroups per CU): raise the
  // wave's issue priority over its MFMA steps (measured 1.3% faster there,
  // slightly slower for the K-major products)
  constexpr bool PRIO = !AK && !BK;
  auto main_loop = [&](auto kf) {
#pragma unroll
    for (int t = 0; t < NS; ++t) fill(kf, t, t);
    wait_vmcnt<L * (NS - 1)>();
    barrier_no_fence();
    read_step(0, 0, ya, xa);
    int st0 = 0;   // ring stage of k-step kt
    for (int kt = 0; kt < nk; ++kt) {
      const int st1 = st0 + 1 == NS ? 0 : st0 + 1;   // of k-step kt + 1
      wait_lds_reads();     // reads of ya/xa, issued one MFMA step ago
      if constexpr (PRIO) __builtin_amdgcn_s_setprio(1);
      read_step(st0, 1, yb, xb);
      mma_all(ya, xa);
      interleave_reads<NRI, NM>();
      if constexpr (PRIO) __builtin_amdgcn_s_setprio(0);
      wait_lds_reads();     // reads of yb/xb
      wait_vmcnt<L * (NS - 2)>();   // tile kt + 1 has landed; kt + 2 .. kt + NS - 1 may be in flight
      barrier_no_fence();
      // Refill the stage of tile kt (every wave has read it) with tile kt + NS,
      // one load at a time between the MFMAs of this step and the reads of
      // the next: the loads of all waves of the CU reach the address unit
      // spread over the step instead of in one burst that holds up the MFMAs
      // (measured faster with every layout once a load is one address add; the
      // weight gradients also raise the wave's issue priority over the step).
      if constexpr (PRIO) __builtin_amdgcn_s_setprio(1);
#pragma unroll
      for (int p = 0; p < L; ++p) {
        fill_one(kf, kt + NS, st0, p);   // tile kt + NS reuses the stage of tile kt
#pragma unroll
        for (int f = p * NF / L; f < (p + 1) * NF / L; ++f) read_frag(st1, 0, f, ya, xa);
#pragma unroll
        for (int q = p * NM / L; q < (p + 1) * NM / L; ++q) mma_one(q, yb, xb);
        __builtin_amdgcn_sched_barrier(0);
      }
      if constexpr (PRIO) __builtin_amdgcn_s_setprio(0);
      st0 = st1;
    }
  };
  if (kfull) main_loop(std::true_type{});
  else main_loop(std::false_type{});
  wait_vmcnt<0>();   // the fills past the last tile, before the ring is reused
  float* cl = reinterpret_cast<float*>(smem);
  auto put = [&](int p) {
    if (wm0 < p * CF::PR || wm0 >= (p + 1) * CF::PR) return;
#pragma unroll
    for (int i = 0; i < WM / 16; ++i)
#pragma unroll
      for (int j = 0; j < WN / 16; ++j)
        *reinterpret_cast<floatx4*>(cl + (wm0 - p * CF::PR + i * 16 + (l & 15)) * CF::LDC + wn0 + j * 16 + 4 * (l >> 4)) =
            acc[i][j];
  };
  staged_epilogue<TO, EPI, CF, PRE>(a, cl, m0, n0, put, pre, pb);
}

// ============================================================================================
// bf16 ping-pong kernel: 256 x BN output tiles (BN = 256 or 128), 8 wavefronts.
//
// The wavefronts form two groups of four, one wavefront of each group per SIMD.
// Time runs in slots that end in a workgroup barrier; a wavefront alternates a
// memory slot (the LDS reads of its next 16 MFMAs, two or three direct-to-LDS
// loads of a later k-tile) with a matrix slot (those 16 MFMAs), and the groups
// are one slot apart, so in every slot one wavefront of each SIMD feeds the
// matrix cores while the other one reads and loads. A loop in which all eight
// wavefronts read, wait and multiply together left the matrix cores idle for
// half of the time (the waits of both wavefronts of a SIMD fell together).
//
// A k-tile is 64 contracted elements. Operands are kept in LDS as sub-tiles of
// 128 rows (16 KB), the layouts of the ring above: K-major [128][8 chunks],
// MN-major [64 k][128]. A wavefront's rows are two pieces, one per A sub-tile h
// (rows 128 h + 64 wm .. at BN = 256, 128 h + 32 wm .. at 128), so that an
// A sub-tile is read in one memory slot and refilled from the next one on.
//
// BN = 256 (2 x 4 wavefronts, four slot pairs per k-tile, two LDS stages):
//   pair 0: A_0 read     A_0 B_0     pair 1: B_1 read       A_0 B_1
//   pair 2: A_1 read     A_1 B_1     pair 3: next B_0 read  A_1 B_0
// 8, 4, 8 and 4 LDS reads per slot. The B fragments alternate between two
// register sets. Refills of k-tile t's stage with tile t + 2: B_0 in pair 1,
// A_0 in 2, B_1 in 3, A_1 in pair 0 of tile t + 1.
// BN = 128 (4 x 2 wavefronts, two pairs per k-tile, three A and four B stages):
//   pair 0: A_0, half of the next B read  A_0 B    pair 1: A_1, other half  A_1 B
// Refills: A_0 of tile t + 2 and half of B of t + 3 in pair 0, A_1 of t + 2 and
// half of B of t + 4 in pair 1.
//
// What bounds it: at 256 x 256 the loop runs at 93% of the MFMA issue rate
// (2205 cycles per k-tile against 2048; the ring kernel's 8-wavefront tiles
// took about 4200), and on random data the card then lowers its clock to
// 1.6-1.9 GHz: 1270 -> 1500 TFLOP/s on an 8192^3 product, where zeros run at
// 2.36 GHz and 1830. 256 x 128 tiles reach 1290 cycles against 1024 in the same
// product, but in the stage their loads come from beyond L2 and the deeper
// prefetch of the ring kernel wins (qkv 67 against 68-74 us), so only the LM
// head's input gradient and narrow window products, whose contractions are
// long, take them.
//
// Ordering. A wavefront waits for its LDS reads at the start of the matrix slot
// that follows them, so a sub-tile read by group 1 in slot s (group 0 is one
// slot earlier) is free for refills from slot s + 2 on, which is where the
// refills above are issued. Loads are waited for (vmcnt, in order) one memory
// slot before their first read, that is four (BN 256) or three (BN 128) memory
// slots after their issue, and a barrier lies between the wait and the read.
// ============================================================================================
template <int BN_> struct PP {
  static constexpr int BM = 256, BN = BN_, NT = 512;
  static constexpr int WR = BN == 256 ? 2 : 4, WC = 8 / WR;       // wavefront grid
  static constexpr int NH = BN / 128;                             // B sub-tiles
  static constexpr int TI = 128 / WR / 16, TJ = 128 / WC / 16;    // 16 x 16 tiles per wavefront and sub-tile pair
  static constexpr int SUB = 1024;                                // 16-byte slots per sub-tile
  static constexpr int SA = BN == 256 ? 2 : 3, SB = BN == 256 ? 2 : 4;   // LDS stages of A and of B
  static constexpr int RING = (SA * 2 + SB * NH) * SUB;
  static constexpr int LDC = BN + 4, PR = BN == 256 ? 128 : 256;  // epilogue panels
  static constexpr int SMEM_SLOTS = RING > PR * LDC / 4 ? RING : PR * LDC / 4;
};
template <int H> struct IC { static constexpr int value = H; };

// The loads of one operand: each sub-tile is 16 wave loads of 64 slots, two per
// wavefront. off: byte offset of load p of sub-tile h from the tile's base at
// the k-tile's first contracted element, rows past the operand clamped into it
// (they feed outputs that are not stored).
template <bool KMAJ, int NH>
struct PPOperand {
  static constexpr int NP = KMAJ ? 2 : 1;   // (MN-major: load 1 is 32 lines after load 0, no clamping between them)
  uint32_t off[NH][NP];
  const bf16* base;   // the tile's first row or column at contracted element 0 (uniform)
  int64_t ld;
  int kk;             // K-major: this thread's first contracted element in the k-tile; else its line of load 0

  __device__ __forceinline__ void init(const bf16* src, int64_t ld_, int row0, int rows_total, int w, int l) {
    ld = ld_;
    if (KMAJ) {
      base = src + (int64_t)row0 * ld;
      kk = 8 * ((l & 7) ^ (((w & 1) * 4 + (l >> 4)) & 7));
    } else {
      base = src + row0;
      kk = w * 4 + (l >> 4);
    }
#pragma unroll
    for (int h = 0; h < NH; ++h)
#pragma unroll
      for (int p = 0; p < NP; ++p) {
        if (KMAJ) {
          const int row = min(row0 + h * 128 + p * 64 + w * 8 + (l >> 3), rows_total - 1) - row0;
          off[h][p] = (uint32_t)(2 * (row * ld + kk));
        } else {
          const int c = (l & 15) ^ trt_swz<128>(kk);
          const int col = min(row0 + h * 128 + c * 8, (rows_total - 1) & ~7) - row0;
          off[h][p] = (uint32_t)(2 * (kk * ld + col));
        }
      }
  }
  // elements from contracted element 0 to k
  __device__ __forceinline__ int64_t at(int k) const { return KMAJ ? (int64_t)k : (int64_t)k * ld; }
  // Load P of sub-tile H of the k-tile whose first contracted element is at g,
  // to LDS byte address lds + IMM + (8 P) KB, lds including this wavefront's KB.
  template <int H, int P, int IMM> __device__ __forceinline__ void load(const bf16* g, uint32_t lds) const {
    dma16s<IMM + P * 8192>(KMAJ ? g : g + P * 32 * ld, off[H][KMAJ ? P : 0], lds);
  }
  // The same for a k-tile with only `valid` contracted elements inside K: slots
  // past them come from the zero page.
  template <int H, int P, int IMM>
  __device__ __forceinline__ void load_tail(const bf16* g, uint32_t lds, int valid, const void* zeros) const {
    const bool ok = KMAJ ? kk < valid : kk + 32 * P < valid;
    const void* q = reinterpret_cast<const char*>(KMAJ ? g : g + P * 32 * ld) + off[H][KMAJ ? P : 0];
    dma16(ok ? q : zeros, lds + IMM + P * 8192);
  }
};

template <typename TO, bool AK, bool BK, int EPI, int BN_, bool GRP = false>
__global__ void __launch_bounds__(512, 2) gemm_pp_kernel(GemmArgs a, int k_per_split) {
  using CF = PP<BN_>;
  constexpr int BM = CF::BM, BN = CF::BN, NT = CF::NT, TI = CF::TI, TJ = CF::TJ, NH = CF::NH, SUB = CF::SUB;
  __shared__ u32x4 smem[CF::SMEM_SLOTS];
  const int tid = threadIdx.x, l = lane_id();
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6), group = w >> 2;
  int m0, n0;
  if (!locate_tile<BM, BN, GRP>(a, m0, n0)) return;
  const int k_begin = blockIdx.y * k_per_split;
  const int k_end = min(a.K, k_begin + k_per_split);
  const int nk = (k_end - k_begin + 63) / 64;
  const int wm = w / CF::WC, wn = w % CF::WC;

  const uint32_t lds0 = (uint32_t)(uintptr_t)((__attribute__((address_space(3))) u32x4*)smem);
  const uint32_t ldsw = lds0 + (uint32_t)w * 1024;
  PPOperand<AK, 2> oa;
  PPOperand<BK, NH> ob;
  oa.init(reinterpret_cast<const bf16*>(a.A), a.lda, m0, a.M, w, l);
  ob.init(reinterpret_cast<const bf16*>(a.B), a.ldb, n0, a.N, w, l);
  // sub-tile h of A or B in LDS stage st, in slots from the start
  auto slot_a = [](int st, int h) { return (st * 2 + h) * SUB; };
  auto slot_b = [](int st, int h) { return (CF::SA * 2 + st * NH + h) * SUB; };
  // Contracted position of the next fills of A and of B: their addresses advance
  // by one k-tile at a time. B may come in segments of seg_rows contracted rows
  // (weight gradients; a k-tile never straddles two).
  const bf16* pa = oa.base + oa.at(k_begin);
  const bf16* pb_ = ob.base;
  const int64_t step_a = oa.at(64), step_b = ob.at(64);
  int seg_left = 0, seg = 0;
  const bool segs = !AK && !BK && !GRP && a.seg_rows > 0;   // uniform
  if (segs) {
    const int sg = k_begin / (int)a.seg_rows, r = k_begin - sg * (int)a.seg_rows;
    seg = (a.seg_first + sg) % a.seg_count;
    seg_left = (int)a.seg_rows - r;
    pb_ += (int64_t)seg * a.seg_stride + (int64_t)r * a.ldb;
  } else {
    pb_ += ob.at(k_begin);
  }
  auto next_a = [&] { pa += step_a; };
  auto next_b = [&] {
    pb_ += step_b;
    if (segs && (seg_left -= 64) <= 0) {
      seg = seg + 1 == a.seg_count ? 0 : seg + 1;
      seg_left = (int)a.seg_rows;
      pb_ = ob.base + (int64_t)seg * a.seg_stride;
    }
  };
  const int nfull = (k_end - k_begin) / 64;   // k-tiles wholly inside K
  // Load of k-tile kt: in the main loop (FULL) it lies wholly inside K; else it
  // may be the partial last one, or lie past the end (no load then).
  auto load_a = [&](auto full, int kt, uint32_t lds, auto h, auto p, auto imm) {
    if (decltype(full)::value || kt < nfull) oa.template load<h.value, p.value, imm.value>(pa, lds);
    else if (kt < nk) oa.template load_tail<h.value, p.value, imm.value>(pa, lds, k_end - k_begin - nfull * 64, a.zeros);
  };
  auto load_b = [&](auto full, int kt, uint32_t lds, auto h, auto p, auto imm) {
    if (decltype(full)::value || kt < nfull) ob.template load<h.value, p.value, imm.value>(pb_, lds);
    else if (kt < nk) ob.template load_tail<h.value, p.value, imm.value>(pb_, lds, k_end - k_begin - nfull * 64, a.zeros);
  };
  floatx4 acc[2][NH][TI][TJ];
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int g = 0; g < NH; ++g)
#pragma unroll
      for (int i = 0; i < TI; ++i)
#pragma unroll
        for (int j = 0; j < TJ; ++j) acc[h][g][i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
  // The bias, in registers by the epilogue. It is loaded after the last k-tile's
  // loads have been issued: vmcnt counts in order, so loaded at the start the first
  // k-tile would wait for it (measured 1.6 us of a 25 us product), and in the middle
  // a later one would. BN = 128 has no epilogue that takes a bias.
  constexpr bool HAS_BIAS = EPI == EPI_BIAS || EPI == EPI_BIAS_RES || EPI == EPI_BIAS_GELU;
  static_assert(BN == 256 || EPI == EPI_STORE || EPI == EPI_ACC || EPI == EPI_ATOMIC, "no loads but the k-tiles'");
  using EG = EpiGeom<TO, BN, CF::PR, NT>;
  u32x4 pre[EG::P];   // (aux rows are loaded panel by panel in the epilogue)
  float pb[EG::U];
  // n_late: the loads in flight behind the k-tiles' when they were all issued
  // unconditionally (whole columns, aligned), else 0 (the waits then cover them)
  constexpr int N_LATE = HAS_BIAS ? EG::U / 4 : 0;
  const bool whole = n0 + BN <= a.N && (reinterpret_cast<uintptr_t>(a.bias) & 15) == 0;   // uniform
  const int n_late = whole ? N_LATE : 0;
  auto late_loads = [&] {
    if constexpr (HAS_BIAS) {
      if (whole) {
        const int n = n0 + (tid % EG::UPR) * EG::U;
#pragma unroll
        for (int q = 0; q < EG::U / 4; ++q) {
          const u32x4 v = ld16g(a.bias + n + 4 * q);
#pragma unroll
          for (int j = 0; j < 4; ++j) pb[4 * q + j] = vget<float>(v, j);
        }
      } else {
        prefetch_bias<TO, BN, CF::PR, NT>(a, n0, tid, pb);
      }
    }
  };

  // Wait until at most n loads are outstanding: n in the main loop, and in the
  // last k-tiles (left = 1 for the last, 2, ..), where later loads are not
  // issued, n less those (l1, l2, ..). late: the epilogue's loads behind them.
  auto wait_but = [&](auto full, auto n, int late, int left, int l1, int l2, int l3 = -1, int l4 = -1) {
    if constexpr (decltype(full)::value) {
      wait_vmcnt<n.value>();
    } else {
      const int m = left <= 1 ? l1 : left == 2 ? l2 : left == 3 && l3 >= 0 ? l3 : left == 4 && l4 >= 0 ? l4 : n.value;
      if (late > 0) {   // (a smaller count waits for more)
        if (m >= 10) wait_vmcnt<10 + N_LATE>();
        else if (m >= 8) wait_vmcnt<8 + N_LATE>();
        else if (m >= 6) wait_vmcnt<6 + N_LATE>();
        else if (m >= 4) wait_vmcnt<4 + N_LATE>();
        else if (m >= 2) wait_vmcnt<2 + N_LATE>();
        else wait_vmcnt<N_LATE>();
        return;
      }
      switch (m) {
        case 10: wait_vmcnt<10>(); break;
        case 9: wait_vmcnt<9>(); break;
        case 8: wait_vmcnt<8>(); break;
        case 7: wait_vmcnt<7>(); break;
        case 6: wait_vmcnt<6>(); break;
        case 4: wait_vmcnt<4>(); break;
        case 2: wait_vmcnt<2>(); break;
        default: wait_vmcnt<0>(); break;
      }
    }
  };

  // fragment addresses: K-major, this lane's slot for step s of row 0 of the
  // sub-tile (16 rows further are 128 slots); MN-major, byte offset per fragment
  int ka[2], kb[2];   // (K-major)
  uint32_t ta[TI], tb[TJ];   // (MN-major)
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    ka[s] = kmaj_slot(wm * 16 * TI + (l & 15), s * 4 + (l >> 4));
    kb[s] = kmaj_slot(wn * 16 * TJ + (l & 15), s * 4 + (l >> 4));
  }
#pragma unroll
  for (int i = 0; i < TI; ++i) ta[i] = AK ? 0u : lds_frag_tr_off<128>((wm * TI + i) * 16);
#pragma unroll
  for (int j = 0; j < TJ; ++j) tb[j] = BK ? 0u : lds_frag_tr_off<128>((wn * TJ + j) * 16);
  auto frag_a = [&](int slot, int i, int s) -> u32x4 {
    if constexpr (AK) return smem[slot + ka[s] + i * 128];
    else return lds_frag_tr_at<128>(lds0 + 16 * slot + ta[i], s);
  };
  auto frag_b = [&](int slot, int j, int s) -> u32x4 {
    if constexpr (BK) return smem[slot + kb[s] + j * 128];
    else return lds_frag_tr_at<128>(lds0 + 16 * slot + tb[j], s);
  };
  u32x4 fa[TI][2], fb0[TJ][2], fb1[TJ][2];
  auto read_a = [&](int slot) {
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int i = 0; i < TI; ++i) fa[i][s] = frag_a(slot, i, s);
  };
  auto read_b = [&](int slot, u32x4 (&f)[TJ][2], int j0, int j1) {
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int j = 0; j < TJ; ++j)
        if (j >= j0 && j < j1) f[j][s] = frag_b(slot, j, s);
  };
  auto end_slot = [&] {
    __builtin_amdgcn_sched_barrier(0);
    barrier_no_fence();
    __builtin_amdgcn_sched_barrier(0);
  };
  auto matrix_slot = [&](floatx4 (&c)[TI][TJ], const u32x4 (&f)[TJ][2]) {
    wait_lds_reads();
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int i = 0; i < TI; ++i)
#pragma unroll
        for (int j = 0; j < TJ; ++j) mma_step<bf16>(c[i][j], f[j][s], fa[i][s]);
    __builtin_amdgcn_s_setprio(0);
    end_slot();
  };

  constexpr std::true_type FULL{};
  constexpr std::false_type TAIL{};
  if constexpr (BN == 256) {
    constexpr int SUBB = SUB * 16, STAGE = 2 * SUBB;   // bytes; A's stages, then B's
    // k-tile kt in stage st (its parity); x holds its B_0 fragments, y receives those of the next one
    auto late = [&](int kt) { return kt >= nk - 2 ? n_late : 0; };
    auto ktile = [&](auto full, int kt, auto st, u32x4 (&x)[TJ][2], u32x4 (&y)[TJ][2]) {
      constexpr int S = decltype(st)::value;
      constexpr IC<S * STAGE> A0{};
      constexpr IC<(S ^ 1) * STAGE + SUBB> A1{};
      constexpr IC<(2 + S) * STAGE> B0{};
      constexpr IC<(2 + S) * STAGE + SUBB> B1{};
      read_a(slot_a(S, 0));
      load_a(full, kt + 1, ldsw, IC<1>{}, IC<0>{}, A1);
      load_a(full, kt + 1, ldsw, IC<1>{}, IC<1>{}, A1);
      next_a();
      if (!decltype(full)::value && kt == nk - 2) late_loads();
      wait_but(full, IC<10>{}, late(kt), nk - kt, 2, 10);
      end_slot();
      matrix_slot(acc[0][0], x);

      read_b(slot_b(S, 1), y, 0, TJ);
      load_b(full, kt + 2, ldsw, IC<0>{}, IC<0>{}, B0);
      load_b(full, kt + 2, ldsw, IC<0>{}, IC<1>{}, B0);
      wait_but(full, IC<10>{}, late(kt), nk - kt, 0, 8);
      end_slot();
      matrix_slot(acc[0][1], y);

      read_a(slot_a(S, 1));
      load_a(full, kt + 2, ldsw, IC<0>{}, IC<0>{}, A0);
      load_a(full, kt + 2, ldsw, IC<0>{}, IC<1>{}, A0);
      wait_but(full, IC<10>{}, late(kt), nk - kt, 0, 6);
      end_slot();
      matrix_slot(acc[1][1], y);

      read_b(slot_b(S ^ 1, 0), y, 0, TJ);
      load_b(full, kt + 2, ldsw, IC<1>{}, IC<0>{}, B1);
      load_b(full, kt + 2, ldsw, IC<1>{}, IC<1>{}, B1);
      next_b();
      wait_but(full, IC<10>{}, late(kt), nk - kt, 0, 4);
      end_slot();
      matrix_slot(acc[1][0], x);
    };
    // the loads of tiles 0 and 1 that the loop does not issue, in the loop's order
    auto first = [&](int t, auto st) {
      constexpr int S = decltype(st)::value;
      load_b(TAIL, t, ldsw, IC<0>{}, IC<0>{}, IC<(2 + S) * STAGE>{});
      load_b(TAIL, t, ldsw, IC<0>{}, IC<1>{}, IC<(2 + S) * STAGE>{});
      load_a(TAIL, t, ldsw, IC<0>{}, IC<0>{}, IC<S * STAGE>{});
      load_a(TAIL, t, ldsw, IC<0>{}, IC<1>{}, IC<S * STAGE>{});
      load_b(TAIL, t, ldsw, IC<1>{}, IC<0>{}, IC<(2 + S) * STAGE + SUBB>{});
      load_b(TAIL, t, ldsw, IC<1>{}, IC<1>{}, IC<(2 + S) * STAGE + SUBB>{});
      if constexpr (S == 0) {
        load_a(TAIL, t, ldsw, IC<1>{}, IC<0>{}, IC<SUBB>{});
        load_a(TAIL, t, ldsw, IC<1>{}, IC<1>{}, IC<SUBB>{});
        next_a();
      }
      next_b();
    };
    first(0, IC<0>{});
    first(1, IC<1>{});
    if (nk < 2) late_loads();
    wait_but(TAIL, IC<10>{}, late(nk > 1 ? -1 : 0), nk + 1, 0, 4);   // B_0 and A_0 of tile 0
    end_slot();
    read_b(slot_b(0, 0), fb0, 0, TJ);
    if (group == 1) end_slot();
    int kt = 0;
    for (; kt + 3 < nfull; kt += 2) {
      ktile(FULL, kt, IC<0>{}, fb0, fb1);
      ktile(FULL, kt + 1, IC<1>{}, fb1, fb0);
    }
    for (; kt < nk; kt += 2) {
      ktile(TAIL, kt, IC<0>{}, fb0, fb1);
      if (kt + 1 < nk) ktile(TAIL, kt + 1, IC<1>{}, fb1, fb0);
    }
    if (group == 0) end_slot();
  } else {
    constexpr int SUBB = SUB * 16, AST = 2 * SUBB;   // bytes: sub-tile, stage of A
    const uint32_t ldsb = ldsw + CF::SA * AST;
    uint32_t sa = 0, sb = 0;   // byte offsets of the stages of A and B of tile kt
    const bf16* pb3 = pb_;     // B of tile kt + 3 (its second half is loaded one slot pair after the first)
    auto ktile = [&](auto full, int kt, u32x4 (&x)[TJ][2], u32x4 (&y)[TJ][2]) {
      const uint32_t sa2 = sa == 0 ? 2 * AST : sa - AST;                          // A of tile kt + 2 (and kt - 1)
      const uint32_t sb1 = (sb + SUBB) & (4 * SUBB - 1), sb3 = (sb + 3 * SUBB) & (4 * SUBB - 1);
      const int fra = (int)(sa >> 4), frb = (int)(sb1 >> 4) + CF::SA * 2 * SUB;
      read_a(fra);
      read_b(frb, y, 0, TJ / 2);
      load_a(full, kt + 2, ldsw + sa2, IC<0>{}, IC<0>{}, IC<0>{});
      load_a(full, kt + 2, ldsw + sa2, IC<0>{}, IC<1>{}, IC<0>{});
      {
        const bf16* cur = pb_;
        pb_ = pb3;
        load_b(full, kt + 3, ldsb + sb3, IC<0>{}, IC<1>{}, IC<0>{});
        pb_ = cur;
      }
      wait_but(full, IC<9>{}, 0, nk - kt, 0, 4, 7);
      end_slot();
      matrix_slot(acc[0][0], x);

      read_a(fra + SUB);
      read_b(frb, y, TJ / 2, TJ);
      load_a(full, kt + 2, ldsw + sa2, IC<1>{}, IC<0>{}, IC<SUBB>{});
      load_a(full, kt + 2, ldsw + sa2, IC<1>{}, IC<1>{}, IC<SUBB>{});
      load_b(full, kt + 4, ldsb + sb, IC<0>{}, IC<0>{}, IC<0>{});
      pb3 = pb_;
      next_a();
      next_b();
      wait_but(full, IC<9>{}, 0, nk - kt, 0, 2, 6, 8);
      end_slot();
      matrix_slot(acc[1][0], x);
      sa = sa == 2 * AST ? 0 : sa + AST;
      sb = sb1;
    };
    // the loads the loop does not issue, in its order
    load_b(TAIL, 0, ldsb, IC<0>{}, IC<0>{}, IC<0>{});
    load_b(TAIL, 0, ldsb, IC<0>{}, IC<1>{}, IC<0>{});
    next_b();
    load_b(TAIL, 1, ldsb, IC<0>{}, IC<0>{}, IC<SUBB>{});
    load_a(TAIL, 0, ldsw, IC<0>{}, IC<0>{}, IC<0>{});
    load_a(TAIL, 0, ldsw, IC<0>{}, IC<1>{}, IC<0>{});
    load_b(TAIL, 1, ldsb, IC<0>{}, IC<1>{}, IC<SUBB>{});
    next_b();
    load_a(TAIL, 0, ldsw, IC<1>{}, IC<0>{}, IC<SUBB>{});
    load_a(TAIL, 0, ldsw, IC<1>{}, IC<1>{}, IC<SUBB>{});
    next_a();
    load_b(TAIL, 2, ldsb, IC<0>{}, IC<0>{}, IC<2 * SUBB>{});
    load_a(TAIL, 1, ldsw, IC<0>{}, IC<0>{}, IC<AST>{});
    load_a(TAIL, 1, ldsw, IC<0>{}, IC<1>{}, IC<AST>{});
    load_b(TAIL, 2, ldsb, IC<0>{}, IC<1>{}, IC<2 * SUBB>{});
    next_b();
    load_a(TAIL, 1, ldsw, IC<1>{}, IC<0>{}, IC<AST + SUBB>{});
    load_a(TAIL, 1, ldsw, IC<1>{}, IC<1>{}, IC<AST + SUBB>{});
    next_a();
    load_b(TAIL, 3, ldsb, IC<0>{}, IC<0>{}, IC<3 * SUBB>{});
    pb3 = pb_;
    next_b();
    wait_but(TAIL, IC<9>{}, 0, nk + 1, 0, 2, 6, 8);   // B of tiles 0 and 1, A_0 of tile 0
    end_slot();
    read_b(slot_b(0, 0), fb0, 0, TJ);
    if (group == 1) end_slot();
    int kt = 0;
    for (; kt + 5 < nfull; kt += 2) {
      ktile(FULL, kt, fb0, fb1);
      ktile(FULL, kt + 1, fb1, fb0);
    }
    for (; kt < nk; kt += 2) {
      ktile(TAIL, kt, fb0, fb1);
      if (kt + 1 < nk) ktile(TAIL, kt + 1, fb1, fb0);
    }
    if (group == 0) end_slot();
  }
  wait_vmcnt<0>();
  wait_lds_reads();
  float* cl = reinterpret_cast<float*>(smem);
  auto put = [&](int p) {   // BN 256: panel p is A sub-tile p; 128: one panel of both
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      if (CF::PR == 128 && h != p) continue;
      const int r0 = (CF::PR == 128 ? 0 : h * 128) + wm * 16 * TI + (l & 15);
#pragma unroll
      for (int g = 0; g < NH; ++g)
#pragma unroll
        for (int i = 0; i < TI; ++i)
#pragma unroll
          for (int j = 0; j < TJ; ++j)
            *reinterpret_cast<floatx4*>(cl + (r0 + i * 16) * CF::LDC + g * 128 + (wn * TJ + j) * 16 + 4 * (l >> 4)) =
                acc[h][g][i][j];
    }
  };
  staged_epilogue<TO, EPI, CF, false>(a, cl, m0, n0, put, pre, pb);
}


// Tile configurations.
typedef Tile<128, 128, 64, 64> T128x128;
typedef Tile<64, 64, 32, 32, 4> T64x64;
typedef Tile<32, 32, 16, 16, 4> T32x32;

typedef PipeTile<256, 128, 64, 64, 3> P256x128;
typedef PipeTile<128, 128, 64, 64, 2, 2> P128x128o2;   // two workgroups per CU
// grids that leave CUs idle on the tiles above
typedef PipeTile<128, 128, 32, 64, 4, 2> P128x128w8;
typedef PipeTile<128, 64, 32, 32, 4, 2> P128x64;
typedef PipeTile<64, 64, 32, 32, 4, 2> P64x64;

template <typename TO, bool AK, bool BK, int EPI, class CF>
hipError_t launch_pipe(const GemmArgs& a, int splits, hipStream_t st) {
  constexpr int BKE = 64;
  const int tiles = ((a.M + CF::BM - 1) / CF::BM) * ((a.N + CF::BN - 1) / CF::BN);
  int kps = (a.K + splits - 1) / splits;
  kps = ((kps + BKE - 1) / BKE) * BKE;
  const int used = (a.K + kps - 1) / kps;
  hipLaunchKernelGGL((gemm_pipe_kernel<TO, AK, BK, EPI, CF>), dim3(tiles, used), dim3(CF::NT), 0, st, a, kps);
  return hipGetLastError();
}

template <typename TO, bool AK, bool BK, int EPI, int BN>
hipError_t launch_pp(const GemmArgs& a, int splits, hipStream_t st) {
  constexpr int BKE = 64;
  const int tiles = ((a.M + 255) / 256) * ((a.N + BN - 1) / BN);
  int kps = (a.K + splits - 1) / splits;
  kps = ((kps + BKE - 1) / BKE) * BKE;
  const int used = (a.K + kps - 1) / kps;
  hipLaunchKernelGGL((gemm_pp_kernel<TO, AK, BK, EPI, BN>), dim3(tiles, used), dim3(512), 0, st, a, kps);
  return hipGetLastError();
}


template <bool AK, bool BK, int EPI, class CF>
hipError_t launch_cf(const GemmArgs& a, int splits, hipStream_t st) {
  constexpr int BKE = KVN * Vec<float>::V;
  const int tiles = ((a.M + CF::BM - 1) / CF::BM) * ((a.N + CF::BN - 1) / CF::BN);
  int kps = (a.K + splits - 1) / splits;
  kps = ((kps + BKE - 1) / BKE) * BKE;
  const int used = (a.K + kps - 1) / kps;
  hipLaunchKernelGGL((gemm_kernel<AK, BK, EPI, CF>), dim3(tiles, used), dim3(CF::NT), 0, st, a, kps);
  return hipGetLastError();
}

template <bool AK, bool BK, int EPI>
hipError_t launch_f32(const GemmArgs& a, int splits, hipStream_t st) {
  if (a.seg_rows > 0) return hipErrorInvalidValue;
  hipError_t e;
  switch (gemm_f32_tile(a.M, a.N, splits)) {
    case 32: e = launch_cf<AK, BK, EPI, T32x32>(a, splits, st); break;
    case 64: e = launch_cf<AK, BK, EPI, T64x64>(a, splits, st); break;
    default: e = launch_cf<AK, BK, EPI, T128x128>(a, splits, st); break;
  }
  if constexpr (EPI != EPI_ATOMIC && EPI != EPI_ACC) {
    // the register-staged epilogue has no column sums: one pass over the output
    if (e == hipSuccess && a.colsum != nullptr) e = colsum_acc(DT_F32, a.C, a.ldc, a.M, a.N, a.colsum, st);
  }
  return e;
}

// The pipelined kernels move whole 16-byte chunks of 8 elements from global
// memory to LDS: bases and leading dimensions must be aligned to them. A chunk
// of a K-major operand that straddles K must be zero past it in A (the other
// operand's contracted rows are masked one by one): K a multiple of 8, or A
// zero-padded and B MN-major; both MN-major: any K. A chunk of an MN-major
// operand that straddles M or N only feeds outputs that are not stored, and
// must exist: M (N) a multiple of 8, or a leading dimension that covers the
// chunk. Other calls are refused: every bf16 operand of a stage is aligned (d and
// f are multiples of 32).
template <bool AK, bool BK>
bool pipe_eligible(const GemmArgs& a) {
  auto al16 = [](const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; };
  auto covers = [](int64_t ld, int n) { return n % 8 == 0 || ld >= (n + 7) / 8 * 8; };
  const bool k_ok = a.K % 8 == 0 || (!AK && !BK) || (AK && !BK && a.a_zero_pad);
  return a.zeros != nullptr && al16(a.A) && al16(a.B) && al16(a.zeros) && k_ok && a.lda % 8 == 0 && a.ldb % 8 == 0 &&
         (AK || covers(a.lda, a.M)) && (BK || covers(a.ldb, a.N));
}

// The ping-pong kernel addresses a sub-tile by a 32-bit byte offset, up to 255
// rows (K-major) or 31 lines (MN-major) from its base; the ring kernel's
// addresses are 64-bit. Longer rows (a vocabulary or FFN width of 8M and more)
// stay on the ring kernel.
template <bool AK, bool BK>
bool pp_reach(const GemmArgs& a) {
  return a.lda < (AK ? 1 << 23 : 1 << 26) && a.ldb < (BK ? 1 << 23 : 1 << 26);
}

// A segmented B: the window weight gradients.
template <int EPI>
hipError_t launch_window(const GemmArgs& a, int splits, hipStream_t st) {
  if (!pipe_eligible<false, false>(a) || !pp_reach<false, false>(a) || a.seg_rows % 64 || a.seg_count < 1 ||
      a.seg_first < 0)
    return hipErrorInvalidValue;
  return gemm_window_plan(a.M, a.N, a.K).bn == 256 ? launch_pp<float, false, false, EPI, 256>(a, splits, st)
                                                   : launch_pp<float, false, false, EPI, 128>(a, splits, st);
}

// Both operands K-major (a block's forward products and, on the transposed
// weights, its input gradients), on the tiles of gemm_kmajor_plan.
template <int EPI>
hipError_t launch_kmajor(const GemmArgs& a, hipStream_t st) {
  KmajorPlan plan = gemm_kmajor_plan(a.M, a.N);
  if (!pp_reach<true, true>(a) && (plan.tile == KT_PP_256x256 || plan.n1 > 0)) plan = {KT_256x128, 0};
  if (plan.n1 > 0) {
    GemmArgs r = a;
    r.N = plan.n1;
    const hipError_t e = launch_kmajor<EPI>(r, st);
    if (e != hipSuccess) return e;
    auto skip = [&](auto* p) { return p == nullptr ? p : p + plan.n1; };
    r.N = a.N - plan.n1;
    r.B = reinterpret_cast<const bf16*>(a.B) + plan.n1 * a.ldb;
    r.C = reinterpret_cast<bf16*>(a.C) + plan.n1;
    r.C2 = skip(reinterpret_cast<bf16*>(a.C2));
    r.bias = skip(a.bias);
    r.aux = skip(reinterpret_cast<const bf16*>(a.aux));
    r.colsum = skip(a.colsum);
    return launch_kmajor<EPI>(r, st);
  }
  switch (plan.tile) {
    case KT_64x64: return launch_pipe<bf16, true, true, EPI, P64x64>(a, 1, st);
    case KT_128x64: return launch_pipe<bf16, true, true, EPI, P128x64>(a, 1, st);
    case KT_128x128: return launch_pipe<bf16, true, true, EPI, P128x128w8>(a, 1, st);
    case KT_PP_256x256: return launch_pp<bf16, true, true, EPI, 256>(a, 1, st);
    default: break;
  }
  // The input gradient through gelu'(u): 128 x 128 tiles, two workgroups per CU, so
  // one's epilogue overlaps the other's loop (3-6% faster, and slower for the other
  // products: qkv 67 -> 69 us).
  if constexpr (EPI == EPI_GELU_GRAD) return launch_pipe<bf16, true, true, EPI, P128x128o2>(a, 1, st);
  else return launch_pipe<bf16, true, true, EPI, P256x128>(a, 1, st);
}

template <bool AK, bool BK, int EPI>
hipError_t launch_bf16(const GemmArgs& a, int splits, hipStream_t st) {
  if (!pipe_eligible<AK, BK>(a)) return hipErrorInvalidValue;
  if constexpr (AK && BK) {
    return launch_kmajor<EPI>(a, st);
  } else if constexpr (AK) {
    // An MN-major weight operand (the LM head's input gradient, K = V): 256 x 128
    // ping-pong tiles, whose partial last k-tile does not slow the others (8192 x
    // 1024 x 50257: 1118 us on the register-staged kernel, 683 now).
    if constexpr (EPI == EPI_STORE) {
      if (pp_reach<AK, BK>(a)) return launch_pp<bf16, AK, BK, EPI, 128>(a, splits, st);
    }
    if constexpr (EPI == EPI_GELU_GRAD) return launch_pipe<bf16, AK, BK, EPI, P128x128o2>(a, splits, st);
    else return launch_pipe<bf16, AK, BK, EPI, P256x128>(a, splits, st);
  } else {
    // weight gradients: 128 x 128 tiles, two workgroups per CU
    return launch_pipe<float, AK, BK, EPI, P128x128o2>(a, splits, st);
  }
}

template <DType DT, bool AK, bool BK, int EPI>
hipError_t launch(const GemmArgs& a, int splits, hipStream_t st) {
  if constexpr (DT == DT_F32) {
    return launch_f32<AK, BK, EPI>(a, splits, st);
  } else {
    if constexpr (!AK && !BK) {
      if (a.seg_rows > 0) return launch_window<EPI>(a, splits, st);
    }
    return a.seg_rows > 0 ? hipErrorInvalidValue : launch_bf16<AK, BK, EPI>(a, splits, st);
  }
}

// The softmax cross-entropy products.
hipError_t launch_ce(bool out_f32, GemmEpi epi, const GemmArgs& a, hipStream_t st) {
  if (!pipe_eligible<true, true>(a) || !pp_reach<true, true>(a) || a.row_tgt == nullptr || a.colsum != nullptr)
    return hipErrorInvalidValue;
  // 256 x 256 ping-pong tiles (8192 x 50257 x 1024: 1111 us storing fp32 logits on 256 x 128
  // ring tiles, 1115 with the statistics, which save a 950 us pass over the logits; without
  // logits 1079 -> 871 and 1203 -> 978 us). About 100 us of each are the exponentials: with a
  // once-rounded argument 2^(x log2 e) they took 1015, 736 and 872 us, but were off by up to
  // |x| 2^-24 where expf is good to an ulp.
  if (epi == EPI_CE_GRAD) {
    if (a.row_lse == nullptr || out_f32) return hipErrorInvalidValue;
    return launch_pp<bf16, true, true, EPI_CE_GRAD, 256>(a, 1, st);
  }
  if (a.ce_part == nullptr || a.ce_zt == nullptr || a.ld_part < (a.N + 63) / 64) return hipErrorInvalidValue;
  if (epi == EPI_STORE_CE) return launch_pp<float, true, true, EPI_STORE_CE, 256>(a, 1, st);
  return launch_pp<float, true, true, EPI_CE_STATS, 256>(a, 1, st);
}

template <DType DT>
hipError_t by_layout(bool out_f32, GemmLayout lay, GemmEpi epi, const GemmArgs& a, int splits, hipStream_t st) {
  if (epi == EPI_ACC || epi == EPI_ATOMIC) {
    // accumulation into fp32 is only used for weight gradients
    if (lay != GEMM_TN) return hipErrorInvalidValue;
    return epi == EPI_ACC ? launch<DT, false, false, EPI_ACC>(a, 1, st)
                          : launch<DT, false, false, EPI_ATOMIC>(a, splits, st);
  }
  if (splits != 1) return hipErrorInvalidValue;
  if (epi == EPI_CE_STATS || epi == EPI_STORE_CE || epi == EPI_CE_GRAD)
    return DT == DT_BF16 && lay == GEMM_NT ? launch_ce(out_f32, epi, a, st) : hipErrorInvalidValue;
  if (out_f32 && (DT == DT_BF16 || lay != GEMM_NT || epi != EPI_STORE)) return hipErrorInvalidValue;
  if (lay == GEMM_NT) {
    switch (epi) {
      case EPI_STORE: return launch<DT, true, true, EPI_STORE>(a, 1, st);
      case EPI_BIAS: return launch<DT, true, true, EPI_BIAS>(a, 1, st);
      case EPI_BIAS_RES: return launch<DT, true, true, EPI_BIAS_RES>(a, 1, st);
      case EPI_BIAS_GELU: return launch<DT, true, true, EPI_BIAS_GELU>(a, 1, st);
      case EPI_GELU_GRAD: return launch<DT, true, true, EPI_GELU_GRAD>(a, 1, st);
      default: return hipErrorInvalidValue;
    }
  }
  if (lay == GEMM_NN) {
    if (epi == EPI_STORE) return launch<DT, true, false, EPI_STORE>(a, 1, st);
    if (epi == EPI_GELU_GRAD) return launch<DT, true, false, EPI_GELU_GRAD>(a, 1, st);
  }
  return hipErrorInvalidValue;
}

}  // namespace

// Grouped weight gradients on 256 x 128 tiles (three-stage ring: 131 us for 256
// of them over 8192 rows, ping-pong 137) or 256 x 256 (ping-pong: 916 -> 814 us
// for 1024 of them), plain fp32 read-modify-write of each output tile.
namespace {
// f(CF{}) for the configuration of a tile shape
template <class F> auto with_tile(WgradTile t, F&& f) {
  switch (t) {
    case WG_256x256: return f(PP<256>{});
    case WG_128x128: return f(P128x128w8{});
    case WG_64x64: return f(P64x64{});
    default: return f(P256x128{});
  }
}
template <class CF> int group_tiles(int M, int N) { return ((M + CF::BM - 1) / CF::BM) * ((N + CF::BN - 1) / CF::BN); }
template <class CF> int group_xcd_m(int M, int N, int K) {
  const int tm = (M + CF::BM - 1) / CF::BM, tn = (N + CF::BN - 1) / CF::BN;
  int best = 0;
  double best_bytes = 0;
  for (int xm = 1; xm <= 8; xm *= 2) {
    const int xn = 8 / xm;
    if (tm % xm || tn % xn) continue;
    // panels one XCD reads: its bm row tiles of A and bn column tiles of B over K rows
    const double bytes = (double)K * 2.0 * ((tm / xm) * CF::BM + (tn / xn) * CF::BN);
    if (best == 0 || bytes < best_bytes) {
      best = xm;
      best_bytes = bytes;
    }
  }
  return best;
}
template <class CF, int EPI>
void launch_grouped(const GemmArgs& a, int total_tiles, int K, hipStream_t st) {
  if constexpr (CF::BN == 256)
    hipLaunchKernelGGL((gemm_pp_kernel<float, false, false, EPI, 256, true>), dim3(total_tiles, 1), dim3(CF::NT), 0, st, a, K);
  else
    hipLaunchKernelGGL((gemm_pipe_kernel<float, false, false, EPI, CF, true>), dim3(total_tiles, 1), dim3(CF::NT), 0, st, a, K);
}
}  // namespace

int wgrad_group_tiles(int M, int N, WgradTile tile) {
  return with_tile(tile, [&](auto cf) { return group_tiles<decltype(cf)>(M, N); });
}

int wgrad_group_xcd_m(int M, int N, int K, WgradTile tile) {
  return with_tile(tile, [&](auto cf) { return group_xcd_m<decltype(cf)>(M, N, K); });
}

int wgrad_group_split(const int* M, const int* N, int n, WgradTile* rest) {
  const int cus = cu_count();
  auto padded = [](int t) { return (t + 7) / 8 * 8; };
  auto total = [&](WgradTile t) {
    int64_t sum = 0;
    for (int p = 0; p < n; ++p) sum += padded(wgrad_group_tiles(M[p], N[p], t));
    return sum;
  };
  // few tiles: smaller ones, so that more CUs share the work (a k-tile takes
  // about 0.2 us on 64 x 64 tiles, 0.36 on 128 x 128 and 0.6-0.8 on 256 x 128)
  *rest = WG_256x128;
  if (total(WG_64x64) <= 2 * cus) *rest = WG_64x64;
  else if (total(WG_128x128) <= cus) *rest = WG_128x128;
  if (*rest != WG_256x128) return 0;
  // cost in rounds of 256 x 128 tiles; n1 = 0 is the single launch
  auto cost = [&](int n1) {
    int t1 = 0, t2 = 0;
    for (int p = 0; p < n; ++p) {
      if (p < n1) t1 += padded(wgrad_group_tiles(M[p], N[p], WG_256x256));
      else t2 += padded(wgrad_group_tiles(M[p], N[p], WG_256x128));
    }
    return 1.8 * ((t1 + cus - 1) / cus) + 1.0 * ((t2 + cus - 1) / cus);
  };
  int best = 0;
  double best_cost = cost(0);
  for (int n1 = n; n1 >= 1; --n1) {
    const double c = cost(n1);
    if (c < best_cost - 1e-9) {
      best = n1;
      best_cost = c;
    }
  }
  return best;
}

hipError_t gemm_wgrad_grouped(const WgradProblem* probs, int n, int total_tiles, int K, const void* zeros,
                              bool overwrite, WgradTile tile, int* nonfinite, hipStream_t st) {
  if (probs == nullptr || n < 1 || total_tiles < 1 || K < 1 || zeros == nullptr ||
      (reinterpret_cast<uintptr_t>(zeros) & 15))
    return hipErrorInvalidValue;
  GemmArgs a{};
  a.K = K;
  a.zeros = zeros;
  a.group = probs;
  a.group_n = n;
  a.nonfinite = nonfinite;
  with_tile(tile, [&](auto cf) {
    using CF = decltype(cf);
    if (overwrite) launch_grouped<CF, EPI_STORE>(a, total_tiles, K, st);
    else launch_grouped<CF, EPI_ACC>(a, total_tiles, K, st);
  });
  return hipGetLastError();
}

int gemm_acc_splits(DType dt, int M, int N, int K) {
  // Split-K count for Cf32 += A^T B. Cost model, in microseconds: rounds of
  // workgroups over the resident slots times the k-tiles each runs, plus the
  // fp32 read-modify-write or atomic adds of the epilogue (about 2 ps per
  // element and split).
  auto best_of = [&](auto cost) {
    int best = 1;
    double best_t = 1e30;
    for (int sp = 1; sp <= 16; sp *= 2) {
      const double t = cost(sp) + sp * 2e-6 * M * N;
      if (t < best_t * 0.97) {
        best_t = t;
        best = sp;
      }
    }
    return best;
  };
  if (dt == DT_BF16) {
    // 128 x 128 tiles, two workgroups per CU: about 2.3 TFLOP/s per CU, shared by them
    constexpr int BM = P128x128o2::BM, BN = P128x128o2::BN, OCC = P128x128o2::OCC;
    const double tiles = (double)((M + BM - 1) / BM) * ((N + BN - 1) / BN), t_k = 2.0 * BM * BN * 64 / (2.3e6 / OCC);
    const int kt = (K + 63) / 64;
    return best_of([&](int sp) {
      return sp > kt ? 1e30 : std::ceil(tiles * sp / (cu_count() * OCC)) * std::ceil((double)kt / sp) * t_k;
    });
  }
  // fp32: k-tiles of 32 on the tile edge for that many splits
  const int kt = (K + 31) / 32;
  return best_of([&](int sp) {
    if (sp > kt) return 1e30;
    const int e = gemm_f32_tile(M, N, sp);
    const double tiles = (double)((M + e - 1) / e) * ((N + e - 1) / e), t_k = e == 128 ? 2.4 : e == 64 ? 0.7 : 0.45;
    return std::ceil(tiles * sp / (2 * cu_count())) * std::ceil((double)kt / sp) * t_k;
  });
}

hipError_t gemm_wgrad(DType dt, const GemmArgs& a, hipStream_t st) {
  if (a.M <= 0 || a.N <= 0 || a.K <= 0 || a.colsum != nullptr || a.seg_rows > 0) return hipErrorInvalidValue;
  GemmArgs r = a;
  // At least one whole round of 256 x 256 tiles: that many whole rounds on the
  // ping-pong kernel and the remaining rows split over K, since a last partial
  // round would leave most CUs idle for as long as a full one. The 50257 x 1024
  // LM head over 8192 rows: 1453 us on the register-staged 128 x 128 kernel,
  // 625 (3 rounds) + 50 us now.
  if (dt == DT_BF16 && pipe_eligible<false, false>(a) && pp_reach<false, false>(a)) {
    const int cus = cu_count(), tn = (a.N + 255) / 256, tm = a.M / 256;
    const int rows_t = tn <= cus ? tm * tn / cus * cus / tn : 0;   // row tiles of the whole rounds
    if (rows_t > 0) {
      r.M = rows_t * 256;
      const hipError_t e = launch_pp<float, false, false, EPI_ACC, 256>(r, 1, st);
      if (e != hipSuccess || r.M == a.M) return e;
      r.A = reinterpret_cast<const bf16*>(a.A) + r.M;
      r.C = reinterpret_cast<float*>(a.C) + (int64_t)r.M * a.ldc;
      r.M = a.M - rows_t * 256;
    }
  }
  const int splits = gemm_acc_splits(dt, r.M, r.N, r.K);
  return gemm(dt, true, GEMM_TN, splits > 1 ? EPI_ATOMIC : EPI_ACC, r, splits, st);
}

hipError_t gemm(DType dt, bool out_f32, GemmLayout lay, GemmEpi epi, const GemmArgs& a, int splits,
                hipStream_t st) {
  if (a.M <= 0 || a.N <= 0 || a.K <= 0 || splits < 1) return hipErrorInvalidValue;
  if (a.colsum != nullptr && (epi == EPI_ACC || epi == EPI_ATOMIC)) return hipErrorInvalidValue;
  if (dt == DT_BF16) return by_layout<DT_BF16>(out_f32, lay, epi, a, splits, st);
  return by_layout<DT_F32>(out_f32, lay, epi, a, splits, st);
}

}  // namespace paci
