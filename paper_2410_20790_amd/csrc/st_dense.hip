// Dense convolutions of the reference pass (gfx950): implicit GEMM on MFMA
// whose operands go from global memory straight into LDS.
//
// The reference frame evaluates every output pixel, so a tile's rows are
// consecutive pixels and its gathered rows follow from the geometry.  What
// bounds these layers is streaming (the f32 state and the emitted rows of a
// 1x1 layer) or the chain load -> LDS -> MFMA of a long reduction with few
// tiles; both want many bytes in flight per CU and little per-tile work:
//
//  - The staged operands bypass the registers (16-byte global-to-LDS loads).
//    S stages are kept in S separate LDS arrays, so a stage's reads are known
//    not to alias the loads in flight and no wait but the counted one is
//    needed: one counted wait and one barrier per stage, with S - 1 stages
//    of loads outstanding.
//  - A staged row is 128 bytes in eight 16-byte slots; slot s of row r holds
//    the row's vector s ^ (r & 7) (weights: an equivalent permutation), set
//    by the address each lane loads from, so the MFMA operand reads are
//    conflict-free without padding.
//  - The weights are the MFMA's first operand: a lane's accumulators are then
//    consecutive channels of one pixel, and with the weight rows of two
//    16-channel blocks interleaved four by four, eight of them -- the lane
//    stores 32 bytes of state and 16 bytes of rows directly.  The accumulators
//    never go through LDS and the epilogue has no barrier.
//  - One block per tile (no persistent loop): a tile's loads never wait for
//    another tile's stores.  Blocks are dealt round-robin over the XCDs, so
//    each XCD takes a contiguous range of tiles, the channel tiles of one
//    pixel tile next to each other (they read the same pixels).
//
// Against the persistent register-staged 64x64 kernel that these layers took
// before (ResNet-50 at 1024x2048, bf16, us per layer): 1x1 64->256 with
// residual on 131072 pixels 93 -> 74 (285 MB, 3.9 TB/s), 1x1 512->128 on
// 32768 23 -> 16, 3x3 256 on 8192 40 (with its split epilogue) -> 21; the
// whole reference pass 2.05 -> 1.45 ms.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "st_device.h"
#include "st_kernels.h"
#include "st_stage.h"

namespace st {

namespace {

constexpr int kDenseXcd = 8;

// Which input rows an offset reads: a 1x1 kernel has one row per pixel; with
// a channel count that is a multiple of the stage's columns a stage lies
// within one offset; otherwise every lane walks its own (offset, channel).
enum { kSrcPoint = 0, kSrcAligned = 1, kSrcAny = 2 };

// One thread's share of the staged loads: PQ pixel vectors and WQ weight
// vectors per stage.
template <typename T, int KIND, int NW, int PQ, int WQ>
struct DenseLoader {
  static constexpr int VEC = 16 / (int)sizeof(T);
  static constexpr int KC = kRowBytes / (int)sizeof(T);
  const T* prow[PQ];  // the pixel vectors' input rows at offset k, or NULL
  const T* wrow[WQ];  // the weight vectors' rows, or NULL
  int iy[PQ], ix[PQ], nb[PQ];  // window origins, image * Hi
  int k, ci, wc;      // offset and channel; column of the weight row
  int next;           // (kSrcAligned) columns left of offset k
  int wave;

  __device__ __forceinline__ void rows_at(const ConvArgs& a) {
    const int ky = k / a.g.kw, kx = k - ky * a.g.kw;
#pragma unroll
    for (int q = 0; q < PQ; ++q) {
      const int y = iy[q] + ky, x = ix[q] + kx;
      const bool in = k < a.K && y >= 0 && y < a.g.Hi && x >= 0 && x < a.g.Wi;
      prow[q] = in ? (const T*)a.din +
                         (int64_t)((nb[q] + y) * a.g.Wi + x) * a.cin_p
                   : nullptr;
    }
  }

  // st: the first stage
  __device__ __forceinline__ void init(const ConvArgs& a, int64_t m0, int n0,
                                       int st, int lane, int wave_) {
    wave = wave_;
    const int lr = lane >> 3, slot = lane & 7;
    const unsigned hwo = (unsigned)a.g.Ho * (unsigned)a.g.Wo;
#pragma unroll
    for (int q = 0; q < PQ; ++q) {
      const int64_t o = m0 + (q * NW + wave) * 8 + lr;
      const unsigned op = o < a.capO ? (unsigned)o : 0u;
      const unsigned n = op / hwo, rem = op - n * hwo;
      const unsigned oy = rem / (unsigned)a.g.Wo;
      const unsigned ox = rem - oy * (unsigned)a.g.Wo;
      nb[q] = (int)n * a.g.Hi;
      iy[q] = (int)oy * a.g.sh - a.g.ph;
      ix[q] = o < a.capO ? (int)ox * a.g.sw - a.g.pw : -(1 << 28);
    }
    k = KIND == kSrcPoint ? 0 : st * KC / a.cin_p;
    next = (k + 1) * a.cin_p - st * KC;
    ci = st * KC - k * a.cin_p + (slot ^ lr) * VEC;
    if (KIND == kSrcAny) {
      while (ci >= a.cin_p) {
        ci -= a.cin_p;
        ++k;
      }
    }
    rows_at(a);
    wc = st * KC + (slot ^ ((lr & 3) | ((wave & 1) << 2))) * VEC;
#pragma unroll
    for (int q = 0; q < WQ; ++q) {
      const int n = n0 + (q * NW + wave) * 8 + lr;
      wrow[q] = n < a.cout_p ? (const T*)a.w + (int64_t)n * a.ktot_p : nullptr;
    }
  }

  // Issues the next stage's loads into the stage buffer `buf` (pixel rows,
  // then weight rows); past the reduction's end they read zeros.
  template <int BM>
  __device__ __forceinline__ void issue(const ConvArgs& a, char* buf) {
    const T* zero = (const T*)a.zero;
#pragma unroll
    for (int q = 0; q < PQ; ++q) {
      const bool ok = prow[q] && (KIND != kSrcPoint || ci < a.cin_p);
      load_to_lds(ok ? prow[q] + ci : zero,
                  buf + (q * NW + wave) * 8 * kRowBytes);
    }
#pragma unroll
    for (int q = 0; q < WQ; ++q) {
      const bool ok = wrow[q] && wc < (int)a.ktot_p;
      load_to_lds(ok ? wrow[q] + wc : zero,
                  buf + (BM + (q * NW + wave) * 8) * kRowBytes);
    }
    wc += KC;
    ci += KC;
    if (KIND == kSrcAligned) {
      next -= KC;
      if (next == 0) {
        next = a.cin_p;
        ci -= a.cin_p;
        ++k;
        rows_at(a);
      }
    } else if (KIND == kSrcAny) {
      if (ci >= a.cin_p) {
        do {
          ci -= a.cin_p;
          ++k;
        } while (ci >= a.cin_p);
        rows_at(a);
      }
    }
  }
};

// How a tile's reduction is summed: in one chain; in `parts` partial sums
// that the block adds in order; or block row y reduces part y of the stages
// and writes f32 partial rows part[y][pixel][channel], which the split
// epilogue adds in order and finishes.
enum { kSumChain = 0, kSumParts = 1, kSumSplit = 2 };

// Tile of BM pixels by BN channels in waves of WM by WN, S stages in LDS.
template <typename T, int KIND, int BM, int BN, int WM, int WN, int S,
          int SUM>
__global__ __launch_bounds__((BM / WM) * (BN / WN) * 64)
void k_dense_conv(ConvArgs a, int tiles_n, int tiles, int chunk, int parts) {
  constexpr bool SPLIT = SUM == kSumSplit;
  constexpr int WAVES_N = BN / WN, NW = BM / WM * WAVES_N;
  constexpr int PQ = BM / 8 / NW, WQ = BN / 8 / NW, L = PQ + WQ;
  constexpr int IM = WM / 16, JN = WN / 16;
  constexpr int KC = kRowBytes / (int)sizeof(T);
  static_assert(PQ * 8 * NW == BM && WQ * 8 * NW == BN && NW % 2 == 0 && JN % 2 == 0, "waves");
  static_assert(S >= 2 && S <= 4, "stages");
  constexpr int STAGE = (BM + BN) * kRowBytes;
  __shared__ __align__(128) char s0[STAGE];
  __shared__ __align__(128) char s1[STAGE];
  __shared__ __align__(128) char s2[S > 2 ? STAGE : 128];
  __shared__ __align__(128) char s3[S > 3 ? STAGE : 128];

  // this XCD's contiguous range of tiles, channel tiles fastest
  const int t = (int)(blockIdx.x % kDenseXcd) * chunk +
                (int)(blockIdx.x / kDenseXcd);
  if ((int)(blockIdx.x / kDenseXcd) >= chunk || t >= tiles) return;
  const int tm = t / tiles_n;
  const int64_t m0 = (int64_t)tm * BM;
  const int n0 = (t - tm * tiles_n) * BN;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int wm = wave / WAVES_N, wn = wave % WAVES_N;
  const int l16 = lane & 15, lg = lane >> 4;
  const int nst = (a.K * a.cin_p + KC - 1) / KC;
  const int st0 = SPLIT ? (int)blockIdx.y * nst / (int)gridDim.y : 0;
  const int st1 = SPLIT ? ((int)blockIdx.y + 1) * nst / (int)gridDim.y : nst;

  DenseLoader<T, KIND, NW, PQ, WQ> ld;
  ld.init(a, m0, n0, st0, lane, wave);

  // the lane's pixels and channels: pixel block i -> pixel pm + 16 i,
  // channel pair p -> channels cn + 32 p + [0, 8)
  const int64_t pm = m0 + wm * WM + l16;
  const int cn = n0 + wn * WN + lg * 8;
  const int cout_p = a.cout_p;

  v4f acc[IM][JN];
#pragma unroll
  for (int i = 0; i < IM; ++i)
#pragma unroll
    for (int j = 0; j < JN; ++j) acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};

  // the residual rows are requested first: they arrive with the first stage
  const T* dskip = !SPLIT && a.mskip ? (const T*)a.dskip : nullptr;
  constexpr int SKV = (int)sizeof(T) / 2;  // 16-byte vectors per 8 channels
  uint4 sk[JN / 2][IM][SKV];
#pragma unroll
  for (int p = 0; p < JN / 2; ++p)
#pragma unroll
    for (int i = 0; i < IM; ++i) {
      const int64_t o = pm + 16 * i;
      const int c = cn + 32 * p;
#pragma unroll
      for (int v = 0; v < SKV; ++v) {
        sk[p][i][v] = make_uint4(0u, 0u, 0u, 0u);
        if (dskip && o < a.capO && c < cout_p)
          sk[p][i][v] = ((const uint4*)(dskip + o * cout_p + c))[v];
      }
    }

  ld.template issue<BM>(a, s0);
  if constexpr (S > 2) ld.template issue<BM>(a, s1);
  if constexpr (S > 3) ld.template issue<BM>(a, s2);
  constexpr int AH = (S - 2) * L;
  const int pr = wm * WM, wr = BM + wn * WN;
  v4f sum[SUM == kSumParts ? IM : 1][SUM == kSumParts ? JN : 1];
  int part_end = nst, part = 0;
  if constexpr (SUM == kSumParts) {
    part_end = nst / parts;
#pragma unroll
    for (int i = 0; i < IM; ++i)
#pragma unroll
      for (int j = 0; j < JN; ++j) sum[i][j] = v4f{0.f, 0.f, 0.f, 0.f};
  }
  // the stage before `next` is done: the last of a part?
  auto part_done = [&](int next) {
    if constexpr (SUM == kSumParts) {
      if (next != part_end) return;
      ++part;
      part_end = (part + 1) * nst / parts;
#pragma unroll
      for (int i = 0; i < IM; ++i)
#pragma unroll
        for (int j = 0; j < JN; ++j) {
          sum[i][j] += acc[i][j];
          acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};
        }
    }
  };
  for (int st = st0; st < st1; st += S) {
    char* const last = S == 2 ? s1 : S == 3 ? s2 : s3;
    stage_turn<T, BM, AH>(a, ld, s0, last, pr, wr, l16, lg, acc);
    part_done(st + 1);
    if (st + 1 >= st1) break;
    stage_turn<T, BM, AH>(a, ld, s1, s0, pr, wr, l16, lg, acc);
    part_done(st + 2);
    if constexpr (S > 2) {
      if (st + 2 >= st1) break;
      stage_turn<T, BM, AH>(a, ld, s2, s1, pr, wr, l16, lg, acc);
      part_done(st + 3);
    }
    if constexpr (S > 3) {
      if (st + 3 >= st1) break;
      stage_turn<T, BM, AH>(a, ld, s3, s2, pr, wr, l16, lg, acc);
      part_done(st + 4);
    }
  }
  if constexpr (SUM == kSumParts) {  // (the last part's end is nst)
#pragma unroll
    for (int i = 0; i < IM; ++i)
#pragma unroll
      for (int j = 0; j < JN; ++j) acc[i][j] = sum[i][j];
  }

  if constexpr (SPLIT) {
    float* part = a.part + (int64_t)blockIdx.y * a.capO * cout_p;
#pragma unroll
    for (int p = 0; p < JN / 2; ++p)
#pragma unroll
      for (int i = 0; i < IM; ++i) {
        const int64_t o = pm + 16 * i;
        const int c = cn + 32 * p;
        if (o >= a.capO || c >= cout_p) continue;
        *(v4f*)(part + o * cout_p + c) = acc[i][2 * p];
        *(v4f*)(part + o * cout_p + c + 4) = acc[i][2 * p + 1];
      }
    return;
  }
  // epilogue: bias, residual row, activation; state and row stores
  T* dout = (T*)a.dout;
  with_act(a.act, [&](auto act_tag) {
    constexpr int ACT = decltype(act_tag)::value;
#pragma unroll
    for (int p = 0; p < JN / 2; ++p) {
      const int c = cn + 32 * p;
      if (c >= cout_p) continue;
      float bias[8];
      load8f(a.bias + c, bias);
#pragma unroll
      for (int i = 0; i < IM; ++i) {
        const int64_t o = pm + 16 * i;
        if (o >= a.capO) continue;
        float v[8], f[8];
        Vec8<T>::load((const T*)sk[p][i], f);
#pragma unroll
        for (int e = 0; e < 8; ++e)
          v[e] = acc[i][2 * p + (e >> 2)][e & 3] + bias[e] + f[e];
        if (a.mode != kModeLinear) {
#pragma unroll
          for (int e = 0; e < 8; ++e) v[e] = state_round(a.p16, v[e]);
          if (a.p16 || a.mode == kModeStateOnly) {
            // (a state without rows is read by the next launch: the pool,
            // the squeeze or the output)
            state_store8(a.P, a.p16, o * cout_p + c, v);
          } else {
            // the next reader of the state is another frame: streamed past
            // the caches, which keep the rows the next layer reads
            v4f* d = (v4f*)(a.P + o * cout_p + c);
            __builtin_nontemporal_store(v4f{v[0], v[1], v[2], v[3]}, d);
            __builtin_nontemporal_store(v4f{v[4], v[5], v[6], v[7]}, d + 1);
          }
          if (a.mode == kModeStateOnly) continue;
#pragma unroll
          for (int e = 0; e < 8; ++e) v[e] = act_c<ACT>(v[e]);
        }
        (void)Vec8<T>::store(dout + o * cout_p + c, v);
        if (a.ynew) store8f_rounded<T>(a.ynew + o * cout_p + c, v);
      }
    }
  });
}

template <typename T, int BM, int BN, int WM, int WN, int S, int SUM>
void dense_launch(hipStream_t s, const ConvArgs& a, int parts) {
  constexpr int KC = kRowBytes / (int)sizeof(T);
  constexpr int NT = (BM / WM) * (BN / WN) * 64;
  const int tiles_n = (a.cout_p + BN - 1) / BN;
  const int tiles = (int)((a.capO + BM - 1) / BM) * tiles_n;
  const int chunk = (tiles + kDenseXcd - 1) / kDenseXcd;
  const dim3 grid(chunk * kDenseXcd, SUM == kSumSplit ? parts : 1);
  if (a.K == 1)
    k_dense_conv<T, kSrcPoint, BM, BN, WM, WN, S, SUM>
        <<<grid, NT, 0, s>>>(a, tiles_n, tiles, chunk, parts);
  else if (a.cin_p % KC == 0)
    k_dense_conv<T, kSrcAligned, BM, BN, WM, WN, S, SUM>
        <<<grid, NT, 0, s>>>(a, tiles_n, tiles, chunk, parts);
  else
    k_dense_conv<T, kSrcAny, BM, BN, WM, WN, S, SUM>
        <<<grid, NT, 0, s>>>(a, tiles_n, tiles, chunk, parts);
}

// Tile shape by the tiles a launch has for the chip's 256 CUs (measured on
// the layers of a ResNet-50 at 1024x2048, bf16, us):
//  - 128x128, 3 stages, where that still makes 224 tiles: half the operand
//    traffic of 64x64 (512->256 on 32768 pixels: 27 against 32; 1024->512 on
//    8192: 18 against 24), one block of eight waves per CU (f32, which the
//    products bound: where the CU with the most tiles then has at most 15%
//    more products to do than with 128x64 tiles; 3x3 256 on 19200 pixels
//    309 against 244, 1152->192 on 50176 307 against 207);
//  - 128x64 where that makes 224 tiles: two blocks per CU with 3 stages (3x3
//    256 on 8192 pixels: 21 against 28 for 128x128), three with 2 stages when
//    the tiles go round the chip several times (3x3 64 on 131072: 27 against
//    30 with 3 stages);
//  - 64x64 with 4 stages else (3x3 512 on 2048 pixels: 28 against 35), and
//    128x32 for at most 32 channels, where half of a 64-channel tile would
//    be padding.
template <typename T, int SUM>
void dense_tiles(hipStream_t s, const ConvArgs& a, int parts) {
  const int64_t m128 = (a.capO + 127) / 128;
  const int64_t n64 = (a.cout_p + 63) / 64, n128 = (a.cout_p + 127) / 128;
  if (a.cout_p <= 32 && m128 >= 224)
    dense_launch<T, 128, 32, 32, 32, 3, SUM>(s, a, parts);
  else if (a.cout_p > 64 && m128 * n128 >= 224 &&
           (sizeof(T) == 2 ||
            40 * ((m128 * n128 + 255) / 256) <= 23 * ((m128 * n64 + 255) / 256)))
    dense_launch<T, 128, 128, 64, 32, 3, SUM>(s, a, parts);
  else if (SUM == kSumChain && m128 * n64 >= 1024)  // (parts: 1023 of 64x64)
    dense_launch<T, 128, 64, 32, 32, 2, kSumChain>(s, a, 1);
  else if (m128 * n64 >= 224)
    dense_launch<T, 128, 64, 32, 32, 3, SUM>(s, a, parts);
  else
    dense_launch<T, 64, 64, 32, 32, 4, SUM>(s, a, parts);
}

// A long reduction is summed in parts, as many as the diff frames' split
// (split_count of the 64x64 tiles, whatever tile the rule above takes), so
// that no chain of sums is longer and, in half precision, a state is the same
// sum in the same order whichever kernel computes it (f32 columns are added
// in another order).  With few tiles every part has a block of its own (half
// precision: fewer than 128; f32, whose products bound it: where the rule
// above would take 64x64), with more the block adds its parts itself.
template <typename T>
int dense_conv(hipStream_t s, const ConvArgs& a) {
  const int64_t tiles = ((a.capO + 63) / 64) * ((a.cout_p + 63) / 64);
  const int64_t t128 = ((a.capO + 127) / 128) * ((a.cout_p + 63) / 64);
  const int parts = split_count(tiles, a.split_max);
  if (parts > 1 && (sizeof(T) == 4 ? t128 < 224 : tiles < 128)) {
    dense_launch<T, 64, 64, 32, 32, 4, kSumSplit>(s, a, parts);
    return parts;
  }
  if (parts > 1)
    dense_tiles<T, kSumParts>(s, a, parts);
  else
    dense_tiles<T, kSumChain>(s, a, 1);
  return 1;
}

// Depthwise convolution of every pixel.  Its streams (rows in, f32 state out)
// would bound it, but on the small grids of the deeper layers the chain of
// dependent steps does, and the instructions a wave fetches: so a block loads
// the input patch of TH x 16 output pixels and OCT 8-channel vectors into LDS
// at once (no register staging, one wait), and rolled loops then read it: a
// thread takes 8 channels of a strip of four pixels, a window row at a time.
// EfficientNet-B0's 16 layers, 32 images of 256x256, bf16: 536 us with a
// thread per pixel, now 262 us; one image of 512x512, f16: 195 us, now 121.
constexpr int kDwPX = 4, kDwTW = 16;

template <typename T, int KS, int ST, int OCT, int TH>
struct DwTile {
  static constexpr int NT = TH * (kDwTW / kDwPX) * OCT, NW = NT / 64;
  static constexpr int RB = OCT * 8 * (int)sizeof(T);  // bytes of a patch row
  static constexpr int LPR = RB / 16, RPI = 64 / LPR;  // lanes per row, rows
  static constexpr int PH = (TH - 1) * ST + KS, PW = (kDwTW - 1) * ST + KS;
  static constexpr int ROWS = (PH * PW + RPI * NW - 1) / (RPI * NW) * RPI * NW;
};

template <typename T, int KS, int ST, int OCT, int TH, int ACT>
__device__ __forceinline__ void dense_dw_tile(const ConvArgs& a, int tiles_x,
                                               char* patch, float* wl) {
  using G = DwTile<T, KS, ST, OCT, TH>;
  constexpr int NX = (kDwPX - 1) * ST + KS;  // input columns of a strip
  constexpr int W = OCT * 8, V4 = W / 4;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int t = blockIdx.x, n = blockIdx.y, cp = a.cout_p;
  const int cb = (int)blockIdx.z * W;
  const Geo& q = a.g;
  // the slab's weights, two vectors per thread requested at a time
  const float* w = (const float*)a.w;
  for (int e0 = tid; e0 < KS * KS * V4; e0 += 2 * G::NT) {
    float4 r[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int e = e0 + G::NT * j, k = e / V4, c = cb + (e % V4) * 4;
      r[j] = *(const float4*)(k < KS * KS && c < cp ? w + k * cp + c
                                                    : (const float*)a.zero);
    }
#pragma unroll
    for (int j = 0; j < 2; ++j)
      if (e0 + G::NT * j < KS * KS * V4) ((float4*)wl)[e0 + G::NT * j] = r[j];
  }
  const int oct = tid % OCT, st = tid / OCT;
  const int ty = st / (kDwTW / kDwPX), sx = st % (kDwTW / kDwPX);
  const int c0 = cb + oct * 8;
  float bias[8];
  load8f(c0 < cp ? a.bias + c0 : (const float*)a.zero, bias);
  const int lrow = lane / G::LPR, lcol = lane % G::LPR * (16 / (int)sizeof(T));
  const int oy0 = t / tiles_x * TH, ox0 = t % tiles_x * kDwTW;
  const int iy0 = oy0 * ST - q.ph, ix0 = ox0 * ST - q.pw;
  // the patch, zeros outside the image
#pragma unroll 2
  for (int r0 = wave * G::RPI; r0 < G::ROWS; r0 += G::NW * G::RPI) {
    const int r = r0 + lrow, py = r / G::PW;
    const int iy = iy0 + py, ix = ix0 + r - py * G::PW;
    const bool in = py < G::PH && iy >= 0 && iy < q.Hi && ix >= 0 &&
                    ix < q.Wi && cb + lcol < cp;
    load_to_lds(in ? (const T*)a.din +
                         (int64_t)((n * q.Hi + iy) * q.Wi + ix) * cp + cb +
                         lcol
                   : (const T*)a.zero,
                patch + r0 * G::RB);
  }
  __syncthreads();  // (waits for the loads into LDS too)
  float acc[kDwPX][8];
#pragma unroll
  for (int p = 0; p < kDwPX; ++p)
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[p][e] = 0.f;
  const char* strip =
      patch + (ty * ST * G::PW + sx * kDwPX * ST) * G::RB +
      oct * 8 * (int)sizeof(T);
#pragma unroll 1
  for (int ky = 0; ky < KS; ++ky) {
    float wk[KS][8];
#pragma unroll
    for (int kx = 0; kx < KS; ++kx)
      load8f(wl + (ky * KS + kx) * W + oct * 8, wk[kx]);
#pragma unroll
    for (int j = 0; j < NX; ++j) {
      float x[8];
      Vec8<T>::load((const T*)(strip + (ky * G::PW + j) * G::RB), x);
#pragma unroll
      for (int p = 0; p < kDwPX; ++p) {
        const int kx = j - p * ST;
        if (kx < 0 || kx >= KS) continue;
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[p][e] += wk[kx][e] * x[e];
      }
    }
  }
  const int oy = oy0 + ty;
  const int64_t pix0 = ((int64_t)n * q.Ho + oy) * q.Wo + ox0 + sx * kDwPX;
  const int np = oy < q.Ho && c0 < cp
                     ? min(kDwPX, q.Wo - ox0 - sx * kDwPX)
                     : 0;
  // (rolled too: the pixel at hand is acc[0])
#pragma unroll 1
  for (int p = 0; p < np; ++p) {
    const int64_t at = (pix0 + p) * cp + c0;
    float v[8], sk[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) sk[e] = 0.f;
    if (a.mskip) Vec8<T>::load((const T*)a.dskip + at, sk);
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = acc[0][e] + bias[e] + sk[e];
#pragma unroll
    for (int r = 1; r < kDwPX; ++r)
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[r - 1][e] = acc[r][e];
    if (a.mode != kModeLinear) {
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = state_round(a.p16, v[e]);
      state_store8(a.P, a.p16, at, v);
      if (a.mode == kModeStateOnly) continue;
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = act_c<ACT>(v[e]);
    }
    (void)Vec8<T>::store((T*)a.dout + at, v);
    if (a.ynew) store8f_rounded<T>(a.ynew + at, v);
  }
}

template <typename T, int KS, int ST, int OCT, int TH>
__global__ __launch_bounds__(TH * (kDwTW / kDwPX) * OCT) void k_dense_dw(
    ConvArgs a, int tiles_x) {
  using G = DwTile<T, KS, ST, OCT, TH>;
  __shared__ __align__(16) char patch[G::ROWS * G::RB];
  __shared__ __align__(16) float wl[KS * KS * OCT * 8];
  with_act(a.act, [&](auto act_tag) {
    dense_dw_tile<T, KS, ST, OCT, TH, decltype(act_tag)::value>(a, tiles_x,
                                                                patch, wl);
  });
}

template <typename T, int KS, int ST, int OCT, int TH>
void dw_launch(hipStream_t s, const ConvArgs& a, int images) {
  const int tiles_x = (a.g.Wo + kDwTW - 1) / kDwTW;
  const dim3 grid(tiles_x * ((a.g.Ho + TH - 1) / TH), images,
                  (a.cout_p / 8 + OCT - 1) / OCT);
  k_dense_dw<T, KS, ST, OCT, TH>
      <<<grid, DwTile<T, KS, ST, OCT, TH>::NT, 0, s>>>(a, tiles_x);
}

// 8 vectors (128 bytes) of a half-precision pixel where that pads the channels
// by less than half a tile, else 4; f32: 4.
inline bool dw_wide(int dtype, const ConvArgs& a) {
  const int rest = a.cout_p / 8 % 8;
  return dtype != 0 && (rest == 0 || rest > 4);
}

// Tile height by what the patch leaves of LDS (stride 2: about four input
// pixels per output).
template <typename T, int KS>
void dense_dw(hipStream_t s, const ConvArgs& a, int images) {
  if constexpr (sizeof(T) == 2) {
    if (dw_wide(1, a)) {
      if (a.g.sh == 1)
        dw_launch<T, KS, 1, 8, 8>(s, a, images);
      else
        dw_launch<T, KS, 2, 8, 4>(s, a, images);
      return;
    }
  }
  constexpr int TH = sizeof(T) == 2 ? 16 : 8;
  if (a.g.sh == 1)
    dw_launch<T, KS, 1, 4, TH>(s, a, images);
  else
    dw_launch<T, KS, 2, 4, TH / 2>(s, a, images);
}

template <typename T>
void dense_dw(hipStream_t s, const ConvArgs& a, int images) {
  if (a.g.kh == 3)
    dense_dw<T, 3>(s, a, images);
  else
    dense_dw<T, 5>(s, a, images);
}

}  // namespace

bool dense_dw_takes(int dtype, const ConvArgs& a, int images) {
  const Geo& g = a.g;
  if (images > 65535 || g.kh != g.kw || (g.kh != 3 && g.kh != 5) ||
      g.sh != g.sw || (g.sh != 1 && g.sh != 2))
    return false;
  const bool wide = dw_wide(dtype, a);
  const int th = (dtype != 0 && !wide ? 16 : 8) / g.sh;
  const int64_t tiles = (int64_t)((g.Wo + kDwTW - 1) / kDwTW) *
                        ((g.Ho + th - 1) / th);
  const int slabs = (a.cout_p / 8 + (wide ? 7 : 3)) / (wide ? 8 : 4);
  // sixteenths of the tiles' pixels that are outputs
  const int64_t full = 16 * (int64_t)g.Ho * g.Wo / (tiles * th * kDwTW);
  if (g.sh == 1) return images * tiles * slabs <= 1024 || full >= 3;
  return images * tiles * slabs <= 512 || full >= (dtype == 0 ? 10 : 6);
}

void launch_dense_dw(const Prof& pf, hipStream_t s, int dtype,
                     const ConvArgs& a, int images) {
  prof_begin(pf, 8 /*ST_K_CONV_DW*/, s);
  if (dtype == 0)
    dense_dw<float>(s, a, images);
  else if (dtype == 1)
    dense_dw<_Float16>(s, a, images);
  else
    dense_dw<bf16_t>(s, a, images);
  prof_end(pf, 8, s);
}

int launch_dense_conv(hipStream_t s, int dtype, const ConvArgs& a) {
  if (dtype == 0) return dense_conv<float>(s, a);
  if (dtype == 1) return dense_conv<_Float16>(s, a);
  return dense_conv<bf16_t>(s, a);
}

}  // namespace st
