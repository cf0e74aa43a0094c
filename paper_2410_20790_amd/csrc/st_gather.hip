// Gathered convolutions of the diff frames (gfx950): the affected rows of a
// layer, whose operands are gathered through the neighbour table straight
// into LDS.
//
// A 64-row by 64-channel tile is a chain of round trips -- its row bounds,
// its lists, the first stage, the states it updates, its stores -- around a
// short reduction (one to a few dozen stages), and that chain, not the bytes
// or the products, bounds it.  Against the register-staged kernel
// (k_conv_gemm, which keeps what this one does not take) the stages cost no
// registers (global-to-LDS loads, S - 1 stages outstanding, one counted wait
// and one barrier each), and the registers so freed hold what the epilogue
// needs -- old states, residual rows -- requested before the first stage and
// arriving with it, where they cost no round trip of their own.  The weights
// are the matrix units' first operand, so a lane owns eight consecutive
// channels of a row: a frame's update leaves straight from the accumulators,
// without LDS or a barrier; only a chunk's site runs, whose frames follow one
// another, go through LDS.
//
// Measured (us of kernel time, before -> after): two live ResNet-50 frames at
// 1024x2048 2000 -> 1580; in its chunk of 9 the seven 3x3 layers here 405 ->
// 367 and the fourteen 1x1 layers without a residual row 767 -> 750;
// EfficientNet-B0's 1x1 layers, whose channels fill no stage
// (and paid a division per vector), of 32 cameras 650 -> 420.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "st_device.h"
#include "st_kernels.h"
#include "st_stage.h"

namespace st {

namespace {

constexpr int kGB = 64;         // tile rows and channels
constexpr int kGWindow = 9;     // largest window with a table in LDS
constexpr int kGCld = kGB + 4;  // f32 row of the accumulator tile
constexpr int kGXcd = 8;
constexpr int kGWalk = 6;       // rows per site run above which a tile walks

// This thread's gathered and weight vectors of a stage: two rows each.
// POINT: 1x1 kernels (any channel count); else channel counts that are a
// multiple of the stage's columns, offsets without an active neighbour in the
// tile skipped.
template <typename T, bool POINT>
struct GatherLoader {
  static constexpr int VEC = 16 / (int)sizeof(T);
  static constexpr int KC = kRowBytes / (int)sizeof(T);
  const T* prow[2];
  const T* wrow[2];
  const int* nbr;  // [offset][tile row] in LDS
  u64 rest;        // active offsets after the current one
  int ci, wc, sub, left, wave, lr;

  __device__ __forceinline__ void offset_rows(const ConvArgs& a, int k) {
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int src = nbr[k * kGB + (q * 4 + wave) * 8 + lr];
      prow[q] = src >= 0 ? (const T*)a.din + (int64_t)src * a.cin_p : nullptr;
    }
  }

  // lo: first of the tile's active stages, n: how many
  __device__ __forceinline__ void init(const ConvArgs& a, int n0, u64 kmask,
                                       const int* src, const int* table,
                                       int lo, int n, int lane, int wave_) {
    wave = wave_;
    lr = lane >> 3;
    left = n;
    nbr = table;
    const int slot = lane & 7;
    const int cv = (slot ^ lr) * VEC;
    const int cw = (slot ^ ((lr & 3) | ((wave & 1) << 2))) * VEC;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int c = n0 + (q * 4 + wave) * 8 + lr;
      wrow[q] = c < a.cout_p ? (const T*)a.w + (int64_t)c * a.ktot_p : nullptr;
    }
    if (POINT) {
#pragma unroll
      for (int q = 0; q < 2; ++q)
        prow[q] = src[q] >= 0
                      ? (const T*)a.din + (int64_t)src[q] * a.cin_p
                      : nullptr;
      ci = cv + lo * KC;
      wc = cw + lo * KC;
    } else {
      const int spk = a.cin_p / KC;
      for (int skip = lo / spk; skip > 0; --skip) kmask &= kmask - 1;
      sub = lo % spk;
      const int k = kmask ? __builtin_ctzll(kmask) : 0;
      rest = kmask & (kmask - 1);
      offset_rows(a, k);
      ci = cv + sub * KC;
      wc = k * a.cin_p + cw + sub * KC;
    }
  }

  template <int BM>
  __device__ __forceinline__ void issue(const ConvArgs& a, char* buf) {
    const T* zero = (const T*)a.zero;
    const bool live = left > 0;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const bool ok = live && prow[q] && (!POINT || ci < a.cin_p);
      load_to_lds(ok ? prow[q] + ci : zero,
                  buf + (q * 4 + wave) * 8 * kRowBytes);
    }
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const bool ok = live && wrow[q] && (!POINT || wc < (int)a.ktot_p);
      load_to_lds(ok ? wrow[q] + wc : zero,
                  buf + (BM + (q * 4 + wave) * 8) * kRowBytes);
    }
    --left;
    ci += KC;
    wc += KC;
    if (!POINT && ++sub == a.cin_p / KC && left > 0) {
      const int k = __builtin_ctzll(rest);
      rest &= rest - 1;
      sub = 0;
      ci -= a.cin_p;
      wc = k * a.cin_p + wc % KC;
      offset_rows(a, k);
    }
  }
};

// A chunk's state update (kModeChunkState): the rows are site runs, of few
// frames (kGatherShortRuns) or of any length; kNoRuns: one frame's rows or
// rows whose update is linear or deferred.
enum { kNoRuns = 0, kShortRuns = 1, kLongRuns = 2 };

// SPLIT: a partial tile for the split epilogue.
template <typename T, bool POINT, int KRUNS, bool SPLIT, int S, int WPE>
__global__ __launch_bounds__(256)
__attribute__((amdgpu_waves_per_eu(WPE))) void k_gather_conv(ConvArgs a) {
  constexpr bool RUNS = KRUNS != kNoRuns, LONG = KRUNS == kLongRuns;
  constexpr int BM = kGB, BN = kGB, IM = 2, JN = 2;
  constexpr int KC = kRowBytes / (int)sizeof(T);
  constexpr int STAGE = (BM + BN) * kRowBytes;
  static_assert(S == 2 || S == 3, "stages");
  __shared__ __align__(128) char s0[STAGE];
  __shared__ __align__(128) char s1[STAGE];
  __shared__ __align__(128) char s2[S > 2 ? STAGE : 128];
  __shared__ int s_nbr[POINT ? 1 : kGWindow * BM];
  __shared__ int s_act[POINT ? 1 : kGWindow];
  __shared__ int s_site[RUNS ? BM : 1];
  __shared__ int s_run[LONG ? BM + 1 : 1];  // the runs' first rows, the end
  __shared__ u64 s_open;  // the rows that open a site run

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int l16 = lane & 15, lg = lane >> 4;
  const int cout_p = a.cout_p, K = a.K;
  const int64_t nO = (int64_t)*a.nO;
  const int rstep = RUNS ? chunk_tile_step(a.nf) : BM;
  const int64_t tiles_m = (nO + rstep - 1) / rstep;
  const int tiles_n = (cout_p + BN - 1) / BN;
  const int64_t ntiles = tiles_m * tiles_n;
  const int spk = (a.cin_p + KC - 1) / KC;  // stages per offset
  const int sp_n = SPLIT ? split_count(ntiles, a.split_max) : 1;
  const int64_t nunits = ntiles * sp_n;
  // each XCD a contiguous range of units (neighbouring tiles gather the same
  // rows), its blocks striding through it
  const int chunk = (int)((nunits + kGXcd - 1) / kGXcd);
  const int xcd = blockIdx.x % kGXcd;
  const int u_end = (int)min(nunits, (int64_t)(xcd + 1) * chunk);
  const int per_xcd = gridDim.x / kGXcd;
  const int u0 = xcd * chunk + blockIdx.x / kGXcd;
  const int row0 = wm * 32 + l16;  // this lane's rows: row0 + 16 i
  for (int u = u0; u < u_end; u += per_xcd) {
    const int sp = SPLIT ? (int)((unsigned)u / (unsigned)ntiles) : 0;
    const int t = SPLIT ? u - sp * (int)ntiles : u;
    const int tm = (int)((unsigned)t / (unsigned)tiles_n);
    const int n0 = (t - tm * tiles_n) * BN;
    const int64_t m0 = RUNS ? (int64_t)a.tstart[tm] : (int64_t)tm * BM;
    const int64_t m1 =
        RUNS ? (int64_t)a.tstart[tm + 1] : min(m0 + BM, nO);
    const int rows = (int)(m1 - m0);
    if (u != u0) __syncthreads();  // the previous unit's LDS reads

    // lists: the gathered rows, the rows' pixels, a chunk's site runs
    int src[2] = {-1, -1};
    if constexpr (POINT) {
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const int r = (q * 4 + wave) * 8 + (lane >> 3);
        if (r < rows) src[q] = a.nbr[m0 + r];
      }
    }
    int epix[IM];
#pragma unroll
    for (int i = 0; i < IM; ++i)
      epix[i] = !SPLIT && (!RUNS || a.mskip) && row0 + 16 * i < rows
                    ? a.O[m0 + row0 + 16 * i]
                    : -1;
    if constexpr (!POINT) {
      // a wave takes an offset's 64 rows at a time, its offsets together
      constexpr int NV = (kGWindow + 3) / 4;
      int v[NV];
#pragma unroll
      for (int j = 0; j < NV; ++j) {
        const int k = wave + 4 * j;
        v[j] = k < K && lane < rows
                   ? a.nbr[(int64_t)k * a.stride + m0 + lane]
                   : -1;
      }
#pragma unroll
      for (int j = 0; j < NV; ++j) {
        const int k = wave + 4 * j;
        const u64 any = __ballot(v[j] >= 0);
        if (k < K) {
          s_nbr[k * BM + lane] = v[j];
          if (lane == 0) s_act[k] = any != 0ull;
        }
      }
    }
    if constexpr (RUNS) {
      if (wave == 0) {
        const int site =
            lane < rows
                ? (int)((unsigned)a.O[m0 + lane] % (unsigned)a.per)
                : -1;
        const int prev = __shfl_up(site, 1, 64);
        const u64 starts =
            __ballot(lane < rows && (lane == 0 || site != prev));
        s_site[lane] = site;
        if (LONG && ((starts >> lane) & 1ull))
          s_run[lane_prefix(starts)] = lane;
        if (lane == 0) {
          s_open = starts;
          if (LONG) s_run[__popcll(starts)] = rows;
          // every run lies in one row tile: its first column tile counts it
          if (n0 == 0 && starts)
            atomicAdd(a.sites + blockIdx.x % kSiteSlots,
                      (u64)__popcll(starts));
        }
      }
    }
    if constexpr (!POINT || RUNS) __syncthreads();
    u64 kmask = 1ull;
    if constexpr (!POINT)
      kmask = __ballot(lane < K && s_act[lane < K ? lane : 0]);
    const int nact = POINT ? spk : (int)__popcll(kmask) * spk;
    // A split's share of the active stages.  Half precision: those of its
    // share of the whole reduction, so that a row's sum does not depend on
    // which rows share its tile; f32: an equal share (CRNN-VGG chunks of 16:
    // 625 us a group against 638).
    auto cut = [&](int j) {
      if (POINT || sizeof(T) == 4) return j * nact / sp_n;
      const int r = j * (K * spk) / sp_n, k = r / spk;
      return (int)__popcll(kmask & ((1ull << k) - 1)) * spk +
             ((kmask >> k) & 1ull ? r - k * spk : 0);
    };
    const int lo = SPLIT ? cut(sp) : 0;
    const int nst = (SPLIT ? cut(sp + 1) : nact) - lo;

    // what the epilogue reads, requested before the first stage
    const int c = n0 + wn * 32 + lg * 8;  // this lane's eight channels
    int rsk[IM];
#pragma unroll
    for (int i = 0; i < IM; ++i)
      rsk[i] = a.mskip && epix[i] >= 0 ? a.mskip[epix[i]] : -1;
    float P[16];
    // a chunk's rows: four adjacent lanes each, channels 8 j + 32 h + [0, 8)
    const int er = tid >> 2, ec = (tid & 3) * 8;
    int64_t sbase = 0;
    if constexpr (RUNS) {
      sbase = (er < rows ? (int64_t)s_site[er] : 0) * cout_p + n0 + ec;
#pragma unroll
      for (int h = 0; h < 2; ++h)
        if (er < rows && n0 + ec + 32 * h < cout_p)
          state_load8(a.P, a.p16, sbase + 32 * h, P + 8 * h);
    } else if (!SPLIT && a.mode == kModeState) {
#pragma unroll
      for (int i = 0; i < IM; ++i) {
        if (epix[i] >= 0 && c < cout_p)
          state_load8(a.P, a.p16, (int64_t)epix[i] * cout_p + c, P + 8 * i);
      }
    }

    GatherLoader<T, POINT> ld;
    ld.init(a, n0, kmask, src, s_nbr, lo, nst, lane, wave);
    ld.template issue<BM>(a, s0);
    if constexpr (S > 2) ld.template issue<BM>(a, s1);

    constexpr int SKV = (int)sizeof(T) / 2;  // 16-byte vectors / 8 channels
    uint4 sk[IM][SKV];
#pragma unroll
    for (int i = 0; i < IM; ++i)
#pragma unroll
      for (int v = 0; v < SKV; ++v) {
        sk[i][v] = make_uint4(0u, 0u, 0u, 0u);
        if (rsk[i] >= 0 && c < cout_p)
          sk[i][v] = ((const uint4*)((const T*)a.dskip +
                                     (int64_t)rsk[i] * cout_p + c))[v];
      }

    v4f acc[IM][JN];
#pragma unroll
    for (int i = 0; i < IM; ++i)
#pragma unroll
      for (int j = 0; j < JN; ++j) acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};
    constexpr int AH = (S - 2) * 4;
    const int pr = wm * 32, wr = BM + wn * 32;
    for (int st = 0; st < nst; st += S) {
      stage_turn<T, BM, AH>(a, ld, s0, S == 2 ? s1 : s2, pr, wr, l16, lg,
                            acc);
      if (st + 1 >= nst) break;
      stage_turn<T, BM, AH>(a, ld, s1, s0, pr, wr, l16, lg, acc);
      if constexpr (S > 2) {
        if (st + 2 >= nst) break;
        stage_turn<T, BM, AH>(a, ld, s2, s1, pr, wr, l16, lg, acc);
      }
    }

    if constexpr (SPLIT) {
      float* part = a.part + (int64_t)sp * a.capO * cout_p;
#pragma unroll
      for (int i = 0; i < IM; ++i) {
        if (row0 + 16 * i >= rows || c >= cout_p) continue;
        float* d = part + (m0 + row0 + 16 * i) * cout_p + c;
        *(v4f*)d = acc[i][0];
        *(v4f*)(d + 4) = acc[i][1];
      }
      continue;
    }

    // the reduced values with the residual deltas
    float v[IM][8];
#pragma unroll
    for (int i = 0; i < IM; ++i) {
      Vec8<T>::load((const T*)sk[i], v[i]);
#pragma unroll
      for (int e = 0; e < 8; ++e) v[i][e] = acc[i][e >> 2][e & 3] + v[i][e];
    }
    T* dout = (T*)a.dout;
    if constexpr (!RUNS) {
      with_act(a.act, [&](auto act_tag) {
        constexpr int ACT = decltype(act_tag)::value;
#pragma unroll
        for (int i = 0; i < IM; ++i) {
          const int64_t o = m0 + row0 + 16 * i;
          const bool ok = row0 + 16 * i < rows && c < cout_p;
          float rm = 0.f;
          if (ok && a.mode == kModeDefer) {
            store8f(a.dP + o * cout_p + c, v[i]);
          } else if (ok) {
            if (a.mode == kModeState) {
              const int64_t at = (int64_t)epix[i] * cout_p + c;
              float pn[8];
#pragma unroll
              for (int e = 0; e < 8; ++e)
                pn[e] = state_round(a.p16, P[8 * i + e] + v[i][e]);
              if (a.gate) {
                // frozen squeeze-excitation: both values scaled by the gates
                float g[8];
                load8f(gate_slot(a.gate, a.gpar, a.gsz, 0) +
                           (epix[i] / a.gate_hw) * cout_p + c,
                       g);
#pragma unroll
                for (int e = 0; e < 8; ++e)
                  v[i][e] = act_c<ACT>(pn[e]) * g[e] -
                            act_c<ACT>(P[8 * i + e]) * g[e];
              } else if (a.yhat) {
                // residual carry: against what the consumers received
                float yh[8];
                load8f(a.yhat + at, yh);
#pragma unroll
                for (int e = 0; e < 8; ++e)
                  v[i][e] = act_c<ACT>(pn[e]) - yh[e];
              } else {
#pragma unroll
                for (int e = 0; e < 8; ++e)
                  v[i][e] = act_c<ACT>(pn[e]) - act_c<ACT>(P[8 * i + e]);
              }
              state_store8(a.P, a.p16, at, pn);
            }
            rm = Vec8<T>::store(dout + o * cout_p + c, v[i]);
          }
          // the four lanes of a row's 32 channels
          rm = fmaxf(rm, __shfl_xor(rm, 16, 64));
          rm = fmaxf(rm, __shfl_xor(rm, 32, 64));
          if (lg == 0 && rm > 0.f && a.rowmax)
            atomicMax(a.rowmax + o, __float_as_uint(rm));
        }
      });
    } else {
      // the accumulator tile to LDS (rows 0..31 in the first stage's buffer,
      // 32..63 in the second's), once no load into them is outstanding
      stage_ready<0>();
      auto crow = [&](int r) {
        return (float*)(r < 32 ? s0 : s1) + (r & 31) * kGCld;
      };
#pragma unroll
      for (int i = 0; i < IM; ++i)
        store8f(crow(row0 + 16 * i) + wn * 32 + lg * 8, v[i]);
      __syncthreads();
      // A row's state is the run's first state and the updates of the run's
      // rows before it, added in frame order; the run's last row stores it.
      // Short runs: every row adds the rows before it for itself (runs are a
      // few rows long, and every lane has a row to emit: walking a run with
      // its own threads left half of them idle and the others a loop of
      // emissions).  Tiles of long runs, where that is quadratic (chunks of
      // 31 frames at 512x1024, 90% changed, ResNet-50: 31.4 ms), walk them in
      // LDS first: the updates become the states after them, the runs' first
      // rows' by their own threads, then two columns of a run per thread, 32
      // threads a run (26.0 ms; 26.3 with the layers of gather_takes).
      const u64 starts = s_open;
      const bool in = er < rows, opens = (starts >> er) & 1ull;
      const int nruns = (int)__popcll(starts);
      const bool walk =
          LONG && __builtin_amdgcn_readfirstlane(rows > kGWalk * nruns);
      if (walk) {
        if (in && opens) {
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            if (n0 + ec + 32 * h >= cout_p) continue;
            float* x = crow(er) + ec + 32 * h;
            float w[8];
            load8f(x, w);
#pragma unroll
            for (int e = 0; e < 8; ++e)
              w[e] = state_round(a.p16, P[8 * h + e] + w[e]);
            store8f(x, w);
          }
        }
        __syncthreads();
        const int wc = (tid & 31) * 2;
        for (int g = tid >> 5; g < nruns; g += 8) {
          const int r0 = s_run[g], r1 = s_run[g + 1];
          float2 p = *(const float2*)(crow(r0) + wc);
#pragma unroll 4
          for (int r = r0 + 1; r < r1; ++r) {
            float2* x = (float2*)(crow(r) + wc);
            p.x = state_round(a.p16, p.x + x->x);
            p.y = state_round(a.p16, p.y + x->y);
            *x = p;
          }
        }
        __syncthreads();
        if (in && !opens) {
#pragma unroll
          for (int h = 0; h < 2; ++h)
            load8f(crow(er - 1) + ec + 32 * h, P + 8 * h);
        }
      } else {
        int rr =
            in ? 63 - __builtin_clzll(starts & (~0ull >> (63 - er))) : er;
        for (; rr < er; ++rr) {
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            float w[8];
            load8f(crow(rr) + ec + 32 * h, w);
#pragma unroll
            for (int e = 0; e < 8; ++e)
              P[8 * h + e] = state_round(a.p16, P[8 * h + e] + w[e]);
          }
        }
      }
      const bool last = er + 1 >= rows || ((starts >> (er + 1)) & 1ull);
      float rm = 0.f;
      with_act(a.act, [&](auto act_tag) {
        constexpr int ACT = decltype(act_tag)::value;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int ch = n0 + ec + 32 * h;
          if (!in || ch >= cout_p) continue;
          float w[8], d[8];
          load8f(crow(er) + ec + 32 * h, w);
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const float po = P[8 * h + e];
            if (!walk) w[e] = state_round(a.p16, po + w[e]);
            d[e] = act_c<ACT>(w[e]) - act_c<ACT>(po);
          }
          rm = fmaxf(rm, Vec8<T>::store(dout + (m0 + er) * cout_p + ch, d));
          if (last) state_store8(a.P, a.p16, sbase + 32 * h, w);
        }
      });
      rm = fmaxf(rm, __shfl_xor(rm, 1, 64));
      rm = fmaxf(rm, __shfl_xor(rm, 2, 64));
      if ((tid & 3) == 0 && in && rm > 0.f)
        atomicMax(a.rowmax + m0 + er, __float_as_uint(rm));
    }
  }
}

template <typename T, bool POINT, int KRUNS, bool SPLIT, int S, int PER_CU>
void gather_launch(hipStream_t s, const ConvArgs& a, int step) {
  const int64_t units = (a.capO + step - 1) / step *
                        ((a.cout_p + kGB - 1) / kGB) *
                        (SPLIT ? a.split_max : 1);
  int64_t grid = units < 256 * PER_CU ? units : 256 * PER_CU;
  grid = (grid + kGXcd - 1) / kGXcd * kGXcd;
  k_gather_conv<T, POINT, KRUNS, SPLIT, S, PER_CU>
      <<<(int)grid, 256, 0, s>>>(a);
}

// Stages and blocks per CU (one wave of a block per SIMD): the chunk build
// keeps 16 state values beside the products and takes three (four, with its
// spills, 2.86 ms of a ResNet-50 chunk of 9 diff frames against 2.65; three
// with a third stage 2.72); the one-frame builds take four, although they
// spill seven to nine registers there, as every mode and activation is in one
// build (linear chunk layers 263 us against 302 with three).  Split
// reductions are long and take a third stage (323 -> 309 us of a frame's),
// and so do, in chunks of long runs, half-precision 1x1 layers of four stages
// or more (the fourteen without a residual row of a ResNet-50 chunk of 9:
// 793 -> 750 us with 10% of the sites changed, 2050 -> 1946 with 40%; the 3x3
// layers 367 -> 381, f32 chunks 4.75 -> 4.80 ms).  128x128 tiles (one block
// per CU) were slower on every layer, and so were the next unit's lists
// requested ahead.
template <typename T, bool POINT>
void gather_conv(hipStream_t s, const ConvArgs& a) {
  if (a.mode == kModeChunkState && a.nf <= kGatherShortRuns)
    gather_launch<T, POINT, kShortRuns, false, 2, 3>(s, a,
                                                     chunk_tile_step(a.nf));
  else if (a.mode == kModeChunkState && POINT && sizeof(T) == 2 &&
           a.cin_p >= 256)
    gather_launch<T, POINT, kLongRuns, false, POINT ? 3 : 2, 3>(
        s, a, chunk_tile_step(a.nf));
  else if (a.mode == kModeChunkState)
    gather_launch<T, POINT, kLongRuns, false, 2, 3>(s, a,
                                                    chunk_tile_step(a.nf));
  else if (a.split_max > 1)
    gather_launch<T, POINT, kNoRuns, true, 3, 3>(s, a, kGB);
  else
    gather_launch<T, POINT, kNoRuns, false, 2, 4>(s, a, kGB);
}

template <typename T>
void gather_conv(hipStream_t s, const ConvArgs& a) {
  if (a.K == 1)
    gather_conv<T, true>(s, a);
  else
    gather_conv<T, false>(s, a);
}

}  // namespace

void launch_gather_conv(hipStream_t s, int dtype, const ConvArgs& a) {
  if (dtype == 0)
    gather_conv<float>(s, a);
  else if (dtype == 1)
    gather_conv<_Float16>(s, a);
  else
    gather_conv<bf16_t>(s, a);
}

}  // namespace st
