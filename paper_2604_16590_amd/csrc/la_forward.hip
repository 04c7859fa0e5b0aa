// la_forward.hip -- gfx950 kernels of the forward pass and of the FP64
// cross-tile combine.
//
// Forward of kernelised linear attention per (b, h):
//   S = phi(K)^T V, z = phi(K)^T 1 over all N tokens (summary_kernel, then
//   combine_kernel), O_i = phi(q_i)^T S / (phi(q_i) . z) (apply_kernel,
//   which can also blend O with another branch's output by a noise gate).
// Both phases stream HBM once: summary reads K and V, apply reads Q and
// writes O.  The d x d contractions run on the matrix cores.
#include "la_kernels.h"
#include "la_profile.h"
#include "la_split.h"
#include "la_summary.h"

namespace la {

// ---------------------------------------------------------------------------
// Summary: per wave, a contiguous token range [p*Tw, p*Tw + Tw) of one head.
// Lane (g, m) owns key/value features [F*m, F*m + F) (F = d/16) of R tokens
// per lane group per step.  Loads are contiguous F-feature runs of a token,
// so one load instruction covers whole token rows.  The feature-major
// operands the matrix core needs (a token run per feature) are assembled in
// registers: for bf16 the two tokens of a pair are packed into one word, so
// the transpose costs nothing beyond the pack that rounds phi(k) anyway.
//
// Tile (i, j) of the accumulator holds rows m <-> key feature F*m + i and
// columns n <-> value feature F*n + j, so lane (g, n) ends with
//   S[F*(4g + r) + i][F*n + j],  r = 0..3.
// These FP32 per-wave sums are written out; combine_kernel adds them in
// FP64 in partial order.
// ---------------------------------------------------------------------------
// Rows past the end of the range load K = -inf (phi = 0) and V = 0, so
// they add exactly nothing to S or z and the step itself needs no masks.
// In the backward mode the per-token pair (1/den, -(dO . O)) is loaded too.
// Addresses split into a wave-uniform part (head + (t0 + r) rows, scalar
// registers) and a loop-invariant 32-bit lane offset (off: the lane group's
// first row and the lane's feature run), so the loads need no per-lane
// address arithmetic.
template <int DT, int D, int MODE>
__device__ __forceinline__ void summary_load(const char* kh, const char* vh, uint32_t off,
                                             const float2* stash,
                                             int64_t row_bytes, int64_t t0, int g, int m,
                                             int64_t t_end, SummaryRegs<DT, D, MODE>& x) {
  using C = SummaryCfg<DT, D, MODE>;
  const uint32_t neg_inf = DT == DT_BF16 ? 0xff80ff80u : 0xff800000u;
  if (t0 + C::STEP <= t_end) {
#pragma unroll
    for (int r = 0; r < C::R; ++r) {
      const int64_t ur = (t0 + r) * row_bytes;
      load_words_nt<C::KB>(kh + ur + off, x.kw[r]);
      load_words_nt<C::VB>(vh + ur + off, x.vw[r]);
    }
  } else {
#pragma unroll
    for (int r = 0; r < C::R; ++r) {
      const int64_t ur = (t0 + r) * row_bytes;
      if (t0 + C::R * g + r < t_end) {
        load_words_nt<C::KB>(kh + ur + off, x.kw[r]);
        load_words_nt<C::VB>(vh + ur + off, x.vw[r]);
      } else {
#pragma unroll
        for (int w = 0; w < C::KW; ++w) x.kw[r][w] = neg_inf;
#pragma unroll
        for (int w = 0; w < C::VW; ++w) x.vw[r][w] = 0;
      }
    }
  }
  if constexpr (MODE == MODE_BWD) {
    const int64_t t = t0 + C::R * g + m;
    x.tok = (m < C::R && t < t_end) ? stash[t] : float2{0.f, 0.f};
  }
}

// A partial's tokens are summed in runs of Tq (summary_run), from zero each,
// and the runs' sums added in order in FP32, so that the same bits come of
// two forms (teams always take the second, and join longer partials' runs in
// FP64, join64):
// NW = 1: a wave to a partial takes its runs one after the other and keeps
// the sum so far in LDS.  One dimension of waves in (partial, (b, h)) order,
// (b, h) fastest: wave w takes partial w / BH of (b, h) = w % BH, so a
// block's four waves are four heads over the same tokens (with heads
// interleaved in a token row, BNHD, one compute unit then reads adjacent
// slices of the same rows: the summary at d = 64, 16 heads, went from 1.55 to
// 1.32 ms; BHND is unaffected).
// NW > 1: one workgroup per (partial, (b, h)), in the same order, a wave to a
// run.  A few heads are NW times as many waves for the same partials in
// memory (a head of 1,700,000 tokens at d = 32: 86 us, 417 with a wave to a
// partial; two of 300,000 at d = 64: 51, 175).  Each XCD takes a contiguous
// share of the items (workgroups go to the eight in turn).
// (fp32 inputs at d >= 32 take summary_split_kernel.)
template <int DT, int D, int MODE, int NW>
__global__ __launch_bounds__(NW == 1 ? 256 : 64 * NW) __attribute__((amdgpu_waves_per_eu(NW == 16 ? 4 : SummaryCfg<DT, D, MODE>::WAVES_PER_SIMD))) void summary_kernel(
    const void* __restrict__ k, const void* __restrict__ v, int64_t sb,
    int64_t sh, int64_t sn, int H, int64_t N, int P, int Tw, int Tq,
    const float2* __restrict__ stash, float* __restrict__ part, int BH, bool join64) {
  using C = SummaryCfg<DT, D, MODE>;
  constexpr int F = C::F;
  constexpr int E = D * D + D;
  const int lane = threadIdx.x & 63, wave = wave_index();
  const int g = lane >> 4, m = lane & 15;
  int64_t item = (int64_t)blockIdx.x * 4 + wave;
  if constexpr (NW > 1) item = (int64_t)(blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
  const int p = (int)(item / BH);
  if (p >= P) return;  // uniform across the waves that share p
  const int bh = (int)(item % BH);
  const int64_t b = bh / H, h = bh % H;
  int64_t t_begin = (int64_t)p * Tw;
  int64_t t_end = min(N, t_begin + (int64_t)Tw);
  if constexpr (NW > 1) {
    // a wave past the partial's end runs one step of masked rows, which
    // adds nothing
    t_begin += (int64_t)wave * Tq;
    t_end = min(t_end, t_begin + (int64_t)Tq);
  }
  const int64_t head = (b * sb + h * sh) * C::ES;
  // lane m reads features [F*m, +F) of rows R*g + r (the host bounds 32 rows
  // of the token stride to 2^24 bytes, so the lane offset fits 32 bits)
  const int64_t row_bytes = sn * C::ES;
  const char* kh = (const char*)k + head;
  const char* vh = (const char*)v + head;
  const uint32_t off = (uint32_t)(C::R * g) * (uint32_t)row_bytes + (uint32_t)(F * m * C::ES);
  const float2* tstash = MODE == MODE_BWD ? stash + (int64_t)bh * N : nullptr;

  f32x4 acc[F][F];
  float zacc[F];
#pragma unroll
  for (int i = 0; i < F; ++i)
#pragma unroll
    for (int j = 0; j < F; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int i = 0; i < F; ++i) zacc[i] = 0.f;
  // the sum of the runs before this one (NW = 1)
  constexpr bool KEEP = NW == 1 && (D == 32 || D == 64);
  __shared__ f32x4 kept[KEEP ? 4 : 1][KEEP ? F * F : 1][64];
  float zkept[F];
  bool first = true;
  auto add_kept = [&] {
#pragma unroll
    for (int i = 0; i < F; ++i) {
      zacc[i] = sum_groups(zacc[i]);
      if (!first) zacc[i] = zkept[i] + zacc[i];
#pragma unroll
      for (int j = 0; j < F; ++j)
        if (!first) acc[i][j] = kept[wave][i * F + j][lane] + acc[i][j];
    }
  };

  // two register sets in turn: while one step computes, the next one's
  // loads are in flight in the other set (no copies between them)
  SummaryRegs<DT, D, MODE> ra, rb;
  auto load = [&](int64_t t0, SummaryRegs<DT, D, MODE>& x) {
    summary_load<DT, D, MODE>(kh, vh, off, tstash, row_bytes, t0, g, m, t_end, x);
  };
  int64_t t0 = t_begin;
  int left = Tq;  // tokens of the run, a multiple of two steps (NW = 1)
  load(t0, ra);
  while (true) {
    const int64_t t1 = t0 + C::STEP;
    if (t1 < t_end) load(t1, rb);
    summary_step<DT, D, MODE>(ra, acc, zacc);
    if (t1 >= t_end) break;
    const int64_t t2 = t1 + C::STEP;
    if (t2 < t_end) load(t2, ra);
    summary_step<DT, D, MODE>(rb, acc, zacc);
    if (t2 >= t_end) break;
    t0 = t2;
    if constexpr (KEEP) {
      left -= 2 * C::STEP;
      if (left == 0) {
        add_kept();
#pragma unroll
        for (int i = 0; i < F; ++i) {
          zkept[i] = zacc[i];
          zacc[i] = 0.f;
#pragma unroll
          for (int j = 0; j < F; ++j) {
            kept[wave][i * F + j][lane] = acc[i][j];
            acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
          }
        }
        first = false;
        left = Tq;
      }
    }
  }

  float* out = part + ((int64_t)bh * P + p) * E;
  if constexpr (NW > 1) {
    // the runs' sums meet in LDS, RT tiles at a time
    constexpr int T = F * F, RT = T < 64 / NW ? T : 64 / NW;
    static_assert(RT % F == 0);
    __shared__ f32x4 red[NW][RT][64];
    __shared__ float zred[NW][D];
    const int runs = (int)((min(N - (int64_t)p * Tw, (int64_t)Tw) + Tq - 1) / Tq);
    // K neighbouring sums, the runs' sums in order.  Only teams of four join
    // in FP64, with all loads in flight (no branch divides them)
    constexpr bool J64 = NW == 4 && D >= 64;
    auto join = [&](auto kc, auto at, float* x) {
      constexpr int K = decltype(kc)::value;
#pragma unroll
      for (int j = 0; j < K; ++j) x[j] = at(0, j);
      if (J64 && join64) {
        float y[NW][K];
#pragma unroll
        for (int w = 1; w < NW; ++w)
#pragma unroll
          for (int j = 0; j < K; ++j) y[w][j] = at(w, j);
#pragma unroll
        for (int j = 0; j < K; ++j) {
          double s = x[j];
#pragma unroll
          for (int w = 1; w < NW; ++w) {
            if (w < runs) s += (double)y[w][j];
          }
          x[j] = (float)s;
        }
      } else {
        for (int w = 1; w < runs; ++w)
#pragma unroll
          for (int j = 0; j < K; ++j) x[j] += at(w, j);
      }
    };
#pragma unroll
    for (int i = 0; i < F; ++i) {
      const float zs = sum_groups(zacc[i]);
      if (g == 0) zred[wave][F * m + i] = zs;
    }
#pragma unroll
    for (int r0 = 0; r0 < T; r0 += RT) {
      if (r0 > 0) __syncthreads();  // the buffers have been read
#pragma unroll
      for (int t = 0; t < RT; ++t) red[wave][t][lane] = acc[(r0 + t) / F][(r0 + t) % F];
      __syncthreads();
      // a wave takes rows 4g + r of a tile row in turn
      for (int u = wave; u < RT / F * 4; u += NW) {
        const int t = u / 4 * F, r = u % 4;
        float x[F];
        join(std::integral_constant<int, F>{}, [&](int w, int j) { return red[w][t + j][lane][r]; }, x);
        uint32_t w[F];
#pragma unroll
        for (int j = 0; j < F; ++j) w[j] = __float_as_uint(x[j]);
        store_words<4 * F>(out + (F * (4 * g + r) + (r0 + t) / F) * D + F * m, w);
      }
    }
    if (threadIdx.x < D)
      join(std::integral_constant<int, 1>{}, [&](int w, int) { return zred[w][threadIdx.x]; },
           out + D * D + threadIdx.x);
    return;
  }

  // this wave's partial: rows of S, F consecutive values a lane, then z
  if constexpr (KEEP) {
    add_kept();
  } else {
#pragma unroll
    for (int i = 0; i < F; ++i) zacc[i] = sum_groups(zacc[i]);
  }
#pragma unroll
  for (int i = 0; i < F; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      uint32_t w[F];
#pragma unroll
      for (int j = 0; j < F; ++j) w[j] = __float_as_uint(acc[i][j][r]);
      store_words<4 * F>(out + (F * (4 * g + r) + i) * D + F * m, w);
    }
#pragma unroll
  for (int i = 0; i < F; ++i)
    if (g == 0) out[D * D + F * m + i] = zacc[i];
}

// ---------------------------------------------------------------------------
// Summary of fp32 inputs at d >= 32, on the bf16 matrix cores (la_split.h).
// A workgroup takes one partial, 4096 / d tokens a step: its threads load
// the step's K and V rows whole (16 bytes a thread), form phi, split every
// value into three bf16 parts and put them in LDS as rows; the transposing
// LDS read gives the token-major operands, and each wave sums its own tiles
// of S over all of the step's tokens, so nothing is left to add up between
// waves.  The next step's rows are in flight while this one is computed, and
// two (d <= 64: three) workgroups share a compute unit.  Steps that leave
// the split's range are taken after the others by the fp32 matrix
// instructions (in the loop, that path's addresses spilled the operands).
//
// What bounds it: per 32 tokens at d = 128 a SIMD has 1,536 cycles of matrix
// products and about 1,700 of vector work (phi, split, sums) in the 2,400
// that HBM takes; they overlap in part.  8 heads of 524,288 tokens at
// d = 128: 0.86 ms, 5.0 TB/s (fp32 matrix instructions: 1.33); 32 heads of
// 20,011 at d = 64: 71 us (81).
// ---------------------------------------------------------------------------
template <int D>
struct SplitCfg {
  // d = 128: eight waves, so that a wave's share of S and its operands take
  // 128 registers and four waves fit a SIMD (0.86 ms for 8 heads of 524,288
  // tokens; four waves of 4 x 4 tiles, two to a SIMD, 0.90)
  static constexpr int NW = D == 128 ? 8 : 4;
  static constexpr int QI = D == 128 ? 2 : D / 32, QJ = D / 32;  // a wave's tiles of S
  static constexpr int WAVES_PER_SIMD = D == 128 ? 4 : 3;
};

template <int D, int MODE>
__global__ __launch_bounds__(64 * SplitCfg<D>::NW) __attribute__((amdgpu_waves_per_eu(SplitCfg<D>::WAVES_PER_SIMD))) void summary_split_kernel(
    const void* __restrict__ k, const void* __restrict__ v, int64_t sb, int64_t sh, int64_t sn,
    int H, int64_t N, int P, int Tw, const float2* __restrict__ stash, float* __restrict__ part,
    int BH) {
  constexpr int E = D * D + D;
  constexpr int TPS = 4096 / D;       // tokens per step
  constexpr int RP = SplitCfg<D>::NW * 256 / D;  // rows per pass of the workgroup's loads
  constexpr int NP = TPS / RP;        // passes
  constexpr int QI = SplitCfg<D>::QI, QJ = SplitCfg<D>::QJ;
  constexpr int TILE = TPS * D * 2;   // LDS bytes of one part of one tensor
  __shared__ __align__(16) char buf[2][3][TILE];
  __shared__ float zred[RP][D];
  constexpr int STEPS = 4096 / TPS;   // at most (a partial's tokens)
  __shared__ int out_of_range[STEPS]; // steps that left the split's range

  const int tid = threadIdx.x, lane = tid & 63, wave = wave_index();
  const int g = lane >> 4, n = lane & 15;
  const int64_t item = (int64_t)(blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
  const int p = (int)(item / BH);
  if (p >= P) return;  // uniform over the workgroup
  const int bh = (int)(item % BH);
  const int64_t head = ((int64_t)(bh / H) * sb + (int64_t)(bh % H) * sh) * 4;
  const char* kh = (const char*)k + head;
  const char* vh = (const char*)v + head;
  const float2* tstash = MODE == MODE_BWD ? stash + (int64_t)bh * N : nullptr;
  const int64_t t_begin = (int64_t)p * Tw, t_end = min(N, t_begin + (int64_t)Tw);
  const int64_t row_bytes = sn * 4;
  if (tid < STEPS) out_of_range[tid] = 0;

  // this thread's part of a pass: row r0, features [4 * c4, +4)
  const int c4 = tid % (D / 4), r0 = tid / (D / 4);
  // LDS rows: 16-byte chunks XOR-swizzled so that the eight rows a half
  // wave reads (32 bytes each) lie in distinct banks
  auto swz = [](int row) { return D == 128 ? 2 * (row & 7) : D == 64 ? 2 * ((row >> 1) & 3) : 2 * ((row >> 2) & 1); };

  struct Regs {
    f32x4 k[NP], v[NP];
    float2 st[MODE == MODE_BWD ? NP : 1];
  };
  auto load = [&](int64_t t0, Regs& x) {
    // rows past the end read the last one again (masked when used); a
    // step's row offsets fit 32 bits (128 rows of at most 2^24 bytes)
    const int64_t tb = min(t0, t_end - 1);
    const int last = (int)min((int64_t)(TPS - 1), t_end - 1 - tb);
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      const uint32_t row = (uint32_t)min(i * RP + r0, last);
      const uint32_t off = row * (uint32_t)row_bytes + (uint32_t)(c4 * 16);
      x.k[i] = __builtin_nontemporal_load((const f32x4*)(kh + tb * row_bytes + off));
      x.v[i] = __builtin_nontemporal_load((const f32x4*)(vh + tb * row_bytes + off));
      if constexpr (MODE == MODE_BWD) x.st[i] = tstash[tb + row];
    }
  };

  float z[4] = {0.f, 0.f, 0.f, 0.f};
  // phi, split, LDS
  auto stage = [&](int64_t t0, Regs& x, int step) {
    SplitRange<4> kr, vr;  // by feature: a row and a column of S each
    if (t0 + TPS > t_end) {  // uniform: rows past the end add nothing
#pragma unroll
      for (int i = 0; i < NP; ++i)
        if (t0 + i * RP + r0 >= t_end) {
          const float ninf = -__builtin_inff();  // phi = 0
          x.k[i] = f32x4{ninf, ninf, ninf, ninf};
          x.v[i] = f32x4{0.f, 0.f, 0.f, 0.f};
          if constexpr (MODE == MODE_BWD) x.st[i] = float2{0.f, 0.f};
        }
    }
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      const int row = i * RP + r0;
      float a[4], b[4];
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        a[c] = phi<DT_FP32>(x.k[i][c]);
        b[c] = x.v[i][c];
        if constexpr (MODE == MODE_BWD) a[c] *= x.st[i].x;
      }
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        if constexpr (MODE == MODE_BWD) z[c] = fmaf(x.st[i].y, a[c], z[c]);
        else z[c] += a[c];
      }
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        kr.see(c, a[c]);
        vr.see(c, b[c]);
      }
      const int at = row * (2 * D) + (((c4 >> 1) ^ swz(row)) * 16) + (c4 & 1) * 8;
      const Split2 a0 = split2(a[0], a[1]), a1 = split2(a[2], a[3]);
      const Split2 b0 = split2(b[0], b[1]), b1 = split2(b[2], b[3]);
      *(u32x2*)(buf[0][0] + at) = u32x2{a0.h, a1.h};
      *(u32x2*)(buf[0][1] + at) = u32x2{a0.m, a1.m};
      *(u32x2*)(buf[0][2] + at) = u32x2{a0.l, a1.l};
      *(u32x2*)(buf[1][0] + at) = u32x2{b0.h, b1.h};
      *(u32x2*)(buf[1][1] + at) = u32x2{b0.m, b1.m};
      *(u32x2*)(buf[1][2] + at) = u32x2{b0.l, b1.l};
    }
    if (kr.bad() || vr.bad()) out_of_range[step] = 1;  // every writer stores the same
  };

  // wave w sums the tiles of rows [16 i0, +16 QI) and columns [16 j0, +16 QJ)
  const int i0 = QI * (wave >> 1), j0 = QJ * (wave & 1);
  f32x4 acc[QI][QJ];
#pragma unroll
  for (int i = 0; i < QI; ++i)
#pragma unroll
    for (int j = 0; j < QJ; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  // operand of feature block f: lane (g, n) addresses row 4g + (n >> 2) of
  // each 16-row half of a 32-token step, features 16f + 4 (n & 3) .. + 3
  const int rrow = 4 * g + (n >> 2);
  auto operand = [&](int tensor, int ks, int f) {
    const int at = (32 * ks + rrow) * (2 * D) + ((2 * f + ((n & 3) >> 1)) ^ swz(rrow)) * 16 + (n & 1) * 8;
    Bf16x3 r;
    bf16x8* o[3] = {&r.h, &r.m, &r.l};
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      const u32x2 lo = lds_read_tr16(buf[tensor][q] + at);
      const u32x2 hi = lds_read_tr16(buf[tensor][q] + at + 16 * 2 * D);
      *o[q] = as_bf16x8(u32x4{lo[0], lo[1], hi[0], hi[1]});
    }
    return r;
  };
  auto compute = [&]() {
#pragma unroll
    for (int ks = 0; ks < TPS / 32; ++ks) {
      Bf16x3 a[QI];
#pragma unroll
      for (int i = 0; i < QI; ++i) a[i] = operand(0, ks, i0 + i);
#pragma unroll
      for (int j = 0; j < QJ; ++j) {
        const Bf16x3 b = operand(1, ks, j0 + j);
#pragma unroll
        for (int i = 0; i < QI; ++i) mfma_split(a[i], b, acc[i][j]);
        __builtin_amdgcn_sched_barrier(0);  // bounded registers
      }
    }
  };
  // a step out of the split's range: the fp32 matrix instructions, with
  // operands read again from memory (four tokens a product)
  auto compute_fp32 = [&](int64_t t0) {
    for (int tt = 0; tt < TPS; tt += 4) {
      const int64_t t = t0 + tt + g;
      const bool ok = t < t_end;
      const int64_t at = min(t, t_end - 1) * row_bytes + n * 4;
      float a[QI], b[QJ];
#pragma unroll
      for (int i = 0; i < QI; ++i) {
        float x = phi<DT_FP32>(*(const float*)(kh + at + 64 * (i0 + i)));
        if constexpr (MODE == MODE_BWD) x *= tstash[min(t, t_end - 1)].x;
        a[i] = ok ? x : 0.f;  // (masked last: 1/den may be infinite)
      }
#pragma unroll
      for (int j = 0; j < QJ; ++j) {
        const float y = *(const float*)(vh + at + 64 * (j0 + j));
        b[j] = ok ? y : 0.f;
      }
#pragma unroll
      for (int i = 0; i < QI; ++i)
#pragma unroll
        for (int j = 0; j < QJ; ++j) acc[i][j] = mfma_f32(a[i], b[j], acc[i][j]);
    }
  };

  Regs x;
  load(t_begin, x);
  __syncthreads();  // out_of_range is set
  const int steps = (int)((t_end - t_begin + TPS - 1) / TPS);
  for (int s = 0; s < steps; ++s) {
    const int64_t t0 = t_begin + s * TPS;
    stage(t0, x, s);
    load(t0 + TPS, x);
    __syncthreads();
    if (!out_of_range[s]) compute();
    __syncthreads();  // before the rows are written again
  }
  for (int s = 0; s < steps; ++s)
    if (out_of_range[s]) compute_fp32(t_begin + s * TPS);

  float* out = part + ((int64_t)bh * P + p) * E;
#pragma unroll
  for (int i = 0; i < QI; ++i)
#pragma unroll
    for (int j = 0; j < QJ; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        out[(16 * (i0 + i) + 4 * g + r) * D + 16 * (j0 + j) + n] = acc[i][j][r];
#pragma unroll
  for (int c = 0; c < 4; ++c) zred[r0][4 * c4 + c] = z[c];
  __syncthreads();
  if (tid < D) {
    double s = 0.0;
    for (int r = 0; r < RP; ++r) s += (double)zred[r][tid];
    out[D * D + tid] = (float)s;
  }
}

// ---------------------------------------------------------------------------
// Combine: FP64 sum of the P partials in a fixed order (so results are
// bitwise reproducible), writing the dense FP64 matrix M (S or dS) and
// vector (z or dz) and the matrix-core operands `what` asks for.
//
// A workgroup takes eight rows of M: four slices of 2 D threads, slice w
// summing quarter w of the partials, four columns a thread, and the quarters
// added as (q0 + q1) + (q2 + q3).  Eight rows by D columns are whole 16-byte
// words of both images (eight contraction indices each), so every store is
// one: the halfword stores this replaces took most of the time (1,024 heads
// of 4 partials at d = 64: 94 -> 37 us; 64 heads of 8: 14 -> 7.5 us).  The
// last workgroup of a head does the same for the vector.
// ---------------------------------------------------------------------------
template <int D, int IDT>
__global__ __launch_bounds__(8 * D) void combine_kernel(
    const float* __restrict__ part, int P,
    double* __restrict__ M64, double* __restrict__ v64, void* __restrict__ img, int what) {
  using IC = ImageCfg<D>;
  constexpr int E = D * D + D;
  __shared__ double qs[4][8][D];
  __shared__ double sum[8][D];
  const int bh = blockIdx.y, t = threadIdx.x;
  const bool vec = blockIdx.x == D / 8;
  const int rows = vec ? 1 : 8, row0 = 8 * blockIdx.x;
  const float* src = part + (int64_t)bh * P * E + (vec ? D * D : row0 * D);
  // slice w, element quad u of the rows; eight loads at a time in flight
  // (the last repeated past the end), added in order
  const int w = t / (2 * D), u = 4 * (t % (2 * D));
  const int pq = (P + 3) / 4, p0 = min(P, w * pq), p1 = min(P, p0 + pq);
  if (u < rows * D) {
    double q[4] = {0.0, 0.0, 0.0, 0.0};
    for (int p = p0; p < p1; p += 8) {
      f32x4 x[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) x[k] = *(const f32x4*)(src + (int64_t)min(p + k, p1 - 1) * E + u);
#pragma unroll
      for (int k = 0; k < 8; ++k)
#pragma unroll
        for (int r = 0; r < 4; ++r) q[r] += p + k < p1 ? (double)x[k][r] : 0.0;
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) (&qs[w][0][0])[u + r] = q[r];
  }
  __syncthreads();
  if (t < rows * D) {
    const double s = ((&qs[0][0][0])[t] + (&qs[1][0][0])[t]) + ((&qs[2][0][0])[t] + (&qs[3][0][0])[t]);
    (&sum[0][0])[t] = s;
    if (vec) v64[(int64_t)bh * D + t] = s;
    else M64[((int64_t)bh * D + row0) * D + t] = s;
  }
  __syncthreads();
  char* head = (char*)img + (int64_t)bh * IC::head_bytes(IDT);
  const bool lo = what & IMG_LO;
  int i, m;
  if (vec) {
    // the z tile: v in each of its 16 rows
    if ((what & IMG_Z) && t < 2 * D) {
      const int c0 = 8 * (t >> 4);
      put_image8<D, IDT>(head, IC::NT, t & 15, c0, &sum[0][c0], lo);
    }
    return;
  }
  // T image: row e, contraction over the eight rows here
  if ((what & IMG_T) && t < D) {
    double x[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) x[k] = sum[k][t];
    image_row<D, IDT>(t, i, m);
    put_image8<D, IDT>(head, i, m, row0, x, lo);
  }
  // N image: row row0 + r, contraction over the columns
  if ((what & IMG_N) && t >= 7 * D) {
    const int u = t - 7 * D, r = u & 7, e0 = 8 * (u >> 3);
    image_row<D, IDT>(row0 + r, i, m);
    put_image8<D, IDT>(head + IC::img_bytes(IDT), i, m, e0, &sum[r][e0], lo);
  }
}

// ---------------------------------------------------------------------------
// Apply: O^T = S^T phi(Q)^T per 16-token tile.  The G workgroups of a head
// take the head's blocks of 4 * 16 * TT tokens in turn (workgroup g: blocks
// g, g + G, g + 2G, ...; each wave 16 * TT tokens of a block), so the waves
// of the whole grid move through every tensor together and the accesses in
// flight at any moment lie in a narrow window of it: a copy stream laid
// out this way reached 5.49 TB/s on MI355X against 5.21 TB/s for the same
// copy with one contiguous range per wave.  Lane (g, n) holds token n
// and a run of Q4 = d/4 query features (Run: 16-byte chunks interleaved
// over the lane groups); the matrix-core result puts the value features of
// the same run positions of the same token in the same lane.  The normaliser den = phi(q) . z comes from
// the same matrix-core pass (the image's z tile: every output row of it is
// den of the lane's token), so the FP64 division and the store stay
// in-lane.  The S^T operands (bf16 hi + lo parts, or fp32) sit in LDS for
// the whole workgroup.
// ---------------------------------------------------------------------------
template <int DT, int D>
struct ApplyCfg {
  // 16-token tiles per step; every LDS operand read feeds TT matrix-core ops
  static constexpr int TT = 2;
  static constexpr int ES = DT == DT_BF16 ? 2 : 4;
  static constexpr int QB = D / 4 * ES;             // bytes of a lane's query run
  static constexpr int QW = QB / 4;
};

//
// MIX: the noise-gated epilogue.  Batch element b's spatial weight
// g_b = sigma_data / (sigma_data + sigma[b]) (FP64, once per workgroup)
// blends this attention with another branch's stored output (same dtype
// and strides as o): o = g_b A + (1 - g_b) other, in FP32 before the
// store.  The other branch's rows travel in the same register sets as the
// queries, a step ahead, where registers allow (bf16 in and out).  `other`
// may be `o` itself: each lane reads its elements before it writes them.
//
// img: the operands as the combine left them; null: each workgroup makes
// them from src, and where that holds partial sums the first of a head
// writes their FP64 sum if it is a result.
struct ApplySrc {
  const double *M, *v;     // FP64 summary, or
  const float* part;       // P partial sums a head, and where their sum goes
  int P;
  double *M_out, *v_out;   // (may be null)
};

template <int DT, int OT, int D, bool MIX>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void apply_kernel(
    const void* __restrict__ q, int64_t sb, int64_t sh, int64_t sn,
    void* o, int64_t osb, int64_t osh, int64_t osn, int H,
    int64_t N, int G, const void* __restrict__ img, ApplySrc src, const void* other,
    const double* __restrict__ sigma, double sigma_data) {
  using IC = ImageCfg<D>;
  using AC = ApplyCfg<DT, D>;
  constexpr int Q4 = D / 4;
  constexpr int NT = D / 16;
  constexpr int ES = AC::ES;
  constexpr int OES = OT == DT_BF16 ? 2 : 4;
  constexpr int QW = AC::QW;
  constexpr int IMG_WORDS = IC::img_bytes(DT) / 16;
  constexpr int TT = AC::TT;
  __shared__ u32x4 simg[IMG_WORDS];

  const int bh = blockIdx.y;
  const int64_t b = bh / H, h = bh % H;
  const int lane = threadIdx.x & 63, wave = wave_index();
  const int g = lane >> 4, n = lane & 15;

  // wave-uniform head pointers plus loop-invariant 32-bit lane offsets
  // (token n of the tile, lane group g's feature run)
  const int64_t row_bytes = sn * ES, orow_bytes = osn * OES;
  const char* qh = (const char*)q + (b * sb + h * sh) * ES;
  char* oh = (char*)o + (b * osb + h * osh) * OES;
  using RN = Run<D, DT>;
  const uint32_t ooff = (uint32_t)n * (uint32_t)orow_bytes + (uint32_t)(g * RN::CH * OES);

  // the gate: spatial weight gw, the other branch's weight hw
  float gw = 1.f, hw = 0.f;
  const char* xh = nullptr;
  if constexpr (MIX) {
    const double gg = sigma_data / (sigma_data + sigma[b]);
    gw = (float)gg;
    hw = (float)(1.0 - gg);
    xh = (const char*)other + (b * osb + h * osh) * OES;
  }
  constexpr int XW = MIX ? Q4 * OES / 4 : 1;  // words of a lane's run of `other`
  // bf16 in and out: `other` rides in the query register sets, a step
  // ahead; otherwise (registers) it is loaded as its step starts
  constexpr bool XPF = MIX && DT == DT_BF16 && OT == DT_BF16;

  struct QRegs {
    uint32_t q[TT][QW];
    uint32_t x[TT][XPF ? XW : 1];
  };
  auto load_x = [&](int64_t tb, uint32_t* xw) {
    load_out_run<D, DT, OT>(xh + tb * orow_bytes + ooff, xw);
  };
  // Rows past the head's last token read that token again (no zero fill
  // and no branch around the loads); their results are not stored.
  auto load_q = [&](int64_t t0, QRegs& r) {
#pragma unroll
    for (int tt = 0; tt < TT; ++tt) {
      const int64_t tb = min(t0 + 16 * tt, N - 1);  // wave-uniform
      const uint32_t row = (uint32_t)min(n, (int)min((int64_t)15, N - 1 - tb));
      load_run<D, DT>(qh + tb * row_bytes + (row * (uint32_t)row_bytes + (uint32_t)(g * RN::CB)),
                      r.q[tt]);
      if constexpr (XPF)
        load_out_run<D, DT, OT>(
            xh + tb * orow_bytes + (row * (uint32_t)orow_bytes + (uint32_t)(g * RN::CH * OES)),
            r.x[tt]);
    }
  };

  auto compute = [&](int64_t t0, const QRegs& r) {
    const auto& qw = r.q;
    // `other` when not prefetched: loaded as the step starts (bf16 queries)
    // or just before its use (fp32 queries, whose runs fill the registers)
    uint32_t xs[TT][MIX && !XPF ? XW : 1];
    if constexpr (MIX && !XPF && DT == DT_BF16) {
#pragma unroll
      for (int tt = 0; tt < TT; ++tt)
        if (t0 + 16 * tt + n < N) load_x(t0 + 16 * tt, xs[tt]);
    }
    // phi(q) as matrix-core operands; acc[tt][NT] is the z tile (den)
    f32x4 acc[TT][NT + 1];
#pragma unroll
    for (int tt = 0; tt < TT; ++tt)
#pragma unroll
      for (int i = 0; i <= NT; ++i) acc[tt][i] = f32x4{0.f, 0.f, 0.f, 0.f};
    if constexpr (DT == DT_BF16) {
      constexpr int NS = IC::NS;
      bf16x8 bq[TT][NS];
#pragma unroll
      for (int tt = 0; tt < TT; ++tt)
#pragma unroll
        for (int s = 0; s < NS; ++s) {
          u32x4 w;
#pragma unroll
          for (int pp = 0; pp < 4; ++pp) {
            const int c0 = 8 * s + 2 * pp;
            if (c0 < Q4) {
              const float p0 = phi<DT>(word_elem<DT>(qw[tt], c0));
              const float p1 = phi<DT>(word_elem<DT>(qw[tt], c0 + 1));
              w[pp] = pack_bf16(p0, p1);
            } else {
              w[pp] = 0;
            }
          }
          bq[tt][s] = as_bf16x8(w);
        }
#pragma unroll
      for (int i = 0; i <= NT; ++i)
#pragma unroll
        for (int s = 0; s < NS; ++s) {
          const bf16x8 hi = as_bf16x8(simg[((i * NS + s) * 2 + 0) * 64 + lane]);
          const bf16x8 lo = as_bf16x8(simg[((i * NS + s) * 2 + 1) * 64 + lane]);
#pragma unroll
          for (int tt = 0; tt < TT; ++tt) {
            // the chain's first product starts from zero (no separate clear)
            acc[tt][i] = mfma_bf16(hi, bq[tt][s], s == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : acc[tt][i]);
            acc[tt][i] = mfma_bf16(lo, bq[tt][s], acc[tt][i]);
          }
          // keep the operand reads next to their use (bounded registers)
          if constexpr (D >= 128) __builtin_amdgcn_sched_barrier(0);
        }
    } else {
      float pq[TT][Q4];
#pragma unroll
      for (int tt = 0; tt < TT; ++tt)
#pragma unroll
        for (int c = 0; c < Q4; ++c) pq[tt][c] = phi<DT>(word_elem<DT>(qw[tt], c));
#pragma unroll
      for (int i = 0; i <= NT; ++i)
#pragma unroll
        for (int s4 = 0; s4 < Q4 / 4; ++s4) {
          const u32x4 a = simg[(i * (Q4 / 4) + s4) * 64 + lane];
#pragma unroll
          for (int t4 = 0; t4 < 4; ++t4)
#pragma unroll
            for (int tt = 0; tt < TT; ++tt)
              acc[tt][i] = mfma_f32(__uint_as_float(a[t4]), pq[tt][4 * s4 + t4],
                                    s4 == 0 && t4 == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : acc[tt][i]);
        }
    }
#pragma unroll
    for (int tt = 0; tt < TT; ++tt) {
      // O = num / den: FP64 reciprocal, applied as its two-float expansion
      // rh + rl (num * rh + num * rl with one rounding: within an ulp of
      // the FP64 product rounded to fp32)
      const double rden = 1.0 / (double)acc[tt][NT][0];
      const float rh = (float)rden, rl = (float)(rden - (double)rh);
      if (t0 + 16 * tt + n < N) {
        float out[Q4];
#pragma unroll
        for (int i = 0; i < NT; ++i)
#pragma unroll
          for (int r = 0; r < 4; ++r)
            out[4 * i + r] = fmaf(acc[tt][i][r], rh, acc[tt][i][r] * rl);
        if constexpr (MIX) {
          if constexpr (!XPF && DT != DT_BF16) load_x(t0 + 16 * tt, xs[tt]);
#pragma unroll
          for (int c = 0; c < Q4; ++c)
            out[c] = fmaf(gw, out[c], hw * word_elem<OT>(XPF ? r.x[tt] : xs[tt], c));
        }
        store_run<D, DT, OT>(oh + (t0 + 16 * tt) * orow_bytes + ooff, out);
      }
    }
  };

  // two register sets in turn: the next step's queries are in flight in
  // one while the other's step computes (no copies between them).  The
  // loads are unconditional and the loop body has no early exit, so the
  // compiler's wait counts cover only the set a step is about to use (an
  // odd step count runs one step with nothing to store); the scheduling
  // barriers keep each load ahead of the step that overlaps it.
  constexpr int BLK = 16 * TT * 4;  // tokens per block
  const int64_t nblk = (N + BLK - 1) / BLK;
  const int64_t blk0 = blockIdx.x;
  const int nk = blk0 < nblk ? (int)((nblk - 1 - blk0) / G + 1) : 0;
  // first token of this wave's part of the k-th block it takes
  auto tok = [&](int k) { return (blk0 + (int64_t)k * G) * BLK + 16 * TT * wave; };
  // the first queries are in flight while the workgroup stages the T image
  // (the first of the head's two, S^T operands) into LDS
  QRegs qa, qb;
  if (nk > 0) load_q(tok(0), qa);
  if (img) {
    const u32x4* from = (const u32x4*)((const char*)img + (int64_t)bh * IC::head_bytes(DT));
    for (int w = threadIdx.x; w < IMG_WORDS; w += 256) simg[w] = from[w];
  } else {
    const MatrixSrc<D> s{src.M ? src.M + (int64_t)bh * D * D : nullptr,
                         src.v ? src.v + (int64_t)bh * D : nullptr,
                         src.part ? src.part + (int64_t)bh * src.P * (D * D + D) : nullptr, src.P};
    constexpr bool MANY = D <= 32;
    __shared__ double sum[MANY ? D * D + D : 1];
    if (MANY && src.part && src.P > 4) {
      sum_partials<MANY ? D : 16, 256>(sum, s.part, src.P);
      const MatrixSrc<D> t{sum, sum + D * D, nullptr, 0};
      make_image<DT, D, 2, true, 0, 256>(simg, t);
      make_z_tile<DT, D, 0>(simg + IC::mat_bytes(DT) / 16, t);
      if (src.M_out && blockIdx.x == 0)
        for (int u = threadIdx.x; u < D * D + D; u += 256) {
          if (u < D * D) src.M_out[(int64_t)bh * D * D + u] = sum[u];
          else src.v_out[(int64_t)bh * D + u - D * D] = sum[u];
        }
    } else if (!src.part) {
      make_image<DT, D, 2, true, 0, 256>(simg, s);
      make_z_tile<DT, D, 0>(simg + IC::mat_bytes(DT) / 16, s);
    } else {
      by_partials(src.P, [&](auto pn) {
        constexpr int PN = decltype(pn)::value;
        make_image<DT, D, 2, true, PN, 256>(simg, s);
        make_z_tile<DT, D, PN>(simg + IC::mat_bytes(DT) / 16, s);
        if (src.M_out && blockIdx.x == 0) {
          double x[2];
          for (int u = threadIdx.x; u < (D * D + D) / 2; u += 256) {
            const bool vec = u >= D * D / 2;
            const int i = 2 * u - (vec ? D * D : 0);
            s.template get<PN, 2>(i, vec, x);
            double* to = vec ? src.v_out + (int64_t)bh * D + i : src.M_out + (int64_t)bh * D * D + i;
            to[0] = x[0]; to[1] = x[1];
          }
        }
      });
    }
  }
  __syncthreads();
  if (nk > 0) {
    for (int k = 0; k < nk; k += 2) {
      load_q(tok(k + 1), qb);
      __builtin_amdgcn_sched_barrier(0);
      compute(tok(k), qa);
      load_q(tok(k + 2), qa);
      __builtin_amdgcn_sched_barrier(0);
      compute(tok(k + 1), qb);
    }
  }
}

// ---------------------------------------------------------------------------
// Host-side launchers
// ---------------------------------------------------------------------------
// Tokens of a summary's runs: four to a partial where the teams take them
// (d >= 64, short sequences), else up to eight (d <= 32: sixteen) of at least
// 256 (128) tokens, so that a wave that takes them all adds up every eight
// (four) steps; at d = 128, where a wave's sum fills 64 KB, one.  (Kept in
// memory between the runs, or in a launch for each, it cost 8 to 25 % of the
// summary of eight heads and more.)
static int summary_run(int D, int Tw, bool team) {
  if (team) return (Tw / 4 + 31) / 32 * 32;
  const int most = D >= 128 ? 1 : D == 64 ? 8 : 16;
  const int runs = std::max(1, std::min(most, Tw / (D == 64 ? 256 : 128)));
  return ((Tw + runs - 1) / runs + 63) / 64 * 64;
}

template <int DT, int D, int MODE>
static void launch_summary_t(const void* k, const void* v, int64_t sb, int64_t sh, int64_t sn,
                             int64_t BH, int64_t H, int64_t N, int P, int Tw, bool team,
                             const float2* stash, float* part, hipStream_t stream) {
  const int64_t items = P * BH;
  const dim3 one((unsigned)((items + 7) / 8 * 8));
  if constexpr (DT == DT_FP32 && D >= 32) {
    summary_split_kernel<D, MODE><<<one, 64 * SplitCfg<D>::NW, 0, stream>>>(
        k, v, sb, sh, sn, (int)H, N, P, Tw, stash, part, (int)BH);
  } else {
#define LA_SUM(NW, GRID)                                                             \
  summary_kernel<DT, D, MODE, NW><<<GRID, NW == 1 ? 256 : 64 * NW, 0, stream>>>(      \
      k, v, sb, sh, sn, (int)H, N, P, Tw, Tq, stash, part, (int)BH, join64)
    const int Tq = summary_run(D, Tw, team);
    // an FP32 sum covers at most 2,048 (d = 128) or 512 tokens of a team's
    // (the join in FP64 takes conversions: 2 us of the 20 of two heads of
    // 1,000 tokens at d = 128, whose partials are shorter)
    const bool join64 = team && Tw > (D >= 128 ? 2048 : 512);
    const int runs = (Tw + Tq - 1) / Tq;
    // A wave to a whole partial where those fill the chip, d = 64: from 832
    // partials (12 heads of 50,000 tokens in 64 each: 40 us by teams, 44; 14:
    // 50, 44); d = 32: from 2,048 unless heads share cache lines (64 heads of
    // 30,001 tokens: 63 us by teams, 60; as views of [B, N, H, d] 76 and 82);
    // d = 16 never (128 heads of 60,000: 164 us, 174).
    const bool whole = D >= 32 && items >= (D == 32 ? 2048 : 832) &&
                       !(D == 32 && lines_shared(sh * SummaryCfg<DT, D, MODE>::ES, H));
    if (runs > 1 && (team || !whole)) {
      if (runs <= 4) {
        LA_SUM(4, one);
      } else if (runs <= 8) {
        if constexpr (D <= 64) LA_SUM(8, one);
      } else {
        if constexpr (D <= 32) LA_SUM(16, one);
      }
    } else {
      LA_SUM(1, dim3((unsigned)((items + 3) / 4)));
    }
#undef LA_SUM
  }
}

template <int D>
static void launch_summary_d(int mode, int dt, const void* k, const void* v, int64_t sb,
                             int64_t sh, int64_t sn, int64_t B, int64_t H, int64_t N, int P,
                             int Tw, bool team, const float2* stash, float* part,
                             hipStream_t stream) {
  ProfScope prof(mode == MODE_FWD ? "summary_fwd" : "summary_bwd", stream);
  const int64_t BH = B * H;
#define LA_SUM(DTI, M) \
  launch_summary_t<DTI, D, M>(k, v, sb, sh, sn, BH, H, N, P, Tw, team, stash, part, stream)
  if (mode == MODE_FWD) {
    if (dt == DT_BF16) LA_SUM(DT_BF16, MODE_FWD); else LA_SUM(DT_FP32, MODE_FWD);
  } else if (dt == DT_FP32) {
    LA_SUM(DT_FP32, MODE_BWD);
  } else if constexpr (D == 16) {  // (wider bf16 heads: la_backward.hip's fused pass)
    LA_SUM(DT_BF16, MODE_BWD);
  }
#undef LA_SUM
}

hipError_t launch_summary_bwd(int dt, int D, const void* q, const void* g, int64_t sb, int64_t sh,
                              int64_t sn, int64_t B, int64_t H, int64_t N, int P, int Tw,
                              const float2* stash, float* part, hipStream_t stream) {
  if (dt == DT_BF16 && D != 16) return hipErrorInvalidValue;  // la_backward.hip's fused pass
#define LA_SUM(D) \
  launch_summary_d<D>(MODE_BWD, dt, q, g, sb, sh, sn, B, H, N, P, Tw, false, stash, part, stream)
  switch (D) {
    case 16: LA_SUM(16); break;
    case 32: LA_SUM(32); break;
    case 64: LA_SUM(64); break;
    case 128: LA_SUM(128); break;
    default: return hipErrorInvalidValue;
  }
#undef LA_SUM
  return hipGetLastError();
}

template <int D>
static void launch_combine_d(const float* part, int P, double* M64, double* v64, void* img,
                             int img_dt, int64_t BH, int what, hipStream_t stream) {
  const dim3 grid(D / 8 + 1, (unsigned)BH);
  if (img_dt == DT_BF16)
    combine_kernel<D, DT_BF16><<<grid, 8 * D, 0, stream>>>(part, P, M64, v64, img, what);
  else
    combine_kernel<D, DT_FP32><<<grid, 8 * D, 0, stream>>>(part, P, M64, v64, img, what);
}

hipError_t launch_combine(const float* part, int P, double* M64, double* v64, void* img,
                          int img_dt, int64_t BH, int D, int what, hipStream_t stream) {
  ProfScope prof("combine", stream);
  switch (D) {
    case 16: launch_combine_d<16>(part, P, M64, v64, img, img_dt, BH, what, stream); break;
    case 32: launch_combine_d<32>(part, P, M64, v64, img, img_dt, BH, what, stream); break;
    case 64: launch_combine_d<64>(part, P, M64, v64, img, img_dt, BH, what, stream); break;
    case 128: launch_combine_d<128>(part, P, M64, v64, img, img_dt, BH, what, stream); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <int D>
static hipError_t launch_apply_only(const FwdArgs& a, const void* img, const ApplySrc& src);

template <int D>
static hipError_t launch_forward_d(const FwdArgs& a) {
  const int BH = (int)(a.B * a.H);
  launch_summary_d<D>(MODE_FWD, a.in_dt, a.k, a.v, a.sb, a.sh, a.sn, a.B, a.H, a.N, a.P, a.Tw,
                      a.team, nullptr, a.part, a.stream);
  // few partials: the apply's workgroups add them up themselves
  if (!fp32_rows(a.in_dt, D) && fold_partials(a.P, a.Ga, BH, D))
    return launch_apply_only<D>(a, nullptr, ApplySrc{nullptr, nullptr, a.part, a.P,
                                                     a.want_summary ? a.S64 : nullptr, a.z64});
  {
    ProfScope prof("combine", a.stream);
    launch_combine_d<D>(a.part, a.P, a.S64, a.z64, a.img, a.in_dt, BH,
                        fp32_rows(a.in_dt, D) ? 0 : IMG_T | IMG_Z | IMG_LO, a.stream);
  }
  return launch_apply_only<D>(a, a.img, ApplySrc{});
}

template <int D>
static hipError_t launch_apply_only(const FwdArgs& a, const void* img, const ApplySrc& src) {
  if (fp32_rows(a.in_dt, D)) return launch_apply_fp32(a);
  const int BH = (int)(a.B * a.H);
  dim3 agrid((unsigned)a.Ga, BH);
  ProfScope prof(a.other ? "apply_gated" : "apply", a.stream);
#define LA_APPLY(DTI, DTO, MIX)                                                   \
  apply_kernel<DTI, DTO, D, MIX><<<agrid, 256, 0, a.stream>>>(                     \
      a.q, a.sb, a.sh, a.sn, a.o, a.osb, a.osh, a.osn, (int)a.H, a.N, a.Ga, img, src, a.other, \
      a.sigma, a.sigma_data)
#define LA_APPLY_DT(MIX)                                                \
  if (a.in_dt == DT_BF16 && a.out_dt == DT_BF16) LA_APPLY(DT_BF16, DT_BF16, MIX); \
  else if (a.in_dt == DT_BF16) LA_APPLY(DT_BF16, DT_FP32, MIX);                   \
  else if constexpr (!fp32_rows(DT_FP32, D)) {                                    \
    if (a.out_dt == DT_BF16) LA_APPLY(DT_FP32, DT_BF16, MIX);                     \
    else LA_APPLY(DT_FP32, DT_FP32, MIX);                                         \
  }
  if (a.other) {
    LA_APPLY_DT(true)
  } else {
    LA_APPLY_DT(false)
  }
#undef LA_APPLY_DT
#undef LA_APPLY
  return hipGetLastError();
}

hipError_t launch_forward(const FwdArgs& a) {
  switch (a.D) {
    case 16: return launch_forward_d<16>(a);
    case 32: return launch_forward_d<32>(a);
    case 64: return launch_forward_d<64>(a);
    case 128: return launch_forward_d<128>(a);
  }
  return hipErrorInvalidValue;
}

template <int D>
static hipError_t launch_apply_d(const FwdArgs& a) {
  if (fp32_rows(a.in_dt, D)) return launch_apply_fp32(a);
  return launch_apply_only<D>(a, nullptr, ApplySrc{a.S64, a.z64, nullptr, 0, nullptr, nullptr});
}

hipError_t launch_apply(const FwdArgs& a) {
  switch (a.D) {
    case 16: return launch_apply_d<16>(a);
    case 32: return launch_apply_d<32>(a);
    case 64: return launch_apply_d<64>(a);
    case 128: return launch_apply_d<128>(a);
  }
  return hipErrorInvalidValue;
}

}  // namespace la
