// la_fp32.hip -- gfx950 row kernels of fp32 inputs at d = 64 and 128: apply,
// query backward and key backward on the bf16 matrix cores (la_split.h).
//
// As in the bf16 kernels, lane (g, n) holds token n of a 16-token tile and a
// run of d/4 features, here features 16 c + 4 g + j at run position 4 c + j,
// and a product A x (runs) puts the output features of the same run
// positions in the same lane: output tile i is features 16 i .. 16 i + 15.
// A is the FP64 d x d matrix (S or dS) itself, split into three bf16 parts
// as a workgroup stages it into LDS, row by row.  One copy serves both
// orientations: the transposing LDS read gives A^T's operands (contraction
// over its rows), plain 8-byte reads give A's (over its columns), so the key
// backward holds dS once (96 KB at d = 128) and reads K and V once, where
// two fp32 images did not fit LDS and took two passes.
//
// Each tile's output is finished and stored as soon as its product is, so
// no accumulators are kept.  A wave leaves out the tiles whose operands are
// outside the split's range and takes them after the others with the fp32
// matrix instructions, operands straight from the FP64 matrix.
//
// What bounds them: HBM and, within 20 %, the matrix cores (per 16 tokens
// and product at d = 128, 216 bf16 instructions of 16 cycles a wave, half of
// what a SIMD has while HBM moves the rows).
#include <algorithm>
#include <type_traits>

#include "la_kernels.h"
#include "la_profile.h"
#include "la_split.h"

namespace la {

template <int D>
struct Rows32 {
  static constexpr int Q4 = D / 4, NT = D / 16, NS = D / 32;
  // d = 128: the matrix leaves room for one workgroup on a compute unit
  static constexpr int NW = D == 128 ? 8 : 4;
  static constexpr int NTH = 64 * NW;
  static constexpr int ROW = 2 * D, PART = D * ROW;  // LDS bytes of a row, of a part
};

// The matrix in LDS: 16-byte chunks of a row are XOR-swizzled so that the
// eight rows (32 bytes each) of a half wave's transposing read and the 16
// rows (16 bytes each) of a half wave's plain read lie in distinct banks.
template <int D>
__device__ __forceinline__ int mat_swz(int row) {
  return (D == 128 ? 2 * (row & 7) : 2 * ((row >> 1) & 3)) ^ ((row >> 3) & 1);
}

template <int D>
struct MatLds {
  __align__(16) char m[3 * Rows32<D>::PART];
  uint16_t v[3][D];  // the vector's parts
  double vd[D];      // the vector
  int out_of_range;
};

// The parts of two FP64 values.
__device__ __forceinline__ Split2 split2(double a, double b) {
  Split2 s;
  s.h = pack_bf16((float)a, (float)b);
  const double a1 = a - (double)bf16lo(s.h), b1 = b - (double)bf16hi(s.h);
  s.m = pack_bf16((float)a1, (float)b1);
  s.l = pack_bf16((float)(a1 - (double)bf16lo(s.m)), (float)(b1 - (double)bf16hi(s.m)));
  return s;
}

// Stage M [D][D] and v [D]; barriers are the caller's (one before, so that
// out_of_range is cleared, is here).  COLS, ROWS: whether M's columns, its
// rows are results of the kernel's products, whose ranges count one by one
// (a thread meets 2 (d = 128: 4) elements of each of its columns and eight of
// a row at a time); VEC: whether v is an operand too.
template <int D, bool COLS, bool ROWS, bool VEC>
__device__ __forceinline__ void stage_matrix(MatLds<D>& L, const double* __restrict__ M,
                                             const double* __restrict__ v) {
  using C = Rows32<D>;
  if (threadIdx.x == 0) L.out_of_range = 0;
  __syncthreads();
  const double vx = threadIdx.x < D ? v[threadIdx.x] : 0.0;  // in flight with the matrix's loads
  SplitRange<8> cols;
  bool bad = false;
  static_assert(C::NTH % (D / 8) == 0, "a thread's elements lie in the same columns");
  for (int u = threadIdx.x; u < D * D / 8; u += C::NTH) {
    const int row = u / (D / 8), ch = u % (D / 8);
    SplitRange<> r;
    double x[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) x[j] = M[row * D + 8 * ch + j];
    u32x4 h, m, l;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float a = (float)x[2 * j], b = (float)x[2 * j + 1];
      if (ROWS) r.see(0, a, b);
      if (COLS) {
        cols.see(2 * j, a);
        cols.see(2 * j + 1, b);
      }
      const Split2 s = split2(x[2 * j], x[2 * j + 1]);
      h[j] = s.h;
      m[j] = s.m;
      l[j] = s.l;
    }
    char* at = L.m + row * C::ROW + ((ch ^ mat_swz<D>(row)) << 4);
    *(u32x4*)at = h;
    *(u32x4*)(at + C::PART) = m;
    *(u32x4*)(at + 2 * C::PART) = l;
    bad |= r.bad();
  }
  bad |= cols.bad();
  if (threadIdx.x < D) {
    const float mag = fabsf((float)vx);  // the vector's elements are summed: judged 64 at a time
    if (VEC) bad |= !(mag < 0x1p63f) || (mag > 0.f && !__any(mag >= 0x1p-90f));
    const Split2 s = split2(vx, 0.0);
    L.v[0][threadIdx.x] = (uint16_t)s.h;
    L.v[1][threadIdx.x] = (uint16_t)s.m;
    L.v[2][threadIdx.x] = (uint16_t)s.l;
    L.vd[threadIdx.x] = vx;
  }
  if (bad) L.out_of_range = 1;  // every writer stores the same
}

__device__ __forceinline__ bf16x8 join(const u32x2& lo, const u32x2& hi) {
  return as_bf16x8(u32x4{lo[0], lo[1], hi[0], hi[1]});
}

// Operands of k-step s (contraction indices 32 s .. 32 s + 31, lane group g
// taking 32 s + 4 g + j and 32 s + 16 + 4 g + j, as the runs do).
// Columns: row m of the operand is matrix column 16 i + m (A^T).
template <int D>
__device__ __forceinline__ Bf16x3 column_operand(const MatLds<D>& L, int base, int i, int s) {
  using C = Rows32<D>;
  const char* p = L.m + (base ^ (i << 5)) + 32 * s * C::ROW;
  Bf16x3 r;
  r.h = join(lds_read_tr16(p), lds_read_tr16(p + 16 * C::ROW));
  r.m = join(lds_read_tr16(p + C::PART), lds_read_tr16(p + C::PART + 16 * C::ROW));
  r.l = join(lds_read_tr16(p + 2 * C::PART), lds_read_tr16(p + 2 * C::PART + 16 * C::ROW));
  return r;
}
template <int D>
__device__ __forceinline__ int column_base(int g, int n) {
  const int row = 4 * g + (n >> 2);
  return row * Rows32<D>::ROW + ((((n & 3) >> 1) ^ mat_swz<D>(row)) << 4) + (n & 1) * 8;
}
// Rows: row m of the operand is matrix row 16 i + m.
template <int D>
__device__ __forceinline__ Bf16x3 row_operand(const MatLds<D>& L, int base, int i, int s) {
  using C = Rows32<D>;
  const char* p0 = L.m + (base ^ (s << 6)) + 16 * i * C::ROW;
  const char* p1 = L.m + (base ^ (s << 6) ^ 32) + 16 * i * C::ROW;
  Bf16x3 r;
  r.h = join(*(const u32x2*)p0, *(const u32x2*)p1);
  r.m = join(*(const u32x2*)(p0 + C::PART), *(const u32x2*)(p1 + C::PART));
  r.l = join(*(const u32x2*)(p0 + 2 * C::PART), *(const u32x2*)(p1 + 2 * C::PART));
  return r;
}
template <int D>
__device__ __forceinline__ int row_base(int g, int n) {
  return n * Rows32<D>::ROW + (((g >> 1) ^ mat_swz<D>(n)) << 4) + (g & 1) * 8;
}
// The vector in every row of the operand.
template <int D>
__device__ __forceinline__ Bf16x3 vector_operand(const MatLds<D>& L, int g, int s) {
  Bf16x3 r;
  bf16x8* o[3] = {&r.h, &r.m, &r.l};
#pragma unroll
  for (int q = 0; q < 3; ++q)
    *o[q] = join(*(const u32x2*)&L.v[q][32 * s + 4 * g], *(const u32x2*)&L.v[q][32 * s + 16 + 4 * g]);
  return r;
}

// The small products of a k-step into `small`, the large one into `big`.
__device__ __forceinline__ void split_products(const Bf16x3& a, const Bf16x3& b, f32x4& big, f32x4& small) {
  small = mfma_bf16(a.h, b.l, small);
  small = mfma_bf16(a.l, b.h, small);
  small = mfma_bf16(a.m, b.m, small);
  small = mfma_bf16(a.h, b.m, small);
  small = mfma_bf16(a.m, b.h, small);
  big = mfma_bf16(a.h, b.h, big);
}

// A run's values at k-step s as an operand.
__device__ __forceinline__ Bf16x3 split_run(const float* x) {
  u32x4 h, m, l;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const Split2 s = split2(x[2 * j], x[2 * j + 1]);
    h[j] = s.h;
    m[j] = s.m;
    l[j] = s.l;
  }
  return Bf16x3{as_bf16x8(h), as_bf16x8(m), as_bf16x8(l)};
}

// Matrix index of run position p of lane group g.
__device__ __forceinline__ int run_feature(int g, int p) { return 16 * (p >> 2) + 4 * g + (p & 3); }

// Blocks of 16 * TT * NW tokens, workgroup g of a head taking g, g + G, ...
// (the whole grid moves through the tensors together); wave w's tiles of the
// k-th block.
template <int D, int TT>
struct Sweep {
  static constexpr int BLK = 16 * TT * Rows32<D>::NW;
  int64_t blk0;
  int G, nk, wave;
  __device__ __forceinline__ Sweep(int64_t N, int G_, int wave_) : blk0(blockIdx.x), G(G_), wave(wave_) {
    const int64_t nblk = (N + BLK - 1) / BLK;
    nk = blk0 < nblk ? (int)((nblk - 1 - blk0) / G + 1) : 0;
  }
  __device__ __forceinline__ int64_t token(int k) const {
    return (blk0 + (int64_t)k * G) * BLK + 16 * TT * wave;
  }
};

// Four consecutive output values of a token.
template <int OT>
__device__ __forceinline__ void store4(char* p, const float* x) {
  if constexpr (OT == DT_BF16) *(u32x2*)p = u32x2{pack_bf16(x[0], x[1]), pack_bf16(x[2], x[3])};
  else *(f32x4*)p = f32x4{x[0], x[1], x[2], x[3]};
}
template <int OT>
struct Out4 {
  typename std::conditional<OT == DT_BF16, u32x2, u32x4>::type w;
  __device__ __forceinline__ void load(const char* p) { w = *(const decltype(w)*)p; }
  __device__ __forceinline__ float operator[](int r) const {
    if constexpr (OT == DT_BF16) return (r & 1) ? bf16hi(w[r >> 1]) : bf16lo(w[r >> 1]);
    else return __uint_as_float(w[r]);
  }
};

// A lane's run of the tile at t0 (rows past the end read the last one again).
template <int D>
__device__ __forceinline__ void load_rows(const char* base, int64_t row_bytes, int64_t t0, int64_t N,
                                          int g, int n, uint32_t* w) {
  const int64_t tb = min(t0, N - 1);  // wave-uniform
  const uint32_t row = (uint32_t)min(n, (int)min((int64_t)15, N - 1 - tb));
  load_run<D, DT_FP32>(base + tb * row_bytes + (row * (uint32_t)row_bytes + (uint32_t)(g * 16)), w);
}

// ---------------------------------------------------------------------------
// Apply: O_i = phi(q_i)^T S / (phi(q_i) . z); MIX: blended with `other` (see
// apply_kernel).
// ---------------------------------------------------------------------------
template <int OT, int D, bool MIX>
__global__ __launch_bounds__(Rows32<D>::NTH) __attribute__((amdgpu_waves_per_eu(2))) void apply_split_kernel(
    const void* __restrict__ q, int64_t sb, int64_t sh, int64_t sn, void* o, int64_t osb,
    int64_t osh, int64_t osn, int H, int64_t N, int G, const double* __restrict__ S64,
    const double* __restrict__ z64, const void* other, const double* __restrict__ sigma,
    double sigma_data) {
  using C = Rows32<D>;
  constexpr int Q4 = C::Q4, NT = C::NT, NS = C::NS, TT = MIX && D == 128 ? 1 : 2;
  constexpr int OES = OT == DT_BF16 ? 2 : 4;
  __shared__ MatLds<D> L;
  const int bh = blockIdx.y;
  const int64_t b = bh / H, h = bh % H;
  const int lane = threadIdx.x & 63, wave = wave_index();
  const int g = lane >> 4, n = lane & 15;
  const int64_t row_bytes = sn * 4, orow_bytes = osn * OES;
  const char* qh = (const char*)q + (b * sb + h * sh) * 4;
  char* oh = (char*)o + (b * osb + h * osh) * OES;
  const double* M = S64 + (int64_t)bh * D * D;
  const double* v = z64 + (int64_t)bh * D;
  float gw = 1.f, hw = 0.f;
  const char* xh = nullptr;
  if constexpr (MIX) {
    const double gg = sigma_data / (sigma_data + sigma[b]);
    gw = (float)gg;
    hw = (float)(1.0 - gg);
    xh = (const char*)other + (b * osb + h * osh) * OES;
  }
  const Sweep<D, TT> sw(N, G, wave);

  uint32_t raw[TT][Q4];
  auto load = [&](int k) {
#pragma unroll
    for (int tt = 0; tt < TT; ++tt) load_rows<D>(qh, row_bytes, sw.token(k) + 16 * tt, N, g, n, raw[tt]);
  };
  // O = num / den by the two-float expansion of the FP64 reciprocal, the
  // blend, and the store, four features of a token at a time
  auto finish = [&](const f32x4& num, float rh, float rl, int64_t t, int i, const Out4<OT>& x) {
    if (t >= N) return;
    const int64_t at = t * orow_bytes + (16 * i + 4 * g) * OES;
    float out[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) out[r] = fmaf(num[r], rh, num[r] * rl);
    if constexpr (MIX) {
#pragma unroll
      for (int r = 0; r < 4; ++r) out[r] = fmaf(gw, out[r], hw * x[r]);
    }
    store4<OT>(oh + at, out);
  };
  auto reciprocal = [](double den, float& rh, float& rl) {
    const double rden = 1.0 / den;
    rh = (float)rden;
    rl = (float)(rden - (double)rh);
  };
  if (sw.nk > 0) load(0);
  stage_matrix<D, true, false, true>(L, M, v);
  __syncthreads();
  const bool all_bad = __builtin_amdgcn_readfirstlane(L.out_of_range);  // uniform over the workgroup
  const int cbase = column_base<D>(g, n);

  Bf16x3 p[TT][NS];
  // phi of the loaded rows as operands; whether all lie in the range
  auto convert = [&]() {
    SplitRange<TT> range;
#pragma unroll
    for (int tt = 0; tt < TT; ++tt)
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        float x[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) x[j] = phi<DT_FP32>(__uint_as_float(raw[tt][8 * s + j]));
#pragma unroll
        for (int j = 0; j < 8; j += 2) range.see(tt, x[j], x[j + 1]);
        p[tt][s] = split_run(x);
      }
    return !all_bad && !__any(range.bad());
  };
  // the other branch's rows of a step
  constexpr int XT = MIX ? NT : 1;
  auto load_other = [&](int k, Out4<OT> (&x)[TT][XT]) {
    if constexpr (MIX) {
#pragma unroll
      for (int tt = 0; tt < TT; ++tt) {
        const int64_t t = min(sw.token(k) + 16 * tt + n, N - 1);
#pragma unroll
        for (int i = 0; i < NT; ++i) x[tt][i].load(xh + t * orow_bytes + (16 * i + 4 * g) * OES);
      }
    }
  };
  bool left_out = false;
  for (int k = 0; k < sw.nk; ++k) {
    const bool good = convert();  // wave-uniform
    Out4<OT> x[TT][XT];
    load_other(k, x);
    load(k + 1);
    __builtin_amdgcn_sched_barrier(0);
    if (!good) {
      left_out = true;
      continue;
    }
    const int64_t t0 = sw.token(k) + n;
    float rh[TT], rl[TT];
    {
      f32x4 big[TT], small[TT];
#pragma unroll
      for (int tt = 0; tt < TT; ++tt) big[tt] = small[tt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        const Bf16x3 a = vector_operand<D>(L, g, s);
#pragma unroll
        for (int tt = 0; tt < TT; ++tt) split_products(a, p[tt][s], big[tt], small[tt]);
      }
#pragma unroll
      for (int tt = 0; tt < TT; ++tt) reciprocal((double)big[tt][0] + (double)small[tt][0], rh[tt], rl[tt]);
    }
#pragma unroll
    for (int i = 0; i < NT; ++i) {
      f32x4 big[TT], small[TT];
#pragma unroll
      for (int tt = 0; tt < TT; ++tt) big[tt] = small[tt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        const Bf16x3 a = column_operand<D>(L, cbase, i, s);
#pragma unroll
        for (int tt = 0; tt < TT; ++tt) split_products(a, p[tt][s], big[tt], small[tt]);
      }
#pragma unroll
      for (int tt = 0; tt < TT; ++tt) finish(big[tt] + small[tt], rh[tt], rl[tt], t0 + 16 * tt, i, x[tt][MIX ? i : 0]);
      __builtin_amdgcn_sched_barrier(0);  // bounded registers
    }
  }
  if (!left_out) return;
  for (int k = 0; k < sw.nk; ++k) {
    load(k);
    if (convert()) continue;
    Out4<OT> x[TT][XT];
    load_other(k, x);
#pragma unroll
    for (int tt = 0; tt < TT; ++tt) {
      f32x4 den = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int c = 0; c < Q4; ++c)
        den = mfma_f32((float)v[run_feature(g, c)], phi<DT_FP32>(__uint_as_float(raw[tt][c])), den);
      float rh, rl;
      reciprocal((double)den[0], rh, rl);
#pragma unroll
      for (int i = 0; i < NT; ++i) {
        f32x4 num = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int c = 0; c < Q4; ++c)
          num = mfma_f32((float)M[run_feature(g, c) * D + 16 * i + n],
                         phi<DT_FP32>(__uint_as_float(raw[tt][c])), num);
        finish(num, rh, rl, sw.token(k) + 16 * tt + n, i, x[tt][MIX ? i : 0]);
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Query backward: X = S G, G . O = phi(q) . X / den, dQ = (X - (G . O) z) /
// den phi'(q), and (1/den, -(G . O)) per token for the dS/dz reduction; the
// per-token arithmetic is FP64.
// ---------------------------------------------------------------------------
template <int OT, int D>
__global__ __launch_bounds__(Rows32<D>::NTH) __attribute__((amdgpu_waves_per_eu(2))) void query_split_kernel(
    const void* __restrict__ q, const void* __restrict__ dout, int64_t sb, int64_t sh, int64_t sn,
    void* __restrict__ dq, int64_t osb, int64_t osh, int64_t osn, int H, int64_t N, int G,
    const double* __restrict__ S64, const double* __restrict__ z64, float2* __restrict__ stash) {
  using C = Rows32<D>;
  constexpr int Q4 = C::Q4, NT = C::NT, NS = C::NS;
  constexpr int OES = OT == DT_BF16 ? 2 : 4;
  __shared__ MatLds<D> L;
  const int bh = blockIdx.y;
  const int64_t b = bh / H, h = bh % H;
  const int lane = threadIdx.x & 63, wave = wave_index();
  const int g = lane >> 4, n = lane & 15;
  const int64_t row_bytes = sn * 4, orow_bytes = osn * OES;
  const char* qh = (const char*)q + (b * sb + h * sh) * 4;
  const char* gh = (const char*)dout + (b * sb + h * sh) * 4;
  char* oh = (char*)dq + (b * osb + h * osh) * OES;
  const double* M = S64 + (int64_t)bh * D * D;
  const double* v = z64 + (int64_t)bh * D;
  const Sweep<D, 1> sw(N, G, wave);

  uint32_t rq[Q4], rg[Q4];
  auto load = [&](int k) {
    load_rows<D>(qh, row_bytes, sw.token(k), N, g, n, rq);
    load_rows<D>(gh, row_bytes, sw.token(k), N, g, n, rg);
  };
  float ph[Q4];  // phi(q)
  Bf16x3 bg[NS];
  auto convert = [&](bool all_bad) {
    SplitRange<> rp, rx;
#pragma unroll
    for (int c = 0; c < Q4; ++c) ph[c] = phi<DT_FP32>(__uint_as_float(rq[c]));
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      float x[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) x[j] = __uint_as_float(rg[8 * s + j]);
#pragma unroll
      for (int j = 0; j < 8; j += 2) {
        rx.see(0, x[j], x[j + 1]);
        rp.see(0, ph[8 * s + j], ph[8 * s + j + 1]);
      }
      bg[s] = split_run(x);
    }
    return !all_bad && !__any(rp.bad() || rx.bad());
  };
  auto finish = [&](const f32x4 (&X)[NT], double den, int64_t t) {
    double gn = 0.0;
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) gn += (double)ph[4 * i + r] * (double)X[i][r];
    gn = sum_groups(gn);
    const double rden = 1.0 / den, go = gn * rden;
    if (t >= N) return;
#pragma unroll
    for (int i = 0; i < NT; ++i) {
      float out[4];
#pragma unroll
      for (int r = 0; r < 4; ++r)
        out[r] = (float)(fma(-go, L.vd[16 * i + 4 * g + r], (double)X[i][r]) * rden) * dphi_of_phi(ph[4 * i + r]);
      store4<OT>(oh + t * orow_bytes + (16 * i + 4 * g) * OES, out);
    }
    if (g == 0) stash[(int64_t)bh * N + t] = float2{(float)rden, (float)(-go)};
  };
  if (sw.nk > 0) load(0);
  stage_matrix<D, false, true, true>(L, M, v);
  __syncthreads();
  const bool all_bad = __builtin_amdgcn_readfirstlane(L.out_of_range);
  const int rbase = row_base<D>(g, n);

  bool left_out = false;
  for (int k = 0; k < sw.nk; ++k) {
    const bool good = convert(all_bad);
    load(k + 1);
    __builtin_amdgcn_sched_barrier(0);
    if (!good) {
      left_out = true;
      continue;
    }
    f32x4 big = f32x4{0.f, 0.f, 0.f, 0.f}, small = big;
#pragma unroll
    for (int s = 0; s < NS; ++s) split_products(vector_operand<D>(L, g, s), split_run(ph + 8 * s), big, small);
    const double den = (double)big[0] + (double)small[0];
    f32x4 X[NT];
#pragma unroll
    for (int i = 0; i < NT; ++i) {
      big = small = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int s = 0; s < NS; ++s) split_products(row_operand<D>(L, rbase, i, s), bg[s], big, small);
      X[i] = big + small;
      __builtin_amdgcn_sched_barrier(0);  // bounded registers
    }
    finish(X, den, sw.token(k) + n);
  }
  if (!left_out) return;
  for (int k = 0; k < sw.nk; ++k) {
    load(k);
    if (convert(all_bad)) continue;
    f32x4 den = f32x4{0.f, 0.f, 0.f, 0.f}, X[NT];
#pragma unroll
    for (int c = 0; c < Q4; ++c) den = mfma_f32((float)v[run_feature(g, c)], ph[c], den);
#pragma unroll
    for (int i = 0; i < NT; ++i) {
      X[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int c = 0; c < Q4; ++c)
        X[i] = mfma_f32((float)M[(16 * i + n) * D + run_feature(g, c)], __uint_as_float(rg[c]), X[i]);
    }
    finish(X, (double)den[0], sw.token(k) + n);
  }
}

// ---------------------------------------------------------------------------
// Key backward: dV = dS^T phi(k) (A^T's operands), dK = (dS v + dz) phi'(k)
// (A's), dz added in FP64.
// ---------------------------------------------------------------------------
template <int OT, int D>
__global__ __launch_bounds__(Rows32<D>::NTH) __attribute__((amdgpu_waves_per_eu(2))) void key_split_kernel(
    const void* __restrict__ k, const void* __restrict__ v, int64_t sb, int64_t sh, int64_t sn,
    void* __restrict__ dk, void* __restrict__ dv, int64_t osb, int64_t osh, int64_t osn, int H,
    int64_t N, int G, const double* __restrict__ dS64, const double* __restrict__ dz64) {
  using C = Rows32<D>;
  constexpr int Q4 = C::Q4, NT = C::NT, NS = C::NS;
  constexpr int OES = OT == DT_BF16 ? 2 : 4;
  __shared__ MatLds<D> L;
  const int bh = blockIdx.y;
  const int64_t b = bh / H, h = bh % H;
  const int lane = threadIdx.x & 63, wave = wave_index();
  const int g = lane >> 4, n = lane & 15;
  const int64_t row_bytes = sn * 4, orow_bytes = osn * OES;
  const char* kh = (const char*)k + (b * sb + h * sh) * 4;
  const char* vh = (const char*)v + (b * sb + h * sh) * 4;
  char* okh = (char*)dk + (b * osb + h * osh) * OES;
  char* ovh = (char*)dv + (b * osb + h * osh) * OES;
  const double* M = dS64 + (int64_t)bh * D * D;
  const Sweep<D, 1> sw(N, G, wave);

  uint32_t rk[Q4], rv[Q4];
  auto load = [&](int kk) {
    load_rows<D>(kh, row_bytes, sw.token(kk), N, g, n, rk);
    load_rows<D>(vh, row_bytes, sw.token(kk), N, g, n, rv);
  };
  float ph[Q4];  // phi(k)
  Bf16x3 bk[NS], bv[NS];
  auto convert = [&](bool all_bad) {
    SplitRange<> rp, rx;
#pragma unroll
    for (int c = 0; c < Q4; ++c) ph[c] = phi<DT_FP32>(__uint_as_float(rk[c]));
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      float x[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) x[j] = __uint_as_float(rv[8 * s + j]);
#pragma unroll
      for (int j = 0; j < 8; j += 2) {
        rx.see(0, x[j], x[j + 1]);
        rp.see(0, ph[8 * s + j], ph[8 * s + j + 1]);
      }
      bv[s] = split_run(x);
      bk[s] = split_run(ph + 8 * s);
    }
    return !all_bad && !__any(rp.bad() || rx.bad());
  };
  auto finish = [&](const f32x4& tv, const f32x4& tk, int i, const float* p, int64_t t) {
    if (t >= N) return;
    const int64_t at = t * orow_bytes + (16 * i + 4 * g) * OES;
    const float ov[4] = {tv[0], tv[1], tv[2], tv[3]};
    float ok[4];
#pragma unroll
    for (int r = 0; r < 4; ++r)
      ok[r] = (float)((double)tk[r] + L.vd[16 * i + 4 * g + r]) * dphi_of_phi(p[r]);
    store4<OT>(ovh + at, ov);
    store4<OT>(okh + at, ok);
  };
  if (sw.nk > 0) load(0);
  stage_matrix<D, true, true, false>(L, M, dz64 + (int64_t)bh * D);
  __syncthreads();
  const bool all_bad = __builtin_amdgcn_readfirstlane(L.out_of_range);
  const int cbase = column_base<D>(g, n), rbase = row_base<D>(g, n);

  bool left_out = false;
  for (int kk = 0; kk < sw.nk; ++kk) {
    const bool good = convert(all_bad);
    load(kk + 1);
    __builtin_amdgcn_sched_barrier(0);
    if (!good) {
      left_out = true;
      continue;
    }
#pragma unroll
    for (int i = 0; i < NT; ++i) {
      f32x4 bigv = f32x4{0.f, 0.f, 0.f, 0.f}, smallv = bigv, bigk = bigv, smallk = bigv;
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        split_products(column_operand<D>(L, cbase, i, s), bk[s], bigv, smallv);
        split_products(row_operand<D>(L, rbase, i, s), bv[s], bigk, smallk);
      }
      finish(bigv + smallv, bigk + smallk, i, ph + 4 * i, sw.token(kk) + n);
      __builtin_amdgcn_sched_barrier(0);  // bounded registers
    }
  }
  if (!left_out) return;
  for (int kk = 0; kk < sw.nk; ++kk) {
    load(kk);
    if (convert(all_bad)) continue;
#pragma unroll
    for (int i = 0; i < NT; ++i) {
      f32x4 tv = f32x4{0.f, 0.f, 0.f, 0.f}, tk = tv;
#pragma unroll
      for (int c = 0; c < Q4; ++c) {
        const int f = run_feature(g, c);
        tv = mfma_f32((float)M[f * D + 16 * i + n], ph[c], tv);
        tk = mfma_f32((float)M[(16 * i + n) * D + f], __uint_as_float(rv[c]), tk);
      }
      finish(tv, tk, i, ph + 4 * i, sw.token(kk) + n);
    }
  }
}

// ---------------------------------------------------------------------------
// Host-side launchers
// ---------------------------------------------------------------------------
namespace {

// Workgroups per head of a sweep in blocks of `blk` tokens: about four
// rounds of the grid's resident workgroups, so that the last one weighs
// little, and while they fill the chip at least four blocks each (each
// stages the matrix first).
template <int D>
unsigned groups(int64_t N, int64_t BH, int64_t blk) {
  const int64_t resident = D == 128 ? 256 : 1024;
  const auto div = [](int64_t a, int64_t b) { return (a + b - 1) / b; };
  int64_t G = std::min(div(N, blk), div(4 * resident, BH));
  G = std::min(G, std::max(div(N, 4 * blk), div(resident, BH)));
  return (unsigned)std::max<int64_t>(1, G);
}

template <int D, int OT, bool MIX>
void apply_d(const FwdArgs& a) {
  constexpr int TT = MIX && D == 128 ? 1 : 2;
  const int64_t BH = a.B * a.H;
  const unsigned G = groups<D>(a.N, BH, Sweep<D, TT>::BLK);
  apply_split_kernel<OT, D, MIX><<<dim3(G, (unsigned)BH), Rows32<D>::NTH, 0, a.stream>>>(
      a.q, a.sb, a.sh, a.sn, a.o, a.osb, a.osh, a.osn, (int)a.H, a.N, (int)G, a.S64, a.z64, a.other,
      a.sigma, a.sigma_data);
}

template <int D, int OT>
hipError_t backward_d(const BwdArgs& a) {
  const int64_t BH = a.B * a.H;
  const unsigned G = groups<D>(a.N, BH, Sweep<D, 1>::BLK);
  const dim3 grid(G, (unsigned)BH);
  hipError_t e;
  {
    ProfScope prof("bwd_query", a.stream);
    query_split_kernel<OT, D><<<grid, Rows32<D>::NTH, 0, a.stream>>>(
        a.q, a.dout, a.sb, a.sh, a.sn, a.dq, a.osb, a.osh, a.osn, (int)a.H, a.N, (int)G, a.S64, a.z64,
        a.stash);
  }
  if ((e = hipGetLastError()) != hipSuccess) return e;
  e = launch_summary_bwd(DT_FP32, D, a.q, a.dout, a.sb, a.sh, a.sn, a.B, a.H, a.N, a.P, a.Tw,
                     a.stash, a.part, a.stream);
  if (e != hipSuccess) return e;
  e = launch_combine(a.part, a.P, a.dS64, a.dz64, nullptr, DT_FP32, BH, D, 0, a.stream);
  if (e != hipSuccess) return e;
  ProfScope prof("bwd_key", a.stream);
  key_split_kernel<OT, D><<<grid, Rows32<D>::NTH, 0, a.stream>>>(
      a.k, a.v, a.sb, a.sh, a.sn, a.dk, a.dv, a.osb, a.osh, a.osn, (int)a.H, a.N, (int)G, a.dS64,
      a.dz64);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_apply_fp32(const FwdArgs& a) {
  ProfScope prof(a.other ? "apply_gated" : "apply", a.stream);
#define LA_APPLY(D)                                                                              \
  if (a.out_dt == DT_BF16) a.other ? apply_d<D, DT_BF16, true>(a) : apply_d<D, DT_BF16, false>(a); \
  else a.other ? apply_d<D, DT_FP32, true>(a) : apply_d<D, DT_FP32, false>(a)
  if (a.D == 64) { LA_APPLY(64); } else { LA_APPLY(128); }
#undef LA_APPLY
  return hipGetLastError();
}

hipError_t launch_backward_fp32(const BwdArgs& a) {
  if (a.D == 64) return a.out_dt == DT_BF16 ? backward_d<64, DT_BF16>(a) : backward_d<64, DT_FP32>(a);
  return a.out_dt == DT_BF16 ? backward_d<128, DT_BF16>(a) : backward_d<128, DT_FP32>(a);
}

}  // namespace la
