// la_kernels.h -- launch arguments, operand-image layout and launcher
// declarations of the gfx950 kernels (internal to liblinattn).
#pragma once
#include "../../include/la.h"
#include "la_device.h"

namespace la {

// Lane runs of the row kernels (apply, query and key backward).  Lane
// (g, n) holds Q4 = d/4 features of token n: chunk w (CH features, 16 bytes
// of the input type) of lane group g is features [4*CH*w + CH*g, +CH), so
// one load or store instruction of the wave covers 4*CH contiguous features
// of each of its 16 tokens.  Run position c = CH*w + j <-> feature
// 4*CH*w + CH*g + j.
template <int D, int DT>
struct Run {
  static constexpr int ES = DT == DT_BF16 ? 2 : 4;
  static constexpr int Q4 = D / 4;
  static constexpr int CH = 16 / ES < Q4 ? 16 / ES : Q4;  // features per chunk
  static constexpr int NCH = Q4 / CH;                      // chunks per run
  static constexpr int CB = CH * ES;                       // bytes per chunk
  static __host__ __device__ constexpr int feature(int g, int c) {
    return (c / CH) * 4 * CH + g * CH + c % CH;
  }
  static __host__ __device__ constexpr int group(int f) { return (f % (4 * CH)) / CH; }
  static __host__ __device__ constexpr int pos(int f) { return (f / (4 * CH)) * CH + f % CH; }
};

// Load a lane's run (p = row start + CB * g) into words, chunk by chunk.
template <int D, int DT>
__device__ __forceinline__ void load_run(const char* p, uint32_t* w) {
  using R = Run<D, DT>;
  constexpr int CW = R::CB / 4;
#pragma unroll
  for (int c = 0; c < R::NCH; ++c) load_words<R::CB>(p + c * 4 * R::CB, w + c * CW);
}

// Store a lane's run of output values x[0..Q4) as type OT (p = row start +
// CH * sizeof(OT) * g), chunk by chunk; bf16 rounds to nearest even.
template <int D, int DT, int OT>
__device__ __forceinline__ void store_run(char* p, const float* x) {
  using R = Run<D, DT>;
  constexpr int OES = OT == DT_BF16 ? 2 : 4;
  constexpr int OCB = R::CH * OES;  // output bytes per chunk
  constexpr int OW = OCB / 4;
#pragma unroll
  for (int c = 0; c < R::NCH; ++c) {
    uint32_t ow[OW];
#pragma unroll
    for (int j = 0; j < R::CH; j += 2) {
      const float a = x[c * R::CH + j], b = x[c * R::CH + j + 1];
      if constexpr (OT == DT_BF16) {
        ow[j >> 1] = pack_bf16(a, b);
      } else {
        ow[j] = __float_as_uint(a);
        ow[j + 1] = __float_as_uint(b);
      }
    }
    store_words<OCB>(p + c * 4 * OCB, ow);
  }
}

// Load a lane's run of stored output values (type OT, the layout store_run
// writes; p = row start + CH * sizeof(OT) * g) as words; element c of the
// run is word_elem<OT>(w, c).
template <int D, int DT, int OT>
__device__ __forceinline__ void load_out_run(const char* p, uint32_t* w) {
  using R = Run<D, DT>;
  constexpr int OES = OT == DT_BF16 ? 2 : 4;
  constexpr int OCB = R::CH * OES;
  constexpr int OW = OCB / 4;
#pragma unroll
  for (int c = 0; c < R::NCH; ++c) load_words<OCB>(p + c * 4 * OCB, w + c * OW);
}

// Matrix-core operand images of a d x d matrix M (S or dS), per head:
//   T image: A[row = value feature e][k = key/query feature c] = M[c][e],
//            followed by a z tile: A[row = any of 16][k = c] = v[c] (the
//            normaliser z, or dz), whose product with phi(q) gives the
//            normaliser of every token in every output row
//   N image: A[row = key/query feature c][k = value feature e] = M[c][e]
// A 16-row output tile i maps row m = 4g + r to the feature at run
// position 4i + r of lane group g (Run above), so a lane's four result rows
// over all tiles are its run of output features.  The contraction index k
// maps to lane group Run::group(k) and run position Run::pos(k), matching
// how the B operand (one token per lane, a feature run per lane group) is
// loaded.  bf16 images store a hi part bf16(M) and a lo part bf16(M - hi);
// fp32 images store float(M).
template <int D>
struct ImageCfg {
  static constexpr int Q4 = D / 4;
  static constexpr int NT = D / 16;                  // output tiles
  static constexpr int NS = D >= 32 ? D / 32 : 1;    // bf16 k-steps of 32
  static constexpr int TILE_BF16 = NS * 2 * 64 * 16;  // one 16-row tile, hi + lo
  static constexpr int TILE_F32 = (Q4 / 4) * 64 * 16;
  static constexpr int tile_bytes(int dt) { return dt == DT_BF16 ? TILE_BF16 : TILE_F32; }
  // the NT matrix tiles of one image
  static constexpr int mat_bytes(int dt) { return NT * tile_bytes(dt); }
  // the T image: matrix tiles + z tile (the N image starts right after it)
  static constexpr int img_bytes(int dt) { return (NT + 1) * tile_bytes(dt); }
  static constexpr int head_bytes(int dt) { return img_bytes(dt) + mat_bytes(dt); }
};

// Which operands of a matrix a combine writes.
enum {
  IMG_T = 1,   // T image
  IMG_Z = 2,   // its z tile
  IMG_N = 4,   // N image
  IMG_LO = 8   // the bf16 lo parts of these
};

// Store x[0..8) = the row of 16-row tile i, row m, at contraction indices
// k0 .. k0 + 7 (k0 a multiple of 8), as bf16 hi (and, with `lo`, lo) parts
// or fp32: whole 16-byte words, one per chunk of the lane runs.  PARTS: bf16
// parts that the image has room for.  A hi part alone is rounded once (beside
// a lo part, which takes up what it leaves, the way is the same and rounding
// through fp32 cheaper: 36 us for a forward of 2 heads x 1,000 at d = 128, 40).
template <int D, int DT, int PARTS = 2>
__device__ __forceinline__ void put_image8(char* base, int i, int m, int k0, const double* x, bool lo) {
  using R = Run<D, DT>;
  using IC = ImageCfg<D>;
  u32x4* img = (u32x4*)base;
#pragma unroll
  for (int c0 = 0; c0 < 8; c0 += R::CH) {
    const int lane = 16 * R::group(k0 + c0) + m, pos = R::pos(k0 + c0);
    if constexpr (DT == DT_BF16) {
      u32x4 h = u32x4{0, 0, 0, 0}, l = u32x4{0, 0, 0, 0};  // d = 16: slots 4..7 are padding
      if (PARTS == 1 || !lo) {
        uint32_t w[R::CH / 2];
        pack_bf16_once<R::CH>(x + c0, w);
#pragma unroll
        for (int j = 0; j < R::CH / 2; ++j) h[j] = w[j];
      } else {
#pragma unroll
        for (int j = 0; j < R::CH; j += 2) {
          const double a = x[c0 + j], b = x[c0 + j + 1];
          h[j >> 1] = pack_bf16((float)a, (float)b);
          l[j >> 1] = pack_bf16((float)(a - (double)bf16lo(h[j >> 1])), (float)(b - (double)bf16hi(h[j >> 1])));
        }
      }
      const int word = ((i * IC::NS + (pos >> 3)) * PARTS) * 64 + lane;
      img[word] = h;
      if (PARTS > 1 && lo) img[word + 64] = l;
    } else {
      const int word = (i * (IC::Q4 / 4) + (pos >> 2)) * 64 + lane;
      img[word] = u32x4{__float_as_uint((float)x[c0]), __float_as_uint((float)x[c0 + 1]),
                        __float_as_uint((float)x[c0 + 2]), __float_as_uint((float)x[c0 + 3])};
    }
  }
}

// (16-row tile, row of it) of matrix row `row`.
template <int D, int DT>
__device__ __forceinline__ void image_row(int row, int& i, int& m) {
  using R = Run<D, DT>;
  const int pos = R::pos(row);
  i = pos >> 2;
  m = 4 * R::group(row) + (pos & 3);
}

// Workgroup g of G of head bh, in a backward row kernel's grid of
// row_grid(G, BH) workgroups.  Normally a head's workgroups are neighbours.  Where heads
// share cache lines (a token's slice of a head is narrower than the 128
// bytes of one, and the heads are interleaved in a token row), the heads of
// one token range are, and each XCD (workgroups go to the eight in turn)
// takes a contiguous share of the ranges, so that a line is read and written
// through one L2 (d = 32, 8 heads of 30,001 tokens: the query backward 65 ->
// 58 us, key 60 -> 58; d = 16: query 49 -> 35, key 49 -> 35; the apply, with
// one tensor in and one out, is slower that way, 35 -> 39 us at d = 32).
struct HeadPart {
  int g, bh;
  bool out;  // beyond the work
};
__device__ __forceinline__ HeadPart head_part(int G, int BH, bool shared_lines) {
  const uint32_t id = blockIdx.x;
  if (!shared_lines) return HeadPart{(int)(id % (uint32_t)G), (int)(id / (uint32_t)G), false};
  const uint32_t item = (id & 7) * (gridDim.x >> 3) + (id >> 3);
  return HeadPart{(int)(item / (uint32_t)BH), (int)(item % (uint32_t)BH),
                  item >= (uint32_t)G * (uint32_t)BH};
}
inline bool lines_shared(int64_t head_stride_bytes, int64_t H) { return H > 1 && head_stride_bytes < 128; }
inline dim3 row_grid(int64_t G, int64_t BH, bool shared) {
  return dim3((unsigned)(shared ? (G * BH + 7) / 8 * 8 : G * BH));
}

// A head's d x d matrix and d vector where a workgroup makes its operands
// itself: in FP64, or (part) as P <= 4 partial sums [d][d], [d] still to be
// added, in the combine's order (more, at d <= 32: sum_partials first).
template <int D>
struct MatrixSrc {
  const double* M;
  const double* v;
  const float* part;
  int P;
  // W neighbouring elements from i (a multiple of W) of the matrix or, vec,
  // of the vector.  PN: 0 for FP64, else the loads an element takes: 1, 2 or
  // 4 >= P (no branch divides them; those past P read the last partial and
  // count 0).
  template <int PN, int W>
  __device__ __forceinline__ void get(int i, bool vec, double* x) const {
    if constexpr (PN == 0) {
      typedef double dw __attribute__((ext_vector_type(W), aligned(8)));
      const dw w = *(const dw*)((vec ? v : M) + i);
#pragma unroll
      for (int c = 0; c < W; ++c) x[c] = w[c];
    } else {
      typedef float fw __attribute__((ext_vector_type(W)));
      const int e = (vec ? D * D : 0) + i;
      fw w[PN];
#pragma unroll
      for (int p = 0; p < PN; ++p) {
        w[p] = *(const fw*)(part + (p < P ? p : P - 1) * (D * D + D) + e);
        if (p >= P) w[p] = 0.f;
      }
#pragma unroll
      for (int c = 0; c < W; ++c) {
        if constexpr (PN == 1) x[c] = (double)w[0][c];
        else if constexpr (PN == 2) x[c] = (double)w[0][c] + (double)w[1][c];
        else x[c] = ((double)w[0][c] + (double)w[1][c]) + ((double)w[2][c] + (double)w[3][c]);
      }
    }
  }
};

// A kernel's operands, made in LDS by NTH threads: the T or N image's matrix
// tiles (bf16, PARTS = 2: hi and lo parts, 1: hi parts), the z tile.  Small
// grids wait for these loads: 8 or 16 bytes wide.
template <int DT, int D, int PARTS, bool TRANSPOSED, int PN, int NTH>
__device__ __forceinline__ void make_image(u32x4* dst, const MatrixSrc<D>& s) {
  if constexpr (TRANSPOSED) {
    constexpr int W = 2;  // eight rows' runs of two columns
#pragma unroll 1
    for (int u = threadIdx.x; u < D * D / (8 * W); u += NTH) {
      const int c0 = W * (u % (D / W)), k0 = 8 * (u / (D / W));
      double x[8][W];
#pragma unroll
      for (int j = 0; j < 8; ++j) s.template get<PN, W>((k0 + j) * D + c0, false, x[j]);
#pragma unroll
      for (int c = 0; c < W; ++c) {
        double y[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) y[j] = x[j][c];
        int i, m;
        image_row<D, DT>(c0 + c, i, m);
        put_image8<D, DT, PARTS>((char*)dst, i, m, k0, y, true);
      }
    }
  } else {
    constexpr int W = PN == 0 ? 2 : 4;
#pragma unroll 1
    for (int u = threadIdx.x; u < D * D / 8; u += NTH) {
      const int row = u / (D / 8), k0 = 8 * (u % (D / 8));
      double x[8];
#pragma unroll
      for (int j = 0; j < 8; j += W) s.template get<PN, W>(row * D + k0 + j, false, x + j);
      int i, m;
      image_row<D, DT>(row, i, m);
      put_image8<D, DT, PARTS>((char*)dst, i, m, k0, x, true);
    }
  }
}
template <int DT, int D, int PN>
__device__ __forceinline__ void make_z_tile(u32x4* dst, const MatrixSrc<D>& s) {
  if (threadIdx.x < 2 * D) {
    const int k0 = 8 * (threadIdx.x >> 4);
    double x[8];
#pragma unroll
    for (int j = 0; j < 8; j += 2) s.template get<PN, 2>(k0 + j, true, x + j);
    put_image8<D, DT>((char*)dst, 0, threadIdx.x & 15, k0, x, true);
  }
}
// f(PN) for the loads that P partials take
template <class F>
__device__ __forceinline__ void by_partials(int P, F&& f) {
  if (P == 1) f(std::integral_constant<int, 1>{});
  else if (P == 2) f(std::integral_constant<int, 2>{});
  else f(std::integral_constant<int, 4>{});
}

// The sum of 5 to 16 partials (d <= 32), in the combine's order: quarters of
// them in order, then (q0 + q1) + (q2 + q3).  NTH threads put the matrix and
// the vector behind it into `sum`, two elements each with all sixteen loads
// in flight (no branch divides them); ends in a barrier.
template <int D, int NTH>
__device__ __forceinline__ void sum_partials(double* sum, const float* part, int P) {
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  constexpr int E = D * D + D;
  const int pq = (P + 3) / 4;
  for (int u = 2 * threadIdx.x; u < E; u += 2 * NTH) {
    f32x2 x[4][4];
#pragma unroll
    for (int w = 0; w < 4; ++w)
#pragma unroll
      for (int k = 0; k < 4; ++k) x[w][k] = *(const f32x2*)(part + min(w * pq + k, P - 1) * E + u);
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      double q[4];
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        q[w] = 0.0;
#pragma unroll
        for (int k = 0; k < 4; ++k) q[w] += k < pq && w * pq + k < P ? (double)x[w][k][r] : 0.0;
      }
      sum[u + r] = (q[0] + q[1]) + (q[2] + q[3]);
    }
  }
  __syncthreads();
}

// Whether the G workgroups of each head add up its P partials themselves
// instead of a combine before them.  On a full chip the partials cost their
// bytes G times over.  Apply and key pass against the same with a combine
// each: 2,048 heads x 256 tokens, d = 128 (P = 1, G = 1 and 2) 161 + 179 us
// and 126 + 198 + 399; 512 heads x 512, d = 64 (P = 2, G = 4) 40 + 43 and 30 +
// 41 + 31; but 1,024 heads x 512, d = 32 (P = 4), the key pass with G = 4 42
// and 32 + 8, and 512 heads x 1,024, d = 64 (P = 4, G = 4 and 8) 64 + 97 and
// 38 + 70 + 42.  A small grid waits some 4 us for 100 KB and 6 us for a
// combine: 4 heads x 1,024, d = 128 (P = 2) 23 + 14 us and 16 + 16 + 13, 4 x
// 2,048 (P = 4) 28 + 20 and 17 + 15 + 13; at d <= 32 up to sixteen partials (2 x
// 8 heads x 4,000, d = 32: 46 us for the pass, 59; with 64 partials of two
// heads x 30,001, d = 16, 58 and 54).
inline bool fold_partials(int P, int G, int64_t heads, int D) {
  if (P > 4) return D <= 32 && P <= 16 && heads * G <= 512;
  return P * G <= 8 || (P * (D * D + D) * 4 <= 144 * 1024 && heads * G <= 512);
}

struct FwdArgs {
  int64_t B, H, N;
  int D, in_dt, out_dt;
  int64_t sb, sh, sn, osb, osh, osn;
  const void *q, *k, *v;
  void* o;
  int P, Tw;           // partials per head, tokens per partial
  bool team;           // bf16 summary: four waves share a partial
  int Ga;              // apply workgroups per head (they take its token blocks in turn)
  float* part;         // [BH][P][D*D + D]: S rows, then z
  double* S64;         // [BH][D][D]
  double* z64;         // [BH][D]
  bool want_summary;   // S64, z64 are results
  void* img;           // [BH][2 images] (forward, but not fp32_rows)
  // noise-gated mix (null `other`: plain output): o = g_b A + (1 - g_b) other,
  // g_b = sigma_data / (sigma_data + sigma[b])
  const void* other;   // output dtype and strides
  const double* sigma; // [B]
  double sigma_data;
  hipStream_t stream;
};

struct BwdArgs {
  int64_t B, H, N;
  int D, in_dt, out_dt;
  int64_t sb, sh, sn, osb, osh, osn;
  const void *q, *k, *v, *dout;
  void *dq, *dk, *dv;
  const double *S64, *z64;
  int P, Tw, Ta;       // Ta: tokens per workgroup of the two-pass query kernel
  int Gk;              // key-backward workgroups per head (they take its token blocks in turn)
  float* part;         // partials of dS, dz
  float2* stash;       // [BH][N] per query token: (1/den, -(dO . O))
  double* dS64;
  double* dz64;
  void* dimg;          // images of dS (not fp32_rows)
  hipStream_t stream;
};

enum { MODE_FWD = 0, MODE_BWD = 1 };

// Keeps a failed hipError_t for la_last_hip_error(); returns LA_ERR_HIP.
int32_t record_hip_error(int32_t e);

hipError_t launch_forward(const FwdArgs& a);
// Apply only, of a given S and z.
hipError_t launch_apply(const FwdArgs& a);
// The dS/dz sums of the two-pass backward (fp32 and d = 16; g = dO, stash =
// per-token (1/den, -(dO . O))).
hipError_t launch_summary_bwd(int dt, int D, const void* q, const void* g, int64_t sb, int64_t sh,
                              int64_t sn, int64_t B, int64_t H, int64_t N, int P, int Tw,
                              const float2* stash, float* part, hipStream_t stream);
// FP64 sum of the P partials [D][D], [D] of each head, and the operands
// `what` (IMG_*) of the result.
hipError_t launch_combine(const float* part, int P, double* M64, double* v64, void* img,
                          int img_dt, int64_t BH, int D, int what, hipStream_t stream);
hipError_t launch_backward(const BwdArgs& a);
// fp32 inputs at d = 64 and 128, where the row kernels take S and dS in FP64
// and need no operand images: the apply, and the whole backward.
constexpr bool fp32_rows(int dt, int D) { return dt == DT_FP32 && D >= 64; }
hipError_t launch_apply_fp32(const FwdArgs& a);
hipError_t launch_backward_fp32(const BwdArgs& a);

// The least workspace, in bytes, with which a pass (as la_workspace_size's) runs.
size_t least_workspace(const la_attn_desc* d, int pass);

}  // namespace la
