// la_api.cpp -- the C ABI of liblinattn (include/la.h): argument checks,
// tiling choices, workspace layout and kernel launches.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>

#include "../../include/la.h"
#include "la_kernels.h"

namespace {

thread_local int32_t g_last_hip_error = 0;

constexpr size_t kAlign = 256;
size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }
int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

la_status hip_fail(hipError_t e) {
  g_last_hip_error = (int32_t)e;
  return LA_ERR_HIP;
}

int elem_size(int32_t dt) { return dt == LA_BF16 ? 2 : 4; }

bool aligned16(const void* p) { return ((uintptr_t)p & 15u) == 0; }

la_status check_desc(const la_attn_desc* d) {
  if (!d) return LA_ERR_INVALID_ARG;
  if (d->B < 1 || d->H < 1 || d->N < 1 || d->d < 1) return LA_ERR_INVALID_ARG;
  if (d->in_dtype != LA_BF16 && d->in_dtype != LA_FP32) return LA_ERR_INVALID_ARG;
  if (d->out_dtype != LA_BF16 && d->out_dtype != LA_FP32) return LA_ERR_INVALID_ARG;
  if (d->feature_map != LA_PHI_ELU1) return LA_ERR_UNSUPPORTED;
  if (d->flags != 0) return LA_ERR_INVALID_ARG;
  if (d->d != 16 && d->d != 32 && d->d != 64 && d->d != 128) return LA_ERR_UNSUPPORTED;
  // the grid's y dimension carries (b, h); token indices are 64-bit, while
  // partials (N / 4096 at most) and workgroups along x (N / 2048 at most)
  // are counted in 32 bits
  if (d->B * d->H > 65535 || d->N > (int64_t(1) << 36)) return LA_ERR_UNSUPPORTED;
  const int64_t s[2][3] = {{d->in_sb, d->in_sh, d->in_sn}, {d->out_sb, d->out_sh, d->out_sn}};
  const int es[2] = {elem_size(d->in_dtype), elem_size(d->out_dtype)};
  for (int t = 0; t < 2; ++t) {
    for (int i = 0; i < 3; ++i) {
      if (s[t][i] < 0) return LA_ERR_INVALID_ARG;
      if ((s[t][i] * es[t]) % 16 != 0) return LA_ERR_INVALID_ARG;
    }
    if (s[t][2] < d->d) return LA_ERR_INVALID_ARG;
    // kernels address 32 consecutive token rows with 32-bit lane offsets
    if (s[t][2] * es[t] > (int64_t(1) << 24)) return LA_ERR_UNSUPPORTED;
  }
  return LA_OK;
}

// Tiling.  Depends only on (N, d, dtype) so that the same (b, h) problem
// gives bitwise the same result whatever batch it is part of.
struct Tiling {
  int P;   // partial sums per (b, h)
  int Tw;  // tokens per partial (a multiple of 64, at most max_fp32_run)
};

// The longest token range any kernel sums in FP32: each partial sum covers
// at most this many tokens, and partials are added in FP64 (the combine),
// so the FP32 part of every sum over tokens is bounded whatever N is.
// The fp32 path, which is held to a tighter tolerance, takes shorter runs.
int64_t max_fp32_run(int dt) { return dt == LA_BF16 ? 16384 : 4096; }

// At most 128 partials at d = 128 and 64 below while that keeps each FP32
// run within max_fp32_run: longer ranges per wave paid off at d = 64
// (summary of 32 heads x 262,144 tokens 0.38 -> 0.33 ms), while 8 heads at
// d = 128 need the 128 to give each SIMD a wave.  Beyond that the partial
// count grows with N (about (d^2 + d) * 4 bytes of workspace per
// max_fp32_run tokens per head: 0.8 % of the inputs' bytes at d = 128).
int64_t max_partials(int d) { return d >= 128 ? 128 : 64; }

// The fused query backward, a workgroup to a partial: at least 2048 (d =
// 128) or 512 tokens each, but up to four partials of at least 4 d (two
// heads of 1,000 tokens at d = 128: 42 us in two partials, 62 in one).
int64_t fused_partials(int64_t N, int d) {
  return std::max(std::min(max_partials(d), ceil_div(N, d >= 128 ? 2048 : 512)),
                  std::min<int64_t>(4, ceil_div(N, 4 * d)));
}

// bf16 summaries with four waves to a partial: sequences too short for 64
// partials of a single wave's 2048 (d = 128) or 512 tokens.  Longer ones
// keep the SIMDs streaming with a wave to a partial, whose four waves of a
// workgroup, four heads of a token range, read a BNHD view best (8 x 8 heads
// of 63,607 tokens at d = 64, BNHD: 200 us, 224 with teams).  A team is one
// workgroup a compute unit at d = 128, so eight heads of more than 131,072
// tokens would take a second round of them: the forward of 8 x 262,144 takes
// 417 us, 441 with teams, gated on BNHD views 545, 574 (one head of 200,001
// would take 121 instead of 181, but the bits may not follow the head count).
// At d <= 32 heads of a BNHD view share cache lines, and a single wave is the
// better form for all (d = 32, 8 heads of 30,001 tokens: 34 us, 38).
bool team_summary(int64_t N, int d, int dt) {
  return dt == LA_BF16 && d >= 64 && N <= 64 * (d >= 128 ? 2048 : 512);
}

// The summary's partials.  A partial's write and read cost 2 (d + 1) * 4
// bytes against 2 * es bytes of K and V a token and feature, so a partial of
// 32 d bf16 tokens adds 6 % and is the rule of the teams (16 d in fp32: the
// same bytes).  Short sequences take up to four (fp32: sixteen) shorter ones,
// not below 4 d (2 d) tokens, so that a few heads still fill compute units:
// one head of 4,096 fp32 tokens (d = 64) takes 14 us in sixteen partials and
// 21 in eight, while 1,024 heads of 8,192 bf16 tokens take 396 + 94 us
// (summary + combine) in four and 430 + 110 in eight.  (fp32 at d = 64: up to
// 1,024 tokens are one FP32 sum, but 32 to an accumulation; S is 1.8e-7 off
// where 512 tokens, four to an accumulation, left 4.0e-7.)  A single wave's
// partials: 2048 (512) tokens, at d <= 32 up to sixteen of at least 4 d.
int64_t summary_partials(int64_t N, int d, int dt) {
  const int64_t unit = dt == LA_BF16 ? 4 * d : 2 * d;
  if (dt == LA_FP32 || team_summary(N, d, dt))
    return std::max(std::min(max_partials(d), ceil_div(N, 8 * unit)),
                    std::min<int64_t>(dt == LA_FP32 ? 16 : 4, ceil_div(N, unit)));
  return std::max(std::min(max_partials(d), ceil_div(N, d >= 128 ? 2048 : 512)),
                  std::min<int64_t>(d <= 32 ? 16 : 1, ceil_div(N, unit)));
}

bool fused_backward(int d, int dt) { return dt == LA_BF16 && d >= 32; }

// The fewest partials a pass takes: one for 2,048 (d = 128) or 512 tokens,
// for workspaces without room for one head's finer ones.
int64_t coarse_partials(int64_t N, int d) {
  return std::min(max_partials(d), ceil_div(N, d >= 128 ? 2048 : 512));
}

Tiling choose_tiling(int64_t N, int d, int dt, bool backward, bool coarse) {
  int64_t P = coarse                                 ? coarse_partials(N, d)
              : backward && fused_backward(d, dt) ? fused_partials(N, d)
                                                  : summary_partials(N, d, dt);
  P = std::max<int64_t>(P, ceil_div(N, max_fp32_run(dt)));
  // a multiple of 64: the summary steps over 32 tokens, the fused
  // backward over 64 (four waves x 16); max_fp32_run is one too, so
  // rounding up keeps Tw <= max_fp32_run
  int64_t Tw = ceil_div(ceil_div(N, P), 64) * 64;
  P = ceil_div(N, Tw);
  Tiling t;
  t.P = (int)P;
  t.Tw = (int)Tw;
  return t;
}

// Partials the workspace has room for: those of the tiling, or as many as
// 512 (d = 128: 2048) tokens each would make, which keeps the size the
// same from 64 (128) of them up to max_fp32_run tokens each.
int64_t partial_room(int64_t N, int d, int P) {
  return std::max<int64_t>(P, coarse_partials(N, d));
}

// Apply workgroups per head: at most one per token block.  Per-token work, so
// this changes no bits and may depend on the batch size.
int apply_groups(int64_t N, int64_t BH, int d) {
  const int64_t blk = 128;  // tokens per block
  if (d >= 128) {
    // A workgroup first makes or copies 72 KB of operands, as much traffic as
    // 270 tokens, and two share a compute unit: one round of 512 workgroups
    // (4 x 16 heads of 4,096: 44 us, 81 with 2,048; 16 of 43,237: 92, 126),
    // more where each still has 8,192 tokens (8 heads of 2,097,152 as views of
    // [B, N, H, d]: 1.72 ms, 1.95 in one round).  Beyond 128 heads a round does
    // not divide evenly: the count, up to sixteen, whose rounds of (tokens each
    // + the operands' 300) are fewest (4,095 tokens: 129 heads, 3 each, 85 us,
    // 125 with 1 and 100 with 2; 256, 2, 127, 145 with 1 and 160 with 3; 300, 3,
    // 165, 197 and 175; 384, 4, 199, 215 and 199; 500, 1, 236, 243 with 2).
    if (BH <= 128)
      return (int)std::max<int64_t>(
          1, std::min(ceil_div(N, blk), std::max(512 / BH, std::min(ceil_div(4096, BH), N / 8192))));
    int64_t ga = 1, least = INT64_MAX;
    for (int64_t g = 1; g <= std::min<int64_t>(16, ceil_div(N, blk)); ++g) {
      const int64_t cost = ceil_div(BH * g, 512) * (ceil_div(ceil_div(N, blk), g) * blk + 300);
      if (cost < least) { least = cost; ga = g; }
    }
    return (int)ga;
  }
  const int64_t grid = 4096;
  int64_t ga = std::min(ceil_div(N, blk), ceil_div(grid, BH));
  // while the grid keeps 1,024 workgroups or more (four to a compute unit), at
  // least four blocks per workgroup: each stages the operands first (d = 64:
  // 4 x 16 heads of 4,096 tokens take 23 us with 16 workgroups a head and 29
  // with 32; of 16,384, 58 us with 32 and 60 with 64 or 16)
  ga = std::min(ga, std::max(ceil_div(N, 4 * blk), ceil_div(1024, BH)));
  return (int)std::max<int64_t>(1, ga);
}

// Bytes of the two matrix-core operand images of one head.
size_t head_image_bytes(int D, int dt) {
  const int idt = dt == LA_BF16 ? la::DT_BF16 : la::DT_FP32;
  switch (D) {
    case 16: return la::ImageCfg<16>::head_bytes(idt);
    case 32: return la::ImageCfg<32>::head_bytes(idt);
    case 64: return la::ImageCfg<64>::head_bytes(idt);
    default: return la::ImageCfg<128>::head_bytes(idt);
  }
}

struct Layout {
  size_t part, S64, z64, img, stash, dS64, dz64, dimg, total;
};

// Forward: [part][S64][z64][img].  Backward: [part][stash][dS64][dz64][dimg];
// the stash holds two floats per query token (1/den, -(dO . O)) between the
// query kernel and the dS reduction, the only part of any workspace that
// grows with N.  bf16 at d >= 32 fuses the two passes and needs no stash;
// fp32 at d >= 64 has no images.  The apply makes its operands in LDS; its
// workspace stays the two images that callers have always brought.
Layout layout_for(const la_attn_desc* d, int pass, bool coarse = false) {
  const int64_t BH = d->B * d->H, D = d->d;
  const Tiling t = choose_tiling(d->N, (int)D, d->in_dtype, pass == 1, coarse);
  const int64_t room = coarse ? t.P : partial_room(d->N, (int)D, t.P);
  const size_t part = align_up((size_t)BH * room * (D * D + D) * sizeof(float));
  const size_t mat = align_up((size_t)BH * D * D * sizeof(double));
  const size_t vec = align_up((size_t)BH * D * sizeof(double));
  const size_t img = pass != 2 && la::fp32_rows(d->in_dtype, (int)D)
                         ? 0
                         : align_up((size_t)BH * head_image_bytes((int)D, d->in_dtype));
  Layout L{};
  size_t off = 0;
  if (pass == 2) {
    off += img;
  } else if (pass == 0) {
    L.part = off; off += part;
    L.S64 = off; off += mat;
    L.z64 = off; off += vec;
    L.img = off; off += img;
  } else {
    L.part = off; off += part;
    L.stash = off;
    if (!fused_backward((int)D, d->in_dtype)) off += align_up((size_t)BH * d->N * 2 * sizeof(float));
    L.dS64 = off; off += mat;
    L.dz64 = off; off += vec;
    L.dimg = off; off += img;
  }
  L.total = off;
  return L;
}

}  // namespace

// The workspace that a pass has always taken: two operand images of S (and dS)
// and the coarse partials.  Short sequences are cut finer now, up to 3.3
// times this (fp32, d = 128); with less than they want, but this much, a
// problem runs in parts of its heads, and where not even one head's finer
// partials fit, with the coarse ones.
namespace la {
size_t least_workspace(const la_attn_desc* d, int pass) {
  const int64_t BH = d->B * d->H, D = d->d;
  const int64_t P = choose_tiling(d->N, (int)D, d->in_dtype, pass == 1, true).P;
  const size_t part = align_up((size_t)BH * P * (D * D + D) * sizeof(float));
  const size_t sums = align_up((size_t)BH * D * D * sizeof(double)) + align_up((size_t)BH * D * sizeof(double));
  const size_t img = align_up((size_t)BH * head_image_bytes((int)D, d->in_dtype));
  if (pass == 2) return img;
  if (pass == 0) return part + sums + img;
  const size_t stash =
      fused_backward((int)D, d->in_dtype) ? 0 : align_up((size_t)BH * d->N * 2 * sizeof(float));
  return part + stash + sums + 2 * img;
}
}  // namespace la

namespace {

// The largest number of batch elements, or of heads of one, whose workspace
// fits ws_bytes (0: not even one head's).
struct Part {
  int64_t B, H;
};
Part part_for(const la_attn_desc* d, int pass, size_t ws_bytes) {
  la_attn_desc p = *d;
  auto most = [&](int64_t& n) {  // the total is monotonic in n
    int64_t lo = 0, hi = n;
    while (lo < hi) {
      n = (lo + hi + 1) / 2;
      if (layout_for(&p, pass).total <= ws_bytes) lo = n; else hi = n - 1;
    }
    return lo;
  };
  if (const int64_t b = most(p.B)) return {b, d->H};
  p.B = 1;
  return {1, most(p.H)};
}

// Calls f(part's descriptor, its first b, its first h, coarse) for parts of the
// problem that fit ws_bytes, one after the other.  A head's result does not
// depend on the others in a call, so the bits are those of one call.  With
// less than one head's layout, one call in coarse partials, which fit the
// least workspace: its sums over tokens round differently.
template <class F>
la_status in_parts(const la_attn_desc* desc, int pass, size_t ws_bytes, F&& f) {
  if (ws_bytes < la::least_workspace(desc, pass)) return LA_ERR_OOM;
  const Part most = part_for(desc, pass, ws_bytes);
  if (!most.H) return f(desc, 0, 0, true);
  for (int64_t b = 0; b < desc->B; b += most.B)
    for (int64_t h = 0; h < desc->H; h += most.H) {
      la_attn_desc p = *desc;
      p.B = std::min(most.B, desc->B - b);
      p.H = std::min(most.H, desc->H - h);
      const la_status st = f(&p, b, h, false);
      if (st != LA_OK) return st;
    }
  return LA_OK;
}

// Byte offsets of element (b, h, 0, 0) of the tensors in in_s*, out_s*.
int64_t in_offset(const la_attn_desc* d, int64_t b, int64_t h) {
  return (b * d->in_sb + h * d->in_sh) * elem_size(d->in_dtype);
}
int64_t out_offset(const la_attn_desc* d, int64_t b, int64_t h) {
  return (b * d->out_sb + h * d->out_sh) * elem_size(d->out_dtype);
}

// Tokens per workgroup of the two-pass query backward (d = 16, fp32 d = 32):
// per-token work as the apply's, up to 2,048 once the grid has 1,024
// workgroups (2 heads of 8,699 fp32 tokens at d = 32: 10 us, 41 with ten
// workgroups; 1,024 of 1,000 bf16 tokens, d = 16, 23 us, 28 with four each).
int query_tokens(int64_t N, int64_t BH, int dt) {
  const int64_t blk = dt == LA_FP32 ? 64 : 128;  // tokens per block (4 waves x 16 x TT)
  const int64_t g = std::min(ceil_div(N, blk), std::max(ceil_div(N, 2048), ceil_div(1024, BH)));
  return (int)(ceil_div(ceil_div(N, g), blk) * blk);
}

// Key-backward workgroups per head, as apply_groups (fp32 takes one tile per
// wave step; at d >= 64 it has its own grid).  A bf16 workgroup stages 64 KB
// of operands at d = 128 and 16 at d = 64: at least 1,024 (512) tokens each
// while the grid keeps 1,024 (2,048) workgroups: 4 x 16 heads of 4,096 tokens
// at d = 128 take 68 us, 80 with 128 tokens each, 8 x 16 of 16,384 430 and
// 495 (256 tokens); at d = 64 8 x 16 of 16,384 take 215 us, 230 (256).
int key_groups(int64_t N, int64_t BH, int d, int dt) {
  const int64_t blk = dt == LA_FP32 ? 64 : 128;  // tokens per block (4 waves x 16 x TT)
  int64_t grid = 8192;
  int64_t g = std::min(ceil_div(N, blk), ceil_div(grid, BH));
  if (d >= 64) {
    const int64_t tokens = d >= 128 ? 1024 : 512, least = d >= 128 ? 1024 : 2048;
    g = std::min(g, std::max(ceil_div(N, tokens), ceil_div(least, BH)));
  }
  return (int)std::max<int64_t>(1, g);
}

// The gate's arguments (the attention's own are checked by the caller).
la_status check_gate(const void* other, const double* sigma, double sigma_data) {
  if (!other || !sigma) return LA_ERR_INVALID_ARG;
  if (!aligned16(other) || ((uintptr_t)sigma & 7u)) return LA_ERR_INVALID_ARG;
  if (!(sigma_data > 0.0) || !std::isfinite(sigma_data)) return LA_ERR_INVALID_ARG;
  return LA_OK;
}

la_status forward_impl(const la_attn_desc* desc, const void* q, const void* k, const void* v,
                       void* o, double* s_out, double* z_out, void* ws, size_t ws_bytes,
                       la_stream stream, const void* other, const double* sigma,
                       double sigma_data, bool coarse = false) {
  la_status st = check_desc(desc);
  if (st != LA_OK) return st;
  if (!q || !k || !v || !o || !ws) return LA_ERR_INVALID_ARG;
  if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(o)) return LA_ERR_INVALID_ARG;
  if (((uintptr_t)ws % kAlign) != 0) return LA_ERR_INVALID_ARG;
  if (((uintptr_t)s_out & 7u) || ((uintptr_t)z_out & 7u)) return LA_ERR_INVALID_ARG;
  const Layout L = layout_for(desc, 0, coarse);
  if (ws_bytes < L.total)
    return in_parts(desc, 0, ws_bytes, [&](const la_attn_desc* p, int64_t b, int64_t h, bool c) {
      const int64_t i = in_offset(desc, b, h), j = out_offset(desc, b, h);
      const int64_t bh = b * desc->H + h, d = desc->d;
      return forward_impl(p, (const char*)q + i, (const char*)k + i, (const char*)v + i, (char*)o + j,
                          s_out ? s_out + bh * d * d : nullptr, z_out ? z_out + bh * d : nullptr, ws,
                          ws_bytes, stream, other ? (const char*)other + j : nullptr,
                          sigma ? sigma + b : nullptr, sigma_data, c);
    });
  const Tiling t = choose_tiling(desc->N, (int)desc->d, desc->in_dtype, false, coarse);
  char* w = (char*)ws;
  la::FwdArgs a{};
  a.B = desc->B; a.H = desc->H; a.N = desc->N; a.D = (int)desc->d;
  a.in_dt = desc->in_dtype; a.out_dt = desc->out_dtype;
  a.sb = desc->in_sb; a.sh = desc->in_sh; a.sn = desc->in_sn;
  a.osb = desc->out_sb; a.osh = desc->out_sh; a.osn = desc->out_sn;
  a.q = q; a.k = k; a.v = v; a.o = o;
  a.P = t.P; a.Tw = t.Tw;
  a.team = team_summary(desc->N, (int)desc->d, desc->in_dtype);
  a.Ga = apply_groups(desc->N, desc->B * desc->H, (int)desc->d);
  a.part = (float*)(w + L.part);
  a.S64 = s_out ? s_out : (double*)(w + L.S64);
  a.z64 = z_out ? z_out : (double*)(w + L.z64);
  a.want_summary = s_out || z_out;
  a.img = w + L.img;
  a.other = other; a.sigma = sigma; a.sigma_data = sigma_data;
  a.stream = (hipStream_t)stream;
  hipError_t e = la::launch_forward(a);
  if (e != hipSuccess) return hip_fail(e);
  return LA_OK;
}

la_status apply_impl(const la_attn_desc* desc, const void* q, const double* s, const double* z,
                     void* o, void* ws, size_t ws_bytes, la_stream stream, const void* other,
                     const double* sigma, double sigma_data) {
  la_status st = check_desc(desc);
  if (st != LA_OK) return st;
  if (!q || !s || !z || !o || !ws) return LA_ERR_INVALID_ARG;
  if (!aligned16(q) || !aligned16(o)) return LA_ERR_INVALID_ARG;
  if (((uintptr_t)s & 7u) || ((uintptr_t)z & 7u)) return LA_ERR_INVALID_ARG;
  if (((uintptr_t)ws % kAlign) != 0) return LA_ERR_INVALID_ARG;
  const Layout L = layout_for(desc, 2);
  if (ws_bytes < L.total) return LA_ERR_OOM;  // (it is not used)
  la::FwdArgs a{};
  a.B = desc->B; a.H = desc->H; a.N = desc->N; a.D = (int)desc->d;
  a.in_dt = desc->in_dtype; a.out_dt = desc->out_dtype;
  a.sb = desc->in_sb; a.sh = desc->in_sh; a.sn = desc->in_sn;
  a.osb = desc->out_sb; a.osh = desc->out_sh; a.osn = desc->out_sn;
  a.q = q; a.o = o;
  a.Ga = apply_groups(desc->N, desc->B * desc->H, (int)desc->d);
  a.S64 = const_cast<double*>(s);
  a.z64 = const_cast<double*>(z);
  a.other = other; a.sigma = sigma; a.sigma_data = sigma_data;
  a.stream = (hipStream_t)stream;
  hipError_t e = la::launch_apply(a);
  if (e != hipSuccess) return hip_fail(e);
  return LA_OK;
}

la_status backward_impl(const la_attn_desc* desc, const void* q, const void* k, const void* v,
                        const double* s, const double* z, const void* dout, void* dq, void* dk,
                        void* dv, void* ws, size_t ws_bytes, la_stream stream, bool coarse = false) {
  la_status st = check_desc(desc);
  if (st != LA_OK) return st;
  if (!q || !k || !v || !s || !z || !dout || !dq || !dk || !dv || !ws) return LA_ERR_INVALID_ARG;
  for (const void* p : {q, k, v, dout, (const void*)dq, (const void*)dk, (const void*)dv})
    if (!aligned16(p)) return LA_ERR_INVALID_ARG;
  if (((uintptr_t)s & 7u) || ((uintptr_t)z & 7u)) return LA_ERR_INVALID_ARG;
  if (((uintptr_t)ws % kAlign) != 0) return LA_ERR_INVALID_ARG;
  const Layout L = layout_for(desc, 1, coarse);
  if (ws_bytes < L.total)
    return in_parts(desc, 1, ws_bytes, [&](const la_attn_desc* p, int64_t b, int64_t h, bool c) {
      const int64_t i = in_offset(desc, b, h), j = out_offset(desc, b, h);
      const int64_t bh = b * desc->H + h, d = desc->d;
      return backward_impl(p, (const char*)q + i, (const char*)k + i, (const char*)v + i, s + bh * d * d,
                           z + bh * d, (const char*)dout + i, (char*)dq + j, (char*)dk + j, (char*)dv + j,
                           ws, ws_bytes, stream, c);
    });
  const Tiling t = choose_tiling(desc->N, (int)desc->d, desc->in_dtype, true, coarse);
  char* w = (char*)ws;
  la::BwdArgs a{};
  a.B = desc->B; a.H = desc->H; a.N = desc->N; a.D = (int)desc->d;
  a.in_dt = desc->in_dtype; a.out_dt = desc->out_dtype;
  a.sb = desc->in_sb; a.sh = desc->in_sh; a.sn = desc->in_sn;
  a.osb = desc->out_sb; a.osh = desc->out_sh; a.osn = desc->out_sn;
  a.q = q; a.k = k; a.v = v; a.dout = dout;
  a.dq = dq; a.dk = dk; a.dv = dv;
  a.S64 = s; a.z64 = z;
  a.P = t.P; a.Tw = t.Tw; a.Ta = query_tokens(desc->N, desc->B * desc->H, desc->in_dtype);
  a.Gk = key_groups(desc->N, desc->B * desc->H, (int)desc->d, desc->in_dtype);
  a.part = (float*)(w + L.part);
  a.stash = (float2*)(w + L.stash);
  a.dS64 = (double*)(w + L.dS64);
  a.dz64 = (double*)(w + L.dz64);
  a.dimg = w + L.dimg;
  a.stream = (hipStream_t)stream;
  hipError_t e = la::launch_backward(a);
  if (e != hipSuccess) return hip_fail(e);
  return LA_OK;
}

}  // namespace

namespace la {
// A failed HIP call seen outside this file: kept for la_last_hip_error().
int32_t record_hip_error(int32_t e) {
  g_last_hip_error = e;
  return LA_ERR_HIP;
}
}  // namespace la

extern "C" {

const char* la_status_string(la_status s) {
  switch (s) {
    case LA_OK: return "LA_OK";
    case LA_ERR_INVALID_ARG: return "LA_ERR_INVALID_ARG";
    case LA_ERR_UNSUPPORTED: return "LA_ERR_UNSUPPORTED";
    case LA_ERR_OOM: return "LA_ERR_OOM";
    case LA_ERR_HIP: return "LA_ERR_HIP";
    case LA_ERR_NOT_FOUND: return "LA_ERR_NOT_FOUND";
    case LA_ERR_SHUTDOWN: return "LA_ERR_SHUTDOWN";
    case LA_ERR_BUSY: return "LA_ERR_BUSY";
  }
  return "LA_ERR_UNKNOWN";
}

int32_t la_last_hip_error(void) { return g_last_hip_error; }

la_status la_version(int32_t* major, int32_t* minor) {
  if (!major || !minor) return LA_ERR_INVALID_ARG;
  *major = 1;
  *minor = 0;
  return LA_OK;
}

la_status la_workspace_size(const la_attn_desc* desc, int32_t pass, size_t* bytes) {
  if (!bytes || pass < 0 || pass > 2) return LA_ERR_INVALID_ARG;
  la_status st = check_desc(desc);
  if (st != LA_OK) return st;
  *bytes = layout_for(desc, pass).total;
  return LA_OK;
}

la_status la_forward(const la_attn_desc* desc, const void* q, const void* k,
                     const void* v, void* o, double* s_out, double* z_out,
                     void* ws, size_t ws_bytes, la_stream stream) {
  return forward_impl(desc, q, k, v, o, s_out, z_out, ws, ws_bytes, stream, nullptr, nullptr, 0.0);
}

la_status la_forward_gated(const la_attn_desc* desc, const void* q, const void* k,
                           const void* v, const void* other, const double* sigma,
                           double sigma_data, void* o, double* s_out, double* z_out,
                           void* ws, size_t ws_bytes, la_stream stream) {
  const la_status st = check_gate(other, sigma, sigma_data);
  if (st != LA_OK) return st;
  return forward_impl(desc, q, k, v, o, s_out, z_out, ws, ws_bytes, stream, other, sigma,
                      sigma_data);
}

la_status la_apply(const la_attn_desc* desc, const void* q, const double* s,
                   const double* z, void* o, void* ws, size_t ws_bytes, la_stream stream) {
  return apply_impl(desc, q, s, z, o, ws, ws_bytes, stream, nullptr, nullptr, 0.0);
}

la_status la_apply_gated(const la_attn_desc* desc, const void* q, const double* s,
                         const double* z, const void* other, const double* sigma,
                         double sigma_data, void* o, void* ws, size_t ws_bytes,
                         la_stream stream) {
  const la_status st = check_gate(other, sigma, sigma_data);
  if (st != LA_OK) return st;
  return apply_impl(desc, q, s, z, o, ws, ws_bytes, stream, other, sigma, sigma_data);
}

la_status la_backward(const la_attn_desc* desc, const void* q, const void* k,
                      const void* v, const double* s, const double* z,
                      const void* dout, void* dq, void* dk, void* dv, void* ws,
                      size_t ws_bytes, la_stream stream) {
  return backward_impl(desc, q, k, v, s, z, dout, dq, dk, dv, ws, ws_bytes, stream);
}

}  // extern "C"
