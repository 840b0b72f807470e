// Sliced decoding ("Feature chunk and Sliced Decoding" section): the latent video, batch and frame axes merged, is
// decoded `slice_frames` frames at a time (1 = frame by frame) by a convolutional decoder and the images are
// merged back in frame order; the workspace is sized by the slice, not by the video. The decoder's operators are
// the kernels of the denoising stage: the fused-loader 3x3 convolution (GroupNorm + SiLU applied on the way in,
// residual added on the way out), the GroupNorm statistics kernels, the linear kernels and the spatial attention.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <new>
#include <string>

#include "../../include/lightcache.h"
#include "lc_internal.h"

using namespace lc;

namespace {

thread_local std::string g_derr = "";
constexpr size_t kAlign = 256;
inline size_t align_up(size_t v) { return (v + kAlign - 1) / kAlign * kAlign; }

struct GnP { float *g, *b; };
struct ConvP { void* w; float* b; };  // w of a bf16 decoder (not `out`): in fragment order

struct DPlan {
  size_t off_a, off_b, off_part, off_scale, off_shift, off_one, off_zero, off_qkv, off_vt, off_ao, total;
  size_t frame_a;               // bytes of one frame in buffer `a`
  size_t lane_off, lane_stride;  // [lane_off, lane_off + lane_stride): what one lane works in
  int lanes;
};

}  // namespace

struct lc_decoder {
  lc_decoder_config cfg;
  hipStream_t s;          // the stream kernels are issued on right now
  hipStream_t s_main, s_aux;  // the caller's stream; the library's own second one
  hipEvent_t ev_fork, ev_join;
  char* lane;             // where the lane's scratch offsets count from
  void* wblob;
  size_t wblob_bytes;
  bool have_weights;
  // packed weights
  float *cin_w, *cin_b;
  void* cin_wp;  // conv_in weights as rows [C][64] of the operand type (k = plane * 9 + tap, zero padded), or nullptr
  GnP res_gn[2 + LC_DEC_MAX_LEVELS]; ConvP res[2 + LC_DEC_MAX_LEVELS];  // mid.res0, mid.res1, up0.res, ...
  GnP at_gn; void *at_wqkv, *at_wo; float* at_bo;
  ConvP upc[LC_DEC_MAX_LEVELS];
  GnP out_gn; ConvP out;
  char* arena;
  size_t arena_bytes;
  std::string err;
};

namespace {

lc_status dfail(lc_decoder* d, lc_status code, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  if (d) d->err = buf; else g_derr = buf;
  return code;
}

#define LCD_HIP(d, expr)                                                                          \
  do {                                                                                            \
    hipError_t e_ = (expr);                                                                       \
    if (e_ != hipSuccess) return dfail(d, LC_ERR_HIP, "%s: %s", #expr, hipGetErrorString(e_));   \
  } while (0)

lc_status check_dcfg(lc_decoder* d, const lc_decoder_config* g) {
  if (!g) return dfail(d, LC_ERR_ARG, "config is NULL");
  if (g->dtype != LC_F32 && g->dtype != LC_BF16) return dfail(d, LC_ERR_ARG, "dtype must be LC_F32 or LC_BF16");
  if (g->N <= 0 || g->H <= 0 || g->W <= 0 || g->C_lat <= 0 || g->C_img <= 0 || g->groups <= 0 || g->heads <= 0 ||
      g->head_dim <= 0)
    return dfail(d, LC_ERR_SHAPE, "all sizes must be positive");
  if (g->levels < 0 || g->levels > LC_DEC_MAX_LEVELS) return dfail(d, LC_ERR_SHAPE, "levels must be in [0, %d]", LC_DEC_MAX_LEVELS);
  if (g->C_lat > 16 || g->C_img > 32) return dfail(d, LC_ERR_SHAPE, "C_lat must be <= 16 and C_img <= 32");
  for (int l = 0; l <= g->levels; ++l) {
    const int C = g->widths[l];
    if (C <= 0 || C % 64 || C > 1024) return dfail(d, LC_ERR_SHAPE, "every width must be a multiple of 64, at most 1024");
    if (C % g->groups || C / g->groups > 512) return dfail(d, LC_ERR_SHAPE, "every width must be divisible by groups");
  }
  if (g->heads * g->head_dim != g->widths[0]) return dfail(d, LC_ERR_SHAPE, "heads * head_dim must equal widths[0]");
  const int hd = g->head_dim;
  if (!(hd == 8 || hd == 16 || hd == 32 || hd == 40 || hd == 64))
    return dfail(d, LC_ERR_SHAPE, "head_dim must be one of 8, 16, 32, 40, 64");
  if (!(g->gn_eps > 0.f)) return dfail(d, LC_ERR_SHAPE, "gn_eps must be positive");
  if (((int64_t)g->H << g->levels) * ((int64_t)g->W << g->levels) > (int64_t)1 << 24)
    return dfail(d, LC_ERR_SHAPE, "decoded frames of more than 2^24 pixels are not supported");
  return LC_OK;
}

// Workspace of a pass over `n` frames. The maps alternate between two fp32 buffers: `a` takes the output of the first
// convolution and of every level's upsampling convolution, `b` the residual blocks', so `b` need not hold the last and
// largest map (the upsampled input of a convolution exists nowhere). Then GroupNorm partial sums and scale / shift, a
// unit scale and a zero shift (the convolution after the upsampling takes its input as it is), and the attention
// block's q,k rows, V^T and normalised rows / output at the latent resolution. The partial sums share their memory with
// the latter: what the block normalises with is folded into scale / shift before q,k,v are written, and nothing behind it
// reads them. Where the scratch of two passes takes no more than two maps of the largest stage with its input upsampled,
// partial sums and attention rows apart (what a pass with a separate upsampling held, as for widths that fall from level to
// level), there are two lanes and alternate slices run on two streams; else one, and no more memory than it needs.
DPlan make_dplan(const lc_decoder_config& g, int n) {
  DPlan p;
  const size_t es = dtype_size(g.dtype);
  const int64_t P0 = (int64_t)g.H * g.W;
  const int C0 = g.widths[0];
  int64_t elems_a = P0 * C0, elems_b = elems_a, elems_up = elems_a, splits_c = 0, rows_c = 0;
  int maxC = C0;
  for (int l = 0; l <= g.levels; ++l) {
    const int H = g.H << l, W = g.W << l;
    const int64_t e = P0 * ((int64_t)1 << 2 * l) * g.widths[l];
    elems_a = std::max(elems_a, e);
    if (l < g.levels) elems_b = std::max(elems_b, e);
    elems_up = std::max({elems_up, e, l ? P0 * ((int64_t)1 << 2 * l) * g.widths[l - 1] : (int64_t)0});
    const int splits = std::max({stat_splits(H * W), conv_stat_splits(H, W), l ? 0 : conv_in_splits(H, W)});
    splits_c = std::max(splits_c, (int64_t)splits * g.widths[l]);
    rows_c = std::max(rows_c, (int64_t)stat_splits(H * W) * g.widths[l]);
    maxC = std::max(maxC, g.widths[l]);
  }
  size_t off = 0;
  auto take = [&](size_t bytes) { size_t o = off; off += align_up(bytes); return o; };
  p.off_one = take((size_t)n * maxC * 4);
  p.off_zero = take((size_t)n * maxC * 4);
  p.lane_off = off;
  p.frame_a = (size_t)elems_a * 4;
  p.off_a = take((size_t)n * elems_a * 4);
  p.off_b = take((size_t)n * elems_b * 4);
  p.off_scale = take((size_t)n * maxC * 4);
  p.off_shift = take((size_t)n * maxC * 4);
  p.off_part = take((size_t)n * splits_c * 2 * 4);
  const size_t end_part = off;
  off = p.off_part;
  const int64_t row_bytes = P0 * C0 * (int64_t)es, vt_bytes = (int64_t)C0 * attn_tp((int)P0) * (int64_t)es;
  p.off_qkv = take((size_t)n * 2 * row_bytes);
  p.off_vt = take((size_t)n * vt_bytes);
  p.off_ao = take((size_t)n * row_bytes);
  off = std::max(off, end_part);
  p.lane_stride = off - p.lane_off;
  // (per frame: the number of lanes is a property of the configuration, never of the slice)
  const int64_t lane = (elems_a + elems_b) * 4 + 2 * maxC * 4 + std::max(splits_c * 8, 3 * row_bytes + vt_bytes);
  const int64_t apart = 2 * elems_up * 4 + rows_c * 8 + 2 * maxC * 4 + 4 * row_bytes + vt_bytes;
  p.lanes = 2 * lane <= apart ? 2 : 1;
  p.total = p.lane_off + p.lanes * p.lane_stride;
  return p;
}

inline int eff_slice(const lc_decoder_config& g, int slice_frames) {
  return (slice_frames <= 0 || slice_frames > g.N) ? g.N : slice_frames;
}

// Partial sums [frame][splits][C][2] of a tensor, written by the kernel that produced it (part == nullptr: none)
struct Stats { const float* part; int splits; };

// scale / shift of GroupNorm(x) for n frames of fp32 rows [rows][C]; st: the partial sums of x if its producer wrote them
lc_status gn(lc_decoder* d, const DPlan& p, const float* x, Stats st, int n, int rows, int C, const GnP& w) {
  const lc_decoder_config& g = d->cfg;
  if (!st.part) {
    float* part = (float*)(d->lane + p.off_part);
    LCD_HIP(d, launch_gn_stats(d->s, kF32, x, part, n, rows, C));
    st = Stats{part, stat_splits(rows)};
  }
  LCD_HIP(d, launch_gn_finalize(d->s, st.part, C, st.splits, rows, 1.f, nullptr, 0, 0, 0, 0.f, w.g, w.b, g.groups, g.gn_eps,
                                (float*)(d->lane + p.off_scale), (float*)(d->lane + p.off_shift), n));
  return LC_OK;
}

// y = [res +] conv3x3(act(x)) at H x W, y fp32 rows with its partial sums. src 2: act = SiLU(GroupNorm(x)) with the scale /
// shift at hand; src 1: x, at half the resolution, nearest 2x upsampled on the way in; src 0: the same with x rounded already.
// act: room for the activated rows, act_bytes of it, or nullptr. y16: y is rounded to bf16 rows instead, without partial sums
// (*st is then what it was).
lc_status conv(lc_decoder* d, const DPlan& p, const ConvP& w, int src, int Cin, int Cout, int n, int H, int W, const void* x,
               const float* res, void* y, Stats* st, void* act = nullptr, size_t act_bytes = 0, bool y16 = false) {
  FusedDesc f;
  memset(&f, 0, sizeof f);
  f.xact = act; f.xact_bytes = act_bytes;
  f.dt = d->cfg.dtype; f.y_f32 = y16 ? 0 : 1; f.taps = 9; f.src = src; f.Cin = Cin; f.Cout = Cout; f.Cout_store = Cout;
  f.w = w.w; f.bias = w.b; f.frames = n; f.H = H; f.W = W; f.x = x; f.res = res; f.y = y; f.up2 = src < 2;
  f.unit_scale = src == 1;  // (off_one, off_zero)
  f.scale = (const float*)(src == 2 ? d->lane + p.off_scale : d->arena + p.off_one);
  f.shift = (const float*)(src == 2 ? d->lane + p.off_shift : d->arena + p.off_zero);
  f.in_map = f.out_map = RowMap{0, 0, 1 << 30};
  if (!y16) { f.stat = (float*)(d->lane + p.off_part); f.stat_splits = conv_stat_splits(H, W); }  // (those of x are folded by now)
  LCD_HIP(d, launch_fused(d->s, f));
  if (!y16) *st = Stats{f.stat, f.stat_splits};
  return LC_OK;
}

// whether launch_conv_dma takes a convolution of these widths over frames of this size
bool conv_covered(lc_decoder* d, const ConvP& w, int Cin, int Cout, int H, int W, bool up2) {
  FusedDesc f;
  memset(&f, 0, sizeof f);
  f.dt = d->cfg.dtype; f.taps = 9; f.Cin = Cin; f.Cout = Cout; f.Cout_store = Cout; f.H = H; f.W = W; f.up2 = up2;
  return launch_conv_dma(d->s, f) == hipSuccess;  // (no frames: nothing is launched)
}

// Room for the activated rows of a residual block's convolution over n frames of H x W x C: behind the map of that size at the
// start of buffer `a`, which holds the largest map of all. A property of the configuration, never of the slice.
void* res_act(lc_decoder* d, const DPlan& p, int C, int n, int H, int W, size_t* bytes) {
  const size_t e = (size_t)H * W * C;
  *bytes = 0;
  if (d->cfg.dtype != kBF16 || e * 6 > p.frame_a) return nullptr;
  *bytes = (size_t)n * e * 2;
  return d->lane + p.off_a + (size_t)n * e * 4;
}

// y16: y as bf16 rows (what a convolution reads that takes them as they are)
lc_status res_block(lc_decoder* d, const DPlan& p, int idx, int C, int n, int H, int W, const float* x, float* y, Stats* st, bool y16 = false) {
  lc_status s = gn(d, p, x, *st, n, H * W, C, d->res_gn[idx]);
  if (s != LC_OK) return s;
  size_t bytes;
  void* act = res_act(d, p, C, n, H, W, &bytes);
  return conv(d, p, d->res[idx], 2, C, C, n, H, W, x, x, y, st, act, bytes, y16);
}

// h += proj(Attn(qkv(GroupNorm(h)))) over the H*W positions of each frame, in place on fp32 rows
lc_status attn_block(lc_decoder* d, const DPlan& p, int n, float* h, Stats* st) {
  const lc_decoder_config& g = d->cfg;
  const int T = g.H * g.W, C = g.widths[0], Tp = attn_tp(T);
  const int64_t rows = (int64_t)n * T;
  lc_status s = gn(d, p, h, *st, n, T, C, d->at_gn);
  if (s != LC_OK) return s;
  *st = Stats{nullptr, 0};
  const float* scale = (const float*)(d->lane + p.off_scale);
  const float* shift = (const float*)(d->lane + p.off_shift);
  char* qk = d->lane + p.off_qkv;
  char* vt = d->lane + p.off_vt;
  char* ao = d->lane + p.off_ao;
  // q (with the softmax scale) and k as rows, V transposed from the projection's epilogue. The streamed linear kernel
  // takes normalised bf16 rows (in the buffer of the attention output, free until then); other widths and types are
  // normalised in the loader.
  const bool dense = g.dtype == kBF16 && lin2_covers(C, 3 * C) && lin2_covers(C, C) && T % 4 == 0;
  if (dense) LCD_HIP(d, launch_gn_apply(d->s, h, scale, shift, ao, rows, C, T, RowMap{0, T, T}));
  FusedDesc f;
  memset(&f, 0, sizeof f);
  f.dt = g.dtype; f.y_f32 = 0; f.taps = 1; f.src = dense ? 0 : 1; f.Cin = C; f.Cout = 3 * C; f.Cout_store = 3 * C; f.w = d->at_wqkv;
  f.rows = rows; f.in_map = RowMap{0, T, T}; f.out_map = RowMap{0, 0, 1 << 30}; f.x = dense ? (void*)ao : (void*)h; f.y = qk;
  f.scale = scale; f.shift = shift;
  f.q_cols = C; f.q_scale = attn_q_scale(g.head_dim);
  f.yt = vt; f.yt_from = 2 * C; f.yt_T = T; f.yt_Tp = Tp;
  LCD_HIP(d, launch_fused(d->s, f));
  LCD_HIP(d, launch_spatial_attention(d->s, g.dtype, qk, 2 * C, vt, Tp, ao, n, T, g.heads, g.head_dim, 0, T, 1, 0));
  memset(&f, 0, sizeof f);
  f.dt = g.dtype; f.y_f32 = 1; f.taps = 1; f.src = 0; f.Cin = C; f.Cout = C; f.Cout_store = C; f.w = d->at_wo; f.bias = d->at_bo;
  f.rows = rows; f.in_map = f.out_map = RowMap{0, 0, 1 << 30}; f.x = ao; f.res = h; f.y = h;
  LCD_HIP(d, launch_fused(d->s, f));
  return LC_OK;
}

// one pass: n frames of latents z -> n decoded images
lc_status decode_pass(lc_decoder* d, const DPlan& p, const void* z, void* img, int n) {
  const lc_decoder_config& g = d->cfg;
  float* a = (float*)(d->lane + p.off_a);
  float* b = (float*)(d->lane + p.off_b);
  int H = g.H, W = g.W;
  const int C0 = g.widths[0];
  Stats st{nullptr, 0};
  {
    float* part = (float*)(d->lane + p.off_part);
    const hipError_t e = d->cin_wp ? launch_conv_in_tile(d->s, g.dtype, z, d->cin_wp, d->cin_b, a, part, n, H, W, g.C_lat, C0, Win{0, 0, 0, 0})
                                   : hipErrorNotSupported;
    if (e == hipSuccess) st = Stats{part, conv_in_splits(H, W)};
    else if (e != hipErrorNotSupported) LCD_HIP(d, e);
    else LCD_HIP(d, launch_conv_in(d->s, g.dtype, z, a, n, H, W, g.C_lat, C0, d->cin_w, d->cin_b));
  }
  lc_status s = res_block(d, p, 0, C0, n, H, W, a, b, &st);
  if (s != LC_OK) return s;
  if ((s = attn_block(d, p, n, b, &st)) != LC_OK) return s;
  if ((s = res_block(d, p, 1, C0, n, H, W, b, a, &st)) != LC_OK) return s;
  for (int l = 0; l < g.levels; ++l) {
    const int Cl = g.widths[l], Cn = g.widths[l + 1];
    // only the upsampling convolution reads the block's output, rounded to bf16 as it contracts it: where both take the
    // kernel over activated rows, the block leaves it so
    size_t bytes;
    const bool y16 = res_act(d, p, Cl, n, H, W, &bytes) && conv_covered(d, d->res[2 + l], Cl, Cl, H, W, false) &&
                     conv_covered(d, d->upc[l], Cl, Cn, 2 * H, 2 * W, true);
    if ((s = res_block(d, p, 2 + l, Cl, n, H, W, a, b, &st, y16)) != LC_OK) return s;
    H *= 2; W *= 2;
    if ((s = conv(d, p, d->upc[l], y16 ? 0 : 1, Cl, Cn, n, H, W, b, nullptr, a, &st)) != LC_OK) return s;
  }
  const int CL = g.widths[g.levels];
  if ((s = gn(d, p, a, st, n, H * W, CL, d->out_gn)) != LC_OK) return s;
  const float* scale = (const float*)(d->lane + p.off_scale);
  const float* shift = (const float*)(d->lane + p.off_shift);
  const hipError_t e = launch_conv_out_tile(d->s, g.dtype, a, scale, shift, d->out.w, d->out.b, img, n, H, W, CL, g.C_img, Win{0, 0, 0, 0});
  if (e == hipSuccess) return LC_OK;
  if (e != hipErrorNotSupported) LCD_HIP(d, e);
  FusedDesc f;
  memset(&f, 0, sizeof f);
  f.dt = g.dtype; f.taps = 9; f.src = 2; f.Cin = CL; f.Cout = 32; f.Cout_store = g.C_img; f.w = d->out.w; f.bias = d->out.b;
  f.frames = n; f.H = H; f.W = W; f.x = a; f.y = img; f.planar_out = 1; f.scale = scale; f.shift = shift;
  f.in_map = f.out_map = RowMap{0, 0, 1 << 30};
  LCD_HIP(d, launch_fused(d->s, f));
  return LC_OK;
}

}  // namespace

extern "C" {

const char* lc_decoder_last_error(const lc_decoder* d) { return d ? d->err.c_str() : g_derr.c_str(); }

lc_status lc_decoder_check_config(const lc_decoder_config* cfg) { return check_dcfg(nullptr, cfg); }

size_t lc_decoder_workspace_bytes(const lc_decoder_config* cfg, int slice_frames) {
  if (check_dcfg(nullptr, cfg) != LC_OK) return 0;
  if (slice_frames < 0) { g_derr = "slice_frames must be >= 0"; return 0; }
  return make_dplan(*cfg, eff_slice(*cfg, slice_frames)).total;
}

lc_status lc_decoder_create(const lc_decoder_config* cfg, void* stream, lc_decoder** out) {
  if (!out) return dfail(nullptr, LC_ERR_ARG, "out is NULL");
  lc_status s = check_dcfg(nullptr, cfg);
  if (s != LC_OK) return s;
  if (!stream) return dfail(nullptr, LC_ERR_ARG, "stream must be a non-default stream");
  lc_decoder* d = new (std::nothrow) lc_decoder();
  if (!d) return dfail(nullptr, LC_ERR_NOMEM, "out of host memory");
  d->cfg = *cfg;
  d->s = d->s_main = (hipStream_t)stream;
  d->s_aux = nullptr; d->ev_fork = d->ev_join = nullptr; d->lane = nullptr;
  if (hipStreamCreateWithFlags(&d->s_aux, hipStreamNonBlocking) != hipSuccess ||
      hipEventCreateWithFlags(&d->ev_fork, hipEventDisableTiming) != hipSuccess ||
      hipEventCreateWithFlags(&d->ev_join, hipEventDisableTiming) != hipSuccess) {
    d->wblob = nullptr;
    lc_decoder_destroy(d);
    return dfail(nullptr, LC_ERR_HIP, "creating the second stream failed");
  }
  d->wblob = nullptr; d->wblob_bytes = 0; d->have_weights = false;
  d->arena = nullptr; d->arena_bytes = 0;
  *out = d;
  return LC_OK;
}

lc_status lc_decoder_destroy(lc_decoder* d) {
  if (!d) return LC_OK;
  (void)hipStreamSynchronize(d->s_main);
  if (d->s_aux) (void)hipStreamDestroy(d->s_aux);
  if (d->ev_fork) (void)hipEventDestroy(d->ev_fork);
  if (d->ev_join) (void)hipEventDestroy(d->ev_join);
  if (d->wblob) (void)hipFree(d->wblob);
  delete d;
  return LC_OK;
}

lc_status lc_decoder_load_weights(lc_decoder* d, const lc_decoder_weights* w) {
  if (!d) return dfail(nullptr, LC_ERR_ARG, "decoder is NULL");
  if (!w) return dfail(d, LC_ERR_ARG, "weights is NULL");
  const lc_decoder_config& g = d->cfg;
  const int dt = g.dtype, L = g.levels, C0 = g.widths[0], CL = g.widths[L];
  const size_t es = dtype_size(dt);
  auto need_gc = [](const lc_gnconv_w& x) { return x.gn_g && x.gn_b && x.w && x.b; };
  bool ok = w->conv_in_w && w->conv_in_b && need_gc(w->mid_res[0]) && need_gc(w->mid_res[1]) && need_gc(w->out) &&
            w->mid_attn.gn_g && w->mid_attn.gn_b && w->mid_attn.wq && w->mid_attn.wk && w->mid_attn.wv && w->mid_attn.wo &&
            w->mid_attn.bo;
  for (int l = 0; l < L; ++l) ok = ok && need_gc(w->up_res[l]) && w->up_conv_w[l] && w->up_conv_b[l];
  if (!ok) return dfail(d, LC_ERR_ARG, "a weight pointer is NULL");
  size_t off = 0;
  auto take = [&](size_t bytes) { size_t o = off; off += align_up(bytes); return o; };
  const size_t o_cin_w = take((size_t)g.C_lat * 9 * C0 * 4), o_cin_b = take((size_t)C0 * 4), o_cin_wp = take((size_t)C0 * 64 * es);
  size_t o_rg[2 + LC_DEC_MAX_LEVELS], o_rb[2 + LC_DEC_MAX_LEVELS], o_rw[2 + LC_DEC_MAX_LEVELS], o_rbias[2 + LC_DEC_MAX_LEVELS];
  for (int i = 0; i < 2 + L; ++i) {
    const int C = i < 2 ? C0 : g.widths[i - 2];
    o_rg[i] = take((size_t)C * 4); o_rb[i] = take((size_t)C * 4); o_rw[i] = take((size_t)C * 9 * C * es); o_rbias[i] = take((size_t)C * 4);
  }
  const size_t o_ag = take((size_t)C0 * 4), o_ab = take((size_t)C0 * 4), o_aqkv = take((size_t)3 * C0 * C0 * es),
               o_awo = take((size_t)C0 * C0 * es), o_abo = take((size_t)C0 * 4);
  size_t o_uw[LC_DEC_MAX_LEVELS], o_ub[LC_DEC_MAX_LEVELS];
  for (int l = 0; l < L; ++l) { o_uw[l] = take((size_t)g.widths[l + 1] * 9 * g.widths[l] * es); o_ub[l] = take((size_t)g.widths[l + 1] * 4); }
  const size_t o_og = take((size_t)CL * 4), o_ob = take((size_t)CL * 4), o_ow = take((size_t)32 * 9 * CL * es), o_obias = take(32 * 4);

  LCD_HIP(d, hipStreamSynchronize(d->s));
  if (d->wblob) { LCD_HIP(d, hipFree(d->wblob)); d->wblob = nullptr; d->have_weights = false; }
  void* blob = nullptr;
  if (hipMalloc(&blob, off) != hipSuccess) return dfail(d, LC_ERR_NOMEM, "hipMalloc of %zu bytes for packed weights failed", off);
  d->wblob = blob; d->wblob_bytes = off;
  char* b = (char*)blob;
  hipStream_t s = d->s;
#define F32(src, dst_off, n, npad) LCD_HIP(d, launch_to_f32(s, dt, src, (float*)(b + dst_off), n, npad))
  // bf16: the fragment order that all kernels of the 3x3 convolutions read
#define CF(src, dst_off, co, ci)                                                                  \
  LCD_HIP(d, dt == kBF16 ? launch_pack_conv_w_frags(s, dt, src, b + dst_off, co, ci) : launch_pack_conv_w(s, dt, src, b + dst_off, co, ci, 9, co))
  LCD_HIP(d, launch_pack_conv_in_w(s, dt, w->conv_in_w, (float*)(b + o_cin_w), C0, g.C_lat));
  F32(w->conv_in_b, o_cin_b, C0, C0);
  d->cin_w = (float*)(b + o_cin_w); d->cin_b = (float*)(b + o_cin_b); d->cin_wp = nullptr;
  if (dt == kBF16 && g.C_lat * 9 <= 64) {
    LCD_HIP(d, launch_pad_rows(s, dt, w->conv_in_w, b + o_cin_wp, C0, g.C_lat * 9, 64));
    d->cin_wp = b + o_cin_wp;
  }
  for (int i = 0; i < 2 + L; ++i) {
    const int C = i < 2 ? C0 : g.widths[i - 2];
    const lc_gnconv_w& r = i < 2 ? w->mid_res[i] : w->up_res[i - 2];
    F32(r.gn_g, o_rg[i], C, C); F32(r.gn_b, o_rb[i], C, C); CF(r.w, o_rw[i], C, C); F32(r.b, o_rbias[i], C, C);
    d->res_gn[i] = GnP{(float*)(b + o_rg[i]), (float*)(b + o_rb[i])};
    d->res[i] = ConvP{b + o_rw[i], (float*)(b + o_rbias[i])};
  }
  F32(w->mid_attn.gn_g, o_ag, C0, C0); F32(w->mid_attn.gn_b, o_ab, C0, C0);
  LCD_HIP(d, launch_copy_rows(s, dt, w->mid_attn.wq, b + o_aqkv, (int64_t)C0 * C0));
  LCD_HIP(d, launch_copy_rows(s, dt, w->mid_attn.wk, b + o_aqkv + (size_t)C0 * C0 * es, (int64_t)C0 * C0));
  LCD_HIP(d, launch_copy_rows(s, dt, w->mid_attn.wv, b + o_aqkv + (size_t)2 * C0 * C0 * es, (int64_t)C0 * C0));
  LCD_HIP(d, launch_copy_rows(s, dt, w->mid_attn.wo, b + o_awo, (int64_t)C0 * C0));
  F32(w->mid_attn.bo, o_abo, C0, C0);
  d->at_gn = GnP{(float*)(b + o_ag), (float*)(b + o_ab)};
  d->at_wqkv = b + o_aqkv; d->at_wo = b + o_awo; d->at_bo = (float*)(b + o_abo);
  for (int l = 0; l < L; ++l) {
    CF(w->up_conv_w[l], o_uw[l], g.widths[l + 1], g.widths[l]);
    F32(w->up_conv_b[l], o_ub[l], g.widths[l + 1], g.widths[l + 1]);
    d->upc[l] = ConvP{b + o_uw[l], (float*)(b + o_ub[l])};
  }
  F32(w->out.gn_g, o_og, CL, CL); F32(w->out.gn_b, o_ob, CL, CL);
  LCD_HIP(d, launch_pack_conv_w(s, dt, w->out.w, b + o_ow, g.C_img, CL, 9, 32)); F32(w->out.b, o_obias, g.C_img, 32);
  d->out_gn = GnP{(float*)(b + o_og), (float*)(b + o_ob)};
  d->out = ConvP{b + o_ow, (float*)(b + o_obias)};
#undef F32
#undef CF
  LCD_HIP(d, hipStreamSynchronize(s));
  d->have_weights = true;
  return LC_OK;
}

lc_status lc_decoder_set_workspace(lc_decoder* d, void* arena, size_t bytes) {
  if (!d) return dfail(nullptr, LC_ERR_ARG, "decoder is NULL");
  if (!arena) return dfail(d, LC_ERR_ARG, "arena is NULL");
  if ((uintptr_t)arena % kAlign) return dfail(d, LC_ERR_ARG, "arena must be 256-byte aligned");
  LCD_HIP(d, hipStreamSynchronize(d->s));
  d->arena = (char*)arena;
  d->arena_bytes = bytes;
  return LC_OK;
}

lc_status lc_decode(lc_decoder* d, const void* z, void* img, int slice_frames) {
  if (!d) return dfail(nullptr, LC_ERR_ARG, "decoder is NULL");
  if (!z || !img) return dfail(d, LC_ERR_ARG, "z and img must not be NULL");
  if (slice_frames < 0) return dfail(d, LC_ERR_ARG, "slice_frames must be >= 0");
  if (!d->have_weights) return dfail(d, LC_ERR_STATE, "weights not loaded");
  if (!d->arena) return dfail(d, LC_ERR_STATE, "workspace not set");
  const lc_decoder_config& g = d->cfg;
  const int n = eff_slice(g, slice_frames);
  const DPlan p = make_dplan(g, n);
  if (p.total > d->arena_bytes)
    return dfail(d, LC_ERR_NOMEM, "a slice of %d frames needs %zu bytes of workspace, %zu are set", n, p.total, d->arena_bytes);
  const size_t es = dtype_size(g.dtype);
  int maxC = 0;
  for (int l = 0; l <= g.levels; ++l) maxC = std::max(maxC, (int)g.widths[l]);
  LCD_HIP(d, launch_fill_f32(d->s, (float*)(d->arena + p.off_one), (int64_t)n * maxC, 1.f));
  LCD_HIP(d, launch_fill_f32(d->s, (float*)(d->arena + p.off_zero), (int64_t)n * maxC, 0.f));
  const size_t zf = (size_t)g.C_lat * g.H * g.W * es;
  const size_t imf = (size_t)g.C_img * ((size_t)g.H << g.levels) * ((size_t)g.W << g.levels) * es;
  // Slices depend on nothing but the weights: alternate ones go to the caller's stream and to one of the library's own,
  // forked from and joined into it here, each with its own scratch. The launches of one frame leave most of the device
  // idle at the latent resolution (64 workgroups), and one slice's fill the other's gaps.
  const int lanes = std::min(p.lanes, (g.N + n - 1) / n);
  if (lanes > 1) {
    LCD_HIP(d, hipEventRecord(d->ev_fork, d->s_main));
    LCD_HIP(d, hipStreamWaitEvent(d->s_aux, d->ev_fork, 0));
  }
  lc_status s = LC_OK;
  for (int n0 = 0, i = 0; n0 < g.N && s == LC_OK; n0 += n, ++i) {
    d->s = i % lanes ? d->s_aux : d->s_main;
    d->lane = d->arena + (i % lanes) * p.lane_stride;
    s = decode_pass(d, p, (const char*)z + n0 * zf, (char*)img + n0 * imf, std::min(n, g.N - n0));
  }
  d->s = d->s_main;
  if (lanes > 1) {  // whatever happened: joined
    LCD_HIP(d, hipEventRecord(d->ev_join, d->s_aux));
    LCD_HIP(d, hipStreamWaitEvent(d->s_main, d->ev_join, 0));
  }
  return s;
}

lc_status lc_decoder_sync(lc_decoder* d) {
  if (!d) return dfail(nullptr, LC_ERR_ARG, "decoder is NULL");
  LCD_HIP(d, hipStreamSynchronize(d->s));
  return LC_OK;
}

}  // extern "C"
