// Linear layers over dense bf16 rows on gfx950: y[rows][N] = x[rows][K] W[N][K]^T (+ bias, + fp32 residual), the
// projections and feed-forward layers of the transformer blocks, where K is a few hundred to a few thousand.
//
// One workgroup = 4 wavefronts = 128 rows x 160 (or 128) output channels; wavefront w owns rows [32 w, 32 w + 32) and
// all channels (5 or 4 accumulator tiles of 32 x 32: every fragment of x feeds five or four MFMAs), and walks K in
// steps of 64 elements without splitting it. Both operands are K-major in memory, so a step's tiles are rows of 128
// bytes, brought from global memory straight into LDS (16 bytes per lane, no registers in between) into a ring of two
// stages: the loads of step s + 1 are issued as soon as those of step s have landed. Two workgroups share a compute
// unit (2 x 74 KB of LDS, 256 registers each) and cover each other's prologue, waits and epilogue. (The first design,
// a 256-row tile with a ring of three stages and one workgroup per compute unit, was slower at every K measured: by
// 6 % at K = 1280, by 13-22 % from K = 1024 to 4096 where the output is narrow.) The 16-byte packet c of row r is
// parked in slot c ^ ((r >> 1) & 7) of its row, which makes the fragment reads (32 consecutive rows, one slot)
// conflict-free without padding. The product is not transposed (rows of x are the rows of the accumulator tile): a
// lane then holds one output channel of 16 rows, and the 32 lanes of a half-wavefront hold 32 consecutive channels of
// one row.
//
// Workgroups are dealt to the eight XCDs round robin in launch order, and each XCD has an L2 of its own: the
// channel tiles of one row tile are mapped to the same XCD, so its L2 fetches that tile of x once.
#include "lc_lin_epi.h"

namespace lc {

namespace {

constexpr int kKB = 128;                        // K bytes per step
constexpr int kStages = 2;
// a workgroup takes 128 rows and 32 NT channels; bytes of one ring stage: the x tile, then the W tile
constexpr int lin2_stage(int NT) { return (128 + NT * 32) * kKB; }
static_assert(2 * kStages * lin2_stage(5) <= 160 * 1024, "two workgroups fit the LDS of a compute unit together");

}  // namespace


// MAPPED: rows go through the row maps (a 64-bit division per row: kept out of the common, dense case, where the
// host folds the maps' offsets into the pointers; the arithmetic, and so every bit of the result, is the same)
template <class OT, int NT, bool MAPPED>
__global__ __launch_bounds__(256, 2) void lin2_kernel(Lin2Args a) {
  typedef Mma32<bf16_t> M;
  constexpr int MR = 1;  // 32-row accumulator tiles per wavefront along the rows
  constexpr int kM = 128 * MR, kN = NT * 32, kStage = lin2_stage(NT);
  constexpr int kXI = 4 * MR, kWI = NT;  // global->LDS instructions per wavefront per stage: x tile, W tile
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lp = lane & 31, hh = lane >> 5;
  // (row tile, channel tile) of this workgroup: all channel tiles of a row tile on one XCD
  const int lin = blockIdx.x, xcd = lin & 7, slot = lin >> 3;
  const int mt = xcd + 8 * (slot / a.ntn), nt = slot - (slot / a.ntn) * a.ntn;
  if (mt >= a.ntm) return;  // the grid is padded to whole rounds of eight row tiles
  const int64_t m0 = (int64_t)mt * kM;
  const int n0 = nt * kN;

  // ---- global -> LDS: instruction i of a tile moves rows 8 i .. 8 i + 7; this lane moves the packet that lands
  //      in slot (lane & 7) of row 8 i + (lane >> 3), i.e. global packet (lane & 7) ^ ((row >> 1) & 7)
  const int lrow = lane >> 3;
  const bf16_t* xsrc[kXI];
  const bf16_t* wsrc[kWI];
#pragma unroll
  for (int j = 0; j < kXI; ++j) {
    const int r = (wid + 4 * j) * 8 + lrow;
    const int c = (lane & 7) ^ ((r >> 1) & 7);
    int64_t gr = min(m0 + r, a.rows - 1);  // rows beyond the end: a valid row, never stored
    if (MAPPED) gr = a.in_map(gr);
    xsrc[j] = a.x + gr * a.K + c * 8;
  }
#pragma unroll
  for (int j = 0; j < kWI; ++j) {
    const int r = (wid + 4 * j) * 8 + lrow;
    const int c = (lane & 7) ^ ((r >> 1) & 7);
    wsrc[j] = a.w + (int64_t)(n0 + r) * a.K + c * 8;
  }
  auto issue = [&](int step, int buf) {
    unsigned char* xb = smem + buf * kStage;
    unsigned char* wb = xb + kM * kKB;
    const int kofs = step * 64;
#ifdef __HIP_DEVICE_COMPILE__  // the host pass only needs the kernel's stub; it does not know this builtin
#pragma unroll
    for (int j = 0; j < kXI; ++j) __builtin_amdgcn_global_load_lds(xsrc[j] + kofs, xb + (wid + 4 * j) * 1024, 16, 0, 0);
#pragma unroll
    for (int j = 0; j < kWI; ++j) __builtin_amdgcn_global_load_lds(wsrc[j] + kofs, wb + (wid + 4 * j) * 1024, 16, 0, 0);
#else
    (void)xb; (void)wb; (void)kofs;
#endif
  };

  f32x16 acc[MR][NT];
#pragma unroll
  for (int j = 0; j < MR; ++j)
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[j][i][r] = 0.f;

  // fragment addresses inside a stage: row * 128 + ((slot ^ key) << 4), slot = hh + 2 kk
  const int xrow0 = wid * (32 * MR) + lp, xkey = (xrow0 >> 1) & 7;  // (+32 does not change the key)
  const int wkey = (lp >> 1) & 7;
  auto xfrag = [&](const unsigned char* st, int j, int kk) {
    return M::load((const bf16_t*)(st + (xrow0 + 32 * j) * kKB + (((hh + 2 * kk) ^ xkey) << 4)));
  };
  auto wfrag = [&](const unsigned char* st, int i, int kk) {
    return M::load((const bf16_t*)(st + kM * kKB + (32 * i + lp) * kKB + (((hh + 2 * kk) ^ wkey) << 4)));
  };

  const int nsteps = a.K / 64;
  issue(0, 0);
  for (int s = 0; s < nsteps; ++s) {
    // the loads of step s have landed (for every wavefront, after the barrier), and every wavefront has read step s - 1
    barrier_keep<0>();
    // the next request goes into the stage that was read in step s - 1
    if (s + 1 < nsteps) issue(s + 1, (s + 1) % kStages);
    const unsigned char* st = smem + (s % kStages) * kStage;
    typename M::Frag xf[2][MR], wf[2][NT];
#pragma unroll
    for (int j = 0; j < MR; ++j) xf[0][j] = xfrag(st, j, 0);
#pragma unroll
    for (int i = 0; i < NT; ++i) wf[0][i] = wfrag(st, i, 0);
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      if (kk + 1 < 4) {  // the fragments of the next k-step are requested before this one's MFMAs
#pragma unroll
        for (int j = 0; j < MR; ++j) xf[(kk + 1) & 1][j] = xfrag(st, j, kk + 1);
#pragma unroll
        for (int i = 0; i < NT; ++i) wf[(kk + 1) & 1][i] = wfrag(st, i, kk + 1);
      }
#pragma unroll
      for (int i = 0; i < NT; ++i)
#pragma unroll
        for (int j = 0; j < MR; ++j) M::mma(xf[kk & 1][j], wf[kk & 1][i], acc[j][i]);
    }
  }

  // ---- epilogue: lane holds channel n0 + 32 i + lp of rows m0 + 32 MR wid + 32 j + 8 (r / 4) + 4 hh + r % 4
  float bias_l[NT], mul_l[NT];
#pragma unroll
  for (int i = 0; i < NT; ++i) {
    const int co = n0 + 32 * i + lp;
    bias_l[i] = a.bias ? a.bias[co] : 0.f;
    mul_l[i] = co < a.q_cols ? a.q_scale : 1.f;
  }
#pragma unroll
  for (int j = 0; j < MR; ++j)
    lin_epilogue<OT, NT, MAPPED, false>(a, acc[j], m0 + wid * (32 * MR) + 32 * j, n0, lane, bias_l, mul_l);
}

// taps == 1, src == 0 of a bf16 stage, Cin % 64 == 0 and Cout % 160 == 0 or % 128 == 0 (rows through any row map);
// hipErrorNotSupported for what it does not cover (the general kernel then runs). Whether it covers a launch depends on
// the layer's widths only, never on the number of rows: a chunked pass must give the bits of the unchunked one (the tiles
// of lc_lin3.hip, which dense launches may take by their rows, give the same bits).
// (hipFuncSetAttribute is called once per instantiation and process: one device.)
template <class OT, int NT, bool MAPPED>
static hipError_t run_lin2_k(hipStream_t s, const Lin2Args& a) {
  constexpr int lds = kStages * lin2_stage(NT);
  static bool done = false;  // per instantiation
  if (!done) {
    hipError_t e = hipFuncSetAttribute((const void*)lin2_kernel<OT, NT, MAPPED>, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
    done = true;
  }
  const unsigned grid = (unsigned)((a.ntm + 7) / 8 * 8 * a.ntn);
  lin2_kernel<OT, NT, MAPPED><<<grid, 256, lds, s>>>(a);
  return hipGetLastError();
}
template <class OT, int NT>
static hipError_t run_lin2(hipStream_t s, Lin2Args a) {
  a.ntn = a.N / (NT * 32);
  a.ntm = (int)((a.rows + 127) / 128);
  // a map that is the identity up to an offset (one segment, or segments that follow each other) is folded into
  // the pointers
  auto plain = [&](const RowMap& m) { return m.rows_per_seg >= a.rows || m.seg_stride == m.rows_per_seg; };
  if (!plain(a.in_map) || !plain(a.out_map)) return a.yt || a.gate ? hipErrorInvalidValue : run_lin2_k<OT, NT, true>(s, a);
  const int64_t nout = a.ldy;
  a.x += a.in_map.base * a.K;
  a.y = (OT*)a.y + a.out_map.base * nout;
  if (a.res) a.res += a.out_map.base * nout;
  if (a.y2) a.y2 += a.out_map.base * nout;
  if constexpr (NT == 4) {  // (yt_from is then a multiple of 128)
    return launch_lin3(s, a, sizeof(OT) == 4);
  } else {
    if (!a.yt || a.yt_from % 64 == 0) {
      const hipError_t e = launch_lin3(s, a, sizeof(OT) == 4);
      if (e != hipErrorNotSupported) return e;
    }
    return a.gate ? hipErrorInvalidValue : run_lin2_k<OT, NT, false>(s, a);
  }
}

hipError_t launch_lin2(hipStream_t s, const FusedDesc& d) {
  if (d.dt != kBF16 || d.taps != 1 || d.src != 0 || d.stat || d.win_w || d.planar_out) return hipErrorNotSupported;
  if (!lin2_covers(d.Cin, d.Cout) || d.Cout_store != d.Cout) return hipErrorNotSupported;
  if (d.in_map.rows_per_seg <= 0 || d.out_map.rows_per_seg <= 0) return hipErrorInvalidValue;
  if (d.res && !d.y_f32) return hipErrorNotSupported;
  if (d.q_cols && d.res) return hipErrorInvalidValue;
  if (d.y2 && !d.y_f32) return hipErrorInvalidValue;
  if (d.act && (d.y_f32 || d.res || d.q_cols || d.act > 2)) return hipErrorInvalidValue;
  if (d.act == 2 && d.Cout % 128) return hipErrorNotSupported;
  if (d.yt) {  // the transposed tail: whole channel tiles of a bf16 output, rows in fours
    const int tile = d.Cout % 160 == 0 ? 160 : 128;
    if (d.y_f32 || d.res || d.act || d.y2) return hipErrorInvalidValue;
    if (d.yt_from <= 0 || d.yt_from >= d.Cout || d.yt_from % tile || d.yt_T <= 0 || d.yt_T % 4 || d.rows % 4 || d.yt_Tp % 64 || d.yt_Tp < d.yt_T)
      return hipErrorNotSupported;
  }
  if (d.gate && (!lin_gate_covers(d.Cin, d.Cout) || !d.y_f32 || !d.res || d.y2 || d.gate_T < 32 || d.gate_n <= 0)) return hipErrorInvalidValue;
  if (d.rows <= 0) return hipSuccess;
  if (d.rows > (int64_t)1 << 30) return hipErrorNotSupported;
  if ((int64_t)d.Cout * 4 * 32 >= (int64_t)1 << 31) return hipErrorNotSupported;  // (32-bit offsets in a block of rows)
  Lin2Args a;
  a.x = (const bf16_t*)d.x; a.w = (const bf16_t*)d.w; a.bias = d.bias; a.res = (const float*)d.res; a.y = d.y;
  a.y2 = (bf16_t*)d.y2;
  a.rows = d.rows; a.K = d.Cin; a.N = d.Cout;
  a.ntm = a.ntn = 0;
  a.q_scale = d.q_cols ? d.q_scale : 1.f; a.q_cols = d.q_cols;
  a.act = d.act;
  a.in_map = d.in_map; a.out_map = d.out_map;
  a.yt = (bf16_t*)d.yt; a.yt_from = d.yt_from; a.yt_T = d.yt_T; a.yt_Tp = d.yt_Tp;
  a.gate = d.gate; a.gate_T = d.gate_T; a.gate_n = d.gate_n; a.gate_ld = d.gate_ld; a.row0 = d.row0;
  a.ldy = d.yt ? d.yt_from : (d.act == 2 ? d.Cout / 2 : d.Cout);
  if (d.act == 2) return run_lin2<bf16_t, 4>(s, a);  // (an even number of column tiles: value / gate pairs)
  if (d.Cout % 160 == 0) return d.y_f32 ? run_lin2<float, 5>(s, a) : run_lin2<bf16_t, 5>(s, a);
  return d.y_f32 ? run_lin2<float, 4>(s, a) : run_lin2<bf16_t, 4>(s, a);
}

}  // namespace lc
