// Linear layers over dense bf16 rows on gfx950: the tiles beside lc_lin2.hip's 128 x 160, wide ones for launches that fill
// the chip several times and small ones for launches that would leave most of it idle.
//
// Where a large launch's time goes (8192 x 4096 x 1024 with GELU, 256 x 256): 49 us per 1024 of K, 1.37 PFLOP/s, as fast as this
// card runs any long contraction, and about 25 us that do not depend on K: first loads, the epilogue and its stores (14 us at
// the rate of a copy), which one workgroup per compute unit does not cover. In small launches a compute unit has one wavefront per
// SIMD, and what a stage consists of adds up: requests, fragment reads, MFMAs, barrier.
// Measured, us (rows x N x K; fp32 outputs with their residual; in all figures of this file each launch behind one of the same shape
// on other buffers, so that short ones are close to what they are in a step and large ones a few percent more): lin2's 128 x 160
// -> this file's, 8192 x 3840 x 1280 86 -> 75 (256 x 256), 2048 x 320 x 1280 fp32 18 -> 8 (64 x 64); 128 x 128 -> the other
// tiles, 8192 x 4096 x 1024 with GELU 76 -> 73 (256 x 256), 3000 x 768 x 3072 fp32 36 -> 23 (64 x 128), 1024 x 1024 x 4096 fp32
// 39 -> 19 (64 x 64).
//
// The K loop: a ring of S stages of 64 K elements (global -> LDS directly, packet c of row r in slot c ^ ((r >> 1) & 7)).
// The one barrier of a step stands before its last group of MFMAs, whose operands are in registers by then: behind it the
// stage is free (every wavefront has read it), its next load is issued, and the first fragments of the next stage are
// requested, so that the barrier and the LDS round trip hide behind that group. K is walked in order by one wavefront per
// output element, as lin2_kernel does: the same bits whatever the tile, so the launch may choose the tile by its rows.
#include "lc_lin_epi.h"

namespace lc {

namespace {
constexpr int kKB3 = 128;  // K bytes per step
constexpr int kRawBuffer = 0x00020000;  // resource word 3: raw 32-bit data
typedef __attribute__((address_space(3))) unsigned char* lds_ptr;
}  // namespace

// WM x WN wavefronts of MT x NT accumulator tiles (32 x 32): a tile of 32 WM MT rows x 32 WN NT channels
template <class OT, int WM, int WN, int MT, int NT, int S>
__global__ __launch_bounds__(WM * WN * 64, 2) void lin3_kernel(Lin2Args a) {
  typedef Mma32<bf16_t> M;
  constexpr int NW = WM * WN, kM = 32 * WM * MT, kN = 32 * WN * NT, kStage = (kM + kN) * kKB3;
  constexpr int kXI = kM / 8 / NW, kWI = kN / 8 / NW, kPer = kXI + kWI;  // global->LDS instructions per wavefront per stage
  static_assert(kM % (8 * NW) == 0 && kN % (8 * NW) == 0, "whole wavefront instructions");
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wid / WN, wn = wid % WN;
  const int lp = lane & 31, hh = lane >> 5;
  // (row tile, channel tile) of this workgroup: workgroups go round the eight XCDs, and each XCD has a block of the tiles
  const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
  const int mt = xcd % a.xm * a.bm + slot / a.bn, nt = xcd / a.xm * a.bn + slot % a.bn;
  if (mt >= a.ntm || nt >= a.ntn) return;  // (the blocks at the ends may be smaller)
  const int64_t m0 = (int64_t)mt * kM;
  const int n0 = nt * kN;

  // ---- global -> LDS: instruction i of a tile moves rows 8 i .. 8 i + 7; this lane moves the packet that lands
  //      in slot (lane & 7) of row 8 i + (lane >> 3), i.e. global packet (lane & 7) ^ ((row >> 1) & 7)
  // Buffer loads: the compiler counts a FLAT-encoded load to LDS as one of LDS too, whose order is unknown, and then
  // waits for every fragment in flight where it needs the oldest; and their bounds check reads rows beyond the end as 0.
  const int lrow = lane >> 3;
  int xofs[kXI], wofs[kWI];  // bytes from the tile's first row
#pragma unroll
  for (int j = 0; j < kXI; ++j) {
    const int r = (wid + NW * j) * 8 + lrow;
    xofs[j] = r * a.K * 2 + (((lane & 7) ^ ((r >> 1) & 7)) << 4);
  }
#pragma unroll
  for (int j = 0; j < kWI; ++j) {
    const int r = (wid + NW * j) * 8 + lrow;
    wofs[j] = r * a.K * 2 + (((lane & 7) ^ ((r >> 1) & 7)) << 4);
  }
#ifdef __HIP_DEVICE_COMPILE__  // the host pass only needs the kernel's stub; it does not know these builtins
  const int xrows = (int)min((int64_t)kM, a.rows - m0);
  const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(a.x + m0 * a.K), 0, xrows * a.K * 2, kRawBuffer);
  const __amdgpu_buffer_rsrc_t wr = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(a.w + (int64_t)n0 * a.K), 0, kN * a.K * 2, kRawBuffer);
#endif
  auto issue = [&](int step, int buf) {
#ifdef __HIP_DEVICE_COMPILE__
    lds_ptr xb = (lds_ptr)(smem + buf * kStage), wb = xb + kM * kKB3;
    const int kofs = step * kKB3;
#pragma unroll
    for (int j = 0; j < kXI; ++j) __builtin_amdgcn_raw_ptr_buffer_load_lds(xr, xb + (wid + NW * j) * 1024, 16, xofs[j], kofs, 0, 0);
#pragma unroll
    for (int j = 0; j < kWI; ++j) __builtin_amdgcn_raw_ptr_buffer_load_lds(wr, wb + (wid + NW * j) * 1024, 16, wofs[j], kofs, 0, 0);
#else
    (void)step; (void)buf; (void)xofs; (void)wofs;
#endif
  };

  f32x16 acc[MT][NT];
#pragma unroll
  for (int j = 0; j < MT; ++j)
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[j][i][r] = 0.f;

  // fragment addresses inside a stage: row * 128 + ((slot ^ key) << 4), slot = hh + 2 kk (rows + 32 do not change the key)
  const int key = (lp >> 1) & 7;
  const int xrow0 = wm * (32 * MT) + lp, wrow0 = kM + wn * (32 * NT) + lp;
  const int nsteps = a.K / 64;
#pragma unroll
  for (int j = 0; j < S; ++j)
    if (j < nsteps) issue(j, j);
  if (nsteps >= S) barrier_keep<(S - 1) * kPer>();
  else barrier_keep<0>();
  // this wavefront has read its last fragments of the stage at hand, and its loads of the next one have landed (those of
  // the S - 2 stages behind it may be on their way; at the end of K there are fewer)
  auto step_end = [&](int s) __attribute__((always_inline)) {
    if (s + S - 1 < nsteps) barrier_keep<(S - 2) * kPer>();
    else barrier_keep<0>();
  };
  int buf = 0;
  if constexpr (MT * NT <= 2) {
    // A wavefront with few accumulators has few MFMAs to put between a fragment's request and its use, and one wavefront per
    // SIMD has nothing else: k-step by k-step an LDS round trip stood in front of each (1024 x 1024 x 4096: 660 clocks a
    // stage for 4 MFMAs). Here all fragments of a stage are in registers when its first MFMA is issued, and behind the
    // last MFMA that needs a fragment the same registers are requested for the next stage.
    typename M::Frag xf[4][MT], wf[4][NT];
    auto frag = [&](const unsigned char* st, int kk) __attribute__((always_inline)) {
      const int so = ((hh + 2 * kk) ^ key) << 4;
#pragma unroll
      for (int j = 0; j < MT; ++j) xf[kk][j] = M::load((const bf16_t*)(st + (xrow0 + 32 * j) * kKB3 + so));
#pragma unroll
      for (int i = 0; i < NT; ++i) wf[kk][i] = M::load((const bf16_t*)(st + (wrow0 + 32 * i) * kKB3 + so));
    };
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) frag(smem, kk);
    for (int s = 0; s < nsteps; ++s) {
      const int bnext = buf + 1 == S ? 0 : buf + 1;
      if (s + 1 < nsteps) step_end(s);
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) {
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < NT; ++i)
#pragma unroll
          for (int j = 0; j < MT; ++j) M::mma(xf[kk][j], wf[kk][i], acc[j][i]);
        __builtin_amdgcn_sched_barrier(0);
        frag(smem + bnext * kStage, kk);  // (behind the last stage they are of no stage: in bounds, never used)
      }
      __builtin_amdgcn_sched_barrier(0);
      if (s + S < nsteps) issue(s + S, buf);
      buf = bnext;
    }
  } else {
    typename M::Frag xf[2][MT], wf[2][NT];
    auto frags = [&](const unsigned char* st, int kk, int b) __attribute__((always_inline)) {
      const int so = ((hh + 2 * kk) ^ key) << 4;
#pragma unroll
      for (int j = 0; j < MT; ++j) xf[b][j] = M::load((const bf16_t*)(st + (xrow0 + 32 * j) * kKB3 + so));
#pragma unroll
      for (int i = 0; i < NT; ++i) wf[b][i] = M::load((const bf16_t*)(st + (wrow0 + 32 * i) * kKB3 + so));
    };
    auto mma = [&](int b) __attribute__((always_inline)) {
#pragma unroll
      for (int i = 0; i < NT; ++i)
#pragma unroll
        for (int j = 0; j < MT; ++j) M::mma(xf[b][j], wf[b][i], acc[j][i]);
    };
    frags(smem, 0, 0);
    for (int s = 0; s < nsteps; ++s) {
      const unsigned char* st = smem + buf * kStage;
      const int bnext = buf + 1 == S ? 0 : buf + 1;
#pragma unroll
      for (int kk = 0; kk < 3; ++kk) {  // the fragments of the next k-step are requested before this one's MFMAs
        frags(st, kk + 1, (kk + 1) & 1);
        __builtin_amdgcn_sched_barrier(0);
        mma(kk & 1);
        __builtin_amdgcn_sched_barrier(0);
      }
      if (s + 1 < nsteps) {
        step_end(s);
        if (s + S < nsteps) issue(s + S, buf);
        frags(smem + bnext * kStage, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      }
      mma(1);  // (left in one place: a copy behind the loop costs the compiler a second set of accumulators)
      buf = bnext;
    }
  }

  // out, two column tiles at a time (their 64 channels of a row are a whole line, and the registers beside the accumulators
  // hold no more); one at a time where the wavefront's channels do not start on a multiple of 64, so that a slice lies on
  // one side of yt_from
  constexpr int SL = NT % 2 ? 1 : 2;
  const int c0 = n0 + wn * (32 * NT);
#pragma unroll
  for (int i = 0; i < NT; i += SL) {
    const int ci = c0 + 32 * i;
    float bias_l[SL], mul_l[SL];
#pragma unroll
    for (int e = 0; e < SL; ++e) {
      const int co = ci + 32 * e + lp;
      bias_l[e] = a.bias ? a.bias[co] : 0.f;
      mul_l[e] = co < a.q_cols ? a.q_scale : 1.f;
    }
#pragma unroll
    for (int j = 0; j < MT; ++j) {
      f32x16 part[SL];
#pragma unroll
      for (int e = 0; e < SL; ++e) part[e] = acc[j][i + e];
      lin_epilogue<OT, SL, false, true>(a, part, m0 + wm * (32 * MT) + 32 * j, ci, lane, bias_l, mul_l);
    }
  }
}

template <class OT, int WM, int WN, int MT, int NT, int S>
static hipError_t run_lin3_k(hipStream_t s, Lin2Args a) {
  constexpr int kM = 32 * WM * MT, kN = 32 * WN * NT, lds = S * (kM + kN) * kKB3;
  static_assert(lds <= 160 * 1024, "one workgroup's ring fits the LDS");
  auto kern = lin3_kernel<OT, WM, WN, MT, NT, S>;
  static bool done = false;  // per instantiation
  if (!done) {
    hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
    done = true;
  }
  if (a.N % kN || (int64_t)(kM > kN ? kM : kN) * a.K * 2 > 0x7fffffff) return hipErrorInvalidValue;  // (32-bit offsets in a tile)
  a.ntn = a.N / kN;
  a.ntm = (int)((a.rows + kM - 1) / kM);
  // Each XCD fetches what its tiles read into an L2 of its own, and for short contractions and few rows that traffic, from beyond
  // the L2, is what a launch waits for. Of the four ways to deal the tiles in blocks, the one with the fewest rounds of
  // workgroups on the fullest XCD, then the fewest rows and channels to fetch.
  constexpr int kRes = 32 * (2 * lds <= 160 * 1024 ? 2 : 1);  // workgroups resident on an XCD
  int64_t best = -1;
  for (int xm = 8; xm >= 1; xm /= 2) {
    const int bm = (a.ntm + xm - 1) / xm, bn = (a.ntn + 8 / xm - 1) / (8 / xm);
    const int64_t cost = ((int64_t)((bm * (int64_t)bn + kRes - 1) / kRes) << 40) + (int64_t)bm * kM + (int64_t)bn * kN;
    if (best < 0 || cost < best) { best = cost; a.xm = xm; a.bm = bm; a.bn = bn; }
  }
  kern<<<(unsigned)(8 * a.bm * a.bn), WM * WN * 64, lds, s>>>(a);
  return hipGetLastError();
}

// The tile of a dense launch. 256 compute units: a launch wants at least about that many workgroups, and the large tiles pay only
// where their last round is nearly full.
LinTile lin3_tile(const Lin2Args& a, bool y_f32) {
  auto tiles = [&](int m, int n) { return (a.rows + m - 1) / m * (a.N / n); };
  auto fills = [&](int64_t t) { return t >= 256 && t * 10 >= (t + 255) / 256 * 256 * 9; };
  if (a.N % 160 == 0 && a.act != 2 && !a.gate) {
    // 128 x 160 and 64 x 64, fp32 (tiles of the former). 320 channels, K = 320: 4096 rows (64) 8.1 and 5.6, 12288 (192) 12.0 and
    // 11.4, 16384 (256) 13.5 and 15.1; K = 1280: 2048 rows (32) 18 and 8, 16384 (256) 25 and 28. At 128 tiles the small ones are
    // level or ahead one launch after the other (8192 rows of 320, K = 320 9.7 and 9.7, K = 1280 21 and 18; 4096 of 640 13.3 and
    // 12.1) and nothing is gained among other kernels: the cache step of the U-Net at 256 x 256, which has them, 1329 and 1330
    // us, its normal step at 512 x 512 15.83 and 15.77 ms
    if (a.N % 64 == 0 && tiles(128, 160) < 128) return LinTile::k64x64;
    // (fp32 outputs stay: 32768 x 640 x 640 58 against 62 with 128 x 128, 32768 x 640 x 2560 131 against 143, 8192 x 1280 x 1280
    // 36 against 43, 131072 x 320 x 320 85 against 119 with 64 x 64)
    if (y_f32) return LinTile::k128x160;
    // 8192 x 3840 x 1280 86 with 128 x 160, 75 with 256 x 256; 131072 x 1280 x 320 207 and 172
    if (a.N % 256 == 0 && fills(tiles(256, 256))) return LinTile::k256x256;
    // 128 x 160 and 256 x 192: 131072 x 960 x 320 136 and 166, the larger tile's epilogue is not covered; 8192 x 2880 x 960 57 and 50,
    // 32768 x 2880 x 960 218 and 210, 65536 x 960 x 1280 189 and 189, 32768 x 1920 x 1280 184 and 188. At the line itself the smaller
    // one has come ahead since its epilogue has no condition per row (32768 x 1920 x 640 110 and 103 before, 109 and 118 now)
    if (a.N % 192 == 0 && a.K >= 640 && fills(tiles(256, 192))) return LinTile::k256x192;
    return LinTile::k128x160;
  }
  if (!y_f32) {
    // 8192 x 4096 x 1024 with GELU 76 with 128 x 128, 73 with 256 x 256; 8192 x 3072 x 1024 (384 tiles, the second round half empty)
    // 52 against 58, and 52 with 256 x 192. Short contractions too: with GEGLU 131072 x 2560 x 320 315 and 289, 65536 x 2560 x 320 158
    // and 151, 32768 x 5120 x 640 270 and 240, 8192 x 10240 x 1280 208 and 192 (their epilogue, two transcendentals for each value
    // that leaves, is uncovered in either)
    if (a.N % 256 == 0 && fills(tiles(256, 256))) return LinTile::k256x256;
    if (a.N % 192 == 0 && a.K >= 640 && a.act != 2 && fills(tiles(256, 192))) return LinTile::k256x192;
  }
  // 128 x 128 and 64 x 128 (tiles of the former): 1024 x 3072 x 1024 (192) 12.9 and 11.8, 1024 x 4096 x 1024 (256) 15.2 and 13.8,
  // 2048 x 2048 x 512 (256) 9.0 and 8.4, 4096 x 1024 x 1024 fp32 (256) 17.6 and 15.4, 1536 x 3072 x 768 (288) 14.5 and 15.3,
  // 3108 x 3072 x 1024 (600) 28.2 and 28.3, 6216 x 3072 x 1024 (1176) 45 and 53. GEGLU: 4096 x 2560 x 320 13.2 and 13.9, 2048 x
  // 5120 x 640 19.5 and 20.4
  if (tiles(128, 128) > 256 || a.act == 2) return LinTile::k128x128;
  // 64 x 128 and 64 x 64 (tiles of the former): 1024 x 4096 x 1024 (512) 13.8 and 16.6, 2048 x 2048 x 512 (512) 8.4 and 10.2, 1024 x
  // 3072 x 1024 (384) 11.8 and 13.2; 1024 x 1024 x 1024 fp32 (128) 9.0 and 7.5. Between the two the small ones are ahead by less since
  // they hold a stage in registers: 512 x 3072 x 1024 (192) 9.2 and 8.1, 640 x 3072 x 1024 (240) 9.2 and 8.4, 1024 x 2048 x 512 (256)
  // 6.5 and 5.9; fp32 1536 x 1024 x 1024 (192) 9.6 and 9.1, 1600 x 1024 x 4096 (200) 27 and 26
  return tiles(64, 128) >= 192 ? LinTile::k64x128 : LinTile::k64x64;
}

hipError_t launch_lin3(hipStream_t s, const Lin2Args& a, bool y_f32) {
  switch (lin3_tile(a, y_f32)) {
    case LinTile::k256x256: return run_lin3_k<bf16_t, 4, 2, 2, 4, 2>(s, a);  // (bf16 outputs only)
    case LinTile::k256x192: return run_lin3_k<bf16_t, 4, 2, 2, 3, 2>(s, a);
    case LinTile::k128x128: return y_f32 ? run_lin3_k<float, 2, 2, 2, 2, 2>(s, a) : run_lin3_k<bf16_t, 2, 2, 2, 2, 2>(s, a);
    case LinTile::k64x128: return y_f32 ? run_lin3_k<float, 2, 2, 1, 2, 3>(s, a) : run_lin3_k<bf16_t, 2, 2, 1, 2, 3>(s, a);
    case LinTile::k64x64: return y_f32 ? run_lin3_k<float, 2, 2, 1, 1, 4>(s, a) : run_lin3_k<bf16_t, 2, 2, 1, 1, 4>(s, a);
    case LinTile::k128x160: break;
  }
  return hipErrorNotSupported;
}

}  // namespace lc
