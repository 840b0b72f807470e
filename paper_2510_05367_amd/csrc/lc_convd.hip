// 3x3 stride-1 convolution of the bf16 stages over activations that are in memory already (gfx950): the rows that the
// contraction reads - SiLU(GroupNorm(x)), or x itself, rounded to bf16 - were written by a pass of their own
// (launch_conv_act), so nothing in this kernel touches a vector register on its way from memory to the matrix cores but
// the MFMA fragments: activations and weights go global -> LDS by buffer loads, whose bounds check delivers the zero
// padding, and the four wavefronts of a workgroup do nothing but fragment reads, MFMAs and requests.
//
// Why a pass of its own: a loader that activates on the way in (lc_convws.hip, lc_gemm.hip) does that work 1.4 times for the
// halo and once more per block of output channels, reads the fp32 rows as often, and needs four wavefronts and the LDS
// for it, so that one workgroup fills a compute unit and nothing covers its prologue and epilogue. Ablations of the
// specialised-wavefront kernel at 32 frames of 64 x 64, 320 channels: 323 us, without its loaders 265, without the
// residual and the stores 272, MFMAs and fragment reads alone 196.
//
// Product and order of the sums are those of the kernels named above (64-channel slab, tap, two k-steps of 16 in each of
// two halves of the slab, the halves added at the end): D[cout][pixel] on 32 x 32 x 16 MFMAs, a workgroup owns CO_T * 32
// channels x 128 pixels (an 8 x 16 tile of one frame), wavefront (pxh, kh) all of its channels x 64 pixels over half of K.
// All widths CO_T and those kernels agree bit for bit, so the width may follow the launch's size.
//
// LDS holds 80 KB at most, so that two workgroups share a compute unit and cover each other's waits:
//  * a ring of four to eight weight sub-steps (16 channels of both halves for one tap: 2 * CO_T fragments of 1 KB in fragment
//    order, as the weights are laid out at load time; reads are 1 KB in a row);
//  * a ring of 16 halo lines of 20 pixels x 64 channels (18 used; 16-byte slots XOR-swizzled by the pixel so that 16
//    consecutive pixels hit all banks). A slab has 10 lines. Lines 0..5 of the next slab lie in no line of this one, lines 6
//    and 7 where lines 0 and 1 of this one were, which its taps 6..8 no longer read, lines 8 and 9 where its lines 2 and 3
//    were: they are requested in the next slab's first sub-step and first read at its tap 3.
// A sub-step u: its fragments are in registers; those of u + 1 are read from LDS while its MFMAs are issued, the weights of
// u + ring are requested into the slot u had, and it ends with a wait for these reads and for the weights of u + 2 (and what
// was requested before them) and the workgroup's barrier.
// A lone workgroup of 160 channels on an idle chip takes 24 us for 90 sub-steps: 12 of MFMAs, 5 of everything else in the loop,
// 7 of launch, first loads and epilogue; 256 of them 34, the rest being the residual and the output (42 MB at the rate of a
// copy), which only a second workgroup per compute unit covers. Eight wavefronts of 32 pixels instead of four of 64 (two per
// SIMD also where a launch has one workgroup per compute unit) measured the same there and 20-40 % slower in larger launches.
#include <type_traits>

#include "lc_internal.h"

namespace lc {

namespace {

constexpr int kdLines = 16;      // halo lines in LDS
constexpr int kdLine = 20 * 128; // bytes of a halo line
constexpr int kdSub = 18;        // sub-steps of a slab: 9 taps x 2
constexpr int kdRawBuffer = 0x00020000;  // buffer descriptor word 3: raw bytes, 32-bit data format

struct ConvDArgs {
  const bf16_t* x;   // channels [0, Cs): rows [frames][H][W][Cs], or at half the resolution if `up`
  const bf16_t* x2;  // channels [Cs, Cin): rows [frames][H/2][W/2][Cin - Cs], or nullptr
  const bf16_t* w;   // fragments [9 * Cin / 32][2][Cout / 32][64][8]
  const float* bias;  // of frame f: bias + (bias_f0 + f) / bias_div * Cout; or nullptr
  const float* res;  // fp32, indexed like y, or nullptr
  void* y;           // [frames][H][W][Cout], fp32 or bf16
  int Cin, Cs, Cout, up, bias_div, bias_f0;
  int H, W, tiles_x, tiles_y, ntiles, ncb;
  float* stat;
  int stat_splits;
};

// weight sub-steps in LDS: as many as fit beside the halo lines. Narrow workgroups have short sub-steps and need more of them
// in flight to cover a request's way from L2 (us; two tiles, 4 frames of 64 x 64, 320 channels: 41.7 with a ring of four, 35.4
// with eight; three tiles, a frame of 256 x 256, 192 channels: 51.3 with four, 46.9 with six)
template <int CO_T> constexpr int cd_ring() { return CO_T == 2 ? 8 : CO_T == 3 ? 6 : 4; }
template <int CO_T> constexpr int cd_lds_bytes() { return cd_ring<CO_T>() * 2 * CO_T * 1024 + kdLines * kdLine; }
// tiles handed over at a time in the epilogue: their fp32 values of four wavefronts and the four patches must fit
template <int CO_T> constexpr int cd_give() {
  int g = CO_T;
  while (4 * g * 4096 + 4 * 32 * 36 * 4 > cd_lds_bytes<CO_T>()) --g;
  return g;
}

// Requests that every wavefront has issued (one of them a fifth instruction for a pair of halo lines, some the extra weight
// fragment of an odd width: these wait for a little more than they need to). Weights of n sub-steps in a row:
constexpr int cd_weights(int n, int cot) { return n / 2 * cot + n % 2 * (cot / 2); }
// halo lines in sub-step t of a slab
constexpr int cd_halo(int t, bool more) { return t == 0 || (more && (t == 2 || t == 4 || t == 6 || t == 12)) ? 1 : 0; }
// Requests that may be in flight at the end of sub-step t: all that are younger than the weights of t + 2, which were requested
// ring - 2 sub-steps ago (a slab begins with the last halo lines of the one before landed); and at the end of sub-steps 4 and 16 all that are younger than the halo lines requested in 0 and 12,
// which are read from the next sub-step but one on
constexpr int cd_keep(int t, bool more, int cot, int ring) {
  int n = more ? ring - 2 : kdSub - 3 - t < ring - 2 ? kdSub - 3 - t : ring - 2;
  int k = cd_weights(n > 0 ? n : 0, cot);
  for (int q = t + 3 - ring > 0 ? t + 3 - ring : 0; q <= t; ++q) k += cd_halo(q, more);
  if (t == 4 || (t == 16 && more)) {
    int h = 0, m = 0;
    for (int q = t - 4; q <= t; ++q) {
      m += more || q + ring < kdSub;
      if (q > t - 4) h += cd_halo(q, more);
    }
    const int k2 = cd_weights(m, cot) + h;
    k = k2 < k ? k2 : k;
  }
  return k;
}

// the sum over the eight lanes that are equal modulo 8, in all of them: by lane distances 8, 16, 32, without LDS
__device__ __forceinline__ float fold8(float x) {
  const int i = __builtin_bit_cast(int, x);
  x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, i, 0x128, 0xf, 0xf, true));  // row_ror:8
  auto r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(unsigned, x), __builtin_bit_cast(unsigned, x), false, false);
  x = __builtin_bit_cast(float, (unsigned)r[0]) + __builtin_bit_cast(float, (unsigned)r[1]);
  r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, x), __builtin_bit_cast(unsigned, x), false, false);
  return __builtin_bit_cast(float, (unsigned)r[0]) + __builtin_bit_cast(float, (unsigned)r[1]);
}

}  // namespace

template <int CO_T, class OT>
__global__ __launch_bounds__(256, 2) void conv_dma_kernel(ConvDArgs a) {
  typedef Mma32<bf16_t> M;
  constexpr int kSlot = 2 * CO_T * 1024;
  constexpr int kRing = cd_ring<CO_T>();
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  unsigned char* const hl = smem + kRing * kSlot;

  const int lane = threadIdx.x & 63, wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lp = lane & 31, hh = lane >> 5;
  const int pxh = wid & 1, kh = wid >> 1;
  // the channel blocks of a tile run one after another on one XCD (workgroups go round the eight), whose L2 then has the tile
  int t0 = (int)blockIdx.x >> 3;
  const int cb = t0 % a.ncb;
  t0 = (t0 / a.ncb) * 8 + ((int)blockIdx.x & 7);
  if (t0 >= a.ntiles) return;
  const int tx0 = (t0 % a.tiles_x) * 16;
  const int ty0 = (t0 / a.tiles_x) % a.tiles_y * 8;
  const int frame = t0 / (a.tiles_x * a.tiles_y);
  const int nslab = a.Cin >> 6, ct = a.Cout >> 5;

  // ---- requests: halo lines. A pair of lines is 320 packets of 16 bytes: instruction k < 4 by wavefront k, the fifth by one of
  // them. hofs: this lane's byte offset for pair 0 of the source at hand; a pixel beyond the left or right edge
  // (or of the two spare ones) gets an offset that stays out of range, lines above and below the frame are out of range anyway
  __amdgpu_buffer_rsrc_t hsrc;
  unsigned hofs[2], hadv;  // hadv: bytes from pair to pair
  auto source = [&](const bf16_t* x, int C, int up) {
    const int Ws = a.W >> up, Hs = a.H >> up;
    hsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(x) + (int64_t)frame * Hs * Ws * C, 0, Hs * Ws * C * 2, kdRawBuffer);
    hadv = (unsigned)((up ? Ws : 2 * Ws) * C * 2);
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int e = (q ? 4 : wid) * 64 + lane;
      const int l = e / 160, px = (e - l * 160) >> 3, pk = (e & 7) ^ ((px >> 1) & 7);
      const int ix = tx0 - 1 + px;
      const int iy = up ? (ty0 >> 1) - 1 + l : ty0 - 1 + l;
      const bool ok = px < 18 && ix >= 0 && ix < a.W;
      hofs[q] = ok ? (unsigned)((iy * Ws + (ix >> up)) * C * 2 + pk * 16) : 0x80000000u;
    }
  };
  // lines 2 p, 2 p + 1 of slab `slab`, whose channels start `cofs` bytes into the source's rows
  auto halo = [&](int slab, int p, int cofs) {
#ifdef __HIP_DEVICE_COMPILE__
    unsigned char* dst = hl + ((10 * slab + 2 * p) & (kdLines - 1)) * kdLine;
    const unsigned adv = p * hadv + cofs;
    __builtin_amdgcn_raw_ptr_buffer_load_lds(hsrc, dst + wid * 1024, 16, hofs[0] + adv, 0, 0, 0);
    if (wid == (p & 3)) __builtin_amdgcn_raw_ptr_buffer_load_lds(hsrc, dst + 4096, 16, hofs[1] + adv, 0, 0, 0);
#endif
  };
  // ---- requests: weights of sub-step u. Fragment f = kh' * CO_T + i. A wavefront takes every fourth one, and the two left over
  // of an odd CO_T go to two wavefronts in even and to the other two in odd sub-steps: CO_T requests each in any two in a row
  constexpr bool ODD = CO_T & 1;
  constexpr int WJ = (CO_T + 1) / 2;  // requests per sub-step; the last one of an odd CO_T not of every wavefront
  auto wfrag = [&](int j) { return ODD && j + 1 == WJ ? j * 4 + (wid & 1) : j * 4 + wid; };
  const __amdgpu_buffer_rsrc_t wsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(a.w), 0, a.Cin * 9 * a.Cout * 2, kdRawBuffer);
  const unsigned wofs = lane * 16;
  int wsub[WJ];  // byte offsets in a sub-step's fragments of all channels
#pragma unroll
  for (int j = 0; j < WJ; ++j) {
    const int f = wfrag(j);
    wsub[j] = ((f >= CO_T ? ct - CO_T : 0) + cb * CO_T + f) * 1024;
  }
  const int wadv = 2 * ct * 1024;
  // request j of the sub-step at source offset uofs into ring offset slot; odd: of the sub-step's number
  auto wreq = [&](int uofs, int slot, int j, int odd) {
#ifdef __HIP_DEVICE_COMPILE__
    if (!ODD || j + 1 < WJ || (wid >> 1) == odd)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(wsrc, smem + slot + wfrag(j) * 1024, 16, wofs, uofs + wsub[j], 0, 0);
#else
    (void)uofs; (void)slot; (void)j; (void)odd; (void)wofs; (void)wsrc;
#endif
  };

  f32x16 acc[CO_T][2];
#pragma unroll
  for (int i = 0; i < CO_T; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  // Tile column 0 of the accumulators is the one this wavefront finishes after the K halves are folded, column 1 the one
  // its partner of the other half finishes: which 32 pixels (two image rows) that is depends on kh, the code does not.
  const int quarter = pxh * 2 + kh;  // the 32 pixels of column 0
  const int ly[2] = {quarter * 2 + (lp >> 4), (quarter ^ 1) * 2 + (lp >> 4)};
  unsigned xofs[3];  // of k-step 0 for dx = 0..2; k-step 1 is 2 packets on: offset ^ 32
#pragma unroll
  for (int dx = 0; dx < 3; ++dx) {
    const int px = (lp & 15) + dx;
    xofs[dx] = px * 128 + (((kh * 4 + hh) ^ ((px >> 1) & 7)) << 4);
  }
  const unsigned wrd = kh * CO_T * 1024 + lane * 16;
  auto wread = [&](int slot, int i) { return M::load((const bf16_t*)(smem + (slot + wrd) + i * 1024)); };
  auto xread = [&](int slab, int t, int j) {  // sub-step t of slab `slab`
    const int tap = t >> 1, dy = tap / 3, dx = tap - dy * 3;
    const unsigned line = (unsigned)(10 * slab + dy + ly[j]) & (kdLines - 1);
    return M::load((const bf16_t*)(hl + line * kdLine + ((t & 1) ? xofs[dx] ^ 32u : xofs[dx])));
  };
  // at most VM requests and no LDS read of this wavefront in flight, then the barrier
  auto step_end = [&](auto vm_c) { barrier_keep<decltype(vm_c)::value>(); };

  // ---- prologue
  source(a.x, a.Cs, a.up);
#pragma unroll
  for (int p = 0; p < 4; ++p) halo(0, p, 0);
#pragma unroll
  for (int u = 0; u < kRing; ++u)
#pragma unroll
    for (int j = 0; j < WJ; ++j) wreq(u * wadv, u * kSlot, j, u & 1);
  barrier_keep<cd_weights(kRing - 2, CO_T)>();  // the weights of sub-steps 0 and 1 and lines 0..7 have landed
  M::Frag w[CO_T], x[2];
#pragma unroll
  for (int i = 0; i < CO_T; ++i) w[i] = wread(0, i);
  x[0] = xread(0, 0, 0);
  x[1] = xread(0, 0, 1);
  barrier_keep<cd_weights(kRing - 2, CO_T)>();

  const int nskip = a.Cs >> 6;
  int slot = 0;             // ring offset of the current sub-step, whose fragments are in registers: the weights of the kRing-th
  int uofs = kRing * wadv;  // one from here go there, from this offset of the source
  auto slab_body = [&](int slab, auto more_c) {
    constexpr bool MORE = decltype(more_c)::value;
    auto cofs = [&](int s) { return (s < nskip ? s : s - nskip) * 128; };
    auto sub = [&](auto t_c) {
      constexpr int t = decltype(t_c)::value;
      M::Frag wn[CO_T], xn[2];
      constexpr bool NEXT = MORE || t + 1 < kdSub;
      const int rd = slot + kSlot == kRing * kSlot ? 0 : slot + kSlot;  // where the weights of the next sub-step are
      if (MORE && t == 1)
        if (slab + 1 == nskip) source(a.x2, a.Cin - a.Cs, 1);
      // one request or fragment read behind each MFMA: several in a row hold the next MFMA up
#pragma unroll
      for (int g = 0; g < 2 * CO_T; ++g) {
        if (NEXT && g < CO_T + 2) {
          const int ns = t + 1 < kdSub ? slab : slab + 1, nt = t + 1 < kdSub ? t + 1 : 0;
          if (g < 2) xn[g] = xread(ns, nt, g);
          else wn[g - 2] = wread(rd, g - 2);
        }
        __builtin_amdgcn_sched_barrier(0);
        M::mma(w[g >> 1], x[g & 1], acc[g >> 1][g & 1]);
        __builtin_amdgcn_sched_barrier(0);
        if (g == 0) {
          if (t == 0) halo(slab, 4, cofs(slab));
          if (MORE && t == 2) halo(slab + 1, 0, cofs(slab + 1));
          if (MORE && t == 4) halo(slab + 1, 1, cofs(slab + 1));
          if (MORE && t == 6) halo(slab + 1, 2, cofs(slab + 1));
          if (MORE && t == 12) halo(slab + 1, 3, cofs(slab + 1));
        }
#pragma unroll
        for (int j = 0; j < WJ; ++j)
          if (g == 2 * CO_T - WJ + j && (MORE || t + kRing < kdSub)) wreq(uofs, slot, j, t & 1);
        __builtin_amdgcn_sched_barrier(0);
      }
      uofs += wadv;
      slot = rd;
      if (NEXT) {
        step_end(std::integral_constant<int, cd_keep(t, MORE, CO_T, kRing)>{});
#pragma unroll
        for (int i = 0; i < CO_T; ++i) w[i] = wn[i];
        x[0] = xn[0];
        x[1] = xn[1];
      }
    };
#define LC_SUB(T) sub(std::integral_constant<int, T>{});
    LC_SUB(0) LC_SUB(1) LC_SUB(2) LC_SUB(3) LC_SUB(4) LC_SUB(5) LC_SUB(6) LC_SUB(7) LC_SUB(8)
    LC_SUB(9) LC_SUB(10) LC_SUB(11) LC_SUB(12) LC_SUB(13) LC_SUB(14) LC_SUB(15) LC_SUB(16) LC_SUB(17)
#undef LC_SUB
  };
  for (int slab = 0; slab + 1 < nslab; ++slab) slab_body(slab, std::true_type{});
  slab_body(nslab - 1, std::false_type{});

  // ---- fold the two K halves and write out: column 1 goes to the partner through LDS (every read of the rings is done, see
  // the barrier of the last sub-step but one, and no request is in flight), each finished 32 x 32 tile is turned
  // through a private patch so that eight lanes store 128 contiguous bytes of a pixel; as many tiles at a time as fit
  constexpr int G = cd_give<CO_T>();
  constexpr int kTile = 16 * 64;
  float* give = reinterpret_cast<float*>(smem) + quarter * (G * kTile);
  const float* take = reinterpret_cast<const float*>(smem) + (quarter ^ 1) * (G * kTile);
  float* patch = reinterpret_cast<float*>(smem + 4 * G * kTile * 4) + quarter * (32 * 36);
  const int prow = lane >> 3, pcol = (lane & 7) * 4;  // patch read-back: rows prow + 8 k, channels pcol..pcol+3
  const int co0 = cb * CO_T * 32;
  // Output and residual through buffer descriptors over the tile's eight image rows: a pixel beyond the edge has an offset out
  // of range, whose load gives zero and whose store is dropped, so neither needs a condition per pixel. No scalar offsets: the
  // range check takes them off the size first, and without a residual that is zero
  const int64_t row0 = ((int64_t)frame * a.H + ty0) * a.W * a.Cout + co0;
  const int rows8 = 8 * a.W * a.Cout;
  const __amdgpu_buffer_rsrc_t ydst = __builtin_amdgcn_make_buffer_rsrc((OT*)a.y + row0, 0, rows8 * (int)sizeof(OT), kdRawBuffer);
  const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(a.res) + (a.res ? row0 : 0), 0, a.res ? rows8 * 4 : 0, kdRawBuffer);
  unsigned opix[4];  // element offset of this lane's channels of pixel k
  bool okk[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int p = quarter * 32 + prow + 8 * k;
    const int dy = p >> 4, ox = tx0 + (p & 15);
    okk[k] = ty0 + dy < a.H && ox < a.W;
    opix[k] = (dy * a.W + ox) * a.Cout + pcol;
  }
  const float* bias = a.bias ? a.bias + (int64_t)((a.bias_f0 + frame) / a.bias_div) * a.Cout : nullptr;
  typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
  typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
  auto far = [&](int k, unsigned bytes) { return okk[k] ? bytes : 0x80000000u; };
  struct Side { f32x4 r[4]; f32x4 b; };
#pragma unroll
  for (int i0 = 0; i0 < CO_T; i0 += G) {
    if (i0) __syncthreads();  // the partner has read the tiles before
#pragma unroll
    for (int i = i0; i < i0 + G && i < CO_T; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) give[((i - i0) * 16 + r) * 64 + lane] = acc[i][1][r];
    asm volatile("" ::: "memory");  // (the requests stay below the hand-over: above it they would not fit)
    Side side[G];
#pragma unroll
    for (int i = i0; i < i0 + G && i < CO_T; ++i) {
      side[i - i0].b = bias ? *reinterpret_cast<const f32x4*>(bias + co0 + i * 32 + pcol) : f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int k = 0; k < 4; ++k)
        side[i - i0].r[k] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, far(k, opix[k] * 4) + i * 128, 0, 0));
    }
    barrier_keep<63>();
#pragma unroll
    for (int i = i0; i < i0 + G && i < CO_T; ++i) {
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        f32x4 v;
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = acc[i][0][g * 4 + e] + take[((i - i0) * 16 + g * 4 + e) * 64 + lane];
        *reinterpret_cast<f32x4*>(patch + lp * 36 + g * 8 + hh * 4) = v;
      }
      // the patch is private to this wavefront, whose LDS operations complete in order
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      float ssum[4] = {0.f, 0.f, 0.f, 0.f}, ssq[4] = {0.f, 0.f, 0.f, 0.f};  // statistics of this lane's pixels
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        f32x4 v = *reinterpret_cast<const f32x4*>(patch + (prow + 8 * k) * 36 + pcol);
        v += side[i - i0].b;
        v += side[i - i0].r[k];
        if constexpr (sizeof(OT) == 4) {
          __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), ydst, far(k, opix[k] * 4) + i * 128, 0, 0);
        } else {
          bf16x4 o;
#pragma unroll
          for (int e = 0; e < 4; ++e) o[e] = (bf16_t)v[e];
          __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, o), ydst, far(k, opix[k] * 2) + i * 64, 0, 0);
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float t = okk[k] ? v[e] : 0.f;
          ssum[e] += t;
          ssq[e] = fmaf(t, t, ssq[e]);
        }
      }
      if (a.stat) {
        // fold the eight lanes that hold the same channels, in a fixed order; the first writes. One split = these 32 pixels
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          ssum[e] = fold8(ssum[e]);
          ssq[e] = fold8(ssq[e]);
        }
        if (prow == 0) {
          const int split = ((ty0 >> 3) * a.tiles_x + (tx0 >> 4)) * 4 + quarter;
          float* sp = a.stat + (((int64_t)frame * a.stat_splits + split) * a.Cout + co0 + i * 32 + pcol) * 2;
          *reinterpret_cast<f32x4*>(sp) = f32x4{ssum[0], ssq[0], ssum[1], ssq[1]};
          *reinterpret_cast<f32x4*>(sp + 4) = f32x4{ssum[2], ssq[2], ssum[3], ssq[3]};
        }
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
    }
  }
}

template <int CO_T, class OT>
static hipError_t run_convd(hipStream_t s, ConvDArgs a) {
  constexpr int lds = cd_lds_bytes<CO_T>();
  static_assert(lds <= 80 * 1024, "two workgroups per compute unit");
  auto kern = conv_dma_kernel<CO_T, OT>;
  static bool attr_done = false;  // per instantiation
  if (!attr_done) {
    hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
    attr_done = true;
  }
  a.ncb = a.Cout / (CO_T * 32);
  const unsigned grid = (unsigned)((a.ntiles + 7) / 8 * 8 * a.ncb);
  kern<<<grid, 256, lds, s>>>(a);
  return hipGetLastError();
}

// Channel tiles per workgroup. Widest first: a wider workgroup reads less per MFMA, and two share a compute unit. Launches that
// would not fill the chip with those (up to 512 workgroups of two tiles are resident at once) take two: 320 channels at
// 3 frames of 36 x 60 27.8 us with five and 22.1 with two, one frame of 64 x 64 25.9 and 15.2, two 28.2 and 22.6; 4 frames of
// 64 x 64 (640 workgroups of two) 33.8 and 35.4, with 960 input channels 82 and 86, 32 frames 227 and 249.
static int conv_dma_tiles(int64_t ntiles, int ct) {
  if (ct % 2 == 0 && ntiles * (ct / 2) <= 512) return 2;
  for (int w = 5; w >= 2; --w)
    if (ct % w == 0) return w;
  return 0;
}

hipError_t launch_conv_dma(hipStream_t s, const FusedDesc& d) {
  if (d.dt != kBF16 || d.taps != 9 || (d.src != 0 && d.src != 3) || d.planar_out || d.yt || d.q_cols || d.win_w || d.general)
    return hipErrorNotSupported;
  if (d.Cin % 64 || d.Cout % 64 || d.Cout_store != d.Cout || d.Cin <= 0 || d.Cout <= 0) return hipErrorNotSupported;
  if (d.src == 3 && (d.up2 || d.Cs % 64 || d.Cs <= 0 || d.Cs >= d.Cin || ((d.H | d.W) & 1))) return hipErrorInvalidValue;
  if (d.up2 && ((d.H | d.W) & 1)) return hipErrorInvalidValue;
  if (d.stat && (!d.y_f32 || d.stat_splits != conv_stat_splits(d.H, d.W))) return hipErrorInvalidValue;
  if (d.bias_div < 0 || d.bias_f0 < 0) return hipErrorInvalidValue;
  // 31-bit byte offsets inside a frame, inside the weights and inside eight image rows of the output
  if ((int64_t)8 * d.W * d.Cout * 4 >= (int64_t)1 << 31) return hipErrorNotSupported;
  if ((int64_t)d.H * d.W * d.Cin * 2 >= (int64_t)1 << 31 || (int64_t)d.Cout * 9 * d.Cin * 2 >= (int64_t)1 << 31) return hipErrorNotSupported;
  if (d.frames <= 0) return hipSuccess;
  ConvDArgs a;
  a.x = (const bf16_t*)d.x; a.x2 = (const bf16_t*)d.x2; a.w = (const bf16_t*)d.w; a.bias = d.bias; a.res = (const float*)d.res; a.y = d.y;
  a.Cin = d.Cin; a.Cs = d.src == 3 ? d.Cs : d.Cin; a.Cout = d.Cout; a.up = d.up2;
  a.bias_div = d.bias_div ? d.bias_div : 1 << 30; a.bias_f0 = d.bias_div ? d.bias_f0 : 0;
  a.H = d.H; a.W = d.W; a.tiles_x = (d.W + 15) / 16; a.tiles_y = (d.H + 7) / 8;
  a.stat = d.stat; a.stat_splits = d.stat_splits;
  const int64_t ntiles = (int64_t)a.tiles_x * a.tiles_y * d.frames;
  if (ntiles * (d.Cout / 32) >= (int64_t)1 << 30) return hipErrorNotSupported;
  a.ntiles = (int)ntiles; a.ncb = 0;
  const int ct = d.Cout / 32;
  switch (conv_dma_tiles(ntiles, ct)) {
    case 5: return d.y_f32 ? run_convd<5, float>(s, a) : run_convd<5, bf16_t>(s, a);
    case 4: return d.y_f32 ? run_convd<4, float>(s, a) : run_convd<4, bf16_t>(s, a);
    case 3: return d.y_f32 ? run_convd<3, float>(s, a) : run_convd<3, bf16_t>(s, a);
    case 2: return d.y_f32 ? run_convd<2, float>(s, a) : run_convd<2, bf16_t>(s, a);
  }
  return hipErrorNotSupported;
}

hipError_t launch_conv_act_dma(hipStream_t s, const FusedDesc& d) {
  if (d.src < 1 || d.src > 3 || (d.src == 1 && !d.unit_scale) || !d.xact || d.xact_bytes < conv_act_bytes(d)) return hipErrorNotSupported;
  FusedDesc c = d;
  c.x = d.xact; c.frames = 0;
  c.src = d.src == 3 ? 3 : 0;
  const hipError_t ok = launch_conv_dma(s, c);  // (no frames: says whether the shape is covered)
  if (ok != hipSuccess) return ok;
  c.frames = d.frames;
  const int T = d.H * d.W;
  hipError_t e;
  if (d.src == 3) {
    char* deep = (char*)d.xact + (size_t)d.frames * T * d.Cs * 2;
    c.x2 = deep;
    e = launch_conv_act(s, kF32, d.x, d.Cs, nullptr, 0, d.scale, d.shift, d.Cin, d.xact, d.frames, T);
    if (e == hipSuccess)
      e = launch_conv_act(s, kBF16, d.x2, d.Cin - d.Cs, nullptr, 0, d.scale + d.Cs, d.shift + d.Cs, d.Cin, deep, d.frames, T / 4);
  } else if (d.src == 2) {
    e = launch_conv_act(s, kF32, d.x, d.Cin, nullptr, 0, d.scale, d.shift, d.Cin, d.xact, d.frames, T);
  } else {  // (a unit scale: the rows are only rounded)
    e = launch_conv_act(s, kF32, d.x, d.Cin, nullptr, 0, nullptr, nullptr, 0, d.xact, d.frames, d.up2 ? T / 4 : T);
  }
  return e == hipSuccess ? launch_conv_dma(s, c) : e;
}

}  // namespace lc
