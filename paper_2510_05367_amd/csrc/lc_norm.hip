// GroupNorm statistics on channels-last activations.
//
// GroupNorm over a frame is done as: (1) per-channel partial sums over blocks of rows (one 16-byte
// packet per lane, coalesced over the channel axis), (2) a tiny kernel that folds the partials of
// whole groups into per-frame, per-channel scale/shift. The apply step (with SiLU, and for the up
// block with the 2x upsampling and skip-concatenation) lives in the loaders of the kernels that
// consume the normalised tensor. The split geometry depends only on the frame size, never on the
// chunking, so chunked and unchunked runs reduce in the same order.
#include "lc_internal.h"

namespace lc {

// ---------------------------------------------------------------------------------------------
template <class T>
__global__ __launch_bounds__(256) void gn_stats_kernel(const T* __restrict__ x, float* __restrict__ partial,
                                                       int rows_per_frame, int C) {
  constexpr int VEC = Vec16<T>::N;
  __shared__ float red[2][256 * VEC];
  // a workgroup covers up to 256 packets of the channel axis; wider tensors take gridDim.z of them side by side
  const int cv0 = blockIdx.z * 256;
  const int cv = min(C / VEC - cv0, 256);
  const int R = 256 / cv;
  const int split = blockIdx.x, frame = blockIdx.y, splits = gridDim.x;
  const int tid = threadIdx.x;
  const int cvec = tid % cv, rsub = tid / cv;
  float s[VEC], q[VEC];
#pragma unroll
  for (int i = 0; i < VEC; ++i) s[i] = q[i] = 0.f;
  const int r0 = split * kStatRows;
  const int r1 = min(r0 + kStatRows, rows_per_frame);
  if (rsub < R) {
    const T* base = x + ((int64_t)frame * rows_per_frame) * C + (cv0 + cvec) * VEC;
    for (int r = r0 + rsub; r < r1; r += R) {
      Vec16<T> v = load16(base + (int64_t)r * C);
#pragma unroll
      for (int i = 0; i < VEC; ++i) {
        float f = v.get(i);
        s[i] += f;
        q[i] = fmaf(f, f, q[i]);
      }
    }
  }
#pragma unroll
  for (int i = 0; i < VEC; ++i) {
    red[0][tid * VEC + i] = s[i];
    red[1][tid * VEC + i] = q[i];
  }
  __syncthreads();
  // channel c of row-slot j sits at red[.][(j*cv)*VEC + c]
  for (int c = tid; c < cv * VEC; c += 256) {
    float ss = 0.f, qq = 0.f;
    for (int j = 0; j < R; ++j) {
      ss += red[0][j * cv * VEC + c];
      qq += red[1][j * cv * VEC + c];
    }
    float* p = partial + (((int64_t)frame * splits + split) * C + cv0 * VEC + c) * 2;
    p[0] = ss;
    p[1] = qq;
  }
}

hipError_t launch_gn_stats(hipStream_t s, int dt, const void* x, float* partial, int frames,
                           int rows_per_frame, int C) {
  if (frames <= 0) return hipSuccess;
  const int vec = dt == kBF16 ? 8 : 4;
  if (C <= 0 || C % vec) return hipErrorInvalidValue;
  dim3 grid(stat_splits(rows_per_frame), frames, (C / vec + 255) / 256);
  if (dt == kBF16)
    gn_stats_kernel<bf16_t><<<grid, 256, 0, s>>>((const bf16_t*)x, partial, rows_per_frame, C);
  else
    gn_stats_kernel<float><<<grid, 256, 0, s>>>((const float*)x, partial, rows_per_frame, C);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// One workgroup folds the partial sums of one group of one frame. The group's (split, channel) cells are dealt to the
// threads in a fixed pattern, each thread adds its cells in double precision in a fixed order, and the results are folded by
// a fixed tree: the result does not depend on scheduling. The tensor may be the concatenation of two sources (A then B along
// the channels) with different row counts per frame; `w` weighs a source's rows (the 2x-upsampled deep feature
// counts each of its pixels four times).
// What it waits for are its loads: two channels a load where the group lies so (V = 2), kBatch of them in flight, no division
// per load, and 1024 threads where there are many splits (a 512 x 512 frame has 8192: 48 us with 256 threads, one channel a
// load and a division for each).
// At most 32 vector registers: it starts beside what another stream has running instead of waiting for a compute unit to drain.
template <int V>
__global__ __launch_bounds__(1024) __attribute__((amdgpu_num_vgpr(32))) void gn_finalize_kernel(const float* __restrict__ partA, int CA, int splitsA,
                                                          int rowsA, float wA, const float* __restrict__ partB,
                                                          int CB, int splitsB, int rowsB, float wB,
                                                          const float* __restrict__ gamma,
                                                          const float* __restrict__ beta, int groups, float eps,
                                                          float* __restrict__ scale, float* __restrict__ shift) {
  typedef float __attribute__((ext_vector_type(2 * V))) vec;
  __shared__ double rs[16], rq[16];
  __shared__ float s_mean, s_rstd;
  const int g = blockIdx.x, f = blockIdx.y, tid = threadIdx.x, nt = blockDim.x;
  const int Ct = CA + CB, cg = Ct / groups;
  const int c_lo = g * cg;
  // channels of the group that lie in A / in B
  const int nA = max(0, min(c_lo + cg, CA) - c_lo), nB = cg - nA;
  double ss = 0.0, qq = 0.0;
  // cells i = tid, tid + nt, ... in batches of kBatch: all loads of a batch are requested before the first is added
  constexpr int kBatch = 3;
  auto fold = [&](const float* part, int C, int splits, int n, int c_first, float w) {
    const int per = n / V, cells = per * splits;  // loads per split, in all
    const float* base = part + ((int64_t)f * splits * C + c_first) * 2;
    int k = tid / per, j = tid - k * per;
    const int dk = nt / per, dj = nt - dk * per;
    for (int i = tid; i < cells; i += nt * kBatch) {
      vec v[kBatch];
#pragma unroll
      for (int b = 0; b < kBatch; ++b) {
        const int kk = min(k, splits - 1);  // (beyond the end: a valid cell, not added)
        v[b] = *reinterpret_cast<const vec*>(base + ((int64_t)kk * C + j * V) * 2);
        k += dk;
        j += dj;
        if (j >= per) { j -= per; ++k; }
      }
#pragma unroll
      for (int b = 0; b < kBatch; ++b) {
        if (i + nt * b < cells) {
#pragma unroll
          for (int e = 0; e < V; ++e) {
            ss += (double)w * (double)v[b][2 * e];
            qq += (double)w * (double)v[b][2 * e + 1];
          }
        }
      }
    }
  };
  if (nA > 0) fold(partA, CA, splitsA, nA, c_lo, wA);
  if (nB > 0) fold(partB, CB, splitsB, nB, max(c_lo, CA) - CA, wB);
#pragma unroll
  for (int m = 32; m > 0; m >>= 1) {
    ss += __shfl_xor(ss, m, 64);
    qq += __shfl_xor(qq, m, 64);
  }
  if ((tid & 63) == 0) {
    rs[tid >> 6] = ss;
    rq[tid >> 6] = qq;
  }
  __syncthreads();
  if (tid == 0) {
#pragma unroll 1  // (registers)
    for (int i = 1; i < nt / 64; ++i) {
      ss += rs[i];
      qq += rq[i];
    }
    const double cnt = (double)nA * rowsA * wA + (double)nB * rowsB * wB;
    const double mean = ss / cnt;
    double var = qq / cnt - mean * mean;
    if (var < 0.0) var = 0.0;
    s_mean = (float)mean;
    s_rstd = (float)(1.0 / sqrt(var + (double)eps));
  }
  __syncthreads();
  for (int j = tid; j < cg; j += nt) {
    const int c = c_lo + j;
    const float a = s_rstd * gamma[c];
    scale[(int64_t)f * Ct + c] = a;
    shift[(int64_t)f * Ct + c] = fmaf(-s_mean, a, beta[c]);
  }
}

hipError_t launch_gn_finalize(hipStream_t s, const float* partA, int CA, int splitsA, int rowsA, float wA,
                              const float* partB, int CB, int splitsB, int rowsB, float wB,
                              const float* gamma, const float* beta, int groups, float eps, float* scale,
                              float* shift, int frames) {
  if (frames <= 0) return hipSuccess;
  if (groups <= 0 || (CA + CB) % groups) return hipErrorInvalidValue;
  const int cg = (CA + CB) / groups;
  if (cg <= 0) return hipErrorInvalidValue;
  // two channels a load: every group's channels of A and of B are pairs on 16-byte boundaries
  const bool pairs = cg % 2 == 0 && CA % 2 == 0 && CB % 2 == 0 && ((uintptr_t)partA | (uintptr_t)partB) % 16 == 0;
  const int64_t cells = (int64_t)cg * (splitsA > splitsB ? splitsA : splitsB) / (pairs ? 2 : 1);
  const dim3 grid(groups, frames);
  // (1024 threads where 256 would take more than two batches; us: 32 x 1 groups, 4 channels: 8192 splits 48 -> 12)
  const int nt = cells > 1536 ? 1024 : 256;
#define LC_FIN(V) \
  gn_finalize_kernel<V><<<grid, nt, 0, s>>>(partA, CA, splitsA, rowsA, wA, partB, CB, splitsB, rowsB, wB, gamma, beta, groups, eps, scale, shift)
  if (pairs) LC_FIN(2);
  else LC_FIN(1);
#undef LC_FIN
  return hipGetLastError();
}

// y[r][:] = bf16(x[m(r)][:] * scale[f][:] + shift[f][:]), f = r / rows_per_frame: GroupNorm applied to fp32 rows and
// rounded once, the operand of the projection into a transformer block. Thread = 8 channels of one row.
// MAPPED: the dense rows are gathered through the row map (a chunk of positions out of every frame).
template <bool MAPPED>
__global__ __launch_bounds__(256) void gn_apply_kernel(const float* __restrict__ x, const float* __restrict__ scale,
                                                       const float* __restrict__ shift, bf16_t* __restrict__ y, int64_t rows,
                                                       int C8, int rows_per_frame, RowMap m) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= rows * C8) return;
  const int64_t r = i / C8;
  const int c = (int)(i - r * C8) * 8;
  const int64_t f = r / rows_per_frame;
  const int64_t sr = MAPPED ? m(r) : r;
  float v[8], sc[8], sh[8];
  load_f<float, 8>(x + sr * C8 * 8 + c, v);
  load_f<float, 8>(scale + f * C8 * 8 + c, sc);
  load_f<float, 8>(shift + f * C8 * 8 + c, sh);
  Vec16<bf16_t> o;
#pragma unroll
  for (int e = 0; e < 8; ++e) o.set(e, fmaf(v[e], sc[e], sh[e]));
  store16(y + r * C8 * 8 + c, o);
}

hipError_t launch_gn_apply(hipStream_t s, const float* x, const float* scale, const float* shift, void* y, int64_t rows, int C,
                           int rows_per_frame, RowMap m) {
  if (rows <= 0) return hipSuccess;
  if (C % 8 || rows_per_frame <= 0 || m.rows_per_seg <= 0) return hipErrorInvalidValue;
  const unsigned blocks = (unsigned)((rows * (C / 8) + 255) / 256);
  if (m.rows_per_seg >= rows || m.seg_stride == m.rows_per_seg)  // consecutive rows from m.base on
    gn_apply_kernel<false><<<blocks, 256, 0, s>>>(x + m.base * C, scale, shift, (bf16_t*)y, rows, C / 8, rows_per_frame, m);
  else
    gn_apply_kernel<true><<<blocks, 256, 0, s>>>(x, scale, shift, (bf16_t*)y, rows, C / 8, rows_per_frame, m);
  return hipGetLastError();
}

// The rows a 3x3 convolution contracts (lc_convd.hip), rounded once to bf16: y = act(x) with act(x) = SiLU(x * scale[f] + shift[f])
// (ACT) or x, x the channel concatenation of two tensors of rows [frames][rows_per_frame][..] (the second may be missing).
// The arithmetic of the loaders of the other convolution kernels, so results do not depend on which of them runs. A thread
// keeps one packet of 8 channels and its scale / shift and takes kActRows rows, all requested before the first is used: bound
// by memory (fp32, 320 channels: 131072 rows 37 us = 6.8 TB/s, 16384 rows 5.5 us = 5.7 TB/s). A workgroup has up to 256 packets
// side by side, wider rows (a concatenation) have several workgroups (gridDim.z).
constexpr int kActRows = 4;
template <class XT, bool ACT>
__global__ __launch_bounds__(256) void conv_act_kernel(const XT* __restrict__ xa, const XT* __restrict__ xb,
                                                       const float* __restrict__ scale, const float* __restrict__ shift, int ld,
                                                       bf16_t* __restrict__ y, int rows_per_frame, int Ca8, int Cb8, int R) {
  constexpr int VN = Vec16<XT>::N;
  const int C8 = Ca8 + Cb8, W8 = min(C8, 256);
  const int c8 = threadIdx.x % W8 + blockIdx.z * 256, sub = threadIdx.x / W8, f = blockIdx.y;
  const int r0 = blockIdx.x * (R * kActRows) + sub;
  if (r0 >= rows_per_frame || c8 >= C8) return;
  const bool in_a = c8 < Ca8;
  const int64_t ldx = (in_a ? Ca8 : Cb8) * 8;
  const XT* x = (in_a ? xa + c8 * 8 : xb + (c8 - Ca8) * 8) + (int64_t)f * rows_per_frame * ldx;
  Vec16<XT> v[kActRows][8 / VN];
#pragma unroll
  for (int j = 0; j < kActRows; ++j) {
    const int r = min(r0 + j * R, rows_per_frame - 1);
#pragma unroll
    for (int q = 0; q < 8 / VN; ++q) v[j][q] = load16(x + r * ldx + q * VN);
  }
  float sc[8], sh[8];
  if (ACT) {
    load_f<float, 8>(scale + (int64_t)f * ld + c8 * 8, sc);
    load_f<float, 8>(shift + (int64_t)f * ld + c8 * 8, sh);
  }
#pragma unroll
  for (int j = 0; j < kActRows; ++j) {
    const int r = r0 + j * R;
    Vec16<bf16_t> o;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float t = v[j][e / VN].get(e % VN);
      o.set(e, ACT ? silu_fast(fmaf(t, sc[e], sh[e])) : t);
    }
    if (r < rows_per_frame) store16(y + ((int64_t)f * rows_per_frame + r) * C8 * 8 + c8 * 8, o);
  }
}

hipError_t launch_conv_act(hipStream_t s, int x_dt, const void* xa, int Ca, const void* xb, int Cb, const float* scale, const float* shift,
                           int ld, void* y, int frames, int rows_per_frame) {
  if (frames <= 0 || rows_per_frame <= 0) return hipSuccess;
  if (Ca <= 0 || Cb < 0 || Ca % 8 || Cb % 8 || (scale && ld % 4) || (scale == nullptr) != (shift == nullptr)) return hipErrorInvalidValue;
  if (frames > 65535 || (x_dt == kBF16 && !scale)) return hipErrorNotSupported;
  const int C8 = (Ca + Cb) / 8, W8 = C8 < 256 ? C8 : 256, R = 256 / W8;
  const dim3 grid((unsigned)((rows_per_frame + R * kActRows - 1) / (R * kActRows)), (unsigned)frames, (unsigned)((C8 + 255) / 256));
#define LC_ACT(XT, A) \
  conv_act_kernel<XT, A><<<grid, W8 * R, 0, s>>>((const XT*)xa, (const XT*)xb, scale, shift, ld, (bf16_t*)y, rows_per_frame, Ca / 8, Cb / 8, R)
  if (x_dt == kBF16) LC_ACT(bf16_t, true);
  else if (scale) LC_ACT(float, true);
  else LC_ACT(float, false);
#undef LC_ACT
  return hipGetLastError();
}

}  // namespace lc
