// What the linear kernels over dense bf16 rows (lc_lin2.hip, lc_lin3.hip) share: their arguments and the way a finished
// accumulator tile leaves a wavefront.
#pragma once
#include <type_traits>

#include "lc_internal.h"

namespace lc {

struct Lin2Args {
  const bf16_t* x;     // [rows][K]
  const bf16_t* w;     // [N][K]
  const float* bias;   // [N] or nullptr
  const float* res;    // fp32 [rows][N] or nullptr (may alias y)
  void* y;             // [rows][N], bf16 or fp32
  bf16_t* y2;          // fp32 output only: a copy of y rounded to bf16 (the next layer's operand), or nullptr
  int64_t rows;
  int K, N, ntm, ntn;
  int xm, bm, bn;      // lc_lin3.hip: XCDs along the row tiles, and the tiles of one XCD: bm row tiles x bn channel tiles
  float q_scale;       // channels below q_cols are multiplied by this before they are rounded
  int q_cols;
  int act;             // 0 none, 1 GELU, 2 GEGLU over alternating 32-channel blocks (y is then N / 2 wide)
  RowMap in_map, out_map;  // dense row r is row in_map(r) of x and row out_map(r) of y / res / y2
  // bf16 output over dense rows only: channels >= yt_from are not stored in y (whose rows then have yt_from channels)
  // but transposed into yt[g / yt_T][N - yt_from][yt_Tp] at column (t & ~63) + vcol(t & 63), g the launch's row, t = g % yt_T:
  // the V^T layout of the spatial attention kernel. nullptr: off. yt_from a multiple of a wavefront's channels, yt_T of 4.
  bf16_t* yt;
  int yt_from, yt_T, yt_Tp;
  // fp32 output over dense rows, with `res` only: y = res + gate[(row0 + r) / gate_T][co] * (x W^T + bias), the gate vectors
  // gate_ld floats apart, gate_n of them, gate_T >= 32 (a 32-row tile meets two at most). nullptr: off.
  const float* gate;
  int gate_T, gate_n;
  int64_t gate_ld;
  int64_t row0;  // gate: the launch's first row within the whole matrix
  int ldy;  // channels per row of y (yt_from with yt, else N; N / 2 after a GEGLU)
};

// The tile of a dense launch by its size: lc_lin3.hip's, or lin2_kernel's 128 x 160 (never with a gate)
enum class LinTile { k64x64, k64x128, k128x128, k256x192, k256x256, k128x160 };
LinTile lin3_tile(const Lin2Args& a, bool y_f32);
// A dense launch (N % 128 == 0 or % 160 == 0; yt_from % 64 == 0) on one of lc_lin3.hip's tiles; hipErrorNotSupported for 128 x 160
hipError_t launch_lin3(hipStream_t s, const Lin2Args& a, bool y_f32);

// bf16 stores of a 32-row block, two channels per lane: lanes l and l ^ 1 hold channels c, c + 1 of the same rows;
// they trade halves so that the even lane holds both channels of the even row of a pair and the odd lane both of the
// odd row, and each stores 4 bytes: a wavefront instruction then writes 64 consecutive bytes of two rows instead of
// 64 bytes of one with 2-byte stores. NV: column tiles (32 channels each) in val's second index. put(rp, i, v): rows
// rp and rp + 1 of the accumulator's 16.
template <int NV, int NTV, class Put>
__device__ __forceinline__ void store_pairs(const float (&val)[16][NTV], int lane, Put put) {
  // v_perm_b32 selectors (bytes 0-3: own pair, 4-7: the neighbour's): even (own lo, neighbour's lo), odd (neighbour's hi, own hi)
  const uint32_t sel = lane & 1 ? 0x03020706u : 0x05040100u;
#pragma unroll
  for (int rp = 0; rp < 16; rp += 2) {
    uint32_t out[NV];
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      bf16x2 p2;
      p2[0] = static_cast<bf16_t>(val[rp][i]);
      p2[1] = static_cast<bf16_t>(val[rp + 1][i]);
      const uint32_t own = __builtin_bit_cast(uint32_t, p2);
      const uint32_t nb = (uint32_t)__builtin_amdgcn_mov_dpp((int)own, 0xB1 /* quad_perm [1,0,3,2] */, 0xF, 0xF, true);
      out[i] = __builtin_amdgcn_perm(nb, own, sel);
    }
    put(rp, out);
  }
}

// The epilogue of one 32-row block of NT column tiles (32 channels each): the lane holds channel c0 + 32 i + lp of rows
// rblk + 8 (r / 4) + 4 hh + r % 4.
// Dense rows go through buffer descriptors over the block: rows beyond the end read as zero and are not stored by the bounds
// check, where 64-bit addresses and a condition per row took most of a short contraction's time (131072 x 2560, K = 64, GEGLU
// 215 us with them, 160 now). The row's offset is part of the vector offset, which is what the check compares with the descriptor's size:
// a scalar offset is taken off that size first, and beyond the end it is the larger of the two.
// GATE: Lin2Args::gate may be set (its own registers: the kernels that never take one stay without them).
template <class OT, int NT, bool MAPPED, bool GATE>
__device__ __forceinline__ void lin_epilogue(const Lin2Args& a, const f32x16 (&acc)[NT], int64_t rblk, int c0, int lane,
                                             const float (&bias_l)[NT], const float (&mul_l)[NT]) {
  constexpr int kRaw = 0x00020000;  // descriptor word 3: raw 32-bit data
  const int lp = lane & 31, hh = lane >> 5;
  const int64_t rbase = rblk + 4 * hh;
  const int left = (int)max((int64_t)0, min((int64_t)32, a.rows - rblk));  // existing rows of the block
  auto rofs = [](int r) { return 8 * (r >> 2) + (r & 3); };
  // rows of ld elements of es bytes from column c on: the block's descriptor, and the lane's offset in its first row
  auto block = [&](const void* p, int64_t ld, int es, int c) {
    return __builtin_amdgcn_make_buffer_rsrc((char*)const_cast<void*>(p) + (rblk * ld + c) * es, 0, (int)max((int64_t)0, (left * ld - c) * es), kRaw);
  };
  // the vector offset of a row; opaque, so that the channel tiles behind it stay immediate offsets (one addition a row)
  auto row_at = [](int vo, int row) {
    int v = vo + row;
    asm("" : "+v"(v));
    return v;
  };
  OT* Y = (OT*)a.y;
  const float* R = a.res;
  // The residual (which may be y itself: every element is read and written by the same lane) is fetched for a whole
  // block at once, before the first store of that block: a load placed after a store that may alias it cannot
  // be moved up by the compiler, and one round trip per element would cost more than the whole contraction.
  float rv[16][NT];
  if (R) {
    if constexpr (MAPPED) {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int64_t row = a.out_map(min(rbase + rofs(r), a.rows - 1));
#pragma unroll
        for (int i = 0; i < NT; ++i) rv[r][i] = R[row * a.N + c0 + 32 * i + lp];
      }
    } else {
      const __amdgpu_buffer_rsrc_t rs = block(R, a.N, 4, c0);
      const int vo = (4 * hh * a.N + lp) * 4;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int vr = row_at(vo, rofs(r) * a.N * 4);
#pragma unroll
        for (int i = 0; i < NT; ++i) rv[r][i] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, vr + 128 * i, 0, 0));
      }
    }
  }
  // all arithmetic of the block first, so that the stores below depend on no load
  float val[16][NT];
  bool gated = false;
  if constexpr (GATE && sizeof(OT) == 4 && !MAPPED) {
    if (a.gate) {
      gated = true;
      const int b0 = (int)((a.row0 + rbase) / a.gate_T);
      const int64_t next = (int64_t)(b0 + 1) * a.gate_T - a.row0;  // the first row of the next vector
      const float* g0 = a.gate + min(b0, a.gate_n - 1) * a.gate_ld + c0 + lp;
      const float* g1 = a.gate + min(b0 + 1, a.gate_n - 1) * a.gate_ld + c0 + lp;
#pragma unroll
      for (int i = 0; i < NT; ++i) {
        const float ga = g0[32 * i], gb = g1[32 * i];
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const float g = rbase + rofs(r) >= next ? gb : ga;
          val[r][i] = fmaf(g, acc[i][r] + bias_l[i], rv[r][i]);
          asm volatile("" : "+v"(val[r][i]));
        }
      }
    }
  }
  if (!gated) {
#pragma unroll
    for (int r = 0; r < 16; ++r)
#pragma unroll
      for (int i = 0; i < NT; ++i) val[r][i] = acc[i][r] + bias_l[i];
    if (a.q_cols) {
#pragma unroll
      for (int r = 0; r < 16; ++r)
#pragma unroll
        for (int i = 0; i < NT; ++i) val[r][i] *= mul_l[i];
    }
    if (R) {
#pragma unroll
      for (int r = 0; r < 16; ++r)
#pragma unroll
        for (int i = 0; i < NT; ++i) val[r][i] += rv[r][i];
    }
    if constexpr (sizeof(OT) == 2) {
      if (a.act == 1) {
#pragma unroll
        for (int r = 0; r < 16; ++r)
#pragma unroll
          for (int i = 0; i < NT; ++i) val[r][i] = gelu_tanh_fast(val[r][i]);
      }
    }
    if constexpr (MAPPED) {  // computed here: left alone, the compiler sinks it into the stores' branches
#pragma unroll
      for (int r = 0; r < 16; ++r)
#pragma unroll
        for (int i = 0; i < NT; ++i) asm volatile("" : "+v"(val[r][i]));
    }
  }
  // NV column tiles of val, rounded, to rows of ld channels from column c on
  auto put16 = [&](bf16_t* y, int ld, int c, auto nv_c) __attribute__((always_inline)) {
    constexpr int NV = decltype(nv_c)::value;
    if constexpr (MAPPED) {
      store_pairs<NV>(val, lane, [&](int rp, const uint32_t (&out)[NV]) __attribute__((always_inline)) {
        const int64_t dr = rbase + rofs(rp) + (lane & 1);
        if (dr >= a.rows) return;
        const int64_t row = a.out_map(dr);
#pragma unroll
        for (int i = 0; i < NV; ++i) *reinterpret_cast<uint32_t*>(y + row * ld + c + 32 * i + (lp & ~1)) = out[i];
      });
    } else {
      const __amdgpu_buffer_rsrc_t ys = block(y, ld, 2, c);
      const int vo = ((4 * hh + (lane & 1)) * ld + (lp & ~1)) * 2;
      store_pairs<NV>(val, lane, [&](int rp, const uint32_t (&out)[NV]) __attribute__((always_inline)) {
        const int vr = row_at(vo, rofs(rp) * ld * 2);
#pragma unroll
        for (int i = 0; i < NV; ++i) __builtin_amdgcn_raw_buffer_store_b32(out[i], ys, vr + 64 * i, 0, 0);
      });
    }
  };
  if constexpr (sizeof(OT) == 2) {
    if (a.yt && c0 >= a.yt_from) {  // (uniform over the wavefront) a lane holds 4 consecutive rows of a channel: 8 bytes of V^T
      const int Cv = a.N - a.yt_from;
      const uint32_t g0 = (uint32_t)rblk, T = (uint32_t)a.yt_T;  // (rows <= 2^30: see launch_lin2)
      const uint32_t f0 = g0 / T, t0 = g0 - f0 * T;
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        if (8 * g + 4 * hh >= left) continue;  // (rows come in fours)
        uint32_t f = f0, t = t0 + 8 * g + 4 * hh;
        if (T >= 32) {
          if (t >= T) { t -= T; ++f; }
        } else {
          const uint32_t q = t / T;
          t -= q * T; f += q;
        }
        bf16_t* dst = a.yt + ((int64_t)f * Cv + (c0 - a.yt_from) + lp) * a.yt_Tp + (t & ~63u) + vcol<bf16_t>((int)(t & 63));
#pragma unroll
        for (int i = 0; i < NT; ++i) {
          bf16x4 o;
#pragma unroll
          for (int e = 0; e < 4; ++e) o[e] = static_cast<bf16_t>(val[4 * g + e][i]);
          *reinterpret_cast<bf16x4*>(dst + (int64_t)32 * i * a.yt_Tp) = o;
        }
      }
      return;
    }
  }
  if constexpr (sizeof(OT) == 2 && NT % 2 == 0) {
    if (a.act == 2) {  // GEGLU: column tile 2 q holds 32 values, tile 2 q + 1 their gates; N / 2 channels leave
#pragma unroll
      for (int r = 0; r < 16; ++r)
#pragma unroll
        for (int q = 0; q < NT / 2; ++q) val[r][q] = val[r][2 * q] * gelu_tanh_fast(val[r][2 * q + 1]);
      put16((bf16_t*)a.y, a.N / 2, c0 / 2, std::integral_constant<int, NT / 2>{});
      return;
    }
  }
  if constexpr (sizeof(OT) == 2) {
    put16((bf16_t*)a.y, a.ldy, c0, std::integral_constant<int, NT>{});
  } else {
    if constexpr (MAPPED) {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int64_t dr = rbase + rofs(r);
        if (dr >= a.rows) continue;
        const int64_t row = a.out_map(dr);
#pragma unroll
        for (int i = 0; i < NT; ++i) Y[row * a.N + c0 + 32 * i + lp] = from_f32<OT>(val[r][i]);
      }
    } else {
      const __amdgpu_buffer_rsrc_t ys = block(Y, a.N, 4, c0);
      const int vo = (4 * hh * a.N + lp) * 4;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int vr = row_at(vo, rofs(r) * a.N * 4);
#pragma unroll
        for (int i = 0; i < NT; ++i) __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, (float)val[r][i]), ys, vr + 128 * i, 0, 0);
      }
    }
    if (a.y2) put16(a.y2, a.N, c0, std::integral_constant<int, NT>{});
  }
}

}  // namespace lc
