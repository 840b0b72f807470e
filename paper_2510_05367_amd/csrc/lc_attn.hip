// Attention cores on gfx950.
//
// Spatial attention (tokens = the H*W positions of one frame) is a flash-style kernel (one for fp32 stages, one for
// bf16 stages): one workgroup owns a block of queries of one (frame, head), walks the keys in tiles of 64 staged in
// LDS and keeps per query what it has summed up and the offset its exponents subtract (fp32: a running maximum; bf16:
// usually none), so the T x T score matrix never exists and the kernel needs no workspace. Scores are produced transposed, S^T[key][query] = K Q^T, with
// 32x32 MFMA tiles: one lane then holds 16 keys of ONE query, so the softmax statistics are
// in-lane plus a single cross-lane exchange, and the exponentials, packed to the storage type,
// are directly the B operand of O^T[dim][query] += V^T[dim][key] P^T[key][query].
//
// Temporal attention (tokens = the F frames of one position) is bandwidth-bound: F is 8..32. bf16 stages
// with 8..32 frames put the scores of a (position, head) on one 16 x 16 or 32 x 32 MFMA tile; otherwise one thread
// owns one (position, head, query frame) and streams the F keys / values.
#include "lc_internal.h"

#include <type_traits>

namespace lc {

constexpr int kKeys = 64;  // keys per LDS stage

namespace {
constexpr int kRawBuffer = 0x00020000;  // resource word 3: raw 32-bit data
typedef __attribute__((address_space(3))) unsigned char* lds_ptr;
}  // namespace

// qk: rows [frame*T + token] of stride ldq holding q at column 0 and k at column C (per head: + head*D).
// vt: V transposed and block-permuted, [frame][C][Tp] with token t of a row at column vcol(t), Tp a
// multiple of 64 (columns beyond T are never trusted: they are zeroed while staging).
// the permutation is an involution on the 4-key blocks (it swaps blocks 1 and 2)
template <class T> __device__ __forceinline__ int vcol_inv(int c) { return vcol<T>(c); }

// Queries: the launch takes nq of them, numbered densely; query number i is token q0 + (i / qw) * qstride + i % qw
// (a window of rows of qw tokens out of image rows of qstride tokens; a plain range has qw >= nq).
// PRE: the q columns already hold q * log2(e) / sqrt(d) (the q,k,v projection scales them before it
// rounds them); `scale_log2e` is then 1.
// KS: wavefronts that share a block of 32 queries. 1: each wavefront has queries of its own and walks all keys, in stages of
// 64 that are double buffered. 4: the four wavefronts share their queries and take 32 keys each of stages of 128 (one buffer,
// the next stage waits in registers); what they summed up is combined through LDS at the end. Either way the fp32 matrix
// instructions bound it (64 cycles each, 256 FLOP per cycle and compute unit); what KS = 4 shortens is the serial chain of
// a wavefront, to a quarter, with four times the workgroups.
// XA (cross-attention): the keys are not the queries' own rows but rows [Tk] of stride ldk at kx, one set (with its
// V^T) per group of kv_div consecutive frames; T_tok then counts the query tokens of a frame only.
template <int D, bool PRE, int KS, bool XA = false>
__global__ __launch_bounds__(256, 2) void spatial_attn_kernel(const float* __restrict__ qk, int ldq,
                                                           const float* __restrict__ vt, int Tp, float* __restrict__ out,
                                                           int T_tok, int C, int q0, int nq, int qw, int qstride,
                                                           float scale_log2e, const float* __restrict__ kx = nullptr,
                                                           int ldk = 0, int Tk = 0, int kv_div = 1) {
  typedef float T;
  typedef Mma32<T> M;
  constexpr int VEC = Vec16<T>::N;
  constexpr int DP = (D + M::K - 1) / M::K * M::K;  // contraction length of Q K^T, padded
  constexpr int KSTEPS = DP / M::K;
  constexpr int DM = (D + 31) / 32;                 // 32-row tiles of O^T
  constexpr int KROW = DP * (int)sizeof(T) + 16;    // LDS row stride of the K tile, bytes
  static_assert(KS == 1 || KS == 4, "the wavefronts of a workgroup share all their queries or none");
  constexpr int SK = KS == 1 ? 64 : 128;            // keys per stage
  constexpr int NB = KS == 1 ? 2 : 1;               // stages in LDS
  constexpr int VROW = SK * (int)sizeof(T) + 16;    // LDS row stride of the V^T tile, bytes
  constexpr int PSTEPS = 32 / M::K;                 // P^T V instructions per 32-key sub-tile
  constexpr int KT = SK / KS / 32;                  // 32-key sub-tiles per stage and wavefront
  constexpr int KBYTES = SK * KROW, VBYTES = DM * 32 * VROW;
  constexpr int PK = D / VEC;                       // 16-byte packets per K / V row
  constexpr int NP = (SK * PK + 255) / 256;         // K (and V) packets per thread per stage
  constexpr int RROW = 33;                          // KS == 4: row stride (floats) of the sums handed over at the end
  static_assert(KS == 1 || NB * (KBYTES + VBYTES) >= 4 * (DM * 32 * RROW + 64) * 4, "the sums of four wavefronts fit");
  __shared__ __attribute__((aligned(16))) unsigned char smem[NB * (KBYTES + VBYTES)];
  unsigned char (*const k_lds)[KBYTES] = reinterpret_cast<unsigned char (*)[KBYTES]>(smem);
  unsigned char (*const v_lds)[VBYTES] = reinterpret_cast<unsigned char (*)[VBYTES]>(smem + NB * KBYTES);

  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  const int lq = lane & 31, hh = lane >> 5;
  // Workgroups are handed to the eight XCDs round robin in launch order, and each XCD has an L2 of its
  // own. All query blocks of one (frame, head) stream the same keys and values, so they are mapped to one
  // XCD (problem p on XCD p % 8): its L2 then fetches that K / V once instead of every XCD fetching all of
  // them. Needs the number of problems to be a multiple of eight; otherwise the plain mapping.
  int qb = blockIdx.x, head = blockIdx.y, frame = blockIdx.z;
  {
    const int nqb = gridDim.x, heads = gridDim.y, nprob = gridDim.y * gridDim.z;
    if (nprob % 8 == 0) {
      const int lin = blockIdx.x + nqb * (blockIdx.y + heads * blockIdx.z);
      const int xcd = lin & 7, slot = lin >> 3;
      const int prob = xcd + 8 * (slot / nqb);
      qb = slot % nqb;
      head = prob % heads;
      frame = prob / heads;
    }
  }
  const int ld = ldq;
  const T* __restrict__ base = qk + (int64_t)frame * T_tok * ld + head * D;
  const int kvf = XA ? frame / kv_div : frame;  // whose keys and values
  const int TK = XA ? Tk : T_tok;               // number of keys
  const int ldkk = XA ? ldk : ld;
  const T* __restrict__ kb = XA ? kx + (int64_t)kvf * Tk * ldk + head * D : base + C;
  const T* __restrict__ vbase = vt + ((int64_t)kvf * C + head * D) * Tp;
  const int qblk = KS == 1 ? qb * (4 * 32) + wid * 32 : qb * 32;  // first query number of this wavefront
  const int sub0 = KS == 1 ? 0 : wid;                             // its first sub-tile of a stage
  auto token_of = [&](int qi) { const int r = qi / qw; return q0 + r * qstride + (qi - r * qw); };

  // zero the buffers once: K columns beyond D and V^T rows beyond D feed padded MFMA lanes
  for (int i = tid; i < NB * (KBYTES + VBYTES) / 4; i += 256) reinterpret_cast<uint32_t*>(smem)[i] = 0u;
  // Softmax denominators for free: when d leaves a spare row in the 32-row tiles of V^T (d = 40:
  // rows 40..63 are padding), row D is set to ones, so O^T[D][q] accumulates the sum over keys of
  // exactly the (rounded) probabilities that multiply V, and is rescaled with the rest of O^T.
  constexpr bool ROWSUM = D % 32 != 0;
  if (ROWSUM) {
    __syncthreads();
    for (int i = tid; i < NB * SK; i += 256)
      reinterpret_cast<T*>(&v_lds[i / SK][D * VROW])[i % SK] = 1.f;
  }

  // ---- staging: K packet i = tid + 256 j of a stage is (key i / PK, packet i % PK); V^T packet i is
  //      (dim i / VPK, packet i % VPK) and is already in LDS order
  constexpr int VPK = SK / VEC;                 // 16-byte packets per V^T row of a stage
  constexpr int NPV = (D * VPK + 255) / 256;
  Vec16<T> kreg[NP], vreg[NPV];
  auto fetch_kv = [&](int k0) {
#pragma unroll
    for (int j = 0; j < NP; ++j) {
      const int i = tid + 256 * j;
      const int key = min(i / PK, SK - 1), pk = i % PK;
      const int gk = min(k0 + key, TK - 1);  // clamped: keys beyond the sequence are masked later
      kreg[j] = load16(kb + (int64_t)gk * ldkk + pk * VEC);
    }
#pragma unroll
    for (int j = 0; j < NPV; ++j) {
      const int i = tid + 256 * j;
      const int dim = min(i / VPK, D - 1), pk = i % VPK;
      // (a row of V^T is whole stages of 64 keys long: of a stage of 128 the second half may lie behind it)
      vreg[j] = load16(vbase + (int64_t)dim * Tp + (KS == 1 ? k0 + pk * VEC : min(k0 + pk * VEC, Tp - VEC)));
    }
  };
  auto stash_kv = [&](int buf, int k0) {
#pragma unroll
    for (int j = 0; j < NP; ++j) {
      const int i = tid + 256 * j;
      if (i < SK * PK) *reinterpret_cast<Vec16<T>*>(&k_lds[buf][(i / PK) * KROW + (i % PK) * 16]) = kreg[j];
    }
    const bool tail = k0 + SK > TK;
#pragma unroll
    for (int j = 0; j < NPV; ++j) {
      const int i = tid + 256 * j;
      if (i < D * VPK) {
        const int dim = i / VPK, pk = i % VPK;
        Vec16<T> v = vreg[j];
        if (tail) {  // column c of the stage holds the token whose vcol is c; zero what lies beyond T
#pragma unroll
          for (int e = 0; e < VEC; ++e)
            if (k0 + vcol_inv<T>(pk * VEC + e) >= TK) v.set(e, 0.f);
        }
        *reinterpret_cast<Vec16<T>*>(&v_lds[buf][dim * VROW + pk * 16]) = v;
      }
    }
  };

  // ---- Q fragments (B operand of S^T = K Q^T): lane holds query lq, k-slots M::LK*hh + M::K*kk
  const int qi = qblk + lq, q = token_of(qi);
  typename M::Frag qf[KSTEPS];
#pragma unroll
  for (int kk = 0; kk < KSTEPS; ++kk) {
    const int e = kk * M::K + hh * M::LK;
    qf[kk] = (qi < nq && e < D) ? M::load(base + (int64_t)q * ld + e) : M::zero();
  }
  f32x16 o[DM];
  float m_run = -INFINITY, l_run = 0.f;  // running max (raw score units) and per-lane partial sum
#pragma unroll
  for (int mt = 0; mt < DM; ++mt)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[mt][r] = 0.f;
  fetch_kv(0);
  __syncthreads();  // zero fill done
  stash_kv(0, 0);
  __syncthreads();

  const int nstage = (TK + SK - 1) / SK;
  for (int st_i = 0; st_i < nstage; ++st_i) {
    const int k0 = st_i * SK, buf = st_i % NB;
    const bool tail = k0 + SK > TK;  // uniform: some keys of this stage lie beyond the sequence
    if (st_i + 1 < nstage) fetch_kv(k0 + SK);
    // (a wavefront none of whose keys of the stage exist; with KS == 1 there is always one)
    if (KS == 1 || k0 + sub0 * 32 < TK) {

    // ---- S^T sub-tiles [32 keys][32 queries]
    f32x16 sc[KT];
#pragma unroll
    for (int kt = 0; kt < KT; ++kt) {
      typename M::Frag kf[KSTEPS];
#pragma unroll
      for (int kk = 0; kk < KSTEPS; ++kk)
        kf[kk] = M::load(reinterpret_cast<const T*>(&k_lds[buf][((sub0 + kt) * 32 + lq) * KROW]) + kk * M::K + hh * M::LK);
#pragma unroll
      for (int r = 0; r < 16; ++r) sc[kt][r] = 0.f;
#pragma unroll
      for (int kk = 0; kk < KSTEPS; ++kk) M::mma(kf[kk], qf[kk], sc[kt]);
    }
    // lane holds keys  k0 + (sub0 + kt)*32 + 8*(r/4) + 4*hh + r%4  of query lq
    if (tail) {
      // (the key indices are built from a value the compiler cannot see through: left alone it hoists
      // these 64 additions out of the branch and every stage pays for them)
      int kbi = k0 + sub0 * 32 + 4 * hh;
      asm volatile("" : "+v"(kbi));
#pragma unroll
      for (int kt = 0; kt < KT; ++kt)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (kbi + kt * 32 + 8 * (r >> 2) + (r & 3) >= TK) sc[kt][r] = -INFINITY;
    }
    float mx = -INFINITY;
#pragma unroll
    for (int kt = 0; kt < KT; ++kt)
#pragma unroll
      for (int r = 0; r < 16; ++r) mx = fmaxf(mx, sc[kt][r]);
    // mx: over this lane's 16 keys of the query. The other half of the query's keys sits in lane l ^ 32; the
    // exchange (a trip through LDS) is only made inside the rare branch below: whether ANY lane of the
    // wavefront exceeds the margin is the same question asked of the per-lane and of the per-query maxima.
    // The offset m subtracted in the exponent need not be the exact running maximum: any m gives the same
    // softmax as long as exp2 stays in range, because the same m enters the probabilities, the denominator
    // and the rescaling. So m is raised (and O^T, l rescaled) only when some query of the wavefront sees a
    // score more than kLazy above its m (in log2 units: probabilities then reach at most 2^kLazy, harmless
    // in fp32). With the exact maximum about 70 % of the 64-key stages
    // took the rescaling branch for some lane; with the margin hardly any after the first. (A lane whose own
    // score stays inside the margin keeps its m when the branch is taken for another: exp2(0) = 1 exactly.)
    constexpr float kLazy = 8.f;
    if (st_i == 0 || __builtin_amdgcn_ballot_w64((mx - m_run) * scale_log2e > kLazy) != 0) {
      mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
      const bool up = st_i == 0 || (mx - m_run) * scale_log2e > kLazy;
      const float m_new = up ? fmaxf(m_run, mx) : m_run;
      // (a sub-tile of scores that are all -inf leaves the maximum there: nothing to rescale, nothing to subtract)
      const float alpha = KS != 1 && m_new == m_run ? 1.f : __builtin_amdgcn_exp2f((m_run - m_new) * scale_log2e);
      m_run = m_new;
      if (!ROWSUM) l_run *= alpha;
#pragma unroll
      for (int mt = 0; mt < DM; ++mt)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[mt][r] *= alpha;
    }
    const float mc = KS != 1 && m_run == -INFINITY ? 0.f : m_run * scale_log2e;
    typename M::Frag pf[KT][PSTEPS];
    float ps = 0.f;
#pragma unroll
    for (int kt = 0; kt < KT; ++kt)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        pf[kt][r] = __builtin_amdgcn_exp2f(fmaf(sc[kt][r], scale_log2e, -mc));
        if (!ROWSUM) ps += pf[kt][r];
      }
    if (!ROWSUM) l_run += ps;
    // ---- O^T += V^T P^T. Step st of sub-tile kt contracts, in lane half hh, the single key 8*(st/4) + 4*hh + st%4.
#pragma unroll
    for (int kt = 0; kt < KT; ++kt)
#pragma unroll
      for (int st = 0; st < PSTEPS; ++st) {
        const int col = (sub0 + kt) * 32 + 8 * (st >> 2) + 4 * hh + (st & 3);
#pragma unroll
        for (int mt = 0; mt < DM; ++mt) {
          const typename M::Frag vf = M::load(reinterpret_cast<const T*>(&v_lds[buf][(mt * 32 + lq) * VROW]) + col);
          M::mma(vf, pf[kt][st], o[mt]);
        }
      }
    }
    if (st_i + 1 < nstage) {
      if (NB == 1) __syncthreads();  // everybody has read the stage
      stash_kv(NB == 1 ? 0 : buf ^ 1, k0 + SK);
    }
    __syncthreads();
  }

  if constexpr (KS != 1) {
    // ---- combine: bring the sums of the four wavefronts to the largest of their offsets and add them, in a fixed order
    float* const red = reinterpret_cast<float*>(smem);  // [wavefront][dim][RROW]: O^T of the 32 queries
    float* const ml = red + 4 * DM * 32 * RROW;          // [wavefront][offset | denominator][32]
    if (!ROWSUM) l_run += __shfl_xor(l_run, 32, 64);
    if (hh == 0) {
      ml[wid * 64 + lq] = m_run;
      ml[wid * 64 + 32 + lq] = l_run;
    }
    __syncthreads();
    float m_all = -INFINITY;
#pragma unroll
    for (int w = 0; w < 4; ++w) m_all = fmaxf(m_all, ml[w * 64 + lq]);
    auto factor = [&](float m, float top) { return m == top ? 1.f : __builtin_amdgcn_exp2f((m - top) * scale_log2e); };
    const float f = factor(m_run, m_all);
#pragma unroll
    for (int mt = 0; mt < DM; ++mt)
#pragma unroll
      for (int r = 0; r < 16; ++r) red[((wid * DM + mt) * 32 + 8 * (r >> 2) + 4 * hh + (r & 3)) * RROW + lq] = o[mt][r] * f;
    __syncthreads();
    const int tq = tid >> 3, td = (tid & 7) * (DM * 4);  // this thread finishes dims td .. td + 4 DM - 1 of query tq
    float l = 0.f, m_top = -INFINITY;
#pragma unroll
    for (int w = 0; w < 4; ++w) m_top = fmaxf(m_top, ml[w * 64 + tq]);
#pragma unroll
    for (int w = 0; w < 4; ++w)
      l += ROWSUM ? red[(w * DM * 32 + D) * RROW + tq] : ml[w * 64 + 32 + tq] * factor(ml[w * 64 + tq], m_top);
    const float inv = 1.f / l;
    if (qblk + tq >= nq) return;
    T* orow = out + ((int64_t)frame * T_tok + token_of(qblk + tq)) * C + head * D;
#pragma unroll
    for (int e = 0; e < DM * 4; ++e) {
      if (td + e < D) {
        float v = 0.f;
#pragma unroll
        for (int w = 0; w < 4; ++w) v += red[(w * DM * 32 + td + e) * RROW + tq];
        orow[td + e] = v * inv;
      }
    }
    return;
  }

  // ---- normalise and store: lane holds O^T[dim = 32*mt + 8*(r/4) + 4*hh + r%4][query lq]
  float l;
  if (ROWSUM) {  // O^T[D][q] sits in register r of the lanes of half hsel
    constexpr int rem = D % 32, hsel = (rem % 8) / 4, r = (rem / 8) * 4 + rem % 4;
    l = __shfl(o[D / 32][r], lq + 32 * hsel, 64);
  } else {
    l = l_run + __shfl_xor(l_run, 32, 64);
  }
  const float inv = 1.f / l;
  if (qi >= nq) return;
  T* orow = out + ((int64_t)frame * T_tok + q) * C + head * D;
#pragma unroll
  for (int mt = 0; mt < DM; ++mt)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const int dim = mt * 32 + 8 * g + 4 * hh;
      if (dim < D) {
#pragma unroll
        for (int e = 0; e < 4; ++e) orow[dim + e] = o[mt][4 * g + e] * inv;
      }
    }
}

// f(0), f(1), .. f(N - 1) with compile-time indexes (the bodies below index register arrays)
template <int I, int N, class F> __device__ __forceinline__ void static_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<I + 1, N>(static_cast<F&&>(f));
  }
}

// Spatial attention of the bf16 stages. What bounds it: the matrix pipe (d = 64: 512 cycles of MFMAs per 32 keys x 64
// queries and wavefront) and, beside it, the vector port (32 exponentials, 16 packs, 16 dot products for the denominator).
// Here the two overlap inside a wavefront. A substep is 32 keys, and three independent pieces of work are issued interleaved, a few vector instructions behind every MFMA:
//   scores of substep j + 1 (K Q^T)  |  probabilities of substep j  |  O^T += V^T P^T of substep j - 1
// Fragments are requested from LDS half a substep ahead of their use. K and V^T go from global memory straight into
// LDS (16 bytes per lane) into a ring of four 64-key stages: stage s + 2 is requested at the start of stage s, one
// barrier per stage. (Four, because the scores run into stage s + 1 and the lagging V fragments are read until late in
// stage s.) 16-byte slots are XOR-swizzled where a row is 128 bytes.
// What the exponents subtract: softmax does not depend on it, and with scores in log2 units of ordinary size exp2 needs
// nothing subtracted in fp32 (bf16 has the same exponent range and rounds relatively). So a query's offset m is zero if the
// largest of its first 32 scores lies within kNear of zero, else that score, rounded; a wavefront whose offsets are all zero
// runs the plain form of a substep, which subtracts nothing, others the safe form, which does and raises an offset (scaling
// what it has summed up) before a score passes it by kRaise. The plain form looks at the denominators after every stage: one
// past kHigh sends its wavefront on in the safe form, and one past kBroken says that a score came that the safe form would
// have raised m for; the workgroup is then done again, safely. Should an output not be finite after all (values near the end
// of their own range), its query is done once more with its exact maximum, found in a sweep over the keys. Every decision
// that shows in a query's bits is its own (x - 0 is x), whoever shares its wavefront.
// Measured (us per launch, with a kernel that ran the two phases in turn / this one): d = 64, 5 x 9216 tokens, 2304
// queries, 5 heads 204 / 170 alone and 157 / 132 with two launches in flight (1.02 PFLOP/s); d = 40, 4 x 4096, 8 heads
// 121 / 101; d = 40, 8 x 9216 1110 / 960; cross-attention to 77 keys, 16 x 4096, 8 heads 48 / 43. Counters, shares of the
// cycles: d = 40, 4 x 4096: matrix pipe 52 % (41 % in turn), exponentials 59 % (47 %), LDS 74 %, clock 2.2 GHz; 32 x 4096: 61 %,
// 69 %, 88 %, 2.0 GHz; d = 64, 2 x 4096, 16 heads: 48 % each, 1.9 GHz. Nothing is full but the LDS of the larger d = 40 launches,
// and the clock falls with the work done in a cycle (with zeros as input it stays at 2.3): the rest is what one wavefront's
// instructions wait for each other.
// Scores out of range (us; this kernel / the plain form alone, every workgroup with such a score done again with exact maxima /
// a kernel with a running maximum throughout; d = 64, 5 x 9216 tokens, 5 heads | d = 40, 4 x 4096, 8 heads, both with the
// pass that transposes V): deviation 1.4 in log2 units 562, 556, 663 | 128, 129, 150; 15: 606, 551, 684 | 141, 118, 150; 40:
// 612, 1542, 673 | 138, 320, 147; 150: 638, 1501, 647 | 157, 303, 142; 500: 688, 1476, 643 | 173, 298, 143; all near -240:
// 594, 1467, 660 | 131, 294, 131; one late key at +150: 1096, 1520, 653 | 224, 304, 132.
// The limits: kNear + a few deviations of ordinary scores stay below kHigh, and kRaise leaves exp2's range (2^128) room for
// values and sums. With kNear = 40 and kHigh = 2^40 scores of deviation 15 took 619, with 60 and 2^80, where more wavefronts
// meet a score beyond kRaise in the plain form, 717.
// NQT: 32-query tiles per wavefront. Two share every fragment read; one is for launches that would otherwise leave
// compute units without a workgroup.
template <int D, int NQT, bool PRE, bool XA>
__global__ __launch_bounds__(256, 2) void spatial_attn_ring_kernel(const bf16_t* __restrict__ qk, int ldq,
                                                                   const bf16_t* __restrict__ vt, int Tp,
                                                                   bf16_t* __restrict__ out, int T_tok, int C, int q0, int nq,
                                                                   int qw, int qstride, float scale_log2e,
                                                                   const bf16_t* __restrict__ kx, int ldk, int Tk, int kv_div) {
  typedef Mma32<bf16_t> M;
  typedef M::Frag Frag;
  constexpr int KSTEPS = (D + 15) / 16;     // MFMAs along d
  constexpr int DM = (D + 31) / 32;         // 32-row tiles of O^T
  constexpr int KP = 2 * KSTEPS;            // 16-byte slots of a K row in LDS (those beyond d are zeros)
  constexpr int KSLOT = kKeys * KP * 16, VSLOT = DM * 32 * 128, SLOT = KSLOT + VSLOT;
  constexpr int NB = 4;                     // stages in LDS
  constexpr bool ROWSUM = D % 32 != 0;      // a spare row of V^T holds ones: O^T[D] is the denominator
  constexpr bool KSWZ = KP == 8;            // 128-byte K rows
  constexpr int NKI = KP, NVI = D / 8;      // wavefront instructions that move one stage of K, of V^T
  constexpr int KJ = (NKI + 3) / 4, VJ = (NVI + 3) / 4;
  constexpr int NQK = NQT * KSTEPS, NPV = NQT * 2 * DM, NM = NQK + NPV;  // MFMAs of a substep
  constexpr int NE = NQT * 16;              // exponentials of a substep
  constexpr int NF = KSTEPS + 2 * DM;       // LDS fragments of a substep, NQT MFMAs each
  constexpr int kAhead = 2 * DM < 6 / NQT ? 2 * DM : 6 / NQT;
  constexpr float kNear = 52.f, kRaise = 100.f, kAbove = 16.f;  // (see above)
  constexpr float kHigh = 0x1p60f, kBroken = 0x1p99f;
  enum Sweep { kPlain, kSafe, kExact };
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  auto kl = [&](int b) { return smem + b * SLOT; };
  auto vl = [&](int b) { return smem + b * SLOT + KSLOT; };
  // sweep again: every query safely; some with their exact maxima, seen behind the first sweep, behind a safe one
  int* flags = reinterpret_cast<int*>(smem + NB * SLOT);

  const int tid = threadIdx.x, lane = tid & 63, wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lq = lane & 31, hh = lane >> 5;
  int qb = blockIdx.x, head = blockIdx.y, frame = blockIdx.z;
  {  // all query blocks of one (frame, head) on one XCD, as above
    const int nqb = gridDim.x, heads = gridDim.y, nprob = gridDim.y * gridDim.z;
    if (nprob % 8 == 0) {
      const int lin = blockIdx.x + nqb * (blockIdx.y + heads * blockIdx.z);
      const int xcd = lin & 7, slot = lin >> 3;
      const int prob = xcd + 8 * (slot / nqb);
      qb = slot % nqb;
      head = prob % heads;
      frame = prob / heads;
    }
  }
  const bf16_t* __restrict__ base = qk + (int64_t)frame * T_tok * ldq + head * D;
  const int kvf = XA ? frame / kv_div : frame, TK = XA ? Tk : T_tok, ldkk = XA ? ldk : ldq;
  const bf16_t* __restrict__ kb = XA ? kx + (int64_t)kvf * Tk * ldk + head * D : base + C;
  const bf16_t* __restrict__ vbase = vt + ((int64_t)kvf * C + head * D) * Tp;
  const int qblk = qb * (4 * NQT * 32) + wid * (NQT * 32);
  auto token_of = [&](int qi) { const int r = qi / qw; return q0 + r * qstride + (qi - r * qw); };

  // rows of V^T beyond d: ones in row D (ROWSUM), zeros below; the loads never touch them
  if constexpr (ROWSUM) {
    constexpr int per = (DM * 32 - D) * 8;  // 16-byte packets of a stage
    for (int i = tid; i < NB * per; i += 256) {
      const int b = i / per, p = i - b * per;
      const uint32_t v = p < 8 ? 0x3f803f80u : 0u;
      *reinterpret_cast<uint4*>(vl(b) + D * 128 + p * 16) = uint4{v, v, v, v};
    }
  }
  if (tid < 3) flags[tid] = 0;

  // ---- global -> LDS. K: packet p of a stage is (key p / KP, slot p % KP); V^T: (row p / 8, slot p % 8). Buffer loads,
  // whose bounds check delivers zeros for the slots of K beyond d (a copy of anything there could meet the zeros of q with
  // an infinity) and for keys beyond the sequence (masked below); the resource moves on by a stage.
  uint32_t koff[KJ], voff[VJ];
#pragma unroll
  for (int j = 0; j < KJ; ++j) {
    const int p = min(wid + 4 * j, NKI - 1) * 64 + lane, key = p / KP, sl = p % KP;
    const int c = KSWZ ? (sl ^ ((key >> 1) & 7)) : sl;
    koff[j] = c < D / 8 ? (uint32_t)(key * ldkk + c * 8) * 2 : 0x7fffff00u;
  }
#pragma unroll
  for (int j = 0; j < VJ; ++j) {
    const int p = min(wid + 4 * j, NVI - 1) * 64 + lane, dim = p / 8, sl = p % 8;
    voff[j] = (uint32_t)(dim * Tp + (sl ^ ((dim >> 1) & 7)) * 8) * 2;
  }
  auto issue = [&](int st) {
#ifdef __HIP_DEVICE_COMPILE__  // the host pass only needs the kernel's stub; it does not know these builtins
    lds_ptr b = (lds_ptr)kl(st & (NB - 1));
    const int keys = min(kKeys, TK - st * kKeys);
    const __amdgpu_buffer_rsrc_t kr = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(kb + (int64_t)st * kKeys * ldkk), 0,
                                                                        ((keys - 1) * ldkk + D) * 2, kRawBuffer);
    const __amdgpu_buffer_rsrc_t vr = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(vbase + (int64_t)st * kKeys), 0,
                                                                        (int)((uint32_t)((D - 1) * Tp + kKeys) * 2), kRawBuffer);
#pragma unroll
    for (int j = 0; j < KJ; ++j)
      if (wid + 4 * j < NKI) __builtin_amdgcn_raw_ptr_buffer_load_lds(kr, b + (wid + 4 * j) * 1024, 16, koff[j], 0, 0, 0);
#pragma unroll
    for (int j = 0; j < VJ; ++j)
      if (wid + 4 * j < NVI) __builtin_amdgcn_raw_ptr_buffer_load_lds(vr, b + KSLOT + (wid + 4 * j) * 1024, 16, voff[j], 0, 0, 0);
#else
    (void)st; (void)koff; (void)voff;
#endif
  };
  // every load has landed (for every wavefront, behind the barrier); LDS reads in flight are left alone: the stage they
  // read is written again two barriers later at the earliest
  auto stage_barrier = [&]() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(7 << 4 | 15 << 8);  // vmcnt(0)
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };

  // ---- Q fragments (B operand of S^T = K Q^T); slots beyond d are zeros
  Frag qf[NQT][KSTEPS];
#pragma unroll
  for (int t = 0; t < NQT; ++t) {
    const int qi = qblk + t * 32 + lq;
    const int q = token_of(min(qi, nq - 1));
#pragma unroll
    for (int kk = 0; kk < KSTEPS; ++kk) {
      const int e = kk * 16 + hh * 8;
      qf[t][kk] = (qi < nq && e < D) ? M::load(base + (int64_t)q * ldq + e) : M::zero();
    }
  }
  const int krow = lq * (KP * 16), kkey = KSWZ ? ((lq >> 1) & 7) : 0;
  const int vrow = lq * 128, vkey = (lq >> 1) & 7;
  auto kfrag = [&](const unsigned char* k, int u, int kk) {
    return M::load((const bf16_t*)(k + u * 32 * KP * 16 + krow + (((kk * 2 + hh) ^ kkey) << 4)));
  };
  // the 8 keys a lane contracts in step st of substep u: V^T columns 32 u + 16 st + 8 hh ..+7
  auto vfrag = [&](const unsigned char* v, int u, int st, int mt) {
    return M::load((const bf16_t*)(v + mt * 32 * 128 + vrow + (((4 * u + 2 * st + hh) ^ vkey) << 4)));
  };
  auto beyond = [&](int key0, int r) { return key0 + 4 * hh + 8 * (r >> 2) + (r & 3) >= TK; };  // accumulator r's key

  const int nstage = (TK + kKeys - 1) / kKeys;
  f32x16 o[NQT][DM];
  float lsum[NQT][2];
  float m[NQT];      // what the exponents subtract, in their own units (log2)
  bool safe, broken;  // this wavefront subtracts it; a score passed kRaise while it did not

  // the denominator, as far as this lane holds it
  auto so_far = [&](int t) {
    if constexpr (ROWSUM) return o[t][D / 32][(D % 32 / 8) * 4 + D % 4];  // (the other half of the lanes: a row of zeros)
    else return fmaxf(lsum[t][0], lsum[t][1]);
  };
  auto sweep = [&](Sweep kind) __attribute__((always_inline)) {
    f32x16 sA[NQT], sB[NQT];     // scores: of this substep, of the next
    Frag pA[NQT][2], pB[NQT][2]; // probabilities as operands: of this substep, of the one before
    Frag kf[KSTEPS], vf[2][DM];
    const f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < NQT; ++t) {
      lsum[t][0] = lsum[t][1] = 0.f;
      pB[t][0] = pB[t][1] = M::zero();
#pragma unroll
      for (int mt = 0; mt < DM; ++mt) o[t][mt] = zero16;
    }
    auto exponent = [&](float x, int t) { return PRE ? x - m[t] : fmaf(x, scale_log2e, -m[t]); };
    // O^T += (V^T of the 32 keys (vp, up)) pp; sn = K Q^T of the keys (ks, us); pc = probabilities of sc (first key key0).
    // The fragment of group g (NQT MFMAs each: V fragments, then K fragments) is requested kAhead groups before its use,
    // the first V fragments of the next substep, (vn, un), in the last groups of this one.
    auto substep = [&](auto safe_c, f32x16 (&sn)[NQT], f32x16 (&sc)[NQT], Frag (&pc)[NQT][2], Frag (&pp)[NQT][2], const unsigned char* vp, int up,
                       const unsigned char* ks, int us, const unsigned char* vn, int un, int key0)
                       __attribute__((always_inline)) {
      constexpr bool SAFE = decltype(safe_c)::value;
      if (key0 + 32 > TK) {  // uniform: some keys lie beyond the sequence
        int kb0 = key0 + 4 * hh;
        asm volatile("" : "+v"(kb0));  // (left alone the compiler computes the sixteen indexes outside the branch)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const bool gone = kb0 + 8 * (r >> 2) + (r & 3) >= TK;
#pragma unroll
          for (int t = 0; t < NQT; ++t)
            if (gone) sc[t][r] = -INFINITY;
        }
      }
      if constexpr (SAFE) {
        float hi[NQT];
        bool any = false;
#pragma unroll
        for (int t = 0; t < NQT; ++t) {
          hi[t] = sc[t][0];
#pragma unroll
          for (int r = 1; r < 16; ++r) hi[t] = fmaxf(hi[t], sc[t][r]);
          hi[t] = exponent(hi[t], t);
          any |= hi[t] > kRaise;
        }
        if (__builtin_amdgcn_ballot_w64(any) != 0) {  // some query's m is raised, and what it has summed up is scaled
#pragma unroll
          for (int t = 0; t < NQT; ++t) {
            hi[t] = fmaxf(hi[t], __shfl_xor(hi[t], 32, 64));
            const float k = hi[t] > kRaise ? rintf(hi[t]) + kAbove : 0.f;
            const int by = -(int)fminf(k, 4096.f);  // (a factor 2^-k could be too small for a float where its products are not)
            m[t] += k;
            lsum[t][0] = ldexpf(lsum[t][0], by);
            lsum[t][1] = ldexpf(lsum[t][1], by);
#pragma unroll
            for (int mt = 0; mt < DM; ++mt)
#pragma unroll
              for (int r = 0; r < 16; ++r) o[t][mt][r] = ldexpf(o[t][mt][r], by);
#pragma unroll
            for (int st = 0; st < 2; ++st)
#pragma unroll
              for (int e = 0; e < 8; ++e) pp[t][st][e] = static_cast<bf16_t>(ldexpf(static_cast<float>(pp[t][st][e]), by));
          }
        }
      }
      static_for<0, NM>([&](auto m_c) __attribute__((always_inline)) {
        constexpr int i = decltype(m_c)::value;
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (i % NQT == 0) {
          constexpr int g = i / NQT + kAhead;
          if constexpr (g < 2 * DM) vf[g / DM][g % DM] = vfrag(vp, up, g / DM, g % DM);
          else if constexpr (g < NF) kf[g - 2 * DM] = kfrag(ks, us, g - 2 * DM);
          else vf[(g - NF) / DM][(g - NF) % DM] = vfrag(vn, un, (g - NF) / DM, (g - NF) % DM);
          __builtin_amdgcn_sched_barrier(0);
          // the group's own fragment has arrived, the kAhead younger ones may be on their way (left alone the compiler
          // waits for all of them at every fourth group)
          __builtin_amdgcn_s_waitcnt(15 | 7 << 4 | kAhead << 8 | 3 << 14);
        }
        if constexpr (i < NPV) {
          constexpr int st = i / (DM * NQT), mt = i / NQT % DM, t = i % NQT;
          M::mma(vf[st][mt], pp[t][st], o[t][mt]);
        } else {
          constexpr int kk = (i - NPV) / NQT, t = i % NQT;
          sn[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[kk], qf[t][kk], kk ? sn[t] : zero16, 0, 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
        constexpr int e0 = (i * NE / NM) & ~1, e1 = i == NM - 1 ? NE : (((i + 1) * NE / NM) & ~1);
        static_for<0, (e1 - e0) / 2>([&](auto e_c) __attribute__((always_inline)) {
          constexpr int e = e0 + 2 * decltype(e_c)::value, t = e / 16, r = e % 16;
          float p[2];
#pragma unroll
          for (int k = 0; k < 2; ++k) {
            p[k] = __builtin_amdgcn_exp2f(SAFE ? exponent(sc[t][r + k], t) : PRE ? sc[t][r + k] : sc[t][r + k] * scale_log2e);
            pc[t][r / 8][r % 8 + k] = static_cast<bf16_t>(p[k]);
          }
          // the denominator sums the probabilities as rounded, like the ones row does: what one key contributes to
          // numerator and denominator then cancels, however peaked the softmax is
          if constexpr (!ROWSUM) {
            bf16x2 p2, one2;
            p2[0] = pc[t][r / 8][r % 8];
            p2[1] = pc[t][r / 8][r % 8 + 1];
            one2[0] = one2[1] = (bf16_t)1.f;
            lsum[t][e / 2 % 2] = __builtin_amdgcn_fdot2_f32_bf16(p2, one2, lsum[t][e / 2 % 2], false);
          }
        });
      });
      // (computed here: left alone the compiler moves them behind the branch of the next substep, which uses them)
#pragma unroll
      for (int t = 0; t < NQT; ++t) asm volatile("" : "+v"(pc[t][0]), "+v"(pc[t][1]));
      __builtin_amdgcn_sched_barrier(0);
    };
    // columns of V^T beyond the sequence hold anything: zeros, so that they meet zero probabilities safely
    auto clear_beyond = [&](int s, int b) {
      for (int i = tid; i < D * kKeys; i += 256) {
        const int dim = i / kKeys, col = i % kKeys;
        if (s * kKeys + vcol_inv<bf16_t>(col) >= TK)
          *reinterpret_cast<bf16_t*>(vl(b) + dim * 128 + (((col >> 3) ^ ((dim >> 1) & 7)) << 4) + (col & 7) * 2) = (bf16_t)0.f;
      }
      __syncthreads();
    };
    // V of "the stage before" the first one: zeros, which meet the zero probabilities of the first substep (stage 3 lands there)
    for (int i = tid; i < D * 8; i += 256) *reinterpret_cast<uint4*>(vl(NB - 1) + i * 16) = uint4{0u, 0u, 0u, 0u};
    issue(0);
    if (nstage > 1) issue(1);
    // this barrier also stands between what the prologue wrote to LDS (the rows of V^T beyond d, the zeros above) and the other wavefronts'
    // first fragments: it waits for LDS too
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(7 << 4);  // vmcnt(0) lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    if (kKeys > TK) clear_beyond(0, 0);  // (before the first fragments of V are requested, below)
    static_for<0, KSTEPS>([&](auto kk) __attribute__((always_inline)) { kf[decltype(kk)::value] = kfrag(kl(0), 0, decltype(kk)::value); });
    static_for<0, NQK>([&](auto i) __attribute__((always_inline)) {
      constexpr int kk = decltype(i)::value / NQT, t = decltype(i)::value % NQT;
      sA[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[kk], qf[t][kk], kk ? sA[t] : zero16, 0, 0, 0);
    });
    if (kind != kExact) {
      // (lane by lane first: the two halves of a query's scores are brought together only if some lane's are far)
      float hi[NQT];
      bool far = false;
#pragma unroll
      for (int t = 0; t < NQT; ++t) {
        hi[t] = -INFINITY;
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (!beyond(0, r)) hi[t] = fmaxf(hi[t], sA[t][r]);
        hi[t] *= PRE ? 1.f : scale_log2e;
        m[t] = 0.f;
        far |= !(fabsf(hi[t]) <= kNear);
      }
      safe = kind == kSafe;
      if (__builtin_amdgcn_ballot_w64(far) != 0) {
        far = false;
#pragma unroll
        for (int t = 0; t < NQT; ++t) {
          hi[t] = fmaxf(hi[t], __shfl_xor(hi[t], 32, 64));
          if (fabsf(hi[t]) > kNear && fabsf(hi[t]) < INFINITY) {
            m[t] = rintf(hi[t]);
            far = true;
          }
        }
        safe |= __builtin_amdgcn_ballot_w64(far) != 0;
      }
    } else {
      safe = true;
    }
    broken = false;
    static_for<0, kAhead>([&](auto g) __attribute__((always_inline)) {
      vf[decltype(g)::value / DM][decltype(g)::value % DM] = vfrag(vl(NB - 1), 1, decltype(g)::value / DM, decltype(g)::value % DM);
    });
    // (Behind the last stage the K requests and scores are of no stage: in bounds, never used.)
    int s = 0;
    auto stage = [&](auto safe_c) __attribute__((always_inline)) {
      if (s) stage_barrier();
      if (s + 2 < nstage) issue(s + 2);
      const int b = s & (NB - 1), bn = (s + 1) & (NB - 1), bp = (s - 1) & (NB - 1);
      if (s && s * kKeys + kKeys > TK) clear_beyond(s, b);
      substep(safe_c, sB, sA, pA, pB, vl(bp), 1, kl(b), 1, vl(b), 0, s * kKeys);
      substep(safe_c, sA, sB, pB, pA, vl(b), 0, kl(bn), 0, vl(b), 1, s * kKeys + 32);
    };
    if (!safe) for (; s < nstage; ++s) {
      stage(std::false_type{});
      bool high = false;
#pragma unroll
      for (int t = 0; t < NQT; ++t) high |= so_far(t) > kHigh;
      if (__builtin_expect(__builtin_amdgcn_ballot_w64(high) != 0, 0)) {
        safe = true;  // (from the next stage on)
        ++s;
#pragma unroll
        for (int t = 0; t < NQT; ++t) {
          broken |= so_far(t) > kBroken;
          if constexpr (ROWSUM) {  // (the last substep's are not in it yet)
#pragma unroll
            for (int st = 0; st < 2; ++st)
#pragma unroll
              for (int e = 0; e < 8; ++e) broken |= static_cast<float>(pB[t][st][e]) > kBroken;
          }
        }
        break;
      }
    }
    for (; s < nstage; ++s) stage(std::true_type{});
    const unsigned char* vlast = vl((nstage - 1) & (NB - 1));
    static_for<0, 2 * DM>([&](auto i) __attribute__((always_inline)) {
      constexpr int st = decltype(i)::value / DM, mt = decltype(i)::value % DM;
      const Frag v = decltype(i)::value < kAhead ? vf[st][mt] : vfrag(vlast, 1, st, mt);
#pragma unroll
      for (int t = 0; t < NQT; ++t) M::mma(v, pB[t][st], o[t][mt]);
    });
  };

  // ---- normalise and store the queries of tile t: lane holds O^T[dim = 32 mt + 8 (r / 4) + 4 hh + r % 4][query lq]
  auto denominator = [&](int t) {
    if constexpr (ROWSUM) {  // O^T[D][q] sits in register r of the lanes of half hsel
      constexpr int rem = D % 32, hsel = (rem % 8) / 4, r = (rem / 8) * 4 + rem % 4;
      return __shfl(o[t][D / 32][r], lq + 32 * hsel, 64);
    } else {
      const float l = lsum[t][0] + lsum[t][1];
      return l + __shfl_xor(l, 32, 64);
    }
  };
  auto store = [&](int t, float inv) {
    const int qi = qblk + t * 32 + lq;
    if (qi >= nq) return;
    bf16_t* orow = out + ((int64_t)frame * T_tok + token_of(qi)) * C + head * D;
#pragma unroll
    for (int mt = 0; mt < DM; ++mt)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int dim = mt * 32 + 8 * g + 4 * hh;
        if (dim < D) {
          bf16x4 ov;
#pragma unroll
          for (int e = 0; e < 4; ++e) ov[e] = static_cast<bf16_t>(o[t][mt][4 * g + e] * inv);
          *reinterpret_cast<bf16x4*>(orow + dim) = ov;
        }
      }
  };

  bool redo[NQT];
  for (Sweep kind = kPlain;;) {  // (every decision here is the workgroup's)
    sweep(kind);
    bool any = false;
#pragma unroll
    for (int t = 0; t < NQT; ++t) {
      const float l = denominator(t);
      float worst = 0.f;  // NaN or infinite if any element is
#pragma unroll
      for (int mt = 0; mt < DM; ++mt)
#pragma unroll
        for (int r = 0; r < 16; ++r) worst = fmaf(o[t][mt][r], 0.f, worst);
      int bad = !(l >= 0x1p-90f && l <= 0x1p125f) || worst != 0.f;
      bad |= __shfl_xor(bad, 32, 64);
      if (kind == kExact ? redo[t] : !bad) store(t, 1.f / l);
      redo[t] = bad && qblk + t * 32 + lq < nq;
      any |= redo[t];
    }
    if (kind == kExact) break;
    if (kind == kPlain) {
#pragma unroll
      for (int t = 0; t < NQT; ++t) broken |= !safe && so_far(t) > kBroken;
      if (__builtin_amdgcn_ballot_w64(broken) != 0 && lane == 0) flags[0] = 1;
    }
    if (__builtin_amdgcn_ballot_w64(any) != 0 && lane == 0) flags[1 + kind] = 1;
    __syncthreads();
    if (kind == kPlain && flags[0]) {  // (what was stored is stored again)
      kind = kSafe;
      continue;
    }
    if (!flags[1 + kind]) break;
    kind = kExact;
    // the exact maxima of every query, for a sweep with them
#pragma unroll
    for (int t = 0; t < NQT; ++t) m[t] = -INFINITY;
    for (int s = 0; s < nstage; ++s) {
      __syncthreads();
      issue(s);
      stage_barrier();
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int t = 0; t < NQT; ++t) {
          f32x16 sc;
#pragma unroll
          for (int r = 0; r < 16; ++r) sc[r] = 0.f;
#pragma unroll
          for (int kk = 0; kk < KSTEPS; ++kk) M::mma(kfrag(kl(s & (NB - 1)), u, kk), qf[t][kk], sc);
#pragma unroll
          for (int r = 0; r < 16; ++r)
            if (!beyond(s * kKeys + 32 * u, r)) m[t] = fmaxf(m[t], sc[r]);
        }
    }
#pragma unroll
    for (int t = 0; t < NQT; ++t) m[t] = fmaxf(m[t], __shfl_xor(m[t], 32, 64)) * (PRE ? 1.f : scale_log2e);
    __syncthreads();
  }
}

template <int D, int NQT, bool PRE, bool XA>
static hipError_t run_ring(hipStream_t s, const bf16_t* qk, int ldq, const bf16_t* vt, int Tp, bf16_t* out, int frames, int T_tok, int heads,
                           int q0, int nq, int qw, int qstride, const bf16_t* kx, int ldk, int Tk, int kv_div) {
  constexpr int lds = 4 * (kKeys * ((D + 15) / 16) * 32 + (D + 31) / 32 * 32 * 128) + 16;
  static_assert(2 * lds <= 160 * 1024, "two workgroups per compute unit");
  auto kern = spatial_attn_ring_kernel<D, NQT, PRE, XA>;
  static bool attr_done = false;  // per instantiation
  if (!attr_done) {
    const hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
    attr_done = true;
  }
  const float sl = PRE ? 1.f : 1.4426950408889634f / sqrtf((float)D);
  dim3 grid((nq + 128 * NQT - 1) / (128 * NQT), heads, frames);
  kern<<<grid, 256, lds, s>>>(qk, ldq, vt, Tp, out, T_tok, heads * D, q0, nq, qw, qstride, sl, kx, ldk, Tk, kv_div);
  return hipGetLastError();
}
template <bool PRE, bool XA>
static hipError_t ring_dispatch(hipStream_t s, const bf16_t* qk, int ldq, const bf16_t* vt, int Tp, bf16_t* out, int frames, int T_tok, int heads,
                                int d, int q0, int nq, int qw, int qstride, const bf16_t* kx = nullptr, int ldk = 0, int Tk = 0,
                                int kv_div = 1) {
  // One query tile per wavefront while two would leave a quarter of the 256 compute units without a workgroup: the extra
  // fragment reads cost less than idle units (d = 40, one frame of 4096 tokens, 8 heads: 128 workgroups 57 us, 256
  // workgroups 43 us; d = 64, 225 against 450 workgroups: 164 and 159 us alone, 133 and 145 us with two launches in flight).
  const bool narrow = (int64_t)((nq + 255) / 256) * heads * frames < 192;
#define LC_GO(D)                                                                                                                        \
  return narrow ? run_ring<D, 1, PRE, XA>(s, qk, ldq, vt, Tp, out, frames, T_tok, heads, q0, nq, qw, qstride, kx, ldk, Tk, kv_div)      \
                : run_ring<D, 2, PRE, XA>(s, qk, ldq, vt, Tp, out, frames, T_tok, heads, q0, nq, qw, qstride, kx, ldk, Tk, kv_div)
  switch (d) {
    case 8: LC_GO(8);
    case 16: LC_GO(16);
    case 32: LC_GO(32);
    case 40: LC_GO(40);
    case 64: LC_GO(64);
    default: return hipErrorInvalidValue;
  }
#undef LC_GO
}

// fp32: whether the wavefronts of a workgroup share their queries and split the keys (KS = 4). Shorter chains and four times
// the workgroups pay while the chip is idle, the staging that is done once per 32 instead of 128 queries costs where it is not:
// 2 frames of 1024 tokens, 1 head of 64 (16 workgroups of 128 queries) 79 us without, 32 us with; 8 heads of 40 (128
// workgroups) 69 and 45 us, 8 frames of 256 (128) 22 and 19 us; 32 frames of 256 (512) 42 and 65 us; 4 frames of 4096 (1024)
// 878 and 1033 us; up to 64 keys, one stage of either, 10.3 and 11.0 us. Beyond one workgroup of 32 queries per compute unit short
// sequences gain little (8 heads of 40, 128 workgroups: 128 tokens 18.5 and 17.2, 192 tokens 21.9 and 21.3), and they lose where
// the problems are no multiple of eight, so that the workgroups of one fetch its keys into several XCDs' L2 (5 heads of 64,
// 128 tokens: 16 frames 21.5 and 19.8, 25 frames 22.9 and 25.4; 192 tokens, 12 frames 27.5 and 29.8; 256 tokens 33.4 and 31.3). The
// two round differently, and a window of queries or a chunk of frames gives the bits of the whole, so the workgroups counted
// are those of the whole problem.
static bool keys_split(int T, int heads, int all_frames) {
  const int64_t problems = (int64_t)heads * all_frames;
  return all_frames > 0 && T > 64 && (T + 127) / 128 * problems <= 128 &&
         ((T + 31) / 32 * problems <= 256 || T > 192 || problems % 8 == 0);
}

template <bool PRE>
static hipError_t spatial_dispatch(hipStream_t s, const float* qk, int ldq, const float* vt, int Tp, float* out, int frames,
                                   int T_tok, int heads, int d, int q0, int nq, int qw, int qstride, int all_frames) {
  const int C = heads * d;
  const float sl = PRE ? 1.f : 1.4426950408889634f / sqrtf((float)d);
  const bool split = keys_split(T_tok, heads, all_frames);
  const int per = split ? 32 : 128;
  dim3 grid((nq + per - 1) / per, heads, frames);
#define LC_ARGS qk, ldq, vt, Tp, out, T_tok, C, q0, nq, qw, qstride, sl
#define LC_GO(D)                                                              \
  if (split) spatial_attn_kernel<D, PRE, 4><<<grid, 256, 0, s>>>(LC_ARGS);    \
  else spatial_attn_kernel<D, PRE, 1><<<grid, 256, 0, s>>>(LC_ARGS)
  switch (d) {
    case 8: LC_GO(8); break;
    case 16: LC_GO(16); break;
    case 32: LC_GO(32); break;
    case 40: LC_GO(40); break;
    case 64: LC_GO(64); break;
    default: return hipErrorInvalidValue;
  }
#undef LC_GO
#undef LC_ARGS
  return hipGetLastError();
}

hipError_t launch_spatial_attention(hipStream_t s, int dt, const void* qk, int ldq, const void* vt, int Tp, void* out,
                                    int frames, int T, int heads, int d, int q0, int q1, int q_prescaled, int all_frames) {
  if (q1 <= q0) return hipSuccess;
  return launch_spatial_attention_window(s, dt, qk, ldq, vt, Tp, out, frames, T, heads, d, q0, q1 - q0, q1 - q0, 0,
                                         q_prescaled, all_frames);
}

hipError_t launch_spatial_attention_window(hipStream_t s, int dt, const void* qk, int ldq, const void* vt, int Tp, void* out,
                                           int frames, int T, int heads, int d, int q0, int nq, int qw, int qstride,
                                           int q_prescaled, int all_frames) {
  if (frames <= 0 || nq <= 0) return hipSuccess;
  if (Tp % kKeys != 0 || Tp < T || qw <= 0 || q0 < 0) return hipErrorInvalidValue;
  {  // the last query must be a token of the frame
    const int r = (nq - 1) / qw;
    if ((int64_t)q0 + (int64_t)r * qstride + (nq - 1 - r * qw) >= T) return hipErrorInvalidValue;
  }
#define LC_ARGS(TT) s, (const TT*)qk, ldq, (const TT*)vt, Tp, (TT*)out, frames, T, heads, d, q0, nq, qw, qstride
  if (dt == kBF16) return q_prescaled ? ring_dispatch<true, false>(LC_ARGS(bf16_t)) : ring_dispatch<false, false>(LC_ARGS(bf16_t));
  return q_prescaled ? spatial_dispatch<true>(LC_ARGS(float), all_frames) : spatial_dispatch<false>(LC_ARGS(float), all_frames);
#undef LC_ARGS
}

// Cross-attention: queries q[frames*Tq] (stride ldq, head h at column h*d) against keys k[(frames/kv_div)*Tk] (stride
// ldk) and their V^T [(frames/kv_div)][C][Tp]; out [frames*Tq][C]. Frame f uses the keys of group f / kv_div.
static hipError_t cross_dispatch(hipStream_t s, const float* q, int ldq, const float* k, int ldk, const float* vt, int Tp, float* out,
                                 int frames, int Tq, int Tk, int kv_div, int heads, int d) {
  const int C = heads * d;
  const float sl = 1.f;  // the queries carry the scale
  dim3 grid((Tq + 127) / 128, heads, frames);
#define LC_GO(D) spatial_attn_kernel<D, true, 1, true><<<grid, 256, 0, s>>>(q, ldq, vt, Tp, out, Tq, C, 0, Tq, Tq, 0, sl, k, ldk, Tk, kv_div)
  switch (d) {
    case 8: LC_GO(8); break;
    case 16: LC_GO(16); break;
    case 32: LC_GO(32); break;
    case 40: LC_GO(40); break;
    case 64: LC_GO(64); break;
    default: return hipErrorInvalidValue;
  }
#undef LC_GO
  return hipGetLastError();
}
hipError_t launch_cross_attention(hipStream_t s, int dt, const void* q, int ldq, const void* k, int ldk, const void* vt, int Tp,
                                  void* out, int frames, int Tq, int Tk, int kv_div, int heads, int d) {
  if (frames <= 0 || Tq <= 0) return hipSuccess;
  if (Tk <= 0 || kv_div <= 0 || frames % kv_div || Tp % kKeys != 0 || Tp < Tk) return hipErrorInvalidValue;
  if (dt == kBF16)
    return ring_dispatch<true, true>(s, (const bf16_t*)q, ldq, (const bf16_t*)vt, Tp, (bf16_t*)out, frames, Tq, heads, d, 0, Tq, Tq, 0,
                                      (const bf16_t*)k, ldk, Tk, kv_div);
  return cross_dispatch(s, (const float*)q, ldq, (const float*)k, ldk, (const float*)vt, Tp, (float*)out, frames, Tq, Tk, kv_div,
                               heads, d);
}

// V^T in the layout the spatial kernel stages: vt[frame][c][vcol(t)] = v[frame*T + t][c] (v rows of stride ldv)
template <class T>
__global__ __launch_bounds__(256) void make_vt_kernel(const T* __restrict__ v, int ldv, T* __restrict__ vt, int T_tok,
                                                      int Tp, int C) {
  __shared__ T tile[32][33];
  const int f = blockIdx.z, t0 = blockIdx.x * 32, c0 = blockIdx.y * 32;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  for (int k = ty; k < 32; k += 8)
    if (t0 + k < T_tok && c0 + tx < C) tile[k][tx] = v[((int64_t)f * T_tok + t0 + k) * ldv + c0 + tx];
  __syncthreads();
  for (int k = ty; k < 32; k += 8) {
    const int t = t0 + tx;
    if (c0 + k < C && t < T_tok) vt[((int64_t)f * C + c0 + k) * Tp + (t & ~63) + vcol<T>(t & 63)] = tile[tx][k];
  }
}
hipError_t launch_make_vt(hipStream_t s, int dt, const void* v, int ldv, void* vt, int frames, int T, int Tp, int C) {
  if (frames <= 0) return hipSuccess;
  dim3 grid((T + 31) / 32, (C + 31) / 32, frames);
  if (dt == kBF16) make_vt_kernel<bf16_t><<<grid, 256, 0, s>>>((const bf16_t*)v, ldv, (bf16_t*)vt, T, Tp, C);
  else make_vt_kernel<float><<<grid, 256, 0, s>>>((const float*)v, ldv, (float*)vt, T, Tp, C);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// Temporal attention over the F frames of one spatial position. A workgroup takes `np` consecutive
// positions of one batch element and brings the q,k,v rows of all F frames at those positions into
// LDS once, with LDS-direct loads (F x np rows of 3C elements; the rows of one frame are contiguous
// in memory). Then thread = (position, query frame f, head h), h fastest: per key frame every lane of
// a wavefront reads the same row and neighbouring lanes neighbouring head slices of it, so the LDS
// reads are broadcasts or conflict-free, where the same loop over global memory had every thread
// pull all F key and value rows through the vector cache again.
// ---------------------------------------------------------------------------------------------
template <class T, int D>
__global__ __launch_bounds__(256) void temporal_attn_kernel(const T* __restrict__ qkv, T* __restrict__ out, int F,
                                                            int P, int heads, int np, float scale_log2e) {
  constexpr int VEC = Vec16<T>::N;
  constexpr int PK = D / VEC;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int C = heads * D, ld = 3 * C;
  const int tid = threadIdx.x, wid = tid >> 6;
  const int b = blockIdx.y, p0 = blockIdx.x * np;
  const int npv = min(np, P - p0);  // positions of this workgroup that exist
  // LDS image [f][np][ld], filled 16 bytes per lane: packet q = (frame, position, packet of the row)
  const int ppr = ld / VEC;         // packets per row
  const int total = F * np * ppr;
  for (int q0 = 0; q0 < total; q0 += 256) {
    const int q = min(q0 + tid, total - 1);
    const int row = q / ppr, pk = q - row * ppr;
    const int f = row / np, pos = min(row - f * np, npv - 1);  // positions beyond the end: a copy nobody reads
    const T* src = qkv + ((int64_t)(b * F + f) * P + p0 + pos) * ld + pk * VEC;
#ifdef __HIP_DEVICE_COMPILE__  // the host pass only needs the kernel's stub; it does not know this builtin
    __builtin_amdgcn_global_load_lds(src, smem + (q0 + wid * 64) * 16, 16, 0, 0);
#else
    (void)src;
#endif
  }
  __builtin_amdgcn_s_waitcnt(0);  // every counter at zero: the rows have landed
  __syncthreads();

  const T* rows = reinterpret_cast<const T*>(smem);
  const int items = npv * F * heads;
  for (int item = tid; item < items; item += 256) {
    const int h = item % heads;
    const int f = (item / heads) % F;
    const int pos = item / (heads * F);
    const T* qrow = rows + (int64_t)(f * np + pos) * ld + h * D;
    float q[D];
#pragma unroll
    for (int k = 0; k < PK; ++k) {
      Vec16<T> v = load16(qrow + k * VEC);
#pragma unroll
      for (int e = 0; e < VEC; ++e) q[k * VEC + e] = v.get(e) * scale_log2e;
    }
    float acc[D];
#pragma unroll
    for (int e = 0; e < D; ++e) acc[e] = 0.f;
    float m = -INFINITY, l = 0.f;
    for (int g = 0; g < F; ++g) {
      const T* krow = rows + (int64_t)(g * np + pos) * ld + C + h * D;
      float s = 0.f;
#pragma unroll
      for (int k = 0; k < PK; ++k) {
        Vec16<T> v = load16(krow + k * VEC);
#pragma unroll
        for (int e = 0; e < VEC; ++e) s = fmaf(q[k * VEC + e], v.get(e), s);
      }
      const float m_new = fmaxf(m, s);
      const float alpha = exp2f(m - m_new);
      const float pe = exp2f(s - m_new);
      m = m_new;
      l = l * alpha + pe;
      const T* vrow = krow + C;
#pragma unroll
      for (int k = 0; k < PK; ++k) {
        Vec16<T> v = load16(vrow + k * VEC);
#pragma unroll
        for (int e = 0; e < VEC; ++e) acc[k * VEC + e] = fmaf(acc[k * VEC + e], alpha, pe * v.get(e));
      }
    }
    const float inv = 1.f / l;
    T* orow = out + ((int64_t)(b * F + f) * P + p0 + pos) * C + h * D;
#pragma unroll
    for (int k = 0; k < PK; ++k) {
      Vec16<T> v;
#pragma unroll
      for (int e = 0; e < VEC; ++e) v.set(e, acc[k * VEC + e] * inv);
      store16(orow + k * VEC, v);
    }
  }
}

// The bf16 case with F <= 16 frames on the matrix cores: the score tile of one (position, head) fits one
// 16 x 16 MFMA tile, so a wavefront takes (position, head) pairs whole instead of a thread taking one query
// (frames beyond F: rows read again from frame F - 1, masked as keys, not stored as queries).
//   S^T[key][query] = K Q^T      16 x 16 x 32 MFMAs over d (packets beyond d are zeros); the lane ends up with
//                                keys 4 (lane / 16) .. + 3 of query lane % 16
//   softmax over the keys        in the lane and across the four lane groups (two shuffles), exact (all 16 keys at once)
//   O^T[d][query] = V^T P^T      16 x 16 x 16 MFMAs, one per 16 channels: the accumulator layout of S^T is the
//                                operand layout of P^T as it stands; V^T is read from the staged rows two bytes
//                                at a time (the four keys of a lane sit in four rows)
// and stores 8 bytes (4 channels of one query frame) per lane. The staging is the one of the kernel above.
// The vector kernel spends 3200 instructions per wavefront on 4 such pairs; this one about 100 on one.
template <int D>
__global__ __launch_bounds__(256) void temporal_attn_mfma_kernel(const bf16_t* __restrict__ qkv, bf16_t* __restrict__ out,
                                                                 int F, int P, int heads, int np, float scale_log2e) {
  static_assert(D % 8 == 0, "whole 16-byte packets per head");
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int C = heads * D, ld = 3 * C;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int b = blockIdx.y, p0 = blockIdx.x * np;
  const int npv = min(np, P - p0);
  const int ppr = ld / 8;
  const int total = F * np * ppr;
  for (int q0 = 0; q0 < total; q0 += 256) {
    const int q = min(q0 + tid, total - 1);
    const int row = q / ppr, pk = q - row * ppr;
    const int f = row / np, pos = min(row - f * np, npv - 1);  // positions beyond the end: a copy nobody reads
    const bf16_t* src = qkv + ((int64_t)(b * F + f) * P + p0 + pos) * ld + pk * 8;
#ifdef __HIP_DEVICE_COMPILE__
    __builtin_amdgcn_global_load_lds(src, smem + (q0 + wid * 64) * 16, 16, 0, 0);
#else
    (void)src;
#endif
  }
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();

  const bf16_t* rows = reinterpret_cast<const bf16_t*>(smem);
  const int i16 = lane & 15, g = lane >> 4;
  const int tasks = npv * heads;
  for (int task = wid; task < tasks; task += 4) {  // uniform over the wavefront
    const int h = task % heads, pos = task / heads;
    const bf16_t* qrow = rows + (min(i16, F - 1) * np + pos) * ld + h * D;  // frame i16: as query (B operand) and, + C, as key (A)
    f32x4 st = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int sl = 0; sl < (D + 31) / 32; ++sl) {
      const int d0 = sl * 32 + 8 * g;
      bf16x8 ka, qb;
#pragma unroll
      for (int e = 0; e < 8; ++e) ka[e] = qb[e] = (bf16_t)0.f;
      if (d0 < D) {
        ka = *reinterpret_cast<const bf16x8*>(qrow + C + d0);
        qb = *reinterpret_cast<const bf16x8*>(qrow + d0);
      }
      st = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ka, qb, st, 0, 0, 0);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (4 * g + r >= F) st[r] = -INFINITY;  // no such key (key 0 always exists: the maximum is finite)
    float mx = fmaxf(fmaxf(st[0], st[1]), fmaxf(st[2], st[3]));
    mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    float pe[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) pe[r] = exp2f((st[r] - mx) * scale_log2e);
    float l = (pe[0] + pe[1]) + (pe[2] + pe[3]);
    l += __shfl_xor(l, 16, 64);
    l += __shfl_xor(l, 32, 64);
    const float inv = 1.f / l;
    bf16x4 pb;
#pragma unroll
    for (int r = 0; r < 4; ++r) pb[r] = static_cast<bf16_t>(pe[r]);
    const bf16_t* vbase = rows + pos * ld + 2 * C + h * D;  // + key * np * ld
    bf16_t* obase = out + ((int64_t)(b * F + i16) * P + p0 + pos) * C + h * D;
#pragma unroll
    for (int t = 0; t < (D + 15) / 16; ++t) {
      const int dv = min(t * 16 + i16, D - 1);  // channels beyond the head: a copy, computed and dropped
      bf16x4 va;
#pragma unroll
      for (int r = 0; r < 4; ++r) va[r] = vbase[min(4 * g + r, F - 1) * np * ld + dv];  // (weight 0 beyond F)
      const f32x4 o = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(va, pb, f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
      const int dd = t * 16 + 4 * g;  // this lane's four channels of query frame i16
      if (dd < D && i16 < F) {
        bf16x4 ov;
#pragma unroll
        for (int r = 0; r < 4; ++r) ov[r] = static_cast<bf16_t>(o[r] * inv);
        *reinterpret_cast<bf16x4*>(obase + dd) = ov;
      }
    }
  }
}

// The same for 17 <= F <= 32 frames on 32 x 32 MFMA tiles. The lane ends up with 16 keys of query lane % 32:
// keys 8 (r / 4) + 4 (lane / 32) + r % 4, r = 0..15. The contraction of O^T = V^T P^T runs over the keys in two slabs
// of 16 whose order inside a slab is free as long as both operands use the same one: slot j of lane group hh in
// slab u stands for key 16 u + 8 (j / 4) + 4 hh + j % 4, which is where accumulator r = 8 u + j already sits.
template <int D>
__global__ __launch_bounds__(256) void temporal_attn_mfma32_kernel(const bf16_t* __restrict__ qkv, bf16_t* __restrict__ out,
                                                                   int F, int P, int heads, int np, float scale_log2e) {
  static_assert(D % 8 == 0, "whole 16-byte packets per head");
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int C = heads * D, ld = 3 * C;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int b = blockIdx.y, p0 = blockIdx.x * np;
  const int npv = min(np, P - p0);
  const int ppr = ld / 8;
  const int total = F * np * ppr;
  for (int q0 = 0; q0 < total; q0 += 256) {
    const int q = min(q0 + tid, total - 1);
    const int row = q / ppr, pk = q - row * ppr;
    const int f = row / np, pos = min(row - f * np, npv - 1);  // positions beyond the end: a copy nobody reads
    const bf16_t* src = qkv + ((int64_t)(b * F + f) * P + p0 + pos) * ld + pk * 8;
#ifdef __HIP_DEVICE_COMPILE__
    __builtin_amdgcn_global_load_lds(src, smem + (q0 + wid * 64) * 16, 16, 0, 0);
#else
    (void)src;
#endif
  }
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();

  const bf16_t* rows = reinterpret_cast<const bf16_t*>(smem);
  const int i32 = lane & 31, hh = lane >> 5;
  const int tasks = npv * heads;
  for (int task = wid; task < tasks; task += 4) {  // uniform over the wavefront
    const int h = task % heads, pos = task / heads;
    const bf16_t* qrow = rows + (min(i32, F - 1) * np + pos) * ld + h * D;  // frame i32: as query (B operand) and, + C, as key (A)
    f32x16 st;
#pragma unroll
    for (int r = 0; r < 16; ++r) st[r] = 0.f;
#pragma unroll
    for (int sl = 0; sl < (D + 15) / 16; ++sl) {
      const int d0 = sl * 16 + 8 * hh;
      bf16x8 ka, qb;
#pragma unroll
      for (int e = 0; e < 8; ++e) ka[e] = qb[e] = (bf16_t)0.f;
      if (d0 < D) {
        ka = *reinterpret_cast<const bf16x8*>(qrow + C + d0);
        qb = *reinterpret_cast<const bf16x8*>(qrow + d0);
      }
      st = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka, qb, st, 0, 0, 0);
    }
    float mx = -INFINITY;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      if (8 * (r >> 2) + 4 * hh + (r & 3) >= F) st[r] = -INFINITY;  // no such key (key 0 always exists: the maximum is finite)
      mx = fmaxf(mx, st[r]);
    }
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    float l = 0.f;
    bf16x8 pb[2];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float pe = exp2f((st[r] - mx) * scale_log2e);
      l += pe;
      pb[r >> 3][r & 7] = static_cast<bf16_t>(pe);
    }
    l += __shfl_xor(l, 32, 64);
    const float inv = 1.f / l;
    const bf16_t* vbase = rows + pos * ld + 2 * C + h * D;  // + key * np * ld
    bf16_t* obase = out + ((int64_t)(b * F + i32) * P + p0 + pos) * C + h * D;
#pragma unroll
    for (int t = 0; t < (D + 31) / 32; ++t) {
      const int dv = min(t * 32 + i32, D - 1);  // channels beyond the head: a copy, computed and dropped
      f32x16 o;
#pragma unroll
      for (int r = 0; r < 16; ++r) o[r] = 0.f;
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        bf16x8 va;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const int key = 16 * u + 8 * (j >> 2) + 4 * hh + (j & 3);
          va[j] = vbase[min(key, F - 1) * np * ld + dv];  // (weight 0 beyond F)
        }
        o = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va, pb[u], o, 0, 0, 0);
      }
#pragma unroll
      for (int g4 = 0; g4 < 4; ++g4) {
        const int dd = t * 32 + 8 * g4 + 4 * hh;  // this lane's channels dd .. dd + 3 of query frame i32
        if (dd < D && i32 < F) {
          bf16x4 ov;
#pragma unroll
          for (int r = 0; r < 4; ++r) ov[r] = static_cast<bf16_t>(o[4 * g4 + r] * inv);
          *reinterpret_cast<bf16x4*>(obase + dd) = ov;
        }
      }
    }
  }
}

// The same computation straight from global memory, for frame counts whose rows do not fit in LDS:
// thread = (batch b, position p, query frame f, head h), h fastest.
template <class T, int D>
__global__ __launch_bounds__(256) void temporal_attn_global_kernel(const T* __restrict__ qkv, T* __restrict__ out, int B,
                                                            int F, int P, int heads, float scale_log2e) {
  constexpr int VEC = Vec16<T>::N;
  constexpr int PK = D / VEC;
  const int C = heads * D, ld = 3 * C;
  const int64_t total = (int64_t)B * P * F * heads;
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= total) return;
  const int h = (int)(i % heads);
  int64_t t = i / heads;
  const int f = (int)(t % F);
  t /= F;
  const int p = (int)(t % P);
  const int b = (int)(t / P);
  // row of (frame n, position p) in the frame-major chunk: n * P + p
  const T* qrow = qkv + ((int64_t)(b * F + f) * P + p) * ld + h * D;
  float q[D];
#pragma unroll
  for (int k = 0; k < PK; ++k) {
    Vec16<T> v = load16(qrow + k * VEC);
#pragma unroll
    for (int e = 0; e < VEC; ++e) q[k * VEC + e] = v.get(e) * scale_log2e;
  }
  float acc[D];
#pragma unroll
  for (int e = 0; e < D; ++e) acc[e] = 0.f;
  float m = -INFINITY, l = 0.f;
  for (int g = 0; g < F; ++g) {
    const T* krow = qkv + ((int64_t)(b * F + g) * P + p) * ld + C + h * D;
    float s = 0.f;
#pragma unroll
    for (int k = 0; k < PK; ++k) {
      Vec16<T> v = load16(krow + k * VEC);
#pragma unroll
      for (int e = 0; e < VEC; ++e) s = fmaf(q[k * VEC + e], v.get(e), s);
    }
    const float m_new = fmaxf(m, s);
    const float alpha = exp2f(m - m_new);
    const float pe = exp2f(s - m_new);
    m = m_new;
    l = l * alpha + pe;
    const T* vrow = krow + C;
#pragma unroll
    for (int k = 0; k < PK; ++k) {
      Vec16<T> v = load16(vrow + k * VEC);
#pragma unroll
      for (int e = 0; e < VEC; ++e) acc[k * VEC + e] = fmaf(acc[k * VEC + e], alpha, pe * v.get(e));
    }
  }
  const float inv = 1.f / l;
  T* orow = out + ((int64_t)(b * F + f) * P + p) * C + h * D;
#pragma unroll
  for (int k = 0; k < PK; ++k) {
    Vec16<T> v;
#pragma unroll
    for (int e = 0; e < VEC; ++e) v.set(e, acc[k * VEC + e] * inv);
    store16(orow + k * VEC, v);
  }
}

template <class T, int D>
static hipError_t temporal_run(hipStream_t s, const T* qkv, T* out, int B, int F, int P, int heads, float sl) {
  const int64_t pos_bytes = (int64_t)F * 3 * heads * D * (int64_t)sizeof(T);  // LDS for one position
  if (pos_bytes + 4096 > 150 * 1024) {
    const int64_t total = (int64_t)B * P * F * heads;
    temporal_attn_global_kernel<T, D><<<(unsigned)((total + 255) / 256), 256, 0, s>>>(qkv, out, B, F, P, heads, sl);
    return hipGetLastError();
  }
  // positions per workgroup: two workgroups per compute unit if possible, at most 16 positions
  int np = (int)(32 * 1024 / pos_bytes);
  np = np < 1 ? 1 : (np > 16 ? 16 : np);
  if (np > P) np = P;
  const int64_t packets = (int64_t)F * np * (3 * heads * D / Vec16<T>::N);
  const int lds = (int)((packets + 255) / 256 * 256 * 16);  // whole rounds of 256 lanes land in LDS
  if constexpr (std::is_same<T, bf16_t>::value && D % 8 == 0) {
    if (F >= 8 && F <= 16) {  // (below 8 frames the vector kernel has less to do than a padded tile)
      auto mk = temporal_attn_mfma_kernel<D>;
      static int mk_attr_bytes = 0;  // per instantiation
      if (lds > mk_attr_bytes) {
        hipError_t e = hipFuncSetAttribute((const void*)mk, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        if (e != hipSuccess) return e;
        mk_attr_bytes = lds;
      }
      dim3 grid((unsigned)((P + np - 1) / np), (unsigned)B);
      mk<<<grid, 256, lds, s>>>(qkv, out, F, P, heads, np, sl);
      return hipGetLastError();
    }
    if (F > 16 && F <= 32) {
      auto mk = temporal_attn_mfma32_kernel<D>;
      static int mk32_attr_bytes = 0;  // per instantiation
      if (lds > mk32_attr_bytes) {
        hipError_t e = hipFuncSetAttribute((const void*)mk, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        if (e != hipSuccess) return e;
        mk32_attr_bytes = lds;
      }
      dim3 grid((unsigned)((P + np - 1) / np), (unsigned)B);
      mk<<<grid, 256, lds, s>>>(qkv, out, F, P, heads, np, sl);
      return hipGetLastError();
    }
  }
  auto kern = temporal_attn_kernel<T, D>;
  static int attr_bytes = 0;  // per instantiation
  if (lds > attr_bytes) {
    hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
    attr_bytes = lds;
  }
  dim3 grid((unsigned)((P + np - 1) / np), (unsigned)B);
  kern<<<grid, 256, lds, s>>>(qkv, out, F, P, heads, np, sl);
  return hipGetLastError();
}

template <class T>
static hipError_t temporal_dispatch(hipStream_t s, const T* qkv, T* out, int B, int F, int P, int heads, int d) {
  const float sl = 1.4426950408889634f / sqrtf((float)d);
  switch (d) {
    case 8: return temporal_run<T, 8>(s, qkv, out, B, F, P, heads, sl);
    case 16: return temporal_run<T, 16>(s, qkv, out, B, F, P, heads, sl);
    case 32: return temporal_run<T, 32>(s, qkv, out, B, F, P, heads, sl);
    case 40: return temporal_run<T, 40>(s, qkv, out, B, F, P, heads, sl);
    case 64: return temporal_run<T, 64>(s, qkv, out, B, F, P, heads, sl);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_temporal_attention(hipStream_t s, int dt, const void* qkv, void* out, int B, int F, int P,
                                     int heads, int d) {
  if (B <= 0 || F <= 0 || P <= 0) return hipSuccess;
  if (dt == kBF16) return temporal_dispatch<bf16_t>(s, (const bf16_t*)qkv, (bf16_t*)out, B, F, P, heads, d);
  return temporal_dispatch<float>(s, (const float*)qkv, (float*)out, B, F, P, heads, d);
}

}  // namespace lc
