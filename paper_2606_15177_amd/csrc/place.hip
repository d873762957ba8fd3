// Source-aware expert placement on the GPU: the online greedy of Sec. 5.3
// over the objective of Sec. 5.2, one workgroup per MoE layer.
//
// The statistics it consumes (the source x expert matrix A and the aggregate
// load B, Sec. 5.1) are accumulated on the device by the routing kernels, so
// the placement runs where they already are.  Per layer:
//   1. every thread sums the source-aware volume V_e = sum_s A_{s,e} of its
//      experts and stages B, V, the current ranks x^0 and the source/rank cost
//      matrix D in LDS;
//   2. every thread ranks its experts by hotness (B descending, then V
//      descending, then lower index) by counting the experts ahead of them;
//   3. hottest first, in chunks: wave 0 places a chunk's experts one at a
//      time while the other waves compute the next chunk's placement-
//      independent terms C^comm = sum_s A_{s,e} D_{s,g} and C^mig (zero on
//      the current rank, else M_{e,g} plus M_{e,x0} when x0 is a rank) into
//      the other of two LDS buffers.  Lane g of wave 0 scores rank g with the
//      load term C^load = (L_g + B_e - Lbar)^2 - (L_g - Lbar)^2 that depends
//      on the experts placed before; a butterfly over the lanes picks the
//      lowest score (ties: the current rank, then fewer experts placed, then
//      the lower rank);
//   4. the placement, each rank's experts and the objective's three terms of
//      the result are written out.
// What bounds it is the chain of E dependent steps.  A step's winner decides
// the next step's score of one lane only, so every lane computes its next
// score for both outcomes while the minimum of this one is found, and the
// chain per step is the butterfly, one comparison and a select; ties, rare in
// fp64, leave the main path.  48 layers of 128 experts on 8 ranks and 58 of 256
// on 64 took 44 and 245 us with each score computed after the last winner, the
// tie phase in every step and the terms between the chunks, and take 36 and
// 101 us: 200 and 290 ns per step, about 90 instructions of one wave.
// Scores are fp64 and evaluated left to right without contraction into fused
// multiply-adds, so the chosen rank is the one any IEEE fp64 evaluation of the
// same expressions chooses.
#include "common.h"
#include "kernels.h"

#pragma clang fp contract(off)

namespace moe {
namespace {

constexpr int kPlaceWaves = 16;  // of a layer's workgroup (WAVES below) at most, see place_waves

struct PlaceKernelArgs {
  const int64_t* A;
  const int64_t* B;
  const double* D;
  const double* M;
  const int32_t* x0;
  int32_t* x;
  int32_t* rank_experts;
  double* cost;
  double alpha, beta, gamma, m_uniform;
  int S, E, G, slots, chunk;
  int cap[kPlaceMaxRanks];
};

typedef int64_t i64x2 __attribute__((ext_vector_type(2)));

struct PlaceLds {
  i64x2* bv;       // [E] (B, V) of each expert: aggregate load, source-aware volume
  double* D;       // [S*G]
  double2* terms;  // [2][chunk*G] (C^comm, C^mig) of a chunk, two buffers
  int64_t* bo;     // [E] B of the expert in hotness position i (FAST: as a double)
  int32_t* order;  // [E] expert in hotness position i
  int32_t* ho;     // [E] x^0 of the expert in hotness position i
  int32_t* xpos;   // [E] rank chosen for hotness position i
  int32_t* xs;     // [E] rank chosen for each expert
  int32_t* fill;   // [kPlaceMaxRanks] experts placed per rank
  int64_t* red_i;  // [2 * WAVES]
  double* A;       // [S*E] this layer's counts when they fit (a_staged), else
                   // piece_a values per wave: a piece of its experts' columns
};

// The layer's A is staged in LDS when it takes at most this many bytes.
constexpr size_t kStageABytes = 32 * 1024;
__host__ __device__ constexpr int piece_a(int waves) { return static_cast<int>(kStageABytes / sizeof(double)) / waves; }
__host__ __device__ inline bool a_staged(int S, int E) {
  return static_cast<size_t>(S) * E * sizeof(int64_t) <= kStageABytes;
}

// Experts that a wave takes at once in the terms phase: as many as fit its
// lanes beside their ranks.
__host__ __device__ inline int place_batch_experts(int G) {
  int gp = 1;
  while (gp < G) gp *= 2;
  return kWave / gp;
}

// Experts per chunk: at most 32, so that the first steps start early, and no
// more than the waves beside wave 0 prepare in one batch each.
__host__ __device__ inline int place_chunk_experts(int E, int G, int waves) {
  int c = (waves - 1) * place_batch_experts(G);
  c = c < 32 ? c : 32;
  return c < E ? c : E;
}

__host__ __device__ inline size_t align16(size_t v) { return (v + 15) & ~static_cast<size_t>(15); }

// Byte offsets of the LDS carve; the same function sizes the launch.
__host__ __device__ inline size_t place_lds_layout(int S, int E, int G, int chunk, int waves, size_t* off) {
  size_t o = 0;
  off[0] = o; o = align16(o + 16 * static_cast<size_t>(E));                 // bv
  off[1] = o; o = align16(o + sizeof(double) * S * G);                      // D
  off[2] = o; o = align16(o + sizeof(double2) * 2 * chunk * G);             // terms
  off[3] = o; o = align16(o + sizeof(int64_t) * E);                         // bo
  off[4] = o; o = align16(o + sizeof(int32_t) * E);                         // order
  off[5] = o; o = align16(o + sizeof(int32_t) * E);                         // ho
  off[6] = o; o = align16(o + sizeof(int32_t) * E);                         // xpos
  off[7] = o; o = align16(o + sizeof(int32_t) * E);                         // xs
  off[8] = o; o = align16(o + sizeof(int32_t) * kPlaceMaxRanks);            // fill
  off[9] = o; o = align16(o + sizeof(int64_t) * 2 * waves);                 // red_i
  off[10] = o;
  o = align16(o + (a_staged(S, E) ? sizeof(double) * S * E : kStageABytes));  // A or its pieces
  return o;
}
constexpr int kLdsParts = 11;

__device__ __forceinline__ double mig_cost(const PlaceKernelArgs& a, int l, int e, int g) {
  return a.M ? a.M[(static_cast<size_t>(l) * a.E + e) * a.G + g] : a.m_uniform;
}

// C^mig of expert e on rank g: zero on its current rank, else the two
// indicator changes M_{e,g} and (when it has a rank) M_{e,home}.
__device__ __forceinline__ double mig_term(const PlaceKernelArgs& a, int l, int e, int g, int home) {
  const bool home_ok = home >= 0 && home < a.G;
  if (home_ok && g == home) return 0.0;
  double m = mig_cost(a, l, e, g);
  if (home_ok) m = m + mig_cost(a, l, e, home);
  return m;
}

// comm + sum_s A_{s,e} D_{s,g} over n sources, in s order, with A_{s,e} =
// col[s * stride] (exactly converted counts) and D_{s,g} = d[s * G];
// eight loads are issued before their products are summed.
__device__ __forceinline__ double comm_term(double comm, const double* col, int stride, const double* d, int n,
                                            int G) {
  int src = 0;
  for (; src + 8 <= n; src += 8) {
    double av[8], dv[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      av[j] = col[(src + j) * stride];
      dv[j] = d[(src + j) * G];
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) comm = comm + av[j] * dv[j];
  }
  for (; src < n; ++src) comm = comm + col[src * stride] * d[src * G];
  return comm;
}

// Orders a wave's own LDS accesses (they complete in order).
__device__ __forceinline__ void wave_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// One wave's share (experts w0, w0 + nw, ... in batches) of a chunk's terms.
// A wave takes as many experts at once as fit its lanes beside their ranks
// and, when A is not staged whole, as leave each a piece of its column.
template <int WAVES>
__device__ __forceinline__ void chunk_terms(const PlaceKernelArgs& a, const PlaceLds& s, int l, int c0, int nc,
                                            int t0, int w0, int nw, int wave, int lane, bool staged) {
  constexpr int kPiece = piece_a(WAVES);
  const int S = a.S, E = a.E, G = a.G;
  const int64_t* A_l = a.A + static_cast<size_t>(l) * S * E;
  int per = place_batch_experts(G);
  const int gp = kWave / per;
  const int sub = lane / gp, g = lane % gp;
  if (!staged)
    while (per > 1 && per * S > kPiece) per /= 2;
  double* own = s.A + wave * kPiece;
  auto expert_at = [&](int i) { return s.order[c0 + (i < nc ? i : nc - 1)]; };
  auto put = [&](int i, double comm) {
    if (sub < per && i < nc && g < G)
      s.terms[t0 + i * G + g] = make_double2(comm, mig_term(a, l, expert_at(i), g, s.ho[c0 + i]));
  };
  if (staged) {
    for (int b = w0 * per; b < nc; b += nw * per)
      put(b + sub, comm_term(0.0, s.A + expert_at(b + sub), E, s.D + min(g, G - 1), S, G));
  } else if (per * S <= kPiece) {
    // the columns of several batches at once, so that their loads overlap
    const int col = per * S, bats = kPiece / col;
    for (int b0 = w0 * per; b0 < nc; b0 += bats * nw * per) {
      const int nb = min(bats, ceil_div(nc - b0, nw * per));
#pragma unroll 4
      for (int q = lane; q < nb * col; q += kWave) {
        const int k = q / S;  // column of the staged batches
        const int i = b0 + (k / per) * nw * per + k % per;
        own[q] = static_cast<double>(A_l[static_cast<size_t>(q - k * S) * E + expert_at(i)]);
      }
      wave_fence();
      for (int k = 0; k < nb; ++k)
        put(b0 + k * nw * per + sub, comm_term(0.0, own + (k * per + min(sub, per - 1)) * S, 1, s.D + min(g, G - 1), S, G));
      wave_fence();
    }
  } else {
    // a column longer than the wave's piece (per == 1): piece by piece
    for (int b = w0; b < nc; b += nw) {
      double comm = 0.0;
      for (int s0 = 0; s0 < S; s0 += kPiece) {
        const int n = min(kPiece, S - s0);
#pragma unroll 4
        for (int q = lane; q < n; q += kWave)
          own[q] = static_cast<double>(A_l[static_cast<size_t>(s0 + q) * E + expert_at(b)]);
        wave_fence();
        comm = comm_term(comm, own, 1, s.D + s0 * G + min(g, G - 1), n, G);
        wave_fence();
      }
      put(b + sub, comm);
    }
  }
}

template <int CTRL>
__device__ __forceinline__ uint32_t dpp_u32(uint32_t v) {
  // every lane has a source under these controls: no old value to keep
  return static_cast<uint32_t>(__builtin_amdgcn_mov_dpp(static_cast<int>(v), CTRL, 0xf, 0xf, true));
}
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v) {
  const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xf, 0xf, true);
  return __hiloint2double(hi, lo);
}
// The minimum of two scores.  A score may be a quiet NaN (never a signalling
// one: it is the result of arithmetic), and the instruction then returns the
// other operand, so a NaN loses; a minimum over NaNs alone equals no score and
// an infinite one is not looked for, and both go to the tie path, which counts
// a NaN as +inf.  Of -0.0 and +0.0 it may return either, which the equality test
// with the scores treats alike.  The builtin would first canonicalise both
// operands (two more instructions of the chain per level), as it cannot know
// that they are no signalling NaNs.
__device__ __forceinline__ double min_f64(double a, double b) {
  double r;
  asm("v_min_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
__device__ __forceinline__ uint32_t min_u32(uint32_t a, uint32_t b) { return b < a ? b : a; }

// DPP controls: swap neighbours, swap pairs, mirror each half row (lane i <->
// 7 - i), mirror each row (lane i <-> 15 - i).  After the four levels every
// lane of a 16-lane row holds the row's minimum.
constexpr int kDppSwap1 = 0xB1;   // quad_perm [1, 0, 3, 2]
constexpr int kDppSwap2 = 0x4E;   // quad_perm [2, 3, 0, 1]
constexpr int kDppHalfMirror = 0x141;
constexpr int kDppMirror = 0x140;

// The minimum of each lane's value and that of the lane ROWS (16 or 32) away:
// the swaps exchange odd rows (the upper half) of one copy with even rows
// (the lower half) of the other, which leaves the pair's two values in every
// lane, without a trip through the LDS crossbar.
template <int ROWS>
__device__ __forceinline__ double min_swapped_f64(double v) {
  const unsigned lo = static_cast<unsigned>(__double2loint(v)), hi = static_cast<unsigned>(__double2hiint(v));
  if constexpr (ROWS == 16) {
    const auto l = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
    const auto h = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
    return min_f64(__hiloint2double(static_cast<int>(h[0]), static_cast<int>(l[0])),
                   __hiloint2double(static_cast<int>(h[1]), static_cast<int>(l[1])));
  } else {
    const auto l = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
    const auto h = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
    return min_f64(__hiloint2double(static_cast<int>(h[0]), static_cast<int>(l[0])),
                   __hiloint2double(static_cast<int>(h[1]), static_cast<int>(l[1])));
  }
}

// Minimum over the first 2^LEVELS lanes (every lane among them gets it;
// lanes past G must hold values that do not win).
__device__ __forceinline__ double lanes_min_level(double v, int level) {
  switch (level) {
    case 0: return min_f64(v, dpp_f64<kDppSwap1>(v));
    case 1: return min_f64(v, dpp_f64<kDppSwap2>(v));
    case 2: return min_f64(v, dpp_f64<kDppHalfMirror>(v));
    case 3: return min_f64(v, dpp_f64<kDppMirror>(v));
    case 4: return min_swapped_f64<16>(v);
    default: return min_swapped_f64<32>(v);
  }
}
template <int LEVELS>
__device__ __forceinline__ double lanes_min_f64(double v) {
#pragma unroll
  for (int lv = 0; lv < LEVELS; ++lv) v = lanes_min_level(v, lv);
  return v;
}
template <int LEVELS>
__device__ __forceinline__ uint32_t lanes_min_u32(uint32_t v) {
  if constexpr (LEVELS > 0) v = min_u32(v, dpp_u32<kDppSwap1>(v));
  if constexpr (LEVELS > 1) v = min_u32(v, dpp_u32<kDppSwap2>(v));
  if constexpr (LEVELS > 2) v = min_u32(v, dpp_u32<kDppHalfMirror>(v));
  if constexpr (LEVELS > 3) v = min_u32(v, dpp_u32<kDppMirror>(v));
  if constexpr (LEVELS > 4) v = min_u32(v, __shfl_xor(v, 16));
  if constexpr (LEVELS > 5) v = min_u32(v, __shfl_xor(v, 32));
  return v;
}

// State of rank g, held by lane g of wave 0: experts placed, load placed (as
// int64, or as an exact double in FAST mode) and u2 = (L_g - Lbar)^2.  comm
// and mig are a lane's share of the placed experts' terms.
struct RankState {
  int placed;
  int64_t load;
  double loadd, u2, comm, mig;
};

// Wave 0's greedy over one chunk of nc <= 32 hotness positions from c0.
// FAST requires every partial load to be an integer below 2^53, so that
// (double)(L + B) equals the double sum of the two exact conversions.
template <bool FAST, int LEVELS>
__device__ __forceinline__ void place_chunk_steps(const PlaceKernelArgs& a, const PlaceLds& s, int t0, int c0, int nc,
                                                  double mean, int lane, int cap_g, RankState& r) {
  const int G = a.G;
  const int gl = lane < G ? lane : G - 1;   // lanes past G read a valid term and stay closed
  const double2* const terms = s.terms + t0;  // (indexed from s: a chosen pointer would make these generic loads)
  struct Load {
    int64_t i;
    double d;
  };
  auto add_load = [&](const Load& have, int64_t be) {
    if constexpr (FAST) return Load{0, have.d + __longlong_as_double(be)};
    else return Load{have.i + be, 0.0};
  };
  auto over_mean = [&](const Load& ld) { return (FAST ? ld.d : static_cast<double>(ld.i)) - mean; };
  // A NaN score needs no care in the main path: the minimum passes it over
  // and it equals no minimum.
  const double inf = __builtin_inf();
  const uint64_t ranks = G < 64 ? (1ull << G) - 1 : ~0ull;
  double2 t = terms[gl];
  int64_t be = s.bo[c0];
  int home = s.ho[c0];
  // the operands of step i + 1, read one step before they are used
  double2 t1 = terms[min(1, nc - 1) * G + gl];
  int64_t be1 = s.bo[c0 + min(1, nc - 1)];
  int home1 = s.ho[c0 + min(1, nc - 1)];
  Load have{r.load, r.loadd}, ld;
  double u2 = r.u2, vv;
  int placed = r.placed;
  ld = add_load(have, be);
  vv = over_mean(ld);
  vv = vv * vv;
  double sc = a.alpha * t.x;
  sc = sc + a.beta * (vv - u2);
  sc = sc + a.gamma * t.y;
  sc = placed < cap_g ? sc : inf;
  uint32_t won_steps = 0;  // bit i: this rank won step i
  // The loop at a fixed place in its cache lines: left where the code before it
  // ends, the same loop takes up to 5% longer (48 layers of 128 experts on 8
  // ranks 36.0 us so, 36.4 to 37.8 up to 28 bytes further on).
  asm volatile(".p2align 6");
  for (int i = 0; i < nc; ++i) {
    const int i2 = min(i + 2, nc - 1);
    const double2 t2 = terms[i2 * G + gl];
    const int64_t be2 = s.bo[c0 + i2];
    const int home2 = s.ho[c0 + i2];
    // step i + 1's score if this rank loses step i (l), and if it wins it (w)
    const double at = a.alpha * t1.x, gt = a.gamma * t1.y;
    const Load ld_l = add_load(have, be1), ld_w = add_load(ld, be1);
    double vv_l = over_mean(ld_l), vv_w = over_mean(ld_w);
    vv_l = vv_l * vv_l;
    vv_w = vv_w * vv_w;
    double sc_l = at + a.beta * (vv_l - u2), sc_w = at + a.beta * (vv_w - vv);
    sc_l = sc_l + gt;
    sc_w = sc_w + gt;

    const double best = lanes_min_f64<LEVELS>(sc);
    // (groups of lanes past G have minima of their own; an infinite minimum
    // may stand for a NaN or a full rank and goes to the tie path)
    uint64_t m = __ballot((sc == best) & (best < inf)) & ranks;
    // both next scores are computed before the branch, beside the minimum
    asm volatile("" : "+v"(sc_l), "+v"(sc_w));
    if (__popcll(m) != 1) {
      // ties: a full rank loses, then the current rank wins, then fewer
      // experts placed, then the lower rank; a NaN score counts as +inf
      const double scn = sc == sc ? sc : inf;
      const double bestn = lanes_min_f64<LEVELS>(scn);
      const uint32_t key = (placed < cap_g ? 0u : 0x80000000u) | (lane == home ? 0u : 0x40000000u) |
                           (static_cast<uint32_t>(placed) << 6) | static_cast<uint32_t>(lane);
      const uint32_t k = lanes_min_u32<LEVELS>(scn == bestn ? key : 0xffffffffu);
      m = 1ull << (__builtin_amdgcn_readfirstlane(k) & 63u);
    }
    const bool won = __builtin_amdgcn_inverse_ballot_w64(m);
    won_steps |= won ? 1u << i : 0u;
    placed += won ? 1 : 0;
    if constexpr (FAST) have.d = won ? ld.d : have.d;
    else have.i = won ? ld.i : have.i;
    u2 = won ? vv : u2;   // the new load's (L - Lbar)^2
    if constexpr (FAST) ld.d = won ? ld_w.d : ld_l.d;
    else ld.i = won ? ld_w.i : ld_l.i;
    vv = won ? vv_w : vv_l;
    sc = won ? sc_w : sc_l;
    sc = placed < cap_g ? sc : inf;
    t1 = t2;
    be1 = be2;
    home = home1;
    home1 = home2;
  }
  r.placed = placed;
  r.load = have.i;
  r.loadd = have.d;
  r.u2 = u2;
  while (won_steps != 0) {
    const int i = __builtin_ctz(won_steps);
    won_steps &= won_steps - 1;
    s.xpos[c0 + i] = lane;
    const double2 own = terms[i * G + lane];
    r.comm = r.comm + own.x;
    r.mig = r.mig + own.y;
  }
}

__device__ __forceinline__ int64_t wave_sum_i64(int64_t v) {
  for (int off = kWave / 2; off > 0; off >>= 1) v += __shfl_xor(v, off);
  return v;
}

__device__ __forceinline__ double wave_sum_f64(double v) {
  for (int off = kWave / 2; off > 0; off >>= 1) v = v + __shfl_xor(v, off);
  return v;
}

template <int WAVES>
__global__ __launch_bounds__(WAVES* kWave) void place_kernel(PlaceKernelArgs a) {
  constexpr int kThreads = WAVES * kWave;
  extern __shared__ __align__(16) unsigned char place_smem[];
  const int l = blockIdx.x;
  const int tid = threadIdx.x;
  const int lane = tid & (kWave - 1);
  const int wave = tid / kWave;
  const int S = a.S, E = a.E, G = a.G;
  const int64_t* A_l = a.A + static_cast<size_t>(l) * S * E;
  const int32_t* x0_l = a.x0 + static_cast<size_t>(l) * E;

  size_t off[kLdsParts];
  place_lds_layout(S, E, G, a.chunk, WAVES, off);
  PlaceLds s;
  s.bv = reinterpret_cast<i64x2*>(place_smem + off[0]);
  s.D = reinterpret_cast<double*>(place_smem + off[1]);
  s.terms = reinterpret_cast<double2*>(place_smem + off[2]);
  s.bo = reinterpret_cast<int64_t*>(place_smem + off[3]);
  s.order = reinterpret_cast<int32_t*>(place_smem + off[4]);
  s.ho = reinterpret_cast<int32_t*>(place_smem + off[5]);
  s.xpos = reinterpret_cast<int32_t*>(place_smem + off[6]);
  s.xs = reinterpret_cast<int32_t*>(place_smem + off[7]);
  s.fill = reinterpret_cast<int32_t*>(place_smem + off[8]);
  s.red_i = reinterpret_cast<int64_t*>(place_smem + off[9]);
  const bool staged = a_staged(S, E);
  s.A = reinterpret_cast<double*>(place_smem + off[10]);

  // 1. hotness signals, D, and the layer's A when it fits in LDS
  int64_t part = 0;
  int negative = 0;
  for (int e = tid; e < E; e += kThreads) {
    int64_t v = 0;
#pragma unroll 16
    for (int src = 0; src < S; ++src) {
      const int64_t c = A_l[static_cast<size_t>(src) * E + e];
      if (staged) s.A[src * E + e] = static_cast<double>(c);
      v += c;
    }
    const int64_t b = a.B ? a.B[static_cast<size_t>(l) * E + e] : v;
    i64x2 bv;
    bv.x = b;
    bv.y = v;
    s.bv[e] = bv;
    part += b;
    negative |= static_cast<int>(b < 0);
  }
  for (int i = tid; i < S * G; i += kThreads) s.D[i] = a.D[i];
  part = wave_sum_i64(part);
  const int64_t neg_w = wave_sum_i64(negative);
  if (lane == 0) {
    s.red_i[wave] = part;
    s.red_i[WAVES + wave] = neg_w;
  }
  __syncthreads();
  int64_t total = 0, n_negative = 0;
  for (int w = 0; w < WAVES; ++w) {
    total += s.red_i[w];
    n_negative += s.red_i[WAVES + w];
  }
  // every expert is placed, so the final average rank load is known up front
  const double mean = static_cast<double>(total) / G;
  // non-negative loads whose total is below 2^53: every partial load is an
  // exactly representable integer
  const bool fast = n_negative == 0 && total < (int64_t{1} << 53);

  // 2. hotness order: an expert's position is the number of experts ahead of
  // it; tpe consecutive lanes split the count of one expert
  int tpe = 1;
  while (tpe < kWave && tpe * 2 * E <= kThreads) tpe *= 2;
  for (int idx = tid; idx < E * tpe; idx += kThreads) {
    const int e = idx / tpe;
    const int sub = idx - e * tpe;
    const i64x2 me = s.bv[e];
    const int home = x0_l[e];  // in flight beside the count
    auto before = [&](const i64x2 o, int f) {
      return static_cast<int>((o.x > me.x) | ((o.x == me.x) & ((o.y > me.y) | ((o.y == me.y) & (f < e)))));
    };
    int ahead = 0;
    int f = sub;
    for (; f + 3 * tpe < E; f += 4 * tpe) {   // four independent loads per round
      const i64x2 o0 = s.bv[f], o1 = s.bv[f + tpe], o2 = s.bv[f + 2 * tpe], o3 = s.bv[f + 3 * tpe];
      ahead += before(o0, f) + before(o1, f + tpe) + before(o2, f + 2 * tpe) + before(o3, f + 3 * tpe);
    }
    for (; f < E; f += tpe) ahead += before(s.bv[f], f);
    for (int m = tpe / 2; m > 0; m >>= 1) ahead += __shfl_xor(ahead, m);
    if (sub == 0) {
      s.order[ahead] = e;
      s.bo[ahead] = fast ? __double_as_longlong(static_cast<double>(me.x)) : me.x;
      s.ho[ahead] = home;
    }
  }
  __syncthreads();

  // 3. greedy, hottest first; wave 0 lane g keeps rank g's state
  RankState r{0, 0, 0.0, mean * mean, 0.0, 0.0};   // u2 = (0 - mean)^2
  const int cap_g = lane < G ? a.cap[lane] : 0;
  int levels = 0;   // butterfly levels that cover G lanes
  while ((1 << levels) < G) ++levels;
  // the first chunk's terms by all waves; then wave 0 places chunk after
  // chunk while the others prepare the next one
  chunk_terms<WAVES>(a, s, l, 0, min(a.chunk, E), 0, wave, WAVES, wave, lane, staged);
  __syncthreads();
  for (int c0 = 0, turn = 0; c0 < E; c0 += a.chunk, turn ^= 1) {
    const int nc = min(a.chunk, E - c0);
    if (wave == 0) {
      const int t0 = turn * a.chunk * G;
      switch ((fast ? 8 : 0) + levels) {
#define PLACE_STEPS(F, LV)                                                     \
  case (F ? 8 : 0) + LV:                                                       \
    place_chunk_steps<F, LV>(a, s, t0, c0, nc, mean, lane, cap_g, r);      \
    break;
        PLACE_STEPS(true, 0) PLACE_STEPS(true, 1) PLACE_STEPS(true, 2) PLACE_STEPS(true, 3)
        PLACE_STEPS(true, 4) PLACE_STEPS(true, 5) PLACE_STEPS(true, 6)
        PLACE_STEPS(false, 0) PLACE_STEPS(false, 1) PLACE_STEPS(false, 2) PLACE_STEPS(false, 3)
        PLACE_STEPS(false, 4) PLACE_STEPS(false, 5) PLACE_STEPS(false, 6)
#undef PLACE_STEPS
        default: break;
      }
    } else if (c0 + a.chunk < E) {
      const int c1 = c0 + a.chunk;
      chunk_terms<WAVES>(a, s, l, c1, min(a.chunk, E - c1), (turn ^ 1) * a.chunk * G, wave - 1, WAVES - 1, wave, lane, staged);
    }
    __syncthreads();
  }

  // 4. results: the objective's terms from the ranks' sums, the placement by
  // expert, and each rank's experts in ascending order
  for (int i = tid; i < E; i += kThreads) s.xs[s.order[i]] = s.xpos[i];
  if (wave == 0) {
    if (lane < G) s.fill[lane] = r.placed;
    if (a.cost) {
      const bool rank = lane < G;
      const double c_comm = wave_sum_f64(r.comm);
      const double c_load = wave_sum_f64(rank ? r.u2 : 0.0);
      const double c_mig = wave_sum_f64(r.mig);
      if (lane == 0) {
        a.cost[static_cast<size_t>(l) * 3 + 0] = c_comm;
        a.cost[static_cast<size_t>(l) * 3 + 1] = c_load;
        a.cost[static_cast<size_t>(l) * 3 + 2] = c_mig;
      }
    }
  }
  __syncthreads();
  for (int e = tid; e < E; e += kThreads) {
    const int g = s.xs[e];
    a.x[static_cast<size_t>(l) * E + e] = g;
    if (a.rank_experts) {
      // experts before e on its rank, four ranks per load
      typedef int32_t i32x4 __attribute__((ext_vector_type(4)));
      int pos = 0, f = 0;
      for (; f + 4 <= e; f += 4) {
        const i32x4 q = *reinterpret_cast<const i32x4*>(s.xs + f);
        pos += static_cast<int>(q.x == g) + static_cast<int>(q.y == g) + static_cast<int>(q.z == g) +
               static_cast<int>(q.w == g);
      }
      for (; f < e; ++f) pos += static_cast<int>(s.xs[f] == g);
      a.rank_experts[(static_cast<size_t>(l) * G + g) * a.slots + pos] = e;
    }
  }
  if (a.rank_experts) {
    for (int i = tid; i < G * a.slots; i += kThreads) {
      const int g = i / a.slots;
      if (i - g * a.slots >= s.fill[g])
        a.rank_experts[static_cast<size_t>(l) * G * a.slots + i] = -1;
    }
  }
}

}  // namespace

namespace {
size_t place_lds_of(int S, int E, int G, int waves) {
  size_t off[kLdsParts];
  return place_lds_layout(S, E, G, place_chunk_experts(E, G, waves), waves, off);
}
}  // namespace

size_t place_lds_bytes(int S, int E, int G) { return place_lds_of(S, E, G, kPlaceWaves); }

// Waves per layer.  Sixteen waves, one workgroup per CU, place a layer
// fastest; where the layers are more than the CUs, smaller workgroups share
// the CUs and one round of them does more (16, 8 and 4 waves, us: 600 layers
// of 64 experts on 8 ranks 59, 45 and 24; 300 of 128 on 8 70, 42 and 43; 200
// 37, 37 and 39).  Counts not staged whole are fetched by the waves beside the
// first all the time, which takes more of them (300 layers of 256 experts on
// 32 ranks 157, 102 and 115; 200 sources, 8 ranks 498, 294 and 291).  Where
// the LDS holds one workgroup anyway they gain nothing (64 sources and ranks
// 204, 268 and 459).
int place_waves(int L, int S, int E, int G) {
  if (L <= device_cu_count()) return kPlaceWaves;
  const int waves = a_staged(S, E) ? 4 : 8;
  return 2 * place_lds_of(S, E, G, waves) <= static_cast<size_t>(kPlaceMaxLdsBytes) ? waves : kPlaceWaves;
}

namespace {
template <int WAVES>
hipError_t launch_place_t(const PlaceArgs& h, PlaceKernelArgs a, hipStream_t st) {
  a.chunk = place_chunk_experts(h.E, h.G, WAVES);
  const size_t lds = place_lds_of(h.S, h.E, h.G, WAVES);
  static unsigned long long lds_set = 0;  // devices with the LDS limit raised
  const hipError_t e_lds = set_max_dynamic_lds(reinterpret_cast<const void*>(&place_kernel<WAVES>), kPlaceMaxLdsBytes, &lds_set);
  if (e_lds != hipSuccess) return e_lds;
  hipLaunchKernelGGL(place_kernel<WAVES>, dim3(h.L), dim3(WAVES * kWave), lds, st, a);
  return hipGetLastError();
}
}  // namespace

hipError_t launch_place(const PlaceArgs& h, hipStream_t st) {
  if (h.L == 0) return hipSuccess;
  PlaceKernelArgs a{};
  a.A = h.A;
  a.B = h.B;
  a.D = h.D;
  a.M = h.M;
  a.x0 = h.x0;
  a.x = h.x;
  a.rank_experts = h.rank_experts;
  a.cost = h.cost;
  a.alpha = h.alpha;
  a.beta = h.beta;
  a.gamma = h.gamma;
  a.m_uniform = h.m_uniform;
  a.S = h.S;
  a.E = h.E;
  a.G = h.G;
  a.slots = h.slots;
  for (int g = 0; g < h.G; ++g) a.cap[g] = h.cap[g];
  switch (place_waves(h.L, h.S, h.E, h.G)) {
    case 4: return launch_place_t<4>(h, a, st);
    case 8: return launch_place_t<8>(h, a, st);
    default: return launch_place_t<kPlaceWaves>(h, a, st);
  }
}

}  // namespace moe
