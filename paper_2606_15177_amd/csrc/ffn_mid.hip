// Expert FFN for decode and mid-sized batches: from a single token to far
// fewer rows per expert than fill 256-row tiles (chunked prefill, decode of
// hundreds of tokens over many experts).  What bounds it is reading the
// active experts' weights once; hot and shared experts add MFMA work.
//
// Items.  One workgroup of four waves takes one item: up to 128 token rows of
// one group (a chunk) times a block of weight rows.  Groups of up to 64 rows
// take narrow items of 128 weight rows, larger groups wide ones of 256 (of
// 128 where a launch has few wide items, which would otherwise run on long
// after the rest: Mixtral down at 100 tokens 318 -> 223 us, DSV2-Lite down at
// 200 tokens 97 -> 71 us; and up to one per CU where few narrow ones keep them
// company: 17 experts of H 2208, I 1064 and a shared one of 1392, 642 tokens,
// layer 153 -> 116 us, while in the DSV3 share of 512 tokens narrow items fill
// the CUs and the halves cost 1%).  A wave owns 32-row blocks of the weights
// (gate/up: 16 gate rows and the 16 up rows of the same columns, which the
// MFMA's C layout puts into one lane) and all token rows of the chunk.
// Dispatched as plain workgroups, two per CU: a persistent grid over 256-row tiles left CUs
// idle in its last round and one workgroup per CU waiting at its barriers.
//
// Pipeline.  Weights and token rows go by buffer_load_dwordx4 ... lds straight
// into a ring of K stages in 80 KB of LDS, D - 1 stages ahead; each wave loads
// its own weights and a quarter of the chunk's token rows; one barrier per
// stage.  Narrow items: 64-wide stages, four (<= 32 rows) or three in the
// ring, 96 and 64 KB of weights in flight per CU.  Wide items: 32-wide stages,
// so that three of 24 KB fit.  Splitting K over the waves as the decode kernel
// does was slower past 64 tokens (Qwen3 down at 256 tokens 77 us against 90
// and 141 with 2 and 4 parts: each part needs token rows of its own); a batch
// with few items halves it (see mid_splits_k).  Also slower: 64-row chunks for
// hot experts (DSV2-Lite layer, 4096 tokens: 971 against 825 us).
//
// Order.  Items are numbered per kind; each XCD (workgroup id mod 8) owns a
// contiguous run of every kind, so an expert's token rows, and the weight
// block that its chunks share, stay in one L2 (DSV2-Lite gate/up at 1021
// tokens fetches 0.95 GB instead of 1.09).  Within an XCD the wide (MFMA
// bound) and narrow (HBM bound) items take turns.  The dispatcher deals
// workgroups to the shader engines strictly in turn, and waits for the engine
// whose turn it is: turns of one item put all wide ones on the same two
// engines of an XCD and left the others idle half the time.  Turns of kTurn
// items give every engine both (Qwen3 layer at 800 tokens 316 -> 286 us,
// DSV2-Lite at 1021 tokens 448 -> 342 us).
//
// Only groups with rows have items: the decode kernel's grid over all groups
// spent most of a small batch's time on empty ones (Qwen3, 1 token, layer 42.8
// -> 34.8 us; DSV2-Lite, 1 token, gate/up 31 -> 18 us, down 35 -> 17 us).
//
// Measured (layer, 256-row tiles -> this kernel): Qwen3, 256 tokens 288 -> 244
// us (gate/up streams 5.6 TB/s); DSV2-Lite, 400 tokens 341 -> 266 us; the
// DSV3 share, 256 tokens 544 -> 430 us; Mixtral, 65 tokens 607 -> 525 us.
#include "ffn_impl.h"

#include <algorithm>
#include <type_traits>

namespace moe {
namespace {

constexpr int kMidRows = 128;        // token rows of a chunk
constexpr int kWideRows = 64;        // groups of more rows take wide items
constexpr int kMidCols = 128;        // weight rows of a narrow item
constexpr int kFewWide = 128;        // fewer wide items than this take 128 weight rows: half the CUs' worth
constexpr int kOneWide = 256;        // ... or fewer than this, one per CU, in a launch of fewer items than
constexpr int kSlots = 512;          // workgroups fit the chip
constexpr int kMidLds = 80 * 1024;   // two workgroups per CU
constexpr int kXcds = 8;
constexpr int kTurn = 8;             // items per turn: a multiple of an XCD's shader engines
constexpr uint32_t kDead = 0x80000000u;  // past the descriptor's range: reads zeros, no traffic

struct MidArgs {
  GemmArgs g;   // the routed experts (device offsets)
  GemmArgs sp;  // static rows (shared experts); sp.static_rows == 0: none
};

// first of n items that XCD x owns (x = kXcds: n)
__device__ __forceinline__ int run_start(int n, int x) {
  return static_cast<int>(static_cast<long long>(n) * x / kXcds);
}

// column blocks of a group of n rows: narrow items cover `cols` output columns, wide ones wide_cols
__device__ __forceinline__ int col_blocks(int n, int N, int cols, int wide_cols) {
  return ceil_div(N, n > kWideRows ? wide_cols : cols);
}

template <bool GATED, int KP>
__global__ __launch_bounds__(kMidThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void mid_kernel(MidArgs ma) {
  constexpr int FULL_COLS = GATED ? kMidCols / 2 : kMidCols;  // output columns of 128 weight rows
  constexpr int OUT_COLS = FULL_COLS / KP;                    // ... of a narrow item
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int lane = lane_id();
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);

  // ---- which item ----
  // Items are numbered per kind (shared, wide, narrow) by group, column block
  // and chunk (fastest); an XCD owns an equal, contiguous run of each kind.
  const int sp_m = ma.sp.static_rows;
  const int sp_chunks = sp_m > 0 ? ceil_div(sp_m, kMidRows) : 0;
  // Offset and rows of groups g0 + 64 i + lane, i < kPasses, their loads in
  // flight together: up to 64 kPasses groups are read once, more in as many
  // batches.  (64 groups at a time, and thrice over, a small batch of 1024
  // experts spent most of its time here: H 512, I 256, 64 tokens, layer 117 us,
  // 90 on the decode kernel.)
  constexpr int kPasses = 4;
  int first_row[kPasses], n_rows[kPasses];
  auto load_groups = [&](int g0) {
#pragma unroll
    for (int i = 0; i < kPasses; ++i) {
      first_row[i] = n_rows[i] = 0;
      if (g0 + i * kWave < ma.g.groups) {
        const int gg = min(g0 + i * kWave + lane, ma.g.groups);  // past the last group: no rows
        first_row[i] = ma.g.offsets[gg];
        n_rows[i] = ma.g.offsets[min(gg + 1, ma.g.groups)];
      }
    }
#pragma unroll
    for (int i = 0; i < kPasses; ++i) n_rows[i] -= first_row[i];
  };
  int c_wide = 0, c_narrow = 0;  // chunks of the routed groups
  for (int g0 = 0; g0 < ma.g.groups; g0 += kPasses * kWave) {
    load_groups(g0);
#pragma unroll
    for (int i = 0; i < kPasses; ++i) {
      c_wide += n_rows[i] > kWideRows ? ceil_div(n_rows[i], kMidRows) : 0;
      c_narrow += n_rows[i] > 0 && n_rows[i] <= kWideRows ? 1 : 0;
    }
  }
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) {
    c_wide += __shfl_xor(c_wide, off);
    c_narrow += __shfl_xor(c_narrow, off);
  }
  c_wide = __builtin_amdgcn_readfirstlane(c_wide);
  c_narrow = __builtin_amdgcn_readfirstlane(c_narrow);
  const int narrow_blocks = ceil_div(ma.g.N, OUT_COLS);
  const int n_narrow = c_narrow * narrow_blocks;
  // items of the shared and of the wide groups where wide items cover `cols` output columns
  auto shared_items = [&](int cols) { return sp_m > 0 ? sp_chunks * col_blocks(sp_m, ma.sp.N, OUT_COLS, cols) : 0; };
  int wide_cols = 2 * FULL_COLS;
  const int heavy = shared_items(wide_cols) + c_wide * ceil_div(ma.g.N, wide_cols);
  if (heavy < kFewWide || (heavy < kOneWide && heavy + n_narrow < kSlots)) wide_cols = FULL_COLS;
  const int n_shared = shared_items(wide_cols);
  const int wide_blocks = ceil_div(ma.g.N, wide_cols);
  const int n_wide = c_wide * wide_blocks;
  const int xcd = blockIdx.x % kXcds, i = blockIdx.x / kXcds;
  const int s_lo = run_start(n_shared, xcd), w_lo = run_start(n_wide, xcd), n_lo = run_start(n_narrow, xcd);
  const int my_shared = run_start(n_shared, xcd + 1) - s_lo;
  const int my_heavy = my_shared + run_start(n_wide, xcd + 1) - w_lo;
  const int my_narrow = run_start(n_narrow, xcd + 1) - n_lo;
  if (i >= my_heavy + my_narrow) return;
  // heavy (shared and wide) and narrow items take turns while there are both
  const int turns = min(my_heavy, my_narrow) / kTurn;
  bool narrow;
  int idx;
  if (i < 2 * turns * kTurn) {
    narrow = (i / kTurn) & 1;
    idx = i / (2 * kTurn) * kTurn + i % kTurn;
  } else {
    idx = i - turns * kTurn;
    narrow = idx >= my_heavy;
    idx = narrow ? i - my_heavy : idx;
  }
  const bool shared = !narrow && idx < my_shared;
  const bool wide = shared ? sp_m > kWideRows : !narrow;
  idx = narrow ? n_lo + idx : shared ? s_lo + idx : w_lo + idx - my_shared;
  int g = 0, row_base = 0, m = sp_m, item = idx;
  if (!shared) {
    // the group of the kind's chunk `at`, the kind's chunks before it in `before`
    const int blocks = wide ? wide_blocks : narrow_blocks;
    const int at = idx / blocks;
    bool found = false;
    for (int g0 = 0, before = 0; !found && g0 < ma.g.groups; g0 += kPasses * kWave) {
      if (ma.g.groups > kPasses * kWave) load_groups(g0);
#pragma unroll
      for (int i = 0; i < kPasses; ++i) {
        if (found || g0 + i * kWave >= ma.g.groups) continue;
        const int own = (n_rows[i] > kWideRows) == wide ? ceil_div(n_rows[i], kMidRows) : 0;
        int inc = own;
#pragma unroll
        for (int off = 1; off < kWave; off <<= 1) {
          const int o = __shfl_up(inc, off);
          if (lane >= off) inc += o;
        }
        const uint64_t past = __ballot(before + inc > at);
        if (past) {
          const int l = __ffsll(static_cast<long long>(past)) - 1;
          g = g0 + i * kWave + l;
          row_base = __builtin_amdgcn_readlane(first_row[i], l);
          m = __builtin_amdgcn_readlane(n_rows[i], l);
          item = idx - (before + __builtin_amdgcn_readlane(inc - own, l)) * blocks;
          found = true;
        } else {
          before += __builtin_amdgcn_readlane(inc, kWave - 1);
        }
      }
    }
    if (!found) return;  // not reached: idx lies within the groups' items
  }
  const int n_chunks = ceil_div(m, kMidRows);
  int nblk = item / n_chunks;
  int chunk = item - nblk * n_chunks;
  g = __builtin_amdgcn_readfirstlane(g);
  row_base = __builtin_amdgcn_readfirstlane(row_base);
  m = __builtin_amdgcn_readfirstlane(m);
  chunk = __builtin_amdgcn_readfirstlane(chunk);
  nblk = __builtin_amdgcn_readfirstlane(nblk);

  const int K = shared ? ma.sp.K : ma.g.K;
  const int N = shared ? ma.sp.N : ma.g.N;
  const int ldw = shared ? ma.sp.ldw : ma.g.ldw;
  const int kseg = shared ? ma.sp.kseg : ma.g.kseg;
  const size_t seg_stride = shared ? ma.sp.seg_stride : ma.g.seg_stride;
  const int32_t* x_rows = shared ? nullptr : ma.g.x_rows;
  // the group's rows in equal chunks of whole 32-row MFMA tiles
  const int chunk_rows = ceil_div(ceil_div(m, ceil_div(m, kMidRows)), 32) * 32;
  const int m0 = chunk * chunk_rows;
  const int rows = min(chunk_rows, m - m0);
  const int n0 = nblk * (wide ? wide_cols : OUT_COLS);

  // ---- loads ----
  const size_t gofs = (shared ? size_t{0} : static_cast<size_t>(g) * ma.g.group_stride) + static_cast<size_t>(n0) * ldw;
  const uint16_t* w0 = (shared ? ma.sp.w0 : ma.g.w0) + gofs;
  const uint16_t* w1 = GATED ? (shared ? ma.sp.w1 : ma.g.w1) + gofs : w0;
  const uint16_t* xb = shared ? ma.sp.x : ma.g.x;
  if (x_rows == nullptr) xb += static_cast<size_t>(row_base + m0) * K;
  const __amdgpu_buffer_rsrc_t rs_w0 =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(w0), 0, 0x7fffffff, 0x00020000);
  const __amdgpu_buffer_rsrc_t rs_w1 =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(w1), 0, 0x7fffffff, 0x00020000);
  const __amdgpu_buffer_rsrc_t rs_x =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(xb), 0, 0x7fffffff, 0x00020000);
  const bool segmented = kseg < K;
  const int lrow = lane & 31, lhalf = lane >> 5;

  auto body = [&](auto nsub_c, auto wb_c, auto kp_c, auto bk_c, auto depth_c) {
    constexpr int NSUB = decltype(nsub_c)::value;
    constexpr int WB = decltype(wb_c)::value;
    constexpr int NK = decltype(kp_c)::value;   // K parts; waves WN apart take the same columns
    constexpr int WN = 4 / NK;                  // waves along the weight rows
    constexpr int BK = decltype(bk_c)::value;
    constexpr int D = decltype(depth_c)::value;
    constexpr int ROW = BK * 2;              // bytes of an LDS row
    constexpr int CPR = ROW / 16;            // 16-byte chunks per row
    constexpr int RPI = kWave / CPR;         // rows per load instruction
    constexpr int SWZ = 16 / CPR;            // rows sharing one swizzle key
    constexpr int XPART = NSUB * 32 * ROW;   // token rows of one K part
    constexpr int STAGE = NK * XPART + 4 * WB * 32 * ROW;
    constexpr int XL = NSUB * 32 / RPI / WN;// token loads per wave and stage
    constexpr int WL = WB * 32 / RPI;           // weight loads per wave and stage
    constexpr int LOADS = XL + WL;
    constexpr int KS = BK / 16;              // MFMA K-steps per stage
    static_assert(D * STAGE <= kMidLds && XL * RPI * WN == NSUB * 32, "the ring fits, whole loads fill the token rows");
    const int lr = lane / CPR;               // row of a load
    const int wn = wave % WN, wk = wave / WN;
    // 16-byte chunk c of LDS row r sits at slot c ^ ((r / SWZ) % CPR); load i
    // of the weights fills the wave's rows RPI i .., load q of the tokens the
    // rows RPI (WN q + wn) ..
    uint32_t woff[WL], xoff[XL];
    int wpiece[WL], xpiece[XL];
#pragma unroll
    for (int i = 0; i < WL; ++i) {
      const int r = RPI * i + lr;
      const int b = WB * wn + r / 32;  // 32-row block of weights
      const int col = GATED ? 16 * b + (r & 15) : 32 * b + r % 32;
      woff[i] = n0 + col < N ? static_cast<uint32_t>(col * ldw * 2) : kDead;
      wpiece[i] = (lane % CPR) ^ ((r / SWZ) % CPR);
    }
#pragma unroll
    for (int q = 0; q < XL; ++q) {
      const int r = RPI * (WN * q + wn) + lr;
      int src = r;
      if (x_rows) src = x_rows[row_base + m0 + min(r, rows - 1)];
      xoff[q] = r < rows ? static_cast<uint32_t>(src * K * 2) : kDead;
      xpiece[q] = (lane % CPR) ^ ((r / SWZ) % CPR);
    }
    const int nst = ceil_div(ceil_div(K, BK), NK);  // stages of a K part (the last part's may lie past K)
    int s_ld = 0, slot_ld = 0;  // next stage to load and its slot
    int kb_ld = static_cast<int>((static_cast<unsigned>(nblk) * 7u + static_cast<unsigned>(g) * 3u) % static_cast<unsigned>(nst));
    auto issue = [&]() {
      unsigned char* st = smem + slot_ld * STAGE;
      const int k0 = (wk * nst + kb_ld) * BK;
      const uint32_t dead = s_ld < nst ? 0u : kDead;
#pragma unroll
      for (int q = 0; q < XL; ++q) {
        const int k = k0 + xpiece[q] * 8;
        const uint32_t kill = dead | (k < K ? 0u : kDead) | (xoff[q] & kDead);
        load_lds16(rs_x, st + wk * XPART + RPI * (WN * q + wn) * ROW, (xoff[q] + static_cast<uint32_t>(k * 2)) | kill);
      }
      unsigned char* wl = st + NK * XPART + wave * (WB * 32 * ROW);
#pragma unroll
      for (int i = 0; i < WL; ++i) {
        const int k = k0 + wpiece[i] * 8;
        const uint32_t kill = dead | (k < K ? 0u : kDead) | (woff[i] & kDead);
        uint32_t col = static_cast<uint32_t>(k * 2);
        if (segmented) {
          const int kc = k < K ? k : 0;
          const int q = kc / kseg;
          col = static_cast<uint32_t>((static_cast<size_t>(q) * seg_stride + (kc - q * kseg)) * 2);
        }
        load_lds16(GATED && ((RPI * i) & 16) ? rs_w1 : rs_w0, wl + i * 1024, (woff[i] + col) | kill);
      }
      ++s_ld;
      if (++slot_ld == D) slot_ld = 0;
      if (++kb_ld == nst) kb_ld = 0;
    };
    f32x16 acc[WB][NSUB];
#pragma unroll
    for (int b = 0; b < WB; ++b)
#pragma unroll
      for (int s = 0; s < NSUB; ++s) acc[b][s] = f32x16{};
#pragma unroll
    for (int s = 0; s < D - 1; ++s) issue();
    int slot = 0;
    for (int j = 0; j < nst; ++j) {
      __builtin_amdgcn_s_waitcnt(wait_vm((D - 2) * LOADS));  // own loads of stage j landed
      phase_barrier();  // everyone's have, and everyone has read stage j - 1
      issue();          // stage j + D - 1 into the slot of stage j - 1
      const unsigned char* xp = smem + slot * STAGE + wk * XPART;
      const unsigned char* wp = smem + slot * STAGE + NK * XPART + wave * (WB * 32 * ROW);
      bf16x8 wf[KS][WB], xf[KS][NSUB];
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        const int cs = ((2 * ks + lhalf) ^ ((lrow / SWZ) % CPR)) << 4;
#pragma unroll
        for (int b = 0; b < WB; ++b)
          wf[ks][b] = as_bf16x8(*reinterpret_cast<const u32x4*>(wp + (32 * b + lrow) * ROW + cs));
#pragma unroll
        for (int s = 0; s < NSUB; ++s)
          xf[ks][s] = as_bf16x8(*reinterpret_cast<const u32x4*>(xp + (32 * s + lrow) * ROW + cs));
      }
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
#pragma unroll
        for (int b = 0; b < WB; ++b)
#pragma unroll
          for (int s = 0; s < NSUB; ++s) acc[b][s] = mfma32x32x16(wf[ks][b], xf[ks][s], acc[b][s]);
      if (++slot == D) slot = 0;
    }
    __builtin_amdgcn_s_waitcnt(wait_vm(0));  // the loads past the last stage: nothing may still write the LDS
    if constexpr (NK > 1) {
      // sum the K parts in order through LDS
      static_assert((NK - 1) * WN * WB * NSUB * 16 * kWave * 4 <= kMidLds, "the partial sums fit the LDS");
      float* red = reinterpret_cast<float*>(smem);
      __syncthreads();  // every wave is past its last stage
      if (wk > 0) {
#pragma unroll
        for (int b = 0; b < WB; ++b)
#pragma unroll
          for (int s = 0; s < NSUB; ++s)
#pragma unroll
            for (int v = 0; v < 16; ++v)
              red[((((wk - 1) * WN + wn) * WB + b) * NSUB + s) * (16 * kWave) + v * kWave + lane] = acc[b][s][v];
      }
      __syncthreads();
      if (wk > 0) return;
#pragma unroll
      for (int p = 0; p < NK - 1; ++p)
#pragma unroll
        for (int b = 0; b < WB; ++b)
#pragma unroll
          for (int s = 0; s < NSUB; ++s)
#pragma unroll
            for (int v = 0; v < 16; ++v)
              acc[b][s][v] += red[(((p * WN + wn) * WB + b) * NSUB + s) * (16 * kWave) + v * kWave + lane];
    }
    // ---- epilogue: lane holds C[n = 8 v4 + 4 lhalf + i][t = lrow] ----
    uint16_t* out = (shared ? ma.sp.out : ma.g.out) + static_cast<size_t>(row_base + m0) * N;
#pragma unroll
    for (int s = 0; s < NSUB; ++s) {
      const int r = 32 * s + lrow;
      constexpr int PAIRS = GATED ? 1 : 2;  // pairs of 8-column groups the wave writes
#pragma unroll
      for (int bp = 0; bp < WB * PAIRS; ++bp) {
        const int b = bp / PAIRS, p = bp % PAIRS;
        uint32_t pk[2][2];
#pragma unroll
        for (int v = 0; v < 2; ++v) {
          float o[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float c0 = acc[b][s][4 * (2 * p + v) + i];
            if constexpr (GATED)
              o[i] = silu(c0) * acc[b][s][4 * (2 + v) + i];
            else
              o[i] = c0;
          }
          pk[v][0] = cvt_pk_bf16(o[0], o[1]);
          pk[v][1] = cvt_pk_bf16(o[2], o[3]);
        }
        // lower lanes take columns 0..7, upper lanes 8..15 of the pair
        const auto s0 = __builtin_amdgcn_permlane32_swap(pk[0][0], pk[1][0], false, false);
        const auto s1 = __builtin_amdgcn_permlane32_swap(pk[0][1], pk[1][1], false, false);
        const u32x4 v = {s0[0], s1[0], s0[1], s1[1]};
        const int col = n0 + (GATED ? 16 * (WB * wn + b) : 32 * (WB * wn + b) + 16 * p) + 8 * lhalf;
        if (r < rows && col < N) store16(out + static_cast<size_t>(r) * N + col, v);
      }
    }
  };
  using std::integral_constant;
  using C1 = integral_constant<int, 1>;
  using C2 = integral_constant<int, 2>;
  using C3 = integral_constant<int, 3>;
  using C4 = integral_constant<int, 4>;
  using C5 = integral_constant<int, 5>;
  using K32 = integral_constant<int, 32>;
  using K64 = integral_constant<int, 64>;
  if (wide && wide_cols > FULL_COLS)
    body(C4{}, C2{}, C1{}, K32{}, C3{});
  else if (wide)
    body(C4{}, C1{}, C1{}, K32{}, C5{});
  else if constexpr (KP == 1) {
    if (rows > 32) body(C2{}, C1{}, C1{}, K64{}, C3{});
    else body(C1{}, C1{}, C1{}, K64{}, C4{});
  } else {
    if (rows > 32) body(C2{}, C1{}, C2{}, K32{}, C5{});
    else body(C1{}, C1{}, C2{}, K64{}, C3{});
  }
}

template <bool GATED, int KP>
hipError_t launch_mid_t(long long blocks, const GemmArgs& g, const GemmArgs& sp, hipStream_t st) {
  static unsigned long long lds_set = 0;  // devices with the LDS limit raised
  const hipError_t e = set_max_dynamic_lds(reinterpret_cast<const void*>(&mid_kernel<GATED, KP>), kMidLds, &lds_set);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((mid_kernel<GATED, KP>), dim3(static_cast<unsigned>(blocks)), dim3(kMidThreads), kMidLds, st,
                     MidArgs{g, sp});
  return hipGetLastError();
}

// Narrow items that an evenly routed batch makes (undivided in K).
long long narrow_items(const Segments& seg, const GemmArgs& a, const GemmArgs* sh, bool gated) {
  const int cols = gated ? kMidCols / 2 : kMidCols;
  return static_cast<long long>(seg.hit_groups) * ceil_div(a.N, cols) + (sh ? ceil_div(sh->N, cols) : 0);
}

}  // namespace

// Whether narrow_items is close: where not all experts are hit, skewed routing
// hits fewer still (24 tokens, top 8 of 96 experts, Zipf 1, 24 of them, gate/up
// of 210 items by even routing: 48 us with K in halves, 59 without).
bool mostly_hit(const Segments& seg) { return 20 * seg.hit_groups >= 19 * seg.groups; }

// Few narrow items leave CUs idle and each runs through its whole K alone:
// half as many columns and the K halves on two pairs of waves then.  Time
// without / with the split: Qwen3, 1 token (96 and 128 items) gate/up 18.0 /
// 14.7 us, down 10.1 / 8.8, 2 tokens (180) gate/up 19.5 / 21.1; long K:
// Mixtral down, 1, 4 and 8 tokens (70, 175, 230) 83.6 / 59.0, 96 / 80 and 112
// / 124 us; DSV3 share gate/up, 14 and 24 tokens (400, 610) 120 / 110 and 130
// / 131 us; a stacked K of the shared experts (DSV2-Lite down, K 2816 among
// 1408), 12 tokens (730) 38 / 31 us.  Not on long K of gate/up alone with a few
// more items than half the CUs over mostly hit experts (8 experts of H 4096, 24
// and 64 tokens: I 1408, 176 items, layer 58 / 60 and 64 / 74 us; 4 of H 8192, I
// 5632, 352 items, 24 tokens 227 / 213).
// A deeper ring there (six stages in 160 KB, one workgroup per CU) does not
// pay: Qwen3, 1 token, gate/up 14.6 -> 14.3 us but down 9.0 -> 10.7, and a layer
// of four 139 -> 147 us, as each kernel waits for whole CUs' LDS.
bool mid_splits_k(const Segments& seg, const GemmArgs& a, const GemmArgs* sh, bool gated) {
  if (seg.max_rows > kWideRows) return false;
  const long long items = narrow_items(seg, a, sh, gated);
  if (items <= 128 || (sh && sh->K > a.K && items <= 768)) return true;
  if (gated && !sh && items <= 220 && mostly_hit(seg)) return false;
  return a.K >= kLongK && items <= (gated ? 400 : 200);
}

long long mid_blocks(const Segments& seg, const GemmArgs& a, const GemmArgs* sh, bool gated) {
  const int cols = (gated ? kMidCols / 2 : kMidCols) / (mid_splits_k(seg, a, sh, gated) ? 2 : 1);
  // at most one partly filled chunk per group; wide items need fewer column blocks
  const long long chunks = seg.total_rows / kMidRows + std::min(seg.groups, seg.total_rows);
  long long items = chunks * ceil_div(a.N, cols);
  if (sh) items += static_cast<long long>(ceil_div(sh->static_rows, kMidRows)) * ceil_div(sh->N, cols);
  return items == 0 ? 0 : (items / kXcds + 3) * kXcds;  // each kind's run on an XCD rounds up by one
}

// Batches of up to 64 tokens: everything but two kinds of launch without
// shared rows, where the decode kernel's finer items, four K parts each, are
// faster (times of its and of this kernel, us, in layers of 2 of E experts).
//   Small ones, a few rows per expert, K up to 1024 and all its workgroups on
//   the CUs at once: it knows its rows without a search over the groups (H
//   1280, I 448, 8 experts, one token, top 3: layer 20 and 21.5).
//   Gate/up of many items over mostly hit experts (E 8, H 4096, 24 and 64
//   tokens: I 2816 112 and 126, 118 and 134; E 16, H 2048, I 2816, 48 tokens 104
//   and 109; 64 experts of H 2048, I 768, top 8, 45 tokens 130 and 138); not on
//   K of 8192 (E 16, I 2816, 64 tokens 410 and 388) unless there are very many
//   (Mixtral, 1.02 at 8 to 24 tokens, 1.00 to 1.02 at 40 to 64), nor with fewer
//   items (E 8, H 4096, I 1408, 24 tokens 64 and 58).
bool mid_streams(const Segments& seg, const GemmArgs& a, const GemmArgs* sh, bool gated) {
  if (sh) return true;
  if (a.K <= 1024 && seg.mean_rows <= 8 && skinny_blocks(seg, a, gated) <= device_cu_count()) return false;
  if (!gated) return true;
  const long long items = narrow_items(seg, a, sh, gated);
  if (a.K >= kLongK && items >= 1024) return false;
  return !(mostly_hit(seg) && a.K < 2 * kLongK && items >= (a.K >= kLongK ? 300 : 600));
}

hipError_t launch_mid(const Segments& seg, const GemmArgs& a, const GemmArgs* sh, bool gated, hipStream_t st) {
  const GemmArgs none{};
  const GemmArgs& sp = sh ? *sh : none;
  const long long blocks = mid_blocks(seg, a, sh, gated);
  if (blocks == 0) return hipSuccess;
  if (mid_splits_k(seg, a, sh, gated))
    return gated ? launch_mid_t<true, 2>(blocks, a, sp, st) : launch_mid_t<false, 2>(blocks, a, sp, st);
  return gated ? launch_mid_t<true, 1>(blocks, a, sp, st) : launch_mid_t<false, 1>(blocks, a, sp, st);
}

}  // namespace moe
