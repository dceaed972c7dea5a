// Grouped SwiGLU expert GEMMs over the permuted route rows and the weighted
// combine (Eq. gated_expert, Eq. moe_output / Eq. folded_moe).
//
// gate_up:  H[r, :] = SiLU(X[tok(r)] W_gate[e]^T) * (X[tok(r)] W_up[e]^T)     (bf16 H)
// down:     Y[r, :] = w(r) * (H[r] W_down[e]^T)                                (fp32 Y)
//           or, when every token owns exactly one row, y[tok(r)] = Y[r] directly
// combine:  y_i = sum over the token's routes (slot order) of Y[row], + shared row
//
// Weights are [rows, K] with K contiguous, so both operands load along K.  Group
// sizes are device data: each kernel walks a device-side tile list built by the
// permutation (no host synchronisation), in an XCD-aware order that keeps the
// tiles sharing one weight tile on one XCD's L2.
//
// expert_gemm_tile: 128x128 macro tile, 4 waves of 32x32x16 bf16 MFMA, BK=64 LDS
// double buffer with an XOR swizzle of 16-byte chunks, two tiles of global loads
// in flight through registers.  The down projection may split its reduction
// (few rows per retained expert): split s writes its own partial Y[s], and the
// combine adds the splits in a fixed order.
#include "common.hpp"
#include "kernels.hpp"

namespace exfold {

struct GemmKArgs {
  const bf16_t *A;  // gate_up: x [T, d] gathered by row_token; down: H [rows, I]
  int lda;
  const int32_t *row_token;
  const int32_t *offsets;
  const int32_t *tile_start;
  int groups, n_experts, n_tiles, ksplit, kc, rows;
  const bf16_t *W, *Ws;  // routed base and shared expert
  long long w_stride;    // elements per routed expert
  int ldw;               // K extent of a weight row
  int inter;             // gate_up: intermediate size (up-row offset, H width)
  int d;                 // down: output width
  bf16_t *H;
  float *Y;
  bf16_t *Yh;  // down, when set: bf16 per-row outputs instead of Y (no split)
  float *P;    // wide tiles: split-remainder partial tiles [workgroups][256 * 256]
  bf16_t *y;
  const float *row_w;
};

// g * sigmoid(g) with the hardware reciprocal (one rounding step instead of
// the IEEE division sequence; the result is rounded to bf16 or kept fp32
// within 1 ulp).
__device__ __forceinline__ float silu(float g) { return g * __builtin_amdgcn_rcpf(1.0f + __expf(-g)); }

constexpr int kBK = 64;

// 16 bytes of a weight row; ONCE: no other tile reads it (TileId::alone), and the
// load is non-temporal.  Such streams neither evict the rows, tables and activations
// that are read again nor wait for the room: Mixtral-shaped decode gate/up 163 ->
// 149 us, down 85 -> 77, GLM-shaped (64 tokens, pool of 32) 141 -> 129 and 79 -> 71.
// Where several m-tiles share a weight row the hint costs more than it gives (64-row
// down tiles of 512 Qwen3-shaped tokens, pool of 64, 55 -> 68 us; every wide tile
// 5%; 256 tokens on 128 Qwen3-shaped experts, some with up to 175 rows, the layer:
// no hint 256, on every weight row 266, on single m-tiles 235).  It loses only where
// the weights fit the last-level cache and nothing else runs between two calls (32
// experts, d 1024, I 512, 300 tokens x 4, skewed: 46.1 -> 48.2 us; with 2 GB of other
// layers between them 50.8 -> 48.3; the most seen: d 2048, I 1408, 4 tokens x 6 on 64
// skewed experts, 56.4 -> 62.4, and 66.5 -> 59.0 with 5 GB of other layers).
template <bool ONCE>
__device__ __forceinline__ u32x4 load_w16(const bf16_t *p) {
  if constexpr (ONCE)
    return __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(p));
  else
    return *reinterpret_cast<const u32x4 *>(p);
}

// Start of a main loop whose weight loads are load_w16<ONCE>, in a kernel that holds
// one of each.  An instruction that the two loops do not have in common: the compiler
// otherwise hoists the first loads out of both as plain ones and waits for all of
// them at the loop head (2-3% of a skinny launch).
template <bool ONCE>
__device__ __forceinline__ void mark_loads() {
  if constexpr (ONCE)
    asm volatile("; weights read once");
  else
    asm volatile("; weights shared");
}

// LDS element offset of 16-byte chunk q of tile row r (8 chunks per 128-byte row).
// The slot is q XOR gray(r): one chunk column of any 8 or 16 consecutive rows
// (the lanes of one LDS cycle of ds_read_b128) then spans distinct banks.
__device__ __forceinline__ int swz(int r, int q) { return (r * 8 + (q ^ ((r ^ (r >> 1)) & 7))) * 8; }

// Tile of workgroup `wg`: group g, n-tile nt, split ks, m-tile mt (m-tile
// fastest, so the m-tiles sharing one weight tile run together).  The grid is an
// upper bound of the tile count; workgroups past the device-side count exit, and
// the XCD-aware remap is taken over the actual count so that every XCD gets an
// equal, contiguous share of the real tiles.
struct TileId {
  int g, nt, ks, mt;
  int dbl;  // wide tiles: a 128-row tail spanning n-tiles nt and nt + 1
  int alone;  // the group has one m-tile: nobody else reads this tile's weights
};
// Tile of logical id L (m-tile fastest within a group and n-tile).
__device__ __forceinline__ void tile_at(const GemmKArgs &p, int L, TileId &t) {
  const int units = p.n_tiles * p.ksplit;
  int lo = 0, hi = p.groups;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (p.tile_start[mid] * units <= L) lo = mid; else hi = mid;
  }
  const int mt_g = p.tile_start[lo + 1] - p.tile_start[lo];
  const int local = L - p.tile_start[lo] * units;
  t.g = lo;
  t.mt = local % mt_g;
  t.alone = mt_g == 1;
  const int u = local / mt_g;
  t.ks = u % p.ksplit;
  t.nt = u / p.ksplit;
}

__device__ __forceinline__ bool decode_tile(const GemmKArgs &p, int wg, TileId &t) {
  const int units = p.n_tiles * p.ksplit;
  const int total = p.tile_start[p.groups] * units;
  if (wg >= total) return false;
  tile_at(p, xcd_remap(wg, total), t);
  return true;
}

// ---------------------------------------------------------------------------
// Macro-tile kernel.
// ---------------------------------------------------------------------------
// PLAIN: one group of p.rows rows read in order (no offsets, tile list or
// gather), partial sums of split ks written unscaled to Y[ks] (a plain
// x W^T with a split reduction: the router logits of large batches).
template <int BM, int BN, bool GATE_UP, bool DIRECT, bool PLAIN = false>
__global__ __launch_bounds__(256, 1) void expert_gemm_tile(const GemmKArgs p) {
  constexpr int WTM = BM / 2, WTN = BN / 2;
  constexpr int TM = WTM / 32, TN = WTN / 32;
  constexpr int PA = BM / 32, PB = BN / 32;  // 16-byte chunks per thread per stage
  static_assert(!GATE_UP || (TN % 2 == 0), "gate/up pairs");

  __shared__ __attribute__((aligned(16))) bf16_t smem[2 * (BM + BN) * kBK];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;

  TileId t;
  int row0, valid;
  const bf16_t *Wg;
  if constexpr (PLAIN) {
    const int mt_n = (p.rows + BM - 1) / BM, total = mt_n * p.n_tiles * p.ksplit;
    if ((int)blockIdx.x >= total) return;
    const int L = xcd_remap(blockIdx.x, total);
    t.g = 0;
    t.mt = L % mt_n;
    t.alone = 0;
    t.ks = (L / mt_n) % p.ksplit;
    t.nt = L / mt_n / p.ksplit;
    row0 = t.mt * BM;
    valid = min(BM, p.rows - row0);
    Wg = p.W;
  } else {
    if (!decode_tile(p, blockIdx.x, t)) return;
    row0 = p.offsets[t.g] + t.mt * BM;
    valid = min(BM, p.offsets[t.g + 1] - row0);
    Wg = (t.g < p.n_experts) ? p.W + (long long)t.g * p.w_stride : p.Ws;
  }

  // global source of this thread's 16-byte chunks (row r = c / 8, chunk q = c % 8)
  // A rows past the group's end are not loaded (their outputs are never stored):
  // a tile with few rows (decode) then reads only its live rows.
  const bf16_t *a_src[PA];
  const bf16_t *b_src[PB];
  bool a_live[PA];
#pragma unroll
  for (int i = 0; i < PA; ++i) {
    const int c = i * 256 + tid;
    const int r = c >> 3;
    a_live[i] = r < valid;
    const int rr = row0 + (r < valid ? r : 0);
    const long long arow = GATE_UP ? (long long)p.row_token[rr] : (long long)rr;
    a_src[i] = p.A + arow * p.lda + t.ks * p.kc + (c & 7) * 8;
  }
#pragma unroll
  for (int i = 0; i < PB; ++i) {
    const int c = i * 256 + tid;
    const int r = c >> 3;
    int wrow;
    if (GATE_UP)
      wrow = (r < BN / 2) ? t.nt * (BN / 2) + r : p.inter + t.nt * (BN / 2) + (r - BN / 2);
    else
      wrow = t.nt * BN + r;
    b_src[i] = Wg + (long long)wrow * p.ldw + t.ks * p.kc + (c & 7) * 8;
  }

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  // LDS row of wave subtile j of B (gate/up pairs for GATE_UP)
  int b_row[TN];
#pragma unroll
  for (int j = 0; j < TN; ++j)
    b_row[j] = GATE_UP ? ((j < TN / 2) ? wn * (WTN / 2) + j * 32 : BN / 2 + wn * (WTN / 2) + (j - TN / 2) * 32)
                       : wn * WTN + j * 32;

  // The prefetch registers are plain arrays indexed only by unrolled constants
  // (macros, not lambdas taking their address), so they stay in VGPRs.
#define EXF_GLOAD(RA, RB, K0)                                                                \
  do {                                                                                       \
    _Pragma("unroll") for (int i_ = 0; i_ < PA; ++i_) if (a_live[i_]) RA[i_] =               \
        *reinterpret_cast<const u32x4 *>(a_src[i_] + (K0));                                  \
    _Pragma("unroll") for (int i_ = 0; i_ < PB; ++i_) RB[i_] = load_w16<ONCE>(b_src[i_] + (K0)); \
  } while (0)
#define EXF_LSTORE(RA, RB, BUF)                                                              \
  do {                                                                                       \
    bf16_t *As_ = smem + (BUF) * BM * kBK;                                                   \
    bf16_t *Bs_ = smem + 2 * BM * kBK + (BUF) * BN * kBK;                                    \
    _Pragma("unroll") for (int i_ = 0; i_ < PA; ++i_) {                                      \
      const int c_ = i_ * 256 + tid;                                                         \
      *reinterpret_cast<u32x4 *>(&As_[swz(c_ >> 3, c_ & 7)]) = RA[i_];                        \
    }                                                                                        \
    _Pragma("unroll") for (int i_ = 0; i_ < PB; ++i_) {                                      \
      const int c_ = i_ * 256 + tid;                                                         \
      *reinterpret_cast<u32x4 *>(&Bs_[swz(c_ >> 3, c_ & 7)]) = RB[i_];                        \
    }                                                                                        \
  } while (0)
// Fragments of k-step s+1 are read while the MFMAs of step s run.
#define EXF_FRAGS(A_, B_, S_)                                                                \
  do {                                                                                       \
    const int ch_ = (S_) * 2 + (lane >> 5);                                                  \
    _Pragma("unroll") for (int i_ = 0; i_ < TM; ++i_) A_[i_] =                               \
        *reinterpret_cast<const bf16x8 *>(&As_[swz(wm * WTM + i_ * 32 + (lane & 31), ch_)]); \
    _Pragma("unroll") for (int j_ = 0; j_ < TN; ++j_) B_[j_] =                               \
        *reinterpret_cast<const bf16x8 *>(&Bs_[swz(b_row[j_] + (lane & 31), ch_)]);           \
  } while (0)
#define EXF_MMA(A_, B_)                                                                      \
  do {                                                                                       \
    _Pragma("unroll") for (int i_ = 0; i_ < TM; ++i_)                                        \
        _Pragma("unroll") for (int j_ = 0; j_ < TN; ++j_) acc[i_][j_] =                      \
            __builtin_amdgcn_mfma_f32_32x32x16_bf16(A_[i_], B_[j_], acc[i_][j_], 0, 0, 0);   \
  } while (0)
#define EXF_COMPUTE(BUF)                                                                     \
  do {                                                                                       \
    const bf16_t *As_ = smem + (BUF) * BM * kBK;                                             \
    const bf16_t *Bs_ = smem + 2 * BM * kBK + (BUF) * BN * kBK;                              \
    bf16x8 a0_[TM], b0_[TN], a1_[TM], b1_[TN];                                               \
    EXF_FRAGS(a0_, b0_, 0);                                                                  \
    EXF_FRAGS(a1_, b1_, 1);                                                                  \
    EXF_MMA(a0_, b0_);                                                                       \
    EXF_FRAGS(a0_, b0_, 2);                                                                  \
    EXF_MMA(a1_, b1_);                                                                       \
    EXF_FRAGS(a1_, b1_, 3);                                                                  \
    EXF_MMA(a0_, b0_);                                                                       \
    EXF_MMA(a1_, b1_);                                                                       \
  } while (0)

  // Schedule of one phase: the next tile's global loads first, fragments of
  // k-step s+1 read while the MFMAs of step s run, and the staged tile written to
  // the other LDS buffer before the last MFMA group.
#define EXF_SCHEDULE()                                                               \
  do {                                                                               \
    __builtin_amdgcn_sched_group_barrier(0x020, PA + PB, 0); /* VMEM read */         \
    __builtin_amdgcn_sched_group_barrier(0x100, 2 * (TM + TN), 0); /* DS read */     \
    __builtin_amdgcn_sched_group_barrier(0x008, TM * TN, 0); /* MFMA */              \
    __builtin_amdgcn_sched_group_barrier(0x100, TM + TN, 0);                          \
    __builtin_amdgcn_sched_group_barrier(0x008, TM * TN, 0);                          \
    __builtin_amdgcn_sched_group_barrier(0x100, TM + TN, 0);                          \
    __builtin_amdgcn_sched_group_barrier(0x008, TM * TN, 0);                          \
    __builtin_amdgcn_sched_group_barrier(0x200, PA + PB, 0); /* DS write */           \
    __builtin_amdgcn_sched_group_barrier(0x008, TM * TN, 0);                          \
  } while (0)

  // Pairs of phases over the two LDS buffers, no early exit (one loop exit keeps
  // the accumulators in one register set); an odd tile count ends with buffer 0.
  // LDS buffer (kt & 1) holds tile kt and the other register set holds tile kt + 1,
  // so each tile's loads are covered by two compute phases.  Loads past the last
  // tile re-read the last tile (k clamped) and land in a buffer that is never read
  // again, so each phase is one straight-line block.
  const int KT = p.kc / kBK;
  const int k_last = (KT - 1) * kBK;
  auto main_loop = [&](auto once) __attribute__((always_inline)) {
    constexpr bool ONCE = decltype(once)::value;
    u32x4 ra0[PA], rb0[PB], ra1[PA], rb1[PB];
    _Pragma("unroll") for (int i_ = 0; i_ < PA; ++i_) ra0[i_] = ra1[i_] = u32x4{0u, 0u, 0u, 0u};
    EXF_GLOAD(ra0, rb0, 0);
    EXF_LSTORE(ra0, rb0, 0);
    EXF_GLOAD(ra1, rb1, min(kBK, k_last));
    __syncthreads();
    int kt = 0;
    for (; kt + 2 <= KT; kt += 2) {
      EXF_GLOAD(ra0, rb0, min((kt + 2) * kBK, k_last));
      EXF_COMPUTE(0);
      EXF_LSTORE(ra1, rb1, 1);
      EXF_SCHEDULE();
      __syncthreads();
      EXF_GLOAD(ra1, rb1, min((kt + 3) * kBK, k_last));
      EXF_COMPUTE(1);
      EXF_LSTORE(ra0, rb0, 0);
      EXF_SCHEDULE();
      __syncthreads();
    }
    if (kt < KT) EXF_COMPUTE(0);
  };
  if (!PLAIN && __builtin_amdgcn_readfirstlane(t.alone))
    main_loop(std::true_type{});
  else
    main_loop(std::false_type{});
#undef EXF_GLOAD
#undef EXF_LSTORE
#undef EXF_COMPUTE
#undef EXF_FRAGS
#undef EXF_MMA
#undef EXF_SCHEDULE

  // ---- epilogue ----
#pragma unroll
  for (int i = 0; i < TM; ++i) {
#pragma unroll
    for (int j = 0; j < (GATE_UP ? TN / 2 : TN); ++j) {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int ml = wm * WTM + i * 32 + (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3);
        if (ml < valid) {
          const int row = row0 + ml;
          if (GATE_UP) {
            const int n = t.nt * (BN / 2) + wn * (WTN / 2) + j * 32 + (lane & 31);
            p.H[(long long)row * p.inter + n] = f32_to_bf16(silu(acc[i][j][r]) * acc[i][j + TN / 2][r]);
          } else {
            const int n = t.nt * BN + wn * WTN + j * 32 + (lane & 31);
            if (PLAIN)
              p.Y[((long long)t.ks * p.rows + row) * p.d + n] = acc[i][j][r];
            else if (DIRECT)
              p.y[(long long)p.row_token[row] * p.d + n] = f32_to_bf16(acc[i][j][r] * p.row_w[row]);
            else if (p.Yh)
              p.Yh[(long long)row * p.d + n] = f32_to_bf16(acc[i][j][r]);
            else
              p.Y[((long long)t.ks * p.rows + row) * p.d + n] = acc[i][j][r] * p.row_w[row];
          }
        }
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Wide tile for the prefill GEMMs (many rows per retained expert): 256x256
// macro tile, eight waves (two per SIMD) of 4x2 MFMA tiles each (gate/up: gate
// columns with the matching up columns); a group's last rows, when at most 128,
// form a 128x512 tile over two n-tiles.  Four waves of 128x128 each (one per
// SIMD, accumulators in AGPRs) measured 7-11% slower against eight waves that
// met one barrier a stage.  The operands go from global memory
// straight into LDS (global_load_lds_dwordx4) through a ring of reduction
// stages: no staging registers and no LDS write instructions.  Against 128x128
// tiles the bytes loaded per flop halve, and the weight panel a tile shares
// with the other m-tiles of its expert is fetched from HBM fewer times: a
// Mixtral-shaped launch reads 3.0-3.1 GB, 2.0 GB of them needed, against 3.8-5
// GB (2.4 GB with one barrier a stage, one stage ahead: tiles whose loads run 1.5
// stages ahead drift further apart, at less time all the same).  Measured with one
// barrier a stage, the 64-wide stages with two ring buffers beat 32-wide stages
// with four or five buffers (more bytes in flight, but 64-byte row pieces and
// twice the barriers).
// ---------------------------------------------------------------------------
constexpr int kWide = 256, kWideWaves = 8, kWideBK = 64;

// LDS byte address of a shared-memory pointer (for M0).
__device__ __forceinline__ uint32_t lds_addr(const void *ptr) {
  return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void *)ptr;
}

// One 16-byte chunk per lane from global g into the 1 KiB LDS block at byte
// address lds (wave-uniform): lane l lands at lds + 16 l.  M0 holds the block
// address; one wait state separates its write from the load.  The statement
// clobbers M0, which the compiler does not save around it: the kernels that
// use it must give the compiler no reason to hold a value in M0 (register
// arrays indexed by compile-time constants only, no indirect register moves).
// The compiler's own LDS-DMA builtin keeps M0 safe but schedules the main loop
// 2% slower (its conservative waits).
__device__ __forceinline__ void lds_dma16(const void *g, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off"
               :
               : "v"(g), "s"(lds)
               : "memory", "m0");
}

// Wide tile of logical id L.  The tile list counts rows of a group in
// 128-row units (u_g = ceil(rows_g / 128), prefix tile_start); per group and
// per pair j of n-tiles (2j, 2j + 1) there are u_g tiles: the M = u_g / 2
// full-height m-tiles of n-tile 2j, then those of n-tile 2j + 1 (m-tile
// fastest: the tiles that share a weight panel run side by side), then, for
// odd u_g, one tail tile of at most 128 rows that spans both n-tiles.  The
// tail costs half a tile and starts and ends with its neighbours, so the tiles
// that share a panel stay in step (a half-height tile on one n-tile would run
// ahead of its siblings and fetch the panel a second time).
__device__ __forceinline__ void wide_tile_at(const GemmKArgs &p, int L, TileId &t) {
  const int pairs = p.n_tiles / 2;
  int lo = 0, hi = p.groups;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (p.tile_start[mid] * pairs <= L) lo = mid; else hi = mid;
  }
  const int u_g = p.tile_start[lo + 1] - p.tile_start[lo];
  const int local = L - p.tile_start[lo] * pairs;
  const int j = local / u_g, u = local % u_g, M = u_g >> 1;
  t.g = lo;
  t.ks = 0;
  if (u < 2 * M) {
    t.nt = 2 * j + u / M;
    t.mt = u % M;
    t.dbl = 0;
  } else {
    t.nt = 2 * j;
    t.mt = M;
    t.dbl = 1;
  }
}

// Slot of 16-byte chunk q in a 128-byte tile row (an involution in q): the
// Gray-code swizzle of the register-staged tiles, so that the chunk columns one
// ds_read_b128 takes from consecutive rows land in distinct LDS banks.
__device__ __forceinline__ int wide_slot(int r, int q) { return q ^ ((r ^ (r >> 1)) & 7); }

// 32x32 MFMA tiles per wave: four row blocks by two column blocks (tail tiles:
// two by four, kept as [2 (pair) + row block][column of the pair])
constexpr int kWideTM = 4, kWideTN = 2;
constexpr int kWideBN = kWide;  // tile columns (gate/up: weight rows)
// LDS ring: two stages of the 256 x 256 tile (128 KiB) or of the 128 x 512 tail (160 KiB)
constexpr int kWideSmemElems = 2 * (kWide / 2 + 2 * kWideBN) * kWideBK;

// Main loop of one wide tile over the reduction stages [k0, k1) of 64 columns
// (at least two): zeroes acc and leaves the products in it.  The LDS ring holds
// two stages in half tiles of 128 rows: A0, A1 (token rows) and B0, B1 (weight
// rows; gate/up: the gate rows and the up rows), or, for a 128 x 512 tail tile
// (DBL), A0 and B0 .. B3 (n-tile nt: B0, B1; nt + 1: B2, B3).  Wave (wm, wn) owns
// rows 64 i + 32 wm .. + 31 (i = 0, 1) of every A half and rows 32 wn .. + 31 of
// every B half: four quadrants of 64 x 32.
//
// A stage takes four phases, one quadrant each.  A phase reads one half tile's
// fragments from LDS, issues the loads of half tiles ahead, meets the barrier,
// and then runs the quadrant's MFMAs alone (each waits for its own fragments),
// up to a second barrier.  The two waves of a SIMD (w and w + 4) run half a phase
// apart: while one issues MFMAs back to back, the other reads fragments and
// issues loads, so the matrix pipe waits for neither.  Full tiles take the
// quadrants of a stage in ring buffer 0 in the order of weight halves 0 1 1 0 and
// in buffer 1 in 1 0 0 1: the last phase of a stage then reads the next stage's
// first weight half into registers that are already free.  Tail tiles go
// through B0 .. B3 on two register sets, the last phase reading B3 and the next
// B0.
//
// Half tiles are issued in the order they are read.  Full tiles: numbered so,
// phase p reads tile p + 1 and issues tile p + 7 (two loads a wave) into the slot
// that phase p - 2 read: the later waves met the barrier that ends their phase
// p - 2 before this phase began, and every wave waits for all its LDS reads
// before that barrier.  (The MFMAs alone do not order them: those of a stage's
// last phase do not use the weight half that it reads for the next stage, and
// no MFMA precedes the first phase.  The reads are a block of MFMAs old by then,
// so the wait costs nothing: Qwen3-shaped prefill 461 us a layer without it, 464
// with it, on two cards.)  Before the phase's barrier tile p + 2 must have landed:
// at most five tiles, 10 loads, stay in flight; a load has six phases (1.5
// stages) to land.  Tail tiles: five tiles a stage on four phases (the second
// issues two), six or seven stay in flight.
//
// One barrier a stage with every wave reading, loading and multiplying at once
// (one stage ahead) kept the MFMA pipes busy 57% of the cycles at 1.88 GHz on a
// Mixtral-shaped gate/up launch of ragged groups, this 66-67% at 1.76 and 1.67 GHz
// (two cards: the launch is held by the chip's power); 4096 rows on 8 such
// experts, 512 each, gate/up 877 -> 842 us (1143 TFLOP/s), down 437 -> 415.  Ragged
// groups gain most, in their tail tiles (8192 Qwen3-shaped tokens, K' = 4: 247 ->
// 229 and 177 -> 156 us; pipes busy 47.5 -> 52% and 36 -> 40%).
//
// TMV: 32-row blocks of the wave that hold rows of the group (full: 2 .. 4, tail:
// 0 .. 2; the others' fragments are not read and their MFMAs not issued).
template <bool GATE_UP, bool DBL, int TMV>
__device__ __forceinline__ void wide_tile_mma(const GemmKArgs &p, const TileId &t, int row0, int valid,
                                              int k0, int k1, bf16_t *smem,
                                              f32x16 (&acc)[kWideTM][kWideTN]) {
  constexpr int HALF = 128 * kWideBK;             // elements of a half tile
  constexpr int NA = DBL ? 1 : 2, NB = DBL ? 4 : 2;  // half tiles of a stage
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave >> 2, wn = wave & 3;
  const bf16_t *Wg = (t.g < p.n_experts) ? p.W + (long long)t.g * p.w_stride : p.Ws;
  // Wave w fills 1 KiB blocks w and w + 8 of a half tile: rows 8 w .. + 7 and 64
  // further, lane l the chunk that the swizzle puts at slot l % 8 of row l / 8.
  const bf16_t *sa[NA][2], *sb[NB][2];
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int rh = (u * 8 + wave) * 8 + (lane >> 3);  // row of the half tile
    const int q = wide_slot(rh, lane & 7);
#pragma unroll
    for (int h = 0; h < NA; ++h) {
      const int r = h * 128 + rh;
      const int rr = row0 + (r < valid ? r : 0);  // padding rows re-read the first one, never stored
      const long long arow = GATE_UP ? (long long)p.row_token[rr] : (long long)rr;
      sa[h][u] = p.A + arow * p.lda + (long long)k0 * kWideBK + q * 8;
    }
#pragma unroll
    for (int g = 0; g < NB; ++g) {
      const int wrow = GATE_UP ? (g & 1) * p.inter + (t.nt + (g >> 1)) * 128 + rh : t.nt * kWideBN + g * 128 + rh;
      sb[g][u] = Wg + (long long)wrow * p.ldw + (long long)k0 * kWideBK + q * 8;
    }
  }
  const uint32_t lds0 = lds_addr(smem) + wave * 1024;
#pragma unroll
  for (int i = 0; i < kWideTM; ++i)
#pragma unroll
    for (int j = 0; j < kWideTN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
  // fragment of k16 step s: row lane % 32 of a 32-row block, chunk 2 s + lane / 32
  const bf16_t *fa_at[4], *fb_at[4];
#pragma unroll
  for (int s_ = 0; s_ < 4; ++s_) {
    const int off = (lane & 31) * kWideBK + wide_slot(lane & 31, 2 * s_ + (lane >> 5)) * 8;
    fa_at[s_] = smem + wm * 32 * kWideBK + off;
    fb_at[s_] = smem + 2 * NA * HALF + wn * 32 * kWideBK + off;
  }
  bf16x8 fa[2][4], fb[2][4];

  // half tiles in LDS: A half h of ring buffer b at slot 2 h + b, B half g at 2 NA + 2 g + b
#define EXF_P_ISSUE(SRC_, SLOT_)                                                        \
  do {                                                                                  \
    _Pragma("unroll") for (int u_ = 0; u_ < 2; ++u_) {                                  \
      lds_dma16(SRC_[u_], lds0 + (uint32_t)(SLOT_) * (HALF * 2) + u_ * 8192);           \
      SRC_[u_] += kWideBK;                                                              \
    }                                                                                   \
  } while (0)
#define EXF_P_ISSUE_A(H_, BUF_) EXF_P_ISSUE(sa[H_], 2 * (H_) + (BUF_))
#define EXF_P_ISSUE_B(G_, BUF_) EXF_P_ISSUE(sb[G_], 2 * NA + 2 * (G_) + (BUF_))
  // blocks of quadrant row half H_ (tail tiles: always the first)
#define EXF_P_LIVE(H_, I_) (2 * (DBL ? 0 : (H_)) + (I_) < TMV)
#define EXF_P_READ_A(H_, BUF_)                                                          \
  do {                                                                                  \
    _Pragma("unroll") for (int s_ = 0; s_ < 4; ++s_)                                    \
        _Pragma("unroll") for (int i_ = 0; i_ < 2; ++i_) if (EXF_P_LIVE(H_, i_))        \
            fa[i_][s_] = *reinterpret_cast<const bf16x8 *>(                             \
                fa_at[s_] + (2 * (H_) + (BUF_)) * HALF + i_ * 64 * kWideBK);            \
  } while (0)
#define EXF_P_READ_B(G_, BUF_)                                                          \
  do {                                                                                  \
    if (TMV > 0)                                                                        \
      _Pragma("unroll") for (int s_ = 0; s_ < 4; ++s_) fb[(G_) & 1][s_] =               \
          *reinterpret_cast<const bf16x8 *>(fb_at[s_] + (2 * (G_) + (BUF_)) * HALF);    \
  } while (0)
#define EXF_P_BARRIER() asm volatile("s_barrier" ::: "memory")
  // the end of a phase: the wave's LDS reads have ended, then the barrier
#define EXF_P_CLOSE() asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory")
  // products of row half H_ (full tiles) or weight pair H_ (tail tiles) with weight half J_ of it
#define EXF_P_MMA(H_, J_)                                                               \
  do {                                                                                  \
    __builtin_amdgcn_sched_barrier(0);                                                  \
    __builtin_amdgcn_s_setprio(1);                                                      \
    _Pragma("unroll") for (int s_ = 0; s_ < 4; ++s_)                                    \
        _Pragma("unroll") for (int i_ = 0; i_ < 2; ++i_) if (EXF_P_LIVE(H_, i_))        \
            acc[2 * (H_) + i_][J_] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(           \
                fb[J_][s_], fa[i_][s_], acc[2 * (H_) + i_][J_], 0, 0, 0);               \
    __builtin_amdgcn_s_setprio(0);                                                      \
    __builtin_amdgcn_sched_barrier(0);                                                  \
    EXF_P_CLOSE();                                                                      \
  } while (0)
  // at most VM_ of the wave's loads are in flight, then the barrier
#define EXF_P_WAIT(VM_) asm volatile("s_waitcnt vmcnt(" #VM_ ")\n\ts_barrier" ::: "memory")
  // One stage of a full tile from ring buffer BUF_.  FILL1_: the first phase issues
  // the last half tile of the next stage; FILL_: the others issue three of the
  // stage after it; V1_ .. V4_: loads in flight allowed; NEXT_: a stage follows.
#define EXF_P_STAGE(BUF_, FILL1_, FILL_, V1_, V2_, V3_, V4_, NEXT_)                     \
  do {                                                                                  \
    EXF_P_READ_A(0, BUF_);                                                              \
    if (FILL1_) EXF_P_ISSUE_A(1, 1 - (BUF_));                                           \
    EXF_P_WAIT(V1_);                                                                    \
    EXF_P_MMA(0, BUF_);                                                                 \
    EXF_P_READ_B(1 - (BUF_), BUF_);                                                     \
    if (FILL_) EXF_P_ISSUE_B(BUF_, BUF_);                                               \
    EXF_P_WAIT(V2_);                                                                    \
    EXF_P_MMA(0, 1 - (BUF_));                                                           \
    EXF_P_READ_A(1, BUF_);                                                              \
    if (FILL_) EXF_P_ISSUE_A(0, BUF_);                                                  \
    EXF_P_WAIT(V3_);                                                                    \
    EXF_P_MMA(1, 1 - (BUF_));                                                           \
    if (NEXT_) EXF_P_READ_B(1 - (BUF_), 1 - (BUF_));                                    \
    if (FILL_) EXF_P_ISSUE_B(1 - (BUF_), BUF_);                                         \
    EXF_P_WAIT(V4_);                                                                    \
    EXF_P_MMA(1, BUF_);                                                                 \
  } while (0)
  // One stage of a tail tile: FILL1_: B2, B3 of the next stage; FILL_: B0, A, B1 of
  // the stage after it.
#define EXF_P_TAIL(BUF_, FILL1_, FILL_, V1_, V2_, V3_, V4_, NEXT_)                      \
  do {                                                                                  \
    EXF_P_READ_A(0, BUF_);                                                              \
    if (FILL1_) EXF_P_ISSUE_B(NB - 2, 1 - (BUF_));                                      \
    EXF_P_WAIT(V1_);                                                                    \
    EXF_P_MMA(0, 0);                                                                    \
    EXF_P_READ_B(1, BUF_);                                                              \
    if (FILL1_) EXF_P_ISSUE_B(NB - 1, 1 - (BUF_));                                      \
    if (FILL_) EXF_P_ISSUE_B(0, BUF_);                                                  \
    EXF_P_WAIT(V2_);                                                                    \
    EXF_P_MMA(0, 1);                                                                    \
    EXF_P_READ_B(NB - 2, BUF_);                                                         \
    if (FILL_) EXF_P_ISSUE_A(0, BUF_);                                                  \
    EXF_P_WAIT(V3_);                                                                    \
    EXF_P_MMA(1, 0);                                                                    \
    EXF_P_READ_B(NB - 1, BUF_);                                                         \
    if (NEXT_) EXF_P_READ_B(0, 1 - (BUF_));                                             \
    if (FILL_) EXF_P_ISSUE_B(1, BUF_);                                                  \
    EXF_P_WAIT(V4_);                                                                    \
    EXF_P_MMA(1, 1);                                                                    \
  } while (0)
  // the loads of the two first stages, in reading order, that no phase issues;
  // then the first weight half (tiles 0 and 1 have landed)
#define EXF_P_BEGIN(BUF_)                                                               \
  do {                                                                                  \
    EXF_P_ISSUE_B(DBL ? 0 : (BUF_), BUF_);                                              \
    EXF_P_ISSUE_A(0, BUF_);                                                             \
    EXF_P_ISSUE_B(DBL ? 1 : 1 - (BUF_), BUF_);                                          \
    if (DBL) {                                                                          \
      EXF_P_ISSUE_B(NB - 2, BUF_);                                                      \
      EXF_P_ISSUE_B(NB - 1, BUF_);                                                      \
      EXF_P_ISSUE_B(0, 1 - (BUF_));                                                     \
      EXF_P_ISSUE_A(0, 1 - (BUF_));                                                     \
      EXF_P_ISSUE_B(1, 1 - (BUF_));                                                     \
      EXF_P_WAIT(12);                                                                   \
    } else {                                                                            \
      EXF_P_ISSUE_A(NA - 1, BUF_);                                                      \
      EXF_P_ISSUE_B(1 - (BUF_), 1 - (BUF_));                                            \
      EXF_P_ISSUE_A(0, 1 - (BUF_));                                                     \
      EXF_P_ISSUE_B(BUF_, 1 - (BUF_));                                                  \
      EXF_P_WAIT(10);                                                                   \
    }                                                                                   \
    EXF_P_READ_B(DBL ? 0 : (BUF_), BUF_);                                               \
  } while (0)

  // an odd count of stages starts in buffer 1, so the last stage is always in buffer 1
  int left = k1 - k0 - 2;
  const bool odd = left & 1;
  if (odd)
    EXF_P_BEGIN(1);
  else
    EXF_P_BEGIN(0);
  if (wave >= 4) EXF_P_CLOSE();  // half a phase behind; the first weight half has been read
  if constexpr (DBL) {
    if (odd) {
      EXF_P_TAIL(1, true, true, 12, 14, 12, 12, true);
      --left;
    }
    for (; left > 0; left -= 2) {
      EXF_P_TAIL(0, true, true, 12, 14, 12, 12, true);
      EXF_P_TAIL(1, true, true, 12, 14, 12, 12, true);
    }
    EXF_P_TAIL(0, true, false, 12, 12, 8, 6, true);
    EXF_P_TAIL(1, false, false, 4, 2, 0, 0, false);
  } else {
    if (odd) {
      EXF_P_STAGE(1, true, true, 10, 10, 10, 10, true);
      --left;
    }
    for (; left > 0; left -= 2) {
      EXF_P_STAGE(0, true, true, 10, 10, 10, 10, true);
      EXF_P_STAGE(1, true, true, 10, 10, 10, 10, true);
    }
    EXF_P_STAGE(0, true, false, 10, 8, 6, 4, true);
    EXF_P_STAGE(1, false, false, 2, 0, 0, 0, false);
  }
  if (wave < 4) EXF_P_BARRIER();
#undef EXF_P_ISSUE
#undef EXF_P_ISSUE_A
#undef EXF_P_ISSUE_B
#undef EXF_P_LIVE
#undef EXF_P_READ_A
#undef EXF_P_READ_B
#undef EXF_P_BARRIER
#undef EXF_P_CLOSE
#undef EXF_P_MMA
#undef EXF_P_WAIT
#undef EXF_P_STAGE
#undef EXF_P_TAIL
#undef EXF_P_BEGIN
}

// Tile row and column of accumulator tile (i, j) of wave (wm, wn), and the
// output column of gate/up pair (i, 0), (i, 1).
template <bool DBL> __device__ __forceinline__ int wide_row(int wm, int i) {
  return (DBL ? 0 : (i >> 1) * 128) + (i & 1) * 64 + wm * 32;
}
template <bool DBL> __device__ __forceinline__ int wide_col(int wn, int i, int j) {
  return (DBL ? (i >> 1) * kWideBN : 0) + j * 128 + wn * 32;
}
template <bool DBL> __device__ __forceinline__ int wide_pair_col(int wn, int i) {
  return (DBL ? (i >> 1) * 128 : 0) + wn * 32;
}

// Accumulator layout: the MFMAs take the weight fragment as their first
// operand, so register r of tile (i, j) of wave (wm, wn) holds tile row (token)
// wide_row + lane % 32 and tile column wide_col + 8 (r / 4) + 4 (lane / 32) +
// r % 4: each lane owns four runs of four consecutive columns of one row,
// stored 8 (bf16) or 16 (fp32) bytes at a time.
__device__ __forceinline__ void store4_bf16(bf16_t *dst, float a, float b, float c, float d) {
  typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
  const bf16x4 v = {(__bf16)a, (__bf16)b, (__bf16)c, (__bf16)d};   // two v_cvt_pk_bf16_f32
  *reinterpret_cast<bf16x4 *>(dst) = v;
}
// The same as a non-temporal store, for the layer output y written by the wide
// down GEMM (nothing in the layer reads it back): its lines are not kept dirty
// in the caches, whose later write-back otherwise lands in the next kernels (a
// decode forward right after the Mixtral-shaped prefill: 265.0-265.2 against
// 268.9-270.1 us, the prefill unchanged).
__device__ __forceinline__ void store4_bf16_nt(bf16_t *dst, float a, float b, float c, float d) {
  typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
  typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
  const bf16x4 v = {(__bf16)a, (__bf16)b, (__bf16)c, (__bf16)d};
  __builtin_nontemporal_store(*reinterpret_cast<const u32x2 *>(&v), reinterpret_cast<u32x2 *>(dst));
}

// Finished tile, from the registers: gate/up writes H = SiLU(gate) * up, the
// direct down projection y, scaled by the row's routing weight.
template <bool GATE_UP, bool DBL>
__device__ __forceinline__ void wide_store(const GemmKArgs &p, const TileId &t, int row0, int valid,
                                           const f32x16 (&acc)[kWideTM][kWideTN]) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wm = wave >> 2, wn = wave & 3;
  const int c4 = 4 * (lane >> 5);
#pragma unroll
  for (int i = 0; i < kWideTM; ++i) {
    const int ml = wide_row<DBL>(wm, i) + (lane & 31);
    if (ml >= valid) continue;
    const int row = row0 + ml;
    if (GATE_UP) {
      bf16_t *dst = p.H + (long long)row * p.inter + t.nt * (kWideBN / 2) + wide_pair_col<DBL>(wn, i) + c4;
      const f32x16 &gt = acc[i][0], &up = acc[i][1];
#pragma unroll
      for (int g = 0; g < 4; ++g)
        store4_bf16(dst + 8 * g, silu(gt[4 * g]) * up[4 * g], silu(gt[4 * g + 1]) * up[4 * g + 1],
                    silu(gt[4 * g + 2]) * up[4 * g + 2], silu(gt[4 * g + 3]) * up[4 * g + 3]);
    } else {
      const float w = p.row_w[row];
      bf16_t *dst = p.y + (long long)p.row_token[row] * p.d + t.nt * kWideBN + c4;
#pragma unroll
      for (int j = 0; j < kWideTN; ++j)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const f32x16 &c = acc[i][j];
          store4_bf16_nt(dst + wide_col<DBL>(wn, i, j) + 8 * g, c[4 * g] * w, c[4 * g + 1] * w, c[4 * g + 2] * w,
                         c[4 * g + 3] * w);
        }
    }
  }
}

// Finished bf16 rows of the down projection through LDS (the ring is free after
// the main loop): each lane writes its runs of four columns into a row-major
// bf16 tile, and the workgroup then stores whole rows 16 bytes a lane, so one
// store instruction covers a few complete rows instead of 32 scattered 16-byte
// pieces (Qwen3-shaped prefill: down 200 -> 177 us).  For H and the direct y it
// gains nothing.
template <bool DBL>
__device__ __forceinline__ void wide_store_lds(const GemmKArgs &p, const TileId &t, int row0, int valid,
                                               const f32x16 (&acc)[kWideTM][kWideTN], bf16_t *smem) {
  constexpr int BM = DBL ? kWide / 2 : kWide;
  constexpr int COLS = (DBL ? 2 : 1) * kWideBN;               // output columns of the tile
  constexpr int PITCH = COLS * 2 + 16;                        // LDS bytes per row (padded)
  static_assert(BM * PITCH <= kWideSmemElems * 2, "staging tile fits the ring");
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wm = wave >> 2, wn = wave & 3;
  const int c4 = 4 * (lane >> 5);
  char *lds = reinterpret_cast<char *>(smem);
#pragma unroll
  for (int i = 0; i < kWideTM; ++i) {
    bf16_t *rowp = reinterpret_cast<bf16_t *>(lds + (wide_row<DBL>(wm, i) + (lane & 31)) * PITCH) + c4;
#pragma unroll
    for (int j = 0; j < kWideTN; ++j)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const f32x16 &c = acc[i][j];
        store4_bf16(rowp + wide_col<DBL>(wn, i, j) + 8 * g, c[4 * g], c[4 * g + 1], c[4 * g + 2], c[4 * g + 3]);
      }
  }
  lds_barrier();
  constexpr int CPR = COLS / 8;                               // 16-byte chunks per row
  for (int q = threadIdx.x; q < BM * CPR; q += 64 * kWideWaves) {
    const int ml = q / CPR, ch = q % CPR;
    if (ml >= valid) continue;
    *reinterpret_cast<u32x4 *>(p.Yh + (long long)(row0 + ml) * p.d + t.nt * kWideBN + ch * 8) =
        *reinterpret_cast<const u32x4 *>(lds + ml * PITCH + ch * 16);
  }
}

// ---------------------------------------------------------------------------
// Wide-tile launches: whole rounds of tiles plus a split remainder.  With one
// workgroup per CU (the ring takes 128 KiB of LDS), tiles run in rounds of G =
// CU count; the last, partial round would leave most CUs idle.  When it holds
// at most half a round, its rem tiles have their reductions cut into s equal
// ranges of stages (s = G / rem, at most kWideMaxSplit, at least four stages a
// range) on separate workgroups: range c of remainder tile r leaves its fp32
// partial tile in P[r s + c], and expert_wide_fixup adds the s partials in
// range order and applies the epilogue.  Whole tiles keep the lock-step order
// in which the m-tiles of one weight panel and the n-tiles of one row block
// share an XCD's L2 (dealing the stages of every tile out evenly instead
// breaks that sharing: measured slower).  The ranges of one remainder tile are
// disjoint in K, so the remainder is laid out range-major: neighbouring
// workgroups take neighbouring tiles over the same stages.  The sums depend on
// the problem and G only, so the result is deterministic.
// ---------------------------------------------------------------------------
constexpr int kWideTileElems = kWide * kWide;
constexpr int kWideMaxSplit = 16;

struct WideSplit {
  int ndp;  // tiles run whole: logical ids 0 .. ndp - 1
  int rem;  // tiles split s ways: logical ids ndp .. ndp + rem - 1
  int s;
};
__device__ __forceinline__ WideSplit wide_split(const GemmKArgs &p, int G) {
  const int total = p.tile_start[p.groups] * (p.n_tiles / 2);
  const int rem = total % G;
  const int s = rem > 0 ? min(G / rem, min(kWideMaxSplit, p.kc / kWideBK / 4)) : 1;
  if (rem > 0 && s >= 2) return WideSplit{total - rem, rem, s};
  return WideSplit{total, 0, 1};
}

// Finished float32 tile through LDS in two halves of 128 rows x 256 columns
// (full tiles: the row halves; tails: the n-tiles), whole rows of 1 KiB a wave
// instead of 32-byte pieces of 32 rows: row ml of half h goes to dst + ml * ld +
// h * kWideBN (tails), scaled by scale(ml).  Kept rows of a calibration (4096
// tokens x 8, d 2048): down 190 -> 170 us; split partials 1-3 us a launch.
template <bool DBL, typename Scale>
__device__ __forceinline__ void wide_store_f32(float *dst, long long ld, int valid, Scale scale,
                                               const f32x16 (&acc)[kWideTM][kWideTN], bf16_t *smem) {
  constexpr int PITCH = kWideBN * 4 + 16;  // LDS bytes per row (padded)
  static_assert(kWide / 2 * PITCH <= kWideSmemElems * 2, "staging half fits the ring");
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave >> 2, wn = wave & 3;
  char *lds = reinterpret_cast<char *>(smem);
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    if (h) lds_barrier();
#pragma unroll
    for (int ib = 0; ib < 2; ++ib) {
      const int i = 2 * h + ib, ml = wide_row<DBL>(wm, i) + (lane & 31);
      const float w = scale(min(ml, valid - 1));
      char *rowp = lds + (wide_row<true>(wm, i) + (lane & 31)) * PITCH + 16 * (lane >> 5);
#pragma unroll
      for (int j = 0; j < kWideTN; ++j)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const f32x16 &c = acc[i][j];
          *reinterpret_cast<float4 *>(rowp + 4 * (wide_col<false>(wn, i, j) + 8 * g)) =
              make_float4(c[4 * g] * w, c[4 * g + 1] * w, c[4 * g + 2] * w, c[4 * g + 3] * w);
        }
    }
    lds_barrier();
    for (int r = wave; r < kWide / 2; r += kWideWaves) {
      const int ml = (DBL ? 0 : h * (kWide / 2)) + r;
      if (ml >= valid) break;
      const float4 v = *reinterpret_cast<const float4 *>(lds + r * PITCH + lane * 16);
      *reinterpret_cast<float4 *>(dst + ml * ld + (DBL ? h * kWideBN : 0) + lane * 4) = v;
    }
  }
}

// Workgroup blockIdx.x of a launch of ndp + rem s workgroups (more exit).
template <bool GATE_UP, bool DIRECT>
__device__ __forceinline__ void wide_gemm(const GemmKArgs &p, int G, bf16_t *smem) {
  const WideSplit w = wide_split(p, G);
  const int KT = p.kc / kWideBK;
  const int b = blockIdx.x;
  TileId t;
  int k0 = 0, k1 = KT;
  float *part = nullptr;
  if (b < w.ndp) {
    wide_tile_at(p, xcd_remap(b, w.ndp), t);
  } else {
    const int j = b - w.ndp, n = w.rem * w.s;
    if (j >= n) return;
    const int lj = xcd_remap(j, n), c = lj / w.rem, r = lj % w.rem;
    wide_tile_at(p, w.ndp + r, t);
    k0 = c * KT / w.s;
    k1 = (c + 1) * KT / w.s;
    part = p.P + (size_t)(r * w.s + c) * kWideTileElems;
  }
  const int row0 = p.offsets[t.g] + t.mt * kWide;
  f32x16 acc[kWideTM][kWideTN];
  // the wave's 32-row blocks that hold rows of the group (wave-uniform)
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // partial tile: row-major, 256 (tail: 512) columns
#define EXF_W_STORE(DBL_)                                                                      \
  do {                                                                                         \
    if (part)                                                                                  \
      wide_store_f32<DBL_>(part, (DBL_ ? 2 : 1) * kWideBN, valid, [](int) { return 1.f; }, acc, smem); \
    else if (!GATE_UP && !DIRECT && p.Yh)                                                      \
      wide_store_lds<DBL_>(p, t, row0, valid, acc, smem);                                      \
    else if (!GATE_UP && !DIRECT)                                                              \
      wide_store_f32<DBL_>(p.Y + (long long)row0 * p.d + t.nt * kWideBN, p.d, valid,           \
                           [&](int ml) { return p.row_w[row0 + ml]; }, acc, smem);             \
    else                                                                                       \
      wide_store<GATE_UP, DBL_>(p, t, row0, valid, acc);                                       \
  } while (0)
#define EXF_W_MAIN(DBL_, TMV_) wide_tile_mma<GATE_UP, DBL_, TMV_>(p, t, row0, valid, k0, k1, smem, acc)
  // the 32-row blocks 64 i + 32 wm of 128 rows, `rows` of which hold rows of the group
  auto live = [&](int rows) { return max(0, min(2, (rows - 32 * (wave >> 2) + 63) >> 6)); };
  if (__builtin_amdgcn_readfirstlane(t.dbl)) {
    const int valid = min(kWide / 2, p.offsets[t.g + 1] - row0);
    switch (live(valid)) {
      case 2: EXF_W_MAIN(true, 2); break;
      case 1: EXF_W_MAIN(true, 1); break;
      default: EXF_W_MAIN(true, 0); break;
    }
    EXF_W_STORE(true);
  } else {
    const int valid = min(kWide, p.offsets[t.g + 1] - row0);  // more than 128
    switch (2 + live(valid - 128)) {
      case 4: EXF_W_MAIN(false, 4); break;
      case 3: EXF_W_MAIN(false, 3); break;
      default: EXF_W_MAIN(false, 2); break;
    }
    EXF_W_STORE(false);
  }
#undef EXF_W_MAIN
#undef EXF_W_STORE
}


__global__ __launch_bounds__(64 * kWideWaves, 1) void expert_gate_up_wide(const GemmKArgs p, int G) {
  __shared__ __attribute__((aligned(1024))) bf16_t smem[kWideSmemElems];
  wide_gemm<true, false>(p, G, smem);
}

template <bool DIRECT>
__global__ __launch_bounds__(64 * kWideWaves, 1) void expert_down_wide(const GemmKArgs p, int G) {
  __shared__ __attribute__((aligned(1024))) bf16_t smem[kWideSmemElems];
  wide_gemm<false, DIRECT>(p, G, smem);
}

// Block (r, c): remainder tile r, tile rows 16 c .. 16 c + 15, sixteen threads
// a row.  The partial tiles are row-major, 256 (tail tile: 512) columns a row.
// Gate/up: H column 128 nt + col from the gate column and the up column 128
// further; down: the output columns scaled by the row's routing weight.
template <bool GATE_UP, bool DIRECT>
__global__ __launch_bounds__(256) void expert_wide_fixup(const GemmKArgs p, int G) {
  const WideSplit w = wide_split(p, G);
  const int r = blockIdx.x;
  if (r >= w.rem) return;
  TileId t;
  wide_tile_at(p, w.ndp + r, t);
  const int bm = t.dbl ? kWide / 2 : kWide, bn = t.dbl ? 2 * kWideBN : kWideBN;
  const int row0 = p.offsets[t.g] + t.mt * kWide;
  const int valid = min(bm, p.offsets[t.g + 1] - row0);
  const int ml = blockIdx.y * 16 + (threadIdx.x >> 4);
  if (ml >= valid) return;
  const int row = row0 + ml;
  const float *P0 = p.P + (size_t)r * w.s * kWideTileElems + (size_t)ml * bn;
  // all s partials of a column group are loaded before the in-order sum (the
  // loads do not wait on each other)
  auto sum4 = [&](int col) {
    float4 q[kWideMaxSplit];
#pragma unroll
    for (int k = 0; k < kWideMaxSplit; ++k)
      if (k < w.s) q[k] = *reinterpret_cast<const float4 *>(P0 + (size_t)k * kWideTileElems + col);
    float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int k = 0; k < kWideMaxSplit; ++k)
      if (k < w.s) {
        v.x += q[k].x;
        v.y += q[k].y;
        v.z += q[k].z;
        v.w += q[k].w;
      }
    return v;
  };
  if (GATE_UP) {
    for (int q = 0; q < bn / 128; ++q) {
      const int col = q * 64 + (threadIdx.x & 15) * 4;
      // H column col of the tile: gate column col % 128 of n-tile col / 128, up 128 further
      const int pc = (col >> 7) * kWideBN + (col & 127);
      const float4 g = sum4(pc), u = sum4(pc + 128);
      const float h[4] = {silu(g.x) * u.x, silu(g.y) * u.y, silu(g.z) * u.z, silu(g.w) * u.w};
      bf16_t *dst = p.H + (long long)row * p.inter + t.nt * (kWideBN / 2) + col;
#pragma unroll
      for (int e = 0; e < 4; ++e) dst[e] = f32_to_bf16(h[e]);
    }
  } else {
    const float rw = p.Yh && !DIRECT ? 1.f : p.row_w[row];
    for (int q = 0; q < bn / 64; ++q) {
      const int col = q * 64 + (threadIdx.x & 15) * 4;
      const float4 a = sum4(col);
      const float v[4] = {a.x * rw, a.y * rw, a.z * rw, a.w * rw};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int n = t.nt * kWideBN + col + e;
        if (DIRECT)
          __builtin_nontemporal_store(f32_to_bf16(v[e]), &p.y[(long long)p.row_token[row] * p.d + n]);
        else if (p.Yh)
          p.Yh[(long long)row * p.d + n] = f32_to_bf16(v[e]);
        else
          p.Y[(long long)row * p.d + n] = v[e];
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Skinny tile for decode (few rows per retained expert): 32 RB rows x 64 output
// columns (gate/up: 32 gate + 32 up columns), BK = 128 per stage (256 contiguous
// bytes of every weight row per load step), and the four waves split each
// stage's reduction (wave w takes k16 steps w and w + 4) instead of the tile, so
// the weights stream through many small workgroups (three per CU by LDS for RB
// = 1, two for RB = 2).  The four partial tiles are added in wave order through
// LDS at the end.  A weight row that skips LDS (each wave loading its own MFMA
// fragments, 64-byte pieces of 16 rows) streams 25-35% slower.
// ---------------------------------------------------------------------------
constexpr int kSkN = 64, kSkK = 128;

// LDS element offset of 16-byte chunk q of row r in a 256-byte row (16 chunks):
// q XOR (r mod 16) spreads one chunk column of 16 consecutive rows over all banks.
__device__ __forceinline__ int swz16(int r, int q) { return (r * 16 + (q ^ (r & 15))) * 8; }

template <int RB, bool GATE_UP, bool DIRECT>
__global__ __launch_bounds__(256, RB == 1 ? 3 : 2) void expert_gemm_skinny(const GemmKArgs p) {
  constexpr int kSkM = 32 * RB, PA = kSkM * 16 / 256, PB = kSkN * 16 / 256;  // 16-byte chunks per thread per stage
  constexpr int STAGE = (kSkM + kSkN) * kSkK;                  // elements per LDS stage
  __shared__ __attribute__((aligned(16))) bf16_t smem[2 * STAGE];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;

  TileId t;
  if (!decode_tile(p, blockIdx.x, t)) return;
  const int row0 = p.offsets[t.g] + t.mt * kSkM;
  const int valid = min(kSkM, p.offsets[t.g + 1] - row0);
  const bf16_t *Wg = (t.g < p.n_experts) ? p.W + (long long)t.g * p.w_stride : p.Ws;

  // chunk c = i * 256 + tid: row c / 16, 16-byte column c % 16
  const bf16_t *a_src[PA];
  const bf16_t *b_src[PB];
#pragma unroll
  for (int i = 0; i < PA; ++i) {
    const int c = i * 256 + tid, r = c >> 4;
    const int rr = row0 + (r < valid ? r : 0);
    const long long arow = GATE_UP ? (long long)p.row_token[rr] : (long long)rr;
    a_src[i] = p.A + arow * p.lda + (long long)t.ks * p.kc + (c & 15) * 8;
  }
#pragma unroll
  for (int i = 0; i < PB; ++i) {
    const int c = i * 256 + tid, r = c >> 4;
    int wrow;
    if (GATE_UP)
      wrow = (r < kSkN / 2) ? t.nt * (kSkN / 2) + r : p.inter + t.nt * (kSkN / 2) + (r - kSkN / 2);
    else
      wrow = t.nt * kSkN + r;
    b_src[i] = Wg + (long long)wrow * p.ldw + (long long)t.ks * p.kc + (c & 15) * 8;
  }

  f32x16 acc[RB][2];
#pragma unroll
  for (int i = 0; i < RB; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
  const bool two = RB == 2 && __builtin_amdgcn_readfirstlane(valid) > 32;  // the second row block holds rows

  // stage KT_ (past the end: the last one again, into a buffer that is not read)
#define EXF_SK_GLOAD(RA_, RB_, KT_)                                                         \
  do {                                                                                      \
    const int k_ = min((KT_) * kSkK, k_last);                                               \
    _Pragma("unroll") for (int i_ = 0; i_ < PA; ++i_) RA_[i_] =                             \
        *reinterpret_cast<const u32x4 *>(a_src[i_] + k_);                                   \
    _Pragma("unroll") for (int i_ = 0; i_ < PB; ++i_) RB_[i_] = load_w16<ONCE>(b_src[i_] + k_); \
  } while (0)
#define EXF_SK_LSTORE(RA, RB, BUF)                                                          \
  do {                                                                                      \
    bf16_t *As_ = smem + (BUF) * STAGE;                                                     \
    bf16_t *Bs_ = As_ + kSkM * kSkK;                                                        \
    _Pragma("unroll") for (int i_ = 0; i_ < PA; ++i_) {                                     \
      const int c_ = i_ * 256 + tid;                                                        \
      *reinterpret_cast<u32x4 *>(&As_[swz16(c_ >> 4, c_ & 15)]) = RA[i_];                   \
    }                                                                                       \
    _Pragma("unroll") for (int i_ = 0; i_ < PB; ++i_) {                                     \
      const int c_ = i_ * 256 + tid;                                                        \
      *reinterpret_cast<u32x4 *>(&Bs_[swz16(c_ >> 4, c_ & 15)]) = RB[i_];                   \
    }                                                                                       \
  } while (0)
  // wave w: k16 steps w and w + 4 of the stage; lane l reads row l % 32, 8 k at (l / 32) * 8
#define EXF_SK_COMPUTE(BUF, KT_)                                                            \
  do {                                                                                      \
    const bf16_t *As_ = smem + (BUF) * STAGE;                                               \
    const bf16_t *Bs_ = As_ + kSkM * kSkK;                                                  \
    _Pragma("unroll") for (int h_ = 0; h_ < 2; ++h_) {                                      \
      if (h_ == 0 && half && (KT_) == KT - 1) continue;                                     \
      const int ch_ = (wave + 4 * h_) * 2 + (lane >> 5);                                    \
      const bf16x8 a_ = *reinterpret_cast<const bf16x8 *>(&As_[swz16(lane & 31, ch_)]);     \
      const bf16x8 b0_ = *reinterpret_cast<const bf16x8 *>(&Bs_[swz16(lane & 31, ch_)]);    \
      const bf16x8 b1_ = *reinterpret_cast<const bf16x8 *>(&Bs_[swz16(32 + (lane & 31), ch_)]); \
      acc[0][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a_, b0_, acc[0][0], 0, 0, 0);     \
      acc[0][1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a_, b1_, acc[0][1], 0, 0, 0);     \
      if (two) {                                                                            \
        const bf16x8 c_ = *reinterpret_cast<const bf16x8 *>(&As_[swz16(32 + (lane & 31), ch_)]); \
        acc[RB - 1][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(c_, b0_, acc[RB - 1][0], 0, 0, 0); \
        acc[RB - 1][1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(c_, b1_, acc[RB - 1][1], 0, 0, 0); \
      }                                                                                     \
    }                                                                                       \
  } while (0)

  // Two register sets: the loads of stage kt + 2 fly during the MFMAs of stage kt.
  // The last stage always ends with the range; when only 64 of its columns are
  // new, the k16 steps of its lower half are not taken again.
  const int KT = (p.kc + kSkK - 1) / kSkK, k_last = p.kc - kSkK;
  const bool half = (p.kc & (kSkK - 1)) != 0;
  auto main_loop = [&](auto once) __attribute__((always_inline)) {
    constexpr bool ONCE = decltype(once)::value;
    mark_loads<ONCE>();
    u32x4 ra0[PA], rb0[PB], ra1[PA], rb1[PB];
    EXF_SK_GLOAD(ra0, rb0, 0);
    EXF_SK_LSTORE(ra0, rb0, 0);
    EXF_SK_GLOAD(ra1, rb1, 1);
    __syncthreads();
    int kt = 0;
    for (; kt + 2 <= KT; kt += 2) {
      EXF_SK_GLOAD(ra0, rb0, kt + 2);
      EXF_SK_COMPUTE(0, kt);
      EXF_SK_LSTORE(ra1, rb1, 1);
      __syncthreads();
      EXF_SK_GLOAD(ra1, rb1, kt + 3);
      EXF_SK_COMPUTE(1, kt + 1);
      EXF_SK_LSTORE(ra0, rb0, 0);
      __syncthreads();
    }
    if (kt < KT) EXF_SK_COMPUTE(0, kt);
  };
  if (__builtin_amdgcn_readfirstlane(t.alone))
    main_loop(std::true_type{});
  else
    main_loop(std::false_type{});
#undef EXF_SK_GLOAD
#undef EXF_SK_LSTORE
#undef EXF_SK_COMPUTE

  // Partial tiles of the four waves, added in wave order (LDS reused).
  float *red = reinterpret_cast<float *>(smem);  // [4][2][16][64] floats = 32 KB
#pragma unroll
  for (int i = 0; i < RB; ++i) {
    if (i > 0 && !two) break;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) red[((wave * 2 + j) * 16 + r) * 64 + lane] = acc[i][j][r];
    __syncthreads();
    // wave w finishes accumulator registers r in [4 w, 4 w + 4) of both column halves:
    // rows (r / 4) * 8 + (lane / 32) * 4 + r % 4 of the 32x32 MFMA layout
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int r = wave * 4 + q;
      float v[2];
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        v[j] = red[((0 * 2 + j) * 16 + r) * 64 + lane];
#pragma unroll
        for (int w = 1; w < 4; ++w) v[j] += red[((w * 2 + j) * 16 + r) * 64 + lane];
      }
      const int ml = i * 32 + (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3);
      if (ml < valid) {
        const int row = row0 + ml;
        if (GATE_UP) {
          const int n = t.nt * (kSkN / 2) + (lane & 31);
          p.H[(long long)row * p.inter + n] = f32_to_bf16(silu(v[0]) * v[1]);
        } else {
          const float w = p.row_w[row];
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            const int n = t.nt * kSkN + j * 32 + (lane & 31);
            if (DIRECT)
              p.y[(long long)p.row_token[row] * p.d + n] = f32_to_bf16(v[j] * w);
            else if (p.Yh)
              p.Yh[(long long)row * p.d + n] = f32_to_bf16(v[j]);
            else
              p.Y[((long long)t.ks * p.rows + row) * p.d + n] = v[j] * w;
          }
        }
      }
    }
  }
}

template <bool GATE_UP, bool DIRECT>
static void launch_skinny(const GemmKArgs &p, const GemmPlan &pl, hipStream_t s) {
  if (pl.bm == 32) expert_gemm_skinny<1, GATE_UP, DIRECT><<<pl.grid, 256, 0, s>>>(p);
  else expert_gemm_skinny<2, GATE_UP, DIRECT><<<pl.grid, 256, 0, s>>>(p);
}

// ---------------------------------------------------------------------------
// float32 layers: 16x16x4 float32 MFMA on tiles of 16 TM rows x 16 TN output
// columns (gate/up: as many gate and up columns).  Small layers are bound by
// the latency of the weight stream, so the four waves of a workgroup split the
// reduction and every operand goes from global memory straight into MFMA
// registers: lane l holds four consecutive columns 4 (l / 16) of row l % 16 and
// MFMA step e takes element e of every lane (any assignment of columns to
// steps is a valid reduction order), so rows load in 64-byte pieces, a batch of
// kF32Batch pieces in flight.  The partial tiles are added in wave order
// through LDS.  One thread an output, walking a weight row alone, read each
// weight row 4 bytes at a time: 64 tokens, 8 experts, d 256, I 512:
// gate/up 63 -> 6.9 us, down 65 -> 5.7 us.
// ---------------------------------------------------------------------------
constexpr int kF32Batch = 4;

template <int TM, int TN, bool GATE_UP>
__global__ __launch_bounds__(256) void expert_gemm_f32(const GemmKArgs p) {
  constexpr int NB = GATE_UP ? 2 : 1, TILES = TM * TN * NB;
  __shared__ float red[4][TILES][256];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  TileId t;
  if (!decode_tile(p, blockIdx.x, t)) return;
  const int row0 = p.offsets[t.g] + t.mt * 16 * TM;
  const int valid = min(16 * TM, p.offsets[t.g + 1] - row0);
  const float *Wg = (t.g < p.n_experts)
                        ? reinterpret_cast<const float *>(p.W) + (long long)t.g * p.w_stride
                        : reinterpret_cast<const float *>(p.Ws);
  const int kq = (lane >> 4) * 4;
  const float *a_src[TM], *b_src[NB][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int r = i * 16 + (lane & 15);
    const int rr = row0 + (r < valid ? r : 0);  // rows past the group's end are never stored
    const long long arow = GATE_UP ? (long long)p.row_token[rr] : (long long)rr;
    a_src[i] = reinterpret_cast<const float *>(p.A) + arow * p.lda + kq;
  }
#pragma unroll
  for (int b = 0; b < NB; ++b)
#pragma unroll
    for (int j = 0; j < TN; ++j)
      b_src[b][j] = Wg + (long long)(b * p.inter + (t.nt * TN + j) * 16 + (lane & 15)) * p.ldw + kq;
  f32x4 acc[TM][TN][NB];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int b = 0; b < NB; ++b) acc[i][j][b] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int span = p.kc / 4, k1 = (wave + 1) * span;  // a multiple of 16 columns a wave
  constexpr int U = TILES >= 8 ? 2 : kF32Batch;
  for (int k0 = wave * span; k0 < k1; k0 += 16 * U) {
    f32x4 va[U][TM], vb[U][TN][NB];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k = k0 + 16 * u;
      if (k < k1) {
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int b = 0; b < NB; ++b) vb[u][j][b] = *reinterpret_cast<const f32x4 *>(b_src[b][j] + k);
#pragma unroll
        for (int i = 0; i < TM; ++i) va[u][i] = *reinterpret_cast<const f32x4 *>(a_src[i] + k);
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (k0 + 16 * u < k1) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
              for (int b = 0; b < NB; ++b)
                acc[i][j][b] =
                    __builtin_amdgcn_mfma_f32_16x16x4f32(va[u][i][e], vb[u][j][b][e], acc[i][j][b], 0, 0, 0);
      }
  }
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int r = 0; r < 4; ++r) red[wave][(i * TN + j) * NB + b][r * 64 + lane] = acc[i][j][b][r];
  __syncthreads();
  // thread (r, l) finishes register r of lane l of every tile: row 4 (l / 16) + r, column l % 16
  const int ml0 = (lane >> 4) * 4 + wave, col = lane & 15, x = threadIdx.x;
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int ml = i * 16 + ml0;
    if (ml >= valid) continue;
    const int row = row0 + ml;
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      float v[NB];
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        const int q = (i * TN + j) * NB + b;
        v[b] = ((red[0][q][x] + red[1][q][x]) + red[2][q][x]) + red[3][q][x];
      }
      const int n = (t.nt * TN + j) * 16 + col;
      if constexpr (GATE_UP) {
        reinterpret_cast<float *>(p.H)[(long long)row * p.inter + n] = silu(v[0]) * v[1];
      } else {
        const float o = v[0] * p.row_w[row];
        if (p.y)
          reinterpret_cast<float *>(p.y)[(long long)p.row_token[row] * p.d + n] = o;
        else
          p.Y[(long long)row * p.d + n] = o;
      }
    }
  }
}

template <bool GATE_UP>
static void launch_gemm_f32(const GemmKArgs &p, const GemmPlan &pl, hipStream_t s) {
  if (pl.bm == 16) expert_gemm_f32<1, 1, GATE_UP><<<pl.grid, 256, 0, s>>>(p);
  else if (pl.bm == 32) expert_gemm_f32<2, 1, GATE_UP><<<pl.grid, 256, 0, s>>>(p);
  else expert_gemm_f32<4, 2, GATE_UP><<<pl.grid, 256, 0, s>>>(p);
}

// ---------------------------------------------------------------------------
// Planning and launch.
// ---------------------------------------------------------------------------
static int largest_divisor_at_most(int n, int cap) {
  for (int v = cap < n ? cap : n; v > 1; --v)
    if (n % v == 0) return v;
  return 1;
}

void plan_expert_gemms(int dtype, int rows, int groups, int active_groups, int d, int inter,
                       int cu_count, GemmPlan *gu, GemmPlan *dn) {
  // The plan depends on the problem only (rows, groups, sizes), never on the
  // phase, so equal problems get equal plans.
  const int active = active_groups < 1 ? 1 : active_groups;
  if (dtype != EXFOLD_BF16) {
    // tiles as high as the rows of a busy expert on average, 64 at most (then
    // 32 output columns, so a weight row feeds as many MFMAs as a token row)
    const int bm = rows <= 16 * active ? 16 : rows <= 32 * active ? 32 : 64, cols = bm == 64 ? 32 : 16;
    const int mt = rows / bm + groups;  // >= sum of ceil(rows_g / bm)
    *gu = GemmPlan{bm, 2 * cols, 1, mt * (inter / cols), kGemmSimt};
    *dn = GemmPlan{bm, cols, 1, mt * (d / cols), kGemmSimt};
    return;
  }
  // Few rows per retained expert (decode): skinny tiles stream the weights through
  // many small workgroups; otherwise 128-column tiles.  The gate/up projection
  // takes 128-row tiles once the experts hold more than about 24 rows each, even
  // where those tiles do not cover the CUs (GLM-shaped, 256 tokens on a static
  // pool of 64, 32 rows each: 255 against 273 us on skinny tiles).  64-row skinny
  // tiles from 12 rows on average, where groups of more than 32 rows appear and
  // 32-row tiles would read their weights twice (the same batch's down: 174 ->
  // 162 us; 1237 tokens, K' = 3: 354 -> 338); below, three workgroups of 32-row
  // tiles a CU (Qwen3-shaped, one token: 54.9 against 56.4 us).  d is a multiple
  // of 128; a reduction shorter than one skinny stage (I = 64) takes the tile.
  const bool gu_skinny = rows <= 24 * active;
  // 64-row skinny tiles only where there are more than four tiles a CU: two of
  // them fit a CU and three of 32 rows, so a launch of few tiles takes a second
  // round as soon as some experts hold more than 64 rows (32 experts, d 1024, I 512,
  // 180 tokens x 4, one expert with 99 rows: 46.0 against 40.7 us a layer; with every
  // expert below 34 rows 37.8 against 39.9).
  const auto skinny_rows = [&](int tiles) {
    return rows <= 12 * active || (rows <= 24 * active && tiles <= 4 * cu_count) ? 32 : 64;
  };
  // Many rows per retained expert (prefill, at least 128 on average): wide
  // tiles.  With the 128-row tail tiles a skewed load pays at most half a tile
  // per group: the Qwen3-shaped prefill (8192 tokens, K' = 4, 98 of 128 experts
  // busy, 334 rows on average, 3974 at most) runs 19% faster than on 128x128.
  // Fewer than a quarter round of wide tiles (then split four ways or more)
  // loses to 128x128 tiles (Qwen3-shaped decode, 256 tokens on a pool of 16,
  // 48 wide tiles: 130.8 against 103.8 us per layer).
  const bool gu_wide = !gu_skinny && inter % kWideBN == 0 && d % 128 == 0 && 2 * rows >= kWide * active &&
                       (long long)(rows / 128) * (inter / kWideBN) * 4 >= cu_count;
  // The down projection keeps skinny tiles up to about 48 rows per expert, or to
  // 20 where there are more than two 128-column tiles a CU: then 64-row tiles of
  // 128 columns (three workgroups a CU) stream as well and fetch the rows of H
  // half as often (GLM-shaped, 256 tokens on a static pool of 64, 32 rows each:
  // 149 against 163 us; 700 Qwen3-shaped prefill tokens, K' = 4: 61 against 71;
  // at 18 rows, 64 tokens on a pool of 32, 75 against 73).  64-row tiles up to 80
  // rows (512 Qwen3-shaped tokens on a pool of 64: 51 us against 66 on skinny and
  // 59 on 128-row tiles, whose second half is padding there; gate/up is not
  // faster on them: 98 against 92 us).
  const bool dn_skinny = inter >= kSkK && rows <= (active * (d / 128) > 2 * cu_count ? 20 : 48) * active;
  const int tile_m = rows <= 80 * active ? 64 : 128;
  if (gu_skinny) {
    const int sk_m = skinny_rows(active * (inter / (kSkN / 2)));
    *gu = GemmPlan{sk_m, kSkN, 1, 0, kGemmSkinny};
    gu->grid = (rows / sk_m + groups) * (inter / (kSkN / 2));  // >= sum of ceil(rows_g / bm) tiles
  } else if (gu_wide) {
    // tile list in 128-row units, one tile per unit and pair of 128-column
    // n-tiles; whole rounds plus the split remainder: at most that + one round
    *gu = GemmPlan{kWide / 2, kWideBN, 1, 0, kGemmWide, cu_count};
    gu->grid = (rows / 128 + groups) * (inter / kWideBN) + cu_count;
  } else {
    *gu = GemmPlan{128, 128, 1, 0, kGemmTile};
    gu->grid = (rows / 128 + groups) * (inter / 64);
  }
  // Down projection on the wide tile where the gate/up projection takes it,
  // also when its tiles do not fill one round (they then all run split along
  // the reduction: Qwen3-shaped decode, 512 tokens on a pool of 32, 150.7
  // against 160.0 us per layer with 128x128 tiles).
  if (!dn_skinny && gu_wide && d % (2 * kWideBN) == 0) {
    *dn = GemmPlan{kWide / 2, kWideBN, 1, 0, kGemmWide, cu_count};
    dn->grid = (rows / 128 + groups) * (d / (2 * kWideBN)) + cu_count;
    return;
  }
  // Few expected tiles: split the down projection's reduction so the workgroups
  // still cover every CU.  Partial sums land in separate buffers and are added
  // in a fixed order by the combine.  Only long reductions are split: every
  // range keeps at least kMinSplitStages stages (an intermediate size of 768
  // split three ways ran 3 us slower per decode layer than unsplit, a 14336
  // one split in two 20 us faster).
  // The split is counted on 32 x 64 tiles, three a CU, where skinny tiles take an
  // even multiple of 64 columns, and on 128 x 128 tiles, two a CU, otherwise,
  // whatever the tile that runs: with one range the rows travel as bf16, with more
  // as float32 partials, so a count on the smaller tiles, which asks for fewer
  // ranges, would take precision from odd multiples of 64 (d 512, I 1728, 1598 rows
  // on 34 experts: three ranges).
  const int bn = dn_skinny ? kSkN : 128;
  const bool fine = dn_skinny && inter % 128 == 0;
  const int split_m = fine ? 32 : 128, split_n = fine ? kSkN : 128, kk = fine ? kSkK : kBK, fill = fine ? 3 : 2;
  *dn = GemmPlan{0, bn, 1, 0, dn_skinny ? kGemmSkinny : kGemmTile};
  const int mt_expect = (rows + split_m - 1) / split_m > active ? (rows + split_m - 1) / split_m : active;
  const int dn_tiles = mt_expect * (d / split_n);
  constexpr int kMinSplitStages = 8;
  const int max_split = (inter / kk) / kMinSplitStages;
  if (dn_tiles < fill * cu_count && max_split >= 2) {
    const int want = (fill * cu_count + dn_tiles - 1) / dn_tiles;
    const int cap = want < max_split ? want : max_split;
    dn->ksplit = largest_divisor_at_most(inter / kk, cap > 8 ? 8 : cap);
  }
  dn->bm = dn_skinny ? skinny_rows(active * (d / kSkN) * dn->ksplit) : tile_m;
  dn->grid = (rows / dn->bm + groups) * (d / bn) * dn->ksplit;
}

hipError_t launch_expert_gemms(const ExpertArgs &a, const GemmPlan &gu, const GemmPlan &dn,
                               hipStream_t s, hipEvent_t ev_mid) {
  if (a.rows <= 0) return hipSuccess;
  GemmKArgs ga{};
  ga.A = static_cast<const bf16_t *>(a.x);
  ga.lda = a.d;
  ga.row_token = a.row_token;
  ga.offsets = a.offsets;
  ga.tile_start = a.tile_start_gu;
  ga.groups = a.groups;
  ga.n_experts = a.n_experts;
  ga.n_tiles = a.inter / (gu.bn / 2);
  ga.ksplit = 1;
  ga.kc = a.d;
  ga.rows = a.rows;
  ga.W = static_cast<const bf16_t *>(a.w_gate_up);
  ga.Ws = static_cast<const bf16_t *>(a.ws_gate_up);
  ga.w_stride = 2LL * a.inter * a.d;
  ga.ldw = a.d;
  ga.inter = a.inter;
  ga.d = a.d;
  ga.H = static_cast<bf16_t *>(a.H);

  GemmKArgs da{};
  da.A = static_cast<const bf16_t *>(a.H);
  da.lda = a.inter;
  da.row_token = a.row_token;
  da.offsets = a.offsets;
  da.tile_start = a.tile_start_dn;
  da.groups = a.groups;
  da.n_experts = a.n_experts;
  da.n_tiles = a.d / dn.bn;
  da.ksplit = dn.ksplit;
  da.kc = a.inter / dn.ksplit;
  da.rows = a.rows;
  da.W = static_cast<const bf16_t *>(a.w_down);
  da.Ws = static_cast<const bf16_t *>(a.ws_down);
  da.w_stride = (long long)a.d * a.inter;
  da.ldw = a.inter;
  da.inter = a.inter;
  da.d = a.d;
  da.Y = a.y_bf16 ? nullptr : a.Y;
  da.Yh = a.y_bf16 ? reinterpret_cast<bf16_t *>(a.Y) : nullptr;
  da.y = static_cast<bf16_t *>(a.y);
  da.row_w = a.row_w;

  if (a.dtype != EXFOLD_BF16) {
    if (!a.direct) da.y = nullptr;
    launch_gemm_f32<true>(ga, gu, s);
    if (ev_mid) (void)hipEventRecord(ev_mid, s);
    launch_gemm_f32<false>(da, dn, s);
    return hipGetLastError();
  }
  if (gu.grid > 0) {
    if (gu.kind == kGemmSkinny) {
      launch_skinny<true, false>(ga, gu, s);
    } else if (gu.kind == kGemmWide) {
      ga.P = a.wide_part;
      expert_gate_up_wide<<<gu.grid, 64 * kWideWaves, 0, s>>>(ga, gu.wgs);
      expert_wide_fixup<true, false><<<dim3(gu.wgs / 2, kWide / 16), 256, 0, s>>>(ga, gu.wgs);
    } else {
      expert_gemm_tile<128, 128, true, false><<<gu.grid, 256, 0, s>>>(ga);
    }
  }
  if (ev_mid) (void)hipEventRecord(ev_mid, s);
  if (dn.grid > 0) {
    if (dn.kind == kGemmWide) {
      da.P = a.wide_part;
      const dim3 fg(dn.wgs / 2, kWide / 16);
      if (a.direct) {
        expert_down_wide<true><<<dn.grid, 64 * kWideWaves, 0, s>>>(da, dn.wgs);
        expert_wide_fixup<false, true><<<fg, 256, 0, s>>>(da, dn.wgs);
      } else {
        expert_down_wide<false><<<dn.grid, 64 * kWideWaves, 0, s>>>(da, dn.wgs);
        expert_wide_fixup<false, false><<<fg, 256, 0, s>>>(da, dn.wgs);
      }
    } else if (dn.kind == kGemmSkinny) {
      if (a.direct)
        launch_skinny<false, true>(da, dn, s);
      else
        launch_skinny<false, false>(da, dn, s);
    } else {
      if (dn.bm == 64 && a.direct)
        expert_gemm_tile<64, 128, false, true><<<dn.grid, 256, 0, s>>>(da);
      else if (dn.bm == 64)
        expert_gemm_tile<64, 128, false, false><<<dn.grid, 256, 0, s>>>(da);
      else if (a.direct)
        expert_gemm_tile<128, 128, false, true><<<dn.grid, 256, 0, s>>>(da);
      else
        expert_gemm_tile<128, 128, false, false><<<dn.grid, 256, 0, s>>>(da);
    }
  }
  return hipGetLastError();
}

int plain_gemm_splits(int M, int N, int K, int cu_count) {
  if (M <= 0 || N % 128 != 0 || K % kBK != 0) return 0;
  const int tiles = (M + 127) / 128 * (N / 128);
  int P = 1;
  // split the reduction until the tiles cover the CUs, every range at least
  // four stages of kBK
  while (tiles * P < cu_count && P < 8 && K % (2 * P * kBK) == 0 && K / (2 * P) >= 4 * kBK) P *= 2;
  return P;
}

hipError_t launch_plain_gemm_nt(const void *A, const void *W, int M, int N, int K, int P, float *part,
                                hipStream_t s) {
  GemmKArgs g{};
  g.A = static_cast<const bf16_t *>(A);
  g.lda = K;
  g.W = static_cast<const bf16_t *>(W);
  g.ldw = K;
  g.rows = M;
  g.d = N;
  g.n_tiles = N / 128;
  g.ksplit = P;
  g.kc = K / P;
  g.Y = part;
  // 64-row tiles: the splits are chosen on 128 rows, which leaves at most one
  // workgroup a CU (1237 tokens x 128 experts x 4096: 13.9 -> 9.9 us; 4096 x 128 x
  // 2048: 14.4 -> 12.0)
  const int grid = (M + 63) / 64 * g.n_tiles * P;
  expert_gemm_tile<64, 128, false, false, true><<<grid, 256, 0, s>>>(g);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Weighted combine: y_i = sum_k Y[row(i,k)] (+ shared row), in slot order;
// float32 accumulation, one rounding to the output dtype.
// ---------------------------------------------------------------------------
template <typename InT>
__device__ __forceinline__ float4 load4(const InT *p);
template <>
__device__ __forceinline__ float4 load4<float>(const float *p) {
  return *reinterpret_cast<const float4 *>(p);
}
template <>
__device__ __forceinline__ float4 load4<bf16_t>(const bf16_t *p) {
  const uint2 u = *reinterpret_cast<const uint2 *>(p);
  return make_float4(__uint_as_float(u.x << 16), __uint_as_float(u.x & 0xffff0000u),
                     __uint_as_float(u.y << 16), __uint_as_float(u.y & 0xffff0000u));
}

template <typename InT, int C>
__device__ __forceinline__ void load_cols(const InT *p, float (&v)[C]) {
#pragma unroll
  for (int q = 0; q < C; q += 4) {
    const float4 f = load4<InT>(p + q);
    v[q] = f.x;
    v[q + 1] = f.y;
    v[q + 2] = f.z;
    v[q + 3] = f.w;
  }
}

template <typename InT, typename OutT, int C, bool PAIRS>
__global__ __launch_bounds__(256) void combine_kernel(const InT *__restrict__ Y, int ksplit,
                                                     int rows, const int32_t *__restrict__ slot_row,
                                                     const float *__restrict__ row_w,
                                                     int k_out, int d, int shared_base,
                                                     OutT *__restrict__ y) {
  // block (i, c): token i, columns [256 C c, 256 C (c + 1)), C per thread.  The
  // token's row indices are loaded first (one round trip), then the rows are
  // loaded four at a time and added in slot order, split partials in order.
  // bf16 rows arrive unscaled: each is multiplied by its routing weight here,
  // in fp32, so two routes of one token to the same expert share one rounded
  // row and their weights add exactly as in the unrounded sum.
  const int i = blockIdx.x;
  const int c = (blockIdx.y * 256 + threadIdx.x) * C;
  if (c >= d) return;
  const long long split = (long long)rows * d;
  const int nr = k_out + (shared_base >= 0 ? 1 : 0);
  int r[kMaxTopK + 1];
#pragma unroll
  for (int k = 0; k <= kMaxTopK; ++k)
    r[k] = (k < k_out) ? slot_row[(long long)i * k_out + k] : (k == k_out && shared_base >= 0) ? shared_base + i : 0;
  constexpr bool kScale = sizeof(InT) == 2;
  float rw[kMaxTopK + 1];
#pragma unroll
  for (int k = 0; k <= kMaxTopK; ++k) rw[k] = (kScale && k < nr) ? row_w[r[k]] : 1.f;
  float acc[C];
#pragma unroll
  for (int q = 0; q < C; ++q) acc[q] = 0.f;
  for (int sp = 0; sp < ksplit; sp += 2) {
    // splits sp and sp + 1 of four rows at a time, all loaded before the adds
    // (rows in slot order, the two splits in order); with one split this is
    // the whole sum in slot order
    const InT *base = Y + sp * split + c;
    const bool two = PAIRS && sp + 1 < ksplit;
#pragma unroll
    for (int k0 = 0; k0 <= kMaxTopK; k0 += 4) {
      if (k0 >= nr) break;
      float v[2][4][C];
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (k0 + u < nr) {
          load_cols<InT, C>(base + (long long)r[k0 + u] * d, v[0][u]);
          if (two) load_cols<InT, C>(base + split + (long long)r[k0 + u] * d, v[1][u]);
        }
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (k0 + u < nr && (h == 0 || two)) {
#pragma unroll
            for (int q = 0; q < C; ++q) acc[q] = kScale ? fmaf(rw[k0 + u], v[h][u][q], acc[q]) : acc[q] + v[h][u][q];
          }
    }
  }
  OutT *o = y + (long long)i * d + c;
#pragma unroll
  for (int q = 0; q < C; q += 4) {
    if constexpr (sizeof(OutT) == 2)
      store4_bf16(reinterpret_cast<bf16_t *>(o) + q, acc[q], acc[q + 1], acc[q + 2], acc[q + 3]);
    else
      *reinterpret_cast<float4 *>(o + q) = make_float4(acc[q], acc[q + 1], acc[q + 2], acc[q + 3]);
  }
}

// The same sums for more rows a token than the registers of combine_kernel hold (only
// exfold_moe_execute takes more than 16 routes): the row indices are read as the rows are.
template <typename InT, typename OutT>
__global__ __launch_bounds__(256) void combine_many_kernel(const InT *__restrict__ Y, int ksplit, int rows,
                                                          const int32_t *__restrict__ slot_row,
                                                          const float *__restrict__ row_w, int k_out, int d,
                                                          int shared_base, OutT *__restrict__ y) {
  const int i = blockIdx.x, c = (blockIdx.y * 256 + threadIdx.x) * 4;
  if (c >= d) return;
  const int nr = k_out + (shared_base >= 0 ? 1 : 0);
  constexpr bool kScale = sizeof(InT) == 2;
  float acc[4] = {0.f, 0.f, 0.f, 0.f};
  for (int sp = 0; sp < ksplit; ++sp) {
    const InT *base = Y + (long long)sp * rows * d + c;
#pragma unroll 4
    for (int k = 0; k < nr; ++k) {
      const int r = k < k_out ? slot_row[(long long)i * k_out + k] : shared_base + i;
      const float w = kScale ? row_w[r] : 1.f;
      float v[4];
      load_cols<InT, 4>(base + (long long)r * d, v);
#pragma unroll
      for (int q = 0; q < 4; ++q) acc[q] = kScale ? fmaf(w, v[q], acc[q]) : acc[q] + v[q];
    }
  }
  OutT *o = y + (long long)i * d + c;
  if constexpr (sizeof(OutT) == 2)
    store4_bf16(reinterpret_cast<bf16_t *>(o), acc[0], acc[1], acc[2], acc[3]);
  else
    *reinterpret_cast<float4 *>(o) = make_float4(acc[0], acc[1], acc[2], acc[3]);
}

template <typename InT, typename OutT>
static void launch_combine_t(const InT *Y, int ksplit, int rows, const int32_t *slot_row, const float *row_w,
                             int T, int k_out, int d, int shared_base, OutT *y, hipStream_t s) {
  if (k_out + (shared_base >= 0 ? 1 : 0) > kMaxTopK + 1) {
    combine_many_kernel<InT, OutT><<<dim3(T, (d + 1023) / 1024), 256, 0, s>>>(Y, ksplit, rows, slot_row, row_w, k_out,
                                                                              d, shared_base, y);
    return;
  }
  // eight columns a thread once the grid covers the CUs a few times over; four below
  if ((long long)T * d >= 256LL * 256 * 8 * 4) {
    const dim3 grid(T, (d + 2047) / 2048);
    if (ksplit > 1)
      combine_kernel<InT, OutT, 8, true><<<grid, 256, 0, s>>>(Y, ksplit, rows, slot_row, row_w, k_out, d,
                                                                   shared_base, y);
    else
      combine_kernel<InT, OutT, 8, false><<<grid, 256, 0, s>>>(Y, ksplit, rows, slot_row, row_w, k_out, d,
                                                                   shared_base, y);
  } else {
    const dim3 grid(T, (d + 1023) / 1024);
    if (ksplit > 1)
      combine_kernel<InT, OutT, 4, true><<<grid, 256, 0, s>>>(Y, ksplit, rows, slot_row, row_w, k_out, d,
                                                                   shared_base, y);
    else
      combine_kernel<InT, OutT, 4, false><<<grid, 256, 0, s>>>(Y, ksplit, rows, slot_row, row_w, k_out, d,
                                                                   shared_base, y);
  }
}

hipError_t launch_combine(int dtype, const float *Y, bool y_bf16, int ksplit, int rows,
                          const int32_t *slot_row, const float *row_w, int T, int k_out, int d,
                          int shared_base, void *y, hipStream_t s) {
  if (T <= 0) return hipSuccess;
  if (dtype == EXFOLD_BF16 && y_bf16)
    launch_combine_t<bf16_t, bf16_t>(reinterpret_cast<const bf16_t *>(Y), ksplit, rows, slot_row, row_w, T, k_out,
                                     d, shared_base, static_cast<bf16_t *>(y), s);
  else if (dtype == EXFOLD_BF16)
    launch_combine_t<float, bf16_t>(Y, ksplit, rows, slot_row, nullptr, T, k_out, d, shared_base,
                                    static_cast<bf16_t *>(y), s);
  else
    launch_combine_t<float, float>(Y, ksplit, rows, slot_row, nullptr, T, k_out, d, shared_base,
                                   static_cast<float *>(y), s);
  return hipGetLastError();
}

}  // namespace exfold
