// Flash-attention forward for gfx950: Alg. 1 (standard safe softmax) and Alg. 3 (stabilised
// normaliser, Sec. 4) of arXiv 2510.04212, one work-group per (batch, head, 128-query block).
//
// Work split: 4 waves, each owning 32 query rows; key tiles of B_c = 64 rows of K and V are
// staged in LDS (double buffered) and shared by the 4 waves.  Per tile a wave computes
//     S^T[key][query] = K_j Q_i^T           (A = K_j from LDS, B = Q_i^T held in registers)
// so that one query row lives in lane r and lane r+32; row max / row sum / near-max count are
// in-register reductions plus one exchange with the partner lane.  P-bar^T in the accumulator
// layout is directly the B operand of
//     O^T[d][query] += V_j^T P-bar^T          (A = V_j^T via transposing LDS reads)
// which keeps the per-query rescale factor uniform over a lane's accumulator registers.
#include "common.hpp"

#include <atomic>
#include <type_traits>

namespace {

constexpr int kBr = 128;   // query rows per work-group
constexpr int kBc = 64;    // key rows per tile

// Optional outputs and switches of the forward (the experiments of Sec. 3.2 / 3.3.2 and the
// tie statistics of Sec. 3.3.2 / 4).  Only kernels instantiated with EXTRAS look at them (EXTRAS = 1; 2: with the
// P-bar V product in E4M3: one kernel for both products takes up to 67 registers more than either, d256 all 512.  us, both in one ->
// apart, with O_hp and counts: B4 H12 N1024 d64 causal 27.6 -> 26.6, B8 H12 44.4 -> 38.4, B2 H16 N2048 d128 full 120 -> 111,
// B2 H8 N2048 d256 causal 111 -> 89, B8 H12 N1024 d32 31.1 -> 30.1).
struct FwdExtras {
  float* O_hp;          // [B,H,N,d] float32: accumulator / l with no bf16 rounding, or null
  int* ones;            // [B,H,N]: number of keys whose rounded P-bar was exactly 1, or null
  int* fired;           // [B,H,N]: number of key tiles in which Alg. 3 moved the normaliser, or null
  int single_rounding;  // nonzero: O-bar is NOT rounded to bf16 before the division by l
  int guard;            // nonzero: Alg. 3's rule is not applied where it would move the normaliser
                        // by more than kGuardLimit (a labelled deviation from Sec. 4, see attn.h)
};

// Largest move of the normaliser the guarded form of Alg. 3 makes, in natural-log units of the
// alpha-scaled scores: the row maximum then still maps to exp(-60) ~ 9e-27, far above the point
// where the hardware exponential returns 0 (2^-126).
constexpr float kGuardLimit = 60.0f;
DEVI bool guard_allows(float r_m, float beta) {
  const float shift_by = r_m > 0.f ? (beta - 1.0f) * r_m : -r_m;
  return shift_by <= kGuardLimit;
}

// Eight float32 values -> eight E4M3 bytes (hardware conversion: round to nearest even).
DEVI long pack_e4m3(const float (&v)[8]) {
  int w0 = 0, w1 = 0;
  w0 = __builtin_amdgcn_cvt_pk_fp8_f32(v[0], v[1], w0, false);
  w0 = __builtin_amdgcn_cvt_pk_fp8_f32(v[2], v[3], w0, true);
  w1 = __builtin_amdgcn_cvt_pk_fp8_f32(v[4], v[5], w1, false);
  w1 = __builtin_amdgcn_cvt_pk_fp8_f32(v[6], v[7], w1, true);
  return (long)(((unsigned long long)(unsigned)w1 << 32) | (unsigned)w0);
}

// VARIANT: 0 = Alg. 1, 1 = Alg. 3 (repeated maximum looked for inside each key tile, as the algorithm is written), and
//   kWholeRow   the tile-size-independent form of Alg. 3 (the rule of Sec. 4 applied to the whole row, as in the paper's
//               untiled analysis), in two passes over the key tiles: scores only, whose two largest per row over ALL keys
//               decide the normaliser (a repeated maximum <=> the second largest is within eps of the largest), and the
//               forward with that fixed normaliser (no running maximum, no accumulator rescale).
// Both passes are one launch: a work-group's rows need nothing of another's.  As two launches, with the normaliser through memory,
// Q was fetched twice, the grid drained twice and short problems waited for the second launch.  Same bits; us, two launches -> one:
// B1 H1 N128 d64 causal 10.1 -> 7.3, B64 H8 N200 22.6 -> 17.7, B4 H12 N1024 26.4 -> 23.3, B32 H12 N512 full 54.5 -> 47.2,
// B1 H16 N768 d128 causal 27.2 -> 24.9, B4 H32 N4096 789 -> 778, B12 H16 N1408 d256 452 -> 407, B4 H16 N1999 d32 44.8 -> 41.6.
constexpr int kWholeRow = 2;

// Which kernels run as a software pipeline over tiles.  It needs 32 more registers for the next tile's scores: at
// D <= 64 that costs a wave per SIMD.  Measured, tile after tile -> pipeline (us): causal B2 H16 N2048 d96 46.7 -> 43.7,
// B8 H16 N512 d96 19.1 -> 18.3, B8 H16 N384 d128 17.4 -> 16.1, B2 H16 N512 d128 15.5 -> 14.6, B2 H32/8 N2048 d128
// 93.5 -> 91, but B16 H16 N200 d128 16.6 -> 17.6; d256 (with kPlacedReads) even, B4 H16 N4096 693 -> 683; not taken: B4 H32
// N4096 d64 342 -> 353, B8 H12 N1024 d64 27.4 -> 28.4, and without a mask B4 H16 N2048 d128 153 -> 205, B2 H16 N2000 d96
// 70 -> 75, B2 H8 N2048 d256 83 -> 143 (spills).
template <int D, bool CAUSAL> constexpr bool kPipelined = CAUSAL && D >= 96;

// Waves per SIMD the compiler has to make room for.  The row sums' selector and four-register result (add_rows) put some
// kernels one to four registers over the 96 that five waves allow (D = 32, causal) or the 128 of four (D = 64, causal);
// asked for the waves they fit without spilling, but for the whole-row rule at D = 32, causal, which spills two outside its tile loops.
// Measured, a wave less -> now (us): d32 B13 H32 N520 Alg. 1 37.0 -> 31.8, Alg. 3 41.7 -> 35.5, B4 H32 N4096 250 -> 244, B8 H12 N1024
// even, whole rows 192 heads N1000 37.0 -> 35.6, 48 heads N4096 106.6 -> 103.1, one tile (768 heads N64) 8.05 -> 8.30; d64 Alg. 1 B64 H8 N200 17.6 -> 15.7, B16 H12 N1999 144 -> 138,
// B8 H12 N1000 even, aligned Alg. 3 B64 H8 N256 18.8 -> 16.8, B4 H32 N4096 354 -> 350, B8 H12 N1024 even.  Not asked of
// the causal Alg. 3 kernel with bounds checks at d64, which would spill two: B16 H12 N1999 154 -> 150, but B8 H12 N1000 27.0 -> 28.3.
template <int D, bool CAUSAL, int VARIANT, bool RAGGED, int EXTRAS> constexpr int kFwdWaves =
    D == 32 && CAUSAL && EXTRAS == 0 ? 5 : D == 64 && CAUSAL && EXTRAS == 0 && (!RAGGED || VARIANT == 0) ? 4 : D <= 128 ? 2 : 1;

// Kernels whose LDS reads are put ahead of their products by hand (a fence per product) where tiles come one after the
// other.  The compiler gives the requested read-ahead up where registers are short: at D = 256 every product waited for
// its own reads, at D = 64 under the mask with bounds checks those of the scores did.  Same bits; us, left to the compiler -> placed:
// d256 B2 H8 N2000 full 104 -> 82, aligned N2048 95 -> 80, B3 H8 N1000 full 56 -> 45, whole-row rule B2 H8 N2048 causal 83 -> 62,
// optional outputs B2 H8 N2048 causal 110 -> 87; d64 causal B2 H8 N1999 Alg. 1 32.3 -> 30.7, Alg. 3 35.0 -> 33.6, whole-row rule
// B4 H12 N1024 11.0 + 18.3 -> 10.1 + 17.6.
template <int D, bool CAUSAL, bool RAGGED, bool SPLIT> constexpr bool kPlacedReads =
    D == 256 || (D == 64 && CAUSAL && RAGGED && !SPLIT);

// ---- sharing a block's key tiles out to several work-groups (SPLIT below)
// Shares of a block of `tiles` key tiles when the grid has `splits` work-groups per block: of two tiles at least,
// three from 2048 keys on (below that, start-up and merging cost more than a shorter chain takes off).
__host__ DEVI int split_shares(int tiles, int splits) {
  const int most = tiles / (tiles < 32 ? 2 : 3);
  return most < 1 ? 1 : most < splits ? most : splits;
}
// floats of a share of 32 rows in the workspace: the 32 x D accumulator, 32 normalisers, 32 row sums
template <int D> constexpr int kPartFloats = 32 * D + 64;
// largest normaliser the first n shares of a 32-row block ask for in row r (16 loads in flight)
template <int D> DEVI float largest_norm(const float* rows, int n, int r) {
  float m = -INFINITY;
  for (int s0 = 0; s0 < n; s0 += 16) {
    float v[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      if (i % 8 == 0 && s0 + i >= n) break;
      v[i] = rows[(size_t)min(s0 + i, n - 1) * kPartFloats<D> + 32 * D + r];
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      if (i % 8 == 0 && s0 + i >= n) break;
      m = fmaxf(m, v[i]);
    }
  }
  return m;
}
// first tile of share s (share `shares` would be the end)
DEVI int share_begin(int tiles, int s, int shares) { return tiles * s / shares; }

// Running maxima of a lane's 32 scores of a tile, fed in 2 x kMaxSteps steps (kb, st) so that a caller can spread
// them over its matrix instructions.  Alg. 3's rule (TWO) needs the two largest (a value met twice is both): two
// more scores x, y make max3(a1, x, y) the largest, and the second largest is the median of {a1, x, y} or the
// old a2 (a2 <= a1): 2.5 vector instructions per two scores and no mask bookkeeping.
constexpr int kMaxSteps = 8;
template <bool TWO> struct TileMax {
  float a1[2], a2[2], mid;
  // step 0 takes scores 0 .. 2, step st = 1 .. 6 scores 2 st + 1 and 2 st + 2, step 7 score 15
  template <int ST> DEVI void step(int kb, const f32x16& s) {
    if constexpr (ST == 0) {
      if (TWO) a2[kb] = __builtin_amdgcn_fmed3f(s[0], s[1], s[2]);
      a1[kb] = fmaxf(fmaxf(s[0], s[1]), s[2]);
    } else if constexpr (ST < 7) {
      const float x = s[2 * ST + 1], y = s[2 * ST + 2];
      if (TWO) {
        const float m = __builtin_amdgcn_fmed3f(a1[kb], x, y);
        if (ST % 2) mid = m; else a2[kb] = fmaxf(fmaxf(a2[kb], mid), m);
      }
      a1[kb] = fmaxf(fmaxf(a1[kb], x), y);
    } else {
      if (TWO) a2[kb] = __builtin_amdgcn_fmed3f(a1[kb], a2[kb], s[15]);
      a1[kb] = fmaxf(a1[kb], s[15]);
    }
  }
  DEVI void all(const f32x16 (&s)[2]) {
    static_for<2>([&](auto kb) { static_for<kMaxSteps>([&](auto st) { step<decltype(st)::value>(decltype(kb)::value, s[decltype(kb)::value]); }); });
  }
  DEVI float largest() const { return fmaxf(a1[0], a1[1]); }
  DEVI float second() const { return fmaxf(fmaxf(fminf(a1[0], a1[1]), a2[0]), a2[1]); }
};

// Normaliser a row asks for in one key tile (the two lanes of the row get the same): Alg. 1 (VARIANT 0) its
// maximum r_m, Alg. 3 (VARIANT 1) what the rule makes of it.  tm: maxima of the raw scores, masked ones -inf.
// In two pieces, which a caller can place apart: the largest (and second largest) raw scores of the row, and the rule.
struct RowMax { float mx, second; };
template <bool TWO> DEVI RowMax row_max(const TileMax<TWO>& tm) {
  if (!TWO) return {max_with_partner32(tm.largest()), 0.f};
  // Alg. 3's count r_s = #{ r_m - S <= eps } over the tile row only matters through "more than one", i.e. through
  // whether the SECOND largest score of the row passes the test: the two lanes that share a query row merge the
  // two largest of their 32 scores.
  const float t1 = tm.largest(), t2 = tm.second();
  const auto w1 = __builtin_amdgcn_permlane32_swap(__float_as_uint(t1), __float_as_uint(t1), false, false);
  const auto w2 = __builtin_amdgcn_permlane32_swap(__float_as_uint(t2), __float_as_uint(t2), false, false);
  const float x1 = __uint_as_float(w1[0]), y1 = __uint_as_float(w1[1]);       // the largest of either lane
  return {fmaxf(x1, y1), fmaxf(fmaxf(fminf(x1, y1), __uint_as_float(w2[0])), __uint_as_float(w2[1]))};
}
// may_be_unseen: a row may see no key of the tile.  allowed(r_m): whether a guard lets the rule apply.
// r_m: the tile row maximum of the alpha-scaled scores.
template <int VARIANT, class AllowedF>
DEVI float asked_normaliser(const RowMax& w, float alpha, float inv_alpha, float beta, float eps,
                            bool may_be_unseen, AllowedF&& allowed, float& r_m) {
  r_m = w.mx * alpha;
  if (VARIANT != 1) return r_m;
  // A repeated maximum moves the normaliser to beta*r_m (r_m > 0) or to 0 (r_m < 0).  The test
  // r_m - alpha*s <= eps  in terms of the raw score:  s >= (r_m - eps) / alpha
  // (a row with nothing visible in this tile has r_m = -inf: no rule, no update)
  const bool repeated = w.second >= (w.mx * alpha - eps) * inv_alpha && (!may_be_unseen || w.mx > -INFINITY) && allowed(r_m);
  const float m_prime = (repeated && r_m > 0.f) ? beta * r_m : r_m;
  return (repeated && r_m < 0.f) ? 0.f : m_prime;
}
template <int VARIANT, class AllowedF>
DEVI float tile_normaliser(const TileMax<VARIANT == 1>& tm, float alpha, float inv_alpha, float beta, float eps,
                           bool may_be_unseen, AllowedF&& allowed, float& r_m) {
  return asked_normaliser<VARIANT>(row_max(tm), alpha, inv_alpha, beta, eps, may_be_unseen, allowed, r_m);
}

// Waves per SIMD are stated as a range, not only as a minimum: at D = 128 two work-groups fit a
// CU (LDS), and told so the compiler spends the registers of the third wave it would otherwise
// keep room for on issuing LDS fragment reads ahead of their matrix instructions.
//
// SPLIT: grids of so few query blocks that most of the chip would idle (few heads, a chunk of queries
// against a long context).  The key tiles of a block are shared out to `splits` work-groups, in
// three launches: attn_fwd_norms_kernel leaves in `part` the largest normaliser each share's tiles ask for;
// this kernel starts every share from the largest normaliser of the shares before it and leaves the
// float32 accumulator and row sum; attn_fwd_merge_kernel joins them.  The running normaliser, and
// with it every rounded P-bar, is then the one of a single pass over the tiles (Alg. 3: a moved
// normaliser stays for the rest of the row), and only the order of the float32 sums differs: 3e-5 .. 1e-4
// relative in O, one bf16 step in 1 .. 5 of 10^4 elements.  Without the first launch a share would
// round P-bar against its own maximum: other roundings, more unit probabilities, 1e-3 .. 2e-3 relative.
template <int D, bool CAUSAL, int VARIANT, bool RAGGED, int EXTRAS, bool SPLIT = false>
__global__ __launch_bounds__(256)
__attribute__((amdgpu_waves_per_eu(kFwdWaves<D, CAUSAL, VARIANT, RAGGED, EXTRAS>, (D == 96 || D == 128) ? 2 : (D > 128 ? 1 : 8)))) void attn_fwd_kernel(
    const bf16_t* __restrict__ Q, const bf16_t* __restrict__ K, const bf16_t* __restrict__ V,
    bf16_t* __restrict__ O, float* __restrict__ LSE, int N, float alpha, float beta, float eps,
    FwdExtras ex, Layout lay, int pairs, float* __restrict__ part, int splits, BlockOrder ord) {
  constexpr int TILE_BYTES = kBc * D * 2;
  constexpr bool PIPE = kPipelined<D, CAUSAL> && VARIANT <= 1 && !EXTRAS && !SPLIT;
  // Row sums by matrix instruction (add_rows) where the vector work is what bounds the kernel: at D <= 64, and without a
  // mask at D <= 128 (us, dot products -> matrix instructions: B8 H12 N1024 d64 causal 29.1 -> 28.0, B32 H12 N512 d64 full
  // 48.5 -> 44.9, B4 H16 N2048 d128 full 156 -> 153, B2 H16 N2000 d96 full 74.3 -> 70.2; not taken: d256 full even (B2 H8 N2048
  // 82.7 -> 82.6, B4 H16 N4096 1211 -> 1225), B4 H32 N4096 d128 causal in the pipeline 601 -> 611).
  // (One rule for all kernels of a head size and mask: they give the same bits.)
  constexpr bool MFMA_SUMS = D <= 64 || (D <= 128 && !CAUSAL);
  extern __shared__ __attribute__((aligned(16))) char smem[];
  // layout: K buffers [2][TILE_BYTES], then V buffers [2][TILE_BYTES]

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int r = lane & 31, h = lane >> 5;

  // RAGGED: the bounds-checking instantiation.  N (queries) need not be a multiple of the block:
  // the last block's missing rows are computed on clamped data and not stored; NK keys, those
  // past the end are masked like future keys; the causal mask is  key <= query + shift.
  const int NK = RAGGED ? lay.Nk : N;
  const int shift = RAGGED ? NK - N : 0;
  // A score of -inf in a row that does see keys (overflowed inputs) is no "nothing visible": the aligned
  // instantiation treats it like any other, and so does SPLIT (always bounds-checking) at its sizes.
  const bool may_be_unseen = RAGGED && !(SPLIT && shift == 0 && N % kBr == 0);
  const int nqt = (N + kBr - 1) / kBr;
  // pairs != 0 (causal problems with enough work-groups): a work-group takes query block
  // nqt-1-idx and then its mirror image idx, which together always meet the same number of key
  // tiles, so every work-group carries the same load, there is no tail of heavy blocks at the
  // end of the grid, and half as many work-groups have to start and drain.  pairs == 0: one
  // block per work-group, for causal grids in the order the table `ord` gives (or, where the
  // table does not apply, heavy blocks first with a per-lap rotation on small grids).
  const int wg_all = logical_wg(ord, blockIdx.x, gridDim.x);
  const int split = SPLIT ? wg_all % splits : 0;        // neighbours share a block (and its Q)
  const int wg = SPLIT ? wg_all / splits : wg_all;
  const int npw = pairs ? (nqt + 1) / 2 : nqt;          // work-groups per head
  const int bh = wg / npw;
  const int idx = wg % npw;
  const size_t head_off = head_base(lay, bh);
  const int sn = lay.sn;
  const bf16_t* Qh = Q + head_off;
  const bf16_t* Kh = K + head_base_kv(lay, bh);
  const bf16_t* Vh = V + head_base_kv(lay, bh);

  TileLoader<D> loader;
  loader.init(tid, sn);
  FragOffsets<D> fo0;
  init_frag_offsets<D>(fo0, lane, lds_address(smem));
  const float c2 = alpha * kLog2e;
  const bf16x8 row_select = make_row_select(lane);
  // Alg. 3's test  r_m - alpha*s <= eps  in terms of the raw score s:  s >= (r_m - eps) / alpha
  const float inv_alpha = 1.0f / alpha;

  for (int half = 0; half < (pairs ? 2 : 1); ++half) {
  if (half > 0) __syncthreads();                      // the first block's output staging is done with the tile buffers
  // heavy (late) query blocks first under the causal mask
  const int qt = pairs ? (half == 0 ? nqt - 1 - idx : idx)
                       : nqt - 1 - (idx + (CAUSAL && !SPLIT && ord.n == 0 ? small_grid_rotation(bh, nqt, gridDim.x, D == 128 ? 768 : 1536) : 0)) % nqt;
  if (half == 1 && qt == nqt - 1 - idx) break;        // odd number of blocks: the middle one has no partner
  const int q0 = qt * kBr;
  const int qw = q0 + 32 * wave;                 // first query row of this wave
  const int q = qw + r;
  const int qc = (RAGGED && q >= N) ? N - 1 : q;   // row actually read for this lane

  // keys [0, kend) can matter to this block; its tiles, or this work-group's share of them
  const int kend = !CAUSAL ? NK : !RAGGED ? q0 + kBr : max(0, min(NK, q0 + kBr + shift));
  const int all_tiles = RAGGED ? (kend + kBc - 1) / kBc : kend / kBc;
  const int shares = SPLIT ? split_shares(all_tiles, splits) : 1;
  if (SPLIT && split >= shares) return;          // the block is too short for all of them
  const int tile0 = SPLIT ? share_begin(all_tiles, split, shares) : 0;
  const int ntiles = SPLIT ? share_begin(all_tiles, split + 1, shares) : all_tiles;
  loader.template load_rows<RAGGED>(smem, Kh, tile0 * kBc, NK);
  // kWholeRow: the buffer that the second pass begins with, filled in one burst ahead of the first pass's last scores, at D = 32 right
  // here.  (Spread over those scores like other transfers, every instruction needs a branch in every tile, which a SIMD with one
  // wave waits for; right here, short sequences wait for it.  us, spread -> here -> burst: H2 N4096 d128 causal 100.6 -> 92.5 -> 94.0,
  // H1 N4096 d96 full 77.6 -> 73.9 -> 74.8, H768 N100 d128 full 23.3 -> 25.0 -> 23.6, but H1 N4096 d32 full 53.9 -> 50.5 -> 52.1.)
  constexpr bool V_FIRST = VARIANT != kWholeRow || D == 32;
  if (V_FIRST) loader.template load_rows<RAGGED>(smem + (2 + (VARIANT == kWholeRow ? ntiles & 1 : 0)) * TILE_BYTES, Vh, tile0 * kBc, NK);
  if (PIPE) loader.template load_rows<RAGGED>(smem + TILE_BYTES, Kh, (ntiles > 1 ? 1 : 0) * kBc, NK);

  // Q_i^T fragments: lane (r,h) holds Q[qw + r][16kc + 8h .. +7] for every kc.
  bf16x8 qf[D / 16];
#pragma unroll
  for (int kc = 0; kc < D / 16; ++kc)
    qf[kc] = *reinterpret_cast<const bf16x8*>(Qh + (size_t)qc * sn + 16 * kc + 8 * h);

  f32x16 acc[D / 32];
#pragma unroll
  for (int db = 0; db < D / 32; ++db)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[db][i] = 0.f;

  int ones_cnt = 0, fired_cnt = 0;   // EXTRAS only
  float top1 = -INFINITY, top2 = -INFINITY;   // kWholeRow: the lane's two largest raw scores so far
  float m = -INFINITY;      // running normaliser, natural-log units of the alpha-scaled scores (kWholeRow: the row's, once chosen)
  float* share = SPLIT ? part + ((size_t)bh * ((N + 31) / 32) + qw / 32) * splits * kPartFloats<D> : nullptr;   // the rows' first share
  if (SPLIT && qw < N) m = largest_norm<D>(share, split, r);
  float lsum = 0.f;         // running row sum (the same in both lanes of a row; without MFMA_SUMS this lane's share of it)

  wait_vmem();
#pragma unroll
  for (int kc = 0; kc < D / 16; ++kc) settle(qf[kc]);
  if (SPLIT) settle(m);
  __syncthreads();

  FragOffsets<D> fo = fo0;
  // One key tile; BUF (which LDS buffer holds it) is a compile-time constant so that every LDS
  // address is a precomputed per-lane offset plus an immediate.
  // STATS (kWholeRow's first pass): scores and their maxima only.
  auto tile_step = [&](auto stats_c, auto buf_c, int j) {
    constexpr bool STATS = decltype(stats_c)::value;
    constexpr int BUF = decltype(buf_c)::value;
    constexpr int tK = BUF * TILE_BYTES;          // byte offsets of this tile's K and V in smem
    constexpr int tV = (2 + BUF) * TILE_BYTES;
    // The next tile lands in the other buffer while this one is being processed.  Its transfer
    // instructions are not issued in one burst (all eight waves of a CU would queue 64 KB of
    // requests right behind the barrier and sit at the head of the tile until the queue takes
    // them) but one per step of the score product.  After the last tile the current one is
    // fetched once more into the idle buffer: harmless, and the instruction stream stays free of
    // branches.
    const bool last = j + 1 >= ntiles;
    const int jn = !last ? j + 1 : STATS ? 0 : j;
    constexpr int NLD = TileLoader<D>::NI;
    const auto pendK = loader.template prepare<RAGGED>(smem + (BUF ^ 1) * TILE_BYTES, Kh, jn * kBc, NK);
    const auto pendV = loader.template prepare<RAGGED>(smem + (2 + (BUF ^ 1)) * TILE_BYTES, Vh, jn * kBc, NK);
    auto issue_part = [&](int i) {
      if (i < NLD) loader.issue(pendK, i);
      else if (i < 2 * NLD && !STATS) loader.issue(pendV, i - NLD);
    };
    if (STATS && !V_FIRST && last)
#pragma unroll
      for (int i = 0; i < NLD; ++i) loader.issue(pendV, i);
    bool issued = false;
    const int k0 = j * kBc;
    // A wave whose 32 rows all lie above this key tile has nothing to do in it (causal); of a chunk of a few queries
    // most waves hold no rows at all and only fetch.
    if ((!CAUSAL || (k0 <= qw + shift + 31)) && (!SPLIT || qw < N)) {
      // ---- S^T = K_j Q_i^T (Alg. 1 step 6); raw scores, alpha not yet applied
      f32x16 s[2];
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int i = 0; i < 16; ++i) s[kb][i] = 0.f;
      if constexpr (kPlacedReads<D, CAUSAL, RAGGED, SPLIT>) {
        constexpr int AHEAD = 2, RING = AHEAD + 1;
        auto fragment = [&](int i) { return lds_row8<D>(tK, fo, 32 * (i % 2), i / 2); };
        bf16x8 ring[RING];
#pragma unroll
        for (int i = 0; i < AHEAD; ++i) ring[i] = fragment(i);
        static_for<D / 8>([&](auto slot) {
          constexpr int sl = decltype(slot)::value;
          if (sl + AHEAD < D / 8) ring[(sl + AHEAD) % RING] = fragment(sl + AHEAD);
          s[sl % 2] = mfma32(ring[sl % RING], qf[sl / 2], s[sl % 2]);
          if (sl % 2) issue_part(sl / 2);
          __builtin_amdgcn_sched_barrier(0);
        });
      } else {
#pragma unroll
        for (int kc = 0; kc < D / 16; ++kc) {
#pragma unroll
          for (int kb = 0; kb < 2; ++kb) s[kb] = mfma32(lds_row8<D>(tK, fo, 32 * kb, kc), qf[kc], s[kb]);
          issue_part(kc);
        }
        sched_reads_ahead_of_mfma<D / 8, 1, 4>();
      }
#pragma unroll
      for (int i = D / 16; i < 2 * NLD; ++i) issue_part(i);
      issued = true;
      // ---- mask: causal (key > query) in the tile that crosses the diagonal, and keys beyond
      // the sequence end in the last, partial tile -> -inf
      if ((CAUSAL && (k0 + kBc - 1 > qw + shift)) || (RAGGED && k0 + kBc > NK)) {
        // element (kb, i) of this lane is key k0 + 4h + c with c = 32 kb + 8 (i / 4) + i % 4 a
        // compile-time constant: masked <=> c > lim, one per-lane limit for both conditions.  (Written
        // out here and not called: as a function its 32 comparisons come first and spill scalar registers.)
        // (At D <= 64 what it needs of the lane is formed here, from an opaque copy: ahead of the loop it costs registers.)
        int ql = q, hl = h;
        if constexpr (D <= 64) {
          int ln = lane;
          asm volatile("" : "+v"(ln));
          ql = __builtin_amdgcn_readfirstlane(qw) + (ln & 31);
          hl = ln >> 5;
        }
        int lim = CAUSAL ? ql + shift - k0 - 4 * hl : 0x7fffffff;
        if (RAGGED) lim = min(lim, NK - 1 - k0 - 4 * hl);
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
          for (int i = 0; i < 16; ++i)
            if (32 * kb + 8 * (i >> 2) + (i & 3) > lim) s[kb][i] = -INFINITY;
      }
      if constexpr (STATS) {
        TileMax<true> tm;                // merged into the two largest this lane has seen
        tm.all(s);
        const float t1 = tm.largest(), t2 = tm.second();
        top2 = fmaxf(fmaxf(fminf(top1, t1), top2), t2);
        top1 = fmaxf(top1, t1);
      } else {
        float corr = 1.f;    // factor the accumulated output and row sum are multiplied by
        float mneg;          // -m log2(e) of the normaliser used for this tile
        if (VARIANT == kWholeRow) {
          mneg = (RAGGED && m == -INFINITY) ? 0.f : -m * kLog2e;   // a query that sees no key at all
        } else {
          float r_m;         // tile row maximum of the alpha-scaled scores
          TileMax<VARIANT == 1> tm;
          tm.all(s);
          const float m_prime = tile_normaliser<VARIANT>(tm, alpha, inv_alpha, beta, eps, may_be_unseen, [&](float r) {
            return !EXTRAS || ex.guard == 0 || guard_allows(r, beta);
          }, r_m);
          if (EXTRAS && VARIANT == 1) fired_cnt += (m_prime != r_m) ? 1 : 0;
          const float m_new = fmaxf(m, m_prime);         // Alg. 1 step 7 / Alg. 3
          const bool unseen = may_be_unseen && m_new == -INFINITY;   // nothing visible so far: P-bar = 0, nothing to rescale
          corr = unseen ? 1.f : __builtin_amdgcn_exp2f((m - m_new) * kLog2e);
          m = m_new;
          mneg = unseen ? 0.f : -m_new * kLog2e;
        }
        if constexpr (EXTRAS == 2) {
          // ---- exploration beyond the paper (its future-work remark on FP8): the same step with
          // P-bar and V_j rounded to E4M3 and multiplied by the FP8 matrix instruction; the row sum
          // is of the rounded P-bar, everything downstream is unchanged.  Same k-slot order in
          // both operands as in the bf16 path.
          long pf8[2][2];
          float psum8 = 0.f;
#pragma unroll
          for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int cc = 0; cc < 2; ++cc) {
              float pv[8];
#pragma unroll
              for (int jj = 0; jj < 8; ++jj)
                pv[jj] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[kb][8 * cc + jj], c2, mneg));
              const long pk = pack_e4m3(pv);
              pf8[kb][cc] = pk;
              const int w0 = (int)(unsigned)pk, w1 = (int)(unsigned)((unsigned long long)pk >> 32);
              const float back[8] = {__builtin_amdgcn_cvt_f32_fp8(w0, 0), __builtin_amdgcn_cvt_f32_fp8(w0, 1),
                                     __builtin_amdgcn_cvt_f32_fp8(w0, 2), __builtin_amdgcn_cvt_f32_fp8(w0, 3),
                                     __builtin_amdgcn_cvt_f32_fp8(w1, 0), __builtin_amdgcn_cvt_f32_fp8(w1, 1),
                                     __builtin_amdgcn_cvt_f32_fp8(w1, 2), __builtin_amdgcn_cvt_f32_fp8(w1, 3)};
#pragma unroll
              for (int jj = 0; jj < 8; ++jj) {
                psum8 += back[jj];
                ones_cnt += back[jj] == 1.0f ? 1 : 0;
              }
            }
          lsum = lsum * corr + (MFMA_SUMS ? sum_with_partner32(psum8) : psum8);
          if (VARIANT != kWholeRow && j > tile0 && __builtin_amdgcn_ballot_w64(corr != 1.f) != 0) {
#pragma unroll
            for (int db = 0; db < D / 32; ++db)
#pragma unroll
              for (int i = 0; i < 16; ++i) acc[db][i] *= corr;
          }
#pragma unroll
          for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int cc = 0; cc < 2; ++cc)
#pragma unroll
              for (int db = 0; db < D / 32; ++db) {
                const bf16x8 v8 = lds_col8<D>(tV, fo, 32 * kb + 16 * cc, db);
                float vv[8];
#pragma unroll
                for (int jj = 0; jj < 8; ++jj) vv[jj] = (float)v8[jj];
                acc[db] = __builtin_amdgcn_mfma_f32_32x32x16_fp8_fp8(pack_e4m3(vv), pf8[kb][cc], acc[db], 0, 0, 0);
              }
        } else {
        // ---- P-bar = exp(S - m), rounded to bf16; row sum of the ROUNDED values
        bf16x8 pf[4];
        f32x4 psum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int c = 0; c < 4; ++c) {
#pragma unroll
          for (int jj = 0; jj < 8; ++jj) {
            const bf16_t p = (bf16_t)__builtin_amdgcn_exp2f(__builtin_fmaf(s[c >> 1][8 * (c & 1) + jj], c2, mneg));
            pf[c][jj] = p;
            if (EXTRAS) ones_cnt += (float)p == 1.0f ? 1 : 0;
          }
          if (MFMA_SUMS) psum = add_rows(pf[c], row_select, psum);
          else psum[0] = add_values(pf[c], psum[0]);
        }
        if (!MFMA_SUMS) lsum = lsum * corr + psum[0];
        // ---- O^T <- diag(corr) O^T + V_j^T P-bar^T (Alg. 1 step 8); in the first tile the
        // accumulator is still zero (corr = exp(-inf) = 0 there), nothing to rescale
        if (VARIANT != kWholeRow && j > tile0 && __builtin_amdgcn_ballot_w64(corr != 1.f) != 0) {
#pragma unroll
          for (int db = 0; db < D / 32; ++db)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[db][i] *= corr;
        }
        const bool not_finite = MFMA_SUMS && __builtin_amdgcn_ballot_w64(psum[0] != psum[0]) != 0;
        if constexpr (D == 256) {       // (kPlacedReads; at D = 64 the compiler keeps these reads ahead)
          constexpr int NDB = D / 32, AHEAD = 3, RING = AHEAD + 1;
          auto fragment = [&](int i) { return lds_col8<D>(tV, fo, 16 * (i / NDB), i % NDB); };
          bf16x8 ring[RING];
#pragma unroll
          for (int i = 0; i < AHEAD; ++i) ring[i] = fragment(i);
          __builtin_amdgcn_sched_barrier(0);
          static_for<4 * NDB>([&](auto slot) {
            constexpr int sl = decltype(slot)::value;
            if (sl + AHEAD < 4 * NDB) ring[(sl + AHEAD) % RING] = fragment(sl + AHEAD);
            acc[sl % NDB] = mfma32(ring[sl % RING], pf[sl / NDB], acc[sl % NDB]);
            __builtin_amdgcn_sched_barrier(0);
          });
        } else {
#pragma unroll
          for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int db = 0; db < D / 32; ++db) acc[db] = mfma32(lds_col8<D>(tV, fo, 16 * c, db), pf[c], acc[db]);
        }
        if (MFMA_SUMS) {
          if (not_finite) psum[0] = row_sum_apart(pf);
          lsum = lsum * corr + psum[0];
        }
        }
      }
    }
    if (!issued) {      // a wave that skipped the tile still has its share of the transfer to issue
#pragma unroll
      for (int i = 0; i < 2 * NLD; ++i) issue_part(i);
    }
    wait_vmem();
    __syncthreads();
  };

  // The same tiles as a software pipeline over tiles: one step holds the scores of tile j + 1 and the output product
  // of tile j as one stream of 4 x D/16 matrix instructions ("slots", a fence each, LDS fragments read AHEAD
  // slots before their use), with the vector work under them: P-bar of tile j under the scores of tile j + 1,
  // the row maxima of tile j + 1 under the output product.  K is read one tile ahead of V.
  // What no product covers makes a lone wave wait: so the first fragments of a step are read ahead of the accumulator's
  // rescale, and the chain from the maxima to the next normaliser lies under the last products.  us, both outside -> now, same
  // bits: B4 H32 N4096 d128 606 -> 596, B4 H16 N1999 d128 86.8 -> 85.5, B1 H8 N2048 d128 38.1 -> 36.5, B2 H16 N2048 d96
  // 40.5 -> 39.8, B8 H16 N512 d128 even.  (These kernels run at the board's power limit on large grids - the same instructions on
  // zeros take 0.71 of the time - where filling gaps gives less than it does on small ones.)
  static_assert(!PIPE || !MFMA_SUMS, "row sums of the pipeline");
  if constexpr (PIPE) {
    constexpr int NS = D / 16, NDB = D / 32, AHEAD = 4, RING = AHEAD + 1;
    // tiles this wave has anything to do with
    const int qu = __builtin_amdgcn_readfirstlane(qw) + shift;      // last key its first row sees
    const int seen = qu + 31 < 0 ? 0 : min(ntiles, (qu + 31) / kBc + 1);
    f32x16 s0[2], s1[2];                               // raw scores of even and odd tiles
    float corr = 1.f, mneg = 0.f;                      // of the tile whose P-bar is next
    const int plain = min(seen, min(RAGGED ? NK / kBc : ntiles, max(0, qu + 1) / kBc));     // tiles that need no mask: the first ones
    auto limit = [&](int j) {                          // last visible c = 32 kb + 8 (i / 4) + i % 4 of tile j
      const int lim = q + shift - j * kBc - 4 * h;
      return RAGGED ? min(lim, NK - 1 - j * kBc - 4 * h) : lim;
    };
    // scores 16 kb + lo .. of a tile that crosses the diagonal or the sequence end
    auto mask = [&](f32x16& s, int kb, int lo, int hi, int lim) {
#pragma unroll
      for (int i = lo; i < hi; ++i)
        s[i] = 32 * kb + 8 * (i >> 2) + (i & 3) > lim ? -INFINITY : s[i];
    };
    // running normaliser after a tile, and what its P-bar needs (m_prime: what the tile asks for)
    auto asked = [&](const RowMax& w) {
      float r_m;
      return asked_normaliser<VARIANT>(w, alpha, inv_alpha, beta, eps, may_be_unseen, [](float) { return true; }, r_m);
    };
    auto advance = [&](float m_prime, float& factor) {
      const float m_new = fmaxf(m, m_prime);         // Alg. 1 step 7 / Alg. 3
      const bool unseen = may_be_unseen && m_new == -INFINITY;   // nothing visible so far: P-bar = 0, nothing to rescale
      factor = unseen ? 1.f : __builtin_amdgcn_exp2f((m - m_new) * kLog2e);
      m = m_new;
      mneg = unseen ? 0.f : -m_new * kLog2e;
    };
    // The LDS buffers change by adding to the fragment addresses (fo.row: the next tile's K, fo.col: this tile's V).
    int par = 0, turn = TILE_BYTES;                    // parity of the tile: its V buffer, the other K buffer
    constexpr int NLD = TileLoader<D>::NI;
    typename TileLoader<D>::Pending pendK, pendV;
    // K of tile j + 2 and V of tile j + 1 (past the last tile: that one once more, harmlessly)
    auto prepare = [&](int j) {
      pendK = loader.template prepare<RAGGED>(smem + par * TILE_BYTES, Kh, min(j + 2, ntiles - 1) * kBc, NK);
      pendV = loader.template prepare<RAGGED>(smem + (2 + (par ^ 1)) * TILE_BYTES, Vh, min(j + 1, ntiles - 1) * kBc, NK);
    };
    auto issue_part = [&](int i) {
      if (i < NLD) loader.template issue<true>(pendK, i);
      else if (i < 2 * NLD) loader.template issue<true>(pendV, i - NLD);
    };
    auto finish = [&]() {
      wait_vmem();
      __syncthreads();
      par ^= 1;
    };
    auto step = [&](auto next_c, auto masked_c, int j, f32x16 (&sc)[2], f32x16 (&sn)[2]) {
      constexpr bool NEXT = decltype(next_c)::value, MASKED = decltype(masked_c)::value;
      constexpr int FIRST = NEXT ? 0 : 2 * NS, SLOTS = 4 * NS;
      auto fragment = [&](int i) -> bf16x8 {
        if (i < 2 * NS) return lds_row8<D>(0, fo, 32 * (i / NS), i % NS);
        return lds_col8<D>(0, fo, 16 * ((i - 2 * NS) / NDB), (i - 2 * NS) % NDB);
      };
      prepare(j);
      bf16x8 ring[RING], pf[4];
      float psum = 0.f;
      TileMax<VARIANT == 1> tm;
      const int lim = MASKED ? limit(j + 1) : 0;
#pragma unroll
      for (int i = 0; i < AHEAD; ++i) ring[(FIRST + i) % RING] = fragment(FIRST + i);
      __builtin_amdgcn_sched_barrier(0);               // (the reads' latency lies under what follows)
      // O^T <- diag(corr) O^T (Alg. 1 step 8); in the first tile the accumulator is still zero.
      // SPREAD: always, and under the scores.  D = 256 has 128 products to rescale and the least vector work per matrix
      // instruction, which hides them: us, B2 H8 N2048 66.1 -> 62.4, B1 H8 64.0 -> 60.7.  At D = 128 B1 H8 N2048 35.0 -> 34.8, but
      // B1 H16 N16384 1005 -> 1043, where two tiles of three need none.
      constexpr bool SPREAD = NEXT && D == 256;
      if (!SPREAD && j > 0 && __builtin_amdgcn_ballot_w64(corr != 1.f) != 0) {
#pragma unroll
        for (int db = 0; db < NDB; ++db)
#pragma unroll
          for (int i = 0; i < 16; ++i) acc[db][i] *= corr;
      }
      RowMax row;
      float m_prime = 0.f, corr_next = 1.f;
      if (NEXT) {
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
          for (int i = 0; i < 16; ++i) sn[kb][i] = 0.f;
      }
      // P-bar = exp(S - m) of entries e0 .. e1 - 1 (of 32), rounded to bf16; row sum of the ROUNDED values
      auto form_p = [&](int e0, int e1) {
#pragma unroll
        for (int e = e0; e < e1; ++e) {
          const bf16_t p = (bf16_t)__builtin_amdgcn_exp2f(__builtin_fmaf(sc[e >> 4][e & 15], c2, mneg));
          pf[e >> 3][e & 7] = p;
          if (e % 8 == 7) psum = add_values(pf[e >> 3], psum);
        }
      };
      if (!NEXT) form_p(0, 8);
      static_for<SLOTS - FIRST>([&](auto slot) {
        constexpr int sl = FIRST + decltype(slot)::value;
        if (sl + AHEAD < SLOTS) ring[(sl + AHEAD) % RING] = fragment(sl + AHEAD);
        const bf16x8 a = ring[sl % RING];
        if constexpr (sl < 2 * NS) sn[sl / NS] = mfma32(a, qf[sl % NS], sn[sl / NS]);
        else acc[(sl - 2 * NS) % NDB] = mfma32(a, pf[(sl - 2 * NS) / NDB], acc[(sl - 2 * NS) % NDB]);
        // (one transfer instruction per two slots: us, one slot -> two, and the immediate offset, B4 H32 N4096 d128 583 -> 575, B1 H8
        // N2048 35.5 -> 34.7, B2 H16 N2048 d96 37.4 -> 37.1, B2 H8 N2048 d256 66.2 -> 64.4)
        if (!NEXT) issue_part(sl - FIRST);
        else if (sl % 2 == 0) issue_part(sl / 2);
        if constexpr (sl < 2 * NS) {
          if constexpr (SPREAD) {
            constexpr int each = 16 * NDB / (2 * NS);
#pragma unroll
            for (int i = each * sl; i < each * (sl + 1); ++i) acc[i / 16][i % 16] *= corr;
          }
          form_p(16 * sl / NS, 16 * (sl + 1) / NS);
        } else {
          constexpr int u = sl - 2 * NS;
          if (!NEXT && u % NDB == 0 && u / NDB < 3) form_p(8 * (u / NDB + 1), 8 * (u / NDB + 2));
          if constexpr (NEXT) {
            // steps of the row maxima, over all but the last quarter of the slots, and there, piece by piece, the chain of
            // dependent instructions from them to the next tile's normaliser
            constexpr int SPAN = NS * 3 / 2, Q = (2 * NS - SPAN) / 3, F = 2 * kMaxSteps * u / SPAN, L = 2 * kMaxSteps * (u + 1) / SPAN;
            static_for<(u < SPAN ? L - F : 0)>([&](auto k) {
              constexpr int t = F + decltype(k)::value, kb = t / kMaxSteps, st = t % kMaxSteps;
              if (MASKED) mask(sn[kb], kb, st == 0 ? 0 : 2 * st + 1, st == 0 ? 3 : st < 7 ? 2 * st + 3 : 16, lim);
              tm.template step<st>(kb, sn[kb]);
            });
            if constexpr (u == SPAN) row = row_max(tm);
            if constexpr (u == SPAN + Q) m_prime = asked(row);
            if constexpr (u == SPAN + 2 * Q) advance(m_prime, corr_next);
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      });
      lsum = lsum * corr + psum;
      corr = corr_next;
#pragma unroll
      for (int p = 0; p < 2; ++p) { fo.row[p] -= turn; fo.col[p] += turn; }
      turn = -turn;
      finish();
    };
    // ---- scores of the first tile
    if (seen > 0) {
      static_for<2 * NS>([&](auto i) {
        constexpr int sl = decltype(i)::value;
        if (sl % NS == 0) {
#pragma unroll
          for (int e = 0; e < 16; ++e) s0[sl / NS][e] = 0.f;
        }
        s0[sl / NS] = mfma32(lds_row8<D>(0, fo, 32 * (sl / NS), sl % NS), qf[sl % NS], s0[sl / NS]);
      });
      sched_reads_ahead_of_mfma<2 * NS, 1, 4>();
      if (plain == 0) {
        const int lim = limit(0);
        mask(s0[0], 0, 0, 16, lim);
        mask(s0[1], 1, 0, 16, lim);
      }
      TileMax<VARIANT == 1> tm;
      tm.all(s0);
      advance(asked(row_max(tm)), corr);
    }
    __syncthreads();                                   // K of the first tile is read out everywhere: its buffer is free
#pragma unroll
    for (int p = 0; p < 2; ++p) { fo.row[p] += TILE_BYTES; fo.col[p] += 2 * TILE_BYTES; }
    // Counted loops, two steps a turn where no mask is needed.  (With the test for the mask between the two steps the loop had
    // another way out, on which the compiler kept the accumulator a second time: 20 moves a tile.  us, that -> now, same bits:
    // B4 H32 N4096 d128 597 -> 589, B1 H16 N16384 1053 -> 1040, B4 H16 N1999 85.4 -> 83.2, B1 H8 N2048 36.4 -> 35.5, B2 H16
    // N2048 d96 39.7 -> 39.2, d256 B1 H8 65.4 -> 64.7.)
    int j = 0;
    for (; j + 2 < plain; j += 2) {
      step(std::true_type{}, std::false_type{}, j, s0, s1);
      step(std::true_type{}, std::false_type{}, j + 1, s1, s0);
    }
    if (j + 1 < plain) {
      step(std::true_type{}, std::false_type{}, j++, s0, s1);
      s0[0] = s1[0];
      s0[1] = s1[1];
    }
    for (; j + 1 < seen; ++j) {
      step(std::true_type{}, std::true_type{}, j, s0, s1);
      s0[0] = s1[0];
      s0[1] = s1[1];
    }
    if (j < seen) {
      step(std::false_type{}, std::false_type{}, j, s0, s1);
      ++j;
    }
    for (; j < ntiles; ++j) {                          // the other waves' tiles: this wave's share of the transfers
      prepare(j);
#pragma unroll
      for (int i = 0; i < 2 * NLD; ++i) issue_part(i);
      finish();
    }
  } else {
    constexpr std::integral_constant<int, 0> buf0;
    constexpr std::integral_constant<int, 1> buf1;
    int begin = tile0;
    if constexpr (VARIANT == kWholeRow) {
      for (int j = 0; j < ntiles; j += 2) {
        tile_step(std::true_type{}, buf0, j);
        if (j + 1 < ntiles) tile_step(std::true_type{}, buf1, j + 1);
      }
      // merge the two lanes of a row, then the rule of Sec. 4 on the whole row
      const float o1 = partner32(top1), o2 = partner32(top2);
      const float M1 = fmaxf(top1, o1);
      const float M2 = fmaxf(fminf(top1, o1), fmaxf(top2, o2));
      const float r_m = M1 * alpha;
      bool repeated = (r_m - M2 * alpha) <= eps;            // r_s > 1
      if (EXTRAS && ex.guard != 0) repeated = repeated && guard_allows(r_m, beta);
      m = (repeated && r_m > 0.f) ? beta * r_m : r_m;
      m = (repeated && r_m < 0.f) ? 0.f : m;
      if (EXTRAS && ex.fired != nullptr && h == 0 && q < N) ex.fired[(size_t)bh * N + q] = (m != r_m) ? 1 : 0;
      begin = -(ntiles & 1);           // the first tile again: in the buffer after the last one's
    }
    for (int j = begin; j < ntiles; j += 2) {
      if (VARIANT != kWholeRow || j >= 0) tile_step(std::false_type{}, buf0, j);
      if (j + 1 < ntiles) tile_step(std::false_type{}, buf1, j + 1);
    }
  }

  if constexpr (SPLIT) {
    // the share's sums, as the registers hold them (16 bytes per lane, lanes consecutive)
    const float l_share = MFMA_SUMS ? lsum : sum_with_partner32(lsum);
    if (qw < N) {
      float* p = share + (size_t)split * kPartFloats<D>;
#pragma unroll
      for (int db = 0; db < D / 32; ++db)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          f32x4 v;
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] = acc[db][4 * g + e];
          *reinterpret_cast<f32x4*>(p + ((db * 4 + g) * 64 + lane) * 4) = v;
        }
      if (h == 0) p[32 * D + 32 + r] = l_share;
    }
    return;
  }
  // ---- epilogue (Alg. 1 steps 10-13).  Rounding points of Sec. 3.3.2: the unnormalised
  // output is rounded to bf16 first, then divided by l, then rounded again.
  const float l = MFMA_SUMS ? lsum : sum_with_partner32(lsum);
  int ones_row = 0;
  if (EXTRAS) {   // the partner lane counted the other 32 keys of every tile
    auto sw = __builtin_amdgcn_permlane32_swap((unsigned)ones_cnt, (unsigned)ones_cnt, false, false);
    ones_row = (int)(sw[0] + sw[1]);
  }
  const bool keep_obar_f32 = EXTRAS && ex.single_rounding != 0;
  // No visible key (more queries than keys): O = 0, LSE = -inf.  A row of NaN scores also leaves m at -inf (the maxima pass
  // NaN over), but its l is NaN: it stays NaN, as in the kernels without this case.
  const bool unseen_row = RAGGED && m == -INFINITY && l == 0.f;
  const Divisor by_l = make_divisor(l);
  auto o_piece = [&](int db, int g) {
    bf16x4 o4;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float a = acc[db][4 * g + e];
      const float obar = keep_obar_f32 ? a : (float)(bf16_t)a;
      o4[e] = (bf16_t)(unseen_row ? 0.f : divide(obar, by_l));
    }
    return o4;
  };
  if constexpr (kCanStage<D / 32>) {
    // the tile buffers are free now (every wave is past the last tile's barrier) and serve as the
    // staging areas of store_rows_staged; the barrier at the top of the part loop keeps the next
    // block's tile transfers from overwriting an area a slower wave is still reading
    store_rows_staged<D / 32>(smem, o_piece, O + head_off + (size_t)qw * sn, sn, RAGGED ? N - qw : 32, tid);
  }
  if (!RAGGED || q < N) {                                  // rows past the sequence end exist only as padding
  if constexpr (!kCanStage<D / 32>) {
    bf16_t* Oq = O + head_off + (size_t)q * sn;
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
      for (int g = 0; g < 4; ++g) *reinterpret_cast<bf16x4*>(Oq + 32 * db + 8 * g + 4 * h) = o_piece(db, g);
  }
  if (EXTRAS && ex.O_hp != nullptr) {
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        f32x4 hp;
#pragma unroll
        for (int e = 0; e < 4; ++e) hp[e] = unseen_row ? 0.f : divide(acc[db][4 * g + e], by_l);
        *reinterpret_cast<f32x4*>(ex.O_hp + ((size_t)bh * N + q) * D + 32 * db + 8 * g + 4 * h) = hp;
      }
  }
  if (h == 0) {
    LSE[(size_t)bh * N + q] = m + __logf(l);
    if (EXTRAS && ex.ones != nullptr) ex.ones[(size_t)bh * N + q] = ones_row;
    if (EXTRAS && VARIANT != kWholeRow && ex.fired != nullptr) ex.fired[(size_t)bh * N + q] = fired_cnt;
  }
  }
  }   // part
}

// First launch of the SPLIT forward: per row and share the largest normaliser its tiles ask for (the same
// score products and rule as the kernel above, bit for bit).  Shares are few tiles long and only K is
// read, so latency bounds it: K comes 128 rows at a time, in the LDS of the other launch's K and V.
template <int D, bool CAUSAL, int VARIANT>
__global__ __launch_bounds__(256)
__attribute__((amdgpu_waves_per_eu(D <= 128 ? 2 : 1, D <= 128 ? 2 : 1))) void attn_fwd_norms_kernel(
    const bf16_t* __restrict__ Q, const bf16_t* __restrict__ K, int N, float alpha, float beta, float eps,
    Layout lay, float* __restrict__ part, int splits) {
  constexpr int STEP = 2 * kBc, STEP_BYTES = STEP * D * 2;
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int r = lane & 31, h = lane >> 5;
  const int NK = lay.Nk, shift = NK - N;
  const bool may_be_unseen = !(shift == 0 && N % kBr == 0);
  const int nqt = (N + kBr - 1) / kBr;
  const int wg_all = xcd_remap(blockIdx.x, gridDim.x);
  const int split = wg_all % splits, wg = wg_all / splits;
  const int bh = wg / nqt, q0 = (nqt - 1 - wg % nqt) * kBr;
  const int qw = q0 + 32 * wave, q = qw + r, qc = min(q, N - 1);
  const int kend = !CAUSAL ? NK : max(0, min(NK, q0 + kBr + shift));
  const int all_tiles = (kend + kBc - 1) / kBc;
  const int shares = split_shares(all_tiles, splits);
  if (split >= shares) return;
  const int tile0 = share_begin(all_tiles, split, shares), ntiles = share_begin(all_tiles, split + 1, shares);
  const bf16_t* Kh = K + head_base_kv(lay, bh);
  TileLoader<D, STEP> loader;
  loader.init(tid, lay.sn);
  loader.template load_rows<true>(smem, Kh, tile0 * kBc, NK);
  const bf16_t* Qr = Q + head_base(lay, bh) + (size_t)qc * lay.sn + 8 * h;
  bf16x8 qf[D / 16];
#pragma unroll
  for (int kc = 0; kc < D / 16; ++kc) qf[kc] = *reinterpret_cast<const bf16x8*>(Qr + 16 * kc);
  FragOffsets<D> fo;
  init_frag_offsets<D>(fo, lane, lds_address(smem));
  const float inv_alpha = 1.0f / alpha;
  float m = -INFINITY;
  wait_vmem();
#pragma unroll
  for (int kc = 0; kc < D / 16; ++kc) settle(qf[kc]);
  __syncthreads();
  auto step = [&](auto buf_c, int j0) {
    constexpr int BUF = decltype(buf_c)::value;
    if (j0 + 2 < ntiles) loader.template load_rows<true>(smem + (BUF ^ 1) * STEP_BYTES, Kh, (j0 + 2) * kBc, NK);
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int k0 = (j0 + t) * kBc;
      if (j0 + t >= ntiles || (CAUSAL && k0 > qw + shift + 31) || qw >= N) continue;
      f32x16 s[2];
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int i = 0; i < 16; ++i) s[kb][i] = 0.f;
#pragma unroll
      for (int kc = 0; kc < D / 16; ++kc)
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
          s[kb] = mfma32(lds_row8<D>(BUF * STEP_BYTES, fo, kBc * t + 32 * kb, kc), qf[kc], s[kb]);
      sched_reads_ahead_of_mfma<D / 8, 1, 4>();
      if ((CAUSAL && k0 + kBc - 1 > qw + shift) || k0 + kBc > NK) {
        const int lim = min(CAUSAL ? q + shift - k0 - 4 * h : 0x7fffffff, NK - 1 - k0 - 4 * h);
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
          for (int i = 0; i < 16; ++i)
            if (32 * kb + 8 * (i >> 2) + (i & 3) > lim) s[kb][i] = -INFINITY;
      }
      float r_m;
      TileMax<VARIANT == 1> tm;
      tm.all(s);
      m = fmaxf(m, tile_normaliser<VARIANT>(tm, alpha, inv_alpha, beta, eps, may_be_unseen, [](float) { return true; }, r_m));
    }
    wait_vmem();
    __syncthreads();
  };
  for (int j = tile0; j < ntiles; j += 4) {
    step(std::integral_constant<int, 0>{}, j);
    if (j + 2 < ntiles) step(std::integral_constant<int, 1>{}, j + 2);
  }
  if (qw < N && h == 0)
    part[(((size_t)bh * ((N + 31) / 32) + qw / 32) * splits + split) * kPartFloats<D> + 32 * D + r] = m;
}

// Joins the shares of the SPLIT forward: one wave per 32 rows x 32 columns.  The normaliser of a row
// is the largest any of its shares asked for; a share's sums stand relative to the largest of its own
// and the shares before it.  They are brought to the row's normaliser in float32, and the roundings of
// the ordinary epilogue follow.  Streams the shares once; work-groups of one wave, as there are few of them and each
// should have a CU to itself.  They take the heads and blocks in the order of the other two launches, so that a block is joined
// on the XCD that summed it: its shares come from that XCD's L2, and the next call's sums are written to lines no other XCD
// holds.  us, sums + merge, rows in their own order in work-groups of four waves -> of one -> now: B2 H4 64 x 4096 d64
// 8.8 + 6.5 -> 8.6 + 10.1 -> 9.0 + 5.9, d32 8.0 + 9.4 -> 7.5 + 9.0 -> 7.5 + 5.8, B1 H8 2048 x 2048 causal d256 35.9 + 12.9
// -> 35.8 + 14.1 -> 35.8 + 13.0, B1 H4 2048 x 2048 causal d128 17.6 + 7.1 -> 18.4 + 6.9 -> 14.8 + 6.7, B2 H16 64 x 8192 d128
// 24.8 + 6.0 -> 24.7 + 5.5 -> 24.8 + 5.6.
template <int D, bool CAUSAL>
__global__ __launch_bounds__(64) void attn_fwd_merge_kernel(
    const float* __restrict__ part, bf16_t* __restrict__ O, float* __restrict__ LSE, int N,
    Layout lay, int splits) {
  constexpr int NDB = D / 32;
  const int lane = threadIdx.x & 63;
  const int r = lane & 31, h = lane >> 5;
  const int nrb = (N + 31) / 32;
  const int id = xcd_remap(blockIdx.x, gridDim.x);
  const int db = id % NDB;
  const int bh = id / (NDB * nrb);
  const int rb = nrb - 1 - id / NDB % nrb;    // 32-row block of the head, last ones first
  const int rows = bh * nrb + rb, qw = rb * 32;
  const int shift = lay.Nk - N;
  const int kend = !CAUSAL ? lay.Nk : max(0, min(lay.Nk, qw / kBr * kBr + kBr + shift));
  const int shares = split_shares((kend + kBc - 1) / kBc, splits);
  const float* p = part + (size_t)rows * splits * kPartFloats<D>;
  // Shares come in batches whose loads are all in flight at once; the first batch's are issued ahead of those of the row's
  // normaliser, so that a row of up to kBatch shares waits for memory once.  All three launches, us, four shares at a time after the
  // normaliser -> now, same bits: B2 H16 64 x 8192 d128 (8 shares) 43.0 -> 41.5, B8 H1 1 x 16384 (32) 36.2 -> 29.9, B3 H5
  // 100 x 3000 full (15) 27.0 -> 24.5, B1 H8 2048 x 2048 (4) 35.5 -> 34.9.
  constexpr int kBatch = 8;
  f32x4 v[kBatch][4];
  float norm[kBatch], sum[kBatch];
  auto fetch = [&](int s0) {
#pragma unroll
    for (int i = 0; i < kBatch; ++i) {
      if (i == kBatch / 2 && s0 + i >= shares) break;
      const float* ps = p + (size_t)min(s0 + i, shares - 1) * kPartFloats<D>;
      norm[i] = ps[32 * D + r];
      sum[i] = ps[32 * D + 32 + r];
#pragma unroll
      for (int g = 0; g < 4; ++g) v[i][g] = *reinterpret_cast<const f32x4*>(ps + ((db * 4 + g) * 64 + lane) * 4);
    }
  };
  fetch(0);
  const float m = largest_norm<D>(p, shares, r);
  f32x16 acc;
#pragma unroll
  for (int i = 0; i < 16; ++i) acc[i] = 0.f;
  float l = 0.f, m_here = -INFINITY;
  for (int s0 = 0; s0 < shares; s0 += kBatch) {
    if (s0 > 0) fetch(s0);
#pragma unroll
    for (int i = 0; i < kBatch; ++i) {
      if (s0 + i >= shares) break;
      m_here = fmaxf(m_here, norm[i]);
      // as long as the row has seen nothing its normaliser is -inf and its sums are zero
      const float w = m_here == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((m_here - m) * kLog2e);
      l = __builtin_fmaf(w, sum[i], l);
#pragma unroll
      for (int g = 0; g < 4; ++g)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[4 * g + e] = __builtin_fmaf(w, v[i][g][e], acc[4 * g + e]);
    }
  }
  if (qw + r >= N) return;
  const bool unseen_row = m == -INFINITY && l == 0.f;      // no visible key: O = 0, LSE = -inf (l is NaN where scores were -inf)
  const Divisor by_l = make_divisor(l);
  bf16_t* Oq = O + head_base(lay, bh) + (size_t)(qw + r) * lay.sn + 32 * db + 4 * h;
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    bf16x4 o4;
#pragma unroll
    for (int e = 0; e < 4; ++e) o4[e] = (bf16_t)(unseen_row ? 0.f : divide((float)(bf16_t)acc[4 * g + e], by_l));
    *reinterpret_cast<bf16x4*>(Oq + 8 * g) = o4;
  }
  if (db == 0 && h == 0) LSE[(size_t)bh * N + qw + r] = m + __logf(l);
}

}  // namespace

extern "C" int attn_fwd_key_tile(int d) { return (d == 32 || d == 64 || d == 96 || d == 128 || d == 256) ? kBc : 0; }

template <int D, bool CAUSAL, int VARIANT, bool RAGGED, int EXTRAS>
static hipError_t launch_fwd(const void* Q, const void* K, const void* V, void* O, float* LSE,
                             int BH, int N, float alpha, float beta, float eps, FwdExtras ex,
                             Layout lay, hipStream_t st) {
  constexpr int smem = 4 * kBc * D * 2;
  static std::atomic<bool> attr_set{false};   // (calls from several host threads may race to set it: harmless, the call is idempotent)
  auto kern = attn_fwd_kernel<D, CAUSAL, VARIANT, RAGGED, EXTRAS>;
  if (!attr_set.load(std::memory_order_acquire)) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, smem);
    if (e != hipSuccess) return e;
    attr_set.store(true, std::memory_order_release);
  }
  // Under the causal mask a work-group takes a query block and its mirror image (equal work for
  // all) when that still leaves at least two full rounds of work-groups (two fit a CU, 256 CUs);
  // smaller grids keep one block per work-group, in a balanced order (below).
  const int nqt = (N + kBr - 1) / kBr;
  const int pairs = (CAUSAL && (long long)BH * ((nqt + 1) / 2) >= 1024) ? 1 : 0;
  dim3 grid(BH * (pairs ? (nqt + 1) / 2 : nqt));
  // one block per work-group: in the order that balances the compute units (block_order.hpp)
  // whenever the table can express the grid (measured: -12..-21 % at one to three rounds of
  // work-groups against heavy-first order)
  static std::atomic<int> resident{0};
  static thread_local OrderCache cache;
  const BlockOrder& ord = (CAUSAL && !pairs)
      ? small_grid_order(cache, (int)grid.x, nqt, resident_per_cu(kern, smem, resident), 8 * kMaxOrder) : kNoOrder;
  hipLaunchKernelGGL(kern, grid, dim3(256), smem, st, (const bf16_t*)Q, (const bf16_t*)K,
                     (const bf16_t*)V, (bf16_t*)O, LSE, N, alpha, beta, eps, ex, lay, pairs,
                     (float*)nullptr, 1, ord);
  return hipGetLastError();
}

template <int D, bool CAUSAL, int VARIANT>
static hipError_t launch_fwd_split(const void* Q, const void* K, const void* V, void* O, float* LSE,
                                   int BH, int N, float alpha, float beta, float eps, Layout lay,
                                   float* part, int splits, hipStream_t st) {
  constexpr int smem = 4 * kBc * D * 2;
  static std::atomic<bool> attr_set{false};
  auto norms = attn_fwd_norms_kernel<D, CAUSAL, VARIANT>;
  auto sums = attn_fwd_kernel<D, CAUSAL, VARIANT, true, 0, true>;
  hipError_t e;
  if (!attr_set.load(std::memory_order_acquire)) {
    for (const void* kern : {reinterpret_cast<const void*>(norms), reinterpret_cast<const void*>(sums)})
      if ((e = hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, smem)) != hipSuccess) return e;
    attr_set.store(true, std::memory_order_release);
  }
  const dim3 grid(BH * ((N + kBr - 1) / kBr) * splits);
  hipLaunchKernelGGL(norms, grid, dim3(256), smem, st, (const bf16_t*)Q, (const bf16_t*)K, N, alpha, beta, eps, lay, part, splits);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  hipLaunchKernelGGL(sums, grid, dim3(256), smem, st, (const bf16_t*)Q, (const bf16_t*)K, (const bf16_t*)V, (bf16_t*)O, LSE, N,
                     alpha, beta, eps, FwdExtras{}, lay, 0, part, splits, kNoOrder);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  const int waves = BH * ((N + 31) / 32) * (D / 32);
  hipLaunchKernelGGL((attn_fwd_merge_kernel<D, CAUSAL>), dim3(waves), dim3(64), 0, st, part,
                     (bf16_t*)O, LSE, N, lay, splits);
  return hipGetLastError();
}

// Work-groups per query block of the SPLIT forward; 1: the ordinary kernel.
// The chip is filled once (256 work-groups); twice under the causal mask when blocks differ in work.
// A tile takes a lone work-group about 1 us (2 us at d = 256); the two extra launches cost 6 to 10 us,
// and up to a third of the score products is done twice.  Measured, one work-group per block -> shares (us,
// launches included; B*H, Nq x Nk):
//   up to 64 blocks: 32, 64 x 8192 d128 154 -> 46, 8, 1 x 16384 d128 296 -> 40, 16, 256 x 4096 d128 81 -> 33, 4, 2048 x 2048 causal
//     d128 41 -> 33, full 39 -> 34, d32 24 -> 20, 1, 8192 x 8192 causal d64 113 -> 46, 64, 64 x 1024 d128 25 -> 22, d64 19.1 -> 18.7;
//   65 to 128 blocks, from 2048 keys on with three work-groups per block (two at d = 256), from 2560 on with two: 8,
//     2048 x 2048 causal d128 42 -> 38, d256 88 -> 71, 80, 64 x 2048 d128 43 -> 35, 1, 16384 x 16384 causal 288 -> 200, 128,
//     64 x 2048 d256 99 -> 88; with two 96, 128 x 3000 causal d32 42 -> 39, d128 63 -> 60, 128, 64 x 4096 d64 59 -> 51, d128
//     80 -> 71, 16, 1000 x 6000 causal d96 100 -> 87, 1, 16000 x 16000 full d64 203 -> 166; even at the limit (4, 4096 x 4096
//     full d64 55.3 -> 53.8, d96 62.2 -> 63.5, 30, 300 x 2500 d32 32.2 -> 31.6); beyond the limits: 8, 2048 x 2048 full d64
//     30 -> 35, d128 40 -> 49, 96, 128 x 2048 causal d96 38.0 -> 39.4, 10, 1536 x 1536 causal d128 33 -> 36;
//   1024 to 1535 keys and many queries, d <= 128, only with 10 work-groups per block: 2, 1024 x 1024 causal d64
//     18.7 -> 17.4, d128 23.4 -> 19.9, 4, 1024 x 1024 causal d128 23.7 -> 22.2, even at the limit (2, 1500 x 1030 full d128
//     25.5 -> 24.6, d64 19.2 -> 19.9, 3, 1024 x 1024 full d64 17.0 -> 18.3); beyond it: 8, 1024 x 1024 causal d64
//     18.9 -> 22.5, 16, 512 x 1024 causal d128 26 -> 28.
int attn_fwd_splits(int BH, int Nq, int Nk, int d, int causal, int variant) {
  const long long blocks = (long long)BH * ((Nq + kBr - 1) / kBr);
  if (variant == 2 || Nk < 1024 || 2 * blocks > kNumCUs) return 1;
  const long long s = (causal && 2LL * Nq > Nk ? 2 : 1) * kNumCUs / blocks;
  if (4 * blocks > kNumCUs && (Nk < 2048 || (s < 3 && d <= 128 && Nk < 2560))) return 1;
  if (4LL * Nq > Nk && Nk < 1536 && d <= 128 && s < 10) return 1;
  return split_shares((Nk + kBc - 1) / kBc, s < 32 ? (int)s : 32);
}

size_t attn_fwd_part_bytes(int BH, int Nq, int d, int splits) {
  return (size_t)BH * ((Nq + 31) / 32) * splits * (32 * d + 64) * sizeof(float);
}

hipError_t attn_fwd_split_dispatch(const void* Q, const void* K, const void* V, void* O, float* LSE,
                                   int BH, int N, int d, int causal, float alpha, int variant,
                                   float beta, float eps, Layout lay, float* part, int splits,
                                   hipStream_t st) {
#define CASE(DD, CC, VV)                                  \
  if (d == DD && (causal != 0) == CC && variant == VV)    \
    return launch_fwd_split<DD, CC, VV>(Q, K, V, O, LSE, BH, N, alpha, beta, eps, lay, part, splits, st);
  CASE(32, false, 0) CASE(32, false, 1) CASE(32, true, 0) CASE(32, true, 1)
  CASE(64, false, 0) CASE(64, false, 1) CASE(64, true, 0) CASE(64, true, 1)
  CASE(128, false, 0) CASE(128, false, 1) CASE(128, true, 0) CASE(128, true, 1)
  CASE(256, false, 0) CASE(256, false, 1) CASE(256, true, 0) CASE(256, true, 1)
  CASE(96, false, 0) CASE(96, false, 1) CASE(96, true, 0) CASE(96, true, 1)
#undef CASE
  return hipErrorInvalidValue;
}

// Host-side dispatch used by the C ABI (api.hip).  Shapes are validated by the caller.
// The optional outputs / switches select further sets of kernels (always the bounds-checking
// instantiation), so that the plain forward carries none of their instructions.
template <int D, bool CAUSAL, int VARIANT>
static hipError_t launch_fwd_form(bool ragged, int extras, const void* Q, const void* K, const void* V, void* O, float* LSE,
                                  int BH, int N, float alpha, float beta, float eps, FwdExtras ex, Layout lay, hipStream_t st) {
  if (extras == 2) return launch_fwd<D, CAUSAL, VARIANT, true, 2>(Q, K, V, O, LSE, BH, N, alpha, beta, eps, ex, lay, st);
  if (extras) return launch_fwd<D, CAUSAL, VARIANT, true, 1>(Q, K, V, O, LSE, BH, N, alpha, beta, eps, ex, lay, st);
  // (whole-row rule: the bounds-checking kernels serve every N)
  return ragged ? launch_fwd<D, CAUSAL, VARIANT, true, 0>(Q, K, V, O, LSE, BH, N, alpha, beta, eps, ex, lay, st)
                : launch_fwd<D, CAUSAL, VARIANT, (VARIANT > 1), 0>(Q, K, V, O, LSE, BH, N, alpha, beta, eps, ex, lay, st);
}

hipError_t attn_fwd_dispatch(const void* Q, const void* K, const void* V, void* O, float* LSE,
                             int BH, int N, int d, int causal, float alpha, int variant,
                             float beta, float eps, float* O_hp, int* ones, int* fired,
                             int flags, Layout lay, hipStream_t st) {
  // flags: bit 0 = single rounding of the output, bit 1 = P-bar V in E4M3, bit 2 = guarded Alg. 3
  const int extras = (flags & 2) ? 2 : (O_hp != nullptr || ones != nullptr || fired != nullptr || flags != 0) ? 1 : 0;
  const FwdExtras ex{O_hp, ones, fired, flags & 1, (flags >> 2) & 1};
  const bool ragged = N % kBr != 0 || lay.Nk != N;
#define CASE(DD, CC)                                                                            \
  if (d == DD && (causal != 0) == CC) {                                                          \
    if (variant == 0) return launch_fwd_form<DD, CC, 0>(ragged, extras, Q, K, V, O, LSE, BH, N, alpha, beta, eps, ex, lay, st); \
    if (variant == 1) return launch_fwd_form<DD, CC, 1>(ragged, extras, Q, K, V, O, LSE, BH, N, alpha, beta, eps, ex, lay, st); \
    if (variant == kWholeRow) return launch_fwd_form<DD, CC, kWholeRow>(ragged, extras, Q, K, V, O, LSE, BH, N, alpha, beta, eps, ex, lay, st); \
    return hipErrorInvalidValue;                                                                 \
  }
  CASE(32, false) CASE(32, true) CASE(64, false) CASE(64, true) CASE(128, false) CASE(128, true)
  CASE(256, false) CASE(256, true) CASE(96, false) CASE(96, true)
#undef CASE
  return hipErrorInvalidValue;
}
