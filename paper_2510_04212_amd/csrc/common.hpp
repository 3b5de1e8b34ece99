// Shared device helpers for the gfx950 attention kernels: vector types, the matrix-core
// wrappers, the LDS tile layout (macro blocks with permuted 16-byte chunks) and cross-lane exchanges.
//
// Matrix-core fragment layouts of the forward (wave64, v_mfma_f32_32x32x16_bf16; those of the backward stand at mfma16,
// D[32x32] += A[32x16] * B[16x32]; lane l, r = l & 31, h = l >> 5):
//   A operand: lane holds A[r][8h .. 8h+7]            (8 consecutive k of one row)
//   B operand: lane holds B[8h .. 8h+7][r]            (8 consecutive k of one column)
//   D / C    : register i of lane holds D[8*(i/4) + 4h + (i%4)][r]
// Because the contraction index may be permuted freely as long as A and B agree, a C-layout
// tile can be fed back as a B operand: registers 8c..8c+7 of a lane are the k-slots (h, 0..7)
// of 16-wide k-chunk c, i.e. k-slot (h, j) of chunk c  <->  tile row 16c + 8*(j/4) + 4h + (j%4).
#pragma once
#include "block_order.hpp"
#include "row_offset.hpp"
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <atomic>
#include <type_traits>
#include <utility>

typedef __bf16 bf16_t;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;

#define DEVI __device__ __forceinline__

// f(0), f(1) ... f(N - 1), each with its index as a compile-time constant
template <class F, int... I> DEVI void static_for_impl(F&& f, std::integer_sequence<int, I...>) { (f(std::integral_constant<int, I>{}), ...); }
template <int N, class F> DEVI void static_for(F&& f) { static_for_impl(f, std::make_integer_sequence<int, N>{}); }

constexpr float kLog2e = 1.4426950408889634f;

DEVI f32x16 mfma32(bf16x8 a, bf16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// ---- LDS tile layout.  A tile of R rows x D bf16 columns is cut into macro blocks of 16 rows x 32
// columns (64 bytes per row), 1024 bytes each: block (rg, cg) lies at (rg * D/32 + cg) * 1024.  Inside a
// block row r (0..15) takes 64 consecutive bytes and its four 16-byte chunks are permuted by
// chunk ^ slot_mask(r >> 2), so that (a) 16 lanes reading the same chunk of the block's 16 rows and (b) a
// transposing read of 8 rows x 64 bytes (512 consecutive bytes) both spread over all 64 LDS banks.
// Everything a fragment's address depends on besides the lane - row block, column block, tile
// buffer - adds a multiple of 1024 bytes: two per-lane registers serve every row-major fragment and
// two every column-major one, the rest is the instruction's immediate offset.  (With whole rows of
// D columns and the chunk index XOR-ed over the full row, D/16 + D/16 such registers were
// needed, and rows had to be a power of two wide: D = 96 moved and held a third more.)
template <int D> constexpr int kColBlocks = D / 32;
// Slot of chunk c of row r: c ^ slot_mask(r >> 2), slot_mask = 0, 2, 3, 1.  A ds_read_b128 serves lanes 0-3, 12-15, 20-23 and 24-27
// together (then the other half of the 32, then the upper 32), a transposing read 32 lanes: with this order neither finds two
// lanes on a bank, whichever of the fragments below they read (clocks per 1 KB and CU, measured in loops of reads only: 16-row
// fragments 4.8 with ds_read_b128 and 6.3 transposing; with 0, 1, 2, 3 8.0 and 8.0, with 0, 2, 1, 3 8.0 and 6.4; 32-row
// fragments 4.8 and 4.3 with either of the first two orders).
__host__ DEVI constexpr int slot_mask(int x) { return (((x ^ (x >> 1)) & 1) << 1) | (x >> 1); }
// D rounded up to a power of two: the lanes (and the summation tree) of one row in rowsum(dO o O)
template <int D> constexpr int kPow2D = (D == 96) ? 128 : D;
// bytes from one 16-row block of a tile to the next
template <int D> constexpr int kRowBlockBytes = kColBlocks<D> * 1024;

template <int D> struct FragOffsets {
  int row[2];               // natural read of row (lane & 31), columns 16kc + 8h .. +7, by parity of kc
  int col[2];               // transposing reads: rows 4h + 8*half + 0..3, column 32db + (lane & 31)
};
// 32-bit LDS address of a pointer into shared memory
DEVI int lds_address(const void* p) {
  typedef __attribute__((address_space(3))) const char lds_char;
  return (int)(unsigned)(unsigned long)((lds_char*)p);
}
// shared_base: LDS address of the array the tiles live in (lds_address(smem)).  The offsets are
// absolute LDS addresses, each passed through an empty asm statement: otherwise the compiler,
// rather than keep the sum in a register, re-adds the array's address (a link-time value) in front of
// every read.
template <int D> DEVI void init_frag_offsets(FragOffsets<D>& fo, int lane, int shared_base) {
  const int r = lane & 31, h = lane >> 5, i = lane & 15;
#pragma unroll
  for (int p = 0; p < 2; ++p) {
    fo.row[p] = shared_base + (r >> 4) * kRowBlockBytes<D> + (r & 15) * 64 + (((2 * p + h) ^ slot_mask((r & 15) >> 2)) << 4);
    asm volatile("" : "+v"(fo.row[p]));
  }
#pragma unroll
  for (int half = 0; half < 2; ++half) {
    const int row = 4 * h + 8 * half + (i >> 2);              // row >> 2 = h + 2 half
    const int chunk = ((lane & 16) >> 3) + ((i & 3) >> 1);
    fo.col[half] = shared_base + row * 64 + ((chunk ^ slot_mask(h + 2 * half)) << 4) + ((i & 1) << 3);
    asm volatile("" : "+v"(fo.col[half]));
  }
}
// `tile`: byte offset of the tile inside the shared-memory array (fo holds absolute addresses).
// 16-byte natural read: 8 consecutive columns (16kc + 8h ..) of row row_base + (lane & 31), row_base
// a multiple of 16: an A/B fragment whose contraction index runs along the tile's columns.
template <int D> DEVI bf16x8 lds_row8(int tile, const FragOffsets<D>& fo, int row_base, int kc) {
  typedef __attribute__((address_space(3))) const bf16x8 lds_bf16x8;
  return *reinterpret_cast<lds_bf16x8*>((unsigned long)(unsigned)(
      fo.row[kc & 1] + tile + (row_base >> 4) * kRowBlockBytes<D> + (kc >> 1) * 1024));
}
// Fragment whose contraction index runs along the tile's ROWS: k-slots (h, 0..7) of the 16-row chunk at
// row_base (a multiple of 16) are rows row_base + 8*(j/4) + 4h + (j%4), j = 0..7; the lane's own
// index selects column 32db + (lane & 31).  Two transposing reads: ds_read_b64_tr_b16 works on groups
// of 16 lanes, lane i of a group supplies the address of 4 consecutive columns (4*(i&3)..) of row
// (i>>2) and receives column i of the four rows.
template <int D> DEVI bf16x8 lds_col8(int tile, const FragOffsets<D>& fo, int row_base, int db) {
  typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
  union { struct { s16x4 lo, hi; } p; bf16x8 v; } u;
  const int at = tile + (row_base >> 4) * kRowBlockBytes<D> + db * 1024;
  u.p.lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(unsigned long)(unsigned)(fo.col[0] + at));
  u.p.hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(unsigned long)(unsigned)(fo.col[1] + at));
  return u.v;
}

// ---- the same tiles read for v_mfma_f32_16x16x32_bf16, D[16x16] += A[16x32] * B[32x16] (lane l, r = l & 15, g = l >> 4):
//   A operand: lane holds A[r][8g .. 8g+7];  B operand: B[8g .. 8g+7][r];  D / C: register i holds D[4g + i][r].
// Two C tiles one above the other (rows 0..15 and 16..31) are a B operand whose k-slot (g, j) is row
// 16*(j/4) + 4g + (j%4).  A fragment (1 KB) is one macro block of a tile and feeds as many multiplications as one of the
// 32x32x16 instruction: two of these, against 16 columns each.
//
// Why this instruction: on large grids the kernels run at the board's power limit (the same instructions on zeros take 0.7 of
// the time), and per multiplication it costs less energy, as an accumulator is read and written half as often.  Loops of
// matrix instructions on N(0,1) data (profiles/matrix_instruction_loops.txt): 32x32x16 1850 TFLOP/s at 1.80 GHz, 16x16x32 2140 at
// 2.14; with a fragment from LDS each 1444 and 1566; with 2.5 vector instructions per fragment as well 1266 and 1383.  On zeros, at 2.39
// GHz, twice as many instructions cost 2.6, 5.4 and 4 %.  The two backward kernels, us, 32x32x16
// -> this, with equal error against 64 bits:  dK/dV, causal  B4 H32 N4096 d128 922 -> 890, B1 H16 N16384 d128 1765 -> 1645,
// B2 H32/8 N2048 d128 139 -> 133, B8 H12 N1024 d64 33.7 -> 32.8, B2 H16 N2048 d96 56.3 -> 53.1, B2 H8 N2048 d256 104.5 -> 95.7,
// full  B4 H16 N4096 d128 865 -> 807, B16 H16 N2048 d64 473 -> 444;  dQ, causal  B4 H32 N4096 d128 681 -> 651, B4 H16 N1999 d128
// 98.3 -> 93.6, B4 H32 N4096 d64 371 -> 364, full  B2 H8 N2000 d256 89.8 -> 83.2.  Grids that leave a SIMD one wave are not at the
// limit and pay for the second instruction: dK/dV B1 H1 N5120 d64 44.3 -> 45.4, d128 66.6 -> 69.6, N496 H6 d128 full 18.3 -> 19.2; dQ, most
// where a score's vector work is largest against its products and no wave groups are taken, without a mask between a half and one block per
// CU: H10 N2048 d64 22.7 -> 25.2, H9 N2048 d96 28.2 -> 30.6, H17 N1024 d128 20.0 -> 21.4.  (There the vector work between the two instructions
// instead of after them gives 1 to 2 % at d64 and takes 2 % at d128, under twice as many products nothing; fragments read four slots ahead
// 0 to 1 %.)
DEVI f32x4 mfma16(bf16x8 a, bf16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}
struct TileFrags {
  int row;                  // natural read of row (lane & 15), columns 32kc + 8g .. +7
  int col[2];               // transposing read of rows 4g .. 4g+3 of a 16-row block, column 16dt + (lane & 15), by parity of dt
};
DEVI void init_tile_frags(TileFrags& fo, int lane, int shared_base) {
  const int r = lane & 15, g = lane >> 4;
  fo.row = shared_base + r * 64 + ((g ^ slot_mask(r >> 2)) << 4);
  asm volatile("" : "+v"(fo.row));                   // (absolute addresses, opaque: see init_frag_offsets)
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    fo.col[c] = shared_base + (4 * g + (r >> 2)) * 64 + (((2 * c + ((r & 3) >> 1)) ^ slot_mask(g)) << 4) + ((r & 1) << 3);
    asm volatile("" : "+v"(fo.col[c]));
  }
}
// A or B operand whose contraction index runs along the tile's columns: rows row_base + (lane & 15) (row_base a multiple of
// 16), columns 32kc + 8g .. +7.
template <int D> DEVI bf16x8 lds_row16(int tile, const TileFrags& fo, int row_base, int kc) {
  typedef __attribute__((address_space(3))) const bf16x8 lds_bf16x8;
  return *reinterpret_cast<lds_bf16x8*>((unsigned long)(unsigned)(fo.row + tile + (row_base >> 4) * kRowBlockBytes<D> + kc * 1024));
}
// Operand whose contraction index runs along the tile's ROWS: k-slot (g, j) is row row_base + 16*(j/4) + 4g + (j%4) (row_base a
// multiple of 16), the lane's own index column 16dt + (lane & 15).
template <int D> DEVI bf16x8 lds_col16(int tile, const TileFrags& fo, int row_base, int dt) {
  typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
  union { struct { s16x4 lo, hi; } p; bf16x8 v; } u;
  const int at = fo.col[dt & 1] + tile + (row_base >> 4) * kRowBlockBytes<D> + (dt >> 1) * 1024;
  u.p.lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(unsigned long)(unsigned)at);
  u.p.hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(unsigned long)(unsigned)(at + kRowBlockBytes<D>));
  return u.v;
}

// Value held by the lane 32 positions away (lane ^ 32).
DEVI float partner32(float x) {
  unsigned u = __float_as_uint(x);
  auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  // r[0] = {lower-half values in all lanes}, r[1] = {upper-half values in all lanes}
  return (threadIdx.x & 32) ? __uint_as_float(r[0]) : __uint_as_float(r[1]);
}
DEVI float max_with_partner32(float x) {
  unsigned u = __float_as_uint(x);
  auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
DEVI float sum_with_partner32(float x) {
  unsigned u = __float_as_uint(x);
  auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Sum over the two lanes 16 positions apart (lane ^ 16), and over the four that share lane & 15.
DEVI float sum_with_partner16(float x) {
  unsigned u = __float_as_uint(x);
  auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
DEVI float sum_over_groups(float x) { return sum_with_partner16(sum_with_partner32(x)); }

// Addressing of the bf16 tensors Q, K, V, O, dO, dQ, dK, dV: element (b, h, n, k) lives at
// b*sb + h*sh + n*sn + k (the last dimension is contiguous).  [B,H,N,d] contiguous is
// (H*N*d, N*d, d); [B,N,H,d] is (N*H*d, d, H*d).  float32 per-row tensors (LSE, delta) and the
// optional float32 / int32 outputs are always contiguous [B,H,N(,d)].
// Grouped-query attention: K, V, dK, dV have H / group heads with their own batch / head strides
// (sb_kv, sh_kv); query head h uses key/value head h / group.  group = 1 is ordinary attention.
// Nk: rows of K, V, dK, dV per head.  The kernels' sequence-length argument N counts the queries
// (rows of Q, O, dO, dQ, LSE, delta).  Only the bounds-checking kernel instantiations read Nk
// (the others are used for N == Nk, multiples of the block size); with Nk != N the causal mask
// is aligned at the bottom right: query r sees keys c <= r + (Nk - N).
struct Layout {
  long long sb, sh;
  int sn;
  int H;
  long long sb_kv, sh_kv;
  int group;
  int Nk;
};
// first element of query-side head bh = b*H + h
DEVI size_t head_base(const Layout& lay, int bh) {
  return (size_t)(bh / lay.H) * (size_t)lay.sb + (size_t)(bh % lay.H) * (size_t)lay.sh;
}
// first element of the key/value head that query-side head bh attends to
DEVI size_t head_base_kv(const Layout& lay, int bh) {
  return (size_t)(bh / lay.H) * (size_t)lay.sb_kv + (size_t)((bh % lay.H) / lay.group) * (size_t)lay.sh_kv;
}

// Asynchronous copy of a R-row x D bf16 tile from global memory straight into LDS
// (global_load_lds_dwordx4: no registers are involved; completion is tracked by vmcnt).
// One wave-instruction moves 64 x 16 bytes to LDS base + 16*lane, i.e. one macro block of the layout
// above: 16 rows x 64 bytes.  The chunk permutation is applied on the GLOBAL side: the lane that
// lands in slot s of row r fetches chunk s ^ slot_mask(r >> 2) of that row.  NW waves share a tile; a wave stays
// inside its own 16-row block(s), so that one per-lane offset (per row block) serves all its instructions
// and only the scalar base moves along the columns.
// The caller must execute wait_vmem() and a barrier before any wave reads the tile.
//
// The instruction is emitted through inline assembly on purpose: when the compiler itself sees a
// pending global->LDS transfer it turns every later LDS wait into "wait for everything"
// (lgkmcnt(0)) and inserts a full vmcnt(0) before the first transposing LDS read, which defeats
// both the fragment read-ahead and the overlap of the transfer with computation.  Hidden from
// its bookkeeping, the transfer only makes the compiler's own vmcnt waits more conservative
// (loads complete in order), and its completion is enforced explicitly by wait_vmem().
// A pointer the caller knows to be the same in every lane, as a scalar-register value (the tile
// loader's instruction takes its base address from scalar registers).
DEVI const bf16_t* wave_uniform(const bf16_t* p) {
  const unsigned long long u = reinterpret_cast<unsigned long long>(p);
  const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)u);
  const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)(u >> 32));
  return reinterpret_cast<const bf16_t*>(((unsigned long long)hi << 32) | lo);
}

template <int D, int R = 64, int NW = 4> struct TileLoader {
  static_assert(R == 32 || R == 64 || R == 128 || R == 256, "rows per tile");
  static constexpr int NRB = R / 16;             // 16-row blocks
  static constexpr int NCB = kColBlocks<D>;
  static constexpr int WPR = NW > NRB ? NW / NRB : 1;    // waves that share a 16-row block ...
  static constexpr int RPW = NRB > NW ? NRB / NW : 1;    // ... or row blocks per wave
  static constexpr int CPW = (NCB + WPR - 1) / WPR;  // column blocks per wave and row block
  static constexpr int NI = RPW * CPW;           // instructions per wave
  static constexpr int kBytes = R * D * 2;
  // A tile of more rows than 32-bit offsets span at the largest row stride: every wave counts its own few rows from the first of them.
  static constexpr bool FROM_WAVE = R > kMaxTileRows;
  static_assert((FROM_WAVE ? 16 * RPW : R) <= kMaxTileRows, "rows that one base address serves");
  int row, chunk;                                // per lane: first row it fetches, from the base address's row; byte offset of its chunk
  int row0_wave;                                 // row of the tile that the wave's base address stands for (scalar)
  int col0;                                      // first column block of this wave (scalar)
  int sn;                                        // distance between consecutive rows of the source, in elements
  unsigned lds_wave;                             // LDS offset of the wave's first macro block (scalar)
  DEVI void init(int tid, int row_stride) {
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rg = wave / WPR * RPW;             // first row block of this wave
    col0 = wave % WPR;
    sn = row_stride;
    row0_wave = FROM_WAVE ? rg * 16 : 0;
    row = (FROM_WAVE ? 0 : rg * 16) + (lane >> 2);
    chunk = ((lane & 3) ^ slot_mask(lane >> 4)) * 16;
    lds_wave = (unsigned)(rg * kRowBlockBytes<D> + col0 * 1024);
  }
  // A tile transfer prepared once (operands) and issued one instruction at a time, so that a caller
  // can spread it over its matrix instructions instead of issuing it in one burst.
  // RAGGED: of the source tile only the first N - row0 rows may exist: rows beyond them re-read the
  // last valid row, so that nothing is fetched out of bounds and the LDS tile holds finite values
  // everywhere (the kernels mask those rows / columns out).
  struct Pending { const bf16_t* src; unsigned base; unsigned voff[RPW]; };
  // tile starting at row `row0` of a tensor with `N` rows (row0 < N)
  template <bool RAGGED>
  DEVI Pending prepare(const char* tile, const bf16_t* tensor, int row0, int N) const {
    Pending p;
    if (FROM_WAVE) row0 = RAGGED ? min(row0 + row0_wave, N - 1) : row0 + row0_wave;
    p.src = wave_uniform(tensor + (size_t)row0 * sn + col0 * 32);
    p.base = __builtin_amdgcn_readfirstlane((unsigned)lds_address(tile)) + lds_wave;
#pragma unroll
    for (int g = 0; g < RPW; ++g) {
      const int rr = row + 16 * g;
      p.voff[g] = row_offset(RAGGED ? min(rr, N - 1 - row0) : rr, sn, chunk);
    }
    return p;
  }
  // Instruction i (0 .. NI-1) of the prepared transfer.  IMM: the column block goes into the immediate offset, which counts for
  // both addresses (m0 makes up for the difference), and two scalar additions are saved.  Pays in the pipelined forward, where a
  // wave has no issue slot to spare (there); in the backward kernels even, and 1 to 2 % slower where a SIMD has one wave.
  template <bool IMM = false> DEVI void issue(const Pending& p, int i) const {
    const int g = i / CPW, c = (i % CPW) * WPR;  // row block and column block, relative to the wave's first
    if (NCB % WPR != 0 && col0 + c >= NCB) return;
    if constexpr (IMM) {
      asm volatile("s_add_u32 m0, %0, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 offset:%4"
                   :
                   : "s"(p.base), "v"(p.voff[g]), "s"(p.src), "i"(g * kRowBlockBytes<D> + c * (1024 - 64)), "i"(c * 64)
                   : "m0", "scc");
      return;
    }
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 :
                 : "s"(p.base + (unsigned)(g * kRowBlockBytes<D> + c * 1024)), "v"(p.voff[g]), "s"(p.src + c * 32)
                 : "m0");
  }
  // the whole transfer at once
  template <bool RAGGED>
  DEVI void load_rows(const char* tile, const bf16_t* tensor, int row0, int N) const {
    const Pending p = prepare<RAGGED>(tile, tensor, row0, N);
#pragma unroll
    for (int i = 0; i < NI; ++i) issue(p, i);
  }
};

// s_waitcnt vmcnt(0): every outstanding global load (including loads into LDS) has landed.
DEVI void wait_vmem() { __builtin_amdgcn_s_waitcnt(0x0F70); }

// Marks a register value as used at this point, so that the compiler waits HERE for the load that
// produces it rather than at its first real use.  The kernels call it on their register-resident
// fragments right after the explicit wait in front of the tile loop: a compiler-generated
// "vmcnt(n)" left inside the loop (needed in its first pass only) would in every later pass also
// wait for the next tile's global->LDS transfers, which the compiler does not know of, and stall
// the wave at the start of each tile until they have landed.
template <class T> DEVI void settle(T& x) { asm volatile("" : "+v"(x)); }

// Sum of the eight bf16 values a lane holds in p, added to acc in float32 (v_dot2c_f32_bf16 with (1,1)).
DEVI float add_values(bf16x8 p, float acc) {
  bf16x2 one;
  one[0] = one[1] = (bf16_t)1.0f;
#pragma unroll
  for (int j = 0; j < 8; j += 2) {
    bf16x2 v;
    v[0] = p[j];
    v[1] = p[j + 1];
    acc = __builtin_amdgcn_fdot2_f32_bf16(v, one, acc, false);
  }
  return acc;
}

// Row sums of a fragment p of 32 rows x 16 columns in operand layout (lane (r, h): columns 8h .. 8h+7 of row r),
// added to acc[0], in float32; both lanes of a row get the whole sum.  One v_mfma_f32_16x16x32_bf16: that
// instruction takes the four 16-lane groups of p as k-slots 8g .. 8g+7 of columns (lane & 15), so that groups g and
// g + 2 hold the same rows; the selector (make_row_select) is 1 where the result's row, which lane group
// (row / 4) receives, asks for groups of its own parity, and 0 elsewhere.  A value that is not finite makes the
// sum of row r ^ 16 NaN as well (0 x inf): the caller looks for NaN and takes row_sum_apart instead.
// 16 matrix clocks; the four v_dot2c_f32_bf16 of add_values take 17 vector clocks and do not overlap with matrix
// instructions (a 32x32x16 product and eight of them: 76 clocks, with eight of any other vector instruction 40
// to 44).  (v_mfma_f32_4x4x4_16b_bf16, which keeps the rows apart, made the forward 2 to 8 % slower than either.)
DEVI bf16x8 make_row_select(int lane) {
  bf16x8 a;
#pragma unroll
  for (int j = 0; j < 8; ++j) a[j] = (bf16_t)((((lane >> 2) ^ (lane >> 4)) & 1) ? 0.f : 1.f);
  return a;
}
DEVI f32x4 add_rows(bf16x8 p, bf16x8 select, f32x4 acc) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(select, p, acc, 0, 0, 0);
}
// Row sum of the four fragments of a tile without add_rows.
DEVI float row_sum_apart(const bf16x8 (&p)[4]) {
  float s = 0.f;
#pragma unroll
  for (int c = 0; c < 4; ++c) s = add_values(p[c], s);
  return sum_with_partner32(s);
}

// x / l for the many x that share one divisor l (a row's outputs): a reciprocal of l refined by
// one Newton step, then per quotient one product and one residual correction.  The result is the
// correctly rounded quotient up to rare last-bit cases, and exact whenever l is a power of two;
// 4 instructions per quotient instead of the ~10 of a full division.  A subnormal or tiny l (the
// reciprocal instruction takes no subnormal inputs) is handled by scaling numerator and
// denominator by 2^64 first, which is exact.  l = 0 gives NaN.
struct Divisor { float l, r, scale; };
DEVI Divisor make_divisor(float l) {
  const float scale = l < 0x1p-64f ? 0x1p64f : 1.0f;
  const float ls = l * scale;
  const float r0 = __builtin_amdgcn_rcpf(ls);
  return Divisor{ls, __builtin_fmaf(__builtin_fmaf(-ls, r0, 1.0f), r0, r0), scale};
}
DEVI float divide(float x, Divisor d) {
  const float xs = x * d.scale;
  const float q = xs * d.r;
  return __builtin_fmaf(__builtin_fmaf(-q, d.l, xs), d.r, q);
}

// Output rows of a wave that holds a 32-row tile transposed in accumulator layout (lane (r,h) has,
// for its row r, the columns 32db + 8g + 4h .. +3 of every (db, g)): written straight from the
// registers, every store instruction would put 8-byte pieces into 32 different rows.  Instead the
// wave passes the tile through an LDS staging area of its own (32 rows of kStagePitch<NDB> bytes,
// wave w's area following wave w-1's from stage_wave0 on) and stores whole rows, 16 bytes per
// lane with consecutive lanes on consecutive chunks.  No barrier is involved: the area belongs to this wave alone, and the LDS executes one wave's
// accesses in order.  piece(db, g) returns the four bf16 values of that position; rows at or
// beyond rows_valid are not stored.  Needs 64 % (4 NDB) == 0.
template <int NDB> constexpr int kStagePitch = 64 * NDB + 16;   // +16: rows start 4 banks apart
template <int NDB> constexpr bool kCanStage = (64 % (4 * NDB)) == 0;
template <int NDB, class PieceF>
DEVI void store_rows_staged(char* stage_wave0, PieceF&& piece, bf16_t* dst_row0, int sn, int rows_valid, int tid) {
  static_assert(kCanStage<NDB>, "row width");
  constexpr int PITCH = kStagePitch<NDB>;
  constexpr int CPR = 4 * NDB;                  // 16-byte chunks per row
  constexpr int RPI = 64 / CPR;                 // rows per store instruction
  // The thread index goes through a copy the compiler cannot see through: every address below
  // depends on it, and computed from the kernel's own copy they would all be formed before the
  // tile loop and held in registers through it.
  asm volatile("" : "+v"(tid));
  const int lane = tid & 63;
  char* stage = stage_wave0 + (tid >> 6) * (32 * PITCH);
  const int r = lane & 31, h = lane >> 5;
#pragma unroll
  for (int db = 0; db < NDB; ++db)
#pragma unroll
    for (int g = 0; g < 4; ++g)
      *reinterpret_cast<bf16x4*>(stage + r * PITCH + (32 * db + 8 * g + 4 * h) * 2) = piece(db, g);
  typedef __attribute__((ext_vector_type(4))) unsigned u32x4;
#pragma unroll
  for (int it = 0; it < 32 / RPI; ++it) {
    const int row = it * RPI + lane / CPR, c = lane % CPR;
    const u32x4 v = *reinterpret_cast<const u32x4*>(stage + row * PITCH + c * 16);
    if (row < rows_valid) *reinterpret_cast<u32x4*>(dst_row0 + (size_t)row * sn + c * 8) = v;
  }
}

// The same for a tile in accumulator layout of 16x16 tiles: lane (r, g) has, for its rows 16n + r (n = 0, 1), the columns
// 16dt + 4g .. +3; NDT = width / 16.  piece(dt, n) returns the four bf16 values of that position.
template <int NDT, class PieceF>
DEVI void store_rows16_staged(char* stage_wave0, PieceF&& piece, bf16_t* dst_row0, int sn, int rows_valid, int tid) {
  static_assert(NDT % 2 == 0 && kCanStage<NDT / 2>, "row width");
  constexpr int PITCH = kStagePitch<NDT / 2>, CPR = 2 * NDT, RPI = 64 / CPR;
  asm volatile("" : "+v"(tid));
  const int lane = tid & 63;
  char* stage = stage_wave0 + (tid >> 6) * (32 * PITCH);
  const int r = lane & 15, g = lane >> 4;
#pragma unroll
  for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
    for (int n = 0; n < 2; ++n)
      *reinterpret_cast<bf16x4*>(stage + (16 * n + r) * PITCH + (16 * dt + 4 * g) * 2) = piece(dt, n);
#pragma unroll
  for (int it = 0; it < 32 / RPI; ++it) {
    const int row = it * RPI + lane / CPR, c = lane % CPR;
    const u32x4 v = *reinterpret_cast<const u32x4*>(stage + row * PITCH + c * 16);
    if (row < rows_valid) *reinterpret_cast<u32x4*>(dst_row0 + (size_t)row * sn + c * 8) = v;
  }
}
// ... and without staging (widths that do not divide 64 lanes): 8 bytes per lane and store.
template <int NDT, class PieceF>
DEVI void store_rows16(PieceF&& piece, bf16_t* dst_row0, int sn, int rows_valid, int lane) {
  const int r = lane & 15, g = lane >> 4;
#pragma unroll
  for (int n = 0; n < 2; ++n)
    if (16 * n + r < rows_valid) {
#pragma unroll
      for (int dt = 0; dt < NDT; ++dt)
        *reinterpret_cast<bf16x4*>(dst_row0 + (size_t)(16 * n + r) * sn + 16 * dt + 4 * g) = piece(dt, n);
    }
}

// Issue-order hints for one scheduling region (basic block) that holds N matrix instructions,
// each fed by PER LDS fragment reads: the reads are issued AHEAD matrix instructions before
// their use, so that LDS latency is covered by matrix-core work instead of stalling the wave.
// (sched_group_barrier masks: 0x008 = MFMA, 0x100 = LDS read.)
template <int N, int PER, int AHEAD_> DEVI void sched_reads_ahead_of_mfma() {
  static_assert(PER == 1 || PER == 2, "PER");
  constexpr int AHEAD = AHEAD_ < N ? AHEAD_ : N;
  __builtin_amdgcn_sched_group_barrier(0x100, AHEAD * PER, 0);
#pragma unroll
  for (int i = 0; i < N - AHEAD; ++i) {
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    __builtin_amdgcn_sched_group_barrier(0x100, PER, 0);
  }
#pragma unroll
  for (int i = 0; i < AHEAD; ++i) __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
}

// Work-group index remap: consecutive hardware work-group ids go round-robin over the 8 XCDs
// (each with its own L2).  Give every XCD a contiguous range of logical ids so that the
// work-groups sharing one head's K/V run on the same L2.  Only applied when the grid is a
// multiple of 8 (otherwise the map would not be a bijection).
DEVI int xcd_remap(int id, int n) {
  if ((n & 7) != 0) return id;
  return (id & 7) * (n >> 3) + (id >> 3);
}

// Logical id of a work-group: with an order table (block_order.hpp) the s-th work-group of an XCD
// takes item pos[s] of the XCD's contiguous share of the grid, otherwise the plain remap above.
// The table is a kernel argument, i.e. read with scalar loads.
DEVI int logical_wg(const BlockOrder& ord, int id, int n) {
  if (ord.n == 0) return xcd_remap(id, n);
  return (id & 7) * (n >> 3) + ord.pos[id >> 3];
}

// Rotation of the causal block order of one head, for grids small enough to be resident all at
// once or nearly so (at most `capacity` work-groups, which callers set to 1.5x what the chip
// holds of that kernel: measured, the rotation wins up to one and a half rounds of work-groups;
// from two rounds on, plain heavy-first order does better and is kept).  Blocks of one head differ in
// work by up to nblk : 1.  Work-groups are handed to the CUs of an XCD round-robin, so with a
// fixed heavy-to-light order the j-th work-group of a CU always lands on the same weight class;
// rotating the order by a different amount for each "lap" over the XCD's 32 CUs gives every CU
// a mix.  The rotation depends on the head only, so every block is still visited once.
DEVI int small_grid_rotation(int bh, int nblk, int grid, int capacity) {
  if (grid > capacity || (grid & 7) != 0) return 0;
  const int first = (bh * nblk) % (grid >> 3);     // dispatch sequence number of the head's first block inside its XCD
  return (3 * (first >> 5)) % nblk;
}

// ---- host side of the order table --------------------------------------------------------------

// Work-groups of `kern` (`threads` threads, `smem` bytes of dynamic LDS) that a compute unit holds at
// once; asked of the runtime once per kernel instantiation.
template <class KernT>
static int resident_per_cu(KernT kern, int smem, std::atomic<int>& cached, int threads = 256) {
  int r = cached.load(std::memory_order_relaxed);
  if (r == 0) {
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&r, reinterpret_cast<const void*>(kern), threads, smem) != hipSuccess || r <= 0) {
      (void)hipGetLastError();   // the answer only steers the block order: not an error of the launch that follows
      r = 1;
    }
    cached.store(r, std::memory_order_relaxed);
  }
  return r;
}

// The table for a causal grid of `grid` one-block work-groups with `nblk` blocks per head; empty
// (n = 0) unless the grid is at most `max_grid`, a multiple of 8, every XCD's share holds whole
// heads and fits the table.  The last table is kept (one per calling thread and kernel
// instantiation), so a training loop computes it once.
struct OrderCache {
  int grid = -1, nblk = -1, resident = -1;
  BlockOrder ord;
};
static const BlockOrder kNoOrder{};
static const BlockOrder& small_grid_order(OrderCache& c, int grid, int nblk, int resident, long long max_grid) {
  if (c.grid != grid || c.nblk != nblk || c.resident != resident) {
    c.grid = grid; c.nblk = nblk; c.resident = resident;
    c.ord.n = 0;
    if ((grid & 7) == 0 && grid <= max_grid) fill_block_order(c.ord, grid >> 3, nblk, resident);
  }
  return c.ord;
}
