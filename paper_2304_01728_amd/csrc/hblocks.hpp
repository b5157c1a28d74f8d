// Sets of dense Hermitian blocks applied as y = sum_b R_b^T A_b R_b x: the
// macro-grid operator (one block per coarse element, Sec. 3 "Prolongation"),
// the additive Schwarz smoother (one inverse per vertex patch, Sec. 3
// "V-cycle and smoother") and the coarsest-level inverse.
//
// Storage: only the upper triangle of 32x32 tiles of each block, tiles of
// block b ordered by tile column J then tile row I <= J.  Inside a tile,
// entry (r, c) sits at [k][lane] with lane = 8 (r/4) + c/4 and
// k = 4 (r%4) + c%4, so that one wave reads a tile with 16 fully coalesced
// 64-lane loads and every lane holds a 4x4 sub-block.  A diagonal tile keeps
// only the sub-blocks on and above its diagonal (36 of 64, the diagonal 4x4
// sub-blocks whole): [k][slot] with 36 slots, 576 entries instead of 1024.
//
// Blocks that are the same matrix (a class) share one copy of its tiles and are
// applied in groups of up to eight: their local vectors are the columns of a
// matrix, and each tile is read once for the blocks of a group (four in FP32).
// Every block gets the arithmetic it would get alone, in the same order: the
// mixed-precision solutions move by 1e-9 and more with the rounding of the
// preconditioner (products of the groups on the matrix cores were as fast but
// moved them), so results do not depend on the grouping.
//
// Apply (three kernels, deterministic):
//  1. gather:  x_loc[b] = R_b x, zero-padded to 32 nt_b entries;
//  2. columns: FP64: one wave per (block, tile column J, segment of two tile
//     rows) loads both tiles before any arithmetic, writes A_IJ x_J (row
//     sums, one 32-vector per tile, laid out tile row by tile row) and
//     sum_{I<J} A_IJ^H x_I over the segment (one 32-vector per segment);
//     FP32: one wave per (block, pair of tile columns J0, J1, chunk of tile
//     rows) writes A_I,J0 x_J0 + A_I,J1 x_J1 per row I (one 32-vector per
//     two tiles) and the column sums of both columns over the chunk;
//  3. rows and scatter: eight lanes per vector entry, one per block holding it,
//     add the column partials of its column and the row partials of its row
//     (contiguous); the blocks' sums are added in a fixed order and the
//     epilogue applied (large sets: the rows first, into y_loc, then the sums
//     of these); the result can also be written into the local vector
//     of the set applied next (the smoother after a residual, the residual
//     after a smoother), whose gather is then left out.
#pragma once
#include "common.hpp"

namespace dpg {

enum { RED_SET = 0, RED_RESID = 1, RED_AXPY = 2, RED_SET_SCALED = 3 };

constexpr int kTileFull = 1024, kTileDiag = 576, kDiagSlots = 36;

// Entry offset of tile (I, J), I <= J, inside its block: the tile columns
// before J hold J (J - 1) / 2 full tiles and J diagonal tiles, and the tiles
// of column J come in order I = 0..J.
__host__ __device__ __forceinline__ int64_t tile_entry(int I, int J) {
  return (int64_t)kTileFull * ((int64_t)J * (J - 1) / 2 + I) + (int64_t)kTileDiag * J;
}

// The stored tile that A_IJ is read from (the transposed one below the diagonal): its
// first entry inside the block, which passes 2^31 bytes from 725 tile columns on in
// FP32 (the coarsest operator is one block), and its entries, in 16 slots `step` apart.
struct TileSpan {
  int64_t first;
  int entries, step;
};
__host__ __device__ __forceinline__ TileSpan tile_span(int I, int J) {
  if (J > I) return {tile_entry(I, J), kTileFull, kTileFull / 16};
  return {tile_entry(J, I), J < I ? kTileFull : kTileDiag, J < I ? kTileFull / 16 : kDiagSlots};
}

// Slot of sub-block (ra, cb), ra <= cb, in a diagonal tile: row-major order
// of the upper triangle of the 8 x 8 sub-block grid.
__host__ __device__ __forceinline__ int diag_slot(int ra, int cb) {
  return ra * 8 - ra * (ra - 1) / 2 + (cb - ra);
}

// Most tile columns of a block (row and strip descriptors hold 12-bit counts).
constexpr int kMaxTiles = 0xfff;

// Blocks of one class that are applied together: column m of a group of gw
// blocks is the local vector of its member m, row i at (base + i gw + m) (times
// the right-hand sides of a block vector, column k of a member at m nr + k).  A
// group of one block is that block's contiguous local vector.
constexpr int kMaxGroup = 8;
struct HermGroup {
  int64_t ent;               // first tile entry of the class
  int32_t base, gw, nt, pad;
};

// Units of the matrix-core apply for nr right-hand sides: chunks of 32 columns;
// chunk c covers the first cnt[c] units (units are sorted by group width).
struct ChunkMap {
  int32_t total = 0;
  int32_t cnt[kMaxGroup] = {};
};

struct HermSet {
  int nblk = 0;
  DevBuf<int4> lists;        // every list below, in one allocation
  int64_t nvec = 0;          // length of the target vector
  // units, packed: of the blocks that are a group of their own
  int64_t ntiles = 0, npart = 0, nunits = 0, nrows = 0, nloc = 0, packed = 0;
  int64_t nent = 0;          // stored tile entries
  int64_t full = 0;          // sum of n_b^2 (entries of the full blocks)
  std::vector<int32_t> n_h;  // block sizes (host)
  std::vector<int64_t> tile_off_h;   // per class: first tile index
  std::vector<int64_t> ent_off_h;    // per block: first entry of its class
  std::vector<int64_t> loc_off_h;    // per block: row 0 of its local vector
  DevList<int32_t> bn;
  DevList<int64_t> ent_off;
  // groups, widest first, and their tile rows (group, I); nrow_w[w]: how many of
  // these belong to groups of at least w blocks
  DevList<HermGroup> grp;
  DevList<int2> grow;
  int64_t nrow_w[kMaxGroup + 2] = {};
  int64_t full_grouped = 0;  // sum of n_b^2 over the blocks in groups of two and more
  DevList<int32_t> gidx;      // [nloc] vector index of each padded local row, -1 = padding
  DevList<int4> units;        // two int4 descriptors per (block, J, tile-row pair), block order
  DevList<int4> rowd;         // per (block, I): column-partial base, row-partial base,
                             // segment count | row-partial count << 12 | row step of the
                             // local vector << 24, local offset
  // the same for the FP32 apply by column pairs (strips); partials in p32;
  // sunits: blocks alone, gunits (three int4 each): up to four blocks of a group;
  // rowd, srowd: the rows of every block
  DevList<int4> sunits, gunits, srowd;
  int64_t snunits = 0, gnunits = 0, snpart = 0;
  DevList<int4> gunits64;     // three int4 per (group, J, tile-row pair), FP64; the first
  int64_t gnunits64 = 0;     // gnunits64 of groups of two and more blocks, gall64 in all
  int64_t gall64 = 0;
  // without groups (FP64): first of gunits64 and first partial slot of each block, in
  // the order of the partials, and where the last one ends; slots of the largest block
  std::vector<int64_t> unit0_h, slot0_h;
  int64_t max_slots = 0;
  DevList<int2> rowb;         // per (block, I): first partial slot of the block, its slots
  DevList<int4> tdesc;        // (representative block, I, J, 0) per stored tile (packing)
  DevList<int32_t> red_ptr;   // CSR over vector entries
  DevList<int32_t> red_ent;   // offsets into the local vectors
  DevList<int32_t> red_row;   // the same rows as 32 (tile row in rowd) + row in it
  DevBuf<double2> t64;       // tiles, FP64
  DevBuf<float2> t32;        // tiles, FP32 (mixed precision)
  DevBuf<double2> p64, xl64, yl64;   // partials and local vectors (yl: large sets, and
  DevBuf<float2> p32, xl32, yl32;    // with recomputed patches)
  Prof *prof = nullptr;      // kernel timing of the owning context
  int64_t bytes_fp64() const { return nent * 16; }
  int64_t bytes_fp32() const { return nent * 8; }
  // algorithmic entries of the blocks applied one by one: packed Hermitian
  // n(n+1)/2 per block
  int64_t packed_entries() const { return packed; }

  // idx: per block the vector index of each local row (concatenated).  cls
  // (or null: every block its own): the class of each block; the blocks of a
  // class are the same matrix and share one copy of its tiles, packed from
  // the class's first block; unless grouping is off, they are applied in
  // groups.
  void build(const std::vector<int32_t> &sizes, const std::vector<int32_t> &idx_concat,
             int64_t nvec_, bool fp64, bool fp32, Budget *bud, hipStream_t s,
             const std::vector<int32_t> *cls = nullptr, bool grouping = true);
  // Fill the tiles from dense column-major sources: block b reads
  // src[src_off[b] + map(i) + map(j) * ld[b]] where map is the identity when
  // map_off[b] < 0, else map[map_off[b] + i].
  void pack(const double2 *src, const int64_t *src_off_dev, const int32_t *ld_dev,
            const int64_t *map_off_dev, const int32_t *map_dev, hipStream_t s, int64_t tile0 = 0,
            int64_t ntile_count = -1);
};

// y <- epilogue(sum_b R_b^T A_b R_b x): RED_SET y = Ax; RED_RESID y = r - Ax;
// RED_AXPY y += theta Ax; RED_SET_SCALED y = theta Ax.
// gathered: the local vector of H already holds R_b x (a previous
// application forwarded x to H), so x is not read.  fwd: a block set on the
// same vector whose local vector receives the new y (its padding rows stay
// zero: they are zeroed at build and never written by a forward), for an
// application of fwd to y that follows with gathered = true.
template <typename T>
void herm_apply(HermSet &H, const cplx_t<T> *x, cplx_t<T> *y, const cplx_t<T> *r, int mode,
                T theta, hipStream_t s, bool gathered = false, HermSet *fwd = nullptr);

// yl = A xl for the nr interleaved columns of every block of a set without
// groups, each tile read once for all of them (FP64).  part holds npart_max >=
// max_slots entries: with fewer than npart nr the blocks are taken in ranges, and with
// fewer than max_slots nr the columns in parts; a column's sums are the same.
void launch_units_cols(HermSet &H, const double2 *xl, double2 *part, int64_t npart_max,
                       double2 *yl, int nr, hipStream_t s);

}  // namespace dpg
