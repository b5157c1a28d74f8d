// Hermitian block sets: packing and apply kernels (see hblocks.hpp).
#include <algorithm>
#include <map>

#include "block.hpp"
#include "hblocks.hpp"
#include "kernels.hpp"

namespace dpg {
namespace {

template <typename C> __device__ __forceinline__ C czero() {
  C r;
  r.x = 0;
  r.y = 0;
  return r;
}

// Cross-lane moves inside rows of 16 lanes (DPP): quad_perm [1,0,3,2],
// quad_perm [2,3,0,1], the mirror inside each group of 8 lanes, and the rotation
// by 8 lanes.
constexpr int kDppXor1 = 0xB1, kDppXor2 = 0x4E, kDppHalfMirror = 0x141, kDppRor8 = 0x128;

template <int CTRL> __device__ __forceinline__ float dpp(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v),
                                                               CTRL, 0xF, 0xF, false));
}
template <int CTRL> __device__ __forceinline__ double dpp(double v) {
  int2 i = __builtin_bit_cast(int2, v);
  i.x = __builtin_amdgcn_update_dpp(0, i.x, CTRL, 0xF, 0xF, false);
  i.y = __builtin_amdgcn_update_dpp(0, i.y, CTRL, 0xF, 0xF, false);
  return __builtin_bit_cast(double, i);
}
template <int CTRL, typename C> __device__ __forceinline__ C dpp_c(C v) {
  C r;
  r.x = dpp<CTRL>(v.x);
  r.y = dpp<CTRL>(v.y);
  return r;
}
template <typename C> __device__ __forceinline__ C csel(bool c, C a, C b) {
  C r;
  r.x = c ? a.x : b.x;
  r.y = c ? a.y : b.y;
  return r;
}

// Reduce-scatter of four row values over the 8 lanes cb = 0..7 of a group:
// lanes cb and cb^1 return the full sum of row cb/2.  Three exchange rounds
// (partners 7-cb, cb^2, cb^1), each moving one value per lane after the
// first, which moves two.
template <typename C> __device__ __forceinline__ C rowsum_scatter(const C rs[4], int cb) {
  const bool lo = cb < 4;
  C k0 = csel(lo, rs[0], rs[2]), k1 = csel(lo, rs[1], rs[3]);
  const C s0 = csel(lo, rs[2], rs[0]), s1 = csel(lo, rs[3], rs[1]);
  k0 = cadd(k0, dpp_c<kDppHalfMirror>(s0));
  k1 = cadd(k1, dpp_c<kDppHalfMirror>(s1));
  const bool b1 = cb & 2;
  C k = csel(b1, k1, k0);
  k = cadd(k, dpp_c<kDppXor2>(csel(b1, k0, k1)));
  return cadd(k, dpp_c<kDppXor1>(k));
}

// The dwords of a pair (p, q) with their rows of 16 lanes (halves of 32) exchanged:
// the sum of the two results is p over both rows of a pair in the even row, q in the
// odd one.
template <int ROW> __device__ __forceinline__ void swap_rows(uint32_t &p, uint32_t &q) {
  if constexpr (ROW == 16) {
    const auto r = __builtin_amdgcn_permlane16_swap(p, q, false, false);
    p = r[0];
    q = r[1];
  } else {
    const auto r = __builtin_amdgcn_permlane32_swap(p, q, false, false);
    p = r[0];
    q = r[1];
  }
}
template <int ROW> __device__ __forceinline__ float swap_sum(float p, float q) {
  uint32_t a = __float_as_uint(p), b = __float_as_uint(q);
  swap_rows<ROW>(a, b);
  return __uint_as_float(a) + __uint_as_float(b);
}
template <int ROW> __device__ __forceinline__ double swap_sum(double p, double q) {
  uint32_t al = __double2loint(p), ah = __double2hiint(p), bl = __double2loint(q),
           bh = __double2hiint(q);
  swap_rows<ROW>(al, bl);
  swap_rows<ROW>(ah, bh);
  return __hiloint2double(ah, al) + __hiloint2double(bh, bl);
}

// Sums of four column values over the lanes ra = 0..7 (8, 16, 32 lanes apart, in
// that order): lane ra returns that of column col_of(ra).  Each exchange halves the
// values a lane carries on, and stays in the vector unit (DPP, row swaps).  Four sums
// one by one through LDS permutations, 12 exchanges instead of 4: solves at 16^3,
// p = 3 24.6 / 23.6 ms, 24^3, p = 4 mixed 108.1 / 104.8.
__device__ __forceinline__ int col_of(int ra) { return 2 * (ra & 1) + (ra >> 1 & 1); }
template <typename C> __device__ __forceinline__ C colsum_scatter(const C v[4], int ra) {
  const bool odd = ra & 1;
  C k0 = csel(odd, v[2], v[0]), k1 = csel(odd, v[3], v[1]);
  const C s0 = csel(odd, v[0], v[2]), s1 = csel(odd, v[1], v[3]);
  k0 = cadd(k0, dpp_c<kDppRor8>(s0));
  k1 = cadd(k1, dpp_c<kDppRor8>(s1));
  C k;
  k.x = swap_sum<16>(k0.x, k1.x);
  k.y = swap_sum<16>(k0.y, k1.y);
  k.x = swap_sum<32>(k.x, k.x);
  k.y = swap_sum<32>(k.y, k.y);
  return k;
}

// Tile entries are read once per application: non-temporal loads keep them
// from displacing the x entries and partials in the caches.
__device__ __forceinline__ double2 ld_nt(const double2 *p) {
  typedef double v2 __attribute__((ext_vector_type(2)));
  const v2 v = __builtin_nontemporal_load(reinterpret_cast<const v2 *>(p));
  return make_double2(v.x, v.y);
}
__device__ __forceinline__ float2 ld_nt(const float2 *p) {
  typedef float v2 __attribute__((ext_vector_type(2)));
  const v2 v = __builtin_nontemporal_load(reinterpret_cast<const v2 *>(p));
  return make_float2(v.x, v.y);
}

template <typename C> __device__ __forceinline__ void load_tile(const C *__restrict__ tp, C t[16]) {
#pragma unroll
  for (int k = 0; k < 16; ++k) t[k] = ld_nt(tp + k * 64);
}

// A tile by its lane's first entry and the stride between its 16 entries: 64
// for a full tile, 36 for a diagonal one, whose lanes below the diagonal
// read slot 0 (in range) and are zeroed by mask_lower once the data is
// needed.  One code path for both kinds: behind a branch, the compiler made
// the loads of either kind wait for those of the other.
template <typename C>
__device__ __forceinline__ void load_strided(const C *__restrict__ tp, int st, C t[16]) {
#pragma unroll
  for (int k = 0; k < 16; ++k) t[k] = ld_nt(tp + k * st);
}
template <typename C> __device__ __forceinline__ void mask_lower(bool keep, C t[16]) {
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    t[k].x = keep ? t[k].x : 0;
    t[k].y = keep ? t[k].y : 0;
  }
}

// Row sums of one tile into its partial slot; column sums accumulated where
// off holds: every sub-block of an off-diagonal tile, the sub-blocks strictly
// above the diagonal of a diagonal tile (their conjugate transposes are the
// sub-blocks below it, which are not stored).
template <typename C>
__device__ __forceinline__ void do_tile(const C t[16], const C xJ[4], const C *xr, bool off,
                                        int ra, int cb, C cacc[4], C *__restrict__ slot) {
  C rs[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    C a;
    a.x = 0;
    a.y = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) a = cfma(t[4 * i + j], xJ[j], a);
    rs[i] = a;
  }
  if (off) {
    C xI[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) xI[i] = xr[4 * ra + i];
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int i = 0; i < 4; ++i) cacc[j] = cfmaconj(t[4 * i + j], xI[i], cacc[j]);
  }
  const C v = rowsum_scatter(rs, cb);
  if (!(cb & 1)) slot[4 * ra + (cb >> 1)] = v;
}

// Tile columns are cut into segments of at most kSeg tiles, one wave each.
// Two tiles, both loaded before any arithmetic, stream fastest: longer
// segments leave only one tile in flight while the other is being used.
constexpr int kSeg = 2;

// Column-sum slots of a block: column J has ceil((J+1)/kSeg) segment slots;
// colbase(J) = 32 sum_{j=1..J} ceil(j/kSeg).
__host__ __device__ __forceinline__ int64_t colbase(int J) {
  const int64_t q = J / kSeg, r = J % kSeg;
  return 32 * (kSeg * q * (q + 1) / 2 + r * (q + 1));
}

// offset of the row-sum slot (I, J), I <= J, inside the row partials of a block
__host__ __device__ __forceinline__ int64_t row_slot(int nt, int I, int J) {
  return ((int64_t)I * nt - (int64_t)I * (I - 1) / 2 + (J - I)) * 32;
}

// The FP32 apply (k_strips) takes tile columns in pairs, "strips" (J0 = 2 s,
// J1 = 2 s + 1; the last strip of a block with an odd tile count has one
// column), whose tile rows 0..J1 are cut into chunks of at most kChunk rows,
// one wave each.  Per row I the wave loads tiles (I, J0) and (I, J1) and
// writes their row sums as one 32-vector (slot (I, s)); the column sums of
// both columns accumulate in registers over the chunk (one slot per column
// and chunk).  Partials per 1024-entry tile: 16 + 8 entries instead of the
// 32 + 16 of the segments above (and the x entries of a row once per two
// tiles), which pays in FP32, where they weigh twice as much against the
// tiles; FP64 streams its 16 KB tiles faster as segments.
constexpr int kChunk = 4;
constexpr int kStripBlocks = 4;   // blocks of a group per wave (k_strips_grp)

// Row-sum slots of a block with nt tile columns (ns = ceil(nt / 2) strips):
// row I is covered by the strips s >= I / 2, its slots are contiguous, and
// rows come in order: slot(I, s) = I ns - floor((I - 1)^2 / 4) + s - I / 2.
__host__ __device__ __forceinline__ int64_t strip_row_slot(int ns, int I, int s) {
  return (int64_t)I * ns - (int64_t)(I - 1) * (I - 1) / 4 + s - I / 2;
}
__host__ __forceinline__ int64_t strip_row_slots(int nt) {
  return (int64_t)nt * ((nt + 1) / 2) - (int64_t)(nt - 1) * (nt - 1) / 4;
}
__host__ __forceinline__ int strip_rows(int nt, int s) { return std::min(2 * s + 2, nt); }
__host__ __forceinline__ int strip_chunks(int nt, int s) {
  return (strip_rows(nt, s) + kChunk - 1) / kChunk;
}

template <typename T>
__global__ __launch_bounds__(256) void k_gather_x(int64_t nloc, const int32_t *__restrict__ gidx,
                                                  const cplx_t<T> *__restrict__ x,
                                                  cplx_t<T> *__restrict__ xl) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= nloc) return;
  const int32_t g = gidx[i];
  cplx_t<T> v;
  v.x = 0;
  v.y = 0;
  if (g >= 0) v = x[g];
  xl[i] = v;
}

// One wave per (block, tile column J, pair of tile rows I0, I0 + 1 <= J).  The
// unit's descriptor (two int4, see HermSet::build) holds every address the
// wave needs and is read with scalar loads (the wave index is made uniform),
// so the tile loads follow it at once and the x loads come after them (with
// x first, the compiler waited for x, and a vector-loaded descriptor, before
// issuing the tiles).  The x entries of the two tile rows are staged in LDS
// (wave-private), which keeps registers for the tiles and the vector memory
// queue for tile data.
template <typename T>
__global__ __launch_bounds__(256) void k_units(const cplx_t<T> *__restrict__ tiles,
                                               const int4 *__restrict__ units, int64_t nunits,
                                               const cplx_t<T> *__restrict__ xloc,
                                               cplx_t<T> *__restrict__ part) {
  static_assert(kSeg == 2, "k_units handles segments of two tile rows");
  using C = cplx_t<T>;
  __shared__ C xs[4][kSeg * 32];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // workgroup g runs on XCD g % 8: each XCD takes a contiguous range of
  // units (the grid is a multiple of 8; workgroups past the end exit)
  const int64_t per = gridDim.x / 8, wg = (int64_t)(blockIdx.x % 8) * per + blockIdx.x / 8;
  const int64_t wv = wg * 4 + wave;
  if (wv >= nunits) return;
  const int lane = threadIdx.x & 63, ra = lane >> 3, cb = lane & 7;
  const int4 d0 = units[2 * wv], d1 = units[2 * wv + 1];
  const int64_t ent = (int64_t)(uint32_t)d0.x | ((int64_t)d0.y << 32);
  // a one-tile segment is a diagonal tile; of two, the first is off-diagonal
  const bool two = d1.w & 1, off0 = d1.w & 2, off1 = d1.w & 4;
  const bool upper = ra <= cb, strict = ra < cb;
  const C *tp = tiles + ent;
  C t0[16], t1[16], xJ[4], cacc[4];
  // tiles first, then x (lanes past the unit's rows read its last row); all
  // of them arrive before any arithmetic
  const int ds = upper ? diag_slot(ra, cb) : 0;
  load_strided(tp + (off0 ? lane : ds), off0 ? 64 : kDiagSlots, t0);
  if (two) load_strided(tp + kTileFull + (off1 ? lane : ds), off1 ? 64 : kDiagSlots, t1);
  const int nx = 32 * (1 + two);
  const C v = xloc[d0.z + min(lane, nx - 1)];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    xJ[j] = xloc[d0.w + 4 * cb + j];
    cacc[j].x = 0;
    cacc[j].y = 0;
  }
  C *xw = xs[wave];
  C w;
  w.x = lane < nx ? v.x : 0;
  w.y = lane < nx ? v.y : 0;
  xw[lane] = w;
  wave_lds_fence();
  if (!off0) mask_lower(upper, t0);
  if (two && !off1) mask_lower(upper, t1);
  do_tile(t0, xJ, xw, off0 || strict, ra, cb, cacc, part + d1.x);
  if (two) do_tile(t1, xJ, xw + 32, off1 || strict, ra, cb, cacc, part + d1.x + d1.y);
  const C cs = colsum_scatter(cacc, ra);
  if (ra < 4) part[d1.z + 4 * cb + col_of(ra)] = cs;
}

// The units of a group's blocks (a group's local vectors are interleaved: row i
// of block m at i gw + m): both tiles are loaded once for all blocks, from a
// cache except for the first group of its class, and every block gets the
// arithmetic of k_units in the same order, so the partials are bit for bit the
// same.  Bound by the vector units and the cross-lane sums, about 1000 cycles per
// block and tile against 7300 for the tile's 16 KB at a SIMD's share of the HBM
// rate.  The x entries of the next block are loaded while one is multiplied.
// The right-hand sides k0 .. k0 + q - 1 of a block alone are taken like the blocks of
// a group (column k at i nr + k), with the partials of the blocks from slot0 on; its
// tiles are read once per application (NT: past the caches).
template <typename T, bool NT>
__global__ __launch_bounds__(256, 2) void k_units_grp(const cplx_t<T> *__restrict__ tiles,
                                                      const int4 *__restrict__ units,
                                                      int64_t nunits, int nr, int k0, int q,
                                                      int64_t slot0,
                                                      const cplx_t<T> *__restrict__ xloc,
                                                      cplx_t<T> *__restrict__ part) {
  using C = cplx_t<T>;
  __shared__ C xs[4][kSeg * 32];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t per = gridDim.x / 8, wg = (int64_t)(blockIdx.x % 8) * per + blockIdx.x / 8;
  const int64_t wv = wg * 4 + wave;
  if (wv >= nunits) return;
  const int lane = threadIdx.x & 63, ra = lane >> 3, cb = lane & 7;
  const int4 d0 = units[3 * wv], d1 = units[3 * wv + 1], d2 = units[3 * wv + 2];
  const int each = d2.x, ld = (d1.w >> 8) * nr, gw = NT ? q : ld;
  const int64_t ent = (int64_t)(uint32_t)d0.x | ((int64_t)d0.y << 32);
  if (NT) {   // slots of the columns of the blocks before this one
    part += (int64_t)d2.y * (q - 1) - slot0 * q;
    xloc += k0;
  }
  const bool two = d1.w & 1, off0 = d1.w & 2, off1 = d1.w & 4;
  const bool upper = ra <= cb, strict = ra < cb;
  const C *tp = tiles + ent;
  C t0[16], t1[16], xJ[4];
  const int ds = upper ? diag_slot(ra, cb) : 0;
  const int s0 = off0 ? 64 : kDiagSlots, s1 = off1 ? 64 : kDiagSlots;
  const C *p0 = tp + (off0 ? lane : ds), *p1 = tp + kTileFull + (off1 ? lane : ds);
#pragma unroll
  for (int k = 0; k < 16; ++k) t0[k] = NT ? ld_nt(p0 + k * s0) : p0[k * s0];
  if (two) {
#pragma unroll
    for (int k = 0; k < 16; ++k) t1[k] = NT ? ld_nt(p1 + k * s1) : p1[k * s1];
  }
  const int nx = 32 * (1 + two);
  const C *xi = xloc + (int64_t)d0.z * nr + min(lane, nx - 1) * ld;
  const C *xj = xloc + (int64_t)d0.w * nr + 4 * cb * ld;
  C v = xi[0];
#pragma unroll
  for (int j = 0; j < 4; ++j) xJ[j] = xj[j * ld];
  if (!off0) mask_lower(upper, t0);
  if (two && !off1) mask_lower(upper, t1);
  C *xw = xs[wave];
#pragma unroll 1
  for (int m = 0; m < gw; ++m) {
    C w, cacc[4], xc[4];
    w.x = lane < nx ? v.x : 0;
    w.y = lane < nx ? v.y : 0;
    wave_lds_fence();   // the block before has read its x
    xw[lane] = w;
    wave_lds_fence();
    const int mn = min(m + 1, gw - 1);
    v = xi[mn];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      xc[j] = xJ[j];
      xJ[j] = xj[j * ld + mn];
      cacc[j] = czero<C>();
    }
    C *pm = part + (int64_t)m * each;
    do_tile(t0, xc, xw, off0 || strict, ra, cb, cacc, pm + d1.x);
    if (two) do_tile(t1, xc, xw + 32, off1 || strict, ra, cb, cacc, pm + d1.x + d1.y);
    const C cs = colsum_scatter(cacc, ra);
    if (ra < 4) pm[d1.z + 4 * cb + col_of(ra)] = cs;
  }
}

// One wave per (block, strip s, chunk of tile rows [Ia, Ib)).  The unit's
// descriptor (two int4, see HermSet::build) is read with scalar loads (the
// wave index is made uniform).  Each row step issues the loads of both tiles,
// then the x entries of the row, before any arithmetic.  A diagonal tile and
// an absent one (row J1 of column J0, the second column of a one-column
// strip) are read through the diagonal tile's 36-slot layout at an address
// inside it, and masked: one load path for every kind (behind branches the
// compiler made the loads of one kind wait for the other's).
template <typename T>
__global__ __launch_bounds__(256) void k_strips(const cplx_t<T> *__restrict__ tiles,
                                               const int4 *__restrict__ units, int64_t nunits,
                                               const cplx_t<T> *__restrict__ xloc,
                                               cplx_t<T> *__restrict__ part) {
  using C = cplx_t<T>;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // workgroup g runs on XCD g % 8: each XCD takes a contiguous range of
  // units (the grid is a multiple of 8; workgroups past the end exit)
  const int64_t per = gridDim.x / 8, wg = (int64_t)(blockIdx.x % 8) * per + blockIdx.x / 8;
  const int64_t wv = wg * 4 + wave;
  if (wv >= nunits) return;
  const int lane = threadIdx.x & 63, ra = lane >> 3, cb = lane & 7;
  const int4 d0 = units[2 * wv], d1 = units[2 * wv + 1];
  const int64_t ent = (int64_t)(uint32_t)d0.x | ((int64_t)d0.y << 32);
  const int J0 = d1.x & 0xffff, nt = d1.x >> 16, J1 = J0 + 1;
  const int Ia = d1.y & 0xffff, Ib = d1.y >> 16;
  const bool two = J1 < nt;
  const int ns = (nt + 1) >> 1, s = J0 >> 1;
  const bool upper = ra <= cb, strict = ra < cb;
  const int ds = upper ? diag_slot(ra, cb) : 0;
  const C *t0 = tiles + ent;                                   // tile (0, J0)
  const C *t1 = two ? t0 + (int64_t)kTileFull * J0 + kTileDiag : t0;   // tile (0, J1)
  const C *xb = xloc + d0.z;
  C *rp = part + d0.w;
  C xJ0[4], xJ1[4], c0[4], c1[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    xJ0[j] = xb[32 * J0 + 4 * cb + j];
    xJ1[j] = xb[32 * (two ? J1 : J0) + 4 * cb + j];
    c0[j].x = 0;
    c0[j].y = 0;
    c1[j].x = 0;
    c1[j].y = 0;
  }
#pragma unroll 1
  for (int I = Ia; I < Ib; ++I) {
    // (I, J0): full for I < J0, diagonal for I == J0, absent for I == J1;
    // (I, J1): full for I < J1, diagonal for I == J1, absent without J1
    const bool fa = I < J0, fb = two && I < J1;
    const bool ka = fa || (I == J0 && upper), kb = fb || (two && I == J1 && upper);
    const C *pa = fa ? t0 + (int64_t)kTileFull * I + lane : t0 + (int64_t)kTileFull * J0 + ds;
    const C *pb = fb ? t1 + (int64_t)kTileFull * I + lane
                     : two ? t1 + (int64_t)kTileFull * J1 + ds : t0 + (int64_t)kTileFull * J0 + ds;
    C ta[16], tb[16], xI[4];
    load_strided(pa, fa ? 64 : kDiagSlots, ta);
    load_strided(pb, fb ? 64 : kDiagSlots, tb);
#pragma unroll
    for (int i = 0; i < 4; ++i) xI[i] = xb[32 * I + 4 * ra + i];
    mask_lower(ka, ta);
    mask_lower(kb, tb);
    C rs[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      C a;
      a.x = 0;
      a.y = 0;
#pragma unroll
      for (int j = 0; j < 4; ++j) a = cfma(ta[4 * i + j], xJ0[j], a);
#pragma unroll
      for (int j = 0; j < 4; ++j) a = cfma(tb[4 * i + j], xJ1[j], a);
      rs[i] = a;
    }
    // column sums: every sub-block of a full tile, the sub-blocks strictly
    // above the diagonal of a diagonal one (masked entries are zero)
    C xa[4], xbb[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      xa[i] = csel(fa || strict, xI[i], czero<C>());
      xbb[i] = csel(fb || strict, xI[i], czero<C>());
    }
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        c0[j] = cfmaconj(ta[4 * i + j], xa[i], c0[j]);
        c1[j] = cfmaconj(tb[4 * i + j], xbb[i], c1[j]);
      }
    const C v = rowsum_scatter(rs, cb);
    if (!(cb & 1)) rp[32 * strip_row_slot(ns, I, s) + 4 * ra + (cb >> 1)] = v;
  }
  const C s0 = colsum_scatter(c0, ra), s1 = colsum_scatter(c1, ra);
  if (ra < 4) {
    part[d1.z + 4 * cb + col_of(ra)] = s0;
    if (two) part[d1.w + 4 * cb + col_of(ra)] = s1;
  }
}

// The strips of up to kStripBlocks equal blocks (a group's local vectors are
// interleaved: row i of block m at i gw + m): each pair of tiles is loaded once
// for all of them, from a cache except for the first group of its class, and
// every block gets the arithmetic of k_strips in the same order, so the partials
// are bit for bit the same.  Bound by the vector units: at 24^3, p = 4 (36 TFLOP/s of
// products, of 78.6) they issue in 81 % of the busy cycles of a compute unit, and a wave
// waits for memory in 17 % of its time; the tiles come from L2 for 66 % of the requests
// and from memory at 0.8 TB/s (counters).  Of some 300 instructions per pair of tiles and
// block 256 are the products.  Four blocks (16 column sums and 16 x entries each) fill
// the 256 registers of two waves per SIMD.  The next tile row's x comes through LDS,
// loaded a row ahead (one load per block and row, waited for at its use, 68.6 -> 66.5 ms
// of a solve).
template <typename T>
__global__ __launch_bounds__(256, 2) void k_strips_grp(const cplx_t<T> *__restrict__ tiles,
                                                       const int4 *__restrict__ units,
                                                       int64_t nunits,
                                                       const cplx_t<T> *__restrict__ xloc,
                                                       cplx_t<T> *__restrict__ part) {
  using C = cplx_t<T>;
  constexpr int G = kStripBlocks, XR = 32 * G + 2 * 8;   // x of a tile row, padded per four rows
  __shared__ C xs[4][XR];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t per = gridDim.x / 8, wg = (int64_t)(blockIdx.x % 8) * per + blockIdx.x / 8;
  const int64_t wv = wg * 4 + wave;
  if (wv >= nunits) return;
  const int lane = threadIdx.x & 63, ra = lane >> 3, cb = lane & 7;
  const int4 d0 = units[3 * wv], d1 = units[3 * wv + 1];
  const int each = units[3 * wv + 2].x;
  const int64_t ent = (int64_t)(uint32_t)d0.x | ((int64_t)d0.y << 32);
  const int cnt = d0.w & 0xff, gw = d0.w >> 8;
  const int J0 = d1.x & 0xffff, nt = d1.x >> 16, J1 = J0 + 1;
  const int Ia = d1.y & 0xffff, Ib = d1.y >> 16;
  const bool two = J1 < nt;
  const int ns = (nt + 1) >> 1, s = J0 >> 1;
  const bool upper = ra <= cb, strict = ra < cb;
  const int ds = upper ? diag_slot(ra, cb) : 0;
  const C *t0 = tiles + ent;                                   // tile (0, J0)
  const C *t1 = two ? t0 + (int64_t)kTileFull * J0 + kTileDiag : t0;   // tile (0, J1)
  const C *xb = xloc + d0.z;
  C xJ0[G][4], xJ1[G][4], c0[G][4], c1[G][4];
#pragma unroll
  for (int m = 0; m < G; ++m) {
    const int mc = min(m, cnt - 1);   // blocks past cnt repeat the last one, unused
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      xJ0[m][j] = xb[(32 * J0 + 4 * cb + j) * gw + mc];
      xJ1[m][j] = xb[(32 * (two ? J1 : J0) + 4 * cb + j) * gw + mc];
      c0[m][j] = czero<C>();
      c1[m][j] = czero<C>();
    }
  }
  // x of the blocks' next tile row: entries lane and lane + 64 of (row, block)
  C *const xw = xs[wave];
  C xn[2];
  auto load_x = [&](int I) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int e = lane + 64 * h;
      xn[h] = xb[(32 * I + e / G) * gw + min(e % G, cnt - 1)];
    }
  };
  static_assert(32 * G == 128, "two x entries per lane");
  load_x(Ia);
#pragma unroll 1
  for (int I = Ia; I < Ib; ++I) {
    wave_lds_fence();   // the row before has been read
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int e = lane + 64 * h;
      xw[e + 2 * (e / (4 * G))] = xn[h];
    }
    wave_lds_fence();
    const bool fa = I < J0, fb = two && I < J1;
    const bool ka = fa || (I == J0 && upper), kb = fb || (two && I == J1 && upper);
    const C *pa = fa ? t0 + (int64_t)kTileFull * I + lane : t0 + (int64_t)kTileFull * J0 + ds;
    const C *pb = fb ? t1 + (int64_t)kTileFull * I + lane
                     : two ? t1 + (int64_t)kTileFull * J1 + ds : t0 + (int64_t)kTileFull * J0 + ds;
    const int sa = fa ? 64 : kDiagSlots, sb = fb ? 64 : kDiagSlots;
    C ta[16], tb[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) ta[k] = pa[k * sa];
#pragma unroll
    for (int k = 0; k < 16; ++k) tb[k] = pb[k * sb];
    load_x(min(I + 1, Ib - 1));
    mask_lower(ka, ta);
    mask_lower(kb, tb);
#pragma unroll
    for (int m = 0; m < G; ++m) {
      if (m >= cnt) break;
      C xI[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) xI[i] = xw[(4 * G + 2) * ra + G * i + m];
      C rs[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        C a = czero<C>();
#pragma unroll
        for (int j = 0; j < 4; ++j) a = cfma(ta[4 * i + j], xJ0[m][j], a);
#pragma unroll
        for (int j = 0; j < 4; ++j) a = cfma(tb[4 * i + j], xJ1[m][j], a);
        rs[i] = a;
      }
      C xa[4], xbb[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        xa[i] = csel(fa || strict, xI[i], czero<C>());
        xbb[i] = csel(fb || strict, xI[i], czero<C>());
      }
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          c0[m][j] = cfmaconj(ta[4 * i + j], xa[i], c0[m][j]);
          c1[m][j] = cfmaconj(tb[4 * i + j], xbb[i], c1[m][j]);
        }
      const C v = rowsum_scatter(rs, cb);
      if (!(cb & 1))
        part[d1.w + m * each + 32 * strip_row_slot(ns, I, s) + 4 * ra + (cb >> 1)] = v;
    }
  }
  const int nc = (min(2 * s + 2, nt) + kChunk - 1) / kChunk;   // chunks of the strip
#pragma unroll
  for (int m = 0; m < G; ++m) {
    if (m >= cnt) break;
    const C s0 = colsum_scatter(c0[m], ra), s1 = colsum_scatter(c1[m], ra);
    if (ra < 4) {
      C *pc = part + d1.z + m * each + 4 * cb + col_of(ra);
      pc[0] = s0;
      if (two) pc[32 * nc] = s1;
    }
  }
}

// Sum of the partial slots of row r of a tile row: the column sums of the
// segments (or strip chunks) of its tile column, then the row sums of its tiles;
// eight loads in flight per lane (a row of a 24-tile block sums 25 slots), summed
// in a fixed order.
template <typename C>
__device__ __forceinline__ C row_total(const int4 d, int r, const C *__restrict__ part) {
  constexpr int U = 8;
  const C *cp = part + d.x + r;
  const C *rp = part + d.y + r;
  const int nseg = d.z & 0xfff, tot = nseg + (d.z >> 12 & 0xfff);
  C acc[U];
#pragma unroll
  for (int u = 0; u < U; ++u) acc[u] = czero<C>();
  for (int q0 = 0; q0 < tot; q0 += U) {
    C v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int q = q0 + u;
      v[u] = czero<C>();
      if (q < tot) v[u] = q < nseg ? cp[q * 32] : rp[(q - nseg) * 32];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) acc[u] = cadd(acc[u], v[u]);
  }
#pragma unroll
  for (int w = U / 2; w >= 1; w /= 2)
#pragma unroll
    for (int u = 0; u < w; ++u) acc[u] = cadd(acc[u], acc[u + w]);
  return acc[0];
}

// Half a wave per (block, tile row I).  With rowb ({first slot of the block, slots of
// the block}): column k0 + blockIdx.y of the local vectors of nr right-hand sides, for
// the blocks whose first slot is in [slot0, slot1), with the partials of gridDim.y
// columns.
template <typename T>
__global__ __launch_bounds__(256) void k_rows(const int4 *__restrict__ rowd,
                                              const int2 *__restrict__ rowb, int64_t nrows, int nr,
                                              int k0, int64_t slot0, int64_t slot1,
                                              const cplx_t<T> *__restrict__ part,
                                              cplx_t<T> *__restrict__ yl) {
  const int64_t hw = ((int64_t)blockIdx.x * 256 + threadIdx.x) >> 5;
  if (hw >= nrows) return;
  const int r = threadIdx.x & 31;
  const int4 d = rowd[hw];
  if (rowb) {
    const int2 b = rowb[hw];
    if (b.x < slot0 || b.x >= slot1) return;
    part += (int64_t)b.x * (gridDim.y - 1) - slot0 * gridDim.y + (int64_t)b.y * blockIdx.y;
  }
  yl[(int64_t)(d.w + r * (d.z >> 24)) * nr + k0 + blockIdx.y] = row_total(d, r, part);
}

// With FWD the result of entry d is also written to every local row of the
// next block set that holds d (its reduction list), which is then applied
// without its own gather: the same values the gather would read.
template <typename T, int MODE, bool FWD>
__global__ __launch_bounds__(256) void k_scatter(int64_t nvec, const int32_t *__restrict__ red_ptr,
                                                 const int32_t *__restrict__ red_ent,
                                                 const cplx_t<T> *__restrict__ yl,
                                                 const cplx_t<T> *__restrict__ r,
                                                 cplx_t<T> *__restrict__ y, T theta,
                                                 const int32_t *__restrict__ fwd_ptr,
                                                 const int32_t *__restrict__ fwd_ent,
                                                 cplx_t<T> *__restrict__ fwd_xl) {
  using C = cplx_t<T>;
  const int64_t d = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (d >= nvec) return;
  C acc;
  acc.x = 0;
  acc.y = 0;
  for (int32_t k = red_ptr[d]; k < red_ptr[d + 1]; ++k) acc = cadd(acc, yl[red_ent[k]]);
  C out;
  if (MODE == RED_SET) out = acc;
  else if (MODE == RED_RESID) out = csub(r[d], acc);
  else if (MODE == RED_AXPY) out = cadd(y[d], cscale(acc, theta));
  else out = cscale(acc, theta);
  y[d] = out;
  if (FWD)
    for (int32_t k = fwd_ptr[d]; k < fwd_ptr[d + 1]; ++k) fwd_xl[fwd_ent[k]] = out;
}

// One column: eight lanes per vector entry d, one for each block that holds it
// (its list: tile row 32 + row of the entry in the block, in block order; longer
// lists take more rounds), each sums its row's partials, and the sums are added
// in list order, 0 + first + second + ..., in the group's first lane, which
// applies the epilogue.  The row sums never go to memory and one launch is
// saved; the partials are read in shorter runs (eight rows of a slot instead of
// 32), which costs more once they exceed the 256 MB Infinity Cache (kFusedBytes).
// Solves with k_rows and k_scatter / with this: 8^3, order levels, 15.3 / 12.1 ms;
// 4^3, p = 2, 1.69 / 1.52; 16^3, p = 3 (118 MB of FP64 partials) 25.9 / 25.5; 24^3,
// p = 4 mixed (400 MB) 108.7 / 113.1.
constexpr int64_t kFusedBytes = 192 << 20;
template <int K, typename C> __device__ __forceinline__ C add_lane(C acc, C v, int cnt) {
  const C o = dpp_c<0x100 | K>(v);   // row_shl: lane i reads lane i + K of its 16
  return csel(K < cnt, cadd(acc, o), acc);
}
template <typename T, int MODE, bool FWD>
__global__ __launch_bounds__(256) void k_rows_scatter(int64_t nvec,
                                                      const int32_t *__restrict__ red_ptr,
                                                      const int32_t *__restrict__ red_row,
                                                      const int4 *__restrict__ rowd,
                                                      const cplx_t<T> *__restrict__ part,
                                                      const cplx_t<T> *__restrict__ r,
                                                      cplx_t<T> *__restrict__ y, T theta,
                                                      const int32_t *__restrict__ fwd_ptr,
                                                      const int32_t *__restrict__ fwd_ent,
                                                      cplx_t<T> *__restrict__ fwd_xl) {
  using C = cplx_t<T>;
  const int64_t d = ((int64_t)blockIdx.x * 256 + threadIdx.x) >> 3;
  const int j = threadIdx.x & 7;
  if (d >= nvec) return;   // whole groups of eight
  const int32_t p0 = red_ptr[d];
  int cnt = red_ptr[d + 1] - p0;
  C rd, yd;
  if (MODE == RED_RESID) rd = r[d];
  if (MODE == RED_AXPY) yd = y[d];
  C acc = czero<C>();
  for (int32_t q = p0;; q += 8, cnt -= 8) {
    C v = czero<C>();
    if (j < cnt) {
      const int32_t e = red_row[q + j];
      v = row_total(rowd[e >> 5], e & 31, part);
    }
    acc = csel(0 < cnt, cadd(acc, v), acc);
    acc = add_lane<1>(acc, v, cnt);
    acc = add_lane<2>(acc, v, cnt);
    acc = add_lane<3>(acc, v, cnt);
    acc = add_lane<4>(acc, v, cnt);
    acc = add_lane<5>(acc, v, cnt);
    acc = add_lane<6>(acc, v, cnt);
    acc = add_lane<7>(acc, v, cnt);
    if (cnt <= 8) break;
  }
  C out;
  if (MODE == RED_SET) out = acc;
  else if (MODE == RED_RESID) out = csub(rd, acc);
  else if (MODE == RED_AXPY) out = cadd(yd, cscale(acc, theta));
  else out = cscale(acc, theta);
  if (j == 0) y[d] = out;
  if (FWD) {
    const int src = threadIdx.x & 0x38;   // the group's first lane
    out.x = __shfl(out.x, src, 64);
    out.y = __shfl(out.y, src, 64);
    for (int32_t k = fwd_ptr[d] + j; k < fwd_ptr[d + 1]; k += 8) fwd_xl[fwd_ent[k]] = out;
  }
}

__global__ __launch_bounds__(256) void k_pack(const int4 *__restrict__ tdesc, int64_t tile0,
                                              const int32_t *__restrict__ bn,
                                              const int64_t *__restrict__ ent_off,
                                              const double2 *__restrict__ src,
                                              const int64_t *__restrict__ src_off,
                                              const int32_t *__restrict__ ld,
                                              const int64_t *__restrict__ map_off,
                                              const int32_t *__restrict__ map,
                                              double2 *__restrict__ t64, float2 *__restrict__ t32) {
  const int64_t t = tile0 + blockIdx.x;
  const int4 td = tdesc[t];
  const int b = td.x, I = td.y, J = td.z, n = bn[b];
  const int64_t mo = map_off ? map_off[b] : -1;
  const int64_t t0 = ent_off[b] + tile_entry(I, J);
  for (int e = threadIdx.x; e < kTileFull; e += 256) {
    const int k = e >> 6, lane = e & 63, ra = lane >> 3, cb = lane & 7;
    if (I == J && ra > cb) continue;   // below the diagonal of a diagonal tile
    const int64_t dst = t0 + (I == J ? k * kDiagSlots + diag_slot(ra, cb) : e);
    const int ri = 4 * ra + (k >> 2), cj = 4 * cb + (k & 3);
    const int row = 32 * I + ri, col = 32 * J + cj;
    double2 v = mk(0.0, 0.0);
    if (row < n && col < n) {
      const int64_t mr = mo >= 0 ? map[mo + row] : row, mc = mo >= 0 ? map[mo + col] : col;
      v = src[src_off[b] + mr + mc * (int64_t)ld[b]];
    }
    if (t64) t64[dst] = v;
    if (t32) t32[dst] = mkf((float)v.x, (float)v.y);
  }
}

}  // namespace

void HermSet::build(const std::vector<int32_t> &sizes, const std::vector<int32_t> &idx_concat,
                    int64_t nvec_, bool fp64, bool fp32, Budget *bud, hipStream_t s,
                    const std::vector<int32_t> *cls, bool grouping) {
  nblk = (int)sizes.size();
  nvec = nvec_;
  n_h = sizes;
  std::vector<int64_t> toff, ceoff, eoff(nblk), cpo(nblk), rpo(nblk), loff(nblk), idx0(nblk);
  std::vector<std::vector<int32_t>> members;   // blocks of each class
  int64_t t = 0, p = 0, lo = 0, ii = 0;
  nent = 0;
  packed = 0;
  full = 0;
  full_grouped = 0;
  std::vector<int4> un;
  std::vector<int2> rw;
  std::vector<int4> td;
  for (int b = 0; b < nblk; ++b) {
    const int n = sizes[b], nt = (n + 31) / 32;
    const int cl = cls ? (*cls)[b] : b;
    const bool first = cl == (int)toff.size();   // classes are numbered by first block
    if (first) {
      toff.push_back(t);
      ceoff.push_back(nent);
      t += (int64_t)nt * (nt + 1) / 2;
      nent += tile_entry(0, nt);
      members.emplace_back();
    }
    eoff[b] = ceoff[cl];
    members[cl].push_back(b);
    idx0[b] = ii;
    full += (int64_t)n * n;
    ii += n;
    for (int J = 0; first && J < nt; ++J)
      for (int I = 0; I <= J; ++I) td.push_back(make_int4(b, I, J, 0));
  }
  if (ii != (int64_t)idx_concat.size()) throw DpgError(-1, "HermSet: index list size mismatch");
  // groups: the members of a class in about equal parts of at most kMaxGroup
  // (in block order, so that the columns of a group are mostly neighbours of
  // one another), stored widest first.  A wave takes its blocks of a group one
  // after the other, so the groups are no wider than leaves two waves per SIMD
  // (2048) to run (8^3 order levels: solve 15.6 ms with each block alone, 21.2
  // ms in groups of 32).
  struct Part { std::vector<int32_t> m; HermGroup g; };
  std::vector<Part> parts;
  auto cut = [&](int most) {
    parts.clear();
    int64_t waves = 0;
    for (size_t k = 0; k < members.size(); ++k) {
      const int cnt = (int)members[k].size(), np = (cnt + most - 1) / most;
      const int nt = (sizes[members[k][0]] + 31) / 32;
      int64_t w = 0;
      for (int J = 0; J < nt; ++J) w += J / kSeg + 1;
      if (fp32) {
        w = 0;
        for (int st = 0; 2 * st < nt; ++st) w += strip_chunks(nt, st);
      }
      for (int q = 0; q < np; ++q) {
        const int m0 = (int)((int64_t)cnt * q / np), m1 = (int)((int64_t)cnt * (q + 1) / np);
        parts.push_back({{members[k].begin() + m0, members[k].begin() + m1},
                         {ceoff[k], 0, m1 - m0, nt, 0}});
        waves += w * (fp32 ? (m1 - m0 + kStripBlocks - 1) / kStripBlocks : 1);
      }
    }
    return waves;
  };
  for (int most = grouping ? kMaxGroup : 1; cut(most) < 2048 && most > 1;) most /= 2;
  std::stable_sort(parts.begin(), parts.end(),
                   [](const Part &x, const Part &y) { return x.g.gw > y.g.gw; });
  std::vector<HermGroup> gs;
  std::vector<int2> gr;
  std::fill(std::begin(nrow_w), std::end(nrow_w), 0);
  std::vector<int32_t> alone, step(nblk, 1);   // blocks that are a group of their own
  for (Part &q : parts) {
    HermGroup &g = q.g;
    if (lo + (int64_t)g.nt * 32 * g.gw >= (1LL << 31))
      throw DpgError(-1, "HermSet: partial or local vectors beyond 32-bit offsets");
    g.base = (int32_t)lo;
    for (int m = 0; m < g.gw; ++m) {
      loff[q.m[m]] = lo + m;
      step[q.m[m]] = g.gw;
    }
    lo += (int64_t)g.nt * 32 * g.gw;
    for (int I = 0; I < g.nt; ++I) gr.push_back(make_int2((int)gs.size(), I));
    for (int w = 0; w <= g.gw; ++w) nrow_w[w] += g.nt;
    if (g.gw == 1) alone.push_back(q.m[0]);
    else full_grouped += (int64_t)g.gw * sizes[q.m[0]] * sizes[q.m[0]];
    gs.push_back(g);
  }
  std::sort(alone.begin(), alone.end());
  std::vector<int32_t> gi(lo, -1);
  for (int b = 0; b < nblk; ++b)
    for (int i = 0; i < sizes[b]; ++i) gi[loff[b] + (int64_t)i * step[b]] = idx_concat[idx0[b] + i];
  for (const Part &q : parts)
    for (int32_t b : q.m) {
      const int nt = q.g.nt;
      cpo[b] = p;
      p += colbase(nt);
      rpo[b] = p;
      p += (int64_t)nt * (nt + 1) / 2 * 32;
    }
  for (int b = 0; b < nblk; ++b)
    for (int J = 0; 32 * J < sizes[b]; ++J) rw.push_back(make_int2(b, J));
  for (int32_t b : alone) {
    const int n = sizes[b], nt = (n + 31) / 32;
    packed += (int64_t)n * (n + 1) / 2;
    for (int J = 0; fp64 && J < nt; ++J)
      for (int seg = 0; seg * kSeg <= J; ++seg) un.push_back(make_int4(b, J, seg * kSeg, seg));
  }
  // units in block order (block, tile column, segment): the waves of
  // neighbouring workgroups stream neighbouring tiles (longest first, the
  // blocks mixed, was 1.3 % slower at 16^3, shuffled slower still)
  ntiles = t;
  npart = p;
  nloc = lo;
  nunits = (int64_t)un.size();
  // of groups (group, tile column, segment): as below with the first block's
  // offsets, flags | blocks << 8, and {slots of a block, first slot of the
  // group, 0, 0}; the blocks that are a group of their own at the end
  //
  // The units of all groups of a class that read the same tiles follow one another,
  // so that the tiles come from memory once per class and not once per group (a
  // class of order 1399 is 8 MB in FP32, twice an L2): 16^3, p = 3 23.6 -> 22.8 ms per
  // solve, 24^3, p = 4 mixed 105 -> 100 (with the x of k_strips_grp through LDS).
  std::vector<std::vector<const Part *>> runs;   // groups of a class; blocks alone last
  {
    std::map<int64_t, size_t> at;
    for (const Part &q : parts) {
      const auto it = q.g.gw > 1 ? at.emplace(q.g.ent, runs.size()).first : at.end();
      if (it == at.end() || it->second == runs.size()) runs.emplace_back();
      runs[it == at.end() ? runs.size() - 1 : it->second].push_back(&q);
    }
  }
  std::vector<int4> gud64;
  gnunits64 = 0;
  for (const auto &run : runs) {
    if (!fp64) break;
    const int nt = run[0]->g.nt;
    const int64_t each = colbase(nt) + (int64_t)nt * (nt + 1) / 2 * 32;
    if (gnunits64 == 0 && run[0]->g.gw == 1) {
      unit0_h.push_back((int64_t)gud64.size() / 3);
      slot0_h.push_back(cpo[run[0]->m[0]]);
      max_slots = std::max(max_slots, each);
    }
    for (int J = 0; J < nt; ++J)
      for (int I0 = 0; I0 <= J; I0 += kSeg) for (const Part *pq : run) {
        const Part &q = *pq;
        const int b = q.m[0];
        const int64_t tile = q.g.ent + tile_entry(I0, J);
        const int64_t rd = I0 + 1 <= J ? row_slot(nt, I0 + 1, J) - row_slot(nt, I0, J) : 0;
        const int flags = (I0 + 1 <= J ? 1 : 0) | (I0 < J ? 2 : 0) | (I0 + 1 < J ? 4 : 0);
        gud64.push_back(make_int4((int)(uint32_t)(tile & 0xffffffff), (int)(tile >> 32),
                                  (int)(loff[b] + (int64_t)32 * I0 * q.g.gw),
                                  (int)(loff[b] + (int64_t)32 * J * q.g.gw)));
        gud64.push_back(make_int4((int)(rpo[b] + row_slot(nt, I0, J)), (int)rd,
                                  (int)(cpo[b] + colbase(J) + I0 / kSeg * 32), flags | q.g.gw << 8));
        gud64.push_back(make_int4((int)each, (int)cpo[b], 0, 0));
      }
    if (run[0]->g.gw > 1) gnunits64 = (int64_t)gud64.size() / 3;
  }
  gall64 = (int64_t)gud64.size() / 3;
  unit0_h.push_back(gall64);
  slot0_h.push_back(npart);
  std::vector<int2> rb;
  for (const int2 &k : rw) {
    if (!fp64) break;
    const int b = k.x, nt = (sizes[b] + 31) / 32;
    rb.push_back(make_int2((int)cpo[b], (int)(colbase(nt) + (int64_t)nt * (nt + 1) / 2 * 32)));
  }
  if ((fp64 && npart >= (1LL << 31)) || nloc >= (1LL << 31))
    throw DpgError(-1, "HermSet: partial or local vectors beyond 32-bit offsets");
  // unit descriptors: {entry offset of tile (I0, J) lo, hi, x offset of tile
  // row I0, of tile column J}, {row-partial slot of (I0, J), step to the slot of (I0 + 1, J),
  // column-partial slot, flags: 1 two tiles, 2 first tile off-diagonal, 4
  // second tile off-diagonal}
  std::vector<int4> ud(2 * un.size());
  for (size_t k = 0; k < un.size(); ++k) {
    const int b = un[k].x, J = un[k].y, I0 = un[k].z, seg = un[k].w;
    const int nt = (sizes[b] + 31) / 32;
    const int64_t tile = eoff[b] + tile_entry(I0, J);
    const int64_t r0 = rpo[b] + row_slot(nt, I0, J);
    const int64_t rd = I0 + 1 <= J ? row_slot(nt, I0 + 1, J) - row_slot(nt, I0, J) : 0;
    const int64_t cs = cpo[b] + colbase(J) + seg * 32;
    const int flags = (I0 + 1 <= J ? 1 : 0) | (I0 < J ? 2 : 0) | (I0 + 1 < J ? 4 : 0);
    ud[2 * k] = make_int4((int)(uint32_t)(tile & 0xffffffff), (int)(tile >> 32),
                          (int)(loff[b] + 32 * I0), (int)(loff[b] + 32 * J));
    ud[2 * k + 1] = make_int4((int)r0, (int)rd, (int)cs, flags);
  }
  nrows = (int64_t)rw.size();
  std::vector<int4> rd(fp64 ? rw.size() : 0);
  for (size_t k = 0; k < rd.size(); ++k) {
    const int b = rw[k].x, I = rw[k].y, nt = (sizes[b] + 31) / 32;
    const int nseg = (I + kSeg) / kSeg, nrw = nt - I;
    if (nt > kMaxTiles) throw DpgError(-1, "HermSet: block too large for row descriptors");
    rd[k] = make_int4((int)(cpo[b] + colbase(I)), (int)(rpo[b] + row_slot(nt, I, I)),
                      nseg | nrw << 12 | step[b] << 24, (int)(loff[b] + (int64_t)32 * I * step[b]));
  }
  // FP32: units (block, strip, chunk), in that order: {entry offset of
  // tile (0, J0) lo, hi, x offset of the block, row-sum base of the block},
  // {J0 | nt << 16, Ia | Ib << 16, column-sum slot of J0, of J1 (0 without
  // J1)}; of groups (up to four blocks, strip, chunk): {entry offset lo, hi, x
  // offset of the first block, blocks | row step << 8}, {J0 | nt << 16, Ia |
  // Ib << 16, column-sum slot of J0 of the first block, its row-sum base},
  // {step of the slots from block to block, 0, 0, 0}; rows: the column sums of
  // tile column I (one slot per chunk of its strip) and the row sums of tile
  // row I (one slot per strip s >= I / 2)
  std::vector<int4> sud, gud, srd;
  if (fp32) {
    std::vector<int64_t> scpo(nblk), srpo(nblk);
    std::map<int, std::vector<int32_t>> cbase;   // by tile count
    int64_t sp = 0;
    for (const Part &q : parts) {
      const int nt = q.g.nt;
      if (nt > kMaxTiles) throw DpgError(-1, "HermSet: block too large for strip descriptors");
      std::vector<int32_t> &cbv = cbase[nt];
      if (cbv.empty()) {
        cbv.assign(nt + 1, 0);
        for (int J = 0; J < nt; ++J) cbv[J + 1] = cbv[J] + strip_chunks(nt, J / 2);
      }
      for (int32_t b : q.m) {
        scpo[b] = sp;
        sp += 32LL * cbv[nt];
        srpo[b] = sp;
        sp += 32 * strip_row_slots(nt);
      }
    }
    snpart = sp;
    if (snpart >= (1LL << 31)) throw DpgError(-1, "HermSet: partials beyond 32-bit offsets");
    for (int32_t b : alone) {
      const int nt = (sizes[b] + 31) / 32;
      for (int st = 0; 2 * st < nt; ++st) {
        const int J0 = 2 * st, J1 = J0 + 1, rws = strip_rows(nt, st);
        const bool two = J1 < nt;
        const int64_t tile = eoff[b] + tile_entry(0, J0);
        for (int c = 0; c * kChunk < rws; ++c) {
          const int Ia = c * kChunk, Ib = std::min(rws, Ia + kChunk);
          sud.push_back(make_int4((int)(uint32_t)(tile & 0xffffffff), (int)(tile >> 32),
                                  (int)loff[b], (int)srpo[b]));
          sud.push_back(make_int4(J0 | (nt << 16), Ia | (Ib << 16),
                                  (int)(scpo[b] + 32LL * (cbase[nt][J0] + c)),
                                  two ? (int)(scpo[b] + 32LL * (cbase[nt][J1] + c)) : 0));
        }
      }
    }
    for (const auto &run : runs) {
      if (run[0]->g.gw == 1) continue;
      const int nt = run[0]->g.nt;
      const int64_t each = 32LL * (cbase[nt][nt] + strip_row_slots(nt));
      for (int st = 0; 2 * st < nt; ++st)
        for (int c = 0; c * kChunk < strip_rows(nt, st); ++c) for (const Part *pq : run) {
          const Part &q = *pq;
          const int np = (q.g.gw + kStripBlocks - 1) / kStripBlocks;
          for (int u = 0; u < np; ++u) {   // blocks m0 .. m1 - 1 of the group
            const int m0 = q.g.gw * u / np, m1 = q.g.gw * (u + 1) / np, b = q.m[m0];
            const int64_t tile = q.g.ent + tile_entry(0, 2 * st);
            gud.push_back(make_int4((int)(uint32_t)(tile & 0xffffffff), (int)(tile >> 32),
                                    (int)loff[b], (m1 - m0) | q.g.gw << 8));
            gud.push_back(make_int4(2 * st | (nt << 16),
                                    c * kChunk | std::min(strip_rows(nt, st), (c + 1) * kChunk) << 16,
                                    (int)(scpo[b] + 32LL * (cbase[nt][2 * st] + c)), (int)srpo[b]));
            gud.push_back(make_int4((int)each, 0, 0, 0));
          }
        }
    }
    snunits = (int64_t)sud.size() / 2;
    gnunits = (int64_t)gud.size() / 3;
    for (const int2 &k : rw) {
      const int b = k.x, I = k.y, nt = (sizes[b] + 31) / 32, ns = (nt + 1) / 2;
      const int nseg = strip_chunks(nt, I / 2), nrw = ns - I / 2;
      srd.push_back(make_int4((int)(scpo[b] + 32LL * cbase[nt][I]),
                              (int)(srpo[b] + 32 * strip_row_slot(ns, I, I / 2)),
                              nseg | nrw << 12 | step[b] << 24,
                              (int)(loff[b] + (int64_t)32 * I * step[b])));
    }
  }
  tile_off_h = toff;
  ent_off_h = eoff;
  loc_off_h = loff;
  // reduction lists: for every vector entry, the local rows holding it
  std::vector<int32_t> cnt(nvec + 1, 0);
  for (int32_t v : idx_concat) {
    if (v < 0 || v >= nvec) throw DpgError(-1, "HermSet: index out of range");
    cnt[v + 1]++;
  }
  for (int64_t d = 0; d < nvec; ++d) cnt[d + 1] += cnt[d];
  std::vector<int32_t> ent(cnt[nvec]), erow(cnt[nvec]);
  std::vector<int32_t> fill(cnt.begin(), cnt.end() - 1);
  if (32 * (int64_t)rw.size() >= (1LL << 31))
    throw DpgError(-1, "HermSet: partial or local vectors beyond 32-bit offsets");
  for (int b = 0, row0 = 0; b < nblk; ++b) {   // in block order, whatever the groups
    for (int i = 0; i < sizes[b]; ++i) {
      const int32_t f = fill[idx_concat[idx0[b] + i]]++;
      ent[f] = (int32_t)(loff[b] + (int64_t)i * step[b]);
      erow[f] = 32 * row0 + i;   // rows of rw: tile row I of block b is row0 + I
    }
    row0 += (sizes[b] + 31) / 32;
  }
  ListPack all;
  auto add = [&](auto &dst, const auto &v) { all.add(dst, v); };
  add(bn, sizes);
  add(ent_off, eoff);
  add(grp, gs);
  add(grow, gr);
  add(gidx, gi);
  add(units, ud);
  add(gunits64, gud64);
  add(rowd, rd);
  add(rowb, rb);
  add(tdesc, td);
  add(red_ptr, cnt);
  add(red_ent, ent);
  add(red_row, erow);
  add(sunits, sud);
  add(gunits, gud);
  add(srowd, srd);
  all.upload(lists, bud, s);
  if (fp64) {
    t64.alloc(nent, bud);
    p64.alloc(npart, bud);
    if (npart * 16 > kFusedBytes) yl64.alloc(nloc, bud);
    xl64.alloc(nloc, bud);
    launch_zero(nloc, xl64.p, s);
  }
  if (fp32) {
    t32.alloc(nent, bud);
    p32.alloc(snpart, bud);
    if (snpart * 8 > kFusedBytes) yl32.alloc(nloc, bud);
    xl32.alloc(nloc, bud);
    launch_zero(nloc, xl32.p, s);
  }
  HIP_OK(hipStreamSynchronize(s));
}

void HermSet::pack(const double2 *src, const int64_t *src_off_dev, const int32_t *ld_dev,
                   const int64_t *map_off_dev, const int32_t *map_dev, hipStream_t s,
                   int64_t tile0, int64_t count) {
  if (count < 0) count = ntiles - tile0;
  if (count <= 0) return;
  hipLaunchKernelGGL(k_pack, dim3((unsigned)count), dim3(256), 0, s, tdesc.p, tile0, bn.p,
                     ent_off.p, src,
                     src_off_dev, ld_dev, map_off_dev, map_dev, t64.p, t32.p);
  LAUNCH_OK();
}

template <typename T, int MODE>
void launch_reduce(const HermSet &H, const cplx_t<T> *part, cplx_t<T> *yl, const cplx_t<T> *r,
                   cplx_t<T> *y, T theta, HermSet *fwd, cplx_t<T> *fxl, hipStream_t s) {
  const dim3 g(cdiv(H.nvec, yl ? 256 : 32));
  const int4 *rowd = sizeof(T) == 8 ? H.rowd.p : H.srowd.p;
  if (yl) {
    hipLaunchKernelGGL((k_rows<T>), dim3(cdiv(H.nrows, 8)), dim3(256), 0, s, rowd,
                       (const int2 *)nullptr, H.nrows, 1, 0, 0, 0, part, yl);
    LAUNCH_OK();
    if (fwd)
      hipLaunchKernelGGL((k_scatter<T, MODE, true>), g, dim3(256), 0, s, H.nvec, H.red_ptr.p,
                         H.red_ent.p, yl, r, y, theta, fwd->red_ptr.p, fwd->red_ent.p, fxl);
    else
      hipLaunchKernelGGL((k_scatter<T, MODE, false>), g, dim3(256), 0, s, H.nvec, H.red_ptr.p,
                         H.red_ent.p, yl, r, y, theta, nullptr, nullptr, nullptr);
    return;
  }
  if (fwd)
    hipLaunchKernelGGL((k_rows_scatter<T, MODE, true>), g, dim3(256), 0, s, H.nvec, H.red_ptr.p,
                       H.red_row.p, rowd, part, r, y, theta, fwd->red_ptr.p, fwd->red_ent.p, fxl);
  else
    hipLaunchKernelGGL((k_rows_scatter<T, MODE, false>), g, dim3(256), 0, s, H.nvec, H.red_ptr.p,
                       H.red_row.p, rowd, part, r, y, theta, nullptr, nullptr, nullptr);
}

template <typename T> cplx_t<T> *local_x(HermSet &H) {
  if constexpr (sizeof(T) == 8) return H.xl64.p;
  else return H.xl32.p;
}

template <typename T>
void herm_apply(HermSet &H, const cplx_t<T> *x, cplx_t<T> *y, const cplx_t<T> *r, int mode,
                T theta, hipStream_t s, bool gathered, HermSet *fwd) {
  const cplx_t<T> *tiles;
  cplx_t<T> *part, *xl, *yl;
  if constexpr (sizeof(T) == 8) {
    tiles = H.t64.p;
    part = H.p64.p;
    yl = H.yl64.p;
  } else {
    tiles = H.t32.p;
    part = H.p32.p;
    yl = H.yl32.p;
  }
  xl = local_x<T>(H);
  if (!tiles) throw DpgError(-6, "block set has no tiles of this precision");
  cplx_t<T> *fxl = fwd ? local_x<T>(*fwd) : nullptr;
  if (fwd && (!fxl || fwd->nvec != H.nvec))
    throw DpgError(-1, "forwarded block set does not match this one");
  if (!gathered) {
    ProfScope ps(H.prof, DPG_K_REDUCE, 0.0, s);
    hipLaunchKernelGGL((k_gather_x<T>), dim3(cdiv(H.nloc, 256)), dim3(256), 0, s, H.nloc,
                       H.gidx.p, x, xl);
    LAUNCH_OK();
  }
  if constexpr (sizeof(T) == 8) {
    if (H.gnunits64 > 0) {
      ProfScope ps(H.prof, DPG_K_APPLYG64, 8.0 * (double)H.full_grouped, s);
      hipLaunchKernelGGL((k_units_grp<T, false>), dim3(8 * cdiv(cdiv(H.gnunits64, 4), 8)),
                         dim3(256), 0, s, tiles, H.gunits64.p, H.gnunits64, 1, 0, 1, 0, xl, part);
      LAUNCH_OK();
    }
    if (H.nunits > 0) {
      ProfScope ps(H.prof, DPG_K_APPLY64, (double)H.packed_entries() * sizeof(cplx_t<T>), s);
      hipLaunchKernelGGL((k_units<T>), dim3(8 * cdiv(cdiv(H.nunits, 4), 8)), dim3(256), 0, s,
                         tiles, H.units.p, H.nunits, xl, part);
      LAUNCH_OK();
    }
  } else {
    if (H.gnunits > 0) {
      ProfScope ps(H.prof, DPG_K_APPLYG32, 8.0 * (double)H.full_grouped, s);
      hipLaunchKernelGGL((k_strips_grp<T>), dim3(8 * cdiv(cdiv(H.gnunits, 4), 8)), dim3(256), 0, s,
                         tiles, H.gunits.p, H.gnunits, xl, part);
      LAUNCH_OK();
    }
    if (H.snunits > 0) {
      ProfScope ps(H.prof, DPG_K_APPLY32, (double)H.packed_entries() * sizeof(cplx_t<T>), s);
      hipLaunchKernelGGL((k_strips<T>), dim3(8 * cdiv(cdiv(H.snunits, 4), 8)), dim3(256), 0, s,
                         tiles, H.sunits.p, H.snunits, xl, part);
      LAUNCH_OK();
    }
  }
  ProfScope ps(H.prof, DPG_K_REDUCE, 0.0, s);
  switch (mode) {
    case RED_SET: launch_reduce<T, RED_SET>(H, part, yl, r, y, theta, fwd, fxl, s); break;
    case RED_RESID: launch_reduce<T, RED_RESID>(H, part, yl, r, y, theta, fwd, fxl, s); break;
    case RED_AXPY: launch_reduce<T, RED_AXPY>(H, part, yl, r, y, theta, fwd, fxl, s); break;
    default: launch_reduce<T, RED_SET_SCALED>(H, part, yl, r, y, theta, fwd, fxl, s);
  }
  LAUNCH_OK();
}

void launch_units_cols(HermSet &H, const double2 *xl, double2 *part, int64_t npart_max,
                       double2 *yl, int nr, hipStream_t s) {
  const int nb = (int)H.slot0_h.size() - 1, q = (int)std::min<int64_t>(nr, npart_max / H.max_slots);
  if (q < 1) throw DpgError(-1, "block apply: no room for the partials");
  for (int k0 = 0; k0 < nr; k0 += q) {
    const int kc = std::min(q, nr - k0);
    for (int b = 0, e; b < nb; b = e) {
      for (e = b + 1; e < nb && (H.slot0_h[e + 1] - H.slot0_h[b]) * kc <= npart_max;) ++e;
      const int64_t u0 = H.unit0_h[b], n = H.unit0_h[e] - u0;
      {
        ProfScope ps(H.prof, DPG_K_APPLYG64,
                     8.0 * (double)H.full * kc * (double)n / (double)H.gall64, s);
        hipLaunchKernelGGL((k_units_grp<double, true>), dim3(8 * cdiv(cdiv(n, 4), 8)), dim3(256),
                           0, s, H.t64.p, H.gunits64.p + 3 * u0, n, nr, k0, kc, H.slot0_h[b], xl,
                           part);
        LAUNCH_OK();
      }
      ProfScope ps(H.prof, DPG_K_REDUCE, 0.0, s);
      hipLaunchKernelGGL((k_rows<double>), dim3(cdiv(H.nrows, 8), kc), dim3(256), 0, s, H.rowd.p,
                         H.rowb.p, H.nrows, nr, k0, H.slot0_h[b], H.slot0_h[e], part, yl);
      LAUNCH_OK();
    }
  }
}

template void herm_apply<double>(HermSet &, const double2 *, double2 *, const double2 *, int,
                                 double, hipStream_t, bool, HermSet *);
template void herm_apply<float>(HermSet &, const float2 *, float2 *, const float2 *, int, float,
                                hipStream_t, bool, HermSet *);

}  // namespace dpg
