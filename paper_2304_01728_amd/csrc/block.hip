// Multi-right-hand-side kernels (see block.hpp).
#include <algorithm>

#include "block.hpp"
#include "kernels.hpp"

namespace dpg {
namespace {

constexpr int kBMaxI = 1024;   // interior unknowns per macro block (as the single path)
constexpr int KC = 4;          // columns per workgroup in the condensation kernels

template <typename C> __device__ inline C czero() {
  C r;
  r.x = 0;
  r.y = 0;
  return r;
}

// ---- Hermitian block sets ------------------------------------------------------------

template <typename T>
__global__ __launch_bounds__(256) void k_gather_blk(int64_t nloc, int nr,
                                                    const int32_t *__restrict__ gidx,
                                                    const cplx_t<T> *__restrict__ x,
                                                    cplx_t<T> *__restrict__ xl) {
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (e >= nloc * nr) return;
  const int64_t i = e / nr;
  const int k = (int)(e % nr);
  const int32_t g = gidx[i];
  xl[e] = g >= 0 ? x[(int64_t)g * nr + k] : czero<cplx_t<T>>();
}

// ---- the block apply on the matrix cores ------------------------------------------------
//
// Columns: the local vectors of the blocks of a group, times the right-hand
// sides (HermGroup).  A unit (group, tile row I) forms Y_I = sum_J A_IJ X_J of a
// chunk of 32 columns over the stored upper tiles of row I (J >= I) and the
// conjugate transposes of the stored tiles of column I (J < I), so no partial
// sums leave it; every tile is read by two units, of which one finds it in a
// cache.  Workgroup g runs on XCD g % 8, so each XCD is given a contiguous range
// of units: the rows of one group then share its tiles and X in one L2.
typedef float v16f __attribute__((ext_vector_type(16)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef double v4d __attribute__((ext_vector_type(4)));

struct RowUnit {
  int64_t ent, base;   // tiles of the class; row 0, first column of the chunk in the local vectors
  int I, nt, ld, nc;   // row step of the local vectors and columns of the chunk
  bool on;
};

__device__ __forceinline__ RowUnit row_unit(const int2 *__restrict__ rows, const ChunkMap &cm,
                                            const HermGroup *__restrict__ grp, int nr) {
  RowUnit u;
  const int per = (cm.total + 7) / 8;
  int w = (int)(blockIdx.x % 8) * per + (int)(blockIdx.x / 8), c = 0;
  u.on = w < cm.total;
  if (!u.on) return u;
  while (w >= cm.cnt[c]) w -= cm.cnt[c++];
  const int2 r = rows[w];
  const HermGroup g = grp[r.x];
  u.ent = g.ent;
  u.I = r.y;
  u.nt = g.nt;
  u.ld = g.gw * nr;
  u.nc = min(32, u.ld - 32 * c);
  u.base = (int64_t)g.base * nr + 32 * c;
  return u;
}

typedef unsigned int v2u __attribute__((ext_vector_type(2)));

// Raw buffer over n entries at p (wave-uniform); reads past them give zero.  Sizes and
// offsets have 32 bits: one tile, or the columns of one group (32 kMaxTiles rows of
// kMaxGroup kMaxCols columns at most).
static_assert(32LL * kMaxTiles * kMaxGroup * kMaxCols * sizeof(float2) < (1LL << 31),
              "X of a group beyond a buffer's offsets");
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_of(const float2 *p, int64_t n) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<float2 *>(p), 0, (int)(n * sizeof(float2)),
                                           0x00020000);
}
// The entry at byte offset vo (per lane) + so (wave-uniform).
__device__ __forceinline__ float2 buffer_at(__amdgpu_buffer_rsrc_t r, int vo, int so) {
  const v2u v = __builtin_amdgcn_raw_buffer_load_b64(r, vo, so, 0);
  return make_float2(__uint_as_float(v.x), __uint_as_float(v.y));
}

// FP32.  Y_I accumulates three real products per tile (the
// three-multiplication complex product: a quarter fewer matrix-core
// operations, and an imaginary part formed as p3 - p1 - p2, which in FP32
// can lose digits when it is small against |A||X|; this path is the
// mixed-precision preconditioner, corrected by the FP64 outer iteration),
// with v_mfma_f32_32x32x2f32 (lane l supplies A[l%32][k] and B[k][l%32] for
// k = l/32 of each two-column slice, and receives result row
// 8(v/4) + 4(l/32) + v%4, column l%32 in register v) or, up to 16 columns,
// two 16-row blocks of v_mfma_f32_16x16x4f32 (half the cycles; lane l: row or
// column l%16, k = l/16 of a four-column slice, result row 4(l/16) + v).  Both
// add the products of a result one by one in the order of k, fused, so the
// results do not depend on the shape.  The tile A_IJ is staged in LDS column by
// column (rows XOR-swizzled per group of four columns); X_J
// goes straight from global memory into the B operands, which for 32 columns
// are contiguous 512-byte rows.  A tile's registers are loaded again as soon as
// it is staged, and an X operand's as soon as it is multiplied, so one register
// set each is in flight through the whole step and three waves fit a SIMD.
template <int NC>
__device__ __forceinline__ void rows32(const RowUnit &u, const float2 *__restrict__ tiles,
                                       const float2 *__restrict__ xl, float2 *__restrict__ yl,
                                       float2 *buf) {
  constexpr int NX = NC / 2;   // X entries per lane and tile
  const int lane = threadIdx.x, a = lane >> 3, q = lane & 7;
  const int kk = NC == 32 ? lane >> 5 : lane >> 4, n = lane & (NC - 1);
  const int I = u.I, nt = u.nt;
  // columns past nc read column nc - 1: B column n only feeds result column
  // n, and those results are not stored
  const int ncl = min(n, u.nc - 1);
  // a diagonal tile stores the sub-blocks a <= q only (slot diag_slot(a, q))
  const bool dup = a <= q;
  const int dsl = dup ? diag_slot(a, q) : 0;
  // tiles (a descriptor each, at a 64-bit address) and X through buffer descriptors: a
  // load is the lane's offset, fixed, and a scalar one, so that no vector instruction
  // forms addresses
  const auto rx = buffer_of(xl + u.base, (int64_t)(32 * nt - 1) * u.ld + u.nc);
  const int xo = (ncl + kk * u.ld) * (int)sizeof(float2);
  const int xs = 64 / NC * u.ld * (int)sizeof(float2);   // step of a lane's X entries
  // Where the lane's entries (4a + i, 4q + j) go: row m of column c at
  // 32 c + (m ^ 2 (c / 4 % 8)).  As A_IJ they are rows 4a + i of columns 4q + j,
  // entry i of a column at up[i / 2] + i % 2 + 32 j; transposed, rows 4q + j of
  // columns 4a + i, at lo[j / 2] + j % 2 + 32 i.
  float2 *const up[2] = {buf + 128 * q + 4 * (a ^ (q >> 1)) + 2 * (q & 1),
                         buf + 128 * q + 4 * (a ^ (q >> 1)) + 2 - 2 * (q & 1)};
  float2 *const lo[2] = {buf + 128 * a + 4 * (q ^ (a >> 1)) + 2 * (a & 1),
                         buf + 128 * a + 4 * (q ^ (a >> 1)) + 2 - 2 * (a & 1)};
  float2 *const away = buf + 32 * 32;   // for lanes of a diagonal tile without an entry
  float2 t[16], x[NX];
  auto load_tile = [&](int J) {
    // lanes below the diagonal of a diagonal tile read slot 0 (in range)
    const TileSpan ts = tile_span(I, J);
    const auto rt = buffer_of(tiles + u.ent + ts.first, ts.entries);
    const int step = ts.step * (int)sizeof(float2);
    const int vo = (J != I ? lane : dsl) * (int)sizeof(float2);
#pragma unroll
    for (int k = 0; k < 16; ++k) t[k] = buffer_at(rt, vo, k * step);
  };
  // three real products (Gauss): p1 = Re A Re X, p2 = Im A Im X,
  // p3 = (Re A + Im A)(Re X + Im X); Re Y = p1 - p2, Im Y = p3 - p1 - p2
  v16f p1, p2, p3;
  v4f q1[2], q2[2], q3[2];
  if constexpr (NC == 32) {
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      p1[v] = 0.f;
      p2[v] = 0.f;
      p3[v] = 0.f;
    }
  } else {
#pragma unroll
    for (int rb = 0; rb < 2; ++rb) q1[rb] = q2[rb] = q3[rb] = v4f{0.f, 0.f, 0.f, 0.f};
  }
  load_tile(0);
#pragma unroll
  for (int s = 0; s < NX; ++s) x[s] = buffer_at(rx, xo, s * xs);
#pragma unroll 1
  for (int J = 0; J < nt; ++J) {
    // the lane holds stored entries (4a + i, 4q + j) at 4i + j; A_IJ is the
    // stored tile (J > I), the conjugate transpose of tile (J, I), or both
    // triangles of the diagonal tile, whose lanes a <= q hold something.
    // (Separate code and fixed addresses for each: choosing row, column and sign
    // per entry took eight vector instructions an entry, and vector instructions
    // take matrix-core time here.  With those and the load addresses gone, about
    // 200 to 50 a tile, and no path on which a load is waited for late, 32 columns
    // of 24^3, p = 3: 282 to 240 ms in this kernel, 123 to 144 TFLOP/s.)
    auto stage_up = [&](float2 *u0, float2 *u1) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) (i >> 1 ? u1 : u0)[(i & 1) + 32 * j] = t[4 * i + j];
    };
    auto stage_lo = [&](float2 *l0, float2 *l1) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          (j >> 1 ? l1 : l0)[(j & 1) + 32 * i] = make_float2(t[4 * i + j].x, -t[4 * i + j].y);
    };
    wave_lds_fence();   // the tile before has been read
    if (J > I) {
      stage_up(up[0], up[1]);
    } else if (J < I) {
      stage_lo(lo[0], lo[1]);
    } else {
      stage_up(dup ? up[0] : away, dup ? up[1] : away);
      stage_lo(a < q ? lo[0] : away, a < q ? lo[1] : away);
    }
    wave_lds_fence();
    const int Jn = min(J + 1, nt - 1);   // the loads after the last tile repeat it
    load_tile(Jn);
    __builtin_amdgcn_sched_barrier(0);
    const int xn = 32 * Jn * u.ld * (int)sizeof(float2);
    if constexpr (NC == 32) {
      float2 av = buf[kk * 32 + n];
#pragma unroll
      for (int s = 0; s < 16; ++s) {
        const float2 ac = av;
        if (s < 15) av = buf[(2 * (s + 1) + kk) * 32 + (n ^ (2 * ((s + 1) >> 1)))];
        p1 = __builtin_amdgcn_mfma_f32_32x32x2f32(ac.x, x[s].x, p1, 0, 0, 0);
        p2 = __builtin_amdgcn_mfma_f32_32x32x2f32(ac.y, x[s].y, p2, 0, 0, 0);
        p3 = __builtin_amdgcn_mfma_f32_32x32x2f32(ac.x + ac.y, x[s].x + x[s].y, p3, 0, 0, 0);
        x[s] = buffer_at(rx, xo, xn + s * xs);
        __builtin_amdgcn_sched_barrier(0);
      }
    } else {
      float2 av[2] = {buf[kk * 32 + n], buf[kk * 32 + 16 + n]};
#pragma unroll
      for (int s = 0; s < 8; ++s) {
        const float2 ac[2] = {av[0], av[1]};
        if (s < 7) {
          av[0] = buf[(4 * (s + 1) + kk) * 32 + (n ^ (2 * (s + 1)))];
          av[1] = buf[(4 * (s + 1) + kk) * 32 + ((16 + n) ^ (2 * (s + 1)))];
        }
        const float xsum = x[s].x + x[s].y;
#pragma unroll
        for (int rb = 0; rb < 2; ++rb)
          q1[rb] = __builtin_amdgcn_mfma_f32_16x16x4f32(ac[rb].x, x[s].x, q1[rb], 0, 0, 0);
#pragma unroll
        for (int rb = 0; rb < 2; ++rb)
          q2[rb] = __builtin_amdgcn_mfma_f32_16x16x4f32(ac[rb].y, x[s].y, q2[rb], 0, 0, 0);
#pragma unroll
        for (int rb = 0; rb < 2; ++rb)
          q3[rb] = __builtin_amdgcn_mfma_f32_16x16x4f32(ac[rb].x + ac[rb].y, xsum, q3[rb], 0, 0, 0);
        x[s] = buffer_at(rx, xo, xn + s * xs);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
  if (n >= u.nc) return;
  float2 *yb = yl + u.base + (int64_t)32 * I * u.ld + n;
  if constexpr (NC == 32) {
#pragma unroll
    for (int v = 0; v < 16; ++v)
      yb[(int64_t)(8 * (v >> 2) + 4 * kk + (v & 3)) * u.ld] =
          make_float2(p1[v] - p2[v], p3[v] - p1[v] - p2[v]);
  } else {
#pragma unroll
    for (int rb = 0; rb < 2; ++rb)
#pragma unroll
      for (int v = 0; v < 4; ++v)
        yb[(int64_t)(16 * rb + 4 * kk + v) * u.ld] =
            make_float2(q1[rb][v] - q2[rb][v], q3[rb][v] - q1[rb][v] - q2[rb][v]);
  }
}

__global__ __launch_bounds__(64, 3) void k_rows_mfma(const float2 *__restrict__ tiles,
                                                     const int2 *__restrict__ rows,
                                                     const ChunkMap cm,
                                                     const HermGroup *__restrict__ grp,
                                                     const float2 *__restrict__ xl,
                                                     float2 *__restrict__ yl, int nr) {
  __shared__ float2 buf[32 * 32 + 128];   // the tile, and entries that nobody reads
  const RowUnit u = row_unit(rows, cm, grp, nr);
  if (!u.on) return;
  if (u.nc <= 16) rows32<16>(u, tiles, xl, yl, buf);
  else rows32<32>(u, tiles, xl, yl, buf);
}

// FP64 form (v_mfma_f64_16x16x4f64: lane l supplies A[l%16][k] and B[k][l%16]
// for k = l/16 of each four-column step, and receives result row 4v + l/16,
// column l%16 in element v).  One wave per unit: Y_I as 2 x (1 or 2) blocks of
// 16 x 16, each complex product as four real ones (the outer-iteration operator
// keeps full FP64 accuracy).  The tile A_IJ is staged in
// LDS column by column (stride 33); X_J goes from global memory straight into
// the B operands; registers are loaded again as soon as they are staged or
// multiplied, as in the FP32 form (two waves per SIMD).
template <int NC>
__device__ __forceinline__ void rows64(const RowUnit &u, const double2 *__restrict__ tiles,
                                       const double2 *__restrict__ xl, double2 *__restrict__ yl,
                                       double2 *buf) {
  constexpr int NB = NC == 32 ? 2 : 1;
  const int lane = threadIdx.x, a = lane >> 3, q = lane & 7;
  const int li = lane & 15, lk = lane >> 4, I = u.I, nt = u.nt;
  // columns past nc read column nc - 1; their results are not stored
  const int c0 = min(li, u.nc - 1), c1 = min(16 + li, u.nc - 1);
  // a diagonal tile stores the sub-blocks a <= q only (slot diag_slot(a, q))
  const bool dup = a <= q;
  const int dsl = dup ? diag_slot(a, q) : 0;
  const double2 *xb = xl + u.base;
  double2 t[16], x[8 * NB];
  auto load_tile = [&](int J) {
    // (wave-uniform branch, constant strides: immediate load offsets); lanes
    // below the diagonal of a diagonal tile read slot 0 (in range), their
    // values are not staged
    if (J != I) {
      const double2 *tp = tiles + u.ent + (J > I ? tile_entry(I, J) : tile_entry(J, I)) + lane;
#pragma unroll
      for (int k = 0; k < 16; ++k) t[k] = tp[k * 64];
    } else {
      const double2 *tp = tiles + u.ent + tile_entry(I, I) + dsl;
#pragma unroll
      for (int k = 0; k < 16; ++k) t[k] = tp[k * kDiagSlots];
    }
  };
  auto load_x = [&](int J, int ks) {
    const double2 *xr = xb + (int64_t)(32 * J + 4 * ks + lk) * u.ld;
    x[NB * ks] = xr[c0];
    if constexpr (NB == 2) x[2 * ks + 1] = xr[c1];
  };
  v4d are[2][NB], aim[2][NB];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      are[i][j] = v4d{0.0, 0.0, 0.0, 0.0};
      aim[i][j] = v4d{0.0, 0.0, 0.0, 0.0};
    }
  load_tile(0);
#pragma unroll
  for (int ks = 0; ks < 8; ++ks) load_x(0, ks);
#pragma unroll 1
  for (int J = 0; J < nt; ++J) {
    const bool up = J >= I;
    // the lane holds stored entries (4a + i, 4q + j) at 4i + j; A_IJ is the
    // stored tile (J >= I) or the conjugate transpose of tile (J, I)
    wave_lds_fence();   // the tile before has been read
    if (J != I) {
      const double sg = up ? 1.0 : -1.0;
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int c = up ? 4 * q + j : 4 * a + i;
          const int m = up ? 4 * a + i : 4 * q + j;
          const double2 v = t[4 * i + j];
          buf[c * 33 + m] = make_double2(v.x, sg * v.y);
        }
    } else {
      // diagonal tile: lanes a <= q write their sub-block, lanes a < q also
      // its conjugate transpose below the diagonal
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int c = 4 * q + j, m = 4 * a + i;
          const double2 v = t[4 * i + j];
          if (dup) buf[c * 33 + m] = v;
          if (a < q) buf[m * 33 + c] = make_double2(v.x, -v.y);
        }
    }
    wave_lds_fence();
    const int Jn = min(J + 1, nt - 1);   // the loads after the last tile repeat it
    load_tile(Jn);
    __builtin_amdgcn_sched_barrier(0);
    double2 an[2] = {buf[lk * 33 + li], buf[lk * 33 + 16 + li]};
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) {
      const double2 ar[2] = {an[0], an[1]};
      if (ks < 7) {
        const int c = 4 * (ks + 1) + lk;
        an[0] = buf[c * 33 + li];
        an[1] = buf[c * 33 + 16 + li];
      }
      double2 xv[NB];
#pragma unroll
      for (int j = 0; j < NB; ++j) xv[j] = x[NB * ks + j];
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j)
          are[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(ar[i].x, xv[j].x, are[i][j], 0, 0, 0);
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j)
          aim[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(ar[i].x, xv[j].y, aim[i][j], 0, 0, 0);
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j)
          are[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(-ar[i].y, xv[j].y, are[i][j], 0, 0, 0);
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j)
          aim[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(ar[i].y, xv[j].x, aim[i][j], 0, 0, 0);
      load_x(Jn, ks);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  double2 *yb = yl + u.base + (int64_t)(32 * I) * u.ld;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      const int col = 16 * j + li;
      if (col >= u.nc) continue;
#pragma unroll
      for (int v = 0; v < 4; ++v)
        yb[(int64_t)(16 * i + 4 * v + lk) * u.ld + col] = make_double2(are[i][j][v], aim[i][j][v]);
    }
}

__global__ __launch_bounds__(64, 2) void k_rows_mfma64(const double2 *__restrict__ tiles,
                                                       const int2 *__restrict__ rows,
                                                       const ChunkMap cm,
                                                       const HermGroup *__restrict__ grp,
                                                       const double2 *__restrict__ xl,
                                                       double2 *__restrict__ yl, int nr) {
  __shared__ double2 buf[32 * 33];
  const RowUnit u = row_unit(rows, cm, grp, nr);
  if (!u.on) return;
  if (u.nc <= 16) rows64<16>(u, tiles, xl, yl, buf);
  else rows64<32>(u, tiles, xl, yl, buf);
}

// With FWD the result (d, k) also goes to the local rows of the next block
// set that hold d (its reduction lists), in that set's block buffers.
template <typename T, int MODE, bool FWD>
__global__ __launch_bounds__(256) void k_scatter_blk(int64_t nvec, int nr,
                                                     const int32_t *__restrict__ red_ptr,
                                                     const int32_t *__restrict__ red_ent,
                                                     const cplx_t<T> *__restrict__ yl,
                                                     const cplx_t<T> *__restrict__ r,
                                                     cplx_t<T> *__restrict__ y, T theta,
                                                     const int32_t *__restrict__ fwd_ptr,
                                                     const int32_t *__restrict__ fwd_ent,
                                                     cplx_t<T> *__restrict__ fwd_xl) {
  using C = cplx_t<T>;
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (e >= nvec * nr) return;
  const int64_t d = e / nr;
  const int k = (int)(e % nr);
  C acc = czero<C>();
  for (int32_t j = red_ptr[d]; j < red_ptr[d + 1]; ++j)
    acc = cadd(acc, yl[(int64_t)red_ent[j] * nr + k]);
  C out;
  if (MODE == RED_SET) out = acc;
  else if (MODE == RED_RESID) out = csub(r[e], acc);
  else if (MODE == RED_AXPY) out = cadd(y[e], cscale(acc, theta));
  else out = cscale(acc, theta);
  y[e] = out;
  if (FWD)
    for (int32_t j = fwd_ptr[d]; j < fwd_ptr[d + 1]; ++j)
      fwd_xl[(int64_t)fwd_ent[j] * nr + k] = out;
}

// Local vectors column by column ([nr][nloc]).
__global__ __launch_bounds__(256) void k_gather_cols(int64_t nloc, int nr,
                                                     const int32_t *__restrict__ gidx,
                                                     const double2 *__restrict__ x,
                                                     double2 *__restrict__ xl) {
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (e >= nloc * nr) return;
  const int64_t i = e % nloc;
  const int k = (int)(e / nloc);
  const int32_t g = gidx[i];
  xl[e] = g >= 0 ? x[(int64_t)g * nr + k] : czero<double2>();
}

template <int MODE>
__global__ __launch_bounds__(256) void k_scatter_cols(int64_t nvec, int64_t nloc, int nr,
                                                      const int32_t *__restrict__ red_ptr,
                                                      const int32_t *__restrict__ red_ent,
                                                      const double2 *__restrict__ yl,
                                                      const double2 *__restrict__ r,
                                                      double2 *__restrict__ y, double theta) {
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (e >= nvec * nr) return;
  const int64_t d = e / nr;
  const int k = (int)(e % nr);
  double2 acc = czero<double2>();
  for (int32_t j = red_ptr[d]; j < red_ptr[d + 1]; ++j)
    acc = cadd(acc, yl[(int64_t)k * nloc + red_ent[j]]);
  if (MODE == RED_SET) y[e] = acc;
  else if (MODE == RED_RESID) y[e] = csub(r[e], acc);
  else if (MODE == RED_AXPY) y[e] = cadd(y[e], cscale(acc, theta));
  else y[e] = cscale(acc, theta);
}

// ---- transfers and condensation ----------------------------------------------------------

template <typename T>
__global__ __launch_bounds__(256) void k_csr_blk(int64_t nrows, int nr,
                                                 const int64_t *__restrict__ ptr,
                                                 const int32_t *__restrict__ col,
                                                 const T *__restrict__ val,
                                                 const cplx_t<T> *__restrict__ x,
                                                 cplx_t<T> *__restrict__ y, int add) {
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (e >= nrows * nr) return;
  const int64_t i = e / nr;
  const int k = (int)(e % nr);
  cplx_t<T> acc = czero<cplx_t<T>>();
  for (int64_t j = ptr[i]; j < ptr[i + 1]; ++j)
    acc = cadd(acc, cscale(x[(int64_t)col[j] * nr + k], val[j]));
  y[e] = add ? cadd(y[e], acc) : acc;
}

// c_b[sl, k] = sum_i WH_b[sl, i] rc[I_b(i), k] for the KC columns of blockIdx.y and
// the 64 boundary slots of blockIdx.z, one per lane.  Bound by latency: a level has
// few blocks, and a lane's sum is one chain over the interior, so the slots of a
// block are spread over workgroups of one wave whose LDS holds only the interior
// values (WH is read once per KC columns, from a cache after the first).  Whole
// blocks in workgroups of 256 with 64 KB of LDS took 91 us for 64 blocks of order
// 169 + 434 and 8 columns in FP32, now 40 (216 blocks, 32 columns 168 / 111; 1728
// blocks, 32 columns in FP64 1840 / 1380).
template <typename T>
__global__ __launch_bounds__(64) void k_condense_local_blk(const cplx_t<T> *__restrict__ WH,
                                                           const int32_t *__restrict__ bcls,
                                                           int nI, int nBf,
                                                           const int32_t *__restrict__ blkI,
                                                           const cplx_t<T> *__restrict__ rc,
                                                           cplx_t<T> *__restrict__ c, int nr) {
  using C = cplx_t<T>;
  extern __shared__ __align__(16) char smem[];
  C(*rI)[KC] = reinterpret_cast<C(*)[KC]>(smem);
  const int b = blockIdx.x, k0 = blockIdx.y * KC, kc = min(KC, nr - k0);
  for (int e = threadIdx.x; e < nI * KC; e += 64) {
    const int i = e / KC, k = e % KC;
    rI[i][k] = k < kc ? rc[(int64_t)blkI[(int64_t)b * nI + i] * nr + k0 + k] : czero<C>();
  }
  __syncthreads();
  const int sl = blockIdx.z * 64 + threadIdx.x;
  if (sl >= nBf) return;
  const C *W = WH + (int64_t)bcls[b] * nBf * nI + sl;
  C acc[KC];
#pragma unroll
  for (int k = 0; k < KC; ++k) acc[k] = czero<C>();
#pragma unroll 8
  for (int i = 0; i < nI; ++i) {
    const C wv = W[(int64_t)i * nBf];
#pragma unroll
    for (int k = 0; k < KC; ++k) acc[k] = cfma(wv, rI[i][k], acc[k]);
  }
  for (int k = 0; k < kc; ++k) c[((int64_t)b * nBf + sl) * nr + k0 + k] = acc[k];
}

template <typename T>
__global__ __launch_bounds__(256) void k_condense_reduce_blk(int64_t nM, int nr,
                                                             const int64_t *__restrict__ macro_B,
                                                             const int32_t *__restrict__ red_ptr,
                                                             const int32_t *__restrict__ red_ent,
                                                             const cplx_t<T> *__restrict__ rc,
                                                             const cplx_t<T> *__restrict__ c,
                                                             cplx_t<T> *__restrict__ rB) {
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (e >= nM * nr) return;
  const int64_t m = e / nr;
  const int k = (int)(e % nr);
  cplx_t<T> acc = rc[macro_B[m] * nr + k];
  for (int32_t j = red_ptr[m]; j < red_ptr[m + 1]; ++j)
    acc = csub(acc, c[(int64_t)red_ent[j] * nr + k]);
  rB[e] = acc;
}

template <typename C> __device__ inline C wave_sum_c(C v) {
  for (int o = 32; o > 0; o >>= 1) {
    v.x += __shfl_xor(v.x, o, 64);
    v.y += __shfl_xor(v.y, o, 64);
  }
  return v;
}

template <typename T>
__global__ __launch_bounds__(256) void k_scatter_macro_blk(int64_t nM, int nr,
                                                           const int64_t *__restrict__ macro_B,
                                                           const cplx_t<T> *__restrict__ eB,
                                                           cplx_t<T> *__restrict__ ec) {
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (e < nM * nr) ec[macro_B[e / nr] * nr + e % nr] = eB[e];
}

// ec[I_b(i), k] = sum_j conj(Tinv[j, i]) rc[I_b(j), k] - sum_sl conj(WH[sl, i]) eB_b[sl, k],
// one wave per interior unknown i at a time, KC columns (blockIdx.y) and the rows of
// blockIdx.z per workgroup.  A coarse level has few blocks, so their rows are spread
// over workgroups until the chip is full: 64 blocks of order 169 + 434, 8 columns in
// FP32, 239 us with all rows in one workgroup, now 36; 27 blocks, 3 columns in FP64
// 253 / 34.  (Four rows per wave at a time, which reads the LDS values once for all,
// needed twice the registers: 216 blocks, 32 columns 551 us, 266 so.)
template <typename T>
__global__ __launch_bounds__(256) void k_expand_blk(const cplx_t<T> *__restrict__ WH,
                                                    const cplx_t<T> *__restrict__ Tinv,
                                                    const int32_t *__restrict__ bcls, int nI,
                                                    int nBf, const int32_t *__restrict__ blkI,
                                                    const int32_t *__restrict__ blkBm,
                                                    const cplx_t<T> *__restrict__ rc,
                                                    const cplx_t<T> *__restrict__ eB,
                                                    cplx_t<T> *__restrict__ ec, int nr, int rows) {
  using C = cplx_t<T>;
  extern __shared__ __align__(16) char smem[];
  C(*eBs)[KC] = reinterpret_cast<C(*)[KC]>(smem);
  C(*rIs)[KC] = reinterpret_cast<C(*)[KC]>(smem + sizeof(C) * KC * nBf);
  const int b = blockIdx.x, k0 = blockIdx.y * KC, kc = min(KC, nr - k0);
  for (int e = threadIdx.x; e < nBf * KC; e += 256) {
    const int sl = e / KC, k = e % KC;
    const int m = blkBm[(int64_t)b * nBf + sl];
    eBs[sl][k] = (m >= 0 && k < kc) ? eB[(int64_t)m * nr + k0 + k] : czero<C>();
  }
  for (int e = threadIdx.x; e < nI * KC; e += 256) {
    const int i = e / KC, k = e % KC;
    rIs[i][k] = k < kc ? rc[(int64_t)blkI[(int64_t)b * nI + i] * nr + k0 + k] : czero<C>();
  }
  __syncthreads();
  const C *W = WH + (int64_t)bcls[b] * nBf * nI;
  const C *Ti = Tinv + (int64_t)bcls[b] * nI * nI;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int r1 = min(nI, ((int)blockIdx.z + 1) * rows);
  for (int i = blockIdx.z * rows + wave; i < r1; i += 4) {
    C acc[KC];
#pragma unroll
    for (int k = 0; k < KC; ++k) acc[k] = czero<C>();
    for (int j = lane; j < nI; j += 64) {
      const C tv = cconj(Ti[j + (int64_t)i * nI]);
#pragma unroll
      for (int k = 0; k < KC; ++k) acc[k] = cfma(tv, rIs[j][k], acc[k]);
    }
    for (int sl = lane; sl < nBf; sl += 64) {
      const C wv = cconj(W[sl + (int64_t)i * nBf]);
#pragma unroll
      for (int k = 0; k < KC; ++k) acc[k] = csub(acc[k], cmul(wv, eBs[sl][k]));
    }
#pragma unroll
    for (int k = 0; k < KC; ++k) acc[k] = wave_sum_c(acc[k]);
    if (lane < kc) {
      C v = acc[0];
#pragma unroll
      for (int k = 1; k < KC; ++k)
        if (lane == k) v = acc[k];
      ec[(int64_t)blkI[(int64_t)b * nI + i] * nr + k0 + lane] = v;
    }
  }
}

__global__ __launch_bounds__(256) void k_interleave(int64_t n, int nr, const double2 *__restrict__ cols,
                                                    double2 *__restrict__ blk, int dir) {
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (e >= n * nr) return;
  const int64_t d = e / nr;
  const int k = (int)(e % nr);
  if (dir == 0) blk[e] = cols[(int64_t)k * n + d];
  else blk[(int64_t)k * n + d] = cols[e];
}

// Column k of an interleaved block of width w: set from a plain vector (or
// zero), or copied out.
__global__ __launch_bounds__(256) void k_col(int64_t n, int w, int k, const double2 *__restrict__ src,
                                             double2 *__restrict__ dst, int dir) {
  const int64_t d = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (d >= n) return;
  if (dir == 0) dst[d * w + k] = src ? src[d] : mk(0.0, 0.0);
  else dst[d] = src[d * w + k];
}

// dst (width w_new) <- src (width w_old): columns k < min(w_old, w_new) kept,
// new columns zero.
__global__ __launch_bounds__(256) void k_rewidth(int64_t n, int w_old, int w_new,
                                                 const double2 *__restrict__ src,
                                                 double2 *__restrict__ dst) {
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (e >= n * w_new) return;
  const int64_t d = e / w_new;
  const int k = (int)(e % w_new);
  dst[e] = k < w_old ? src[d * w_old + k] : mk(0.0, 0.0);
}

// A column joining a block solve: rz = 1 (so that its first flexible beta is
// finite; it multiplies a zero search direction), every other scalar 0.
__global__ void k_col_reset(double *sc, int k) {
  const int q = threadIdx.x;
  if (q < 8) sc[q * kMaxCols + k] = q == 0 ? 1.0 : 0.0;
}

// ---- per-column CG --------------------------------------------------------------------

// Per workgroup and column: sums of Re(a^H b) (and Re(a^H c) when c).
__global__ __launch_bounds__(256) void k_coldot(int64_t n, int nr, const double2 *__restrict__ a,
                                                const double2 *__restrict__ bv,
                                                const double2 *__restrict__ cv,
                                                double *__restrict__ partial) {
  __shared__ double sh[2][256];
  const int t = threadIdx.x, rpb = 256 / nr, k = t % nr;
  const bool on = t < rpb * nr;
  double s = 0.0, u = 0.0;
  if (on)
#pragma unroll 4
    for (int64_t i = (int64_t)blockIdx.x * rpb + t / nr; i < n; i += (int64_t)gridDim.x * rpb) {
      const double2 x = a[i * nr + k], y = bv[i * nr + k];
      s += x.x * y.x + x.y * y.y;
      if (cv) {
        const double2 z = cv[i * nr + k];
        u += x.x * z.x + x.y * z.y;
      }
    }
  sh[0][t] = s;
  sh[1][t] = u;
  __syncthreads();
  if (t < nr) {
    double ss = 0.0, uu = 0.0;
    for (int j = 0; j < rpb; ++j) {
      ss += sh[0][t + j * nr];
      uu += sh[1][t + j * nr];
    }
    partial[(int64_t)blockIdx.x * kMaxCols + t] = ss;
    partial[(int64_t)(kColDotBlocks + blockIdx.x) * kMaxCols + t] = uu;
  }
}

// Column reductions and the scalar updates of the CG step (mode: 0 store the
// dot in slot q, 1 alpha, 2 ||r||^2, 3 flexible beta).  One column's partials are
// added in order by one lane; they come through LDS, kFinRows at a time, so that the
// chain waits for LDS and not for memory (15 us, now 7).
constexpr int kFinRows = 64;
__global__ __launch_bounds__(256) void k_colfinal(const double *__restrict__ partial, int nr,
                                                  double *__restrict__ sc,
                                                  const int *__restrict__ act, int mode, int q) {
  __shared__ double sh[2][kFinRows][kMaxCols];
  const int k = threadIdx.x;
  double s = 0.0, u = 0.0;
  for (int j0 = 0; j0 < kColDotBlocks; j0 += kFinRows) {
    double v[kFinRows * kMaxCols / 256], w[kFinRows * kMaxCols / 256];
#pragma unroll
    for (int e = 0; e < kFinRows * kMaxCols / 256; ++e) {
      const int64_t at = (int64_t)j0 * kMaxCols + e * 256 + threadIdx.x;
      v[e] = partial[at];
      w[e] = mode == 3 ? partial[(int64_t)kColDotBlocks * kMaxCols + at] : 0.0;
    }
    if (j0) __syncthreads();
#pragma unroll
    for (int e = 0; e < kFinRows * kMaxCols / 256; ++e) {
      (&sh[0][0][0])[e * 256 + threadIdx.x] = v[e];
      (&sh[1][0][0])[e * 256 + threadIdx.x] = w[e];
    }
    __syncthreads();
    if (k < nr) {
#pragma unroll 16
      for (int j = 0; j < kFinRows; ++j) {
        s += sh[0][j][k];
        u += sh[1][j][k];
      }
    }
  }
  if (k >= nr) return;
  double *S = sc;
  const bool on = act ? act[k] != 0 : true;
  if (mode == 0) {
    S[q * kMaxCols + k] = s;
  } else if (mode == 1) {
    S[1 * kMaxCols + k] = s;
    if (on && (!(s > 0.0) || !isfinite(s))) S[6 * kMaxCols + k] = 1.0;
    S[2 * kMaxCols + k] = on ? S[0 * kMaxCols + k] / s : 0.0;
  } else if (mode == 2) {
    S[4 * kMaxCols + k] = s;
  } else {
    // flexible (Polak-Ribiere) beta = Re(r^H (z - z_old)) / Re(r_old^H z_old)
    const double beta = on ? (s - u) / S[0 * kMaxCols + k] : 0.0;
    S[3 * kMaxCols + k] = beta;
    S[7 * kMaxCols + k] = u;
    S[0 * kMaxCols + k] = s;
    if (on && !isfinite(beta)) S[6 * kMaxCols + k] = 1.0;
  }
}

__global__ __launch_bounds__(256) void k_update_xr_blk(int64_t n, int nr, double2 *__restrict__ x,
                                                       double2 *__restrict__ r,
                                                       const double2 *__restrict__ p,
                                                       const double2 *__restrict__ qv,
                                                       double *__restrict__ partial,
                                                       const double *__restrict__ sc) {
  __shared__ double sh[256];
  const int t = threadIdx.x, rpb = 256 / nr, k = t % nr;
  const bool on = t < rpb * nr;
  const double al = on ? sc[2 * kMaxCols + k] : 0.0;
  double s = 0.0;
  if (on)
    for (int64_t i = (int64_t)blockIdx.x * rpb + t / nr; i < n; i += (int64_t)gridDim.x * rpb) {
      const int64_t e = i * nr + k;
      x[e] = mk(x[e].x + al * p[e].x, x[e].y + al * p[e].y);
      const double2 ri = mk(r[e].x - al * qv[e].x, r[e].y - al * qv[e].y);
      r[e] = ri;
      s += ri.x * ri.x + ri.y * ri.y;
    }
  sh[t] = s;
  __syncthreads();
  if (t < nr) {
    double ss = 0.0;
    for (int j = 0; j < rpb; ++j) ss += sh[t + j * nr];
    partial[(int64_t)blockIdx.x * kMaxCols + t] = ss;
    partial[(int64_t)(kColDotBlocks + blockIdx.x) * kMaxCols + t] = 0.0;
  }
}

__global__ __launch_bounds__(256) void k_update_p_blk(int64_t n, int nr, double2 *__restrict__ p,
                                                      const double2 *__restrict__ z,
                                                      const double *__restrict__ sc) {
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (e >= n * nr) return;
  const double be = sc[3 * kMaxCols + (int)(e % nr)];
  p[e] = mk(z[e].x + be * p[e].x, z[e].y + be * p[e].y);
}

}  // namespace

void HermBlockBufs::ensure(const HermSet &H, int nr, bool fp64, bool fp32, Budget *bud,
                           hipStream_t s) {
  if (nr <= cap) return;
  if (fp64) {
    xl64.alloc(H.nloc * nr, bud);
    yl64.alloc(H.nloc * nr, bud);
    launch_zero(H.nloc * nr, xl64.p, s);
  }
  if (fp32) {
    xl32.alloc(H.nloc * nr, bud);
    yl32.alloc(H.nloc * nr, bud);
    launch_zero(H.nloc * nr, xl32.p, s);
  }
  cap = nr;
}

// (not in mixed precision, whose solutions feel the last bit of the outer iteration)
bool units_for(const HermSet &H, int nr) {
  return H.t64.p && !H.t32.p && H.gnunits64 == 0 && nr > 1 && nr <= kUnitCols &&
         H.npart * nr <= kPartMost;
}

template <typename T>
void launch_rows(HermSet &H, const cplx_t<T> *xl, cplx_t<T> *yl, int nr, hipStream_t s) {
  constexpr bool F64 = sizeof(T) == 8;
  const int64_t *cw = H.nrow_w;
  // chunk c: the units of the groups with more than 32 c columns
  ChunkMap cm;
  int64_t total = 0;
  for (int c = 0; c < kMaxGroup; ++c) {
    const int w = 32 * c / nr + 1;
    if (w > kMaxGroup || cw[w] == 0) break;
    cm.cnt[c] = (int32_t)cw[w];
    total += cw[w];
  }
  const int64_t per = (total + 7) / 8;
  if (8 * per > INT32_MAX) throw DpgError(-1, "block apply: too many tile rows");
  cm.total = (int32_t)total;
  ProfScope ps(H.prof, F64 ? DPG_K_APPLYB64 : DPG_K_APPLYB32,
               8.0 * (double)H.full * nr, s);
  if constexpr (F64)
    hipLaunchKernelGGL(k_rows_mfma64, dim3((unsigned)(8 * per)), dim3(64), 0, s, H.t64.p, H.grow.p,
                       cm, H.grp.p, xl, yl, nr);
  else
    hipLaunchKernelGGL(k_rows_mfma, dim3((unsigned)(8 * per)), dim3(64), 0, s, H.t32.p, H.grow.p,
                       cm, H.grp.p, xl, yl, nr);
  LAUNCH_OK();
}

template <typename T, int MODE>
void launch_scatter_blk(const HermSet &H, int nr, const cplx_t<T> *yl, const cplx_t<T> *R,
                        cplx_t<T> *Y, T theta, const HermSet *fwd, cplx_t<T> *fxl,
                        hipStream_t s) {
  const dim3 g(cdiv(H.nvec * nr, 256));
  if (fwd)
    hipLaunchKernelGGL((k_scatter_blk<T, MODE, true>), g, dim3(256), 0, s, H.nvec, nr,
                       H.red_ptr.p, H.red_ent.p, yl, R, Y, theta, fwd->red_ptr.p,
                       fwd->red_ent.p, fxl);
  else
    hipLaunchKernelGGL((k_scatter_blk<T, MODE, false>), g, dim3(256), 0, s, H.nvec, nr,
                       H.red_ptr.p, H.red_ent.p, yl, R, Y, theta, nullptr, nullptr, nullptr);
}

template <typename T>
void herm_apply_blk(HermSet &H, HermBlockBufs &W, const cplx_t<T> *X, cplx_t<T> *Y,
                    const cplx_t<T> *R, int mode, T theta, int nr, hipStream_t s, bool gathered,
                    HermSet *fwd, HermBlockBufs *fwd_bufs) {
  if (nr < 1 || nr > kMaxCols || nr > W.cap) throw DpgError(-1, "block apply: bad column count");
  if (nr == 1) {   // one column: the HBM-bound single-vector apply (same layout)
    herm_apply<T>(H, X, Y, R, mode, theta, s, gathered, fwd);
    return;
  }
  cplx_t<T> *fxl = nullptr;
  if (fwd) {
    if (!fwd_bufs || fwd->nvec != H.nvec || nr > fwd_bufs->cap)
      throw DpgError(-1, "forwarded block set does not match this one");
    if constexpr (sizeof(T) == 8) fxl = fwd_bufs->xl64.p;
    else fxl = fwd_bufs->xl32.p;
    if (!fxl) throw DpgError(-1, "forwarded block set has no local vectors of this precision");
  }
  const cplx_t<T> *tiles;
  cplx_t<T> *xl, *yl;
  if constexpr (sizeof(T) == 8) {
    tiles = H.t64.p;
    xl = W.xl64.p;
    yl = W.yl64.p;
  } else {
    tiles = H.t32.p;
    xl = W.xl32.p;
    yl = W.yl32.p;
  }
  if (!tiles || !xl) throw DpgError(-6, "block set has no tiles of this precision");
  if (!gathered) {
    ProfScope ps(H.prof, DPG_K_REDUCE, 0.0, s);
    hipLaunchKernelGGL((k_gather_blk<T>), dim3(cdiv(H.nloc * nr, 256)), dim3(256), 0, s, H.nloc,
                       nr, H.gidx.p, X, xl);
    LAUNCH_OK();
  }
  bool rows = true;
  if constexpr (sizeof(T) == 8) {
    if (W.part && units_for(H, nr)) {
      const bool own = W.part->n < H.max_slots;   // (also: of a larger block than it holds)
      launch_units_cols(H, xl, own ? H.p64.p : W.part->p, own ? H.npart : W.part->n, yl, nr, s);
      rows = false;
    }
  }
  if (rows) launch_rows<T>(H, xl, yl, nr, s);
  ProfScope ps(H.prof, DPG_K_REDUCE, 0.0, s);
  switch (mode) {
    case RED_SET: launch_scatter_blk<T, RED_SET>(H, nr, yl, R, Y, theta, fwd, fxl, s); break;
    case RED_RESID: launch_scatter_blk<T, RED_RESID>(H, nr, yl, R, Y, theta, fwd, fxl, s); break;
    case RED_AXPY: launch_scatter_blk<T, RED_AXPY>(H, nr, yl, R, Y, theta, fwd, fxl, s); break;
    default: launch_scatter_blk<T, RED_SET_SCALED>(H, nr, yl, R, Y, theta, fwd, fxl, s);
  }
  LAUNCH_OK();
}

void herm_gather_cols(const HermSet &H, const double2 *X, double2 *xl, int nr, hipStream_t s) {
  if (nr < 1 || nr > kMaxCols) throw DpgError(-1, "column gather: bad column count");
  ProfScope ps(H.prof, DPG_K_REDUCE, 0.0, s);
  hipLaunchKernelGGL(k_gather_cols, dim3(cdiv(H.nloc * nr, 256)), dim3(256), 0, s, H.nloc, nr,
                     H.gidx.p, X, xl);
  LAUNCH_OK();
}

void herm_scatter_cols(const HermSet &H, const double2 *yl, double2 *Y, const double2 *R,
                       int mode, double theta, int nr, hipStream_t s) {
  if (nr < 1 || nr > kMaxCols) throw DpgError(-1, "column scatter: bad column count");
  ProfScope ps(H.prof, DPG_K_REDUCE, 0.0, s);
  const dim3 g(cdiv(H.nvec * nr, 256));
  switch (mode) {
    case RED_SET:
      hipLaunchKernelGGL((k_scatter_cols<RED_SET>), g, dim3(256), 0, s, H.nvec, H.nloc, nr, H.red_ptr.p, H.red_ent.p, yl, R, Y, theta);
      break;
    case RED_RESID:
      hipLaunchKernelGGL((k_scatter_cols<RED_RESID>), g, dim3(256), 0, s, H.nvec, H.nloc, nr, H.red_ptr.p, H.red_ent.p, yl, R, Y, theta);
      break;
    case RED_AXPY:
      hipLaunchKernelGGL((k_scatter_cols<RED_AXPY>), g, dim3(256), 0, s, H.nvec, H.nloc, nr, H.red_ptr.p, H.red_ent.p, yl, R, Y, theta);
      break;
    default:
      hipLaunchKernelGGL((k_scatter_cols<RED_SET_SCALED>), g, dim3(256), 0, s, H.nvec, H.nloc, nr, H.red_ptr.p, H.red_ent.p, yl, R, Y, theta);
  }
  LAUNCH_OK();
}

template <typename T>
void launch_csr_blk(int64_t nrows, const int64_t *ptr, const int32_t *col, const T *val,
                    const cplx_t<T> *x, cplx_t<T> *y, int add, int nr, hipStream_t s) {
  if (nrows <= 0) return;
  hipLaunchKernelGGL((k_csr_blk<T>), dim3(cdiv(nrows * nr, 256)), dim3(256), 0, s, nrows, nr, ptr,
                     col, val, x, y, add);
  LAUNCH_OK();
}

template <typename T>
void launch_condense_blk(const cplx_t<T> *WH, const int32_t *bcls, int nI, int nBf,
                         const int32_t *blkI, int nblk, int64_t nM, const int64_t *macro_B,
                         const int32_t *red_ptr,
                         const int32_t *red_ent, const cplx_t<T> *rc, cplx_t<T> *c,
                         cplx_t<T> *rB, int nr, hipStream_t s) {
  if (nI > kBMaxI) throw DpgError(-1, "macro block too large");
  // 64 KB of LDS at most: kBMaxI interior unknowns in FP64
  hipLaunchKernelGGL((k_condense_local_blk<T>), dim3(nblk, cdiv(nr, KC), cdiv(nBf, 64)), dim3(64),
                     sizeof(cplx_t<T>) * KC * nI, s, WH, bcls, nI, nBf, blkI, rc, c, nr);
  LAUNCH_OK();
  hipLaunchKernelGGL((k_condense_reduce_blk<T>), dim3(cdiv(nM * nr, 256)), dim3(256), 0, s, nM, nr,
                     macro_B, red_ptr, red_ent, rc, c, rB);
  LAUNCH_OK();
}

constexpr int64_t kExpandWgs = 2048;

template <typename T>
void launch_expand_blk(const cplx_t<T> *WH, const cplx_t<T> *Tinv, const int32_t *bcls, int nI,
                       int nBf, const int32_t *blkI, const int32_t *blkBm, int nblk,
                       const cplx_t<T> *rc, const cplx_t<T> *eB, int64_t nM,
                       const int64_t *macro_B, cplx_t<T> *ec, int nr, hipStream_t s) {
  // the boundary and interior values of KC columns of one macro block stay in
  // LDS; beyond 64 KB (order 4 in FP64) the kernel asks for more, up to the
  // 160 KB a gfx950 workgroup can hold
  const size_t lds = sizeof(cplx_t<T>) * KC * ((size_t)nBf + nI);
  if (lds > 160 * 1024) throw DpgError(-1, "macro block too large for the block expansion");
  if (lds > 64 * 1024)
    HIP_OK(hipFuncSetAttribute(reinterpret_cast<const void *>(&k_expand_blk<T>),
                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
  hipLaunchKernelGGL((k_scatter_macro_blk<T>), dim3(cdiv(nM * nr, 256)), dim3(256), 0, s, nM, nr,
                     macro_B, eB, ec);
  LAUNCH_OK();
  // rows of a workgroup, in sixteens: workgroups enough to fill the chip eight deep
  // (27 blocks, 32 columns: 65 us at four deep, 51 at eight)
  const int64_t wgs = (int64_t)nblk * cdiv(nr, KC), want = cdiv(kExpandWgs, wgs);
  const int rows = (int)std::max<int64_t>(16, 16 * cdiv(cdiv(nI, 16), want));
  hipLaunchKernelGGL((k_expand_blk<T>), dim3(nblk, cdiv(nr, KC), cdiv(nI, rows)), dim3(256), lds, s,
                     WH, Tinv, bcls, nI, nBf, blkI, blkBm, rc, eB, ec, nr, rows);
  LAUNCH_OK();
}

void launch_interleave(int64_t n, int nr, const double2 *cols, double2 *blk, hipStream_t s) {
  hipLaunchKernelGGL(k_interleave, dim3(cdiv(n * nr, 256)), dim3(256), 0, s, n, nr, cols, blk, 0);
  LAUNCH_OK();
}
void launch_deinterleave(int64_t n, int nr, const double2 *blk, double2 *cols, hipStream_t s) {
  hipLaunchKernelGGL(k_interleave, dim3(cdiv(n * nr, 256)), dim3(256), 0, s, n, nr, blk, cols, 1);
  LAUNCH_OK();
}

void launch_set_col(int64_t n, int w, int k, const double2 *src, double2 *blk, hipStream_t s) {
  if (n <= 0) return;
  hipLaunchKernelGGL(k_col, dim3(cdiv(n, 256)), dim3(256), 0, s, n, w, k, src, blk, 0);
  LAUNCH_OK();
}
void launch_get_col(int64_t n, int w, int k, const double2 *blk, double2 *dst, hipStream_t s) {
  if (n <= 0) return;
  hipLaunchKernelGGL(k_col, dim3(cdiv(n, 256)), dim3(256), 0, s, n, w, k, blk, dst, 1);
  LAUNCH_OK();
}
void launch_rewidth(int64_t n, int w_old, int w_new, const double2 *src, double2 *dst,
                    hipStream_t s) {
  if (n <= 0) return;
  hipLaunchKernelGGL(k_rewidth, dim3(cdiv(n * w_new, 256)), dim3(256), 0, s, n, w_old, w_new,
                     src, dst);
  LAUNCH_OK();
}
void cgb_reset_col(double *sc, int k, hipStream_t s) {
  hipLaunchKernelGGL(k_col_reset, dim3(1), dim3(64), 0, s, sc, k);
  LAUNCH_OK();
}

void cgb_dot(int64_t n, int nr, const double2 *a, const double2 *b, double *partial, double *sc,
             int q, hipStream_t s) {
  hipLaunchKernelGGL(k_coldot, dim3(kColDotBlocks), dim3(256), 0, s, n, nr, a, b,
                     (const double2 *)nullptr, partial);
  hipLaunchKernelGGL(k_colfinal, dim3(1), dim3(256), 0, s, partial, nr, sc, (const int *)nullptr, 0,
                     q);
  LAUNCH_OK();
}

void cgb_alpha(int64_t n, int nr, const double2 *p, const double2 *qv, double *partial,
               double *sc, const int *act, hipStream_t s) {
  hipLaunchKernelGGL(k_coldot, dim3(kColDotBlocks), dim3(256), 0, s, n, nr, p, qv,
                     (const double2 *)nullptr, partial);
  hipLaunchKernelGGL(k_colfinal, dim3(1), dim3(256), 0, s, partial, nr, sc, act, 1, 0);
  LAUNCH_OK();
}

void cgb_update_xr(int64_t n, int nr, double2 *x, double2 *r, const double2 *p, const double2 *qv,
                   double *partial, double *sc, hipStream_t s) {
  hipLaunchKernelGGL(k_update_xr_blk, dim3(kColDotBlocks), dim3(256), 0, s, n, nr, x, r, p, qv,
                     partial, sc);
  hipLaunchKernelGGL(k_colfinal, dim3(1), dim3(256), 0, s, partial, nr, sc, (const int *)nullptr, 2,
                     0);
  LAUNCH_OK();
}

void cgb_beta(int64_t n, int nr, const double2 *r, const double2 *z, const double2 *zold,
              double *partial, double *sc, const int *act, hipStream_t s) {
  hipLaunchKernelGGL(k_coldot, dim3(kColDotBlocks), dim3(256), 0, s, n, nr, r, z, zold, partial);
  hipLaunchKernelGGL(k_colfinal, dim3(1), dim3(256), 0, s, partial, nr, sc, act, 3, 0);
  LAUNCH_OK();
}

void cgb_update_p(int64_t n, int nr, double2 *p, const double2 *z, const double *sc,
                  hipStream_t s) {
  hipLaunchKernelGGL(k_update_p_blk, dim3(cdiv(n * nr, 256)), dim3(256), 0, s, n, nr, p, z, sc);
  LAUNCH_OK();
}

template void launch_rows<double>(HermSet &, const double2 *, double2 *, int, hipStream_t);
template void launch_rows<float>(HermSet &, const float2 *, float2 *, int, hipStream_t);
template void herm_apply_blk<double>(HermSet &, HermBlockBufs &, const double2 *, double2 *,
                                     const double2 *, int, double, int, hipStream_t, bool,
                                     HermSet *, HermBlockBufs *);
template void herm_apply_blk<float>(HermSet &, HermBlockBufs &, const float2 *, float2 *,
                                    const float2 *, int, float, int, hipStream_t, bool,
                                    HermSet *, HermBlockBufs *);
template void launch_csr_blk<double>(int64_t, const int64_t *, const int32_t *, const double *,
                                     const double2 *, double2 *, int, int, hipStream_t);
template void launch_csr_blk<float>(int64_t, const int64_t *, const int32_t *, const float *,
                                    const float2 *, float2 *, int, int, hipStream_t);
template void launch_condense_blk<double>(const double2 *, const int32_t *, int, int,
                                          const int32_t *, int, int64_t, const int64_t *,
                                          const int32_t *, const int32_t *, const double2 *,
                                          double2 *, double2 *, int, hipStream_t);
template void launch_condense_blk<float>(const float2 *, const int32_t *, int, int,
                                         const int32_t *, int, int64_t, const int64_t *,
                                         const int32_t *, const int32_t *, const float2 *,
                                         float2 *, float2 *, int, hipStream_t);
template void launch_expand_blk<double>(const double2 *, const double2 *, const int32_t *, int,
                                        int, const int32_t *, const int32_t *, int,
                                        const double2 *, const double2 *, int64_t,
                                        const int64_t *, double2 *, int, hipStream_t);
template void launch_expand_blk<float>(const float2 *, const float2 *, const int32_t *, int, int,
                                       const int32_t *, const int32_t *, int, const float2 *,
                                       const float2 *, int64_t, const int64_t *, float2 *, int,
                                       hipStream_t);

}  // namespace dpg
