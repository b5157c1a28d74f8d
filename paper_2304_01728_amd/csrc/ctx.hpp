// Internal context of libdpgmg.
#pragma once
#include <chrono>
#include <memory>
#include <string>
#include <vector>

#include "../../include/dpgmg.h"
#include "block.hpp"
#include "common.hpp"
#include "dense.hpp"
#include "element.hpp"
#include "hblocks.hpp"
#include "kernels.hpp"
#include "topology.hpp"

namespace dpg {

// Classes of equal matrices.  All elements are translated copies of one box, so
// two of them with the same wave speed and the same faces on Gamma have equal
// element matrices; two macro blocks with equal children (and two patches with
// equal blocks around them) are equal in turn.  Each class is computed and
// stored once, by the arithmetic its first member would go through alone, so
// the matrices are bit for bit those of a setup without classes.  Classes are
// numbered by their first members; with too little to share (more than three
// quarters as many classes as members) every member is a class of its own.
struct Classes {
  int n = 0;                         // classes
  std::vector<int32_t> of_h, rep_h;  // class of each member; first member of each class
  const int32_t *of = nullptr, *rep = nullptr;   // the same on the device (dpg_ctx::classes)
  bool shared() const { return n < (int)of_h.size(); }
};

// Prepared once per mesh (and per number of loads): item tables on the device
// and fixed workspaces, so that the setup phases only queue kernels.

// Loads of the elements of one chunk of element classes: a range of the
// elements sorted by class, with the items of the products and solves by the
// chunk's factors (one item per class of the chunk, some without columns).
struct LoadPiece {
  int chunk = 0, j0 = 0, cnt = 0, max_cols = 0;
  DevBuf<TrsmItem> tl, tk;
  DevBuf<GemmItem> gl, gs, gr;
};

// Element stage: chunks of C elements are dealt to ns streams, each with its
// own G, [B l], K and diagonal-block-inverse buffers.
struct ElemPlan {
  int C = 0, mp = -1, nel = -1, ns = 2;
  DevBuf<double2> G[4], BL[4], K[4], wk[4];   // one set per stream
  DevBuf<PotrfItem> pG, pK;
  DevBuf<TrsmItem> tG, tK;
  DevBuf<GemmItem> gK, gS;
  DevBuf<int> info;    // [2 nel]: Gram factor, then field block, per element
  // error-indicator pass: per-stream element unknowns [C][nr][m] and the
  // residual products' items (for gR_nr columns, chunks of gR_C)
  DevBuf<double2> X[4];
  DevBuf<GemmItem> gR;
  int gR_nr = 0, gR_C = 0, gR_mp = 0;
  // with shared classes (nel = their number, mp = m): the loads by pieces
  DevBuf<double2> LB[4], KL[4], wkK[4];
  DevBuf<int32_t> mlist;             // elements sorted by class
  std::vector<LoadPiece> pieces;
  int pieces_nr = -1, pieces_C = 0;
};

// Load updates by maps per element class.  Elements with equal wave speed and
// the same faces on Gamma have equal G and B (translated boxes), so one linear
// map T_c takes an element's load vector l (over the test functions) to its
// condensed trace load s = K_tl - K_tf K_ff^-1 K_fl, and F_c to its
// field-recovery data L_f^-1 K_fl; both are formed once by the element chain
// with identity load columns on one element of each class.
struct LoadMaps {
  int state = 0;                     // 0 not built, 1 built, -1 not used (too many classes)
  int nclass = 0;
  std::vector<int32_t> cls_h;        // class of every finest element
  DevBuf<double2> T, F;              // [nclass] n_tr x n_test, n_field x n_test (column-major)
  DevBuf<double2> lbuf;              // load vectors of a chunk of elements [C][nr][n_test]
  DevBuf<GemmItem> items;            // per update: s_e = T_c l_e, then Yb_e = F_c l_e
};

// Macro condensation and Galerkin step of one level (workspaces shared by
// all levels: the levels run one after the other on one stream).
struct MacroPlan {
  bool ready = false;
  int CB = 0;
  DevBuf<double2> Ploc;
  DevBuf<PotrfItem> pII;
  DevBuf<TrsmItem> tIB, tLi;
  DevBuf<GemmItem> gS, gTi, gWH, gX, gA;
  DevBuf<int64_t> idoff, soff, moff;
  DevBuf<int32_t> idn, cmap, sld, map;
  DevBuf<int> info;    // [block classes]
};

// Patch factors and inverses of one level, in batches that fit the patch
// workspaces.
struct PatchBatch {
  int half = 0;                      // part: 0 .. 2 on the extra streams, 3 on the main
                                     // stream (each part with its own workspaces)
  int v0 = 0, cnt = 0, nmax = 0;     // patch classes v0 .. v0 + cnt - 1
  int64_t t0 = 0, t1 = 0;
  double fp = 0, ft = 0, fg = 0;
  DevBuf<int64_t> off;
  DevBuf<int32_t> nn;
  std::vector<int32_t> hn;           // the orders nn on the host (kernel statistics)
  DevBuf<PotrfItem> pi;
  DevBuf<TrsmItem> ti;
  DevBuf<GemmItem> gi;
  DevBuf<GemmItem> gyc, gzc;         // recomputed inverses, t = X x_v and y_v = X^H t for
                                     // nr = 1 .. kMaxCols columns stored column by
                                     // column: items (nr - 1) mcnt + i over the
                                     // patches of the batch's classes
  int mcnt = 0;
};
struct PatchPlan {
  bool ready = false;
  std::vector<PatchBatch> batches;
  DevBuf<int64_t> soff_all;
  DevBuf<int32_t> ld_all;
  DevBuf<int> info;    // [patch classes]
};

// One mesh of the hierarchy.  Level 0 is the coarsest mesh, level L the finest.
struct LevelData {
  int N = 0, nel = 0;
  int q = 0, ntr = 0, ntr_c = 0;     // order, element trace size, that of the coarser level
  bool order = false;                // the coarser level has the same mesh (order q - 1)
  ElementLayout el;
  Numbering num;
  std::vector<int32_t> edofs_h;
  DevBuf<int4> lists;                // the index and value lists below
  DevList<int32_t> edofs;
  Classes ec, bc, pc;                // of the elements, macro blocks and vertex patches
  DevBuf<double2> E;                 // element matrices [ec.n][n_tr^2]
  DevBuf<double> kappa, Zel;         // per element c^-2 and Z on a coarser mesh whose
                                     // operator is assembled directly ("store")
  // macro grid (levels >= 1)
  bool macro = false;
  MacroLevel mc;
  Prolongation P;
  int nblk = 0, nBf = 0, nI = 0;
  int64_t nM = 0;
  DevBuf<double2> Mfull;             // [bc.n][nBf^2] condensed blocks, full local layout
  DevBuf<double2> Tinv, WH;          // [bc.n][nI^2], [bc.n][nBf nI]
  DevBuf<float2> Tinv32, WH32;
  DevList<int32_t> blkI, blkBm;       // [nblk][nI] canonical, [nblk][nBf] macro index / -1
  DevList<int64_t> macroB;            // [nM] canonical index of each macro unknown
  DevList<int32_t> cred_ptr, cred_ent;
  DevList<int64_t> patch_ptr;
  DevList<int32_t> patch_slot;
  DevList<int32_t> mpidx;             // [nblk][nBf] packed position of each macro-block slot
                                     // (recomputed patch inverses)
  HermSet Mset, Sset;
  DevList<int64_t> Pptr, Ptptr;
  DevList<int32_t> Pcol, Ptcol;
  DevList<double> Pval, Ptval;
  DevList<float> Pval32, Ptval32;
  // V-cycle work vectors: r, x, res on this macro grid; rc, ec on the coarser
  // mesh's traces; c = per-block condensation contributions of this level.
  DevBuf<double2> r64, x64, res64, rc64, ec64, c64;
  DevBuf<float2> r32, x32, res32, rc32, ec32, c32;
  // the same for block (multi-right-hand-side) solves, dpg_ctx::bcap columns
  DevBuf<double2> br64, bx64, bres64, brc64, bec64, bc64;
  DevBuf<float2> br32, bx32, bres32, brc32, bec32, bc32;
  HermBlockBufs Mb, Sb;
  MacroPlan mp;
  PatchPlan pp;
};

// Instantiated HIP graphs of the PCG iteration: (A) matvec, alpha, x and r;
// (B) V-cycle, beta, search direction, in two versions (z and z_old swap
// every iteration).  Destroyed with the object.
struct GraphSet {
  hipGraphExec_t a = nullptr, b[2] = {nullptr, nullptr};
  GraphSet() = default;
  GraphSet(const GraphSet &) = delete;
  GraphSet &operator=(const GraphSet &) = delete;
  ~GraphSet() {
    for (hipGraphExec_t g : {a, b[0], b[1]})
      if (g) (void)hipGraphExecDestroy(g);
  }
};

// A block PCG whose columns join and leave while it runs (continuous
// batching; dpg_batch_* and the block path of dpg_solve).  Slot k is column
// k of the interleaved block vectors of the context (width w).
struct BatchSession {
  bool open = false;
  int max = 0, w = 0;                // capacity, current width (a power of two or max)
  int cur = 0;                       // which of bz / bzo holds z
  int state[kMaxCols] = {};          // 0 free, 1 running, 2 converged, 3 maxit, 4 breakdown
  int iters[kMaxCols] = {};
  double tol[kMaxCols] = {}, bb[kMaxCols] = {}, rr[kMaxCols] = {};
  bool act_dirty = true;
  std::vector<int> done;             // finished slots not taken yet, in finishing order
  std::unique_ptr<GraphSet> graphs;  // captured for width gw
  int gw = 0;
  int lw = 0;                        // width of the last iteration
};

}  // namespace dpg

struct dpg_ctx {
  std::string err;
  int stage = 0;                     // 1 set up, 2 assembled, 3 hierarchy built
  bool released = false;             // setup-only data freed (dpg_release_setup)
  int N = 0, p = 0, dp = 1, nrhs = 0;
  double omega = 0, side = 1, org[3] = {0, 0, 0};
  dpg_options opt{};
  int device = 0;                    // the device current at dpg_setup
  hipStream_t stream = nullptr;
  hipStream_t own_stream = nullptr;  // created when the options give no stream
  hipStream_t aux = nullptr;         // second stream of the setup phases
  hipStream_t paux[2] = {nullptr, nullptr};   // third and fourth setup streams
  hipEvent_t ev_pjoin[2] = {nullptr, nullptr};
  hipEvent_t ev_fork = nullptr, ev_join = nullptr;
  std::vector<hipEvent_t> ev_level;  // per level: macro blocks ready for the patches
  dpg::Budget bud;
  dpg::ElementLayout el;
  int n_test = 0, n_field = 0, n_tr = 0, m = 0;
  std::vector<double> c_h;
  dpg::DevBuf<double> kappa, Zel;
  dpg::ElemTables tables_h{};
  dpg::DevBuf<dpg::ElemTables> tables;
  dpg::DevBuf<int4> testd, triald;
  std::vector<dpg::LoadDesc> ld_h;
  std::vector<double> src_h;
  dpg::DevBuf<dpg::LoadDesc> ld;
  dpg::DevBuf<double> src;
  dpg::DevBuf<double2> u0q;          // impedance data at the boundary load points, all loads
  std::vector<dpg::LevelData> lv;
  dpg::DevBuf<int32_t> classes;      // the class lists of every level
  int L = 0;
  bool keep_recovery = false;
  dpg::DevBuf<double2> s_elem;       // [nrhs][nel][n_tr] condensed element loads
  dpg::DevBuf<double2> s_asm;        // [nrhs][n_trace] assembled loads
  dpg::DevBuf<int32_t> asm_ptr, asm_ent;
  dpg::DevBuf<double2> rec_L, rec_Y, rec_Yb;  // [ec.n][nf^2], [ec.n][nf n_tr], [nel][nrhs nf]
  dpg::DevBuf<int32_t> elist;        // elements of a point-source load update
  dpg::LoadMaps lm;                  // load updates without the element chain
  // coarsest mesh
  dpg::DevBuf<double2> T0;
  dpg::HermSet T0set;
  // setup-phase plans and workspaces
  dpg::ElemPlan ep;
  dpg::DevBuf<double2> mT[2], mLinv[2], mX[2], mwk[2];   // macro levels, one set per stream
  dpg::DevBuf<double2> pS[4], pX[4], pwk[4];       // patches, one set per part
  dpg::DevBuf<double2> ptmp;                       // recomputed inverses: X x_v, local layout
  dpg::DevBuf<double2> zF, zLi, zTi, zwk;          // coarsest
  dpg::DevBuf<dpg::PotrfItem> zpi;
  dpg::DevBuf<dpg::TrsmItem> zti;
  dpg::DevBuf<dpg::GemmItem> zgi;
  dpg::DevBuf<int64_t> zoff;
  dpg::DevBuf<int32_t> znn, zld, zptr, zent;   // zptr, zent: elements holding each unknown
  dpg::DevBuf<int> zinfo;
  // outer CG (FP64, finest macro grid)
  dpg::DevBuf<double2> b, x, r, z, zo, pv, q, xfull, sB;
  dpg::DevBuf<double> partial, sc;
  double *host_sc = nullptr;         // pinned
  double *host_report = nullptr, *dev_report = nullptr;   // pinned, and its device address
  // block PCG (interleaved [n][nr] vectors), allocated at the first block solve
  int bcap = 0;
  dpg::HermBlockBufs T0b;
  dpg::DevBuf<double2> bpart;        // partials of few FP64 columns, of every block set in turn
  dpg::DevBuf<double2> bb, bx, br, bz, bzo, bp, bq, bsv, bxf, bcols;
  dpg::DevBuf<double> bpartial, bsc;
  dpg::DevBuf<int> bact;
  double *host_bsc = nullptr;        // pinned, 8 x kMaxCols
  int *host_bact = nullptr;          // pinned, kMaxCols
  dpg::BatchSession bs;
  bool nonfinite = false;            // a column of a block solve ended in a breakdown
  double ms[4] = {0, 0, 0, 0};
  dpg::Prof prof;
};
