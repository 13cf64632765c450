// Overlapped patches: a level's Gauss-Seidel sweeps, residual and transfers as two launches.
//
// A level is cut into patches of consecutive rows in spatial (Morton) order. A patch also holds the
// halo of rows that its own rows' results depend on through every colour pass of the sweeps, found by
// walking the passes backwards: before a pass of colour c, the needed values are the ones needed
// after it without colour c, and the neighbours of the needed rows of colour c. One block keeps the
// patch's x in LDS and its matrix rows in registers, runs all passes with a block barrier between
// them, and writes its own rows only; halo rows are computed redundantly (the same arithmetic in the
// same order as their owner's, so every patch sees the same values). A row whose inputs lie outside the
// patch computes a value that no needed row reads.
//
// `down` (forward sweeps from zero): b -> x on the own rows, then the residual, then the restriction of
// the coarse rows that the patch owns (their fine rows belong to the halo as well).
// `up` (backward sweeps): x + P e on every cell that the first pass reads, then the passes.
//
// Layout of a patch: its rows sorted by colour, inside a colour by row length, in slices of 64 rows
// (one per lane), dealt to the waves in turn, and cell 64 k + lane of the LDS image is its row. Cells
// that are read but never computed follow the last slice. The cells whose value counts before the first
// backward pass form slices of their own (start rows), by the length of their prolongation row. Matrix entries come in pairs: two values and
// two 16-bit cell numbers, 64 lanes side by side; shorter rows of a slice are filled up with products 0 * the
// row's own first neighbour. A row without any neighbour has no such cell, and another row's may hold anything (a
// cell that `up` does not write, a non-finite value of another mesh of a batch): those rows form slices of their
// own, of width 0. A prolongation row without entries takes a neighbour's column for its padding, and a restriction
// row whose entries are all left out (zero residuals) one of their cells: slices of their own for them made the upward
// launches of a graded mesh longer (1M rows, FP32 application 0.560 ms against 0.554). Only those that find none form
// slices of width 0. Matrices with few distinct values (the level matrices
// of a constant coefficient) keep a 4-bit code above each 12-bit cell number instead of the value, and
// so do prolongations, whose entries are 1 and 1/2 (above the column number).
#pragma once

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdint>
#include <memory>
#include <mutex>
#include <vector>

#include "common.hpp"
#include "host_parallel.hpp"

namespace asmg {

// Geometry of the patch kernels: waves of a block, slices per wave, entry pairs of a row kept in registers
// (FP64, FP32), bits of a cell number in 16 (a code sits above it).
//   PatchSmall: up to 2048 rows, two blocks per CU; the 2-D levels.
//   PatchBig: up to 6144 rows, the whole register file and LDS of a CU; 3-D levels of many colours, whose
//   halo through all passes is several times the own rows.
template <int Waves, int Slots, int Pairs64, int Pairs32, int Bits>
struct PatchGeom {
  static constexpr int waves = Waves, slots = Slots, bits = Bits;
  static constexpr int threads = 64 * Waves, slices = Waves * Slots;
  template <class T>
  static constexpr int pairs = sizeof(T) == 8 ? Pairs64 : Pairs32;
};
using PatchSmall = PatchGeom<8, 4, 4, 4, 12>;
using PatchBig = PatchGeom<16, 6, 2, 4, 13>;

struct PatchShape {
  int waves, slices, cell_slices, bits;
};
static constexpr PatchShape kPatchSmall{PatchSmall::waves, PatchSmall::slices, 38, PatchSmall::bits};
static constexpr PatchShape kPatchBig{PatchBig::waves, PatchBig::slices, 104, PatchBig::bits};
static_assert(64 * kPatchSmall.cell_slices <= 1 << PatchSmall::bits, "cell numbers fit below the codes");
static_assert(64 * kPatchBig.cell_slices <= 1 << PatchBig::bits, "cell numbers fit below the codes");

static constexpr int kPatchHeadCoarse = 16;  // coarse slices whose entry offsets are in the head
static constexpr int kPatchColours = 15;
static constexpr int kPatchHalo = 1 << 30;   // gidx: a halo row or cell (its result is not written)
static constexpr int kPatchCodes = 16;       // matrix codes (PatchSmall)

struct alignas(64) PatchHead {
  int ns, ncs;          // matrix slices, cell slices (the first ns are the matrix slices)
  int start0, nst;      // first slice of start rows, slices
  int coarse0, nco;     // first slice of coarse rows, slices
  int cell0;            // first slice of the cells that are no rows (on request)
  uint64_t sc[PatchBig::slots];         // colour of slice (waves j + i) in bits 4 i of sc[j], 15 = none
  int poff[kPatchBig.slices + 1];       // first pair row of each matrix slice
  int uoff[kPatchBig.cell_slices + 1];  // first prolongation row of each slice of start rows
  int roff[kPatchHeadCoarse + 1];       // first pair row of the first coarse slices
};

// a vector whose plain resize leaves the new elements unwritten: parallel tasks copy into them, and the first
// touch of the pages is theirs
template <class T>
struct RawAlloc : std::allocator<T> {
  template <class U>
  struct rebind {
    using other = RawAlloc<U>;
  };
  template <class U>
  void construct(U *p) {
    ::new ((void *)p) U;
  }
  template <class U, class... A>
  void construct(U *p, A &&...a) {
    ::new ((void *)p) U(std::forward<A>(a)...);
  }
};
template <class T>
using RawVector = std::vector<T, RawAlloc<T>>;

// host image of a level's patches, or of a run of them
struct PatchHost {
  std::vector<PatchHead> head;
  RawVector<int> gidx;              // level row per matrix lane, -1 = none; as many slices a patch as fit
  RawVector<uint32_t> pidx;         // two cells per pair
  RawVector<double> pval;           // two values
  RawVector<int> cgidx;             // level row of each cell that is no row, -1 = none (on request)
  RawVector<int> ugidx, ucell;      // start rows: level row (-1 = none), cell
  RawVector<int> ucol;              // and prolongation row
  RawVector<double> uval;
  RawVector<int> roff, rrow;        // coarse rows owned, and their restriction over cells
  RawVector<uint32_t> ridx;
  RawVector<double> rval;
  int64_t rows = 0, own = 0;
  PatchHost() { roff.push_back(0); }

  // appends b in two steps: room for its elements, then (any thread) the elements. The values of coded entries
  // are left out.
  struct Place {
    size_t head, gidx, pidx, cgidx, start, ucol, coarse, ridx;
  };
  void reserve(const std::vector<PatchHost> &parts, bool pvals, bool tvals) {
    Place n{};
    for (const PatchHost &b : parts) {
      n.head += b.head.size();
      n.gidx += b.gidx.size();
      n.pidx += b.pidx.size();
      n.cgidx += b.cgidx.size();
      n.start += b.ugidx.size();
      n.ucol += b.ucol.size();
      n.coarse += b.rrow.size();
      n.ridx += b.ridx.size();
    }
    head.reserve(n.head);
    gidx.reserve(n.gidx);
    pidx.reserve(n.pidx);
    if (pvals) pval.reserve(2 * n.pidx);
    cgidx.reserve(n.cgidx);
    ugidx.reserve(n.start);
    ucell.reserve(n.start);
    ucol.reserve(n.ucol);
    if (tvals) uval.reserve(n.ucol);
    rrow.reserve(n.coarse);
    roff.reserve(n.coarse / 64 + 1);
    ridx.reserve(n.ridx);
    if (tvals) rval.reserve(2 * n.ridx);
  }
  Place room(const PatchHost &b, bool pvals, bool tvals) {
    const Place at{head.size(), gidx.size(), pidx.size(), cgidx.size(), ugidx.size(), ucol.size(), rrow.size(), ridx.size()};
    head.resize(at.head + b.head.size());
    gidx.resize(at.gidx + b.gidx.size());
    pidx.resize(at.pidx + b.pidx.size());
    if (pvals) pval.resize(2 * pidx.size());
    cgidx.resize(at.cgidx + b.cgidx.size());
    ugidx.resize(at.start + b.ugidx.size());
    ucell.resize(at.start + b.ucell.size());
    ucol.resize(at.ucol + b.ucol.size());
    if (tvals) uval.resize(ucol.size());
    rrow.resize(at.coarse + b.rrow.size());
    roff.resize(rrow.size() / 64 + 1);
    ridx.resize(at.ridx + b.ridx.size());
    if (tvals) rval.resize(2 * ridx.size());
    rows += b.rows;
    own += b.own;
    return at;
  }
  void put(const PatchHost &b, const Place &at, bool pvals, bool tvals) {
    const int c0 = (int)(at.start / 64), r0 = (int)(at.coarse / 64), l0 = (int)(at.cgidx / 64);
    const int p0 = (int)(at.pidx / 64), u0 = (int)(at.ucol / 64), q0 = (int)(at.ridx / 64);
    for (size_t i = 0; i < b.head.size(); ++i) {
      PatchHead h = b.head[i];
      h.start0 += c0;
      h.coarse0 += r0;
      h.cell0 += l0;
      for (int &o : h.poff) o += p0;
      for (int &o : h.uoff) o += u0;
      for (int &o : h.roff) o += q0;
      head[at.head + i] = h;
    }
    auto copy = [](const auto &x, auto &y, size_t o) { std::copy(x.begin(), x.end(), y.begin() + o); };
    copy(b.gidx, gidx, at.gidx);
    copy(b.pidx, pidx, at.pidx);
    if (pvals) copy(b.pval, pval, 2 * at.pidx);
    copy(b.cgidx, cgidx, at.cgidx);
    copy(b.ugidx, ugidx, at.start);
    copy(b.ucell, ucell, at.start);
    copy(b.ucol, ucol, at.ucol);
    if (tvals) copy(b.uval, uval, at.ucol);
    for (size_t i = 1; i < b.roff.size(); ++i) roff[at.coarse / 64 + i] = b.roff[i] + q0;
    copy(b.rrow, rrow, at.coarse);
    copy(b.ridx, ridx, at.ridx);
    if (tvals) copy(b.rval, rval, 2 * at.ridx);
  }
};

// One level's matrices in its internal numbering, as the builder reads them. M has rp, ci, v.
template <class M>
struct PatchSource {
  const M *A = nullptr;       // off-diagonal part, symmetric pattern
  int n = 0;                  // rows (all smoothed)
  std::vector<uint8_t> col;   // colour per row
  int C = 0;
  std::vector<int> order;     // rows in spatial order
  int nu = 1;                 // sweeps per side
  const M *P = nullptr;       // prolongation: rows of this level, columns of the coarser one
  int ncoarse = 0;            // rows of the coarser level
  const M *R = nullptr;       // restriction: all rows of the coarser level; null = write the residual
  bool want_cells = false;    // list the cells that are no rows (patch_map reads them)
  bool lone = false;          // original grid of a 2-D single-mesh handle above a level that runs passes
  PatchShape shape = kPatchSmall;
  bool use[2] = {true, true}; // whether the patches are faster in an FP64, an FP32 cycle (patch_plan)
  bool alone(int r) const { return A->rp[r] == A->rp[r + 1]; }  // no neighbours
  // filled by prepare()
  std::vector<int> pos;           // position of each row in the order
  std::vector<int> cpos0, clist;  // coarse rows by the position of the row that decides their owner

  void prepare() {
    pos.resize(n);
    for (int i = 0; i < n; ++i) pos[order[i]] = i;
    if (!R) return;
    const int nc = (int)R->rp.size() - 1;
    std::vector<int> at(nc);
    cpos0.assign((size_t)n + 1, 0);
    for (int k = 0; k < nc; ++k) {
      int best = -1;
      double w = -1;
      for (int p = R->rp[k]; p < R->rp[k + 1]; ++p) {
        const double a = std::fabs(R->v[p]);
        if (a > w) {
          w = a;
          best = R->ci[p];
        }
      }
      at[k] = best >= 0 ? pos[best] : (int)((int64_t)k * n / nc);
      cpos0[at[k] + 1]++;
    }
    for (int i = 0; i < n; ++i) cpos0[i + 1] += cpos0[i];
    clist.resize(nc);
    std::vector<int> fill(cpos0.begin(), cpos0.end() - 1);
    for (int k = 0; k < nc; ++k) clist[fill[at[k]]++] = k;
  }
};

// marks over a level's rows
struct PatchMarks {
  std::vector<int> need, uni, cell, row;
  std::vector<int> list[2];
  int epoch = 0;
  void size(int n) {
    if ((int)need.size() < n) {
      need.resize(n, 0);
      uni.resize(n, 0);
      cell.resize(n, 0);
      row.resize(n, 0);
    }
    ++epoch;
  }
};

// the marks of the threads that build a set of levels
struct PatchPool {
  std::mutex mu;
  std::vector<std::unique_ptr<PatchMarks>> idle;
  std::unique_ptr<PatchMarks> take() {
    std::lock_guard<std::mutex> g(mu);
    if (idle.empty()) return std::make_unique<PatchMarks>();
    std::unique_ptr<PatchMarks> w = std::move(idle.back());
    idle.pop_back();
    return w;
  }
  void give(std::unique_ptr<PatchMarks> w) {
    std::lock_guard<std::mutex> g(mu);
    idle.push_back(std::move(w));
  }
};

// Rows and cells of the patch of order[a..b): `uni` all of them (`row` marks the computed ones), `need` the
// cells whose value before the first backward pass counts; false where they cannot fit.
template <class M>
static bool patch_closure(const PatchSource<M> &S, int a, int b, PatchMarks &W, std::vector<int> &need,
                          std::vector<int> &uni) {
  const M &A = *S.A;
  const int C = S.C;
  W.size(S.n);
  const int E = W.epoch;
  std::vector<int> next, cur;
  need.clear();
  uni.clear();
  auto add = [&](int r) {
    if (W.need[r] != E) {
      W.need[r] = E;
      need.push_back(r);
    }
    if (W.uni[r] != E) {
      W.uni[r] = E;
      uni.push_back(r);
    }
  };
  auto later = [&](int c, bool earlier_only, bool rows) {  // undo one pass of colour c
    next.clear();
    cur.clear();
    for (int r : need)
      if (S.col[r] == c) {
        W.need[r] = E - 1;
        cur.push_back(r);
        if (rows) W.row[r] = E;
      } else if (!(earlier_only && S.col[r] > c)) {
        next.push_back(r);
      } else {
        W.need[r] = E - 1;
      }
    need.swap(next);
    for (int r : cur)
      for (int p = A.rp[r]; p < A.rp[r + 1]; ++p)
        if (!earlier_only || S.col[A.ci[p]] < c) add(A.ci[p]);
  };
  // rows computed going down
  for (int i = a; i < b; ++i) add(S.order[i]);
  auto residual_of = [&](int r) {
    add(r);
    for (int p = A.rp[r]; p < A.rp[r + 1]; ++p)
      if (S.nu > 1 || S.col[A.ci[p]] > S.col[r]) add(A.ci[p]);
  };
  if (S.R) {
    for (int q = S.cpos0[a]; q < S.cpos0[b]; ++q) {
      const int k = S.clist[q];
      for (int p = S.R->rp[k]; p < S.R->rp[k + 1]; ++p)
        if (S.col[S.R->ci[p]] != C - 1) residual_of(S.R->ci[p]);
    }
  } else {
    for (int i = a; i < b; ++i)
      if (S.col[S.order[i]] != C - 1) residual_of(S.order[i]);
  }
  for (int k = S.nu - 1; k >= 0; --k)
    for (int c = C - 1; c >= 0; --c) later(c, k == 0, false);
  for (int r : uni) W.row[r] = E;
  if ((int)uni.size() > 64 * S.shape.slices) return false;
  // rows computed and cells read going up
  for (int r : need) W.need[r] = E - 1;
  need.clear();
  for (int i = a; i < b; ++i) add(S.order[i]);
  for (int k = 0; k < S.nu; ++k)
    for (int c = 0; c < C; ++c) later(c, false, true);
  return true;
}

// computed rows of a patch, 0 where it does not fit
template <class M>
static int patch_rows(const PatchSource<M> &S, int a, int b, PatchMarks &W, std::vector<int> &need,
                      std::vector<int> &uni) {
  if (!patch_closure(S, a, b, W, need, uni)) return 0;
  std::vector<int> count(2 * S.C, 0);
  int rows = 0;
  for (int r : uni) {
    if (W.row[r] != W.epoch) continue;
    count[2 * S.col[r] + S.alone(r)]++;
    ++rows;
  }
  int ns = 0;
  for (int k : count) ns += (k + 63) / 64;
  return ns > S.shape.slices || ns + ((int)uni.size() - rows + 63) / 64 > S.shape.cell_slices ? 0 : rows;
}

// Patch of the rows order[a..b): appended to out; false (nothing appended) where it does not fit.
template <class M>
static bool patch_one(const PatchSource<M> &S, int a, int b, PatchMarks &W, PatchHost &out) {
  const M &A = *S.A;
  const int C = S.C;
  std::vector<int> &need = W.list[0], &uni = W.list[1];
  if (!patch_closure(S, a, b, W, need, uni)) return false;
  const int E = W.epoch;
  std::vector<std::vector<int>> by(2 * C);  // rows of each colour with neighbours, and without
  std::vector<int> cells;
  for (int i : uni)
    if (W.row[i] == E)
      by[2 * S.col[i] + S.alone(i)].push_back(i);
    else
      cells.push_back(i);
  int ns = 0;
  for (auto &v : by) ns += ((int)v.size() + 63) / 64;
  const int ncs = ns + ((int)cells.size() + 63) / 64;
  if (ns > S.shape.slices || ncs > S.shape.cell_slices) return false;
  // start rows: the cells that some backward pass reads as they were
  auto plen = [&](int r) { return S.P->rp[r + 1] - S.P->rp[r]; };
  // column that pads a row's entries: its first, or where it has none the first of a neighbour (of the same mesh of
  // a batch); -1 = none
  auto pad_column = [&](int r) {
    if (plen(r) > 0) return S.P->ci[S.P->rp[r]];
    for (int p = A.rp[r]; p < A.rp[r + 1]; ++p)
      if (plen(A.ci[p]) > 0) return S.P->ci[S.P->rp[A.ci[p]]];
    return -1;
  };
  std::vector<std::pair<int, int>> start[2];  // with a column, without
  for (int r : need)
    if (W.need[r] == E && S.col[r] != C - 1) start[pad_column(r) < 0].push_back({plen(r), r});
  if ((start[0].size() + 63) / 64 + (start[1].size() + 63) / 64 > (size_t)kPatchBig.cell_slices) return false;
  // spatial order inside a colour: internal numbers ascend with the spatial order there
  PatchHead h{};
  h.start0 = (int)(out.ugidx.size() / 64);
  h.coarse0 = (int)out.roff.size() - 1;
  h.ns = ns;
  h.ncs = ncs;
  auto kept = [&](int r) {
    int w = 0;
    for (int p = A.rp[r]; p < A.rp[r + 1]; ++p) w += W.uni[A.ci[p]] == E;
    return w;
  };
  std::vector<int> list;  // row per cell, -1 = empty lane
  std::vector<std::pair<int, int>> key;
  for (uint64_t &x : h.sc) x = ~0ull;
  for (int i = 0; i < 2 * C; ++i) {
    const int c = i / 2, k0 = (int)list.size() / 64;
    std::sort(by[i].begin(), by[i].end());
    key.clear();
    for (int r : by[i]) key.push_back({(kept(r) + 1) / 2, r});
    std::stable_sort(key.begin(), key.end(), [](auto &x, auto &y) { return x.first > y.first; });
    for (auto &kr : key) list.push_back(kr.second);
    while (list.size() % 64) list.push_back(-1);
    for (int k = k0; k < (int)list.size() / 64; ++k) {
      const int bit = 4 * (k % S.shape.waves);
      h.sc[k / S.shape.waves] = (h.sc[k / S.shape.waves] & ~(15ull << bit)) | (uint64_t)c << bit;
    }
  }
  std::sort(cells.begin(), cells.end());
  for (int r : cells) list.push_back(r);
  while (list.size() % 64) list.push_back(-1);
  for (size_t i = 0; i < list.size(); ++i)
    if (list[i] >= 0) W.cell[list[i]] = (int)i;
  h.cell0 = (int)(out.cgidx.size() / 64);
  if (S.want_cells) out.cgidx.insert(out.cgidx.end(), list.begin() + 64 * ns, list.end());
  // own rows: marked by position
  std::vector<uint8_t> own(list.size(), 0);
  for (int i = a; i < b; ++i) own[W.cell[S.order[i]]] = 1;
  for (int i = 0; i < 64 * S.shape.slices; ++i) {
    const int r = i < 64 * ns ? list[i] : -1;
    out.gidx.push_back(r < 0 ? -1 : own[i] ? r : r | kPatchHalo);
  }
  // matrix pairs
  for (int k = 0; k < ns; ++k) {
    int w = 0;
    for (int l = 0; l < 64; ++l)
      if (list[64 * k + l] >= 0) w = std::max(w, (kept(list[64 * k + l]) + 1) / 2);
    const size_t base = out.pidx.size();
    h.poff[k] = (int)(base / 64);
    out.pidx.resize(base + (size_t)w * 64, 0);
    out.pval.resize(2 * (base + (size_t)w * 64), 0.0);
    for (int l = 0; l < 64; ++l) {
      const int r = list[64 * k + l];
      if (r < 0) continue;
      int q = 0, first = 0;
      for (int p = A.rp[r]; p < A.rp[r + 1]; ++p) {
        if (W.uni[A.ci[p]] != E) continue;
        const int c = W.cell[A.ci[p]];
        if (q == 0) first = c;
        const size_t e = base + (size_t)(q >> 1) * 64 + l;
        out.pidx[e] |= (uint32_t)c << (q & 1 ? 16 : 0);
        out.pval[2 * e + (q & 1)] = A.v[p];
        ++q;
      }
      for (; q < 2 * w; ++q)  // padding: the row's first neighbour with value 0
        out.pidx[base + (size_t)(q >> 1) * 64 + l] |= (uint32_t)first << (q & 1 ? 16 : 0);
    }
  }
  for (int k = ns; k <= kPatchBig.slices; ++k) h.poff[k] = (int)(out.pidx.size() / 64);
  for (auto &st : start) {
    // in spatial order (the gathers of a slice then share lines), by length inside windows
    std::sort(st.begin(), st.end(), [&](auto &x, auto &y) { return S.pos[x.second] < S.pos[y.second]; });
    for (size_t k = 0; k < st.size(); k += 256)
      std::stable_sort(st.begin() + k, st.begin() + std::min(k + 256, st.size()),
                       [](auto &x, auto &y) { return x.first > y.first; });
    for (size_t k = 0; k < st.size(); k += 64) {
      const int w = st[k].first;
      const size_t base = out.ucol.size();
      h.uoff[h.nst++] = (int)(base / 64);
      out.ucol.resize(base + (size_t)w * 64, 0);
      out.uval.resize(base + (size_t)w * 64, 0.0);
      for (size_t l = 0; l < 64; ++l) {
        const int r = k + l < st.size() ? st[k + l].second : -1;
        out.ugidx.push_back(r);
        out.ucell.push_back(r < 0 ? 0 : W.cell[r]);
        if (r < 0) continue;
        const int m = plen(r), pad = m < w ? pad_column(r) : 0;
        for (int q = 0; q < w; ++q) {
          const size_t e = base + (size_t)q * 64 + l;
          out.ucol[e] = q < m ? S.P->ci[S.P->rp[r] + q] : pad;
          if (q < m) out.uval[e] = S.P->v[S.P->rp[r] + q];
        }
      }
    }
  }
  for (int k = h.nst; k <= kPatchBig.cell_slices; ++k) h.uoff[k] = (int)(out.ucol.size() / 64);
  // coarse rows
  if (S.R) {
    auto len = [&](int k) {
      int w = 0;
      for (int p = S.R->rp[k]; p < S.R->rp[k + 1]; ++p) w += S.col[S.R->ci[p]] != C - 1;
      return w;
    };
    // cell of an own row that a coarse row weighs (the one that made the patch its owner is among them)
    auto own_cell = [&](int k) {
      for (int p = S.R->rp[k]; p < S.R->rp[k + 1]; ++p) {
        const int at = S.pos[S.R->ci[p]];
        if (at >= a && at < b) return W.cell[S.R->ci[p]];
      }
      return 0;
    };
    std::vector<std::pair<int, int>> coarse[2];  // with entries (left out or not), without
    for (int q = S.cpos0[a]; q < S.cpos0[b]; ++q) {
      const int k = S.clist[q];
      coarse[S.R->rp[k] == S.R->rp[k + 1]].push_back({(len(k) + 1) / 2, k});
    }
    for (auto &rows : coarse) {
      std::stable_sort(rows.begin(), rows.end(), [](auto &x, auto &y) { return x.first > y.first; });
      for (size_t k = 0; k < rows.size(); k += 64) {
        const int w = rows[k].first;
        const size_t base = (size_t)out.roff.back() * 64;
        out.ridx.resize(base + (size_t)w * 64, 0);
        out.rval.resize(2 * (base + (size_t)w * 64), 0.0);
        for (size_t l = 0; l < 64; ++l) {
          if (k + l >= rows.size()) {
            out.rrow.push_back(-1);
            continue;
          }
          const int row = rows[k + l].second;
          out.rrow.push_back(row);
          int q = 0, first = own_cell(row);
          for (int p = S.R->rp[row]; p < S.R->rp[row + 1]; ++p) {
            if (S.col[S.R->ci[p]] == C - 1) continue;
            const int c = W.cell[S.R->ci[p]];
            if (q == 0) first = c;
            const size_t e = base + (size_t)(q >> 1) * 64 + l;
            out.ridx[e] |= (uint32_t)c << (q & 1 ? 16 : 0);
            out.rval[2 * e + (q & 1)] = S.R->v[p];
            ++q;
          }
          for (; q < 2 * w; ++q) out.ridx[base + (size_t)(q >> 1) * 64 + l] |= (uint32_t)first << (q & 1 ? 16 : 0);
        }
        out.roff.push_back(out.roff.back() + w);
        ++h.nco;
      }
    }
  }
  for (int k = 0; k <= kPatchHeadCoarse; ++k) h.roff[k] = out.roff[h.coarse0 + std::min(k, h.nco)];
  out.head.push_back(h);
  out.rows += (int64_t)uni.size() - (int64_t)cells.size();
  out.own += b - a;
  return true;
}

template <class M>
static bool patch_range(const PatchSource<M> &S, int a, int b, PatchMarks &W, PatchHost &out) {
  if (a >= b) return true;
  if (patch_one(S, a, b, W, out)) return true;
  if (b - a < 2) return false;
  const int m = a + (b - a) / 2;
  return patch_range(S, a, m, W, out) && patch_range(S, m, b, W, out);
}

// Own rows per patch that a plan starts from: enough patches for the chip where that is possible, no fewer own rows
// than kPatchOwnMin (the halo grows against them: measured flat from 256 to 1024 within 4 %), no more than
// kPatchOwnMax. Where such patches do not fit, a fifth less at a time, down to 128; where the halo outweighs the own
// rows (3-D levels), as many as fit.
static constexpr int kPatchOwnMin = 256;
static constexpr int kPatchOwnMax = 1536;

// Estimated us of a level's two patch launches in an FP64 (p = 0) or FP32 cycle, from measured ones: 5 us each, and
// beyond that 4 us for every 512 patches of PatchSmall (two per CU at a time), for every 256 of PatchBig 14 and 1.2
// for each pass, or its rows (own and halo) at 4 TB/s and some 70 bytes; and the prolongation's gathers, 1.6 us for
// each entry of a row beyond two (the original grid: 2-D 6 entries, up 15 us; 3-D 12, 29 us).
// Where the levels below run passes (local smoothing, near-boundary correction), their launch shapes are tuned and
// the original grid's passes cost a first solve nothing more, so the line is drawn more exactly there: an FP64
// block has a CU to itself, and beyond 256 patches the second round of blocks costs more than the passes save; FP32
// rows take 22 ps, and beyond 512 patches the next level's own first pass and restriction weigh as well. Measured, us
// an iteration that the patches gain with local smoothing: FP64 102k rows +15, 249k +9 (256 patches), 489k -34
// (398), 998k -41 (813); FP32 +18, +11, +9, -14; with the near-boundary correction: FP64 55k +15, 218k +16, 869k -55;
// FP32 +16, +26, -39. (Where every level has patches a first FP64 solve of 998k rows takes 19 ms with passes on the
// original grid, 8 without, and a later one 6.0 against 6.4.)
template <class M>
static double patch_cost(const PatchSource<M> &S, bool big, int np, double rows, double pw, int p) {
  const double gathers = 1.6 * std::max(0.0, pw - 2);
  if (S.lone && p == 0 && np > 256) return 40.0 * ((np + 255) / 256);
  if (S.lone && p == 1)
    return 2 * (5 + std::max(4.0 * ((np + 511) / 512), 2.2e-5 * rows)) + gathers + (np > 512 ? 25 : 0);
  const double one = big ? (14 + 1.2 * S.nu * S.C) * ((np + 255) / 256) : 4.0 * ((np + 511) / 512);
  return 2 * (5 + std::max(one, 1.75e-5 * rows)) + gathers;
}

// and of its passes one by one: one per colour, sweep and direction, the residual and the transfers, 3 us
// each and 18 more per million rows of their colour (measured in a graph: 2.9 us at 2000 rows, 4.75 at
// 125,000, 12.5 at 540,000; on the 2-D original grid 32 in FP64, 21 in FP32). Where the patches write the
// residual, the restriction is a launch of its own on both sides.
template <class M>
static double pass_cost(const PatchSource<M> &S, int p) {
  const double slope = !S.lone ? 1.8e-5 : p == 0 ? 3.2e-5 : 2.1e-5;
  return (2 * S.nu * S.C + (S.lone && !S.R ? 2 : 3)) * (3.0 + slope * S.n / S.C);
}

// Plan of one level's patches: the chunk boundaries in the spatial order, and in S the shape and the precisions
// that gain; empty = the passes are faster in both. `big`: the larger shape may be used.
template <class M>
static std::vector<int> patch_plan(PatchSource<M> &S, bool big) {
  std::vector<int> cut;
  if (S.n < 1 || S.C < 1 || S.C > kPatchColours || S.n >= 1 << 27) return cut;
  if (S.ncoarse >= 1 << 27) return cut;
  PatchMarks W;
  const double pw = (double)S.P->ci.size() / S.n, passes[2] = {pass_cost(S, 0), pass_cost(S, 1)};
  double best = 0;  // us gained
  int best_np = 0;
  PatchShape shape = kPatchSmall;
  // computed rows per own row of `np` patches, from up to 5 of them; 0 where one does not fit
  auto try_plan = [&](int np) {
    const int tries = std::min(np, 5);
    double rows = 0, own = 0;
    for (int i = 0; i < tries; ++i) {
      const int64_t p = tries > 1 ? (int64_t)i * (np - 1) / (tries - 1) : 0;
      const int a = (int)(p * S.n / np), b = (int)((p + 1) * S.n / np);
      const int r = patch_rows(S, a, b, W, W.list[0], W.list[1]);
      if (r == 0) return 0.0;
      rows += r;
      own += b - a;
    }
    return rows / own;
  };
  for (int k = 0; k < (big ? 2 : 1); ++k) {
    S.shape = k ? kPatchBig : kPatchSmall;
    int target = std::max(kPatchOwnMin, std::min(k ? 2 * kPatchOwnMax : kPatchOwnMax, (S.n + 255) / 256));
    int np = 0;
    double ratio = 0;
    for (; target >= 128 && ratio == 0; target -= target / 5) {
      np = (S.n + target - 1) / target;
      ratio = try_plan(np);
    }
    if (ratio == 0) continue;
    while (ratio > 2 && np > 1) {  // fewer, larger patches while they fit
      const int fewer = np - std::max(1, np / 5);
      const double r = try_plan(fewer);
      if (r == 0) break;
      np = fewer;
      ratio = r;
    }
    // the larger shape has to be clearly better: its patches take longer to lay out
    double gain[2];
    for (int p = 0; p < 2; ++p) gain[p] = passes[p] - patch_cost(S, k == 1, np, ratio * S.n, pw, p) * (k ? 1.25 : 1.0);
    if (std::max(gain[0], gain[1]) > best) {
      best = std::max(gain[0], gain[1]);
      best_np = np;
      shape = S.shape;
      for (int p = 0; p < 2; ++p) S.use[p] = gain[p] > 0;
    }
    if (ratio <= 2) break;
  }
  S.shape = shape;
  for (int p = 0; p <= best_np && best_np > 0; ++p) cut.push_back((int)((int64_t)p * S.n / best_np));
  return cut;
}

// the distinct values of v in ascending order, added to d; false: more than kPatchCodes
template <class V>
static bool patch_codes(const V &v, std::vector<double> &d) {
  for (double x : v) {
    auto it = std::lower_bound(d.begin(), d.end(), x);
    if (it != d.end() && *it == x) continue;
    if (d.size() == kPatchCodes || !(x == x)) return false;
    d.insert(it, x);
  }
  return true;
}

// Codes of a level: of its matrix entries (code, the index of the value in `dict`) and of its transfers
// (tcode: 0 for the value 1, 1 for 1/2, 2 for the padding's 0).
struct PatchCodes {
  bool matrix = false, transfer = false;
  std::vector<double> dict;
  int used = 0;  // values in dict
};

// what a run's values allow
struct PatchValues {
  std::vector<double> distinct;
  bool few = false, simple = false;
  void read(const PatchHost &H, bool matrix) {
    auto weights = [](const auto &v) {
      for (double x : v)
        if (x != 1.0 && x != 0.5 && x != 0.0) return false;
      return true;
    };
    few = matrix && patch_codes(H.pval, distinct);
    int most = 0;
    for (int c : H.ucol) most = std::max(most, c);
    simple = most < 1 << 28 && weights(H.uval) && weights(H.rval);
  }
};

static inline PatchCodes patch_code(const std::vector<PatchValues> &V) {
  PatchCodes K;
  K.dict.assign(kPatchCodes, 0.0);
  std::vector<double> d{0.0};  // the padding's, whether there is any or not: patch_recode decides by the matrix alone
  K.matrix = K.transfer = !V.empty();
  for (const PatchValues &v : V) {
    K.matrix = K.matrix && v.few && patch_codes(v.distinct, d);
    K.transfer = K.transfer && v.simple;
  }
  if (K.matrix) {
    std::copy(d.begin(), d.end(), K.dict.begin());
    K.used = (int)d.size();
  }
  return K;
}

// the codes of a run's entries, into their cell and column numbers
static inline void patch_encode(PatchHost &H, const PatchCodes &K, int bits) {
  auto halves = [bits](auto &idx, const auto &v, auto &&code) {
    for (size_t e = 0; e < idx.size(); ++e)
      idx[e] |= (uint32_t)code(v[2 * e]) << bits | (uint32_t)code(v[2 * e + 1]) << (16 + bits);
  };
  if (K.matrix) {
    const auto end = K.dict.begin() + K.used;
    halves(H.pidx, H.pval, [&](double x) { return std::lower_bound(K.dict.begin(), end, x) - K.dict.begin(); });
  }
  if (K.transfer) {
    auto code = [](double x) { return x == 1.0 ? 0 : x == 0.5 ? 1 : 2; };
    for (size_t e = 0; e < H.ucol.size(); ++e)
      H.ucol[e] = (int)((uint32_t)H.ucol[e] | (uint32_t)code(H.uval[e]) << 28);
    halves(H.ridx, H.rval, code);
  }
}

// A level's patches under construction; one task builds a run of kPatchRun patches.
static constexpr int kPatchRun = 8;

template <class M>
struct PatchJob {
  PatchSource<M> src;
  std::vector<int> cuts;  // patch boundaries in the spatial order; empty: none
  std::vector<PatchHost> parts;
  std::vector<PatchValues> values;
  std::vector<PatchHost::Place> place;
  PatchHost all;
  PatchCodes codes;
  bool code_matrix = true;
  std::atomic<bool> fits{true};
  int runs() const { return cuts.empty() ? 0 : ((int)cuts.size() - 2 + kPatchRun) / kPatchRun; }
};

// builds the patches of every job that has cuts; a level one of whose rows alone does not fit gets none
template <class M>
static void patch_build(int threads, std::vector<PatchJob<M>> &jobs) {
  std::vector<std::pair<int, int>> runs;
  for (size_t j = 0; j < jobs.size(); ++j) {
    jobs[j].parts.resize(jobs[j].runs());
    jobs[j].values.resize(jobs[j].runs());
    for (int t = 0; t < jobs[j].runs(); ++t) runs.push_back({(int)j, t});
  }
  PatchPool pool;
  host_parallel(threads, (int)runs.size(), [&](int i) {
    PatchJob<M> &J = jobs[runs[i].first];
    const int t = runs[i].second, np = (int)J.cuts.size() - 1;
    std::unique_ptr<PatchMarks> W = pool.take();
    for (int p = t * kPatchRun; p < std::min(np, (t + 1) * kPatchRun) && J.fits; ++p)
      if (!patch_range(J.src, J.cuts[p], J.cuts[p + 1], *W, J.parts[t])) J.fits = false;
    pool.give(std::move(W));
    J.values[t].read(J.parts[t], J.code_matrix && J.src.shape.bits == kPatchSmall.bits);
  });
  for (PatchJob<M> &J : jobs) {
    if (!J.fits) {
      J.cuts.clear();
      J.parts.clear();
      J.values.clear();
    }
    J.codes = patch_code(J.values);
    J.all.reserve(J.parts, !J.codes.matrix, !J.codes.transfer);
    for (const PatchHost &p : J.parts) J.place.push_back(J.all.room(p, !J.codes.matrix, !J.codes.transfer));
  }
  host_parallel(threads, (int)runs.size(), [&](int i) {
    PatchJob<M> &J = jobs[runs[i].first];
    if (J.parts.empty()) return;
    PatchHost &p = J.parts[runs[i].second];
    patch_encode(p, J.codes, J.src.shape.bits);
    J.all.put(p, J.place[runs[i].second], !J.codes.matrix, !J.codes.transfer);
    p = PatchHost();
  });
}

// Whether the FP32 cycle may run patches. In 3-D it keeps the passes: a patch adds up a row in another order, and CG
// on some cubes takes a change in the last bits of an FP32 cycle to 1e-9 of the solution (30^3 unknowns, 15 steps:
// 1e-14 on most, 3e-12 to 4e-9 on one, by either path, from scaling f alone), so the same sums stay. The precision
// is chosen call by call, so 3-D handles hold both; one created for the FP32 cycle builds no patches.
static inline bool patch_fp32(int dim) { return dim == 2; }

// device arrays of a level's patches, values in precision T
template <class T>
struct PatchView {
  const PatchHead *head;
  const int *gidx;
  const uint32_t *pidx;
  const T *pval;  // values; the dictionary where they are coded
  const int *ugidx, *ucell, *ucol;
  const T *uval;
  const int *roff, *rrow;
  const uint32_t *ridx;
  const T *rval;
};

struct DPatch {
  int np = 0;
  bool big = false;    // PatchBig
  bool fused = false;  // `down` restricts (else it writes the residual)
  bool mcode = false, tcode = false;  // matrix entries, transfer entries coded
  bool use[2] = {true, true};         // whether the FP64 and the FP32 cycle run them (else the level's passes)
  template <class T>
  bool on() const { return np > 0 && use[sizeof(T) == 4]; }
  int cells = 0, lrows = 0;  // LDS cells and matrix lanes of the largest patch
  PatchHead *head = nullptr;
  int *gidx = nullptr, *cgidx = nullptr, *ugidx = nullptr, *ucell = nullptr, *ucol = nullptr, *roff = nullptr, *rrow = nullptr;
  uint32_t *pidx = nullptr, *ridx = nullptr;
  // the dictionary or the plain values, as mcode says; a level that has been both holds both
  double *dict64 = nullptr, *plain64 = nullptr, *uval64 = nullptr, *rval64 = nullptr;
  float *dict32 = nullptr, *plain32 = nullptr, *uval32 = nullptr, *rval32 = nullptr;
  int *map = nullptr;  // matrix entry of each stored value (patch_map), made when the values first change
  RawVector<int> cells_host;  // cgidx where only a host update can make the map: most handles never need it
  int64_t npair = 0, nu = 0, nr = 0, rows = 0, nstart = 0, ncoarse = 0;  // stored pairs, entries, rows
  template <class T>
  PatchView<T> view() const {
    PatchView<T> v{head, gidx, pidx, nullptr, ugidx, ucell, ucol, nullptr, roff, rrow, ridx, nullptr};
    if constexpr (sizeof(T) == 8) {
      v.pval = mcode ? dict64 : plain64;
      v.uval = uval64;
      v.rval = rval64;
    } else {
      v.pval = mcode ? dict32 : plain32;
      v.uval = uval32;
      v.rval = rval32;
    }
    return v;
  }
};

// Algorithmic bytes of a level's two launches (n rows, nnz off-diagonal entries, NR values a row): every entry once,
// as its 2-byte cell or 4-byte column and, where it is not coded, its value; the vectors and diagonals once.
template <int NR, class T, class BT>
static double patch_down_bytes(const DPatch &D, double n, double nnz) {
  const double sz = sizeof(T), value = D.mcode ? 0 : sz, weight = D.tcode ? 0 : sz;
  // b, the diagonal (and in FP32 its reciprocal), x written; the restriction's entries and result, or the residual
  const double rows = 4 + NR * sizeof(BT) + (sizeof(T) == 4 ? 2 : 1) * sz + NR * sz;
  return nnz * (2 + value) + n * rows +
         (D.fused ? (double)D.nr * 2 * (2 + weight) + (double)D.ncoarse * (4 + NR * sz) : n * NR * sz);
}
template <int NR, class T, class BT>
static double patch_up_bytes(const DPatch &D, double n, double nnz) {
  const double sz = sizeof(T), value = D.mcode ? 0 : sz, weight = D.tcode ? 0 : sz;
  // b, the reciprocal of the diagonal, x read and the result written; the prolongation's entries and input
  return nnz * (2 + value) + n * (4 + NR * sizeof(BT) + sz + 2 * NR * sz) + (double)D.nu * (4 + weight) +
         (double)D.ncoarse * NR * sz;
}

// what the handles export of a level's patches
static inline std::vector<int64_t> patch_info(const DPatch &D) {
  return {D.np, D.big, D.mcode, D.tcode, D.on<double>(), D.on<float>()};
}

static __global__ __launch_bounds__(BS) void k_patch_round(int64_t n, const double *__restrict__ a,
                                                           float *__restrict__ b) {
  const int64_t i = (int64_t)blockIdx.x * BS + threadIdx.x;
  if (i < n) b[i] = (float)a[i];
}

static inline void patch_round(int64_t n, const double *a, float *b) {
  if (n > 0) hipLaunchKernelGGL(k_patch_round, dim3(nblk(n)), dim3(BS), 0, nullptr, n, a, b);
}

// room for a level's matrix values, coded or plain
template <class Room64, class Room32>
static void patch_values(DPatch &D, bool coded, Room64 &&room64, Room32 &&room32) {
  double *&v64 = coded ? D.dict64 : D.plain64;
  float *&v32 = coded ? D.dict32 : D.plain32;
  const int64_t n = coded ? kPatchCodes : 2 * D.npair;
  if (!v64) v64 = room64(n);
  if (!v32) v32 = room32(n);
}

// matrix values of a level, coded or plain, in both precisions; the room is there
static inline void patch_put_values(const PatchHost &H, const PatchCodes &K, DPatch &D) {
  double *v64 = D.mcode ? D.dict64 : D.plain64;
  const int64_t n = D.mcode ? kPatchCodes : 2 * D.npair;
  if (n == 0) return;
  HIPCHECK(hipMemcpy(v64, D.mcode ? K.dict.data() : H.pval.data(), (size_t)n * 8, hipMemcpyHostToDevice));
  patch_round(n, v64, D.mcode ? D.dict32 : D.plain32);
}

// uploads a level's patches; up(vector) -> device copy, room64(n), room32(n) -> n values
template <class Up, class Room64, class Room32>
static void patch_commit(const PatchHost &H, const PatchCodes &K, DPatch &D, bool fused, Up &&up, Room64 &&room64,
                         Room32 &&room32) {
  D.np = (int)H.head.size();
  D.fused = fused;
  if (!D.np) return;
  for (const PatchHead &h : H.head) {
    D.cells = std::max(D.cells, 64 * h.ncs);
    D.lrows = std::max(D.lrows, 64 * h.ns);
  }
  D.mcode = K.matrix;
  D.pidx = up(H.pidx);
  D.npair = (int64_t)H.pidx.size();
  patch_values(D, D.mcode, room64, room32);
  patch_put_values(H, K, D);
  D.head = up(H.head);
  D.gidx = up(H.gidx);
  if (!H.cgidx.empty()) D.cgidx = up(H.cgidx);
  D.ugidx = up(H.ugidx);
  D.ucell = up(H.ucell);
  D.ucol = up(H.ucol);
  D.nstart = (int64_t)H.ugidx.size();
  D.roff = up(H.roff);
  D.rrow = up(H.rrow);
  D.ridx = up(H.ridx);
  D.nu = (int64_t)H.ucol.size();
  D.nr = (int64_t)H.ridx.size();
  D.rows = H.rows;
  D.ncoarse = (int64_t)H.rrow.size();
  D.tcode = K.transfer;
  if (D.tcode) return;
  D.uval64 = up(H.uval);
  D.rval64 = up(H.rval);
  D.uval32 = room32(D.nu);
  D.rval32 = room32(2 * D.nr);
  patch_round(D.nu, D.uval64, D.uval32);
  patch_round(2 * D.nr, D.rval64, D.rval32);
}

// ---------------------------------------------------------------------------
// kernels
// ---------------------------------------------------------------------------

template <int NR, class T>
struct alignas(sizeof(T) * NR) PVec {
  T v[NR];
};

template <class T>
struct alignas(2 * sizeof(T)) PPair {
  T a, b;
};

// base[i], with the offset in 32 bits so that the address is a scalar base and one offset register (a
// level with patches has fewer than 2^27 rows, and so has the coarser one: 4 GiB of four FP64 values)
template <class X>
__device__ __forceinline__ X at32(const X *base, uint32_t i) {
  return *reinterpret_cast<const X *>(reinterpret_cast<const char *>(base) + (size_t)(uint32_t)(i * (uint32_t)sizeof(X)));
}
template <class X>
__device__ __forceinline__ void put32(X *base, uint32_t i, const X &v) {
  *reinterpret_cast<X *>(reinterpret_cast<char *>(base) + (size_t)(uint32_t)(i * (uint32_t)sizeof(X))) = v;
}

// transfer value of a code
template <class T>
__device__ __forceinline__ T patch_weight(uint32_t code) {
  return code == 0 ? T(1) : code == 1 ? T(0.5) : T(0);
}

// a0 += v.a x[first cell], a1 += v.b x[second cell]; UP: only cells above `above`
template <int BITS, bool UP, int NR, class T>
__device__ __forceinline__ void pair_add(PVec<NR, T> &a0, PVec<NR, T> &a1, uint32_t id, PPair<T> v,
                                         const PVec<NR, T> *xs, int above) {
  constexpr uint32_t mask = (1u << BITS) - 1;
  const int i0 = (int)(id & mask), i1 = (int)(id >> 16 & mask);
  if (UP) {
    v.a = i0 > above ? v.a : T(0);
    v.b = i1 > above ? v.b : T(0);
  }
  const PVec<NR, T> x0 = xs[i0], x1 = xs[i1];
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    a0.v[r] += v.a * x0.v[r];
    a1.v[r] += v.b * x1.v[r];
  }
}

// matrix entries of a wave's slices in registers: N pairs of each row (longer rows read the rest again
// in every pass), with their values unless MC (coded: looked up in `dict`, in LDS). Rows of the 2-D
// auxiliary levels hold at most 6 entries: N = 3 there leaves registers for two FP64 blocks per CU.
template <class G, class T, bool MC, int N>
struct PatchRows {
  uint32_t id[G::slots][N];
  PPair<T> v[G::slots][N];
  int o[G::slots], w[G::slots];

  __device__ __forceinline__ PPair<T> value(uint32_t c, const T *dict) const {
    return PPair<T>{dict[c >> G::bits & 15u], dict[c >> (16 + G::bits)]};
  }

  template <int J0, int J1>
  __device__ __forceinline__ void load(const PatchView<T> &V, const PatchHead &h, int wv, uint32_t lane) {
#pragma unroll
    for (int j = J0; j < J1; ++j) {
      const int k = j * G::waves + wv;
      o[j] = h.poff[k];
      w[j] = h.poff[k + 1] - o[j];
      const uint32_t *ip = V.pidx + (size_t)o[j] * 64;
      const PPair<T> *vp = reinterpret_cast<const PPair<T> *>(V.pval) + (size_t)o[j] * 64;
#pragma unroll
      for (int q = 0; q < N; ++q)
        if (q < w[j]) {
          id[j][q] = at32(ip + q * 64, lane);
          if constexpr (!MC) v[j][q] = at32(vp + q * 64, lane);
        }
    }
  }
  // values of the codes (after the dictionary is in LDS)
  __device__ __forceinline__ void decode(const T *dict) {
    if constexpr (MC) {
#pragma unroll
      for (int j = 0; j < G::slots; ++j)
#pragma unroll
        for (int q = 0; q < N; ++q)
          if (q < w[j]) v[j][q] = value(id[j][q], dict);
    }
  }

  // the first W pairs: every LDS read before the first product
  template <int W, bool UP, int NR>
  __device__ __forceinline__ void add_w(PVec<NR, T> &a0, PVec<NR, T> &a1, int j, const PVec<NR, T> *xs,
                                        int above) const {
    PVec<NR, T> x0[W], x1[W];
    int i0[W], i1[W];
#pragma unroll
    for (int q = 0; q < W; ++q) {
      // unpacked here, not kept unpacked across the passes (32 more registers)
      uint32_t c = id[j][q];
      asm volatile("" : "+v"(c));
      i0[q] = (int)(c & ((1u << G::bits) - 1));
      i1[q] = (int)(c >> 16 & ((1u << G::bits) - 1));
      x0[q] = xs[i0[q]];
      x1[q] = xs[i1[q]];
    }
#pragma unroll
    for (int q = 0; q < W; ++q) {
      PPair<T> m = v[j][q];
      if (UP) {
        m.a = i0[q] > above ? m.a : T(0);
        m.b = i1[q] > above ? m.b : T(0);
      }
#pragma unroll
      for (int r = 0; r < NR; ++r) {
        a0.v[r] += m.a * x0[q].v[r];
        a1.v[r] += m.b * x1[q].v[r];
      }
    }
  }

  template <bool UP, int NR>
  __device__ __forceinline__ PVec<NR, T> dot(const PatchView<T> &V, int j, const PVec<NR, T> *xs, const T *dict,
                                             uint32_t lane, int above = 0) const {
    PVec<NR, T> a0, a1;
#pragma unroll
    for (int r = 0; r < NR; ++r) a0.v[r] = a1.v[r] = T(0);
    switch (w[j] < N ? w[j] : N) {
      case 0: break;
      case 1: add_w<1, UP, NR>(a0, a1, j, xs, above); break;
      case 2: add_w<2, UP, NR>(a0, a1, j, xs, above); break;
      case 3: add_w<3, UP, NR>(a0, a1, j, xs, above); break;
      case 4:
        if constexpr (N >= 4) add_w<4, UP, NR>(a0, a1, j, xs, above);
        break;
      default:
        if constexpr (N >= 5) add_w<5, UP, NR>(a0, a1, j, xs, above);
        break;
    }
    for (int q = N; q < w[j]; q += 4) {  // the rest of long rows, four pairs at a time
      uint32_t c[4];
      PPair<T> m[4];
#pragma unroll
      for (int t = 0; t < 4; ++t)
        if (q + t < w[j]) {
          c[t] = at32(V.pidx + (size_t)(o[j] + q + t) * 64, lane);
          if constexpr (!MC) m[t] = at32(reinterpret_cast<const PPair<T> *>(V.pval) + (size_t)(o[j] + q + t) * 64, lane);
        }
#pragma unroll
      for (int t = 0; t < 4; ++t)
        if (q + t < w[j]) {
          if constexpr (MC) m[t] = value(c[t], dict);
          pair_add<G::bits, UP, NR, T>(a0, a1, c[t], m[t], xs, above);
        }
    }
#pragma unroll
    for (int r = 0; r < NR; ++r) a0.v[r] += a1.v[r];
    return a0;
  }
};

__device__ __forceinline__ int patch_row(int g) { return g < 0 ? 0 : g & (kPatchHalo - 1); }
__device__ __forceinline__ bool patch_owns(int g) { return g >= 0 && !(g & kPatchHalo); }

// coarse slices of a wave loaded before the sweeps (coded transfers)
template <class T>
constexpr int kPatchCoarse = sizeof(T) == 8 ? 1 : 2;
static constexpr int kCoarsePairs = 4;  // entry pairs of each

// Waves per SIMD that the registers are held to: four (two blocks of PatchSmall per CU, one of PatchBig),
// or two where 64-bit values leave no room for that: on the original grid (rows of four pairs, gathers of
// Pi) and with four values a row. Six for one FP32 value (three blocks) spill: 9.0 ms a solve at 1M rows
// against 8.7.
template <class G, class T, bool TC>
constexpr int patch_waves(int NR) {
  return G::waves > 8 || sizeof(T) == 4 || (TC && NR <= 2) ? 4 : 2;
}

// whether `down` keeps the diagonal in LDS between the sweeps and the residual (else it is read again):
// two FP64 values a row leave no room for it beside a second block
template <class T, bool TC>
constexpr bool patch_diag(int NR) { return !(sizeof(T) == 8 && NR == 2 && TC); }

// RS: the vectors hold RS * NR values a row, and block p RS + k serves values k NR .. of patch p. Four
// FP64 values at once leave one block per CU (LDS, registers) and the memory idle while it computes; two
// halves run side by side and share the patch's matrix rows in L2 (40 meshes, 2860 patches: `down` 193 ->
// 187 us, `up` 185 -> 171). The original grid's kernels are bound by their gathers, each half of which
// fetches the same lines: one block there (`up` 362 us in two halves, 234 in one).
template <class T, bool TC>
constexpr int patch_split(int NR) { return NR * sizeof(T) > 16 && TC ? 2 : 1; }

// The FP64 reciprocal of the diagonal is computed (id holds the same bits); in FP32 id is 1/a_ii rounded
// once, the value that `up` multiplies with, where the reciprocal of the rounded diagonal can differ in the
// last bit.
// Forward sweeps from zero on b (BT: its type; FP64 on the original grid in both precisions), x on the
// own rows, and either the restricted residual bc on the coarse rows owned (fused) or the residual r.
template <class G, int NR, class T, class BT, bool MC, bool TC, int RS = 1>
__global__ __launch_bounds__(G::threads, (patch_waves<G, T, TC>(NR))) void k_patch_down(
    PatchView<T> V, int cells, int rows, int C, int nu, int fused, const BT *__restrict__ b, const T *__restrict__ dg,
    const T *__restrict__ id, T *__restrict__ x, T *__restrict__ r, T *__restrict__ bc, const int *__restrict__ done) {
  extern __shared__ __align__(32) unsigned char patch_lds[];
  __shared__ T dict[kPatchCodes];
  using X = PVec<NR, T>;
  X *xs = reinterpret_cast<X *>(patch_lds);
  const uint32_t lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int block = xcd_block(), patch = block / RS;
  const uint32_t sub = block % RS;
  int g[G::slots];
#pragma unroll
  for (int j = 0; j < G::slots; ++j)
    g[j] = at32(V.gidx + (size_t)(patch * G::slices + j * G::waves + wv) * 64, lane);
  const PatchHead &h = V.head[patch];
  const int ns = h.ns, nco = fused ? h.nco : 0;
  const int stop = done ? *done : 0;  // the solve has ended: nothing is written
  int turn[G::slots];  // colour of each slice, in scalar registers: the passes read no memory but LDS
#pragma unroll
  for (int j = 0; j < G::slots; ++j) turn[j] = (int)(h.sc[j] >> 4 * wv & 15);
  if (MC && threadIdx.x < kPatchCodes) dict[threadIdx.x] = V.pval[threadIdx.x];
  // (the rows of the 2-D auxiliary levels hold at most 6 entries: three pairs fit two FP64 blocks per CU)
  constexpr int pairs = G::waves > 8 ? G::template pairs<T> : TC ? 3 : G::template pairs<T>;
  PatchRows<G, T, MC, pairs> A;
  // the last slot's 64-bit values wait until b and the diagonal are out of their registers
  constexpr int early = sizeof(T) == 8 || G::waves > 8 ? G::slots - 1 : G::slots;
  A.template load<0, early>(V, h, wv, lane);
  X *bs = xs + cells;
  T *ds = reinterpret_cast<T *>(bs + rows);
  T iv[G::slots];
  {
    X bv[G::slots];
    T dv[G::slots];
#pragma unroll
    for (int j = 0; j < G::slots; ++j) {
      const int i = patch_row(g[j]);
      const PVec<NR, BT> t = at32(reinterpret_cast<const PVec<NR, BT> *>(b) + sub, i * RS);
#pragma unroll
      for (int q = 0; q < NR; ++q) bv[j].v[q] = (T)t.v[q];
      dv[j] = at32(dg, i);
      if constexpr (sizeof(T) == 4) iv[j] = at32(id, i);
    }
    if (stop) return;
    // colour 0 of the first sweep; every other cell starts from zero
#pragma unroll
    for (int j = 0; j < G::slots; ++j) {
      const int k = j * G::waves + wv;
      if (k >= ns) continue;
      if constexpr (sizeof(T) == 8) iv[j] = T(1) / dv[j];
      bs[k * 64 + lane] = bv[j];
      if constexpr (patch_diag<T, TC>(NR)) ds[k * 64 + lane] = dv[j];
      X o;
#pragma unroll
      for (int q = 0; q < NR; ++q) o.v[q] = turn[j] == 0 ? bv[j].v[q] * iv[j] : T(0);
      xs[k * 64 + lane] = o;
    }
    for (int k = ns + wv; k < h.ncs; k += G::waves) {
      X o;
#pragma unroll
      for (int q = 0; q < NR; ++q) o.v[q] = T(0);
      xs[k * 64 + lane] = o;
    }
  }
  // coarse rows of the restriction: their loads are in flight during the sweeps
  int crow[kPatchCoarse<T>], co[kPatchCoarse<T>], cw[kPatchCoarse<T>];
  uint32_t cid[kPatchCoarse<T>][kCoarsePairs];
  if (TC) {
#pragma unroll
    for (int j = 0; j < kPatchCoarse<T>; ++j) {
      const int k = j * G::waves + wv;
      co[j] = cw[j] = 0;
      crow[j] = -1;
      if (k < nco) {
        const bool in_head = k < kPatchHeadCoarse;
        co[j] = in_head ? h.roff[k] : V.roff[h.coarse0 + k];
        cw[j] = (in_head ? h.roff[k + 1] : V.roff[h.coarse0 + k + 1]) - co[j];
        crow[j] = at32(V.rrow + (size_t)(h.coarse0 + k) * 64, lane);
      }
#pragma unroll
      for (int q = 0; q < kCoarsePairs; ++q)
        if (q < cw[j]) cid[j][q] = at32(V.ridx + (size_t)(co[j] + q) * 64, lane);
    }
  }
  A.template load<early, G::slots>(V, h, wv, lane);
  __syncthreads();
  A.decode(dict);
  for (int s = 0; s < nu; ++s)
    for (int c = s == 0 ? 1 : 0; c < C; ++c) {
#pragma unroll
      for (int j = 0; j < G::slots; ++j) {
        const int k = j * G::waves + wv;
        if (turn[j] == c) {
          X a = A.template dot<false, NR>(V, j, xs, dict, lane);
#pragma unroll
          for (int q = 0; q < NR; ++q) a.v[q] = (bs[k * 64 + lane].v[q] - a.v[q]) * iv[j];
          xs[k * 64 + lane] = a;
        }
      }
      __syncthreads();
    }
  T dv[G::slots];
  if constexpr (!patch_diag<T, TC>(NR))
#pragma unroll
    for (int j = 0; j < G::slots; ++j) dv[j] = at32(dg, patch_row(g[j]));
  // x out; residual in b's place (zero on the last colour: its pass came last)
#pragma unroll
  for (int j = 0; j < G::slots; ++j) {
    const int k = j * G::waves + wv;
    if (k >= ns) continue;
    const X xi = xs[k * 64 + lane];
    if (patch_owns(g[j])) put32(reinterpret_cast<X *>(x) + sub, g[j] * RS, xi);
    X rv;
    if (turn[j] == C - 1) {
#pragma unroll
      for (int q = 0; q < NR; ++q) rv.v[q] = T(0);
    } else if (nu == 1) {  // after a single sweep from zero only the later colours' terms remain
      rv = A.template dot<true, NR>(V, j, xs, dict, lane, k * 64 + lane);
#pragma unroll
      for (int q = 0; q < NR; ++q) rv.v[q] = -rv.v[q];
    } else {
      rv = A.template dot<false, NR>(V, j, xs, dict, lane);
      const X bi = bs[k * 64 + lane];
      T d;
      if constexpr (patch_diag<T, TC>(NR))
        d = ds[k * 64 + lane];
      else
        d = dv[j];
#pragma unroll
      for (int q = 0; q < NR; ++q) rv.v[q] = bi.v[q] - d * xi.v[q] - rv.v[q];
    }
    bs[k * 64 + lane] = rv;
    if (!fused && patch_owns(g[j])) put32(reinterpret_cast<X *>(r) + sub, g[j] * RS, rv);
  }
  if (!fused) return;
  __syncthreads();
  auto add = [&](X &a0, X &a1, uint32_t id) {
    const PPair<T> v{patch_weight<T>(id >> G::bits & (65535u >> G::bits)), patch_weight<T>(id >> (16 + G::bits))};
    pair_add<G::bits, false, NR, T>(a0, a1, id, v, bs, 0);
  };
  auto put = [&](int row, X a0, const X &a1) {
    if (row < 0) return;
#pragma unroll
    for (int q = 0; q < NR; ++q) a0.v[q] += a1.v[q];
    put32(reinterpret_cast<X *>(bc) + sub, row * RS, a0);
  };
  int k = wv;
  if (TC) {
#pragma unroll
    for (int j = 0; j < kPatchCoarse<T>; ++j, k += G::waves)
      if (k < nco) {
        X a0, a1;
#pragma unroll
        for (int q = 0; q < NR; ++q) a0.v[q] = a1.v[q] = T(0);
#pragma unroll
        for (int q = 0; q < kCoarsePairs; ++q)
          if (q < cw[j]) add(a0, a1, cid[j][q]);
        for (int q = kCoarsePairs; q < cw[j]; ++q) add(a0, a1, at32(V.ridx + (size_t)(co[j] + q) * 64, lane));
        put(crow[j], a0, a1);
      }
  }
  for (; k < nco; k += G::waves) {
    const int row = at32(V.rrow + (size_t)(h.coarse0 + k) * 64, lane);
    const int o = V.roff[h.coarse0 + k], w = V.roff[h.coarse0 + k + 1] - o;
    X a0, a1;
#pragma unroll
    for (int q = 0; q < NR; ++q) a0.v[q] = a1.v[q] = T(0);
    for (int q = 0; q < w; q += 4) {
      uint32_t ids[4];
      PPair<T> vs[4];
#pragma unroll
      for (int t = 0; t < 4; ++t)
        if (q + t < w) {
          ids[t] = at32(V.ridx + (size_t)(o + q + t) * 64, lane);
          if constexpr (!TC)
            vs[t] = at32(reinterpret_cast<const PPair<T> *>(V.rval) + (size_t)(o + q + t) * 64, lane);
        }
#pragma unroll
      for (int t = 0; t < 4; ++t)
        if (q + t < w) {
          if constexpr (TC)
            add(a0, a1, ids[t]);
          else
            pair_add<G::bits, false, NR, T>(a0, a1, ids[t], vs[t], bs, 0);
        }
    }
    put(row, a0, a1);
  }
}

// Backward sweeps on b from x + P e, result in xo on the own rows (other patches still read x); with
// `part` also each patch's share of b.xo.
template <class G, int NR, class T, class BT, bool MC, bool TC, bool DOT = false, int RS = 1>
__global__ __launch_bounds__(G::threads, (patch_waves<G, T, TC>(NR))) void k_patch_up(
    PatchView<T> V, int cells, int C, int nu, const BT *__restrict__ b, const T *__restrict__ id,
    const T *__restrict__ x, const T *__restrict__ e, T *__restrict__ xo, double *__restrict__ part, const int *__restrict__ done) {
  extern __shared__ __align__(32) unsigned char patch_lds[];
  __shared__ T dict[kPatchCodes];
  using X = PVec<NR, T>;
  X *xs = reinterpret_cast<X *>(patch_lds);
  const uint32_t lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int block = xcd_block(), patch = block / RS;
  const uint32_t sub = block % RS;
  int g[G::slots];
#pragma unroll
  for (int j = 0; j < G::slots; ++j)
    g[j] = at32(V.gidx + (size_t)(patch * G::slices + j * G::waves + wv) * 64, lane);
  const PatchHead &h = V.head[patch];
  const int ns = h.ns, nst = h.nst;
  const int stop = done ? *done : 0;
  int turn[G::slots];
#pragma unroll
  for (int j = 0; j < G::slots; ++j) turn[j] = (int)(h.sc[j] >> 4 * wv & 15);
  if (MC && threadIdx.x < kPatchCodes) dict[threadIdx.x] = V.pval[threadIdx.x];
  X *bs = xs + cells;
  T iv[G::slots];
  // (the rows of the 2-D auxiliary levels hold at most 6 entries: three pairs fit two FP64 blocks per CU)
  constexpr int pairs = G::waves > 8 ? G::template pairs<T> : TC ? 3 : G::template pairs<T>;
  PatchRows<G, T, MC, pairs> A;
  // with 64-bit values the second half of the matrix rows is loaded after the prolongation: both at
  // once do not fit in the registers of two blocks per CU
  constexpr int early = G::waves > 8 || (sizeof(T) == 8 && TC) ? G::slots / 2 : G::slots;
  auto column = [](int c) { return TC ? c & 0xfffffff : c; };
  // Start rows, UB slices of a wave at a time: their indices (and values) come in while the slices before
  // gather, so a step waits for memory once, not twice (original grid, 1M rows in FP32: 79 -> 49 us, 122k rows
  // in FP64: 16.5 -> 13.5; two FP32 slices at a time 53). PW entries of a row are held (coded rows hold at most two, the
  // rows of Pi 6 on average); longer rows read the rest PW at a time.
  constexpr int PW = TC ? 2 : 8, UB = TC ? 3 : sizeof(T) == 8 && NR == 1 ? 2 : 1;
  struct Start {
    int ug[UB], cell[UB], o[UB], w[UB], uc[UB][PW];
    T uv[UB][PW];
  };
  auto fetch = [&](int k0, Start &t) {
#pragma unroll
    for (int i = 0; i < UB; ++i) {
      const int k = k0 + i * G::waves;
      t.ug[i] = -1;
      t.o[i] = t.w[i] = 0;
      if (k < nst) {
        t.ug[i] = at32(V.ugidx + (size_t)(h.start0 + k) * 64, lane);
        t.cell[i] = at32(V.ucell + (size_t)(h.start0 + k) * 64, lane);
        t.o[i] = h.uoff[k];
        t.w[i] = h.uoff[k + 1] - t.o[i];
      }
#pragma unroll
      for (int q = 0; q < PW; ++q)
        if (q < t.w[i]) {
          t.uc[i][q] = at32(V.ucol + (size_t)(t.o[i] + q) * 64, lane);
          if constexpr (!TC) t.uv[i][q] = at32(V.uval + (size_t)(t.o[i] + q) * 64, lane);
        }
    }
  };
  auto start = [&](int k0, const Start &t) {
    X a[UB], ev[UB][PW];
#pragma unroll
    for (int i = 0; i < UB; ++i) {
      if (k0 + i * G::waves < nst) a[i] = at32(reinterpret_cast<const X *>(x) + sub, t.ug[i] < 0 ? 0 : t.ug[i] * RS);
#pragma unroll
      for (int q = 0; q < PW; ++q)
        if (q < t.w[i]) ev[i][q] = at32(reinterpret_cast<const X *>(e) + sub, column(t.uc[i][q]) * RS);
    }
#pragma unroll
    for (int i = 0; i < UB; ++i) {
#pragma unroll
      for (int q = 0; q < PW; ++q)
        if (q < t.w[i]) {
          const T v = TC ? patch_weight<T>((uint32_t)t.uc[i][q] >> 28) : t.uv[i][q];
#pragma unroll
          for (int m = 0; m < NR; ++m) a[i].v[m] += v * ev[i][q].v[m];
        }
      for (int p = PW; p < t.w[i]; p += PW) {
        int c[PW];
        T v[PW];
        X ex[PW];
#pragma unroll
        for (int q = 0; q < PW; ++q)
          if (p + q < t.w[i]) {
            c[q] = at32(V.ucol + (size_t)(t.o[i] + p + q) * 64, lane);
            if constexpr (!TC) v[q] = at32(V.uval + (size_t)(t.o[i] + p + q) * 64, lane);
          }
#pragma unroll
        for (int q = 0; q < PW; ++q)
          if (p + q < t.w[i]) ex[q] = at32(reinterpret_cast<const X *>(e) + sub, column(c[q]) * RS);
#pragma unroll
        for (int q = 0; q < PW; ++q)
          if (p + q < t.w[i]) {
            const T f = TC ? patch_weight<T>((uint32_t)c[q] >> 28) : v[q];
#pragma unroll
            for (int m = 0; m < NR; ++m) a[i].v[m] += f * ex[q].v[m];
          }
      }
      if (t.ug[i] >= 0) xs[t.cell[i]] = a[i];
    }
  };
  // right-hand side and diagonal of the rows: their gathers fly with the first start rows'
  PVec<NR, BT> bv[G::slots];
  Start t0;
  fetch(wv, t0);
#pragma unroll
  for (int j = 0; j < G::slots; ++j) {
    const int i = patch_row(g[j]);
    bv[j] = at32(reinterpret_cast<const PVec<NR, BT> *>(b) + sub, i * RS);
    iv[j] = at32(id, i);
  }
  if constexpr (TC) A.template load<0, early>(V, h, wv, lane);
  if (stop) return;
  {
    Start t1;
    fetch(wv + UB * G::waves, t1);
    start(wv, t0);
    t0 = t1;
  }
#pragma unroll
  for (int j = 0; j < G::slots; ++j)
    if (j * G::waves + wv < ns) {
      X o;
#pragma unroll
      for (int q = 0; q < NR; ++q) o.v[q] = (T)bv[j].v[q];
      bs[(j * G::waves + wv) * 64 + lane] = o;
    }
  for (int k = wv + UB * G::waves; k < nst; k += UB * G::waves) {
    Start t1;
    fetch(k + UB * G::waves, t1);
    start(k, t0);
    t0 = t1;
  }
  if constexpr (!TC) A.template load<0, early>(V, h, wv, lane);
  A.template load<early, G::slots>(V, h, wv, lane);
  __syncthreads();
  A.decode(dict);
  for (int s = 0; s < nu; ++s)
    for (int c = C - 1; c >= 0; --c) {
#pragma unroll
      for (int j = 0; j < G::slots; ++j) {
        const int k = j * G::waves + wv;
        if (turn[j] == c) {
          X y = A.template dot<false, NR>(V, j, xs, dict, lane);
#pragma unroll
          for (int q = 0; q < NR; ++q) y.v[q] = (bs[k * 64 + lane].v[q] - y.v[q]) * iv[j];
          xs[k * 64 + lane] = y;
          // the last sweep's value is final
          if (s == nu - 1 && patch_owns(g[j])) put32(reinterpret_cast<X *>(xo) + sub, g[j] * RS, y);
        }
      }
      __syncthreads();
    }
  // partial sum of b.x over the own rows (FP64 b: the residual of the original grid)
  if constexpr (DOT) {
    double v = 0;
#pragma unroll
    for (int j = 0; j < G::slots; ++j)
      if (patch_owns(g[j])) v += at32(b, g[j]) * (double)xs[(j * G::waves + wv) * 64 + lane].v[0];
    __shared__ double sm[G::waves];
    v = group_sum<64>(v);
    if (lane == 0) sm[wv] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
      v = 0;
      for (int i = 0; i < G::waves; ++i) v += sm[i];
      part[patch] = v;
    }
  }
}

// map[slot] = entry of the level's matrix (CSR rp, ci, columns ascending) that each stored value of a patch
// came from, -1 = padding (a repeat of the row's first cell). One block per patch: the rows of its cells go
// to LDS, every pair looks its two columns up. Run once, at the first change of the coefficient; the host's patches
// built again for it took 65 of that call's 200 ms at 250k rows.
static __global__ __launch_bounds__(512) void k_patch_map(const PatchHead *head, const int *__restrict__ gidx,
                                                          const int *__restrict__ cgidx, const uint32_t *__restrict__ pidx,
                                                          int slices, int bits, const int *__restrict__ rp,
                                                          const int *__restrict__ ci, int *__restrict__ map) {
  extern __shared__ int row_of[];
  const PatchHead &h = head[blockIdx.x];
  const int *g = gidx + (size_t)blockIdx.x * slices * 64, *cg = cgidx + (size_t)h.cell0 * 64;
  for (int i = threadIdx.x; i < 64 * h.ncs; i += 512) {
    const int r = i < 64 * h.ns ? g[i] : cg[i - 64 * h.ns];
    row_of[i] = r < 0 ? -1 : patch_row(r);
  }
  __syncthreads();
  const uint32_t mask = (1u << bits) - 1;
  for (int i = threadIdx.x; i < 64 * h.ns; i += 512) {
    const int row = row_of[i], k = i >> 6;
    const int a = row < 0 ? 0 : rp[row], b = row < 0 ? 0 : rp[row + 1];
    auto entry = [&](int cell) {
      const int c = row_of[cell];
      int lo = a, hi = b;
      while (lo < hi) {
        const int m = (lo + hi) >> 1;
        if (ci[m] < c)
          lo = m + 1;
        else
          hi = m;
      }
      return lo < b && ci[lo] == c ? lo : -1;
    };
    for (int o = h.poff[k], q = o; q < h.poff[k + 1]; ++q) {
      const size_t at = (size_t)q * 64 + (i & 63);
      const int c0 = (int)(pidx[at] & mask), c1 = (int)(pidx[at] >> 16 & mask);
      const int first = (int)(pidx[(size_t)o * 64 + (i & 63)] & mask);
      map[2 * at] = q > o && c0 == first ? -1 : entry(c0);
      map[2 * at + 1] = c1 == first ? -1 : entry(c1);
    }
  }
}

static void patch_map(const DPatch &D, const int *rp, const int *ci, int *map, hipStream_t s) {
  const PatchShape sh = D.big ? kPatchBig : kPatchSmall;
  hipLaunchKernelGGL(k_patch_map, dim3(D.np), dim3(512), (size_t)D.cells * sizeof(int), s, D.head, D.gidx, D.cgidx,
                     D.pidx, sh.slices, sh.bits, rp, ci, map);
  HIPCHECK(hipGetLastError());
}

// new values of a coded matrix: the codes of its entries above their cell numbers (dict: `used` values, ascending)
static __global__ __launch_bounds__(BS) void k_patch_recode(int64_t npair, int bits, const int *__restrict__ map,
                                                            const double *__restrict__ v, int used,
                                                            const double *__restrict__ dict, uint32_t *__restrict__ pidx) {
  const int64_t i = (int64_t)blockIdx.x * BS + threadIdx.x;
  if (i >= npair) return;
  const uint32_t cells = (1u << bits) - 1;
  uint32_t c = pidx[i] & (cells | cells << 16);
  for (int h = 0; h < 2; ++h) {
    const int p = map[2 * i + h];
    const double x = p >= 0 ? v[p] : 0.0;
    uint32_t k = 0;
    while ((int)k < used - 1 && dict[k] < x) ++k;
    c |= k << (16 * h + bits);
  }
  pidx[i] = c;
}

// dictionary of a matrix's values; empty: more than kPatchCodes, it stays plain
template <class V>
static std::vector<double> patch_dict(const V &v) {
  std::vector<double> d{0.0};
  if (!patch_codes(v, d)) d.clear();
  return d;
}

// launch of a patch kernel; LDS: x on the cells, b (then the residual) and the
// diagonal on the rows, `vec` and `scalar` bytes each. The kernel's limit is set to what its largest patch can take,
// the same value at every launch: handles of other sizes launch it from other threads.
template <class G, class K, class... A>
static void launch_patch(K kernel, int grid, const DPatch &D, size_t vec, size_t scalar, hipStream_t s, hipEvent_t e0,
                         hipEvent_t e1, A... args) {
  constexpr PatchShape sh = G::waves == PatchBig::waves ? kPatchBig : kPatchSmall;
  const size_t lds = (size_t)D.cells * vec + (size_t)D.lrows * (vec + scalar);
  const size_t most = 64 * ((size_t)sh.cell_slices * vec + (size_t)sh.slices * (vec + scalar));
  if (most > 64 * 1024)
    HIPCHECK(hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                 (int)most));
  if (e0) {
    hipExtLaunchKernelGGL(kernel, dim3(grid), dim3(G::threads), lds, s, e0, e1, 0, args...);
    HIPCHECK(hipGetLastError());
  } else {
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(G::threads), lds, s, args...);
  }
}

// calls f(geometry, matrix coded, transfers coded) with the level's variant as compile-time values; BIG:
// the larger geometry is possible (its matrices are not coded)
template <bool BIG, class F>
static void with_codes(const DPatch &D, F &&f) {
  if constexpr (BIG)
    if (D.big) {
      if (D.tcode)
        f(PatchBig(), std::false_type(), std::true_type());
      else
        f(PatchBig(), std::false_type(), std::false_type());
      return;
    }
  if (D.mcode && D.tcode)
    f(PatchSmall(), std::true_type(), std::true_type());
  else if (D.tcode)
    f(PatchSmall(), std::false_type(), std::true_type());
  else if (D.mcode)
    f(PatchSmall(), std::true_type(), std::false_type());
  else
    f(PatchSmall(), std::false_type(), std::false_type());
}

}  // namespace asmg
