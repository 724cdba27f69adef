// The fused batched Krylov solvers (paper Sec. 3.2-3.6): one kernel launch, one
// team of lanes per system, the whole solve of each system inside the kernel.
//
// Control flow.  Teams that share a wave (16- or 32-lane teams) run in lockstep
// through the same instruction stream: every cross-lane operation is executed by
// all lanes, and per-team state changes are committed under per-team
// predicates.  A team that has finished keeps executing (its results are
// discarded) until every team of its wave has finished.  Multi-wave teams make
// identical decisions in every wave because every wave reads the same reduced
// bits, so all their barriers match.
//
// Stop test.  ||r||_2 <= tol*||b||_2 on the recurrence residual, confirmed on the
// true residual b - A x; if the confirmation fails and iterations remain, the
// method restarts from the true residual.  (The paper's Alg. 1 tests |r.z|
// against a threshold; its Tab. 2 lists a relative criterion, which is used.)
#pragma once
#include <type_traits>

#include "bs_device.hpp"

namespace bs {

__device__ __forceinline__ bool finite(double v) { return __builtin_isfinite(v); }

// Stop level on ||r||_2 (Tab. 2): tol * ||b||_2 (relative) or tol (absolute).
template <class G>
__device__ __forceinline__ double stop_limit(const G& g, double bn) {
  return (g.flags & kFlagAbsTol) ? g.tol : g.tol * bn;
}

// ------------------------------------------------------------ block Jacobi
// v of lane src of this wave (a cross-lane permute through the LDS crossbar,
// no memory access); every lane must be active.
__device__ __forceinline__ double shfl(double v, int src) {
  const int a = src << 2;
  const int lo = __builtin_amdgcn_ds_bpermute(a, __double2loint(v));
  const int hi = __builtin_amdgcn_ds_bpermute(a, __double2hiint(v));
  return __hiloint2double(hi, lo);
}

// Blocks of bs consecutive rows (bs = 2, 4 or 8; the last block may be
// shorter); M = the inverse of the block diagonal of A.  Per team in LDS: the
// inverse stored by columns, binv[j*rows + i] = entry (i, b0 + j) (b0 = i - i %
// bs), so that the lanes of a wave touch consecutive elements, and a
// row-indexed exchange buffer pbuf[rows].  The rows of one block always sit in
// one wave, on consecutive lanes (bs divides the rows a wave holds, and block
// Jacobi runs with row i on lane i of its team), so a wavefront-scope fence
// orders the exchanges.
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront", "local");
  __builtin_amdgcn_wave_barrier();
}

// Inverse of every diagonal block by Gauss-Jordan elimination without
// pivoting: for each pivot p, row p is scaled by the pivot's reciprocal (its
// diagonal entry becoming 1/pivot), then every other row r subtracts a_rp times
// it (its entry p becoming -a_rp/pivot).  A zero or non-finite pivot, or a
// non-finite entry of the result, makes the block the identity.  The block's
// entries are scattered from the register slots (their columns found by
// gathering a vector that holds each row's own index), the elimination runs in
// registers, and the result is stored by columns.  All lanes of the workgroup
// call it together.
//
// After the gather, every LDS access stays inside the wave that owns the rows:
// a block's rows lie in one wave, and its failure flag is the exchange entry
// of its first row.  Waves of a multi-wave team may therefore leave at
// different times and go straight into bj_apply, which writes only the
// entries of its own rows.
template <class TM, class RW>
__device__ void bj_setup(TM& tm, RW& A, const KArgs& g) {
  constexpr int R = RW::R;
  const int bs = g.block, n = A.nrows(g), rows = tm.bj_rows(), per = rows / R;
  double* binv = tm.bj_region(g);
  double* pbuf = binv + (size_t)rows * bs;
  const int lane = tm.lane;
  // clear the exchange buffer (also the per-block failure flags) and the rows
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int i = lane + r * per;
    pbuf[i] = 0.0;
#pragma unroll 1
    for (int j = 0; j < bs; ++j) binv[j * rows + i] = 0.0;
  }
  // each row's own index into buffer 1, then gather it through the slots
#pragma unroll
  for (int r = 0; r < R; ++r)
    if (A.ok[r]) lds_store<double>(A.vrow[r] + RW::kBuf, (double)A.row[r]);
  tm.sync();
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int i = A.row[r], b0 = i - (i & (bs - 1));
#pragma unroll
    for (int k0 = 0; k0 < RW::NZ; k0 += 4) {
      int col[4];
#pragma unroll
      for (int k = k0; k < k0 + 4 && k < RW::NZ; ++k)
        col[k - k0] = (int)lds_load<double>(A.c[r][k] + RW::kBuf);
#pragma unroll
      for (int k = k0; k < k0 + 4 && k < RW::NZ; ++k)
        if (A.ok[r] && A.real(r, k) && col[k - k0] >= b0 && col[k - k0] < b0 + bs)
          binv[(col[k - k0] - b0) * rows + i] = A.a[r][k];
      // four gathers in flight at a time
      __asm__ volatile("" ::: "memory");
    }
  }
  wave_lds_fence();
  // Gauss-Jordan in registers.  The rows of a block sit on consecutive lanes
  // of one wave (row i on lane i of its team: the plain layout), so each lane
  // reads the pivot row from its lane with a cross-lane permute.  Every row
  // other than p subtracts its entry p times row p scaled by one reciprocal of
  // the pivot; row p takes the scaled row.  A zero or non-finite pivot, or a
  // non-finite entry of the result, raises the block's flag (the exchange
  // entry of its first row, in the same wave) and the block becomes the
  // identity.  All lanes run every step (the permutes read every lane).
  const int me = threadIdx.x & (kWave - 1);
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int i = A.row[r], ib = i & (bs - 1), b0 = i - ib;
    double m[kMaxBlock];
    bool bad = false;
#pragma unroll
    for (int j = 0; j < kMaxBlock; ++j) m[j] = (A.ok[r] && j < bs) ? binv[j * rows + i] : 0.0;
#pragma unroll 1
    for (int p = 0; p < bs; ++p) {
      const int src = me - ib + p;  // lane of row b0 + p
      double q[kMaxBlock];
#pragma unroll
      for (int j = 0; j < kMaxBlock; ++j) q[j] = j < bs ? shfl(m[j], src) : 0.0;
      double piv = q[0], f = m[0];
#pragma unroll
      for (int j = 1; j < kMaxBlock; ++j) {
        piv = j == p ? q[j] : piv;
        f = j == p ? m[j] : f;
      }
      const bool act = A.ok[r] && b0 + p < n, own = ib == p;
      if (act && (piv == 0.0 || !__builtin_isfinite(piv))) bad = true;
      const double rp = 1.0 / piv;
#pragma unroll
      for (int j = 0; j < kMaxBlock; ++j) {
        const double qs = (j == p ? 1.0 : q[j]) * rp;  // row p after this step
        const double upd = own ? qs : fma(-f, qs, j == p ? 0.0 : m[j]);
        m[j] = act ? upd : m[j];
      }
    }
#pragma unroll
    for (int j = 0; j < kMaxBlock; ++j) bad = bad || (j < bs && !__builtin_isfinite(m[j]));
    if (A.ok[r] && bad) pbuf[b0] = 1.0;
    wave_lds_fence();
    if (A.ok[r]) {
      const bool ident = pbuf[b0] != 0.0;
#pragma unroll
      for (int j = 0; j < kMaxBlock; ++j)
        if (j < bs) binv[j * rows + i] = ident ? (j == ib ? 1.0 : 0.0) : m[j];
    }
  }
  wave_lds_fence();
#pragma unroll
  for (int r = 0; r < R; ++r) pbuf[lane + r * per] = 0.0;
  wave_lds_fence();
}

// z = M v for the block-Jacobi M (rows past n give 0).  All lanes of a wave call
// it together.
template <class T, class TM, class RW>
__device__ __forceinline__ void bj_apply(TM& tm, const RW& A, const KArgs& g,
                                         const T (&v)[RW::R], T (&z)[RW::R]) {
  constexpr int R = RW::R;
  const int bs = g.block, rows = tm.bj_rows();
  const double* binv = tm.bj_region(g);
  double* pbuf = tm.bj_region(g) + (size_t)rows * bs;
#pragma unroll
  for (int r = 0; r < R; ++r)
    if (A.ok[r]) pbuf[A.row[r]] = (double)v[r];
  wave_lds_fence();
#pragma unroll
  for (int r = 0; r < R; ++r) {
    T acc = (T)0;
    if (A.ok[r]) {
      const int i = A.row[r], b0 = i - (i & (bs - 1));
      // four columns of the inverse row and of the block's slice of v per
      // batch of loads
#pragma unroll
      for (int h = 0; h < kMaxBlock; h += 4) {
        if (h >= bs) break;
        double w[4], u[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          w[j] = h + j < bs ? binv[(h + j) * rows + i] : 0.0;
          u[j] = h + j < bs ? pbuf[b0 + h + j] : 0.0;
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) acc = fma((T)w[j], (T)u[j], acc);
      }
    }
    z[r] = acc;
  }
  wave_lds_fence();
}

// ------------------------------------------------------------------ ILU(0)
// ILU(0) for one-wave teams (row i on lane i, one row per lane, n <= 64).  The
// factors live in the team's LDS region as F, row-major with an odd stride
// (the rows of a wave fall on distinct bank pairs) and zero columns padding
// each row to a multiple of 8: L strictly below the diagonal (unit diagonal
// implied), U on and above, zero off the pattern.

// Lanes past lane k (all 64-bit shifts stay below 64).
__device__ __forceinline__ uint64_t lanes_past(int k) { return (~0ull << k) << 1; }

// Factorization (Saad 2003, Sec. 10.3.2), right-looking: for pivot k, every row
// i > k that holds column k replaces that entry by l_ik = a_ik / u_kk (a
// division, as the IKJ form writes it) and subtracts l_ik u_kj from each of
// its entries j > k.  The pattern's schedule lists the pivots' columns, four
// per record, each with the rows that hold it below the pivot: a record comes
// through the scalar cache while the one before it is worked on, so a column
// costs its two reads, its update and its store (the lanes that do not hold
// it store to their own cell of a vector buffer, which nothing reads before it
// is written again).  Finding the columns and their rows from bit masks here
// took about 25 instructions per column, most of them one scalar chain: 0.79
// against 0.44 ms for loading and factoring 16384 systems of 54 rows.  What is
// left is the LDS: three operations of a whole wave per column, about 80 % of
// the LDS cycles of this phase; reading the pivot row once and its entries out
// of the lanes takes a third of them away and is slower (0.49 ms).  Each entry
// receives its updates in increasing k, as in the IKJ form.  d gets the pivot
// u_ii (1 on idle lanes), which the backward sweep divides by.  A zero pivot
// or a non-finite factor entry anywhere in the system turns M into the
// identity (F zero, d = 1).
template <class TM, class RW>
__device__ void ilu_setup(TM& tm, RW& A, const KArgs& g, double (&d)[RW::R]) {
  static_assert(RW::R == 1 && RW::TEAM == kWave, "ILU(0) runs on one-wave teams");
  const int n = g.n, st = ilu_stride(n);
  const unsigned F = lds_addr(tm.bj_region(g));
  const int lane = tm.lane;
  const bool ok = A.ok[0];
  const int i = ok ? A.row[0] : 0;  // rows past n address row 0 and never store
  const unsigned fi = F + (unsigned)(i * st) * 8, spare = A.vrow[0];
  auto clear = [&]() {
    for (unsigned e = 16u * (unsigned)lane; e < (unsigned)ilu_bytes(n); e += 16u * kWave)
      lds_store<uint4v>(F + e, uint4v{0, 0, 0, 0});
  };
  clear();
  wave_lds_fence();
  // slot s holds column (c - b0) / 8: its place in the row is c moved from the
  // vector buffer to the row; empty slots go to the spare cell.  (The zero
  // cell's address is opaque per system: the slots' masks would otherwise be
  // formed once per kernel and spill.)
  unsigned zc = A.zc;
  __asm__ volatile("" : "+v"(zc));
#pragma unroll
  for (int s = 0; s < RW::NZ; ++s)
    lds_store<double>(A.c[0][s] != zc ? A.c[0][s] - A.b0 + fi : spare, A.a[0][s]);
  wave_lds_fence();
  // Three sets of registers in turn: a record's load is issued two records
  // ahead, once the LDS reads of that time have arrived (scalar loads share
  // the LDS counter out of order, and a load in flight at the reads' wait has
  // to arrive too: issued just ahead of the reads it set the pace).
  typedef const __attribute__((address_space(4))) uint16v* Records;
  Records rec = (Records)(uintptr_t)g.ilu64;
  double l = 0.0;
  auto work = [&](const uint16v& w, uint16v& fresh, int ahead) {
    unsigned fk = F + w[15];  // row k
    const unsigned k8 = w[14] & 0x7fffffffu;
    const bool first = w[14] >> 31;  // first record of pivot k
    double piv = 1.0, aik = 0.0, u[4], f[4];
    wave_lds_fence();
    if (first) {
      piv = lds_load<double>(fk + k8);
      aik = lds_load<double>(fi + k8);
    }
    __asm__ volatile("" : "+v"(fk));  // one vector addition per column
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      u[q] = lds_load<double>(fk + w[8 + q]);
      f[q] = lds_load<double>(fi + w[8 + q]);
    }
    __asm__ volatile("" : "+v"(u[0]), "+v"(u[1]), "+v"(u[2]), "+v"(u[3]), "+v"(f[0]), "+v"(f[1]),
                          "+v"(f[2]), "+v"(f[3]), "+v"(piv), "+v"(aik));
    __builtin_amdgcn_sched_barrier(0);
    fresh = rec[ahead];
    if (first) {
      l = aik / piv;
      const uint64_t below = (uint64_t)w[13] << 32 | w[12];
      lds_store<double>(__builtin_amdgcn_inverse_ballot_w64(below) ? fi + k8 : spare, l);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const uint64_t rows = (uint64_t)w[2 * q + 1] << 32 | w[2 * q];
      lds_store<double>(__builtin_amdgcn_inverse_ballot_w64(rows) ? fi + w[8 + q] : spare,
                        fma(-l, u[q], f[q]));
    }
  };
  uint16v w0 = rec[0], w1 = rec[1], w2;
  // a multiple of three records, and two empty ones that are read ahead
  for (int r = g.ilu64_records; r > 0; r -= 3, rec += 3) {
    work(w0, w2, 2);
    work(w1, w0, 3);
    work(w2, w1, 4);
  }
  wave_lds_fence();
  // a zero pivot or a non-finite entry: the identity for the whole system
  // (0 * entry, summed over the row, is not a number then)
  const double pivot = ok ? lds_load<double>(fi + i * 8) : 1.0;
  double sum[2] = {0.0, 0.0};
  for (int j = 0; j < st - 1; j += 8) {
    double f[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) f[q] = lds_load<double>(fi + (j + q) * 8);
#pragma unroll
    for (int q = 0; q < 8; ++q) sum[q & 1] = fma(f[q], 0.0, sum[q & 1]);
  }
  const bool bad = pivot == 0.0 || !__builtin_isfinite(sum[0] + sum[1]);
  if (wave_any(bad)) {
    wave_lds_fence();
    clear();
    d[0] = 1.0;
  } else {
    d[0] = pivot;
  }
  wave_lds_fence();
}

// G consecutive doubles of a lane's row.  ILU(0) takes groups of eight (its rows
// are padded to that), BatchTrsv of four, which still cover a read's latency and
// hold 16 registers less.
template <int G>
struct Group {
  double v[G];
};
template <int G>
__device__ __forceinline__ Group<G> group_at(unsigned at) {
  Group<G> e;
#pragma unroll
  for (int q = 0; q < G; ++q) e.v[q] = lds_load<double>(at + q * 8);
  return e;
}

// A column sweep over columns 0..cols-1 (a multiple of G, at most 64) of a
// lane's row at fi, in increasing (UP) or decreasing order: step(k, entry).
// Unrolled over all 64 columns, so that lanes and masks are constants (a lane
// number from a scalar register costs a step 16 more cycles) and the reads of
// the next G entries issue in the gaps of a group's chain; groups past cols
// are skipped.  A group reads ahead up to G doubles past the row.  CUT: the
// columns n .. cols-1 hold other rows' entries, taken as zero (decreasing order,
// where they are the first group's).
template <bool UP, int G, bool CUT = false, class STEP>
__device__ __forceinline__ void sweep_columns(unsigned fi, int cols, STEP step, [[maybe_unused]] int n = 0) {
  static_assert(!UP || !CUT, "an increasing sweep masks its own columns past the rows");
  Group<G> t = group_at<G>(fi + (UP ? 0 : cols - G) * 8);
  if constexpr (CUT) {
#pragma unroll
    for (int q = 1; q < G; ++q) t.v[q] = cols - G + q < n ? t.v[q] : 0.0;
  }
#pragma unroll
  for (int h = 0; h < kWave / G; ++h) {
    const int k0 = UP ? G * h : kWave - G - G * h;
    if (k0 < cols) {
      // this group's entries first (read a group ago): issued behind the next
      // group's reads, their wait would cover those too
#pragma unroll
      for (int q = 0; q < G; ++q) __asm__ volatile("" : "+v"(t.v[q]));
      Group<G> next = t;
      if (h < kWave / G - 1) next = group_at<G>(fi + (UP ? k0 + G : k0 - G) * 8);
#pragma unroll
      for (int q = 0; q < G; ++q) step(k0 + (UP ? q : G - 1 - q), t.v[UP ? q : G - 1 - q]);
      t = next;
    }
  }
}

// a / d from 1 / d in two words, r + e: the error of the sum that is rounded is
// under 2^-104 of the quotient, so the result is the correctly rounded one
// unless the quotient lies that near to the middle of two doubles; two
// dependent operations where the division takes about a dozen.  Holds while no
// intermediate leaves the normal range, which quotient_safe() makes sure of.
__device__ __forceinline__ double quotient(double a, double r, double e) { return fma(a, r, a * e); }
__device__ __forceinline__ bool quotient_safe(double a, double d) {
  const double x = fabs(a), y = fabs(d);
  return (x == 0.0 || (x > 0x1p-500 && x < 0x1p500)) && y > 0x1p-400 && y < 0x1p400;
}

// z = (L U)^{-1} v by two column sweeps: forward, y_k (final on lane k) is
// read out and every row i > k subtracts l_ik y_k; backward, z_j = y_j / u_jj
// (the quotient by the pivot d of lane j) and every row i < j subtracts u_ij
// z_j.  The lanes that subtract are a mask formed in scalar registers.  Entries
// off the pattern and the padding columns add nothing.  The sums run in
// increasing k (forward) and decreasing j (backward).  With M the identity F
// is zero and d = 1, so z = v.
//
// The sweeps are chains of n dependent steps and bound by a step's latency
// (30 cycles forward, most of them the read-out of a lane and its first use):
// 100 us per BiCGSTAB iteration of 16384 systems of 54 rows, where the rolled
// form with divisions took 150.
// A lane's value no longer changes once its step has passed, so one test
// behind the backward sweep covers every quotient taken; out of range, the
// sweep is repeated with divisions.
template <class T, class TM, class RW>
__device__ __forceinline__ void ilu_apply(TM& tm, const RW& A, const KArgs& g,
                                          const T (&d)[RW::R], const T (&v)[RW::R],
                                          T (&z)[RW::R]) {
  const int n = g.n, st = ilu_stride(n), n8 = st - 1;
  const bool ok = A.ok[0];
  const unsigned fi = lds_addr(tm.bj_region(g)) + (unsigned)((ok ? A.row[0] : 0) * st) * 8;
  const uint64_t rows = ~0ull >> (kWave - n);  // idle lanes take no term
  const double dv = (double)d[0], r = 1.0 / dv, e = fma(-dv, r, 1.0) * r;
  double acc = ok ? (double)v[0] : 0.0;
  sweep_columns<true, 8>(fi, n8, [&](int k, double f) {
    const double y = rdlane(acc, k);
    if (__builtin_amdgcn_inverse_ballot_w64(lanes_past(k) & rows)) acc = fma(-f, y, acc);
  });
  const double y0 = acc;
  sweep_columns<false, 8>(fi, n8, [&](int j, double f) {
    const double zj = rdlane(quotient(acc, r, e), j);
    if (__builtin_amdgcn_inverse_ballot_w64(~(~0ull << j) & rows)) acc = fma(-f, zj, acc);
  });
  double zz = quotient(acc, r, e);
  if (wave_any(!quotient_safe(acc, dv))) {
    acc = y0;
    for (int j = n - 1; j > 0; --j) {
      const double zj = rdlane(acc / dv, j);
      if (__builtin_amdgcn_inverse_ballot_w64(~(~0ull << j)))
        acc = fma(-lds_load<double>(fi + j * 8), zj, acc);
    }
    zz = acc / dv;
  }
  z[0] = ok ? (T)zz : (T)0;
}

// ------------------------------------------------ ILU(0), multi-wave teams
// Teams of 2..16 waves (row i on lane i, one row per lane, up to 1024 rows)
// keep the factors sparse (bs::IluMw) and run the factorization and both sweeps
// level by level (level scheduling; Saad 2003, Ch. 11): a row's level in the
// lower triangle is one more than the largest level among the rows its strictly
// lower entries name (0 if none), and its level in the upper triangle is
// defined the same way from its strictly upper entries.  Rows of one level
// depend only on earlier levels.  The factorization takes one level per team
// barrier, each lane its own row; the sweeps run on the team's first wave
// alone, whose LDS operations complete in issue order, so that levels follow
// one another without a barrier.  The levels and schedules come with the
// pattern.

// The region's constant cells, once per kernel: the zero of the factor array
// and the one behind the sweep vector.  (The next barrier orders them.)
template <class TM>
__device__ __forceinline__ void tri_cells(TM& tm, const KArgs& g, unsigned reg, const IluMw& L) {
  if (tm.lists) return;
  if (threadIdx.x == 0) {
    lds_store<double>(reg + L.f + (g.noff + g.n) * 8, 0.0);
    lds_store<double>(reg + L.f + (g.noff + g.n + 1) * 8, 0.0);
    lds_store<double>(reg + L.y + g.n * 8, 0.0);
    // a record's four values of a one-row system reach one cell further
    if (g.n == 1) lds_store<double>(reg + L.f + 3 * 8, 0.0);
  }
  tm.lists = true;
}

// One triangular sweep by the team's first wave: for the rows of each level
// in turn, out_r <- (in_r - sum_c t_rc out_c) [/ d_r] (DIV), the row's strictly
// lower or upper terms in increasing column, rows at their places in the
// sweep's order.  COPY also stores the result at the row's place in the upper
// order.  SEL: the values may be other than finite, so the ones past a row's
// last term are replaced by zero (otherwise they meet the zero cell).  ONE: no
// row takes more than one segment; lanes without a row then store like the
// others, to the cell kept for them.  `divide`: by division instead of the
// reciprocal in two words.
//
// A segment (the four first terms of a level's rows, then the next four ..) is
// one record per lane, read from memory four segments ahead; everything but the
// gathers of the sweep vector is read from LDS one segment ahead, so a level
// waits for its gathers, four multiplications, the quotient and the store.
// Bound by the issue of one wave's instructions, about 40 per segment.
// Finding a row, its list range, its list words and then its values and
// gathers one after another in LDS took 700 cycles per level of the 992-row
// stencil (up to 16 rows), now 200.
template <bool DIV, bool SEL, bool COPY, bool ONE>
__device__ __forceinline__ void tri_sweep(const int4* __restrict__ segs, int nseg, int w, unsigned F,
                                          unsigned in, unsigned out, unsigned D, unsigned RE,
                                          unsigned copy, bool divide) {
  const int4* rec = segs + (threadIdx.x & ((1 << w) - 1));
  struct Seg {
    double f[4], a, r, e;
    unsigned c0, c1, own, tag;
  };
  auto fetch = [&](const int4& q) {
    Seg s;
    s.c0 = (unsigned)q.x;
    s.c1 = (unsigned)q.y;
    s.own = (unsigned)q.z;
    s.tag = (unsigned)q.w;
    const unsigned fa = F + (s.tag & 0x7fffu) * 8, o = s.own & 0xffffu;
#pragma unroll
    for (int k = 0; k < 4; ++k) s.f[k] = lds_load<double>(fa + k * 8);
    s.a = lds_load<double>(in + o);
    if constexpr (DIV) {
      typedef double double2v __attribute__((ext_vector_type(2)));
      const double2v re = lds_load<double2v>(RE + o * 2);
      s.r = re.x;
      s.e = re.y;
    } else {
      s.r = s.e = 0.0;
    }
    return s;
  };
  int4 q[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) q[u] = rec[u << w];
  rec += 4 << w;
  Seg s = fetch(q[0]);
  double acc = 0.0;
  for (int t = 0; t < nseg; t += 4, rec += 4 << w) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      double y[4];
      y[0] = lds_load<double>(out + (s.c0 & 0xffffu));
      y[1] = lds_load<double>(out + (s.c0 >> 16));
      y[2] = lds_load<double>(out + (s.c1 & 0xffffu));
      y[3] = lds_load<double>(out + (s.c1 >> 16));
      const Seg next = fetch(q[(u + 1) & 3]);
      q[u] = rec[u << w];
      const int terms = (int)(s.tag >> 16) & 7;
      acc = ONE || (s.tag & (1u << 30)) ? s.a : acc;
#pragma unroll
      for (int k = 0; k < 4; ++k) acc = fma(SEL && k >= terms ? 0.0 : -s.f[k], y[k], acc);
      double v = acc;
      if constexpr (DIV) {
        v = quotient(acc, s.r, s.e);
        if (divide) v = acc / lds_load<double>(D + (s.own & 0xffffu));
      }
      if (ONE || (int)s.tag < 0) {
        lds_store<double>(out + (s.own & 0xffffu), v);
        if constexpr (COPY) lds_store<double>(copy + (s.own >> 16), v);
      }
      __asm__ volatile("" ::: "memory");
      s = next;
    }
  }
}

// The sweep of a triangle by the first wave, between two team barriers, for a
// sweep that divides; x is this lane's result, read at place `me`.  The
// quotients are those of a division while |d| and the result stay within
// 2^-400 .. 2^400 (or the result is zero): outside, the sweep is run again with
// divisions.
template <bool SEL, class TM>
__device__ __forceinline__ double divided_sweep(TM& tm, const KArgs& g, const IluMw& L, unsigned reg,
                                                bool lower, bool ok, unsigned me, bool divide) {
  const unsigned F = reg + L.f, Y = reg + L.y, V = reg + L.v, D = F + g.noff * 8, RE = reg + L.re;
  const int4* segs = lower ? g.seg_l : g.seg_u;
  const int nseg = lower ? g.nseg_l : g.nseg_u, w = lower ? g.wseg_l : g.wseg_u;
  for (;;) {
    if (threadIdx.x < kWave) {
      if (lower ? g.one_l : g.one_u) tri_sweep<true, SEL, false, true>(segs, nseg, w, F, V, Y, D, RE, 0, divide);
      else tri_sweep<true, SEL, false, false>(segs, nseg, w, F, V, Y, D, RE, 0, divide);
    }
    tm.sync();
    const double x = ok ? lds_load<double>(Y + me) : 0.0;
    const bool far = !divide && x != 0.0 && !(fabs(x) > 0x1p-400 && fabs(x) < 0x1p400);
    if (__syncthreads_or(far) == 0) return x;
    divide = true;
  }
}

// A pivot's reciprocal in two words (see quotient), as the sweeps read them.
__device__ __forceinline__ void store_reciprocal(unsigned at, double d) {
  const double r = 1.0 / d;
  lds_store<double>(at, r);
  lds_store<double>(at + 8, fma(-d, r, 1.0) * r);
}

// Factorization, the IKJ form of the one-wave code, from the pattern's
// schedule: at its level, row i takes the columns k < i it holds in increasing
// order, replaces f_ik by f_ik / u_kk and subtracts f_ik u_kj from each of its
// entries (i,j), j > k, that row k holds.  Row k is final by then; row i's
// values are updated in place in LDS, where no other row of its level reads
// them.  Each entry so receives its updates in increasing k.  The row then
// stores its pivot's reciprocal.  Lane q takes the q-th row in lower order, so
// that one wave or two work on a level and the others only meet its barrier
// (with row i on lane i, up to 16 waves had a row each); a pivot and four of
// its updates are one group of schedule words, whose LDS reads go out together.
// 204 us per system of 992 rows with every update waiting for its own reads,
// now 121 (reading the system included).  A zero pivot or a non-finite factor
// entry anywhere in the system turns M into the identity (row values 0, pivots
// 1).
template <class TM, class RW>
__device__ void ilu_setup_mw(TM& tm, const RW& A, const KArgs& g) {
  static_assert(RW::R == 1 && RW::TEAM > kWave, "multi-wave ILU(0): one row per lane");
  constexpr int NZ = RW::NZ;
  const IluMw L = ilu_mw_layout(g.n, g.nnz);
  const unsigned reg = lds_addr(tm.bj_region(g));
  const unsigned F = reg + L.f, D = F + g.noff * 8, RE = reg + L.re;
  tri_cells(tm, g, reg, L);
  const bool ok = A.ok[0];
  int i = ok ? A.row[0] : 0;
  // opaque once per system: everything below derives from the pattern, and
  // would otherwise be loaded or formed once per kernel and pin registers
  // through the whole solve
  __asm__ volatile("" : "+v"(i));
  const int e0 = g.fmt == 0 ? A.w[0] : g.row_ptr[i];  // CSR position of register slot 0
  tm.place = (unsigned)g.tri_place[i];
  // the lane's row in lower order (ok also tells whether there is one)
  const int lv = ok ? g.lev[i] : -1;
  const unsigned up = (unsigned)g.tri_up[i];
  // Shapes of up to 16 slots load the row's first groups before the level loop
  // (all lanes at once); wider ones, short of registers, load them when the
  // row's level comes.
  constexpr int kEarly = NZ <= 16 ? 4 : 0;
  const int o0 = g.ilu_ptr[i], o1 = ok ? g.ilu_ptr[i + 1] : o0;
  unsigned w[kEarly > 0 ? kEarly : 1][5];
#pragma unroll
  for (int q = 0; q < kEarly; ++q)
#pragma unroll
    for (int u = 0; u < 5; ++u) w[q][u] = o0 + 5 * q < o1 ? (unsigned)g.ilu_ops[o0 + 5 * q + u] : 0u;
  // publish row i's values (a row without a stored diagonal has pivot 0)
  if (ok) {
    if (A.dslot[0] < 0) lds_store<double>(D + (tm.place >> 16) * 8, 0.0);
#pragma unroll
    for (int s = 0; s < NZ; ++s)
      if (A.real(0, s)) lds_store<double>(F + g.tri_pos[e0 + s] * 8, A.a[0][s]);
  }
  tm.sync();
  double lik = 0.0;
  auto group = [&](const unsigned (&v)[5]) {
    const bool head = v[0] >> 31;
    const unsigned aik = F + (v[0] & 0x7fffu) * 8, kk = (v[0] >> 15) & 0xffffu;
    double a = 0.0, d = 1.0, r = 1.0, e = 0.0, x[4], y[4];
    if (head) {
      a = lds_load<double>(aik);
      d = lds_load<double>(F + kk * 8);
      r = lds_load<double>(RE + (kk - g.noff) * 16);
      e = lds_load<double>(RE + (kk - g.noff) * 16 + 8);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      x[q] = lds_load<double>(F + (v[1 + q] & 0xffffu) * 8);
      y[q] = lds_load<double>(F + (v[1 + q] >> 16) * 8);
    }
    if (head) {
      lik = quotient(a, r, e);
      if (!quotient_safe(a, d)) lik = a / d;
      lds_store<double>(aik, lik);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) lds_store<double>(F + (v[1 + q] & 0xffffu) * 8, fma(-lik, y[q], x[q]));
  };
  for (int l = 0; l < g.nlev; ++l) {
    if (lv == l) {
#pragma unroll
      for (int q = 0; q < kEarly; ++q)
        if (o0 + 5 * q < o1) group(w[q]);
      for (int o = o0 + 5 * kEarly; o < o1; o += 5) {
        unsigned v[5];
#pragma unroll
        for (int u = 0; u < 5; ++u) v[u] = (unsigned)g.ilu_ops[o + u];
        group(v);
      }
      store_reciprocal(RE + up * 16, lds_load<double>(D + up * 8));
    }
    tm.sync();
  }
  // an infinite quotient of this system left no number in the discard cell,
  // which the records of the smallest systems read (against the zero cell)
  if (threadIdx.x == 0) lds_store<double>(F + (g.noff + g.n) * 8, 0.0);
  bool bad = false, wide = false;
  if (ok) {
    const double d = lds_load<double>(D + (tm.place >> 16) * 8);
    double sum = 0.0;  // of 0 * entry: not a number when one is not finite
#pragma unroll
    for (int s = 0; s < NZ; ++s)
      if (A.real(0, s)) sum = fma(lds_load<double>(F + g.tri_pos[e0 + s] * 8), 0.0, sum);
    bad = d == 0.0 || !__builtin_isfinite(sum);
    wide = !quotient_safe(0.0, d);
  }
  tm.divide = __syncthreads_or(wide) != 0;
  if (__syncthreads_or(bad)) {
    tm.divide = false;
    if (ok) {
#pragma unroll
      for (int s = 0; s < NZ; ++s)
        if (A.real(0, s)) lds_store<double>(F + g.tri_pos[e0 + s] * 8, 0.0);
      lds_store<double>(D + (tm.place >> 16) * 8, 1.0);
      store_reciprocal(RE + (tm.place >> 16) * 16, 1.0);
    }
    tm.sync();
  }
}

// z = (L U)^{-1} v by the two row-oriented substitutions of the oracle's
// default form on the team's first wave: forward, y_i = v_i - sum_{k<i} l_ik
// y_k; backward, z_i = (y_i - sum_{j>i} u_ij z_j) / u_ii, each row's terms in
// increasing column.  With M the identity the row values are zero and the
// pivots 1, so z = v.
template <class T, class TM, class RW>
__device__ __forceinline__ void ilu_apply_mw(TM& tm, const RW& A, const KArgs& g,
                                             const T (&v)[RW::R], T (&z)[RW::R]) {
  const IluMw L = ilu_mw_layout(g.n, g.nnz);
  const unsigned reg = lds_addr(tm.bj_region(g));
  const unsigned F = reg + L.f, Y = reg + L.y, V = reg + L.v;
  const bool ok = A.ok[0];
  if (ok) lds_store<double>(Y + (tm.place & 0xffffu) * 8, (double)v[0]);
  tm.sync();
  if (threadIdx.x < kWave) {
    if (g.one_l) tri_sweep<false, false, true, true>(g.seg_l, g.nseg_l, g.wseg_l, F, Y, Y, 0, 0, V, false);
    else tri_sweep<false, false, true, false>(g.seg_l, g.nseg_l, g.wseg_l, F, Y, Y, 0, 0, V, false);
  }
  z[0] = (T)divided_sweep<false>(tm, g, L, reg, false, ok, (tm.place >> 16) * 8, tm.divide);
}

// z = M v: block Jacobi or ILU(0) in their instances, else the diagonal d
// (scalar Jacobi, or 1 without a preconditioner).
template <int PK, class T, class TM, class RW>
__device__ __forceinline__ void precond(TM& tm, const RW& A, const KArgs& g, const T (&d)[RW::R],
                                        const T (&v)[RW::R], T (&z)[RW::R]) {
  if constexpr (PK == kPkBlock) {
    bj_apply(tm, A, g, v, z);
  } else if constexpr (PK == kPkIlu) {
    if constexpr (RW::TEAM > kWave) ilu_apply_mw(tm, A, g, v, z);
    else ilu_apply(tm, A, g, d, v, z);
  } else {
#pragma unroll
    for (int r = 0; r < RW::R; ++r) z[r] = d[r] * v[r];
  }
}

// Shared epilogue: true residual for teams that do not have it, then outputs.
template <class TM, class RW>
__device__ __forceinline__ void finish(TM& tm, const RW& A, const KArgs& g,
                                       const double (&b)[RW::R], const double (&x)[RW::R], int st,
                                       int k, int outer, double bn, double rn, bool have_rn) {
  // the output addresses first: their scalar loads then overlap the residual
  // below instead of waiting one after another before each store
  double* const gx = g.x;
  int* const gi = g.iters;
  double* const gr = g.resid;
  const bool has_status = g.status != nullptr;
  int* const gs = has_status ? g.status : g.sink;
  int* const go = g.outer;
  const int flags = g.flags;
  __asm__ volatile("" ::"s"(gx), "s"(gi), "s"(gr), "s"(gs), "s"(go), "s"(flags));
  const bool need = tm.live && !have_rn;
  if (tm.any(need)) {
    double t[RW::R], q[1];
    A.template spmv<0>(tm, A.a, x, t);
    double p[RW::R];
#pragma unroll
    for (int r = 0; r < RW::R; ++r) { const double e = b[r] - t[r]; p[r] = e * e; }
    q[0] = sum_rows(p);
    tm.sum(q);
    if (need) rn = sqrt(q[0]);
  }
  if (!tm.live) return;
#pragma unroll
  for (int r = 0; r < RW::R; ++r)
    if (A.ok[r]) gx[tm.row0 + A.row[r]] = x[r];
  if (tm.lane == 0) {
    gi[tm.sys] = k;
    // the true residual, relative to ||b|| unless the criterion is absolute
    gr[tm.sys] = !finite(bn) ? bn : ((bn == 0.0 || (flags & kFlagAbsTol)) ? rn : rn / bn);
    // always one store (to the sink when no status is wanted): the persistent
    // loop counts on a fixed number of stores after each prefetch
    gs[has_status ? tm.sys : 0] = st;
    if (go) go[tm.sys] = outer;
  }
}

// Shared prologue: load the system, its Jacobi diagonal, b, x0 and the initial
// residual r0 = b - A x0 (r0 = b when x0 = 0 is promised).
template <int R>
struct Prologue {
  double b[R], x[R], r[R], d[R];
};

template <int PK, class TM, class RW>
__device__ __forceinline__ void prologue(TM& tm, RW& A, const KArgs& g, Prologue<RW::R>& P) {
  A.jacobi(g.precond, P.d);
  if constexpr (PK == kPkBlock) bj_setup(tm, A, g);
  if constexpr (PK == kPkIlu) {
    if constexpr (RW::TEAM > kWave) ilu_setup_mw(tm, A, g);
    else ilu_setup(tm, A, g, P.d);
  }
  const bool x0zero = (g.flags & 1) != 0;
#pragma unroll
  for (int r = 0; r < RW::R; ++r) {
    P.b[r] = A.bval[r];
    P.x[r] = A.xval[r];
  }
  if (!x0zero) {
    double t[RW::R];
    A.template spmv<0>(tm, A.a, P.x, t);
#pragma unroll
    for (int r = 0; r < RW::R; ++r) P.r[r] = P.b[r] - t[r];
    if (g.x_alt) {
      // Second candidate start: keep whichever has the smaller residual
      // norm (x on a tie; x_alt also when only x's norm is not a number).
      // The other buffer: lanes may still gather from buffer 0.
      double ta[RW::R], ra[RW::R], p0[RW::R], p1[RW::R];
      A.template spmv<1>(tm, A.a, A.xalt, ta);
#pragma unroll
      for (int r = 0; r < RW::R; ++r) {
        ra[r] = P.b[r] - ta[r];
        p0[r] = P.r[r] * P.r[r];
        p1[r] = ra[r] * ra[r];
      }
      double q[2] = {sum_rows(p0), sum_rows(p1)};
      tm.sum(q);
      const bool alt = q[1] < q[0] || (q[0] != q[0] && q[1] == q[1]);
#pragma unroll
      for (int r = 0; r < RW::R; ++r) {
        P.x[r] = alt ? A.xalt[r] : P.x[r];
        P.r[r] = alt ? ra[r] : P.r[r];
      }
      if (g.alt_used && tm.live && tm.lane == 0) g.alt_used[tm.sys] = alt ? 1 : 0;
    }
  } else {
#pragma unroll
    for (int r = 0; r < RW::R; ++r) P.r[r] = P.b[r];
  }
}

// =================================================================== BiCGSTAB
// Right-preconditioned BiCGSTAB (van der Vorst 1992), the solver the paper
// evaluates on all application inputs (Sec. 4.3).  Per iteration: two SpMVs and
// three fused reductions (r^.v; s.s, t.t, t.s; r.r, r^.r).  The second SpMV is
// issued before the half-step test so that ||s|| joins the t-reduction; it is
// discarded when the half step already converges.
//
// MIXED: the Krylov vectors, the FP32 copy of A and the inner reductions are
// FP32 and solve for a correction to the FP64 x, scaled by 1/||r||; the "true
// residual confirmation" becomes the FP64 outer refinement step r = b - A x,
// which also ends the inner solve when it meets inner_tol or breaks down.
// Vectors of the lean form (see kVarLean), in the lane's LDS cells.
constexpr int kLeanX = 0, kLeanB = 1, kLeanD = 2, kLeanRh = 3, kLeanVectors = 4;

template <bool MIXED, int PK, bool LEAN = false, class TM, class RW>
__device__ __forceinline__ void bicgstab_system(TM& tm, RW& A, const KArgs& g) {
  using T = typename std::conditional<MIXED, float, double>::type;
  Prologue<RW::R> P;
  prologue<PK>(tm, A, g, P);
  constexpr int R = RW::R;
  static_assert(!LEAN || (!MIXED && PK == kPkScalar), "lean: FP64, scalar Jacobi or none");
  constexpr bool kUniform = LEAN || (!MIXED && RW::NZ >= 64 && RW::ROWS > kWave);
  // LEAN: vectors kept in the lane's own LDS cells
  auto keep = [&](int q, const double(&u)[R]) {
    if constexpr (LEAN) {
#pragma unroll
      for (int i = 0; i < R; ++i) lds_store<double>(tm.lean_cell(q, i), u[i]);
    }
  };
  auto kept = [&](int q, double(&u)[R]) {
    if constexpr (LEAN) {
#pragma unroll
      for (int i = 0; i < R; ++i) u[i] = lds_load<double>(tm.lean_cell(q, i));
    }
  };
  // LEAN, and rows of 64 slots on several waves: a team's scalar moved to scalar
  // registers
  auto uni = [&](auto u) {
    if constexpr (kUniform) return wave_uniform(u);
    else return u;
  };

  // FP32 copy of the rows and of the Jacobi diagonal for the inner solve.
  using AT = typename std::conditional<MIXED, float, double>::type;
  AT a_in[R][RW::NZ];
  T d_in[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    d_in[r] = (T)P.d[r];
#pragma unroll
    for (int k = 0; k < RW::NZ; ++k) {
      // slots without an entry of the row may hold other rows' values: zero
      // them so that a value beyond FP32 range cannot meet the zero cell as Inf
      if constexpr (MIXED) a_in[r][k] = A.real(r, k) ? (AT)A.a[r][k] : (AT)0;
      else a_in[r][k] = (AT)A.a[r][k];
    }
  }

  double q2[2];
  {
    double p0[R], p1[R];
#pragma unroll
    for (int r = 0; r < R; ++r) { p0[r] = P.b[r] * P.b[r]; p1[r] = P.r[r] * P.r[r]; }
    q2[0] = sum_rows(p0);
    q2[1] = sum_rows(p1);
    tm.sum(q2);
  }
  const double bn = uni(sqrt(q2[0]));
  double rn = uni(sqrt(q2[1]));  // FP64 norm of the outer (or only) residual
  const double lim = uni(stop_limit(g, bn));
  int st = tm.live ? ST_RUNNING : ST_IDLE;
  bool rtrue = true;
  if (st == ST_RUNNING) {
    if (!finite(bn)) st = ST_NONFINITE;
    else if (bn == 0.0) {
      st = ST_CONVERGED;
#pragma unroll
      for (int r = 0; r < R; ++r) P.x[r] = 0.0;
      rn = 0.0;
    }
  }
  int k = 0, outer = 0;

  // Krylov state.
  T r[R], rh[R], p[R], v[R];
  T rho, rho0, alpha, omega, rr_in;  // rr_in: squared norm of the inner residual
  double scale;  // x += scale * (inner update)
  double rn_prev = rn;
  auto restart = [&](double rtrue_norm) {
    // r_in = r / scale; r^ = r_in; p = v = 0; rho0 = alpha = omega = 1
    scale = MIXED ? rtrue_norm : 1.0;
    const double inv = MIXED ? (rtrue_norm > 0.0 ? 1.0 / rtrue_norm : 0.0) : 1.0;
#pragma unroll
    for (int i = 0; i < R; ++i) {
      r[i] = (T)(MIXED ? P.r[i] * inv : P.r[i]);
      rh[i] = r[i];
      p[i] = 0;
      v[i] = 0;
    }
    rho0 = alpha = omega = (T)1;
  };
  restart(rn);
  keep(kLeanX, P.x);
  keep(kLeanB, P.b);
  keep(kLeanD, P.d);
  if constexpr (LEAN) keep(kLeanRh, rh);
  if constexpr (MIXED) {
    T q[1];
    T pr[R];
#pragma unroll
    for (int i = 0; i < R; ++i) pr[i] = r[i] * r[i];
    q[0] = sum_rows(pr);
    tm.sum(q);
    rho = q[0];
    rr_in = q[0];
  } else {
    rho = (T)q2[1];  // r^ = r, so r^.r is the same sum as r.r
    rr_in = (T)q2[1];
  }
  // Inner stop level: absolute on the same scale as r_in.
  auto inner_lim = [&]() -> T {
    if constexpr (MIXED) {
      const double want = 0.5 * lim / (rn > 0.0 ? rn : 1.0);
      return (T)(want > g.inner_tol ? want : g.inner_tol);
    } else {
      return (T)lim;
    }
  };
  // The recurrence tests compare squared norms (no square root per test);
  // the true-residual confirmation below compares the norm itself.
  T ilim = inner_lim();
  T ilim2 = uni(ilim * ilim);
  bool inner_end = false;  // MIXED: inner solve ended (met inner tol or broke down)

  for (;;) {
    // ---- top: convergence / budget checks, per team
    bool need_chk = false;
    if (st == ST_RUNNING) {
      if (MIXED ? !finite(rn) : !finite((double)rr_in)) {
        st = ST_NONFINITE;
      } else if (MIXED ? (rn <= lim || inner_end || rr_in <= ilim2) : (rr_in <= ilim2)) {
        if (!MIXED && rtrue) st = ST_CONVERGED;
        else if (MIXED && rtrue && rn <= lim) st = ST_CONVERGED;
        else need_chk = true;
      } else if (k >= g.max_iter) {
        st = ST_MAX_ITER;
      }
    }
    bool any_run;
    if (tm.any_first(need_chk, st == ST_RUNNING, any_run)) {
      // ---- true residual (plain) / outer refinement step (mixed), FP64
      double t[R], pr[R], q[1];
      kept(kLeanX, P.x);
      A.template spmv<0>(tm, A.a, P.x, t);
      kept(kLeanB, P.b);
#pragma unroll
      for (int i = 0; i < R; ++i) {
        const double e = P.b[i] - t[i];
        if (need_chk) P.r[i] = e;
        pr[i] = e * e;
      }
      q[0] = sum_rows(pr);
      tm.sum(q);
      if (need_chk) {
        const double rnc = uni(sqrt(q[0]));
        rtrue = true;
        if constexpr (MIXED) outer += 1;
        const bool stagnant = MIXED && !(rnc < rn_prev);
        rn = rnc;
        rn_prev = rnc;
        if (!finite(rnc)) st = ST_NONFINITE;
        else if (rnc <= lim) st = ST_CONVERGED;
        else if (k >= g.max_iter) st = ST_MAX_ITER;
        else if (stagnant) st = ST_BREAKDOWN;
        else {
          restart(rnc);
          if constexpr (LEAN) keep(kLeanRh, rh);
          inner_end = false;
          ilim = inner_lim();
          ilim2 = ilim * ilim;
        }
      }
      if constexpr (MIXED) {
        // new inner residual norm and rho for restarted teams
        T qq[1], pp[R];
#pragma unroll
        for (int i = 0; i < R; ++i) pp[i] = r[i] * r[i];
        qq[0] = sum_rows(pp);
        tm.sum(qq);
        if (need_chk && st == ST_RUNNING) { rho = qq[0]; rr_in = qq[0]; }
      } else {
        if (need_chk && st == ST_RUNNING) { rho = (T)q[0]; rr_in = (T)q[0]; }
      }
      continue;
    }
    if (!tm.any_second(st == ST_RUNNING, any_run)) break;

    // ---- one BiCGSTAB iteration; committed for teams still running
    bool go = st == ST_RUNNING;
    if (go) {
      k += 1;
      if (!finite((double)rho)) {
        if (MIXED) inner_end = true; else st = ST_NONFINITE;
        go = false;
      } else if (rho == (T)0) {
        if (MIXED) inner_end = true; else st = ST_BREAKDOWN;
        go = false;
      }
    }
    const T beta = (rho * alpha) / (rho0 * omega);
    T ph[R], s[R], sh[R], t[R];
    if constexpr (LEAN) kept(kLeanD, d_in);
#pragma unroll
    for (int i = 0; i < R; ++i) p[i] = r[i] + beta * (p[i] - omega * v[i]);
    precond<PK>(tm, A, g, d_in, p, ph);
    A.template spmv<0>(tm, a_in, ph, v);
    T q1[1];
    {
      T pr[R];
      if constexpr (LEAN) kept(kLeanRh, rh);
#pragma unroll
      for (int i = 0; i < R; ++i) pr[i] = rh[i] * v[i];
      q1[0] = sum_rows(pr);
    }
    tm.sum(q1);
    const T sigma = q1[0];
    if (go) {
      if (!finite((double)sigma)) { if (MIXED) inner_end = true; else st = ST_NONFINITE; go = false; }
      else if (sigma == (T)0) { if (MIXED) inner_end = true; else st = ST_BREAKDOWN; go = false; }
    }
    const T al = uni(rho / sigma);
    if constexpr (LEAN) kept(kLeanD, d_in);
#pragma unroll
    for (int i = 0; i < R; ++i) s[i] = r[i] - al * v[i];
    precond<PK>(tm, A, g, d_in, s, sh);
    A.template spmv<1>(tm, a_in, sh, t);
    T q3[3];
    {
      T p0[R], p1[R], p2[R];
#pragma unroll
      for (int i = 0; i < R; ++i) { p0[i] = s[i] * s[i]; p1[i] = t[i] * t[i]; p2[i] = t[i] * s[i]; }
      q3[0] = sum_rows(p0);
      q3[1] = sum_rows(p1);
      q3[2] = sum_rows(p2);
    }
    tm.sum(q3);
    const T ss = q3[0], tt = q3[1], ts = q3[2];
    bool half = false;
    if (go) {
      if (!finite((double)ss)) { if (MIXED) inner_end = true; else st = ST_NONFINITE; go = false; }
      else if (ss <= ilim2) half = true;
      else if (!finite((double)tt) || !finite((double)ts)) {
        if (MIXED) inner_end = true; else st = ST_NONFINITE;
        go = false;
      }
    }
    const double sal = scale * (double)al;
    if constexpr (LEAN) {
      // z = M p and M s are formed again rather than held through the products
      kept(kLeanD, d_in);
#pragma unroll
      for (int i = 0; i < R; ++i) {
        __asm__ volatile("" : "+v"(p[i]), "+v"(s[i]));
        ph[i] = d_in[i] * p[i];
        sh[i] = d_in[i] * s[i];
      }
      if (half || go) kept(kLeanX, P.x);
    }
    if (half) {
#pragma unroll
      for (int i = 0; i < R; ++i) {
        P.x[i] = fma(sal, (double)ph[i], P.x[i]);
        r[i] = s[i];
      }
      keep(kLeanX, P.x);
      rtrue = false;
      rr_in = ss;
      go = false;
    }
    const T om = uni((tt == (T)0) ? (T)0 : ts / tt);
    if (go) {
      const double som = scale * (double)om;
#pragma unroll
      for (int i = 0; i < R; ++i) {
        P.x[i] = fma(som, (double)sh[i], fma(sal, (double)ph[i], P.x[i]));
        r[i] = s[i] - om * t[i];
      }
      keep(kLeanX, P.x);
      rtrue = false;
      rho0 = rho;
      alpha = al;
      omega = om;
    }
    T q4[2];
    {
      T p0[R], p1[R];
      if constexpr (LEAN) kept(kLeanRh, rh);
#pragma unroll
      for (int i = 0; i < R; ++i) { p0[i] = r[i] * r[i]; p1[i] = rh[i] * r[i]; }
      q4[0] = sum_rows(p0);
      q4[1] = sum_rows(p1);
    }
    tm.sum(q4);
    if (go) {
      rr_in = q4[0];
      rho = q4[1];
      if (om == (T)0 && !(rr_in <= ilim2)) {
        if (MIXED) inner_end = true; else st = ST_BREAKDOWN;
      }
    }
  }
  kept(kLeanX, P.x);
  kept(kLeanB, P.b);
  finish(tm, A, g, P.b, P.x, st, k, outer, bn, rn, st == ST_CONVERGED || st == ST_IDLE);
}

// =================================================================== Trsv
// BatchTrsv (Tab. 2): T x = b for T the lower (upper) triangle of A, diagonal
// included, one-wave teams (row i on lane i, n <= 64).  The row's register
// values outside the triangle are zeroed, so the shared epilogue's true
// residual is that of T; the triangle goes to the LDS region, packed by rows
// (entry (i,j) of the lower one at i(i+1)/2 + j, of the upper one at i n -
// i(i-1)/2 + j - i: half the square's LDS, twice the resident waves, and the
// rows of a wave still start in distinct banks), and one column sweep solves
// it: x_k = acc_k / t_kk (final on lane k when column k is reached) is read
// out, and every later row subtracts t_ik x_k.  A sweep reads a lane's row at
// every column; what lies there outside the triangle belongs to other rows,
// and the lanes that would meet it take no term.  The columns past n, which an
// upper sweep reaches first with every row, are cut to zero: the x there is
// zero too, but another row's infinite diagonal (a row whose x is zero, and no
// error) would make its product no number.  A zero diagonal entry is a
// breakdown (x = 0); iterations: 0.
template <bool LOWER, class TM, class RW>
__device__ __forceinline__ void trsv_system_w64(TM& tm, RW& A, const KArgs& g) {
  static_assert(RW::R == 1 && RW::TEAM == kWave, "one-wave BatchTrsv");
  const int n = g.n;
  const unsigned F = lds_addr(tm.bj_region(g));
  const int lane = tm.lane;
  const bool ok = A.ok[0];
  const int i = ok ? A.row[0] : 0;
  // byte address of column 0 of this lane's row
  const unsigned fi = F + (unsigned)(LOWER ? i * (i + 1) / 2 : i * n - i * (i - 1) / 2 - i) * 8;
  for (unsigned e = 16u * (unsigned)lane; e < (unsigned)trsv_bytes(n); e += 16u * kWave)
    lds_store<uint4v>(F + e, uint4v{0, 0, 0, 0});
  wave_lds_fence();
  // slot s holds column (c - b0) / 8 (the zero cell, past all of them, when
  // empty); entries outside the triangle go to the lane's own cell of buffer
  // 0.  (vrow is opaque per system: the slots' masks would otherwise be formed
  // once per kernel and spill.)
  unsigned own = A.vrow[0];
  __asm__ volatile("" : "+v"(own));
#pragma unroll
  for (int s = 0; s < RW::NZ; ++s) {
    const bool keep = LOWER ? A.c[0][s] <= own : A.c[0][s] - own < A.zc - own;
    lds_store<double>(keep ? A.c[0][s] - A.b0 + fi : own, A.a[0][s]);
    A.a[0][s] = keep ? A.a[0][s] : 0.0;
  }
  wave_lds_fence();
  double b[1] = {A.bval[0]}, x[1] = {A.xval[0]}, q[1] = {b[0] * b[0]};
  tm.sum(q);
  const double bn = sqrt(q[0]);
  const double tii = ok ? lds_load<double>(fi + i * 8) : 1.0;
  int stt = tm.live ? ST_CONVERGED : ST_IDLE;
  if (tm.live && !finite(bn)) {
    stt = ST_NONFINITE;
  } else if (bn == 0.0 || wave_any(tm.live && tii == 0.0)) {
    if (tm.live && bn != 0.0) stt = ST_BREAKDOWN;
    x[0] = 0.0;
  } else {
    const double dv = ok ? 1.0 / tii : 0.0;
    const uint64_t rows = ~0ull >> (kWave - n);  // idle lanes take no term
    double acc = ok ? b[0] : 0.0;
    sweep_columns<LOWER, 4, !LOWER>(
        fi, (n + 3) & ~3,
        [&](int k, double f) {
          const double xk = rdlane(acc * dv, k);
          if (__builtin_amdgcn_inverse_ballot_w64((LOWER ? lanes_past(k) : ~(~0ull << k)) & rows))
            acc = fma(-f, xk, acc);
        },
        n);
    x[0] = ok ? acc * dv : 0.0;
    if (tm.live && wave_any(ok && !finite(x[0]))) stt = ST_NONFINITE;
  }
  wave_lds_fence();
  finish(tm, A, g, b, x, stt, 0, 0, bn, 0.0, false);
}

// BatchTrsv for multi-wave teams (row i on lane i, up to 1024 rows): the
// row-oriented substitution of the oracle on the team's first wave, level by
// level (the sweep of the ILU(0) form with the triangle's own diagonal):
// x_i = (b_i - sum_j t_ij x_j) / t_ii over the row's strictly lower (upper)
// entries in increasing column.  Entries outside the triangle are zeroed in
// registers as in the one-wave form, so the epilogue's residual is that of
// the triangle; a zero diagonal entry anywhere is a breakdown.
template <bool LOWER, class TM, class RW>
__device__ __forceinline__ void trsv_system_mw(TM& tm, RW& A, const KArgs& g) {
  static_assert(RW::R == 1 && RW::TEAM > kWave, "multi-wave BatchTrsv: one row per lane");
  constexpr int NZ = RW::NZ;
  const IluMw L = ilu_mw_layout(g.n, g.nnz);
  const unsigned reg = lds_addr(tm.bj_region(g));
  const unsigned F = reg + L.f, D = F + g.noff * 8, RE = reg + L.re, V = reg + L.v;
  tri_cells(tm, g, reg, L);
  const bool ok = A.ok[0];
  int i = ok ? A.row[0] : 0;
  __asm__ volatile("" : "+v"(i));  // per system: keeps the row's addresses out of the kernel-wide registers
  const int e0 = g.fmt == 0 ? A.w[0] : g.row_ptr[i];  // CSR position of register slot 0
  const int place = g.tri_place[i];
  const unsigned me = (unsigned)(LOWER ? place & 0xffff : place >> 16) * 8;
  const double tii = ok ? A.dval[0] : 1.0;
  if (ok) {
    // the triangle's entries off the diagonal; the diagonal in the sweep's order
#pragma unroll
    for (int s = 0; s < NZ; ++s)
      if (A.real(0, s) && s != A.dslot[0]) lds_store<double>(F + g.tri_pos[e0 + s] * 8, A.a[0][s]);
    lds_store<double>(D + me, tii);
    store_reciprocal(RE + me * 2, tii);
    lds_store<double>(V + me, A.bval[0]);
  }
#pragma unroll
  for (int s = 0; s < NZ; ++s) {
    const bool keep = ok && A.real(0, s) && (LOWER ? A.c[0][s] <= A.vrow[0] : A.c[0][s] >= A.vrow[0]);
    A.a[0][s] = keep ? A.a[0][s] : 0.0;
  }
  double b[1] = {A.bval[0]}, x[1] = {A.xval[0]}, q[1] = {b[0] * b[0]};
  tm.sum(q);  // also makes the stores above visible to the team
  const double bn = sqrt(q[0]);
  const bool zero_diag = __syncthreads_or(ok && tii == 0.0) != 0;
  const bool wide = __syncthreads_or(!quotient_safe(0.0, tii)) != 0;
  int stt = tm.live ? ST_CONVERGED : ST_IDLE;
  if (tm.live && !finite(bn)) {
    stt = ST_NONFINITE;
  } else if (bn == 0.0 || zero_diag) {
    if (tm.live && bn != 0.0) stt = ST_BREAKDOWN;
    x[0] = 0.0;
  } else {
    x[0] = divided_sweep<true>(tm, g, L, reg, LOWER, ok, me, wide);
    const bool nf = __syncthreads_or(ok && !finite(x[0])) != 0;
    if (tm.live && nf) stt = ST_NONFINITE;
  }
  finish(tm, A, g, b, x, stt, 0, 0, bn, 0.0, false);
}

template <bool LOWER, class TM, class RW>
__device__ __forceinline__ void trsv_system(TM& tm, RW& A, const KArgs& g) {
  if constexpr (RW::TEAM > kWave) trsv_system_mw<LOWER>(tm, A, g);
  else trsv_system_w64<LOWER>(tm, A, g);
}

// =================================================================== CG
// Preconditioned CG, Sec. 3.5 Alg. 1 step for step, with the relative-residual
// stop test.  Per iteration: one SpMV and two reductions (p.t; r.z, r.r).
template <int PK, class TM, class RW>
__device__ __forceinline__ void cg_system(TM& tm, RW& A, const KArgs& g) {
  Prologue<RW::R> P;
  prologue<PK>(tm, A, g, P);
  constexpr int R = RW::R;
  double z[R], p[R];
  precond<PK>(tm, A, g, P.d, P.r, z);
#pragma unroll
  for (int i = 0; i < R; ++i) p[i] = z[i];
  double q3[3];
  {
    double p0[R], p1[R], p2[R];
#pragma unroll
    for (int i = 0; i < R; ++i) { p0[i] = P.b[i] * P.b[i]; p1[i] = P.r[i] * P.r[i]; p2[i] = P.r[i] * z[i]; }
    q3[0] = sum_rows(p0); q3[1] = sum_rows(p1); q3[2] = sum_rows(p2);
  }
  tm.sum(q3);
  const double bn = sqrt(q3[0]);
  double rn = sqrt(q3[1]), rho = q3[2];
  double rsq = q3[1];  // squared recurrence residual (the loop compares squares)
  const double lim = stop_limit(g, bn), lim2 = lim * lim;
  int st = tm.live ? ST_RUNNING : ST_IDLE;
  if (st == ST_RUNNING) {
    if (!finite(bn)) st = ST_NONFINITE;
    else if (bn == 0.0) {
      st = ST_CONVERGED;
#pragma unroll
      for (int i = 0; i < R; ++i) P.x[i] = 0.0;
      rn = 0.0;
    }
  }
  bool rtrue = true;
  int k = 0;
  for (;;) {
    bool need_chk = false;
    if (st == ST_RUNNING) {
      if (!finite(rsq) || !finite(rho)) st = ST_NONFINITE;
      else if (rsq <= lim2) { if (rtrue) st = ST_CONVERGED; else need_chk = true; }
      else if (k >= g.max_iter) st = ST_MAX_ITER;
    }
    bool any_run;
    if (tm.any_first(need_chk, st == ST_RUNNING, any_run)) {
      double t[R], rc[R], zc[R], p0[R], p1[R], q[2];
      A.template spmv<0>(tm, A.a, P.x, t);
#pragma unroll
      for (int i = 0; i < R; ++i) rc[i] = P.b[i] - t[i];
      precond<PK>(tm, A, g, P.d, rc, zc);
#pragma unroll
      for (int i = 0; i < R; ++i) {
        p0[i] = rc[i] * rc[i];
        p1[i] = rc[i] * zc[i];
      }
      q[0] = sum_rows(p0); q[1] = sum_rows(p1);
      tm.sum(q);
      if (need_chk) {
        rn = sqrt(q[0]);
        rsq = q[0];
        rtrue = true;
        if (!finite(rn)) st = ST_NONFINITE;
        else if (rn <= lim) st = ST_CONVERGED;
        else if (k >= g.max_iter) st = ST_MAX_ITER;
        else {
#pragma unroll
          for (int i = 0; i < R; ++i) { P.r[i] = rc[i]; z[i] = zc[i]; p[i] = zc[i]; }
          rho = q[1];
        }
      }
      continue;
    }
    if (!tm.any_second(st == ST_RUNNING, any_run)) break;
    bool go = st == ST_RUNNING;
    if (go && rho == 0.0) { st = ST_BREAKDOWN; go = false; }
    double t[R];
    A.template spmv<0>(tm, A.a, p, t);
    double q1[1];
    {
      double pr[R];
#pragma unroll
      for (int i = 0; i < R; ++i) pr[i] = p[i] * t[i];
      q1[0] = sum_rows(pr);
    }
    tm.sum(q1);
    const double pt = q1[0];
    if (go) {
      if (!finite(pt)) { st = ST_NONFINITE; go = false; }
      else if (pt == 0.0) { st = ST_BREAKDOWN; go = false; }
    }
    const double alpha = rho / pt;
    double rr[R];
#pragma unroll
    for (int i = 0; i < R; ++i) {
      rr[i] = go ? fma(-alpha, t[i], P.r[i]) : P.r[i];
      if (go) P.x[i] = fma(alpha, p[i], P.x[i]);
    }
    precond<PK>(tm, A, g, P.d, rr, z);
    double q2[2];
    {
      double p0[R], p1[R];
#pragma unroll
      for (int i = 0; i < R; ++i) { p0[i] = rr[i] * z[i]; p1[i] = rr[i] * rr[i]; }
      q2[0] = sum_rows(p0); q2[1] = sum_rows(p1);
    }
    tm.sum(q2);
    if (go) {
      const double beta = q2[0] / rho;
#pragma unroll
      for (int i = 0; i < R; ++i) { P.r[i] = rr[i]; p[i] = fma(beta, p[i], z[i]); }
      rho = q2[0];
      rsq = q2[1];
      rtrue = false;
      k += 1;
    }
  }
  finish(tm, A, g, P.b, P.x, st, k, 0, bn, rn, st == ST_CONVERGED || st == ST_IDLE);
}

// =================================================================== GMRES(m)
// Right-preconditioned restarted GMRES with Gram-Schmidt Arnoldi and Givens
// rotations (Saad 2003, Alg. 6.9 with right preconditioning): modified
// Gram-Schmidt for teams narrower than a wave, block modified Gram-Schmidt
// (blocks of four, classical inside a block) for teams of a wave or more, whose
// reductions then fuse four dots at a time.  The m+1
// basis vectors stay on chip (one element per row per lane, in registers, or
// partly in LDS for 1024-lane teams), so a cycle never touches HBM.  The Hessenberg column, the rotated triangle R, the
// rotations, g and y are per-team LDS scalars written once per cycle: every lane
// of the team computes the same bits and writes them, and reads only entries it
// has written itself, so no barrier is needed around them.  The last entry of g
// changes at every step and is kept in a register.  At the end of a cycle
// y = R^{-1} g by back substitution and x += M V y.
//
// MIXED: every cycle is an iterative-refinement step.  The cycle start forms
// the FP64 true residual r = b - A x (as the plain method does at a restart);
// the cycle's Arnoldi steps run in FP32 (basis, SpMV with an FP32 copy of A,
// dots and norms), ending when |g| <= max(inner_tol * beta, tol ||b|| / 2) or
// after m steps; the rotations and the triangular solve stay FP64 and x is
// updated in FP64.  A cycle that does not lower the FP64 residual ends the
// solve with BREAKDOWN.
// Where a team keeps the GMRES scalars (Hessenberg column, packed R, the
// rotations, g, y) and its LDS basis vectors: behind the fixed-size team's
// vector buffers.  Teams of other kernels provide their own overloads.
template <class S>
__device__ __forceinline__ double* gmres_scalar_base(const Team<S>& tm, int rows) {
  return reinterpret_cast<double*>(tm.lds + kVecBuffers * vec_buf_bytes(rows));
}
template <class S>
__device__ __forceinline__ unsigned gmres_basis_base(const Team<S>& tm, int rows) {
  return lds_addr(tm.lds) + gmres_basis_offset(rows);
}

template <bool MIXED, int PK, class TM, class RW>
__device__ __forceinline__ void gmres_system(TM& tm, RW& A, const KArgs& g) {
  static_assert(RW::R == 1, "GMRES keeps one row per lane");
  using T = typename std::conditional<MIXED, float, double>::type;
  constexpr int M = kMaxRestart;
  Prologue<RW::R> P;
  prologue<PK>(tm, A, g, P);
  const int m = g.restart;
  // LDS scalars of this team
  double* hcol = gmres_scalar_base(tm, RW::ROWS);
  double* Rt = hcol + (M + 2);               // packed by columns: R[i][j] at j(j+1)/2 + i
  double* cs = Rt + M * (M + 1) / 2;
  double* sn = cs + M;
  double* gv = sn + M;
  double* yv = gv + (M + 1);

  // the arithmetic copy of the rows (FP32 for MIXED; slots without an entry
  // zeroed so that no value beyond FP32 range meets the zero cell)
  T a_in[1][RW::NZ];
#pragma unroll
  for (int k = 0; k < RW::NZ; ++k) {
    if constexpr (MIXED) a_in[0][k] = A.real(0, k) ? (T)A.a[0][k] : (T)0;
    else a_in[0][k] = A.a[0][k];
  }

  double q1[1];
  {
    double pr[1] = {P.b[0] * P.b[0]};
    q1[0] = pr[0];
  }
  tm.sum(q1);
  const double bn = sqrt(q1[0]);
  const double lim = stop_limit(g, bn);
  int st = tm.live ? ST_RUNNING : ST_IDLE;
  double rn = 0.0;
  if (st == ST_RUNNING) {
    if (!finite(bn)) st = ST_NONFINITE;
    else if (bn == 0.0) { st = ST_CONVERGED; P.x[0] = 0.0; }
  }
  // Basis vectors 0..NL-1 live in LDS (this lane's element of vector i at
  // vb + i * ROWS * sizeof(T)), vectors NL..M in registers V[i - NL].
  constexpr int NL = gmres_lds_vectors(RW::WG, MIXED);
  constexpr int NV = M + 1 - NL;
  T V[NV > 0 ? NV : 1];
  const unsigned vb = gmres_basis_base(tm, RW::ROWS) + (unsigned)tm.lane * sizeof(T);
  constexpr unsigned vstride = RW::ROWS * sizeof(T);
#pragma unroll
  for (int i = 0; i < NV; ++i) V[i] = (T)0;
#pragma unroll
  for (int i = 0; i < NL; ++i) lds_store<T>(vb + i * vstride, (T)0);
  // basis element i of this lane (i is a compile-time index after unrolling)
  auto basis = [&](int i) -> T {
    return i < NL ? lds_load<T>(vb + i * vstride) : V[i >= NL ? i - NL : 0];
  };

  int k = 0, j = 0, cycles = 0;
  T vcur = (T)0;       // the basis vector the next Arnoldi step multiplies
  double gcur = 0.0;   // g_j, the entry the next rotation acts on
  double ilim = lim;   // the cycle's stopping level for |g|
  double beta_prev = INFINITY;
  bool start = true;   // at a cycle start (true residual due)
  const double d = P.d[0];
  const T dT = (T)d;
  for (;;) {
    // ---- cycle start: true residual, convergence, V0 = r/beta
    if (tm.any(st == ST_RUNNING && start)) {
      const bool me = st == ST_RUNNING && start;
      double t[1];
      A.template spmv<0, false>(tm, A.a, P.x, t);
      const double rc = P.b[0] - t[0];
      double q[1] = {rc * rc};
      tm.sum(q);
      if (me) {
        const double beta = sqrt(q[0]);
        rn = beta;
        if (!finite(beta)) st = ST_NONFINITE;
        else if (beta <= lim) st = ST_CONVERGED;
        else if (k >= g.max_iter) st = ST_MAX_ITER;
        else if (MIXED && !(beta < beta_prev)) st = ST_BREAKDOWN;
        else {
          vcur = (T)(rc / beta);
          if constexpr (NL > 0) lds_store<T>(vb, vcur);
          else V[0] = vcur;
          gcur = beta;
          if constexpr (MIXED) ilim = fmax(g.inner_tol * beta, 0.5 * lim);
          beta_prev = beta;
          cycles += 1;
          j = 0;
          start = false;
        }
      }
    }
    if (!tm.any(st == ST_RUNNING)) break;
    // ---- one Arnoldi step for every running team (all of them are mid-cycle)
    const bool act = st == ST_RUNNING;
    T z[1], w[1];
    {
      const T vv[1] = {vcur}, dd[1] = {dT};
      precond<PK>(tm, A, g, dd, vv, z);
    }
    A.template spmv<0, false>(tm, a_in, z, w);
    const int jmax = wave_max(act ? j : -1);
    if constexpr (RW::TEAM >= 64) {
      // Block Gram-Schmidt: blocks of four basis vectors taken in order, as
      // modified Gram-Schmidt takes single vectors; within a block the four
      // dots use the same w (classical Gram-Schmidt) and share one fused
      // reduction, then w -= V_block q.
      [[maybe_unused]] double* const hq =
          hcol + ((lane_id() >> 5) | ((lane_id() >> 3) & 2));  // rows 0..3: values 0, 2, 1, 3
#pragma unroll
      for (int g = 0; g < M; g += 4) {
        if (g <= jmax) {
          // the last block may reach past vector j: what those hold (earlier
          // cycles' vectors) gives sums that nothing uses
          T vq[4], q[4];
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            vq[t] = g + t < M ? basis(g + t) : (T)0;
            q[t] = w[0] * vq[t];
          }
          if constexpr (RW::WG == kWave) {
            // each row of the wave stores its value (entries past j unused)
            const T own = wave_sums_rows(q);
            if (act) hq[g] = (double)own;
          } else {
            tm.sum(q);
          }
          if (act) {
            if (g + 3 < M && g + 3 <= j) {
#pragma unroll
              for (int t = 0; t < 4; ++t) {
                w[0] = fma(-q[t], vq[t], w[0]);
                if constexpr (RW::WG != kWave) hcol[g + t] = (double)q[t];
              }
            } else {
#pragma unroll
              for (int t = 0; t < 3; ++t) {
                if (g + t < M && g + t <= j) {
                  w[0] = fma(-q[t], vq[t], w[0]);
                  if constexpr (RW::WG != kWave) hcol[g + t] = (double)q[t];
                }
              }
            }
          }
        }
      }
    } else {
#pragma unroll
      for (int i = 0; i < M; ++i) {
        if (i <= jmax) {
          const T vi = basis(i);
          T q[1] = {w[0] * vi};
          tm.sum(q);
          if (act && i <= j) {
            w[0] = fma(-q[0], vi, w[0]);
            hcol[i] = (double)q[0];
          }
        }
      }
    }
    T qn[1] = {w[0] * w[0]};
    tm.sum(qn);
    bool end = false;
    if (act) {
      const double hn = sqrt((double)qn[0]);
      k += 1;
      if (!finite(hn)) {
        st = ST_NONFINITE;
      } else {
        // apply the previous rotations to column j
        double hp;
        const int cj = j * (j + 1) / 2;
        if constexpr (RW::TEAM >= 64 && RW::TEAM <= 512) {
          // The chain hp_{i+1} = c_i h_{i+1} - s_i hp_i takes its operands from
          // LDS at one address for all lanes, a group of G steps ahead, and
          // leaves the hp_i there; lane i then forms R_ij from hp_i.  (One entry
          // per lane and six v_readlane per step made this loop 14 vector
          // instructions and 46 cycles a step before any arithmetic: with the
          // other changes to a step, 16384 stiff systems of 54 rows took 2.40 ms,
          // now 1.84.)  Groups of four take 48 registers: one-wave shapes afford
          // them, their LDS holds them to two or three waves per SIMD as it is
          // (8928 of 60 rows, 28 entries each: 349 us, 378 in groups of two).  Teams
          // of several waves would lose a resident wave or two to them (3906 systems
          // of 120 rows, 32 entries each: 640 us, 438 in groups of two, 494 with the
          // readlane form), and the 4-slot shapes one to groups of two as well
          // (10000 of 500 rows, 3 each, block Jacobi on 512 lanes: 25 ms, 19 with
          // single steps, 23 with the readlane form).
          const int ju = __builtin_amdgcn_readfirstlane(j);
          constexpr int G = RW::WG == kWave ? 4 : RW::NZ <= 4 ? 1 : 2;
          hp = hcol[0];
          double c4[G], s4[G], h4[G];
#pragma unroll
          for (int u = 0; u < G; ++u) { c4[u] = cs[u]; s4[u] = sn[u]; h4[u] = hcol[u + 1]; }
          for (int i = 0; i < ju; i += G) {
            const int nx = i + G < M ? i + G : 0;  // the group after the last is not used
#pragma unroll
            for (int u = 0; u < G; ++u) {
              if (i + u < ju) {
                yv[i + u] = hp;
                hp = fma(h4[u], c4[u], -(hp * s4[u]));
              }
              c4[u] = cs[nx + u];
              s4[u] = sn[nx + u];
              h4[u] = hcol[nx + u + 1];
            }
          }
          const int l = (int)lane_id();
          if (l < ju) Rt[cj + l] = fma(cs[l], yv[l], sn[l] * hcol[l + 1]);
        } else if constexpr (RW::TEAM > 512) {
          // 16 waves would each read the chain's operands from the LDS they
          // share (700 systems of 992 rows: 1.93 ms): column j and the rotations
          // are loaded one entry per lane and read with readlane (1.18 ms)
          const int ju = __builtin_amdgcn_readfirstlane(j);
          const int l = (int)lane_id();
          const double hreg = l <= ju ? hcol[l] : 0.0;
          const double creg = l < ju ? cs[l] : 0.0, sreg = l < ju ? sn[l] : 0.0;
          hp = rdlane(hreg, 0);
          for (int i = 0; i < ju; ++i) {
            const double hnx = rdlane(hreg, i + 1), c = rdlane(creg, i), s = rdlane(sreg, i);
            Rt[cj + i] = c * hp + s * hnx;
            hp = -s * hp + c * hnx;
          }
        } else {
          hp = hcol[0];
          for (int i = 0; i < j; ++i) {
            const double hnx = hcol[i + 1];
            const double c = cs[i], s = sn[i];
            Rt[cj + i] = c * hp + s * hnx;
            hp = -s * hp + c * hnx;
          }
        }
        const double dd = sqrt(hp * hp + hn * hn);
        if (dd == 0.0) {
          st = ST_BREAKDOWN;
        } else {
          const double c = hp / dd, s = hn / dd;
          cs[j] = c;
          sn[j] = s;
          Rt[cj + j] = dd;
          gv[j] = c * gcur;
          gcur = -s * gcur;
          end = fabs(gcur) <= ilim || hn == 0.0 || k >= g.max_iter || j == m - 1;
          if (!end) {
            const T vn = (T)((double)w[0] / hn);
            vcur = vn;
            if constexpr (NL > 0) {
              if (j + 1 < NL) lds_store<T>(vb + (unsigned)(j + 1) * vstride, vn);
            }
            // teams of a wave or more: j is the same in every lane
            const int jn = RW::TEAM >= 64 ? __builtin_amdgcn_readfirstlane(j + 1) : j + 1;
            // by groups of four, each behind a scalar branch
#pragma unroll
            for (int i = (NL > 1 ? NL : 1) & ~3; i <= M; i += 4) {
              if (RW::TEAM < 64 || (jn >> 2) == (i >> 2)) {
#pragma unroll
                for (int u = 0; u < 4; ++u)
                  if (i + u >= (NL > 1 ? NL : 1) && i + u <= M && jn == i + u) V[i + u - NL < NV ? i + u - NL : 0] = vn;
              }
            }
            j += 1;
          }
        }
      }
    }
    // ---- cycle end: y = R^{-1} g (back substitution), x += M V y
    if (tm.any(end)) {
      const int jend = wave_max(end ? j : -1);
      double zacc = 0.0;
      if constexpr (RW::TEAM >= 64) {
        // column by column: lane l keeps g_l minus the known terms of row l;
        // y_i = (that of lane i) / R_ii, then the rows above drop R_li y_i
        if (end) {
          const int je = __builtin_amdgcn_readfirstlane(j);
          const int l = (int)lane_id();
          double acc = l <= je ? gv[l] : 0.0;
#pragma unroll
          for (int i = M - 1; i >= 0; --i) {
            if (i <= je) {
              const double yi = rdlane(acc, i) / Rt[i * (i + 1) / 2 + i];
              if (l < i) acc = fma(-Rt[i * (i + 1) / 2 + l], yi, acc);
              zacc = fma(yi, (double)basis(i), zacc);
            }
          }
        }
      } else {
#pragma unroll
        for (int i = M - 1; i >= 0; --i) {
          if (i <= jend) {
            if (end && i <= j) {
              double acc = gv[i];
              for (int l = i + 1; l <= j; ++l) acc = fma(-Rt[l * (l + 1) / 2 + i], yv[l], acc);
              const double yi = acc / Rt[i * (i + 1) / 2 + i];
              yv[i] = yi;
              zacc = fma(yi, (double)basis(i), zacc);
            }
          }
        }
      }
      // x += M V y (every lane of the wave applies M together)
      double mz[1];
      {
        const double zz[1] = {zacc}, dd[1] = {d};
        precond<PK>(tm, A, g, dd, zz, mz);
      }
      if (end) {
        if constexpr (PK != kPkScalar) P.x[0] = P.x[0] + mz[0];
        else P.x[0] = fma(d, zacc, P.x[0]);
        start = true;
      }
    }
  }
  finish(tm, A, g, P.b, P.x, st, k, MIXED ? cycles : 0, bn, rn,
         st == ST_CONVERGED || st == ST_IDLE || (st == ST_MAX_ITER && start) ||
             (MIXED && st == ST_BREAKDOWN && start));
}

// =================================================================== kernels
// Each workgroup loads the shared pattern into registers once and then walks
// over the batch: in every round the G workgroups take G consecutive slots of
// T systems (T teams each), workgroup b the slot xcd_slot(b) of the round,
// team t the system slot * T + t.  Single-wave groups prefetch the next
// round's systems into LDS while the current round is solved: wait for the
// prefetch, copy the block into registers, wait for those LDS reads, start the
// next prefetch, solve.
// Vector memory operations retire in issue order.  After the first round the
// last ones a wave issued are the previous system's four output stores (x,
// iters, resid, status), all after this round's prefetch: waiting until at most
// four are outstanding (and for LDS) means the prefetch has landed, without
// waiting for the stores to be acknowledged.  s_waitcnt vmcnt(4) expcnt(7)
// lgkmcnt(0).
constexpr int kWaitPrefetch = 0x0074;
// Multi-wave teams wait for all of their vector memory operations (their
// waves issue different numbers of output stores after the prefetch):
// s_waitcnt vmcnt(0) expcnt(7) lgkmcnt(15).
constexpr int kWaitAllVm = 0x0F70;

// Workgroups are placed on the 8 XCDs round-robin (workgroup b on XCD b mod 8),
// and each XCD has its own L2.  Slot of workgroup b in a round of the grid:
// XCD x takes the contiguous slots x*G/8 .. (x+1)*G/8-1, so
// neighbouring systems (whose values, right-hand sides and outputs share cache
// lines at their edges) are handled inside one XCD and their partial lines
// merge in one L2.  Identity when G is not a multiple of 8.
__device__ __forceinline__ unsigned xcd_slot(unsigned b, unsigned G) {
  return (G & 7u) ? b : (b & 7u) * (G >> 3) + (b >> 3);
}

// The loop body reads the arguments through ga, at an address offset by a
// zero the compiler cannot see through: otherwise it hoists every argument
// load out of the loop and keeps them all in scalar registers through the
// solve, where they spill into vector-register lanes.
#define BS_PERSISTENT_LOOP(MX, PF, CALL)                                            \
  extern __shared__ __align__(16) char smem[];                                     \
  Team<S> tm(smem, g);                                                             \
  Rows<S, MX> A;                                                                   \
  A.load_pattern(tm, g);                                                           \
  const int64_t stride = (int64_t)gridDim.x * S::TEAMS;                            \
  const int64_t slot0 = (int64_t)xcd_slot(blockIdx.x, gridDim.x) * S::TEAMS;      \
  bool staged = false;                                                             \
  [[maybe_unused]] RegBlock<(PF)> pf;                                              \
  if constexpr ((PF) > 0) {                                                        \
    if (g.stage == 3 && slot0 < g.n_batch) A.prefetch_regs(tm, g, slot0, pf);      \
  } else if constexpr (S::WAVES == 1) {                                            \
    staged = g.stage == 1;                                                         \
    if (staged) A.prefetch(tm, g, slot0);                                          \
  } else if constexpr (S::NZ >= kStageMinSlots) {                                  \
    staged = g.stage == 2;                                                         \
    if (staged && slot0 < g.n_batch) A.prefetch_group(tm, g, slot0);               \
  }                                                                                \
  bool first_round = true;                                                         \
  for (int64_t base = slot0; base < g.n_batch; base += stride) {                   \
    int opaque_zero;                                                               \
    __asm__ volatile("s_mov_b32 %0, 0" : "=s"(opaque_zero));                       \
    const KArgs& ga = (&g)[opaque_zero];                                           \
    tm.sys = base + tm.tix;                                                        \
    tm.live = tm.sys < ga.n_batch;                                                 \
    tm.row0 = tm.live ? tm.sys * ga.n : 0;                                         \
    if constexpr ((PF) > 0) {                                                      \
      if (ga.stage == 3) A.put_regs(tm, ga, pf);                                   \
    } else if constexpr (S::WAVES == 1) {                                          \
      if (staged) { /* the prefetch of this round has landed */                    \
        if (first_round) __builtin_amdgcn_s_waitcnt(0);                            \
        else __builtin_amdgcn_s_waitcnt(kWaitPrefetch);                            \
        first_round = false;                                                       \
        __asm__ volatile("" ::: "memory");                                         \
      }                                                                            \
    } else {                                                                       \
      if (staged) { /* every wave's part of the prefetch has landed */             \
        __builtin_amdgcn_s_waitcnt(kWaitAllVm);                                    \
        __asm__ volatile("" ::: "memory");                                         \
        __syncthreads();                                                           \
      }                                                                            \
    }                                                                              \
    A.load_values(tm, ga);                                                         \
    if constexpr ((PF) > 0) {                                                      \
      if (ga.stage == 3 && base + stride < ga.n_batch)                             \
        A.prefetch_regs(tm, ga, base + stride, pf);                                \
    } else if constexpr (S::WAVES == 1) {                                          \
      if (staged && base + stride < ga.n_batch) {                                  \
        __builtin_amdgcn_s_waitcnt(0xC07F); /* staging reads done (lgkmcnt 0) */   \
        __asm__ volatile("" ::: "memory");                                         \
        A.prefetch(tm, ga, base + stride);                                         \
      }                                                                            \
    } else if constexpr (S::NZ >= kStageMinSlots) {                                \
      if (staged && base + stride < ga.n_batch) {                                  \
        __syncthreads(); /* every wave has read its rows from the block */         \
        A.prefetch_group(tm, ga, base + stride);                                   \
      }                                                                            \
    }                                                                              \
    CALL;                                                                          \
  }

// Mixed kernels keep their FP32 vectors at a 4-byte LDS stride when a team
// holds more rows than a wave: the gathers of the large systems then meet
// fewer bank conflicts (the 992-row stencil solves 8% faster), while the
// one-wave systems (54 rows) lose more to the extra address arithmetic of the
// FP64 residual SpMVs than they gain.
template <class S, bool MIXED>
constexpr bool kLds32 = MIXED && (S::ROWS > kWave);

// One-wave ILU(0) and BatchTrsv: KiB of the next system's values kept in
// registers through a solve (65536 triangular solves of 54 rows: 0.41 ms with
// every lane reading its row from memory and a square triangle in LDS, 0.21 ms
// with this and the packed one).  Their LDS goes to more resident waves instead of
// a staging area, and a lane that reads its own row from memory touches a
// line of its own with every load.
template <class S, bool TRSV>
constexpr int kRegBlock = S::TEAM == kWave && S::R == 1 ? pf_chunks(S::NZ, TRSV) : 0;

// ILU(0) on one-wave teams: the dense factors (about 25 KB of LDS per wave
// for 54 rows) leave room for fewer than two waves per SIMD, so the register
// budget is that of two (no spills) rather than three.
// Multi-wave ones: the sweep's records and values one segment ahead take about
// 40 registers, which would cost a resident wave per SIMD where the rows are
// short; held to the count that the rows alone allow, the compiler parks a few
// of the row's own across the sweep instead (1024 triangular solves of 256
// rows: 34.4 us without the limit, 24.6 with it; 700 systems of 182 rows with
// ILU(0): 325 and 191 us).
// One-wave BatchTrsv of 4 slots: the packed triangle of a small system leaves
// room for many waves, whose loads hide one another; six per SIMD at 80
// registers (16384 lower triangles of 12 rows, 3 entries each: 17.3 us at five,
// 16.2 at six; 19 at three and with groups of eight columns).
template <class S, bool TRSV>
constexpr int kTriOcc = S::TEAM > kWave && S::TEAM < 1024 && S::NZ <= (TRSV ? 32 : 16)
                            ? (S::NZ <= (TRSV ? 16 : 8) ? 4 : 3)
                        : TRSV && S::TEAM == kWave && S::NZ == 4 ? 6
                                                                 : S::OCC_MIXED;

template <class S, bool MIXED, int PK = kPkScalar>
__global__ __launch_bounds__(S::WG) __attribute__((amdgpu_waves_per_eu(PK == kPkIlu ? kTriOcc<S, false> : MIXED ? S::OCC_MIXED : PK == kPkBlock ? S::OCC_BLOCK : S::OCC))) void k_bicgstab(const KArgs g) {
  BS_PERSISTENT_LOOP((kLds32<S, MIXED>), (PK == kPkIlu ? kRegBlock<S, false> : 0),
                     (bicgstab_system<MIXED, PK>(tm, A, ga)))
}

template <class S, bool LOWER>
__global__ __launch_bounds__(S::WG) __attribute__((amdgpu_waves_per_eu(kTriOcc<S, true>))) void k_trsv(const KArgs g) {
  BS_PERSISTENT_LOOP(false, (kRegBlock<S, true>), (trsv_system<LOWER>(tm, A, ga)))
}

template <class S, int PK = kPkScalar>
__global__ __launch_bounds__(S::WG) __attribute__((amdgpu_waves_per_eu(PK == kPkBlock ? S::OCC_BLOCK : S::OCC))) void k_cg(const KArgs g) {
  BS_PERSISTENT_LOOP(false, 0, (cg_system<PK>(tm, A, ga)))
}

// GMRES keeps its basis in registers beside the row: held to three waves per
// SIMD, the one-wave shapes of 24..32 slots spill (60..148 bytes per lane),
// and their LDS (staging plus the Hessenberg scalars, about 16 KB per wave)
// leaves room for only 2.5 anyway, so they are held to two, as the mixed ones.
template <class S, bool MIXED, int PK = kPkScalar>
__global__ __launch_bounds__(S::WG) __attribute__((amdgpu_waves_per_eu(S::OCC_MIXED))) void k_gmres(const KArgs g) {
  BS_PERSISTENT_LOOP((kLds32<S, MIXED>), 0, (gmres_system<MIXED, PK>(tm, A, ga)))
}

#undef BS_PERSISTENT_LOOP

}  // namespace bs
