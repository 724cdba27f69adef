// Host side of the C ABI declared in include/batchsolve.h: argument and pattern
// validation, one-time pattern preprocessing (Sec. 3.1: one pattern copy for the
// whole batch), the kernel-shape planner (Sec. 3.3 multi-level dispatch,
// Sec. 3.5 on-chip placement, Sec. 3.6 size-dependent work-group choice) and the
// launch of the fused solver kernel.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <string>
#include <mutex>
#include <vector>

#include "../../include/batchsolve.h"
#include "bs_layout.hpp"
#include "bs_registry.hpp"
#include "bs_shape.hpp"

struct bs_pattern_s {
  int n = 0, nnz = 0, width = 0, max_row = 0, device = -1;
  std::vector<int> row_ptr, col, slot_col, row_len, diag_slot;
  // Multi-wave ILU(0) and BatchTrsv (patterns of up to 1024 rows).  The rows
  // are taken by level in the lower (upper) triangle's dependency graph, the
  // lower (upper) order; levels of the rows in lower order, their number, and
  // the same rows' places in the upper order.
  std::vector<int> lev, up;
  int nlev = 0;
  // Places of a row in the two orders (lower | upper << 16), and of each entry (CSR order) in the factor array
  // (bs::IluMw); noff: entries off the diagonal.
  std::vector<int> place;
  std::vector<unsigned short> pos;
  int noff = 0;
  // ILU(0) schedule: the groups of row i, the q-th in lower order (from word
  // ilu_ptr[q]), in increasing pivot column k, five words each: 1 << 31 | place of (k,k) << 15 | place of (i,k),
  // or 0 when the group goes on with the last pivot; then four updates, place
  // of (k,j) << 16 | place of (i,j), one per entry (i,j), j > k, that row k
  // holds (filled up with the zero and the discard cell).
  std::vector<int> ilu_ptr, ilu_ops;
  // Sweep segments: the rows of a level (at most 64 per step) with four of their
  // strictly lower (upper) terms in increasing column, 2^w records of four
  // words per segment, one per lane:
  //   0, 1  byte offsets of the terms' columns in the sweep vector, 16 bits each
  //         (the zero cell past the row's last term)
  //   2     byte offsets of the row in the sweep's order and in the upper order
  //         (the cell behind the zero cell on lanes without a row)
  //   3     place of the first term in the factor array, terms << 16, 1 << 30 on
  //         a row's first segment, 1 << 31 on its last
  // Segments without rows make their number a multiple of four and are read
  // four ahead.
  std::vector<int> seg[2];
  int nseg[2] = {0, 0}, wseg[2] = {0, 0};
  bool one_seg[2] = {true, true};  // no row takes more than one segment
  // ILU(0) schedule of the one-wave factorization (patterns of up to 64 rows;
  // F is the factor array, row-major with stride ilu_stride(n)): for each pivot
  // k that a later row holds, in increasing order, its columns j > k that such
  // a row holds too, four per record of 16 words:
  //   0..7   per column, the rows i > k that hold both k and j (64 bits each,
  //          none past the pivot's last column)
  //   8..11  per column, its byte offset in a row (that of k past the last)
  //   12, 13 the rows i > k that hold k
  //   14     byte offset of column k, bit 31 on the pivot's first record
  //   15     byte offset of row k
  // Empty records make their number a multiple of three, and two more are read
  // ahead.
  std::vector<int> ilu64;
  int ilu64_records = 0;
  // bank-aware layout for one-wave teams of layout_nz register slots (0: none)
  std::vector<int> layout;
  int layout_nz = 0;
  // one allocation: ilu64 | seg[0] | seg[1] | row_ptr | slot_col | row_len |
  // diag_slot | lev | up | place | ilu_ptr | ilu_ops | pos | layout
  int* d_base = nullptr;
  int *d_seg[2] = {nullptr, nullptr};
  int *d_row_ptr = nullptr, *d_slot_col = nullptr, *d_row_len = nullptr, *d_diag = nullptr;
  int *d_lev = nullptr, *d_up = nullptr, *d_place = nullptr, *d_ilu_ptr = nullptr, *d_ilu_ops = nullptr, *d_pos = nullptr;
  int* d_layout = nullptr;
};

namespace {
thread_local std::string g_last_error = "";
}  // namespace

namespace bs {
// The streamed placement of shared-pattern batches (bs_stream_api.hip).
int stream_plan(int n, bs_solver solver, bs_precond precond, const bs_options* o,
                bs_plan_info* info);
int stream_launch(const KArgs& a, const bs_plan_info& info, bs_solver solver, int mixed, int cus,
                  hipStream_t s);

// Shared by every translation unit of the library (bs_last_error reads it).
void set_last_error(const std::string& msg) { g_last_error = msg; }

// A device word per device that kernels may write instead of an output the
// caller did not ask for (allocated once, kept until the process ends).
int* device_sink() {
  static std::mutex mu;
  static std::vector<int*> sinks;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return nullptr;
  std::lock_guard<std::mutex> lock(mu);
  if ((int)sinks.size() <= dev) sinks.resize(dev + 1, nullptr);
  if (!sinks[dev]) {
    void* p = nullptr;
    if (hipMalloc(&p, 256) != hipSuccess) {
      g_last_error = "sink allocation failed";
      return nullptr;
    }
    sinks[dev] = static_cast<int*>(p);
  }
  return sinks[dev];
}

// Compute units of the current device (cached per device); -1 on an error.
int device_cus() {
  static int cache[64] = {0};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return -1;
  if (cache[dev] == 0) {
    int v = 0;
    if (hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
      return -1;
    cache[dev] = v;
  }
  return cache[dev];
}
}  // namespace bs

namespace {

int hip_fail(hipError_t e, const char* what) {
  g_last_error = std::string(what) + ": " + hipGetErrorString(e);
  return BS_ERR_HIP;
}

constexpr int kLdsPerCu = 160 * 1024;

// The multi-wave triangular schedules hold rows and entries in 16-bit words.
constexpr int kTriRows = 1024;

// Level scheduling of a pattern's triangles (see bs_pattern_s): a row's lower
// level is one more than the largest lower level among the columns j < i it
// holds (0 if none), its upper level likewise over the columns j > i, taken
// from the last row up.  Every pattern that a multi-wave shape can take pays
// for this when it is created, whatever it is used for, so it works on flat
// arrays of known size (1000 rows of 9 entries, the whole creation: 442 us with a
// list per row and growing vectors, now 213).
void tri_schedule(bs_pattern_s& p) {
  const int n = p.n;
  // the strictly lower (0) and upper (1) entries of each row in increasing
  // column: row i's are terms[base[t][i] .. +count[t][i]], and that index is
  // the entry's place in the factor array
  std::vector<int> terms(p.nnz), base[2], count[2], level[2], order[2], at[2];
  for (int t = 0; t < 2; ++t) {
    base[t].resize(n);
    count[t].resize(n);
    level[t].assign(n, 0);
    order[t].resize(n);
    at[t].resize(n);
  }
  p.pos.assign(p.nnz, 0);
  p.noff = 0;
  std::vector<std::pair<int, int>> row;
  for (int i = 0; i < n; ++i) {
    const int e0 = p.row_ptr[i], e1 = p.row_ptr[i + 1];
    bool sorted = true;
    for (int e = e0 + 1; e < e1; ++e) sorted = sorted && p.col[e - 1] < p.col[e];
    row.clear();
    if (!sorted) {
      for (int e = e0; e < e1; ++e) row.push_back({p.col[e], e});
      std::sort(row.begin(), row.end());
    }
    base[0][i] = p.noff;
    count[0][i] = count[1][i] = 0;
    for (int q = e0; q < e1; ++q) {
      const int j = sorted ? p.col[q] : row[q - e0].first, e = sorted ? q : row[q - e0].second;
      if (j == i) continue;
      ++count[j > i][i];
      p.pos[e] = (unsigned short)p.noff;
      terms[p.noff++] = j;
    }
    base[1][i] = base[0][i] + count[0][i];
  }
  auto of = [&](int t, int i) { return terms.data() + base[t][i]; };
  for (int i = 0; i < n; ++i)
    for (int q = 0; q < count[0][i]; ++q) level[0][i] = std::max(level[0][i], level[0][of(0, i)[q]] + 1);
  for (int i = n - 1; i >= 0; --i)
    for (int q = 0; q < count[1][i]; ++q) level[1][i] = std::max(level[1][i], level[1][of(1, i)[q]] + 1);
  // rows by level, in increasing order inside one, and each row's place among them
  std::vector<int> first;
  for (int t = 0; t < 2; ++t) {
    first.assign(n + 1, 0);
    for (int i = 0; i < n; ++i) ++first[level[t][i] + 1];
    for (int l = 0; l < n; ++l) first[l + 1] += first[l];
    for (int i = 0; i < n; ++i) order[t][at[t][i] = first[level[t][i]]++] = i;
  }
  p.place.resize(n);
  p.lev.resize(n);
  p.up.resize(n);
  for (int i = 0; i < n; ++i) p.place[i] = at[0][i] | (at[1][i] << 16);
  for (int q = 0; q < n; ++q) {
    p.lev[q] = level[0][order[0][q]];
    p.up[q] = at[1][order[0][q]];
  }
  p.nlev = p.lev.back() + 1;
  const int diag0 = p.noff;
  for (int i = 0; i < n; ++i)
    if (p.diag_slot[i] >= 0) p.pos[p.row_ptr[i] + p.diag_slot[i]] = (unsigned short)(diag0 + at[1][i]);
  // sweep segments
  struct Step { int first, rows, most; };  // place of the first row, rows, their longest row
  std::vector<Step> steps;
  for (int t = 0; t < 2; ++t) {
    steps.clear();
    int w = 0, total = 0;
    p.one_seg[t] = true;
    for (int q = 0; q < n;) {
      Step st{q, 0, 1};
      const int l = level[t][order[t][q]];
      for (; st.rows < bs::kWave && q < n && level[t][order[t][q]] == l; ++q, ++st.rows)
        st.most = std::max(st.most, count[t][order[t][q]]);
      while ((1 << w) < st.rows) ++w;
      total += (st.most + 3) / 4;
      p.one_seg[t] = p.one_seg[t] && st.most <= 4;
      steps.push_back(st);
    }
    p.wseg[t] = w;
    p.nseg[t] = (total + 3) / 4 * 4;
    // records without a row, then the rows' over them
    const unsigned zero = (unsigned)n * 8 * 0x10001u, spare = (unsigned)(n + 1) * 8 * 0x10001u;
    p.seg[t].resize(((size_t)(p.nseg[t] + 4) << w) * 4);
    unsigned* r = reinterpret_cast<unsigned*>(p.seg[t].data());
    for (size_t k = 0; k < p.seg[t].size(); k += 4) {
      r[k] = r[k + 1] = zero;
      r[k + 2] = spare;
      r[k + 3] = 0;
    }
    for (const Step& st : steps) {
      for (int l = 0; l < st.rows; ++l) {
        const int i = order[t][st.first + l],* tm = of(t, i), own = at[t][i] * 8 | (at[1][i] * 8 << 16);
        unsigned* s = r + (size_t)l * 4;
        for (int k0 = 0; k0 < st.most; k0 += 4, s += (size_t)4 << w) {
          unsigned col[4];
          int c = 0;
          for (; c < 4 && k0 + c < count[t][i]; ++c) col[c] = (unsigned)at[t][tm[k0 + c]] * 8;
          for (int q = c; q < 4; ++q) col[q] = (unsigned)n * 8;
          s[0] = col[0] | (col[1] << 16);
          s[1] = col[2] | (col[3] << 16);
          s[2] = (unsigned)own;
          s[3] = (unsigned)(c ? base[t][i] + k0 : 0) | ((unsigned)c << 16) | (k0 == 0 ? 1u << 30 : 0u) |
                 (k0 + 4 >= st.most ? 1u << 31 : 0u);
        }
      }
      r += ((size_t)((st.most + 3) / 4) << w) * 4;
    }
  }
  // The ILU(0) schedule (symbolic factorization, the IKJ form): for a lower
  // entry (i,k) at most a group per four upper entries of row k, and at least one.
  size_t most = 0;
  for (int i = 0; i < n; ++i)
    for (int q = 0; q < count[0][i]; ++q) most += (size_t)std::max((count[1][of(0, i)[q]] + 3) / 4, 1);
  const unsigned discard = (unsigned)(diag0 + n), zero = discard + 1;
  p.ilu_ptr.assign(n + 1, 0);
  p.ilu_ops.resize(most * 5);
  unsigned* ops = reinterpret_cast<unsigned*>(p.ilu_ops.data());
  unsigned* out = ops;
  std::vector<int> where(n, -1);  // place of (i, j), for the row i at hand
  for (int q0 = 0; q0 < n; ++q0) {
    const int i = order[0][q0];
    for (int e = p.row_ptr[i]; e < p.row_ptr[i + 1]; ++e) where[p.col[e]] = p.pos[e];
    for (int q = 0; q < count[0][i]; ++q) {
      const int k = of(0, i)[q], * uk = of(1, k);
      unsigned head = 1u << 31 | (unsigned)(diag0 + at[1][k]) << 15 | (unsigned)(base[0][i] + q);
      int u = 0;
      for (int c = 0; c < count[1][k]; ++c) {
        const int w = where[uk[c]];
        if (w < 0) continue;
        if ((u & 3) == 0) {
          *out++ = head;
          head = 0;
        }
        *out++ = (unsigned)(base[1][k] + c) << 16 | (unsigned)w;
        ++u;
      }
      if (u == 0) *out++ = head;
      for (; u == 0 || (u & 3); ++u) *out++ = zero << 16 | discard;
    }
    for (int e = p.row_ptr[i]; e < p.row_ptr[i + 1]; ++e) where[p.col[e]] = -1;
    p.ilu_ptr[q0 + 1] = (int)(out - ops);
  }
  p.ilu_ops.resize(out - ops);
}

const bs::KernelEntry* find_kernel(int variant, int team, int r, int nz_min);

// Whether some multi-wave shape can take the pattern for ILU(0) or BatchTrsv:
// the schedule of a pattern that none holds would only cost its creation time
// (a dense one of 150 rows: 2 ms).
bool takes_tri_schedule(const bs_pattern_s& p) {
  if (p.n > kTriRows || p.nnz >= (1 << 15) || bs::tri_limit_bytes(p.n, p.nnz) > kLdsPerCu)
    return false;
  for (int t = 2 * bs::kWave; t <= 1024; t *= 2)
    if (t >= p.n && (find_kernel(bs::V_BICGSTAB_ILU, t, 1, std::max(p.max_row, 1)) ||
                     find_kernel(bs::V_TRSV_LOWER, t, 1, std::max(p.max_row, 1))))
      return true;
  return false;
}

// Derived per-row data shared by the CSR and ELL forms.
void derive(bs_pattern_s& p) {
  const int n = p.n;
  p.row_len.resize(n);
  p.diag_slot.assign(n, -1);
  p.max_row = 0;
  for (int i = 0; i < n; ++i) {
    const int len = p.row_ptr[i + 1] - p.row_ptr[i];
    p.row_len[i] = len;
    p.max_row = std::max(p.max_row, len);
    for (int k = 0; k < len; ++k)
      if (p.col[p.row_ptr[i] + k] == i && p.diag_slot[i] < 0) p.diag_slot[i] = k;
  }
  p.width = p.max_row;
  p.slot_col.assign((size_t)p.width * n, -1);
  for (int s = 0; s < p.width; ++s)
    for (int i = 0; i < n; ++i)
      if (s < p.row_len[i]) p.slot_col[(size_t)s * n + i] = p.col[p.row_ptr[i] + s];
  if (takes_tri_schedule(p)) tri_schedule(p);
  // The one-wave schedule: rows and columns as 64-bit masks.
  p.ilu64.clear();
  if (n <= bs::kWave) {
    uint64_t row[bs::kWave] = {0}, col[bs::kWave] = {0};
    for (int i = 0; i < n; ++i)
      for (int e = p.row_ptr[i]; e < p.row_ptr[i + 1]; ++e) {
        row[i] |= 1ull << p.col[e];
        col[p.col[e]] |= 1ull << i;
      }
    const int stride = bs::ilu_stride(n) * 8;
    // a pivot has at most a record for every four of its columns, and one
    p.ilu64.resize(((size_t)n * (bs::kWave / 4 + 1) + 4) * 16);
    unsigned* w = reinterpret_cast<unsigned*>(p.ilu64.data());
    for (int k = 0; k + 1 < n; ++k) {
      const uint64_t later = (~0ull << k) << 1, below = col[k] & later;
      if (!below) continue;
      uint64_t js = row[k] & later;  // columns of row k ..
      for (uint64_t m = js; m; m &= m - 1)  // .. that a row below holds
        if (!(col[__builtin_ctzll(m)] & below)) js &= ~(m & -m);
      bool head = true;
      do {
        for (int q = 0; q < 4; ++q) {
          const int j = js ? __builtin_ctzll(js) : k;
          const uint64_t rows = js ? col[j] & below : 0;
          js &= js - 1;
          w[2 * q] = (unsigned)rows;
          w[2 * q + 1] = (unsigned)(rows >> 32);
          w[8 + q] = (unsigned)j * 8;
        }
        w[12] = (unsigned)below;
        w[13] = (unsigned)(below >> 32);
        w[14] = (unsigned)(k * 8) | (head ? 1u << 31 : 0u);
        w[15] = (unsigned)(k * stride);
        head = false;
        w += 16;
      } while (js);
    }
    const int records = (int)(w - reinterpret_cast<unsigned*>(p.ilu64.data())) / 16;
    p.ilu64_records = (records + 2) / 3 * 3;
    p.ilu64.resize((size_t)records * 16);  // the empty ones behind them are zero
    p.ilu64.resize((size_t)(p.ilu64_records + 2) * 16, 0);
  }
}

int upload(bs_pattern_s& p) {
  int count = 0;
  if (hipGetDeviceCount(&count) != hipSuccess || count < 1) {
    (void)hipGetLastError();
    g_last_error = "no HIP device";
    return BS_ERR_NO_DEVICE;
  }
  hipError_t e = hipGetDevice(&p.device);
  if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
  // the regions in order: the schedules read 16 or 64 bytes at a time first
  std::vector<int> h;
  auto put = [&](const auto& v, size_t least = 0) {
    const size_t off = h.size();
    h.insert(h.end(), v.begin(), v.end());
    h.resize(std::max(h.size(), off + least), -1);
    return off;
  };
  h.reserve(p.ilu64.size() + p.seg[0].size() + p.seg[1].size() + p.row_ptr.size() + p.slot_col.size() + 1 +
            p.row_len.size() + p.diag_slot.size() + p.lev.size() + p.up.size() + p.place.size() +
            p.ilu_ptr.size() + p.ilu_ops.size() + (p.pos.size() + 1) / 2 + p.layout.size());
  std::vector<int> pos((p.pos.size() + 1) / 2, 0);
  if (!p.pos.empty()) std::memcpy(pos.data(), p.pos.data(), p.pos.size() * sizeof(unsigned short));
  put(p.ilu64);
  const size_t o_seg0 = put(p.seg[0]), o_seg1 = put(p.seg[1]);
  const size_t o_rp = put(p.row_ptr), o_sc = put(p.slot_col, 1), o_rl = put(p.row_len),
               o_ds = put(p.diag_slot), o_lev = put(p.lev), o_up = put(p.up), o_place = put(p.place),
               o_ptr = put(p.ilu_ptr), o_ops = put(p.ilu_ops), o_pos = put(pos), o_lay = put(p.layout);
  const size_t total = h.size();
  e = hipMalloc(&p.d_base, total * sizeof(int));
  if (e != hipSuccess) return hip_fail(e, "hipMalloc(pattern)");
  p.d_seg[0] = p.d_base + o_seg0;
  p.d_seg[1] = p.d_base + o_seg1;
  p.d_row_ptr = p.d_base + o_rp;
  p.d_slot_col = p.d_base + o_sc;
  p.d_row_len = p.d_base + o_rl;
  p.d_diag = p.d_base + o_ds;
  p.d_lev = p.d_base + o_lev;
  p.d_up = p.d_base + o_up;
  p.d_place = p.d_base + o_place;
  p.d_ilu_ptr = p.d_base + o_ptr;
  p.d_ilu_ops = p.d_base + o_ops;
  p.d_pos = p.d_base + o_pos;
  p.d_layout = p.layout.empty() ? nullptr : p.d_base + o_lay;
  e = hipMemcpy(p.d_base, h.data(), total * sizeof(int), hipMemcpyHostToDevice);
  if (e != hipSuccess) {
    (void)hipFree(p.d_base);
    p.d_base = nullptr;
    return hip_fail(e, "hipMemcpy(pattern)");
  }
  return BS_OK;
}

// Columns of one row must be in range and distinct.
bool row_ok(const int* cols, int len, int n, std::vector<int>& mark, int stamp) {
  for (int k = 0; k < len; ++k) {
    const int c = cols[k];
    if (c < 0 || c >= n || mark[c] == stamp) return false;
    mark[c] = stamp;
  }
  return true;
}

// block: block-Jacobi block size (0 without); block Jacobi is FP64 only.
int variant_of(bs_solver solver, int precision, int block = 0, bool ilu = false) {
  if (solver == BS_TRSV_LOWER || solver == BS_TRSV_UPPER) {
    if (precision == BS_MIXED) return -1;
    return solver == BS_TRSV_LOWER ? bs::V_TRSV_LOWER : bs::V_TRSV_UPPER;
  }
  if (ilu) {
    if (precision == BS_MIXED) return -1;
    if (solver == BS_BICGSTAB) return bs::V_BICGSTAB_ILU;
    if (solver == BS_GMRES) return bs::V_GMRES_ILU;
    return -1;  // CG needs a symmetric preconditioner
  }
  if (block > 1) {
    if (precision == BS_MIXED) return -1;
    if (solver == BS_CG) return bs::V_CG_BJ;
    if (solver == BS_BICGSTAB) return bs::V_BICGSTAB_BJ;
    if (solver == BS_GMRES) return bs::V_GMRES_BJ;
    return -1;
  }
  if (solver == BS_CG) return precision == BS_MIXED ? -1 : bs::V_CG;
  if (solver == BS_BICGSTAB) return precision == BS_MIXED ? bs::V_BICGSTAB_MIXED : bs::V_BICGSTAB;
  if (solver == BS_GMRES) return precision == BS_MIXED ? bs::V_GMRES_MIXED : bs::V_GMRES;
  return -1;
}

bs::KernelTable table_of(int variant) {
  switch (variant) {
    case bs::V_CG: return bs::kernels_cg();
    case bs::V_BICGSTAB: return bs::kernels_bicgstab();
    case bs::V_BICGSTAB_MIXED: return bs::kernels_bicgstab_mixed();
    case bs::V_GMRES: return bs::kernels_gmres();
    case bs::V_GMRES_MIXED: return bs::kernels_gmres_mixed();
    case bs::V_CG_BJ: return bs::kernels_cg_bj();
    case bs::V_BICGSTAB_BJ: return bs::kernels_bicgstab_bj();
    case bs::V_GMRES_BJ: return bs::kernels_gmres_bj();
    case bs::V_BICGSTAB_ILU: return bs::kernels_bicgstab_ilu();
    case bs::V_GMRES_ILU: return bs::kernels_gmres_ilu();
    case bs::V_TRSV_LOWER: return bs::kernels_trsv_lower();
    case bs::V_TRSV_UPPER: return bs::kernels_trsv_upper();
    default: return {nullptr, 0};
  }
}

const bs::KernelEntry* find_kernel(int variant, int team, int r, int nz_min) {
  const bs::KernelTable t = table_of(variant);
  const bs::KernelEntry* best = nullptr;
  for (int i = 0; i < t.count; ++i) {
    const bs::KernelEntry& e = t.entries[i];
    if (e.team == team && e.r == r && e.nz >= nz_min && (!best || e.nz < best->nz)) best = &e;
  }
  return best;
}

// Rows of 33..64 entries are solved by one-wave teams (one row per lane); such a
// pattern gets its bank-aware layout for the register-slot count the planner
// takes for it.
constexpr int kLayoutSteps = 20000;

void choose_layout(bs_pattern_s& p) {
  p.layout.clear();
  p.layout_nz = 0;
  if (p.n <= 32 || p.n > bs::kLayoutLanes) return;
  const bs::KernelEntry* k = find_kernel(bs::V_BICGSTAB, bs::kWave, 1, std::max(p.max_row, 1));
  if (!k || p.nnz < k->nz) return;
  const bs::WaveLayout L =
      bs::choose_wave_layout(p.n, p.nnz, p.row_ptr.data(), p.col.data(), k->nz, kLayoutSteps);
  if (L.cost >= L.plain_cost) return;
  p.layout.reserve(2 * bs::kLayoutLanes + p.n);
  p.layout.insert(p.layout.end(), L.lane_row.begin(), L.lane_row.end());
  p.layout.insert(p.layout.end(), L.lane_win.begin(), L.lane_win.end());
  p.layout.insert(p.layout.end(), L.col_pos.begin(), L.col_pos.end());
  p.layout_nz = k->nz;
}

bool pow2_team(int t) { return t >= 16 && t <= 1024 && (t & (t - 1)) == 0; }

// Block-Jacobi block size of a request: 0 without block Jacobi, else 2, 4 or
// 8 (0 selects 8); -1 when the size is not one of these.
int block_of(const bs_options* o, int precond = BS_PREC_BLOCK_JACOBI) {
  if (precond != BS_PREC_BLOCK_JACOBI) return 0;
  const int b = o ? o->block_size : 0;
  if (b == 0) return 8;
  return (b == 2 || b == 4 || b == 8) ? b : -1;
}

// Staging of CSR values through LDS is used while a workgroup's staging area
// stays within this budget.
constexpr int kStageBudget = 48 * 1024;

struct Plan {
  bs_plan_info info;
  const bs::KernelEntry* k;
};

// block: block-Jacobi block size (0 without block Jacobi); ilu: ILU(0).
// ILU(0) and the triangular solves take one row per lane: a one-wave team up
// to 64 rows (dense factors), else the smallest power-of-two team of at least
// n lanes, up to 1024 (sparse factors, level-scheduled sweeps); a forced team
// must hold n rows and be at least a wave.
int make_plan(bs_format fmt, int n, int nnz, int max_row, int width, bs_solver solver,
              const bs_options* o, int block, bool ilu, Plan* out) {
  const int precision = o ? o->precision : BS_FP64;
  const int variant = variant_of(solver, precision, block, ilu);
  if (variant < 0) return BS_ERR_UNSUPPORTED;
  if (n > BS_MAX_ROWS || max_row > BS_MAX_ROW_NNZ) return BS_ERR_UNSUPPORTED;
  const bool trsv = solver == BS_TRSV_LOWER || solver == BS_TRSV_UPPER;
  const bool tri = ilu || trsv;
  if (tri && (n > 1024 || (o && ((o->team != 0 && (o->team < bs::kWave || o->team < n)) ||
                                 o->rows_per_lane > 1))))
    return BS_ERR_UNSUPPORTED;
  int tri_team = bs::kWave;
  while (tri_team < n) tri_team *= 2;
  // the multi-wave schedules address entries with 15 bits
  if (tri && n > bs::kWave && nnz >= (1 << 15)) return BS_ERR_UNSUPPORTED;
  const int force_team = tri ? (o && o->team ? o->team : tri_team) : o ? o->team : 0,
            force_r = o ? o->rows_per_lane : 0;
  if (force_team != 0 && !pow2_team(force_team)) return BS_ERR_INVALID_ARG;
  if (force_r != 0 && force_r != 1 && force_r != 2 && force_r != 4) return BS_ERR_INVALID_ARG;
  // Sec. 3.6: at least one lane per row, rounded up to a power of two no
  // smaller than the 16-lane DPP row; systems beyond one workgroup of lanes take
  // 2 or 4 rows per lane.  Shapes are tried from the fewest rows per lane and the
  // narrowest team upwards; the first compiled shape whose register slots cover
  // the longest row is taken.
  const bs::KernelEntry* k = nullptr;
  int team = 0, r = 0;
  for (int rr = 1; rr <= 4 && !k; rr *= 2) {
    if (force_r && rr != force_r) continue;
    int t = 16;
    while (t * rr < n && t < 1024) t *= 2;
    if (force_team) t = force_team;
    for (; t <= 1024 && !k; t *= 2) {
      if (t * rr < n) break;
      k = find_kernel(variant, t, rr, std::max(max_row, 1));
      team = t;
      r = rr;
      if (force_team) break;
    }
  }
  if (!k) return BS_ERR_UNSUPPORTED;
  const int rows = team * r;
  const int wg = k->wg, teams = wg / team, waves = wg / bs::kWave;
  const bool gm = variant == bs::V_GMRES || variant == bs::V_GMRES_MIXED ||
                  variant == bs::V_GMRES_BJ || variant == bs::V_GMRES_ILU;
  const int stored = fmt == BS_CSR ? nnz : width * n;
  const bool mixed = variant == bs::V_GMRES_MIXED;
  const int vec = teams * (bs::team_vec_bytes(rows, gm, wg, mixed) + bs::bj_bytes(rows, block) +
                           (tri ? bs::tri_region_bytes(team, n, nnz, trsv) : 0)) +
                  bs::red_lds_bytes(waves);
  int stage = 0;
  // ILU(0) and the triangular solves are bound by their substitution chains,
  // not by loading the values: their LDS goes to more resident waves instead
  // of staging
  // Nor is anything staged where nothing is stored: the copy would read from
  // an array of no element.
  if (waves == 1 && !tri && stored > 0 &&
      bs::stage_total_bytes(teams, stored, n, k->nz) <= kStageBudget)
    stage = 1;
  // Multi-wave teams, CSR, rows of many slots: each system's values copied
  // into LDS by the whole group (coalesced direct-to-LDS loads issued during
  // the previous system's solve), where they fit beside the vectors; the
  // launch keeps it only where it costs no resident group.
  if (waves > 1 && fmt == BS_CSR && !tri && k->nz >= bs::kStageMinSlots &&
      vec + bs::stage_vals_bytes(teams, stored, k->nz) <= kLdsPerCu)
    stage = 2;
  out->k = k;
  out->info.team = team;
  out->info.rows_per_lane = r;
  out->info.slots = k->nz;
  out->info.group_size = wg;
  out->info.systems_per_group = teams;
  out->info.lds_bytes = vec + (stage == 1   ? bs::stage_total_bytes(teams, stored, n, k->nz)
                               : stage == 2 ? bs::stage_vals_bytes(teams, stored, k->nz)
                                            : 0);
  out->info.stage_values = stage;
  // a workgroup's LDS is at most that of a compute unit
  if (out->info.lds_bytes > kLdsPerCu) return BS_ERR_UNSUPPORTED;
  if (tri && team > bs::kWave &&
      vec - bs::tri_region_bytes(team, n, nnz, trsv) + bs::tri_limit_bytes(n, nnz) > kLdsPerCu)
    return BS_ERR_UNSUPPORTED;
  return BS_OK;
}

__global__ void k_csr_to_ell(int64_t n_batch, int n, int nnz, int width, const int* row_ptr,
                             const int* row_len, const double* src, double* dst) {
  const int64_t per = (int64_t)width * n;
  const int64_t total = n_batch * per;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t s = e / per;
    const int rem = (int)(e - s * per);
    const int slot = rem / n, i = rem - slot * n;
    dst[e] = slot < row_len[i] ? src[s * nnz + row_ptr[i] + slot] : 0.0;
  }
}

}  // namespace

extern "C" {

const char* bs_error_string(int code) {
  switch (code) {
    case BS_OK: return "success";
    case BS_ERR_INVALID_ARG: return "invalid argument";
    case BS_ERR_PATTERN: return "malformed sparsity pattern";
    case BS_ERR_UNSUPPORTED: return "unsupported shape or option";
    case BS_ERR_HIP: return "HIP runtime error";
    case BS_ERR_NO_DEVICE: return "no HIP device";
    default: return "unknown error";
  }
}

const char* bs_last_error(void) { return g_last_error.c_str(); }

int bs_pattern_create_csr(int32_t n_rows, int32_t nnz, const int32_t* row_ptr,
                          const int32_t* col_idx, bs_pattern* out) {
  if (!out || !row_ptr || (nnz > 0 && !col_idx) || n_rows < 1 || nnz < 0)
    return BS_ERR_INVALID_ARG;
  *out = nullptr;
  if (row_ptr[0] != 0 || row_ptr[n_rows] != nnz) return BS_ERR_PATTERN;
  for (int i = 0; i < n_rows; ++i)
    if (row_ptr[i + 1] < row_ptr[i]) return BS_ERR_PATTERN;
  std::vector<int> mark(n_rows, -1);
  for (int i = 0; i < n_rows; ++i)
    if (!row_ok(col_idx + row_ptr[i], row_ptr[i + 1] - row_ptr[i], n_rows, mark, i))
      return BS_ERR_PATTERN;
  bs_pattern_s* p = new bs_pattern_s();
  p->n = n_rows;
  p->nnz = nnz;
  p->row_ptr.assign(row_ptr, row_ptr + n_rows + 1);
  p->col.assign(col_idx, col_idx + nnz);
  derive(*p);
  choose_layout(*p);
  const int rc = upload(*p);
  if (rc != BS_OK) {
    delete p;
    return rc;
  }
  *out = p;
  return BS_OK;
}

int bs_pattern_create_dense(int32_t n_rows, bs_pattern* out) {
  if (!out || n_rows < 1 || n_rows > 46340) return BS_ERR_INVALID_ARG;
  *out = nullptr;
  const int n = n_rows;
  std::vector<int32_t> rp(n + 1), col((size_t)n * n);
  for (int i = 0; i <= n; ++i) rp[i] = i * n;
  for (int i = 0; i < n; ++i)
    for (int j = 0; j < n; ++j) col[(size_t)i * n + j] = j;
  return bs_pattern_create_csr(n, n * n, rp.data(), col.data(), out);
}

int bs_pattern_create_ell(int32_t n_rows, int32_t ell_width, const int32_t* ell_col,
                          bs_pattern* out) {
  if (!out || n_rows < 1 || ell_width < 0 || (ell_width > 0 && !ell_col))
    return BS_ERR_INVALID_ARG;
  *out = nullptr;
  std::vector<int> rp(n_rows + 1, 0), col;
  for (int i = 0; i < n_rows; ++i) {
    int len = 0;
    bool pad = false;
    for (int s = 0; s < ell_width; ++s) {
      const int c = ell_col[(size_t)s * n_rows + i];
      if (c == -1) {
        pad = true;
      } else {
        if (pad || c < -1 || c >= n_rows) return BS_ERR_PATTERN;
        ++len;
      }
    }
    rp[i + 1] = rp[i] + len;
  }
  col.resize(rp[n_rows]);
  for (int i = 0; i < n_rows; ++i)
    for (int s = 0; s < rp[i + 1] - rp[i]; ++s) col[rp[i] + s] = ell_col[(size_t)s * n_rows + i];
  std::vector<int> mark(n_rows, -1);
  for (int i = 0; i < n_rows; ++i)
    if (!row_ok(col.data() + rp[i], rp[i + 1] - rp[i], n_rows, mark, i)) return BS_ERR_PATTERN;
  bs_pattern_s* p = new bs_pattern_s();
  p->n = n_rows;
  p->nnz = rp[n_rows];
  p->row_ptr = std::move(rp);
  p->col = std::move(col);
  derive(*p);
  // Keep the caller's width (it may include all-padding slots).
  if (ell_width > p->width) {
    p->slot_col.resize((size_t)ell_width * n_rows, -1);
    p->width = ell_width;
  }
  choose_layout(*p);
  const int rc = upload(*p);
  if (rc != BS_OK) {
    delete p;
    return rc;
  }
  *out = p;
  return BS_OK;
}

int bs_pattern_destroy(bs_pattern p) {
  if (!p) return BS_OK;
  if (p->d_base) (void)hipFree(p->d_base);
  delete p;
  return BS_OK;
}

int bs_wave_layout(int32_t n_rows, int32_t nnz, const int32_t* row_ptr, const int32_t* col_idx,
                   int32_t slots, int32_t steps, int32_t* lane_row, int32_t* lane_win,
                   int32_t* col_pos, int64_t* cost) {
  if (!row_ptr || (nnz > 0 && !col_idx) || !lane_row || !lane_win || !col_pos || !cost ||
      n_rows < 1 || nnz < 0 || slots < 1 || steps < 0)
    return BS_ERR_INVALID_ARG;
  if (row_ptr[0] != 0 || row_ptr[n_rows] != nnz) return BS_ERR_PATTERN;
  int max_row = 0;
  for (int i = 0; i < n_rows; ++i) {
    if (row_ptr[i + 1] < row_ptr[i]) return BS_ERR_PATTERN;
    max_row = std::max(max_row, row_ptr[i + 1] - row_ptr[i]);
  }
  std::vector<int> mark(n_rows, -1);
  for (int i = 0; i < n_rows; ++i)
    if (!row_ok(col_idx + row_ptr[i], row_ptr[i + 1] - row_ptr[i], n_rows, mark, i))
      return BS_ERR_PATTERN;
  if (n_rows <= 32 || n_rows > bs::kLayoutLanes || nnz < slots || max_row > slots)
    return BS_ERR_UNSUPPORTED;
  const bs::WaveLayout L = bs::choose_wave_layout(n_rows, nnz, row_ptr, col_idx, slots, steps);
  std::copy(L.lane_row.begin(), L.lane_row.end(), lane_row);
  std::copy(L.lane_win.begin(), L.lane_win.end(), lane_win);
  std::copy(L.col_pos.begin(), L.col_pos.end(), col_pos);
  cost[0] = L.cost;
  cost[1] = L.plain_cost;
  return BS_OK;
}

int bs_pattern_layout(bs_pattern p, int32_t* slots, int32_t* layout) {
  if (!p || !slots) return BS_ERR_INVALID_ARG;
  *slots = p->layout_nz;
  if (layout) std::copy(p->layout.begin(), p->layout.end(), layout);
  return BS_OK;
}

int bs_pattern_query(bs_pattern p, int32_t* n_rows, int32_t* nnz, int32_t* ell_width,
                     int32_t* max_row_nnz) {
  if (!p) return BS_ERR_INVALID_ARG;
  if (n_rows) *n_rows = p->n;
  if (nnz) *nnz = p->nnz;
  if (ell_width) *ell_width = p->width;
  if (max_row_nnz) *max_row_nnz = p->max_row;
  return BS_OK;
}

int bs_pattern_ell_cols(bs_pattern p, int32_t* out) {
  if (!p || (!out && p->width > 0)) return BS_ERR_INVALID_ARG;
  std::copy(p->slot_col.begin(), p->slot_col.end(), out);
  return BS_OK;
}

int bs_values_csr_to_ell(bs_pattern p, int64_t n_batch, const double* csr, double* ell,
                         void* stream) {
  if (!p || n_batch < 0) return BS_ERR_INVALID_ARG;
  if (n_batch == 0 || p->width == 0) return BS_OK;
  if (!csr || !ell) return BS_ERR_INVALID_ARG;
  const int64_t total = n_batch * (int64_t)p->width * p->n;
  const int64_t blocks = std::min<int64_t>((total + 255) / 256, 1 << 20);
  hipLaunchKernelGGL(k_csr_to_ell, dim3((unsigned)blocks), dim3(256), 0, (hipStream_t)stream,
                     n_batch, p->n, p->nnz, p->width, p->d_row_ptr, p->d_row_len, csr, ell);
  const hipError_t e = hipGetLastError();
  return e == hipSuccess ? BS_OK : hip_fail(e, "k_csr_to_ell");
}

int bs_matrix_storage(bs_format fmt, int64_t n_batch, int32_t n_rows, int32_t nnz,
                      int32_t ell_width, int64_t* value_count, int64_t* index_count) {
  if (n_batch < 0 || n_rows < 1 || nnz < 0 || ell_width < 0 || !value_count || !index_count)
    return BS_ERR_INVALID_ARG;
  if (fmt == BS_CSR) {
    *value_count = n_batch * (int64_t)nnz;
    *index_count = (int64_t)n_rows + 1 + nnz;
  } else if (fmt == BS_DENSE) {
    *value_count = n_batch * (int64_t)n_rows * n_rows;
    *index_count = 0;
  } else if (fmt == BS_ELL) {
    *value_count = n_batch * (int64_t)ell_width * n_rows;
    *index_count = (int64_t)ell_width * n_rows;
  } else {
    return BS_ERR_INVALID_ARG;
  }
  return BS_OK;
}

int bs_plan(bs_format fmt, int32_t n_rows, int32_t nnz, int32_t max_row_nnz, bs_solver solver,
            const bs_options* opts, bs_plan_info* out) {
  if (!out || n_rows < 1 || nnz < 0 || max_row_nnz < 0 ||
      (fmt != BS_CSR && fmt != BS_ELL && fmt != BS_DENSE) ||
      (solver < BS_CG || solver > BS_TRSV_UPPER))
    return BS_ERR_INVALID_ARG;
  if (fmt == BS_DENSE) {  // the full pattern in CSR order
    nnz = n_rows * n_rows;
    max_row_nnz = n_rows;
    fmt = BS_CSR;
  }
  Plan pl;
  // planned with the block-Jacobi region when opts asks for a block size
  const int block = opts && opts->block_size != 0 ? block_of(opts) : 0;
  if (block < 0) return BS_ERR_INVALID_ARG;
  const int rc =
      make_plan(fmt, n_rows, nnz, max_row_nnz, max_row_nnz, solver, opts, block, false, &pl);
  if (rc == BS_OK) *out = pl.info;
  // no register shape: the streamed placement, where the request allows it
  if (rc == BS_ERR_UNSUPPORTED && block <= 1)
    return bs::stream_plan(n_rows, solver, BS_PREC_JACOBI, opts, out);
  return rc;
}

int bs_plan_precond(bs_format fmt, int32_t n_rows, int32_t nnz, int32_t max_row_nnz,
                    bs_solver solver, bs_precond precond, const bs_options* opts,
                    bs_plan_info* out) {
  if (!out || n_rows < 1 || nnz < 0 || max_row_nnz < 0 ||
      (fmt != BS_CSR && fmt != BS_ELL && fmt != BS_DENSE) ||
      (solver < BS_CG || solver > BS_TRSV_UPPER) ||
      (precond != BS_PREC_NONE && precond != BS_PREC_JACOBI && precond != BS_PREC_BLOCK_JACOBI &&
       precond != BS_PREC_ILU))
    return BS_ERR_INVALID_ARG;
  if (fmt == BS_DENSE) {
    nnz = n_rows * n_rows;
    max_row_nnz = n_rows;
    fmt = BS_CSR;
  }
  const int block = block_of(opts, precond);
  if (block < 0) return BS_ERR_INVALID_ARG;
  Plan pl;
  const int rc = make_plan(fmt, n_rows, nnz, max_row_nnz, max_row_nnz, solver, opts, block,
                           precond == BS_PREC_ILU, &pl);
  if (rc == BS_OK) *out = pl.info;
  if (rc == BS_ERR_UNSUPPORTED) return bs::stream_plan(n_rows, solver, precond, opts, out);
  return rc;
}

size_t bs_workspace_size(bs_format fmt, int64_t n_batch, int32_t n_rows, bs_pattern pattern,
                         bs_solver solver, const bs_options* opts) {
  (void)fmt;
  (void)n_batch;
  (void)n_rows;
  (void)pattern;
  (void)solver;
  (void)opts;
  return 0;
}

int bs_batch_solve(bs_format fmt, int64_t n_batch, int32_t n_rows, bs_pattern pattern,
                   const double* values, const double* b, double* x, bs_solver solver,
                   bs_precond precond, double tol, int32_t max_iter, int32_t* iters,
                   double* resid, int32_t* status, const bs_options* opts, void* stream) {
  if (!pattern || n_batch < 0 || n_rows != pattern->n) return BS_ERR_INVALID_ARG;
  if (fmt != BS_CSR && fmt != BS_ELL && fmt != BS_DENSE) return BS_ERR_INVALID_ARG;
  // BatchDense: row-major [n][n] values are the CSR values of the full pattern
  if (fmt == BS_DENSE) {
    if ((int64_t)pattern->nnz != (int64_t)pattern->n * pattern->n) return BS_ERR_PATTERN;
    fmt = BS_CSR;
  }
  if (solver < BS_CG || solver > BS_TRSV_UPPER) return BS_ERR_INVALID_ARG;
  if (precond != BS_PREC_NONE && precond != BS_PREC_JACOBI && precond != BS_PREC_BLOCK_JACOBI &&
      precond != BS_PREC_ILU)
    return BS_ERR_INVALID_ARG;
  if (!(tol > 0.0) || !std::isfinite(tol) || max_iter < 0) return BS_ERR_INVALID_ARG;
  // the triangular solves take no preconditioner
  const bool trsv = solver == BS_TRSV_LOWER || solver == BS_TRSV_UPPER;
  const bool ilu = precond == BS_PREC_ILU && !trsv;
  const int block = trsv ? 0 : block_of(opts, precond);
  if (block < 0) return BS_ERR_INVALID_ARG;
  int restart = bs::kMaxRestart;
  double inner_tol = 1e-6;
  int flags = 0;
  if (opts) {
    if (opts->restart < 0 || opts->restart > bs::kMaxRestart) return BS_ERR_INVALID_ARG;
    if (opts->restart > 0) restart = opts->restart;
    if (opts->precision != BS_FP64 && opts->precision != BS_MIXED) return BS_ERR_INVALID_ARG;
    if (opts->inner_tol < 0.0 || !std::isfinite(opts->inner_tol)) return BS_ERR_INVALID_ARG;
    if (opts->inner_tol > 0.0) inner_tol = opts->inner_tol;
    flags = opts->flags;
  }
  // several right-hand sides per matrix: one solve per (matrix, right-hand side)
  const int nrhs = opts && opts->n_rhs > 0 ? opts->n_rhs : 1;
  if (opts && opts->n_rhs < 0) return BS_ERR_INVALID_ARG;
  if (n_batch > INT64_MAX / nrhs) return BS_ERR_INVALID_ARG;
  const int64_t n_solves = n_batch * nrhs;
  if (n_batch == 0) return BS_OK;
  if (!values || !b || !x || !iters || !resid) return BS_ERR_INVALID_ARG;
  Plan pl;
  int rc = make_plan(fmt, pattern->n, pattern->nnz, pattern->max_row, pattern->width, solver,
                     opts, block, ilu, &pl);
  // no register shape holds the rows: the streamed placement, if it applies
  bool streamed = false;
  if (rc == BS_ERR_UNSUPPORTED && !trsv) {
    rc = bs::stream_plan(pattern->n, solver, precond, opts, &pl.info);
    streamed = rc == BS_OK;
  }
  if (rc != BS_OK) return rc;
  // multi-wave ILU(0) and BatchTrsv need the pattern's schedules
  if (!streamed && (ilu || trsv) && pl.info.team > bs::kWave && pattern->lev.empty())
    return BS_ERR_UNSUPPORTED;
  bs::KArgs a{};
  a.n_batch = n_solves;
  a.nrhs = nrhs;
  a.n = pattern->n;
  a.nnz = pattern->nnz;
  a.width = pattern->width;
  a.fmt = fmt == BS_CSR ? 0 : 1;
  a.precond = precond == BS_PREC_JACOBI ? 1 : 0;
  a.flags = flags;
  a.max_iter = max_iter;
  a.restart = restart;
  a.stage = pl.info.stage_values;
  a.gmres = solver == BS_GMRES ? 1 : 0;
  const int stored = fmt == BS_CSR ? pattern->nnz : pattern->width * pattern->n;
  if (!streamed) {
    const int rows = pl.info.team * pl.info.rows_per_lane;
    const int teams = pl.info.systems_per_group, waves = pl.info.group_size / bs::kWave;
    a.team_bytes = bs::team_vec_bytes(rows, a.gmres, pl.info.group_size,
                                      a.gmres && opts && opts->precision == BS_MIXED);
    // block Jacobi (inverse and exchange buffer) or ILU(0) (factors) after the
    // vectors
    a.block = block;
    a.bj_offset = a.team_bytes;
    a.team_bytes += bs::bj_bytes(rows, block) +
                    (ilu || trsv ? bs::tri_region_bytes(pl.info.team, pattern->n, pattern->nnz, trsv)
                                 : 0);
    a.stage_vals_bytes = bs::stage_vals_bytes(teams, stored, pl.info.slots);
    a.stage_team_bytes = a.stage_vals_bytes + bs::stage_b_bytes(teams, pattern->n);
    a.stage_offset = teams * a.team_bytes + bs::red_lds_bytes(waves);
    // One-wave ILU(0) (BiCGSTAB) and BatchTrsv: the next system's values travel
    // in registers during a solve and pass through the region of the factors
    // or the triangle, which the solve no longer needs by then; where the
    // block is longer than the registers kept for it, or than the region, the
    // rows are read straight from memory.
    if (stored > 0 && (ilu || trsv) && solver != BS_GMRES && pl.info.team == bs::kWave &&
        a.stage_vals_bytes <= bs::pf_chunks(pl.info.slots, trsv) * 1024 &&
        a.stage_vals_bytes + bs::round16(pattern->n * 8) + 16 <= a.team_bytes - a.bj_offset)
      a.stage = 3;
    // CSR rows go through a fixed window when the block holds a full window
    a.window = (fmt == BS_CSR && pattern->nnz >= pl.info.slots) ? 1 : 0;
  }
  a.tol = tol;
  a.inner_tol = inner_tol;
  a.row_ptr = pattern->d_row_ptr;
  a.slot_col = pattern->d_slot_col;
  a.row_len = pattern->d_row_len;
  a.diag_slot = pattern->d_diag;
  a.lev = pattern->d_lev;
  a.nlev = pattern->nlev;
  a.tri_up = pattern->d_up;
  a.ilu_ptr = pattern->d_ilu_ptr;
  a.ilu_ops = pattern->d_ilu_ops;
  a.tri_place = pattern->d_place;
  a.tri_pos = reinterpret_cast<const unsigned short*>(pattern->d_pos);
  a.seg_l = reinterpret_cast<const int4*>(pattern->d_seg[0]);
  a.seg_u = reinterpret_cast<const int4*>(pattern->d_seg[1]);
  a.nseg_l = pattern->nseg[0];
  a.nseg_u = pattern->nseg[1];
  a.wseg_l = pattern->wseg[0];
  a.wseg_u = pattern->wseg[1];
  a.one_l = pattern->one_seg[0];
  a.one_u = pattern->one_seg[1];
  a.noff = pattern->noff;
  a.ilu64 = pattern->d_base;
  a.ilu64_records = pattern->ilu64_records;
  a.b = b;
  a.x = x;
  a.iters = iters;
  a.resid = resid;
  a.status = status;
  a.outer = opts ? opts->outer_iters : nullptr;
  a.sink = bs::device_sink();
  if (!a.sink) return BS_ERR_HIP;
  // Slots without an entry read a system's first value and drop it; where no
  // system has one they read the sink instead.
  a.values = stored > 0 ? values : reinterpret_cast<const double*>(a.sink);
  a.x_alt = opts ? opts->x_alt : nullptr;
  a.alt_used = opts ? opts->alt_used : nullptr;
  if (a.x_alt && (flags & BS_FLAG_X0_ZERO)) return BS_ERR_INVALID_ARG;
  if (streamed) {
    a.layout = nullptr;
    a.block = 0;
    const int cus = bs::device_cus();
    if (cus < 1) return BS_ERR_HIP;
    const int mixed = opts && opts->precision == BS_MIXED;
    const int src = bs::stream_launch(a, pl.info, solver, mixed, cus, (hipStream_t)stream);
    return src == BS_OK ? BS_OK : hip_fail(hipGetLastError(), "streamed solver launch");
  }
  a.layout = (pattern->d_layout && pl.info.team == bs::kWave && pl.info.rows_per_lane == 1 &&
              a.window && pl.k->nz == pattern->layout_nz && !(flags & BS_FLAG_PLAIN_LAYOUT) &&
              a.block <= 1 && !ilu && !trsv)  // these need row i on lane i
                 ? pattern->d_layout
                 : nullptr;
  // Persistent grid: as many workgroups as can be resident at once, each
  // walking over the batch (never more than there are systems).
  const int64_t groups = (n_solves + pl.info.systems_per_group - 1) / pl.info.systems_per_group;
  const int cus = bs::device_cus();
  if (cus < 1) return BS_ERR_HIP;
  // Resident groups per CU, asked with 1 KiB more LDS per group than used: a
  // group count that would fill the CU's LDS to the last granule is not always
  // placed at once, and a group left over runs only after another one ends.
  int lds = pl.info.lds_bytes;
  // the group-wide copy lands in whole KiB behind the vectors: inside the launch's LDS
  if (a.stage == 2 && (a.stage_vals_bytes % 1024 != 0 || a.stage_offset + a.stage_vals_bytes > lds))
    return BS_ERR_UNSUPPORTED;
  // The group-wide copy of the values only where no group is lost to it; rows of
  // more than 56 slots keep it at that price: lanes that read such rows from
  // memory touch a line each and load (967 systems of 250 rows, 62 entries each, two
  // groups without the copy and one with it: BiCGSTAB 207 and 137 us, CG 196 and
  // 121; 2016 of 120 rows, four and two: 179 and 132).
  if (a.stage == 2 && pl.k->nz <= 56) {
    const int without = lds - a.stage_vals_bytes;
    if (pl.k->occupancy((unsigned)lds + 1024) < pl.k->occupancy((unsigned)without + 1024)) {
      a.stage = 0;
      lds = without;
    }
  }
  // A call of no more groups than compute units has them all resident whatever
  // the runtime's occupancy query would say (its cost is a fraction of a
  // microsecond, within the noise of a small call of 18 us).
  const int64_t resident =
      groups <= cus ? groups : (int64_t)pl.k->occupancy((unsigned)lds + 1024) * cus;
  const int64_t grid = std::min(groups, resident);
  const hipError_t e = pl.k->launch(a, (unsigned)grid, (unsigned)lds, (hipStream_t)stream);
  return e == hipSuccess ? BS_OK : hip_fail(e, "solver launch");
}

}  // extern "C"

namespace {
// Patterns of bs_batch_solve_dev, keyed by what identifies the caller's arrays.
struct DevPatKey {
  int device, fmt, n, nnz, width;
  const void* rp;
  const void* ci;
  int32_t generation;
  bool operator==(const DevPatKey& o) const {
    return device == o.device && fmt == o.fmt && n == o.n && nnz == o.nnz && width == o.width &&
           rp == o.rp && ci == o.ci && generation == o.generation;
  }
};
struct DevPatEntry {
  DevPatKey key;
  bs_pattern pattern = nullptr;
  uint64_t used = 0;
};
std::mutex g_dp_mu;
std::vector<DevPatEntry> g_dp_cache;
uint64_t g_dp_clock = 0;
constexpr size_t kDevPatEntries = 8;

int read_ints(std::vector<int32_t>& dst, const int32_t* src, int64_t count, hipStream_t st) {
  dst.resize((size_t)std::max<int64_t>(count, 0));
  if (count <= 0) return BS_OK;
  hipError_t e = hipMemcpyAsync(dst.data(), src, (size_t)count * sizeof(int32_t),
                                hipMemcpyDeviceToHost, st);
  if (e == hipSuccess) e = hipStreamSynchronize(st);
  return e == hipSuccess ? BS_OK : hip_fail(e, "read pattern arrays");
}
}  // namespace

extern "C" {

int bs_batch_solve_dev(bs_format fmt, int64_t n_batch, int32_t n_rows,
                       const bs_pattern_dev* pattern, const double* values, const double* b,
                       double* x, bs_solver solver, bs_precond precond, double tol,
                       int32_t max_iter, int32_t* iters, double* resid, int32_t* status,
                       const bs_options* opts, void* workspace, size_t workspace_bytes,
                       void* stream) {
  (void)workspace;  // the solve needs none (bs_workspace_size returns 0)
  (void)workspace_bytes;
  if (n_batch < 0 || n_rows < 1) return BS_ERR_INVALID_ARG;
  if (fmt != BS_CSR && fmt != BS_ELL && fmt != BS_DENSE) return BS_ERR_INVALID_ARG;
  DevPatKey key{};
  key.fmt = fmt;
  key.n = n_rows;
  key.generation = opts ? opts->structure_generation : 0;
  if (fmt != BS_DENSE) {
    if (!pattern) return BS_ERR_INVALID_ARG;
    if (fmt == BS_CSR && (!pattern->row_ptr || pattern->nnz < 0 || (pattern->nnz > 0 && !pattern->col_idx)))
      return BS_ERR_INVALID_ARG;
    if (fmt == BS_ELL && (pattern->ell_width < 0 ||
                          (int64_t)pattern->nnz != (int64_t)pattern->ell_width * n_rows ||
                          (pattern->ell_width > 0 && !pattern->col_idx)))
      return BS_ERR_INVALID_ARG;
    key.nnz = pattern->nnz;
    key.width = fmt == BS_ELL ? pattern->ell_width : 0;
    key.rp = fmt == BS_CSR ? pattern->row_ptr : nullptr;
    key.ci = pattern->col_idx;
  }
  if (n_batch == 0) return BS_OK;
  int count = 0;
  if (hipGetDeviceCount(&count) != hipSuccess || count < 1) {
    (void)hipGetLastError();
    g_last_error = "no HIP device";
    return BS_ERR_NO_DEVICE;
  }
  hipError_t e = hipGetDevice(&key.device);
  if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
  const hipStream_t st = (hipStream_t)stream;
  std::lock_guard<std::mutex> lock(g_dp_mu);
  DevPatEntry* ent = nullptr;
  for (DevPatEntry& d : g_dp_cache)
    if (d.key == key) ent = &d;
  if (!ent) {
    bs_pattern p = nullptr;
    int rc = BS_OK;
    if (fmt == BS_DENSE) {
      rc = bs_pattern_create_dense(n_rows, &p);
    } else if (fmt == BS_CSR) {
      std::vector<int32_t> rp, ci;
      rc = read_ints(rp, pattern->row_ptr, (int64_t)n_rows + 1, st);
      if (rc == BS_OK) rc = read_ints(ci, pattern->col_idx, pattern->nnz, st);
      if (rc == BS_OK) rc = bs_pattern_create_csr(n_rows, pattern->nnz, rp.data(), ci.data(), &p);
    } else {
      std::vector<int32_t> ci;
      rc = read_ints(ci, pattern->col_idx, (int64_t)pattern->ell_width * n_rows, st);
      if (rc == BS_OK) rc = bs_pattern_create_ell(n_rows, pattern->ell_width, ci.data(), &p);
    }
    if (rc != BS_OK) return rc;
    if (g_dp_cache.size() >= kDevPatEntries) {  // drop the least recently used
      size_t lru = 0;
      for (size_t i = 1; i < g_dp_cache.size(); ++i)
        if (g_dp_cache[i].used < g_dp_cache[lru].used) lru = i;
      (void)bs_pattern_destroy(g_dp_cache[lru].pattern);
      g_dp_cache.erase(g_dp_cache.begin() + (long)lru);
    }
    DevPatEntry fresh;
    fresh.key = key;
    fresh.pattern = p;
    g_dp_cache.push_back(fresh);
    ent = &g_dp_cache.back();
  }
  ent->used = ++g_dp_clock;
  return bs_batch_solve(fmt, n_batch, n_rows, ent->pattern, values, b, x, solver, precond, tol,
                        max_iter, iters, resid, status, opts, stream);
}

}  // extern "C"
