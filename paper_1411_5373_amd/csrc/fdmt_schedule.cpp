// Pass schedule of the fused FDMT (host).
//
// A pass fuses iterations l0+1 .. l1. Its work item ("block") is a range of
// consecutive rows of one sub-band of plane l1 over one time tile
// [T0, T0 + W). Walking the delay tables down from the block gives, at every
// fused iteration, the rows each sub-band must supply: because d_lo, d_hi and
// s are non-decreasing in dt, they are the contiguous range between the
// children of the block's first and last rows. The lower half is read at the
// same times as its parent; the upper half t - s back, so its time window is
// the parent's widened by the spread of s over the block.
#include "fdmt_schedule.h"

#include <algorithm>
#include <array>

namespace fdmt {

namespace {

struct Tree {
  std::vector<Node> nodes;  // level by level, leaves first
  int need[2] = {0, 0};     // elements of LDS buffers A (even levels) and B (odd levels)
};

// Builds the tree of a block and its LDS layout; levels i = 0..k of the pass.
Tree build_tree(const Tables &t, bool from_input, int l0, int l1, int sub, int r0, int nr, int tile) {
  const int k = l1 - l0;
  Tree tr;
  tr.nodes.resize((size_t(2) << k) - 1);
  // the 2^(k-i) nodes of level i
  const auto level = [&](int i) { return tr.nodes.data() + ((2 << k) - (2 << (k - i))); };
  *level(k) = Node{static_cast<int32_t>(t.row_off[l1][sub] + r0), nr, 0, tile, 0, sub, 0, 0};
  for (int i = k; i >= 1; --i) {
    const int l = l0 + i;
    for (int j = 0; j < 1 << (k - i); ++j) {
      const Node &n = level(i)[j];
      const MergeRow &a = t.merge[l][n.row0];
      const MergeRow &b = t.merge[l][n.row0 + n.nrows - 1];
      level(i - 1)[2 * j] = Node{a.lo, b.lo - a.lo + 1, n.win, n.width, 0, 2 * n.sub, 0, 0};
      level(i - 1)[2 * j + 1] =
          Node{a.hi, b.hi - a.hi + 1, n.win + b.s, n.width + (b.s - a.s), 0, 2 * n.sub + 1, 0, 0};
    }
  }
  if (from_input) {
    // Leaves become staged input rows: the Option-1 chain of partial-sum row d
    // reads d samples further back, so the window grows by the largest d.
    for (int j = 0; j < 1 << k; ++j) {
      Node &n = level(0)[j];
      const int ch = n.sub;
      const int d_last = n.row0 + n.nrows - 1 - t.leaf_off[ch];
      n.win += d_last;
      n.width += d_last;
      n.row0 = t.leaf_off[ch];
      n.nrows = 1;
    }
  }
  for (int i = 0; i <= k; ++i) {
    int off = 0, cum = 0;
    for (int j = 0; j < 1 << (k - i); ++j) {
      Node &n = level(i)[j];
      n.lds = i < k ? off : 0;
      n.rowcum = cum;
      off += n.nrows * n.width;
      cum += n.nrows;
    }
    if (i < k) tr.need[i & 1] = std::max(tr.need[i & 1], off);
  }
  return tr;
}

// Checks, for every block, that each merge reads only rows its children hold
// and only columns inside their windows, and that every node fits its LDS
// buffer: the bounds the fused kernel relies on.
std::string audit_pass(const Tables &t, const Pass &ps, const Node *nodes) {
  const int k = ps.l1 - ps.l0;
  for (int b = 0; b < ps.nblocks; ++b) {
    const Node *nd = nodes + static_cast<int64_t>(b) * ps.nodes_per_block;
    int base = 0;
    std::vector<int> level_base(k + 2);
    for (int i = 0; i <= k; ++i) {
      level_base[i] = base;
      base += 1 << (k - i);
    }
    level_base[k + 1] = base;
    for (int i = 0; i < k; ++i) {
      const int cap = (i & 1) ? ps.lds_b : ps.lds_a;
      for (int j = level_base[i]; j < level_base[i + 1]; ++j)
        if (nd[j].lds < 0 || nd[j].lds + static_cast<int64_t>(nd[j].nrows) * nd[j].width > cap)
          return "node outside its LDS buffer";
    }
    const Node &top = nd[level_base[k]];
    if (top.win != 0 || top.width != ps.tile) return "top node window";
    for (int i = 1; i <= k; ++i) {
      const int l = ps.l0 + i;
      for (int j = level_base[i]; j < level_base[i + 1]; ++j) {
        const Node &n = nd[j];
        const Node &lo = nd[level_base[i - 1] + 2 * (j - level_base[i])];
        const Node &hi = nd[level_base[i - 1] + 2 * (j - level_base[i]) + 1];
        if (n.row0 < 0 || n.row0 + n.nrows > t.total[l]) return "node rows outside plane";
        for (int r = 0; r < n.nrows; ++r) {
          const MergeRow &m = t.merge[l][n.row0 + r];
          const int dl = m.lo - lo.row0, dh = m.hi - hi.row0;
          if (ps.from_input && i == 1) {
            // chain over the staged input row: columns c + lo.win - n.win - d, d <= dl
            if (dl < 0 || dh < 0) return "partial-sum row below the channel";
            if (lo.win - n.win - dl < 0 || n.width - 1 + lo.win - n.win > lo.width - 1)
              return "lower input window";
            if (hi.win - n.win - m.s - dh < 0 || n.width - 1 - m.s + hi.win - n.win > hi.width - 1)
              return "upper input window";
            if (t.leaf_rows[lo.sub] <= dl || t.leaf_rows[hi.sub] <= dh) return "partial-sum row";
          } else {
            if (dl < 0 || dl >= lo.nrows || dh < 0 || dh >= hi.nrows) return "child row outside node";
            if (lo.win != n.win || lo.width < n.width) return "lower window";
            if (hi.win - n.win - m.s < 0 || n.width - 1 - m.s + hi.win - n.win > hi.width - 1)
              return "upper window";
          }
        }
      }
    }
  }
  return "";
}

// Flattens a block's tree into kernel records (see Rec).
void emit_records(const Tables &t, bool from_input, int l0, int k, const Node *nd,
                  std::vector<Rec> &recs, int32_t *head) {
  std::vector<int> level_base(k + 2);
  int base = 0;
  for (int i = 0; i <= k; ++i) {
    level_base[i] = base;
    base += 1 << (k - i);
  }
  level_base[k + 1] = base;
  const int32_t first = static_cast<int32_t>(recs.size());
  head[0] = first;
  for (int j = level_base[0]; j < level_base[1]; ++j) {
    const Node &n = nd[j];
    for (int r = 0; r < n.nrows; ++r)
      recs.push_back(Rec{from_input ? n.sub : n.row0 + r, 0, n.lds + r * n.width, n.win, n.width, 0, 0, 0});
  }
  head[1] = static_cast<int32_t>(recs.size()) - first;
  for (int i = 1; i <= k; ++i) {
    const int l = l0 + i;
    for (int j = level_base[i]; j < level_base[i + 1]; ++j) {
      const Node &n = nd[j];
      const Node &lo = nd[level_base[i - 1] + 2 * (j - level_base[i])];
      const Node &hi = nd[level_base[i - 1] + 2 * (j - level_base[i]) + 1];
      for (int r = 0; r < n.nrows; ++r) {
        const MergeRow &m = t.merge[l][n.row0 + r];
        Rec e{};
        if (from_input && i == 1) {
          e.a = lo.lds + (lo.win - n.win);
          e.b = hi.lds + (hi.win - n.win) - m.s;
          e.g = m.lo - lo.row0;
          e.h = m.hi - hi.row0;
        } else {
          e.a = lo.lds + (m.lo - lo.row0) * lo.width + (lo.win - n.win);
          e.b = hi.lds + (m.hi - hi.row0) * hi.width + (hi.win - n.win) - m.s;
        }
        e.c = i == k ? n.row0 + r : n.lds + r * n.width;
        e.d = m.s + n.win;
        e.e = n.width;
        e.f = n.win;
        recs.push_back(e);
      }
    }
    head[1 + i] = static_cast<int32_t>(recs.size()) - first;
  }
}

// Bounds of every record as the kernel will use it: LDS reads and writes
// inside their buffers, source rows inside the consumed plane (or channel
// range), destination rows inside the produced plane.
std::string audit_records(const Tables &t, const Pass &ps, const Rec *recs, const int32_t *heads) {
  const int k = ps.l1 - ps.l0;
  const int64_t src_rows = ps.from_input ? t.slots : t.total[ps.l0];
  for (int b = 0; b < ps.nblocks; ++b) {
    const int32_t *h = heads + static_cast<int64_t>(b) * kRecHeader;
    const Rec *r = recs + h[0];
    if (h[1 + k] > ps.max_recs) return "record count";
    for (int q = 0; q < h[1]; ++q) {
      if (r[q].a < 0 || r[q].a >= src_rows) return "staged row outside source";
      if (r[q].c < 0 || r[q].c + r[q].e > ps.lds_a || r[q].e < 1) return "staged row outside LDS";
    }
    for (int i = 1; i <= k; ++i) {
      const int64_t src_cap = (i & 1) ? ps.lds_a : ps.lds_b;  // level i-1 buffer
      const int64_t dst_cap = (i & 1) ? ps.lds_b : ps.lds_a;
      for (int q = h[i]; q < h[1 + i]; ++q) {
        const Rec &e = r[q];
        const int back_lo = (ps.from_input && i == 1) ? e.g : 0;
        const int back_hi = (ps.from_input && i == 1) ? e.h : 0;
        if (e.e < 1 || e.a - back_lo < 0 || e.a + e.e > src_cap) return "lower operand outside LDS";
        if (e.b - back_hi < 0 || e.b + e.e > src_cap) return "upper operand outside LDS";
        if (i == k) {
          if (e.c < 0 || e.c >= t.total[ps.l1] || e.e != ps.tile) return "top row";
        } else if (e.c < 0 || e.c + e.e > dst_cap) {
          return "merged row outside LDS";
        }
      }
    }
  }
  return "";
}

// Staged pass layout of one block. Leaves are packed in LDS with row
// strides padded to 4 elements. In the first pass a leaf is one staged input
// row per channel plus, after all of them, the channel's Option-1 partial-sum
// rows 0 .. d_last computed from it in LDS.
struct StagedLayout {
  int64_t stage_elems = 0;  // staged rows (input or plane rows)
  int64_t psum_elems = 0;   // partial-sum rows (first pass)
  std::vector<int> psum_lds;
};

StagedLayout staged_layout(const Tables &t, bool from_input, std::vector<Node> &leaves,
                           const std::vector<Node> &generic) {
  StagedLayout lay;
  int64_t off = 0;
  for (Node &n : leaves) {
    n.lds = static_cast<int32_t>(off);
    off += static_cast<int64_t>(n.nrows) * ((n.width + 3) / 4 * 4);
  }
  lay.stage_elems = off;
  if (from_input) {
    for (size_t j = 0; j < leaves.size(); ++j) {
      const Node &g = generic[j];  // partial-sum rows and window before widening
      const int d_last = g.row0 + g.nrows - 1 - t.leaf_off[g.sub];
      lay.psum_lds.push_back(static_cast<int>(off));
      off += static_cast<int64_t>(d_last + 1) * ((g.width + 3) / 4 * 4);
    }
    lay.psum_elems = off - lay.stage_elems;
  }
  return lay;
}

// Emits the staging records, partial-sum records, terms and header of one
// staged block and checks every LDS access the kernel will make for it.
std::string emit_staged(const Tables &t, bool from_input, int l0, int l1, int sub, int r0, int nr,
                        int tile, const std::vector<Node> &leaves, const std::vector<Node> &generic,
                        const StagedLayout &lay, Schedule &s, const Pass &ps) {
  const int k = l1 - l0;
  const int n_terms = 1 << k;
  const int64_t lds_total = lay.stage_elems + lay.psum_elems;
  int32_t head[kStagedHeader] = {};
  head[0] = static_cast<int32_t>(s.stage.size() - ps.rec_offset);
  int max_w4 = 0;
  for (const Node &n : leaves) {
    const int w4 = (n.width + 3) / 4 * 4;
    max_w4 = std::max(max_w4, w4);
    for (int r = 0; r < n.nrows; ++r) {
      if (n.lds + static_cast<int64_t>(r + 1) * w4 > lay.stage_elems) return "staged row outside LDS";
      s.stage.push_back(Rec{from_input ? n.sub : n.row0 + r, 0, n.lds + r * w4, n.win, w4, 0, 0, 0});
    }
  }
  head[1] = static_cast<int32_t>(s.stage.size() - ps.rec_offset) - head[0];
  head[2] = static_cast<int32_t>(s.sterms.size() - ps.term_offset);
  head[3] = nr;
  head[4] = static_cast<int32_t>(t.row_off[l1][sub] + r0);
  const int qpr = max_w4 / 4;  // quads per staged row
  head[5] = qpr;
  head[6] = static_cast<int32_t>((0x100000000ull + qpr - 1) / qpr);  // ceil(2^32 / qpr)
  if (static_cast<int64_t>(head[1]) * qpr >= 65536) return "staged block too large";
  head[7] = static_cast<int32_t>(s.psums.size() - ps.psum_offset);
  head[8] = from_input ? static_cast<int32_t>(leaves.size()) : 0;
  if (from_input) {
    for (size_t j = 0; j < leaves.size(); ++j) {
      const Node &x = leaves[j], &g = generic[j];
      const int d_last = g.row0 + g.nrows - 1 - t.leaf_off[g.sub];
      const int w4 = (g.width + 3) / 4 * 4;
      // input column of time T0 - g.win + c is c + (x.win - g.win); the chain
      // reads d_last samples back from there
      const int ahead = x.win - g.win;
      if (ahead != d_last || x.width != g.width + d_last) return "partial-sum window";
      if (lay.psum_lds[j] + static_cast<int64_t>(d_last + 1) * w4 > lds_total) return "partial sums outside LDS";
      s.psums.push_back(Rec{lay.psum_lds[j], x.lds, d_last, w4, g.width, ahead, 0, 0});
    }
  }
  std::vector<Term> cur, nxt;
  for (int r = 0; r < nr; ++r) {
    cur.assign(1, Term{static_cast<int32_t>(t.row_off[l1][sub] + r0 + r), 0});
    for (int l = l1; l > l0; --l) {
      nxt.clear();
      for (const Term &x : cur) {
        const MergeRow &m = t.merge[l][x.row];
        nxt.push_back(Term{m.lo, x.shift});
        nxt.push_back(Term{m.hi, x.shift + m.s});
      }
      cur.swap(nxt);
    }
    for (int j = 0; j < n_terms; ++j) {
      StagedTerm st{};
      int64_t row_start, row_end;
      int col0;
      if (from_input) {
        const Node &g = generic[j];
        const int d = cur[j].row - t.leaf_off[g.sub];  // partial-sum row of the channel
        const int d_last = g.row0 + g.nrows - 1 - t.leaf_off[g.sub];
        if (d < 0 || d > d_last) return "partial-sum row of a term";
        const int w4 = (g.width + 3) / 4 * 4;
        col0 = g.win - cur[j].shift;
        if (col0 < 0 || col0 + tile > g.width) return "partial-sum term window";
        row_start = lay.psum_lds[j] + static_cast<int64_t>(d) * w4;
        row_end = row_start + w4;
      } else {
        const Node &n = leaves[j];
        const int w4 = (n.width + 3) / 4 * 4;
        const int rl = cur[j].row - n.row0;
        if (rl < 0 || rl >= n.nrows) return "staged term row outside leaf";
        col0 = n.win - cur[j].shift;  // column of time T0 - sigma
        if (col0 < 0 || col0 + tile > n.width) return "staged term window";
        row_start = n.lds + static_cast<int64_t>(rl) * w4;
        row_end = row_start + w4;
      }
      st.lds = static_cast<int32_t>(row_start + col0);
      if (row_start < 0 || row_end > lds_total || st.lds + tile > row_end) return "staged term outside LDS";
      s.sterms.push_back(st);
    }
  }
  s.sheads.insert(s.sheads.end(), head, head + kStagedHeader);
  return "";
}

} // namespace

// Builds one pass of k iterations starting at plane l0 and appends it.
std::string build_pass(Schedule &s, const Tables &t, const ScheduleParams &p, int l0, int k_req,
                       bool from_input) {
  const int L = t.levels;
  const int64_t budget = p.lds_bytes / p.acc_bytes;
  {
    const bool first = from_input;
    const PassKind kind = first ? p.first_kind : p.later_kind;
    // The d_min pre-shift enters through the input terms of a register pass
    // (and the initialisation kernels); passes that stage input rows in LDS do
    // not apply it.
    if (first && kind != PassKind::Register)
      for (int k = 0; k < t.nf; ++k)
        if (t.pre[k] != 0) return "the d_min pre-shift needs the first pass to gather from the input";
    if (kind == PassKind::Staged) {
      const int k = std::min(k_req, L - l0);
      // five would hold 32 terms of 4 runs per thread: past the register
      // budget of its workgroup (it spilled)
      if (k > 4) return "at most 4 iterations per staged pass";
      if (p.tile % 256 != 0) return "staged passes need a tile that is a multiple of 256";
      Pass ps;
      ps.kind = PassKind::Staged;
      ps.from_input = first;
      ps.l0 = l0;
      ps.l1 = l0 + k;
      ps.tile = p.tile;
      ps.rows_in = first ? t.slots : t.total[l0];
      ps.rows_out = t.total[ps.l1];
      ps.rec_offset = static_cast<int64_t>(s.stage.size());
      ps.term_offset = static_cast<int64_t>(s.sterms.size());
      ps.head_offset = static_cast<int64_t>(s.sheads.size());
      ps.psum_offset = static_cast<int64_t>(s.psums.size());
      int max_stage = 0, max_rows = 0;
      int64_t leaf_max = 0, psum_max = 0;
      for (int sub = 0; sub < (t.slots >> ps.l1); ++sub) {
        const int n = t.rows[ps.l1][sub];
        int r0 = 0;
        while (r0 < n) {
          int nr = std::min(p.max_block_rows, n - r0);
          std::vector<Node> leaves, generic;
          StagedLayout lay;
          int nstage = 0;
          for (;;) {
            Tree tr = build_tree(t, first, l0, ps.l1, sub, r0, nr, p.tile);
            leaves.assign(tr.nodes.begin(), tr.nodes.begin() + (1 << k));
            if (first) {
              Tree g = build_tree(t, false, l0, ps.l1, sub, r0, nr, p.tile);
              generic.assign(g.nodes.begin(), g.nodes.begin() + (1 << k));
            }
            lay = staged_layout(t, first, leaves, generic);
            nstage = 0;
            for (const Node &x : leaves) nstage += x.nrows;
            // LDS: leaves, partial sums, staging records (4 ints each),
            // partial-sum records (4 ints per channel), terms (2 ints each)
            int max_w4 = 0;
            for (const Node &x : leaves) max_w4 = std::max(max_w4, (x.width + 3) / 4 * 4);
            const int64_t quads = static_cast<int64_t>(nstage) * (max_w4 / 4);
            const int64_t need = lay.stage_elems + lay.psum_elems + 4LL * nstage +
                                 (first ? 8LL * (1 << k) : 0) + 2LL * nr * (1 << k);
            if (need <= budget && quads <= kMaxStagedQuads) break;
            if (nr == 1) return "LDS budget too small for one row of pass " + std::to_string(l0);
            nr = std::max(1, nr * 3 / 4);
          }
          ps.staged_rows += nstage;
          const std::string err =
              emit_staged(t, first, l0, ps.l1, sub, r0, nr, p.tile, leaves, generic, lay, s, ps);
          if (!err.empty()) return "audit of pass " + std::to_string(l0) + ": " + err;
          leaf_max = std::max(leaf_max, lay.stage_elems);
          psum_max = std::max(psum_max, lay.psum_elems);
          max_stage = std::max(max_stage, nstage);
          max_rows = std::max(max_rows, nr);
          ++ps.nblocks;
          r0 += nr;
        }
      }
      // LDS areas (4-byte units): staged rows | partial sums | staging records |
      // partial-sum records | terms. Partial-sum offsets are relative to the
      // start of LDS, so the partial-sum area follows the largest staged area.
      ps.lds_a = static_cast<int>((leaf_max + 3) / 4 * 4);
      ps.lds_p = static_cast<int>((psum_max + 3) / 4 * 4);
      ps.stage_ints = 4 * max_stage;
      ps.lds_b = ps.stage_ints + (first ? 8 * (1 << k) : 0);
      ps.max_recs = 2 * max_rows * (1 << k);
      s.passes.push_back(ps);
      return "";
    }
    if (kind == PassKind::Register) {
      // Iterations as register gathers: walking the tables down from each
      // output row gives its 2^k (row, shift) terms of plane l0, in the order
      // the recursion adds them (lower half before upper half). From the
      // input, a plane-0 term is channel ch's Option-1 partial-sum row d:
      // the chain of input samples at shifts sigma .. sigma + d.
      const int k = std::min(k_req, L - l0);
      if (k > 4) return "at most 4 iterations per register pass";
      Pass ps;
      ps.gather = true;
      ps.kind = PassKind::Register;
      ps.from_input = first;
      ps.l0 = l0;
      ps.l1 = l0 + k;
      ps.rows_in = first ? t.slots : t.total[l0];
      ps.rows_out = t.total[ps.l1];
      ps.term_offset = static_cast<int64_t>(first ? s.iterms.size() : s.terms.size());
      std::vector<int32_t> channel_of;
      if (first) {
        channel_of.resize(t.total[0]);
        for (int ch = 0; ch < t.slots; ++ch)
          for (int d = 0; d < t.leaf_rows[ch]; ++d) channel_of[t.leaf_off[ch] + d] = ch;
      }
      std::vector<Term> cur, nxt;
      for (int64_t r = 0; r < ps.rows_out; ++r) {
        cur.assign(1, Term{static_cast<int32_t>(r), 0});
        for (int l = ps.l1; l > l0; --l) {
          nxt.clear();
          for (const Term &x : cur) {
            const MergeRow &m = t.merge[l][x.row];
            nxt.push_back(Term{m.lo, x.shift});
            nxt.push_back(Term{m.hi, x.shift + m.s});
          }
          cur.swap(nxt);
        }
        for (const Term &x : cur)
          if (x.row < 0 || x.row >= t.total[l0] || x.shift < 0) return "gather term out of range";
        if (first) {
          for (const Term &x : cur) {
            const int ch = channel_of[x.row];
            const int d = x.row - t.leaf_off[ch];
            // a position without a channel reads a zero row of the padded input
            s.iterms.push_back(InTerm{ch, x.shift + (ch < t.nf ? t.pre[ch] : 0), d, 0});
            ps.staged_rows += d + 1;
            ps.max_chain = std::max(ps.max_chain, d);
          }
        } else {
          s.terms.insert(s.terms.end(), cur.begin(), cur.end());
          ps.staged_rows += static_cast<int64_t>(cur.size());
        }
      }
      ps.nblocks = static_cast<int>(ps.rows_out);
      s.passes.push_back(ps);
      return "";
    }
    const int k = std::min(k_req, L - l0);
    if (k > 8) return "at most 8 iterations per pass";
    Pass ps;
    ps.kind = PassKind::Recursive;
    ps.from_input = first;
    ps.l0 = l0;
    ps.l1 = l0 + k;
    ps.tile = p.tile;
    ps.nodes_per_block = (1 << (k + 1)) - 1;
    ps.node_offset = static_cast<int64_t>(s.nodes.size());
    ps.rec_offset = static_cast<int64_t>(s.recs.size());
    ps.head_offset = static_cast<int64_t>(s.heads.size());
    ps.rows_in = first ? t.slots : t.total[l0];
    ps.rows_out = t.total[ps.l1];
    for (int sub = 0; sub < (t.slots >> ps.l1); ++sub) {
      const int n = t.rows[ps.l1][sub];
      int r0 = 0;
      while (r0 < n) {
        int nr = std::min(p.max_block_rows, n - r0);
        Tree tr;  // level-by-level LDS pass
        for (;;) {
          tr = build_tree(t, first, l0, ps.l1, sub, r0, nr, p.tile);
          if (tr.need[0] + tr.need[1] + 2 * kLdsSlack <= budget) break;
          if (nr == 1) return "LDS budget too small for one row of pass " + std::to_string(l0);
          nr = std::max(1, nr * 3 / 4);
        }
        ps.lds_a = std::max(ps.lds_a, tr.need[0]);
        ps.lds_b = std::max(ps.lds_b, tr.need[1]);
        for (int j = 0; j < (1 << k); ++j) ps.staged_rows += tr.nodes[j].nrows;
        s.nodes.insert(s.nodes.end(), tr.nodes.begin(), tr.nodes.end());
        int32_t head[kRecHeader] = {};
        const size_t before = s.recs.size();
        emit_records(t, first, l0, k, tr.nodes.data(), s.recs, head);
        head[0] -= static_cast<int32_t>(ps.rec_offset);
        ps.max_recs = std::max(ps.max_recs, static_cast<int>(s.recs.size() - before));
        s.heads.insert(s.heads.end(), head, head + kRecHeader);
        ++ps.nblocks;
        r0 += nr;
      }
    }
    ps.lds_a = (ps.lds_a + 3) / 4 * 4;  // keeps the record area 16-byte aligned
    ps.lds_b = (ps.lds_b + 3) / 4 * 4;
    std::string err = audit_pass(t, ps, s.nodes.data() + ps.node_offset);
    if (err.empty())
      err = audit_records(t, ps, s.recs.data() + ps.rec_offset, s.heads.data() + ps.head_offset);
    if (!err.empty()) return "audit of pass " + std::to_string(l0) + ": " + err;
    s.passes.push_back(ps);
  }
  return "";
}

std::string build_schedule(Schedule &s, const Tables &t, const ScheduleParams &p) {
  s = Schedule();
  const int L = t.levels;
  if (L == 0) return "";
  if (p.tile < 1 || p.first_levels < 1 || p.later_levels < 1) return "bad schedule parameters";
  int l0 = 0;
  while (l0 < L) {
    const bool first = l0 == 0 && !s.init_separate;
    const bool automatic = first ? p.first_auto : p.later_auto;
    int k = std::min(first ? p.first_levels : p.later_levels, L - l0);
    for (;;) {
      // Remember the sizes so a pass that does not fit can be taken back.
      const size_t n_nodes = s.nodes.size(), n_recs = s.recs.size(), n_heads = s.heads.size(),
                   n_terms = s.terms.size(), n_iterms = s.iterms.size(), n_sterms = s.sterms.size(),
                   n_stage = s.stage.size(),
                   n_psums = s.psums.size(), n_sheads = s.sheads.size();
      const std::string err = build_pass(s, t, p, l0, k, first);
      if (err.empty()) break;
      s.nodes.resize(n_nodes);
      s.recs.resize(n_recs);
      s.heads.resize(n_heads);
      s.terms.resize(n_terms);
      s.iterms.resize(n_iterms);
      s.sterms.resize(n_sterms);
      s.stage.resize(n_stage);
      s.psums.resize(n_psums);
      s.sheads.resize(n_sheads);
      const bool too_big = err.find("LDS budget too small") != std::string::npos ||
                           err.find("at most") != std::string::npos;
      if (!automatic || !too_big) return err;
      if (k == 1) {
        // Not even one fused iteration fits: run the Option-1 initialisation
        // as its own step (writing plane 0) and fuse from plane 0 on.
        if (!first) return err;
        s.init_separate = true;
        break;
      }
      --k;
    }
    if (!s.passes.empty()) l0 = s.passes.back().l1;
  }
  return "";
}

namespace {

// Ranges of at most `most` rows that a sub-band's n rows are split into, one of
// `subs` sub-bands: with few sub-bands as many as make the blocks a multiple of
// the 8 XCDs, so that a range of blocks stays on its XCD from one time tile to
// the next (57 blocks instead of 64 made a pass 12% slower).
int row_parts(int n, int most, int subs) {
  const int parts = (n + most - 1) / most;
  const int step = subs >= 8 ? 1 : 8 / subs;
  return parts < step ? parts : (parts + step - 1) / step * step;
}

// How a block pass of k iterations splits over its stages: two iterations
// loaded through the caches, at most three from LDS at a time (five iterations
// of 32-bit sums as 2 + 1 + 2 were 9% slower than as 2 + 3).
struct BlockSplit {
  int k1, k2, k3;
};
BlockSplit block_split(int k, bool packed) {
  switch (k) {
    case 3: return {1, 0, 2};
    case 4: return {2, 0, 2};
    case 5: return packed ? BlockSplit{2, 1, 2} : BlockSplit{2, 0, 3};
    default: return {2, 2, 2};
  }
}

// The 2^k terms (k <= 3) of row `row` of plane l, k iterations down, in the
// order the recursion adds them.
void walk_terms(const Tables &t, int l, int k, int64_t row, Term (&out)[8]) {
  out[0] = Term{static_cast<int32_t>(row), 0};
  for (int i = 0; i < k; ++i, --l)
    for (int j = (1 << i) - 1; j >= 0; --j) {
      const Term x = out[j];
      const MergeRow &m = t.merge[l][x.row];
      out[2 * j] = Term{m.lo, x.shift};
      out[2 * j + 1] = Term{m.hi, x.shift + m.s};
    }
}

// LDS offsets of the rows of `tops` (nodes k levels above `leaves`, which lie
// in LDS from row base[i] on): appended to offs, in row order.
std::string block_offsets(const Tables &t, int l, int k, const Node *tops, int ntops, const Node *leaves,
                          const std::vector<int> &base, int lead, const Pass &ps, std::vector<int32_t> &offs) {
  Term cur[8];
  const int terms = 1 << k;
  for (int j = 0; j < ntops; ++j) {
    const Node &n = tops[j];
    for (int r = 0; r < n.nrows; ++r) {
      walk_terms(t, l, k, n.row0 + r, cur);
      for (int q = 0; q < terms; ++q) {
        const int i = j * terms + q;
        const Node &x = leaves[i];
        const int rl = cur[q].row - x.row0;
        if (rl < 0 || rl >= x.nrows) return "block term row outside its node";
        const int col = lead + x.win - n.win - cur[q].shift;  // column of the top row's first sample
        if (col < lead || col + n.width > lead + x.width ||
            lead + x.width + ps.tile > ps.pitch - (ps.packed ? 2 : 1) * kBlockTail)
          return "block term window";
        offs.push_back((base[i] + rl) * ps.pitch + col);
      }
    }
  }
  return "";
}

// `many`: whole blocks, for batches of so many records that they fill the GPU.
std::string build_block_pass(Schedule &s, const Tables &t, int64_t nt, int l0, int k, bool from_input, bool bytes,
                             bool many, Pass &ps) {
  ps.kind = PassKind::Block;
  ps.from_input = from_input;
  ps.l0 = l0;
  ps.l1 = l0 + k;
  ps.rows_in = from_input ? t.slots : t.total[l0];
  ps.rows_out = t.total[ps.l1];
  ps.term_offset = static_cast<int64_t>(from_input ? s.iterms.size() : s.terms.size());
  ps.offs_offset = static_cast<int64_t>(s.block_offs.size());
  ps.head_offset = static_cast<int64_t>(s.block_heads.size());
  std::vector<int32_t> channel_of;
  if (from_input) {
    channel_of.resize(t.total[0]);
    for (int ch = 0; ch < t.slots; ++ch)
      for (int d = 0; d < t.leaf_rows[ch]; ++d) channel_of[t.leaf_off[ch] + d] = ch;
  }
  // Blocks of at most max_rows rows, each sub-band's rows split evenly.
  int max_rows = k == 6 ? 16 : 18;
  const int64_t tiles = (nt + kBlockPitch - 33) / (kBlockPitch - 32);
  const auto count_blocks = [&]() {
    int64_t n = 0;
    for (int32_t r : t.rows[ps.l1]) n += row_parts(r, max_rows, t.slots >> ps.l1);
    return n;
  };
  if (!many)
    while (max_rows > 4 && count_blocks() * tiles < 256) {
      max_rows /= 2;
      ps.few = true;
    }
  // Packed 16-bit sums: exact while 255 (2^l1 + rows - 1), the largest sum of
  // uint8 samples, fits, and worth it once the wider tiles fill the GPU.
  int widest = 0;
  for (int32_t r : t.rows[ps.l1]) widest = std::max(widest, r);
  ps.packed = from_input && bytes && 255 * ((int64_t(1) << ps.l1) + widest - 1) <= 65535 &&
              count_blocks() * ((nt + 447) / 448) >= 1024;
  ps.pitch = ps.packed ? 2 * kBlockPitch : kBlockPitch;
  const BlockSplit sp = block_split(k, ps.packed);
  ps.k1 = sp.k1;
  ps.k2 = sp.k2;
  ps.k3 = sp.k3;
  // The trees of the rows in LDS, area A's first (level 0; level i's nodes start at
  // 2^(kl+1) - 2^(kl+1-i)). A node's width with a tile of 0 samples is the spread of
  // its shifts.
  const int kl = k - ps.k1;
  struct Range {
    int sub, r0, nr;
    Tree tree;
  };
  std::vector<Range> blocks;
  blocks.reserve(count_blocks());
  int spread = 0;
  size_t lds_rows = 0;
  for (int sub = 0; sub < (t.slots >> ps.l1); ++sub) {
    const int n = t.rows[ps.l1][sub];
    const int nb = row_parts(n, max_rows, t.slots >> ps.l1);
    for (int b = 0; b < nb; ++b) {
      const int r0 = static_cast<int>(static_cast<int64_t>(n) * b / nb);
      const int r1 = static_cast<int>(static_cast<int64_t>(n) * (b + 1) / nb);
      blocks.push_back({sub, r0, r1 - r0, build_tree(t, false, l0 + ps.k1, ps.l1, sub, r0, r1 - r0, 0)});
      const Tree &tr = blocks.back().tree;
      for (const Node &x : tr.nodes) spread = std::max(spread, x.width);
      for (int j = 0; j < 1 << kl; ++j) lds_rows += tr.nodes[j].nrows;
    }
  }
  const int lead = (from_input ? kBlockLead : 0) * (ps.packed ? 2 : 1);
  ps.tile = (ps.pitch - (ps.packed ? 2 : 1) * kBlockTail - spread - lead) / 32 * 32;
  if (ps.tile < 128) return "block shifts spread too far";
  if (from_input && static_cast<int64_t>(blocks.size()) * ((nt + ps.tile - 1) / ps.tile) >= (ps.packed ? 8192 : 4096))
    ps.tiles_per_wg = 2;
  Term cur[8];
  const int terms1 = 1 << ps.k1;
  std::vector<int> base_a, base_b;
  ps.term_count = static_cast<int64_t>(lds_rows * terms1);
  if (from_input) s.iterms.resize(ps.term_offset + ps.term_count);
  else s.terms.resize(ps.term_offset + ps.term_count);
  InTerm *iterm = s.iterms.data() + ps.term_offset;  // used by a pass from the input
  Term *term = s.terms.data() + ps.term_offset;      // used by one from a plane
  int32_t terms = 0;
  for (const Range &b : blocks) {
    const auto level = [&](int i) { return b.tree.nodes.data() + ((2 << kl) - (2 << (kl - i))); };
    const auto bases = [](const Node *n, int count, std::vector<int> &base) {
      int rows = 0;
      base.resize(count);
      for (int j = 0; j < count; ++j) {
        base[j] = rows;
        rows += n[j].nrows;
      }
      return rows;
    };
    int32_t head[kBlockHeader] = {};
    head[0] = terms;
    // stage 1: the rows of area A, each term's shift counted from the row's column 0
    const Node *na = level(0);
    const int count_a = 1 << kl;
    const int rows_a = bases(na, count_a, base_a);
    int reach = 0, complete = 0;
    for (int j = 0; j < count_a; ++j) {
      // positions without a channel are the last ones, so are the nodes that have them
      const bool whole = !from_input || (na[j].sub + 1) << ps.k1 <= t.nf;
      if (whole) complete = base_a[j] + na[j].nrows;
      for (int r = 0; r < na[j].nrows; ++r) {
        walk_terms(t, l0 + ps.k1, ps.k1, na[j].row0 + r, cur);
        for (int q = 0; q < terms1; ++q) {
          const Term &x = cur[q];
          if (x.row < 0 || x.row >= t.total[l0] || x.shift < 0) return "block term out of range";
          const int shift = x.shift + na[j].win + lead;
          if (from_input) {
            const int ch = channel_of[x.row];
            const int d = x.row - t.leaf_off[ch];
            // a position without a channel: past the start of every record, so zero
            const InTerm y = ch < t.nf ? InTerm{ch, shift + t.pre[ch], d, 0} : InTerm{0, kNoChannelPre, 0, 0};
            iterm[terms++] = y;
            if (whole) reach = std::max(reach, y.shift);
            ps.staged_rows += d + 1;
            ps.max_chain = std::max(ps.max_chain, d);
          } else {
            term[terms++] = Term{x.row, shift};
            reach = std::max(reach, shift);
            ++ps.staged_rows;
          }
        }
      }
    }
    head[1] = rows_a;
    head[7] = reach;
    head[8] = complete;
    head[2] = static_cast<int32_t>(s.block_offs.size() - ps.offs_offset);
    const Node *below = na;
    std::vector<int> *base = &base_a;
    int rows_b = 0;
    std::string err;
    if (ps.k2 > 0) {
      const Node *nb = level(ps.k2);
      const int count_b = 1 << ps.k3;
      rows_b = bases(nb, count_b, base_b);
      err = block_offsets(t, l0 + ps.k1 + ps.k2, ps.k2, nb, count_b, na, base_a, lead, ps, s.block_offs);
      if (!err.empty()) return err;
      below = nb;
      base = &base_b;
    }
    head[3] = rows_b;
    head[4] = static_cast<int32_t>(s.block_offs.size() - ps.offs_offset);
    err = block_offsets(t, ps.l1, ps.k3, level(kl), 1, below, *base, ps.k2 > 0 ? 0 : lead, ps, s.block_offs);
    if (!err.empty()) return err;
    head[5] = b.nr;
    head[6] = static_cast<int32_t>(t.row_off[ps.l1][b.sub] + b.r0);
    s.block_heads.insert(s.block_heads.end(), head, head + kBlockHeader);
    ps.rows_a = std::max(ps.rows_a, rows_a);
    ps.rows_b = std::max(ps.rows_b, rows_b);
  }
  if ((ps.rows_a + ps.rows_b + 1) * kBlockPitch * 4 > 64 * 1024) return "block rows do not fit LDS";
  ps.nblocks = static_cast<int>(blocks.size());
  return "";
}

} // namespace

std::string build_block_schedule(Schedule &s, const Tables &t, int64_t nt, bool search, bool bytes) {
  s = Schedule();
  const int L = search ? t.levels - 3 : t.levels;  // iterations of the block passes
  if (L < 3) return "fewer than three iterations";
  int chain = 0;
  for (int k = 0; k < t.nf; ++k) chain = std::max(chain, t.leaf_rows[k] - 1);
  s.init_separate = chain > kBlockMaxChain;
  const int passes = (L + kBlockLevels - 1) / kBlockLevels;
  int l0 = 0;
  for (int i = 0; i < passes; ++i) {
    const int k = (L - l0 + passes - i - 1) / (passes - i);
    const bool from_input = i == 0 && !s.init_separate;
    Pass one, many;
    const std::string err = build_block_pass(s, t, nt, l0, k, from_input, bytes, false, one);
    if (!err.empty()) return err;
    // Blocks of 4 rows load two to three times the terms per output of blocks of 16
    // or 18: a batch takes whole ones where they come to two workgroups per CU (256
    // records of Nf=64, Nt=1024, Nd=64 FP32 159 -> 77 us, 64 of Nf=256, Nt=500,
    // Nd=256 121 -> 90 us). With fewer the smaller blocks can be the faster ones (8 of
    // the latter 22.7 us, 23.4 us with whole ones; 4 of the former 7.8 and 10.2 us).
    if (one.few && build_block_pass(s, t, nt, l0, k, from_input, bytes, true, many).empty()) {
      many.samples = (511 + many.nblocks) / many.nblocks * static_cast<int64_t>(kBlockTile);
    } else {
      many = Pass();
    }
    s.passes.push_back(one);
    s.many.push_back(many);
    l0 += k;
  }
  if (search) {
    ScheduleParams p;
    return build_pass(s, t, p, l0, 3, false);
  }
  return "";
}

namespace {

// Depth-first walk of one adjoint output row (see AdjLeaf).
struct AdjWalker {
  const Tables &t;
  int l_hi;
  std::vector<AdjLeaf> &out;

  // Row r of plane l at accumulated shift sigma, tree depth d; `branch` is
  // the branch depth handed to the first leaf below this node.
  void visit(int l, int r, int sigma, int d, int branch) {
    if (l == l_hi) {
      out.push_back(AdjLeaf{r, sigma, branch, 0});
      return;
    }
    const AdjRow &a = t.adj[l + 1][r];
    for (int q = 0; q < a.count; ++q) {
      const int p = a.first + q;
      const int s = a.upper ? t.merge[l + 1][p].s : 0;
      visit(l + 1, p, sigma + s, d + 1, q == 0 ? branch : d);
    }
  }
};

} // namespace

std::string build_adjoint_schedule(AdjSchedule &s, const Tables &t, int levels_per_pass, int last_levels,
                                   bool lag_reuse) {
  s = AdjSchedule();
  const int L = t.levels;
  if (L == 0) return "";
  if (levels_per_pass < 1 || last_levels < 1) return "bad adjoint schedule parameters";
  // Fold the init transpose into the last pass only while its fan-out (the
  // (d, i) pairs of a channel, quadratic in its partial-sum rows) is small;
  // otherwise the passes stop at plane 0 and the transpose runs on its own.
  int fan = 0, rows_max = 0;
  for (int k = 0; k < t.nf; ++k) {
    fan = std::max(fan, t.leaf_rows[k] * (t.leaf_rows[k] + 1) / 2);
    rows_max = std::max(rows_max, t.leaf_rows[k]);
  }
  s.init_separate = fan > 16;
  int l_hi = L;
  while (l_hi > 0) {
    AdjPass ps;
    ps.l_hi = l_hi;
    // The last pass (down to the channels) takes the init transpose too.
    if (l_hi <= last_levels && !s.init_separate) {
      ps.l_lo = 0;
      ps.to_input = true;
      ps.depth = l_hi + 1;
      ps.nrows = t.nf;
      ps.lagged = lag_reuse && rows_max > 1 && rows_max <= kMaxLags;
    } else {
      ps.l_lo = std::max(l_hi - levels_per_pass, s.init_separate ? 0 : last_levels);
      ps.depth = l_hi - ps.l_lo;
      ps.nrows = static_cast<int>(t.total[ps.l_lo]);
    }
    if (ps.depth > 5) return "adjoint pass deeper than 5";
    ps.leaf_offset = static_cast<int64_t>(s.leaves.size());
    ps.start_offset = static_cast<int64_t>(s.starts.size());
    ps.order_offset = static_cast<int64_t>(s.order.size());
    // Leaves of every output row, then the rows ordered by the first plane-l_hi
    // row they read.
    std::vector<std::vector<AdjLeaf>> per_row(ps.nrows);
    for (int r = 0; r < ps.nrows; ++r) {
      AdjWalker w{t, l_hi, per_row[r]};
      if (ps.lagged) {
        // channel r: the subtree of each partial-sum row d once, at lag 0
        // (plus the channel's pre-shift), its first leaf carrying the d + 1
        // lags it is added at
        for (int d = 0; d < t.leaf_rows[r]; ++d) {
          const size_t first = per_row[r].size();
          w.visit(0, t.leaf_off[r] + d, t.pre[r], 1, 0);
          per_row[r][first].lags = (d + 1) | static_cast<int32_t>(per_row[r].size() - first) << 3;
        }
      } else if (ps.to_input) {
        // channel r: partial-sum rows d at lags i (plus the channel's
        // pre-shift), in (d, i) order; each starts a new child of the root
        // (branch depth 0)
        for (int d = 0; d < t.leaf_rows[r]; ++d)
          for (int i = 0; i <= d; ++i) w.visit(0, t.leaf_off[r] + d, t.pre[r] + i, 1, 0);
      } else {
        w.visit(ps.l_lo, r, 0, 0, 0);
      }
    }
    std::vector<int32_t> ord(ps.nrows);
    for (int r = 0; r < ps.nrows; ++r) ord[r] = r;
    std::stable_sort(ord.begin(), ord.end(), [&](int32_t a, int32_t b) {
      return per_row[a].front().row < per_row[b].front().row;
    });
    for (int i = 0; i < ps.nrows; ++i) {
      s.starts.push_back(static_cast<int32_t>(s.leaves.size() - ps.leaf_offset));
      s.order.push_back(ord[i]);
      const std::vector<AdjLeaf> &lv = per_row[ord[i]];
      s.leaves.insert(s.leaves.end(), lv.begin(), lv.end());
    }
    s.starts.push_back(static_cast<int32_t>(s.leaves.size() - ps.leaf_offset));
    ps.leaves = static_cast<int64_t>(s.leaves.size()) - ps.leaf_offset;
    if (s.leaves.size() > static_cast<size_t>(INT32_MAX)) return "adjoint schedule too large";
    // Audit: rows inside plane l_hi, shifts non-negative, branch depths valid.
    for (int64_t x = ps.leaf_offset; x < static_cast<int64_t>(s.leaves.size()); ++x) {
      const AdjLeaf &e = s.leaves[x];
      if (e.row < 0 || e.row >= t.total[l_hi] || e.shift < 0 || e.branch < 0 || e.branch >= ps.depth)
        return "adjoint leaf out of range";
      if (!ps.lagged && e.lags != 0) return "adjoint leaf lags";
      ps.max_shift = std::max(ps.max_shift, e.shift);
    }
    // A lagged pass: each row is a sequence of subtrees, each opened by a leaf
    // at branch 0 that holds its lags (1..kMaxLags) and leaf count, the other
    // leaves below the root.
    if (ps.lagged) {
      for (int i = 0; i < ps.nrows; ++i) {
        const int64_t end = ps.leaf_offset + s.starts[ps.start_offset + i + 1];
        for (int64_t x = ps.leaf_offset + s.starts[ps.start_offset + i]; x < end;) {
          const AdjLeaf &e = s.leaves[x];
          const int lags = e.lags & 7, count = e.lags >> 3;
          if (e.branch != 0 || lags < 1 || lags > kMaxLags || count < 1 || x + count > end)
            return "adjoint leaf lags";
          for (int64_t y = x + 1; y < x + count; ++y)
            if (s.leaves[y].branch == 0 || s.leaves[y].lags != 0) return "adjoint leaf lags";
          x += count;
        }
      }
    }
    s.passes.push_back(ps);
    l_hi = ps.l_lo;
  }
  return "";
}

namespace {

// One output row of a block pass.
struct AdjOutRow {
  int32_t row, sub;     // plane l_lo row (or channel) and its sub-band
  int32_t first, last;  // its leaves in plane m (row, shift, branch): [first, last) of a common list
  int32_t lead;         // plane m row of the first leaf, its smallest
};

std::string build_adjoint_block_pass(AdjSchedule &s, const Tables &t, int64_t nt, int l_hi, int l_lo, bool to_input) {
  AdjPass shape;
  shape.block = true;
  shape.l_hi = l_hi;
  shape.l_lo = l_lo;
  shape.to_input = to_input;
  const int k = l_hi - l_lo;
  shape.k1 = k >= 3 ? 2 : 1;
  const int m = l_hi - shape.k1;
  shape.depth2 = k - shape.k1 + (to_input ? 1 : 0);
  shape.depth = k + (to_input ? 1 : 0);
  shape.nrows = static_cast<int>(to_input ? t.nf : t.total[l_lo]);
  // Output rows of every sub-band of plane m with channels, by their first row.
  const int subs = (t.nf + (1 << m) - 1) >> m;
  std::vector<AdjOutRow> outs;
  std::vector<size_t> out_of(subs + 1, 0);  // first output of each sub-band of plane m
  std::vector<AdjLeaf> pool;
  outs.reserve(shape.nrows);
  pool.reserve(static_cast<size_t>(shape.nrows) * 5);
  int64_t rows = 0;
  for (int x = 0; x < subs; ++x) {
    rows += t.rows[m][x];
    for (int q = x << (m - l_lo); q < (x + 1) << (m - l_lo) && (static_cast<int64_t>(q) << l_lo) < t.nf; ++q) {
      const int n = to_input ? 1 : t.rows[l_lo][q];
      for (int r = 0; r < n; ++r) {
        AdjOutRow o{to_input ? q : static_cast<int32_t>(t.row_off[l_lo][q] + r), q, static_cast<int32_t>(pool.size()), 0, 0};
        AdjWalker w{t, m, pool};
        if (to_input) {
          for (int d = 0; d < t.leaf_rows[q]; ++d)
            for (int i = 0; i <= d; ++i) w.visit(0, t.leaf_off[q] + d, t.pre[q] + i, 1, 0);
        } else {
          w.visit(l_lo, o.row, 0, 0, 0);
        }
        o.last = static_cast<int32_t>(pool.size());
        if (o.first == o.last) return "output row without leaves";
        o.lead = pool[o.first].row;
        outs.push_back(o);
      }
    }
    out_of[x + 1] = outs.size();
    std::stable_sort(outs.begin() + out_of[x], outs.end(),
                     [](const AdjOutRow &a, const AdjOutRow &b) { return a.lead < b.lead; });
  }
  // The pass with ranges of rows for one record, or for a batch of many.
  const auto build = [&](bool many, AdjPass &ps) -> std::string {
    ps = shape;
    ps.head_offset = static_cast<int64_t>(s.block_heads.size());
    ps.mid_offset = static_cast<int64_t>(s.block_mids.size());
    ps.out_offset = static_cast<int64_t>(s.block_outs.size());
    ps.leaf_offset = static_cast<int64_t>(s.block_leaves1.size());
    ps.leaf2_offset = static_cast<int64_t>(s.block_leaves2.size());
    // Windows of 512 samples, outputs on whole 128-byte lines, where that leaves
    // each CU's two workgroups of 1024 threads more than once their work (Nf=4096,
    // Nt=65536, Nd=2048: 1.05 ms against 1.20 ms with windows of 256); below, twice
    // the workgroups of half the size (Nf=Nd=1024, Nt=8192: 75 us against 86 us).
    int own = 28;
    const auto workgroups = [&](int pitch) { return (rows + own - 1) / own * ((nt + pitch - 33) / (pitch - 32)); };
    ps.pitch = workgroups(512) >= 1024 ? 512 : 256;
    const int align = ps.pitch == 512 ? 32 : 4;
    // Fewer rows of plane m per range where the blocks would leave CUs idle: ranges
    // are halved while there are less than 768 workgroups of the 1024 that run at
    // once (Nf=64, Nt=20000, Nd=64 15.8 us, 22 us with 256 of them; Nf=1024, Nt=Nd=1000
    // 24.6 and 32.6 us; at 1024 other shapes lost up to 10%). A batch has them anyway,
    // and larger ranges make fewer rows twice; so do few rows in one or two blocks,
    // which are halved below 256 only (Nf=100, Nt=100000, Nd=16 28 us, 28.7 us). A
    // sub-band of no more than `most` rows stays whole, no row of it made twice,
    // unless half the GPU would be idle.
    int most = kAdjBlockRows;
    const int enough = many || rows <= 2 * own ? 256 : 768;
    while (own > 7 && ps.pitch == 256 && workgroups(ps.pitch) < enough) {
      ps.few = ps.few || workgroups(ps.pitch) >= 256;
      own /= 2;
      if (enough == 256 || workgroups(ps.pitch) < 600) most = own;
    }
    // Ranges, gathered into blocks while their rows fit LDS and their outputs'
    // offsets lie together: a block runs the windows between its smallest and its
    // largest offset for all of its rows.
    const int64_t apart = std::max<int64_t>(ps.pitch, nt / 2);
    typedef std::array<int32_t, kAdjBlockHeader> Head;
    struct Block {
      Head head;
      int32_t row;  // its first row of plane l_hi
    };
    std::vector<Block> blocks;
    Block block{};
    int block_rows = 0, spread = 0;
    std::vector<AdjLeaf> leaves;
    std::vector<int32_t> betas;
    s.block_leaves1.reserve(s.block_leaves1.size() + static_cast<size_t>(rows) * 6);
    s.block_leaves2.reserve(s.block_leaves2.size() + pool.size());
    s.block_outs.reserve(s.block_outs.size() + outs.size());
    const auto flush = [&]() {
      if (block_rows == 0) return;
      block.head[1] = block_rows;
      block.head[3] = static_cast<int32_t>(s.block_outs.size() - ps.out_offset) - block.head[2];
      blocks.push_back(block);
      ps.rows_mid = std::max(ps.rows_mid, block_rows);
      block_rows = 0;
    };
    // Outputs [first, last), with their rows lo .. hi of plane m.
    const auto add_range = [&](size_t first, size_t last, int32_t lo, int32_t hi) {
      // The range's smallest stage-1 shift moves its window instead of its
      // leaves: every range then reads plane l_hi over one and the same time.
      int32_t lag = INT32_MAX;
      const int32_t mid = static_cast<int32_t>(s.block_mids.size() - ps.mid_offset);
      const size_t leaf = s.block_leaves1.size();
      for (int32_t r = lo; r <= hi; ++r) {
        leaves.clear();
        AdjWalker w{t, l_hi, leaves};
        w.visit(m, r, 0, 0, 0);
        s.block_mids.push_back(static_cast<int32_t>(s.block_leaves1.size() - ps.leaf_offset));
        for (const AdjLeaf &e : leaves) {
          s.block_leaves1.push_back(AdjBlockLeaf{e.row, 4 * e.shift + e.branch});
          lag = std::min(lag, e.shift);
        }
      }
      // each output sub-band's smallest shift in this range is its offset (the
      // sub-bands under one of plane m are few and consecutive)
      const int sub0 = (outs[first].sub >> (m - l_lo)) << (m - l_lo);
      betas.assign(size_t(1) << (m - l_lo), INT32_MAX);
      for (size_t i = first; i < last; ++i)
        for (int32_t x = outs[i].first; x < outs[i].last; ++x)
          betas[outs[i].sub - sub0] = std::min(betas[outs[i].sub - sub0], pool[x].shift);
      int32_t near = INT32_MAX, far = 0;
      for (int32_t &b : betas)
        if (b != INT32_MAX) {
          b -= (b + lag) & (align - 1);
          near = std::min(near, b + lag);
          far = std::max(far, b + lag);
        }
      const int have = hi - lo + 1;
      if (block_rows > 0 && (block_rows + have > kAdjBlockRows || block_rows >= own ||
                             std::max(block.head[5], far) - std::min(block.head[6], near) > apart))
        flush();
      if (block_rows == 0) {
        block = Block{};
        block.head[0] = mid;
        block.head[2] = static_cast<int32_t>(s.block_outs.size() - ps.out_offset);
        block.head[6] = INT32_MAX;
        block.row = s.block_leaves1[leaf].row;
      }
      for (size_t x = leaf; x < s.block_leaves1.size(); ++x) {
        s.block_leaves1[x].shift4 -= 4 * lag;
        block.head[4] = std::max(block.head[4], s.block_leaves1[x].shift4 >> 2);
      }
      block.head[5] = std::max(block.head[5], far);
      block.head[6] = std::min(block.head[6], near);
      for (size_t i = first; i < last; ++i) {
        const AdjOutRow &o = outs[i];
        const int32_t beta = betas[o.sub - sub0];
        AdjBlockOut b{static_cast<int32_t>(s.block_leaves2.size() - ps.leaf2_offset), 0, o.row, beta + lag};
        for (int32_t x = o.first; x < o.last; ++x) {
          const AdjLeaf &e = pool[x];
          s.block_leaves2.push_back(((block_rows + e.row - lo) * ps.pitch + e.shift - beta) * 4 + e.branch);
          spread = std::max(spread, e.shift - beta);
        }
        b.last = static_cast<int32_t>(s.block_leaves2.size() - ps.leaf2_offset);
        s.block_outs.push_back(b);
      }
      block_rows += have;
    };
    for (int x = 0; x < subs; ++x) {
      const int n = t.rows[m][x];
      const int32_t off = static_cast<int32_t>(t.row_off[m][x]);
      // A range's stage 1 has a leaf for each row of plane l_hi that it reads: under
      // a wide sub-band of plane l_hi 28 rows read up to 300, against 60 and 150 in
      // the blocks beside them, and a few such blocks were the tail of a pass
      // (Nf=Nd=1024, Nt=16384, 0.4-0.8 GHz, one record: first pass 72 us in 38 blocks,
      // 67 us in 40 that are no lighter, 43 us in these 40; the adjoint 144 and 120 us,
      // of 16 records 1845 and 1780 us). Bounds of 185 to 245 leaves measure alike,
      // 160 and less make too many rows twice (1.1-1.9 GHz 5% slower), 270 changes
      // nothing. Where heavy blocks were no tail, the rows made twice cost up to 4%
      // (Nt=8192, 0.3-0.9 GHz).
      const int64_t leaves1 = t.rows[l_hi][x >> shape.k1];
      const int each = static_cast<int>(std::clamp<int64_t>(int64_t(n) * 240 / leaves1, std::min(own, 7), own));
      const int parts = n <= most ? 1 : row_parts(n, each, subs);
      size_t i = out_of[x];
      for (int b = 0; b < parts; ++b) {
        const int32_t end = off + static_cast<int32_t>(static_cast<int64_t>(n) * (b + 1) / parts);
        const size_t first = i;
        int32_t lo = INT32_MAX, hi = -1;
        for (; i < out_of[x + 1] && outs[i].lead < end; ++i)
          for (int32_t y = outs[i].first; y < outs[i].last; ++y) {
            lo = std::min(lo, pool[y].row);
            hi = std::max(hi, pool[y].row);
          }
        if (first == i) continue;
        if (hi - lo + 1 > kAdjBlockRows) return "block rows do not fit LDS";
        add_range(first, i, lo, hi);
      }
    }
    flush();
    s.block_mids.push_back(static_cast<int32_t>(s.block_leaves1.size() - ps.leaf_offset));
    // blocks of several sub-bands read the same rows of plane l_hi: run them next
    // to each other, on one XCD
    std::stable_sort(blocks.begin(), blocks.end(), [](const Block &a, const Block &b) { return a.row < b.row; });
    ps.leaf1_count = static_cast<int64_t>(s.block_leaves1.size()) - ps.leaf_offset;
    ps.leaves = ps.leaf1_count;
    ps.tile = (ps.pitch - spread) / align * align;
    if (ps.tile < 128 || spread > 128) return "block shifts spread too far";
    // T0 = 0 is the same time in every block where the record is longer than the
    // offsets: blocks then read plane l_hi over one time (three beams of Nf=1024,
    // Nt=3283, Nd=1823, offsets half a record, 55 us for the first pass, 61 us each
    // from its own). A smallest delay, or a shorter record, would make most of them
    // windows that no output of the block lies in: there T0 = 0 is each block's own
    // first window (Nf=1024, Nt=1024, Nd=64, smallest delay 100000: 32481 workgroups
    // of the last pass, now 1568, and the adjoint 72 us, now 17 us; register gathers
    // 19 us).
    for (const Block &b : blocks) ps.extra = std::max(ps.extra, b.head[5]);
    const bool own_start = to_input || ps.extra > nt;
    ps.extra = 0;
    for (Block &b : blocks) {
      if (const int32_t first = own_start ? b.head[6] / ps.tile * ps.tile : 0) {
        if (first > 1 << 28) return "offsets too large";
        const int32_t *mids = s.block_mids.data() + ps.mid_offset + b.head[0];
        for (int32_t x = mids[0]; x < mids[b.head[1]]; ++x) s.block_leaves1[ps.leaf_offset + x].shift4 += 4 * first;
        for (int32_t x = 0; x < b.head[3]; ++x) s.block_outs[ps.out_offset + b.head[2] + x].beta -= first;
        b.head[4] += first;
        b.head[5] -= first;
        b.head[6] -= first;
      }
      ps.extra = std::max(ps.extra, b.head[5]);
      s.block_heads.insert(s.block_heads.end(), b.head.begin(), b.head.end());
    }
    ps.nblocks = static_cast<int>(blocks.size());
    if (ps.extra > 2 * nt + 4 * ps.pitch) return "offsets of a block spread past its records";
    if (s.block_leaves1.size() > static_cast<size_t>(INT32_MAX) || s.block_leaves2.size() > static_cast<size_t>(INT32_MAX))
      return "adjoint schedule too large";
    for (int64_t x = ps.leaf_offset; x < ps.leaf_offset + ps.leaf1_count; ++x) {
      const AdjBlockLeaf &e = s.block_leaves1[x];
      if (e.row < 0 || e.row >= t.total[l_hi] || e.shift4 < 0 || (e.shift4 & 3) >= ps.k1) return "adjoint leaf out of range";
    }
    for (size_t x = ps.leaf2_offset; x < s.block_leaves2.size(); ++x) {
      const int32_t e = s.block_leaves2[x];
      if (e < 0 || (e & 3) >= ps.depth2 || e / 4 / ps.pitch >= ps.rows_mid) return "adjoint LDS leaf out of range";
    }
    return "";
  };
  AdjPass one, many;
  const std::string err = build(false, one);
  if (!err.empty()) return err;
  if (one.few && build(true, many).empty())
    many.samples = (1023 + many.nblocks) / many.nblocks * static_cast<int64_t>(kBlockTile);
  else
    many = AdjPass();
  s.passes.push_back(one);
  s.many.push_back(many);
  return "";
}

} // namespace

std::string build_adjoint_block_schedule(AdjSchedule &s, const Tables &t, int64_t nt) {
  s = AdjSchedule();
  const int L = t.levels;
  if (L < 2) return "fewer than two iterations";
  int fan = 0;
  for (int k = 0; k < t.nf; ++k) fan = std::max(fan, t.leaf_rows[k] * (t.leaf_rows[k] + 1) / 2);
  s.init_separate = fan > 16;
  const int passes = (L + 3) / 4;
  int l_hi = L;
  for (int i = 0; i < passes; ++i) {
    const int k = (l_hi + passes - i - 1) / (passes - i);
    const std::string err =
        build_adjoint_block_pass(s, t, nt, l_hi, l_hi - k, i == passes - 1 && !s.init_separate);
    if (!err.empty()) return err;
    l_hi -= k;
  }
  return "";
}

} // namespace fdmt
