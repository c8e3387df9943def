// How the window driver runs a window plan's phases: the same values, fewer
// passes over the versioned signals.  A window's signals are far larger than
// the caches (a 1024-neuron layer of 256 batch columns and 50 steps is 52 MB),
// so each phase that only resets, copies or scales is a pass at the copy rate.
//
//   * A reset (or a copy of a parameter) that only prepares rows for one
//     increment goes: the increment starts from its value.
//   * A copy of a whole row into a row that nothing else writes goes: its
//     readers read the source.
//   * A neuron phase whose input current is such a started increment J = bias +
//     gain (.) x computes J itself, and runs the synaptic filter that yields x
//     when nothing else reads that filter.
//
// Each row's value is formed by the same operations in the same order, so the
// results are the same (a copied -0 may become +0 and back).
#include <algorithm>

#include "host.hpp"

namespace ms {

namespace {

int64_t row_at(const LOperand& o, int64_t r) { return o.idx.empty() ? o.start + r : o.idx[(size_t)r]; }

LOperand operand_of(int32_t base, std::vector<int32_t> rows) {
  LOperand o;
  o.base = base;
  bool run = !rows.empty();
  for (size_t k = 1; k < rows.size() && run; ++k) run = rows[k] == rows[0] + (int32_t)k;
  if (run) o.start = rows[0];
  else o.idx = std::move(rows);
  return o;
}

int64_t entries(const LGroup& g) { return g.ptr.empty() ? g.rows : (int64_t)g.ptr.back(); }

struct Fuser {
  const Plan& p;
  const WindowPlan& w;
  std::vector<WRun>& run;
  std::vector<Phases> writers, readers;   // per versioned row
  std::vector<char> probed;

  bool batched(const LOperand& o) const { return o.base >= 0 && p.ir.bases[o.base].cls == SC_BATCHED; }

  // f(row) for every versioned row that phase k writes.
  template <class F>
  void each_write(int32_t k, F&& f) const {
    const LGroup& g = run[k].g;
    if (g.type == OP_DOT_INC) {
      for (int32_t d : g.d_row)
        for (int32_t m = 0; m < g.M; ++m) f((int64_t)d + m);
    } else if (g.type == OP_ENS) {
      for (size_t o = 0; o < g.ens_n.size(); ++o) {
        for (size_t fn = 0; fn < g.ens_df.size(); ++fn)
          for (int32_t q = 0; q < g.ens_df[fn]; ++q) f((int64_t)g.ens_dd[fn][o] + q);
        if (g.ens_s[o] >= 0)
          for (int32_t r = 0; r < g.ens_n[o]; ++r) f((int64_t)g.ens_s[o] + r);
        if (!g.ens_chain.empty() && g.ens_chain[kChainInts * o + 1] > 0)
          for (int32_t m = 0; m < g.ens_chain[kChainInts * o + 4]; ++m) f((int64_t)g.ens_chain[kChainInts * o + 3] + m);
      }
    } else {
      for (int64_t r = 0; r < g.rows; ++r) f(row_at(g.dst, r));
    }
  }

  // f(row) for every versioned row that phase k reads as an operand.
  template <class F>
  void each_read(int32_t k, F&& f) const {
    const LGroup& g = run[k].g;
    switch (g.type) {
      case OP_COPY: case OP_COPY_INC: case OP_ELEM_INC: case OP_LIF: case OP_LIF_RATE: case OP_LOWPASS:
        if (batched(g.src))
          for (int64_t e = 0; e < entries(g); ++e) f(row_at(g.src, e));
        if (g.type == OP_ELEM_INC && batched(g.a))
          for (int64_t e = 0; e < entries(g); ++e) f(row_at(g.a, e));
        break;
      case OP_DOT_INC:
        for (int32_t x : g.x_row)
          for (int32_t q = 0; q < g.K; ++q) f((int64_t)x + q);
        break;
      case OP_ENS:
        for (size_t o = 0; o < g.ens_n.size(); ++o) {
          const bool chain = !g.ens_chain.empty() && g.ens_chain[kChainInts * o + 1] > 0;
          const int32_t x = chain ? g.ens_chain[kChainInts * o] : g.ens_x[o];
          const int32_t n = chain ? g.ens_chain[kChainInts * o + 1] : g.ens_d;
          for (int32_t q = 0; x >= 0 && q < n; ++q) f((int64_t)x + q);
        }
        break;
      default: break;
    }
  }

  void index() {
    writers.resize((size_t)w.rows_v);
    readers.resize((size_t)w.rows_v);
    for (Phases& v : writers) v.n = 0;
    for (Phases& v : readers) v.n = 0;
    for (int32_t k = 0; k < (int32_t)run.size(); ++k) {
      if (run[k].skip) continue;
      each_write(k, [&](int64_t r) { if (!writers[r].ends_with(k)) writers[r].push_back(k); });
      each_read(k, [&](int64_t r) { if (!readers[r].ends_with(k)) readers[r].push_back(k); });
    }
  }

  // Increments that are the first writer after a reset or a parameter copy.
  void start_increments() {
    const int32_t n = (int32_t)run.size();
    std::vector<int64_t> where((size_t)w.rows_v, -1);   // row -> position in its first writer
    for (int32_t k = 0; k < n; ++k)
      if (run[k].g.type == OP_RESET || run[k].g.type == OP_COPY)
        for (int64_t r = 0; r < run[k].g.rows; ++r) where[row_at(run[k].g.dst, r)] = r;
    std::vector<int32_t> from((size_t)n, -1);           // increment -> the phase its rows come from
    for (int32_t k = 0; k < n; ++k) {
      const LGroup& g = run[k].g;
      if (g.type != OP_COPY_INC && g.type != OP_ELEM_INC && g.type != OP_DOT_INC) continue;
      bool ok = g.rows > 0;
      int32_t src = -1;
      std::vector<int64_t> rows;
      each_write(k, [&](int64_t r) {
        if (!ok) return;
        rows.push_back(r);
        const Phases& ws = writers[r];
        if (ws.size() < 2 || ws[1] != k || (src >= 0 && ws[0] != src)) { ok = false; return; }
        src = ws[0];
        const LGroup& f = run[src].g;
        if (f.type == OP_RESET) {
          if (g.type == OP_DOT_INC && !f.values.empty() && f.values[(size_t)where[r]] != 0.0f) ok = false;
        } else if (f.type != OP_COPY || batched(f.src) || g.type == OP_DOT_INC) {
          ok = false;
        }
      });
      std::sort(rows.begin(), rows.end());
      if (!ok || std::adjacent_find(rows.begin(), rows.end()) != rows.end()) continue;
      from[k] = src;
    }
    // a parameter copy goes only as a whole (its reverse stays in use)
    for (int32_t k = 0; k < n; ++k) {
      if (run[k].g.type != OP_COPY) continue;
      int64_t used = 0;
      for (int32_t q = 0; q < n; ++q)
        if (from[q] == k) each_write(q, [&](int64_t) { ++used; });
      if (used == 0) continue;
      if (used == run[k].g.rows) { run[k].skip = true; continue; }
      for (int32_t q = 0; q < n; ++q) if (from[q] == k) from[q] = -1;
    }
    std::vector<std::vector<char>> gone((size_t)n);
    for (int32_t k = 0; k < n; ++k) {
      if (from[k] < 0) continue;
      const LGroup& f = run[from[k]].g;
      WRun& r = run[k];
      if (f.type == OP_COPY) {
        r.init = 2;
        std::vector<int32_t> rows;
        each_write(k, [&](int64_t d) { rows.push_back((int32_t)row_at(f.src, where[d])); });
        r.init_src = operand_of(f.src.base, std::move(rows));
      } else {
        r.init = 1;
        if (!f.values.empty()) {
          each_write(k, [&](int64_t d) { r.init_vals.push_back(f.values[(size_t)where[d]]); });
          if (std::all_of(r.init_vals.begin(), r.init_vals.end(), [](float v) { return v == 0.0f; })) r.init_vals.clear();
        }
        gone[from[k]].resize((size_t)f.rows, 0);
        each_write(k, [&](int64_t d) { gone[from[k]][(size_t)where[d]] = 1; });
      }
    }
    for (int32_t k = 0; k < n; ++k) {
      if (gone[k].empty()) continue;
      LGroup& f = run[k].g;
      std::vector<int32_t> rows;
      std::vector<float> vals;
      for (int64_t r = 0; r < f.rows; ++r)
        if (!gone[k][(size_t)r]) {
          rows.push_back((int32_t)row_at(f.dst, r));
          if (!f.values.empty()) vals.push_back(f.values[(size_t)r]);
        }
      f.rows = (int64_t)rows.size();
      f.values = std::move(vals);
      f.dst = operand_of(f.dst.base, std::move(rows));
      if (f.rows == 0) run[k].skip = true;
    }
  }

  // Row `r` read at block offset blk through the copies alias[row] = (source,
  // block offset).
  static bool through(const std::vector<std::pair<int32_t, int32_t>>& alias, int32_t r, int32_t blk, int32_t* nr, int32_t* nb) {
    *nr = r;
    *nb = blk;
    if (alias[r].first < 0) return true;
    *nr = alias[r].first;
    *nb = blk - 1 + alias[r].second;
    return *nb >= 0;
  }

  // Rewrites the operands of phase q that read rows of `alias`; false (nothing
  // changed) when an operand cannot express it.
  bool rewrite(WRun& q, const std::vector<std::pair<int32_t, int32_t>>& alias) const {
    LGroup& g = q.g;
    auto operand = [&](LOperand& o, int32_t& blk) {
      std::vector<int32_t> rows;
      int32_t nb = -1;
      for (int64_t e = 0; e < entries(g); ++e) {
        int32_t r, b;
        if (!through(alias, (int32_t)row_at(o, e), blk, &r, &b) || (nb >= 0 && b != nb)) return false;
        nb = b;
        rows.push_back(r);
      }
      if (nb < 0) return true;
      o = operand_of(o.base, std::move(rows));
      blk = nb;
      return true;
    };
    auto runs = [&](std::vector<int32_t>& first, int32_t len, int32_t& blk) {
      std::vector<int32_t> out = first;
      int32_t nb = -1;
      for (size_t o = 0; o < first.size(); ++o)
        for (int32_t k = 0; first[o] >= 0 && k < len; ++k) {
          int32_t r, b;
          if (!through(alias, first[o] + k, blk, &r, &b) || (nb >= 0 && b != nb)) return false;
          nb = b;
          if (k == 0) out[o] = r;
          else if (r != out[o] + k) return false;
        }
      first = std::move(out);
      if (nb >= 0) blk = nb;
      return true;
    };
    const WRun old = q;
    bool ok = true;
    switch (g.type) {
      case OP_COPY: case OP_COPY_INC: case OP_LIF: case OP_LIF_RATE: case OP_LOWPASS: case OP_ELEM_INC:
        if (batched(g.src)) ok = operand(g.src, q.src_blk);
        if (ok && g.type == OP_ELEM_INC && batched(g.a)) ok = operand(g.a, q.a_blk);
        break;
      case OP_DOT_INC: ok = runs(g.x_row, g.K, q.src_blk); break;
      case OP_ENS: ok = g.ens_chain.empty() && runs(g.ens_x, g.ens_d, q.src_blk); break;
      default: ok = false;
    }
    if (!ok) q = old;
    return ok;
  }

  // Copies of whole rows whose readers can read the source instead.
  void drop_copies() {
    std::vector<char> state((size_t)w.rows_v, 0);
    for (size_t k = 0; k < p.ir.sigs.size(); ++k)
      if (p.ir.sigs[k].cls == SC_BATCHED && p.ir.sigs[k].state && !w.priv[k])
        for (int32_t r = 0; r < p.ir.sigs[k].rows; ++r) state[(size_t)(w.sig_row[k] + r)] = 1;
    std::vector<std::pair<int32_t, int32_t>> alias((size_t)w.rows_v, {-1, 1});
    for (int32_t k = 0; k < (int32_t)run.size(); ++k) {
      const LGroup& g = run[k].g;
      if (run[k].skip || !batched(g.src)) continue;
      if (!(g.type == OP_COPY || (g.type == OP_COPY_INC && run[k].init == 1 && run[k].init_vals.empty() && entries(g) == g.rows)))
        continue;
      bool ok = true;
      for (int64_t r = 0; r < g.rows && ok; ++r) {
        const int64_t d = row_at(g.dst, r);
        ok = writers[d].size() == 1 && !probed[d] && !state[d];
      }
      if (!ok) continue;
      std::vector<int32_t> rd;
      for (int64_t r = 0; r < g.rows; ++r) {
        const int64_t d = row_at(g.dst, r);
        alias[d] = {(int32_t)row_at(g.src, r), run[k].src_blk};
        rd.insert(rd.end(), readers[d].begin(), readers[d].end());
      }
      std::sort(rd.begin(), rd.end());
      rd.erase(std::unique(rd.begin(), rd.end()), rd.end());
      std::vector<WRun> saved;
      size_t done = 0;
      for (; done < rd.size() && ok; ++done) {
        saved.push_back(run[rd[done]]);
        ok = rd[done] > k && rewrite(run[rd[done]], alias);
      }
      if (ok) {   // the sources' readers are now the copies' readers as well, but not phase k
        run[k].skip = true;
        std::vector<int32_t> both;
        for (int64_t r = 0; r < g.rows; ++r) {
          const int64_t d = row_at(g.dst, r);
          readers[row_at(g.src, r)].take(readers[d], k, both);
          readers[d].n = writers[d].n = 0;
        }
      } else {
        for (size_t i = 0; i < saved.size(); ++i) run[rd[i]] = saved[i];
      }
      for (int64_t r = 0; r < g.rows; ++r) alias[row_at(g.dst, r)] = {-1, 1};
    }
  }

  // Neuron phases that compute their own input current, and the filter
  // before it (spiking neurons, which run step after step; keep: every signal
  // stays stored for the backward pass, so the filter is not taken in).
  void fuse_currents(bool keep) {
    std::vector<int64_t> where((size_t)w.rows_v, -1);
    for (int32_t k = 0; k < (int32_t)run.size(); ++k) {
      WRun& q = run[k];
      if (q.skip || (q.g.type != OP_LIF && q.g.type != OP_LIF_RATE) || q.src_blk != 1 || !batched(q.g.src)) continue;
      auto only = [&](int64_t row, int32_t writer) {   // written by `writer` alone, read by phase k alone
        return writers[row].size() == 1 && writers[row][0] == writer && readers[row].size() == 1 &&
               readers[row][0] == k && !probed[row];
      };
      const int64_t n = q.g.rows;
      const int64_t r0 = row_at(q.g.src, 0);
      if (n == 0 || writers[r0].size() != 1) continue;
      const int32_t pe = writers[r0][0];
      WRun& e = run[pe];
      if (e.g.type != OP_ELEM_INC || e.init == 0 || entries(e.g) != e.g.rows || e.g.rows != n || !batched(e.g.src) ||
          batched(e.g.a))
        continue;
      bool ok = true;
      for (int64_t r = 0; r < n && ok; ++r) ok = only(row_at(q.g.src, r), pe);
      if (!ok) continue;
      for (int64_t r = 0; r < n; ++r) where[row_at(e.g.dst, r)] = r;
      std::vector<int32_t> x, a, is;
      for (int64_t r = 0; r < n; ++r) {
        const int64_t j = where[row_at(q.g.src, r)];
        x.push_back((int32_t)row_at(e.g.src, j));
        a.push_back((int32_t)row_at(e.g.a, j));
        if (e.init == 2) is.push_back((int32_t)row_at(e.init_src, j));
        else q.init_vals.push_back(e.init_vals.empty() ? 0.0f : e.init_vals[(size_t)j]);
      }
      q.init = e.init;
      if (e.init == 2) q.init_src = operand_of(e.init_src.base, std::move(is));
      q.jx = operand_of(e.g.src.base, x);
      q.ja = operand_of(e.g.a.base, std::move(a));
      q.jx_blk = e.src_blk;
      e.skip = true;
      // the filter that x is
      const Phases& wx = writers[x[0]];
      if (keep || q.g.type != OP_LIF || e.src_blk != 0 || wx.size() != 1 || run[wx[0]].g.type != OP_LOWPASS) continue;
      const int32_t pl = wx[0];
      WRun& f = run[pl];
      for (int64_t r = 0; r < n && ok; ++r) {
        const int64_t y = x[(size_t)r];
        ok = writers[y].size() == 1 && writers[y][0] == pl && readers[y].size() == 1 && readers[y][0] == pe && !probed[y];
      }
      std::vector<int32_t> ys = x;
      std::sort(ys.begin(), ys.end());
      if (!ok || f.skip || f.g.rows != n || std::adjacent_find(ys.begin(), ys.end()) != ys.end()) continue;
      for (int64_t r = 0; r < n; ++r) where[row_at(f.g.dst, r)] = r;
      std::vector<int32_t> v;
      for (int64_t r = 0; r < n; ++r) {
        const int64_t j = where[x[(size_t)r]];
        v.push_back((int32_t)row_at(f.g.src, j));
        q.fa.push_back(f.g.ca.size() > 1 ? f.g.ca[(size_t)j] : f.g.ca[0]);
        q.fb.push_back(f.g.cb.size() > 1 ? f.g.cb[(size_t)j] : f.g.cb[0]);
      }
      q.fy = q.jx;
      q.jx = operand_of(f.g.src.base, std::move(v));
      q.jx_blk = f.src_blk;
      f.skip = true;
    }
  }
};

}  // namespace

std::vector<WRun> fuse_window(const Plan& p, const WindowPlan& w) {
  std::vector<WRun> run(w.phases.size());
  for (size_t k = 0; k < run.size(); ++k) {
    run[k].g = w.phases[k].g;
    run[k].src_blk = w.phases[k].src_blk;
    run[k].a_blk = w.phases[k].a_blk;
  }
  Fuser f{p, w, run, {}, {}, std::vector<char>((size_t)std::max<int64_t>(1, w.rows_v), 0)};
  for (int32_t r : w.probe_rows) f.probed[(size_t)r] = 1;
  // a model that can be trained (built without simplification) keeps every
  // operand where the reverse of its phases reads it
  const bool trainable = !p.opts.simplify;
  f.index();
  f.start_increments();
  f.index();
  if (!trainable) f.drop_copies();
  f.fuse_currents(trainable);
  return run;
}

}  // namespace ms
