// The resident program: a small model's whole step as tables for k_resident,
// one workgroup per batch column with every neuron in registers.
//
// The merged groups of the plan, without the resets and whole-row copies that
// only prepare rows for one reader, become levels: a group runs after every
// earlier group that it conflicts with (one writes a row the other reads or
// writes), and groups of one level run without a barrier between them.  Rows
// other than neuron state get places in LDS, in row order, and every operand
// becomes such a place; each wavefront gets its own list of entries for the
// step (k_resident runs it without any lookup in global memory).
#include <algorithm>
#include <cmath>

#include "host.hpp"

namespace ms {

namespace {

int64_t row_at(const LOperand& o, int64_t r) { return o.idx.empty() ? o.start + r : o.idx[(size_t)r]; }
int64_t entries(const LGroup& g) { return g.ptr.empty() ? g.rows : (int64_t)g.ptr.back(); }
int32_t bits(float f) { return __builtin_bit_cast(int32_t, f); }

// One merged group on its way into the program.
struct Item {
  LGroup g;
  bool skip = false, init = false;   // init: the increment starts from vals (empty: zero)
  std::vector<float> vals;
};

struct Prep {
  const Plan& p;
  std::vector<Item>& G;
  int64_t nrows;
  std::vector<char> probed;
  std::vector<Phases> writers, readers;   // per row

  bool batched(const LOperand& o) const { return o.base >= 0 && p.ir.bases[o.base].cls == SC_BATCHED; }

  template <class F>
  void each_write(const LGroup& g, F&& f) const {
    if (g.type == OP_ENS) {
      for (size_t o = 0; o < g.ens_n.size(); ++o) {
        for (size_t k = 0; k < g.ens_df.size(); ++k)
          for (int32_t q = 0; q < g.ens_df[k]; ++q) f((int64_t)g.ens_dd[k][o] + q);
        for (int32_t r = 0; g.ens_s[o] >= 0 && r < g.ens_n[o]; ++r) f((int64_t)g.ens_s[o] + r);
      }
    } else if (g.type == OP_DOT_INC) {
      for (int32_t d : g.d_row)
        for (int32_t m = 0; m < g.M; ++m) f((int64_t)d + m);
    } else {
      for (int64_t r = 0; r < g.rows; ++r) f(row_at(g.dst, r));
    }
  }
  template <class F>
  void each_read(const LGroup& g, F&& f) const {
    if (g.type == OP_ENS) {
      for (int32_t x : g.ens_x)
        for (int32_t q = 0; x >= 0 && q < g.ens_d; ++q) f((int64_t)x + q);
    } else if (g.type == OP_DOT_INC) {
      for (int32_t x : g.x_row)
        for (int32_t q = 0; q < g.K; ++q) f((int64_t)x + q);
    } else if (batched(g.src)) {
      for (int64_t e = 0; e < entries(g); ++e) f(row_at(g.src, e));
    }
  }
  void index() {
    writers.resize((size_t)nrows);
    readers.resize((size_t)nrows);
    for (Phases& v : writers) v.n = 0;
    for (Phases& v : readers) v.n = 0;
    for (int32_t k = 0; k < (int32_t)G.size(); ++k) {
      if (G[k].skip) continue;
      each_write(G[k].g, [&](int64_t r) { if (!writers[r].ends_with(k)) writers[r].push_back(k); });
      each_read(G[k].g, [&](int64_t r) { if (!readers[r].ends_with(k)) readers[r].push_back(k); });
    }
  }

  // Increments that are the first to touch rows after their reset.
  void start_increments() {
    std::vector<int64_t> where((size_t)nrows, -1);
    for (const Item& it : G)
      if (it.g.type == OP_RESET)
        for (int64_t r = 0; r < it.g.rows; ++r) where[row_at(it.g.dst, r)] = r;
    std::vector<std::vector<char>> gone(G.size());
    for (int32_t k = 0; k < (int32_t)G.size(); ++k) {
      Item& it = G[k];
      if (it.g.type != OP_COPY_INC && it.g.type != OP_ELEM_INC && it.g.type != OP_DOT_INC) continue;
      bool ok = it.g.rows > 0;
      int32_t from = -1;
      std::vector<int64_t> rows;
      std::vector<float> vals;
      each_write(it.g, [&](int64_t r) {
        const Phases& w = writers[r];
        if (!ok || w.size() < 2 || w[1] != k || G[w[0]].g.type != OP_RESET || (from >= 0 && w[0] != from)) { ok = false; return; }
        from = w[0];
        for (int32_t q : readers[r]) if (q > from && q < k) ok = false;   // would see the reset value
        const LGroup& f = G[from].g;
        vals.push_back(f.values.empty() ? 0.0f : f.values[(size_t)where[r]]);
        if (it.g.type == OP_DOT_INC && vals.back() != 0.0f) ok = false;
        rows.push_back(r);
      });
      std::sort(rows.begin(), rows.end());
      if (!ok || std::adjacent_find(rows.begin(), rows.end()) != rows.end()) continue;
      it.init = true;
      if (!std::all_of(vals.begin(), vals.end(), [](float v) { return v == 0.0f; })) it.vals = std::move(vals);
      gone[from].resize((size_t)G[from].g.rows, 0);
      for (int64_t r : rows) gone[from][(size_t)where[r]] = 1;
    }
    for (size_t k = 0; k < G.size(); ++k) {
      if (gone[k].empty()) continue;
      LGroup& f = G[k].g;
      std::vector<int32_t> rows;
      std::vector<float> vals;
      for (int64_t r = 0; r < f.rows; ++r)
        if (!gone[k][(size_t)r]) {
          rows.push_back((int32_t)row_at(f.dst, r));
          if (!f.values.empty()) vals.push_back(f.values[(size_t)r]);
        }
      f.rows = (int64_t)rows.size();
      f.values = std::move(vals);
      f.dst.idx = std::move(rows);
      G[k].skip = f.rows == 0;
    }
  }

  // Fed rows that only increments and filters read, after the feed in the step:
  // those read the feed places themselves.
  void drop_feeds(std::vector<int32_t>& feed_of) {
    for (int32_t k = 0; k < (int32_t)G.size(); ++k) {
      const LGroup& g = G[k].g;
      if (g.type != OP_FEED || G[k].skip) continue;
      bool ok = true;
      for (int64_t r = 0; r < g.rows && ok; ++r) {
        const int64_t d = row_at(g.dst, r);
        ok = writers[d].size() == 1 && !probed[d];
        for (int32_t q : readers[d]) {
          const OpType t = G[q].g.type;
          ok = ok && q > k && (t == OP_COPY || t == OP_COPY_INC || t == OP_ELEM_INC || t == OP_LOWPASS);
        }
      }
      if (!ok) continue;
      for (int64_t r = 0; r < g.rows; ++r) feed_of[row_at(g.dst, r)] = g.feed_rows[(size_t)r];
      G[k].skip = true;
    }
  }

  // Copies of whole rows whose readers, later in the step, find the source
  // unchanged: they read it instead.
  void drop_copies() {
    std::vector<int32_t> alias((size_t)nrows, -1), both;
    for (int32_t k = 0; k < (int32_t)G.size(); ++k) {
      const LGroup& g = G[k].g;
      if (G[k].skip || !batched(g.src)) continue;
      if (!(g.type == OP_COPY || (g.type == OP_COPY_INC && G[k].init && G[k].vals.empty() && entries(g) == g.rows))) continue;
      std::vector<int32_t> rd;
      bool ok = true;
      for (int64_t r = 0; r < g.rows && ok; ++r) {
        const int64_t d = row_at(g.dst, r), s = row_at(g.src, r);
        ok = writers[d].size() == 1 && !probed[d];
        for (int32_t q : readers[d]) {
          if (q <= k) ok = false;   // reads the previous step's value
          for (int32_t wk : writers[s]) if (wk > k && wk <= q) ok = false;
        }
      }
      if (!ok) continue;
      for (int64_t r = 0; r < g.rows; ++r) {
        const int64_t d = row_at(g.dst, r);
        alias[d] = (int32_t)row_at(g.src, r);
        rd.insert(rd.end(), readers[d].begin(), readers[d].end());
      }
      std::sort(rd.begin(), rd.end());
      rd.erase(std::unique(rd.begin(), rd.end()), rd.end());
      std::vector<Item> saved;
      for (size_t i = 0; i < rd.size() && ok; ++i) {
        saved.push_back(G[rd[i]]);
        ok = rewrite(G[rd[i]].g, alias);
      }
      if (ok) {   // the sources' readers are now the copies' readers as well, but not group k
        G[k].skip = true;
        for (int64_t r = 0; r < g.rows; ++r) {
          const int64_t d = row_at(g.dst, r);
          readers[row_at(g.src, r)].take(readers[d], k, both);
          readers[d].n = writers[d].n = 0;
        }
      } else {
        for (size_t i = 0; i < saved.size(); ++i) G[rd[i]] = saved[i];
      }
      for (int64_t r = 0; r < g.rows; ++r) alias[row_at(g.dst, r)] = -1;
    }
  }

  bool rewrite(LGroup& g, const std::vector<int32_t>& alias) const {
    auto runs = [&](std::vector<int32_t>& first, int32_t len) {
      for (int32_t& x : first) {
        if (x < 0 || len == 0) continue;
        const int32_t y = alias[x] >= 0 ? alias[x] : x;
        for (int32_t q = 1; q < len; ++q)
          if ((alias[x + q] >= 0 ? alias[x + q] : x + q) != y + q) return false;
        x = y;
      }
      return true;
    };
    if (g.type == OP_ENS) return runs(g.ens_x, g.ens_d);
    if (g.type == OP_DOT_INC) return runs(g.x_row, g.K);
    std::vector<int32_t> rows;
    for (int64_t e = 0; e < entries(g); ++e) {
      const int64_t r = row_at(g.src, e);
      rows.push_back(alias[r] >= 0 ? alias[r] : (int32_t)r);
    }
    g.src.idx = std::move(rows);
    return true;
  }
};

}  // namespace

ResProgram make_resident(const Plan& p, int32_t B, int64_t lds_bytes, bool graph_order,
                         const std::vector<std::vector<float>>* params) {
  ResProgram R;
  auto no = [&](const char* why) { R.why = why; return R; };
  const IR& ir = p.ir;
  auto batched = [&](const LOperand& o) { return o.base >= 0 && ir.bases[o.base].cls == SC_BATCHED; };
  int64_t nrows = 0;
  for (size_t b = 0; b < ir.bases.size(); ++b)
    if (ir.bases[b].cls == SC_BATCHED) nrows = p.base_rows[b];
  if (nrows == 0) return no("no batched signals");
  std::vector<std::vector<float>> base(ir.bases.size());
  auto param = [&](int32_t b) -> const std::vector<float>& {
    if (params) return (*params)[(size_t)b];
    std::vector<float>& v = base[(size_t)b];
    if (v.empty()) {
      v.assign((size_t)std::max<int64_t>(1, p.base_rows[b] * ir.bases[b].cols), 0.0f);
      for (size_t k = 0; k < ir.sigs.size(); ++k)
        if (ir.sigs[k].base == b)
          for (size_t j = 0; j < ir.sigs[k].value.size(); ++j)
            v[(size_t)(p.sig_offset[k] * ir.bases[b].cols) + j] = (float)ir.sigs[k].value[j];
    }
    return v;
  };
  // ---- is the model of the kind the kernel runs
  const LGroup* first = nullptr;
  int64_t slots = 0, tree = 0, dot = 0;   // work of the products: units of 8 rows, columns taken one by one
  R.d = R.ndec = 1;
  for (const LGroup& g : p.lowered) {
    switch (g.type) {
      case OP_FEED: case OP_RESET: case OP_LOWPASS: case OP_COPY: case OP_COPY_INC: break;
      case OP_ELEM_INC:
        if (batched(g.a) || !batched(g.src)) return no("an elementwise product of two batched rows");
        break;
      case OP_DOT_INC:
        if (batched(g.a) || ir.bases[g.a.base].cols != g.K) return no("a product with batched or strided weights");
        if (graph_order && g.K > 128) return no("a long product, which many workgroups share better");
        if (g.K >= 64 && graph_order && B <= 4) tree += g.rows * (int64_t)((g.M + 7) / 8);
        else if (graph_order) dot += g.rows * (int64_t)((g.M + 63) / 64) * g.K;
        break;
      case OP_ENS: {
        int32_t nd = 0;
        for (int32_t d : g.ens_df) nd += d;
        if (g.ens_type != MS_NEURON_LIF) return no("rate neurons");
        if (g.ens_d > kResD || nd < 1 || nd > kResDec) return no("an ensemble of more dimensions or decoded outputs, or none");
        if (g.tau_rc.size() > 1 || g.tau_ref.size() > 1 || g.amp.size() > 1) return no("neuron parameters differ");
        if (!first) first = &g;
        if (g.tau_rc[0] != first->tau_rc[0] || g.tau_ref[0] != first->tau_ref[0] || g.amp[0] != first->amp[0])
          return no("neuron parameters differ between ensembles");
        R.d = std::max(R.d, g.ens_d);
        R.ndec = std::max(R.ndec, nd);
        for (int32_t n : g.ens_n) {
          if (graph_order && n > 256) return no("an ensemble of more than 256 neurons");
          slots += (n + 63) / 64;
          ++R.ensembles;
        }
        break;
      }
      default: return no("an operator the resident kernel does not run");
    }
  }
  if (!first) return no("no ensembles");
  // against the launch drivers, which spread products over the whole chip: at
  // most 16 units (about 3 us a step) or 64 columns a wavefront, and few columns
  if (graph_order && (B >= 8 || tree > 16 * kResWaves || dot > 64 * kResWaves)) return no("products too large for one workgroup");
  if (!((float)p.dt * (float)(1.0 / (double)first->tau_rc[0]) <= 0.0625f)) return no("a step past tau_rc / 16");
  if (R.d > 1 || R.ndec > 1) R.d = kResD, R.ndec = kResDec;   // the two forms the kernel is compiled for
  // (found out before any table is built; by wavefront, it is checked once the
  // ensembles have theirs)
  if (slots > (int64_t)kResWaves * (R.d == 1 ? kResSlots[2] : kResSlots[1])) return no("more neurons than the wavefronts' registers hold");
  R.tau_rc = first->tau_rc[0]; R.tau_ref = first->tau_ref[0]; R.amp = first->amp[0];
  R.chunks = (int32_t)slots;
  R.waves = (int32_t)std::min<int64_t>(kResWaves, std::max<int64_t>(1, (slots + 3) / 4));   // about four slots each
  if (ir.feed_rows > 2 * 64 * R.waves) return no("more feed rows than the workgroup fetches ahead");
  std::vector<Item> G;
  for (const LGroup& g : p.lowered) G.push_back({g, false, false, {}});
  Prep P{p, G, nrows, std::vector<char>((size_t)nrows, 0), {}, {}};
  for (int32_t r : p.probe_src_rows) P.probed[(size_t)r] = 1;
  P.index();
  P.start_increments();
  P.index();
  P.drop_copies();
  std::vector<int32_t> feed_of((size_t)nrows, -1);
  P.drop_feeds(feed_of);
  // ---- levels, and places in row order for every row used; place 0 holds 1.0
  // and place 1 zero
  std::vector<char> state((size_t)nrows, 0);
  for (const LGroup& g : p.lowered)
    if (g.type == OP_ENS)
      for (size_t o = 0; o < g.ens_n.size(); ++o)
        for (int32_t r = 0; r < g.ens_n[o]; ++r) state[(size_t)(g.ens_V[o] + r)] = state[(size_t)(g.ens_ref[o] + r)] = 1;
  std::vector<int32_t> wl((size_t)nrows, -1), rl((size_t)nrows, -1), place((size_t)nrows, -1), level(G.size(), -1);
  int32_t nlev = 0;
  for (size_t k = 0; k < G.size(); ++k) {
    if (G[k].skip) continue;
    int32_t lv = 0;
    P.each_read(G[k].g, [&](int64_t r) { lv = std::max(lv, wl[r] + 1); });
    P.each_write(G[k].g, [&](int64_t r) { lv = std::max(lv, std::max(wl[r], rl[r]) + 1); });
    P.each_read(G[k].g, [&](int64_t r) { rl[r] = std::max(rl[r], lv); place[(size_t)r] = 0; });
    P.each_write(G[k].g, [&](int64_t r) { wl[r] = std::max(wl[r], lv); place[(size_t)r] = 0; });
    level[k] = lv;
    nlev = std::max(nlev, lv + 1);
  }
  for (int32_t r : p.probe_src_rows) place[(size_t)r] = 0;
  R.row_of.push_back(-1);
  R.row_of.push_back(-1);
  for (int64_t r = 0; r < nrows; ++r) {
    if (place[(size_t)r] < 0 || feed_of[(size_t)r] >= 0) continue;
    if (state[(size_t)r]) return no("neuron state read as a signal");
    place[(size_t)r] = (int32_t)R.row_of.size();
    R.row_of.push_back((int32_t)r);
  }
  if ((int64_t)R.row_of.size() + ir.feed_rows >= 65536) return no("more rows than 16-bit places");
  auto at = [&](int64_t row) { return place[(size_t)row]; };
  // an operand: a place, or a feed place (which moves with the step)
  auto src_at = [&](int64_t row) { return feed_of[(size_t)row] >= 0 ? feed_of[(size_t)row] | kResFeed : at(row); };
  auto together = [&](int64_t row, int64_t n) {   // n rows at consecutive places
    for (int64_t q = 1; q < n; ++q) if (at(row + q) != at(row) + q) return false;
    return true;
  };
  // k_persistent takes a product's sums in parts
  auto parts_of = [&](const LGroup& g) {
    const int64_t out = g.rows * (int64_t)g.M, threads = nrows <= 4096 ? 256 : 1024;
    int32_t parts = 1;
    while (!graph_order && parts < 64 && out * parts * 2 <= threads && parts * 2 <= g.K) parts *= 2;
    return parts;
  };
  auto tree_sums = [&](const LGroup& g) { return graph_order && g.K >= 64 && B <= 4; };
  // ---- wavefronts: also about two entries of the level with the most rows and
  // products (16 columns of a product count as one more), or of the probes.  By
  // the neurons alone one ensemble of 50 neurons had one wavefront: beside a
  // product of 500 x 500 a step took 279 us (k_persistent 99), with eight 38.
  std::vector<double> busy((size_t)nlev, 0.0);
  for (size_t k = 0; k < G.size(); ++k) {
    if (G[k].skip || G[k].g.type == OP_ENS) continue;
    const LGroup& g = G[k].g;
    double e = (double)g.rows / 64;
    if (g.type == OP_DOT_INC && tree_sums(g)) {
      e = (double)g.rows * ((g.M + 7) / 8);
    } else if (g.type == OP_DOT_INC) {
      const int32_t parts = parts_of(g);
      e *= (double)g.M * parts * (1.0 + (double)((g.K + parts - 1) / parts) / 16);
    }
    busy[(size_t)level[k]] += e;
  }
  const double most_busy = std::max(*std::max_element(busy.begin(), busy.end()), (double)p.probe_src_rows.size() / 64);
  R.waves = std::max(R.waves, (int32_t)std::min<double>(kResWaves, std::ceil(most_busy / 2)));
  // ---- tables
  struct Slot { int32_t x = 0, d = 0, s = -1, n = 0, flags = 0, V = 0, ref = 0; std::vector<float> enc, bias, dec; };
  std::vector<std::vector<Slot>> ws((size_t)R.waves);
  typedef std::array<int32_t, 4> Entry;
  std::vector<std::vector<Entry>> sched((size_t)R.waves);
  for (int32_t lv = 0; lv < nlev; ++lv) {
    std::vector<size_t> lo;
    for (const auto& w : ws) lo.push_back(w.size());
    std::vector<std::vector<Entry>> rest((size_t)R.waves);
    // 64-item pieces to the wavefronts in turn, the least busy one first
    auto least = [&]() {
      size_t w = 0;
      for (size_t q = 1; q < rest.size(); ++q)
        if (rest[q].size() < rest[w].size()) w = q;
      return w;
    };
    auto chunk = [&](int32_t type, int32_t M, int32_t parts, const std::vector<std::array<int32_t, 4>>& it) {
      for (size_t i = 0; i < it.size(); i += 64) {
        const size_t n = std::min<size_t>(64, it.size() - i);
        rest[least()].push_back({type, (int32_t)R.items.size(), (int32_t)n, M | parts << 24});
        R.items.insert(R.items.end(), it.begin() + (int64_t)i, it.begin() + (int64_t)(i + n));
      }
    };
    std::vector<std::array<int32_t, 4>> simple, sum4;   // of every group of the level
    struct Unit { int32_t d, x, K, w, n, init; };
    std::vector<Unit> units;   // products summed across a wavefront: up to 8 rows each
    for (size_t k = 0; k < G.size(); ++k) {
      if (G[k].skip || level[k] != lv) continue;
      const LGroup& g = G[k].g;
      const Item& gi = G[k];
      std::vector<std::array<int32_t, 4>> it;
      switch (g.type) {
        case OP_FEED:   // d = 1 src - 0, which keeps the sign of a zero
          for (int64_t r = 0; r < g.rows; ++r)
            simple.push_back({at(row_at(g.dst, r)), g.feed_rows[(size_t)r] | kResFeed | kResInit, bits(1.0f), bits(-0.0f)});
          break;
        case OP_RESET:  // d = -0 place 0 + value
          for (int64_t r = 0; r < g.rows; ++r)
            simple.push_back({at(row_at(g.dst, r)), kResInit, bits(-0.0f), bits(g.values.empty() ? 0.0f : g.values[(size_t)r])});
          break;
        case OP_COPY:
          for (int64_t r = 0; r < g.rows; ++r) {
            if (batched(g.src)) simple.push_back({at(row_at(g.dst, r)), src_at(row_at(g.src, r)) | kResInit, bits(1.0f), bits(-0.0f)});
            else simple.push_back({at(row_at(g.dst, r)), kResInit, bits(-0.0f), bits(param(g.src.base)[(size_t)row_at(g.src, r)])});
          }
          break;
        case OP_COPY_INC: case OP_ELEM_INC:
          for (int64_t r = 0; r < g.rows; ++r) {
            const int64_t e0 = g.ptr.empty() ? r : g.ptr[(size_t)r], e1 = g.ptr.empty() ? r + 1 : g.ptr[(size_t)r + 1];
            const int32_t d = at(row_at(g.dst, r)), start = bits(gi.vals.empty() ? 0.0f : gi.vals[(size_t)r]);
            // entries {place, factor}: a factor of 1 makes the fma an add, and
            // a parameter to add is the factor of place 0, which holds 1.0
            std::vector<std::pair<int32_t, int32_t>> en;
            bool adds = true;   // plain adds of places: up to four go into one item
            for (int64_t e = e0; e < e1; ++e) {
              const bool bt = batched(g.src);
              const int32_t f = bits(g.type == OP_ELEM_INC ? param(g.a.base)[(size_t)row_at(g.a, e)]
                                     : bt                  ? 1.0f
                                                           : param(g.src.base)[(size_t)row_at(g.src, e)]);
              en.push_back({bt ? src_at(row_at(g.src, e)) : 0, f});
              // by type and not by the factor's value, which may be set later
              adds = adds && bt && g.type == OP_COPY_INC && !(en.back().first & kResFeed);
            }
            if (en.size() == 1) {
              simple.push_back({d, en[0].first | (gi.init ? kResInit : 0), en[0].second, start});
            } else if (adds && en.size() <= 4 && gi.init && start == 0) {
              while (en.size() < 4) en.push_back({1, 0});
              sum4.push_back({d, en[0].first | en[1].first << 16, en[2].first | en[3].first << 16, 0});
            } else {
              it.push_back({d, (int32_t)(R.entries.size() / 2), (int32_t)en.size() | (gi.init ? kResInit : 0), start});
              for (const auto& q : en) {
                R.entries.push_back(q.first);
                R.entries.push_back(q.second);
              }
            }
          }
          chunk(RES_INC, 0, 0, it);
          break;
        case OP_LOWPASS:
          for (int64_t r = 0; r < g.rows; ++r)
            simple.push_back({at(row_at(g.dst, r)), src_at(row_at(g.src, r)) | kResLowpass,
                              bits(g.ca.size() > 1 ? g.ca[(size_t)r] : g.ca[0]), bits(g.cb.size() > 1 ? g.cb[(size_t)r] : g.cb[0])});
          break;
        case OP_DOT_INC: {
          const std::vector<float>& W = param(g.a.base);
          for (int64_t o = 0; o < g.rows; ++o)
            if (!together(g.x_row[o], g.K) || !together(g.d_row[o], g.M)) return no("a product whose rows are apart");
          if (tree_sums(g)) {   // rows of W across the lanes
            for (int64_t o = 0; o < g.rows; ++o)
              for (int32_t m = 0; m < g.M; m += 8) {
                const int32_t n = std::min(8, g.M - m);
                units.push_back({at((int64_t)g.d_row[o] + m), at(g.x_row[o]), g.K, (int32_t)R.weights.size(), n, gi.init});
                for (int32_t q = 0; q < 8; ++q)   // [row][128], zero past the rows and K
                  for (int32_t c = 0; c < 128; ++c)
                    R.weights.push_back(q < n && c < g.K ? W[(size_t)((g.w_row[o] + m + q) * (int64_t)g.K + c)] : 0.0f);
              }
            break;
          }
          const int32_t parts = parts_of(g);   // a row per lane, W transposed
          for (int64_t o = 0; o < g.rows; ++o) {
            const int32_t off = (int32_t)R.weights.size();
            for (int32_t q = 0; q < g.K; ++q)
              for (int32_t m = 0; m < g.M; ++m) R.weights.push_back(W[(size_t)((g.w_row[o] + m) * (int64_t)g.K + q)]);
            // a lane per (row, part), a row's parts in consecutive lanes
            std::vector<std::array<int32_t, 4>> io;
            const int32_t len = (g.K + parts - 1) / parts;
            for (int32_t m = 0; m < g.M; ++m)
              for (int32_t q = 0; q < parts; ++q) {
                const int32_t q0 = std::min(g.K, q * len), n = std::min(g.K, q0 + len) - q0;
                io.push_back({at((int64_t)g.d_row[o] + m) | (gi.init ? kResInit : 0), at(g.x_row[o]) + q0, n, off + q0 * g.M + m});
              }
            if (g.M >= 1 << 24) return no("a product of too many rows");
            chunk(RES_DOT, g.M, parts, io);
          }
          break;
        }
        case OP_ENS:
          for (size_t o = 0; o < g.ens_n.size(); ++o) {
            size_t w = 0;   // the wavefront with the fewest slots
            for (size_t q = 1; q < ws.size(); ++q)
              if (ws[q].size() < ws[w].size()) w = q;
            const int32_t n = g.ens_n[o], d = g.ens_x[o] >= 0 ? g.ens_d : 0, nch = (n + 63) / 64;
            int32_t nd = 0;
            const int32_t drow = at(g.ens_dd[0][o]);
            for (size_t f = 0; f < g.ens_df.size(); ++f)
              for (int32_t q = 0; q < g.ens_df[f]; ++q, ++nd)
                if (at((int64_t)g.ens_dd[f][o] + q) != drow + nd) return no("decoded outputs apart");
            if (d > 0 && !together(g.ens_x[o], d)) return no("an input whose rows are apart");
            if (g.ens_s[o] >= 0 && !together(g.ens_s[o], n)) return no("neuron outputs apart");
            for (int32_t c = 0; c < nch; ++c) {
              Slot t;
              t.x = d > 0 ? at(g.ens_x[o]) : 0;
              t.d = drow;
              t.n = std::min(64, n - 64 * c);
              t.flags = (c == 0 ? 1 : 0) | (c + 1 == nch ? 2 : 0) | (nd << 2) | (d << 8) | (c << 12);
              t.s = g.ens_s[o] >= 0 ? at(g.ens_s[o]) + 64 * c : -1;
              t.V = g.ens_V[o] + 64 * c;
              t.ref = g.ens_ref[o] + 64 * c;
              t.enc.assign((size_t)(64 * R.d), 0.0f);
              t.bias.assign(64, 0.0f);
              t.dec.assign((size_t)(64 * R.ndec), 0.0f);
              for (int32_t r = 0; r < t.n; ++r) {
                const int64_t i = 64 * c + r;
                t.bias[(size_t)r] = param(g.ens_bias_base)[(size_t)(g.ens_bias[o] + i)];
                for (int32_t q = 0; q < d; ++q)
                  t.enc[(size_t)(64 * q + r)] = param(g.a.base)[(size_t)((g.ens_enc[o] + i) * g.ens_d + q)];
                int32_t qd = 0;
                for (size_t f = 0; f < g.ens_df.size(); ++f) {
                  const int64_t cols = ir.bases[g.ens_Dbase[f]].cols;
                  for (int32_t q = 0; q < g.ens_df[f]; ++q, ++qd)
                    t.dec[(size_t)(64 * qd + r)] = param(g.ens_Dbase[f])[(size_t)(((int64_t)g.ens_D[f][o] + q) * cols + i)];
                }
              }
              ws[w].push_back(std::move(t));
            }
          }
          break;
        default: return no("an operator the resident kernel does not run");
      }
    }
    chunk(RES_SUM4, 0, 0, sum4);
    chunk(RES_SIMPLE, 0, 0, simple);
    for (size_t w = 0; w < sched.size(); ++w) {
      std::vector<Entry> e;
      if (ws[w].size() > lo[w]) e.push_back({RES_ENS, 0, (int32_t)lo[w], (int32_t)ws[w].size()});
      const size_t u0 = units.size() * w / sched.size(), u1 = units.size() * (w + 1) / sched.size();
      if (u1 > u0) {
        e.push_back({RES_TREE, 0, (int32_t)(R.units.size() / 4), (int32_t)(u1 - u0)});
        for (size_t u = u0; u < u1; ++u) {
          const Unit& q = units[u];
          R.units.insert(R.units.end(), {q.d | q.n << 20 | (q.init ? 1 << 28 : 0), q.x, q.K, q.w});
        }
      }
      e.insert(e.end(), rest[w].begin(), rest[w].end());
      if (e.empty()) e.push_back({RES_NONE, 0, 0, 0});
      e.back()[0] |= kResBar | (lv + 1 == nlev ? kResPut : 0);
      sched[w].insert(sched[w].end(), e.begin(), e.end());
    }
  }
  size_t most = 0;
  for (const auto& w : ws) most = std::max(most, w.size());
  for (int32_t s : kResSlots)
    if (R.slots == 0 && most <= (size_t)s && (s <= 16 || R.d == 1)) R.slots = s;
  if (R.slots == 0) return no("more neurons than the wavefronts' registers hold");
  // a wavefront's list sits in its lanes: entry i in lane i, one more past the end
  for (auto& w : sched) {
    if (w.size() > 63) return no("more entries a step than lanes");
  }
  for (auto& w : sched) {
    const size_t n = w.size();
    w.resize(64, {RES_NONE, 0, 0, 0});
    for (const Entry& e : w) R.sched.insert(R.sched.end(), e.begin(), e.end());
    R.sched_n.push_back((int32_t)n);
  }
  // probes read their rows after the last level: a barrier has to stand between
  // them and the next step's first level only if that level writes one of them
  for (int32_t r : p.probe_src_rows) R.probe_at.push_back(at(r));
  for (size_t k = 0; k < G.size(); ++k)
    if (level[k] == 0) P.each_write(G[k].g, [&](int64_t r) { R.probe_barrier |= P.probed[(size_t)r]; });
  // per (wavefront, slot): record and parameters (unused: a neuron that never spikes)
  for (int32_t w = 0; w < R.waves; ++w)
    for (int32_t s = 0; s < R.slots; ++s) {
      Slot t;
      t.enc.assign((size_t)(64 * R.d), 0.0f);
      t.bias.assign(64, 0.0f);
      t.dec.assign((size_t)(64 * R.ndec), 0.0f);
      if (s < (int32_t)ws[(size_t)w].size()) t = ws[(size_t)w][(size_t)s];
      if ((t.flags >> 12) > 0) R.multi = 1;
      if (t.s >= 0) R.spikes = 1;
      R.slot_rec.insert(R.slot_rec.end(), {t.x, t.d, t.s, t.n, t.flags, t.V, t.ref, 0});
      R.slot_par.insert(R.slot_par.end(), t.enc.begin(), t.enc.end());
      R.slot_par.insert(R.slot_par.end(), t.bias.begin(), t.bias.end());
      R.slot_dec.insert(R.slot_dec.end(), t.dec.begin(), t.dec.end());
    }
  R.split_sums = graph_order ? 1 : 0;
  // items are fetched ahead for entries of any kind: 64 past the last stay in range
  R.items.resize(R.items.size() + 64, {0, 0, 0, 0});
  // LDS of k_resident: rows, two steps of feed rows, chunk sums, then (16-byte
  // aligned) items, units, slot records, decoders, entries
  const int64_t nslot = (int64_t)R.waves * R.slots;
  if (R.units.empty()) R.units.assign(4, 0);
  R.lds = ((int64_t)R.row_of.size() + 2 * ir.feed_rows + nslot * R.ndec + 3) / 4 * 16 + (int64_t)R.items.size() * 16 +
          (int64_t)R.units.size() * 4 + nslot * 32 + (int64_t)R.slot_dec.size() * 4 + (int64_t)R.entries.size() * 4;
  if (R.lds > lds_bytes) return no("rows and tables past the LDS");
  if ((int64_t)R.weights.size() > (1 << 20)) return no("products too large for one workgroup");
  // k_persistent runs models of more than 4096 rows on 1024 threads, which take
  // large products better than 512, while its ensembles are the slower ones: with
  // 300 x 300 weights 30 ensembles of 100 neurons take 25.8 us a step on it, 27.3
  // here, 300 of 64 50.3 and 33.9; with 500 x 500 the 30 take 36 and 48, with 500 x
  // 100 0.88 times as long here.  Smaller models run on 256 threads there, and
  // several columns share a CU, where 16 slots' registers let one column alone have
  // it: with 300 columns 4 ensembles of 400 neurons and 500 x 100 weights 35 and
  // 46, with 100 x 100 level, with 64 columns half as long here.
  int64_t nweight = 0;
  for (const LGroup& g : p.lowered)
    if (g.type == OP_DOT_INC) nweight += g.rows * (int64_t)g.M * g.K;
  if (!graph_order && (nrows > 4096 ? nweight > 48 * 1024 + 300 * (int64_t)R.chunks
                                    : B > 256 && R.slots > kResSlots[0] && nweight > 8192))
    return no("products that k_persistent runs faster");
  R.ok = true;
  return R;
}

// A step of the launch drivers takes about 2.2 us a launch and 2 us more, so the
// program is the faster one past three launches: 5 of them take 11.7 to 16.8 us, the
// same models 4.5 to 9.6 with it.  Two or three (one fused ensemble launch, one
// of synapses, the feed's) use the whole chip for 7.2 or 10.4 us, about 2 more
// where the ensembles' workgroups no longer fit at once (1024 of 256 threads).
// The program's step grows with the chunks a wavefront holds, by the form of its
// neurons, and with its items.  Of 388 models of two or three launches measured
// on both (80 to 320 chunks, 1 to 7 columns, 1 to 16 connections an ensemble),
// those this lets through are up to twice as fast and one is slower, by 3%
// (8.08, 7.87 us); a ring of 320 ensembles of 50 neurons takes 7.7 us with the
// program and 7.3 as launches, 80 of 250 9.7 and 7.1, 160 of 50 5.3 and 7.1.
bool resident_beats_launches(const Plan& p, int32_t B, const ResProgram& r) {
  const size_t launches = make_launch_plan(p).step.size();
  if (launches > 3) return true;
  const double per_wave = (r.chunks + r.waves - 1) / r.waves;
  const double neurons = r.d == 2 ? 4.8 + per_wave * (r.spikes ? 0.09 : 0.055)
                         : r.spikes ? 3.7 + per_wave * 0.19
                                    : 2.5 + per_wave * (r.multi ? 0.17 : 0.12);
  return neurons + 0.0005 * (double)(r.items.size() + r.entries.size() / 2) <=
         (launches == 3 ? 10.4 : 7.2) + ((int64_t)r.ensembles * B > 1024 ? 2.2 : 0.0);
}

}  // namespace ms
