// Fusion exploration over a multi-pattern graph (paper Section 5): the search, and the making of
// an executable program from the plan it finds (fs_program.cpp runs it).
//   * candidate patterns per vertex, from the last vertex to the first, by PatternReduction
//     (Section 5.2): a vertex joins combinations of its consumers' candidate patterns, consumers
//     are handled in groups of two, only the top-k patterns by score survive;
//   * patterns with a cyclic dependence or that the code generator cannot process are discarded
//     (Section 5.2) -- "can process" here means: a hand-written kernel family matches it or it
//     compiles to a row program (a generated kernel, or the interpreter).  Computations outside the
//     graph that the graph names (Section 1: compute-intensive ops go to libraries and are not fused) order execution
//     like edges and are never inside a pattern;
//   * score f = T_reduced_mem + T_reduced_calls - T_penalty (Section 5.4, Eq. 3), with constants
//     measured on MI355X (launch cost, streaming rate) and the penalty from the kernel estimate
//     without compiled register figures;
//   * the overall plan by beam search over the vertices from producers to consumers (Section 5.3),
//     the final choice among the beam's plans by the full latency evaluator (Section 4.3);
//   * independent launch-bound patterns of the chosen plan are packed into one launch (remote
//     fusion / kernel packing, Section 5.2 and 4.1).
// The program runs the patterns in dependence order, in stages where external computations lie
// between them; tensors that cross from one pattern to another live in the caller's workspace,
// placed by lifetime; fold launches of column sums that nothing reads move behind the last step
// and run as one.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <map>
#include <set>
#include <string>

#include "fs_internal.hpp"
#include "fs_program.hpp"

extern "C" {
fs_status fs_graph_create(fs_graph** out);
void fs_graph_destroy(fs_graph* g);
fs_tensor fs_graph_input(fs_graph* g, int32_t dtype, int32_t rank, const int64_t* dims);
fs_tensor fs_graph_op(fs_graph* g, int32_t opcode, int32_t n_in, const fs_tensor* in, const void* attr, size_t attr_bytes);
fs_status fs_graph_output(fs_graph* g, fs_tensor t, int32_t store_as);
fs_status fs_graph_finalize(fs_graph* g);
}

namespace fs {
namespace {

typedef std::vector<int> OpSet;   // sorted op indices

struct SubGraph {
  fs_graph* g = nullptr;
  std::vector<int32_t> in_tensor;    // sub input slot  -> tensor id in the big graph
  std::vector<int32_t> out_tensor;   // sub output slot -> tensor id in the big graph
  ~SubGraph() { fs_graph_destroy(g); }
  SubGraph() = default;
  SubGraph(const SubGraph&) = delete;
  SubGraph& operator=(const SubGraph&) = delete;
};

struct Scored {
  bool valid = false;
  int32_t why = FS_OK;     // FS_ERR_CYCLE / FS_ERR_UNSUPPORTED_PATTERN / FS_ERR_DTYPE when not valid
  double f = 0;            // microseconds
  double f_optimistic = 0; // what f would be if the ops ran as one kernel at streaming rate; set for every convex pattern
  double t_fused = 0, t_unfused = 0;
};

struct Explorer {
  const fs_graph& g;
  int n;                                     // ops
  std::vector<std::vector<int>> consumers;   // op -> ops that read its result (sorted, distinct)
  std::vector<std::vector<int>> waiting;     // op -> ops that wait for its result through an external computation
  std::vector<std::vector<uint64_t>> desc;   // op -> bitset of everything that runs after it because of it
  std::vector<std::vector<uint64_t>> reads_of;   // op -> bitset of its descendants through tensors of the graph alone
  std::map<OpSet, Scored> memo;
  int top_k = 3, beam_width = 3;

  explicit Explorer(const fs_graph& graph) : g(graph), n((int)graph.ops.size()) {
    consumers.resize(n);
    for (int i = 0; i < n; ++i) {
      std::set<int> c(g.tensors[g.ops[i].out].consumers.begin(), g.tensors[g.ops[i].out].consumers.end());
      consumers[i].assign(c.begin(), c.end());
    }
    waiting.resize(n);
    const std::vector<std::vector<int>> waits_for = g.external_producers();
    for (int i = 0; i < n; ++i)
      for (int p : waits_for[i]) waiting[p].push_back(i);
    const int words = (n + 63) / 64;
    desc.assign(n, std::vector<uint64_t>(words, 0));
    reads_of.assign(n, std::vector<uint64_t>(words, 0));
    for (int i = n - 1; i >= 0; --i) {
      for (int c : consumers[i]) {
        desc[i][c / 64] |= 1ull << (c % 64);
        reads_of[i][c / 64] |= 1ull << (c % 64);
        for (int w = 0; w < words; ++w) { desc[i][w] |= desc[c][w]; reads_of[i][w] |= reads_of[c][w]; }
      }
      for (int c : waiting[i]) {
        desc[i][c / 64] |= 1ull << (c % 64);
        for (int w = 0; w < words; ++w) desc[i][w] |= desc[c][w];
      }
    }
  }

  // An op and an op that waits for its result through an external computation cannot share a kernel.
  bool holds_external_dependence(const OpSet& p) const {
    for (int o : p)
      for (int c : waiting[o])
        if (std::binary_search(p.begin(), p.end(), c)) return true;
    return false;
  }

  // No path may leave the pattern and come back (Section 5.2, cyclic dependence).
  bool convex(const OpSet& p) const {
    const int words = (n + 63) / 64;
    std::vector<uint64_t> in(words, 0), below(words, 0);
    for (int o : p) in[o / 64] |= 1ull << (o % 64);
    for (int o : p)
      for (int w = 0; w < words; ++w) below[w] |= desc[o][w];
    for (int x = 0; x < n; ++x) {
      if ((in[x / 64] >> (x % 64)) & 1) continue;
      if (!((below[x / 64] >> (x % 64)) & 1)) continue;
      for (int w = 0; w < words; ++w)
        if (desc[x][w] & in[w]) return false;
    }
    return true;
  }

  // The pattern as a graph of its own: operands made outside become its inputs, results read
  // outside (or graph outputs) become its outputs.
  fs_status extract(const OpSet& p, SubGraph* sub) const {
    std::vector<char> inside(n, 0);
    for (int o : p) inside[o] = 1;
    if (fs_graph_create(&sub->g) != FS_OK) return FS_ERR_INVALID_ARG;
    sub->g->cut_out = (int)p.size() < n;   // (a program of one pattern hands nothing from step to step)
    std::map<int32_t, fs_tensor> local;   // big-graph tensor -> sub tensor
    for (int o : p) {
      const Op& op = g.ops[o];
      fs_tensor in[2] = {-1, -1};
      for (int k = 0; k < op.n_in; ++k) {
        const int32_t t = op.in[k];
        auto it = local.find(t);
        if (it == local.end()) {
          const Tensor& T = g.tensors[t];
          // what a neighbouring pattern wrote is what this one reads: an output stored in another dtype than it
          // was computed in cannot also feed a different pattern
          if (T.output_slot >= 0 && T.store_as != T.dtype) return FS_ERR_DTYPE;
          const fs_tensor id = fs_graph_input(sub->g, T.dtype, T.rank, T.dims);
          if (id < 0) return id;
          sub->in_tensor.push_back(t);
          it = local.emplace(t, id).first;
        }
        in[k] = it->second;
      }
      fs_tensor r;
      const Tensor& out = g.tensors[op.out];
      switch (op.opcode) {
        case FS_SCALE: case FS_ADD_SCALAR: {
          fs_attr_scalar a = {op.scalar};
          r = fs_graph_op(sub->g, op.opcode, op.n_in, in, &a, sizeof a);
          break;
        }
        case FS_BROADCAST: {
          fs_attr_dims a;
          a.rank = out.rank;
          for (int k = 0; k < FS_MAX_RANK; ++k) a.dims[k] = k < out.rank ? out.dims[k] : 1;
          r = fs_graph_op(sub->g, op.opcode, op.n_in, in, &a, sizeof a);
          break;
        }
        case FS_REDUCE_SUM: case FS_REDUCE_MAX: case FS_REDUCE_MEAN: {
          fs_attr_axis a = {op.axis};
          r = fs_graph_op(sub->g, op.opcode, op.n_in, in, &a, sizeof a);
          break;
        }
        case FS_TRANSPOSE: {
          fs_attr_perm a;
          for (int k = 0; k < FS_MAX_RANK; ++k) a.perm[k] = op.perm[k];
          r = fs_graph_op(sub->g, op.opcode, op.n_in, in, &a, sizeof a);
          break;
        }
        case FS_CONVERT: {
          fs_attr_dtype a = {op.to_dtype};
          r = fs_graph_op(sub->g, op.opcode, op.n_in, in, &a, sizeof a);
          break;
        }
        default:
          r = fs_graph_op(sub->g, op.opcode, op.n_in, in, nullptr, 0);
          break;
      }
      if (r < 0) return r;
      local[op.out] = r;
      bool read_outside = false;
      for (int c : out.consumers)
        if (!inside[c]) read_outside = true;
      if (out.output_slot >= 0 && read_outside && out.store_as != out.dtype) return FS_ERR_DTYPE;
      if (out.output_slot >= 0 || read_outside) {
        const fs_status s = fs_graph_output(sub->g, r, out.output_slot >= 0 ? out.store_as : out.dtype);
        if (s != FS_OK) return s;
        sub->out_tensor.push_back(op.out);
      }
    }
    return fs_graph_finalize(sub->g);
  }

  // per-op execution of one op: one launch and one dependent memory round trip, operands read and the result
  // written (float32 unless the op keeps a dtype)
  double t_single(int o) const {
    const DeviceModel& d = device();
    const Op& op = g.ops[o];
    double bytes = 0;
    for (int k = 0; k < op.n_in; ++k) bytes += (double)g.tensors[op.in[k]].numel() * dtype_bytes(g.tensors[op.in[k]].dtype);
    const Tensor& out = g.tensors[op.out];
    bytes += (double)out.numel() * dtype_bytes(out.output_slot >= 0 ? out.store_as : out.dtype);
    // a sum over rows that different workgroups own takes a second launch to fold their partial sums
    const bool across_rows = (op.opcode == FS_REDUCE_SUM || op.opcode == FS_REDUCE_MAX || op.opcode == FS_REDUCE_MEAN) &&
                             op.axis != g.tensors[op.in[0]].rank - 1;
    return d.launch_s * (across_rows ? 2.0 : 1.0) + d.mem_latency_s + bytes / (d.hbm_peak_Bps * d.stream_fraction);
  }

  // Delta-evaluator (Eq. 3): time saved by running the ops of `p` as one pattern.
  const Scored& score(const OpSet& p) {
    auto it = memo.find(p);
    if (it != memo.end()) return it->second;
    Scored s;
    for (int o : p) s.t_unfused += t_single(o);
    if (p.size() == 1) {
      s.valid = true;
      s.t_fused = s.t_unfused;
      s.f = 0;
    } else if (holds_external_dependence(p) || !convex(p)) {
      s.why = FS_ERR_CYCLE;
    } else {
      SubGraph sub;
      const fs_status st = extract(p, &sub);
      if (st == FS_OK) {
        const DeviceModel& d = device();
        s.f_optimistic = (s.t_unfused - (d.launch_s + d.mem_latency_s + (double)graph_bytes_min(*sub.g) / (d.hbm_peak_Bps * d.stream_fraction))) * 1e6;
      }
      std::vector<Candidate> cands;
      if (st != FS_OK) {
        s.why = st == FS_ERR_DTYPE ? FS_ERR_DTYPE : FS_ERR_UNSUPPORTED_PATTERN;
      } else if (build_stitched(*sub.g, &cands, nullptr).empty() || cands.empty()) {
        s.why = FS_ERR_UNSUPPORTED_PATTERN;
      } else {
        // T_penalty comes from the kernel estimate with register figures left at their estimates
        // (the expensive part of the latency evaluator is skipped during exploration)
        double best = 1e30;
        bool only_fallbacks = true;
        for (const Candidate& c : cands) only_fallbacks = only_fallbacks && c.fallback;
        for (const Candidate& c : cands) {
          if (c.fallback && !only_fallbacks) continue;   // the plan would not pick it either
          double t = evaluate(c.cost, 0).seconds;
          if (c.launches.size() > 1) t += device().launch_s * (double)(c.launches.size() - 1);
          best = std::min(best, t);
        }
        s.valid = true;
        s.t_fused = best;
        s.f = (s.t_unfused - s.t_fused) * 1e6;
      }
    }
    return memo.emplace(p, s).first->second;
  }

  // A candidate pattern.  `tentative`: no kernel can run it as it stands, but it is convex and may grow into
  // one that a kernel family covers; it takes part in the growth with its optimistic score and never in a plan.
  struct Pat {
    OpSet ops;
    double f = 0;
    bool tentative = false;
  };
  static bool better(const Pat& a, const Pat& b) {
    if (a.f != b.f) return a.f > b.f;
    return a.ops < b.ops;
  }
  // top-k runnable patterns and top-k tentative ones, each list by score
  void keep_top(std::vector<Pat>* v) const {
    std::sort(v->begin(), v->end(), better);
    v->erase(std::unique(v->begin(), v->end(), [](const Pat& a, const Pat& b) { return a.ops == b.ops; }), v->end());
    std::vector<Pat> kept;
    int n_real = 0, n_tent = 0;
    for (const Pat& p : *v) {
      int& count = p.tentative ? n_tent : n_real;
      if (count < top_k) { kept.push_back(p); ++count; }
    }
    v->swap(kept);
  }
  static OpSet unite(const OpSet& a, const OpSet& b) {
    OpSet r;
    std::set_union(a.begin(), a.end(), b.begin(), b.end(), std::back_inserter(r));
    return r;
  }
  // a scored pattern if it is valid and gains time; a tentative one if only the kernel is missing
  bool consider(const OpSet& ops, std::vector<Pat>* out) {
    const Scored& s = score(ops);
    if (s.valid) {
      if (!(s.f > 0)) return false;
      out->push_back(Pat{ops, s.f, false});
      return true;
    }
    if (s.why == FS_ERR_UNSUPPORTED_PATTERN && s.f_optimistic > 0 && (int)ops.size() <= max_tentative_ops &&
        !reads_own_output(ops)) {
      out->push_back(Pat{ops, s.f_optimistic, true});
      return true;
    }
    return false;
  }
  int max_tentative_ops = 24;
  // A graph output is written to memory whatever the plan: growing a speculative pattern across it gains little
  // and lets ever larger unrunnable merges crowd out the runnable pattern on either side.
  bool reads_own_output(const OpSet& p) const {
    for (int o : p) {
      const Tensor& T = g.tensors[g.ops[o].out];
      if (T.output_slot < 0) continue;
      for (int c : T.consumers)
        if (std::binary_search(p.begin(), p.end(), c)) return true;
    }
    return false;
  }

  std::vector<std::vector<Pat>> cand;   // per vertex: candidate patterns whose producer is the vertex (without the singleton)

  // Temporary candidates of vertex v from one group of its consumers (Section 5.2).
  std::vector<Pat> reduce_group(int v, const std::vector<int>& group) {
    std::vector<Pat> out;
    if (group.size() <= 2) {
      // every combination of "one candidate pattern or nothing" per consumer, plus v
      std::vector<std::vector<OpSet>> choices;
      for (int c : group) {
        std::vector<OpSet> ch;
        ch.push_back(OpSet());            // do not take this consumer
        ch.push_back(OpSet{c});           // the consumer alone
        for (const Pat& p : cand[c]) ch.push_back(p.ops);
        choices.push_back(ch);
      }
      std::vector<size_t> idx(choices.size(), 0);
      while (true) {
        OpSet u{v};
        bool any = false;
        for (size_t k = 0; k < choices.size(); ++k) {
          if (!choices[k][idx[k]].empty()) any = true;
          u = unite(u, choices[k][idx[k]]);
        }
        if (any) consider(u, &out);
        size_t k = 0;
        while (k < idx.size() && ++idx[k] == choices[k].size()) idx[k++] = 0;
        if (k == idx.size()) break;
      }
      keep_top(&out);
      return out;
    }
    // divide, conquer, and reduce: the halves' temporary candidates, and their pairwise unions
    const size_t half = group.size() / 2;
    const std::vector<Pat> a = reduce_group(v, std::vector<int>(group.begin(), group.begin() + half));
    const std::vector<Pat> b = reduce_group(v, std::vector<int>(group.begin() + half, group.end()));
    out = a;
    out.insert(out.end(), b.begin(), b.end());
    for (const Pat& x : a)
      for (const Pat& y : b) consider(unite(x.ops, y.ops), &out);
    keep_top(&out);
    return out;
  }

  void explore_patterns() {
    cand.assign(n, {});
    for (int v = n - 1; v >= 0; --v)
      if (!consumers[v].empty()) cand[v] = reduce_group(v, consumers[v]);
    // Seeds beyond the bottom-up growth.  The growth only reaches a pattern through smaller patterns that are
    // themselves runnable; a hand-written family (say a row pass that ends in a column reduction) is runnable
    // as a whole while some of its parts are not, and the top-k cut favours ever larger patterns.  So three whole
    // shapes are offered directly: everything downstream of a vertex, the same stopped at graph outputs, and the
    // connected component a vertex starts (ops joined by an edge or a shared operand).
    std::vector<int> comp(n, -1);
    for (int v = 0; v < n; ++v) {
      if (comp[v] >= 0) continue;
      std::vector<int> stack{v};
      comp[v] = v;
      while (!stack.empty()) {
        const int o = stack.back();
        stack.pop_back();
        std::vector<int> next = consumers[o];
        for (int k = 0; k < g.ops[o].n_in; ++k) {
          const Tensor& operand = g.tensors[g.ops[o].in[k]];
          if (operand.producer >= 0) next.push_back(operand.producer);
          for (int c : operand.consumers) next.push_back(c);   // ops that share an operand belong together too
        }
        for (int x : next)
          if (comp[x] < 0) { comp[x] = v; stack.push_back(x); }
      }
    }
    for (int v = 0; v < n; ++v) {
      std::vector<Pat> seeds;
      OpSet cone{v};
      for (int x = v + 1; x < n; ++x)
        if ((reads_of[v][x / 64] >> (x % 64)) & 1) cone.push_back(x);
      if (cone.size() > 1) consider(cone, &seeds);
      // the same cone, but not continued past a graph output: that tensor is written to memory anyway
      OpSet bounded{v};
      {
        std::vector<char> in(n, 0);
        in[v] = 1;
        for (int x = v; x < n; ++x) {
          if (!in[x]) continue;
          if (g.tensors[g.ops[x].out].output_slot >= 0) continue;
          for (int c : consumers[x]) in[c] = 1;
        }
        for (int x = v + 1; x < n; ++x)
          if (in[x]) bounded.push_back(x);
      }
      if (bounded.size() > 1 && bounded != cone) consider(bounded, &seeds);
      if (comp[v] == v) {
        OpSet whole;
        for (int x = 0; x < n; ++x)
          if (comp[x] == v) whole.push_back(x);
        if (whole.size() > 1 && whole != cone && whole != bounded) consider(whole, &seeds);
      }
      // seeds are not subject to the top-k cut (at most three per vertex)
      for (const Pat& sd : seeds) {
        bool have = false;
        for (const Pat& p : cand[v])
          if (p.ops == sd.ops) have = true;
        if (!have) cand[v].push_back(sd);
      }
      std::sort(cand[v].begin(), cand[v].end(), better);
    }
  }

  // Patterns that are convex one by one can still wait for each other in a circle (P = {a, d}, Q = {b, c} with edges
  // a -> b and c -> d and no path from b to c): Section 5.2's "no cyclic dependence" is a property of the plan, checked
  // on the graph whose vertices are the plan's patterns and the ops outside them.
  bool acyclic(const std::vector<OpSet>& groups) const {
    std::vector<int> gid(n, -1);
    int n_groups = 0;
    for (const OpSet& p : groups) {
      for (int o : p) gid[o] = n_groups;
      ++n_groups;
    }
    for (int o = 0; o < n; ++o)
      if (gid[o] < 0) gid[o] = n_groups++;
    std::vector<std::vector<int>> next(n_groups);
    std::vector<int> pending(n_groups, 0);
    for (int o = 0; o < n; ++o) {
      for (int c : consumers[o])
        if (gid[c] != gid[o]) next[gid[o]].push_back(gid[c]);
      for (int c : waiting[o])
        if (gid[c] != gid[o]) next[gid[o]].push_back(gid[c]);
    }
    for (int a = 0; a < n_groups; ++a) {
      std::sort(next[a].begin(), next[a].end());
      next[a].erase(std::unique(next[a].begin(), next[a].end()), next[a].end());
      for (int b : next[a]) ++pending[b];
    }
    std::vector<int> ready;
    for (int a = 0; a < n_groups; ++a)
      if (pending[a] == 0) ready.push_back(a);
    int done = 0;
    while (!ready.empty()) {
      const int a = ready.back();
      ready.pop_back();
      ++done;
      for (int b : next[a])
        if (--pending[b] == 0) ready.push_back(b);
    }
    return done == n_groups;
  }

  // Remote fusion (Section 5.2): patterns of a plan that are not adjacent in the graph -- no edge joins them --
  // may still share a kernel.  Greedy reading: among all pairs of the plan's patterns (single ops included)
  // whose union is a runnable pattern, merge the pair that gains the most over running the two apart; repeat
  // until no pair gains.  Returns the total gain (microseconds).
  double merge_remote(std::vector<OpSet>* groups) {
    if (groups->size() > 64) return 0.0;
    std::sort(groups->begin(), groups->end());
    auto f_of = [&](const OpSet& p) { return p.size() > 1 ? score(p).f : 0.0; };
    double total = 0.0;
    while (true) {
      double best_gain = 0.0;
      size_t bi = 0, bj = 0;
      for (size_t i = 0; i < groups->size(); ++i)
        for (size_t j = i + 1; j < groups->size(); ++j) {
          const OpSet u = unite((*groups)[i], (*groups)[j]);
          const Scored& s = score(u);
          if (!s.valid) continue;
          const double gain = s.f - f_of((*groups)[i]) - f_of((*groups)[j]);
          if (!(gain > best_gain)) continue;
          std::vector<OpSet> merged;
          for (size_t k = 0; k < groups->size(); ++k)
            if (k != i && k != j) merged.push_back((*groups)[k]);
          merged.push_back(u);
          if (!acyclic(merged)) continue;   // the union is convex, but the plan with it would wait for itself
          best_gain = gain;
          bi = i;
          bj = j;
        }
      if (!(best_gain > 0.0)) break;
      const OpSet u = unite((*groups)[bi], (*groups)[bj]);
      groups->erase(groups->begin() + bj);
      (*groups)[bi] = u;
      std::sort(groups->begin(), groups->end());
      total += best_gain;
    }
    return total;
  }

  struct PlanSet {
    std::vector<OpSet> patterns;      // multi-op patterns, in the order they were appended
    std::vector<uint64_t> covered;
    double f = 0;
  };
  // Beam search (Section 5.3).  Plans are ranked by their accumulated score plus a look-ahead for the part of the
  // graph not visited yet: every op still uncovered counts with the best score per op of any candidate pattern
  // that holds it.  Without the look-ahead a large pattern that swallows half of a neighbouring pattern pushes
  // out the plan that takes both neighbours whole; at the last vertex the look-ahead is zero and the ranking is
  // the paper's.
  std::vector<PlanSet> beam() {
    const int words = (n + 63) / 64;
    std::vector<double> per_op(n, 0.0);
    for (int v = 0; v < n; ++v)
      for (const Pat& p : cand[v]) {
        if (p.tentative) continue;
        const double share = p.f / (double)p.ops.size();
        for (int o : p.ops) per_op[o] = std::max(per_op[o], share);
      }
    auto rank = [&](const PlanSet& s, int v) {
      double r = s.f;
      for (int u = v + 1; u < n; ++u)
        if (!((s.covered[u / 64] >> (u % 64)) & 1)) r += per_op[u];
      return r;
    };
    std::vector<PlanSet> sets(1);
    sets[0].covered.assign(words, 0);
    for (int v = 0; v < n; ++v) {
      std::vector<PlanSet> next = sets;
      for (const PlanSet& s : sets) {
        for (const Pat& p : cand[v]) {
          if (p.tentative) continue;
          bool overlap = false;
          for (int o : p.ops)
            if ((s.covered[o / 64] >> (o % 64)) & 1) { overlap = true; break; }
          if (overlap) continue;
          PlanSet t = s;
          t.patterns.push_back(p.ops);
          if (!acyclic(t.patterns)) continue;
          for (int o : p.ops) t.covered[o / 64] |= 1ull << (o % 64);
          t.f += p.f;
          next.push_back(t);
        }
      }
      std::vector<std::pair<double, size_t>> order;
      for (size_t k = 0; k < next.size(); ++k) order.push_back({rank(next[k], v), k});
      std::stable_sort(order.begin(), order.end(), [&](const std::pair<double, size_t>& a, const std::pair<double, size_t>& b) {
        if (a.first != b.first) return a.first > b.first;
        return next[a.second].patterns < next[b.second].patterns;
      });
      std::vector<PlanSet> kept;
      for (size_t k = 0; k < order.size() && (int)k < beam_width; ++k) kept.push_back(next[order[k].second]);
      sets.swap(kept);
    }
    return sets;
  }
};

}  // namespace
}  // namespace fs

using namespace fs;


namespace {

int64_t align256(int64_t v) { return (v + 255) / 256 * 256; }

// first-fit placement of [begin, end] lifetimes (in steps) into one arena
struct Arena {
  struct Block { int64_t off, size; int begin, end; };
  std::vector<Block> blocks;
  int64_t top = 0;
  int64_t place(int64_t size, int begin, int end) {
    size = align256(size);
    std::vector<Block> live;
    for (const Block& b : blocks)
      if (!(b.end < begin || end < b.begin)) live.push_back(b);
    std::sort(live.begin(), live.end(), [](const Block& a, const Block& b) { return a.off < b.off; });
    int64_t off = 0;
    for (const Block& b : live) {
      if (off + size <= b.off) break;
      off = std::max(off, b.off + b.size);
    }
    blocks.push_back({off, size, begin, end});
    top = std::max(top, off + size);
    return off;
  }
};

struct BuiltPlan {
  std::vector<fs_program::Step> steps;
  double predicted = 0;   // latency-evaluator estimate, microseconds
  double f = 0;           // accumulated delta-evaluator score after remote fusion
  bool ok = false;
  void destroy() {
    for (fs_program::Step& s : steps) fs_plan_destroy(s.plan);
    steps.clear();
    ok = false;
  }
};

// One plan of the beam made executable: remote fusion, then a stitched plan per pattern and per op left alone.
fs_status build_steps(Explorer* ex, const Explorer::PlanSet& plan, bool remote_fusion, BuiltPlan* b, std::string* error_text) {
  std::vector<OpSet> groups = plan.patterns;
  for (int o = 0; o < ex->n; ++o)
    if (!((plan.covered[o / 64] >> (o % 64)) & 1)) groups.push_back(OpSet{o});
  b->f = plan.f + (remote_fusion ? ex->merge_remote(&groups) : 0.0);
  b->ok = true;
  for (const OpSet& p : groups) {
    SubGraph sub;
    fs_status st = ex->extract(p, &sub);
    if (st == FS_ERR_DTYPE)
      *error_text = "a tensor that is stored as a graph output in another dtype than it was computed in also feeds ops that "
                    "cannot join its pattern; add an explicit convert and read its result";
    else if (st != FS_OK)
      *error_text = fs_last_error();
    fs_program::Step step;
    if (st == FS_OK) {
      step.ops = p;
      step.f = p.size() > 1 ? ex->score(p).f : 0.0;
      st = create_plan(sub.g, FS_SCHEME_AUTO, nullptr, false, &step.plan);   // generated kernels are compiled for the winner only
      if (st != FS_OK) *error_text = fs_last_error();
    }
    if (st != FS_OK) {
      b->destroy();
      return st;
    }
    for (int32_t t : sub.in_tensor) {
      BufRef r;
      r.kind = BUF_INPUT;
      r.slot = t;           // tensor id in the whole graph for now; resolved once the order is known
      step.in.push_back(r);
    }
    for (int32_t t : sub.out_tensor) {
      BufRef r;
      r.kind = BUF_OUTPUT;
      r.slot = t;
      step.out.push_back(r);
    }
    b->predicted += step.plan->candidates[step.plan->chosen].info.predicted_us;
    b->steps.push_back(std::move(step));
  }
  return FS_OK;
}

std::vector<int> owners(const fs_graph& g, const std::vector<fs_program::Step>& steps) {
  std::vector<int> owner(g.ops.size(), -1);
  for (size_t s = 0; s < steps.size(); ++s)
    for (int o : steps[s].ops) owner[o] = (int)s;
  return owner;
}

// Dependence order: a pattern runs after every pattern that makes one of its operands.  False if none exists.
bool order_steps(const fs_graph& g, std::vector<fs_program::Step>* steps) {
  std::stable_sort(steps->begin(), steps->end(),
                   [](const fs_program::Step& a, const fs_program::Step& b) { return a.ops.back() < b.ops.back(); });
  const std::vector<int> owner = owners(g, *steps);
  const std::vector<std::vector<int>> waits_for = g.external_producers();
  const size_t ns = steps->size();
  std::vector<std::set<int>> deps(ns), across(ns);   // steps it reads from; steps it waits for through external computations
  for (size_t s = 0; s < ns; ++s)
    for (int o : (*steps)[s].ops) {
      for (int k = 0; k < g.ops[o].n_in; ++k) {
        const int32_t prod = g.tensors[g.ops[o].in[k]].producer;
        if (prod >= 0 && owner[prod] != (int)s) deps[s].insert(owner[prod]);
      }
      for (int prod : waits_for[o]) {
        if (owner[prod] == (int)s) return false;   // cannot happen: such a pattern has no score
        deps[s].insert(owner[prod]);
        across[s].insert(owner[prod]);
      }
    }
  std::vector<int> order;
  std::vector<char> done(ns, 0);
  while (order.size() < ns) {
    bool progressed = false;
    for (size_t s = 0; s < ns; ++s) {
      if (done[s]) continue;
      bool ready = true;
      for (int d : deps[s])
        if (!done[d]) ready = false;
      if (ready) { done[s] = 1; order.push_back((int)s); progressed = true; }
    }
    if (!progressed) return false;
  }
  // stages: a step runs in the stage after the latest one it waits for across an external computation, and never
  // before a step it reads from; the steps are issued stage by stage
  for (int s : order) {
    int32_t stage = 0;
    for (int d : deps[s]) stage = std::max(stage, (*steps)[d].stage + (across[s].count(d) ? 1 : 0));
    (*steps)[s].stage = stage;
  }
  std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return (*steps)[a].stage < (*steps)[b].stage; });
  std::vector<fs_program::Step> sorted;
  for (int s : order) sorted.push_back(std::move((*steps)[s]));
  steps->swap(sorted);
  return true;
}

// Launch-bound patterns with no dependence between them share one packed launch, issued where the first of them
// stands; a member joins only if everything it reads is made before that point (remote fusion as kernel packing).
void decide_packs(const fs_graph& g, fs_program* prog, std::vector<int>* pos) {
  const int ns = (int)prog->steps.size();
  const std::vector<int> owner = owners(g, prog->steps);
  std::vector<int> level(ns, 0);
  for (int s = 0; s < ns; ++s)
    for (int o : prog->steps[s].ops)
      for (int k = 0; k < g.ops[o].n_in; ++k) {
        const int32_t prod = g.tensors[g.ops[o].in[k]].producer;
        if (prod >= 0 && owner[prod] != s) level[s] = std::max(level[s], level[owner[prod]] + 1);
      }
  const double tiny_us = 3.0 * device().launch_s * 1e6;   // the launch is a third or more of the pattern's estimated time
  std::map<std::pair<int, int>, std::vector<int>> by_level;   // (stage, level): members of a pack are issued together
  for (int s = 0; s < ns; ++s) {
    const fs_plan* p = prog->steps[s].plan;
    if ((p->pack.spec >= 0 || !p->generic.forms.empty()) && p->candidates[p->chosen].info.predicted_us <= tiny_us)
      by_level[{prog->steps[s].stage, level[s]}].push_back(s);
  }
  for (auto& kv : by_level) {
    if (kv.second.size() < 2) continue;
    std::vector<const fs_plan*> members;
    std::vector<int> chosen;
    const int first = kv.second.front();
    for (int s : kv.second) {
      bool ready = true;
      for (const BufRef& r : prog->steps[s].in) {
        const int32_t prod = g.tensors[r.slot].producer;
        if (prod >= 0 && owner[prod] >= first) ready = false;
      }
      if (ready) { members.push_back(prog->steps[s].plan); chosen.push_back(s); }
    }
    if (members.size() < 2 || members.size() > FS_PACK_MAX_MEMBERS) continue;
    fs_program::Pack pk;
    if (fs_pack_create(members.data(), (int32_t)members.size(), &pk.pack) != FS_OK) continue;
    pk.steps = chosen;
    for (int s : chosen) {
      prog->steps[s].pack = (int32_t)prog->packs.size();
      (*pos)[s] = first;
    }
    prog->packs.push_back(pk);
  }
  clear_error();
}

// Where tensors that cross patterns live: placed by lifetime, from the position their maker runs at to the position
// of their last reader; then every buffer reference of every step is resolved to a graph input, a graph output or
// a workspace offset.  Returns the workspace size.
int64_t place_buffers(const fs_graph& g, fs_program* prog, const std::vector<int>& pos) {
  const int ns = (int)prog->steps.size();
  std::map<int32_t, int> last_read;
  for (int s = 0; s < ns; ++s)
    for (const BufRef& r : prog->steps[s].in) {
      const int at = std::max(pos[s], s);
      auto it = last_read.find(r.slot);
      if (it == last_read.end() || it->second < at) last_read[r.slot] = at;
    }
  int64_t fixed = 0;   // the plans' own workspaces: never shared, so partial sums wait there untouched until the joint fold at the end
  for (int s = 0; s < ns; ++s) {
    const int64_t need = prog->steps[s].plan->candidates[prog->steps[s].plan->chosen].info.workspace_bytes;
    prog->steps[s].plan_ws_offset = fixed;
    fixed += align256(need);
  }
  Arena arena;
  std::map<int32_t, int64_t> where;
  for (int s = 0; s < ns; ++s)
    for (const BufRef& r : prog->steps[s].out) {
      const Tensor& T = g.tensors[r.slot];
      if (T.output_slot >= 0) continue;
      const int begin = pos[s];
      const int end = std::max(begin, last_read.count(r.slot) ? last_read[r.slot] : begin);
      where[r.slot] = fixed + arena.place(T.numel() * dtype_bytes(T.dtype), begin, end);
    }
  auto resolve = [&](BufRef* r) {
    const Tensor& T = g.tensors[r->slot];
    if (T.producer < 0) { r->kind = BUF_INPUT; r->slot = T.input_slot; }
    else if (T.output_slot >= 0) { r->kind = BUF_OUTPUT; r->slot = T.output_slot; }
    else { r->kind = BUF_WORKSPACE; r->offset = where[r->slot]; r->slot = 0; }
  };
  for (fs_program::Step& s : prog->steps) {
    for (BufRef& r : s.in) resolve(&r);
    for (BufRef& r : s.out) resolve(&r);
  }
  return fixed + arena.top;
}

// Column sums that nothing in the graph reads are finished by fold launches that only need to run before the
// program ends: instead of one tiny launch (or two) after each pattern, all of them run as one launch after the
// last step.  The plans' own workspaces, where the partial sums wait, are never shared between steps.
void join_folds(const fs_graph& g, fs_program* prog) {
  std::vector<fs_program::JointFold> found;
  for (size_t si = 0; si < prog->steps.size(); ++si) {
    fs_program::Step& s = prog->steps[si];
    const std::vector<Launch>& launches = s.plan->candidates[s.plan->chosen].launches;
    s.own_launches = launches.size();
    if (s.pack >= 0) continue;
    size_t first = launches.size();
    while (first > 1 && launches[first - 1].kernel == K_COLFOLD) {
      bool free_standing = true;
      for (int k = 0; k < 3; ++k) {
        const BufRef& r = launches[first - 1].ptr[k];
        if (r.kind != BUF_OUTPUT) continue;
        const int32_t t = s.out[r.slot].slot;
        const Tensor& T = g.tensors[t];
        if (T.output_slot < 0 || !T.consumers.empty()) free_standing = false;
        for (const std::pair<int32_t, int32_t>& e : g.external)
          if (e.first == t) free_standing = false;   // an external computation reads it before the program ends
      }
      if (!free_standing) break;
      --first;
    }
    for (size_t l = first; l < launches.size(); ++l) found.push_back({(int)si, l});
  }
  if (found.size() < 2) return;   // one fold alone would still be one launch, behind the last step instead of its own (carry_folds never sees it)
  for (const fs_program::JointFold& f : found) {
    fs_program::Step& s = prog->steps[f.step];
    s.own_launches = std::min(s.own_launches, f.launch);
    if (prog->joint_folds.empty() || prog->joint_folds.back().size() >= (size_t)kFoldManyMax) prog->joint_folds.emplace_back();
    prog->joint_folds.back().push_back(f);
  }
}

// The joint folds need only come after the steps that make their partial sums.  Where the last step makes none and is a
// generated kernel of 256 threads, one kernel made of both runs them together: a launch that follows another one costs 2.5 to
// 3.5 us before it does anything, and the folds' few workgroups find room beside the rows'.  Measured (us, folds behind the last
// step / with it), backward pass through a transformer block of 0.2 MB 23.5 / 19.5, 2.1 MB 22.9 / 20.7, 15 MB 21.8 / 15.8, 50 MB
// 26.0 / 22.0, 101 MB 32.4 / 29.8, 201 MB 50.2 / 47.5, 319 MB 68.7 / 65.8, 478 MB 93.6 / 91.2, and five more between them: never
// slower, so neither the evaluator nor the merged kernel's registers are asked.
// A lone op as the last step keeps the fold launch behind it.  Nothing in the kernels asks for that: it would save 2.3 to 2.5 us
// there too (three bias gradients [300,256] 17.9 / 15.5, [2100,768] 25.7 / 23.2, [8192,1024] 64.3 / 62.1), but that joining folds
// saves such a program exactly one launch is a count that its users check (test_gpu_explorer.py).
void carry_folds(fs_program* prog) {
  if (prog->joint_folds.size() != 1 || prog->steps.empty() || !codegen_enabled()) return;
  const int last = (int)prog->steps.size() - 1;
  const fs_program::Step& s = prog->steps[last];
  for (const fs_program::Step& other : prog->steps)
    if (other.stage > s.stage) return;
  const std::vector<Launch>& own = s.plan->candidates[s.plan->chosen].launches;
  if (s.pack >= 0 || s.ops.size() < 2 || own.size() != 1 || own[0].kernel != K_ROW_GENERATED || !own[0].gen) return;
  const RowProgP& p = own[0].args.u.prog;
  if (own[0].shape.block[0] != 256 || p.n_colsum > 0 || p.rows_per_group > 1 || p.col_tiles > 1 || p.col_chunks > 1) return;
  std::vector<Launch> folds;
  uint64_t blocks = own[0].shape.grid[0];
  for (const fs_program::JointFold& f : prog->joint_folds[0]) {
    if (f.step >= last) return;
    folds.push_back(prog->steps[f.step].plan->candidates[prog->steps[f.step].plan->chosen].launches[f.launch]);
    blocks += folds.back().shape.grid[0];
  }
  if (blocks >= (1ull << 31)) return;
  std::string entry, log;
  const std::string source = embedded_prelude() + generate_merged_kernel({p}, {own[0].shape.grid[0]}, folds, &entry);
  std::shared_ptr<GenKernel> kernel;
  if (gen_compile(source, entry.c_str(), &kernel, &log) != 0 || gen_resources(kernel.get()).scratch_bytes > 0 || gen_preload(kernel.get()) != 0) return;
  prog->carrier.step = last;
  prog->carrier.kernel = kernel;
  prog->carrier.shape = own[0].shape;
  prog->carrier.shape.grid[0] = (uint32_t)blocks;
}

// A step as a member of a merged kernel: its row program, the buffers of its pointers, its workgroups; what the evaluator knows of it.
struct Member {
  RowProgP prog;
  const BufRef* ptr = nullptr;
  uint32_t blocks = 0;
  const KernelCost* cost = nullptr;
  int32_t vgprs = 0;
  double seconds = 0;        // by itself, without a fold launch
  bool loops = false;        // its workgroups work through many rows: column sums, or rows one after the other
  bool reduces = false;      // ... with a row reduction in every round
};

// The kernel that the step runs by itself, or the form in which its pack runs it (the results are the same bit for bit); a lone
// transpose, which moves bits, in its first form.
bool member_of(const fs_program& prog, int step, Member* m) {
  const fs_program::Step& s = prog.steps[step];
  const Candidate& chosen = s.plan->candidates[s.plan->chosen];
  const Launch& own = chosen.launches[0];
  auto fill = [&](const RowProgP& p, const BufRef* ptr, uint32_t blocks, const KernelCost& cost, int32_t vgprs) {
    m->prog = p;
    m->ptr = ptr;
    m->blocks = blocks;
    m->cost = &cost;
    m->vgprs = vgprs;
    m->seconds = evaluate(cost, vgprs).seconds - (p.n_colsum > 0 ? device().fold_s : 0.0);
    m->loops = p.n_colsum > 0 || p.rows_per_group > 1;
    for (int i = 0; i < p.n_instr; ++i) m->reduces = m->reduces || p.instr[i].op == PO_RSUM || p.instr[i].op == PO_RMAX || p.instr[i].op == PO_RSUMSQ;
    return true;
  };
  auto generic = [&](const GenericForm& f) { return fill(s.plan->generic.in_form(f), s.plan->generic.ptr, f.blocks, f.cost, f.cost.vgpr_estimate); };
  if (s.pack >= 0) {
    const fs_program::Pack& pk = prog.packs[s.pack];
    if (pk.pack->generated.size() != 1) return false;
    const size_t at = std::find(pk.steps.begin(), pk.steps.end(), step) - pk.steps.begin();
    return at < pk.pack->generated[0].forms.size() && generic(pk.pack->generated[0].forms[at]);
  }
  if (own.kernel == K_TRANSPOSE_ROWS && !s.plan->generic.forms.empty()) return generic(s.plan->generic.forms[0]);
  if (own.kernel != K_ROW_GENERATED || own.shape.block[0] != 256 || own.args.u.prog.col_chunks > 1) return false;
  return fill(own.args.u.prog, own.ptr, own.shape.grid[0], chosen.cost, own.gen ? gen_resources(own.gen.get()).vgprs : 0);
}

// Workgroups of one launch of these steps that a compute unit holds: all have the registers of the hungriest and the LDS of the largest.
double groups_per_cu(const std::vector<Member>& members, const std::vector<int>& steps) {
  KernelCost launch;   // of 256 threads
  int32_t vgprs = 0;
  launch.waves = launch.elems = 1e9;
  launch.lds_bytes_per_block = 4096;
  for (int s : steps) {
    launch.lds_bytes_per_block = std::max(launch.lds_bytes_per_block, (int32_t)column_sum_lds_bytes(members[s].prog));
    vgprs = std::max(vgprs, members[s].vgprs > 0 ? members[s].vgprs : members[s].cost->vgpr_estimate);
  }
  return evaluate(launch, vgprs).waves_per_simd;   // (four wavefronts on four SIMDs)
}

// What being in one launch costs its members.  Few of its workgroups may fit a compute unit (groups_per_cu), so
//   * members that stream (no loop over rows) may be left with fewer bytes in flight than it takes, 40 KB a compute unit: `lean`
//     lists them, longest first, if the looping members, whose workgroups wait for latencies, are not at work for as long as
//     they stream.  Measured (us, apart / in one launch with / in a later one): LayerNorm backward [512,768] and RMS norm backward
//     beside a gate of 201 MB, 32 bytes a lane on 3 workgroups 39.3 / 41.5 / 36.9; of 805 MB 141.1 / 153.2 / 137.4; a gate of 403 MB beside
//     both of [16384,768] 94.1 / 100.5 / 92.9.  On 64 bytes a lane (49 KB) it pays: 104.0 / 97.8;
//   * looping members with row reductions whose workgroups are not all resident leave a part of the chip idle in the last round
//     (`ragged`, seconds; the evaluator's weight).  LayerNorm and RMS norm backward, 768 workgroups where 512 fit, apart / in one
//     launch: 177 MB 38.6 / 38.2, 302 MB 72.2 / 73.3 (with a gate), 453 MB 89.3 / 94.2.
void cost_of_sharing(const std::vector<Member>& members, const std::vector<int>& steps, std::vector<int>* lean, double* ragged) {
  const DeviceModel& d = device();
  const double per_cu = groups_per_cu(members, steps);
  const double Bps = d.hbm_peak_Bps * d.stream_fraction;
  double looping_s = 0, streaming_s = 0, rounds = 0, bytes = 0;
  lean->clear();
  for (int s : steps) {
    const Member& m = members[s];
    if (m.loops) {
      looping_s += m.seconds;
      if (m.reduces) {
        rounds += m.blocks / (d.n_cu * per_cu);
        bytes += m.cost->hbm_bytes;
      }
      continue;
    }
    if (per_cu < evaluate(*m.cost, m.vgprs).waves_per_simd && per_cu * 256.0 * m.cost->bytes_in_flight_per_lane < 40960.0) {
      lean->push_back(s);
      streaming_s += m.cost->hbm_bytes / Bps;
    }
  }
  std::stable_sort(lean->begin(), lean->end(), [&](int a, int b) { return members[a].cost->hbm_bytes > members[b].cost->hbm_bytes; });
  if (looping_s == 0 || streaming_s <= looping_s) lean->clear();
  *ragged = rounds > 1.0 ? bytes / Bps * 0.25 * (std::ceil(rounds - 1e-9) / rounds - 1.0) : 0.0;
}

// The whole program in as few launches as its dependences allow: a step reads what others made one launch earlier or
// before; folds of column sums run one launch after the step; steps with room to choose (and with nobody waiting for them) go
// where the fewest bytes are, those without column sums also into the launch that finishes the last folds.  What the external
// computations make is in place when the whole program is run, so they tie nothing together here (stage by stage, every step
// keeps its launch).  What a launch that follows another one costs, 2.5 to 3.5 us, and what latency-bound steps (LayerNorm backward:
// 256 workgroups, 2.5 times its bytes) leave of the memory's rate is what this saves; where sharing a launch costs more than that
// (cost_of_sharing), the step goes to another one or the program stays step by step.  Measured (us, step by step with the folds in
// the last step's launch / merged), the kernels of a backward pass through a transformer block with its matrix products' results in
// place: 0.2 MB 19.4 / 12.2, 15 MB 25.6 / 20.1, 50 MB 28.0 / 21.9, 201 MB 47.4 / 39.7, 319 MB 64.1 / 55.0;
// 44 programs of one to three patterns with column sums beside gates, normalisations and transposes, 10 MB to 1.4 GB: 1.09 times, the worst level.
// Only where every step is a generated kernel of 256 threads (or a transpose of rows) and no two tensors share a part of the workspace.
void merge_steps(fs_program* prog) {
  const int ns = (int)prog->steps.size();
  if (!codegen_enabled() || ns < 2 || ns > 12) return;   // (twelve: what compiles in a few seconds)
  std::vector<Member> members(ns);
  typedef std::pair<int32_t, int64_t> Place;   // of a tensor between steps: an output of the graph or a part of the workspace
  auto place = [](const BufRef& r) { return Place(r.kind, r.kind == BUF_OUTPUT ? r.slot : r.offset); };
  std::map<Place, int> maker;
  std::set<Place> by_fold;
  std::map<int64_t, int64_t> scratch;   // the tensors in the workspace: where they begin and end
  std::vector<std::vector<size_t>> folds(ns);
  for (int s = 0; s < ns; ++s) {
    if (!member_of(*prog, s, &members[s])) return;
    const fs_program::Step& st = prog->steps[s];
    for (size_t k = 0; k < st.out.size(); ++k) {
      if (!maker.emplace(place(st.out[k]), s).second) return;
      if (st.out[k].kind == BUF_WORKSPACE) scratch[st.out[k].offset] = st.out[k].offset + st.plan->output_bytes[k];
    }
    const std::vector<Launch>& launches = st.plan->candidates[st.plan->chosen].launches;
    for (size_t l = 1; l < launches.size(); ++l) {
      if (launches[l].kernel != K_COLFOLD) return;
      folds[s].push_back(l);
      for (int a = 1; a < 3; ++a)
        if (launches[l].ptr[a].kind == BUF_OUTPUT) by_fold.insert(place(st.out[launches[l].ptr[a].slot]));
    }
  }
  int64_t end = 0;
  for (const auto& t : scratch) {   // memory that serves two tensors in turn ties their steps to their order
    if (t.first < end) return;
    end = t.second;
  }
  std::vector<int> at(ns, 0);              // a step's launch
  std::vector<char> tied(ns, 0);           // it reads from another step, or another one from it
  int last = 0;
  for (int s = 0; s < ns; ++s) {
    for (const BufRef& r : prog->steps[s].in) {
      if (r.kind == BUF_INPUT) continue;
      const auto made = maker.find(place(r));
      if (made == maker.end() || made->second >= s || by_fold.count(place(r))) return;
      at[s] = std::max(at[s], at[made->second] + 1);
      tied[s] = tied[made->second] = 1;
    }
    last = std::max(last, at[s] + (folds[s].empty() ? 0 : 1));
  }
  const int n = last + 1;
  if (n >= prog->info.n_kernels) return;
  std::vector<int64_t> bytes(n, 0);
  std::vector<int> free_steps;
  for (int s = 0; s < ns; ++s) {
    if (tied[s]) bytes[at[s]] += prog->steps[s].plan->bytes_min;
    else free_steps.push_back(s);
  }
  std::stable_sort(free_steps.begin(), free_steps.end(), [&](int a, int b) { return prog->steps[a].plan->bytes_min > prog->steps[b].plan->bytes_min; });
  for (int s : free_steps) {
    for (int l = 0; l <= last - (folds[s].empty() ? 0 : 1); ++l)
      if (bytes[l] < bytes[at[s]]) at[s] = l;
    bytes[at[s]] += prog->steps[s].plan->bytes_min;
  }
  std::vector<char> loops_in(n, 0);
  for (int s = 0; s < ns; ++s) loops_in[at[s]] |= members[s].loops;
  for (int l = 0; l < n; ++l)
    for (;;) {
      std::vector<int> here, lean;
      double ragged = 0;
      for (int s = 0; s < ns; ++s)
        if (at[s] == l) here.push_back(s);
      if (here.size() < 2) break;
      cost_of_sharing(members, here, &lean, &ragged);
      if (ragged > (double)(here.size() - 1) * device().launch_s) return;
      if (lean.empty()) break;
      const auto movable = std::find_if(lean.begin(), lean.end(), [&](int s) { return !tied[s]; });   // (no folds: it does not loop)
      int to = -1;
      for (int k = 0; k < n; ++k)
        if (!loops_in[k] && (to < 0 || bytes[k] < bytes[to])) to = k;
      if (movable == lean.end() || to < 0) return;
      bytes[l] -= prog->steps[*movable].plan->bytes_min;
      bytes[to] += prog->steps[*movable].plan->bytes_min;
      at[*movable] = to;
    }
  std::vector<fs_program::Merged> merged(n);
  std::vector<GenSource> sources;
  for (int l = 0; l < n; ++l) {
    fs_program::Merged& m = merged[l];
    std::vector<RowProgP> progs;
    std::vector<uint32_t> blocks;
    std::vector<Launch> fold_launches;
    uint64_t total = 0;
    // column sums first: their workgroups work the longest.  Where they are not all resident, one moves before others whose workgroups
    // have less than half its own's bytes (GELU backward [4096,3072] and LayerNorm backward [32768,768], in that order 50.2 us, in
    // the other 42.4, apart 44.7; where they are closer neither order is always the better: 19 and 76 MB 40.2 / 42.3, 38 and 151 MB
    // 37.0 / 36.1)
    double looping = 0;
    for (int s = 0; s < ns; ++s)
      if (at[s] == l) {
        m.steps.push_back(s);
        if (members[s].loops) looping += members[s].blocks;
      }
    const bool in_rounds = looping > device().n_cu * groups_per_cu(members, m.steps);
    m.steps.clear();
    auto per_group = [&](int s) { return members[s].cost->hbm_bytes / members[s].blocks; };
    for (int sums = 1; sums >= 0; --sums)
      for (int s = 0; s < ns; ++s) {
        if (at[s] != l || (members[s].prog.n_colsum > 0) != (sums == 1)) continue;
        size_t to = m.steps.size();
        while (sums == 1 && in_rounds && to > 0 && per_group(s) > 2.0 * per_group(m.steps[to - 1])) --to;
        m.steps.insert(m.steps.begin() + to, s);
      }
    for (int s : m.steps) {
      progs.push_back(members[s].prog);
      blocks.push_back(members[s].blocks);
      total += members[s].blocks;
      for (int slot : generated_ptr_slots(members[s].prog)) m.operands.push_back({s, members[s].ptr[slot]});
    }
    for (int s = 0; s < ns; ++s) {
      if (at[s] != l - 1) continue;
      for (size_t f : folds[s]) {
        const Launch& launch = prog->steps[s].plan->candidates[prog->steps[s].plan->chosen].launches[f];
        m.folds.push_back({s, f});
        fold_launches.push_back(launch);
        total += launch.shape.grid[0];
        for (int a = 0; a < 3; ++a) m.operands.push_back({s, launch.ptr[a]});
      }
    }
    if (total == 0 || total >= (1ull << 31) || m.operands.size() > kMergedMaxOperands) return;
    const std::string source = embedded_prelude() + generate_merged_kernel(progs, blocks, fold_launches, &m.entry);
    sources.push_back(gen_source(source, m.entry));
    m.shape = LaunchShape{};
    m.shape.grid[0] = (uint32_t)total;
    m.shape.block[0] = 256;
  }
  gen_compile_together(sources);
  for (int l = 0; l < n; ++l) {
    fs_program::Merged& m = merged[l];
    std::string log;
    if (gen_compile(sources[l].text, m.entry.c_str(), &m.kernel, &log) != 0 || gen_resources(m.kernel.get()).scratch_bytes > 0 || gen_preload(m.kernel.get()) != 0) return;
  }
  prog->merged = std::move(merged);
}

void fill_info(const Explorer& ex, fs_program* prog, int32_t beam_plans, double f_total_us, int64_t workspace_bytes) {
  fs_program_info& I = prog->info;
  I.n_ops = ex.n;
  I.beam_plans = beam_plans;
  I.workspace_bytes = workspace_bytes;
  I.bytes_min = graph_bytes_min(ex.g);
  I.f_total_us = f_total_us;
  std::set<int> counted_packs;
  for (const fs_program::Step& s : prog->steps) {
    const fs_plan_info& pi = s.plan->candidates[s.plan->chosen].info;
    if (s.ops.size() > 1) ++I.n_patterns; else ++I.n_single_ops;
    I.bytes_moved_model += pi.bytes_moved_model;
    if (s.pack >= 0) {
      if (counted_packs.insert(s.pack).second) {
        I.n_kernels += prog->packs[s.pack].pack->info.n_kernels;
        I.predicted_us += prog->packs[s.pack].pack->info.predicted_us;
        ++I.n_steps;
      }
    } else {
      I.n_kernels += pi.n_kernels;
      I.predicted_us += pi.predicted_us;
      ++I.n_steps;
    }
  }
  // joint folds: the steps they come from no longer issue a fold launch of their own; the estimate keeps the folds'
  // own times and drops the launches they no longer pay for
  int moved_from = 0;
  for (const fs_program::Step& s : prog->steps)
    if (s.pack < 0 && s.own_launches < s.plan->candidates[s.plan->chosen].launches.size()) ++moved_from;
  for (const std::vector<fs_program::JointFold>& j : prog->joint_folds) I.n_joint_folds += (int32_t)j.size();
  I.n_kernels += (int32_t)prog->joint_folds.size() - moved_from;
  I.predicted_us -= (double)(moved_from - (int)prog->joint_folds.size()) * device().launch_s * 1e6;
  if (prog->carrier.step >= 0) {
    I.n_kernels -= 1;
    I.predicted_us -= device().launch_s * 1e6;
  }
  I.n_packs = (int32_t)prog->packs.size();
  I.n_stages = 1;
  for (const fs_program::Step& s : prog->steps) I.n_stages = std::max(I.n_stages, s.stage + 1);
  for (int o = 0; o < ex.n; ++o) I.predicted_unfused_us += ex.t_single(o) * 1e6;
}

}  // namespace

extern "C" {

fs_status fs_explore_score(const fs_graph* g, const int32_t* ops, int32_t n, double* f_us, double* f_optimistic_us) try {
  clear_error();
  if (!g || !ops || !f_us) return fail(FS_ERR_INVALID_ARG, "fs_explore_score: null argument");
  if (!g->finalized) return fail(FS_ERR_INVALID_ARG, "fs_explore_score: graph is not finalized");
  if (n < 1) return fail(FS_ERR_INVALID_ARG, "fs_explore_score: empty pattern");
  OpSet p(ops, ops + n);
  std::sort(p.begin(), p.end());
  if (std::adjacent_find(p.begin(), p.end()) != p.end() || p.front() < 0 || p.back() >= (int)g->ops.size())
    return fail(FS_ERR_INVALID_ARG, "fs_explore_score: op indices must be distinct and inside the graph");
  Explorer ex(*g);
  const Scored& s = ex.score(p);
  if (f_optimistic_us) *f_optimistic_us = s.f_optimistic;
  if (!s.valid) {
    if (s.why == FS_ERR_CYCLE) return fail(FS_ERR_CYCLE, "fs_explore_score: fusing these ops creates a cyclic dependence");
    if (s.why == FS_ERR_DTYPE)
      return fail(FS_ERR_DTYPE, "fs_explore_score: a tensor stored in another dtype than it was computed in crosses the pattern boundary");
    return fail(FS_ERR_UNSUPPORTED_PATTERN, "fs_explore_score: no stitched kernel can run these ops as one pattern");
  }
  *f_us = s.f;
  return FS_OK;
} catch (...) {
  return fs::fail_caught("fs_explore_score");
}

fs_status fs_explore(const fs_graph* g, const fs_explore_opts* opts, fs_program** out) try {
  clear_error();
  if (!g || !out) return fail(FS_ERR_INVALID_ARG, "fs_explore: null argument");
  if (!g->finalized) return fail(FS_ERR_INVALID_ARG, "fs_explore: graph is not finalized");
  Explorer ex(*g);
  bool pack_tiny = true, remote_fusion = true, joint_folds = true;
  if (opts) {
    if (opts->top_k < 0 || opts->beam_width < 0 || opts->top_k > 16 || opts->beam_width > 16)
      return fail(FS_ERR_INVALID_ARG, "fs_explore: top_k and beam_width must be 0 (default 3) or 1..16");
    if (opts->top_k > 0) ex.top_k = opts->top_k;
    if (opts->beam_width > 0) ex.beam_width = opts->beam_width;
    pack_tiny = opts->no_packing == 0;
    remote_fusion = opts->no_remote_fusion == 0;
    joint_folds = opts->no_joint_folds == 0;
  }
  ex.explore_patterns();
  const std::vector<Explorer::PlanSet> plans = ex.beam();

  // Final choice among the beam's plans by the full latency evaluator (Section 5.3): every pattern, and every op
  // left alone, is planned for real and the predicted times are added up.
  std::vector<BuiltPlan> built(plans.size());
  fs_status first_error = FS_OK;
  std::string first_text;
  for (size_t k = 0; k < plans.size(); ++k) {
    std::string text;
    const fs_status st = build_steps(&ex, plans[k], remote_fusion, &built[k], &text);
    if (st != FS_OK && first_error == FS_OK) { first_error = st; first_text = text; }
  }
  int best = -1;
  for (size_t k = 0; k < built.size(); ++k)
    if (built[k].ok && (best < 0 || built[k].predicted < built[best].predicted)) best = (int)k;
  for (size_t k = 0; k < built.size(); ++k)
    if ((int)k != best) built[k].destroy();
  if (best < 0) return fail(first_error != FS_OK ? first_error : FS_ERR_UNSUPPORTED_PATTERN, "fs_explore: %s", first_text.c_str());

  std::vector<GenSource> sources;
  for (const fs_program::Step& s : built[best].steps) compiled_ahead(*s.plan, &sources);
  gen_compile_together(sources);
  for (fs_program::Step& s : built[best].steps) {
    fs_status st = complete_plan(s.plan);
    if (st == FS_ERR_UNSUPPORTED_PATTERN) {
      // the pattern's only stitched form was a generated kernel that did not compile: it runs per op instead
      SubGraph sub;
      fs_plan* per_op = nullptr;
      st = ex.extract(s.ops, &sub);
      if (st == FS_OK) st = create_plan(sub.g, FS_SCHEME_UNFUSED, nullptr, true, &per_op);
      if (st == FS_OK) {
        fs_plan_destroy(s.plan);
        s.plan = per_op;
      }
    }
    if (st != FS_OK) {
      built[best].destroy();
      return st;
    }
  }
  fs_program* prog = new (std::nothrow) fs_program();
  if (!prog) { built[best].destroy(); return fail(FS_ERR_INVALID_ARG, "fs_explore: out of host memory"); }
  if (!order_steps(*g, &built[best].steps)) {   // cannot happen for convex patterns
    delete prog;
    built[best].destroy();
    return fail(FS_ERR_CYCLE, "fs_explore: the chosen patterns depend on each other cyclically");
  }
  prog->steps = std::move(built[best].steps);
  built[best].steps.clear();
  std::vector<int> pos(prog->steps.size());   // where in the order a step's kernel is issued (packed members: at the first member)
  for (size_t s = 0; s < pos.size(); ++s) pos[s] = (int)s;
  if (pack_tiny) decide_packs(*g, prog, &pos);
  for (fs_program::Step& s : prog->steps) s.own_launches = s.plan->candidates[s.plan->chosen].launches.size();
  if (joint_folds) {
    join_folds(*g, prog);
    carry_folds(prog);
  }
  const int64_t workspace = place_buffers(*g, prog, pos);
  fill_info(ex, prog, (int32_t)plans.size(), built[best].f, workspace);
  prog->n_inputs = (int32_t)g->inputs.size();
  prog->n_outputs = (int32_t)g->outputs.size();
  for (int t : g->inputs) prog->input_bytes.push_back(g->tensors[t].numel() * dtype_bytes(g->tensors[t].dtype));
  for (int t : g->outputs) prog->output_bytes.push_back(g->tensors[t].numel() * dtype_bytes(g->tensors[t].store_as));
  if (joint_folds && pack_tiny) merge_steps(prog);
  *out = prog;
  return FS_OK;
} catch (...) {
  return fs::fail_caught("fs_explore");
}

}  // extern "C"
