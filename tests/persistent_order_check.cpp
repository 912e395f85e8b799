// The order in which the one-launch step of few rows uses the memory that its blocks hand on (persist_hand()): a model of its wavefronts,
// each a list of what it asks for, marks and stores between the barriers of its workgroup.  Whoever asks for a place finds what
// was stored there in that block or the mark ahead of it, never what an earlier block left and never what a later one put over it,
// and no wavefront is kept waiting for good, however long any one of them is held up anywhere.
// Compiled and run by test_few_rows.py; exits non-zero at the first order that does not hold.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

#include "persistent_cut.h"

using namespace mtmc::bf16;

enum Kind { X, SS0, XO, SS1, QKV, O, ACT, PART, kKinds };
enum Do { ASK, MARK, STORE, BARRIER };
struct Op {
  Do what;
  Kind kind;
  int block, first, last;  // places first .. last - 1 of what block `block` hands on (X, SS0: of what goes into it)
};
constexpr int kBlocks = 8, kGrid = 10, kCompute = 4, kControl = 2, kWaves = kCompute + kControl, kPlaces = 64;
struct Wave {
  std::vector<Op> ops;
  size_t at = 0;
};

// Which workgroup has what: row tiles of the residual for the first nt_d, the rest drawn.
struct Cut {
  int nt_d, qkv[kGrid], unit[kGrid], acts[kGrid], parts[kGrid], heads;
  bool empty[kGrid];  // the unit's chunk holds no part of the context
  int n_qkv = 0, n_units = 0, n_acts = 0, n_parts = 0, first_qkv[kGrid], first_act[kGrid], first_part[kGrid];
  explicit Cut(std::mt19937& rng) {
    auto upto = [&](int n) { return (int)(rng() % (n + 1)); };
    nt_d = 1 + upto(3);
    heads = 1 + upto(7);
    for (int g = 0; g < kGrid; ++g) {
      qkv[g] = upto(2);
      first_qkv[g] = n_qkv;
      n_qkv += qkv[g];
      unit[g] = g % 3 == 2 || upto(1) ? n_units++ : -1;
      empty[g] = upto(2) == 0;
      acts[g] = g < 3 ? 1 + upto(2) : g < 6 ? upto(2) : 0;  // some have none, and nothing of the down projection
      first_act[g] = n_acts;
      n_acts += acts[g];
      parts[g] = g < 2 ? 1 + upto(1) : g < 5 ? upto(2) : 0;
      first_part[g] = n_parts;
      n_parts += parts[g];
    }
    empty[2] = true;
  }
};

// What is stored by wavefront w of a unit: half of the place pair if its threads store at all (16 threads per head, 64 a wavefront).
static bool stores(int w, int heads) { return w * 64 < heads * 16; }

static void write_program(const Cut& c, int g, int w, bool all_ask, std::vector<Op>& p) {
  const bool control = w >= kCompute, lead = w == kCompute, tile = g < c.nt_d;
  const int k = w - kCompute;
  auto ask = [&](Kind kind, int l, int first, int last) { if (first < last) p.push_back({ASK, kind, l, first, last}); };
  auto put = [&](Do what, Kind kind, int l, int at) { p.push_back({what, kind, l, at, at + 1}); };
  auto barrier = [&] { p.push_back({BARRIER, X, 0, 0, 0}); };
  for (int l = 0; l < kBlocks; ++l) {
    const bool more = l + 1 < kBlocks;
    // QKV projection
    if (control) {
      for (int u = k; more && u < c.qkv[g]; u += kControl) put(MARK, QKV, l + 1, c.first_qkv[g] + u);
      if (lead && l && c.qkv[g]) ask(SS1, l - 1, 0, c.nt_d), ask(SS0, l, 0, c.nt_d);
    }
    for (int u = 0; u < c.qkv[g]; ++u) {
      if (!control && l) ask(X, l, 0, c.nt_d);
      barrier();
      if (control && u % kControl == k) put(STORE, QKV, l, c.first_qkv[g] + u);
    }
    barrier();
    // attention; the places of a unit: one for each of two wavefronts that may store
    const int u = c.unit[g];
    if (control) {
      if (u >= 0 && !c.empty[g]) barrier(), barrier();
    } else if (u >= 0) {
      const bool mine = stores(w, c.heads);
      if (more && mine) put(MARK, O, l + 1, 2 * u + w);
      if (!c.empty[g]) ask(QKV, l, 0, c.n_qkv), barrier(), barrier();
      else if (all_ask || persist_empty_unit_asks(w, c.heads)) ask(QKV, l, 0, c.n_qkv);
      if (mine) put(STORE, O, l, 2 * u + w);
    }
    barrier();
    // O projection
    if (tile) {
      if (control) {
        if (lead && more) put(MARK, XO, l + 1, g), put(MARK, SS1, l + 1, g);
        if (lead && l) ask(SS0, l, 0, c.nt_d);
        barrier();
        if (lead) put(STORE, XO, l, g), put(STORE, SS1, l, g);
      } else {
        for (int v = 0; v < c.n_units; ++v) ask(O, l, 2 * v, 2 * v + (c.heads > 4 ? 2 : 1));
        barrier();
      }
    }
    barrier();
    // gate / up projection
    if (c.acts[g]) {
      if (control) {
        for (int a = k; more && a < c.acts[g]; a += kControl) put(MARK, ACT, l + 1, c.first_act[g] + a);
        if (lead) {
          if (l) ask(SS0, l, 0, c.nt_d);
          ask(SS1, l, 0, c.nt_d);
        }
        barrier();
        for (int a = k; a < c.acts[g]; a += kControl) put(STORE, ACT, l, c.first_act[g] + a);
      } else {
        ask(XO, l, 0, c.nt_d);
        barrier();
      }
    }
    barrier();
    // down projection
    if (control) {
      if (more && k < c.parts[g]) put(MARK, PART, l + 1, c.first_part[g] + k);
      if (lead && tile) ask(SS1, l, 0, c.nt_d);
      barrier();
      if (k < c.parts[g]) put(STORE, PART, l, c.first_part[g] + k);
    } else {
      if (c.parts[g]) ask(ACT, l, 0, c.n_acts);
      barrier();
    }
    barrier();
    // sum of the splits
    if (lead && tile) {
      if (l + 2 < kBlocks) put(MARK, X, l + 2, g), put(MARK, SS0, l + 2, g);
      int stored = 0;  // parts without a control wavefront are not stored
      for (int h = 0; h < kGrid; ++h, stored = 0)
        while (stored < std::min(c.parts[h], kControl)) ask(PART, l, c.first_part[h] + stored, c.first_part[h] + stored + 1), ++stored;
      if (more) put(STORE, X, l + 1, g), put(STORE, SS0, l + 1, g);
    }
  }
}

// What a place holds: 2 block + 1 what the block stored, 2 block its mark; -1 anything.
struct Run {
  std::vector<Wave> waves;
  int place[kKinds][kPlaces][kPersistPieces];
  bool late;  // marks come when they are waited for, ahead of the wavefront's next store; else at once
  std::vector<std::vector<Op>> due;
  int arrived[kGrid] = {};
  const char* fault = nullptr;
  Run(const Cut& c, bool late_, bool all_ask) : waves(kGrid * kWaves), late(late_), due(kGrid * kWaves) {
    for (auto& kind : place)
      for (auto& at : kind)
        for (int s = 0; s < kPersistPieces; ++s) at[s] = s < 2 ? 2 * s : -1;
    for (int i = 0; i < kGrid * kWaves; ++i) write_program(c, i / kWaves, i % kWaves, all_ask, waves[i].ops);
  }
  // -1: it waits, 0: it is done, 1: a step further
  int step(int i) {
    Wave& w = waves[i];
    if (w.at == w.ops.size()) return 0;
    const Op& op = w.ops[w.at];
    if (op.what == BARRIER) {
      const int g = i / kWaves;
      int here = 0;
      for (int v = 0; v < kWaves; ++v) {
        const Wave& o = waves[g * kWaves + v];
        here += o.at < o.ops.size() && o.ops[o.at].what == BARRIER;
      }
      if (here < kWaves) return -1;
      for (int v = 0; v < kWaves; ++v) ++waves[g * kWaves + v].at;
      return 1;
    }
    if (op.what == ASK) {
      for (int p = op.first; p < op.last; ++p) {
        const int v = place[op.kind][p][op.block % kPersistPieces];
        if (v != 2 * op.block && v != 2 * op.block + 1) {
          fault = v < 2 * op.block ? "an earlier block's data where there should be a mark" : "gone before it was read";
          return -1;
        }
        if (v == 2 * op.block) return -1;
      }
    } else if (op.what == MARK && late) {
      due[i].push_back(op);
    } else {
      if (op.what == STORE) {
        for (const Op& m : due[i]) place[m.kind][m.first][m.block % kPersistPieces] = 2 * m.block;
        due[i].clear();
      }
      place[op.kind][op.first][op.block % kPersistPieces] = 2 * op.block + (op.what == STORE);
    }
    ++w.at;
    return 1;
  }
  // everybody but `held` as far as they come
  void all(int held) {
    for (bool on = true; on && !fault;) {
      on = false;
      for (int i = 0; i < kGrid * kWaves; ++i)
        while (i != held && !fault && step(i) == 1) on = true;
    }
  }
  bool done() const {
    return std::all_of(waves.begin(), waves.end(), [](const Wave& w) { return w.at == w.ops.size(); });
  }
};

// Each wavefront in turn is held up ahead of each of its operations (all others go on as far as they can), then let go.
static const char* first_fault(const Cut& c, bool late, bool all_ask) {
  for (int held = 0; held < kGrid * kWaves; ++held) {
    Run r(c, late, all_ask);
    while (!r.done()) {
      r.all(held);
      if (r.fault) return r.fault;
      const int s = r.step(held);
      if (r.fault) return r.fault;
      if (s == 1) continue;
      r.all(-1);
      if (r.fault) return r.fault;
      if (!r.done()) return "wavefronts that wait for good";
    }
  }
  return nullptr;
}

int main() {
  std::mt19937 rng(7);
  bool seen = false;
  for (int n = 0; n < 12; ++n) {
    const Cut c(rng);
    for (bool late : {false, true}) {
      const char* fault = first_fault(c, late, false);
      if (fault) {
        std::printf("cut %d, marks %s: %s\n", n, late ? "late" : "at once", fault);
        return 1;
      }
      seen |= first_fault(c, late, true) != nullptr;
    }
  }
  // the model tells: with a wavefront that asks and has no store behind it (all eight of a unit with nothing to attend to) it fails
  if (!seen) {
    std::printf("a reader without a store behind it goes unnoticed\n");
    return 1;
  }
  std::printf("ok\n");
  return 0;
}
