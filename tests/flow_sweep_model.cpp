// Host model of the push-relabel sweeps: the node step of the GPU kernel (flow_sweep.h) run by one
// coroutine per node, interleaved at every memory operation, with atomics that return nothing applied
// late and in any order across addresses (in order per address, and before the node's own loads of it).
// The rounds around the sweeps are those of max_flow: exact relabels, an exact relabel when a node is
// stuck at 2N, and another pass from saturated sources while the sources reach a sink (not with "plain").
// Usage: flow_sweep_model FIRST_SEED COUNT RELABEL_EVERY [plain]; prints one line of counts.
#include <limits.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include <ucontext.h>

#include <algorithm>
#include <deque>
#include <queue>
#include <random>
#include <vector>

struct Pending {
  int64_t *p, d;
};
struct Thread {
  ucontext_t ctx;
  std::vector<char> stack;
  std::deque<Pending> pend;
  bool done = true;
  int ex_loads = 0;
  int64_t last_ex = 0;
};
static std::vector<Thread> threads;
static ucontext_t scheduler;
static int running;
static std::mt19937 rng;

static void step() { swapcontext(&threads[running].ctx, &scheduler); }
static void settle(Thread &t, const void *p) {
  for (size_t i = 0; i < t.pend.size();) {
    if (t.pend[i].p == p) {
      *t.pend[i].p += t.pend[i].d;
      t.pend.erase(t.pend.begin() + i);
    } else {
      ++i;
    }
  }
}
static void settle_one(Thread &t) {  // any pending operation that is the first on its address
  if (t.pend.empty()) return;
  int64_t *p = t.pend[rng() % t.pend.size()].p;
  size_t j = 0;
  while (t.pend[j].p != p) ++j;
  *p += t.pend[j].d;
  t.pend.erase(t.pend.begin() + j);
}

static std::vector<int64_t> res, ex;
template <typename T>
static T model_load(const T *p) {
  step();
  Thread &t = threads[running];
  settle(t, p);
  if ((const void *)p == (const void *)&ex[running]) {
    ++t.ex_loads;
    t.last_ex = (int64_t)*p;
  }
  return *p;
}
template <typename T>
static void model_store(T *p, T v) {
  step();
  *p = v;
}
static void atomicAdd(unsigned long long *p, unsigned long long d) {
  step();
  threads[running].pend.push_back({(int64_t *)p, (int64_t)d});
}

#define __device__
#define __forceinline__ inline
#define __HIP_MEMORY_SCOPE_AGENT 0
#define __hip_atomic_load(p, order, scope) model_load(p)
#define __hip_atomic_store(p, v, order, scope) model_store(p, v)
#include "../paper_2504_12013_amd/csrc/flow_sweep.h"

// a Lawler network in the layout of the kernels
static int64_t N, A;
static int32_t nv;
static std::vector<int32_t> head, tail_, h, rends;
static std::vector<int64_t> voffn, vadj, rbase, cap;
static std::vector<uint8_t> term;
static std::vector<std::vector<int64_t>> arcs;  // out-arcs per node, for the searches

static void build(int seed) {
  rng.seed(seed);
  const int vertices = 3 + rng() % 10, nets = 4 + rng() % 14;
  nv = 2 + vertices;
  N = nv + 2 * nets;
  std::vector<std::vector<int32_t>> pins(nets);
  std::vector<int64_t> w(nets);
  for (int e = 0; e < nets; ++e) {
    w[e] = 1 + rng() % 2;
    for (int i = 2 + rng() % 3; i > 0; --i) {
      const int32_t x = rng() % nv;
      if (std::find(pins[e].begin(), pins[e].end(), x) == pins[e].end()) pins[e].push_back(x);
    }
  }
  rbase.clear();
  rends.clear();
  A = 0;
  std::vector<std::vector<int64_t>> at(nv);
  for (int e = 0; e < nets; ++e) {
    rbase.push_back(A);
    rends.push_back((int32_t)pins[e].size());
    for (size_t j = 0; j < pins[e].size(); ++j) at[pins[e][j]].push_back(A + 2 + 4 * (int64_t)j);
    A += 2 + 4 * (int64_t)pins[e].size();
  }
  head.assign(A, 0);
  tail_.assign(A, 0);
  res.assign(A, 0);
  auto arc = [&](int64_t a, int32_t u, int32_t v, int64_t c) {
    tail_[a] = u;
    head[a] = v;
    res[a] = c;
  };
  for (int e = 0; e < nets; ++e) {
    const int32_t in = nv + 2 * e, out = in + 1;
    arc(rbase[e], in, out, w[e]);
    arc(rbase[e] + 1, out, in, 0);
    for (size_t j = 0; j < pins[e].size(); ++j) {
      const int64_t a = rbase[e] + 2 + 4 * (int64_t)j;
      const int32_t x = pins[e][j];
      arc(a, x, in, 1000);
      arc(a + 1, in, x, 0);
      arc(a + 2, out, x, 1000);
      arc(a + 3, x, out, 0);
    }
  }
  voffn.assign(nv + 1, 0);
  vadj.clear();
  for (int x = 0; x < nv; ++x) {
    vadj.insert(vadj.end(), at[x].begin(), at[x].end());
    voffn[x + 1] = (int64_t)vadj.size();
  }
  arcs.assign(N, {});
  for (int64_t a = 0; a < A; ++a) arcs[tail_[a]].push_back(a);
  for (int64_t u = 0; u < N; ++u) {  // the kernels' arc index names the same arcs
    const jet::OutArcs o = jet::out_arcs(u, nv, voffn.data(), rbase.data(), rends.data());
    std::vector<int64_t> mine;
    for (int32_t i = 0; i < o.count; ++i) mine.push_back(jet::out_arc(o, vadj.data(), i));
    std::sort(mine.begin(), mine.end());
    if (mine != arcs[u]) abort();
  }
  cap = res;
  term.assign(N, 0);
  term[0] = 1;
  term[1] = 2;
  h.assign(N, 0);
  ex.assign(N, 0);
}

// nodes that the terminals of `side` reach (back: that reach them) over residual arcs r
static std::vector<uint8_t> reached(const std::vector<int64_t> &r, int side, bool back) {
  std::vector<uint8_t> f(N, 0);
  std::queue<int32_t> q;
  for (int64_t u = 0; u < N; ++u)
    if (term[u] == side) f[u] = 1, q.push((int32_t)u);
  while (!q.empty()) {
    const int32_t u = q.front();
    q.pop();
    for (int64_t a : arcs[u])
      if ((back ? r[a ^ 1] : r[a]) > 0 && !f[head[a]]) f[head[a]] = 1, q.push(head[a]);
  }
  return f;
}

static int64_t augment(std::vector<int64_t> &r) {  // shortest augmenting paths
  for (int64_t F = 0;;) {
    std::vector<int64_t> by(N, -2);
    std::queue<int32_t> q;
    by[0] = -1;
    q.push(0);
    while (!q.empty() && by[1] == -2) {
      const int32_t u = q.front();
      q.pop();
      for (int64_t a : arcs[u])
        if (r[a] > 0 && by[head[a]] == -2) by[head[a]] = a, q.push(head[a]);
    }
    if (by[1] == -2) return F;
    int64_t d = INT64_MAX;
    for (int32_t v = 1; v != 0; v = tail_[by[v]]) d = std::min(d, r[by[v]]);
    for (int32_t v = 1; v != 0; v = tail_[by[v]]) r[by[v]] -= d, r[by[v] ^ 1] += d;
    F += d;
  }
}

static void relabel() {
  for (int64_t u = 0; u < N; ++u) h[u] = term[u] == 2 ? 0 : term[u] == 1 ? (int32_t)N : -1;
  for (int side = 2; side >= 1; --side) {
    std::queue<int32_t> q;
    for (int64_t u = 0; u < N; ++u)
      if (term[u] == side) q.push((int32_t)u);
    while (!q.empty()) {
      const int32_t v = q.front();
      q.pop();
      for (int64_t a : arcs[v])
        if (res[a ^ 1] > 0 && term[head[a]] == 0 && h[head[a]] == -1) h[head[a]] = h[v] + 1, q.push(head[a]);
    }
  }
  for (int64_t u = 0; u < N; ++u)
    if (h[u] == -1) h[u] = (int32_t)(2 * N);
}

static int64_t waited;  // turns that ended with excess and no residual arc in sight
static void turn(int u) {
  jet::sweep_node(u, N, nv, term.data(), h.data(), ex.data(), res.data(), head.data(), voffn.data(), vadj.data(),
                  rbase.data(), rends.data());
  const Thread &t = threads[u];
  if (term[u] == 0 && t.last_ex > 0 && h[u] < 2 * N && t.ex_loads <= jet::kPushCycles) ++waited;
  threads[u].done = true;
  swapcontext(&threads[u].ctx, &scheduler);
}
static void sweep() {
  std::vector<int> live;
  for (int u = 0; u < (int)N; ++u) {
    Thread &t = threads[u];
    t.done = false;
    t.ex_loads = 0;
    t.last_ex = 0;
    if (t.stack.empty()) t.stack.resize(1 << 16);
    getcontext(&t.ctx);
    t.ctx.uc_stack.ss_sp = t.stack.data();
    t.ctx.uc_stack.ss_size = t.stack.size();
    t.ctx.uc_link = &scheduler;
    makecontext(&t.ctx, (void (*)())turn, 1, u);
    live.push_back(u);
  }
  while (!live.empty()) {
    const size_t k = rng() % live.size();
    running = live[k];
    for (int n = 1 + rng() % 12; n > 0 && !threads[running].done; --n) swapcontext(&scheduler, &threads[running].ctx);
    for (int n = rng() % 3; n > 0; --n) settle_one(threads[rng() % N]);
    if (threads[running].done) live[k] = live.back(), live.pop_back();
  }
  for (int u = 0; u < (int)N; ++u)
    while (!threads[u].pend.empty()) settle_one(threads[u]);
}

static void count(int64_t *active, int64_t *stuck) {
  *active = *stuck = 0;
  for (int64_t u = 0; u < N; ++u)
    if (term[u] == 0 && ex[u] > 0) ++(h[u] < 2 * N ? *active : *stuck);
}

int main(int argc, char **argv) {
  const int first = atoi(argv[1]), trials = atoi(argv[2]), every = atoi(argv[3]);
  const bool plain = argc > 4 && strcmp(argv[4], "plain") == 0;
  threads.resize(64);
  int64_t refused = 0, unfinished = 0, wrong = 0, again = 0;
  for (int t = 0; t < trials; ++t) {
    build(first + t);
    bool open = true, failed = false;
    for (int round = 0; open && !failed; ++round) {
      again += round > 0;
      for (int64_t a = 0; a < A; ++a) {  // saturate the sources' arcs
        const int64_t d = res[a];
        if (term[tail_[a]] != 1 || term[head[a]] == 1 || d <= 0) continue;
        res[a] -= d, res[a ^ 1] += d, ex[tail_[a]] -= d, ex[head[a]] += d;
      }
      relabel();
      int64_t active = 1;
      for (int check = 0; active > 0 && !failed; ++check) {
        if (check == 4000) ++unfinished, failed = true;
        if (check % every == every - 1) relabel();
        sweep();
        int64_t stuck;
        count(&active, &stuck);
        if (stuck == 0) continue;
        relabel();
        count(&active, &stuck);
        if (stuck > 0) ++refused, failed = true;
      }
      open = !plain && !failed && reached(res, 1, false)[1];
    }
    if (failed) continue;
    std::vector<int64_t> r = cap;
    const int64_t F = augment(r);
    wrong += ex[1] != F || reached(r, 1, false) != reached(res, 1, false) ||
             reached(r, 2, true) != reached(res, 2, true);
  }
  printf("refused %lld unfinished %lld wrong %lld again %lld waited %lld\n", (long long)refused, (long long)unfinished,
         (long long)wrong, (long long)again, (long long)waited);
  return 0;
}
