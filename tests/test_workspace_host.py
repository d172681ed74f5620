"""The workspace that the observables keep between calls, on the host with counted
allocations: growing requests free the blocks they outgrow instead of adding up, a
repeated run allocates nothing, at most the stated amount stays after a run, a run
that fails leaves nothing, and live blocks never overlap (random scopes)."""
from tests.host_util import run_host

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include <map>
#include <random>
#include "runtime.hpp"
static std::map<char*, size_t> live;
static size_t held = 0, peak = 0, n_malloc = 0, limit = (size_t)1 << 60;
static char* next_p = (char*)((size_t)1 << 40);
extern "C" hipError_t hipMalloc(void** p, size_t n) {
  if (held + n > limit) return hipErrorOutOfMemory;
  *p = next_p;
  live[next_p] = n;
  next_p += n + 4096;
  held += n;
  n_malloc++;
  if (held > peak) peak = held;
  return hipSuccess;
}
extern "C" hipError_t hipFree(void* p) {
  auto it = live.find((char*)p);
  if (it == live.end()) { std::printf("bad free\n"); std::exit(0); }
  held -= it->second;
  live.erase(it);
  return hipSuccess;
}
#define CHECK(c) do { if (!(c)) { std::printf("line %d: %s (held %zu peak %zu)\n", __LINE__, #c, held, peak); return 0; } } while (0)
struct Scope {
  rt::Workspace& w;
  rt::Workspace::Mark m;
  explicit Scope(rt::Workspace& ws) : w(ws), m(ws.mark()) {}
  ~Scope() { w.reset(m); }
};
int main() {
  const size_t MB = (size_t)1 << 20;
  {   // scopes of growing size beside a live one
    rt::Workspace w;
    Scope outer(w);
    w.get(3 * MB);
    size_t big = 0;
    for (size_t n = MB; n < 4096 * MB; n += n / 2) {
      Scope s(w);
      w.get(n);
      big = n;
    }
    CHECK(peak <= big + 8 * MB);
    w.trim(0);
    CHECK(held == 0);
  }
  {   // a repeated run allocates nothing; what stays is bounded
    rt::Workspace a, b;
    for (int rep = 0; rep < 3; rep++) {
      const size_t before = n_malloc;
      rt::WorkspaceRun run(a, b);
      Scope keep(a);
      for (int k = 0; k < 20; k++) {
        a.get(k * MB / 8);
        Scope s(b);
        b.get((size_t)(1 + 7 * k % 13) * MB);
        b.get(MB / 2);
      }
      run.ok = true;
      CHECK(rep == 0 || n_malloc == before);
    }
    {
      rt::WorkspaceRun run(a, b);
      Scope keep(a), tmp(b);
      for (int k = 0; k < 9; k++) { a.get(200 * MB); b.get(100 * MB); }
      run.ok = true;
    }
    CHECK(a.held() <= rt::Workspace::kKeep && b.held() <= rt::Workspace::kKeep);
    CHECK(held == a.held() + b.held());
    // a run that fails gives everything back, and the next one works
    limit = 1500 * MB;
    bool threw = false;
    try {
      rt::WorkspaceRun run(a, b);
      Scope keep(a);
      for (int k = 0; k < 40; k++) {
        Scope s(b);
        a.get(100 * MB);
        b.get(300 * MB);
      }
      run.ok = true;
    } catch (const rt::HipFail&) { threw = true; }
    CHECK(threw && held == 0 && a.blocks.empty() && b.blocks.empty());
    limit = (size_t)1 << 60;
    {
      rt::WorkspaceRun run(a, b);
      Scope s(b);
      CHECK(b.get(MB) != nullptr);
    }
  }
  // random nested scopes: no two live ranges overlap, every range inside a live block
  std::mt19937 g(1);
  rt::Workspace w;
  std::vector<std::pair<char*, size_t>> rs;
  struct Frame { rt::Workspace::Mark m; size_t n; };
  std::vector<Frame> st;
  for (int step = 0; step < 20000; step++) {
    const int op = g() % 10;
    if (op < 2) st.push_back({w.mark(), rs.size()});
    else if (op < 4 && !st.empty()) { w.reset(st.back().m); rs.resize(st.back().n); st.pop_back(); }
    else if (rs.size() < 60) {
      const size_t n = (size_t)(g() % 1000 + 1) << (g() % 18);
      limit = g() % 8 ? (size_t)1 << 60 : held;   // some requests for new memory fail
      char* p;
      try { p = (char*)w.get(n); } catch (const rt::HipFail&) { continue; }
      for (auto& r : rs) CHECK(p + n <= r.first || r.first + r.second <= p);
      auto it = live.upper_bound(p);
      CHECK(it != live.begin() && (--it, p + n <= it->first + it->second));
      for (auto& r : rs) { auto q = live.upper_bound(r.first); CHECK(q != live.begin() && (--q, r.first + r.second <= q->first + q->second)); }
      rs.push_back({p, n});
    }
  }
  std::printf("ok\n");
}
"""


def test_workspace_blocks(tmp_path):
    out = run_host(PROGRAM, tmp_path)
    assert out == "ok\n", out
