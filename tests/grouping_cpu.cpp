// The one-wave grouping's own text (group_few.inc, taken out of the kernel source
// by the test) run on the CPU: 64 threads as the wave's lanes, in any order
// between the points where the wave waits for all its lanes, on arrays that
// check every index and start with leftovers; the groups against union-find.
#include <algorithm>
#include <atomic>
#include <barrier>
#include <climits>
#include <cstdio>
#include <cstdlib>
#include <map>
#include <numeric>
#include <random>
#include <set>
#include <thread>
#include <vector>
using std::max;
using std::min;
struct int2 {
  int x, y;
};
static int2 make_int2(int x, int y) { return {x, y}; }
struct Cell {
  std::atomic<int> v{0};
  operator int() const { return v; }
  int operator=(int i) { return v = i; }
  int operator=(const Cell& o) { return v = o.v.load(); }
};
static void bad(const char* what, int i, int n) {
  printf("%s: index %d of %d\n", what, i, n);
  fflush(stdout);
  _Exit(2);
}
struct Arr {
  std::vector<Cell> d;
  explicit Arr(int n) : d(n) {}
  Cell& operator[](int i) {
    if (i < 0 || i >= (int)d.size()) bad("array", i, (int)d.size());
    return d[i];
  }
};
struct Ptr {  // a pointer to such an array, or null
  Arr* a;
  explicit operator bool() const { return a; }
  Cell& operator[](int i) const { return (*a)[i]; }
};
struct Pairs {
  const int2* p;
  int n;
  const int2& operator[](int i) const {
    if (i < 0 || i >= n) bad("pair list", i, n);
    return p[i];
  }
};
struct Stat {
  unsigned ctl;
  int maxg, ngroups, ncand;
  unsigned long long enc_total;
};
struct EncArgs {
  Pairs encij;
  Ptr goff, gmem;
  Stat* st;
};
template <int N>
struct Lds {
  static constexpr int kN = N;
  Arr link{N}, first{N}, gid{N}, gsz{N / 2 + 1}, gof{N / 2 + 1}, roots{N / 2}, shw{4};
  Cell nroot;
};
static thread_local struct {
  int x;
} threadIdx;
static thread_local std::minstd_rand rng;
static std::barrier<> wave_bar(64);
static long long slot[64];
static void jitter() {
  if (rng() % 8 == 0) std::this_thread::yield();
}
static void wsync() {
  jitter();
  wave_bar.arrive_and_wait();
}
static void __syncthreads() { wave_bar.arrive_and_wait(); }
template <class F>
static auto all_lanes(long long v, F f) {
  slot[threadIdx.x] = v;
  wave_bar.arrive_and_wait();
  const auto r = f();
  wave_bar.arrive_and_wait();
  return r;
}
static unsigned long long __ballot(bool b) {
  return all_lanes(b, [] {
    unsigned long long m = 0;
    for (int i = 0; i < 64; ++i) m |= (unsigned long long)(slot[i] != 0) << i;
    return m;
  });
}
static int wave_incl_scan(int v) {
  return all_lanes(v, [] { return (int)std::accumulate(slot, slot + threadIdx.x + 1, 0ll); });
}
static int wave_max_i(int v) {
  return all_lanes(v, [] { return (int)*std::max_element(slot, slot + 64); });
}
static int read_lane(int v, int l) {
  return all_lanes(v, [l] { return (int)slot[l]; });
}
#define __device__
#define __forceinline__ inline
#define __builtin_amdgcn_readlane read_lane
#define __builtin_amdgcn_readfirstlane(x) ((int)(x))
static int __popc(unsigned v) { return __builtin_popcount(v); }
static int __ffs(int v) { return __builtin_ffs(v); }
static int atomicMin(Cell* p, int v) {
  jitter();
  int o = p->v.load();
  while (o > v && !p->v.compare_exchange_weak(o, v)) {
  }
  return o;
}
static int atomicAdd(Cell* p, int v) { return jitter(), p->v.fetch_add(v); }
static int atomicOr(Cell* p, int v) { return jitter(), p->v.fetch_or(v); }
static int clear_rows(const EncArgs&, int, int) { return 0; }

#include "group_few.inc"

template <int N>
static int run(std::mt19937& R, int trials) {
  Lds<N> L;
  Arr gm(N), goff(N + 1), gmem(N);
  for (int t = 0; t < trials; ++t) {
    // random pairs, a chain, stars, disjoint pairs, neighbours; sometimes all 256
    const int n = 2 + R() % (N - 1), kind = R() % 5;
    const int want = (int)min<long long>((long long)n * (n - 1) / 2, t % 5 == 0 ? 256 : R() % 257);
    std::vector<int2> P;
    std::set<std::pair<int, int>> seen;
    auto add = [&](int i, int j) {
      if (i > j) std::swap(i, j);
      if (i != j && (int)P.size() < 256 && seen.emplace(i, j).second) P.push_back({i, j});
    };
    for (int k = 0; k < want; ++k) {
      if (kind == 0) add(R() % n, R() % n);
      if (kind == 1 && k + 1 < n) add(k, k + 1);
      if (kind == 2 && k + 1 < n) add(R() % 2 ? 0 : n - 1, k + 1);
      if (kind == 3 && 2 * k + 1 < n) add(2 * k, 2 * k + 1);
      if (kind == 4) {
        const int b = R() % n;
        add(b, min<int>(n - 1, b + R() % 6));
      }
    }
    std::vector<int> perm(n);
    std::iota(perm.begin(), perm.end(), 0);
    if (R() % 2) std::shuffle(perm.begin(), perm.end(), R);
    std::shuffle(P.begin(), P.end(), R);
    for (int2& p : P) p = {min(perm[p.x], perm[p.y]), max(perm[p.x], perm[p.y])};
    const int ne = (int)P.size();
    for (int i = 0; i < N; ++i) {
      L.link[i] = (int)(R() % 100000) - 50000;
      L.first[i] = -7;
      L.gid[i] = 12345;
    }
    for (int i = 0; i < N / 2; ++i) L.roots[i] = -1;
    for (int i = 0; i <= N / 2; ++i) L.gsz[i] = L.gof[i] = 99999;
    Stat st{};
    const EncArgs a{{P.data(), ne}, {&goff}, {&gmem}, &st};
    int ret[64];
    const unsigned seed = R();
    std::vector<std::thread> th;
    for (int l = 0; l < 64; ++l)
      th.emplace_back([&, l] {
        threadIdx.x = l;
        rng.seed(seed + l * 7919);
        ret[l] = group_few<64, Lds<N>>(a, ne, L, Ptr{&gm}, true, l < ne ? P[l] : int2{0, 0});
      });
    for (auto& x : th) x.join();
    // union-find: the groups in order of their smallest member
    std::vector<int> u(n);
    std::iota(u.begin(), u.end(), 0);
    auto root = [&](int i) {
      while (u[i] != i) i = u[i] = u[u[i]];
      return i;
    };
    std::set<int> in;
    for (const int2& p : P) {
      const int x = root(p.x), y = root(p.y);
      u[max(x, y)] = min(x, y);
      in.insert({p.x, p.y});
    }
    std::map<int, std::vector<int>> groups;
    for (int i : in) groups[root(i)].push_back(i);
    bool ok = st.ngroups == (int)groups.size() && (int)st.enc_total == ne;
    for (int l = 0; l < 64; ++l) ok = ok && ret[l] == st.ngroups;
    int g = 0, off = 0, most = 0;
    for (auto& [r, m] : groups) {
      if (!ok) break;
      most = max<int>(most, m.size());
      ok = L.gof[g] == off && goff[g] == off;
      std::vector<int> h, w;
      for (size_t k = 0; ok && k < m.size(); ++k) {
        h.push_back(gm[off + (int)k]);
        w.push_back(gmem[off + (int)k]);
      }
      std::sort(h.begin(), h.end());
      std::sort(w.begin(), w.end());
      ok = ok && h == m && w == m;
      off += (int)m.size();
      ++g;
    }
    ok = ok && L.gof[g] == off && goff[g] == off && st.maxg == most;
    if (!ok) {
      printf("wrong groups: %d bodies of %d, %d pairs, kind %d\n", n, N, ne, kind);
      return 1;
    }
  }
  return 0;
}

int main() {
  std::mt19937 R(20250);
  return run<2048>(R, 60) || run<32>(R, 50) || run<16>(R, 50);
}
