// Runs a kernel's source as it stands on the CPU, a fiber per thread, in any order of the threads between two barriers, and stops at
// the first access that a GPU would let pass: an index behind an array, a shared element that nothing has written, two
// threads at one element between the same barriers (not both atomic), a loop that does not end.
#include <climits>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <functional>
#include <memory>
#include <vector>
#include <ucontext.h>

#define __global__ static
#define __device__ static
#define __forceinline__ inline
#define __launch_bounds__(n)

struct Index { int x, y, z; };
static Index threadIdx, blockIdx;
static int epoch_;            // barriers passed
static long accesses_;        // of one thread since its last barrier
static std::function<void()> barrier_;
static void __syncthreads() { barrier_(); }

[[noreturn]] static void fault(const char* what, const char* array, long i) {
  printf("FAULT %s: %s[%ld], thread %d, block %d, behind barrier %d\n", what, array, i, threadIdx.x, blockIdx.x, epoch_);
  fflush(stdout);
  _exit(3);
}
static void count(const char* name) {
  if (++accesses_ > 2000000) fault("a loop does not end", name, -1);
}

// ---- global memory: bounds ----
template <class T>
struct Global {
  const char* name = "null"; T* p = nullptr; long n = 0;
  T& operator[](long i) const {
    count(name);
    if (i < 0 || i >= n) fault("index out of range", name, i);
    return p[i];
  }
  explicit operator bool() const { return p != nullptr; }
};

// ---- shared memory: bounds, initialisation, races ----
struct Track { int w = -1, w_at = -1, r = -1, r_at = -1; bool w_atomic = false, many = false, written = false; };
static std::vector<std::function<void()>> shared_resets_;   // shared arrays are new for every workgroup
template <class T>
struct Ref {
  const char* name; long i; T* p; Track* k;
  T get() const {
    if (!k->written) fault("read of what nothing wrote", name, i);
    if (k->w_at == epoch_ && k->w != threadIdx.x) fault("race (read)", name, i);
    if (k->r_at != epoch_) { k->r_at = epoch_; k->r = threadIdx.x; k->many = false; }
    else if (k->r != threadIdx.x) k->many = true;
    return *p;
  }
  void put(T v, bool atomic = false) const {
    if (k->w_at == epoch_ && k->w != threadIdx.x && !(atomic && k->w_atomic)) fault("race (write)", name, i);
    if (k->r_at == epoch_ && (k->many || k->r != threadIdx.x)) fault("race (write after read)", name, i);
    k->w = threadIdx.x; k->w_at = epoch_; k->w_atomic = atomic; k->written = true;
    *p = v;
  }
  operator T() const { return get(); }
  const Ref& operator=(T v) const { put(v); return *this; }
  const Ref& operator=(const Ref& o) const { put(o.get()); return *this; }
  Ref(const char* n, long at, T* x, Track* t) : name(n), i(at), p(x), k(t) {}
  Ref(const Ref&) = default;
  const Ref& operator|=(T v) const { put(get() | v); return *this; }
  const Ref& operator+=(T v) const { put(get() + v); return *this; }
  Ref operator&() const { return *this; }
};
template <class T, int N, int M = 1>
struct Shared {
  const char* name; std::vector<T> v; std::vector<Track> k;
  explicit Shared(const char* n) : name(n) {
    shared_resets_.push_back([this] { v.assign(N * M, (T)7); k.assign(N * M, Track{}); });
    shared_resets_.back()();
  }
  Ref<T> at(long i) {
    count(name);
    if (i < 0 || i >= N * M) fault("index out of range", name, i);
    return Ref<T>(name, i, &v[i], &k[i]);
  }
  struct Row { Shared& s; long i; Ref<T> operator[](long j) const { if (j < 0 || j >= M) fault("index out of range", s.name, j); return s.at(i * M + j); } };
  auto operator[](long i) {
    if constexpr (M == 1) return at(i);
    else { if (i < 0 || i >= N) fault("index out of range", name, i); return Row{*this, i}; }
  }
  operator T() { return at(0); }                    // (a single variable)
  void operator=(T x) { at(0) = x; }
  Ref<T> operator&() { return at(0); }
};
template <class T> static void atomicAdd(const Ref<T>& r, T v) { if (!r.k->written) fault("atomic on what nothing wrote", r.name, r.i); r.put(*r.p + v, true); }
template <class T> static void atomicMin(const Ref<T>& r, T v) { if (!r.k->written) fault("atomic on what nothing wrote", r.name, r.i); r.put(v < *r.p ? v : *r.p, true); }

// ---- a launch: `threads` fibers per block, resumed in the order of a permutation drawn from `seed` (0: ascending, 1: descending) ----
struct Fiber { ucontext_t at; std::unique_ptr<char[]> stack; bool done; };
static ucontext_t main_;
static std::vector<Fiber> fibers_;
static int running_;
static std::function<void()> body_;
static void enter() { body_(); fibers_[running_].done = true; }
static void launch(int blocks, int threads, unsigned seed, std::function<void()> body) {
  body_ = body;
  barrier_ = [] { swapcontext(&fibers_[running_].at, &main_); };
  for (int b = 0; b < blocks; ++b) {
    blockIdx = {b, 0, 0};
    epoch_ = 0;
    for (auto& f : shared_resets_) f();
    fibers_.resize(threads);
    std::vector<int> order(threads);
    for (int t = 0; t < threads; ++t) order[t] = seed == 1 ? threads - 1 - t : t;
    srand(seed);
    if (seed > 1)
      for (int t = threads - 1; t > 0; --t) std::swap(order[t], order[rand() % (t + 1)]);
    for (int t = 0; t < threads; ++t) {
      Fiber& f = fibers_[t];
      if (!f.stack) f.stack.reset(new char[65536]);
      getcontext(&f.at);
      f.at.uc_stack.ss_sp = f.stack.get();
      f.at.uc_stack.ss_size = 65536;
      f.at.uc_link = &main_;
      f.done = false;
      makecontext(&f.at, enter, 0);
    }
    for (bool any = true; any; ++epoch_) {
      any = false;
      for (int t : order) {
        if (fibers_[t].done) continue;
        running_ = t;
        threadIdx = {t, 0, 0};
        accesses_ = 0;
        swapcontext(&main_, &fibers_[t].at);
        any = any || !fibers_[t].done;
      }
    }
  }
}
