// The cases of tests/test_host_sources.py, one by name: prints "ok" or what
// went wrong.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <new>

#include "../../include/dl.h"
#include "../../paper_1608_00139_amd/csrc/ctx.h"
#include "runtime.h"

static long g_fail_new = 0;  // the how manyth allocation from now fails (0: none)
void* operator new(size_t bytes) {
  if (g_fail_new > 0 && --g_fail_new == 0) throw std::bad_alloc();
  if (void* p = std::malloc(bytes ? bytes : 1)) return p;
  throw std::bad_alloc();
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, size_t) noexcept { std::free(p); }

namespace {

int bad(const char* what, long long got) {
  std::printf("%s: %lld (%s)\n", what, got, dl_last_error());
  return 1;
}

const char* kClosure = "tc(X,Y) :- e(X,Y).\ntc(X,Y) :- e(X,Z), tc(Z,Y).\n";
uint8_t* const kSome = (uint8_t*)64;  // a matrix that nothing reads here

// A relation bound at another size after a run: the results of the last run
// stay what they were until the next one.
int fetch_after_rebind() {
  dl_ctx* ctx = nullptr;
  dl_program* p = nullptr;
  if (int rc = dl_create(&ctx, 0, 0)) return bad("create", rc);
  if (int rc = dl_program_create(ctx, kClosure, &p)) return bad("program", rc);
  if (int rc = dl_program_bind(p, "e", 300, kSome, 300)) return bad("bind", rc);
  if (int rc = dl_program_run(p, DL_EVAL_ITERATION, nullptr)) return bad("run", rc);
  for (const int64_t n : {3000, 100, 0, 300}) {
    if (int rc = dl_program_bind(p, "e", n, kSome, n)) return bad("bind again", rc);
    int64_t ones = -1;
    for (const bool count : {true, false}) {
      fake::emits.clear();
      if (int rc = dl_program_fetch(p, "tc", kSome, 3000, count ? &ones : nullptr, nullptr)) return bad("fetch", rc);
      if (fake::emits.size() != 1) return bad("launches of a fetch", (long long)fake::emits.size());
      const fake::Emit e = fake::emits[0];
      if (e.n != 300 || e.Np != 512 || e.ld != 3000) return bad("constants fetched", e.n);
    }
    if (ones != 77) return bad("ones", ones);
    if (dl_program_fetch(p, "tc", kSome, 299, &ones, nullptr) != DL_EINVAL) return bad("stride 299 taken", n);
  }
  if (int rc = dl_program_bind(p, "e", 600, kSome, 600)) return bad("bind", rc);
  if (int rc = dl_program_run(p, DL_EVAL_ITERATION, nullptr)) return bad("run", rc);
  fake::emits.clear();
  if (int rc = dl_program_fetch(p, "tc", kSome, 600, nullptr, nullptr)) return bad("fetch", rc);
  if (fake::emits[0].n != 600 || fake::emits[0].Np != 768) return bad("constants of the second run", fake::emits[0].n);
  dl_program_destroy(p);
  dl_destroy(ctx);
  return fake::live ? bad("bytes left", (long long)fake::live) : 0;
}

// Memory that a program's matrices are kept in is given back before another
// allocation of the context is refused: a batch's pool and the temporary
// memory of its tuner.
int kept_matrices_given_up() {
  dl_ctx* ctx = nullptr;
  dl_program* p = nullptr;
  dl_batch* b = nullptr;
  if (int rc = dl_create(&ctx, 0, 0)) return bad("create", rc);
  const size_t before = fake::live;
  if (int rc = dl_program_create(ctx, kClosure, &p)) return bad("program", rc);
  auto fill = [&]() -> int {
    if (int rc = dl_program_bind(p, "e", 2000, kSome, 2000)) return rc;
    if (int rc = dl_program_run(p, DL_EVAL_ITERATION, nullptr)) return rc;
    if (int rc = dl_program_bind(p, "e", 0, nullptr, 0)) return rc;
    return dl_program_run(p, DL_EVAL_ITERATION, nullptr);  // gives its matrices back
  };
  if (int rc = fill()) return bad("run", rc);
  const size_t kept = fake::live - before;
  if (kept < (size_t)8 << 20) return bad("nothing was kept", (long long)kept);
  fake::limit = fake::live + ((size_t)4 << 20);
  if (int rc = dl_batch_create(ctx, 0, (size_t)8 << 20, 4, &b)) return bad("batch", rc);
  fake::limit = ~(size_t)0;
  if (int rc = fill()) return bad("run", rc);
  const int64_t sizes[] = {2048};  // eight requests of 16 MB and their descriptors
  fake::limit = fake::live + ((size_t)126 << 20);
  if (int rc = dl_batch_tune(b, sizes, 1, nullptr, nullptr, nullptr)) return bad("tune", rc);
  fake::limit = fake::live;  // and nothing left to give
  dl_batch* c = nullptr;
  if (dl_batch_create(ctx, 0, (size_t)8 << 20, 4, &c) != DL_ENOMEM || c) return bad("batch without memory", 0);
  dl_batch_destroy(b);
  dl_program_destroy(p);
  dl_destroy(ctx);
  return fake::live ? bad("bytes left", (long long)fake::live) : 0;
}

// Host memory that runs out is DL_ENOMEM, not an exception: one allocation
// after the other refused, in the calls that create and where matrices are
// given back to be kept.
int host_memory_runs_out() {
  for (long k = 1; k < 40; ++k) {
    dl_ctx* ctx = nullptr;
    dl_batch* b = nullptr;
    const char* at = "create";
    try {
      g_fail_new = k;
      int rc = dl_create(&ctx, 0, 0);
      g_fail_new = 0;
      if (rc != DL_OK && rc != DL_ENOMEM) return bad("create", rc);
      if (rc == DL_OK) {
        at = "batch";
        g_fail_new = k;
        rc = dl_batch_create(ctx, 0, 1 << 20, 4, &b);
        g_fail_new = 0;
        if (rc != DL_OK && rc != DL_ENOMEM) return bad("batch", rc);
        if ((rc == DL_OK) != (b != nullptr)) return bad("batch after", rc);
      }
      at = "put";
      MatPool pool;
      void* m = nullptr;
      if (pool.get(4096, &m) != hipSuccess) return bad("get", k);
      g_fail_new = k;
      pool.put(m, 4096);
      g_fail_new = 0;
    } catch (const std::bad_alloc&) {
      g_fail_new = 0;
      return bad(at, k);
    }
    dl_batch_destroy(b);
    dl_destroy(ctx);
    if (fake::live) return bad("bytes left", (long long)fake::live);
  }
  // what is kept stays under its limit, the oldest given back first
  MatPool pool;
  void* m[3];
  for (void*& q : m) pool.get(MatPool::kMaxKept / 2, &q);
  for (void* q : m) pool.put(q, MatPool::kMaxKept / 2);
  if (fake::live != MatPool::kMaxKept) return bad("kept", (long long)fake::live);
  pool.drop();
  return fake::live ? bad("bytes left", (long long)fake::live) : 0;
}

// The step numbers of the one-launch plain series' exchanged words: no launch
// uses one that an earlier launch has used since the words were cleared, none
// is zero, none runs over.
int launch_tags() {
  const uint64_t top = (uint64_t)~0u;
  unsigned last = 0u;
  bool clear = false;
  if (dl::fix_small_tag(&last, &clear) != dl::kFixSmallTags || clear) return bad("first tag", last);
  for (unsigned from : {~0u - 4 * dl::kFixSmallTags, ~0u - 3 * dl::kFixSmallTags + 1, ~0u - 2 * dl::kFixSmallTags,
                        ~0u - 2 * dl::kFixSmallTags + 1, ~0u}) {
    last = from;
    uint64_t used = from + (uint64_t)512 + 2;  // the last launch's highest
    for (int k = 0; k < 4; ++k) {
      clear = false;
      const unsigned tag = dl::fix_small_tag(&last, &clear);
      if (clear) used = 0;
      if (tag != last || tag + (uint64_t)1 <= used || tag == 0u) return bad("tag in use", tag);
      used = tag + (uint64_t)512 + 2;
      if (used > top) return bad("tag runs over", tag);
    }
  }
  return 0;
}

struct Case {
  const char* name;
  int (*run)();
};
const Case kCases[] = {{"fetch_after_rebind", fetch_after_rebind},
                        {"kept_matrices_given_up", kept_matrices_given_up},
                        {"host_memory_runs_out", host_memory_runs_out},
                        {"launch_tags", launch_tags}};

}  // namespace

int main(int argc, char** argv) {
  for (const Case& c : kCases)
    if (argc > 1 && !std::strcmp(argv[1], c.name)) {
      const int rc = c.run();
      if (!rc) std::printf("ok\n");
      return rc;
    }
  std::printf("no such case\n");
  return 2;
}
