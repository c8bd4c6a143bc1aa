// Checks of stream_pool.hpp against a stand-in for the HIP calls it makes.
// Prints "ok", or the line of the first check that fails.
#include <cstdio>
#include <cstdlib>
#include <set>
#include <vector>

typedef int hipError_t;
typedef struct Stream* hipStream_t;
enum { hipSuccess = 0, hipErrorOutOfMemory = 2, hipErrorUnknown = 999, hipStreamNonBlocking = 1 };

static long made = 0;
static std::set<hipStream_t> alive;
static std::vector<int> create_fails;   // numbers of the creations (from 1) that fail
static hipStream_t broken = nullptr;    // its synchronization fails

static hipError_t hipStreamCreateWithFlags(hipStream_t* s, int) {
  ++made;
  for (int f : create_fails)
    if (f == made) return hipErrorOutOfMemory;
  *s = reinterpret_cast<hipStream_t>(made * 16);
  alive.insert(*s);
  return hipSuccess;
}
static hipError_t hipStreamDestroy(hipStream_t s) {
  if (!alive.erase(s)) std::abort();
  return hipSuccess;
}
static hipError_t hipStreamSynchronize(hipStream_t s) { return s == broken ? hipErrorUnknown : hipSuccess; }
static hipError_t hipGetLastError() { return hipSuccess; }

#include "stream_pool.hpp"

#define CHECK(x)                           \
  do {                                     \
    if (!(x)) {                            \
      std::printf("%d: %s\n", __LINE__, #x); \
      return 1;                            \
    }                                      \
  } while (0)

int main() {
  using namespace gls;
  auto yes = [](hipStream_t, hipStream_t) { return true; };
  auto no = [](hipStream_t, hipStream_t) { return false; };
  {  // a failed second creation leaves nothing behind, and the next try makes a whole pair
    StreamPool pool;
    StreamPair p;
    create_fails = {2};
    CHECK(pool.take_pair(0, yes, &p) == hipErrorOutOfMemory);
    CHECK(!p.there() && !p.st[0] && !p.st[1] && alive.empty());
    CHECK(pool.take_pair(0, yes, &p) == hipSuccess && p.there() && p.checked);
    pool.give_pair(0, &p);
    CHECK(!p.st[0] && !p.st[1] && alive.size() == 2);
    StreamPair q;
    const long before = made;
    CHECK(pool.take_pair(0, no, &q) == hipSuccess && made == before && q.checked);   // kept pairs have passed
    pool.give_pair(0, &q);
    CHECK(pool.take_pair(1, yes, &q) == hipSuccess && made == before + 2);   // another device's
    pool.give_pair(1, &q);
  }
  alive.clear();
  {  // a pair that no copy stream made pass is used, but not kept
    StreamPool pool;
    StreamPair p;
    int looks = 0;
    create_fails = {};
    CHECK(pool.take_pair(0, [&](hipStream_t, hipStream_t) { return ++looks, false; }, &p) == hipSuccess);
    CHECK(p.there() && !p.checked && looks == 5 && alive.size() == 2);
    pool.give_pair(0, &p);
    CHECK(alive.empty());
    looks = 0;   // the third copy stream passes
    CHECK(pool.take_pair(0, [&](hipStream_t, hipStream_t) { return ++looks == 3; }, &p) == hipSuccess);
    CHECK(p.there() && p.checked && alive.size() == 2);
    create_fails = {(int)made + 3};   // of another pair's, the first replacement fails: the pair stays, unchecked
    StreamPair q;
    CHECK(pool.take_pair(0, no, &q) == hipSuccess && q.there() && !q.checked && alive.size() == 4);
    pool.give_pair(0, &q);
    broken = p.st[1];   // a stream with an error is not kept
    pool.give_pair(0, &p);
    CHECK(alive.empty());
  }
  {  // at most POOL_MAX are kept
    StreamPool pool;
    StreamPair p[6];
    hipStream_t s[6];
    broken = nullptr;
    create_fails = {};
    for (auto& x : p) CHECK(pool.take_pair(0, yes, &x) == hipSuccess);
    for (auto& x : s) CHECK(pool.take_side(0, &x) == hipSuccess);
    CHECK(alive.size() == 18);
    for (auto& x : p) pool.give_pair(0, &x);
    for (auto& x : s) pool.give_side(0, x);
    CHECK(alive.size() == 3 * StreamPool::POOL_MAX);
    StreamPair empty;
    pool.give_pair(0, &empty);   // a handle that never streamed
    CHECK(alive.size() == 3 * StreamPool::POOL_MAX);
  }
  std::puts("ok");
  return 0;
}
