// Which upload buffers of released layouts are handed to other layouts (upload_staging.h), with a runtime of counters in
// place of HIP.
#include "upload_staging.h"

#include <cstdio>
#include <cstdlib>

static bool no_memory = false;
void* operator new(size_t n) {
  if (no_memory) throw std::bad_alloc();
  return std::malloc(n ? n : 1);
}
void* operator new(size_t n, const std::nothrow_t&) noexcept { return no_memory ? nullptr : std::malloc(n ? n : 1); }
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, size_t) noexcept { std::free(p); }

struct Event_ {
  int device;
  bool done;
  bool refuses = false;   // cannot be asked
};
struct Runtime {
  typedef Event_* Event;
  static inline int waits = 0, destroyed = 0, freed = 0, last_error = 0;
  static bool query(Event e) {
    if (!e->done || e->refuses) last_error = e->refuses ? 2 : 1;
    return e->done && !e->refuses;
  }
  static void forget_error() { last_error = 0; }
  static void wait(Event e) { ++waits; e->done = true; }
  static void destroy(Event e) { ++destroyed; delete e; }
  static void free_host(void*) { ++freed; }
};
typedef UploadStaging<Runtime> Staging;
typedef StagingPool<Staging, Runtime> Pool;

#define REQUIRE(x) do { if (!(x)) { std::printf("FAILED line %d: %s\n", __LINE__, #x); std::exit(1); } } while (0)

static Staging* used(int device0, int device1, bool done = true) {   // two uploads behind it (device -1: not made)
  Staging* s = new Staging;
  const int device[2] = {device0, device1};
  for (int i = 0; i < 2; ++i)
    if (device[i] >= 0) {
      s->done[i] = new Event_{device[i], done};
      s->device[i] = device[i];
      s->in_use[i] = true;
      s->buffer[i] = s;
      s->capacity[i] = 4096;
    }
  return s;
}

static void events_of_two_devices() {
  Pool pool;
  pool.give(used(0, 1));
  REQUIRE(Runtime::freed == 2);                     // such a pair serves no one else
  Staging* one = used(1, -1);
  pool.give(one);
  Staging* fresh = pool.take(0);
  REQUIRE(fresh != one && !fresh->done[0]);
  REQUIRE(pool.take(1) == one);
  pool.give(fresh);
  pool.give(one);
  pool.drain();
}

static void finished_and_bounded() {
  Pool pool;
  Staging* busy = used(0, 0, false);
  pool.give(busy);
  Staging* other = pool.take(0);
  REQUIRE(other != busy);                           // nobody waits for another layout's stream
  busy->done[0]->done = busy->done[1]->done = true;
  REQUIRE(pool.take(0) == busy && !busy->in_use[0] && !busy->in_use[1]);
  delete other;
  delete busy;
  const int freed = Runtime::freed;
  for (size_t i = 0; i < Pool::kKept + 3; ++i) pool.give(used(0, 0));
  REQUIRE(Runtime::freed == freed + 2 * 3);
  Staging* large = used(0, 0);
  large->capacity[1] = Pool::kBytes + 1;
  pool.give(large);
  REQUIRE(Runtime::freed == freed + 2 * 4);
  pool.drain();
  REQUIRE(Runtime::freed == freed + 2 * (4 + int(Pool::kKept)));
}

static void answers_of_events_are_no_errors() {
  for (bool refuses : {false, true}) {
    Pool pool;
    Staging* s = used(0, 0, refuses);
    s->done[0]->refuses = s->done[1]->refuses = refuses;
    pool.give(s);
    Staging* fresh = pool.take(0);
    REQUIRE(fresh != s && Runtime::last_error == 0);
    delete fresh;
    pool.drain();
  }
}

static void giving_back_needs_no_memory() {
  Pool pool;
  for (int round = 0; round < 3; ++round) {
    Staging* s[Pool::kKept + 1];
    for (Staging*& one : s) one = used(0, 0);
    no_memory = true;
    for (Staging* one : s) pool.give(one);          // (from a destructor: an exception would end the process)
    pool.drain();                                   // the last block pool is destroyed
    no_memory = false;
  }
}

static void copies_without_an_event() {
  Pool pool;
  Staging* s = used(0, 0);
  s->in_use[1] = false;
  s->unrecorded = true;                             // the upload went out, its event was refused
  const int freed = Runtime::freed;
  pool.give(s);
  REQUIRE(Runtime::freed == freed + 2);
  pool.drain();
}

int main() {
  events_of_two_devices();
  finished_and_bounded();
  answers_of_events_are_no_errors();
  giving_back_needs_no_memory();
  copies_without_an_event();
  std::puts("ok");
  return 0;
}
