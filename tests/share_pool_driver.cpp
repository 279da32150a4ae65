// SharePool (csrc/share_pool.h) on a runtime of counters: streams are queues whose work ends when the test says so, and
// a destroyed stream's handle goes to the next one created. After every lend: whoever used the buffer before has
// finished, or is this very stream, or is waited for.
#include "../paper_2507_17245_amd/csrc/share_pool.h"

#include <cstdio>
#include <cstdlib>
#include <map>
#include <random>
#include <set>
#include <vector>

#define CHECK(x) \
  do { \
    if (!(x)) { \
      std::printf("line %d: %s\n", __LINE__, #x); \
      std::exit(1); \
    } \
  } while (0)

struct Queue {          // one stream's life; work items are numbered
  long queued = 0, finished = 0;
};
struct Mark {           // an item of a queue
  int life = -1;
  long item = 0;
};
std::vector<Queue> lives;
std::map<int, int> life_of;                         // handle -> the life it names now
std::map<int, Mark> events;
std::map<std::pair<int, int>, long> waited_item;    // (life, life it waits for) -> item
std::set<void*> memory;
int next_event = 1, fail_allocate = 0, fail_record = 0, most_memory = 0;

struct Fake {
  typedef int Stream;
  typedef int Event;
  static bool allocate(void** p) {
    if (fail_allocate) return false;
    *p = std::malloc(1);
    memory.insert(*p);
    if ((int)memory.size() > most_memory) most_memory = (int)memory.size();
    return true;
  }
  static bool deallocate(void* p) {
    CHECK(memory.erase(p) == 1);
    std::free(p);
    return true;
  }
  static bool create(Event* e) {
    events[*e = next_event++] = Mark();
    return true;
  }
  static bool destroy(Event e) { return events.erase(e) == 1; }
  static bool record(Event e, Stream s) {
    if (fail_record) return false;
    CHECK(events.count(e));
    CHECK(!lasting(s));
    events[e] = Mark{life_of.at(s), lives[life_of.at(s)].queued};
    return true;
  }
  static bool wait(Stream s, Event e) {
    const Mark m = events.at(e);
    if (m.life >= 0) waited_item[{life_of.at(s), m.life}] = m.item;
    return true;
  }
  static bool lasting(Stream s) { return s == 0; }
  static bool done(Event e) {
    const Mark m = events.at(e);
    return m.life < 0 || lives[m.life].finished >= m.item;
  }
};

da::SharePool<Fake> pool;
std::map<void*, Mark> last_user;   // of a buffer (it came after those before it)

int create_stream(int handle) {
  lives.push_back(Queue());
  life_of[handle] = (int)lives.size() - 1;
  return handle;
}
void finish(int handle) { lives[life_of.at(handle)].finished = lives[life_of.at(handle)].queued; }

// One call: lend, queue work, give back.
void* call(int stream) {
  const int life = life_of.at(stream);
  void* p = pool.lend(stream);
  if (!p) return nullptr;
  CHECK(memory.count(p));
  const Mark m = last_user[p];
  const auto w = waited_item.find({life, m.life});
  CHECK(m.life < 0 || m.life == life || lives[m.life].finished >= m.item || (w != waited_item.end() && w->second >= m.item));
  last_user[p] = Mark{life, ++lives[life].queued};
  pool.give_back();
  return p;
}

int main() {
  // one live stream: one buffer, also while its work is in flight
  create_stream(1);
  void* a = call(1);
  CHECK(a && call(1) == a && call(1) == a && memory.size() == 1);
  finish(1);
  // streams one after the other take it over
  for (int i = 0; i < 100; ++i) {
    create_stream(100 + i);
    CHECK(call(100 + i) == a);
    finish(100 + i);
  }
  CHECK(memory.size() == 1);
  // a stream destroyed with work in flight, its handle given to the next: the new stream waits
  create_stream(2);
  CHECK(call(2) == a);
  const int before = life_of[2];
  create_stream(2);
  CHECK(call(2) == a && waited_item.count({life_of[2], before}));
  // a lasting stream: a buffer that no other stream gets, in flight or not
  create_stream(0);
  void* own = call(0);
  finish(0);
  CHECK(own && own != a && call(0) == own && memory.size() == 2);
  for (int i = 0; i < 40; ++i) CHECK(call(create_stream(2)) == a);
  // streams at work at the same time have buffers of their own, as many as the pool holds
  for (int i = 0; i < 14; ++i) CHECK(call(create_stream(10 + i)));
  CHECK(memory.size() == 16 && call(create_stream(50)) == nullptr);
  finish(12);
  CHECK(call(50));
  // an event that cannot be recorded: the buffer stays out
  finish(13);
  create_stream(60);
  fail_record = 1;
  void* out = call(60);
  fail_record = 0;
  CHECK(out);
  finish(60);
  for (int i = 0; i < 40; ++i) CHECK(call(60) != out);
  CHECK(memory.size() == 16);
  CHECK(pool.clear() && memory.empty() && events.empty() && pool.empty());
  last_user.clear();
  // no memory to have
  fail_allocate = 1;
  CHECK(call(create_stream(70)) == nullptr && pool.empty() && events.empty());
  fail_allocate = 0;
  // any order of all this
  std::mt19937 rng(1);
  most_memory = 0;
  for (int step = 0; step < 200000; ++step) {
    const int h = (int)(rng() % 24), what = (int)(rng() % 16);
    if (!life_of.count(h) || (what == 0 && h != 0)) create_stream(h);
    else if (what < 4) finish(h);
    else call(h);
    if (step % 50000 == 49999) {
      CHECK(pool.clear() && memory.empty());
      last_user.clear();
    }
  }
  CHECK(most_memory == 16);
  CHECK(pool.clear());
  std::printf("ok\n");
  return 0;
}
