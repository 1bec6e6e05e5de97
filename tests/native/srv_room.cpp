// Host test of the server scheduler's choice of workspace (srv_core.hpp): a request that runs
// faster with more memory than it needs gets it only where no other request loses its place.
// The executor holds every launch until it is told to finish.
#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <map>
#include <thread>

#include "srv_core.hpp"

#define CHECK(c)                                                                   \
  do {                                                                             \
    if (!(c)) {                                                                    \
      std::fprintf(stderr, "CHECK failed at %s:%d: %s\n", __FILE__, __LINE__, #c); \
      std::abort();                                                                \
    }                                                                              \
  } while (0)

using cqsrv::Req;

constexpr size_t MB = 1 << 20;

class HoldExec final : public cqsrv::Executor {
 public:
  void dispatch(int slot, const std::vector<Req*>& reqs, bool grouped, size_t, size_t len) override {
    std::lock_guard<std::mutex> lk(mu_);
    CHECK(!grouped && reqs.size() == 1);
    CHECK(len == cqsrv::req_footprint(*reqs[0]));
    ws_[reqs[0]->id] = reqs[0]->ws_bytes;
    at_[slot] = reqs[0]->id;
  }
  bool finished(int slot) override {
    std::lock_guard<std::mutex> lk(mu_);
    return free_.count(at_[slot]) != 0;
  }
  void collect(int, const std::vector<Req*>&, bool) override {}
  void finish(uint64_t id) {
    std::lock_guard<std::mutex> lk(mu_);
    free_[id] = true;
  }
  size_t workspace_of(uint64_t id) {  // 0: not started
    std::lock_guard<std::mutex> lk(mu_);
    return ws_.count(id) ? ws_[id] : 0;
  }

 private:
  std::mutex mu_;
  std::map<uint64_t, size_t> ws_;
  std::map<int, uint64_t> at_;
  std::map<uint64_t, bool> free_;
};

struct Sim {
  HoldExec ex;
  cqsrv::Scheduler s;
  Sim(int slots, size_t budget) : s(config(slots, budget), &ex) {}
  static cqsrv::Config config(int slots, size_t budget) {
    cqsrv::Config c;
    c.num_slots = slots;
    c.arena_bytes = budget;
    return c;
  }
  uint64_t submit(size_t least, size_t more) {
    Req* r = new Req();
    r->n = 64;
    r->ws_bytes = least;
    r->ws_more = more;
    uint64_t t = 0;
    CHECK(s.submit(r, &t, nullptr) == CQ_OK);
    return t;
  }
  // the request's workspace once it runs
  size_t runs_with(uint64_t t) {
    for (int i = 0; i < 20000; ++i) {
      if (const size_t w = ex.workspace_of(t)) return w;
      std::this_thread::sleep_for(std::chrono::microseconds(100));
    }
    return 0;
  }
  void end(uint64_t t) {
    ex.finish(t);
    CHECK(s.wait(t, -1, nullptr, nullptr) == CQ_OK);
  }
};

int main() {
  {  // two at once fit a budget of 8 MB by their least sizes; the larger of one would keep the other out
    Sim m(2, 8 * MB);
    m.s.start();
    const uint64_t a = m.submit(3 * MB, 6 * MB);
    CHECK(m.runs_with(a) == 3 * MB);
    const uint64_t b = m.submit(3 * MB, 6 * MB);
    CHECK(m.runs_with(b) == 3 * MB);  // beside a
    m.end(a);
    m.end(b);
  }
  {  // the larger size where the other still fits, the least one where no more is left
    Sim m(2, 8 * MB);
    m.s.start();
    const uint64_t a = m.submit(3 * MB, 4 * MB);
    CHECK(m.runs_with(a) == 4 * MB);
    const uint64_t b = m.submit(3 * MB, 4 * MB);
    CHECK(m.runs_with(b) == 3 * MB);
    m.end(a);
    m.end(b);
  }
  {  // a larger request queued behind counts with its own size
    Sim m(2, 8 * MB);
    const uint64_t a = m.submit(3 * MB, 4 * MB), b = m.submit(4 * MB + MB / 2, 0);
    m.s.start();
    CHECK(m.runs_with(a) == 3 * MB);
    CHECK(m.runs_with(b) == 4 * MB + MB / 2);
    m.end(a);
    m.end(b);
  }
  {  // and so does the largest one seen, though it has finished
    Sim m(2, 8 * MB);
    const uint64_t a = m.submit(4 * MB + MB / 2, 0);
    m.s.start();
    CHECK(m.runs_with(a) == 4 * MB + MB / 2);
    m.end(a);
    const uint64_t b = m.submit(3 * MB, 4 * MB);
    CHECK(m.runs_with(b) == 3 * MB);
    m.end(b);
  }
  {  // one slot: nothing can run beside it
    Sim m(1, 8 * MB);
    m.s.start();
    const uint64_t a = m.submit(3 * MB, 7 * MB);
    CHECK(m.runs_with(a) == 7 * MB);
    const uint64_t b = m.submit(3 * MB, 9 * MB);  // more than the arena
    m.end(a);
    CHECK(m.runs_with(b) == 3 * MB);
    m.end(b);
    CHECK(m.s.arena_in_use() == 0);
  }
  {  // a request that waits for memory may still get the larger size when its turn comes
    Sim m(2, 8 * MB);
    m.s.start();
    const uint64_t a = m.submit(6 * MB, 0);
    CHECK(m.runs_with(a) == 6 * MB);
    const uint64_t b = m.submit(3 * MB, 3 * MB + MB / 2);
    std::this_thread::sleep_for(std::chrono::milliseconds(5));
    CHECK(m.ex.workspace_of(b) == 0);
    const uint64_t c = m.submit(3 * MB, 0);
    m.end(a);
    CHECK(m.runs_with(b) == 3 * MB + MB / 2);
    CHECK(m.runs_with(c) == 3 * MB);
    m.end(b);
    m.end(c);
    CHECK(m.s.arena_in_use() == 0 && m.s.arena_free_blocks() == 1);
  }
  std::printf("srv_room: all passed\n");
}
