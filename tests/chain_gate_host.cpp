// The order of chains (csrc/chain_gate.hpp) with a fake device that logs what is asked of it.
// Prints the name of every check that fails.
#include "chain_gate.hpp"

#include <atomic>
#include <chrono>
#include <cstdio>
#include <string>
#include <thread>
#include <vector>

using namespace nc;

static std::vector<std::string> events;  // by number - 1: what the event was last recorded behind
static std::vector<std::string> calls;
static std::vector<std::string> streams(16);  // by stream: its last launch
static bool record_fails = false;
static std::mutex log_m;

struct Fake {
  using Stream = int;
  using Event = int;
  static void wait(int s, int e) {
    std::lock_guard<std::mutex> l(log_m);
    calls.push_back("s" + std::to_string(s) + " waits for " + events[e - 1]);
  }
  static bool record(int& e, int s) {
    std::lock_guard<std::mutex> l(log_m);
    if (record_fails) return false;
    if (!e) {
      events.push_back("");
      e = (int)events.size();
    }
    events[e - 1] = streams[s];
    return true;
  }
  static void destroy(int e) {
    if (e) events[e - 1] = "destroyed";
  }
};

static int failed = 0;
static void check(const char* what, const std::vector<std::string>& want) {
  if (calls != want) {
    std::printf("%s:", what);
    for (auto& c : calls) std::printf(" [%s]", c.c_str());
    std::printf("\n");
    ++failed;
  }
  calls.clear();
}

constexpr int kRoom = 256;
static int go(ChainGate<Fake>& g, const void* owner, int s, int tiles, const char* name, int result = 0) {
  return g.launch(owner, s, tiles, kRoom, [&] {
    std::lock_guard<std::mutex> l(log_m);
    if (!result) {
      streams[s] = name;
      calls.push_back(name);
    }
    return result;
  });
}

int main() {
  int A, B, C;
  {
    ChainGate<Fake> g;
    go(g, &A, 1, 255, "a1");
    go(g, &A, 1, 255, "a2");
    check("one stream: nothing but launches", {"a1", "a2"});
    go(g, &B, 2, 255, "b1");  // a2 was launched when nobody else was there: no event
    go(g, &A, 1, 255, "a3");
    go(g, &B, 2, 255, "b2");
    check("two large ones alternate", {"b1", "s1 waits for b1", "a3", "s2 waits for a3", "b2"});
    streams[1] = "other work of stream 1";
    go(g, &B, 2, 255, "b3");
    check("a wait is for the chain, not for what follows it", {"s2 waits for a3", "b3"});
    g.leave(&A);
    go(g, &B, 2, 255, "b4");
    check("a context that has gone is not waited for", {"b4"});
  }
  {
    ChainGate<Fake> g;
    go(g, &A, 1, 104, "a1");
    go(g, &B, 2, 104, "b1");
    go(g, &A, 1, 104, "a2");
    go(g, &B, 2, 104, "b2");
    check("two that fit together do not wait", {"a1", "b1", "a2", "b2"});
    go(g, &C, 3, 104, "c1");
    check("a third waits for the oldest", {"s3 waits for a2", "c1"});
    go(g, &A, 1, 104, "a3");
    check("and the first then for the second", {"s1 waits for b2", "a3"});
    go(g, &C, 4, 510, "c2");
    check("more tiles than room: after all others", {"s4 waits for b2", "s4 waits for c1", "s4 waits for a3", "c2"});
  }
  {
    ChainGate<Fake> g;
    go(g, &A, 1, 200, "a1");
    go(g, &B, 2, 10, "b1");
    go(g, &C, 1, 10, "c1");  // behind a1 on the same stream, which may still run
    go(g, &B, 2, 100, "b2");
    check("a small chain behind a large one counts as the large one", {"a1", "b1", "c1", "s2 waits for c1", "b2"});
    g.leave(&A);             // c1 is the stream's last chain
    go(g, &B, 2, 250, "b3");
    check("its entry stays with the last launch", {"s2 waits for c1", "b3"});
  }
  {
    ChainGate<Fake> g;
    go(g, &A, 1, 255, "a1");
    go(g, &B, 2, 255, "b1");
    if (go(g, &A, 1, 255, "a2", 7) != 7) ++failed;
    calls.clear();
    go(g, &B, 2, 255, "b2");
    check("a launch that failed leaves no trace", {"b2"});
    record_fails = true;
    go(g, &A, 1, 255, "a3");
    record_fails = false;
    go(g, &B, 2, 255, "b3");
    check("an event that could not be recorded is not waited for", {"s1 waits for b2", "a3", "b3"});
  }
  {
    // a second thread comes between the first one's look around and its launch
    ChainGate<Fake> g;
    go(g, &A, 1, 255, "a0");
    go(g, &B, 2, 255, "b0");
    calls.clear();
    std::atomic<bool> inside{false}, second{false};
    std::thread a([&] {
      g.launch(&A, 1, 255, kRoom, [&] {
        inside = true;
        while (!second) std::this_thread::yield();
        std::this_thread::sleep_for(std::chrono::milliseconds(50));
        std::lock_guard<std::mutex> l(log_m);
        streams[1] = "a1";
        calls.push_back("a1");
        return 0;
      });
    });
    while (!inside) std::this_thread::yield();
    std::thread b([&] {
      second = true;
      go(g, &B, 2, 255, "b1");
    });
    a.join();
    b.join();
    check("launches are one after the other, each behind the last", {"s1 waits for b0", "a1", "s2 waits for a1", "b1"});
  }
  return failed ? 1 : 0;
}
