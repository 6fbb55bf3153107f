// Checks of the blocking calls' idle sessions (bn_sessions.h) over a counting
// host device: what is kept, handed out, destroyed after an error, released when
// memory runs out or on request, and forgotten when the device was reset.
#include <cstdio>
#include <cstdlib>
#include <map>
#include <thread>
#include <vector>

#include "../../paper_1408_1664_amd/csrc/bn_sessions.h"

struct Fake {
    struct Events {
        int made = 0;
    };
    static std::mutex mu;
    static int dev, events_alive, bad_frees;
    static bool have_device, events_fail;
    static size_t limit, used;
    static uint64_t next;
    struct Block {
        size_t bytes;
        uint64_t id;
    };
    static std::map<char *, Block> live;
    static bool get(size_t bytes, char **p, uint64_t *id) {
        std::lock_guard<std::mutex> lk(mu);
        *p = nullptr;
        if (used + bytes > limit) return false;
        *p = (char *)malloc(1);
        *id = ++next;
        live[*p] = Block{bytes, *id};
        used += bytes;
        return true;
    }
    static void put(char *p) {
        std::lock_guard<std::mutex> lk(mu);
        auto it = live.find(p);
        if (it == live.end()) {
            ++bad_frees;
            return;
        }
        used -= it->second.bytes;
        live.erase(it);
        free(p);
    }
    static void reset() {
        for (auto &kv : live) free(kv.first);
        live.clear();
        used = 0;
    }
    static bool current(int *d) {
        *d = dev;
        return have_device;
    }
    static bool holds(char *p, uint64_t id) {
        std::lock_guard<std::mutex> lk(mu);
        auto it = live.find(p);
        return it != live.end() && it->second.id == id;
    }
    static bool alloc(size_t bytes, char **p, uint64_t *id, bool *lost) {
        *lost = !have_device;
        return !*lost && get(bytes, p, id);
    }
    static bool alloc_pinned(size_t bytes, char **p, uint64_t *id) { return get(bytes, p, id); }
    static void release(char *p) { put(p); }
    static void release_pinned(char *p) { put(p); }
    static bool make_events(Events &e) {
        if (events_fail) return false;
        e.made = 1;
        ++events_alive;
        return true;
    }
    static void destroy_events(Events &e) {
        events_alive -= e.made;
        e.made = 0;
    }
};
std::mutex Fake::mu;
int Fake::dev = 0, Fake::events_alive = 0, Fake::bad_frees = 0;
bool Fake::have_device = true, Fake::events_fail = false;
size_t Fake::limit = (size_t)1 << 40, Fake::used = 0;
uint64_t Fake::next = 0;
std::map<char *, Fake::Block> Fake::live;

using Pool = bnk::SessionPool<Fake>;
using S = Pool::S;
static constexpr size_t kMB = (size_t)1 << 20;
static int failed = 0;
static void expect(const char *name, bool ok) {
    failed += ok ? 0 : 1;
    printf("%s %s\n", ok ? "ok  " : "FAIL", name);
}

int main() {
    Pool pool;
    S a, b, c;
    expect("a first call allocates", pool.take(10 * kMB, true, &a) == Pool::Got::ok && a.ws && a.pin &&
                                         a.events && a.bytes == 10 * kMB);
    char *ws = a.ws;
    pool.give(a, true);
    expect("the next one takes it over", pool.take(8 * kMB, false, &a) == Pool::Got::ok && a.ws == ws &&
                                             a.bytes == 10 * kMB && a.events);
    expect("a call beside it gets its own", pool.take(8 * kMB, false, &b) == Pool::Got::ok && b.ws != ws &&
                                                b.pin != a.pin && !b.events);
    pool.give(a, false);
    expect("a failed call's session is destroyed", !a.ws && !a.pin && Fake::live.size() == 2 &&
                                                       Fake::events_alive == 0);
    pool.give(b, true);
    expect("only the other one is handed out", pool.take(1 * kMB, false, &a) == Pool::Got::ok &&
                                                   a.bytes == 8 * kMB);
    Fake::events_fail = true;
    expect("failed events are no events", pool.take(1 * kMB, true, &b) == Pool::Got::ok && !b.events);
    Fake::events_fail = false;
    pool.give(b, true);
    expect("and are created later", pool.take(1 * kMB, true, &b) == Pool::Got::ok && b.events);
    pool.give(a, true);
    pool.give(b, true);
    pool.release();
    expect("release frees everything idle", Fake::live.empty() && Fake::used == 0 && Fake::events_alive == 0);
    pool.take(100 * kMB, false, &a);
    pool.give(a, true);
    expect("large memory is not kept", Fake::used == Pool::kPinBytes);
    pool.release();
    std::vector<S> many(7);
    for (S &s : many) pool.take(64 * kMB, true, &s);
    for (S &s : many) pool.give(s, true);
    expect("at most four are kept", Fake::used == 4 * (64 * kMB + Pool::kPinBytes) && Fake::events_alive == 4);
    Fake::limit = 300 * kMB;
    expect("idle memory goes when an allocation needs it",
           pool.take(250 * kMB, false, &a) == Pool::Got::ok && a.bytes == 250 * kMB && Fake::used <= Fake::limit);
    expect("no memory", pool.take(100 * kMB, false, &b) == Pool::Got::no_memory && !b.ws && !b.pin);
    pool.give(a, true);
    Fake::limit = (size_t)1 << 40;
    pool.take(5 * kMB, true, &a);
    pool.take(6 * kMB, true, &b);
    pool.take(7 * kMB, true, &c);
    S busy;
    pool.take(3 * kMB, true, &busy);
    pool.give(c, true);
    pool.give(a, true);
    pool.give(b, true);
    expect("the smallest that fits", pool.take(6 * kMB, false, &a) == Pool::Got::ok && a.bytes == 6 * kMB);
    pool.give(a, true);
    Fake::dev = 1;
    expect("another device has its own", pool.take(1 * kMB, false, &a) == Pool::Got::ok && a.dev == 1 &&
                                             a.bytes == 1 * kMB);
    pool.give(a, true);
    Fake::dev = 0;
    Fake::reset();
    expect("after a device reset old memory is neither used nor freed",
           pool.take(1 * kMB, false, &a) == Pool::Got::ok && a.bytes == 1 * kMB &&
               Fake::holds(a.ws, a.ws_id) && Fake::holds(a.pin, a.pin_id) && Fake::bad_frees == 0);
    pool.give(a, true);
    Fake::reset();
    pool.release();
    expect("nor on release", Fake::bad_frees == 0);
    Fake::have_device = false;
    expect("no device", pool.take(1, false, &a) == Pool::Got::no_device);
    Fake::have_device = true;
    std::vector<std::thread> th;
    std::map<char *, int> seen;
    std::mutex mu;
    bool shared = false;
    for (int t = 0; t < 8; ++t)
        th.emplace_back([&] {
            for (int k = 0; k < 2000; ++k) {
                S s;
                pool.take((k % 5 + 1) * kMB, k & 1, &s);
                {
                    std::lock_guard<std::mutex> lk(mu);
                    shared = shared || ++seen[s.ws] > 1;
                }
                std::this_thread::yield();
                {
                    std::lock_guard<std::mutex> lk(mu);
                    --seen[s.ws];
                }
                pool.give(s, k % 7 != 0);
                if (k % 100 == 0) pool.release();
            }
        });
    for (auto &t : th) t.join();
    pool.release();
    expect("threads never share one", !shared && Fake::bad_frees == 0);
    expect("nothing is left", Fake::live.empty() && Fake::used == 0);
    return failed ? 1 : 0;
}
