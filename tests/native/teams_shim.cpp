// Host build of batch_teams.h for the CPU tests: a thread per workgroup of one
// XCD, and slots with tags written and read as the exchange of the batch
// sampler does.  One workgroup can be held back before it reads an exchange.
#include <atomic>
#include <chrono>
#include <thread>
#include <vector>

#include "../../paper_2606_06255_amd/csrc/batch_teams.h"

namespace {

using Word = std::atomic<unsigned long long>;

struct World {
    int per_xcd, batch;
    const uint32_t *level_first;  // [kBatchLevels + 1]
    const int *exchanges;         // [batch] of every place in the order; 0: needs none
    int slow, at_exchange;        // the workgroup held back and before which of its exchanges
    bool wait;                    // whether a team waits for its workgroups before it splits
    std::vector<Word> slots, posts, counts, taken, epochs, samples;
    std::atomic<bool> over{false};

    World(int x, int b)
        : per_xcd(x), batch(b), slots(2 * x), posts(rfps::kBatchLevels * x), counts(rfps::kBatchLevels * x),
          taken(rfps::kBatchLevels), epochs(x), samples(b)
    {
    }
};

struct Io {
    World &w;
    int me;
    uint32_t epoch = 0;
    bool lost = false;
    uint32_t kSpins = 1u << 30, looks = 0;  // (`over` ends every wait)

    unsigned long long look(const Word &v)
    {
        if (w.over) {
            lost = true;
            kSpins = 0;
        }
        if (++looks % 64 == 0)
            std::this_thread::sleep_for(std::chrono::microseconds(20));
        return v.load();
    }
    uint32_t next(int lev) { return (uint32_t)w.taken[lev].fetch_add(1); }
    bool wanted(uint32_t q) { return w.exchanges[q] > 0; }
    void post(int lev, int T, unsigned long long v) { w.posts[lev * w.per_xcd + (me & ~(T - 1))] = v; }
    unsigned long long posted(int lev, int T)
    {
        return look(w.posts[lev * w.per_xcd + (me & ~(T - 1))]);
    }
    void arrive(int lev, int T) { w.counts[lev * w.per_xcd + (me & ~(T - 1))].fetch_add(1); }
    unsigned long long arrived(int lev, int T)
    {
        const unsigned long long v = look(w.counts[lev * w.per_xcd + (me & ~(T - 1))]);
        return w.wait ? v : ~0ull;
    }
    uint32_t first(int lev) { return w.level_first[lev]; }
    template <class F>
    uint32_t one(F f)
    {
        return f();
    }
    bool sample(int, int T, int rank, uint32_t q)
    {
        for (int e = 0; e < w.exchanges[q] && T > 1; ++e) {
            ++epoch;
            const int team = me - rank;
            w.slots[2 * me + (epoch & 1u)] = epoch;
            w.epochs[me] = epoch;
            if (me == w.slow && (int)epoch == w.at_exchange) {
                // held back until another workgroup is two exchanges ahead, or
                // all have had time to be
                const auto end = std::chrono::steady_clock::now() + std::chrono::milliseconds(60);
                bool ahead = false;
                while (!ahead && std::chrono::steady_clock::now() < end) {
                    for (const Word &v : w.epochs)
                        ahead |= v.load() >= epoch + 2;
                    std::this_thread::yield();
                }
            }
            for (int g = team; g < team + T; ++g) {
                for (;;) {
                    const unsigned long long v = look(w.slots[2 * g + (epoch & 1u)]);
                    if (v == epoch)
                        break;
                    if (v > epoch || lost) {  // written again before it was read
                        lost = true;
                        w.over = true;
                        return false;
                    }
                }
            }
        }
        w.samples[q].fetch_add(1);
        return !lost;
    }
};

}  // namespace

// Runs a batch; members[q] counts the workgroups that sampled the cloud at
// place q.  Returns 0, or 1 when a read was lost or a workgroup gave up.
extern "C" int shim_teams(int per_xcd, int batch, const unsigned *level_first, const int *exchanges, int slow,
                          int at_exchange, int wait, int *members)
{
    World w(per_xcd, batch);
    w.level_first = level_first;
    w.exchanges = exchanges;
    w.slow = slow;
    w.at_exchange = at_exchange;
    w.wait = wait != 0;
    std::atomic<int> failed{0};
    std::vector<std::thread> all;
    for (int g = 0; g < per_xcd; ++g)
        all.emplace_back([&, g] {
            Io io{w, g};
            if (!rfps::walk_levels(io, per_xcd, g) || io.lost) {
                failed = 1;
                w.over = true;
            }
        });
    for (std::thread &t : all)
        t.join();
    for (int q = 0; q < batch; ++q)
        members[q] = (int)w.samples[q].load();
    return failed;
}

extern "C" int shim_levels() { return rfps::kBatchLevels; }
