// Every order in which the accesses of a few threads can meet, over the library's own union-find
// walks (sc_union.hpp): a thread is a fibre that stops before each access, and the orders are
// walked one after the other by replay.
#include <ucontext.h>

#include <cstdio>
#include <cstdlib>
#include <functional>
#include <memory>
#include <vector>

#define __device__
#define __forceinline__ inline
#include "sc_union.hpp"

namespace {

using Parents = std::vector<uint32_t>;

struct Fibre {
    ucontext_t ctx;
    std::vector<char> stack;
    std::function<void()> body;
    bool done = false;
};

ucontext_t scheduler;
Fibre* running = nullptr;

void stop() { swapcontext(&running->ctx, &scheduler); }
void enter()
{
    running->body();
    running->done = true;
    swapcontext(&running->ctx, &scheduler);
}

struct Mem {
    Parents* p;
    uint32_t load(uint32_t i) const { stop(); return (*p)[i]; }
    void store(uint32_t i, uint32_t v) const { stop(); (*p)[i] = v; }
    uint32_t min(uint32_t i, uint32_t v) const
    {
        stop();
        const uint32_t old = (*p)[i];
        if (v < old) (*p)[i] = v;
        return old;
    }
};

using Body = std::function<void(Mem)>;

// Runs the bodies over `start` in every order; returns how many orders end with `ok` false.
long wrong_orders(const Parents& start, const std::vector<Body>& bodies,
                  const std::function<bool(const Parents&)>& ok, long* orders)
{
    std::vector<int> choice, width;  // of the threads that can go on at each access, which went
    long bad = 0;
    *orders = 0;
    while (true) {
        Parents p = start;
        std::vector<std::unique_ptr<Fibre>> fibres;
        for (const Body& b : bodies) {
            auto f = std::make_unique<Fibre>();
            f->stack.resize(32768);
            f->body = [&p, &b] { b(Mem{&p}); };
            getcontext(&f->ctx);
            f->ctx.uc_stack.ss_sp = f->stack.data();
            f->ctx.uc_stack.ss_size = f->stack.size();
            f->ctx.uc_link = nullptr;
            makecontext(&f->ctx, enter, 0);
            fibres.push_back(std::move(f));
        }
        auto resume = [&](Fibre* f) { running = f; swapcontext(&scheduler, &f->ctx); };
        for (auto& f : fibres) resume(f.get());  // up to the first access
        for (size_t depth = 0;; ++depth) {
            std::vector<Fibre*> ready;
            for (auto& f : fibres)
                if (!f->done) ready.push_back(f.get());
            if (ready.empty()) break;
            if (depth == choice.size()) {
                choice.push_back(0);
                width.push_back((int)ready.size());
            }
            resume(ready[(size_t)choice[depth]]);
        }
        ++*orders;
        if (!ok(p)) ++bad;
        while (!choice.empty() && choice.back() + 1 == width.back()) {
            choice.pop_back();
            width.pop_back();
        }
        if (choice.empty()) return bad;
        ++choice.back();
    }
}

uint32_t root_of(const Parents& p, uint32_t x)
{
    while (p[x] != x) x = p[x];
    return x;
}

long total = 0, failed = 0;
void report(const char* what, int a, int b, long bad, long orders)
{
    total += orders;
    if (bad) {
        ++failed;
        std::printf("%s %d %d: %ld of %ld orders end wrong\n", what, a, b, bad, orders);
    }
}

}  // namespace

int main()
{
    long orders = 0;
    // a chain n - 1 -> .. -> 1 -> 0, two entries settled at once: both hold the root, and no entry
    // leaves its tree
    for (int n = 2; n <= 7; ++n) {
        Parents chain(n);
        for (int i = 0; i < n; ++i) chain[i] = (uint32_t)(i ? i - 1 : 0);
        for (int a = 0; a < n; ++a)
            for (int b = a + 1; b < n; ++b) {
                const long bad = wrong_orders(
                    chain,
                    {[a](Mem m) { sc::union_settle(m, (uint32_t)a); },
                     [b](Mem m) { sc::union_settle(m, (uint32_t)b); }},
                    [&](const Parents& p) {
                        bool good = p[a] == 0 && p[b] == 0;
                        for (int i = 0; i < n; ++i) good = good && root_of(p, (uint32_t)i) == 0;
                        return good;
                    },
                    &orders);
                report("settle", a, b, bad, orders);
            }
    }
    // three entries of a chain at once, every entry by a thread of its own
    {
        const Parents chain{0, 0, 1, 2};
        const long bad = wrong_orders(chain,
                                      {[](Mem m) { sc::union_settle(m, 1); },
                                       [](Mem m) { sc::union_settle(m, 2); },
                                       [](Mem m) { sc::union_settle(m, 3); }},
                                      [](const Parents& p) { return p == Parents{0, 0, 0, 0}; },
                                      &orders);
        report("settle", 3, 3, bad, orders);
    }
    // two unions at once, of every pair of links among three entries over three starts: their sets
    // are joined, and the walks that halve paths return the smallest entry
    const int links[3][2] = {{0, 1}, {1, 2}, {0, 2}};
    for (const Parents& start : {Parents{0, 1, 2}, Parents{0, 0, 2}, Parents{0, 1, 1}})
        for (int a = 0; a < 3; ++a)
            for (int b = 0; b < 3; ++b) {
                Parents want = start;  // the same links one after the other
                for (int l : {a, b}) {
                    const uint32_t x = root_of(want, (uint32_t)links[l][0]);
                    const uint32_t y = root_of(want, (uint32_t)links[l][1]);
                    want[x < y ? y : x] = x < y ? x : y;
                }
                auto unite = [&links](int l) -> Body {
                    return [&links, l](Mem m) {
                        sc::union_unite(m, (uint32_t)links[l][0], (uint32_t)links[l][1]);
                    };
                };
                const long bad = wrong_orders(
                    start, {unite(a), unite(b)},
                    [&](const Parents& p) {
                        bool good = true;
                        for (uint32_t i = 0; i < 3; ++i)
                            good = good && root_of(p, i) == root_of(want, i);
                        return good;
                    },
                    &orders);
                report("unite", a, b, bad, orders);
            }
    // two unions that halve a path while they meet at its end
    {
        const long bad = wrong_orders(
            Parents{0, 0, 1, 3},
            {[](Mem m) { sc::union_unite(m, 2, 3); }, [](Mem m) { sc::union_unite(m, 3, 2); }},
            [](const Parents& p) {
                bool good = true;
                for (uint32_t i = 0; i < 4; ++i) good = good && root_of(p, i) == 0;
                return good;
            },
            &orders);
        report("halve", 2, 3, bad, orders);
    }
    std::printf("%ld orders, %ld cases wrong\n", total, failed);
    return failed ? 1 : 0;
}
