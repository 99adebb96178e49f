// Runs the operations on the word of a tile split along K (csrc/split_word.hpp) in random orders against a memory that lets a
// plain store arrive late, over several chains that use the same word.  Exit code 0: every slice of every chain was finished
// once, from partials that had been left, and the word was zero at the end.
//   split_word_check RUNS            the code as it is
//   split_word_check RUNS no-drain   a memory whose drain() waits for nothing: the check has to see it
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <random>
#include <vector>

#include <ucontext.h>

#include "split_word.hpp"

using namespace depsync;

namespace {

constexpr uint32_t CHAINS = 3, MAX_S = 8;
constexpr size_t STACK = 64 << 10;
bool g_drains = true;

struct Part {
    ucontext_t ctx;
    std::vector<char> stack;
    uint32_t chain, z;
    bool running, done, clear_pending;
    bool left[MAX_S];       // slices of its partials that are in memory
};

struct World {
    std::mt19937 rng;
    uint32_t S = 0, word = 0, slots = 0;
    bool outlives = false;
    std::vector<bool> has_slice;
    std::vector<Part> parts;
    uint32_t finished[CHAINS][MAX_S], posted[CHAINS];
    ucontext_t main;
    Part* now = nullptr;
    const char* error = nullptr;
    void yield() { swapcontext(&now->ctx, &main); }
    void fail(const char* what) { if (!error) error = what; }
    uint32_t pick(uint32_t n) { return std::uniform_int_distribution<uint32_t>(0, n - 1)(rng); }
    void flush(Part& p) { if (p.clear_pending) { p.clear_pending = false; word = 0; } }
};
World* g;

struct Mem {
    uint32_t load() { g->yield(); return g->word; }
    uint32_t add(uint32_t v) {
        g->yield();
        g->flush(*g->now);                       // operations of one lane on one address keep their order
        const uint32_t old = g->word;
        g->word += v;
        return old;
    }
    void clear() { g->yield(); g->now->clear_pending = true; }
    void drain() { g->yield(); if (g_drains) g->flush(*g->now); }
    bool wait_published(uint32_t S) {
        while (split_published(load()) != S) {}
        return true;
    }
};

// One part of the tile, as in gemm_tile.hpp.
void run_part() {
    Part& p = *g->now;
    const uint32_t S = g->S, z = p.z, c = p.chain;
    Mem m;
    m.add(SPLIT_STARTED);
    for (uint32_t i = g->pick(8); i > 0; --i) g->yield();
    const uint32_t seen = m.load();
    for (uint32_t i = 0; i < S; ++i) p.left[i] = i != z;
    uint32_t todo = split_publish(m, S, z, g->has_slice[z], split_all_started(seen, S));
    if (todo == SPLIT_AGAIN) {
        p.left[z] = true;
        todo = split_publish_whole(m, S, z);
    }
    for (uint32_t i = 0; i < S; ++i) {
        if (!((todo >> i) & 1u)) continue;
        g->yield();
        for (uint32_t o = 0; o < S; ++o)
            if (!(o == z && i == z) && !g->parts[c * S + o].left[i]) g->fail("a slice was summed before all parts had left it");
        g->finished[c][i] += 1;
    }
    split_leave(m, S, g->outlives, [&] {
        g->yield();
        for (uint32_t i = 0; i < S; ++i)
            if (g->finished[c][i] != (g->has_slice[i] ? 1u : 0u)) g->fail("posted with a slice missing or finished twice");
        g->posted[c] += 1;
    });
    p.running = false;
    p.done = true;
    for (;;) g->yield();
}

const char* run(uint32_t seed) {
    World w;
    g = &w;
    w.rng.seed(seed);
    w.S = 2 + w.pick(MAX_S - 1);
    w.slots = 1 + w.pick(2 * w.S);               // resident workgroups: fewer than parts, or more
    w.outlives = w.pick(2) != 0;
    for (uint32_t i = 0; i < w.S; ++i) w.has_slice.push_back(w.pick(5) != 0);
    std::memset(w.finished, 0, sizeof(w.finished));
    std::memset(w.posted, 0, sizeof(w.posted));
    w.parts.resize(CHAINS * w.S);
    for (uint32_t i = 0; i < w.parts.size(); ++i) {
        Part& p = w.parts[i];
        p.chain = i / w.S; p.z = i % w.S;
        p.running = p.done = p.clear_pending = false;
        std::memset(p.left, 0, sizeof(p.left));
        p.stack.resize(STACK);
        getcontext(&p.ctx);
        p.ctx.uc_stack.ss_sp = p.stack.data();
        p.ctx.uc_stack.ss_size = STACK;
        p.ctx.uc_link = &w.main;
        makecontext(&p.ctx, run_part, 0);
    }
    uint32_t next = 0;                           // parts are started in order, as slots come free
    for (uint64_t step = 0; !w.error; ++step) {
        if (step > 200000) { w.fail("no progress"); break; }
        std::vector<uint32_t> can;
        uint32_t resident = 0, done = 0;
        for (const Part& p : w.parts) { resident += p.running; done += p.done; }
        if (done == w.parts.size()) break;
        if (next < w.parts.size() && resident < w.slots) {
            const uint32_t c = w.parts[next].chain;
            bool may = true;                     // a chain begins when the one before has posted, or when its launch has ended
            if (c > 0 && w.outlives) may = w.posted[c - 1] != 0;
            else if (c > 0)
                for (uint32_t z = 0; z < w.S; ++z) may = may && w.parts[(c - 1) * w.S + z].done;
            if (may) {
                if (c > 0 && !w.outlives)
                    for (uint32_t z = 0; z < w.S; ++z) w.flush(w.parts[(c - 1) * w.S + z]);
                can.push_back(2 * (uint32_t)w.parts.size());
            }
        }
        for (uint32_t i = 0; i < w.parts.size(); ++i) {
            if (w.parts[i].running) can.push_back(i);
            if (w.parts[i].clear_pending && w.pick(4) == 0) can.push_back((uint32_t)w.parts.size() + i);
        }
        if (can.empty()) {
            bool pending = false;
            for (const Part& p : w.parts) pending = pending || p.clear_pending;
            if (!pending) { w.fail("nothing can run"); break; }
            continue;
        }
        const uint32_t e = can[w.pick((uint32_t)can.size())], n = (uint32_t)w.parts.size();
        if (e == 2 * n) { w.parts[next++].running = true; continue; }
        if (e >= n) { w.flush(w.parts[e - n]); continue; }
        w.now = &w.parts[e];
        swapcontext(&w.main, &w.parts[e].ctx);
    }
    if (!w.error) {
        for (Part& p : w.parts) w.flush(p);
        if (w.word != 0) w.fail("the word is not zero after the chains");
        for (uint32_t c = 0; c < CHAINS; ++c)
            if (w.posted[c] != 1) w.fail("a chain posted not once");
    }
    return w.error;
}

}  // namespace

int main(int argc, char** argv) {
    const uint32_t runs = argc > 1 ? (uint32_t)std::atoi(argv[1]) : 1000;
    g_drains = !(argc > 2 && std::strcmp(argv[2], "no-drain") == 0);
    for (uint32_t seed = 0; seed < runs; ++seed)
        if (const char* e = run(seed)) { std::printf("seed %u: %s\n", seed, e); return 1; }
    std::printf("%u orders\n", runs);
    return 0;
}
