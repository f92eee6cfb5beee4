// The claim of a sequence call's sets (csrc/rnn_seq_placement.hpp) on the host: its workgroups as coroutines that hand over before every
// access to the claim's words, in an order drawn at random.  As on the GPU, workgroups start in the order of their ids, no more of
// them run at once than there is room for, and those of a set stay until the whole set has come together.
#include <ucontext.h>

#include <cstdint>
#include <random>
#include <vector>

#include "rnn_seq_placement.hpp"

namespace {
struct Group {
    ucontext_t context;
    std::vector<char> stack;
    unsigned int xcd;
    int set = -1, unit = -1;
    bool running = false, claimed = false, gone = false;
};
struct Call {
    grim::SeqClaim claim = {};
    std::vector<Group> groups;
    ucontext_t scheduler;
    Group *now = nullptr;
    int sets, wgs, polls;
} *g_call;

void hand_over() { swapcontext(&g_call->now->context, &g_call->scheduler); }

struct Memory {
    static unsigned int add_one(unsigned int *at) { hand_over(); return (*at)++; }
    static unsigned int load(unsigned int *at) { hand_over(); return *at; }
    static void store_and_wait(unsigned int *at, unsigned int v) { hand_over(); *at = v; }
    static unsigned int set_if_zero(unsigned int *at, unsigned int v) { hand_over(); const unsigned int was = *at; if (was == 0) *at = v; return was; }
    static void pause() { hand_over(); }
};

void body() {
    Call *const c = g_call;
    Group *const g = c->now;
    grim::seq_claim(&c->claim, Memory{}, g->xcd, c->sets, c->wgs, c->polls, &g->set, &g->unit);
    g->claimed = true;
    hand_over();
}
}  // namespace

// The mode the claim ended in, or < 0: -1 a (set, unit) that is nobody's or out of range, -2 one that two workgroups have, -3 a set
// that is placed and runs on several XCDs, -4 workgroups that wait for each other for ever.
// xcds: 0: ids are dealt to eight XCDs in turn, 1: all on one, 2: at random, 3: at random to two.  room: workgroups that run at once.
extern "C" int seq_claim_outcome(int sets, int wgs, int xcds, int polls, int room, int seed) {
    std::mt19937 rng(seed);
    Call c;
    c.sets = sets;
    c.wgs = wgs;
    c.polls = polls;
    c.groups.resize((size_t)8 * ((sets + 7) / 8 * wgs));
    g_call = &c;
    for (size_t i = 0; i < c.groups.size(); ++i) {
        Group &g = c.groups[i];
        g.xcd = xcds == 0 ? i % 8 : xcds == 1 ? 3 : xcds == 2 ? rng() % 8 : rng() % 2;
        g.stack.resize(32 * 1024);
        getcontext(&g.context);
        g.context.uc_stack.ss_sp = g.stack.data();
        g.context.uc_stack.ss_size = g.stack.size();
        g.context.uc_link = nullptr;
        makecontext(&g.context, body, 0);
    }
    std::vector<int> seen((size_t)sets * wgs, 0), together((size_t)sets, 0);
    std::vector<Group *> active;
    size_t next = 0;
    int held = 0, left = (int)c.groups.size();                     // workgroups that occupy a place; that have not gone
    while (left > 0) {
        while (next < c.groups.size() && held < room) {
            active.push_back(&c.groups[next++]);
            ++held;
        }
        if (active.empty()) return -4;
        const size_t at = rng() % active.size();
        c.now = active[at];
        swapcontext(&c.scheduler, &c.now->context);
        Group *const g = c.now;
        if (!g->claimed) continue;
        active.erase(active.begin() + at);
        if (g->set < 0) {
            --held;
            --left;
            continue;
        }
        if (g->set >= sets || g->unit < 0 || g->unit >= wgs) return -1;
        if (seen[(size_t)g->set * wgs + g->unit]++) return -2;
        if (++together[g->set] == wgs) {                           // the set has come together: it runs and leaves
            held -= wgs;
            left -= wgs;
        }
    }
    for (int n : seen)
        if (n != 1) return -1;
    if (c.claim.mode == grim::kClaimPlaced) {
        std::vector<int> home((size_t)sets, -1);
        for (const Group &g : c.groups) {
            if (g.set < 0) continue;
            if (home[g.set] >= 0 && home[g.set] != (int)g.xcd) return -3;
            home[g.set] = (int)g.xcd;
        }
    }
    return (int)c.claim.mode;
}
