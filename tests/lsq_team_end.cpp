// A model of a least-squares team (paper_1910_12308_amd/csrc/lsq_team.hip) on the host: its workgroups are fibers that a seeded
// generator runs in any order, changing after every access to what they share, and every look for words that are not there may be the
// last one that a workgroup has patience for.  What such a workgroup does then is the kernel's own code (lsq_team_end.hpp).
//   lsq_team_end schedules reducers [wrong]
// runs so many random schedules and prints how many of them did not end, in how many a slice of a node was not written, and in how many
// a workgroup gave up with an error.  wrong: a claim that nobody made lies on the way, so that workgroups wait for what does not come.
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <functional>
#include <memory>
#include <random>
#include <vector>

#include <ucontext.h>

#include "lsq_team_end.hpp"

using swarm::TeamClaim;
using swarm::TeamWait;

namespace {

// Fibers, and a scheduler that goes to any of those that have not ended.
struct Fiber {
    ucontext_t context;
    std::vector<char> stack;
    std::function<void()> body;
    bool ended = false;
};
ucontext_t scheduler;
Fiber *running = nullptr;
void yield() { swapcontext(&running->context, &scheduler); }
void enter_fiber() {
    running->body();
    running->ended = true;
    yield();
}

struct Team {
    uint32_t columns, reducers, steps_each, nodes;        // nodes: that the team takes one after the other in a launch
    std::vector<uint32_t> part[2], total[2];              // numbers of the words, by the parity of the number
    TeamClaim claim = ~0ull;
    uint32_t number = 0;                                  // of the next launch's first step
    std::vector<std::vector<bool>> written;               // [node][column]
    std::mt19937_64 gen;
    double patience;                                      // chance that a workgroup waits on
    bool wrong = false, lost = false;

    bool tired() { return std::generate_canonical<double, 32>(gen) > patience; }
    TeamWait give_up(uint32_t first, uint32_t done, bool overdue) {
        return swarm::out_of_patience(first, done, overdue, [&] { yield(); return claim; },
                                      [&](TeamClaim expected, TeamClaim mine) {
                                          yield();
                                          const TeamClaim before = claim;
                                          if (before == expected) claim = mine;
                                          return before;
                                      });
    }
    // Until all the words carry the number; whoever makes no claim ends when it has waited long enough.
    TeamWait wait(const std::vector<uint32_t> &words, uint32_t first, uint32_t with, bool claims) {
        for (uint32_t looks = 0;; ++looks) {
            bool there = true;
            for (const uint32_t &w : words) {
                yield();
                there = there && w == with;
            }
            if (there) return TeamWait::GO_ON;
            if (tired()) {
                if (!claims) return TeamWait::END;
                const TeamWait then = give_up(first, with - first, looks > 500);
                lost = lost || then == TeamWait::LOST;
                if (then != TeamWait::GO_ON) return then;
            }
        }
    }
    void alone(uint32_t step) {
        for (uint32_t node = step / steps_each; node < nodes; ++node)
            for (uint32_t c = 0; c < columns; ++c) {
                yield();
                written[node][c] = true;
            }
    }
    bool claimed(uint32_t first) {
        yield();
        return (uint32_t)(claim >> 32) == first;
    }
    void column(uint32_t c) {
        yield();
        const uint32_t first = number, steps = nodes * steps_each;
        if (claimed(first)) return;
        for (uint32_t k = 0; k < steps; ++k) {
            const uint32_t tag = first + k;
            yield();
            part[tag & 1u][c] = tag;
            const TeamWait then = wait(total[tag & 1u], first, tag, true);
            if (then == TeamWait::ALONE) return alone(k);
            if (then != TeamWait::GO_ON) return;
            if (k % steps_each == steps_each - 1) {
                yield();
                written[k / steps_each][c] = true;
            }
        }
        if (c == 0 && !claimed(first)) {                  // the kernel's is one compare and exchange
            const TeamClaim mine = (TeamClaim)first << 32 | steps;
            if ((uint32_t)(claim >> 32) != first) claim = mine;
        }
    }
    void reducer(uint32_t j) {
        yield();
        const uint32_t first = number, steps = nodes * steps_each;
        if (claimed(first)) return;
        for (uint32_t k = 0; k < steps; ++k) {
            const uint32_t tag = first + k;
            if (wait(part[tag & 1u], first, tag, false) == TeamWait::END) return;
            yield();
            total[tag & 1u][j] = tag;
        }
    }
    // One launch; false: not all its workgroups end.
    bool launch() {
        std::vector<std::unique_ptr<Fiber>> fibers;
        written.assign(nodes, std::vector<bool>(columns, false));
        for (uint32_t m = 0; m < columns + reducers; ++m) {
            auto f = std::make_unique<Fiber>();
            f->stack.resize(32768);
            f->body = [this, m] { m < columns ? column(m) : reducer(m - columns); };
            getcontext(&f->context);
            f->context.uc_stack.ss_sp = f->stack.data();
            f->context.uc_stack.ss_size = f->stack.size();
            f->context.uc_link = nullptr;
            makecontext(&f->context, enter_fiber, 0);
            fibers.push_back(std::move(f));
        }
        size_t left = fibers.size();
        for (size_t turns = 0; left; ++turns) {
            if (turns == 10000 * fibers.size()) return false;
            running = fibers[gen() % fibers.size()].get();
            if (running->ended) continue;
            const uint32_t some = 1 + gen() % 8;          // accesses in a row
            for (uint32_t k = 0; k < some && !running->ended; ++k) swapcontext(&scheduler, &running->context);
            left -= running->ended;
            if (wrong && (uint32_t)(claim >> 32) != number && gen() % 16 == 0) claim = (TeamClaim)number << 32 | (1 + gen() % (nodes * steps_each));
        }
        number += nodes * steps_each;
        return true;
    }
};

}  // namespace

int main(int argc, char **argv) {
    if (argc < 3) return 2;
    const uint32_t schedules = (uint32_t)std::atoi(argv[1]), reducers = (uint32_t)std::atoi(argv[2]);
    uint32_t endless = 0, unwritten = 0, lost = 0;
    for (uint32_t seed = 0; seed < schedules; ++seed) {
        Team t;
        t.gen.seed(seed);
        t.columns = 2 + seed % 2;
        t.reducers = reducers;
        t.steps_each = 1 + seed / 2 % 3;
        t.nodes = 2;
        t.wrong = argc > 3;
        t.patience = seed % 3 == 0 ? 0.5 : seed % 3 == 1 ? 0.9 : 0.98;
        for (auto &w : t.part) w.assign(t.columns, ~0u);
        for (auto &w : t.total) w.assign(t.reducers, ~0u);
        bool ended = true, whole = true;
        for (int launch = 0; launch < 3 && ended && whole; ++launch) {
            ended = t.launch();
            for (const auto &node : t.written)
                for (const bool w : node) whole = whole && w;
        }
        endless += !ended;
        unwritten += ended && !whole;
        lost += t.lost;
    }
    std::printf("endless %u unwritten %u lost %u\n", endless, unwritten, lost);
    return 0;
}
