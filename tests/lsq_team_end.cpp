// A model of a least-squares team (paper_1910_12308_amd/csrc/lsq_team.hip) on the host: its workgroups are fibers that a seeded
// generator runs in any order, changing after every access to what they share, and every look for words that are not there may be the
// last one that a workgroup has patience for.  What such a workgroup does then is the kernel's own code (lsq_team_end.hpp).
//   lsq_team_end schedules reducers [wrong]
// runs so many random schedules and prints how many of them did not end, in how many a slice of a node was not written, in how many a
// workgroup gave up with an error, and in how many the next launch's numbers were not the same for all, or had been used.  wrong: a claim that nobody made lies on the way, so that workgroups wait for what does not come.
#include <algorithm>
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
    TeamClaim claim = ~0ull, claim_before = ~0ull;        // and what a load that is late still finds
    std::vector<uint32_t> number;                         // of the next launch's first step, a copy for each workgroup
    uint32_t highest = 0;                                 // number that a word has carried
    std::vector<std::vector<bool>> written;               // [node][column]
    std::mt19937_64 gen;
    double patience;                                      // chance that a workgroup waits on
    bool wrong = false, lost = false, numbered = true;

    bool tired() { return std::generate_canonical<double, 32>(gen) > patience; }
    TeamWait give_up(uint32_t first, uint32_t done, bool overdue) {
        return swarm::out_of_patience(first, done, overdue, [&] { return seen(); },
                                      [&](TeamClaim expected, TeamClaim mine) { return swap(expected, mine); });
    }
    TeamClaim seen() {
        yield();
        return gen() % 4 ? claim : claim_before;
    }
    TeamClaim swap(TeamClaim expected, TeamClaim mine) {
        yield();
        const TeamClaim before = claim;
        if (before == expected) { claim_before = claim; claim = mine; }
        return before;
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
    void carry(uint32_t tag) { highest = std::max(highest, tag); }
    void alone(uint32_t step, uint32_t tag) {
        for (uint32_t k = step / steps_each * steps_each; k < nodes * steps_each; ++k) {
            carry(++tag);
            for (uint32_t c = 0; c < columns; ++c) {
                yield();
                if (k % steps_each == steps_each - 1) written[k / steps_each][c] = true;
            }
        }
    }
    void move_on(uint32_t m, uint32_t first) {
        yield();
        number[m] = swarm::next_number(first, nodes * steps_each);
    }
    void column(uint32_t c) {
        yield();
        const uint32_t first = number[c], steps = nodes * steps_each;
        const TeamClaim there = seen();
        TeamWait then = (uint32_t)(there >> 32) == first ? TeamWait::END : TeamWait::GO_ON;
        uint32_t k = 0;
        for (; k < steps && then == TeamWait::GO_ON; ++k) {
            const uint32_t tag = first + k;
            yield();
            carry(part[tag & 1u][c] = tag);
            then = wait(total[tag & 1u], first, tag, true);
            if (then != TeamWait::GO_ON) break;
            if (k % steps_each == steps_each - 1) {
                yield();
                written[k / steps_each][c] = true;
            }
        }
        move_on(c, first);
        if (then == TeamWait::ALONE) alone(k, first + k);
        if (then == TeamWait::GO_ON && c == 0) swap(there, (TeamClaim)first << 32 | steps);
    }
    void reducer(uint32_t j) {
        yield();
        const uint32_t first = number[columns + j], steps = nodes * steps_each;
        const TeamClaim there = seen();
        TeamWait then = (uint32_t)(there >> 32) == first ? TeamWait::END : TeamWait::GO_ON;
        for (uint32_t k = 0; k < steps && then == TeamWait::GO_ON; ++k) {
            const uint32_t tag = first + k;
            then = wait(part[tag & 1u], first, tag, false);
            if (then != TeamWait::GO_ON) break;
            yield();
            carry(total[tag & 1u][j] = tag);
        }
        move_on(columns + j, first);
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
        size_t left = fibers.size(), late = gen() % 3 ? 0 : 1 + gen() % left;          // the last to be let in when all others have ended
        const size_t order = gen() % left;
        for (size_t turns = 0; left; ++turns) {
            if (turns == 10000 * fibers.size()) return false;
            const size_t some_one = gen() % fibers.size();
            if (left > late && (some_one + order) % fibers.size() < late) continue;
            if (left <= late) late = 0;
            running = fibers[some_one].get();
            if (running->ended) continue;
            const uint32_t some = 1 + gen() % 8;          // accesses in a row
            for (uint32_t k = 0; k < some && !running->ended; ++k) swapcontext(&scheduler, &running->context);
            left -= running->ended;
            if (wrong && (uint32_t)(claim >> 32) != number[0] && gen() % 16 == 0) claim = (TeamClaim)number[0] << 32 | (1 + gen() % (nodes * steps_each));
        }
        claim_before = claim;                             // a launch finds what the ones before it have left
        for (const uint32_t v : number) numbered = numbered && v == number[0] && v > highest;
        return true;
    }
};

}  // namespace

int main(int argc, char **argv) {
    if (argc < 3) return 2;
    const uint32_t schedules = (uint32_t)std::atoi(argv[1]), reducers = (uint32_t)std::atoi(argv[2]);
    uint32_t endless = 0, unwritten = 0, lost = 0, misnumbered = 0;
    for (uint32_t seed = 0; seed < schedules; ++seed) {
        Team t;
        t.gen.seed(seed);
        t.columns = 2 + seed % 2;
        t.reducers = reducers;
        t.steps_each = 1 + seed / 2 % 3;
        t.nodes = 2;
        t.wrong = argc > 3;
        t.patience = seed % 3 == 0 ? 0.5 : seed % 3 == 1 ? 0.9 : 0.98;
        t.number.assign(t.columns + reducers, 0);
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
        misnumbered += !t.numbered;
    }
    std::printf("endless %u unwritten %u lost %u misnumbered %u\n", endless, unwritten, lost, misnumbered);
    return 0;
}
