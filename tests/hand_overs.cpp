// csrc/hands.hpp on the host: workgroups' waves as sets of fibers that a scheduler with a seed runs operation by operation, in any order that the
// hardware may, with stores that arrive late unless they are waited for and a clock that jumps, so that every wait runs out now and then.
// Launch after launch with the same tag, as a replayed graph has it.  usage: hand_overs rows|apart|levels|overlap seeds
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include <ucontext.h>

#include <algorithm>
#include <functional>
#include <memory>
#include <random>
#include <vector>

typedef unsigned long long u64;
typedef uint32_t u32;
using std::min;
#define __device__
#define __forceinline__ inline

namespace {
std::mt19937 rng;
int pick(int n) { return (int)(rng() % (u32)n); }
u32 seed_now;
#define CHECK(c, ...) \
    do { \
        if (!(c)) { printf("seed %u: ", seed_now); printf(__VA_ARGS__); printf("\n"); exit(1); } \
    } while (0)

enum Kind { NONE, BALLOT, DRAIN, TICKS };
struct Lane {
    ucontext_t context;
    std::unique_ptr<char[]> stack;
    int wave, lane;
    bool done = false, vote = false;
    Kind waits = NONE;
    u64 result = 0;
    std::vector<std::pair<u64 *, u64>> late;  // stores on their way
};
struct Wave {
    std::function<void(int)> body;
    u32 xcd;
    int first, lanes, start;  // not before that many steps
};
std::vector<Lane> lanes;
std::vector<Wave> waves;
ucontext_t scheduler;
Lane *now;
u32 clock_ticks;

void yield() { swapcontext(&now->context, &scheduler); }
u64 together(Kind kind, bool vote) {  // the lanes of a wave wait for each other
    now->waits = kind;
    now->vote = vote;
    yield();
    return now->result;
}
void arrive(Lane &l, u64 *p) {
    for (auto &s : l.late)
        if (!p || s.first == p) *s.first = s.second;
    l.late.erase(std::remove_if(l.late.begin(), l.late.end(), [&](auto &s) { return !p || s.first == p; }), l.late.end());
}
}  // namespace

namespace dt {
void put_agent(u64 *p, u64 v) {
    yield();
    for (auto &s : now->late)
        if (s.first == p) { s.second = v; return; }
    now->late.push_back({p, v});
}
u64 get_agent(u64 *p) {
    yield();
    for (auto &s : now->late)
        if (s.first == p) return s.second;
    return *p;
}
u64 swap_agent(u64 *p, u64 v) {
    yield();
    arrive(*now, p);
    return std::exchange(*p, v);
}
void put_local(u64 *p, u64 v) {
    yield();
    *p = v;
}
u64 swap_local(u64 *p, u64 from, u64 to) {
    yield();
    const u64 was = *p;
    if (was == from) *p = to;
    return was;
}
void drain() {
    arrive(*now, nullptr);
    together(DRAIN, false);
}
u64 ballot(bool b) { return together(BALLOT, b); }
u32 ticks() { return (u32)together(TICKS, false); }
u32 xcc_id() { return waves[now->wave].xcd; }
}  // namespace dt
#include "../paper_2601_12212_amd/csrc/hands.hpp"
using namespace dt;

namespace {
void entry() {
    waves[now->wave].body(now->lane);
    arrive(*now, nullptr);
    now->done = true;
    yield();
}
// A launch of what `waves` holds.
void run(int lanes_of_a_wave) {
    lanes.clear();
    lanes.resize(waves.size() * lanes_of_a_wave);
    for (size_t w = 0; w < waves.size(); ++w) {
        waves[w].first = (int)w * lanes_of_a_wave;
        waves[w].lanes = lanes_of_a_wave;
        waves[w].start = pick(3) ? 0 : pick(4000);
        for (int i = 0; i < lanes_of_a_wave; ++i) {
            Lane &l = lanes[waves[w].first + i];
            l.wave = (int)w;
            l.lane = i;
            l.stack.reset(new char[32768]);
            getcontext(&l.context);
            l.context.uc_stack.ss_sp = l.stack.get();
            l.context.uc_stack.ss_size = 32768;
            l.context.uc_link = nullptr;
            makecontext(&l.context, entry, 0);
        }
    }
    int left = (int)waves.size();
    for (int step = 0; left; ++step) {
        CHECK(step < 4000000, "a wait without an end");
        Wave &w = waves[pick((int)waves.size())];
        if (step < w.start) continue;
        // the wave's next lane that can run; all of them waiting for each other: on
        const int at = pick(w.lanes);
        Lane *next = nullptr;
        int waiting = 0, ended = 0;
        for (int i = 0; i < w.lanes; ++i) {
            Lane &l = lanes[w.first + (at + i) % w.lanes];
            ended += l.done;
            waiting += l.waits != NONE;
            if (!next && !l.done && l.waits == NONE) next = &l;
        }
        if (ended == w.lanes) continue;
        if (next) {
            if (!next->late.empty() && !pick(4)) arrive(*next, next->late[pick((int)next->late.size())].first);
            now = next;
            swapcontext(&scheduler, &now->context);
            if (next->done) {
                bool all = true;
                for (int i = 0; i < w.lanes; ++i) all = all && lanes[w.first + i].done;
                left -= all;
            }
            continue;
        }
        CHECK(waiting == w.lanes, "lanes of a wave part");
        u64 bits = 0;
        const Kind kind = lanes[w.first].waits;
        for (int i = 0; i < 64; ++i) bits |= (u64)lanes[w.first + min(i, w.lanes - 1)].vote << i;  // lanes past the last do as that one
        if (kind == TICKS) clock_ticks += pick(8) ? 1 : pick(2) ? 600 : 4000;
        for (int i = 0; i < w.lanes; ++i) {
            Lane &l = lanes[w.first + i];
            CHECK(l.waits == kind, "lanes of a wave part");
            l.waits = NONE;
            l.result = kind == BALLOT ? bits : clock_ticks;
        }
    }
}

const u64 TAG = 0x9e3779b97f4a0000ull;
struct Data {
    int local = 0, memory = 0;  // the launch whose result lies in the writer's L2, at the memory side
    u32 xcd = 0;
};
struct Row {
    std::vector<u64> offers, marks;
    u64 claim;
    std::vector<Data> data;
    int result = 0, taken = 0;
};

void launches(int rows, int members, bool level, bool apart, int n_launches, bool overlap = false) {
    const u64 litter = pick(3) == 0 ? 0 : pick(2) ? 0xEEEEEEEEEEEEEEEEull : TAG + (5ull << 20) + 1;
    std::vector<Row> row(rows);
    for (Row &r : row) {
        r.offers.assign(members, litter);
        r.marks.assign(members + 1, litter);
        r.claim = litter;
        r.data.resize(members + 1);
    }
    std::vector<u64> words(MARK_WORDS, litter);
    const Marks marks = {words.data(), TAG, (1ull << rows) - 1ull};
    int version = 0, expanded = 0;
    auto expand = [&](int lane) {
        if (lane < rows) CHECK(overlap || row[lane].result == version, "a level from another launch's row");
        if (lane == 0) ++expanded;
        drain();
        mark_clear(marks, lane);
    };
    auto take = [&](int r, const Hands<1> &h, int me, int lane, bool taking) {
        Row &of = row[r];
        yield();
        if (lane <= members && lane != me) {
            const Data &d = of.data[lane];
            CHECK(overlap || (d.xcd == xcc_id() ? std::max(d.local, d.memory) : d.memory) == version, "a result of another launch");
        }
        const u64 was = hand_take(h, lane, taking);
        hand_settle(h, lane, taking, was);
        if (lane == 0) {
            ++of.taken;
            of.result = version;
        }
        if (!level) return;
        drain();
        if (mark_done(marks, r, lane)) expand(lane);
    };
    for (version = 1; version <= n_launches; ++version) {
        waves.clear();
        expanded = 0;
        for (int r = 0; r < rows; ++r) {
            Row &of = row[r];
            of.taken = 0;
            const u32 home = (u32)pick(8);
            for (int m = 0; m <= members; ++m) {
                of.data[m].xcd = pick(6) ? home : (u32)pick(8);
                waves.push_back({[&, r, m](int lane) {
                                     Row &mine = row[r];
                                     const Hands<1> h = {mine.offers.data(), mine.marks.data(), &mine.claim, TAG, members};
                                     bool taking = false;
                                     if (m < members) {
                                         mine.data[m].local = version;
                                         drain();
                                         if (!apart && hand_offer(h, m, lane)) return;
                                         mine.data[m].memory = version;
                                         drain();
                                         if (!hand_mark(h, m, lane)) return;
                                     } else if (!hand_await(h, lane, taking)) {
                                         mine.data[m].memory = version;
                                         drain();
                                         if (!hand_leave(h, lane)) return;
                                     }
                                     take(r, h, m, lane, taking);
                                 },
                                 of.data[m].xcd, 0, 0, 0});
            }
        }
        if (level) waves.push_back({[&](int lane) { if (mark_await(marks, lane)) expand(lane); }, (u32)pick(8), 0, 0, 0});
        if (overlap)  // a launch that writes to the same memory meanwhile
            waves.push_back({[&](int lane) {
                                 for (int i = 0; lane == 0 && i < 40; ++i) {
                                     Row &r = row[pick(rows)];
                                     u64 *const words[] = {&r.offers[pick(members)], &r.marks[pick(members + 1)], &r.claim};
                                     const u64 values[] = {0, litter, (TAG + (7ull << 20)) | (u64)pick(17), ~TAG};
                                     put_local(words[pick(3)], values[pick(4)]);
                                     for (int n = pick(40); n; --n) yield();
                                 }
                             },
                             0, 0, 0, 0});
        run(level ? MARK_CLAIM : members + 2);
        if (overlap) continue;  // what such launches leave is not defined, but they end
        for (const Row &r : row) {
            CHECK(r.taken == 1, "launch %d: a row taken %d times", version, r.taken);
            for (u64 o : r.offers) CHECK(apart || o == 0, "launch %d: an offer %llx is left", version, o);
            for (u64 m : r.marks) CHECK((m & ~0xffffull) != TAG, "launch %d: a mark %llx is left", version, m);
        }
        if (level) {
            CHECK(expanded == 1, "launch %d: a level chosen %d times", version, expanded);
            for (int i = 0; i <= MARK_GONE; ++i) CHECK(words[i] != TAG, "launch %d: word %d of the level is left", version, i);
        }
    }
}
}  // namespace

int main(int argc, char **argv) {
    if (argc != 3) return 2;
    for (seed_now = 1; (int)seed_now <= atoi(argv[2]); ++seed_now) {
        rng.seed(seed_now);
        clock_ticks = rng();
        if (!strcmp(argv[1], "rows")) launches(1, 1 + pick(4), false, false, 8);
        else if (!strcmp(argv[1], "apart")) launches(1, 1 + pick(4), false, true, 8);
        else if (!strcmp(argv[1], "levels")) launches(1 + pick(2), 1 + pick(2), true, false, 6);
        else if (!strcmp(argv[1], "overlap")) launches(1 + pick(2), 1 + pick(3), pick(2), false, 4, true);
        else return 2;
    }
    printf("ok\n");
    return 0;
}
