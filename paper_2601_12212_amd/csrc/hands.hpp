// Words by which the workgroups of a launch hand each other results.  The including file has the operations on memory (common.hpp; tests/hand_overs.cpp tries
// every order of them on the host):
//   put_agent, get_agent, swap_agent  at the memory side
//   put_local, swap_local             in the XCD's L2; swap_local(p, from, to) exchanges *p if it is `from` and returns what it was
//   drain                             what the wave has written so is there
//   ballot, xcc_id, ticks (of 10 ns)
#pragma once

namespace dt {

#define LINE_WORDS 16  // of 64 bits in a cache line
// How long, in ticks, a workgroup that began to wait at t0 stays for the others of its launch, and how long it offers them what it has in its XCD's L2.
// SHORT_WAITS: a second build, for tests, whose waits end after 0 to 1.2 us, by the clock, so that every way out of them is taken.
#ifdef SHORT_WAITS
#define STAY_TICKS(t0) (((t0) >> 2 & 3) * 40)
#define OFFER_TICKS(t0) (((t0) & 3) * 40)
#else
#define STAY_TICKS(t0) 5000
#define OFFER_TICKS(t0) 1000
#endif

// n members that hand what they have to one more, which waits for them; one wave of each speaks for it.
//
// What they have goes in one of two ways.  On the waiting one's XCD it is left in that L2 and offered by a word, with the XCD's number in it, which the waiting
// one exchanges for 0 when it takes what is there.  An offer that nobody has taken for OFFER_TICKS is withdrawn the same way; then all of it is written
// to the memory side and marked there, for a reader anywhere.  Nothing depends on which workgroups run at once or where: if the waiting one has
// waited for STAY_TICKS and taken nothing, it leaves a mark as well and goes; the offers run out, and of those that mark what they have the last to come
// sees all marks and does its work.  Of the last two both may: the first to claim it does, alone (of a row that two had taken the second mark for
// its level could come behind the level's choice, and stay).
//
// No wait is for anything but a limited time.  Offers end as 0, and marks are taken away by who has seen them all: a replayed graph has the same
// tag.  The claim is not: another may be on the way to it.  It is cleared by the waiting one before its own mark, without which nobody claims.
template <int STRIDE>
struct Hands {
    u64 *offers;  // of member m at m * STRIDE: `tag` and an XCD's number while something is on offer in its L2
    u64 *marks;   // [n + 1]: `tag` once it is at the memory side; the last one's, once it has gone
    u64 *claim;
    u64 tag;      // of this launch, the low 16 bits free: what the memory held before it never looks like an offer or a mark
    int n;        // up to 63
};
#define HAND_HAD 0x100  // with the tag, in the place of a member's mark: the waiting one has what it is about to mark; of the claim: made
// What is offered has reached the L2.  True if it has been taken.
template <int STRIDE>
__device__ __forceinline__ bool hand_offer(const Hands<STRIDE> &h, int me, int lane) {
    const u64 here = h.tag | (xcc_id() + 1);
    u64 *const own = h.offers + me * STRIDE;
    if (lane == 0) put_local(own, here);
    drain();
    const u32 t0 = ticks();
    while (ballot(lane == 0 && get_agent(own) == here)) {
        if (ticks() - t0 > OFFER_TICKS(t0)) break;
    }
    u64 was = here;
    if (lane == 0) was = swap_local(own, here, 0);
    return ballot(lane == 0 && was == 0) != 0ull;  // (anything else is not this launch's: as if nobody had taken it)
}
__device__ __forceinline__ bool hand_claim(u64 *claim, u64 tag, int lane) {
    u64 was = 0;
    if (lane == 0) was = swap_agent(claim, tag | HAND_HAD);
    return ballot(was == (tag | HAND_HAD)) == 0ull;
}
// What is marked has reached the memory side.  True for one, if all are there, the waiting one's mark among them.
template <int STRIDE>
__device__ __forceinline__ bool hand_mark(const Hands<STRIDE> &h, int me, int lane) {
    u64 was = 0;
    if (lane == 0) was = swap_agent(h.marks + me, h.tag);
    drain();
    if (ballot(was == (h.tag | HAND_HAD))) {
        if (lane == 0) put_agent(h.marks + me, 0);
        return false;
    }
    return ballot(get_agent(h.marks + min(lane, h.n)) != h.tag) == 0ull && hand_claim(h.claim, h.tag, lane);
}
// The waiting one: true if all are there, with `taking` in the lanes of offers that hand_take is to take.  False if it has waited for long enough.
template <int STRIDE>
__device__ __forceinline__ bool hand_await(const Hands<STRIDE> &h, int lane, bool &taking) {
    const u64 here = h.tag | (xcc_id() + 1);
    const int peer = min(lane, h.n - 1);
    const u32 t0 = ticks();
    for (;;) {
        const bool offered = get_agent(h.offers + peer * STRIDE) == here, marked = get_agent(h.marks + peer) == h.tag;
        taking = offered && !marked && lane < h.n;
        if (ballot(offered || marked) == ~0ull) return true;
        if (ticks() - t0 > STAY_TICKS(t0)) {
            taking = false;
            return false;
        }
    }
}
// The waiting one goes; what it has itself has reached the memory side.  As hand_mark.
template <int STRIDE>
__device__ __forceinline__ bool hand_leave(const Hands<STRIDE> &h, int lane) {
    if (lane == 0) put_agent(h.claim, 0);
    drain();
    return hand_mark(h, h.n, lane);
}
// What the offers were that were to be taken, once what was on offer has been asked for.
template <int STRIDE>
__device__ __forceinline__ u64 hand_take(const Hands<STRIDE> &h, int lane, bool taking) {
    const u64 here = h.tag | (xcc_id() + 1);
    return taking ? swap_local(h.offers + min(lane, h.n - 1) * STRIDE, here, 0) : here;
}
// Whoever has all.  Who withdrew its offer a moment ago is on the way to its mark, with what it had offered: it finds there that it is not needed any more, and
// takes that away.  (Nobody waits for the other: where two launches overlap on one memory, against the rules, it may never come.)
template <int STRIDE>
__device__ __forceinline__ void hand_settle(const Hands<STRIDE> &h, int lane, bool taking, u64 was) {
    const bool late = taking && was != (h.tag | (xcc_id() + 1));
    u64 mark = h.tag;
    if (late) mark = swap_agent(h.marks + min(lane, h.n), h.tag | HAND_HAD);
    if (lane <= h.n && (!taking || (late && mark == h.tag))) put_agent(h.marks + lane, 0);
}

// Marks alone: who waits for others' results at the memory side and has nothing of its own there.  One word to each of them, one of the waiting one if it
// has waited for STAY_TICKS and goes, in whose place the last of the others to come then does its work, and a claim, as above.  All but the claim are 0 again
// at the end (mark_clear).
#define MARK_GONE 32  // most of them
#define MARK_CLAIM 33
#define MARK_WORDS 40
struct Marks {
    u64 *words;  // [MARK_WORDS]
    u64 tag;
    u64 all;     // bits of the words that are waited for
};
__device__ __forceinline__ u64 marks_there(const Marks &m, int lane) { return ballot(get_agent(m.words + min(lane, MARK_GONE)) == m.tag); }
// One whose results have reached the memory side; true: the work is this one's to do.
__device__ __forceinline__ bool mark_done(const Marks &m, int me, int lane) {
    if (lane == 0) put_agent(m.words + me, m.tag);
    drain();
    const u64 all = m.all | 1ull << MARK_GONE;
    return (marks_there(m, lane) & all) == all && hand_claim(m.words + MARK_CLAIM, m.tag, lane);
}
// The waiting one; true: as above.
__device__ __forceinline__ bool mark_await(const Marks &m, int lane) {
    const u32 t0 = ticks();
    while ((marks_there(m, lane) & m.all) != m.all) {
        if (ticks() - t0 > STAY_TICKS(t0)) {
            if (lane == 0) put_agent(m.words + MARK_CLAIM, 0);
            drain();
            return mark_done(m, MARK_GONE, lane);
        }
    }
    return true;
}
__device__ __forceinline__ void mark_clear(const Marks &m, int lane) {
    if (lane <= MARK_GONE) put_agent(m.words + lane, 0);
}

}  // namespace dt
