// The choice of a level's nodes: what the tree kernel and the workgroups that expand a level beside its rows have in common.
#pragma once
#include "common.hpp"
#include "kernels.hpp"

namespace dt {

// order-preserving integer image of a score (ord32; adding zero folds -0 onto +0)
__device__ __forceinline__ u32 score_key(float s) {
    const u32 u = __float_as_uint(s + 0.0f);
    return u ^ ((u32)((int)u >> 31) | 0x80000000u);
}
#define NARROW_K 16               // levels of at most NARROW_K^2 candidates: one wave
#define KEY_NEG_INF 0x007FFFFFu   // key of -inf: a candidate that does not exist

// x / dv for 0 <= x < 8192 and 1 <= dv <= 1024 with inv = 1.0f / dv (any rounding within two ulp):
// (x + 0.5) / dv is at least 0.5 / dv away from every integer, far more than the product's error.
__device__ __forceinline__ int fdiv(int x, float inv) { return (int)(((float)x + 0.5f) * inv); }

struct Decoded {
    int level, slot, rank, row;
};
struct PoolShape {
    int k, kk;
    float inv_k, inv_kk;
};
__device__ __forceinline__ PoolShape pool_shape(int k) {
    PoolShape s;
    s.k = k; s.kk = k * k;
    s.inv_k = 1.0f / (float)k; s.inv_kk = 1.0f / (float)(k * k);
    return s;
}
// pool index -> (level, slot of the parent in its level's expanded set, rank in the parent's row, draft row)
__device__ __forceinline__ Decoded decode(int p, const PoolShape &s) {
    Decoded d;
    if (p < s.k) {
        d.level = 1; d.slot = 0; d.rank = p; d.row = 0;
    } else {
        const int q = p - s.k;
        const int l2 = fdiv(q, s.inv_kk), rem = q - l2 * s.kk;
        d.level = l2 + 2; d.slot = fdiv(rem, s.inv_k); d.rank = rem - d.slot * s.k;
        d.row = 1 + l2 * s.k + d.slot;
    }
    return d;
}

// An expanded node: score, pool index, and the slots of its ancestors and itself, five bits per level.
struct __attribute__((aligned(16))) Parent {
    float score;
    int index;
    u64 path;
};

// How many nodes the levels have expanded, the state's word of a sequence: that of the last call in the half of its level's parity, the level times 64 and the
// nodes, and in the other half the one before's.  What a level finds about the level before it (-1: nothing, which is so where a level is asked for again after later
// ones) is the same before and after its own note: the rows of a launch may look while the level is chosen in that launch.
__device__ __forceinline__ int level_count(u32 word, int level) {
    const u32 half = word >> (level & 1 ? 16 : 0) & 0xFFFFu;
    return (int)(half >> 6) == level ? (int)(half & 63u) : -1;
}
__device__ __forceinline__ int level_note(u32 before, int level, int n) {
    const u32 other = level & 1 ? before & 0xFFFFu : before >> 16, kept = (int)(other >> 6) > level ? 0u : other;
    const u32 own = (u32)(level << 6 | n);
    return (int)(level & 1 ? own << 16 | kept : kept << 16 | own);
}

// What the expansion of level l hands on to that of level l + 1 when the tree is built level by level: the nodes it chose, how many, the
// token count, and which level it was.  It lies in the last rows of the sequence's state, which belong to the deepest level's pass and are
// free until then.  Without it, or with another level's (a level asked for again), the levels before are gone through again, from the
// row results.  (How many, in the same word as the level: the state's own word may have been a later level's since.)  Each level gone through again took 0.5 us with k up to 16 and 1.7 beyond.  All calls of a step, replayed: (60, 6, 10), 128,256 tokens
// 78.2 -> 74.7 us (with the kernels of their own); 16 sequences of up to (123, 8, 23), 1,152 tokens 125.6 -> 101.7; 4 of (66, 3, 8) 32.0 -> 31.7.
// Up to k = NARROW_K there is room for every level's, and the tree is finished from them where all are there: the candidates scored side by side in
// place of a chain of levels.  A level that is chosen takes away what later ones have left.  (All calls, replayed, the chain | so: (60, 6, 10) 68.4 | 67.1 us, (96, 8, 12)
// 90.0 | 85.9, 16 sequences of (60, 6, 16) 77.1 | 73.5.)
#define CARRY_ROW (DT_STATE_ROWS - 4)  // four rows of values: DT_K_MAX Parents; two words of the ids
#define CARRY_FROM 2  // level 1 expands the root's children: nothing to go through
#define CARRY_LEVELS ((CARRY_ROW - 1) / DT_K_MAX)  // levels whose nodes' rows, at most l DT_K_MAX, end before it
static_assert(1 + (DT_D_MAX - 1) * NARROW_K <= CARRY_ROW - 4 * (DT_D_MAX - 1), "rows of narrow levels end before all of these");
static_assert(4 * DT_K_MAX * sizeof(float) == DT_K_MAX * sizeof(Parent), "four rows");
#define CARRY_COUNT 0x3F0  // where the tag holds the number of nodes
__device__ __forceinline__ int carry_tag(int level, int n_exp, int early_stop) { return 0x7A5C3000 | (early_stop ? 0x400 : 0) | n_exp << 4 | level; }
static_assert(DT_D_MAX < 16 && DT_K_MAX <= CARRY_COUNT >> 4, "the tag's fields");
__device__ __forceinline__ int64_t carry_at(int64_t seq_rows, int b, int level, bool narrow) { return (b * seq_rows + CARRY_ROW - (narrow ? 4 * level : 0)) * DT_K_MAX; }
__device__ __forceinline__ bool carries(int level, bool narrow) { return narrow ? level >= 1 : level >= CARRY_FROM && level <= CARRY_LEVELS; }
// The level to start from, its nodes and the token count: level 0, nothing.
struct Start {
    int level, n_exp, tok_count;
};

// ---- selection inside a wave ---------------------------------------------------------------------------
// The `keep` best of the keys that a wave holds (key q of lane i is candidate i + 64 q), equal keys by ascending candidate;
// all viable ones if they are fewer.  The caller knows bounds: lo is KEY_NEG_INF or lies below at
// least `keep` keys, no key lies above hi.  Returns how many were chosen (uniform).
template <int G>
__device__ __forceinline__ int wave_select(const u32 (&key)[G], int keep, u32 lo, u32 hi, bool (&chosen)[G]) {
    int c = count_above<G>(key, lo), equal = 0;  // equal > 0: that many of the keys equal to lo are chosen too
    if (c > keep) {
        // more than `keep` above lo, fewer above hi = lo + width
        u32 width = hi - lo;
        for (int step = 0; step < (G < 4 ? 7 : 10); ++step) {
            const u32 half = width >> 1, mid = lo + half;
            c = count_above<G>(key, mid);
            width -= half;
            lo = c >= keep ? mid : lo;
            if (c == keep) break;
        }
        hi = lo + width;
        // Candidates close together, or equal: from here on a candidate of those in (lo, hi] divides them.
        while (c != keep) {
            u32 any = 0u;
#pragma unroll
            for (int q = 0; q < G; ++q) any = key[q] > lo && key[q] <= hi ? key[q] : any;
            const u32 pivot = (u32)__builtin_amdgcn_readlane((int)any, __builtin_ctzll(__builtin_amdgcn_ballot_w64(any != 0u)));
            c = count_above<G>(key, pivot - 1u);
            if (c < keep) hi = pivot - 1u;
            else if (c == keep) lo = pivot - 1u;
            else {
                lo = pivot;
                c = count_above<G>(key, pivot);
                if (c < keep) { equal = keep - c; c = keep; }
            }
        }
    }
#pragma unroll
    for (int q = 0; q < G; ++q) chosen[q] = key[q] > lo;
    if (equal) {
#pragma unroll
        for (int q = 0; q < G; ++q) {
            const u64 eq = __builtin_amdgcn_ballot_w64(key[q] == lo);
            chosen[q] = chosen[q] || (key[q] == lo && (int)lanes_below(eq) < equal);
            equal -= min(equal, (int)__popcll(eq));
        }
    }
    return c;
}

// Bounds of a level's cut: the best children of k nodes (lane s < k: key `fk` of slot s's, rows descend) are k candidates, so
// at least k lie above `lo`; none lies above `hi`.
__device__ __forceinline__ void level_bounds(u32 fk, int k, u32 &lo, u32 &hi) {
    const bool viable = lane_id() < k && fk > KEY_NEG_INF;
    u32 x = viable ? fk : 0u, y = viable ? ~fk : 0u;  // the maxima over lanes 0 .. 31 end in lane 31
#define STEP(CTRL, ROWS)                                          \
    x = max(x, (u32)dpp_mov<CTRL, ROWS>(0, (int)x));              \
    y = max(y, (u32)dpp_mov<CTRL, ROWS>(0, (int)y));
    STEP(0x111, 0xf) STEP(0x112, 0xf) STEP(0x114, 0xf) STEP(0x118, 0xf) STEP(0x142, 0xa)
#undef STEP
    hi = (u32)__builtin_amdgcn_readlane((int)x, 31);
    lo = __popcll(__builtin_amdgcn_ballot_w64(viable)) == k ? ~(u32)__builtin_amdgcn_readlane((int)y, 31) - 1u : KEY_NEG_INF;
}
// The head of what level l hands on, by one thread.
__device__ __forceinline__ void carry_head(const TreeArgs &a, int b, int l, int k, int n_exp, int tok_count) {
    const bool narrow = k <= NARROW_K;
    if (carries(l, narrow)) *(int2 *)(a.state_id + carry_at(a.seq_rows, b, l, narrow)) = make_int2(carry_tag(l, n_exp, a.early_stop), tok_count);
    if (narrow)
        for (int j = l + 1; j < DT_D_MAX; ++j) a.state_id[carry_at(a.seq_rows, b, j, true)] = 0;
}
// What the draft model is handed for its next pass, by one wave: node s of the set chosen at level l, node(s, token).
template <typename F>
__device__ __forceinline__ void emit_level(const TreeArgs &a, int b, int l, int k, int n_exp, int tok_count, u32 before, int prefix, F node) {
    const int lane = lane_id();
    const bool carry = carries(l, k <= NARROW_K);
    const int64_t at = carry_at(a.seq_rows, b, l, k <= NARROW_K);
    if (lane < n_exp) {
        int token;
        const Parent pr = node(lane, token);
        if (carry) ((Parent *)(a.state_val + at))[lane] = pr;
        const Decoded dc = decode(pr.index, pool_shape(k));
        const int64_t e = (int64_t)b * DT_K_MAX + lane;
        a.exp_token[e] = token;
        a.exp_parent_slot[e] = l == 1 ? -1 : dc.slot;
        a.exp_row[e] = 1 + (l - 1) * k + lane;
        a.exp_pos[e] = max(prefix, 0) + l;
        // draft-side mask over draft rows: the root's row, the rows of the ancestors, its own
        u64 w0 = 1ull, w1 = 0ull, w2 = 0ull, w3 = 0ull;
        for (int j = 1; j <= l; ++j) {
            const int r = 1 + (j - 1) * k + (int)((pr.path >> (5 * (j - 1))) & 31);
            const u64 bit = 1ull << (r & 63);
            const int wd = r >> 6;
            w0 |= wd == 0 ? bit : 0ull; w1 |= wd == 1 ? bit : 0ull;
            w2 |= wd == 2 ? bit : 0ull; w3 |= wd == 3 ? bit : 0ull;
        }
        a.exp_mask[e * 4] = w0; a.exp_mask[e * 4 + 1] = w1;
        a.exp_mask[e * 4 + 2] = w2; a.exp_mask[e * 4 + 3] = w3;
    }
    if (lane == 0) {
        a.n_expand[b] = n_exp;
        a.state_n_exp[b] = level_note(before, l, n_exp);
        carry_head(a, b, l, k, n_exp, tok_count);
    }
}

// Nothing is expanded at level l, by one thread.
__device__ __forceinline__ void emit_nothing(const TreeArgs &a, int b, int l, u32 before) {
    a.n_expand[b] = 0;
    a.state_n_exp[b] = level_note(before, l, 0);
}

// ---- a level chosen in the launch that reduces its rows ----------------------------------------------------
// A workgroup to a sequence waits for the workgroups of the sequence's rows and chooses the level's nodes, one wave with a candidate to a lane, or four (k up to
// NARROW_K; with two up to k = 11 as well, (96, 8, 12) took 92.3 us, 90.9 so), nothing of the earlier levels but what the last one has handed on.  A kernel of its own behind the rows' is a launch more, and reads its parameters, what
// was handed on and the rows one after the other where this has the first two before the rows are done.  All calls of a step, called | replayed, with the kernel
// of its own -> so: one sequence of (60, 6, 10) and 128,256 tokens 70 to 78 | 71.4 -> 66.7 | 68.8 us, 1,000 tokens 69 to 76 | 58.0 -> 55 | 52.3; (64, 7, 8), 8,192 80 to 89 |
// 65.2 -> 63 | 58.9; 16 of (60, 6, 16), 4,001 69 to 78 | 67.8 -> 62 | 64.5.
//
// The words of a sequence (Marks): one for each row that is reduced and one for its log-sum-exp where a workgroup of its own makes that, at the memory
// side like the results.  Who does the waiting one's work has claimed it: what is handed on must not be read by one while another writes it.
static_assert(2 * NARROW_K <= MARK_GONE, "a row's and its log-sum-exp's");
struct LevelTail {
    TreeArgs t;
    u64 *words;     // [batch, MARK_WORDS]
    u64 tag;
    int first_wg;   // of the workgroups that wait
    int rows;       // rows of a sequence in the launch
    int lse_apart;
};
struct LevelLds {
    Parent par[2][DT_K_MAX + 1];  // of the level's parity
    int tok[DT_K_MAX];
};
// Of a sequence: its limits, what the state has, and the row of its root.
struct LevelIn {
    int TT, d, k, rows, tok_count, n_exp, prefix;  // rows: of the launch, that are reduced
    u32 word;
    bool carried;
    uint4 node;
    float root_val, root_lse;
    int root_id;
};
template <typename T>
__device__ __forceinline__ T get32_agent(const T *p) {
    static_assert(sizeof(T) == 4, "a word");
    return __builtin_bit_cast(T, __hip_atomic_load((const u32 *)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}
template <typename T>
__device__ __forceinline__ void put32_agent(T *p, T v) {
    static_assert(sizeof(T) == 4, "a word");
    __hip_atomic_store((u32 *)p, __builtin_bit_cast(u32, v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// The marks of a sequence's level, `rows` of its rows being reduced.
__device__ __forceinline__ Marks level_marks(const LevelTail &h, int b, int rows) {
    const u64 m = (1ull << rows) - 1ull;
    return {h.words + (int64_t)b * MARK_WORDS, h.tag, h.lse_apart ? m | m << NARROW_K : m};
}
__device__ __forceinline__ LevelIn level_in(const TreeArgs &a, int rows, int b, int lane) {
    LevelIn in;
    const int xl = a.expand_level;
    const int64_t at = carry_at(a.seq_rows, b, max(xl - 1, 1), true), r0 = (int64_t)b * a.seq_rows;
    const dt_params prm = a.params[b];
    in.word = (u32)a.state_n_exp[b];
    in.prefix = a.prefix_len ? a.prefix_len[b] : 0;
    in.root_val = a.top_val[r0 * DT_K_MAX + (lane & (DT_K_MAX - 1))];  // (of level 1 not there yet)
    in.root_id = 0;
    in.root_lse = a.lse[r0];
    in.node = ((const uint4 *)(a.top_val + at))[lane & (DT_K_MAX - 1)];
    const int2 head = *(const int2 *)(a.top_id + at);
    in.TT = min(max(prm.TT, 1), a.TT_cap);
    in.d = min(max(prm.d, 1), DT_D_MAX);
    in.k = min(max(prm.k, 1), min(DT_K_MAX, a.V));
    const int last = level_count(in.word, xl - 1);
    in.rows = min(xl == 1 ? 1 : last >= 0 ? min(last, in.k) : in.k, rows);
    in.carried = xl > 1 && (head.x & ~CARRY_COUNT) == carry_tag(xl - 1, 0, a.early_stop);
    in.n_exp = min((head.x & CARRY_COUNT) >> 4, in.k);
    in.tok_count = head.y;
    return in;
}
// From the nodes of level l to those of level l + 1; none if there are none, or if the token count ends the expansion.
template <int G>
__device__ __forceinline__ int level_next(const TreeArgs &a, LevelLds &L, int b, int l, int k, int TT, int n_exp, int &tok_count) {
    const int lane = lane_id(), kk = k * k;
    const float inv_k = 1.0f / (float)k;
    const int64_t row0 = (int64_t)b * a.seq_rows + 1 + (l - 1) * k;
    Parent *const from = L.par[l & 1], *const to = L.par[(l + 1) & 1];
    const int64_t best_row = row0 + min(lane, k - 1);
    const float best_val = get32_agent(a.top_val + best_row * DT_K_MAX), best_lse = get32_agent(a.lse + best_row);
    int parent[G], tok[G];
    float val[G], lse[G];
#pragma unroll
    for (int q = 0; q < G; ++q) {
        const int c = min(lane + 64 * q, kk - 1), slot = fdiv(c, inv_k);
        const int64_t row = row0 + slot, at = row * DT_K_MAX + c - slot * k;
        val[q] = get32_agent(a.top_val + at);
        lse[q] = get32_agent(a.lse + row);
        tok[q] = get32_agent(a.top_id + at);
        parent[q] = lane + 64 * q < kk ? slot : DT_K_MAX;  // no candidate: a parent that does not exist
    }
    if (lane >= n_exp && lane <= DT_K_MAX) from[lane].score = -INFINITY;
    auto own = [](float v, float row_lse) {
        const float lp = v - row_lse;
        return lp < INFINITY ? lp : -INFINITY;  // neither +inf nor a NaN, see tree_kernel
    };
    const float f = from[min(lane, DT_K_MAX)].score + own(best_val, best_lse);
    float sc[G];
    u32 key[G], lo, hi;
    bool chosen[G];
#pragma unroll
    for (int q = 0; q < G; ++q) {
        sc[q] = from[parent[q]].score + own(val[q], lse[q]);
        key[q] = score_key(sc[q]);
    }
    if (a.early_stop) {
#pragma unroll
        for (int q = 0; q < G; ++q) tok_count += __popcll(__builtin_amdgcn_ballot_w64(sc[q] > -INFINITY));
        if (tok_count >= TT) return 0;
    }
    level_bounds(score_key(f), k, lo, hi);
    const int n = wave_select<G>(key, k, lo, hi, chosen);
    int before = 0;
#pragma unroll
    for (int q = 0; q < G; ++q) {
        const u64 m = __builtin_amdgcn_ballot_w64(chosen[q]);
        const int pos = before + (int)lanes_below(m);
        if (chosen[q]) {
            const u64 path = from[fdiv(lane + 64 * q, inv_k)].path;  // (read with the score and held, registers that a workgroup of 1,024 has not)
            to[pos] = {sc[q], k + (l - 1) * kk + lane + 64 * q, path | (u64)pos << (5 * l)};
            L.tok[pos] = tok[q];
        }
        before += __popcll(m);
    }
    return n;
}
// The level, by one wave; its rows' results are at the memory side.
__device__ __forceinline__ void level_expand(const LevelTail &h, const Marks &marks, LevelLds &L, int b, LevelIn in, int lane) {
    const TreeArgs &a = h.t;
    const int xl = a.expand_level;
    // (rows_per_seq reaches every k: of more than NARROW_K nodes there is level 1 only)
    const int k = xl > 1 ? min(in.k, NARROW_K) : in.k;
    int l = xl - 1, n_exp = in.n_exp, tok_count = in.tok_count;
    if (in.carried) {
        if (lane < DT_K_MAX) *(uint4 *)&L.par[l & 1][lane] = in.node;
    } else {
        const int64_t r0 = (int64_t)b * a.seq_rows;
        if (xl == 1) {
            in.root_val = get32_agent(a.top_val + r0 * DT_K_MAX + (lane & (DT_K_MAX - 1)));
            in.root_id = get32_agent(a.top_id + r0 * DT_K_MAX + (lane & (DT_K_MAX - 1)));
            in.root_lse = get32_agent(a.lse + r0);
        }
        const float lp = in.root_val - in.root_lse, sc = lane < k && lp < INFINITY ? lp : -INFINITY;
        const u64 m = __builtin_amdgcn_ballot_w64(score_key(sc) > KEY_NEG_INF);  // every viable one is expanded
        tok_count = 1 + __popcll(m);
        l = 1;
        n_exp = a.early_stop && tok_count >= in.TT ? 0 : __popcll(m);
        if ((m >> lane) & 1ull) {
            const int pos = (int)lanes_below(m);
            L.par[1][pos] = {sc, lane, (u64)pos};
            L.tok[pos] = in.root_id;
        }
    }
    for (; n_exp > 0 && l < xl; ++l)
        n_exp = k <= 8 ? level_next<1>(a, L, b, l, k, in.TT, n_exp, tok_count) : level_next<NARROW_K * NARROW_K / 64>(a, L, b, l, k, in.TT, n_exp, tok_count);
    if (n_exp > 0) {
        emit_level(a, b, xl, k, n_exp, tok_count, in.word, in.prefix, [&](int s, int &token) {
            token = L.tok[s];
            return L.par[xl & 1][s];
        });
    } else if (lane == 0) {
        emit_nothing(a, b, xl, in.word);
        carry_head(a, b, xl, k, 0, tok_count);
    }
    drain();
    mark_clear(marks, lane);
}
// The waiting workgroup of sequence b, one wave.
__device__ __forceinline__ void level_wait_and_expand(const LevelTail &h, LevelLds &L, int b, int lane) {
    const LevelIn in = level_in(h.t, h.rows, b, lane);
    if (in.TT == 1 || h.t.expand_level >= in.d) {  // nothing is drafted below level d; the rows leave no marks
        if (lane == 0) emit_nothing(h.t, b, h.t.expand_level, in.word);
        return;
    }
    const Marks marks = level_marks(h, b, in.rows);
    if (mark_await(marks, lane)) level_expand(h, marks, L, b, in, lane);
}

}  // namespace dt
