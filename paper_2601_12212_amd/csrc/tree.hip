// Tree kernel: layer-wise expansion, rerank, and emission of the node arrays and the
// ancestor bitsets.  One workgroup of eight waves per sequence; the whole candidate pool (at most
// k + (d-1)k^2 = 7200 scores) lives in LDS.
//
// Selections ("the n best by (score desc, pool index asc)") never sort.  What bounds the kernel is a chain of dependent
// instructions, LDS trips and barriers (a lone wave issues one instruction in about eight cycles), not the work in it:
//  * Levels of up to 256 candidates (k <= 16) are expanded by one wave from start to end, without a barrier.  The worst of the
//    k parents' best children is a bound that at least k candidates reach; from there the wave bisects the
//    order-preserving integer image of the scores: a step counts the keys above a scalar by ballots, 5 steps on average.
//  * Larger levels are scored by all waves, which also collect what lies above that bound (2 to 7 k); one wave cuts the list.
//  * The rerank over the pool is cut by score buckets: one LDS histogram and one scan name the bucket that holds the
//    cut, the few candidates inside it rank themselves one against the other, everything in a better bucket is taken.
//    A pool of more than 1024 is thinned first, by a bound that enough of the threads' best candidates reach.
//  * A bucket, or a thinned list, that equal scores make too crowded goes through a radix selection over the integer image
//    (four 8-bit digits, one histogram and one barrier per digit, every wave scanning the 256 bins by itself).
// Eight waves that shared every level (pairs counted for k <= 11, score buckets beyond), two to five barriers per level, took
// 11.0 us for (TT, d, k) = (60, 6, 10), 10.9 for (64, 7, 8), 20 for (96, 8, 12) and 30 for the slowest of a batch with k up to
// 32; this takes 7.8, 7.8, 12.6 and 21.2 (averages of kernel traces; other machines 0.1 to 0.5 off).  What a lane, a thread or a list holds is sized in steps by k and by the pool, since each
// element more is instructions more in the chain (figures beside the steps: launches replayed one behind the other).
#include <stddef.h>

#include <type_traits>

#include "level.hpp"

namespace dt {

#define DT_P_MAX (DT_K_MAX + (DT_D_MAX - 1) * DT_K_MAX * DT_K_MAX)
#define TREE_NT 512               // threads of the workgroup
#define TREE_NW (TREE_NT / 64)    // its waves
#define LIST_CAP 1024             // most candidates that a thinning may leave
#define CAND_CAP 512              // most candidates of a wide level that its bound may leave
#define BUCKET_CAP 64             // most candidates of one score bucket that are ranked one against the other
#define SHARE_MAX 15              // most candidates per thread of a pool, an odd number

struct TreeLds {
    float score[DT_P_MAX];         // cumulative score of a candidate
    float lp[DT_P_MAX];            // its own log-probability (finite, or -inf: does not exist) and token, kept for the
    int tok[DT_P_MAX];             // emission: the kernel then ends without another trip to memory
    int16_t node[DT_P_MAX];        // node number after the rerank, -1: not kept
    int8_t slot[DT_P_MAX];         // slot in its level's expanded set, -1: not expanded
    Parent par[DT_D_MAX][DT_K_MAX + 1];  // slot s of level l; slots without a node, and the last entry: score -inf
    u32 hist[4][256];              // one histogram per radix digit
    u32 best[TREE_NT];             // best key of every thread's share of a large pool
    u64 mem[BUCKET_CAP];           // (key, index) of the candidates in the bucket that holds the cut
    Parent cand[CAND_CAP];         // candidates of a wide level above its bound, in pool order; `path`: their parents'
    float list_score[LIST_CAP];    // what a thinning leaves, in pool order
    int16_t list[LIST_CAP];
    int16_t sel[DT_TT_MAX];        // the kept candidates, in pool order
    int wtot[2 * TREE_NW];         // per-wave totals
    int p_end, n_exp, memn;
};

// ---- radix selection ---------------------------------------------------------------------------------
// Key of the keep-th best of score[0..n), keep = min(keep_max, #viable): returns keep (uniform), thr and
// need_eq = how many candidates with key == thr belong to the chosen set.  Whole workgroup; ends
// with every thread past the last barrier it contains.
__device__ __forceinline__ int block_radix_cut(const float *score, int n, int keep_max, TreeLds &S, u32 &thr,
                                               int &need_eq) {
    const int tid = threadIdx.x, lane = lane_id();
    for (int i = tid; i < 4 * 256; i += TREE_NT) (&S.hist[0][0])[i] = 0u;
    __syncthreads();
    u32 prefix = 0;
    int above = 0, keep = 0;
    thr = 0xFFFFFFFFu;
    need_eq = 0;
#pragma unroll 1
    for (int p = 0; p < 4; ++p) {
        const int shift = 24 - 8 * p;
        for (int i = tid; i < n; i += TREE_NT) {
            const u32 key = score_key(score[i]);
            const bool in = key > KEY_NEG_INF && (p == 0 || (key >> (shift + 8)) == (prefix >> (shift + 8)));
            if (in) atomicAdd(&S.hist[p][(key >> shift) & 255u], 1u);
        }
        __syncthreads();
        // every wave: lane L holds bins 4(63-L) .. 4(63-L)+3, so an ascending lane scan walks the bins downwards
        const uint4 h = *(const uint4 *)&S.hist[p][4 * (63 - lane)];
        const int c = (int)(h.x + h.y + h.z + h.w);
        const int incl = wave_scan_incl_i32(c);
        if (p == 0) {
            keep = min(keep_max, __builtin_amdgcn_readlane(incl, 63));
            if (keep <= 0) return 0;
        }
        const int need = keep - above;  // rank of the wanted key among those sharing the digits found so far
        const u64 m = __ballot(incl >= need);
        const int ls = __ffsll((long long)m) - 1;
        int acc = __builtin_amdgcn_readlane(incl - c, ls);
        const int h3 = __builtin_amdgcn_readlane((int)h.w, ls), h2 = __builtin_amdgcn_readlane((int)h.z, ls),
                  h1 = __builtin_amdgcn_readlane((int)h.y, ls);
        int dg;
        if (acc + h3 >= need) dg = 3;
        else {
            acc += h3;
            if (acc + h2 >= need) dg = 2;
            else {
                acc += h2;
                if (acc + h1 >= need) dg = 1;
                else { acc += h1; dg = 0; }
            }
        }
        above += acc;
        prefix |= (u32)(4 * (63 - ls) + dg) << shift;
        const int hd = dg == 3 ? h3 : dg == 2 ? h2 : dg == 1 ? h1 : __builtin_amdgcn_readlane((int)h.x, ls);
        if (keep - above == hd && p < 3 && prefix != 0u) {
            // every key that shares these digits belongs to the set: cut just below the smallest of them
            thr = prefix - 1u;
            need_eq = 0;
            return keep;
        }
    }
    thr = prefix;
    need_eq = keep - above;
    return keep;
}

// Positions in ascending index of the chosen candidates of score[0..n): those above thr and the first
// need_eq of those equal to it; f(index, position).  Returns how many were chosen (uniform).  Whole
// workgroup; one barrier inside, none after the calls of f.
template <typename F>
__device__ __forceinline__ int block_enumerate(const float *score, int n, u32 thr, int need_eq, TreeLds &S, F f) {
    const int tid = threadIdx.x, lane = lane_id(), w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int C = (n + TREE_NT - 1) / TREE_NT;  // consecutive candidates per thread
    const int i0 = tid * C;
    int own = 0;  // low half: keys above thr, high half: keys equal to thr
    for (int c = 0; c < C; ++c) {
        const int i = i0 + c;
        const u32 kv = score_key(score[min(i, n - 1)]);
        const u32 key = i < n ? kv : 0u;
        own += (key > thr ? 1 : 0) + (key == thr ? 0x10000 : 0);
    }
    const int incl = wave_scan_incl_i32(own);
    if (lane == 63) S.wtot[w] = incl;
    __syncthreads();
    int base = 0, total = 0;
#pragma unroll
    for (int v = 0; v < TREE_NW; ++v) {
        const int t = S.wtot[v];
        base += v < w ? t : 0;
        total += t;
    }
    int before = base + incl - own;
    for (int c = 0; c < C; ++c) {
        const int i = i0 + c;
        const u32 kv = score_key(score[min(i, n - 1)]);
        const u32 key = i < n ? kv : 0u;
        const int gt = before & 0xFFFF, eq = before >> 16;
        if (key > thr || (key == thr && eq < need_eq)) f(i, gt + min(eq, need_eq));
        before += (key > thr ? 1 : 0) + (key == thr ? 0x10000 : 0);
    }
    return (total & 0xFFFF) + min(total >> 16, need_eq);
}

// ---- expansion ---------------------------------------------------------------------------------------
__device__ __forceinline__ void put_parent(TreeLds &S, int l, int pos, float score, int index, u64 above) {
    Parent pr;
    pr.score = score;
    pr.index = index;
    pr.path = above | (u64)pos << (5 * (l - 1));
    S.par[l][pos] = pr;
    S.slot[index] = (int8_t)pos;
}
// Level 1, by one wave: every viable candidate is expanded.
__device__ __forceinline__ int choose_first(TreeLds &S, int k, float sc) {
    const int lane = lane_id();
    const u64 m = __builtin_amdgcn_ballot_w64(lane < k && score_key(sc) > KEY_NEG_INF);
    if ((m >> lane) & 1ull) put_parent(S, 1, (int)lanes_below(m), sc, lane, 0ull);
    return __popcll(m);
}
__device__ __forceinline__ Parent node_of(const TreeLds &S, int l, int slot, int &token) {
    const Parent pr = S.par[l][slot];
    token = S.tok[pr.index];
    return pr;
}

// All levels, by one wave: G candidates per lane, 64 G >= k^2.  Returns the end of the pool (levels computed so far), or -1
// when only level `xl` was wanted and has been written.  LDS is written and read by this wave alone, in order.
template <int G, bool EXPAND>
__device__ __forceinline__ int levels_narrow(const TreeArgs &a, TreeLds &S, int b, int k, int d, int TT, const Start &from, u32 word) {
    const int lane = lane_id(), xl = EXPAND ? a.expand_level : 0, kk = k * k;
    const int skip = from.level > 0 ? (from.level - 1) * kk : 0;  // candidates of the levels that are not gone through
    const PoolShape ps = pool_shape(k);
    int parent[G], at[G];  // of candidate lane + 64 q: its parent's slot, its pool index
    float own[G];          // of the next level: own log-probabilities, and of slot `lane`'s best child
    int best_at = k + skip + min(lane, k - 1) * k;
    float best_own = S.lp[best_at];
#pragma unroll
    for (int q = 0; q < G; ++q) {
        parent[q] = lane + 64 * q < kk ? fdiv(lane + 64 * q, ps.inv_k) : DT_K_MAX;
        at[q] = k + skip + min(lane + 64 * q, kk - 1);  // no candidate: the last one's place, and a parent that does not exist
        own[q] = S.lp[at[q]];
    }
    if (lane < DT_D_MAX) S.par[lane][DT_K_MAX].score = -INFINITY;
    const float sc1 = lane < k ? S.lp[lane] : -INFINITY;
    if (lane < k) S.score[lane] = sc1;
    // token count of Algorithm 2's expansion loop: the root plus the viable candidates proposed so far
    int tok_count = 1 + __popcll(__builtin_amdgcn_ballot_w64(sc1 > -INFINITY));
    const int l_end = xl > 0 ? xl + 1 : d;
    int l = 1, p_end = k, n_exp = 0;
    if (from.level > 0) {
        l = from.level;
        n_exp = from.n_exp;
        tok_count = from.tok_count;
    } else if (l < l_end && !(a.early_stop && tok_count >= TT)) {
        n_exp = choose_first(S, k, sc1);
    }
    while (n_exp > 0) {
        if (l == xl) {
            emit_level(a, b, l, k, n_exp, tok_count, word, a.prefix_len ? a.prefix_len[b] : 0, [&](int s, int &token) { return node_of(S, l, s, token); });
            return -1;
        }
        // slots beyond the expanded set own no node: their candidates do not exist
        if (n_exp < k && lane >= n_exp && lane < DT_K_MAX) S.par[l][lane].score = -INFINITY;
        // level l + 1: score = score[parent] + lp
        float sc[G];
        u64 path[G];
        const float f = S.par[l][min(lane, DT_K_MAX)].score + best_own;
#pragma unroll
        for (int q = 0; q < G; ++q) {
            const Parent pr = S.par[l][parent[q]];
            sc[q] = pr.score + own[q];
            path[q] = pr.path;
        }
#pragma unroll
        for (int q = 0; q < G; ++q)
            if (lane + 64 * q < kk) S.score[at[q]] = sc[q];
        p_end += kk;
        ++l;
        if (l == l_end) break;  // the deepest level is not expanded
        if (a.early_stop) {
#pragma unroll
            for (int q = 0; q < G; ++q) tok_count += __popcll(__builtin_amdgcn_ballot_w64(sc[q] > -INFINITY));
            n_exp = 0;
            if (tok_count >= TT) break;
        }
        // asked for before the choice (past the deepest level: whatever is there)
        best_at += kk;
        best_own = S.lp[best_at];
#pragma unroll
        for (int q = 0; q < G; ++q) own[q] = S.lp[at[q] + kk];
        u32 key[G], lo, hi;
        bool chosen[G];
#pragma unroll
        for (int q = 0; q < G; ++q) key[q] = score_key(sc[q]);
        level_bounds(score_key(f), k, lo, hi);
        n_exp = wave_select<G>(key, k, lo, hi, chosen);
        int before = 0;
#pragma unroll
        for (int q = 0; q < G; ++q) {
            const u64 m = __builtin_amdgcn_ballot_w64(chosen[q]);
            const int pos = (int)__builtin_amdgcn_mbcnt_hi((u32)(m >> 32), __builtin_amdgcn_mbcnt_lo((u32)m, (u32)before));
            if (chosen[q]) put_parent(S, l, pos, sc[q], at[q], path[q]);
            before += __popcll(m);
            at[q] += kk;
        }
    }
    if (xl > 0) {  // an earlier level had nothing viable to expand, or the token count ended the expansion
        if (lane == 0) {
            emit_nothing(a, b, xl, word);
            carry_head(a, b, xl, k, 0, tok_count);
        }
        return -1;
    }
    return p_end;
}

// A bound close below the k best of a level: the best and second best children of k nodes (lane s: the best of slot s, lane 32 + s: the
// second; rows descend) are candidates, so what k of those 64 keys lie above, at least k candidates do.  `lo` and `hi` as level_bounds has them.
__device__ __forceinline__ u32 raise_bound(u32 key, int k, u32 lo, u32 hi) {
    u32 width = hi - lo;
    for (int step = 0; step < 7; ++step) {  // uniform
        const u32 half = width >> 1, mid = lo + half;
        const int c = __popcll(__builtin_amdgcn_ballot_w64(key > mid));
        width -= half;
        lo = c >= k ? mid : lo;
        if (c == k) break;
    }
    return lo;
}
// The k best of n candidates of level l, by one wave; cand: one of them, with its parent's path.
template <int G, typename C>
__device__ __forceinline__ int choose_wide(TreeLds &S, int l, int k, int n, u32 lo_key, u32 hi_key, C cand) {
    const int lane = lane_id();
    Parent pr[G];
    u32 key[G];
    bool chosen[G];
#pragma unroll
    for (int q = 0; q < G; ++q) {
        pr[q] = cand(min(lane + 64 * q, n - 1));
        key[q] = lane + 64 * q < n ? score_key(pr[q].score) : 0u;
    }
    const int c = wave_select<G>(key, k, lo_key, hi_key, chosen);
    int before = 0;
#pragma unroll
    for (int q = 0; q < G; ++q) {
        const u64 m = __builtin_amdgcn_ballot_w64(chosen[q]);
        const int pos = (int)__builtin_amdgcn_mbcnt_hi((u32)(m >> 32), __builtin_amdgcn_mbcnt_lo((u32)m, (u32)before));
        if (chosen[q]) put_parent(S, l, pos, pr[q].score, pr[q].index, pr[q].path);
        before += __popcll(m);
    }
    return c;
}
// All levels of more than NARROW_K^2 candidates, by all waves: Q candidates per thread, k^2 <= Q TREE_NT.  As above.  (Two per thread,
// and lists of up to 128 candidates cut four to a lane instead of two: (TT, d, k) = (80, 6, 20) 14.1 us, 13.3 so.)
template <int Q, bool EXPAND>
__device__ __forceinline__ int levels_wide(const TreeArgs &a, TreeLds &S, int b, int k, int d, int TT, const Start &from, u32 word) {
    const int tid = threadIdx.x, lane = lane_id(), w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int xl = EXPAND ? a.expand_level : 0, kk = k * k;
    const PoolShape ps = pool_shape(k);
    int parent[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) parent[q] = tid + TREE_NT * q < kk ? fdiv(tid + TREE_NT * q, ps.inv_k) : DT_K_MAX;
    if (tid < DT_D_MAX) S.par[tid][DT_K_MAX].score = -INFINITY;
    const float sc1 = lane < k ? S.lp[lane] : -INFINITY;
    if (tid < k) S.score[tid] = sc1;
    int tok_count = 1 + __popcll(__builtin_amdgcn_ballot_w64(sc1 > -INFINITY));
    u32 lo_key = KEY_NEG_INF, hi_key = 0u;
    int lo = 0, p_end = k, c = 0;
    const int l_end = xl > 0 ? xl + 1 : d;
    if (from.level > 0) tok_count = from.tok_count;
    for (int l = max(from.level, 1); l < l_end; ++l) {
        if (a.early_stop && tok_count >= TT) break;  // uniform
        const int nlo = k + (l - 1) * kk;
        float first = -INFINITY, own[Q] = {};
        if (l != xl) {
            first = S.lp[nlo + min(lane & 31, k - 1) * k + (lane >> 5)];  // k > 1
#pragma unroll
            for (int q = 0; q < Q; ++q) own[q] = S.lp[nlo + min(tid + TREE_NT * q, kk - 1)];
        }
        if (w == 0) {
            int n;
            if (l == from.level) n = from.n_exp;
            else if (l == 1) n = choose_first(S, k, sc1);
            else if (c == 0) n = 0;
            else if (c <= 64) n = choose_wide<1>(S, l, k, c, lo_key, hi_key, [&](int i) { return S.cand[i]; });
            else if (c <= 128) n = choose_wide<2>(S, l, k, c, lo_key, hi_key, [&](int i) { return S.cand[i]; });
            else if (c <= CAND_CAP) n = choose_wide<CAND_CAP / 64>(S, l, k, c, lo_key, hi_key, [&](int i) { return S.cand[i]; });
            else  // equal scores
                n = choose_wide<16>(S, l, k, kk, lo_key, hi_key, [&](int i) {
                    Parent pr;
                    pr.score = S.score[lo + i];
                    pr.index = lo + i;
                    pr.path = S.par[l - 1][fdiv(i, ps.inv_k)].path;
                    return pr;
                });
            if (lane >= n && lane < DT_K_MAX) S.par[l][lane].score = -INFINITY;
            if (lane == 0) S.n_exp = n;
            if (l == xl) emit_level(a, b, l, k, n, tok_count, word, a.prefix_len ? a.prefix_len[b] : 0, [&](int s, int &token) { return node_of(S, l, s, token); });
        }
        if (l == xl) return -1;
        __syncthreads();
        if (S.n_exp == 0) break;
        // every wave: the bound; Q candidates per thread scored; those above it into the list
        const float f = S.par[l][(lane & 31) < k ? lane & 31 : DT_K_MAX].score + first;
        Parent pr[Q];
        u32 key[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            pr[q] = S.par[l][parent[q]];
            pr[q].score += own[q];
            pr[q].index = nlo + tid + TREE_NT * q;
        }
        const u32 fk = score_key(f);
        level_bounds(fk, k, lo_key, hi_key);
        lo_key = raise_bound(fk, k, lo_key, hi_key);
        u64 m[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            key[q] = score_key(pr[q].score);
            if (tid + TREE_NT * q < kk) S.score[nlo + tid + TREE_NT * q] = pr[q].score;
            m[q] = __builtin_amdgcn_ballot_w64(key[q] > lo_key);
        }
        if (lane == 0) {
            S.wtot[w] = __popcll(m[0]);
            S.wtot[TREE_NW + w] = Q == 2 ? __popcll(m[Q - 1]) : 0;
        }
        if (a.early_stop) {
            tok_count += __syncthreads_count(pr[0].score > -INFINITY);
            if (Q == 2) tok_count += __syncthreads_count(pr[Q - 1].score > -INFINITY);
        } else {
            __syncthreads();
        }
        const int wt = S.wtot[lane & (2 * TREE_NW - 1)], upto = wave_scan_incl_i32(wt);  // lanes 0 .. 15
        const int at[2] = {__builtin_amdgcn_readlane(upto - wt, w), __builtin_amdgcn_readlane(upto - wt, TREE_NW + w)};
        c = __builtin_amdgcn_readlane(upto, 2 * TREE_NW - 1);
        if (c <= CAND_CAP)
#pragma unroll
            for (int q = 0; q < Q; ++q)
                if (key[q] > lo_key) S.cand[at[q] + (int)lanes_below(m[q])] = pr[q];
        __syncthreads();
        lo = nlo;
        p_end = nlo + kk;
    }
    if (xl > 0) {
        if (tid == 0) {
            emit_nothing(a, b, xl, word);
            carry_head(a, b, xl, k, 0, tok_count);
        }
        return -1;
    }
    return p_end;
}

// ---- rerank ---------------------------------------------------------------------------------------------
// 64 keys reach the worst of the lanes' best ones, 128 the worst of their second best (keep < 128).
template <int G>
__device__ __forceinline__ void lane_bounds(const u32 (&key)[G], int keep, u32 &lo, u32 &hi) {
    u32 m1 = 0u, m2 = 0u;
#pragma unroll
    for (int q = 0; q < G; ++q) {
        m2 = max(m2, min(m1, key[q]));
        m1 = max(m1, key[q]);
    }
    const u32 bound = ~wave_max_u32(~(keep <= 64 ? m1 : m2));
    lo = bound > KEY_NEG_INF ? bound - 1u : KEY_NEG_INF;
    hi = wave_max_u32(m1);
}
// The keep_max best of score[0..n) (fewer if fewer are viable), f(index, position) in ascending index.  Whole workgroup,
// n <= CT TREE_NT, hist[0], mem and memn cleared.
//
// floor(scale (top - score)), kept within 0 .. 255, spreads the scores over buckets that are
// ordered like them.  One histogram and one scan name the bucket that holds the cut; the few
// candidates inside it are ranked one against the other by (key desc, index asc), everything in a better
// bucket is taken.  A bucket with more than BUCKET_CAP candidates (many equal scores, or the last one)
// goes through the radix selection instead.
// (clamped as a float first: converting a float beyond the int range would be undefined)
__device__ __forceinline__ u64 member_key(u32 key, int i) { return ((u64)key << 32) | (u32)(0x7FFFFFFF - i); }

template <int CT, typename F>
__device__ __forceinline__ int block_select(const float *score, int n, float top, float scale, int keep_max, TreeLds &S, F f) {
    auto score_bucket = [&](float s) { return (int)fmaxf(fminf((top - s) * scale, 255.0f), 0.0f); };
    const int tid = threadIdx.x, lane = lane_id(), w = __builtin_amdgcn_readfirstlane(tid >> 6);
    float sc[CT];
#pragma unroll
    for (int c = 0; c < CT; ++c) {
        const float v = score[min(tid * CT + c, n - 1)];
        sc[c] = tid * CT + c < n ? v : -INFINITY;
        if (sc[c] > -INFINITY) atomicAdd(&S.hist[0][score_bucket(sc[c])], 1u);
    }
    __syncthreads();
    // every wave: lane L holds buckets 4L .. 4L+3, best scores first
    const uint4 h = *(const uint4 *)&S.hist[0][4 * lane];
    const int c4 = (int)(h.x + h.y + h.z + h.w);
    const int incl = wave_scan_incl_i32(c4);
    const int keep = min(keep_max, __builtin_amdgcn_readlane(incl, 63));
    if (keep <= 0) return 0;
    const int ls = __ffsll((long long)__builtin_amdgcn_ballot_w64(incl >= keep)) - 1;
    int above = __builtin_amdgcn_readlane(incl - c4, ls);
    const int h0 = __builtin_amdgcn_readlane((int)h.x, ls), h1 = __builtin_amdgcn_readlane((int)h.y, ls),
              h2 = __builtin_amdgcn_readlane((int)h.z, ls), h3 = __builtin_amdgcn_readlane((int)h.w, ls);
    int dg, hB;
    if (above + h0 >= keep) { dg = 0; hB = h0; }
    else {
        above += h0;
        if (above + h1 >= keep) { dg = 1; hB = h1; }
        else {
            above += h1;
            if (above + h2 >= keep) { dg = 2; hB = h2; }
            else { above += h2; dg = 3; hB = h3; }
        }
    }
    const int B = 4 * ls + dg;
    const int need = keep - above;  // how many of bucket B belong to the set: 1 .. hB
    if (hB > BUCKET_CAP) {
        __syncthreads();  // the histogram has been read
        u32 thr;
        int need_eq;
        if (block_radix_cut(score, n, keep_max, S, thr, need_eq) <= 0) return 0;
        return block_enumerate(score, n, thr, need_eq, S, f);
    }
    // the candidates in better buckets, and those in bucket B
    bool sure[CT], inb[CT];
#pragma unroll
    for (int c = 0; c < CT; ++c) {
        const int bk = score_bucket(sc[c]);
        sure[c] = sc[c] > -INFINITY && bk < B;
        inb[c] = sc[c] > -INFINITY && bk == B;
    }
    if (need < hB) {  // the cut runs through bucket B: its members rank themselves
#pragma unroll
        for (int c = 0; c < CT; ++c)
            if (inb[c]) S.mem[atomicAdd(&S.memn, 1)] = member_key(score_key(sc[c]), tid * CT + c);
        __syncthreads();
        bool any = false;
        u64 mine[CT];
        int rank[CT];
#pragma unroll
        for (int c = 0; c < CT; ++c) {
            any = any || inb[c];
            mine[c] = member_key(score_key(sc[c]), tid * CT + c);
            rank[c] = 0;
        }
        if (any)
            for (int j0 = 0; j0 < hB; j0 += 8) {  // entries past the hB members are zero and rank below every member
                u64 o[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) o[j] = S.mem[j0 + j];
#pragma unroll
                for (int c = 0; c < CT; ++c)
#pragma unroll
                    for (int j = 0; j < 8; ++j) rank[c] += o[j] > mine[c] ? 1 : 0;
            }
#pragma unroll
        for (int c = 0; c < CT; ++c) sure[c] = sure[c] || (inb[c] && rank[c] < need);
    } else {
#pragma unroll
        for (int c = 0; c < CT; ++c) sure[c] = sure[c] || inb[c];
    }
    // positions in ascending index
    int below = 0, own = 0;
#pragma unroll
    for (int c = 0; c < CT; ++c) {
        const u64 m = __builtin_amdgcn_ballot_w64(sure[c]);
        below += (int)lanes_below(m);
        own += __popcll(m);
    }
    if (lane == 0) S.wtot[w] = own;
    __syncthreads();
    int pos = below, total = 0;
#pragma unroll
    for (int v = 0; v < TREE_NW; ++v) {
        const int t = S.wtot[v];
        pos += v < w ? t : 0;
        total += t;
    }
#pragma unroll
    for (int c = 0; c < CT; ++c)
        if (sure[c]) f(tid * CT + c, pos++);
    return total;
}

// ---- rows of small trees ------------------------------------------------------------------------------------
// The k best entries of a row that the wave holds, place(rank, value, token) by some lane for every rank below k (value -inf: there are no more), and its log-sum-exp.
// As row_topk_kernel does it, with a slot to a lane: T, the k-th best of the lanes' best entries or little below, and the entries that reach it ranked one against the
// other in `list`.
#define ROW_LIST 64
template <typename F>
__device__ __forceinline__ float wave_row_topk(int V, int k, const float (&x)[ROW_NG][8], const float (&gmx)[ROW_NG], float mx, u64 *list, F place) {
    const int lane = lane_id();
    auto id_of = [&](int n, int e) { return row_group(V, n) + e; };
    auto for_groups = [&](auto f) __attribute__((always_inline)) {
#pragma unroll
        for (int n = 0; n < ROW_NG; ++n)
            if (n == 0 || 512 * n < V) f(n);  // uniform
    };
    const u32 key16[1] = {ord32(mx) >> 16};
    const float T = key_edge(wave_kth<1>(key16, k)), T1 = fmaxf(T, -__FLT_MAX__);  // -inf does not count
    list[lane] = 0ull;
    u32 hits = 0;  // bit 8 n + e: element e of group n
    for_groups([&](int n) {
#pragma unroll
        for (int e = 0; e < 8; ++e) hits |= (x[n][e] >= T1 ? 1u : 0u) << (8 * n + e);
    });
    int n_hits = wave_sum_i32(__popc(hits));
    if (n_hits > ROW_LIST) {
        // Clusters or equal values: the k-th key by bisection, then, of the entries equal to it, the last id.
        auto mask = [&](auto in) {
            u32 m = 0;
            for_groups([&](int n) {
#pragma unroll
                for (int e = 0; e < 8; ++e) m |= (in(x[n][e], id_of(n, e)) ? 1u : 0u) << (8 * n + e);
            });
            return m;
        };
        auto count = [&](u32 m) { return wave_sum_i32(__popc(m)); };
        u32 lo = max(ord32(T1), 0x00800000u), hi = 0xFFFFFFFFu;  // at least k keys reach lo, or all there are; none lies above hi
        int c = n_hits;
        while (hi > lo && c > k) {
            const u32 mid = lo + ((hi - lo) >> 1) + 1u;
            const int m = count(mask([&](float v, int) { return ord32(v) >= mid; }));
            if (m >= k) { lo = mid; c = m; }
            else hi = mid - 1u;
        }
        int id_hi = 0x7FFFFFFF;  // of the entries equal to lo: those up to this id
        if (c > k) {
            const int need = k - count(mask([&](float v, int) { return ord32(v) > lo; }));
            int id_lo = 0;  // the smallest id with `need` of them at or below it
            id_hi = V - 1;
            while (id_hi > id_lo) {
                const int mid = (id_lo + id_hi) >> 1;
                if (count(mask([&](float v, int id) { return ord32(v) == lo && id <= mid; })) >= need) id_hi = mid;
                else id_lo = mid + 1;
            }
        }
        hits = mask([&](float v, int id) { return ord32(v) > lo || (ord32(v) == lo && id <= id_hi); });
        n_hits = count(hits);
    }
    const int own = __popc(hits);
    int at = wave_scan_incl_i32(own) - own;
    for_groups([&](int n) {
        u32 left = hits >> (8 * n) & 0xFFu;
        if (__builtin_amdgcn_ballot_w64(left != 0u))  // uniform
            for (; left; left &= left - 1) {
                const int e = __builtin_ctz(left);
                float v = x[n][0];
#pragma unroll
                for (int j = 1; j < 8; ++j) v = e == j ? x[n][j] : v;
                if (at < ROW_LIST) list[at] = make_key(v, (u32)id_of(n, e));
                ++at;
            }
    });
    const float M = wave_max(mx), sum = wave_row_sum(V, x, M, 1.0f);
    __builtin_amdgcn_wave_barrier();
    const u64 mine = list[lane];
    int rank = 0;
    for (int j0 = 0; j0 < n_hits; j0 += 8) {  // zeros behind the keys
        u64 o[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) o[j] = list[j0 + j];
#pragma unroll
        for (int j = 0; j < 8; ++j) rank += o[j] > mine ? 1 : 0;
    }
    if (lane < n_hits && rank < k) place(rank, key_val(mine), (int)key_idx(mine));
    else if (lane >= n_hits && lane < k) place(lane, -INFINITY, -1);
    return M == -INFINITY ? -INFINITY : M + __logf(sum);
}

// EXPAND: one level's choice; otherwise the whole tree.  (Kernels of their own: what one of them does not do would be instructions to fetch and scalar
// registers spilled in the other's chain.)
// FROM: whose rows have been reduced: the launch's before (ONE_SHOT), level by level (LEVELS); or reduced here, a wave to a row (LOGITS_F32, LOGITS_BF16), in
// the place of a launch in front of this one.  (The finish of a tree built level by level in the kernel of the one-shot build cost that 0.7 us of 7.6, k = 27.)
enum { ONE_SHOT, LEVELS, LOGITS_F32, LOGITS_BF16 };
template <bool EXPAND, int FROM>
__global__ __launch_bounds__(TREE_NT) void tree_kernel(TreeArgs a) {
    constexpr bool ROWS = FROM == LOGITS_F32 || FROM == LOGITS_BF16, FINISH = !EXPAND && FROM == LEVELS;
    const int b = blockIdx.x, tid = threadIdx.x;
    // Row results of sequence b: rows b * seq_rows .. (the same block layout for the one-shot build and
    // the level-at-a-time state), so nothing about them depends on the sequence's parameters.  The first
    // 96 rows are requested before the parameters have arrived: one trip to memory instead of two.
    const int64_t r0 = (int64_t)b * a.seq_rows;
    const float *tv = a.top_val + r0 * DT_K_MAX;
    const int32_t *ti = a.top_id + r0 * DT_K_MAX;
    const float *lse = a.lse + r0;
    constexpr int EARLY = 6;  // entries per thread read ahead: rows 0 .. EARLY * TREE_NT / DT_K_MAX - 1
    float ev[EARLY], el[EARLY];
    int et[EARLY];
    uint4 raw[ROW_NG][2];
    const int row_wave = __builtin_amdgcn_readfirstlane(tid >> 6), early_row = min(row_wave, a.total_rows - 1);  // the first sequence's, as a rule the only one's
    if constexpr (ROWS) wave_row_request<FROM == LOGITS_BF16>(a.logits, early_row * a.row_stride, a.V, raw);
#pragma unroll
    for (int j = 0; j < (ROWS ? 0 : EARLY); ++j) {
        const int e = tid + j * TREE_NT;  // entry (row e / 32, rank e % 32)
        ev[j] = tv[e];
        et[j] = ti[e];
        el[j] = lse[e / DT_K_MAX];
    }
    // The parameters and the root's token, in one trip.  (The token, asked for where it is stored, was a trip more before anything else was
    // done: four trees of a 70B step 13.2 -> 12.8 us, sixteen ragged ones 8.9 -> 8.6, one of (64, 7, 8) 7.6 -> 7.05.)
    const dt_params prm = a.params[b];
    int root = EXPAND ? 0 : a.root_token[b];
    const u32 word = EXPAND ? (u32)a.state_n_exp[b] : 0u;
    int64_t row_begin = 0, row_end = 0;
    if (a.row_off) { row_begin = a.row_off[b]; row_end = a.row_off[b + 1]; }
    // what the level before has left, in the same trip
    const int xl = EXPAND ? a.expand_level : 0;  // > 0: only the nodes of level xl that are expanded next
    int2 head = make_int2(0, 0), narrow_head = make_int2(0, 0);
    uint4 node = make_uint4(0, 0, 0, 0), narrow_node = make_uint4(0, 0, 0, 0);
    if (xl > 1) {
        const int64_t at = carry_at(a.seq_rows, b, xl - 1, false), narrow_at = carry_at(a.seq_rows, b, xl - 1, true);
        head = *(const int2 *)(a.top_id + at);
        node = ((const uint4 *)(a.top_val + at))[tid & (DT_K_MAX - 1)];
        narrow_head = *(const int2 *)(a.top_id + narrow_at);
        narrow_node = ((const uint4 *)(a.top_val + narrow_at))[tid & (DT_K_MAX - 1)];
    }
    // or all levels have left: lane l - 1 of every wave the head of level l's, thread 16 (l - 1) + s its node s
    if constexpr (FINISH) {
        narrow_head = *(const int2 *)(a.top_id + carry_at(a.seq_rows, b, min((tid & 63) + 1, DT_D_MAX - 1), true));
        narrow_node = ((const uint4 *)(a.top_val + carry_at(a.seq_rows, b, min(tid / NARROW_K + 1, DT_D_MAX - 1), true)))[tid % NARROW_K];
    }
    extern __shared__ __attribute__((aligned(16))) unsigned char s_dyn[];  // 135 KB: more than a static array may hold
    TreeLds &S = *reinterpret_cast<TreeLds *>(s_dyn);
    static_assert(DT_P_MAX % 16 == 0 && offsetof(TreeLds, node) % 16 == 0 && offsetof(TreeLds, slot) % 16 == 0, "16-byte stores");
    if constexpr (!EXPAND) {
        for (int i = tid; i < DT_P_MAX / 8; i += TREE_NT) ((uint4 *)S.node)[i] = make_uint4(~0u, ~0u, ~0u, ~0u);
        for (int i = tid; i < DT_P_MAX / 16; i += TREE_NT) ((uint4 *)S.slot)[i] = make_uint4(~0u, ~0u, ~0u, ~0u);
        if (tid < 256) S.hist[0][tid] = 0u;
        if (tid < BUCKET_CAP) S.mem[tid] = 0ull;
        if (tid == 0) S.memn = 0;
    }
    // one-shot build: rows past the span the sequence owns were never reduced; they count as rows
    // without a viable token (the level-at-a-time state has no such span: its rows arrive level by level)
    const int64_t span = a.row_off ? row_end - row_begin : (int64_t)DT_STATE_ROWS;
    const int TT = min(max(prm.TT, 1), a.TT_cap), d = min(max(prm.d, 1), DT_D_MAX);
    const int k = min(max(prm.k, 1), min(DT_K_MAX, a.V));
    const int64_t o = (int64_t)b * a.TT_cap;
    if constexpr (!EXPAND) asm volatile("" : "+s"(root));  // here: the compiler would move the load to the store

    if (xl > 0 && (TT == 1 || xl >= d)) {  // nothing is drafted below level d
        if (tid == 0) emit_nothing(a, b, xl, word);
        return;
    }
    if (tid == 0 && xl == 0) {
        a.tokens[o] = root;
        a.parents[o] = -1;
        a.depth[o] = 0;
        a.score[o] = 0.f;
        a.logp[o] = 0.f;
        a.src_row[o] = 0;
        a.anc_mask[o * DT_MASK_WORDS] = 1ull;
        a.anc_mask[o * DT_MASK_WORDS + 1] = 0ull;
    }
    if (TT == 1) {
        if (tid == 0) a.n_nodes[b] = 1;
        return;
    }
    // Candidates through level d, or through level xl when only that level's choice is wanted (the
    // rows of deeper levels do not exist yet).  Every candidate's own log-probability is known up front: the draft row that would
    // produce pool index p is fixed by p alone (only its parent is decided later).
    // Entry (row, rank) with rank < k is candidate p = rank (row 0) or k + (row - 1) k + rank.
    const int R = xl > 0 ? 1 + (xl - 1) * k : 1 + (d - 1) * k;  // rows that hold candidates
    Start from = {0, 0, 0};
    if (EXPAND && k <= NARROW_K) {
        head = narrow_head;
        node = narrow_node;
    }
    const int tag = __builtin_amdgcn_readfirstlane(head.x);
    if (carries(xl - 1, k <= NARROW_K) && (tag & ~CARRY_COUNT) == carry_tag(xl - 1, 0, a.early_stop))
        from = {xl - 1, min((tag & CARRY_COUNT) >> 4, k), __builtin_amdgcn_readfirstlane(head.y)};
    if (from.level > 0 && tid < DT_K_MAX) {
        if (tid >= from.n_exp) node.x = __float_as_uint(-INFINITY);
        *(uint4 *)&S.par[from.level][tid] = node;
    }
    const int R0 = from.level > 0 ? 1 + (xl - 2) * k : 0;  // the first of them that is needed
    const int owned = (int)min(max(span, (int64_t)0), (int64_t)DT_STATE_ROWS);
    auto place = [&](int e, float v, int token, float row_lse) {
        const int row = e / DT_K_MAX, rank = e % DT_K_MAX;
        if (row < R && rank < k) {
            const int p = row == 0 ? rank : k + (row - 1) * k + rank;
            // Neither +inf nor a NaN: children of slots without a node (score -inf) count on -inf plus this being -inf,
            // and their rows may hold anything: a state row of an earlier step, logits that belong to no node.
            const float lp = v - row_lse;
            S.lp[p] = lp < INFINITY && row < owned ? lp : -INFINITY;
            S.tok[p] = token;
        }
    };
    if constexpr (ROWS) {
        for (int row = row_wave; row < R; row += TREE_NW) {
            if (row < owned) {
                const int64_t g = row_begin + row;
                if (g != early_row) wave_row_request<FROM == LOGITS_BF16>(a.logits, g * a.row_stride, a.V, raw);
                float x[ROW_NG][8], gmx[ROW_NG];
                const float mx = wave_row_unpack<FROM == LOGITS_BF16>(a.V, raw, x, gmx);
                float *const lp = S.lp + (row == 0 ? 0 : k + (row - 1) * k);
                int *const tok = S.tok + (row == 0 ? 0 : k + (row - 1) * k);
                const float row_lse = wave_row_topk(a.V, k, x, gmx, mx, (u64 *)S.cand + row_wave * ROW_LIST, [&](int rank, float v, int token) {
                    lp[rank] = v;
                    tok[rank] = token;
                });
                __builtin_amdgcn_wave_barrier();
                if (lane_id() < k) {
                    const float own = lp[lane_id()] - row_lse;
                    lp[lane_id()] = own < INFINITY ? own : -INFINITY;
                }
            } else if (lane_id() < k) {
                S.lp[k + (row - 1) * k + lane_id()] = -INFINITY;
            }
        }
        static_assert(sizeof(S.cand) >= TREE_NW * ROW_LIST * sizeof(u64), "the waves' lists");
    }
    // The other rows in one more trip, asked for before the early ones are placed (behind them the trip began 0.4 us later: a step of one sequence, (67, 7, 29),
    // 2,368 entries, 25.0 -> 24.6 us).
    constexpr int MORE = (DT_STATE_ROWS * DT_K_MAX + TREE_NT - 1) / TREE_NT - EARLY;
    const int more = ROWS ? 0 : (R * DT_K_MAX + TREE_NT - 1) / TREE_NT - EARLY;
    float xv[MORE], xs[MORE];
    int xt[MORE];
    auto place_early = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < (ROWS ? 0 : EARLY); ++j) place(tid + j * TREE_NT, ev[j], et[j], el[j]);
    };
    if (more > 0) {
#pragma unroll
        for (int j = 0; j < MORE; ++j)
            if (j < more && (EARLY + j + 1) * TREE_NT > R0 * DT_K_MAX) {
                const int e = min(tid + (EARLY + j) * TREE_NT, R * DT_K_MAX - 1);
                xv[j] = tv[e];
                xt[j] = ti[e];
                xs[j] = lse[e / DT_K_MAX];
            }
        place_early();
#pragma unroll
        for (int j = 0; j < MORE; ++j)
            if (j < more && (EARLY + j + 1) * TREE_NT > R0 * DT_K_MAX) place(tid + (EARLY + j) * TREE_NT, xv[j], xt[j], xs[j]);
    } else {
        place_early();
    }
    int levels = -1;  // whose nodes are known
    if (FINISH && k <= NARROW_K) {
        const int l = (tid & 63) + 1, n = (narrow_head.x & CARRY_COUNT) >> 4;
        const bool there = l < DT_D_MAX && (narrow_head.x & ~CARRY_COUNT) == carry_tag(l, 0, a.early_stop) && n <= k;
        const u64 ok = __builtin_amdgcn_ballot_w64(there), last = __builtin_amdgcn_ballot_w64(there && n == 0) | 1ull << (d - 1);
        const int up_to = __builtin_ctzll(last);  // levels with nodes; the one behind them has none, or is the deepest
        const u64 needed = (2ull << min(up_to, max(d - 2, 0))) - 1ull;
        if (d == 1 || (ok & needed) == needed) levels = up_to;
        const int of = tid / NARROW_K + 1, mine = __shfl(n, of - 1);
        if (of <= levels) {
            if (tid % NARROW_K >= mine) narrow_node.x = __float_as_uint(-INFINITY);
            *(uint4 *)&S.par[of][tid % NARROW_K] = narrow_node;
        }
    }
    __syncthreads();

    // ---- expansion -------------------------------------------------------------------------------
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = lane_id();
    int p_end = 0;
    if (FINISH && levels >= 0) {  // uniform
        p_end = k + levels * k * k;
        const int of = tid / NARROW_K + 1;
        const Parent own = __builtin_bit_cast(Parent, narrow_node);
        if (of <= levels && own.score > -INFINITY) S.slot[min(max(own.index, 0), DT_P_MAX - 1)] = (int8_t)(tid % NARROW_K);
        const PoolShape ps = pool_shape(k);
        for (int p = tid; p < p_end; p += TREE_NT) {
            const Decoded dc = decode(p, ps);
            S.score[p] = p < k ? S.lp[p] : S.par[dc.level - 1][dc.slot].score + S.lp[p];
        }
        __syncthreads();
    } else if (k > NARROW_K) {
        p_end = k * k <= TREE_NT ? levels_wide<1, EXPAND>(a, S, b, k, d, TT, from, word) : levels_wide<2, EXPAND>(a, S, b, k, d, TT, from, word);
        if constexpr (EXPAND) return;
        __syncthreads();  // the levels may have ended without one
    } else {
        if (w == 0) {
            if (k <= 8) p_end = levels_narrow<1, EXPAND>(a, S, b, k, d, TT, from, word);
            else if (k <= 11) p_end = levels_narrow<2, EXPAND>(a, S, b, k, d, TT, from, word);
            else if (k <= 13) p_end = levels_narrow<3, EXPAND>(a, S, b, k, d, TT, from, word);  // four per lane: (96, 8, 12) 10.8 us, 10.4 so
            else p_end = levels_narrow<4, EXPAND>(a, S, b, k, d, TT, from, word);
            if (lane == 0) S.p_end = p_end;
        }
        if constexpr (EXPAND) return;
        __syncthreads();
        p_end = S.p_end;
    }

    // ---- rerank: the TT-1 best of the whole pool ----------------------------------------------
    auto kept = [&](int i, int pos) {
        S.node[i] = (int16_t)(pos + 1);
        S.sel[pos] = (int16_t)i;
    };
    // 256 buckets over the best 32 or 16 nats: the larger the pool, the closer to its top the cut
    const float scale = p_end <= 256 ? 8.0f : 16.0f;
    int keep;
    if (p_end <= TREE_NT) {
        keep = block_select<1>(S.score, p_end, S.score[0], scale, TT - 1, S, kept);
    } else if (p_end <= 2 * TREE_NT) {
        keep = block_select<2>(S.score, p_end, S.score[0], scale, TT - 1, S, kept);
    } else {
        // Consecutive candidates per thread, an odd number of them (64 lanes then read 64 banks).  The loops over them are unrolled, and
        // three lengths of them there: with the longest for every pool, and every index held to the pool's end, (80, 6, 16) took 10.5
        // us and (80, 6, 20) 13.3; 9.7 and 12.6 so.  Past the pool's end they read what follows the scores in LDS, and use none of it.
        const int C = ((p_end + TREE_NT - 1) / TREE_NT) | 1;
        static_assert((TREE_NT - 1) * SHARE_MAX + SHARE_MAX <= 2 * DT_P_MAX, "the scores and what follows them");
        auto by_share = [&](auto f) __attribute__((always_inline)) {
            using std::integral_constant;
            if (C <= 5) f(integral_constant<int, 5>());
            else if (C <= 9) f(integral_constant<int, 9>());
            else f(integral_constant<int, SHARE_MAX>());
        };
        const float *pool = (const float *)s_dyn;  // S.score
        static_assert(offsetof(TreeLds, score) == 0 && offsetof(TreeLds, lp) == DT_P_MAX * sizeof(float), "the scores come first");
        // the threads' best ones, each of candidates TREE_NT apart (the children of one node are neighbours)
        u32 best = 0u;
        by_share([&](auto share) __attribute__((always_inline)) {
#pragma unroll
            for (int c = 0; c < decltype(share)::value; ++c) {
                const int i = tid + TREE_NT * c;
                const u32 kv = score_key(pool[i]);
                best = max(best, i < p_end ? kv : 0u);
            }
        });
        S.best[tid] = best;
        __syncthreads();
        // every wave by itself: a bound that TT - 1 of them reach, and not many more
        u32 bk[TREE_NW], lo, hi;
#pragma unroll
        for (int q = 0; q < TREE_NW; ++q) bk[q] = S.best[64 * q + lane];
        lane_bounds<TREE_NW>(bk, TT - 1, lo, hi);
        int n = count_above<TREE_NW>(bk, lo);
        while (n > 320 && hi - lo > 1u) {
            const u32 mid = lo + ((hi - lo) >> 1);
            const int nm = count_above<TREE_NW>(bk, mid);
            if (nm >= TT - 1) { lo = mid; n = nm; }
            else hi = mid;
        }
        // what lies above, in pool order
        u32 over = 0u;
        by_share([&](auto share) __attribute__((always_inline)) {
#pragma unroll
            for (int c = 0; c < decltype(share)::value; ++c) {
                const u32 kv = score_key(pool[tid * C + c]);
                over |= (c < C && tid * C + c < p_end && kv > lo ? 1u : 0u) << c;
            }
        });
        const int own = __popc(over), incl = wave_scan_incl_i32(own);
        if (lane == 63) S.wtot[w] = incl;
        __syncthreads();
        int at = incl - own, total = 0;
#pragma unroll
        for (int v = 0; v < TREE_NW; ++v) {
            const int nv = S.wtot[v];
            at += v < w ? nv : 0;
            total += nv;
        }
        if (total <= LIST_CAP) {  // uniform
            for (; over; over &= over - 1u) S.list[at++] = (int16_t)(tid * C + __builtin_ctz(over));
            __syncthreads();
            // every thread the scores that it is going to look at (read where the list is made, one behind the other, they cost (128, 8, 32)
            // 0.35 us more)
            const int share = total <= TREE_NT ? 1 : 2;
            for (int c = 0; c < share; ++c)
                if (tid * share + c < total) S.list_score[tid * share + c] = S.score[S.list[tid * share + c]];
            auto kept_of_list = [&](int i, int pos) { kept(S.list[i], pos); };
            const float top = S.score[0], range = top - (lo > KEY_NEG_INF ? unord32(lo) : top - 32.0f);
            const float fit = range > 0.0f ? 255.0f / range : 8.0f;
            if (total <= TREE_NT) keep = total == 0 ? 0 : block_select<1>(S.list_score, total, top, fit, TT - 1, S, kept_of_list);
            else keep = block_select<2>(S.list_score, total, top, fit, TT - 1, S, kept_of_list);
        } else {  // equal scores
            __syncthreads();  // wtot has been read
            u32 thr;
            int need_eq;
            keep = block_radix_cut(S.score, p_end, TT - 1, S, thr, need_eq);
            if (keep > 0) keep = block_enumerate(S.score, p_end, thr, need_eq, S, kept);
        }
    }
    __syncthreads();
    if (tid == 0) a.n_nodes[b] = keep + 1;

    // ---- emission -------------------------------------------------------------------------------
    // (a wave issues one instruction in eight cycles at best, two waves twice as many: two threads per node)
    const int t = tid & (DT_TT_MAX - 1);
    if (t >= keep || tid >= 2 * DT_TT_MAX) return;
    const int p = S.sel[t], n = t + 1;
    const Decoded dc = decode(p, pool_shape(k));
    if (tid >= DT_TT_MAX) {
        const int slot = S.slot[p];
        a.tokens[o + n] = S.tok[p];
        a.depth[o + n] = dc.level;
        a.score[o + n] = S.score[p];
        a.logp[o + n] = S.lp[p];
        a.src_row[o + n] = slot >= 0 ? 1 + (dc.level - 1) * k + slot : -1;
        return;
    }
    // the ancestors: their slots stand in the parent's path
    const u64 path = dc.level > 1 ? S.par[dc.level - 1][dc.slot].path : 0ull;
    int up[DT_D_MAX - 1], parent = 0;
#pragma unroll
    for (int j = 1; j < DT_D_MAX; ++j) {
        const int index = S.par[j][(path >> (5 * (j - 1))) & 31].index;
        up[j - 1] = j < dc.level ? index : 0;
    }
#pragma unroll
    for (int j = 1; j < DT_D_MAX; ++j) up[j - 1] = j < dc.level ? max((int)S.node[up[j - 1]], 0) : 0;
    u64 m0 = 1ull | (n < 64 ? 1ull << n : 0ull), m1 = n < 64 ? 0ull : 1ull << (n - 64);  // the root and itself
#pragma unroll
    for (int j = 1; j < DT_D_MAX; ++j) {
        const u64 bit = 1ull << (up[j - 1] & 63);
        m0 |= up[j - 1] < 64 ? bit : 0ull;
        m1 |= up[j - 1] < 64 ? 0ull : bit;
        parent = j < dc.level ? up[j - 1] : parent;
    }
    a.parents[o + n] = parent;
    a.anc_mask[(o + n) * DT_MASK_WORDS] = m0;
    a.anc_mask[(o + n) * DT_MASK_WORDS + 1] = m1;
}


// LDS beyond 64 KB has to be asked for, once per device (dt_init)
hipError_t tree_init() {
    const void *const kernels[] = {(const void *)tree_kernel<false, ONE_SHOT>, (const void *)tree_kernel<false, LEVELS>, (const void *)tree_kernel<true, LEVELS>,
                                   (const void *)tree_kernel<false, LOGITS_F32>, (const void *)tree_kernel<false, LOGITS_BF16>};
    hipError_t e = hipSuccess;
    for (const void *k : kernels)
        if (e == hipSuccess) e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)sizeof(TreeLds));
    return e;
}

// Rows that a wave holds, few enough for a wave of the workgroup to each, whichever sequence has more than the one that all have: one launch in place of two.
// us a step, two launches -> one, graph | eager: 5 rows of 1,024 fp32 entries 21.4 -> 19.5 | 18.0 -> 16.3, bf16 22.1 -> 20.2 | 18.5 -> 17.1; 7 of 2,048 22.4 -> 21.3 | 18.9 -> 18.0, bf16
// 22.7 -> 21.8 | 19.2 -> 18.2; but two rows to a wave, 10 of 2,047 22.6 -> 23.0, 16 of 2,048 22.8 -> 24.3, bf16 23.1 -> 25.0.
// While every sequence has a compute unit to itself (the tree's LDS leaves room for one): 256 sequences of 2,048 bf16 entries, one of eight rows, the others of one, 9.3 -> 8.2, 257 12.1 -> 13.0, 1,031 rows
// 22.6 -> 24.8; fp32 9.6 -> 8.4, 12.2 -> 13.3, 23.4 -> 25.8.
#define TREE_ROWS_BATCH 256
bool tree_takes_rows(int64_t total_rows, int batch, int V) {
    return batch <= TREE_ROWS_BATCH && total_rows - (batch - 1) <= TREE_NW && V >= 8 && V <= ROW_V_MAX;
}

hipError_t tree_launch(const TreeArgs &a, hipStream_t st) {
    if (a.batch <= 0) return hipSuccess;
    auto go = [&](auto kernel) { launch_kernel(KID_TREE, st, kernel, dim3(a.batch), dim3(TREE_NT), sizeof(TreeLds), a); };
    if (a.expand_level > 0) go(tree_kernel<true, LEVELS>);
    else if (!a.row_off) go(tree_kernel<false, LEVELS>);
    else if (!a.logits) go(tree_kernel<false, ONE_SHOT>);
    else if (a.dtype == DT_BF16) go(tree_kernel<false, LOGITS_BF16>);
    else go(tree_kernel<false, LOGITS_F32>);
    return hipGetLastError();
}

}  // namespace dt
