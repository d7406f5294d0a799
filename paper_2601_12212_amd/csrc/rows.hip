// Row kernels: top-k and log-sum-exp over vocabulary rows (draft rows: k best + lse;
// target rows: arg max, and lse of row/T for stochastic acceptance).
//
// Top-k rows of up to 16,384 entries are held by one workgroup each (row_topk_kernel).  Longer ones take two passes, of one launch while
// that has room on the chip (row_select_kernel).  The
// first is a pure stream: a row is cut into chunks of
// 256*8*NL elements, each lane reads 8*NL of them with coalesced 16-byte loads, and a pair of lanes leaves
// only its maximum (plus one (max, sum-exp) pair per wave).  The second works on those lane
// maxima, 16*NL times fewer than the logits: the k-th largest lane maximum bounds the k-th
// largest element from below, so only the ~k pairs that reach it are read again and their
// elements ranked by 64-bit (value, id) keys -- exact under (value desc, id asc).  Where
// that bound leaves too many, a pass over them keeps the k best so far.
#include <stddef.h>

#include <type_traits>

#include "level.hpp"

namespace dt {

// ---------------------------------------------------------------- row -> (valid, k) ----
struct RowMeta {
    bool valid;
    int k;
    int64_t out;  // row index of the results (top-k values, ids, lse)
    int seq, slot, rows;  // ROWS_LEVEL, ROWS_CHOOSE: the sequence, which of its rows, how many are reduced
    bool expands;         // and whether its level is to be chosen
};

template <int MODE>
__device__ __forceinline__ RowMeta row_meta(const RowArgs &a, int64_t g) {
    RowMeta m;
    m.valid = true;
    m.k = a.k_uniform;
    m.out = g;
    if constexpr (MODE == ROWS_LEVEL || MODE == ROWS_CHOOSE) {
        // level-at-a-time build: row s of sequence b in this call is the row of the s-th node expanded
        // one level up (level 1: the root's row); its results go to the sequence's row slot in the state
        const int b = (int)((u32)g / (u32)a.rows_per_seq), s = (int)((u32)g % (u32)a.rows_per_seq);  // fewer than 2^31 rows
        const dt_params p = a.params[b];
        const int TT = min(max(p.TT, 1), a.TT_cap), d = min(max(p.d, 1), DT_D_MAX);
        const int k = min(max(p.k, 1), min(DT_K_MAX, a.V));
        // Where what the level before expanded is not known (this one is asked for again after later ones), every row: results of rows that belong to no
        // node are not used.
        const int last = level_count((u32)a.n_exp_prev[b], a.level - 1);
        const int cnt = a.level == 1 ? 1 : last >= 0 ? min(last, k) : k;
        m.k = k;
        m.valid = TT > 1 && a.level <= d && s < cnt;
        m.out = (int64_t)b * a.state_rows + (a.level == 1 ? 0 : 1 + (a.level - 2) * k + s);
        m.seq = b;
        m.slot = s;
        m.rows = min(cnt, a.rows_per_seq);
        m.expands = a.level < d;
    } else if constexpr (MODE == ROWS_DRAFT) {
        // sequence b with row_off[b] <= g < row_off[b+1].  A few sequences: bisection, every step one scalar read.  More:
        // lane j looks at sequence j (of each group of 64), offsets and limits together, one trip to memory instead of
        // one per step (a launch that looks before it reads has all of them in front of its loads: 1.4 GB of draft rows
        // of 64 sequences streamed in 261 us instead of 273).
        int lo = 0;
        int64_t r_lo, r_hi;
        dt_params p;
        if (a.batch <= 4) {
            int hi = a.batch;
            while (hi - lo > 1) {
                const int mid = (lo + hi) >> 1;
                if (a.row_off[mid] <= g) lo = mid; else hi = mid;
            }
            r_lo = a.row_off[lo];
            r_hi = a.row_off[lo + 1];
            p = a.params[lo];
        } else {
            r_lo = r_hi = 0;
            p.TT = p.d = p.k = 0;
            for (int b0 = 0; b0 < a.batch; b0 += 64) {
                const int b = min(b0 + lane_id(), a.batch - 1);
                const int64_t o0 = a.row_off[b], o1 = a.row_off[b + 1];
                const dt_params q = a.params[b];
                const int n = __popcll(__ballot(b0 + lane_id() < a.batch && o0 <= g));  // offsets do not decrease
                if (n == 0) break;
                lo = b0 + n - 1;
                r_lo = (int64_t)readlane_u64((u64)o0, n - 1);
                r_hi = (int64_t)readlane_u64((u64)o1, n - 1);
                p.TT = __builtin_amdgcn_readlane(q.TT, n - 1);
                p.d = __builtin_amdgcn_readlane(q.d, n - 1);
                p.k = __builtin_amdgcn_readlane(q.k, n - 1);
                if (n < 64) break;
            }
        }
        const int r = (int)(g - r_lo);
        const int TT = min(max(p.TT, 1), a.TT_cap), d = min(max(p.d, 1), DT_D_MAX);
        const int k = min(max(p.k, 1), min(DT_K_MAX, a.V));
        m.k = k;
        m.valid = (TT > 1) && (r < 1 + (d - 1) * k) && (g < r_hi);
        m.out = (int64_t)lo * DT_STATE_ROWS + r;  // results in the sequence's own block of rows
    } else if constexpr (MODE == ROWS_TARGET) {
        const int b = (int)((u32)g / (u32)a.TT_cap), i = (int)((u32)g % (u32)a.TT_cap);
        m.k = 1;
        m.valid = i < a.n_nodes[b];
    }
    return m;
}

// -------------------------------------------------------------------- chunk loading -----
// Element (n, e) of a lane, n < NL, e < 8, has id = base + n*512 + e with
// base = chunk*256*8*NL + wave*64*8*NL + lane*8: one coalesced 16-byte load per (lane, n).
// Two halves, so that a kernel can put other waits (the row's metadata) or another chunk's arithmetic between them:
// chunk_request asks for a lane's NL groups of eight, unconditionally, so that they are in flight together -- a load
// inside a divergent branch is waited for inside that branch, and the NL trips to memory would follow one another.  A
// group that reaches past the row is taken from the row's last eight elements instead (V >= 8 on the vector path):
// group_start says where it really starts, and chunk_finish hides the elements that belong to the group before it.
// Without VEC (V < 8) everything happens in chunk_finish.
template <int NL, bool BF16>
struct RawChunk {
    uint4 r[BF16 ? NL : 2 * NL];
};
__device__ __forceinline__ int group_start(int V, int id0) { return min(id0, V - 8); }

template <int NL, bool BF16, bool VEC, bool KEEP = false>
__device__ __forceinline__ void chunk_request(const RowArgs &a, int64_t g, int base, RawChunk<NL, BF16> &raw) {
    if (!VEC) return;
    const int V = a.V;
    if (BF16) {
        const uint16_t *row = (const uint16_t *)a.logits + g * a.row_stride;
#pragma unroll
        for (int n = 0; n < NL; ++n) raw.r[n] = load16<KEEP>(row + group_start(V, base + n * 512));
    } else {
        const float *row = (const float *)a.logits + g * a.row_stride;
#pragma unroll
        for (int n = 0; n < NL; ++n) {
            const float *p = row + group_start(V, base + n * 512);
            raw.r[2 * n] = load16<KEEP>(p);
            raw.r[2 * n + 1] = load16<KEEP>(p + 4);
        }
    }
    __builtin_amdgcn_sched_barrier(0);  // every request is out before anything that follows
}
// cend: first element past the chunk (the same for all lanes).  PASS: groups of the last chunk that end inside the row are passed over.
template <int NL, bool BF16, bool VEC, bool PASS = true>
__device__ __forceinline__ void chunk_finish(const RowArgs &a, int64_t g, int base, int cend, const RawChunk<NL, BF16> &raw,
                                             float (&x)[8 * NL]) {
    const int V = a.V;
    if (!VEC) {
#pragma unroll
        for (int n = 0; n < NL; ++n)
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int id = base + n * 512 + e;
                x[n * 8 + e] = -INFINITY;
                if (id < V)
                    x[n * 8 + e] = BF16 ? bf16_bits_to_float(((const uint16_t *)a.logits)[g * a.row_stride + id])
                                        : ((const float *)a.logits)[g * a.row_stride + id];
            }
        return;
    }
    if (BF16) {
#pragma unroll
        for (int n = 0; n < NL; ++n) {
            const u32 rr[4] = {raw.r[n].x, raw.r[n].y, raw.r[n].z, raw.r[n].w};
#pragma unroll
            for (int p = 0; p < 4; ++p) {
                x[n * 8 + 2 * p] = __uint_as_float(rr[p] << 16);
                x[n * 8 + 2 * p + 1] = __uint_as_float(rr[p] & 0xFFFF0000u);
            }
        }
    } else {
#pragma unroll
        for (int n = 0; n < 2 * NL; ++n) {
            x[n * 4 + 0] = __uint_as_float(raw.r[n].x); x[n * 4 + 1] = __uint_as_float(raw.r[n].y);
            x[n * 4 + 2] = __uint_as_float(raw.r[n].z); x[n * 4 + 3] = __uint_as_float(raw.r[n].w);
        }
    }
    const int wave0 = __builtin_amdgcn_readfirstlane(base);
    if (BF16 && wave0 < 0) x[0] = base < 0 ? -INFINITY : x[0];  // the entry before the row (row_shift)
    if (cend > V) {  // the row's last chunk
#pragma unroll
        for (int n = 0; n < NL; ++n) {
            if (PASS && wave0 + (n + 1) * 512 <= V) continue;  // uniform
            const int first = base + n * 512 - group_start(V, base + n * 512);  // eight and more: none of the group exists
#pragma unroll
            for (int e = 0; e < 8; ++e) x[n * 8 + e] = e >= first ? x[n * 8 + e] : -INFINITY;
        }
    }
}

// (max, sum of exp((x - max) * inv_t)) of a wave's elements, from the lane maxima.
template <int E>
__device__ __forceinline__ float2 wave_lse_partial(const float (&x)[E], float mx, float inv_t) {
    const float cexp = 1.4426950408889634f * inv_t;
    const float mref = mx == -INFINITY ? 0.f : mx;
    const float nm = -mref * cexp;
    float s = 0.f;
#pragma unroll
    for (int j = 0; j < E; ++j) s += __builtin_amdgcn_exp2f(fmaf(x[j], cexp, nm));
    const float M = wave_max(mx);
    const float Mref = M == -INFINITY ? 0.f : M;
    float term = s > 0.f ? s * __builtin_amdgcn_exp2f((mref - Mref) * cexp) : 0.f;
    return make_float2(M, wave_sum(term));
}

// ------------------------------------------------------------ streaming kernel (top-k rows) --
// Pure stream: every wave reads its 64*8*NL elements once and leaves behind one maximum per
// pair of lanes and one (max, sum) pair per wave.  No LDS, no barrier.  All selection happens later on
// the lane maxima, which are 16*NL times fewer than the logits.
// (One per lane, the four waves of a chunk interleaved, was 3 % of the traffic, in 2-byte pieces eight bytes apart: 1.55 GB of
// rows 299 us, 292 with a pair's maximum and a wave's side by side; 156 MB 31.9 and 30.2.)
template <bool BF16>
using LaneMax = std::conditional_t<BF16, uint16_t, float>;
template <bool BF16>
__device__ __forceinline__ LaneMax<BF16> lane_max_pack(float v) {
    if constexpr (BF16) return (uint16_t)(__float_as_uint(v) >> 16);
    else return v;
}
template <bool BF16>
__device__ __forceinline__ float lane_max_value(LaneMax<BF16> v) {
    if constexpr (BF16) return bf16_bits_to_float(v);
    else return v;
}

// CPW chunks of a row per workgroup, one after the other, the next one's elements on their way while one is worked on.
template <int MODE, int NL, bool BF16, int CPW>
__global__ __launch_bounds__(256) void row_stream_kernel(RowArgs a, int S) {
    constexpr int E = 8 * NL;
    // workgroup (chunks c0 .., row g): the chunks ride in grid x, the row in y and -- past 65,535 rows -- z
    // (no division in front of the loads: a streaming workgroup's life is one trip to memory long)
    const int64_t g = (int64_t)blockIdx.z * gridDim.y + blockIdx.y;
    const int c0 = blockIdx.x * CPW;
    const int lane = lane_id(), w = threadIdx.x >> 6;
    const int base = c0 * (256 * E) + w * (64 * E) + lane * 8 - row_shift(a.logits, BF16, a.V, a.row_stride, g);
    // (S stands at the end of the arguments: a comparison with it here cost launches of short chunks 1 %)
    if (g >= a.n_rows || c0 * (256 * E) >= a.V) return;
    // early: the row's elements are on their way while the (dependent, scalar) reads of its metadata are waited for
    RawChunk<NL, BF16> raw[CPW > 1 ? 2 : 1];
    if (a.early_load) chunk_request<NL, BF16, true>(a, g, base, raw[0]);
    if (!row_meta<MODE>(a, g).valid) return;
    if (!a.early_load) chunk_request<NL, BF16, true>(a, g, base, raw[0]);
#pragma unroll
    for (int i = 0; i < CPW; ++i) {
        const int c = c0 + i;
        if (CPW > 1 && c >= S) return;
        if (i + 1 < CPW && c + 1 < S) chunk_request<NL, BF16, true>(a, g, base + (i + 1) * (256 * E), raw[(i + 1) & 1]);
        float x[E];
        // (passing over groups gains nothing in fp32, where the branches cost registers, 42 -> 62: 1,000 rows of 128,257 entries 93.6 -> 94.3 us, 2,000 of 70,001
        // 103.5 -> 104.2)
        chunk_finish<NL, BF16, true, BF16>(a, g, base + i * (256 * E), (c + 1) * (256 * E), raw[i & 1], x);
        float mx = x[0];
#pragma unroll
        for (int j = 1; j < E; ++j) mx = fmaxf(mx, x[j]);
        // maxima of two lanes in the row's own precision (exact)
        const int64_t chunk = g * S + c;
        const float mx2 = fmaxf(mx, __int_as_float(dpp_mov<0xB1, 0xf>(0, __float_as_int(mx))));  // lane ^ 1
        if ((lane & 1) == 0) {
            LaneMax<BF16> *lm = (LaneMax<BF16> *)a.lane_max + chunk * 128 + w * 32 + (lane >> 1);
            if (CPW > 1) __builtin_nontemporal_store(lane_max_pack<BF16>(mx2), lm);
            else *lm = lane_max_pack<BF16>(mx2);
        }
        if (a.want_lse) {
            const float2 p = wave_lse_partial<E>(x, mx, a.inv_t);
            if (lane == 0) a.part_ms[chunk * 4 + w] = p;
        }
    }
}

// ------------------------------------------------------------- selection kernel (top-k rows) --
// One workgroup per row, working on the row's S*128 lane maxima:
//   1. every thread takes the maximum of some lane maxima; the 256 thread maxima meet in LDS as 16-bit keys
//      (the upper half of the ordered integer image: all of it for bf16 data) and every wave finds the k-th largest by
//      itself, four keys to a lane, by bisection over ballots.  T, the lower edge of that key, is a lower bound of the
//      row's k-th largest ELEMENT (k threads have one >= T), and because a thread's lane maxima come from places far
//      apart in the row (spread_max), little more than k lane maxima reach it, also where the best are neighbours;
//   2. the 16*NL elements of the pairs of lanes that reach T are read again, (pair, group of eight) over the threads, and the elements
//      >= T are keyed by (value, id) and ranked by counting.
// More than SEL_CAP such elements (clusters, ties), or a vocabulary of more than 16 chunks, take a second bound first: a
// histogram of the lane maxima that reach T names the bin of the k-th largest lane maximum.  If that leaves too many as
// well (the best of the row in fewer pairs than k, ties, fewer than k finite entries), one pass over the pairs left keeps the k best so far.
// The kernel is two dependent trips to memory (2 x 1.5 us) and the wave arithmetic between them.
// Candidates before another bound is taken.  (128, when a lane maximum stood for half as many elements; with pairs 702 rows of 128,256, k = 12, and 150
// neighbours raised by 20 were 51.8 us, 38.1 so, 51 rows, k = 28, 100 of them 16.4 and 12.1; 2,000 held rows of 8,000, k = 20, 150 of them 81 and 16.8.)
#define SEL_CAP 256
#define SEL_LIST (SEL_CAP + 256)
#define SEL_WAVE_CAP 64  // hot lanes of one wave
// The eight elements from id0 on of row g; returns where they really start (group_start), those before id0 and past the
// row are -inf.
template <bool BF16, bool KEEP>
__device__ __forceinline__ int load_octet(const RowArgs &a, int64_t g, int id0, float (&xv)[8]) {
    const int start = group_start(a.V, id0);
    if (BF16) {
        const uint4 r = load16<KEEP>((const uint16_t *)a.logits + g * a.row_stride + start);
        const u32 rr[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            xv[2 * p] = __uint_as_float(rr[p] << 16);
            xv[2 * p + 1] = __uint_as_float(rr[p] & 0xFFFF0000u);
        }
    } else {
        const float *src = (const float *)a.logits + g * a.row_stride + start;
        const uint4 r0 = load16<KEEP>(src), r1 = load16<KEEP>(src + 4);
        const u32 rr[8] = {r0.x, r0.y, r0.z, r0.w, r1.x, r1.y, r1.z, r1.w};
#pragma unroll
        for (int e = 0; e < 8; ++e) xv[e] = __uint_as_float(rr[e]);
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) xv[e] = start + e >= max(id0, 0) ? xv[e] : -INFINITY;
    return start;
}
// Candidates: of a thread's N elements those that reach T, value x(e), id id_of(e), behind the *n keys already in the list (past its end they
// only count).  A bit for each hit and a loop over the bits, one as a rule, behind one LDS add: a branch and an add for each element, in
// waves that run alone or wait for each other at the next barrier, cost a selection of k = 28 0.25 us and rows that a workgroup holds
// 0.3 to 0.7 of 5 to 7 (128 rows of 32,000 entries, k = 12, 6.93 -> 6.26, 500 of 4,000 5.71 -> 5.13, 2,000 of 8,000 12.8 -> 12.0).
// A hit of the loop costs five times an element of the row of branches, so a wave with more than two to a lane takes the branches: where the
// best of a row are neighbours, eight and more come to one lane (28 rows of 115,042, k = 28, 32 neighbours raised by 20 12.7 us by the loop, 9.5
// so; 50 of 32,000, k = 12, 7.7 and 6.6; two and three to a lane the same).
#define HITS_ONE_BY_ONE 2
template <int N, class X, class Id>
__device__ __forceinline__ void keep_hits(X x, Id id_of, float T, int *n, u64 *list) {
    u32 hits = 0;
#pragma unroll
    for (int e = 0; e < N; ++e) hits |= (x(e) >= T ? 1u : 0u) << e;
    if (hits) {
        const int c = __popc(hits);
        int slot = atomicAdd(n, c);
        if (__builtin_amdgcn_ballot_w64(c > HITS_ONE_BY_ONE)) {  // uniform
#pragma unroll
            for (int e = 0; e < N; ++e) {
                if ((hits >> e & 1u) && slot < SEL_CAP) {
                    float v = x(e);
                    int id = id_of(e);
                    asm("" : "+v"(v), "+v"(id));  // here, for the hits: the compiler would work out every element's key in front of the branch
                    list[slot] = make_key(v, (u32)id);
                }
                slot += hits >> e & 1;
            }
            return;
        }
        for (; hits; hits &= hits - 1) {
            const int at = __builtin_ctz(hits);
            float v = x(0);
#pragma unroll
            for (int e = 1; e < N; ++e) v = at == e ? x(e) : v;
            if (slot < SEL_CAP) list[slot] = make_key(v, (u32)id_of(at));
            ++slot;
        }
    }
}

// A slot's maximum from the two quadruples of neighbouring lane maxima that each lane holds: the lanes L, L ^ 16, L ^ 32 and L ^ 48 exchange
// until each has one of the four places of all their quadruples, 4,096 and more entries of the row apart (v_permlane32_swap and
// v_permlane16_swap exchange halves and odd and even rows of sixteen lanes of two registers, so this deals the maxima out anew
// and loses none).  With a quadruple's four in one slot, the best of a row whose best are neighbours fell into few slots, the bound among the rest
// and too much was read again.  Calls of 51 rows of 128,256 bf16 entries, k = 10, with 256 / 512 / 1,024 neighbours raised by 20: 16.9 / 18.5 / 19.7 us so,
// 9.2 / 9.3 / 9.1 with places far apart (rows without neighbours 8.5 to 8.9 both).
__device__ __forceinline__ float spread_max(const float (&it)[8]) {
    float m[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) m[j] = fmaxf(it[j], it[j + 4]);
    asm volatile("s_nop 1\n\tv_permlane32_swap_b32 %0, %2\n\tv_permlane32_swap_b32 %1, %3\n\ts_nop 1"
                 : "+v"(m[0]), "+v"(m[1]), "+v"(m[2]), "+v"(m[3]));
    float lo = fmaxf(m[0], m[2]), hi = fmaxf(m[1], m[3]);
    asm volatile("s_nop 1\n\tv_permlane16_swap_b32 %0, %1\n\ts_nop 1" : "+v"(lo), "+v"(hi));
    return fmaxf(lo, hi);
}

// A lane maximum, or four, that another workgroup of the launch may have written (SAME) or an earlier launch.
template <bool BF16>
struct alignas(4 * sizeof(LaneMax<BF16>)) Quad { LaneMax<BF16> v[4]; };
template <bool BF16, bool SAME>
__device__ __forceinline__ Quad<BF16> quad_at(const LaneMax<BF16> *lm, int i) {
    const Quad<BF16> *p = (const Quad<BF16> *)lm + i;
    if constexpr (!SAME) return *p;
    else {
        u64 v[sizeof(Quad<BF16>) / 8];
#pragma unroll
        for (int j = 0; j < (int)(sizeof(Quad<BF16>) / 8); ++j) v[j] = get_agent((u64 *)p + j);
        return __builtin_bit_cast(Quad<BF16>, v);
    }
}
template <bool BF16, bool SAME>
__device__ __forceinline__ LaneMax<BF16> lane_max_at(const LaneMax<BF16> *lm, int i) {
    if constexpr (SAME) return __hip_atomic_load(lm + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else return lm[i];
}
// ---- rows of a level whose nodes are chosen in the same launch ----
// (ROWS_CHOOSE, kernels of their own: where the level's nodes are chosen by a launch behind it, two sequences of up to (83, 6, 31) and 16,640 entries, the tail's
// test and stores to the memory side cost a launch of rows 6.99 -> 7.57 us.)
struct NoTail {};
template <int MODE>
using Tail = std::conditional_t<MODE == ROWS_CHOOSE, LevelTail, NoTail>;
// A row's results, which another workgroup of the launch may read.
template <int MODE, typename T>
__device__ __forceinline__ void put_result(T *p, T v) {
    if constexpr (MODE == ROWS_CHOOSE) put32_agent(p, v);
    else *p = v;
}
// The tail's arguments, at `offset` of the kernel's.  Read from there and not as the argument that it is: its twenty pointers would be asked for
// at the kernel's start and held, 60 scalar registers spilled to vector ones in every workgroup of a row.
__device__ __forceinline__ const LevelTail &tail_at(size_t offset) {
    typedef __attribute__((address_space(4))) const char Arg;
    Arg *p = (Arg *)__builtin_amdgcn_kernarg_segment_ptr() + offset;
    asm volatile("" : "+s"(p));
    return *(const LevelTail *)p;
}
struct SelectArgs { RowArgs a; int nl, S; float *top_val; int32_t *top_id; float *lse; int out_stride; u64 tag; LevelTail tail; };  // as the kernels have them
struct HeldArgs { RowArgs a; float *top_val; int32_t *top_id; float *lse; int out_stride; LevelTail tail; };
__device__ __forceinline__ LevelLds &level_lds() {
    __shared__ LevelLds s_level;
    return s_level;
}
// The end of a row's workgroup.
template <int MODE, size_t OFFSET>
__device__ __forceinline__ void level_row_end(const RowMeta &meta, bool lse_wg) {
    if constexpr (MODE == ROWS_CHOOSE) {
        if (!meta.expands) return;
        const LevelTail &tail = tail_at(OFFSET);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (threadIdx.x >= 64) return;
        const int lane = lane_id(), b = __builtin_amdgcn_readfirstlane(meta.seq);
        const Marks marks = level_marks(tail, b, meta.rows);
        if (!mark_done(marks, meta.slot + (lse_wg ? NARROW_K : 0), lane)) return;
        level_expand(tail, marks, level_lds(), b, level_in(tail.t, tail.rows, b, lane), lane);
    }
}
// True for the workgroups that wait for a sequence's rows, which have then done so; wg: the workgroup's number.
template <int MODE, size_t OFFSET>
__device__ __forceinline__ bool level_waits(const Tail<MODE> &arg, u32 wg) {
    if constexpr (MODE == ROWS_CHOOSE) {
        if (wg >= (u32)arg.first_wg) {
            const LevelTail &tail = tail_at(OFFSET);
            const int b = (int)(wg - (u32)tail.first_wg);
            if (threadIdx.x < 64 && b < tail.t.batch) level_wait_and_expand(tail, level_lds(), b, lane_id());
            return true;
        }
    }
    return false;
}

#define ROW_MARKS 18  // marks of a row's chunks and of the workgroup that waits for them, and a claim
// PASS: the maxima are made in the same launch, in chunks of 2,048 PASS entries, up to 16 of them.  0: by the launch before.
// Both passes in one launch: workgroups of the stream, and one to a row that waits for the row's chunks and selects.  Between two launches lie the first one's end, the
// second's start, its arguments and its rows' metadata; here the maxima go through the L2 of the XCD that has the row, in three trips of 0.4 us (written, offered, read),
// and what is read again mostly comes from there as well.  51 rows of 128,256 bf16 entries, from memory: elements there after 2.1 us on average
// (3.2 the last), their maxima 0.5 later, all of a row's at its selecting workgroup after 4.0, bound 1.6 later, hits 1.1, end 0.5.  (As many of
// a row's entries to a workgroup as it can hold, each finding its own k best, and lists of those merged: 11.7 us a call against 9.6 in two launches: 16
// waves take 1.7 us to their bound, and the merge 2.7.)
// (eight waves per SIMD: left alone the compiler takes 76 registers in one mode, 29.3 us for 64 sequences instead of 26.3)
template <int MODE, bool BF16, int PASS>
__global__ __launch_bounds__(256, 8) void row_select_kernel(RowArgs a, int nl_, int S, float *top_val, int32_t *top_id, float *lse, int out_stride, u64 tag, Tail<MODE> tail) {
    constexpr bool SAME = PASS > 0, KEEP = SAME && MODE == ROWS_UNIFORM && !BF16;
    if constexpr (SAME)
        if (level_waits<MODE, offsetof(SelectArgs, tail)>(tail, blockIdx.y * gridDim.x + blockIdx.x)) return;
    const int nl = SAME ? PASS : nl_;
    // (PASS: the workgroups of a row are eight apart: dealt to the XCDs in turn, they fall to one)
    const int64_t g = SAME ? 8 * blockIdx.y + (blockIdx.x & 7) : blockIdx.x;
    const int tid = threadIdx.x, lane = lane_id(), w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int V = a.V, E = 8 * nl;
    const int n_lm = S * 128;
    typedef LaneMax<BF16> LM;
    const LM *lm = (const LM *)a.lane_max + g * n_lm;
    Quad<BF16> q[2];
    const bool lse_wave = w == 3 && a.want_lse && lse;
    float2 pm = make_float2(-INFINITY, 0.f);
    RowMeta meta;
    if constexpr (SAME) {
        const int c = blockIdx.x >> 3;
        if (g >= a.n_rows) return;
        __shared__ int s_go;
        // offers, and marks and a claim, behind the maxima, whose room is twice what they take
        u64 *const words = (u64 *)((char *)a.lane_max + a.n_rows * S * 512), *const marks = words + a.n_rows * LINE_WORDS + g * ROW_MARKS;
        const Hands<1> hands = {words + g * LINE_WORDS, marks, marks + ROW_MARKS - 1, tag, S};
        if (c < S) {
            constexpr int EC = 8 * PASS;
            const int base = c * (256 * EC) + w * (64 * EC) + lane * 8 - row_shift(a.logits, BF16, a.V, a.row_stride, g);
            RawChunk<PASS, BF16> raw;
            chunk_request<PASS, BF16, true, KEEP>(a, g, base, raw);
            meta = row_meta<MODE>(a, g);
            if (!meta.valid) return;
            float x[EC];
            chunk_finish<PASS, BF16, true, BF16>(a, g, base, (c + 1) * (256 * EC), raw, x);
            float mx = x[0];
#pragma unroll
            for (int j = 1; j < EC; ++j) mx = fmaxf(mx, x[j]);
            const float mx2 = fmaxf(mx, __int_as_float(dpp_mov<0xB1, 0xf>(0, __float_as_int(mx))));  // lane ^ 1
            const LM pair = lane_max_pack<BF16>(mx2);
            float2 p = make_float2(0.f, 0.f);
            if (a.want_lse) p = wave_lse_partial<EC>(x, mx, a.inv_t);
            LM *own = (LM *)a.lane_max + (g * S + c) * 128 + w * 32 + (lane >> 1);
            u64 *ms = (u64 *)(a.part_ms + (g * S + c) * 4 + w);
            if ((lane & 1) == 0) *own = pair;
            if (lane == 0) *ms = __builtin_bit_cast(u64, p);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __syncthreads();
            if (w == 0) {
                const bool taken = hand_offer(hands, c, lane);
                if (lane == 0) s_go = !taken;
            }
            __syncthreads();
            if (!s_go) return;
            if ((lane & 1) == 0) __hip_atomic_store(own, pair, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (lane == 0) put_agent(ms, __builtin_bit_cast(u64, p));
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __syncthreads();
        } else {
            meta = row_meta<MODE>(a, g);
            if (!meta.valid) return;
        }
        bool taking = false;
        if (w == 0) {
            const bool all = c < S ? hand_mark(hands, c, lane) : hand_await(hands, lane, taking) || hand_leave(hands, lane);
            if (lane == 0) s_go = all;
        }
        __syncthreads();
        if (!s_go) return;
#pragma unroll
        for (int i = 0; i < 2; ++i) q[i] = quad_at<BF16, true>(lm, 4 * min(64 * i + lane, 8 * S - 1) + w);
        if (lse_wave) pm = __builtin_bit_cast(float2, get_agent((u64 *)(a.part_ms + g * S * 4 + min(lane, S * 4 - 1))));
        if (w == 0) hand_settle(hands, lane, taking, hand_take(hands, lane, taking));
    } else {
        // the lane maxima do not depend on the row's metadata (two dependent global reads): ask for them
        // first, and wave 3 for the row's (max, sum) partials.  Rows that turn out to be dead have their
        // slots in the workspace all the same.
        // A quarter of them to a wave, every fourth of the 32 S quadruples: lane l holds those in places l and l + 64 of its wave's (so far as there
        // are any).  So the waves share what is read again also where the best are in one part of the row: with a quarter of the row to a wave,
        // 51 rows of 128,256 bf16 entries, k = 28, that fall by 12 along the row 13.0 us, 9.35 so, by ln(1 + id) 12.8 and 10.2, evenly spread ones 9.3 and 9.1.
        // (As they came: converted here, they were waited for before the metadata was asked for, a trip more.  Traced inside steps: 51 rows of 128,256 4.85 ->
        // 4.56 us, 569 6.14 -> 5.93, ten of a level 4.92 -> 4.61.)
        if (S <= 16) {
#pragma unroll
            for (int i = 0; i < 2; ++i) q[i] = quad_at<BF16, false>(lm, 4 * min(64 * i + lane, 8 * S - 1) + w);
        }
        if (lse_wave && S <= 16) pm = a.part_ms[g * S * 4 + min(lane, S * 4 - 1)];
        meta = row_meta<MODE>(a, g);
        if (!meta.valid) return;
    }
    const int k = meta.k;

    __shared__ __attribute__((aligned(16))) uint16_t s_key[256];
    __shared__ __attribute__((aligned(16))) u32 s_hist[256];
    __shared__ int s_hot[4 * SEL_WAVE_CAP];
    __shared__ int s_h;
    __shared__ __attribute__((aligned(16))) u64 s_fin[SEL_LIST];
    __shared__ int s_n2, s_cnt[3];

    float *tv = top_val + meta.out * out_stride;
    int32_t *ti = top_id ? top_id + meta.out * out_stride : nullptr;
    auto emit = [&](int r, u64 key) {
        float v = key_val(key);
        u32 id = key_idx(key);
        bool viable = (v > -INFINITY) && (id < (u32)V);
        put_result<MODE>(tv + r, viable ? v : -INFINITY);
        if (ti) put_result<MODE>(ti + r, viable ? (int32_t)id : -1);
    };
    // ---- the row's log-sum-exp, by wave 3 ----------------------------------------------------------------
    auto row_lse = [&]() {
        if (!lse_wave) return;
        const float cexp = 1.4426950408889634f * a.inv_t;
        float M = -INFINITY, Ssum = 0.f;
        if (SAME || S <= 16) {
            if (lane < S * 4) { M = pm.x; Ssum = pm.y; }
        } else {
            for (int i = lane; i < S * 4; i += 64) {
                const float2 p = a.part_ms[g * S * 4 + i];
                const float M2 = fmaxf(M, p.x);
                if (M2 != -INFINITY)
                    Ssum = Ssum * __builtin_amdgcn_exp2f((M - M2) * cexp) + p.y * __builtin_amdgcn_exp2f((p.x - M2) * cexp);
                M = M2;
            }
        }
        const float Mw = wave_max(M);
        float term = (Ssum > 0.f) ? Ssum * __builtin_amdgcn_exp2f((M - Mw) * cexp) : 0.f;
        term = wave_sum(term);
        if (lane == 0) put_result<MODE>(lse + meta.out, (Mw == -INFINITY) ? -INFINITY : Mw * a.inv_t + __logf(term));
    };
    // Eight elements of lane maximum i (chunk, wave, pair of lanes), those of load n / 2 and lane n % 2 of the pair: the ones that
    // reach T become candidates, room for them with one LDS add.
    const int per_log2 = nl == 4 ? 3 : nl == 2 ? 2 : 1;  // groups of eight: chunk multipliers are 1, 2 or 4
    const int shift = row_shift(a.logits, BF16, V, a.row_stride, g);
    auto octet_of = [&](int i, int n) {
        return (i >> 7) * (256 * E) + ((i >> 5) & 3) * (64 * E) + (2 * (i & 31) + (n & 1)) * 8 + (n >> 1) * 512 - shift;
    };
    auto reread = [&](int i, int n, float T) {
        float xv[8];
        const int start = load_octet<BF16, KEEP>(a, g, octet_of(i, n), xv);
        keep_hits<8>([&](int e) { return xv[e]; }, [&](int e) { return start + e; }, T, &s_n2, s_fin);
    };
    // candidate t ranks itself against all n2 keys (LDS broadcasts, eight in flight)
    auto rank_and_emit = [&](int n2) {
        if (tid < SEL_CAP && (tid & ~63) < n2) {  // the waves that hold a candidate
            const u64 mine = s_fin[tid];
            int r0 = 0, r1 = 0;
#pragma unroll 2  // more would spill
            for (int j0 = 0; j0 < n2; j0 += 8) {  // the list is zero behind its n2 keys
                u64 o[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) o[j] = s_fin[j0 + j];
#pragma unroll
                for (int j = 0; j < 8; j += 2) {
                    r0 += o[j] > mine ? 1 : 0;
                    r1 += o[j + 1] > mine ? 1 : 0;
                }
            }
            if (tid < n2 && r0 + r1 < k) emit(r0 + r1, mine);
        }
    };

    do {
        // ---- 1. thread maxima and T -------------------------------------------------------------------
        float it[8], tmax = -INFINITY;
        if (SAME || S <= 16) {
#pragma unroll
            for (int j = 0; j < 8; ++j) it[j] = 64 * (j >> 2) + lane < 8 * S ? lane_max_value<BF16>(q[j >> 2].v[j & 3]) : -INFINITY;
            tmax = spread_max(it);
        } else {
            for (int i = tid; i < n_lm; i += 256) tmax = fmaxf(tmax, lane_max_value<BF16>(lm[i]));
        }
        s_key[tid] = (uint16_t)(ord32(tmax) >> 16);
        if (tid < SEL_CAP) s_fin[tid] = 0ull;
        if (tid == 0) { s_n2 = 0; s_h = 0; }
        __syncthreads();
        const uint2 k4 = ((const uint2 *)s_key)[lane];
        const u32 ky[4] = {k4.x & 0xFFFFu, k4.x >> 16, k4.y & 0xFFFFu, k4.y >> 16};
        const u32 key0 = wave_kth<4>(ky, k);
        const float T0 = key_edge(key0);

        // ---- 2. the lanes that reach T, read again ------------------------------------------------------
        if (SAME || S <= 16) {
            // Every wave by itself: its hot lanes into a list of its own (a prefix sum over the lanes instead of an LDS
            // counter, no barrier), then (hot lane, load n) pairs over its lanes.
            u32 hot = 0;
#pragma unroll
            for (int j = 0; j < 8; ++j) hot |= (it[j] >= T0 ? 1u : 0u) << j;
            const int mine = __popc(hot), incl = wave_scan_incl_i32(mine);
            const int h = __builtin_amdgcn_readlane(incl, 63);
            if (h > SEL_WAVE_CAP) {  // ties: this bound does not cut
                if (lane == 0) s_n2 = SEL_CAP + 1;
            } else {
                int *list = s_hot + w * SEL_WAVE_CAP;
                for (int at = incl - mine; hot; hot &= hot - 1) {
                    const int j = __builtin_ctz(hot);
                    list[at++] = 4 * (4 * (64 * (j >> 2) + lane) + w) + (j & 3);
                }
                __builtin_amdgcn_wave_barrier();
                // A group to a lane, or the two neighbours of a load where there are more: k = 28 is some sixty groups to a wave.  (Each launch
                // between two events, one group to a lane after the other and lane maxima dealt so that of twelve chunks' two waves held two
                // thirds: 336 rows of 12 chunks, k = 27, 11.4 us; dealt evenly and two groups asked for at a time 10.0.  Top-k calls of 28 rows of
                // 115,042, k = 28, replayed: so 9.8 us, with neighbours in a lane 9.65, with the loop over hits 9.05.)
                const int total = h << per_log2;
                if (total <= 64) {
                    if (lane < total) reread(list[lane >> per_log2], lane & ((1 << per_log2) - 1), T0);
                } else {
                    const int pairs_log2 = per_log2 - 1, mask = (1 << pairs_log2) - 1;
                    for (int q = lane; q < total >> 1; q += 64) {
                        float x[2][8];
                        const int i = list[q >> pairs_log2], n = 2 * (q & mask);
                        const int s0 = load_octet<BF16, KEEP>(a, g, octet_of(i, n), x[0]);
                        const int s1 = load_octet<BF16, KEEP>(a, g, octet_of(i, n + 1), x[1]);
                        keep_hits<16>([&](int e) { return x[e >> 3][e & 7]; }, [&](int e) { return (e < 8 ? s0 : s1 - 8) + e; }, T0, &s_n2, s_fin);
                    }
                }
            }
            __syncthreads();
            const int n2 = s_n2;
            row_lse();
            if (n2 <= SEL_CAP) {
                rank_and_emit(n2);
                break;
            }
            __syncthreads();  // s_n2 has been read
            if (tid < SEL_CAP) s_fin[tid] = 0ull;
            if (tid == 0) s_n2 = 0;
        } else {
            row_lse();
        }

        // ---- second bound: histogram of the lane maxima >= T0; its scan from the top gives T1 ------------
        auto lane_val = [&](int i) { return lane_max_value<BF16>(lane_max_at<BF16, SAME>(lm, i)); };
        s_hist[tid] = 0u;
        __syncthreads();
        for (int i = tid; i < n_lm; i += 256) {
            const float v = lane_val(i);
            if (v >= T0) atomicAdd(&s_hist[min((ord32(v) >> 16) - key0, 255u)], 1u);
        }
        __syncthreads();
        // every wave by itself: lane L holds bins 4(63-L) .. 4(63-L)+3, so an ascending lane scan walks the
        // bins downwards; at least k lane maxima reach T0, so the scan finds its bin
        int n_hot;      // lane maxima >= T1
        float T1;
        {
            const uint4 hb = *(const uint4 *)&s_hist[4 * (63 - lane)];
            const int c4 = (int)(hb.x + hb.y + hb.z + hb.w);
            const int incl = wave_scan_incl_i32(c4);
            const u64 m = __ballot(incl >= k);
            const int ls = m ? (int)__builtin_ctzll(m) : 63;
            int acc = __builtin_amdgcn_readlane(incl - c4, ls);
            const int h3 = __builtin_amdgcn_readlane((int)hb.w, ls), h2 = __builtin_amdgcn_readlane((int)hb.z, ls),
                      h1 = __builtin_amdgcn_readlane((int)hb.y, ls), h0 = __builtin_amdgcn_readlane((int)hb.x, ls);
            int dg;
            if (acc + h3 >= k) { dg = 3; acc += h3; }
            else if (acc + h3 + h2 >= k) { dg = 2; acc += h3 + h2; }
            else if (acc + h3 + h2 + h1 >= k) { dg = 1; acc += h3 + h2 + h1; }
            else { dg = 0; acc += h3 + h2 + h1 + h0; }
            n_hot = acc;
            // the lower edge of that bin: the smallest float whose upper 16 key bits are the bin's (bin 255 also
            // holds everything farther up: its lower edge still bounds all of it)
            T1 = key_edge(key0 + (u32)(4 * (63 - ls) + dg));
        }
        if (n_hot <= SEL_CAP) {  // uniform over the workgroup
            for (int i = tid; i < n_lm; i += 256)
                if (lane_val(i) >= T1) {
                    const int at = atomicAdd(&s_h, 1);
                    if (at < SEL_CAP) s_hot[at] = i;
                }
            __syncthreads();
            for (int q = tid; q < n_hot << per_log2; q += 256) reread(s_hot[q >> per_log2], q & ((1 << per_log2) - 1), T1);
            __syncthreads();
            const int n2 = s_n2;
            if (n2 <= SEL_CAP) {
                rank_and_emit(n2);
                break;
            }
        }

        // ---- too many still: one pass over the elements of the lane maxima that reach T1 -----------------------------------------
        // Two groups of eight to a thread at a time.  What reaches the threshold goes on the list; when the list is long, the k best of it
        // stay and the k-th becomes the threshold, so that equal values later in the row no longer reach it.  -inf does not count.
        // (51 rows of 128,256 bf16 entries, k = 28: 256 to 400 neighbours raised by 20, in fewer pairs than k, 28 to 30 us, all equal 78, all -inf 59, where
        // taking the best k times from the whole row took 2,330; k = 10 23, 78 and 59 against 840; k = 1 9, 73 and 59 against 9, 101 and 95.)
        auto keep_best = [&](int n) {
            u64 key[2];
            int rank[2] = {0, 0};
#pragma unroll
            for (int h = 0; h < 2; ++h) key[h] = tid + 256 * h < SEL_LIST ? s_fin[tid + 256 * h] : 0ull;
            for (int j0 = 0; j0 < n; j0 += 4) {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const u64 o = s_fin[j0 + j];
                    rank[0] += o > key[0] ? 1 : 0;
                    rank[1] += o > key[1] ? 1 : 0;
                }
            }
            __syncthreads();
#pragma unroll
            for (int h = 0; h < 2; ++h)
                if (tid + 256 * h < SEL_LIST) s_fin[tid + 256 * h] = 0ull;
            __syncthreads();
#pragma unroll
            for (int h = 0; h < 2; ++h)
                if (tid + 256 * h < n && rank[h] < k) s_fin[rank[h]] = key[h];
            if (tid == 0) s_n2 = k;
            __syncthreads();
            return s_fin[k - 1] + 1ull;
        };
        __syncthreads();  // s_n2 has been read
        for (int i = tid; i < SEL_LIST; i += 256) s_fin[i] = 0ull;
        if (tid == 0) s_n2 = 0;
        if (tid < 3) s_cnt[tid] = 0;
        __syncthreads();
        u64 threshold = (u64)max(ord32(T1), 0x00800000u) << 32;
        const bool listed = n_hot <= SEL_CAP;
        const int pairs_log2 = per_log2 - 1, total = (listed ? n_hot : n_lm) << pairs_log2;
        int n = 0, step = 0;
        for (int q0 = 0; q0 < total; q0 += 256) {
            const int q = q0 + tid, at = min(q, total - 1) >> pairs_log2, i = listed ? s_hot[at] : at;
            float x[2][8];
            int s0 = 0, s1 = 0;
            u32 todo = 0;
            if (q < total && (listed || lane_val(i) >= T1)) {
                const int m = 2 * (q & ((1 << pairs_log2) - 1));
                s0 = load_octet<BF16, KEEP>(a, g, octet_of(i, m), x[0]);
                s1 = load_octet<BF16, KEEP>(a, g, octet_of(i, m + 1), x[1]);
#pragma unroll
                for (int e = 0; e < 16; ++e)
                    todo |= (make_key(x[e >> 3][e & 7], (u32)((e < 8 ? s0 : s1 - 8) + e)) >= threshold ? 1u : 0u) << e;
            }
            for (bool all = false; !all;) {
                // how many of the workgroup's elements wait; three counters in turn, so that one barrier does
                const int sum = wave_sum_i32(__popc(todo));
                if (lane == 0 && sum) atomicAdd(&s_cnt[step % 3], sum);
                __syncthreads();
                const int waiting = s_cnt[step % 3];
                if (tid == 0) s_cnt[(step + 2) % 3] = 0;
                ++step;
                if (waiting == 0) break;
                all = n + waiting <= SEL_LIST;  // else one of each thread's: at most 256 behind at most SEL_CAP
                for (u32 now = all ? todo : todo & (0u - todo); now; now &= now - 1) {
                    const int e = __builtin_ctz(now);
                    float v = x[0][0];
#pragma unroll
                    for (int j = 1; j < 16; ++j) v = e == j ? x[j >> 3][j & 7] : v;
                    const u64 key = make_key(v, (u32)((e < 8 ? s0 : s1 - 8) + e));
                    if (key >= threshold) s_fin[atomicAdd(&s_n2, 1)] = key;
                }
                todo &= todo - 1;
                __syncthreads();
                n = s_n2;
                if (n > SEL_CAP) {
                    threshold = keep_best(n);
                    n = k;
                }
            }
        }
        rank_and_emit(n);
        if (tid >= n && tid < k) emit(tid, make_key(-INFINITY, 0u));
    } while (false);
    level_row_end<MODE, offsetof(SelectArgs, tail)>(meta, false);
}

// ---------------------------------------------------- rows that one workgroup holds (top-k rows) --
// A row of up to 32,768 entries stays in the registers of one workgroup, 8 NL elements per thread: the thread maxima meet in LDS,
// T is found as in the selection kernel, and the elements that reach it come straight from the registers.  One launch and one
// trip to memory where the two passes take two and three.  NT threads: the fewest that hold the row with NL <= 4.
// Behind that trip the waves' instructions bound it, four waves to a SIMD with 1,024 threads: T is found by wave 0 alone while the
// others sum their exponentials (ONE), not by every wave for itself (by all, 50 rows of 8,000 / 16,000 / 32,000 bf16 entries 5.0 / 6.0 /
// 7.1 us, 2,000 of 1,000 / 8,000 / 16,000 7.3 / 13.7 / 24.9; by one 4.6 / 5.2 / 6.7 and 6.4 / 12.3 / 20.9;
// both before hits went by bits, see keep_hits).  In a small launch with a wave to a SIMD
// the barrier that this takes costs what it saves, or more (5 rows of 1,024 fp32 entries 3.53 and 3.61): there every wave finds T.
template <int MODE, int NL, bool BF16, bool VEC, int NT, bool ONE>
__global__ __launch_bounds__(NT, NL == 4 ? 4 : 8) void row_topk_kernel(RowArgs a, float *top_val, int32_t *top_id, float *lse, int out_stride, Tail<MODE> tail) {
    if (level_waits<MODE, offsetof(HeldArgs, tail)>(tail, blockIdx.x)) return;
    constexpr int E = 8 * NL, NW = NT / 64;
    const bool lse_wg = NT == 1024 && a.lse_apart && (int64_t)blockIdx.x >= a.n_rows;
    const int64_t g = lse_wg ? (int64_t)blockIdx.x - a.n_rows : (int64_t)blockIdx.x;
    const int tid = threadIdx.x, lane = lane_id(), w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int V = a.V, base = w * (64 * E) + lane * 8 - row_shift(a.logits, BF16 && VEC, a.V, a.row_stride, g);
    RawChunk<NL, BF16> raw;
    if (a.early_load) chunk_request<NL, BF16, VEC>(a, g, base, raw);
    const RowMeta meta = row_meta<MODE>(a, g);
    if (!meta.valid) return;
    const int k = meta.k;
    if (!a.early_load) chunk_request<NL, BF16, VEC>(a, g, base, raw);

    // [lane][wave].  Twice the room with 1,024 threads: the compiler places by size, and with the list of candidates in front of the keys
    // 50 rows of 16,000 bf16 entries take 4.92 us, with the keys at offset 0 4.84.
    __shared__ __attribute__((aligned(16))) uint16_t s_key[NT == 1024 ? 2 * NT : NT];
    __shared__ float2 s_ms[NW];
    __shared__ __attribute__((aligned(16))) u64 s_fin[SEL_CAP];
    __shared__ int s_n, s_cnt[3];
    __shared__ float s_T;
    if (tid < SEL_CAP) s_fin[tid] = 0ull;
    if (tid < 3) s_cnt[tid] = 0;
    if (tid == 0) s_n = 0;

    float x[E];
    chunk_finish<NL, BF16, VEC>(a, g, base, NT * E, raw, x);
    float gmx[NL], mx = -INFINITY;  // of each group of eight, and of all
#pragma unroll
    for (int n = 0; n < NL; ++n) {
        gmx[n] = x[8 * n];
#pragma unroll
        for (int e = 1; e < 8; ++e) gmx[n] = fmaxf(gmx[n], x[8 * n + e]);
        mx = fmaxf(mx, gmx[n]);
    }
    s_key[lane * NW + w] = (uint16_t)(ord32(mx) >> 16);
    const bool want_lse = a.want_lse && (NT < 1024 || lse_wg == a.lse_apart);
    auto lse_partial = [&]() {
        const float2 p = wave_lse_partial<E>(x, mx, a.inv_t);
        if (lane == 0) s_ms[w] = p;
    };
    auto row_lse = [&]() {  // by one wave, from the waves' partials
        const float cexp = 1.4426950408889634f * a.inv_t;
        const float2 p = lane < NW ? s_ms[min(lane, NW - 1)] : make_float2(-INFINITY, 0.f);
        const float M = wave_max(p.x);
        const float sum = wave_sum(p.y > 0.f ? p.y * __builtin_amdgcn_exp2f((p.x - M) * cexp) : 0.f);
        if (lane == 0) put_result<MODE>(lse + meta.out, M == -INFINITY ? -INFINITY : M * a.inv_t + __logf(sum));
    };
    do {
        if (lse_wg) {  // uniform over the workgroup
            lse_partial();
            __syncthreads();
            if (w == 0) row_lse();
            break;
        }
        if (!ONE && want_lse) lse_partial();
        __syncthreads();
        // 256 slots of NW / 4 threads each: k slots that reach T hold k elements that do
        float T;
        if (!ONE || w == 0) {
            u32 ky[4];
            uint16_t kv[NW];
            __builtin_memcpy(kv, __builtin_assume_aligned(&s_key[lane * NW], NW * 2), NW * 2);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                ky[i] = kv[i];
#pragma unroll
                for (int j = i + 4; j < NW; j += 4) ky[i] = max(ky[i], (u32)kv[j]);
            }
            T = key_edge(wave_kth<4>(ky, k));
        }
        if constexpr (ONE) {
            if (w == 0) {
                if (lane == 0) s_T = T;
            } else if (want_lse) {
                lse_partial();
            }
            __syncthreads();
            T = s_T;
            if (w == 0 && want_lse) lse_partial();
        }
        auto id_of = [&](int n, int e) {
            const int id0 = base + n * 512;
            return (VEC ? group_start(V, id0) : id0) + e;
        };
        auto push = [&](bool in, int j) {
            if (__builtin_amdgcn_ballot_w64(in)) {  // uniform: few elements get here
                if (in) {
                    const int at = atomicAdd(&s_n, 1);
                    if (at < SEL_CAP) s_fin[at] = make_key(x[j], (u32)id_of(j >> 3, j & 7));
                }
            }
        };
        const float T1 = fmaxf(T, -__FLT_MAX__);  // -inf does not count
#pragma unroll
        for (int n = 0; n < NL; ++n)
            if (__builtin_amdgcn_ballot_w64(gmx[n] >= T1))
                keep_hits<8>([&](int e) { return x[8 * n + e]; }, [&](int e) { return id_of(n, e); }, T1, &s_n, s_fin);
        __syncthreads();
        int n = s_n;
        if (n > SEL_CAP) {
            // Clusters or equal values: the exact k-th key by bisection, then, of the elements equal to it, the exact last id.
            int step = 0;
            auto total = [&](int own) {  // sum over the workgroup; three counters in turn, so that one barrier does
                const int sum = wave_sum_i32(own);
                if (lane == 0) atomicAdd(&s_cnt[step % 3], sum);
                __syncthreads();
                const int v = s_cnt[step % 3];
                if (tid == 0) s_cnt[(step + 2) % 3] = 0;
                ++step;
                return v;
            };
            u32 lo = ord32(T), hi = 0xFFFFFFFFu;  // at least k keys reach lo, none lies above hi
            if (lo <= 0x007FFFFFu) lo = 0x00800000u;  // -inf does not count
            int c = n;
            while (hi > lo && c > k) {
                const u32 mid = lo + ((hi - lo) >> 1) + 1u;
                int own = 0;
#pragma unroll
                for (int j = 0; j < E; ++j) own += ord32(x[j]) >= mid ? 1 : 0;
                const int m = total(own);
                if (m >= k) { lo = mid; c = m; }
                else hi = mid - 1u;
            }
            int id_hi = 0x7FFFFFFF;  // of the elements equal to lo: those up to this id
            if (c > k) {
                int own = 0;
#pragma unroll
                for (int j = 0; j < E; ++j) own += ord32(x[j]) > lo ? 1 : 0;
                const int need = k - total(own);
                int id_lo = 0;  // the smallest id with `need` of them at or below it
                id_hi = V - 1;
                while (id_hi > id_lo) {
                    const int mid = (id_lo + id_hi) >> 1;
                    own = 0;
#pragma unroll
                    for (int j = 0; j < E; ++j) own += ord32(x[j]) == lo && id_of(j >> 3, j & 7) <= mid ? 1 : 0;
                    if (total(own) >= need) id_hi = mid;
                    else id_lo = mid + 1;
                }
            }
            __syncthreads();  // the count has been read
            if (tid < SEL_CAP) s_fin[tid] = 0ull;
            if (tid == 0) s_n = 0;
            __syncthreads();
#pragma unroll
            for (int j = 0; j < E; ++j) push(ord32(x[j]) > lo || (ord32(x[j]) == lo && id_of(j >> 3, j & 7) <= id_hi), j);
            __syncthreads();
            n = s_n;
        }
        float *tv = top_val + meta.out * out_stride;
        int32_t *ti = top_id + meta.out * out_stride;
        if (tid < SEL_CAP && (tid & ~63) < n) {  // candidate tid ranks itself against all (zeros behind the n keys)
            const u64 mine = s_fin[tid];
            int rank = 0;
            for (int j0 = 0; j0 < n; j0 += 8) {
                u64 o[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) o[j] = s_fin[j0 + j];
#pragma unroll
                for (int j = 0; j < 8; ++j) rank += o[j] > mine ? 1 : 0;
            }
            if (tid < n && rank < k) {
                put_result<MODE>(tv + rank, key_val(mine));
                put_result<MODE>(ti + rank, (int32_t)key_idx(mine));
            }
        }
        if (w == NW - 1) {
            if (lane >= n && lane < k) {  // fewer than k viable entries
                put_result<MODE>(tv + lane, -INFINITY);
                put_result<MODE>(ti + lane, (int32_t)-1);
            }
            if (want_lse) row_lse();
        }
    } while (false);
    level_row_end<MODE, offsetof(HeldArgs, tail)>(meta, lse_wg);
}

// ------------------------------------------------- bf16 rows of large launches (top-k rows) --
// Where rows come by the thousand the kernel above is bound by vector instructions, most of them not spent on the elements: every wave of a
// row looks its row up, reduces, and takes part in the search, and lanes past the row's end work like the others (2,040 entries, k = 24:
// 1,240 instructions a row, 250 of them on elements; 16,000 in 1,024 threads 6,900).  Here a lane holds 32 or 64 elements, as they came from
// memory: unpacked once for the maxima and once more for the exponentials, they leave room for eight waves to a SIMD.  The slots are the groups of
// eight at the same place of all waves, four to a lane, so that a row of one wave needs no exchange; the groups that reach T are listed, and their
// elements read again, one to a lane, in place of a search of every lane's elements; keys are 32 bits, value and place.  Groups past the end are passed
// over.  Draft rows, us, before | now: 10,309 rows of 2,040 entries, k = 24, 29 | 19; 5,408 of 9,411 67 | 31, of 16,000 69 | 34, of 32,000 114 | 62 (two passes
// before; the bytes are 55 us); calls of 2,600 rows of 16,000, k = 16, 26.4 | 18.5, of 25,000 37 | 28.
#define MANY_LIST (SEL_CAP * 4)  // bytes of the list of candidates
#define MANY_WAVE (64 * 16)      // of a wave: its slots' keys, later its groups that reach T
template <int MODE, int NG>
__global__ __launch_bounds__(1024, 8) void row_many_kernel(RowArgs a, float *top_val, int32_t *top_id, float *lse, int out_stride) {
    static_assert(NG == 4 || NG == 8, "groups of eight to a lane");
    constexpr int WAVE = 512 * NG;  // entries of a wave
    const int64_t g = blockIdx.x;
    const int tid = threadIdx.x, lane = lane_id(), w = __builtin_amdgcn_readfirstlane(tid >> 6), NW = blockDim.x >> 6;
    const int V = a.V, wave0 = w * WAVE - row_shift(a.logits, true, a.V, a.row_stride, g), base = wave0 + lane * 8;
    RawChunk<NG, true> raw;
    const bool early = MODE == ROWS_UNIFORM || a.early_load;
    if (early) chunk_request<NG, true, true>(a, g, base, raw);
    const RowMeta meta = row_meta<MODE>(a, g);
    if (!meta.valid) return;
    const int k = meta.k;
    if (!early) chunk_request<NG, true, true>(a, g, base, raw);

    extern __shared__ __attribute__((aligned(16))) unsigned char s_dyn[];
    __shared__ float2 s_ms[16];
    __shared__ int s_n, s_cnt[3];
    __shared__ float s_T;
    u32 *s_list = (u32 *)s_dyn;
    uint2 *s_key = (uint2 *)(s_dyn + MANY_LIST + w * MANY_WAVE);  // this wave's
    auto clear = [&]() {
        ((uint4 *)s_list)[lane] = make_uint4(0, 0, 0, 0);
        if (lane == 0) s_n = 0;
    };
    if (w == 0) {
        clear();
        if (lane < 3) s_cnt[lane] = 0;
    }
    auto key_of = [](float v, int id) { return (ord32(v) & 0xFFFF0000u) | (0xFFFFu - (u32)id); };
    auto unpack = [&](int n, float (&x)[8]) {
        const u32 rr[4] = {raw.r[n].x, raw.r[n].y, raw.r[n].z, raw.r[n].w};
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            x[2 * p] = __uint_as_float(rr[p] << 16);
            x[2 * p + 1] = __uint_as_float(rr[p] & 0xFFFF0000u);
        }
        if (n == 0 && wave0 < 0) x[0] = lane == 0 ? -INFINITY : x[0];
        if (wave0 + (n + 1) * 512 > V) {  // uniform: reaches past the row's end
            const int id0 = base + n * 512, first = id0 - group_start(V, id0);
#pragma unroll
            for (int e = 0; e < 8; ++e) x[e] = e >= first ? x[e] : -INFINITY;
        }
    };
    float gmx[NG];
#pragma unroll
    for (int n = 0; n < NG; ++n) {
        gmx[n] = -INFINITY;
        if (n && wave0 + n * 512 >= V) continue;  // uniform
        float x[8];
        unpack(n, x);
        float m = -INFINITY;
        asm("v_max3_f32 %0, %1, %2, %0\n\tv_max3_f32 %0, %3, %4, %0\n\tv_max3_f32 %0, %5, %6, %0\n\tv_max3_f32 %0, %7, %8, %0"
            : "+v"(m) : "v"(x[0]), "v"(x[1]), "v"(x[2]), "v"(x[3]), "v"(x[4]), "v"(x[5]), "v"(x[6]), "v"(x[7]));
        gmx[n] = m;
    }
    float sl[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        sl[i] = gmx[i];
        if constexpr (NG == 8) asm("v_max_f32 %0, %1, %0" : "+v"(sl[i]) : "v"(gmx[i + 4]));
    }
    // the upper halves as keys: x ^ (negative ? 0xFFFF : 0x8000), two at a time.  (-0 below +0: T is only a bound.)
    auto pair_key = [](float lo, float hi) {
        typedef short s2 __attribute__((ext_vector_type(2)));
        const u32 p = __builtin_amdgcn_perm(__float_as_uint(hi), __float_as_uint(lo), 0x07060302u);
        const u32 sign = __builtin_bit_cast(u32, __builtin_bit_cast(s2, p) >> (short)15);
        return p ^ (sign | 0x80008000u);
    };
    const uint2 own = make_uint2(pair_key(sl[0], sl[1]), pair_key(sl[2], sl[3]));
    if (NW > 1 && w) s_key[lane] = own;
    if (a.want_lse) {
        const float cexp = 1.4426950408889634f * a.inv_t;
        float mx = sl[0];
        asm("v_max3_f32 %0, %1, %2, %0\n\tv_max_f32 %0, %3, %0" : "+v"(mx) : "v"(sl[1]), "v"(sl[2]), "v"(sl[3]));
        const float M = wave_max(mx), nm = M == -INFINITY ? 0.f : -M * cexp;
#pragma unroll
        for (int i = 0; i < NG; ++i)  // keep the compiler from holding the elements
            asm volatile("" : "+v"(raw.r[i].x), "+v"(raw.r[i].y), "+v"(raw.r[i].z), "+v"(raw.r[i].w));
        float s = 0.f;
#pragma unroll
        for (int n = 0; n < NG; ++n) {
            if (n && wave0 + n * 512 >= V) continue;
            float x[8];
            unpack(n, x);
#pragma unroll
            for (int e = 0; e < 8; ++e) s += __builtin_amdgcn_exp2f(fmaf(x[e], cexp, nm));
        }
        s = wave_sum(s > 0.f ? s : 0.f);
        if (NW == 1) {
            if (lane == 0) lse[meta.out] = M == -INFINITY ? -INFINITY : M * a.inv_t + __logf(s);
        } else if (lane == 0) s_ms[w] = make_float2(M, s);
    }
    __syncthreads();
    if (w == 0) {  // the row's 256 slots: group (n, lane) of all waves
        typedef unsigned short us4 __attribute__((ext_vector_type(4)));
        us4 m = __builtin_bit_cast(us4, own);
#pragma unroll 4
        for (int j = 1; j < NW; ++j) {
            const uint2 o = *(const uint2 *)((const unsigned char *)s_key + j * MANY_WAVE + lane * 8);
            m = __builtin_elementwise_max(m, __builtin_bit_cast(us4, o));
        }
        const u32 ky[4] = {m.x, m.y, m.z, m.w};
        const u32 t = wave_kth<4>(ky, k);
        if (lane == 0) s_T = key_edge(t);
    }
    __syncthreads();
    const float T = s_T;
    const float T1 = fmaxf(T, -__FLT_MAX__);  // -inf does not count
    uint16_t *s_hot = (uint16_t *)s_key;  // the groups that reach T (in the place of the slots, which have been read)
    int hot = 0;
#pragma unroll
    for (int n = 0; n < NG; ++n) {
        const bool in = gmx[n] >= T1;
        const u64 m = __builtin_amdgcn_ballot_w64(in);
        if (m) {
            if (in) s_hot[hot + lanes_below(m)] = (uint16_t)(64 * n + lane);
            hot += __popcll(m);
        }
    }
    // their entries again, one to a lane
    const uint16_t *row = (const uint16_t *)a.logits + g * a.row_stride;
    auto entry = [&](int id) { return bf16_bits_to_float(row[id]); };
    __builtin_amdgcn_wave_barrier();
    for (int q0 = 0; q0 < 8 * hot; q0 += 64) {  // uniform
        const int q = s_hot[min((q0 + lane) >> 3, hot - 1)];
        const int id0 = wave0 + q * 8, id = group_start(V, id0) + (lane & 7);
        const float v = entry(id);
        const bool in = v >= T1 && id >= max(id0, 0) && q0 + lane < 8 * hot;
        const u64 m = __builtin_amdgcn_ballot_w64(in);
        if (m) {
            int at = 0;
            if (lane == 0) at = atomicAdd(&s_n, (int)__popcll(m));
            at = __builtin_amdgcn_readfirstlane(at);
            at += lanes_below(m);
            if (in && at < SEL_CAP) s_list[at] = key_of(v, id);
        }
    }
    __syncthreads();
    int n = s_n;
    if (n > SEL_CAP) {
        // Clusters or equal values: the k-th value by bisection, then, of the entries equal to it, the last id.  Over the registers, filled again here (held
        // until now they would cost waves), with the 16 bits that a value has as keys, two to a word.  Calls of equal rows, every step over the row in memory
        // with 32-bit keys | so: 2,000 of 8,000 entries 563 | 73 us, 5,000 of 4,001 1,081 | 97, 300 of 16,384 260 | 42, 200 of 30,000 248 | 43 (by the kernel that holds
        // rows 121, 133, 66; in two passes 68).
        typedef unsigned short us2 __attribute__((ext_vector_type(2)));
        typedef short s2 __attribute__((ext_vector_type(2)));
        int first0 = base;
        asm volatile("" : "+v"(first0));  // the addresses are worked out again
        chunk_request<NG, true, true>(a, g, first0, raw);
        auto word = [&](int i, int p) -> u32 & { return p == 0 ? raw.r[i].x : p == 1 ? raw.r[i].y : p == 2 ? raw.r[i].z : raw.r[i].w; };
#pragma unroll
        for (int i = 0; i < NG; ++i) {
            const int id0 = first0 + i * 512, first = id0 < 0 ? 1 : id0 - group_start(V, id0);  // elements before it are not the group's
#pragma unroll
            for (int p = 0; p < 4; ++p) {
                u32 &x = word(i, p);
                const u32 sign = __builtin_bit_cast(u32, __builtin_bit_cast(s2, x) >> (short)15);
                const us2 y = __builtin_bit_cast(us2, x ^ (sign | 0x80008000u)), minus_zero = {0x7FFF, 0x7FFF};
                const u32 key = __builtin_bit_cast(u32, y + us2{1, 1} - __builtin_elementwise_min(y ^ minus_zero, us2{1, 1}));  // -0 as +0
                x = key & ((2 * p >= first ? 0xFFFFu : 0u) | (2 * p + 1 >= first ? 0xFFFF0000u : 0u));
                asm volatile("" : "+v"(x));
            }
        }
        int step = 0;
        auto total = [&](int own_n) {  // sum over the workgroup; three counters in turn, so that one barrier does
            const int sum = wave_sum_i32(own_n);
            if (lane == 0) atomicAdd(&s_cnt[step % 3], sum);
            __syncthreads();
            const int v = s_cnt[step % 3];
            if (tid == 0) s_cnt[(step + 2) % 3] = 0;
            ++step;
            return v;
        };
        auto reach = [&](u32 key) {  // this lane's entries that reach a key of 1 and more
            const unsigned short below = (unsigned short)(key - 1u);
            us2 sum = {0, 0};
#pragma unroll
            for (int i = 0; i < 4 * NG; ++i)
                sum += __builtin_elementwise_min(__builtin_elementwise_sub_sat(__builtin_bit_cast(us2, word(i / 4, i % 4)), us2{below, below}), us2{1, 1});
            return (int)sum.x + (int)sum.y;
        };
        u32 lo = ord32(T) >> 16, hi = 0xFFFFu;  // at least k keys reach lo, none lies above hi
        if (lo <= 0x007Fu) lo = 0x0080u;  // -inf does not count
        int c = n;
        while (hi > lo && c > k) {
            const u32 mid = lo + ((hi - lo) >> 1) + 1u;
            const int m = total(reach(mid));
            if (m >= k) { lo = mid; c = m; }
            else hi = mid - 1u;
        }
        u64 above = 0, equal = 0;  // bit 8 i + e: element e of group i
#pragma unroll
        for (int i = 0; i < 4 * NG; ++i) {
            const u32 y = word(i / 4, i % 4), y0 = y & 0xFFFFu, y1 = y >> 16;
            above |= (u64)((y0 > lo ? 1u : 0u) | (y1 > lo ? 2u : 0u)) << (2 * i);
            equal |= (u64)((y0 == lo ? 1u : 0u) | (y1 == lo ? 2u : 0u)) << (2 * i);
            asm volatile("" : "+v"(above), "+v"(equal));
        }
        if (c > k) {
            const int need = k - total(__popcll(above));
            auto up_to = [&](int id) {  // of those equal to lo
                u64 m = 0;
#pragma unroll
                for (int i = 0; i < NG; ++i) {
                    const int last = min(id - group_start(V, first0 + i * 512), 7);
                    m |= (u64)(last < 0 ? 0u : (2u << last) - 1u) << (8 * i);
                }
                return equal & m;
            };
            int id_lo = 0, id_hi = V - 1;  // the smallest id with `need` of them at or below it
            while (id_hi > id_lo) {
                const int mid = (id_lo + id_hi) >> 1;
                if (total(__popcll(up_to(mid))) >= need) id_hi = mid;
                else id_lo = mid + 1;
            }
            equal = up_to(id_hi);
        }
        __syncthreads();  // the count has been read
        if (w == 0) clear();
        __syncthreads();
        for (u64 left = above | equal; left; left &= left - 1) {  // k of the row's
            const int i = (int)__builtin_ctzll(left), id = group_start(V, first0 + (i >> 3) * 512) + (i & 7);
            const int at = atomicAdd(&s_n, 1);
            if (at < SEL_CAP) s_list[at] = key_of(entry(id), id);
        }
        __syncthreads();
        n = s_n;
    }
    float *tv = top_val + meta.out * out_stride;
    int32_t *ti = top_id ? top_id + meta.out * out_stride : nullptr;
    for (int c = tid; c < SEL_CAP && (c & ~63) < n; c += blockDim.x) {  // candidate c ranks itself against all (zeros behind the n keys)
        const u32 mine = s_list[c];
        int rank = 0;
#pragma unroll 1
        for (int j0 = 0; j0 < n; j0 += 8) {
            u32 o[8];
            __builtin_memcpy(o, __builtin_assume_aligned(&s_list[j0], 16), sizeof(o));
#pragma unroll
            for (int j = 0; j < 8; ++j) rank += o[j] > mine ? 1 : 0;
        }
        if (c < n && rank < k) {
            tv[rank] = unord32(mine & 0x80000000u ? mine & 0xFFFF0000u : mine | 0xFFFFu);
            if (ti) ti[rank] = (int32_t)(0xFFFFu - (mine & 0xFFFFu));
        }
    }
    if (w == NW - 1) {
        if (lane >= n && lane < k) {  // fewer than k viable entries
            tv[lane] = -INFINITY;
            if (ti) ti[lane] = -1;
        }
        if (NW > 1 && a.want_lse) {
            const float cexp = 1.4426950408889634f * a.inv_t;
            const float2 p = lane < NW ? s_ms[min(lane, NW - 1)] : make_float2(-INFINITY, 0.f);
            const float M = wave_max(p.x);
            const float sum = wave_sum(p.y > 0.f ? p.y * __builtin_amdgcn_exp2f((p.x - M) * cexp) : 0.f);
            if (lane == 0) lse[meta.out] = M == -INFINITY ? -INFINITY : M * a.inv_t + __logf(sum);
        }
    }
}

// ------------------------------------------------------------- arg max kernel (target rows) --
// k = 1: every workgroup leaves the best (value, id) key of its chunk, and optionally the
// (max, sum) pair of row/T; the acceptance kernel merges the chunks of a row.
// Small vocabularies in large launches are bound by vector instructions: rows of one chunk have only the waves that they fill, groups that end inside the
// row are not masked, the first of the best entries is looked for in the one group that has it, and the exponentials refer to the wave's maximum.
// (7,686 rows of 1,728 entries, greedy: 266 instructions in each of four waves -> 125 in one, 17.2 -> 8.9 us; with sums 22.7 -> 8.3; 3,200 rows of 128,256 with sums, which were bound so too, 145 -> 126.)
template <int NL, bool BF16, bool VEC>
__global__ __launch_bounds__(256) void row_argmax_kernel(RowArgs a) {
    constexpr int E = 8 * NL;
    const int64_t g = (int64_t)blockIdx.z * gridDim.y + blockIdx.y;
    const int c = blockIdx.x;
    const int lane = lane_id(), w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), NW = blockDim.x >> 6;
    __shared__ u64 s_wout[4];
    __shared__ float s_m[4], s_s[4];

    const int wave0 = c * (256 * E) + w * (64 * E) - row_shift(a.logits, BF16 && VEC, a.V, a.row_stride, g), base = wave0 + lane * 8;
    if (g >= a.n_rows) return;
    // early: the row's elements are on their way while the (dependent, scalar) reads of its metadata are waited for
    float x[E];
    RawChunk<NL, BF16> raw;
    if (a.early_load) chunk_request<NL, BF16, VEC>(a, g, base, raw);
    const RowMeta meta = row_meta<ROWS_TARGET>(a, g);
    if (!meta.valid) return;
    u64 key = 0ull;
    float T = -INFINITY, s = 0.f;
    if (wave0 < a.V) {  // uniform
        if (!a.early_load) chunk_request<NL, BF16, VEC>(a, g, base, raw);
        chunk_finish<NL, BF16, VEC>(a, g, base, (c + 1) * (256 * E), raw, x);
        float gmx[NL], mx = -INFINITY;
#pragma unroll
        for (int n = 0; n < NL; ++n) {
            gmx[n] = x[8 * n];
#pragma unroll
            for (int e = 1; e < 8; ++e) gmx[n] = fmaxf(gmx[n], x[8 * n + e]);
            mx = fmaxf(mx, gmx[n]);
        }
        T = wave_max(mx);
        if (a.want_lse) {
            const float cexp = 1.4426950408889634f * a.inv_t, nm = T == -INFINITY ? 0.f : -T * cexp;
#pragma unroll
            for (int j = 0; j < E; ++j) s += __builtin_amdgcn_exp2f(fmaf(x[j], cexp, nm));
            s = wave_sum(s > 0.f ? s : 0.f);
        }
        // the wave's best key: the first group that holds its maximum, the first lane of that, the first such element
#pragma unroll
        for (int n = 0; n < NL; ++n) {
            const u64 m = __builtin_amdgcn_ballot_w64(gmx[n] == T);
            if (m && key == 0ull) {  // uniform
                const int first = (int)__builtin_ctzll(m), id0 = wave0 + n * 512 + 8 * first;
                int at = 0;
#pragma unroll
                for (int e = 7; e >= 0; --e) at = x[8 * n + e] == T ? e : at;
                // (a row without a finite entry: its first, not the one before it)
                key = make_key(T, (u32)max((VEC ? group_start(a.V, id0) : id0) + __builtin_amdgcn_readlane(at, first), 0));
            }
        }
    }
    if (lane == 0) {
        s_wout[w] = key;
        s_m[w] = T;
        s_s[w] = s;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        const int64_t slot = g * gridDim.x + c;
        for (int q = 1; q < NW; ++q) key = s_wout[q] > key ? s_wout[q] : key;
        a.part_keys[slot] = key;
        if (a.want_lse) {
            const float cexp = 1.4426950408889634f * a.inv_t;
            float M = T, S = s;
            for (int q = 1; q < NW; ++q) {
                const float M2 = fmaxf(M, s_m[q]);
                if (M2 != -INFINITY)
                    S = S * __builtin_amdgcn_exp2f((M - M2) * cexp) + s_s[q] * __builtin_amdgcn_exp2f((s_m[q] - M2) * cexp);
                M = M2;
            }
            a.part_ms[slot] = make_float2(M, S);
        }
    }
}

// ------------------------------------------------------------------------ launchers ------

int rows_chunks_per_row(int V, int nl) { return (V + 256 * 8 * nl - 1) / (256 * 8 * nl); }

// Chunk multiplier for the top-k rows: the smallest that keeps a row within 16 chunks (so that
// the selection kernel holds its lane maxima in registers); 4 beyond that.
int rows_topk_nl(int V) {
    for (int nl = 1; nl <= 4; nl <<= 1)
        if (rows_chunks_per_row(V, nl) <= 16) return nl;
    return 4;
}

// Chunk multiplier for the arg max rows: few, fat chunks (the acceptance kernel merges the
// chunks of a row, and measured kernel time does not depend on the chunk size), but at least
// about one workgroup per compute unit.
int rows_pick_nl(int64_t n_rows, int V) {
    for (int nl = 4; nl > 1; nl >>= 1)
        if (n_rows * rows_chunks_per_row(V, nl) >= 256) return nl;
    return 1;
}

// (chunks, rows) as a launch grid: rows beyond what grid y holds continue in z; the last z-slab may
// overhang, its workgroups leave at once
static dim3 rows_grid(int chunks, int64_t n_rows) {
    const int64_t ny = n_rows < 65535 ? n_rows : 65535;
    return dim3((unsigned)chunks, (unsigned)ny, (unsigned)((n_rows + ny - 1) / ny));
}

// f(MODE, BF16) with both as compile-time constants
template <typename F>
static void by_mode_and_type(const RowArgs &a, F f) {
    using std::integral_constant;
    auto typed = [&](auto mode) {
        if (a.dtype == DT_BF16) f(mode, integral_constant<bool, true>());
        else f(mode, integral_constant<bool, false>());
    };
    if (a.mode == ROWS_DRAFT) typed(integral_constant<int, ROWS_DRAFT>());
    else if (a.mode == ROWS_LEVEL) typed(integral_constant<int, ROWS_LEVEL>());
    else typed(integral_constant<int, ROWS_UNIFORM>());
}
// the same for launches that may choose a level's nodes
template <typename F>
static void by_mode_and_type(const RowArgs &a, const TreeArgs *tree, F f) {
    using std::integral_constant;
    if (!tree) by_mode_and_type(a, f);
    else if (a.dtype == DT_BF16) f(integral_constant<int, ROWS_CHOOSE>(), integral_constant<bool, true>());
    else f(integral_constant<int, ROWS_CHOOSE>(), integral_constant<bool, false>());
}

// Launches of at most this many workgroups are latency bound: their rows are read before they are known
// to be live.  Larger ones are bandwidth bound, and the bytes of a dead row would cost time: a launch sized for the limits
// that a policy may set on the device is mostly dead rows (two sequences, 450 rows of 128,256 for the widest action:
// 21.8 us when all were read, 8-13 us when a row's liveness is looked up first).
static const int64_t EARLY_LOAD_WGS = 2048;
// Launches of more chunks than this take two to a workgroup if the rows are looked up or the chunks are short: the trip in front of the loads
// (whose row is it, is it live) is made half as often, and the second chunk's elements are on their way under the exponentials of the first.
// Draft rows, one | two to a workgroup, traced: of 128,256 entries, 17,900 chunks 46.7 | 48.0 us, 25,800 70 | 69, 33,500 94 | 88, 60,600 174 | 163; of 128,257 57.5 | 57.5,
// 82 | 82, 111 | 106, 204 | 187; of 90,001, 17,700 chunks 57 | 59, 24,200 80 | 80, 42,000 141 | 137; of 50,257, 18,200 38 | 34, 24,400 50 | 46, 61,300 125 | 111.  Below: 156 MB (9,700
// chunks) 30.1 | 30.6, 87 MB (5,400) 18.4 | 19.8.  Rows that need no look-up gain only where a workgroup's life is short, chunks of 2,048: calls of 1,900 rows of 18,944
// 29.9 | 24.7 us, of 22,976 32.8 | 26.5, of 30,976 41.0 | 31.9, of 31,001 41.8 | 33.8; of 40,001 (chunks of 4,096) 36.9 | 39.0, of 128,256 (8,192), 17,000 chunks 53.2 | 54.9, of 119,331
// 53.8 | 60.6.
static const int64_t PAIR_CHUNKS = 16384;
// How many workgroups a row has in launches bound by bandwidth.  They go to the eight XCDs in turn: with sixteen, or eight of two chunks, a
// row's last, shorter one falls to the same XCD in every row.  One more, which leaves at once, deals every chunk to every XCD.  Sixteen | seventeen, calls
// of 1,000 rows of 128,257 bf16 entries 48.8 | 47.8 us, of 128,256 49.2 | 48.4, of 125,001 50.9 | 47.2, of 65,001 30.1 | 29.2; eight | nine, draft rows of 61
// sequences of 125,001 504 | 489, of 119,331 489 | 467.  With ten, twelve or fourteen it gains nothing, and it costs where the
// last one is whole (65,536 27.7 | 28.1, 98,304 in twelve 36.6 | 37.6).
static int workgroups_per_row(const RowArgs &a, int64_t S, int nl, int cpw) {
    const int wgs = (int)((S + cpw - 1) / cpw);
    const bool last_is_whole = a.V % (256 * 8 * nl * cpw) == 0 && a.row_stride % 2 == 0;
    return (wgs % 8 == 0 || (cpw == 2 && wgs % 2 == 0)) && !last_is_whole ? wgs + 1 : wgs;
}

// top-k rows, pass 1: lane maxima and (max, sum) partials
static hipError_t launch_stream(const RowArgs &a_in, int64_t n_rows, int nl, hipStream_t st) {
    RowArgs a = a_in;
    const int64_t S = rows_chunks_per_row(a.V, nl);
    a.early_load = n_rows * S <= EARLY_LOAD_WGS;
    const int kid = a.mode == ROWS_DRAFT ? KID_ROWS_DRAFT : KID_ROWS_UNIFORM;
    a.n_rows = n_rows;
    using std::integral_constant;
    auto go = [&](auto mode, auto bf16) {
        constexpr int MODE = decltype(mode)::value;
        constexpr bool BF = decltype(bf16)::value;
        auto launch = [&](auto nl_c) {
            constexpr int NL = decltype(nl_c)::value;
            auto with = [&](auto kernel, int cpw) {
                const int wgs = a.early_load ? (int)S : workgroups_per_row(a, S, nl, cpw);
                launch_kernel(kid, st, kernel, rows_grid(wgs, n_rows), dim3(256), 0, a, (int)S);
            };
            if constexpr (MODE != ROWS_UNIFORM || NL == 1)
                if (n_rows * S > PAIR_CHUNKS) return with(row_stream_kernel<MODE, NL, BF, 2>, 2);
            with(row_stream_kernel<MODE, NL, BF, 1>, 1);
        };
        if (nl == 4) launch(integral_constant<int, 4>());
        else if (nl == 2) launch(integral_constant<int, 2>());
        else launch(integral_constant<int, 1>());
    };
    by_mode_and_type(a, go);
    return hipGetLastError();
}

// top-k rows, pass 2: selection on the lane maxima
// What a launch of a level's rows needs to choose the level's nodes, with `first_wg` workgroups of rows and its words at `words`.
template <int MODE>
static Tail<MODE> level_tail(const RowArgs &a, const TreeArgs *tree, void *words, unsigned first_wg) {
    if constexpr (MODE == ROWS_CHOOSE) {
        LevelTail h = {};
        h.t = *tree;
        h.words = (u64 *)words;
        h.tag = launch_tag();
        h.first_wg = (int)first_wg;
        h.rows = a.rows_per_seq;
        h.lse_apart = a.lse_apart;
        return h;
    } else {
        return NoTail();
    }
}

static hipError_t launch_select(const RowArgs &a, int64_t n_rows, int nl, float *top_val, int32_t *top_id, float *lse,
                                int out_stride, hipStream_t st) {
    const int S = rows_chunks_per_row(a.V, nl);
    by_mode_and_type(a, [&](auto mode, auto bf16) {
        launch_kernel(KID_ROWS_MERGE, st, row_select_kernel<decltype(mode)::value, decltype(bf16)::value, 0>, dim3((unsigned)n_rows),
                      dim3(256), 0, a, nl, S, top_val, top_id, lse, out_stride, 0ull, level_tail<decltype(mode)::value>(a, nullptr, nullptr, 0));
    });
    return hipGetLastError();
}

// Both passes in one launch: while all its workgroups are on the chip at once, and in bf16 up to some 13 MB of entries.  Beyond, the stream is bound by bandwidth and
// the exponentials, and what the launch saves goes into more workgroups to a compute unit; fp32 rows, without the exponentials' weight, gain
// throughout, since a row is selected while others still stream.  Calls, k = 12, two launches | one: bf16 of 128,256 entries 10 rows 7.8 | 6.7 us, 28 8.1 | 7.2, 44
// 8.4 | 8.1, 64 9.0 | 9.5, 80 9.6 | 10.1; of 90,001 48 rows 9.0 | 7.2, 72 9.1 | 8.7, 100 9.6 | 9.6; of 50,001 28 8.0 | 6.6, 64 8.0 | 7.1, 112 9.0 | 8.3, 144 9.2 | 9.5; of
// 36,000 112 8.9 | 7.5; fp32 of 128,256 28 rows 9.2 | 8.8, 64 11.9 | 11.5, 120 17.1 | 15.6; of 50,001 61 9.15 | 8.19, 144 12.0 | 11.5; of 20,001 112 8.9 | 7.6.
// Beside a busy stream the workgroups that wait have no place, or others have none because of them, and a launch less is still worth more: 51 bf16 rows of 128,256, two launches | one, beside
// a product of 4,096 cubed 160 | 119 us a call, beside an elementwise pass over 512 MB 27.3 | 22.6, to which a call adds 3.7 | 4.6; 61 fp32 rows of 50,001 172 | 116, 29.6 | 22.0, 3.7 | 4.3.
#define PASS_WGS 2048
#define PASS_ENTRIES ((int64_t)13 << 19)
static bool takes_pass(const RowArgs &a, int64_t n_rows, int nl) {
    const int64_t S = rows_chunks_per_row(a.V, nl);
    return S <= 16 && (n_rows + 7) / 8 * 8 * (S + 1) <= PASS_WGS && (a.dtype == DT_F32 || n_rows * a.V <= PASS_ENTRIES);
}
static hipError_t launch_pass(const RowArgs &a_in, int64_t n_rows, int nl, float *top_val, int32_t *top_id, float *lse, int out_stride, hipStream_t st, const TreeArgs *tree) {
    RowArgs a = a_in;
    const int S = rows_chunks_per_row(a.V, nl);
    a.early_load = 1;
    a.n_rows = n_rows;
    const int kid = a.mode == ROWS_DRAFT ? KID_ROWS_DRAFT : KID_ROWS_UNIFORM;
    by_mode_and_type(a, tree, [&](auto mode, auto bf16) {
        constexpr int MODE = decltype(mode)::value;
        constexpr bool BF = decltype(bf16)::value;
        auto go = [&](auto kernel) {
            const unsigned x = 8 * (S + 1), y = (unsigned)((n_rows + 7) / 8), more = tree ? (unsigned)((tree->batch + x - 1) / x) : 0;
            // a level's words lie behind those of the rows (row_select_kernel)
            const auto tail = level_tail<MODE>(a, tree, (char *)a.lane_max + n_rows * (S * 512 + (LINE_WORDS + ROW_MARKS) * 8), x * y);
            launch_kernel(kid, st, kernel, dim3(x, y + more), dim3(256), 0, a, nl, S, top_val, top_id, lse, out_stride, launch_tag(), tail);
        };
        if (nl == 4) go(row_select_kernel<MODE, BF, 4>);
        else if (nl == 2) go(row_select_kernel<MODE, BF, 2>);
        else go(row_select_kernel<MODE, BF, 1>);
    });
    return hipGetLastError();
}

// Rows that a workgroup holds.
static int held_threads(int V) { return V <= 256 * 16 ? 256 : V <= 512 * 16 ? 512 : 1024; }
// While every row of 1,024 threads leaves another compute unit idle, its exponentials are summed there, by a workgroup of its own that
// reads the row as well: 16 waves sum 32,000 exponentials in 0.6 us (50 rows of 32,000 bf16 entries 6.7 -> 6.1 us, 120 rows 7.1 -> 6.2,
// 16,000 entries 5.2 -> 4.95 and 5.4 -> 5.05; 50 rows of 8,000, 512 threads, 4.65 -> 4.80).
// With another stream busy the other half of the chip is not idle, and neither side gains: the same calls beside a bf16 product of 4,096
// cubed, without | with, 20.2 | 19.7, 20.4 | 19.7, 19.0 | 18.8, 18.9 | 18.7 us, the product 114.3 | 115.0, 112.9 | 113.8, 113.6 | 113.2, 111.5 | 110.9; beside
// an elementwise pass over 512 MB 15.4 | 15.2, 16.2 | 15.9, 13.0 | 13.7, 14.1 | 14.4, the pass 87.1 | 87.4, 87.3 | 88.1, 86.9 | 87.0, 87.2 | 87.7.
#define APART_ROWS 128
#define SMALL_ROWS 512  // most rows of a launch that leaves a SIMD a wave or two of 256-thread workgroups
static hipError_t launch_held(const RowArgs &a_in, int64_t n_rows, float *top_val, int32_t *top_id, float *lse, int out_stride,
                              hipStream_t st, const TreeArgs *tree) {
    RowArgs a = a_in;
    a.early_load = n_rows * rows_chunks_per_row(a.V, 4) <= EARLY_LOAD_WGS;
    a.n_rows = n_rows;
    a.lse_apart = a.want_lse && n_rows <= APART_ROWS && held_threads(a.V) == 1024;
    const int64_t wgs = a.lse_apart ? 2 * n_rows : n_rows;
    const int kid = a.mode == ROWS_DRAFT ? KID_ROWS_DRAFT : KID_ROWS_UNIFORM;
    by_mode_and_type(a, tree, [&](auto mode, auto bf16) {
        constexpr int MODE = decltype(mode)::value;
        constexpr bool BF = decltype(bf16)::value;
        auto go = [&](auto kernel, int nt) {
            launch_kernel(kid, st, kernel, dim3((unsigned)(wgs + (tree ? tree->batch : 0))), dim3(nt), 0, a, top_val, top_id, lse, out_stride,
                          level_tail<MODE>(a, tree, a.lane_max, (unsigned)wgs));
        };
        const bool one = n_rows > SMALL_ROWS;
        if (a.V < 8) go(row_topk_kernel<MODE, 1, BF, false, 256, false>, 256);  // no 16-byte group: element loads
        else if (a.V <= 256 * 8 && one) go(row_topk_kernel<MODE, 1, BF, true, 256, true>, 256);
        else if (a.V <= 256 * 8) go(row_topk_kernel<MODE, 1, BF, true, 256, false>, 256);
        else if (a.V <= 256 * 16 && one) go(row_topk_kernel<MODE, 2, BF, true, 256, true>, 256);
        else if (a.V <= 256 * 16) go(row_topk_kernel<MODE, 2, BF, true, 256, false>, 256);
        else if (a.V <= 512 * 16) go(row_topk_kernel<MODE, 2, BF, true, 512, true>, 512);
        else if (!BF || a.V <= 1024 * 16) go(row_topk_kernel<MODE, 2, BF, true, 1024, true>, 1024);
        else if constexpr (BF) go(row_topk_kernel<MODE, 4, BF, true, 1024, true>, 1024);
    });
    return hipGetLastError();
}

// bf16 rows that the kernel for large launches takes, in waves of 512 ng entries.  Four groups of eight to a lane while all rows then fit on the chip at
// once, else eight: calls of 1,000 rows of 16,000 entries, four | eight, 9.2 | 9.7 us, of 25,000 16.6 | 12.8; 2,600 of 4,096 8.1 | 8.7, of 9,411 15.9 | 16.4, of 32,000 37 | 33;
// draft rows, 776 of 16,000 10.6 | 10.3, 5,408 44 | 34.
static int many_waves(int V, int ng) { return (V + 512 * ng - 1) / (512 * ng); }
static int many_groups(int64_t n_rows, int V) { return V <= 2048 || n_rows <= 256 * (32 / many_waves(V, 4)) ? 4 : 8; }
static hipError_t launch_many(const RowArgs &a_in, int64_t n_rows, float *top_val, int32_t *top_id, float *lse, int out_stride, hipStream_t st) {
    RowArgs a = a_in;
    a.early_load = n_rows * rows_chunks_per_row(a.V, 4) <= EARLY_LOAD_WGS;
    a.n_rows = n_rows;
    const int kid = a.mode == ROWS_DRAFT ? KID_ROWS_DRAFT : KID_ROWS_UNIFORM, ng = many_groups(n_rows, a.V), waves = many_waves(a.V, ng);
    by_mode_and_type(a, [&](auto mode, auto bf16) {
        if constexpr (decltype(bf16)::value)
            launch_kernel(kid, st, ng == 4 ? row_many_kernel<decltype(mode)::value, 4> : row_many_kernel<decltype(mode)::value, 8>, dim3((unsigned)n_rows),
                          dim3(64 * waves), MANY_LIST + waves * MANY_WAVE, a, top_val, top_id, lse, out_stride);
    });
    return hipGetLastError();
}

// Top-k rows.  a: its scratch (lane_max, part_ms) is that of rows_topk_nl(V) chunks.
// One workgroup holds rows of up to 16,384 entries: 51 rows of 1,000 / 4,000 / 8,192 / 16,000 bf16 entries 7.4 / 8.0 / 7.8 / 8.4
// us in two passes, 4.6 / 5.4 / 5.4 / 6.7 held; 2,000 rows 13.8 / 16.2 / 19.9 / 29, held 8.1 / 10.1 / 15.4 / 29.  Up to twice as long
// ones in bf16 while every row has a compute unit to itself (32,000 entries: 51 rows 8.7 -> 8.1, 200 rows 11.6 -> 8.9, but
// 600 rows 18.5 -> 21.1: the two passes spread a row over more of the chip; fp32 51 rows 9.2 -> 10.3).
// A workgroup takes a row in grid x, where a launch may have 2^32 - 1 threads: more rows of 512 or 1,024 threads than that go
// through the two passes, whose 256 threads a row reach further.  (Rows on in grid y, and a test for its overhang, cost every
// launch 0.3 us.)
#define HELD_V_MAX 16384
#define HELD_ROWS_MAX 256  // of 2 HELD_V_MAX entries
// bf16 rows of up to 32,768 entries, from 128 to 2,048 rows on by their length: row_many_kernel.  Calls, k = 16, held or in two passes | many: 1,600 rows of 2,048
// entries 6.1 | 6.1 us, 2,600 7.8 | 6.8; 800 of 4,096 5.6 | 5.6, 2,000 7.9 | 6.8; 400 of 8,192 5.1 | 5.5, 640 6.1 | 5.9; 256 of 16,000 5.3 | 5.3, 330 6.7 | 6.4, of 9,411 7.3 | 6.4; 128 of
// 32,000 5.9 | 6.2, 200 7.0 | 6.5, of 25,000 6.7 | 5.7.  In fp32, whose elements take the registers of half the waves, it gains nothing (2,600 rows of 4,000 11.2 | 12.1).
// Rows beyond 16,384 entries that need no look-up only while all are on the chip at once: past that the two passes gain least from it
// (1,990 rows of 26,944 25 | 23, 2,600 of 20,000 31 | 24), and their time grows more slowly with the number of rows, which the tests hold them to.
#define MANY_V_MAX 32768
static bool takes_many(const RowArgs &a, int64_t n_rows) {
    if (a.dtype != DT_BF16 || a.V < 8 || a.V > MANY_V_MAX || n_rows * 64 * many_waves(a.V, 4) > 0xFFFFFFFFll) return false;
    if (a.mode == ROWS_UNIFORM && a.V > HELD_V_MAX && n_rows > 256 * (32 / many_waves(a.V, 8))) return false;
    int64_t room = 2048;  // entries, a power of two
    while (room < a.V) room *= 2;
    return n_rows * room > ((int64_t)1 << 22);
}
hipError_t rows_launch_topk(const RowArgs &a, int64_t n_rows, float *top_val, int32_t *top_id, float *lse, int out_stride,
                            hipStream_t st, const TreeArgs *tree, bool *to_expand) {
    if (n_rows <= 0) return hipSuccess;
    // A level's nodes are chosen by one wave (level_expand): the first level's, or those of up to NARROW_K parents.
    if (tree && a.level > 1 && a.rows_per_seq > NARROW_K) tree = nullptr;
    if (takes_many(a, n_rows)) return launch_many(a, n_rows, top_val, top_id, lse, out_stride, st);
    const int nt = held_threads(a.V);
    if ((a.V <= HELD_V_MAX && (nt == 256 || n_rows * nt <= 0xFFFFFFFFll)) ||
        (a.V <= 2 * HELD_V_MAX && a.dtype == DT_BF16 && n_rows <= HELD_ROWS_MAX)) {
        if (tree && (n_rows + tree->batch) * nt > 0xFFFFFFFFll) tree = nullptr;  // no room for the workgroups that wait
        if (tree) *to_expand = false;
        return launch_held(a, n_rows, top_val, top_id, lse, out_stride, st, tree);
    }
    // Chunks of 4,096 entries, for launches that have too few of 8,192, cost larger ones 3 to 18 %: calls of 1,000 rows of 50,257 entries, 4,096 | 8,192, 25.3 | 23.4 us,
    // of 65,536 29.3 | 26.9, 200 of 36,000 9.0 | 9.1, fp32 500 of 40,001 21.9 | 21.9, 1,000 38.8 | 36.6; draft rows 776 of 64,960 31.8 | 26.0, 10,309 293 | 264.  (The scratch
    // was sized for the smaller ones.)
    int nl = rows_topk_nl(a.V);
    if (nl == 2 && n_rows * rows_chunks_per_row(a.V, 4) > EARLY_LOAD_WGS) nl = 4;
    if (takes_pass(a, n_rows, nl)) {
        if (tree) *to_expand = false;
        return launch_pass(a, n_rows, nl, top_val, top_id, lse, out_stride, st, tree);
    }
    const hipError_t e = launch_stream(a, n_rows, nl, st);
    return e != hipSuccess ? e : launch_select(a, n_rows, nl, top_val, top_id, lse, out_stride, st);
}

// arg max rows (target logits)
hipError_t rows_launch_argmax(const RowArgs &a_in, int64_t n_rows, int nl, hipStream_t st) {
    if (n_rows <= 0) return hipSuccess;
    RowArgs a = a_in;
    a.early_load = n_rows * rows_chunks_per_row(a.V, nl) <= EARLY_LOAD_WGS;
    a.n_rows = n_rows;
    const dim3 grid = rows_grid(rows_chunks_per_row(a.V, nl), n_rows);
    auto go = [&](auto bf16) {
        constexpr bool BF = decltype(bf16)::value;
        // a row of one chunk: the waves that it fills
        const int threads = a.V <= 3 * 512 * nl ? 64 * ((a.V + 512 * nl - 1) / (512 * nl)) : 256;
        auto launch = [&](auto kernel) { launch_kernel(KID_ROWS_TARGET, st, kernel, grid, dim3(threads), 0, a); };
        if (a.V < 8) launch(row_argmax_kernel<1, BF, false>);  // no 16-byte group: element loads
        else if (nl == 4) launch(row_argmax_kernel<4, BF, true>);
        else if (nl == 2) launch(row_argmax_kernel<2, BF, true>);
        else launch(row_argmax_kernel<1, BF, true>);
    };
    if (a.dtype == DT_BF16) go(std::integral_constant<bool, true>());
    else go(std::integral_constant<bool, false>());
    return hipGetLastError();
}

}  // namespace dt
