// Tree-masked attention of the tree tokens against [KV prefix | tree keys].
//
// bf16 path (MFMA).  Query rows of one kv head are the (node, group head) pairs, packed as
// the N dimension of S^T = K Q^T so that every lane owns ONE query column of the 32x32
// score block: the softmax statistics are lane-local plus one exchange with lane^32.  The
// probabilities come out of the S^T accumulator in exactly the register layout the B
// operand of O^T = V^T P^T wants, so P never leaves registers; 128-wide heads round it to bf16 for that
// product, 64-wide heads keep it whole.  K and V tiles are staged in LDS
// row-major; the V operand comes from the transposing LDS read.  The keys of a sequence may be split
// across workgroups, which leave partial max / sum / O, when a batch offers too few
// (sequence, kv head, row tile) items to fill the chip (small batches, merged by those that wait for the others) or items of
// different lengths (large batches, merged by the workgroup that comes last, or by all that stayed to see it come).
// The ancestor bitset is applied only to key blocks that contain tree keys.
//
// fp32 heads of 64 and 128: sixteen lanes to a key (attn_f32_kernel); every other head size and type, and bf16 caches whose
// strides are not multiples of 16 bytes: attn_simple_kernel.  Plain ALU kernels, one workgroup per (node, head).

#include <algorithm>
#include <type_traits>

#include "common.hpp"
#include "kernels.hpp"

namespace dt {


typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
// Global-address-space views: pointers fetched from memory (the per-sequence prefix pointers)
// would otherwise be generic, and generic loads also count against the LDS wait counter.
typedef const __bf16 __attribute__((address_space(1))) *gbf16p;
typedef const bf16x8 __attribute__((address_space(1))) *gbf16x8p;
__device__ __forceinline__ bf16x8 gload8(gbf16p p) { return *(gbf16x8p)p; }
typedef const char __attribute__((address_space(1))) *gbytep;

// LDS transpose read of gfx950 (ds_read_b64_tr_b16).  Within each group of 16 lanes, lane p
// supplies the address of 4 consecutive 16-bit values; with X the concatenation of the 16
// quadruples in lane order, lane i receives X[i], X[16+i], X[32+i], X[48+i].  Pointing lane
// p = 4j+q at row j, columns 4q..4q+3 of a row-major tile therefore hands lane i the column
// i of rows 0..3: a 4x16 -> 16x4 transpose, which is what a K-contiguous MFMA operand needs
// from a matrix stored with the other index contiguous.
typedef short s16x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ bf16x4 lds_read_tr4(const __bf16 *p) {
    s16x4 v = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3))) *)p);
    return __builtin_bit_cast(bf16x4, v);
}

// Four global_load_lds_dwordx4, 64 bytes apart in memory and STEP bytes apart in LDS, with the address split into a
// wave-uniform base (scalar registers) and a 32-bit per-lane byte offset, the LDS destination (wave-uniform, the lanes' 16 bytes
// follow each other) in M0: no vector arithmetic per load, and no 64-bit per-lane pointers to keep and advance.  The
// instruction adds its offset to the LDS address as well, so M0 holds the destination less that.
// The hardware asks for five wait states between a vector instruction that writes a scalar register (readfirstlane, the
// reload of a spilled one) and a memory instruction that reads it, and the compiler does not see the memory instructions in
// here: the group keeps that distance itself in front of its first load, and is one statement, so that nothing can be put
// between the loads.
template <int STEP>
__device__ __forceinline__ void load4_to_lds16(const void __attribute__((address_space(1))) *base, u32 lane_off, u32 lds_addr) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 3\n\tglobal_load_lds_dwordx4 %0, %1\n\t"
                 "s_add_u32 m0, m0, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 offset:64\n\t"
                 "s_add_u32 m0, m0, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 offset:128\n\t"
                 "s_add_u32 m0, m0, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 offset:192" ::"v"(lane_off),
                 "s"(base), "s"(lds_addr), "n"(STEP - 64)
                 : "memory", "m0", "scc");
}
// a pointer that is the same in every lane, moved to scalar registers where the compiler has not seen that
__device__ __forceinline__ gbf16p uniform_ptr(gbf16p p) {
    const u64 v = (u64)(uintptr_t)p;
    const u32 lo = __builtin_amdgcn_readfirstlane((u32)v), hi = __builtin_amdgcn_readfirstlane((u32)(v >> 32));
    return (gbf16p)(uintptr_t)(((u64)hi << 32) | lo);
}
// The same two LDS reads as bare instructions, for loops that keep the wait counters by hand: the
// compiler neither counts them nor guards them with a wait for outstanding global_load_lds traffic
// (it cannot tell a read of one tile from a read of the tile still being filled).  lds_wait<N> lets at
// most N later LDS operations stay outstanding and ties the wait to the register it releases.
template <int OFF>
__device__ __forceinline__ bf16x8 lds_load128_at(u32 addr) {
    bf16x8 v;
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFF));
    return v;
}
template <int N>
__device__ __forceinline__ void lds_wait2(bf16x8 &a, bf16x8 &b) {
    asm volatile("s_waitcnt lgkmcnt(%2)" : "+v"(a), "+v"(b) : "n"(N));
}
template <int N>
__device__ __forceinline__ void lds_wait4(bf16x4 &a, bf16x4 &b, bf16x4 &c, bf16x4 &d) {
    asm volatile("s_waitcnt lgkmcnt(%4)" : "+v"(a), "+v"(b), "+v"(c), "+v"(d) : "n"(N));
}
template <int OFF>
__device__ __forceinline__ bf16x4 lds_load_tr4(u32 addr) {
    bf16x4 v;
    asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFF));
    return v;
}
template <int N>
__device__ __forceinline__ void lds_wait(bf16x8 &v) {
    asm volatile("s_waitcnt lgkmcnt(%1)" : "+v"(v) : "n"(N));
}

// The value of the partner lane (lane ^ 32) next to the own one, without a trip through the LDS
// crossbar: v_permlane32_swap exchanges the upper half of one register with the lower half of another,
// so from two copies of x every lane ends up holding {x[lane], x[lane ^ 32]} in the two registers (in
// either order; layout checked on the device).  Written as an instruction: the compiler's builtin
// returned the same element for both results when they met in one expression.  The waits around it
// cover the vector-write -> swap-read distance the hardware asks for.
__device__ __forceinline__ void half_swap(float x, float &a, float &b) {
    a = x;
    b = x;
    asm volatile("s_nop 1\n\tv_permlane32_swap_b32 %0, %1\n\ts_nop 1" : "+v"(a), "+v"(b));
}
__device__ __forceinline__ float half_swap_max(float x) {
    float a, b;
    half_swap(x, a, b);
    return fmaxf(a, b);
}
__device__ __forceinline__ float half_swap_sum(float x) {
    float a, b;
    half_swap(x, a, b);
    return a + b;
}

#define ATT_KB 32           // keys per block
#define ATT_ROWS_PER_WAVE 32
#define ATT_WAVES 4
#define ATT_MTILE (ATT_ROWS_PER_WAVE * ATT_WAVES)
#define NEAR_LIMIT 0x1p8f     // sums of probabilities that cannot hurt, and
#define REF_LIMIT 0x1p64f     // that send a key range of the large-batch kernel through a second time
#define LAZY_LOG2 8.0f        // how far (in powers of two) a probability may exceed 1 before a reference that moves does

// 32-bit visibility window of one query over keys t0 .. t0+31, where off = t0 - L (uniform): the
// prefix keys (negative positions) are visible, tree key j is visible iff bit j of the node's
// ancestor set is set (bits at and past the node count are 0, which also hides the padding
// keys past the end of the sequence).
__device__ __forceinline__ u32 vis_window(int off, u64 mask0, u64 mask1) {
    if (off <= -32) return ~0u;
    if (off < 0) return ((u32)mask0 << (-off)) | ((1u << (-off)) - 1u);
    if (off >= 128) return 0u;
    const u64 lo = off < 64 ? mask0 : mask1, hi = off < 64 ? mask1 : 0ull;
    const int sh = off & 63;
    return (u32)((lo >> sh) | (sh ? hi << (64 - sh) : 0ull));
}

// ------------------------------------------------------------------- large-batch kernel -----
// One workgroup = 128 query rows of one (sequence, kv head) (wave w: rows 32w .. 32w+31) times
// one contiguous range of 64-key blocks.  The four waves share each K/V block through LDS, so a
// block crosses the L2 -> LDS path once per 128 rows.  The blocks are loaded straight into LDS
// (global_load_lds_dwordx4: a wave's 64 x 16 B land contiguously, lane after lane), double
// buffered with one barrier per block: the loads of block i+1 are in flight while block i is
// multiplied, and cost neither registers nor LDS-write instructions.
//
// A tile is four sub-tiles of 64 keys x 64 bytes (32 columns), row after row.  A 1 KB load is sixteen keys of one sub-tile;
// the operand reads find everything but a lane's own row at immediate offsets (two address registers for K, one for V), and
// no read has a bank conflict:
//   K: chunk c (16 bytes) of row r sits at position c ^ (r / 4 % 4) of its 64 bytes (the permutation is applied on the
//      global side), so that the A-operand read of S^T = K Q^T, the same chunk of 16 consecutive rows, takes 16 different
//      16-byte slots of 256 bytes;
//   V: the transposing read takes 4 rows x 64 B per 32 lanes, 256 consecutive bytes.
#define TILE_KEYS 64
#define TILE_BYTES (TILE_KEYS * 256)     // one K or V tile
#define SUB_BYTES (TILE_KEYS * 64)       // a quarter of its columns
#define TILE_LDS_BYTES(NS) (2 * (NS) * TILE_BYTES)  // NS K tiles, then NS V tiles
typedef char __attribute__((address_space(3))) *ldsp;

// One key range of a (sequence, row tile): the `me`-th of `parts`.  With more than one, the workgroups leave partials
// (unnormalised O, running max, sum) and the one that comes last puts them together; partial i lies at index
// 2 (slot + i step), the first at 2 slot + 1.  Values are 64-bit words in the order in which a row block's lanes hold them,
// since the same lanes of another workgroup read them.
struct TileParts {
    int parts, me;
    int slot, step;
    u64 *o;       // [.., D / 4, 256]
    u64 *ml;      // [.., 128]
    u64 *count;   // partials left so far, in the low 16 bits, if the others are `tag`; anything else counts as none
    u64 tag;
};
// One more partial is there: true for the last of `parts`, which also clears the count.  `old`: what the count was a moment ago (the
// reader of the count before the partials, handed on: a trip less, 12 shapes of 80 to 144 tiles 38.5 -> 38.3 us on average).
__device__ __forceinline__ bool arrive_last(u64 *count, u64 tag, int parts, u64 old) {
    for (;;) {  // a failed exchange means that another of the parts came: at most `parts` turns
        const int n = (old & ~(u64)0xffff) == tag ? (int)(old & 0xffff) + 1 : 1;
        if (__hip_atomic_compare_exchange_strong(count, &old, n == parts ? 0 : tag | n, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_AGENT))
            return n == parts;
    }
}

// Many parts: a batch of few kv heads with one sequence far longer than the others.  Counted in one after the other on one
// word, and read one after the other by one workgroup at the rate that a compute unit is fed, they took 1 to 1.6 us each.  More
// than SERIAL_PARTS leave marks on words of their own instead, and their workgroups stay to see the last mark (for at most
// STAY_TICKS: nothing depends on who is still there); whoever sees all of them takes slices of the tile, one after the other,
// until there are none left.  Two kv heads, one sequence of 32,768 keys among 63 of 256 (170 parts): 208 us before, 40 so; seven
// query heads to each of two kv heads, one of 16,384 among 15 of 128 (52 parts): 130 and 42; eight kv heads, one of 8,192
// among 15 of 256 (18 parts): 55 and 46.  (Marks, but all parts read by the last to come: 132, 78, 54; a merge kernel: 53,
// 46, 51.)
// Fewer parts are read faster by one workgroup that has the last of them in registers than left, marked and shared: 16 ragged
// sequences in up to 3 parts 155 us a step, 177 shared; 8 of up to 5, four layers, 497 and 507 to 522.
#define SERIAL_PARTS 8
#define MERGE_SLICES 16
struct SharedMerge {
    TileParts pt;
    u64 *marks;   // [slots, 2] `tag` once a partial has been left, anything else before
    bool stay;    // nothing else waits for this workgroup
    __bf16 *out;  // of (sequence, kv head): row node * Hq + group head
    int m0, rb, M, G, Hq;
    float c;
};
__device__ __forceinline__ int64_t part_at(const TileParts &pt, int i) { return 2 * (int64_t)(pt.slot + i * pt.step) + (i == 0); }
// The next slice to take.  Part 1 lies inside its sequence, so nothing in this launch leaves a mark as a first part there.
__device__ __forceinline__ u64 *next_slice(const SharedMerge &s) { return s.marks + 2 * (int64_t)(s.pt.slot + s.pt.step) + 1; }
// One wave: marks its part and looks for the others'.  True if all of them are there and the merge has not been taken entirely.
__device__ __forceinline__ bool mark_and_stay(const SharedMerge &s, int lane) {
    if (s.pt.me == 0) {  // before the mark: whoever sees all marks sees a number of this launch
        if (lane == 0) put_agent(next_slice(s), 0);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }
    if (lane == 0) put_agent(s.marks + part_at(s.pt, s.pt.me), s.pt.tag);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // of the last two parts at least one sees the other's mark
    const u32 t0 = (u32)__builtin_amdgcn_s_memrealtime();
    for (;;) {
        bool all = true, mine = false;
        for (int i0 = 0; i0 < s.pt.parts; i0 += 64) {
            const int i = min(i0 + lane, s.pt.parts - 1);
            const bool there = get_agent(s.marks + part_at(s.pt, i)) == s.pt.tag;
            all = all && __builtin_amdgcn_ballot_w64(!there) == 0ull;
            mine = mine || __builtin_amdgcn_ballot_w64(there && i == s.pt.me) != 0ull;
        }
        if (all) return true;
        if (!mine || !s.stay || (u32)__builtin_amdgcn_s_memrealtime() - t0 > STAY_TICKS(t0)) return false;
        __builtin_amdgcn_s_sleep(8);
    }
}
template <int D>
__device__ __forceinline__ void merge_shared(SharedMerge s) {
    __shared__ int s_word[2];
    int tid = threadIdx.x, one = 1;
    asm volatile("" : "+v"(tid), "+v"(one), "+s"(s.pt.tag));  // what follows from these stays out of the key loop's registers
    const int lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6), half = lane >> 5;
    const int row = 32 * s.rb + (lane & 31), mq = s.m0 + row;
    if (w == 0) {
        const bool help = mark_and_stay(s, lane);
        if (lane == 0) s_word[0] = help;
    }
    __syncthreads();
    if (!s_word[0]) return;
    asm volatile("" ::: "memory");
    constexpr int E = D / 4 / MERGE_SLICES, U = 16;  // 64-bit words of a slice per thread, parts in flight
    int slice;
    for (;;) {
        if (tid == 0) s_word[1] = (int)__hip_atomic_fetch_add(next_slice(s), one, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
        slice = s_word[1];
        __syncthreads();
        if (slice >= MERGE_SLICES) break;    // uniform
        if (s.m0 + 32 * s.rb >= s.M) continue;  // a wave without rows
        float m = -INFINITY, l = 0.f;
        float2 acc[E];
#pragma unroll
        for (int e = 0; e < E; ++e) acc[e] = make_float2(0.f, 0.f);
        for (int i0 = 0; i0 < s.pt.parts; i0 += U) {
            u64 mlw[U], ow[U][E];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int64_t at = part_at(s.pt, min(i0 + u, s.pt.parts - 1));
                mlw[u] = get_agent(s.pt.ml + at * ATT_MTILE + row);
#pragma unroll
                for (int e = 0; e < E; ++e) ow[u][e] = get_agent(s.pt.o + at * (D / 4 * 256) + (slice * E + e) * 256 + 64 * s.rb + lane);
            }
            __builtin_amdgcn_sched_barrier(0);  // all requests before the first use
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const float2 ml = __builtin_bit_cast(float2, mlw[u]);
                if (i0 + u < s.pt.parts && ml.y > 0.f) {  // a range whose keys were all hidden weighs nothing
                    const float m2 = fmaxf(m, ml.x);
                    const float keep = __builtin_amdgcn_exp2f((m - m2) * s.c);  // first partial: exp2(-inf) = 0
                    const float wgt = __builtin_amdgcn_exp2f((ml.x - m2) * s.c);
#pragma unroll
                    for (int e = 0; e < E; ++e) {
                        const float2 v = __builtin_bit_cast(float2, ow[u][e]);
                        acc[e].x = acc[e].x * keep + v.x * wgt;
                        acc[e].y = acc[e].y * keep + v.y * wgt;
                    }
                    l = l * keep + ml.y * wgt;
                    m = m2;
                }
            }
        }
        if (mq >= s.M) continue;
        const float inv = l > 0.f ? 1.0f / l : 0.f;
        __bf16 *op = s.out + ((int64_t)(mq / s.G) * s.Hq + mq % s.G) * D + 4 * half;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int i = 2 * (slice * E + e);  // element i of the lane's: column 32 (i / 16) + 8 (i % 16 / 4) + 4 half + i % 4
            const bf16x2 v = {(__bf16)(acc[e].x * inv), (__bf16)(acc[e].y * inv)};
            *(bf16x2 *)(op + 32 * (i >> 4) + 8 * ((i & 15) >> 2) + (i & 3)) = v;
        }
    }
    // The first to find nothing left takes the marks away: a replayed graph has the same tag.
    if (slice == MERGE_SLICES)
        for (int i = tid; i < s.pt.parts; i += 256) put_agent(s.marks + part_at(s.pt, i), 0);
}

// The words of a sequence, the same in all lanes.
struct SeqWords {
    int N, L;
    u64 kpre, vpre;  // of the caches, as addresses
};
// x / G for 0 <= x < 2^31: with 2^shift < G <= 2^(shift + 1) and magic = 2^(32 + shift) / G rounded up, x * magic / 2^(32 + shift) is too large by
// x (magic G / 2^(32 + shift) - 1) / G < 1 / G, which no quotient notices.  (A remainder that puts a coarser one right cost 64-wide heads 0.05 us of 7.7.)
struct GroupDiv {
    int G;
    u32 magic, shift;
    __device__ __forceinline__ int div(int x) const { return G == 1 ? x : (int)(__umulhi((u32)x, magic) >> shift); }
};
static GroupDiv group_div(int G) {
    u32 shift = 0;
    while ((2ll << shift) < G) ++shift;
    return {G, G == 1 ? 0u : (u32)((((u64)1 << (32 + shift)) + G - 1) / G), shift};
}

// Rows m0 .. m0+127 of (sequence b, kv head h) against key blocks kb0 .. kb1-1 of that sequence.
// Called by all 256 threads of the workgroup; ends behind a barrier, so calls can follow each other.
//
// NS tiles of K and of V are in LDS.  Two (64 KB) where two workgroups share a compute unit and each covers the other's waits.  Four where a
// workgroup is alone: with two its loads are asked for one block before they are read, and a block of a cache that comes from memory then takes
// 1.3 us in place of 0.7; with four they are asked for three blocks before.  us per layer, two | four: 16 layers of 8 sequences of 1,100 keys (8B
// shape) 32.6 | 27.5, 32 of 400 18.1 | 17.1; one layer, its cache in the last level: 200 keys 13.0 | 13.6, 1,100 25.2 | 26.6 (the counted waits and
// stages found at run time).
template <int D, int NS>
__device__ __forceinline__ bool tile_segment(const AttnArgs &a, const GroupDiv &gd, const SeqWords &sq, unsigned char *s_dyn, int h,
                                             int b, int m0, int rot, int kb0, int kb1, const TileParts &pt, int slots, bool stay, bool exact) {
    static_assert(D == 128 && (NS == 2 || NS == 4), "shape");
    constexpr int KSTEPS = D / 16, DBLK = D / 32;
    int G = gd.G, N = sq.N, L = sq.L;
    asm volatile("" : "+s"(G), "+s"(N), "+s"(L));
    const int M = N * G;
    const int Tk = L + N;

    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid), "+s"(h), "+s"(b), "+s"(m0));  // what follows from these is worked out here, not kept in registers from segment to segment
    const int lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = lane >> 5, col = lane & 31;
    // Wave w works on rows 32 rb .. of the tile.  Waves past the last row only help with the loads; `rot` spreads them over
    // the SIMDs, so that two half-filled tiles on one compute unit do not leave the same ones idle.
    const int rb = (w + rot) & 3;
    const bool active = m0 + 32 * rb < M;
    const int mq = m0 + 32 * rb + col;
    const bool qvalid = mq < M;
    const int mr = qvalid ? mq : 0;  // rows past M read node 0: unused
    const int node = gd.div(mr), hq = h * G + (mr - node * G);

    f32x16 oacc[DBLK];
#pragma unroll
    for (int db = 0; db < DBLK; ++db)
#pragma unroll
        for (int i = 0; i < 16; ++i) oacc[db][i] = 0.f;
    float m_run = -INFINITY, l_run = 0.f;
    const float c = a.scale * 1.4426950408889634f;

    const gbf16p kpre = uniform_ptr((gbf16p)(uintptr_t)sq.kpre + (int64_t)h * a.kv_stride_head);
    const gbf16p vpre = uniform_ptr((gbf16p)(uintptr_t)sq.vpre + (int64_t)h * a.kv_stride_head);
    const gbf16p ktree = (gbf16p)a.k_tree + ((int64_t)b * a.TT_cap * a.Hkv + h) * D;
    const gbf16p vtree = (gbf16p)a.v_tree + ((int64_t)b * a.TT_cap * a.Hkv + h) * D;
    const int64_t stok = a.kv_stride_tok, stree = (int64_t)a.Hkv * D;
    // Loading role of a thread: load i takes 64-byte column group i of keys 16 w .. 16 w + 15 of the block, lane l key
    // 16 w + l / 4 and chunk position l % 4 of it: consecutive lanes fill consecutive 16 bytes of the sub-tile.
    const int krow = 16 * w + (lane >> 2), vchunk = lane & 3, kchunk = vchunk ^ ((lane >> 4) & 3);
    // inside the prefix: a lane's byte offset from the block's first row (the same for the four loads, 64 bytes apart)
    const u32 koffp = (u32)(krow * stok + 8 * kchunk) * 2u, voffp = (u32)(krow * stok + 8 * vchunk) * 2u;
    const bool small_stride = (int64_t)TILE_KEYS * stok * 2 < ((int64_t)1 << 31);

    // Every load is unconditional.  Keys past the end are read from the last valid row; their
    // scores are masked to -inf below, so their probabilities are exactly 0 and the duplicated V
    // rows contribute nothing.
    auto fetch = [&](auto inside, int kb, u32 tile, gbf16p pre, gbf16p tree, u32 poff, int chunk) __attribute__((always_inline)) {
        const ldsp dst = (ldsp)s_dyn + tile + w * 1024;
        if (decltype(inside)::value || (small_stride && kb * TILE_KEYS + TILE_KEYS <= L)) {  // block inside the prefix (uniform test)
            const u32 dl = (u32)(uintptr_t)dst;
            const gbytep base = (gbytep)(pre + (int64_t)kb * TILE_KEYS * stok);
            load4_to_lds16<SUB_BYTES>(base, poff, dl);
        } else {                                                 // block touching the tree keys or the end
            const int t = min(kb * TILE_KEYS + krow, Tk - 1);
            const gbf16p src = (t < L ? pre + (int64_t)t * stok : tree + (int64_t)(t - L) * stree) + 8 * chunk;
#pragma unroll
            for (int i = 0; i < 4; ++i)
                __builtin_amdgcn_global_load_lds((gbytep)(src + 32 * i), dst + i * SUB_BYTES, 16, 0, 0);
        }
    };
    const std::false_type anywhere;
    auto stage_of = [&](int kb) { return (u32)((kb - kb0) & (NS - 1)); };
    auto fetch_k = [&](auto inside, int kb, u32 stage) { fetch(inside, kb, stage * TILE_BYTES, kpre, ktree, koffp, kchunk); };
    auto fetch_v = [&](auto inside, int kb, u32 stage) { fetch(inside, kb, (NS + stage) * TILE_BYTES, vpre, vtree, voffp, vchunk); };

    // Operand read addresses; everything but the lane's own part is an immediate offset.
    // K, A operand of S^T: lane (col, half), k-step s reads chunk 2s + half of row 32 j + col: sub-tile s / 2, chunk
    // 2 (s % 2) + half of it, at position chunk ^ (row / 4 % 4).
    const u32 lds0 = (u32)(uintptr_t)(ldsp)s_dyn;
    const u32 koff[2] = {lds0 + (u32)(col * 64 + ((half ^ ((col >> 2) & 3)) << 4)),
                         lds0 + (u32)(col * 64 + (((2 + half) ^ ((col >> 2) & 3)) << 4))};
    // V, A operand of O^T = V^T P^T through the transposing read.  Lane (column d = 32 db + col,
    // half) needs, for e = 0..7, V[key 16 st + 8 (e/4) + 4 half + e%4][d]: two reads of 4 keys.  In
    // a 16-lane group lane p16 = 4 r0 + q points at key r0 of the quadruple, columns 4q .. 4q+3 of
    // the group's 16 columns: sub-tile db, byte 32 grp + 8 q of the row (grp = second 16-lane group of the half).
    const int p16 = lane & 15, r0 = p16 >> 2, q4 = p16 & 3, grp = (lane >> 4) & 1;
    const u32 voff = lds0 + NS * TILE_BYTES + (u32)((4 * half + r0) * 64 + 32 * grp + 8 * q4);

    bf16x8 qreg[KSTEPS];
    // Scores of a block: two 32x32 blocks, S[j] = keys 32 j .. 32 j + 31.
    struct Scores { f32x16 v[2]; };
    f32x16 zero16;
#pragma unroll
    for (int i = 0; i < 16; ++i) zero16[i] = 0.f;
    // only blocks that contain tree keys (or the end) need the mask
    auto mask = [&](int kb, Scores &S) {
        const int tbase = kb * TILE_KEYS;
        if (tbase + TILE_KEYS <= L) return;
        // read where it is needed, at most three blocks of a sequence: four registers fewer in all others
        const u64 *am = a.anc_mask + ((int64_t)b * a.TT_cap + node) * DT_MASK_WORDS;
        const u64 mask0 = am[0], mask1 = am[1];
        __builtin_amdgcn_s_waitcnt(0x0f70);  // or the compiler waits for them, and for the tiles, in every block
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const u32 vis = vis_window(tbase + 32 * j - L, mask0, mask1) >> (4 * half);
#pragma unroll
            for (int i = 0; i < 16; ++i) S.v[j][i] = ((vis >> (8 * (i >> 2) + (i & 3))) & 1u) ? S.v[j][i] : -INFINITY;
        }
    };
    // m_run is a reference, not the running maximum: the maximum of the range's first block, and it stays (unless one of the wave's
    // queries sees nothing there).  Later scores may lie above it, and their probabilities above 1, which neither 32-bit sums nor bf16's relative precision
    // mind as long as everything stays a number: sums of a lane's probabilities up to NEAR_LIMIT cannot hurt; above that the range's accumulators are
    // looked at when it ends, and past REF_LIMIT, or if one of them is not finite, the workgroup goes through the range once more (`exact`).  Then the
    // reference moves when a block's maximum lies more than LAZY_LOG2 binary orders above it, so that probabilities stay below 2^LAZY_LOG2,
    // at the price of a maximum over every block and, when it moves, of 64 multiplies.  A maximum in every block, in the shadow of
    // the second product, cost a lone workgroup of a compute unit 0.1 us of 0.95 a block, four sequences of a 70B step 3.4 % of their attention.
    // (-inf - -inf is NaN: a fully hidden block moves nothing.)
    float nmc = 0.f;
    auto move_reference = [&](float mloc) {
        mloc = half_swap_max(mloc);
        const bool move = (mloc - m_run) * c > LAZY_LOG2;
        const float m_new = move ? mloc : m_run;
        const float m_use = m_new == -INFINITY ? 0.f : m_new;
        const float alpha = move ? __builtin_amdgcn_exp2f((m_run - m_use) * c) : 1.0f;  // m_run = -inf -> 0
        nmc = -m_use * c;
        l_run *= alpha;
        m_run = m_new;
        if (__builtin_expect(__ballot(alpha != 1.0f) != 0, 0)) {  // the reference moved for some query of this wave
#pragma unroll
            for (int db = 0; db < DBLK; ++db)
#pragma unroll
                for (int i = 0; i < 16; ++i) oacc[db][i] *= alpha;
        }
    };

    // (as instructions: fmaxf on MFMA results costs two more per pair to quiet NaNs)
    auto block_max = [](const Scores &S) {
        asm volatile("s_nop 15\n\ts_nop 3");  // the distance from the last MFMA, which the compiler does not keep for what it does not know
        float m = -INFINITY, m1 = -INFINITY;
#pragma unroll
        for (int i = 0; i < 16; i += 2) {
            asm volatile("v_max3_f32 %0, %0, %1, %2" : "+v"(m) : "v"(S.v[0][i]), "v"(S.v[0][i + 1]));
            asm volatile("v_max3_f32 %0, %0, %1, %2" : "+v"(m1) : "v"(S.v[1][i]), "v"(S.v[1][i + 1]));
        }
        return fmaxf(m, m1);
    };
    __shared__ int s_again;
    auto sums_fine = [&]() {  // uniform
        if (!__builtin_amdgcn_ballot_w64(!(l_run <= NEAR_LIMIT))) return true;
        asm volatile("s_nop 15\n\ts_nop 3");  // as above
        float top[DBLK];
#pragma unroll
        for (int db = 0; db < DBLK; ++db) {
            top[db] = 0.f;
#pragma unroll
            for (int i = 0; i < 16; i += 2)
                asm volatile("v_maximum3_f32 %0, %0, |%1|, |%2|" : "+v"(top[db]) : "v"(oacc[db][i]), "v"(oacc[db][i + 1]));
        }
        asm volatile("v_maximum3_f32 %0, %0, %1, %2" : "+v"(top[0]) : "v"(top[1]), "v"(top[2]));
        const bool fine = l_run <= REF_LIMIT && top[0] < INFINITY && top[3] < INFINITY;  // false for a NaN
        return !__builtin_amdgcn_ballot_w64(!fine);
    };
    // One block: O += V(kb)^T P(kb)^T, and under it the scores of block kb + 1.  A wave that runs S^T, softmax and O^T of
    // the same block one after the other leaves the matrix pipe idle during its softmax and the vector pipe during its
    // MFMAs, and two such waves on a SIMD fall into step.  Here the two products of different blocks are independent of
    // the softmax arithmetic between them, so every MFMA is followed by a few vector instructions of the other block, which
    // issue while it runs:
    //   MFMA s of K(kb + 1) Q^T:  exponentials of block kb (16 of a lane's 32)
    //   MFMA n of V(kb)^T P^T:    the other 16, in time for the MFMA that takes them
    // What bounds a wave that has its SIMD to itself is the bytes of its instructions (some eight cycles for eight of them), and two to
    // a SIMD the power that the chip may draw (long sequences hold it at 1,350 to 1,400 of 1,400 W, where it clocks at 1.73 to 1.94 GHz of 2.4) and the loads into LDS:
    // a layer of the 70B step takes 113 us, for timing without the loads 97, without the exponentials 110, without both 93; eight long sequences of
    // the 8B shape 117, 94, 113 and 92; sixteen ragged ones (2.25 GHz), whose time is not in this loop alone, 64, 61, 63 and 59.
    // All LDS operand reads are bare instructions with hand-kept waits, eight K reads or seven V read pairs ahead of their
    // MFMA (V pairs start behind the last K reads).  P: CUR is the stage of V(kb); K(kb + 1) is in stage CUR ^ 1.
    // EXP_A(e), EXP_B(e): elements 2e and 2e + 1 of the lane's 32 (element i of S[j] is 16 j + i).  The multiply-add as an
    // instruction and the empty asm statements keep each of them where it is written: left alone, the compiler gathers the
    // multiply-adds in front of all MFMAs and the conversions behind them.
#define PIN(x) asm volatile("" : "+v"(x));
    // Behind a statement of this kind whose result one of the next two instructions reads, the compiler puts an s_nop.  So multiply-add and
    // exponential are one statement, and one wait releases the operands of two MFMAs, in front of the vector work of the MFMA before them.
    // A block of a lone workgroup, with the maxima left out as well: 0.95 -> 0.83 us.
#define SCALED_EXP(p, e)                                                                                      \
        asm volatile("v_fma_f32 %0, %1, %2, %3\n\tv_exp_f32 %0, %0" : "=v"(p) : "v"(S.v[(e) >> 4][(e) & 15]), "v"(c), "v"(nmc));
#define EXP_A(e) SCALED_EXP(pe, 2 * (e))
#define EXP_B(e)                                                                                              \
        {                                                                                                      \
            float pf;                                                                                          \
            SCALED_EXP(pf, 2 * (e) + 1)                                                                        \
            psum0 += pe;                                                                                       \
            psum1 += pf;                                                                                       \
            bf16x2 pk = {(__bf16)pe, (__bf16)pf};                                                              \
            pw[e] = __builtin_bit_cast(u32, pk);                                                               \
            PIN(pw[e])                                                                                         \
        }
#define K_READ(i) ka[i] = lds_load128_at<(NS == 2 ? (CUR ^ 1) * TILE_BYTES : 0) + ((i) >> 2) * SUB_BYTES + ((i) & 1) * 32 * 64>(kat[((i) >> 1) & 1]);
#define K_WAIT(i, W) lds_wait<W>(ka[i]);
#define K_WAIT2(i, W) lds_wait2<W>(ka[i], ka[(i) + 1]);
#define QK_MFMA(i)                                                                                            \
        T.v[(i) & 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[i], qreg[(i) >> 1], (i) < 2 ? zero16 : T.v[(i) & 1], 0, 0, 0); \
        __builtin_amdgcn_sched_barrier(0);
#define V_READ(n)                                                                                             \
        vlo[n] = lds_load_tr4<(NS == 2 ? CUR * TILE_BYTES : 0) + ((n) & 3) * SUB_BYTES + 16 * ((n) >> 2) * 64>(vat);         \
        vhi[n] = lds_load_tr4<(NS == 2 ? CUR * TILE_BYTES : 0) + ((n) & 3) * SUB_BYTES + (16 * ((n) >> 2) + 8) * 64>(vat);
#define V_WAIT2(n, W) lds_wait4<W>(vlo[n], vhi[n], vlo[(n) + 1], vhi[(n) + 1]);
#define PV_MFMA(n)                                                                                            \
        oacc[(n) & 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(                                               \
            __builtin_shufflevector(vlo[n], vhi[n], 0, 1, 2, 3, 4, 5, 6, 7), p_operand(&pw[4 * ((n) >> 2)]),   \
            oacc[(n) & 3], 0, 0, 0);                                                                           \
        __builtin_amdgcn_sched_barrier(0);
#define FENCE __builtin_amdgcn_sched_barrier(0);
    auto p_operand = [](const u32 *wd) {
        const uint4 v = make_uint4(wd[0], wd[1], wd[2], wd[3]);
        return __builtin_bit_cast(bf16x8, v);
    };
    // inside: the blocks up to kb + NS are there and hold prefix keys only, and nothing else is to be asked either: no branches
    // (some fifteen in a block; taken ones cost a lone wave up to twenty cycles).
    auto block = [&](auto cur_c, auto inside, int kb, Scores &S, Scores &T) {
        constexpr int CUR = decltype(cur_c)::value;
        constexpr bool IN = decltype(inside)::value;
        const bool next = IN || kb + 1 < kb1;  // uniform
        // K(kb) was last read before the previous barrier, V(kb - 1) too: their stages take K(kb + NS) and V(kb + NS - 1)
        if (IN || kb + NS < kb1) fetch_k(inside, kb + NS, NS == 2 ? CUR : stage_of(kb));
        if (IN || kb + NS - 1 < kb1) fetch_v(inside, kb + NS - 1, NS == 2 ? CUR ^ 1 : stage_of(kb - 1));
        const u32 kst = NS == 2 ? 0 : stage_of(kb + 1) * TILE_BYTES, vst = NS == 2 ? 0 : stage_of(kb) * TILE_BYTES;
        const u32 kat[2] = {koff[0] + kst, koff[1] + kst}, vat = voff + vst;
        if (IN || active) {
            float psum0 = 0.f, psum1 = 0.f, pe;
            u32 pw[16];  // the probabilities as pairs of bf16
            bf16x4 vlo[16], vhi[16];
            if (next) {
                bf16x8 ka[16];  // read i: k-step i / 2, half i % 2
                K_READ(0) K_READ(1) K_READ(2) K_READ(3) K_READ(4) K_READ(5) K_READ(6) K_READ(7) FENCE
                K_WAIT2(0, 6) FENCE
                QK_MFMA(0) K_READ(8) K_WAIT2(2, 5) EXP_A(0) FENCE
                QK_MFMA(1) K_READ(9) EXP_B(0) FENCE
                QK_MFMA(2) K_READ(10) K_WAIT2(4, 5) EXP_A(1) FENCE
                QK_MFMA(3) K_READ(11) EXP_B(1) FENCE
                QK_MFMA(4) K_READ(12) K_WAIT2(6, 5) EXP_A(2) FENCE
                QK_MFMA(5) K_READ(13) EXP_B(2) FENCE
                QK_MFMA(6) K_READ(14) K_WAIT2(8, 5) EXP_A(3) FENCE
                QK_MFMA(7) K_READ(15) EXP_B(3) FENCE
                QK_MFMA(8) V_READ(0) K_WAIT2(10, 6) EXP_A(4) FENCE
                QK_MFMA(9) V_READ(1) EXP_B(4) FENCE
                QK_MFMA(10) V_READ(2) K_WAIT2(12, 8) EXP_A(5) FENCE
                QK_MFMA(11) V_READ(3) EXP_B(5) FENCE
                QK_MFMA(12) V_READ(4) K_WAIT2(14, 10) EXP_A(6) FENCE
                QK_MFMA(13) V_READ(5) EXP_B(6) FENCE
                QK_MFMA(14) V_READ(6) V_WAIT2(0, 10) EXP_A(7) FENCE
                QK_MFMA(15) EXP_B(7) FENCE
            } else {
                V_READ(0) V_READ(1) V_READ(2) V_READ(3) V_READ(4) V_READ(5) V_READ(6) FENCE
                EXP_A(0) EXP_B(0) EXP_A(1) EXP_B(1) EXP_A(2) EXP_B(2) EXP_A(3) EXP_B(3)
                EXP_A(4) EXP_B(4) EXP_A(5) EXP_B(5) EXP_A(6) EXP_B(6) V_WAIT2(0, 10) EXP_A(7) EXP_B(7) FENCE
            }
            PV_MFMA(0) V_READ(7) V_WAIT2(2, 8) EXP_A(8) FENCE
            PV_MFMA(1) V_READ(8) EXP_B(8) FENCE
            if (!IN && next) mask(kb + 1, T);
            PV_MFMA(2) V_READ(9) V_WAIT2(4, 8) EXP_A(9) FENCE
            PV_MFMA(3) V_READ(10) EXP_B(9) EXP_A(10) FENCE
            PV_MFMA(4) V_READ(11) V_WAIT2(6, 8) EXP_B(10) FENCE
            PV_MFMA(5) V_READ(12) EXP_A(11) FENCE
            PV_MFMA(6) V_READ(13) V_WAIT2(8, 8) EXP_B(11) EXP_A(12) FENCE
            PV_MFMA(7) V_READ(14) EXP_B(12) FENCE
            PV_MFMA(8) V_READ(15) V_WAIT2(10, 8) EXP_A(13) FENCE
            PV_MFMA(9) EXP_B(13) EXP_A(14) FENCE
            PV_MFMA(10) V_WAIT2(12, 4) EXP_B(14) EXP_A(15) FENCE
            PV_MFMA(11) EXP_B(15) FENCE
            PV_MFMA(12) V_WAIT2(14, 0) FENCE
            PV_MFMA(13) FENCE
            PV_MFMA(14) FENCE
            PV_MFMA(15)
            l_run += psum0 + psum1;
            if (!IN && __builtin_expect(exact && next, 0)) move_reference(block_max(T));
            if (!next && !exact && !sums_fine() && lane == 0) s_again = 1;
            // the "memory" clobber keeps the next block's loads into these stages behind this block's reads
            asm volatile("" ::: "memory");
        }
        if constexpr (NS == 2) {
            __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0): this wave's part of the next tiles has landed
            __syncthreads();
        } else {
            // K(kb + 2) and V(kb + 1), asked for two blocks ago, have to be there; what was asked for since (four loads a tile) may be on its way
            const int left = kb1 - kb;
            if (IN || left > 4) asm volatile("s_waitcnt vmcnt(16)" ::: "memory");
            else if (left == 4) asm volatile("s_waitcnt vmcnt(12)" ::: "memory");
            else if (left == 3) asm volatile("s_waitcnt vmcnt(4)" ::: "memory");
            else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
        }
    };
    Scores S0, S1;
    const __bf16 *qp = (const __bf16 *)a.q + (((int64_t)b * a.TT_cap + node) * a.Hq + hq) * D + 8 * half;
    if constexpr (NS == 2) {
        fetch_k(anywhere, kb0, 0);
#pragma unroll
        for (int s = 0; s < KSTEPS; ++s) qreg[s] = *(const bf16x8 *)(qp + 16 * s);
        fetch_v(anywhere, kb0, 0);
        if (kb0 + 1 < kb1) fetch_k(anywhere, kb0 + 1, 1);
        __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0): this wave's part of the tiles is in LDS
        __syncthreads();
    } else {
        // in the order in which they are needed; the queries as instructions, since the compiler would wait for everything behind them
        fetch_k(anywhere, kb0, 0);
#define Q_LOAD(s) asm volatile("global_load_dwordx4 %0, %1, off offset:%2" : "=v"(qreg[s]) : "v"(qp), "n"(32 * (s)) : "memory");
        Q_LOAD(0) Q_LOAD(1) Q_LOAD(2) Q_LOAD(3) Q_LOAD(4) Q_LOAD(5) Q_LOAD(6) Q_LOAD(7)
#undef Q_LOAD
        fetch_v(anywhere, kb0, 0);
        for (int i = 1; i < 4; ++i)
            if (kb0 + i < kb1) {
                fetch_k(anywhere, kb0 + i, i);
                if (i < 3) fetch_v(anywhere, kb0 + i, i);
            }
        const int n = kb1 - kb0;  // the first K tile and the queries
        if (n >= 4) asm volatile("s_waitcnt vmcnt(24)" ::: "memory");
        else if (n == 3) asm volatile("s_waitcnt vmcnt(20)" ::: "memory");
        else if (n == 2) asm volatile("s_waitcnt vmcnt(12)" ::: "memory");
        else asm volatile("s_waitcnt vmcnt(4)" ::: "memory");
        asm volatile("" : "+v"(qreg[0]), "+v"(qreg[1]), "+v"(qreg[2]), "+v"(qreg[3]), "+v"(qreg[4]), "+v"(qreg[5]), "+v"(qreg[6]), "+v"(qreg[7]));
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    }
    if (tid == 0) s_again = 0;  // every wave has read the segment before's
    if (active) {  // scores of the first block
        constexpr int CUR = 1;
        const u32 kat[2] = {koff[0], koff[1]};
        Scores &T = S0;
        bf16x8 ka[16];
        K_READ(0) K_READ(1) K_READ(2) K_READ(3) K_READ(4) K_READ(5) K_READ(6) K_READ(7) FENCE
        K_WAIT(0, 7) QK_MFMA(0) K_READ(8) FENCE K_WAIT(1, 7) QK_MFMA(1) K_READ(9) FENCE
        K_WAIT(2, 7) QK_MFMA(2) K_READ(10) FENCE K_WAIT(3, 7) QK_MFMA(3) K_READ(11) FENCE
        K_WAIT(4, 7) QK_MFMA(4) K_READ(12) FENCE K_WAIT(5, 7) QK_MFMA(5) K_READ(13) FENCE
        K_WAIT(6, 7) QK_MFMA(6) K_READ(14) FENCE K_WAIT(7, 7) QK_MFMA(7) K_READ(15) FENCE
        K_WAIT(8, 7) QK_MFMA(8) FENCE K_WAIT(9, 6) QK_MFMA(9) FENCE
        K_WAIT(10, 5) QK_MFMA(10) FENCE K_WAIT(11, 4) QK_MFMA(11) FENCE
        K_WAIT(12, 3) QK_MFMA(12) FENCE K_WAIT(13, 2) QK_MFMA(13) FENCE
        K_WAIT(14, 1) QK_MFMA(14) FENCE K_WAIT(15, 0) QK_MFMA(15)
        mask(kb0, S0);
        move_reference(block_max(S0));
        // Nothing of the block for some query (a range that begins among the tree's keys, a mask without them): no reference to stay with, and the scores to
        // come may be so low that 0 in its place would leave nothing of them.  This wave's moves.
        exact = exact || __builtin_amdgcn_ballot_w64(m_run == -INFINITY) != 0;
        asm volatile("" ::: "memory");
    }
    if constexpr (NS == 2) {
        __syncthreads();  // K stage 0 is free
    } else {              // and V(kb0) and K(kb0 + 1) are there
        const int n = kb1 - kb0;
        if (n >= 4) asm volatile("s_waitcnt vmcnt(16)" ::: "memory");
        else if (n == 3) asm volatile("s_waitcnt vmcnt(12)" ::: "memory");
        else if (n == 2) asm volatile("s_waitcnt vmcnt(4)" ::: "memory");
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    }
    // The two workgroups of a compute unit have equal work, but a SIMD issues the older of two ready waves, so the first to
    // arrive finished 15 us of 110 before the second, which then ran alone at 60 % of the pair's rate.  The wave in the odd slot
    // goes first in every other block instead: both end within 5 us (4 sequences of a 70B step 121 -> 117 us, 64 wide trees
    // 240 -> 231; odd slots first in every block: 120 and 236).
    const bool odd_slot = __builtin_amdgcn_s_getreg((3 << 11) | 4) & 1;  // HW_ID, 4 bits from bit 0: wave slot of the SIMD
    const std::integral_constant<int, 0> even;
    const std::integral_constant<int, 1> odd;
    int kb = kb0;
    if (active && small_stride && !exact)
        for (const int end = min(kb1, L / TILE_KEYS); kb + NS + 1 < end; kb += 2) {
            if (odd_slot) __builtin_amdgcn_s_setprio(1);
            block(even, std::true_type(), kb, S0, S1);
            if (odd_slot) __builtin_amdgcn_s_setprio(0);
            block(odd, std::true_type(), kb + 1, S1, S0);
        }
    for (; kb < kb1; kb += 2) {
        if (odd_slot) __builtin_amdgcn_s_setprio(1);
        block(even, anywhere, kb, S0, S1);
        if (odd_slot) __builtin_amdgcn_s_setprio(0);
        if (kb + 1 < kb1) block(odd, anywhere, kb + 1, S1, S0);
    }
    if (__builtin_expect(s_again, 0)) return true;
#undef PIN
#undef SCALED_EXP
#undef EXP_A
#undef EXP_B
#undef K_READ
#undef K_WAIT
#undef K_WAIT2
#undef QK_MFMA
#undef V_READ
#undef V_WAIT2
#undef PV_MFMA
#undef FENCE

    // ---- epilogue -------------------------------------------------------------------------------
    float l_tot = half_swap_sum(l_run);
    if (pt.parts > 1) {
        int word = lane;
        asm volatile("" : "+v"(word));  // as above: the addresses are worked out here
        // The last part's workgroup usually finds the others' partials there, and then leaves none of its own.
        __shared__ int s_last[2];
        const bool many = __builtin_expect(pt.parts > SERIAL_PARTS, 0);
        u64 seen = 0;
        if (tid == 0) {
            seen = get_agent(pt.count);
            s_last[0] = !many && seen == (pt.tag | (pt.parts - 1));
        }
        __syncthreads();
        const int mine = 32 * rb + col;
        if (!s_last[0]) {
            if (active) {
                const int64_t at = 2 * (pt.slot + pt.me * pt.step) + (pt.me == 0);
                u64 *op = pt.o + at * (D / 4 * 256) + 64 * rb + word;
#pragma unroll
                for (int i = 0; i < D / 4; ++i)
                    put_agent(op + i * 256, __builtin_bit_cast(u64, make_float2(oacc[i >> 3][(2 * i) & 15], oacc[i >> 3][(2 * i + 1) & 15])));
                if (half == 0) put_agent(pt.ml + at * ATT_MTILE + mine, __builtin_bit_cast(u64, make_float2(m_run, l_tot)));
            }
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the stores are there before the count says so
            __syncthreads();
            if (many) {
                SharedMerge sm;
                sm.pt = pt;
                sm.marks = pt.ml + (int64_t)slots * (2 * ATT_MTILE + 1);
                sm.stay = stay;
                sm.out = (__bf16 *)a.out + ((int64_t)b * a.TT_cap * a.Hq + h * G) * D;
                sm.m0 = m0; sm.rb = rb; sm.M = M; sm.G = G; sm.Hq = a.Hq;
                sm.c = c;
                merge_shared<D>(sm);
                return false;
            }
            if (tid == 0) s_last[1] = arrive_last(pt.count, pt.tag, pt.parts, seen);
            __syncthreads();
            if (!s_last[1]) return false;
        } else if (tid == 0) {
            put_agent(pt.count, 0);
        }
        asm volatile("" ::: "memory");
        if (active) {
            // in the order of the parts, whoever came last: the same sum each time
            float M = -INFINITY, l = 0.f;
            f32x16 acc[DBLK];
#pragma unroll
            for (int db = 0; db < DBLK; ++db)
#pragma unroll
                for (int i = 0; i < 16; ++i) acc[db][i] = 0.f;
            for (int i = 0; i < pt.parts; ++i) {
                float2 ml = make_float2(m_run, l_tot);
                f32x16 o[DBLK];
                if (i == pt.me) {
#pragma unroll
                    for (int db = 0; db < DBLK; ++db) o[db] = oacc[db];
                } else {
                    const int64_t at = 2 * (pt.slot + i * pt.step) + (i == 0);
                    u64 *op = pt.o + at * (D / 4 * 256) + 64 * rb + word;
                    ml = __builtin_bit_cast(float2, get_agent(pt.ml + at * ATT_MTILE + mine));
#pragma unroll
                    for (int e = 0; e < D / 4; ++e) {
                        const float2 v = __builtin_bit_cast(float2, get_agent(op + e * 256));
                        o[e >> 3][(2 * e) & 15] = v.x;
                        o[e >> 3][(2 * e + 1) & 15] = v.y;
                    }
                }
                const bool some = ml.y > 0.f;  // a range whose keys were all hidden weighs nothing
                const float M2 = some ? fmaxf(M, ml.x) : M;
                const float keep = some ? __builtin_amdgcn_exp2f((M - M2) * c) : 1.f;  // first partial: exp2(-inf) = 0
                const float wgt = some ? __builtin_amdgcn_exp2f((ml.x - M2) * c) : 0.f;
#pragma unroll
                for (int db = 0; db < DBLK; ++db)
#pragma unroll
                    for (int e = 0; e < 16; ++e) acc[db][e] = acc[db][e] * keep + o[db][e] * wgt;
                l = l * keep + ml.y * wgt;
                M = M2;
            }
            l_tot = l;
#pragma unroll
            for (int db = 0; db < DBLK; ++db) oacc[db] = acc[db];
        }
    }
    if (!qvalid) return false;
    const float inv = l_tot > 0.f ? 1.0f / l_tot : 0.f;
    int h4 = 4 * half;
    asm volatile("" : "+v"(h4));  // as above
    __bf16 *op = (__bf16 *)a.out + h4 + (((int64_t)b * a.TT_cap + node) * a.Hq + hq) * D;
#pragma unroll
    for (int db = 0; db < DBLK; ++db)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            bf16x4 o4;
#pragma unroll
            for (int e = 0; e < 4; ++e) o4[e] = (__bf16)(oacc[db][q * 4 + e] * inv);
            *(bf16x4 *)(op + 32 * db + 8 * q) = o4;
        }
    return false;
}

// One workgroup per (kv head, row tile, sequence), the whole key range: for short sequences, and for batches that the balanced
// schedule below does not take.  blockIdx.x = kv head: workgroups are dealt to the 8 XCDs
// round-robin by linear id, so all row tiles of one kv head land on one XCD and share its L2
// copy of that head's K/V.
template <int D, int NS>
__global__ __launch_bounds__(256, 2) void attn_tile_kernel(AttnArgs a, GroupDiv gd) {
    extern __shared__ __attribute__((aligned(16))) unsigned char s_dyn[];
    const int b = blockIdx.z, h = blockIdx.x, m0 = blockIdx.y * ATT_MTILE;
    // the four words in one trip to memory: the compiler would fetch the others behind the test of the first
    int n_raw = a.n_nodes[b], l_raw = a.prefix_len[b];
    u64 kp_raw = (u64)(uintptr_t)a.k_prefix[b], vp_raw = (u64)(uintptr_t)a.v_prefix[b];
    asm volatile("" : "+s"(n_raw), "+s"(l_raw), "+s"(kp_raw), "+s"(vp_raw));
    const SeqWords sq = {min(max(n_raw, 1), a.TT_cap), max(l_raw, 0), kp_raw, vp_raw};
    if (m0 >= sq.N * gd.G) return;
    const int nb = (sq.L + sq.N + TILE_KEYS - 1) / TILE_KEYS;
    TileParts whole = {};
    whole.parts = 1;
    bool exact = false;
    while (tile_segment<D, NS>(a, gd, sq, s_dyn, h, b, m0, blockIdx.y + blockIdx.z, 0, nb, whole, 0, false, exact)) exact = true;
}

// ---- balanced schedule -----------------------------------------------------------------------------
// Each kv head gets P workgroup slots (two per compute unit over all heads).  Sequences are
// grouped into classes by their number of row tiles m; the key blocks of a class's sequences,
// concatenated in batch order, form its C_m "columns" of cost m each.  Class m is given g_m
// "gangs" of m slots (one per row tile, neighbours in launch order, so the tiles of a sequence walk
// its K/V together and share it in L2); gang j takes columns [j T_m, (j+1) T_m) of the class, with
// T_m = ceil(C_m / g_m), and the g_m are the ones that minimise max_m T_m under sum m g_m <= P, or the next ones where fewer cuts
// are worth more than slots (below); or every sequence has a gang of its own, where there are slots for all and that is cheaper still.
// A slot therefore works through a few (sequence, tile, key range) segments of near-equal total
// length.  A sequence cut by a range boundary leaves partials: per slot at most one "head" (its first
// segment, when that sequence began in an earlier gang) and one "tail" (a sequence that began
// here and runs on), and the slot of its first gang holds the count of them.  The last workgroup to come merges them, or, if
// they are many, those that have stayed for it together: a merge kernel of its own read every partial back from memory after
// all had been written, 9 to 16 us of a launch of 62 to 240, while here a head is written early and read once by the workgroup
// that ends with the tail.
// Every wave derives the plan by itself from n_nodes / prefix_len with wave
// operations (sequence b in lane b: batch <= 64; class m in lane m), so no barrier is involved.
// How long a plan takes, in twentieths of a microsecond: a block of a slot that has its compute unit to itself, or shares it; a sequence in
// parts (its partials written, counted in and, part after part, read back), and in so many that its workgroups share the merge.
// A cut that fills the chip is not worth its partials where sequences are short: two workgroups of a compute unit take nearly twice as long for a
// block as one.  The smallest T that fits, always, against this (us per layer, 8B shape unless said): 8 sequences of 112 nodes, 40 keys 23.2 | 13.1,
// 400 26.7 | 18.9, 1,100 43.7 | 31.8; 14 of 64, 400 27.0 | 18.8, of 112, 400 33.5 | 25.4; 5 of 64, 1,600 keys 45.7 | 30.4, 2,400 40.8 | 30.4; four of
// the 70B shape, 64 nodes, 1,600 38.4 | 28.6; 20 of seven query heads to each of two kv heads, 64 nodes, 400 39.9 | 18.5, 2,400 ragged 46.9 | 39.0.
// Where the chip is full or one sequence is far longer than the others, the smallest T stays.
#define COST_BLOCK 22
#define COST_BLOCK_PAIR 36
#define COST_CUT 60
#define COST_PART 60
#define COST_SHARED 500
struct GangPartial {
    u64 *o;       // [Hkv, P, 2, D / 4, 256]
    u64 *ml;      // [Hkv, P, 2, 128]
    u64 *count;   // [Hkv, P], and behind them the marks, [Hkv, P, 2]
    u64 tag;      // of this launch: what the memory held before it never looks like a count or a mark
};

// x / d for 0 <= x < 2^31 and d >= 1: two steps from the reciprocal, each off by a few units of its own result at most, and the last
// unit by the remainder.  (The compiler's division is some forty instructions, and the plan has ten in a row.)
__device__ __forceinline__ int div_small(int x, int d) {
    const float inv = __builtin_amdgcn_rcpf((float)d);
    int q = (int)((float)x * inv), r = x - q * d;
    const int q1 = (int)((float)r * inv);
    q += q1;
    r -= q1 * d;
    return q + (r >= d ? 1 : 0) - (r < 0 ? 1 : 0);
}

struct GangPlan {
    int mt, nb;        // lane b: row tiles and key blocks of sequence b (0 past the batch)
    u64 classes;       // bit m: there are sequences of m row tiles
    int C, g, T;       // lane m: columns, gangs and columns per gang of class m
    int pitch;         // > 0: every sequence has a gang of its own, `pitch` columns wide; 0: columns follow each other
};

__device__ __forceinline__ GangPlan gang_plan(const SeqWords &mine, int G, int batch, int P, int lane) {
    GangPlan p;
    p.mt = 0;
    p.nb = 0;
    if (lane < batch) {
        p.mt = (mine.N * G + ATT_MTILE - 1) / ATT_MTILE;
        p.nb = (mine.L + mine.N + TILE_KEYS - 1) / TILE_KEYS;
    }
    p.classes = 0;
    p.C = 0;
    int W = 0, tiles = 0, count = 0;
    for (u64 left = __builtin_amdgcn_ballot_w64(p.mt > 0); left;) {
        const int m = __builtin_amdgcn_readlane(p.mt, __builtin_ctzll(left));
        const int c = wave_sum_i32(p.mt == m ? p.nb : 0);
        const u64 members = __builtin_amdgcn_ballot_w64(p.mt == m);
        const int n = __popcll(members);
        if (lane == m) {
            p.C = c;
            count = n;
        }
        W += m * c;
        tiles += m * n;
        p.classes |= 1ull << m;
        left &= ~members;
    }
    // smallest T with sum_m m ceil(C_m / T) <= P: lane i probes T0 + i.  T = max C_m always fits
    // (the host checks P >= 1 + 2 + .. + mt_max), so the loop ends.
    auto slots_of = [&](int t) {
        int slots = 0;
        for (u64 left = p.classes; left; left &= left - 1) {
            const int m = (int)__builtin_ctzll(left);
            slots += m * div_small(__builtin_amdgcn_readlane(p.C, m) + t - 1, t);
        }
        return slots;
    };
    int T0 = max(1, div_small(W + P - 1, P)), T;
    for (;;) {
        const u64 ok = __builtin_amdgcn_ballot_w64(slots_of(T0 + lane) <= P);
        if (ok) {
            T = T0 + (int)__builtin_ctzll(ok);
            break;
        }
        T0 += 64;
    }
    // What the plan costs with T and up to 63 larger ones, one to a lane; and with every sequence whole.
    const int longest = wave_max_i32(p.nb);
    const int step = max(1, (longest - T + 62) / 63);
    const int t = T + step * lane, parts = div_small(longest + t - 1, t);
    const int block = slots_of(t) <= P / 2 ? COST_BLOCK : COST_BLOCK_PAIR;
    const u32 cost = (u32)(block * t + (parts > SERIAL_PARTS ? COST_SHARED : COST_CUT + COST_PART * max(parts, 2)));
    const u32 best = ~wave_max_u32(~(cost << 6 | (u32)lane));  // of equal ones the smallest
    T += step * (int)(best & 63u);
    p.pitch = tiles <= P && (u32)((tiles <= P / 2 ? COST_BLOCK : COST_BLOCK_PAIR) * longest) <= best >> 6 ? longest : 0;
    p.g = p.pitch ? count : div_small(p.C + T - 1, T);
    p.T = p.pitch ? longest : p.g > 0 ? div_small(p.C + p.g - 1, p.g) : 0;
    if (p.pitch) p.C = count * longest;
    return p;
}

template <int D>
__global__ __launch_bounds__(256, 2) void attn_gang_kernel(AttnArgs a, GroupDiv gd, int P, GangPartial part) {
    extern __shared__ __attribute__((aligned(16))) unsigned char s_dyn[];
    const int h = blockIdx.x, y = blockIdx.y, lane = threadIdx.x & 63;
    // lane b: the words of sequence b, in one trip to memory (read again by every segment, a sequence's pointers behind its lengths,
    // and with the compiler's divisions in the plan, a launch took 1.0 to 1.7 us longer: 8 sequences of the 8B shape, 112 nodes, 40 keys 23.7 us, now
    // 22.8; 64 nodes, 1,100 keys 41.8 and 40.2; 4 of the 70B shape, 2,048 keys 45.8 and 44.8)
    const int bl = min(lane, a.batch - 1);
    const int n_raw = a.n_nodes[bl], l_raw = a.prefix_len[bl];
    const SeqWords mine = {min(max(n_raw, 1), a.TT_cap), max(l_raw, 0), (u64)(uintptr_t)a.k_prefix[bl], (u64)(uintptr_t)a.v_prefix[bl]};
    const GangPlan p = gang_plan(mine, gd.G, a.batch, P, lane);
    // class, gang and row tile of slot y
    int base = 0, cls = 0;
    for (u64 left = p.classes; left; left &= left - 1) {
        const int m = (int)__builtin_ctzll(left), span = m * __builtin_amdgcn_readlane(p.g, m);
        if (y < base + span) {
            cls = m;
            break;
        }
        base += span;
    }
    if (cls == 0) return;  // spare slot
    const int j = __builtin_amdgcn_readfirstlane(div_small(y - base, cls)), tile = y - base - j * cls;
    const int Tc = __builtin_amdgcn_readlane(p.T, cls), Cc = __builtin_amdgcn_readlane(p.C, cls);
    const int lo = j * Tc, hi = min(Cc, lo + Tc);
    // first column of every sequence of this class
    const int val = p.mt == cls ? p.nb : 0;
    const int cs = p.pitch ? (int)lanes_below(__builtin_amdgcn_ballot_w64(val > 0)) * p.pitch : wave_scan_incl_i32(val) - val;
    u64 segs = __builtin_amdgcn_ballot_w64(val > 0 && cs < hi && cs + val > lo);
    // What a segment needs of its sequence, out of the registers of the loop over its blocks.  Every wave writes the same.
    __shared__ struct { SeqWords w; int cs, nb; } s_seq[64];
    s_seq[lane].w = mine;
    s_seq[lane].cs = cs;
    s_seq[lane].nb = val;
    bool exact = false;
    while (segs) {
        const int b = (int)__builtin_ctzll(segs);
        asm volatile("" ::: "memory");
        const int csb = __builtin_amdgcn_readfirstlane(s_seq[b].cs), nbb = __builtin_amdgcn_readfirstlane(s_seq[b].nb);
        const SeqWords sq = {__builtin_amdgcn_readfirstlane(s_seq[b].w.N), __builtin_amdgcn_readfirstlane(s_seq[b].w.L),
                             readlane_u64(s_seq[b].w.kpre, 0), readlane_u64(s_seq[b].w.vpre, 0)};
        const int kb0 = max(lo, csb) - csb, kb1 = min(hi, csb + nbb) - csb;
        // its first and its last gang
        const int jf = __builtin_amdgcn_readfirstlane(div_small(csb, Tc)), jl = __builtin_amdgcn_readfirstlane(div_small(csb + nbb - 1, Tc));
        TileParts pt;
        pt.parts = jl - jf + 1;
        pt.me = j - jf;
        pt.slot = h * P + base + jf * cls + tile;
        pt.step = cls;
        pt.o = part.o;
        pt.ml = part.ml;
        pt.count = part.count + pt.slot;
        pt.tag = part.tag;
        exact = tile_segment<D, 2>(a, gd, sq, s_dyn, h, b, tile * ATT_MTILE, j, kb0, kb1, pt, a.Hkv * P, !(segs & (segs - 1)), exact);
        if (!exact) segs &= segs - 1;
    }
}

// ------------------------------------------------------------------- small-batch kernel -----
// When a batch offers only a few (sequence, kv head) pairs, latency matters more than reuse:
// one workgroup owns 32 query rows, its NW waves take the key blocks round-robin and stream
// them PRIVATELY (coalesced 16-byte loads, a wave-private LDS tile to bring K into operand
// layout and V into transposed operand layout, next block prefetched into registers), so the
// main loop has no barrier at all.  The partial results meet in LDS once at the end; nothing
// goes through global scratch.  Two variants: eight waves that stage each block through registers
// into padded tiles (one workgroup per unit, short key ranges), and four waves that load straight
// into LDS (DIRECT: several workgroups per unit, one wave per SIMD, so latency is hidden inside the
// wave by having every operand read of a block in flight at once).
// What bounds a launch is the chain of its trips to memory and, with one wave per SIMD, the number of its instructions (one
// in eight cycles or so): hence one trip for the four words of a sequence, no division, accumulators in plain registers
// (moved to and from the accumulator file, rescaling them cost 3,300 cycles of 16,800) and no rescaling of
// accumulators that are still zero.  8B shape, 1,024 keys, kernel and merge: 12.6 -> 10.9 us per layer; 256 keys 9.0 -> 8.7;
// 4,096 keys 19.2 -> 18.0.
// Staged layout, both tiles row-major with padded rows of bf16 elements.  K: the 16 B reads of 16 consecutive rows fall
// into 16 different slots of 256 B (pitch 272 B at D = 128, 144 B at D = 64).  V: the transposing read takes 4 rows x 64 B
// per 32 lanes, which fall into four different 64-byte groups (pitch 320 B, 192 B).
template <int D>
struct WaveTile {
    static constexpr int K_PITCH = D + 8, V_PITCH = D + 32, K_ELEMS = ATT_KB * K_PITCH, ELEMS = K_ELEMS + ATT_KB * V_PITCH;
};
#define WD_TILE (ATT_KB * 256)                  // direct layout: one K or V tile of a wave
#define WD_SUB (ATT_KB * 128)                   // half of its columns
#define WD_STAGE (2 * WD_TILE)                  // K tile + V tile of one stage
// LDS of a wave: its tiles, and at the end its partial results
template <int D, bool DIRECT>
struct WaveArea {
    static constexpr int BYTES = DIRECT ? 2 * WD_STAGE : WaveTile<D>::ELEMS * 2;
    static_assert(BYTES >= 32 * D * 4, "a wave's accumulators go where its tiles were");
};
#define WD_LDS_BYTES (4 * 2 * WD_STAGE)         // four waves, two stages: 128 KB

// With KS > 1 the key blocks are additionally dealt over KS workgroups per (sequence, kv head, row block), whose waves put their
// partials together in the same launch (join_splits).
struct SplitBuf {
    float4 *o;     // [unit, D/32 waves, KS, 4, 64 lanes]: a wave's output registers
    float2 *ml;    // [unit, D/32 waves, KS, 32]: (max, sum) per query row
    u64 *offers;   // [unit, D/32 waves, KS], a cache line each (Hands)
    u64 *marks;    // [unit, D/32 waves, KS]
    u64 tag;       // of this launch
    GroupDiv gd, hd, md;  // by the query heads per kv head, the kv heads, the row blocks
    int units;
    u32 ks_magic;  // x / KS = x * ks_magic / 4096 for x < 64
};
#define MAX_SPLITS 8

// Sixteen and eight bytes to the memory side, past the L2s (not coherent between the XCDs inside a launch): a relaxed atomic at
// agent scope for more than a word.
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ void put16_agent(float4 *p, f32x4 v) { asm volatile("global_store_dwordx4 %0, %1, off sc1" ::"v"(p), "v"(v) : "memory"); }
__device__ __forceinline__ void put8_agent(float2 *p, f32x2 v) { asm volatile("global_store_dwordx2 %0, %1, off sc1" ::"v"(p), "v"(v) : "memory"); }
// N partials (four times 1,024 bytes of a wave from o[u] on, with STATS the statistics at ml[u] too) in one trip, past the L1: from this XCD's L2 what
// was written there, else from the memory side.  With them, in the lanes of `lanes`, *word is exchanged for the first half of `swap` where it is the
// second (within the XCD); `was`, in those lanes, is what it was.  One statement, since the registers hold nothing that may be copied before the wait.
template <int N, bool STATS>
__device__ __forceinline__ void get_partials(const float4 *const (&o)[N], const u64 *const (&ml)[N], f32x4 (&p)[N][4], u64 (&st)[N], u64 lanes, u64 *word,
                                             u64x2 swap, u64 &was) {
#define PART_LOADS(o, p0, p1, p2, p3)                                                                              \
    "global_load_dwordx4 " p0 ", " o ", off sc1\n\tglobal_load_dwordx4 " p1 ", " o ", off offset:1024 sc1\n\t"    \
    "global_load_dwordx4 " p2 ", " o ", off offset:2048 sc1\n\tglobal_load_dwordx4 " p3 ", " o ", off offset:3072 sc1\n\t"
#define PART_STAT(st, ml) "global_load_dwordx2 " st ", " ml ", off sc1\n\t"
#define PART_SWAP "s_mov_b64 %1, exec\n\ts_mov_b64 exec, %[lanes]\n\tglobal_atomic_cmpswap_x2 %0, %[word], %[swap], off sc0\n\ts_mov_b64 exec, %1\n\t"
#define PART_OUT(u) "=&v"(p[u][0]), "=&v"(p[u][1]), "=&v"(p[u][2]), "=&v"(p[u][3])
#define PART_SWAP_OUT "=&v"(was), "=&s"(all)
#define PART_SWAP_IN [lanes] "s"(lanes), [word] "v"(word), [swap] "v"(swap)
    u64 all;
    if constexpr (!STATS && N == 1)
        asm volatile(PART_SWAP PART_LOADS("%6", "%2", "%3", "%4", "%5") "s_waitcnt vmcnt(0)"
                     : PART_SWAP_OUT, PART_OUT(0) : "v"(o[0]), PART_SWAP_IN : "memory");
    else if constexpr (!STATS && N == 2)
        asm volatile(PART_SWAP PART_LOADS("%10", "%2", "%3", "%4", "%5") PART_LOADS("%11", "%6", "%7", "%8", "%9") "s_waitcnt vmcnt(0)"
                     : PART_SWAP_OUT, PART_OUT(0), PART_OUT(1) : "v"(o[0]), "v"(o[1]), PART_SWAP_IN : "memory");
    else if constexpr (!STATS)
        asm volatile(PART_SWAP PART_LOADS("%14", "%2", "%3", "%4", "%5") PART_LOADS("%15", "%6", "%7", "%8", "%9")
                     PART_LOADS("%16", "%10", "%11", "%12", "%13") "s_waitcnt vmcnt(0)"
                     : PART_SWAP_OUT, PART_OUT(0), PART_OUT(1), PART_OUT(2) : "v"(o[0]), "v"(o[1]), "v"(o[2]), PART_SWAP_IN : "memory");
    else if constexpr (N == 1)
        asm volatile(PART_SWAP PART_STAT("%6", "%8") PART_LOADS("%7", "%2", "%3", "%4", "%5") "s_waitcnt vmcnt(0)"
                     : PART_SWAP_OUT, PART_OUT(0), "=&v"(st[0]) : "v"(o[0]), "v"(ml[0]), PART_SWAP_IN : "memory");
    else if constexpr (N == 2)
        asm volatile(PART_SWAP PART_STAT("%10", "%14") PART_STAT("%11", "%15") PART_LOADS("%12", "%2", "%3", "%4", "%5")
                     PART_LOADS("%13", "%6", "%7", "%8", "%9") "s_waitcnt vmcnt(0)"
                     : PART_SWAP_OUT, PART_OUT(0), PART_OUT(1), "=&v"(st[0]), "=&v"(st[1]) : "v"(o[0]), "v"(o[1]), "v"(ml[0]), "v"(ml[1]), PART_SWAP_IN : "memory");
    else
        asm volatile(PART_SWAP PART_STAT("%14", "%20") PART_STAT("%15", "%21") PART_STAT("%16", "%22") PART_LOADS("%17", "%2", "%3", "%4", "%5")
                     PART_LOADS("%18", "%6", "%7", "%8", "%9") PART_LOADS("%19", "%10", "%11", "%12", "%13") "s_waitcnt vmcnt(0)"
                     : PART_SWAP_OUT, PART_OUT(0), PART_OUT(1), PART_OUT(2), "=&v"(st[0]), "=&v"(st[1]), "=&v"(st[2])
                     : "v"(o[0]), "v"(o[1]), "v"(o[2]), "v"(ml[0]), "v"(ml[1]), "v"(ml[2]), PART_SWAP_IN : "memory");
#undef PART_LOADS
#undef PART_STAT
#undef PART_SWAP
#undef PART_OUT
#undef PART_SWAP_OUT
#undef PART_SWAP_IN
}

// Split ks of KS of a row block: one wave's column block, res (unnormalised), M and Lsum (of the lane's query), against those of its
// fellows in the other splits; `at` is the column block's number in the launch.  One split owns the block (another one for each wave, so that
// its workgroup reads little): it keeps its own partial in registers, waits for the others' and adds them up (Hands).  True for a wave that
// has them all, with the results in res and Lsum.
//
// The workgroups of a row block are numbered so that the same XCD gets them all (but `apart`, whose partials go to the memory side at once): what is handed over
// is left in its L2, and loads at agent scope find what lies written in their own XCD's L2.
//
// What bounds it are trips within the XCD, about 0.4 us each when all workgroups make them at once: the partial is written, the offer seen, the partials and the exchange
// of the offer fetched together, 1.7 us of a layer where a merge kernel took 2.9 and a launch of the host (8B shape, 64 nodes, 1,024 keys, three splits: 32 layers
// 352 -> 331 us; 16 layers, whose caches lie closer, 10.8 -> 9.3 a layer; one of 40 heads 2,048 keys 12.8 -> 11.5).  Through the memory side only, as far fellows go, 336.
template <int DBLK>
__device__ __forceinline__ bool join_splits(const SplitBuf &sb, int64_t at, int KS, int ks, bool apart, int w, int lane, float c, float (&res)[16], float M, float &Lsum) {
    const int col = lane & 31;
    float4 *const o = sb.o + at * KS * 4 * 64 + lane;
    float2 *const ml = sb.ml + at * KS * 32 + col;
    // the members are the other splits in their order; the line of an offer more holds the claim
    u64 *const offers = sb.offers + at * KS * LINE_WORDS;
    const Hands<LINE_WORDS> hands = {offers, sb.marks + at * KS, offers + (KS - 1) * LINE_WORDS, sb.tag, KS - 1};
    const int owner = KS - 1 - (w >= KS ? w - KS : w);  // w % KS: four waves, two splits and more
    auto leave = [&]() {  // at the memory side
#pragma unroll
        for (int q = 0; q < 4; ++q) put16_agent(o + (ks * 4 + q) * 64, f32x4{res[4 * q], res[4 * q + 1], res[4 * q + 2], res[4 * q + 3]});
        if (lane < 32) put8_agent(ml + ks * 32, f32x2{M, Lsum});
        drain();
    };
    bool taking = false;
    if (ks == owner) {
        if (!hand_await(hands, lane, taking)) {
            leave();
            if (!hand_leave(hands, lane)) return false;
        }
    } else {
        const int me = ks - (ks > owner);
        if (!apart) {
#pragma unroll
            for (int q = 0; q < 4; ++q) *(f32x4 *)(o + (ks * 4 + q) * 64) = f32x4{res[4 * q], res[4 * q + 1], res[4 * q + 2], res[4 * q + 3]};
            if (lane < 32) *(f32x2 *)(ml + ks * 32) = f32x2{M, Lsum};
            drain();
            if (hand_offer(hands, me, lane)) return false;
        }
        leave();
        if (!hand_mark(hands, me, lane)) return false;
    }
    asm volatile("" ::: "memory");
    // Partial j of the others is split j + (j >= ks)'s.  All their statistics, and three partials at a time, are in flight together; the sum is over the
    // splits in their order, whoever makes it.
    const u64 take = ballot(taking), here = sb.tag | (xcc_id() + 1);
    u64 *const offer = offers + min(lane, KS - 2) * LINE_WORDS;
    u64 was = here;
    float acc[16], l = 0.f;
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[i] = 0.f;
    auto add = [&](auto n_c) __attribute__((always_inline)) {  // sized for every number of splits: branches for each partial cost 0.4 us
        constexpr int n = decltype(n_c)::value;
        constexpr bool one = n <= 3;  // all in one statement
        u64 st[n];
        const u64 *mp[n];
#pragma unroll
        for (int j = 0; j < n; ++j) mp[j] = (const u64 *)(ml + (j + (j >= ks)) * 32);
        if constexpr (!one)
#pragma unroll
            for (int j = 0; j < n; ++j) st[j] = get_agent((u64 *)mp[j]);
        float mu = M, f_own = 0.f, f[n];
        auto weights = [&]() {
#pragma unroll
            for (int j = 0; j < n; ++j) mu = fmaxf(mu, __builtin_bit_cast(f32x2, st[j]).x);
            mu = mu == -INFINITY ? 0.f : mu;
            f_own = __builtin_amdgcn_exp2f((M - mu) * c);
#pragma unroll
            for (int j = 0; j < n; ++j) f[j] = __builtin_amdgcn_exp2f((__builtin_bit_cast(f32x2, st[j]).x - mu) * c);
        };
        auto own = [&]() {
            l += Lsum * f_own;
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[i] += res[i] * f_own;
        };
        auto some = [&](auto j_c) __attribute__((always_inline)) {
            constexpr int j0 = decltype(j_c)::value, m = n - j0 < 3 ? n - j0 : 3;
            if constexpr (m > 0) {
                const float4 *op[m];
#pragma unroll
                for (int u = 0; u < m; ++u) op[u] = o + (j0 + u + (j0 + u >= ks)) * 4 * 64;
                f32x4 p[m][4];
                u64 none;
                if constexpr (one) get_partials<m, true>(op, mp, p, st, take, offer, u64x2{0, here}, was);
                else {
                    const u64 *no_stats[m];
                    u64 stats[m];
                    get_partials<m, false>(op, no_stats, p, stats, j0 == 0 ? take : 0, offer, u64x2{0, here}, j0 == 0 ? was : none);
                }
                if constexpr (j0 == 0) weights();
#pragma unroll
                for (int u = 0; u < m; ++u) {
                    if (j0 + u == ks) own();
                    l += __builtin_bit_cast(f32x2, st[j0 + u]).y * f[j0 + u];
#pragma unroll
                    for (int i = 0; i < 16; ++i) acc[i] += p[u][i >> 2][i & 3] * f[j0 + u];
                }
            }
        };
        some(std::integral_constant<int, 0>());
        some(std::integral_constant<int, 3>());
        some(std::integral_constant<int, 6>());
        if (ks == n) own();
    };
    using std::integral_constant;
    if (KS == 3) add(integral_constant<int, 2>());
    else if (KS == 4) add(integral_constant<int, 3>());
    else if (KS == 2) add(integral_constant<int, 1>());
    else if (KS == 5) add(integral_constant<int, 4>());
    else if (KS == 6) add(integral_constant<int, 5>());
    else if (KS == 7) add(integral_constant<int, 6>());
    else add(integral_constant<int, MAX_SPLITS - 1>());
    hand_settle(hands, lane, taking, was);
#pragma unroll
    for (int i = 0; i < 16; ++i) res[i] = acc[i];
    Lsum = l;
    return true;
}

// APART: the units past the last multiple of eight have their workgroups dealt one to an XCD in turn (a compilation of its own: the test took 0.17 us a launch).
template <int D, int NW, bool DIRECT, bool APART>
__global__ __launch_bounds__(64 * NW, 2) void attn_wave_kernel(AttnArgs a, int KS, SplitBuf sb) {
    static_assert((D == 128 || D == 64) && (NW == 4 || NW == 8) && (!DIRECT || (NW == 4 && D == 128)), "shape");
    constexpr int KSTEPS = D / 16, DBLK = D / 32;
    constexpr int K_PITCH = WaveTile<D>::K_PITCH, V_PITCH = WaveTile<D>::V_PITCH;
    const int G = sb.gd.G;
    // Workgroups are dealt to the 8 XCDs round-robin by linear id.  With the kv head in x (or in the unit's number, kv heads
    // first), every row block of a kv head lands on one XCD, where their number is a multiple of eight, and shares its L2 copy of that head's K/V; the splits
    // of a unit are eight apart.
    int b = blockIdx.z, h = blockIdx.x, ks = 0, rows = blockIdx.y, unit = 0;
    bool apart = false;  // this unit's are
    if constexpr (NW == 4) {
        unit = 8 * blockIdx.y + (blockIdx.x & 7);
        ks = blockIdx.x >> 3;
        if constexpr (APART)
            if ((int)blockIdx.y == sb.units >> 3) {
                const int i = (int)(blockIdx.x * sb.ks_magic >> 12);
                unit = (sb.units & ~7) + i;
                ks = blockIdx.x - i * KS;
                apart = true;
            }
        if (unit >= sb.units) return;
        const int t = __builtin_amdgcn_readfirstlane(sb.hd.div(unit));
        h = unit - t * sb.hd.G;
        b = __builtin_amdgcn_readfirstlane(sb.md.div(t));
        rows = t - b * sb.md.G;
    }
    // The four per-sequence words in one trip to memory: the compiler would fetch the others behind the test of the first.
    int n_raw = a.n_nodes[b], l_raw = a.prefix_len[b];
    u64 kp_raw = (u64)(uintptr_t)a.k_prefix[b], vp_raw = (u64)(uintptr_t)a.v_prefix[b];
    asm volatile("" : "+s"(n_raw), "+s"(l_raw), "+s"(kp_raw), "+s"(vp_raw));
    const int N = min(max(n_raw, 1), a.TT_cap);
    const int M = N * G;
    const int m0 = rows * 32;
    if (m0 >= M) return;
    const int L = max(l_raw, 0);
    const int Tk = L + N;
    const int nb = (Tk + ATT_KB - 1) / ATT_KB;

    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave index, known uniform
    const int half = lane >> 5, col = lane & 31;
    const int mq = m0 + col;
    const bool qvalid = mq < M;
    const int mr = qvalid ? mq : 0;  // rows past M read node 0: unused
    const int node = sb.gd.div(mr);
    const int hq = h * G + (mr - node * G);

    // LDS: NW private tiles during the loop, then the exchange area of the partial results
    extern __shared__ __attribute__((aligned(16))) unsigned char s_dyn[];
    __shared__ float s_m[NW][32], s_l[NW][32];
    __bf16 *kt = (__bf16 *)s_dyn + w * WaveTile<D>::ELEMS;   // staged layout (!DIRECT): padded rows
    __bf16 *vt = kt + WaveTile<D>::K_ELEMS;
    unsigned char *wtile = s_dyn + w * 2 * WD_STAGE;  // direct layout: two stages of (K tile, V tile)

    bf16x8 qreg[KSTEPS];
    {
        const __bf16 *qp = (const __bf16 *)a.q + (((int64_t)b * a.TT_cap + node) * a.Hq + hq) * D;
#pragma unroll
        for (int s = 0; s < KSTEPS; ++s) qreg[s] = *(const bf16x8 *)(qp + 16 * s + 8 * half);  // rows past M read node 0: unused
    }
    const u64 mask0 = a.anc_mask[((int64_t)b * a.TT_cap + node) * DT_MASK_WORDS];
    const u64 mask1 = a.anc_mask[((int64_t)b * a.TT_cap + node) * DT_MASK_WORDS + 1];

    f32x16 oacc[DBLK];
#pragma unroll
    for (int db = 0; db < DBLK; ++db)
#pragma unroll
        for (int i = 0; i < 16; ++i) oacc[db][i] = 0.f;
    float m_run = -INFINITY, l_run = 0.f;
    const float c = a.scale * 1.4426950408889634f;

    const gbf16p kpre = (gbf16p)(uintptr_t)kp_raw + (int64_t)h * a.kv_stride_head;
    const gbf16p vpre = (gbf16p)(uintptr_t)vp_raw + (int64_t)h * a.kv_stride_head;
    const gbf16p ktree = (gbf16p)a.k_tree + ((int64_t)b * a.TT_cap * a.Hkv + h) * D;
    const gbf16p vtree = (gbf16p)a.v_tree + ((int64_t)b * a.TT_cap * a.Hkv + h) * D;
    const int64_t stok = a.kv_stride_tok, stree = (int64_t)a.Hkv * D;
    const int kstep = KS * NW;  // the blocks are dealt round-robin over all waves of all splits
    // 64-wide heads keep their probabilities in 32 bits: as the sum of three bf16 numbers, 24 bits of significand, which
    // multiply the same V operand one after the other.  Error against 64-bit arithmetic over 1 to 8 sequences of 16 to 4,000
    // keys: 1.6616e-3 of the result, what the plain kernel has (the rounding of the result itself), against 2.0231e-3 with
    // probabilities rounded to bf16.  It costs a step of three sequences 0.6 us of 43.8, and where every compute unit has work
    // for several rounds a third: 16 sequences of 96 nodes and 2,000 keys 74 -> 100 us, 64 of 1,000 keys 188 -> 234.
    constexpr int PARTS = D == 64 ? 3 : 1;
    if constexpr (DIRECT) {
        // Blocks go straight from global memory into the wave's own LDS tiles (global_load_lds_dwordx4:
        // a wave's 64 x 16 B land contiguously), so no staging registers and no LDS-write instructions.  A tile is two
        // sub-tiles of 32 keys x 128 bytes, a load eight keys of one: whole cache lines.  No operand read has a bank conflict:
        //   K: chunk c (16 bytes) of row r sits at position c ^ (r / 2 % 8) of its 128 bytes (the permutation is applied on
        //      the global side);
        //   V: at c ^ 4 (r / 2 % 2), so that the transposing read's 4 rows x 64 B fall into four different groups of banks.
        // Two stages, one block asked for ahead.  (Two ahead were slower at every length, 11.3 us per layer against 10.9 at
        // 1,024 keys, 20.7 against 18.1 at 4,096.)
        const int krow = lane >> 3, cpos = lane & 7;
        u32 koffp[2][2], voffp[2];  // inside the prefix: byte offsets from the first of eight rows, even and odd eights; sub-tile
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            koffp[0][s] = (u32)(krow * stok + 8 * (cpos ^ (lane >> 4))) * 2u + 128u * s;
            koffp[1][s] = (u32)(krow * stok + 8 * (cpos ^ (4 + (lane >> 4)))) * 2u + 128u * s;
            voffp[s] = (u32)(krow * stok + 8 * (cpos ^ (((lane >> 4) & 1) << 2))) * 2u + 128u * s;
        }
        const int64_t rows8 = 16 * stok;  // bytes
        const bool small_stride = (int64_t)ATT_KB * stok * 2 < ((int64_t)1 << 31);
        // Every load is unconditional: keys past the end are read from the last valid row, their scores
        // are masked to -inf below, so the duplicated V rows contribute nothing.
        auto fetch = [&](int kb, int stage) {
            const ldsp kdst = (ldsp)wtile + stage * WD_STAGE;
            const ldsp vdst = kdst + WD_TILE;
            if (small_stride && kb * ATT_KB + ATT_KB <= L) {  // block inside the prefix (uniform test)
                gbytep kbase = (gbytep)(kpre + (int64_t)kb * ATT_KB * stok), vbase = (gbytep)(vpre + (int64_t)kb * ATT_KB * stok);
#pragma unroll
                for (int g = 0; g < 4; ++g) {
#pragma unroll
                    for (int s = 0; s < 2; ++s) {
                        __builtin_amdgcn_global_load_lds(kbase + koffp[g & 1][s], kdst + s * WD_SUB + g * 1024, 16, 0, 0);
                        __builtin_amdgcn_global_load_lds(vbase + voffp[s], vdst + s * WD_SUB + g * 1024, 16, 0, 0);
                    }
                    kbase += rows8;
                    vbase += rows8;
                }
            } else {                                           // block touching the tree keys or the end
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const int t = min(kb * ATT_KB + 8 * g + krow, Tk - 1);
                    const int64_t o = t < L ? (int64_t)t * stok : (int64_t)(t - L) * stree;
                    const gbf16p kp = (t < L ? kpre : ktree) + o + 8 * (cpos ^ (4 * (g & 1) + (lane >> 4)));
                    const gbf16p vp = (t < L ? vpre : vtree) + o + 8 * (cpos ^ (((lane >> 4) & 1) << 2));
#pragma unroll
                    for (int s = 0; s < 2; ++s) {
                        __builtin_amdgcn_global_load_lds((gbytep)(kp + 64 * s), kdst + s * WD_SUB + g * 1024, 16, 0, 0);
                        __builtin_amdgcn_global_load_lds((gbytep)(vp + 64 * s), vdst + s * WD_SUB + g * 1024, 16, 0, 0);
                    }
                }
            }
        };
        int kb = ks * NW + w, cur = 0;
        if (kb < nb) fetch(kb, 0);
        // operand read offsets (bytes)
        const u32 lds0 = (u32)(uintptr_t)(ldsp)wtile;
        u32 koff[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) koff[s] = lds0 + (u32)(col * 128 + (((2 * s + half) ^ ((col >> 1) & 7)) << 4));
        const int p16 = lane & 15, r0 = p16 >> 2, q4 = p16 & 3, grp = (lane >> 4) & 1;
        const u32 voff[2] = {lds0 + (u32)((4 * half + r0) * 128 + 64 * (r0 >> 1) + 32 * grp + 8 * q4),
                             lds0 + (u32)((4 * half + r0) * 128 + 64 * ((r0 >> 1) ^ 1) + 32 * grp + 8 * q4)};

        for (; kb < nb; kb += kstep, cur ^= 1) {
            __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0): this block has landed
            if (kb + kstep < nb) fetch(kb + kstep, cur ^ 1);  // the other stage was last read one block ago
            // Every operand of the block is asked for before it is needed (with one wave per SIMD nothing
            // else hides LDS latency): the eight K reads first, the sixteen transposing V reads between the
            // MFMAs of S^T, whose accumulator chain leaves the issue slots free.  K read s is followed by
            // 7 - s K reads and 2 s V reads when its MFMA comes up.
            const u32 stage = cur * WD_STAGE, va0 = voff[0] + stage, va1 = voff[1] + stage;
            bf16x8 ka[KSTEPS];
#pragma unroll
            for (int s = 0; s < 4; ++s) ka[s] = lds_load128_at<0>(koff[s] + stage);
#pragma unroll
            for (int s = 0; s < 4; ++s) ka[4 + s] = lds_load128_at<WD_SUB>(koff[s] + stage);
            bf16x4 vlo[DBLK][2], vhi[DBLK][2];
            f32x16 sacc;
#pragma unroll
            for (int i = 0; i < 16; ++i) sacc[i] = 0.f;
#define QK_STEP(s, db, st)                                                                  \
            lds_wait<7 + s>(ka[s]);                                                          \
            sacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[s], qreg[s], sacc, 0, 0, 0);   \
            vlo[db][st] = lds_load_tr4<WD_TILE + (db >> 1) * WD_SUB + 16 * st * 128>((db) & 1 ? va1 : va0);       \
            vhi[db][st] = lds_load_tr4<WD_TILE + (db >> 1) * WD_SUB + (16 * st + 8) * 128>((db) & 1 ? va1 : va0); \
            __builtin_amdgcn_sched_barrier(0);
            QK_STEP(0, 0, 0) QK_STEP(1, 1, 0) QK_STEP(2, 2, 0) QK_STEP(3, 3, 0)
            QK_STEP(4, 0, 1) QK_STEP(5, 1, 1) QK_STEP(6, 2, 1) QK_STEP(7, 3, 1)
#undef QK_STEP

            const int tbase = kb * ATT_KB;
            if (tbase + ATT_KB > L) {  // only blocks that contain tree keys (or the end) need the mask
                // 32-bit visibility window of this lane's query over keys tbase .. tbase+31: prefix keys
                // are visible, tree key j is visible iff bit j of the node's ancestor set (bits >= N are 0)
                const int off = tbase - L;  // uniform
                u32 vis;
                if (off >= 0) {
                    const u64 lo = off < 64 ? mask0 : mask1, hi = off < 64 ? mask1 : 0ull;
                    const int sh = off & 63;
                    vis = (u32)((lo >> sh) | (sh ? hi << (64 - sh) : 0ull));
                } else {
                    vis = ((u32)mask0 << (-off)) | ((1u << (-off)) - 1u);
                }
                vis >>= 4 * half;
#pragma unroll
                for (int i = 0; i < 16; ++i) sacc[i] = ((vis >> (8 * (i >> 2) + (i & 3))) & 1u) ? sacc[i] : -INFINITY;
            }
            float mloc = sacc[0];
#pragma unroll
            for (int i = 1; i < 16; ++i) mloc = fmaxf(mloc, sacc[i]);
            mloc = half_swap_max(mloc);
            // lazily moved reference maximum, as in the large-batch kernel
            const bool move = (mloc - m_run) * c > LAZY_LOG2;
            const float m_new = move ? mloc : m_run;
            const float m_use = m_new == -INFINITY ? 0.f : m_new;
            const float alpha = move ? __builtin_amdgcn_exp2f((m_run - m_use) * c) : 1.0f;
            const float nmc = -m_use * c;
            float psum = 0.f;
            bf16x8 pb[2];
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const float p = __builtin_amdgcn_exp2f(fmaf(sacc[i], c, nmc));
                psum += p;
                pb[i >> 3][i & 7] = (__bf16)p;
            }
            l_run = l_run * alpha + psum;
            // the running maximum moved away from a value for some query of this wave: not in the first block, whose
            // accumulators are zero
            const bool rescale = __ballot(move && m_run > -INFINITY);
            m_run = m_new;
            if (rescale) {
#pragma unroll
                for (int db = 0; db < DBLK; ++db)
#pragma unroll
                    for (int i = 0; i < 16; ++i) oacc[db][i] *= alpha;
            }

            // All V reads have landed (they had the whole softmax).  The wait is tied to the very registers
            // the reads fill, and the halves are joined only behind it: a register copy made before the
            // data arrives would copy the old contents.  The "memory" clobber also keeps the next
            // iteration's loads into this stage behind this block's reads.
            asm volatile("s_waitcnt lgkmcnt(0)"
                         : "+v"(vlo[0][0]), "+v"(vhi[0][0]), "+v"(vlo[1][0]), "+v"(vhi[1][0]), "+v"(vlo[2][0]), "+v"(vhi[2][0]),
                           "+v"(vlo[3][0]), "+v"(vhi[3][0]), "+v"(vlo[0][1]), "+v"(vhi[0][1]), "+v"(vlo[1][1]), "+v"(vhi[1][1]),
                           "+v"(vlo[2][1]), "+v"(vhi[2][1]), "+v"(vlo[3][1]), "+v"(vhi[3][1])
                         :
                         : "memory");
#pragma unroll
            for (int st = 0; st < 2; ++st)
#pragma unroll
                for (int db = 0; db < DBLK; ++db)
                    oacc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                        __builtin_shufflevector(vlo[db][st], vhi[db][st], 0, 1, 2, 3, 4, 5, 6, 7), pb[st], oacc[db], 0, 0, 0);
        }
    } else {
    // Loading role of a lane, the same for K and V: load i takes key RPL i + lane / LPR of the block, columns 8 dc ..
    // 8 dc + 7, so the LPR lanes of a row cover it (fully coalesced).
    // Inside the prefix the address is a uniform block base plus a fixed 32-bit lane offset.
    constexpr int LPR = D / 8, RPL = 64 / LPR, NLD = ATT_KB / RPL;
    const int kq = lane / LPR, dc = lane % LPR;
    u32 loff[NLD];
#pragma unroll
    for (int i = 0; i < NLD; ++i) loff[i] = (u32)((RPL * i + kq) * stok + 8 * dc) * 2u;
    const bool small_stride = (int64_t)ATT_KB * stok * 2 < ((int64_t)1 << 31);

    // Every load is unconditional, so the loads of a block are in flight together.  Keys
    // past the end are read from the last valid row; their scores are masked to -inf below, so
    // their probabilities are exactly 0 and the duplicated V rows contribute nothing.
    bf16x8 kn[NLD], vn[NLD];
    auto fetch = [&](int kb) {
        if (small_stride && kb * ATT_KB + ATT_KB <= L) {  // block inside the prefix (uniform test)
            const gbytep kbase = (gbytep)(kpre + (int64_t)kb * ATT_KB * stok);
            const gbytep vbase = (gbytep)(vpre + (int64_t)kb * ATT_KB * stok);
#pragma unroll
            for (int i = 0; i < NLD; ++i) {
                kn[i] = *(gbf16x8p)(kbase + loff[i]);
                vn[i] = *(gbf16x8p)(vbase + loff[i]);
            }
        } else {                                           // block touching the tree keys or the end
#pragma unroll
            for (int i = 0; i < NLD; ++i) {
                const int t = min(kb * ATT_KB + RPL * i + kq, Tk - 1);
                const int64_t o = (t < L ? (int64_t)t * stok : (int64_t)(t - L) * stree) + 8 * dc;
                kn[i] = gload8((t < L ? kpre : ktree) + o);
                vn[i] = gload8((t < L ? vpre : vtree) + o);
            }
        }
    };

    // All blocks of this wave; by_key: the second product in 32 bits, key by key (a loop of its own: a branch in the other one
    // made the compiler copy the accumulators in every block, 10 % of it)
    auto walk = [&](auto by_key) __attribute__((always_inline)) {
    int kb = ks * NW + w;
    if (kb < nb) fetch(kb);
    for (; kb < nb; kb += kstep) {
        // The prefetched block goes straight into the wave's two LDS tiles, both row-major, which
        // frees its registers for the next prefetch, issued before any arithmetic on this block.
#pragma unroll
        for (int i = 0; i < NLD; ++i) {
            const int r = RPL * i + kq;
            *(bf16x8 *)(kt + r * K_PITCH + 8 * dc) = kn[i];
            *(bf16x8 *)(vt + r * V_PITCH + 8 * dc) = vn[i];
        }
        if (kb + kstep < nb) fetch(kb + kstep);

        f32x16 sacc;
#pragma unroll
        for (int i = 0; i < 16; ++i) sacc[i] = 0.f;
#pragma unroll
        for (int s = 0; s < KSTEPS; ++s) {
            const bf16x8 ka = *(const bf16x8 *)(kt + col * K_PITCH + 16 * s + 8 * half);
            sacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka, qreg[s], sacc, 0, 0, 0);
        }

        const int tbase = kb * ATT_KB;
        if (tbase + ATT_KB > L) {  // only blocks that contain tree keys (or the end) need the mask
            // 32-bit visibility window of this lane's query over keys tbase .. tbase+31: prefix keys
            // are visible, tree key j is visible iff bit j of the node's ancestor set (bits >= N are 0)
            const int off = tbase - L;  // uniform
            u32 vis;
            if (off >= 0) {
                const u64 lo = off < 64 ? mask0 : mask1, hi = off < 64 ? mask1 : 0ull;
                const int sh = off & 63;
                vis = (u32)((lo >> sh) | (sh ? hi << (64 - sh) : 0ull));
            } else {
                vis = ((u32)mask0 << (-off)) | ((1u << (-off)) - 1u);
            }
            vis >>= 4 * half;
#pragma unroll
            for (int i = 0; i < 16; ++i) sacc[i] = ((vis >> (8 * (i >> 2) + (i & 3))) & 1u) ? sacc[i] : -INFINITY;
        }
        float mloc = sacc[0];
#pragma unroll
        for (int i = 1; i < 16; ++i) mloc = fmaxf(mloc, sacc[i]);
        mloc = half_swap_max(mloc);
        // lazily moved reference maximum, as in the large-batch kernel
        const bool move = (mloc - m_run) * c > LAZY_LOG2;
        const float m_new = move ? mloc : m_run;
        const float m_use = m_new == -INFINITY ? 0.f : m_new;
        const float alpha = move ? __builtin_amdgcn_exp2f((m_run - m_use) * c) : 1.0f;
        const float nmc = -m_use * c;
        float psum = 0.f;
        bf16x8 pb[PARTS][2];
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const float p = __builtin_amdgcn_exp2f(fmaf(sacc[i], c, nmc));
            psum += p;
            if constexpr (decltype(by_key)::value) sacc[i] = p;
            if constexpr (PARTS == 1) pb[0][i >> 3][i & 7] = (__bf16)p;
            else {
                float rest = p;
#pragma unroll
                for (int q = 0; q < PARTS; ++q) {  // the upper half of what is left; every remainder is exact
                    const u32 part = __float_as_uint(rest) & 0xFFFF0000u;
                    pb[q][i >> 3][i & 7] = __builtin_bit_cast(__bf16, (uint16_t)(part >> 16));
                    rest -= __uint_as_float(part);
                }
            }
        }
        l_run = l_run * alpha + psum;
        const bool rescale = __ballot(move && m_run > -INFINITY);  // (as above)
        m_run = m_new;
        if (rescale) {
#pragma unroll
            for (int db = 0; db < DBLK; ++db)
#pragma unroll
                for (int i = 0; i < 16; ++i) oacc[db][i] *= alpha;
        }

        // O^T += V^T P^T.  The A operand of lane (column d = 32db + col, half) holds, for e = 0..7,
        // V[key 16st + 8(e/4) + 4half + e%4][d]: two transposing LDS reads of 4 keys each.  In a
        // 16-lane group lane p = 4j+q points at key j of the quadruple, columns d0 + 4q..4q+3.
        if constexpr (!decltype(by_key)::value) {
            const int p16 = lane & 15;
            const __bf16 *vbase = vt + (4 * half + (p16 >> 2)) * V_PITCH + 16 * ((lane >> 4) & 1) + 4 * (p16 & 3);
#pragma unroll
            for (int db = 0; db < DBLK; ++db)
#pragma unroll
                for (int st = 0; st < 2; ++st) {
                    const bf16x4 lo = lds_read_tr4(vbase + (16 * st) * V_PITCH + 32 * db);
                    const bf16x4 hi = lds_read_tr4(vbase + (16 * st + 8) * V_PITCH + 32 * db);
                    const bf16x8 va = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
#pragma unroll
                    for (int q = 0; q < PARTS; ++q)
                        oacc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va, pb[q][st], oacc[db], 0, 0, 0);
                }
        } else {
            float *pt = (float *)kt;  // [32 keys][32 queries], in the place of the K tile, which has been read
            static_assert(ATT_KB * 32 * 4 <= WaveTile<D>::K_ELEMS * 2, "probabilities in the K tile");
            asm volatile("" ::: "memory");  // the tile changes its type: nothing moves across
#pragma unroll
            for (int i = 0; i < 16; ++i) pt[(8 * (i >> 2) + 4 * half + (i & 3)) * 32 + col] = sacc[i];
            __builtin_amdgcn_wave_barrier();
#pragma unroll 1
            for (int j = 0; j < ATT_KB; ++j) {
                const float p = pt[j * 32 + col];
#pragma unroll
                for (int db = 0; db < DBLK; ++db)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const bf16x4 v = *(const bf16x4 *)(vt + j * V_PITCH + 32 * db + 8 * q + 4 * half);
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            oacc[db][4 * q + e] = p != 0.f ? fmaf(p, (float)v[e], oacc[db][4 * q + e]) : oacc[db][4 * q + e];
                    }
            }
            asm volatile("" ::: "memory");
        }
    }
    };
    walk(std::false_type());
    if constexpr (PARTS > 1) {
        // An infinity or a NaN in V must not reach the queries that give its key no weight, and the parts of a probability must
        // not meet it with different signs.  Whatever it meets, it leaves an accumulator that is not finite: then the wave
        // starts again and takes its second products in 32 bits, key by key.
        float odd = 0.f;
#pragma unroll
        for (int db = 0; db < DBLK; ++db)
#pragma unroll
            for (int i = 0; i < 16; ++i) odd = fmaf(oacc[db][i], 0.f, odd);
        if (__builtin_amdgcn_ballot_w64(odd != 0.f)) {
            m_run = -INFINITY;
            l_run = 0.f;
#pragma unroll
            for (int db = 0; db < DBLK; ++db)
#pragma unroll
                for (int i = 0; i < 16; ++i) oacc[db][i] = 0.f;
            walk(std::true_type());
        }
    }

    }

    // ---- the partial results meet ----------------------------------------------------------------
    float l_tot = half_swap_sum(l_run);
    // Each wave's go where its own tiles were, which it alone reads: no barrier in front, and none between the two stages (with one
    // slice area for all, the first to end waited for the last before it wrote: per layer of the 8B shape 11.20 us at 1,024 keys
    // and 8.46 at 256, 11.12 and 8.30 so).  float4 slot (q, lane) of wave v at xv(v)[q*64 + lane], q = 4 db + i/4
    asm volatile("" ::: "memory");  // the tiles change their type: nothing moves across
    auto xv = [&](int v) { return (float4 *)(s_dyn + v * WaveArea<D, DIRECT>::BYTES); };
    if (NW == 8) {
        // stage A: wave w+4 hands its whole partial to wave w
        if (w >= 4) {
            if (half == 0) { s_m[w][col] = m_run; s_l[w][col] = l_tot; }
#pragma unroll
            for (int db = 0; db < DBLK; ++db)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    xv(w)[(db * 4 + q) * 64 + lane] =
                        make_float4(oacc[db][4 * q], oacc[db][4 * q + 1], oacc[db][4 * q + 2], oacc[db][4 * q + 3]);
        }
        __syncthreads();
        if (w < 4) {
            const float m2 = s_m[w + 4][col], l2 = s_l[w + 4][col];
            const float Mn = fmaxf(m_run, m2), Mu = Mn == -INFINITY ? 0.f : Mn;
            const float f1 = __builtin_amdgcn_exp2f((m_run - Mu) * c), f2 = __builtin_amdgcn_exp2f((m2 - Mu) * c);
#pragma unroll
            for (int db = 0; db < DBLK; ++db)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const float4 o = xv(w + 4)[(db * 4 + q) * 64 + lane];
                    oacc[db][4 * q] = oacc[db][4 * q] * f1 + o.x * f2;
                    oacc[db][4 * q + 1] = oacc[db][4 * q + 1] * f1 + o.y * f2;
                    oacc[db][4 * q + 2] = oacc[db][4 * q + 2] * f1 + o.z * f2;
                    oacc[db][4 * q + 3] = oacc[db][4 * q + 3] * f1 + o.w * f2;
                }
            l_tot = l_tot * f1 + l2 * f2;
            m_run = Mn;
        }
    }
    // stage B: waves 0..3; wave w < D/32 finishes output columns [32w, 32w+32)
    if (w < 4) {
        if (half == 0) { s_m[w][col] = m_run; s_l[w][col] = l_tot; }
#pragma unroll
        for (int db = 0; db < DBLK; ++db) {
            if (db == w) continue;
#pragma unroll
            for (int q = 0; q < 4; ++q)
                xv(w)[(db * 4 + q) * 64 + lane] =
                    make_float4(oacc[db][4 * q], oacc[db][4 * q + 1], oacc[db][4 * q + 2], oacc[db][4 * q + 3]);
        }
    }
    __syncthreads();
    if (w >= DBLK) return;
    // the fellows' shares in turn from the next wave on, all of them asked for before the first is used (behind a branch for each fellow they came two at
    // a time)
    float4 o[3][4];
    float mw[4], lw[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        mw[j] = s_m[(w + j) & 3][col];
        lw[j] = s_l[(w + j) & 3][col];
    }
#pragma unroll
    for (int j = 1; j < 4; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) o[j - 1][q] = xv((w + j) & 3)[(w * 4 + q) * 64 + lane];
    __builtin_amdgcn_sched_barrier(0);
    float Mx = fmaxf(fmaxf(mw[0], mw[1]), fmaxf(mw[2], mw[3]));
    const float Mu = Mx == -INFINITY ? 0.f : Mx;
    float f[4], Lsum = 0.f;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        f[j] = __builtin_amdgcn_exp2f((mw[j] - Mu) * c);
        Lsum += f[j] * lw[j];
    }
    float res[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) res[i] = 0.f;
#pragma unroll
    for (int db = 0; db < DBLK; ++db)  // own block (db == w) from registers; static indexing only
        if (db == w)
#pragma unroll
            for (int i = 0; i < 16; ++i) res[i] = oacc[db][i] * f[0];
#pragma unroll
    for (int j = 1; j < 4; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            res[4 * q] += o[j - 1][q].x * f[j];
            res[4 * q + 1] += o[j - 1][q].y * f[j];
            res[4 * q + 2] += o[j - 1][q].z * f[j];
            res[4 * q + 3] += o[j - 1][q].w * f[j];
        }
    if constexpr (NW == 4) {  // (eight waves take all keys of a unit)
        if (!join_splits<DBLK>(sb, (int64_t)unit * DBLK + w, KS, ks, apart, w, lane, c, res, Mx, Lsum)) return;
    }
    if (!qvalid) return;
    const float inv = Lsum > 0.f ? 1.0f / Lsum : 0.f;
    __bf16 *op = (__bf16 *)a.out + (((int64_t)b * a.TT_cap + node) * a.Hq + hq) * D + 32 * w;
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4) {
        bf16x4 o4;
#pragma unroll
        for (int e = 0; e < 4; ++e) o4[e] = (__bf16)(res[q4 * 4 + e] * inv);
        *(bf16x4 *)(op + 8 * q4 + 4 * half) = o4;
    }
}

// --------------------------------------------------------------- fp32 path, other head sizes --
// One workgroup per (node, head), four waves that take 64-key blocks in turn: lane j scores key j, the wave agrees on the
// running maximum, then lane c accumulates output columns c (and c + 64, NC = 2).  The waves' results meet in LDS.  What
// bounds it at the sizes it is meant for is trips to memory: the K row of a lane (16-byte loads, VEC) and half of the
// block's V rows are asked for together, the other half behind the scores.  One wave per (node, head) that walked all keys
// with 4-byte loads took 16.5 us on the tiny fp32 configuration (8 nodes, 4 heads, 136 keys).
template <typename T>
__device__ __forceinline__ float ld(const T *p);
template <>
__device__ __forceinline__ float ld<float>(const float *p) { return *p; }
template <>
__device__ __forceinline__ float ld<uint16_t>(const uint16_t *p) { return bf16_bits_to_float(*p); }
// sixteen bytes at any element address
__device__ __forceinline__ void ld16(const float *p, float *x) {
    const u32x4_any4 v = *(const u32x4_any4 *)p;
    x[0] = __uint_as_float(v.x); x[1] = __uint_as_float(v.y); x[2] = __uint_as_float(v.z); x[3] = __uint_as_float(v.w);
}
__device__ __forceinline__ void ld16(const uint16_t *p, float *x) {
    const u32x4_any2 v = *(const u32x4_any2 *)p;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        x[2 * i] = __uint_as_float(v[i] << 16);
        x[2 * i + 1] = __uint_as_float(v[i] & 0xFFFF0000u);
    }
}

template <typename T, int NC, bool VEC>
__global__ __launch_bounds__(256) void attn_simple_kernel(AttnArgs a) {
    const int node = blockIdx.x, hq = blockIdx.y, b = blockIdx.z, tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n_raw = a.n_nodes[b], l_raw = a.prefix_len[b];
    const T *kpre = (const T *)a.k_prefix[b], *vpre = (const T *)a.v_prefix[b];
    const int N = min(max(n_raw, 1), a.TT_cap);
    if (node >= N) return;
    const int D = a.D, G = a.Hq / a.Hkv, h = hq / G;
    const int L = max(l_raw, 0), Tk = L + N;
    const int64_t row = ((int64_t)b * a.TT_cap + node) * a.Hq + hq;
    const T *q = (const T *)a.q + row * D;
    const T *ktree = (const T *)a.k_tree + ((int64_t)b * a.TT_cap * a.Hkv + h) * D;
    const T *vtree = (const T *)a.v_tree + ((int64_t)b * a.TT_cap * a.Hkv + h) * D;
    kpre += (int64_t)h * a.kv_stride_head;
    vpre += (int64_t)h * a.kv_stride_head;
    const u64 mask0 = a.anc_mask[((int64_t)b * a.TT_cap + node) * DT_MASK_WORDS];
    const u64 mask1 = a.anc_mask[((int64_t)b * a.TT_cap + node) * DT_MASK_WORDS + 1];

    __shared__ __attribute__((aligned(16))) float s_q[128];
    __shared__ float s_m[4], s_l[4], s_o[4][128];
    if (tid < 128) s_q[tid] = tid < D ? ld(q + tid) : 0.f;
    __syncthreads();

    constexpr int PER = 16 / sizeof(T);  // elements of a 16-byte load
    constexpr int VB = 32;               // V rows in flight together
    float m_run = -INFINITY, l_lane = 0.f, o[NC];
#pragma unroll
    for (int i = 0; i < NC; ++i) o[i] = 0.f;
    for (int t0 = w * 64; t0 < Tk; t0 += 256) {
        const int t = t0 + lane, tc = min(t, Tk - 1);
        bool vis = t < Tk;
        if (vis && t >= L) {
            const int j = t - L;
            vis = ((j < 64 ? mask0 : mask1) >> (j & 63)) & 1ull;
        }
        const T *kp = tc < L ? kpre + (int64_t)tc * a.kv_stride_tok : ktree + (int64_t)(tc - L) * a.Hkv * D;
        // V rows j0 .. j0 + VB - 1 of the block, lane's columns (columns past D repeat the last one and are never stored,
        // rows past the end repeat the last one and weigh 0): unconditional, a load in a branch is waited for there
        float v[VB][NC];
        auto v_request = [&](int j0) {
#pragma unroll
            for (int u = 0; u < VB; ++u) {
                const int tj = min(t0 + j0 + u, Tk - 1);
                const T *vp = tj < L ? vpre + (int64_t)tj * a.kv_stride_tok : vtree + (int64_t)(tj - L) * a.Hkv * D;
#pragma unroll
                for (int i = 0; i < NC; ++i) v[u][i] = ld(vp + min(lane + 64 * i, D - 1));
            }
        };
        float d4[4] = {0.f, 0.f, 0.f, 0.f};
        bool first = true;
        int c0 = 0;
        if (VEC) {
            for (; c0 + 64 <= D; c0 += 64) {
                float kv[64];
#pragma unroll
                for (int u = 0; u < 64; u += PER) ld16(kp + c0 + u, kv + u);
                if (first) v_request(0);
                first = false;
                __builtin_amdgcn_sched_barrier(0);  // all requests before the first use
#pragma unroll
                for (int u = 0; u < 64; ++u) d4[u & 3] = fmaf(s_q[c0 + u], kv[u], d4[u & 3]);
            }
            for (; c0 + PER <= D; c0 += PER) {
                float kv[PER];
                ld16(kp + c0, kv);
#pragma unroll
                for (int u = 0; u < PER; ++u) d4[u & 3] = fmaf(s_q[c0 + u], kv[u], d4[u & 3]);
            }
        }
        for (; c0 < D; ++c0) d4[0] = fmaf(s_q[c0], ld(kp + c0), d4[0]);
        if (first) v_request(0);
        const float s = vis ? ((d4[0] + d4[1]) + (d4[2] + d4[3])) * a.scale : -INFINITY;
        const float m_new = fmaxf(m_run, wave_max(s));
        if (m_new == -INFINITY) continue;
        const float alpha = __expf(m_run - m_new);
        const float p = vis ? __expf(s - m_new) : 0.f;
        l_lane = l_lane * alpha + p;
#pragma unroll
        for (int i = 0; i < NC; ++i) o[i] *= alpha;
        m_run = m_new;
#pragma unroll
        for (int j0 = 0; j0 < 64; j0 += VB) {
            if (j0 > 0) {
                if (t0 + j0 >= Tk) break;
                v_request(j0);
            }
#pragma unroll
            for (int u = 0; u < VB; ++u) {
                const float pj = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(p), j0 + u));
#pragma unroll
                for (int i = 0; i < NC; ++i)
                    o[i] = pj != 0.f ? fmaf(pj, v[u][i], o[i]) : o[i];  // a hidden key's row is not even multiplied by 0
            }
        }
    }
    const float l_run = wave_sum(l_lane);
    if (lane == 0) { s_m[w] = m_run; s_l[w] = l_run; }
#pragma unroll
    for (int i = 0; i < NC; ++i) s_o[w][lane + 64 * i] = o[i];
    __syncthreads();
    if (tid >= D) return;
    const float M = fmaxf(fmaxf(s_m[0], s_m[1]), fmaxf(s_m[2], s_m[3])), Mu = M == -INFINITY ? 0.f : M;
    float lt = 0.f, ot = 0.f;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const float f = __expf(s_m[v] - Mu);
        lt = fmaf(s_l[v], f, lt);
        ot = fmaf(s_o[v][tid], f, ot);
    }
    const float res = lt > 0.f ? ot * (1.0f / lt) : 0.f;
    if (sizeof(T) == 4) ((float *)a.out)[row * D + tid] = res;
    else ((__bf16 *)a.out)[row * D + tid] = (__bf16)res;
}

// Heads of 64 and 128 in fp32: one workgroup per (node, head), eight waves, 32 keys of each in turn.  Sixteen lanes share a
// key, lane c of them columns 4c .. 4c+3 of every 64, so that K and V rows come in whole and a lane that has summed a score
// (four DPP rotations) has the V columns that it weighs: each group of sixteen lanes keeps a softmax of its own over every
// fourth key, nothing crosses groups before the end.  What bounds it is the chain of trips to memory, two: the words of
// the sequence (with the query), then all of a wave's K and V rows.  Tiny fp32 configuration (8 nodes, 4 heads, 136 keys):
// 8.7 us in the kernel above (64-key blocks of four waves, one key to a lane, 4-byte V loads), 4.6 here.
typedef const float __attribute__((address_space(1))) *gfloatp;
__device__ __forceinline__ void ld16(gfloatp p, float *x) {
    typedef const u32x4_any4 __attribute__((address_space(1))) *g16;
    const u32x4_any4 v = *(g16)p;
    x[0] = __uint_as_float(v.x); x[1] = __uint_as_float(v.y); x[2] = __uint_as_float(v.z); x[3] = __uint_as_float(v.w);
}
template <int CTRL>
__device__ __forceinline__ float row_rotate_add(float v) {
    return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}
template <int D>
__global__ __launch_bounds__(512) void attn_f32_kernel(AttnArgs a) {
    constexpr int C = D / 64, U = 8, W = 8;  // 16-byte pieces of a lane's row, keys of a group in flight, waves
    const int node = blockIdx.x, hq = blockIdx.y, b = blockIdx.z, tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6), grp = lane >> 4, col = (lane & 15) * 4;
    int n_raw = a.n_nodes[b], l_raw = a.prefix_len[b];
    const float *kpre = (const float *)a.k_prefix[b], *vpre = (const float *)a.v_prefix[b];
    const int h = hq / (a.Hq / a.Hkv);
    const int64_t row = ((int64_t)b * a.TT_cap + node) * a.Hq + hq;
    u64 mask0 = a.anc_mask[((int64_t)b * a.TT_cap + node) * DT_MASK_WORDS];
    u64 mask1 = a.anc_mask[((int64_t)b * a.TT_cap + node) * DT_MASK_WORDS + 1];
    float q[C][4];
#pragma unroll
    for (int i = 0; i < C; ++i) ld16((gfloatp)a.q + row * D + 64 * i + col, q[i]);
    // here, all at once (left alone, the words are read one behind the other, where they are first used)
    asm volatile("" : "+s"(n_raw), "+s"(l_raw), "+s"(kpre), "+s"(vpre), "+s"(mask0), "+s"(mask1));
    const int N = min(max(n_raw, 1), a.TT_cap);
    if (node >= N) return;
    const int L = max(l_raw, 0), Tk = L + N;
    const float *ktree = (const float *)a.k_tree + ((int64_t)b * a.TT_cap * a.Hkv + h) * D + col;
    const float *vtree = (const float *)a.v_tree + ((int64_t)b * a.TT_cap * a.Hkv + h) * D + col;
    kpre += (int64_t)h * a.kv_stride_head + col;
    vpre += (int64_t)h * a.kv_stride_head + col;
    const float c2 = a.scale * 1.4426950408889634f;

    float m_run = -INFINITY, l_run = 0.f, o[C][4];
#pragma unroll
    for (int i = 0; i < C; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) o[i][e] = 0.f;
    for (int t0 = w * (4 * U); t0 < Tk; t0 += W * 4 * U) {
        float k[U][C][4], v[U][C][4], s[U];
        const float *vp[U];
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const int t = min(t0 + 4 * j + grp, Tk - 1);
            const bool pre = t < L;
            const int64_t off = pre ? (int64_t)((u64)(u32)t * (u64)a.kv_stride_tok) : (int64_t)((t - L) * (a.Hkv * D));
            const float *kp = (pre ? kpre : ktree) + off;
            vp[j] = (pre ? vpre : vtree) + off;
#pragma unroll
            for (int i = 0; i < C; ++i) ld16((gfloatp)kp + 64 * i, k[j][i]);
        }
#pragma unroll
        for (int j = 0; j < U; ++j)
#pragma unroll
            for (int i = 0; i < C; ++i) ld16((gfloatp)vp[j] + 64 * i, v[j][i]);
        __builtin_amdgcn_sched_barrier(0);  // all requests before the first use
        float m_new = m_run;
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const int t = t0 + 4 * j + grp, tt = t - L;
            const u32 bit = (u32)((tt < 64 ? mask0 : mask1) >> (tt & 63)) & 1u;
            const bool vis = (t < Tk) & ((tt < 0) | (bit != 0u));
            float d = 0.f;
#pragma unroll
            for (int i = 0; i < C; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e) d = fmaf(q[i][e], k[j][i][e], d);
            d = row_rotate_add<0x128>(d);
            d = row_rotate_add<0x124>(d);
            d = row_rotate_add<0x122>(d);
            d = row_rotate_add<0x121>(d);
            s[j] = vis ? d * c2 : -INFINITY;
            m_new = fmaxf(m_new, s[j]);
        }
        const float m_ref = m_new == -INFINITY ? 0.f : m_new;  // a group without a visible key yet
        const float alpha = __builtin_amdgcn_exp2f(m_run - m_ref);
        l_run *= alpha;
#pragma unroll
        for (int i = 0; i < C; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) o[i][e] *= alpha;
        m_run = m_new;
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const float p = __builtin_amdgcn_exp2f(s[j] - m_ref);
            l_run += p;
#pragma unroll
            for (int i = 0; i < C; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    o[i][e] = s[j] != -INFINITY ? fmaf(p, v[j][i][e], o[i][e]) : o[i][e];  // a hidden key's row is not even multiplied by 0
        }
    }
    // the four groups of the wave, then the waves
    __shared__ __attribute__((aligned(16))) float s_o[W][D];
    __shared__ float s_m[W], s_l[W];
    const float M = wave_max(m_run), Mr = M == -INFINITY ? 0.f : M;
    const float f = __builtin_amdgcn_exp2f(m_run - Mr);
    auto over_groups = [&](float x) {
        x += __shfl_xor(x, 16, 64);
        return half_swap_sum(x);
    };
    const float l_wave = over_groups(l_run * f);
#pragma unroll
    for (int i = 0; i < C; ++i) {
        float4 r;
        r.x = over_groups(o[i][0] * f); r.y = over_groups(o[i][1] * f);
        r.z = over_groups(o[i][2] * f); r.w = over_groups(o[i][3] * f);
        if (grp == 0) *(float4 *)&s_o[w][64 * i + col] = r;
    }
    if (lane == 0) { s_m[w] = M; s_l[w] = l_wave; }
    __syncthreads();
    if (tid >= D) return;
    float Mt = s_m[0];
#pragma unroll
    for (int v = 1; v < W; ++v) Mt = fmaxf(Mt, s_m[v]);
    const float Mu = Mt == -INFINITY ? 0.f : Mt;
    float lt = 0.f, ot = 0.f;
#pragma unroll
    for (int v = 0; v < W; ++v) {
        const float g = __builtin_amdgcn_exp2f(s_m[v] - Mu);
        lt = fmaf(s_l[v], g, lt);
        ot = fmaf(s_o[v][tid], g, ot);
    }
    ((float *)a.out)[row * D + tid] = lt > 0.f ? ot * (1.0f / lt) : 0.f;
}

// ------------------------------------------------------------------------------- launchers --
// LDS beyond 64 KB has to be asked for, once per device (dt_init)
hipError_t attn_init() {
    hipError_t e = hipFuncSetAttribute((const void *)attn_wave_kernel<128, 8, false, false>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                       8 * WaveTile<128>::ELEMS * 2);
    if (e == hipSuccess)
        e = hipFuncSetAttribute((const void *)attn_wave_kernel<64, 8, false, false>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                8 * WaveTile<64>::ELEMS * 2);
    if (e == hipSuccess)
        e = hipFuncSetAttribute((const void *)attn_wave_kernel<128, 4, true, false>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                WD_LDS_BYTES);
    if (e == hipSuccess)
        e = hipFuncSetAttribute((const void *)attn_wave_kernel<128, 4, true, true>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                WD_LDS_BYTES);
    if (e == hipSuccess)
        e = hipFuncSetAttribute((const void *)attn_tile_kernel<128, 2>, hipFuncAttributeMaxDynamicSharedMemorySize, TILE_LDS_BYTES(2));
    if (e == hipSuccess)
        e = hipFuncSetAttribute((const void *)attn_tile_kernel<128, 4>, hipFuncAttributeMaxDynamicSharedMemorySize, TILE_LDS_BYTES(4));
    if (e == hipSuccess)
        e = hipFuncSetAttribute((const void *)attn_gang_kernel<128>, hipFuncAttributeMaxDynamicSharedMemorySize, TILE_LDS_BYTES(2));
    return e;
}

// scratch of the balanced large-batch schedule: (kv heads x slots per head) <= 2 x compute units
// slots, two partials of 128 rows with their marks and a count each
static size_t gang_slot_bytes(int D) { return 2 * ATT_MTILE * ((size_t)D * 4 + 8) + 3 * 8; }
static size_t gang_bytes(int D, int n_cu) { return (size_t)2 * n_cu * gang_slot_bytes(D); }

// scratch of one key split of the small-batch kernel, per (sequence, kv head, 32-row block)
static size_t wave_unit_bytes(int D) { return (size_t)(D / 32) * (4 * 64 * 16 + 32 * 8 + LINE_WORDS * 8 + 8); }

size_t attn_workspace_bytes(int batch, int TT_cap, int Hq, int D, int n_cu) {
    if (D != 128 && D != 64) return 0;
    const size_t units = (size_t)batch * ((TT_cap * Hq + 31) / 32 + Hq);
    const size_t w8 = units * wave_unit_bytes(D) * MAX_SPLITS, g = D == 128 ? gang_bytes(D, n_cu) : 0;
    const size_t cap = (size_t)256 << 20;
    const size_t want = w8 > g ? w8 : g;
    return want < cap ? want : cap;
}

// Over how many workgroups the keys of a (sequence, kv head, 32-row block) are dealt: nb blocks of 32 keys, `units` such row blocks.
// At most one workgroup per compute unit, and MAX_SPLITS.  Split, the four waves of a workgroup take ceil(nb / 4 KS) rounds of about 0.75 us (0.84 of
// 64-wide heads), and the exchange costs the more the more partials an owner reads: from four splits on each workgroup owns one column block or none.
// Unsplit, eight waves share the four SIMDs, 0.55 us for every four blocks, and there is nothing to exchange.  Whatever is cheapest by that, in 1/100 us, from six
// blocks on.
// us per layer, 16 layers, unsplit | two | three | four | eight splits:
//   128-wide heads, 4 units: 5 blocks 6.6 | 6.6 | 6.7 | 6.8 | 7.4, 7: 7.1 | 6.3 | 6.6 | 6.5 | 7.4, 32: 12.5 | 8.9 | 8.4 | 7.8 | 8.0, 63: 18.2 | 11.3 | 10.2 | 9.0 | 8.7;
//     64 units: 7: 7.7 | 7.1 | 7.6 | 7.3, 9: 8.0 | 8.1 | 7.7 | 7.6, 13: 9.6 | 8.4 | 8.4 | 7.5, 34: 13.0 | 10.2 | 9.3 | 9.1, 127: 33.2 | 20.6 | 16.5 | 14.3;
//     128 units: 7: 7.8 | 7.6, 9: 8.4 | 8.4, 11: 8.6 | 8.6, 13: 9.8 | 8.6, 34: 13.2 | 10.6;
//   64-wide heads, 28 units: 7: 6.1 | 6.4 | 6.6 | 6.4 | 7.2, 11: 6.5 | 7.1 | 6.6 | 6.6 | 7.2, 15: 7.5 | 7.1 | 7.3 | 6.7 | 7.2, 46: 12.0 | 10.7 | 9.3 | 8.6 | 8.4;
//     128 units: 10: 6.5 | 7.4, 15: 7.8 | 7.8, 26: 8.8 | 9.3, 46: 12.1 | 10.9.
// (With a merge kernel behind them, splits paid from 9 to 13 blocks on, 29 to 60 of 64-wide heads: 64 units of 13 blocks 9.8, of 34 10.8, 28 units of 46 9.8.)
static int wave_splits(int D, int64_t units, int64_t nb) {
    const int most = (int)std::min<int64_t>(MAX_SPLITS, 256 / units);
    auto cost = [&](int64_t n) -> int64_t {
        if (n == 1) return 55 * ((nb + 3) / 4);
        const int64_t rounds = (nb + 4 * n - 1) / (4 * n);
        return (D == 128 ? 25 + 75 * rounds : 80 + 84 * rounds) + (n > 4 ? 20 + 15 * (n - 4) : 5 * (n - 2));
    };
    int best = 1;
    for (int n = 2; n <= most && nb > 5; ++n)
        if (cost(n) < cost(best)) best = n;
    return best;
}

// 32-key blocks of the longest sequence
static int64_t max_blocks(const AttnArgs &a) { return ((int64_t)a.max_prefix_len + a.TT_cap + ATT_KB - 1) / ATT_KB; }

// 128-wide heads: which kernel, by what the caller allows for (max_prefix_len, TT_cap; in a step that is captured once the most that any replay will have):
// units of (sequence, kv head, 32 rows), tiles of (sequence, kv head, 128 rows), blocks of 32 keys of the longest sequence.
//   1. up to 256 units:                                                    small-batch
//   2. up to 144 tiles and 56 blocks, and up to 320 units (400 beyond 32 blocks): small-batch
//   3. up to 40 blocks, 56 where every tile has a compute unit to itself:   whole tiles, four of K and V in LDS where it has, else two
//   4. otherwise, if the plan fits:                                        balanced (if not, as 3, or with fewer than 128 tiles as 1)
// us per layer, all sequences as long as said, or from a quarter of it up ("ragged"); 8B shape and 64 nodes unless said.
//   1: every unit has a compute unit.  Small-batch | balanced | whole: 4 sequences of 40 keys 7 | 9 | 9, 400 12 | 15 | 16, 2,400 26 | 40 | 47, 4,000 36 | 35 | 70; 32 heads without groups,
//      4 of 2,400 33 | 40 | 45, 8 of 32 nodes 54 | 66 | 65.  Longer ones gain by the schedule, 8,000 keys 62 | 55, 3 of 12,000 81 | 63, and stay: the lengths are bounds, and under a
//      bound that far above them the short ones would lose more.
//   3: four row blocks share a key block, and short sequences are not worth cutting, which the schedule finds too, in 1 us.  Balanced | whole: 32 of the 70B shape, ragged 200
//      keys 42 | 31, 1,100 73 | 67; 54 of 40 heads without groups 400 153 | 138, 1,100 316 | 289; 16 of them 1,100 103 | 96, 1,600 136 | 134, 2,400 181 | 199.  A compute unit to each
//      tile, caches from memory, balanced | whole with two | with four tiles in LDS (means over 4 to 14 sequences, 20 of 2 kv heads, 6 of 32): ragged 400 18.5 | 17.0 | 16.6, 1,100 32.3 | 30.8 | 27.1, 1,600 36.0 | 39.0 |
//      32.9, 2,400 46.8 | 56.9 | 46.9; equal 1,600 43.0 | 43.5 | 37.2.
//   4: small-batch | balanced: 5 sequences (320 units) 1,600 keys 33 | 30, 2,400 44 | 30; 4 of 112 nodes (448) 4,000 66 | 57; whole | balanced: 64 of 256 to 4,096 keys 295 | 231.
//   2: a compromise between batches that these bounds do not tell apart.  Where sequences end early or their trees are smaller than the largest, the units that are left have a
//      compute unit each, and a few tiles take as long as the longest sequence; where all are equal, whole tiles are ahead.  Small-batch | whole, from the best to the worst of the rule:
//      260 to 320 units ragged 8.2 | 11.5, 12.1 | 17.2, 16.6 | 20.5, 21.5 | 20.7, 13.0 | 10.0 (22 shapes 0.70 to 1.3 times as long, 0.95 on average); 336 to 400 beyond 32 blocks
//      ragged 15.4 | 21.0, 19.8 | 22.8, 22.4 | 25.6, equal 28.4 | 25.9.  Not taken: 336 to 400 up to 32 blocks 17.1 | 15.8, 13.2 | 11.1; 448 to 512 22.7 | 23.2, 25.5 | 22.7, equal 39.0 | 33.7.
#define SMALL_UNITS 256
#define FEW_TILES 144
#define FEW_TILES_UNITS 320        // at any length
#define FEW_TILES_UNITS_LONG 400   // beyond FEW_TILES_BLOCKS
#define FEW_TILES_BLOCKS 32
#define WHOLE_BLOCKS 40
#define WHOLE_BLOCKS_ONE 56

// The small-batch kernel.
template <int D>
static int wave_launch(const AttnArgs &a, hipStream_t st, hipError_t *err) {
    const int G = a.Hq / a.Hkv;
    const int mblocks = (a.TT_cap * G + 31) / 32;
    const int64_t units = (int64_t)a.batch * a.Hkv * mblocks;
    int KS = wave_splits(D, units, max_blocks(a));
    const size_t per_split = (size_t)units * wave_unit_bytes(D);
    if (KS > 1 && (!a.ws || (size_t)KS * per_split > a.ws_bytes)) KS = a.ws ? (int)(a.ws_bytes / per_split) : 1;
    if (KS < 1) KS = 1;
    SplitBuf sb = {};
    sb.gd = group_div(G);
    if (KS > 1) {  // several workgroups per unit: four waves each
        const size_t parts = (size_t)units * (D / 32) * KS;
        sb.offers = (u64 *)a.ws;
        sb.o = (float4 *)(sb.offers + parts * LINE_WORDS);
        sb.ml = (float2 *)(sb.o + parts * 4 * 64);
        sb.marks = (u64 *)(sb.ml + parts * 32);
        sb.tag = launch_tag();
        sb.hd = group_div(a.Hkv);
        sb.md = group_div(mblocks);
        sb.units = (int)units;
        sb.ks_magic = (u32)((4096 + KS - 1) / KS);
        const dim3 grid(8 * KS, (unsigned)((units + 7) / 8));
        auto go = [&](auto kernel, size_t lds) { launch_kernel(KID_ATTN, st, kernel, grid, dim3(256), lds, a, KS, sb); };
        // Where an XCD has no compute unit for one more unit, the last of them, fewer than eight, are spread over all (84 units of 64-wide heads in
        // three splits of 127 blocks 18.1 us with 33 workgroups on an XCD, 15.8 so; 4 units of 7 blocks, spread 7.7, on four XCDs 6.6).
        const bool apart = (units + 7) / 8 * KS * 8 > a.n_cu;
        if constexpr (D == 128) {  // one workgroup per compute unit (128 KB of LDS)
            if (apart) go(attn_wave_kernel<D, 4, true, true>, WD_LDS_BYTES);
            else go(attn_wave_kernel<D, 4, true, false>, WD_LDS_BYTES);
        } else {
            if (apart) go(attn_wave_kernel<D, 4, false, true>, 4 * WaveTile<D>::ELEMS * 2);
            else go(attn_wave_kernel<D, 4, false, false>, 4 * WaveTile<D>::ELEMS * 2);
        }
    } else {       // one workgroup per unit: eight waves (two per SIMD)
        const dim3 grid(a.Hkv, mblocks, a.batch);
        launch_kernel(KID_ATTN, st, attn_wave_kernel<D, 8, false, false>, grid, dim3(512), 8 * WaveTile<D>::ELEMS * 2, a, KS, sb);
    }
    *err = hipGetLastError();
    return *err == hipSuccess ? DT_OK : DT_ERR_HIP;
}

int attn_launch(const AttnArgs &a, hipStream_t st, hipError_t *err) {
    *err = hipSuccess;
    if (a.batch <= 0) return DT_OK;
    const bool mfma = a.dtype == DT_BF16 && (a.D == 128 || a.D == 64) && a.kv_stride_tok % 8 == 0 && a.kv_stride_head % 8 == 0;
    if (!mfma) {
        if (a.D > 128) return DT_ERR_LIMIT;
        const dim3 grid(a.TT_cap, a.Hq, a.batch);
        auto go = [&](auto kernel) { launch_kernel(KID_ATTN, st, kernel, grid, dim3(256), 0, a); };
        // 16-byte loads of a K row need no alignment, only a row that is long enough for them to be worth it
        if (a.dtype == DT_BF16) {
            if (a.D > 64) go(attn_simple_kernel<uint16_t, 2, true>);
            else if (a.D >= 8) go(attn_simple_kernel<uint16_t, 1, true>);
            else go(attn_simple_kernel<uint16_t, 1, false>);
        } else if (a.D == 64 || a.D == 128) {
            if (a.D == 64) launch_kernel(KID_ATTN, st, attn_f32_kernel<64>, grid, dim3(512), 0, a);
            else launch_kernel(KID_ATTN, st, attn_f32_kernel<128>, grid, dim3(512), 0, a);
        } else {
            if (a.D > 64) go(attn_simple_kernel<float, 2, true>);
            else if (a.D >= 4) go(attn_simple_kernel<float, 1, true>);
            else go(attn_simple_kernel<float, 1, false>);
        }
        *err = hipGetLastError();
        return *err == hipSuccess ? DT_OK : DT_ERR_HIP;
    }
    const int G = a.Hq / a.Hkv;
    const int mtiles = (a.TT_cap * G + ATT_MTILE - 1) / ATT_MTILE;
    const int base_wgs = a.batch * a.Hkv * mtiles;
    // 64-wide heads take the small-batch kernel at every batch: the
    // large-batch tiles are laid out for 128 columns, and against the plain kernel (the same call on a cache whose strides keep
    // it off the matrix cores) it is ahead at both ends, one sequence of 8 nodes and 40 keys 5.1 us against 7.5, 3 of 64 and
    // 1,500 12.9 against 206, 64 of 128 and 4,000 455 against 19,500.
    if (a.D == 64) return wave_launch<64>(a, st, err);
    // The balanced schedule needs a lane for every sequence and a slot for every tile count.
    const int P = 2 * a.n_cu / a.Hkv;
    const bool gang = a.batch <= 64 && mtiles <= 63 && P >= mtiles * (mtiles + 1) / 2 && a.ws &&
                      (size_t)a.Hkv * P * gang_slot_bytes(a.D) <= a.ws_bytes;
    const int mblocks = (a.TT_cap * G + 31) / 32;
    const int64_t units = (int64_t)a.batch * a.Hkv * mblocks;
    if (units <= SMALL_UNITS || (base_wgs < 128 && !gang)) return wave_launch<128>(a, st, err);
    const bool one = base_wgs <= a.n_cu;
    if (base_wgs <= FEW_TILES && max_blocks(a) <= WHOLE_BLOCKS_ONE &&
        units <= (max_blocks(a) > FEW_TILES_BLOCKS ? FEW_TILES_UNITS_LONG : FEW_TILES_UNITS))
        return wave_launch<128>(a, st, err);
    if (!gang || max_blocks(a) <= (one ? WHOLE_BLOCKS_ONE : WHOLE_BLOCKS)) {
        const dim3 grid(a.Hkv, mtiles, a.batch);
        if (one) launch_kernel(KID_ATTN, st, attn_tile_kernel<128, 4>, grid, dim3(256), TILE_LDS_BYTES(4), a, group_div(G));
        else launch_kernel(KID_ATTN, st, attn_tile_kernel<128, 2>, grid, dim3(256), TILE_LDS_BYTES(2), a, group_div(G));
        *err = hipGetLastError();
        return *err == hipSuccess ? DT_OK : DT_ERR_HIP;
    }
    const size_t slots = (size_t)a.Hkv * P;
    GangPartial part;
    part.o = (u64 *)a.ws;
    part.ml = part.o + slots * 2 * ATT_MTILE * (a.D / 2);
    part.count = part.ml + slots * 2 * ATT_MTILE;
    part.tag = launch_tag();
    launch_kernel(KID_ATTN, st, attn_gang_kernel<128>, dim3(a.Hkv, P), dim3(256), TILE_LDS_BYTES(2), a, group_div(G), P, part);
    *err = hipGetLastError();
    return *err == hipSuccess ? DT_OK : DT_ERR_HIP;
}

}  // namespace dt
