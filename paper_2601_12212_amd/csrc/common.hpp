// Device-side helpers shared by the gfx950 kernels: order-preserving keys, wave64
// reductions, bf16 access.  Wavefront size is 64 everywhere.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#define DT_WAVE 64

namespace dt {

typedef unsigned long long u64;
typedef uint32_t u32;

// ---- order-preserving integer image of a float (larger float <=> larger key) ----------
// -0 is folded onto +0 so that the integer order agrees with the float order exactly.
__device__ __forceinline__ u32 ord32(float f) {
    u32 u = __float_as_uint(f);
    if (u == 0x80000000u) u = 0u;
    return u ^ ((u >> 31) ? 0xFFFFFFFFu : 0x80000000u);
}
__device__ __forceinline__ float unord32(u32 k) {
    u32 u = (k & 0x80000000u) ? (k ^ 0x80000000u) : ~k;
    return __uint_as_float(u);
}
// 64-bit key of (value, index): larger value first, then SMALLER index.  Keys of distinct
// indices are distinct, so "greater key" is a strict total order.
__device__ __forceinline__ u64 make_key(float v, u32 idx) {
    return ((u64)ord32(v) << 32) | (u64)(0xFFFFFFFFu - idx);
}
__device__ __forceinline__ float key_val(u64 k) { return unord32((u32)(k >> 32)); }
__device__ __forceinline__ u32 key_idx(u64 k) { return 0xFFFFFFFFu - (u32)k; }

__device__ __forceinline__ float bf16_bits_to_float(uint16_t b) { return __uint_as_float((u32)b << 16); }

// 16 bytes of a logit row.  The address is only known to be a multiple of the element size: one load all the same (the
// hardware takes any address), so a row of an odd vocabulary streams like an aligned one.  Non-temporal: a step reads a
// logit once, and lines that do not displace each other in the caches on the way stream faster (1.25 GB of target rows:
// 192 us, 6.5 TB/s, against 207 us).
typedef u32 u32x4_any2 __attribute__((ext_vector_type(4), aligned(2)));
typedef u32 u32x4_any4 __attribute__((ext_vector_type(4), aligned(4)));
// KEEP: left in the caches, to be read again from the same XCD: fp32 rows in calls of rows on their own, both passes in one launch.  On rows that are new to each call, without | with: from
// memory (1.2 GB of them in turn) 61 of 50,001 entries 9.5 | 9.4 us, 28 of 128,256 10.3 | 9.9, 144 of 50,001 13.5 | 12.7, 120 of 128,256 19.3 | 18.0; from the last-level cache 9.7 | 9.0,
// 10.9 | 9.5, 13.5 | 12.3; the call and what has just written them: a product 59.0 | 59.0, 66.9 | 67.5, 91 | 90, 210 | 206, a conversion from bf16 16.5 | 16.9, 18.0 | 18.1, 22.7 | 22.7, 35.2 | 31.0, a copy from
// memory 15.6 | 16.5, 17.5 | 18.0, 26.4 | 24.7, 43 | 39.  (The same rows again 8.0 | 7.8.)  Not in bf16: from memory 10 of 128,256 7.2 | 7.7, 44 9.2 | 9.5, 61 of 50,001 8.0 | 8.4, 112 of 36,000 8.5 | 8.8;
// from the last level 7.3 | 7.4, 9.3 | 9.3, 8.2 | 8.1, 8.9 | 8.6, behind a copy 28 of 128,256 14.2 | 14.6.  Not in a step: left in the caches, the draft rows displace the keys and values that the attention behind them finds on the memory side,
// 11.4 us a launch against 10.45, a step of the 8B shape over 16 input sets 36.8 us against 35.3; a tree level by level takes 65.1 us and 64.6.
template <bool KEEP = false>
__device__ __forceinline__ uint4 load16(const uint16_t *p) {
    const u32x4_any2 v = KEEP ? *(const u32x4_any2 *)p : __builtin_nontemporal_load((const u32x4_any2 *)p);
    return make_uint4(v.x, v.y, v.z, v.w);
}
template <bool KEEP = false>
__device__ __forceinline__ uint4 load16(const float *p) {
    const u32x4_any4 v = KEEP ? *(const u32x4_any4 *)p : __builtin_nontemporal_load((const u32x4_any4 *)p);
    return make_uint4(v.x, v.y, v.z, v.w);
}

// A bf16 row of an odd vocabulary at an odd two-byte address is read from one entry before its first on (the last of the row before, masked), at
// multiples of four bytes: the loads of such rows took more than twice as long, those at four-byte addresses as long as aligned ones (4,324
// target rows of 9,664 / 9,665 / 9,666 entries 16.1 / 27.0 / 17.6 us, 1,024 of 128,256 / 128,257 / 128,258 40.4 / 54.0 / 39.8; 9,665 and 128,257 so 17.7 and 39.7).
// Everything that finds a place in the row by chunk, lane and group counts from there.  (An even vocabulary may end with its last chunk; the
// first row has nothing before it.)
__device__ __forceinline__ int row_shift(const void *logits, bool bf16, int V, int64_t row_stride, int64_t g) {
    return bf16 && (V & 1) && V >= 8 && g > 0 ? (int)(((uintptr_t)logits >> 1) + (uint64_t)(g * row_stride)) & 1 : 0;
}

// ---- wave64 primitives -------------------------------------------------------------------
__device__ __forceinline__ int lane_id() { return (int)(threadIdx.x & 63); }

__device__ __forceinline__ u32 lanes_below(u64 mask) {  // number of set bits of mask below this lane
    return __builtin_amdgcn_mbcnt_hi((u32)(mask >> 32), __builtin_amdgcn_mbcnt_lo((u32)mask, 0u));
}

// Wave-wide reductions with DPP row shifts and row broadcasts: six VALU steps, no LDS
// traffic.  The total lands in lane 63 and is broadcast from there, so the result is uniform.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ int dpp_mov(int ident, int v) {
    return __builtin_amdgcn_update_dpp(ident, v, CTRL, ROW_MASK, 0xf, false);
}
#define DT_DPP_REDUCE(v, ident, OP, TO_I, FROM_I)                          \
    v = OP(v, FROM_I(dpp_mov<0x111, 0xf>(TO_I(ident), TO_I(v))));          \
    v = OP(v, FROM_I(dpp_mov<0x112, 0xf>(TO_I(ident), TO_I(v))));          \
    v = OP(v, FROM_I(dpp_mov<0x114, 0xf>(TO_I(ident), TO_I(v))));          \
    v = OP(v, FROM_I(dpp_mov<0x118, 0xf>(TO_I(ident), TO_I(v))));          \
    v = OP(v, FROM_I(dpp_mov<0x142, 0xa>(TO_I(ident), TO_I(v))));          \
    v = OP(v, FROM_I(dpp_mov<0x143, 0xc>(TO_I(ident), TO_I(v))));

__device__ __forceinline__ float f_add(float a, float b) { return a + b; }
__device__ __forceinline__ u32 u_max(u32 a, u32 b) { return a > b ? a : b; }
__device__ __forceinline__ int i_max(int a, int b) { return a > b ? a : b; }
__device__ __forceinline__ int i_add(int a, int b) { return a + b; }
__device__ __forceinline__ int id_i(int x) { return x; }
__device__ __forceinline__ int u2i(u32 x) { return (int)x; }
__device__ __forceinline__ u32 i2u(int x) { return (u32)x; }

__device__ __forceinline__ float wave_max(float v) {
    DT_DPP_REDUCE(v, -INFINITY, fmaxf, __float_as_int, __int_as_float)
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}
__device__ __forceinline__ float wave_sum(float v) {
    DT_DPP_REDUCE(v, 0.f, f_add, __float_as_int, __int_as_float)
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}
__device__ __forceinline__ u32 wave_max_u32(u32 v) {
    DT_DPP_REDUCE(v, 0u, u_max, u2i, i2u)
    return (u32)__builtin_amdgcn_readlane((int)v, 63);
}
__device__ __forceinline__ int wave_max_i32(int v) {
    DT_DPP_REDUCE(v, (int)0x80000000, i_max, id_i, id_i)
    return __builtin_amdgcn_readlane(v, 63);
}
__device__ __forceinline__ int wave_sum_i32(int v) {
    DT_DPP_REDUCE(v, 0, i_add, id_i, id_i)
    return __builtin_amdgcn_readlane(v, 63);
}
// inclusive prefix sum over the lanes of a wave (the same row shifts and row broadcasts)
__device__ __forceinline__ int wave_scan_incl_i32(int v) {
    DT_DPP_REDUCE(v, 0, i_add, id_i, id_i)
    return v;
}
// the same in double (two moves a step instead of two trips through LDS)
__device__ __forceinline__ double wave_scan_incl_f64(double v) {
#define STEP(CTRL, ROWS)                                                                           \
    v += __hiloint2double(dpp_mov<CTRL, ROWS>(0, __double2hiint(v)), dpp_mov<CTRL, ROWS>(0, __double2loint(v)));
    STEP(0x111, 0xf) STEP(0x112, 0xf) STEP(0x114, 0xf) STEP(0x118, 0xf) STEP(0x142, 0xa) STEP(0x143, 0xc)
#undef STEP
    return v;
}
// 64-bit maximum: the high words first, then the low words of the lanes that hold that high word.
__device__ __forceinline__ u64 wave_max_u64(u64 v) {
    const u32 hi = wave_max_u32((u32)(v >> 32));
    const u32 lo = wave_max_u32((u32)(v >> 32) == hi ? (u32)v : 0u);
    return ((u64)hi << 32) | lo;
}
__device__ __forceinline__ u64 shfl_xor_u64(u64 v, int o) {
    u32 lo = __shfl_xor((u32)v, o, 64), hi = __shfl_xor((u32)(v >> 32), o, 64);
    return ((u64)hi << 32) | lo;
}
__device__ __forceinline__ u64 readlane_u64(u64 v, int lane) {
    u32 lo = __builtin_amdgcn_readlane((u32)v, lane), hi = __builtin_amdgcn_readlane((u32)(v >> 32), lane);
    return ((u64)hi << 32) | lo;
}

__device__ __forceinline__ double readlane_f64(double v, int lane) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane), __builtin_amdgcn_readlane(__double2loint(v), lane));
}

// How many of the keys that a wave holds lie above t (uniform).  The compares go to scalar register pairs of their own, four
// at a time (the compiler's sequence sends each through VCC and waits for it before the next).
template <int G>
__device__ __forceinline__ int count_above(const u32 (&key)[G], u32 t) {
    int c = 0;
    if constexpr (G % 4 == 0) {
#pragma unroll
        for (int q = 0; q < G; q += 4) {
            u64 m0, m1, m2, m3;
            asm("v_cmp_lt_u32_e64 %0, %8, %4\n\tv_cmp_lt_u32_e64 %1, %8, %5\n\tv_cmp_lt_u32_e64 %2, %8, %6\n\tv_cmp_lt_u32_e64 %3, %8, %7"
                : "=&s"(m0), "=&s"(m1), "=&s"(m2), "=&s"(m3)
                : "v"(key[q]), "v"(key[q + 1]), "v"(key[q + 2]), "v"(key[q + 3]), "s"(t));
            c += (__popcll(m0) + __popcll(m1)) + (__popcll(m2) + __popcll(m3));
        }
    } else {
#pragma unroll
        for (int q = 0; q < G; ++q) c += __popcll(__builtin_amdgcn_ballot_w64(key[q] > t));
    }
    return c;
}

// Philox4x32-10 (Salmon et al., SC'11): first output word for counter (c0,c1,c2,c3), key (k0,k1).
__device__ __forceinline__ u32 philox4x32_10_word0(u32 c0, u32 c1, u32 c2, u32 c3, u32 k0, u32 k1) {
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const u32 hi0 = __umulhi(0xD2511F53u, c0), lo0 = 0xD2511F53u * c0;
        const u32 hi1 = __umulhi(0xCD9E8D57u, c2), lo1 = 0xCD9E8D57u * c2;
        const u32 n0 = hi1 ^ c1 ^ k0, n2 = hi0 ^ c3 ^ k1;
        c0 = n0; c1 = lo1; c2 = n2; c3 = lo0;
        k0 += 0x9E3779B9u; k1 += 0xBB67AE85u;
    }
    return c0;
}
__device__ __forceinline__ float philox_uniform(u64 seed, u64 step, u32 seq, u32 node) {
    u32 x = philox4x32_10_word0(node, seq, (u32)step, (u32)(step >> 32), (u32)seed, (u32)(seed >> 32));
    return (float)(x >> 8) * (1.0f / 16777216.0f);
}

// ---- rows ---------------------------------------------------------------------------------------
// smallest float whose ordered image has these upper 16 bits (the bin of -inf holds nothing else)
__device__ __forceinline__ float key_edge(u32 k16) { return k16 <= 0x007Fu ? -INFINITY : unord32(k16 << 16); }
// The k-th largest, or a key between it and the next, of the 16-bit keys that a wave holds, G to a lane (k <= 64).
// Bisection between the worst and the best of the lanes' best keys (64 keys reach the worst), about four steps of a
// hundred cycles (the exact k-th between fixed ends, counted pair by pair, was nine steps and 1,600 cycles of the 10,200 that
// a workgroup took; 1,000 now).
template <int G>
__device__ __forceinline__ u32 wave_kth(const u32 (&ky)[G], int k) {
    u32 best = ky[0];
    if constexpr (G == 4) best = max(max(ky[0], ky[1]), max(ky[2], ky[3]));
    static_assert(G == 1 || G == 4, "keys of a lane");
    // Groups without an element (past the row's end, where a wave's last lanes may hold nothing else) do not set the bottom: from -inf
    // on the bisection is sixteen steps (28 rows of 74,365, k = 28, 10.3 us a call, 9.7 so).
    const bool some = best > 0x007Fu;
    u32 hi = best, rest = some ? ~best : 0u;
#define STEP(CTRL, ROWS)                                               \
    hi = max(hi, (u32)dpp_mov<CTRL, ROWS>(0, (int)hi));                \
    rest = max(rest, (u32)dpp_mov<CTRL, ROWS>(0, (int)rest));
    STEP(0x111, 0xf) STEP(0x112, 0xf) STEP(0x114, 0xf) STEP(0x118, 0xf) STEP(0x142, 0xa) STEP(0x143, 0xc)
#undef STEP
    hi = (u32)__builtin_amdgcn_readlane((int)hi, 63);
    // reached by k keys, hi + 1 by none
    u32 lo = __popcll(__ballot(some)) >= k ? ~(u32)__builtin_amdgcn_readlane((int)rest, 63) : 0x007Fu;
    while (hi > lo) {
        const u32 mid = lo + ((hi - lo + 1u) >> 1);
        const int n = count_above<G>(ky, mid - 1u);
        if (n >= k) lo = mid;
        else hi = mid - 1u;
        if (n == k) break;
    }
    return lo;
}
// A row of 8 to ROW_V_MAX entries that one wave holds, groups of eight to a lane, 512 entries apart: asked for, and unpacked, with the groups' maxima and the
// lane's.  A group that reaches past the row's end is its last eight entries, those before the group -inf; of groups behind the end there is only the maximum, -inf.
#define ROW_V_MAX 2048
#define ROW_NG (ROW_V_MAX / 512)
__device__ __forceinline__ int row_group(int V, int n) { return min(512 * n + 8 * lane_id(), V - 8); }
template <bool BF16>
__device__ __forceinline__ void wave_row_request(const void *logits, int64_t at, int V, uint4 (&raw)[ROW_NG][2]) {
#pragma unroll
    for (int n = 0; n < ROW_NG; ++n) {
        if (BF16) raw[n][0] = load16((const uint16_t *)logits + at + row_group(V, n));
        else {
            const float *p = (const float *)logits + at + row_group(V, n);
            raw[n][0] = load16(p);
            raw[n][1] = load16(p + 4);
        }
    }
    __builtin_amdgcn_sched_barrier(0);
}
template <bool BF16>
__device__ __forceinline__ float wave_row_unpack(int V, const uint4 (&raw)[ROW_NG][2], float (&x)[ROW_NG][8], float (&gmx)[ROW_NG]) {
    float mx = -INFINITY;
#pragma unroll
    for (int n = 0; n < ROW_NG; ++n) {
        gmx[n] = -INFINITY;
        if (n && 512 * n >= V) continue;  // uniform
        const u32 lo[4] = {raw[n][0].x, raw[n][0].y, raw[n][0].z, raw[n][0].w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if (BF16) {
                x[n][2 * e] = __uint_as_float(lo[e] << 16);
                x[n][2 * e + 1] = __uint_as_float(lo[e] & 0xFFFF0000u);
            } else {
                const u32 hi[4] = {raw[n][1].x, raw[n][1].y, raw[n][1].z, raw[n][1].w};
                x[n][e] = __uint_as_float(lo[e]);
                x[n][4 + e] = __uint_as_float(hi[e]);
            }
        }
        if (512 * (n + 1) > V) {  // uniform
            const int first = 512 * n + 8 * lane_id() - row_group(V, n);
#pragma unroll
            for (int e = 0; e < 8; ++e) x[n][e] = e >= first ? x[n][e] : -INFINITY;
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) gmx[n] = fmaxf(gmx[n], x[n][e]);
        mx = fmaxf(mx, gmx[n]);
    }
    return mx;
}
// Sum of exp((x - T) inv_t), T the row's maximum.
__device__ __forceinline__ float wave_row_sum(int V, const float (&x)[ROW_NG][8], float T, float inv_t) {
    const float cexp = 1.4426950408889634f * inv_t, nm = T == -INFINITY ? 0.f : -T * cexp;
    float s = 0.f;
#pragma unroll
    for (int n = 0; n < ROW_NG; ++n) {
        if (n && 512 * n >= V) continue;
#pragma unroll
        for (int e = 0; e < 8; ++e) s += __builtin_amdgcn_exp2f(fmaf(x[n][e], cexp, nm));
    }
    return wave_sum(s > 0.f ? s : 0.f);
}

// ---- words between the workgroups of a launch ----------------------------------------------------
// They may sit on different XCDs, whose L2 caches are not coherent: relaxed atomics at agent scope go through to the memory side word by
// word, where a fence would write back and drop the whole L2.  A load at agent scope finds what lies written in its own XCD's L2.
__device__ __forceinline__ void put_agent(u64 *p, u64 v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ u64 get_agent(u64 *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ u64 swap_agent(u64 *p, u64 v) { return __hip_atomic_exchange(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void put_local(u64 *p, u64 v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP); }
__device__ __forceinline__ u64 swap_local(u64 *p, u64 from, u64 to) {
    __hip_atomic_compare_exchange_strong(p, &from, to, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    return from;
}
__device__ __forceinline__ void drain() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
__device__ __forceinline__ u64 ballot(bool b) { return __builtin_amdgcn_ballot_w64(b); }
__device__ __forceinline__ u32 xcc_id() { return __builtin_amdgcn_s_getreg(20 | 3 << 11); }  // HW_REG_XCC_ID, four bits
__device__ __forceinline__ u32 ticks() { return (u32)__builtin_amdgcn_s_memrealtime(); }
typedef u64 u64x2 __attribute__((ext_vector_type(2)));

}  // namespace dt

#include "hands.hpp"
