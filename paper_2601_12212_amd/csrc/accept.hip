// Acceptance kernel: per-node accept decision (greedy arg max match, or stochastic
// min(1, P_T/P_d) against a Philox uniform), then the longest accepted root path via the
// ancestor bitsets, and the bonus token.  One workgroup per sequence.  The vocabulary
// rows themselves were reduced by the row kernels; this kernel merges their per-chunk
// partials (arg max key, and (max, sum) of row/T for the stochastic mode).
#include "common.hpp"
#include "kernels.hpp"

namespace dt {

__device__ __forceinline__ float load_logit(const void *base, int dtype, int64_t idx) {
    return dtype == DT_BF16 ? bf16_bits_to_float(((const uint16_t *)base)[idx]) : ((const float *)base)[idx];
}

// The up to 32 consecutive entries id0 .. id0 + epl - 1 of a row that a thread owns (epl a multiple of 8; entries
// at or past `hi`, and octets past epl, read as -inf), as four octets.  Every load is unconditional, so that all
// of a thread's loads are in flight together (a load inside a branch is waited for inside that branch): an
// bf16 octet that lies wholly inside the range is one 16-byte load (at whatever address), any other octet asks for the
// row's first entries instead and is patched with element loads afterwards (at most one octet of a chunk straddles the
// end of the row).  vec_ok: the row holds at least 8 entries.
__device__ __forceinline__ void load_logits32(const void *row, int dtype, int id0, int epl, int hi, bool vec_ok,
                                              float x[4][8]) {
    if (dtype == DT_BF16 && vec_ok) {  // uniform
        uint4 raw[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int id = id0 + 8 * j;
            const bool full = 8 * j < epl && id + 8 <= hi;
            raw[j] = load16((const uint16_t *)row + (full ? id : 0));
        }
        __builtin_amdgcn_sched_barrier(0);  // every request is out before the first conversion
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const u32 wds[4] = {raw[j].x, raw[j].y, raw[j].z, raw[j].w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                x[j][2 * e] = __uint_as_float(wds[e] << 16);
                x[j][2 * e + 1] = __uint_as_float(wds[e] & 0xFFFF0000u);
            }
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int id = id0 + 8 * j;
            if (!(8 * j < epl && id + 8 <= hi)) {
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    x[j][e] = 8 * j < epl && id + e < hi ? load_logit(row, dtype, id + e) : -INFINITY;
            }
        }
    } else {
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int id = id0 + 8 * j + e;
                x[j][e] = load_logit(row, dtype, 8 * j < epl && id < hi ? id : 0);
            }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int id = id0 + 8 * j + e;
                x[j][e] = 8 * j < epl && id < hi ? x[j][e] : -INFINITY;
            }
    }
}

// Inverse-CDF sample of softmax(row g / T) at the uniform u, by the whole workgroup (256 threads; contains
// barriers; s_wtot and *s_out are not in use).  p: the (max, sum exp((x - max)/T)) that the row kernel left for chunk
// `lane` of the row (lane < S <= 64), the same in every wave.  The chunks' masses
// relative to the row maximum Mrow, accumulated in double, locate the chunk that holds the crossing; only
// that chunk is read again (thread t owns `epl` <= 32 consecutive ids), element masses in fp32, running sums in
// double.  The comparison is "cumulative mass > u * total", the un-normalised form of the cdf > u test;
// it differs from an all-double evaluation by ~1e-6 in probability.  The token is returned to thread 0.
__device__ __forceinline__ int sample_row_block(const AcceptArgs &a, int64_t g, float2 p, float Mrow, float u, float inv_t,
                                                double *s_wtot, int *s_out) {
    const int tid = threadIdx.x, lane = lane_id(), w = __builtin_amdgcn_readfirstlane(tid >> 6), S = a.S;
    const void *row = (const char *)a.target + g * a.row_stride * (a.dtype == DT_BF16 ? 2 : 4);
    const float cexp = 1.4426950408889634f * inv_t;
    double mass = 0.0;
    if (lane < S && p.y > 0.f) mass = (double)p.y * (double)__builtin_amdgcn_exp2f((p.x - Mrow) * cexp);
    const double cum = wave_scan_incl_f64(mass);  // over the chunks
    const double Z = readlane_f64(cum, 63);
    const double target_mass = (double)u * Z;
    // first chunk whose cumulative mass passes the target; if rounding leaves none, the last with mass
    const u64 passed = __ballot(cum > target_mass), massy = __ballot(mass > 0.0);
    const int cstar = passed ? (int)__builtin_ctzll(passed) : massy ? 63 - (int)__builtin_clzll(massy) : 0;
    const double before = readlane_f64(cum - mass, cstar);
    const int epl = a.chunk_elems / 256;
    const int begin = cstar * a.chunk_elems - row_shift(a.target, a.dtype == DT_BF16, a.V, a.row_stride, g);  // as the row kernel counts
    const int lo = max(begin, 0), hi = min(a.V, begin + a.chunk_elems);
    const int id0 = begin + tid * epl;
    const bool vec_ok = a.V >= 8;
    // a thread owns at most 32 entries (four octets): all asked for at once, their masses kept, so that the thread that
    // holds the crossing finds it in its registers
    float x[4][8];
    load_logits32(row, a.dtype, id0, epl, hi, vec_ok, x);
    if (id0 < 0) x[0][0] = -INFINITY;
    double oct[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        oct[j] = 0.0;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            x[j][e] = __builtin_amdgcn_exp2f((x[j][e] - Mrow) * cexp);  // past epl: 0
            oct[j] += (double)x[j][e];
        }
    }
    const double mine = (oct[0] + oct[1]) + (oct[2] + oct[3]);
    const double incl = wave_scan_incl_f64(mine);
    if (lane == 63) s_wtot[w] = incl;
    if (tid == 0) *s_out = -1;
    __syncthreads();
    // the first crossing thread of the first crossing wave
    double run = before;
    bool earlier = false;
    for (int q = 0; q < w; ++q) {
        run += s_wtot[q];
        earlier = earlier || run > target_mass;
    }
    const u64 m = __ballot(run + incl > target_mass);
    if (!earlier && m && lane == (int)__builtin_ctzll(m)) {
        // the octet that crosses (the last one if rounding leaves none), then the entry
        double cm = run + incl - mine;
        int jc = 3;
        double c0 = cm;
        bool found = false;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (!found) { jc = j; c0 = cm; }
            cm += oct[j];
            found = found || cm > target_mass;
        }
        int id = min(id0 + epl, hi) - 1;
        bool done = false;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float v = jc < 2 ? (jc == 0 ? x[0][e] : x[1][e]) : (jc == 2 ? x[2][e] : x[3][e]);
            c0 += (double)v;
            if (!done && c0 > target_mass) { id = id0 + 8 * jc + e; done = true; }
        }
        *s_out = id;
    }
    __syncthreads();
    int out = *s_out;
    if (tid == 0 && out < 0) {
        // the chunk's re-computed mass falls just short of the crossing (rounding), or the row
        // carries no mass at all: last token of the chunk that carries mass, else token 0
        int id = hi - 1;
        while (id > lo && !(__builtin_amdgcn_exp2f((load_logit(row, a.dtype, id) - Mrow) * cexp) > 0.f)) --id;
        out = Z > 0.0 ? id : 0;
    }
    return out;
}

// Target-sampled verification: node i of sequence b draws the target's own next token from
// softmax(row i / T) at the uniform of its depth.  One workgroup per (sequence, node): two trips to memory, one for
// everything that leads to the chunk (the uniforms of all depths are made meanwhile, one to a lane) and the chunk itself.
// With four trips, scans through LDS and every exponential taken twice by the lane that holds the crossing: 6.9 us for 3 x 64
// nodes of a 50,001-entry vocabulary, 5.0 now.
__global__ __launch_bounds__(256) void node_sample_kernel(AcceptArgs a) {
    const int b = (int)((u32)blockIdx.x / (u32)a.TT_cap), i = (int)((u32)blockIdx.x % (u32)a.TT_cap), lane = lane_id();
    const int64_t g = blockIdx.x;
    __shared__ double s_wtot[4];
    __shared__ int s_out;
    const int n_raw = a.n_nodes[b];
    const int c = min(lane, a.S - 1);
    u64 key = a.part_keys[g * a.S + c];  // dead nodes have their slots in the workspace all the same
    const float2 p = a.part_ms[g * a.S + c];
    const int dep_raw = a.depth[g];
    const float u_lane = philox_uniform(a.seed, a.step, (u32)b, 0x80000000u + (u32)lane);
    __builtin_amdgcn_sched_barrier(0);
    if (i >= min(max(n_raw, 1), a.TT_cap)) return;
    // the row maximum: the largest of the chunks' best keys
    key = wave_max_u64(key);
    const int dep = __builtin_amdgcn_readfirstlane(min(max(dep_raw, 0), DT_D_MAX));
    const float u = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(u_lane), dep));
    const int tok = sample_row_block(a, g, p, key_val(key), u, 1.0f / a.temperature, s_wtot, &s_out);
    if (threadIdx.x == 0) a.samples[g] = tok;
}

// The best (value, id) key of row g and, with SUM, its (max, sum exp((x - max) inv_t)), by one wave that holds the row, 8 to ROW_V_MAX
// entries.  What row_argmax_kernel leaves for a row of one chunk, and as there.
#define ACCEPT_WAVES 16
template <bool BF16, bool SUM>
__device__ __forceinline__ u64 wave_row(const AcceptArgs &a, int64_t g, float inv_t, float2 &ms) {
    constexpr int NG = ROW_NG;
    const int V = a.V;
    uint4 raw[NG][2];
    wave_row_request<BF16>(a.target, g * a.row_stride, V, raw);
    float x[NG][8], gmx[NG];
    const float T = wave_max(wave_row_unpack<BF16>(V, raw, x, gmx));
    if constexpr (SUM) ms = make_float2(T, wave_row_sum(V, x, T, inv_t));
    // the first group that holds the maximum, the first lane of that, the first such element
    u64 key = 0ull;
#pragma unroll
    for (int n = 0; n < NG; ++n) {
        if (n && 512 * n >= V) continue;
        const u64 m = __builtin_amdgcn_ballot_w64(gmx[n] == T);
        if (m && key == 0ull) {  // uniform
            const int first = (int)__builtin_ctzll(m);
            int at = 0;
#pragma unroll
            for (int e = 7; e >= 0; --e) at = x[n][e] == T ? e : at;
            key = make_key(T, (u32)(min(512 * n + 8 * first, V - 8) + __builtin_amdgcn_readlane(at, first)));
        }
    }
    return key;
}

// ROWS: the rows are reduced here as well, a wave to a row, in the place of a launch in front of this one.
//
// The stochastic mode asks for a node's own logit and makes its uniforms while the row partials are on their way or being
// merged, and keeps the partials for the bonus token: 10.2 -> 8.5 us for four sequences of 96 nodes.
template <bool ROWS>
__global__ __launch_bounds__(ROWS ? 64 * ACCEPT_WAVES : 256) void accept_kernel(AcceptArgs a) {
    const int b = blockIdx.x, tid = threadIdx.x, lane = lane_id(), w = tid >> 6;
    const int n_raw = a.n_nodes[b];
    const int64_t o = (int64_t)b * a.TT_cap;
    const bool stochastic = a.mode == DT_ACCEPT_STOCHASTIC;
    const bool sampled = a.mode == DT_ACCEPT_SAMPLED;  // node_sample_kernel has drawn every node's token
    const float inv_t = stochastic ? 1.0f / a.temperature : 1.0f;
    const int S = a.S;

    __shared__ int s_amax[DT_TT_MAX];
    __shared__ float s_rowmax[DT_TT_MAX];
    __shared__ float s_lse[DT_TT_MAX];
    __shared__ u64 s_acc[2];
    __shared__ int s_best[4];
    __shared__ double s_wtot[4];
    __shared__ int s_bonus;
    __shared__ float2 s_ms[DT_TT_MAX][16];  // a row's chunk partials, for the bonus token

    // ---- everything a node needs later, and the row partials, are requested before the node count is back: one trip to
    //      memory instead of two (padded entries and rows belong to the buffers; what they hold is not used) --------------
    const int me = min(tid, a.TT_cap - 1);
    const int my_tok = a.tokens[o + me], my_par = a.parents[o + me], my_dep = a.depth[o + me];
    const u64 my_m0 = a.anc_mask[(o + me) * DT_MASK_WORDS], my_m1 = a.anc_mask[(o + me) * DT_MASK_WORDS + 1];
    const float my_logp = stochastic ? a.logp[o + me] : 0.f;
    // four adjacent lanes share a row, each takes every fourth chunk; rows tid / 4 and 64 + tid / 4
    const int part = tid & 3;
    u64 key0[2][4];
    float2 p0[2][4];
    __shared__ u64 s_key[ROWS ? ACCEPT_WAVES : 1];
    __shared__ float2 s_sum[ROWS ? ACCEPT_WAVES : 1];
    if constexpr (ROWS) {
        auto row = [&](int i) {
            float2 ms = make_float2(0.f, 0.f);
            const u64 key = a.dtype == DT_BF16 ? stochastic ? wave_row<true, true>(a, o + i, inv_t, ms) : wave_row<true, false>(a, o + i, inv_t, ms)
                                               : stochastic ? wave_row<false, true>(a, o + i, inv_t, ms) : wave_row<false, false>(a, o + i, inv_t, ms);
            if (lane == 0) {
                s_key[i] = key;
                s_sum[i] = ms;
            }
        };
        const int wave = __builtin_amdgcn_readfirstlane(w);
        if (wave < a.TT_cap) row(wave);  // a wave to a row, without waiting for the node count: the row is inside the buffer either way
        __syncthreads();
        if (wave >= 4) return;  // (a barrier waits for the waves that are left)
    }
#pragma unroll
    for (int h = 0; h < 2; ++h)
        if (!ROWS && 64 * h < a.TT_cap) {  // uniform
            const int64_t g = o + min(64 * h + (tid >> 2), a.TT_cap - 1);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int c = min(part + 4 * u, S - 1);  // past the end: the last chunk again, ignored below
                key0[h][u] = a.part_keys[g * S + c];
                if (stochastic) p0[h][u] = a.part_ms[g * S + c];
            }
        }
    // the uniforms, meanwhile
    const float my_u = stochastic ? philox_uniform(a.seed, a.step, (u32)b, (u32)tid) : 0.f;
    const float bonus_u = stochastic ? philox_uniform(a.seed, a.step, (u32)b, 0xFFFFFFFFu) : 0.f;
    __builtin_amdgcn_sched_barrier(0);
    const int N = min(max(n_raw, 1), a.TT_cap);
    // the logit of a node's own token in its parent's row, on its way while the partials are merged
    const int par = min(max(my_par, 0), N - 1);
    const float my_x = stochastic ? load_logit(a.target, a.dtype, (o + par) * a.row_stride + min(max(my_tok, 0), a.V - 1)) : 0.f;
    __builtin_amdgcn_sched_barrier(0);

    // ---- merge the row partials --------------------------------------------------------------------
    {
        const float cexp = 1.4426950408889634f * inv_t;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int i0 = 64 * h;
            if (i0 >= N) break;  // uniform
            const int i = i0 + (tid >> 2);
            const int64_t g = o + min(i, N - 1);
            u64 best = 0ull;
            float M = -INFINITY, Ssum = 0.f;
            auto take = [&](int c0, const u64 (&key)[4], const float2 (&p)[4]) {
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    if (c0 + 4 * u >= S) continue;
                    best = key[u] > best ? key[u] : best;
                    if (stochastic) {
                        const float M2 = fmaxf(M, p[u].x);
                        if (M2 != -INFINITY)
                            Ssum = Ssum * __builtin_amdgcn_exp2f((M - M2) * cexp) +
                                   p[u].y * __builtin_amdgcn_exp2f((p[u].x - M2) * cexp);
                        M = M2;
                    }
                }
            };
            if constexpr (ROWS) {
                best = s_key[min(i, N - 1)];
                if (stochastic) {
                    const float2 p = s_sum[min(i, N - 1)];
                    M = p.x;
                    Ssum = part == 0 ? p.y : 0.f;
                    if (part == 0) s_ms[i][0] = p;
                }
            } else take(part, key0[h], p0[h]);
            if (!ROWS && stochastic && S <= 16)
#pragma unroll
                for (int u = 0; u < 4; ++u) s_ms[i][part + 4 * u] = p0[h][u];
            for (int c0 = part + 16; !ROWS && c0 < S; c0 += 16) {  // four chunks per trip to memory
                u64 key[4];
                float2 p[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int c = min(c0 + 4 * u, S - 1);
                    key[u] = a.part_keys[g * S + c];
                    if (stochastic) p[u] = a.part_ms[g * S + c];
                }
                take(c0, key, p);
            }
#pragma unroll
            for (int off = 1; off <= 2; off <<= 1) {  // the four lanes of the row
                const u64 ob = shfl_xor_u64(best, off);
                best = ob > best ? ob : best;
                if (stochastic) {
                    const float M2 = __shfl_xor(M, off, 64), S2 = __shfl_xor(Ssum, off, 64);
                    const float Mn = fmaxf(M, M2);
                    if (Mn != -INFINITY)
                        Ssum = Ssum * __builtin_amdgcn_exp2f((M - Mn) * cexp) + S2 * __builtin_amdgcn_exp2f((M2 - Mn) * cexp);
                    M = Mn;
                }
            }
            if (part == 0 && i < N) {
                const int choice = sampled ? a.samples[o + i] : (int)key_idx(best);
                s_amax[i] = choice;
                s_rowmax[i] = key_val(best);
                s_lse[i] = stochastic ? M * inv_t + __logf(Ssum) : 0.f;
                if (a.node_argmax) a.node_argmax[o + i] = choice;
            }
        }
    }
    __syncthreads();

    // ---- per-node accept bit ----------------------------------------------------------------
    if (tid < DT_TT_MAX) {  // waves 0 and 1: wave w owns bits [64w, 64w+64)
        bool acc = false;
        if (tid < N) {
            if (tid == 0) {
                acc = true;
            } else {
                if (!stochastic) {
                    acc = my_tok == s_amax[par];
                } else if (my_tok >= 0 && my_tok < a.V) {
                    const float lpT = my_x * inv_t - s_lse[par];
                    const float alpha = fminf(1.0f, __expf(lpT - my_logp));
                    acc = my_u < alpha;
                }
            }
        }
        const u64 m = __ballot(acc);
        if (lane == 0) s_acc[w] = m;
    }
    __syncthreads();

    // ---- deepest node whose ancestors are all accepted; ties -> lowest index -------------
    if (tid < DT_TT_MAX) {
        int key = -1;
        if (tid < N) {
            const bool ok = ((my_m0 & ~s_acc[0]) | (my_m1 & ~s_acc[1])) == 0ull;
            if (ok) key = (my_dep << 8) | (255 - tid);
        }
        key = wave_max_i32(key);
        if (lane == 0) s_best[w] = key;
    }
    __syncthreads();
    const int bkey = max(s_best[0], s_best[1]);
    const int best = 255 - (bkey & 255);
    const int len = bkey >> 8;

    // ---- the accepted path: exactly the nodes in the ancestor set of `best`, which its owner
    //      thread publishes (the accept bits in s_acc are no longer needed) -----------------------
    if (tid == best) { s_acc[0] = my_m0; s_acc[1] = my_m1; }
    if (tid <= DT_D_MAX && tid > len) {  // unused slots; slot len of out_tokens is the bonus token
        a.path_nodes[(int64_t)b * (DT_D_MAX + 1) + tid] = -1;
        a.out_tokens[(int64_t)b * (DT_D_MAX + 1) + tid] = -1;
    }
    __syncthreads();
    if (tid < N) {
        const bool on_path = ((tid < 64 ? s_acc[0] : s_acc[1]) >> (tid & 63)) & 1ull;
        if (on_path && my_dep <= DT_D_MAX) {
            a.path_nodes[(int64_t)b * (DT_D_MAX + 1) + my_dep] = tid;
            if (tid > 0) a.out_tokens[(int64_t)b * (DT_D_MAX + 1) + my_dep - 1] = my_tok;
        }
    }
    if (tid == 0) { a.accept_len[b] = len; a.best_node[b] = best; }

    // ---- bonus token --------------------------------------------------------------------------
    int bonus;
    if (!stochastic) {
        bonus = s_amax[best];
    } else {
        // inverse CDF of softmax(row best / T) at the bonus uniform
        const int c = min(lane, S - 1);
        const float2 p = S <= 16 ? s_ms[best][c] : a.part_ms[(o + best) * S + c];
        bonus = sample_row_block(a, o + best, p, s_rowmax[best], bonus_u, inv_t, s_wtot, &s_bonus);
    }
    if (tid == 0 && len <= DT_D_MAX) a.out_tokens[(int64_t)b * (DT_D_MAX + 1) + len] = bonus;
}

// Rows that a wave holds, a wave of the workgroup to each: one launch in place of two.  us a step, graph | eager, two launches -> one: 8 rows of 1,024 fp32
// entries 22.5 -> 21.9 | 19.0 -> 16.9; graphs, greedy and stochastic, 16 rows of 1,000 bf16 entries 23.7 -> 22.5, 26.8 -> 26.4, of 2,000 fp32 22.3 -> 21.5,
// 26.3 -> 25.4; but two rows to a wave, 32 of 1,001 24.4 -> 25.1, 27.5 -> 29.1.  (Longer rows, 2,048 entries at a time, and four waves: 16 rows of 2,000 23.5 -> 25.2.)
// Beyond a compute unit to a sequence they come in turns of a whole acceptance, and rows past a sequence's nodes are read for nothing: greedy | stochastic, three nodes of 16,
// two launches -> one, 256 sequences of 1,000 bf16 entries 7.5 -> 4.5 | 11.3 -> 8.3, 264 7.6 -> 7.1 | 12.0 -> 14.6, 1,024 13.4 -> 14.3 | 20.1 -> 29.9; of 2,048 fp32 320 7.8 -> 12.3 | 12.4 -> 19.3.
// And from 32 sequences on more than 120 KB of rows to a workgroup take longer than a launch that passes over the dead ones: fp32 of 1,920 entries, 64 sequences 6.3 -> 5.0 | 9.6 -> 8.5, of 2,000
// 6.1 -> 6.8 | 9.5 -> 10.3 (32 5.9 -> 6.4), of 2,048 192 sequences 6.8 -> 7.9 | 10.4 -> 11.4, with room for 10 nodes 6.7 -> 5.0 | 10.2 -> 8.6.
#define ACCEPT_BATCH 256
#define ACCEPT_BATCH_LONG 16
#define ACCEPT_LONG (120 << 10)
bool accept_takes_rows(const AcceptArgs &a) {
    const int bytes = a.TT_cap * a.V * (a.dtype == DT_BF16 ? 2 : 4);
    return a.mode != DT_ACCEPT_SAMPLED && a.V >= 8 && a.V <= ROW_V_MAX && a.TT_cap <= ACCEPT_WAVES && a.batch <= (bytes > ACCEPT_LONG ? ACCEPT_BATCH_LONG : ACCEPT_BATCH);
}

hipError_t accept_launch(const AcceptArgs &a, hipStream_t st) {
    if (a.batch <= 0) return hipSuccess;
    if (a.mode == DT_ACCEPT_SAMPLED) {
        launch_kernel(KID_NODE_SAMPLE, st, node_sample_kernel, dim3(a.batch * a.TT_cap), dim3(256), 0, a);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    launch_kernel(KID_ACCEPT, st, a.rows_here ? accept_kernel<true> : accept_kernel<false>, dim3(a.batch), dim3(a.rows_here ? 64 * ACCEPT_WAVES : 256), 0, a);
    return hipGetLastError();
}

}  // namespace dt
