// Routing, part 3: block importance and top-n selection per (sequence, verifier query, KV group)
// (the top-n reduction of the routing launch, Section 5.1; mandatory initial and local blocks that count toward n, Section 7.3).
//
//   imp[j] = sum_{m < l'/d} sum_{n' < l/d} colsum[(l'/d) j + m - n']      (terms outside [0, visible) are 0)
//   candidates j = 0..J, J = block of the query's own slot; forced blocks are ranked first;
//   the n_eff = min(n, J+1) best by (importance descending, index ascending) are written ascending.
//
// One workgroup per (b, i, g); in the approximate shared-index variant (Section 4.3) one per (b, group, g):
// it selects for the group's representative and writes the set to the row of every member.  Keys are packed as (float bits << 32) | ~index so that a plain
// unsigned 64-bit comparison implements "larger importance, then smaller index"; importances are
// sums of probabilities, hence non-negative, and their IEEE bit patterns order like the values.
//
// Selection without a serial argmax loop: every thread owns the blocks j = tid (mod 256) and keeps
// its best key.  The n_eff-th largest of the 64 per-thread bests of one wavefront is a lower bound of
// the n_eff-th largest key overall (they are n_eff distinct keys), so every winner is >= the largest of
// the four wavefronts' bounds; the (few) keys at or above it are compacted into a candidate list and
// ranked by counting.  If the list overflows (massive ties), a
// plain serial argmax over LDS takes over.  LDS keeps the importances as their 32-bit patterns (the index is the position;
// keys are composed on the fly): 18 KB at 2048 blocks, eight workgroups per CU.
#pragma once
#include <type_traits>

#include "device_common.hpp"
#include "topn_fold.hpp"

namespace ssv {

struct TopnArgs {
    const float* colsum;     // [B, T, H_kv, nc_pitch]
    const int32_t *seq_lens, *n_cmp, *n_query, *parents;
    int32_t* sel_idx;        // [B, T, H_kv, n_sel]
    int B, T, H_kv;
    int l, d, l_sel, n_sel, n_init, n_local;
    int max_seq_len, max_n_cmp;   // host-side bounds the lengths read from device memory are clamped to
    int nc_pitch;
    int max_blocks;          // capacity of the key array in LDS
    int share;               // 0: every query selects for itself; > 0: groups of `share` queries share a set
};

constexpr int kMaxNSel = 32;
constexpr int kMaxImpTerms = 8;     // (l'/d) + (l/d) - 1 compressed columns feed one selection block
constexpr int kBlocksPerBatch = 4;  // blocks whose column loads are issued together
constexpr int kMaxCand = 512;

__device__ __forceinline__ uint64_t wave_max_u64(uint64_t v) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        const uint32_t lo = __shfl_xor((uint32_t)v, off), hi = __shfl_xor((uint32_t)(v >> 32), off);
        const uint64_t o = ((uint64_t)hi << 32) | lo;
        v = o > v ? o : v;
    }
    return v;
}

__host__ __device__ inline size_t topn_lds_bytes(int max_blocks) {
    return (((size_t)max_blocks * 4 + 15) & ~(size_t)15) + kThreads * 8 + kMaxCand * 8 + 16 * 8 + kMaxNSel * 4 + kMaxT * 28 + 64;
}

// ---- The same selection by ONE wavefront, for callers that have several queries to select for at once (the
// selected-branch launch selects for the queries of its own group, each wavefront taking a query, instead of
// waiting for a separate launch).  Importances are kept in LDS as their 32-bit patterns (the index is the
// position), keys are composed on the fly, and the result is the one k_topn writes: the same importances, summed
// in the same order, the same (importance, index) order.

struct WaveTopnScratch {             // one per wavefront, in LDS
    uint32_t* bits;                  // [J + 1] importance bit patterns (forced blocks: +inf)
    uint64_t* cand;                  // [kWaveMaxCand + 8]
    int* pick;                       // [kMaxNSel]
};
constexpr int kWaveMaxCand = 256;
__host__ __device__ inline size_t wave_topn_lds_bytes(int max_blocks) {   // per wavefront, 16-byte multiple
    return (((size_t)max_blocks * 4 + 15) & ~(size_t)15) + (kWaveMaxCand + 8) * 8 + kMaxNSel * 4;
}
__device__ __forceinline__ WaveTopnScratch wave_topn_scratch(char* base, int max_blocks) {
    WaveTopnScratch w;
    w.bits = reinterpret_cast<uint32_t*>(base);
    w.cand = reinterpret_cast<uint64_t*>(base + (((size_t)max_blocks * 4 + 15) & ~(size_t)15));
    w.pick = reinterpret_cast<int*>(w.cand + kWaveMaxCand + 8);
    return w;
}
// LDS written by some lanes of a wavefront is read by others: the LDS unit takes a wavefront's operations in order,
// so only the compiler has to be kept from reordering them.
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
__device__ __forceinline__ uint64_t topn_key(uint32_t bits, int j) {
    return ((uint64_t)bits << 32) | (uint32_t)(0xFFFFFFFFu - (uint32_t)j);
}

// cs: colsum row of the (representative) query; ncv: its visible compressed rows; J: block of its own slot.
// Writes the n_sel entries (ascending, -1 padding) to out[] (LDS or global).  WIDE: 1024 blocks in flight instead of 512 (80
// registers; not where they would cost the caller's third workgroup per CU, at d = 64).
template <bool WIDE>
__device__ __forceinline__ void wave_topn(const float* cs, int ncv, int J, int l, int d, int l_sel, int n_sel, int n_init,
                                          int n_local, const WaveTopnScratch& w, int lane, int32_t* out) {
    const int a_ratio = l_sel / d, b_ratio = l / d;
    const int n_eff = min(n_sel, J + 1);
    const int n_terms = a_ratio + b_ratio - 1;
    const int j_last_scored = fold_last_scored(J, n_local);
    uint32_t best = 0;         // largest importance among the blocks of this lane (index mod 64), as its bit pattern
    for (int j = max(j_last_scored + 1, 0); j <= J; ++j) {     // forced trailing local blocks, each with its owner lane
        if ((j & 63) != lane) continue;
        w.bits[j] = 0x7F800000u;
        best = max(best, 0x7F800000u);
    }
    constexpr int NB = 4;     // blocks per lane whose column loads are issued together
    if (a_ratio == 4 && b_ratio == 2) {
        // The standard geometry: block j takes columns 4j-1 .. 4j+3 with weights 1 2 2 2 1; one 16-byte and one 4-byte load
        // per block (same terms in the same order as the general form).  This is one wavefront on its SIMD, a vector
        // instruction every five clocks: groups of 64 blocks whose columns are all visible take none for conditions, and up to
        // 1024 blocks are in flight together.  (2048 blocks: 13 us of the selected launch of 40-node trees at 128K with the
        // conditions at every block and 512 in flight.)
        auto block_loads = [&](int j, f32x4& x, float& xm) {
            x = *reinterpret_cast<const f32x4*>(cs + fold_column(j, j_last_scored, ncv));
            xm = cs[fold_left_column(j, j_last_scored, ncv)];
        };
        auto put = [&](int j, float imp) {
            const uint32_t bits = j < n_init ? 0x7F800000u : __float_as_uint(imp);
            w.bits[j] = bits;
            best = max(best, bits);
        };
        auto block_any = [&](int j, const f32x4& x, float xm) {
            if (j > j_last_scored) return;
            const int c0 = 4 * j;
            float imp = 0.f;
            if (c0 >= 1 && c0 - 1 < ncv) imp += 1.f * xm;
            if (c0 < ncv) imp += 2.f * x[0];
            if (c0 + 1 < ncv) imp += 2.f * x[1];
            if (c0 + 2 < ncv) imp += 2.f * x[2];
            if (c0 + 3 < ncv) imp += 1.f * x[3];
            put(j, imp);
        };
        const int groups = fold_full_groups(j_last_scored, ncv);
        constexpr int NR = 2;      // the remainder's loads go first (it rarely has more groups)
        f32x4 rx[NR];
        float rm[NR];
#pragma unroll
        for (int v = 0; v < NR; ++v) block_loads((groups + v) * 64 + lane, rx[v], rm[v]);
        int last63 = 0;        // (uniform) column before the group's first one: the last column of lane 63 of the group before
        auto full_groups = [&](auto nf, int g0) {
            constexpr int NF = decltype(nf)::value;
            f32x4 x[NF];
#pragma unroll
            for (int v = 0; v < NF; ++v) x[v] = *reinterpret_cast<const f32x4*>(cs + 4 * (min(g0 + v, groups - 1) * 64 + lane));
            // Past the last group: that group again (no branches: the loads would sink into them, behind each other).  The
            // column before a block's own comes from the lane below, not from memory: its load would be as expensive as theirs.
#pragma unroll
            for (int v = 0; v < NF; ++v) {
                const int j = min(g0 + v, groups - 1) * 64 + lane;
                const float xm = __int_as_float(__builtin_amdgcn_update_dpp(last63, __float_as_int(x[v][3]), 0x138, 0xf, 0xf, false));   // lane l: x[3] of l - 1
                const float imp = (((xm + 2.f * x[v][0]) + 2.f * x[v][1]) + 2.f * x[v][2]) + x[v][3];
                w.bits[j] = __float_as_uint(imp);
                best = max(best, __float_as_uint(imp));
                last63 = g0 + v + 1 < groups ? __builtin_amdgcn_readlane(__float_as_int(x[v][3]), 63) : last63;
            }
        };
        int g0 = 0;
        if constexpr (WIDE) {
            for (; groups - g0 > 8; g0 += 16) full_groups(std::integral_constant<int, 16>{}, g0);
        }
        for (; g0 < groups; g0 += 8) full_groups(std::integral_constant<int, 8>{}, g0);
        if (groups > 0 && lane < n_init) {         // (n_init <= n_sel <= 32: forced blocks are in the first group)
            w.bits[lane] = 0x7F800000u;
            best = 0x7F800000u;
        }
#pragma unroll
        for (int v = 0; v < NR; ++v) block_any((groups + v) * 64 + lane, rx[v], rm[v]);
        for (int j = (groups + NR) * 64 + lane; j <= j_last_scored; j += 64) {
            f32x4 x;
            float xm;
            block_loads(j, x, xm);
            block_any(j, x, xm);
        }
    } else
    for (int j0 = lane; j0 <= j_last_scored; j0 += 64 * NB) {
        float imp[NB];
        if (n_terms <= kMaxImpTerms) {
            float x[NB][kMaxImpTerms];
#pragma unroll
            for (int v = 0; v < NB; ++v)
#pragma unroll
                for (int u = 0; u < kMaxImpTerms; ++u) {
                    const int c = a_ratio * (j0 + v * 64) + u - (b_ratio - 1);
                    x[v][u] = cs[(u < n_terms && c >= 0 && c < ncv) ? c : 0];
                }
#pragma unroll
            for (int v = 0; v < NB; ++v) {
                imp[v] = 0.f;
#pragma unroll
                for (int u = 0; u < kMaxImpTerms; ++u) {
                    const int delta = u - (b_ratio - 1);
                    const int c = a_ratio * (j0 + v * 64) + delta;
                    const int pairs = min(min(a_ratio, b_ratio), min(delta + b_ratio, a_ratio - delta));
                    if (u < n_terms && c >= 0 && c < ncv) imp[v] += (float)pairs * x[v][u];
                }
            }
        } else {
            for (int v = 0; v < NB; ++v) {
                imp[v] = 0.f;
                const int j = j0 + v * 64;
                for (int m = 0; m < a_ratio && j <= J; ++m)
                    for (int n2 = 0; n2 < b_ratio; ++n2) {
                        const int c = a_ratio * j + m - n2;
                        if (c >= 0 && c < ncv) imp[v] += cs[c];
                    }
            }
        }
#pragma unroll
        for (int v = 0; v < NB; ++v) {
            const int j = j0 + v * 64;
            if (j <= j_last_scored) {
                const uint32_t bits = j < n_init ? 0x7F800000u : __float_as_uint(imp[v]);
                w.bits[j] = bits;
                best = max(best, bits);
            }
        }
    }
    // Threshold on the importance bits alone: the largest value (to 23 bits) that at least n_eff of the 64 per-lane
    // bests reach, found by bisection with wave-wide votes.  The lanes' bests are distinct blocks, so at least n_eff
    // blocks reach it and every winner does; blocks that reach it are the candidates (lanes without blocks hold 0,
    // and with fewer than n_eff bests the threshold stays 0: every block is a candidate).
    uint32_t thr_bits = 0;
    {
        for (int bit = 30; bit >= 8; --bit) {
            const uint32_t trial = thr_bits | (1u << bit);
            if (__popcll(__builtin_amdgcn_ballot_w64(best >= trial)) >= n_eff) thr_bits = trial;
        }
    }
    wave_lds_sync();      // the importance bits written above are read by other lanes below
    int n_cand = 0;
    constexpr int NC = 8;     // blocks per lane whose LDS reads are in flight together
    for (int jb = 0; jb <= J; jb += 64 * NC) {
        uint32_t bits[NC];
#pragma unroll
        for (int u = 0; u < NC; ++u) bits[u] = w.bits[min(jb + 64 * u + lane, J)];
#pragma unroll
        for (int u = 0; u < NC; ++u) {
            const int j = jb + 64 * u + lane;
            if (jb + 64 * u > J) break;               // uniform
            const bool is = j <= J && bits[u] >= thr_bits;
            const uint64_t m = __builtin_amdgcn_ballot_w64(is);
            if (m == 0) continue;                     // uniform
            const int pos = n_cand + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
            if (is && pos < kWaveMaxCand) w.cand[pos] = topn_key(bits[u], j);
            n_cand += __popcll(m);
        }
    }
    if (n_cand <= 64) {
        // One candidate per lane, in index order: the value of the n_eff-th largest, exactly, by bisection; the winners are
        // the larger ones and the first of the equal ones, and their order is the output's: no ranking, no sorting.
        wave_lds_sync();
        const uint64_t key = lane < n_cand ? w.cand[lane] : 0ull;
        const uint32_t bits = (uint32_t)(key >> 32);
        uint32_t t = 0;
        for (int bit = 31; bit >= 0; --bit) {
            const uint32_t trial = t | (1u << bit);
            if (__popcll(__builtin_amdgcn_ballot_w64(bits >= trial)) >= n_eff) t = trial;      // (trial > 0: no lane without a candidate)
        }
        auto before = [&](uint64_t m) { return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u)); };
        const bool gt = lane < n_cand && bits > t, eq = lane < n_cand && bits == t;
        const int need = n_eff - __popcll(__builtin_amdgcn_ballot_w64(gt));
        const bool win = gt || (eq && before(__builtin_amdgcn_ballot_w64(eq)) < need);
        const uint64_t m = __builtin_amdgcn_ballot_w64(win);
        if (win) out[before(m)] = (int)(0xFFFFFFFFu - (uint32_t)key);
        if (lane >= n_eff && lane < n_sel) out[lane] = -1;
        return;
    }
    // pad the list to a multiple of 8 with keys that are larger than none (the counting loop below reads in eights)
    if (lane < 8 && n_cand + lane < kWaveMaxCand + 8) w.cand[min(n_cand, kWaveMaxCand) + lane] = 0ull;
    wave_lds_sync();
    if (n_cand <= kWaveMaxCand) {
        for (int e = lane; e < n_cand; e += 64) {      // rank candidates by counting; ranks below n_eff are the selection
            const uint64_t key = w.cand[e];
            int rank = 0;
            for (int f = 0; f < n_cand; f += 8) {
                uint64_t c[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) c[u] = w.cand[f + u];
#pragma unroll
                for (int u = 0; u < 8; ++u) rank += c[u] > key;
            }
            if (rank < n_eff) w.pick[rank] = (int)(0xFFFFFFFFu - (uint32_t)key);
        }
    } else {
        // massive ties: serial argmax, one winner per round; the owner (index mod 64) retires it and rescans
        uint64_t best_key = 0;
        for (int j = lane; j <= J; j += 64) {
            const uint64_t key = topn_key(w.bits[j], j);
            best_key = key > best_key ? key : best_key;
        }
        for (int round = 0; round < n_eff; ++round) {
            const uint64_t top = wave_max_u64(best_key);
            const int j_top = (int)(0xFFFFFFFFu - (uint32_t)top);
            if (lane == 0) w.pick[round] = top ? j_top : 0;
            if (!top) continue;       // (cannot happen: there are at least n_eff blocks)
            if ((j_top & 63) == lane) {
                w.bits[j_top] = 0xFFFFFFFFu;      // retired (no importance has this pattern)
                best_key = 0;
                for (int j = lane; j <= J; j += 64) {
                    const uint32_t bits = w.bits[j];
                    const uint64_t key = topn_key(bits, j);
                    if (bits != 0xFFFFFFFFu && key > best_key) best_key = key;
                }
            }
        }
    }
    wave_lds_sync();
    // ascending order: pick e goes to position (number of smaller picks); picks are distinct
    if (lane < n_sel) {
        int pick = -1, rank = lane;       // lanes beyond n_eff write the -1 padding at their own position
        if (lane < n_eff) {
            pick = w.pick[lane];
            rank = 0;
            int p[kMaxNSel];
#pragma unroll
            for (int f = 0; f < kMaxNSel; ++f) p[f] = w.pick[f];      // (entries past n_eff are not used)
#pragma unroll
            for (int f = 0; f < kMaxNSel; ++f) rank += (f < n_eff && p[f] < pick) ? 1 : 0;
        }
        out[rank] = pick;
    }
}

// (eight workgroups per CU: 64 registers)
__global__ void __launch_bounds__(kThreads, 8) k_topn(const TopnArgs a) {
    extern __shared__ __align__(16) char smem[];
    uint32_t* s_bits = reinterpret_cast<uint32_t*>(smem);                 // [max_blocks] importance bit patterns (forced: +inf)
    uint64_t* s_best = reinterpret_cast<uint64_t*>(smem + (((size_t)a.max_blocks * 4 + 15) & ~(size_t)15));   // [256] per-thread best keys
    uint64_t* s_cand = s_best + kThreads;                                 // [kMaxCand]
    uint64_t* s_red = s_cand + kMaxCand;                                  // [16]: threshold, counter, argmax scratch
    int* s_pick = reinterpret_cast<int*>(s_red + 16);                     // [kMaxNSel]
    AncSet* s_anc = reinterpret_cast<AncSet*>(s_pick + kMaxNSel);
    int* s_par = reinterpret_cast<int*>(s_anc + kMaxT);
    int* s_depth = s_par + kMaxT;
    int* s_cmax = s_depth + kMaxT;

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int g = blockIdx.x % a.H_kv;
    const int x = (blockIdx.x / a.H_kv) % a.T;
    const int b = blockIdx.x / (a.H_kv * a.T);

    const MetaFetch mf = fetch_tree_meta(b, a.T, a.seq_lens, a.n_query, a.n_cmp);
    const SeqMeta sm = build_tree_meta(tid, mf, b, a.T, a.parents, a.l, a.d, a.max_seq_len, a.max_n_cmp, s_par, s_depth, s_cmax, s_anc);
    if (x >= sm.Tq) {
        if (tid < a.n_sel) a.sel_idx[(((int64_t)b * a.T + x) * a.H_kv + g) * a.n_sel + tid] = -1;
        return;
    }
    // rows [m0, m1) receive the set selected for query i
    int i = x, m0 = x, m1 = x + 1;
    if (a.share) {
        m0 = x * a.share;
        if (m0 >= sm.Tq) return;
        m1 = min(m0 + a.share, sm.Tq);
        i = group_representative(s_depth, m0, m1);
    }
    const int ncv = min(s_cmax[i], a.nc_pitch);
    const int J = min((sm.L + i) / a.l_sel, a.max_blocks - 1);
    const int a_ratio = a.l_sel / a.d, b_ratio = a.l / a.d;
    const float* cs = a.colsum + (((int64_t)b * a.T + i) * a.H_kv + g) * a.nc_pitch;
    const int n_eff = min(a.n_sel, J + 1);
    if (tid == 0) s_red[1] = 0;     // candidate counter
    if (tid < 4) s_red[12 + tid] = 0;   // per-wavefront thresholds

    // imp[j] = sum_delta wt[delta] * colsum[a_ratio * j + delta], delta in [-(b_ratio-1), a_ratio-1], where wt counts
    // the (m, n') pairs with m - n' = delta.  Loads are unconditional (clamped column, zero weight) and issued
    // for several blocks at once so that they are in flight together.
    const int n_terms = a_ratio + b_ratio - 1;
    uint64_t best = 0;   // best key among the blocks owned by this thread (index % 256 == tid)
    // The trailing local blocks are forced and need no importance: leaving them out of the load loop saves a
    // whole batch of loads whenever J + 1 is just above a multiple of the batch (contexts of 2^k tokens).
    const int j_last_scored = J - max(a.n_local, 0);
    for (int j = max(j_last_scored + 1, 0); j <= J; ++j) {
        if ((j % kThreads) == tid) {          // the owner of block j
            s_bits[j] = 0x7F800000u;
            const uint64_t key = topn_key(0x7F800000u, j);
            best = key > best ? key : best;
        }
    }
    if (a_ratio == 4 && b_ratio == 2) {
        // the standard geometry: block j takes columns 4j-1 .. 4j+3 with weights 1 2 2 2 1; one 16-byte and one 4-byte
        // load per block, four blocks per thread in flight (the same terms in the same order as the general form below;
        // eight in flight would not fit the 64 registers that eight workgroups per CU leave)
        constexpr int NF = 4;
        for (int j0 = tid; j0 <= j_last_scored; j0 += kThreads * NF) {
            f32x4 x[NF];
            float xm[NF];
#pragma unroll
            for (int v = 0; v < NF; ++v) {
                const int j = j0 + v * kThreads;
                const int c0 = j <= j_last_scored ? 4 * j : 0;
                // (a row holds nc_pitch columns, a multiple of 64: a block starting past it has no visible column)
                x[v] = *reinterpret_cast<const f32x4*>(cs + (c0 < ncv ? c0 : 0));
                xm[v] = cs[(c0 >= 1 && c0 - 1 < ncv) ? c0 - 1 : 0];
            }
#pragma unroll
            for (int v = 0; v < NF; ++v) {
                const int j = j0 + v * kThreads;
                if (j > j_last_scored) continue;
                const int c0 = 4 * j;
                float imp = 0.f;
                if (c0 >= 1 && c0 - 1 < ncv) imp += 1.f * xm[v];
                if (c0 < ncv) imp += 2.f * x[v][0];
                if (c0 + 1 < ncv) imp += 2.f * x[v][1];
                if (c0 + 2 < ncv) imp += 2.f * x[v][2];
                if (c0 + 3 < ncv) imp += 1.f * x[v][3];
                const uint32_t bits = j < a.n_init ? 0x7F800000u : __float_as_uint(imp);
                s_bits[j] = bits;
                const uint64_t key = topn_key(bits, j);
                best = key > best ? key : best;
            }
        }
    } else
    for (int j0 = tid; j0 <= j_last_scored; j0 += kThreads * kBlocksPerBatch) {
        float imp[kBlocksPerBatch];
        if (n_terms <= kMaxImpTerms) {
            float x[kBlocksPerBatch][kMaxImpTerms];
#pragma unroll
            for (int v = 0; v < kBlocksPerBatch; ++v)
#pragma unroll
                for (int u = 0; u < kMaxImpTerms; ++u) {
                    const int c = a_ratio * (j0 + v * kThreads) + u - (b_ratio - 1);
                    x[v][u] = cs[(u < n_terms && c >= 0 && c < ncv) ? c : 0];
                }
#pragma unroll
            for (int v = 0; v < kBlocksPerBatch; ++v) {
                imp[v] = 0.f;
#pragma unroll
                for (int u = 0; u < kMaxImpTerms; ++u) {
                    const int delta = u - (b_ratio - 1);
                    const int c = a_ratio * (j0 + v * kThreads) + delta;
                    const int pairs = min(min(a_ratio, b_ratio), min(delta + b_ratio, a_ratio - delta));
                    if (u < n_terms && c >= 0 && c < ncv) imp[v] += (float)pairs * x[v][u];
                }
            }
        } else {
            for (int v = 0; v < kBlocksPerBatch; ++v) {
                imp[v] = 0.f;
                const int j = j0 + v * kThreads;
                for (int m = 0; m < a_ratio && j <= J; ++m)
                    for (int n2 = 0; n2 < b_ratio; ++n2) {
                        const int c = a_ratio * j + m - n2;
                        if (c >= 0 && c < ncv) imp[v] += cs[c];
                    }
            }
        }
#pragma unroll
        for (int v = 0; v < kBlocksPerBatch; ++v) {
            const int j = j0 + v * kThreads;
            if (j <= j_last_scored) {
                const bool forced = j < a.n_init;
                const uint32_t bits = forced ? 0x7F800000u : __float_as_uint(imp[v]);
                s_bits[j] = bits;
                const uint64_t key = topn_key(bits, j);
                best = key > best ? key : best;
            }
        }
    }
    s_best[tid] = best;
    __syncthreads();

    // threshold: per wavefront, the n_eff-th largest of its per-thread bests (keys are distinct; threads without
    // blocks hold 0; a wavefront with fewer than n_eff keys leaves 0)
    {
        int rank = 0;
        const uint64_t* wb = s_best + wave * 64;
#pragma unroll 16
        for (int k = 0; k < 64; ++k) rank += wb[k] > best;   // broadcast LDS reads, 16 in flight
        if (best != 0 && rank == n_eff - 1) s_red[12 + wave] = best;
    }
    __syncthreads();
    uint64_t thr = s_red[12];
#pragma unroll
    for (int k = 1; k < 4; ++k) thr = s_red[12 + k] > thr ? s_red[12 + k] : thr;
    for (int j = tid; j <= J; j += kThreads) {
        const uint64_t key = topn_key(s_bits[j], j);
        if (key >= thr) {
            const unsigned slot = atomicAdd(reinterpret_cast<unsigned*>(&s_red[1]), 1u);
            if (slot < kMaxCand) s_cand[slot] = key;
        }
    }
    __syncthreads();
    const int n_cand = (int)*reinterpret_cast<unsigned*>(&s_red[1]);
    if (n_cand <= kMaxCand) {
        // rank candidates by counting; ranks below n_eff are the selection
        for (int e = tid; e < n_cand; e += kThreads) {
            const uint64_t key = s_cand[e];
            int rank = 0;
            int f = 0;
            for (; f + 8 <= n_cand; f += 8) {
                uint64_t c[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) c[u] = s_cand[f + u];
#pragma unroll
                for (int u = 0; u < 8; ++u) rank += c[u] > key;
            }
            for (; f < n_cand; ++f) rank += s_cand[f] > key;
            if (rank < n_eff) s_pick[rank] = (int)(0xFFFFFFFFu - (uint32_t)key);
        }
    } else {
        // fallback for massive ties: serial argmax, one winner per round
        for (int round = 0; round < n_eff; ++round) {
            const uint64_t wbest = wave_max_u64(best);
            uint64_t* red = s_red + 4 + (round & 1) * 4;
            if (lane == 0) red[wave] = wbest;
            __syncthreads();
            uint64_t top = red[0];
#pragma unroll
            for (int k = 1; k < 4; ++k) top = red[k] > top ? red[k] : top;
            const int j_top = (int)(0xFFFFFFFFu - (uint32_t)top);
            if (tid == 0) s_pick[round] = j_top;
            if ((j_top % kThreads) == tid) {       // the owner retires the winner and rescans its blocks
                s_bits[j_top] = 0xFFFFFFFFu;       // retired (no importance has this pattern)
                best = 0;
                for (int j = tid; j <= J; j += kThreads) {
                    const uint32_t bits = s_bits[j];
                    const uint64_t key = topn_key(bits, j);
                    if (bits != 0xFFFFFFFFu && key > best) best = key;
                }
            }
        }
    }
    __syncthreads();
    // ascending order: pick e goes to position (number of smaller picks); picks are distinct
    if (tid < a.n_sel) {
        int pick = 0x7fffffff, rank = tid;   // threads beyond n_eff write the -1 padding at their own position
        if (tid < n_eff) {
            pick = s_pick[tid];
            rank = 0;
            int p[kMaxNSel];
#pragma unroll
            for (int f = 0; f < kMaxNSel; ++f) p[f] = s_pick[f < n_eff ? f : 0];
#pragma unroll
            for (int f = 0; f < kMaxNSel; ++f) rank += (f < n_eff && p[f] < pick) ? 1 : 0;
        }
        for (int m = m0; m < m1; ++m)
            a.sel_idx[(((int64_t)b * a.T + m) * a.H_kv + g) * a.n_sel + rank] = tid < n_eff ? pick : -1;
    }
}

}  // namespace ssv
