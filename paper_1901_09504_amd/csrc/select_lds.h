// Device-side pieces of the greedy channel selection of Sec. 3.4, shared by the selector kernel
// and by the weight pass that runs the selection in its own prologue.
//
// The list of channel maxima lives in LDS: `vals` holds one slot per expanded channel, `src` and
// `dep` the original channel and the number of halvings of each.  The paper splits one channel at a
// time, always the one with the largest value, the lowest expanded index among equals.  That
// sequence does not have to be walked step by step: with M the largest value of the list, every
// entry above M/2 is split before any half that these splits leave behind (a half is at most M/2),
// so a whole ROUND of splits is the entries above M/2 in descending order, lowest index first among
// equals, and the i-th of them appends expanded channel cur + i.  After the round the largest value
// is exactly M/2 (the halves of M), and the next round holds at least twice as many entries as there
// were halves of M: s splits take at most log2(s) + 2 rounds, whatever the values.  A round is a
// handful of passes over the list by the whole workgroup; a split costs no sequential step.
#pragma once
#include "ocs_internal.h"

namespace ocs {

// Channel maxima from the column maxima of `blocks` row blocks, colmax[blocks][K = C * g], into vals[0 .. C), src/dep set to
// the identity.  Independent 16-byte loads, a lane's eight or sixteen on their way together (the maxima were written a moment ago by
// other CUs and every load waits a whole trip through the fabric), folded per channel with LDS atomics on the bit
// pattern.  Lanes are dealt over a block's groups of four columns first, then over the blocks; the last group of a block is
// its last four columns, some of which may be another group's as well (K >= 4 with several blocks).  Called by all NT lanes of the workgroup;
// contains barriers, and ends with one.
// BLOCKS: more than one, in an instance of its own.
template <int NT, bool BLOCKS>
__device__ __forceinline__ void channel_maxima_to_lds(const float* __restrict__ colmax, int blocks, int C, int g,
                                                      float* vals, unsigned short* src, unsigned short* dep) {
    const int tid = threadIdx.x;
    for (int j = tid; j < C; j += NT) {
        vals[j] = 0.0f;
        src[j] = (unsigned short)j;
        dep[j] = 0;
    }
    __syncthreads();
    const int K = C * g;
    unsigned* vbits = reinterpret_cast<unsigned*>(vals);
    if constexpr (!BLOCKS) {
        // (a column per lane: four atomics behind one 16-byte load are longer than the loads, 256 x 256 x 9 7.1 against 7.6 us.
        // The compiler keeps a load behind the LDS atomic that precedes it in program order, so a plain loop, unrolled or
        // not, makes one trip per column of a lane: several are requested before the first value is used.)
        constexpr int U1 = NT >= 1024 ? 4 : 16;
        for (int k0 = tid; k0 < K; k0 += U1 * NT) {
            float v[U1];
#pragma unroll
            for (int u = 0; u < U1; ++u) {
                const int k = k0 + u * NT;
                v[u] = colmax[k < K ? k : K - 1];
            }
#pragma unroll
            for (int u = 0; u < U1; ++u) {
                const int k = k0 + u * NT;
                if (k < K) atomicMax(&vbits[k / g], __float_as_uint(v[u]));
            }
        }
    } else {
        constexpr int UN = NT >= 1024 ? 16 : 8;
        const int units = (K + 3) / 4;
        const int groups = units < NT ? NT / units : 1;           // blocks walked side by side
        const int b0 = units < NT ? tid / units : 0, u0 = tid - b0 * units;
        if (b0 < groups) {
            for (int u = u0; u < units; u += NT) {                // (one trip where units < NT)
                const int col = 4 * u < K - 4 ? 4 * u : K - 4;
                f32x4 m = {0.0f, 0.0f, 0.0f, 0.0f};
                for (int b = b0; b < blocks; b += UN * groups) {
                    f32x4 v[UN] = {};
#pragma unroll
                    for (int q = 0; q < UN; ++q)
                        if (b + q * groups < blocks) v[q] = *reinterpret_cast<const f32x4u*>(colmax + (int64_t)(b + q * groups) * K + col);
#pragma unroll
                    for (int q = 0; q < UN; ++q)
#pragma unroll
                        for (int e = 0; e < 4; ++e) m[e] = fmaxf(m[e], v[q][e]);
                }
#pragma unroll
                for (int e = 0; e < 4; ++e) atomicMax(&vbits[(col + e) / g], __float_as_uint(m[e]));
            }
        }
    }
    __syncthreads();
}

// Scratch of greedy_rounds in LDS.
constexpr int kGreedyBins = 256;
struct GreedyScratch {
    unsigned hist[kGreedyBins];
    unsigned red[16];
    unsigned count[2], bin, before, size;
};
// LDS of the list: the keys of a round's entries, the values, sources and depths (in this order).
__host__ __device__ inline unsigned greedy_list_bytes(int E) { return (unsigned)E * 16u; }

// Largest of `v` over the workgroup (bit patterns of non-negative floats).  Two barriers.
template <int NT>
__device__ __forceinline__ unsigned group_umax(unsigned v, unsigned* red) {
    v = wave_umax32(v);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    v = red[0];
#pragma unroll
    for (int w = 1; w < NT / 64; ++w) v = red[w] > v ? red[w] : v;
    __syncthreads();
    return v;
}

// A few steps on a short list, one after the other by the first wave alone: lane l keeps entries l, l + 64, ... of the
// list (values only) and the copies, one per lane, in registers.  A step is the wave's maximum and, for the lowest index
// that holds it, one comparison per register whose result is a scalar mask: no barrier, no read from LDS.  A
// round costs the same whatever it holds, and most when it is cut (a bound on its keys is searched first):
// 256 x 256 x 9 with 3 splits, selector alone 8.9 -> 7.2 us, the whole preparation 11.1 -> 9.8; 1024 x 256 12.4 -> 11.1.
template <int S>
__device__ __forceinline__ void greedy_few(float* vals, unsigned short* src, unsigned short* dep, int C, int s,
                                           int32_t* split_src) {
    if (threadIdx.x < 64) {
        const int lane = (int)threadIdx.x;
        int v[S];                                                // bit patterns; -1: no such entry
#pragma unroll
        for (int q = 0; q < S; ++q) {
            const bool in = q * 64 + lane < C;
            const int bits = (int)__float_as_uint(vals[in ? q * 64 + lane : 0]);
            v[q] = in ? bits : -1;
        }
        int w = -1, wsrc = 0, wdep = 0, wsplit = -1;             // lane i: value, source and depth of copy i; what step i split
        for (int i = 0; i < s; ++i) {
            int best = w > 0 ? w : 0;
#pragma unroll
            for (int q = 0; q < S; ++q) best = v[q] > best ? v[q] : best;
            const int top = (int)wave_umax32((unsigned)best);
            unsigned long long at = __ballot(w == top);
            int js = C + __ffsll((long long)at) - 1;
#pragma unroll
            for (int q = S - 1; q >= 0; --q) {
                at = __ballot(v[q] == top);
                js = at != 0 ? q * 64 + __ffsll((long long)at) - 1 : js;
            }
            js = __builtin_amdgcn_readfirstlane(js);
            const float half = __int_as_float(top) * 0.5f;
            const int hbits = __float_as_int(half);
            const bool copy = js >= C;
            const int k = copy ? js - C : 0, cur = C + i;
            const int from = copy ? __builtin_amdgcn_readlane(wsrc, k) : js;
            const int d = 1 + (copy ? __builtin_amdgcn_readlane(wdep, k) : __popcll(__ballot(wsplit == js)));
            const int here = (copy ? -64 : js) - lane;           // 64 q in the lane and register of the split entry
#pragma unroll
            for (int q = 0; q < S; ++q) v[q] = here == 64 * q ? hbits : v[q];
            const bool changed = lane == i || (copy && lane == k);
            w = changed ? hbits : w;
            wdep = changed ? d : wdep;
            wsrc = lane == i ? from : wsrc;
            wsplit = lane == i ? js : wsplit;
            if (lane == 0) {
                vals[js] = half;
                vals[cur] = half;
                dep[js] = (unsigned short)d;
                dep[cur] = (unsigned short)d;
                src[cur] = (unsigned short)from;
                if (split_src) split_src[i] = js;
            }
        }
    }
    __syncthreads();
}
// Where that is ahead of the rounds: 0.35 us a step up to 256 channels, 0.5 up to 640, 0.65 above.  Level with the rounds at 3 to
// 4 splits of 64 channels (so few entries are ranked without the search), at 7 of 256, 6 of 512, 4 of 800.
__host__ __device__ inline bool few_steps(int C, int s) {
    return s <= (C <= 96 ? 3 : (C <= 640 ? 6 : 4)) && C <= 1024;
}

// The s greedy steps on a list of C entries, by all NT lanes.  split_src (may be null) receives the
// expanded index chosen at every step.  Contains barriers, and ends with one.
//   Sort key of an entry of the round: (M - value) in units of the last place (below 2^23: values lie
//   in (M/2, M]) above the index (13 bits): ascending keys are the order of the splits, and no two are
//   equal.  An entry's place is the number of smaller keys of the round, counted by all lanes; when a
//   round holds more entries than splits are left and too many to count over, a bound on the largest
//   key that still takes part is found first, digit by digit (8 bits at a time, a histogram in LDS per
//   digit) until few enough entries lie below it.
//   HELD: the list is at most HELD pieces of NT entries.
template <int NT, int HELD>
__device__ __forceinline__ void greedy_rounds(float* vals, unsigned short* src, unsigned short* dep,
                                              unsigned long long* cand, GreedyScratch& sc, int C, int s,
                                              int32_t* split_src) {
    static_assert(NT % 64 == 0 && NT / 64 <= 16 && NT >= kGreedyBins, "waves of the workgroup");
    const int tid = (int)threadIdx.x, lane = tid & 63;
    const unsigned* vbits = reinterpret_cast<const unsigned*>(vals);
    if (s <= 0) return;
    unsigned m = 0;
    if (tid == 0) sc.count[0] = 0;
    for (int j = tid; j < C; j += NT) m = vbits[j] > m ? vbits[j] : m;
    unsigned mbits = group_umax<NT>(m, sc.red);
    int cur = C, rem = s, turn = 0;
    while (rem > 0) {
        const unsigned hbits = __float_as_uint(__uint_as_float(mbits) * 0.5f);
        if (!(mbits > hbits)) {
            // nothing but zeros left (or an infinite channel): halving changes no value any more, and
            // every remaining step takes the lowest index that holds the largest value
            unsigned low = 0;                                    // complemented index: largest = lowest index
            for (int j = tid; j < cur; j += NT)
                if (vbits[j] == mbits) { low = 0xFFFFFFFFu - (unsigned)j; break; }
            const int js = (int)(0xFFFFFFFFu - group_umax<NT>(low, sc.red));
            const unsigned short s0 = src[js];
            const int d0 = dep[js];
            __syncthreads();                                     // everyone has read entry js
            for (int i = tid; i < rem; i += NT) {
                vals[cur + i] = __uint_as_float(hbits);
                src[cur + i] = s0;
                dep[cur + i] = (unsigned short)(d0 + i + 1);
                if (split_src) split_src[cur + i - C] = js;
            }
            if (tid == 0) {
                vals[js] = __uint_as_float(hbits);
                dep[js] = (unsigned short)(d0 + rem);
            }
            __syncthreads();
            return;
        }
        auto key_of = [&](unsigned v, int j) { return ((unsigned long long)(mbits - v) << 13) | (unsigned long long)j; };
        auto before = [&](unsigned long long mask) {
            return (int)__builtin_amdgcn_mbcnt_hi((unsigned)(mask >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)mask, 0));
        };
        // (counting costs in_round^2 / NT look-ups per lane, a digit three barriers: level at about 32
        // look-ups)
        auto countable = [&](int n) { return n * n <= 32 * NT; };
        // The round's entries, in no order yet.  Sixteen waves on four SIMDs, once through code that no cache holds: what a round costs is its
        // instructions, their fetches, and the trips to LDS that wait for each other.  A wave reads its part of the list once, a
        // value a lane and piece, all on their way together, and keeps it for the round; it takes the places of all its entries
        // with one LDS atomic, and makes their keys at once unless its own are too many for a round that is not cut.  Kernel alone in
        // a graph, us, keys made piece by piece with an atomic each / counted first and read again / so: 2000 channels, 40 splits,
        // heavy tails 12.1 / 12.6 / 11.3, 3700 x 185 16.2 / 15.5 / 14.6, 7000 x 350 27.2 / 26.7 / 24.5; 300 x 512 whole
        // preparation, 26 splits, 12.5 / 11.8 / 11.5.  Instances for two, four and eight pieces: eight for all 8.7 -> 9.7 at 1024.
        unsigned v[HELD], own = 0, first = 0;
        unsigned long long mask[HELD];
#pragma unroll
        for (int q = 0; q < HELD; ++q) v[q] = vbits[q * NT + tid < cur ? q * NT + tid : cur - 1];
#pragma unroll
        for (int q = 0; q < HELD; ++q) {
            mask[q] = __ballot(v[q] > hbits && q * NT + tid < cur);
            own += (unsigned)__popcll(mask[q]);
        }
        // f(value, entries of this wave's piece, index) for every piece that has any
        auto each = [&](auto&& f) {
#pragma unroll
            for (int q = 0; q < HELD; ++q)
                if (mask[q] != 0) f(v[q], mask[q], q * NT + tid);
        };
        if (own != 0 && lane == 0) first = atomicAdd(&sc.count[turn], own);
        if ((int)own <= rem || countable((int)own)) {
            int base = __builtin_amdgcn_readfirstlane((int)first);
            each([&](unsigned u, unsigned long long m, int j) {
                if ((m >> lane) & 1) cand[base + before(m)] = key_of(u, j);
                base += __popcll(m);
            });
        }
        __syncthreads();
        int in_round = __builtin_amdgcn_readfirstlane((int)sc.count[turn]);
        turn ^= 1;
        if (tid == 0) sc.count[turn] = 0;                        // (last read before the barrier that ended the round before)
        if (in_round > rem && !countable(in_round)) {
            // the rem smallest keys: find the largest of them
            unsigned long long prefix = 0;       // digits fixed so far
            int need = rem;
            unsigned long long cut = 0;
            int shift = 28;                      // 36 key bits: digits at 28, 20, 12, 4 and the last 4 bits
            for (;;) {
                const int width = shift == 0 ? 4 : 8;
                if (tid < kGreedyBins) sc.hist[tid] = 0;
                __syncthreads();
                each([&](unsigned u, unsigned long long m, int j) {
                    const unsigned long long k = key_of(u, j);
                    if (((m >> lane) & 1) && (k >> (shift + width)) == prefix)
                        atomicAdd(&sc.hist[(unsigned)(k >> shift) & ((1u << width) - 1u)], 1u);
                });
                __syncthreads();
                if (tid < 64) {                  // first bin at which the running count reaches `need`
                    unsigned h4[4], sum = 0;
#pragma unroll
                    for (int e = 0; e < 4; ++e) { h4[e] = sc.hist[4 * tid + e]; sum += h4[e]; }
                    unsigned incl = sum;
#pragma unroll
                    for (int o = 1; o < 64; o <<= 1) {
                        const unsigned up = (unsigned)__shfl_up((int)incl, o);
                        if (tid >= o) incl += up;
                    }
                    unsigned run = incl - sum;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        if (run < (unsigned)need && run + h4[e] >= (unsigned)need) {
                            sc.bin = 4 * tid + e;
                            sc.before = run;
                            sc.size = h4[e];
                        }
                        run += h4[e];
                    }
                }
                __syncthreads();
                prefix = (prefix << width) | sc.bin;
                need -= (int)sc.before;
                in_round = rem - need + (int)sc.size;            // entries up to and in that bin
                if (in_round == rem || countable(in_round) || shift == 0) {
                    cut = ((prefix + 1) << shift) - 1;
                    break;
                }
                shift = shift >= 12 ? shift - 8 : 0;
            }
            each([&](unsigned u, unsigned long long m, int j) {
                const unsigned long long k = key_of(u, j), in = __ballot(((m >> lane) & 1) && k <= cut);
                unsigned base = 0;
                if (lane == 0) base = atomicAdd(&sc.count[turn], (unsigned)__popcll(in));
                base = (unsigned)__builtin_amdgcn_readfirstlane((int)base);
                if ((in >> lane) & 1) cand[(int)base + before(in)] = k;
            });
            __syncthreads();
        }
        const int take = in_round < rem ? in_round : rem;
        // rank of every entry of the round = how many keys are smaller; G lanes share one entry's count
        int log2_G = 0;
        while (log2_G < 4 && (in_round << (log2_G + 1)) <= NT) ++log2_G;
        const int G = 1 << log2_G;
        const int per = NT >> log2_G;
        for (int i0 = 0; i0 < in_round; i0 += per) {
            const int i = i0 + (tid >> log2_G);
            const unsigned long long mine = i < in_round ? cand[i] : 0ull;
            int rank = 0;
            if (i < in_round) {
                int k = tid & (G - 1);
                for (; k + 3 * G < in_round; k += 4 * G)
                    rank += (cand[k] < mine) + (cand[k + G] < mine) + (cand[k + 2 * G] < mine) +
                            (cand[k + 3 * G] < mine);
                for (; k < in_round; k += G) rank += cand[k] < mine;
            }
            for (int o = 1; o < G; o <<= 1) rank += __shfl_xor(rank, o);
            if (i < in_round && rank < take && (tid & (G - 1)) == 0) {
                const int j = (int)(mine & 0x1FFFull), n = cur + rank;
                const float half = vals[j] * 0.5f;
                const unsigned short s0 = src[j], d = (unsigned short)(dep[j] + 1);
                vals[j] = half;
                vals[n] = half;
                dep[j] = d;
                dep[n] = d;
                src[n] = s0;
                if (split_src) split_src[n - C] = j;
            }
        }
        __syncthreads();
        cur += take;
        rem -= take;
        mbits = hbits;          // the halves of M are the largest entries now (a cut round is the last one)
    }
}

// One or the other, as the launch says (FEW: few_steps holds), in instances of their own: the rounds' kernels stay what
// they are without the steps' code.
template <int NT, bool FEW, int HELD>
__device__ __forceinline__ void greedy_select(float* vals, unsigned short* src, unsigned short* dep, unsigned long long* cand,
                                              GreedyScratch& sc, int C, int s, int32_t* split_src) {
    if constexpr (FEW) {
        if (C <= 256) greedy_few<4>(vals, src, dep, C, s, split_src);
        else if (C <= 320) greedy_few<5>(vals, src, dep, C, s, split_src);
        else if (C <= 512) greedy_few<8>(vals, src, dep, C, s, split_src);
        else if (C <= 640) greedy_few<10>(vals, src, dep, C, s, split_src);
        else greedy_few<16>(vals, src, dep, C, s, split_src);
    } else {
        greedy_rounds<NT, HELD>(vals, src, dep, cand, sc, C, s, split_src);
    }
}

}  // namespace ocs
