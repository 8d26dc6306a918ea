// Exchange of the split partials inside the attention kernel, and the merge of a query row: used by the split kernels,
// whose workgroups then merge their sequence's rows themselves, and by the merge kernel.
#pragma once
#include "rapid_internal.h"

namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

// Reductions over 32 values, one per lane of the wave's lower and again of its upper half; result in every lane.
template <int ROR>
__device__ __forceinline__ float row_ror(float v)      // rotation inside rows of 16 lanes, without LDS
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x120 + ROR, 0xf, 0xf, false));
}
__device__ __forceinline__ float lane_of(float v, int lane) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane)); }
__device__ __forceinline__ float max32(float v)
{
    v = fmaxf(v, row_ror<8>(v));
    v = fmaxf(v, row_ror<4>(v));
    v = fmaxf(v, row_ror<2>(v));
    v = fmaxf(v, row_ror<1>(v));
    return fmaxf(lane_of(v, 0), lane_of(v, 16));
}
__device__ __forceinline__ float sum32(float v)
{
    v += row_ror<8>(v);
    v += row_ror<4>(v);
    v += row_ror<2>(v);
    v += row_ror<1>(v);
    return lane_of(v, 0) + lane_of(v, 16);
}

constexpr int kMergeBlock = 32;        // splits whose weights are formed together, one per lane

// ---- one launch for the whole call.
// Every workgroup of a team, the splits of a (sequence, kv head), publishes its partial, or that it holds no tokens, and then merges its share of the
// team's output, every share as many elements.  What it publishes are 64-bit words, 32 bits of payload under a tag that no
// earlier call on the same memory used; whoever needs a word looks until it carries the tag, so no fence, flag or counter
// stands between a store and its reader.  The memory holds nothing but such words and starts as zeros.  The tag is the number of the call, and never 0,
// the tag of a word that nobody has written.  (32 bits: a word that exactly 2^32 - 1 calls have left alone would pass for new.)
// Every possible team has a copy of it, moved by a plain store once the first share of a team has been merged: all
// workgroups of the team have read it then.  Replays of a captured graph move it too.  Two calls that overlap in time on one memory can leave unequal
// copies, and then a team may later meet words of another one under its own tag: the memory has to be cleared (rapid.h).
//
// No workgroup depends on another one for its end.  It looks for a bounded time; then it marks its share as left over and looks
// once more.  Every wave, after its own words have arrived in memory, looks at the marks, and its workgroup merges what is left
// over where all words are there.  Store, then look, on both sides: of the one who marks and the one whose word was missing,
// the later one sees what the other has stored, and the last of a team to publish finds everything.  (Two may merge the same
// share, to the same bits.)
//
// What bounds it: round trips past the dies' L2s (0.7 us each: the own words' arrival, one or two looks) and code that every
// workgroup meets for the first time, about 3 us from the last tile to the end at 4 rows where a store, a second launch and its
// gap took 3.6.  So everything that is missing is asked for at once, one element of the output a thread, and partials keep
// the order of the merge kernel.  Measured: 2K tokens, 4/1 heads of 64, 5 positions, enqueued one by one 9.9 -> 7.9 us, in a graph 8.2 -> 8.0; 4 rows 7.1 -> 6.8.  Not kept (a graph
// of 16 calls on 8K tokens with the head and the draw, 290 us with two launches, 277 like this): a counter of arrivals per team (256 atomic additions on a few
// lines: 345); a wave per row asking for 32 splits (304); asking for words only where (maximum, sum) had come (282 to 292).
struct Exchange {
    AttnExchangeHead* head;
    __amdgpu_buffer_rsrc_t words;
    uint32_t tag;
};
constexpr int kDeviceScope = 16;       // sc1: past the dies' own L2s

// The number of this call, read by every workgroup beside its sequence's length.
__device__ __forceinline__ uint32_t exchange_call(const AttnLaunch& a, int team, int& L)
{
    uint32_t calls = a.xhead->calls[team];
    calls = __builtin_amdgcn_readfirstlane(calls);
    L = __builtin_amdgcn_readfirstlane(L);
    asm volatile("" : "+s"(calls), "+s"(L));
    return calls;
}
__device__ __forceinline__ Exchange make_exchange(const AttnLaunch& a, uint32_t calls)
{
    Exchange x;
    x.head = a.xhead;
    x.words = __builtin_amdgcn_make_buffer_rsrc(a.xwords, 0, a.xbytes, 0x00027000);
    x.tag = calls + 1 ? calls + 1 : 1;
    return x;
}
// Two values side by side; `at` in words.
__device__ __forceinline__ void publish_pair(const Exchange& x, uint32_t at, float v0, float v1)
{
    const u32x4 w = {__float_as_uint(v0), x.tag, __float_as_uint(v1), x.tag};
    __builtin_amdgcn_raw_buffer_store_b128(w, x.words, at * 8, 0, kDeviceScope);
}

// A query row's state while its splits are folded in, 32 at a time.
struct RowMerge {
    float M = -INFINITY, den = 0.f;
    // weight of this lane's split of the block (lane % 32); resc: what the sums so far are multiplied by
    __device__ __forceinline__ float block(float m, float l, float* resc)
    {
        const float Mn = fmaxf(M, max32(m));
        const float Mu = (Mn == -INFINITY) ? 0.f : Mn;
        *resc = __builtin_amdgcn_exp2f(M - Mu);
        M = Mn;
        const float w = __builtin_amdgcn_exp2f(m - Mu);
        den = den * *resc + sum32(w * l);
        return w;
    }
};

// What lies in LDS while a workgroup merges.
template <int ROWS, int NWAVES>
struct MergeLds {
    float weight[ROWS][kMergeBlock];                   // of the share's rows, for each split
    float den[ROWS], top[ROWS];                        // sum and maximum of a row
    uint32_t missing[NWAVES], seen[NWAVES];            // not all words there; marks of the team, by wave
    float vals[];                                      // [split][element of the share]
};

// One try at a share (`share` of n) of a team whose partials start at row slot `base`: every wave looks until `ticks` have passed, or
// once (ticks < 0).  False: words are missing.
// The shares are those of all splits, so that a thread has one element whatever the length of the sequence is (plan_exchange).
template <int D, int ROWS, int NWAVES>
__device__ __forceinline__ bool merge_share(const AttnLaunch& a, const Exchange& x, char* smem, int team, uint32_t base, int live, int R,
                                            int share, int64_t ticks, bool first, uint32_t* marks)
{
    constexpr int NT = NWAVES * 64;
    MergeLds<ROWS, NWAVES>& lds = *reinterpret_cast<MergeLds<ROWS, NWAVES>*>(smem);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int RP = a.RB * 16, total = a.Qmax * a.G * D, n = a.nsplit;
    const int E = ((total + n - 1) / n + 15) & ~15;    // elements of a share; whole 32-byte pieces of the output
    const int e0 = share * E, e1 = min(e0 + E, total), er = min(e1, R * D);      // from er on: rows that this sequence does not have
    const int row0 = e0 / D, row1 = (er + D - 1) / D;
    const int64_t t0 = (int64_t)wall_clock64();
    bool missing = false;
    // Words of the share, two a time: pair p of split s.
    constexpr int U = ROWS * D / 2 / NT + 1;
    const int pairs = live ? max(er - e0, 0) / 2 : 0;
    uint32_t off[U];
    int at[U];                                         // place in LDS; -1: it is there
    {
        const int step = max(pairs, 1);
        const int ds = NT / step, dp = NT - ds * step;
        int s = tid / step, p = tid - s * step;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            at[u] = s < live && pairs ? s * E + p * 2 : -1;
            off[u] = ((base + s * RP) * D + e0 + p * 2) * 8;
            s += ds;
            p += dp;
            if (p >= step) { p -= step; ++s; }
        }
    }
    // Every look asks for all that is missing at once: the words, (maximum, sum) of the wave's first row, the marks of the team, one
    // per lane.  Marks count once this wave's own words have arrived, which is after the first look; they are needed in the end.
    int row = row0 + wave;
    const int sl = min(lane & (kMergeBlock - 1), n - 1);
    const uint32_t ml_at = a.xml_offset + (base + sl * RP + min(row, max(row1 - 1, 0))) * 16;
    const uint32_t* marks_at = &x.head->marks[team][lane & (kMaxShares - 1)];
    uint32_t mark = 0;
    u32x4 ml = {0, 0, 0, 0};
    for (bool early = true;; early = false) {
        ml = __builtin_amdgcn_raw_buffer_load_b128(x.words, ml_at, 0, kDeviceScope);
        mark = __hip_atomic_load(marks_at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        u32x4 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (at[u] >= 0) v[u] = __builtin_amdgcn_raw_buffer_load_b128(x.words, off[u], 0, kDeviceScope);
        bool open = row0 < row1 && (ml.y != x.tag || ml.w != x.tag);
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (at[u] >= 0) {
                if (v[u].y == x.tag && v[u].w == x.tag) {
                    *reinterpret_cast<float2*>(lds.vals + at[u]) = float2{__uint_as_float(v[u].x), __uint_as_float(v[u].z)};
                    at[u] = -1;
                } else {
                    open = true;
                }
            }
        missing = __any(open);
        if (!missing || ticks < 0 || (int64_t)wall_clock64() - t0 >= ticks) {
            if (early) {
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                mark = __hip_atomic_load(marks_at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            break;
        }
        asm volatile("" ::: "memory");
    }
    if (share == 0 && wave == NWAVES - 1 && !missing) {
        // this team's copy of the number, and those of the teams that this call does not have
        const int teams = a.B * a.Hkv;
        for (int t = team + teams * lane; t < kAttnTeams; t += teams * 64) x.head->calls[t] = x.tag;
    }
    // weights: a wave per row, split j in lane j
    for (; row < row1; row += NWAVES) {
        const bool real = (lane & (kMergeBlock - 1)) < live;
        float resc;
        RowMerge r;
        const float w = r.block(real ? __uint_as_float(ml.x) : -INFINITY, real ? __uint_as_float(ml.z) : 0.f, &resc);
        if (lane < kMergeBlock) lds.weight[row - row0][lane] = w;
        if (lane == 0) {
            lds.den[row - row0] = r.den;
            lds.top[row - row0] = r.M;
        }
        if (row + NWAVES < row1) {                     // (all have published)
            ml = __builtin_amdgcn_raw_buffer_load_b128(x.words, a.xml_offset + (base + sl * RP + row + NWAVES) * 16, 0, kDeviceScope);
            if (!__all(ml.y == x.tag && ml.w == x.tag)) missing = true;
        }
    }
    if (lane == 0) lds.missing[wave] = missing;
    __syncthreads();
    uint32_t any = 0;
#pragma unroll
    for (int w = 0; w < NWAVES; ++w) any |= lds.missing[w];
    const int b = team / a.Hkv, hkv = team - b * a.Hkv;
    for (int e = any ? e1 : e0 + tid; e < e1; e += NT) {
        const int row = e / D, d = e % D;
        const int qi = row / a.G, h = hkv * a.G + row % a.G;
        float num = 0.f;
        if (row < R) {
            const float* w = lds.weight[row - row0];
            const float* val = lds.vals + (e - e0);
            float acc[2] = {0.f, 0.f};
            int s = 0;
            for (; s + 16 <= live; s += 16) {
                floatx4 w4[4];
                float y[16];
#pragma unroll
                for (int i = 0; i < 4; ++i) w4[i] = *reinterpret_cast<const floatx4*>(w + s + i * 4);
#pragma unroll
                for (int i = 0; i < 16; ++i) y[i] = val[(s + i) * E];
#pragma unroll
                for (int i = 0; i < 16; ++i) acc[i & 1] = fmaf(w4[i / 4][i % 4], y[i], acc[i & 1]);
            }
            for (; s < live; s += 2) {
                acc[0] = fmaf(w[s], val[s * E], acc[0]);
                if (s + 1 < live) acc[1] = fmaf(w[s + 1], val[(s + 1) * E], acc[1]);
            }
            const float den = lds.den[row - row0];
            num = den > 0.f ? (acc[0] + acc[1]) / den : 0.f;
        }
        const __bf16 ob = (__bf16)num;
        a.out[(((int64_t)b * a.Qmax + qi) * a.Hq + h) * D + d] = __builtin_bit_cast(uint16_t, ob);
        if (a.lse_out && d == 0) {
            float lse = 0.f;
            if (row < R) lse = (lds.top[row - row0] + log2f(lds.den[row - row0])) * 0.6931471805599453f;
            a.lse_out[((int64_t)b * a.Hq + h) * a.Qmax + qi] = lse;
        }
    }
    if (first) {
        const uint32_t seen = (uint32_t)__ballot(mark == x.tag);
        if (lane == 0) lds.seen[wave] = seen;
        __syncthreads();
        uint32_t left = 0;
#pragma unroll
        for (int w = 0; w < NWAVES; ++w) left |= lds.seen[w];
        *marks = left;
    }
    return !any;
}

// What a workgroup does after it has published its partial (`live` splits hold tokens; the others say so here).
template <int D, int ROWS, int NWAVES>
__device__ __forceinline__ void exchange_finish(const AttnLaunch& a, uint32_t calls, char* smem, int team, int split, int live, int R)
{
    const Exchange x = make_exchange(a, calls);
    const uint32_t base = (uint32_t)team * a.nsplit * (a.RB * 16);
    uint32_t left = 0;
    int64_t ticks = a.xwait_ticks;
    int share = split;
    // What this workgroup published has been read out of LDS; and one without tokens publishes only now that all of its waves have read
    // the number of the call, which moves once all have published.
    __syncthreads();
    if (split >= live && (int)threadIdx.x < R)
        publish_pair(x, a.xml_offset / 8 + (base + split * (a.RB * 16) + threadIdx.x) * 2, -INFINITY, 0.f);
    for (;;) {
        const bool done = merge_share<D, ROWS, NWAVES>(a, x, smem, team, base, live, R, share, ticks, ticks >= 0, &left);
        if (!done && ticks >= 0) {
            if (threadIdx.x == 0) {
                __hip_atomic_store(&x.head->marks[team][share], x.tag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            }
            left |= 1u << share;                       // once more, without waiting
        }
        ticks = -1;
        if (!left) return;
        share = __ffs(left) - 1;
        left &= left - 1;
        __syncthreads();
    }
}

}  // namespace
