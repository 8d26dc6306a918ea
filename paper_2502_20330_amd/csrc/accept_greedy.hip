// The greedy limit T -> 0 of RAPID's validation loop (Alg. 1) for gfx950.
//
// As T -> 0, p and q become one-hot on the arg-max of their logits, the mixing term
// eta T (q - p) of Eq. new_target vanishes, and the ratio of the accept test behaves like
// exp(((z_x' - max z) - (zq_x' - max zq)) / T): it tends to infinity, 1 or 0 as the target's
// gap at the drafted token is above, equal to or below the drafter's gap.  A rejection and the
// bonus position emit the target's arg-max of that row (the limit of the residual for a draft
// that is the drafter's own arg-max, which is what a drafter proposes at T -> 0).  Equal maxima:
// the lowest index.  The accept test stays the literal r <= min(1, limit of the ratio).
//
// Two launches, every logit read once:
//   greedy_slice_argmax  per slice of every row: (max, lowest index of the max); bound by HBM
//   greedy_decide        one workgroup per sequence: rows combined, gaps compared in fp64 (the
//                        difference of two fp32 numbers is exact there), prefix length, token; bound by
//                        the latency of its chain of loads
#include <algorithm>

#include "logit_rows.h"
#include "rapid_internal.h"

namespace {

constexpr int kThreads = 256;
constexpr int kDecideWaves = 16;                       // waves of greedy_decide at most
constexpr int kSlice = kThreads * 16;

struct GreedyWs {
    int32_t* status;      // same place and meaning as in the general accept pass
    float* smax;          // [B][2 gmax + 1][W]
    int32_t* sidx;        // [B][2 gmax + 1][W]
    int W;
    size_t bytes;
};
__host__ __device__ inline size_t galign(size_t x) { return (x + 255) / 256 * 256; }
__host__ __device__ inline GreedyWs gcarve(void* base, int B, int gmax, int V)
{
    GreedyWs w;
    w.W = (V + kSlice - 1) / kSlice;
    char* p = static_cast<char*>(base);
    w.status = reinterpret_cast<int32_t*>(p); p += 256;
    const size_t n = (size_t)B * (2 * gmax + 1) * w.W;
    w.smax = reinterpret_cast<float*>(p); p += galign(n * sizeof(float));
    w.sidx = reinterpret_cast<int32_t*>(p); p += galign(n * sizeof(int32_t));
    w.bytes = (size_t)(p - static_cast<char*>(base));
    return w;
}

__device__ __forceinline__ int seq_gamma(const AcceptLaunch& a, int b)
{
    return a.gammas ? min(max(a.gammas[b], 0), a.gmax) : a.gmax;
}
// (value, index) pairs ordered by larger value, then lower index
__device__ __forceinline__ void take_better(float& m, int& i, float m2, int i2)
{
    if (m2 > m || (m2 == m && i2 < i)) { m = m2; i = i2; }
}

// The best pair of a wave, in every lane: the maximum (never a NaN: maxima start at -inf and NaN entries do not pass), then the lowest
// index that has it; lane permutes on the way to the vector unit, no LDS.  Lanes without a source keep their own value.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ int dpp_or_own(int v) { return __builtin_amdgcn_update_dpp(v, v, CTRL, ROW_MASK, 0xf, false); }
template <class Op>
__device__ __forceinline__ int wave_fold(int v, Op op)
{
    v = op(v, dpp_or_own<0x111, 0xf>(v));                     // row_shr 1, 2, 4, 8 inside rows of 16 lanes
    v = op(v, dpp_or_own<0x112, 0xf>(v));
    v = op(v, dpp_or_own<0x114, 0xf>(v));
    v = op(v, dpp_or_own<0x118, 0xf>(v));
    v = op(v, dpp_or_own<0x142, 0xa>(v));                     // lane 15 of a row into the next: rows 1 and 3
    v = op(v, dpp_or_own<0x143, 0xc>(v));                     // lane 31 into the upper half
    return __builtin_amdgcn_readlane(v, 63);
}
__device__ __forceinline__ void wave_best(float& m, int& idx)
{
    const float best = __int_as_float(wave_fold(__float_as_int(m), [](int x, int y) { return __float_as_int(fmaxf(__int_as_float(x), __int_as_float(y))); }));
    idx = wave_fold(m == best ? idx : 0x7fffffff, [](int x, int y) { return min(x, y); });
    m = best;
}

// Row y of sequence b: y <= gmax the target rows, then the draft rows.  Bound by the read: four 128-bit loads per thread, all in flight
// at once, STREAM: with the streaming hint (see launch_accept_greedy; 64 sequences of 128256 entries and 8 drafts, 558 MB, both launches: 97.0 us
// without it, 88.5 = 6.3 TB/s with it; 16 sequences of 4 to 8 drafts 21.0 and 20.4).  512 threads take 86.6 and 21.4, and 24 instead of 16 for 4096 rows of 100; eight loads
// 88.0 and 22.7 against 22.2 at 16 sequences of 6 drafts.  A thread's entries come in index order, so equal maxima keep the lowest index by themselves.
template <bool STREAM>
__global__ void __launch_bounds__(kThreads) greedy_slice_argmax(AcceptLaunch a, GreedyWs ws)
{
    __shared__ float shm[kThreads / 64];
    __shared__ int shi[kThreads / 64];
    const int w = blockIdx.x, y = blockIdx.y, b = blockIdx.z;
    // only the two status words: the words behind them are the general pass's call counters, which persist
    if (w == 0 && y == 0 && b == 0 && threadIdx.x < 2) ws.status[threadIdx.x] = 0;
    const int g = seq_gamma(a, b);
    const bool is_t = y <= a.gmax;
    const int k = is_t ? y : y - (a.gmax + 1);
    if (is_t ? (k > g) : (k >= g)) return;
    const float* row = is_t ? a.zt + ((int64_t)b * (a.gmax + 1) + k) * a.V : a.zd + ((int64_t)b * a.gmax + k) * a.V;
    constexpr int NV = kSlice / (4 * kThreads);
    const int i0 = w * kSlice + threadIdx.x * 4;
    const bool full = (int64_t)(w + 1) * kSlice <= a.V;
    floatx4 x[NV];
    load_runs<NV, STREAM>(x, row, i0, kThreads * 4, a.V, full);
    shift_runs(x, i0, kThreads * 4, a.V, full);
    float m = -INFINITY;
    int idx = 0x7fffffff;
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        if (!full && i0 + v * kThreads * 4 >= a.V) break;     // short rows: nothing left for this thread (whole waves leave)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int i = i0 + v * kThreads * 4 + j;
            // (-inf is a maximum like any other as long as it is an entry of the row)
            const bool first = x[v][j] == m && idx == 0x7fffffff && i < a.V;
            if (x[v][j] > m || first) { m = x[v][j]; idx = i; }
        }
    }
    wave_best(m, idx);
    if ((threadIdx.x & 63) == 0) { shm[threadIdx.x >> 6] = m; shi[threadIdx.x >> 6] = idx; }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int s = 1; s < kThreads / 64; ++s) take_better(m, idx, shm[s], shi[s]);
        const int64_t slot = ((int64_t)b * (2 * a.gmax + 1) + y) * ws.W + w;
        ws.smax[slot] = m;
        ws.sidx[slot] = idx;
    }
}

// One wave combines the slices of row y of sequence b; the result is valid in every lane.  first: the row's first 64 slices, one per lane,
// fetched before (so that the loads of several rows are in flight together).
struct Best { float m; int i; };
__device__ __forceinline__ Best fetch_slice(const GreedyWs& ws, int64_t row, int s)
{
    return s < ws.W ? Best{ws.smax[row * ws.W + s], ws.sidx[row * ws.W + s]} : Best{-INFINITY, 0x7fffffff};
}
__device__ __forceinline__ void row_argmax(const GreedyWs& ws, int64_t row, Best first, float& m, int& idx)
{
    m = -INFINITY;
    idx = 0x7fffffff;
    take_better(m, idx, first.m, first.i);
    for (int s = (threadIdx.x & 63) + 64; s < ws.W; s += 64) take_better(m, idx, ws.smax[row * ws.W + s], ws.sidx[row * ws.W + s]);
    wave_best(m, idx);
}

// One wave per position: the drafted token, its two logits and the slices of both rows are fetched side by side, and the
// wave of position k leaves the arg-max of target row k in LDS, where the decision finds that of row n (the first kKept rows:
// gmax has no small bound; beyond them row n is combined once more).
constexpr int kKept = 1024;
__global__ void __launch_bounds__(kDecideWaves * 64) greedy_decide(AcceptLaunch a, GreedyWs ws)
{
    __shared__ int target_arg[kKept];
    __shared__ int first_fail;
    const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int nrows = 2 * a.gmax + 1;
    if (tid == 0) first_fail = 0x7fffffff;
    __syncthreads();
    const int g = seq_gamma(a, b);
    for (int k = wave; k <= a.gmax; k += blockDim.x / 64) {
        // what does not depend on the sequence's own count of drafts is requested before that has arrived (rows past it hold whatever
        // an earlier call left, and are not used)
        const int64_t at = (int64_t)b * a.gmax + k;
        const Best first_t = fetch_slice(ws, (int64_t)b * nrows + k, lane);
        const Best first_d = k < a.gmax ? fetch_slice(ws, (int64_t)b * nrows + a.gmax + 1 + k, lane) : Best{-INFINITY, 0x7fffffff};
        const int drafted = k < a.gmax ? a.tokens[at] : 0;
        if (k > g) break;
        const bool pair = k < g;
        const int x = pair ? drafted : 0;
        const bool in_range = pair && x >= 0 && x < a.V;
        const float zx_t = in_range ? a.zt[((int64_t)b * (a.gmax + 1) + k) * a.V + x] : 0.f;
        const float zx_d = in_range ? a.zd[at * a.V + x] : 0.f;
        const double u = (double)a.uniforms[(int64_t)b * (a.gmax + 1) + k];
        float mt, md = 0.f;
        int it, id;
        row_argmax(ws, (int64_t)b * nrows + k, first_t, mt, it);
        if (pair) row_argmax(ws, (int64_t)b * nrows + a.gmax + 1 + k, first_d, md, id);
        if (lane != 0) continue;
        if (k < kKept) target_arg[k] = it;
        if (!pair) continue;
        double rho = 0.0;
        bool ok = false;
        if (in_range) {
            // gaps of the drafted token to the row maxima; differences of fp32 values are exact in fp64
            const double gap_t = (double)zx_t - (double)mt, gap_d = (double)zx_d - (double)md;
            rho = gap_t > gap_d ? INFINITY : (gap_t < gap_d ? 0.0 : 1.0);
            ok = u <= fmin(1.0, rho);
        } else {
            atomicAdd(ws.status + 0, 1);                      // id outside the vocabulary: rejected, and counted
        }
        if (a.ratio) a.ratio[at] = (float)rho;
        if (!ok) atomicMin(&first_fail, k);
    }
    __syncthreads();
    const int n = min(first_fail, g);
    if (n >= kKept) {                                         // uniform
        float m;
        int it;
        if (wave == 0) row_argmax(ws, (int64_t)b * nrows + n, fetch_slice(ws, (int64_t)b * nrows + n, lane), m, it);
        if (tid == 0) target_arg[0] = it;
        __syncthreads();
    }
    for (int k = tid; k <= a.gmax; k += blockDim.x) {
        int tok = -1;
        if (k < n) tok = a.tokens[(int64_t)b * a.gmax + k];
        else if (k == n) {                                    // target row n: rejection or bonus position
            tok = target_arg[n < kKept ? n : 0];
            if (tok < 0 || tok >= a.V) tok = 0;               // a row of NaNs has no arg-max: any valid id
        }
        a.out_tokens[(int64_t)b * (a.gmax + 1) + k] = tok;
    }
    if (a.fill_ratio)
        for (int k = g + tid; k < a.gmax; k += blockDim.x) a.ratio[(int64_t)b * a.gmax + k] = 0.f;
    if (tid == 0) a.n_accepted[b] = n;
}

}  // namespace

size_t accept_greedy_workspace_bytes(int B, int gmax, int V)
{
    return gcarve(nullptr, B, gmax, V).bytes;
}

hipError_t launch_accept_greedy(const AcceptLaunch& a, hipStream_t stream)
{
    GreedyWs ws = gcarve(a.workspace, a.B, a.gmax, a.V);
    // The streaming hint from 80 MiB of logits on.  Logits that are still in the caches, as when the head has just written them, are
    // read faster without it in smaller calls, others with it in all (calls in a graph, us without and with it; one set of logits again and again, sets past the
    // caches): 35 MB 9.1 and 9.7, 11.6 and 10.8; 46 MB of rows of 8192 10.2 and 11.3, 13.3 and 12.1; 74 MB of 32000 14.4 and 14.8, 16.8 and 15.7; 87 MB
    // 15.8 and 15.5, 18.1 and 17.0; 174 MB 25.1 and 25.0, 28.3 and 26.2; 349 MB 42.6 and 42.9, 49.4 and 45.1; 558 MB 74.8 and 66.2, 73.3 and 65.6.
    const bool streams = (int64_t)a.B * (2 * a.gmax + 1) * a.V * 4 >= 80 << 20;
    hipLaunchKernelGGL(streams ? greedy_slice_argmax<true> : greedy_slice_argmax<false>, dim3(ws.W, 2 * a.gmax + 1, a.B), dim3(kThreads), 0,
                       stream, a, ws);
    // A wave per position while every sequence has a compute unit to itself (the decision is then one chain of loads), four
    // beyond, where the chip is full: 4096 sequences of one draft (vocabulary 100) took 53 us a call with 16 waves, 28 with four,
    // and 21 since the row pass also leaves out what lies past a short row.
    const int waves = std::min(a.gmax + 1, a.B <= a.n_cu ? kDecideWaves : 4);
    hipLaunchKernelGGL(greedy_decide, dim3(a.B), dim3(waves * 64), 0, stream, a, ws);
    return hipGetLastError();
}
