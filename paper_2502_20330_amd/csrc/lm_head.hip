// Output head of the target model for the verification rows, for gfx950 (MI355X):
//     z[r][v] = sum_k h[r][k] * W[v][k]          ("LogitsOf", Alg. 1)
// for the rows of a verification step (gamma+1 rows of one sequence, or of a batch: up to 96),
// with the per-chunk softmax statistics of every row (max z, sum exp((z - max)/T)) produced in
// the epilogue, so that the acceptance pass does not have to form them from the logits.
//
// With so few rows every weight is used 2 x rows times, so the kernel is bound by streaming W
// (vocab x hidden bf16, about 1 GB for a 128K vocabulary) from HBM, which is read once whatever
// the row count.  NR = number of 16-row blocks of h (1..6).
//
//  * One workgroup owns up to 512 consecutive vocabulary rows (4 MiB of W at hidden = 4096); the
//    host picks the row count (a multiple of 16) so that the grid fills the chip in whole rounds:
//    501 rows x 251 workgroups would leave a second round of 41 workgroups that cannot saturate
//    HBM, 304 rows x 501 workgroups does not.
//  * The four waves split the vocabulary range: wave w takes the 16-row blocks w, w + 4, ... (eight
//    at most) and runs over the whole hidden dimension for them, one slab of SK = 256 or 128 hidden
//    elements at a time.  Its accumulators (8 blocks x NR row blocks x 4 registers) stay in
//    registers across all slabs, and the logits leave straight from them: no exchange between
//    waves except four (max, sum) pairs per row at the very end.  (A first version split the
//    hidden dimension over the waves and met in LDS; its accumulators then limited a workgroup to
//    512 / NR vocabulary rows and the grid to NR times as many short-lived workgroups, each ending
//    in that exchange: 456 us at 72 rows where this one takes 202 us, and no faster at 9 rows.)
//  * W travels HBM -> LDS directly (global_load_lds_dwordx4, 1 KiB per instruction) in tiles of
//    16 rows x SK (8 KiB / 4 KiB) through a 32 KiB ring per wave, three / seven tiles ahead of the
//    math; the wave counts its own outstanding loads, so the main loop has no workgroup barrier.
//  * Where rows of W are a multiple of 4 KiB, but no power of two from 16 KiB on, a 256-wide slab is two runs of 256 bytes of a row, 2 KiB apart
//    (Slabs below).  All waves of the chip run through the hidden dimension nearly in step, so with contiguous slabs they ask for the same 512
//    of every 4 KiB at a time, which is half of the memory channels (bit 11 of the address is one of the bits that select them; the upper
//    bits make up for it in some placements of W and not in others, and at pitches of 16 and 32 KiB by themselves).  Means over placements of W, contiguous ->
//    two runs: 9 rows of 2048 x 128256 98 -> 82 us, 6144 x 64000 148 -> 122, 10240 x 32000 127 -> 99, 14336 x 50000 233 -> 227, 24576 x 16000 136 -> 122; 12288 x
//    50000 195 -> 194; 32768 x 16000 166 -> 163; 4096 x 128256 160 -> 161, 164 -> 163 and 184 -> 164 in three runs (154 to 194 by placement -> 155 to 170), one row 166 -> 162, 72
//    rows 200 -> 180, 9 of 4096 x 152064 200 -> 195, but of 4096 x 12000 18.2 -> 18.8; 8192 x 80000 201 -> 203, 8192 x 32000 88 -> 93, 16384 x 16000 87 -> 102,
//    16384 x 32000 160 -> 177, and a first pass right after a kernel that wrote W 219 -> 246 and 181 -> 219 at these two pitches (4096 x 128256: 196 -> 204 with
//    9 rows, 243 -> 223 with 72).  The order of the sum is the same for every logit.
//  * Up to three row blocks of h: the matching slab of h (NR tiles of 16 rows; rows past the last real one repeat it) comes
//    through the same ring at the head of every slab (from cache: every wave of every workgroup
//    reads the same h) and is then held in registers as the B operand of
//    v_mfma_f32_16x16x32_bf16 for the W tiles that follow.  From four row blocks on that would be a third of all
//    tiles, all out of one or two channels of the L2: there the workgroup shares a slab of h (lm_head_shared).
//  * A 16-byte-chunk XOR swizzle applied by the load addressing makes the operand reads
//    (ds_read_b128, 16 rows of 512 / 256 B) bank-conflict free without padding.
//  * Epilogue: fp32 logits from the accumulators (16-byte stores where the row stride allows);
//    per row the wave's own (max, sum exp) over its blocks, combined over the four waves by the
//    first threads of the workgroup.
#include "rapid_internal.h"

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

namespace {

constexpr int kWaves = 4;
constexpr int kNB = 32;                      // 16-row vocabulary blocks per workgroup
constexpr int kRing = 32768;                 // LDS ring per wave
// Tile geometry for a slab width of SK hidden elements (256, or 128 for hidden sizes
// that are a multiple of 128 but not of 256).
template <int SK>
struct Tile {
    static constexpr int BYTES = 16 * SK * 2;          // 8 KiB / 4 KiB
    static constexpr int NLD = BYTES / 1024;           // 1 KiB load instructions per tile
    static constexpr int RPI = 1024 / (SK * 2);        // rows moved by one instruction
    static constexpr int CPR = SK * 2 / 16;            // 16-byte chunks per row
    static constexpr int KS = SK / 32;                 // MFMA k-steps per tile
    static constexpr int SLOTS = kRing / BYTES;        // 4 / 8
    static constexpr int AHEAD = SLOTS - 1;            // tiles requested ahead of the math
};
constexpr float kLog2e = 1.4426950408889634f;

// Where the slabs of a row lie.  128-wide slabs: one run of 256 bytes.  256-wide ones: two, the second kHalf bytes behind the first: in
// rows that are a multiple of 4 KiB (TWO), the runs of eight slabs fill either half of 4 KiB in turn; else they adjoin (a pitch that is no
// multiple of 4 KiB spreads the rows of a tile by itself, and whole lines of 512 bytes are 1 % faster: 9 rows of 3072 x 128256
// 118.4 us against 120.1, 5 of 2304 x 100000 69.9 against 71.1; for powers of two see above).  A template parameter: told apart
// at every load it made heads of a few thousand entries 3 to 10 % slower.
template <int SK, bool TWO>
struct Slabs {
    static_assert(SK == 256 || !TWO, "");
    static constexpr uint32_t kHalf = TWO ? 2048u : 256u;
    static __device__ __forceinline__ int64_t byte(int s) { return TWO ? (int64_t)(s >> 3) * 4096 + (s & 7) * 256 : (int64_t)s * SK * 2; }
};

__device__ __forceinline__ void dma16(const char* base, uint32_t byte_off, uint32_t lds_addr)
{
    asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dwordx4 %0, %1 nt"
                 :
                 : "v"(byte_off), "s"(base), "s"(lds_addr)
                 : "memory", "m0");
}
// h is re-read by every workgroup: no streaming hint, it should stay in cache
__device__ __forceinline__ void dma16_keep(const char* base, uint32_t byte_off, uint32_t lds_addr)
{
    asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dwordx4 %0, %1"
                 :
                 : "v"(byte_off), "s"(base), "s"(lds_addr)
                 : "memory", "m0");
}
template <int N>
__device__ __forceinline__ void wait_loads()
{
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
__device__ __forceinline__ void lds_reads_done() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

constexpr int kNBW = kNB / kWaves;                      // vocabulary blocks per wave at most
constexpr int lds_bytes() { return kWaves * kRing + kWaves * 96 * 2 * 4; }   // rings + (max, sum) of 96 rows per wave

// First vocabulary row of a block as loaded: a block that reaches past the vocabulary reads the last 16 rows instead (the
// epilogue drops the rows that belong to the block before).
__device__ __forceinline__ int loaded_row0(const LmHeadLaunch& a, int nominal) { return min(nominal, a.vocab - 16); }

// acc[jj][rb]: lane (ln, lg) holds, for row rb*16 + ln of h, the four vocabulary
// entries loaded_row0 + lg*4 .. +3 of block jj.  Logits go out from the registers; the chunk statistics
// are formed per wave (own maximum) and combined over the four waves by the first threads; red: [kWaves][NR * 16][2].
template <int NR>
__device__ __forceinline__ void epilogue(const LmHeadLaunch& a, const floatx4 (&acc)[kNBW][NR], int nbw, int v0, float* red)
{
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ln = lane & 15, lg = lane >> 4;
    const float c = a.inv_T * kLog2e;
    const bool vec_ok = (a.ldz & 3) == 0 && (reinterpret_cast<uintptr_t>(a.logits) & 15) == 0;
#pragma unroll
    for (int rb = 0; rb < NR; ++rb) {
        const int hrow = rb * 16 + ln;
        const bool row_ok = hrow < a.n_rows;
        float m = -INFINITY;
#pragma unroll
        for (int jj = 0; jj < kNBW; ++jj) {
            const int nominal = v0 + (jj * kWaves + wave) * 16;
            if (jj < nbw && nominal < a.vocab && row_ok) {
                const int vi = loaded_row0(a, nominal) + lg * 4;
                float* dst = a.logits + (int64_t)hrow * a.ldz + vi;
                if (vec_ok && vi >= nominal && (vi & 3) == 0) {
                    *reinterpret_cast<floatx4*>(dst) = acc[jj][rb];
#pragma unroll
                    for (int i = 0; i < 4; ++i) m = fmaxf(m, acc[jj][rb][i]);
                } else {
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if (vi + i >= nominal) { dst[i] = acc[jj][rb][i]; m = fmaxf(m, acc[jj][rb][i]); }
                }
            }
        }
        if (!a.stats) continue;                                // uniform
        m = fmaxf(m, __shfl_xor(m, 16));
        m = fmaxf(m, __shfl_xor(m, 32));
        float sum = 0.f;
        if (m > -INFINITY) {
#pragma unroll
            for (int jj = 0; jj < kNBW; ++jj) {
                const int nominal = v0 + (jj * kWaves + wave) * 16;
                if (jj < nbw && nominal < a.vocab && row_ok) {
                    const int vi = loaded_row0(a, nominal) + lg * 4;
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if (vi + i >= nominal) sum += __builtin_amdgcn_exp2f((acc[jj][rb][i] - m) * c);
                }
            }
        }
        sum += __shfl_xor(sum, 16);
        sum += __shfl_xor(sum, 32);
        if (lg == 0) {
            red[((wave * NR * 16) + hrow) * 2 + 0] = m;
            red[((wave * NR * 16) + hrow) * 2 + 1] = sum;
        }
    }
    if (!a.stats) return;
    __syncthreads();
    if (tid < a.n_rows) {
        float M = -INFINITY;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) M = fmaxf(M, red[((w * NR * 16) + tid) * 2]);
        float S = 0.f;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            const float mw = red[((w * NR * 16) + tid) * 2], sw = red[((w * NR * 16) + tid) * 2 + 1];
            if (sw > 0.f) S += sw * __builtin_amdgcn_exp2f((mw - M) * c);
        }
        a.stats[((int64_t)tid * gridDim.x + blockIdx.x) * 2 + 0] = M;
        a.stats[((int64_t)tid * gridDim.x + blockIdx.x) * 2 + 1] = S;
    }
}

template <int SK, int NR, bool TWO>
__global__ void __launch_bounds__(kWaves * 64) lm_head_stream(LmHeadLaunch a)
{
    using T = Tile<SK>;
    using At = Slabs<SK, TWO>;
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ln = lane & 15, lg = lane >> 4;
    const int nb = a.nb;                                 // 16-row vocabulary blocks per workgroup (<= 32)
    const int nbw = (nb + kWaves - 1 - wave) / kWaves;   // blocks of this wave: wave, wave + 4, ...
    const int v0 = blockIdx.x * nb * 16;
    const uint32_t row_bytes = (uint32_t)a.hidden * 2u;
    const int nslab = a.hidden / SK;
    char* ring = smem + wave * kRing;
    const uint32_t ring_lds = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)smem + wave * kRing;

    // Per-lane byte offsets of the loads of a tile, relative to the tile's first row and the slab:
    // instruction e moves RPI consecutive rows; lane i writes LDS bytes [16 i, 16 i + 16) of that
    // 1 KiB and fetches the chunk the swizzle assigns there (chunks 16..31: the slab's second run).
    uint32_t woff[T::NLD], coff[T::NLD];
    int rrow[T::NLD];
#pragma unroll
    for (int e = 0; e < T::NLD; ++e) {
        rrow[e] = T::RPI * e + lane / T::CPR;
        coff[e] = (uint32_t)((lane % 16) ^ (rrow[e] & 15)) * 16u + (uint32_t)((lane % T::CPR) / 16) * At::kHalf;
        woff[e] = (uint32_t)rrow[e] * row_bytes + coff[e];
    }
    auto block_row0 = [&](int jj) { return loaded_row0(a, v0 + (jj * kWaves + wave) * 16); };

    // tile j of slab s: j = 0..NR-1 the row blocks of the h slab, j = NR.. the wave's W blocks
    auto issue = [&](int s, int j, int slot) {
        const int64_t kbyte = At::byte(s);
        const uint32_t dst = ring_lds + slot * T::BYTES;
        if (j < NR) {
            const char* base = reinterpret_cast<const char*>(a.h) + kbyte;
#pragma unroll
            for (int e = 0; e < T::NLD; ++e)
                dma16_keep(base, (uint32_t)min(j * 16 + rrow[e], a.n_rows - 1) * row_bytes + coff[e], dst + e * 1024);
            return;
        }
        const char* base = reinterpret_cast<const char*>(a.w) + (int64_t)block_row0(j - NR) * row_bytes + kbyte;
#pragma unroll
        for (int e = 0; e < T::NLD; ++e) dma16(base, woff[e], dst + e * 1024);
    };

    floatx4 acc[kNBW][NR];
#pragma unroll
    for (int j = 0; j < kNBW; ++j)
#pragma unroll
        for (int rb = 0; rb < NR; ++rb) acc[j][rb] = floatx4{0.f, 0.f, 0.f, 0.f};

    if (nbw > 0) {                                       // (a wave without blocks: ranges of fewer than four blocks)
        int ps = 0, pj = 0, pt = 0;                      // next tile to request: slab, index, linear number
        auto request_next = [&]() {
            const int sl = pt & (T::SLOTS - 1);
            if (ps < nslab) issue(ps, pj, sl);
            else issue(nslab - 1, 0, sl);                // past the end: a cached h tile keeps the count uniform
            ++pt;
            if (++pj >= NR + nbw) { pj = 0; ++ps; }
        };
#pragma unroll
        for (int j = 0; j < T::AHEAD; ++j) request_next();

        bf16x8 hreg[NR][T::KS];
        const int rd_row = ln * (SK * 2);
        const int rd_swz = ln & 15;
        int t = 0;
        for (int s = 0; s < nslab; ++s) {
#pragma unroll
            for (int j = 0; j < NR + kNBW; ++j) {
                if (j < NR + nbw) {
                    wait_loads<(T::AHEAD - 1) * T::NLD>();     // tile (s, j) has landed
                    request_next();
                    const char* tile = ring + (t & (T::SLOTS - 1)) * T::BYTES;
                    ++t;
                    if (j < NR) {
#pragma unroll
                        for (int ks = 0; ks < T::KS; ++ks)
                            hreg[j < NR ? j : 0][ks] = *reinterpret_cast<const bf16x8*>(tile + rd_row + (((ks * 4 + lg) ^ rd_swz) * 16));
                    } else {
#pragma unroll
                        for (int ks = 0; ks < T::KS; ++ks) {
                            bf16x8 wa = *reinterpret_cast<const bf16x8*>(tile + rd_row + (((ks * 4 + lg) ^ rd_swz) * 16));
#pragma unroll
                            for (int rb = 0; rb < NR; ++rb)
                                acc[j >= NR ? j - NR : 0][rb] =
                                    __builtin_amdgcn_mfma_f32_16x16x32_bf16(wa, hreg[rb][ks], acc[j >= NR ? j - NR : 0][rb], 0, 0, 0);
                        }
                    }
                    lds_reads_done();
                }
            }
        }
        wait_loads<0>();
    }

    epilogue<NR>(a, acc, nbw, v0, reinterpret_cast<float*>(smem + kWaves * kRing));
}

// ---------------------------------------------------------------- many rows: one copy of h per workgroup
// From four row blocks on.  The four waves load a slab of h together (256-wide, NR tiles) and all read it into their registers; two
// barriers a slab, eight tiles of W apart, and the loads of the next slab of h go out right behind them.  What the
// LDS has left is the rings of W, in units of half a tile (one of the slab's two runs: 16 rows x 256 bytes), five or six units
// ahead of the math.  Against h through every wave's own ring: 72 rows of 4096 x 128256 179 -> 171 us, 96 rows 190 -> 175, 72
// rows of 2048 x 128256 100 -> 95; 60 rows 171 -> 168; 40 rows 162 -> 164, so three row blocks stay there.  Two or four
// passes over the hidden dimension, so that the logits of the first leave under the loads of the second: 184 and 224 us.
template <int NR>
struct Shared {
    static constexpr int HBYTES = NR * 16 * 512;                              // a slab of h
    static constexpr int RED = kWaves * NR * 16 * 2 * 4;
    static constexpr int UNIT = 16 * 256;                                     // half a tile of W
    static constexpr int ULD = UNIT / 1024;                                   // loads per unit
    static constexpr int HLD = NR * 8 / kWaves;                               // loads of a wave per slab of h
    static constexpr int SLOTS = (160 * 1024 - HBYTES - RED) / kWaves / UNIT;
    static constexpr int AHEAD = SLOTS - 1;
    static constexpr int LDS = HBYTES + RED + kWaves * SLOTS * UNIT;
};

template <int NR, bool TWO>
__global__ void __launch_bounds__(kWaves * 64) lm_head_shared(LmHeadLaunch a)
{
    using S = Shared<NR>;
    using At = Slabs<256, TWO>;
    constexpr int KH = 4;                                // k-steps of a unit
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ln = lane & 15, lg = lane >> 4;
    const int nb = a.nb;                                 // 16-row vocabulary blocks per workgroup (<= 32)
    const int nbw = (nb + kWaves - 1 - wave) / kWaves;   // blocks of this wave: wave, wave + 4, ...
    const int v0 = blockIdx.x * nb * 16;
    const uint32_t row_bytes = (uint32_t)a.hidden * 2u;
    const int nslab = a.hidden / 256;
    char* hbuf = smem;
    char* ring = smem + S::HBYTES + wave * (S::SLOTS * S::UNIT);
    const uint32_t h_lds = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)smem;
    const uint32_t ring_lds = h_lds + S::HBYTES + wave * (S::SLOTS * S::UNIT);

    // Loads of a unit: instruction e moves rows 4 e .. 4 e + 3; the swizzle as above, within 16 chunks.
    uint32_t woff[S::ULD];
#pragma unroll
    for (int e = 0; e < S::ULD; ++e) {
        const int row = 4 * e + lane / 16;
        woff[e] = (uint32_t)row * row_bytes + (uint32_t)((lane & 15) ^ (row & 15)) * 16u;
    }
    // This wave's share of slab s of h: 1 KiB (two rows) of every 4.
    auto issue_h = [&](int s) {
        const char* base = reinterpret_cast<const char*>(a.h) + At::byte(s);
#pragma unroll
        for (int i = 0; i < S::HLD; ++i) {
            const int e = i * kWaves + wave, row = 2 * e + lane / 32;
            const uint32_t c = (uint32_t)((lane & 15) ^ (row & 15)) * 16u + (uint32_t)((lane & 31) / 16) * At::kHalf;
            dma16_keep(base, (uint32_t)min(row, a.n_rows - 1) * row_bytes + c, h_lds + e * 1024);
        }
    };
    // The next unit to request: half pq of slab ps of block pj; past the end any valid one keeps the count uniform.
    int ps = 0, pj = 0, pq = 0, pslot = 0;
    auto request_next = [&]() {
        const char* base = reinterpret_cast<const char*>(a.w) +
                           (int64_t)loaded_row0(a, v0 + (pj * kWaves + wave) * 16) * row_bytes + At::byte(min(ps, nslab - 1)) + (pq ? At::kHalf : 0u);
#pragma unroll
        for (int e = 0; e < S::ULD; ++e) dma16(base, woff[e], ring_lds + pslot * S::UNIT + e * 1024);
        if (++pslot == S::SLOTS) pslot = 0;
        pq ^= 1;
        if (pq == 0 && ++pj >= nbw) { pj = 0; ++ps; }
    };

    floatx4 acc[kNBW][NR];
#pragma unroll
    for (int j = 0; j < kNBW; ++j)
#pragma unroll
        for (int rb = 0; rb < NR; ++rb) acc[j][rb] = floatx4{0.f, 0.f, 0.f, 0.f};

    // (a wave without blocks, in ranges of fewer than four, only loads its share of h and meets the barriers)
    issue_h(0);
    if (nbw > 0)
#pragma unroll
        for (int j = 0; j < S::AHEAD; ++j) request_next();
    int slot = 0;
    for (int s = 0; s < nslab; ++s) {
        // The own share of h has landed: AHEAD units at least were requested after it, unless the wave has too few blocks.
        if (s == 0 ? nbw > 0 : 2 * nbw >= S::AHEAD) wait_loads<S::AHEAD * S::ULD>();
        else wait_loads<0>();
        __syncthreads();                                 // everybody's has
        bf16x8 hreg[NR][2 * KH];
#pragma unroll
        for (int rb = 0; rb < NR; ++rb)
#pragma unroll
            for (int ks = 0; ks < 2 * KH; ++ks)
                hreg[rb][ks] = *reinterpret_cast<const bf16x8*>(hbuf + rb * 8192 + ln * 512 + (((ks * 4 + lg) ^ ln) * 16));
        lds_reads_done();
        __syncthreads();                                 // everybody has read it
        issue_h(min(s + 1, nslab - 1));                  // (the last one again: the count stays uniform)
#pragma unroll
        for (int j = 0; j < kNBW; ++j)
            if (j < nbw) {
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    // the slab's first AHEAD units were requested before the loads of h just issued, so those are behind them too
                    if (2 * j + q < S::AHEAD) wait_loads<(S::AHEAD - 1) * S::ULD + S::HLD>();
                    else wait_loads<(S::AHEAD - 1) * S::ULD>();
                    request_next();
                    const char* unit = ring + slot * S::UNIT;
                    if (++slot == S::SLOTS) slot = 0;
#pragma unroll
                    for (int ks = 0; ks < KH; ++ks) {
                        const bf16x8 wa = *reinterpret_cast<const bf16x8*>(unit + ln * 256 + (((ks * 4 + lg) ^ ln) * 16));
#pragma unroll
                        for (int rb = 0; rb < NR; ++rb)
                            acc[j][rb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wa, hreg[rb][q * KH + ks], acc[j][rb], 0, 0, 0);
                    }
                    lds_reads_done();
                }
            }
    }
    wait_loads<0>();
    epilogue<NR>(a, acc, nbw, v0, reinterpret_cast<float*>(smem + S::HBYTES + kWaves * S::SLOTS * S::UNIT));
}

}  // namespace

namespace {
// Calls f(kernel, bytes of LDS) for a build: 128-wide slabs, 256-wide ones in adjoining or in two runs, and these with h shared.
enum Kind { kNarrow, kAdjoining, kTwoRuns, kSharedAdjoining, kSharedTwoRuns };
template <int NR, class F>
hipError_t for_build(Kind kind, F f)
{
    if constexpr (NR >= 4) {
        if (kind == kSharedAdjoining) return f(lm_head_shared<NR, false>, Shared<NR>::LDS);
        if (kind == kSharedTwoRuns) return f(lm_head_shared<NR, true>, Shared<NR>::LDS);
    } else {
        if (kind == kTwoRuns) return f(lm_head_stream<256, NR, true>, lds_bytes());
    }
    if (kind == kNarrow) return f(lm_head_stream<128, NR, false>, lds_bytes());
    return f(lm_head_stream<256, NR, false>, lds_bytes());
}
// The 256-wide slab when the hidden size allows, else the 128-wide one; from four row blocks on the workgroup shares h, except at pitches that are
// a power of two from 16 KiB on where a wave has at least as many blocks of W as there are row blocks.  There its half tiles (256 bytes of a row at
// a time) cost more than the copies of h: 8192 x 128256 with 52, 72, 96 rows 326, 332, 346 us through the rings, 347, 348, 371 shared; x 64000 (four
// blocks a wave) 169, 180, 199 and 179, 181, 188; x 50257 (three) 154, 168, 191 and 152, 142, 148; 16384 x 64000 323, 345, 383 and 343, 348, 356.
Kind kind_of(const LmHeadLaunch& a, int nr)
{
    if (a.hidden % 256 != 0) return kNarrow;
    const bool large_power = a.hidden >= 8192 && (a.hidden & (a.hidden - 1)) == 0;
    const bool two_runs = a.hidden % 2048 == 0 && !large_power;
    if (nr >= 4 && (!large_power || a.nb < kWaves * nr)) return two_runs ? kSharedTwoRuns : kSharedAdjoining;
    return two_runs ? kTwoRuns : kAdjoining;
}
template <int NR>
hipError_t configure_rows()
{
    for (Kind kind : {kNarrow, kAdjoining, kTwoRuns, kSharedAdjoining, kSharedTwoRuns}) {
        const hipError_t e = for_build<NR>(kind, [](auto kernel, int lds) {
            return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        });
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}
template <int NR>
hipError_t launch_rows(const LmHeadLaunch& a, hipStream_t stream)
{
    const int nwg = (a.vocab + a.nb * 16 - 1) / (a.nb * 16);
    return for_build<NR>(kind_of(a, NR), [&](auto kernel, int lds) {
        hipLaunchKernelGGL(kernel, dim3(nwg), dim3(kWaves * 64), lds, stream, a);
        return hipGetLastError();
    });
}
}  // namespace

hipError_t configure_lm_head()
{
    hipError_t e;
    if ((e = configure_rows<1>()) != hipSuccess) return e;
    if ((e = configure_rows<2>()) != hipSuccess) return e;
    if ((e = configure_rows<3>()) != hipSuccess) return e;
    if ((e = configure_rows<4>()) != hipSuccess) return e;
    if ((e = configure_rows<5>()) != hipSuccess) return e;
    return configure_rows<6>();
}

hipError_t launch_lm_head(const LmHeadLaunch& a, hipStream_t stream)
{
    const int nr = (a.n_rows + 15) / 16;                 // row blocks of 16 rows of h
    if (a.hidden % 128 != 0 || a.nb < 1 || a.nb > kNB) return hipErrorInvalidValue;
    switch (nr) {
        case 1: return launch_rows<1>(a, stream);
        case 2: return launch_rows<2>(a, stream);
        case 3: return launch_rows<3>(a, stream);
        case 4: return launch_rows<4>(a, stream);
        case 5: return launch_rows<5>(a, stream);
        case 6: return launch_rows<6>(a, stream);
    }
    return hipErrorInvalidValue;
}
