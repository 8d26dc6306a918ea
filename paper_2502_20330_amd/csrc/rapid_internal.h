// Internal declarations shared by the translation units of librapid.so.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include "rapid.h"

struct rapid_ctx {
    int device;
    int n_cu;
    int last_hip_error;
    void* static_scratch;   // device address of this GPU's copy of the library's static scratch array
    int64_t accept_wait_ticks;   // bound of every inter-workgroup wait of the accept pass, 10 ns ticks
    int64_t attn_wait_ticks;     // the same of the attention call's exchange
    int accept_slice;            // entries per workgroup of the accept row pass (0 = automatic)
    int probe_skew;              // streaming probe: 32nds of the mean share moved from odd to even workgroups
};

// ---- verify attention (verify_attn.hip)
struct AttnExchangeHead;
struct AttnLaunch {
    const uint16_t* q;
    const uint16_t* k;
    const uint16_t* v;
    const int32_t* ctx_lens;
    const int32_t* gammas;
    const int32_t* page_table;
    uint16_t* out;
    float* lse_out;
    float* part_o;      // [B, Hkv, nsplit, RB*16, D] fp32, relative to the maximum in part_ml; balanced shares:
                        // [Hkv, nslots, RB*16, D], slot g + b for group g's piece of sequence b
    float* part_ml;     // the same slots, [.., RB*16, 2] (running max in log2 units, sum)
    int32_t B, Qmax, Hq, Hkv, G, D, gamma;
    int32_t max_ctx;    // host bound of ctx_lens
    int32_t chunk, nsplit, RB;   // RB: 16-row blocks of the partials (wide: two teams of (RB + 1) / 2 and RB / 2 blocks)
    int32_t wide;       // 1: eight-wave kernel with two row teams (from five row blocks on)
    int32_t rot;        // 1: dispatch slot x serves head (x + split) mod Hkv, 0: head x
    int32_t groups;     // > 0: balanced shares of a ragged batch, one workgroup per (kv head, group); even
    int32_t nslots;     // balanced shares: partial slots per kv head (groups + B - 1)
    int32_t skew;       // tokens moved from the splits on odd dispatch slots to those on even ones
                        // (balanced shares: 32nds of the mean share)
    int64_t bstride, tstride, hstride, pstride;   // elements
    int32_t page_shift, page_mask, max_pages;     // page_shift < 0: contiguous
    int32_t page_hi;    // largest page id the kernels will use (ids are clamped to [0, page_hi])
    float scale_log2e;
    // one launch: the workgroups exchange their partials and merge them themselves (null: a second kernel merges)
    AttnExchangeHead* xhead;
    void* xwords;            // tagged words: partials [B, Hkv, nsplit, RB*16, D], behind them (max, sum) of the rows
    uint32_t xbytes;         // of the words
    uint32_t xml_offset;     // bytes from xwords to the (max, sum) words
    int64_t xwait_ticks;     // bound of a wait in wall-clock ticks (100 MHz)
};
constexpr int kAttnTeams = 256;  // largest grid that merges by itself
// Row counts (in blocks of 16) for which the workgroups merge their partials themselves, up to 16 rows of 128 or 32 of 64.  In graphs
// of calls, two launches against one: 4 rows of 128, 500 tokens 8.30 and 7.90 us, 16 rows, 4000 tokens 9.73 and 9.28; 32 rows of 64, 4000 tokens 8.50 and 8.20.  Beyond, the words (twice the
// partials) take longer to go through memory and back than a second launch: 20 rows of 128, 8K tokens 14.3 and 14.7, 36 rows 17.0
// and 18.3, 72 rows 20.2 and 23.0; 40 rows of 64, 2K tokens 8.6 and 9.2.  Calls that the host cannot enqueue as fast as they run gain a launch.
constexpr bool attn_in_one_launch(int row_blocks, int D) { return row_blocks * D <= 128; }
constexpr int kMaxShares = 32;   // workgroups of a (sequence, kv head) that merge rows
// Head of the exchange memory of the attention call (attn_exchange.h).
struct AttnExchangeHead {
    uint32_t calls[kAttnTeams];                  // calls so far, a copy per (sequence, kv head)
    uint32_t marks[kAttnTeams][kMaxShares];      // number of the last call that left this share to others
};
constexpr size_t kAttnExchangeHeadBytes = (sizeof(AttnExchangeHead) + 255) / 256 * 256;
size_t attn_exchange_bytes(int B, int Hkv, int nsplit, int RB, int D);
hipError_t launch_verify_attn(const AttnLaunch& a, hipStream_t stream);
hipError_t configure_verify_attn();   // per device, before the first launch
size_t attn_workspace_bytes(int B, int Hkv, int nsplit, int RB, int D);

// ---- accept pass (accept.hip)
struct AcceptLaunch {
    const float* zt;
    const float* zd;
    const int32_t* tokens;
    const int32_t* gammas;
    const float* uniforms;
    int32_t* n_accepted;
    int32_t* out_tokens;
    float* ratio;
    void* workspace;
    int32_t B, gmax, V;
    float eta, inv_T, tail_alpha;
    double inv_T_exact;   // 1 / (double)temperature
    // row statistics computed elsewhere (the output head's epilogue), or null:
    // (max z, sum exp((z - max)/T)) per chunk, [B*(gmax+1)][nch_t] and [B*gmax][nch_d] pairs
    const float* ext_t;
    const float* ext_d;
    int32_t nch_t, nch_d;
    int64_t wait_ticks;   // bound of an exchange wait in wall-clock ticks (100 MHz); 0 = publish nothing, compute every slice
    int32_t n_cu;         // compute units of the device (sizes the slices)
    int32_t fill_ratio;   // 1: ratios of positions past a sequence's drafts are written as 0, else left alone
    int32_t force_slice;  // 4096 / 8192 / 10240 / 16384 entries per slice; 0 = automatic
};
hipError_t launch_accept(const AcceptLaunch& a, hipStream_t stream);
size_t accept_workspace_bytes(int B, int gmax, int V);
// the greedy limit T -> 0 (accept_greedy.hip); uses zt, zd, tokens, gammas, uniforms, outputs, workspace
hipError_t launch_accept_greedy(const AcceptLaunch& a, hipStream_t stream);
size_t accept_greedy_workspace_bytes(int B, int gmax, int V);

// ---- streaming-read probe (hbm_probe.hip)
hipError_t configure_hbm_read_probe();
hipError_t launch_hbm_read_probe(const rapid_ctx* ctx, const void* buf, size_t bytes, uint32_t* sink, hipStream_t stream);

// ---- output head (lm_head.hip)
struct LmHeadLaunch {
    const uint16_t* h;      // [n_rows][hidden] bf16
    const uint16_t* w;      // [vocab][hidden] bf16
    float* logits;          // [n_rows][ldz]
    float* stats;           // [n_rows][ceil(vocab / (16 nb))][2] or null
    int32_t n_rows, hidden, vocab;
    int32_t nb;             // 16-row vocabulary blocks per workgroup, 1..32 (statistics chunk = 16 nb)
    int64_t ldz;
    float inv_T;
};
hipError_t launch_lm_head(const LmHeadLaunch& a, hipStream_t stream);
hipError_t configure_lm_head();

// ---- cache bookkeeping (kv_cache.hip)
struct KvAppendLaunch {
    const uint16_t* k_new;      // [B][Qmax][Hkv][D]
    const uint16_t* v_new;
    const int32_t* ctx_lens;
    const int32_t* gammas;
    const int32_t* page_table;
    uint16_t* k_cache;
    uint16_t* v_cache;
    int32_t B, Qmax, Hkv, D, gamma;
    int32_t max_ctx;
    int64_t bstride, tstride, hstride, pstride;   // elements
    int32_t page_shift, page_mask, max_pages;     // page_shift < 0: contiguous
    int32_t page_hi;            // page ids are clamped to [0, page_hi]
};
struct KvCommitPagesLaunch {
    const int32_t* gammas;
    const int32_t* n_accepted;
    const int32_t* page_table;
    int32_t* ctx_lens;
    int32_t* released;          // [B][cap]
    int32_t* n_released;        // [B]
    int32_t B, Qmax, gamma, max_ctx, page_shift, max_pages, cap, page_hi;
};
hipError_t launch_kv_commit_pages(const KvCommitPagesLaunch& a, hipStream_t stream);
hipError_t launch_kv_append(const KvAppendLaunch& a, hipStream_t stream);
hipError_t launch_kv_commit(int B, int gamma, const int32_t* gammas, const int32_t* n_accepted, int32_t* ctx_lens,
                            hipStream_t stream);

// ---- retrieval chunk selection (retrieve.hip)
struct RetrieveLaunch {
    const float* emb;       // [n][dim]
    const float* query;     // [dim]
    float* sim;             // [n]
    int32_t* selected;      // [top_k], unused tail = -1
    int32_t* n_selected;    // [1]
    int32_t n, dim, top_k;
    float threshold;
};
hipError_t launch_retrieve(const RetrieveLaunch& a, hipStream_t stream);
