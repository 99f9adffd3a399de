// C ABI of libcard: argument checks and the launch sequence of one verification step.
#include <algorithm>
#include <atomic>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <hip/hip_runtime.h>

#include <vector>

#include "card.h"

#ifndef CARD_STATIC_SCRATCH_BYTES
#define CARD_STATIC_SCRATCH_BYTES (32u << 20)
#endif
#include "card_pack.hip"
#include "card_verify.hip"
#include "card_prompt.hip"
#include "card_level.hip"

using namespace card;

namespace {

inline hipStream_t as_stream(void* s) { return reinterpret_cast<hipStream_t>(s); }

inline int launch_status() { return hipGetLastError() == hipSuccess ? CARD_OK : CARD_EDEVICE; }

unsigned long long* g_ts_buf = nullptr;
int g_ts_layer = 0;

// Benchmark hook: event pairs around the verify kernel.  One user at a time (the lock only keeps
// enable / disable / collect and a concurrent card_verify from tearing the vectors).  The events
// are destroyed by card_profile_disable, never by a static destructor: at process exit the HIP
// runtime may already be gone.
struct Profile {
    std::mutex mu;
    std::atomic<bool> on{false};
    int used = 0;
    std::vector<hipEvent_t> start, stop;
};
Profile& prof() {
    static Profile* p = new Profile;  // leaked on purpose: no destructor runs after HIP teardown
    return *p;
}

struct ProfScope {
    hipStream_t st;
    hipEvent_t stop = nullptr;
    explicit ProfScope(hipStream_t s) : st(s) {
        Profile& p = prof();
        if (!p.on) return;
        std::lock_guard<std::mutex> g(p.mu);
        if (p.on && p.used < int(p.start.size())) {
            const int idx = p.used++;
            (void)hipEventRecord(p.start[idx], st);
            stop = p.stop[idx];
        }
    }
    ~ProfScope() {
        if (stop) (void)hipEventRecord(stop, st);
    }
};

constexpr int kMaxDevices = 64;

// Compute units of the current device (cached per device id).
int cu_count() {
    static std::atomic<int> cus[kMaxDevices];
    int dev = 0, n = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return 0;
    n = cus[dev].load(std::memory_order_relaxed);
    if (n == 0) {
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
        cus[dev].store(n, std::memory_order_relaxed);
    }
    return n;
}

// Workgroups of the verify kernel: cfg->grid_wgs if the caller fixed it, else one per compute
// unit; at most 256 (the barrier polls 256 flags), never more than the compute units there are
// (every workgroup needs a compute unit of its own: the grid meets at barriers).
int grid_size(const card_model_cfg* cfg) {
    const int cus = cu_count();
    int n = cus > 256 ? 256 : cus;
    if (cfg && cfg_grid(cfg) > 0) {
        if (cfg_grid(cfg) > n) return 0;
        n = cfg_grid(cfg);
    }
    return n;
}

// The kernel synchronises its workgroups through flags in memory, so all of them have to be
// resident at once.  It is launched as an ordinary kernel: one workgroup fills a compute unit
// (158.6 of its 160 KiB of LDS, 512 threads with 256 registers each), the grid is no larger than the
// number of compute units, and the occupancy query below confirms that the device can hold a
// workgroup per compute unit, so on an otherwise idle device the dispatcher places all of them.
// Should other work hold compute units for longer than the kernel's bounded waits, the step ends
// with accepted_len = -1 instead of hanging.
template <int MT, int H, bool PK, bool DR, bool PC, bool CODED>
int launch_kernel(MegaArgs& a, hipStream_t st) {
    static std::atomic<int> fits[kMaxDevices];  // 0 unknown, 1 yes, -1 no
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return CARD_EDEVICE;
    int f = fits[dev].load(std::memory_order_relaxed);
    if (f == 0) {
        int per_cu = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_verify<MT, H, PK, DR, PC, CODED>, kBlockThreads, 0) != hipSuccess)
            return CARD_EDEVICE;
        f = per_cu >= 1 ? 1 : -1;
        fits[dev].store(f, std::memory_order_relaxed);
    }
    if (f < 0 || a.nwg > cu_count()) return CARD_EDEVICE;
    hipLaunchKernelGGL((k_verify<MT, H, PK, DR, PC, CODED>), dim3(a.nwg), dim3(kBlockThreads), 0, st, a);
    return launch_status();
}
template <int MT, int H, bool PK, bool DR, bool PC = false>
int launch_mega(MegaArgs& a, hipStream_t st) {
    return a.cbase ? launch_kernel<MT, H, PK, DR, PC, true>(a, st) : launch_kernel<MT, H, PK, DR, PC, false>(a, st);
}

// Scratch of the entry point that allocates nothing: what card_verify takes as `workspace_dev`,
// at a fixed place in the code object.  In host code the name is a stand-in, not a device address:
// the address of this device's copy comes from hipGetSymbolAddress, once per device.
constexpr size_t kStaticWsBytes = size_t(CARD_STATIC_SCRATCH_BYTES);
static __device__ __align__(256) unsigned char scratch[kStaticWsBytes];

struct StaticWs {
    void* ptr = nullptr;       // device address of `scratch` on this device
    bool prepared = false;     // k_ws_init has been enqueued for `cfg`'s layout
    card_model_cfg cfg = {};
};
StaticWs g_static[kMaxDevices];
std::mutex g_static_mu;

// Draft-side options of a step (card_draft_level): tree rows and the per-row top-k.
struct TreeOpt {
    const int32_t* row_pos;
    int32_t first_slot;
    const uint32_t* mask;
    int32_t mask_words, mask_base;
    int32_t topk;
    int32_t* topk_tok;
    float* topk_prob;
    bool piece;  // one of several calls, perhaps at the same time, that forward the level in these slots
    int32_t level_first, level_end;
};

// one layer of a page pool is addressed with 32-bit byte offsets
bool pool_fits(const card_model_cfg* cfg, const card_kv* kv) {
    return size_t(kv->n_pages) * cfg->n_kv_heads * 16 * cfg->head_dim * 2 < (size_t(1) << 32);
}

// How attention cuts the list of pages of a step of r rows.  A workgroup's share fits the page buffers of its wavefronts (all of
// its old-context pages are then in flight before the barrier in front of attention), as long
// as every task still gets a workgroup of its own; beyond that the shares grow instead.
// The cut length is a function of the context length in steps of 512 tokens, the grid and
// the kernel (r <= 8, <= 16, <= 32), not of r itself: a row's keys are then cut, summed and
// merged in the same order whether a step of eight rows or a plain decode step computes it,
// and verification reproduces the plain decode's logits bit for bit (same kernel, same
// 512-token stretch).
void attn_cuts(const card_model_cfg* cfg, const Layout& L, int nwg, int r, int pages_used, int32_t& pages_per_cut, int32_t& cuts) {
    const int G = cfg->n_q_heads / cfg->n_kv_heads;
    const int share = kMegaWaves * (cfg->head_dim == 128 ? 2 : 4);
    const int r_kernel = r <= 8 ? 8 : (r <= 16 ? 16 : 32);
    const int max_cuts = std::min<int>(L.m_attn_max_splits, std::max(1, nwg / (cfg->n_kv_heads * ceil_div(G * r_kernel, 16))));
    const int pages_stretch = ceil_div(pages_used, 32) * 32;
    pages_per_cut = std::max(share, ceil_div(pages_stretch, max_cuts));
    cuts = ceil_div(pages_used, pages_per_cut);
}

// Workgroups of a step: all of the grid, or as many as have a tile of some matrix or an attention task.  A small model's step is a chain of
// grid-wide hand-overs, cheaper among fewer workgroups (2 layers of 256 columns, 88 instead of 256: 74.5 -> 67.2 us).
// The weights need no other layout: a matrix of at most n tiles lies in memory the same way for every grid of n positions and more.  Nor
// does any sum change its order: attention is cut for the grid, and multiples of eight (or none) keep the
// down-projection's groups; of head_dim / 8, the rotation factors in LDS.
int step_workgroups(const card_model_cfg* cfg, const Layout& L, int grid, int attn_tasks) {
    const int unit = cfg->head_dim / 8;
    if (grid % unit) return grid;
    const int busy = std::max({L.qkv.Nt, L.wo.Nt, L.gu.Nt, L.wd.Nt, L.lm.Nt, attn_tasks});
    return std::min(grid, ceil_div(busy, unit) * unit);
}

// One persistent kernel runs the whole step (card_verify.hip).
int verify_impl(const card_model_cfg* cfg, const void* packed, const card_kv* kv, int32_t ctx_len,
                const int32_t* cand, int32_t r, void* workspace, void* stream, card_verify_result* out,
                int32_t* row_argmax, float* logits, const card_sampling* sampling = nullptr,
                const TreeOpt* tree = nullptr) {
    if (!cfg || !packed || !kv || !cand || !workspace || (!out && !tree)) return CARD_EINVAL;
    const Layout L = make_layout(cfg);
    if (!L.ok) return CARD_EINVAL;
    if (!kv->k_pages || !kv->v_pages || !kv->block_table || kv->n_pages <= 0) return CARD_EINVAL;
    if (!pool_fits(cfg, kv)) return CARD_EINVAL;
    if (r < 1 || r > cfg->max_r) return CARD_ERANGE;
    if (ctx_len < 0) return CARD_EINVAL;
    const int32_t slot0 = tree ? tree->first_slot : ctx_len;
    if (int64_t(slot0) + r > cfg->max_ctx) return CARD_ECAPACITY;
    if (tree) {
        if (!tree->row_pos || !tree->mask || !tree->topk_tok || !tree->topk_prob) return CARD_EINVAL;
        if (tree->mask_words < 1 || tree->mask_words > 32 || tree->topk < 1 || tree->topk > 16) return CARD_ERANGE;
        if (tree->mask_base < 0 || tree->mask_base % kKvBlock || tree->mask_base > ctx_len) return CARD_EINVAL;
        if (slot0 < ctx_len || int64_t(slot0) + r > int64_t(tree->mask_base) + 32 * tree->mask_words) return CARD_ERANGE;
        if (tree->piece) {
            if (tree->level_first < ctx_len || tree->level_first > slot0 || tree->level_end < slot0 + r) return CARD_ERANGE;
            if (tree->level_end > cfg->max_ctx) return CARD_ECAPACITY;
        }
    }
    const int grid = grid_size(cfg);
    if (grid <= 0) return CARD_EDEVICE;

    char* ws = static_cast<char*>(workspace);
    const int h = cfg->head_dim;
    MegaArgs a = {};
    a.L = cfg->n_layers;
    a.d = cfg->d_model;
    a.qd = cfg->n_q_heads * h;
    a.kvd = cfg->n_kv_heads * h;
    a.h = h;
    a.Hkv = cfg->n_kv_heads;
    a.G = cfg->n_q_heads / cfg->n_kv_heads;
    a.F = cfg->d_ffn;
    a.V = cfg->vocab;
    a.r = r;
    a.rp = r;
    a.ctx_len = ctx_len;
    a.eps = cfg->rms_eps;
    a.inv_d = 1.0f / float(cfg->d_model);
    a.theta = cfg->rope_theta;
    a.inv_sqrt_h = 1.4426950408889634f / sqrtf(float(h));  // log2(e)/sqrt(h): the softmax runs on exp2
    a.wbase = static_cast<const char*>(packed);
    a.embed_off = L.embed_off;
    a.g_final_off = L.g_final_off;
    a.layer0_off = L.layer0_off;
    a.stamp = reinterpret_cast<const uint32_t*>(a.wbase + L.stamp_off);
    a.layer_stride = L.layer_stride;
    a.g_attn_off = L.g_attn_off;
    a.g_ffn_off = L.g_ffn_off;
    a.qkv = L.qkv;
    a.wo = L.wo;
    a.gu = L.gu;
    a.wd = L.wd;
    a.lm = L.lm;
    if (cfg_coded(cfg)) {
        a.cbase = a.wbase + L.coded_off;
        a.c_layer0_off = L.c_layer0_off;
        a.c_layer_stride = L.c_layer_stride;
        a.c_code_off = L.c_code_off;
        a.c_lm_code_off = L.c_lm_code_off;
        const auto desc = [&](CodedDesc c, const MatDesc& m) {
            c.fl_run = flag_run_words(m.Nt, m.Ks, m.NB, grid);
            c.fl2_run = grouped_run_words(m.Nt, m.Ks, grid);
            return c;
        };
        a.c_qkv = desc(L.c_qkv, L.qkv);
        a.c_wo = desc(L.c_wo, L.wo);
        a.c_gu = desc(L.c_gu, L.gu);
        a.c_wd = desc(L.c_wd, L.wd);
        a.c_lm = desc(L.c_lm, L.lm);
    }
    a.kpool = static_cast<__bf16*>(kv->k_pages);
    a.vpool = static_cast<__bf16*>(kv->v_pages);
    a.pool_layer_elems = size_t(kv->n_pages) * cfg->n_kv_heads * 16 * h;
    a.block_table = kv->block_table;
    a.pages_used = ceil_div(slot0 + r, kKvBlock);
    a.slot0 = slot0;
    a.old_end = tree ? tree->mask_base : ctx_len;
    a.clear_from = tree && tree->piece ? tree->level_end : 0;
    a.level_first = tree && tree->piece ? tree->level_first : 0;
    a.row_tiles = ceil_div(a.G * r, 16);
    attn_cuts(cfg, L, grid, r, a.pages_used, a.pages_per_split, a.a_splits);
    a.grid = grid;
    a.nwg = g_ts_buf ? grid : step_workgroups(cfg, L, grid, a.Hkv * a.row_tiles * a.a_splits);  // (a timeline is one of the whole grid)
    a.xres = reinterpret_cast<float*>(ws + L.m_xres_off);
    a.xfrag = reinterpret_cast<__bf16*>(ws + L.m_xfrag_off);
    a.ss = reinterpret_cast<float*>(ws + L.m_ss_off);
    a.qfrag = reinterpret_cast<__bf16*>(ws + L.m_qfrag_off);
    a.attfrag = reinterpret_cast<__bf16*>(ws + L.m_attfrag_off);
    a.actfrag = reinterpret_cast<__bf16*>(ws + L.m_actfrag_off);
    a.apart = reinterpret_cast<float*>(ws + L.m_apart_off);
    a.xfrag_stride = L.xfrag_stride;
    a.attfrag_stride = L.attfrag_stride;
    a.actfrag_stride = L.actfrag_stride;
    a.qfrag_stride = L.qfrag_stride;
    a.rope = reinterpret_cast<float*>(ws + L.m_rope_off);
    a.best = reinterpret_cast<unsigned long long*>(ws + L.m_best_off);
    a.bar = reinterpret_cast<uint32_t*>(ws + L.m_bar_off);
    a.acount = reinterpret_cast<uint32_t*>(ws + L.m_acount_off);
    a.dpart = reinterpret_cast<float*>(ws + L.m_dpart_off);
    a.dcount = reinterpret_cast<uint32_t*>(ws + L.m_dcount_off);
    a.flags = reinterpret_cast<uint32_t*>(ws + L.m_flags_off);
    a.cand = cand;
    if (tree) {
        a.row_pos = tree->row_pos;
        a.tmask = tree->mask;
        a.tmask_words = tree->mask_words;
        a.tmask_base = tree->mask_base;
        a.topk = tree->topk;
        a.topk_tok = tree->topk_tok;
        a.topk_prob = tree->topk_prob;
        a.topk_part = reinterpret_cast<unsigned long long*>(ws + L.m_topk_off);
        a.lse_part = reinterpret_cast<float*>(ws + L.m_lse_off);
        if (!out) out = reinterpret_cast<card_verify_result*>(ws + L.m_out_off);
    }
    a.pending = kv->pending_token;
    if (sampling && sampling->temperature > 0.f) {
        a.inv_temp = 1.0f / sampling->temperature;
        a.seed_lo = uint32_t(sampling->seed & 0xffffffffull);
        a.seed_hi = uint32_t(sampling->seed >> 32);
    }
    a.out = out;
    a.row_argmax = row_argmax;
    a.logits = logits;
    a.ts = g_ts_buf;
    a.ts_layer = g_ts_layer;
    hipStream_t st = as_stream(stream);
    ProfScope ps(st);
    if (tree && tree->piece) {
        if (r <= 8) return h == 128 ? launch_mega<1, 128, true, true, true>(a, st) : launch_mega<1, 64, true, true, true>(a, st);
        if (r <= 16) return h == 128 ? launch_mega<1, 128, false, true, true>(a, st) : launch_mega<1, 64, false, true, true>(a, st);
        return h == 128 ? launch_mega<2, 128, false, true, true>(a, st) : launch_mega<2, 64, false, true, true>(a, st);
    }
    if (tree) {
        if (r <= 8) return h == 128 ? launch_mega<1, 128, true, true>(a, st) : launch_mega<1, 64, true, true>(a, st);
        if (r <= 16) return h == 128 ? launch_mega<1, 128, false, true>(a, st) : launch_mega<1, 64, false, true>(a, st);
        return h == 128 ? launch_mega<2, 128, false, true>(a, st) : launch_mega<2, 64, false, true>(a, st);
    }
    if (r <= 8) return h == 128 ? launch_mega<1, 128, true, false>(a, st) : launch_mega<1, 64, true, false>(a, st);
    if (r <= 16) return h == 128 ? launch_mega<1, 128, false, false>(a, st) : launch_mega<1, 64, false, false>(a, st);
    return h == 128 ? launch_mega<2, 128, false, false>(a, st) : launch_mega<2, 64, false, false>(a, st);
}

int draft_impl(const card_model_cfg* cfg, const void* packed, const card_kv* kv, int32_t ctx_len, const card_tree_rows* rows,
               int32_t n_rows, int32_t k, void* workspace, void* stream, int32_t* topk_tokens, float* topk_probs, float* logits,
               bool piece, int32_t level_first, int32_t level_end) {
    if (!rows || !kv) return CARD_EINVAL;
    const TreeOpt t = {rows->positions_dev, rows->first_slot, rows->mask_dev, rows->mask_words, rows->mask_base, k,
                       topk_tokens, topk_probs, piece, level_first, level_end};
    card_kv kv2 = *kv;
    kv2.pending_token = -1;
    return verify_impl(cfg, packed, &kv2, ctx_len, rows->tokens_dev, n_rows, workspace, stream, nullptr, nullptr, logits, nullptr, &t);
}

// ---- prompt pass (card_prompt.hip) -----------------------------------------------------------------
constexpr int kPromptMaxRows = 1024;  // rows per pass: the chip is full (more rows per pass measured no gain)

// How a product is run: workgroups of `waves` wavefronts on 4 * waves weight tiles x `tiles` row tiles, K in `splits` ranges.
struct PromptPlan {
    int waves, tiles, splits;
};
// The plan with the least estimated time.  A workgroup's time goes with its k-steps, plus 5-6 for filling and draining:
// of four wavefronts 0.43 us a step alone on a compute unit, 0.75 with a second one beside it (512 at a time, a third of a last
// round that is not full is lost); of eight, one per compute unit, 0.70 us with four row tiles and 1.16 with seven, in whole rounds
// of 256.  Every K range writes the product once more in fp32 (4.4 TB/s) and the next kernel reads it (5 TB/s); a cut
// gate/up product needs a kernel of its own behind it (4 us).
// Against the fastest of all plans with 1, 2, ... 8, 12 or 16 ranges on the 1B, 7B, 8B and 70B shapes with 16-1024 rows (240 products, with what the
// next kernel pays): within 5 % in 95 % of them, at worst 9 % slower (7B gate/up, 64 rows: 55 us, another plan 50).  The wide
// workgroups read less of the activations and weights per matrix instruction: from 200 rows on they give 3-8 %.
PromptPlan prompt_plan(int Nt, int Ks, int mts, bool swiglu) {
    const int turns = ceil_div(Ks, kPgUnroll);
    PromptPlan best = {4, 4, 1};
    double best_us = 1e30;
    for (const PromptPlan& v : {PromptPlan{4, 4, 0}, PromptPlan{8, 4, 0}, PromptPlan{8, 7, 0}}) {
        if (v.tiles > 4 && mts <= 4) continue;
        const int64_t blocks = int64_t(ceil_div(Nt, v.waves * kPgN)) * ceil_div(mts, v.tiles);
        for (int s = 1; s <= 16 && (s == 1 || turns / s >= 2); ++s) {
            const int64_t wgs = blocks * s;
            const double steps = ceil_div(turns, s) * kPgUnroll;
            double us;
            if (v.waves == 8) us = (steps + 4.8) * (v.tiles == 4 ? 0.70 : 1.16) * ceil_div(wgs, 256);
            else if (wgs <= 256) us = (steps + 6) * 0.43;
            else us = (steps + 6) * 0.75 * std::max(1.0, 0.68 * double(wgs) / 512 + 0.32 * ceil_div(wgs, 512));
            if (!swiglu || s > 1) us += double(s) * Nt * mts * 1024.0 * (1 / 4.4e6 + 1 / 5e6) + (swiglu ? 4.0 : 0.0);
            if (us < best_us) {
                best_us = us;
                best = {v.waves, v.tiles, s};
            }
        }
    }
    return best;
}

struct PromptLayout {
    size_t x, xf, ss, att, act, q, rope, best, part;  // part: the last one, of prompt_part_bytes
    int mcap, groups;
};
PromptLayout prompt_layout(const card_model_cfg* cfg, const Layout& L, int rows) {
    PromptLayout p = {};
    p.mcap = ceil_div(rows, 16 * kPgTiles) * kPgTiles;
    p.groups = ceil_div(cfg->d_model, kPgGroup);
    const size_t cap = size_t(p.mcap) * 16, h = cfg->head_dim;
    size_t w = 0;
    auto take = [&](size_t bytes) {
        const size_t at = w;
        w = align_up(w + bytes, 1024);
        return at;
    };
    p.x = take(cap * cfg->d_model * 4);
    p.xf = take(size_t(L.qkv.Ks) * p.mcap * 2048);
    p.ss = take(cap * p.groups * 4);
    p.att = take(size_t(L.wo.Ks) * p.mcap * 2048);
    p.act = take(size_t(L.wd.Ks) * p.mcap * 2048);
    p.q = take(cap * cfg->n_q_heads * h * 4);
    p.rope = take(cap * h * 4);
    p.best = take(8);
    p.part = w;
    return p;
}
// Room for the partial products of up to mcap row tiles (256 plans per 1024 rows: for the size query, not for each prompt).
size_t prompt_part_bytes(const Layout& L, int mcap) {
    size_t part = 0;
    for (int m = 1; m <= mcap; ++m)
        for (const MatDesc* d : {&L.qkv, &L.wo, &L.gu, &L.wd}) {
            const int s = prompt_plan(d->Nt, d->Ks, m, d == &L.gu).splits;
            if (d != &L.gu || s > 1) part = std::max(part, size_t(s) * d->Nt * m * 1024);
        }
    return part;
}

// The product of the row tiles [g.mt0, g.mts).
template <int EPI>
void prompt_gemm(PgemmArgs g, const PromptPlan& plan, hipStream_t st) {
    g.splits = plan.splits;
    g.nblk = ceil_div(g.Nt, plan.waves * kPgN);
    g.mblk = ceil_div(g.mts - g.mt0, plan.tiles);
    const dim3 grid(uint32_t(ceil_div(int64_t(g.nblk) * g.mblk * g.splits, 8) * 8)), block(uint32_t(plan.waves) * 64);
    if constexpr (EPI != PG_ARGMAX) {  // (one row tile)
        if (plan.waves == 8) {
            if (plan.tiles == 4) hipLaunchKernelGGL((k_prompt_gemm<EPI, 8, 4>), grid, block, 0, st, g);
            else hipLaunchKernelGGL((k_prompt_gemm<EPI, 8, 7>), grid, block, 0, st, g);
            return;
        }
    }
    hipLaunchKernelGGL((k_prompt_gemm<EPI, 4, 4>), grid, block, 0, st, g);
}

// One pass: `rows` tokens at positions ctx_len .. (a multiple of 16).  next_token: where the arg-max behind the
// last row goes, or null.
int prompt_pass(const card_model_cfg* cfg, const Layout& L, const PromptLayout& P, const char* packed, const card_kv* kv,
                int ctx_len, const int32_t* tokens, int rows, char* ws, int nwg, hipStream_t st, int32_t* next_token) {
    const int mts = ceil_div(rows, 16), h = cfg->head_dim, d = cfg->d_model, G = cfg->n_q_heads / cfg->n_kv_heads;
    const int mpad = ceil_div(mts, kPgTiles) * kPgTiles;
    __bf16* xf = reinterpret_cast<__bf16*>(ws + P.xf);
    __bf16* att = reinterpret_cast<__bf16*>(ws + P.att);
    __bf16* act = reinterpret_cast<__bf16*>(ws + P.act);
    PepiArgs e = {};
    e.part = reinterpret_cast<float*>(ws + P.part);
    e.d = d;
    e.rows = rows;
    e.x = reinterpret_cast<float*>(ws + P.x);
    e.xf = xf;
    e.ss = reinterpret_cast<float*>(ws + P.ss);
    e.ss_groups = P.groups;
    e.embed = reinterpret_cast<const __bf16*>(packed + L.embed_off);
    e.tokens = tokens;
    e.V = cfg->vocab;
    e.best = reinterpret_cast<unsigned long long*>(ws + P.best);
    e.qd = cfg->n_q_heads * h;
    e.kvd = cfg->n_kv_heads * h;
    e.h = h;
    e.Hkv = cfg->n_kv_heads;
    e.G = G;
    e.ctx_len = ctx_len;
    e.qcap = mpad * 16 * G;
    e.inv_d = 1.0f / float(d);
    e.eps = cfg->rms_eps;
    e.inv_sqrt_h = 1.4426950408889634f / sqrtf(float(h));
    e.rope = reinterpret_cast<float*>(ws + P.rope);
    e.rope_rows = mpad * 16;
    e.q = reinterpret_cast<__bf16*>(ws + P.q);
    e.block_table = kv->block_table;
    const auto gain = [&](int l, bool ffn) {
        if (l == cfg->n_layers) return reinterpret_cast<const float*>(packed + L.g_final_off);
        const char* lb = packed + L.layer0_off + size_t(l) * L.layer_stride;
        return reinterpret_cast<const float*>(lb + (ffn ? L.g_ffn_off : L.g_attn_off));
    };
    const auto gemm = [&](const MatDesc& m, const char* base, const __bf16* in, PgemmEpi epi, int mt0) {
        PgemmArgs g = {};
        g.w = base + m.off;
        g.bytes = uint32_t(m.bytes());
        g.Nt = m.Nt;
        g.Ks = m.Ks;
        g.NB = m.NB;
        g.nwg = nwg;
        g.x = in;
        g.mts = mts;
        g.mt0 = e.mp0 = mt0;  // (a tile that goes on alone may be cut many ways: its partials get few rows)
        g.mcap = e.mcap = mts - mt0;
        g.part = const_cast<float*>(e.part);
        g.ss = e.ss;
        g.ss_groups = P.groups;
        g.inv_d = e.inv_d;
        g.eps = e.eps;
        g.act = act;
        g.Ks_out = L.wd.Ks;
        g.row = rows - 1;
        g.V = cfg->vocab;
        g.best = e.best;
        const PromptPlan plan = epi == PG_ARGMAX ? PromptPlan{4, 4, 1} : prompt_plan(m.Nt, m.Ks, mts - mt0, epi == PG_SWIGLU);
        e.splits = plan.splits;
        e.Nt = m.Nt;
        if (epi == PG_ARGMAX) {
            prompt_gemm<PG_ARGMAX>(g, plan, st);
        } else if (epi == PG_SWIGLU && plan.splits == 1) {
            prompt_gemm<PG_SWIGLU>(g, plan, st);
        } else {
            prompt_gemm<PG_PART>(g, plan, st);
            if (epi == PG_SWIGLU) {
                e.mt0 = mt0;
                hipLaunchKernelGGL(k_prompt_swiglu, dim3(uint32_t(ceil_div(m.Nt, 2 * kPgWaves)), uint32_t(mts - mt0)), dim3(256), 0, st, e,
                                   act, L.wd.Ks);
            }
        }
    };
    const auto resid = [&](const float* next_gain, int mt0) {
        e.gain = next_gain;
        e.mt0 = mt0;
        hipLaunchKernelGGL(k_prompt_resid<false>, dim3(uint32_t(P.groups), uint32_t(mts - mt0)), dim3(256), 0, st, e);
    };
    const size_t pool_layer = size_t(kv->n_pages) * cfg->n_kv_heads * 16 * h;
    e.gain = gain(0, false);
    hipLaunchKernelGGL(k_prompt_resid<true>, dim3(uint32_t(P.groups), uint32_t(mts)), dim3(256), 0, st, e);
    hipLaunchKernelGGL(k_prompt_rope, dim3(uint32_t(ceil_div(int64_t(rows) * (h / 2), 256))), dim3(256), 0, st,
                       reinterpret_cast<float*>(ws + P.rope), rows, mpad * 16, h / 2, ctx_len, cfg->rope_theta, h);
    for (int l = 0; l < cfg->n_layers; ++l) {
        const char* lb = packed + L.layer0_off + size_t(l) * L.layer_stride;
        const bool last = l + 1 == cfg->n_layers;
        gemm(L.qkv, lb, xf, PG_PART, 0);
        e.kpool = static_cast<__bf16*>(kv->k_pages) + size_t(l) * pool_layer;
        e.vpool = static_cast<__bf16*>(kv->v_pages) + size_t(l) * pool_layer;
        hipLaunchKernelGGL(k_prompt_qkv, dim3(uint32_t(ceil_div(L.qkv.Nt, kPgWaves)), uint32_t(mts)), dim3(256), 0, st, e);
        // behind the last layer's K and V only the row that predicts is still of use: its row tile goes on alone
        if (last && !next_token) break;
        const int mt0 = last ? mts - 1 : 0;
        const PattnArgs t = {e.q, e.kpool, e.vpool, kv->block_table, e.qcap, rows, G, e.Hkv, ctx_len, ceil_div(int64_t(rows) * G, 16),
                             L.wo.Ks, att};
        const dim3 ag(uint32_t(ceil_div(last ? std::min(G, t.row_tiles) : t.row_tiles, kPgWaves) * e.Hkv));
        if (h == 128) hipLaunchKernelGGL(k_prompt_attn<128>, ag, dim3(256), 0, st, t);
        else hipLaunchKernelGGL(k_prompt_attn<64>, ag, dim3(256), 0, st, t);
        gemm(L.wo, lb, att, PG_PART, mt0);
        resid(gain(l, true), mt0);
        gemm(L.gu, lb, xf, PG_SWIGLU, mt0);
        gemm(L.wd, lb, act, PG_PART, mt0);
        resid(gain(l + 1, false), mt0);
    }
    if (next_token) {
        gemm(L.lm, packed, xf, PG_ARGMAX, mts - 1);
        hipLaunchKernelGGL(k_prompt_token, dim3(1), dim3(1), 0, st, e.best, reinterpret_cast<const uint32_t*>(packed + L.stamp_off),
                           nwg, next_token);
    }
    return launch_status();
}

// ---- wide levels (card_level.hip) -------------------------------------------------------------------
struct LevelLayout {
    size_t x, xf, ss, att, act, q, rope, part, apart, counts, logits, lse, best, bytes;
    int n_counts;
};
LevelLayout level_layout(const card_model_cfg* cfg, const Layout& L) {
    LevelLayout p = {};
    constexpr size_t rows = kLvTiles * 16;
    const size_t h = cfg->head_dim, G = cfg->n_q_heads / cfg->n_kv_heads;
    size_t w = 0;
    auto take = [&](size_t bytes) {
        const size_t at = w;
        w = align_up(w + bytes, 1024);
        return at;
    };
    p.x = take(rows * cfg->d_model * 4);
    p.xf = take(size_t(L.qkv.Ks) * kLvTiles * 2048);
    p.ss = take(rows * (cfg->d_model / 16) * 4);
    p.att = take(size_t(L.wo.Ks) * kLvTiles * 2048);
    p.act = take(size_t(L.wd.Ks) * kLvTiles * 2048);
    p.q = take(rows * cfg->n_q_heads * h * 4);
    p.rope = take(rows * h * 4);
    p.part = take(size_t(4) * std::max(L.qkv.Nt, std::max(L.wo.Nt, L.wd.Nt)) * kLvTiles * 1024);
    // (a row tile's cuts never outnumber the grid, unless its heads do)
    p.apart = take(kLvTiles * std::max<size_t>(256, cfg->n_kv_heads * G) * 16 * (h + 2) * 4);
    p.n_counts = int(kLvTiles * cfg->n_kv_heads * G);
    p.counts = take(size_t(p.n_counts) * 4);
    p.logits = take(rows * L.lm.Nt * 16 * 4);
    p.lse = take(rows * 256 * 8);
    p.best = take(rows * 256 * 16 * 8);
    p.bytes = w;
    return p;
}

template <int EPI, int N, int MT>
void level_gemm(LvGemmArgs g, hipStream_t st) {
    g.nblk = ceil_div(g.Nt, kLvWaves * N);
    g.mblk = ceil_div(g.n_tiles, MT);
    const int64_t wgs = int64_t(g.nblk) * g.mblk * (EPI == LV_PART ? 4 : 1);
    hipLaunchKernelGGL((k_level_gemm<EPI, N, MT>), dim3(uint32_t(ceil_div(wgs, 8) * 8)), dim3(kLvWaves * 64), 0, st, g);
}
template <int EPI>
void level_product(const LvGemmArgs& g, hipStream_t st) {
    // whole rounds of 256 workgroups, times what they bring into a compute unit per k-step
    const auto rounds = [&](int n, int mt) {
        return ceil_div(int64_t(ceil_div(g.Nt, kLvWaves * n)) * ceil_div(g.n_tiles, mt) * (EPI == LV_PART ? 4 : 1), 256) * (kLvWaves * n + 2 * mt);
    };
    if constexpr (EPI == LV_PART) {
        if (rounds(1, 2) <= rounds(2, 2)) level_gemm<EPI, 1, 2>(g, st);
        else level_gemm<EPI, 2, 2>(g, st);
    } else {
        if (g.n_tiles > 4 && rounds(2, 8) < std::min(rounds(1, 4), rounds(2, 4))) level_gemm<EPI, 2, 8>(g, st);
        else if (rounds(1, 4) <= rounds(2, 4)) level_gemm<EPI, 1, 4>(g, st);
        else level_gemm<EPI, 2, 4>(g, st);
    }
}

// The rows of `e.t` (of the n_rows of the level) through the model.
int level_pass(const card_model_cfg* cfg, const Layout& L, const LevelLayout& P, const char* packed, const card_kv* kv, LvArgs e,
               int tasks, const card_tree_rows* rows, int k, char* ws, int nwg, hipStream_t st, int32_t* tok, float* prob) {
    const int h = cfg->head_dim;
    uint32_t pk_tiles = 0;
    for (int i = 0; i < e.n_tiles; ++i) pk_tiles |= uint32_t(e.t[i].pk) << i;
    const auto gain = [&](int l, bool ffn) {
        if (l == cfg->n_layers) return reinterpret_cast<const float*>(packed + L.g_final_off);
        const char* lb = packed + L.layer0_off + size_t(l) * L.layer_stride;
        return reinterpret_cast<const float*>(lb + (ffn ? L.g_ffn_off : L.g_attn_off));
    };
    const auto product = [&](const MatDesc& m, const char* base, const __bf16* in) {
        LvGemmArgs g = {};
        g.w = base + m.off;
        g.bytes = uint32_t(m.bytes());
        g.Nt = e.Nt = m.Nt;
        g.Ks = m.Ks;
        g.NB = m.NB;
        g.nwg = nwg;
        g.x = in;
        g.n_tiles = e.n_tiles;
        g.pk_tiles = pk_tiles;
        g.part = const_cast<float*>(e.part);
        g.ss = e.ss;
        g.n_part = cfg->d_model / 16;
        g.Ks_out = L.wd.Ks;
        g.inv_d = e.inv_d;
        g.eps = e.eps;
        g.act = reinterpret_cast<__bf16*>(ws + P.act);
        g.logits = reinterpret_cast<float*>(ws + P.logits);
        g.ldl = L.lm.Nt * 16;
        return g;
    };
    const dim3 cols(uint32_t(cfg->d_model / 64), uint32_t(e.n_tiles));
    e.gain = gain(0, false);
    hipLaunchKernelGGL(k_level_resid<true>, cols, dim3(256), 0, st, e);
    hipLaunchKernelGGL(k_level_rope, dim3(uint32_t(ceil_div(e.n_tiles * 16 * (h / 2), 256))), dim3(256), 0, st, e,
                       reinterpret_cast<float*>(ws + P.rope), rows->positions_dev, cfg->rope_theta);
    const size_t pool_layer = size_t(kv->n_pages) * cfg->n_kv_heads * 16 * h;
    for (int l = 0; l < cfg->n_layers; ++l) {
        const char* lb = packed + L.layer0_off + size_t(l) * L.layer_stride;
        level_product<LV_PART>(product(L.qkv, lb, e.xf), st);
        e.kpool = static_cast<__bf16*>(kv->k_pages) + size_t(l) * pool_layer;
        e.vpool = static_cast<__bf16*>(kv->v_pages) + size_t(l) * pool_layer;
        hipLaunchKernelGGL(k_level_qkv, dim3(uint32_t(ceil_div(L.qkv.Nt, 4)), uint32_t(e.n_tiles)), dim3(256), 0, st, e);
        if (h == 128) hipLaunchKernelGGL(k_level_attn<128>, dim3(uint32_t(tasks)), dim3(256), 0, st, e);
        else hipLaunchKernelGGL(k_level_attn<64>, dim3(uint32_t(tasks)), dim3(256), 0, st, e);
        level_product<LV_PART>(product(L.wo, lb, e.att), st);
        e.gain = gain(l, true);
        hipLaunchKernelGGL(k_level_resid<false>, cols, dim3(256), 0, st, e);
        level_product<LV_SWIGLU>(product(L.gu, lb, e.xf), st);
        LvGemmArgs g = product(L.wd, lb, reinterpret_cast<const __bf16*>(ws + P.act));
        g.grouped = (nwg & 7) == 0 && (L.wd.Nt & 3) == 0;
        level_product<LV_PART>(g, st);
        e.gain = gain(l + 1, false);
        hipLaunchKernelGGL(k_level_resid<false>, cols, dim3(256), 0, st, e);
    }
    level_product<LV_LOGITS>(product(L.lm, packed, e.xf), st);
    LvTopkArgs t = {};
    t.logits = reinterpret_cast<const float*>(ws + P.logits);
    t.ldl = L.lm.Nt * 16;
    t.V = cfg->vocab;
    t.Nt = L.lm.Nt;
    t.nwg = nwg;
    t.n_tiles = e.n_tiles;
    t.k = k;
    t.stamp = reinterpret_cast<const uint32_t*>(packed + L.stamp_off);
    std::copy(e.t, e.t + kLvTiles, t.t);
    t.lse = reinterpret_cast<float*>(ws + P.lse);
    t.best = reinterpret_cast<unsigned long long*>(ws + P.best);
    t.tok = tok;
    t.prob = prob;
    hipLaunchKernelGGL(k_level_lse, dim3(uint32_t(ceil_div(nwg, 32)), uint32_t(e.n_tiles * 16)), dim3(256), 0, st, t);
    hipLaunchKernelGGL(k_level_topk, dim3(uint32_t(e.n_tiles * 16)), dim3(256), 0, st, t);
    return launch_status();
}

}  // namespace

extern "C" {

const char* card_strerror(int status) {
    switch (status) {
        case CARD_OK: return "ok";
        case CARD_EINVAL: return "invalid argument";
        case CARD_ERANGE: return "value out of range";
        case CARD_ECAPACITY: return "KV cache capacity exceeded";
        case CARD_EDEVICE: return "device error";
        case CARD_ESTALE: return "stale cache epoch";
        case CARD_ETOOBIG: return "workspace of this model exceeds the static scratch buffer";
        default: return "unknown status";
    }
}

size_t card_packed_weight_bytes(const card_model_cfg* cfg) {
    const Layout L = make_layout(cfg);
    return L.ok ? L.weight_bytes : 0;
}

size_t card_workspace_bytes(const card_model_cfg* cfg) {
    const Layout L = make_layout(cfg);
    return L.ok ? L.ws_bytes : 0;
}

size_t card_kv_pool_bytes(const card_model_cfg* cfg, int32_t n_pages) {
    if (!cfg_valid(cfg) || n_pages <= 0) return 0;
    return size_t(cfg->n_layers) * n_pages * cfg->n_kv_heads * 16 * cfg->head_dim * 2;
}

int64_t card_stream_frag_index(int32_t n_tiles, int32_t k_steps, int32_t batch, int32_t grid, int32_t t, int32_t s) {
    if (n_tiles <= 0 || k_steps <= 0 || batch <= 0 || grid <= 0 || t < 0 || t >= n_tiles || s < 0 || s >= k_steps)
        return -1;
    return stream_frag_index(n_tiles, k_steps, batch, grid, t, s);
}

int card_weights_pack_tensor(const card_model_cfg* cfg, int32_t tensor, int32_t layer, const void* src_dev,
                             void* packed_dev, void* stream) {
    if (!src_dev || !packed_dev) return CARD_EINVAL;
    const Layout L = make_layout(cfg);
    if (!L.ok) return CARD_EINVAL;
    if (tensor < CARD_T_EMBED || tensor > CARD_T_G_FINAL) return CARD_EINVAL;
    const bool per_layer = !(tensor == CARD_T_EMBED || tensor == CARD_T_LM_HEAD || tensor == CARD_T_G_FINAL);
    if (per_layer && (layer < 0 || layer >= cfg->n_layers)) return CARD_ERANGE;
    hipStream_t st = as_stream(stream);
    char* pb = static_cast<char*>(packed_dev);
    char* lb = pb + L.layer0_off + size_t(per_layer ? layer : 0) * L.layer_stride;
    const int d = cfg->d_model, h = cfg->head_dim, qd = cfg->n_q_heads * h, kvd = cfg->n_kv_heads * h;

    auto copy = [&](char* dst, size_t bytes) {
        return hipMemcpyAsync(dst, src_dev, bytes, hipMemcpyDeviceToDevice, st) == hipSuccess ? CARD_OK
                                                                                               : CARD_EDEVICE;
    };
    // coded copy: of the vocabulary head or of the layer
    char* cb = pb + L.coded_off;
    char* clb = per_layer ? cb + L.c_layer0_off + size_t(layer) * L.c_layer_stride : cb;
    auto pack = [&](char* dst, const MatDesc& m, int src_rows, int n_rows, int prow0, int map, const CodedDesc& c, int which) {
        PackArgs a = {};
        a.src = static_cast<const __bf16*>(src_dev);
        a.dst = reinterpret_cast<__bf16*>(dst + m.off);
        a.src_rows = src_rows;
        a.K = m.K;
        a.Ks = m.Ks;
        a.prow0 = prow0;
        a.map = map;
        a.head_dim = h;
        a.Nt = m.Nt;
        a.NB = m.NB;
        a.nwg = grid_size(cfg);
        if (a.nwg <= 0) return int(CARD_EDEVICE);
        const bool half = map == MAP_GATE || map == MAP_UP;  // eight rows of every tile
        a.t0 = half ? 0 : prow0 / 16;
        a.tiles = half ? m.Nt : n_rows / 16;
        a.stamp = reinterpret_cast<uint32_t*>(pb + L.stamp_off);
        const int slot = per_layer ? layer : cfg->n_layers;
        if (slot < kCopySlots) a.copy_word = a.stamp + kCopyWord + slot / 4;
        a.copy_bit = 1u << (slot % 4 * 8 + which);
        if (cfg_coded(cfg)) {
            uint32_t* code = reinterpret_cast<uint32_t*>(clb + (per_layer ? L.c_code_off : L.c_lm_code_off));
            a.planes = clb + c.off;
            a.fl = reinterpret_cast<unsigned long long*>(clb + (map == MAP_UP ? c.fl2 : c.fl));
            // (only grids that can take it in groups: elsewhere a run of the grouped order has no room of its own)
            if (tensor == CARD_T_WD && (m.Nt & 3) == 0 && ((a.nwg & 7) == 0 || m.Nt <= a.nwg))
                a.gfl = reinterpret_cast<unsigned long long*>(clb + c.fl2);
            a.base4 = code + which;
            a.counts = code + kCodeCounts + 128 * which;
        }
        hipLaunchKernelGGL(k_pack_begin, dim3(1), dim3(128), 0, st, a);
        if (cfg_coded(cfg)) {
            const int64_t pieces = (int64_t(src_rows) * m.K / 8 + 255) / 256;
            hipLaunchKernelGGL(k_pack_count, dim3(uint32_t(std::min<int64_t>(pieces, 1024))), dim3(256), 0, st, a);
            hipLaunchKernelGGL(k_pack_base, dim3(1), dim3(128), 0, st, a);
        }
        hipLaunchKernelGGL(k_pack, dim3(uint32_t((int64_t(a.tiles) * m.Ks + 3) / 4)), dim3(256), 0, st, a);
        return launch_status();
    };
    switch (tensor) {
        case CARD_T_EMBED: return copy(pb + L.embed_off, size_t(cfg->vocab) * d * 2);
        case CARD_T_G_FINAL: return copy(pb + L.g_final_off, size_t(d) * 4);
        case CARD_T_G_ATTN: return copy(lb + L.g_attn_off, size_t(d) * 4);
        case CARD_T_G_FFN: return copy(lb + L.g_ffn_off, size_t(d) * 4);
        case CARD_T_WQ: return pack(lb, L.qkv, qd, qd, 0, MAP_ROPE, L.c_qkv, CT_Q);
        case CARD_T_WK: return pack(lb, L.qkv, kvd, kvd, qd, MAP_ROPE, L.c_qkv, CT_K);
        case CARD_T_WV: return pack(lb, L.qkv, kvd, kvd, qd + kvd, MAP_IDENT, L.c_qkv, CT_V);
        case CARD_T_WO: return pack(lb, L.wo, d, L.wo.Nt * 16, 0, MAP_IDENT, L.c_wo, CT_O);
        case CARD_T_WG: return pack(lb, L.gu, cfg->d_ffn, cfg->d_ffn, 0, MAP_GATE, L.c_gu, CT_G);
        case CARD_T_WU: return pack(lb, L.gu, cfg->d_ffn, cfg->d_ffn, 0, MAP_UP, L.c_gu, CT_U);
        case CARD_T_WD: return pack(lb, L.wd, d, L.wd.Nt * 16, 0, MAP_IDENT, L.c_wd, CT_D);
        default: {
            MatDesc m = L.lm;
            m.off = 0;
            return pack(pb + L.lm_off, m, cfg->vocab, L.lm.Nt * 16, 0, MAP_IDENT, L.c_lm, 0);
        }
    }
}

int card_verify(const card_model_cfg* cfg, const void* packed_weights_dev, const card_kv* kv, int32_t ctx_len,
                const int32_t* cand_tokens_dev, int32_t r, void* workspace_dev, void* stream,
                card_verify_result* out_dev, int32_t* row_argmax_dev) {
    return verify_impl(cfg, packed_weights_dev, kv, ctx_len, cand_tokens_dev, r, workspace_dev, stream, out_dev,
                       row_argmax_dev, nullptr);
}

int card_verify_sampled(const card_model_cfg* cfg, const void* packed_weights_dev, const card_kv* kv, int32_t ctx_len,
                        const int32_t* cand_tokens_dev, int32_t r, const card_sampling* sampling, void* workspace_dev,
                        void* stream, card_verify_result* out_dev, int32_t* row_token_dev, float* logits_dev) {
    if (!sampling || !(sampling->temperature >= 0.f)) return CARD_EINVAL;
    return verify_impl(cfg, packed_weights_dev, kv, ctx_len, cand_tokens_dev, r, workspace_dev, stream, out_dev,
                       row_token_dev, logits_dev, sampling);
}

int card_draft_level(const card_model_cfg* cfg, const void* packed_weights_dev, const card_kv* kv, int32_t ctx_len,
                     const card_tree_rows* rows, int32_t n_rows, int32_t k, void* workspace_dev, void* stream,
                     int32_t* topk_tokens_dev, float* topk_probs_dev, float* logits_dev) {
    return draft_impl(cfg, packed_weights_dev, kv, ctx_len, rows, n_rows, k, workspace_dev, stream, topk_tokens_dev, topk_probs_dev,
                      logits_dev, false, 0, 0);
}

int card_draft_level_piece(const card_model_cfg* cfg, const void* packed_weights_dev, const card_kv* kv, int32_t ctx_len,
                           const card_tree_rows* rows, int32_t n_rows, int32_t level_first, int32_t level_end, int32_t k,
                           void* workspace_dev, void* stream, int32_t* topk_tokens_dev, float* topk_probs_dev, float* logits_dev) {
    return draft_impl(cfg, packed_weights_dev, kv, ctx_len, rows, n_rows, k, workspace_dev, stream, topk_tokens_dev, topk_probs_dev,
                      logits_dev, true, level_first, level_end);
}

int card_tree_mask_level(const uint32_t* parent_mask_host, const int32_t* parent_idx_host, int32_t n_rows,
                         int32_t first_slot, int32_t ctx_len, int32_t mask_base, int32_t mask_words,
                         uint32_t* out_mask_host) {
    if (!parent_idx_host || !out_mask_host || n_rows < 1) return CARD_EINVAL;
    if (mask_words < 1 || mask_words > 32 || mask_base < 0 || mask_base % kKvBlock || mask_base > ctx_len) return CARD_EINVAL;
    if (first_slot < ctx_len || int64_t(first_slot) + n_rows > int64_t(mask_base) + 32 * mask_words) return CARD_ERANGE;
    for (int i = 0; i < n_rows; ++i) {
        uint32_t* row = out_mask_host + size_t(i) * mask_words;
        const int p = parent_idx_host[i];
        if (p >= 0) {
            if (!parent_mask_host) return CARD_EINVAL;
            // inherit the parent's causal history
            for (int w = 0; w < mask_words; ++w) row[w] = parent_mask_host[size_t(p) * mask_words + w];
        } else {
            // a root of the tree sees the committed context only
            for (int w = 0; w < mask_words; ++w) row[w] = 0u;
            for (int s = mask_base; s < ctx_len; ++s) row[(s - mask_base) >> 5] |= 1u << ((s - mask_base) & 31);
        }
        const int own = first_slot + i - mask_base;  // ... plus the node itself; peers stay invisible
        row[own >> 5] |= 1u << (own & 31);
    }
    return CARD_OK;
}

int card_cache_select(const float* sigma_dev, const int32_t* topk_tokens_dev, const float* topk_probs_dev, int32_t n_parents,
                      int32_t k, int32_t K, int32_t* out_tokens_dev, float* out_scores_dev, int32_t* out_parents_dev,
                      void* stream) {
    if (!sigma_dev || !topk_tokens_dev || !topk_probs_dev || !out_tokens_dev || !out_scores_dev || !out_parents_dev)
        return CARD_EINVAL;
    if (n_parents < 1 || k < 1 || k > 16 || K < 1 || int64_t(n_parents) * k > kSelMax) return CARD_ERANGE;
    SelectArgs a = {sigma_dev, topk_tokens_dev, topk_probs_dev, n_parents, k, K, out_tokens_dev, out_scores_dev,
                    out_parents_dev};
    int threads = 64;  // two keys each
    while (2 * threads < n_parents * k) threads *= 2;
    hipLaunchKernelGGL(k_cache_select, dim3(1), dim3(uint32_t(threads)), 0, as_stream(stream), a);
    const int st = launch_status();
    return st != CARD_OK ? st : (K < n_parents * k ? K : n_parents * k);
}

static int step_begin_impl(card_cache* cache, const card_model_cfg* cfg, const void* packed_weights_dev, const card_kv* kv,
                    int32_t ctx_len, int32_t max_len, int32_t* cand_staging, void* workspace_dev, void* stream,
                    card_verify_result* out, int32_t* row_argmax_dev, card_step* step_host, const card_sampling* sampling) {
    if (!cache || !cfg || !kv || !cand_staging || !step_host) return CARD_EINVAL;
    if (max_len < 1 || max_len > cfg->max_r || max_len > kMaxR) return CARD_ERANGE;
    if (kv->pending_token < 0) return CARD_EINVAL;  // the query key is the token just verified
    int32_t n = 0;
    float score = 0.f;
    const int hit = card_cache_query(cache, kv->pending_token, max_len, step_host->cand, &n, &score);
    if (hit < 0) return hit;
    if (hit == 0 || n < 1) {  // miss: a plain decode step on the verified token
        n = 1;
        step_host->cand[0] = kv->pending_token;
    }
    step_host->hit = hit > 0 ? 1 : 0;
    step_host->r = n;
    step_host->path_score = hit > 0 ? score : 0.f;
    for (int i = 0; i < n; ++i) cand_staging[i] = step_host->cand[i];
    return verify_impl(cfg, packed_weights_dev, kv, ctx_len, cand_staging, n, workspace_dev, stream, out, row_argmax_dev,
                       nullptr, sampling);
}


int card_step_begin(card_cache* cache, const card_model_cfg* cfg, const void* packed_weights_dev, const card_kv* kv,
                    int32_t ctx_len, int32_t max_len, int32_t* cand_staging, void* workspace_dev, void* stream,
                    card_verify_result* out, int32_t* row_argmax_dev, card_step* step_host) {
    return step_begin_impl(cache, cfg, packed_weights_dev, kv, ctx_len, max_len, cand_staging, workspace_dev, stream, out,
                           row_argmax_dev, step_host, nullptr);
}

int card_step_begin_sampled(card_cache* cache, const card_model_cfg* cfg, const void* packed_weights_dev, const card_kv* kv,
                    int32_t ctx_len, int32_t max_len, int32_t* cand_staging, void* workspace_dev, void* stream,
                    card_verify_result* out, int32_t* row_argmax_dev, card_step* step_host,
                            const card_sampling* sampling) {
    if (!sampling || !(sampling->temperature >= 0.f)) return CARD_EINVAL;
    return step_begin_impl(cache, cfg, packed_weights_dev, kv, ctx_len, max_len, cand_staging, workspace_dev, stream, out,
                           row_argmax_dev, step_host, sampling);
}

int card_step_end(card_cache* cache, const card_step* step_host, const card_verify_result* out_host, int32_t flags,
                  int32_t* emitted_host, int32_t* n_emitted_host) {
    if (!cache || !step_host || !out_host || !emitted_host || !n_emitted_host) return CARD_EINVAL;
    const int a = out_host->accepted_len;
    if (a < 1 || a > step_host->r) return CARD_EDEVICE;  // the step failed (or was not a CARD step)
    // what the step has verified beyond the query key: the accepted part of the path, then the target's own token
    int n = 0;
    for (int i = 1; i < a; ++i) emitted_host[n++] = step_host->cand[i];
    emitted_host[n++] = out_host->correction_token;
    *n_emitted_host = n;
    if (flags & CARD_STEP_NO_CORRECT) return CARD_OK;
    // the accepted candidates (query key first) are walked down the tree: the children of the last
    // one become level 0, where the next query looks the target's own token up
    const int st = card_cache_correct(cache, step_host->cand, a);
    return st < 0 ? st : CARD_OK;
}

int card_verify_static(const card_model_cfg* cfg, const void* packed_weights_dev, const card_kv* kv, int32_t ctx_len,
                       const int32_t* cand_tokens_dev, int32_t r, void* stream, card_verify_result* out_dev,
                       int32_t* row_argmax_dev) {
    const Layout L = make_layout(cfg);
    if (!L.ok || !packed_weights_dev || !kv || !cand_tokens_dev || !out_dev) return CARD_EINVAL;
    if (L.ws_bytes > kStaticWsBytes) return CARD_ETOOBIG;
    if (r < 1 || r > cfg->max_r) return CARD_ERANGE;  // nothing is enqueued for a call that will be refused
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return CARD_EDEVICE;
    void* ws = nullptr;
    {
        std::lock_guard<std::mutex> g(g_static_mu);
        StaticWs& sw = g_static[dev];
        if (!sw.ptr) {
            void* p = nullptr;
            if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return CARD_EDEVICE;
            sw.ptr = p;
        }
        // The layout of the control words depends on the model: a call for another model than the
        // last one (or the first call) clears the part it uses and sets the mark, stream-ordered in
        // front of the step.  The array keeps the last call's contents otherwise.
        if (!sw.prepared || memcmp(&sw.cfg, cfg, sizeof(card_model_cfg)) != 0) {
            hipLaunchKernelGGL(k_ws_init, dim3(1024), dim3(256), 0, as_stream(stream), static_cast<uint4v*>(sw.ptr),
                               L.ws_bytes / 16, reinterpret_cast<uint32_t*>(static_cast<char*>(sw.ptr) + L.m_bar_off) + kBarMagic);
            if (launch_status() != CARD_OK) return CARD_EDEVICE;
            sw.cfg = *cfg;
            sw.prepared = true;
        }
        ws = sw.ptr;
    }
    return verify_impl(cfg, packed_weights_dev, kv, ctx_len, cand_tokens_dev, r, ws, stream, out_dev, row_argmax_dev,
                       nullptr);
}

size_t card_static_scratch_bytes(void) { return kStaticWsBytes; }

int card_static_scratch_reset(void) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return CARD_EDEVICE;
    std::lock_guard<std::mutex> g(g_static_mu);
    g_static[dev].prepared = false;
    return CARD_OK;
}

int card_verify_debug_logits(const card_model_cfg* cfg, const void* packed_weights_dev, const card_kv* kv,
                             int32_t ctx_len, const int32_t* cand_tokens_dev, int32_t r, void* workspace_dev,
                             void* stream, card_verify_result* out_dev, int32_t* row_argmax_dev,
                             float* logits_dev) {
    if (!logits_dev) return CARD_EINVAL;
    return verify_impl(cfg, packed_weights_dev, kv, ctx_len, cand_tokens_dev, r, workspace_dev, stream, out_dev,
                       row_argmax_dev, logits_dev);
}

size_t card_prompt_workspace_bytes(const card_model_cfg* cfg, int32_t rows) {
    const Layout L = make_layout(cfg);
    if (!L.ok || rows < 1) return 0;
    const PromptLayout P = prompt_layout(cfg, L, std::min(rows, kPromptMaxRows));
    return align_up(P.part + prompt_part_bytes(L, P.mcap), 1024);
}

int card_prompt(const card_model_cfg* cfg, const void* packed_weights_dev, const card_kv* kv, int32_t ctx_len,
                const int32_t* tokens_dev, int32_t n, void* workspace_dev, int32_t workspace_rows, void* stream,
                int32_t* next_token_dev) {
    if (!cfg || !packed_weights_dev || !kv || !tokens_dev || !workspace_dev) return CARD_EINVAL;
    const Layout L = make_layout(cfg);
    if (!L.ok) return CARD_EINVAL;
    if (!kv->k_pages || !kv->v_pages || !kv->block_table || kv->n_pages <= 0) return CARD_EINVAL;
    if (!pool_fits(cfg, kv)) return CARD_EINVAL;  // (no step could follow)
    if (ctx_len < 0 || ctx_len % kKvBlock || n < 1 || workspace_rows < 1) return CARD_EINVAL;
    if (reinterpret_cast<uintptr_t>(workspace_dev) % 16) return CARD_EINVAL;  // 16-byte loads and stores
    if (int64_t(ctx_len) + n > cfg->max_ctx) return CARD_ECAPACITY;
    const int nwg = grid_size(cfg);
    if (nwg <= 0) return CARD_EDEVICE;
    const PromptLayout P = prompt_layout(cfg, L, std::min(workspace_rows, kPromptMaxRows));
    // passes of about equal size, whole blocks of row tiles
    const int passes = ceil_div(n, P.mcap * 16), per = ceil_div(ceil_div(n, passes), 16 * kPgTiles) * 16 * kPgTiles;
    for (int at = 0; at < n; at += per) {
        const int st = prompt_pass(cfg, L, P, static_cast<const char*>(packed_weights_dev), kv, ctx_len + at, tokens_dev + at,
                                   std::min(per, n - at), static_cast<char*>(workspace_dev), nwg, as_stream(stream),
                                   at + per >= n ? next_token_dev : nullptr);
        if (st != CARD_OK) return st;
    }
    return CARD_OK;
}

size_t card_level_workspace_bytes(const card_model_cfg* cfg) {
    const Layout L = make_layout(cfg);
    return L.ok ? level_layout(cfg, L).bytes : 0;
}

int card_draft_level_wide(const card_model_cfg* cfg, const void* packed_weights_dev, const card_kv* kv, int32_t ctx_len,
                          const card_tree_rows* rows, int32_t n_rows, int32_t rows_per_call, int32_t k, void* workspace_dev,
                          void* stream, int32_t* topk_tokens_dev, float* topk_probs_dev) {
    if (!cfg || !packed_weights_dev || !kv || !rows || !workspace_dev || !topk_tokens_dev || !topk_probs_dev) return CARD_EINVAL;
    if (!rows->tokens_dev || !rows->positions_dev || !rows->mask_dev) return CARD_EINVAL;
    const Layout L = make_layout(cfg);
    if (!L.ok) return CARD_EINVAL;
    if (!kv->k_pages || !kv->v_pages || !kv->block_table || kv->n_pages <= 0 || !pool_fits(cfg, kv)) return CARD_EINVAL;
    if (reinterpret_cast<uintptr_t>(workspace_dev) % 16 || ctx_len < 0) return CARD_EINVAL;
    if (n_rows < 1 || rows_per_call <= 8 || rows_per_call > cfg->max_r) return CARD_ERANGE;
    const int first = rows->first_slot;
    if (int64_t(first) + n_rows > cfg->max_ctx) return CARD_ECAPACITY;
    if (rows->mask_words < 1 || rows->mask_words > 32 || k < 1 || k > 16) return CARD_ERANGE;
    if (rows->mask_base < 0 || rows->mask_base % kKvBlock || rows->mask_base > ctx_len) return CARD_EINVAL;
    if (first < ctx_len || int64_t(first) + n_rows > int64_t(rows->mask_base) + 32 * rows->mask_words) return CARD_ERANGE;
    const int nwg = grid_size(cfg);
    if (nwg <= 0) return CARD_EDEVICE;
    const LevelLayout P = level_layout(cfg, L);
    char* ws = static_cast<char*>(workspace_dev);
    LvArgs e = {};
    e.d = cfg->d_model;
    e.Ks = L.qkv.Ks;
    e.x = reinterpret_cast<float*>(ws + P.x);
    e.xf = reinterpret_cast<__bf16*>(ws + P.xf);
    e.ss = reinterpret_cast<float*>(ws + P.ss);
    e.part = reinterpret_cast<float*>(ws + P.part);
    e.embed = reinterpret_cast<const __bf16*>(static_cast<const char*>(packed_weights_dev) + L.embed_off);
    e.tokens = rows->tokens_dev;
    e.V = cfg->vocab;
    e.n_counts = P.n_counts;
    e.counts = reinterpret_cast<uint32_t*>(ws + P.counts);
    e.h = cfg->head_dim;
    e.qd = cfg->n_q_heads * e.h;
    e.kvd = cfg->n_kv_heads * e.h;
    e.Hkv = cfg->n_kv_heads;
    e.G = cfg->n_q_heads / cfg->n_kv_heads;
    e.first_slot = e.level_first = first;
    e.level_end = first + n_rows;
    e.last_row = n_rows - 1;
    e.inv_d = 1.0f / float(cfg->d_model);
    e.eps = cfg->rms_eps;
    e.inv_sqrt_h = 1.4426950408889634f / sqrtf(float(e.h));
    e.rope = reinterpret_cast<const float*>(ws + P.rope);
    e.q = reinterpret_cast<__bf16*>(ws + P.q);
    e.block_table = kv->block_table;
    e.mask = rows->mask_dev;
    e.mask_words = rows->mask_words;
    e.mask_base = rows->mask_base;
    e.apart = reinterpret_cast<float*>(ws + P.apart);
    e.att = reinterpret_cast<__bf16*>(ws + P.att);
    e.Ks_att = L.wo.Ks;
    // passes of whole calls, eight row tiles at most
    for (int c0 = 0; c0 < n_rows;) {
        int tasks = 0, counts = 0;
        e.n_tiles = 0;
        while (c0 < n_rows) {
            const int r = std::min(rows_per_call, n_rows - c0), tiles = ceil_div(r, 16);
            if (e.n_tiles + tiles > kLvTiles) break;
            for (int i = 0; i < tiles; ++i) {
                LvTile& t = e.t[e.n_tiles++];
                t.row0 = c0 + 16 * i;
                t.n = std::min(16, r - 16 * i);
                t.pk = r <= 8;
                t.wide = r > 16;
                t.pages = ceil_div(first + c0 + r, kKvBlock);
                attn_cuts(cfg, L, nwg, r, t.pages, t.per_cut, t.cuts);
                t.subs = ceil_div(t.n * e.G, 16);
                t.task0 = tasks;
                t.count0 = counts;
                tasks += e.Hkv * t.subs * t.cuts;
                counts += e.Hkv * t.subs;
            }
            c0 += r;
        }
        const int st = level_pass(cfg, L, P, static_cast<const char*>(packed_weights_dev), kv, e, tasks, rows, k, ws, nwg,
                                  as_stream(stream), topk_tokens_dev, topk_probs_dev);
        if (st != CARD_OK) return st;
    }
    return CARD_OK;
}

int card_profile_timeline(void* buf_dev, int32_t layer) {
    g_ts_buf = static_cast<unsigned long long*>(buf_dev);
    g_ts_layer = layer;
    return CARD_OK;
}

int card_profile_enable(int32_t max_launches) {
    if (max_launches <= 0) return CARD_EINVAL;
    Profile& p = prof();
    std::lock_guard<std::mutex> g(p.mu);
    while (int(p.start.size()) < max_launches) {
        hipEvent_t a, b;
        if (hipEventCreate(&a) != hipSuccess) return CARD_EDEVICE;
        if (hipEventCreate(&b) != hipSuccess) {
            (void)hipEventDestroy(a);
            return CARD_EDEVICE;
        }
        p.start.push_back(a);
        p.stop.push_back(b);
    }
    p.used = 0;
    p.on = true;
    return CARD_OK;
}

int card_profile_collect(float* ms_host, int32_t* n_host) {
    if (!ms_host || !n_host) return CARD_EINVAL;
    Profile& p = prof();
    std::lock_guard<std::mutex> g(p.mu);
    const int n = p.used;
    p.on = false;
    p.used = 0;
    for (int i = 0; i < n; ++i) {
        if (hipEventSynchronize(p.stop[i]) != hipSuccess) return CARD_EDEVICE;
        if (hipEventElapsedTime(&ms_host[i], p.start[i], p.stop[i]) != hipSuccess) return CARD_EDEVICE;
    }
    *n_host = n;
    return CARD_OK;
}

int card_profile_disable(void) {
    Profile& p = prof();
    std::lock_guard<std::mutex> g(p.mu);
    p.on = false;
    p.used = 0;
    int st = CARD_OK;
    for (hipEvent_t e : p.start)
        if (hipEventDestroy(e) != hipSuccess) st = CARD_EDEVICE;
    for (hipEvent_t e : p.stop)
        if (hipEventDestroy(e) != hipSuccess) st = CARD_EDEVICE;
    p.start.clear();
    p.stop.clear();
    return st;
}

int card_workspace_init(const card_model_cfg* cfg, void* workspace_dev, void* stream) {
    if (!workspace_dev) return CARD_EINVAL;
    const Layout L = make_layout(cfg);
    if (!L.ok) return CARD_EINVAL;
    char* ws = static_cast<char*>(workspace_dev);
    if (reinterpret_cast<uintptr_t>(ws) % 16 || L.ws_bytes % 16) return CARD_EINVAL;
    hipLaunchKernelGGL(k_ws_init, dim3(1024), dim3(256), 0, as_stream(stream), reinterpret_cast<uint4v*>(ws),
                       L.ws_bytes / 16, reinterpret_cast<uint32_t*>(ws + L.m_bar_off) + kBarMagic);
    return launch_status();
}

int card_kv_gather(const card_model_cfg* cfg, const card_kv* kv, int32_t layer, int32_t first_slot, int32_t count,
                   float* k_out_dev, float* v_out_dev, void* stream) {
    if (!cfg_valid(cfg) || !kv || !kv->k_pages || !kv->v_pages || !kv->block_table || !k_out_dev || !v_out_dev)
        return CARD_EINVAL;
    if (layer < 0 || layer >= cfg->n_layers || count <= 0 || first_slot < 0) return CARD_ERANGE;
    if (int64_t(first_slot) + count > cfg->max_ctx) return CARD_ECAPACITY;
    const size_t pool_layer_elems = size_t(kv->n_pages) * cfg->n_kv_heads * 16 * cfg->head_dim;
    GatherArgs a = {};
    a.kpool = static_cast<const __bf16*>(kv->k_pages) + size_t(layer) * pool_layer_elems;
    a.vpool = static_cast<const __bf16*>(kv->v_pages) + size_t(layer) * pool_layer_elems;
    a.block_table = kv->block_table;
    a.first = first_slot;
    a.count = count;
    a.n_kv_heads = cfg->n_kv_heads;
    a.head_dim = cfg->head_dim;
    a.k_out = k_out_dev;
    a.v_out = v_out_dev;
    const int64_t total = int64_t(count) * cfg->n_kv_heads * cfg->head_dim;
    hipLaunchKernelGGL(k_kv_gather, dim3(uint32_t((total + 255) / 256)), dim3(256), 0, as_stream(stream), a);
    return launch_status();
}

}  // extern "C"
