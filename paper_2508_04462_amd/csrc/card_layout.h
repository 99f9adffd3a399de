// Host-side description of where everything lives: the packed weight blob, the workspace,
// of the persistent verify kernel.  Plain structs, passed to kernels by value.
#pragma once
#include <stddef.h>
#include <stdint.h>

#include "card.h"

namespace card {

constexpr int kTileN = 16;     // rows of one matrix-instruction tile (output features)
constexpr int kTileK = 32;     // contraction depth of one bf16 16x16x32 matrix instruction
constexpr int kMaxR = 32;
constexpr int kKvBlock = 16;
// tiles a workgroup accumulates side by side (batch width) per kind of matrix
constexpr int kNbQkv = 2, kNbOne = 1, kNbWide = 8;
constexpr int kFlagCopies = 32;  // copies of the barrier flags (256 words each): pollers spread over them
constexpr uint32_t kStampMagic = 0x43415244u;  // "CARD"
constexpr uint32_t kWsMagic = 0x57534b31u;     // workspace control words initialised ("WSK1"), word kBarMagic
// words of the barrier block: [1] exit counter, [2] error flag, [3] barrier epoch, [4] magic
constexpr int kBarExit = 1, kBarError = 2, kBarEpoch = 3, kBarMagic = 4;

#ifdef __HIPCC__
#define CARD_HD __host__ __device__
#else
#define CARD_HD
#endif

constexpr int kStreamWaves = 4;  // wavefront pairs of a workgroup: they cut the contraction four ways

// One matrix as Nt n-tiles x Ks k-steps of 1 KiB fragments [64 lanes][8 bf16]: lane l of
// fragment (t, s) holds row 16t + l%16, columns 32s + 8*(l/16) .. +8; rows / columns beyond
// N / K are zero.  Fragments are stored in STREAM ORDER, the order in which the verify kernel
// consumes them on a grid of nwg workgroups: tile t belongs to position p = t % nwg of the grid
// (its j-th tile, j = t / nwg), k-step s to the wavefront pair w with w*Ks/4 <= s < (w+1)*Ks/4.
// Memory holds position after position, inside a position pair after pair, and inside a pair
// the tiles NB at a time ("batch"): batch, then k-step, then tile of the batch.  Every wavefront
// pair therefore reads ONE contiguous run per matrix.
struct MatDesc {
    size_t off;  // byte offset inside the packed blob (layer matrices: relative to the layer base)
    int32_t N, K, Nt, Ks, NB;
    size_t bytes() const { return size_t(Nt) * Ks * 1024; }
};

// Tiles of grid position p, the k-steps [s0, s1) of pair w, and the index of the pair's first
// fragment in the matrix.
struct StreamRun {
    int32_t cnt, s0, s1;
    int64_t first;
};
CARD_HD inline StreamRun stream_run(int32_t Nt, int32_t Ks, int32_t nwg, int32_t p, int32_t w) {
    StreamRun r;
    const int32_t full = Nt / nwg, rem = Nt % nwg;
    r.cnt = full + (p < rem ? 1 : 0);
    r.s0 = (w * Ks) / kStreamWaves;
    r.s1 = ((w + 1) * Ks) / kStreamWaves;
    r.first = (int64_t(full) * p + (p < rem ? p : rem)) * Ks + int64_t(r.cnt) * r.s0;
    return r;
}
// Index of fragment (tile t, k-step s) in stream order.
CARD_HD inline int64_t stream_frag_index(int32_t Nt, int32_t Ks, int32_t NB, int32_t nwg, int32_t t, int32_t s) {
    const int32_t p = t % nwg, j = t / nwg;
    int32_t w = 0;
    while (w + 1 < kStreamWaves && s >= ((w + 1) * Ks) / kStreamWaves) ++w;
    const StreamRun r = stream_run(Nt, Ks, nwg, p, w);
    const int32_t b = j / NB, i = j % NB;
    const int32_t nv = r.cnt - b * NB < NB ? r.cnt - b * NB : NB;
    return r.first + int64_t(b) * NB * (r.s1 - r.s0) + int64_t(s - r.s0) * nv + i;
}

// ---- the coded copy of the matrices (CARD_CODED) -----------------------------------------------
// Which tensors the copy holds stands in the stamp block, which every blob has: from word kCopyWord on a byte per layer, bit i for
// tensor i of CodeTensor, and behind the last layer one for the vocabulary head (bit 0).  Packing a tensor sets its bit or, without a copy, clears
// it, whatever the memory held before; so once everything has been packed the bits are right.  Steps on the copy need all of them.
constexpr int kCopyWord = 4, kCopySlots = (256 - kCopyWord) * 4;  // (the block has 256 words)
CARD_HD inline int32_t copy_words(int32_t n_layers) { return n_layers / 4 + 1; }
CARD_HD inline uint32_t copy_bits_needed(int32_t n_layers, int32_t word) {
    uint32_t need = 0;
    for (int32_t b = 0; b < 4; ++b) {
        const int32_t slot = word * 4 + b;
        need |= (slot < n_layers ? 0x7fu : slot == n_layers ? 1u : 0u) << (8 * b);
    }
    return need;
}
// The verify kernel's steps are bound by the bytes of the weights, and of a bf16 weight's sixteen bits four are nearly always
// known: weights with a bell-shaped distribution spread over few exponents.  A coded matrix holds its fragments (in stream order, n = Nt * Ks of
// them) in three planes:
//   low  512 B at f * 512:                bits 0-7 of the lane's eight weights
//   high 256 B at n * 512 + f * 256:      four bits each: the sign, and the low three bits c of bits 8-14 less `base`
//   rest 256 B at n * 768 + f * 256:      four bits each: what is left of bits 8-14, zero for the weights whose
//                                         exponent is one of the sixteen from 2 * base on
// The base is that of the tensor, chosen when it is packed as the one that leaves out fewest weights.  The kernel reads a
// fragment's rest only where a bit per fragment says that it holds something: 12 bits per weight instead of 16,
// lossless, for any bit pattern.  (6 % of the fragments have a rest if the weights are normally distributed.)
struct CodedDesc {
    size_t off;  // of the planes, from the coded layer's base (vocabulary head: from the copy's)
    size_t fl;   // of the bits that say which fragments have a rest, in stream order (stream_flag)
    size_t fl2;  // gate/up: those of the up rows (`fl`: of the gate rows); down-projection: those in grouped order (grouped_flag)
    int32_t fl_run, fl2_run;  // words of 64 bits per run (filled in for the grid in use)
};
// The bits in stream order: every run (pair w of position p: number 4 p + w) has its own words, every batch of a run begins with a word.
// As the verify kernel's down-projection for more than eight rows takes them (four positions share their tiles: position 4 g + q takes
// quarter q of K of all four, pair w the w-th quarter of that, the four tiles of a k-step in turn): "grouped".
struct FlagPlace {
    int64_t word;
    int32_t bit;
};
CARD_HD inline int32_t flag_words(int32_t bits) { return (bits + 63) / 64; }
CARD_HD inline int32_t flag_run_words(int32_t Nt, int32_t Ks, int32_t NB, int32_t nwg) {
    const int32_t cnt = (Nt + nwg - 1) / nwg, wide = cnt < NB ? cnt : NB;
    return (cnt + NB - 1) / NB * flag_words(wide * ((Ks + kStreamWaves - 1) / kStreamWaves));
}
CARD_HD inline int32_t grouped_run_words(int32_t Nt, int32_t Ks, int32_t nwg) {
    const int32_t quarter = (Ks + 3) / 4, steps = (quarter + 3) / 4;
    return (Nt + nwg - 1) / nwg * flag_words(4 * steps);
}
CARD_HD inline FlagPlace stream_flag(int32_t Nt, int32_t Ks, int32_t NB, int32_t nwg, int32_t t, int32_t s) {
    const int32_t p = t % nwg, j = t / nwg;
    int32_t w = 0;
    while (w + 1 < kStreamWaves && s >= ((w + 1) * Ks) / kStreamWaves) ++w;
    const StreamRun r = stream_run(Nt, Ks, nwg, p, w);
    const int32_t b = j / NB, steps = r.s1 - r.s0, nv = r.cnt - b * NB < NB ? r.cnt - b * NB : NB;
    const int32_t at = (s - r.s0) * nv + j % NB;
    return {int64_t(p * kStreamWaves + w) * flag_run_words(Nt, Ks, NB, nwg) + b * flag_words(NB * steps) + at / 64, at % 64};
}
CARD_HD inline FlagPlace grouped_flag(int32_t Nt, int32_t Ks, int32_t nwg, int32_t t, int32_t s) {
    const int32_t p = t % nwg, j = t / nwg;
    int32_t q = 0, w = 0;
    while (q < 3 && s >= ((q + 1) * Ks) / 4) ++q;
    const int32_t q0 = (q * Ks) / 4, len = ((q + 1) * Ks) / 4 - q0;
    while (w < 3 && s >= q0 + ((w + 1) * len) / 4) ++w;
    const int32_t s0 = q0 + (w * len) / 4, steps = q0 + ((w + 1) * len) / 4 - s0;
    const int32_t at = (s - s0) * 4 + (p & 3);
    return {int64_t(((p & ~3) + q) * kStreamWaves + w) * grouped_run_words(Nt, Ks, nwg) + j * flag_words(4 * steps) + at / 64, at % 64};
}
// Room for them on any grid of up to 256 workgroups.  (The kernel reads a word ahead.)
inline size_t flag_bytes(int32_t Nt, int32_t Ks, int32_t NB) {
    const size_t steps = (Ks + kStreamWaves - 1) / kStreamWaves;
    return (4 * ((size_t(Nt) + 256 * size_t(NB)) * steps / 64 + size_t(Nt) / NB + 520) + 8) * 8;
}
inline size_t grouped_bytes(int32_t Nt, int32_t Ks) { return (4 * (size_t(Nt) + 260) * ((size_t(Ks) + 15) / 16 / 16 + 2) + 8) * 8; }
// Words of a layer's `code` block: a base per tensor (four times in its bytes), then 128 counters per tensor (packing only).
enum CodeTensor { CT_Q = 0, CT_K = 1, CT_V = 2, CT_O = 3, CT_G = 4, CT_U = 5, CT_D = 6 };
constexpr int kCodeCounts = 64;  // first counter (tensor i: 128 i behind it)

struct Layout {
    bool ok;
    // packed weights
    size_t embed_off, lm_off, g_final_off, stamp_off, layer0_off, layer_stride, weight_bytes;
    MatDesc qkv, wo, gu, wd, lm;  // layer matrices relative to the layer base; lm absolute
    size_t g_attn_off, g_ffn_off; // relative to the layer base
    // coded copy: where it begins in the blob (behind everything else), from there: the vocabulary head's planes and code block, the layers
    CodedDesc c_qkv, c_wo, c_gu, c_wd, c_lm;
    size_t coded_off, c_lm_code_off, c_layer0_off, c_layer_stride, c_code_off;  // c_code_off: in a layer
    size_t ws_bytes;
    // workspace of the persistent kernel (byte offsets) and strides in elements
    size_t m_xres_off, m_xfrag_off, m_ss_off, m_qfrag_off, m_attfrag_off, m_actfrag_off, m_apart_off, m_bar_off,
        m_acount_off, m_flags_off, m_best_off, m_rope_off, m_topk_off, m_lse_off, m_out_off, m_dpart_off,
        m_dcount_off;
    size_t xfrag_stride, attfrag_stride, actfrag_stride, qfrag_stride;
    int32_t m_attn_max_splits;
};

inline int32_t ceil_div(int64_t a, int64_t b) { return int32_t((a + b - 1) / b); }
inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

inline MatDesc make_mat(size_t off, int32_t N, int32_t K, int32_t NB) {
    MatDesc m;
    m.off = off;
    m.N = N;
    m.K = K;
    m.NB = NB;
    m.Nt = ceil_div(N, kTileN);
    m.Ks = ceil_div(K, kTileK);
    return m;
}

inline int32_t cfg_grid(const card_model_cfg* c) { return c->grid_wgs & ~CARD_CODED; }
inline bool cfg_coded(const card_model_cfg* c) { return (c->grid_wgs & CARD_CODED) != 0; }

inline bool cfg_valid(const card_model_cfg* c) {
    if (!c) return false;
    if (c->n_layers <= 0 || c->d_model <= 0 || c->n_q_heads <= 0 || c->n_kv_heads <= 0 || c->d_ffn <= 0 ||
        c->vocab <= 1)
        return false;
    if (c->head_dim != 64 && c->head_dim != 128) return false;
    if (c->d_model % 64 || c->d_ffn % 8) return false;
    if (c->n_q_heads % c->n_kv_heads) return false;
    if (c->kv_block != kKvBlock) return false;
    if (c->max_ctx <= 0 || c->max_ctx % kKvBlock) return false;
    if (c->max_r < 1 || c->max_r > kMaxR) return false;
    if (!(c->rope_theta > 0.f) || !(c->rms_eps >= 0.f)) return false;
    if (cfg_grid(c) < 0 || cfg_grid(c) > 256) return false;
    if (cfg_coded(c) && c->n_layers >= kCopySlots) return false;
    return true;
}

inline Layout make_layout(const card_model_cfg* c) {
    Layout L = {};
    if (!cfg_valid(c)) return L;
    const int32_t d = c->d_model, h = c->head_dim, qd = c->n_q_heads * h, kvd = c->n_kv_heads * h;
    size_t off = 0;
    L.embed_off = off;
    off = align_up(off + size_t(c->vocab) * d * 2, 1024);
    L.lm = make_mat(off, c->vocab, d, kNbWide);
    L.lm_off = off;
    off = align_up(off + L.lm.bytes(), 1024);
    L.g_final_off = off;
    off = align_up(off + size_t(d) * 4, 1024);
    L.stamp_off = off;  // {magic, grid size the stream order was laid out for}; from word kCopyWord on: what the coded copy holds
    off += 1024;
    L.layer0_off = off;
    size_t lo = 0;
    L.qkv = make_mat(lo, qd + 2 * kvd, d, kNbQkv);
    lo += L.qkv.bytes();
    L.wo = make_mat(lo, d, qd, kNbOne);
    lo += L.wo.bytes();
    L.gu = make_mat(lo, 2 * c->d_ffn, d, kNbWide);
    lo += L.gu.bytes();
    L.wd = make_mat(lo, d, c->d_ffn, kNbOne);
    lo += L.wd.bytes();
    L.g_attn_off = lo;
    lo = align_up(lo + size_t(d) * 4, 1024);
    L.g_ffn_off = lo;
    lo = align_up(lo + size_t(d) * 4, 1024);
    L.layer_stride = lo;
    L.weight_bytes = L.layer0_off + size_t(c->n_layers) * L.layer_stride;
    L.coded_off = align_up(L.weight_bytes, 1024);
    {
        size_t at = 0;
        auto coded = [&](const MatDesc& m, int sets, bool grouped) {
            CodedDesc c = {};
            c.off = at;
            at += m.bytes();
            c.fl = at;
            at = align_up(at + flag_bytes(m.Nt, m.Ks, m.NB), 1024);
            c.fl2 = at;
            if (grouped) at = align_up(at + grouped_bytes(m.Nt, m.Ks), 1024);
            else if (sets > 1) at = align_up(at + flag_bytes(m.Nt, m.Ks, m.NB), 1024);
            return c;
        };
        L.c_lm = coded(L.lm, 1, false);
        L.c_lm_code_off = at;
        L.c_layer0_off = at + 1024;
        at = 0;
        L.c_qkv = coded(L.qkv, 1, false);
        L.c_wo = coded(L.wo, 1, false);
        L.c_gu = coded(L.gu, 2, false);
        L.c_wd = coded(L.wd, 1, true);
        L.c_code_off = at;
        at = align_up(at + (kCodeCounts + 7 * 128) * 4, 1024);
        L.c_layer_stride = at;
        if (cfg_coded(c)) L.weight_bytes = L.coded_off + L.c_layer0_off + size_t(c->n_layers) * L.c_layer_stride;
    }
    // the kernel addresses a matrix with 32-bit byte offsets
    constexpr size_t k4G = size_t(1) << 32;
    if (L.qkv.bytes() >= k4G || L.wo.bytes() >= k4G || L.gu.bytes() >= k4G || L.wd.bytes() >= k4G || L.lm.bytes() >= k4G)
        return L;

    // workspace
    size_t w = 0;
    auto take = [&](size_t bytes) {
        size_t at = w;
        w = align_up(w + bytes, 256);
        return at;
    };
    const int32_t G = c->n_q_heads / c->n_kv_heads;
    // persistent kernel: one copy of every hand-over buffer per layer and phase
    auto frag_elems = [](int32_t K) { return size_t(ceil_div(K, kTileK)) * 4 * kMaxR * 16; };
    const int32_t versions = 2 * c->n_layers + 1;
    L.xfrag_stride = frag_elems(d);
    L.attfrag_stride = frag_elems(qd);
    L.actfrag_stride = frag_elems(c->d_ffn);
    L.qfrag_stride = size_t(c->n_q_heads) * kMaxR * h * 2;
    L.m_xres_off = take(size_t(versions) * kMaxR * d * 4);
    L.m_xfrag_off = take(size_t(versions) * L.xfrag_stride * 2);
    L.m_ss_off = take(size_t(versions) * (d / 16) * kMaxR * 4);
    L.m_qfrag_off = take(size_t(c->n_layers) * L.qfrag_stride * 2);
    L.m_attfrag_off = take(size_t(c->n_layers) * L.attfrag_stride * 2);
    L.m_actfrag_off = take(size_t(c->n_layers) * L.actfrag_stride * 2);
    L.m_attn_max_splits = 32;
    L.m_apart_off = take(size_t(c->n_kv_heads) * (2 * G) * L.m_attn_max_splits * 16 * (h + 2) * 4);
    L.m_bar_off = take(256);
    L.m_flags_off = take(size_t(kFlagCopies) * 1024);
    L.m_acount_off = take(size_t(c->n_kv_heads) * (2 * G) * 4);
    L.m_best_off = take(size_t(kMaxR) * 8);
    L.m_rope_off = take(size_t(kMaxR) * h * 4);
    L.m_topk_off = take(size_t(256) * kMaxR * 16 * 8);  // per workgroup and row: up to sixteen best keys
    L.m_lse_off = take(size_t(256) * kMaxR * 2 * 4);    // per workgroup and row: (max, sum of exp)
    L.m_out_off = take(64);                             // where a draft-side call parks the verify result
    // down-projection at r > 8: the four workgroups of a group each hold a quarter of K of the
    // group's tiles; per tile four partial blocks of 16 x 32 fp32, and one arrival counter per
    // four tiles
    L.m_dpart_off = take(size_t(L.wd.Nt) * kStreamWaves * 16 * kMaxR * 4);
    L.m_dcount_off = take(size_t(ceil_div(L.wd.Nt, 4)) * 4);
    L.ws_bytes = w;
    L.ok = true;
    return L;
}

}  // namespace card
