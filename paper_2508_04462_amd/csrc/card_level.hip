// A wide level of the draft's tree in one pass: up to 128 rows as a sequence of ordinary kernels.
//
// Why not calls of the verify kernel: they carry at most 32 rows, so a level of 100 nodes streams every
// weight four times, and each of the four crosses five grid barriers per layer.  Here the weights are
// streamed once, and a layer is eight kernels of 4-20 us.
//
// The results are those of the calls (card_draft_level_piece) bit for bit: every sum is taken in the order in which
// the verify kernel's wavefronts take it.  A product's contraction is four chains of k-steps (its four
// wavefronts' shares of K), added in order; the grouped down-projection's is four times four; a row's keys are walked in
// the same cuts by the same four wavefronts; calls of at most eight rows ("packed halves") add the products of the low activation
// halves behind those of the high ones instead of in between.  So which calls a level would have been cut into decides the
// order of some sums: the host describes the rows as row tiles that never cross a call's end (LvTile).
//
// Weights and activations as in the prompt pass (card_prompt.hip).  A tile of packed halves holds its (at most eight)
// rows' high halves in columns 0-7 and their low halves in columns 8-15 of the high fragment, zeros in the low one: the
// products need not know.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "card_prompt.hip"

namespace card {

constexpr int kLvTiles = 8;  // row tiles of a pass
constexpr int kLvWaves = 8;  // wavefronts per workgroup of the product kernel

// Rows [row0, row0 + n) of the level, n <= 16, all of one call.
struct LvTile {
    int32_t row0, n;
    int32_t pk;                    // the call is one of at most eight rows
    int32_t wide;                  // the call has two row tiles: eight lanes share a row's columns in the vocabulary phase, not sixteen
    int32_t pages, per_cut, cuts;  // the call's page list and its cuts
    int32_t subs, task0, count0;   // attention: tiles of 16 (row, head) pairs, first task, first arrival counter
};

struct LvArgs {
    int32_t n_tiles, d, Ks;
    LvTile t[kLvTiles];
    // residual
    float* x;            // [n_tiles * 16][d]
    __bf16* xf;
    const float* gain;
    float* ss;           // [n_tiles * 16][d / 16]
    const float* part;   // [4][Nt][n_tiles][64][4]
    int32_t Nt;
    // embedding
    const __bf16* embed;
    const int32_t* tokens;
    int32_t V, n_counts;
    uint32_t* counts;
    // QKV
    int32_t qd, kvd, h, Hkv, G, first_slot, level_first, level_end, last_row;
    float inv_d, eps, inv_sqrt_h;
    const float* rope;   // [n_tiles * 16][h / 2] cos, then the same of sin
    __bf16* q;           // [Hkv][n_tiles * 16 * G][h / 8][16]
    __bf16* kpool;
    __bf16* vpool;
    const int32_t* block_table;
    // attention
    const uint32_t* mask;
    int32_t mask_words, mask_base;
    float* apart;        // [tasks][16 * (h + 2)]
    __bf16* att;
    int32_t Ks_att;
};

// High and low halves h, l of four (eight) consecutive values of row m of tile mt at column k, in place.
template <int W>
__device__ __forceinline__ void lv_put(__bf16* x, int Ks, int mt, bool pk, int m, int k, const __bf16 (&h)[W], const __bf16 (&l)[W]) {
    static_assert(W == 4 || W == 8, "8 or 16 bytes");
    typedef __attribute__((ext_vector_type(W / 2))) unsigned int word;
    word hi, lo;
#pragma unroll
    for (int e = 0; e < W; e += 2) {
        hi[e / 2] = pack_bf16(h[e], h[e + 1]);
        lo[e / 2] = pack_bf16(l[e], l[e + 1]);
    }
    __bf16* p = x + px_frag(Ks, k >> 5, mt) + (((k >> 3) & 3) * 16 + m) * 8 + (k & 7);
    *reinterpret_cast<word*>(p) = hi;
    if (!pk) {
        *reinterpret_cast<word*>(p + 512) = lo;
    } else {
        *reinterpret_cast<word*>(p + 64) = lo;
        *reinterpret_cast<word*>(p + 512) = word(0u);
        *reinterpret_cast<word*>(p + 576) = word(0u);
    }
}
// Values v.
template <int W>
__device__ __forceinline__ void lv_store(__bf16* x, int Ks, int mt, bool pk, int m, int k, const float (&v)[W]) {
    __bf16 h[W], l[W];
#pragma unroll
    for (int e = 0; e < W; ++e) split_bf16(v[e], h[e], l[e]);
    lv_put<W>(x, Ks, mt, pk, m, k, h, l);
}
// Halves of f * g: the low one is rounded from the exact product less the high one, which is what the compiler makes of
// the product and the split in the verify kernel.
__device__ __forceinline__ void split_product(float f, float g, __bf16& hi, __bf16& lo) {
    hi = static_cast<__bf16>(f * g);
    lo = static_cast<__bf16>(fmaf(f, g, -static_cast<float>(hi)));
}

// RMSNorm scale of a row by eight neighbouring lanes, in the order of the verify kernel
__device__ __forceinline__ float lv_row_scale(const float* ss, int n_part, int sub, float inv_d, float eps) {
    float sq = 0.f;
    for (int g = sub; g < n_part >> 2; g += 8) {
        const floatx4 v = *reinterpret_cast<const floatx4*>(ss + 4 * g);
        sq += (v[0] + v[1]) + (v[2] + v[3]);
    }
    sq = group_sum<8>(sq);
    return 1.0f / sqrtf(sq * inv_d + eps);
}

// ---- product ------------------------------------------------------------------------------------
struct LvGemmArgs {
    const char* w;
    uint32_t bytes;
    int32_t Nt, Ks, NB, nwg;  // tiles, k-steps, batch width and grid of the stream order
    const __bf16* x;
    int32_t n_tiles, nblk, mblk;
    uint32_t pk_tiles;        // bit mt: packed halves
    int32_t grouped;          // the verify kernel's down-projection for more than eight rows
    float* part;              // LV_PART: sums over the quarters of K
    const float* ss;
    int32_t n_part, Ks_out;
    float inv_d, eps;
    __bf16* act;
    float* logits;            // [n_tiles * 16][ldl]
    int32_t ldl;
};

enum LvEpi { LV_PART = 0, LV_SWIGLU = 1, LV_LOGITS = 2 };

// As k_prompt_gemm (weights of a wavefront's N tiles straight into registers, MT row tiles of activations through LDS
// for all eight wavefronts), but K is walked in the verify kernel's chains: at the end of each the accumulators are
// added to the running sums and start again from zero.  LV_PART: a workgroup takes one quarter of K (one chain, or the four of
// the grouped down-projection), the next kernel adds the quarters; narrow matrices then still fill the chip.
// The others walk all of K.
// Bound by the bytes that enter a compute unit (57 GB/s of weights and activations together): 0.15 us per k-step for eight weight tiles
// and 0.07 for two row tiles.  1B shape, 100 rows, us: QKV 10.4 (N = 2, MT = 2; four wavefronts on four row tiles 11.8), O and down 12.9 on
// average (N = 1, MT = 2; 13.9), gate/up 27.9 (N = 1, MT = 4; 28.6), vocabulary 131 (N = 2, MT = 8; 174).
template <int EPI, int N, int MT>
__global__ __launch_bounds__(kLvWaves * 64, 2) void k_level_gemm(LvGemmArgs a) {
    // k-steps between two barriers (a "turn"), turns in the rings of registers, weights in the ring
    constexpr int KB = MT > 4 ? 2 : 4, UT = 2, DA = KB * UT;
    constexpr int XF = KB * 2 * MT, XW = XF / kLvWaves;
    static_assert(XF % kLvWaves == 0 && UT == 2, "fragments dealt evenly; turn u reads LDS buffer u & 1");
    constexpr bool FULL = EPI != LV_PART;
    __shared__ uint4v xs[2][XF][64];
    __shared__ __align__(16) float scale[FULL ? MT * 16 : 4];
    __shared__ floatx4 pkq[FULL ? kLvWaves : 1][4][N][64];  // a packed tile's four quarters
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int splits = FULL ? 1 : 4;
    // a compute die gets a contiguous range of the blocks in (weight block, quarter, row block) order
    const int total = a.nblk * splits * a.mblk, per = (total + 7) >> 3;
    const int L = int(blockIdx.x & 7) * per + int(blockIdx.x >> 3);
    if (int(blockIdx.x >> 3) >= per || L >= total) return;
    const int mb = L % a.mblk, sp = (L / a.mblk) % splits, nb = L / (a.mblk * splits);
    const int v0 = (nb * kLvWaves + wave) * N, mt0 = mb * MT;
    const uint32_t pk = (a.pk_tiles >> mt0) & ((1u << MT) - 1u);
    const int q0 = (sp * a.Ks) / kStreamWaves, qlen = ((sp + 1) * a.Ks) / kStreamWaves - q0;
    const int n_chains = FULL ? kStreamWaves : (a.grouped ? 4 : 1);
    auto chain = [&](int i, int& b, int& e) {
        if constexpr (FULL) {
            b = (i * a.Ks) / kStreamWaves;
            e = ((i + 1) * a.Ks) / kStreamWaves;
        } else {
            b = q0 + (i * qlen) / n_chains;
            e = q0 + ((i + 1) * qlen) / n_chains;
        }
    };
    // the k-steps in order, every chain filled up to whole turns with steps that read zeros
    struct Cursor {
        int i, s, e, left;
    };
    auto next = [&](Cursor& c) {  // at a chain's end: the next one that is not empty; true if c.s jumped
        bool moved = false;
        while (c.left == 0 && c.i + 1 < n_chains) {
            int b, e;
            chain(++c.i, b, e);
            c.s = b;
            c.e = e;
            c.left = (e - b + KB - 1) / KB * KB;
            moved = true;
        }
        return moved;
    };

    const __amdgpu_buffer_rsrc_t wr = make_rsrc(a.w, a.bytes);
    const PgemmArgs order = {a.w, a.bytes, a.Nt, a.Ks, a.NB, a.nwg};
    PgTile tl[N];
#pragma unroll
    for (int i = 0; i < N; ++i) tl[i].init(order, min(v0 + i, a.Nt - 1));
    uint32_t woff[N];
    Cursor ca = {-1, 0, 0, 0}, cb = {-1, 0, 0, 0};
    // (`first`: the k-step is the first of a turn; chains begin with turns)
    auto load_a = [&](bf16x8 (&r)[N], bool first) {
        if (first && ca.left == 0 && next(ca)) {
            int w = 0;
            while (w + 1 < kStreamWaves && ca.s >= ((w + 1) * a.Ks) / kStreamWaves) ++w;
#pragma unroll
            for (int i = 0; i < N; ++i) woff[i] = tl[i].at(ca.s, (w * a.Ks) / kStreamWaves, ((w + 1) * a.Ks) / kStreamWaves);
        }
        int voff = ca.left > 0 && ca.s < ca.e ? lane * 16 : kOutOfRange;
        asm volatile("" : "+v"(voff));  // (one load here, not one per way to this offset: the second would wait for the first)
#pragma unroll
        for (int i = 0; i < N; ++i) {
            r[i] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(wr, voff, int(woff[i]), 0));
            woff[i] += uint32_t(tl[i].nv) << 10;
        }
        ++ca.s;
        ca.left -= ca.left > 0 ? 1 : 0;
    };
    // fragment f of a turn: k-step f / (2 MT), row tile f / 2 % MT, half f % 2; the wavefront brings XW consecutive ones
    const __amdgpu_buffer_rsrc_t xr = make_rsrc(a.x, uint32_t(a.Ks) * uint32_t((a.n_tiles + kPgTiles - 1) / kPgTiles * kPgTiles) * 2048u);
    uint32_t xoff[XW];
    int xstep[XW];
#pragma unroll
    for (int q = 0; q < XW; ++q) {
        const int f = wave * XW + q, mt = mt0 + f / 2 % MT;
        xstep[q] = mt < a.n_tiles ? f / (2 * MT) : 1 << 24;  // (no such row tile: no such k-step)
        xoff[q] = uint32_t(px_frag(a.Ks, f / (2 * MT), mt)) * 2u + uint32_t(f & 1) * 1024u;
    }
    auto load_b = [&](uint4v (&r)[XW]) {
        if (cb.left == 0) next(cb);
#pragma unroll
        for (int q = 0; q < XW; ++q) {
            int voff = cb.left > 0 && cb.s + xstep[q] < cb.e ? lane * 16 : kOutOfRange;
            asm volatile("" : "+v"(voff));
            r[q] = __builtin_amdgcn_raw_buffer_load_b128(xr, voff, int(xoff[q] + uint32_t(cb.s) * (kPgTiles * 2048u)), 0);
        }
        cb.s += KB;
        cb.left -= cb.left > 0 ? KB : 0;
    };
    auto store_b = [&](int buf, const uint4v (&r)[XW]) {
#pragma unroll
        for (int q = 0; q < XW; ++q) xs[buf][wave * XW + q][lane] = r[q];
    };
    auto sync = [&]() {  // LDS writes done, everybody here; loads stay in flight
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(kWaitLds);
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };

    floatx4 acc[N][MT], tot[N][MT];
#pragma unroll
    for (int i = 0; i < N; ++i)
#pragma unroll
        for (int j = 0; j < MT; ++j) acc[i][j] = tot[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
    bf16x8 wa[DA][N];
    uint4v xb[UT][XW];
    load_b(xb[0]);
#pragma unroll
    for (int q = 0; q + 1 < DA; ++q) load_a(wa[q], q % KB == 0);
    store_b(0, xb[0]);
#pragma unroll
    for (int q = 1; q <= UT; ++q) load_b(xb[q % UT]);
    sync();
    int c = -1, turns = 0, total_turns = 0;  // the chain that is being multiplied, what is left of it
    for (int i = 0; i < n_chains; ++i) {
        int b, e;
        chain(i, b, e);
        total_turns += (e - b + KB - 1) / KB;
    }
    auto next_chain = [&]() {
        while (turns == 0 && c + 1 < n_chains) {
            int b, e;
            chain(++c, b, e);
            turns = (e - b + KB - 1) / KB;
            if (FULL && turns == 0) {
#pragma unroll
                for (int i = 0; i < N; ++i) pkq[wave][c][i][lane] = floatx4{0.f, 0.f, 0.f, 0.f};
            }
        }
    };
    next_chain();
    for (int t = 0; t < total_turns; t += UT) {  // (a turn behind the last one multiplies zeros)
#pragma unroll
        for (int u = 0; u < UT; ++u) {
            px_half_turn<N, MT, KB>(xs[u & 1], lane, acc, [&](int k) -> const bf16x8(&)[N] { return wa[u * KB + k]; }, [&](int k) {
                load_a(wa[(u * KB + k + DA - 1) % DA], (k + DA - 1) % KB == 0);
            });
            store_b((u + 1) & 1, xb[(u + 1) % UT]);
            load_b(xb[(u + 1) % UT]);
            sync();
            // the chain's end.  (A packed tile's quarter is one chain in the grouped down-projection too.)
            if (turns > 0 && --turns == 0) {
#pragma unroll
                for (int j = 0; j < MT; ++j) {
                    const bool packed = (pk >> j) & 1u;
                    if (FULL || !packed) {
#pragma unroll
                        for (int i = 0; i < N; ++i) {
                            if (FULL && packed) pkq[wave][c][i][lane] = acc[i][j];
                            tot[i][j] += acc[i][j];
                            acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
                        }
                    }
                }
                next_chain();
            }
        }
    }

    if constexpr (EPI == LV_PART) {
#pragma unroll
        for (int i = 0; i < N; ++i) {
            if (v0 + i >= a.Nt) continue;
            float* p = a.part + ((size_t(sp) * a.Nt + tl[i].t) * a.n_tiles + mt0) * 256 + lane * 4;
#pragma unroll
            for (int j = 0; j < MT; ++j)
                if (mt0 + j < a.n_tiles) *reinterpret_cast<floatx4*>(p + j * 256) = (pk >> j) & 1u ? acc[i][j] : tot[i][j];
        }
    } else {
        for (int e = tid; e < MT * 16 * 8; e += kLvWaves * 64) {
            const int row = mt0 * 16 + (e >> 3);
            if (mt0 + (e >> 7) < a.n_tiles) {
                const float sc = lv_row_scale(a.ss + size_t(row) * a.n_part, a.n_part, e & 7, a.inv_d, a.eps);
                if ((e & 7) == 0) scale[e >> 3] = sc;
            }
        }
        sync();
        const int m = lane & 15;
#pragma unroll
        for (int j = 0; j < MT; ++j) {
            if (mt0 + j >= a.n_tiles) continue;
            const bool packed = (pk >> j) & 1u;
            if (packed) {  // the low halves' products, quarter by quarter
#pragma unroll
                for (int i = 0; i < N; ++i)
#pragma unroll
                    for (int q = 0; q < 4; ++q) tot[i][j] += pkq[wave][q][i][min(lane + 8, 63)];
            }
            const float sc = scale[j * 16 + m];
            if constexpr (EPI == LV_SWIGLU) {
                // (one tile: the lanes from 32 on get what the others have)
#pragma unroll
                for (int i = 0; i < N; i += 2) {
                    const int i1 = N > 1 ? i + 1 : i;
                    float v[4];
                    const bool low = lane < 32;
                    px_swiglu_values(lane, sc, tot[i][j], tot[i1][j], v);
                    const int t = low ? tl[i].t : tl[i1].t;
                    if (v0 + (low ? i : i + 1) >= (N > 1 || low ? a.Nt : 0) || (packed && m >= 8)) continue;
                    const int k = t * 8 + ((lane >> 4) & 1) * 4;
                    lv_store<4>(a.act, a.Ks_out, mt0 + j, packed, m, k, v);
                    const float z[4] = {0.f, 0.f, 0.f, 0.f};
                    if (t == a.Nt - 1)
                        for (int kz = k + 8; kz < a.Ks_out * 32; kz += 8) lv_store<4>(a.act, a.Ks_out, mt0 + j, packed, m, kz, z);
                }
            } else {
#pragma unroll
                for (int i = 0; i < N; ++i) {
                    if (v0 + i >= a.Nt) continue;
                    floatx4 v = tot[i][j];
                    v *= sc;
                    *reinterpret_cast<floatx4*>(a.logits + size_t((mt0 + j) * 16 + m) * a.ldl + tl[i].t * 16 + (lane >> 4) * 4) = v;
                }
            }
        }
    }
}

// ---- what stands between the products ----------------------------------------------------------------
// the four quarters of tile t for row tile mt, then (packed halves) those of the low halves' products
__device__ __forceinline__ floatx4 lv_sum(const LvArgs& a, int t, int mt, int lane, bool pk) {
    const float* p = a.part + (size_t(t) * a.n_tiles + mt) * 256 + lane * 4;
    const size_t st = size_t(a.Nt) * a.n_tiles * 256;
    floatx4 w[4], l[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) w[q] = *reinterpret_cast<const floatx4*>(p + size_t(q) * st);
    if (pk && (lane & 15) < 8) {
#pragma unroll
        for (int q = 0; q < 4; ++q) l[q] = *reinterpret_cast<const floatx4*>(p + size_t(q) * st + 32);
    }
    floatx4 v = ((w[0] + w[1]) + w[2]) + w[3];
    if (pk && (lane & 15) < 8) v = (((v + l[0]) + l[1]) + l[2]) + l[3];
    return v;
}

// Residual update (or, FIRST, the embedding) of 16 rows x 64 columns, a tile per wavefront.
template <bool FIRST>
__global__ __launch_bounds__(256) void k_level_resid(LvArgs a) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int mt = blockIdx.y, m = lane & 15, kq = lane >> 4, t = blockIdx.x * 4 + wave, n0 = t * 16 + kq * 4;
    const LvTile& T = a.t[mt];
    float* xp = a.x + size_t(mt * 16 + m) * a.d + n0;
    floatx4 v = floatx4{0.f, 0.f, 0.f, 0.f};
    if (FIRST) {
        if (blockIdx.x == 0 && mt == 0)
            for (int c = tid; c < a.n_counts; c += 256) a.counts[c] = 0u;
        if (m < T.n) {
            int tok = a.tokens[T.row0 + m];
            tok = tok < 0 ? 0 : (tok >= a.V ? a.V - 1 : tok);
            const uint2v e = *reinterpret_cast<const uint2v*>(a.embed + size_t(tok) * a.d + n0);
            v = floatx4{__uint_as_float(e[0] << 16), __uint_as_float(e[0] & 0xffff0000u), __uint_as_float(e[1] << 16),
                        __uint_as_float(e[1] & 0xffff0000u)};
        }
    } else {
        v = *reinterpret_cast<const floatx4*>(xp) + lv_sum(a, t, mt, lane, T.pk != 0);
    }
    *reinterpret_cast<floatx4*>(xp) = v;
    const floatx4 g = *reinterpret_cast<const floatx4*>(a.gain + n0);
    __bf16 hi[4], lo[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) split_product(v[e], g[e], hi[e], lo[e]);
    if (!(T.pk && m >= 8)) lv_put<4>(a.xf, a.Ks, mt, T.pk != 0, m, n0, hi, lo);
    // sums of squares of eight columns each, one behind the other, then of the tile's two halves
    // (the second square is the rounded one, as the compiler has it in the verify kernel)
    const float sq = fmaf(v[3], v[3], fmaf(v[2], v[2], fmaf(v[0], v[0], v[1] * v[1])));
    float s8 = __shfl_xor(sq, 16);
#pragma unroll
    for (int e = 0; e < 4; ++e) s8 = fmaf(v[e], v[e], s8);  // (of use in the odd quarters of the wavefront)
    const float tile = s8 + __shfl_xor(s8, 32);
    if (kq == 1) a.ss[size_t(mt * 16 + m) * (a.d >> 4) + t] = tile;
}

// Rotation table of the rows' positions, angles in fp64 as in the verify kernel.
__global__ __launch_bounds__(256) void k_level_rope(LvArgs a, float* rope, const int32_t* positions, float theta) {
    const int half = a.h >> 1, e = blockIdx.x * 256 + threadIdx.x;
    if (e >= a.n_tiles * 16 * half) return;
    const int row = e / half, j = e % half;
    const LvTile& T = a.t[row >> 4];
    if ((row & 15) >= T.n) return;
    const double ang = double(positions[T.row0 + (row & 15)]) * pow(double(theta), -2.0 * j / a.h);
    rope[e] = float(cos(ang));
    rope[size_t(a.n_tiles) * 16 * half + e] = float(sin(ang));
}

// QKV: sums, RMSNorm scale, rotation; q for the attention kernel, K and V into the rows' slots.
__global__ __launch_bounds__(256) void k_level_qkv(LvArgs a) {
    __shared__ float scale[16];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int mt = blockIdx.y, m = lane & 15, kq = lane >> 4, row = mt * 16 + m;
    const LvTile& T = a.t[mt];
    if (tid < 128) {
        const float sc = lv_row_scale(a.ss + size_t(mt * 16 + (tid >> 3)) * (a.d >> 4), a.d >> 4, tid & 7, a.inv_d, a.eps);
        if ((tid & 7) == 0) scale[tid >> 3] = sc;
    }
    __syncthreads();
    const int t = blockIdx.x * 4 + wave;
    if (t >= a.Nt) return;
    const float sc = scale[m];
    const int h = a.h, half = h >> 1, prow = t * 16;
    floatx4 v = lv_sum(a, t, mt, lane, T.pk != 0);
    v *= sc;
    const bool on = m < T.n;
    const int slot = a.first_slot + T.row0 + (on ? m : 0), tk = slot & 15;
    const size_t block = size_t(a.block_table[slot >> 4]) * a.Hkv;
    if (prow < a.qd + a.kvd) {
        if (!on) return;
        const bool is_q = prow < a.qd;
        const int rel = is_q ? prow : prow - a.qd;
        const int head = rel / h, p0 = ((rel % h) >> 1) + kq * 2;  // pairs p0, p0 + 1
        const float* cp = a.rope + size_t(row) * half + p0;
        const float* sp = cp + size_t(a.n_tiles) * 16 * half;
        float o2[2][2];  // [which half of the head][pair]
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            o2[0][q] = rotate_first(v[2 * q], v[2 * q + 1], cp[q], sp[q]);
            o2[1][q] = rotate_second(v[2 * q], v[2 * q + 1], cp[q], sp[q]);
        }
        if (is_q) {
            const int kvh = head / a.G, gl = head % a.G;
            __bf16* qp = a.q + (size_t(kvh) * a.n_tiles * 16 * a.G + size_t(row) * a.G + gl) * (2 * h);
#pragma unroll
            for (int w = 0; w < 2; ++w) {
                const int j = p0 + w * half;
                __bf16 h0, l0, h1, l1;
                split_product(o2[w][0], a.inv_sqrt_h, h0, l0);
                split_product(o2[w][1], a.inv_sqrt_h, h1, l1);
                *reinterpret_cast<uint32_t*>(qp + (j >> 3) * 16 + (j & 7)) = pack_bf16(h0, h1);
                *reinterpret_cast<uint32_t*>(qp + (j >> 3) * 16 + (j & 7) + 8) = pack_bf16(l0, l1);
            }
        } else {
            __bf16* kp = a.kpool + (block + head) * (16 * h) + tk * 8;
#pragma unroll
            for (int w = 0; w < 2; ++w) {
                const int j = p0 + w * half;
                *reinterpret_cast<uint32_t*>(kp + (j >> 3) * 128 + (j & 7)) =
                    pack_bf16(static_cast<__bf16>(o2[w][0]), static_cast<__bf16>(o2[w][1]));
            }
        }
        return;
    }
    const int rel = prow - a.qd - a.kvd, head = rel / h, jg = rel % h + kq * 4;
    if (on) {
        __bf16* vp = a.vpool + (block + head) * (16 * h);
#pragma unroll
        for (int e = 0; e < 4; ++e) vp[v_page_index(jg + e, tk)] = static_cast<__bf16>(v[e]);
    }
    // a page that the level opens is cleared behind the level's last slot
    const int end = a.level_end, open = end & ~15;
    if (a.last_row >= T.row0 && a.last_row < T.row0 + T.n && open >= a.level_first && m >= (end & 15) && open < end) {
        __bf16* vp = a.vpool + (size_t(a.block_table[open >> 4]) * a.Hkv + head) * (16 * h);
#pragma unroll
        for (int e = 0; e < 4; ++e) vp[v_page_index(jg + e, m)] = static_cast<__bf16>(0.f);
    }
}

// Attention of one (kv head, 16 (row, head) pairs, cut): the four wavefronts take the cut's pages in turn, two per round,
// and meet in LDS; cuts meet in memory, merged by the last to arrive.
template <int H>
__global__ __launch_bounds__(256, 2) void k_level_attn(LvArgs a) {
    constexpr int ST = H / 32, HT = H / 16, PART = 16 * (H + 2);
    __shared__ float parts[4 * PART];
    __shared__ float wgt[4 * 16], ml[2 * 16];
    __shared__ int last;
    const int tid = threadIdx.x, lane = tid & 63, col = lane & 15, kq = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int mt = 0;
    while (mt + 1 < a.n_tiles && int(blockIdx.x) >= a.t[mt + 1].task0) ++mt;
    const LvTile& T = a.t[mt];
    const int local = int(blockIdx.x) - T.task0, cut = local % T.cuts, sub = (local / T.cuts) % T.subs, kvh = local / (T.cuts * T.subs);
    const int pg0 = cut * T.per_cut, pg1 = min(T.pages, pg0 + T.per_cut);
    const int rho = sub * 16 + col;
    const bool row_ok = rho < T.n * a.G;
    const int mrow = row_ok ? rho / a.G : 0, gl = row_ok ? rho % a.G : 0;
    const uint32_t* mask = a.mask + size_t(T.row0 + mrow) * a.mask_words;
    const int shared = a.level_first >> 4;  // pages from here on hold slots of the level
    bf16x8 qh[ST], ql[ST];
    {
        const bf16x8* qp = reinterpret_cast<const bf16x8*>(
            a.q + (size_t(kvh) * a.n_tiles * 16 * a.G + size_t(mt * 16 + mrow) * a.G + gl) * (2 * H));
#pragma unroll
        for (int st = 0; st < ST; ++st) {
            qh[st] = qp[(st * 4 + kq) * 2];
            ql[st] = qp[(st * 4 + kq) * 2 + 1];
        }
    }
    floatx4 o[HT];
#pragma unroll
    for (int i = 0; i < HT; ++i) o[i] = floatx4{0.f, 0.f, 0.f, 0.f};
    float mx = -1e30f, sum = 0.f;
    MegaArgs pa = {};
    pa.Hkv = a.Hkv;
    bf16x8 ka[ST], kb[ST];
    short4v va[HT], vb[HT];
    auto id = [&](int pg) { return __builtin_amdgcn_readfirstlane(a.block_table[pg < pg1 ? pg : pg1 - 1]); };
    // the 16 visibility bits of a page
    auto bits = [&](int pg) -> uint32_t {
        const int off = pg * 16 - a.mask_base;
        if (!row_ok || pg >= pg1) return 0u;
        if (off < 0) return 0xffffu;
        return (off >> 5) < a.mask_words ? (mask[off >> 5] >> (off & 31)) & 0xffffu : 0u;
    };
    int pg = pg0 + wave;
    int ida = id(pg), idb = id(pg + 4);
    if (pg < pg1) {
        attn_load_k<H>(pa, a.kpool, kvh, ida, lane, ka);
        attn_load_k<H>(pa, a.kpool, kvh, idb, lane, kb);
    }
    for (; pg < pg1; pg += 8) {
        attn_load_v<H>(pa, a.vpool, kvh, ida, lane, va);
        attn_load_v<H>(pa, a.vpool, kvh, idb, lane, vb);
        const uint32_t ba = bits(pg), bb = bits(pg + 4);
        bool oka[4], okb[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            oka[v] = ((ba >> (kq * 4 + v)) & 1u) != 0;
            okb[v] = ((bb >> (kq * 4 + v)) & 1u) != 0;
        }
        px_two_pages<H>(ka, kb, va, vb, qh, ql, oka, okb, o, mx, sum, [&]() {
            ida = id(pg + 8);
            idb = id(pg + 12);
            if (pg + 8 < pg1) {
                attn_load_k<H>(pa, a.kpool, kvh, ida, lane, ka);
                attn_load_k<H>(pa, a.kpool, kvh, idb, lane, kb);
            }
        }, [&]() {
            // A page of the level may hold slots that nobody has written (0 x NaN): V of the slots that none of the
            // tile's rows sees becomes zero.  So does that of a pair's second page where there is none.
            if (pg + 4 < shared && pg + 4 < pg1) return;
            short4v ma, mb;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int sh = lane >> 4 << 4;
                ma[v] = pg < shared || ((__builtin_amdgcn_ballot_w64(oka[v]) >> sh) & 0xffffull) != 0ull ? short(-1) : short(0);
                mb[v] = (pg + 4 < shared && pg + 4 < pg1) || ((__builtin_amdgcn_ballot_w64(okb[v]) >> sh) & 0xffffull) != 0ull
                            ? short(-1) : short(0);
            }
#pragma unroll
            for (int i = 0; i < HT; ++i) {
                va[i] &= ma;
                vb[i] &= mb;
            }
        });
    }
    float* mine = parts + wave * PART;
    if (kq == 0) {
        mine[col] = mx;
        mine[16 + col] = sum;
    }
#pragma unroll
    for (int i = 0; i < HT; ++i)
#pragma unroll
        for (int v = 0; v < 4; ++v) mine[32 + col * H + i * 16 + kq * 4 + v] = o[i][v];
    __syncthreads();
    if (tid < 16) {
        float mg = -1e30f;
        for (int w = 0; w < 4; ++w) mg = fmaxf(mg, parts[w * PART + tid]);
        float l = 0.f;
        for (int w = 0; w < 4; ++w) {
            const float f = __builtin_amdgcn_exp2f(parts[w * PART + tid] - mg);
            wgt[w * 16 + tid] = f;
            l += f * parts[w * PART + 16 + tid];
        }
        ml[tid] = mg;
        ml[16 + tid] = l;
    }
    __syncthreads();
    const int row = tid / (H / 8), ch = tid % (H / 8);  // work item: (pair, eight head elements)
    const bool item = tid < 16 * (H / 8);
    float v8[8];
    if (item) {
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            float acc = 0.f;
            for (int w = 0; w < 4; ++w) acc += wgt[w * 16 + row] * parts[w * PART + 32 + row * H + ch * 8 + q];
            v8[q] = acc;
        }
    }
    float inv_l = 0.f;
    if (T.cuts == 1) {
        if (item) inv_l = 1.0f / ml[16 + row];
    } else {
        float* mine_cut = a.apart + size_t(blockIdx.x) * PART;
        if (item) st_dev_f32x8(mine_cut, 32 + row * H + ch * 8, v8);
        if (tid < 16) {
            st_agent(mine_cut + tid, ml[tid]);
            st_agent(mine_cut + 16 + tid, ml[16 + tid]);
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        if (tid == 0) {
            uint32_t* count = a.counts + T.count0 + kvh * T.subs + sub;
            const uint32_t prev = __hip_atomic_fetch_add(count, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            last = prev == uint32_t(T.cuts) - 1;
            if (last) __hip_atomic_store(count, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        __syncthreads();
        if (!last) return;
        const __amdgpu_buffer_rsrc_t prs = make_rsrc(a.apart + size_t(int(blockIdx.x) - cut) * PART, uint32_t(T.cuts) * PART * 4);
        float mg = -1e30f, lg = 0.f;
#pragma unroll
        for (int q = 0; q < 8; ++q) v8[q] = 0.f;
        constexpr int CH = 10;
        for (int s0 = 0; s0 < T.cuts; s0 += CH) {
            uint32_t mw[CH], lw[CH];
            uint4v p0[CH], p1[CH];
#pragma unroll
            for (int c = 0; c < CH; ++c) {
                const uint32_t at = uint32_t(s0 + c) * PART * 4;
                const int lane_off = (item && s0 + c < T.cuts) ? 0 : kOutOfRange;
                mw[c] = __builtin_amdgcn_raw_buffer_load_b32(prs, lane_off + row * 4, int(at), kAuxDev);
                lw[c] = __builtin_amdgcn_raw_buffer_load_b32(prs, lane_off + (16 + row) * 4, int(at), kAuxDev);
                p0[c] = __builtin_amdgcn_raw_buffer_load_b128(prs, lane_off + (32 + row * H + ch * 8) * 4, int(at), kAuxDev);
                p1[c] = __builtin_amdgcn_raw_buffer_load_b128(prs, lane_off + (32 + row * H + ch * 8) * 4 + 16, int(at), kAuxDev);
            }
            float mnew = mg;
#pragma unroll
            for (int c = 0; c < CH; ++c)
                if (s0 + c < T.cuts) mnew = fmaxf(mnew, __uint_as_float(mw[c]));
            const float resc = __builtin_amdgcn_exp2f(mg - mnew);
            lg *= resc;
#pragma unroll
            for (int q = 0; q < 8; ++q) v8[q] *= resc;
#pragma unroll
            for (int c = 0; c < CH; ++c) {
                const float f = s0 + c < T.cuts ? __builtin_amdgcn_exp2f(__uint_as_float(mw[c]) - mnew) : 0.f;
                lg += f * __uint_as_float(lw[c]);
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    v8[q] += f * __uint_as_float(p0[c][q]);
                    v8[4 + q] += f * __uint_as_float(p1[c][q]);
                }
            }
            mg = mnew;
        }
        if (item) inv_l = 1.0f / lg;
    }
    const int rr = sub * 16 + row;
    if (item && rr < T.n * a.G) {
        __bf16 hi[8], lo[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) split_product(v8[q], inv_l, hi[q], lo[q]);
        lv_put<8>(a.att, a.Ks_att, mt, T.pk != 0, rr / a.G, (kvh * a.G + rr % a.G) * H + ch * 8, hi, lo);
    }
}

// ---- top-k of the vocabulary phase -----------------------------------------------------------------------
struct LvTopkArgs {
    const float* logits;  // [n_tiles * 16][ldl]
    int32_t ldl, V, Nt, nwg, n_tiles, k;
    const uint32_t* stamp;  // {magic, grid size} the weights were laid out for
    LvTile t[kLvTiles];
    float* lse;                  // [n_tiles * 16][nwg][2] (max, sum of exp) of the columns of each position of the stream order
    unsigned long long* best;    // [n_tiles * 16][16 * nwg] largest key of each lane's columns
    int32_t* tok;                // [rows][k]
    float* prob;
};

__device__ __forceinline__ unsigned long long lv_key(float v, int n) {
    return (static_cast<unsigned long long>(float_key(v)) << 32) | (0xffffffffu - uint32_t(n));
}

// The log-sum-exp in the verify kernel's order: there the columns of grid position p (tiles p, p + nwg, ...) are taken by a row's
// lanes in groups of tiles (four and eight lanes where a call has two row tiles, else eight and sixteen), lane l
// the half l & 1 of the group's tile l >> 1; then the lanes are added pairwise.  Here a thread is such a lane, a wavefront 32
// positions and both halves: consecutive threads read consecutive 32 bytes.
__global__ __launch_bounds__(256) void k_level_lse(LvTopkArgs a) {
    __shared__ float pm[16][32], ps[16][32];
    const int row = blockIdx.y, mt = row >> 4, tid = threadIdx.x;
    const LvTile& T = a.t[mt];
    if ((row & 15) >= T.n) return;
    const int group = T.wide ? 4 : 8, lpr = 2 * group;
    const int lane = tid & 63, pl = lane >> 1, p = blockIdx.x * 32 + pl, half = lane & 1;
    const float* src = a.logits + size_t(row) * a.ldl + half * 8;
    for (int i = tid >> 6; i < group; i += 4) {
        float m = -1e30f, s = 0.f;
        unsigned long long best = 0ull;
        if (p < a.nwg)
            for (int t = p + i * a.nwg; t < a.Nt; t += group * a.nwg) {
                const floatx4 c0 = *reinterpret_cast<const floatx4*>(src + size_t(t) * 16);
                const floatx4 c1 = *reinterpret_cast<const floatx4*>(src + size_t(t) * 16 + 4);
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    const int n = t * 16 + half * 8 + q;
                    if (n >= a.V) continue;
                    const float val = q < 4 ? c0[q & 3] : c1[q & 3];
                    const unsigned long long key = lv_key(val, n);
                    best = key > best ? key : best;
                    if (val > m) {
                        s = s * __expf(m - val) + 1.f;
                        m = val;
                    } else {
                        s += __expf(val - m);
                    }
                }
            }
        pm[2 * i + half][pl] = m;
        ps[2 * i + half][pl] = s;
        if (p < a.nwg) a.best[size_t(row) * (16 * a.nwg) + size_t(2 * i + half) * a.nwg + p] = best;
    }
    __syncthreads();
    if (tid < 32 && blockIdx.x * 32 + tid < a.nwg) {
        float mx = pm[0][tid];
        for (int l = 1; l < lpr; ++l) mx = fmaxf(mx, pm[l][tid]);
        float s[16];
#pragma unroll
        for (int l = 0; l < 16; ++l) s[l] = l < lpr ? ps[l][tid] * __expf(pm[l][tid] - mx) : 0.f;
#pragma unroll
        for (int o = 1; o < 16; o <<= 1)
#pragma unroll
            for (int l = 0; l < 16; l += 2 * o)
                if (o < lpr) s[l] += s[l + o];
        float* dst = a.lse + (size_t(row) * a.nwg + blockIdx.x * 32 + tid) * 2;
        dst[0] = mx;
        dst[1] = s[0];
    }
}

// One workgroup per row.  The row's k best tokens lie in the columns of the k lanes whose best keys are the largest: k
// rounds of "largest key below the last one" over the lanes' best, and k more over the columns of the lanes found.
__global__ __launch_bounds__(256) void k_level_topk(LvTopkArgs a) {
    __shared__ unsigned long long wbest[2][4];
    __shared__ float red[8];
    __shared__ int lanes[16];
    const int row = blockIdx.x, mt = row >> 4, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const LvTile& T = a.t[mt];
    if ((row & 15) >= T.n) return;
    const int group = T.wide ? 4 : 8, n_lanes = 2 * group * a.nwg;  // (at most 4096)
    float pm = -1e30f, psum = 0.f;
    if (tid < a.nwg) {
        pm = a.lse[(size_t(row) * a.nwg + tid) * 2];
        psum = a.lse[(size_t(row) * a.nwg + tid) * 2 + 1];
    }
    unsigned long long mine[16];
#pragma unroll
    for (int c = 0; c < 16; ++c) mine[c] = tid + c * 256 < n_lanes ? a.best[size_t(row) * (16 * a.nwg) + tid + c * 256] : 0ull;
    float mx = pm;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) mx = fmaxf(mx, __shfl_xor(mx, o));
    if (lane == 0) red[wave] = mx;
    __syncthreads();
    mx = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
    float sx = psum * __expf(pm - mx);
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) sx += __shfl_xor(sx, o);
    if (lane == 0) red[4 + wave] = sx;
    __syncthreads();
    const float lse = mx + __logf((red[4] + red[5]) + (red[6] + red[7]));
    int round = 0;
    auto block_max = [&](unsigned long long best) {
        best = group_max<16>(best);
#pragma unroll
        for (int o = 16; o < 64; o <<= 1) {
            const unsigned long long other = __shfl_xor(best, o);
            best = other > best ? other : best;
        }
        unsigned long long* slot = wbest[round++ & 1];
        if (lane == 0) slot[wave] = best;
        __syncthreads();
        best = slot[0];
#pragma unroll
        for (int w = 1; w < 4; ++w) best = slot[w] > best ? slot[w] : best;
        return best;
    };
    unsigned long long prev = ~0ull;
    int found = 0;
    for (; found < a.k; ++found) {
        unsigned long long best = 0ull;
#pragma unroll
        for (int c = 0; c < 16; ++c) best = mine[c] < prev && mine[c] > best ? mine[c] : best;
        best = block_max(best);
        if (best == 0ull) break;
#pragma unroll
        for (int c = 0; c < 16; ++c)
            if (mine[c] == best) lanes[found] = tid + c * 256;
        prev = best;
    }
    __syncthreads();
    // column u of the found lanes: eight of each tile
    const int per_lane = (a.Nt + group * a.nwg - 1) / (group * a.nwg) * 8, total = found * per_lane;
    auto key_of = [&](int u) -> unsigned long long {
        if (u >= total) return 0ull;
        const int at = lanes[u / per_lane], l = at / a.nwg, p = at % a.nwg, c = u % per_lane;
        const int t = p + ((l >> 1) + (c >> 3) * group) * a.nwg, n = t * 16 + (l & 1) * 8 + (c & 7);
        return t < a.Nt && n < a.V ? lv_key(a.logits[size_t(row) * a.ldl + n], n) : 0ull;
    };
    // (as many as fit are kept: k <= 16 lanes of 128 columns on 256 positions and a vocabulary of 131 072 with group 4)
#pragma unroll
    for (int c = 0; c < 16; ++c) mine[c] = key_of(tid + c * 256);
    prev = ~0ull;
    const bool bad_layout = a.stamp[0] != kStampMagic || a.stamp[1] != uint32_t(a.nwg);
    for (int j = 0; j < a.k; ++j) {
        unsigned long long best = 0ull;
#pragma unroll
        for (int c = 0; c < 16; ++c) best = mine[c] < prev && mine[c] > best ? mine[c] : best;
        for (int u = tid + 4096; u < total; u += 256) {
            const unsigned long long key = key_of(u);
            best = key < prev && key > best ? key : best;
        }
        best = block_max(best);
        if (tid == 0) {
            const uint32_t kb = uint32_t(best >> 32);
            const float logit = __uint_as_float((kb & 0x80000000u) ? (kb & 0x7fffffffu) : ~kb);
            const size_t at = size_t(T.row0 + (row & 15)) * a.k + j;
            const bool is = best != 0ull && !bad_layout;
            a.tok[at] = is ? int(0xffffffffu - uint32_t(best & 0xffffffffull)) : -1;
            a.prob[at] = is ? __expf(logit - lse) : 0.f;
        }
        prev = best;
    }
}

}  // namespace card
