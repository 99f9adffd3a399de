// Prompt pass: K and V of many context tokens in one go, as a sequence of ordinary kernels.
//
// Why not the persistent verify kernel: its calls carry at most 32 rows, so a prompt streams every
// weight once per 32 tokens and is bound by HBM (8B shape: 4.1 ms per 32 tokens).  With hundreds
// of rows a decoder layer is bound by the matrix pipe instead (each weight fragment meets hundreds
// of rows), hand-overs cost microseconds against hundreds of them, and separate kernels with
// thousands of workgroups are the simpler and the faster form.
//
// The packed weights are the same blob: a 1 KiB fragment is already in the register order of the
// matrix instruction's A operand, so a wavefront loads it straight into registers, no LDS pass.
// Activations are kept in the B operand's order, high and low bf16 halves side by side:
// [block of 4 row tiles][k-step][4 row tiles][hi, lo][64 lanes][8]; a workgroup's share of one
// k-step is 8 contiguous KiB.  As in the verify kernel a normalised row is the gained row (split
// into halves) times its RMSNorm scale, which the consuming kernel applies after its product.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "card_common.hip"
#include "card_layout.h"
#include "card_verify.hip"

namespace card {

constexpr int kPgTiles = 4;      // row tiles per block of the activation layout
constexpr int kPgGroup = 64;     // residual columns per partial sum of squares
constexpr int kPgWaves = 4;      // wavefronts per workgroup of the small kernels
constexpr int kPgN = 4;          // weight tiles per wavefront
constexpr int kPgUnroll = 4;     // k-steps per turn of the product kernel

// element offset of (k-step s, row tile mt) of an activation with Ks k-steps: hi fragment, lo 512 behind
__device__ __forceinline__ size_t px_frag(int Ks, int s, int mt) {
    return ((size_t(mt / kPgTiles) * Ks + s) * kPgTiles + mt % kPgTiles) * 1024;
}
// four consecutive values of row m of tile mt at column k (k % 4 == 0) -> halves in place
__device__ __forceinline__ void px_store4(__bf16* x, int Ks, int mt, int m, int k, const float (&v)[4]) {
    __bf16 h[4], l[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) split_bf16(v[e], h[e], l[e]);
    __bf16* p = x + px_frag(Ks, k >> 5, mt) + (((k >> 3) & 3) * 16 + m) * 8 + (k & 7);
    *reinterpret_cast<uint2v*>(p) = uint2v{pack_bf16(h[0], h[1]), pack_bf16(h[2], h[3])};
    *reinterpret_cast<uint2v*>(p + 512) = uint2v{pack_bf16(l[0], l[1]), pack_bf16(l[2], l[3])};
}

// SwiGLU of two gate/up tiles a and b and 16 rows: a tile holds eight gate rows (lanes 0-31 of the accumulator)
// and the eight up rows that belong to them (lanes 32-63).  The tiles trade halves: lanes 0-31 finish a, lanes 32-63 b.
// sc: the RMSNorm scale of row lane & 15.
__device__ __forceinline__ void px_swiglu_values(int lane, float sc, const floatx4& a, const floatx4& b, float (&v)[4]) {
    const bool low = lane < 32;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const float give = low ? b[e] : a[e];
        const float got = __shfl_xor(give, 32);
        const float g = (low ? a[e] : got) * sc, u = (low ? got : b[e]) * sc;
        v[e] = g * __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(-1.4426950408889634f * g)) * u;
    }
}
// ... of tiles ta and tb (of Nt); `on`: whether this lane's tile exists.
__device__ __forceinline__ void px_swiglu(__bf16* act, int Ks_out, int Nt, int mt, int lane, float sc, const floatx4& a,
                                          const floatx4& b, int ta, int tb, bool on) {
    const int t = lane < 32 ? ta : tb, m = lane & 15;
    float v[4];
    px_swiglu_values(lane, sc, a, b, v);
    if (!on) return;
    const int k = t * 8 + ((lane >> 4) & 1) * 4;
    px_store4(act, Ks_out, mt, m, k, v);
    // whoever writes the last tile fills the rest of the next product's last k-step with zeros
    const float z[4] = {0.f, 0.f, 0.f, 0.f};
    if (t == Nt - 1)
        for (int kz = k + 8; kz < Ks_out * 32; kz += 8) px_store4(act, Ks_out, mt, m, kz, z);
}

// ---- product ------------------------------------------------------------------------------------
struct PgemmArgs {
    const char* w;       // packed matrix
    uint32_t bytes;
    int32_t Nt, Ks, NB, nwg;  // tiles, k-steps, batch width and grid of the stream order
    const __bf16* x;     // activations [blocks][Ks][kPgTiles][2][64][8]
    int32_t mts;         // end of the row tiles in use
    int32_t mt0, mcap;   // first row tile, and how many the partials have room for
    int32_t nblk, mblk, splits;
    float* part;         // [splits][Nt][mcap][64][4]
    // SwiGLU
    const float* ss;     // [rows][ss_groups]
    int32_t ss_groups, Ks_out;
    float inv_d, eps;
    __bf16* act;
    // arg-max over the vocabulary, of one row
    int32_t row, V;
    unsigned long long* best;
};

enum PgemmEpi { PG_PART = 0, PG_SWIGLU = 1, PG_ARGMAX = 2 };

// RMSNorm scale of a row from its partial sums of squares, by LPR neighbouring lanes.
template <int LPR>
__device__ __forceinline__ float px_row_scale(const float* ss, int groups, int sub, float inv_d, float eps) {
    float sq = 0.f;
    for (int g = sub; g < groups; g += LPR) sq += ss[g];
#pragma unroll
    for (int o = 1; o < LPR; o <<= 1) sq += __shfl_xor(sq, o);
    return 1.0f / sqrtf(sq * inv_d + eps);
}

// Where the fragments of one weight tile lie: stream order inside a wavefront pair's share of K is
// one fixed step per k-step.
// Tiles are dealt in memory order: position after position, the tiles of a position in a row, so that
// a workgroup's sixteen fragments of a k-step lie in one or two contiguous runs where a position owns several.
struct PgTile {
    uint32_t base;       // fragment index of the tile's position
    int32_t cnt, skip, nv, i;
    int32_t t;           // tile number in the matrix
    __device__ __forceinline__ void init(const PgemmArgs& a, int v) {
        const int full = a.Nt / a.nwg, rem = a.Nt % a.nwg, wide = rem * (full + 1);
        const int p = v < wide ? v / (full + 1) : rem + (v - wide) / max(full, 1);
        const int j = v < wide ? v % (full + 1) : (v - wide) % max(full, 1);
        t = p + j * a.nwg;
        cnt = full + (p < rem ? 1 : 0);
        base = uint32_t(full * p + (p < rem ? p : rem)) * uint32_t(a.Ks);
        skip = (j / a.NB) * a.NB;
        nv = min(cnt - skip, a.NB);
        i = j % a.NB;
    }
    // byte offset of k-step s, which belongs to the pair with k-steps [s0, s1)
    __device__ __forceinline__ uint32_t at(int s, int s0, int s1) const {
        return (base + uint32_t(cnt * s0 + skip * (s1 - s0) + (s - s0) * nv + i)) << 10;
    }
};

// The matrix instructions of KB k-steps on a wavefront's N weight tiles (weights(k)) and MT row tiles, whose halves lie in LDS.
// A row tile's fragments are read AHEAD steps before they are used: left to itself the compiler reads them right in front of their first
// use, and a wavefront then waits for LDS four times a k-step (gate/up of the 1B shape, 203 rows: 39.7 -> 35.3 us).  before(k) runs in front of k-step k.
template <int N, int MT, int KB, typename W, typename F>
__device__ __forceinline__ void px_half_turn(const uint4v (&x)[KB * MT * 2][64], int lane, floatx4 (&acc)[N][MT], W&& weights, F&& before) {
    constexpr int J = N >= 4 ? 1 : 2;      // row tiles per step: at least four independent instructions in a row (two of N = 1)
    constexpr int STEPS = KB * MT / J, AHEAD = N == 1 || (N >= 4 && MT < 8) ? 2 : 1;
    static_assert(MT % J == 0 && STEPS >= AHEAD, "steps");
    bf16x8 fr[STEPS][2 * J];
    auto read = [&](int i) {
#pragma unroll
        for (int q = 0; q < 2 * J; ++q) fr[i][q] = __builtin_bit_cast(bf16x8, x[i * 2 * J + q][lane]);
    };
#pragma unroll
    for (int i = 0; i < AHEAD; ++i) read(i);
#pragma unroll
    for (int i = 0; i < STEPS; ++i) {
        const int k = i * J / MT;
        if (i * J % MT == 0) before(k);
        if (i + AHEAD < STEPS) read(i + AHEAD);
        __builtin_amdgcn_sched_barrier(0);
        const bf16x8(&w)[N] = weights(k);
#pragma unroll
        for (int half = 0; half < 2; ++half)
#pragma unroll
            for (int q = 0; q < J; ++q)
#pragma unroll
                for (int n = 0; n < N; ++n) {
                    floatx4& c = acc[n][(i * J + q) % MT];
                    c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[n], fr[i][2 * q + half], c, 0, 0, 0);
                }
    }
}

// One workgroup of W wavefronts: 4 W weight tiles (four per wavefront, straight from memory into registers: no
// other wavefront needs them) x MT row tiles (staged through LDS: all of them need them), a range of K.
// Per k-step a wavefront issues 8 MT matrix instructions (high and low halves).  W = 8 fills a compute unit with one
// workgroup, W = 4 with two; either way two wavefronts share a SIMD.
// A compute unit brings in about 57 GB/s of weights (HBM) and activations (L2) together, so wide workgroups pay by what they do not
// read again: per k-step 46 KiB for 448 matrix instructions at 8 x 7, 24 for 128 at 4 x 4.  Measured on the 8B shape, 1000 rows, us,
// 4 x 4 / 8 x 4 / 8 x 7: gate/up 371 / 381 / 326 (1.45 PFLOP/s issued, halves counted; in other sessions 338-348), QKV 88 / 90 / 82, O 58 /
// 55 / 62, down 180 / 166 / 174; with zeros as operands gate/up takes 276: the card's power.  Eight row tiles spill (383).
template <int EPI, int W, int MT>
__global__ __launch_bounds__(W * 64, 2) void k_prompt_gemm(PgemmArgs a) {
    constexpr int KB = kPgUnroll;                 // k-steps between two barriers, and in the ring of weights
    constexpr int XF = KB * 2 * MT, XW = XF / W;  // their activation fragments, per wavefront
    static_assert(XF % W == 0, "fragments dealt evenly");
    __shared__ uint4v xs[2][XF][64];
    __shared__ __align__(8) float scale[MT * 16];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // Workgroups go to the eight compute dies in turn: a die gets a contiguous range of the blocks in
    // (weight block, K range, row block) order, so its L2 sees few weight panels, each used by every row block.
    const int total = a.nblk * a.splits * a.mblk, per = (total + 7) >> 3;
    const int L = int(blockIdx.x & 7) * per + int(blockIdx.x >> 3);
    if (int(blockIdx.x >> 3) >= per || L >= total) return;
    const int mb = L % a.mblk, sp = (L / a.mblk) % a.splits, nb = L / (a.mblk * a.splits);
    const int kc = (a.Ks + KB - 1) / KB;  // K in whole turns
    const int k0 = kc * sp / a.splits * KB, k1 = kc * (sp + 1) / a.splits * KB, ke = min(k1, a.Ks);
    const int v0 = (nb * W + wave) * kPgN, mt0 = a.mt0 + mb * MT;

    const __amdgpu_buffer_rsrc_t wr = make_rsrc(a.w, a.bytes);
    PgTile tl[kPgN];
#pragma unroll
    for (int i = 0; i < kPgN; ++i) tl[i].init(a, min(v0 + i, a.Nt - 1));
    uint32_t woff[kPgN];
    int sa = k0, seg_end = k0;  // next k-step to load; first one behind the pair's share that woff is valid in
    auto load_a = [&](bf16x8 (&r)[kPgN]) {
        if (sa >= seg_end && sa < a.Ks) {
            int w = 0;
            while (w + 1 < kStreamWaves && sa >= ((w + 1) * a.Ks) / kStreamWaves) ++w;
            const int s0 = (w * a.Ks) / kStreamWaves;
            seg_end = ((w + 1) * a.Ks) / kStreamWaves;
#pragma unroll
            for (int i = 0; i < kPgN; ++i) woff[i] = tl[i].at(sa, s0, seg_end);
        }
        int voff = sa < ke ? lane * 16 : kOutOfRange;
        asm volatile("" : "+v"(voff));  // (one load here, not one per way to this offset: the second would wait for the first)
#pragma unroll
        for (int i = 0; i < kPgN; ++i) {
            r[i] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(wr, voff, int(woff[i]), 0));
            woff[i] += uint32_t(tl[i].nv) << 10;
        }
        ++sa;
    };
    // fragment f of a turn: k-step f / (2 MT), row tile f / 2 % MT, half f % 2; the wavefront brings XW consecutive ones
    const __amdgpu_buffer_rsrc_t xr = make_rsrc(a.x, uint32_t(a.Ks) * uint32_t((a.mts + kPgTiles - 1) / kPgTiles * kPgTiles) * 2048u);
    uint32_t xoff[XW];
    int xstep[XW];
#pragma unroll
    for (int q = 0; q < XW; ++q) {
        const int f = wave * XW + q, mt = mt0 + f / 2 % MT;
        xstep[q] = mt < a.mts ? f / (2 * MT) : 1 << 24;  // (no such row tile: no such k-step)
        xoff[q] = uint32_t(px_frag(a.Ks, f / (2 * MT), mt)) * 2u + uint32_t(f & 1) * 1024u;
    }
    int sb = k0;
    uint4v xb[XW];
    auto load_b = [&]() {
#pragma unroll
        for (int q = 0; q < XW; ++q) {
            int voff = sb + xstep[q] < ke ? lane * 16 : kOutOfRange;
            asm volatile("" : "+v"(voff));
            xb[q] = __builtin_amdgcn_raw_buffer_load_b128(xr, voff, int(xoff[q] + uint32_t(sb) * (kPgTiles * 2048u)), 0);
        }
        sb += KB;
    };
    auto store_b = [&](int buf) {
#pragma unroll
        for (int q = 0; q < XW; ++q) xs[buf][wave * XW + q][lane] = xb[q];
    };

    floatx4 acc[kPgN][MT];
#pragma unroll
    for (int i = 0; i < kPgN; ++i)
#pragma unroll
        for (int j = 0; j < MT; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
    bf16x8 wa[KB][kPgN];
    load_b();
#pragma unroll
    for (int q = 0; q + 1 < KB; ++q) load_a(wa[q]);
    store_b(0);
    auto sync = [&]() {  // LDS writes done, everybody here; loads stay in flight
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(kWaitLds);
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    sync();
    // A turn: request the next one's activations, multiply this one's (requesting weights KB - 1 k-steps on), then put
    // the next one's into the other LDS buffer, which everybody left at the last barrier.
    for (int s = k0, h = 0; s < k1; s += KB, h ^= 1) {
        load_b();
        px_half_turn<kPgN, MT, KB>(xs[h], lane, acc, [&](int k) -> const bf16x8(&)[kPgN] { return wa[k]; },
                                   [&](int k) { load_a(wa[(k + KB - 1) % KB]); });
        store_b(h ^ 1);
        sync();
    }

    if constexpr (EPI == PG_PART) {
#pragma unroll
        for (int i = 0; i < kPgN; ++i) {
            if (v0 + i >= a.Nt) continue;
            float* p = a.part + ((size_t(sp) * a.Nt + tl[i].t) * a.mcap + mt0 - a.mt0) * 256 + lane * 4;
#pragma unroll
            for (int j = 0; j < MT; ++j)
                if (mt0 + j < a.mts) *reinterpret_cast<floatx4*>(p + j * 256) = acc[i][j];
        }
    } else if constexpr (EPI == PG_SWIGLU) {
        for (int e = tid; e < MT * 64; e += W * 64) {
            if (mt0 + (e >> 6) >= a.mts) continue;
            const float sc = px_row_scale<4>(a.ss + size_t(mt0 * 16 + (e >> 2)) * a.ss_groups, a.ss_groups, e & 3, a.inv_d, a.eps);
            if ((e & 3) == 0) scale[e >> 2] = sc;
        }
        sync();
#pragma unroll
        for (int i = 0; i < kPgN; i += 2)
#pragma unroll
            for (int j = 0; j < MT; ++j)
                px_swiglu(a.act, a.Ks_out, a.Nt, mt0 + j, lane, scale[j * 16 + (lane & 15)], acc[i][j], acc[i + 1][j], tl[i].t,
                          tl[i + 1].t, v0 + i + (lane < 32 ? 0 : 1) < a.Nt && mt0 + j < a.mts);
    } else {
        // arg-max of one row: (ordered logit, ~token) keys, the lowest token among equals
        const float sc = px_row_scale<64>(a.ss + size_t(a.row) * a.ss_groups, a.ss_groups, lane, a.inv_d, a.eps);
        unsigned long long best = 0ull;
#pragma unroll
        for (int j = 0; j < MT; ++j)
            if (mt0 + j == a.row >> 4 && (lane & 15) == (a.row & 15)) {
#pragma unroll
                for (int i = 0; i < kPgN; ++i)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int n = tl[i].t * 16 + (lane >> 4) * 4 + e;
                        const unsigned long long key =
                            (static_cast<unsigned long long>(float_key(acc[i][j][e] * sc)) << 32) | (0xffffffffu - uint32_t(n));
                        if (n < a.V && key > best) best = key;
                    }
            }
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const unsigned long long other = __shfl_xor(best, o);
            best = other > best ? other : best;
        }
        unsigned long long* wb = reinterpret_cast<unsigned long long*>(scale);
        if (lane == 0) wb[wave] = best;
        sync();
        if (tid == 0) {
#pragma unroll
            for (int w = 1; w < W; ++w) best = wb[w] > best ? wb[w] : best;
            __hip_atomic_fetch_max(a.best, best, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
}

// stamp: as in the verify kernel, weights laid out for another grid size are in the wrong order: no token
__global__ void k_prompt_token(const unsigned long long* best, const uint32_t* stamp, int nwg, int32_t* out) {
    const bool bad_layout = stamp[0] != kStampMagic || stamp[1] != uint32_t(nwg);
    *out = bad_layout ? -1 : int32_t(0xffffffffu - uint32_t(*best & 0xffffffffull));
}

// ---- what stands between the products ----------------------------------------------------------------
struct PepiArgs {
    const float* part;   // [splits][Nt][mcap][64][4]
    int32_t splits, Nt, mp0, mcap;
    int32_t d, rows, mt0;  // mt0: first row tile to work on
    // residual
    float* x;            // [mcap * 16][d]
    __bf16* xf;
    const float* gain;
    float* ss;
    int32_t ss_groups;
    // embedding
    const __bf16* embed;
    const int32_t* tokens;
    int32_t V;
    unsigned long long* best;
    // QKV
    int32_t qd, kvd, h, Hkv, G, ctx_len, qcap;
    float inv_d, eps, inv_sqrt_h;
    const float* rope;   // [rope_rows][h/2] cos, then the same of sin
    int32_t rope_rows;
    __bf16* q;           // [Hkv][qcap][h/8][16]
    __bf16* kpool;
    __bf16* vpool;
    const int32_t* block_table;
};

__device__ __forceinline__ floatx4 part_sum(const PepiArgs& a, int t, int mt, int lane) {
    const float* p = a.part + (size_t(t) * a.mcap + mt - a.mp0) * 256 + lane * 4;
    const size_t st = size_t(a.Nt) * a.mcap * 256;
    floatx4 v = *reinterpret_cast<const floatx4*>(p);
    int s = 1;
    for (; s + 3 < a.splits; s += 4) {  // four loads on their way at a time, added in order
        floatx4 w[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) w[q] = *reinterpret_cast<const floatx4*>(p + size_t(s + q) * st);
#pragma unroll
        for (int q = 0; q < 4; ++q) v += w[q];
    }
    for (; s < a.splits; ++s) v += *reinterpret_cast<const floatx4*>(p + size_t(s) * st);
    return v;
}

// Residual update (or, FIRST, the embedding): x += sum of the K ranges; the next product's operand
// (x times the next norm's gain, split) and the sums of squares behind its RMSNorm scale.
// One workgroup: 16 rows x 64 columns, a tile per wavefront: a short prompt has few row tiles, and
// the sums over many K ranges need every compute unit.
template <bool FIRST>
__global__ __launch_bounds__(256) void k_prompt_resid(PepiArgs a) {
    __shared__ float red[kPgWaves][16];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int mt = a.mt0 + blockIdx.y, grp = blockIdx.x, m = lane & 15, row = mt * 16 + m;
    const int Ks = a.d >> 5, t = grp * kPgWaves + wave, n0 = t * 16 + (lane >> 4) * 4;
    float* xp = a.x + size_t(row) * a.d + n0;
    floatx4 v = floatx4{0.f, 0.f, 0.f, 0.f};
    if (FIRST) {
        if (blockIdx.x == 0 && blockIdx.y == 0 && tid == 0) *a.best = 0ull;
        if (row < a.rows) {
            int tok = a.tokens[row];
            tok = tok < 0 ? 0 : (tok >= a.V ? a.V - 1 : tok);
            const uint2v e = *reinterpret_cast<const uint2v*>(a.embed + size_t(tok) * a.d + n0);
            v = floatx4{__uint_as_float(e[0] << 16), __uint_as_float(e[0] & 0xffff0000u), __uint_as_float(e[1] << 16),
                        __uint_as_float(e[1] & 0xffff0000u)};
        }
    } else {
        v = *reinterpret_cast<const floatx4*>(xp) + part_sum(a, t, mt, lane);
    }
    *reinterpret_cast<floatx4*>(xp) = v;
    const floatx4 g = *reinterpret_cast<const floatx4*>(a.gain + n0);
    float gv[4], sq = 0.f;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        sq += v[e] * v[e];
        gv[e] = v[e] * g[e];
    }
    px_store4(a.xf, Ks, mt, m, n0, gv);
    sq += __shfl_xor(sq, 16);
    sq += __shfl_xor(sq, 32);
    if (lane < 16) red[wave][lane] = sq;
    __syncthreads();
    if (tid < 16) a.ss[size_t(mt * 16 + tid) * a.ss_groups + grp] = (red[0][tid] + red[1][tid]) + (red[2][tid] + red[3][tid]);
}

// SwiGLU of a gate/up product that was cut along K.  One workgroup: 16 rows, a tile pair per wavefront.
__global__ __launch_bounds__(256) void k_prompt_swiglu(PepiArgs a, __bf16* act, int Ks_out) {
    __shared__ float scale[16];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, mt = a.mt0 + blockIdx.y;
    const float rsc = px_row_scale<16>(a.ss + size_t(mt * 16 + (tid >> 4)) * a.ss_groups, a.ss_groups, tid & 15, a.inv_d, a.eps);
    if ((tid & 15) == 0) scale[tid >> 4] = rsc;
    __syncthreads();
    const int ta = (blockIdx.x * kPgWaves + wave) * 2, tb = min(ta + 1, a.Nt - 1);
    if (ta >= a.Nt) return;
    const floatx4 pa = part_sum(a, ta, mt, lane), pb = part_sum(a, tb, mt, lane);
    px_swiglu(act, Ks_out, a.Nt, mt, lane, scale[lane & 15], pa, pb, ta, ta + 1, (lane < 32 ? ta : ta + 1) < a.Nt);
}

// Rotation table of the pass's positions, angles in fp64 as in the verify kernel.
__global__ __launch_bounds__(256) void k_prompt_rope(float* rope, int rows, int cap_rows, int half, int ctx_len, float theta, int h) {
    const int e = blockIdx.x * 256 + threadIdx.x;
    if (e >= rows * half) return;
    const int m = e / half, j = e % half;
    const double ang = double(ctx_len + m) * pow(double(theta), -2.0 * j / h);
    rope[size_t(m) * half + j] = float(cos(ang));
    rope[size_t(cap_rows) * half + size_t(m) * half + j] = float(sin(ang));
}

// QKV: sum of the K ranges, RMSNorm scale, rotation; q (scaled by log2(e)/sqrt(h), split) for the
// attention kernel, K and V into their pages.  A row tile is one page (a pass starts on one).
// One workgroup: 16 rows, a tile per wavefront (four: 9.1 instead of 5.4 us on 203 rows of the 1B shape).
__global__ __launch_bounds__(256) void k_prompt_qkv(PepiArgs a) {
    __shared__ float scale[16];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int mt = blockIdx.y, m = lane & 15, kq = lane >> 4, row = mt * 16 + m;
    const float rsc = px_row_scale<16>(a.ss + size_t(mt * 16 + (tid >> 4)) * a.ss_groups, a.ss_groups, tid & 15, a.inv_d, a.eps);
    if ((tid & 15) == 0) scale[tid >> 4] = rsc;
    __syncthreads();
    const float sc = scale[m];
    const int h = a.h, half = h >> 1, slot = a.ctx_len + row, tk = slot & 15;
    const bool on = row < a.rows;
    const int page = a.block_table[slot >> 4];  // (a tile has at least one row, and is one page)
    const int t = blockIdx.x * kPgWaves + wave;
    if (t >= a.Nt) return;
    floatx4 v = part_sum(a, t, mt, lane);
    v *= sc;
    const int prow = t * 16;
    if (prow < a.qd + a.kvd) {
        const bool is_q = prow < a.qd;
        const int rel = is_q ? prow : prow - a.qd;
        const int head = rel / h, p0 = ((rel % h) >> 1) + kq * 2;  // pairs p0, p0 + 1
        if (!on) return;
        const float* cp = a.rope + size_t(row) * half + p0;
        const float* sp = cp + size_t(a.rope_rows) * half;
        float lo2[2], hi2[2];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            lo2[q] = v[2 * q] * cp[q] - v[2 * q + 1] * sp[q];
            hi2[q] = v[2 * q + 1] * cp[q] + v[2 * q] * sp[q];
        }
        if (is_q) {
            const int kvh = head / a.G, gl = head % a.G;
            __bf16* qp = a.q + (size_t(kvh) * a.qcap + size_t(row) * a.G + gl) * (2 * h);
#pragma unroll
            for (int w = 0; w < 2; ++w) {
                const int j = p0 + w * half;
                __bf16 h0, l0, h1, l1;
                split_bf16((w ? hi2[0] : lo2[0]) * a.inv_sqrt_h, h0, l0);
                split_bf16((w ? hi2[1] : lo2[1]) * a.inv_sqrt_h, h1, l1);
                *reinterpret_cast<uint32_t*>(qp + (j >> 3) * 16 + (j & 7)) = pack_bf16(h0, h1);
                *reinterpret_cast<uint32_t*>(qp + (j >> 3) * 16 + (j & 7) + 8) = pack_bf16(l0, l1);
            }
        } else {
            __bf16* kp = a.kpool + (size_t(page) * a.Hkv + head) * (16 * h) + tk * 8;
#pragma unroll
            for (int w = 0; w < 2; ++w) {
                const int j = p0 + w * half;
                *reinterpret_cast<uint32_t*>(kp + (j >> 3) * 128 + (j & 7)) =
                    w ? pack_bf16(static_cast<__bf16>(hi2[0]), static_cast<__bf16>(hi2[1]))
                      : pack_bf16(static_cast<__bf16>(lo2[0]), static_cast<__bf16>(lo2[1]));
            }
        }
    } else {  // (the slots behind the prompt's last token are cleared: the page is opened here)
        if (!on) v = floatx4{0.f, 0.f, 0.f, 0.f};
        const int rel = prow - a.qd - a.kvd, head = rel / h, jg = rel % h + kq * 4;
        __bf16* vp = a.vpool + (size_t(page) * a.Hkv + head) * (16 * h);
#pragma unroll
        for (int e = 0; e < 4; ++e) vp[v_page_index(jg + e, tk)] = static_cast<__bf16>(v[e]);
    }
}

// ---- attention -----------------------------------------------------------------------------------------
struct PattnArgs {
    const __bf16* q;
    const __bf16* kpool;
    const __bf16* vpool;
    const int32_t* block_table;
    int32_t qcap, rows, G, Hkv, ctx_len, row_tiles, Ks_out;
    __bf16* att;
};

// One round of a wavefront's walk over the cache, two pages of 16 keys, for 16 query rows: scores, online softmax, output.
// oka / okb: which keys of the lane's four its row sees.  scores_done runs once the K operands have been used,
// weights_done before V is.
template <int H, typename F1, typename F2>
__device__ __forceinline__ void px_two_pages(const bf16x8 (&ka)[H / 32], const bf16x8 (&kb)[H / 32], const short4v (&va)[H / 16],
                                             const short4v (&vb)[H / 16], const bf16x8 (&qh)[H / 32], const bf16x8 (&ql)[H / 32],
                                             const bool (&oka)[4], const bool (&okb)[4], floatx4 (&o)[H / 16], float& mx,
                                             float& sum, F1&& scores_done, F2&& weights_done) {
    floatx4 sa = floatx4{0.f, 0.f, 0.f, 0.f}, sb = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int st = 0; st < H / 32; ++st) {
        sa = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ka[st], qh[st], sa, 0, 0, 0);
        sb = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kb[st], qh[st], sb, 0, 0, 0);
        sa = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ka[st], ql[st], sa, 0, 0, 0);
        sb = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kb[st], ql[st], sb, 0, 0, 0);
    }
    scores_done();
    float pmax = -1e30f;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        if (oka[v]) pmax = fmaxf(pmax, sa[v]);
        if (okb[v]) pmax = fmaxf(pmax, sb[v]);
    }
    pmax = max_across_rows(pmax);
    const float mnew = fmaxf(mx, pmax);
    const float alpha = __builtin_amdgcn_exp2f(mx - mnew);
    float psum = 0.f;
    short4v pah, pal, pbh, pbl;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const float xa = oka[v] ? __builtin_amdgcn_exp2f(sa[v] - mnew) : 0.f;
        const float xb = okb[v] ? __builtin_amdgcn_exp2f(sb[v] - mnew) : 0.f;
        psum += xa + xb;
        __bf16 hi, lo;
        split_bf16(xa, hi, lo);
        pah[v] = __builtin_bit_cast(short, hi);
        pal[v] = __builtin_bit_cast(short, lo);
        split_bf16(xb, hi, lo);
        pbh[v] = __builtin_bit_cast(short, hi);
        pbl[v] = __builtin_bit_cast(short, lo);
    }
    psum = sum_across_rows(psum);
    sum = sum * alpha + psum;
    mx = mnew;
    weights_done();
#pragma unroll
    for (int i = 0; i < H / 16; ++i) {
        floatx4 acc = o[i];
        acc[0] *= alpha; acc[1] *= alpha; acc[2] *= alpha; acc[3] *= alpha;
        acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(va[i], pah, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(vb[i], pbh, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(va[i], pal, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(vb[i], pbl, acc, 0, 0, 0);
        o[i] = acc;
    }
}

// Causal attention of the pass's rows over the paged cache.  A wavefront owns 16 rows (of the G query
// heads that share a KV head, row (m, g) = m * G + g) and walks the pages up to its last row's position,
// two per round, as the verify kernel does; the four wavefronts of a workgroup own neighbouring row tiles
// of one KV head, so they read the same pages at about the same time.
template <int H>
__global__ __launch_bounds__(256, 2) void k_prompt_attn(PattnArgs a) {
    constexpr int ST = H / 32, HT = H / 16;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kvh = blockIdx.x % a.Hkv;
    const int rt = a.row_tiles - 1 - (int(blockIdx.x / a.Hkv) * kPgWaves + wave);  // the longest first
    if (rt < 0) return;
    const int R = a.rows * a.G, col = lane & 15, kq = lane >> 4;
    const int rho = rt * 16 + col;
    const bool row_ok = rho < R;
    const int mrow = row_ok ? rho / a.G : 0, gl = row_ok ? rho % a.G : 0;
    const int limit = row_ok ? a.ctx_len + mrow : -1;
    const int last = min(rt * 16 + 15, R - 1) / a.G;
    const int n_pages = (a.ctx_len + last) / 16 + 1;
    bf16x8 qh[ST], ql[ST];
    {
        const bf16x8* qp = reinterpret_cast<const bf16x8*>(a.q + (size_t(kvh) * a.qcap + (row_ok ? rho : 0)) * (2 * H));
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
    auto id = [&](int pg) { return __builtin_amdgcn_readfirstlane(a.block_table[pg < n_pages ? pg : n_pages - 1]); };
    int ida = id(0), idb = id(1);
    attn_load_k<H>(pa, a.kpool, kvh, ida, lane, ka);
    attn_load_k<H>(pa, a.kpool, kvh, idb, lane, kb);
    for (int pg = 0; pg < n_pages; pg += 2) {
        attn_load_v<H>(pa, a.vpool, kvh, ida, lane, va);
        attn_load_v<H>(pa, a.vpool, kvh, idb, lane, vb);
        bool oka[4], okb[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            oka[v] = pg * 16 + kq * 4 + v <= limit;
            okb[v] = pg * 16 + 16 + kq * 4 + v <= limit;
        }
        px_two_pages<H>(ka, kb, va, vb, qh, ql, oka, okb, o, mx, sum, [&]() {
            ida = id(pg + 2);
            idb = id(pg + 3);
            if (pg + 2 < n_pages) {
                attn_load_k<H>(pa, a.kpool, kvh, ida, lane, ka);
                attn_load_k<H>(pa, a.kpool, kvh, idb, lane, kb);
            }
        }, []() {});
    }
    if (!row_ok) return;
    const float inv = 1.0f / sum;
#pragma unroll
    for (int i = 0; i < HT; ++i) {
        float v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = o[i][e] * inv;
        px_store4(a.att, a.Ks_out, mrow >> 4, mrow & 15, (kvh * a.G + gl) * H + i * 16 + kq * 4, v);
    }
}

}  // namespace card
