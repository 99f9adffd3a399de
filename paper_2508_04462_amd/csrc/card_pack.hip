// Weight re-layout (canonical row-major -> matrix-instruction fragments in stream order) and the KV read-back helper.
#pragma once
#include "card_common.hip"

namespace card {

// ------------------------------------------------------------------------------------------
// Weight re-layout: canonical row-major bf16 -> fragments in stream order, and the coded copy.  One wavefront per fragment: its
// stores are whole lines (one thread per chunk of a row: 8B shape with the coded copy 42 ms longer than without, now 4).
// ------------------------------------------------------------------------------------------
enum RowMap { MAP_IDENT = 0, MAP_ROPE = 1, MAP_GATE = 2, MAP_UP = 3 };

struct PackArgs {
    const __bf16* src;  // [src_rows][K]
    __bf16* dst;        // packed matrix base
    int32_t src_rows, K, Ks;
    int32_t Nt, NB, nwg;              // stream order: tiles of the matrix, batch width, grid size
    int32_t prow0;      // first packed row (MAP_IDENT / MAP_ROPE)
    int32_t map, head_dim;
    int32_t t0, tiles;  // tiles of the matrix that hold rows of this tensor
    uint32_t* stamp;    // {magic, grid size}
    uint32_t *copy_word, copy_bit;  // where the stamp block says that the coded copy holds this tensor (or null)
    // coded copy (or null): its planes, the bits of this tensor's fragments in stream order and in grouped order (or null)
    char* planes;
    unsigned long long *fl, *gfl;
    uint32_t *base4, *counts;  // base in all four bytes; 128 counters
};

// Whoever verifies with these weights must run the grid they are laid out for.
__global__ __launch_bounds__(128) void k_pack_begin(PackArgs a) {
    const int i = threadIdx.x;
    if (a.planes) a.counts[i] = 0u;
    if (i == 0) {
        a.stamp[0] = kStampMagic;
        a.stamp[1] = uint32_t(a.nwg);
        // (a word is shared with other tensors, which may be packed at the same time)
        if (a.planes) atomicOr(a.copy_word, a.copy_bit);
        else if (a.copy_word) atomicAnd(a.copy_word, ~a.copy_bit);
    }
}
// Coded copy: weights counted by bits 8-14 (of large tensors an eighth, spread over all of it: it is the usual ones that count), and
// the window of eight values that holds most of them.
__global__ __launch_bounds__(256) void k_pack_count(PackArgs a) {
    __shared__ uint32_t n[128 * 32];  // 32 copies: neighbouring lanes mostly count the same value
    for (int i = threadIdx.x; i < 128 * 32; i += 256) n[i] = 0u;
    __syncthreads();
    const int64_t chunks = int64_t(a.src_rows) * a.K / 8, pieces = (chunks + 255) / 256, every = pieces >= 1024 ? 8 : 1;
    for (int64_t p = int64_t(blockIdx.x) * every; p < pieces; p += int64_t(gridDim.x) * every) {
        const int64_t i = p * 256 + threadIdx.x;
        if (i >= chunks) break;
        const uint4v v = reinterpret_cast<const uint4v*>(a.src)[i];
#pragma unroll
        for (int e = 0; e < 8; ++e) atomicAdd(&n[((v[e >> 1] >> ((e & 1) * 16 + 8)) & 127u) * 32 + (threadIdx.x & 31)], 1u);
    }
    __syncthreads();
    if (threadIdx.x < 128) {
        uint32_t sum = 0;
        for (int c = 0; c < 32; ++c) sum += n[threadIdx.x * 32 + ((c + threadIdx.x) & 31)];
        if (sum) atomicAdd(a.counts + threadIdx.x, sum);
    }
}
__global__ __launch_bounds__(128) void k_pack_base(PackArgs a) {
    __shared__ uint32_t n[136];
    __shared__ unsigned long long best;
    const int i = threadIdx.x;
    n[i] = a.counts[i];
    if (i == 0) best = 0ull;
    __syncthreads();
    if (i <= 120) {
        uint32_t sum = 0;
        for (int q = 0; q < 8; ++q) sum += n[i + q];
        atomicMax(&best, (static_cast<unsigned long long>(sum) << 32) | uint32_t(i));
    }
    __syncthreads();
    if (i == 0) *a.base4 = uint32_t(best & 0xffffffffull) * 0x01010101u;
}

__global__ __launch_bounds__(256) void k_pack(PackArgs a) {
    const int64_t id = int64_t(blockIdx.x) * 4 + (threadIdx.x >> 6);
    if (id >= int64_t(a.tiles) * a.Ks) return;
    const int lane = threadIdx.x & 63, t = a.t0 + int(id / a.Ks), s = int(id % a.Ks);
    const int row = lane & 15, idx = t * 16 + row - a.prow0;
    int srow = idx;
    bool mine = true;
    if (a.map == MAP_ROPE) {
        const int h = a.head_dim, i = idx % h;
        srow = (idx / h) * h + (i >> 1) + (i & 1) * (h >> 1);
    } else if (a.map != MAP_IDENT) {  // eight gate rows, then the eight up rows that belong to them
        srow = t * 8 + (row & 7);
        mine = (row >= 8) == (a.map == MAP_UP);
    }
    const int k0 = s * 32 + (lane >> 4) * 8;
    bf16x8 v;
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = static_cast<__bf16>(0.f);
    if (mine && srow < a.src_rows && k0 < a.K) v = *reinterpret_cast<const bf16x8*>(a.src + size_t(srow) * a.K + k0);
    const size_t f = size_t(stream_frag_index(a.Nt, a.Ks, a.NB, a.nwg, t, s));
    if (mine) reinterpret_cast<bf16x8*>(a.dst)[f * 64 + lane] = v;
    if (!a.planes) return;
    const size_t n = size_t(a.Nt) * a.Ks;
    const uint4v c = encode_weights(v, *a.base4 & 127u);
    if (mine) {
        *reinterpret_cast<unsigned long long*>(a.planes + f * 512 + lane * 8) = uint64_t(c[0]) | (uint64_t(c[1]) << 32);
        *reinterpret_cast<uint32_t*>(a.planes + n * 512 + f * 256 + lane * 4) = c[2];
        *reinterpret_cast<uint32_t*>(a.planes + n * 768 + f * 256 + lane * 4) = c[3];
    }
    // (a word is shared with other fragments and other tensors, which may be packed at the same time)
    const bool rest = __builtin_amdgcn_ballot_w64(mine && c[3] != 0u) != 0ull;
    auto mark = [&](unsigned long long* words, const FlagPlace& p) {
        if (rest) atomicOr(words + p.word, 1ull << p.bit);
        else atomicAnd(words + p.word, ~(1ull << p.bit));
    };
    if (lane == 0) {
        mark(a.fl, stream_flag(a.Nt, a.Ks, a.NB, a.nwg, t, s));
        if (a.gfl) mark(a.gfl, grouped_flag(a.Nt, a.Ks, a.nwg, t, s));
    }
}

// A workspace is prepared by clearing all of it (control words must start at zero; the kernel
// multiplies hand-over bytes it never wrote - rows beyond r, k-steps beyond a wavefront's share
// - with zero weights, so those bytes have to be finite) and setting the mark that says so.
__global__ __launch_bounds__(256) void k_ws_init(uint4v* ws, size_t n16, uint32_t* magic_word) {
    const size_t stride = size_t(gridDim.x) * 256;
    for (size_t i = size_t(blockIdx.x) * 256 + threadIdx.x; i < n16; i += stride) ws[i] = uint4v{0u, 0u, 0u, 0u};
    // the mark lives in a 16-byte unit that this same thread has just cleared
    const size_t mi = size_t(reinterpret_cast<char*>(magic_word) - reinterpret_cast<char*>(ws)) / 16;
    if (mi % stride == size_t(blockIdx.x) * 256 + threadIdx.x) *magic_word = kWsMagic;
}

// Cache construction, eqs. (3)-(7): score every (parent, top-k token) pair w = p * sigma(parent),
// pool the M * k tuples and keep the K best, best first; equal scores in (parent, rank) order.  Keys are
// unique and sorted in LDS (bitonic network) by one workgroup, which has read every input before it writes an
// output: the outputs may lie over the inputs.  Bound by the latency of the network's steps, 55 for 1024 keys;
// a wavefront compares pairs of its own 128 keys, so only steps of larger distance need a barrier.
// M = 100, k = 8, K = 100, a call among others: 10 us; keys ranked by many workgroups that each count the larger ones 14
// (and no output over an input); K rounds of "largest key left", two barriers each, 68.  M = 32, K = 50: 6.2; ranked 5.6.
constexpr int kSelMax = 2048;
struct SelectArgs {
    const float* sigma;     // [M] cumulative probability of each parent sequence, eq. (4)
    const int32_t* tok;     // [M][k] eq. (2)
    const float* prob;      // [M][k]
    int32_t M, k, K;
    int32_t* out_tok;       // [K]
    float* out_score;       // [K] eq. (3)
    int32_t* out_parent;    // [K]
};

__global__ __launch_bounds__(kSelMax / 2) void k_cache_select(SelectArgs a) {
    __shared__ unsigned long long keys[kSelMax];
    __shared__ int toks[kSelMax];
    const int tid = threadIdx.x, total = a.M * a.k, n = 2 * blockDim.x;  // n: a power of two
    for (int flat = tid; flat < n; flat += blockDim.x) {
        unsigned long long key = 0ull;  // an empty tuple
        const int tok = flat < total ? a.tok[flat] : -1;
        if (tok >= 0) {
            const float w = a.prob[flat] * a.sigma[flat / a.k];
            // non-negative floats order like their bit patterns; +1 keeps a zero score above "empty"
            key = ((static_cast<unsigned long long>(__float_as_uint(w)) + 1ull) << 32) | (0xffffffffu - uint32_t(flat));
        }
        keys[flat] = key;
        toks[flat] = tok;
    }
    for (int size = 2; size <= n; size <<= 1)
        for (int dist = size >> 1; dist > 0; dist >>= 1) {
            // this step touches other wavefronts' keys, or the step before did (or it was the load)
            if (dist >= 128 || (dist == 64 && size > 128) || size == 2) __syncthreads();
            const int lo = 2 * tid - (tid & (dist - 1)), hi = lo + dist;
            const unsigned long long x = keys[lo], y = keys[hi];
            if ((x < y) == ((lo & size) == 0)) {
                keys[lo] = y;
                keys[hi] = x;
            }
            asm volatile("" ::: "memory");
        }
    __syncthreads();
    const int n_out = a.K < total ? a.K : total;
    for (int j = tid; j < n_out; j += blockDim.x) {
        const unsigned long long key = keys[j];
        const int flat = int(0xffffffffu - uint32_t(key & 0xffffffffull));
        // fewer tuples than places: the rest is marked empty
        a.out_tok[j] = key != 0ull ? toks[flat] : -1;
        a.out_score[j] = key != 0ull ? __uint_as_float(uint32_t((key >> 32) - 1ull)) : 0.f;
        a.out_parent[j] = key != 0ull ? flat / a.k : -1;
    }
}

struct GatherArgs {
    const __bf16* kpool;
    const __bf16* vpool;
    const int32_t* block_table;
    int32_t first, count, n_kv_heads, head_dim;
    float* k_out;
    float* v_out;
};

__global__ __launch_bounds__(256) void k_kv_gather(GatherArgs a) {
    const int64_t id = int64_t(blockIdx.x) * 256 + threadIdx.x;
    const int h = a.head_dim;
    if (id >= int64_t(a.count) * a.n_kv_heads * h) return;
    const int j = int(id % h), head = int((id / h) % a.n_kv_heads), i = int(id / (int64_t(h) * a.n_kv_heads));
    const int slot = a.first + i;
    const int page = a.block_table[slot >> 4], tk = slot & 15;
    const size_t base = (size_t(page) * a.n_kv_heads + head) * (16 * h);
    a.k_out[id] = static_cast<float>(a.kpool[base + ((j >> 3) * 16 + tk) * 8 + (j & 7)]);
    a.v_out[id] = static_cast<float>(a.vpool[base + v_page_index(j, tk)]);
}

}  // namespace card
