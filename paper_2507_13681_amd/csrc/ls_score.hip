// Window scoring: attention of the newest query window over the whole context, reduced to
// per-column ("vertical") and per-diagonal ("slash") sums and maxima (Alg. 2: the softmax step,
// SlashSum and VerticalSum; Sec. 3.1 defines the two kinds of line).  The same kernels, in
// "column sums only, summed over the query heads of a KV head" mode, produce the retention score
// of Alg. 3 (Sec. 5.2).
//
// The softmax normaliser of a row is only known after all keys were seen, and the line sums mix
// rows with different normalisers, so the pass is split:
//   stats_kernel, range_stats_kernel   per (row, 128 keys), for the retention score per (row, range of keys): a reference and the sum of exp of the scaled logits against it;
//   merge_kernel   per row: global max m and 1/l;
//   lines_kernel   recomputes the logits, forms A = exp2(x - m) / l, and reduces it
//                  - over rows, in registers, to column sums / maxima (written once, in order);
//                  - over diagonals through an LDS copy of 32 rows of the 128-key slab at a time, one
//                    thread per diagonal adding the rows in fixed order; a diagonal crosses at most two
//                    key blocks, whose two partial results finish_kernel adds, or the block of the two that is done last.
// With explicit scoring positions (q_pos given) the diagonals of a slab are not a contiguous range: the
// matrix A is then written out, band by band of as many KV heads and rows as the workspace takes, and
// diagonals_kernel adds each diagonal's cells in row order, on from where the band before it stopped.
// Everything is summed in a fixed order, so results are bit-reproducible from run to run.
//
// Tile products run on 32x32 MFMA.  In lines_kernel and stats_kernel each wave owns 32 keys of a block, whose fragments it keeps in
// registers, and meets every query head of the KV group and every 32-row group with them.  Those chunks of 32 query rows
// come through LDS by global -> LDS transfers, two buffers, one barrier per chunk.  K rows go through LDS on
// their way to the registers as well: read straight from global memory a fragment load touches 32 rows with
// 32 bytes each.  What bounds lines_kernel is vector instruction issue (52 % of all SIMD cycles at 131072 keys, 4 cycles each)
// and LDS: what counts is few instructions (no masks where every row sees every key, no address arithmetic in the diagonal sums), and little enough
// LDS (33 to 38 KB) for four workgroups per CU.  Whole windows of 64 rows in LDS (100 KB, one workgroup per CU),
// as one step: 131072 keys 832 us, by chunks 310; retention score, 16384 keys, B 4: 102 us, by chunks 43.
#include <type_traits>

#include "ls_device.h"
#include "ls_internal.h"

namespace ls {

constexpr int SB = 128;           // keys per block
constexpr int SCORE_THREADS = 256;
constexpr int SLAB = 33;          // floats per diagonal of the LDS slab: 32 rows, odd so that neighbouring diagonals lie in
constexpr int SLAB_DIAGS = SB + 31;   // neighbouring banks; key k of row r lies on diagonal k - r + 31.  The cells no key falls into stay zero
constexpr int SLAB_BYTES = (SLAB_DIAGS * SLAB * 4 + 15) / 16 * 16;
constexpr int RED_CHUNKS = 8;     // chunks whose wave results stats_kernel keeps before merging them

// 32 rows of T x D in LDS, row-major, the 8-element fragment units of a row XOR-swizzled with the row so that
// the rows one fragment read touches fall into different banks; filled by transfers of 1 KB.
template <typename T, int D>
struct RowTile {
    static constexpr int FB = 8 * Elem<T>::bytes;         // bytes of one fragment unit
    static constexpr int UPR = D / 8;                     // units per row
    static constexpr int RB = D * Elem<T>::bytes;         // bytes per row
    static constexpr int BYTES = 32 * RB;
    static constexpr int SPR = RB / 16;                   // 16-byte slots per row
    static constexpr int RPI = 64 / SPR > 0 ? 64 / SPR : 1;   // rows per transfer
    static constexpr int NI = BYTES / 1024;               // transfers
    static_assert(SPR <= 64, "a row fits one transfer");
    // transfers first, first + step, ... of the tile; row r of it comes from src + min(r, rows - 1) * RB
    __device__ static void fetch(const unsigned char* src, int rows, uint32_t lds, int lane, int first, int step) {
        const int tr = lane / SPR, sl = lane % SPR;
        src = uniform_ptr(src);
        lds = (uint32_t)__builtin_amdgcn_readfirstlane((int)lds);
        for (int i = first; i < NI; i += step) {
            const int row = RPI * i + tr;
            const int u = FB == 16 ? sl ^ (row & (UPR - 1)) : 2 * ((sl >> 1) ^ (row & (UPR - 1))) + (sl & 1);
            dma16(src, (uint32_t)((row < rows ? row : rows - 1) * RB + 16 * u), lds + (uint32_t)(i * 1024));
        }
    }
    __device__ static void frags(Frag<T> (&f)[D / 16], const unsigned char* tile, int row, int g) {
#pragma unroll
        for (int c = 0; c < D / 16; ++c) load_frag(f[c], tile + row * RB + FB * ((2 * c + g) ^ (row & (UPR - 1))));
    }
};

__device__ __forceinline__ uint32_t lds_address(const void* p) { return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const unsigned char*)p; }

// The rows of a KV head's G windows in chunks of up to 32: chunk c covers the rows start .. start + cnt - 1 of the
// G * w rows, which lie one after the other in memory.  Windows of 8 or 16 rows share a chunk with their neighbours
// (`packed`); otherwise a chunk stays inside one head's window.
struct Chunk { int start, cnt, t0; };         // t0: window row of the first one (row r of the chunk: (t0 + r) % w)
struct Chunks {
    int w, rows, rgs, count, first, end;      // `first`: window row at which a head's chunks begin; they reach row end - 1
    __host__ __device__ __forceinline__ Chunks(int w_, int G, bool packed) : w(w_), rows(G * w_), rgs(packed ? 0 : (w_ + 31) / 32), count(packed ? (G * w_ + 31) / 32 : G * ((w_ + 31) / 32)), first(0), end(w_) {}
    // the chunks that hold window rows t0 .. t1 - 1
    __device__ __forceinline__ Chunks(int w_, int G, int t0, int t1) : w(w_), rows(G * w_), rgs((t1 + 31) / 32 - t0 / 32), count(G * rgs), first(t0 & ~31), end(t1) {}
    __device__ __forceinline__ Chunk at(int c) const {
        if (rgs == 0) { const int s = 32 * c; return {s, rows - s < 32 ? rows - s : 32, 0}; }
        const int h = c / rgs, r0 = first + 32 * (c - h * rgs);
        return {h * w + r0, w - r0 < 32 ? w - r0 : 32, r0};
    }
};
// The accumulator registers of a product hold its rows in groups of eight, so that a head of 8 or 16 rows ends with a group and
// its sums can be taken there; one of 1, 2 or 4 rows would end inside a group.  ls_kv_compress, B 4, 64 / 8 heads of 128, 16384
// keys, a chunk a head / packed: 16 rows 148 / 90 us, 8 rows 147 / 74; 4 rows 145.
__host__ __device__ static bool packs(int w) { return w == 8 || w == 16; }

// This wave's K fragments of 32 keys, through its own 32 rows of LDS (keys beyond the context repeat the last one; every
// row's mask excludes them)
template <typename T, int D>
__device__ __forceinline__ void k_frags(Frag<T> (&kf)[D / 16], const T* Kg, int64_t key0, int64_t n, unsigned char* stage, int lane) {
    using RT = RowTile<T, D>;
    const int64_t left = n - key0;
    const int64_t k0 = left > 0 ? key0 : n - 1;
    RT::fetch(reinterpret_cast<const unsigned char*>(Kg + k0 * D), left > 32 ? 32 : left > 0 ? (int)left : 1, lds_address(stage), lane, 0, 1);
    wait_transfers();
    RT::frags(kf, stage, lane & 31, lane >> 5);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");     // the stage may be filled again
}

// dynamic LDS ahead of the per-row arrays: the K stage, and what later takes its place
template <typename T, int D>
__host__ __device__ constexpr int stats_front() {
    using RT = RowTile<T, D>;
    return 4 * RT::BYTES > 2 * RT::BYTES + RED_CHUNKS * 1024 ? 4 * RT::BYTES : 2 * RT::BYTES + RED_CHUNKS * 1024;
}
template <typename T, int D>
__host__ __device__ constexpr int lines_front(int mode) {
    using RT = RowTile<T, D>;
    return (mode != 0 && mode != 4) || 2 * RT::BYTES > SLAB_BYTES ? 4 * RT::BYTES : 2 * RT::BYTES + SLAB_BYTES;
}
// the larger / the sum of this lane's and lane ^ 32's value
__device__ __forceinline__ float halves_max(float x) {
    const auto b = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, x), __builtin_bit_cast(uint32_t, x), false, false);
    return fmaxf(__builtin_bit_cast(float, (uint32_t)b[0]), __builtin_bit_cast(float, (uint32_t)b[1]));
}
__device__ __forceinline__ float halves_sum(float x) {
    const auto b = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, x), __builtin_bit_cast(uint32_t, x), false, false);
    return __builtin_bit_cast(float, (uint32_t)b[0]) + __builtin_bit_cast(float, (uint32_t)b[1]);
}

// What the key blocks of a head leave each other (MODE 4 of lines_kernel).  Block kb and the next share the w - 1 diagonals from
// omin(kb) on: two sides' {sum, maximum}; a head's total has shares of so many blocks each (as in finish_kernel: the same sums in the same order); and for each KV head and share of
// its heads the counts of two neighbours that are done, and of the blocks of a share (all counting in one place, which lies in one line of memory for 32 heads, took
// 8 ns each: 16 heads of 20000 keys 50 us instead of 30).  All of it takes no more than 16 bytes a head and key.
constexpr int FINISH_SPLIT = 8;            // shares of a total
__host__ __device__ __forceinline__ int64_t share_keys(int64_t n) { return ((n + FINISH_SPLIT - 1) / FINISH_SPLIT + 1023) / 1024 * 1024; }      // whole rounds of 1024
__device__ __forceinline__ int edge_groups(const ScoreArgs& a) { const int blocks = (int)(share_keys(a.n) / SB); return (a.nkb + blocks - 1) / blocks; }
__device__ __forceinline__ int edge_counters(const ScoreArgs& a) { return a.nkb - 1 + edge_groups(a); }
__device__ __forceinline__ float* edge(const ScoreArgs& a, int bh, int kb, int side) { return a.spart + (((int64_t)bh * (a.nkb - 1) + kb) * 2 + side) * (2 * (a.w - 1)); }
__device__ __forceinline__ float* edge_share(const ScoreArgs& a, int bh) { return a.spart + (int64_t)a.BH * (a.nkb - 1) * (4 * (a.w - 1)) + (int64_t)bh * edge_groups(a); }
__device__ __forceinline__ uint32_t* edge_done(const ScoreArgs& a, int bk, int share) {
    return reinterpret_cast<uint32_t*>(edge_share(a, a.BH)) + ((int64_t)bk * a.shares + share) * edge_counters(a);
}
// by the first workgroup of a KV head that gets to stats_kernel, for the kernels behind it
__device__ __forceinline__ void clear_counters(const ScoreArgs& a, int bk, int tid) {
    if (a.done) for (int h = tid; h < a.G; h += SCORE_THREADS) clear_shared(a.done + bk * a.G + h);
    if (a.join) for (int i = tid; i < a.shares * edge_counters(a); i += SCORE_THREADS) clear_shared(edge_done(a, bk, 0) + i);
}

// a share of a total from what 16 times 64 places of its range have, and the total from its shares
__device__ __forceinline__ float share_of(float (&r)[16]) {
#pragma unroll
    for (int s = 8; s > 0; s >>= 1)
#pragma unroll
        for (int w = 0; w < s; ++w) r[w] += r[w + s];
    return wave_sum(r[0]);
}
__device__ __forceinline__ float total_of(const float (&p)[FINISH_SPLIT]) { return ((p[0] + p[1]) + (p[2] + p[3])) + ((p[4] + p[5]) + (p[6] + p[7])); }

// window row t's position in the context
__device__ __forceinline__ int position_of(const ScoreArgs& a, int t) {
    int64_t p = a.q_pos ? a.q_pos[t] : a.n - a.w + t;
    if (p > a.n - 1) p = a.n - 1;                          // positions outside the context are clipped
    return (int)(p < -1 ? -1 : p);
}

// ---- pass 1: per row max and sum of exp2 over a range or a block of keys -----------------------------------------
// The retention score's, bf16.  grid (ranges of keys, B*Hkv, shares of the heads).  part[(bk * a.parts + range) * G w + row] = {max, sum} over the range's keys.
// Bound by the reads of K where there are few rows, by vector and matrix issue where there are many.
// A wave keeps 32 or 64 query rows in registers and meets the tiles of its range with them, three buffers of 64 keys
// that the four waves fill and read together, the tile after the next under way at the barrier; a row is in a lane, and
// its sum stays there until the end.  No maximum is looked for on the way: the reference is the maximum of the first 32 keys and moves
// where a sum exceeds 2^30 (fp32 sums are as exact there; a reference of zero, with no look at the first keys, was not): three vector instructions a cell.
// Against a workgroup per 128 keys with all rows passing through LDS (nine instructions a cell, K of all resident workgroups asked for at once
// and nothing meanwhile, statistics of every 128 keys written), us: 16384 keys, B 4, 64 heads of 16 rows, 35 -> 27 (134 MB: 5 TB/s), 131072 keys, 32 heads of 128 rows, 193 -> 138.
// Everything in 56 KB of LDS, two workgroups a CU: 155 at 131072 keys.
template <int D>
struct KeyTile {
    static constexpr int KEYS = 64, BUFFERS = 3;
    static constexpr int RB = D * 2, DS = RB / 16, RPI = 64 / DS, NI = KEYS / RPI, IPW = NI / 4;
    static constexpr int ISTR = D == 128 ? 1088 : 1024;   // LDS bytes from one transfer to the next
    static constexpr int BYTES = NI * ISTR, HALF = BYTES / 2;
    static constexpr int KA = D == 128 ? 2 : 4;           // fragment address registers
    // slot s of row r holds chunk s ^ swz(r): a fragment read touches every bank once a pass
    __device__ static constexpr int swz(int row) { return D == 128 ? (row & 3) : (((row >> 1) & 3) | (((row >> 3) & 1) << 2)); }
};
constexpr int STATS_CHUNKS = 8;           // chunks of 32 rows of a workgroup
constexpr float STATS_LIMIT = 1073741824.f;
template <int D>
__host__ __device__ constexpr int stats_lds() { return KeyTile<D>::BUFFERS * KeyTile<D>::BYTES; }

//
// BLOCKS (the scores of a turn): the same way past the keys, but statistics of every 128 keys, in stats_kernel's operations and order (stats_split).
template <int D, bool BLOCKS>
__global__ __launch_bounds__(SCORE_THREADS, 3) void range_stats_kernel(ScoreArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    using C = KeyTile<D>;
    using T = bf16_t;
    constexpr int NS = D / 16;
    float2 (*red)[STATS_CHUNKS][32] = reinterpret_cast<float2 (*)[STATS_CHUNKS][32]>(smem);      // [2 halves of a tile], once the tiles are done with
    static_assert(C::BYTES >= 2 * STATS_CHUNKS * 32 * 8, "room for the waves' results");
    const int tid = threadIdx.x, lane = tid & 63, r32 = lane & 31, g = lane >> 5;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int bk = blockIdx.y, b = bk / a.Hkv, kvh = bk % a.Hkv;
    const int64_t n = a.n;
    const unsigned char* Kg = reinterpret_cast<const unsigned char*>(a.k) + (int64_t)bk * n * C::RB;
    const unsigned char* Q0 = reinterpret_cast<const unsigned char*>(a.q) + (int64_t)(b * a.Hq + kvh * a.G) * a.w * C::RB;
    const Chunks ch(a.w, a.G, packs(a.w));
    const int c0 = a.stat_chunks * (int)blockIdx.z, here = ch.count - c0 < a.stat_chunks ? ch.count - c0 : a.stat_chunks;
    // rows: waves side by side on chunks; few chunks: two waves share one, a half of each tile each (of one chunk, two waves only read K)
    const int rw = here > 2 ? 4 : here, kw = BLOCKS || here > 2 ? 1 : 2;
    const int kh = wv / rw;                                // where they share: this wave's half
    const bool works = kh < kw && wv % rw < here;          // (of three chunks, the fourth wave only reads K)
    const int cw = works ? wv % rw : 0;                    // its first chunk
    const int mine = !works ? 0 : cw + rw < here ? 2 : 1;  // chunks cw, cw + 4
    const int nt = (int)((n + C::KEYS - 1) / C::KEYS);
    constexpr int UNIT = BLOCKS ? SB / C::KEYS : 1;        // BLOCKS: whole blocks
    const uint32_t units = BLOCKS ? (uint32_t)a.nkb : (uint32_t)nt;
    const int t0 = UNIT * (int)range_begin(units, gridDim.x, blockIdx.x);
    int t1 = UNIT * (int)range_begin(units, gridDim.x, blockIdx.x + 1);
    if (t1 > nt) t1 = nt;
    if (BLOCKS && blockIdx.x == 0 && blockIdx.z == 0) clear_counters(a, bk, tid);

    // ---- transfers: wave wv fetches rows 16 wv .. 16 wv + 15 of a tile; keys beyond the context repeat the last one
    const int rowlane = 16 * wv + lane / C::DS, sl = lane % C::DS;
    const uint32_t part0 = 16u * (uint32_t)(sl ^ C::swz(rowlane));
    const uint32_t lds0 = lds_address(smem) + (uint32_t)(wv * C::IPW * C::ISTR);
    auto fetch = [&](int t, int buf) {
        const int64_t key0 = (int64_t)t * C::KEYS, left = n - key0;
        const int last = left < C::KEYS ? (int)left - 1 : C::KEYS - 1;
        const unsigned char* src = uniform_ptr(Kg + key0 * C::RB);
        const uint32_t dst = (uint32_t)__builtin_amdgcn_readfirstlane((int)(lds0 + (uint32_t)(buf * C::BYTES)));
#pragma unroll
        for (int i = 0; i < C::IPW; ++i) {
            const int row = rowlane + C::RPI * i;
            dma16(src, (uint32_t)(row < last ? row : last) * C::RB + (D == 128 ? part0 : part0 ^ (uint32_t)(64 * (i & 1))), dst + (uint32_t)(i * C::ISTR));
        }
    };
    fetch(t0, 0);
    // ---- the rows: fragments, by way of LDS like the keys (the last two buffers have a half for each wave), and the position each lane's row ends at
    const int x = C::swz(r32);
    int kaddr[C::KA];
#pragma unroll
    for (int j = 0; j < C::KA; ++j) kaddr[j] = (r32 / C::RPI) * C::ISTR + (r32 % C::RPI) * C::RB + 32 * (j ^ (x >> 1)) + 16 * (g ^ (x & 1));
    Frag<T> q[2][NS];
    int pos[2], start[2], cnt[2];
    const uint32_t stage = (uint32_t)__builtin_amdgcn_readfirstlane((int)(lds_address(smem) + (uint32_t)(C::BYTES + wv * C::HALF)));
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const Chunk k = ch.at(c0 + (i < mine ? cw + rw * i : cw));
        start[i] = k.start; cnt[i] = k.cnt;
        if (i == 0 || mine == 2) {
            const unsigned char* src = uniform_ptr(Q0 + (int64_t)k.start * C::RB);
#pragma unroll
            for (int j = 0; j < C::NI / 2; ++j) {
                const int row = lane / C::DS + C::RPI * j;
                dma16(src, (uint32_t)(row < k.cnt ? row : k.cnt - 1) * C::RB + 16u * (uint32_t)(sl ^ C::swz(row)), stage + (uint32_t)(j * C::ISTR));
            }
            wait_transfers();
#pragma unroll
            for (int c = 0; c < NS; ++c) load_frag(q[i][c], smem + C::BYTES + wv * C::HALF + kaddr[c & (C::KA - 1)] + 32 * (c & ~(C::KA - 1)));
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");     // the stage may be filled again
        }
        int t = k.t0 + r32;
        if (ch.rgs == 0) t &= a.w - 1;                     // packed windows: w is a power of two
        pos[i] = t < a.w ? position_of(a, t) : INT_MAX;  // (rows that are none: not kept)
    }
    wait_transfers();
    __syncthreads();                                       // the stages are free
    if (t0 + 1 < t1) fetch(t0 + 1, 1);
    const float sc = a.scale_log2e;
    float mneg[2] = {INFINITY, INFINITY}, l[2] = {0.f, 0.f};      // reference of the lane's row in base 2, negated (+inf: no cell seen yet), and the sum against it
    // BLOCKS: {max, sum} of a block's halves of 32 keys, those of its first tile and those of its second; a lane of the first 32 has the first half of each, one of the others the second
    float2 one[2], two[2] = {make_float2(-INFINITY, 0.f), make_float2(-INFINITY, 0.f)};
    int buf = 0;
    for (int t = t0; t < t1; ++t) {
        // this wave's transfers of tile t have landed (those of the next are under way), and every wave is done with the tile before
        if (t + 1 < t1) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(C::IPW) : "memory"); else wait_transfers();
        lds_barrier();
        const int next = buf + 2 < 3 ? buf + 2 : buf - 1;
        if (t + 2 < t1) fetch(t + 2, next);
        const int64_t key0 = (int64_t)t * C::KEYS;
        const bool open = __ballot((pos[0] < pos[1] ? pos[0] : pos[1]) < (int)key0 + C::KEYS - 1) == 0ull;      // this wave's rows see every key (of a context: n is an int's)
        auto half = [&](int h, auto TWO, auto OPEN) {
            constexpr int N = decltype(TWO)::value ? 2 : 1;
            const unsigned char* base = smem + buf * C::BYTES + h * C::HALF;
            f32x16 s[N];
            {
                Frag<T> kf[NS];
                constexpr int AHEAD = 4;
#pragma unroll
                for (int c = 0; c < AHEAD; ++c) load_frag(kf[c], base + kaddr[c & (C::KA - 1)] + 32 * (c & ~(C::KA - 1)));
#pragma unroll
                for (int i = 0; i < N; ++i)
#pragma unroll
                    for (int r = 0; r < 16; ++r) s[i][r] = 0.f;
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int c = 0; c < NS; ++c) {
#pragma unroll
                    for (int i = 0; i < N; ++i) mma(s[i], kf[c], q[i][c]);           // s[r] = <k_{8(r/4)+4g+r%4}, q_row>
                    if (c + AHEAD < NS) load_frag(kf[c + AHEAD], base + kaddr[(c + AHEAD) & (C::KA - 1)] + 32 * ((c + AHEAD) & ~(C::KA - 1)));
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
#pragma unroll
            for (int i = 0; i < N; ++i) {
                if constexpr (!decltype(OPEN)::value) {
                    const int lim = pos[i] - ((int)key0 + 32 * h + 4 * g);           // register r holds key 4g + 8(r/4) + r%4 of the half
                    if (__ballot(lim >= 0) == 0ull) continue;
#pragma unroll
                    for (int r = 0; r < 16; ++r) if (8 * (r >> 2) + (r & 3) > lim) s[i][r] = -INFINITY;
                }
                if constexpr (BLOCKS) {
                    float mx = -INFINITY;
#pragma unroll
                    for (int r = 0; r < 16; ++r) { s[i][r] *= sc; mx = fmaxf(mx, s[i][r]); }
                    mx = halves_max(mx);
                    const float ms = mx == -INFINITY ? 0.f : mx;
                    float sum = 0.f;
#pragma unroll
                    for (int r = 0; r < 16; ++r) sum += fast_exp2(s[i][r] - ms);
                    sum = halves_sum(sum);
                    if (g == h) two[i] = make_float2(mx, sum);
                    continue;
                }
                float s0 = 0.f, s1 = 0.f;
#pragma unroll
                for (int r = 0; r < 16; r += 2) {
                    s0 += fast_exp2(__builtin_fmaf(s[i][r], sc, mneg[i]));
                    s1 += fast_exp2(__builtin_fmaf(s[i][r + 1], sc, mneg[i]));
                }
                float sum = s0 + s1;
                if (__ballot(!(sum <= STATS_LIMIT)) != 0ull) {     // once more against the maximum (a row's first cells: mneg = inf)
                    float mx = -INFINITY;
#pragma unroll
                    for (int r = 0; r < 16; ++r) mx = fmaxf(mx, s[i][r] * sc);
                    const float m = fmaxf(mx, -mneg[i]);
                    l[i] *= m > -INFINITY ? fast_exp2(-mneg[i] - m) : 1.f;
                    mneg[i] = -m;
                    const float safe = m > -INFINITY ? -m : 0.f;
                    sum = 0.f;
#pragma unroll
                    for (int r = 0; r < 16; ++r) sum += fast_exp2(__builtin_fmaf(s[i][r], sc, safe));
                }
                l[i] += sum;
            }
        };
        auto tile = [&](auto TWO, auto OPEN) { for (int h = kh; h < 2; h += kw) half(h, TWO, OPEN); };
        if (mine == 2) { if (open) tile(std::true_type{}, std::true_type{}); else tile(std::true_type{}, std::false_type{}); }
        else if (mine == 1) { if (open) tile(std::false_type{}, std::true_type{}); else tile(std::false_type{}, std::false_type{}); }
        buf = buf + 1 < 3 ? buf + 1 : 0;
        if (BLOCKS) {
            if ((t & 1) == 0) { one[0] = two[0]; one[1] = two[1]; two[0] = two[1] = make_float2(-INFINITY, 0.f); }
            if ((t & 1) != 0 || t + 1 == t1) {             // the block's last tile: four halves, in order
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    if (i >= mine) break;
                    const float M = halves_max(fmaxf(one[i].x, two[i].x)), Ms = M == -INFINITY ? 0.f : M;
                    const float u = one[i].y * fast_exp2(one[i].x - Ms), v = two[i].y * fast_exp2(two[i].x - Ms);
                    const auto uu = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, u), __builtin_bit_cast(uint32_t, u), false, false);
                    const auto vv = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, v), __builtin_bit_cast(uint32_t, v), false, false);
                    const float L = ((__builtin_bit_cast(float, (uint32_t)uu[0]) + __builtin_bit_cast(float, (uint32_t)uu[1])) + __builtin_bit_cast(float, (uint32_t)vv[0])) + __builtin_bit_cast(float, (uint32_t)vv[1]);
                    if (lane < cnt[i]) reinterpret_cast<float2*>(a.part)[((int64_t)bk * a.nkb + (t >> 1)) * (a.G * a.w) + start[i] + lane] = make_float2(M, L);
                    two[i] = make_float2(-INFINITY, 0.f);
                }
            }
        }
    }
    wait_transfers();                                      // (none is under way)
    if (BLOCKS) return;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        if (i >= mine) break;
        const float m = -mneg[i], M = halves_max(m);
        const float sum = halves_sum(m > -INFINITY ? l[i] * fast_exp2(m - M) : 0.f);
        if (g == 0) red[kh][cw + rw * i][r32] = make_float2(M, sum);
    }
    __syncthreads();
    const int c = tid >> 5;
    if (c < here) {
        const Chunk k = ch.at(c0 + c);
        float2 v = red[0][c][r32];
        if (kw == 2) {
            const float2 u = red[1][c][r32];
            const float M = fmaxf(v.x, u.x), Ms = M > -INFINITY ? M : 0.f;
            v = make_float2(M, v.y * fast_exp2(v.x - Ms) + u.y * fast_exp2(u.x - Ms));
        }
        if (r32 < k.cnt) reinterpret_cast<float2*>(a.part)[((int64_t)bk * a.parts + blockIdx.x) * (a.G * a.w) + k.start + r32] = v;
    }
}
// Per (row, key block) max and sum, the scores of short turns and of fp32: a workgroup per 128 keys, which it keeps in registers while the chunks of rows pass.  grid (nkb, B*Hkv, shares
// of the G heads).  part[(bk * nkb + kb) * G w + row].  (These sums are taken in one order, whichever kernel does it: another one, as the retention score's, moves a head's last line now and
// then, of 256 heads of 16384 keys one in 250, of 32 of 131072 one in 30, and with it rows of the output that are not the same any more.)
template <typename T, int D>
__global__ __launch_bounds__(SCORE_THREADS, (Elem<T>::bytes == 2 ? 4 : 1)) void stats_kernel(ScoreArgs a) {
    using RT = RowTile<T, D>;
    extern __shared__ __align__(16) unsigned char smem[];
    unsigned char* kst = smem;                             // [4 waves] K rows on their way to registers, then
    unsigned char* qs = smem;                              // [2] chunks of queries and
    float2 (*red)[4][32] = reinterpret_cast<float2 (*)[4][32]>(smem + 2 * RT::BYTES);   // [RED_CHUNKS] results of the waves
    int32_t* pos = reinterpret_cast<int32_t*>(smem + stats_front<T, D>());              // [w]
    const int tid = threadIdx.x, lane = tid & 63, r32 = lane & 31, g = lane >> 5;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kb = blockIdx.x, bk = blockIdx.y;
    const int b = bk / a.Hkv, kvh = bk % a.Hkv;
    const int64_t n = a.n;
    const T* Kg = reinterpret_cast<const T*>(a.k) + (int64_t)bk * n * D;
    const unsigned char* Q0 = reinterpret_cast<const unsigned char*>(a.q) + (int64_t)(b * a.Hq + kvh * a.G) * a.w * RT::RB;
    const Chunks ch(a.w, a.G, packs(a.w));
    const int c0 = ch.count / (int)gridDim.z * (int)blockIdx.z, c1 = c0 + ch.count / (int)gridDim.z;
    const uint32_t qs_lds = lds_address(qs);
    auto fetch = [&](int c) {
        const Chunk k = ch.at(c);
        RT::fetch(Q0 + (int64_t)k.start * RT::RB, k.cnt, qs_lds + (uint32_t)((c & 1) * RT::BYTES), lane, wv, 4);
    };
    for (int t = tid; t < a.w; t += SCORE_THREADS) pos[t] = position_of(a, t);
    Frag<T> kf[D / 16];
    k_frags<T, D>(kf, Kg, (int64_t)kb * SB + 32 * wv, n, kst + wv * RT::BYTES, lane);
    __syncthreads();
    fetch(c0);
    if (c0 + 1 < c1) fetch(c0 + 1);
    // every key of the block is visible to every row of a contiguous window: no masks (all but the last blocks)
    const bool open = a.q_pos == nullptr && (int64_t)(kb + 1) * SB - 1 <= n - a.w;
    const int rows = a.G * a.w;
    if (kb == 0 && blockIdx.z == 0) clear_counters(a, bk, tid);
    wait_transfers();
    __syncthreads();
    int first = c0;                                        // first chunk whose wave results are still in `red`
    for (int c = c0; c < c1; ++c) {
        const Chunk k = ch.at(c);
        f32x16 s;
        {
            Frag<T> qf[D / 16];
            RT::frags(qf, qs + (c & 1) * RT::BYTES, r32, g);
#pragma unroll
            for (int r = 0; r < 16; ++r) s[r] = 0.f;
#pragma unroll
            for (int cc = 0; cc < D / 16; ++cc) mma(s, kf[cc], qf[cc]);      // s[r] = <k_{8(r/4)+4g+r%4}, q_row>
        }
        float mx = -INFINITY;
        if (open) {
#pragma unroll
            for (int r = 0; r < 16; ++r) { s[r] *= a.scale_log2e; mx = fmaxf(mx, s[r]); }
        } else {
            int t = k.t0 + r32;
            if (ch.rgs == 0) t &= a.w - 1;                 // packed windows: w is a power of two
            const int p = t < a.w ? pos[t] : -1;
            const int64_t lim64 = (int64_t)p - ((int64_t)kb * SB + 32 * wv) - 4 * g;      // register r holds key 4g + 8(r/4) + r%4
            const int lim = lim64 < -1 ? -1 : (lim64 > 64 ? 64 : (int)lim64);
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const float x = (8 * (r >> 2) + (r & 3) <= lim) ? s[r] * a.scale_log2e : -INFINITY;
                s[r] = x;
                mx = fmaxf(mx, x);
            }
        }
        mx = halves_max(mx);
        const float ms = (mx == -INFINITY) ? 0.f : mx;
        float sum = 0.f;
#pragma unroll
        for (int r = 0; r < 16; ++r) sum += fast_exp2(s[r] - ms);
        sum = halves_sum(sum);
        if (g == 0) red[c - first][wv][r32] = make_float2(mx, sum);
        wait_transfers();                                  // chunk c + 1
        __syncthreads();
        if (c + 2 < c1) fetch(c + 2);
        if (c - first == RED_CHUNKS - 1 || c == c1 - 1) {
            for (int i = tid; i < (c - first + 1) * 32; i += SCORE_THREADS) {
                const int r = i & 31, cc = i >> 5;
                const Chunk kk = ch.at(first + cc);
                if (r >= kk.cnt) continue;
                float2 v[4];
                float M = -INFINITY;
#pragma unroll
                for (int w4 = 0; w4 < 4; ++w4) { v[w4] = red[cc][w4][r]; M = fmaxf(M, v[w4].x); }
                const float Ms = (M == -INFINITY) ? 0.f : M;
                float L = 0.f;
#pragma unroll
                for (int w4 = 0; w4 < 4; ++w4) L += v[w4].y * fast_exp2(v[w4].x - Ms);
                reinterpret_cast<float2*>(a.part)[((int64_t)bk * a.parts + kb) * rows + kk.start + r] = make_float2(M, L);
            }
            first = c + 1;
            if (first < c1) __syncthreads();         // `red` is written again
        }
    }
}

// ---- merge: sixteen rows per workgroup; 64 threads of a row stride over the key blocks, then a fixed butterfly ----
// grid (rows of a KV head / 16, B*Hkv).  Bound by the reads of `part`, and where there are few by its steps (shuffles through LDS instead of DPP, and a barrier more
// for each: merge and finish together 0.4 to 0.6 us more): the threads of sixteen neighbouring rows read 128
// contiguous bytes (a wave per two rows, 16 bytes at a time: 25 us at 131072 keys).
__global__ __launch_bounds__(1024) void merge_kernel(ScoreArgs a) {
    __shared__ float x[64][17], most[16];
    const int rows = a.G * a.w, bk = blockIdx.y;
    const int row = blockIdx.x * 16 + (threadIdx.x & 15), k0 = threadIdx.x >> 4;           // as a reader of `part`
    const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;                                // as a lane of row wv
    const float2* p = reinterpret_cast<const float2*>(a.part) + (int64_t)bk * a.parts * rows + (row < rows ? row : rows - 1);
    constexpr int KEEP = 4;                                // values a thread keeps from the first look (contexts up to 32768)
    float2 v[KEEP];
    float M = -INFINITY, L = 0.f;
#pragma unroll
    for (int i = 0; i < KEEP; ++i) {
        const int kb = k0 + 64 * i;
        v[i] = make_float2(-INFINITY, 0.f);
        if (kb < a.parts) v[i] = p[(int64_t)kb * rows];
    }
#pragma unroll
    for (int i = 0; i < KEEP; ++i) M = fmaxf(M, v[i].x);
#pragma unroll 4
    for (int kb = k0 + 64 * KEEP; kb < a.parts; kb += 64) M = fmaxf(M, p[(int64_t)kb * rows].x);
    x[k0][threadIdx.x & 15] = M;
    __syncthreads();
    M = x[lane][wv];
    M = wave_largest(M);
    if (lane == 0) most[wv] = M;
    __syncthreads();
    const float Mr = most[threadIdx.x & 15];
#pragma unroll
    for (int i = 0; i < KEEP; ++i)
        if (v[i].x != -INFINITY) L += v[i].y * fast_exp2(v[i].x - Mr);
#pragma unroll 4
    for (int kb = k0 + 64 * KEEP; kb < a.parts; kb += 64) {
        const float2 u = p[(int64_t)kb * rows];
        if (u.x != -INFINITY) L += u.y * fast_exp2(u.x - Mr);
    }
    x[k0][threadIdx.x & 15] = L;
    __syncthreads();
    L = x[lane][wv];
    L = wave_sum(L);
    if (lane == 0 && blockIdx.x * 16 + wv < rows)
        reinterpret_cast<float2*>(a.rowstat)[(int64_t)bk * rows + blockIdx.x * 16 + wv] = make_float2(M, L > 0.f ? 1.0f / L : 0.f);
}

// Short windows and contexts: lines_kernel merges the statistics of its rows itself, every workgroup again, which takes a launch away: the
// retention score of 4096 entries, 8 rows of 32 heads (2 MB read so) 22.6 -> 20.6 us.  Beyond a few MB that costs more than the launch: ls_score of 5003
// keys, d = 64 (10 MB) 35.8 -> 36.8, 8192 keys (50 MB) 38.2 -> 44.6.
constexpr int FOLD_PARTS = 64, FOLD_CHUNKS = 32;
constexpr int64_t FOLD_BYTES = 4 << 20;
static int score_chunks(const ScoreArgs& a) { return a.G * ((a.w + 31) / 32); }           // at most: packed windows take fewer
// LANES neighbouring lanes (one or four) share a row's ranges, sixteen each at most; all of them get {max, 1 / sum}.
template <int LANES>
__device__ __forceinline__ float2 row_stats(const ScoreArgs& a, int bk, int row, int part) {
    constexpr int PER = 16;
    const int rows = a.G * a.w;
    const float2* p = reinterpret_cast<const float2*>(a.part) + (int64_t)bk * a.parts * rows + row;
    float2 v[PER];
    float M = -INFINITY;
#pragma unroll
    for (int q = 0; q < PER / 4; ++q) {                    // as many loads at once as there are ranges
#pragma unroll
        for (int u = 4 * q; u < 4 * q + 4; ++u) v[u] = make_float2(-INFINITY, 0.f);
        if (4 * LANES * q < a.parts) {
#pragma unroll
            for (int u = 4 * q; u < 4 * q + 4; ++u) v[u] = p[(int64_t)(LANES * u + part < a.parts ? LANES * u + part : 0) * rows];
        }
    }
#pragma unroll
    for (int u = 0; u < PER; ++u) if (LANES * u + part >= a.parts) v[u] = make_float2(-INFINITY, 0.f);
#pragma unroll
    for (int u = 0; u < PER; ++u) M = fmaxf(M, v[u].x);
    if (LANES == 4) {
        M = fmaxf(M, __shfl_xor(M, 1, 64));
        M = fmaxf(M, __shfl_xor(M, 2, 64));
    }
#pragma unroll
    for (int u = 0; u < PER; ++u) v[u].y = v[u].x != -INFINITY ? v[u].y * fast_exp2(v[u].x - M) : 0.f;
#pragma unroll
    for (int off = PER / 2; off > 0; off >>= 1)            // (merge_kernel's order)
#pragma unroll
        for (int u = 0; u < off; ++u) v[u].y += v[u + off].y;
    float L = v[0].y;
    if (LANES == 4) {
        L += __shfl_xor(L, 2, 64);
        L += __shfl_xor(L, 1, 64);
    }
    return make_float2(M, L > 0.f ? 1.0f / L : 0.f);
}

// ---- pass 2 of the retention score with few rows: all of them stay in LDS, the keys come by ----------------
// grid (workgroups that share a KV head's key blocks, B*Hkv).  Bound by the reads of K.  A wave has its 32 keys of a block in registers and those of
// the workgroup's next block on their way to its own stage; between blocks nobody waits for anybody.  Against a workgroup per block past which the chunks
// come, a barrier each, us: 16384 entries, B 4, 128 rows a KV head 39 -> 31, 32768, B 2, d = 64 18.4 -> 13.8, 65536, 8 KV heads of 16 rows 26 -> 21.
// Two chunks at once: B 4, 64 / 8 heads of 16384 entries, 16 rows 32.0 -> 30.2 us (134 MB: 4.4 TB/s), the whole ls_kv_compress 85.0 -> 83.4; 32768 entries, B 1, 52.8 -> 52.2.  (The products of one chunk beside
// the probabilities of the one before, 193 registers: the same, the reads of K bound it.)
// Four chunks of 32 rows: room for eight leaves a CU one workgroup at d = 128.  The whole ls_kv_compress, four / eight, us: 128 rows 73 / 82; 192 129 / 123, 256 120 / 124, 32768 entries, B 1, 81 / 82.  At d = 64
// it leaves two, and more rows would gain: 192 99.6 / 79.2, 256 90.6 / 79.9, 32768 entries, B 1, 65 / 60.
constexpr int RETAIN_CHUNKS = 4;
template <int D>
__host__ __device__ constexpr int retain_lds() { return (4 + RETAIN_CHUNKS) * RowTile<bf16_t, D>::BYTES + RETAIN_CHUNKS * 32 * 8; }
// (The LDS leaves two workgroups a CU at d = 128, three at 64: no need for fewer than 256 registers.  A kernel of its own: inside lines_kernel, small retentions had its registers.)
template <int D>
__global__ __launch_bounds__(SCORE_THREADS, 2) void retain_kernel(ScoreArgs a) {
    using T = bf16_t;
    using RT = RowTile<T, D>;
    extern __shared__ __align__(16) unsigned char smem[];
    unsigned char* qs = smem + 4 * RT::BYTES;              // the chunks
    float2* rst = reinterpret_cast<float2*>(smem + (4 + RETAIN_CHUNKS) * RT::BYTES);          // max and 1 / sum of their rows
    const int tid = threadIdx.x, lane = tid & 63, r32 = lane & 31, g = lane >> 5;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int bk = a.bk0 + blockIdx.y, bh0 = bk * a.G;     // (heads of a KV head lie together)
    const int64_t n = a.n;
    const unsigned char* Kg = reinterpret_cast<const unsigned char*>(a.k) + (int64_t)bk * n * RT::RB;
    const unsigned char* Q0 = reinterpret_cast<const unsigned char*>(a.q) + (int64_t)bh0 * a.w * RT::RB;
    const Chunks ch(a.w, a.G, packs(a.w));
    unsigned char* stage = smem + wv * RT::BYTES;
    auto fetch = [&](int kb) {                             // keys beyond the context repeat the last one
        const int64_t key0 = (int64_t)kb * SB + 32 * wv, left = n - key0;
        RT::fetch(Kg + (left > 0 ? key0 : n - 1) * RT::RB, left > 32 ? 32 : left > 0 ? (int)left : 1, lds_address(stage), lane, 0, 1);
    };
    int kb = blockIdx.x;
    fetch(kb);
    if (wv < ch.count) {
        const Chunk k = ch.at(wv);
        RT::fetch(Q0 + (int64_t)k.start * RT::RB, k.cnt, lds_address(qs + wv * RT::BYTES), lane, 0, 1);
        if (lane < 32) rst[32 * wv + lane] = lane < k.cnt ? reinterpret_cast<const float2*>(a.rowstat)[(int64_t)bh0 * a.w + k.start + lane] : make_float2(INFINITY, 0.f);      // (no row: probabilities of zero)
    }
    wait_transfers();
    __syncthreads();
    for (;;) {
        Frag<T> kf[D / 16];
        RT::frags(kf, stage, r32, g);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");         // the stage may be filled again
        const int here = kb;
        kb += (int)gridDim.x;
        if (kb < a.nkb) fetch(kb);
        const int64_t blk0 = (int64_t)here * SB, mykey = blk0 + 32 * wv + r32;
        const bool open = blk0 + SB - 1 <= n - a.w;        // every row sees every key
        float sum = 0.f;
        auto chunks = [&](auto OPEN) {
            // N chunks at once: two, whose products do not wait for each other, in a pinned order (as many registers as two workgroups a CU leave: 163; one at a time 106).
            // At d = 64, where a chunk's chain is half as long, one: the whole ls_kv_compress, two / one, us: B 2, 16 / 4 heads of 61338 entries, 16 rows 54.2 / 53.1, 65111, 8 / 2, 32 rows 43.8 / 42.6, B 4, 64 / 8, 16384 59.8 / 58.9.
            auto some = [&](auto COUNT, int c0) {
                constexpr int N = decltype(COUNT)::value, NS = D / 16, AHEAD = N == 1 ? NS : 2;
                f32x16 s[N];
#pragma unroll
                for (int i = 0; i < N; ++i)
#pragma unroll
                    for (int r = 0; r < 16; ++r) s[i][r] = 0.f;
                {
                    Frag<T> qf[NS][N];
                    auto load = [&](int cc, int i) { load_frag(qf[cc][i], qs + (c0 + i) * RT::BYTES + r32 * RT::RB + RT::FB * ((2 * cc + g) ^ (r32 & (RT::UPR - 1)))); };
#pragma unroll
                    for (int cc = 0; cc < AHEAD; ++cc)
#pragma unroll
                        for (int i = 0; i < N; ++i) load(cc, i);
                    if (N > 1) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int cc = 0; cc < NS; ++cc) {
#pragma unroll
                        for (int i = 0; i < N; ++i) mma(s[i], qf[cc][i], kf[cc]);    // s[r] = <q_{8(r/4)+4g+r%4}, k_lane>
                        if (cc + AHEAD < NS) {
#pragma unroll
                            for (int i = 0; i < N; ++i) load(cc + AHEAD, i);
                        }
                        if (N > 1) __builtin_amdgcn_sched_barrier(0);
                    }
                }
#pragma unroll
                for (int i = 0; i < N; ++i) {
                    const int c = c0 + i, t0 = ch.at(c).t0;
                    float ps = 0.f;                        // of the chunk: one sum through all chunks costs precision (128 rows of 65536 keys, relative error 1.14e-7, so 0.81e-7)
#pragma unroll
                    for (int q4 = 0; q4 < 4; ++q4) {
                        const int rq = 8 * q4 + 4 * g;
                        const f32x4 sa = *reinterpret_cast<const f32x4*>(rst + 32 * c + rq), sb = *reinterpret_cast<const f32x4*>(rst + 32 * c + rq + 2);
                        const float mm[4] = {sa.x, sa.z, sb.x, sb.z}, il[4] = {sa.y, sa.w, sb.y, sb.w};
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const float p = fast_exp2(__builtin_fmaf(s[i][4 * q4 + e], a.scale_log2e, -mm[e]));
                            if constexpr (decltype(OPEN)::value) ps = __builtin_fmaf(p, il[e], ps);
                            else {
                                int t = t0 + rq + e;
                                if (ch.rgs == 0) t &= a.w - 1; // packed windows: w is a power of two
                                ps += mykey <= n - a.w + t ? p * il[e] : 0.f;
                            }
                        }
                    }
                    sum += ps;
                }
            };
            int c = 0;
            if constexpr (D == 128) {
                for (; c + 2 <= ch.count; c += 2) some(std::integral_constant<int, 2>{}, c);
                if (c < ch.count) some(std::integral_constant<int, 1>{}, c);
            } else {
                for (; c < ch.count; ++c) some(std::integral_constant<int, 1>{}, c);
            }
        };
        if (open) chunks(std::true_type{}); else chunks(std::false_type{});
        sum = halves_sum(sum);
        if (g == 0 && mykey < n) a.gscore[(int64_t)bk * n + mykey] = sum;
        if (kb >= a.nkb) break;
        wait_transfers();                                  // this wave's keys of the next block
    }
}

// ---- pass 2: line sums ------------------------------------------------------------------------
// grid (nkb, KV heads from a.bk0 on, shares of the G heads; one share in mode 2)
// MODE 0: vert/vmax per head + diagonal partials (contiguous window, q_pos == NULL)
// MODE 1: vert/vmax per head + a band of the matrix A of these KV heads, [heads][t1 - t0][n], zero beyond each row's position.
//         The chunks that hold the band's rows are passed; their columns are added to those of the chunks before them.
// MODE 2: column sums only, summed over the G heads of the KV head (retention score)
// MODE 3: the matrix A only
// MODE 4: as 0; the block that is done last adds what it shares with its neighbours, and the total (joins)
// Four workgroups per CU leave bf16 128 registers (little data).  In MODE 0 and 4 what a row sees is arithmetic: with a table of the rows' limits in LDS, as for explicit
// positions, ls_score took, us, 131072 keys 464 instead of 448, 16384, B 4, 64 heads, 267 / 248, 32768 88 / 82, 8192 37.5 / 35.2, 61 rows of 12347, half
// of whose chunks have 29 rows, 51.5 / 47.9 (its reads beside the slab's, 13 more registers, four of them spilled).
template <typename T, int D, int MODE, bool FOLD>
__global__ __launch_bounds__(SCORE_THREADS, (Elem<T>::bytes == 2 ? 4 : 1)) void lines_kernel(ScoreArgs a) {
    using RT = RowTile<T, D>;
    constexpr bool LINES = MODE == 0 || MODE == 4;
    extern __shared__ __align__(16) unsigned char smem[];
    unsigned char* kst = smem;                             // [4 waves] K rows on their way to registers, then
    float* slab = reinterpret_cast<float*>(smem);          // [SLAB_DIAGS][SLAB] A by diagonals (MODE 0) and
    unsigned char* qs = smem + (LINES ? SLAB_BYTES : 0);           // [2] chunks of queries
    int32_t* ql = reinterpret_cast<int32_t*>(smem + lines_front<T, D>(MODE));    // [w] last visible key of a row, relative to the block
    float* rst = reinterpret_cast<float*>(ql + (a.w + 3) / 4 * 4);     // [2][32][2] max and 1 / sum of the chunks' rows (FOLD: of all chunks)
    const int tid = threadIdx.x, lane = tid & 63, r32 = lane & 31, g = lane >> 5;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kb = blockIdx.x, bk = a.bk0 + blockIdx.y;
    const int b = bk / a.Hkv, kvh = bk % a.Hkv;
    const int64_t n = a.n;
    const T* Kg = reinterpret_cast<const T*>(a.k) + (int64_t)bk * n * D;
    const int64_t blk0 = (int64_t)kb * SB;
    const int klocal = 32 * wv + r32;                      // this lane's key in the block
    const int64_t mykey = blk0 + klocal;
    const int bh0 = b * a.Hq + kvh * a.G;
    const unsigned char* Q0 = reinterpret_cast<const unsigned char*>(a.q) + (int64_t)bh0 * a.w * RT::RB;
    const float* st0 = a.rowstat + 2 * (int64_t)bh0 * a.w;
    const bool packed = MODE == 2 && packs(a.w);
    const Chunks ch = MODE == 1 ? Chunks(a.w, a.G, a.t0, a.t1) : Chunks(a.w, a.G, packed);
    const int c0 = ch.count / (int)gridDim.z * (int)blockIdx.z, c1 = c0 + ch.count / (int)gridDim.z;
    const uint32_t qs_lds = lds_address(qs), rst_lds = lds_address(rst);
    auto fetch = [&](int c) {
        const Chunk k = ch.at(c);
        RT::fetch(Q0 + (int64_t)k.start * RT::RB, k.cnt, qs_lds + (uint32_t)((c & 1) * RT::BYTES), lane, wv, 4);
        if (wv == 3 && !FOLD) dma4(uniform_ptr(st0), (uint32_t)(8 * (k.start + ((lane >> 1) < k.cnt ? lane >> 1 : k.cnt - 1)) + 4 * (lane & 1)), (uint32_t)__builtin_amdgcn_readfirstlane((int)(rst_lds + (uint32_t)((c & 1) * 256))));
    };
    if (!LINES) for (int t = tid; t < a.w; t += SCORE_THREADS) {
        const int64_t rel = position_of(a, t) - blk0;      // key klocal of the block is visible to row t iff klocal <= rel
        ql[t] = rel < -1 ? -1 : (rel > SB ? SB : (int32_t)rel);
    }
    if (FOLD) {
        auto stats = [&](auto LANES) {
            constexpr int N = decltype(LANES)::value;
            for (int i0 = tid; i0 < 32 * N * (c1 - c0); i0 += SCORE_THREADS) {
                const int i = i0 / N;
                const Chunk k = ch.at(c0 + i / 32);
                const float2 st = row_stats<N>(a, bk, k.start + (i % 32 < k.cnt ? i % 32 : k.cnt - 1), i0 % N);
                if (i0 % N == 0) reinterpret_cast<float2*>(rst)[i] = st;
            }
        };
        // (256 rows of 16 ranges by four lanes a row: the whole retention of 2048 entries 27.2 us instead of 25.1)
        if (a.parts <= 16) stats(std::integral_constant<int, 1>{}); else stats(std::integral_constant<int, 4>{});
    }
    Frag<T> kf[D / 16];
    k_frags<T, D>(kf, Kg, blk0 + 32 * wv, n, kst + wv * RT::BYTES, lane);
    __syncthreads();
    fetch(c0);
    if (c0 + 1 < c1) fetch(c0 + 1);
    if (LINES) for (int i = tid; i < SLAB_DIAGS * SLAB; i += SCORE_THREADS) slab[i] = 0.f;
    // every key of the block is visible to every row of a contiguous window (all but the last blocks)
    const bool open = a.q_pos == nullptr && blk0 + SB - 1 <= n - a.w;
    const int64_t omin = n - a.w - (blk0 + SB - 1);        // MODE 0, 4: this thread adds diagonal omin + tid of the slab (at most 255, w <= 128)
    float gsum = 0.f, vsum = 0.f, vmx = 0.f, dsum = 0.f, dmax = 0.f;
    wait_transfers();
    __syncthreads();
    for (int c = c0; c < c1; ++c) {
        const Chunk k = ch.at(c);
        const int bh = bh0 + k.start / a.w;                // head of the chunk (of its first row when packed)
        const float* rs = rst + (FOLD ? c - c0 : c & 1) * 64;
        if (MODE == 1 && ch.first > 0 && k.t0 == ch.first && mykey < n) {
            vsum = a.vert[(int64_t)bh * n + mykey];
            vmx = a.vmax[(int64_t)bh * n + mykey];
        }
        f32x16 s;
        {
            Frag<T> qf[D / 16];
            RT::frags(qf, qs + (c & 1) * RT::BYTES, r32, g);
#pragma unroll
            for (int r = 0; r < 16; ++r) s[r] = 0.f;
#pragma unroll
            for (int cc = 0; cc < D / 16; ++cc) mma(s, qf[cc], kf[cc]);      // s[r] = <q_{8(r/4)+4g+r%4}, k_lane>
        }
        float ps = 0.f, pm = 0.f;
        // of the chunk's rows, lo .. lo + cells - 1 are written out; `cell`: this lane's key in row 4 g
        const int lo = MODE == 1 && a.t0 > k.t0 ? a.t0 - k.t0 : 0;
        const int cells = (MODE == 1 && a.t1 - k.t0 < k.cnt ? a.t1 - k.t0 : k.cnt) - lo;
        float* cell = MODE == 1 || MODE == 3 ? a.a_win + ((int64_t)(bh - a.bh_first) * (a.t1 - a.t0) + k.t0 - a.t0 + 4 * g) * n + mykey : nullptr;
        // MODE 0, 4: the rows that see this lane's key are those from its own on, see + 4 g .. see + 4 g + seen - 1 of the chunk
        const int own = mykey - (n - a.w) - k.t0 > 0 ? (int)(mykey - (n - a.w)) - k.t0 : 0, see = own - 4 * g, seen = k.cnt > own ? k.cnt - own : 0;
        // MASKED: there are rows that do not exist (the last one is repeated) or keys that a row does not see
        auto rows = [&](auto MASKED) {
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4) {
                const int rq = 8 * q4 + 4 * g;             // registers 4*q4 .. 4*q4+3 hold the chunk's rows rq .. rq+3
                const f32x4 sa = *reinterpret_cast<const f32x4*>(rs + 2 * rq);            // m, 1/l of rows rq, rq+1
                const f32x4 sb = *reinterpret_cast<const f32x4*>(rs + 2 * rq + 4);        // ... rq+2, rq+3
                // (1 / sum in the exponent instead would take the product away, and cost six times the error: the offset has 2^-20 and more)
                float pe[4];
                const float mm[4] = {sa.x, sa.z, sb.x, sb.z}, il[4] = {sa.y, sa.w, sb.y, sb.w};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int row = rq + e;
                    float p = fast_exp2(MODE == 2 ? __builtin_fmaf(s[4 * q4 + e], a.scale_log2e, -mm[e]) : s[4 * q4 + e] * a.scale_log2e - mm[e]) * il[e];
                    if constexpr (decltype(MASKED)::value) {
                        if (LINES) p = (unsigned)(8 * q4 + e - see) < (unsigned)seen ? p : 0.f;
                        else {
                            int t = k.t0 + row;
                            if (MODE == 2 && packed) t &= a.w - 1;
                            p = ((row < k.cnt) & (klocal <= ql[t < a.w ? t : a.w - 1])) ? p : 0.f;
                        }
                    }
                    ps += p;
                    pe[e] = p;
                    if (LINES) slab[(klocal - row + 31) * SLAB + row] = p;
                    if ((MODE == 1 || MODE == 3) && (unsigned)(row - lo) < (unsigned)cells && mykey < n) cell[(8 * q4 + e) * n] = p;
                }
                if (LINES || MODE == 1) { pm = fmaxf(fmaxf(pm, pe[0]), pe[1]); pm = fmaxf(fmaxf(pm, pe[2]), pe[3]); }
                if (MODE == 2 && packed && (8 * (q4 + 1)) % a.w == 0) {                  // the last rows of a head
                    gsum += halves_sum(ps);                // (rows past the last head add zeros)
                    ps = 0.f;
                }
            }
        };
        if (open && k.cnt == 32) rows(std::false_type{}); else rows(std::true_type{});
        if (!(MODE == 2 && packed)) {
            vsum += halves_sum(ps);
            if (LINES || MODE == 1) vmx = fmaxf(vmx, halves_max(pm));
        }
        if (LINES) {
            lds_barrier();                                 // the slab is whole
            const int u = k.t0 + (SB - 1) - tid + 31;      // this thread's diagonal in the slab
            if (tid < SB - 1 + a.w && u >= 0 && u < SLAB_DIAGS) {
                int at = u * SLAB;
                asm("" : "+v"(at));                        // (one address for all reads, constants in their offsets)
                // rows in ascending order, sixteen reads in flight
#pragma unroll
                for (int rb = 0; rb < 32; rb += 16) {
                    float p[16];
#pragma unroll
                    for (int e = 0; e < 16; ++e) p[e] = slab[at + rb + e];
#pragma unroll
                    for (int e = 0; e < 16; e += 2) { dsum += p[e]; dsum += p[e + 1]; dmax = fmaxf(fmaxf(dmax, p[e]), p[e + 1]); }
                }
            }
        }
        wait_transfers();                                  // chunk c + 1
        __syncthreads();
        if (c + 2 < c1) fetch(c + 2);
        if (!(MODE == 2 && packed) && k.t0 + 32 >= ch.end) {   // the head's last chunk
            if (MODE == 2) gsum += vsum;
            if ((LINES || (MODE == 1 && a.sums)) && g == 0 && mykey < n) {
                if (MODE == 4) put_shared(a.vert + (int64_t)bh * n + mykey, vsum); else a.vert[(int64_t)bh * n + mykey] = vsum;
                a.vmax[(int64_t)bh * n + mykey] = vmx;
            }
            if (LINES) {
                const int64_t o = omin + tid;
                if (tid < SB - 1 + a.w && o >= 0) {        // the first w - 1 the next block has too, those from SB on the one before
                    if (MODE != 4) reinterpret_cast<float2*>(a.spart)[((int64_t)(kb & 1) * a.BH + bh) * n + o] = make_float2(dsum, dmax);
                    else if (tid < a.w - 1) put_shared2(edge(a, bh, kb, 0) + 2 * tid, dsum, dmax);
                    else if (tid >= SB && kb > 0) put_shared2(edge(a, bh, kb - 1, 1) + 2 * (tid - SB), dsum, dmax);
                    else { a.slash[(int64_t)bh * n + o] = dsum; a.smax[(int64_t)bh * n + o] = dmax; }
                }
                dsum = 0.f; dmax = 0.f;
            }
            vsum = 0.f; vmx = 0.f;
        }
    }
    if (MODE == 2 && g == 0 && mykey < n) a.gscore[(int64_t)bk * n + mykey] = gsum;
    if constexpr (MODE == 4) {
        // Of two neighbouring blocks the one that is done last adds the diagonals that they share, of a share's blocks the last one that share, of all
        // the last one the total; nobody waits for anybody.
        __shared__ uint32_t met[3];                        // how many were done before: of the block before and this one, of this one and the next, of the share
        const int heads = a.G / (int)gridDim.z, first = bh0 + heads * (int)blockIdx.z;
        const int blocks = (int)(share_keys(n) / SB), part = kb / blocks, left = a.nkb - part * blocks;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this wave's sides and columns are written
        __syncthreads();
        if (tid < 3) {
            const int at = tid == 2 ? a.nkb - 1 + part : kb - 1 + tid;
            met[tid] = tid == 2 || (at >= 0 && at < a.nkb - 1) ? count_shared(edge_done(a, bk, (int)blockIdx.z) + at) : 0u;
        }
        __syncthreads();
        const int each = a.w - 1, all = heads * each;
        const bool take[2] = {met[0] == 1u, met[1] == 1u};
        constexpr int NT = SCORE_THREADS, U = 2;           // (all of a side's reads at once for four heads of 128 rows)
        for (int i0 = tid; i0 < all; i0 += U * NT) {
            float2 x[2][U], y[2][U];
            int h[U], u[U];
#pragma unroll
            for (int e = 0; e < U; ++e) {
                const int i = i0 + e * NT < all ? i0 + e * NT : i0;
                h[e] = i / each; u[e] = i - h[e] * each;
            }
#pragma unroll
            for (int side = 0; side < 2; ++side)
                if (take[side]) {
#pragma unroll
                    for (int e = 0; e < U; ++e) {
                        x[side][e] = get_shared2(edge(a, first + h[e], kb - 1 + side, 0) + 2 * u[e]);
                        y[side][e] = get_shared2(edge(a, first + h[e], kb - 1 + side, 1) + 2 * u[e]);
                    }
                }
#pragma unroll
            for (int side = 0; side < 2; ++side) {
                if (!take[side]) continue;
                const int64_t o0 = n - a.w - ((int64_t)(kb - 1 + side) * SB + SB - 1);
#pragma unroll
                for (int e = 0; e < U; ++e) {
                    if (i0 + e * NT >= all || o0 + u[e] < 0) continue;
                    a.slash[(int64_t)(first + h[e]) * n + o0 + u[e]] = x[side][e].x + y[side][e].x;      // lower key block first
                    a.smax[(int64_t)(first + h[e]) * n + o0 + u[e]] = fmaxf(x[side][e].y, y[side][e].y);
                }
            }
        }
        if (met[2] + 1u != (uint32_t)(left < blocks ? left : blocks)) return;
        for (int h = wv; h < heads; h += 4) {
            const float* col = a.vert + (int64_t)(first + h) * n;
            const int64_t beg = (int64_t)part * share_keys(n), end = beg + share_keys(n) < n ? beg + share_keys(n) : n;
            float r[16];
#pragma unroll
            for (int w = 0; w < 16; ++w) r[w] = 0.f;
            for (int64_t i0 = beg + lane; i0 - lane < end; i0 += 1024) {
                float v[16];
#pragma unroll
                for (int w = 0; w < 16; ++w) v[w] = get_shared(col + (i0 + 64 * w < end ? i0 + 64 * w : beg));
#pragma unroll
                for (int w = 0; w < 16; ++w) if (i0 + 64 * w < end) r[w] += v[w];
            }
            const float share = share_of(r);
            if (lane == 0) put_shared(edge_share(a, first + h) + part, share);
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (wv > 0) return;
        const int groups = edge_groups(a);
        int last = 0;
        if (lane == 0) last = count_shared(a.done + first) + 1u == (uint32_t)groups;
        if (__builtin_amdgcn_readfirstlane(last) == 0) return;
        for (int h = lane; h < heads; h += 64) {
            float p[FINISH_SPLIT];
#pragma unroll
            for (int i = 0; i < FINISH_SPLIT; ++i) p[i] = i < groups ? get_shared(edge_share(a, first + h) + i) : 0.f;
            a.total[first + h] = total_of(p);
        }
    }
}

// ---- diagonals from the written matrix (explicit positions) ---------------------------------------
// grid (n / 256, heads bh_first ..): thread o adds A[t][p_t - o] over the band's rows in order, to what the bands before it
// gave; neighbouring threads read neighbouring cells.
__global__ __launch_bounds__(256) void diagonals_kernel(ScoreArgs a) {
    __shared__ int32_t pos[256];
    if (threadIdx.x < (unsigned)a.w) pos[threadIdx.x] = position_of(a, threadIdx.x);
    __syncthreads();
    const int64_t o = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (o >= a.n) return;
    const float* A = a.a_win + ((int64_t)blockIdx.y * (a.t1 - a.t0) - a.t0) * a.n;
    const int64_t at = (int64_t)(a.bh_first + blockIdx.y) * a.n + o;
    float sum = 0.f, mx = 0.f;
    if (a.t0 > 0) { sum = a.slash[at]; mx = a.smax[at]; }
    for (int t0 = a.t0; t0 < a.t1; t0 += 8) {
        float p[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int t = t0 + e < a.t1 ? t0 + e : a.t1 - 1;
            const int64_t key = pos[t] - o;
            p[e] = t0 + e < a.t1 && key >= 0 ? A[(int64_t)t * a.n + key] : 0.f;
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) { sum += p[e]; mx = fmaxf(mx, p[e]); }
    }
    a.slash[at] = sum;
    a.smax[at] = mx;
}

// ---- finish: add the two diagonal partials, reduce the total ------------------------------------
// grid (B*Hq, FINISH_SPLIT).  Diagonal o is met by keys n-w-o .. n-1-o (clipped at 0), i.e. by key blocks
// kA = max(0, n-w-o)/SB and kB = (n-1-o)/SB, which are equal or adjacent.  The last of a head's workgroups to get to its
// end (a counter per head, which the statistics pass has cleared) adds their shares of the total, in a fixed tree order.
__global__ __launch_bounds__(1024) void finish_kernel(ScoreArgs a, int contiguous) {
    __shared__ float red[1024];
    const int bh = blockIdx.x, part = blockIdx.y, tid = threadIdx.x;
    const int64_t n = a.n;
    const int64_t per = share_keys(n);                     // this workgroup's range
    const int64_t beg = (int64_t)part * per, end = beg + per < n ? beg + per : n;
    // (asked for ahead of the diagonals' partials: one round trip for both)
    float v4[4];
    auto ask = [&](int64_t i0) {
#pragma unroll
        for (int j = 0; j < 4; ++j) { const int64_t i = i0 + j * 1024; v4[j] = i < end ? a.vert[(int64_t)bh * n + i] : 0.f; }
    };
    ask(beg + tid);
    if (contiguous) {
        for (int64_t o0 = beg + tid; o0 < end; o0 += 4 * 1024) {   // four diagonals per thread, all loads first
            float2 va[4], vb[4]; bool two[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int64_t o = o0 + j * 1024 < end ? o0 + j * 1024 : end - 1;
                int64_t lo = n - a.w - o; if (lo < 0) lo = 0;
                const int64_t kA = lo / SB, kB = (n - 1 - o) / SB;
                two[j] = kB != kA;
                va[j] = reinterpret_cast<const float2*>(a.spart)[((kA & 1) * a.BH + bh) * n + o];
                vb[j] = reinterpret_cast<const float2*>(a.spart)[((kB & 1) * a.BH + bh) * n + o];
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int64_t o = o0 + j * 1024;
                if (o < end) {
                    a.slash[(int64_t)bh * n + o] = two[j] ? va[j].x + vb[j].x : va[j].x;      // lower key block first
                    a.smax[(int64_t)bh * n + o] = two[j] ? fmaxf(va[j].y, vb[j].y) : va[j].y;
                }
            }
        }
    }
    // this range's share of total = sum of the column sums: per thread in index order, then a fixed tree
    float acc = 0.f;
    for (int64_t i0 = beg + tid; i0 < end;) {
#pragma unroll
        for (int j = 0; j < 4; ++j) if (i0 + j * 1024 < end) acc += v4[j];
        i0 += 4 * 1024;
        ask(i0);
    }
    red[tid] = acc;
    __syncthreads();
    if (tid >= 64) return;
    float r[16];
#pragma unroll
    for (int w = 0; w < 16; ++w) r[w] = red[64 * w + tid];
    acc = share_of(r);
    if (tid == 0) {
        float* share = a.part + (int64_t)bh * FINISH_SPLIT;            // `part` is free again once merge_kernel has run
        put_shared(share + part, acc);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        if (count_shared(a.done + bh) == FINISH_SPLIT - 1u) {
            float p[FINISH_SPLIT];
#pragma unroll
            for (int i = 0; i < FINISH_SPLIT; ++i) p[i] = get_shared(share + i);
            a.total[bh] = total_of(p);
        }
    }
}

// Workgroups that share a KV head's query heads over one key block.  A grid of less than four workgroups per CU
// (what the LDS takes) leaves SIMDs with too few waves to cover the chunks' barriers: the heads are then shared
// out, at the price of reading K once more per share, which the L2 mostly answers.  No further: a second round of workgroups costs more than it spreads.  ls_score, up to 2048 workgroups where
// they keep four chunks / 1024, us: 64 heads, 64 rows of 8192 keys 54.4 / 49.9, B 4, 3000 keys 73.9 / 70.2, 32 heads, 16384 keys 55.9 / 52.9, 128 rows 82.1 / 80.7, 12347 keys
// 48.4 / 47.8; ls_score_window, 64 rows of 16384 keys 60.5 / 56.0, 128 of 8192 57.5 / 53.3.  1024 fp32 keys, 4 -> 16 workgroups per key block: 15.1 -> 6.2 us.
// `band`: chunks of a band of explicit positions.  The band's launches wait for each other, and a second round fills the end of one: up to 2048 workgroups where they keep four of the band's chunks.
// 1024 / so, us: B 4, 64 heads, 64 rows of 16384 keys 718 / 711, d = 64 645 / 629; where they keep two: 131072 keys, 128 rows 1306 / 1463, 32768 keys, 64 rows 180 / 194.
static int head_shares(const ScoreArgs& a, int kv_heads, int band = 0) {
    const int64_t wgs = (int64_t)a.nkb * kv_heads;
    int z = 1;
    while (a.G % (2 * z) == 0 && wgs * 2 * z <= (band >= 8 * z ? 2048 : 1024)) z *= 2;
    return z;
}
// Whether lines_kernel adds what neighbouring key blocks have of a diagonal, and the totals, itself.  That saves finish_kernel's launch and round trips, and costs a
// workgroup three round trips at its end, in which others of its CU have to keep it busy: where nearly all are there at once (1024 are).
// The whole ls_score, finish_kernel / so, us: 1024 keys, fp32, 16.1 / 15.3; 32 heads, 64 rows, of 2048 keys 19.7 / 18.5, 8192 36.0 / 34.8, B 2 52.7 / 50.5, 12347 50.8 / 49.7, 16384 51.5 /
// 50.8; 16 heads of 64, 48 rows of 5003 keys 22.2 / 20.8; 1536 workgroups, B 8, 3000 keys 75.4 / 74.0, B 3, 8192 70.7 / 70.8; 2048: B 4, 8192 89.0 / 85.2, but with fewer chunks of rows a workgroup,
// MHA, four of 16384 44.6 / 47.7, two of 8192 45.2 / 46.7, one 38.9 / 40.8.  Beyond 16384 keys a share of the total is more than two reads a lane: 20000 60.8 / 63.5, 8 rows of 8 heads 29.7 / 32.7, 65536, 4 heads
// 30.4 / 35.8.
static bool joins(const ScoreArgs& a, int kv_heads) { return (int64_t)a.nkb * kv_heads * a.shares <= 1600 && a.n <= 16384; }
// The ranges of keys of range_stats_kernel; 0: stats_kernel, where there is little work, or so few rows that waves would stand idle.
// As many as fill the chip with three workgroups a CU; for the retention score, which keeps their statistics apart, no more than the blocks of 128 keys that `part` has room for, and
// no more than give every CU two workgroups (64 to 256 of them: beyond, merge_kernel takes what they save).  The whole ls_kv_compress, us, stats_kernel / 64 ranges / so: one KV head, 64
// rows of 262144 keys 67 / 78 / 51, 128 of 131072 49 / 65 / 45, 256 67 / 75 / 56; two, 64 of 262144 87 / 90 / 74; four, 128 of 131072, d = 64, 74 / 72 / 64; eight, 64 ranges / 96: 131 / 133.  Four chunks of rows a workgroup, eight where there is much work: eight / four, us, 131072 keys 140 / 157, 16384 keys, B 4, 75 / 81, 32768
// 24.0 / 24.4, 12347 16.0 / 13.8.
// The lines.  The whole call, stats_kernel / range_stats_kernel, us.  Retention score of 16 rows: 8 heads, 16384 keys (1024 of the products below) 25.7 / 27.8, 32 / 8 heads (2048) 28.8 / 29.1, 20000 keys
// (2512) 39.2 / 37.2, 32768 (4096) 47.3 / 45.1, 4 / 1 heads, 32768 (512) 25.7 / 26.2, 131072 (2048) 43.4 / 40.1.  ls_score: 8192 keys, 32 heads, 64 rows (4096) 34.9 / 35.1, 12347 (6208) 50.1 / 48.2, 16384 (8192) 55.0 /
// 50.0, 32768 91.1 / 84.3, 131072, 16 heads of 64, 32 rows 86.8 / 84.7, 4 heads, 100 rows 93 / 88, 32 heads, 128 rows 520 / 491, 16384, B 4, 64 heads 288 / 269.
//
// Explicit positions see parts of a context that differ from row to row, and the ranges of a KV head come out uneven: few and long ones are worse than none.  The whole ls_score, us,
// stats_kernel / range_stats_kernel, d = 128: 3 to 12 ranges of eleven blocks, B 4, 64 heads, 16384 keys 703 / 715, B 8, 8192 701 / 720, B 16, 4096 725 / 741; 6 of four, B 4, 3000 162 / 159;
// 24 of five, B 4, 32 heads, 16384 347 / 345; 96 of three, 32768 183 / 180; 48 of 21, 131072, 128 rows 1322 / 1306.  d = 64, whose keys are half as much to read, gains nothing:
// 613 / 624, 623 / 658 (B 8), 320 / 324 (32 heads), 167 / 168 (32768), 1214 / 1240 (131072).
constexpr int STATS_PARTS = 64, STATS_PARTS_MOST = 256, STATS_FEW = 16, STATS_LONG = 8;
static int stats_split(ScoreArgs& a, bool bf16, int d, bool retention) {
    a.parts = a.nkb; a.stat_chunks = STATS_CHUNKS;
    const int count = Chunks(a.w, a.G, packs(a.w)).count;
    const int64_t work = (int64_t)a.B * a.Hkv * a.nkb * count;       // 128 keys by 32 rows
    if (!bf16 || work < (retention ? 3072 : 8192) || (!retention && count < 3)) return 0;
    if (work <= 24576) a.stat_chunks = 4;
    int r = 768 / (a.B * a.Hkv * ((count + a.stat_chunks - 1) / a.stat_chunks));
    if (retention) {
        const int two = 512 / (a.B * a.Hkv), most = two < STATS_PARTS ? STATS_PARTS : two < STATS_PARTS_MOST ? two : STATS_PARTS_MOST;
        r = r > most ? most : r;
    }
    r = r < 1 ? 1 : r < a.nkb ? r : a.nkb;
    if (a.q_pos && (d == 64 || (r < STATS_FEW && a.nkb >= STATS_LONG * r))) { a.stat_chunks = STATS_CHUNKS; return 0; }
    if (retention) a.parts = r;
    return r;
}
template <typename T, int D>
static void launch_stats(const ScoreArgs& a, int ranges, bool retention, hipStream_t st) {
    if constexpr (Elem<T>::bytes == 2) {
        if (ranges > 0) {
            const int z = (Chunks(a.w, a.G, packs(a.w)).count + a.stat_chunks - 1) / a.stat_chunks;
            const dim3 grid(ranges, a.B * a.Hkv, z);
            if (retention) hipLaunchKernelGGL((range_stats_kernel<D, false>), grid, dim3(SCORE_THREADS), stats_lds<D>(), st, a);
            else hipLaunchKernelGGL((range_stats_kernel<D, true>), grid, dim3(SCORE_THREADS), stats_lds<D>(), st, a);
            return;
        }
    }
    const size_t smem = stats_front<T, D>() + (size_t)a.w * 4;
    hipLaunchKernelGGL((stats_kernel<T, D>), dim3(a.nkb, a.B * a.Hkv, packs(a.w) ? 1 : head_shares(a, a.B * a.Hkv)), dim3(SCORE_THREADS), smem, st, a);
}
// whether lines_kernel merges the statistics (of all KV heads: bands of explicit positions do it again)
static bool folds(const ScoreArgs& a, int mode) {
    const int64_t bytes = (int64_t)a.nkb * a.B * a.Hkv * (a.G * a.w) * a.parts * 8;      // of all workgroups together (each takes its share of the heads)
    return a.parts <= FOLD_PARTS && score_chunks(a) <= FOLD_CHUNKS && (bytes <= FOLD_BYTES || (mode != 1 && a.nkb <= 16));
}
static int band_chunks(const ScoreArgs& a) { return a.G * ((a.t1 + 31) / 32 - a.t0 / 32); }
template <typename T, int D, int MODE>
static void launch_lines(const ScoreArgs& a, int kv_heads, hipStream_t st) {
    const bool fold = folds(a, MODE);
    const size_t smem = lines_front<T, D>(MODE) + (size_t)(a.w + 3) / 4 * 16 + (fold ? (size_t)score_chunks(a) * 256 : 512);
    const dim3 grid(a.nkb, kv_heads, MODE == 2 ? 1 : head_shares(a, kv_heads, MODE == 1 ? band_chunks(a) : 0));
    if (fold) hipLaunchKernelGGL((lines_kernel<T, D, MODE, true>), grid, dim3(SCORE_THREADS), smem, st, a);
    else hipLaunchKernelGGL((lines_kernel<T, D, MODE, false>), grid, dim3(SCORE_THREADS), smem, st, a);
}

// Explicit positions: how many KV heads and window rows a band of the matrix has, `fit` rows of one KV head at most.  Whole
// chunks of 32 rows (or the whole window), so many of them that the bands are fewest, and of those the ones with most rows: K
// is read once a band.  A buffer of less than a chunk takes parts of one, and the chunk is passed again for each.  A band costs
// two launches that wait for each other: 32768 keys, two KV heads of four, 32 rows a band: 22 + 14 us for 34 MB written and read.
static void window_bands(int64_t fit, int BK, int w, int* heads, int* rows) {
    int64_t fewest = INT64_MAX;
    *heads = 1;
    *rows = (int)(fit < w ? fit : w);
    for (int r = w; r > 0; r = (r - 1) / 32 * 32) {
        if (fit < r) continue;
        const int64_t h = fit / r < BK ? fit / r : BK, bands = ((BK + h - 1) / h) * ((w + r - 1) / r);
        if (bands < fewest) { fewest = bands; *heads = (int)h; *rows = r; }
    }
}

// Which kernels a call takes (run_score_t launches them), and what they find of it in `a`.
ScoreRoute score_route(ScoreArgs& a, bool bf16, int d, int mode) {
    ScoreRoute r{};
    const int BK = a.B * a.Hkv;
    if (mode == 0) { a.shares = head_shares(a, BK); a.join = joins(a, BK); }
    r.ranges = stats_split(a, bf16, d, mode == 2);
    r.unit = mode == 2 ? KeyTile<128>::KEYS : SB;
    r.chunks = a.stat_chunks;
    r.folds = folds(a, mode);
    r.shares = packs(a.w) ? 1 : head_shares(a, BK);
    r.joins = a.join;
    if (mode == 1) {
        window_bands(a.win_rows, BK, a.w, &r.band_heads, &r.band_rows);
        ScoreArgs first = a;
        first.t0 = 0; first.t1 = r.band_rows;
        r.band_shares = head_shares(first, r.band_heads, band_chunks(first));
    }
    r.streams = a.retain = mode == 2 && bf16 && !r.folds && Chunks(a.w, a.G, packs(a.w)).count <= RETAIN_CHUNKS;
    return r;
}

template <typename T, int D>
static hipError_t run_score_t(const ScoreArgs& a0, int mode, hipStream_t st) {
    ScoreArgs a = a0;
    const int BK = a.B * a.Hkv;
    a.t0 = 0; a.t1 = a.w;
    const ScoreRoute r = score_route(a, Elem<T>::bytes == 2, D, mode);
    launch_stats<T, D>(a, r.ranges, mode == 2, st);
    if (!r.folds) hipLaunchKernelGGL(merge_kernel, dim3((a.G * a.w + 15) / 16, BK), dim3(1024), 0, st, a);
    if (mode == 0) {
        if (a.join) {
            launch_lines<T, D, 4>(a, BK, st);
            return hipGetLastError();
        }
        launch_lines<T, D, 0>(a, BK, st);
    } else if (mode == 1) {
        const int most = r.band_heads, rows = r.band_rows;
        for (a.bk0 = 0; a.bk0 < BK; a.bk0 += most) {
            const int heads = BK - a.bk0 < most ? BK - a.bk0 : most;
            a.bh_first = a.bk0 * a.G;
            for (a.t0 = 0; a.t0 < a.w; a.t0 = a.t1) {
                const int chunk_end = rows < 32 ? (a.t0 / 32 + 1) * 32 : a.w;      // a band of less than a chunk lies inside one
                a.t1 = a.t0 + rows < a.w ? a.t0 + rows : a.w;
                if (a.t1 > chunk_end) a.t1 = chunk_end;
                a.sums = a.t0 % 32 == 0;
                launch_lines<T, D, 1>(a, heads, st);
                hipLaunchKernelGGL(diagonals_kernel, dim3((unsigned)((a.n + 255) / 256), heads * a.G), dim3(256), 0, st, a);
            }
        }
    } else if (mode == 3) {
        launch_lines<T, D, 3>(a, BK, st);
        return hipGetLastError();
    } else {
        const int share = 512 / BK < 1 ? 1 : 512 / BK < a.nkb ? 512 / BK : a.nkb;      // (64 KB of LDS: two workgroups a CU)
        if constexpr (Elem<T>::bytes == 2) {
            if (a.retain) hipLaunchKernelGGL(retain_kernel<D>, dim3(share, BK), dim3(SCORE_THREADS), retain_lds<D>(), st, a);
        }
        if (!a.retain) launch_lines<T, D, 2>(a, BK, st);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(finish_kernel, dim3(a.BH, FINISH_SPLIT), dim3(1024), 0, st, a, mode == 0 ? 1 : 0);
    return hipGetLastError();
}

template <typename T, int D>
static hipError_t init_score_t() {
    hipError_t e;
    if ((e = allow_full_lds(&stats_kernel<T, D>)) != hipSuccess) return e;
    if constexpr (Elem<T>::bytes == 2)
        if ((e = allow_full_lds(&range_stats_kernel<D, false>)) != hipSuccess || (e = allow_full_lds(&range_stats_kernel<D, true>)) != hipSuccess || (e = allow_full_lds(&retain_kernel<D>)) != hipSuccess) return e;
    if ((e = allow_full_lds(&lines_kernel<T, D, 0, false>)) != hipSuccess || (e = allow_full_lds(&lines_kernel<T, D, 0, true>)) != hipSuccess) return e;
    if ((e = allow_full_lds(&lines_kernel<T, D, 4, false>)) != hipSuccess || (e = allow_full_lds(&lines_kernel<T, D, 4, true>)) != hipSuccess) return e;
    if ((e = allow_full_lds(&lines_kernel<T, D, 1, false>)) != hipSuccess || (e = allow_full_lds(&lines_kernel<T, D, 1, true>)) != hipSuccess) return e;
    if ((e = allow_full_lds(&lines_kernel<T, D, 2, false>)) != hipSuccess || (e = allow_full_lds(&lines_kernel<T, D, 2, true>)) != hipSuccess) return e;
    if ((e = allow_full_lds(&lines_kernel<T, D, 3, false>)) != hipSuccess) return e;
    return allow_full_lds(&lines_kernel<T, D, 3, true>);
}
hipError_t init_score_kernels() {
    hipError_t e;
    if ((e = init_score_t<bf16_t, 128>()) != hipSuccess) return e;
    if ((e = init_score_t<bf16_t, 64>()) != hipSuccess) return e;
    if ((e = init_score_t<float, 128>()) != hipSuccess) return e;
    return init_score_t<float, 64>();
}

hipError_t run_score(const ScoreArgs& a, int dtype, int d, int mode, hipStream_t st) {
    if (dtype == 0 && d == 128) return run_score_t<bf16_t, 128>(a, mode, st);
    if (dtype == 0 && d == 64) return run_score_t<bf16_t, 64>(a, mode, st);
    if (dtype == 1 && d == 128) return run_score_t<float, 128>(a, mode, st);
    if (dtype == 1 && d == 64) return run_score_t<float, 64>(a, mode, st);
    return hipErrorInvalidValue;
}

}  // namespace ls
