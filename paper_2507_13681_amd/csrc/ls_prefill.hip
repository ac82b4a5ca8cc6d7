// Sparse prefill attention over selected key columns and diagonals (gfx950).
//
// Computes, for every row a of the newest turn (absolute position p = n - n_hat + a),
//     out[a] = sum_b softmax_b( scale * <q_a, k_b> ) v_b   over the allowed cells
//     allowed(a, b)  <=>  b <= p  and  ( b is a selected column  or  p - b is a selected diagonal )
// which is the masked attention Softmax(QK^T/sqrt(d_k) - c(1 - M)) V of Sec. 2.2 with the mask M
// built from the vertical and slash lines chosen by Alg. 2 (Sec. 5.1), masked entries weighing zero.
//
// Work decomposition.  One workgroup (4 waves) owns 128 query rows of one (batch, head); blocks of
// rows are aligned to absolute positions that are multiples of 128, so the diagonals a 128 x 64 tile
// touches depend only on j = (row block start)/64 - (key block): offsets 64j - 63 .. 64j + 127.  A
// per-head table built by plan_kernel says, for each j, whether any (or every) diagonal in that range
// is selected.
//   phase 1: key blocks whose diagonal range holds a selected diagonal are streamed as contiguous
//            64-key tiles; the cell mask is the diagonal bit, read from the head's bitmap.
//   phase 2: the selected columns (up to the block's last row) are gathered, 64 at a time, into
//            packed tiles; a cell is dropped there if its diagonal is selected (phase 1 counted it).
// So every allowed cell is visited exactly once.  Each wave owns 32 rows and skips the 32 x 32
// sub-tiles in which none of its rows has an allowed cell.
//
// Tile products: S^T = K_tile * Q^T and O^T += V_tile^T * P^T on 32x32 MFMA, fp32 accumulation, softmax
// in the base-2 domain.  bf16 (prefill_bf16_kernel): K and V rows go to LDS as they are, V is read back transposed, and the softmax
// reference moves only where a sum of probabilities exceeds a limit.  fp32 (prefill_kernel): online softmax with the tile's maximum,
// K staged row-major in LDS, V transposed (see vt_col).
#include <type_traits>
#include <hip/hip_ext.h>
#include "ls_device.h"
#include "ls_internal.h"

namespace ls {

constexpr int RING_S = 4;        // K fragments in flight ahead of the QK^T products
constexpr int RING_P = 3;        // V^T fragments in flight ahead of the P*V products
constexpr int RING_P_QUEUES = 2; // ... with queues, where there are fewer registers
constexpr int BM = 128;   // query rows per workgroup
constexpr int BN = 64;    // keys per tile
constexpr int PREFILL_THREADS = 256;

// Work is counted in eighths of a contiguous tile: a packed tile takes longer (its rows are gathered, and its loop has more to see to), and an item takes as long as
// four tiles beside its own (queries, lists, the first tile's way from memory, the results; one tile in fp32, whose tiles take long).
// bf16: with packed tiles at nine eighths, as before the loop of contiguous tiles had its own short form, the pieces of heads of columns came last, 258 to 336 us where those of diagonals took 219 to 272 (2000
// of 20000 rows).  9 / 10 / 11 / 12, the whole call, us: that turn 488 / 469 / 465 / 467, 3000 rows 611 / 592 / 581 / 584, 1000 of 32768 439 / 429 / 419 / 419, 500 of 65536 647 / 628 / 621 / 622;
// fp32 has nine.
constexpr uint32_t WORK_TILE = 8;
// What an item is: the contiguous tiles (at most 4097) and the columns (at most 262144) of a row block.
__host__ __device__ __forceinline__ uint32_t pack_item(uint32_t n1, uint32_t cols) { return n1 | cols << 13; }
__host__ __device__ __forceinline__ int item_blocks(uint32_t r) { return (int)(r & 0x1FFFu); }
__host__ __device__ __forceinline__ int item_cols(uint32_t r) { return (int)(r >> 13); }
__host__ __device__ __forceinline__ uint32_t work_base(int dtype) { return dtype == 0 ? 32 : 8; }
__host__ __device__ __forceinline__ uint32_t work_cols(uint32_t base) { return base == 32 ? 11 : 9; }        // of a packed tile
__host__ __device__ __forceinline__ uint32_t item_work(uint32_t base, uint32_t n1, uint32_t n2) { return base + n1 * WORK_TILE + n2 * work_cols(base); }
// A half's probabilities (relative to the running reference) may sum to this in a lane before the reference moves to the half's maximum;
// in an item's first tiles to less (4, 8, 16: twice as much every tile).  bf16 is as exact up there as around one, but the probability
// that is the reference is one, without rounding, and a row's largest cells mostly come early (the band beside the
// diagonal).  Error of the output against 64 bits, rms relative to it, 1e-3, with 65536 throughout / 16 / this / a maximum per tile and
// moves beyond 2^8, as it was: 3000 of 6000 rows 2.05 / 1.97 / 1.98 / 1.99, 61 of 12347 2.09 / 1.92 / 1.87 / 1.92, 8192 rows, all new, 2.14 / 1.89 /
// 1.91 / 2.06, 2000 of 30000 2.10 / 1.95 / 1.96 / 2.04, d = 64, 1777 of 5003 2.02 / 1.89 / 1.90 / 1.92.  It costs 0.5 % of the attention of
// a long turn, 4 % of one of 61 rows, and most where items have a handful of tiles: the 300 newest diagonals, 4402 rows of 13466, B 16, 16 heads 410 us,
// at 16 from the second tile on 398, with a maximum per tile 382; d = 64, 7390 of 9251 rows 410, 390, 363.  (The first reference over both halves of
// the first tile: nothing.  Errors at 16 from the second tile on 2.041, 1.983, 2.036e-3 instead of 2.037, 1.973, 2.035: not taken.)
constexpr float SOFT_LIMIT = 32.f, SOFT_FIRST = 2.f;
// Where a row's logits rise along the keys (heads that look at the newest keys most), nearly every half would be done again.  A wave whose
// halves exceed the limit that often (SOFT_OFTEN: 4 for each, less 1 a tile) sets its references 2^32 above the maxima from then on, until
// the last two contiguous tiles, where such rows have their largest cells: those are done with the maxima as the references again.
// (In between, what values of V below 2^-94 add is too small for fp32.)
// 4096 of 16384 rows, 8 dense heads whose logits rise by 0 / 1 / 4 / 16 / 32 (base 2) in 64 keys, us: without 326 / 363 / 387 / 402 / 396, with
// 316 / 342 / 325 / 328 / 354 (a maximum per tile 361 / 365 / 344 / 341 / 340); d = 64 196 / 221 / 264 / 259 / 258, with 194 / 210 / 208 / 205 / 229.
// Error against 64 bits 2.32 / 2.27 / 2.11 / 1.90 / 1.83e-3, with 2.32 / 2.17 / 2.01 / 1.90 / 1.84e-3 (without the last two tiles' part
// 2.32 / 2.34 / 2.30 / 2.21 / 2.09e-3).  Other rows pay 0.1 to 0.5 % of the attention for the count.
constexpr int SOFT_OFTEN = 40, SOFT_RISING = 1 << 29;      // (what the count is from then on)
constexpr float SOFT_AHEAD = 32.f;

// ---------------------------------------------------------------------------------------------
// plan: per (batch, head) bitmap of the selected diagonals, the per-j activity table, a head flag.
//   obits : [BH][4 + words] uint32: four zero words, then bit o in word 4 + o/32; words = n/32 rounded up + 8 zero words
//   tab   : [BH][tab_len] bytes, entry j+1 for j = -1 .. ; bit0 = some diagonal of
//           [64j-63, 64j+127] is selected, bit1 = all of them are (and none is cut off at 0 or n-1)
//   elist : [BH][tab_len + 1] the entries of tab with bit0, ascending: a row block's key blocks are a run of them
//   rec   : [BH][nqb] of each row block the length of that run and the columns it gathers (none if every diagonal is
//           selected: the mask is plain causal then, or if the column list is not strictly ascending inside [0, n): its columns
//           are ignored); upto, head_work: running sums of the work that is
// ---------------------------------------------------------------------------------------------
// Exclusive prefix sum over the 1024 threads of a workgroup: returns the sum of `v` over the threads before this one and, in
// `total`, the sum over all threads.  `wsum`: 16 words, FREE: that no earlier call's threads still read (a barrier less).
template <bool FREE = false>
__device__ __forceinline__ uint32_t block_scan_1024(uint32_t v, uint32_t* wsum, uint32_t& total) {
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t upto = lanes_upto(v);
    if (!FREE) __syncthreads();
    if (lane == 63) wsum[wv] = upto;
    __syncthreads();
    return waves_before(wsum, lane, wv, total) + upto - v;
}

constexpr int OB_PAD = 4;                    // zero words in front of a head's bitmap (rows above a tile's keys)
// The same for the maximum, with `wsum` free: the largest `v` of the threads before this one (0 for the first).
template <int CTRL, int ROWS> __device__ __forceinline__ uint32_t dpp_larger(uint32_t x) { const uint32_t o = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, ROWS, 0xF, false); return o > x ? o : x; }
__device__ __forceinline__ uint32_t block_max_1024(uint32_t v, uint32_t* wsum) {
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    auto row = [](uint32_t x) { x = dpp_larger<0x111, 0xF>(x); x = dpp_larger<0x112, 0xF>(x); x = dpp_larger<0x114, 0xF>(x); return dpp_larger<0x118, 0xF>(x); };      // row_shr:1, 2, 4, 8
    uint32_t upto = row(v);
    upto = dpp_larger<0x142, 0xA>(upto);                   // row_bcast15 into rows 1 and 3
    upto = dpp_larger<0x143, 0xC>(upto);                   // row_bcast31 into rows 2 and 3
    if (lane == 63) wsum[wv] = upto;
    const uint32_t ex = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)upto, 0x138 /* wave_shr:1 */, 0xF, 0xF, false);
    __syncthreads();
    const uint32_t waves = row(wsum[lane & 15]), before = wv > 0 ? (uint32_t)__builtin_amdgcn_readlane((int)waves, wv - 1) : 0u;
    return ex > before ? ex : before;
}

// grid (BH).  Bound by the round trips of one workgroup through the lists of its head: so many loads of 16 bytes are in flight as
// there are registers for without losing a wave, and the bitmap is put together from neighbouring entries (one entry a lane, eight
// loads of 4 bytes in flight: 131072 rows 81 us, now 52; 32768 26 -> 19.5, B 4, 64 heads of 16384 17.1 -> 14.7).  Where the lists are short it is the steps behind
// one another, a thousand cycles each: scans by DPP with a barrier instead of shuffles with two, the six words of a table entry read at once, 32-bit
// column arithmetic: 5003 lines 11.2 -> 9.6 us, 8192 11.7 -> 9.4, 12347 7.2 -> 5.9 (start 1500 cycles, columns 1000 to 2000, diagonals 900 to 2400, bitmap out 1000,
// table 630, entries 1400, row blocks 1700).
constexpr int LS_MAX_BLOCKS = 262144 / 128 + 2;   // row blocks at the largest supported context
constexpr int LS_MAX_TAB = 262144 / 64 + 8;  // table entries at the largest supported context
__global__ __launch_bounds__(1024) void plan_kernel(PlanArgs a) {
    extern __shared__ uint32_t sm[];
    __shared__ int total_bits;
    __shared__ uint8_t tabs[LS_MAX_TAB];
    __shared__ uint32_t colh[LS_MAX_BLOCKS];               // list position behind the last column that each row block is the first to see
    __shared__ uint32_t wsum[3][16];
    const int bh = blockIdx.x;
    const int64_t n = a.n;
    const int words = a.words;
    const int tid = threadIdx.x;
    int nvl = a.v_cnt[bh]; if (nvl > a.cap_v) nvl = a.cap_v; if (nvl < 0) nvl = 0;
    int ns = a.s_cnt[bh]; if (ns > a.cap_s) ns = a.cap_s; if (ns < 0) ns = 0;
    const int32_t* si = a.s_idx + (int64_t)bh * a.cap_s;
    for (int i = tid; i < words; i += blockDim.x) sm[i] = 0u;
    for (int i = tid; i < a.nqb; i += blockDim.x) colh[i] = 0u;
    if (tid == 0) total_bits = 0;
    __syncthreads();
    // The column list must be strictly ascending and inside [0, n) (the attention kernel gathers K / V rows through
    // a prefix of it): a head whose list is not has its columns ignored and the context's status word says so.  Diagonals outside [0, n) are skipped below and reported likewise.
    const int32_t* vl = a.v_idx + (int64_t)bh * a.cap_v;
    bool v_bad = false, s_bad = false;
    // the last column that each row block is the first to see leaves its list position behind (columns before the turn
    // count for the first block)
    const int pos0 = (int)a.pos0, n32 = (int)n;
    static_assert(BM == 128, "a shift by 7");
    auto block_of = [&](int32_t c) -> int { return c > pos0 ? (c - pos0) >> 7 : 0; };
    auto mark_col = [&](int i, int32_t c, int block, int next, bool last) {        // (next: the next entry's block)
        if (c >= 0 && c < n32 && (last || next != block)) colh[block] = (uint32_t)i + 1u;
    };
    if ((reinterpret_cast<uintptr_t>(vl) & 15) == 0 && a.cap_v % 4 == 0) {     // four entries per load (and the one before them)
        typedef __attribute__((ext_vector_type(4))) int32_t i32x4;
        constexpr int AT_ONCE = 4;                         // loads of a thread in flight, 4096 entries apart
        for (int b0 = 4 * tid; b0 < nvl; b0 += AT_ONCE * 4 * (int)blockDim.x) {
            i32x4 c4[AT_ONCE];
            int32_t before[AT_ONCE], next[AT_ONCE];
#pragma unroll
            for (int u = 0; u < AT_ONCE; ++u) {
                const int i0 = b0 + u * 4 * (int)blockDim.x, at = i0 < nvl ? i0 : b0;
                c4[u] = *reinterpret_cast<const i32x4*>(vl + at);      // entries past nvl (inside the capacity, a multiple of 4 here) are not looked at
                before[u] = vl[at > 0 ? at - 1 : 0];
                next[u] = vl[at + 4 < nvl ? at + 4 : at];
            }
#pragma unroll
            for (int u = 0; u < AT_ONCE; ++u) {
                const int i0 = b0 + u * 4 * (int)blockDim.x;
                if (i0 >= nvl) break;
                int32_t prev = i0 > 0 ? before[u] : -1;
                const int32_t c[4] = {c4[u].x, c4[u].y, c4[u].z, c4[u].w};
                const int block[5] = {block_of(c[0]), block_of(c[1]), block_of(c[2]), block_of(c[3]), block_of(next[u])};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if (i0 + e < nvl) { v_bad = v_bad || c[e] <= prev || c[e] >= n32; prev = c[e]; }
                    if (i0 + e < nvl) mark_col(i0 + e, c[e], block[e], block[e + 1], i0 + e == nvl - 1);
                }
            }
        }
    } else {
        for (int i = tid; i < nvl; i += blockDim.x) {
            const int32_t c = vl[i];
            v_bad = v_bad || c < 0 || c >= n || (i > 0 && vl[i - 1] >= c);
            mark_col(i, c, block_of(c), block_of(i + 1 < nvl ? vl[i + 1] : 0), i == nvl - 1);
        }
    }
    v_bad = __syncthreads_or(v_bad);
    // every diagonal selected (a head the walk gave up sparsifying): the list is 0 .. n-1, checked while it is read
    typedef int32_t i32x4u __attribute__((ext_vector_type(4), aligned(4)));
    bool ident = ns == (int)n && ns >= 4;
    if (ident) {
        for (int i0 = 4 * tid; i0 < ns; i0 += 4 * 4 * 1024) {
            i32x4u x[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) { const int i = i0 + j * 4096; x[j] = *reinterpret_cast<const i32x4u*>(si + (i + 4 <= ns ? i : ns - 4)); }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int i = i0 + j * 4096, at = i + 4 <= ns ? i : ns - 4;
#pragma unroll
                for (int e = 0; e < 4; ++e) ident = ident && x[j][e] == at + e;
            }
        }
        ident = __syncthreads_and(ident);
        if (ident) for (int i = tid; i < (int)((n + 31) / 32); i += blockDim.x) sm[i] = (i == (int)(n / 32)) ? ((1u << (n & 31)) - 1u) : 0xFFFFFFFFu;
    }
    // sixteen entries that follow each other per thread; the list is ascending, so most of them fall into few words of the bitmap,
    // and a word's bits are collected first.  (Correct for any order of the list.)
    for (int i0 = 16 * tid; i0 < (ident ? 0 : ns); i0 += 16 * 1024) {
        int32_t o[16];
        if (i0 + 16 <= ns) {
            i32x4u x[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) x[j] = *reinterpret_cast<const i32x4u*>(si + i0 + 4 * j);
#pragma unroll
            for (int j = 0; j < 16; ++j) o[j] = x[j >> 2][j & 3];
        } else {
#pragma unroll
            for (int j = 0; j < 16; ++j) o[j] = si[i0 + j < ns ? i0 + j : i0];
        }
        int word = -1;
        uint32_t m = 0u;
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const bool ok = o[j] >= 0 && o[j] < n;
            s_bad = s_bad || !ok;
            const int wd = ok ? o[j] >> 5 : word;
            if (wd != word && word >= 0) { atomicOr(&sm[word], m); m = 0u; }
            word = wd;
            m |= ok ? 1u << (o[j] & 31) : 0u;
        }
        if (word >= 0) atomicOr(&sm[word], m);
    }
    __syncthreads();
    int mine = 0;
    uint32_t* og = a.obits + (int64_t)bh * (OB_PAD + words);  // zero words, then the bitmap
    if (tid < OB_PAD) og[tid] = 0u;
    for (int i = tid; i < words; i += blockDim.x) { og[OB_PAD + i] = sm[i]; mine += __popc(sm[i]); }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) mine += __shfl_down(mine, off, 64);       // one atomic per wave, not per thread
    if ((tid & 63) == 0) atomicAdd(&total_bits, mine);
    // activity table
    for (int e = tid; e < a.tab_len; e += blockDim.x) {
        // the diagonals 64 j - 63 .. 64 j + 127 that there are: six words (bits beyond the context are zero)
        const int j = e - 1;
        int cnt = 0;
#pragma unroll
        for (int k = 0; k < 6; ++k) {
            const int wd = 2 * j - 2 + k;
            const uint32_t m = sm[wd < 0 ? 0 : wd < words ? wd : words - 1];
            cnt += wd >= 0 && wd < words ? __popc(k == 0 ? m & ~1u : m) : 0;
        }
        uint8_t f = 0;
        if (cnt > 0) f |= 1;
        if (cnt == 191) f |= 2;
        a.tab[(int64_t)bh * a.tab_len + e] = f;
        tabs[e] = f;                                       // LDS copy for the counts below
    }
    __syncthreads();
    // the active entries in ascending order, and in LDS how many lie below each entry
    const int chunk = (a.tab_len + (int)blockDim.x - 1) / (int)blockDim.x;
    const int e0 = tid * chunk < a.tab_len ? tid * chunk : a.tab_len, e1 = (e0 + chunk < a.tab_len) ? e0 + chunk : a.tab_len;
    int mine2 = 0;
    for (int e = e0; e < e1; ++e) mine2 += tabs[e] & 1;
    uint32_t active_entries;
    uint32_t run = block_scan_1024<true>((uint32_t)mine2, wsum[0], active_entries);
    uint16_t* el = a.elist + (int64_t)bh * (a.tab_len + 1);
    uint16_t* below = reinterpret_cast<uint16_t*>(sm);     // [tab_len + 1]; the bitmap has been written out (the scan's barriers lie between)
    for (int e = e0; e < e1; ++e) {
        below[e] = (uint16_t)run;
        if (tabs[e] & 1) el[run++] = (uint16_t)e;
    }
    if (tid == 0) below[a.tab_len] = (uint16_t)active_entries;
    // what each row block visits and gathers: the columns up to its last row (none where every diagonal is selected, phase 1 covers
    // all cells then, or where the list is unusable), and the work that is
    {
        const bool none = total_bits == (int)n || v_bad;
        const int per = (a.nqb + (int)blockDim.x - 1) / (int)blockDim.x;
        const int q0 = tid * per < a.nqb ? tid * per : a.nqb, q1 = q0 + per < a.nqb ? q0 + per : a.nqb;
        uint32_t top = 0;                                  // positions grow with the block: a running maximum fills the gaps
        for (int q = q0; q < q1; ++q) top = top > colh[q] ? top : colh[q];
        const uint32_t before = block_max_1024(top, wsum[1]);          // (its barrier publishes `below`)
        const uint32_t base = work_base(a.dtype);
        uint32_t work = 0, all;
        auto visit = [&](int q, uint32_t& cols) -> uint2 {                       // {key blocks, columns}
            const int64_t blockpos = a.pos0 + (int64_t)q * BM;
            const int64_t posmax = (blockpos + BM - 1 < n - 1) ? blockpos + BM - 1 : n - 1;
            const int jb = (int)(blockpos / BN), kb_hi = (int)(posmax / BN);
            cols = cols > colh[q] ? cols : colh[q];
            return make_uint2(below[jb + 2] - below[jb - kb_hi + 1], none ? 0u : cols);             // entries jb-kb_hi+1 .. jb+1
        };
        uint32_t cols = before;
        for (int q = q0; q < q1; ++q) { const uint2 r = visit(q, cols); work += item_work(base, r.x, (r.y + BN - 1) / BN); }
        uint32_t pre = block_scan_1024<true>(work, wsum[2], all);
        cols = before;
        for (int q = q0; q < q1; ++q) {
            const uint2 r = visit(q, cols);
            pre += item_work(base, r.x, (r.y + BN - 1) / BN);
            a.rec[(int64_t)bh * a.nqb + q] = pack_item(r.x, r.y);
            if (a.upto) a.upto[(int64_t)bh * a.nqb + q] = pre;
            if (a.arrived) a.arrived[(int64_t)bh * a.nqb + q] = 0u;
        }
        if (tid == 0) a.head_work[bh] = all;
    }
    s_bad = __syncthreads_or(s_bad);
    if (bh == 0 && tid < 2) a.split_count[tid] = 0;
    if (tid == 0) {
        if (v_bad) atomicOr(a.status, STAT_V_INVALID);
        if (s_bad) atomicOr(a.status, STAT_S_RANGE);
    }
}

// ---------------------------------------------------------------------------------------------
// pieces: which part of the work each workgroup of the attention kernel takes, up to PIECES_TILES.
//
// The items (row blocks of heads) lie in one row, head by head, and the row is cut into as many pieces of about equal work
// as there are workgroups.  Every workgroup finds its own piece from the running sums that plan_kernel left behind: a scan over
// the heads, a look through one head's row blocks.  Neighbouring pieces go to the same XCD, so that the query heads that
// share K and V meet in one L2.  An item that a cut goes through is done in parts, whose unnormalised results go to slots of the
// workspace and which combine_kernel puts together (join_parts, where there are many items); a cut that would leave a few tiles on one side is moved to the
// end of the item.  A workspace that does not hold all parts gets fewer pieces, or queues (prefill_pieces_for).
//
// Against the work queues of sched_kernel (which serve what is larger) this saves a launch of one workgroup per XCD, a look at the
// queues per item, and the wait for the longest item, which a short turn feels most.  The whole call, bf16, 32 heads of d = 128, queues -> pieces,
// us: 2048 rows, all new, 92 -> 68; 1024 new of 8192 152 -> 124; 300 of 16384 89 -> 70; 100 of 131072 254 -> 230; 61 of 12347
// 32.7 -> 30.3; 4 heads fp32, 256 of 1024 44 -> 38, 2048 all new 65 -> 37.
// fp32: a tile keeps a workgroup's matrix cores busy for 8200 cycles, all that comes before the first one takes 13000: a few items' tiles
// go to a workgroup each.  Two tiles a piece and on either side of a cut / one, us: 4 heads of 64, 256 rows of 1024 38.6 / 30.2, 8 heads, 40 of 700 29.0 / 21.8, 20 of
// 4096 35.2 / 22.4, 700 of 3001 59.4 / 56.8, 4096, all new, 58.2 / 52.8.
// The line.  What the pieces' estimates miss nothing evens out, and the row spreads the heads of a moment wider than the queues
// do: the longer the run, the more both cost.  In bf16 the queues' kernel also has a workgroup more per CU (prefill_bf16_kernel).
// Tiles here are those that dense heads would have, and a tile of d = 64 counts half.  Pieces / queues, the whole call, us, d = 128, up to
// 262144 tiles: 4096 rows, all new, 114 / 150, 2500 of 12347 253 / 285, 2000 of 32768 660 / 692, 500 of 65536, 64 heads, 1030 / 1064 (but 1000 of 65536 773 / 752).
// Up to 524288 what it takes beside the length is a few items a workgroup: fewer and longer ones are cut too often, and more of them the queues even out.  Items and tiles: 752 of 385024 (16 heads, 6000 of 32768)
// 787 / 815, 768 of 393216 861 / 876, 1024 of 524288 (4000 of 32768) 949 / 1013, 1504 of 385024 581 / 589, 1536 of 288768 428 / 433, 1600 of 377600 836 / 851, 1664 of 520832 (64 heads, 3114 of 20000) 1041 /
// 1122, 2560 of 401920 661 / 679; 192 of 393216 (700 of 131072) 1534 / 1482, 512 of 524288 1081 / 1046 and 1194 / 1178, 640 of 500480 1110 / 1087, 3072 of 433152 595 / 590, 4096 of 524288 (B 4, 4096 of 8192) 816 / 746.  (Rows scored at random
// positions have no dense heads among the others, and pieces gain 5 to 10 %: 1504 items 380 / 420, 1600 537 / 571.)  At d = 64, where a workgroup has two thirds of the work, few items gain too, and more of them: 320 of
// 289920 (64 heads, 547 of 115957) 1327 / 1433, 512 of 524288 1427 / 1596, 1536 of 393216 965 / 1054, 2048 of 524288 1563 / 1539 and 1170 / 1214, 2560 of 480000 901 / 942, 4032 of 516096 783 / 782, 5120 of 481280 859 / 863, 8192 of
// 524288 616 / 600.  Turns that are all of the context see half of their tiles: 64 heads, 6000 rows (141376 seen) 337 / 363, 10000, 32 heads, 434 / 436, at d = 64 9000 417 / 447; 12000, 32 heads (283000), 497 / 490.
// More: 3072 of 589824 1127 / 1066, 10923 of 32768 1957 / 1527.  fp32, whose kernel is the same for both: 524288.
// ---------------------------------------------------------------------------------------------
constexpr int64_t PIECES_TILES = 262144, PIECES_TILES_MOST = 524288, PIECES_SEEN = 204800;
// fewest tiles on either side of a cut (a part costs its result written and read: the time of two bf16 tiles; one of fp32 takes four times as long)
__host__ __device__ __forceinline__ int cut_tiles(uint32_t base) { return base == 32 ? 2 : 1; }
__host__ __device__ __forceinline__ uint32_t piece_work(uint32_t base) { return base == 32 ? 64 : WORK_TILE; }    // the most of a piece while there are workgroups left: four bf16 tiles, one of fp32

struct Cut { int item, tile; };                            // a piece begins at this tile of this item
// The cut `u` into an item of n1 contiguous and n2 packed tiles.
__host__ __device__ __forceinline__ Cut cut_item(uint32_t base, uint32_t u, int item, int n1, int n2) {
    const int tiles = n1 + n2;
    int t = 0;
    if (u >= base + cut_tiles(base) * WORK_TILE) {
        const uint32_t v = u - base;
        t = v < n1 * WORK_TILE ? (int)(v / WORK_TILE) : n1 + (int)((v - n1 * WORK_TILE) / work_cols(base));
        if (t + cut_tiles(base) > tiles) t = tiles;
    }
    return t > 0 && t >= tiles ? Cut{item + 1, 0} : Cut{item, t};
}
// Results of parts that so many pieces may have to keep: one for each that begins inside an item, and one for what was left unfinished
// before it (by item or by piece, whichever are fewer).
__host__ __device__ __forceinline__ int part_slots(int64_t items, int pieces) { return pieces - 1 + (items < pieces ? (int)items : pieces - 1); }
// Number of pieces, no more than `most`, and no more than the workgroups of the launch
__host__ __device__ __forceinline__ int piece_count(uint32_t base, uint32_t work, int64_t items, uint32_t most) {
    uint32_t pieces = (base == 32 ? work : work + WORK_TILE - 1) / piece_work(base), least = items < most ? (uint32_t)items : most;
    if (base != 32 && pieces > 256) pieces = work / work_cols(base) > 256 ? work / work_cols(base) : 256;      // two on some CUs are not the better for it: 4096 rows, all new, 8 heads of 64, 76.6 us, else 78.3
    pieces = pieces > most ? most : pieces < least ? least : pieces;
    // (Two bf16 tiles or one of fp32 a piece, and more.  Pieces a little shorter than a tile leave two cuts in one now and then, and what lies between
    // them is a part without tiles, which is written and weighs nothing; pieces a little longer than one take up two, and the kernel lasts as
    // long as these: 4 heads of 64, 256 rows of 1024, 18.3 us with 9 units a piece, 14.3 with 8; 40 rows of 300, the whole call, 26.7 / 22.1.)
    const uint32_t fewest = base == 32 ? 2 * WORK_TILE : WORK_TILE - 1;
    return pieces <= work / fewest ? (int)pieces : work >= fewest ? (int)(work / fewest) : 1;
}
// where piece p begins
//
// Of the workgroups of a CU the one that came first is served first: of equal pieces, one per place, those of workgroups 0 to 255
// took 220 us, 256 to 511 262 (first turn of 8192 rows), at d = 64 41, 50 and 60 us (5003 rows carried), and a CU left to its last
// workgroup is not busy.  So where every place is taken the pieces of a place are that much larger or smaller.  Shares of
// 64 / 64, 67 / 61, 70 / 58, 73 / 55, 76 / 52, the whole call, us: 8192 rows, all new, 300 / 296 / 291 / 290 / 297, 2048 of 32768 481 / 473 / 465 /
// 460 / 475; at d = 64 64, 69, 74, 79, 84 for the first of three 90 / 88 / 88 / 88 / 87, 5003 rows, all new, 73 / 71 / 71 / 71 / 70.  That was with 72 and 80; the loops as they are leave the first place 5 %
// early so, and 72 and 80 / 74 and 84 / 76 and 88 take 3000 of 20000 rows 590 / 581 / 580, 8192, all new, 289.5 / 286 / 286, 100 of 131072 731 / 731 / 743, at d = 64 8000 of 16384 466 / 459 / 455, 1777 of 5003 150 / 148 / 147.
//
// But not where items of alike work come out in whole pieces, or pieces in whole items (few row blocks a head, `equal` in my_span): then equal
// pieces leave most items uncut, and the query heads of a group, cut at the same tiles, meet at the same keys in the L2.  By place / equal,
// us: 8 dialogues, 8 heads of 128, 2 rows of 98648 keys 551 / 326; 4, 64 heads, 4 rows of 11569, every diagonal, 237 / 164; 4, 32 heads of 64, columns, 331
// rows of 9141 28 / 24; the other way 4, 32 heads, 84 rows of 1435 53 / 57, 2, 64 heads, one of them dense, 3 rows of 116925 115 / 124.  (Short turns of 10 to 130000
// keys, 1 to 64 dialogues: of 108 that are so 27 gain more than 3 %, 7 lose more; of 51 that are not, 12 and 10.  fp32, whose tiles wait for no memory: 52 / 56.)
constexpr uint32_t FIRST_OF_2 = 74, FIRST_OF_3 = 84;       // of 128, of 192 (the second of three: 64)
__host__ __device__ __forceinline__ uint32_t cut_at(uint32_t total, int p, int pieces, bool equal) {
    if (!equal && (pieces == 512 || pieces == 768)) {                  // 32 CUs an XCD, whose workgroups take neighbouring pieces
        const uint32_t places = pieces / 256, xcd = (uint32_t)p / (32 * places), j = (uint32_t)p % (32 * places);
        const uint32_t w0 = places == 2 ? FIRST_OF_2 : FIRST_OF_3, w1 = places == 2 ? 128 - FIRST_OF_2 : 64, w2 = 192 - w0 - w1;
        const uint32_t at = xcd * 32 * 64 * places + (j < 32 ? j * w0 : j < 64 ? 32 * w0 + (j - 32) * w1 : 32 * (w0 + w1) + (j - 64) * w2);
        const uint32_t all = 256 * 64 * places;            // (total % all * at: less than 2^32)
        return total / all * at + total % all * at / all;
    }
    const uint32_t q = total / (uint32_t)pieces, r = total % (uint32_t)pieces;
    return q * (uint32_t)p + ((uint32_t)p < r ? (uint32_t)p : r);
}
// piece of workgroup `id`, or -1
__host__ __device__ __forceinline__ int piece_of(int id, int pieces) {
    const int x = id & 7, j = id >> 3, q = pieces / 8, r = pieces % 8;
    return j < q + (x < r ? 1 : 0) ? x * q + (x < r ? x : r) + j : -1;
}

struct Span { int piece, pieces; Cut from, to; uint32_t rec; };          // from `from` up to, not including, `to`; rec: of from.item where known (else 0)
// The span of this workgroup (all of its 256 threads call; the result is uniform).  piece -1: none.  Two round trips to memory.
__device__ __forceinline__ Span my_span(const PrefillArgs& a, uint32_t* sh) {              // sh: 8 words of LDS
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int per = (a.BH + 255) / 256, h0 = tid * per < a.BH ? tid * per : a.BH, h1 = h0 + per < a.BH ? h0 + per : a.BH;
    uint32_t mine = 0;                                     // (all work there is: less than 2^25, prefill_in_pieces)
    for (int h = h0; h < h1; ++h) mine += a.head_work[h];
    uint32_t inc = mine;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) { const uint32_t t = __shfl_up(inc, off, 64); if (lane >= off) inc += t; }
    if (lane == 63) sh[wv] = inc;
    __syncthreads();
    uint32_t before = inc - mine, total = 0;
#pragma unroll
    for (int w = 0; w < 4; ++w) { const uint32_t t = sh[w]; if (w < wv) before += t; total += t; }
    total = (uint32_t)__builtin_amdgcn_readfirstlane((int)total);
    const int items = a.BH * a.nqb;
    const uint32_t base = work_base(a.dtype);
    Span s;
    s.pieces = piece_count(base, total, items, (uint32_t)a.grid);
    s.piece = piece_of((int)blockIdx.x, s.pieces);
    s.from = s.to = Cut{items, 0};
    s.rec = 0u;
    if (s.piece < 0) return s;
    const bool equal = a.nqb <= 2 && a.dtype == 0 && (s.pieces % items == 0 || items % s.pieces == 0);
    const uint32_t x0 = cut_at(total, s.piece, s.pieces, equal), x1 = cut_at(total, s.piece + 1, s.pieces, equal);
    if (x0 < before + mine && x1 >= before) {
        uint32_t at = before;
        for (int h = h0; h < h1; ++h) {
            const uint32_t next = at + a.head_work[h];
            if (x0 >= at && x0 < next) { sh[4] = (uint32_t)h; sh[5] = x0 - at; }
            if (x1 >= at && x1 < next) { sh[6] = (uint32_t)h; sh[7] = x1 - at; }
            at = next;
        }
    }
    __syncthreads();
    // every wave looks for both ends in the sums of their heads, with the records beside them
    const bool more = s.piece + 1 < s.pieces;
    const int hb = __builtin_amdgcn_readfirstlane((int)sh[4]), he = more ? __builtin_amdgcn_readfirstlane((int)sh[6]) : hb;
    const uint32_t rb = (uint32_t)__builtin_amdgcn_readfirstlane((int)sh[5]), re = (uint32_t)__builtin_amdgcn_readfirstlane((int)sh[7]);
    const uint32_t *ub = a.upto + (int64_t)hb * a.nqb, *ue = a.upto + (int64_t)he * a.nqb;
    const uint32_t *cb = a.rec + (int64_t)hb * a.nqb, *ce = a.rec + (int64_t)he * a.nqb;
    const int l = lane < a.nqb ? lane : a.nqb - 1;
    uint32_t u0 = ub[l], c0 = cb[l], u1 = ue[l], c1 = ce[l];
    auto find = [&](const uint32_t* upto, const uint32_t* recs, uint32_t u, uint32_t c, int h, uint32_t r, uint32_t* rec) -> Cut {
        uint32_t at = 0;                                   // work of the row blocks before q
        for (int q = 0;;) {
            const int n = __popcll(__ballot(q + lane < a.nqb && u <= r));
            if (n > 0) at = (uint32_t)__builtin_amdgcn_readlane((int)u, n - 1);
            if (n < 64) {
                const uint32_t e = (uint32_t)__builtin_amdgcn_readlane((int)c, n);
                const Cut k = cut_item(base, r - at, h * a.nqb + q + n, item_blocks(e), (item_cols(e) + BN - 1) / BN);
                if (rec && k.item == h * a.nqb + q + n) *rec = e;
                return k;
            }
            q += 64;
            const int i = q + lane < a.nqb ? q + lane : a.nqb - 1;
            u = upto[i]; c = recs[i];
        }
    };
    uint32_t rec = 0xFFFFFFFFu;
    s.from = find(ub, cb, u0, c0, hb, rb, &rec);
    if (more) s.to = find(ue, ce, u1, c1, he, re, nullptr);
    s.rec = rec != 0xFFFFFFFFu || s.from.item >= items ? rec : a.rec[s.from.item];      // (a cut moved to the next item: its record)
    if (tid == 0) {                                        // for whoever puts the parts together
        if (!a.arrived) a.cuts[1 + s.piece] = make_int2(s.from.item, s.from.tile);
        else put_shared_word(reinterpret_cast<uint64_t*>(a.cuts + 1 + s.piece), (uint32_t)s.from.item, (uint32_t)s.from.tile | (s.to.item == s.from.item && s.to.tile > 0 ? CUT_ON : 0u));
        if (s.piece == 0) a.cuts[0] = make_int2(s.pieces, 0);
    }
    return s;
}
// Slot of the part with which an item begins on piece p; the one that takes an item up on piece p goes to slot p - 1.
__host__ __device__ __forceinline__ int begin_slot(int item, int p, int64_t items, int pieces) { return pieces - 1 + (items < pieces ? item : p); }

// ---------------------------------------------------------------------------------------------
// sched: builds the 8 work queues of turns beyond PIECES_TILES.  The query heads of one KV head stay together (they share K/V
// tiles in one L2); KV groups are dealt to the XCDs heaviest first, each to the XCD with the least
// work so far.
// One workgroup per queue; groups beyond SCHED_MAX_GROUPS fall back to round-robin dealing.  Inside a
// queue entries are ordered by decreasing tile count, so the long ones start first.
//
// Split items.  A (head, row block) item of a dense head late in the context has hundreds of tiles, and a short turn
// has fewer items than the chip has compute units: one workgroup walking such an item alone decides the kernel's time.
// An item with more than lmax tiles is therefore cut into equal parts that are queued like items; their unnormalised
// results go to `slots` of the workspace and combine_kernel puts them together.  lmax is the mean number of tiles per
// resident workgroup over SPLIT_SHARE, so the longest entry is a fraction of the run, but at least SPLIT_MIN: a part costs a
// 64 KB result written and read (3-4 us of one CU's share of the memory bandwidth) against about 2 us per tile.
// SPLIT_WGS is the resident workgroups of d = 128 for all types and dimensions.  Attention with 256 / 512 / 768, us: first turn of
// 8192 rows 211 / 230 / 230 (d 64: 131 / 147 / 148), 10923 rows of 32768 1596 / 1543 / 1529, 5000 of 16384 at d 64 342 / 350 / 350, 1777
// of 5003 at d 64 108 / 112 / 113, fp32 1024 of 4096 64 / 64 / 64: fewer, longer parts suit short contexts, more the long ones.
// SPLIT_ITEMS is what a copy of all costs in LDS holds.  With 8192 instead: 24000 of 32768 rows (6016 items) 2993 -> 2961 us, first turn of
// 20000 rows (5024 items) 1114 -> 1096, B 2, 64 heads, 7000 of 16384 rows (7040 items) 1687 -> 1696: so many items balance by themselves.
// ---------------------------------------------------------------------------------------------
constexpr int SCHED_MAX_GROUPS = 2048;
constexpr int SCHED_MAX_HEADS = 8192;      // heads one XCD's queue can take
constexpr int SCHED_THREADS = 1024;
constexpr int SPLIT_ITEMS = 4096;          // most items for which splitting is considered
constexpr int SPLIT_SLOTS = 1024;          // most parts of split items
constexpr int SPLIT_MIN = 4;               // tiles
constexpr int SPLIT_SHARE = 2;
constexpr int SPLIT_WGS = 512;
constexpr int SPLIT_MAX_PARTS = 64;
__global__ __launch_bounds__(SCHED_THREADS) void sched_kernel(SchedArgs a) {
    __shared__ uint32_t gcost[SCHED_MAX_GROUPS];
    __shared__ uint16_t order[SCHED_MAX_GROUPS];          // groups by decreasing cost
    __shared__ uint16_t bin_of[SCHED_MAX_GROUPS];
    __shared__ uint32_t hist[4097];
    __shared__ uint16_t heads[SCHED_MAX_HEADS];
    __shared__ uint16_t cost_s[SPLIT_ITEMS];              // costs of all items, where they are few
    __shared__ int nheads;
    __shared__ uint32_t wsum[16], base;                    // base: entries of the queues before this one, which lie ahead of it
    const int tid = threadIdx.x;
    const int groups = a.BH / a.G;
    const bool sorted = groups <= SCHED_MAX_GROUPS;
    const int x = blockIdx.x;
    auto item_cost = [&](uint32_t it) -> int {             // tiles
        const uint32_t r = a.rec[it];
        const int c = item_blocks(r) + (item_cols(r) + BN - 1) / BN;
        return c > 4095 ? 4095 : c;
    };
    const uint32_t all_items = (uint32_t)a.BH * (uint32_t)a.nqb, nqb = (uint32_t)a.nqb;      // at most 8192 * 2050
    const bool cached = all_items <= SPLIT_ITEMS;
    if (cached)
        for (uint32_t it = tid; it < all_items; it += SCHED_THREADS) cost_s[it] = (uint16_t)item_cost(it);
    for (int i = tid; i < 4097; i += SCHED_THREADS) hist[i] = 0u;
    if (tid == 0) { nheads = 0; base = 0u; }
    if (sorted) {                                          // every block repeats this small computation
        for (int gi = tid; gi < groups; gi += SCHED_THREADS) {
            const int b = gi / a.Hkv, kvh = gi % a.Hkv;
            uint32_t c = 0;
            for (int g = 0; g < a.G; ++g) c += a.head_work[b * a.Hq + kvh * a.G + g] / (WORK_TILE * 8);
            gcost[gi] = c;
        }
        __syncthreads();
        for (int gi = tid; gi < groups; gi += SCHED_THREADS) {   // rank sort (ties: smaller index first)
            const uint32_t c = gcost[gi];
            int rank = 0;
            for (int o = 0; o < groups; ++o) { const uint32_t d = gcost[o]; rank += (d > c) || (d == c && o < gi); }
            order[rank] = (uint16_t)gi;
        }
        __syncthreads();
        if (tid < 64) {                                    // one wave deals them out; lane l < 8 holds bin l's load
            uint32_t load = 0;                             // (eights of tiles: all heads together have less than 2^28)
            for (int r = 0; r < groups; ++r) {
                const int gi = order[r];
                uint32_t best = tid < 8 ? (load << 3 | tid) : 0xFFFFFFFFu;           // least load, then least index
#pragma unroll
                for (int off = 4; off > 0; off >>= 1) { const uint32_t o = __shfl_xor(best, off, 64); best = o < best ? o : best; }
                const int bin = (int)(__builtin_amdgcn_readfirstlane((int)best) & 7);
                if (tid == bin) load += gcost[gi] + 1;
                if (tid == 0) bin_of[gi] = (uint16_t)bin;
            }
        }
    }
    __syncthreads();
    uint8_t* head_bin = reinterpret_cast<uint8_t*>(gcost);  // (the costs of the groups have been used; at most 8192 heads)
    static_assert(SCHED_MAX_HEADS <= sizeof(gcost), "a byte for every head");
    for (int bh = tid; bh < a.BH; bh += SCHED_THREADS) {   // heads of this bin (order inside the list is free)
        const int b = bh / a.Hq, h = bh % a.Hq, gi = b * a.Hkv + h / a.G;
        const int bin = sorted ? (int)bin_of[gi] : (gi & 7);
        head_bin[bh] = (uint8_t)bin;
        if (bin == x) { const int i = atomicAdd(&nheads, 1); if (i < SCHED_MAX_HEADS) heads[i] = (uint16_t)bh; }
    }
    // what is cut into parts: the same in every block, from the costs of all items
    int lmax = 1 << 30;
    if (cached) {
        int c4[SPLIT_ITEMS / SCHED_THREADS];
        uint32_t mine = 0, total, used = 0;
#pragma unroll
        for (int j = 0; j < SPLIT_ITEMS / SCHED_THREADS; ++j) {
            const int it = tid + j * SCHED_THREADS;
            c4[j] = it < (int)all_items ? cost_s[it] : 0;
            mine += (uint32_t)c4[j];
        }
        (void)block_scan_1024(mine, wsum, total);
        if (a.slots > 0) {
            lmax = (int)(total / (SPLIT_WGS * SPLIT_SHARE));
            if (lmax < SPLIT_MIN) lmax = SPLIT_MIN;
            for (;;) {                                     // until the parts fit the slots (lmax >= 4096: nothing is split)
                mine = 0;
#pragma unroll
                for (int j = 0; j < SPLIT_ITEMS / SCHED_THREADS; ++j) {
                    int parts = (c4[j] + lmax - 1) / lmax;
                    if (parts > SPLIT_MAX_PARTS) parts = SPLIT_MAX_PARTS;
                    mine += parts > 1 ? (uint32_t)parts : 0u;
                }
                (void)block_scan_1024(mine, wsum, used);
                if (used <= (uint32_t)a.slots || lmax >= 4096) break;
                lmax += (lmax + 1) / 2;
            }
            if (used > (uint32_t)a.slots) lmax = 1 << 30;
        }
    }
    const bool splits = lmax < 4096;
    auto parts_of = [&](int c) -> int {
        const int p = splits ? (c + lmax - 1) / lmax : 1;
        return p < 1 ? 1 : p > SPLIT_MAX_PARTS ? SPLIT_MAX_PARTS : p;
    };
    __syncthreads();
    uint32_t ahead = 0;
    if (splits) {
        for (uint32_t it = tid; it < all_items; it += SCHED_THREADS) if (head_bin[it / nqb] < x) ahead += (uint32_t)parts_of(cost_s[it]);
    } else {
        for (int bh = tid; bh < a.BH; bh += SCHED_THREADS) if (head_bin[bh] < x) ahead += nqb;
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) ahead += __shfl_xor(ahead, off, 64);
    if ((tid & 63) == 0 && ahead) atomicAdd(&base, ahead);
    const int nh_ = nheads < SCHED_MAX_HEADS ? nheads : SCHED_MAX_HEADS;
    const uint32_t items = (uint32_t)nh_ * nqb;
    for (uint32_t i = tid; i < items; i += SCHED_THREADS) {
        const uint32_t it = heads[i / nqb] * nqb + i % nqb;
        const int c = cached ? cost_s[it] : item_cost(it), p = parts_of(c);
        atomicAdd(&hist[4095 - (c + p - 1) / p], (uint32_t)p);
    }
    __syncthreads();
    uint32_t entries;
    {                                                      // exclusive scan in decreasing-cost order
        uint32_t h4[4], mine = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) { h4[q] = hist[4 * tid + q]; mine += h4[q]; }
        uint32_t run = block_scan_1024(mine, wsum, entries);
#pragma unroll
        for (int q = 0; q < 4; ++q) { hist[4 * tid + q] = run; run += h4[q]; }
    }
    __syncthreads();
    for (uint32_t i = tid; i < items; i += SCHED_THREADS) {
        const uint32_t it = heads[i / nqb] * nqb + i % nqb;
        const int c = cached ? cost_s[it] : item_cost(it), p = parts_of(c);
        const uint32_t posn = atomicAdd(&hist[4095 - (c + p - 1) / p], (uint32_t)p);
        uint32_t slot0 = 0;
        if (p > 1) {                                       // slots and the list of split items are shared by the 8 blocks
            slot0 = (uint32_t)atomicAdd(&a.split_count[0], p);
            a.split[atomicAdd(&a.split_count[1], 1)] = make_uint2(it, (uint32_t)p | (slot0 << 16));
        }
        const uint32_t r = a.rec[it];
        uint4* q = a.queue + base + posn;
        for (int e = 0; e < p; ++e) q[e] = make_uint4(it, (uint32_t)e | ((uint32_t)p << 8) | (slot0 << 16), (uint32_t)item_blocks(r), (uint32_t)item_cols(r));
    }
    if (tid == 0) { a.qlen[x] = (int)entries; a.qbase[x] = (int)base; a.qhead[x] = (a.grid - x + 7) / 8; }
}

// Launch of the attention kernel: the workgroups that are resident at once (256 CUs x per_cu, see prefill_bf16_kernel); any number drains the
// queues, but a surplus one only starts when another ends and lengthens the run by its look at the queues.
//
// Pieces: as many to an item as fill the chip, but no more than combine_kernel adds up in the time that they save.  The whole call, us, 12 / 24 / 48 of
// an item: bf16, heads of 128, 64 rows of 65536, 4 heads 132 / 82 / 61, 61 rows, 32 heads (384 workgroups / 512) 177 / 152, with lists of few lines 82 / 84; one head of 64, 64 rows of 16384 43 / 34 / 31.
// fp32, whose tiles keep a CU's matrix cores busy, up to one workgroup a CU; a few more would be two on some CUs: one head of 64, 64 rows of 16384 126 / 77 / 53,
// 4 heads, 16 of 4096 47 / 35 / 34, but 512 of 4096 (240 workgroups / 480 / 512) 53 / 54 / 68, 32 heads, 64 of 2048 (384 / 512) 48 / 55.
// No more than there can be work for: 4 heads, 64 rows of 1024 keys, 192 workgroups / 20 28.5 / 28.0.  Where a dozen parts each take less than 15 MB of workspace, more do not take more than that: a caller's fixed 16 MB hold the same shapes as with a dozen.
// (A step, no bound: at d = 128 18 row blocks are cut into 220 parts, 15 MB, 19 into 512, 35 MB, as from 43 on a dozen parts each are.  In a workspace made for a dozen they go in a dozen.)
constexpr int ITEM_PARTS = 12, ITEM_PIECES = 48;
constexpr int64_t PIECES_BYTES = 15 << 20;
int prefill_grid(int dtype, int d, int64_t n, int64_t items, bool pieces) {
    const int per_cu = dtype == 0 ? (d == 128 ? 2 : 3) + (pieces ? 0 : 1) : (d == 128 ? 1 : 2);
    int64_t most;
    if (pieces) {
        const int64_t keys = (n + BN - 1) / BN, base = work_base(dtype), piece = piece_work(base);
        const int64_t each = (base + keys * (WORK_TILE + work_cols(base)) + piece - 1) / piece;      // pieces of an item that visits every key both ways
        const int64_t all = each < 2 ? 2 : each;           // (of one there is nothing to put together: a workspace without room for that takes the queues)
        const int64_t dozen = items * (all < ITEM_PARTS ? all : ITEM_PARTS), fit = PIECES_BYTES / (int64_t)prefill_slot_bytes(d) - items;
        most = items * (all < ITEM_PIECES ? all : ITEM_PIECES);
        if (dtype != 0 && most > 256) most = 256;
        if (dozen <= fit && most > fit) most = fit;
        if (most < dozen) most = dozen;
    } else most = items + prefill_split_slots(items, 0, false);
    return (int)(most < 256 * per_cu ? most : 256 * per_cu);
}
int prefill_split_slots(int64_t items, int grid, bool pieces) {
    if (pieces) return part_slots(items, grid);
    return items > SPLIT_ITEMS ? 0 : items * ITEM_PARTS < SPLIT_SLOTS ? (int)items * ITEM_PARTS : SPLIT_SLOTS;
}
bool prefill_in_pieces(int BH, int64_t n, int nqb, int dtype, int d) {
    const int64_t items = (int64_t)BH * nqb, keys = (n + BN - 1) / BN, tiles = items * keys * d / 128;
    if (dtype != 0) return tiles <= PIECES_TILES_MOST;
    const bool alike = d == 64 ? items <= 5120 : items >= 704 && items <= 2560;
    return tiles <= (alike ? PIECES_TILES_MOST : PIECES_TILES) || items * (keys - (BM / BN) * (nqb - 1) / 2) * d / 128 <= PIECES_SEEN;
}

// Pieces, of up to `grid`, whose parts `slots` hold; 0: the queues serve the call better.  Fewer pieces than workgroups make the run about
// grid / pieces as long (of three places a CU only 5 % where two are filled), queues about a quarter of grid / items longer.  The whole
// call with all slots / 90, 75, 67, 50, 40, 25 % of them, us, pieces; and queues:
// 8192 rows, all new, 32 heads of 128 (4 items a workgroup) 274 / 295 337 371 396 484 736; 294 to 307. 16 heads of 64 (1.3) 75 / 79 85 76 94 110 131;
// 96 to 115.  6000 of 9000, 32 heads (3) 242 / 265 305 337 349 423 649; 259 to 268.  4096, all new, 8 heads of 128 (0.5) 62 / 64 70 68 78 86 117;
// 72 to 94.  300 of 16384, 32 heads (0.2) 62 / 62 62 64 67 79 122; 76 to 94.  1777 of 5003, 16 heads of 64 (0.3) 50 / 53 53 53 61 63 84; 74 to 104.
int prefill_pieces_for(int64_t items, int grid, int slots) {
    if (slots >= part_slots(items, grid)) return grid;
    const int64_t pieces = 1 + (slots > 2 * items ? slots - items : slots / 2);
    if (grid > 512 && pieces >= 512) return items <= 5 * (int64_t)grid ? 512 : 0;
    return pieces > 1 && 4 * items * (grid - pieces) <= grid * pieces ? (int)pieces : 0;
}
bool prefill_joins(int dtype, int64_t items, int grid) { return dtype == 0 && items >= 2 * (int64_t)grid; }
int prefill_piece_xcd(int p, int pieces) {
    for (int id = 0; id < 8; ++id)
        for (int j = id; piece_of(j, pieces) >= 0; j += 8) if (piece_of(j, pieces) == p) return id;
    return -1;
}

// Queue entries for this workgroup, called by one whole wave.  The first entry is the workgroup's own place in its
// XCD's queue (sched_kernel starts the counters behind those), later ones come from the counters: the own queue while
// it has any, then the others in ring order, all eight looked at in one round trip.  While the own queue is far from
// its end the counter is updated without a look, and beside the other waves' stores of the last results (`ahead`); near
// the end every workgroup would update it once for nothing, and updates of one counter take turns.  item = ~0 when every
// queue is drained (each queue hands out each entry once and never refills, so the search ends).
struct QueueSource {
    int own;
    int at;                                   // place taken in the own queue, -1: none
    bool plenty;
    // [8] lengths, [8] first entries of the queues (in LDS: one wave looks at them once an entry)
    __device__ __forceinline__ static int* queues() { __shared__ int q[16]; return q; }
    __device__ __forceinline__ void init(const PrefillArgs& a, int) {
        own = blockIdx.x & 7; at = (int)(blockIdx.x >> 3); plenty = true;
        if (threadIdx.x < 16) queues()[threadIdx.x] = threadIdx.x < 8 ? a.qlen[threadIdx.x] : a.qbase[threadIdx.x - 8];      // (read by the same wave)
    }
    __device__ __forceinline__ void ahead(const PrefillArgs& a, int lane) {
        if (!plenty) return;
        int i = 0;
        if (lane == 0) i = atomicAdd(&a.qhead[own], 1);
        at = __builtin_amdgcn_readfirstlane(i);
    }
    __device__ __forceinline__ uint4 next(const PrefillArgs& a, int lane) {
        asm volatile("" : "+v"(lane));      // (addresses made of it are not to be kept through an entry)
        const int x = (own + lane) & 7, len = lane < 8 ? queues()[x] : 0, base = queues()[8 + x];      // lane l < 8: queue (own + l) % 8
        const int own_len = __builtin_amdgcn_readfirstlane(len);
        if (at >= 0 && at < own_len) {
            const int i = at;
            at = -1;
            plenty = own_len - i > 128;
            return a.queue[__builtin_amdgcn_readfirstlane(base) + i];
        }
        at = -1;
        plenty = false;
        for (;;) {
            const bool some = lane < 8 && __atomic_load_n(&a.qhead[x], __ATOMIC_RELAXED) < len;
            const uint64_t any = __ballot(some);
            if (any == 0ull) return make_uint4(0xFFFFFFFFu, 0u, 0u, 0u);
            const int src = __ffsll((unsigned long long)any) - 1;
            int i = 0;
            if (lane == src) i = atomicAdd(&a.qhead[x], 1);
            i = __builtin_amdgcn_readlane(i, src);
            if (i < __builtin_amdgcn_readlane(len, src)) {
                plenty = src == 0 && own_len - i > 128;
                return a.queue[__builtin_amdgcn_readlane(base, src) + i];
            }
        }
    }
};

// What a workgroup does next: an item, or a part of one.
struct Entry {
    int item, blocks, cols;                   // the item's contiguous tiles and columns
    int lo, hi;                               // queues: part lo of hi; pieces: from tile lo on, up to tile hi (-1: the last)
    int slot0, slot1;                         // queues: -1, slot of the part; pieces: slots for the part that begins and for the one that goes on
    __device__ __forceinline__ int begin(int tiles) const { return slot0 < 0 ? tiles * lo / hi : lo; }
    __device__ __forceinline__ int end(int tiles) const { return slot0 < 0 ? tiles * (lo + 1) / hi : hi < 0 ? tiles : hi; }
    __device__ __forceinline__ bool in_parts(int tiles) const { return slot0 < 0 ? hi > 1 : lo > 0 || (hi >= 0 && hi < tiles); }
    __device__ __forceinline__ int slot() const { return slot0 < 0 || lo > 0 ? slot1 : slot0; }
};
template <bool QUEUES> struct Entries;
template <> struct Entries<true> {
    QueueSource src;
    __device__ __forceinline__ Span span() const { return Span{}; }
    __device__ __forceinline__ void init(const PrefillArgs& a, int lane) { src.init(a, lane); }
    __device__ __forceinline__ void ahead(const PrefillArgs& a, int lane, int wv) { if (wv == 0) src.ahead(a, lane); }
    __device__ __forceinline__ bool next(const PrefillArgs& a, int lane, int wv, Entry& e) {
        __shared__ uint4 entry_s;
        if (wv == 0) {                        // (the other waves have read the last entry: barriers came after it)
            const uint4 t = src.next(a, lane);
            if (lane == 0) entry_s = t;
        }
        __syncthreads();
        const uint32_t item = (uint32_t)__builtin_amdgcn_readfirstlane((int)entry_s.x), info = (uint32_t)__builtin_amdgcn_readfirstlane((int)entry_s.y);
        e.blocks = __builtin_amdgcn_readfirstlane((int)entry_s.z); e.cols = __builtin_amdgcn_readfirstlane((int)entry_s.w);
        e.item = (int)item; e.lo = info & 0xFF; e.hi = (info >> 8) & 0xFF; e.slot0 = -1; e.slot1 = (int)(info >> 16) + e.lo;
        return item != 0xFFFFFFFFu;
    }
};
template <> struct Entries<false> {
    Span s;
    int at, last;
    uint32_t rec;                             // of item `at`
    __device__ __forceinline__ const Span& span() const { return s; }
    __device__ __forceinline__ void init(const PrefillArgs& a, int lane) {
        __shared__ uint32_t span_s[8];
        s = my_span(a, span_s);
        at = s.from.item;
        last = s.to.item - (s.to.tile > 0 ? 0 : 1);
        rec = s.rec;
    }
    __device__ __forceinline__ void ahead(const PrefillArgs& a, int, int) { if (at <= last) rec = a.rec[at]; }
    __device__ __forceinline__ bool next(const PrefillArgs& a, int, int, Entry& e) {
        const uint32_t r = (uint32_t)__builtin_amdgcn_readfirstlane((int)rec);
        e.item = at; e.blocks = item_blocks(r); e.cols = item_cols(r); e.slot0 = begin_slot(at, s.piece, (int64_t)a.BH * a.nqb, s.pieces); e.slot1 = s.piece - 1;
        e.lo = at == s.from.item ? s.from.tile : 0;
        e.hi = at == s.to.item ? s.to.tile : -1;
        return at++ <= last;
    }
};

// Word of a.cuts: the tile at which a piece begins, and whether the piece ends inside the same item
__device__ __forceinline__ int cut_tile(int y) { return y & (int)~CUT_ON; }

// Unnormalised result of one part of a split item: accumulators lane by lane (16 bytes a lane, 1 KB a store) and
// {reference, normaliser} per row.
template <int DBLK>
__device__ __forceinline__ void store_part(const PrefillArgs& a, int slot, int wv, int lane, const f32x16 (&oacc)[DBLK], float m, float l) {
    float* o = a.part_o + (int64_t)slot * (BM * 32 * DBLK) + wv * (DBLK * 4 * 256) + lane * 4;
#pragma unroll
    for (int i = 0; i < DBLK; ++i)
#pragma unroll
        for (int rq = 0; rq < 4; ++rq)
            *reinterpret_cast<f32x4*>(o + (i * 4 + rq) * 256) = f32x4{oacc[i][4 * rq], oacc[i][4 * rq + 1], oacc[i][4 * rq + 2], oacc[i][4 * rq + 3]};
    if (lane < 32) reinterpret_cast<float2*>(a.part_ml)[(int64_t)slot * BM + 32 * wv + lane] = make_float2(m, l);
}

// Pieces, where there are at least two items to a workgroup: an item's parts are put together by the workgroup that comes to the end of its part last
// (the count of the item's tiles that are done tells; plan_kernel has cleared it).  Where all others are there, its own part is not stored at all:
// mostly the one at the end of a piece, since the next piece began with the other.  The parts are added in the order of their tiles,
// so the result does not depend on who comes last, and nobody waits for anybody.  All threads of the workgroup call; returns whether oacc, m and l are
// the item's now.
//
// Against combine_kernel this saves a launch and a write and a read of half of the parts: the attention of 8192 rows, all new, 32 heads of 128 266 -> 257 us,
// of 64 216 -> 211, B 1, 64 heads, 2000 of 3000 rows 121 -> 114; one head dense and 100 diagonals of the others 114 -> 112, 82 -> 83, 65 -> 63.  What bounds it is what a
// compute unit alone can read, 30 to 50 KB a us, part after part.  So not where an item has many parts (with combine_kernel / so,
// us: 16 heads of 64, 1024 rows of 8192 47 / 57, 20 of 40000 66 / 112), nor where one dense head among others gives a few items many (16 heads of 64, 8192 of 20000 rows,
// 1.3 items a workgroup 90 / 97).
template <int DBLK, int NB>
__device__ __forceinline__ bool join_parts(const PrefillArgs& a, const Entry& en, const Span& s, int total, int here, int wv, int lane, bool rows_here, f32x16 (&oacc)[DBLK], float& m, float& l) {
    __shared__ uint32_t count_s;
    uint32_t* count = a.arrived + en.item;
    if (threadIdx.x == 0) count_s = __hip_atomic_load(count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    bool last = __builtin_amdgcn_readfirstlane((int)count_s) + here == total;
    __syncthreads();
    const int64_t at = wv * (DBLK * 16 * 64) + 2 * lane;   // two values of a lane at a time, 512 bytes a store
    const int piece = s.piece, pieces = s.pieces;
    if (!last) {
        if (rows_here) {
            float* o = a.part_o + (int64_t)en.slot() * (BM * 32 * DBLK) + at;
#pragma unroll
            for (int i = 0; i < DBLK; ++i)
#pragma unroll
                for (int r = 0; r < 16; r += 2) put_shared2(o + (16 * i + r) * 64, oacc[i][r], oacc[i][r + 1]);
            if (lane < 32) put_shared2(a.part_ml + 2 * ((int64_t)en.slot() * BM + 32 * wv + lane), m, l);
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (threadIdx.x == 0) count_s = __hip_atomic_fetch_add(count, (uint32_t)here, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
        last = __builtin_amdgcn_readfirstlane((int)count_s) + here == total;
    }
    if (!last) return false;
    if (!rows_here) return true;
    // the item's pieces: from the one that does not begin inside it to the one that does not end inside it
    auto cut = [&](int p) -> int2 {
        const uint64_t u = __hip_atomic_load(reinterpret_cast<const uint64_t*>(a.cuts + 1 + p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return make_int2(__builtin_amdgcn_readfirstlane((int)(uint32_t)u), __builtin_amdgcn_readfirstlane((int)(uint32_t)(u >> 32)));
    };
    int first = piece, end = piece;
    if (en.lo > 0)
        for (;;) { --first; const int2 c = cut(first); if (c.x != en.item || cut_tile(c.y) == 0) break; }
    if (en.hi >= 0)
        for (;;) { ++end; if (!(cut(end).y & (int)CUT_ON)) break; }
    auto slot_of = [&](int p) -> int64_t { return p == first ? begin_slot(en.item, first, (int64_t)a.BH * a.nqb, pieces) : p - 1; };
    const int row = 32 * wv + (lane & 31);
    f32x16 acc[DBLK];
#pragma unroll
    for (int i = 0; i < DBLK; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][r] = 0.f;
    float M = -INFINITY, L = 0.f;
    for (int p0 = first; p0 <= end; p0 += NB) {            // so many parts' loads in flight (the last part is repeated with weight 0)
        float2 ml[NB], x[NB][DBLK * 8];
#pragma unroll
        for (int e = 0; e < NB; ++e) {
            const int p = p0 + e < end ? p0 + e : end;
            const float* o = a.part_o + slot_of(p) * (BM * 32 * DBLK) + at;
            ml[e] = get_shared2(a.part_ml + 2 * (slot_of(p) * BM + row));
#pragma unroll
            for (int k = 0; k < DBLK * 8; ++k) x[e][k] = get_shared2(o + k * 128);
        }
        float m_new = M;
#pragma unroll
        for (int e = 0; e < NB; ++e) {
            if (p0 + e == piece) {                         // (uniform; what is read of its slot may be anything)
                ml[e] = make_float2(m, l);
#pragma unroll
                for (int k = 0; k < DBLK * 8; ++k) x[e][k] = make_float2(oacc[k / 8][2 * (k % 8)], oacc[k / 8][2 * (k % 8) + 1]);
            }
            if (p0 + e > end) ml[e].x = -INFINITY;
            m_new = fmaxf(m_new, ml[e].x);
        }
        const float corr = M > -INFINITY ? fast_exp2(M - m_new) : 0.f;
        M = m_new;
        L *= corr;
#pragma unroll
        for (int i = 0; i < DBLK; ++i) acc[i] *= corr;
#pragma unroll
        for (int e = 0; e < NB; ++e) {
            if (p0 + e > end) break;
            const float wgt = ml[e].x > -INFINITY ? fast_exp2(ml[e].x - M) : 0.f;
            L += ml[e].y * wgt;
#pragma unroll
            for (int k = 0; k < DBLK * 8; ++k) {
                acc[k / 8][2 * (k % 8)] += x[e][k].x * wgt;
                acc[k / 8][2 * (k % 8) + 1] += x[e][k].y * wgt;
            }
        }
    }
#pragma unroll
    for (int i = 0; i < DBLK; ++i) oacc[i] = acc[i];
    m = M; l = L;
    return true;
}

// ---------------------------------------------------------------------------------------------
// the attention kernel
// ---------------------------------------------------------------------------------------------
template <typename T, int D>
struct TileCfg {
    static constexpr int EB = Elem<T>::bytes;
    static constexpr int EPC = Elem<T>::per16;            // elements per 16-byte chunk
    static constexpr int CPR = D / EPC;                   // 16-byte chunks per K/V row
    static constexpr int CPT = CPR / 4;                   // chunks each thread moves per tile and operand
    static constexpr int K_STRIDE = D * EB + 16;          // bytes per staged K row
    static constexpr int VT_STRIDE = BN * EB + 16;        // bytes per staged V^T row
    static constexpr int K_BYTES = BN * K_STRIDE;
    static constexpr int VT_BYTES = D * VT_STRIDE;
    static constexpr int KSTEPS = D / 16;                 // k chunks of the QK^T product
    static constexpr int DBLK = D / 32;                   // 32-wide output column blocks
};

// raw holds 16 bytes of one V row: elements d0 .. d0 + 3; scatter them down column `col`.
__device__ __forceinline__ void store_vt(unsigned char* vt, int stride, int d0, int col, const f32x4 raw) {
    *reinterpret_cast<float*>(vt + (d0 + 0) * stride + col * 4) = raw.x;
    *reinterpret_cast<float*>(vt + (d0 + 1) * stride + col * 4) = raw.y;
    *reinterpret_cast<float*>(vt + (d0 + 2) * stride + col * 4) = raw.z;
    *reinterpret_cast<float*>(vt + (d0 + 3) * stride + col * 4) = raw.w;
}

__device__ __forceinline__ void store_out4(bf16_t* p, float a, float b, float c, float d) {
    typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
    *reinterpret_cast<bf16x4*>(p) = __builtin_convertvector((f32x4{a, b, c, d}), bf16x4);      // round to nearest even
}
__device__ __forceinline__ void store_out4(float* p, float a, float b, float c, float d) {
    const f32x4 v = {a, b, c, d};
    *reinterpret_cast<f32x4*>(p) = v;
}

// Puts the parts of the split items together.  Queues: `split` lists them.  Pieces: the cuts tell; the part that begins an item
// lies in the slot of the item (or of its piece, where there are more items than pieces) behind those of the cuts, the
// others in the slots of theirs.  A unit is one wave's 32 rows of a split item, taken by one workgroup in the layout store_part
// wrote: wave w adds the groups w, w + 4, ... of 16 bytes a lane.  Queues: grid-stride over the units.  Pieces: four units a cut, a
// workgroup each (512 workgroups in all: 5003 rows carried, d = 64, 13.4 us instead of 10.3, first turn of 8192 rows 17.6 instead of 15.7,
// which is 65 MB read at 4.2 TB/s).
template <typename T, int D, bool QUEUES>
__global__ __launch_bounds__(256) void combine_kernel(PrefillArgs a) {
    constexpr int DBLK = D / 32;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, r32 = lane & 31, g = lane >> 5;
    const int units = QUEUES ? a.split_count[1] * 4 : (a.grid - 1) * 4;
    for (int u = blockIdx.x; u < units; u += gridDim.x) {
        const int wv = u & 3;
        int item, parts, begin, rest;                      // begin: slot of part 0; rest + p: slot of part p > 0
        if constexpr (QUEUES) {
            const uint2 e = a.split[u >> 2];
            item = (int)e.x; parts = (int)(e.y & 0xFFFF); begin = rest = (int)(e.y >> 16);
        } else {
            const int first = u >> 2, p = first + 1 + lane;              // the item's first piece, if the next begins inside it
            const int2* cuts = a.cuts + 1;
            const int pieces = a.cuts[0].x;
            const int2 c0 = cuts[first], c1 = cuts[first + 1];
            int2 c = cuts[p < a.grid ? p : a.grid - 1];                  // (asked for at once; those of no piece are not looked at)
            if (first + 1 >= pieces || c1.y == 0 || (c0.x == c1.x && c0.y > 0)) continue;       // no cut through an item, or not its first
            item = c1.x; parts = 1;                        // the first, and one for every piece that begins inside the item
            for (;;) {
                const uint64_t no = ~__ballot(first + parts + lane < pieces && c.x == item);
                const int more = no ? __ffsll((unsigned long long)no) - 1 : 64;
                parts += more;
                if (more < 64) break;
                const int q = first + parts + lane;
                c = cuts[q < a.grid ? q : a.grid - 1];
            }
            begin = begin_slot(item, first, a.BH * (int64_t)a.nqb, pieces); rest = first - 1;
        }
        const int bh = item / a.nqb, qb = item % a.nqb;
        const int64_t row0 = a.n - a.n_hat, pos = a.pos0 + (int64_t)qb * BM + 32 * wv + r32;
        if (pos < row0 || pos >= a.n) continue;
        auto slot_of = [&](int p) -> int64_t { return p == 0 ? begin : rest + p; };
        const float2* ml = reinterpret_cast<const float2*>(a.part_ml) + 32 * wv + r32;
        const float* o = a.part_o + wv * (DBLK * 4 * 256) + lane * 4;
        f32x4 acc[DBLK];
#pragma unroll
        for (int k = 0; k < DBLK; ++k) acc[k] = f32x4{0.f, 0.f, 0.f, 0.f};
        float m = -INFINITY, l = 0.f;
        for (int p0 = 0; p0 < parts; p0 += 4) {            // four parts' loads in flight (the last part is repeated with weight 0)
            float2 t[4];
            f32x4 x[4][DBLK];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int p = p0 + e < parts ? p0 + e : parts - 1;
                t[e] = ml[slot_of(p) * BM];
                if (p0 + e >= parts) t[e].x = -INFINITY;
#pragma unroll
                for (int k = 0; k < DBLK; ++k) x[e][k] = *reinterpret_cast<const f32x4*>(o + slot_of(p) * (BM * D) + (w + 4 * k) * 256);
            }
            const float m_new = fmaxf(fmaxf(fmaxf(m, t[0].x), fmaxf(t[1].x, t[2].x)), t[3].x);
            const float corr = m > -INFINITY ? fast_exp2(m - m_new) : 0.f;
            m = m_new;
            l *= corr;
#pragma unroll
            for (int k = 0; k < DBLK; ++k) acc[k] *= corr;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float wgt = t[e].x > -INFINITY ? fast_exp2(t[e].x - m) : 0.f;
                l += t[e].y * wgt;
#pragma unroll
                for (int k = 0; k < DBLK; ++k) acc[k] += x[e][k] * wgt;
            }
        }
        const float inv = l > 0.f ? 1.0f / l : 0.f;
        T* orow = reinterpret_cast<T*>(a.out) + ((int64_t)bh * a.n_hat + (pos - row0)) * D;
#pragma unroll
        for (int k = 0; k < DBLK; ++k) {
            const int grp = w + 4 * k, d0 = 32 * (grp >> 2) + 8 * (grp & 3) + 4 * g;
            store_out4(orow + d0, acc[k].x * inv, acc[k].y * inv, acc[k].z * inv, acc[k].w * inv);
        }
        if (a.lse && g == 0 && w == 0)
            a.lse[(int64_t)bh * a.n_hat + (pos - row0)] = l > 0.f ? (m + log2f(l)) * 0.69314718055994531f : -INFINITY;
    }
}

// ---- cell masks -------------------------------------------------------------------------------
// A wave's 32 rows start at a position that is a multiple of 32 and a contiguous tile at a key that is one of 64, so
// row i and key k of the tile meet on diagonal 32 Q + i - k with a wave-uniform Q: three words of the bitmap cover the
// wave's part of the tile, and the bits a lane needs are a shift by its row.  The words are uniform (scalar loads,
// requested one tile ahead), and so are the questions whether a 32 x 32 sub-tile has an allowed cell at all and
// whether all of its cells are allowed.  (Bit by bit windows with 64-bit index arithmetic per lane and a ballot per
// question took 103 instructions per wave and tile of about 600.)
typedef const __attribute__((address_space(4))) uint32_t* const_words;    // read-only for the whole kernel: scalar loads

struct DiagWords { uint32_t x0, x1, x2; };                // diagonals 32 Q - 64 .. 32 Q + 31
__device__ __forceinline__ DiagWords diag_words(const_words ob, int posw, int key0) {
    const int q = (posw - key0) >> 5;                     // >= -2
    return {ob[q - 2 + OB_PAD], ob[q - 1 + OB_PAD], ob[q + OB_PAD]};
}
// What a wave may see of a 64-key tile: bit 8 (r/4) + r % 4 of am[h] = key 32 h + 8 (r/4) + 4 g + r % 4 is allowed for
// this lane's row (the key that accumulator register r of the lane holds)
struct TileMask { uint32_t am[2]; bool act[2], full[2]; };
__device__ __forceinline__ TileMask diag_mask(const DiagWords& w, int r32, int g) {
    TileMask m;
    m.act[0] = ((w.x1 & ~1u) | w.x2) != 0u;
    m.act[1] = ((w.x0 & ~1u) | w.x1) != 0u;
    m.full[0] = (w.x2 & (w.x1 | 1u)) == 0xFFFFFFFFu;
    m.full[1] = (w.x1 & (w.x0 | 1u)) == 0xFFFFFFFFu;
    m.am[0] = __brev((uint32_t)((((uint64_t)w.x2 << 32) | w.x1) >> (r32 + 1))) >> (4 * g);
    m.am[1] = __brev((uint32_t)((((uint64_t)w.x1 << 32) | w.x0) >> (r32 + 1))) >> (4 * g);
    return m;
}
// 32 x 32 bit transpose inside each half of the wave: bit c of lane r <- bit r of lane c
__device__ __forceinline__ uint32_t transpose32(uint32_t x, int lane) {
    // (written without a choice between two expressions: the compiler made branches of those)
#define LS_STEP(b, m, moved)                                                                          \
    { const uint32_t p = (uint32_t)(moved), hi = (uint32_t)__builtin_amdgcn_sbfe(lane, b, 1), mk = (m) ^ ~hi;   \
      const uint32_t y = ((p >> (1 << (b))) & hi) | ((p << (1 << (b))) & ~hi); x = (y & mk) | (x & ~mk); }
    LS_STEP(4, 0x0000FFFFu, __builtin_amdgcn_ds_swizzle((int)x, 0x401F))                              // lane ^ 16
    LS_STEP(3, 0x00FF00FFu, __builtin_amdgcn_update_dpp(0, (int)x, 0x128 /* row_ror:8 */, 0xF, 0xF, false))
    LS_STEP(2, 0x0F0F0F0Fu, __builtin_amdgcn_ds_swizzle((int)x, 0x101F))                               // lane ^ 4
    LS_STEP(1, 0x33333333u, __builtin_amdgcn_update_dpp(0, (int)x, 0x4E /* quad_perm 2,3,0,1 */, 0xF, 0xF, false))
    LS_STEP(0, 0x55555555u, __builtin_amdgcn_update_dpp(0, (int)x, 0xB1 /* quad_perm 1,0,3,2 */, 0xF, 0xF, false))
#undef LS_STEP
    return x;
}
// The same in pieces: what a lane sees of a half whose words are hi and lo, and whether the half has an allowed cell (1) and nothing else (4)
__device__ __forceinline__ uint32_t diag_cells(uint32_t hi, uint32_t lo, int r32, int g) {
    const uint64_t w = (((uint64_t)hi << 32) | lo) >> 1;   // (uniform)
    return __brev(__builtin_amdgcn_alignbit((uint32_t)(w >> 32), (uint32_t)w, (uint32_t)r32)) >> (4 * g);
}
__device__ __forceinline__ int diag_half(uint32_t hi, uint32_t lo) {      // (as asm statements it stays in scalar registers)
    uint32_t any, out;
    asm("s_min_u32 %0, %1, 1" : "=s"(any) : "s"((lo & ~1u) | hi) : "scc");
    asm("s_min_u32 %0, %1, 1" : "=s"(out) : "s"(~(hi & (lo | 1u))) : "scc");
    return (int)(any | (out ^ 1u) << 2);
}
// Packed columns: lane l answers for column `col` (slot l of the tile; -1: none) and all 32 rows of the wave at once,
// 32 bits of the bitmap in two words, and one bit transpose hands the rows their columns.  (Each lane testing the
// columns of its row one after the other was a chain of up to 64 LDS reads per tile.)  A cell whose diagonal is selected
// is left out: phase 1 counted it.
struct ColWords { uint32_t lo, hi; };
__device__ __forceinline__ int col_offset(int posw, int col) { return posw - col < -96 ? -96 : posw - col; }   // row i meets the column on diagonal offset + i
__device__ __forceinline__ ColWords col_words(const uint32_t* ob, int posw, int col, bool diags) {
    ColWords w = {0u, 0u};
    if (diags && col >= 0) {
        const int q = (col_offset(posw, col) >> 5) + OB_PAD;
        w.lo = ob[q]; w.hi = ob[q + 1];
    }
    return w;
}
__device__ __forceinline__ TileMask col_mask(const ColWords& w, int posw, int col, int lane) {
    const int o = col_offset(posw, col);
    const uint32_t sel = (uint32_t)((((uint64_t)w.hi << 32) | w.lo) >> (o & 31));
    uint32_t rows = (o >= 0 ? 0xFFFFFFFFu : o > -32 ? 0xFFFFFFFFu << (-o & 31) : 0u) & ~sel;
    if (col < 0) rows = 0u;
    const uint32_t t = transpose32(rows, lane);
    const auto both = __builtin_amdgcn_permlane32_swap(t, t, false, false);   // every lane: its row's columns 0-31 and 32-63
    TileMask m;
    m.act[0] = __ballot(both[0] != 0u) != 0ull;
    m.act[1] = __ballot(both[1] != 0u) != 0ull;
    m.full[0] = m.full[1] = false;
    const int g4 = (lane >> 5) * 4;
    m.am[0] = both[0] >> g4; m.am[1] = both[1] >> g4;
    return m;
}
__device__ __forceinline__ float masked(float x, uint32_t am, int r) {      // x, or -inf if register r's key is not allowed
    const uint32_t keep = (uint32_t)__builtin_amdgcn_sbfe((int)am, 8 * (r >> 2) + (r & 3), 1);     // 0 or ~0
    return __builtin_bit_cast(float, (__builtin_bit_cast(uint32_t, x) & keep) | (0xFF800000u & ~keep));
}
__device__ __forceinline__ float max32(float x) {                           // the larger of this lane's and lane ^ 32's value
    const auto b = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, x), __builtin_bit_cast(uint32_t, x), false, false);
    return fmaxf(__builtin_bit_cast(float, (uint32_t)b[0]), __builtin_bit_cast(float, (uint32_t)b[1]));
}

__device__ __forceinline__ float sum32(float x) {                           // the sum of this lane's and lane ^ 32's value
    const auto b = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, x), __builtin_bit_cast(uint32_t, x), false, false);
    return __builtin_bit_cast(float, (uint32_t)b[0]) + __builtin_bit_cast(float, (uint32_t)b[1]);
}

// Tile sequence of one workgroup: first the n1 key blocks crossed by a selected diagonal (ascending),
// then n2 packed tiles of 64 selected columns each.  K/V rows of tile t+1 are fetched into registers
// while tile t is multiplied out of LDS buffer t&1, then written to buffer (t+1)&1; one barrier per tile.
template <typename T, int D, bool QUEUES>
__global__ __launch_bounds__(PREFILL_THREADS, 2) void prefill_kernel(PrefillArgs a) {
    using C = TileCfg<T, D>;
    extern __shared__ __align__(16) unsigned char smem[];
    unsigned char* k_lds = smem;                                         // [2][K_BYTES]
    unsigned char* vt_lds = smem + 2 * C::K_BYTES;                       // [2][VT_BYTES]
    int32_t* colring = reinterpret_cast<int32_t*>(smem + 2 * C::K_BYTES + 2 * C::VT_BYTES);   // [2][64]
    int32_t* wcnt = colring + 128;                                       // [8]
    uint16_t* kbl = reinterpret_cast<uint16_t*>(wcnt + 8);               // [tab_len] active key blocks

    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r32 = lane & 31, g = lane >> 5;

    Entries<QUEUES> entries;
    entries.init(a, lane);
    Entry en;
    while (entries.next(a, lane, wv, en)) {
    __syncthreads();                                       // everyone is done with the previous entry's LDS
    const int item = en.item, bh = item / a.nqb, qb = item % a.nqb;
    const int bkv = bh / a.Hq * a.Hkv + bh % a.Hq / a.G;
    const int nv = en.cols;                                // columns phase 2 gathers (those up to the block's last row)
    const int64_t n = a.n, row0 = n - a.n_hat;
    const int64_t blockpos = a.pos0 + (int64_t)qb * BM;                  // multiple of 128
    const int64_t posmax = (blockpos + BM - 1 < n - 1) ? blockpos + BM - 1 : n - 1;
    const T* Kg = reinterpret_cast<const T*>(a.k) + (int64_t)bkv * n * D;
    const T* Vg = reinterpret_cast<const T*>(a.v) + (int64_t)bkv * n * D;
    const T* Qg = reinterpret_cast<const T*>(a.q) + (int64_t)bh * a.n_hat * D;

    const uint8_t* tab = a.tab + (int64_t)bh * a.tab_len;
    const uint32_t* obg = a.obits + (int64_t)bh * (OB_PAD + a.words);    // zero words + bitmap of this head

    // this lane's query row and its fragments (a row that does not exist has zeros: its results are finite and unused)
    const int64_t pos = blockpos + 32 * wv + r32;
    const int posw = (int)blockpos + 32 * wv;              // the wave's first row
    const bool row_ok = (pos >= row0) && (pos < n);
    const bool rows_here = posw < n && posw + 31 >= row0;
    const int64_t jb = blockpos / BN;                      // even
    const int kb_hi = (int)(posmax / BN);
    const uint8_t tab0 = tab[jb - (tid <= kb_hi ? tid : kb_hi) + 1];     // (with the queries: the list below waits for it)
    Frag<T> qf[C::KSTEPS];
    if (row_ok) {
        const T* qrow = Qg + (pos - row0) * D;
#pragma unroll
        for (int c = 0; c < C::KSTEPS; ++c) load_frag(qf[c], qrow + 16 * c + 8 * g);
    } else {
#pragma unroll
        for (int c = 0; c < C::KSTEPS; ++c) zero_frag(qf[c]);
    }
    __syncthreads();

    // ---- ordered list of the key blocks phase 1 visits
    int n1 = 0;
    for (int base = 0; base <= kb_hi; base += PREFILL_THREADS) {
        const int kb = base + tid;
        const bool act = kb <= kb_hi && ((base == 0 ? tab0 : tab[jb - kb + 1]) & 1);
        const uint64_t bal = __ballot(act);
        if (lane == 0) wcnt[wv] = __popcll(bal);
        __syncthreads();
        int off = n1;
        for (int w2 = 0; w2 < wv; ++w2) off += wcnt[w2];
        if (act) kbl[off + __popcll(bal & ((1ull << lane) - 1ull))] = (uint16_t)kb;
        n1 += wcnt[0] + wcnt[1] + wcnt[2] + wcnt[3];
        __syncthreads();
    }
    const int32_t* vi = a.v_idx + (int64_t)bh * a.cap_v;
    const int n2 = (nv + BN - 1) / BN;
    const int tbeg = en.begin(n1 + n2), ntiles = en.end(n1 + n2);        // tiles tbeg .. ntiles - 1

    f32x16 oacc[C::DBLK];
#pragma unroll
    for (int i = 0; i < C::DBLK; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[i][r] = 0.f;
    float m_run = -INFINITY, l_run = 0.f;                  // m_run in raw logit units
    const float sc2 = a.scale_log2e;

    // ---- one staged tile
    auto process = [&](const unsigned char* kt, const unsigned char* vt, const TileMask& tm) {
        f32x16 s[2];
        if (!tm.act[0] && !tm.act[1]) return;
#pragma unroll
        for (int sub = 0; sub < 2; ++sub) {
#pragma unroll
            for (int r = 0; r < 16; ++r) s[sub][r] = 0.f;
            if (tm.act[sub]) {
                const unsigned char* krow = kt + (32 * sub + r32) * C::K_STRIDE + 8 * g * C::EB;
#pragma unroll
                for (int c = 0; c < C::KSTEPS; ++c) {
                    Frag<T> kf;
                    load_frag(kf, krow + 16 * c * C::EB);
                    mma(s[sub], kf, qf[c]);        // s[r] = <k_{8(r/4)+4g+r%4}, q_row>
                }
            }
        }
        float mx = -INFINITY;
#pragma unroll
        for (int sub = 0; sub < 2; ++sub) {
            if (!tm.full[sub]) {
#pragma unroll
                for (int r = 0; r < 16; ++r) s[sub][r] = masked(s[sub][r], tm.am[sub], r);
            }
#pragma unroll
            for (int r = 0; r < 16; ++r) mx = fmaxf(mx, s[sub][r]);
        }
        mx = fmaxf(mx, xor32(mx));
        const float m_new = fmaxf(m_run, mx);
        const float m_safe = (m_new == -INFINITY) ? 0.f : m_new;
        const float corr = fast_exp2((m_run - m_safe) * sc2);
        const float mneg = -m_safe * sc2;
        m_run = m_new;
        float psum = 0.f;
#pragma unroll
        for (int sub = 0; sub < 2; ++sub)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const float p = fast_exp2(__builtin_fmaf(s[sub][r], sc2, mneg));
                s[sub][r] = p;
                psum += p;
            }
        l_run = l_run * corr + psum;
        if (__ballot(corr != 1.0f) != 0ull) {
#pragma unroll
            for (int i = 0; i < C::DBLK; ++i)
#pragma unroll
                for (int r = 0; r < 16; ++r) oacc[i][r] *= corr;
        }
#pragma unroll
        for (int sub = 0; sub < 2; ++sub) {
            if (!tm.act[sub]) continue;
#pragma unroll
            for (int hh = 0; hh < 2; ++hh) {
                float pv[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) pv[e] = s[sub][8 * hh + e];
                Frag<T> pf;
                pack_frag(pf, pv);
#pragma unroll
                for (int i = 0; i < C::DBLK; ++i) {
                    Frag<T> vf;
                    load_frag(vf, vt + (32 * i + r32) * C::VT_STRIDE + (32 * sub + 16 * hh + 8 * g) * C::EB);
                    mma(oacc[i], vf, pf);          // O^T[d][row] += V^T[d][key] P^T[key][row]
                }
            }
        }
    };

    // ---- staging: thread -> (row tid/4, chunks tid%4 + 4i) for K, (row tid%64, chunks (tid/64)*CPT + i) for V
    const int rk = tid >> 2, ck0 = tid & 3;
    const int rv = tid & 63, cv0 = (tid >> 6) * C::CPT;
    const int vcol = vt_col(rv);
    f32x4 kreg[C::CPT], vreg[C::CPT];
    int32_t colk = -1, colv = -1;                          // gathered rows of the tile being fetched

    // global row feeding slot r of tile t (or -1): contiguous tiles read key block kbl[t]
    auto src_row = [&](int t, int r, int32_t gathered) -> int64_t {
        if (t < n1) { const int64_t kr = (int64_t)kbl[t] * BN + r; return kr < n ? kr : -1; }
        return gathered;
    };
    auto load_cols = [&](int t) {                          // column indices of gathered tile t -> registers
        colk = -1; colv = -1;
        if (t >= n1 && t < ntiles) {
            const int base = (t - n1) * BN;
            if (base + rk < nv) colk = vi[base + rk];
            if (base + rv < nv) colv = vi[base + rv];
        }
    };
    auto fetch = [&](int t) {                              // global -> registers, no divergent branches
        const int64_t gk = src_row(t, rk, colk), gv = src_row(t, rv, colv);
        const unsigned char* pk = reinterpret_cast<const unsigned char*>(Kg + (gk < 0 ? 0 : gk) * D) + 16 * ck0;
        const unsigned char* pv = reinterpret_cast<const unsigned char*>(Vg + (gv < 0 ? 0 : gv) * D) + 16 * cv0;
#pragma unroll
        for (int i = 0; i < C::CPT; ++i) {
            kreg[i] = *reinterpret_cast<const f32x4*>(pk + 64 * i);
            vreg[i] = *reinterpret_cast<const f32x4*>(pv + 16 * i);
        }
        if (__ballot(gk < 0 || gv < 0) != 0ull) {          // a slot without a row (tail of the context or of the list)
            const f32x4 z = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int i = 0; i < C::CPT; ++i) {
                if (gk < 0) kreg[i] = z;
                if (gv < 0) vreg[i] = z;
            }
        }
    };
    auto stash = [&](int t) {                              // registers -> LDS buffer t & 1 (+ column ids)
        unsigned char* kt = k_lds + (t & 1) * C::K_BYTES;
        unsigned char* vt = vt_lds + (t & 1) * C::VT_BYTES;
#pragma unroll
        for (int i = 0; i < C::CPT; ++i) {
            *reinterpret_cast<f32x4*>(kt + rk * C::K_STRIDE + 16 * (ck0 + 4 * i)) = kreg[i];
            store_vt(vt, C::VT_STRIDE, (cv0 + i) * C::EPC, vcol, vreg[i]);
        }
        if (t >= n1 && tid < BN) colring[(t & 1) * BN + tid] = colv;
    };

    if (tbeg < ntiles) {
        load_cols(tbeg);
        fetch(tbeg);
        stash(tbeg);
        load_cols(tbeg + 1);
    }
    __syncthreads();

    for (int t = tbeg; t < ntiles; ++t) {
        const bool more = t + 1 < ntiles;
        if (more) fetch(t + 1);                            // uses the columns loaded one iteration ago
        const int32_t colv_next = colv;
        if (more) load_cols(t + 2);
        // ---- masks of tile t
        TileMask tm;
        if (t < n1) {
            tm = diag_mask(diag_words((const_words)obg, posw, __builtin_amdgcn_readfirstlane((int)kbl[t]) * BN), r32, g);
        } else {
            const int col = colring[(t & 1) * BN + lane];
            tm = col_mask(col_words(obg, posw, col, n1 > 0), posw, col, lane);
        }
        if (!rows_here) tm.act[0] = tm.act[1] = false;
        process(k_lds + (t & 1) * C::K_BYTES, vt_lds + (t & 1) * C::VT_BYTES, tm);
        if (more) {
            const int32_t keep = colv; colv = colv_next;   // stash() records the columns of tile t+1
            stash(t + 1);
            colv = keep;
        }
        __syncthreads();
    }

    // ================= epilogue =================
    const float l_tot = l_run + xor32(l_run);
    const float inv = l_tot > 0.f ? 1.0f / l_tot : 0.f;
    entries.ahead(a, lane, wv);
    if (en.in_parts(n1 + n2)) {
        store_part<C::DBLK>(a, en.slot(), wv, lane, oacc, m_run * sc2, l_tot);
    } else if (row_ok) {
        T* orow = reinterpret_cast<T*>(a.out) + ((int64_t)bh * a.n_hat + (pos - row0)) * D;
#pragma unroll
        for (int i = 0; i < C::DBLK; ++i)
#pragma unroll
            for (int rq = 0; rq < 4; ++rq) {
                const int d0 = 32 * i + 8 * rq + 4 * g;
                store_out4(orow + d0, oacc[i][4 * rq] * inv, oacc[i][4 * rq + 1] * inv,
                           oacc[i][4 * rq + 2] * inv, oacc[i][4 * rq + 3] * inv);
            }
        if (a.lse && g == 0)
            a.lse[(int64_t)bh * a.n_hat + (pos - row0)] =
                l_tot > 0.f ? (m_run * sc2 + log2f(l_tot)) * 0.69314718055994531f : -INFINITY;
    }
    }                                                      // next entry
}

// ---------------------------------------------------------------------------------------------
// bf16 kernel: same tile sequence, masks and softmax as prefill_kernel, but staged the CDNA4 way.
//   * K and V rows go straight from global memory into LDS (global_load_lds, 16 bytes per lane, no
//     registers, no LDS store instructions).  A lane's 16 bytes land at LDS base + 16 * lane, so one
//     wave-wide transfer fills 1024 consecutive bytes: RPI whole rows of DS 16-byte slots.  Where a
//     lane's bytes land is fixed; which bytes it fetches is free, so slot s of row r receives chunk
//     s ^ swizzle(r) of that row.  The swizzles (kswz, vswz) are chosen so that the fragment reads
//     below touch every LDS bank once per pass; for d = 128 the K transfers are also spaced 64 bytes
//     apart.  All transfers of a wave then differ only in uniform addresses: one per-lane
//     offset register per operand serves the whole kernel.
//   * V stays row-major; the V^T fragments of the P*V product come from the LDS transpose read
//     ds_read_b64_tr_b16: in a block of 16 lanes, lane s addresses 4 consecutive 16-bit values and
//     lane L receives value L%4 of the lanes L/4, L/4+4, L/4+8, L/4+12.  With lane s pointing at key
//     (s/4) and at d-offset 4*(s%4), lane L ends up with four keys of column d = L: two reads give the
//     eight keys of a fragment.
// Rows that do not exist (tail of the context or of the column list) re-load an existing row; their
// keys are masked, so only finiteness of the staged values matters.
//
// Two ways through the tiles.  What bounds the kernel is instruction issue, and the card's power: of the cycles of a SIMD the products
// take half, and the clock falls as they take more.
//   Queues (long runs): half a tile, 32 keys, from barrier to barrier, and nothing of a half overlaps in its own wave: that takes 166 registers and
//   37 KB of LDS, so that three workgroups share a CU (four at d = 64) and one wave's softmax runs beside another's products.
//   Pieces (short runs): a whole tile from barrier to barrier, by halves, the softmax of one beside the products of the other: two workgroups
//   a CU (three at d = 64), but a wave that has the SIMD to itself, as where a workgroup has a handful of tiles, is faster: 61 rows of 12347
//   30.5 us a call against 32.0 by halves, d = 64, 1777 of 5003 rows, carried lines, 83.6 against 87.2.
// A tile of the 32768 keys' turn, three quarters diagonals, took a SIMD 2060 cycles with two halves and their transfers in one burst, 1830 with the
// transfers in between the products and fewer scalar instructions, 1600 by halves.  The whole call, us (as it was / tiles / halves): 10923 of 32768 rows 1700 / 1615 /
// 1580, all heads dense 4840 / 4750 / 4240, diagonals only 2055 / 1890 / 1850; 16384 of 131072 14670 / 13660 / 13600, B 4, 64 heads, 5462 of 16384 4120 / 3900 / 3660;
// 8192 rows, all new (pieces) 275 / 266.  (What the clock gives back: 2.24 GHz as it was, 2.0 by halves.  A workgroup of 2000 to 3000 of 20000 rows takes 13 % fewer
// cycles in pieces than it did, at a clock that is 7 % lower: 2.15 to 2.19 GHz instead of 2.30 to 2.35.)
// ---------------------------------------------------------------------------------------------
template <int D>
struct DirectCfg {
    static_assert(D == 128 || D == 64, "head dimension");
    static constexpr int RB = D * 2;                      // bytes per row
    static constexpr int DS = RB / 16;                    // 16-byte slots per row
    static constexpr int RPI = 64 / DS;                   // rows per transfer instruction
    static constexpr int HB = BN / 2;                     // keys of a half, which is what a buffer holds
    static constexpr int NI = HB / RPI;                   // transfer instructions per operand and half
    static constexpr int IPW = NI / 4;                    // ... per wave
    static constexpr int K_ISTR = D == 128 ? 1088 : 1024; // LDS bytes from one K transfer to the next
    static constexpr int V_ISTR = 1024;
    static constexpr int K_BYTES = NI * K_ISTR, V_BYTES = NI * V_ISTR, HALF_BYTES = K_BYTES + V_BYTES;
    static constexpr int FRONT = (128 + 512) * 4;         // LDS ahead of the buffers
    static constexpr int OUT_ROW = RB + 16;               // results on their way out: LDS bytes from row to row
    static constexpr int lds(bool queues) {
        const int halves = (queues ? 2 : 4) * HALF_BYTES;
        return FRONT + (halves > BM * OUT_ROW ? halves : BM * OUT_ROW);
    }
    static constexpr int KSTEPS = D / 16, DBLK = D / 32;
    static constexpr int KA = D == 128 ? 2 : 4;           // K fragment address registers
    // slot swizzles (XOR on the 16-byte slot index inside a row)
    __device__ static constexpr int kswz(int row) { return D == 128 ? (row & 3) : (((row >> 1) & 3) | (((row >> 3) & 1) << 2)); }
    __device__ static constexpr int vswz(int row) { return D == 128 ? ((row & 3) << 2) : (((row >> 1) & 1) << 2); }
};

template <int D, bool QUEUES>
__global__ __launch_bounds__(PREFILL_THREADS, (D == 64 ? 3 : 2) + (QUEUES ? 1 : 0)) void prefill_bf16_kernel(PrefillArgs a) {
    using C = DirectCfg<D>;
    using T = bf16_t;
    using std::integral_constant;
    extern __shared__ __align__(16) unsigned char smem[];
    int32_t* colring = reinterpret_cast<int32_t*>(smem);                 // [2][64] column ids of packed tiles
    uint32_t* colbits = reinterpret_cast<uint32_t*>(colring + 128);      // [4 waves][2][64] bitmap words for the masks of a packed tile
    unsigned char* tiles = smem + C::FRONT;                              // [2 halves, or two tiles of 2][HALF_BYTES]: K rows, V rows
    const uint32_t tiles_lds = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)tiles;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t colring_lds = tiles_lds - (uint32_t)C::FRONT, colbits_lds = colring_lds + 512u + (uint32_t)wv * 512u;
    const int r32 = lane & 31, g = lane >> 5;
    auto uniform = [](int x) { return __builtin_amdgcn_readfirstlane(x); };
    // a value made anew: addresses and masks computed from it are needed now and then, and would otherwise be kept in registers (20 of them)
    auto again = [](int x) { asm volatile("" : "+v"(x)); return x; };
    auto apart = [](int x) { asm volatile("" : "+v"(x)); return __builtin_amdgcn_readfirstlane(x); };      // a condition that is not joined with others

    // ---- per-lane constants of the transfers: this lane fills slot sl of row rowlane (+ RPI for the wave's second instruction)
    // of a half and fetches the chunk the swizzle assigns to that slot
    const int rowlane = C::IPW * C::RPI * wv + lane / C::DS;
    const int sl = lane % C::DS;
    const uint32_t kcpart = 16u * (uint32_t)(sl ^ C::kswz(rowlane)), vcpart = 16u * (uint32_t)(sl ^ C::vswz(rowlane));
    static_assert(C::IPW == 1 || (C::kswz(C::RPI) == 0 && C::vswz(C::RPI) == 0), "a wave's instructions share their swizzles");
    // ---- K fragment reads: row r32, chunk 2c+g sits in slot (2c+g) ^ kswz
    int kaddr[C::KA];
    {
        const int x = C::kswz(r32);
        const int krow = (r32 / C::RPI) * C::K_ISTR + (r32 % C::RPI) * C::RB;
#pragma unroll
        for (int j = 0; j < C::KA; ++j) kaddr[j] = krow + 32 * (j ^ (x >> 1)) + 16 * (g ^ (x & 1));
    }
    // ---- V^T fragment reads (see the header comment): key 4g + L16/4 (+8, +16 q4), 64-byte block i
    int vaddr[C::DBLK];
    {
        const int L16 = lane & 15, beta = (lane >> 4) & 1;
        const int lrow = 4 * g + (L16 >> 2);
        const int y = C::vswz(lrow) >> 2;
#pragma unroll
        for (int i = 0; i < C::DBLK; ++i) vaddr[i] = C::K_BYTES + lrow * C::RB + 64 * (i ^ y) + 32 * beta + 8 * (L16 & 3);
    }

    Entries<QUEUES> entries;
    entries.init(a, lane);
    Entry en;
    while (entries.next(a, lane, wv, en)) {
    const int item = uniform(en.item), bh = item / a.nqb, qb = item % a.nqb;
    const int n1 = en.blocks, nv = en.cols;                // key blocks phase 1 visits, columns phase 2 gathers (those up to the block's last row)
    const int bkv = bh / a.Hq * a.Hkv + bh % a.Hq / a.G;
    const int n2 = (nv + BN - 1) / BN;
    const int tbeg = uniform(en.begin(n1 + n2)), ntiles = uniform(en.end(n1 + n2));      // tiles tbeg .. ntiles - 1
    const int64_t n = a.n, row0 = n - a.n_hat;
    const int64_t blockpos = a.pos0 + (int64_t)qb * BM;                  // multiple of 128
    const unsigned char* Kg = reinterpret_cast<const unsigned char*>(a.k) + (int64_t)bkv * n * C::RB;
    const unsigned char* Vg = reinterpret_cast<const unsigned char*>(a.v) + (int64_t)bkv * n * C::RB;
    const T* Qg = reinterpret_cast<const T*>(a.q) + (int64_t)bh * a.n_hat * D;

    const uint32_t* obg = a.obits + (int64_t)bh * (OB_PAD + a.words);     // zero words + bitmap of this head
    const int posw = (int)blockpos + 32 * wv;              // the wave's first row
    const bool rows_here = posw < n && posw + 31 >= row0;
    // ---- key blocks of the contiguous tiles, ascending: a run of the head's list of active table entries, backwards; entry e is key block
    // jb + 1 - e.  Lane l keeps that of tile tile0 + l.  The first are asked for ahead of the queries.
    const int jb = (int)(blockpos / BN);
    const uint16_t* el = a.elist + (int64_t)bh * (a.tab_len + 1) + n1 - 1;         // of tile 0, the others below it
    if (n - 1 < blockpos + BN && n1 > 0 && uniform((int)a.elist[(int64_t)bh * (a.tab_len + 1)]) == 0) ++el;      // half a row block: entry 0 belongs to key blocks beyond it
    const int blocks = ntiles < n1 ? ntiles : n1;                        // contiguous tiles of this part end here
    int kbv = 0, tile0 = tbeg;
    auto ask_blocks = [&]() { const int i = tile0 + lane < blocks ? tile0 + lane : blocks - 1; kbv = jb + 1 - (int)el[-i]; };
    auto keep_blocks = [&](int t) {                        // tile t among them
        if (t - tile0 < 64) return;
        tile0 = t;
        ask_blocks();
        wait_transfers();
    };
    auto block_at = [&](int t) -> int { return __builtin_amdgcn_readlane(kbv, t - tile0); };
    if (tbeg < blocks) ask_blocks();
    asm volatile("" ::: "memory");
    Frag<T> qf[C::KSTEPS];
    {
        const int64_t pos = posw + again(r32);
        if (pos >= row0 && pos < n) {                      // a row that does not exist has zeros: finite results, not stored
            const T* qrow = Qg + (pos - row0) * D;
#pragma unroll
            for (int c = 0; c < C::KSTEPS; ++c) load_frag(qf[c], qrow + 16 * c + 8 * g);
        } else {
#pragma unroll
            for (int c = 0; c < C::KSTEPS; ++c) zero_frag(qf[c]);
        }
    }
    const int32_t* vi = a.v_idx + (int64_t)bh * a.cap_v;

    f32x16 oacc[C::DBLK];
#pragma unroll
    for (int i = 0; i < C::DBLK; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[i][r] = 0.f;
    // mneg: the softmax reference of this lane's row in base 2, negated (+inf: no cell seen yet).  It moves only when a probability
    // might exceed the limit, so that most tiles need no rescaling of the accumulators.
    const float sc2 = a.scale_log2e;
    float mneg = INFINITY, l_run = 0.f, limit = SOFT_FIRST;
    int often = 0, doubled = -1;                           // how often halves exceed the limit; the tile for which the limit was doubled last (uniform)

    // ---- staging.  Of a half's K and V wave wv fetches rows 8 wv .. 8 wv + 7, IPW instructions of RPI rows each.  A row beyond the context
    // re-loads the last row, a missing column the last column: every slot is always written with finite data and needs no exec masking.
    const uint32_t kdst0 = tiles_lds + (uint32_t)(wv * C::IPW * C::K_ISTR), vdst0 = tiles_lds + (uint32_t)(C::K_BYTES + wv * C::IPW * C::V_ISTR);
    auto buffer = [](int s) -> uint32_t { return (uint32_t)(s & (QUEUES ? 1 : 3)) * (uint32_t)C::HALF_BYTES; };       // of half s, counted through the tiles
    auto issue_half = [&](int kh, int s) {                 // keys 32 kh ..
        const int64_t left = n - (int64_t)kh * C::HB;      // none left: the last key throughout
        const int64_t key0 = left > 0 ? (int64_t)kh * C::HB : n - 1;
        const int last = left > C::HB ? C::HB - 1 : left > 0 ? (int)left - 1 : 0, r0 = again(rowlane);
#pragma unroll
        for (int i = 0; i < C::IPW; ++i) {
            const int row = r0 + C::RPI * i;
            const uint32_t at = (uint32_t)(row <= last ? row : last) * C::RB;
            dma16(Kg + key0 * C::RB, at + kcpart, kdst0 + buffer(s) + (uint32_t)(i * C::K_ISTR));
            dma16(Vg + key0 * C::RB, at + vcpart, vdst0 + buffer(s) + (uint32_t)(i * C::V_ISTR));
        }
    };
    auto issue_cols = [&](int s) {                         // the columns of half s & 1 of packed tile s / 2
        const int32_t* cols = colring + (s >> 1 & 1) * BN + (s & 1) * C::HB + again(rowlane);
#pragma unroll
        for (int i = 0; i < C::IPW; ++i) {
            const uint32_t at = (uint32_t)cols[C::RPI * i] * C::RB;
            dma16(Kg, at + kcpart, kdst0 + buffer(s) + (uint32_t)(i * C::K_ISTR));
            dma16(Vg, at + vcpart, vdst0 + buffer(s) + (uint32_t)(i * C::V_ISTR));
        }
    };

    // ---- masks.  halves: of the tile at hand, 1, 2 = the half has an allowed cell (for this wave), 4, 8 = all of it is allowed; am: which.
    // (Queues, contiguous tiles: of the half at hand, in the first place.)
    // The bitmap words of contiguous tiles come out of a register: lane l keeps word wq - l, good for some 60 neighbouring
    // halves, and a half's words are lane reads.  (Scalar loads ahead of the tile's transfers, waited for there, were 200 cycles a tile.)
    const int rows_mask = rows_here ? 15 : 0, pw = posw / 32;
    uint32_t am[2] = {0u, 0u};
    int halves = 0, kh_next = 0;                           // kh_next: the keys (in 32s) of the half (pieces: the tile) after the one at hand (phase 1)
    uint32_t wc = 0u;
    int wq = -1000000;
    auto keep_words = [&](int kh) {
        const int q = pw - kh;                             // >= -3
        if ((uint32_t)(wq - q) > (QUEUES ? 62u : 61u)) {
            const int at = q - lane + OB_PAD;              // (below the bitmap: zero words)
            wc = obg[at < 0 ? 0 : at];
            wq = q;
            wait_transfers();
        }
    };
    uint32_t x0 = 0u, x1 = 0u, x2 = 0u;
    auto mask_step = [&](int k) {                          // masks of the contiguous half or tile kh_next, in four steps
        if (k == 0) {
            const int l = wq - pw + kh_next;
            x2 = (uint32_t)__builtin_amdgcn_readlane((int)wc, l);
            x1 = (uint32_t)__builtin_amdgcn_readlane((int)wc, l + 1);
            if (!QUEUES) x0 = (uint32_t)__builtin_amdgcn_readlane((int)wc, l + 2);
        } else if (k == 1) am[0] = diag_cells(x2, x1, r32, g);
        else if (k == 2) { if (!QUEUES) am[1] = diag_cells(x1, x0, r32, g); }
        else halves = (diag_half(x2, x1) | (QUEUES ? 0 : diag_half(x1, x0) << 1)) & rows_mask;
    };

    // ---- products and softmax.  Order is pinned (a scheduling barrier after each product), the LDS fragment reads run a fixed number
    // of products ahead.
    // No maximum is looked for on the way: the exponentials are taken with the reference as it stands, and where a lane's
    // sum says that one of them may exceed the limit (or is no number, as with the first cells of a row: -mneg = -inf), the half is
    // done again with a new reference.  s keeps the logits for that.
    constexpr int NS = C::KSTEPS, NV = 2 * C::DBLK;        // products of a half
    constexpr int RS = RING_S, RV = QUEUES ? RING_P_QUEUES : RING_P;
    static_assert(RS <= NS && RV <= NV, "fragments in flight");
    const f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    struct Soft { uint32_t p[8]; float sum[2]; };          // packed probabilities and their sums
    auto kload = [&](Frag<T>& f, const unsigned char* base, int c) { load_frag(f, base + kaddr[c & (C::KA - 1)] + 32 * (c & ~(C::KA - 1))); };
    auto vload = [&](Frag<T>& f, const unsigned char* base, int k) {         // keys 16 (k / DBLK).., output block k % DBLK
        const unsigned char* va = base + vaddr[k % C::DBLK] + 16 * (k / C::DBLK) * C::RB;
        load_frag_tr(f, va, va + 8 * C::RB);
    };
    auto pack2 = [&](float lo, float hi) {
        typedef __attribute__((ext_vector_type(2))) float f32x2;
        typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
        uint32_t u = __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{lo, hi}), bf16x2));   // v_cvt_pk_bf16_f32, round to nearest even
        asm volatile("" : "+v"(u));                        // here, and not where it is used
        return u;
    };
    auto pfrag = [&](const Soft& o, int h) {
        struct U { uint32_t w[4]; } u = {o.p[4 * h], o.p[4 * h + 1], o.p[4 * h + 2], o.p[4 * h + 3]};
        Frag<T> f;
        f.v = __builtin_bit_cast(bf16x8, u);
        return f;
    };
    // registers r .. r + E - 1 of a half, in step k of 16 / E; x: their exponents, one step ahead
    auto exponents = [&](auto MASKED, auto EC, float (&x)[4], f32x16& s, uint32_t cells, int k) {
        constexpr int E = decltype(EC)::value;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int r = E * k + e;
            if constexpr (decltype(MASKED)::value) s[r] = masked(s[r], cells, r);
            x[e] = __builtin_fmaf(s[r], sc2, mneg);
        }
    };
    auto soft_step = [&](auto MASKED, auto EC, float (&x)[4], f32x16& s, uint32_t cells, Soft& o, int k) {
        constexpr int E = decltype(EC)::value;
        float p[E];
#pragma unroll
        for (int e = 0; e < E; ++e) p[e] = fast_exp2(x[e]);
        if (k + 1 < 16 / E) exponents(MASKED, EC, x, s, cells, k + 1);
#pragma unroll
        for (int e = 0; e < E; ++e) { if (E * k + e < 2) o.sum[e] = p[e]; else o.sum[e & 1] += p[e]; }
#pragma unroll
        for (int e = 0; e < E; e += 2) o.p[(E * k + e) / 2] = pack2(p[e], p[e + 1]);
    };
    auto soft_alone = [&](auto MASKED, auto EC, f32x16& s, uint32_t cells, Soft& o) {
        float x[4];
        exponents(MASKED, EC, x, s, cells, 0);
#pragma unroll
        for (int k = 0; k < 16 / decltype(EC)::value; ++k) soft_step(MASKED, EC, x, s, cells, o, k);
    };
    auto settle = [&](int t, f32x16& s, Soft& o) {         // the sums in, or the half once more with a new reference
        float sum = o.sum[0] + o.sum[1];
        if (__ballot(!(sum <= limit)) != 0ull) {
            float mx = -INFINITY;
#pragma unroll
            for (int r = 0; r < 16; ++r) mx = fmaxf(mx, s[r]);
            mx = max32(mx) * sc2;
            float m_new = fmaxf(mx, -mneg);                // in base 2
            often = (often > t ? often : t) + 4;
            if (often - t > SOFT_OFTEN) {
                asm volatile("");                          // (rare: a branch, no selects)
                often = SOFT_RISING;
                if (limit < 0.f) {                         // back to the maxima, once
                    if (limit == -2.f) m_new = fmaxf(mx, -mneg - SOFT_AHEAD);
                    limit = t < n1 ? -4.f : SOFT_LIMIT;
                } else if (t + 2 < n1) {
                    m_new = mx > -mneg ? mx + SOFT_AHEAD : -mneg;
                }
            }
            const float corr = m_new > -INFINITY ? fast_exp2(-mneg - m_new) : 1.f;
            mneg = -m_new;
            const float safe = m_new > -INFINITY ? mneg : 0.f;
            l_run *= corr;
#pragma unroll
            for (int i = 0; i < C::DBLK; ++i)
#pragma unroll
                for (int r = 0; r < 16; ++r) oacc[i][r] *= corr;
            sum = 0.f;
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int r = 0; r < 16; r += 4) {
                float p[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) { p[e] = fast_exp2(__builtin_fmaf(s[r + e], sc2, safe)); sum += p[e]; }
                o.p[r / 2] = pack2(p[0], p[1]);
                o.p[r / 2 + 1] = pack2(p[2], p[3]);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        l_run += sum;
    };
    // S of a half, beside it PER-th of SN transfers (none: 0)
    auto scores = [&](auto SENDS, f32x16& x, const unsigned char* base, auto send) {
        constexpr int SN = decltype(SENDS)::value;
        static_assert(SN <= NS, "at most a transfer beside a product");
        Frag<T> kf[NS];
#pragma unroll
        for (int c = 0; c < RS; ++c) kload(kf[c], base, c);
        __builtin_amdgcn_sched_barrier(0);
        x = zero16;
#pragma unroll
        for (int c = 0; c < NS; ++c) {
            mma(x, kf[c], qf[c]);                          // x[r] = <k_{8(r/4)+4g+r%4}, q_row>
            if (c + RS < NS) kload(kf[c + RS], base, c + RS);
            if constexpr (SN > 0) if (c % (NS / SN) == NS / SN / 2) send(c / (NS / SN));
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    // O += P V of a half, beside it the masks of what comes next
    auto values = [&](Frag<T> (&vf)[NV], const Soft& p, const unsigned char* base) {
#pragma unroll
        for (int k = 0; k < NV; ++k) {
            mma(oacc[k % C::DBLK], vf[k], pfrag(p, k / C::DBLK));
            if (k + RV < NV) vload(vf[k + RV], base, k + RV);
            if (k < 4) mask_step(k);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    // Queues: one half after the other; the other waves of the SIMD (three, four at d = 64) keep the matrix pipe busy beside a wave's softmax.
    auto process_half = [&](auto SENDS, int t, const unsigned char* base, auto send) {
        f32x16 x;
        Soft o;
        if (t != doubled) { doubled = t; limit = fminf(limit * 2.f, SOFT_LIMIT); }
        scores(SENDS, x, base, send);
        Frag<T> vf[NV];
#pragma unroll
        for (int k = 0; k < RV; ++k) vload(vf[k], base, k);                  // ahead of the softmax
        auto soft = [&](auto MASKED) {
#pragma unroll
            for (int r = 0; r < 16; r += 2) {
                if constexpr (decltype(MASKED)::value) { x[r] = masked(x[r], am[0], r); x[r + 1] = masked(x[r + 1], am[0], r + 1); }
                const float e0 = fast_exp2(__builtin_fmaf(x[r], sc2, mneg)), e1 = fast_exp2(__builtin_fmaf(x[r + 1], sc2, mneg));
                o.sum[0] = r ? o.sum[0] + e0 : e0;
                o.sum[1] = r ? o.sum[1] + e1 : e1;
                o.p[r / 2] = pack2(e0, e1);
            }
        };
        if (halves & 4) soft(std::false_type{}); else soft(std::true_type{});
        settle(t, x, o);
        __builtin_amdgcn_sched_barrier(0);
        values(vf, o, base);
    };
    // Pieces: a tile by halves; halves without an allowed cell are passed by.  With two halves the vector work of one runs beside the
    // products of the other: S(1) beside the softmax of 0, P V of 0 beside the softmax of 1.  A product is followed by its share of the
    // other half's 16 registers (a product takes its wave 33 cycles, a masked register 27, an unmasked one 18).
    auto process_tile = [&](auto SENDS, int t, auto send) {
        constexpr int ES = 16 / NS, EV = 16 / NV;          // registers of the other half's softmax per product
        constexpr int SN = decltype(SENDS)::value / 2;     // transfers beside the products of a half's S
        f32x16 sa, sb;
        Soft pa, pb;
        limit = fminf(limit * 2.f, SOFT_LIMIT);
        // (The accumulators change in straight code and under conditions without an else only: where both sides of a choice
        // changed them, the compiler, which gives every choice the form of two guarded parts, kept them twice and moved them.)
        const unsigned char *t0 = tiles + buffer(2 * t), *t1 = t0 + C::HALF_BYTES;
        const int two = (halves & 3) == 3, h0 = (halves & 3) == 2;
        const uint32_t am0 = h0 ? am[1] : am[0];
        scores(integral_constant<int, SN>{}, sa, h0 ? t1 : t0, send);
        if (two) {
            auto first = [&](auto MASKED) {                // S of the second half beside the softmax of the first
                Frag<T> kf[NS];
                float x[4];
#pragma unroll
                for (int c = 0; c < RS; ++c) kload(kf[c], t1, c);
                __builtin_amdgcn_sched_barrier(0);
                sb = zero16;
#pragma unroll
                for (int c = 0; c < NS; ++c) {
                    mma(sb, kf[c], qf[c]);
                    if (c + RS < NS) kload(kf[c + RS], t1, c + RS);
                    if constexpr (SN > 0) if (c % (NS / SN) == NS / SN / 2) send(SN + c / (NS / SN));
                    if (c == 0) exponents(MASKED, integral_constant<int, ES>{}, x, sa, am0, 0);
                    else soft_step(MASKED, integral_constant<int, ES>{}, x, sa, am0, pa, c - 1);
                    __builtin_amdgcn_sched_barrier(0);
                }
                soft_step(MASKED, integral_constant<int, ES>{}, x, sa, am0, pa, NS - 1);
            };
            if (halves & 4) first(std::false_type{}); else first(std::true_type{});
        } else {
#pragma unroll
            for (int i = 0; i < SN; ++i) send(SN + i);
            soft_alone(std::true_type{}, integral_constant<int, 4>{}, sa, am0, pa);
        }
        settle(t, sa, pa);
        pb = pa;
        if (apart(two)) {
            Frag<T> vf[NV];                                // P V of the first half beside the softmax of the second
            float x[4];
#pragma unroll
            for (int k = 0; k < RV; ++k) vload(vf[k], t0, k);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int k = 0; k < NV; ++k) {
                mma(oacc[k % C::DBLK], vf[k], pfrag(pa, k / C::DBLK));
                if (k + RV < NV) vload(vf[k + RV], t0, k + RV);
                if (k == 0) exponents(std::true_type{}, integral_constant<int, EV>{}, x, sb, am[1], 0);
                else soft_step(std::true_type{}, integral_constant<int, EV>{}, x, sb, am[1], pb, k - 1);
                __builtin_amdgcn_sched_barrier(0);
            }
            soft_step(std::true_type{}, integral_constant<int, EV>{}, x, sb, am[1], pb, NV - 1);
            settle(t, sb, pb);
        }
        const unsigned char* tv = (halves & 2) ? t1 : t0;
        Frag<T> vf[NV];
#pragma unroll
        for (int k = 0; k < RV; ++k) vload(vf[k], tv, k);
        __builtin_amdgcn_sched_barrier(0);
        values(vf, pb, tv);
    };

    // What a packed tile needs besides its rows goes through LDS by transfers of its own: the ids of its columns ahead of them
    // (slots past the end of the list repeat the last column), the bitmap words of its masks beside them.
    // (As loads into registers they made the compiler put waits for all outstanding memory operations, the transfers of
    // the next tile among them, into the tile loop.)
    auto request_cols = [&](int t) {                       // column ids of packed tile t -> slot t & 1
        if (wv == 0) {
            int i = (t - n1) * BN + lane;
            if (i > nv - 1) i = nv - 1;
            dma4(vi, (uint32_t)i * 4u, colring_lds + (uint32_t)((t & 1) * BN * 4));
        }
    };
    int32_t mycol = -1;
    auto col_words_of = [&](int t) {                       // what the masks of packed tile t are made of, ahead of its transfers
        const int l = again(lane);
        const int32_t col = colring[(t & 1) * BN + l];
        mycol = (t - n1) * BN + l < nv ? col : -1;
        if (n1 > 0) {
            const uint32_t off = (uint32_t)((col_offset(posw, mycol < 0 ? 0 : mycol) >> 5) + OB_PAD) * 4u;
            dma4(obg, off, colbits_lds);
            dma4(obg, off + 4u, colbits_lds + 256u);
        }
    };
    auto masks_cols = [&]() {                              // once the transfers have landed
        ColWords cw = {0u, 0u};
        const int l = again(lane);
        if (n1 > 0) { cw.lo = colbits[wv * 128 + l]; cw.hi = colbits[wv * 128 + 64 + l]; }
        const TileMask tm = col_mask(cw, posw, mycol, l);
        am[0] = tm.am[0]; am[1] = tm.am[1];
        halves = uniform(((tm.act[0] ? 1 : 0) | (tm.act[1] ? 2 : 0)) & rows_mask);
    };

    // transfers of two halves inside the context, one at a time
    const unsigned char *ka = Kg, *va = Vg;
    uint32_t to = 0u;                                      // K and V rows of up to two halves from ka, va on -> buffers from `to` on
    auto send = [&](int i) {
        const int h = i / (2 * C::IPW), j = i % (2 * C::IPW) / 2, rows = h * C::HB + j * C::RPI;
        if (i & 1) dma16(va + rows * C::RB, (uint32_t)rowlane * C::RB + vcpart, vdst0 + to + (uint32_t)(h * C::HALF_BYTES + j * C::V_ISTR));
        else dma16(ka + rows * C::RB, (uint32_t)rowlane * C::RB + kcpart, kdst0 + to + (uint32_t)(h * C::HALF_BYTES + j * C::K_ISTR));
    };
    auto aim = [&](int kh, uint32_t buf) {
        const uint64_t at = (uint64_t)(uint32_t)kh * (uint32_t)(C::HB * C::RB);
        ka = Kg + at; va = Vg + at; to = buf;
    };
    // The part's halves are 2 tbeg .. end - 1 (the second half of the last packed tile may have no columns).  Queues: the next half is
    // fetched beside every half, the columns of a packed tile are requested a tile ahead; pieces: the next tile beside every tile, two ahead.
    const int end = 2 * ntiles - (ntiles > n1 && (ntiles - n1) * BN - nv >= C::HB ? 1 : 0);
    auto fetch = [&](int s) {                              // half s
        if (s >= end) return;
        if ((s >> 1) >= blocks) { issue_cols(s); return; }
        const int kh = 2 * block_at(s >> 1) + (s & 1);
        if ((int64_t)(kh + 1) * C::HB > n) { issue_half(kh, s); return; }
        aim(kh, buffer(s));
#pragma unroll
        for (int i = 0; i < 2 * C::IPW; ++i) send(i);
    };
    if (tbeg < ntiles && tbeg + (QUEUES ? 0 : 1) >= n1) {  // a packed tile among the first ones
        if (tbeg >= n1) request_cols(tbeg);
        if (!QUEUES && tbeg + 1 < ntiles) request_cols(tbeg + 1);
        wait_transfers();
    }
    __syncthreads();                                       // the first column ids are visible, and the buffers are free
    if (tbeg < blocks) {
        kh_next = 2 * block_at(tbeg);
        keep_words(kh_next);
    } else if (tbeg < ntiles) {
        col_words_of(tbeg);
    }
    fetch(2 * tbeg);
    if (!QUEUES) fetch(2 * tbeg + 1);
    if (tbeg < blocks) for (int k = 0; k < 4; ++k) mask_step(k);
    wait_transfers();                                      // (on every path: the compiler has loads of its own under way)
    if (tbeg >= blocks && tbeg < ntiles) masks_cols();
    __syncthreads();

    // As long as the next tile is a contiguous one ahead of the item's last, its halves lie inside the context, and there is little else to see to:
    // 20 scalar instructions a tile instead of 90, its transfers in between the products of S (one after the other ahead of them they kept
    // the wave for 600 of its 4000 cycles a tile).
    const int plain = ntiles < n1 ? ntiles - 1 : n1 - 2;
    int t = tbeg;
    for (; t < plain; ++t) {
        if constexpr (QUEUES) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                if (h == 0) ++kh_next;
                else { keep_blocks(t + 1); kh_next = 2 * block_at(t + 1); }
                keep_words(kh_next);
                aim(kh_next, buffer(h + 1));
                const int active = halves & 1;
                if (active) process_half(integral_constant<int, 2 * C::IPW>{}, t, tiles + buffer(h), send);
                if (apart(active) == 0) {
#pragma unroll
                    for (int i = 0; i < 2 * C::IPW; ++i) send(i);
                    for (int k = 0; k < 4; ++k) mask_step(k);
                }
                wait_transfers();                          // this wave's transfers have landed
                __syncthreads();
            }
        } else {
            keep_blocks(t + 1);
            kh_next = 2 * block_at(t + 1);
            keep_words(kh_next);
            aim(kh_next, buffer(2 * t + 2));
            const int active = halves & 3;
            if (active) process_tile(integral_constant<int, 4 * C::IPW>{}, t, send);
            if (apart(active) == 0) {
#pragma unroll
                for (int i = 0; i < 4 * C::IPW; ++i) send(i);
                for (int k = 0; k < 4; ++k) mask_step(k);
            }
            wait_transfers();
            __syncthreads();
        }
    }
    auto none = [](int) {};
    if constexpr (QUEUES) {
        for (int s = 2 * t; s < end; ++s) {
            const int odd = s & 1;
            t = s >> 1;
            const bool next = s + 1 < end, packed = next && t + odd >= n1;         // of the next half
            if (odd && t + 1 < blocks) keep_blocks(t + 1);
            if (next && !packed) {
                kh_next = odd ? 2 * block_at(t + 1) : kh_next + 1;
                keep_words(kh_next);
            }
            if (!odd) {
                if (t + 1 >= n1 && t + 1 < ntiles) request_cols(t + 1);
                if (t + 2 == n1 && often == SOFT_RISING) limit = -1.f;       // (no sum is less: every half from here on)
            } else if (packed) {
                col_words_of(t + 1);
            }
            fetch(s + 1);
            const int active = halves & 1, second = halves >> 1;
            const uint32_t am1 = am[1];
            if (active) process_half(integral_constant<int, 0>{}, t, tiles + buffer(s), none);
            if (apart(active) == 0) for (int k = 0; k < 4; ++k) mask_step(k);
            wait_transfers();
            if (packed) {
                if (odd) masks_cols();
                else { am[0] = am1; halves = second; }
            }
            __syncthreads();
        }
    } else {
        for (; t < ntiles; ++t) {
            const bool next = t + 1 < ntiles, packed = next && t + 1 >= n1;        // of the next tile
            if (next && !packed) {
                keep_blocks(t + 1);
                kh_next = 2 * block_at(t + 1);
                keep_words(kh_next);
            }
            if (t + 2 >= n1 && t + 2 < ntiles) request_cols(t + 2);
            if (t + 2 == n1 && often == SOFT_RISING) limit = -1.f;
            if (packed) col_words_of(t + 1);
            fetch(2 * t + 2);
            fetch(2 * t + 3);
            const int active = halves & 3;
            if (active) process_tile(integral_constant<int, 0>{}, t, none);
            if (apart(active) == 0) for (int k = 0; k < 4; ++k) mask_step(k);
            wait_transfers();
            if (packed) masks_cols();
            __syncthreads();
        }
    }

    float l_tot = sum32(l_run), m_tot = -mneg;
    entries.ahead(a, lane, wv);                            // the next entry's place in the queue, under the stores below
    const int ln = again(lane), rl = ln & 31, gl = ln >> 5;
    bool whole = !en.in_parts(n1 + n2);
    if (!whole) {
        if (!QUEUES && __builtin_expect(a.arrived != nullptr, 0)) whole = join_parts<C::DBLK, (D == 64 ? 2 : 1)>(a, en, entries.span(), n1 + n2, ntiles - tbeg, wv, ln, rows_here, oacc, m_tot, l_tot);
        else store_part<C::DBLK>(a, en.slot(), wv, ln, oacc, m_tot, l_tot);
    }
    const float inv = l_tot > 0.f ? 1.0f / l_tot : 0.f;
    if (whole && rows_here) {
        // A lane holds four neighbouring values of its row at a time; through LDS (32 rows of this wave in the tile
        // buffers, which nobody reads any more) they become whole rows, 1 KB a store.  (Stored as they are, 8 bytes a
        // lane in 32 rows, they kept a wave for 4.5-7 thousand cycles an entry.)
        constexpr int OS = C::OUT_ROW;
        unsigned char* ow = tiles + wv * (32 * OS);
#pragma unroll
        for (int i = 0; i < C::DBLK; ++i)
#pragma unroll
            for (int rq = 0; rq < 4; ++rq)
                store_out4(reinterpret_cast<T*>(ow + rl * OS) + 32 * i + 8 * rq + 4 * gl, oacc[i][4 * rq] * inv, oacc[i][4 * rq + 1] * inv,
                           oacc[i][4 * rq + 2] * inv, oacc[i][4 * rq + 3] * inv);
        __builtin_amdgcn_wave_barrier();
        unsigned char* og = reinterpret_cast<unsigned char*>(a.out) + ((int64_t)bh * a.n_hat + (posw - row0)) * C::RB;   // row posw may lie before the turn
        const int cr = ln / C::DS, cs = ln % C::DS;
#pragma unroll
        for (int j = 0; j < 32 / C::RPI; ++j) {
            const int r = C::RPI * j + cr;
            const f32x4 v = *reinterpret_cast<const f32x4*>(ow + r * OS + 16 * cs);
            if (posw + r >= row0 && posw + r < n) *reinterpret_cast<f32x4*>(og + (int64_t)r * C::RB + 16 * cs) = v;
        }
        if (a.lse && gl == 0 && posw + rl >= row0 && posw + rl < n)
            a.lse[(int64_t)bh * a.n_hat + (posw + rl - row0)] =
                l_tot > 0.f ? (log2f(l_tot) + m_tot) * 0.69314718055994531f : -INFINITY;
    }
    }                                                      // next entry
}

template <typename T, int D, bool QUEUES>
static void launch_combine(const PrefillArgs& a, hipStream_t st, const hipEvent_t* ev) {
    if (a.slots == 0) return;
    const dim3 grid(QUEUES ? (a.slots < 256 ? 2 * a.slots : 512) : 4 * a.grid);
    if (ev) hipExtLaunchKernelGGL((combine_kernel<T, D, QUEUES>), grid, dim3(256), 0, st, ev[2], ev[3], 0, a);
    else hipLaunchKernelGGL((combine_kernel<T, D, QUEUES>), grid, dim3(256), 0, st, a);
}

template <typename T, int D>
static size_t prefill_smem_t(int tab_len) {
    using C = TileCfg<T, D>;
    return 2 * (size_t)C::K_BYTES + 2 * (size_t)C::VT_BYTES + 128 * 4 + 8 * 4 + (size_t)((tab_len + 7) & ~7) * 2 + 16;
}

template <typename T, int D, bool QUEUES>
static hipError_t launch_prefill_t(const PrefillArgs& a, hipStream_t st, const hipEvent_t* ev) {
    // with events: they take the start and stop time stamps of this dispatch itself, no marker goes into the stream
    if constexpr (std::is_same<T, float>::value) {
        const size_t smem = prefill_smem_t<T, D>(a.tab_len);
        if (ev) hipExtLaunchKernelGGL((prefill_kernel<T, D, QUEUES>), dim3(a.grid), dim3(PREFILL_THREADS), (uint32_t)smem, st, ev[0], ev[1], 0, a);
        else hipLaunchKernelGGL((prefill_kernel<T, D, QUEUES>), dim3(a.grid), dim3(PREFILL_THREADS), smem, st, a);
    } else {
        const size_t smem = DirectCfg<D>::lds(QUEUES);
        if (ev) hipExtLaunchKernelGGL((prefill_bf16_kernel<D, QUEUES>), dim3(a.grid), dim3(PREFILL_THREADS), (uint32_t)smem, st, ev[0], ev[1], 0, a);
        else hipLaunchKernelGGL((prefill_bf16_kernel<D, QUEUES>), dim3(a.grid), dim3(PREFILL_THREADS), smem, st, a);
    }
    if (!a.arrived) launch_combine<T, D, QUEUES>(a, st, ev);
    return hipGetLastError();
}
template <typename T, int D>
static hipError_t launch_prefill_d(const PrefillArgs& a, hipStream_t st, const hipEvent_t* ev) {
    return a.queue ? launch_prefill_t<T, D, true>(a, st, ev) : launch_prefill_t<T, D, false>(a, st, ev);
}

hipError_t init_prefill_kernels() {
    hipError_t e;
    if ((e = allow_full_lds(&prefill_bf16_kernel<128, true>)) != hipSuccess) return e;
    if ((e = allow_full_lds(&prefill_bf16_kernel<128, false>)) != hipSuccess) return e;
    if ((e = allow_full_lds(&prefill_bf16_kernel<64, true>)) != hipSuccess) return e;
    if ((e = allow_full_lds(&prefill_bf16_kernel<64, false>)) != hipSuccess) return e;
    if ((e = allow_full_lds(&prefill_kernel<float, 128, true>)) != hipSuccess) return e;
    if ((e = allow_full_lds(&prefill_kernel<float, 128, false>)) != hipSuccess) return e;
    if ((e = allow_full_lds(&prefill_kernel<float, 64, true>)) != hipSuccess) return e;
    if ((e = allow_full_lds(&prefill_kernel<float, 64, false>)) != hipSuccess) return e;
    return allow_full_lds(&plan_kernel);
}

size_t prefill_smem_bytes(int dtype, int d, int tab_len) {
    if (dtype == 0) return d == 128 ? DirectCfg<128>::lds(false) : DirectCfg<64>::lds(false);
    if (dtype == 1 && d == 128) return prefill_smem_t<float, 128>(tab_len);
    return prefill_smem_t<float, 64>(tab_len);
}

hipError_t launch_plan(const PlanArgs& a, int BH, hipStream_t st) {
    const size_t smem = (size_t)a.words * 4;
    hipLaunchKernelGGL(plan_kernel, dim3(BH), dim3(1024), smem, st, a);
    return hipGetLastError();
}

int prefill_block_rows() { return BM; }

size_t prefill_slot_bytes(int d) { return (size_t)BM * d * 4 + BM * 2 * 4; }

hipError_t launch_sched(const SchedArgs& a, hipStream_t st) {
    hipLaunchKernelGGL(sched_kernel, dim3(8), dim3(SCHED_THREADS), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_prefill(const PrefillArgs& a, int dtype, int d, hipStream_t st, const hipEvent_t* ev) {
    if (dtype == 0 && d == 128) return launch_prefill_d<bf16_t, 128>(a, st, ev);
    if (dtype == 0 && d == 64) return launch_prefill_d<bf16_t, 64>(a, st, ev);
    if (dtype == 1 && d == 128) return launch_prefill_d<float, 128>(a, st, ev);
    if (dtype == 1 && d == 64) return launch_prefill_d<float, 64>(a, st, ev);
    return hipErrorInvalidValue;
}

}  // namespace ls
