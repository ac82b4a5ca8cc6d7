// Per-head line selection (Alg. 2 from Desc_Sort on) and top-B retention (Alg. 3), gfx950.
//
//   order_kernel  Desc_Sort: the n line weights of a list in descending order, equal weights in ascending index order.
//                 The weights' range is cut into ranges of about as many lines each, a workgroup per range: it picks its
//                 lines out of the list and ranks them inside LDS, so nothing is left to merge.  The last ranges of long lists
//                 are left out where the ones before them outweigh what a walk can take.
//   walk_kernel   one workgroup of six waves per head: the greedy loop of Alg. 2 in binary32 with the operands
//                 and operation order of the definition.  One wave decides runs of up to 1024 picks from one
//                 list with its lanes, one accumulates the running sum pick by pick behind it and finds
//                 the pick that reaches the target, and two waves per list stage the sorted list and its
//                 overlap prefix sums in LDS ahead of both.
//   emit_kernel   one workgroup per (head, list): the chosen prefix of a sorted list becomes an
//                 ascending index list (bitmap in LDS + prefix popcount); a walk that came to the end of what is in order is
//                 done again here.
//   topb_*        Alg. 3: the `budget` largest scores per KV head, ties broken towards smaller indices, ascending output.
//                 Up to TB_ONE_LEN scores one workgroup a head narrows the threshold by bins of equal span; beyond, a radix
//                 select on the float bit patterns is spread over many, one launch per step.
#include <type_traits>
#include "ls_device.h"
#include "ls_internal.h"

namespace ls {

// order-preserving map float -> uint32 (ascending), then inverted so ascending keys = descending floats
__device__ __forceinline__ uint32_t desc_key(float x) {
    const uint32_t u = __builtin_bit_cast(uint32_t, x);
    const uint32_t asc = u ^ ((u >> 31) ? 0xFFFFFFFFu : 0x80000000u);
    return ~asc;
}
__device__ __forceinline__ float key_to_float(uint32_t key) {
    const uint32_t asc = ~key;
    const uint32_t u = (asc >> 31) ? (asc ^ 0x80000000u) : ~asc;
    return __builtin_bit_cast(float, u);
}

constexpr int WALK_BLK = 1024;                 // entries of a sorted list the walk stages at a time
static_assert(WALK_BLK == SELECT_HEAD_LINES, "order_kernel writes the walk's first block in order");
constexpr int ORDER_THREADS = 1024;
constexpr int ORDER_WAVES = 16;
static_assert(ORDER_WAVES == 16, "waves_before adds a row of lanes");
constexpr int ORDER_CHUNKS = 10;               // most lines of a workgroup, in 1024
constexpr int ORDER_ONE = 5120;                // longest list that one workgroup puts in order, whatever the number of lists
constexpr int ORDER_SAMPLES = 2048;            // of a list, for the bounds of its ranges
constexpr int ORDER_WIDE = 65536;              // lists beyond: shorter ranges, with more room
constexpr float ORDER_GOAL = 1.f + 1.f / 512;  // of the target: what lines before a range have to have of it for the range to be left out (its sums round otherwise than the walk's)
constexpr int LAZY_LINES = 8193;               // shorter lists are put in order throughout: 32 heads of 8192 lines 17.3 us, lazily 17.4
constexpr int ORDER_FULL = 32;                 // lines of the fullest bin that are still ranked against each other
// ... and of the last bin of a list in one range: where rows are sampled a percent or two of the columns and diagonals are seen by none of them and weigh nothing, and another spread of the
// whole list only for these takes 4 us (16 heads of 5003 lines 34.0 -> 28.6, 64 of 6500 40.5 -> 33.6, 32 of 3500 28.2 -> 24.1, of 2000 22.5 -> 19.9).  Of any bin: 64 heads of 8192 lines that crowd 72 -> 78.
constexpr int ORDER_LAST = 128;
constexpr int order_fine(int pt) { return pt * 2 * ORDER_THREADS; }        // fine bins, where a thread has `pt` words of them
constexpr size_t order_lds_bytes(int pt, int cap) { return (size_t)order_fine(pt) * 2 + 16 + 1024 * 4 + (size_t)cap * 12; }
static_assert(order_fine(4) * 2 >= 4096 * 4 && order_fine(8) >= 1024 * ORDER_CHUNKS, "room for order_bounds, a bin per line");
constexpr int ORDER_SEGS = 320;                // most bins with more lines than that
static_assert(1024 * ORDER_CHUNKS / (ORDER_FULL + 1) < ORDER_SEGS && 2 * ORDER_SEGS <= 1024 && 1024 * ORDER_CHUNKS <= 1 << 14, "words for each of them, places 14 bits");

// smallest / largest of the wave's, in lane 63
template <int CTRL, int ROWS> __device__ __forceinline__ uint32_t dpp_min(uint32_t x) { const uint32_t o = (uint32_t)__builtin_amdgcn_update_dpp((int)x, (int)x, CTRL, ROWS, 0xF, false); return o < x ? o : x; }
__device__ __forceinline__ uint32_t lanes_min(uint32_t x) {
    x = dpp_min<0x111, 0xF>(x); x = dpp_min<0x112, 0xF>(x); x = dpp_min<0x114, 0xF>(x); x = dpp_min<0x118, 0xF>(x);       // row_shr:1, 2, 4, 8
    x = dpp_min<0x142, 0xA>(x);                            // row_bcast15 into rows 1 and 3
    return dpp_min<0x143, 0xC>(x);                         // row_bcast31 into rows 2 and 3
}
__device__ __forceinline__ uint32_t lanes_max(uint32_t x) { return ~lanes_min(~x); }
// bits of a number
__device__ __forceinline__ int width_of(uint32_t x) { return x == 0u ? 0 : 32 - __builtin_clz(x); }

// What the workgroup keeps beside the keys: `red` for sums over the waves (two rounds that follow each other use different halves).
struct OrderSync { uint32_t red[4][ORDER_WAVES], count[4 * ORDER_WAVES], bin[2], rest[2], many[2], next; float mass[4 * ORDER_WAVES]; int32_t cross[4]; uint16_t lines[ORDER_SEGS]; };

// Smallest and largest over the waves, of what each left in the two halves of `red`
__device__ __forceinline__ void waves_extremes(const uint32_t (*red)[ORDER_WAVES], int lane, uint32_t& least, uint32_t& most) {
    least = (uint32_t)__builtin_amdgcn_readlane((int)lanes_min(red[0][lane & 15]), 63);
    most = (uint32_t)__builtin_amdgcn_readlane((int)lanes_max(red[1][lane & 15]), 63);
}

// Sum of `x` over the threads before this one, and over all of them.  One barrier; `red` must not be in use.
__device__ __forceinline__ uint32_t order_scan(uint32_t x, uint32_t* red, int lane, int wv, uint32_t& total) {
    const uint32_t upto = lanes_upto(x);
    if (lane == 63) red[wv] = upto;
    __syncthreads();
    return waves_before(red, lane, wv, total) + upto - x;
}

// Where a range begins: lines of a lighter weight come behind it, and lines of its weight from `line` on.  -1: all of them.
// earlier, later: the bound before or behind it lies among the lines of the same weight as well.
struct OrderBound { uint32_t key; int32_t line; bool earlier, later; };

// The bounds of range `b` of `nb`: the samples of rank b S / nb and (b + 1) S / nb among S = 2048 of them, two a thread (sample i before
// sample i + 1 in the list).  The key is found to 20 bits of the samples' span, and to the last bit where more than `few`
// samples lie in one such step; the line is given where as many samples have one weight: its lines then fall
// to several ranges.  The same numbers in every workgroup of the list: a bound depends on its rank alone.
// next: of the first line of range `next` (that is to have one) a key that is not greater.
// hist: 4096 words of LDS.
__device__ __forceinline__ void order_bounds(const uint32_t (&key)[2], const int32_t (&pos)[2], int b, int nb, int next, uint32_t few, uint32_t* hist, OrderSync& sync, OrderBound& from, OrderBound& to, uint32_t& next_key) {
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    constexpr int PER = 2, S = ORDER_SAMPLES;
    static_assert(S == PER * ORDER_THREADS, "two a thread");
    uint32_t lo = 0xFFFFFFFFu, hi = 0u;
    hist[tid] = 0u; hist[1024 + tid] = 0u;
#pragma unroll
    for (int j = 0; j < PER; ++j) { lo = key[j] < lo ? key[j] : lo; hi = key[j] > hi ? key[j] : hi; }
    lo = lanes_min(lo); hi = lanes_max(hi);
    if (lane == 63) { sync.red[0][wv] = lo; sync.red[1][wv] = hi; }
    __syncthreads();
    waves_extremes(sync.red, lane, lo, hi);
    const int width = width_of(hi - lo), sh = width > 20 ? width - 20 : 0;
    uint32_t at[PER];
#pragma unroll
    for (int j = 0; j < PER; ++j) { at[j] = (key[j] - lo) >> sh; atomicAdd(&hist[at[j] >> 10], 1u); }
    __syncthreads();
    // bins of the two ranks, then the bins inside those (of both at once, in the halves of a word)
    const uint32_t t0 = (uint32_t)(b * S / nb), t1 = (uint32_t)((b + 1) * S / nb), t2 = (uint32_t)(next * S / nb);
    uint32_t all;
    uint32_t v = hist[tid], e = order_scan(v, sync.red[0], lane, wv, all);
    if (t0 >= e && t0 < e + v) { sync.bin[0] = (uint32_t)tid; sync.rest[0] = t0 - e; }
    if (t1 >= e && t1 < e + v) { sync.bin[1] = (uint32_t)tid; sync.rest[1] = t1 - e; }
    if (t2 >= e && t2 < e + v) sync.next = (uint32_t)tid;
    if (b == nb - 1 && tid == 0) { sync.bin[1] = 1023u; sync.rest[1] = 0u; }             // (no bound: not looked at)
    __syncthreads();
    const uint32_t bin0 = sync.bin[0], bin1 = sync.bin[1];
    next_key = next < nb ? lo + (sync.next << 10 << sh) : 0u;
    uint32_t rest0 = sync.rest[0], rest1 = sync.rest[1];
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const uint32_t add = ((at[j] >> 10) == bin0 ? 1u : 0u) | ((at[j] >> 10) == bin1 ? 0x10000u : 0u);
        if (add) atomicAdd(&hist[1024 + (at[j] & 1023u)], add);
    }
    __syncthreads();
    v = hist[1024 + tid]; e = order_scan(v, sync.red[1], lane, wv, all);
    if (rest0 >= (e & 0xFFFFu) && rest0 < (e & 0xFFFFu) + (v & 0xFFFFu)) { sync.bin[0] = (uint32_t)tid; sync.rest[0] = rest0 - (e & 0xFFFFu); sync.many[0] = v & 0xFFFFu; }
    if (b < nb - 1 && rest1 >= (e >> 16) && rest1 < (e >> 16) + (v >> 16)) { sync.bin[1] = (uint32_t)tid; sync.rest[1] = rest1 - (e >> 16); sync.many[1] = v >> 16; }
    __syncthreads();
    uint32_t f0 = bin0 << 10 | sync.bin[0], f1 = bin1 << 10 | sync.bin[1];
    uint32_t many0 = b > 0 ? sync.many[0] : 0u, many1 = b < nb - 1 ? sync.many[1] : 0u;
    rest0 = sync.rest[0]; rest1 = sync.rest[1];
    from = OrderBound{lo + (f0 << sh), -1, false, false};
    to = OrderBound{lo + (f1 << sh), -1, false, false};
    if (many0 <= few && many1 <= few) return;              // (uniform, as all of this)
    if (sh > 0) {                                          // the last bits, at most 12
#pragma unroll
        for (int j = 0; j < 4; ++j) hist[4 * tid + j] = 0u;
        __syncthreads();
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            const uint32_t add = (at[j] == f0 ? 1u : 0u) | (at[j] == f1 ? 0x10000u : 0u);
            if (add) atomicAdd(&hist[(key[j] - lo) & ((1u << sh) - 1u)], add);
        }
        __syncthreads();
        uint32_t h[4], sum = 0u;
#pragma unroll
        for (int j = 0; j < 4; ++j) { h[j] = hist[4 * tid + j]; sum += h[j]; }
        e = order_scan(sum, sync.red[0], lane, wv, all);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint32_t x = h[j] & 0xFFFFu, y = h[j] >> 16, ex = e & 0xFFFFu, ey = e >> 16;
            if (rest0 >= ex && rest0 < ex + x) { sync.bin[0] = (uint32_t)(4 * tid + j); sync.rest[0] = rest0 - ex; sync.many[0] = x; }
            if (rest1 >= ey && rest1 < ey + y) { sync.bin[1] = (uint32_t)(4 * tid + j); sync.rest[1] = rest1 - ey; sync.many[1] = y; }
            e += h[j];
        }
        __syncthreads();
        f0 = f0 << sh | sync.bin[0]; f1 = f1 << sh | sync.bin[1];
        rest0 = sync.rest[0]; rest1 = sync.rest[1];
        if (many0 > few) { from.key = lo + f0; many0 = sync.many[0]; }
        if (many1 > few) { to.key = lo + f1; many1 = sync.many[1]; }
        if (many0 <= few && many1 <= few) return;
    }
    // samples of the bound's weight, in the list's order
    uint32_t upto = 0u;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const bool is0 = many0 > few && key[j] == from.key, is1 = many1 > few && key[j] == to.key;
        const uint32_t n = upto + order_scan((is0 ? 1u : 0u) | (is1 ? 0x10000u : 0u), sync.red[j ^ 1], lane, wv, all);
        if (is0 && (n & 0xFFFFu) == rest0) sync.bin[0] = (uint32_t)pos[j];
        if (is1 && (n >> 16) == rest1) sync.bin[1] = (uint32_t)pos[j];
        upto += all;
    }
    __syncthreads();
    auto rank = [&](int r) -> int { return r * S / nb; };
    auto finish = [&](OrderBound& x, int r, uint32_t bin, uint32_t rest, uint32_t many) {      // r: the range that it begins
        x.line = (int32_t)bin;
        const int first = rank(r) - (int)rest;
        x.earlier = r > 1 && rank(r - 1) >= first;
        x.later = r + 1 < nb && rank(r + 1) < first + (int)many;
    };
    if (many0 > few) finish(from, b, sync.bin[0], rest0, many0);
    if (many1 > few) finish(to, b + 1, sync.bin[1], rest1, many1);
}

// Desc_Sort.  grid (lists, nb); list 2 bh + 0 = diagonals (slash), + 1 = columns (vert) of a head.  (Workgroups of a list are
// `lists` apart: with a multiple of eight lists in one XCD, whose L2 then fetches the list once.)
// Workgroup b puts the b-th of nb ranges of weights in order (WHOLE: the list, of up to `cap` lines).  It
//   - finds the range's bounds from 2048 samples of the list, so that each range has about as many lines;
//   - counts the range's lines and those before it, and takes the former into LDS, in index order;
//   - spreads them over bins, about one line each (below), and ranks the few lines of a bin against each other, by weight
//     and then by index; bins with too many lines are spread again, each over as many bins as it has lines;
//   - writes their indices (sidx), weights and maxima (sorted_w, sorted_m: of as many lines as there is room for, 1024 at least) where they belong, so that
//     the walk reads what it needs as it lies.  (Fetched by the walk through the indices, 1024 lines took it 2500 cycles and more, of which it can go through them in 1500.)
// The lines of a weight that has ranges to itself are written as they come, by one workgroup, and so are many lines of weights that
// two ranges meet in.  A range of more than `cap` lines all the same (the samples missed them) is halved until it fits.
//
// What bounds it: the instructions of sixteen waves that look through the whole list twice, and latencies; one workgroup per CU.  32768 lines in eight ranges, cycles of a workgroup:
// bounds 8000, count 11000, lines into LDS 9000, their span 1700, bins 9500, ranks and results 11000.  So the two looks take four lines a lane at once, eight instructions a line, with
// the weights as they are where their sign allows it, in a short loop with the next lines under way (unrolled over 1024 lines it was half as long again: a workgroup runs through its
// code once and has to fetch it), and two lists of lines that are not needed are not ranked.  A maximum is fetched when its line is placed and written with the next one.
// 32 heads, the kernel alone, us, everything in order and only the first 1024 lines' weights / now: 32768 lines 28.6 / 25.5, 12347 18.5 / 17.0, 8192 15.5 / 17.2, 5003 (16 heads) 12.6 / 14.0 (in one range 13.3),
// 131072 226 / 141, 256 heads of 16384 104 / 92; the walk, which gains what short lists lose here, 24.0 / 15.5, 12.7 / 10.6, 16.1 / 13.8, 14.4 / 12.2, 123 / 52, 25.8 / 18.5.
// (Keys and bins in registers, ten lines a thread, ranks by indirection and many equal weights by digits, 30 KB of code and 88 bytes of scratch: 32 heads of 32768 lines 35 us where the
// bins in LDS took 30.)
// Lists that crowd, 32 heads, the kernel alone, us, by digits / now / segments of 8192 sorted by digits and merged:
// all but ten lines within 2^12 numbers 1024 lines 13.6 / 10.7 / 7.7, 4096 27.9 / 17.1 / 14.4, 32768 122 / 48 / 54, 131072 320 / 354 / 323; two thirds of one
// weight, the others of 59 4096 31.9 / 21.6 / 17.7, 32768 96 / 47 / 59, 131072 300 / 238 / 326; two fifths zero 4096 25.6 / 18.3 / 15.0, 32768 34 / 33 / 53,
// 131072 233 / 219 / 317; 59 weights 4096 26.6 / 16.9 / 17.0, 32768 69 / 57 / 56.
// Where a range begins or ends inside a weight its looks through the list take longer.  So weights of less than two fifths of a range are left whole
// beyond ORDER_WIDE lines, where there is room for them, and lines at the ends are ranked with the others unless they are more than
// half.  ls_select that ends after its first pick, by digits / every weight shared that has a sixteenth, its lines written apart / now / segments:
// 59 weights 80862 lines 332 / 284 / 217 / 199, 131072 432 / 466 / 387 / 309, 262144 1020 / 1300 / 1240 / 880 (there each has two thirds of a range);
// 300 weights 131072 406 / 462 / 329 / 315; two thirds of one weight 131072 356 / 281 / 215 / 328; within 2^12 numbers 262144 1745 / 1230 / 934 / 946.
// (WHOLE: two workgroups per CU; 256 heads of 1500 lines, the whole ls_select, 29.4 -> 27.9.)
//
// LAZY: range b, unless the lines of the ranges before it have `goal` of weight between them, which is more than a walk takes from a list: picks from
// one list alone reach the target with that, and where columns and diagonals are both taken the overlaps stop the walk after a few of them, or each takes fewer (32 heads of 8192 to
// 32768 lines went no deeper than 9100 lines, the mixed ones 170).  A walk that needs more, because overlaps are there but smaller than the last lines' weights, is emit_kernel's.
// a.info of the range then says how many lines those are.  Whether the lines before range `next`, the workgroup's next one, have
// as much is known as well once the lines have been counted: false, and said in a.info, if they have.
template <int PT, bool WHOLE, bool LAZY>
__device__ __forceinline__ bool order_range(const SelectArgs& a, const int list, const int bh, const int b, const int nb, const int next, const int cap, const float goal, unsigned char* order_lds, OrderSync& sync) {
    constexpr int FINE = order_fine(PT);
    uint32_t* words = reinterpret_cast<uint32_t*>(order_lds);                            // of the fine bins: lines, then places, in pairs
    uint16_t* fine = reinterpret_cast<uint16_t*>(order_lds);                             // [FINE + 1] bin f's at f + 1; in the end bin f has the places from fine[f] up to fine[f + 1]
    uint32_t* coarse = reinterpret_cast<uint32_t*>(order_lds + FINE * 2 + 16);           // [1024]; later least and largest key of the bins that are too full
    uint32_t* keys = coarse + 1024;                                                      // [cap] of the range's lines, in index order
    uint32_t* spread = keys + cap;                                                       // [cap] by fine bin: how far into the bin << 14 | place in `keys`
    uint16_t* line = reinterpret_cast<uint16_t*>(spread + cap);                          // [cap] index, low half
    uint16_t* bins = line + cap;                                                         // [cap] fine bin | DONE | EQUAL; between two spreads, place in the order | DONE or first place of its bin
    constexpr uint32_t PLACE = 0x3FFFu, DONE = 0x4000u, EQUAL = 0x8000u;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = (int)a.n;
    const float* src = (list == 0 ? a.slash : a.vert) + (int64_t)bh * n;
    const float* mx = (list == 0 ? a.smax : a.vmax) + (int64_t)bh * n;
    int32_t* out = a.sidx + ((int64_t)list * a.BH + bh) * n;
    const int kept = (int)a.kept;                          // lines of the order whose weight and maximum are written as well
    float* sorted_w = a.sorted_w + ((int64_t)list * a.BH + bh) * kept;
    float* sorted_m = a.sorted_m ? a.sorted_m + ((int64_t)list * a.BH + bh) * kept : nullptr;
    auto say = [&](int range, int what) { if (!WHOLE && a.info && tid == 0) a.info[((int64_t)list * a.BH + bh) * SELECT_RANGES + range] = what; };
    const int per = (n + 4 * ORDER_THREADS - 1) / (4 * ORDER_THREADS) * 256;
    const int w0 = wv * per < n ? wv * per : n, w1 = w0 + per < n ? w0 + per : n;         // this wave's lines
    typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
    // f(first line, weights, how many of the four there are) for the wave's lines, four a lane, in the list's order, 256 at a time with the next under way; the last, of which
    // there may be fewer, by themselves.
    auto lines4 = [&](auto f) {
        int i0 = w0;
        const int rest = w0 + (w1 - w0) / 256 * 256 + 4 * lane, from = rest < n - 4 ? rest : n - 4;
        f32x4u y = f32x4u{0.f, 0.f, 0.f, 0.f};
        if (w1 == n && w0 < n) y = *reinterpret_cast<const f32x4u*>(src + from);
        if (i0 + 256 <= w1) {
            const float* at = src + w0 + 4 * lane;
            f32x4u next4 = *reinterpret_cast<const f32x4u*>(at);
#pragma unroll 1
            for (;;) {
                const f32x4u x = next4;
                const bool again = i0 + 512 <= w1;
                at += 256;
                if (again) next4 = *reinterpret_cast<const f32x4u*>(at);
                f(i0 + 4 * lane, x, std::integral_constant<int, 4>{});
                i0 += 256;
                if (!again) break;
            }
        }
        if (i0 < w1) {                                     // (the list's end: a lane whose four would reach beyond it has the list's last four, and takes of them what is its own)
            const int by = rest - from, some = w1 - rest;
            const float p = (by & 1) ? y[1] : y[0], q = (by & 1) ? y[2] : y[1], r = (by & 1) ? y[3] : y[2];
            const f32x4u x = {(by & 2) ? r : p, (by & 2) ? y[3] : q, r, y[3]};
            f(rest, x, some < 0 ? 0 : some < 4 ? some : 4);
        }
    };
    // f(line, key, whether there is such a line) for the wave's lines, 64 at a time
    auto read = [&](auto f) {
        for (int i0 = w0; i0 < w1; i0 += 64 * 8) {
            float x[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) { const int i = i0 + 64 * j + lane; x[j] = src[i < n ? i : n - 1]; }
#pragma unroll
            for (int j = 0; j < 8; ++j) { const int i = i0 + 64 * j + lane; f(i, desc_key(x[j]), i < w1); }
        }
    };
    // (a maximum is written when the thread has its next one to ask for, which then does not wait for it)
    float top = 0.f;
    int top_at = -1;
    bool odd = false;                                      // one of them is negative or no number
    auto settle = [&]() {
        if (top_at < 0) return;
        sorted_m[top_at] = top;
        if (!WHOLE) odd = odd || !(top >= 0.f);
        top_at = -1;
    };
    auto put = [&](int at, int i, uint32_t k) {            // line i is the `at`-th of the order
        out[at] = i;
        if (at < kept) {
            sorted_w[at] = key_to_float(k);
            if (sorted_m) { settle(); top = mx[i]; top_at = at; }
        }
    };
    auto lanes_before = [](uint64_t who) -> int { return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(who >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)who, 0u)); };
    // The range: the weights from `lo` to `end`.  With `ends` it begins or ends among lines of one weight, has all lines from key << 32 | index of
    // `lo_line` to that of `end_line`, and `lo` to `end` are the weights between `front` and `back`, its first and the first behind it.
    uint32_t lo = 0u, end = 0xFFFFFFFFu, front = 0u, back = 0u;
    uint64_t lo_line = 0u, end_line = ~0ull;
    bool ends = false, alone = false;                      // alone: `front` is its only weight
    uint32_t next_key = 0u;
    bool more = true;
    if (!WHOLE) {
        uint32_t sample[2];
        int32_t where[2];
        OrderBound from, to;
#pragma unroll
        for (int j = 0; j < 2; ++j) {                      // somewhere in the i-th 2048th of the list, so that no period of it is met
            const int i = tid + j * ORDER_THREADS, len = n / (2 * ORDER_THREADS);
            where[j] = (int)((int64_t)i * n / (2 * ORDER_THREADS)) + (int)((((uint32_t)i * 0x9E3779B1u) >> 16) * (uint32_t)len >> 16);
            sample[j] = desc_key(src[where[j]]);
        }
        // weights of so many samples are shared: two fifths of a range where it has room for that beside its own, a sixteenth where they would leave the
        // ranges unequal
        const uint32_t few = (uint32_t)(n > ORDER_WIDE ? 2 * ORDER_SAMPLES / (5 * nb) : ORDER_SAMPLES / (16 * nb));
        order_bounds(sample, where, b, nb, next, few, words, sync, from, to, next_key);
        const bool last = b == nb - 1;
        if (b == 0) from = OrderBound{0u, -1, false, false};
        // A weight that has ranges to itself: the first of them takes all its lines, those at its ends none
        if (!last && to.line >= 0 && (to.earlier || to.later)) {
            if (from.line >= 0 && from.key == to.key) {
                if (from.earlier) { say(b, 0); return true; }
                from.line = 0; to.line = 0x7FFFFFFF;
            } else {
                to.line = -1;
            }
        }
        if (from.line >= 0 && (from.earlier || from.later) && (last || from.key != to.key)) {
            if (from.key == 0xFFFFFFFFu) { say(b, 0); return true; }
            from.line = -1; ++from.key;
        }
        lo_line = (uint64_t)from.key << 32 | (uint32_t)(from.line > 0 ? from.line : 0);
        lo = from.key;
        if (!last) {
            const uint64_t behind = (uint64_t)to.key << 32 | (uint32_t)(to.line > 0 ? to.line : 0);
            if (behind <= lo_line) { say(b, 0); return true; }   // nothing (the bounds are the same for every thread)
            end_line = behind - 1u;
            end = to.key - 1u;
        }
        if (from.line >= 0 || (!last && to.line >= 0)) {
            ends = true;
            alone = !last && to.key == from.key;
            front = lo++; back = last ? front : to.key;
        }
    }
    uint32_t hi = end;
    int base = WHOLE ? 0 : -1;                             // place of the range's first line in the order
    if (!WHOLE && tid < 4) sync.cross[tid] = 0x7FFFFFFF;
    for (;;) {
        int before = w0, m = n;                            // lines of the range in the waves before, and in all (a list in one range: all lines)
        bool picked = false, plain = false;
        const uint32_t span = hi - lo;
        if (!WHOLE) {
            // Weights as integers in the order of the floats: t, largest first.  (That of a weight of 0 or more is its bits, and of others the sign is enough where
            // a range begins at 0 or more and ends there as well or nowhere.)
            const int t_last = (int)(hi ^ 0x7FFFFFFFu), t_first = (int)(lo ^ 0x7FFFFFFFu), t_next = (int)(next_key ^ 0x7FFFFFFFu);
            plain = t_first >= 0 && t_next >= 0 && (t_last >= 0 || t_last == (int)0x80000000);
            // of this lane's lines: in the range, before it, before range `next`, of the weights at its ends; the weight of those before each
            uint32_t here = 0u, below = 0u, short_of = 0u, fronts = 0u, backs = 0u;
            float mass = 0.f, next_mass = 0.f;
            if (ends) {
                lines4([&](int i, const f32x4u& w, auto some) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const uint32_t k = desc_key(w[e]);
                        const uint64_t x = (uint64_t)k << 32 | (uint32_t)(i + e);
                        const bool any = e < some, in = any && x - lo_line <= end_line - lo_line, less = any && x < lo_line, before_next = any && k < next_key;
                        here += in ? 1u : 0u; below += less ? 1u : 0u; fronts += in && k == front ? 1u : 0u; backs += in && k == back && front != back ? 1u : 0u;
                        if (LAZY) { short_of += before_next ? 1u : 0u; mass += less ? w[e] : 0.f; next_mass += before_next ? w[e] : 0.f; }
                    }
                });
            } else {
                lines4([&](int, const f32x4u& w, auto some) {
                    int t[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) { const float x = w[e]; t[e] = __builtin_bit_cast(int, x); }      // (not of the vector's element: that is always the first)
                    if (!plain) {
#pragma unroll
                        for (int e = 0; e < 4; ++e) t[e] ^= (t[e] >> 31) & 0x7FFFFFFF;
                    }
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const bool any = e < some, less = any && t[e] > t_first, before_next = any && t[e] > t_next;
                        here += any && (uint32_t)t[e] - (uint32_t)t_last <= span ? 1u : 0u; below += less ? 1u : 0u;
                        if (LAZY) { short_of += before_next ? 1u : 0u; mass += less ? w[e] : 0.f; next_mass += before_next ? w[e] : 0.f; }
                    }
                });
            }
            {
                const uint32_t two = lanes_upto(here | below << 16);                     // (at most 16384 lines a wave)
                if (LAZY) { short_of = lanes_upto(short_of); mass = wave_sum(mass); next_mass = wave_sum(next_mass); }
                __syncthreads();                           // `red` and the last range's lines are free again
                if (lane == 63) {
                    sync.count[wv] = two & 0xFFFFu; sync.count[ORDER_WAVES + wv] = two >> 16; sync.count[2 * ORDER_WAVES + wv] = short_of;
                    if (LAZY) { sync.mass[wv] = mass; sync.mass[ORDER_WAVES + wv] = next_mass; }
                }
                if (ends) {
                    fronts = lanes_upto(fronts); backs = lanes_upto(backs);
                    if (lane == 63) { sync.red[2][wv] = fronts; sync.red[3][wv] = backs; }
                }
            }
            __syncthreads();
            // sums over the waves, three at once in rows of sixteen lanes
            int sums = (int)sync.count[lane];
            sums += __builtin_amdgcn_update_dpp(0, sums, 0x111, 0xF, 0xF, false);        // row_shr:1, 2, 4, 8
            sums += __builtin_amdgcn_update_dpp(0, sums, 0x112, 0xF, 0xF, false);
            sums += __builtin_amdgcn_update_dpp(0, sums, 0x114, 0xF, 0xF, false);
            sums += __builtin_amdgcn_update_dpp(0, sums, 0x118, 0xF, 0xF, false);
            m = __builtin_amdgcn_readlane(sums, 15);
            before = wv > 0 ? __builtin_amdgcn_readlane(sums, wv - 1) : 0;
            const int ahead = __builtin_amdgcn_readlane(sums, 31);
            if (LAZY && base < 0) {
                float g = sync.mass[lane];
                auto fl = [](int x) { return __builtin_bit_cast(float, x); };
                g += fl(__builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, g), 0x111, 0xF, 0xF, false));
                g += fl(__builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, g), 0x112, 0xF, 0xF, false));
                g += fl(__builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, g), 0x114, 0xF, 0xF, false));
                g += fl(__builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, g), 0x118, 0xF, 0xF, false));
                if (b > 0 && fl(__builtin_amdgcn_readlane(__builtin_bit_cast(int, g), 15)) >= goal) {
                    say(b, -1 - ahead);
                    if (next < nb) say(next, -1 - ahead);
                    return false;
                }
                more = !(next < nb && fl(__builtin_amdgcn_readlane(__builtin_bit_cast(int, g), 31)) >= goal);
                if (!more) say(next, -1 - __builtin_amdgcn_readlane(sums, 47));
            }
            if (base < 0) base = ahead;
            if (ends) {
                uint32_t f_all, r_all;
                const int f_before = (int)waves_before(sync.red[2], lane, wv, f_all), r_before = (int)waves_before(sync.red[3], lane, wv, r_all);
                if (m > cap || 2 * (int)(f_all + r_all) > m) {               // the order of the lines at the ends is there: they are written now, the others picked on the way
                    before -= f_before + r_before; m -= (int)(f_all + r_all);
                    int f_at = base + f_before, at = before;
                    base += (int)f_all;
                    int r_at = base + m + r_before;
                    picked = m <= cap;
                    if (!alone || (w1 > (int)(uint32_t)lo_line && w0 <= (int)(uint32_t)end_line)) read([&](int i, uint32_t k, bool any) {
                        const uint64_t x = (uint64_t)k << 32 | (uint32_t)i;
                        const bool in = any && x - lo_line <= end_line - lo_line, f = in && k == front, r = in && k == back && !f, mid = in && !f && !r;
                        const uint64_t fs = __ballot(f), rs = __ballot(r), who = __ballot(mid);
                        if ((i & 0xFFFF) == 0 && any) sync.cross[i >> 16] = at;
                        if (mid && picked) { const int p = at + lanes_before(who); keys[p] = k; line[p] = (uint16_t)i; }
                        if (f || r) put((f ? f_at : r_at) + lanes_before(f ? fs : rs), i, k);
                        f_at += __popcll(fs); r_at += __popcll(rs); at += __popcll(who);
                    });
                    ends = false;
                }
            }
        }
        uint32_t least = 0xFFFFFFFFu, most = 0u;
        auto extremes = [&](uint32_t k, bool in) { least = in && k < least ? k : least; most = in && k > most ? k : most; };
        auto agree = [&]() {                               // (all threads; `red` must have been read)
            least = lanes_min(least); most = lanes_max(most);
            if (lane == 63) { sync.red[0][wv] = least; sync.red[1][wv] = most; }
            __syncthreads();
            waves_extremes(sync.red, lane, least, most);
        };
        if (!WHOLE && m > cap) {                           // more than expected (the samples missed them)
            read([&](int, uint32_t k, bool any) { extremes(k, any && k - lo <= span); });
            __syncthreads();
            agree();
            if (least < most) { lo = least; hi = least + (most - least) / 2; continue; }           // the lower half of the span that its weights have
            read([&](int i, uint32_t k, bool any) {        // equal weights: the order is there
                const bool in = any && k == least;
                const uint64_t who = __ballot(in);
                if (in) put(base + before + lanes_before(who), i, k);
                before += __popcll(who);
            });
        } else if (m > 0) {
            for (int i = tid; i <= FINE / 2; i += ORDER_THREADS) words[i] = 0u;
            coarse[tid] = 0u;
            if (WHOLE) {
                for (int p = tid; p < m; p += ORDER_THREADS) { const uint32_t k = desc_key(src[p]); keys[p] = k; extremes(k, true); }
            } else {
                if (ends) {
                    read([&](int i, uint32_t k, bool any) {
                        const bool in = any && ((uint64_t)k << 32 | (uint32_t)i) - lo_line <= end_line - lo_line;
                        const uint64_t who = __ballot(in);
                        const int at = before + lanes_before(who);
                        if (in) { keys[at] = k; line[at] = (uint16_t)i; }
                        if ((i & 0xFFFF) == 0 && any) sync.cross[i >> 16] = before;
                        before += __popcll(who);
                    });
                } else if (!picked) {                      // (the bits of their weights, for now)
                    const int t_last = (int)(hi ^ 0x7FFFFFFFu);
                    lines4([&](int i, const f32x4u& w, auto some) {
                        bool in[4];
                        float x[4];
                        uint32_t mine = 0u;
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            x[e] = w[e];
                            int t = __builtin_bit_cast(int, x[e]);
                            if (!plain) t ^= (t >> 31) & 0x7FFFFFFF;
                            in[e] = e < some && (uint32_t)t - (uint32_t)t_last <= span;
                            mine += in[e] ? 1u : 0u;
                        }
                        const uint32_t upto = lanes_upto(mine);
                        int p = before + (int)(upto - mine);
                        if (n > 65536 && (i & 0xFFFF) == 0 && some > 0) sync.cross[i >> 16] = p;
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            if (in[e]) { keys[p] = __builtin_bit_cast(uint32_t, x[e]); line[p] = (uint16_t)(i + e); }
                            p += in[e] ? 1 : 0;
                        }
                        before += __builtin_amdgcn_readlane((int)upto, 63);
                    });
                }
                __syncthreads();
                const bool bits = !ends && !picked;
                for (int p = tid; p < m; p += ORDER_THREADS) {
                    uint32_t k = keys[p];
                    if (bits) { k = desc_key(__builtin_bit_cast(float, k)); keys[p] = k; }
                    extremes(k, true);
                }
            }
            agree();
            const int c1 = sync.cross[1], c2 = sync.cross[2], c3 = sync.cross[3];
            auto line_at = [&](int p) -> int {             // (index of the p-th line of the range)
                if (WHOLE) return p;
                return (int)line[p] + (n > 65536 ? (p >= c1 ? 65536 : 0) + (p >= c2 ? 65536 : 0) + (p >= c3 ? 65536 : 0) : 0);
            };
            const int width = __builtin_amdgcn_readfirstlane(width_of(most - least));
            if (width == 0) {                              // equal weights: the order is there
                for (int p = tid; p < m; p += ORDER_THREADS) put(base + p, line_at(p), least);
            } else {
                // 1024 coarse bins of equal span, and of each as many fine bins of equal span as it has lines (or a few times
                // that): a fine bin then has about one line wherever the weights crowd
                const int sh = width > 10 ? width - 10 : 0, place_sh = 32 - width_of((uint32_t)m - 1u);
                const uint32_t times = (uint32_t)(FINE / m);
                for (int p = tid; p < m; p += ORDER_THREADS) {                  // (lines of the first lane's bin at once: all may be in one)
                    const uint32_t c = (keys[p] - least) >> sh;
                    const bool same = c == (uint32_t)__builtin_amdgcn_readfirstlane((int)c);
                    const uint64_t who = __ballot(same);
                    if (!same || lanes_before(who) == 0) atomicAdd(&coarse[c], same ? (uint32_t)__popcll(who) : 1u);
                }
                __syncthreads();
                uint32_t all;
                const uint32_t mine = coarse[tid], ahead_of = order_scan(mine, sync.red[2], lane, wv, all);
                coarse[tid] = ahead_of * times | (mine * times) << 16;      // (at most 16384: first bin below it or no line, number)
                __syncthreads();
                // The 18 bits tell all keys of a bin apart where its coarse bin has so many fine ones, and always in later spreads, whose
                // bins span less than 2^18 numbers.
                const uint32_t tell = sh > 18 ? 1u << (sh - 18) : 0u;
                for (bool again = false;; again = true) {
                    // fine bin of line p | DONE | EQUAL, and how far into the bin it lies, in 2^-32 of it
                    auto locate = [&](int p, uint32_t& into) -> uint32_t {
                        uint32_t first, lines, step, flags = 0u;
                        if (!again) {
                            const uint32_t d = keys[p] - least, w = coarse[d >> sh];
                            first = w & 0xFFFFu; lines = w >> 16; step = sh ? d << (32 - sh) : 0u;
                        } else {
                            const uint32_t x = bins[p], at = x & PLACE, s = at / (ORDER_FULL + 1);
                            first = at * times; into = 0u;
                            if (x & DONE) return first | DONE;
                            const uint32_t low = coarse[s], wide = coarse[ORDER_SEGS + s] - low;
                            lines = sync.lines[s] * times;
                            step = wide ? (keys[p] - low) << (32 - width_of(wide)) : (uint32_t)p << place_sh;
                            flags = wide ? 0u : EQUAL;
                        }
                        const uint64_t x = (uint64_t)step * lines;
                        into = (uint32_t)x;
                        return (first + (uint32_t)(x >> 32)) | flags;
                    };
                    auto meet = [&](uint32_t f) -> uint32_t {                  // its count goes up by one
                        const uint32_t h = (f & PLACE) + 1u;
                        return atomicAdd(&words[h >> 1], 1u << (16 * (h & 1u))) >> (16 * (h & 1u)) & 0xFFFFu;
                    };
                    for (int p = tid; p < m; p += ORDER_THREADS) { uint32_t into; meet(locate(p, into)); }
                    __syncthreads();
                    bool full;
                    {                                      // where each fine bin begins
                        uint32_t t[PT], sum = 0u, fullest = 0u;
#pragma unroll
                        for (int j = 0; j < PT; ++j) t[j] = words[PT * tid + j];
                        const uint32_t very_last = words[FINE / 2];
#pragma unroll
                        for (int j = 0; j < PT; ++j) {
                            const uint32_t x = t[j] & 0xFFFFu, y = t[j] >> 16;
                            sum += x + y; fullest = x > fullest ? x : fullest; fullest = y > fullest ? y : fullest;
                        }
                        fullest = very_last > fullest ? very_last : fullest;
                        // (with it, above the lines, how many threads saw too full a bin)
                        uint32_t at = order_scan(sum | (fullest > (uint32_t)ORDER_FULL ? 0x10000u : 0u), sync.red[again ? 0 : 1], lane, wv, all) & 0xFFFFu;
                        full = all >> 16 != 0u;
#pragma unroll
                        for (int j = 0; j < PT; ++j) {
                            words[PT * tid + j] = at | (at + (t[j] & 0xFFFFu)) << 16;
                            at += (t[j] & 0xFFFFu) + (t[j] >> 16);
                        }
                        if (tid == ORDER_THREADS - 1) words[FINE / 2] = at;
                        __syncthreads();
                    }
                    for (int p = tid; p < m; p += ORDER_THREADS) {
                        uint32_t into;
                        const uint32_t f = locate(p, into);
                        spread[meet(f)] = (into & ~PLACE) | (uint32_t)p;
                        bins[p] = (uint16_t)f;
                    }
                    __syncthreads();
                    // a line's place in its bin: the lines of it that go before, four at once.  Their keys are looked at only where they are
                    // as far into it to 18 bits.
                    bool more = false;
                    for (int q = tid; q < m; q += ORDER_THREADS) {
                        const uint32_t self = spread[q], p = self & PLACE, x = bins[p], f = x & PLACE;
                        const uint32_t from = fine[f], to = fine[f + 1];
                        if (x & DONE) { bins[p] = (uint16_t)(from | DONE); continue; }
                        if (__builtin_expect(to - from > (uint32_t)ORDER_FULL && !(x & EQUAL), 0)) {
                            if (!WHOLE || to - from > (uint32_t)ORDER_LAST || (int)to != m) {
                                bins[p] = (uint16_t)from;
                                sync.lines[from / (ORDER_FULL + 1)] = (uint16_t)(to - from);
                                more = true;
                                continue;
                            }
                        }
                        uint32_t at = from;
                        if (to - from > 1u) {
                            uint32_t nearest = 0xFFFFFFFFu;            // least difference, but one, to another line: below PLACE if the 18 bits are the same
                            uint32_t o[4], r = from;
                            auto tally = [&]() {
#pragma unroll
                                for (int e = 0; e < 4; ++e) {
                                    at += o[e] < self ? 1u : 0u;
                                    const uint32_t z = (o[e] ^ self) - 1u;
                                    nearest = z < nearest ? z : nearest;
                                }
                            };
                            for (; r + 4u <= to; r += 4u) {
#pragma unroll
                                for (int e = 0; e < 4; ++e) o[e] = spread[r + e];
                                tally();
                            }
                            if (r < to) {
#pragma unroll
                                for (int e = 0; e < 4; ++e) { const uint32_t y = spread[r + e]; o[e] = r + e < to ? y : self; }
                                tally();
                            }
                            const uint32_t k = keys[p];
                            if (nearest < PLACE && !again && coarse[(k - least) >> sh] >> 16 < tell) {
                                for (r = from; r < to; ++r) {
                                    const uint32_t y = spread[r];
                                    if ((y ^ self) - 1u >= PLACE) continue;
                                    const uint32_t j = keys[y & PLACE];
                                    at += j == k ? 0u : (j < k ? 1u : 0u) - (y < self ? 1u : 0u);
                                }
                            }
                        }
                        if (full) bins[p] = (uint16_t)(at | DONE);
                        put(base + (int)at, line_at((int)p), keys[p]);
                    }
                    if (!full || !__syncthreads_or(more)) break;           // (too full a bin may have been one of equal keys)
                    // Bins with more lines than are ranked against each other: each is spread once more over as many bins as it has
                    // lines (or a few times that), by equal steps from its least key to its largest, or if all its keys are equal, by
                    // place.  (Each time the least and the largest part, so it ends; of equal keys no bin gets many more than the root of
                    // `cap`.)  Such bins begin more than ORDER_FULL places apart, which numbers them.
                    for (int i = tid; i <= FINE / 2; i += ORDER_THREADS) words[i] = 0u;
                    for (int p = tid; p < m; p += ORDER_THREADS) {
                        const uint32_t x = bins[p], s = x / (ORDER_FULL + 1);
                        if (!(x & DONE)) { coarse[s] = keys[p]; coarse[ORDER_SEGS + s] = keys[p]; }
                    }
                    __syncthreads();
                    for (int p = tid; p < m; p += ORDER_THREADS) {
                        const uint32_t x = bins[p], s = x / (ORDER_FULL + 1), k = keys[p];
                        if (!(x & DONE)) {
                            if (k < __atomic_load_n(&coarse[s], __ATOMIC_RELAXED)) atomicMin(&coarse[s], k);
                            if (k > __atomic_load_n(&coarse[ORDER_SEGS + s], __ATOMIC_RELAXED)) atomicMax(&coarse[ORDER_SEGS + s], k);
                        }
                    }
                    __syncthreads();
                }
            }
        }
        base += m;
        if (hi == end) break;
        lo = hi + 1u; hi = end;
    }
    settle();
    if (!WHOLE && a.info) {                                // (the maxima that the range has written: of lines that nobody has put in order nobody takes any unseen)
        const int any = __syncthreads_or(odd);
        say(b, any ? 1 : 0);
    }
    return more;
}
// grid (lists, nb or half as many: workgroup w then takes range w, and the one as many behind it if that is wanted)
// WHOLE: a list in one range.  (Two workgroups a CU where their LDS leaves room for them.)
template <int PT, bool WHOLE, bool LAZY>
__global__ __launch_bounds__(ORDER_THREADS, WHOLE && PT <= 4 ? 8 : 4) void order_kernel(SelectArgs a, int cap) {
    extern __shared__ __align__(16) unsigned char order_lds[];
    __shared__ OrderSync sync;
    const int list = blockIdx.x & 1, bh = blockIdx.x >> 1, nb = a.ranges;
    const float goal = LAZY ? a.alpha * a.total[bh] * ORDER_GOAL : 0.f;
    for (int b = blockIdx.y; b < nb; b += (int)gridDim.y) {
        if (!order_range<PT, WHOLE, LAZY>(a, list, bh, b, nb, b + (int)gridDim.y, cap, goal, order_lds, sync)) break;
        if (WHOLE) break;
        __syncthreads();
    }
}

// ---- running sums in binary32, many additions at a time ------------------------------------------
// s <- fl(s + g[i]) for one i after the other is a chain of dependent additions, 5 cycles each for a wave by itself.
// But while s stays inside one binade, with u the spacing of its numbers and s = m u, what a stretch of additions
// adds to m depends on m only through its parity (to which the ties round).  So each lane runs its stretch of
// entries twice, from an even and an odd m in the middle of the binade, a scan over the lanes composes the pairs of
// increments and gives every lane the exact sum it starts from, and the lane's entries are then added to that.  All of
// it is valid up to the first lane that leaves the binade (itself included: its additions are ordinary ones), or
// whose gains are not small against the sum or negative; the next step goes on behind that lane.  64 entries are added
// the ordinary way where that is the first lane (the first entries of a chain: the sum is not yet large against
// them).  16 entries a lane: 700 cycles a step, 1024 additions one by one 5700.

// increments of a stretch of the chain that starts at an even (e) or odd (o) m
struct ChainInc { int32_t e, o; };
__device__ __forceinline__ ChainInc chain_then(ChainInc a, ChainInc b) {
    return {a.e + ((a.e & 1) ? b.o : b.e), a.o + ((a.o & 1) ? b.e : b.o)};
}
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ ChainInc chain_dpp(ChainInc x) {        // lanes without a source receive the empty stretch
    return {__builtin_amdgcn_update_dpp(0, x.e, CTRL, ROW_MASK, 0xF, false), __builtin_amdgcn_update_dpp(0, x.o, CTRL, ROW_MASK, 0xF, false)};
}
// of the lanes to the left, in order
__device__ __forceinline__ ChainInc chain_before(ChainInc x) {
    if (__ballot(x.e != x.o) == 0ull) {                    // no tie anywhere: plain sums (most stretches of a long chain)
        int32_t s = x.e;
        s += __builtin_amdgcn_update_dpp(0, s, 0x111, 0xF, 0xF, false);
        s += __builtin_amdgcn_update_dpp(0, s, 0x112, 0xF, 0xF, false);
        s += __builtin_amdgcn_update_dpp(0, s, 0x114, 0xF, 0xF, false);
        s += __builtin_amdgcn_update_dpp(0, s, 0x118, 0xF, 0xF, false);
        s += __builtin_amdgcn_update_dpp(0, s, 0x142, 0xA, 0xF, false);
        s += __builtin_amdgcn_update_dpp(0, s, 0x143, 0xC, 0xF, false);
        s -= x.e;
        return {s, s};
    }
    x = chain_then(chain_dpp<0x111, 0xF>(x), x);           // row_shr:1, 2, 4, 8
    x = chain_then(chain_dpp<0x112, 0xF>(x), x);
    x = chain_then(chain_dpp<0x114, 0xF>(x), x);
    x = chain_then(chain_dpp<0x118, 0xF>(x), x);
    x = chain_then(chain_dpp<0x142, 0xA>(x), x);           // row_bcast15 into rows 1 and 3
    x = chain_then(chain_dpp<0x143, 0xC>(x), x);           // row_bcast31 into rows 2 and 3
    return chain_dpp<0x138, 0xF>(x);                       // wave_shr:1
}

// index of the first entry any lane has found, entries in the order entry 0 of lane 0, entry 1 of lane 0, ... (64 E if
// there is none); fe: the first of this lane's E entries (E: none)
template <int E>
__device__ __forceinline__ int first_entry(int fe) {
    const uint64_t any = __ballot(fe < E);
    if (any == 0ull) return 64 * E;
    const int l = __ffsll((unsigned long long)any) - 1;
    return E * l + __builtin_amdgcn_readlane(fe, l);
}
// entry i of the wave's 64 E (i uniform).  The lane's registers are read first and the choice is among scalars: a choice among
// the registers becomes an array in scratch memory, E stores and a load in the chain of every run.  (walk_exact_kernel, which
// waits for that chain, a tenth less; walk_kernel, whose other waves go on meanwhile, 13.2 us both at 12347.)
template <int E>
__device__ __forceinline__ float pick_entry(const float (&v)[E], int i) {
    const int l = i / E;
    int x = __builtin_amdgcn_readlane(__builtin_bit_cast(int, v[0]), l);
#pragma unroll
    for (int e = 1; e < E; ++e) {
        const int y = __builtin_amdgcn_readlane(__builtin_bit_cast(int, v[e]), l);
        x = (i % E) == e ? y : x;
    }
    return __builtin_bit_cast(float, x);
}

// Lane l holds the gains of the entries E l .. E l + E - 1.  x[e] = the sum behind entry e, starting from `sum` ahead of
// lane `first`; valid in the lanes from `first` to the one returned.
// SIGNED: gains may be a little less than 0 (differences of sums that are the same but for their rounding); the sum then has to stay in the binade all the way.
template <int E, bool SIGNED = false>
__device__ __forceinline__ int chain_step(const float (&g)[E], int lane, int first, float sum, bool plain, float (&x)[E]) {
    const uint32_t sb = __builtin_bit_cast(uint32_t, sum), binade = sb & 0x7F800000u;
    if (plain || sb < (64u << 23) || sb > (250u << 23)) {  // (the first sum is 0, and gains may be negative in the end)
#pragma unroll
        for (int e = 0; e < E; ++e) x[e] = 0.f;
        for (int p = 0; p < 64 / E; ++p) {                 // pass p settles lane first + p
            float left = __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x[E - 1]), 0x138 /* wave_shr:1 */, 0xF, 0xF, true));
            left = lane == first ? sum : left;
            x[0] = __fadd_rn(left, g[0]);
#pragma unroll
            for (int e = 1; e < E; ++e) x[e] = __fadd_rn(x[e - 1], g[e]);
        }
        return first + 64 / E < 64 ? first + 64 / E - 1 : 63;
    }
    const uint32_t even = binade | 0x400000u;              // 1.5 times the binade's first number, and the next one
    float xe = __builtin_bit_cast(float, even), xo = __builtin_bit_cast(float, even + 1u), least = g[0];
#pragma unroll
    for (int e = 0; e < E; ++e) { xe = __fadd_rn(xe, g[e]); xo = __fadd_rn(xo, g[e]); least = fminf(least, g[e]); }
    const bool idle = lane < first;
    bool small = xo < __builtin_bit_cast(float, binade + 0x800000u) && least >= 0.f;
    int32_t low = 0, high = 0;                             // how far below the start the stretch gets, and above it
    if constexpr (SIGNED) {
        if (__ballot(!idle && !(least >= 0.f)) != 0ull) {
            float y = __builtin_bit_cast(float, even), lo = y, hi = y;
#pragma unroll
            for (int e = 0; e < E; ++e) { y = __fadd_rn(y, g[e]); lo = fminf(lo, y); hi = fmaxf(hi, y); }
            small = hi < __builtin_bit_cast(float, binade + 0x7FFFFEu) && lo >= __builtin_bit_cast(float, binade + 2u);      // (a NaN is neither: an ordinary step)
            low = (int32_t)(__builtin_bit_cast(uint32_t, lo) - even) - 2; high = (int32_t)(__builtin_bit_cast(uint32_t, hi) - even) + 2;      // (from an odd start a step more at most)
        }
    }
    ChainInc inc = {0, 0};
    if (small && !idle) inc = {(int32_t)(__builtin_bit_cast(uint32_t, xe) - even), (int32_t)(__builtin_bit_cast(uint32_t, xo) - (even + 1u))};
    const ChainInc before = chain_before(inc);
    const int32_t m0 = (int32_t)(sb & 0x7FFFFFu);
    const int32_t m = m0 + ((m0 & 1) ? before.o : before.e);               // less 2^23
    const uint64_t leave = __ballot(!idle && (!small || m + ((m & 1) ? inc.o : inc.e) >= 1 << 23 || (SIGNED && (m + low < 0 || m + high >= 1 << 23))));
    x[0] = __fadd_rn(__builtin_bit_cast(float, binade | ((uint32_t)m & 0x7FFFFFu)), g[0]);
#pragma unroll
    for (int e = 1; e < E; ++e) x[e] = __fadd_rn(x[e - 1], g[e]);
    return leave != 0ull ? __ffsll((unsigned long long)leave) - 1 : 63;
}
// All entries added to `sum` in one step, if it then stays in its binade and below `target` (no gain is negative, so that it was below it all the way):
// the scan alone says so, without the lanes' own sums.  False, and nothing done, where it might not.
// POSITIVE: every gain is known to be above 0.
template <int E, bool POSITIVE = false>
__device__ __forceinline__ bool chain_all(const float (&g)[E], float target, float& sum) {
    const uint32_t sb = __builtin_bit_cast(uint32_t, sum), binade = sb & 0x7F800000u;
    if (sb < (64u << 23) || sb > (250u << 23)) return false;
    const uint32_t even = binade | 0x400000u;
    float xe = __builtin_bit_cast(float, even), xo = __builtin_bit_cast(float, even + 1u), least = g[0];
#pragma unroll
    for (int e = 0; e < E; ++e) { xe = __fadd_rn(xe, g[e]); xo = __fadd_rn(xo, g[e]); if (!POSITIVE) least = fminf(least, g[e]); }
    // (a NaN leaves xo a NaN)
    if (__ballot(!(xo < __builtin_bit_cast(float, binade + 0x800000u) && (POSITIVE || least >= 0.f))) != 0ull) return false;
    const ChainInc inc = {(int32_t)(__builtin_bit_cast(uint32_t, xe) - even), (int32_t)(__builtin_bit_cast(uint32_t, xo) - (even + 1u))};
    const ChainInc all = chain_then(chain_before(inc), inc);       // of lane 63: 63 lanes of less than 2^22 each
    const int32_t m0 = (int32_t)(sb & 0x7FFFFFu);
    const int32_t m = m0 + __builtin_amdgcn_readlane((m0 & 1) ? all.o : all.e, 63);
    const float x = __builtin_bit_cast(float, binade | (uint32_t)m);
    if (m >= 1 << 23 || !(x < target)) return false;
    sum = x;
    return true;
}
// Adds entries 0 .. `limit` - 1 (the gains are 0 from there on) to `sum`, which is below `target`, in order until it
// reaches the target or they are used up; returns how many were added.
template <int E, bool SIGNED = false>
__device__ __forceinline__ int chain_until(const float (&g)[E], int lane, int limit, float target, float& sum) {
    if (limit == 0) return 0;
    int first = 0;
    bool plain = false;
    for (;;) {
        float x[E];
        const int last = chain_step<E, SIGNED>(g, lane, first, sum, plain, x);
        int fe = E;
#pragma unroll
        for (int e = E - 1; e >= 0; --e) fe = x[e] < target ? fe : e;
        const int j = first_entry<E>(lane >= first && lane <= last ? fe : E);
        if (j < limit) { sum = pick_entry(x, j); return j + 1; }
        const bool end = E * (last + 1) >= limit;          // (the entries behind `limit` add 0)
        sum = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, x[E - 1]), end ? (limit - 1) / E : last));
        if (end) return limit;
        plain = !plain && last == first;
        first = last + 1;
    }
}
// Writes pre[i] = acc + (the entries before entry i, added left to right in binary32) for the 64 E entries, and returns
// the sum behind the last one.  The first `again_end` of them (whole lanes) go to `again` as well.  E is even.
template <int E>
__device__ __forceinline__ float chain_prefix(const float (&g)[E], int lane, float acc, float* pre, float* again, int again_end) {
    float x[E];                                            // the sum behind each entry
    float sum = acc;
    int first = 0;
    bool plain = false;
    while (first < 64) {
        float y[E];
        const int last = chain_step<E>(g, lane, first, sum, plain, y);
#pragma unroll
        for (int e = 0; e < E; ++e) x[e] = lane >= first ? y[e] : x[e];    // (behind `last` it is written again)
        sum = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, y[E - 1]), last));
        plain = !plain && last == first;
        first = last + 1;
    }
    const float left = __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x[E - 1]), 0x138 /* wave_shr:1 */, 0xF, 0xF, true));
    auto put = [&](float* p) {
        float2* dst = reinterpret_cast<float2*>(p + E * lane);
        dst[0] = make_float2(lane == 0 ? acc : left, x[0]);
#pragma unroll
        for (int e = 2; e < E; e += 2) dst[e / 2] = make_float2(x[e - 1], x[e]);
    };
    put(pre);
    if (E * lane < again_end) put(again);
    return sum;
}
// The same for up to CHAIN_FEW entries, an entry a lane, one after the other: 400 cycles, a step of the scan 900
constexpr int CHAIN_FEW = 16;
__device__ __forceinline__ int chain_few(float g, int lane, int limit, float target, float& sum) {
    if (limit == 0) return 0;
    float x = 0.f;
#pragma unroll
    for (int p = 0; p < CHAIN_FEW; ++p) {                   // pass p settles lane p
        float left = __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x138 /* wave_shr:1 */, 0xF, 0xF, true));
        left = lane == 0 ? sum : left;
        x = __fadd_rn(left, g);
    }
    const uint64_t reached = __ballot(lane < limit && !(x < target));
    const int last = reached != 0ull ? __ffsll((unsigned long long)reached) - 1 : limit - 1;
    sum = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, x), last));
    return last + 1;
}
// the same with the gains in LDS (64 E floats, 16-byte aligned)
template <int E>
__device__ __forceinline__ int chain_lds(const float* gains, int lane, int limit, float target, float& sum) {
    float g[E];
#pragma unroll
    for (int e = 0; e < E; ++e) { g[e] = gains[E * lane + e]; g[e] = E * lane + e < limit ? g[e] : 0.f; }
    return chain_until<E, true>(g, lane, limit, target, sum);
}

// ---- the greedy loop ----------------------------------------------------------------------------
// One workgroup of six waves per head.  The loop of Alg. 2 is sequential, but three things about it are not:
//   * ol_s after k slashes were taken is the left-to-right binary32 sum of the first k maxima of
//     the slash list, whatever the interleaving with verticals was (likewise ol_v), so both
//     running overlaps are prefix arrays that can be filled ahead of the walk (still added one
//     element after the other, so every value is the one the sequential loop would hold);
//   * while the walk keeps taking from one list, the state of the other list is frozen, so the
//     next 64 ratio tests can be evaluated by the 64 lanes at once; a ballot gives the length of
//     the run of equal decisions.
//   * which list the next pick comes from does not depend on `sum`; only the end of the walk does.  So the
//     decisions can run ahead of the sum: they are handed over run by run (the gain of every pick, in pick
//     order) through a small ring in LDS, and whatever was decided beyond the pick that reaches the target
//     is dropped.
// What stays sequential are two chains of binary32 additions, one add per line each: the overlap prefix sums
// and `sum` with its exit test after every pick.  Both are evaluated by the integer scan above, whose values are the
// ones the sequential loop would hold: each pick sees exactly the operands, operation order and roundings of the
// definition.
constexpr int WALK_THREADS = 384;              // wave 0 decides the runs, wave 2 sums them; per list, waves 1 / 3 stage its
                                               // weights and lengths and waves 4 / 5 its overlap prefix sums
// A lane looks at E list entries: a run has up to 64 E picks.  Short lists have short runs, long ones long: 4 / 8 / 16, ls_select of
// 32 heads, us: 2048 lines 22.0 / 23.1 / 24.3, 4096 24.2 / 24.0 / 25.3, 12347 34.9 / 35.5 / 36.4, 16384 56.2 / 49.3 / 45.7, 32768 76.8 / 67.2 / 63.1,
// 65536 157 / 137 / 128; 256 heads of 1500 lines 27.5 / 29.0 / 29.9.
constexpr int64_t WALK_SHORT = 2048, WALK_LONG = 8192;         // up to: 4; from: 16
// (With long runs taken unseen, below, sixteen pay from 8192 lines on: 8 / 16, the walk alone, 8192 lines 15.9 / 13.8, 5003 12.2 / 13.5.)
// Where the picks go back and forth between the lists a run is one or a few, and its price is that of looking at all E entries.
// The deciding wave then looks at these few only, from the beginning and from three runs in a row of up to half of what they hold until one fills them.  (From one such run, where the runs of
// one list are long and those of the other short: 32 heads of 32768 lines by the thousand picks 3743 / 3653 us, 64 of 8192 1208 / 1178, 32 of 12000 427 / 418, the whole ls_select.)  The walk alone
// with sixteen throughout / so, 32 heads of 32768 lines, us: runs of one to five picks 76.5 / 54.7, of one 489 / 320.
constexpr int WALK_NARROW = 4;
constexpr int WALK_NBLK = 4;                   // blocks of a list resident in LDS (a ring over sorted positions)
constexpr int WALK_CAP = WALK_BLK * WALK_NBLK;
constexpr int WALK_EB = WALK_BLK / 64;         // entries per lane when a block's prefix sums are added
static_assert(WALK_EB % 2 == 0 && 64 * 16 <= WALK_BLK, "a run never reaches beyond the block after the head's");

// The resident part of one sorted list, indexed by sorted position modulo WALK_CAP: weights, line lengths, and
// pre[p] = the overlap sum when the first p lines of the list have been taken.  The first 64 E entries are
// there a second time behind the last one, so that a run's entries are consecutive wherever it starts.
template <int E> struct WalkList { float cw[WALK_CAP + 64 * E], cl[WALK_CAP + 64 * E], pre[WALK_CAP + 64 * E]; };
// One run of picks from one list: the gain of each pick, how many of them count, and whether the walk ends
// after them because no line is left that adds anything.
template <int E> struct WalkRun {
    float g[72 * E];                                       // pick p at p + 2 (p / 16): lanes that read 4, 8 or 16 picks each meet all banks
    int which, limit, last, pad;                           // (read as one)
};
// What the lanes need of a list when its head is at `h`: lane l looks at the entries h + l, h + 64 + l, ... (weight,
// overlap prefix, length; whatever lies there past the end of the list), every lane at the head's own three values.
// Re-read only when the head of that list moves.  (All of them lie in the head's block or the one after it.)
template <int N> struct WalkView { float cw[N], pre[N], cl[N], w0, l0, ol0; };
struct WalkSync { int staged[2], summed_blk[2], cur[2], summed, stop, done, err, runs, decided, cnt_s, cnt_v, falls[2], need[2], cut, open; float tot[2]; };      // falls: a list's prefix sums do not rise throughout; need: blocks whose prefix sums are wanted; cut: a list is wanted further than it is in order; open: and the sum had not reached the target
static_assert(offsetof(WalkSync, summed) % 8 == 0 && offsetof(WalkSync, stop) == offsetof(WalkSync, summed) + 4, "summed and stop are read as one 8-byte word");   // tot: a list's whole overlap sum
constexpr int RUN_WHOLE = 2;                   // a run's `last`: it has all its picks, and every gain is above 0
constexpr int WALK_RING = 4;                   // runs decided ahead of the running sum
template <int E> constexpr size_t WALK_LDS_BYTES = 2 * sizeof(WalkList<E>) + WALK_RING * sizeof(WalkRun<E>) + sizeof(WalkSync);

__device__ __forceinline__ int walk_ld(const int* p) { return __builtin_amdgcn_readfirstlane(__atomic_load_n(p, __ATOMIC_RELAXED)); }
__device__ __forceinline__ void walk_st(int* p, int v) { __atomic_store_n(p, v, __ATOMIC_RELAXED); }

// The lines of a bitmap of up to 1024 words, ascending: line0 + bit goes to out[at + how many are before it] while that is below `cap`.  NT
// threads from t = 0 on call, whole waves, of which wave wv0 is the first (of a workgroup whose other threads do the same for another map of as many
// words); returns the number of lines.  stage: 32 * words numbers of LDS.  wsum: a word for each wave, not in use.
//
// A thread takes a word, several, or down to a quarter of one, whichever gives all of them something to do, and puts its lines into LDS: they go out
// in whole lines of memory.  (Straight from the words each store instruction met up to 64 lines of memory: emit_kernel, 32 heads of 32768 lines
// 9.5 -> 6.9 us, 12347 5.6 -> 4.6; merge_lines_kernel, 16 heads of 5003 lines, 10.5 -> 8.2; the walk of 1024 lines, which does it itself, 11.2 -> 9.3.)
template <int NT>
__device__ __forceinline__ uint32_t put_lines(const uint32_t* bm, int words, int line0, uint16_t* stage, uint32_t* wsum, int wv0, int32_t* out, uint32_t at, int cap, int t) {
    const int lane = t & 63, wv = wv0 + __builtin_amdgcn_readfirstlane(t >> 6);
    const int sh = 4 * words <= NT ? 2 : 2 * words <= NT ? 1 : 0, units = words << sh, bits = 32 >> sh;
    const int per = (units + NT - 1) / NT, u0 = t * per < units ? t * per : units, u1 = u0 + per < units ? u0 + per : units;
    auto unit = [&](int u) -> uint32_t { const uint32_t w = bm[u >> sh]; return sh == 0 ? w : (w >> ((u & ((1 << sh) - 1)) * bits)) & ((1u << bits) - 1u); };
    uint32_t mine = 0u;
    for (int u = u0; u < u1; ++u) mine += (uint32_t)__popc(unit(u));
    const uint32_t upto = lanes_upto(mine);
    if (lane == 63) wsum[wv] = upto;
    __syncthreads();
    uint32_t p = upto - mine, all = 0u;
    for (int w = 0; w < NT / 64; ++w) { const uint32_t x = wsum[wv0 + w]; p += wv0 + w < wv ? x : 0u; all += x; }
    for (int u = u0; u < u1; ++u)
        for (uint32_t m = unit(u); m; m &= m - 1u) stage[p++] = (uint16_t)(u * bits + __ffs(m) - 1);
    __syncthreads();
    const uint32_t room = at < (uint32_t)cap ? (uint32_t)cap - at : 0u, go = all < room ? all : room;
    for (uint32_t i = (uint32_t)t; i < go; i += NT) out[at + i] = line0 + (int32_t)stage[i];
    return all;
}
constexpr int PUT_WORDS = 1024;
constexpr size_t put_lines_bytes(int64_t n) { return (size_t)(n < 32 * PUT_WORDS ? (n + 31) / 32 * 32 : 32 * PUT_WORDS) * 2; }

// Chosen prefixes -> ascending index lists of both lists of a head, by the workgroup that has walked them (half of its NT
// threads a list).  bm: 2 * ceil(n / 32) words of LDS and 2 * put_lines_bytes(n) behind them.  Up to EMIT_LINES lines; beyond, the 192 threads a list (walk_kernel; walk_exact_kernel
// 512) take longer than emit_kernel's 1024 and its launch.  ls_select, 32 heads, launch / here, us: 1024 lines 17.1 / 16.1, 4096 24.7 / 24.7, 8192
// 33.5 / 34.8, 12288 39.4 / 41.2, 16384 42.1 / 45.0; 256 heads of 1500 27.0 / 24.7; with exact overlaps (six seeds in turn; the walk differs more from seed to seed) 1024 69.8 / 69.3,
// 4097 87.2 / 88.8, 6000 106.8 / 108.1, 64 heads 108.5 / 109.2, 8192 80.0 / 80.1, 64 heads 130.3 / 131.1.
constexpr int64_t EMIT_LINES = 4096;
template <int NT>
__device__ __forceinline__ void emit_both(const SelectArgs& a, int bh, int cnt_s, int cnt_v, uint32_t* bm) {
    __shared__ uint32_t wsum[NT / 64];
    constexpr int H = NT / 2;
    const int tid = threadIdx.x, list = tid >= H ? 1 : 0, t = tid - list * H;
    const int n = (int)a.n, words = (n + 31) / 32, cnt = list == 0 ? cnt_s : cnt_v, cap = list == 0 ? a.cap_s : a.cap_v;
    const int32_t* sorted_idx = a.sidx + ((int64_t)list * a.BH + bh) * n;
    int32_t* out = list == 0 ? a.s_idx + (int64_t)bh * cap : a.v_idx + (int64_t)bh * cap;
    bm += list * words;
    for (int i = t; i < words; i += H) bm[i] = cnt >= n ? 0xFFFFFFFFu >> (i == words - 1 ? 32 * words - n : 0) : 0u;
    if (t == 0 && cnt > cap) atomicOr(a.status, list == 0 ? STAT_S_TRUNCATED : STAT_V_TRUNCATED);
    __syncthreads();
    if (cnt < n)
        for (int i0 = t; i0 < cnt; i0 += 8 * H) {          // eight independent loads in flight per thread
            int32_t x8[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) x8[j] = sorted_idx[i0 + j * H < cnt ? i0 + j * H : cnt - 1];
#pragma unroll
            for (int j = 0; j < 8; ++j) atomicOr(&bm[x8[j] >> 5], 1u << (x8[j] & 31));
        }
    __syncthreads();
    put_lines<H>(bm, words, 0, reinterpret_cast<uint16_t*>(bm + (2 - list) * words) + list * 32 * words, wsum, list * (H / 64), out, 0u, cap, t);
}

// ix[e] = the line at sorted position pos + e (the last line's index past the end of the list)
template <int E>
__device__ __forceinline__ void walk_indices(const int32_t* i_l, int pos, int n, int32_t (&ix)[E]) {
    typedef __attribute__((ext_vector_type(4))) int32_t i32x4;
    // (a wave-uniform choice: the list starts on a 16-byte boundary and the wave's last entry is inside it)
    const bool whole = (reinterpret_cast<uintptr_t>(i_l) & 15) == 0 && (pos & 3) == 0 &&
                       __builtin_amdgcn_readfirstlane(pos) + 64 * E <= n;
    if (E % 4 == 0 && whole) {
#pragma unroll
        for (int e = 0; e < E; e += 4) {
            const i32x4 v = *reinterpret_cast<const i32x4*>(i_l + pos + e);
            ix[e] = v.x; ix[e + 1] = v.y; ix[e + 2] = v.z; ix[e + 3] = v.w;
        }
    } else {
#pragma unroll
        for (int e = 0; e < E; ++e) { const int i = pos + e; ix[e] = i_l[i < n ? i : n - 1]; }
    }
}
// m[e] = the largest entry of line ix[e], the line at sorted position pos + e (0 past the end of the list)
template <int E>
__device__ __forceinline__ void walk_maxima(const float* m_l, const int32_t (&ix)[E], int pos, int n, float (&m)[E]) {
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const float t = m_l[ix[e]];
        m[e] = pos + e < n ? t : 0.f;
    }
}

// Position of the first entry for which `p` holds, in the order entry 0 of lane 0, entry 0 of lane 1, ..., entry 1 of
// lane 0, ... (64 E if it holds nowhere)
template <int E>
__device__ __forceinline__ int walk_first(const bool (&p)[E]) {
    int at = 64 * E;
#pragma unroll
    for (int e = E - 1; e >= 0; --e) {
        const uint64_t any = __ballot(p[e]);
        at = any != 0ull ? 64 * e + __ffsll((unsigned long long)any) - 1 : at;
    }
    return at;
}

// grid (BH).  Reads the sorted lists (weights, maxima, indices) and writes taken counts.
//
// The waves share only LDS.  Each list is staged in blocks of WALK_BLK sorted positions into a ring of WALK_NBLK
// blocks: waves 1 / 3 write the weights and line lengths of a block (staged[l] = blocks written), waves 4 / 5
// its overlap prefix sums (summed_blk[l]), 2700 cycles a block and only of blocks that the deciding wave has asked for (need[l]); both load the next
// two blocks while they work on the current one.  Block b may be written once the deciding wave's head of that list
// has reached block b - WALK_NBLK + 1 (cur[l] = the head's block): nothing before the head is read again.  The
// deciding wave (0) needs the head's block and the one after it; it publishes cur[l] and runs = the number of
// runs it has put into the ring of runs; the summing wave (2) publishes summed = the number of runs it has
// taken out, and stop when the walk is over.  The summing wave writes the result; the deciding wave ends the
// stagers through `done`.  Every wait is a bounded spin that also ends when another wave has reported a failed
// wait, so all six waves leave in every case.
// Most walks are one run from one list to the target (32 heads of 32768 lines: 29 of them, 96 to 9071 picks).  Once the other list's head adds nothing any more, 1024 picks need no look
// at each, nor their overlap prefix sums (quick, below: 1300 cycles, looked at 3900), and their sum comes from the scan alone (chain_all: 1500, from 2500).
// SORTED: the lists' weights and maxima lie in order; otherwise only those of the first block do.
template <int E, bool SORTED>
__device__ __forceinline__ void walk_head(const SelectArgs& a, const int bh, unsigned char* walk_lds) {
    using List = WalkList<E>;
    using Run = WalkRun<E>;
    constexpr int RUN = 64 * E;
    List* lists = reinterpret_cast<List*>(walk_lds);
    Run* ring = reinterpret_cast<Run*>(walk_lds + 2 * sizeof(List));
    WalkSync* sync = reinterpret_cast<WalkSync*>(walk_lds + 2 * sizeof(List) + WALK_RING * sizeof(Run));
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = (int)a.n;
    const int nblk = (n + WALK_BLK - 1) / WALK_BLK;
    // order_kernel has looked at the maxima (not of lists that are one range); it may have left ranges out (not of shorter lists, and not any more where a head is walked again)
    static_assert(WALK_SHORT <= ORDER_ONE && LAZY_LINES > WALK_LONG, "lists that are walked four entries a lane are one range, those that lack ranges are walked by sixteen");
    const bool informed = SORTED && E > 4 && a.info != nullptr;
    constexpr bool SOME = SORTED && E == 16;
    // how far list l is in order, and (odd) whether a maximum of the lines up to there is negative or no number
    auto reach = [&](int l, int* odd) {
        const int64_t of = ((int64_t)l * a.BH + bh) * SELECT_RANGES;
        int p = 0, q = 0, far = n;
        if (informed) { p = lane < a.ranges ? a.info[of + lane] : 0; q = lane + 64 < a.ranges ? a.info[of + lane + 64] : 0; }
        if (SOME && a.open) {
            const int at = p < 0 ? -1 - p : n, at2 = q < 0 ? -1 - q : n;
            far = __builtin_amdgcn_readlane((int)lanes_min((uint32_t)(at < at2 ? at : at2)), 63);
        }
        if (odd) *odd = __ballot(p > 0 || q > 0) != 0ull ? 1 : 0;
        return far;
    };
    const int64_t nh = a.n_hat;
    const int spin_limit = a.spin_limit;       // bound of every wait between the waves
    const int64_t seg_s = ((int64_t)0 * a.BH + bh) * a.n, seg_v = ((int64_t)1 * a.BH + bh) * a.n;

    if (threadIdx.x == 0) {
        sync->staged[0] = sync->staged[1] = 0; sync->summed_blk[0] = sync->summed_blk[1] = 0;
        sync->cur[0] = sync->cur[1] = 0; sync->done = 0; sync->err = 0;
        sync->runs = 0; sync->summed = 0; sync->decided = 0; sync->stop = 0; sync->falls[0] = sync->falls[1] = 0; sync->need[0] = sync->need[1] = 2; sync->cut = 0;
    }
    // (every wave comes to one barrier here, the stagers once their first loads are under way)
    // Its blocks by `even` and `odd` in turn, as the ring has room for them; `ready`: how many are there.  (In straight code: what one has
    // asked for is still under way when the other waits for its own.)
    int far = n;                               // a stager's list is in order up to there
    auto stage_blocks = [&](const int* cur, const int* need, int* ready, auto even, auto odd) {
        int b = 0, spins = 0;
        const int blocks = (far + WALK_BLK - 1) / WALK_BLK;
        auto room = [&]() {
            for (;;) {
                if (b >= blocks || walk_ld(&sync->done) != 0) return false;
                if (b <= walk_ld(cur) + WALK_NBLK - 1 && (!need || b < walk_ld(need))) break;
                __builtin_amdgcn_s_sleep(2);
                if (++spins > spin_limit) { walk_st(&sync->err, 1); return false; }
            }
            spins = 0;
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
            return true;
        };
        auto publish = [&]() {
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
            __builtin_amdgcn_wave_barrier();
            ++b;
            if (lane == 0) walk_st(ready, b);
        };
        while (room()) {
            even(b);
            publish();
            if (!room()) break;
            odd(b);
            publish();
        }
    };
    if (wv == 1 || wv == 3) {
        // ------------------------------------------------------------------ weights and lengths of one list
        const int l = wv == 1 ? 0 : 1;
        List& L = lists[l];
        const int64_t seg = l == 0 ? seg_s : seg_v;
        const float* w_l = (l == 0 ? a.slash : a.vert) + (int64_t)bh * a.n;   // weights by line index
        const float* sw = a.sorted_w + ((int64_t)l * a.BH + bh) * a.kept;     // ... in order
        const int32_t* i_l = a.sidx + seg;
        const int nh32 = (int)nh;
        constexpr int PER = WALK_BLK / 64;
        // (What lies behind the list is read as well, inside the workspace, and nothing made of it.  One address for a block's loads:
        // with a look at each entry's place a wave had 2 KB of code to fetch before its first one was asked for.)
        struct Block { float w[PER]; int32_t x[PER]; };
        auto fetch_idx = [&](int b, int32_t (&x)[PER]) {
            if (b >= nblk) return;
            const int32_t* at = i_l + b * WALK_BLK + lane;
#pragma unroll
            for (int j = 0; j < PER; ++j) x[j] = at[j * 64];
        };
        auto fetch_sorted = [&](int b, Block& f) {
            if (b >= nblk) return;
            const float* at = sw + b * WALK_BLK + lane;
#pragma unroll
            for (int j = 0; j < PER; ++j) f.w[j] = at[j * 64];
            fetch_idx(b, f.x);
        };
        auto write = [&](int b, const Block& f) {
            const int slot = (b & (WALK_NBLK - 1)) * WALK_BLK;
            float *cw = L.cw + slot + lane, *cl = L.cl + slot + lane;
            auto length = [&](int x) { return (float)(n - x < nh32 ? n - x : nh32); };     // line length in the n_hat x n block
            auto put = [&](auto WHOLE, int to) {
#pragma unroll
                for (int j = 0; j < (decltype(WHOLE)::value == 2 ? E : PER); ++j) {
                    const bool in = decltype(WHOLE)::value == 1 || b * WALK_BLK + lane + j * 64 < n;
                    cw[to + j * 64] = in ? f.w[j] : 0.f;
                    cl[to + j * 64] = in ? length(f.x[j]) : 1.f;
                }
            };
            if ((b + 1) * WALK_BLK <= n) put(std::integral_constant<int, 1>{}, 0); else put(std::integral_constant<int, 0>{}, 0);
            if (slot == 0) put(std::integral_constant<int, 2>{}, WALK_CAP);       // the first entries once more
        };
        if constexpr (SORTED) {                            // two blocks under way, in turn
            Block even, odd;
            fetch_sorted(0, even);
            fetch_sorted(1, odd);
            far = reach(l, nullptr);
            __syncthreads();
            stage_blocks(&sync->cur[l], nullptr, &sync->staged[l], [&](int b) { write(b, even); fetch_sorted(b + 2, even); }, [&](int b) { write(b, odd); fetch_sorted(b + 2, odd); });
        } else {
            // the block after the last one written to LDS (indices and weights), and the indices of the one after it:
            // the weights are fetched through the indices, so the indices are requested a block earlier
            Block f;
            int32_t next[PER];
            fetch_sorted(0, f);                            // (its weights are there in order)
            fetch_idx(1, next);
            __syncthreads();
            auto block = [&](int b) {
                write(b, f);
#pragma unroll
                for (int j = 0; j < PER; ++j) { f.x[j] = next[j]; f.w[j] = (b + 1) * WALK_BLK + lane + j * 64 < n ? w_l[f.x[j]] : 0.f; }
                fetch_idx(b + 2, next);
            };
            stage_blocks(&sync->cur[l], nullptr, &sync->staged[l], block, block);
        }
        return;
    }

    if (wv == 4 || wv == 5) {
        // ------------------------------------------------------------------ overlap prefix sums of one list
        // (one addition after the other took 5700 cycles a block)
        const int l = wv - 4;
        List& L = lists[l];
        const int32_t* i_l = a.sidx + (l == 0 ? seg_s : seg_v);
        const float* m_l = (l == 0 ? a.smax : a.vmax) + (int64_t)bh * a.n;     // maxima by line index
        const float* sm = a.sorted_m + ((int64_t)l * a.BH + bh) * a.kept;      // ... in order
        struct Block { float m[WALK_EB]; };
        float acc = 0.f;                       // overlap sum behind the last entry summed so far
        auto add = [&](int b, const Block& f) {
            acc = chain_prefix<WALK_EB>(f.m, lane, acc, L.pre + (b & (WALK_NBLK - 1)) * WALK_BLK, L.pre + WALK_CAP, (b & (WALK_NBLK - 1)) == 0 ? RUN : 0);
            if (!informed) {                               // (else order_kernel has said so)
                bool odd = false;
#pragma unroll
                for (int e = 0; e < WALK_EB; ++e) odd = odd || !(f.m[e] >= 0.f);
                if (__ballot(odd) != 0ull && lane == 0) walk_st(&sync->falls[l], 1);
            }
            if (b == nblk - 1 && lane == 0) sync->tot[l] = acc;
        };
        typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
        auto fetch_sorted = [&](int b, Block& f) {         // (past the end of the list, as above)
            if (b >= nblk) return;
            const float* at = sm + b * WALK_BLK + WALK_EB * lane;
#pragma unroll
            for (int e = 0; e < WALK_EB; e += 4) {
                const f32x4u v = *reinterpret_cast<const f32x4u*>(at + e);
                f.m[e] = v.x; f.m[e + 1] = v.y; f.m[e + 2] = v.z; f.m[e + 3] = v.w;
            }
        };
        auto ends = [&](int b, Block& f) {                 // the list ends in this block
            if ((b + 1) * WALK_BLK <= n) return;
#pragma unroll
            for (int e = 0; e < WALK_EB; ++e) f.m[e] = b * WALK_BLK + WALK_EB * lane + e < n ? f.m[e] : 0.f;
        };
        if constexpr (SORTED) {
            Block even, odd;
            fetch_sorted(0, even);
            fetch_sorted(1, odd);
            far = reach(l, nullptr);
            __syncthreads();
            stage_blocks(&sync->cur[l], &sync->need[l], &sync->summed_blk[l], [&](int b) { ends(b, even); add(b, even); fetch_sorted(b + 2, even); }, [&](int b) { ends(b, odd); add(b, odd); fetch_sorted(b + 2, odd); });
        } else {
            Block f, g;
            int32_t ix[WALK_EB];               // line indices of the block after the next one's maxima
            fetch_sorted(0, f);
            ends(0, f);
            walk_indices<WALK_EB>(i_l, WALK_BLK + WALK_EB * lane, n, ix);
            __syncthreads();
            auto block = [&](int b) {
                walk_maxima<WALK_EB>(m_l, ix, (b + 1) * WALK_BLK + WALK_EB * lane, n, g.m);
                walk_indices<WALK_EB>(i_l, (b + 2) * WALK_BLK + WALK_EB * lane, n, ix);
                add(b, f);
                f = g;
            };
            stage_blocks(&sync->cur[l], &sync->need[l], &sync->summed_blk[l], block, block);
        }
        return;
    }

    if (wv == 2) {
        // ------------------------------------------------------------------ the running sum
        // Takes the runs in the order they were decided and adds their gains pick by pick; the first pick whose
        // sum reaches the target ends the walk.
        const float target = a.alpha * a.total[bh];
        float sum = 0.f;
        int cnt_s = 0, cnt_v = 0;              // lines taken from each list
        __syncthreads();
        int k = 0;                             // runs summed
        bool failed = false, all = false, open = false;
        while (sum < target) {
            bool have = false;
            int spins = 0;
            for (;;) {
                if (walk_ld(&sync->runs) > k) { have = true; break; }
                if (walk_ld(&sync->decided)) {                       // stored after the last run was published
                    have = walk_ld(&sync->runs) > k;
                    failed = !have && walk_ld(&sync->err) != 0;
                    open = !have && walk_ld(&sync->cut) != 0;
                    break;
                }
                if (++spins > spin_limit || walk_ld(&sync->err)) { failed = true; break; }
                __builtin_amdgcn_s_sleep(1);
            }
            if (!have) break;                  // both lists were used up (or a wait ran into its bound)
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
            const Run& R = ring[k & (WALK_RING - 1)];
            const int4 about = *reinterpret_cast<const int4*>(&R.which);
            const int which = __builtin_amdgcn_readfirstlane(about.x), limit = __builtin_amdgcn_readfirstlane(about.y), last = __builtin_amdgcn_readfirstlane(about.z);
            // pick by pick, as the loop of the definition adds them; it stops after the pick that reaches the target
            // (one addition after the other took 3900 cycles a run)
            int taken = 0;
            auto add = [&](auto ENTRIES) {
                constexpr int N = decltype(ENTRIES)::value;
                float g[N];
                const float* at = &R.g[N * lane + 2 * (N * lane / 16)];
#pragma unroll
                for (int e = 0; e < N; e += 2) {
                    const float2 t = *reinterpret_cast<const float2*>(at + e);
                    g[e] = t.x; g[e + 1] = t.y;
                }
                if (N != E || last != RUN_WHOLE) {
#pragma unroll
                    for (int e = 0; e < N; ++e) g[e] = N * lane + e < limit ? g[e] : 0.f;
                }
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");         // the slot may be written again
                ++k;
                if (lane == 0) walk_st(&sync->summed, k);
                if (N == E && last == RUN_WHOLE && chain_all<N, true>(g, target, sum)) taken = limit;
                else taken = chain_until<N>(g, lane, limit, target, sum);
            };
            if (E > WALK_NARROW && limit <= 64 * WALK_NARROW) add(std::integral_constant<int, WALK_NARROW>{}); else add(std::integral_constant<int, E>{});
            const bool reached = !(sum < target);
            cnt_s += which == 0 ? taken : 0;
            cnt_v += which == 0 ? 0 : taken;
            if (!reached && last == 1) { all = true; break; }  // the pick after the last one has no positive gain
        }
        if (lane == 0) {
            walk_st(&sync->stop, 1);
            if (failed) walk_st(&sync->err, 1);
            // A wait that ran into its bound (never observed with the default bound) reports the conservative
            // result, every line selected: the coverage target of Alg. 2 still holds for it, and the context's
            // status word tells the caller.
            sync->cnt_s = (failed || all) ? n : cnt_s;
            sync->cnt_v = (failed || all) ? n : cnt_v;
            sync->open = open ? 1 : 0;
            if (failed) atomicOr(a.status, STAT_WALK_TIMEOUT);
            if (a.accounted) a.accounted[bh] = sum;
        }
        return;
    }

    // ---------------------------------------------------------------------- the decisions (wave 0)
    const bool early = a.accounted == nullptr;
    int is = 0, iv = 0;                        // heads of the two lists (plain scalars: an array indexed by the
    int blk_s = 0, blk_v = 0;                  // list would be kept in scratch memory); block each head is in
    int have_s = 0, have_v = 0;                // blocks of each list known to be resident (staged and summed)
    int published = 0;                         // runs handed to the summing wave
    int ended = 0;                             // OVER: the sum has reached the target, FAILED: a wait has run into its bound
    constexpr int OVER = 1, FAILED = 2, CUT = 3;           // CUT: a head has come to where its list is no longer in order
    int need_s = 2, need_v = 2;                // blocks whose prefix sums have been asked for
    int full = 1;                              // the last run had as many picks as were looked at
    int few_picks = 0;                         // wide looks in a row that found a short run
    int column = 0;                            // it ended where the next pick is a column: no need to see that again
    int falls_s = 0, falls_v = 0;
    const int far_s = reach(0, &falls_s), far_v = reach(1, &falls_v);
    // until the head's block and the one after it (the first `want` blocks of list l) are resident
    auto wait_blocks = [&](int l, int want, bool sums = true) __attribute__((always_inline)) {
        int spins = 0, have;
        for (;;) {
            const int st = walk_ld(&sync->staged[l]), su = sums ? walk_ld(&sync->summed_blk[l]) : st;
            have = st < su ? st : su;
            if (have >= want) break;
            if (walk_ld(&sync->stop)) { ended = OVER; break; }
            __builtin_amdgcn_s_sleep(1);
            if (++spins > spin_limit || walk_ld(&sync->err)) { ended = FAILED; break; }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
        return __builtin_amdgcn_readfirstlane(have);
    };

    auto uniform = [](int x) { return __builtin_amdgcn_readfirstlane(x); };      // (what the compiler does not see to be: its branches then go by scalar conditions)
    auto lane0 = [](float x) { return __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, x))); };
    // blocks a view at head h reads: through the block of entry h + RUN - 1, and pre[h] itself
    auto blocks_for = [&](int h, int far) {
        const int want = (h + RUN - 1) / WALK_BLK + 1, all = (far + WALK_BLK - 1) / WALK_BLK;
        return want < all ? want : all;
    };
    __syncthreads();
    have_s = wait_blocks(0, blocks_for(0, far_s));
    have_v = wait_blocks(1, blocks_for(0, far_v));
    // the last head whose view is resident, given the resident blocks (of a list that is all there and in order: any)
    auto good = [&](int have, int far) {
        if (have * WALK_BLK >= far) return far < n ? far - 1 : 0x7FFFFFFF;
        return have * WALK_BLK - RUN;
    };
    int good_s = good(have_s, far_s), good_v = good(have_v, far_v);
    // A free slot of the ring: published runs less runs taken out (one read with whether the walk is over, which ends the waiting as well)
    auto slot_free = [&]() __attribute__((always_inline)) {
        int spins = 0;
        for (;;) {
            const unsigned long long ss = __atomic_load_n(static_cast<const unsigned long long*>(__builtin_assume_aligned(&sync->summed, 8)), __ATOMIC_RELAXED);
            if (__builtin_amdgcn_readfirstlane((int)(ss >> 32))) { ended = OVER; return false; }
            if (published - __builtin_amdgcn_readfirstlane((int)ss) < WALK_RING) break;
            __builtin_amdgcn_s_sleep(1);
            if (++spins > spin_limit || walk_ld(&sync->err)) { ended = FAILED; return false; }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
        return true;
    };
    auto hand_over = [&](Run& R, int which, int limit, int last) __attribute__((always_inline)) {
        if (lane == 0) { R.which = which; R.limit = limit; R.last = last; }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        ++published;
        if (lane == 0) walk_st(&sync->runs, published);
    };
    // Runs of RUN picks (at the list's end, of what is left) from list l, whose head is at h, without a look at each, where nothing can come between: the head adds something, the other list's head
    // does not, and adds the less the more lines of this list are taken; the overlap of the other list's lines with these is `ol` throughout.  As long as the last
    // of RUN picks adds something, mine * cost > 0 >= other * cost for all of them, since costs are 1 or more.  (Lines come in descending order, so that no gain
    // between is less than the last, nor a NaN; the prefix sums rise where all maxima are 0 or more.)  So the prefix sums are not needed meanwhile (informed: not
    // even to know that they rise).  Returns the head behind the runs; `have`: the list's blocks that are known to be there.
    auto quick = [&](int l, int h, float ol, int have, int falls, int far) __attribute__((always_inline)) -> int {
        const List& L = lists[l];
        int blk = h / WALK_BLK;
        while (h < far && !falls) {
            if (have < blocks_for(h, far)) {
                if (!informed && lane == 0) walk_st(&sync->need[l], blocks_for(h, far) + 1);
                have = wait_blocks(l, blocks_for(h, far), !informed);
                if (ended) break;
            }
            const int at = (h & (WALK_CAP - 1)) + lane, picks = far - h < RUN ? far - h : RUN;
            float gain[E];
#pragma unroll
            for (int e = 0; e < E; ++e) gain[e] = __fsub_rn(L.cw[at + 64 * e], ol);
            if (!informed) falls = walk_ld(&sync->falls[l]);
            float last = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, gain[E - 1]), 63));
            if (picks < RUN) last = __fsub_rn(lane0(L.cw[(h & (WALK_CAP - 1)) + picks - 1]), ol);
            if (uniform(falls || !(last > 0.f))) break;
            if (!slot_free()) break;
            Run& R = ring[published & (WALK_RING - 1)];
#pragma unroll
            for (int e = 0; e < E; ++e) R.g[72 * e + lane + 2 * (lane / 16)] = gain[e];
            hand_over(R, l, picks, picks < RUN ? 0 : RUN_WHOLE);
            h = uniform(h + picks);
            if (h < n && h / WALK_BLK != blk) {            // done reading the blocks left behind
                blk = h / WALK_BLK;
                if (lane == 0) walk_st(&sync->cur[l], blk);
            }
        }
        return h;
    };

    // the prefix sums of the first `want` blocks of list l are wanted (those of one more than the views meet, so that they are there in time)
    auto need_more = [&](int l, int want, int need) __attribute__((always_inline)) -> int {
        if (want <= need) return need;
        if (lane == 0) walk_st(&sync->need[l], want);
        return want;
    };
    // Decides run after run with N entries a lane, until the walk is over (false) or runs of another length would suit N better.
    auto decide = [&](auto ENTRIES) __attribute__((always_inline)) -> bool {
        constexpr int N = decltype(ENTRIES)::value;
        using View = WalkView<N>;
        auto view = [&](int l, int h) __attribute__((always_inline)) {
            const List& L = lists[l];
            View r;
            const int at = (h & (WALK_CAP - 1)) + lane;
#pragma unroll
            for (int e = 0; e < N; ++e) { r.cw[e] = L.cw[at + 64 * e]; r.pre[e] = L.pre[at + 64 * e]; r.cl[e] = L.cl[at + 64 * e]; }
            if (h < n) { r.w0 = lane0(r.cw[0]); r.l0 = lane0(r.cl[0]); r.ol0 = lane0(r.pre[0]); }
            else { r.w0 = 0.f; r.l0 = 1.f; r.ol0 = lane0(sync->tot[l]); }  // an exhausted list: no weight, and its overlap sum
            return r;                                                      // sits right behind its last line
        };
        View S = view(0, is), V = view(1, iv);
        bool old_s = false, old_v = false;     // the list's head has moved on, or its blocks were not all there
        auto head = [&](int l, int h, View& r) __attribute__((always_inline)) {
            const int at = h & (WALK_CAP - 1);
            r.w0 = h < n ? lane0(lists[l].cw[at]) : 0.f;
            r.ol0 = h < n ? lane0(lists[l].pre[at]) : lane0(sync->tot[l]);
        };
        while (!ended) {
            if (is >= n && iv >= n) break;
            // a head that has entered a new block frees the blocks behind it; a view that reaches into a block not
            // known to be resident yet is read again once that block is
            if (is / WALK_BLK != blk_s && is < n) {
                blk_s = is / WALK_BLK;
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");     // done reading the blocks left behind
                if (lane == 0) walk_st(&sync->cur[0], blk_s);
            }
            if (iv / WALK_BLK != blk_v && iv < n) {
                blk_v = iv / WALK_BLK;
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
                if (lane == 0) walk_st(&sync->cur[1], blk_v);
            }
            if (is > good_s) {
                if (is >= far_s && is < n) { ended = CUT; break; }
                if (have_s < blocks_for(is, far_s)) {      // (an exhausted list: all of them, for its whole overlap sum)
                    need_s = need_more(0, blocks_for(is, far_s) + 1, need_s);
                    have_s = wait_blocks(0, blocks_for(is, far_s));
                    if (ended) break;
                    old_s = true;
                }
                good_s = good(have_s, far_s);
            }
            if (iv > good_v) {
                if (iv >= far_v && iv < n) { ended = CUT; break; }
                if (have_v < blocks_for(iv, far_v)) {
                    need_v = need_more(1, blocks_for(iv, far_v) + 1, need_v);
                    have_v = wait_blocks(1, blocks_for(iv, far_v));
                    if (ended) break;
                    old_v = true;
                }
                good_v = good(have_v, far_v);
            }
            // long runs (after one that took all it could: where picks go back and forth the look would cost a tenth)
            if (full) {
                if (old_s) head(0, is, S);
                if (old_v) head(1, iv, V);
                const float ds = __fsub_rn(S.w0, V.ol0), dv = __fsub_rn(V.w0, S.ol0);
                const int to_s = uniform(is < n && (iv >= n || dv <= 0.f) && ds > 0.f), to_v = uniform(iv < n && (is >= n || ds <= 0.f) && dv > 0.f);
                if (to_s | to_v) {
                    const int from = to_s ? is : iv, to = quick(to_s ? 0 : 1, from, to_s ? V.ol0 : S.ol0, to_s ? have_s : have_v, to_s ? falls_s : falls_v, to_s ? far_s : far_v);
                    if (ended) break;
                    // (no choice between two variables to write to: they would lie in scratch memory)
                    if (to != from) {
                        is = to_s ? to : is; iv = to_s ? iv : to;
                        blk_s = to_s && to < n ? to / WALK_BLK : blk_s; blk_v = to_s || to >= n ? blk_v : to / WALK_BLK;
                        old_s = old_s || to_s; old_v = old_v || to_v;
                        full = 0;
                        continue;
                    }
                }
            }
            if (old_s) { S = view(0, is); old_s = false; }
            if (old_v) { V = view(1, iv); old_v = false; }
            // entry e of lane l: the decision if the walk has taken 64 e + l more slashes (iv frozen)
            float gain[N];
            bool turn[N];                     // the pick goes to the other list
            const float fs = (float)is, fv = (float)iv;
            int run = 0, which = 0, turns = 0;
            if (is < n && !column) {
#pragma unroll
                for (int e = 0; e < N; ++e) {
                    const float ds = __fsub_rn(S.cw[e], V.ol0), dv = __fsub_rn(V.w0, S.pre[e]);
                    const float cs = fmaxf(__fsub_rn(S.cl[e], fv), 1.0f), cv = fmaxf(__fsub_rn(V.l0, fs + (float)(64 * e + lane)), 1.0f);
                    turn[e] = !(__fmul_rn(ds, cv) >= __fmul_rn(dv, cs));
                    gain[e] = ds;
                }
                run = iv < n ? walk_first(turn) : 64 * N;
                turns = run < 64 * N && run < far_s - is;
                run = uniform(run < far_s - is ? run : far_s - is);
            }
            if (run == 0) {
                // the head pick is a vertical; entry e of lane l: the decision if 64 e + l more verticals are taken (is frozen)
                which = 1;
#pragma unroll
                for (int e = 0; e < N; ++e) {
                    const float dv = __fsub_rn(V.cw[e], S.ol0), ds = __fsub_rn(S.w0, V.pre[e]);
                    const float cv = fmaxf(__fsub_rn(V.cl[e], fs), 1.0f), cs = fmaxf(__fsub_rn(S.l0, fv + (float)(64 * e + lane)), 1.0f);
                    turn[e] = __fmul_rn(ds, cv) >= __fmul_rn(dv, cs);      // not a vertical again
                    gain[e] = dv;
                }
                run = is < n ? walk_first(turn) : 64 * N;
                run = uniform(run < far_v - iv ? run : far_v - iv);
            }
            if (run == 0) break;                   // cannot happen (entry 0 of lane 0 repeats the head's test); never spin
            // picks 0 .. run-1 come from list `which`; the walk ends early at a pick with no positive gain left
            // (the gains of a run do not increase: none is 0 or less if the last entry's is not)
            int stop_dead = 64 * N;
            if (early && __ballot(!(gain[N - 1] > 0.f)) != 0ull) {
                const bool has = which == 0 ? iv < n : is < n;
                bool dead[N];                 // no gain is left in either list
#pragma unroll
                for (int e = 0; e < N; ++e)
                    dead[e] = !(gain[e] > 0.f) && (!has || !((which == 0 ? __fsub_rn(V.w0, S.pre[e]) : __fsub_rn(S.w0, V.pre[e])) > 0.f));
                stop_dead = walk_first(dead);
            }
            const int limit = uniform(run < stop_dead ? run : stop_dead);
            full = limit == 64 * N;
            column = which == 0 && turns;
            // the list's view after the run (read again above if it reaches into a block that is not resident yet)
            const View nxt = view(which, (which == 0 ? is : iv) + limit);
            // hand the run over: a free slot of the ring, the gains, then the count of published runs
            if (!slot_free()) break;
            Run& R = ring[published & (WALK_RING - 1)];
#pragma unroll
            for (int e = 0; e < N; ++e) R.g[72 * e + lane + 2 * (lane / 16)] = gain[e];
            hand_over(R, which, limit, stop_dead < run ? 1 : 0);
            if (stop_dead < run) break;            // nothing after this run can add to the sum
            if (which == 0) { is = uniform(is + limit); S = nxt; } else { iv = uniform(iv + limit); V = nxt; }
            if (N == E) few_picks = limit <= 32 * WALK_NARROW ? few_picks + 1 : 0;
            if (E > WALK_NARROW && (N == E ? few_picks >= 3 : limit == 64 * WALK_NARROW)) { few_picks = 0; return true; }
        }
        return false;
    };
    bool wide = false;
    while (wide ? decide(std::integral_constant<int, E>{}) : decide(std::integral_constant<int, WALK_NARROW>{})) wide = !wide;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    if (lane == 0) {
        if (ended == FAILED) walk_st(&sync->err, 1);
        if (ended == CUT) walk_st(&sync->cut, 1);
        walk_st(&sync->decided, 1);
        walk_st(&sync->done, 1);
    }
}

// grid (BH); dynamic LDS: WALK_LDS_BYTES<E>
static_assert(2 * SELECT_RANGES <= WALK_THREADS, "a thread each");
template <int E, bool SORTED>
__global__ __launch_bounds__(WALK_THREADS) void walk_kernel(SelectArgs a) {
    extern __shared__ __align__(16) unsigned char walk_lds[];
    walk_head<E, SORTED>(a, blockIdx.x, walk_lds);
    __syncthreads();
    const WalkSync* sync = reinterpret_cast<const WalkSync*>(walk_lds + 2 * sizeof(WalkList<E>) + WALK_RING * sizeof(WalkRun<E>));
    const int bh = blockIdx.x, cnt_s = sync->cnt_s, cnt_v = sync->cnt_v;
    if constexpr (E == 16 && SORTED) {
        if (a.open) {
            int missing = 0;                               // ranges that were left out, of a head that needs them
            if (sync->open) {
                const int l = (int)threadIdx.x >= a.ranges ? 1 : 0, b = (int)threadIdx.x - l * a.ranges;
                missing = __syncthreads_count((int)threadIdx.x < 2 * a.ranges && a.info[((int64_t)l * a.BH + bh) * SELECT_RANGES + b] < 0);
            }
            if (threadIdx.x == 0) { a.open[bh] = missing; a.open[a.BH + bh] = 0; }
        }
    }
    if (threadIdx.x == 0) { a.s_cnt[bh] = cnt_s; a.v_cnt[bh] = cnt_v; }
    if (a.n > EMIT_LINES) return;
    emit_both<WALK_THREADS>(a, bh, cnt_s, cnt_v, reinterpret_cast<uint32_t*>(walk_lds));      // (not where `sync` lies)
}
static_assert(2 * sizeof(WalkList<4>) > EMIT_LINES / 4 + 4 * EMIT_LINES, "the bitmaps and their lines lie ahead of the rings");

// ---- Alg. 2 with the overlap of a candidate counted cell by cell ----------------------------------
// The loop of Alg. 2 compares the marginal contributions of the two list heads (Sec. 5.1); the listing bounds the
// part of a line that is already covered by the sum of w^max of the lines taken from the other list.  This variant
// adds that part up exactly: a diagonal o and a column b share the cell of the scored row at position b + o, if
// there is one, so
//     overlap(slash o)  = sum over scored rows t with key c = p_t - o >= 0 and c taken  of A[t][c]
//     overlap(column b) = sum over scored rows t with o = p_t - b >= 0 and o taken      of A[t][b]
// Everything else is the loop of walk_kernel (binary32, single roundings, cross-multiplied test).
//
// One workgroup per head.  The loop takes runs from one list (up to a few dozen a walk, of one to thousands of picks),
// and during a run the other list's head and taken set stand still.  So a round looks at many candidates of one
// list at once: 64 when the list has just changed, then up to 1024, one per thread.  It needs
//   - what the other list's taken set covers of each candidate: a bitmap says which of its W cells count;
//   - what of the other head is covered at each candidate: of its W cells those whose line is taken already, and those that earlier
//     candidates lie on: a running sum over the candidates;
//   - the first candidate that fails the test, and the gains before it added in order.
// What bounds it is the latency of a round, so the head with most rounds (a dozen at 8192 lines): cells that miss the L2 take 2000 cycles, a step of a wave by itself five
// cycles an instruction.  So a round of 64 candidates has two steps: four waves read what is covered of the candidates, a quarter of the rows each, a fifth what is covered of the other head, a
// sixth what the candidates cover of it; then one wave does all the rest.  Cycles of such a round, 8192 lines: 5000 to 5500, of 1024 candidates 10000 and as many more as
// cells take that are covered.  With one candidate in sixteen threads, the other head's cells added one after the other, and five barriers 7000 (13000 where the head crosses many candidates); the
// cells of a list's next candidates fetched a turn ahead 6400 to 10000 (as many more of them are fetched as a CU has lines in flight).  The whole ls_select_exact, us, so / now: 32 heads, 8192
// lines, six inputs, 60.9 / 47.2, 73.7 / 55.0, 67.4 / 50.4, 77.9 / 58.8, 73.9 / 54.2, 117.0 / 85.7; 32 heads, 1101 lines 53.7 / 36.8, 16 heads, 715 57.8 / 31.5, 4 heads, 3393 94.8 / 55.9.
// Taken pick by pick it was 0.37 us a pick: up to 3074 picks or 14 runs a head 1160 us.

// Sum of a double over the 64 lanes, the same value in every lane.  Data-parallel-primitive moves on the two
// halves of the value instead of cross-lane reads through LDS: a shuffle of a double is two LDS round trips, six
// steps of them were most of the time of a pick.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ double dpp_f64(double x) {      // lanes outside ROW_MASK receive 0
    const uint64_t u = __builtin_bit_cast(uint64_t, x);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, CTRL, ROW_MASK, 0xF, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), CTRL, ROW_MASK, 0xF, false);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ double wave_sum_f64(double x) {
    x += dpp_f64<0xB1, 0xF>(x);                            // quad_perm [1,0,3,2]
    x += dpp_f64<0x4E, 0xF>(x);                            // quad_perm [2,3,0,1]: every lane holds its quad's sum
    x += dpp_f64<0x141, 0xF>(x);                           // row_half_mirror: sums of 8
    x += dpp_f64<0x140, 0xF>(x);                           // row_mirror: every lane holds its row's (16 lanes) sum
    x += dpp_f64<0x142, 0xA>(x);                           // row_bcast15 into rows 1 and 3
    x += dpp_f64<0x143, 0xC>(x);                           // row_bcast31 into rows 2 and 3: lane 63 holds the total
    const uint64_t u = __builtin_bit_cast(uint64_t, x);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)u, 63), hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), 63);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}


// of the lanes to the left
__device__ __forceinline__ double lanes_before_f64(double x, double& all) {
    x += dpp_f64<0x111, 0xF>(x);                           // row_shr:1, 2, 4, 8
    x += dpp_f64<0x112, 0xF>(x);
    x += dpp_f64<0x114, 0xF>(x);
    x += dpp_f64<0x118, 0xF>(x);
    x += dpp_f64<0x142, 0xA>(x);                           // row_bcast15 into rows 1 and 3
    x += dpp_f64<0x143, 0xC>(x);                           // row_bcast31 into rows 2 and 3
    const uint64_t u = __builtin_bit_cast(uint64_t, x);
    all = __builtin_bit_cast(double, (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), 63) << 32 | (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)u, 63));
    return dpp_f64<0x138, 0xF>(x);                         // wave_shr:1
}

constexpr int XW_THREADS = 1024;
constexpr int XW_ROWS = 256;                   // longest window
constexpr int XW_FEW = 64;                     // candidates of the first round of a run
constexpr int XW_AGAIN = 768;                  // entries of a block of the sorted list behind the head before the next one is loaded
static_assert(XW_FEW == 64 && XW_AGAIN + XW_FEW <= XW_THREADS, "a lane each; the next candidates lie in the block");

// grid (BH).  Dynamic LDS: two bitmaps of n bits.
__global__ __launch_bounds__(XW_THREADS) void walk_exact_kernel(SelectArgs a) {
    extern __shared__ uint32_t xw_maps[];
    __shared__ __align__(16) float gains[XW_THREADS];
    __shared__ int32_t lines[2][XW_THREADS];   // the block of each sorted list that its head is in
    __shared__ float weights[2][XW_THREADS];
    __shared__ int32_t pos[XW_ROWS];           // positions of the scored rows
    __shared__ double parts[4][XW_FEW];        // few candidates: a quarter of what is covered of each
    __shared__ double before[XW_FEW];          // ... what the candidates before it cover of the other head
    __shared__ double crossed[XW_THREADS / 64];            // many: what each wave's cover of it
    __shared__ double head_part;               // what the lines taken cover of it
    __shared__ int32_t leaves;
    struct Round { int32_t end, taken; float sum; };
    __shared__ Round done[2];                  // (in turn: a wave may come to the next round's while another has yet to read this)
    constexpr int32_t XW_NEVER = 0x7FFFFFFF;
    const int bh = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = (int)a.n, W = a.w, words = (int)((a.n + 31) / 32);
    uint32_t *const map_s = xw_maps, *const map_v = xw_maps + words;       // lines taken
    for (int i = tid; i < 2 * words; i += XW_THREADS) xw_maps[i] = 0u;
    const bool window = a.q_pos == nullptr;    // the scored rows are the last W positions
    if (tid < W) {
        const int64_t p = window ? (int64_t)n - W + tid : a.q_pos[tid];
        pos[tid] = (int)(p > n - 1 ? n - 1 : p < -1 ? -1 : p);
    }
    const float target = a.alpha * a.total[bh], nh = (float)a.n_hat;
    const float* A = a.a_win + (int64_t)bh * W * a.n;
    auto length = [&](int line) { const float rest = (float)(n - line); return rest < nh ? rest : nh; };
    auto is_taken = [](const uint32_t* map, int line) -> bool { return line >= 0 && ((map[line >> 5] >> (line & 31)) & 1u); };

    // Of a list: its lines taken, and the place in its order of the first line of the block in `lines`.
    struct List { int id, taken, base; };
    auto load = [&](List& l) {
        l.base = l.taken;
        const int i = l.base + tid < n ? l.base + tid : n - 1;
        const int32_t x = a.sidx[((int64_t)l.id * a.BH + bh) * a.n + i];
        lines[l.id][tid] = x;
        weights[l.id][tid] = i < a.kept ? a.sorted_w[((int64_t)l.id * a.BH + bh) * a.kept + i] : ((l.id == 0 ? a.slash : a.vert) + (int64_t)bh * a.n)[x];
    };
    List X = {0, 0, 0}, O = {1, 0, 0};         // the list whose lines are the candidates, and the other one
    load(X);
    load(O);
    __syncthreads();
    float sum = 0.f;
    int most = XW_FEW, round = 0;              // candidates of the next round
    bool decided = false;                      // its first candidate is known to be the next pick
    while (sum < target && (X.taken < n || O.taken < n)) {
        bool change = false;                   // to the other list
        if (X.taken == n) change = decided = true;
        else {
            uint32_t* const map_x = X.id == 0 ? map_s : map_v;
            const uint32_t* const map_o = X.id == 0 ? map_v : map_s;
            const bool has_o = O.taken < n, few = most == XW_FEW;
            const int off = X.taken - X.base;  // the first candidate's place in the block: at most XW_AGAIN
            int C = XW_THREADS - off < most ? XW_THREADS - off : most;
            C = n - X.taken < C ? n - X.taken : C;
            const int j = few ? lane : tid;    // this thread's candidate
            const bool cand = j < C;
            const int32_t x = lines[X.id][off + (cand ? j : 0)], o = has_o ? lines[O.id][O.taken - O.base] : 0;
            const float weight = weights[X.id][off + (cand ? j : 0)], head_weight = has_o ? weights[O.id][O.taken - O.base] : 0.f;
            // the rows from t0 on, up to 64, whose cell of line x lies on a taken line of the other list
            auto rows_taken = [&](int t0) -> uint64_t {
                auto word = [&](int wi) { return wi >= 0 && wi < words ? map_o[wi] : 0u; };
                uint64_t on = 0ull;
                if (window) {
                    const int b = n - W + t0 - x, wi = b >> 5, sh = b & 31;
                    const uint64_t lo = ((uint64_t)word(wi + 1) << 32) | word(wi), hi = word(wi + 2);
                    on = lo >> sh | (sh ? hi << (64 - sh) : 0ull);
                    if (W - t0 < 64) on &= (1ull << (W - t0)) - 1ull;
                } else {
                    for (int t = 0; t < 64 && t0 + t < W; ++t) on |= (uint64_t)(is_taken(map_o, pos[t0 + t] - x) ? 1u : 0u) << t;
                }
                return on;
            };
            // of line x in row t, and (window) from where on the rows' lie how far apart
            const uint32_t step = (uint32_t)n + (X.id == 0 ? 1u : 0u), row0 = (uint32_t)(X.id == 0 ? n - W - x : x);
            auto row_cell = [&](int t) -> uint32_t { return window ? row0 + (uint32_t)t * step : (uint32_t)t * (uint32_t)n + (uint32_t)(X.id == 0 ? pos[t] - x : x); };
            auto head_cell = [&](int t) { return (int64_t)t * a.n + (O.id == 0 ? pos[t] - o : o); };       // of the other head
            // what of the other head is covered already, by one wave
            auto head_taken = [&]() {
                double part = 0.0;
                bool any = false;
                for (int t = lane; t < W; t += 64) {
                    const bool in = is_taken(map_x, pos[t] - o);
                    any |= in;
                    const float v = A[in ? head_cell(t) : 0];
                    part += in ? (double)v : 0.0;
                }
                part = __ballot(any) == 0ull ? 0.0 : wave_sum_f64(part);
                if (lane == 0) head_part = part;
            };
            // what line x covers of it: the cell where they cross, if a scored row has one
            auto crossing = [&]() -> double {
                if (window) {
                    const int t = x + o - (n - W);
                    const bool in = cand && t >= 0 && t < W;
                    const float v = A[in ? head_cell(t) : 0];
                    return in ? (double)v : 0.0;
                }
                double c = 0.0;
                for (int t = 0; t < W; ++t) if (cand && pos[t] == x + o) c += (double)A[head_cell(t)];
                return c;
            };
            // candidate j is taken before the other head
            auto stays_at = [&](float gain, double head_covered) -> bool {
                const float other_gain = __fsub_rn(head_weight, (float)head_covered);
                float cx = __fsub_rn(length(x), (float)O.taken); if (cx < 1.0f) cx = 1.0f;
                float co = __fsub_rn(length(o), (float)(X.taken + j)); if (co < 1.0f) co = 1.0f;
                const float mine = __fmul_rn(gain, co), other = __fmul_rn(other_gain, cx);
                return (X.id == 0 ? mine >= other : !(other >= mine)) || (j == 0 && decided);
            };
            if (few) {
                if (wv < 4) {                  // a quarter of the rows each
                    double p0 = 0.0, p1 = 0.0;
                    for (int t0 = 0; O.taken > 0 && t0 < W; t0 += 64) {
                        const uint32_t on = cand ? (uint32_t)(rows_taken(t0) >> (16 * wv)) & 0xFFFFu : 0u;
                        if (__ballot(on != 0u) == 0ull) continue;
                        float v[16];
                        if (window) {          // (a row's cells from W before its first on: where there is none to be read, the one W behind that)
                            const uint32_t at = (row0 + (uint32_t)W) * 4u, none = (uint32_t)W * 4u;
#pragma unroll
                            for (int u = 0; u < 16; ++u) {
                                const int t = t0 + 16 * wv + u < W ? t0 + 16 * wv + u : W - 1;
                                const unsigned char* row = reinterpret_cast<const unsigned char*>(A + (int64_t)t * step - W);
                                v[u] = *reinterpret_cast<const float*>(row + (on >> u & 1u ? at : none));
                            }
                        } else {
#pragma unroll
                            for (int u = 0; u < 16; ++u) v[u] = A[on >> u & 1u ? row_cell(t0 + 16 * wv + u) : 0u];
                        }
#pragma unroll
                        for (int u = 0; u < 16; ++u) {
                            const uint32_t keep = (uint32_t)__builtin_amdgcn_sbfe((int)on, u, 1);
                            (u & 1 ? p1 : p0) += (double)__builtin_bit_cast(float, __builtin_bit_cast(uint32_t, v[u]) & keep);
                        }
                    }
                    parts[wv][lane] = p0 + p1;
                } else if (wv == 4) {
                    if (has_o) head_taken();
                } else if (wv == 5) {
                    double c = has_o ? crossing() : 0.0, all;
                    if (__ballot(c != 0.0) != 0ull) c = lanes_before_f64(c, all);
                    before[lane] = c;
                }
                __syncthreads();
                if (wv == 0) {
                    const float covered = (float)((parts[0][lane] + parts[1][lane]) + (parts[2][lane] + parts[3][lane]));
                    const float gain = cand ? __fsub_rn(weight, covered) : 0.f;
                    const bool stays = cand && (!has_o || stays_at(gain, head_part + before[lane]));
                    const uint64_t leave = __ballot(cand && !stays);
                    const int end = leave != 0ull ? __ffsll((unsigned long long)leave) - 1 : XW_NEVER, run = end < C ? end : C;
                    float s = sum;
                    const float g[1] = {lane < run ? gain : 0.f};
                    const int got = run <= CHAIN_FEW ? chain_few(g[0], lane, run, target, s) : chain_until<1, true>(g, lane, run, target, s);
                    if (lane < got) atomicOr(&map_x[x >> 5], 1u << (x & 31));
                    if (lane == 0) done[round & 1] = Round{end, got, s};
                }
            } else {
                const bool busy = 64 * wv < C;
                double part = 0.0, c = 0.0;
                if (tid == 0) leaves = XW_NEVER;
                if (has_o && busy) c = crossing();
                if (O.taken > 0 && cand)
                    for (int t0 = 0; t0 < W; t0 += 64) {
                        uint64_t on = rows_taken(t0);
                        while (on) {           // eight cells in flight
                            float v[8];
                            uint64_t left = on;
#pragma unroll
                            for (int u = 0; u < 8; ++u) {
                                v[u] = A[left ? row_cell(t0 + __ffsll((unsigned long long)left) - 1) : 0];
                                left &= left - 1ull;
                            }
#pragma unroll
                            for (int u = 0; u < 8; ++u) { part += on ? (double)v[u] : 0.0; on &= on - 1ull; }
                        }
                    }
                if (has_o && wv == 0) head_taken();
                const float gain = cand ? __fsub_rn(weight, (float)part) : 0.f;
                double all = 0.0;
                if (__ballot(c != 0.0) != 0ull) c = lanes_before_f64(c, all);
                if (lane == 0) crossed[wv] = all;
                if (busy) gains[tid] = gain;
                __syncthreads();
                if (busy) {
                    bool stays = cand;
                    if (has_o) {
                        double waves = head_part;
                        for (int w = 0; w < wv; ++w) waves += crossed[w];
                        stays = cand && stays_at(gain, waves + c);
                    }
                    const uint64_t leave = __ballot(cand && !stays);
                    if (leave != 0ull && lane == 0) atomicMin(&leaves, 64 * wv + __ffsll((unsigned long long)leave) - 1);
                }
                __syncthreads();
                if (wv == 0) {
                    const int end = leaves, run = end < C ? end : C;
                    float s = sum;
                    const int got = run <= 64 ? chain_lds<1>(gains, lane, run, target, s) : chain_lds<16>(gains, lane, run, target, s);
                    for (int i = lane; i < got; i += 64) { const int32_t y = lines[X.id][off + i]; atomicOr(&map_x[y >> 5], 1u << (y & 31)); }
                    if (lane == 0) done[round & 1] = Round{end, got, s};
                }
            }
            __syncthreads();
            const Round r = done[round & 1];
            const int run = r.end < C ? r.end : C;
            sum = r.sum;
            ++round;
            X.taken += r.taken;
            if (r.taken == run && X.taken < n && X.taken - X.base > XW_AGAIN) {
                load(X);
                __syncthreads();
            }
            change = decided = r.end < C;      // then the first pick of the other list has been decided
            most = XW_THREADS;
        }
        if (change) { const List t = X; X = O; O = t; most = XW_FEW; }
    }
    const int cnt_s = X.id == 0 ? X.taken : O.taken, cnt_v = X.id == 0 ? O.taken : X.taken;
    if (tid == 0) {
        a.s_cnt[bh] = cnt_s;
        a.v_cnt[bh] = cnt_v;
        if (a.accounted) a.accounted[bh] = sum;
    }
    if (a.n > EMIT_LINES) return;
    __syncthreads();                           // the maps are done with
    emit_both<XW_THREADS>(a, bh, cnt_s, cnt_v, xw_maps);
}

// ---- chosen prefix -> ascending index list --------------------------------------------------------
// The list of a head by a workgroup.  bm: bitmap of n bits, lines of up to 1024 of its words.
__device__ __forceinline__ void emit_list(const SelectArgs& a, const int bh, const int list, const int cnt, uint32_t* bm, uint32_t* wsum) {
    const int tid = threadIdx.x;
    const int64_t n = a.n;
    const int words = (int)((n + 31) / 32);
    const int32_t* sorted_idx = a.sidx + ((int64_t)list * a.BH + bh) * n;
    int32_t* out = list == 0 ? a.s_idx + (int64_t)bh * a.cap_s : a.v_idx + (int64_t)bh * a.cap_v;
    const int cap = list == 0 ? a.cap_s : a.cap_v;
    if (tid == 0 && cnt > cap) atomicOr(a.status, list == 0 ? STAT_S_TRUNCATED : STAT_V_TRUNCATED);
    if (cnt >= n) {                                        // every line was taken: the list is 0 .. n-1
        for (int64_t i = tid; i < n && i < cap; i += 1024) out[i] = (int32_t)i;
        return;
    }
    for (int i = tid; i < words; i += 1024) bm[i] = 0u;
    __syncthreads();
    for (int i0 = tid; i0 < cnt; i0 += 8 * 1024) {          // eight independent loads in flight per thread
        int32_t x8[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) { const int i = i0 + j * 1024; x8[j] = i < cnt ? sorted_idx[i] : -1; }
#pragma unroll
        for (int j = 0; j < 8; ++j) if (x8[j] >= 0) atomicOr(&bm[x8[j] >> 5], 1u << (x8[j] & 31));
    }
    __syncthreads();
    uint16_t* stage = reinterpret_cast<uint16_t*>(bm + words);
    uint32_t at = 0u;
    for (int w0 = 0; w0 < words; w0 += PUT_WORDS) {
        if (w0 > 0) __syncthreads();                       // the last lines are out of `stage`
        at += put_lines<1024>(bm + w0, words - w0 < PUT_WORDS ? words - w0 : PUT_WORDS, 32 * w0, stage, wsum, 0, out, at, cap, tid);
    }
}

// Heads whose walk came to where a list is no longer in order (a.open) are walked again, by the whole launch: its workgroups share out such heads, those of a head put
// its missing ranges in order, and the one of them that is done last walks.  Nobody waits for anybody.  At least BH workgroups.
// The whole ls_select, us, everything in order beforehand / so, and where only one head in twenty needs it: 8 heads of 12347 lines 57 / 112, 55 / 100; 32 of 32768 107 / 195,
// 102 / 165; 96 of 12347 90 / 226, 80 / 152; 256 of 16384 186 / 436, 159 / 261; 16 of 131072 369 / 528, 347 / 432.  (By two to eight workgroups of each head's own: 127, 107; 280, 164; 234, 151; 569, 251; 619, 517.)
constexpr int REDO_CAP = 5120;
constexpr size_t REDO_LDS_BYTES = order_lds_bytes(4, REDO_CAP) > WALK_LDS_BYTES<8> ? order_lds_bytes(4, REDO_CAP) : WALK_LDS_BYTES<8>;
__device__ __forceinline__ int heads_open(const SelectArgs& a) {       // (each wave by itself)
    int heads = 0;
    for (int h0 = 0; h0 < a.BH; h0 += 64) heads += __popcll(__ballot(h0 + ((int)threadIdx.x & 63) < a.BH && a.open[h0 + (threadIdx.x & 63)] != 0));
    return heads;
}
__device__ __forceinline__ void redo_heads(const SelectArgs& a, const int heads, uint32_t* bm, uint32_t* wsum) {
    if (heads == 0) return;
    __shared__ OrderSync sync;
    __shared__ int last;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wgs = (int)(gridDim.x * gridDim.y), me = (int)(blockIdx.y * gridDim.x + blockIdx.x);
    unsigned char* lds = reinterpret_cast<unsigned char*>(bm);
    const int j = me % heads, part = me / heads, most = (wgs - 1 - j) / heads + 1;       // workgroups for the j-th of them
    int bh = 0;
    for (int h0 = 0, seen = 0; h0 < a.BH; h0 += 64) {
        uint64_t who = __ballot(h0 + lane < a.BH && a.open[h0 + lane] != 0);
        const int here = __popcll(who);
        if (j >= seen && j < seen + here) {
            for (int k = seen; k < j; ++k) who &= who - 1ull;
            bh = h0 + __ffsll((unsigned long long)who) - 1;
        }
        seen += here;
    }
    bh = __builtin_amdgcn_readfirstlane(bh);
    const int missing = __builtin_amdgcn_readfirstlane(a.open[bh]), parts = most < missing ? most : missing;
    if (part >= parts) return;
    __syncthreads();                                       // the workgroup's own list has been written
    for (int r = part; r < 2 * a.ranges; r += parts) {
        const int l = r >= a.ranges ? 1 : 0, b = r - l * a.ranges;
        if (__builtin_amdgcn_readfirstlane(a.info[((int64_t)l * a.BH + bh) * SELECT_RANGES + b]) >= 0) continue;
        (void)order_range<4, false, false>(a, l, bh, b, a.ranges, a.ranges, REDO_CAP, 0.f, lds, sync);
        __syncthreads();
    }
    __threadfence();                                       // (the others' L2 may be another: what was written goes to memory, and comes from there)
    __syncthreads();
    if (tid == 0) last = count_shared(reinterpret_cast<uint32_t*>(a.open) + a.BH + bh) + 1u == (uint32_t)parts;
    __syncthreads();
    if (__builtin_amdgcn_readfirstlane(last) == 0) return;
    __threadfence();
    if (tid < WALK_THREADS) walk_head<8, true>(a, bh, lds); else __syncthreads();
    __syncthreads();
    const WalkSync* walk = reinterpret_cast<const WalkSync*>(lds + 2 * sizeof(WalkList<8>) + WALK_RING * sizeof(WalkRun<8>));
    const int cnt_s = walk->cnt_s, cnt_v = walk->cnt_v;
    __syncthreads();
    if (tid == 0) { a.s_cnt[bh] = cnt_s; a.v_cnt[bh] = cnt_v; }
    for (int list = 0; list < 2; ++list) {
        emit_list(a, bh, list, list == 0 ? cnt_s : cnt_v, bm, wsum);
        __syncthreads();
    }
}

// grid (2, BH), or more than two; dynamic LDS as emit_list has it, REDO: at least REDO_LDS_BYTES.
// REDO (up to EMIT_REDO_HEADS heads): the launch walks heads again as well.  Its 109 registers and its LDS leave a CU one workgroup, where the small kernel has two; where two workgroups a head are more
// than the CUs that is a kernel of its own (redo_kernel), whose launch costs no more than the lists take longer: the whole ls_select, us, in one / by itself, 192 heads of 16384 lines 82.0 / 82.1, 256
// 99.7 / 99.9, of 40000 214.5 / 213.6, 512 of 9000 142.9 / 142.3; 32 of 32768 43.8 / 44.6.  Calls that leave nothing out, and ls_select_exact, have the small kernel: 256 heads of 8000 lines 59.7 -> 57.9.
template <bool REDO>
__global__ __launch_bounds__(1024) void emit_kernel(SelectArgs a) {
    extern __shared__ __align__(16) uint32_t bm[];
    __shared__ uint32_t wsum[16];
    const int bh = blockIdx.y;
    const int open = a.open ? a.open[bh] : 0, cnt = blockIdx.x == 0 ? a.s_cnt[bh] : a.v_cnt[bh];
    const int heads = REDO ? heads_open(a) : 0;
    if (blockIdx.x < 2 && !__builtin_amdgcn_readfirstlane(open)) emit_list(a, bh, blockIdx.x, cnt, bm, wsum);
    if constexpr (REDO) redo_heads(a, heads, bm, wsum);
}
__global__ __launch_bounds__(1024) void redo_kernel(SelectArgs a) {
    extern __shared__ __align__(16) uint32_t bm[];
    __shared__ uint32_t wsum[16];
    redo_heads(a, heads_open(a), bm, wsum);
}

// ---- union of two selections ------------------------------------------------------------------------
// Alg. 1 keeps the lines selected in every turn so far (its set L); Sec. 5, Step 1 notes that selected lines can be
// reused in later turns.  Column indices are key positions and diagonal indices are offsets, both unchanged when the
// context grows, so carrying a selection into a later turn is a union of index sets.  grid (2, BH): list 0 =
// diagonals, list 1 = columns; both inputs are marked in an LDS bitmap of n bits, which is then written out in order.
__global__ __launch_bounds__(1024) void merge_lines_kernel(MergeArgs a) {
    extern __shared__ uint32_t bm[];
    __shared__ uint32_t wsum[16];
    const int list = blockIdx.x, bh = blockIdx.y, tid = threadIdx.x;
    const int64_t n = a.n;
    const int words = (int)((n + 31) / 32);
    for (int i = tid; i < words; i += 1024) bm[i] = 0u;
    __syncthreads();
    bool dropped = false;
    for (int src = 0; src < 2; ++src) {
        const int32_t* idx = (src ? a.idx_b[list] : a.idx_a[list]) + (int64_t)bh * (src ? a.cap_b[list] : a.cap_a[list]);
        int cnt = (src ? a.cnt_b[list] : a.cnt_a[list])[bh];
        const int cap = src ? a.cap_b[list] : a.cap_a[list];
        if (cnt > cap) cnt = cap;
        for (int i = tid; i < cnt; i += 1024) {
            const int32_t x = idx[i];
            if (x >= 0 && x < n) atomicOr(&bm[x >> 5], 1u << (x & 31)); else dropped = true;
        }
    }
    dropped = __syncthreads_or(dropped);
    int32_t* out = a.idx[list] + (int64_t)bh * a.cap[list];
    const int cap = a.cap[list];
    uint32_t total = 0;
    for (int w0 = 0; w0 < words; w0 += PUT_WORDS) {
        if (w0 > 0) __syncthreads();
        total += put_lines<1024>(bm + w0, words - w0 < PUT_WORDS ? words - w0 : PUT_WORDS, 32 * w0, reinterpret_cast<uint16_t*>(bm + words), wsum, 0, out, total, cap, tid);
    }
    if (tid == 0) {
        a.cnt[list][bh] = (int32_t)total;
        if (total > (uint32_t)cap) atomicOr(a.status, list == 0 ? STAT_S_TRUNCATED : STAT_V_TRUNCATED);
        if (dropped) atomicOr(a.status, STAT_MERGE_RANGE);
    }
}

hipError_t run_merge_lines(const MergeArgs& a, hipStream_t st) {
    const size_t smem = (size_t)((a.n + 31) / 32) * 4 + put_lines_bytes(a.n);
    hipLaunchKernelGGL(merge_lines_kernel, dim3(2, a.BH), dim3(1024), smem, st, a);
    return hipGetLastError();
}

// ---- top-B retention ------------------------------------------------------------------------------
// keep_idx [BK][budget] ascending; keep_cnt = min(budget, len).
// Radix select on the descending keys in three digits (11 + 11 + 10 bits, most significant first) finds the
// key K* of the budget-th largest score; then every element above K* and the first few equal to it are
// written in index order.  One KV head has too few elements to need a chip but too many for one CU to be
// quick, so a head's scores are cut into chunks of TB_CHUNK, one workgroup each, and the steps are separate
// launches that meet in small global arrays: hist [BK][3][TB_BINS] (zeroed by the first launch), state
// [BK][3][2] (prefix and elements still wanted after each digit) and cnt [BK][chunks][2].
constexpr int TB_THREADS = 1024;
constexpr int TB_CHUNK = 2048;
constexpr int TB_BINS = 2048;

__device__ __forceinline__ uint32_t tb_digit(uint32_t key, int pass) {
    return pass == 0 ? key >> 21 : pass == 1 ? (key >> 10) & 2047u : key & 1023u;
}
__device__ __forceinline__ uint32_t tb_himask(int pass) { return pass == 0 ? 0u : pass == 1 ? 0xFFE00000u : 0xFFFFFC00u; }
__device__ __forceinline__ int tb_shift(int pass) { return pass == 0 ? 21 : pass == 1 ? 10 : 0; }

// All threads of a workgroup: from the histogram of digit `pass` (among the keys that match `prefix`) and the
// number of elements still wanted, the digit that holds the wanted-th element; returns the longer prefix and
// what is still wanted inside it.
__device__ __forceinline__ void tb_pick(const uint32_t* hist, int pass, uint32_t prefix, uint32_t rem,
                                        uint32_t* wsum, uint32_t* res, uint32_t& prefix_out, uint32_t& rem_out) {
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const uint32_t h0 = hist[2 * tid], h1 = hist[2 * tid + 1];
    const uint32_t v = h0 + h1;
    uint32_t inc = v;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) { const uint32_t t = __shfl_up(inc, off, 64); if (lane >= off) inc += t; }
    __syncthreads();                                       // wsum / res may still be read from an earlier call
    if (lane == 63) wsum[wv] = inc;
    __syncthreads();
    uint32_t ex = inc - v;
    for (int w = 0; w < wv; ++w) ex += wsum[w];
    if (ex < rem && rem <= ex + v) {                       // exactly one thread: the total is at least rem
        const uint32_t r = rem - ex;
        const uint32_t d = 2u * tid + (r > h0 ? 1u : 0u);
        res[0] = prefix | (d << tb_shift(pass));
        res[1] = r > h0 ? r - h0 : r;
    }
    __syncthreads();
    prefix_out = res[0]; rem_out = res[1];
}

__global__ void topb_zero_kernel(uint32_t* p, int count) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) p[i] = 0u;
}

// grid (chunks, BK): histogram of digit PASS over this chunk's keys that match the prefix found so far
template <int PASS>
__global__ __launch_bounds__(TB_THREADS) void topb_hist_kernel(TopbArgs a) {
    __shared__ uint32_t lh[TB_BINS];
    __shared__ uint32_t wsum[16], res[2];
    const int chunk = blockIdx.x, bk = blockIdx.y, tid = threadIdx.x, lane = tid & 63;
    const int64_t len = a.len;
    const int64_t keep = a.budget < len ? a.budget : len;
    if (keep == len) return;                               // everything is kept: the write step needs no threshold
    uint32_t* hist = a.hist + (int64_t)bk * 3 * TB_BINS;
    uint32_t* state = a.state + (int64_t)bk * 6;
    uint32_t prefix = 0u, rem = (uint32_t)keep;
    if (PASS >= 1) {
        if (PASS == 2) { prefix = state[0]; rem = state[1]; }
        tb_pick(hist + (PASS - 1) * TB_BINS, PASS - 1, prefix, rem, wsum, res, prefix, rem);
        if (chunk == 0 && tid == 0) { state[2 * (PASS - 1)] = prefix; state[2 * (PASS - 1) + 1] = rem; }
    }
    for (int i = tid; i < TB_BINS; i += TB_THREADS) lh[i] = 0u;
    __syncthreads();
    const float* sc = a.score + (int64_t)bk * len;
    uint32_t kb[TB_CHUNK / TB_THREADS];
#pragma unroll
    for (int q = 0; q < TB_CHUNK / TB_THREADS; ++q) {
        const int64_t i = (int64_t)chunk * TB_CHUNK + q * TB_THREADS + tid;
        const uint32_t k = desc_key(sc[i < len ? i : len - 1]);
        kb[q] = i < len ? k : 0xFFFFFFFFu;
    }
#pragma unroll
    for (int q = 0; q < TB_CHUNK / TB_THREADS; ++q) {
        // scores of one head crowd into few digits: lanes with the same digit add once, through their first lane
        const int64_t i = (int64_t)chunk * TB_CHUNK + q * TB_THREADS + tid;
        const bool on = i < len && (kb[q] & tb_himask(PASS)) == prefix;
        const uint32_t digit = tb_digit(kb[q], PASS);
        uint64_t peers = __ballot(on);
#pragma unroll
        for (int b = 0; b < 11; ++b) {
            const bool bit = (digit >> b) & 1u;
            const uint64_t m = __ballot(bit);
            peers &= bit ? m : ~m;
        }
        if (on && __ffsll((unsigned long long)peers) - 1 == lane) atomicAdd(&lh[digit], (uint32_t)__popcll(peers));
    }
    __syncthreads();
    for (int i = tid; i < TB_BINS; i += TB_THREADS) if (lh[i]) atomicAdd(&hist[PASS * TB_BINS + i], lh[i]);
}

// grid (chunks, BK): K* and the number of elements equal to it that are kept; per chunk, how many of its
// elements lie above K* and how many equal it
__global__ __launch_bounds__(TB_THREADS) void topb_count_kernel(TopbArgs a) {
    __shared__ uint32_t wsum[16], res[2], wg[16], we[16];
    const int chunk = blockIdx.x, bk = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int64_t len = a.len;
    const int64_t keep = a.budget < len ? a.budget : len;
    if (keep == len) return;
    uint32_t* state = a.state + (int64_t)bk * 6;
    uint32_t kstar, need_eq;
    tb_pick(a.hist + ((int64_t)bk * 3 + 2) * TB_BINS, 2, state[2], state[3], wsum, res, kstar, need_eq);
    if (chunk == 0 && tid == 0) { state[4] = kstar; state[5] = need_eq; }
    const float* sc = a.score + (int64_t)bk * len;
    uint32_t g = 0, e = 0;
#pragma unroll
    for (int q = 0; q < TB_CHUNK / TB_THREADS; ++q) {
        const int64_t i = (int64_t)chunk * TB_CHUNK + q * TB_THREADS + tid;
        const uint32_t key = desc_key(sc[i < len ? i : len - 1]);
        g += (uint32_t)__popcll(__ballot(i < len && key < kstar));
        e += (uint32_t)__popcll(__ballot(i < len && key == kstar));
    }
    if (lane == 0) { wg[wv] = g; we[wv] = e; }
    __syncthreads();
    if (tid == 0) {
        uint32_t tg = 0, te = 0;
        for (int w = 0; w < 16; ++w) { tg += wg[w]; te += we[w]; }
        a.cnt[((int64_t)bk * a.chunks + chunk) * 2] = tg;
        a.cnt[((int64_t)bk * a.chunks + chunk) * 2 + 1] = te;
    }
}

// grid (chunks, BK): slot of a kept element = kept elements before it; kept = above K*, or equal to it among
// the first need_eq of those
__global__ __launch_bounds__(TB_THREADS) void topb_write_kernel(TopbArgs a) {
    __shared__ uint32_t seg_g[TB_CHUNK / 64], seg_e[TB_CHUNK / 64], base_s[2];
    const int chunk = blockIdx.x, bk = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int64_t len = a.len;
    const int64_t keep = a.budget < len ? a.budget : len;
    int32_t* out = a.keep_idx + (int64_t)bk * a.budget;
    if (chunk == 0 && tid == 0) a.keep_cnt[bk] = (int32_t)keep;
    if (keep == len) {
#pragma unroll
        for (int q = 0; q < TB_CHUNK / TB_THREADS; ++q) {
            const int64_t i = (int64_t)chunk * TB_CHUNK + q * TB_THREADS + tid;
            if (i < len) out[i] = (int32_t)i;
        }
        return;
    }
    const uint32_t* state = a.state + (int64_t)bk * 6;
    const uint32_t kstar = state[4], need_eq = state[5];
    const float* sc = a.score + (int64_t)bk * len;
    // elements above / equal to K* in the chunks before this one (one wave adds them up, lanes striding)
    if (wv == 0) {
        uint32_t g = 0, e = 0;
        for (int c = lane; c < chunk; c += 64) { g += a.cnt[((int64_t)bk * a.chunks + c) * 2]; e += a.cnt[((int64_t)bk * a.chunks + c) * 2 + 1]; }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) { g += __shfl_xor(g, off, 64); e += __shfl_xor(e, off, 64); }
        if (lane == 0) { base_s[0] = g; base_s[1] = e; }
    }
    uint32_t kb[TB_CHUNK / TB_THREADS];
#pragma unroll
    for (int q = 0; q < TB_CHUNK / TB_THREADS; ++q) {
        const int64_t i = (int64_t)chunk * TB_CHUNK + q * TB_THREADS + tid;
        const uint32_t k = desc_key(sc[i < len ? i : len - 1]);
        kb[q] = i < len ? k : 0xFFFFFFFFu;
        const uint64_t gm = __ballot(i < len && kb[q] < kstar), em = __ballot(i < len && kb[q] == kstar);
        if (lane == 0) { seg_g[q * 16 + wv] = (uint32_t)__popcll(gm); seg_e[q * 16 + wv] = (uint32_t)__popcll(em); }
    }
    __syncthreads();
    if (wv == 0) {                                         // exclusive scan over the chunk's 64-element segments
        uint32_t g = lane < TB_CHUNK / 64 ? seg_g[lane] : 0u, e = lane < TB_CHUNK / 64 ? seg_e[lane] : 0u;
        uint32_t ig = g, ie = e;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t ug = __shfl_up(ig, off, 64), ue = __shfl_up(ie, off, 64);
            if (lane >= off) { ig += ug; ie += ue; }
        }
        if (lane < TB_CHUNK / 64) { seg_g[lane] = base_s[0] + ig - g; seg_e[lane] = base_s[1] + ie - e; }
    }
    __syncthreads();
    const uint64_t below = (1ull << lane) - 1ull;
#pragma unroll
    for (int q = 0; q < TB_CHUNK / TB_THREADS; ++q) {
        const int64_t i = (int64_t)chunk * TB_CHUNK + q * TB_THREADS + tid;
        const bool gt = i < len && kb[q] < kstar, eq = i < len && kb[q] == kstar;
        const uint64_t gm = __ballot(gt), em = __ballot(eq);
        const uint32_t gt_before = seg_g[q * 16 + wv] + (uint32_t)__popcll(gm & below);
        const uint32_t eq_before = seg_e[q * 16 + wv] + (uint32_t)__popcll(em & below);
        const uint32_t eq_kept_before = eq_before < need_eq ? eq_before : need_eq;
        if (gt || (eq && eq_before < need_eq)) out[gt_before + eq_kept_before] = (int32_t)i;
    }
}

// One workgroup per KV head, up to 1024 PER entries, does all steps with the keys in registers, a wave holding
// consecutive entries.  The threshold lies in one of 1024 bins of equal span between the smallest and the largest key, and so
// on inside that bin, until the few keys left are ranked directly or wanted as a whole: mostly one round, a few hundred keys
// at most sharing a bin.  (Digits of the keys as bins, into few of which a head's scores crowd, took 16 us of LDS atomics that take
// turns; two bits a step, counted in registers, 8 to 10 steps, 15.9 for 32 heads of 16384 entries, now 9.9.)
// Lanes that add to one word take turns, four cycles each: a bin has a word for every eighth lane.  ls_kv_compress, 32 heads, one word a
// bin / eight / two bits a step: 16384 entries of which 90 % weigh nothing 131 / 92 / 96 us, all but equal 122 / 89 / 95; 32768 77 / 56 / 57,
// 130 / 59 / 57; scores as they mostly are 93 / 93 / 98, 55 / 55 / 58.
// Beyond 32 keys a thread the launches below, 4.5 us each, are spread over the chip; 64 keys do not stay in registers.  The whole of
// ls_kv_compress (d 64, 8 rows), spread / one workgroup a head, us: 16500 entries 35.5 / 28.9 (8 heads), 93.5 / 73.8 (64); 32768
// entries 40.5 / 35.8 (8), 84.2 / 75.5 (32), 148 / 122 (64); 33000 entries 41.8 / 75.5 (8), 157 / 179 (64).
constexpr int TB_ONE_LEN = 32768, TB_RANKED = 256, TB_COPIES = 8;
template <int PER>
__global__ __launch_bounds__(TB_THREADS) void topb_one_kernel(TopbArgs a) {
    __shared__ uint4 bins[TB_THREADS][TB_COPIES / 4];
    __shared__ uint32_t left[TB_RANKED], most[2][16], place[3], nleft, found[2], wg[16], we[16];
    const int bk = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int len = (int)a.len, keep = a.budget < len ? a.budget : len;
    int32_t* out = a.keep_idx + (int64_t)bk * a.budget;
    if (tid == 0) a.keep_cnt[bk] = keep;
    if (keep == len) {
        for (int i = tid; i < len; i += TB_THREADS) out[i] = i;
        return;
    }
    const float* sc = a.score + (int64_t)bk * len;
    const int first = wv * (64 * PER) + lane;              // entry j of this thread: first + 64 j
    uint32_t key[PER];
#pragma unroll
    for (int j = 0; j < PER; ++j) key[j] = desc_key(sc[first + 64 * j < len ? first + 64 * j : len - 1]);      // (all loads in flight)
    if (tid == 0) nleft = 0u;
    auto clear = [&]() {
#pragma unroll
        for (int c = 0; c < TB_COPIES / 4; ++c) bins[tid][c] = make_uint4(0u, 0u, 0u, 0u);
    };
    clear();
    uint32_t* const copy = reinterpret_cast<uint32_t*>(bins) + (lane & (TB_COPIES - 1));
    uint32_t lo = 0xFFFFFFFFu, hi = 0u;                    // (entries behind the last one repeat it)
#pragma unroll
    for (int j = 0; j < PER; ++j) { lo = key[j] < lo ? key[j] : lo; hi = key[j] > hi ? key[j] : hi; }
    lo = lanes_min(lo); hi = lanes_max(hi);
    if (lane == 63) { most[0][wv] = lo; most[1][wv] = hi; }
    __syncthreads();
    lo = (uint32_t)__builtin_amdgcn_readlane((int)lanes_min(most[0][lane & 15]), 63);
    hi = (uint32_t)__builtin_amdgcn_readlane((int)lanes_max(most[1][lane & 15]), 63);
    // the rem-th smallest key of those not below lo lies among the `within` keys of [lo, lo + 2^bit)
    uint32_t rem = (uint32_t)keep, within;
    int bit;
    for (;;) {
        const int width = width_of(hi - lo);
        bit = width > 10 ? width - 10 : 0;
#pragma unroll
        for (int j = 0; j < PER; ++j)
            if (first + 64 * j < len && key[j] - lo <= hi - lo) atomicAdd(copy + ((key[j] - lo) >> bit) * TB_COPIES, 1u);
        __syncthreads();
        uint32_t mine = 0u;
#pragma unroll
        for (int c = 0; c < TB_COPIES / 4; ++c) { const uint4 b = bins[tid][c]; mine += b.x + b.y + b.z + b.w; }
        const uint32_t upto = lanes_upto(mine);
        if (lane == 63) wg[wv] = upto;
        __syncthreads();
        const uint32_t before = (uint32_t)__builtin_amdgcn_readlane((int)lanes_upto(lane < wv ? wg[lane & 15] : 0u), 63) + upto - mine;
        if (rem > before && rem <= before + mine) { place[0] = (uint32_t)tid; place[1] = before; place[2] = mine; }
        clear();
        __syncthreads();
        lo += place[0] << bit; rem -= place[1]; within = place[2];
        if (rem == within || within <= (uint32_t)TB_RANKED || bit == 0) break;
        hi = lo + ((1u << bit) - 1u);
    }
    // every key below kstar is kept, and need_eq of those equal to it
    uint32_t kstar = lo + (1u << bit) - 1u, need_eq = 0xFFFFFFFFu;
    if (rem != within) {
        if (within <= (uint32_t)TB_RANKED && bit > 0) {
#pragma unroll
            for (int j = 0; j < PER; ++j)
                if (first + 64 * j < len && key[j] - lo < 1u << bit) { const uint32_t at = atomicAdd(&nleft, 1u); if (at < (uint32_t)TB_RANKED) left[at] = key[j]; }
            __syncthreads();
            {                                              // four threads a key
                const uint32_t k = left[tid >> 2];
                uint32_t less = 0u, same = 0u;
                for (uint32_t i = tid & 3; i < within; i += 4) { const uint32_t o = left[i]; less += o < k; same += o == k; }
                less += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)less, 0xB1, 0xF, 0xF, false);        // quad_perm [1,0,3,2], [2,3,0,1]
                less += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)less, 0x4E, 0xF, 0xF, false);
                same += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)same, 0xB1, 0xF, 0xF, false);
                same += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)same, 0x4E, 0xF, 0xF, false);
                if (tid >> 2 < (int)within && less < rem && rem <= less + same) { found[0] = k; found[1] = rem - less; }       // (equal keys store the same)
            }
            __syncthreads();
            kstar = found[0]; need_eq = found[1];
        } else { kstar = lo; need_eq = rem; }
    }
    // places in index order: the waves before this one, the chunks before this one, the lanes before this one
    uint32_t g = 0u, e = 0u;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const bool in = first + 64 * j < len;
        g += (uint32_t)__popcll(__ballot(in && key[j] < kstar));
        e += (uint32_t)__popcll(__ballot(in && key[j] == kstar));
    }
    if (lane == 0) { wg[wv] = g; we[wv] = e; }
    __syncthreads();
    const uint32_t ag = lanes_upto(wg[lane & 15]), ae = lanes_upto(we[lane & 15]);        // (row 0 holds the sums)
    g = wv == 0 ? 0u : (uint32_t)__builtin_amdgcn_readlane((int)ag, wv - 1);
    e = wv == 0 ? 0u : (uint32_t)__builtin_amdgcn_readlane((int)ae, wv - 1);
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const bool in = first + 64 * j < len, gt = in && key[j] < kstar, eq = in && key[j] == kstar;
        const uint64_t gm = __ballot(gt), em = __ballot(eq);
        const uint32_t eb = e + __builtin_amdgcn_mbcnt_hi((uint32_t)(em >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)em, 0u));
        const uint32_t at = g + __builtin_amdgcn_mbcnt_hi((uint32_t)(gm >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)gm, 0u)) + (eb < need_eq ? eb : need_eq);
        if (gt || (eq && eb < need_eq)) out[at] = first + 64 * j;
        g += (uint32_t)__popcll(gm);
        e += (uint32_t)__popcll(em);
    }
}

// gather kept rows of up to two tensors: dst [BK][budget][row_bytes] <- src [BK][len][row_bytes]; grid (slot blocks, BK, tensors).
// 16 bytes a thread and row, four rows in flight: bound by HBM, 67 MB moved in 12 us (a row per 64-thread workgroup, a launch a
// tensor: 33 us).
constexpr int GATHER_THREADS = 256, GATHER_ROWS = 4;
struct GatherArgs { const unsigned char* src[2]; unsigned char* dst[2]; };
__global__ __launch_bounds__(GATHER_THREADS) void gather_rows_kernel(GatherArgs t, const int32_t* keep_idx, const int32_t* keep_cnt,
                                                                     int64_t len, int budget, int row_bytes) {
    const int lanes = row_bytes / 16, per = GATHER_THREADS / lanes;        // rows at a time (row_bytes: 128, 256 or 512)
    const int bk = blockIdx.y, cnt = keep_cnt[bk];
    const int slot = blockIdx.x * (GATHER_ROWS * per) + threadIdx.x / lanes, off = 16 * (threadIdx.x % lanes);
    const unsigned char* s = t.src[blockIdx.z] + (int64_t)bk * len * row_bytes + off;
    unsigned char* d = t.dst[blockIdx.z] + (int64_t)bk * budget * row_bytes + off;
    if (slot >= cnt) return;
    int32_t r[GATHER_ROWS];
    f32x4 v[GATHER_ROWS];
#pragma unroll
    for (int u = 0; u < GATHER_ROWS; ++u) r[u] = keep_idx[(int64_t)bk * budget + (slot + u * per < cnt ? slot + u * per : slot)];
#pragma unroll
    for (int u = 0; u < GATHER_ROWS; ++u) v[u] = *reinterpret_cast<const f32x4*>(s + (int64_t)r[u] * row_bytes);
#pragma unroll
    for (int u = 0; u < GATHER_ROWS; ++u)
        if (slot + u * per < cnt) *reinterpret_cast<f32x4*>(d + (int64_t)(slot + u * per) * row_bytes) = v[u];
}

constexpr int EMIT_REDO_HEADS = 128, REDO_MORE = 6;        // (with few heads up to six workgroups each more than the two that write the lists)
static void launch_emit(const SelectArgs& a, hipStream_t st) {
    if (a.n <= EMIT_LINES) return;
    const size_t bytes = (size_t)((a.n + 31) / 32) * 4 + put_lines_bytes(a.n), redo_bytes = REDO_LDS_BYTES > bytes ? REDO_LDS_BYTES : bytes;
    if (!a.open || a.BH > EMIT_REDO_HEADS) hipLaunchKernelGGL(emit_kernel<false>, dim3(2, a.BH), dim3(1024), bytes, st, a);
    if (!a.open) return;
    const int more = 256 / a.BH - 2, wgs = 2 + (more < REDO_MORE ? more : REDO_MORE);
    if (a.BH > EMIT_REDO_HEADS) hipLaunchKernelGGL(redo_kernel, dim3(a.BH < 256 ? 256 : a.BH), dim3(1024), redo_bytes, st, a);
    else hipLaunchKernelGGL(emit_kernel<true>, dim3(wgs, a.BH), dim3(1024), redo_bytes, st, a);
}
// Ranges of 8192 lines, a fifth less than a workgroup takes (the samples miss by 4 % at most; beyond 65536 lines by more, and a halved
// range counts again), and more of them, down to 512 lines, as long as there are compute units for one each: 8 heads of 8192 lines
// 33.2 us in 16 ranges, 36.7 in one; 512 workgroups instead of 256 take turns: 32 heads of 32768 lines 63.0 -> 75.5, of 8192 36.6 -> 45.8.
// One range saves the looks for its bounds and for its lines, which is more than fewer lines a workgroup save: up to 5120 lines, and where lists could have three or two ranges up to 6144 and 8192.  In ranges / in one, us:
// 4 heads of 4200 lines 23.7 / 22.7, 16 26.1 / 24.8, of 5003 27.2 / 26.9, 32 of 4500 29.1 / 27.0, of 6000 30.8 / 30.9, of 8192 32.7 / 35.0; 40 of 5500 30.5 / 29.3, of 7000 33.5 / 34.0; 64 of 4200 30.7 / 27.8, of 7000 35.5 / 34.4, of 8192 36.9 / 36.7.
// lazy: the last ranges are put in order only where a walk may come to them.  A workgroup then has two ranges of half the length, far apart, as long as they have 1024 lines (up to
// ORDER_WIDE): 32 heads of 32768 lines 33.0 -> 25.5 us, 12347 18.7 -> 17.0; of lists whose lines are all needed, 16500 of 32768 each, the whole ls_select 117 -> 122.
struct OrderPlan { int wgs, ranges; bool lazy; };          // of each list
static OrderPlan order_plan(const SelectArgs& a, bool lazy) {
    int64_t wgs = 1;
    if (a.n > ORDER_ONE) {
        wgs = a.n > ORDER_WIDE ? (a.n + 6553) / 6554 : (a.n + 8191) / 8192;
        const int64_t fill = 256 / (2 * (int64_t)a.BH), most = (a.n + 511) / 512;
        const int64_t more = fill < most ? fill : most;
        if (wgs < more) wgs = more;
        if (a.n <= (wgs == 2 ? 8192 : wgs == 3 ? 6144 : 0)) wgs = 1;
    }
    lazy = lazy && wgs > 1 && a.open && a.n >= LAZY_LINES;
    const int64_t nb = lazy && a.n <= ORDER_WIDE && 2 * wgs <= SELECT_RANGES && a.n >= 2048 * wgs ? 2 * wgs : wgs;
    return OrderPlan{(int)wgs, (int)nb, lazy};
}
int select_ranges_left_out(const SelectArgs& a) { const OrderPlan p = order_plan(a, a.accounted == nullptr); return p.lazy ? p.ranges : 0; }
static hipError_t sort_lines(SelectArgs& a, bool want_lazy, hipStream_t st) {
    const OrderPlan p = order_plan(a, want_lazy);
    const int nb = p.ranges;
    const bool lazy = p.lazy;
    int64_t chunks = nb == 1 ? (a.n + 1023) / 1024 : (a.n * 5 / (4 * nb) + 256 + 1023) / 1024;
    if (chunks > ORDER_CHUNKS || a.n > ORDER_WIDE) chunks = ORDER_CHUNKS;
    const int cap = (int)chunks * 1024;
    a.ranges = nb;
    if (!lazy) a.open = nullptr;
    if (nb == 1) a.info = nullptr;                         // (the walk's own look at the maxima comes as early)
    const dim3 grid(2 * (unsigned)a.BH, (unsigned)p.wgs);
    auto launch = [&](auto kernel, int pt) { hipLaunchKernelGGL(kernel, grid, dim3(ORDER_THREADS), order_lds_bytes(pt, cap), st, a, cap); };
    // (Lists in one range have an instance without these looks at any length: 256 heads of 4500 lines, the whole ls_select, 45.1 -> 41.7, of 8000 56.8 -> 53.0, 128 of 8192 39.2 -> 37.6.)
    if (a.n <= 1024) launch(&order_kernel<1, true, false>, 1);
    else if (nb == 1) { if (cap <= 6144) launch(&order_kernel<4, true, false>, 4); else launch(&order_kernel<8, true, false>, 8); }
    else if (cap <= 6144) { if (lazy) launch(&order_kernel<4, false, true>, 4); else launch(&order_kernel<4, false, false>, 4); }
    else { if (lazy) launch(&order_kernel<8, false, true>, 8); else launch(&order_kernel<8, false, false>, 8); }
    return hipGetLastError();
}

hipError_t init_select_kernels() {
    hipError_t e;
    if ((e = allow_full_lds(&order_kernel<1, true, false>)) != hipSuccess || (e = allow_full_lds(&order_kernel<4, true, false>)) != hipSuccess) return e;
    if ((e = allow_full_lds(&order_kernel<8, true, false>)) != hipSuccess || (e = allow_full_lds(&order_kernel<4, false, false>)) != hipSuccess) return e;
    if ((e = allow_full_lds(&order_kernel<4, false, true>)) != hipSuccess || (e = allow_full_lds(&order_kernel<8, false, false>)) != hipSuccess || (e = allow_full_lds(&order_kernel<8, false, true>)) != hipSuccess) return e;
    if ((e = allow_full_lds(&walk_kernel<4, true>)) != hipSuccess || (e = allow_full_lds(&walk_kernel<4, false>)) != hipSuccess) return e;
    if ((e = allow_full_lds(&walk_kernel<8, true>)) != hipSuccess || (e = allow_full_lds(&walk_kernel<8, false>)) != hipSuccess) return e;
    if ((e = allow_full_lds(&walk_kernel<16, true>)) != hipSuccess || (e = allow_full_lds(&walk_kernel<16, false>)) != hipSuccess) return e;
    if ((e = allow_full_lds(&walk_exact_kernel)) != hipSuccess) return e;
    if ((e = allow_full_lds(&merge_lines_kernel)) != hipSuccess) return e;
    if ((e = allow_full_lds(&emit_kernel<false>)) != hipSuccess || (e = allow_full_lds(&emit_kernel<true>)) != hipSuccess) return e;
    return allow_full_lds(&redo_kernel);
}

hipError_t run_select(const SelectArgs& a0, hipStream_t st) {
    SelectArgs a = a0;
    hipError_t e = sort_lines(a, a.accounted == nullptr, st);
    if (e != hipSuccess) return e;
    auto walk = [&](auto E) {
        constexpr int N = decltype(E)::value;
        if (a.sorted) hipLaunchKernelGGL((walk_kernel<N, true>), dim3(a.BH), dim3(WALK_THREADS), WALK_LDS_BYTES<N>, st, a);
        else hipLaunchKernelGGL((walk_kernel<N, false>), dim3(a.BH), dim3(WALK_THREADS), WALK_LDS_BYTES<N>, st, a);
    };
    if (a.n <= WALK_SHORT) walk(std::integral_constant<int, 4>{});
    else if (a.n < WALK_LONG) walk(std::integral_constant<int, 8>{});
    else walk(std::integral_constant<int, 16>{});
    launch_emit(a, st);
    return hipGetLastError();
}

hipError_t run_select_exact(const SelectArgs& a0, hipStream_t st) {
    SelectArgs a = a0;
    hipError_t e = sort_lines(a, false, st);
    if (e != hipSuccess) return e;
    const size_t smem = (size_t)((a.n + 31) / 32) * 4;
    hipLaunchKernelGGL(walk_exact_kernel, dim3(a.BH), dim3(XW_THREADS), 2 * smem + (a.n <= EMIT_LINES ? 2 * put_lines_bytes(a.n) : 0), st, a);
    launch_emit(a, st);
    return hipGetLastError();
}

int topb_chunks(int64_t len) { return (int)((len + TB_CHUNK - 1) / TB_CHUNK); }
size_t topb_scratch_words(int BK, int64_t len) { return (size_t)BK * (3 * TB_BINS + 6 + 2 * (size_t)topb_chunks(len)); }

hipError_t run_topb(const TopbArgs& a0, int BK, uint32_t* scratch, hipStream_t st) {
    if (a0.len < 1 || a0.len > TOPB_MAX_LEN || a0.budget < 1) return hipErrorInvalidValue;
    TopbArgs a = a0;
    if (a.len <= TB_ONE_LEN) {
        if (a.len <= 4096) hipLaunchKernelGGL(topb_one_kernel<4>, dim3(BK), dim3(TB_THREADS), 0, st, a);
        else if (a.len <= 16384) hipLaunchKernelGGL(topb_one_kernel<16>, dim3(BK), dim3(TB_THREADS), 0, st, a);
        else hipLaunchKernelGGL(topb_one_kernel<32>, dim3(BK), dim3(TB_THREADS), 0, st, a);
        return hipGetLastError();
    }
    a.chunks = topb_chunks(a.len);
    a.hist = scratch;
    a.state = a.hist + (size_t)BK * 3 * TB_BINS;
    a.cnt = a.state + (size_t)BK * 6;
    const dim3 grid(a.chunks, BK);
    const int nz = BK * 3 * TB_BINS;
    hipLaunchKernelGGL(topb_zero_kernel, dim3((nz + 255) / 256), dim3(256), 0, st, a.hist, nz);
    hipLaunchKernelGGL(topb_hist_kernel<0>, grid, dim3(TB_THREADS), 0, st, a);
    hipLaunchKernelGGL(topb_hist_kernel<1>, grid, dim3(TB_THREADS), 0, st, a);
    hipLaunchKernelGGL(topb_hist_kernel<2>, grid, dim3(TB_THREADS), 0, st, a);
    hipLaunchKernelGGL(topb_count_kernel, grid, dim3(TB_THREADS), 0, st, a);
    hipLaunchKernelGGL(topb_write_kernel, grid, dim3(TB_THREADS), 0, st, a);
    return hipGetLastError();
}

hipError_t run_gather_rows(const void* const* src, void* const* dst, int tensors, const int32_t* keep_idx, const int32_t* keep_cnt,
                           int BK, int64_t len, int budget, int row_bytes, hipStream_t st) {
    GatherArgs t{};
    for (int i = 0; i < tensors; ++i) { t.src[i] = static_cast<const unsigned char*>(src[i]); t.dst[i] = static_cast<unsigned char*>(dst[i]); }
    const int rows = GATHER_ROWS * (GATHER_THREADS / (row_bytes / 16));
    hipLaunchKernelGGL(gather_rows_kernel, dim3((budget + rows - 1) / rows, BK, tensors), dim3(GATHER_THREADS), 0, st,
                       t, keep_idx, keep_cnt, len, budget, row_bytes);
    return hipGetLastError();
}

}  // namespace ls
