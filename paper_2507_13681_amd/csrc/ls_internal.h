// Host-side argument blocks and launchers shared by the translation units of libloopserve.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace ls {

struct ScoreArgs {
    const void* q;            // [B,Hq,w,d]
    const void* k;            // [B,Hkv,n,d]
    const int64_t* q_pos;     // [w] or null
    int64_t n;
    int w, G, Hq, Hkv, B, BH, nkb;
    float scale_log2e;
    float* part;              // [B*Hkv][nkb][G*w][2] per key block max / sum of every row; later the shares of the totals
    float* rowstat;           // [BH*w][2]        row max, 1 / row sum
    float* spart;             // [2][BH][n][2]    mode 0: diagonal partial sum / max by key-block parity, or what neighbouring key blocks leave each other (edge, edge_share, edge_done)
    float *vert, *slash, *vmax, *smax, *total;
    float* gscore;            // [B*Hkv][n]       group-summed column sums (retention score)
    float* a_win;             // [BH][w][n]       the window matrix (mode 3), or [heads from bh_first on][t1 - t0][n] a band of it (mode 1)
    int64_t win_rows;         // mode 1: how many rows of a KV head's G heads the buffer takes, at least one
    // set by run_score for each launch
    bool retain;              // mode 2: all rows in LDS
    int parts, stat_chunks;   // ranges of keys whose row statistics lie in `part`; chunks of rows of a workgroup of range_stats_kernel, at most
    bool join;                // mode 0: lines_kernel joins the key blocks' results itself
    int shares;               // mode 0: workgroups that share a KV head's query heads
    int bk0, bh_first;        // first KV head / query head
    int t0, t1;               // window rows whose matrix is written out
    int sums;                 // mode 1: the column sums of the chunks are added here (not on a chunk's later bands)
    uint32_t* done;           // [BH] workgroups of lines_kernel or finish_kernel that are done, of a head (the first of a share), cleared by stats_kernel or range_stats_kernel (null: not used)
};

// Where range x of `ranges` begins among `count` tiles or blocks of keys: floor(count * x / ranges).  That product passes 2^32 in ls_score, which has up to 768
// ranges and takes up to 2^31 keys (2^24 blocks); these do not, with at most 2^16 ranges.
__host__ __device__ inline uint32_t range_begin(uint32_t count, uint32_t ranges, uint32_t x) {
    const uint32_t each = count / ranges, rest = count % ranges;
    return each * x + rest * x / ranges;
}
// What of the scoring passes serves a call.
struct ScoreRoute {
    int ranges, unit;         // range_stats_kernel: ranges of keys, cut at multiples of `unit` keys; 0: stats_kernel
    int chunks;               // of 32 query rows, a workgroup of range_stats_kernel at most
    int shares;               // workgroups of stats_kernel that share a KV head's query heads
    bool folds;               // no merge_kernel: lines_kernel merges the row statistics
    bool joins;               // no finish_kernel: lines_kernel joins the key blocks' results
    bool streams;             // retention: all query rows stay in LDS while the keys come by
    int band_heads, band_rows, band_shares;        // mode 1: KV heads and window rows of a band of the matrix, workgroups of the first that share a KV head's query heads
};
ScoreRoute score_route(ScoreArgs& a, bool bf16, int d, int mode);

constexpr int SELECT_RANGES = 128;         // most ranges that a list is put in order by
constexpr int SELECT_HEAD_LINES = 1024;   // lines at the front of each sorted list whose weight and maximum are stored in order at least

// (The order decides which of its pointers walk_exact_kernel keeps in vector registers; with `w` last and `spin_limit` between the
// pointers it takes 73.9 instead of 69.6 us for 16 heads of 907 lines, 51.2 instead of 49.7 for 32 of 8192.)
struct SelectArgs {
    int64_t n, n_hat;
    int BH;
    float alpha;
    int spin_limit;           // bound of every wait between the waves of walk_kernel
    int w;                    // rows of a_win
    const float *vert, *slash, *vmax, *smax, *total;
    int32_t* sidx;            // [2][BH][n] line indices in sorted order
    int64_t kept;             // of each sorted list, the first lines whose weight and largest entry are there in order: n, or SELECT_HEAD_LINES
    float *sorted_w, *sorted_m;            // [2][BH][kept] (sorted_m: null where nobody wants it)
    int32_t* info;            // [2][BH][SELECT_RANGES] of a range of the list: 0: in order, 1: and one of its largest entries is negative or no number, -1 - k: left out, and k of the
                              // lines before it are in order (only with `open`); null: nobody has looked
    int32_t* open;            // [BH] ranges that were left out, of heads whose walk came to the end of what is in order (else 0), [BH] workgroups that have put their share of the rest in order; null: all of it is
    int ranges;               // of a list
    bool sorted;              // kept == n, and a block of lines may be read past the lists' ends
    int32_t *v_idx, *v_cnt, *s_idx, *s_cnt;
    int cap_v, cap_s;
    float* accounted;         // may be null
    int32_t* status;          // device status word of the context (bits LS_STAT_*), OR-ed into
    // exact-overlap variant (run_select_exact) only
    const float* a_win;       // [BH][w][n] window matrix
    const int64_t* q_pos;     // [w] positions of the scored rows, or null (the last w)
};

constexpr int64_t TOPB_MAX_LEN = 262144;   // longest score row run_topb takes

struct TopbArgs {
    const float* score;       // [BK][len]
    int64_t len;              // <= TOPB_MAX_LEN
    int budget;
    int32_t *keep_idx, *keep_cnt;
    // filled in by run_topb from its scratch block
    int chunks;
    uint32_t *hist, *state, *cnt;
};

constexpr uint32_t CUT_ON = 1u << 30;     // in a cut's tile word: the piece ends inside the item in which it begins

struct PlanArgs {
    int64_t n;
    int words, tab_len;
    const int32_t *v_idx, *v_cnt, *s_idx, *s_cnt;
    int cap_v, cap_s;
    uint32_t* obits;          // [BH][4 + words], four zero words first
    uint8_t* tab;             // [BH][tab_len]
    int nqb;                  // row blocks of the turn
    int64_t pos0;             // position of the first
    int dtype;
    uint16_t* elist;          // [BH][tab_len + 1] the table entries with a selected diagonal, ascending
    uint32_t* rec;            // [BH][nqb] of each row block: key blocks it visits | columns it gathers << 13
    uint32_t* upto;           // [BH][nqb] work of the head's row blocks up to and including this one (null: not wanted)
    uint32_t* arrived;        // [BH][nqb] cleared here for the parts of items (wanted with `upto`)
    uint32_t* head_work;      // [BH] work of all of them
    int32_t* split_count;     // [2] cleared here for sched_kernel
    int32_t* status;          // device status word of the context (bits LS_STAT_*), OR-ed into
};

// Work queues of the sparse attention kernel: one list per XCD of (head, row block) items or parts of them.
struct SchedArgs {
    int BH, G, Hq, Hkv, nqb;
    const uint32_t* rec;      // [BH][nqb], as plan_kernel left them
    const uint32_t* head_work;
    uint4* queue;             // [items + slots] entries, one queue behind the other: {item, part | parts << 8 | first slot << 16, key blocks, columns}
    int32_t* qlen;            // [8]
    int32_t* qbase;           // [8] first entry of each queue
    int32_t* qhead;           // [8] next entry to hand out (the first ones go by workgroup number)
    int grid;                 // workgroups of the attention kernel
    int slots;                // results of parts that the workspace holds (0: no item is split)
    uint2* split;             // [slots] split items: {item, parts | first slot << 16}
    int32_t* split_count;     // [2] slots in use, split items; cleared by plan_kernel
};

struct PrefillArgs {
    const void *q, *k, *v;
    void* out;
    float* lse;
    int64_t n, n_hat, pos0;
    int Hq, Hkv, G, BH, nqb, words, tab_len, dtype;
    float scale_log2e;
    const uint32_t* obits;
    const uint8_t* tab;
    const int32_t* v_idx;
    int cap_v;
    const uint16_t* elist;    // as plan_kernel left them
    int grid;                 // workgroups
    int slots;                // results of parts that may be kept
    // pieces (ls_prefill.hip): at most `grid`
    const uint32_t* rec;
    const uint32_t *upto, *head_work;
    int2* cuts;               // [1 + pieces] their number, and where each piece begins {item, tile | CUT_ON (that flag with `arrived` only)}
    uint32_t* arrived;        // [BH][nqb] tiles of the item's parts that are done, cleared by plan_kernel; null: combine_kernel puts the parts together
    // or work queues built by sched_kernel
    const uint4* queue;       // null: pieces
    const int32_t *qlen, *qbase;
    int32_t* qhead;
    const uint2* split;
    const int32_t* split_count;
    float *part_o, *part_ml;  // [slots][128][d] accumulators in lane order, [slots][128][2] reference and normaliser
};

struct DecodeArgs {
    const void *q;            // [B][Hq][d]
    const void *kc, *vc;      // [B][Hkv][cap][d] retained entries (first cnt rows valid)
    const void *kt, *vt;      // [B][Hkv][T][d] tokens since the retention
    const int32_t* cnt;       // [B][Hkv] or NULL (all cap rows)
    void* out;                // [B][Hq][d]
    float* lse;               // [B][Hq] or NULL
    float* part;              // [B*Hkv][nsplit][G][d + 4] per-split output, reference, normaliser
    uint32_t* done;           // [B*Hkv] splits finished; zero between calls
    uint32_t* done_clear;     // [clear_heads] the counters of the call after the next, cleared here; clear_heads >= B*Hkv
    int clear_heads;
    int B, Hq, Hkv, G, cap, T, nsplit, chunk;
    float scale_log2e;
};

// status bits (mirrors of LS_STAT_* in loopserve.h)
constexpr int STAT_WALK_TIMEOUT = 1, STAT_S_TRUNCATED = 2, STAT_V_TRUNCATED = 4, STAT_S_RANGE = 8, STAT_V_INVALID = 16,
              STAT_MERGE_RANGE = 32;
constexpr int WALK_SPIN_DEFAULT = 1 << 22;   // never reached in practice (about a second of polling)

// Lets a kernel use all of a compute unit's LDS (160 KB, less what the kernel declares statically) as
// dynamic LDS; the launches then only have to name the size they need.
template <typename K>
inline hipError_t allow_full_lds(K kernel) {
    hipFuncAttributes fa;
    hipError_t e = hipFuncGetAttributes(&fa, reinterpret_cast<const void*>(kernel));
    if (e != hipSuccess) return e;
    return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                               160 * 1024 - (int)fa.sharedSizeBytes);
}

// Once per device, with that device current: lets every kernel that asks for dynamic LDS use the whole 160 KB.
hipError_t init_score_kernels();
hipError_t init_select_kernels();
hipError_t init_prefill_kernels();
hipError_t init_decode_kernels();

hipError_t run_score(const ScoreArgs& a, int dtype, int d, int mode, hipStream_t st);
hipError_t run_decode(const DecodeArgs& a, int d, hipStream_t st);
size_t decode_smem_bytes(int d, int G, int nsplit);
size_t decode_part_floats(int d);                                   // floats of one partial result
void decode_split(int BK, int cap, int T, int limit, int* nsplit, int* chunk);   // at most `limit` splits; chunk: 32-key tiles per workgroup
constexpr int DECODE_MAX_SPLITS = 128;
// Union of two selections per head (the accumulated line set of Alg. 1): lists a and b in, ascending unique list out.
struct MergeArgs {
    int64_t n;
    int BH;
    const int32_t *idx_a[2], *cnt_a[2], *idx_b[2], *cnt_b[2];   // [0] diagonals, [1] columns
    int cap_a[2], cap_b[2];
    int32_t *idx[2], *cnt[2];
    int cap[2];
    int32_t* status;
};
hipError_t run_merge_lines(const MergeArgs& a, hipStream_t st);
hipError_t run_select(const SelectArgs& a, hipStream_t st);
int select_ranges_left_out(const SelectArgs& a);                      // ranges of each list of a call that may leave some of them out; else 0
hipError_t run_select_exact(const SelectArgs& a, hipStream_t st);   // a_win, q_pos, w set; vmax / smax unused
hipError_t run_topb(const TopbArgs& a, int BK, uint32_t* scratch, hipStream_t st);   // scratch: topb_scratch_words(BK, len) words
size_t topb_scratch_words(int BK, int64_t len);
hipError_t run_gather_rows(const void* const* src, void* const* dst, int tensors, const int32_t* keep_idx, const int32_t* keep_cnt,
                           int BK, int64_t len, int budget, int row_bytes, hipStream_t st);      // one or two tensors
hipError_t launch_plan(const PlanArgs& a, int BH, hipStream_t st);
hipError_t launch_sched(const SchedArgs& a, hipStream_t st);
// ev (null or four events): the start and stop time of the attention kernel's own dispatch, and, where a.slots > 0, of combine_kernel's
hipError_t launch_prefill(const PrefillArgs& a, int dtype, int d, hipStream_t st, const hipEvent_t* ev = nullptr);
size_t prefill_smem_bytes(int dtype, int d, int tab_len);
int prefill_block_rows();
bool prefill_in_pieces(int BH, int64_t n, int nqb, int dtype, int d);               // the work is shared out in pieces, or by queues
int prefill_grid(int dtype, int d, int64_t n, int64_t items, bool pieces);
int prefill_split_slots(int64_t items, int grid, bool pieces);      // parts' results that a call with so many (head, row block) items may use
size_t prefill_slot_bytes(int d);
int prefill_pieces_for(int64_t items, int grid, int slots);              // workgroups of a call in pieces with room for so many parts' results (0: queues)
bool prefill_joins(int dtype, int64_t items, int grid);               // pieces: whether the attention kernel puts the parts together itself
int prefill_piece_xcd(int p, int pieces);                                // XCD whose workgroup takes piece p

}  // namespace ls
