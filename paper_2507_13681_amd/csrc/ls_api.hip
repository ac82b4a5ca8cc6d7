// C-ABI entry points of libloopserve: argument checks, workspace carving, kernel dispatch.
#include <math.h>
#include <stdarg.h>
#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <array>
#include <mutex>
#include <new>
#include <vector>

#include "../../include/loopserve.h"
#include "../../include/loopserve_test_hooks.h"
#include "ls_internal.h"

static_assert(ls::TOPB_MAX_LEN == LS_MAX_N, "ls_kv_compress documents LS_MAX_N as its longest cache");
static_assert(ls::STAT_WALK_TIMEOUT == LS_STAT_WALK_TIMEOUT && ls::STAT_S_TRUNCATED == LS_STAT_S_TRUNCATED &&
              ls::STAT_V_TRUNCATED == LS_STAT_V_TRUNCATED && ls::STAT_S_RANGE == LS_STAT_S_RANGE &&
              ls::STAT_V_INVALID == LS_STAT_V_INVALID && ls::STAT_MERGE_RANGE == LS_STAT_MERGE_RANGE,
              "status bits of the kernels and of the header");

struct ls_ctx {
    int device;
    unsigned char* ws;
    size_t ws_bytes;
    int32_t* status;          // device status word (bits LS_STAT_*), OR-ed into by kernels, read and cleared by ls_poll_status
    // [COUNTER_SETS][MAX_HEADS] workgroups finished per head or KV head inside a launch.  Set 0: ls_score, cleared by the call's
    // first kernel.  The others take turns call by call in ls_decode_attend, one launch with nobody to clear a set ahead of it:
    // a launch leaves zeros in its own and clears the one after the next.  So calls that overlapped against the rules, and left a
    // set off, spoil the next user of that set and no more.
    uint32_t* counters;
    unsigned decode_calls;    // calls of ls_decode_attend that used a set
    int decode_heads;         // most KV heads of such a call: the part of a set that is cleared
    int walk_spin_limit;      // bound of the waits inside walk_kernel (test hook)
    char err[256];
    // optional timing of the sparse attention (ls_profile_*), per call: start and stop of the attention kernel, and of the launch
    // that puts parts together (null where there is none)
    bool profile;
    std::vector<std::array<hipEvent_t, 4>> events;
};

namespace {

constexpr size_t ALIGN = 256;
constexpr size_t MAX_HEADS = 65536;         // B * Hq (ls_score), B * Hkv (ls_decode_attend) <= 65535
constexpr unsigned DECODE_SETS = 4, COUNTER_SETS = 1 + DECODE_SETS;
constexpr size_t COUNTER_BYTES = COUNTER_SETS * MAX_HEADS * sizeof(uint32_t);
inline uint32_t* decode_set(const ls_ctx* c, unsigned call) { return c->counters + (1 + call % DECODE_SETS) * MAX_HEADS; }
inline size_t up(size_t x) { return (x + ALIGN - 1) / ALIGN * ALIGN; }

int fail(ls_ctx* c, int code, const char* fmt, ...) {
    if (c) {
        va_list ap;
        va_start(ap, fmt);
        vsnprintf(c->err, sizeof(c->err), fmt, ap);
        va_end(ap);
    }
    return code;
}

void drop_events(ls_ctx* c) {
    for (auto& call : c->events)
        for (hipEvent_t e : call) if (e) (void)hipEventDestroy(e);
    c->events.clear();
}

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// Scratch of the entry point that allocates nothing (ls_kv_compress_static): a fixed block of device memory
// that is part of the loaded code object.  Every GPU the library runs on holds its own copy at its own
// address until the process ends; host code reaches it only through the address that hipGetSymbolAddress
// returns on that device (scratch_on[device]), never through the array's name.
constexpr size_t STATIC_SCRATCH_BYTES = LS_STATIC_SCRATCH_BYTES;
static __device__ __align__(256) unsigned char scratch[STATIC_SCRATCH_BYTES];
std::vector<unsigned char*> scratch_on;      // per device, filled by init_device_once
char static_err[256] = "";                   // last error of a call that has no context

// Kernel attributes and the scratch address are per device: set once for each device the library is used on,
// with that device current.
hipError_t init_device_once(int device) {
    static std::mutex mu;
    static std::vector<char> done;
    std::lock_guard<std::mutex> lock(mu);
    try {                                    // (no exception may leave through the C entry points)
        if ((int)done.size() <= device) { scratch_on.resize(device + 1, nullptr); done.resize(device + 1, 0); }
    } catch (...) { return hipErrorOutOfMemory; }
    if (done[device]) return hipSuccess;
    hipError_t e;
    unsigned char* sp = nullptr;
    if ((e = hipGetSymbolAddress(reinterpret_cast<void**>(&sp), HIP_SYMBOL(scratch))) != hipSuccess) return e;
    scratch_on[device] = sp;
    if ((e = ls::init_score_kernels()) != hipSuccess) return e;
    if ((e = ls::init_select_kernels()) != hipSuccess) return e;
    if ((e = ls::init_prefill_kernels()) != hipSuccess) return e;
    if ((e = ls::init_decode_kernels()) != hipSuccess) return e;
    done[device] = 1;
    return hipSuccess;
}

struct Bump {
    unsigned char* base; size_t cap, off;
    template <typename T> T* take(size_t count) {
        const size_t bytes = up(count * sizeof(T));
        if (off + bytes > cap) { off = cap + 1; return nullptr; }
        T* p = reinterpret_cast<T*>(base + off);
        off += bytes;
        return p;
    }
    bool ok() const { return off <= cap; }
};

// common shape checks; `what` selects which fields matter
const char* check_shape(const ls_shape* s, bool need_nhat, bool need_w, bool cap_n) {
    if (!s) return "shape is NULL";
    if (s->B <= 0 || s->Hq <= 0 || s->Hkv <= 0) return "B, Hq, Hkv must be positive";
    if (s->Hq % s->Hkv) return "Hq must be a multiple of Hkv";
    if (s->d != 64 && s->d != 128) return "d must be 64 or 128";
    if (s->dtype != LS_BF16 && s->dtype != LS_F32) return "dtype must be LS_BF16 or LS_F32";
    if (s->n <= 0 || s->n > 2147483000LL) return "n out of range";
    if (cap_n && s->n > LS_MAX_N) return "n exceeds LS_MAX_N";
    if (need_nhat && (s->n_hat <= 0 || s->n_hat > s->n)) return "need 1 <= n_hat <= n";
    if (need_w && (s->w <= 0 || s->w > LS_MAX_W || s->w > s->n)) return "need 1 <= w <= min(n, LS_MAX_W)";
    if ((int64_t)s->B * s->Hq > 65535) return "B * Hq too large";
    return nullptr;
}

inline int nkb_of(int64_t n) { return (int)((n + 127) / 128); }
inline float scale_log2e(const ls_shape* s) {
    const float sc = s->scale > 0.f ? s->scale : 1.0f / sqrtf((float)s->d);
    return sc * 1.44269504088896340736f;
}

ls::ScoreArgs score_args(const ls_shape* s) {
    ls::ScoreArgs a{};
    a.n = s->n; a.w = s->w; a.G = s->Hq / s->Hkv; a.Hq = s->Hq; a.Hkv = s->Hkv; a.B = s->B; a.BH = s->B * s->Hq; a.nkb = nkb_of(s->n);
    a.scale_log2e = scale_log2e(s);
    return a;
}

// per key block max / sum of every scored row; later the 8 partial totals of every head
inline size_t part_floats(const ls_shape* s) {
    const size_t BH = (size_t)s->B * s->Hq;
    const size_t a = BH * s->w * nkb_of(s->n) * 2, b = BH * 8;
    return a > b ? a : b;
}
void row_scratch(ls::ScoreArgs& a, const ls_shape* s, Bump& bp) {
    a.part = bp.take<float>(part_floats(s));
    a.rowstat = bp.take<float>((size_t)a.BH * a.w * 2);
}
// ... and bands of the window matrix in what is left
void window_scratch(ls::ScoreArgs& a, const ls_shape* s, Bump& bp) {
    row_scratch(a, s, bp);
    const size_t row = (size_t)a.G * (size_t)a.n * 4;              // of a KV head's matrices
    a.win_rows = bp.ok() ? (int64_t)((bp.cap - bp.off) / row) : 0;
    a.a_win = reinterpret_cast<float*>(bp.base + bp.off);
}
// The window matrix of explicit scoring positions passes through what is left of the workspace, band by band.  The partial sums
// of the diagonals, which that path does not need, leave room for four rows of every head, and any call gets by with those.
// Asked for is room for the whole matrix up to WIN_BYTES, as much as the parts of long attention items take (ws_prefill).
// ls_score, 32 / 8 heads of 128, 64 rows, 32768 keys: 331 us through 16 MiB, 262 through 47, 189 through 64, 172 through 224, 158 with the whole matrix (256);
// 12347 keys: 195 us through 16 MiB, 109 through 47, 92 through 64, 84 whole (96); 131072 keys, 128 rows: 2130 through 47, 1387 through 64, 1284 through 224, 1012 whole (2048).
constexpr size_t WIN_BYTES = 64u << 20;
size_t ws_score(const ls_shape* s, bool lines) {
    const size_t BH = (size_t)s->B * s->Hq;
    size_t b = up(part_floats(s) * 4) + up(BH * s->w * 2 * 4);
    if (lines) {
        const size_t diag = 2 * BH * (size_t)s->n * 2 * 4, all = BH * s->w * (size_t)s->n * 4, win = all < WIN_BYTES ? all : WIN_BYTES;
        b += up(diag > win ? diag : win);
    }
    return b;
}
// The order of a list, and with it each line's weight and maximum.  (Calls get by with those of the first lines, as contexts made for less may have
// room for no more.)
size_t ws_select(const ls_shape* s) {
    const size_t BH = (size_t)s->B * s->Hq;
    return 3 * up(2 * BH * (size_t)s->n * 4) + 2 * up(2 * BH * ls::SELECT_HEAD_LINES * 4);
}
void order_scratch(ls::SelectArgs& a, Bump& bp) {
    const size_t lists = 2 * (size_t)a.BH, info = lists * ls::SELECT_RANGES;
    a.sidx = bp.take<int32_t>(lists * (size_t)a.n);
    const size_t more = up(info * 4) + up(2 * (size_t)a.BH * 4) + up(ls::SELECT_HEAD_LINES * 4);       // (the walk reads whole blocks of lines)
    const int64_t whole = a.n > ls::SELECT_HEAD_LINES ? a.n : ls::SELECT_HEAD_LINES;
    a.sorted = bp.ok() && bp.cap - bp.off >= 2 * up(lists * (size_t)whole * 4) + more;
    a.kept = a.sorted ? whole : ls::SELECT_HEAD_LINES;
    a.sorted_w = bp.take<float>(lists * (size_t)a.kept); a.sorted_m = bp.take<float>(lists * (size_t)a.kept);
    if (a.sorted) { a.info = bp.take<int32_t>(info); a.open = bp.take<int32_t>(2 * (size_t)a.BH); }
}
inline int words_of(int64_t n) { return (int)((n + 31) / 32) + 8; }
inline int tab_len_of(int64_t n) { return (int)(n / 64) + 4; }
// row blocks of the turn; they start at multiples of the block
inline int64_t row_blocks(int64_t n, int64_t n_hat) {
    const int64_t bm = ls::prefill_block_rows(), pos0 = (n - n_hat) / bm * bm;
    return (n - pos0 + bm - 1) / bm;
}
size_t ws_prefill(const ls_shape* s) {
    const size_t BH = (size_t)s->B * s->Hq;
    const int64_t n_hat = s->n_hat > 0 && s->n_hat <= s->n ? s->n_hat : s->n;
    const size_t items = BH * (size_t)row_blocks(s->n, n_hat);   // (head, row block) work items
    const bool pieces = ls::prefill_in_pieces((int)BH, s->n, (int)row_blocks(s->n, n_hat), s->dtype, s->d);
    const int grid = ls::prefill_grid(s->dtype, s->d, s->n, (int64_t)items, pieces);
    const size_t slots = (size_t)ls::prefill_split_slots((int64_t)items, grid, pieces);
    return up(BH * (size_t)(words_of(s->n) + 4) * 4) + up(BH * (size_t)tab_len_of(s->n)) + up(items * 4) + up(BH * 4) + up(BH * (size_t)(tab_len_of(s->n) + 1) * 2) +
           up(26 * 4) + up((items + slots) * 16) + up(pieces ? ((size_t)grid + 1) * 8 : slots * 8) + up(slots * ls::prefill_slot_bytes(s->d)) + ALIGN;
}
size_t ws_compress(const ls_shape* s) {
    return ws_score(s, false) + up((size_t)s->B * s->Hkv * (size_t)s->n * 4) +
           up(ls::topb_scratch_words(s->B * s->Hkv, s->n) * 4);
}

}  // namespace

extern "C" {

size_t ls_workspace_bytes(const ls_shape* s, int32_t budget) {
    (void)budget;
    if (check_shape(s, false, false, false)) return 0;
    ls_shape t = *s;
    if (t.w <= 0) t.w = 1;
    size_t m = ws_score(&t, true);
    if (ws_select(&t) > m) m = ws_select(&t);
    if (ws_prefill(&t) > m) m = ws_prefill(&t);
    if (ws_compress(&t) > m) m = ws_compress(&t);
    return m + ALIGN;
}

int ls_create(ls_ctx** out, int device, size_t workspace_bytes) {
    if (!out) return LS_EINVAL;
    *out = nullptr;
    int ndev = 0;
    if (hipGetDeviceCount(&ndev) != hipSuccess || device < 0 || device >= ndev) return LS_EHIP;
    if (hipSetDevice(device) != hipSuccess) return LS_EHIP;
    ls_ctx* c = new (std::nothrow) ls_ctx();
    if (!c) return LS_EINVAL;
    c->device = device; c->ws = nullptr; c->ws_bytes = workspace_bytes; c->err[0] = 0; c->profile = false;
    c->status = nullptr; c->decode_calls = 0; c->decode_heads = 0; c->walk_spin_limit = ls::WALK_SPIN_DEFAULT;
    if (init_device_once(device) != hipSuccess) { delete c; return LS_EHIP; }
    {
        void* p = nullptr;
        const size_t bytes = ALIGN + COUNTER_BYTES;
        if (hipMalloc(&p, bytes) != hipSuccess || hipMemset(p, 0, bytes) != hipSuccess) { if (p) (void)hipFree(p); delete c; return LS_EWORKSPACE; }
        c->status = static_cast<int32_t*>(p);
        c->counters = reinterpret_cast<uint32_t*>(static_cast<unsigned char*>(p) + ALIGN);
    }
    if (workspace_bytes) {
        void* p = nullptr;
        if (hipMalloc(&p, workspace_bytes) != hipSuccess) { (void)hipFree(c->status); delete c; return LS_EWORKSPACE; }
        c->ws = static_cast<unsigned char*>(p);
    }
    // (hipMemset returns at once, and calls may come on a stream that does not wait for the default one)
    if (hipStreamSynchronize(nullptr) != hipSuccess) { ls_destroy(c); return LS_EHIP; }
    *out = c;
    return LS_OK;
}

void ls_destroy(ls_ctx* c) {
    if (!c) return;
    (void)hipSetDevice(c->device);
    drop_events(c);
    if (c->ws) (void)hipFree(c->ws);
    if (c->status) (void)hipFree(c->status);
    delete c;
}

const char* ls_last_error(const ls_ctx* c) { return c ? c->err : static_err; }

int ls_score(ls_ctx* c, const ls_shape* s, const void* q_win, const int64_t* q_pos, const void* k,
             float* vert, float* slash, float* vmax, float* smax, float* total, void* stream) {
    if (!c) return LS_EINVAL;
    if (const char* m = check_shape(s, false, true, false)) return fail(c, LS_ESHAPE, "ls_score: %s", m);
    if (!q_win || !k || !vert || !slash || !vmax || !smax || !total) return fail(c, LS_EINVAL, "ls_score: NULL tensor");
    if (!aligned16(q_win) || !aligned16(k) || !aligned16(vert) || !aligned16(slash) || !aligned16(vmax) ||
        !aligned16(smax) || (q_pos && (reinterpret_cast<uintptr_t>(q_pos) & 7u)))
        return fail(c, LS_EINVAL, "ls_score: misaligned tensor");
    ls::ScoreArgs a = score_args(s);
    a.q = q_win; a.k = k; a.q_pos = q_pos;
    Bump bp{c->ws, c->ws_bytes, 0};
    const int mode = (q_pos == nullptr && s->w <= 128) ? 0 : 1;
    if (mode == 0) {
        row_scratch(a, s, bp);
        a.spart = bp.take<float>(2 * (size_t)a.BH * (size_t)a.n * 2);
    } else {
        window_scratch(a, s, bp);
        if (a.win_rows == 0) return fail(c, LS_EWORKSPACE, "ls_score: workspace of %zu bytes is too small", c->ws_bytes);
    }
    a.done = c->counters;
    if (!bp.ok()) return fail(c, LS_EWORKSPACE, "ls_score: workspace of %zu bytes is too small", c->ws_bytes);
    a.vert = vert; a.slash = slash; a.vmax = vmax; a.smax = smax; a.total = total; a.gscore = nullptr;
    if (hipSetDevice(c->device) != hipSuccess) return fail(c, LS_EHIP, "ls_score: hipSetDevice failed");
    const hipError_t e = ls::run_score(a, s->dtype, s->d, mode, static_cast<hipStream_t>(stream));
    if (e != hipSuccess) return fail(c, LS_EHIP, "ls_score: %s", hipGetErrorString(e));
    return LS_OK;
}

int ls_score_window(ls_ctx* c, const ls_shape* s, const void* q_win, const int64_t* q_pos, const void* k,
                    float* a_win, void* stream) {
    if (!c) return LS_EINVAL;
    if (const char* m = check_shape(s, false, true, false)) return fail(c, LS_ESHAPE, "ls_score_window: %s", m);
    if (!q_win || !k || !a_win) return fail(c, LS_EINVAL, "ls_score_window: NULL tensor");
    if (!aligned16(q_win) || !aligned16(k) || !aligned16(a_win) || (q_pos && (reinterpret_cast<uintptr_t>(q_pos) & 7u)))
        return fail(c, LS_EINVAL, "ls_score_window: misaligned tensor");
    ls::ScoreArgs a = score_args(s);
    a.q = q_win; a.k = k; a.q_pos = q_pos;
    Bump bp{c->ws, c->ws_bytes, 0};
    row_scratch(a, s, bp);
    if (!bp.ok()) return fail(c, LS_EWORKSPACE, "ls_score_window: workspace of %zu bytes is too small", c->ws_bytes);
    a.a_win = a_win;
    if (hipSetDevice(c->device) != hipSuccess) return fail(c, LS_EHIP, "ls_score_window: hipSetDevice failed");
    const hipError_t e = ls::run_score(a, s->dtype, s->d, 3, static_cast<hipStream_t>(stream));
    if (e != hipSuccess) return fail(c, LS_EHIP, "ls_score_window: %s", hipGetErrorString(e));
    return LS_OK;
}

int ls_select_exact(ls_ctx* c, const ls_shape* s, float alpha, const float* a_win, const int64_t* q_pos,
                    const float* vert, const float* slash, const float* total,
                    int32_t* v_idx, int32_t* v_cnt, int32_t cap_v, int32_t* s_idx, int32_t* s_cnt, int32_t cap_s,
                    float* accounted, void* stream) {
    if (!c) return LS_EINVAL;
    if (const char* m = check_shape(s, true, true, true)) return fail(c, LS_ESHAPE, "ls_select_exact: %s", m);
    if (!(alpha >= 0.f && alpha <= 1.f)) return fail(c, LS_EALPHA, "ls_select_exact: alpha %g outside [0, 1]", (double)alpha);
    if (!a_win || !vert || !slash || !total || !v_idx || !v_cnt || !s_idx || !s_cnt)
        return fail(c, LS_EINVAL, "ls_select_exact: NULL tensor");
    if (q_pos && (reinterpret_cast<uintptr_t>(q_pos) & 7u)) return fail(c, LS_EINVAL, "ls_select_exact: misaligned q_pos");
    if (cap_v <= 0 || cap_s <= 0) return fail(c, LS_ESHAPE, "ls_select_exact: capacities must be positive");
    ls::SelectArgs a{};
    a.n = s->n; a.n_hat = s->n_hat; a.BH = s->B * s->Hq; a.alpha = alpha;
    a.vert = vert; a.slash = slash; a.vmax = vert; a.smax = slash; a.total = total;   // the maxima are not used: any readable array
    Bump bp{c->ws, c->ws_bytes, 0};
    order_scratch(a, bp);
    a.sorted_m = nullptr; a.info = nullptr; a.open = nullptr;
    if (!bp.ok()) return fail(c, LS_EWORKSPACE, "ls_select_exact: workspace of %zu bytes is too small", c->ws_bytes);
    a.v_idx = v_idx; a.v_cnt = v_cnt; a.s_idx = s_idx; a.s_cnt = s_cnt; a.cap_v = cap_v; a.cap_s = cap_s;
    a.accounted = accounted; a.status = c->status; a.spin_limit = c->walk_spin_limit;
    a.a_win = a_win; a.q_pos = q_pos; a.w = s->w;
    if (hipSetDevice(c->device) != hipSuccess) return fail(c, LS_EHIP, "ls_select_exact: hipSetDevice failed");
    const hipError_t e = ls::run_select_exact(a, static_cast<hipStream_t>(stream));
    if (e != hipSuccess) return fail(c, LS_EHIP, "ls_select_exact: %s", hipGetErrorString(e));
    return LS_OK;
}

int ls_select(ls_ctx* c, const ls_shape* s, float alpha,
              const float* vert, const float* slash, const float* vmax, const float* smax, const float* total,
              int32_t* v_idx, int32_t* v_cnt, int32_t cap_v, int32_t* s_idx, int32_t* s_cnt, int32_t cap_s,
              float* accounted, void* stream) {
    if (!c) return LS_EINVAL;
    if (const char* m = check_shape(s, true, false, true)) return fail(c, LS_ESHAPE, "ls_select: %s", m);
    if (!(alpha >= 0.f && alpha <= 1.f)) return fail(c, LS_EALPHA, "ls_select: alpha %g outside [0, 1]", (double)alpha);
    if (!vert || !slash || !vmax || !smax || !total || !v_idx || !v_cnt || !s_idx || !s_cnt)
        return fail(c, LS_EINVAL, "ls_select: NULL tensor");
    if (cap_v <= 0 || cap_s <= 0) return fail(c, LS_ESHAPE, "ls_select: capacities must be positive");
    ls::SelectArgs a{};
    a.n = s->n; a.n_hat = s->n_hat; a.BH = s->B * s->Hq; a.alpha = alpha;
    a.vert = vert; a.slash = slash; a.vmax = vmax; a.smax = smax; a.total = total;
    Bump bp{c->ws, c->ws_bytes, 0};
    order_scratch(a, bp);
    if (!bp.ok()) return fail(c, LS_EWORKSPACE, "ls_select: workspace of %zu bytes is too small", c->ws_bytes);
    a.v_idx = v_idx; a.v_cnt = v_cnt; a.s_idx = s_idx; a.s_cnt = s_cnt; a.cap_v = cap_v; a.cap_s = cap_s;
    a.accounted = accounted; a.status = c->status; a.spin_limit = c->walk_spin_limit;
    if (hipSetDevice(c->device) != hipSuccess) return fail(c, LS_EHIP, "ls_select: hipSetDevice failed");
    const hipError_t e = ls::run_select(a, static_cast<hipStream_t>(stream));
    if (e != hipSuccess) return fail(c, LS_EHIP, "ls_select: %s", hipGetErrorString(e));
    return LS_OK;
}

int ls_merge_lines(ls_ctx* c, const ls_shape* s,
                   const int32_t* v_idx_a, const int32_t* v_cnt_a, int32_t cap_va,
                   const int32_t* s_idx_a, const int32_t* s_cnt_a, int32_t cap_sa,
                   const int32_t* v_idx_b, const int32_t* v_cnt_b, int32_t cap_vb,
                   const int32_t* s_idx_b, const int32_t* s_cnt_b, int32_t cap_sb,
                   int32_t* v_idx, int32_t* v_cnt, int32_t cap_v, int32_t* s_idx, int32_t* s_cnt, int32_t cap_s, void* stream) {
    if (!c) return LS_EINVAL;
    if (const char* m = check_shape(s, false, false, true)) return fail(c, LS_ESHAPE, "ls_merge_lines: %s", m);
    if (!v_idx_a || !v_cnt_a || !s_idx_a || !s_cnt_a || !v_idx_b || !v_cnt_b || !s_idx_b || !s_cnt_b || !v_idx || !v_cnt || !s_idx || !s_cnt)
        return fail(c, LS_EINVAL, "ls_merge_lines: NULL tensor");
    if (cap_va <= 0 || cap_sa <= 0 || cap_vb <= 0 || cap_sb <= 0 || cap_v <= 0 || cap_s <= 0)
        return fail(c, LS_ESHAPE, "ls_merge_lines: capacities must be positive");
    ls::MergeArgs a{};
    a.n = s->n; a.BH = s->B * s->Hq; a.status = c->status;
    a.idx_a[0] = s_idx_a; a.cnt_a[0] = s_cnt_a; a.cap_a[0] = cap_sa; a.idx_a[1] = v_idx_a; a.cnt_a[1] = v_cnt_a; a.cap_a[1] = cap_va;
    a.idx_b[0] = s_idx_b; a.cnt_b[0] = s_cnt_b; a.cap_b[0] = cap_sb; a.idx_b[1] = v_idx_b; a.cnt_b[1] = v_cnt_b; a.cap_b[1] = cap_vb;
    a.idx[0] = s_idx; a.cnt[0] = s_cnt; a.cap[0] = cap_s; a.idx[1] = v_idx; a.cnt[1] = v_cnt; a.cap[1] = cap_v;
    if (hipSetDevice(c->device) != hipSuccess) return fail(c, LS_EHIP, "ls_merge_lines: hipSetDevice failed");
    const hipError_t e = ls::run_merge_lines(a, static_cast<hipStream_t>(stream));
    if (e != hipSuccess) return fail(c, LS_EHIP, "ls_merge_lines: %s", hipGetErrorString(e));
    return LS_OK;
}

namespace {
// Where ls_sparse_prefill keeps its per-call state in the workspace (one place, so that the test hook that
// reads the work queues back finds them where the call put them).
struct PrefillCarve {
    uint32_t* obits; uint32_t* upto; uint32_t* head_work; uint16_t* elist; uint8_t* tab; int32_t* misc;
    uint32_t* rec; uint32_t* arrived; uint4* queue; uint2* split; int2* cuts; float* part_o; float* part_ml;
    bool pieces;
    int nqb, grid, slots; int64_t pos0; int code;
};
const char* carve_prefill(ls_ctx* c, const ls_shape* s, PrefillCarve& w) {
    const int BH = s->B * s->Hq;
    const int words = words_of(s->n), tab_len = tab_len_of(s->n);
    Bump bp{c->ws, c->ws_bytes, 0};
    w.obits = bp.take<uint32_t>((size_t)BH * (words + 4));
    w.head_work = bp.take<uint32_t>((size_t)BH);
    w.elist = bp.take<uint16_t>((size_t)BH * (tab_len + 1));
    const int bm = ls::prefill_block_rows();
    w.pos0 = (s->n - s->n_hat) / bm * bm;
    w.nqb = (int)row_blocks(s->n, s->n_hat);
    w.code = LS_ESHAPE;
    if (w.nqb > 65535) return "too many row blocks";
    if (BH > 8192) return "B * Hq exceeds 8192";
    const size_t items = (size_t)BH * w.nqb;
    uint32_t* per_item = bp.take<uint32_t>(items);         // pieces: `upto`, the records lie where the queues would; queues: the records
    w.tab = bp.take<uint8_t>((size_t)BH * tab_len);
    w.misc = bp.take<int32_t>(26);                         // of the queues: lengths, heads, first entries, slots in use and split items
    w.code = LS_EWORKSPACE;
    if (!bp.ok()) return "workspace is too small";
    // long items are cut as far as the workspace has room for their parts' results (sized for it by ls_workspace_bytes; a smaller
    // workspace that holds the rest still works)
    const Bump mark = bp;
    auto take = [&](int slots) {
        bp = mark;
        w.slots = slots;
        w.queue = bp.take<uint4>(items + slots);
        w.rec = w.pieces ? reinterpret_cast<uint32_t*>(w.queue) : per_item;
        w.upto = w.pieces ? per_item : nullptr;
        w.arrived = w.pieces && ls::prefill_joins(s->dtype, (int64_t)items, w.grid) ? w.rec + items : nullptr;    // (the queues' entries would have four words an item)
        w.cuts = w.pieces ? bp.take<int2>((size_t)w.grid + 1) : nullptr;
        w.split = slots && !w.pieces ? bp.take<uint2>((size_t)slots) : nullptr;
        w.part_o = slots ? bp.take<float>((size_t)slots * 128 * s->d) : nullptr;
        w.part_ml = slots ? bp.take<float>((size_t)slots * 128 * 2) : nullptr;
        return bp.ok();
    };
    auto most_slots = [&]() {                              // of those wanted, as many as fit
        int slots = ls::prefill_split_slots((int64_t)items, w.grid, w.pieces);
        const size_t queues = up(items * 16), room = mark.cap - mark.off > queues ? mark.cap - mark.off - queues : 0;
        if ((size_t)slots > room / ls::prefill_slot_bytes(s->d)) slots = (int)(room / ls::prefill_slot_bytes(s->d));
        while (slots > 0 && !take(slots)) --slots;         // (a slot has a few more bytes than its results, rounded up together)
        return slots;
    };
    w.pieces = ls::prefill_in_pieces(BH, s->n, w.nqb, s->dtype, s->d);
    w.grid = ls::prefill_grid(s->dtype, s->d, s->n, (int64_t)items, w.pieces);
    if (w.pieces) {
        w.grid = ls::prefill_pieces_for((int64_t)items, w.grid, most_slots());
        w.pieces = w.grid > 0;
        if (w.pieces && !take(ls::prefill_split_slots((int64_t)items, w.grid, true))) return "workspace is too small";
    }
    if (!w.pieces) {
        w.grid = ls::prefill_grid(s->dtype, s->d, s->n, (int64_t)items, false);
        if (!take(most_slots())) return "workspace is too small";
    }
    w.code = LS_OK;
    return nullptr;
}
}  // namespace

int ls_sparse_prefill(ls_ctx* c, const ls_shape* s, const void* q, const void* k, const void* v,
                      const int32_t* v_idx, const int32_t* v_cnt, int32_t cap_v,
                      const int32_t* s_idx, const int32_t* s_cnt, int32_t cap_s,
                      void* out, float* lse, void* stream) {
    if (!c) return LS_EINVAL;
    if (const char* m = check_shape(s, true, false, true)) return fail(c, LS_ESHAPE, "ls_sparse_prefill: %s", m);
    if (!q || !k || !v || !out || !v_idx || !v_cnt || !s_idx || !s_cnt)
        return fail(c, LS_EINVAL, "ls_sparse_prefill: NULL tensor");
    if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(out))
        return fail(c, LS_EINVAL, "ls_sparse_prefill: misaligned tensor");
    if (cap_v <= 0 || cap_s <= 0) return fail(c, LS_ESHAPE, "ls_sparse_prefill: capacities must be positive");
    const int BH = s->B * s->Hq;
    const int words = words_of(s->n), tab_len = tab_len_of(s->n);
    if (ls::prefill_smem_bytes(s->dtype, s->d, tab_len) > 160 * 1024)
        return fail(c, LS_ESHAPE, "ls_sparse_prefill: n too large for the LDS bitmaps");
    PrefillCarve w;
    if (const char* m = carve_prefill(c, s, w)) return fail(c, w.code, "ls_sparse_prefill: %s", m);
    const int nqb = w.nqb; const int64_t pos0 = w.pos0;
    if (hipSetDevice(c->device) != hipSuccess) return fail(c, LS_EHIP, "ls_sparse_prefill: hipSetDevice failed");
    ls::PlanArgs p{};
    p.n = s->n; p.words = words; p.tab_len = tab_len; p.v_idx = v_idx; p.v_cnt = v_cnt; p.s_idx = s_idx; p.s_cnt = s_cnt;
    p.cap_v = cap_v; p.cap_s = cap_s; p.obits = w.obits; p.tab = w.tab; p.nqb = nqb; p.pos0 = pos0; p.dtype = s->dtype;
    p.elist = w.elist; p.rec = w.rec; p.upto = w.upto; p.arrived = w.arrived; p.head_work = w.head_work; p.split_count = w.misc + 24; p.status = c->status;
    hipError_t e = ls::launch_plan(p, BH, static_cast<hipStream_t>(stream));
    if (e != hipSuccess) return fail(c, LS_EHIP, "ls_sparse_prefill(plan): %s", hipGetErrorString(e));
    if (!w.pieces) {
        ls::SchedArgs sa{};
        sa.BH = BH; sa.G = s->Hq / s->Hkv; sa.Hq = s->Hq; sa.Hkv = s->Hkv; sa.nqb = nqb; sa.rec = w.rec; sa.head_work = w.head_work;
        sa.queue = w.queue; sa.qlen = w.misc; sa.qhead = w.misc + 8; sa.qbase = w.misc + 16;
        sa.grid = w.grid; sa.slots = w.slots; sa.split = w.split; sa.split_count = w.misc + 24;
        e = ls::launch_sched(sa, static_cast<hipStream_t>(stream));
        if (e != hipSuccess) return fail(c, LS_EHIP, "ls_sparse_prefill(sched): %s", hipGetErrorString(e));
    }
    ls::PrefillArgs a{};
    a.q = q; a.k = k; a.v = v; a.out = out; a.lse = lse; a.n = s->n; a.n_hat = s->n_hat;
    a.elist = w.elist; a.rec = w.rec; a.upto = w.upto; a.head_work = w.head_work;
    a.queue = w.pieces ? nullptr : w.queue; a.qlen = w.misc; a.qhead = w.misc + 8; a.qbase = w.misc + 16;
    a.split = w.split; a.split_count = w.misc + 24;
    a.grid = w.grid; a.slots = w.slots; a.cuts = w.cuts; a.arrived = w.arrived; a.part_o = w.part_o; a.part_ml = w.part_ml;
    a.pos0 = pos0;
    a.Hq = s->Hq; a.Hkv = s->Hkv; a.G = s->Hq / s->Hkv; a.BH = BH;
    a.nqb = nqb; a.dtype = s->dtype;
    a.words = words; a.tab_len = tab_len; a.scale_log2e = scale_log2e(s);
    a.obits = w.obits; a.tab = w.tab; a.v_idx = v_idx; a.cap_v = cap_v;
    std::array<hipEvent_t, 4> ev{};
    if (c->profile) {
        try { c->events.reserve(c->events.size() + 1); } catch (...) { return fail(c, LS_EHIP, "ls_sparse_prefill: out of memory for events"); }
        for (size_t i = 0; i < (w.slots > 0 && !a.arrived ? 4u : 2u); ++i)
            if (hipEventCreate(&ev[i]) != hipSuccess) {
                for (size_t j = 0; j < i; ++j) (void)hipEventDestroy(ev[j]);
                return fail(c, LS_EHIP, "ls_sparse_prefill: hipEventCreate failed");
            }
    }
    e = ls::launch_prefill(a, s->dtype, s->d, static_cast<hipStream_t>(stream), c->profile ? ev.data() : nullptr);
    if (c->profile) c->events.push_back(ev);
    if (e != hipSuccess) return fail(c, LS_EHIP, "ls_sparse_prefill: %s", hipGetErrorString(e));
    return LS_OK;
}

namespace {
// Where a call's errors go: the context's message buffer, or the library's own for calls without a context.
struct ErrSink {
    ls_ctx* c;
    int operator()(int code, const char* fmt, ...) const {
        char* dst = c ? c->err : static_err;
        va_list ap;
        va_start(ap, fmt);
        vsnprintf(dst, 256, fmt, ap);
        va_end(ap);
        return code;
    }
};

// ls_kv_compress on an explicit scratch block (the context's workspace, or the static scratch)
int kv_compress_on(const ErrSink& fail, const char* who, int device, unsigned char* ws, size_t ws_bytes,
                   const ls_shape* s, int32_t budget, const void* q_obs, const void* k, const void* v,
                   int32_t* keep_idx, int32_t* keep_cnt, void* k_out, void* v_out, void* stream) {
    if (const char* m = check_shape(s, false, true, false)) return fail(LS_ESHAPE, "%s: %s", who, m);
    if (budget <= 0) return fail(LS_ESHAPE, "%s: budget must be positive", who);
    if (s->n > ls::TOPB_MAX_LEN) return fail(LS_ESHAPE, "%s: cache length %lld exceeds LS_MAX_N", who, (long long)s->n);
    if (!q_obs || !k || !keep_idx || !keep_cnt || (v_out && !v)) return fail(LS_EINVAL, "%s: NULL tensor", who);
    if (!aligned16(q_obs) || !aligned16(k) || !aligned16(v) || !aligned16(k_out) || !aligned16(v_out))
        return fail(LS_EINVAL, "%s: misaligned tensor", who);
    ls::ScoreArgs a = score_args(s);
    a.q = q_obs; a.k = k; a.q_pos = nullptr;
    const int BK = s->B * s->Hkv;
    Bump bp{ws, ws_bytes, 0};
    row_scratch(a, s, bp);
    a.gscore = bp.take<float>((size_t)BK * (size_t)a.n);
    uint32_t* tb_scratch = bp.take<uint32_t>(ls::topb_scratch_words(BK, s->n));
    if (!bp.ok()) return fail(LS_EWORKSPACE, "%s: needs %zu bytes of scratch, %zu are there", who, ws_compress(s), ws_bytes);
    if (hipSetDevice(device) != hipSuccess) return fail(LS_EHIP, "%s: hipSetDevice failed", who);
    hipStream_t st = static_cast<hipStream_t>(stream);
    hipError_t e = ls::run_score(a, s->dtype, s->d, 2, st);
    if (e != hipSuccess) return fail(LS_EHIP, "%s(score): %s", who, hipGetErrorString(e));
    ls::TopbArgs t{};
    t.score = a.gscore; t.len = s->n; t.budget = budget; t.keep_idx = keep_idx; t.keep_cnt = keep_cnt;
    e = ls::run_topb(t, BK, tb_scratch, st);
    if (e != hipSuccess) return fail(LS_EHIP, "%s(topb): %s", who, hipGetErrorString(e));
    const int row_bytes = s->d * (s->dtype == LS_BF16 ? 2 : 4);
    const void* src[2]; void* dst[2]; int tensors = 0;
    if (k_out) { src[tensors] = k; dst[tensors++] = k_out; }
    if (v_out) { src[tensors] = v; dst[tensors++] = v_out; }
    if (tensors) {
        e = ls::run_gather_rows(src, dst, tensors, keep_idx, keep_cnt, BK, s->n, budget, row_bytes, st);
        if (e != hipSuccess) return fail(LS_EHIP, "%s(gather): %s", who, hipGetErrorString(e));
    }
    return LS_OK;
}
}  // namespace

int ls_kv_compress(ls_ctx* c, const ls_shape* s, int32_t budget, const void* q_obs, const void* k, const void* v,
                   int32_t* keep_idx, int32_t* keep_cnt, void* k_out, void* v_out, void* stream) {
    if (!c) return LS_EINVAL;
    return kv_compress_on(ErrSink{c}, "ls_kv_compress", c->device, c->ws, c->ws_bytes, s, budget, q_obs, k, v,
                          keep_idx, keep_cnt, k_out, v_out, stream);
}

size_t ls_static_scratch_bytes(void) { return STATIC_SCRATCH_BYTES; }

int ls_kv_compress_static(int device, const ls_shape* s, int32_t budget, const void* q_obs, const void* k, const void* v,
                          int32_t* keep_idx, int32_t* keep_cnt, void* k_out, void* v_out, void* stream) {
    const ErrSink fail{nullptr};
    int ndev = 0;
    if (hipGetDeviceCount(&ndev) != hipSuccess || device < 0 || device >= ndev)
        return fail(LS_EHIP, "ls_kv_compress_static: no GPU %d", device);
    if (hipSetDevice(device) != hipSuccess) return fail(LS_EHIP, "ls_kv_compress_static: hipSetDevice failed");
    const hipError_t e = init_device_once(device);      // first call on this device: kernel attributes, scratch address
    if (e != hipSuccess) return fail(LS_EHIP, "ls_kv_compress_static: %s", hipGetErrorString(e));
    return kv_compress_on(fail, "ls_kv_compress_static", device, scratch_on[device], STATIC_SCRATCH_BYTES, s, budget,
                          q_obs, k, v, keep_idx, keep_cnt, k_out, v_out, stream);
}

size_t ls_decode_workspace_bytes(const ls_shape* s, int32_t cap, int32_t T) {
    if (!s || s->B <= 0 || s->Hq <= 0 || s->Hkv <= 0 || s->Hq % s->Hkv || (s->d != 64 && s->d != 128) || cap < 1 || T < 0) return 0;
    int nsplit, chunk;
    ls::decode_split(s->B * s->Hkv, cap, T, ls::DECODE_MAX_SPLITS, &nsplit, &chunk);
    return up((size_t)s->B * s->Hq * nsplit * ls::decode_part_floats(s->d) * 4) + ALIGN;
}

int ls_decode_attend(ls_ctx* c, const ls_shape* s, int32_t cap, int32_t T, const void* q, const void* k_c, const void* v_c,
                     const int32_t* cnt, const void* k_t, const void* v_t, void* out, float* lse, void* stream) {
    if (!c) return LS_EINVAL;
    if (!s) return fail(c, LS_ESHAPE, "ls_decode_attend: shape is NULL");
    if (s->B <= 0 || s->Hq <= 0 || s->Hkv <= 0 || s->Hq % s->Hkv) return fail(c, LS_ESHAPE, "ls_decode_attend: need positive B, Hq, Hkv with Hkv dividing Hq");
    if (s->d != 64 && s->d != 128) return fail(c, LS_ESHAPE, "ls_decode_attend: d must be 64 or 128");
    if (s->dtype != LS_BF16) return fail(c, LS_ESHAPE, "ls_decode_attend: dtype must be LS_BF16");
    if (s->Hq / s->Hkv > 32) return fail(c, LS_ESHAPE, "ls_decode_attend: at most 32 query heads per KV head");
    if ((int64_t)s->B * s->Hkv > 65535) return fail(c, LS_ESHAPE, "ls_decode_attend: B * Hkv too large");
    if (cap < 1 || T < 0 || (int64_t)cap + T > 2147483000LL / 256) return fail(c, LS_ESHAPE, "ls_decode_attend: need cap >= 1, T >= 0, cap + T < 2^23");
    if (!q || !k_c || !v_c || !out || (T > 0 && (!k_t || !v_t))) return fail(c, LS_EINVAL, "ls_decode_attend: NULL tensor");
    if (!aligned16(q) || !aligned16(k_c) || !aligned16(v_c) || !aligned16(k_t) || !aligned16(v_t) || !aligned16(out))
        return fail(c, LS_EINVAL, "ls_decode_attend: misaligned tensor");
    ls::DecodeArgs a{};
    a.q = q; a.kc = k_c; a.vc = v_c; a.kt = k_t; a.vt = v_t; a.cnt = cnt; a.out = out; a.lse = lse;
    a.B = s->B; a.Hq = s->Hq; a.Hkv = s->Hkv; a.G = s->Hq / s->Hkv; a.cap = cap; a.T = T;
    a.scale_log2e = scale_log2e(s);
    a.done = decode_set(c, c->decode_calls);
    a.done_clear = decode_set(c, c->decode_calls + 2);
    a.clear_heads = c->decode_heads > s->B * s->Hkv ? c->decode_heads : s->B * s->Hkv;
    // as many splits as the workspace has room for.  (The result of one split goes to `out`; a workspace that would not hold it is
    // refused all the same.)
    Bump bp{nullptr, 0, 0};
    for (int limit = ls::DECODE_MAX_SPLITS; limit > 0; limit = a.nsplit - 1) {
        ls::decode_split(s->B * s->Hkv, cap, T, limit, &a.nsplit, &a.chunk);
        bp = Bump{c->ws, c->ws_bytes, 0};
        a.part = bp.take<float>((size_t)s->B * s->Hq * a.nsplit * (a.nsplit > 1 ? ls::decode_part_floats(s->d) : (size_t)s->d + 2));
        if (bp.ok()) break;
    }
    if (ls::decode_smem_bytes(s->d, a.G, a.nsplit) > 156 * 1024) return fail(c, LS_ESHAPE, "ls_decode_attend: group too large for LDS");
    if (!bp.ok()) return fail(c, LS_EWORKSPACE, "ls_decode_attend: workspace of %zu bytes is too small", c->ws_bytes);
    if (hipSetDevice(c->device) != hipSuccess) return fail(c, LS_EHIP, "ls_decode_attend: hipSetDevice failed");
    hipError_t e = ls::run_decode(a, s->d, static_cast<hipStream_t>(stream));
    if (a.nsplit > 1) { ++c->decode_calls; c->decode_heads = a.clear_heads; }
    if (e != hipSuccess) return fail(c, LS_EHIP, "ls_decode_attend: %s", hipGetErrorString(e));
    return LS_OK;
}

int ls_profile_enable(ls_ctx* c, int on) {
    if (!c) return LS_EINVAL;
    (void)hipSetDevice(c->device);
    drop_events(c);
    c->profile = on != 0;
    return LS_OK;
}

int ls_profile_prefill_kernel_ms(ls_ctx* c, double* mean_ms, int32_t* launches) {
    if (!c || !mean_ms || !launches) return LS_EINVAL;
    double tot = 0.0;
    int cnt = 0;
    for (auto& e : c->events) {
        for (int k = 0; k < 4 && e[k]; k += 2) {
            if (hipEventSynchronize(e[k + 1]) != hipSuccess) return fail(c, LS_EHIP, "ls_profile: hipEventSynchronize failed");
            float ms = 0.f;
            if (hipEventElapsedTime(&ms, e[k], e[k + 1]) != hipSuccess) return fail(c, LS_EHIP, "ls_profile: hipEventElapsedTime failed");
            tot += ms;
        }
        ++cnt;
    }
    *mean_ms = cnt ? tot / cnt : 0.0;
    *launches = cnt;
    return LS_OK;
}

int ls_poll_status(ls_ctx* c, int32_t* host_out, void* stream) {
    if (!c || !host_out) return LS_EINVAL;
    if (hipSetDevice(c->device) != hipSuccess) return fail(c, LS_EHIP, "ls_poll_status: hipSetDevice failed");
    hipStream_t st = static_cast<hipStream_t>(stream);
    int32_t word = 0;
    // stream-ordered: read the word behind everything queued so far, then clear it
    if (hipMemcpyAsync(&word, c->status, sizeof(word), hipMemcpyDeviceToHost, st) != hipSuccess ||
        hipMemsetAsync(c->status, 0, sizeof(word), st) != hipSuccess || hipStreamSynchronize(st) != hipSuccess)
        return fail(c, LS_EHIP, "ls_poll_status: reading the status word failed");
    *host_out = word;
    return LS_OK;
}

int ls_debug_set_walk_spin_limit(ls_ctx* c, int32_t limit) {
    if (!c) return LS_EINVAL;
    c->walk_spin_limit = limit < 0 ? ls::WALK_SPIN_DEFAULT : limit;
    return LS_OK;
}

int ls_debug_set_counters(ls_ctx* c, int32_t value, void* stream) {
    if (!c) return LS_EINVAL;
    if (hipSetDevice(c->device) != hipSuccess ||
        hipMemsetD32Async(reinterpret_cast<hipDeviceptr_t>(c->counters), value, COUNTER_BYTES / 4, static_cast<hipStream_t>(stream)) != hipSuccess)
        return fail(c, LS_EHIP, "ls_debug_set_counters: hipMemsetD32Async failed");
    return LS_OK;
}

int ls_debug_fill_workspace(ls_ctx* c, int32_t value, void* stream) {
    if (!c) return LS_EINVAL;
    if (hipSetDevice(c->device) != hipSuccess ||
        hipMemsetD32Async(reinterpret_cast<hipDeviceptr_t>(c->ws), value, c->ws_bytes / 4, static_cast<hipStream_t>(stream)) != hipSuccess)
        return fail(c, LS_EHIP, "ls_debug_fill_workspace: hipMemsetD32Async failed");
    return LS_OK;
}

/* Debug / test hook: the items that the last ls_sparse_prefill call on this context gave to each XCD
 * (host_queue: [8][B*Hq*nqb] item words = (head << 16) | row block, host_qlen: [8]) and how often it cut one, as its kernels left
 * them in the workspace; synchronises the stream. */
int ls_debug_copy_prefill_queues(ls_ctx* c, const ls_shape* s, uint32_t* host_queue, int32_t* host_qlen, int32_t* nqb_out, int32_t* cuts_out, void* stream) {
    if (!c || !s || !host_queue || !host_qlen || !nqb_out || !cuts_out) return LS_EINVAL;
    if (check_shape(s, true, false, true)) return LS_ESHAPE;
    PrefillCarve w;
    if (carve_prefill(c, s, w)) return w.code;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const size_t items = (size_t)s->B * s->Hq * w.nqb;
    std::vector<uint4> q;
    std::vector<int2> cuts;
    try { q.resize(items + w.slots); cuts.resize((size_t)w.grid + 1); } catch (...) { return fail(c, LS_EHIP, "ls_debug_copy_prefill_queues: out of memory"); }
    int32_t misc[24];
    if (hipSetDevice(c->device) != hipSuccess) return LS_EHIP;
    auto word = [&](size_t i) { return (uint32_t)(i / w.nqb) << 16 | (uint32_t)(i % w.nqb); };
    for (int x = 0; x < 8; ++x) host_qlen[x] = 0;
    *cuts_out = 0;
    if (w.pieces) {
        auto read = [&](int2* to, const int2* from, size_t count) {
            return hipMemcpyAsync(to, from, count * sizeof(int2), hipMemcpyDeviceToHost, st) == hipSuccess && hipStreamSynchronize(st) == hipSuccess;
        };
        if (!read(cuts.data(), w.cuts, 1)) return LS_EHIP;
        const int pieces = cuts[0].x;
        if (pieces < 1 || pieces > w.grid) return fail(c, LS_EHIP, "ls_debug_copy_prefill_queues: no call of this shape came before");
        if (!read(cuts.data(), w.cuts, 1 + (size_t)pieces)) return LS_EHIP;
        // an item belongs to the piece on which it begins
        for (int p = 0; p < pieces; ++p) {
            const int x = ls::prefill_piece_xcd(p, pieces);
            cuts[1 + p].y &= (int)~ls::CUT_ON;
            if (p + 2 <= pieces) cuts[2 + p].y &= (int)~ls::CUT_ON;
            *cuts_out += cuts[1 + p].y > 0 ? 1 : 0;
            const int2 from = cuts[1 + p], to = p + 1 < pieces ? cuts[2 + p] : make_int2((int)items, 0);
            for (int64_t i = from.x + (from.y > 0 ? 1 : 0); i < to.x + (to.y > 0 ? 1 : 0); ++i)
                if (i >= 0 && (size_t)i < items && (size_t)host_qlen[x] < items) host_queue[x * items + host_qlen[x]++] = word((size_t)i);
        }
    } else {
        if (hipMemcpyAsync(q.data(), w.queue, q.size() * sizeof(uint4), hipMemcpyDeviceToHost, st) != hipSuccess) return LS_EHIP;
        if (hipMemcpyAsync(misc, w.misc, sizeof(misc), hipMemcpyDeviceToHost, st) != hipSuccess) return LS_EHIP;
        if (hipStreamSynchronize(st) != hipSuccess) return LS_EHIP;
        for (int x = 0; x < 8; ++x)                        // an item in parts is listed once, by its first part
            for (int i = 0; i < misc[x] && (size_t)misc[16 + x] + i < q.size(); ++i) {
                const uint4 e = q[(size_t)misc[16 + x] + i];
                *cuts_out += (e.y & 0xFF) != 0 ? 1 : 0;
                if ((e.y & 0xFF) == 0 && (size_t)host_qlen[x] < items) host_queue[x * items + host_qlen[x]++] = word(e.x);
            }
    }
    *nqb_out = w.nqb;
    return LS_OK;
}

int ls_debug_copy_select_order(ls_ctx* c, const ls_shape* s, int32_t* host_left, int32_t* host_again, int32_t* ranges, void* stream) {
    if (!c || !s || !host_left || !host_again || !ranges) return LS_EINVAL;
    if (check_shape(s, true, false, true)) return LS_ESHAPE;
    ls::SelectArgs a{};
    a.n = s->n; a.BH = s->B * s->Hq;
    Bump bp{c->ws, c->ws_bytes, 0};
    order_scratch(a, bp);
    if (!bp.ok()) return LS_EWORKSPACE;
    *ranges = ls::select_ranges_left_out(a);
    const size_t heads = (size_t)a.BH, lists = 2 * heads;
    std::fill(host_left, host_left + lists, 0);
    std::fill(host_again, host_again + heads, 0);
    if (*ranges == 0) return LS_OK;
    std::vector<int32_t> info;
    try { info.resize(lists * ls::SELECT_RANGES); } catch (...) { return fail(c, LS_EHIP, "ls_debug_copy_select_order: out of memory"); }
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (hipSetDevice(c->device) != hipSuccess || hipMemcpyAsync(info.data(), a.info, info.size() * 4, hipMemcpyDeviceToHost, st) != hipSuccess ||
        hipMemcpyAsync(host_again, a.open, heads * 4, hipMemcpyDeviceToHost, st) != hipSuccess || hipStreamSynchronize(st) != hipSuccess)
        return fail(c, LS_EHIP, "ls_debug_copy_select_order: reading the workspace failed");
    for (size_t l = 0; l < lists; ++l)
        for (int b = 0; b < *ranges; ++b) host_left[l] += info[l * ls::SELECT_RANGES + (size_t)b] < 0 ? 1 : 0;
    return LS_OK;
}

int ls_debug_prefill_in_pieces(const ls_shape* s) {
    if (check_shape(s, true, false, true)) return LS_ESHAPE;
    return ls::prefill_in_pieces(s->B * s->Hq, s->n, (int)row_blocks(s->n, s->n_hat), s->dtype, s->d) ? 1 : 0;
}

int ls_debug_score_route(const ls_shape* s, int32_t mode, int32_t positions, int32_t route[9], int64_t* begins) {
    if (!route || mode < 0 || mode > 3 || check_shape(s, false, true, false)) return LS_EINVAL;
    ls::ScoreArgs a = score_args(s);
    const int64_t any = 0;
    if (positions) a.q_pos = &any;                         // (not looked at)
    if (mode == 1) {
        Bump bp{nullptr, ls_workspace_bytes(s, 0), 0};
        window_scratch(a, s, bp);
    }
    const ls::ScoreRoute r = ls::score_route(a, s->dtype == LS_BF16, s->d, mode);
    const int32_t words[9] = {r.ranges, r.chunks, r.shares, r.folds, r.joins, r.streams, r.band_heads, r.band_rows, r.band_shares};
    memcpy(route, words, sizeof(words));
    const uint32_t units = (uint32_t)((s->n + r.unit - 1) / r.unit);
    for (int x = 0; begins && x <= r.ranges && r.ranges > 0; ++x) {
        const int64_t key = (int64_t)ls::range_begin(units, (uint32_t)r.ranges, (uint32_t)x) * r.unit;
        begins[x] = key < s->n ? key : s->n;
    }
    return LS_OK;
}

/* Debug / test hook: the group-summed retention score of the last ls_kv_compress call on this
 * context lives at the start of the third workspace block; exposed so tests can compare scores. */
int ls_debug_copy_compress_score(ls_ctx* c, const ls_shape* s, float* dst_device, void* stream) {
    if (!c || !s || !dst_device) return LS_EINVAL;
    const size_t BH = (size_t)s->B * s->Hq;
    const size_t off = up(part_floats(s) * 4) + up(BH * s->w * 2 * 4);
    const size_t bytes = (size_t)s->B * s->Hkv * (size_t)s->n * 4;
    if (off + bytes > c->ws_bytes) return LS_EWORKSPACE;
    if (hipMemcpyAsync(dst_device, c->ws + off, bytes, hipMemcpyDeviceToDevice, static_cast<hipStream_t>(stream)) != hipSuccess)
        return LS_EHIP;
    return LS_OK;
}

}  // extern "C"
