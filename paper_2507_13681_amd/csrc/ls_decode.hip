// Decode step over a compressed cache (Alg. 3, the Decoding step; Sec. 5.2): the newest token's query
// attends over the entries its KV head retained at the last retention step followed by the tokens
// generated since (Alg. 3 adds every generated token to the retained set), all of them visible:
//     out = softmax(scale * q [K_c; K_t]^T) [V_c; V_t].
//
// The step reads every retained K and V row once and does 4 d FLOP per (query head, key): it is bound
// by HBM bandwidth, at small sizes by latency.  The query heads of a KV head are the columns of the
// 16x16 MFMA tile products (NH blocks of 16), so the rows are read once for all of them.
//   decode_kernel  grid (splits, B*Hkv).  The keys of a KV head are cut into `splits` chunks of whole
//                  32-key tiles; the waves of a workgroup take the chunk's tiles in turn.  K fragments
//                  come straight from global memory (a key per lane, 64 contiguous bytes of a row per
//                  load), S^T = K Q^T, online softmax per head in a lane, P -> bf16, O^T += V^T P^T with
//                  the V^T fragments read transposed from a wave-private, swizzled LDS copy of the 32 V
//                  rows that a global -> LDS transfer filled.  A wave has 16 KB in flight, a workgroup of
//                  8 waves 128 KB: enough for its CU's share of the HBM bandwidth without prefetching
//                  across tiles.  The waves' partial results (reference, normaliser, unnormalised output)
//                  are merged through LDS; with one split that is the result, else they are written per
//                  split and the workgroup that finishes a KV head last (a counter per KV head) merges
//                  the splits.
// One launch instead of a partial and a combine kernel: a launch costs 2-4 us in the stream and 2 us of
// host time.  Merging splits costs about 3 us of memory round trips (write, counter, read), so the keys are
// spread over the waves of a workgroup first and over workgroups second.  Measured (whole call, against
// 32x32 tiles, 4 waves, two launches): B 4, 64 / 8 heads of 128, 2048 + 16 rows (34 MB) 19.2 -> 12.6 us, B 1,
// 32 / 8 heads, 16384 rows (67 MB) 33.9 -> 18.0 us, 512 + 7 rows 12.0 -> 8.0 us, of which 4.7 us are those of
// an empty kernel.  4 waves: 14.0 / 20.5 / 7.5-8.4 us; 16 waves: 14.9 / 19.5 / 9.1-10.2 us (one CU takes in no
// more than 64 bytes a clock).
// bf16 only (the transpose read is 16-bit).
#include "ls_device.h"
#include "ls_internal.h"

namespace ls {

constexpr int DEC_TILE = 32;                   // keys per wave tile
constexpr int DEC_WAVES = 8;                   // waves per workgroup
constexpr int DEC_THREADS = 64 * DEC_WAVES;

template <int D, int NH>
struct DecCfg {
    static_assert(D == 128 || D == 64, "head dimension");
    static_assert(NH == 1 || NH == 2, "16 or 32 query heads");
    static constexpr int RB = D * 2;                      // bytes per row
    static constexpr int DS = RB / 16;                    // 16-byte slots per row
    static constexpr int RPI = 64 / DS;                   // rows per transfer instruction
    static constexpr int NIV = DEC_TILE / RPI;            // transfers per V tile
    static constexpr int V_BYTES = DEC_TILE * RB;         // one wave's V stage
    static constexpr int KC = D / 32;                     // 32-wide contraction chunks of a row
    static constexpr int DB = D / 16;                     // 16-wide output blocks
    static constexpr int PS = D + 4;                      // floats of a partial result: output, reference, normaliser, 2 unused
    // slot swizzle of the staged V rows (XOR on the 16-byte slot index): the 16 rows a transpose read touches fall
    // into different banks, two per bank as its 512 bytes need anyway
    __device__ static constexpr int vswz(int row) { return D == 128 ? 2 * (row & 7) : 2 * ((row >> 1) & 3); }
};

template <int D, int NH>
__global__ __launch_bounds__(DEC_THREADS) void decode_kernel(DecodeArgs a) {
    using C = DecCfg<D, NH>;
    using T = bf16_t;
    extern __shared__ __align__(16) unsigned char dec_lds[];   // a V stage per wave; later the waves' partial results
    __shared__ int last_s;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int m16 = lane & 15, q = lane >> 4;
    const int split = blockIdx.x, bk = blockIdx.y;
    const int b = bk / a.Hkv, kvh = bk % a.Hkv;
    const int G = a.G;
    const int cnt_raw = a.cnt ? a.cnt[bk] : a.cap;             // asked for ahead of everything else
    const unsigned char* kc = reinterpret_cast<const unsigned char*>(a.kc) + (int64_t)bk * a.cap * C::RB;
    const unsigned char* vc = reinterpret_cast<const unsigned char*>(a.vc) + (int64_t)bk * a.cap * C::RB;
    const unsigned char* kt = reinterpret_cast<const unsigned char*>(a.kt) + (int64_t)bk * a.T * C::RB;
    const unsigned char* vt = reinterpret_cast<const unsigned char*>(a.vt) + (int64_t)bk * a.T * C::RB;

    unsigned char* stage = dec_lds + wv * C::V_BYTES;
    const uint32_t stage_lds = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)stage;
    const int trow = lane / C::DS, sl = lane % C::DS;          // a transfer: this lane fills slot sl of tile row RPI * i + trow
    // rows r0 .. r0 + 31 of `v` -> LDS, of `k` -> fragments; rows from `rows` on repeat the last one
    auto request_v = [&](const unsigned char* v, int r0, int rows) {
#pragma unroll
        for (int i = 0; i < C::NIV; ++i) {
            const int row = C::RPI * i + trow;
            const int r = r0 + row < rows ? r0 + row : rows - 1;
            dma16(v + (int64_t)r * C::RB + 16 * (sl ^ C::vswz(row)), stage_lds + (uint32_t)(i * 1024));
        }
    };
    bf16x8 kf[2][C::KC];                                       // keys m16 and 16 + m16 of the tile, 8 values from 32 c + 8 q on
    auto request_k = [&](const unsigned char* k, int r0, int rows) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int r = r0 + 16 * h + m16 < rows ? r0 + 16 * h + m16 : rows - 1;
            const unsigned char* krow = k + (int64_t)r * C::RB;
#pragma unroll
            for (int c = 0; c < C::KC; ++c) kf[h][c] = *reinterpret_cast<const bf16x8*>(krow + 64 * c + 16 * q);
        }
    };
    // Tiles of a KV head: first those of the retained rows, then those of the tail.  This wave's first tile is requested
    // before the count is here, as if every row of the cache were retained: right for all but a tile of the tail behind
    // a cache that is not full, which is requested again.  Rows past the count may be read then; they are masked (K)
    // and zeroed (V) below, whatever they hold.
    const int tail_tiles = (a.T + DEC_TILE - 1) / DEC_TILE;
    const int tile0 = split * a.chunk;
    int t = tile0 + wv;
    auto request_at = [&](int tile, int ctiles, int rows_c, bool v_part, bool k_part) {
        const bool tail = tile >= ctiles;
        const int r0 = DEC_TILE * (tail ? tile - ctiles : tile), rows = tail ? a.T : rows_c;
        if (v_part) request_v(tail ? vt : vc, r0, rows);
        if (k_part) request_k(tail ? kt : kc, r0, rows);
    };
    const int cap_tiles = (a.cap + DEC_TILE - 1) / DEC_TILE;
    const bool early = wv < a.chunk && t < cap_tiles + tail_tiles;
    if (early) request_at(t, cap_tiles, a.cap, true, true);

    bf16x8 qf[NH][C::KC];                                      // head 16 h + m16 of the group
#pragma unroll
    for (int h = 0; h < NH; ++h)
#pragma unroll
        for (int c = 0; c < C::KC; ++c) {
            const f32x4 z = {0.f, 0.f, 0.f, 0.f};
            qf[h][c] = __builtin_bit_cast(bf16x8, z);
            if (16 * h + m16 < G)
                qf[h][c] = *reinterpret_cast<const bf16x8*>(reinterpret_cast<const T*>(a.q) + ((int64_t)b * a.Hq + kvh * G + 16 * h + m16) * D + 32 * c + 8 * q);
        }
    int nc = cnt_raw < 0 ? 0 : cnt_raw;
    if (nc > a.cap) nc = a.cap;
    nc = __builtin_amdgcn_readfirstlane(nc);
    const int ctiles = (nc + DEC_TILE - 1) / DEC_TILE;         // tiles of this KV head: ctiles + tail_tiles
    const int tend = tile0 + a.chunk < ctiles + tail_tiles ? tile0 + a.chunk : ctiles + tail_tiles;
    if (t < tend && t >= ctiles && ctiles != cap_tiles) {
        wait_transfers();                                      // the rows asked for early have landed: the stage is free
        request_at(t, ctiles, nc, true, true);
    }
    f32x4 oacc[NH][C::DB];                                     // O^T: element r of block i is d = 16 i + 4 q + r of head m16
    float m_run[NH], l_run[NH];                                // reference in raw logit units; this lane's share of the normaliser
#pragma unroll
    for (int h = 0; h < NH; ++h) {
        m_run[h] = -INFINITY; l_run[h] = 0.f;
#pragma unroll
        for (int i = 0; i < C::DB; ++i) oacc[h][i] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    const float sc2 = a.scale_log2e;
    // transpose reads: in a block of 16 lanes lane s points at key 4q + s/4 (+ 16) and d-offset 4 (s%4) of block i, and
    // receives four keys of column d = 16 i + s
    const int vrow = 4 * q + (m16 >> 2);
    const int vbase = vrow * C::RB + 8 * (m16 & 1);
    const int vslot = (m16 >> 1) & 1;                          // 16-byte slot inside block i's 32 bytes

    for (; t < tend; t += DEC_WAVES) {
        wait_transfers();                                              // this tile's rows are here (the same wave reads them)
        const int left = t < ctiles ? nc - DEC_TILE * t : a.T - DEC_TILE * (t - ctiles);      // keys of the tile that exist
        if (left < DEC_TILE) {                                         // the V rows of masked keys meet weight 0: make them finite
#pragma unroll
            for (int i = 0; i < C::NIV; ++i)
                if (C::RPI * i + trow >= left) *reinterpret_cast<f32x4*>(stage + i * 1024 + 16 * lane) = f32x4{0.f, 0.f, 0.f, 0.f};
        }
        f32x4 s[NH][2];
#pragma unroll
        for (int h = 0; h < NH; ++h)
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                s[h][e] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int c = 0; c < C::KC; ++c)                        // s[h][e][r] = <k_{16 e + 4 q + r}, q_{head 16 h + m16}>
                    s[h][e] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[e][c], qf[h][c], s[h][e], 0, 0, 0);
            }
        const bool more = t + DEC_WAVES < tend;
        if (more) request_at(t + DEC_WAVES, ctiles, nc, false, true);
        bf16x8 pf[NH];
#pragma unroll
        for (int h = 0; h < NH; ++h) {
            float x[8], mx = -INFINITY;
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                x[r] = 16 * (r >> 2) + 4 * q + (r & 3) < left ? s[h][r >> 2][r & 3] : -INFINITY;
                mx = fmaxf(mx, x[r]);
            }
            mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
            mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
            const float m_new = fmaxf(m_run[h], mx);                   // finite: the tile holds at least one key
            const float corr = fast_exp2((m_run[h] - m_new) * sc2);
            const float mneg = -m_new * sc2;
            m_run[h] = m_new;
            float ps = 0.f;
#pragma unroll
            for (int r = 0; r < 8; ++r) { x[r] = fast_exp2(__builtin_fmaf(x[r], sc2, mneg)); ps += x[r]; }
            l_run[h] = l_run[h] * corr + ps;
            if (__ballot(corr != 1.0f) != 0ull) {
#pragma unroll
                for (int i = 0; i < C::DB; ++i) oacc[h][i] *= corr;
            }
            Frag<T> f;
            pack_frag(f, x);                                           // contraction index 8 q + r <-> key 16 (r / 4) + 4 q + r % 4
            pf[h] = f.v;
        }
#pragma unroll
        for (int i = 0; i < C::DB; ++i) {
            const unsigned char* va = stage + vbase + 16 * ((2 * i + vslot) ^ C::vswz(vrow));      // vswz(vrow + 16) is the same
            Frag<T> vf;
            load_frag_tr(vf, va, va + 16 * C::RB);
#pragma unroll
            for (int h = 0; h < NH; ++h) oacc[h][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf.v, pf[h], oacc[h][i], 0, 0, 0);
        }
        if (more) {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");         // the stage has been read
            request_at(t + DEC_WAVES, ctiles, nc, true, false);
        }
    }

    // ---- merge the waves through LDS: part[wv][head][PS]
    // (the wait: a wave whose early request lies past the count has not waited for it, and neither the compiler nor the
    // barrier does so; it could still be landing where other waves write their results)
    wait_transfers();
    __syncthreads();                                                   // every wave is done with its V stage
    float* part = reinterpret_cast<float*>(dec_lds);
    constexpr int PS = C::PS;
#pragma unroll
    for (int h = 0; h < NH; ++h) {
        float l = l_run[h] + __shfl_xor(l_run[h], 16, 64);
        l += __shfl_xor(l, 32, 64);
        if (16 * h + m16 < G) {
            float* mine = part + (wv * G + 16 * h + m16) * PS;
#pragma unroll
            for (int i = 0; i < C::DB; ++i) *reinterpret_cast<f32x4*>(mine + 16 * i + 4 * q) = oacc[h][i];
            if (q == 0) { mine[D] = m_run[h]; mine[D + 1] = l; }
        }
    }
    __syncthreads();
    bf16_t* out = reinterpret_cast<bf16_t*>(a.out) + ((int64_t)b * a.Hq + kvh * G) * D;
    float* lse = a.lse ? a.lse + (int64_t)b * a.Hq + kvh * G : nullptr;
    auto finish = [&](int head, int dd, float m, float o0, float o1, float l) {   // two output elements (dd == 0 also writes lse)
        *reinterpret_cast<uint32_t*>(out + head * D + dd) = (uint32_t)f2bf(l > 0.f ? o0 / l : 0.f) | ((uint32_t)f2bf(l > 0.f ? o1 / l : 0.f) << 16);
        if (lse && dd == 0) lse[head] = l > 0.f ? (m * sc2 + log2f(l)) * 0.69314718055994531f : -INFINITY;
    };
    float* shared_part = a.part + (int64_t)bk * a.nsplit * G * PS;     // [split][head][PS]
    const int items = G * (D / 2);                                     // two neighbouring elements of a head
    for (int idx = tid; idx < items; idx += DEC_THREADS) {
        const int head = idx / (D / 2), dd = 2 * (idx % (D / 2));
        float m = -INFINITY, o0 = 0.f, o1 = 0.f, l = 0.f;
        float2 ml[DEC_WAVES], x[DEC_WAVES];                                    // (a wave without a tile: reference -inf, zeros)
#pragma unroll
        for (int w = 0; w < DEC_WAVES; ++w) {
            const float* pw = part + (w * G + head) * PS;
            ml[w] = *reinterpret_cast<const float2*>(pw + D);
            x[w] = *reinterpret_cast<const float2*>(pw + dd);
            m = fmaxf(m, ml[w].x);
        }
#pragma unroll
        for (int w = 0; w < DEC_WAVES; ++w) {
            const float wgt = ml[w].x > -INFINITY ? fast_exp2((ml[w].x - m) * sc2) : 0.f;
            o0 += x[w].x * wgt; o1 += x[w].y * wgt;
            l += ml[w].y * wgt;
        }
        if (a.nsplit == 1) { finish(head, dd, m, o0, o1, l); continue; }
        float* dst = shared_part + ((int64_t)split * G + head) * PS;
        put_shared2(dst + dd, o0, o1);
        if (dd == 0) put_shared2(dst + D, m, l);
    }
    if (a.nsplit == 1) return;

    // ---- the last workgroup of this KV head to get here merges the splits
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");                   // this wave's part of the result has been written
    __syncthreads();
    if (tid == 0) {
        last_s = count_shared(a.done + bk) == (uint32_t)a.nsplit - 1u;
        if (last_s) clear_shared(a.done + bk);                         // for the call that uses these counters next
    }
    if (split == 0)                                                    // whatever an earlier call has left there
        for (int h = bk + tid * (int)gridDim.y; h < a.clear_heads; h += DEC_THREADS * (int)gridDim.y) clear_shared(a.done_clear + h);
    __syncthreads();
    if (!last_s) return;
    // A thread owns two elements of a head and every `subs`-th split; the subsets are added through LDS.
    const int subs = items >= DEC_THREADS ? 1 : DEC_THREADS / items;
    float2* ml = reinterpret_cast<float2*>(dec_lds);                   // [head][split] reference, normaliser
    float* add = reinterpret_cast<float*>(dec_lds) + 2 * G * a.nsplit; // [sub][item][2]
    constexpr int BATCH = 8;                                           // splits whose values are in flight together
    for (int idx0 = 0; idx0 < items; idx0 += DEC_THREADS) {
        const int idx = idx0 + (subs == 1 ? tid : tid % items), sub = subs == 1 ? 0 : tid / items;
        const bool on = idx < items && sub < subs;
        const int head = on ? idx / (D / 2) : 0, dd = on ? 2 * (idx % (D / 2)) : 0;
        const float* src = shared_part + (int64_t)head * PS + dd;
        float2 x[BATCH];
        auto fetch = [&](int s0) {
#pragma unroll
            for (int e = 0; e < BATCH; ++e) {
                const int s = s0 + e * subs;
                x[e] = get_shared2(src + (int64_t)(s < a.nsplit ? s : a.nsplit - 1) * G * PS);
            }
        };
        fetch(sub);
        if (idx0 == 0) {
            for (int i = tid; i < G * a.nsplit; i += DEC_THREADS) ml[i] = get_shared2(shared_part + ((int64_t)(i % a.nsplit) * G + i / a.nsplit) * PS + D);
            __syncthreads();
        }
        const float2* mh = ml + head * a.nsplit;
        float m = -INFINITY, o0 = 0.f, o1 = 0.f, l = 0.f;
        for (int s = 0; s < a.nsplit; ++s) m = fmaxf(m, mh[s].x);
        for (int s0 = sub; s0 < a.nsplit; s0 += BATCH * subs) {
            if (s0 != sub) fetch(s0);
#pragma unroll
            for (int e = 0; e < BATCH; ++e) {
                const int s = s0 + e * subs;
                if (s < a.nsplit && mh[s].x > -INFINITY) {
                    const float wgt = fast_exp2((mh[s].x - m) * sc2);
                    o0 += x[e].x * wgt; o1 += x[e].y * wgt;
                    l += mh[s].y * wgt;
                }
            }
        }
        if (subs > 1) {
            if (on && sub > 0) { float* p = add + 4 * ((sub - 1) * items + idx); p[0] = o0; p[1] = o1; p[2] = l; }
            __syncthreads();
            if (on && sub == 0)
                for (int u = 1; u < subs; ++u) { const float* p = add + 4 * ((u - 1) * items + idx); o0 += p[0]; o1 += p[1]; l += p[2]; }
        }
        if (on && sub == 0) finish(head, dd, m, o0, o1, l);
    }
}

template <int D, int NH>
static size_t decode_smem_t(int G, int nsplit) {
    using C = DecCfg<D, NH>;
    const size_t stages = (size_t)DEC_WAVES * C::V_BYTES;
    const size_t merge = (size_t)DEC_WAVES * G * C::PS * 4;
    const size_t splits = nsplit == 1 ? 0 : 2 * (size_t)G * nsplit * 4 + 4 * (size_t)DEC_THREADS * 4;
    const size_t m = stages > merge ? stages : merge;
    return m > splits ? m : splits;
}
size_t decode_smem_bytes(int d, int G, int nsplit) {
    if (d == 128) return G <= 16 ? decode_smem_t<128, 1>(G, nsplit) : decode_smem_t<128, 2>(G, nsplit);
    return G <= 16 ? decode_smem_t<64, 1>(G, nsplit) : decode_smem_t<64, 2>(G, nsplit);
}
size_t decode_part_floats(int d) { return (size_t)d + 4; }

// Split of the key axis: `chunk` tiles of a KV head per workgroup.  As many workgroups as the chip has compute units,
// but at least four tiles in each (512 workgroups instead of 256 cost 10 to 50 % on large caches), and no split at all while
// the waves of one workgroup get through with two tiles each or little more.  Measured, one workgroup / splits of four tiles,
// us: 8 KV heads, full caches of 14 tiles 7.7 / 7.9, 16 tiles 8.1 / 7.6, 18 tiles 8.6 / 8.0, 22 tiles 10.0 / 8.1, 34 tiles 12.8 /
// 8.4; caches filled to three quarters 15 tiles 7.7 / 8.1, 16 tiles 7.8 / 7.8, 18 tiles 8.3 / 8.1; 64 KV heads, full 16 tiles 8.2 /
// 8.7, 18 tiles 8.7 / 8.8.  The count is on the device: the line lies between what full and what partly filled caches ask for.
void decode_split(int BK, int cap, int T, int limit, int* nsplit, int* chunk) {
    const int tiles = (cap + DEC_TILE - 1) / DEC_TILE + (T + DEC_TILE - 1) / DEC_TILE;
    int want = 256 / BK;
    const int most = tiles <= 2 * DEC_WAVES + 2 ? 1 : tiles / 4;
    if (want > most) want = most;
    if (want > limit) want = limit;
    if (want < 1) want = 1;
    *chunk = (tiles + want - 1) / want;
    *nsplit = (tiles + *chunk - 1) / *chunk;
}

template <int D, int NH>
static hipError_t run_decode_t(const DecodeArgs& a, hipStream_t st) {
    const size_t smem = decode_smem_t<D, NH>(a.G, a.nsplit);
    hipLaunchKernelGGL((decode_kernel<D, NH>), dim3(a.nsplit, a.B * a.Hkv), dim3(DEC_THREADS), smem, st, a);
    return hipGetLastError();
}

hipError_t init_decode_kernels() {
    hipError_t e;
    if ((e = allow_full_lds(&decode_kernel<128, 1>)) != hipSuccess) return e;
    if ((e = allow_full_lds(&decode_kernel<128, 2>)) != hipSuccess) return e;
    if ((e = allow_full_lds(&decode_kernel<64, 1>)) != hipSuccess) return e;
    return allow_full_lds(&decode_kernel<64, 2>);
}

hipError_t run_decode(const DecodeArgs& a, int d, hipStream_t st) {
    if (d == 128) return a.G <= 16 ? run_decode_t<128, 1>(a, st) : run_decode_t<128, 2>(a, st);
    if (d == 64) return a.G <= 16 ? run_decode_t<64, 1>(a, st) : run_decode_t<64, 2>(a, st);
    return hipErrorInvalidValue;
}

}  // namespace ls
