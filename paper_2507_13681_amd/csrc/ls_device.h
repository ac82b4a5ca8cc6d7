// Device-side building blocks shared by the LoopServe kernels (gfx950 only).
//
// The tile products use the 32x32 MFMA shapes of CDNA4.  One "fragment" is the
// 8 contraction-index values a lane feeds into a 32x32x16 product: lane l holds
// row (or column) l % 32 of the operand and the eight k values 8*(l/32) .. +7 of
// the current 16-wide k chunk.  For bf16 that is one v_mfma_f32_32x32x16_bf16;
// for fp32 the same fragment is consumed by eight v_mfma_f32_32x32x2_f32, the
// i-th pairing element i of both lane halves (a permutation of k, applied to
// both operands alike, so the product is unchanged).
//
// Accumulator layout of every 32x32 product D = A * B (A is M x K, B is K x N):
//   lane l, register r (0..15) holds D[8*(r/4) + 4*(l/32) + r%4][l % 32].
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ls {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;

struct bf16_t { uint16_t bits; };   // storage type tag for bf16 tensors

template <typename T> struct Frag;
template <> struct Frag<bf16_t> { bf16x8 v; };
template <> struct Frag<float>  { float v[8]; };

template <typename T> struct Elem;
template <> struct Elem<bf16_t> { static constexpr int bytes = 2; static constexpr int per16 = 8; };
template <> struct Elem<float>  { static constexpr int bytes = 4; static constexpr int per16 = 4; };

// acc += A(32 x 16 chunk) * B(16 chunk x 32)
__device__ __forceinline__ void mma(f32x16& acc, const Frag<bf16_t>& a, const Frag<bf16_t>& b) {
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.v, b.v, acc, 0, 0, 0);
}
__device__ __forceinline__ void mma(f32x16& acc, const Frag<float>& a, const Frag<float>& b) {
#pragma unroll
    for (int i = 0; i < 8; ++i) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.v[i], b.v[i], acc, 0, 0, 0);
}

// Load the 8 consecutive elements starting at p (16-byte aligned) as a fragment.
__device__ __forceinline__ void load_frag(Frag<bf16_t>& f, const void* p) {
    f.v = *reinterpret_cast<const bf16x8*>(p);
}
__device__ __forceinline__ void load_frag(Frag<float>& f, const void* p) {
    const f32x4 a = reinterpret_cast<const f32x4*>(p)[0], b = reinterpret_cast<const f32x4*>(p)[1];
    f.v[0] = a.x; f.v[1] = a.y; f.v[2] = a.z; f.v[3] = a.w;
    f.v[4] = b.x; f.v[5] = b.y; f.v[6] = b.z; f.v[7] = b.w;
}
__device__ __forceinline__ void zero_frag(Frag<bf16_t>& f) {
    const f32x4 z = {0.f, 0.f, 0.f, 0.f};
    f.v = __builtin_bit_cast(bf16x8, z);
}
__device__ __forceinline__ void zero_frag(Frag<float>& f) {
#pragma unroll
    for (int i = 0; i < 8; ++i) f.v[i] = 0.f;
}

// float -> bf16 bits, round to nearest even (finite inputs).
__device__ __forceinline__ uint16_t f2bf(float x) {
    uint32_t u = __builtin_bit_cast(uint32_t, x);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}
__device__ __forceinline__ float bf2f(uint16_t b) {
    return __builtin_bit_cast(float, (uint32_t)b << 16);
}

// Pack 8 probabilities into a fragment (operand of the P*V product).
__device__ __forceinline__ void pack_frag(Frag<bf16_t>& f, const float* p) {
    typedef __attribute__((ext_vector_type(8))) float f32x8;
    const f32x8 x = {p[0], p[1], p[2], p[3], p[4], p[5], p[6], p[7]};
    f.v = __builtin_convertvector(x, bf16x8);          // v_cvt_pk_bf16_f32, round to nearest even
}
__device__ __forceinline__ void pack_frag(Frag<float>& f, const float* p) {
#pragma unroll
    for (int i = 0; i < 8; ++i) f.v[i] = p[i];
}

typedef __attribute__((ext_vector_type(4))) short s16x4;

// One wave-wide global -> LDS transfer (global_load_lds_dwordx4): lane l fetches 16 bytes and they land
// at LDS byte address lds + 16 * l; `lds` (and `gbase`) are wave-uniform.  Written as asm statements so
// that the compiler does not count the transfers among the memory operations it tracks: it cannot tell
// which LDS bytes a transfer fills and would make every later LDS read wait for all outstanding
// transfers, serialising a prefetch with the work on the data already there.  A kernel waits for its
// transfers itself (wait_transfers, then a barrier if other waves read the data).  M0 is listed as
// clobbered so that the compiler never keeps a value of its own in M0 across a transfer.
__device__ __forceinline__ void dma16(const unsigned char* gbase, uint32_t voff, uint32_t lds) {   // address = gbase + voff
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds), "v"(voff), "s"(gbase) : "memory", "m0");
}
__device__ __forceinline__ void dma16(const unsigned char* gptr, uint32_t lds) {                    // per-lane address
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(lds), "v"(gptr) : "memory", "m0");
}
// A wave-uniform address, told so to the compiler (which may compute it in vector registers all the same).
__device__ __forceinline__ const unsigned char* uniform_ptr(const void* p) {
    const uint64_t u = reinterpret_cast<uint64_t>(p);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)u), hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(u >> 32));
    return reinterpret_cast<const unsigned char*>(((uint64_t)hi << 32) | lo);
}
// dma16 with 4 bytes per lane, landing at lds + 4 * l.
__device__ __forceinline__ void dma4(const void* gbase, uint32_t voff, uint32_t lds) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2" ::"s"(lds), "v"(voff), "s"(gbase) : "memory", "m0");
}
// (The builtin says the same to the compiler, which does not look into asm statements: it then knows that its own loads
// have landed too.  Without it, one of them that may still be pending on some path made it wait for every outstanding
// transfer ahead of the products of each tile: 5 % of the attention kernel.)
__device__ __forceinline__ void wait_transfers() {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0x0F70);                    // vmcnt(0), the other counters unconstrained
}

// Workgroup barrier that orders LDS traffic only, and lets the wave's transfers and global accesses stay under way.
// (Nor does __syncthreads() wait for those: on gfx950 neither the barrier nor the fences around it wait for vector memory,
// apart from what the compiler puts there for its own loads, and it does not count the transfers.)  As an asm statement it
// says so to the compiler too.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// LDS transpose read of a bf16 tile stored row-major: in a block of 16 lanes, lane s addresses 4
// consecutive 16-bit values and lane L receives value L % 4 of the lanes L/4, L/4+4, L/4+8, L/4+12.
// Two reads (rows r .. and r + 8 ..) give a lane the eight contraction-index values of a fragment.
__device__ __forceinline__ void load_frag_tr(Frag<bf16_t>& f, const unsigned char* lo_addr, const unsigned char* hi_addr) {
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)(lo_addr));
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)(hi_addr));
    struct U { s16x4 a, b; } u = {lo, hi};
    f.v = __builtin_bit_cast(bf16x8, u);
}

// Results exchanged between workgroups of one launch, which may run on different XCDs, each with an L2 of its own: these
// accesses go to the memory all of them see.  A writer waits for its stores (vmcnt) before it counts itself.
__device__ __forceinline__ void put_shared(float* p, float x) { __hip_atomic_store(p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ float get_shared(const float* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void put_shared2(float* p, float x, float y) {
    __hip_atomic_store(reinterpret_cast<uint64_t*>(p), (uint64_t)__builtin_bit_cast(uint32_t, x) | ((uint64_t)__builtin_bit_cast(uint32_t, y) << 32),
                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void put_shared_word(uint64_t* p, uint32_t lo, uint32_t hi) { __hip_atomic_store(p, (uint64_t)lo | (uint64_t)hi << 32, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ float2 get_shared2(const float* p) {
    const uint64_t u = __hip_atomic_load(reinterpret_cast<const uint64_t*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return make_float2(__builtin_bit_cast(float, (uint32_t)u), __builtin_bit_cast(float, (uint32_t)(u >> 32)));
}
__device__ __forceinline__ uint32_t count_shared(uint32_t* c) { return __hip_atomic_fetch_add(c, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void clear_shared(uint32_t* c) { __hip_atomic_store(c, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// sum over the lanes to the left and this one
__device__ __forceinline__ uint32_t lanes_upto(uint32_t x) {
    int32_t s = (int32_t)x;
    s += __builtin_amdgcn_update_dpp(0, s, 0x111, 0xF, 0xF, false);       // row_shr:1, 2, 4, 8
    s += __builtin_amdgcn_update_dpp(0, s, 0x112, 0xF, 0xF, false);
    s += __builtin_amdgcn_update_dpp(0, s, 0x114, 0xF, 0xF, false);
    s += __builtin_amdgcn_update_dpp(0, s, 0x118, 0xF, 0xF, false);
    s += __builtin_amdgcn_update_dpp(0, s, 0x142, 0xA, 0xF, false);       // row_bcast15 into rows 1 and 3
    s += __builtin_amdgcn_update_dpp(0, s, 0x143, 0xC, 0xF, false);       // row_bcast31 into rows 2 and 3
    return (uint32_t)s;
}

// Sums over the sixteen waves before this one, and over all, of what each left in `red` (the sixteen in a row of lanes: a tenth of the
// instructions that a loop over them takes, which a kernel that runs through its code once has to fetch)
__device__ __forceinline__ uint32_t waves_before(const uint32_t* red, int lane, int wv, uint32_t& total) {
    int32_t s = (int32_t)red[lane & 15];
    s += __builtin_amdgcn_update_dpp(0, s, 0x111, 0xF, 0xF, false);       // row_shr:1, 2, 4, 8
    s += __builtin_amdgcn_update_dpp(0, s, 0x112, 0xF, 0xF, false);
    s += __builtin_amdgcn_update_dpp(0, s, 0x114, 0xF, 0xF, false);
    s += __builtin_amdgcn_update_dpp(0, s, 0x118, 0xF, 0xF, false);
    total = (uint32_t)__builtin_amdgcn_readlane(s, 15);
    return wv > 0 ? (uint32_t)__builtin_amdgcn_readlane(s, wv - 1) : 0u;
}
// Sum / largest over the wave, in every lane, as halves of 32, 16, 8, 4, 2 and 1 lanes put together one after the other.  (Where the halves of a
// row agree already, row_ror:4 brings what lane ^ 4 has.  Six shuffles through LDS wait a hundred cycles each.)
template <typename F>
__device__ __forceinline__ float wave_join(float x, F f) {
    auto u = [](float v) { return __builtin_bit_cast(uint32_t, v); };
    auto fl = [](uint32_t v) { return __builtin_bit_cast(float, v); };
    const auto h = __builtin_amdgcn_permlane32_swap(u(x), u(x), false, false);
    x = f(fl((uint32_t)h[0]), fl((uint32_t)h[1]));
    const auto q = __builtin_amdgcn_permlane16_swap(u(x), u(x), false, false);
    x = f(fl((uint32_t)q[0]), fl((uint32_t)q[1]));
    x = f(x, fl((uint32_t)__builtin_amdgcn_update_dpp(0, (int)u(x), 0x128 /* row_ror:8 */, 0xF, 0xF, false)));
    x = f(x, fl((uint32_t)__builtin_amdgcn_update_dpp(0, (int)u(x), 0x124 /* row_ror:4 */, 0xF, 0xF, false)));
    x = f(x, fl((uint32_t)__builtin_amdgcn_update_dpp(0, (int)u(x), 0x4E /* quad_perm 2,3,0,1 */, 0xF, 0xF, false)));
    return f(x, fl((uint32_t)__builtin_amdgcn_update_dpp(0, (int)u(x), 0xB1 /* quad_perm 1,0,3,2 */, 0xF, 0xF, false)));
}
__device__ __forceinline__ float wave_sum(float x) { return wave_join(x, [](float a, float b) { return a + b; }); }
__device__ __forceinline__ float wave_largest(float x) { return wave_join(x, [](float a, float b) { return fmaxf(a, b); }); }

__device__ __forceinline__ float to_float(bf16_t x) { return bf2f(x.bits); }
__device__ __forceinline__ float to_float(float x) { return x; }

__device__ __forceinline__ float xor32(float x) { return __shfl_xor(x, 32, 64); }

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// Key row `key` (0..63 inside a tile) sits at this column of the transposed V tile,
// so that the 8 keys one lane half needs for a P*V chunk are contiguous:
// bits 2 and 3 of the key index are swapped.
__device__ __forceinline__ int vt_col(int key) {
    return (key & ~12) | ((key & 8) >> 1) | ((key & 4) << 1);
}

}  // namespace ls
