// rd_device.h -- device helpers shared by every kernel file (gfx950, wave64).
//
// The per-voxel update lives here once (rd_update) so that every kernel variant
// (block edge 4 or 8, batched, graph-replayed, solver, adjoint) performs the same
// FP32 operations in the same order and therefore gives bitwise-identical results.
// Kernel files are compiled with -ffp-contract=off; fused multiply-adds are
// explicit.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "rd_internal.h"

// ---- storage types ----------------------------------------------------------
// FP32 storage, BF16 storage (uint16 bit pattern, round-to-nearest-even on store)
// and FP16 storage (IEEE binary16, RNE on store).  Arithmetic is always FP32.
struct bf16_t {
    uint16_t bits;
};

__device__ __forceinline__ float rd_ld(const float *p, int64_t i) { return p[i]; }
__device__ __forceinline__ float rd_ld(const bf16_t *p, int64_t i)
{
    return __uint_as_float((uint32_t)p[i].bits << 16);
}
__device__ __forceinline__ float rd_ld(const _Float16 *p, int64_t i) { return (float)p[i]; }

// BF16 round to nearest even; NaN stays NaN (quiet bit set).  One conversion instruction
// of gfx950, equal to adding 0x7fff + (bit 16) to the FP32 pattern and cutting its lower half
// on all 2^32 patterns.
__device__ __forceinline__ uint16_t bf16_rne(float v) { return __builtin_bit_cast(uint16_t, (__bf16)v); }

// FP32 fields are streamed (written once per step, read by the next step), so their
// stores are nontemporal (measured faster on the 512^3 soil volume).
__device__ __forceinline__ void rd_st(float *p, int64_t i, float v) { __builtin_nontemporal_store(v, p + i); }
__device__ __forceinline__ void rd_st(bf16_t *p, int64_t i, float v) { p[i].bits = bf16_rne(v); }
__device__ __forceinline__ void rd_st(_Float16 *p, int64_t i, float v) { p[i] = (_Float16)v; }
// The value a round-to-nearest store into T holds when read back.
template <typename T> __device__ __forceinline__ float rd_round(float v);
template <> __device__ __forceinline__ float rd_round<float>(float v) { return v; }
template <> __device__ __forceinline__ float rd_round<bf16_t>(float v)
{
    return __uint_as_float((uint32_t)bf16_rne(v) << 16);
}
template <> __device__ __forceinline__ float rd_round<_Float16>(float v) { return (float)(_Float16)v; }

// Plain (cached) store with round to nearest, for vectors that are read again soon
// (the solver's).
__device__ __forceinline__ void rd_st_keep(float *p, int64_t i, float v) { p[i] = v; }
__device__ __forceinline__ void rd_st_keep(bf16_t *p, int64_t i, float v) { p[i].bits = bf16_rne(v); }
__device__ __forceinline__ void rd_st_keep(_Float16 *p, int64_t i, float v) { p[i] = (_Float16)v; }

// ---- predicated loads ---------------------------------------------------------
// A kernel that skips inactive voxels loads raw storage words under a predicate
// (ld_raw, 0 where the predicate is false) and converts them to FP32 only after all of
// its loads are issued (from_raw).  The conversion of BF16 / FP16 words is opaque
// inline asm: written as plain C it is folded into each predicated load's branch,
// which then waits for its own load, so the loads would no longer overlap.
__device__ __forceinline__ float ld_raw(const float *p, int64_t i, bool pred)
{
    return pred ? p[i] : 0.0f;
}
__device__ __forceinline__ uint32_t ld_raw(const bf16_t *p, int64_t i, bool pred)
{
    return pred ? (uint32_t)p[i].bits : 0u;
}
__device__ __forceinline__ uint32_t ld_raw(const _Float16 *p, int64_t i, bool pred)
{
    return pred ? (uint32_t)__builtin_bit_cast(uint16_t, p[i]) : 0u;
}
// unpredicated forms, for several loads under one predicate
__device__ __forceinline__ float ld_raw(const float *p, int64_t i) { return p[i]; }
__device__ __forceinline__ uint32_t ld_raw(const bf16_t *p, int64_t i) { return (uint32_t)p[i].bits; }
__device__ __forceinline__ uint32_t ld_raw(const _Float16 *p, int64_t i)
{
    return (uint32_t)__builtin_bit_cast(uint16_t, p[i]);
}
template <typename T> struct RawOf { typedef uint32_t type; };
template <> struct RawOf<float> { typedef float type; };

template <typename T> __device__ __forceinline__ float from_raw(typename RawOf<T>::type r);
template <> __device__ __forceinline__ float from_raw<float>(float r) { return r; }
template <> __device__ __forceinline__ float from_raw<bf16_t>(uint32_t r)
{
    float f;  // BF16 is the upper half of an FP32 pattern
    asm("v_lshlrev_b32 %0, 16, %1" : "=v"(f) : "v"(r));
    return f;
}
template <> __device__ __forceinline__ float from_raw<_Float16>(uint32_t r)
{
    float f;  // exact FP16 -> FP32 conversion of the low half
    asm("v_cvt_f32_f16 %0, %1" : "=v"(f) : "v"(r));
    return f;
}

// ---- store granularity ------------------------------------------------------
// The step kernels write a slot when any voxel of its aligned sector of
// RD_STORE_SECTOR bytes is active; the inactive slots of such a sector store the 0
// they already hold.  Sectors without an active voxel are never written, and the
// memory side only ever sees whole sectors (no partially written ones).
#ifndef RD_STORE_SECTOR
#define RD_STORE_SECTOR 128
#endif
// W: a 64-slot activity word, bit: the slot's bit in it (slots are consecutive in
// memory within the word).
template <typename T>
__device__ __forceinline__ bool sector_active(uint64_t W, int bit)
{
    // slots per sector, at most the 64 slots of one activity word
    constexpr int V = RD_STORE_SECTOR / (int)sizeof(T) < 64 ? RD_STORE_SECTOR / (int)sizeof(T) : 64;
    static_assert(V >= 1 && (V & (V - 1)) == 0, "sector of 1..64 slots");
    if constexpr (V == 64) return W != 0ull;
    else return ((W >> (bit & ~(V - 1))) & ((1ull << V) - 1ull)) != 0ull;
}

// Wave-level forms for the one-wave-per-block kernels, where slot bit l of a plane
// word belongs to lane l and the word is wave-uniform: lane_bit gives lane l bit l of
// W (the word becomes the execution mask; no per-lane shift), sector_lanes the
// uniform mask of the lanes whose sector holds an active slot (scalar ops only).
__device__ __forceinline__ bool lane_bit(uint64_t W) { return __builtin_amdgcn_inverse_ballot_w64(W); }
template <typename T>
__device__ __forceinline__ uint64_t sector_lanes(uint64_t W)
{
    constexpr int V = RD_STORE_SECTOR / (int)sizeof(T) < 64 ? RD_STORE_SECTOR / (int)sizeof(T) : 64;
    if constexpr (V == 64) {
        return W != 0ull ? ~0ull : 0ull;
    } else if constexpr (V == 32) {
        // by halves (the readfirstlane keeps them 32-bit: a compare of the 64-bit word would go
        // to the vector unit)
        const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)W);
        const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(W >> 32));
        return (uint64_t)(hi != 0u ? ~0u : 0u) << 32 | (lo != 0u ? ~0u : 0u);
    } else {
        constexpr uint64_t ONE = (1ull << V) - 1ull;
        uint64_t m = 0ull;
#pragma unroll
        for (int s = 0; s < 64; s += V) m |= ((W >> s) & ONE) != 0ull ? ONE << s : 0ull;
        return m;
    }
}

// ---- addressing -----------------------------------------------------------------
// p advanced by a 32-bit byte offset: a wave-uniform base plus a zero-extended 32-bit
// offset, the form of a global access with a scalar base and a 32-bit vector offset (no
// 64-bit address arithmetic per access).  The offsets fit: a compact species buffer holds
// fewer than 2^30 values, and block-layout offsets stay inside one block's slab.
template <typename T>
__device__ __forceinline__ T *at_byte(T *p, uint32_t off)
{
    return (T *)((char *)p + (uint64_t)off);
}
template <typename T>
__device__ __forceinline__ const T *at_byte(const T *p, uint32_t off)
{
    return (const T *)((const char *)p + (uint64_t)off);
}
// A wave-uniform pointer pinned to scalar registers, so that the compiler keeps it as the
// scalar base of the accesses above instead of folding it into each 64-bit vector address.
// (The field buffers are device memory: the pointer is rebuilt in the global address
// space, so the accesses stay global ones.)
template <typename T>
__device__ __forceinline__ T *uniform_ptr(T *p)
{
    typedef __attribute__((address_space(1))) T GT;
    const uint64_t v = (uint64_t)p;
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return (T *)(GT *)(((uint64_t)hi << 32) | lo);
}

// ---- stochastic rounding --------------------------------------------------
// 32-bit finaliser of MurmurHash3 (Appleby): a bijective avalanche mix, used as
// a counter-based generator keyed by (slot, species, step, seed).
__device__ __forceinline__ uint32_t mix32(uint32_t x)
{
    x ^= x >> 16;
    x *= 0x85ebca6bu;
    x ^= x >> 13;
    x *= 0xc2b2ae35u;
    x ^= x >> 16;
    return x;
}

// The random bits of a store come in layers so that a kernel spends little per voxel:
// a key per (step, seed), wave-uniform; a column word from the key and the voxel's
// (x, y) column in its box and a plane word from the key and its z plane (so the bits
// do not depend on the block layout, and a kernel that walks a z-column hashes the
// column once and each plane once per wave); their XOR, finalised by one
// xorshift-multiply-xorshift round (the first half of the MurmurHash3 finaliser), is the
// voxel's 32-bit word; 16 bits per species out of it (species 2 and 3 mix the voxel word
// once more).  For a fixed voxel the word is a bijection of the uniformly distributed
// column-plane XOR, so its bits are uniform over the steps' keys.
__device__ __forceinline__ uint32_t sr_key(uint32_t step, uint32_t seed)
{
    return mix32(step ^ mix32(seed + 0x9e3779b9u));
}
__device__ __forceinline__ uint32_t sr_column(const GeomInfo &g, int gx, int gy, uint32_t key)
{
    return mix32(((uint32_t)gy * (uint32_t)g.nx + (uint32_t)gx) ^ key);
}
__device__ __forceinline__ uint32_t sr_plane(int gz, uint32_t key)
{
    return mix32((uint32_t)gz ^ mix32(key ^ 0x3c6ef372u));
}
__device__ __forceinline__ uint32_t sr_combine(uint32_t column, uint32_t plane)
{
    uint32_t x = column ^ plane;
    x ^= x >> 16;
    x *= 0x85ebca6bu;
    x ^= x >> 13;
    return x;
}
__device__ __forceinline__ uint32_t sr_voxel(const GeomInfo &g, int gx, int gy, int gz, uint32_t key)
{
    return sr_combine(sr_column(g, gx, gy, key), sr_plane(gz, key));
}
__device__ __forceinline__ uint32_t sr_species(uint32_t h, int species)
{
    const uint32_t w = species < 2 ? h : mix32(h ^ 0x165667b1u);
    return (species & 1) ? (w >> 16) : (w & 0xffffu);
}

// Store with stochastic rounding: round up with probability equal to the distance
// from the lower neighbour, in units of the storage spacing (unbiased on average).
// Both forms add random bits below the cut of the FP32 pattern and truncate there, so
// the magnitude rounds up exactly when the added bits carry across the cut; no branches.
__device__ __forceinline__ uint16_t bf16_sr(float v, uint32_t rnd)
{
    // BF16 is the upper half of the FP32 pattern: 16 random bits below the cut round the
    // magnitude up with probability (low bits) / 2^16; infinities stay, a NaN stays a (quiet)
    // NaN.  The conversion instruction takes the 16 bits from the upper half of its operand
    // and equals that sum on all 2^32 patterns.
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    const bf16x2 r = __builtin_amdgcn_cvt_sr_bf16_f32(bf16x2{}, v, rnd << 16, false);
    return __builtin_bit_cast(uint16_t, r[0]);
}

// FP16 in software: FP16 keeps 10 mantissa bits down to 2^-14 (13 FP32 bits below its cut)
// and a fixed spacing of 2^-24 below (d = 126 - biased exponent bits below the cut, up to
// 23); d random bits (the 16 given, shifted into the top of the d) are added to the
// magnitude's pattern and the low d bits cleared, which leaves a multiple of the FP16
// spacing (a carry into the exponent is the next power of two).  Below 2^-24 the result is
// 2^-24 with probability |v| / 2^-24, else 0.  Infinities and NaNs convert as they are.
__device__ __forceinline__ _Float16 f16_sr_any(float v, uint32_t rnd)
{
    const uint32_t u = __float_as_uint(v);
    const uint32_t ua = u & 0x7fffffffu;
    const int eb = (int)(ua >> 23);
    const int d = min(max(126 - eb, 13), 23);
    const uint32_t r = ((rnd & 0xffffu) << 16) >> (32 - d);
    uint32_t m = (ua + r) & (0xffffffffu << d);
    if (eb < 103) m = (float)(rnd & 0xffffu) < __uint_as_float(ua) * 0x1p40f ? 0x33800000u : 0u;
    const float q = __uint_as_float(m | (u & 0x80000000u));
    return (_Float16)(eb == 255 ? v : q);
}
// The conversion instruction (random bits in the upper half of its operand) rounds every
// value of FP16's normal range like f16_sr_any (checked on all of them); a wave that holds
// another value (other than 0) takes the software form.
__device__ __forceinline__ _Float16 f16_sr(float v, uint32_t rnd)
{
    typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
    const uint32_t ua = __float_as_uint(v) & 0x7fffffffu;
    if (__any(ua - 0x38800000u >= 0x477fe000u - 0x38800000u && ua != 0u)) return f16_sr_any(v, rnd);
    return __builtin_amdgcn_cvt_sr_f16_f32(f16x2{}, v, rnd << 16, false)[0];
}

__device__ __forceinline__ void rd_st_sr(float *p, int64_t i, float v, uint32_t)
{
    __builtin_nontemporal_store(v, p + i);
}
__device__ __forceinline__ void rd_st_sr(bf16_t *p, int64_t i, float v, uint32_t rnd)
{
    p[i].bits = bf16_sr(v, rnd);
}
__device__ __forceinline__ void rd_st_sr(_Float16 *p, int64_t i, float v, uint32_t rnd)
{
    p[i] = f16_sr(v, rnd);
}

// ---- paired access: two x-adjacent slots (index i even) in one 8- or 4-byte access
typedef _Float16 half2_t __attribute__((ext_vector_type(2)));

__device__ __forceinline__ void rd_ld2(const float *p, int64_t i, float &a, float &b)
{
    const float2 v = *reinterpret_cast<const float2 *>(p + i);
    a = v.x;
    b = v.y;
}
__device__ __forceinline__ void rd_ld2(const bf16_t *p, int64_t i, float &a, float &b)
{
    const uint32_t u = *reinterpret_cast<const uint32_t *>(p + i);
    a = __uint_as_float(u << 16);
    b = __uint_as_float(u & 0xffff0000u);
}
__device__ __forceinline__ void rd_ld2(const _Float16 *p, int64_t i, float &a, float &b)
{
    const half2_t v = *reinterpret_cast<const half2_t *>(p + i);
    a = (float)v.x;
    b = (float)v.y;
}

// Store a pair; sr selects stochastic rounding with the per-slot random words r0, r1.
__device__ __forceinline__ void rd_st2(float *p, int64_t i, float a, float b, bool, uint32_t,
                                       uint32_t)
{
    *reinterpret_cast<float2 *>(p + i) = make_float2(a, b);
}
__device__ __forceinline__ void rd_st2(bf16_t *p, int64_t i, float a, float b, bool sr, uint32_t r0,
                                       uint32_t r1)
{
    const uint32_t lo = sr ? bf16_sr(a, r0) : bf16_rne(a);
    const uint32_t hi = sr ? bf16_sr(b, r1) : bf16_rne(b);
    *reinterpret_cast<uint32_t *>(p + i) = lo | (hi << 16);
}
__device__ __forceinline__ void rd_st2(_Float16 *p, int64_t i, float a, float b, bool sr,
                                       uint32_t r0, uint32_t r1)
{
    half2_t v;
    v.x = sr ? f16_sr(a, r0) : (_Float16)a;
    v.y = sr ? f16_sr(b, r1) : (_Float16)b;
    *reinterpret_cast<half2_t *>(p + i) = v;
}

// ---- compact layout (B = 8) --------------------------------------------------
// A block stores only its active voxels, in slot order, starting at cbase[b]; the
// plane prefix counts sit in words 14-15 of the block's mask record.
// Number of set bits of the wave-uniform word W in the lanes below this one.
__device__ __forceinline__ uint32_t lanes_below(uint64_t W)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(W >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)W, 0u));
}
// Active slots below plane z of a block (from its mask record).
__device__ __forceinline__ uint32_t plane_prefix(const uint64_t *rec, int z)
{
    return (uint32_t)(rec[14 + (z >> 2)] >> (16 * (z & 3))) & 0xffffu;
}
// Element index of (active) slot `slot` of block b: block-major (cbase NULL) or compact.
__device__ __forceinline__ int64_t slot_index8(const uint32_t *cbase, const uint64_t *mask, int64_t b,
                                               int slot)
{
    if (!cbase) return b * 512 + slot;
    const uint64_t *rec = mask + b * 16;
    const int z = slot >> 6, bit = slot & 63;
    const uint64_t below = bit ? (rec[z] & (~0ull >> (64 - bit))) : 0ull;
    return (int64_t)cbase[b] + plane_prefix(rec, z) + (uint32_t)__popcll(below);
}

// ---- block geometry helpers -------------------------------------------------
template <int B>
struct Blk {
    static constexpr int NS = B * B * B;   // slots per block
    static constexpr int E = B + 2;        // tile edge with halo
    static constexpr int TL = E * E * E;   // tile size (corners unused)
    static constexpr int MW = mask_words(B);
    __device__ static __forceinline__ int tidx(int lx, int ly, int lz)
    {
        return ((lz + 1) * E + (ly + 1)) * E + (lx + 1);
    }
};

// Own active bit of slot s in a mask record.
template <int B>
__device__ __forceinline__ bool own_bit(const uint64_t *rec, int s)
{
    if constexpr (B == 8) return (rec[s >> 6] >> (s & 63)) & 1ull;
    else return (rec[0] >> s) & 1ull;
}

// Face bit `bit` of face f (the neighbour voxel across that face is active).
template <int B>
__device__ __forceinline__ bool face_bit(const uint64_t *rec, int f, int bit)
{
    if constexpr (B == 8) return (rec[8 + f] >> bit) & 1ull;
    else {
        const int w = f < 4 ? 1 : 2;
        const int sh = f < 4 ? 16 * f : 16 * (f - 4);
        return (rec[w] >> (sh + bit)) & 1ull;
    }
}

// Six neighbour activity bits (bit d for direction d in -x,+x,-y,+y,-z,+z order)
// and the wall count (in-box inactive neighbours) of slot (lx,ly,lz) at global
// position (gx,gy,gz) in a box nx*ny*nz.
template <int B>
__device__ __forceinline__ unsigned nb_bits(const uint64_t *rec, int lx, int ly, int lz, int gx,
                                            int gy, int gz, int nx, int ny, int nz, int *nwall)
{
    const int s = (lz * B + ly) * B + lx;
    unsigned m = 0;
    m |= (lx > 0 ? own_bit<B>(rec, s - 1) : face_bit<B>(rec, 0, lz * B + ly)) ? 1u : 0u;
    m |= (lx < B - 1 ? own_bit<B>(rec, s + 1) : face_bit<B>(rec, 1, lz * B + ly)) ? 2u : 0u;
    m |= (ly > 0 ? own_bit<B>(rec, s - B) : face_bit<B>(rec, 2, lz * B + lx)) ? 4u : 0u;
    m |= (ly < B - 1 ? own_bit<B>(rec, s + B) : face_bit<B>(rec, 3, lz * B + lx)) ? 8u : 0u;
    m |= (lz > 0 ? own_bit<B>(rec, s - B * B) : face_bit<B>(rec, 4, ly * B + lx)) ? 16u : 0u;
    m |= (lz < B - 1 ? own_bit<B>(rec, s + B * B) : face_bit<B>(rec, 5, ly * B + lx)) ? 32u : 0u;
    unsigned inbox = 0;
    inbox |= gx > 0 ? 1u : 0u;
    inbox |= gx < nx - 1 ? 2u : 0u;
    inbox |= gy > 0 ? 4u : 0u;
    inbox |= gy < ny - 1 ? 8u : 0u;
    inbox |= gz > 0 ? 16u : 0u;
    inbox |= gz < nz - 1 ? 32u : 0u;
    *nwall = __popc(inbox & ~m);
    return m;
}

// Is a voxel at (gx,gy,gz) on a Dirichlet face plane of a species (dir bits)?
__device__ __forceinline__ bool on_dirichlet(uint32_t dir, int gx, int gy, int gz, int nx, int ny,
                                             int nz)
{
    return ((dir & 1u) && gx == 0) || ((dir & 2u) && gx == nx - 1) ||
           ((dir & 4u) && gy == 0) || ((dir & 8u) && gy == ny - 1) ||
           ((dir & 16u) && gz == 0) || ((dir & 32u) && gz == nz - 1);
}

// The FTCS update of one free voxel of one species (see rd.h):
//   lap = sum over active neighbours q of (c_q - c_p)
//   c'  = c + alpha*lap - (beta + gamma*n_wall)*c + sum_b K_b c_b
// Every caller stages inactive and missing neighbours as exactly 0 (inactive slots
// hold 0 in every field buffer), so the sum over the active neighbours is the sum
// of all six values, and the mirror rule enters through the active count:
//   lap = (((((n_-x + n_+x) + n_-y) + n_+y) + n_-z) + n_+z) - popc(nbm) * c_p
// (one rounding order for every kernel; 6 operations instead of 18).
// The increment  alpha lap - (beta + gamma n_wall) c + sum_b K_b c_b  is formed first and
// added to c once, so c is rounded once per step (forming c + alpha lap and then applying
// each term to it rounded c up to four times).  DTH (FP32 storage with stochastic
// rounding): `dith` (fp32_dither) is added to the increment before that final addition.
// rd_update_n takes the active-neighbour count and the wall count as floats (exact small
// integers), rd_update the neighbour bits; both round identically.
// self: the species' own index, whose K is 0 (a reaction's product is another species).
template <int S, bool DTH = false>
__device__ __forceinline__ float rd_update_n(float uc, const float nbv[6], float nact, float nwall,
                                             const SpeciesCoef &k, const float *cen, int self, float dith = 0.0f)
{
    float sum = nbv[0];
#pragma unroll
    for (int d = 1; d < 6; ++d) sum = sum + nbv[d];
    const float lap = fmaf(-nact, uc, sum);
    float inc = k.alpha * lap;
    const float loss = fmaf(k.gamma, nwall, k.beta);
    inc = fmaf(-loss, uc, inc);
#pragma unroll
    for (int b = 0; b < S; ++b)
        if (b != self) inc = fmaf(k.K[b], cen[b], inc);
    if constexpr (DTH) inc = inc + dith;
    return uc + inc;
}
template <int S, bool DTH = false>
__device__ __forceinline__ float rd_update(float uc, const float nbv[6], unsigned nbm, int nwall,
                                           const SpeciesCoef &k, const float *cen, int self, float dith = 0.0f)
{
    return rd_update_n<S, DTH>(uc, nbv, (float)__popc(nbm & 63u), (float)nwall, k, cen, self, dith);
}

// Stochastic rounding of FP32 values: a dither (u - 1/2) ulp(c), u in [0, 1) from 16
// random bits, added to the increment makes the round-to-nearest of c + increment + dither
// equal c + increment on average.  Without it, increments below half an ulp of c are lost
// at every step, and a field close to its steady state stops converging about
// (ulp / 2) / (dt * slowest decay rate) away from it.  0 for zero and subnormal c.
__device__ __forceinline__ float fp32_dither(float uc, uint32_t bits16)
{
    // 2^-23 (1 + u) with the 16 bits as the leading mantissa bits, minus 1.5 * 2^-23, is
    // (u - 1/2) 2^-23 exactly; times the power of two of c (c's exponent bits) it is
    // (u - 1/2) ulp(c)
    const float v = __uint_as_float(0x34000000u | (bits16 << 7)) - 0x1.8p-23f;
    return v * __uint_as_float(__float_as_uint(uc) & 0x7f800000u);
}

// Linear index of a voxel in its (nz, ny, nx) box: the key of the stochastic-rounding
// hash, so the random bits do not depend on the block layout.
__device__ __forceinline__ int64_t voxel_id(const GeomInfo &g, int gx, int gy, int gz)
{
    return g.dense0 + ((int64_t)gz * g.ny + gy) * g.nx + gx;
}

// Bit d set: the voxel lies on box face d (-x, +x, -y, +y, -z, +z).
__device__ __forceinline__ unsigned box_faces(const GeomInfo &g, int gx, int gy, int gz)
{
    return (gx == 0 ? 1u : 0u) | (gx == g.nx - 1 ? 2u : 0u) | (gy == 0 ? 4u : 0u) |
           (gy == g.ny - 1 ? 8u : 0u) | (gz == 0 ? 16u : 0u) | (gz == g.nz - 1 ? 32u : 0u);
}

// Block position of list entry b.
__device__ __forceinline__ void block_pos(const BlockInfo &bi, int *bx, int *by, int *bz, int *gid)
{
    *bx = bi.xy & 0xffff;
    *by = (bi.xy >> 16) & 0xffff;
    *bz = bi.zg & 0xffff;
    *gid = (bi.zg >> 16) & 0xffff;
}

// Slot of a neighbour block that lies across face f at face coordinates (u, v),
// and the tile index it is staged at.
template <int B>
__device__ __forceinline__ void halo_slot(int f, int u, int v, int *nslot, int *tix)
{
    using K = Blk<B>;
    switch (f) {
    case 0: *nslot = (v * B + u) * B + (B - 1); *tix = ((v + 1) * K::E + (u + 1)) * K::E + 0; break;
    case 1: *nslot = (v * B + u) * B + 0; *tix = ((v + 1) * K::E + (u + 1)) * K::E + (B + 1); break;
    case 2: *nslot = (v * B + (B - 1)) * B + u; *tix = ((v + 1) * K::E + 0) * K::E + (u + 1); break;
    case 3: *nslot = (v * B + 0) * B + u; *tix = ((v + 1) * K::E + (B + 1)) * K::E + (u + 1); break;
    case 4: *nslot = ((B - 1) * B + v) * B + u; *tix = ((0) * K::E + (v + 1)) * K::E + (u + 1); break;
    default: *nslot = (0 * B + v) * B + u; *tix = ((B + 1) * K::E + (v + 1)) * K::E + (u + 1); break;
    }
}

// Generic per-block workgroup shape: B = 8 one block per 256-thread workgroup (two
// voxels per thread); B = 4 four blocks per workgroup, one wave per block.
template <int B>
struct Cfg {
    static constexpr int BPW = B == 8 ? 1 : 4;    // blocks per workgroup
    static constexpr int TPB = 256 / BPW;         // threads per block
    static constexpr int VPT = Blk<B>::NS / TPB;  // voxels per thread
};

// The group of blocks of a workgroup in the order of rd_xcd_order.
__device__ __forceinline__ int map_group(int wg, int order)
{
    if (order > 0) return (wg & 7) * order + (wg >> 3);
    if (order == 0) return wg;
    const int run = -order, r = wg & (8 * run - 1);
    return wg - r + (r & 7) * run + (r >> 3);
}

// Stage S fields (species-major, sstride apart) of block b and its six face halos
// into an LDS tile of (B+2)^3 words per field (FP32).  Missing neighbours give 0.
template <typename T, int B>
__device__ __forceinline__ void stage_tile(float (*tile)[Blk<B>::TL], const T *c, int64_t sstride,
                                           int S, int b, const BlockInfo &bi, int lt, bool valid)
{
    using K = Blk<B>;
    using C = Cfg<B>;
    if (!valid) return;
    const int64_t base = (int64_t)b * K::NS;
    for (int s = 0; s < S; ++s) {
#pragma unroll
        for (int k = 0; k < C::VPT; ++k) {
            const int slot = lt + k * C::TPB;
            const int lx = slot % B, ly = (slot / B) % B, lz = slot / (B * B);
            tile[s][K::tidx(lx, ly, lz)] = rd_ld(c, s * sstride + base + slot);
        }
    }
    for (int h = lt; h < 6 * B * B; h += C::TPB) {
        const int f = h / (B * B);
        const int r = h % (B * B);
        int nslot, tix;
        halo_slot<B>(f, r % B, r / B, &nslot, &tix);
        const int n = bi.nbr[f];
        for (int s = 0; s < S; ++s)
            tile[s][tix] = n >= 0 ? rd_ld(c, s * sstride + (int64_t)n * K::NS + nslot) : 0.0f;
    }
}

// ---- activity of the neighbours, as lane masks (B = 8 column kernels) ------------
// Bit r * 8 + c of x at bit c * 8 + r.
__device__ __forceinline__ uint64_t transpose8x8(uint64_t x)
{
    // bit r*8+c -> bit c*8+r: delta swaps of 1x1, 2x2 and 4x4 sub-blocks
    uint64_t t = (x ^ (x >> 7)) & 0x00AA00AA00AA00AAull;
    x = x ^ t ^ (t << 7);
    t = (x ^ (x >> 14)) & 0x0000CCCC0000CCCCull;
    x = x ^ t ^ (t << 14);
    t = (x ^ (x >> 28)) & 0x00000000F0F0F0F0ull;
    x = x ^ t ^ (t << 28);
    return x;
}
// The mask record of a block in scalar registers; the -x / +x face words also transposed
// (bit y * 8 + z).
struct BlockMasks {
    uint64_t Wo[8], Wf[6], tx0, tx1;
    __device__ __forceinline__ void load(const uint64_t *rec)
    {
#pragma unroll
        for (int z = 0; z < 8; ++z) Wo[z] = rec[z];
#pragma unroll
        for (int f = 0; f < 6; ++f) Wf[f] = rec[8 + f];
        tx0 = transpose8x8(Wf[0]);
        tx1 = transpose8x8(Wf[1]);
    }
    // the active lanes of plane z whose neighbour in direction d (-x, +x, -y, +y, -z, +z) is
    // active too.  On the scalar unit; the vector unit then needs one select per neighbour
    // where testing code bits takes three instructions.
    __device__ __forceinline__ uint64_t pair(int z, int d) const
    {
        constexpr uint64_t COL0 = 0x0101010101010101ull;  // lanes with x = 0
        const uint64_t P = Wo[z];
        switch (d) {
        case 0: return P & (((P << 1) & ~COL0) | ((tx0 >> z) & COL0));
        case 1: return P & (((P >> 1) & ~(COL0 << 7)) | (((tx1 >> z) & COL0) << 7));
        case 2: return P & ((P << 8) | ((Wf[2] >> (8 * z)) & 0xffull));
        case 3: return P & ((P >> 8) | (((Wf[3] >> (8 * z)) & 0xffull) << 56));
        case 4: return P & (z > 0 ? Wo[z > 0 ? z - 1 : 0] : Wf[4]);
        default: return P & (z < 7 ? Wo[z < 7 ? z + 1 : 7] : Wf[5]);
        }
    }
};

// ---- values handed to another workgroup of the same launch ------------------------
// v at p, performed where every XCD sees it when this returns (an exchange, whose old value
// is waited for); get_agent reads it there.  A count raised afterwards (arrive_agent, relaxed)
// then needs no release fence, which would write back the dirty lines of the XCD's L2.
// That order is this hardware's, not the memory model's, where relaxed operations on two
// addresses have none: it holds for values written by put_agent and read by get_agent only,
// in the wave that raises the count and after the count was read.  An ordinary store or load
// on either side needs the release and acquire.
__device__ __forceinline__ void put_agent(double *p, double v)
{
    const double old = __hip_atomic_exchange(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("" ::"v"(old) : "memory");
}
__device__ __forceinline__ double get_agent(const double *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint32_t arrive_agent(uint32_t *count)
{
    return __hip_atomic_fetch_add(count, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Wave-level FP64 sum in a fixed butterfly order (deterministic): partners 32, 16, 8, 4, 2
// and 1 lanes away.  All 64 lanes must be active.  The half and row swaps and the row
// rotations stay in the vector unit (after the step of distance 2 d every value repeats
// with period 2 d inside a row, so a rotation by d brings the partner's), where a shuffle
// through LDS takes two permutes and their latency per step.
__device__ __forceinline__ double wave_sum(double v)
{
    auto join = [](uint32_t lo, uint32_t hi) { return __hiloint2double((int)hi, (int)lo); };
    uint32_t lo = (uint32_t)__double2loint(v), hi = (uint32_t)__double2hiint(v);
    auto l = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
    auto h = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
    v = join(l[0], h[0]) + join(l[1], h[1]);
    lo = (uint32_t)__double2loint(v), hi = (uint32_t)__double2hiint(v);
    l = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
    h = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
    v = join(l[0], h[0]) + join(l[1], h[1]);
#define RD_ROT_ADD(D)                                                                               \
    v += join((uint32_t)__builtin_amdgcn_update_dpp(0, __double2loint(v), 0x120 + D, 0xf, 0xf, true), \
              (uint32_t)__builtin_amdgcn_update_dpp(0, __double2hiint(v), 0x120 + D, 0xf, 0xf, true))
    RD_ROT_ADD(8);
    RD_ROT_ADD(4);
    RD_ROT_ADD(2);
    RD_ROT_ADD(1);
#undef RD_ROT_ADD
    return v;
}
