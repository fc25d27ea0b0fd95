// Device code of the quantized paths: the table, loads, stores and scales
// that int8 and E4M3 plans share, and the int8 rule -- ES on symmetric int8
// codes with per-row binary32 scales, theta_j = s_r(j) q_j, q_j in
// [-127, 127].  The paper lists quantized ES as future work (Appendix A.2):
// noise must respect the quantization scale, updates must stay numerically
// stable, and perturbations must remain replayable from a seed.  Here a
// perturbation or update step d_j (in units of the row's quantum s) becomes
// the integer offset
//   k_j = floor(d_j + r_j 2^-16),   E[k_j] = d_j,
// with a 16-bit draw r_j, and q_j <- clamp(q_j + k_j, -127, 127).
//   * perturb / restore: d_j = sign sigma eps_j / s, eps_j the bf16 path's
//     noise (domain 0) under the member seed, and
//     k_j = floor(d_j + (2 r_j + 1) 2^-10) with r_j the top 9 bits of word
//     j & 3 of element j's own noise call (the uniform map reads only the low
//     23 bits, so these are free); restore subtracts the very same k_j, so it
//     is exact wherever the perturbation did not clamp.
//   * update: d_j = sum_d w_d eps_j(seed_d) / s and
//     k_j = floor(d_j + r_j 2^-16) with a 16-bit r_j from domain 1 under the
//     update's rounding seed: one Philox call at counter
//     (g lo, g hi, tensor_id, 1), g = j >> 3, serves elements 8g .. 8g+7;
//     element j takes word (j & 7) >> 1, low half for even j, high for odd.
// Elements whose scale is not a normal positive finite binary32 value are
// left unchanged.
//
// Layout: a lane owns 16 consecutive codes (one 16-byte access, four Philox
// blocks in lockstep); a tile is T lanes x U groups x 16 codes, taken in steps
// of 256 groups.  All passes are VALU-bound (16 normals per 16 bytes).  Of the
// int8 perturbation's 24.4 instructions per code 15.2 are the noise; the
// step's float work is done for the 16 codes in a simple phase and its
// conversions, saturating sums, clamps and packing in a heavy one (swap over
// the 0.5B-shaped set 563 us without the split, 524 with it).
#pragma once

#include <hip/hip_runtime.h>
#include <cstdint>

#include "es_noise.hpp"

namespace esq {

constexpr int kQGroup = 16;                     // one-byte codes per lane-group

// Quantized tensor table entry (a tensor, a contiguous shard of one or a
// strided block of one).  Tiles are numbered as in the bf16 path: full tiles
// (16-byte aligned base, in bounds) across all tensors, then tail tiles.
// Element j of the entry (its index in the entry's own storage) is element
//   n(j) = noise0 + j + (j / cols) * skip
// of its whole tensor: skip = 0 for a tensor or a contiguous shard; a block
// of rows of `cols` codes out of rows of cols + skip has skip > 0.  n(j)
// selects the noise, the rounding draws and the checksum term; j selects the
// code and its scale.  Every n(j) < 2^31 and numel < 2^31, so indices, and
// the end of the last tile, fit 32 bits.  n(0) and, for a block, cols and
// skip are multiples of 16, so a 16-code group of the entry is a 16-code
// group of the whole tensor.  The divisions j / row (scale index) and
// j / cols are mulhi(j, magic) >> shift, exact for every j < 2^31 (Granlund
// and Montgomery, 1994: magic = ceil(2^(31 + l) / d), l = ceil(log2 d),
// shift = l - 1).
struct DevQTensor {
    int8_t* data;
    const float* scales;
    uint32_t numel;
    uint32_t noise0;                            // whole-tensor index of element 0
    uint64_t first_full;
    uint64_t first_tail;
    uint32_t row;                               // codes per scale; 0: one scale
    uint32_t tensor_id;
    uint32_t magic;
    uint32_t shift;
    uint32_t first_step;                        // steps of the tails before this one's (a pass's
                                                //   workgroups over the tails, numbered in order)
    uint32_t skip;                              // 0, or whole-tensor codes between block rows
    uint32_t cmagic;                            // j / cols (read only when skip > 0)
    uint32_t cshift;
    uint32_t pad[2];
};
static_assert(sizeof(DevQTensor) == 80, "quantized tensor table entry layout");

struct QTileRef {
    int8_t* data;
    const float* scales;
    uint32_t numel;
    uint32_t noise0;
    uint32_t elem0;
    uint32_t row;
    uint32_t tensor_id;
    uint32_t magic;
    uint32_t shift;
    uint32_t skip;
    uint32_t cmagic;
    uint32_t cshift;
};

// n(e) of the entry above: the whole-tensor index of local element e.
__device__ __forceinline__ uint32_t qnoise_index(const QTileRef& r, uint32_t e) {
    uint32_t n = r.noise0 + e;
    if (r.skip != 0u) n += (__umulhi(e, r.cmagic) >> r.cshift) * r.skip;
    return n;
}

// The entry that owns global tile (or tail step) `tile`: the last one, of the n
// before the sentinel, whose first(i) is not beyond it (first() does not decrease, and
// first(0) = 0).  One load per 64-fold step: the lanes of a wave probe the
// range in parallel, so a workgroup that starts anywhere in the list finds its
// tensor in two round trips for up to 4096 tensors.  All lanes must be active.
template <class First>
__device__ __forceinline__ uint32_t find_tensor(uint64_t tile, uint32_t n, First first) {
    uint32_t lo = 0, span = n;                  // the owner is one of lo .. lo + span - 1
    while (span > 1u) {
        const uint32_t step = (span + 63u) / 64u;
        const uint32_t at = (threadIdx.x & 63u) * step;
        const bool below = at < span && first(lo + (at < span ? at : 0u)) <= tile;
        const uint32_t last = __popcll(__ballot(below)) - 1u;
        lo += last * step;
        span = min(step, span - last * step);
    }
    return lo;
}

__device__ __forceinline__ QTileRef qtile_ref(const DevQTensor& d, uint32_t elem0) {
    return QTileRef{d.data, d.scales, d.numel, d.noise0, elem0, d.row, d.tensor_id, d.magic,
                    d.shift, d.skip, d.cmagic, d.cshift};
}

// Full tile `tile` of the plan, and tail tile `tile`.
__device__ __forceinline__ QTileRef qlocate_full(const DevQTensor* __restrict__ tab, uint32_t n,
                                                 uint64_t tile, uint32_t tile_elems) {
    const uint32_t t = find_tensor(tile, n, [tab](uint32_t i) { return tab[i].first_full; });
    return qtile_ref(tab[t], static_cast<uint32_t>(tile - tab[t].first_full) * tile_elems);
}

__device__ __forceinline__ QTileRef qlocate_tail(const DevQTensor* __restrict__ tab, uint32_t n,
                                                 uint64_t tile, uint32_t tile_elems) {
    const uint32_t t = find_tensor(tile, n, [tab](uint32_t i) { return tab[i].first_tail; });
    const uint64_t n_full = tab[t + 1].first_full - tab[t].first_full;
    return qtile_ref(tab[t],
                     static_cast<uint32_t>(n_full + tile - tab[t].first_tail) * tile_elems);
}

// Tail step `step` of the plan, of part_codes codes: from its first code on.
__device__ __forceinline__ QTileRef qlocate_step(const DevQTensor* __restrict__ tab, uint32_t n,
                                                 uint32_t step, uint32_t tile_elems,
                                                 uint32_t part_codes) {
    const uint32_t t = find_tensor(step, n, [tab](uint32_t i) { return tab[i].first_step; });
    const uint32_t n_full = static_cast<uint32_t>(tab[t + 1].first_full - tab[t].first_full);
    return qtile_ref(tab[t], n_full * tile_elems + (step - tab[t].first_step) * part_codes);
}

typedef uint32_t q32x4_t __attribute__((ext_vector_type(4)));
#define ESQ_GLOBAL __attribute__((address_space(1)))

// 16 codes of one group in 4 words (byte i of word k is code 4k + i).  The
// checked path (tail tiles) takes the 16-byte access too for every group that
// lies wholly inside the tensor, at any byte alignment (global memory accesses
// need none on this part; the type says so to the compiler).
typedef uint32_t q32x4_any_t __attribute__((ext_vector_type(4), aligned(1)));

template <bool kFast>
__device__ __forceinline__ void qload(const int8_t* __restrict__ p, uint32_t e, uint32_t numel,
                                      uint32_t raw[4]) {
    if (kFast) {
        const q32x4_t v = __builtin_nontemporal_load((const ESQ_GLOBAL q32x4_t*)(p + e));
        raw[0] = v.x; raw[1] = v.y; raw[2] = v.z; raw[3] = v.w;
    } else if (e + 16 <= numel) {
        const q32x4_t v = __builtin_nontemporal_load((const ESQ_GLOBAL q32x4_any_t*)(p + e));
        raw[0] = v.x; raw[1] = v.y; raw[2] = v.z; raw[3] = v.w;
    } else {
        const ESQ_GLOBAL uint8_t* g = (const ESQ_GLOBAL uint8_t*)p;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            uint32_t w = 0;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const uint32_t j = e + 4 * k + i;
                if (j < numel) w |= uint32_t(g[j]) << (8 * i);
            }
            raw[k] = w;
        }
    }
}

template <bool kFast>
__device__ __forceinline__ void qstore(int8_t* __restrict__ p, uint32_t e, uint32_t numel,
                                       const uint32_t out[4]) {
    const q32x4_t v = {out[0], out[1], out[2], out[3]};
    if (kFast) {
        __builtin_nontemporal_store(v, (ESQ_GLOBAL q32x4_t*)(p + e));
    } else if (e + 16 <= numel) {
        __builtin_nontemporal_store(v, (ESQ_GLOBAL q32x4_any_t*)(p + e));
    } else {
        ESQ_GLOBAL uint8_t* g = (ESQ_GLOBAL uint8_t*)p;
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const uint32_t j = e + 4 * k + i;
                if (j < numel) g[j] = static_cast<uint8_t>(out[k] >> (8 * i));
            }
    }
}

// The scale of the 8 codes starting at element j (j is a multiple of 8 and the
// row length a multiple of 8, so the 8 codes share one scale); 0 beyond the
// last code.
__device__ __forceinline__ float load_scale(const QTileRef& r, uint32_t j) {
    if (j >= r.numel) return 0.0f;
    const ESQ_GLOBAL float* s = (const ESQ_GLOBAL float*)r.scales;
    return s[r.row == 0u ? 0u : __umulhi(j, r.magic) >> r.shift];
}

// The two scales of a 16-code group (codes 0-7 and 8-15); one lookup when the
// row length is a multiple of 16 (both halves in one row).
__device__ __forceinline__ void group_scales(const QTileRef& r, uint32_t e, float s[2]) {
    s[0] = load_scale(r, e);
    s[1] = (r.row & 15u) == 0u ? s[0] : load_scale(r, e + 8);
}

// The reciprocal of a scale, or 0 when it is not a normal positive finite
// value.  The hardware reciprocal (1 ulp) is well inside the offsets'
// tolerance.
__device__ __forceinline__ float inv_scale(float v) {
    const bool ok = v >= 0x1p-126f && v <= 0x1.fffffep127f;
    return ok ? __builtin_amdgcn_rcpf(v) : 0.0f;
}

// One noise stream of the 16 codes of a group whose first code has
// whole-tensor index n (a multiple of 16): the words of its four blocks, the
// radius factors and the trigonometric values (es_noise.hpp).
struct GroupNoise {
    es::Words w[4];
    float rad[8], c[8], sn[8];
};

__device__ __forceinline__ void group_noise(uint32_t n, uint32_t tensor_id, uint32_t k0,
                                            uint32_t k1, GroupNoise& g) {
    const uint32_t q0 = n >> 2;                 // multiple of 4: q0 + 3 does not carry
    const uint32_t q[4] = {q0, q0 + 1u, q0 + 2u, q0 + 3u};
    es::philox_quads<4>(q, 0u, tensor_id, k0, k1, g.w);
    es::box_muller_quads<4>(g.w, g.rad, g.c, g.sn);
}

// The low bytes of four 32-bit codes packed into one word (code i in byte
// i): two byte permutes and an OR.
__device__ __forceinline__ uint32_t pack_codes(int32_t c0, int32_t c1, int32_t c2, int32_t c3) {
    // v_perm_b32 numbers the second operand's bytes 0-3 and the first's 4-7;
    // selector byte 0x0c yields zero
    const uint32_t lo = __builtin_amdgcn_perm(uint32_t(c1), uint32_t(c0), 0x0c0c0400u);
    const uint32_t hi = __builtin_amdgcn_perm(uint32_t(c3), uint32_t(c2), 0x04000c0cu);
    return lo | hi;
}

// floor(x) as an integer in one instruction (the compiler emits a floor and
// a conversion), saturating at the ends of int32.
__device__ __forceinline__ int32_t floor_to_int(float x) {
    int32_t r;
    asm("v_cvt_flr_i32_f32 %0, %1" : "=v"(r) : "v"(x));
    return r;
}

// 1 + (2 r + 1) 2^-10 as a binary32 from the top 9 bits r of a noise word:
// ((w >> 9) & 0x007FC000) | 0x3F802000 with both constants in vector registers
// (SpareBits), one shift and one bitop3, which two waves can issue together.
struct SpareBits {
    uint32_t mask = 0x007FC000u, one_plus = 0x3F802000u;
    __device__ __forceinline__ SpareBits() {
        asm("" : "+v"(mask));
        asm("" : "+v"(one_plus));
    }
};
__device__ __forceinline__ float spare_one_plus(uint32_t w, const SpareBits& k) {
    return __uint_as_float(__builtin_amdgcn_bitop3_b32(w >> 9, k.mask, k.one_plus, 0xEA));
}

// Perturb / restore code: clamp(q +- floor(d + (2 r + 1) 2^-10), lo, 127)
// from v = d + f, f = 1 + (2 r + 1) 2^-10 (formed by the caller as one FMA;
// finite): the step is floor(v) - 1.  The conversion saturates at the ends of
// int32 and so does the sum, so a step far beyond what any code can absorb
// clamps to the right end without a bound on v first.  lo is -127; a caller
// whose scale is invalid passes d = 0 (so the step is 0) and lo = -128, which
// returns every code unchanged without a branch.
template <bool kNegate>
__device__ __forceinline__ int32_t qstep9(int32_t q, float v, int32_t lo) {
    const int32_t k = floor_to_int(v);
    int32_t x, r;
    if constexpr (kNegate) {
        asm("v_sub_i32 %0, %1, %2 clamp" : "=v"(x) : "v"(q + 1), "v"(k));
    } else {
        asm("v_add_i32 %0, %1, %2 clamp" : "=v"(x) : "v"(q - 1), "v"(k));
    }
    // min(max(x, lo), 127) in one v_med3_i32 (lo <= 127 always; the compiler
    // only forms the median for constant bounds)
    asm("v_med3_i32 %0, %1, %2, %3" : "=v"(r) : "v"(x), "v"(lo), "s"(127));
    return r;
}

// Update code: clamp(q + floor(d + r 2^-16), -127, 127).  d + r 2^-16 is one
// fused multiply-add (one rounding of the exact sum).  |d| is capped at 2^30
// quanta, far beyond what any code can absorb, so the integer arithmetic cannot
// overflow.
__device__ __forceinline__ int32_t qstep(int32_t q, float d, uint32_t draw16) {
    const float dc = __builtin_amdgcn_fmed3f(d, -0x1p30f, 0x1p30f);
    const float v = __builtin_fmaf(static_cast<float>(draw16), 0x1p-16f, dc);
    return min(max(q + floor_to_int(v), -127), 127);
}

}  // namespace esq
