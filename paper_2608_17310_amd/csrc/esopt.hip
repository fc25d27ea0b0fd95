// ES parameter path for MI355X (gfx950): perturb / restore / fused N-member
// update / reward z-score over a list of bf16 tensors, behind the C ABI of
// include/esopt.h.
//
// Method (arXiv 2608.17310): Section 3 (perturb theta + sigma eps_i, revert
// by subtraction, z-score rewards, theta += (alpha/G) sum zhat_i eps_i, noise
// regenerated from seeds), Section 3.1 (cosine sigma schedule), Appendix C.1
// (1/(G sigma) estimator), Appendix D.6 (order of apply / evaluate / revert /
// regenerate).
//
// Layout and launch shape:
//   * A plan cuts every tensor into tiles of T x U x 8 elements (T lanes per
//     workgroup, U 8-element groups per lane; by default 1024 x 8 x 8 =
//     65536 elements, 128 KB): full tiles on tile-sized boundaries of the
//     address space, then tail tiles (each tensor's head and remainder, or
//     every tile of an unaligned tensor), each described by a 32-byte
//     descriptor.  One launch covers the whole parameter list (several where it
//     would have 2^32 lanes), the full tiles and then the tails, reading a
//     workgroup's descriptor with scalar loads, so a tile's tensor, address and
//     noise identity are wave-uniform.
//   * Within a step of 256 x G groups, lane l of group slot g owns elements
//     e0 + 8 (256 g + l) .. +7: one 16-byte load and one 16-byte store, 64
//     lanes covering 1 KB contiguous per instruction.  Its two Philox calls
//     are the quads 2 n and 2 n + 1 of that group (tiles start at multiples
//     of 8 elements); no tile crosses a multiple of 2^34 elements, so the
//     counter's high word is uniform per tile.
//   * The passes run in 256-lane workgroups of one step each (StepShape): two
//     or four 8-element groups per lane, loaded in one burst and stored in
//     one, dispatched in the order of the plan's memory, the tail tiles' steps
//     (TailIndex) after the full tiles'.  Perturb is
//     HBM-bound: 0.5B-shaped set, perturb and restore, 678 -> 600 us (5.70 ->
//     6.44 TB/s), against one 1024-lane workgroup per CU that strode over the
//     tiles with its next tile's loads in flight.  The update is VALU-bound
//     (N noise streams per element): two groups per lane, so that four Philox
//     blocks run in lockstep (es_noise.hpp) and the waves of a SIMD (70 - 76
//     VGPRs: seven or six; 84 into masters: five) pair their issue.  4B-shaped
//     set, N = 32: 50.8 -> 43.0 ms.  Swap is the perturb kernel with two streams
//     and a bf16 rounding between them.
//   * The quantized path (int8 codes, es_quant.hpp; fp8 E4M3 codes,
//     es_fp8.hpp) has a tensor table, searched once per workgroup, and
//     256-lane workgroups of up to eight steps of one 16-code group per lane;
//     all its passes are VALU-bound.  0.5B-shaped set, int8 swap 602 -> 506
//     us; an eighth of it, fp8 update of 8 members 254 -> 196 us.
//   * Perturb/restore read and write each parameter once (4 bytes of HBM
//     traffic per parameter).  The update regenerates the noise of all
//     distinct member seeds for the same 8 elements in registers,
//     accumulates sum_d w_d eps_d in binary32, and then does the single
//     read-modify-write, so its HBM traffic does not depend on N.
//   * Tail tiles take a bounds-checked path with identical arithmetic:
//     16-byte accesses for whole groups (at any address), 2-byte accesses for
//     a partial one.
//   * Blocks of row-major tensors that are not one contiguous range (column
//     shards) are tiled by address like tensors; their tiles carry a row map
//     from the element's place in the block to its whole-tensor index, the
//     noise index, and run in a second launch of the same kernels
//     instantiated with it (kRows).
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstddef>
#include <cstring>
#include <atomic>
#include <mutex>
#include <new>
#include <string>
#include <type_traits>
#include <limits>
#include <unordered_map>
#include <vector>
#include <algorithm>

#include "../../include/esopt.h"
#include "es_fp8.hpp"
#include "es_noise.hpp"
#include "es_quant.hpp"

namespace {

constexpr int kAuxBlock = 256;              // lanes per workgroup of the small kernels
constexpr int kGroupElems = 8;              // bf16 per lane-group (one 16-byte access)
constexpr int kStepThreads = 256;           // lanes per workgroup of the step kernels
// Default tile shape of a plan, and the lanes per workgroup and workgroups per
// CU of the checksum kernels, which stride over whole tiles.
constexpr int kDefaultThreads = 1024;
constexpr int kDefaultGroups = 8;
constexpr int kDefaultUpdateWgPerCu = 8;
constexpr int kDefaultQGroups = 4;          // int8 tiles: 1024 x 4 x 16 codes (64 KB)
constexpr double kSqrt2Ln2Double = 1.1774100225154746910;   // sqrt(2 ln 2)

// Tile descriptor.  A plan lists its tiles in runs, indexed by tile number:
// full tiles first (kThreads * kU * 8 elements of one tensor, starting on a
// tile-sized boundary of the address space), then tail tiles (the part of a
// tensor before its first such boundary, the part after its last full tile,
// or every tile of a tensor whose base is not 16-byte aligned); the tiles of
// strided blocks (es_plan_create_blocks) follow in two more runs of the same
// kinds, each with a row map (DevRows), and are passed over in a second
// launch.  A workgroup reads a full tile's descriptor with a single scalar
// load and no search (searching a per-tensor table is a chain of dependent
// scalar loads), a tail tile's after one of its guide.
// Full tiles aligned to the address space, not to their tensor's base: with
// hundreds of tensors at unrelated offsets, tiles at mixed offsets streamed
// ~4 % slower.  32 bytes per 65 536-element tile.
struct TileDesc {
    uint16_t* data;                         // the tensor's base
    uint64_t elem0;                         // the tile's first element in its tensor
    uint32_t len;                           // its elements, at most a full tile's
    uint32_t tensor_id;
    uint32_t first, guide;                  // tail tiles: see TailIndex
};
static_assert(sizeof(TileDesc) == 32, "tile descriptor layout");

// A tile as the host lays it out.
struct DevTile {
    uint16_t* data;
    uint64_t elem0;
    uint64_t limit;                         // one past its last element
    uint32_t tensor_id;
    uint32_t aligned16;                     // the tensor's base is 16-byte aligned
};

// Row map of a tile of a strided block (es_block_t with rows > 1 and
// cols < row_len): the block is cut into pieces of whole rows, each tiled by
// address as a tensor of its own, so a tile's element index e is local to
// its piece (e < 2^31), and local element e is whole-tensor element
//   n0 + e + (e / cols) (row_len - cols),
// n0 being the piece's first whole-tensor index.  cols is a multiple of 8, so
// a group of 8 never spans two rows and its elements keep consecutive
// indices (one quad pair).  The row division is a multiply-high and a shift
// and skip = row_len - cols is below 2^32, so the map costs one 32 x 32-bit
// multiply-add and a 64-bit add per group.  As with contiguous tiles, no tile
// spans a multiple of 2^34 whole-tensor elements (the host splits it there),
// so the counter's high word `hi` is the tile's, wave-uniform.  One entry per
// tile, beside its descriptor.
struct DevRows {
    uint64_t n0;
    uint32_t skip;                          // row_len - cols
    uint32_t magic, shift;                  // e / cols = mulhi(e, magic) >> shift
    uint32_t hi;                            // whole-tensor index >> 34, the same for the tile
    uint32_t pad[2];
};
static_assert(sizeof(DevRows) == 32, "row map layout");

// Whole-tensor index of local element e (< 2^31) under a row map; the host
// tests call this same function.
__host__ __device__ __forceinline__ uint64_t rows_index(uint64_t n0, uint32_t skip, uint32_t magic,
                                                        uint32_t shift, uint64_t e) {
    const uint32_t el = static_cast<uint32_t>(e);
    const uint32_t row = static_cast<uint32_t>((uint64_t(el) * magic) >> 32) >> shift;
    return n0 + (uint64_t(row) * skip + el);
}

struct MemberIn {                           // one population member, CSR order
    uint32_t reward_index;
    int32_t sign;
};
struct DistinctIn {                         // one distinct seed and its members
    uint32_t k0, k1;
    uint32_t first;
    uint32_t count;
};
struct Member {                             // merged weight of one distinct seed
    uint32_t k0, k1;
    float w_k;                              // weight times sqrt(2 ln 2)
    uint32_t pad;
};
struct UpdateHeader {
    uint32_t n_distinct;
    uint32_t n_live;                        // distinct seeds with w != 0
    int32_t status;                         // 1: non-finite reward, update skipped
    uint32_t pad;
};

// Plan scratch layout (bytes).
constexpr size_t kOffMembersIn = 0;
constexpr size_t kOffDistinctIn = kOffMembersIn + sizeof(MemberIn) * ES_MAX_MEMBERS;
constexpr size_t kOffMembers = kOffDistinctIn + sizeof(DistinctIn) * ES_MAX_MEMBERS;
constexpr size_t kOffHeader = kOffMembers + sizeof(Member) * ES_MAX_MEMBERS;
constexpr size_t kScratchBytes = kOffHeader + 256;

constexpr int kStageWords = 256;            // 1 KB of kernel arguments per launch
constexpr uint64_t kMaxLayoutTiles = uint64_t(1) << 22;   // es_tile_layout's bound
struct StageChunk {
    uint32_t words[kStageWords];
};

thread_local std::string g_last_error;

int fail(int code, const std::string& msg) {
    g_last_error = msg;
    return code;
}

int hip_fail(hipError_t e, const std::string& what) {
    return fail(ES_ERR_HIP, what + ": " + hipGetErrorString(e));
}

// A failure of call `name`: the message is formatted only here, so a call
// that succeeds builds no strings (no host allocation on its way).
int fail_in(int code, const char* name, const char* msg) {
    return fail(code, std::string(name) + ": " + msg);
}

// ------------------------------------------------------------------------
// Device code
// ------------------------------------------------------------------------

typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
// Tile descriptors and tensor tables hold generic pointers; every parameter
// lives in global memory, and saying so lets the compiler use global_load /
// global_store (vector-memory counters only) instead of flat accesses.
#define ES_GLOBAL __attribute__((address_space(1)))

// Load the 8 bf16 of one group (packed in 4 words): one 16-byte load
// (nontemporal: the parameters are streamed once per pass).  The
// checked path (tail tiles) takes it for every group that lies wholly below
// the bound `limit`, and 2-byte loads below the bound for a partial group.  A
// tensor whose base is only 2-byte aligned takes the same 16-byte accesses at
// its own addresses (global memory accesses need no alignment on this part;
// the type says so to the compiler): a wave then touches nine 128-byte lines
// for its eight.
typedef uint32_t u32x4_any_t __attribute__((ext_vector_type(4), aligned(2)));

template <bool kFast>
__device__ __forceinline__ void load_group(const uint16_t* __restrict__ p, uint64_t e,
                                           uint64_t limit, uint32_t raw[4]) {
    if (kFast) {
        const ES_GLOBAL u32x4_t* a = (const ES_GLOBAL u32x4_t*)(p + e);
        const u32x4_t v = __builtin_nontemporal_load(a);
        raw[0] = v.x; raw[1] = v.y; raw[2] = v.z; raw[3] = v.w;
    } else if (e + 8 <= limit) {
        const ES_GLOBAL u32x4_any_t* a = (const ES_GLOBAL u32x4_any_t*)(p + e);
        const u32x4_t v = __builtin_nontemporal_load(a);
        raw[0] = v.x; raw[1] = v.y; raw[2] = v.z; raw[3] = v.w;
    } else {
        const ES_GLOBAL uint16_t* g = (const ES_GLOBAL uint16_t*)p;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const uint32_t lo = (e + 2 * k < limit) ? g[e + 2 * k] : 0u;
            const uint32_t hi = (e + 2 * k + 1 < limit) ? g[e + 2 * k + 1] : 0u;
            raw[k] = lo | (hi << 16);
        }
    }
}

template <bool kFast>
__device__ __forceinline__ void store_group(uint16_t* __restrict__ p, uint64_t e, uint64_t limit,
                                            const uint32_t out[4]) {
    const u32x4_t v = {out[0], out[1], out[2], out[3]};
    if (kFast) {
        ES_GLOBAL u32x4_t* a = (ES_GLOBAL u32x4_t*)(p + e);
        __builtin_nontemporal_store(v, a);
    } else if (e + 8 <= limit) {
        ES_GLOBAL u32x4_any_t* a = (ES_GLOBAL u32x4_any_t*)(p + e);
        __builtin_nontemporal_store(v, a);
    } else {
        ES_GLOBAL uint16_t* g = (ES_GLOBAL uint16_t*)p;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (e + 2 * k < limit) g[e + 2 * k] = static_cast<uint16_t>(out[k] & 0xFFFFu);
            if (e + 2 * k + 1 < limit) g[e + 2 * k + 1] = static_cast<uint16_t>(out[k] >> 16);
        }
    }
}

// The binary32 master copies of a group's 8 elements (es_plan_set_master):
// element e's master sits at mb + 4 e, mb being the tile's master base.  A
// tensor's masters are 16-byte aligned and its groups start at multiples of 8
// elements of it, so a whole group takes two 16-byte accesses whatever the
// bf16 base; element-wise accesses below the bound otherwise.
typedef float f32x4_t __attribute__((ext_vector_type(4)));

__device__ __forceinline__ void load_master(uintptr_t mb, uint64_t e, uint64_t limit, float m[8]) {
    if (e + 8 <= limit) {
        const ES_GLOBAL f32x4_t* a = (const ES_GLOBAL f32x4_t*)(mb + 4 * e);
        const f32x4_t v0 = __builtin_nontemporal_load(a), v1 = __builtin_nontemporal_load(a + 1);
        m[0] = v0.x; m[1] = v0.y; m[2] = v0.z; m[3] = v0.w;
        m[4] = v1.x; m[5] = v1.y; m[6] = v1.z; m[7] = v1.w;
    } else {
        const ES_GLOBAL float* g = (const ES_GLOBAL float*)mb;
#pragma unroll
        for (int k = 0; k < 8; ++k) m[k] = (e + k < limit) ? g[e + k] : 0.0f;
    }
}

__device__ __forceinline__ void store_master(uintptr_t mb, uint64_t e, uint64_t limit,
                                             const float m[8]) {
    if (e + 8 <= limit) {
        ES_GLOBAL f32x4_t* a = (ES_GLOBAL f32x4_t*)(mb + 4 * e);
        const f32x4_t v0 = {m[0], m[1], m[2], m[3]};
        const f32x4_t v1 = {m[4], m[5], m[6], m[7]};
        __builtin_nontemporal_store(v0, a);
        __builtin_nontemporal_store(v1, a + 1);
    } else {
        ES_GLOBAL float* g = (ES_GLOBAL float*)mb;
#pragma unroll
        for (int k = 0; k < 8; ++k)
            if (e + k < limit) g[e + k] = m[k];
    }
}

// Noise streams applied by one perturb-style pass.  kM = 1: one stream,
// theta <- RNE(theta + c_0 eps_0) (perturb / restore).  kM = 2: two streams
// applied in turn with a bf16 rounding in between,
// theta <- RNE(RNE(theta + c_0 eps_0) + c_1 eps_1), which is es_restore of
// one member followed by es_perturb of the next, bit for bit, in one pass
// (swap).  kM = 3: the same with both streams on one key (an antithetic
// partner), whose noise is generated once.  coef_k = c sqrt(2 ln 2).
struct Streams {
    uint32_t k0[2], k1[2];
    float coef_k[2];
};

// x[8 g + k] += scale * eps of two groups from their four blocks' radius
// factors and trigonometric values (pair p feeds elements 2 p and 2 p + 1);
// scale_k = scale * sqrt(2 ln 2).
__device__ __forceinline__ void pair_axpy(const float rad[8], const float c[8], const float sn[8],
                                          float scale_k, float x[16]) {
#pragma unroll
    for (int p = 0; p < 8; ++p) {
        const float t = scale_k * rad[p];
        x[2 * p] = __builtin_fmaf(t, c[p], x[2 * p]);
        x[2 * p + 1] = __builtin_fmaf(t, sn[p], x[2 * p + 1]);
    }
}

// The quads of two groups whose first elements have whole-tensor indices n[g]
// (multiples of 8, so a group's second quad does not carry).
__device__ __forceinline__ void pair_quads(const uint64_t n[2], uint32_t q[4]) {
#pragma unroll
    for (int g = 0; g < 2; ++g) {
        q[2 * g] = static_cast<uint32_t>(n[g] >> 2);
        q[2 * g + 1] = q[2 * g] + 1u;
    }
}

__device__ __forceinline__ void unpack_pair(const uint32_t raw[2][4], float x[16]) {
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        x[2 * k] = es::bf16_lo(raw[k / 4][k % 4]);
        x[2 * k + 1] = es::bf16_hi(raw[k / 4][k % 4]);
    }
}
__device__ __forceinline__ void pack_pair(const float x[16], uint32_t raw[2][4]) {
#pragma unroll
    for (int k = 0; k < 8; ++k) raw[k / 4][k % 4] = es::pack_bf16x2(x[2 * k], x[2 * k + 1]);
}

// Apply the streams to two 8-element groups in registers (raw, in place):
// each stream adds one FMA per element to the binary32 value, rounded to bf16
// after each stream.  Four Philox blocks in lockstep (es_noise.hpp).
template <int kM>
__device__ __forceinline__ void perturb_pair(uint32_t raw[2][4], const uint64_t n[2],
                                             uint32_t q_hi, uint32_t tensor_id,
                                             const Streams& st) {
    uint32_t q[4];
    pair_quads(n, q);
    es::Words w[4];
    float rad[8], c[8], sn[8], x[16];
#pragma unroll
    for (int m = 0; m < (kM == 2 ? 2 : 1); ++m) {
        es::philox_quads<4>(q, q_hi, tensor_id, st.k0[m], st.k1[m], w);
        es::box_muller_quads<4>(w, rad, c, sn);
        unpack_pair(raw, x);
        pair_axpy(rad, c, sn, st.coef_k[m], x);
        pack_pair(x, raw);
    }
    if constexpr (kM == 3) {
        unpack_pair(raw, x);
        pair_axpy(rad, c, sn, st.coef_k[1], x);
        pack_pair(x, raw);
    }
}

// A tile: up to kThreads * kU * 8 consecutive elements of one tensor, from
// element elem0 on; accesses of a tail tile stay below `limit`.  A tile of a
// strided block also carries its piece's row map (DevRows): its elements are
// then addressed by elem0 + ... and draw the noise of their whole-tensor
// index.  Every field is wave-uniform (scalar registers).
struct TileRef {
    uint16_t* data;
    uint64_t limit;
    uint64_t elem0;
    uint32_t tensor_id;
    uint64_t n0 = 0;                        // row map (strided blocks only)
    uint32_t skip = 0, magic = 0, shift = 0, hi = 0;
};

__device__ __forceinline__ TileRef tile_ref(const TileDesc& d) {
    return TileRef{d.data, d.elem0 + d.len, d.elem0, d.tensor_id};
}

__device__ __forceinline__ TileRef tile_ref(const TileDesc& d, const DevRows& m) {
    return TileRef{d.data, d.elem0 + d.len, d.elem0, d.tensor_id, m.n0, m.skip, m.magic, m.shift,
                   m.hi};
}

// Tile i of a launch: its descriptor, and with kRows its row map.
template <bool kRows>
__device__ __forceinline__ TileRef load_ref(const TileDesc* __restrict__ tiles,
                                            const DevRows* __restrict__ rows, uint64_t i) {
    if constexpr (kRows) return tile_ref(tiles[i], rows[i]);
    else return tile_ref(tiles[i]);
}

// Noise index of the group starting at element e of a tile: e itself, or
// the whole-tensor index through the tile's row map.
template <bool kRows>
__device__ __forceinline__ uint64_t noise_index(const TileRef& r, uint64_t e) {
    if constexpr (kRows) return rows_index(r.n0, r.skip, r.magic, r.shift, e);
    else return e;
}

// The counter's high word (whole-tensor index >> 34), uniform over a tile.
template <bool kRows>
__device__ __forceinline__ uint32_t tile_high_word(const TileRef& r) {
    if constexpr (kRows) return r.hi;
    else return static_cast<uint32_t>(r.elem0 >> 34);
}

// How a launch of kStepThreads-lane workgroups covers a plan's tiles, one step
// per workgroup: a full tile is 2^full_shift steps of kG 8-element groups per
// lane (256 x 8 kG elements), and a tail tile as many steps of two groups as it
// needs (TailIndex).  Workgroups are dispatched in order, so those in flight work
// on one contiguous stretch of the plan's memory, and a step's loads leave in one
// burst and its stores in another.  In place over the 0.5B-shaped set (perturb
// and restore, kG = 4): 6.41 TB/s with one step per workgroup, 6.22 with two,
// 5.66 with four; 5.67 with two steps over a grid that strides (the order is
// lost), 5.70 with one 1024-lane workgroup per CU striding over 128 KB tiles
// with its next tile's loads in flight.
constexpr uint32_t kTailStep = kStepThreads * 2 * kGroupElems;   // elements of a tail's step

// The steps of a run of tail tiles, numbered tile by tile: tail t's are first(t)
// .. first(t + 1) - 1.  The tail of step j is found from guide(k), k = j n_tail /
// n_steps, which is the tail of the first step with that k (a guide table: a k
// stands for n_steps / n_tail steps, so the search goes on over the few tails
// that these lie in).  So every workgroup has a step, whatever the tails'
// lengths, and none has two: with every tail cut for the longest, a plan of
// many short tensors and a longer one launched mostly empty workgroups, which
// cost 0.7 (perturb) to 2 ns each (update of 4), and with several steps per
// workgroup where the tails are many, those of an unaligned plan, whose every
// tile is a tail, lost their order.  10 000 tensors of 64 elements and one of
// 60 000, perturb 53 -> 8 us and update of 4 members 163 -> 29; 6 G unaligned
// elements, perturb 5.35 -> 4.29 ms.  Two groups per lane in every pass: 200 M
// unaligned elements, perturb 138 us with two and 144 with four, swap 200 with
// either.
struct TailIndex {
    uint32_t n_tail;
    uint32_t n_steps;
    uint64_t ratio;                         // n_tail / n_steps in units of 2^-32
};
struct StepShape {
    uint32_t full_shift;
    uint32_t step0;                         // the launch's first tail step
    uint64_t tail0;                         // the first tail tile, from the launch's first tile
    TailIndex tails;
};

// Workgroups go to the 8 XCDs in turn.  Within each 512 of them, item
// xcd_run_item(i) of workgroup i gives every XCD a run of 64 consecutive steps
// (1 MB with kG = 4), so that its L2 and address translation see a contiguous
// stretch and the chip as a whole still 8 MB in order.  Perturb, mean of a
// perturb and its restore: 4B-shaped set 2.745 -> 2.647 ms, 27B 15.58 -> 15.16;
// runs of 8: 2.701 and 15.67, of 512: 2.731 and 15.18.
constexpr uint32_t kXcds = 8, kXcdRun = 64;
__host__ __device__ __forceinline__ uint64_t xcd_run_item(uint64_t i) {
    const uint64_t j = i / kXcds;
    return (j / kXcdRun) * (kXcds * kXcdRun) + (i % kXcds) * kXcdRun + j % kXcdRun;
}

// What workgroup i of a step launch takes, first the n_full full tiles' steps
// and then tail steps: part `part` of tile `tile`.  The host tests call this
// same function.
struct StepItem {
    bool full;
    uint32_t part;
    uint64_t tile;
    TileDesc desc;                          // the tile's
};
__host__ __device__ __forceinline__ StepItem step_item(uint64_t i, uint64_t n_full,
                                                       const StepShape& sh,
                                                       const TileDesc* __restrict__ tiles) {
    const uint64_t full_items = n_full << sh.full_shift;
    if (i < (full_items & ~uint64_t(kXcds * kXcdRun - 1))) i = xcd_run_item(i);
    if (i < full_items) {
        const uint64_t tile = i >> sh.full_shift;
        return StepItem{true, static_cast<uint32_t>(i) & ((1u << sh.full_shift) - 1u), tile,
                        tiles[tile]};
    }
    const uint32_t j = static_cast<uint32_t>(i - full_items) + sh.step0;
    const TileDesc* const tails = tiles + sh.tail0;
    if (sh.tails.n_steps == sh.tails.n_tail)               // a step per tail
        return StepItem{false, 0u, sh.tail0 + j, tails[j]};
    const uint32_t last = sh.tails.n_tail - 1u;
    uint32_t t = tails[(j * sh.tails.ratio) >> 32].guide;
    TileDesc d = tails[t];
    uint32_t end = tails[min(t + 1u, last)].first;         // of t's steps (not the last tail's)
    while (t < last && end <= j) {
        ++t;
        d = tails[t];
        end = tails[min(t + 1u, last)].first;
    }
    return StepItem{false, j - d.first, sh.tail0 + t, d};
}

// The step of this workgroup: step(full, tile reference, tile number, the
// lane's first element); its group g starts 8 kStepThreads g elements on.  For a
// tail tile the first group starts below the bound (lanes beyond it are left
// out) and the second may not.
template <bool kRows, int kG, class Step>
__device__ __forceinline__ void for_steps(const TileDesc* __restrict__ tiles, uint64_t n_full,
                                          const DevRows* __restrict__ rows, const StepShape& sh,
                                          Step step) {
    constexpr uint32_t kElems = kStepThreads * kG * kGroupElems;
    const StepItem it = step_item(blockIdx.x, n_full, sh, tiles);
    TileRef r;
    if constexpr (kRows) r = tile_ref(it.desc, rows[it.tile]);
    else r = tile_ref(it.desc);
    const uint64_t e = r.elem0 + it.part * (it.full ? kElems : kTailStep) +
                       threadIdx.x * uint32_t(kGroupElems);
    if (it.full) step(std::true_type{}, r, it.tile, e);
    else if (e < r.limit) step(std::false_type{}, r, it.tile, e);
}

// One pass over the whole parameter list applying kM noise streams: each lane
// loads its kG groups, generates their noise (two groups at a time, which the
// loads' latency lies under), and stores them in one burst.  HBM-bound with
// one stream, VALU-bound with two.  kRows: the launch over the tiles of strided
// blocks, each with its row map in `rows` (same index as its descriptor);
// otherwise `rows` is unused.
template <int kM, bool kRows, int kG>
__global__ __launch_bounds__(kStepThreads) void es_perturb_kernel(const TileDesc* __restrict__ tiles,
                                                                  uint64_t n_full,
                                                                  const DevRows* __restrict__ rows,
                                                                  Streams st, StepShape sh) {
    constexpr uint64_t kSlab = uint64_t(kStepThreads) * kGroupElems;
    for_steps<kRows, kG>(tiles, n_full, rows, sh,
                         [&](auto full, const TileRef& r, uint64_t, uint64_t e) {
        constexpr bool kFast = decltype(full)::value;
        constexpr int kN = kFast ? kG : 2;
        uint32_t raw[kN][4];
#pragma unroll
        for (int g = 0; g < kN; ++g) {
            if (kFast || e + g * kSlab < r.limit)
                load_group<kFast>(r.data, e + g * kSlab, r.limit, raw[g]);
            else
                raw[g][0] = raw[g][1] = raw[g][2] = raw[g][3] = 0u;
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int g = 0; g < kN; g += 2) {
            const uint64_t n[2] = {noise_index<kRows>(r, e + g * kSlab),
                                   noise_index<kRows>(r, e + (g + 1) * kSlab)};
            perturb_pair<kM>(raw + g, n, tile_high_word<kRows>(r), r.tensor_id, st);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int g = 0; g < kN; ++g)
            if (kFast || e + g * kSlab < r.limit)
                store_group<kFast>(r.data, e + g * kSlab, r.limit, raw[g]);
    });
}

// A tile's master base: its bf16 base times two plus the tensor's delta.
__device__ __forceinline__ uintptr_t master_base(const uint64_t* __restrict__ mdelta,
                                                 const TileRef& r, uint64_t i) {
    return mdelta[i] + 2 * reinterpret_cast<uintptr_t>(r.data);
}

// A member applied from binary32 masters (es_perturb_master) with sigma > 0:
// bf16 values RNE(m + c eps) from the masters at mb + 4 e, the masters only
// read -- the arithmetic of es_perturb on the masters' values.  HBM-bound, 6
// bytes per parameter.  In a full tile a lane takes the quads at elements 4 t
// and 4 (256 + t) of each slab of 2048: a 16-byte master load then covers 1 KB
// of consecutive masters per wave (one lane's 8 consecutive masters would take
// two loads of 16 bytes at a 32-byte stride, and streamed lines were fetched
// twice), and an 8-byte bf16 store 512 consecutive bytes.  A quad is one Philox
// block: its two Box-Muller pairs are its elements.  Tail tiles take the groups
// of the other passes with bounds-checked accesses.  Two groups per lane (57
// VGPRs, eight waves per SIMD) and four (88, five): 0.5B-shaped set 465 and 477
// us, 4B 3875 and 3961, 503 M in column blocks 498 and 507.
template <bool kRows>
__global__ __launch_bounds__(kStepThreads) void es_apply_master_kernel(
    const TileDesc* __restrict__ tiles, uint64_t n_full, const DevRows* __restrict__ rows,
    Streams st, const uint64_t* __restrict__ mdelta, StepShape sh) {
    typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
    constexpr uint64_t kSlab = uint64_t(kStepThreads) * kGroupElems;
    for_steps<kRows, 2>(tiles, n_full, rows, sh,
                         [&](auto full, const TileRef& r, uint64_t tile, uint64_t e) {
        constexpr bool kFast = decltype(full)::value;
        const uintptr_t mb = master_base(mdelta, r, tile);
        const uint32_t q_hi = tile_high_word<kRows>(r);
        float m[2][8];
        if constexpr (kFast) {
            const uint64_t e4 = e - threadIdx.x * 4u;        // the lane's first quad
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const f32x4_t v = __builtin_nontemporal_load(
                    (const ES_GLOBAL f32x4_t*)(mb + 4 * (e4 + i * (kSlab / 2))));
                float* x = m[i / 2] + 4 * (i % 2);
                x[0] = v.x; x[1] = v.y; x[2] = v.z; x[3] = v.w;
            }
        } else {
#pragma unroll
            for (int g = 0; g < 2; ++g) {
                if (e + g * kSlab < r.limit)
                    load_master(mb, e + g * kSlab, r.limit, m[g]);
                else
                    for (int k = 0; k < 8; ++k) m[g][k] = 0.0f;
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        uint32_t out[2][4];
        uint32_t q[4];
        if constexpr (kFast) {
#pragma unroll
            for (int i = 0; i < 4; ++i)
                q[i] = static_cast<uint32_t>(
                    noise_index<kRows>(r, e - threadIdx.x * 4u + i * (kSlab / 2)) >> 2);
        } else {
            const uint64_t n[2] = {noise_index<kRows>(r, e), noise_index<kRows>(r, e + kSlab)};
            pair_quads(n, q);
        }
        es::Words w[4];
        float rad[8], c[8], sn[8];
        es::philox_quads<4>(q, q_hi, r.tensor_id, st.k0[0], st.k1[0], w);
        es::box_muller_quads<4>(w, rad, c, sn);
        pair_axpy(rad, c, sn, st.coef_k[0], &m[0][0]);
        pack_pair(&m[0][0], out);
        if constexpr (kFast) {
            const uint64_t e4 = e - threadIdx.x * 4u;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const u32x2_t v = {out[i / 2][2 * (i % 2)], out[i / 2][2 * (i % 2) + 1]};
                __builtin_nontemporal_store(v,
                                            (ES_GLOBAL u32x2_t*)(r.data + e4 + i * (kSlab / 2)));
            }
        } else {
#pragma unroll
            for (int g = 0; g < 2; ++g)
                if (e + g * kSlab < r.limit)
                    store_group<false>(r.data, e + g * kSlab, r.limit, out[g]);
        }
    });
}

// The in-place streaming ceiling of a plan (es_stream_pass): every element
// is read and written back as itself (XOR with `flip`, which the host passes
// as 0, so the compiler keeps the stores), over the same steps and 16-byte
// nontemporal accesses as the passes above but without arithmetic, so it
// bounds what any pass over the plan can reach.
template <int kG>
__global__ __launch_bounds__(kStepThreads) void es_stream_kernel(const TileDesc* __restrict__ tiles,
                                                                 uint64_t n_full, uint32_t flip,
                                                                 StepShape sh) {
    constexpr uint64_t kSlab = uint64_t(kStepThreads) * kGroupElems;
    for_steps<false, kG>(tiles, n_full, nullptr, sh,
                         [&](auto full, const TileRef& r, uint64_t, uint64_t e) {
        constexpr bool kFast = decltype(full)::value;
        constexpr int kN = kFast ? kG : 2;
        uint32_t raw[kN][4];
#pragma unroll
        for (int g = 0; g < kN; ++g)
            if (kFast || e + g * kSlab < r.limit)
                load_group<kFast>(r.data, e + g * kSlab, r.limit, raw[g]);
        __builtin_amdgcn_sched_barrier(0);      // all loads issued before the first wait
#pragma unroll
        for (int g = 0; g < kN; ++g)
            if (kFast || e + g * kSlab < r.limit) {
#pragma unroll
                for (int k = 0; k < 4; ++k) raw[g][k] ^= flip;
                store_group<kFast>(r.data, e + g * kSlab, r.limit, raw[g]);
            }
    });
}

// Parameter checksum (es_plan_checksum):
//   H = sum over every element of mix64(j K_J + tensor_id K_T + b K_B)  mod 2^64
// with j the element's index in its whole tensor, b its 16 bits and mix64
// the 64-bit finalizer of SplitMix64 (Steele, Lea and Flood, OOPSLA 2014).
// Addition mod 2^64 does not depend on the order of its terms, so H does not
// depend on the launch shape, and the checksums of disjoint shards of a tensor
// add up to the whole tensor's.  Read-only and VALU-bound (about 24
// instructions per element: 64-bit products and shifts on 32-bit lanes).
constexpr uint64_t kSumJ = 0x9E3779B97F4A7C15ull;
constexpr uint64_t kSumT = 0xC2B2AE3D27D4EB4Full;
constexpr uint64_t kSumB = 0x165667B19E3779F9ull;

__device__ __forceinline__ uint64_t mix64(uint64_t z) {
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

__device__ __forceinline__ uint64_t wave_sum_u64(uint64_t x) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off, 64);
    return x;
}

// The checksum terms of kN consecutive elements from whole-tensor index e,
// their values taken kBits at a time from `raw` (element k in bits
// kBits*k.. of the word array); with kChecked only elements below `limit`
// count.
template <int kN, int kBits, bool kChecked>
__device__ __forceinline__ uint64_t checksum_terms(const uint32_t* raw, uint64_t e,
                                                   uint64_t limit, uint64_t salt) {
    constexpr int kPerWord = 32 / kBits;
    constexpr uint32_t kMask = (1u << kBits) - 1u;
    uint64_t x = e * kSumJ + salt, acc = 0;
#pragma unroll
    for (int k = 0; k < kN; ++k) {
        const uint64_t b = (raw[k / kPerWord] >> (kBits * (k % kPerWord))) & kMask;
        const uint64_t f = mix64(x + b * kSumB);
        acc += (!kChecked || e + k < limit) ? f : 0ull;
        x += kSumJ;
    }
    return acc;
}

// Adds the workgroup's lane sums to *out: a lane-shuffle sum per wave, then
// one 64-bit atomic per workgroup.
template <int kThreads>
__device__ __forceinline__ void add_workgroup_sum(uint64_t acc, unsigned long long* out) {
    __shared__ uint64_t part[kThreads / 64];
    acc = wave_sum_u64(acc);
    if ((threadIdx.x & 63u) == 0u) part[threadIdx.x / 64] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint64_t s = 0;
#pragma unroll
        for (int w = 0; w < kThreads / 64; ++w) s += part[w];
        atomicAdd(out, static_cast<unsigned long long>(s));
    }
}

// bf16 plan: full tiles with 16-byte loads and no per-element bound, then
// tail tiles bounds-checked.  With kRows (tiles of strided blocks) each
// term takes the element's whole-tensor index from the tile's row map.
// kCut: a small plan's tiles are cut into 2^shift items each, since its few
// tiles would keep as few CUs at eight group slots in a row (with the slots of
// an item known to the compiler otherwise: 1 % on large plans).
template <int kThreads, int kU, bool kRows, bool kCut>
__global__ __launch_bounds__(kThreads) void es_checksum_kernel(const TileDesc* __restrict__ tiles,
                                                               uint64_t n_full, uint64_t n_tail,
                                                               const DevRows* __restrict__ rows,
                                                               uint32_t shift,
                                                               unsigned long long* __restrict__ out) {
    uint64_t acc = 0;
    const uint32_t cut = kCut ? shift : 0u, slots = kU >> cut, parts = (1u << cut) - 1u;
    for (uint64_t i = blockIdx.x; i < n_full << cut; i += gridDim.x) {
        const TileRef r = load_ref<kRows>(tiles, rows, i >> cut);
        const uint32_t u0 = (static_cast<uint32_t>(i) & parts) * slots;
        const uint64_t salt = uint64_t(r.tensor_id) * kSumT;
#pragma unroll 1
        for (uint32_t u = u0; u < u0 + slots; ++u) {
            const uint64_t e = r.elem0 + uint64_t(u * kThreads + threadIdx.x) * kGroupElems;
            uint32_t raw[4];
            load_group<true>(r.data, e, r.limit, raw);
            acc += checksum_terms<kGroupElems, 16, false>(raw, noise_index<kRows>(r, e), r.limit,
                                                          salt);
        }
    }
    for (uint64_t i = blockIdx.x; i < n_tail << cut; i += gridDim.x) {
        const TileRef r = load_ref<kRows>(tiles, rows, n_full + (i >> cut));
        const uint32_t u0 = (static_cast<uint32_t>(i) & parts) * slots;
        const uint64_t salt = uint64_t(r.tensor_id) * kSumT;
#pragma unroll 1
        for (uint32_t u = u0; u < u0 + slots; ++u) {
            const uint64_t e = r.elem0 + uint64_t(u * kThreads + threadIdx.x) * kGroupElems;
            if (e >= r.limit) break;
            uint32_t raw[4];
            load_group<false>(r.data, e, r.limit, raw);
            const uint64_t n = noise_index<kRows>(r, e);
            // the bound moves with the index: n + (limit - e) for a row map
            acc += checksum_terms<kGroupElems, 16, true>(raw, n, kRows ? n + (r.limit - e) : r.limit,
                                                         salt);
        }
    }
    add_workgroup_sum<kThreads>(acc, out);
}

// *p = 0 before a checksum's atomics (a kernel, not a memset, so the call
// stays capturable into a HIP graph).
__global__ __launch_bounds__(64) void es_zero_u64_kernel(unsigned long long* __restrict__ p) {
    if (threadIdx.x == 0) *p = 0ull;
}

// HBM calibration over a caller's flat buffer (es_hbm_calibrate): tiles of
// kThreads lanes x kU 16-byte words, each loaded whole and then stored, with nontemporal accesses
// (kNT, the passes' policy) or ordinary ones.  kMode 0 reads every word
// (their XOR leaves in one atomic per wave, so the loads are live), 1 writes
// every word (the pattern tile, u, lane, 0), 2 reads every word and writes it
// back (XOR with `flip`, which the host passes as 0, so the stores are kept).
template <bool kNT>
__device__ __forceinline__ u32x4_t cal_load(const ES_GLOBAL u32x4_t* a) {
    if constexpr (kNT) return __builtin_nontemporal_load(a);
    else return *a;
}
template <bool kNT>
__device__ __forceinline__ void cal_store(u32x4_t v, ES_GLOBAL u32x4_t* a) {
    if constexpr (kNT) __builtin_nontemporal_store(v, a);
    else *a = v;
}

template <int kThreads, int kU, int kMode, bool kNT>
__global__ __launch_bounds__(kThreads) void es_calibrate_kernel(u32x4_t* __restrict__ buf,
                                                                uint64_t n_tiles,
                                                                uint32_t* __restrict__ sink,
                                                                uint32_t flip) {
    uint32_t acc = 0;
    for (uint64_t tile = blockIdx.x; tile < n_tiles; tile += gridDim.x) {
        ES_GLOBAL u32x4_t* base =
            (ES_GLOBAL u32x4_t*)buf + tile * (uint64_t(kThreads) * kU) + threadIdx.x;
        u32x4_t v[kU];
        if constexpr (kMode != 1) {
#pragma unroll
            for (int u = 0; u < kU; ++u) v[u] = cal_load<kNT>(base + u * kThreads);
        }
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (kMode == 0) {
#pragma unroll
            for (int u = 0; u < kU; ++u) acc ^= v[u].x ^ v[u].y ^ v[u].z ^ v[u].w;
        } else {
#pragma unroll
            for (int u = 0; u < kU; ++u) {
                if constexpr (kMode == 1) {
                    v[u] = u32x4_t{static_cast<uint32_t>(tile), uint32_t(u), threadIdx.x, 0u};
                } else {
                    v[u].x ^= flip; v[u].y ^= flip; v[u].z ^= flip; v[u].w ^= flip;
                }
                cal_store<kNT>(v[u], base + u * kThreads);
            }
        }
    }
    if constexpr (kMode == 0) {
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) acc ^= __shfl_xor(acc, off, 64);
        if ((threadIdx.x & 63u) == 0u) atomicXor(sink, acc);
    }
}

// w == +-0, tested on the bit pattern so that the member loop's skip stays on
// the scalar unit (a binary32 compare would be a vector instruction).
__device__ __forceinline__ bool is_zero_weight(float w) {
    return (__float_as_uint(w) << 1) == 0u;
}

struct RoundKey {
    uint32_t k0, k1;
};

// The member reverted in the same pass as an update (es_restore_update): its
// entry in the distinct-seed table and coef * sqrt(2 ln 2), coef = -sign sigma.
struct RestoreArg {
    uint32_t d;
    float coef_k;
};

// One step of the fused update: a lane's two 8-element groups at elements e
// and e + 8 kStepThreads.  acc = sum_d w_d eps_d (binary32, members in table
// order, zero weights skipped), theta <- round(theta + acc), store it.
// Rounding is to nearest even, or stochastic (kSR) with the draws of one
// domain-1 Philox call per group under the rounding key.
// kRestore: one member (rst) is reverted first, in registers, exactly as the
// perturb kernel does it (RNE(theta + coef eps)), and the update is added to
// the reverted values; with no live weight (add == false) the reverted values
// are stored as they are, as es_update would then leave them.
// kMaster == 1 (ES_UPDATE_MASTER): the update is added to the binary32
// masters at mb + 4 e instead (one rounding to binary32), and the bf16 values
// are rewritten as the masters rounded to nearest-even -- also with no live
// weight, when the masters are not written -- without reading them.
// kMaster == 2 (es_perturb_master): the members' terms are added to the
// masters in registers, m + sum w eps with one rounding for one member (the
// accumulation starts from m), and only the bf16 values are written.
//
// VALU-bound (es_noise.hpp): four Philox blocks in lockstep, and the step's
// input is loaded before the member loop and first used after it (or by the
// reverted member), so its latency lies under the loop.
template <bool kFast, bool kSR, bool kRows, bool kRestore, int kMaster>
__device__ __forceinline__ void update_step(const TileRef& r, uint64_t e,
                                            const Member* __restrict__ members,
                                            uint32_t n_distinct, RoundKey rk, RestoreArg rst,
                                            bool add, uintptr_t mb) {
    constexpr int kIn = kMaster != 0 ? 8 : 4;            // words of a group's input
    const uint32_t q_hi = tile_high_word<kRows>(r);
    const uint32_t g_hi = q_hi >> 1;                     // index >> 35
    // the masters of a full tile are taken in quads, lane t those at 4 t of
    // each 1024 elements, so that a 16-byte access covers 1 KB of consecutive
    // masters per wave (as in es_apply_master_kernel): with the member applied
    // first, 0.5B-shaped set, 1426 us by groups and 1385 by quads
    constexpr bool kQuads = kFast && kMaster != 0;
    constexpr uint32_t kQuadSlab = kStepThreads * 4;
    const uint64_t e4 = e - threadIdx.x * 4u;
    uint64_t eg[2], n[2];
    bool in[2];
    uint32_t raw[2][kIn];
    if constexpr (kQuads) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const f32x4_t v = __builtin_nontemporal_load(
                (const ES_GLOBAL f32x4_t*)(mb + 4 * (e4 + i * kQuadSlab)));
            uint32_t* x = raw[i / 2] + 4 * (i % 2);
            x[0] = __float_as_uint(v.x); x[1] = __float_as_uint(v.y);
            x[2] = __float_as_uint(v.z); x[3] = __float_as_uint(v.w);
        }
    }
#pragma unroll
    for (int g = 0; g < 2; ++g) {
        if constexpr (kQuads) break;
        eg[g] = e + uint64_t(g) * (kStepThreads * kGroupElems);
        in[g] = kFast || eg[g] < r.limit;
        n[g] = noise_index<kRows>(r, eg[g]);
        if (in[g]) {
            if constexpr (kMaster != 0) {
                float m[8];
                load_master(mb, eg[g], r.limit, m);
#pragma unroll
                for (int k = 0; k < 8; ++k) raw[g][k] = __builtin_bit_cast(uint32_t, m[k]);
            } else {
                load_group<kFast>(r.data, eg[g], r.limit, raw[g]);
            }
        } else {
#pragma unroll
            for (int k = 0; k < kIn; ++k) raw[g][k] = 0u;
        }
    }
    uint32_t q[4];
    if constexpr (kQuads) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
            q[i] = static_cast<uint32_t>(noise_index<kRows>(r, e4 + i * kQuadSlab) >> 2);
    } else {
        pair_quads(n, q);
    }
    float acc[16];
#pragma unroll
    for (int k = 0; k < 16; ++k)
        acc[k] = kMaster == 2 ? __builtin_bit_cast(float, raw[k / 8][k % 8]) : 0.0f;
    for (uint32_t d = 0; d < n_distinct; ++d) {
        const Member m = members[d];
        const bool live = !is_zero_weight(m.w_k);
        if constexpr (kRestore) {
            if (!live && d != rst.d) continue;
        } else {
            if (!live) continue;
        }
        es::Words w[4];
        float rad[8], c[8], sn[8];
        es::philox_quads<4>(q, q_hi, r.tensor_id, m.k0, m.k1, w);
        es::box_muller_quads<4>(w, rad, c, sn);
        if constexpr (kRestore) {
            if (d == rst.d) {
                float x[16];
                unpack_pair(raw, x);
                pair_axpy(rad, c, sn, rst.coef_k, x);
                pack_pair(x, raw);
            }
            if (!live) continue;
        }
        pair_axpy(rad, c, sn, m.w_k, acc);
    }
    if constexpr (kQuads) {
        typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t* x = raw[i / 2] + 4 * (i % 2);
            float m[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                m[k] = kMaster == 2 ? acc[4 * i + k] : __uint_as_float(x[k]);
                if (kMaster == 1 && add) m[k] += acc[4 * i + k];
            }
            if (kMaster == 1 && add) {
                const f32x4_t v = {m[0], m[1], m[2], m[3]};
                __builtin_nontemporal_store(v, (ES_GLOBAL f32x4_t*)(mb + 4 * (e4 + i * kQuadSlab)));
            }
            const u32x2_t b = {es::pack_bf16x2(m[0], m[1]), es::pack_bf16x2(m[2], m[3])};
            __builtin_nontemporal_store(b, (ES_GLOBAL u32x2_t*)(r.data + e4 + i * kQuadSlab));
        }
        return;
    }
#pragma unroll
    for (int g = 0; g < 2; ++g) {
        if constexpr (kQuads) break;
        if (!in[g]) break;
        const float* a = acc + 8 * g;
        uint32_t out[4];
        if constexpr (kMaster == 2) {
#pragma unroll
            for (int k = 0; k < 4; ++k) out[k] = es::pack_bf16x2(a[2 * k], a[2 * k + 1]);
        } else if constexpr (kMaster == 1) {
            float m[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) m[k] = __builtin_bit_cast(float, raw[g][k]);
            if (add) {
#pragma unroll
                for (int k = 0; k < 8; ++k) m[k] += a[k];
                store_master(mb, eg[g], r.limit, m);
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) out[k] = es::pack_bf16x2(m[2 * k], m[2 * k + 1]);
        } else if (kRestore && !add) {
#pragma unroll
            for (int k = 0; k < 4; ++k) out[k] = raw[g][k];
        } else if constexpr (kSR) {
            const es::Words d =
                es::philox4x32_10(static_cast<uint32_t>(n[g] >> 3), g_hi, r.tensor_id,
                                  es::kDomainRounding, rk.k0, rk.k1);
            const uint32_t draws[4] = {d.w0, d.w1, d.w2, d.w3};
#pragma unroll
            for (int k = 0; k < 4; ++k)
                out[k] = es::pack_bf16x2_sr(es::bf16_lo(raw[g][k]) + a[2 * k],
                                            es::bf16_hi(raw[g][k]) + a[2 * k + 1], draws[k]);
        } else {
#pragma unroll
            for (int k = 0; k < 4; ++k)
                out[k] = es::pack_bf16x2(es::bf16_lo(raw[g][k]) + a[2 * k],
                                         es::bf16_hi(raw[g][k]) + a[2 * k + 1]);
        }
        store_group<kFast>(r.data, eg[g], r.limit, out);
    }
}

// Fused update over the whole parameter list (member table and header
// written by es_prepare_kernel): the steps of the full tiles, then those of
// the tail tiles; with kRows the tiles of strided blocks, through their row
// maps; with kRestore the member rst reverted in the same pass.
template <bool kSR, bool kRows, bool kRestore, int kMaster>
__global__ __launch_bounds__(kStepThreads) void es_update_kernel(
    const TileDesc* __restrict__ tiles, uint64_t n_full, const DevRows* __restrict__ rows,
    const Member* __restrict__ members, const UpdateHeader* __restrict__ hdr, RoundKey rk, RestoreArg rst,
    const uint64_t* __restrict__ mdelta, StepShape sh) {
    const bool add = hdr->n_live != 0u;
    if (!kRestore && kMaster == 0 && !add) return;   // nothing to add: theta is not written
    const uint32_t n_distinct = hdr->n_distinct;
    auto mbase = [&](const TileRef& r, uint64_t i) -> uintptr_t {
        if constexpr (kMaster != 0) return master_base(mdelta, r, i);
        else return 0;
    };
    for_steps<kRows, 2>(tiles, n_full, rows, sh,
                        [&](auto full, const TileRef& r, uint64_t tile, uint64_t e) {
        update_step<decltype(full)::value, kSR, kRows, kRestore, kMaster>(
            r, e, members, n_distinct, rk, rst, add, mbase(r, tile));
    });
}

// The scratch of es_update_noalloc: one update's staged member tables, merged
// weights and header (the layout of a plan's scratch), in a fixed device
// array instead of memory allocated with a plan.  Each device holds its own
// copy until the process ends; host code reaches it only through the address
// hipGetSymbolAddress returns for the current device.
__device__ __align__(256) uint8_t scratch[kScratchBytes];

// Copy up to 1 KB of host-packed words (passed as kernel arguments) into
// device scratch: how es_update hands its member tables to the device
// without a host-side staging buffer or synchronisation.
__global__ __launch_bounds__(kAuxBlock) void es_stage_kernel(uint32_t* __restrict__ dst,
                                                          uint32_t n_words, StageChunk chunk) {
    for (uint32_t i = threadIdx.x; i < n_words; i += blockDim.x) dst[i] = chunk.words[i];
}

// Wave-wide reductions (one wavefront of 64 lanes).
__device__ __forceinline__ double wave_sum(double x) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off, 64);
    return x;
}
__device__ __forceinline__ float wave_min(float x) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) x = fminf(x, __shfl_xor(x, off, 64));
    return x;
}
__device__ __forceinline__ float wave_max(float x) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) x = fmaxf(x, __shfl_xor(x, off, 64));
    return x;
}

// Population z-score of n rewards by one wavefront, fp64, into LDS z[].
// Returns the status (1 if any reward is not finite; then z = 0).  All
// rewards equal gives z = 0 exactly.
__device__ int wave_zscore(const float* __restrict__ r, uint32_t n, double eps, double* z) {
    const uint32_t lane = threadIdx.x;
    double s = 0.0;
    float lo = INFINITY, hi = -INFINITY;
    int bad = 0;
    for (uint32_t i = lane; i < n; i += 64) {   // each lane's entries of z[] stay its own
        const float x = r[i];
        bad |= !isfinite(x);
        s += static_cast<double>(x);
        lo = fminf(lo, x);
        hi = fmaxf(hi, x);
        z[i] = static_cast<double>(x);
    }
    bad = __any(bad);
    lo = wave_min(lo);
    hi = wave_max(hi);
    if (bad || lo == hi) {
        for (uint32_t i = lane; i < n; i += 64) z[i] = 0.0;
        return bad ? 1 : 0;
    }
    const double mu = wave_sum(s) / static_cast<double>(n);
    double q = 0.0;
    for (uint32_t i = lane; i < n; i += 64) {
        const double d = z[i] - mu;
        q += d * d;
    }
    const double sd = sqrt(wave_sum(q) / static_cast<double>(n));
    for (uint32_t i = lane; i < n; i += 64) z[i] = (z[i] - mu) / (sd + eps);
    return 0;
}

__global__ __launch_bounds__(64) void es_zscore_kernel(const float* __restrict__ r, uint32_t n,
                                                       double eps, float* __restrict__ z_out,
                                                       int32_t* __restrict__ status_out) {
    __shared__ double z[ES_MAX_MEMBERS];
    const int status = wave_zscore(r, n, eps, z);
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < n; i += 64) z_out[i] = static_cast<float>(z[i]);
    if (status_out != nullptr && threadIdx.x == 0) *status_out = status;
}

// The population's tables, staged in device scratch or inline in the kernel
// arguments (up to kInlineMembers members, 2 KB: one launch instead of three).
struct StagedTables {
    const MemberIn* __restrict__ min;
    const DistinctIn* __restrict__ din;
    __device__ __forceinline__ DistinctIn distinct(uint32_t d) const { return din[d]; }
    __device__ __forceinline__ MemberIn member(uint32_t m) const { return min[m]; }
};
constexpr uint32_t kInlineMembers = 128;
struct InlineTables {
    uint32_t k0[kInlineMembers], k1[kInlineMembers];
    uint16_t first[kInlineMembers], count[kInlineMembers];
    int16_t member_index[kInlineMembers];        // reward index, or its complement for sign -1
    __device__ __forceinline__ DistinctIn distinct(uint32_t d) const {
        return DistinctIn{k0[d], k1[d], first[d], count[d]};
    }
    __device__ __forceinline__ MemberIn member(uint32_t m) const {
        const int32_t v = member_index[m];
        return MemberIn{static_cast<uint32_t>(v < 0 ? ~v : v), v < 0 ? -1 : 1};
    }
};

// z-score (or rewards as weights), then one merged weight per distinct seed:
// w_d = sum over its members (in member order) of c * sign * zhat, fp64,
// stored as binary32 with the seed's key for es_update_kernel.  One wave,
// latency-bound: a generation of 4 over 1 M parameters takes 38.0 us with the
// tables inline, 44.6 us with them staged by two launches before this one.
template <class Tables>
__global__ __launch_bounds__(64) void es_prepare_kernel(const float* __restrict__ r, uint32_t n,
                                                        double eps, uint32_t flags, double c,
                                                        Tables tab, uint32_t n_distinct,
                                                        Member* __restrict__ out,
                                                        UpdateHeader* __restrict__ hdr,
                                                        float* __restrict__ z_out,
                                                        int32_t* __restrict__ status_out) {
    __shared__ double z[ES_MAX_MEMBERS];
    const uint32_t lane = threadIdx.x;
    int status;
    if (flags & ES_REWARDS_ARE_WEIGHTS) {
        int bad = 0;
        for (uint32_t i = lane; i < n; i += 64) {
            const float x = r[i];
            bad |= !isfinite(x);
            z[i] = static_cast<double>(x);
        }
        status = __any(bad) ? 1 : 0;
    } else {
        status = wave_zscore(r, n, eps, z);
    }
    __syncthreads();
    if (z_out != nullptr)
        for (uint32_t i = lane; i < n; i += 64) z_out[i] = static_cast<float>(status ? 0.0 : z[i]);
    uint32_t live = 0;
    for (uint32_t d = lane; d < n_distinct; d += 64) {
        const DistinctIn di = tab.distinct(d);
        double w = 0.0;
        for (uint32_t m = di.first; m < di.first + di.count; ++m) {
            const MemberIn mi = tab.member(m);
            w += c * static_cast<double>(mi.sign) * z[mi.reward_index];
        }
        const float wf = status ? 0.0f : static_cast<float>(w * kSqrt2Ln2Double);
        out[d] = Member{di.k0, di.k1, wf, 0u};
        live += (wf != 0.0f) ? 1u : 0u;
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) live += __shfl_xor(live, off, 64);
    if (lane == 0) {
        *hdr = UpdateHeader{n_distinct, live, status, 0u};
        if (status_out != nullptr) *status_out = status;
    }
}

__global__ __launch_bounds__(kAuxBlock) void es_philox_words_kernel(uint32_t k0, uint32_t k1,
                                                                 uint32_t tensor_id, uint32_t domain,
                                                                 uint64_t quad0, uint64_t n_quads,
                                                                 uint4* __restrict__ out) {
    const uint64_t i = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i >= n_quads) return;
    const uint64_t q = quad0 + i;
    const es::Words w = es::philox4x32_10(static_cast<uint32_t>(q), static_cast<uint32_t>(q >> 32),
                                          tensor_id, domain, k0, k1);
    out[i] = make_uint4(w.w0, w.w1, w.w2, w.w3);
}

__global__ __launch_bounds__(kAuxBlock) void es_normals_kernel(uint32_t k0, uint32_t k1,
                                                            uint32_t tensor_id, uint64_t elem0,
                                                            uint64_t n, float* __restrict__ out) {
    const uint64_t q = (elem0 >> 2) + uint64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (4 * q >= elem0 + n) return;
    float e[4];
    es::quad_normals(static_cast<uint32_t>(q), static_cast<uint32_t>(q >> 32), tensor_id, k0, k1, e);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const uint64_t j = 4 * q + k;
        if (j >= elem0 && j < elem0 + n) out[j - elem0] = e[k];
    }
}

using PerturbKernel = void (*)(const TileDesc*, uint64_t, const DevRows*, Streams, StepShape);
using UpdateKernel = void (*)(const TileDesc*, uint64_t, const DevRows*, const Member*,
                              const UpdateHeader*, RoundKey, RestoreArg, const uint64_t*,
                              StepShape);
using ApplyMasterKernel = void (*)(const TileDesc*, uint64_t, const DevRows*, Streams,
                                   const uint64_t*, StepShape);

// streams: 1 (perturb / restore), 2 (swap, two keys), 3 (swap, one key);
// rows: the launch over strided blocks' tiles; kG: groups per lane and step.
template <int kG>
PerturbKernel perturb_kernel(int streams, bool rows) {
    switch (streams) {
        case 1: return rows ? es_perturb_kernel<1, true, kG> : es_perturb_kernel<1, false, kG>;
        case 2: return rows ? es_perturb_kernel<2, true, kG> : es_perturb_kernel<2, false, kG>;
        default: return rows ? es_perturb_kernel<3, true, kG> : es_perturb_kernel<3, false, kG>;
    }
}

ApplyMasterKernel apply_master_kernel(bool rows) {
    return rows ? es_apply_master_kernel<true> : es_apply_master_kernel<false>;
}

// Tile shapes instantiated: T lanes per workgroup x U groups per lane.
#define ES_TILE_SHAPES(X) X(256, 4) X(256, 8) X(512, 4) X(512, 8) X(1024, 4) X(1024, 8)

using ChecksumKernel = void (*)(const TileDesc*, uint64_t, uint64_t, const DevRows*, uint32_t,
                                unsigned long long*);

ChecksumKernel checksum_kernel(int threads, int groups, bool rows, bool cut) {
#define ES_CASE(T, U)                                                                   \
    if (threads == T && groups == U)                                                    \
        return rows ? (cut ? es_checksum_kernel<T, U, true, true>                       \
                           : es_checksum_kernel<T, U, true, false>)                     \
                    : (cut ? es_checksum_kernel<T, U, false, true>                      \
                           : es_checksum_kernel<T, U, false, false>);
    ES_TILE_SHAPES(ES_CASE)
#undef ES_CASE
    return nullptr;
}

template <bool kRestore>
UpdateKernel update_kernel_for(bool stochastic, bool rows) {
    if (rows)
        return stochastic ? es_update_kernel<true, true, kRestore, 0>
                          : es_update_kernel<false, true, kRestore, 0>;
    return stochastic ? es_update_kernel<true, false, kRestore, 0>
                      : es_update_kernel<false, false, kRestore, 0>;
}

// The update into binary32 masters (mode 1) and the application of members
// from the masters (mode 2), both rewriting the bf16 values.
UpdateKernel update_master_kernel(bool rows, bool apply = false) {
    if (apply)
        return rows ? es_update_kernel<false, true, false, 2>
                    : es_update_kernel<false, false, false, 2>;
    return rows ? es_update_kernel<false, true, false, 1>
                : es_update_kernel<false, false, false, 1>;
}

// restore: the update with one member reverted in the same pass.
UpdateKernel update_kernel(bool stochastic, bool rows, bool restore) {
    return restore ? update_kernel_for<true>(stochastic, rows)
                   : update_kernel_for<false>(stochastic, rows);
}

// ---- quantized path: int8 and E4M3 codes (helpers in es_quant.hpp, es_fp8.hpp) ----

// Kernel arguments of one quantized pass: the key of the update's rounding
// draws, and for perturb / restore the single member inline (for a swap, m is
// the member applied and m_from the member reverted before it).
struct QPass {
    uint32_t dk0, dk1;
    uint32_t pad0, pad1;
    Member m;
    Member m_from;
};

// Perturb / restore of one 16-code group from its noise: per quad of codes one
// block, whose words give the four normals and the four rounding draws.  The
// scale's reciprocal is folded into the pair's radius factor, and d + f is one
// FMA.
template <bool kNegate>
__device__ __forceinline__ void qperturb_group(const uint32_t raw[4], const esq::GroupNoise& gn,
                                               float w_k, const float inv[2], uint32_t out[4]) {
    // an invalid scale has inv = 0: its step is 0 and its codes clamp to
    // [-128, 127], i.e. they are left as they are; the bound keeps a step in
    // quanta finite (it saturates every code long before), so that no product
    // with a zero cosine is a NaN
    const float wk_inv[2] = {__builtin_amdgcn_fmed3f(w_k * inv[0], -0x1p100f, 0x1p100f),
                             __builtin_amdgcn_fmed3f(w_k * inv[1], -0x1p100f, 0x1p100f)};
    const int32_t lo[2] = {inv[0] != 0.0f ? -127 : -128, inv[1] != 0.0f ? -127 : -128};
    const esq::SpareBits bits;
    float v[16];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const uint32_t ws[4] = {gn.w[c].w0, gn.w[c].w1, gn.w[c].w2, gn.w[c].w3};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int p = 2 * c + i / 2;
            const float t = wk_inv[c >> 1] * gn.rad[p];
            v[4 * c + i] = __builtin_fmaf(t, (i & 1) ? gn.sn[p] : gn.c[p],
                                          esq::spare_one_plus(ws[i], bits));
        }
    }
    es::heavy_phase();
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        int32_t code[4];
#pragma unroll
        for (int i = 0; i < 4; ++i)
            code[i] = esq::qstep9<kNegate>(static_cast<int8_t>(raw[c] >> (8 * i)), v[4 * c + i],
                                           lo[c >> 1]);
        out[c] = esq::pack_codes(code[0], code[1], code[2], code[3]);
    }
    es::simple_phase();
}

// Code formats of a quantized plan.
constexpr int kFmtInt8 = 0;
constexpr int kFmtE4M3 = 1;

// fp8 perturb / restore of one 16-code group from its noise (as above).  The
// scale's reciprocal is folded into the pair's radius factor; x = v -+ d is
// one fused multiply-add, and the restore rounds with the complementary
// rule (operand ~U for U), so it undoes the perturbation inside a binade.
template <bool kNegate>
__device__ __forceinline__ void f8perturb_group(const uint32_t raw[4], const esq::GroupNoise& gn,
                                                float w_k, const float inv[2], uint32_t out[4]) {
    const float wk_inv[2] = {w_k * inv[0], w_k * inv[1]};
    const esf::DrawBits bits;
    float x[16];
    uint32_t a[16];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const uint32_t ws[4] = {gn.w[c].w0, gn.w[c].w1, gn.w[c].w2, gn.w[c].w3};
        esf::decode4(raw[c], x + 4 * c);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int p = 2 * c + i / 2;
            const float t = wk_inv[c >> 1] * gn.rad[p];
            const uint32_t u = esf::draw9_fixed(ws[i], bits);
            x[4 * c + i] = __builtin_fmaf(kNegate ? -t : t, (i & 1) ? gn.sn[p] : gn.c[p],
                                          x[4 * c + i]);
            a[4 * c + i] = kNegate ? ~u : u;
        }
    }
    esf::round16(x, a, out);
}

// Perturb (kNegate false) or restore of one 16-code group in the plan's
// format, codes with an invalid scale or a not-a-number code left as they are.
template <bool kNegate, int kFmt>
__device__ __forceinline__ void qmember_group(const uint32_t raw[4], const esq::GroupNoise& gn,
                                              float w_k, const float inv[2], uint32_t out[4]) {
    if constexpr (kFmt == kFmtE4M3) {
        f8perturb_group<kNegate>(raw, gn, w_k, inv, out);
        esf::keep_special(raw, inv[0], inv[1], out);
    } else {
        qperturb_group<kNegate>(raw, gn, w_k, inv, out);
    }
}

// The quantized passes.
enum class QKind { kPerturb, kRestore, kUpdate, kSwap };

// One step of a quantized pass (int8 or E4M3 codes, kFmt): the lane's 16-code
// group at code e of its tensor, the step in scale units (binary32) and the
// stochastically rounded, clamped code.  e indexes the codes and scales at
// hand; n, the whole-tensor index of code e, selects the noise and the
// rounding draws.  A swap reverts the member ps.m_from and applies ps.m in
// registers, the codes of the two separate passes; members that share a key
// (antithetic partners) share their noise.
//
// VALU-bound: four Philox blocks in lockstep per group and stream
// (es_noise.hpp); the codes and scales are loaded first and used after the
// noise, which their latency lies under.
template <bool kFast, QKind kKind, int kFmt>
__device__ __forceinline__ void qstep_group(const esq::QTileRef& r, uint32_t e,
                                            const Member* __restrict__ members,
                                            uint32_t n_members, const QPass& ps) {
    const uint32_t n = esq::qnoise_index(r, e);
    uint32_t raw[4], out[4];
    float sc[2], inv[2];
    esq::qload<kFast>(r.data, e, r.numel, raw);
    esq::group_scales(r, e, sc);
    if constexpr (kKind != QKind::kUpdate) {
        esq::GroupNoise gn;
        const Member& first = kKind == QKind::kSwap ? ps.m_from : ps.m;
        esq::group_noise(n, r.tensor_id, first.k0, first.k1, gn);
        inv[0] = esq::inv_scale(sc[0]);
        inv[1] = esq::inv_scale(sc[1]);
        constexpr bool kNegate = kKind != QKind::kPerturb;
        qmember_group<kNegate, kFmt>(raw, gn, first.w_k, inv, out);
        if constexpr (kKind == QKind::kSwap) {
            if (ps.m.k0 != ps.m_from.k0 || ps.m.k1 != ps.m_from.k1)
                esq::group_noise(n, r.tensor_id, ps.m.k0, ps.m.k1, gn);
#pragma unroll
            for (int k = 0; k < 4; ++k) raw[k] = out[k];
            qmember_group<false, kFmt>(raw, gn, ps.m.w_k, inv, out);
        }
    } else {
        float acc[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[i] = 0.0f;
        for (uint32_t d = 0; d < n_members; ++d) {
            const Member m = members[d];
            if (is_zero_weight(m.w_k)) continue;
            esq::GroupNoise gn;
            esq::group_noise(n, r.tensor_id, m.k0, m.k1, gn);
            pair_axpy(gn.rad, gn.c, gn.sn, m.w_k, acc);
        }
        inv[0] = esq::inv_scale(sc[0]);
        inv[1] = esq::inv_scale(sc[1]);
        const es::Words da =
            es::philox4x32_10(n >> 3, 0u, r.tensor_id, es::kDomainRounding, ps.dk0, ps.dk1);
        const es::Words db =
            es::philox4x32_10((n >> 3) + 1u, 0u, r.tensor_id, es::kDomainRounding, ps.dk0, ps.dk1);
        const uint32_t dw[8] = {da.w0, da.w1, da.w2, da.w3, db.w0, db.w1, db.w2, db.w3};
        if constexpr (kFmt == kFmtE4M3) {
            // x = v + acc / s (one fused multiply-add), rounded onto the
            // grid with the threshold 1 - r 2^-16 (operand r 2^16)
            float x[16];
            uint32_t a[16];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                esf::decode4(raw[k], x + 4 * k);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int c = 4 * k + i;
                    const uint32_t d = dw[c >> 1];
                    a[c] = (c & 1) ? (d & 0xFFFF0000u) : (d << 16);
                    x[c] = __builtin_fmaf(acc[c], inv[c / 8], x[c]);
                }
            }
            esf::round16(x, a, out);
            esf::keep_special(raw, inv[0], inv[1], out);
        } else {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                uint32_t w = 0;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int c = 4 * k + i;
                    const int32_t q = static_cast<int8_t>(raw[k] >> (8 * i));
                    const uint32_t draw = (dw[c >> 1] >> (16 * (c & 1))) & 0xFFFFu;
                    const int32_t v =
                        inv[c / 8] != 0.0f ? esq::qstep(q, acc[c] * inv[c / 8], draw) : q;
                    w |= (static_cast<uint32_t>(v) & 0xFFu) << (8 * i);
                }
                out[k] = w;
            }
        }
    }
    esq::qstore<kFast>(r.data, e, r.numel, out);
}

// A pass over the whole quantized parameter list: perturb / restore (one
// inline member, draws from its own noise words), swap (two inline members)
// or the update (member table and header written by es_prepare_kernel, draws
// of domain 1 under the rounding seed).  A workgroup takes `steps` steps of 256
// lanes x 16 codes, 2^full_shift workgroups per full tile of tile_elems codes; a
// tensor's codes beyond its full tiles have as many workgroups as they need, so
// that short tensors leave none without work (10 000 tensors of 64 codes and one
// of 60 000: swap 24 us, update of 4 36; with every tail cut alike, for the
// longest, 155 and 205).
// first_full and first_step are the launch's first full tile and tail workgroup.
struct QShape {
    uint32_t tile_elems, n_tensors;
    uint32_t full_shift, steps;
    uint64_t first_full;
    uint32_t first_step;
};
constexpr uint32_t kQStepCodes = kStepThreads * esq::kQGroup;

template <QKind kKind, int kFmt>
__global__ __launch_bounds__(kStepThreads) void es_qpass_kernel(
    const esq::DevQTensor* __restrict__ tab, uint64_t n_full, const Member* __restrict__ members,
    const UpdateHeader* __restrict__ hdr, QPass ps, QShape sh) {
    uint32_t n_members = 1;
    if constexpr (kKind == QKind::kUpdate) {
        if (hdr->n_live == 0u) return;      // nothing to add: codes are not written
        n_members = hdr->n_distinct;
    }
    const uint64_t full_items = n_full << sh.full_shift;
    const uint64_t i = blockIdx.x;
    if (i < full_items) {
        const uint32_t part = static_cast<uint32_t>(i) & ((1u << sh.full_shift) - 1u);
        const esq::QTileRef r = esq::qlocate_full(
            tab, sh.n_tensors, sh.first_full + (i >> sh.full_shift), sh.tile_elems);
        const uint32_t e0 = r.elem0 + part * sh.steps * kQStepCodes + threadIdx.x * esq::kQGroup;
#pragma unroll 1
        for (uint32_t k = 0; k < sh.steps; ++k)
            qstep_group<true, kKind, kFmt>(r, e0 + k * kQStepCodes, members, n_members, ps);
        return;
    }
    const esq::QTileRef r =
        esq::qlocate_step(tab, sh.n_tensors, static_cast<uint32_t>(i - full_items) + sh.first_step,
                          sh.tile_elems, sh.steps * kQStepCodes);
    const uint32_t e0 = r.elem0 + threadIdx.x * esq::kQGroup;
#pragma unroll 1
    for (uint32_t k = 0; k < sh.steps; ++k) {
        const uint32_t e = e0 + k * kQStepCodes;
        if (e >= r.numel) return;
        qstep_group<false, kKind, kFmt>(r, e, members, n_members, ps);
    }
}

using QPassKernel = void (*)(const esq::DevQTensor*, uint64_t, const Member*, const UpdateHeader*,
                             QPass, QShape);

template <int kFmt>
QPassKernel qpass_kernel_for(QKind kind) {
    switch (kind) {
        case QKind::kPerturb: return es_qpass_kernel<QKind::kPerturb, kFmt>;
        case QKind::kRestore: return es_qpass_kernel<QKind::kRestore, kFmt>;
        case QKind::kUpdate: return es_qpass_kernel<QKind::kUpdate, kFmt>;
        default: return es_qpass_kernel<QKind::kSwap, kFmt>;
    }
}

QPassKernel qpass_kernel(QKind kind, int format) {
    return format == kFmtE4M3 ? qpass_kernel_for<kFmtE4M3>(kind) : qpass_kernel_for<kFmtInt8>(kind);
}

// Quantized plan: the same sum with b the code's 8 bits and j the element's
// whole-tensor index (qnoise_index; a 16-code group's indices are
// consecutive).
template <int kThreads, int kU, bool kCut>
__global__ __launch_bounds__(kThreads) void es_qchecksum_kernel(
    const esq::DevQTensor* __restrict__ tab, uint64_t n_full, uint64_t n_tail, uint32_t n_tensors,
    uint32_t shift, unsigned long long* __restrict__ out) {
    constexpr uint32_t kTileElems = uint32_t(kThreads) * kU * esq::kQGroup;
    const uint32_t cut = kCut ? shift : 0u, slots = kU >> cut, parts = (1u << cut) - 1u;
    uint64_t acc = 0;
    for (uint64_t i = blockIdx.x; i < n_full << cut; i += gridDim.x) {
        const esq::QTileRef r = esq::qlocate_full(tab, n_tensors, i >> cut, kTileElems);
        const uint32_t u0 = (static_cast<uint32_t>(i) & parts) * slots;
        const uint64_t salt = uint64_t(r.tensor_id) * kSumT;
#pragma unroll 1
        for (uint32_t u = u0; u < u0 + slots; ++u) {
            const uint32_t e = r.elem0 + (u * kThreads + threadIdx.x) * esq::kQGroup;
            uint32_t raw[4];
            esq::qload<true>(r.data, e, r.numel, raw);
            acc += checksum_terms<esq::kQGroup, 8, false>(raw, esq::qnoise_index(r, e), 0, salt);
        }
    }
    for (uint64_t i = blockIdx.x; i < n_tail << cut; i += gridDim.x) {
        const esq::QTileRef r = esq::qlocate_tail(tab, n_tensors, i >> cut, kTileElems);
        const uint32_t u0 = (static_cast<uint32_t>(i) & parts) * slots;
        const uint64_t salt = uint64_t(r.tensor_id) * kSumT;
#pragma unroll 1
        for (uint32_t u = u0; u < u0 + slots; ++u) {
            const uint32_t e = r.elem0 + (u * kThreads + threadIdx.x) * esq::kQGroup;
            if (e >= r.numel) break;
            uint32_t raw[4];
            esq::qload<false>(r.data, e, r.numel, raw);
            const uint32_t n = esq::qnoise_index(r, e);
            acc += checksum_terms<esq::kQGroup, 8, true>(raw, n, uint64_t(n) + (r.numel - e),
                                                         salt);
        }
    }
    add_workgroup_sum<kThreads>(acc, out);
}

using QChecksumKernel = void (*)(const esq::DevQTensor*, uint64_t, uint64_t, uint32_t, uint32_t,
                                 unsigned long long*);

QChecksumKernel qchecksum_kernel(int threads, int groups, bool cut) {
#define ES_CASE(T, U)                                                                   \
    if (threads == T && groups == U)                                                    \
        return cut ? es_qchecksum_kernel<T, U, true> : es_qchecksum_kernel<T, U, false>;
    ES_TILE_SHAPES(ES_CASE)
#undef ES_CASE
    return nullptr;
}

}  // namespace

// ------------------------------------------------------------------------
// Host side
// ------------------------------------------------------------------------

struct es_plan {
    int device = -1;
    uint32_t n_tensors = 0;
    uint64_t numel = 0;
    uint64_t n_full = 0;            // full tiles (16-byte path)
    uint64_t n_tail = 0;            // tail tiles (bounds-checked path)
    uint64_t n_rfull = 0;           // full and tail tiles of strided blocks, after the
    uint64_t n_rtail = 0;           //   others, each with a row map
    TailIndex tails = {};           // the tail tiles' steps,
    TailIndex rtails = {};          //   and those of strided blocks
    int cus = 0;                    // compute units of the device
    uint32_t grid_sum = 0;          // workgroups of the checksum launch
    uint32_t grid_sum_rows = 0;     //   and of its launch over strided blocks
    int threads = kDefaultThreads;  // lanes per workgroup of the tile kernels
    int groups = kDefaultGroups;    // 8-element groups per lane per tile
    uint64_t tile_elems = 0;        // threads * groups * 8
    TileDesc* d_tiles = nullptr;    // n_full full-tile then n_tail tail-tile descriptors, then
                                    //   n_rfull + n_rtail of strided blocks
    DevRows* d_rows = nullptr;      // their row maps (same allocation, after the descriptors)
    uint8_t* d_scratch = nullptr;   // kScratchBytes
    // each tensor's or block's bf16 data and element count, in plan order
    std::vector<std::pair<uintptr_t, uint64_t>> owners;
    // binary32 masters (es_plan_set_master): per tile, the delta D with
    // master address = D + 2 * bf16 address (its tensor's master minus twice
    // its bf16 data pointer, mod 2^64); null when none are attached
    uint64_t* d_master = nullptr;
};

struct es_qplan {
    int device = -1;
    uint32_t n_tensors = 0;
    uint64_t numel = 0;
    uint64_t n_full = 0;
    uint64_t n_tail = 0;
    uint32_t steps = 1;             // steps per workgroup of a pass
    uint32_t n_tail_steps = 0;      // its workgroups over the tail tiles
    uint32_t grid = 0;              // workgroups of the checksum launch
    int threads = kDefaultThreads;
    int groups = kDefaultQGroups;   // 16-code groups per lane per tile
    int format = kFmtInt8;          // ES_QFORMAT_INT8 or ES_QFORMAT_E4M3 (one per plan)
    esq::DevQTensor* d_tab = nullptr;
    uint8_t* d_scratch = nullptr;   // kScratchBytes, as the bf16 plan's
};

namespace {

// Integer from the environment within [lo, hi], else the default.
int env_int(const char* name, int dflt, int lo, int hi) {
    const char* v = std::getenv(name);
    if (v == nullptr) return dflt;
    const int x = std::atoi(v);
    return (x >= lo && x <= hi) ? x : dflt;
}

int check_device(const es_plan_t* p) {
    int dev = -1;
    const hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
    if (dev != p->device)
        return fail(ES_ERR_DEVICE, "current device " + std::to_string(dev) +
                                       " differs from the plan's device " +
                                       std::to_string(p->device));
    return ES_OK;
}

// The launches of a pass over a plan: one over the tiles of tensors and
// contiguous blocks, and one over the tiles of strided blocks with their
// row maps; a part with no tiles is left out.
struct Segment {
    const TileDesc* tiles;
    uint64_t n_full, n_tail;
    const DevRows* rows;            // null for the first part
    TailIndex tails;
    uint32_t grid_sum;
};

int plan_segments(const es_plan_t* p, Segment seg[2]) {
    int n = 0;
    if (p->n_full + p->n_tail > 0)
        seg[n++] = Segment{p->d_tiles, p->n_full, p->n_tail, nullptr, p->tails, p->grid_sum};
    if (p->n_rfull + p->n_rtail > 0)
        seg[n++] = Segment{p->d_tiles + p->n_full + p->n_tail, p->n_rfull, p->n_rtail, p->d_rows,
                           p->rtails, p->grid_sum_rows};
    return n;
}

// Steps per full tile of tile_elems elements (a power of two, at least 8192)
// with `groups` groups per lane.
uint32_t full_tile_shift(uint64_t tile_elems, int groups) {
    const uint64_t step = uint64_t(kStepThreads) * groups * kGroupElems;
    uint32_t shift = 0;
    while ((step << shift) < tile_elems) ++shift;
    return shift;
}

// The device's descriptor of a tile.
TileDesc tile_desc(const DevTile& d) {
    return TileDesc{d.data, d.elem0, static_cast<uint32_t>(d.limit - d.elem0), d.tensor_id, 0u,
                    0u};
}

// The first and guide entries of n tail descriptors, and their index.  A plan
// has fewer than 2^32 tail steps: each is 8 KB of the device's memory or the end
// of one of 2^20 tensors or 2^28 rows.
TailIndex index_tails(TileDesc* tails, uint64_t n) {
    uint64_t steps = 0;
    for (uint64_t t = 0; t < n; ++t) {
        tails[t].first = static_cast<uint32_t>(steps);
        steps += (tails[t].len + kTailStep - 1) / kTailStep;
    }
    const TailIndex ix{static_cast<uint32_t>(n), static_cast<uint32_t>(steps),
                       steps > 0 ? (n << 32) / steps : 0};
    uint64_t next = 0;                      // first guide entry not yet written
    for (uint64_t t = 0, j = 0; t < n; ++t)
        for (const uint64_t end = t + 1 < n ? tails[t + 1].first : steps; j < end; ++j)
            if ((j * ix.ratio) >> 32 == next) tails[next++].guide = static_cast<uint32_t>(t);
    while (next < n) tails[next++].guide = static_cast<uint32_t>(n - 1);
    return ix;
}

// The launches of a pass, in order: of n_full full tiles in 2^full_shift
// workgroups each, then of n_steps tail steps in a workgroup each.  A launch has fewer than 2^32 lanes (HIP's limit for a dimension), and a
// plan's memory can hold more steps than that (an update from 2^36 elements,
// 137 GB, on), so a pass over a larger plan is several launches:
// launch(first full tile, full tiles, first tail step, workgroups) for each,
// until one fails.  `cap` (at least a tile's workgroups) is the most of them in a
// launch.
constexpr uint64_t kMaxStepGrid = (uint64_t(1) << 32) / kStepThreads - 1;

template <class Launch>
int for_step_launches(uint64_t n_full, uint64_t n_steps, uint32_t full_shift, Launch launch,
                      uint64_t cap = kMaxStepGrid) {
    uint64_t f = 0, t = 0;
    while (f < n_full || t < n_steps) {
        const uint64_t full = std::min(n_full - f, cap >> full_shift);
        const uint64_t room = f + full < n_full ? 0 : cap - (full << full_shift);
        const uint64_t tail = std::min(n_steps - t, room);
        const int rc = launch(f, full, static_cast<uint32_t>(t),
                              static_cast<uint32_t>((full << full_shift) + tail));
        if (rc != ES_OK) return rc;
        f += full;
        t += tail;
    }
    return ES_OK;
}

// The arguments of one launch over part of a segment: its tiles, the full ones
// among them, and their row maps and master deltas (each null where the pass
// takes none).
struct StepLaunch {
    const TileDesc* tiles;
    uint64_t n_full;
    const DevRows* rows;
    const uint64_t* mdelta;
    StepShape shape;
    dim3 grid;
};

// launch(StepLaunch) for each launch of a pass of `groups` groups per lane over
// a segment.  One that fails is named by the call and the kernel (formatted only
// then).
template <class Launch>
int launch_steps(const es_plan_t* p, const Segment& g, int groups, const uint64_t* mdelta,
                 const char* call, const char* kernel, Launch launch) {
    const uint32_t shift = full_tile_shift(p->tile_elems, groups);
    return for_step_launches(
        g.n_full, g.tails.n_steps, shift,
        [&](uint64_t first, uint64_t full, uint32_t step0, uint32_t grid) {
            launch(StepLaunch{
                g.tiles + first, full, g.rows != nullptr ? g.rows + first : nullptr,
                mdelta != nullptr ? mdelta + first : nullptr,
                StepShape{shift, step0, g.n_full - first, g.tails},
                dim3(grid)});
            const hipError_t e = hipGetLastError();
            return e != hipSuccess ? hip_fail(e, std::string(call) + kernel + " launch") : ES_OK;
        });
}

// Groups per lane and step of perturb, swap and the stream pass in full tiles:
// four, or two where four would leave wave slots empty (fewer than eight
// workgroups per CU, 16.8 M elements).  Two and four groups, us:
//   perturb: 1 M elements 2.8 and 3.4, 8.4 M 7.7 and 8.0, 21 M 14.3 and 14.5,
//   50 M 33.0 and 32.7, 134 M 85.7 and 84.7, 537 M 338.4 and 337.5;
//   same-key swap: 21 M 14.4 and 14.8, 134 M 85.3 and 84.0, 537 M 340 and 335;
//   two-key swap: 17 M 19.6 and 19.8, 21 M 21.6 and 20.6, 134 M 123 and 119,
//   4 G 3780 and 3640, 22.7 G 21 560 and 20 880 (eight waves per SIMD with two,
//   five with four: these passes don't lack waves).
// Over the largest sets two are better for a single key, perturb 4 G 2527 and
// 2584, 22.7 G 14 250 and 15 000, the stream pass alike, and follow the same rule.
bool four_groups(const es_plan_t* p, const Segment& g) {
    const uint64_t elems = g.n_full * p->tile_elems;
    return elems >= uint64_t(p->cus) * 8 * (kStepThreads * 4 * kGroupElems);
}

// A checksum launch: tiles cut in halves down to single group slots while that
// gives at most kSumItems workgroups, each with one atomic on the result, else
// whole tiles over `grid` workgroups.  1 M parameters: 29 us whole, 12 in
// slots; 24 M in 200 odd-sized tensors 46 whole, 34 in halves (800 workgroups),
// 54 in slots (3600); 60 M in 216 (1800 halves) stay whole, 51 us.
struct SumLaunch {
    uint32_t shift, grid;
};
SumLaunch sum_launch(uint64_t n_full, uint64_t n_tail, int groups, uint32_t grid) {
    constexpr uint64_t kSumItems = 1024;
    const uint64_t tiles = std::max<uint64_t>(std::max(n_full, n_tail), 1);
    SumLaunch l{0u, grid};
    while ((2 << l.shift) <= groups && (tiles << (l.shift + 1)) <= kSumItems) ++l.shift;
    if (l.shift > 0) l.grid = static_cast<uint32_t>(tiles << l.shift);
    return l;
}

// One pass of the perturb kernel: streams = 1 (seed[0], coef[0]), 2 (two
// keys) or 3 (both coefficients on seed[0]).
int launch_streams(es_plan_t* p, int streams, const uint64_t* seed, const double* coef,
                   hipStream_t s) {
    Streams st = {};
    const int terms = streams == 1 ? 1 : 2;
    for (int m = 0; m < terms; ++m) {
        const uint64_t sd = streams == 3 ? seed[0] : seed[m];
        st.k0[m] = static_cast<uint32_t>(sd);
        st.k1[m] = static_cast<uint32_t>(sd >> 32);
        st.coef_k[m] = static_cast<float>(coef[m] * kSqrt2Ln2Double);
    }
    Segment seg[2];
    const int n_seg = plan_segments(p, seg);
    for (int k = 0; k < n_seg; ++k) {
        const Segment& g = seg[k];
        const bool four = four_groups(p, g);
        const bool strided = g.rows != nullptr;
        const PerturbKernel kernel = four ? perturb_kernel<4>(streams, strided)
                                          : perturb_kernel<2>(streams, strided);
        const int rc = launch_steps(
            p, g, four ? 4 : 2, nullptr, "", "es_perturb_kernel", [&](const StepLaunch& l) {
                hipLaunchKernelGGL(kernel, l.grid, dim3(kStepThreads), 0, s, l.tiles, l.n_full,
                                   l.rows, st, l.shape);
            });
        if (rc != ES_OK) return rc;
    }
    return ES_OK;
}

int perturb_impl(es_plan_t* p, uint64_t seed, int32_t sign, float sigma, es_stream_t stream,
                 const char* name) {
    if (p == nullptr) return fail(ES_ERR_INVALID_ARG, std::string(name) + ": null plan");
    if (sign != 1 && sign != -1)
        return fail(ES_ERR_INVALID_ARG, std::string(name) + ": sign must be +1 or -1");
    if (!std::isfinite(sigma) || sigma < 0.0f)
        return fail(ES_ERR_INVALID_ARG, std::string(name) + ": sigma must be finite and >= 0");
    if (sigma == 0.0f) return ES_OK;
    const int rc = check_device(p);
    if (rc != ES_OK) return rc;
    const double coef = sign > 0 ? double(sigma) : -double(sigma);
    return launch_streams(p, 1, &seed, &coef, static_cast<hipStream_t>(stream));
}

int check_qdevice(const es_qplan_t* p) {
    int dev = -1;
    const hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
    if (dev != p->device)
        return fail(ES_ERR_DEVICE, "current device " + std::to_string(dev) +
                                       " differs from the plan's device " +
                                       std::to_string(p->device));
    return ES_OK;
}

// Steps per workgroup of a quantized pass: up to eight (it looks its tensor up
// once), as many as leave three workgroups per slot of the chip.  int8 swap
// over the 0.5B-shaped set 557 us with one, 524, 510 and 506 with two, four and
// eight; fp8 update of 8 over an eighth of it 198, 195 and 204 us with one, two
// and four.
uint32_t qsteps_per_workgroup(uint64_t numel, uint64_t tile_elems, int cus) {
    const uint64_t slots = uint64_t(cus) * 8;
    uint32_t steps = 1;
    while (steps < 8 && 2 * steps * kQStepCodes <= tile_elems &&
           numel / (2 * steps * kQStepCodes) >= 3 * slots)
        steps *= 2;
    return steps;
}

// The tail steps' numbers, of part_codes codes, in the n entries of a table (and
// its sentinel).
void index_qtails(esq::DevQTensor* tab, uint32_t n, uint64_t tile_elems, uint64_t part_codes) {
    uint64_t steps = 0;
    for (uint32_t i = 0; i <= n; ++i) {
        tab[i].first_step = static_cast<uint32_t>(steps);
        if (i == n) break;
        const uint64_t tail = tab[i].numel - (tab[i + 1].first_full - tab[i].first_full) * tile_elems;
        steps += (tail + part_codes - 1) / part_codes;
    }
}

int launch_qpass(es_qplan_t* p, QKind kind, const QPass& ps, hipStream_t s) {
    const uint32_t tile_elems = static_cast<uint32_t>(p->threads) * p->groups * esq::kQGroup;
    QShape sh{tile_elems, p->n_tensors, 0u, p->steps, 0u, 0u};
    while ((p->steps * kQStepCodes << sh.full_shift) < tile_elems) ++sh.full_shift;
    const QPassKernel kernel = qpass_kernel(kind, p->format);
    return for_step_launches(
        p->n_full, p->n_tail_steps, sh.full_shift,
        [&](uint64_t first, uint64_t full, uint32_t step0, uint32_t grid) {
            sh.first_full = first;
            sh.first_step = step0;
            hipLaunchKernelGGL(kernel, dim3(grid), dim3(kStepThreads), 0, s, p->d_tab, full,
                               reinterpret_cast<const Member*>(p->d_scratch + kOffMembers),
                               reinterpret_cast<const UpdateHeader*>(p->d_scratch + kOffHeader),
                               ps, sh);
            const hipError_t e = hipGetLastError();
            return e != hipSuccess ? hip_fail(e, "es_qpass_kernel launch") : ES_OK;
        });
}

// The kernel argument of one perturbation member of a quantized pass: its
// key and sign * sigma * sqrt(2 ln 2) (a restore negates in the kernel), kept
// finite so that its product with the zero that stands for an invalid scale's
// reciprocal is zero and not a NaN.
Member qmember(uint64_t seed, int32_t sign, float sigma) {
    const double w = std::min(double(sigma) * kSqrt2Ln2Double,
                              double(std::numeric_limits<float>::max()));
    return Member{static_cast<uint32_t>(seed), static_cast<uint32_t>(seed >> 32),
                  static_cast<float>(sign > 0 ? w : -w), 0u};
}

int qperturb_impl(es_qplan_t* p, uint64_t seed, int32_t sign, float sigma, es_stream_t stream,
                  QKind kind, const char* name) {
    if (p == nullptr) return fail(ES_ERR_INVALID_ARG, std::string(name) + ": null plan");
    if (sign != 1 && sign != -1)
        return fail(ES_ERR_INVALID_ARG, std::string(name) + ": sign must be +1 or -1");
    if (!std::isfinite(sigma) || sigma < 0.0f)
        return fail(ES_ERR_INVALID_ARG, std::string(name) + ": sigma must be finite and >= 0");
    if (sigma == 0.0f) return ES_OK;
    const int rc = check_qdevice(p);
    if (rc != ES_OK) return rc;
    QPass ps = {};
    ps.m = qmember(seed, sign, sigma);
    return launch_qpass(p, kind, ps, static_cast<hipStream_t>(stream));
}

// The `bytes` bytes at p must be memory that kernels on `device` can access:
// device or managed memory of that device, the whole range inside one
// allocation (checked when the runtime knows the allocation's extent), or
// mapped pinned host memory.  Catches host pointers, other devices' memory
// and overstated sizes before a kernel would fault on them.  A failed query
// leaves no error behind for later launch checks.
// (The name of the checked array is `name` followed by `part`; it is
// formatted only on failure.)
int check_access(const void* p, uint64_t bytes, int device, const char* name, const char* part) {
    if (bytes == 0) return ES_OK;
    auto what = [&]() { return std::string(name) + part; };
    hipPointerAttribute_t a{};
    hipError_t e = hipPointerGetAttributes(&a, p);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        return fail(ES_ERR_INVALID_ARG, what() + ": not memory the device can access");
    }
    if (a.type == hipMemoryTypeHost) {
        if (a.devicePointer == nullptr)
            return fail(ES_ERR_INVALID_ARG, what() + ": host memory not mapped for the device");
        return ES_OK;
    }
    if (a.type != hipMemoryTypeDevice && a.type != hipMemoryTypeManaged &&
        a.type != hipMemoryTypeUnified)
        return fail(ES_ERR_INVALID_ARG, what() + ": not device memory");
    if (a.type == hipMemoryTypeDevice && a.device != device)
        return fail(ES_ERR_INVALID_ARG, what() + ": memory of device " + std::to_string(a.device) +
                                            ", not of device " + std::to_string(device));
    hipDeviceptr_t base = nullptr;
    size_t size = 0;
    e = hipMemGetAddressRange(&base, &size, const_cast<void*>(p));
    if (e != hipSuccess) {                   // allocator that does not report extents
        (void)hipGetLastError();
        return ES_OK;
    }
    const uintptr_t b = reinterpret_cast<uintptr_t>(base), q = reinterpret_cast<uintptr_t>(p);
    if (q < b || q - b > size || bytes > size - (q - b))
        return fail(ES_ERR_INVALID_ARG, what() + ": " + std::to_string(bytes) +
                                            " bytes extend past the end of its allocation");
    return ES_OK;
}
int check_access(const void* p, uint64_t bytes, int device, const std::string& what) {
    return check_access(p, bytes, device, what.c_str(), "");
}

// Free a plan's tile table and scratch on the plan's device: that device is made
// current for the call (the caller's is restored) and synchronised first, so
// no queued launch still reads them.  Every step runs; the first error is
// returned.
int release_device_memory(int device, void* tab, void* scratch, const char* name) {
    const std::string nm(name);
    int rc = ES_OK;
    int caller = -1;
    hipError_t e = hipGetDevice(&caller);
    if (e != hipSuccess) rc = hip_fail(e, nm + ": hipGetDevice");
    const bool switched = e == hipSuccess && caller != device;
    if (switched) {
        e = hipSetDevice(device);
        if (e != hipSuccess && rc == ES_OK) rc = hip_fail(e, nm + ": hipSetDevice");
    }
    e = hipDeviceSynchronize();
    if (e != hipSuccess && rc == ES_OK) rc = hip_fail(e, nm + ": hipDeviceSynchronize");
    e = hipFree(tab);
    if (e != hipSuccess && rc == ES_OK) rc = hip_fail(e, nm + ": hipFree");
    e = hipFree(scratch);
    if (e != hipSuccess && rc == ES_OK) rc = hip_fail(e, nm + ": hipFree");
    if (switched) {
        e = hipSetDevice(caller);
        if (e != hipSuccess && rc == ES_OK) rc = hip_fail(e, nm + ": hipSetDevice");
    }
    return rc;
}

// Division by a row length r >= 2 as a multiply-high and a shift:
// j / r = mulhi(j, magic) >> shift for every j < 2^31 (Granlund and
// Montgomery, 1994: magic = ceil(2^(31 + l) / r) with 2^(l-1) < r <= 2^l,
// which lies in [2^31, 2^32)).
void row_divisor(uint32_t r, uint32_t& magic, uint32_t& shift) {
    uint32_t l = 0;
    while ((uint64_t(1) << l) < r) ++l;
    magic = static_cast<uint32_t>(((uint64_t(1) << (31 + l)) + r - 1) / r);
    shift = l - 1;
}

// Launch shape of the bf16 tile kernels: the defaults, or overrides for
// launch-shape sweeps.
void launch_shape(int& threads, int& groups) {
    threads = env_int("ESOPT_THREADS", kDefaultThreads, 256, 1024);
    groups = env_int("ESOPT_GROUPS", kDefaultGroups, 2, 8);
    if (checksum_kernel(threads, groups, false, false) == nullptr) {
        threads = kDefaultThreads;
        groups = kDefaultGroups;
    }
}

// The tiles of one bf16 tensor (see DevTile), appended to `full` and `tail`.
// Full tiles start where the address is a multiple of the tile's byte size
// (the tensor's base is 16-byte aligned, so such an element index is a
// multiple of 8 and groups keep their Philox quads); the elements before the
// first one and after the last one are tail tiles.  A shard (`offset`
// elements into its whole tensor, a multiple of 8) is tiled by address the
// same way, but its descriptors count elements of the whole tensor: elem0
// and limit are offset, and the base is moved back by as many elements, so
// base + element is still the address and the element is the noise index.
// Every tile keeps its counter's high word uniform: a tile that would cross
// a multiple of 2^34 elements of the whole tensor is split there into tail
// tiles.
void tile_tensor(uint16_t* data, uint64_t numel, uint64_t offset, uint32_t tensor_id,
                 uint64_t tile_elems, std::vector<DevTile>& full, std::vector<DevTile>& tail) {
    if (numel == 0) return;
    constexpr uint64_t kHiBlock = uint64_t(1) << 34;      // elements per counter high word
    // base - offset, as an address: the kernels only ever add an element
    // index of at least `offset` to it
    uint16_t* const base =
        reinterpret_cast<uint16_t*>(reinterpret_cast<uintptr_t>(data) - 2 * offset);
    auto add_tail = [&](uint64_t e0, uint64_t e1, uint32_t aligned) {   // local indices
        e0 += offset;
        e1 += offset;
        while (e0 < e1) {                                   // split at high-word boundaries
            const uint64_t cut = std::min(e1, (e0 / kHiBlock + 1) * kHiBlock);
            tail.push_back(DevTile{base, e0, cut, tensor_id, aligned});
            e0 = cut;
        }
    };
    const uintptr_t a = reinterpret_cast<uintptr_t>(data);
    if (a % 16 != 0) {                                      // tail tiles throughout
        for (uint64_t e0 = 0; e0 < numel; e0 += tile_elems)
            add_tail(e0, std::min(numel, e0 + tile_elems), 0u);
        return;
    }
    const uint64_t tile_bytes = 2 * tile_elems;
    const uint64_t head = std::min<uint64_t>(numel, ((tile_bytes - a % tile_bytes) % tile_bytes) / 2);
    add_tail(0, head, 1u);
    uint64_t e0 = head;
    for (; e0 + tile_elems <= numel; e0 += tile_elems) {
        const uint64_t g0 = offset + e0;
        if (g0 / kHiBlock != (g0 + tile_elems - 1) / kHiBlock)
            add_tail(e0, e0 + tile_elems, 1u);
        else
            full.push_back(DevTile{base, g0, g0 + tile_elems, tensor_id, 1u});
    }
    add_tail(e0, numel, 1u);
}

int current_device(int* dev) {
    const hipError_t e = hipGetDevice(dev);
    if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
    return ES_OK;
}

// The device arrays of an update call: rewards and z (n floats), status.
int check_update_arrays(const char* name, int device, const float* rewards_dev, uint32_t n,
                        const float* z_out_dev, const int32_t* status_out_dev) {
    int rc = check_access(rewards_dev, uint64_t(4) * n, device, name, ": rewards");
    if (rc == ES_OK && z_out_dev != nullptr)
        rc = check_access(z_out_dev, uint64_t(4) * n, device, name, ": z output");
    if (rc == ES_OK && status_out_dev != nullptr)
        rc = check_access(status_out_dev, 4, device, name, ": status output");
    return rc;
}

// Argument checks shared by the update entry points.
int validate_update(const char* name, const uint64_t* seeds, const int32_t* signs,
                    const float* rewards_dev, uint32_t n_members, const es_update_opts_t* opts) {
    if (seeds == nullptr || signs == nullptr || rewards_dev == nullptr || opts == nullptr)
        return fail_in(ES_ERR_INVALID_ARG, name, "null pointer");
    if (n_members == 0 || n_members > ES_MAX_MEMBERS)
        return fail_in(ES_ERR_INVALID_ARG, name, "n_members out of range (1 .. 1024)");
    if ((opts->flags & ~(ES_UPDATE_DIV_SIGMA | ES_REWARDS_ARE_WEIGHTS |
                         ES_UPDATE_STOCHASTIC_ROUND | ES_UPDATE_MASTER)) != 0)
        return fail_in(ES_ERR_INVALID_ARG, name, "unknown flags");
    if ((opts->flags & ES_UPDATE_MASTER) && (opts->flags & ES_UPDATE_STOCHASTIC_ROUND))
        return fail_in(ES_ERR_INVALID_ARG, name,
                       "ES_UPDATE_MASTER rounds the bf16 copy to nearest-even: no "
                       "ES_UPDATE_STOCHASTIC_ROUND with it");
    if (!std::isfinite(opts->alpha)) return fail_in(ES_ERR_INVALID_ARG, name, "alpha not finite");
    if ((opts->flags & ES_UPDATE_DIV_SIGMA) && !(std::isfinite(opts->sigma) && opts->sigma > 0.0f))
        return fail_in(ES_ERR_INVALID_ARG, name,
                       "sigma must be finite and > 0 with ES_UPDATE_DIV_SIGMA");
    if (!std::isfinite(opts->zscore_eps) || opts->zscore_eps < 0.0f)
        return fail_in(ES_ERR_INVALID_ARG, name, "zscore_eps must be finite and >= 0");
    for (uint32_t i = 0; i < n_members; ++i)
        if (signs[i] != 1 && signs[i] != -1)
            return fail_in(ES_ERR_INVALID_ARG, name, "signs must be +1 or -1");
    return ES_OK;
}

// The population as tables (host side, fixed arrays, no allocation):
// distinct seeds in order of first appearance, each with its members grouped
// in member order (CSR).  Members are sorted by (seed, index) in place, each
// run of one seed is a distinct seed whose first appearance is its smallest
// index, and the runs are ordered by that index.
struct MemberTables {
    MemberIn min[ES_MAX_MEMBERS];
    DistinctIn din[ES_MAX_MEMBERS];
    uint32_t n_distinct;
};

void build_member_tables(const uint64_t* seeds, const int32_t* signs, uint32_t n,
                         MemberTables& t) {
    struct SeedIndex {
        uint64_t seed;
        uint32_t index;
    };
    struct Run {
        uint32_t first, start, count;       // smallest member index, position in `order`, size
    };
    SeedIndex order[ES_MAX_MEMBERS];
    Run runs[ES_MAX_MEMBERS];
    for (uint32_t i = 0; i < n; ++i) order[i] = SeedIndex{seeds[i], i};
    std::sort(order, order + n, [](const SeedIndex& a, const SeedIndex& b) {
        return a.seed != b.seed ? a.seed < b.seed : a.index < b.index;
    });
    uint32_t nd = 0;
    for (uint32_t i = 0; i < n;) {
        uint32_t j = i + 1;
        while (j < n && order[j].seed == order[i].seed) ++j;
        runs[nd++] = Run{order[i].index, i, j - i};
        i = j;
    }
    std::sort(runs, runs + nd, [](const Run& a, const Run& b) { return a.first < b.first; });
    uint32_t pos = 0;
    for (uint32_t d = 0; d < nd; ++d) {
        const uint64_t sd = order[runs[d].start].seed;
        t.din[d] = DistinctIn{static_cast<uint32_t>(sd), static_cast<uint32_t>(sd >> 32), pos,
                              runs[d].count};
        for (uint32_t k = 0; k < runs[d].count; ++k) {
            const uint32_t m = order[runs[d].start + k].index;
            t.min[pos++] = MemberIn{m, signs[m]};
        }
    }
    t.n_distinct = nd;
}

// Host words into device scratch at dst_off, in launches of es_stage_kernel
// carrying 1 KB of kernel arguments each (no staging buffer, no host
// synchronisation).
int stage_words(uint8_t* d_scratch, size_t dst_off, const void* src, size_t bytes,
                hipStream_t s) {
    const uint32_t* words = static_cast<const uint32_t*>(src);
    const size_t n_words = bytes / 4;
    for (size_t w0 = 0; w0 < n_words; w0 += kStageWords) {
        StageChunk chunk;
        const uint32_t nw = static_cast<uint32_t>(std::min<size_t>(kStageWords, n_words - w0));
        std::memcpy(chunk.words, words + w0, nw * 4);
        hipLaunchKernelGGL(es_stage_kernel, dim3(1), dim3(kAuxBlock), 0, s,
                           reinterpret_cast<uint32_t*>(d_scratch + dst_off) + w0, nw, chunk);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return hip_fail(e, "es_stage_kernel launch");
    }
    return ES_OK;
}

// Hand the population to the device: the member tables go through kernel
// arguments (staged into the scratch first when they are too many), and one wave
// z-scores the rewards and merges the weights per distinct seed, leaving the
// weighted member table and its header in the scratch.  Allocates nothing.  With
// `find`, *found is set to the distinct-table entry of seed *find before anything
// is launched (or the call fails with INVALID_ARG when no member has that seed).
int prepare_update(uint8_t* d_scratch, const uint64_t* seeds, const int32_t* signs,
                   const float* rewards_dev, uint32_t n_members, const es_update_opts_t* opts,
                   float* z_out_dev, int32_t* status_out_dev, hipStream_t s,
                   const uint64_t* find = nullptr, uint32_t* found = nullptr) {
    MemberTables t;
    build_member_tables(seeds, signs, n_members, t);
    const uint32_t nd = t.n_distinct;
    if (find != nullptr) {
        uint32_t d = 0;
        while (d < nd && (uint64_t(t.din[d].k0) | (uint64_t(t.din[d].k1) << 32)) != *find) ++d;
        if (d == nd)
            return fail(ES_ERR_INVALID_ARG,
                        "es_restore_update: the restored member's seed is not among the seeds");
        *found = d;
    }

    double c = static_cast<double>(opts->alpha) / static_cast<double>(n_members);
    if (opts->flags & ES_UPDATE_DIV_SIGMA) c /= static_cast<double>(opts->sigma);
    const double eps = static_cast<double>(opts->zscore_eps);
    Member* const members = reinterpret_cast<Member*>(d_scratch + kOffMembers);
    UpdateHeader* const header = reinterpret_cast<UpdateHeader*>(d_scratch + kOffHeader);
    if (n_members <= kInlineMembers) {
        InlineTables it;
        for (uint32_t d = 0; d < nd; ++d) {
            it.k0[d] = t.din[d].k0;
            it.k1[d] = t.din[d].k1;
            it.first[d] = static_cast<uint16_t>(t.din[d].first);
            it.count[d] = static_cast<uint16_t>(t.din[d].count);
        }
        for (uint32_t m = 0; m < n_members; ++m) {
            const int32_t i = static_cast<int32_t>(t.min[m].reward_index);
            it.member_index[m] = static_cast<int16_t>(t.min[m].sign < 0 ? ~i : i);
        }
        hipLaunchKernelGGL(es_prepare_kernel<InlineTables>, dim3(1), dim3(64), 0, s, rewards_dev,
                           n_members, eps, opts->flags, c, it, nd, members, header, z_out_dev,
                           status_out_dev);
    } else {
        int rc = stage_words(d_scratch, kOffMembersIn, t.min, sizeof(MemberIn) * n_members, s);
        if (rc == ES_OK)
            rc = stage_words(d_scratch, kOffDistinctIn, t.din, sizeof(DistinctIn) * nd, s);
        if (rc != ES_OK) return rc;
        const StagedTables st{reinterpret_cast<const MemberIn*>(d_scratch + kOffMembersIn),
                              reinterpret_cast<const DistinctIn*>(d_scratch + kOffDistinctIn)};
        hipLaunchKernelGGL(es_prepare_kernel<StagedTables>, dim3(1), dim3(64), 0, s, rewards_dev,
                           n_members, eps, opts->flags, c, st, nd, members, header, z_out_dev,
                           status_out_dev);
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "es_prepare_kernel launch");
    return ES_OK;
}

// The member es_restore_update reverts: its seed and the perturbation
// coefficient es_restore would apply (-sign sigma).
struct RestoreMember {
    uint64_t seed;
    double coef;
};

// The fused update of a bf16 plan with its member tables in `d_scratch`
// (the plan's, or the static array of es_update_noalloc); with `restore`,
// that member reverted in the same pass.
int update_impl(const char* name, es_plan_t* plan, uint8_t* d_scratch, const uint64_t* seeds,
                const int32_t* signs, const float* rewards_dev, uint32_t n_members,
                const es_update_opts_t* opts, float* z_out_dev, int32_t* status_out_dev,
                hipStream_t s, const RestoreMember* restore = nullptr) {
    if (opts->flags & ES_UPDATE_MASTER) {
        if (restore != nullptr)
            return fail_in(ES_ERR_INVALID_ARG, name,
                           "ES_UPDATE_MASTER rewrites the bf16 values from the masters, so no "
                           "member needs reverting first: use es_update");
        if (plan->d_master == nullptr)
            return fail_in(ES_ERR_INVALID_ARG, name,
                           "ES_UPDATE_MASTER on a plan without masters (es_plan_set_master)");
    }
    RestoreArg rst{0u, 0.0f};
    int rc = prepare_update(d_scratch, seeds, signs, rewards_dev, n_members, opts, z_out_dev,
                            status_out_dev, s, restore ? &restore->seed : nullptr, &rst.d);
    if (rc != ES_OK) return rc;
    if (restore) rst.coef_k = static_cast<float>(restore->coef * kSqrt2Ln2Double);
    const bool sr = (opts->flags & ES_UPDATE_STOCHASTIC_ROUND) != 0;
    const bool master = (opts->flags & ES_UPDATE_MASTER) != 0;
    const RoundKey rk{static_cast<uint32_t>(opts->round_seed),
                      static_cast<uint32_t>(opts->round_seed >> 32)};
    Segment seg[2];
    const int n_seg = plan_segments(plan, seg);
    for (int k = 0; k < n_seg; ++k) {
        const Segment& g = seg[k];
        const bool strided = g.rows != nullptr;
        const UpdateKernel kernel =
            master ? update_master_kernel(strided)
                   : update_kernel(sr, strided, restore != nullptr);
        // the segment's masters: the delta table runs parallel to the tiles
        const uint64_t* mdelta =
            master ? plan->d_master + (strided ? plan->n_full + plan->n_tail : 0) : nullptr;
        rc = launch_steps(
            plan, g, 2, mdelta, name, ": es_update_kernel", [&](const StepLaunch& l) {
                hipLaunchKernelGGL(kernel, l.grid, dim3(kStepThreads), 0, s, l.tiles, l.n_full,
                                   l.rows, reinterpret_cast<const Member*>(d_scratch + kOffMembers),
                                   reinterpret_cast<const UpdateHeader*>(d_scratch + kOffHeader),
                                   rk, rst, l.mdelta, l.shape);
            });
        if (rc != ES_OK) return rc;
    }
    return ES_OK;
}

// Per-device address of the static scratch, looked up once per device (with
// that device current) and kept; a fixed table, so lookups allocate nothing.
constexpr int kMaxScratchDevices = 64;
std::atomic<uint8_t*> g_static_scratch[kMaxScratchDevices];
std::mutex g_static_scratch_mutex;

int static_scratch(int device, uint8_t** out) {
    if (device < 0 || device >= kMaxScratchDevices)
        return fail_in(ES_ERR_DEVICE, "es_update_noalloc", "device index above 63");
    uint8_t* p = g_static_scratch[device].load(std::memory_order_acquire);
    if (p == nullptr) {
        std::lock_guard<std::mutex> lock(g_static_scratch_mutex);
        p = g_static_scratch[device].load(std::memory_order_relaxed);
        if (p == nullptr) {
            void* addr = nullptr;
            const hipError_t e = hipGetSymbolAddress(&addr, HIP_SYMBOL(scratch));
            if (e != hipSuccess || addr == nullptr)
                return hip_fail(e, "es_update_noalloc: hipGetSymbolAddress of the static scratch");
            p = static_cast<uint8_t*>(addr);
            g_static_scratch[device].store(p, std::memory_order_release);
        }
    }
    *out = p;
    return ES_OK;
}

// The tiles of a plan under construction: those of tensors and contiguous
// blocks, and those of strided blocks with one row map each.
struct PlanTiles {
    std::vector<DevTile> full, tail;
    std::vector<DevTile> rfull, rtail;
    std::vector<DevRows> rows_full, rows_tail;
};

// Strided blocks are cut into pieces of at most this many elements, so that
// a piece's local element indices stay below 2^31 (the row division's
// range).  A block whose rows are longer than half of that, or whose rows lie
// 2^32 or more elements apart, is laid out row by row instead, each row a
// contiguous shard of its own.
constexpr uint64_t kPieceElems = uint64_t(1) << 31;

// Appends a tile of a strided piece with its row map, cut into tail tiles
// where the whole-tensor index reaches a multiple of 2^34 (so that the
// counter's high word is the tile's).  Such a multiple lies at the start of
// a group: indices within a row are consecutive from a multiple of 8 and
// rows start at multiples of 8.  The index is increasing in e, so each cut
// is found by bisection over the tile's groups.
void split_at_high_words(const DevTile& d, DevRows m, bool full, PlanTiles& t) {
    constexpr uint64_t kHiBlock = uint64_t(1) << 34;
    auto index = [&](uint64_t e) { return rows_index(m.n0, m.skip, m.magic, m.shift, e); };
    uint64_t e0 = d.elem0;
    const uint64_t hi_last = index(d.limit - 1) / kHiBlock;
    if (index(e0) / kHiBlock == hi_last) {
        m.hi = static_cast<uint32_t>(hi_last);
        (full ? t.rfull : t.rtail).push_back(d);
        (full ? t.rows_full : t.rows_tail).push_back(m);
        return;
    }
    while (e0 < d.limit) {
        const uint64_t hi = index(e0) / kHiBlock;
        uint64_t lo_g = (e0 - d.elem0) / 8, hi_g = (d.limit - d.elem0 + 7) / 8;  // groups
        while (lo_g + 1 < hi_g) {          // last group of [e0, ...) still on `hi`
            const uint64_t mid = (lo_g + hi_g) / 2;
            if (index(d.elem0 + 8 * mid) / kHiBlock == hi) lo_g = mid;
            else hi_g = mid;
        }
        const uint64_t cut = std::min(d.limit, d.elem0 + 8 * hi_g);
        DevTile part = d;
        part.elem0 = e0;
        part.limit = cut;
        m.hi = static_cast<uint32_t>(hi);
        t.rtail.push_back(part);
        t.rows_tail.push_back(m);
        e0 = cut;
    }
}

// Tiles of one block (already validated).  A block that is one contiguous
// range of its tensor is tiled as a shard at its first index.  A strided
// block is cut into pieces of whole rows, each tiled by address with local
// element indices, and every tile of a piece gets the piece's row map.
void tile_block(const es_block_t& b, uint64_t tile_elems, PlanTiles& t) {
    const uint64_t numel = b.rows * b.cols;
    if (numel == 0) return;
    uint16_t* const data = static_cast<uint16_t*>(b.data);
    const uint64_t n0 = b.row0 * b.row_len + b.col0;
    if (b.rows == 1 || b.cols == b.row_len) {
        tile_tensor(data, numel, n0, b.tensor_id, tile_elems, t.full, t.tail);
        return;
    }
    if (b.cols > kPieceElems / 2 || b.row_len - b.cols > 0xFFFFFFFFull) {
        for (uint64_t i = 0; i < b.rows; ++i)
            tile_tensor(data + i * b.cols, b.cols, n0 + i * b.row_len, b.tensor_id, tile_elems,
                        t.full, t.tail);
        return;
    }
    DevRows m{};
    m.skip = static_cast<uint32_t>(b.row_len - b.cols);
    row_divisor(static_cast<uint32_t>(b.cols), m.magic, m.shift);
    const uint64_t piece_rows = kPieceElems / b.cols;
    std::vector<DevTile> full, tail;
    for (uint64_t r = 0; r < b.rows; r += piece_rows) {
        const uint64_t nr = std::min(piece_rows, b.rows - r);
        m.n0 = n0 + r * b.row_len;
        full.clear();
        tail.clear();
        tile_tensor(data + r * b.cols, nr * b.cols, 0, b.tensor_id, tile_elems, full, tail);
        for (int k = 0; k < 2; ++k)
            for (const DevTile& d : k == 0 ? full : tail) split_at_high_words(d, m, k == 0, t);
    }
}

// A plan over tiles laid out by the caller (es_plan_create,
// es_plan_create_blocks): launch grids, one device allocation for the
// descriptors and row maps, the scratch.
int finish_plan(const char* name, int device, uint32_t n_tensors, uint64_t numel, int threads,
                int groups, PlanTiles& t, es_plan_t** out) {
    const std::string nm(name);
    const uint64_t n_full = t.full.size(), n_tail = t.tail.size();
    const uint64_t n_rfull = t.rfull.size(), n_rtail = t.rtail.size();
    std::vector<TileDesc> tiles;
    tiles.reserve(n_full + n_tail + n_rfull + n_rtail);
    for (const std::vector<DevTile>* v : {&t.full, &t.tail, &t.rfull, &t.rtail})
        for (const DevTile& d : *v) tiles.push_back(tile_desc(d));
    const TailIndex tails = index_tails(tiles.data() + n_full, n_tail);
    const TailIndex rtails = index_tails(tiles.data() + n_full + n_tail + n_rfull, n_rtail);
    std::vector<DevRows> rows;
    rows.reserve(n_rfull + n_rtail);
    rows.insert(rows.end(), t.rows_full.begin(), t.rows_full.end());
    rows.insert(rows.end(), t.rows_tail.begin(), t.rows_tail.end());
    es_plan_t* p = new (std::nothrow) es_plan_t;
    if (p == nullptr) return fail(ES_ERR_NOMEM, nm + ": host allocation");
    p->device = device;
    int cus = 0;
    hipError_t e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, p->device);
    if (e != hipSuccess) { delete p; return hip_fail(e, "hipDeviceGetAttribute"); }
    const int wg_update = env_int("ESOPT_UPDATE_WG_PER_CU", kDefaultUpdateWgPerCu, 1, 32);
    p->threads = threads;
    p->groups = groups;
    p->tile_elems = uint64_t(threads) * groups * kGroupElems;
    p->n_tensors = n_tensors;
    p->numel = numel;
    p->n_full = n_full;
    p->n_tail = n_tail;
    p->n_rfull = n_rfull;
    p->n_rtail = n_rtail;
    auto grid = [&](uint64_t a, uint64_t b, int per_cu) {   // checksum: a grid that strides
        const uint64_t cap = std::max<uint64_t>(std::max(a, b), 1);
        return static_cast<uint32_t>(std::min<uint64_t>(cap, uint64_t(cus) * per_cu));
    };
    p->grid_sum = grid(n_full, n_tail, wg_update);
    p->grid_sum_rows = grid(n_rfull, n_rtail, wg_update);
    p->cus = cus;
    p->tails = tails;
    p->rtails = rtails;
    const size_t tile_bytes = sizeof(TileDesc) * std::max<size_t>(tiles.size(), 1);
    const size_t rows_bytes = sizeof(DevRows) * rows.size();
    e = hipMalloc(reinterpret_cast<void**>(&p->d_tiles), tile_bytes + rows_bytes);
    if (e != hipSuccess) { delete p; return fail(ES_ERR_NOMEM, std::string("hipMalloc: ") + hipGetErrorString(e)); }
    p->d_rows = rows.empty() ? nullptr
                             : reinterpret_cast<DevRows*>(reinterpret_cast<uint8_t*>(p->d_tiles) +
                                                          tile_bytes);
    e = hipMalloc(reinterpret_cast<void**>(&p->d_scratch), kScratchBytes);
    if (e != hipSuccess) {
        (void)hipFree(p->d_tiles);
        delete p;
        return fail(ES_ERR_NOMEM, std::string("hipMalloc: ") + hipGetErrorString(e));
    }
    if (!tiles.empty())
        e = hipMemcpy(p->d_tiles, tiles.data(), sizeof(TileDesc) * tiles.size(), hipMemcpyHostToDevice);
    if (e == hipSuccess && !rows.empty())
        e = hipMemcpy(p->d_rows, rows.data(), rows_bytes, hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipMemset(p->d_scratch, 0, kScratchBytes);
    if (e != hipSuccess) {
        (void)hipFree(p->d_tiles);
        (void)hipFree(p->d_scratch);
        delete p;
        return hip_fail(e, nm + ": tile table upload");
    }
    *out = p;
    return ES_OK;
}

// Checks of one block's geometry (es_block_t's requirements), in 128-bit
// arithmetic so that no product or sum wraps; an empty string when it holds.
std::string block_geometry_error(const es_block_t& b) {
    typedef unsigned __int128 u128;
    const u128 two60 = u128(1) << 60;
    const u128 numel = u128(b.rows) * b.cols;
    if (numel > two60) return "rows * cols above 2^60";
    if (numel == 0) return "";
    if (u128(b.col0) + b.cols > b.row_len) return "col0 + cols above row_len";
    const u128 first = u128(b.row0) * b.row_len + b.col0;
    const u128 end = u128(b.row0 + u128(b.rows - 1)) * b.row_len + b.col0 + b.cols;
    if (end > two60) return "an element index at or above 2^60";
    if (first % 8 != 0) return "first index row0 * row_len + col0 not a multiple of 8";
    if (b.rows > 1 && b.cols < b.row_len && (b.cols % 8 != 0 || b.row_len % 8 != 0))
        return "strided block: cols and row_len must be multiples of 8";
    return "";
}


// One entry of a quantized plan, from an es_qtensor_t (with a shard start)
// or an es_qblock_t: `numel` codes at `data` with their scales, the
// whole-tensor index n0 of code 0 and, for a strided block, rows of `cols`
// codes that lie cols + skip apart in the whole tensor (skip 0 otherwise).
struct QSpec {
    void* data;
    const float* scales;
    uint64_t numel;
    uint32_t row, tensor_id;
    uint64_t n0, cols, skip;
};

// The geometry of a quantized block as a QSpec, or what is wrong with it.
std::string qblock_geometry(const es_qblock_t& b, QSpec& spec) {
    typedef unsigned __int128 u128;
    const u128 two31 = u128(1) << 31;
    const u128 numel = u128(b.rows) * b.cols;
    if (numel >= two31) return "rows * cols must be below 2^31";
    spec = QSpec{b.data, b.scales, uint64_t(numel), b.row, b.tensor_id, 0, b.cols, 0};
    if (numel == 0) return "";
    if (u128(b.col0) + b.cols > b.row_len) return "col0 + cols above row_len";
    const u128 first = u128(b.row0) * b.row_len + b.col0;
    const u128 end = (u128(b.row0) + b.rows - 1) * b.row_len + b.col0 + b.cols;
    if (end >= two31) return "(row0 + rows - 1) * row_len + col0 + cols must be below 2^31";
    if (first % 16 != 0) return "first index row0 * row_len + col0 not a multiple of 16";
    const bool strided = b.rows > 1 && b.cols < b.row_len;
    if (strided && (b.cols % 16 != 0 || b.row_len % 16 != 0))
        return "strided block: cols and row_len must be multiples of 16";
    spec.n0 = uint64_t(first);
    spec.skip = strided ? b.row_len - b.cols : 0;
    return "";
}

// A quantized plan over checked entries (whole-tensor indices below 2^31):
// the per-entry rules shared by tensors and blocks, the table, the device
// checks and the allocations.  `name` and `kind` label the errors.
int qplan_build(const std::vector<QSpec>& specs, uint32_t format, es_qplan_t** out,
                const char* name, const char* kind) {
    const std::string nm(name);
    if (format != ES_QFORMAT_INT8 && format != ES_QFORMAT_E4M3)
        return fail(ES_ERR_INVALID_ARG, nm + ": format not ES_QFORMAT_INT8 or ES_QFORMAT_E4M3");
    int threads = env_int("ESOPT_THREADS", kDefaultThreads, 256, 1024);
    int groups = env_int("ESOPT_QGROUPS", kDefaultQGroups, 2, 8);
    if (qchecksum_kernel(threads, groups, false) == nullptr) {
        threads = kDefaultThreads;
        groups = kDefaultQGroups;
    }
    const uint64_t tile_elems = uint64_t(threads) * groups * esq::kQGroup;
    const uint32_t n_tensors = static_cast<uint32_t>(specs.size());
    std::vector<esq::DevQTensor> tab(n_tensors + 1);
    std::unordered_map<uint32_t, uint32_t> ids;
    std::vector<std::pair<uintptr_t, uintptr_t>> ranges;
    uint64_t n_full = 0, n_tail = 0, numel = 0;
    for (uint32_t i = 0; i < n_tensors; ++i) {
        const QSpec& t = specs[i];
        const std::string where = nm + ": " + kind + " " + std::to_string(i);
        if (!ids.emplace(t.tensor_id, i).second)
            return fail(ES_ERR_INVALID_ARG, where + ": duplicate tensor_id " + std::to_string(t.tensor_id));
        if (t.numel > 0 && (t.data == nullptr || t.scales == nullptr))
            return fail(ES_ERR_INVALID_ARG, where + ": null data or scales");
        if (t.row % 8 != 0)
            return fail(ES_ERR_INVALID_ARG, where + ": row must be a multiple of 8 (or 0)");
        if (t.numel > 0 && (reinterpret_cast<uintptr_t>(t.scales) & 3u))
            return fail(ES_ERR_ALIGN, where + ": scales not 4-byte aligned");
        const uintptr_t a = reinterpret_cast<uintptr_t>(t.data);
        const uint64_t full = (a % 16 == 0) ? t.numel / tile_elems : 0;
        const uint64_t tail = (t.numel - full * tile_elems + tile_elems - 1) / tile_elems;
        uint32_t magic = 0, shift = 0, cmagic = 0, cshift = 0;
        if (t.row != 0) row_divisor(t.row, magic, shift);
        if (t.skip != 0) row_divisor(static_cast<uint32_t>(t.cols), cmagic, cshift);
        tab[i] = esq::DevQTensor{static_cast<int8_t*>(t.data), t.scales,
                                 static_cast<uint32_t>(t.numel), static_cast<uint32_t>(t.n0),
                                 n_full, n_tail, t.row, t.tensor_id, magic, shift, 0u,
                                 static_cast<uint32_t>(t.skip), cmagic, cshift, {0u, 0u}};
        if (t.numel > 0) ranges.emplace_back(a, a + t.numel);
        n_full += full;
        n_tail += tail;
        numel += t.numel;
    }
    std::sort(ranges.begin(), ranges.end());
    for (size_t i = 1; i < ranges.size(); ++i)
        if (ranges[i].first < ranges[i - 1].second)
            return fail(ES_ERR_INVALID_ARG, nm + ": " + kind + "s overlap in memory");
    tab[n_tensors] = esq::DevQTensor{nullptr, nullptr, 0u, 0u, n_full, n_tail, 0u, 0xFFFFFFFFu,
                                     0u, 0u, 0u, 0u, 0u, 0u, {0u, 0u}};

    int device = -1;
    int rc = current_device(&device);
    if (rc != ES_OK) return rc;
    for (uint32_t i = 0; i < n_tensors && rc == ES_OK; ++i) {
        const QSpec& t = specs[i];
        const std::string where = nm + ": " + kind + " " + std::to_string(i);
        const uint64_t n_scales = t.row == 0 ? 1 : (t.numel + t.row - 1) / t.row;
        rc = check_access(t.data, t.numel, device, where + " codes");
        if (rc == ES_OK && t.numel > 0)
            rc = check_access(t.scales, 4 * n_scales, device, where + " scales");
    }
    if (rc != ES_OK) return rc;
    int cus = 0;
    hipError_t e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device);
    if (e != hipSuccess) return hip_fail(e, "hipDeviceGetAttribute");
    const uint32_t steps = qsteps_per_workgroup(numel, tile_elems, cus);
    index_qtails(tab.data(), n_tensors, tile_elems, uint64_t(steps) * kQStepCodes);
    es_qplan_t* p = new (std::nothrow) es_qplan_t;
    if (p == nullptr) return fail(ES_ERR_NOMEM, nm + ": host allocation");
    p->device = device;
    const int wg = env_int("ESOPT_UPDATE_WG_PER_CU", kDefaultUpdateWgPerCu, 1, 32);
    p->steps = steps;
    p->n_tail_steps = tab[n_tensors].first_step;
    p->threads = threads;
    p->groups = groups;
    p->format = static_cast<int>(format);
    p->n_tensors = n_tensors;
    p->numel = numel;
    p->n_full = n_full;
    p->n_tail = n_tail;
    const uint64_t cap = std::max<uint64_t>(std::max(n_full, n_tail), 1);
    p->grid = static_cast<uint32_t>(std::min<uint64_t>(cap, uint64_t(cus) * wg));
    e = hipMalloc(reinterpret_cast<void**>(&p->d_tab), sizeof(esq::DevQTensor) * tab.size());
    if (e != hipSuccess) { delete p; return fail(ES_ERR_NOMEM, std::string("hipMalloc: ") + hipGetErrorString(e)); }
    e = hipMalloc(reinterpret_cast<void**>(&p->d_scratch), kScratchBytes);
    if (e != hipSuccess) {
        (void)hipFree(p->d_tab);
        delete p;
        return fail(ES_ERR_NOMEM, std::string("hipMalloc: ") + hipGetErrorString(e));
    }
    e = hipMemcpy(p->d_tab, tab.data(), sizeof(esq::DevQTensor) * tab.size(), hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipMemset(p->d_scratch, 0, kScratchBytes);
    if (e != hipSuccess) {
        (void)hipFree(p->d_tab);
        (void)hipFree(p->d_scratch);
        delete p;
        return hip_fail(e, nm + ": table upload");
    }
    *out = p;
    return ES_OK;
}

}  // namespace

extern "C" {

int es_plan_create(const es_tensor_t* tensors, uint32_t n_tensors, es_plan_t** out) try {
    if (out == nullptr) return fail(ES_ERR_INVALID_ARG, "es_plan_create: null output pointer");
    *out = nullptr;
    if (tensors == nullptr) return fail(ES_ERR_INVALID_ARG, "es_plan_create: null tensor list");
    if (n_tensors == 0 || n_tensors > ES_MAX_TENSORS)
        return fail(ES_ERR_INVALID_ARG, "es_plan_create: n_tensors out of range");
    int threads = 0, groups = 0;
    launch_shape(threads, groups);
    const uint64_t tile_elems = uint64_t(threads) * groups * kGroupElems;
    std::unordered_map<uint32_t, uint32_t> ids;
    std::vector<std::pair<uintptr_t, uintptr_t>> ranges;
    uint64_t numel = 0;
    for (uint32_t i = 0; i < n_tensors; ++i) {
        const es_tensor_t& t = tensors[i];
        const std::string where = "es_plan_create: tensor " + std::to_string(i);
        if (!ids.emplace(t.tensor_id, i).second)
            return fail(ES_ERR_INVALID_ARG, where + ": duplicate tensor_id " + std::to_string(t.tensor_id));
        if (t.numel > 0 && t.data == nullptr) return fail(ES_ERR_INVALID_ARG, where + ": null data");
        if (t.numel > (uint64_t(1) << 60) - 8 * uint64_t(t.offset8))
            return fail(ES_ERR_INVALID_ARG, where + ": 8 * offset8 + numel above 2^60");
        const uintptr_t a = reinterpret_cast<uintptr_t>(t.data);
        if (t.numel > 0 && (a & 1u)) return fail(ES_ERR_ALIGN, where + ": data not 2-byte aligned");
        if (t.numel > 0) ranges.emplace_back(a, a + 2 * t.numel);
        numel += t.numel;
    }
    std::sort(ranges.begin(), ranges.end());
    for (size_t i = 1; i < ranges.size(); ++i)
        if (ranges[i].first < ranges[i - 1].second)
            return fail(ES_ERR_INVALID_ARG, "es_plan_create: tensors overlap in memory");

    int device = -1;
    int rc = current_device(&device);
    if (rc != ES_OK) return rc;
    for (uint32_t i = 0; i < n_tensors && rc == ES_OK; ++i)
        rc = check_access(tensors[i].data, 2 * tensors[i].numel, device,
                          "es_plan_create: tensor " + std::to_string(i));
    if (rc != ES_OK) return rc;
    // the tile descriptors (built after the accesses are known to be valid:
    // every tensor lies inside one device allocation)
    PlanTiles t;
    for (uint32_t i = 0; i < n_tensors; ++i)
        tile_tensor(static_cast<uint16_t*>(tensors[i].data), tensors[i].numel,
                    8 * uint64_t(tensors[i].offset8), tensors[i].tensor_id, tile_elems, t.full,
                    t.tail);
    rc = finish_plan("es_plan_create", device, n_tensors, numel, threads, groups, t, out);
    if (rc == ES_OK)
        for (uint32_t i = 0; i < n_tensors; ++i)
            (*out)->owners.emplace_back(reinterpret_cast<uintptr_t>(tensors[i].data),
                                        tensors[i].numel);
    return rc;
} catch (const std::bad_alloc&) {
    return fail(ES_ERR_NOMEM, "es_plan_create: host allocation failed");
}

int es_plan_create_blocks(const es_block_t* blocks, uint32_t n_blocks, es_plan_t** out) try {
    if (out == nullptr) return fail(ES_ERR_INVALID_ARG, "es_plan_create_blocks: null output pointer");
    *out = nullptr;
    if (blocks == nullptr) return fail(ES_ERR_INVALID_ARG, "es_plan_create_blocks: null block list");
    if (n_blocks == 0 || n_blocks > ES_MAX_TENSORS)
        return fail(ES_ERR_INVALID_ARG, "es_plan_create_blocks: n_blocks out of range");
    int threads = 0, groups = 0;
    launch_shape(threads, groups);
    const uint64_t tile_elems = uint64_t(threads) * groups * kGroupElems;
    std::unordered_map<uint32_t, uint32_t> ids;
    std::vector<std::pair<uintptr_t, uintptr_t>> ranges;
    uint64_t numel = 0;
    for (uint32_t i = 0; i < n_blocks; ++i) {
        const es_block_t& b = blocks[i];
        const std::string where = "es_plan_create_blocks: block " + std::to_string(i);
        if (b.reserved != 0) return fail(ES_ERR_INVALID_ARG, where + ": reserved field not 0");
        if (!ids.emplace(b.tensor_id, i).second)
            return fail(ES_ERR_INVALID_ARG, where + ": duplicate tensor_id " + std::to_string(b.tensor_id));
        const std::string bad = block_geometry_error(b);
        if (!bad.empty()) return fail(ES_ERR_INVALID_ARG, where + ": " + bad);
        const uint64_t n = b.rows * b.cols;
        if (n > 0 && b.data == nullptr) return fail(ES_ERR_INVALID_ARG, where + ": null data");
        const uintptr_t a = reinterpret_cast<uintptr_t>(b.data);
        if (n > 0 && (a & 1u)) return fail(ES_ERR_ALIGN, where + ": data not 2-byte aligned");
        if (n > 0) ranges.emplace_back(a, a + 2 * n);
        numel += n;
    }
    std::sort(ranges.begin(), ranges.end());
    for (size_t i = 1; i < ranges.size(); ++i)
        if (ranges[i].first < ranges[i - 1].second)
            return fail(ES_ERR_INVALID_ARG, "es_plan_create_blocks: blocks overlap in memory");

    int device = -1;
    int rc = current_device(&device);
    if (rc != ES_OK) return rc;
    for (uint32_t i = 0; i < n_blocks && rc == ES_OK; ++i)
        rc = check_access(blocks[i].data, 2 * blocks[i].rows * blocks[i].cols, device,
                          "es_plan_create_blocks: block " + std::to_string(i));
    if (rc != ES_OK) return rc;
    PlanTiles t;
    for (uint32_t i = 0; i < n_blocks; ++i) tile_block(blocks[i], tile_elems, t);
    rc = finish_plan("es_plan_create_blocks", device, n_blocks, numel, threads, groups, t, out);
    if (rc == ES_OK)
        for (uint32_t i = 0; i < n_blocks; ++i)
            (*out)->owners.emplace_back(reinterpret_cast<uintptr_t>(blocks[i].data),
                                        blocks[i].rows * blocks[i].cols);
    return rc;
} catch (const std::bad_alloc&) {
    return fail(ES_ERR_NOMEM, "es_plan_create_blocks: host allocation failed");
}

int es_plan_destroy(es_plan_t* plan) {
    if (plan == nullptr) return ES_OK;
    int rc = release_device_memory(plan->device, plan->d_tiles, plan->d_scratch,
                                   "es_plan_destroy");
    if (plan->d_master != nullptr) {
        const int rc2 = release_device_memory(plan->device, plan->d_master, nullptr,
                                              "es_plan_destroy");
        if (rc == ES_OK) rc = rc2;
    }
    delete plan;
    return rc;
}

int es_plan_set_master(es_plan_t* plan, void* const* masters, uint32_t n) try {
    if (plan == nullptr) return fail(ES_ERR_INVALID_ARG, "es_plan_set_master: null plan");
    if (masters == nullptr) {                         // detach
        if (plan->d_master == nullptr) return ES_OK;
        uint64_t* old = plan->d_master;
        plan->d_master = nullptr;
        return release_device_memory(plan->device, old, nullptr, "es_plan_set_master");
    }
    if (n != plan->owners.size())
        return fail(ES_ERR_INVALID_ARG, "es_plan_set_master: " + std::to_string(n) +
                                            " masters for a plan of " +
                                            std::to_string(plan->owners.size()) + " tensors");
    int rc = check_device(plan);
    if (rc != ES_OK) return rc;
    // validation: 16-byte aligned, inside one allocation of this device, and
    // overlapping no other master and no bf16 tensor of the plan
    std::vector<std::pair<uintptr_t, uintptr_t>> ranges;
    for (uint32_t i = 0; i < n; ++i) {
        const uint64_t numel = plan->owners[i].second;
        if (numel == 0) continue;
        const std::string where = "es_plan_set_master: master " + std::to_string(i);
        const uintptr_t a = reinterpret_cast<uintptr_t>(masters[i]);
        if (a == 0) return fail(ES_ERR_INVALID_ARG, where + ": null");
        if (a % 16 != 0) return fail(ES_ERR_ALIGN, where + ": not 16-byte aligned");
        rc = check_access(masters[i], 4 * numel, plan->device, where);
        if (rc != ES_OK) return rc;
        ranges.emplace_back(a, a + 4 * numel);
        ranges.emplace_back(plan->owners[i].first, plan->owners[i].first + 2 * numel);
    }
    std::sort(ranges.begin(), ranges.end());
    for (size_t i = 1; i < ranges.size(); ++i)
        if (ranges[i].first < ranges[i - 1].second)
            return fail(ES_ERR_INVALID_ARG,
                        "es_plan_set_master: masters overlap each other or the bf16 tensors");
    // each tile's owner: the tensor whose bf16 bytes hold the tile's first
    // element (tensors do not overlap), found by bisection over their starts
    const uint64_t n_tiles = plan->n_full + plan->n_tail + plan->n_rfull + plan->n_rtail;
    std::vector<TileDesc> tiles(n_tiles);
    hipError_t e = hipSuccess;
    if (n_tiles > 0)
        e = hipMemcpy(tiles.data(), plan->d_tiles, sizeof(TileDesc) * n_tiles,
                      hipMemcpyDeviceToHost);
    if (e != hipSuccess) return hip_fail(e, "es_plan_set_master: tile table read-back");
    std::vector<std::pair<uintptr_t, uint32_t>> starts;      // (bf16 start, owner)
    for (uint32_t i = 0; i < n; ++i)
        if (plan->owners[i].second > 0) starts.emplace_back(plan->owners[i].first, i);
    std::sort(starts.begin(), starts.end());
    std::vector<uint64_t> delta(std::max<uint64_t>(n_tiles, 1), 0);
    for (uint64_t k = 0; k < n_tiles; ++k) {
        const uintptr_t first = reinterpret_cast<uintptr_t>(tiles[k].data) + 2 * tiles[k].elem0;
        auto it = std::upper_bound(starts.begin(), starts.end(),
                                   std::make_pair(first, std::numeric_limits<uint32_t>::max()));
        const uint32_t i = std::prev(it)->second;
        delta[k] = reinterpret_cast<uintptr_t>(masters[i]) - 2 * plan->owners[i].first;
    }
    uint64_t* d = nullptr;
    e = hipMalloc(reinterpret_cast<void**>(&d), sizeof(uint64_t) * delta.size());
    if (e != hipSuccess) return fail(ES_ERR_NOMEM, std::string("hipMalloc: ") + hipGetErrorString(e));
    e = hipMemcpy(d, delta.data(), sizeof(uint64_t) * delta.size(), hipMemcpyHostToDevice);
    if (e != hipSuccess) {
        (void)hipFree(d);
        return hip_fail(e, "es_plan_set_master: table upload");
    }
    uint64_t* old = plan->d_master;
    plan->d_master = d;
    if (old != nullptr) return release_device_memory(plan->device, old, nullptr,
                                                     "es_plan_set_master");
    return ES_OK;
} catch (const std::bad_alloc&) {
    return fail(ES_ERR_NOMEM, "es_plan_set_master: host allocation failed");
}

int es_perturb_master(es_plan_t* plan, uint64_t seed, int32_t sign, float sigma,
                      es_stream_t stream) {
    if (plan == nullptr) return fail(ES_ERR_INVALID_ARG, "es_perturb_master: null plan");
    if (sign != 1 && sign != -1)
        return fail(ES_ERR_INVALID_ARG, "es_perturb_master: sign must be +1 or -1");
    if (!std::isfinite(sigma) || sigma < 0.0f)
        return fail(ES_ERR_INVALID_ARG, "es_perturb_master: sigma must be finite and >= 0");
    if (plan->d_master == nullptr)
        return fail(ES_ERR_INVALID_ARG, "es_perturb_master: the plan has no masters "
                                        "(es_plan_set_master)");
    int rc = check_device(plan);
    if (rc != ES_OK) return rc;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const double coef = sign > 0 ? double(sigma) : -double(sigma);
    Segment seg[2];
    const int n_seg = plan_segments(plan, seg);
    if (sigma != 0.0f) {
        Streams st = {};
        st.k0[0] = static_cast<uint32_t>(seed);
        st.k1[0] = static_cast<uint32_t>(seed >> 32);
        st.coef_k[0] = static_cast<float>(coef * kSqrt2Ln2Double);
        for (int k = 0; k < n_seg; ++k) {
            const Segment& g = seg[k];
            const bool strided = g.rows != nullptr;
            const ApplyMasterKernel kernel = apply_master_kernel(strided);
            rc = launch_steps(
                plan, g, 2,
                plan->d_master + (strided ? plan->n_full + plan->n_tail : 0),
                "es_perturb_master", ": es_apply_master_kernel", [&](const StepLaunch& l) {
                    hipLaunchKernelGGL(kernel, l.grid, dim3(kStepThreads), 0, s, l.tiles,
                                       l.n_full, l.rows, st, l.mdelta, l.shape);
                });
            if (rc != ES_OK) return rc;
        }
        return ES_OK;
    }
    // sigma == 0 rewrites the bf16 values as the masters rounded to nearest
    // even (-0 stays -0: no term is added): the update kernel's application
    // of members with a one-member table of zero weight in the plan's scratch
    const Member m{static_cast<uint32_t>(seed), static_cast<uint32_t>(seed >> 32),
                   static_cast<float>(coef * kSqrt2Ln2Double), 0u};
    const UpdateHeader h{1u, 0u, 0, 0u};
    rc = stage_words(plan->d_scratch, kOffMembers, &m, sizeof(m), s);
    if (rc == ES_OK) rc = stage_words(plan->d_scratch, kOffHeader, &h, sizeof(h), s);
    if (rc != ES_OK) return rc;
    for (int k = 0; k < n_seg; ++k) {
        const Segment& g = seg[k];
        const bool strided = g.rows != nullptr;
        const UpdateKernel kernel = update_master_kernel(strided, true);
        rc = launch_steps(
            plan, g, 2, plan->d_master + (strided ? plan->n_full + plan->n_tail : 0),
            "es_perturb_master", ": es_update_kernel", [&](const StepLaunch& l) {
                hipLaunchKernelGGL(
                    kernel, l.grid, dim3(kStepThreads), 0, s, l.tiles, l.n_full, l.rows,
                    reinterpret_cast<const Member*>(plan->d_scratch + kOffMembers),
                    reinterpret_cast<const UpdateHeader*>(plan->d_scratch + kOffHeader),
                    RoundKey{0u, 0u}, RestoreArg{0u, 0.0f}, l.mdelta, l.shape);
            });
        if (rc != ES_OK) return rc;
    }
    return ES_OK;
}

uint64_t es_plan_numel(const es_plan_t* plan) { return plan ? plan->numel : 0; }

uint64_t es_plan_device_bytes(const es_plan_t* plan) {
    if (plan == nullptr) return 0;
    const uint64_t tiles =
        std::max<uint64_t>(plan->n_full + plan->n_tail + plan->n_rfull + plan->n_rtail, 1);
    return sizeof(TileDesc) * tiles + sizeof(DevRows) * (plan->n_rfull + plan->n_rtail) +
           kScratchBytes + (plan->d_master != nullptr ? sizeof(uint64_t) * tiles : 0);
}
uint64_t es_plan_tiles(const es_plan_t* plan) {
    return plan ? plan->n_full + plan->n_tail + plan->n_rfull + plan->n_rtail : 0;
}

int es_perturb(es_plan_t* plan, uint64_t seed, int32_t sign, float sigma, es_stream_t stream) {
    return perturb_impl(plan, seed, sign, sigma, stream, "es_perturb");
}

int es_restore(es_plan_t* plan, uint64_t seed, int32_t sign, float sigma, es_stream_t stream) {
    if (sign != 1 && sign != -1)
        return fail(ES_ERR_INVALID_ARG, "es_restore: sign must be +1 or -1");
    return perturb_impl(plan, seed, -sign, sigma, stream, "es_restore");
}

int es_zscore(const float* rewards_dev, uint32_t n, float eps, float* z_dev, int32_t* status_dev,
              es_stream_t stream) {
    if (rewards_dev == nullptr || z_dev == nullptr)
        return fail(ES_ERR_INVALID_ARG, "es_zscore: null pointer");
    if (n == 0 || n > ES_MAX_MEMBERS) return fail(ES_ERR_INVALID_ARG, "es_zscore: n out of range");
    if (!std::isfinite(eps) || eps < 0.0f)
        return fail(ES_ERR_INVALID_ARG, "es_zscore: eps must be finite and >= 0");
    int device = -1;
    int rc = current_device(&device);
    if (rc == ES_OK) rc = check_update_arrays("es_zscore", device, rewards_dev, n, z_dev, status_dev);
    if (rc != ES_OK) return rc;
    hipLaunchKernelGGL(es_zscore_kernel, dim3(1), dim3(64), 0, static_cast<hipStream_t>(stream),
                       rewards_dev, n, static_cast<double>(eps), z_dev, status_dev);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "es_zscore_kernel launch");
    return ES_OK;
}

int es_update(es_plan_t* plan, const uint64_t* seeds, const int32_t* signs,
              const float* rewards_dev, uint32_t n_members, const es_update_opts_t* opts,
              float* z_out_dev, int32_t* status_out_dev, es_stream_t stream) try {
    if (plan == nullptr) return fail(ES_ERR_INVALID_ARG, "es_update: null plan");
    int rc = validate_update("es_update", seeds, signs, rewards_dev, n_members, opts);
    if (rc != ES_OK) return rc;
    rc = check_device(plan);
    if (rc == ES_OK)
        rc = check_update_arrays("es_update", plan->device, rewards_dev, n_members, z_out_dev,
                                 status_out_dev);
    if (rc != ES_OK) return rc;
    return update_impl("es_update", plan, plan->d_scratch, seeds, signs, rewards_dev, n_members,
                       opts, z_out_dev, status_out_dev, static_cast<hipStream_t>(stream));
} catch (const std::bad_alloc&) {
    return fail(ES_ERR_NOMEM, "es_update: host allocation failed");
}

int es_restore_update(es_plan_t* plan, uint64_t restore_seed, int32_t restore_sign,
                      float restore_sigma, const uint64_t* seeds, const int32_t* signs,
                      const float* rewards_dev, uint32_t n_members, const es_update_opts_t* opts,
                      float* z_out_dev, int32_t* status_out_dev, es_stream_t stream) try {
    if (plan == nullptr) return fail(ES_ERR_INVALID_ARG, "es_restore_update: null plan");
    if (restore_sign != 1 && restore_sign != -1)
        return fail(ES_ERR_INVALID_ARG, "es_restore_update: restore_sign must be +1 or -1");
    if (!std::isfinite(restore_sigma) || restore_sigma < 0.0f)
        return fail(ES_ERR_INVALID_ARG,
                    "es_restore_update: restore_sigma must be finite and >= 0");
    int rc = validate_update("es_restore_update", seeds, signs, rewards_dev, n_members, opts);
    if (rc != ES_OK) return rc;
    rc = check_device(plan);
    if (rc == ES_OK)
        rc = check_update_arrays("es_restore_update", plan->device, rewards_dev, n_members,
                                 z_out_dev, status_out_dev);
    if (rc != ES_OK) return rc;
    // es_restore with sigma 0 changes nothing: the update alone, as es_update
    const RestoreMember rm{restore_seed, restore_sign > 0 ? -double(restore_sigma)
                                                          : double(restore_sigma)};
    return update_impl("es_restore_update", plan, plan->d_scratch, seeds, signs, rewards_dev,
                       n_members, opts, z_out_dev, status_out_dev,
                       static_cast<hipStream_t>(stream), restore_sigma != 0.0f ? &rm : nullptr);
} catch (const std::bad_alloc&) {
    return fail(ES_ERR_NOMEM, "es_restore_update: host allocation failed");
}

int es_update_noalloc(es_plan_t* plan, const uint64_t* seeds, const int32_t* signs,
                      const float* rewards_dev, uint32_t n_members, const es_update_opts_t* opts,
                      float* z_out_dev, int32_t* status_out_dev, es_stream_t stream) try {
    if (plan == nullptr) return fail_in(ES_ERR_INVALID_ARG, "es_update_noalloc", "null plan");
    int rc = validate_update("es_update_noalloc", seeds, signs, rewards_dev, n_members, opts);
    if (rc != ES_OK) return rc;
    rc = check_device(plan);
    if (rc == ES_OK)
        rc = check_update_arrays("es_update_noalloc", plan->device, rewards_dev, n_members,
                                 z_out_dev, status_out_dev);
    uint8_t* d_scratch = nullptr;
    if (rc == ES_OK) rc = static_scratch(plan->device, &d_scratch);
    if (rc != ES_OK) return rc;
    return update_impl("es_update_noalloc", plan, d_scratch, seeds, signs, rewards_dev,
                       n_members, opts, z_out_dev, status_out_dev,
                       static_cast<hipStream_t>(stream));
} catch (const std::bad_alloc&) {
    return fail(ES_ERR_NOMEM, "es_update_noalloc: host allocation failed (error reporting)");
}

int es_swap(es_plan_t* plan, uint64_t seed_from, int32_t sign_from, float sigma_from,
            uint64_t seed_to, int32_t sign_to, float sigma_to, es_stream_t stream) {
    if (plan == nullptr) return fail(ES_ERR_INVALID_ARG, "es_swap: null plan");
    if ((sign_from != 1 && sign_from != -1) || (sign_to != 1 && sign_to != -1))
        return fail(ES_ERR_INVALID_ARG, "es_swap: signs must be +1 or -1");
    if (!std::isfinite(sigma_from) || sigma_from < 0.0f || !std::isfinite(sigma_to) ||
        sigma_to < 0.0f)
        return fail(ES_ERR_INVALID_ARG, "es_swap: sigmas must be finite and >= 0");
    // es_restore(from) then es_perturb(to); a zero sigma makes its half the
    // identity, as in those calls, and its stream is dropped.
    uint64_t sd[2];
    double cf[2];
    int m = 0;
    if (sigma_from != 0.0f) {
        sd[m] = seed_from;
        cf[m] = sign_from > 0 ? -double(sigma_from) : double(sigma_from);
        ++m;
    }
    if (sigma_to != 0.0f) {
        sd[m] = seed_to;
        cf[m] = sign_to > 0 ? double(sigma_to) : -double(sigma_to);
        ++m;
    }
    if (m == 0) return ES_OK;
    const int rc = check_device(plan);
    if (rc != ES_OK) return rc;
    const int streams = (m == 2 && sd[0] == sd[1]) ? 3 : m;
    return launch_streams(plan, streams, sd, cf, static_cast<hipStream_t>(stream));
}

int es_qplan_create(const es_qtensor_t* tensors, uint32_t n_tensors, es_qplan_t** out) {
    return es_qplan_create_format(tensors, n_tensors, ES_QFORMAT_INT8, out);
}

int es_qplan_create_format(const es_qtensor_t* tensors, uint32_t n_tensors, uint32_t format,
                           es_qplan_t** out) {
    return es_qplan_create_shards(tensors, nullptr, n_tensors, format, out);
}

int es_qplan_create_shards(const es_qtensor_t* tensors, const uint64_t* elem0, uint32_t n_tensors,
                           uint32_t format, es_qplan_t** out) try {
    if (out == nullptr) return fail(ES_ERR_INVALID_ARG, "es_qplan_create: null output pointer");
    *out = nullptr;
    if (tensors == nullptr) return fail(ES_ERR_INVALID_ARG, "es_qplan_create: null tensor list");
    if (n_tensors == 0 || n_tensors > ES_MAX_TENSORS)
        return fail(ES_ERR_INVALID_ARG, "es_qplan_create: n_tensors out of range");
    std::vector<QSpec> specs(n_tensors);
    for (uint32_t i = 0; i < n_tensors; ++i) {
        const es_qtensor_t& t = tensors[i];
        const std::string where = "es_qplan_create: tensor " + std::to_string(i);
        const uint64_t n0 = elem0 == nullptr ? 0 : elem0[i];
        if (t.numel >= (uint64_t(1) << 31))
            return fail(ES_ERR_INVALID_ARG, where + ": numel must be below 2^31");
        if (n0 >= (uint64_t(1) << 31) - t.numel)
            return fail(ES_ERR_INVALID_ARG, where + ": elem0 + numel must be below 2^31");
        if (n0 % 16 != 0)
            return fail(ES_ERR_INVALID_ARG, where + ": elem0 must be a multiple of 16");
        if (t.row != 0 && n0 % t.row != 0)
            return fail(ES_ERR_INVALID_ARG, where + ": elem0 must be a multiple of row");
        specs[i] = QSpec{t.data, t.scales, t.numel, t.row, t.tensor_id, n0, t.numel, 0};
    }
    return qplan_build(specs, format, out, "es_qplan_create", "tensor");
} catch (const std::bad_alloc&) {
    return fail(ES_ERR_NOMEM, "es_qplan_create: host allocation failed");
}

int es_qplan_create_blocks(const es_qblock_t* blocks, uint32_t n_blocks, uint32_t format,
                           es_qplan_t** out) try {
    if (out == nullptr) return fail(ES_ERR_INVALID_ARG, "es_qplan_create_blocks: null output pointer");
    *out = nullptr;
    if (blocks == nullptr) return fail(ES_ERR_INVALID_ARG, "es_qplan_create_blocks: null block list");
    if (n_blocks == 0 || n_blocks > ES_MAX_TENSORS)
        return fail(ES_ERR_INVALID_ARG, "es_qplan_create_blocks: n_blocks out of range");
    std::vector<QSpec> specs(n_blocks);
    for (uint32_t i = 0; i < n_blocks; ++i) {
        const std::string bad = qblock_geometry(blocks[i], specs[i]);
        if (!bad.empty())
            return fail(ES_ERR_INVALID_ARG,
                        "es_qplan_create_blocks: block " + std::to_string(i) + ": " + bad);
    }
    return qplan_build(specs, format, out, "es_qplan_create_blocks", "block");
} catch (const std::bad_alloc&) {
    return fail(ES_ERR_NOMEM, "es_qplan_create_blocks: host allocation failed");
}

int es_qplan_destroy(es_qplan_t* plan) {
    if (plan == nullptr) return ES_OK;
    const int rc = release_device_memory(plan->device, plan->d_tab, plan->d_scratch,
                                         "es_qplan_destroy");
    delete plan;
    return rc;
}

uint64_t es_qplan_numel(const es_qplan_t* plan) { return plan ? plan->numel : 0; }

uint64_t es_qplan_device_bytes(const es_qplan_t* plan) {
    return plan ? sizeof(esq::DevQTensor) * (plan->n_tensors + 1) + kScratchBytes : 0;
}

int es_qperturb(es_qplan_t* plan, uint64_t seed, int32_t sign, float sigma, es_stream_t stream) {
    return qperturb_impl(plan, seed, sign, sigma, stream, QKind::kPerturb, "es_qperturb");
}

int es_qrestore(es_qplan_t* plan, uint64_t seed, int32_t sign, float sigma, es_stream_t stream) {
    return qperturb_impl(plan, seed, sign, sigma, stream, QKind::kRestore, "es_qrestore");
}

int es_qswap(es_qplan_t* plan, uint64_t seed_from, int32_t sign_from, float sigma_from,
             uint64_t seed_to, int32_t sign_to, float sigma_to, es_stream_t stream) {
    if (plan == nullptr) return fail(ES_ERR_INVALID_ARG, "es_qswap: null plan");
    if ((sign_from != 1 && sign_from != -1) || (sign_to != 1 && sign_to != -1))
        return fail(ES_ERR_INVALID_ARG, "es_qswap: signs must be +1 or -1");
    if (!std::isfinite(sigma_from) || sigma_from < 0.0f || !std::isfinite(sigma_to) ||
        sigma_to < 0.0f)
        return fail(ES_ERR_INVALID_ARG, "es_qswap: sigmas must be finite and >= 0");
    // es_qrestore(from) then es_qperturb(to); a zero sigma makes its half the
    // identity, as in those calls (its pass would still clamp codes)
    if (sigma_from == 0.0f)
        return qperturb_impl(plan, seed_to, sign_to, sigma_to, stream, QKind::kPerturb, "es_qswap");
    if (sigma_to == 0.0f)
        return qperturb_impl(plan, seed_from, sign_from, sigma_from, stream, QKind::kRestore,
                             "es_qswap");
    const int rc = check_qdevice(plan);
    if (rc != ES_OK) return rc;
    QPass ps = {};
    ps.m = qmember(seed_to, sign_to, sigma_to);
    ps.m_from = qmember(seed_from, sign_from, sigma_from);
    return launch_qpass(plan, QKind::kSwap, ps, static_cast<hipStream_t>(stream));
}

int es_qupdate(es_qplan_t* plan, const uint64_t* seeds, const int32_t* signs,
               const float* rewards_dev, uint32_t n_members, const es_update_opts_t* opts,
               float* z_out_dev, int32_t* status_out_dev, es_stream_t stream) try {
    if (plan == nullptr) return fail(ES_ERR_INVALID_ARG, "es_qupdate: null plan");
    int rc = validate_update("es_qupdate", seeds, signs, rewards_dev, n_members, opts);
    if (rc != ES_OK) return rc;
    if (opts->flags & ES_UPDATE_MASTER)
        return fail(ES_ERR_INVALID_ARG, "es_qupdate: quantized plans have no binary32 masters");
    rc = check_qdevice(plan);
    if (rc == ES_OK)
        rc = check_update_arrays("es_qupdate", plan->device, rewards_dev, n_members, z_out_dev,
                                 status_out_dev);
    if (rc != ES_OK) return rc;
    hipStream_t s = static_cast<hipStream_t>(stream);
    rc = prepare_update(plan->d_scratch, seeds, signs, rewards_dev, n_members, opts, z_out_dev,
                        status_out_dev, s);
    if (rc != ES_OK) return rc;
    QPass ps = {};
    ps.dk0 = static_cast<uint32_t>(opts->round_seed);
    ps.dk1 = static_cast<uint32_t>(opts->round_seed >> 32);
    return launch_qpass(plan, QKind::kUpdate, ps, s);
} catch (const std::bad_alloc&) {
    return fail(ES_ERR_NOMEM, "es_qupdate: host allocation failed");
}

int es_stream_pass(es_plan_t* plan, es_stream_t stream) {
    if (plan == nullptr) return fail(ES_ERR_INVALID_ARG, "es_stream_pass: null plan");
    const int rc = check_device(plan);
    if (rc != ES_OK) return rc;
    Segment seg[2];
    const int n_seg = plan_segments(plan, seg);
    for (int k = 0; k < n_seg; ++k) {
        const Segment& g = seg[k];
        const bool four = four_groups(plan, g);
        const int rc2 = launch_steps(
            plan, g, four ? 4 : 2, nullptr, "", "es_stream_kernel", [&](const StepLaunch& l) {
                hipLaunchKernelGGL(four ? es_stream_kernel<4> : es_stream_kernel<2>, l.grid,
                                   dim3(kStepThreads), 0, static_cast<hipStream_t>(stream),
                                   l.tiles, l.n_full, 0u, l.shape);
            });
        if (rc2 != ES_OK) return rc2;
    }
    return ES_OK;
}

int es_hbm_calibrate(void* buf_dev, uint64_t bytes, int32_t mode, uint32_t* sink_dev,
                     es_stream_t stream) {
    constexpr uint64_t kTileBytes = uint64_t(kDefaultThreads) * kDefaultGroups * 16;
    const int32_t kind = mode & ~ES_CALIBRATE_TEMPORAL;
    const bool nt = (mode & ES_CALIBRATE_TEMPORAL) == 0;
    if (mode < 0 || kind > 2)
        return fail(ES_ERR_INVALID_ARG,
                    "es_hbm_calibrate: mode not 0, 1 or 2 (optionally | ES_CALIBRATE_TEMPORAL)");
    if (buf_dev == nullptr || (kind == 0 && sink_dev == nullptr))
        return fail(ES_ERR_INVALID_ARG, "es_hbm_calibrate: null pointer");
    if (bytes == 0 || bytes % kTileBytes != 0)
        return fail(ES_ERR_INVALID_ARG, "es_hbm_calibrate: bytes not a positive multiple of 131072");
    if (reinterpret_cast<uintptr_t>(buf_dev) % 16 != 0 ||
        (kind == 0 && reinterpret_cast<uintptr_t>(sink_dev) % 4 != 0))
        return fail(ES_ERR_ALIGN, "es_hbm_calibrate: buffer not 16-byte aligned");
    int device = -1;
    int rc = current_device(&device);
    if (rc == ES_OK) rc = check_access(buf_dev, bytes, device, "es_hbm_calibrate: buffer");
    if (rc == ES_OK && kind == 0)
        rc = check_access(sink_dev, 4, device, "es_hbm_calibrate: sink");
    if (rc != ES_OK) return rc;
    int cus = 0;
    hipError_t e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device);
    if (e != hipSuccess) return hip_fail(e, "hipDeviceGetAttribute");
    const uint64_t n_tiles = bytes / kTileBytes;
    const dim3 grid(static_cast<uint32_t>(std::min<uint64_t>(n_tiles, uint64_t(cus))));
    const hipStream_t s = static_cast<hipStream_t>(stream);
    u32x4_t* buf = static_cast<u32x4_t*>(buf_dev);
    using CalKernel = void (*)(u32x4_t*, uint64_t, uint32_t*, uint32_t);
    constexpr int kT = kDefaultThreads, kG = kDefaultGroups;
    const CalKernel kernels[2][3] = {
        {es_calibrate_kernel<kT, kG, 0, false>, es_calibrate_kernel<kT, kG, 1, false>,
         es_calibrate_kernel<kT, kG, 2, false>},
        {es_calibrate_kernel<kT, kG, 0, true>, es_calibrate_kernel<kT, kG, 1, true>,
         es_calibrate_kernel<kT, kG, 2, true>}};
    hipLaunchKernelGGL(kernels[nt ? 1 : 0][kind], grid, dim3(kDefaultThreads), 0, s, buf, n_tiles,
                       sink_dev, 0u);
    e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "es_calibrate_kernel launch");
    return ES_OK;
}

int es_plan_checksum(es_plan_t* plan, uint64_t* out_dev, es_stream_t stream) {
    if (plan == nullptr || out_dev == nullptr)
        return fail(ES_ERR_INVALID_ARG, "es_plan_checksum: null pointer");
    if (reinterpret_cast<uintptr_t>(out_dev) % 8 != 0)
        return fail(ES_ERR_ALIGN, "es_plan_checksum: output not 8-byte aligned");
    int rc = check_device(plan);
    if (rc == ES_OK) rc = check_access(out_dev, 8, plan->device, "es_plan_checksum: output");
    if (rc != ES_OK) return rc;
    const hipStream_t s = static_cast<hipStream_t>(stream);
    unsigned long long* out = reinterpret_cast<unsigned long long*>(out_dev);
    hipLaunchKernelGGL(es_zero_u64_kernel, dim3(1), dim3(64), 0, s, out);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "es_zero_u64_kernel launch");
    Segment seg[2];
    const int n_seg = plan_segments(plan, seg);
    for (int k = 0; k < n_seg; ++k) {
        const Segment& g = seg[k];
        const SumLaunch l = sum_launch(g.n_full, g.n_tail, plan->groups, g.grid_sum);
        hipLaunchKernelGGL(checksum_kernel(plan->threads, plan->groups, g.rows != nullptr,
                                           l.shift > 0),
                           dim3(l.grid), dim3(plan->threads), 0, s, g.tiles, g.n_full, g.n_tail,
                           g.rows, l.shift, out);
        e = hipGetLastError();
        if (e != hipSuccess) return hip_fail(e, "es_checksum_kernel launch");
    }
    return ES_OK;
}

int es_qplan_checksum(es_qplan_t* plan, uint64_t* out_dev, es_stream_t stream) {
    if (plan == nullptr || out_dev == nullptr)
        return fail(ES_ERR_INVALID_ARG, "es_qplan_checksum: null pointer");
    if (reinterpret_cast<uintptr_t>(out_dev) % 8 != 0)
        return fail(ES_ERR_ALIGN, "es_qplan_checksum: output not 8-byte aligned");
    int rc = check_qdevice(plan);
    if (rc == ES_OK) rc = check_access(out_dev, 8, plan->device, "es_qplan_checksum: output");
    if (rc != ES_OK) return rc;
    const hipStream_t s = static_cast<hipStream_t>(stream);
    unsigned long long* out = reinterpret_cast<unsigned long long*>(out_dev);
    hipLaunchKernelGGL(es_zero_u64_kernel, dim3(1), dim3(64), 0, s, out);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "es_zero_u64_kernel launch");
    if (plan->n_full + plan->n_tail == 0) return ES_OK;
    const SumLaunch l = sum_launch(plan->n_full, plan->n_tail, plan->groups, plan->grid);
    hipLaunchKernelGGL(qchecksum_kernel(plan->threads, plan->groups, l.shift > 0), dim3(l.grid),
                       dim3(plan->threads), 0, s, plan->d_tab, plan->n_full, plan->n_tail,
                       plan->n_tensors, l.shift, out);
    e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "es_qchecksum_kernel launch");
    return ES_OK;
}

double es_sigma_cosine(double sigma0, double sigma_T, uint32_t t, uint32_t T) {
    if (T == 0 || t > T) return NAN;
    return sigma_T + (sigma0 - sigma_T) * (1.0 + std::cos(M_PI * double(t) / double(T))) / 2.0;
}

int es_philox_words(uint64_t seed, uint32_t tensor_id, uint32_t domain, uint64_t quad0,
                    uint64_t n_quads, uint32_t* out_dev, es_stream_t stream) {
    if (out_dev == nullptr) return fail(ES_ERR_INVALID_ARG, "es_philox_words: null output");
    if (n_quads > (uint64_t(1) << 28)) return fail(ES_ERR_INVALID_ARG, "es_philox_words: n_quads too large");
    if (reinterpret_cast<uintptr_t>(out_dev) % 16 != 0)
        return fail(ES_ERR_ALIGN, "es_philox_words: output not 16-byte aligned");
    if (n_quads == 0) return ES_OK;
    int device = -1;
    int rc = current_device(&device);
    if (rc == ES_OK) rc = check_access(out_dev, 16 * n_quads, device, "es_philox_words: output");
    if (rc != ES_OK) return rc;
    const uint32_t blocks = static_cast<uint32_t>((n_quads + kAuxBlock - 1) / kAuxBlock);
    hipLaunchKernelGGL(es_philox_words_kernel, dim3(blocks), dim3(kAuxBlock), 0,
                       static_cast<hipStream_t>(stream), static_cast<uint32_t>(seed),
                       static_cast<uint32_t>(seed >> 32), tensor_id, domain, quad0, n_quads,
                       reinterpret_cast<uint4*>(out_dev));
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "es_philox_words_kernel launch");
    return ES_OK;
}

int es_normals(uint64_t seed, uint32_t tensor_id, uint64_t elem0, uint64_t n, float* out_dev,
               es_stream_t stream) {
    if (out_dev == nullptr) return fail(ES_ERR_INVALID_ARG, "es_normals: null output");
    if (n > (uint64_t(1) << 30)) return fail(ES_ERR_INVALID_ARG, "es_normals: n too large");
    if (elem0 > (uint64_t(1) << 62) - n) return fail(ES_ERR_INVALID_ARG, "es_normals: element range beyond 2^62");
    if (n == 0) return ES_OK;
    int device = -1;
    int rc = current_device(&device);
    if (rc == ES_OK) rc = check_access(out_dev, 4 * n, device, "es_normals: output");
    if (rc != ES_OK) return rc;
    const uint64_t quads = ((elem0 + n - 1) >> 2) - (elem0 >> 2) + 1;
    const uint32_t blocks = static_cast<uint32_t>((quads + kAuxBlock - 1) / kAuxBlock);
    hipLaunchKernelGGL(es_normals_kernel, dim3(blocks), dim3(kAuxBlock), 0,
                       static_cast<hipStream_t>(stream), static_cast<uint32_t>(seed),
                       static_cast<uint32_t>(seed >> 32), tensor_id, elem0, n, out_dev);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "es_normals_kernel launch");
    return ES_OK;
}

int es_tile_layout(uint64_t addr, uint64_t numel, uint32_t offset8, es_tile_info_t* out,
                   uint64_t cap, uint64_t* n_tiles) try {
    if (n_tiles == nullptr) return fail(ES_ERR_INVALID_ARG, "es_tile_layout: null n_tiles");
    *n_tiles = 0;
    if (numel > (uint64_t(1) << 60) - 8 * uint64_t(offset8))
        return fail(ES_ERR_INVALID_ARG, "es_tile_layout: 8 * offset8 + numel above 2^60");
    if (cap > 0 && out == nullptr) return fail(ES_ERR_INVALID_ARG, "es_tile_layout: null output");
    if (numel > 0 && (addr & 1u)) return fail(ES_ERR_ALIGN, "es_tile_layout: address not 2-byte aligned");
    int threads = 0, groups = 0;
    launch_shape(threads, groups);
    const uint64_t tile_elems = uint64_t(threads) * groups * kGroupElems;
    if (numel / tile_elems > kMaxLayoutTiles)
        return fail(ES_ERR_INVALID_ARG, "es_tile_layout: more than 2^22 tiles");
    std::vector<DevTile> full, tail;
    tile_tensor(reinterpret_cast<uint16_t*>(static_cast<uintptr_t>(addr)), numel,
                8 * uint64_t(offset8), 0u, tile_elems, full, tail);
    const uint64_t n = full.size() + tail.size();
    for (uint64_t i = 0; i < std::min(cap, n); ++i) {
        const DevTile& d = i < full.size() ? full[i] : tail[i - full.size()];
        out[i] = es_tile_info_t{d.elem0, d.limit, i < full.size() ? 1u : 0u, d.aligned16};
    }
    *n_tiles = n;
    return ES_OK;
} catch (const std::bad_alloc&) {
    return fail(ES_ERR_NOMEM, "es_tile_layout: host allocation failed");
}

const char* es_strerror(int code) {
    switch (code) {
        case ES_OK: return "ES_OK";
        case ES_ERR_INVALID_ARG: return "ES_ERR_INVALID_ARG";
        case ES_ERR_ALIGN: return "ES_ERR_ALIGN";
        case ES_ERR_HIP: return "ES_ERR_HIP";
        case ES_ERR_DEVICE: return "ES_ERR_DEVICE";
        case ES_ERR_NOMEM: return "ES_ERR_NOMEM";
        default: return "ES_ERR_UNKNOWN";
    }
}

const char* es_last_error(void) { return g_last_error.c_str(); }

}  // extern "C"
