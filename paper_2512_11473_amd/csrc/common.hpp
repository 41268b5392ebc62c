// Internal helpers shared by the sgrid HIP sources: status reporting, the
// grid handle, launch checks and small device utilities for gfx950.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stdio.h>
#include <string>

#include "../../include/sgrid.h"

namespace sgrid {

void set_error(const char *fmt, ...);
void clear_error();

// Device memory of the library (tables, workspaces) comes from a small
// per-process caching allocator: freed blocks are kept and handed out again
// to requests of the same rounded size, so repeated builds make no driver
// allocation calls.  dev_free must only be called once no queued work uses
// the block.
sgrid_status dev_alloc(void **p, size_t bytes, const char *what);
void dev_free(void *p);

// Compute units of the current device (cached).
int cu_count();

// *p = 0 on `st` by a one-lane kernel (no memset node in a captured graph).
sgrid_status launch_zero_u32(uint32_t *p, hipStream_t st);

// Far-field package ids and the far-field constant in units of h.
constexpr uint32_t kFarNeg = 0u;
constexpr uint32_t kFarPos = 1u;
constexpr uint32_t kNoCell = 0xFFFFFFFFu;
constexpr double kFarFieldInH = 16.0;

// Sweep groups: 64 consecutive worklist entries (Morton order) are swept by one
// workgroup, which shares their rows through LDS.
constexpr int kGroup = 64;
constexpr uint32_t kLocal = 0x80000000u;

// Face slots of the 27-entry neighbour table, in the order the sweeps use:
// -x, +x, -y, +y, -z, +z.
constexpr int kFaceSlot[6] = {12, 14, 10, 16, 4, 22};

}  // namespace sgrid

struct sgrid_grid {
    int32_t M = 0;
    double h = 0.0;
    int64_t P = 0;        // activated packages
    int64_t n_core = 0;
    int device = 0;
    uint32_t *cell_pkg = nullptr;   // [M^3]
    uint32_t *pkg_cell = nullptr;   // [P+2]
    uint8_t *pkg_type = nullptr;    // [P+2]
    uint32_t *nbr = nullptr;        // [P+2][27]
    uint32_t *face = nullptr;       // [P+2][8]: the six face slots of nbr, then two pads
    uint32_t *core_list = nullptr;  // [n_core]
    uint32_t *work = nullptr;       // [P]: activated package ids in Morton order of their cells
    uint32_t *wface = nullptr;      // [P][8]: per worklist position: six face neighbours, own id, pad
    uint32_t *sface = nullptr;      // [P][8]: per worklist position: six face neighbours (package id, or
                                    // group slot | kLocal when in the same 64-package group), own id, pad
    uint32_t *wpos = nullptr;       // [P+2]: position of each package in the worklist
    uint32_t *mface = nullptr;      // [P][8]: per worklist position e: the six face neighbours' rows in the
                                    // worklist-ordered field copy (2 + position, far fields 0 and 1), own id, pad
    void *workspace = nullptr;      // build scratch, kept until destroy
    // compact form of cell_pkg for position lookups: per 32 cells of a row,
    // {activated bits, negative-sign bits, activated cells before them, 0}
    uint4 *rank_map = nullptr;      // [M * M * W32]
    int32_t W32 = 0;                // entries per row: ceil(M / 32)
    int64_t total() const { return P + 2; }
};

#define SG_CHECK_HIP(expr)                                                            \
    do {                                                                              \
        hipError_t _e = (expr);                                                       \
        if (_e != hipSuccess) {                                                       \
            sgrid::set_error("%s failed: %s (%s:%d)", #expr, hipGetErrorString(_e),   \
                             __FILE__, __LINE__);                                     \
            return SGRID_E_HIP;                                                       \
        }                                                                             \
    } while (0)

#define SG_CHECK_LAUNCH(name)                                                         \
    do {                                                                              \
        hipError_t _e = hipGetLastError();                                            \
        if (_e != hipSuccess) {                                                       \
            sgrid::set_error("launch of %s failed: %s", name, hipGetErrorString(_e)); \
            return SGRID_E_HIP;                                                       \
        }                                                                             \
    } while (0)

#define SG_REQUIRE(cond, ...)                              \
    do {                                                   \
        if (!(cond)) {                                     \
            sgrid::set_error(__VA_ARGS__);                 \
            return SGRID_E_INVALID;                        \
        }                                                  \
    } while (0)

static inline bool sg_aligned(const void *p, size_t a) { return (reinterpret_cast<uintptr_t>(p) % a) == 0; }

static inline hipStream_t sg_stream(void *s) { return reinterpret_cast<hipStream_t>(s); }

// Grids of more than 2^31 - 1 blocks are not launched; callers loop or stride.
constexpr int64_t kMaxGrid = 0x7FFFFFFF;

// ---------------------------------------------------------------------------
// Device utilities
// ---------------------------------------------------------------------------

// Neighbour values of a package's four-value row in y and z.  A package is one
// 16-lane DPP row; lane r = j + 4 k holds row (j, k), so its y neighbours are lanes
// r -+ 1 and its z neighbours lanes r -+ 4.  Lanes at the package's face take the
// halo value h instead: lo gets it on the lanes of mask LO, hi on those of mask HI.
// Each neighbour value is one select whose first operand moves between lanes; the
// compiler, which wants the move and the select (or a copy of h, kept twice) as two
// instructions, needs 28 for the sixteen of a row.  A sweep with these and with
// 32-bit offsets, before and now: torus at 256^3 points 4.7 and 4.55 us, prism512
// 12.2 and 12.05, torus at 768^3 23.5 and 22.2, at 2048^3 221.7 and 217.6.
// The select's mask is VCC.  The
// block's first two instructions give the two wait states that the hardware asks
// for between a vector write and a DPP read of its result.  Must run in every lane
// of a package: a lane outside the active mask supplies 0 to its neighbours, so a
// call inside a lane-dependent branch reads wrong values.
constexpr uint64_t kLanesJ0 = 0x1111111111111111ull, kLanesJ3 = 0x8888888888888888ull;
constexpr uint64_t kLanesK0 = 0x000F000F000F000Full, kLanesK3 = 0xF000F000F000F000ull;

#define SG_DPP_SELECT(D, S, H, CTRL) \
    "v_cndmask_b32_dpp %" #D ", %" #S ", %" #H ", vcc " CTRL " row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
#define SG_ROW_NEIGHBOURS(DOWN, UP, LO, HI)                                                                       \
    asm("s_mov_b64 vcc, %16\n\ts_nop 1\n\t"                                                                     \
        SG_DPP_SELECT(0, 8, 12, DOWN) SG_DPP_SELECT(1, 9, 13, DOWN)                                               \
        SG_DPP_SELECT(2, 10, 14, DOWN) SG_DPP_SELECT(3, 11, 15, DOWN)                                             \
        "s_mov_b64 vcc, %17\n\t"                                                                                 \
        SG_DPP_SELECT(4, 8, 12, UP) SG_DPP_SELECT(5, 9, 13, UP)                                                   \
        SG_DPP_SELECT(6, 10, 14, UP) SG_DPP_SELECT(7, 11, 15, UP)                                                 \
        : "=&v"(lo[0]), "=&v"(lo[1]), "=&v"(lo[2]), "=&v"(lo[3]), "=&v"(hi[0]), "=&v"(hi[1]), "=&v"(hi[2]),       \
          "=&v"(hi[3])                                                                                            \
        : "v"(c[0]), "v"(c[1]), "v"(c[2]), "v"(c[3]), "v"(h[0]), "v"(h[1]), "v"(h[2]), "v"(h[3]), "s"(LO), "s"(HI) \
        : "vcc")

__device__ __forceinline__ void neighbours_y(const uint32_t (&c)[4], const uint32_t (&h)[4], uint32_t (&lo)[4],
                                             uint32_t (&hi)[4]) {
    SG_ROW_NEIGHBOURS("row_shr:1", "row_shl:1", kLanesJ0, kLanesJ3);
}
__device__ __forceinline__ void neighbours_z(const uint32_t (&c)[4], const uint32_t (&h)[4], uint32_t (&lo)[4],
                                             uint32_t (&hi)[4]) {
    SG_ROW_NEIGHBOURS("row_shr:4", "row_shl:4", kLanesK0, kLanesK3);
}
#undef SG_ROW_NEIGHBOURS
#undef SG_DPP_SELECT

// The same for four values of type T, by 32-bit words.
template <bool Z, typename T>
__device__ __forceinline__ void row_neighbours(const T (&c)[4], const T (&h)[4], T (&lo)[4], T (&hi)[4]) {
    constexpr int W = sizeof(T) / 4;
    struct Words { uint32_t w[W]; };
    uint32_t l[W][4], u[W][4];
#pragma unroll
    for (int w = 0; w < W; ++w) {
        uint32_t cw[4], hw[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            cw[i] = __builtin_bit_cast(Words, c[i]).w[w];
            hw[i] = __builtin_bit_cast(Words, h[i]).w[w];
        }
        if (Z)
            neighbours_z(cw, hw, l[w], u[w]);
        else
            neighbours_y(cw, hw, l[w], u[w]);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        Words a, b;
#pragma unroll
        for (int w = 0; w < W; ++w) {
            a.w[w] = l[w][i];
            b.w[w] = u[w][i];
        }
        lo[i] = __builtin_bit_cast(T, a);
        hi[i] = __builtin_bit_cast(T, b);
    }
}

// The same moves as the compiler's own instructions, two per neighbour: for kernels
// that keep a set's loads in flight with the one before it or behind a barrier,
// where the block above, which waits for all its operands at once, is the slower.
// row_move: lanes whose source lies outside their 16-lane row read 0 and must not
// use the result.  row_move_keep: lanes of the banks (groups of four lanes of a row)
// left out of BANKS keep `keep`.
constexpr int kRowShl1 = 0x101, kRowShl4 = 0x104, kRowShr1 = 0x111, kRowShr4 = 0x114;

template <int CTRL>
__device__ __forceinline__ uint32_t row_move(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, CTRL, 0xF, 0xF, true);
}
template <int CTRL, int BANKS>
__device__ __forceinline__ uint32_t row_move_keep(uint32_t v, uint32_t keep) {
    return (uint32_t)__builtin_amdgcn_update_dpp((int)keep, (int)v, CTRL, 0xF, BANKS, false);
}
// `op` on a value's 32-bit words.
template <typename T, class Op>
__device__ __forceinline__ T by_words(T a, T b, Op op) {
    struct Words { uint32_t w[sizeof(T) / 4]; };
    Words x = __builtin_bit_cast(Words, a);
    const Words y = __builtin_bit_cast(Words, b);
#pragma unroll
    for (unsigned i = 0; i < sizeof(T) / 4; ++i) x.w[i] = op(x.w[i], y.w[i]);
    return __builtin_bit_cast(T, x);
}

// 16-byte store written through the L2 (device scope, sc1) instead of left
// dirty in it.  The eight XCDs' L2 caches (4 MiB each) do not see each other's
// lines, so a kernel's dirty lines are written back when it ends, after its last
// wavefront; a pass whose output the next kernel reads from everywhere pays for
// that as a tail (prism512's sweep leaves all of its 31 MiB there).  Written
// through, the rows leave while the kernel runs, and stay in the Infinity Cache
// (which the streaming hint would bypass).  Sweeps with plain stores and with
// these: torus at 256^3 points 5.8 and 5.2 us, prism512 14.6 and 13.6, torus at
// 768^3 26.0 and 25.1, at 1024^3 41.3 and 40.4.  The compiler does not see a
// store in the asm: it does not count it in its waits for loads, which makes them
// at most longer, and it does not keep the two wait states that gfx940 and later
// (earlier chips: one) ask for between a store of more than 8 bytes and a vector
// write to its data registers, so the asm ends with them.
typedef float f32x4_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ void store_through(void *p, f32x4_t v) {
    asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 1" : : "v"(p), "v"(v) : "memory");
}
__device__ __forceinline__ void store_through(void *base, uint32_t off, f32x4_t v) {
    asm volatile("global_store_dwordx4 %0, %1, %2 sc1\n\ts_nop 1" : : "v"(off), "v"(v), "s"(base) : "memory");
}
__device__ __forceinline__ void store_through(void *base, int64_t off, f32x4_t v) {
    store_through(static_cast<char *>(base) + off, v);
}

// Point order of the packed (phi, g) probe field: the 64 points of a package
// in 2 x 2 x 2 blocks, so the eight corners of a trilinear cell that lies
// inside one block share one 128-byte line (FP32).
__host__ __device__ __forceinline__ int blocked_index(int i, int j, int k) {
    return 8 * ((i >> 1) + 2 * (j >> 1) + 4 * (k >> 1)) + ((i & 1) + 2 * (j & 1) + 4 * (k & 1));
}

// XCD-aware block order: the hardware deals consecutive workgroups round-robin
// to the 8 XCDs; remapping gives each XCD one contiguous range of block ids,
// so packages that are neighbours in id order share that XCD's L2.
__device__ __forceinline__ int64_t xcd_block(int64_t b, int64_t nb) {
    const int64_t per = (nb + 7) / 8;
    const int64_t x = b % 8, r = b / 8;
    const int64_t full = nb % 8 == 0 ? 8 : nb % 8;   // XCDs that receive `per` blocks
    // XCDs 0..full-1 own ranges of length per, the rest ranges of length per - 1
    return x < full ? x * per + r : full * per + (x - full) * (per - 1) + r;
}
// A workgroup's block in that order, with arithmetic in I (nb < 2^31, as every
// grid's: 32 bits do, and take a third of the scalar instructions).
template <typename I>
__device__ __forceinline__ I block_of(I nb) {
    const I per = (nb + 7) / 8, x = blockIdx.x % 8, r = blockIdx.x / 8;
    const I full = nb % 8 == 0 ? 8 : nb % 8;
    return x < full ? x * per + r : full * per + (x - full) * (per - 1) + r;
}

// Byte offset of value `at` of package row `row` in a field, in the index type I.
// With 32-bit offsets from a base that is the same for every lane an address is
// one vector instruction (shift and or); with 64-bit ones it takes five or six,
// and the sweeps form six addresses per lane: 157 vector instructions per
// wavefront become 134.
template <typename T, typename I>
__device__ __forceinline__ I row_offset(uint32_t row, int at) {
    return (I)row * (I)(64 * sizeof(T)) + (I)(at * (int)sizeof(T));
}
template <typename T, typename I>
__device__ __forceinline__ const T *at_offset(const T *base, I off) {
    return reinterpret_cast<const T *>(reinterpret_cast<const char *>(base) + off);
}
template <typename T, typename I>
__device__ __forceinline__ T *at_offset(T *base, I off) {
    return reinterpret_cast<T *>(reinterpret_cast<char *>(base) + off);
}
