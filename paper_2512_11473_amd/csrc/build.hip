// Package activation, numbering and neighbour tables (Sec. 4, Sec. 5 and
// Sec. 7.1 steps 1-3 and 5 of the paper), plus the handle lifecycle and error
// reporting of the C ABI.
//
// Pipeline on the caller's stream (coarse cells held as bitmaps, 64 cells of a
// row per word):
//   bits_kernel     one wavefront per 16 words: core flag |d| < l_c and sign of d,
//                   one ballot each;
//   dilate_kernel   one lane per word: activated = core dilated by one cell in
//                   x, y, z (word shifts and ORs); per-group counts;
//   scan_counts     exclusive scan of the counts (one workgroup while it can,
//                   else block sums, one workgroup over them, block scans);
//   (host)          P and n_core once, from a pinned word; the package tables;
//   scatter_kernel  16 words per wavefront in steps of four, four cells per lane: rank by
//                   popcount below the cell plus word offsets from the scan,
//                   id = 2 + rank in ascending linear order (no sort needed);
//                   the cell map in 16-byte stores, the rank map;
//   nbr_kernel      nine lanes per package: the neighbour table and the six
//                   face slots copied into a 32-byte row per package;
//   morton_*        the sweep worklist in Morton order of the cells, one lane
//                   per 4 x 4 x 4 box of codes.
// The next layer of the multi-resolution construction replaces bits_kernel by
// refine_bits_kernel (the parent layer's rank map and the children's
// distances) and shares the rest.
#include <stdarg.h>
#include <stdlib.h>
#include <string.h>

#include <atomic>
#include <mutex>
#include <unordered_map>
#include <vector>

#include "common.hpp"

namespace sgrid {

static thread_local std::string g_last_error;

void set_error(const char *fmt, ...) {
    char buf[1024];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_last_error = buf;
}

void clear_error() { g_last_error.clear(); }

namespace {
struct CachedBlock {
    void *ptr;
    size_t bytes;
    int device;
};
std::mutex g_alloc_mu;
std::vector<CachedBlock> g_free_blocks;
std::unordered_map<void *, CachedBlock> g_live_blocks;

size_t round_bytes(size_t b) {
    const size_t q = b <= (1u << 20) ? 4096 : (2u << 20);
    return (b + q - 1) / q * q;
}
}  // namespace

sgrid_status dev_alloc(void **p, size_t bytes, const char *what) {
    int dev = 0;
    (void)hipGetDevice(&dev);
    const size_t rb = round_bytes(bytes == 0 ? 1 : bytes);
    {
        std::lock_guard<std::mutex> lk(g_alloc_mu);
        for (size_t i = 0; i < g_free_blocks.size(); ++i) {
            if (g_free_blocks[i].bytes == rb && g_free_blocks[i].device == dev) {
                CachedBlock b = g_free_blocks[i];
                g_free_blocks[i] = g_free_blocks.back();
                g_free_blocks.pop_back();
                g_live_blocks[b.ptr] = b;
                *p = b.ptr;
                return SGRID_OK;
            }
        }
    }
    hipError_t e = hipMalloc(p, rb);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        // give cached blocks back to the driver and retry once
        std::vector<CachedBlock> drop;
        {
            std::lock_guard<std::mutex> lk(g_alloc_mu);
            drop.swap(g_free_blocks);
        }
        for (auto &b : drop) (void)hipFree(b.ptr);
        e = hipMalloc(p, rb);
    }
    if (e != hipSuccess) {
        (void)hipGetLastError();
        *p = nullptr;
        set_error("allocation of %zu bytes for %s failed: %s", bytes, what, hipGetErrorString(e));
        return SGRID_E_NOMEM;
    }
    std::lock_guard<std::mutex> lk(g_alloc_mu);
    g_live_blocks[*p] = CachedBlock{*p, rb, dev};
    return SGRID_OK;
}

void dev_free(void *p) {
    if (!p) return;
    std::lock_guard<std::mutex> lk(g_alloc_mu);
    auto it = g_live_blocks.find(p);
    if (it == g_live_blocks.end()) return;
    g_free_blocks.push_back(it->second);
    g_live_blocks.erase(it);
}

int cu_count() {
    static std::atomic<int> cached[64];   // 0 until first asked; threads that race store the same value
    int dev = 0;
    (void)hipGetDevice(&dev);
    if (dev < 0 || dev >= 64) return 256;
    int n = cached[dev].load(std::memory_order_relaxed);
    if (n == 0) {
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = 256;
        cached[dev].store(n, std::memory_order_relaxed);
    }
    return n;
}

}  // namespace sgrid

extern "C" const char *sgrid_last_error(void) { return sgrid::g_last_error.c_str(); }

extern "C" int32_t sgrid_version(void) { return 10000; }

namespace {

constexpr int kTagBlock = 256;

__device__ __forceinline__ uint64_t lanemask_lt() {
    const unsigned lane = threadIdx.x & 63u;
    return lane == 0 ? 0ull : (~0ull >> (64 - lane));
}

// Quotient of a word or row index by a row length, in 32-bit arithmetic when
// the index fits (M^2 W words stay below 2^32 up to M = 4096): a few
// instructions instead of the fifty of a 64-bit division.
__device__ __forceinline__ int64_t quot(int64_t a, int b) {
    return a < 0x100000000ll ? (int64_t)((uint32_t)a / (uint32_t)b) : a / b;
}

// Bitmaps of the background grid.  Row r = y + M z holds its M cells in
// W = ceil(M / 64) words; bit b of word r W + i is the cell x = 64 i + b.
// Bits of x >= M are zero.  Word order is linear cell order.

// Pass 1: one wavefront per word: the core flag |d| < l_c (compared in double,
// so that a non-representable l_c rounds as the definition does) and the sign
// of d, each one ballot.
constexpr int kBitsWords = 16;   // words per wavefront of bits_kernel

__global__ __launch_bounds__(256) void bits_kernel(const float *__restrict__ d, int M, int W, int64_t n_words,
                                                   double lc, uint64_t *__restrict__ core,
                                                   uint64_t *__restrict__ neg) {
    // kBitsWords consecutive words per wavefront, their loads issued together
    // (4 KiB in flight per wavefront); the words' rows and offsets advance
    // from the first word's (one division per wavefront)
    const int64_t w0 = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * kBitsWords;
    if (w0 >= n_words) return;   // whole wavefronts
    const int lane = threadIdx.x & 63;
    const int64_t r0 = quot(w0, W);
    const int i0 = (int)(w0 - r0 * W);
    float v[kBitsWords];
    bool in[kBitsWords];
    {
        int64_t r = r0;
        int i = i0;
#pragma unroll
        for (int k = 0; k < kBitsWords; ++k) {
            const int x = i * 64 + lane;
            in[k] = w0 + k < n_words && x < M;
            v[k] = d[in[k] ? r * M + x : 0];   // every lane loads, in bounds
            if (++i == W) {
                i = 0;
                ++r;
            }
        }
    }
#pragma unroll
    for (int k = 0; k < kBitsWords; ++k) {
        const int64_t w = w0 + k;
        const uint64_t bc = __ballot(in[k] && fabs((double)v[k]) < lc);
        const uint64_t bn = __ballot(in[k] && v[k] < 0.0f);
        if (lane == 0 && w < n_words) {
            core[w] = bc;
            neg[w] = bn;
        }
    }
}

// Pass 2: one lane per word: the activated cells are the core cells dilated by
// one cell along x, y and z (the cell and its 26 neighbours, Sec. 7.1 steps
// 1-2: inner = not core with a core neighbour); per group of 16 words, the
// counts of activated and of core cells feed the scan.
__global__ __launch_bounds__(256) void dilate_kernel(const uint64_t *__restrict__ core, int M, int W,
                                                     int64_t n_words, uint64_t *__restrict__ act,
                                                     uint32_t *__restrict__ cnt_act,
                                                     uint32_t *__restrict__ cnt_core) {
    const int64_t w = (int64_t)blockIdx.x * 256 + threadIdx.x;
    uint64_t a = 0, own = 0;
    if (w < n_words) {
        const int64_t r = quot(w, W);
        const int i = (int)(w - r * W);
        const int64_t rz = quot(r, M);
        const int y = (int)(r - rz * M), z = (int)rz;
        for (int dz = -1; dz <= 1; ++dz) {
            const int zz = z + dz;
            if (zz < 0 || zz >= M) continue;
            for (int dy = -1; dy <= 1; ++dy) {
                const int yy = y + dy;
                if (yy < 0 || yy >= M) continue;
                const int64_t b = ((int64_t)yy + (int64_t)M * zz) * W + i;
                const uint64_t c = core[b];
                const uint64_t lo = i > 0 ? core[b - 1] : 0ull, hi = i < W - 1 ? core[b + 1] : 0ull;
                a |= c | (c << 1) | (c >> 1) | (lo >> 63) | (hi << 63);
            }
        }
        if (i == W - 1 && (M & 63)) a &= (1ull << (M & 63)) - 1ull;
        own = core[w];
    }
    uint32_t na = (uint32_t)__popcll(a), nc = (uint32_t)__popcll(own);
#pragma unroll
    for (int off = 8; off >= 1; off >>= 1) {
        na += __shfl_xor(na, off, 16);
        nc += __shfl_xor(nc, off, 16);
    }
    if (w < n_words) {
        act[w] = a;
        if ((threadIdx.x & 15) == 0) {
            cnt_act[w >> 4] = na;
            cnt_core[w >> 4] = nc;
        }
    }
}

// Exclusive scan of one or two count arrays (N) in three passes: per-block
// sums of kScanBlock entries, one workgroup scanning the block sums (and
// writing the totals), then every block scanning its entries from its offset.
// Few counts take the one workgroup alone.
constexpr int kScanThreads = 1024;
constexpr int kScanTile = kScanThreads * 4;
constexpr int kScanBlock = 1024;   // entries per block of the first and last pass (256 lanes x 4)

template <int N>
struct Counts {
    uint32_t *p[N];
};

template <int N>
__global__ __launch_bounds__(256) void scan_reduce_kernel(Counts<N> a, int64_t n, Counts<N> sums) {
    __shared__ uint32_t ra[N][4];
    const int64_t base = (int64_t)blockIdx.x * kScanBlock + threadIdx.x * 4;
#pragma unroll
    for (int c = 0; c < N; ++c) {
        uint32_t x = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (base + k < n) x += a.p[c][base + k];
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) x += __shfl_xor(x, off);
        if ((threadIdx.x & 63) == 0) ra[c][threadIdx.x >> 6] = x;
    }
    __syncthreads();
    if (threadIdx.x < N) {
        const uint32_t *r = ra[threadIdx.x];
        sums.p[threadIdx.x][blockIdx.x] = r[0] + r[1] + r[2] + r[3];
    }
}

// Inclusive scan over the lanes of a wavefront.
template <typename U>
__device__ __forceinline__ U wave_scan(U v, int lane) {
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const U u = __shfl_up(v, off);
        if (lane >= off) v += u;
    }
    return v;
}

// One workgroup, in tiles of kScanTile entries, four per thread: a scan of the
// thread sums inside each wavefront, the wavefronts' totals through LDS (two
// barriers a tile), and a running carry between tiles.  totals (nullable, in
// pinned host memory) = the sums, then 1 in the word after them.
// Latency-bound: a Hillis-Steele scan over LDS, twenty barriers a tile, took
// 4.9 us on the 64 counts of a 16^3 grid, this one 2.4 (one array) and 3.8 (two).
template <int N>
__global__ __launch_bounds__(kScanThreads) void scan_kernel(Counts<N> a, int64_t n, uint64_t *__restrict__ totals) {
    __shared__ uint64_t wsum[2][N][kScanThreads / 64];
    uint64_t carry[N] = {};
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
    int buf = 0;
    for (int64_t base = 0; base < n; base += kScanTile, buf ^= 1) {
        uint32_t v[N][4];
        uint64_t x[N], inc[N];
#pragma unroll
        for (int c = 0; c < N; ++c) {
            x[c] = 0;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int64_t g = base + 4 * t + k;
                v[c][k] = g < n ? a.p[c][g] : 0u;
            }
        }
#pragma unroll
        for (int c = 0; c < N; ++c) {
#pragma unroll
            for (int k = 0; k < 4; ++k) x[c] += v[c][k];
            inc[c] = wave_scan(x[c], lane);
            if (lane == 63) wsum[buf][c][wv] = inc[c];
        }
        __syncthreads();
#pragma unroll
        for (int c = 0; c < N; ++c) {
            uint64_t before = 0, all = 0;
#pragma unroll
            for (int k = 0; k < kScanThreads / 64; ++k) {
                const uint64_t s = wsum[buf][c][k];
                if (k < wv) before += s;
                all += s;
            }
            uint64_t o = carry[c] + before + inc[c] - x[c];
            carry[c] += all;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int64_t g = base + 4 * t + k;
                if (g < n) a.p[c][g] = (uint32_t)o;
                o += v[c][k];
            }
        }
    }
    if (t == 0 && totals != nullptr) {
#pragma unroll
        for (int c = 0; c < N; ++c) __hip_atomic_store(totals + c, carry[c], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        __hip_atomic_store(totals + N, 1ull, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

template <int N>
__global__ __launch_bounds__(256) void scan_apply_kernel(Counts<N> a, int64_t n, Counts<N> offsets) {
    __shared__ uint32_t wsum[N][4];
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
    const int64_t base = (int64_t)blockIdx.x * kScanBlock + t * 4;
    uint32_t v[N][4], x[N], inc[N];
#pragma unroll
    for (int c = 0; c < N; ++c) {
        x[c] = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            v[c][k] = base + k < n ? a.p[c][base + k] : 0u;
            x[c] += v[c][k];
        }
        inc[c] = wave_scan(x[c], lane);
        if (lane == 63) wsum[c][wv] = inc[c];
    }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < N; ++c) {
        uint32_t o = offsets.p[c][blockIdx.x] + inc[c] - x[c];
        for (int k = 0; k < wv; ++k) o += wsum[c][k];
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (base + k < n) {
                a.p[c][base + k] = o;
                o += v[c][k];
            }
    }
}

// Exclusive scan of the N arrays a[n] in place; totals (nullable) = their
// sums.  part holds N * ceil(n / kScanBlock) words.
template <int N>
static void scan_counts(Counts<N> a, int64_t n, uint32_t *part, uint64_t *totals, hipStream_t st) {
    const int64_t nb = (n + kScanBlock - 1) / kScanBlock;
    if (n <= kScanTile) {
        hipLaunchKernelGGL(scan_kernel<N>, dim3(1), dim3(kScanThreads), 0, st, a, n, totals);
        return;
    }
    Counts<N> sums;
    for (int c = 0; c < N; ++c) sums.p[c] = part + c * nb;
    hipLaunchKernelGGL(scan_reduce_kernel<N>, dim3((unsigned)nb), dim3(256), 0, st, a, n, sums);
    hipLaunchKernelGGL(scan_kernel<N>, dim3(1), dim3(kScanThreads), 0, st, sums, nb, totals);
    hipLaunchKernelGGL(scan_apply_kernel<N>, dim3((unsigned)nb), dim3(256), 0, st, a, n, sums);
}

// Pass 4: numbering.  One workgroup per group of 16 words, four words per
// wavefront.  Cell x of word w gets id = 2 + (activated cells before the word:
// the group's offset from the scan plus the words before it in the group) +
// (activated cells of the word below x), which is ascending linear order, so
// no sort is needed.  Cells not activated take the far-field package of their
// sign.
__global__ __launch_bounds__(256) void scatter_kernel(const uint64_t *__restrict__ act,
                                                      const uint64_t *__restrict__ core,
                                                      const uint64_t *__restrict__ neg, int M, int W,
                                                      int64_t n_words, const uint32_t *__restrict__ off_act,
                                                      const uint32_t *__restrict__ off_core,
                                                      uint32_t *__restrict__ cell_pkg,
                                                      uint32_t *__restrict__ pkg_cell,
                                                      uint8_t *__restrict__ pkg_type,
                                                      uint32_t *__restrict__ core_list,
                                                      uint4 *__restrict__ rank_map, int W32) {
    // a wavefront owns one group of 16 words, in four steps of four
    // consecutive words; in a step lane l takes the four cells of bits
    // 4 (l mod 16) .. 4 (l mod 16) + 3 of word l / 16, stored with one 16-byte
    // write where the row allows it.  Lane l < 16 loads word l of the group
    // (the loads issued together) and the counts before each word come from
    // one scan over the 16 lanes; the other lanes read words and counts from
    // them.
    const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int64_t grp = (int64_t)blockIdx.x * 4 + wv;
    const int64_t g0 = grp * 16;
    if (blockIdx.x == 0 && threadIdx.x < 2) {   // the far-field packages
        pkg_cell[threadIdx.x] = sgrid::kNoCell;
        pkg_type[threadIdx.x] = 0;
    }
    if (g0 >= n_words) return;   // the same for the whole wavefront
    const int64_t wl = g0 + (lane & 15);
    const bool inl = wl < n_words;
    const uint64_t la = inl ? act[wl] : 0ull, lcw = inl ? core[wl] : 0ull, ln = inl ? neg[wl] : 0ull;
    uint32_t ea = (uint32_t)__popcll(la), ec = (uint32_t)__popcll(lcw);   // inclusive, then exclusive, counts
#pragma unroll
    for (int o = 1; o < 16; o <<= 1) {
        const uint32_t ta = __shfl_up(ea, o, 16), tc = __shfl_up(ec, o, 16);
        if ((lane & 15) >= o) {
            ea += ta;
            ec += tc;
        }
    }
    ea -= (uint32_t)__popcll(la);
    ec -= (uint32_t)__popcll(lcw);
    const uint32_t pa = off_act[grp], pc = off_core[grp];
    auto word = [](uint64_t v, int src) {
        return ((uint64_t)(uint32_t)__shfl((int)(v >> 32), src) << 32) | (uint32_t)__shfl((int)(uint32_t)v, src);
    };
#pragma unroll
    for (int step = 0; step < 4; ++step) {
        const int64_t w0 = g0 + 4 * step;
        if (w0 >= n_words) break;
        // the rank map entries of the four words' 32-cell halves (lanes 0..7)
        {
            const int k = (lane >> 1) & 3, hf = lane & 1;
            const int j = 4 * step + k;
            const uint64_t aj = word(la, j), nj = word(ln, j);
            const uint32_t before_j = (uint32_t)__shfl((int)ea, j);
            const int64_t w = w0 + k;
            if (lane < 8 && w < n_words) {
                const int64_t r = quot(w, W);
                const int half = (int)(w - r * W) * 2 + hf;
                if (half < W32) {
                    const uint32_t before = pa + before_j + (hf ? (uint32_t)__popc((uint32_t)aj) : 0u);
                    rank_map[r * W32 + half] = make_uint4((uint32_t)(hf ? aj >> 32 : aj),
                                                          (uint32_t)(hf ? nj >> 32 : nj), before, 0u);
                }
            }
        }
        const int k = lane >> 4, b0 = 4 * (lane & 15);
        const int j = 4 * step + k;
        const uint64_t ak = word(la, j), ck = word(lcw, j), nk = word(ln, j);
        uint32_t ra = pa + (uint32_t)__shfl((int)ea, j), rc = pc + (uint32_t)__shfl((int)ec, j);
        const int64_t w = w0 + k;
        if (w >= n_words) continue;
        const uint64_t below = (1ull << b0) - 1ull;
        ra += (uint32_t)__popcll(ak & below);
        rc += (uint32_t)__popcll(ck & below);
        const int64_t r = quot(w, W);
        const int x0 = (int)(w - r * W) * 64 + b0;
        if (x0 >= M) continue;
        uint32_t v[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int bit = b0 + i;
            const int64_t c = r * M + x0 + i;
            if ((ak >> bit) & 1ull) {
                const uint32_t id = 2u + ra++;
                v[i] = id;
                if (x0 + i < M) {
                    pkg_cell[id] = (uint32_t)c;
                    const bool is_core = (ck >> bit) & 1ull;
                    pkg_type[id] = is_core ? 1 : 2;
                    if (is_core) core_list[rc++] = id;
                }
            } else {
                v[i] = ((nk >> bit) & 1ull) ? sgrid::kFarNeg : sgrid::kFarPos;
            }
        }
        uint32_t *dst = cell_pkg + r * M + x0;
        if ((M & 3) == 0) {   // x0 and M multiples of 4: the four cells are in the row and 16-byte aligned
            *reinterpret_cast<uint4 *>(dst) = make_uint4(v[0], v[1], v[2], v[3]);
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (x0 + i < M) dst[i] = v[i];
        }
    }
}

// Sweep order: the activated packages listed in Morton (Z-curve) order of
// their coarse cells, so the packages one workgroup sweeps together are
// spatial neighbours and share their halo lines in the caches.  The codes run
// over the enclosing power-of-two cube; codes outside the grid are skipped.
// One lane per 64 consecutive codes, which cover a 4 x 4 x 4 box of cells:
// the box's activation is 16 four-bit pieces of the bitmap (one per (y, z)
// row, never straddling a word as the box is 4-aligned), gathered into one
// 64-bit mask, bit lx + 4 ly + 16 lz.  Most boxes of a narrow band are empty
// and cost 16 word reads; a box with activated cells is walked in Morton order
// and reads the package id of its activated cells only.
constexpr int kBoxesPerGroup = 64;   // boxes per count, and per workgroup of the scatter

// Bits 0, 3, 6, .. of v (at most ten of them) together.
__device__ __forceinline__ uint32_t every_third(uint32_t v) {
    v &= 0x09249249u;
    v = (v | (v >> 2)) & 0x030C30C3u;
    v = (v | (v >> 4)) & 0x0300F00Fu;
    v = (v | (v >> 8)) & 0x030000FFu;
    return (v | (v >> 16)) & 0x3FFu;
}

// The 64 boxes of a group, consecutive in code order, are a 4 x 4 x 4 block too; its
// origin in groups (at most seven bits per axis).
__device__ __forceinline__ void group_origin(uint32_t group, int &gx, int &gy, int &gz) {
    gx = (int)every_third(group);
    gy = (int)every_third(group >> 1);
    gz = (int)every_third(group >> 2);
}
// The place of a group's masks, -1 when it lies past the grid (of ng groups per axis).
// The masks hold the groups that meet the grid: in code order where these fill the
// enclosing cube of codes, else x fastest, for the cube has up to eight times as many
// (1 GiB of masks at 1025 cells per axis, where these take 0.14 GiB).  The same for the
// wavefront that asks.
__device__ __forceinline__ int64_t group_masks(uint32_t group, int64_t n_groups, int ng) {
    if ((int64_t)ng * ng * ng == n_groups) return (int64_t)group * kBoxesPerGroup;
    int gx, gy, gz;
    group_origin(group, gx, gy, gz);
    if (gx >= ng || gy >= ng || gz >= ng) return -1;
    return (gx + (int64_t)ng * (gy + (int64_t)ng * gz)) * kBoxesPerGroup;
}
// Place t in code order of a 4 x 4 x 4 block: x = t0 + 2 t3, y = t1 + 2 t4, z = t2 + 2 t5.
__device__ __forceinline__ void block_place(int t, int &x, int &y, int &z) {
    x = (t & 1) | ((t >> 2) & 2);
    y = ((t >> 1) & 1) | ((t >> 3) & 2);
    z = ((t >> 2) & 1) | ((t >> 4) & 2);
}

// Activation mask of the box at (bx, by, bz); 0 when it lies past the grid.
__device__ __forceinline__ uint64_t box_mask(const uint64_t *__restrict__ act, int M, int W, int bx, int by, int bz) {
    const int ox = 4 * bx, oy = 4 * by, oz = 4 * bz;
    if (ox >= M || oy >= M || oz >= M) return 0ull;
    const int nx = M - ox;
    const uint64_t xm = nx >= 4 ? 0xFull : ((1ull << nx) - 1ull);
    uint64_t m = 0;
#pragma unroll
    for (int lz = 0; lz < 4; ++lz)
#pragma unroll
        for (int ly = 0; ly < 4; ++ly) {
            const int y = oy + ly, z = oz + lz;
            const uint64_t w = (y < M && z < M) ? act[((int64_t)y + (int64_t)M * z) * W + (ox >> 6)] : 0ull;
            m |= ((w >> (ox & 63)) & xm) << (4 * (ly + 4 * lz));
        }
    return m;
}

// Every box's mask, and the activated cells of every 64 boxes.
__global__ __launch_bounds__(kTagBlock) void morton_count_kernel(const uint64_t *__restrict__ act, int M, int W,
                                                                 int64_t n_groups, int ng, uint64_t *__restrict__ mask,
                                                                 uint32_t *__restrict__ cnt) {
    const int lane = threadIdx.x & 63;
    const uint32_t group = blockIdx.x * (kTagBlock / 64) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (group >= n_groups) return;   // whole wavefronts
    const int64_t at = group_masks(group, n_groups, ng);
    if (at < 0) {
        if (lane == 0) cnt[group] = 0u;
        return;
    }
    int gx, gy, gz, bx, by, bz;
    group_origin(group, gx, gy, gz);
    block_place(lane, bx, by, bz);
    const uint64_t m = box_mask(act, M, W, 4 * gx + bx, 4 * gy + by, 4 * gz + bz);
    mask[at + lane] = m;
    uint32_t n = (uint32_t)__popcll(m);
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) n += __shfl_xor(n, d);
    if (lane == 0) cnt[group] = n;
}

// Writes the worklist and every package's position in it: a workgroup takes
// 64 boxes.  Every wavefront holds a box's mask and place in the list per lane;
// the wavefronts share the boxes with activated cells, each taking kBoxes in
// turn, one lane per code of a box (code order is lane order, so the ballot of
// the activated lanes gives each its place), with the map reads of kBoxes boxes
// in flight.  A lane that walked its own box, one dependent load and store after
// another, took 14 us on the smallest grids and 57 us at 512^3 cells; now 6.4 us
// with eight wavefronts per workgroup (8.1 with four) and 30 us with four (38
// with eight, which the many empty groups of a large grid only start and end).
constexpr int kBoxes = 4;
constexpr int kScatterWaves = 8;          // most of a workgroup
constexpr int kScatterFewGroups = 2048;   // eight per CU: below, more wavefronts for each

__global__ __launch_bounds__(64 * kScatterWaves) void morton_scatter_kernel(const uint32_t *__restrict__ cell_pkg,
                                                                            const uint64_t *__restrict__ mask, int M,
                                                                            int64_t n_groups, int ng,
                                                                            const uint32_t *__restrict__ off,
                                                                            uint32_t *__restrict__ work,
                                                                            uint32_t *__restrict__ wpos) {
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, n_waves = blockDim.x >> 6;
    const int64_t masks = group_masks(blockIdx.x, n_groups, ng);
    if (masks < 0) return;
    const uint64_t m = mask[masks + lane];
    uint64_t todo = __ballot(m != 0ull);
    if (!todo) return;   // the same for the whole workgroup
    const uint32_t n = (uint32_t)__popcll(m);
    const uint32_t pos = off[blockIdx.x] + wave_scan(n, lane) - n;
    int gx, gy, gz, bx, by, bz;
    group_origin(blockIdx.x, gx, gy, gz);
    block_place(lane, bx, by, bz);   // of a box in the group, and of a cell in its box
    const int lx = bx, ly = by, lz = bz, bit = lx + 4 * ly + 16 * lz;
    bx += 4 * gx;
    by += 4 * gy;
    bz += 4 * gz;
    for (int k = 0; k < wv * kBoxes && todo; ++k) todo &= todo - 1ull;
    while (todo) {   // the same for the whole wavefront
        uint32_t id[kBoxes], at[kBoxes];
        bool on[kBoxes];
#pragma unroll
        for (int k = 0; k < kBoxes; ++k) {
            const bool live = todo != 0ull;
            const int src = live ? __builtin_ctzll(todo) : 0;
            todo &= todo - 1ull;
            const uint64_t mk = ((uint64_t)(uint32_t)__shfl((int)(m >> 32), src) << 32) | (uint32_t)__shfl((int)m, src);
            on[k] = live && ((mk >> bit) & 1ull);
            const uint64_t placed = __ballot(on[k]);
            at[k] = (uint32_t)__shfl((int)pos, src) + (uint32_t)__popcll(placed & lanemask_lt());
            const int x = 4 * __shfl(bx, src) + lx, y = 4 * __shfl(by, src) + ly, z = 4 * __shfl(bz, src) + lz;
            id[k] = on[k] ? cell_pkg[x + (int64_t)M * (y + (int64_t)M * z)] : 0u;
        }
#pragma unroll
        for (int k = 0; k < kBoxes; ++k)
            if (on[k]) {
                work[at[k]] = id[k];
                wpos[id[k]] = at[k];
            }
        for (int k = 0; k < (n_waves - 1) * kBoxes && todo; ++k) todo &= todo - 1ull;
    }
}

// Face rows in worklist order, three times: wface holds the six face
// neighbours' package ids and the package's own id; sface marks a neighbour
// in the same group of kGroup entries by its slot in the group (flagged with
// kLocal); mface gives the neighbours' rows in the worklist-ordered copy of a
// field (row 2 + e holds the package at worklist position e, rows 0 and 1 the
// far fields), then the own id.  Eight lanes per entry (one per row slot),
// each taking kFacePkgs consecutive entries whose loads are issued together.
constexpr int kFacePkgs = 4;

__global__ __launch_bounds__(256) void sweep_face_kernel(const uint32_t *__restrict__ work,
                                                         const uint32_t *__restrict__ face,
                                                         const uint32_t *__restrict__ wpos, int64_t P,
                                                         uint32_t *__restrict__ wface, uint32_t *__restrict__ sface,
                                                         uint32_t *__restrict__ mface) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int f = (int)(t & 7);
    const int64_t e0 = (t >> 3) * kFacePkgs;
    if (e0 >= P) return;
    uint32_t p[kFacePkgs], n[kFacePkgs], en[kFacePkgs];
#pragma unroll
    for (int g = 0; g < kFacePkgs; ++g) p[g] = work[e0 + g < P ? e0 + g : P - 1];
#pragma unroll
    for (int g = 0; g < kFacePkgs; ++g) n[g] = f < 6 ? face[(int64_t)p[g] * 8 + f] : 0u;
#pragma unroll
    for (int g = 0; g < kFacePkgs; ++g) en[g] = wpos[n[g]];   // n < 2: a far-field row's entry, not used
#pragma unroll
    for (int g = 0; g < kFacePkgs; ++g) {
        const int64_t e = e0 + g;
        if (e >= P) break;
        uint32_t v, w, m;
        if (f < 6) {
            v = w = n[g];
            m = n[g] < 2u ? n[g] : 2u + en[g];
            if (n[g] >= 2u && (int64_t)en[g] / sgrid::kGroup == e / sgrid::kGroup)
                v = sgrid::kLocal | (en[g] % sgrid::kGroup);
        } else {
            v = w = m = f == 6 ? p[g] : 0u;
        }
        wface[e * 8 + f] = w;
        sface[e * 8 + f] = v;
        mface[e * 8 + f] = m;
    }
}

// Neighbour table and face rows: nine lanes per package, one per row (dy, dz)
// of the 27-entry neighbourhood, whose three cells are adjacent in the map (one
// 12-byte load) and whose three slots are adjacent in the table (one 12-byte
// store); seven packages per wavefront and step, kNbrPkgs steps with their loads
// issued together.  Bound by its scattered map reads and by 140 bytes of table
// per package: in the torus's chain of layers up to 2048^3 points (three builds) a
// lane per slot took 72 us a build on average, this takes 47.
constexpr int kNbrPkgs = 4;                  // steps of a wavefront
constexpr int kNbrWave = 7;                  // packages per wavefront and step
constexpr int kNbrBlock = 4 * kNbrWave * kNbrPkgs;

struct Cells3 {
    uint32_t v[3];
};

template <bool WIDE>   // M >= 3: a row's three cells as one load
__global__ __launch_bounds__(256) void nbr_kernel(const uint32_t *__restrict__ cell_pkg,
                                                  const uint32_t *__restrict__ pkg_cell, int M,
                                                  int64_t n_total, uint32_t *__restrict__ nbr,
                                                  uint32_t *__restrict__ face) {
    const int lane = threadIdx.x & 63;
    if (lane >= 9 * kNbrWave) return;
    const int64_t p0 = (int64_t)blockIdx.x * kNbrBlock + (int64_t)(threadIdx.x >> 6) * (kNbrWave * kNbrPkgs) + lane / 9;
    const int row = lane % 9;
    const int dy = row % 3 - 1, dz = row / 3 - 1;
    const uint32_t um = (uint32_t)M;
    uint32_t c[kNbrPkgs];
#pragma unroll
    for (int g = 0; g < kNbrPkgs; ++g) {
        const int64_t p = p0 + kNbrWave * g;
        c[g] = (p >= 2 && p < n_total) ? pkg_cell[p] : 0u;
    }
    Cells3 m[kNbrPkgs];
    int x[kNbrPkgs];
    bool in[kNbrPkgs];   // the row lies in the grid
#pragma unroll
    for (int g = 0; g < kNbrPkgs; ++g) {
        const uint32_t cyz = c[g] / um;
        x[g] = (int)(c[g] - cyz * um);
        const int y = (int)(cyz % um) + dy, z = (int)(cyz / um) + dz;
        in[g] = y >= 0 && z >= 0 && y < M && z < M;
        const int64_t base = in[g] ? (int64_t)M * y + (int64_t)M * M * z : 0;
        if (WIDE) {   // three cells from x - 1, moved into the row at its ends
            m[g] = *reinterpret_cast<const Cells3 *>(cell_pkg + base + min(max(x[g] - 1, 0), M - 3));
        } else {
#pragma unroll
            for (int k = 0; k < 3; ++k) m[g].v[k] = cell_pkg[base + min(max(x[g] - 1 + k, 0), M - 1)];
        }
    }
#pragma unroll
    for (int g = 0; g < kNbrPkgs; ++g) {
        const int64_t p = p0 + kNbrWave * g;
        if (p >= n_total) break;
        uint32_t v[3];
        if (p < 2) {
            v[0] = v[1] = v[2] = (uint32_t)p;   // the far-field packages neighbour themselves
        } else {
            const bool first = x[g] == 0, last = x[g] == M - 1;
            const Cells3 &u = m[g];
            if (WIDE) {
                v[0] = first ? sgrid::kFarPos : (last ? u.v[1] : u.v[0]);
                v[1] = first ? u.v[0] : (last ? u.v[2] : u.v[1]);
                v[2] = last ? sgrid::kFarPos : (first ? u.v[1] : u.v[2]);
            } else {
                v[0] = first ? sgrid::kFarPos : u.v[0];
                v[1] = u.v[1];
                v[2] = last ? sgrid::kFarPos : u.v[2];
            }
            if (!in[g]) v[0] = v[1] = v[2] = sgrid::kFarPos;
        }
        uint32_t *o = nbr + p * 27 + 3 * row;
        o[0] = v[0];
        o[1] = v[1];
        o[2] = v[2];
        // face row: -x, +x, -y, +y, -z, +z, then the package itself twice
        uint32_t *f = face + p * 8;
        if (row == 4) {
            *reinterpret_cast<uint2 *>(f) = make_uint2(v[0], v[2]);
            *reinterpret_cast<uint2 *>(f + 6) = make_uint2(v[1], v[1]);
        } else if (row == 3) {
            f[2] = v[1];
        } else if (row == 5) {
            f[3] = v[1];
        } else if (row == 1) {
            f[4] = v[1];
        } else if (row == 7) {
            f[5] = v[1];
        }
    }
}

// Multi-resolution layers (Sec. 7, Sec. 7.1 step 1): the layer of doubled
// resolution evaluates distances only in the cells its parent layer's core
// cells cover.  core_slot[id] = position of core package `id` in the parent's
// core list (the rows of the caller's child distances).
__global__ __launch_bounds__(256) void core_slot_kernel(const uint32_t *__restrict__ core_list, int64_t n_core,
                                                        uint32_t *__restrict__ core_slot) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n_core) core_slot[core_list[i]] = (uint32_t)i;
}

// Core and sign bits of the refined layer.  A fine cell under a core parent
// takes its own distance (child b = bx + 2 by + 4 bz of the parent's row); any
// other cell takes the parent's sign from the parent layer's rank map and is
// not core (the parent is not core, so its distance is at least the parent
// cell size, twice the fine one).  The 64 cells of a word lie under the 32
// parents of one rank-map entry: a lane takes a word, and most of a narrow
// band's words have no activated parent, so their bits follow from the entry
// alone.  The others are listed in LDS, and each wavefront takes kRefineWords
// listed words at a time, a lane per cell, with the three dependent loads
// (package type, core slot, distance) of all of them in flight.  One wavefront
// per word, empty or not, took 340 us at 512^3 cells; this takes 45 us.
constexpr int kRefineWords = 4;

// Bit i of v at bits 2i and 2i + 1.
__device__ __forceinline__ uint64_t doubled_bits(uint32_t v) {
    uint64_t x = v;
    x = (x | (x << 16)) & 0x0000FFFF0000FFFFull;
    x = (x | (x << 8)) & 0x00FF00FF00FF00FFull;
    x = (x | (x << 4)) & 0x0F0F0F0F0F0F0F0Full;
    x = (x | (x << 2)) & 0x3333333333333333ull;
    x = (x | (x << 1)) & 0x5555555555555555ull;
    return x | (x << 1);
}

__global__ __launch_bounds__(256) void refine_bits_kernel(const uint4 *__restrict__ rank_map, int W32c,
                                                          const uint8_t *__restrict__ pkg_type,
                                                          const uint32_t *__restrict__ core_slot,
                                                          const float *__restrict__ child_d, int Mc, int W,
                                                          int64_t n_words, double lc, uint64_t *__restrict__ core,
                                                          uint64_t *__restrict__ neg) {
    __shared__ uint4 s_entry[256];
    __shared__ uint32_t s_word[256];   // listed: word within the workgroup, parity of y and z
    __shared__ uint32_t s_n;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int Mf = 2 * Mc;
    const int64_t w0 = (int64_t)blockIdx.x * 256, w = w0 + threadIdx.x;
    if (threadIdx.x == 0) s_n = 0u;
    __syncthreads();
    if (w < n_words) {
        const int64_t r = quot(w, W);
        const int i = (int)(w - r * W);
        const int64_t rz = quot(r, Mf);
        const int y = (int)(r - rz * Mf), z = (int)rz;
        const uint4 e = rank_map[((int64_t)(y >> 1) + (int64_t)Mc * (z >> 1)) * W32c + i];
        if (e.x == 0u) {
            const int left = Mf - 64 * i;
            core[w] = 0ull;
            neg[w] = doubled_bits(e.y) & (left >= 64 ? ~0ull : (1ull << left) - 1ull);
        } else {
            const uint32_t at = atomicAdd(&s_n, 1u);
            s_entry[at] = make_uint4(e.x, e.y, e.z, (uint32_t)min(64, Mf - 64 * i));
            s_word[at] = threadIdx.x | ((uint32_t)(y & 1) << 8) | ((uint32_t)(z & 1) << 9);
        }
    }
    __syncthreads();
    const uint32_t n = s_n;
    const uint32_t bit = 1u << (lane >> 1);
    for (uint32_t k0 = wv * kRefineWords; k0 < n; k0 += 4 * kRefineWords) {   // the same for a wavefront
        uint4 e[kRefineWords];
        uint32_t word[kRefineWords], id[kRefineWords], slot[kRefineWords];
        uint8_t type[kRefineWords];
        float v[kRefineWords];
#pragma unroll
        for (int k = 0; k < kRefineWords; ++k) {
            const uint32_t at = k0 + k < n ? k0 + k : n - 1;
            e[k] = s_entry[at];
            word[k] = s_word[at];
            // 2 + rank of an activated parent; else package 0, a far field
            id[k] = (e[k].x & bit) ? 2u + e[k].z + (uint32_t)__popc(e[k].x & (bit - 1u)) : 0u;
        }
#pragma unroll
        for (int k = 0; k < kRefineWords; ++k) type[k] = pkg_type[id[k]];
#pragma unroll
        for (int k = 0; k < kRefineWords; ++k) slot[k] = type[k] == 1 ? core_slot[id[k]] : 0u;
#pragma unroll
        for (int k = 0; k < kRefineWords; ++k) {
            const uint32_t b = (lane & 1) + 2 * ((word[k] >> 8) & 1u) + 4 * ((word[k] >> 9) & 1u);
            v[k] = type[k] == 1 ? child_d[(int64_t)slot[k] * 8 + b] : 0.f;
        }
#pragma unroll
        for (int k = 0; k < kRefineWords; ++k) {
            const bool in = lane < (int)e[k].w, own = in && type[k] == 1;
            const uint64_t bc = __ballot(own && fabs((double)v[k]) < lc);
            const uint64_t bn = __ballot(in && (own ? v[k] < 0.0f : (e[k].y & bit) != 0u));
            if (lane == 0 && k0 + k < n) {
                core[w0 + (word[k] & 255u)] = bc;
                neg[w0 + (word[k] & 255u)] = bn;
            }
        }
    }
}

void free_grid(sgrid_grid *g) {
    if (!g) return;
    void *ptrs[] = {g->cell_pkg, g->pkg_cell, g->pkg_type, g->nbr,  g->face, g->core_list,
                    g->workspace, g->rank_map, g->work, g->sface, g->wface,     g->wpos,
                    g->mface};
    for (void *p : ptrs) sgrid::dev_free(p);
    delete g;
}

// Pinned host words for the one readback of a build (per thread): P, the core
// packages and a flag, written by the scan kernel itself.
uint64_t *pinned_totals() {
    static thread_local uint64_t *buf = nullptr;
    if (!buf && hipHostMalloc((void **)&buf, 3 * sizeof(uint64_t),
                              hipHostMallocCoherent | hipHostMallocMapped | hipHostMallocPortable) != hipSuccess) {
        (void)hipGetLastError();
        buf = nullptr;
    }
    return buf;
}

// Waits for the flag of `host`.  The word arrives while later kernels of the
// stream run, which a copy and a stream synchronisation would wait for (and
// cost about 10 us more).  When the flag stays away the stream itself is
// asked, so a failed launch or a stream being captured ends the wait with the
// runtime's error.  The thread looks for as long as the stream's earlier work
// takes, as in the runtime's own synchronisation (behind 429 ms of products either
// takes 429 ms of processor time).
hipError_t wait_totals(uint64_t *host, hipStream_t st) {
    for (int spin = 0;; ++spin) {
        if (__atomic_load_n(host + 2, __ATOMIC_ACQUIRE) != 0) return hipSuccess;
        __builtin_ia32_pause();
        if ((spin & 16383) == 16383) {
            const hipError_t e = hipStreamQuery(st);
            if (e != hipErrorNotReady) {
                const hipError_t f = e == hipSuccess ? hipStreamSynchronize(st) : e;
                if (f != hipSuccess) return f;
                return __atomic_load_n(host + 2, __ATOMIC_ACQUIRE) != 0 ? hipSuccess : hipErrorUnknown;
            }
            (void)hipGetLastError();
        }
    }
}

}  // namespace

#define SG_ALLOC(ptr, bytes, what)                                                  \
    do {                                                                            \
        sgrid_status _s = sgrid::dev_alloc((void **)&(ptr), (size_t)(bytes), what); \
        if (_s != SGRID_OK) { free_grid(g); return _s; }                            \
    } while (0)

#define SG_HIP_OR_FREE(expr)                                                          \
    do {                                                                              \
        hipError_t _e = (expr);                                                       \
        if (_e != hipSuccess) {                                                       \
            sgrid::set_error("%s failed: %s", #expr, hipGetErrorString(_e));          \
            free_grid(g);                                                             \
            return SGRID_E_HIP;                                                       \
        }                                                                             \
    } while (0)

namespace {

// A new grid of M^3 cells at spacing h with its build workspace: three
// bitmaps (core, negative sign, activated), the per-group counts and the scan's
// block sums; the masks, counts and block sums of the worklist's boxes.
struct BuildWs {
    int64_t W, n_words, n_groups;
    int64_t n_box_groups;   // of the enclosing cube of codes
    int ng;                 // box groups that meet the grid per axis
    uint64_t *core_bits, *neg_bits, *act_bits, *box_masks;
    uint32_t *ca, *cc, *part, *box_counts, *box_part;
};

sgrid_status new_grid(int64_t M, double h, sgrid_grid **out, BuildWs &ws) {
    const int64_t n_cells = M * M * M;
    if (n_cells + 2 > (int64_t)0xFFFFFFFFll || (n_cells + 2) * 64 > ((int64_t)1 << 40)) {
        sgrid::set_error("n_coarse = %lld gives %lld coarse cells, beyond the 32-bit package ids",
                         (long long)M, (long long)n_cells);
        return SGRID_E_CAPACITY;
    }
    sgrid_grid *g = new sgrid_grid();
    g->M = (int32_t)M;
    g->h = h;
    SG_HIP_OR_FREE(hipGetDevice(&g->device));
    ws.W = (M + 63) / 64;
    ws.n_words = M * M * ws.W;
    ws.n_groups = (ws.n_words + 15) / 16;
    const int64_t n_sblocks = (ws.n_groups + kScanBlock - 1) / kScanBlock;
    const size_t ws_bits = ((size_t)ws.n_words * 8 + 255) / 256 * 256;
    const size_t ws_counts = ((size_t)ws.n_groups * 4 + 255) / 256 * 256;
    const size_t ws_part = ((size_t)n_sblocks * 8 + 255) / 256 * 256;
    ws.ng = (int)((M + 15) / 16);
    int64_t cube = 1;   // groups per axis of the enclosing cube of codes
    while (cube < ws.ng) cube *= 2;
    ws.n_box_groups = cube * cube * cube;
    const size_t ws_masks = (size_t)ws.ng * ws.ng * ws.ng * kBoxesPerGroup * 8;
    const size_t ws_boxes = ((size_t)ws.n_box_groups * 4 + 255) / 256 * 256;
    const size_t ws_box_part = (size_t)((ws.n_box_groups + kScanBlock - 1) / kScanBlock) * 4;
    SG_ALLOC(g->workspace, 3 * ws_bits + 2 * ws_counts + ws_part + ws_masks + ws_boxes + ws_box_part, "build workspace");
    ws.core_bits = (uint64_t *)g->workspace;
    ws.neg_bits = (uint64_t *)((uint8_t *)ws.core_bits + ws_bits);
    ws.act_bits = (uint64_t *)((uint8_t *)ws.neg_bits + ws_bits);
    ws.ca = (uint32_t *)((uint8_t *)ws.act_bits + ws_bits);
    ws.cc = (uint32_t *)((uint8_t *)ws.ca + ws_counts);
    ws.part = (uint32_t *)((uint8_t *)ws.cc + ws_counts);
    ws.box_masks = (uint64_t *)((uint8_t *)ws.part + ws_part);
    ws.box_counts = (uint32_t *)((uint8_t *)ws.box_masks + ws_masks);
    ws.box_part = (uint32_t *)((uint8_t *)ws.box_counts + ws_boxes);
    SG_ALLOC(g->cell_pkg, n_cells * 4, "cell_pkg");
    *out = g;
    return SGRID_OK;
}

// Everything after the core and sign bitmaps: dilation, numbering (one host
// synchronisation learns P), tables, neighbours, the Morton worklist and the
// worklist face rows.
#define SG_TRY_ALLOC(ptr, bytes, what)                                              \
    do {                                                                            \
        sgrid_status _s = sgrid::dev_alloc((void **)&(ptr), (size_t)(bytes), what); \
        if (_s != SGRID_OK) return _s;                                              \
    } while (0)

sgrid_status fill_grid(sgrid_grid *g, const BuildWs &ws, hipStream_t st) {
    const int64_t M = g->M, W = ws.W, n_words = ws.n_words, n_groups = ws.n_groups;
    uint64_t *core_bits = ws.core_bits, *neg_bits = ws.neg_bits, *act_bits = ws.act_bits;
    uint64_t *host = pinned_totals();
    if (host == nullptr) {
        sgrid::set_error("pinned host words could not be allocated");
        return SGRID_E_NOMEM;
    }
    __atomic_store_n(host + 2, 0ull, __ATOMIC_RELEASE);
    uint32_t *ca = ws.ca, *cc = ws.cc, *part = ws.part;
    hipLaunchKernelGGL(dilate_kernel, dim3((unsigned)((n_words + 255) / 256)), dim3(256), 0, st, core_bits, (int)M,
                       (int)W, n_words, act_bits, ca, cc);
    SG_CHECK_HIP(hipGetLastError());
    scan_counts(Counts<2>{{ca, cc}}, n_groups, part, host, st);
    SG_CHECK_HIP(hipGetLastError());
    // the worklist's boxes need no package ids: counted while the host waits
    hipLaunchKernelGGL(morton_count_kernel, dim3((unsigned)((ws.n_box_groups * 64 + kTagBlock - 1) / kTagBlock)),
                       dim3(kTagBlock), 0, st, act_bits, (int)M, (int)W, ws.n_box_groups, ws.ng, ws.box_masks, ws.box_counts);
    SG_CHECK_HIP(hipGetLastError());
    scan_counts(Counts<1>{{ws.box_counts}}, ws.n_box_groups, ws.box_part, nullptr, st);
    SG_CHECK_HIP(hipGetLastError());
    SG_CHECK_HIP(wait_totals(host, st));
    g->P = (int64_t)host[0];
    g->n_core = (int64_t)host[1];
    const int64_t nt = g->total();
    SG_TRY_ALLOC(g->pkg_cell, nt * 4, "pkg_cell");
    SG_TRY_ALLOC(g->pkg_type, nt, "pkg_type");
    SG_TRY_ALLOC(g->nbr, nt * 27 * 4, "pkg_nbr");
    SG_TRY_ALLOC(g->face, nt * 8 * 4, "face table");
    SG_TRY_ALLOC(g->core_list, (g->n_core > 0 ? g->n_core : 1) * 4, "core_list");
    g->W32 = (int32_t)((M + 31) / 32);
    SG_TRY_ALLOC(g->rank_map, M * M * g->W32 * 16, "rank map");
    hipLaunchKernelGGL(scatter_kernel, dim3((unsigned)((n_groups + 3) / 4)), dim3(256), 0, st, act_bits, core_bits,
                       neg_bits,
                       (int)M, (int)W, n_words, ca, cc, g->cell_pkg, g->pkg_cell, g->pkg_type, g->core_list,
                       g->rank_map, g->W32);
    SG_CHECK_HIP(hipGetLastError());
    hipLaunchKernelGGL(M >= 3 ? nbr_kernel<true> : nbr_kernel<false>,
                       dim3((unsigned)((nt + kNbrBlock - 1) / kNbrBlock)), dim3(256), 0, st, g->cell_pkg,
                       g->pkg_cell, (int)M, nt, g->nbr, g->face);
    SG_CHECK_HIP(hipGetLastError());
    SG_TRY_ALLOC(g->work, (g->P > 0 ? g->P : 1) * 4, "sweep worklist");
    SG_TRY_ALLOC(g->wpos, nt * 4, "worklist positions");
    hipLaunchKernelGGL(morton_scatter_kernel, dim3((unsigned)ws.n_box_groups),
                       dim3(ws.n_box_groups < kScatterFewGroups ? 64 * kScatterWaves : 32 * kScatterWaves), 0, st,
                       g->cell_pkg, ws.box_masks, (int)M, ws.n_box_groups, ws.ng, ws.box_counts, g->work, g->wpos);
    SG_CHECK_HIP(hipGetLastError());
    // group-relative face rows of the sweep order, through the position of
    // every package in the worklist (kept with the handle)
    {
        SG_TRY_ALLOC(g->sface, (g->P > 0 ? g->P : 1) * 32, "sweep face table");
        SG_TRY_ALLOC(g->wface, (g->P > 0 ? g->P : 1) * 32, "worklist face table");
        SG_TRY_ALLOC(g->mface, (g->P > 0 ? g->P : 1) * 32, "worklist-ordered face table");
        if (g->P > 0) {
            const int64_t groups = (g->P + kFacePkgs - 1) / kFacePkgs;
            hipLaunchKernelGGL(sweep_face_kernel, dim3((unsigned)((groups * 8 + 255) / 256)), dim3(256), 0, st,
                               g->work, g->face, g->wpos, g->P, g->wface, g->sface, g->mface);
            SG_CHECK_HIP(hipGetLastError());
        }
    }
    return SGRID_OK;
}

// The same; on failure the grid is freed once its queued kernels have ended.
sgrid_status finish_grid(sgrid_grid *g, const BuildWs &ws, hipStream_t st) {
    const sgrid_status s = fill_grid(g, ws, st);
    if (s != SGRID_OK) {
        (void)hipStreamSynchronize(st);
        free_grid(g);
    }
    return s;
}

}  // namespace

extern "C" sgrid_status sgrid_build_packages(const sgrid_desc *desc, const float *coarse_sdf, void *stream,
                                             sgrid_grid **out) {
    sgrid::clear_error();
    SG_REQUIRE(out != nullptr, "out is NULL");
    *out = nullptr;
    SG_REQUIRE(desc != nullptr, "desc is NULL");
    SG_REQUIRE(coarse_sdf != nullptr, "coarse_sdf is NULL");
    SG_REQUIRE(sg_aligned(coarse_sdf, 4), "coarse_sdf is not 4-byte aligned");
    SG_REQUIRE(desc->n_coarse >= 1, "n_coarse must be >= 1 (got %d)", desc->n_coarse);
    SG_REQUIRE(desc->h > 0.0 && desc->h < 1e30, "h must be positive and finite");
    const int64_t M = desc->n_coarse;
    hipStream_t st = sg_stream(stream);
    sgrid_grid *g = nullptr;
    BuildWs ws;
    sgrid_status s = new_grid(M, desc->h, &g, ws);
    if (s != SGRID_OK) return s;
    const double lc = 4.0 * desc->h;
    hipLaunchKernelGGL(bits_kernel, dim3((unsigned)((ws.n_words + 4 * kBitsWords - 1) / (4 * kBitsWords))), dim3(256), 0,
                       st, coarse_sdf, (int)M,
                       (int)ws.W, ws.n_words, lc, ws.core_bits, ws.neg_bits);
    SG_HIP_OR_FREE(hipGetLastError());
    s = finish_grid(g, ws, st);
    if (s != SGRID_OK) return s;
    *out = g;
    return SGRID_OK;
}

extern "C" sgrid_status sgrid_build_packages_refined(const sgrid_grid *coarse, const float *child_sdf, void *stream,
                                                     sgrid_grid **out) {
    sgrid::clear_error();
    SG_REQUIRE(out != nullptr, "out is NULL");
    *out = nullptr;
    SG_REQUIRE(coarse != nullptr, "coarse grid is NULL");
    SG_REQUIRE(child_sdf != nullptr || coarse->n_core == 0, "child_sdf is NULL");
    SG_REQUIRE(child_sdf == nullptr || sg_aligned(child_sdf, 4), "child_sdf is not 4-byte aligned");
    SG_REQUIRE(coarse->M <= (1 << 29), "the coarse grid is too large to refine");
    const int64_t M = 2 * (int64_t)coarse->M;
    hipStream_t st = sg_stream(stream);
    sgrid_grid *g = nullptr;
    BuildWs ws;
    sgrid_status s = new_grid(M, 0.5 * coarse->h, &g, ws);
    if (s != SGRID_OK) return s;
    // the parent's core slots live in the new cell_pkg until it is written
    static_assert(sizeof(uint32_t) == 4, "");
    uint32_t *core_slot = g->cell_pkg;   // M^3 >= 8 (P_parent + 2) entries
    if (coarse->n_core > 0) {
        hipLaunchKernelGGL(core_slot_kernel, dim3((unsigned)((coarse->n_core + 255) / 256)), dim3(256), 0, st,
                           coarse->core_list, coarse->n_core, core_slot);
        SG_HIP_OR_FREE(hipGetLastError());
    }
    const double lc = 4.0 * g->h;
    hipLaunchKernelGGL(refine_bits_kernel, dim3((unsigned)((ws.n_words + 255) / 256)), dim3(256), 0, st, coarse->rank_map,
                       coarse->W32, coarse->pkg_type, core_slot, child_sdf, coarse->M, (int)ws.W, ws.n_words, lc,
                       ws.core_bits, ws.neg_bits);
    SG_HIP_OR_FREE(hipGetLastError());
    s = finish_grid(g, ws, st);
    if (s != SGRID_OK) return s;
    *out = g;
    return SGRID_OK;
}

extern "C" sgrid_status sgrid_get_info(const sgrid_grid *g, sgrid_info *out) {
    sgrid::clear_error();
    SG_REQUIRE(g != nullptr && out != nullptr, "NULL argument");
    out->n_coarse = g->M;
    out->h = g->h;
    out->n_packages = g->P;
    out->n_core = g->n_core;
    out->cell_pkg = g->cell_pkg;
    out->pkg_cell = g->pkg_cell;
    out->pkg_type = g->pkg_type;
    out->pkg_nbr = g->nbr;
    out->core_list = g->core_list;
    out->sweep_order = g->work;
    out->rank_map = (const uint32_t *)g->rank_map;
    out->rank_row = g->W32;
    return SGRID_OK;
}

extern "C" sgrid_status sgrid_destroy(sgrid_grid *g) {
    sgrid::clear_error();
    if (!g) return SGRID_OK;
    hipError_t e = hipDeviceSynchronize();
    free_grid(g);
    if (e != hipSuccess) {
        sgrid::set_error("hipDeviceSynchronize before destroy failed: %s", hipGetErrorString(e));
        return SGRID_E_HIP;
    }
    return SGRID_OK;
}
