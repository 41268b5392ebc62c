// Consistency (sign) correction of a layer's distances (Sec. 7.2), the coarse
// step on the mesh cells.  Where an inside/outside test is unreliable (a
// leaky triangle mesh), only the signs of cells near the surface are used as
// given: the core cells, |d| < lc.  Every other cell gets its sign by
// diffusion from them: in rounds of simultaneous updates, a cell without a
// sign takes one when a face neighbour has one, positive if any such
// neighbour is positive, else negative, until a round changes nothing.
//
// The state lives in two bitmaps of 64 cells per word along x (W = ceil(M /
// 64) words per row): positive and negative cells, interleaved, a cell
// without a sign in neither.  Word (b, y, z) is at (z W + b) M + y, so that
// lanes along y read consecutive 16-byte pairs.
//
// A round moves a sign by one cell, and a large grid takes hundreds of them;
// one launch per round was bound by launches, not by its few megabytes of
// bits.  A launch therefore makes kSignRounds rounds on tiles held in
// registers, with a halo of as many cells (sign_rounds_kernel).  The flags of
// every round are kept, so the round count is that of single rounds; a launch
// whose predecessor's last round changed nothing returns at once, and the
// host reads the flags of a batch of launches at a time.
#include "common.hpp"

#include <mutex>
#include <vector>

namespace {

constexpr int kSignRounds = 16;                       // rounds per launch = halo of a tile
constexpr int kSignOwn = 32;                          // rows a tile writes, in y and in z
constexpr int kSignTile = kSignOwn + 2 * kSignRounds; // rows it holds: one per lane in y
constexpr int kSignStrips = 4;                        // z rows per wavefront
constexpr int kSignWaves = kSignTile / kSignStrips;
constexpr int kSignBatch = 8;                         // launches per check of the host
constexpr int kSignLoads = 8;                         // rows per wavefront of the passes over d
static_assert(kSignTile == 64 && kSignRounds == 16, "a lane per y row, 16 halo bits on either side of a word");

// Pinned flag buffers: kept after a call for the next one (at most
// kPinnedKept of them), one per call in flight.
constexpr size_t kPinnedKept = 4;
constexpr int kFlags = kSignBatch * kSignRounds;
std::mutex g_pinned_mu;
std::vector<uint32_t *> g_pinned;

uint32_t *pinned_flags() {
    {
        std::lock_guard<std::mutex> lk(g_pinned_mu);
        if (!g_pinned.empty()) {
            uint32_t *p = g_pinned.back();
            g_pinned.pop_back();
            return p;
        }
    }
    uint32_t *p = nullptr;
    if (hipHostMalloc((void **)&p, kFlags * sizeof(uint32_t), hipHostMallocPortable) != hipSuccess) {
        (void)hipGetLastError();
        return nullptr;
    }
    return p;
}

void pinned_release(uint32_t *p) {
    {
        std::lock_guard<std::mutex> lk(g_pinned_mu);
        if (g_pinned.size() < kPinnedKept) {
            g_pinned.push_back(p);
            return;
        }
    }
    (void)hipHostFree(p);
}

// The rows of one wavefront of the passes over d: word b of the rows y0 ..
// y0 + kSignLoads - 1 of slice z.
__device__ __forceinline__ bool sign_rows(int M, int W, int64_t n_waves, int &b, int &y0, int64_t &z) {
    const int64_t w = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (w >= n_waves) return false;   // whole wavefronts
    const int groups = (M + kSignLoads - 1) / kSignLoads;
    const int64_t q = w / W;
    b = (int)(w - q * W);
    z = q / groups;
    y0 = (int)(q - z * groups) * kSignLoads;
    return true;
}

// HBM-bound: 4 B of d per cell.  Eight rows per wavefront with their loads
// issued together (one row and one 64-bit division per wavefront before: 37 us
// at 256^3, 3.6 times the time of its bytes).
__global__ __launch_bounds__(256) void sign_init_kernel(const float *__restrict__ d, int M, int W, int64_t n_waves,
                                                        double lc, ulonglong2 *__restrict__ state) {
    int b, y0;
    int64_t z;
    if (!sign_rows(M, W, n_waves, b, y0, z)) return;
    const int lane = threadIdx.x & 63;
    const int x = b * 64 + lane;
    float v[kSignLoads];
#pragma unroll
    for (int i = 0; i < kSignLoads; ++i) {
        const int y = min(y0 + i, M - 1);
        v[i] = d[(z * M + y) * M + min(x, M - 1)];
    }
    ulonglong2 mine = make_ulonglong2(0, 0);
#pragma unroll
    for (int i = 0; i < kSignLoads; ++i) {
        const bool core = x < M && fabs((double)v[i]) < lc;
        const uint64_t n = __ballot(core && v[i] < 0.0f), p = __ballot(core && !(v[i] < 0.0f));
        if (lane == i) mine = make_ulonglong2(p, n);
    }
    if (lane < kSignLoads && y0 + lane < M) state[(z * W + b) * M + y0 + lane] = mine;
}

// The value of the lane below (above) in y; 0 past the ends of the tile.
__device__ __forceinline__ uint32_t lane_below(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x138 /* wave_shr:1 */, 0xF, 0xF, true);
}
__device__ __forceinline__ uint32_t lane_above(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x130 /* wave_shl:1 */, 0xF, 0xF, true);
}

// One row of a tile: 16 bits of the word below, a word, 16 bits of the word
// above (bits 0..95), as positive, negative and undecided cells.
struct SignStrip {
    uint32_t p[3], n[3], u[3];
};

// kSignRounds rounds on the tile of one word column b and kSignOwn x kSignOwn
// rows.  The tile and a halo of kSignRounds cells on every side (96 x 64 x 64
// cells) stay in registers: lane = y row, each wavefront kSignStrips rows of
// z; x neighbours are bit shifts, y neighbours lane shifts, z neighbours the
// wavefront's other rows, and only its first and last row pass through LDS.
// After k rounds every cell at least k from the tile's edge is right, so the
// tile's own cells are; rows nearer the edge are skipped as the rounds go on.
// A tile whose own cells are all decided, or which holds no decided cell, or
// in which a round changes nothing, ends early.  Bound by its integer
// instructions (about 60 per row of 96 cells and round).  At 256^3 cells and
// 213 rounds they took 1.6 ms with one launch a round and
// 0.46 ms in 14 launches of this kernel (0.63 ms with eight z rows per wavefront
// instead of four: two wavefronts per SIMD did not cover the barriers).
__global__ __launch_bounds__(64 * kSignWaves) void sign_rounds_kernel(const ulonglong2 *__restrict__ in, int M, int W,
                                                                      int tiles, const uint32_t *__restrict__ prev,
                                                                      ulonglong2 *__restrict__ out,
                                                                      uint32_t *__restrict__ changed) {
    __shared__ uint32_t edge[2][kSignWaves][2][6][64];
    __shared__ uint32_t moved[3];
    if (prev != nullptr && *prev == 0u) return;
    const int b = (int)(blockIdx.x % (unsigned)W);
    const int t = (int)(blockIdx.x / (unsigned)W);
    const int ty = t % tiles, tz = t / tiles;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int y = ty * kSignOwn - kSignRounds + lane;
    const int z0 = tz * kSignOwn - kSignRounds + wave * kSignStrips;
    if (threadIdx.x < 3) moved[threadIdx.x] = 0u;
    uint32_t valid[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        // bits lo .. hi - 1 of this third lie in the grid
        const int x0 = 64 * b - kSignRounds + 32 * k;
        const int lo = x0 < 0 ? min(-x0, 32) : 0, hi = max(0, min(32, M - x0));
        const uint32_t below_hi = hi >= 32 ? ~0u : ((1u << hi) - 1u);
        valid[k] = lo >= 32 ? 0u : below_hi & (~0u << lo);
    }
    const bool own_y = lane >= kSignRounds && lane < kSignRounds + kSignOwn && y < M;
    SignStrip s[kSignStrips];
    uint32_t open = 0, have = 0;
#pragma unroll
    for (int k = 0; k < kSignStrips; ++k) {
        const int z = z0 + k;
        const bool in_grid = y >= 0 && y < M && z >= 0 && z < M;
        ulonglong2 c = make_ulonglong2(0, 0), l = c, r = c;
        if (in_grid) {
            const ulonglong2 *row = in + ((int64_t)z * W + b) * M + y;
            c = row[0];
            if (b > 0) l = row[-(int64_t)M];
            if (b + 1 < W) r = row[M];
        }
        auto spread = [](uint64_t l, uint64_t c, uint64_t r, uint32_t *v) {
            v[0] = (uint32_t)(l >> 48) | ((uint32_t)c << 16);
            v[1] = (uint32_t)(c >> 16);
            v[2] = (uint32_t)(c >> 48) | ((uint32_t)r << 16);
        };
        spread(l.x, c.x, r.x, s[k].p);
        spread(l.y, c.y, r.y, s[k].n);
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            s[k].u[i] = in_grid ? valid[i] & ~(s[k].p[i] | s[k].n[i]) : 0u;
            have |= s[k].p[i] | s[k].n[i];
        }
        const int zi = wave * kSignStrips + k;
        if (own_y && zi >= kSignRounds && zi < kSignRounds + kSignOwn)
            open |= (s[k].u[0] & 0xFFFF0000u) | s[k].u[1] | (s[k].u[2] & 0xFFFFu);
    }
    const bool busy = __syncthreads_or(open != 0) && __syncthreads_or(have != 0);
    for (int round = 0; busy && round < kSignRounds; ++round) {
        uint32_t(*e)[2][6][64] = edge[round & 1];
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            e[wave][0][i][lane] = s[0].p[i];
            e[wave][0][3 + i][lane] = s[0].n[i];
            e[wave][1][i][lane] = s[kSignStrips - 1].p[i];
            e[wave][1][3 + i][lane] = s[kSignStrips - 1].n[i];
        }
        __syncthreads();
        // the previous round's flag is complete; the one after next is free
        if (round > 0 && moved[(round + 2) % 3] == 0u) break;
        if (threadIdx.x == 0) moved[(round + 1) % 3] = 0u;
        uint32_t bp[3], bn[3];   // the row below in z, as it was before this round
        uint32_t tp[3], tn[3];   // the row above the wavefront's last
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            bp[i] = wave > 0 ? e[wave > 0 ? wave - 1 : 0][1][i][lane] : 0u;
            bn[i] = wave > 0 ? e[wave > 0 ? wave - 1 : 0][1][3 + i][lane] : 0u;
            tp[i] = wave + 1 < kSignWaves ? e[wave + 1 < kSignWaves ? wave + 1 : wave][0][i][lane] : 0u;
            tn[i] = wave + 1 < kSignWaves ? e[wave + 1 < kSignWaves ? wave + 1 : wave][0][3 + i][lane] : 0u;
        }
        uint32_t fresh = 0, fresh_own = 0;
#pragma unroll
        for (int k = 0; k < kSignStrips; ++k) {
            const int zi = wave * kSignStrips + k;
            uint32_t cp[3], cn[3];
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                cp[i] = s[k].p[i];
                cn[i] = s[k].n[i];
            }
            const bool wanted = zi > round && kSignTile - 1 - zi > round;   // uniform over the wavefront
            if (wanted && __any((s[k].u[0] | s[k].u[1] | s[k].u[2]) != 0u)) {
                uint32_t f[3];
#pragma unroll
                for (int i = 0; i < 3; ++i) {
                    uint32_t ap, an;   // the row above in z
                    if (k + 1 < kSignStrips) {
                        ap = s[k + 1 < kSignStrips ? k + 1 : k].p[i];
                        an = s[k + 1 < kSignStrips ? k + 1 : k].n[i];
                    } else {
                        ap = tp[i];
                        an = tn[i];
                    }
                    auto along_x = [&](const uint32_t *v) {
                        const uint32_t up = i > 0 ? __builtin_amdgcn_alignbit(v[i], v[i > 0 ? i - 1 : 0], 31) : v[0] << 1;
                        const uint32_t dn = i < 2 ? __builtin_amdgcn_alignbit(v[i < 2 ? i + 1 : 2], v[i], 1) : v[2] >> 1;
                        return up | dn;
                    };
                    const uint32_t pn = along_x(cp) | lane_below(cp[i]) | lane_above(cp[i]) | bp[i] | ap;
                    const uint32_t nn = along_x(cn) | lane_below(cn[i]) | lane_above(cn[i]) | bn[i] | an;
                    const uint32_t u = s[k].u[i];
                    f[i] = u & (pn | nn);
                    s[k].p[i] = cp[i] | (u & pn);
                    s[k].n[i] = cn[i] | (u & nn & ~pn);
                    s[k].u[i] = u & ~f[i];
                }
                fresh |= f[0] | f[1] | f[2];
                if (own_y && zi >= kSignRounds && zi < kSignRounds + kSignOwn)
                    fresh_own |= (f[0] & 0xFFFF0000u) | f[1] | (f[2] & 0xFFFFu);
            }
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                bp[i] = cp[i];
                bn[i] = cn[i];
            }
        }
        if (__any(fresh != 0u) && lane == 0) moved[round % 3] = 1u;
        if (__any(fresh_own != 0u) && lane == 0) changed[round] = 1u;
    }
#pragma unroll
    for (int k = 0; k < kSignStrips; ++k) {
        const int zi = wave * kSignStrips + k;
        if (!own_y || zi < kSignRounds || zi >= kSignRounds + kSignOwn || z0 + k >= M) continue;
        auto word = [](const uint32_t *v) {
            return (uint64_t)(v[0] >> 16) | ((uint64_t)v[1] << 16) | ((uint64_t)(v[2] & 0xFFFFu) << 48);
        };
        out[((int64_t)(z0 + k) * W + b) * M + y] = make_ulonglong2(word(s[k].p), word(s[k].n));
    }
}

// Corrected distances: core cells and cells without a sign keep d; the rest
// take |d| with their diffused sign.  HBM-bound: 8 B per cell.
__global__ __launch_bounds__(256) void sign_apply_kernel(const float *d, const ulonglong2 *__restrict__ state, int M,
                                                         int W, int64_t n_waves, double lc, float *out) {
    int b, y0;
    int64_t z;
    if (!sign_rows(M, W, n_waves, b, y0, z)) return;
    const int lane = threadIdx.x & 63;
    const int x = b * 64 + lane;
    float v[kSignLoads];
    ulonglong2 s[kSignLoads];
#pragma unroll
    for (int i = 0; i < kSignLoads; ++i) {
        const int y = min(y0 + i, M - 1);
        v[i] = d[(z * M + y) * M + min(x, M - 1)];
        s[i] = state[(z * W + b) * M + y];
    }
#pragma unroll
    for (int i = 0; i < kSignLoads; ++i) {
        const bool core = fabs((double)v[i]) < lc;
        float o = v[i];
        if (!core && ((s[i].x >> lane) & 1ull)) o = fabsf(v[i]);
        if (!core && ((s[i].y >> lane) & 1ull)) o = -fabsf(v[i]);
        if (x < M && y0 + i < M) out[(z * M + y0 + i) * M + x] = o;
    }
}

__global__ __launch_bounds__(256) void clear_flags_kernel(uint32_t *__restrict__ f, int n) {
    if ((int)threadIdx.x < n) f[threadIdx.x] = 0u;
}
static_assert(kFlags <= 256, "one workgroup clears the flags");

// Rounds whose flag is set, up to the first that is not; true when one is not.
bool count_rounds(const uint32_t *flags, int n, int32_t *rounds) {
    for (int k = 0; k < n; ++k) {
        if (!flags[k]) return true;
        ++*rounds;
    }
    return false;
}

}  // namespace

extern "C" sgrid_status sgrid_correct_signs(const sgrid_desc *desc, const float *d, float *out, void *stream,
                                            int32_t *rounds_out) {
    sgrid::clear_error();
    SG_REQUIRE(desc != nullptr, "desc is NULL");
    SG_REQUIRE(d != nullptr && out != nullptr, "d or out is NULL");
    SG_REQUIRE(sg_aligned(d, 4) && sg_aligned(out, 4), "d / out must be 4-byte aligned");
    SG_REQUIRE(desc->n_coarse >= 1 && desc->n_coarse <= 4096, "n_coarse must be in 1..4096 (got %d)",
               desc->n_coarse);
    SG_REQUIRE(desc->h > 0.0 && desc->h < 1e30, "h must be positive and finite");
    const int64_t M = desc->n_coarse, W = (M + 63) / 64, n_words = M * M * W;
    const int64_t n_waves = M * ((M + kSignLoads - 1) / kSignLoads) * W;
    const int64_t tiles = (M + kSignOwn - 1) / kSignOwn;
    const double lc = 4.0 * desc->h;
    hipStream_t st = sg_stream(stream);
    const size_t bits = (size_t)n_words * 16;
    uint8_t *mem = nullptr;
    sgrid_status s = sgrid::dev_alloc((void **)&mem, 2 * bits + kFlags * sizeof(uint32_t), "sign correction bitmaps");
    if (s != SGRID_OK) return s;
    ulonglong2 *state[2] = {(ulonglong2 *)mem, (ulonglong2 *)(mem + bits)};
    uint32_t *flags = (uint32_t *)(mem + 2 * bits);
    uint32_t *host = pinned_flags();
    if (host == nullptr) {
        sgrid::dev_free(mem);
        sgrid::set_error("pinned host flags could not be allocated");
        return SGRID_E_NOMEM;
    }
    auto fail = [&](hipError_t e, const char *what) {
        (void)hipStreamSynchronize(st);
        sgrid::dev_free(mem);
        pinned_release(host);
        sgrid::set_error("%s failed: %s", what, hipGetErrorString(e));
        return SGRID_E_HIP;
    };
    const dim3 wave_grid((unsigned)((n_waves + 3) / 4)), round_grid((unsigned)(W * tiles * tiles));
    hipLaunchKernelGGL(sign_init_kernel, wave_grid, dim3(256), 0, st, d, (int)M, (int)W, n_waves, lc, state[0]);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(e, "sign init");
    int cur = 0;
    int32_t rounds = 0;
    // every round that decides a cell is followed by one more; at most one
    // face step per round separates any cell from a core cell (3 (M - 1)),
    // so the loop ends by then
    const int64_t max_rounds = 3 * M + kSignRounds;
    bool done = false;
    for (int64_t base = 0; !done && base < max_rounds; base += kFlags) {
        hipLaunchKernelGGL(clear_flags_kernel, dim3(1), dim3(256), 0, st, flags, kFlags);
        for (int k = 0; k < kSignBatch; ++k)
            hipLaunchKernelGGL(sign_rounds_kernel, round_grid, dim3(64 * kSignWaves), 0, st, state[(cur + k) & 1],
                               (int)M, (int)W, (int)tiles, k > 0 ? flags + k * kSignRounds - 1 : nullptr,
                               state[(cur + k + 1) & 1], flags + k * kSignRounds);
        e = hipGetLastError();
        if (e != hipSuccess) return fail(e, "sign rounds");
        e = hipMemcpyAsync(host, flags, kFlags * sizeof(uint32_t), hipMemcpyDeviceToHost, st);
        if (e == hipSuccess) e = hipStreamSynchronize(st);
        if (e != hipSuccess) return fail(e, "sign round flags");
        const int32_t before = rounds;
        done = count_rounds(host, kFlags, &rounds);
        // launches that ran: up to the one with the first round that changed nothing
        const int ran = done ? (rounds - before) / kSignRounds + 1 : kSignBatch;
        cur = (cur + ran) & 1;
    }
    hipLaunchKernelGGL(sign_apply_kernel, wave_grid, dim3(256), 0, st, d, state[cur], (int)M, (int)W, n_waves, lc,
                       out);
    e = hipGetLastError();
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    if (e != hipSuccess) return fail(e, "sign apply");
    sgrid::dev_free(mem);
    pinned_release(host);
    if (rounds_out) *rounds_out = rounds;
    return SGRID_OK;
}

// ---------------------------------------------------------------------------
// The refined step on the data packages (Sec. 7.2: on a refined layer the
// operation is limited to the inner packages).  The points of core packages
// keep their sign, as the core cells do in the coarse step, and so do the
// far-field packages (their constants; a neighbour outside the domain is the
// positive far field, as in the neighbour table).  The points of inner
// packages get their sign by the same rounds of diffusion over face
// neighbours, reached through the six face slots of the package's face row.
//
// The state is a pair of 64-bit words per package, its positive and its
// negative points (bit i + 4 j + 16 k): a round takes one lane per package,
// with shifts inside the package and six neighbour pairs.  One byte per point
// and one lane per point took 50 us a round at 37 M points.
// ---------------------------------------------------------------------------
namespace {

constexpr int kPkgBatch = 8;    // rounds per check of the host
constexpr int kPkgLoads = 8;    // packages per wavefront of the passes over phi
static_assert(kPkgBatch <= kFlags, "the pinned buffer holds a batch of flags");

template <typename T>
__device__ __forceinline__ bool sign_bit(T v) { return __builtin_signbit(v); }

// HBM-bound: one read of phi.  `bits` gets the sign bits, so that the last
// pass need not read phi again.
template <typename T>
__global__ __launch_bounds__(256) void point_sign_init_kernel(const T *__restrict__ phi,
                                                              const uint8_t *__restrict__ pkg_type, int64_t n_pkgs,
                                                              ulonglong2 *__restrict__ state,
                                                              uint64_t *__restrict__ bits) {
    const int64_t p0 = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * kPkgLoads;
    if (p0 >= n_pkgs) return;   // whole wavefronts
    const int lane = threadIdx.x & 63;
    T v[kPkgLoads];
#pragma unroll
    for (int i = 0; i < kPkgLoads; ++i) v[i] = phi[(p0 + i < n_pkgs ? p0 + i : n_pkgs - 1) * 64 + lane];
    uint64_t mine = 0, sign = 0;
#pragma unroll
    for (int i = 0; i < kPkgLoads; ++i) {
        const uint64_t n = __ballot(v[i] < T(0)), b = __ballot(sign_bit(v[i]));
        if (lane == i) {
            mine = n;
            sign = b;
        }
    }
    const int64_t p = p0 + lane;
    if (lane < kPkgLoads && p < n_pkgs) {
        state[p] = pkg_type[p] == 2 ? make_ulonglong2(0, 0) : make_ulonglong2(~mine, mine);
        bits[p] = sign;
    }
}

__global__ __launch_bounds__(256) void point_sign_round_kernel(const ulonglong2 *__restrict__ state,
                                                               const uint32_t *__restrict__ face, int64_t n_pkgs,
                                                               const uint32_t *__restrict__ prev,
                                                               ulonglong2 *__restrict__ next,
                                                               uint32_t *__restrict__ changed) {
    if (prev != nullptr && *prev == 0u) return;
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n_pkgs) return;
    const ulonglong2 s = state[p];
    const uint64_t open = ~(s.x | s.y);
    if (!open) {
        next[p] = s;
        return;
    }
    const uint4 f0 = *reinterpret_cast<const uint4 *>(face + p * 8);
    const uint2 f1 = *reinterpret_cast<const uint2 *>(face + p * 8 + 4);
    const ulonglong2 xm = state[f0.x], xp = state[f0.y], ym = state[f0.z], yp = state[f0.w], zm = state[f1.x],
                     zp = state[f1.y];
    constexpr uint64_t kI0 = 0x1111111111111111ull, kI3 = 0x8888888888888888ull;
    constexpr uint64_t kJ0 = 0x000F000F000F000Full, kJ3 = 0xF000F000F000F000ull;
    auto near = [&](uint64_t c, uint64_t a, uint64_t b, uint64_t d, uint64_t e, uint64_t f, uint64_t g) {
        return ((c << 1) & ~kI0) | ((a >> 3) & kI0) | ((c >> 1) & ~kI3) | ((b << 3) & kI3) |
               ((c << 4) & ~kJ0) | ((d >> 12) & kJ0) | ((c >> 4) & ~kJ3) | ((e << 12) & kJ3) |
               (c << 16) | (f >> 48) | (c >> 16) | (g << 48);
    };
    const uint64_t pn = near(s.x, xm.x, xp.x, ym.x, yp.x, zm.x, zp.x);
    const uint64_t nn = near(s.y, xm.y, xp.y, ym.y, yp.y, zm.y, zp.y);
    next[p] = make_ulonglong2(s.x | (open & pn), s.y | (open & nn & ~pn));
    if (open & (pn | nn)) *changed = 1u;
}

// The points of inner packages whose sign bit is not that of their decided
// sign; nothing else of phi is touched.
template <typename T>
__global__ __launch_bounds__(256) void point_sign_apply_kernel(T *__restrict__ phi, const uint8_t *__restrict__ pkg_type,
                                                               const ulonglong2 *__restrict__ state,
                                                               const uint64_t *__restrict__ bits, int64_t n_pkgs) {
    const int64_t p0 = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * 64;
    if (p0 >= n_pkgs) return;   // whole wavefronts
    const int lane = threadIdx.x & 63;
    const int64_t p = p0 + lane;
    uint64_t flip = 0;
    if (p < n_pkgs && pkg_type[p] == 2) {
        const ulonglong2 s = state[p];
        flip = (s.x | s.y) & (s.y ^ bits[p]);
    }
    for (uint64_t todo = __ballot(flip != 0ull); todo; todo &= todo - 1ull) {
        const int k = __builtin_ctzll(todo);
        const uint64_t f = ((uint64_t)(uint32_t)__shfl((int)(flip >> 32), k) << 32) | (uint32_t)__shfl((int)flip, k);
        if ((f >> lane) & 1ull) {
            T *v = phi + (p0 + k) * 64 + lane;
            *v = sign_bit(*v) ? fabs(*v) : -fabs(*v);
        }
    }
}

template <typename T>
sgrid_status correct_package_signs(const sgrid_grid *g, T *phi, hipStream_t st, int32_t *rounds_out) {
    const int64_t n_pkgs = g->total();
    const dim3 load_grid((unsigned)((n_pkgs + 4 * kPkgLoads - 1) / (4 * kPkgLoads)));
    const dim3 pkg_grid((unsigned)((n_pkgs + 255) / 256));
    uint8_t *mem = nullptr;
    sgrid_status s = sgrid::dev_alloc((void **)&mem, (size_t)n_pkgs * 40 + kPkgBatch * sizeof(uint32_t),
                                      "sign correction state");
    if (s != SGRID_OK) return s;
    ulonglong2 *state[2] = {(ulonglong2 *)mem, (ulonglong2 *)mem + n_pkgs};
    uint64_t *bits = (uint64_t *)((ulonglong2 *)mem + 2 * n_pkgs);
    uint32_t *flags = (uint32_t *)(bits + n_pkgs);
    uint32_t *host = pinned_flags();
    if (host == nullptr) {
        sgrid::dev_free(mem);
        sgrid::set_error("pinned host flags could not be allocated");
        return SGRID_E_NOMEM;
    }
    auto fail = [&](hipError_t e, const char *what) {
        (void)hipStreamSynchronize(st);
        sgrid::dev_free(mem);
        pinned_release(host);
        sgrid::set_error("%s failed: %s", what, hipGetErrorString(e));
        return SGRID_E_HIP;
    };
    hipLaunchKernelGGL(point_sign_init_kernel<T>, load_grid, dim3(256), 0, st, phi, g->pkg_type, n_pkgs, state[0],
                       bits);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(e, "point sign init");
    int cur = 0;
    int32_t rounds = 0;
    bool done = false;
    // every inner point lies within a few face steps of a core package, but
    // the loop only ends on a round that changes nothing (or after as many
    // rounds as there are points)
    for (int64_t base = 0; !done && base < n_pkgs * 64 + kPkgBatch; base += kPkgBatch) {
        hipLaunchKernelGGL(clear_flags_kernel, dim3(1), dim3(256), 0, st, flags, kPkgBatch);
        for (int k = 0; k < kPkgBatch; ++k)
            hipLaunchKernelGGL(point_sign_round_kernel, pkg_grid, dim3(256), 0, st, state[(cur + k) & 1], g->face,
                               n_pkgs, k > 0 ? flags + k - 1 : nullptr, state[(cur + k + 1) & 1], flags + k);
        e = hipGetLastError();
        if (e != hipSuccess) return fail(e, "point sign rounds");
        e = hipMemcpyAsync(host, flags, kPkgBatch * sizeof(uint32_t), hipMemcpyDeviceToHost, st);
        if (e == hipSuccess) e = hipStreamSynchronize(st);
        if (e != hipSuccess) return fail(e, "point sign round flags");
        const int32_t before = rounds;
        done = count_rounds(host, kPkgBatch, &rounds);
        const int ran = done ? rounds - before + 1 : kPkgBatch;
        cur = (cur + ran) & 1;
    }
    hipLaunchKernelGGL(point_sign_apply_kernel<T>, pkg_grid, dim3(256), 0, st, phi, g->pkg_type, state[cur], bits,
                       n_pkgs);
    e = hipGetLastError();
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    if (e != hipSuccess) return fail(e, "point sign apply");
    sgrid::dev_free(mem);
    pinned_release(host);
    if (rounds_out) *rounds_out = rounds;
    return SGRID_OK;
}

}  // namespace

extern "C" sgrid_status sgrid_correct_package_signs(const sgrid_grid *g, sgrid_dtype dtype, void *phi, void *stream,
                                                    int32_t *rounds_out) {
    sgrid::clear_error();
    SG_REQUIRE(g != nullptr && phi != nullptr, "NULL argument");
    SG_REQUIRE(dtype == SGRID_F32 || dtype == SGRID_F64, "unknown dtype %d", (int)dtype);
    SG_REQUIRE(sg_aligned(phi, dtype == SGRID_F32 ? 4 : 8), "phi is not aligned to its element size");
    hipStream_t st = sg_stream(stream);
    if (dtype == SGRID_F32) return correct_package_signs<float>(g, (float *)phi, st, rounds_out);
    return correct_package_signs<double>(g, (double *)phi, st, rounds_out);
}
