// Batched reinitialisation: many grids (shapes of uneven size) swept by one
// persistent launch per iteration over a global package worklist, the
// iteration loop replayed as a HIP graph, and an autotuner that times the
// candidate kernels on the caller's data.
//
// Layout: the fields of all grids are concatenated, grid s occupying package
// ids [base_s, base_s + P_s + 2) (its two far-field rows first).  The
// worklist lists the activated packages of every grid, each grid's in the
// Morton order of its cells (the grids' own sweep order), and holds one row
// per entry: (-x, +x, -y, +y, -z, +z, g, s) with the neighbours and the
// package g rebased to global ids and the grid index s, which selects that
// grid's (h^2, 1/h, h/2) in a small parameter table.  Each wavefront walks a
// contiguous range of the worklist, four packages at a time.
//
// A batch whose two buffers exceed the Infinity Cache goes in segments of whole
// grids that fit it, each through all its iterations before the next (the grids
// do not depend on each other), so that a sweep finds the rows that the one
// before it wrote.  24 random unions of up to 512^3 points (594 k packages, 318
// MB with the worklist) take 53 us per iteration over all in two segments,
// from 78 in one.
//
// The per-point update is the same function as the single-grid sweep with the
// same per-grid constants, so every grid's result is bit-identical to its own
// sgrid_reinitialize.
#include <string.h>

#include <vector>

#include "common.hpp"
#include "upwind.hpp"

namespace sgrid {
template <typename T>
struct SweepParams {
    T h2, inv_h, dt;
};
}  // namespace sgrid

namespace {

template <typename T>
struct Row4 { T v[4]; };

__device__ __forceinline__ Row4<float> ld_row(const float *__restrict__ p) {
    const float4 a = *reinterpret_cast<const float4 *>(p);
    return Row4<float>{{a.x, a.y, a.z, a.w}};
}
// How a sweep stores its rows.  Streamed (non-temporal hint): ping-pong buffers
// larger than the last-level cache, where the written rows would only push out
// lines the running sweep still reads.  Through: written through the L2, by sweeps
// of one set per wavefront over kThroughPackages and more (23 unions, 56 k
// packages: 9.6 -> 8.9 us an iteration).  A wavefront that goes on to its next set
// waits for such a store with the set's loads (one workgroup per CU: 16.9 and
// 19.5 us, four: 10.4 and 11.1), and a small sweep leaves little to write back (5.8 k
// packages: 3.76 and 3.86 us): plain stores there.
enum class Store : int { kPlain, kThrough, kStreamed };
constexpr int64_t kThroughPackages = 16384;

template <typename I>
__device__ __forceinline__ void st_row(float *__restrict__ base, I off, const Row4<float> &r, Store mode) {
    typedef float f4v __attribute__((ext_vector_type(4)));
    const f4v v = {r.v[0], r.v[1], r.v[2], r.v[3]};
    f4v *p = reinterpret_cast<f4v *>(at_offset(base, off));
    if (mode == Store::kStreamed)
        __builtin_nontemporal_store(v, p);
    else if (mode == Store::kThrough)
        store_through(base, off, v);
    else
        *p = v;
}

struct Halo {
    Row4<float> c, yh, zh;
    float xm, xp;
};

// Loads of worklist entry e: its row of the worklist table (face neighbours,
// package id g, grid index), then the package row and its halos.
template <typename I>
__device__ __forceinline__ void batch_loads(const float *__restrict__ src, const uint32_t *__restrict__ wrow, I e,
                                            int r, Halo &l, uint32_t &g, uint32_t &shape) {
    const int j = r & 3, k = r >> 2;
    const uint4 f0 = *reinterpret_cast<const uint4 *>(at_offset(wrow, e * 32));
    const uint4 f1 = *reinterpret_cast<const uint4 *>(at_offset(wrow, e * 32 + 16));
    g = f1.z;
    shape = f1.w;
    auto value = [&](uint32_t row, int at) { return at_offset(src, row_offset<float, I>(row, at)); };
    l.c = ld_row(value(g, r * 4));
    l.xm = *value(f0.x, r * 4 + 3);
    l.xp = *value(f0.y, r * 4);
    // unconditional, so the halo loads issue together instead of behind a
    // branch that waits: a lane without a y / z halo loads that of its
    // neighbour lane on the same side (unused), touching no other lines
    l.yh = ld_row(value(j < 2 ? f0.z : f0.w, (j < 2 ? 3 + 4 * k : 4 * k) * 4));
    l.zh = ld_row(value(k < 2 ? f1.x : f1.y, (k < 2 ? j + 12 : j) * 4));
}

__device__ __forceinline__ Row4<float> update_row_dpp(const Halo &l, const sgrid::SweepParams<float> &sp) {
    Row4<float> o, ym, yp, zm, zp;
    row_neighbours<false>(l.c.v, l.yh.v, ym.v, yp.v);
    row_neighbours<true>(l.c.v, l.zh.v, zm.v, zp.v);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float xm = i > 0 ? l.c.v[i - 1] : l.xm;
        const float xp = i < 3 ? l.c.v[i + 1] : l.xp;
        o.v[i] = sgrid::upwind_update(l.c.v[i], xm, xp, ym.v[i], yp.v[i], zm.v[i], zp.v[i], sp.h2, sp.inv_h, sp.dt);
    }
    return o;
}

// Persistent worklist sweep, DPP exchange.  Wavefront w processes the sets
// [w * spw, (w + 1) * spw) of four worklist entries.
template <typename I>   // byte offsets in the concatenated field
__global__ __launch_bounds__(256) void batch_dpp_kernel(const float *__restrict__ src, float *__restrict__ dst,
                                                        const uint32_t *__restrict__ wrow, I n_work,
                                                        const sgrid::SweepParams<float> *__restrict__ params,
                                                        I n_blocks, I spw, Store mode) {
    const I b = block_of(n_blocks);
    const int lane = threadIdx.x & 63, r = lane & 15;
    const I wave = b * 4 + (threadIdx.x >> 6);
    const I n_sets = (n_work + 3) / 4;
    const I s0 = wave * spw, s1 = s0 + spw < n_sets ? s0 + spw : n_sets;
    for (I s = s0; s < s1; ++s) {
        const I e = 4 * s + (lane >> 4);
        const bool live = e < n_work;
        Halo l;
        uint32_t shape = 0, g = 0;
        if (live) batch_loads(src, wrow, e, r, l, g, shape);
        const sgrid::SweepParams<float> sp = params[shape];
        const Row4<float> o = update_row_dpp(l, sp);
        if (live) st_row(dst, row_offset<float, I>(g, r * 4), o, mode);
    }
}

// Persistent worklist sweep, LDS tile (package + one-cell face halo).
__global__ __launch_bounds__(256) void batch_lds_kernel(const float *__restrict__ src, float *__restrict__ dst,
                                                        const uint32_t *__restrict__ wrow, int64_t n_work,
                                                        const sgrid::SweepParams<float> *__restrict__ params,
                                                        int64_t n_blocks, int64_t spw, Store mode) {
    __shared__ float tile[16][216];
    const int64_t b = xcd_block(blockIdx.x, n_blocks);
    const int lane = threadIdx.x & 63, r = lane & 15, j = r & 3, k = r >> 2;
    float *t = tile[threadIdx.x >> 4];
    auto at = [](int x, int y, int z) { return (x + 1) + 6 * ((y + 1) + 6 * (z + 1)); };
    const int64_t wave = b * 4 + (threadIdx.x >> 6);
    const int64_t n_sets = (n_work + 3) / 4;
    const int64_t s0 = wave * spw, s1 = s0 + spw < n_sets ? s0 + spw : n_sets;
    // every wavefront of the block runs the same number of iterations (barriers)
    for (int64_t it = 0; it < spw; ++it) {
        const int64_t s = s0 + it;
        const int64_t e = 4 * s + (lane >> 4);
        const bool live = s < s1 && e < n_work;
        Halo l;
        uint32_t shape = 0, g = 0;
        if (live) {
            batch_loads(src, wrow, e, r, l, g, shape);
#pragma unroll
            for (int i = 0; i < 4; ++i) t[at(i, j, k)] = l.c.v[i];
            t[at(-1, j, k)] = l.xm;
            t[at(4, j, k)] = l.xp;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (j == 0) t[at(i, -1, k)] = l.yh.v[i];
                if (j == 3) t[at(i, 4, k)] = l.yh.v[i];
                if (k == 0) t[at(i, j, -1)] = l.zh.v[i];
                if (k == 3) t[at(i, j, 4)] = l.zh.v[i];
            }
        }
        __syncthreads();
        if (live) {
            const sgrid::SweepParams<float> sp = params[shape];
            Row4<float> o;
#pragma unroll
            for (int i = 0; i < 4; ++i)
                o.v[i] = sgrid::upwind_update(t[at(i, j, k)], t[at(i - 1, j, k)], t[at(i + 1, j, k)], t[at(i, j - 1, k)],
                                t[at(i, j + 1, k)], t[at(i, j, k - 1)], t[at(i, j, k + 1)], sp.h2, sp.inv_h, sp.dt);
            st_row(dst, row_offset<float, int64_t>(g, r * 4), o, mode);
        }
        __syncthreads();
    }
}

// Worklist rows of grid s: its sweep-order face rows (wface) rebased to global
// ids, with the grid index in the last slot.
__global__ __launch_bounds__(256) void rebase_kernel(const uint32_t *__restrict__ wface_s, int64_t P_s, uint32_t base,
                                                     uint32_t shape, uint32_t *__restrict__ wrow, int64_t work_base) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= P_s) return;
    uint32_t *o = wrow + (work_base + t) * 8;
    const uint32_t *in = wface_s + t * 8;
#pragma unroll
    for (int f = 0; f < 7; ++f) o[f] = base + in[f];
    o[7] = shape;
}

// Copies the far-field rows of every grid from one buffer to the other.
__global__ __launch_bounds__(128) void far_rows_copy_kernel(const float *__restrict__ src, float *__restrict__ dst,
                                                            const uint32_t *__restrict__ bases) {
    const int64_t base = bases[blockIdx.x];
    const int t = threadIdx.x;   // 128 values: rows base and base + 1
    dst[base * 64 + t] = src[base * 64 + t];
}

}  // namespace

struct sgrid_batch {
    int device = 0;
    int32_t n = 0;
    int64_t n_total = 0;      // concatenated package rows
    int64_t n_work = 0;
    uint32_t *wrow = nullptr;         // [n_work][8] worklist rows
    uint32_t *bases = nullptr;        // device copy of grid bases
    sgrid::SweepParams<float> *params = nullptr;
    std::vector<int64_t> base_host, total_host;
    // worklist ranges of whole grids, each swept through all its iterations
    struct Segment { int64_t first, count; };
    std::vector<Segment> segments;
    // the configuration; until it is set or tuned, one wavefront per four packages
    // (against four workgroups per CU: 23 unions up to 128^3 9.0 and 10.5 us an
    // iteration, 64 up to 512^3 107 and 129)
    int32_t variant = 0, blocks_per_cu = 0;
    // captured iteration loop
    hipGraphExec_t exec = nullptr;
    hipGraph_t graph = nullptr;
    hipStream_t cap_stream = nullptr;
    const void *g_phi = nullptr, *g_scratch = nullptr;
    int32_t g_iter = -1, g_variant = -1, g_bpc = -1;
};

namespace {

// Packages of a segment: two rows of 256 B and a worklist row of 32 B each in
// 95 % of the 256 MiB Infinity Cache (with 88 % a batch of 457 k packages, 249 MB,
// was two segments, and the launches of the second cost more than its rows: 50.4 us
// an iteration against 48.4).
constexpr double kCacheBytes = 256.0 * 1024 * 1024;
constexpr int64_t kPackageBytes = 2 * 256 + 32;
constexpr int64_t kSegmentPackages = (int64_t)(0.95 * kCacheBytes) / kPackageBytes;

// The grids' worklist ranges in as few segments of at most kSegmentPackages as
// their number needs, of about equal size (a larger grid is its own segment).
std::vector<sgrid_batch::Segment> plan_segments(const std::vector<int64_t> &packages) {
    int64_t all = 0;
    for (int64_t p : packages) all += p;
    const int64_t n = (all + kSegmentPackages - 1) / kSegmentPackages;
    const int64_t target = n > 0 ? (all + n - 1) / n : 0;
    std::vector<sgrid_batch::Segment> out;
    int64_t first = 0, count = 0;
    for (int64_t p : packages) {
        // the grid starts a new segment where that leaves this one nearer its share
        if (count > 0 && (count + p > kSegmentPackages || count + p - target > target - count)) {
            out.push_back({first, count});
            first += count;
            count = 0;
        }
        count += p;
    }
    if (count > 0) out.push_back({first, count});
    return out;
}

sgrid_status launch_batch_sweep(const sgrid_batch *b, const sgrid_batch::Segment &seg, const float *src, float *dst,
                                int variant, int bpc, hipStream_t st) {
    // bpc workgroups per CU walk the worklist persistently; bpc = 0 launches
    // one wavefront per set of four packages instead
    const int64_t n_sets = (seg.count + 3) / 4;
    int64_t nb = bpc > 0 ? (int64_t)sgrid::cu_count() * bpc : (n_sets + 3) / 4;
    const int64_t spw = (n_sets + nb * 4 - 1) / (nb * 4);
    nb = (n_sets + spw * 4 - 1) / (spw * 4);
    const bool streamed = 2.0 * (double)seg.count * 64.0 * sizeof(float) > kCacheBytes;
    const Store mode = streamed ? Store::kStreamed
                                : (spw == 1 && seg.count >= kThroughPackages ? Store::kThrough : Store::kPlain);
    const uint32_t *wrow = b->wrow + seg.first * 8;
    if (variant == 1)
        hipLaunchKernelGGL(batch_lds_kernel, dim3((unsigned)nb), dim3(256), 0, st, src, dst, wrow, seg.count,
                           b->params, nb, spw, mode);
    else if ((double)b->n_total * 256.0 <= 4294967296.0)   // 32-bit byte offsets
        hipLaunchKernelGGL(batch_dpp_kernel<uint32_t>, dim3((unsigned)nb), dim3(256), 0, st, src, dst, wrow,
                           (uint32_t)seg.count, b->params, (uint32_t)nb, (uint32_t)spw, mode);
    else
        hipLaunchKernelGGL(batch_dpp_kernel<int64_t>, dim3((unsigned)nb), dim3(256), 0, st, src, dst, wrow, seg.count,
                           b->params, nb, spw, mode);
    SG_CHECK_LAUNCH("batch sweep");
    return SGRID_OK;
}

// The iteration loop on `st`: far-field rows into the scratch buffer, then
// n_iter ping-pong sweeps of every segment; an odd count leaves the result in
// scratch.
sgrid_status enqueue_loop(const sgrid_batch *b, float *phi, float *scratch, int32_t n_iter, int variant, int bpc,
                          hipStream_t st) {
    hipLaunchKernelGGL(far_rows_copy_kernel, dim3((unsigned)b->n), dim3(128), 0, st, phi, scratch, b->bases);
    SG_CHECK_LAUNCH("far-field rows");
    for (const sgrid_batch::Segment &seg : b->segments) {
        float *a = phi, *c = scratch;
        for (int32_t it = 0; it < n_iter; ++it) {
            sgrid_status s = launch_batch_sweep(b, seg, a, c, variant, bpc, st);
            if (s != SGRID_OK) return s;
            float *t = a;
            a = c;
            c = t;
        }
    }
    return SGRID_OK;
}

void drop_graph(sgrid_batch *b) {
    if (b->exec) (void)hipGraphExecDestroy(b->exec);
    if (b->graph) (void)hipGraphDestroy(b->graph);
    b->exec = nullptr;
    b->graph = nullptr;
    b->g_iter = -1;
}

}  // namespace

extern "C" sgrid_status sgrid_batch_create(const sgrid_grid *const *grids, int32_t n, void *stream,
                                           sgrid_batch **out) {
    sgrid::clear_error();
    SG_REQUIRE(out != nullptr, "out is NULL");
    *out = nullptr;
    SG_REQUIRE(grids != nullptr && n >= 1, "need at least one grid");
    int64_t total = 0, work = 0;
    for (int32_t s = 0; s < n; ++s) {
        SG_REQUIRE(grids[s] != nullptr, "grid %d is NULL", s);
        total += grids[s]->total();
        work += grids[s]->P;
    }
    if (total >= (int64_t)0xFFFFFFFFll) {
        sgrid::set_error("batch of %lld package rows exceeds 32-bit ids", (long long)total);
        return SGRID_E_CAPACITY;
    }
    hipStream_t st = sg_stream(stream);
    sgrid_batch *b = new sgrid_batch();
    (void)hipGetDevice(&b->device);
    b->n = n;
    b->n_total = total;
    b->n_work = work;
    auto fail = [&](sgrid_status s) {
        sgrid::dev_free(b->wrow);
        sgrid::dev_free(b->bases);
        sgrid::dev_free(b->params);
        delete b;
        return s;
    };
    sgrid_status s;
    if ((s = sgrid::dev_alloc((void **)&b->wrow, (size_t)(work > 0 ? work : 1) * 32, "worklist rows")) != SGRID_OK)
        return fail(s);
    if ((s = sgrid::dev_alloc((void **)&b->bases, (size_t)n * 4, "grid bases")) != SGRID_OK) return fail(s);
    if ((s = sgrid::dev_alloc((void **)&b->params, (size_t)n * sizeof(sgrid::SweepParams<float>), "grid params")) !=
        SGRID_OK)
        return fail(s);
    std::vector<uint32_t> bases(n);
    std::vector<int64_t> packages;
    std::vector<sgrid::SweepParams<float>> params(n);
    int64_t base = 0, wbase = 0;
    for (int32_t k = 0; k < n; ++k) {
        const sgrid_grid *g = grids[k];
        bases[k] = (uint32_t)base;
        b->base_host.push_back(base);
        b->total_host.push_back(g->total());
        packages.push_back(g->P);
        // the same constants as the single-grid sweep
        params[k] = sgrid::SweepParams<float>{(float)(g->h * g->h), (float)(1.0 / g->h), (float)(0.5 * g->h)};
        const int64_t nt = g->total();
        if (g->P > 0)
            hipLaunchKernelGGL(rebase_kernel, dim3((unsigned)((g->P + 255) / 256)), dim3(256), 0, st, g->wface, g->P,
                               (uint32_t)base, (uint32_t)k, b->wrow, wbase);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) {
            sgrid::set_error("batch table launch failed: %s", hipGetErrorString(e));
            return fail(SGRID_E_HIP);
        }
        base += nt;
        wbase += g->P;
    }
    hipError_t e = hipMemcpyAsync(b->bases, bases.data(), (size_t)n * 4, hipMemcpyHostToDevice, st);
    if (e == hipSuccess)
        e = hipMemcpyAsync(b->params, params.data(), (size_t)n * sizeof(params[0]), hipMemcpyHostToDevice, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    if (e != hipSuccess) {
        sgrid::set_error("batch table upload failed: %s", hipGetErrorString(e));
        return fail(SGRID_E_HIP);
    }
    b->segments = plan_segments(packages);
    *out = b;
    return SGRID_OK;
}

extern "C" sgrid_status sgrid_batch_destroy(sgrid_batch *b) {
    sgrid::clear_error();
    if (!b) return SGRID_OK;
    hipError_t e = hipDeviceSynchronize();
    drop_graph(b);
    if (b->cap_stream) (void)hipStreamDestroy(b->cap_stream);
    sgrid::dev_free(b->wrow);
    sgrid::dev_free(b->bases);
    sgrid::dev_free(b->params);
    delete b;
    if (e != hipSuccess) {
        sgrid::set_error("hipDeviceSynchronize before destroy failed: %s", hipGetErrorString(e));
        return SGRID_E_HIP;
    }
    return SGRID_OK;
}

extern "C" sgrid_status sgrid_batch_info(const sgrid_batch *b, int64_t *n_total, int64_t *n_work,
                                         int64_t *bases_host) {
    sgrid::clear_error();
    SG_REQUIRE(b != nullptr, "batch is NULL");
    if (n_total) *n_total = b->n_total;
    if (n_work) *n_work = b->n_work;
    if (bases_host)
        for (int32_t k = 0; k < b->n; ++k) bases_host[k] = b->base_host[k];
    return SGRID_OK;
}

extern "C" sgrid_status sgrid_batch_set_config(sgrid_batch *b, int32_t variant, int32_t blocks_per_cu) {
    sgrid::clear_error();
    SG_REQUIRE(b != nullptr, "batch is NULL");
    SG_REQUIRE(variant == 0 || variant == 1, "batch variant must be 0 or 1");
    SG_REQUIRE(blocks_per_cu >= 0 && blocks_per_cu <= 16, "blocks_per_cu must be in 0..16");
    b->variant = variant;
    b->blocks_per_cu = blocks_per_cu;
    return SGRID_OK;
}

extern "C" sgrid_status sgrid_batch_autotune(sgrid_batch *b, const float *phi, float *scratch, int32_t reps,
                                             void *stream, int32_t *variant_out, int32_t *bpc_out,
                                             float *us_table /* [2][6] */) {
    sgrid::clear_error();
    SG_REQUIRE(b != nullptr && phi != nullptr && scratch != nullptr, "NULL argument");
    SG_REQUIRE(reps >= 1 && reps <= 1000, "reps must be in 1..1000");
    hipStream_t st = sg_stream(stream);
    static const int kBpc[6] = {1, 2, 4, 8, 16, 0};
    hipEvent_t e0, e1;
    SG_CHECK_HIP(hipEventCreate(&e0));
    SG_CHECK_HIP(hipEventCreate(&e1));
    float best = 1e30f;
    int bv = 0, bb = 4;
    for (int v = 0; v < 2; ++v)
        for (int i = 0; i < 6; ++i) {
            // phi is only read: every timed sweep writes scratch; a segment's
            // sweeps follow each other, as in the iteration loop.  (A segment
            // beyond the Infinity Cache then finds phi in it, and all candidates
            // look faster than in a call, 57 us and 89 for the torus at 1200^3, but
            // in the same order: six batches looked at.)
            auto sweeps = [&](int n_sweeps) {
                for (const sgrid_batch::Segment &seg : b->segments)
                    for (int k = 0; k < n_sweeps; ++k) {
                        const sgrid_status s = launch_batch_sweep(b, seg, phi, scratch, v, kBpc[i], st);
                        if (s != SGRID_OK) return s;
                    }
                return SGRID_OK;
            };
            sgrid_status s = sweeps(1);
            if (s != SGRID_OK) return s;
            SG_CHECK_HIP(hipEventRecord(e0, st));
            s = sweeps(reps);
            if (s != SGRID_OK) return s;
            SG_CHECK_HIP(hipEventRecord(e1, st));
            SG_CHECK_HIP(hipEventSynchronize(e1));
            float ms = 0.f;
            SG_CHECK_HIP(hipEventElapsedTime(&ms, e0, e1));
            const float us = 1e3f * ms / reps;
            if (us_table) us_table[v * 6 + i] = us;
            if (us < best) {
                best = us;
                bv = v;
                bb = kBpc[i];
            }
        }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    b->variant = bv;
    b->blocks_per_cu = bb;
    if (variant_out) *variant_out = bv;
    if (bpc_out) *bpc_out = bb;
    return SGRID_OK;
}

extern "C" sgrid_status sgrid_batch_reinitialize(sgrid_batch *b, float *phi, float *scratch, int32_t n_iter,
                                                 int32_t use_graph, void *stream) {
    sgrid::clear_error();
    SG_REQUIRE(b != nullptr && phi != nullptr && scratch != nullptr, "NULL argument");
    SG_REQUIRE(phi != scratch, "phi and scratch must be distinct");
    SG_REQUIRE(sg_aligned(phi, 16) && sg_aligned(scratch, 16), "phi / scratch must be 16-byte aligned");
    SG_REQUIRE(n_iter >= 0, "n_iter must be >= 0");
    if (n_iter == 0) return SGRID_OK;
    hipStream_t st = sg_stream(stream);
    if (!use_graph) {
        sgrid_status s = enqueue_loop(b, phi, scratch, n_iter, b->variant, b->blocks_per_cu, st);
        if (s != SGRID_OK) return s;
    } else {
        if (b->g_phi != phi || b->g_scratch != scratch || b->g_iter != n_iter || b->g_variant != b->variant ||
            b->g_bpc != b->blocks_per_cu || !b->exec) {
            drop_graph(b);
            if (!b->cap_stream) SG_CHECK_HIP(hipStreamCreateWithFlags(&b->cap_stream, hipStreamNonBlocking));
            SG_CHECK_HIP(hipStreamBeginCapture(b->cap_stream, hipStreamCaptureModeThreadLocal));
            sgrid_status s = enqueue_loop(b, phi, scratch, n_iter, b->variant, b->blocks_per_cu, b->cap_stream);
            hipGraph_t g = nullptr;
            hipError_t e = hipStreamEndCapture(b->cap_stream, &g);
            if (s != SGRID_OK) {
                if (g) (void)hipGraphDestroy(g);
                return s;
            }
            if (e != hipSuccess) {
                sgrid::set_error("graph capture failed: %s", hipGetErrorString(e));
                return SGRID_E_HIP;
            }
            b->graph = g;
            e = hipGraphInstantiate(&b->exec, g, nullptr, nullptr, 0);
            if (e != hipSuccess) {
                drop_graph(b);
                sgrid::set_error("graph instantiation failed: %s", hipGetErrorString(e));
                return SGRID_E_HIP;
            }
            b->g_phi = phi;
            b->g_scratch = scratch;
            b->g_iter = n_iter;
            b->g_variant = b->variant;
            b->g_bpc = b->blocks_per_cu;
        }
        SG_CHECK_HIP(hipGraphLaunch(b->exec, st));
    }
    if (n_iter & 1) {
        // the result sits in scratch: copy the activated rows of every grid back
        for (int32_t k = 0; k < b->n; ++k) {
            const int64_t r0 = b->base_host[k] + 2, nr = b->total_host[k] - 2;
            if (nr > 0)
                SG_CHECK_HIP(hipMemcpyAsync(phi + r0 * 64, scratch + r0 * 64, (size_t)nr * 64 * 4,
                                            hipMemcpyDeviceToDevice, st));
        }
    }
    return SGRID_OK;
}
