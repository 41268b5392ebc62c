// The 9^3 phi window of a package (local coordinates -2..6 per axis), gathered
// through the package's 27-entry neighbour row with the index shift of
// Sec. 5.2 (slot = (s + 4) / 4, data = s + 4 - 4 slot per axis).
#pragma once

#include "common.hpp"

namespace sgrid {

constexpr int kWin = 9, kWinN = kWin * kWin * kWin;

// Window point q (x fastest) of the package whose neighbour ids are ids[27]:
// the flat index of its value in the field.
__device__ __forceinline__ int64_t window_source(const uint32_t *ids, int q) {
    const int x = q % kWin - 2, y = (q / kWin) % kWin - 2, z = q / (kWin * kWin) - 2;
    const int kx = (x + 4) >> 2, ky = (y + 4) >> 2, kz = (z + 4) >> 2;
    const int d = (x + 4 - 4 * kx) + 4 * (y + 4 - 4 * ky) + 16 * (z + 4 - 4 * kz);
    return (int64_t)ids[kx + 3 * ky + 9 * kz] * 64 + d;
}

// Thread t of NT stages its share of the window into s_phi.  All of the
// thread's loads are issued before any is used (a plain strided loop would
// wait for each load before the next: one memory round trip per iteration).
template <int NT>
__device__ __forceinline__ void stage_window_part(const float *__restrict__ phi, const uint32_t *ids, int t,
                                                  float *s_phi) {
    constexpr int kIters = (kWinN + NT - 1) / NT;
    float v[kIters];
#pragma unroll
    for (int u = 0; u < kIters; ++u) {
        const int q = t + u * NT;
        v[u] = phi[window_source(ids, q < kWinN ? q : kWinN - 1)];
    }
#pragma unroll
    for (int u = 0; u < kIters; ++u) {
        const int q = t + u * NT;
        if (q < kWinN) s_phi[q] = v[u];
    }
}

// LDS layout of the 7^3 cut fractions V around a package (window coordinates
// -1..5): rows of 8 along x (x = 0..5 at 0..5, x = -1 at 7, 6 unused), 8 floats
// per y step and 60 per z step.  A row is two aligned 16-byte words, and the 32
// lanes of a half-wavefront (i, j in 0..3, k in 0..1) read 32 distinct banks at
// any tap.
constexpr int kVol = 7, kVolN = kVol * kVol * kVol;
constexpr int kVRow = 8, kVPlane = 60, kVWinN = kVol * kVPlane;
__device__ __forceinline__ int vidx(int x, int y, int z) { return (x & 7) + kVRow * (y + 1) + kVPlane * (z + 1); }

// The 9^3 phi window of a package, one window row of 9 per lane and step (81
// rows, NT lanes): x = -2, -1 from the -x neighbour's row (8-byte load), x =
// 0..3 the package's own row (16-byte load), x = 4..6 from the +x neighbour's
// row (16-byte load, the fourth value unused).  Row r is y = r % 9 - 2, z = r /
// 9 - 2.
template <int NT>
struct WindowRows {
    static constexpr int kRows = kWin * kWin, kSteps = (kRows + NT - 1) / NT;
    int row[kSteps], slot[kSteps];   // the lane's rows: offset in a package, neighbour slot of x = -1
    float2 m[kSteps];
    float4 c[kSteps], q[kSteps];

    __device__ __forceinline__ explicit WindowRows(int t) {
#pragma unroll
        for (int u = 0; u < kSteps; ++u) {
            const int r = min(t + NT * u, kRows - 1);
            const int y = r % kWin - 2, z = r / kWin - 2;
            const int ky = (y + 4) >> 2, kz = (z + 4) >> 2;
            row[u] = 4 * ((y + 4 - 4 * ky) + 4 * (z + 4 - 4 * kz));
            slot[u] = 3 * ky + 9 * kz;
        }
    }
    // id(s): the package in neighbour slot s
    template <class Id>
    __device__ __forceinline__ void load(const float *__restrict__ phi, const Id &id) {
#pragma unroll
        for (int u = 0; u < kSteps; ++u) {
            const uint32_t im = id(slot[u]), ic = id(slot[u] + 1), ip = id(slot[u] + 2);
            m[u] = *reinterpret_cast<const float2 *>(phi + (int64_t)im * 64 + row[u] + 2);
            c[u] = *reinterpret_cast<const float4 *>(phi + (int64_t)ic * 64 + row[u]);
            q[u] = *reinterpret_cast<const float4 *>(phi + (int64_t)ip * 64 + row[u]);
        }
    }
    __device__ __forceinline__ void values(int u, float (&v)[kWin]) const {
        v[0] = m[u].x; v[1] = m[u].y;
        v[2] = c[u].x; v[3] = c[u].y; v[4] = c[u].z; v[5] = c[u].w;
        v[6] = q[u].x; v[7] = q[u].y; v[8] = q[u].z;
    }
};

}  // namespace sgrid
