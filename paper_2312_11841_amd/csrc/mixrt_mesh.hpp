// Internal interface of the geometry stage, which produces the G-buffer of
// the coarse mesh (Fig. 2 step 1): the uploaded mesh (triangle records and the
// uniform grid of triangle lists, built on the host in mixrt_mesh.cpp), the
// rasteriser (mixrt_raster.hip) and the ray-casting kernel that walks the grid
// (mixrt_raycast.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <vector>

#include "mixrt.h"
#include "mixrt_device.hpp"

namespace mixrt {

inline constexpr int kMaxGridAxis = 1024;
inline constexpr int64_t kMaxGridCells = int64_t(1) << 26;
// Triangle boxes are padded by this fraction of a cell when binned, so that
// a hit computed in fp32 near a cell face is listed in the cell on either side.
inline constexpr double kBinPad = 1.0 / 500.0;

// Device view of an uploaded mesh.  Cell (x, y, z) is index (z*ny + y)*nx + x
// and cells[c] = (first, count): a cell with triangles lists them in
// refs[first .. first+count); an empty cell (count 0) holds in `first` its
// Chebyshev distance D (in cells, 1..255) to the nearest cell with
// triangles, so every cell within D-1 of it on each axis is empty as well.
// A ref is three float4: (v0, triangle index bits), (e1, 0), (e2, 0).
// attr[tri] is two float4: (uv0, uv1), (uv2, 0, 0).
struct MeshGridK {
    float lo[3], hi[3], cell[3], inv_cell[3];
    int32_t n[3];
    const uint2 *cells;
    const float4 *refs;
    const float4 *attr;
    const float4 *tris;   // [n_faces] records like refs, in triangle order
    int32_t n_faces;
};

// A ray's walk through the grid, in units of cells: the ray is o + s d from the
// point o where it enters the grid (its own origin inside), with o and d scaled
// by the cell size and s = t - t_in, a cell is its integer coordinates held as
// floats, and tn[a] = (c + face[a]) inv[a] is the distance s to its next face on
// axis a (face holds -o and which of the two faces; inf where the ray does not
// move on the axis).
//
// o is the point at t_in rounded once, so a face crossing errs with the cells of
// its axis and not with the camera's distance: by at most 2.7e-4 of a cell at
// 1024 cells, from 0 to 10^4 extents away, a seventh of kBinPad.  (Scaled from
// the camera's own position it erred by 4.1e-3 from 10 extents away, twice
// kBinPad, and by 5.6 cells from 10^4.)
struct Walk {
    float o[3], d[3], inv[3], face[3], st[3];
    float c[3], tn[3];
};

__host__ __device__ inline void walk_faces(Walk &w)
{
#pragma unroll
    for (int a = 0; a < 3; ++a) w.tn[a] = (w.c[a] + w.face[a]) * w.inv[a];
}

// The walk of the ray o + t d (world space) at its first cell; false when the
// ray does not meet the grid's box.
__host__ __device__ inline bool walk_enter(const MeshGridK &g, const float o[3], const float d[3],
                                           Walk &w, float &t_in)
{
    constexpr float kInf = __builtin_inff();
    float t0 = 0.0f, t1 = kInf, inv[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        inv[a] = 1.0f / d[a];
        const float ta = (g.lo[a] - o[a]) * inv[a], tb = (g.hi[a] - o[a]) * inv[a];
        t0 = fmaxf(t0, fminf(ta, tb));
        t1 = fminf(t1, fmaxf(ta, tb));
    }
    t_in = t0;
    if (!(t0 <= t1) || !(t0 < kInf)) return false;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        w.o[a] = (fmaf(t0, d[a], o[a]) - g.lo[a]) * g.inv_cell[a];
        w.d[a] = d[a] * g.inv_cell[a];
        const bool moves = d[a] > 0.0f || d[a] < 0.0f;
        w.st[a] = moves ? copysignf(1.0f, d[a]) : 0.0f;
        w.inv[a] = moves ? inv[a] * g.cell[a] : 1.0f;
        w.face[a] = moves ? (d[a] > 0.0f ? 1.0f : 0.0f) - w.o[a] : kInf;
        w.c[a] = fminf(fmaxf(floorf(w.o[a]), 0.0f), (float)(g.n[a] - 1));
    }
    walk_faces(w);
    return true;
}

// The grid as built on the host, before upload.
struct MeshGridHost {
    int32_t n[3] = {0, 0, 0};
    double lo[3] = {0, 0, 0}, hi[3] = {0, 0, 0}, cell[3] = {0, 0, 0};
    int64_t n_refs = 0;
    std::vector<uint32_t> cells;        // 2 per cell: (first or distance, count)
    std::vector<float> refs;            // n_refs * 12
    std::vector<float> attr;            // n_faces * 8
    std::vector<float> tris;            // n_faces * 12, triangle order
};

// Validate desc and choose bounds and resolution; with fill, also count and
// fill the cell lists (otherwise only n_refs is computed).  Returns a
// mixrt_status and writes a message to msg on failure.
int build_mesh_grid(const mixrt_mesh_desc *desc, bool fill, MeshGridHost &g, char *msg,
                    size_t cap);

// Bytes of device memory an uploaded grid occupies (each array 256-aligned).
int64_t mesh_device_bytes(const MeshGridHost &g, int64_t n_faces);

struct RaycastLaunch {
    MeshGridK grid;
    CamK cams[MIXRT_MAX_VIEWS];
    int32_t views, W, H;
    float4 *g0;
    float4 *g1;
};

hipError_t launch_raycast(const RaycastLaunch &L, hipStream_t stream);

// The rasteriser: per view, triangles are clipped at camera depth near_z
// (chosen on the host so that no hit with t > MIXRT_RAY_T_MIN is closer).
// Pixels per view must be below 2^26 (box areas of a wave sum in 32 bits).
struct RasterLaunch {
    const float4 *tris;
    const float4 *attr;
    int32_t n_faces;
    CamK cams[MIXRT_MAX_VIEWS];
    float near_z[MIXRT_MAX_VIEWS];
    int32_t views, W, H;
    int32_t cus;
    float4 *g0;
    float4 *g1;
    int32_t per_wave;   // triangles per wave (1..64)
    int32_t list_from;  // boxes of more pixels go to the list (0: none do)
};

hipError_t launch_rasterize(const RasterLaunch &L, hipStream_t stream);

}  // namespace mixrt
