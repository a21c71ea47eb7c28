// The coarse-mesh hit per pixel (Fig. 2 step 1) by rasterisation, as the
// paper obtains it, on compute units: a visibility buffer of 64-bit keys
// (t bits << 32 | triangle) kept with atomic min, so the closest hit wins and
// equal t goes to the lower triangle index.  Coverage and depth come from the
// same fp32 ray-triangle test, on the same per-pixel rays, as the ray cast
// (mixrt_raycast.hip).
//
//   clear:   every pixel's key = all ones (no hit);
//   raster:  each wave takes up to 64 triangles of one view (strided over the
//            mesh, for balance between waves), one per lane, clips them against
//            a plane just in front of the camera, projects them and bounds
//            their pixels (one pixel of margin).  Large boxes go to a list.  Of
//            the others the (triangle, pixel) pairs, in box order, are cut into
//            64 equal runs, one per lane, so large and small triangles balance
//            within the wave; a lane finds its first box by binary search and
//            then steps pixel by pixel, box by box, testing with the pixel's ray
//            direction before normalisation (same order of hits).  The boxes
//            with pixels stand first in LDS, so the next box is the next
//            entry: skipping the triangles out of view one by one cost a
//            chain of LDS reads at nearly every step (64x64 15.5 -> 14.1 us).
//            Boxes of kWideMean pixels and more on average are drawn one after
//            another instead, 64 consecutive pixels at a time;
//   list:    the listed boxes, one wave per 1024 pixels of them;
//   resolve: per pixel, the winning triangle's hit is recomputed to write t,
//            the barycentric uv and the face normal.
// The winner of a pixel is the fp32 closest hit of its ray as the ray cast
// finds it, except where two triangles' hits lie within rounding of each
// other.  The keys live in the first 8 bytes of each 16-byte G-buffer record and
// the list in the second: the launches need no memory beyond the caller's output.
//
// What bounds it: the pairs' VALU work in view, the set-up of every triangle and
// the launches out of it.
#include "mixrt_common.hpp"
#include "mixrt_mesh.hpp"

namespace mixrt {

namespace {

constexpr uint64_t kNoHit = ~0ull;

__device__ __forceinline__ bool tri_hit(const float4 &A, const float4 &E1, const float4 &E2,
                                        const Ray &ray, float &t, float &b1, float &b2)
{
    const float px = ray.dy * E2.z - ray.dz * E2.y;
    const float py = ray.dz * E2.x - ray.dx * E2.z;
    const float pz = ray.dx * E2.y - ray.dy * E2.x;
    const float det = E1.x * px + E1.y * py + E1.z * pz;
    const float inv = __builtin_amdgcn_rcpf(det);
    const float sx = ray.ox - A.x, sy = ray.oy - A.y, sz = ray.oz - A.z;
    b1 = (sx * px + sy * py + sz * pz) * inv;
    const float qx = sy * E1.z - sz * E1.y;
    const float qy = sz * E1.x - sx * E1.z;
    const float qz = sx * E1.y - sy * E1.x;
    b2 = (ray.dx * qx + ray.dy * qy + ray.dz * qz) * inv;
    t = (E2.x * qx + E2.y * qy + E2.z * qz) * inv;
    return b1 >= 0.0f && b2 >= 0.0f && b1 + b2 <= 1.0f && t > MIXRT_RAY_T_MIN;
}

// The same test for a ray o + s D with D not normalised: s = t / |D|, so the
// order of hits along the ray is that of t, and t > t_min reads
// s^2 |D|^2 > t_min^2 (dd = |D|^2).  Returns s in `key_t`.
__device__ __forceinline__ bool tri_hit_scaled(const float4 &A, const float4 &E1, const float4 &E2,
                                               float ox, float oy, float oz, float dx, float dy,
                                               float dz, float dd, float &key_t)
{
    const float px = dy * E2.z - dz * E2.y;
    const float py = dz * E2.x - dx * E2.z;
    const float pz = dx * E2.y - dy * E2.x;
    const float det = E1.x * px + E1.y * py + E1.z * pz;
    const float inv = __builtin_amdgcn_rcpf(det);
    const float sx = ox - A.x, sy = oy - A.y, sz = oz - A.z;
    const float b1 = (sx * px + sy * py + sz * pz) * inv;
    const float qx = sy * E1.z - sz * E1.y;
    const float qy = sz * E1.x - sx * E1.z;
    const float qz = sx * E1.y - sy * E1.x;
    const float b2 = (dx * qx + dy * qy + dz * qz) * inv;
    const float s = (E2.x * qx + E2.y * qy + E2.z * qz) * inv;
    key_t = s;
    return b1 >= 0.0f && b2 >= 0.0f && b1 + b2 <= 1.0f && s > 0.0f &&
           s * s * dd > MIXRT_RAY_T_MIN * MIXRT_RAY_T_MIN;
}

__global__ __launch_bounds__(kBlock) void clear_kernel(uint4 *__restrict__ g0, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i < n) g0[i] = make_uint4(0xffffffffu, 0xffffffffu, 0u, 0u);
}

struct Box {
    float4 a, e1, e2;
    int x0, y0, bw, bh;
    uint32_t end;   // inclusive prefix sum of the wave's box areas
};

// Pixel box of a triangle in view c (empty: bw = bh = 0).
__device__ __forceinline__ void pixel_box(const RasterLaunch &L, const CamK &c, float zn,
                                          const float4 &A, const float4 &E1, const float4 &E2,
                                          int &x0, int &y0, int &bw, int &bh)
{
    // camera-space corners: R^T (p - o)
    float X[3], Y[3], Z[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const float wx = A.x + (k == 1 ? E1.x : (k == 2 ? E2.x : 0.0f)) - c.o[0];
        const float wy = A.y + (k == 1 ? E1.y : (k == 2 ? E2.y : 0.0f)) - c.o[1];
        const float wz = A.z + (k == 1 ? E1.z : (k == 2 ? E2.z : 0.0f)) - c.o[2];
        X[k] = c.R[0] * wx + c.R[3] * wy + c.R[6] * wz;
        Y[k] = c.R[1] * wx + c.R[4] * wy + c.R[7] * wz;
        Z[k] = c.R[2] * wx + c.R[5] * wy + c.R[8] * wz;
    }
    // clip against Z = -zn (the polygon in front has at most 4 corners) and
    // bound its projection; pixel i's centre is at W/2 + X/(-Z) f - ... (i + 0.5)
    const float f = 1.0f / c.inv_f;
    float lox = INFINITY, hix = -INFINITY, loy = INFINITY, hiy = -INFINITY;
    auto add = [&](float x, float y, float z) {
        const float s = f / (-z);
        const float sx = 0.5f * (float)L.W + x * s, sy = 0.5f * (float)L.H - y * s;
        lox = fminf(lox, sx);
        hix = fmaxf(hix, sx);
        loy = fminf(loy, sy);
        hiy = fmaxf(hiy, sy);
    };
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const int n = k == 2 ? 0 : k + 1;
        const bool in_k = Z[k] < -zn, in_n = Z[n] < -zn;
        if (in_k) add(X[k], Y[k], Z[k]);
        if (in_k != in_n) {
            const float s = (-zn - Z[k]) / (Z[n] - Z[k]);
            add(X[k] + s * (X[n] - X[k]), Y[k] + s * (Y[n] - Y[k]), -zn);
        }
    }
    x0 = y0 = bw = bh = 0;
    if (!(lox <= hix) || !(loy <= hiy)) return;   // nothing in front, or NaN
    // centres i + 0.5 in [lox, hix], one pixel of margin, clamped in float
    // before the conversion
    const float fx0 = fmaxf(floorf(lox - 0.5f) - 1.0f, 0.0f);
    const float fx1 = fminf(ceilf(hix - 0.5f) + 1.0f, (float)(L.W - 1));
    const float fy0 = fmaxf(floorf(loy - 0.5f) - 1.0f, 0.0f);
    const float fy1 = fminf(ceilf(hiy - 0.5f) + 1.0f, (float)(L.H - 1));
    if (!(fx0 <= fx1) || !(fy0 <= fy1)) return;
    x0 = (int)fx0;
    y0 = (int)fy0;
    bw = (int)fx1 - x0 + 1;
    bh = (int)fy1 - y0 + 1;
}

// One (triangle, pixel) pair: the test with the pixel's ray direction before
// normalisation (as in camera_ray), and the key's atomic minimum.
__device__ __forceinline__ void test_pair(const RasterLaunch &L, const CamK &c, int64_t view_base,
                                          const float4 &A, const float4 &E1, const float4 &E2,
                                          int px, int py)
{
    const float cx = ((float)px + 0.5f - 0.5f * (float)L.W) * c.inv_f;
    const float cy = -(((float)py + 0.5f - 0.5f * (float)L.H) * c.inv_f);
    const float dx = c.R[0] * cx + c.R[1] * cy - c.R[2];
    const float dy = c.R[3] * cx + c.R[4] * cy - c.R[5];
    const float dz = c.R[6] * cx + c.R[7] * cy - c.R[8];
    float st;
    if (tri_hit_scaled(A, E1, E2, c.o[0], c.o[1], c.o[2], dx, dy, dz, dx * dx + dy * dy + dz * dz,
                       st)) {
        const uint64_t key = ((uint64_t)__float_as_uint(st) << 32) | (uint32_t)__float_as_int(A.w);
        atomicMin((unsigned long long *)L.g0 + 2 * (view_base + (int64_t)py * L.W + px),
                  (unsigned long long)key);
    }
}

// The list of large boxes of a view, in the second 8 bytes of the view's G-buffer
// records (which the clear leaves zero and the keys do not touch): kLists parts,
// so that no counter takes every wave's atomic, each with its counter in record
// 16 p (a line of its own) and its entries, (triangle + 1, slice), from record
// kListHead + p part on.  An entry of zero was reserved and not used.
constexpr int kLists = kWave;           // the list kernel's lanes read a counter each
constexpr int kListHead = 16 * kLists;
constexpr int kSlicePixels = 1024, kMaxSlices = 256;
// (499,712 triangles from outside at 1280x720: 60 us, 79 with 40, 129 with 32)
constexpr uint32_t kWideMean = 64;

__device__ __forceinline__ unsigned long long *list_word(const RasterLaunch &L, int64_t view_base,
                                                         int64_t record)
{
    return (unsigned long long *)L.g0 + 2 * (view_base + record) + 1;
}

__device__ __forceinline__ uint32_t list_part(const RasterLaunch &L)
{
    return ((uint32_t)L.W * (uint32_t)L.H - kListHead) / kLists;
}

// Waves that share a listed box: one per kSlicePixels, at most kMaxSlices.
__device__ __forceinline__ uint32_t box_slices(uint32_t area)
{
    const uint32_t n = (area + kSlicePixels - 1) / kSlicePixels;
    return n < kMaxSlices ? n : kMaxSlices;
}

// Sum of v over lanes 0..lane.
__device__ __forceinline__ uint32_t wave_inclusive_sum(uint32_t v, int lane)
{
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        const uint32_t o = __shfl_up(v, d);
        if (lane >= d) v += o;
    }
    return v;
}

// Every n-th 64 pixels of one box, from the `slice`-th on, by a wave whose lanes
// take consecutive pixels (the box and its triangle are uniform).
__device__ __forceinline__ void draw_box(const RasterLaunch &L, const CamK &c, int64_t view_base,
                                         const float4 &A, const float4 &E1, const float4 &E2,
                                         int x0, int y0, int bw, int bh, int slice, int n, int lane)
{
    const int area = bw * bh;   // fewer than 2^26 pixels
    int q = slice * kWave + lane;
    if (q >= area) return;
    const int step = kWave * n;
    int j = q / bw, i = q - j * bw;
    const int dj = step / bw, di = step - dj * bw;
    for (; q < area; q += step) {
        test_pair(L, c, view_base, A, E1, E2, x0 + i, y0 + j);
        i += di;
        j += dj;
        if (i >= bw) {
            i -= bw;
            ++j;
        }
    }
}

// The listed boxes, in slices: a wave draws every n-th 64 pixels of its entry's
// box.  The grid does not know how many entries there are; its waves stride over
// them.
__global__ __launch_bounds__(kBlock) void raster_list_kernel(const RasterLaunch L)
{
    const int view = blockIdx.y;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = threadIdx.x & (kWave - 1);
    const int64_t view_base = (int64_t)view * L.H * L.W;
    const uint32_t part = list_part(L);
    // (64 lines: read once per block)
    __shared__ uint32_t s_count[kLists];
    if (wv == 0) s_count[lane] = (uint32_t)*list_word(L, view_base, 16 * lane);
    __syncthreads();
    const uint32_t count = s_count[lane];
    const uint32_t ends = wave_inclusive_sum(count < part ? count : part, lane);
    const uint32_t total = __builtin_amdgcn_readlane(ends, kWave - 1);
    const CamK &c = L.cams[view];
    for (uint32_t e = blockIdx.x * kWavesPerBlock + wv; e < total; e += gridDim.x * kWavesPerBlock) {
        const int p = __popcll(__ballot(ends <= e));
        const uint32_t first = p ? __builtin_amdgcn_readlane(ends, p - 1) : 0u;
        const uint64_t entry =
            *list_word(L, view_base, kListHead + (int64_t)p * part + (e - first));
        const uint32_t tri1 = __builtin_amdgcn_readfirstlane((uint32_t)entry);
        if (tri1 == 0) continue;
        const int64_t tri = (int64_t)tri1 - 1;
        const float4 A = L.tris[3 * tri], E1 = L.tris[3 * tri + 1], E2 = L.tris[3 * tri + 2];
        int x0, y0, bw, bh;
        pixel_box(L, c, L.near_z[view], A, E1, E2, x0, y0, bw, bh);
        draw_box(L, c, view_base, A, E1, E2, x0, y0, bw, bh, (int)(entry >> 32),
                 (int)box_slices(bw * bh), lane);
    }
}

__device__ __forceinline__ float lane_value(float v, int lane)
{
    return __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(v), lane));
}

__device__ __forceinline__ float4 lane_value(const float4 &v, int lane)
{
    return make_float4(lane_value(v.x, lane), lane_value(v.y, lane), lane_value(v.z, lane),
                       lane_value(v.w, lane));
}

__global__ __launch_bounds__(kBlock) void raster_kernel(const RasterLaunch L)
{
    __shared__ Box s_box[kWavesPerBlock][kWave];
    const int view = blockIdx.y;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = threadIdx.x & (kWave - 1);
    // Triangles are dealt to waves with a stride of the wave count, so that
    // the large boxes of a nearby object (consecutive triangles) spread over
    // many waves instead of piling into a few.
    const int64_t n_waves = (int64_t)gridDim.x * kWavesPerBlock;
    const int64_t wave = (int64_t)blockIdx.x * kWavesPerBlock + wv;
    const int64_t tri = (int64_t)lane * n_waves + wave;
    const int64_t view_base = (int64_t)view * L.H * L.W;
    const CamK &c = L.cams[view];
    Box b;
    b.a = b.e1 = b.e2 = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    b.x0 = b.y0 = b.bw = b.bh = 0;
    if (lane < L.per_wave && tri < L.n_faces) {
        b.a = L.tris[3 * tri];
        b.e1 = L.tris[3 * tri + 1];
        b.e2 = L.tris[3 * tri + 2];
        pixel_box(L, c, L.near_z[view], b.a, b.e1, b.e2, b.x0, b.y0, b.bw, b.bh);
    }
    uint32_t area = (uint32_t)b.bw * (uint32_t)b.bh;
    if (L.list_from > 0) {
        // large boxes go to the list, unless this wave's do not all fit in its
        // part (a part that is full is left alone, so that its counter cannot
        // wrap)
        const uint32_t n = area > (uint32_t)L.list_from ? box_slices(area) : 0u;
        if (__ballot(n > 0)) {
            const uint32_t end = wave_inclusive_sum(n, lane);
            const uint32_t all = __builtin_amdgcn_readlane(end, kWave - 1);
            const uint32_t part = list_part(L);
            const int p = (int)(wave & (kLists - 1));
            unsigned int *const ctr = (unsigned int *)list_word(L, view_base, 16 * p);
            uint32_t base = part;
            if (lane == 0 && __hip_atomic_load(ctr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < part)
                base = atomicAdd(ctr, all);
            base = __builtin_amdgcn_readfirstlane(base);
            if (base + all <= part) {
                unsigned long long *const word =
                    list_word(L, view_base, kListHead + (int64_t)p * part + base + end - n);
                for (uint32_t k = 0; k < n; ++k)
                    __hip_atomic_store(word + 2 * k,
                                       (unsigned long long)k << 32 | (uint32_t)(tri + 1),
                                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (n > 0) area = 0;
            }
        }
    }
    // inclusive prefix sum of the areas of the boxes drawn here
    const uint32_t end = wave_inclusive_sum(area, lane);
    b.end = end;
    // the boxes with pixels first, in order, then the others (whose ends, the
    // total, no run reaches): a lane's next box is the next entry
    const uint64_t live = __ballot(area > 0);
    const int rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(live >> 32),
                                               __builtin_amdgcn_mbcnt_lo((uint32_t)live, 0u));
    const uint32_t total = __builtin_amdgcn_readlane(end, kWave - 1);
    if (total == 0) return;   // (the whole wave)
    if (total >= kWideMean * (uint32_t)__popcll(live)) {
        // one box after another, 64 consecutive pixels at a time
        for (uint64_t m = live; m; m &= m - 1) {
            const int l = __builtin_ctzll(m);
            draw_box(L, c, view_base, lane_value(b.a, l), lane_value(b.e1, l), lane_value(b.e2, l),
                     __builtin_amdgcn_readlane(b.x0, l), __builtin_amdgcn_readlane(b.y0, l),
                     __builtin_amdgcn_readlane(b.bw, l), __builtin_amdgcn_readlane(b.bh, l), 0, 1,
                     lane);
        }
        return;
    }
    if (area > 0)
        s_box[wv][rank] = b;
    else
        s_box[wv][__popcll(live) + lane - rank].end = total;
    wave_lds_sync();
    // this lane's run of pairs [q0, q1)
    const uint32_t q0 = (uint32_t)(((uint64_t)total * lane) >> 6);
    const uint32_t q1 = (uint32_t)(((uint64_t)total * (lane + 1)) >> 6);
    if (q0 >= q1) return;
    // first box whose end exceeds q0
    int cur = 0;
#pragma unroll
    for (int step = kWave / 2; step > 0; step >>= 1)
        if (s_box[wv][cur + step - 1].end <= q0) cur += step;
    const Box *bx = &s_box[wv][cur];
    uint32_t local = q0 - (cur ? s_box[wv][cur - 1].end : 0u);
    int j = (int)(local / (uint32_t)bx->bw);
    int i = (int)(local - (uint32_t)j * (uint32_t)bx->bw);
    float4 A = bx->a, E1 = bx->e1, E2 = bx->e2;
    int x0 = bx->x0, y0 = bx->y0, bw = bx->bw, bh = bx->bh;
    for (uint32_t q = q0; q < q1; ++q) {
        test_pair(L, c, view_base, A, E1, E2, x0 + i, y0 + j);
        if (++i == bw) {
            i = 0;
            if (++j == bh && q + 1 < q1) {
                bx = &s_box[wv][++cur];
                A = bx->a;
                E1 = bx->e1;
                E2 = bx->e2;
                x0 = bx->x0;
                y0 = bx->y0;
                bw = bx->bw;
                bh = bx->bh;
                j = 0;
            }
        }
    }
}

__global__ __launch_bounds__(kBlock) void resolve_kernel(const RasterLaunch L)
{
    const int64_t pix = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const int64_t hw = (int64_t)L.H * L.W;
    if (pix >= (int64_t)L.views * hw) return;
    const uint64_t key = ((const uint64_t *)L.g0)[2 * pix];
    if (key == kNoHit) {
        L.g0[pix] = make_float4(-1.0f, 0.0f, 0.0f, 0.0f);
        if (L.g1) L.g1[pix] = make_float4(0.0f, 0.0f, 0.0f, __int_as_float(-1));
        return;
    }
    const int32_t id = (int32_t)(uint32_t)key;
    const int view = (int)(pix / hw);
    const int64_t rem = pix - (int64_t)view * hw;
    const int py = (int)(rem / L.W), px = (int)(rem - (int64_t)py * L.W);
    const Ray r = camera_ray(L.cams[view], L.W, L.H, (uint32_t)px, (uint32_t)py);
    const float4 A = L.tris[3 * (int64_t)id], E1 = L.tris[3 * (int64_t)id + 1],
                 E2 = L.tris[3 * (int64_t)id + 2];
    float t, b1, b2;
    tri_hit(A, E1, E2, r, t, b1, b2);   // the same arithmetic that won the pixel
    const float4 a0 = L.attr[2 * (int64_t)id], a1 = L.attr[2 * (int64_t)id + 1];
    const float b0 = 1.0f - b1 - b2;
    L.g0[pix] = make_float4(t, b0 * a0.x + b1 * a0.z + b2 * a1.x, b0 * a0.y + b1 * a0.w + b2 * a1.y,
                            0.0f);
    if (L.g1) {
        const float nx = E1.y * E2.z - E1.z * E2.y;
        const float ny = E1.z * E2.x - E1.x * E2.z;
        const float nz = E1.x * E2.y - E1.y * E2.x;
        const float nn = sqrtf(nx * nx + ny * ny + nz * nz);
        const float s = nn > 0.0f ? 1.0f / nn : 0.0f;
        L.g1[pix] = make_float4(nx * s, ny * s, nz * s, __int_as_float(id));
    }
}

}  // namespace

// How a frame's triangles are dealt.  What a view shows is not known here, so the
// deal costs no more than a set-up per triangle, 64 to a wave, where the mesh
// is out of view, and the waves find out what is large:
//  - as few triangles per wave as leave one wave per slot of the card (8 per
//    SIMD): more waves would only queue;
//  - boxes go to the list from the size on at which they would keep their wave
//    busy after the others: 128 pixels where a wave holds 16 triangles or more
//    (499,712 triangles at 1920x1080 115 us, 149 from 256 on; seen from outside
//    at 1280x720 60 us, 71 from 64 on, where most waves pay for an atomic), 768
//    where it holds few (32,000 from outside at 1280x720 33 us from 512 on, 31
//    from 1024; 3,632 inside 33.9 and 35.0);
//  - no list in views of fewer than 2^17 pixels, where its launch costs more
//    than the boxes it would spread.
// Measured, us, 64 triangles in every wave and no list / a wave or more per
// triangle from 6 pixels per triangle on / this; room seen from inside, from
// 120 units away, and behind the camera:
//   499,712 at 1280x720    98 /  88 /  81    32 /  51 /  35    18 /  24 /  23
//   499,712 at 2560x1440  330 / 220 / 166    52 / 226 /  55    36 / 117 /  39
//   125,000 at 1280x720    96 /  66 /  57    20 /  60 /  24    14 /  32 /  19
//     3,632 at 1280x720   896 /  32 /  34    24 /  23 /  19    12 /  18 /  18
// and with one wall close by (499,712 at 2560x1440) 497 / 397 / 96.
static void raster_split(RasterLaunch &L)
{
    constexpr int64_t kListPixels = 1 << 17;
    static_assert(kListPixels >= kListHead + kLists, "the list needs a record per part");
    L.per_wave = 1;
    while (L.per_wave < 64 && (int64_t)L.n_faces * L.views > (int64_t)L.per_wave * 32 * L.cus)
        L.per_wave *= 2;
    L.list_from = (int64_t)L.W * L.H < kListPixels ? 0 : L.per_wave >= 16 ? 128 : 768;
}

hipError_t launch_rasterize(const RasterLaunch &L, hipStream_t stream)
{
    const int64_t pixels = (int64_t)L.views * L.H * L.W;
    const int pix_blocks = (int)((pixels + kBlock - 1) / kBlock);
    hipLaunchKernelGGL(clear_kernel, dim3(pix_blocks), dim3(kBlock), 0, stream, (uint4 *)L.g0,
                       pixels);
    RasterLaunch R = L;
    raster_split(R);
    const int64_t waves = ((int64_t)L.n_faces + R.per_wave - 1) / R.per_wave;
    const unsigned blocks = (unsigned)((waves + kWavesPerBlock - 1) / kWavesPerBlock);
    hipLaunchKernelGGL(raster_kernel, dim3(blocks, L.views), dim3(kBlock), 0, stream, R);
    if (R.list_from > 0)
        // one wave per slot of the card
        hipLaunchKernelGGL(raster_list_kernel, dim3((8 * L.cus + L.views - 1) / L.views, L.views),
                           dim3(kBlock), 0, stream, R);
    hipLaunchKernelGGL(resolve_kernel, dim3(pix_blocks), dim3(kBlock), 0, stream, L);
    return hipGetLastError();
}

}  // namespace mixrt
