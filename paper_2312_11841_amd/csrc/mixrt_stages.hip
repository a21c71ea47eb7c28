// Stage kernels of the MixRT path (the entry points that expose one stage's
// intermediates): they call the same device functions as render_kernel.
#include "mixrt_common.hpp"
#include "mixrt_launch.hpp"

namespace mixrt {

// A block takes kBlock / K whole rays, so that lanes divide only small numbers to
// find their sample.  Bound by VALU issue.  Collected in LDS and stored in whole
// lines, with the camera of a block of one view in scalar registers, it took
// longer (1280x720 at K = 8, the along-ray fp16 map 46.9 against 42.6 us, the
// fp16 vector map of run-time degree 1 82.1 against 73.8), but for the fp16 map
// of degree 2 (88.8 against 97.0; at K = 1 36.0 against 33.0).
constexpr uint32_t kSetupBlocks = (1u << 24) - 1u;   // blocks of one row of the grid

template <int TEX>
__global__ __launch_bounds__(kBlock) void ray_setup_kernel(RayParams rp, float *__restrict__ out_x,
                                                           int32_t *__restrict__ out_hit)
{
    typedef TapsAhead<typename TexOf<TEX>::type, TEX == kTexU8Vec3> TK;
    const uint32_t t = threadIdx.x, K = (uint32_t)rp.K;
    const uint32_t R = kBlock / K;
    // t / K: exact for t < 2^8 and K <= 64
    const uint32_t inv = (65536u + K - 1u) / K;
    const uint32_t r = (t * inv) >> 16, k = t - r * K;
    const uint32_t ray = (blockIdx.y * kSetupBlocks + blockIdx.x) * R + r;
    if (r >= R || ray >= (uint32_t)rp.rays) return;
    const Ray ry = pixel_ray(rp, (int32_t)ray);
    float x0, x1, x2;
    const bool hit = sample_position<TK>(rp, ry, rp.g0[ray], (int)k, x0, x1, x2);
    float *const o = out_x + ((int64_t)ray * K + k) * 3;
    o[0] = x0;
    o[1] = x1;
    o[2] = x2;
    if (out_hit && k == 0) out_hit[ray] = hit ? 1 : 0;
}

template <int F, bool TF16>
__global__ __launch_bounds__(kBlock) void hash_encode_kernel(GridParams gp, const float *__restrict__ x,
                                                             int64_t n, int32_t *out_corner,
                                                             uint32_t *out_idx, float *out_w,
                                                             float *out_feat)
{
    const int64_t s = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (s >= n) return;
    const float x0 = x[3 * s], x1 = x[3 * s + 1], x2 = x[3 * s + 2];
    for (int l = 0; l < gp.L; ++l) {
        // the render kernel's arithmetic, one level at a time (the render
        // kernel's queries lie in [0, 1]^3; here a coordinate outside it is
        // clamped to the grid)
        LevelSetup st;
        float v[8][F], f[F];
        const bool dense = l < gp.n_dense;
        constexpr uint32_t eb = TableEntry<F, TF16>::kBytes;
        level_setup<eb, false>(gp, l, dense, x0, x1, x2, st);
        const void *base = level_base(gp, l, F, TF16);
        if (dense)
            level_fetch<F, TF16, true>(base, st, v);
        else
            level_fetch<F, TF16, false>(base, st, v);
        level_accumulate<F>(st, v, f);
        const int64_t sl = s * gp.L + l;
        if (out_corner)
            for (int a = 0; a < 3; ++a) out_corner[sl * 3 + a] = (int32_t)st.c[a];
        if (out_idx)
            for (int b = 0; b < 8; ++b) out_idx[sl * 8 + b] = st.off[b] / eb;
        if (out_w)
            for (int b = 0; b < 8; ++b) out_w[sl * 8 + b] = corner_weight(st, b);
        if (out_feat)
            for (int i = 0; i < F; ++i) out_feat[s * gp.L * F + l * F + i] = f[i];
    }
}

// Block -> logical block: runs of `run` consecutive blocks go to one XCD
// (hardware block b runs on XCD b mod 8), the XCDs' runs one after another.
// The grid is a multiple of 8 run.
__device__ __forceinline__ int xcd_run_block(int b, int run)
{
    const int turn = b / (8 * run), i = b - turn * (8 * run);
    return turn * (8 * run) + (i & 7) * run + (i >> 3);
}

constexpr int kFeatCols = 32;               // features collected at a time
constexpr int kFeatRow = kFeatCols + 4;     // LDS row, 16-byte multiple

template <int F, bool TF16, int G, bool DENSE, int FORM>
__device__ __forceinline__ void features_of(const GridParams &gp, int l, float x0, float x1,
                                            float x2, float *col)
{
    float f[G][F];
    hash_group<F, TF16, G, DENSE, FORM, false>(gp, l, x0, x1, x2, f);
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
        for (int i = 0; i < F; ++i) col[g * F + i] = f[g][i];
}

// The features alone, which is what a program that keeps them asks for.  A
// wave takes 64 queries, one or two levels' gathers in flight, and collects up to
// 32 features of each in LDS; they leave in rows of 16-byte stores past the
// caches (written once, and the table's lines stay).  Written from the lanes
// as they come, one 4-byte store per feature touches 64 lines and most lines
// come back to memory in pieces: 489 us for the 640x360 view's 1.84 M queries of
// 16 levels against 164 (236 MB written).  Neighbouring waves go to one XCD, whose L2
// serves the voxels they share.
template <int F, bool TF16>
__global__ __launch_bounds__(kBlock) void hash_features_kernel(GridParams gp,
                                                               const float *__restrict__ x,
                                                               int64_t n, int wide, int run,
                                                               float *__restrict__ out)
{
    __shared__ __attribute__((aligned(16))) float s_f[kWavesPerBlock][kWave * kFeatRow];
    const int lane = threadIdx.x & (kWave - 1);
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int64_t base =
        ((int64_t)xcd_run_block((int)blockIdx.x, run) * kWavesPerBlock + wv) * kWave;
    if (base >= n) return;
    const int rows = n - base < kWave ? (int)(n - base) : kWave;
    float x0 = 0.0f, x1 = 0.0f, x2 = 0.0f;   // (lanes past n: voxel 0, never stored)
    if (lane < rows) {
        const float *p = x + 3 * (base + lane);
        x0 = p[0];
        x1 = p[1];
        x2 = p[2];
    }
    float *const buf = s_f[wv];
    const int L = gp.L, LF = L * F;
    constexpr int kLevels = kFeatCols / F;
    // Levels' gathers in flight: two of 4-byte entries (1.84 M scattered queries of
    // 16 levels 1023 us, 1084 with one), one of larger ones, whose queries of small
    // tables they kept waiting (8 levels of 2^14 fp32 pairs 236 us, 252 with two;
    // 8 levels of 2^17 fp32 quads 79 and 89; Tab. 3's 14,400 queries 16.4 and 17.6).
    constexpr int G = F == 2 && TF16 ? 2 : 1;
    for (int l0 = 0; l0 < L; l0 += kLevels) {
        const int l1 = l0 + kLevels < L ? l0 + kLevels : L;
        const int ld = gp.n_dense < l1 ? gp.n_dense : l1;
        const int lb = gp.block_from < l1 ? gp.block_from : l1;
        float *const row = buf + lane * kFeatRow - l0 * F;
        int l = l0;
        for (; l + G <= ld; l += G) features_of<F, TF16, G, true, kEntries>(gp, l, x0, x1, x2, row + l * F);
        for (; l < ld; ++l) features_of<F, TF16, 1, true, kEntries>(gp, l, x0, x1, x2, row + l * F);
        for (; l + G <= lb; l += G) features_of<F, TF16, G, false, kEntries>(gp, l, x0, x1, x2, row + l * F);
        for (; l < lb; ++l) features_of<F, TF16, 1, false, kEntries>(gp, l, x0, x1, x2, row + l * F);
        if constexpr (kBlockPairs<F, TF16> || kBlockPairs8<F, TF16>)
            for (; l < l1; ++l)
                features_of<F, TF16, 1, false, kBlocksWithFar>(gp, l, x0, x1, x2, row + l * F);
        wave_lds_sync();
        const int cols = (l1 - l0) * F;
        float *const o = out + base * LF + l0 * F;
        if (wide) {
            const int per = cols / 4;   // 16-byte chunks per row
            for (int e = lane; e < rows * per; e += kWave) {
                const int r = e / per, c = 4 * (e - r * per);
                __builtin_nontemporal_store(*(const f4 *)(buf + r * kFeatRow + c),
                                            (f4 *)(o + (int64_t)r * LF + c));
            }
        } else {
            for (int e = lane; e < rows * cols; e += kWave) {
                const int r = e / cols, c = e - r * cols;
                __builtin_nontemporal_store(buf[r * kFeatRow + c], o + (int64_t)r * LF + c);
            }
        }
        wave_lds_sync();
    }
}

#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"   // M0 is clobbered on purpose
// One 16-byte chunk per lane straight from global memory into LDS
// (global_load_lds_dwordx4): lane l's chunk lands at lds + 16 l.  M0 is set
// in the same statement; nothing else in this kernel uses it.  The rows are
// read once, so the load is marked non-temporal (nt), as are the output
// stores below: with both, the stage runs about 5% faster than with the
// default cache policy (0.161 against 0.169 ms for 7.37M rows), the writes
// disturbing the read stream less.
__device__ __forceinline__ void lds_load16(const void *g, uint32_t lds)
{
    asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, off nt" ::"s"(
                     __builtin_amdgcn_readfirstlane(lds)),
                 "v"(g)
                 : "memory", "m0");
}
#pragma clang diagnostic pop

// A 16-byte non-temporal vector store, issued as assembly like the loads
// above.
__device__ __forceinline__ void store16(void *g, f4 v)
{
    asm volatile("global_store_dwordx4 %0, %1, off nt" ::"v"(g), "v"(v) : "memory");
}

// Wait until at most N vector-memory operations (loads and stores) of this
// wave are outstanding; they complete in issue order.
template <int N>
__device__ __forceinline__ void wait_vm()
{
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// wait_vm<n> for a wave-uniform n in 0..N
template <int N>
__device__ __forceinline__ void wait_vm_upto(int n)
{
    if constexpr (N == 0) {
        wait_vm<0>();
    } else {
        if (n >= N)
            wait_vm<N>();
        else
            wait_vm_upto<N - 1>(n);
    }
}

// Persistent: weights are loaded once per wave, then 64-row tiles.  A tile's
// rows are one contiguous block of 64 * CH 16-byte chunks, copied to LDS in
// CH coalesced loads, DEPTH tiles ahead of the one being computed; its 64
// outputs are gathered in LDS and written with one coalesced 1 KiB store
// (lane l: row l), the same access pattern as the stream the stage is
// measured against.
//
// The loads and stores of the tile loop are issued as assembly, so that the
// compiler, which sees no memory operation of its own there, places no wait
// of its own: its form of the LDS loads waits for every outstanding vector
// operation before any LDS read, and before inline assembly it drains its
// pending stores; either would serialise the pipelining.  The waits are
// counted instead.  Every tile issues exactly CH loads (the chunks of rows
// past n are read from the last row, and their outputs never stored) and
// exactly kStores stores (the lanes of rows past n masked off; a tile always
// has a row below n).  After the loads of tile k come the stores of the
// min(k, DEPTH) tiles before it and the loads of the tiles after it that are
// already in flight, and that is the count to wait for.
constexpr int kStores = 1;

template <int IN, int HID, int NHID, int DEPTH>
__global__ __launch_bounds__(kBlock) void mlp_kernel(const _Float16 *__restrict__ weights,
                                                     int hid_w, const _Float16 *__restrict__ in,
                                                     int64_t n, float4 *__restrict__ out4)
{
    static_assert(IN % 8 == 0, "rows are moved in 16-byte chunks");
    static_assert(DEPTH >= 1 && DEPTH <= 2, "tiles in flight");
    constexpr int CH = IN / 8;   // 16-byte chunks per row; a tile is CH 1-KiB loads
    constexpr int NB = DEPTH + 1;
    static_assert(DEPTH * (CH + kStores) <= 63, "vmcnt range");
    // NB tile buffers per wave, rows of IN halves back to back
    __shared__ __attribute__((aligned(16))) _Float16 s_rows[kWavesPerBlock][NB][kWave * IN];
    __shared__ f4 s_res[kWavesPerBlock][kWave];
    const int lane = threadIdx.x & (kWave - 1);
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    MlpWeights<IN, HID, NHID> Wt;
    Wt.load(weights, lane, hid_w);
    const int64_t n_tiles = (n + kWave - 1) / kWave;
    const int64_t total = (int64_t)gridDim.x * kWavesPerBlock;
    const int64_t first = (int64_t)blockIdx.x * kWavesPerBlock + wv;
    if (first >= n_tiles) return;
    const int count = (int)((n_tiles - 1 - first) / total) + 1;   // tiles of this wave
    const int64_t last_chunk = n * CH - 1;
    const h8 *chunks = (const h8 *)in;
    const int c = lane & 15, g = lane >> 4;
    auto issue = [&](int k) {
        const int64_t base = (first + (int64_t)k * total) * kWave * CH;
        const uint32_t lds = (uint32_t)(uintptr_t)s_rows[wv][k % NB];
#pragma unroll
        for (int e = 0; e < CH; ++e) {
            const int64_t q = base + lane + kWave * e;
            lds_load16(chunks + (q < last_chunk ? q : last_chunk), lds + 1024u * (uint32_t)e);
        }
    };
    for (int k = 0; k < DEPTH && k < count; ++k) issue(k);
    for (int k = 0; k < count; ++k) {
        if (k + DEPTH < count) issue(k + DEPTH);
        const int ahead = count - 1 - k < DEPTH ? count - 1 - k : DEPTH;
        const int stored = k < DEPTH ? k : DEPTH;
        wait_vm_upto<DEPTH *(CH + kStores)>(ahead * CH + stored * kStores);
        const _Float16 *rows = s_rows[wv][k % NB];
        const int64_t base = (first + (int64_t)k * total) * kWave;
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) {
            const f4 o = mlp_tile<IN, HID, NHID>(Wt, rows + nt * 16 * IN, IN, lane);
            if (g == 0) {
                const float4 a = mlp_activate(o);
                s_res[wv][nt * 16 + c] = f4{a.x, a.y, a.z, a.w};
            }
        }
        wave_lds_sync();
        if (base + lane < n) store16(out4 + base + lane, s_res[wv][lane]);
    }
    wait_vm<0>();
}

// The MLP removed: inputs summed per component (input i feeds output i mod 4).
__global__ __launch_bounds__(kBlock) void sum_head_kernel(const _Float16 *__restrict__ in, int width,
                                                          int64_t n, float4 *__restrict__ out4)
{
    const int64_t s = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (s >= n) return;
    float acc[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    for (int i = 0; i < width; ++i) acc[i & 3] += (float)in[s * width + i];
    out4[s] = mlp_activate(f4{acc[0], acc[1], acc[2], acc[3]});
}

// One lane per ray, each loading its ray's samples: see composite_by_lane for
// where.
__global__ __launch_bounds__(kBlock) void composite_lane_kernel(const float4 *__restrict__ srgb,
                                                                int64_t rays, int K, float delta,
                                                                float t_term, float bg0, float bg1,
                                                                float bg2, float4 *__restrict__ out)
{
    const int64_t r = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (r >= rays) return;
    Composite cp;
    for (int k = 0; k < K; ++k)
        if (!cp.add(srgb[r * K + k], delta, t_term)) break;
    out[r] = cp.finish(bg0, bg1, bg2);
}

// A wave composites 64 rays, kCompSamples samples of each at a time: a ray's
// are one contiguous run, which the wave loads in 16-byte lanes, takes to
// opacities at once, and leaves in LDS for the ray's lane to add in order.
// With one lane reading its ray's samples from memory, each load touches 64
// lines of which the next needs the same 64 again, more than the L1 keeps:
// 123 us for 921,600 rays of 8 samples against 22 (133 MB moved, 6 TB/s).  Once
// every ray of the wave has stopped the rest is not read.
constexpr int kCompSamples = 8;
constexpr int kCompRow = kCompSamples + 1;   // LDS row in samples, against bank conflicts

__global__ __launch_bounds__(kBlock) void composite_kernel(const float4 *__restrict__ srgb,
                                                           int64_t rays, int K, float delta,
                                                           float t_term, float bg0, float bg1,
                                                           float bg2, float4 *__restrict__ out)
{
    __shared__ float4 s_s[kWavesPerBlock][kWave * kCompRow];
    const int lane = threadIdx.x & (kWave - 1);
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int64_t base = ((int64_t)blockIdx.x * kWavesPerBlock + wv) * kWave;
    if (base >= rays) return;
    const int n = rays - base < kWave ? (int)(rays - base) : kWave;
    float4 *const buf = s_s[wv];
    const f4 *const src = (const f4 *)srgb + base * K;
    Composite cp;
    bool going = lane < n;
    for (int k0 = 0; k0 < K && __ballot(going); k0 += kCompSamples) {
        const int kc = K - k0 < kCompSamples ? K - k0 : kCompSamples;
        if (n == kWave && kc == kCompSamples) {
            // the usual case: all loads in flight, 8 lanes on a ray's 128 bytes
            f4 v[kCompSamples];
            const f4 *const p = src + (int64_t)(lane >> 3) * K + k0 + (lane & 7);
#pragma unroll
            for (int i = 0; i < kCompSamples; ++i)
                v[i] = __builtin_nontemporal_load(p + (int64_t)(8 * i) * K);
#pragma unroll
            for (int i = 0; i < kCompSamples; ++i)
                buf[((lane >> 3) + 8 * i) * kCompRow + (lane & 7)] = Composite::opacity(
                    make_float4(v[i][0], v[i][1], v[i][2], v[i][3]), delta);
        } else {
            for (int e = lane; e < n * kc; e += kWave) {
                const int r = e / kc, k = e - r * kc;
                const f4 v = __builtin_nontemporal_load(src + (int64_t)r * K + k0 + k);
                buf[r * kCompRow + k] =
                    Composite::opacity(make_float4(v[0], v[1], v[2], v[3]), delta);
            }
        }
        wave_lds_sync();
        for (int k = 0; k < kc && going; ++k) going = cp.blend(buf[lane * kCompRow + k], t_term);
        wave_lds_sync();
    }
    if (lane < n) out[base + lane] = cp.finish(bg0, bg1, bg2);
}

#define MIXRT_MLP_VARIANTS(X) \
    X(32, 16, 2)              \
    X(16, 32, 1)              \
    X(32, 32, 1)              \
    X(48, 64, 2)              \
    X(32, 64, 2)              \
    X(16, 64, 2)

bool mlp_variant_supported(int in, int hid, int nhid)
{
    if (nhid == 0) return in >= 4 && in % 4 == 0;
#define X(d, e, f) \
    if (in == d && hid == e && nhid == f) return true;
    MIXRT_MLP_VARIANTS(X)
#undef X
    return false;
}

hipError_t launch_ray_setup(const RayParams &rp, int tex, float *out_x, int32_t *out_hit,
                            hipStream_t stream)
{
    if (rp.rays == 0) return hipSuccess;
    const int R = kBlock / rp.K;   // rays per block (K is at most 64)
    // A launch holds fewer than 2^32 threads in x.  A block whose K does not
    // divide it leaves lanes idle, so frames of fewer than 2^32 samples may
    // need a second row of blocks.
    const int64_t blocks = ((int64_t)rp.rays + R - 1) / R;
    const dim3 grid((unsigned)(blocks < kSetupBlocks ? blocks : kSetupBlocks),
                    (unsigned)((blocks + kSetupBlocks - 1) / kSetupBlocks));
#define T(ID)                                                                                  \
    case ID:                                                                                   \
        hipLaunchKernelGGL(ray_setup_kernel<ID>, grid, dim3(kBlock), 0, stream, rp, out_x, out_hit); \
        break;
    switch (tex) {
        T(kTexF32Ray) T(kTexF16Ray) T(kTexU8Ray) T(kTexF32Vec3D1) T(kTexF16Vec3D2) T(kTexU8Vec3D2)
        T(kTexNone) T(kTexF32Vec3) T(kTexF16Vec3) T(kTexU8Vec3)
    default: return hipErrorInvalidValue;
    }
#undef T
    return hipGetLastError();
}

hipError_t launch_hash_encode(const GridParams &gp, int F, bool tf16, const float *x, int64_t n,
                              int32_t *oc, uint32_t *oi, float *ow, float *of, hipStream_t stream)
{
    if (n == 0) return hipSuccess;
    if (of && !oc && !oi && !ow) {
        GridParams g = gp;
        // the finest hashed levels in 16-byte blocks: 6 of 4-byte entries, 3 of
        // 8-byte ones (the 640x360 view's 1.84 M queries along rays 167 us with 3,
        // 164 with 6 and with 9; Tab. 3's 8 levels of 8-byte entries 126 with none,
        // 130 with 3, 132 with 6, and 4 levels of 2^21 of them at scattered
        // positions 543, 532)
        const int from = tf16 ? g.L - (F == 2 ? 6 : 3) : g.L;
        g.block_from = from > g.n_dense ? from : g.n_dense;
        const int wide = (g.L * F) % 4 == 0 && ((uintptr_t)of & 15) == 0;
        const int64_t nb = (n + kBlock - 1) / kBlock;
        // Runs of 64 blocks keep neighbouring queries in one L2 (1280x720 queries
        // of one sample per pixel 157 us without runs, 139 in runs of 16, 130 of
        // 64), 8 or more of them per XCD keep the XCDs evenly loaded (the 1.84 M
        // queries in one run per XCD: 227 us)
        const int64_t run = nb / 64 < 1 ? 1 : nb / 64 > 64 ? 64 : nb / 64;
        const dim3 grid((unsigned)((nb + 8 * run - 1) / (8 * run) * (8 * run)));
#define LAUNCH(FF, TT)                                                                         \
    hipLaunchKernelGGL((hash_features_kernel<FF, TT>), grid, dim3(kBlock), 0, stream, g, x, n,  \
                       wide, (int)run, of)
        if (F == 2 && tf16) LAUNCH(2, true);
        else if (F == 2) LAUNCH(2, false);
        else if (F == 4 && tf16) LAUNCH(4, true);
        else if (F == 4) LAUNCH(4, false);
        else return hipErrorInvalidValue;
#undef LAUNCH
        return hipGetLastError();
    }
    const dim3 grid((unsigned)((n + kBlock - 1) / kBlock));
#define LAUNCH(FF, TT)                                                                         \
    hipLaunchKernelGGL((hash_encode_kernel<FF, TT>), grid, dim3(kBlock), 0, stream, gp, x, n, oc, \
                       oi, ow, of)
    if (F == 2 && tf16) LAUNCH(2, true);
    else if (F == 2) LAUNCH(2, false);
    else if (F == 4 && tf16) LAUNCH(4, true);
    else if (F == 4) LAUNCH(4, false);
    else return hipErrorInvalidValue;
#undef LAUNCH
    return hipGetLastError();
}

// Tiles each wave has in flight beyond the one it computes.  One tile ahead
// leaves room in LDS for 3 blocks per CU (2 at two ahead) and, with the
// non-temporal loads and stores, runs about 2.5% faster (0.157 against 0.161
// ms for 7.37M rows of 48).
constexpr int kMlpDepth = 1;

hipError_t launch_mlp(int in, int hid, int nhid, int hid_w, const _Float16 *weights,
                      const _Float16 *x, int64_t n, float4 *out4, int cus, hipStream_t stream)
{
    if (n == 0) return hipSuccess;
    if (nhid == 0) {
        hipLaunchKernelGGL(sum_head_kernel, dim3((unsigned)((n + kBlock - 1) / kBlock)),
                           dim3(kBlock), 0, stream, x, in, n, out4);
        return hipGetLastError();
    }
    const int64_t want = ((n + kWave - 1) / kWave + kWavesPerBlock - 1) / kWavesPerBlock;
#define X(d, e, f)                                                                           \
    if (in == d && hid == e && nhid == f) {                                                  \
        auto fn = mlp_kernel<d, e, f, kMlpDepth>;                                            \
        static std::atomic<int> per_cu{0};                                                   \
        const int64_t resident = (int64_t)blocks_per_cu((const void *)fn, per_cu) * cus;     \
        const int64_t blocks = want < resident ? want : resident;                            \
        hipLaunchKernelGGL(fn, dim3((unsigned)blocks), dim3(kBlock), 0, stream, weights, hid_w, \
                           x, n, out4);                                                      \
        return hipGetLastError();                                                            \
    }
    MIXRT_MLP_VARIANTS(X)
#undef X
    return hipErrorInvalidValue;
}

// Whether each lane loads its own ray's samples.  Up to 4 samples are half a line,
// which the L1 keeps until the lane's next ones (921,600 rays, us by lane / through
// LDS, from the last level cache: K = 2 6.8 / 10.8, 3 11.4 / 13.9, 4 16.3 / 17.1, 5
// 30.1 / 20.0; from memory 9.8 / 11.3, 13.3 / 14.7, 17.9 / 17.9, 31.8 / 20.8).  With
// fewer than three waves per CU the L1 keeps every ray's lines, and the lane's
// chain of loads is shorter than the chunks' (K = 64: 14,400 rays 10.3 / 12.7, 32,768
// 11.4 / 13.4, 65,536 15.7 / 15.1; K = 32: 6.2 / 7.6, 6.5 / 8.0, 7.0 / 8.4).
static bool composite_by_lane(int64_t rays, int K) { return K <= 4 || rays < 3 * 256 * kWave; }

hipError_t launch_composite(const float4 *srgb, int64_t rays, int K, float delta, float t_term,
                            const float *bg, float4 *out, hipStream_t stream)
{
    if (rays == 0) return hipSuccess;
    const dim3 grid((unsigned)((rays + kBlock - 1) / kBlock));
    hipLaunchKernelGGL(composite_by_lane(rays, K) ? composite_lane_kernel : composite_kernel, grid,
                       dim3(kBlock), 0, stream, srgb, rays, K, delta, t_term, bg[0], bg[1], bg[2],
                       out);
    return hipGetLastError();
}

}  // namespace mixrt
