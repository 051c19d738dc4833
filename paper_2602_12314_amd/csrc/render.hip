// Query-map rendering (paper Eq. 2 and Eq. 4) and its adjoint on gfx950.
//
// Pipeline of one forward call (one HIP stream, no host synchronisation):
//   k_preprocess      one thread per (camera, Gaussian) record, float32 projection:
//                     screen mean, conic, opacity, integer footprint, depth key
//   sort              visible records by float32 depth bits (stable: ties by
//                     record): in one launch up to 4096 records, else by radix
//   scan + k_emit     (tile id, record) pairs emitted in depth order
//   radix sort        pairs by tile id (stable, so each tile stays depth-ordered)
//   k_ranges          [start, end) of every tile's list
//   k_raster_fwd      one workgroup per tile, one wave per 64 pixels of it; a
//                     wave takes the list 64 entries at a time, keeps those that
//                     reach its pixels and blends them on the matrix cores
// The backward (k_raster_bwd, after k_clear_grads) walks each pixel's list back
// to front in batches of 16 entries, rebuilding the transmittance by division,
// forms the per-Gaussian sums over the wave's pixels by matrix and vector
// operations and adds them to memory with one atomic per sum and wave;
// k_preprocess_bwd chains the screen-space gradients to the raw parameters.
#include "common.h"
#include "kernels.h"

namespace lam {

// ------------------------------------------------------------- preprocess

// exp(x) in float32 by Cody-Waite reduction and a Taylor polynomial: k =
// rint(x log2 e), r = (x - k ln2_hi) - k ln2_lo with ln2_hi carrying 15
// significant bits (so k ln2_hi is exact for |k| < 256), exp(r) to degree 7 by
// Horner with fused multiply-adds (|r| <= ln2 / 2: truncation below 2^-25),
// scaled by 2^k.  Every step is a correctly rounded float32 operation, so the
// result is a fixed function of x, reproducible bit for bit by any IEEE float32
// implementation of the same steps.
__device__ inline float exp_cw(float x)
{
#pragma clang fp contract(off)
    x = fminf(fmaxf(x, -87.0f), 88.0f);
    const float k = rintf(x * 1.44269504f);
    const float r = (x - k * 0.693145751953125f) - k * 1.42860677e-06f;
    float p = 1.0f / 5040.0f;
    p = fmaf(p, r, 1.0f / 720.0f);
    p = fmaf(p, r, 1.0f / 120.0f);
    p = fmaf(p, r, 1.0f / 24.0f);
    p = fmaf(p, r, 1.0f / 6.0f);
    p = fmaf(p, r, 0.5f);
    p = fmaf(p, r, 1.0f);
    p = fmaf(p, r, 1.0f);
    return ldexpf(p, (int)k);
}

// Record outputs: rec0 = (u, v, first tile, tiles per footprint row | tiles per
// view row << 16) (the last two words as bits, for k_emit), rec1 = (A, B, C,
// opacity) with power = -0.5 (A dx^2 + C dy^2) - B dx dy, foot = (x0 | x1 << 16,
// y0 | y1 << 16) the inclusive pixel footprint.
//
// The projection is float32 with every operation written out and rounded on
// its own (no contraction; division and square root correctly rounded;
// exp_cw above), in the order below, so that the integer decisions it takes
// (culling, radius, footprint, depth key) are a fixed function of the float32
// inputs.
//
// The launch also clears the forward's counters and look-back scratch
// (zero[0 .. zero_words)), which the sorts after it need at zero: one launch
// fewer than a separate fill.
__global__ __launch_bounds__(256) void k_preprocess(
    CamSet cs, int N, const float* __restrict__ means, const float* __restrict__ log_scales,
    const float* __restrict__ quats, const float* __restrict__ logits, float4* __restrict__ rec0,
    float4* __restrict__ rec1, uint2* __restrict__ foot, uint32_t* __restrict__ depth_key,
    uint32_t* __restrict__ ntiles, uint32_t* __restrict__ zero, size_t zero_words)
{
#pragma clang fp contract(off)
    {
        const size_t nthreads = (size_t)gridDim.x * gridDim.y * blockDim.x;
        for (size_t k = ((size_t)blockIdx.y * gridDim.x + blockIdx.x) * blockDim.x + threadIdx.x; k < zero_words;
             k += nthreads)
            zero[k] = 0u;
    }
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= N) return;
    const Cam& cam = cs.c[blockIdx.y];
    const size_t r = (size_t)blockIdx.y * N + i;

    const float mx = means[3 * i], my = means[3 * i + 1], mz = means[3 * i + 2];
    float Wm[3][3], t[3];
    for (int a = 0; a < 3; ++a) {
        for (int b = 0; b < 3; ++b) Wm[a][b] = cam.vm[4 * a + b];
        t[a] = cam.vm[4 * a + 3];
    }
    const float x = ((Wm[0][0] * mx + Wm[0][1] * my) + Wm[0][2] * mz) + t[0];
    const float y = ((Wm[1][0] * mx + Wm[1][1] * my) + Wm[1][2] * mz) + t[1];
    const float z = ((Wm[2][0] * mx + Wm[2][1] * my) + Wm[2][2] * mz) + t[2];

    bool vis = z > kNear;
    float s[3], qn[4];
    if (vis) {
        for (int k = 0; k < 3; ++k) s[k] = exp_cw(log_scales[3 * i + k]);
        const float q0 = quats[4 * i], q1 = quats[4 * i + 1], q2 = quats[4 * i + 2], q3 = quats[4 * i + 3];
        const float nrm = sqrtf(((q0 * q0 + q1 * q1) + q2 * q2) + q3 * q3);
        vis = nrm > 0.0f;
        qn[0] = q0 / nrm; qn[1] = q1 / nrm; qn[2] = q2 / nrm; qn[3] = q3 / nrm;
    }
    float a = 0, b = 0, c = 0, det = 0, u = 0, v = 0, radius = 0;
    if (vis) {
        const float w = qn[0], qx = qn[1], qy = qn[2], qz = qn[3];
        const float Rg[3][3] = {
            {1.0f - 2.0f * (qy * qy + qz * qz), 2.0f * (qx * qy - w * qz), 2.0f * (qx * qz + w * qy)},
            {2.0f * (qx * qy + w * qz), 1.0f - 2.0f * (qx * qx + qz * qz), 2.0f * (qy * qz - w * qx)},
            {2.0f * (qx * qz - w * qy), 2.0f * (qy * qz + w * qx), 1.0f - 2.0f * (qx * qx + qy * qy)}};
        float S3[3][3], Sc[3][3];
        for (int p = 0; p < 3; ++p)
            for (int q = 0; q < 3; ++q) {
                float acc = 0.0f;
                for (int k = 0; k < 3; ++k) acc = acc + ((Rg[p][k] * s[k]) * s[k]) * Rg[q][k];
                S3[p][q] = acc;
            }
        for (int p = 0; p < 3; ++p)
            for (int q = 0; q < 3; ++q) {
                float acc = 0.0f;
                for (int k = 0; k < 3; ++k)
                    for (int l = 0; l < 3; ++l) acc = acc + (Wm[p][k] * S3[k][l]) * Wm[q][l];
                Sc[p][q] = acc;
            }
        const float fx = cam.fx, fy = cam.fy;
        const float limx = kFovClamp * ((float)cam.w / (2.0f * fx));
        const float limy = kFovClamp * ((float)cam.h / (2.0f * fy));
        float tx = x / z, ty = y / z;
        tx = tx < -limx ? -limx : (tx > limx ? limx : tx);
        ty = ty < -limy ? -limy : (ty > limy ? limy : ty);
        const float J[2][3] = {{fx / z, 0.0f, (-fx * tx) / z}, {0.0f, fy / z, (-fy * ty) / z}};
        float cov[2][2];
        for (int p = 0; p < 2; ++p)
            for (int q = 0; q < 2; ++q) {
                float acc = 0.0f;
                for (int k = 0; k < 3; ++k)
                    for (int l = 0; l < 3; ++l) acc = acc + (J[p][k] * Sc[k][l]) * J[q][l];
                cov[p][q] = acc;
            }
        a = cov[0][0] + kDilation;
        b = cov[0][1];
        c = cov[1][1] + kDilation;
        det = a * c - b * b;
        vis = det > 0.0f;
        if (vis) {
            const float mid = 0.5f * (a + c);
            const float lam = mid + sqrtf(fmaxf(kEigFloor, mid * mid - det));
            radius = ceilf(kSigmas * sqrtf(lam));
            u = (fx * x) / z + cam.cx;
            v = (fy * y) / z + cam.cy;
            vis = (u + radius >= 0.0f) && (u - radius <= (float)(cam.w - 1)) && (v + radius >= 0.0f) &&
                  (v - radius <= (float)(cam.h - 1));
        }
    }
    int x0 = 0, x1 = -1, y0 = 0, y1 = -1;
    if (vis) {
        const float fx0 = ceilf(u - radius), fx1 = floorf(u + radius);
        const float fy0 = ceilf(v - radius), fy1 = floorf(v + radius);
        x0 = fx0 < 0.0f ? 0 : (int)fx0;
        x1 = fx1 > (float)(cam.w - 1) ? cam.w - 1 : (int)fx1;
        y0 = fy0 < 0.0f ? 0 : (int)fy0;
        y1 = fy1 > (float)(cam.h - 1) ? cam.h - 1 : (int)fy1;
        vis = x0 <= x1 && y0 <= y1;
    }
    if (!vis) {
        depth_key[r] = 0xFFFFFFFFu;
        ntiles[r] = 0u;
        foot[r] = make_uint2(0u, 0u);
        return;
    }
    const float o = 1.0f / (1.0f + exp_cw(-logits[i]));
    rec1[r] = make_float4(c / det, -b / det, a / det, o);
    foot[r] = make_uint2((uint32_t)x0 | ((uint32_t)x1 << 16), (uint32_t)y0 | ((uint32_t)y1 << 16));
    depth_key[r] = __float_as_uint(z);
    const int nx = (x1 >> cs.tile_shift_x) - (x0 >> cs.tile_shift_x) + 1;
    const int ny = (y1 >> cs.tile_shift_y) - (y0 >> cs.tile_shift_y) + 1;
    ntiles[r] = (uint32_t)(nx * ny);
    const int tx0 = x0 >> cs.tile_shift_x, ty0 = y0 >> cs.tile_shift_y;
    rec0[r] = make_float4(u, v, __uint_as_float((uint32_t)(cam.tile_base + ty0 * cam.tiles_x + tx0)),
                          __uint_as_float((uint32_t)nx | ((uint32_t)cam.tiles_x << 16)));
}

// One thread per emitted (tile id, record) pair, so Gaussians covering many
// tiles do not serialise one thread.  Pair o belongs to the depth-sorted
// record s with offsets[s] <= o < offsets[s + 1], and is that record's
// (o - offsets[s])-th tile of its footprint, rows outer.  A workgroup takes
// chunks of 256 consecutive pairs, a contiguous range of them: every visible
// record emits at least one pair and culled records are not in the sorted
// list, so a chunk's pairs belong to a run of at most 256 consecutive
// records (counters[5] of them).  The run's offsets are staged in LDS and each thread finds its
// record there.  The first record of the workgroup's first chunk is found by
// rounds of 256 probes, each narrowing the range 256-fold (three rounds for
// up to 2^24 records instead of one dependent load per halving); that of each
// later chunk is read off the staged run of the chunk before it, unless the
// run ends first (then the probes again).
__global__ __launch_bounds__(256) void k_emit(const uint32_t* __restrict__ sorted_rec,
                                             const uint32_t* __restrict__ offsets,
                                             const float4* __restrict__ rec0,
                                             const uint32_t* __restrict__ counters, uint32_t cap,
                                             uint32_t* __restrict__ keys,
                                             uint32_t* __restrict__ vals)
{
    __shared__ uint32_t run[257];
    __shared__ uint32_t next_s0;
    const uint32_t total = counters[0] < cap ? counters[0] : cap, R = counters[5];
    const uint32_t nchunks = (total + 255) / 256;
    const uint32_t per = (nchunks + gridDim.x - 1) / gridDim.x;
    const uint32_t c0 = blockIdx.x * per;
    const uint32_t c1 = c0 + per < nchunks ? c0 + per : nchunks;
    bool known = false;  // next_s0 holds the first record of chunk c
    for (uint32_t c = c0; c < c1; ++c) {
        const uint32_t o0 = c * 256u;
        uint32_t s0;
        if (known) {
            s0 = next_s0;
        } else {
            // largest s in [lo, hi) with offsets[s] <= o0 (offsets[0] = 0 <= o0)
            uint32_t lo = 0, hi = R;
            while (hi - lo > 1) {
                const uint32_t stride = (hi - lo + 255) / 256;
                const uint32_t idx = lo + threadIdx.x * stride;
                const int le = idx < hi && offsets[idx] <= o0;
                const uint32_t k = (uint32_t)__syncthreads_count(le);  // a prefix of the probes
                const uint32_t nlo = lo + (k - 1) * stride;
                hi = nlo + stride < hi ? nlo + stride : hi;
                lo = nlo;
            }
            s0 = lo;
        }
        const uint32_t si = s0 + threadIdx.x;
        run[threadIdx.x] = si < R ? offsets[si] : 0xFFFFFFFFu;
        if (threadIdx.x == 0) run[256] = s0 + 256 < R ? offsets[s0 + 256] : 0xFFFFFFFFu;
        __syncthreads();
        const uint32_t o = o0 + threadIdx.x;
        if (o < total) {
            uint32_t a = 0, b = 257;  // largest j with run[j] <= o; run[0] <= o
            while (b - a > 1) {
                const uint32_t m = (a + b) >> 1;
                if (run[m] <= o) a = m;
                else b = m;
            }
            const uint32_t s = s0 + a;
            const uint32_t r = sorted_rec[s];
            const float2 z = *reinterpret_cast<const float2*>(&rec0[r].z);
            const uint32_t first = __float_as_uint(z.x), nx = __float_as_uint(z.y) & 0xFFFFu;
            // row and column of the footprint's k-th tile: the reciprocal is
            // within one of k / nx (k is below 2^21)
            const uint32_t k = o - run[a];
            uint32_t row = (uint32_t)((float)k * __builtin_amdgcn_rcpf((float)nx));
            if (row * nx > k) --row;
            uint32_t colm = k - row * nx;
            if (colm >= nx) {
                ++row;
                colm -= nx;
            }
            keys[o] = first + row * (__float_as_uint(z.y) >> 16) + colm;
            vals[o] = r;
        }
        // the next chunk's first record: the largest j with run[j] <= o0 + 256,
        // if the run reaches past that pair (run[256] > o0 + 256)
        const uint32_t on = o0 + 256u;
        known = run[256] > on;
        if (known && threadIdx.x == 0) {
            uint32_t a = 0, b = 257;
            while (b - a > 1) {
                const uint32_t m = (a + b) >> 1;
                if (run[m] <= on) a = m;
                else b = m;
            }
            next_s0 = s0 + a;
        }
        __syncthreads();  // run[] is rewritten by the next chunk; next_s0 is read
    }
}

__global__ __launch_bounds__(256) void k_fill_u32(uint32_t* p, size_t n, uint32_t v)
{
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n;
         i += (size_t)gridDim.x * blockDim.x)
        p[i] = v;
}

// [start, end) of every tile's list in the tile-sorted pairs, empty tiles
// included, with no fill first: boundary i (0 <= i <= n) looks at the keys on
// both sides and, where they differ, ends the tile before, starts the tile
// after and gives every tile id strictly between them the empty range (0, 0).
__global__ __launch_bounds__(256) void k_ranges(const uint32_t* __restrict__ keys,
                                               const uint32_t* __restrict__ counters, uint32_t cap,
                                               uint32_t tiles, uint2* __restrict__ ranges)
{
    const uint32_t n = counters[0] < cap ? counters[0] : cap;
    // four boundaries a thread, their keys one 16-byte load
    for (uint32_t i0 = (blockIdx.x * blockDim.x + threadIdx.x) * 4; i0 <= n; i0 += gridDim.x * blockDim.x * 4) {
        uint32_t k[5];
        k[0] = i0 > 0 ? keys[i0 - 1] : 0u;
        if (i0 + 4 <= n) {
            const uint4 v = *reinterpret_cast<const uint4*>(keys + i0);
            k[1] = v.x; k[2] = v.y; k[3] = v.z; k[4] = v.w;
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) k[j + 1] = i0 + j < n ? keys[i0 + j] : tiles;
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint32_t i = i0 + j, a = k[j], b = k[j + 1];
            if (i > n || (i > 0 && i < n && a == b)) continue;
            if (i > 0 && a < tiles) ranges[a].y = i;
            for (uint32_t t = i > 0 ? a + 1 : 0u; t < b && t < tiles; ++t) ranges[t] = make_uint2(0u, 0u);
            if (i < n && b < tiles) ranges[b].x = i;
        }
    }
}

// ------------------------------------------------------ compositing: blocks

// The compositing kernels work wave by wave: a wave owns a block of 64 pixels
// of its tile (8 x 8 where the tile is at least that in both directions; lane
// p is pixel (p % bw, p / bw) of it) and walks the tile's list by itself, with
// no barrier.  It takes the list 64 entries at a time, one per lane: the lane
// builds the 64-bit mask of the block's pixels inside its entry's footprint
// and drops the entry when the footprint misses the block or no pixel of the
// block can reach the alpha threshold (block_reached).  Only the entries that
// are left are visited, by all lanes, in list order.
//
// The sums over the query channels run on the matrix cores in float32: the
// blend acc[pixel][k] += w[pixel] q[k] as a K = 1 outer product (lane = pixel
// on one side, lane = channel on the other), and in the backward the dot
// products q . dQ and the sums over the pixels as K = 4 products.  With one
// lane per pixel and the channels in registers, the same sums read every
// channel of every entry through LDS broadcasts (8 cycles of the CU's one LDS
// pipe per 16 bytes and wave) and the backward spent most of its vector
// operations per entry on channels and wave sums.  Measured, that -> now:
// forward 106 -> 49 us and backward 256 -> 109 us at 640x480 with 100k
// Gaussians (d = 16), 333 -> 151 us and 830 -> 392 us at 1200x680 with 2M
// (d = 32).

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kList = 64;  // list entries taken at a time, one per lane
constexpr int kGroup = 4;  // entries left of them that the forward visits at a time

// The wave's block of the tile: x0, y0 its first pixel, width 1 << sx.
// rows has the bit of each row's first pixel.
struct Block {
    int x0, y0, sx, w, h;
    unsigned long long rows;
};

__device__ inline Block wave_block(const CamSet& cs, const Cam& cam, int tile)
{
    const int lt = tile - cam.tile_base;
    const int tyi = lt / cam.tiles_x, txi = lt - tyi * cam.tiles_x;
    Block b;
    b.sx = min(6 - min(3, cs.tile_shift_y), cs.tile_shift_x);
    b.w = 1 << b.sx;
    b.h = kWave >> b.sx;
    const int nx = cs.tile_shift_x - b.sx;  // log2 of the blocks per tile row
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    b.x0 = (txi << cs.tile_shift_x) + ((w & ((1 << nx) - 1)) << b.sx);
    b.y0 = (tyi << cs.tile_shift_y) + (w >> nx) * b.h;
    b.rows = 0ull;
    for (int y = 0; y < b.h; ++y) b.rows |= 1ull << (y << b.sx);
    return b;
}

// Mask of the block's pixels (bit = lane) inside footprint f.
__device__ inline unsigned long long block_mask(const Block& b, uint2 f)
{
    const int xa = max((int)(f.x & 0xFFFF) - b.x0, 0), xb = min((int)(f.x >> 16) - b.x0, b.w - 1);
    const int ya = max((int)(f.y & 0xFFFF) - b.y0, 0), yb = min((int)(f.y >> 16) - b.y0, b.h - 1);
    if (xa > xb || ya > yb) return 0ull;
    const unsigned long long cols = (2ull << xb) - (1ull << xa);
    return (cols * b.rows) & ((2ull << (((yb + 1) << b.sx) - 1)) - (1ull << (ya << b.sx)));
}

// o G(p) of one pair.  Both directions take their decisions (alpha threshold,
// clamp, termination) from these float32 steps, written out so that they
// round alike wherever they are inlined.
__device__ inline float pair_og(float u, float v, float A, float B, float C, float o, float px, float py)
{
#pragma clang fp contract(off)
    const float dx = u - px, dy = v - py;
    const float q = fmaf(dx, dx * A, dy * (dy * C));
    const float power = fmaf(q, -0.5f, -(dy * (dx * B)));
    return o * __builtin_amdgcn_exp2f(power * 1.44269504f);
}

// False only when every pixel of the block has o G < 1/255: the least of
// q(dx, dy) = A dx^2 + 2 B dx dy + C dy^2 over the block's rectangle (zero if
// it holds the centre, else on one of its edges) is compared with
// 2 ln(255 o).  The slack covers the rounding of pair_og (a few ulp of the
// terms of q, which may cancel) many times over; anything undecided (NaN, a
// conic that is not positive definite) is kept.
__device__ inline bool block_reached(const Block& b, float u, float v, float A, float B, float C, float o)
{
    const float xl = u - (float)(b.x0 + b.w - 1), xh = u - (float)b.x0;
    const float yl = v - (float)(b.y0 + b.h - 1), yh = v - (float)b.y0;
    if (!(A > 0.0f && C > 0.0f && A * C > B * B)) return true;
    if (xl <= 0.0f && xh >= 0.0f && yl <= 0.0f && yh >= 0.0f) return true;
    const float ra = -B * __builtin_amdgcn_rcpf(A), rc = -B * __builtin_amdgcn_rcpf(C);
    auto q = [&](float x, float y) { return A * x * x + 2.0f * B * x * y + C * y * y; };
    auto cl = [](float x, float lo, float hi) { return fminf(fmaxf(x, lo), hi); };
    const float m = fminf(fminf(q(xl, cl(rc * xl, yl, yh)), q(xh, cl(rc * xh, yl, yh))),
                          fminf(q(cl(ra * yl, xl, xh), yl), q(cl(ra * yh, xl, xh), yh)));
    const float xm = fmaxf(xl * xl, xh * xh), ym = fmaxf(yl * yl, yh * yh);
    const float lim = 1.38629436f * __builtin_amdgcn_logf(255.0f * o);  // log2
    return !(m > lim + 0.02f + 1e-5f * (A * xm + C * ym));
}

// One list entry as its lane loads it.
struct Entry {
    uint32_t rec;
    float u, v;
    float4 con;  // A, B, C, opacity
    uint2 fp;
};

__device__ inline Entry load_entry(uint32_t r, const float4* __restrict__ rec0, const float4* __restrict__ rec1,
                                   const uint2* __restrict__ foot)
{
    Entry e;
    e.rec = r;
    const float2 uv = *reinterpret_cast<const float2*>(rec0 + r);
    e.u = uv.x;
    e.v = uv.y;
    e.con = rec1[r];
    e.fp = foot[r];
    return e;
}

// Colour and depth of one record; the depth is the float32 camera-space z the
// depth sort keys hold (positive, so its bits are the key).
__device__ inline float4 rgbz(const float* __restrict__ colors, const uint32_t* __restrict__ depth_key,
                              uint32_t r, uint32_t g)
{
    return make_float4(colors[3 * (size_t)g], colors[3 * (size_t)g + 1], colors[3 * (size_t)g + 2],
                       __uint_as_float(depth_key[r]));
}

// ------------------------------------------------------------- raster fwd

// Entries left of the 64 a wave holds, in list order: (u, v, A, B),
// (C, opacity, list position + 1, -), the pixel mask and the query row; with
// RGBD also (colour r, g, b, camera-space depth z), blended with the same
// weights (Eq. 2: colour; depth by the same alpha blending).
template <int DQ, bool RGBD>
struct FwdStage {
    float4 ab[kList + kGroup];
    float4 cd[kList + kGroup];
    uint2 mask[kList + kGroup];
    float q[(kList + kGroup) * DQ];
    float4 x[RGBD ? kList + kGroup : 1];
};

// Bound by vector issue: per entry and wave some 25 operations (mask, alpha, T),
// and 32 matrix cycles per 16 channels beside them.  Four entries are visited
// without a branch between them: one at a time, with a branch past entries that
// hit nothing, the register copies at each merge and the serial latency of the
// alphas made it 71 us at 640x480 instead of 48.  The K = 1 product adds
// w q to each channel by one fused multiply-add per entry, in list order, so
// Q is what a chain of them per pixel gives.
template <int DQ, bool RGBD>
__device__ inline void raster_fwd_tile(
    FwdStage<DQ, RGBD>& st, const int tile, const CamSet& cs, int N, const uint2* __restrict__ ranges,
    const uint32_t* __restrict__ tile_recs, const float4* __restrict__ rec0,
    const float4* __restrict__ rec1, const uint2* __restrict__ foot,
    const float* __restrict__ queries, float* __restrict__ Q, float* __restrict__ T_final,
    float* __restrict__ T_save, uint32_t* __restrict__ n_contrib, const float* __restrict__ colors,
    const uint32_t* __restrict__ depth_key, float* __restrict__ rgb, float* __restrict__ depth)
{
    constexpr int NC = DQ / 16;  // 16-channel accumulators
    const int c = cam_of_tile(cs, tile);
    const Cam& cam = cs.c[c];
    const Block b = wave_block(cs, cam, tile);
    const int lane = (int)__lane_id(), l16 = lane & 15, lg = lane >> 4, half = lane >> 5;
    const int px = b.x0 + (lane & (b.w - 1)), py = b.y0 + (lane >> b.sx);
    const bool inside = px < cam.w && py < cam.h;
    const uint2 rg = ranges[tile];
    const uint32_t rbase = (uint32_t)c * (uint32_t)N;

    f32x16 acc[NC];
#pragma unroll
    for (int k = 0; k < NC; ++k) acc[k] = f32x16{};
    float4 accx = make_float4(0.f, 0.f, 0.f, 0.f);
    float T = 1.0f;
    uint32_t last = 0;
    // this lane's bit of its half of the pixel mask; zero once the pixel is done
    uint32_t bit = inside ? 1u << (lane & 31) : 0u;
    float fpx = (float)px, fpy = (float)py;
    asm volatile("" : "+v"(fpx), "+v"(fpy));  // held as floats, not converted again at each entry
    const unsigned long long below = (1ull << lane) - 1ull;

    // list entries and record ids are requested a step and two steps ahead
    Entry en{};
    if (rg.x + lane < rg.y) en = load_entry(tile_recs[rg.x + lane], rec0, rec1, foot);
    uint32_t rnext = rg.x + kList + lane < rg.y ? tile_recs[rg.x + kList + lane] : 0u;
    for (uint32_t base = rg.x; base < rg.y; base += kList) {
        if (__ballot(bit != 0u) == 0ull) break;
        const Entry e = en;
        const uint32_t r = e.rec;
        unsigned long long mask = 0ull;
        if (base + lane < rg.y) {
            mask = block_mask(b, e.fp);
            if (mask && !block_reached(b, e.u, e.v, e.con.x, e.con.y, e.con.z, e.con.w)) mask = 0ull;
        }
        if (base + kList + lane < rg.y) {
            en = load_entry(rnext, rec0, rec1, foot);
            if (base + 2 * kList + lane < rg.y) rnext = tile_recs[base + 2 * kList + lane];
        }
        const unsigned long long kept = __ballot(mask != 0ull);
        const int nk = __popcll(kept);
        if (nk == 0) continue;
        float z = 0.0f;  // NaN if a value of the entry is not finite
        if (mask) {
            const int pos = __popcll(kept & below);
            st.ab[pos] = make_float4(e.u, e.v, e.con.x, e.con.y);
            st.cd[pos] = make_float4(e.con.z, e.con.w, __uint_as_float(base - rg.x + lane + 1u), 0.0f);
            st.mask[pos] = make_uint2((uint32_t)mask, (uint32_t)(mask >> 32));
            const float4* qs = reinterpret_cast<const float4*>(queries + (size_t)(r - rbase) * DQ);
            float4* qd = reinterpret_cast<float4*>(st.q + pos * DQ);
#pragma unroll
            for (int k = 0; k < DQ / 4; ++k) {
                const float4 v = qs[k];
                qd[k] = v;
                z += 0.0f * v.x + 0.0f * v.y + 0.0f * v.z + 0.0f * v.w;
            }
            if constexpr (RGBD) {
                const float4 x = rgbz(colors, depth_key, r, r - rbase);
                st.x[pos] = x;
                z += 0.0f * x.x + 0.0f * x.y + 0.0f * x.z;
            }
        }
        if (lane < kGroup - 1) {  // fills the last group with entries of no pixel
            st.mask[nk + lane] = make_uint2(0u, 0u);
#pragma unroll
            for (int k = 0; k < DQ / 4; ++k)
                reinterpret_cast<float4*>(st.q + (nk + lane) * DQ)[k] = make_float4(0.f, 0.f, 0.f, 0.f);
            if constexpr (RGBD) st.x[nk + lane] = make_float4(0.f, 0.f, 0.f, 0.f);
        }
        const bool finite = __ballot(z != z) == 0ull;
        wave_sync();

        // one entry's step: its weight per pixel (zero where it does not count)
        auto step = [&](float oG, uint32_t m, float pos1) {
            const float al = oG < kAlphaMax ? oG : kAlphaMax;
            const bool in = (m & bit) != 0u && !(al < kAlphaMin);
            const float Tn = T * (1.0f - al);
            const bool stop = in && Tn < kTStop, hit = in && !stop;
            bit = stop ? 0u : bit;
            const float wgt = hit ? al * T : 0.0f;
            T = hit ? Tn : T;
            last = hit ? __float_as_uint(pos1) : last;
            return wgt;
        };
        if (finite) {
            // kGroup entries at a time and no branch in between: their alphas do
            // not wait for each other, the transmittance then takes them in order
            for (int j0 = 0; j0 < nk; j0 += kGroup) {
                float og[kGroup], pos1[kGroup], qv[kGroup][NC];
                uint32_t mk[kGroup];
#pragma unroll
                for (int i = 0; i < kGroup; ++i) {
                    const float4 a = st.ab[j0 + i];
                    const float4 d = st.cd[j0 + i];
                    mk[i] = reinterpret_cast<const uint32_t*>(st.mask)[2 * (j0 + i) + half];
                    pos1[i] = d.z;
#pragma unroll
                    for (int k = 0; k < NC; ++k) qv[i][k] = st.q[(j0 + i) * DQ + 16 * k + l16];
                    og[i] = pair_og(a.x, a.y, a.z, a.w, d.x, d.y, fpx, fpy);
                }
#pragma unroll
                for (int i = 0; i < kGroup; ++i) {
                    const float wgt = step(og[i], mk[i], pos1[i]);
#pragma unroll
                    for (int k = 0; k < NC; ++k)
                        acc[k] = __builtin_amdgcn_mfma_f32_16x16x1f32(wgt, qv[i][k], acc[k], 0, 0, 0);
                    if constexpr (RGBD) {
                        const float4 x = st.x[j0 + i];
                        accx.x += wgt * x.x;
                        accx.y += wgt * x.y;
                        accx.z += wgt * x.z;
                        accx.w += wgt * x.w;
                    }
                }
                if (__ballot(bit != 0u) == 0ull) break;
            }
        } else {
            // a value that is not finite reaches only the pixels it is blended
            // into (in the product, 0 x inf would reach the whole block)
#pragma unroll 1
            for (int j = 0; j < nk; ++j) {
                const float4 a = st.ab[j], d = st.cd[j];
                const uint32_t m = reinterpret_cast<const uint32_t*>(st.mask)[2 * j + half];
                const float wgt = step(pair_og(a.x, a.y, a.z, a.w, d.x, d.y, fpx, fpy), m, d.z);
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const float wp = __shfl(wgt, 16 * (i >> 2) + 4 * lg + (i & 3), kWave);
#pragma unroll
                    for (int k = 0; k < NC; ++k)
                        acc[k][i] = wp != 0.0f ? fmaf(wp, st.q[j * DQ + 16 * k + l16], acc[k][i]) : acc[k][i];
                }
                if constexpr (RGBD) {
                    const float4 x = st.x[j];
                    if (wgt != 0.0f) {
                        accx.x += wgt * x.x;
                        accx.y += wgt * x.y;
                        accx.z += wgt * x.z;
                        accx.w += wgt * x.w;
                    }
                }
            }
        }
        wave_sync();
    }
    // accumulator register 4 j + i holds pixel 16 j + 4 (lane / 16) + i, channel lane % 16
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int p = 16 * (i >> 2) + 4 * lg + (i & 3);
        const int qx = b.x0 + (p & (b.w - 1)), qy = b.y0 + (p >> b.sx);
        if (qx < cam.w && qy < cam.h) {
            float* qo = Q + ((size_t)cam.pix_base + (size_t)qy * cam.w + qx) * DQ + l16;
#pragma unroll
            for (int k = 0; k < NC; ++k) qo[16 * k] = acc[k][i];
        }
    }
    if (inside) {
        const size_t p = (size_t)cam.pix_base + (size_t)py * cam.w + px;
        T_final[p] = T;
        T_save[p] = T;
        n_contrib[p] = last;
        if constexpr (RGBD) {
            rgb[3 * p] = accx.x;
            rgb[3 * p + 1] = accx.y;
            rgb[3 * p + 2] = accx.z;
            depth[p] = accx.w;
        }
    }
}

// PERSIST = false: one workgroup per tile.  PERSIST = true: a grid of resident
// workgroups takes tiles from the queue counter until all are done, which
// evens out views of uneven size and tiles of uneven list length.
template <int DQ, bool PERSIST, bool RGBD>
__global__ __launch_bounds__(256) void k_raster_fwd(
    CamSet cs, int N, const uint2* __restrict__ ranges, const uint32_t* __restrict__ tile_recs,
    const float4* __restrict__ rec0, const float4* __restrict__ rec1,
    const uint2* __restrict__ foot, const float* __restrict__ queries, float* __restrict__ Q,
    float* __restrict__ T_final, float* __restrict__ T_save, uint32_t* __restrict__ n_contrib,
    uint32_t* __restrict__ queue, const float* __restrict__ colors,
    const uint32_t* __restrict__ depth_key, float* __restrict__ rgb, float* __restrict__ depth)
{
    extern __shared__ __align__(16) char smem[];  // one stage per wave
    FwdStage<DQ, RGBD>& st = reinterpret_cast<FwdStage<DQ, RGBD>*>(smem)[threadIdx.x / kWave];
    if (!PERSIST) {
        raster_fwd_tile<DQ, RGBD>(st, blockIdx.x, cs, N, ranges, tile_recs, rec0, rec1, foot, queries, Q,
                                  T_final, T_save, n_contrib, colors, depth_key, rgb, depth);
        return;
    }
    __shared__ int s_tile;
    for (;;) {
        __syncthreads();  // every wave has read the last tile index
        if (threadIdx.x == 0) s_tile = (int)atomicAdd(queue, 1u);
        __syncthreads();
        const int tile = __builtin_amdgcn_readfirstlane(s_tile);
        if (tile >= cs.total_tiles) break;
        raster_fwd_tile<DQ, RGBD>(st, tile, cs, N, ranges, tile_recs, rec0, rec1, foot, queries, Q, T_final,
                                  T_save, n_contrib, colors, depth_key, rgb, depth);
    }
}

// ------------------------------------------------------------- raster bwd

constexpr int kBatch = 16;  // entries whose sums one set of matrix products forms

// A wave's queue of entries to visit (what a list step leaves plus fewer than
// kBatch from before) and its exchange buffers: weights w and dL/d(power) dp
// of a batch as [pixel][16 entries], and the batch's screen-space gradients.
// slot(p, e): four entries of a pixel are one 16-byte chunk, and a pixel's four
// chunks are permuted by its position so that the chunk writes (lane = pixel)
// and the word reads (lane = entry) both cover all banks.
struct BwdStage {
    float4 ab[kBatch + kList];    // u, v, A, B
    float4 cd[kBatch + kList];    // C, opacity, list position, record
    uint2 mask[kBatch + kList];   // the block's pixels inside the footprint
    float w[kWave * kBatch];
    float dp[kWave * kBatch];
    float grad[kBatch * 8];
    static __device__ int chunk(int p, int q) { return p * kBatch + 4 * ((q ^ (p >> 1)) & 3); }
    static __device__ int slot(int p, int e) { return chunk(p, e >> 2) + (e & 3); }
};

// f over the 16 lanes of a group, in every lane.
template <class F>
__device__ inline float over16(float x, F f)
{
    x = f(x, dpp_f<0xB1, 0xF, 0xF, false>(x));   // lane ^ 1
    x = f(x, dpp_f<0x4E, 0xF, 0xF, false>(x));   // lane ^ 2
    x = f(x, dpp_f<0x141, 0xF, 0xF, false>(x));  // the mirror lane of the half row
    return f(x, dpp_f<0x140, 0xF, 0xF, false>(x));  // the mirror lane of the row
}

// Whether c holds in a lane of this lane's 16-lane group.
__device__ inline bool any16(bool c)
{
    const unsigned long long m = __ballot(c);
    const uint32_t h = __lane_id() & 32 ? (uint32_t)(m >> 32) : (uint32_t)m;
    return ((h >> (__lane_id() & 16)) & 0xFFFFu) != 0u;
}

// Whether x - ref is larger than x, so that it would round to fewer of x's digits.
__device__ inline bool too_far(float x, float ref) { return fabsf(x - ref) > fabsf(x); }

// A reference for the 16 values x of a lane group that is too far from none of
// them: their mean, or where that is too far the one nearest to zero, or zero
// where they are of both signs.  Values that are not finite are left out.
__device__ inline float reference16(float x)
{
    const bool ok = fabsf(x) <= 3.4e38f;
    // magnitudes compare as their bits
    const float least = over16(fabsf(x), [](float a, float b) {
        return __uint_as_float(min(__float_as_uint(a), __float_as_uint(b)));
    });
    const float mean = over16(ok ? x * (1.0f / 16.0f) : 0.0f, [](float a, float b) { return a + b; });
    const bool neg = any16(x < 0.0f), pos = any16(x > 0.0f);
    const float near = neg ? -least : least;
    return (neg & pos) || least > 3.4e38f ? 0.0f : too_far(near, mean) ? near : mean;
}

// Four 16-lane groups by four registers, transposed: register j of lane group
// g becomes register g of lane group j.
__device__ inline void transpose_groups(float& a, float& b, float& c, float& d)
{
    auto swap32 = [](float& x, float& y) {
        const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false);
        x = __uint_as_float(r[0]);
        y = __uint_as_float(r[1]);
    };
    auto swap16 = [](float& x, float& y) {
        const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(y), false, false);
        x = __uint_as_float(r[0]);
        y = __uint_as_float(r[1]);
    };
    swap32(a, c);
    swap32(b, d);
    swap16(a, b);
    swap16(c, d);
}

// Sum over the four 16-lane groups, in every lane.
__device__ inline float sum_groups(float x)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    const auto t = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(t[0]) + __uint_as_float(t[1]);
}

// Everything that the backward adds into starts at zero, in one launch: the
// gradient sums of the visible records (those of the others are not read), the
// query gradients and, with RGBD, the depth sums and the colour gradients.
// Bound by memory: four threads clear one record's 64-byte line.  One launch for
// two fills (four with RGBD): with the record lines below, 1026 to 983 us for
// the whole colour and depth pass at 1200x680.
__global__ __launch_bounds__(256) void k_clear_grads(const uint32_t* __restrict__ ntiles, size_t records,
                                                     double* __restrict__ rec_grad,
                                                     float* __restrict__ rec_dz,
                                                     float* __restrict__ d_queries, size_t nq,
                                                     float* __restrict__ d_colors, size_t nc)
{
    const size_t i0 = blockIdx.x * (size_t)blockDim.x + threadIdx.x, step = (size_t)gridDim.x * blockDim.x;
    for (size_t i = i0; i < records * 4; i += step) {
        const size_t r = i >> 2;
        if (ntiles[r] == 0) continue;
        reinterpret_cast<double2*>(rec_grad)[i] = make_double2(0.0, 0.0);
        if (rec_dz && (i & 3) == 0) rec_dz[r] = 0.0f;
    }
    for (size_t i = i0; i < nq; i += step) d_queries[i] = 0.0f;
    if (d_colors)
        for (size_t i = i0; i < nc; i += step) d_colors[i] = 0.0f;
}

// rec_grad[r] = (du, dv, dA, dB, dC, dopacity) accumulated over pixels, the sums
// over the waves in float64: the gradients of a large Gaussian's rotation and
// scales cancel among the three conic terms, and the rounding of float32 atomics
// in their order of arrival showed in them (a component that cancels moved by up
// to 7e-4 of itself from run to run).  The order is as arbitrary in float64, but
// seldom survives the rounding to float32: seven runs of four scenes gave the
// same bits.  The sums of queries, colours and depths (and with the depths'
// the means' gradient) are float32 and move by up to 3e-6 of the largest.  A
// record's sums have a 64-byte line of their own, so that its atomics never
// touch two: the backward of eight views takes 927 us with records of 24 bytes
// in float32, 1091 us with 48 in float64 and 869 us with 64.
// With RGBD also d_colors[g] and rec_dz[r] (the gradient of the record's depth).
//
// A pixel walks its list back to front, rebuilding the transmittance by
// division.  With s_j = q_j . dQ the gradient of alpha_j is T_j (s_j - b_j),
// where b_j, the blend of the s behind entry j, follows b <- b + alpha (s - b):
// one scalar per pixel in place of a blended query.  Batches of 16 entries:
//   s      [16 entries x 64 pixels] = q dQ^T by MFMA (K = channels), then a
//          transposition of lane groups puts one pixel on each lane;
//   walk   per entry and pixel: alpha, T, w = alpha T, dp = dL/d(power);
//   sums   through LDS (lane = pixel to lane = entry, a quarter of the pixels):
//          d_queries [16 x DQ] = w^T dQ by MFMA (K = pixels), and the sums of
//          dp (1, dx, dy, dx^2, dx dy, dy^2) that the six screen-space
//          gradients need by vector operations (as moments about the block's
//          centre they would also be a product, but small Gaussians away from
//          the centre then lose digits to cancellation).
// Per entry and wave about 45 vector operations and 4 DQ MFMA cycles.  Its
// time at 640x480 is 109 us.  With float32 sums at 24 bytes a record it was 118 us, of which 22
// us were the prologue and the list steps, 26 us the atomics (32 cache lines of
// them per batch) and the rest the walk at two to three waves per SIMD.
template <int DQ, bool RGBD>
__device__ inline void raster_bwd_tile(
    BwdStage& st, const int tile, const CamSet& cs, int N,
    const uint2* __restrict__ ranges, const uint32_t* __restrict__ tile_recs,
    const float4* __restrict__ rec0, const float4* __restrict__ rec1,
    const uint2* __restrict__ foot, const float* __restrict__ queries,
    const float* __restrict__ T_final, const uint32_t* __restrict__ n_contrib,
    const float* __restrict__ dQ, double* __restrict__ rec_grad, float* __restrict__ d_queries,
    const float* __restrict__ colors, const uint32_t* __restrict__ depth_key,
    const float* __restrict__ d_rgb, const float* __restrict__ d_depth, float* __restrict__ d_colors,
    float* __restrict__ rec_dz)
{
    constexpr int NC = DQ / 16;  // 16-channel column blocks
    constexpr int KD = DQ / 4;   // channels per lane group in the dot products
    constexpr int KX = KD + (RGBD ? 1 : 0);
    const int c = cam_of_tile(cs, tile);
    const Cam& cam = cs.c[c];
    const Block b = wave_block(cs, cam, tile);
    const int lane = (int)__lane_id(), l16 = lane & 15, lg = lane >> 4, half = lane >> 5;
    const int px = b.x0 + (lane & (b.w - 1)), py = b.y0 + (lane >> b.sx);
    const bool inside = px < cam.w && py < cam.h;
    const uint2 rg = ranges[tile];
    const uint32_t rbase = (uint32_t)c * (uint32_t)N;
    // pixel of the block -> row of the pixel arrays, or -1 outside the image
    auto row_of = [&](int p) -> long long {
        const int x = b.x0 + (p & (b.w - 1)), y = b.y0 + (p >> b.sx);
        return x < cam.w && y < cam.h ? cam.pix_base + (long long)y * cam.w + x : -1ll;
    };
    const long long prow = row_of(lane);
    float T = inside ? T_final[prow] : 1.0f;
    const uint32_t last = inside ? n_contrib[prow] : 0u;
    // dQ as the B operand of the dot products (K = channels: lane group lg
    // holds channels KD lg .. + KD - 1 of pixel 16 j + l16) and of the sums
    // over the pixels (step s: lane group lg holds pixel 4 s + lg, lane l16 a channel)
    float gd[4][KD], gs[NC][16], gdx[RGBD ? 4 : 1], gsx[RGBD ? 16 : 1];
    float z = 0.0f;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const long long p = row_of(16 * j + l16);
#pragma unroll
        for (int k = 0; k < KD; k += 4) {
            float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
            if (p >= 0) v = *reinterpret_cast<const float4*>(dQ + p * DQ + KD * lg + k);
            gd[j][k] = v.x; gd[j][k + 1] = v.y; gd[j][k + 2] = v.z; gd[j][k + 3] = v.w;
            z += 0.0f * v.x + 0.0f * v.y + 0.0f * v.z + 0.0f * v.w;
        }
        if constexpr (RGBD) {
            gdx[j] = p < 0 ? 0.0f : lg < 3 ? d_rgb[3 * p + lg] : d_depth[p];
            z += 0.0f * gdx[j];
        }
    }
#pragma unroll
    for (int s = 0; s < 16; ++s) {
        const int q = 4 * s + lg;
        const long long p = row_of(q);
#pragma unroll
        for (int k = 0; k < NC; ++k) gs[k][s] = p >= 0 ? dQ[p * DQ + 16 * k + l16] : 0.0f;
        if constexpr (RGBD) gsx[s] = p < 0 || l16 > 3 ? 0.0f : l16 < 3 ? d_rgb[3 * p + l16] : d_depth[p];
    }
    int maxlast = (int)last;
    for (int o = 32; o >= 1; o >>= 1) maxlast = max(maxlast, __shfl_xor(maxlast, o, kWave));

    if (maxlast == 0) return;
    // A pixel whose upstream gradient is not finite reaches only the entries
    // blended into it: its column of the pixel sums is cleared (0 x inf would
    // reach every entry of the batch) and its terms are added one by one.
    unsigned long long bad = 0ull;
    if (__ballot(z != 0.0f) != 0ull) {
        float y = 0.0f;
        if (inside) {
            #pragma unroll 1
            for (int k = 0; k < DQ; ++k) y += 0.0f * dQ[prow * DQ + k];
            if constexpr (RGBD) y += 0.0f * d_rgb[3 * prow] + 0.0f * d_rgb[3 * prow + 1] + 0.0f * d_rgb[3 * prow + 2] + 0.0f * d_depth[prow];
        }
        bad = __ballot(y != 0.0f);
#pragma unroll
        for (int s = 0; s < 16; ++s) {
            if (!((bad >> (4 * s + lg)) & 1ull)) continue;
#pragma unroll
            for (int k = 0; k < NC; ++k) gs[k][s] = 0.0f;
            if constexpr (RGBD) gsx[s] = 0.0f;
        }
    }
    const bool mine_bad = ((bad >> lane) & 1ull) != 0ull;
    const uint32_t bit = 1u << (lane & 31);
    float fpx = (float)px, fpy = (float)py;
    asm volatile("" : "+v"(fpx), "+v"(fpy));
    const unsigned long long below = (1ull << lane) - 1ull;
    float behind = 0.0f;

    // s[e] = value of entry e (rows; lane group lg holds its channels KD lg ..)
    // times dQ of this lane's pixel
    auto dots = [&](const float* q, float* sv) {
        f32x4 s4[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            s4[j] = f32x4{};
#pragma unroll
            for (int k = 0; k < KD; ++k) s4[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(q[k], gd[j][k], s4[j], 0, 0, 0);
            if constexpr (RGBD) s4[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(q[KD], gdx[j], s4[j], 0, 0, 0);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float t0 = s4[0][i], t1 = s4[1][i], t2 = s4[2][i], t3 = s4[3][i];
            transpose_groups(t0, t1, t2, t3);
            sv[i] = t0; sv[4 + i] = t1; sv[8 + i] = t2; sv[12 + i] = t3;
        }
    };
    // The dot products are taken with q - qref, qref the mean query of the
    // wave's first batch: where the queries share an offset, s - b would lose
    // the digits of it.  With rref = qref . dQ and past = the product of
    // (1 - alpha) of the entries behind, s - b = (s' - b') + rref past.
    // The entries of a batch need not share a pixel, and q - qref rounds to the
    // digits of the larger: so that no query costs another one digits, no
    // channel of qref is too far from any query visited: reference16 takes it
    // so for the first batch, and a later query that it does not suit sets that
    // channel of it to zero (it is then less than half of it or of the other
    // sign, and there is not much of an offset to keep).
    bool first_ref = true;
    float qref[KX], rref = 0.0f, past = 1.0f;
#pragma unroll
    for (int k = 0; k < KX; ++k) qref[k] = 0.0f;

    // The sums of a batch are added to memory once the next batch's queries are
    // requested: memory operations complete in order, so a load issued after
    // the atomics would wait for them.
    bool pending = false;
    f32x4 pq[NC], pxz = {};
    uint32_t pr[4], pgr[2];
    float pg[2];
    auto flush = [&]() {
        if (!pending) return;
        // result register i of lane group lg is entry 4 lg + i, column l16
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const size_t g = (size_t)(pr[i] - rbase);
#pragma unroll
            for (int k = 0; k < NC; ++k)
                if (pq[k][i] != 0.0f) unsafeAtomicAdd(d_queries + g * DQ + 16 * k + l16, pq[k][i]);
            if constexpr (RGBD) {
                if (l16 < 4 && pxz[i] != 0.0f) unsafeAtomicAdd(l16 < 3 ? d_colors + g * 3 + l16 : rec_dz + pr[i], pxz[i]);
            }
        }
#pragma unroll
        for (int i = 0; i < 2; ++i)
            if ((lane & 7) < 6 && pg[i] != 0.0f) unsafeAtomicAdd(rec_grad + (size_t)pgr[i] * kRecGrad + (lane & 7), (double)pg[i]);
    };

    auto batch = [&](int q0) {  // queue entries q0 .. q0 + 15
        // the queries of entry l16, channels KD lg ..; in flight during the alphas
        const uint32_t er = __float_as_uint(st.cd[q0 + l16].w);
        const float* qrow = queries + (size_t)(er - rbase) * DQ + KD * lg;
        float qv[KX];
#pragma unroll
        for (int k = 0; k < KD; k += 4) {
            const float4 v = *reinterpret_cast<const float4*>(qrow + k);
            qv[k] = v.x; qv[k + 1] = v.y; qv[k + 2] = v.z; qv[k + 3] = v.w;
        }
        if constexpr (RGBD) qv[KD] = lg < 3 ? colors[3 * (size_t)(er - rbase) + lg] : __uint_as_float(depth_key[er]);
        __builtin_amdgcn_sched_barrier(0);
        flush();
        __builtin_amdgcn_sched_barrier(0);
        float og[kBatch];  // o G where the pair counts, else 0
#pragma unroll
        for (int e = 0; e < kBatch; ++e) {
            const float4 a = st.ab[q0 + e], d = st.cd[q0 + e];
            const uint32_t m = reinterpret_cast<const uint32_t*>(st.mask)[2 * (q0 + e) + half];
            const float oG = pair_og(a.x, a.y, a.z, a.w, d.x, d.y, fpx, fpy);
            const float al = oG < kAlphaMax ? oG : kAlphaMax;
            const bool hit = ((m & bit) != 0u) & (__float_as_uint(d.z) < last) & (al >= kAlphaMin);
            og[e] = hit ? oG : 0.0f;
            // formed here, four entries' LDS reads in flight (sunk to its use it
            // would keep the operands of all sixteen in registers)
            asm volatile("" : "+v"(og[e]));
            if (e % 4 == 3) __builtin_amdgcn_sched_barrier(0);
        }
        bool far = first_ref;
#pragma unroll
        for (int k = 0; k < KX; ++k) far |= too_far(qv[k], qref[k]);
        if (__ballot(far) != 0ull) {
            float sv[kBatch];
#pragma unroll
            for (int k = 0; k < KX; ++k)
                qref[k] = first_ref ? reference16(qv[k]) : any16(too_far(qv[k], qref[k])) ? 0.0f : qref[k];
            first_ref = false;
            dots(qref, sv);
            // b' relative to the new reference (past = 1: nothing behind yet)
            behind += past < 1.0f ? (rref - sv[0]) * (1.0f - past) : 0.0f;
            rref = sv[0];
        }
#pragma unroll
        for (int k = 0; k < KX; ++k) qv[k] -= qref[k];
        float sv[kBatch];  // s of entry e for this lane's pixel
        dots(qv, sv);
#pragma unroll
        for (int e4 = 0; e4 < 4; ++e4) {
            float w4[4], p4[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int e = 4 * e4 + i;
                const bool hit = og[e] != 0.0f;
                const float al = og[e] < kAlphaMax ? og[e] : kAlphaMax;
                // 1 - al >= 0.01: the hardware reciprocal (1 ulp) replaces the
                // IEEE division sequence; 1 where the pair does not count
                const float om = 1.0f - al;
                T = T * __builtin_amdgcn_rcpf(om);
                w4[i] = al * T;
                const float d0 = sv[e] - behind, t = hit ? d0 : 0.0f;
                behind += al * t;
                const float f = fmaf(rref, past, t) * T * og[e];
                p4[i] = (hit & (og[e] < kAlphaMax)) ? f : 0.0f;
                past *= om;
            }
            *reinterpret_cast<float4*>(st.w + BwdStage::chunk(lane, e4)) = make_float4(w4[0], w4[1], w4[2], w4[3]);
            *reinterpret_cast<float4*>(st.dp + BwdStage::chunk(lane, e4)) = make_float4(p4[0], p4[1], p4[2], p4[3]);
        }
        wave_sync();
        if (mine_bad) {
#pragma unroll 1
            for (int e = 0; e < kBatch; ++e) {
                const float w = st.w[BwdStage::slot(lane, e)];
                if (w == 0.0f) continue;
                const uint32_t r = __float_as_uint(st.cd[q0 + e].w);
                const size_t g = (size_t)(r - rbase);
#pragma unroll 1
                for (int k = 0; k < DQ; ++k) unsafeAtomicAdd(d_queries + g * DQ + k, w * dQ[prow * DQ + k]);
                if constexpr (RGBD) {
                    for (int k = 0; k < 3; ++k) unsafeAtomicAdd(d_colors + g * 3 + k, w * d_rgb[3 * prow + k]);
                    unsafeAtomicAdd(rec_dz + r, w * d_depth[prow]);
                }
            }
        }
        // from here a lane is entry l16 and the pixels 4 s + lg
        f32x4 dq4[NC], dx4 = {};
#pragma unroll
        for (int k = 0; k < NC; ++k) dq4[k] = f32x4{};
        float da[16];
        // slot(4 s + lg, l16): two bases, 128 words further for every other s
        const float *we = st.w + BwdStage::slot(lg, l16), *wo = st.w + BwdStage::slot(4 + lg, l16);
#pragma unroll
        for (int s = 0; s < 16; ++s) {
            const float* at = (s & 1 ? wo : we) + 128 * (s >> 1);
            const float wa = at[0];
            da[s] = at[kWave * kBatch];  // st.dp
#pragma unroll
            for (int k = 0; k < NC; ++k) dq4[k] = __builtin_amdgcn_mfma_f32_16x16x4f32(wa, gs[k][s], dq4[k], 0, 0, 0);
            if constexpr (RGBD) dx4 = __builtin_amdgcn_mfma_f32_16x16x4f32(wa, gsx[s], dx4, 0, 0, 0);
        }
        // sums of dp (1, dx, dy, dx^2, dx dy, dy^2) over the lane's pixels,
        // each product formed from the pair's own offsets
        const float4 ea = st.ab[q0 + l16], ed = st.cd[q0 + l16];
        float m0 = 0.f, sx = 0.f, sy = 0.f, sxx = 0.f, sxy = 0.f, syy = 0.f;
        if (b.sx == 3) {
            // 8 x 8: pixels 8 y + lg and 8 y + 4 + lg of row y, summed by rows first
            const float xa = ea.x - (float)(b.x0 + lg), xb = ea.x - (float)(b.x0 + 4 + lg);
            const float xa2 = xa * xa, xb2 = xb * xb;
#pragma unroll
            for (int y = 0; y < 8; ++y) {
                const float dy = ea.y - (float)(b.y0 + y);
                const float r0 = da[2 * y] + da[2 * y + 1];
                const float r1 = da[2 * y] * xa + da[2 * y + 1] * xb;
                m0 += r0;
                sx += r1;
                sxx += da[2 * y] * xa2 + da[2 * y + 1] * xb2;
                const float t = r0 * dy;
                sy += t;
                syy += t * dy;
                sxy += r1 * dy;
            }
        } else {
            int lq = lg;
            asm volatile("" : "+v"(lq));  // the 16 pixel positions are formed here, not kept across the batches
#pragma unroll
            for (int s = 0; s < 16; ++s) {
                const int q = 4 * s + lq;
                const float dx = ea.x - (float)(b.x0 + (q & (b.w - 1))), dy = ea.y - (float)(b.y0 + (q >> b.sx));
                const float tx = da[s] * dx, ty = da[s] * dy;
                m0 += da[s];
                sx += tx;
                sy += ty;
                sxx += tx * dx;
                sxy += tx * dy;
                syy += ty * dy;
            }
        }
        m0 = sum_groups(m0); sx = sum_groups(sx); sy = sum_groups(sy);
        sxx = sum_groups(sxx); sxy = sum_groups(sxy); syy = sum_groups(syy);
        if (lane < kBatch) {
            *reinterpret_cast<float4*>(st.grad + 8 * lane) =
                make_float4(-(ea.z * sx + ea.w * sy), -(ed.x * sy + ea.w * sx), -0.5f * sxx, -sxy);
            *reinterpret_cast<float2*>(st.grad + 8 * lane + 4) =
                make_float2(-0.5f * syy, m0 != 0.0f ? m0 / ed.y : 0.0f);
        }
        wave_sync();
#pragma unroll
        for (int k = 0; k < NC; ++k) pq[k] = dq4[k];
        if constexpr (RGBD) pxz = dx4;
#pragma unroll
        for (int i = 0; i < 4; ++i) pr[i] = __float_as_uint(st.cd[q0 + 4 * lg + i].w);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int e = 8 * i + (lane >> 3);
            pg[i] = st.grad[8 * e + (lane & 7)];
            pgr[i] = __float_as_uint(st.cd[q0 + e].w);
        }
        pending = true;
        wave_sync();
    };

    int nq = 0;  // entries in the queue
    // list entries and record ids are requested a step and two steps ahead
    const int jl = maxlast - 1 - lane;  // back to front
    Entry en{};
    if (jl >= 0) en = load_entry(tile_recs[rg.x + jl], rec0, rec1, foot);
    uint32_t rnext = jl - kList >= 0 ? tile_recs[rg.x + jl - kList] : 0u;
    for (int end = maxlast; end > 0; end -= kList) {
        const int j = end - 1 - lane;
        const Entry e = en;
        const uint32_t r = e.rec;
        unsigned long long mask = 0ull;
        if (j >= 0) {
            mask = block_mask(b, e.fp);
            if (mask && !block_reached(b, e.u, e.v, e.con.x, e.con.y, e.con.z, e.con.w)) mask = 0ull;
        }
        if (j - kList >= 0) {
            en = load_entry(rnext, rec0, rec1, foot);
            if (j - 2 * kList >= 0) rnext = tile_recs[rg.x + j - 2 * kList];
        }
        const unsigned long long kept = __ballot(mask != 0ull);
        if (mask) {
            const int pos = nq + __popcll(kept & below);
            st.ab[pos] = make_float4(e.u, e.v, e.con.x, e.con.y);
            st.cd[pos] = make_float4(e.con.z, e.con.w, __uint_as_float((uint32_t)j), __uint_as_float(r));
            st.mask[pos] = make_uint2((uint32_t)mask, (uint32_t)(mask >> 32));
        }
        nq += __popcll(kept);
        if (end <= kList && (nq & (kBatch - 1)) != 0) {
            // the last list step: fill the last batch with entries of no pixel
            // (the last entry's record, so that no other query is read)
            const int pad = kBatch - (nq & (kBatch - 1));
            wave_sync();
            if (lane < pad) {
                st.ab[nq + lane] = make_float4(0.f, 0.f, 0.f, 0.f);
                st.cd[nq + lane] = make_float4(0.f, 1.f, 0.f, st.cd[nq - 1].w);
                st.mask[nq + lane] = make_uint2(0u, 0u);
            }
            nq += pad;
        }
        wave_sync();
        int q0 = 0;
        for (; q0 + kBatch <= nq; q0 += kBatch) batch(q0);
        // what is left moves to the front (fewer than kBatch entries)
        nq -= q0;
        if (q0 > 0 && nq > 0) {
            float4 ta, td;
            uint2 tm;
            if (lane < nq) {
                ta = st.ab[q0 + lane];
                td = st.cd[q0 + lane];
                tm = st.mask[q0 + lane];
            }
            wave_sync();
            if (lane < nq) {
                st.ab[lane] = ta;
                st.cd[lane] = td;
                st.mask[lane] = tm;
            }
            wave_sync();
        }
    }
    flush();
}

template <int DQ, bool PERSIST, bool RGBD>
__global__ __launch_bounds__(256, DQ == 16 && !RGBD ? 3 : 2) void k_raster_bwd(
    CamSet cs, int N, const uint2* __restrict__ ranges, const uint32_t* __restrict__ tile_recs,
    const float4* __restrict__ rec0, const float4* __restrict__ rec1,
    const uint2* __restrict__ foot, const float* __restrict__ queries,
    const float* __restrict__ T_final, const uint32_t* __restrict__ n_contrib,
    const float* __restrict__ dQ, double* __restrict__ rec_grad, float* __restrict__ d_queries,
    uint32_t* __restrict__ queue, const float* __restrict__ colors,
    const uint32_t* __restrict__ depth_key, const float* __restrict__ d_rgb,
    const float* __restrict__ d_depth, float* __restrict__ d_colors, float* __restrict__ rec_dz)
{
    extern __shared__ __align__(16) char smem[];  // one stage per wave
    BwdStage& st = reinterpret_cast<BwdStage*>(smem)[threadIdx.x / kWave];
    if (!PERSIST) {
        raster_bwd_tile<DQ, RGBD>(st, blockIdx.x, cs, N, ranges, tile_recs, rec0, rec1, foot, queries,
                                  T_final, n_contrib, dQ, rec_grad, d_queries, colors, depth_key, d_rgb,
                                  d_depth, d_colors, rec_dz);
        return;
    }
    __shared__ int s_tile;
    for (;;) {
        __syncthreads();
        if (threadIdx.x == 0) s_tile = (int)atomicAdd(queue, 1u);
        __syncthreads();
        const int tile = __builtin_amdgcn_readfirstlane(s_tile);
        if (tile >= cs.total_tiles) break;
        raster_bwd_tile<DQ, RGBD>(st, tile, cs, N, ranges, tile_recs, rec0, rec1, foot, queries,
                                  T_final, n_contrib, dQ, rec_grad, d_queries, colors, depth_key, d_rgb,
                                  d_depth, d_colors, rec_dz);
    }
}

// ------------------------------------------------------ preprocess adjoint

// Chains rec_grad of every camera back to the raw parameters of Gaussian i
// (FP32, matrix form of the chain rule), and rec_dz (nullable: the gradient of
// each record's rendered depth z = row 3 of the view transform applied to the
// mean) to the mean.  Outputs are overwritten.
__global__ __launch_bounds__(256) void k_preprocess_bwd(
    CamSet cs, int N, const float* __restrict__ means, const float* __restrict__ log_scales,
    const float* __restrict__ quats, const float* __restrict__ logits,
    const uint32_t* __restrict__ ntiles, const double* __restrict__ rec_grad,
    const float* __restrict__ rec_dz, float* __restrict__ d_means, float* __restrict__ d_log_scales,
    float* __restrict__ d_quats, float* __restrict__ d_logits)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= N) return;
    const float m0 = means[3 * i], m1 = means[3 * i + 1], m2 = means[3 * i + 2];
    float s[3];
    for (int k = 0; k < 3; ++k) s[k] = __expf(log_scales[3 * i + k]);
    const float q0 = quats[4 * i], q1 = quats[4 * i + 1], q2 = quats[4 * i + 2], q3 = quats[4 * i + 3];
    const float qnorm = sqrtf(q0 * q0 + q1 * q1 + q2 * q2 + q3 * q3);
    const float iq = 1.0f / qnorm;
    const float w = q0 * iq, x = q1 * iq, y = q2 * iq, z = q3 * iq;
    float Rm[3][3] = {{1.f - 2.f * (y * y + z * z), 2.f * (x * y - w * z), 2.f * (x * z + w * y)},
                      {2.f * (x * y + w * z), 1.f - 2.f * (x * x + z * z), 2.f * (y * z - w * x)},
                      {2.f * (x * z - w * y), 2.f * (y * z + w * x), 1.f - 2.f * (x * x + y * y)}};
    float Mm[3][3];  // M = R diag(s)
    for (int a = 0; a < 3; ++a)
        for (int b = 0; b < 3; ++b) Mm[a][b] = Rm[a][b] * s[b];
    float S3[3][3];
    for (int a = 0; a < 3; ++a)
        for (int b = 0; b < 3; ++b)
            S3[a][b] = Mm[a][0] * Mm[b][0] + Mm[a][1] * Mm[b][1] + Mm[a][2] * Mm[b][2];
    const float sig = 1.0f / (1.0f + __expf(-logits[i]));

    float gmean[3] = {0.f, 0.f, 0.f}, gS3[3][3] = {{0.f}}, glogit = 0.f;
    for (int ci = 0; ci < cs.n; ++ci) {
        const size_t r = (size_t)ci * N + i;
        if (ntiles[r] == 0) continue;
        const Cam& cam = cs.c[ci];
        const double2* gr = reinterpret_cast<const double2*>(rec_grad + kRecGrad * r);
        const double2 g0 = gr[0], g1 = gr[1], g2 = gr[2];
        const float du = (float)g0.x, dv = (float)g0.y, dA = (float)g1.x, dB = (float)g1.y;
        const float dC = (float)g2.x, dO = (float)g2.y;
        glogit += dO * sig * (1.0f - sig);
        float W[3][3];
        for (int a = 0; a < 3; ++a)
            for (int b = 0; b < 3; ++b) W[a][b] = cam.vm[4 * a + b];
        const float cx = W[0][0] * m0 + W[0][1] * m1 + W[0][2] * m2 + cam.vm[3];
        const float cy = W[1][0] * m0 + W[1][1] * m1 + W[1][2] * m2 + cam.vm[7];
        const float cz = W[2][0] * m0 + W[2][1] * m1 + W[2][2] * m2 + cam.vm[11];
        const float limx = (float)kFovClamp * (cam.w / (2.0f * cam.fx));
        const float limy = (float)kFovClamp * (cam.h / (2.0f * cam.fy));
        const float rx = cx / cz, ry = cy / cz;
        const bool inx = rx >= -limx && rx <= limx, iny = ry >= -limy && ry <= limy;
        const float tx = inx ? rx : (rx < 0.f ? -limx : limx);
        const float ty = iny ? ry : (ry < 0.f ? -limy : limy);
        const float iz = 1.0f / cz;
        const float J[2][3] = {{cam.fx * iz, 0.f, -cam.fx * tx * iz}, {0.f, cam.fy * iz, -cam.fy * ty * iz}};
        // camera covariance Sc = W S3 W^T
        float WS[3][3], Sc[3][3];
        for (int a = 0; a < 3; ++a)
            for (int b = 0; b < 3; ++b) WS[a][b] = W[a][0] * S3[0][b] + W[a][1] * S3[1][b] + W[a][2] * S3[2][b];
        for (int a = 0; a < 3; ++a)
            for (int b = 0; b < 3; ++b) Sc[a][b] = WS[a][0] * W[b][0] + WS[a][1] * W[b][1] + WS[a][2] * W[b][2];
        // screen covariance and its inverse (the conic)
        float JS[2][3];
        for (int a = 0; a < 2; ++a)
            for (int b = 0; b < 3; ++b) JS[a][b] = J[a][0] * Sc[0][b] + J[a][1] * Sc[1][b] + J[a][2] * Sc[2][b];
        const float sa = JS[0][0] * J[0][0] + JS[0][1] * J[0][1] + JS[0][2] * J[0][2] + (float)kDilation;
        const float sb = JS[0][0] * J[1][0] + JS[0][1] * J[1][1] + JS[0][2] * J[1][2];
        const float sc = JS[1][0] * J[1][0] + JS[1][1] * J[1][1] + JS[1][2] * J[1][2] + (float)kDilation;
        const float idet = 1.0f / (sa * sc - sb * sb);
        const float Ci[2][2] = {{sc * idet, -sb * idet}, {-sb * idet, sa * idet}};
        // gradient w.r.t. the conic matrix (off-diagonal shared), then -Ci G Ci
        const float Gc[2][2] = {{dA, 0.5f * dB}, {0.5f * dB, dC}};
        float T1[2][2], G2[2][2];
        for (int a = 0; a < 2; ++a)
            for (int b = 0; b < 2; ++b) T1[a][b] = Ci[a][0] * Gc[0][b] + Ci[a][1] * Gc[1][b];
        for (int a = 0; a < 2; ++a)
            for (int b = 0; b < 2; ++b) G2[a][b] = -(T1[a][0] * Ci[0][b] + T1[a][1] * Ci[1][b]);
        // Sigma2 = J Sc J^T: G_Sc = J^T G2 J ; G_J = 2 G2 J Sc
        float GJ[2][3];
        for (int a = 0; a < 2; ++a)
            for (int b = 0; b < 3; ++b)
                GJ[a][b] = 2.0f * (G2[a][0] * JS[0][b] + G2[a][1] * JS[1][b]);
        float GSc[3][3];
        for (int a = 0; a < 3; ++a)
            for (int b = 0; b < 3; ++b)
                GSc[a][b] = J[0][a] * (G2[0][0] * J[0][b] + G2[0][1] * J[1][b]) +
                            J[1][a] * (G2[1][0] * J[0][b] + G2[1][1] * J[1][b]);
        // Sc = W S3 W^T: G_S3 += W^T G_Sc W
        float GW[3][3];
        for (int a = 0; a < 3; ++a)
            for (int b = 0; b < 3; ++b) GW[a][b] = GSc[a][0] * W[0][b] + GSc[a][1] * W[1][b] + GSc[a][2] * W[2][b];
        for (int a = 0; a < 3; ++a)
            for (int b = 0; b < 3; ++b) gS3[a][b] += W[0][a] * GW[0][b] + W[1][a] * GW[1][b] + W[2][a] * GW[2][b];
        // camera-space centre through J and through (u, v)
        float gx = du * cam.fx * iz, gy = dv * cam.fy * iz;
        float gz = -(du * cam.fx * cx + dv * cam.fy * cy) * iz * iz;
        gz += -(GJ[0][0] * cam.fx + GJ[1][1] * cam.fy) * iz * iz;
        // J02 = -fx tx / z, tx = x / z when not clamped
        gz += (GJ[0][2] * cam.fx * tx + GJ[1][2] * cam.fy * ty) * iz * iz;
        if (inx) { gx += -GJ[0][2] * cam.fx * iz * iz; gz += GJ[0][2] * cam.fx * cx * iz * iz * iz; }
        if (iny) { gy += -GJ[1][2] * cam.fy * iz * iz; gz += GJ[1][2] * cam.fy * cy * iz * iz * iz; }
        if (rec_dz) gz += rec_dz[r];
        for (int k = 0; k < 3; ++k) gmean[k] += W[0][k] * gx + W[1][k] * gy + W[2][k] * gz;
    }
    // S3 = M M^T: G_M = 2 G_S3 M ; M = R diag(s)
    float GM[3][3];
    for (int a = 0; a < 3; ++a)
        for (int b = 0; b < 3; ++b) GM[a][b] = 2.0f * (gS3[a][0] * Mm[0][b] + gS3[a][1] * Mm[1][b] + gS3[a][2] * Mm[2][b]);
    float GR[3][3];
    for (int a = 0; a < 3; ++a)
        for (int b = 0; b < 3; ++b) GR[a][b] = GM[a][b] * s[b];
    for (int k = 0; k < 3; ++k)
        d_log_scales[3 * i + k] = (GM[0][k] * Rm[0][k] + GM[1][k] * Rm[1][k] + GM[2][k] * Rm[2][k]) * s[k];
    // rotation entries as functions of the unit quaternion, grouped per component
    const float gw = 2.f * (-z * GR[0][1] + y * GR[0][2] + z * GR[1][0] - x * GR[1][2] - y * GR[2][0] + x * GR[2][1]);
    const float gxq = 2.f * (y * GR[0][1] + z * GR[0][2] + y * GR[1][0] - 2.f * x * GR[1][1] - w * GR[1][2] +
                             z * GR[2][0] + w * GR[2][1] - 2.f * x * GR[2][2]);
    const float gyq = 2.f * (-2.f * y * GR[0][0] + x * GR[0][1] + w * GR[0][2] + x * GR[1][0] + z * GR[1][2] -
                             w * GR[2][0] + z * GR[2][1] - 2.f * y * GR[2][2]);
    const float gzq = 2.f * (-2.f * z * GR[0][0] - w * GR[0][1] + x * GR[0][2] + w * GR[1][0] - 2.f * z * GR[1][1] +
                             y * GR[1][2] + x * GR[2][0] + y * GR[2][1]);
    const float dot = gw * w + gxq * x + gyq * y + gzq * z;
    d_quats[4 * i + 0] = (gw - w * dot) * iq;
    d_quats[4 * i + 1] = (gxq - x * dot) * iq;
    d_quats[4 * i + 2] = (gyq - y * dot) * iq;
    d_quats[4 * i + 3] = (gzq - z * dot) * iq;
    for (int k = 0; k < 3; ++k) d_means[3 * i + k] = gmean[k];
    d_logits[i] = glogit;
}

// ------------------------------------------------------------- launchers

hipError_t launch_fill_u32(uint32_t* p, size_t n, uint32_t v, hipStream_t st)
{
    if (n == 0) return hipSuccess;
    size_t blocks = (n + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(k_fill_u32, dim3((unsigned)blocks), dim3(256), 0, st, p, n, v);
    return hipGetLastError();
}

// ------------------------------------------------------------- scheduling

// The context's tile schedule: 0 one workgroup per tile, 1 persistent, 2 the
// library's choice, which is one workgroup per tile: a workgroup's waves walk
// their blocks independently, and meeting at the queue after every tile costs
// more than the even spread saves (eight views of uneven size: forward 291
// against 313 us, backward 943 against 993 us; 640x480: 49 against 58 us, 117
// against 118 us, all with float32 gradient sums).
static bool use_persistent(const lam_ctx* ctx) { return ctx->raster_schedule.load() == 1; }

hipError_t render_forward_launch(lam_ctx* ctx, const RenderArgs& A, const RenderLayout& L, hipStream_t st)
{
    const CamSet& cs = L.cams;
    const uint32_t R = (uint32_t)L.records;
    const uint32_t cap = (uint32_t)L.capacity;
    // counters and every look-back scratch of the sorts start at zero (cleared
    // by the projection launch when there is one)
    hipError_t e = hipSuccess;
    const size_t zero_words = (size_t)(L.zero_end - L.counters);
    if (A.n > 0 && cs.n > 0) {
        ProfScope ps(ctx, "preprocess", st);
        hipLaunchKernelGGL(k_preprocess, dim3((A.n + 255) / 256, cs.n), dim3(256), 0, st, cs, A.n,
                           A.means, A.log_scales, A.quats, A.logits, L.rec0, L.rec1, L.foot,
                           L.depth_key, L.ntiles, L.counters, zero_words);
    } else {
        e = launch_fill_u32(L.counters, zero_words, 0u, st);
        if (e != hipSuccess) return e;
    }
    bool in_b = false;
    const uint32_t* tkeys;
    const uint32_t* trecs;
    {
        ProfScope ps(ctx, "render_sort", st);
        if (R <= (uint32_t)kSmallSort)
            e = launch_sort_small(L.depth_key, R, L.recs_a, L.counters + 5, st);
        else
            e = launch_radix_sort(L.depth_key, L.depth_a, L.recs_a, L.depth_b, L.recs_b, true, nullptr,
                                  R, 32, L.sort_scratch, L.counters + 4, &in_b, st, L.counters + 5);
        if (e != hipSuccess) return e;
        const uint32_t* sorted_rec = in_b ? L.recs_b : L.recs_a;
        // pair offsets of the depth-ordered records; the last tile of the scan
        // writes the pairs needed and the overflow flag
        e = launch_excl_scan(L.ntiles, sorted_rec, L.counters + 5, R, L.offsets, L.counters, L.counters + 1, cap,
                             L.scan_scratch, L.counters + 4, st);
        if (e != hipSuccess) return e;
        if (R > 0 && cap > 0)
            hipLaunchKernelGGL(k_emit, dim3(std::min<uint32_t>((cap + 255) / 256, 8192u)), dim3(256),
                               0, st, sorted_rec, (const uint32_t*)L.offsets,
                               (const float4*)L.rec0, (const uint32_t*)L.counters, cap, L.ikeys_a,
                               L.ivals_a);
        e = launch_radix_sort(nullptr, L.ikeys_a, L.ivals_a, L.ikeys_b, L.ivals_b, false,
                              L.counters, cap, L.tile_bits, L.tile_scratch, L.counters + 4, &in_b, st);
        if (e != hipSuccess) return e;
        tkeys = in_b ? L.ikeys_b : L.ikeys_a;
        trecs = in_b ? L.ivals_b : L.ivals_a;
        if (cs.total_tiles > 0)
            hipLaunchKernelGGL(k_ranges, dim3(std::min<uint32_t>(cap / 1024 + 1, 8192u)), dim3(256), 0, st,
                               tkeys, (const uint32_t*)L.counters, cap, (uint32_t)cs.total_tiles,
                               L.ranges);
    }
    if (cs.total_tiles > 0) {
        const bool pers = use_persistent(ctx);
        const int threads = cs.tile_w * cs.tile_h;
        const bool rgbd = A.rgbd;
        auto kern = rgbd ? (A.d == 16 ? (pers ? k_raster_fwd<16, true, true> : k_raster_fwd<16, false, true>)
                                      : (pers ? k_raster_fwd<32, true, true> : k_raster_fwd<32, false, true>))
                         : (A.d == 16 ? (pers ? k_raster_fwd<16, true, false> : k_raster_fwd<16, false, false>)
                                      : (pers ? k_raster_fwd<32, true, false> : k_raster_fwd<32, false, false>));
        int grid = cs.total_tiles;
        const size_t stage = A.d == 16 ? (rgbd ? sizeof(FwdStage<16, true>) : sizeof(FwdStage<16, false>))
                                       : (rgbd ? sizeof(FwdStage<32, true>) : sizeof(FwdStage<32, false>));
        const size_t lds = stage * (threads / kWave);
        if (pers)  // its work counter, counters[2], was cleared with the sort scratch
            grid = std::min(grid, ctx_resident_blocks(ctx, (const void*)kern, threads, lds));
        ProfScope ps(ctx, "raster_fwd", st);
        hipLaunchKernelGGL(kern, dim3(grid), dim3(threads), lds, st, cs, A.n, (const uint2*)L.ranges,
                           trecs, (const float4*)L.rec0, (const float4*)L.rec1, (const uint2*)L.foot,
                           A.queries, A.Q, A.T_final, L.t_final, L.n_contrib, L.counters + 2, A.colors,
                           (const uint32_t*)L.depth_key, A.rgb, A.depth);
    }
    return hipGetLastError();
}

hipError_t render_backward_launch(lam_ctx* ctx, const RenderArgs& A, const RenderLayout& L, hipStream_t st)
{
    const CamSet& cs = L.cams;
    const bool rgbd = A.rgbd;
    hipError_t e = hipSuccess;
    if (A.n > 0) {
        const size_t work = std::max((size_t)L.records * 4, (size_t)A.n * A.d);
        const size_t blocks = std::min<size_t>((work + 255) / 256, 8192);
        hipLaunchKernelGGL(k_clear_grads, dim3((unsigned)blocks), dim3(256), 0, st,
                           (const uint32_t*)L.ntiles, (size_t)L.records, L.rec_grad,
                           rgbd ? L.rec_dz : nullptr, A.d_queries, (size_t)A.n * A.d,
                           rgbd ? A.d_colors : nullptr, (size_t)A.n * 3);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    const uint32_t* trecs = L.tile_in_b ? L.ivals_b : L.ivals_a;
    if (cs.total_tiles > 0) {
        const bool pers = use_persistent(ctx);
        const int threads = cs.tile_w * cs.tile_h;
        auto kern = rgbd ? (A.d == 16 ? (pers ? k_raster_bwd<16, true, true> : k_raster_bwd<16, false, true>)
                                      : (pers ? k_raster_bwd<32, true, true> : k_raster_bwd<32, false, true>))
                         : (A.d == 16 ? (pers ? k_raster_bwd<16, true, false> : k_raster_bwd<16, false, false>)
                                      : (pers ? k_raster_bwd<32, true, false> : k_raster_bwd<32, false, false>));
        int grid = cs.total_tiles;
        const size_t lds = sizeof(BwdStage) * (threads / kWave);
        if (pers) {
            e = launch_fill_u32(L.counters + 3, 1, 0u, st);
            if (e != hipSuccess) return e;
            grid = std::min(grid, ctx_resident_blocks(ctx, (const void*)kern, threads, lds));
        }
        ProfScope ps(ctx, "raster_bwd", st);
        hipLaunchKernelGGL(kern, dim3(grid), dim3(threads), lds, st, cs, A.n, (const uint2*)L.ranges,
                           trecs, (const float4*)L.rec0, (const float4*)L.rec1, (const uint2*)L.foot,
                           A.queries, (const float*)L.t_final, (const uint32_t*)L.n_contrib, A.dQ,
                           L.rec_grad, A.d_queries, L.counters + 3, A.colors, (const uint32_t*)L.depth_key,
                           A.d_rgb, A.d_depth, A.d_colors, L.rec_dz);
    }
    if (A.n > 0) {
        ProfScope ps(ctx, "preprocess_bwd", st);
        hipLaunchKernelGGL(k_preprocess_bwd, dim3((A.n + 255) / 256), dim3(256), 0, st, cs, A.n,
                           A.means, A.log_scales, A.quats, A.logits, (const uint32_t*)L.ntiles,
                           (const double*)L.rec_grad, rgbd ? (const float*)L.rec_dz : nullptr, A.d_means,
                           A.d_log_scales, A.d_quats, A.d_logits);
    }
    return hipGetLastError();
}

}  // namespace lam
