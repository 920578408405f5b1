// Decoding of the global (non-blocked) first-order Lorenzo predictor
// (Sec. 3.1's Lorenzo predictor with neighbours anywhere in the field).  The
// Huffman decoders leave every residual in the row-major residual field;
// the inverse is a prefix sum along each axis over the whole field.  2D
// fields, and 3D ones by the rule at launch_global_inverse:
//   k_gl_rows, k_gl_segs, k_gl_out - y in segments of 8 rows: segment sums,
//             their prefix, then x, y (and z) together with dequantised
//             stores
// 3D fields with enough planes (rows of at most 4096 values):
//   k_gl_xy    - lines along x and y together, workgroup = plane, in place
//   k_gl_z_out - lines along z, dequantised stores
// otherwise one axis per launch, in place:
//   k_gl_y  - lines along y (2D/3D): thread = (x, z), carrying the sum
//   k_gl_z  - lines along z (3D): thread = (x, y)
//   k_gl_x  - lines along x, last: one wave per row, 256 values per step by
//             in-lane and cross-lane prefix sums, dequantised row stores
//   1D  k_gl_scan1 - one prefix sum over the field: tiles of 2048 values
//             taken in order from a counter, tile sums chained by decoupled
//             look-back, dequantised stores
// Sums are modulo 2^32 (unsigned arithmetic).
#include "fz_common.h"
#include "fz_kernels.h"

namespace fz {

// Prefix sum of the n values p[0], p[st], ...: D loads in flight.
template <uint32_t D>
__device__ __forceinline__ void line_sum(uint32_t* p, uint64_t st, uint32_t n) {
    uint32_t run = 0, i = 0;
    for (; i + D <= n; i += D, p += D * st) {
        uint32_t v[D];
#pragma unroll
        for (uint32_t k = 0; k < D; k++) v[k] = p[k * st];
#pragma unroll
        for (uint32_t k = 0; k < D; k++) {
            run += v[k];
            p[k * st] = run;
        }
    }
    for (; i < n; i++, p += st) {
        run += *p;
        *p = run;
    }
}

// Line along y (2D/3D): thread = (x, z), consecutive threads on
// consecutive x, so every step reads and writes one contiguous run.
template <uint32_t D>
__global__ __launch_bounds__(256) void k_gl_y(Geom g, uint32_t* __restrict__ R) {
    const uint64_t gid = (uint64_t)blockIdx.x * 256 + threadIdx.x;
    if (gid >= (uint64_t)g.n[0] * g.n[2]) return;
    const uint64_t x = gid % g.n[0], z = gid / g.n[0];
    line_sum<D>(R + x + (uint64_t)g.n[0] * g.n[1] * z, g.n[0], g.n[1]);
}

// Line along z (3D): thread = (x, y).
template <uint32_t D>
__global__ __launch_bounds__(256) void k_gl_z(Geom g, uint32_t* __restrict__ R) {
    const uint64_t plane = (uint64_t)g.n[0] * g.n[1];
    const uint64_t gid = (uint64_t)blockIdx.x * 256 + threadIdx.x;
    if (gid >= plane) return;
    line_sum<D>(R + gid, plane, g.n[2]);
}

// Line along x (last pass, 2D/3D) with dequantisation: one wave per row,
// 256 values per step (4 per lane: a 16-byte load and store where the rows
// are aligned), in-lane and cross-lane prefix sums plus the row's carry.
__global__ __launch_bounds__(256) void k_gl_x(Geom g, const uint32_t* __restrict__ R, double e2,
                                              float* __restrict__ out, int vec) {
    const uint32_t lane = threadIdx.x & 63;
    const uint64_t row = (uint64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= (uint64_t)g.n[1] * g.n[2]) return;  // uniform per wave
    const uint64_t base = row * g.n[0];
    const uint32_t* src = R + base;
    float* dst = out + base;
    auto dq = [&](uint32_t q) { return (float)((double)(int32_t)q * e2); };
    uint32_t carry = 0;
    for (uint32_t x0 = 0; x0 < g.n[0]; x0 += 256) {
        const uint32_t x = x0 + 4 * lane;
        uint32_t v[4] = {0, 0, 0, 0};
        const bool full = vec && x + 4 <= g.n[0];
        if (full) {
            const uint4 a = *reinterpret_cast<const uint4*>(src + x);
            v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
        } else {
#pragma unroll
            for (int k = 0; k < 4; k++)
                if (x + k < g.n[0]) v[k] = src[x + k];
        }
        v[1] += v[0];
        v[2] += v[1];
        v[3] += v[2];
        const uint32_t incl = (uint32_t)wave_incl_scan(v[3]);
        const uint32_t pre = carry + incl - v[3];
        carry += (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
        if (full) {
            const f32x4 w = {dq(pre + v[0]), dq(pre + v[1]), dq(pre + v[2]), dq(pre + v[3])};
            __builtin_nontemporal_store(w, reinterpret_cast<f32x4*>(dst + x));
        } else {
#pragma unroll
            for (int k = 0; k < 4; k++)
                if (x + k < g.n[0]) dst[x + k] = dq(pre + v[k]);
        }
    }
}

// Lines along x and y together (3D, rows of at most 4096 values):
// workgroup = one plane z, wave w = the x range [256 C w, 256 C (w + 1)) of
// every row; the waves walk the rows in order with the running sums along
// y in registers (the next D - 1 rows' loads in flight), and per row take
// the prefix along x of their range plus the row totals of the waves to
// their left (LDS, two slots alternating by row, one barrier per row).  In
// place; the z pass follows and writes the output.
template <int C>
__global__ __launch_bounds__(256) void k_gl_xy(Geom g, uint32_t* __restrict__ R, int vec) {
    constexpr int D = 4;  // rows in flight per wave (8 measured the same)
    __shared__ uint32_t tot[2][4];
    const uint32_t lane = threadIdx.x & 63, w = threadIdx.x >> 6, W = blockDim.x >> 6;
    const uint32_t n0 = g.n[0], n1 = g.n[1];
    uint32_t* P = R + (uint64_t)n0 * n1 * blockIdx.x;
    const uint32_t xb = 256u * C * w + 4 * lane;  // chunk c starts at xb + 256 c
    const bool v4 = vec && (n0 & 3) == 0;
    auto load = [&](uint32_t y, uint32_t (&v)[C][4]) {
        const uint32_t* row = P + (uint64_t)n0 * y;
#pragma unroll
        for (int c = 0; c < C; c++) {
            const uint32_t x = xb + 256u * c;
            if (v4 && x + 4 <= n0) {
                const uint4 a = *reinterpret_cast<const uint4*>(row + x);
                v[c][0] = a.x; v[c][1] = a.y; v[c][2] = a.z; v[c][3] = a.w;
            } else {
#pragma unroll
                for (int k = 0; k < 4; k++) v[c][k] = x + k < n0 ? row[x + k] : 0u;
            }
        }
    };
    uint32_t cy[C][4];  // sums along y of the rows so far
#pragma unroll
    for (int c = 0; c < C; c++)
#pragma unroll
        for (int k = 0; k < 4; k++) cy[c][k] = 0;
    uint32_t buf[D][C][4];
#pragma unroll
    for (int d = 0; d < D; d++)
        if ((uint32_t)d < n1) load(d, buf[d]);
    for (uint32_t y0 = 0; y0 < n1; y0 += D) {
#pragma unroll
        for (int d = 0; d < D; d++) {
            const uint32_t y = y0 + d;  // uniform over the workgroup
            if (y >= n1) break;
            uint32_t a[C][4];
#pragma unroll
            for (int c = 0; c < C; c++)
#pragma unroll
                for (int k = 0; k < 4; k++) {
                    cy[c][k] += buf[d][c][k];
                    a[c][k] = cy[c][k];
                }
            if (y + D < n1) load(y + D, buf[d]);
            uint32_t carry = 0;
#pragma unroll
            for (int c = 0; c < C; c++) {
                a[c][1] += a[c][0];
                a[c][2] += a[c][1];
                a[c][3] += a[c][2];
                const uint32_t incl = wave_incl_scan(a[c][3]);
                const uint32_t pre = carry + incl - a[c][3];
#pragma unroll
                for (int k = 0; k < 4; k++) a[c][k] += pre;
                carry += (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
            }
            if (lane == 0) tot[y & 1][w] = carry;
            __syncthreads();
            uint32_t left = 0;
            for (uint32_t u = 0; u < W; u++) left += u < w ? tot[y & 1][u] : 0u;
            uint32_t* row = P + (uint64_t)n0 * y;
#pragma unroll
            for (int c = 0; c < C; c++) {
                const uint32_t x = xb + 256u * c;
                if (v4 && x + 4 <= n0) {
                    *reinterpret_cast<uint4*>(row + x) =
                        make_uint4(a[c][0] + left, a[c][1] + left, a[c][2] + left, a[c][3] + left);
                } else {
#pragma unroll
                    for (int k = 0; k < 4; k++)
                        if (x + k < n0) row[x + k] = a[c][k] + left;
                }
            }
        }
    }
}

// Line along z with dequantisation (3D, after k_gl_xy): thread = 4
// consecutive x of one (x, y) row segment, walking z.
__global__ __launch_bounds__(256) void k_gl_z_out(Geom g, const uint32_t* __restrict__ R, double e2,
                                                  float* __restrict__ out, int vec) {
    const uint64_t plane = (uint64_t)g.n[0] * g.n[1];
    const uint64_t i0 = 4 * ((uint64_t)blockIdx.x * 256 + threadIdx.x);
    if (i0 >= plane) return;
    auto dq = [&](uint32_t q) { return (float)((double)(int32_t)q * e2); };
    const bool v4 = vec && (plane & 3) == 0;  // then i0 + 4 <= plane
    uint32_t c[4] = {0, 0, 0, 0};
    for (uint32_t z = 0; z < g.n[2]; z++) {
        const uint64_t i = i0 + plane * z;
        if (v4) {
            const uint4 a = *reinterpret_cast<const uint4*>(R + i);
            c[0] += a.x; c[1] += a.y; c[2] += a.z; c[3] += a.w;
            const f32x4 o = {dq(c[0]), dq(c[1]), dq(c[2]), dq(c[3])};
            __builtin_nontemporal_store(o, reinterpret_cast<f32x4*>(out + i));
        } else {
#pragma unroll
            for (int k = 0; k < 4; k++)
                if (i0 + k < plane) {
                    c[k] += R[i + k];
                    out[i + k] = dq(c[k]);
                }
        }
    }
}

// Two-pass inverse along y, z and x together (2D/3D, rows of at most 4096
// values), the y axis cut into segments of kGlSeg rows:
//   k_gl_rows - column sums of each segment's rows in each plane, left in the
//               segment's first row of the output field
//   k_gl_segs - exclusive prefix of those sums along the segments
//   k_gl_out  - one workgroup per segment and whole rows, walking z
// Reads the residuals twice and writes the output once, where a pass per
// axis reads and writes the field three times; bound by memory (26 x 1800 x
// 3600: 2.1 GB in 497 us, 4.3 TB/s; a pass per axis 903 us).
constexpr uint32_t kGlSeg = 8;

// thread = 4 consecutive x of one segment and plane
__global__ __launch_bounds__(256) void k_gl_rows(Geom g, const uint32_t* __restrict__ R, uint32_t nseg,
                                                 uint32_t* __restrict__ S, int vec) {
    const uint32_t n0 = g.n[0], n1 = g.n[1], X = (n0 + 3) / 4;
    const uint32_t gid = blockIdx.x * 256 + threadIdx.x;
    const uint32_t r = gid / X, x = 4 * (gid - r * X);
    const uint32_t z = r / nseg, s = r - z * nseg;
    if (z >= g.n[2]) return;
    const uint32_t y0 = s * kGlSeg, rows = min(kGlSeg, n1 - y0);
    const uint64_t i0 = x + (uint64_t)n0 * (y0 + (uint64_t)n1 * z);
    uint32_t c[4] = {0, 0, 0, 0};
    if (vec && (n0 & 3) == 0) {
#pragma unroll
        for (uint32_t y = 0; y < kGlSeg; y++)
            if (y < rows) {
                const uint4 a = *reinterpret_cast<const uint4*>(R + i0 + (uint64_t)n0 * y);
                c[0] += a.x; c[1] += a.y; c[2] += a.z; c[3] += a.w;
            }
        *reinterpret_cast<uint4*>(S + i0) = make_uint4(c[0], c[1], c[2], c[3]);
    } else {
#pragma unroll
        for (uint32_t y = 0; y < kGlSeg; y++)
#pragma unroll
            for (uint32_t k = 0; k < 4; k++)
                if (y < rows && x + k < n0) c[k] += R[i0 + (uint64_t)n0 * y + k];
#pragma unroll
        for (uint32_t k = 0; k < 4; k++)
            if (x + k < n0) S[i0 + k] = c[k];
    }
}

// thread = (x, z), walking the segments, 16 loads in flight
__global__ __launch_bounds__(256) void k_gl_segs(Geom g, uint32_t nseg, uint32_t* __restrict__ S) {
    const uint64_t gid = (uint64_t)blockIdx.x * 256 + threadIdx.x;
    if (gid >= (uint64_t)g.n[0] * g.n[2]) return;
    const uint64_t z = gid / g.n[0], x = gid - z * g.n[0], st = (uint64_t)g.n[0] * kGlSeg;
    uint32_t* p = S + x + (uint64_t)g.n[0] * g.n[1] * z;
    uint32_t run = 0;
    for (uint32_t s = 0; s < nseg; s += 16, p += 16 * st) {
        uint32_t v[16];
#pragma unroll
        for (uint32_t k = 0; k < 16; k++) v[k] = s + k < nseg ? p[k * st] : 0u;
#pragma unroll
        for (uint32_t k = 0; k < 16; k++) {
            if (s + k < nseg) p[k * st] = run;
            run += v[k];
        }
    }
}

// Workgroup = segment of 8 rows, thread = 4 consecutive x of every row, the
// sums along z (of the prefix along y) in registers; the next plane's rows
// are loaded before this one's are summed.  The prefix along x is taken per
// wave, then the totals of the waves to the left are added (LDS, two slots
// alternating by plane, one barrier each).  `carry`: the segment's sums of
// the rows above, in the rows of `out` that this thread writes afterwards.
__global__ __launch_bounds__(1024) void k_gl_out(Geom g, const uint32_t* __restrict__ R, uint32_t nseg,
                                                 uint32_t nz, double e2, float* out, int vec) {
    constexpr int S = (int)kGlSeg;
    __shared__ uint32_t tot[2][S * 16];
    const uint32_t lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const uint32_t n0 = g.n[0], n1 = g.n[1];
    const uint32_t zr = blockIdx.x / nseg, y0 = (blockIdx.x - zr * nseg) * S, rows = min((uint32_t)S, n1 - y0);
    const uint32_t x = 4 * threadIdx.x;
    const bool v4 = vec && (n0 & 3) == 0;
    const uint64_t plane = (uint64_t)n0 * n1;
    const uint64_t i0 = x + (uint64_t)n0 * y0 + plane * nz * zr;
    auto dq = [&](uint32_t q) { return (float)((double)(int32_t)q * e2); };
    auto load4 = [&](const uint32_t* p, uint32_t (&v)[4]) {
        if (v4 && x < n0) {
            const uint4 a = *reinterpret_cast<const uint4*>(p);
            v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
        } else {
#pragma unroll
            for (int k = 0; k < 4; k++) v[k] = x + k < n0 ? p[k] : 0u;
        }
    };
    uint32_t acc[S][4], buf[S][4], top[4] = {0, 0, 0, 0};
#pragma unroll
    for (int y = 0; y < S; y++)
#pragma unroll
        for (int k = 0; k < 4; k++) acc[y][k] = buf[y][k] = 0;
    auto load = [&](uint32_t z) {
        const uint64_t i = i0 + plane * z;
        if (nseg > 1) load4(reinterpret_cast<const uint32_t*>(out + i), top);
#pragma unroll
        for (int y = 0; y < S; y++)
            if ((uint32_t)y < rows) load4(R + i + (uint64_t)n0 * y, buf[y]);
    };
    load(0);
    for (uint32_t z = 0; z < nz; z++) {
        uint32_t c[4];
#pragma unroll
        for (int k = 0; k < 4; k++) c[k] = top[k];
#pragma unroll
        for (int y = 0; y < S; y++)
#pragma unroll
            for (int k = 0; k < 4; k++) {
                c[k] += buf[y][k];
                acc[y][k] += c[k];
            }
        if (z + 1 < nz) load(z + 1);
        uint32_t pre[S];
        uint32_t* T = tot[z & 1];
#pragma unroll
        for (int y = 0; y < S; y++) {
            const uint32_t sum = (acc[y][0] + acc[y][1]) + (acc[y][2] + acc[y][3]);
            const uint32_t incl = wave_incl_scan(sum);
            pre[y] = incl - sum;
            if (lane == 63) T[y * 16 + w] = incl;
        }
        __syncthreads();
#pragma unroll
        for (int h = 0; h < S / 4; h++) {
            // lane = (row 4 h + lane / 16, wave lane % 16)
            uint32_t t = (lane & 15) < w ? T[64 * h + lane] : 0u;
            t += dpp32<0x111, 0xf>(t);
            t += dpp32<0x112, 0xf>(t);
            t += dpp32<0x114, 0xf>(t);
            t += dpp32<0x118, 0xf>(t);
#pragma unroll
            for (int j = 0; j < 4; j++)
                pre[4 * h + j] += (uint32_t)__builtin_amdgcn_readlane((int)t, 16 * j + 15);
        }
        float* o = out + i0 + plane * z;
#pragma unroll
        for (int y = 0; y < S; y++) {
            if ((uint32_t)y >= rows) break;
            float* oy = o + (uint64_t)n0 * y;
            const uint32_t q0 = pre[y] + acc[y][0], q1 = q0 + acc[y][1], q2 = q1 + acc[y][2], q3 = q2 + acc[y][3];
            if (v4 && x < n0) {
                const f32x4 f = {dq(q0), dq(q1), dq(q2), dq(q3)};
                __builtin_nontemporal_store(f, reinterpret_cast<f32x4*>(oy));
            } else {
                if (x < n0) oy[0] = dq(q0);
                if (x + 1 < n0) oy[1] = dq(q1);
                if (x + 2 < n0) oy[2] = dq(q2);
                if (x + 3 < n0) oy[3] = dq(q3);
            }
        }
    }
}

constexpr uint32_t kScan1 = 2048;  // values per tile of the 1D scan

__global__ __launch_bounds__(256) void k_gl_scan1(uint64_t N, const uint32_t* __restrict__ R, uint32_t ntiles,
                                                  uint64_t* desc, Misc* misc, double e2, float* __restrict__ out) {
    __shared__ uint32_t s_tile;
    __shared__ uint32_t wsum[4];
    __shared__ uint64_t s_excl;
    const uint32_t t = threadIdx.x, lane = t & 63, wave = t >> 6;
    if (t == 0) s_tile = atomicAdd(&misc->mtile_ctr, 1u);
    __syncthreads();
    const uint32_t tile = s_tile;
    if (tile >= ntiles) return;  // uniform: the grid is exactly ntiles
    const uint64_t i0 = (uint64_t)tile * kScan1 + 8ull * t;
    uint32_t v[8];
#pragma unroll
    for (int k = 0; k < 8; k++) v[k] = i0 + k < N ? R[i0 + k] : 0u;
#pragma unroll
    for (int k = 1; k < 8; k++) v[k] += v[k - 1];
    const uint32_t incl = (uint32_t)wave_incl_scan(v[7]);
    if (lane == 63) wsum[wave] = incl;
    __syncthreads();
    uint32_t wpre = 0, total = 0;
#pragma unroll
    for (uint32_t w = 0; w < 4; w++) {
        wpre += w < wave ? wsum[w] : 0u;
        total += wsum[w];
    }
    if (wave == 0) {
        const uint64_t ex = lookback(desc, tile, (uint64_t)total, OpAdd(), &misc->flags);
        if (lane == 0) s_excl = ex;
    }
    __syncthreads();
    const uint32_t base = (uint32_t)s_excl + wpre + incl - v[7];
#pragma unroll
    for (int k = 0; k < 8; k++)
        if (i0 + k < N) __builtin_nontemporal_store((float)((double)(int32_t)(base + v[k]) * e2), out + i0 + k);
}

uint32_t global_scan_tiles(uint64_t N) { return (uint32_t)((N + kScan1 - 1) / kScan1); }

// The fused x/y pass walks each plane's rows in order, one workgroup per
// plane: it needs at least this many waves to keep HBM busy (1024^3: 4096
// waves, 4.9 -> 3.4 ms for the inverse; 512^3 has 1024 waves and runs the
// separate passes, 0.56 ms against 0.64 fused)
constexpr uint64_t kGlFusedWaves = 2048;

// Lines of a pass along y or z from which 4 loads in flight per thread
// reach the memory's rate; with fewer lines 16 (560 x 40 x 560, z lines
// 22400: 116 us with 4, 80 with 16; 512^3, 262144 lines: 549 with 4, 570
// with 16)
constexpr uint64_t kGlDeep = 131072;

// Segments (k_gl_rows, k_gl_segs, k_gl_out) or a pass per axis, microseconds
// per axis / segments:
//   2D always: 1800 x 3600 234/36, 500 x 500 60/18, 3600 x 64 230/39,
//     64 x 3600 22/18
//     (whole calls of long, narrow fields, a serial chain either way:
//     20000 x 200 2401/226, 100000 x 40 10017/720, 2000000 x 3 93537/12575)
//   3D, enough waves (2048 full ones) to walk z inside k_gl_out: 26 x 1800 x 3600
//     903/497 (256^3 would take 938 so: 4 us a plane, one after the other)
//   3D, fewer: a z pass first, then k_gl_out takes every plane on its own:
//     128^3 39/27, 256^3 93/67, 500 x 500 x 100 178/131, 512^3 572/544;
//     not where the field is small (below 2^17 values, one launch more:
//     40^3 17/20), nor where the line passes fill the chip and the field
//     stays in the last-level cache (384^3: 217/232)
constexpr uint64_t kGlWalk = 2048 * 256, kGlSmall = 1u << 17, kGlCached = 1u << 26;

void launch_global_inverse(hipStream_t st, const Geom& g, int32_t* res, uint64_t* desc, Misc* misc, double e2,
                           float* out, int vec) {
    uint32_t* R = reinterpret_cast<uint32_t*>(res);
    auto grid = [](uint64_t threads) { return dim3((uint32_t)((threads + 255) / 256)); };
    const uint32_t C = g.n[0] <= 1024 ? 1u : (g.n[0] <= 2048 ? 2u : 4u);  // chunks of 256 per wave and row
    const uint32_t W = (g.n[0] + 256 * C - 1) / (256 * C);                 // waves per plane
    const uint64_t ly = (uint64_t)g.n[0] * g.n[2], lz = (uint64_t)g.n[0] * g.n[1];
    auto line_z = [&]() {
        if (lz < kGlDeep) hipLaunchKernelGGL(k_gl_z<16>, grid(lz), dim3(256), 0, st, g, R);
        else hipLaunchKernelGGL(k_gl_z<4>, grid(lz), dim3(256), 0, st, g, R);
    };
    const bool xy = g.ndim == 3 && g.n[0] <= 4096 && (uint64_t)g.n[2] * W >= kGlFusedWaves;
    const uint32_t nseg = (g.n[1] + kGlSeg - 1) / kGlSeg, WS = (g.n[0] + 255) / 256;
    const bool walk = g.ndim == 2 || (uint64_t)nseg * g.n[0] >= kGlWalk;
    const bool lines = g.N < kGlSmall || (ly >= kGlDeep && lz >= kGlDeep && g.N < kGlCached);
    if (g.ndim >= 2 && g.n[0] <= 4096 && (walk || (!xy && !lines))) {
        uint32_t* S = reinterpret_cast<uint32_t*>(out);
        if (!walk) line_z();
        if (nseg > 1) {
            hipLaunchKernelGGL(k_gl_rows, grid((uint64_t)((g.n[0] + 3) / 4) * nseg * g.n[2]), dim3(256), 0, st, g, R,
                               nseg, S, vec);
            hipLaunchKernelGGL(k_gl_segs, grid((uint64_t)g.n[0] * g.n[2]), dim3(256), 0, st, g, nseg, S);
        }
        hipLaunchKernelGGL(k_gl_out, dim3(walk ? nseg : nseg * g.n[2]), dim3(64 * WS), 0, st, g, R, nseg,
                           walk ? g.n[2] : 1u, e2, out, vec);
    } else if (xy) {
        // x and y together in place, then z with the dequantised stores
        if (C == 1) hipLaunchKernelGGL(k_gl_xy<1>, dim3(g.n[2]), dim3(64 * W), 0, st, g, R, vec);
        else if (C == 2) hipLaunchKernelGGL(k_gl_xy<2>, dim3(g.n[2]), dim3(64 * W), 0, st, g, R, vec);
        else hipLaunchKernelGGL(k_gl_xy<4>, dim3(g.n[2]), dim3(64 * W), 0, st, g, R, vec);
        const uint64_t plane = (uint64_t)g.n[0] * g.n[1];
        hipLaunchKernelGGL(k_gl_z_out, grid((plane + 3) / 4), dim3(256), 0, st, g, R, e2, out, vec);
    } else if (g.ndim >= 2) {
        // y (and z) in place, then x, the output's contiguous axis, with the
        // dequantised stores
        if (ly < kGlDeep) hipLaunchKernelGGL(k_gl_y<16>, grid(ly), dim3(256), 0, st, g, R);
        else hipLaunchKernelGGL(k_gl_y<4>, grid(ly), dim3(256), 0, st, g, R);
        if (g.ndim == 3) line_z();
        const int xvec = vec && (g.n[0] & 3) == 0;
        hipLaunchKernelGGL(k_gl_x, grid(64ull * g.n[1] * g.n[2]), dim3(256), 0, st, g, R, e2, out, xvec);
    } else {
        const uint32_t nt = global_scan_tiles(g.N);
        launch_fill32(st, reinterpret_cast<uint32_t*>(desc), 2ull * nt, 0u);
        hipLaunchKernelGGL(k_gl_scan1, dim3(nt), dim3(256), 0, st, g.N, R, nt, desc, misc, e2, out);
    }
}

}  // namespace fz
