// k_edt.hip -- signed distance of a voxel image on the GPU (exact Euclidean distance
// transform), the level-set description of the pore space (paper: section "Level-set
// method for image-based geometry reconstruction", eq. SDF; building it on the GPU is
// the future work named in section "Discussion and conclusions").
//
// phi at an active voxel is (distance to the nearest inactive voxel centre - 1/2) dx, at
// an inactive voxel -(distance to the nearest active voxel centre - 1/2) dx; with no
// voxel of the other phase it is +-(box diagonal) dx.  Squared distances are exact
// integers, built one axis at a time as in every separable transform (the squared distance
// to a set is the minimum over a line of offset^2 plus the squared distance within the
// axes done so far).  Both phases share one array: at a voxel only the distance to the
// other phase is needed, and seen from the other phase the voxel is itself a feature
// (distance 0), so a value and a phase bit per voxel serve both transforms.
//   k_edt_x   one wave per row: ballots of the row's voxels, the nearest bit of the other
//             phase by leading / trailing zero counts
//   k_edt_y   one wave per 64 voxels of x by 8 rows: outward search along y (edt_tile)
//   k_edt_z   the same along z, with the square root and the sign
// The search stops where the offset alone reaches the best value of every lane, so its
// length is the distance (a few voxels in a porous medium) and voxels are independent,
// where a lower envelope of parabolas walks each line in one serial chain per thread.
// Measured on a soil image of 365 x 411 x 320 (48 M voxels, 5 bytes per voxel in and out):
// x 148 us, y 250 us, z 244 us, bound by vector instructions (4 + 4 bytes per voxel and
// pass would take 80 us); one wave per row of 64 voxels and a load per candidate took
// 888 / 643 us for y / z, envelope passes 2870 us each and twice (one per phase).  With
// distances as long as the lines (512^3, one voxel of the other phase): 3.5 ms, against
// 17.9 ms without the windows of edt_tile and 5.7 ms for the envelopes; 1024^3 17.2 and 34.0
// ms, with 1e-3 of the voxels of the other phase 12.2 and 113 ms; 4096 x 4096 x 1 22.5 and 24.1.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <mutex>
#include <string>

#include "rd_host.h"

namespace {

// Words of every pass: the squared distance v >= 1 within the axes done so far as +v at an
// active voxel, -v at an inactive one; v = EDT_FAR: none.  Squared distances stay below
// EDT_FAR: 2 * 32767^2 does, and with two axes of 32768 voxels the scratch of a third
// longer than 32 would not fit any GPU.
constexpr int EDT_FAR = 0x7fffffff;
constexpr int EDT_ROWS = 8;  // rows of a tile, of its margins and of a far window
// Lines up to EDT_LONG are searched by rows' summaries alone (RUNS = 0), longer ones also by
// those of runs of 64 rows (1) and, above EDT_LONGER, of 512 (2).  ms with 0, 1 and 2 (512^3: 0
// and 2): one voxel of the other phase in 512^3 3.5 / 1.9, 768^3 15.8 / 6.8 / 6.8, 1024^3 47.4
// / 17.2 / 16.6; packed balls of an eighth of the edge 2.60 / 2.70, 8.6 / 8.8 / 8.9, 25.1 / 25.7 /
// 26.0; one voxel in 4096 x 4096 x 1 to x 64 165 with 0, 22.6 with 2.
constexpr int EDT_LONG = 512, EDT_LONGER = 2048;

// n workgroups in rows of at most 2^20, a multiple of 8: one dimension of a grid holds fewer
// than 2^32 threads, and images of flat or thin shape (32768 x 1 x 32768) need more.
constexpr int64_t EDT_GRID_ROW = 1 << 20;
dim3 edt_grid(int64_t n)
{
    const int64_t row = n < EDT_GRID_ROW ? (n + 7) / 8 * 8 : EDT_GRID_ROW;
    return dim3((unsigned)row, (unsigned)((n + row - 1) / row));
}

// Workgroup id of such a grid (a few come out past the last one) so that each XCD
// (consecutive workgroups go round-robin to the 8 of them) walks one contiguous range of ids
// in a row: the lines it reads are then shared in its own L2.
__device__ __forceinline__ uint32_t xcd_range()
{
    return blockIdx.y * (uint32_t)EDT_GRID_ROW + (blockIdx.x & 7u) * (gridDim.x >> 3) + (blockIdx.x >> 3);
}

// The summary word of a wave's 64 words: the one nearest 0 if all are of one phase, else 0
// (for either viewer the row then holds a feature).
__device__ __forceinline__ int edt_summary(int w, bool valid)
{
    const uint64_t v = __ballot(valid), on = __ballot(valid && w > 0);
    if (on != 0ull && on != v) return 0;
    int m = valid ? max(w, -w) : EDT_FAR;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) m = min(m, __shfl_xor(m, o, 64));
    return on ? m : -m;
}

__global__ __launch_bounds__(256) void k_edt_x(const uint8_t *__restrict__ img, int nx, int ny, int64_t nrows,
                                               int *__restrict__ g, int *__restrict__ sum)
{
    extern __shared__ uint64_t words[];  // 4 waves x chunks of 64 voxels
    const int64_t row = ((int64_t)blockIdx.y * EDT_GRID_ROW + blockIdx.x) * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (row >= nrows) return;  // whole waves; no workgroup barrier below
    const int nc = (nx + 63) / 64;
    uint64_t *W = words + (threadIdx.x >> 6) * nc;
    const uint8_t *r = img + row * nx;
    int *out = g + row * nx;
    int *rs = sum + (row / ny) * nc * ny + row % ny;  // [z][chunk][y]
    for (int c0 = 0; c0 < nc; c0 += 8) {  // eight chunks' loads in flight
        uint8_t v[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) v[k] = (c0 + k) * 64 + lane < nx ? r[(c0 + k) * 64 + lane] : (uint8_t)0;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const uint64_t w = __ballot(v[k] != 0);
            if (lane == 0 && c0 + k < nc) W[c0 + k] = w;
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    // A voxel's nearest neighbours of the other phase are just outside its run of equal
    // voxels: T marks the first voxel of every run but the row's first, so the run of lane i
    // starts at the highest mark at or below i and ends before the lowest mark above it.
    auto marks = [&](int c) {
        const uint64_t w = W[c], first = c > 0 ? W[c - 1] >> 63 : w & 1ull;
        const uint64_t t = w ^ (w << 1 | first);
        return c + 1 < nc || !(nx & 63) ? t : t & ((1ull << (nx & 63)) - 1ull);
    };
    const uint64_t upto = ~0ull >> (63 - lane), above = ~upto;
    int start = -1;         // the run reaching into the chunk (-1: the row's first)
    int next = -1, at = 0;  // first mark after the chunk, in chunk `at` (nc: none)
    for (int c = 0; c < nc; ++c) {
        const uint64_t T = marks(c);
        if (at <= c) {  // searched again only once that chunk is reached: the row is walked once
            uint64_t m = 0ull;
            for (at = c + 1; at < nc; ++at)
                if ((m = marks(at)) != 0ull) break;
            next = m ? at * 64 + __builtin_ctzll(m) : -1;
        }
        const int i = c * 64 + lane;
        const uint64_t lo = T & upto, hi = T & above;
        const int l = lo ? c * 64 + 63 - __builtin_clzll(lo) : start;
        const int h = hi ? c * 64 + __builtin_ctzll(hi) : next;
        const uint32_t d = min(l >= 0 ? (uint32_t)(i - l + 1) : ~0u, h >= 0 ? (uint32_t)(h - i) : ~0u);
        const int v = d == ~0u ? EDT_FAR : (int)(d * d);
        const bool own = (W[c] >> lane) & 1ull;
        if (i < nx) out[i] = own ? v : -v;
        if (T == 0ull || T == 1ull) {  // one phase: the least distance is at an end
            const int e = min(__builtin_amdgcn_readfirstlane(v), __builtin_amdgcn_readlane(v, min(63, nx - 1 - c * 64)));
            if (lane == 0) rs[(int64_t)c * ny] = own ? e : -e;
        } else if (lane == 0) {
            rs[(int64_t)c * ny] = 0;
        }
        if (T) start = c * 64 + 63 - __builtin_clzll(T);
    }
}

// What 8 rows hold for the viewers of either phase: act for active voxels (0 at an
// inactive one), ina for inactive voxels.
struct EdtRows {
    int act[EDT_ROWS], ina[EDT_ROWS];
    // rows r0 .. r0 + 7 of the line, clamped to its n rows: an end row seen once more at a
    // larger offset never wins
    __device__ __forceinline__ void load(const int *line, int64_t stride, int n, int r0, uint32_t x)
    {
        int w[EDT_ROWS];
#pragma unroll
        for (int s = 0; s < EDT_ROWS; ++s) w[s] = (line + min(max(r0 + s, 0), n - 1) * stride)[x];
        set(w);
    }
    __device__ __forceinline__ void set(const int w[EDT_ROWS])
    {
#pragma unroll
        for (int s = 0; s < EDT_ROWS; ++s) {
            act[s] = max(w[s], 0);
            ina[s] = act[s] - w[s];
        }
    }
};

// The squared distances of the lane's voxels in rows p0 .. p0 + 7 of a line of n rows,
// as words.  line + r * stride is row r at x = 0 (wave-uniform), x the lane's column, sum[r]
// the summary word of row r.  The near candidates come from the tile and its two margins
// (24 rows in registers, loaded once).  Farther away, windows of 8 rows are
// read outward, each only if its summaries can still improve a voxel of the tile: across
// a large void or solid that is one scalar load per 8 rows, or with RUNS one per 64 or 512
// (c64: summaries of the line's rows in aligned runs of 64).
template <int RUNS>
__device__ __forceinline__ void edt_tile(const int *line, int64_t stride, const int *sum, const int *c64, int p0, int n,
                                         uint32_t x, int out[EDT_ROWS])
{
    constexpr int R = EDT_ROWS;
    EdtRows own, lo, hi;
    own.load(line, stride, n, p0, x);
    lo.load(line, stride, n, p0 - R, x);
    hi.load(line, stride, n, p0 + R, x);
    uint32_t best[R];
    bool act[R];
#pragma unroll
    for (int t = 0; t < R; ++t) {
        act[t] = own.act[t] > 0;
        best[t] = (uint32_t)(own.act[t] + own.ina[t]);
    }
    // row p0 + q (-8 <= q < 16) for voxel t
    auto seen = [&](int t, int q) {
        const EdtRows &e = q < 0 ? lo : q < R ? own : hi;
        const int j = q & (R - 1);
        return (uint32_t)(act[t] ? e.act[j] : e.ina[j]);
    };
#pragma unroll
    for (int t = 0; t < R; ++t) {
#pragma unroll
        for (int k = 1; k <= R; ++k) best[t] = min(best[t], min(seen(t, t - k), seen(t, t + k)) + (uint32_t)(k * k));
        // the rest of the margins, on one side only
        if (!__any(best[t] > (uint32_t)((R + 1) * (R + 1)))) continue;
#pragma unroll
        for (int k = R + 1; k < 2 * R; ++k) {
            if (t - k >= -R) best[t] = min(best[t], seen(t, t - k) + (uint32_t)(k * k));
            if (t + k < 2 * R) best[t] = min(best[t], seen(t, t + k) + (uint32_t)(k * k));
        }
    }
    int skip[2] = {0, 0};  // RUNS: rows nearer than this are known not to help, below and above
    for (int k0 = R + 1;; k0 += R) {
        const int e = p0 + 1 - k0, b = p0 + R - 1 + k0;  // rows below e and from b on are not seen yet
        if (e <= 0 && b >= n) break;
        uint32_t ma = 0u, mi = 0u;  // the worst of the tile's active and of its inactive voxels
#pragma unroll
        for (int t = 0; t < R; ++t) {
            ma = max(ma, act[t] ? best[t] : 0u);
            mi = max(mi, act[t] ? 0u : best[t]);
        }
        if (!__any(max(ma, mi) > (uint32_t)(k0 * k0))) break;
        // RUNS: no row with one of these summaries, at least k0 away, improves a voxel of the tile
        auto useless = [&](const int *w, int count) {
            int sa = EDT_FAR, si = EDT_FAR;
#pragma unroll
            for (int s = 0; s < count; ++s) {
                sa = min(sa, max(w[s], 0));
                si = min(si, max(-w[s], 0));
            }
            return !__any(ma > (uint32_t)sa + (uint32_t)(k0 * k0) || mi > (uint32_t)si + (uint32_t)(k0 * k0));
        };
#pragma unroll
        for (int dir = 0; dir < 2; ++dir) {
            if (dir ? b >= n : e <= 0) continue;
            if constexpr (RUNS > 0) {
                if (k0 < skip[dir]) continue;
                const int row = dir ? b : e, r64 = dir ? row >> 6 : (row >> 6) - 1, n64 = (n + 63) >> 6;
                if (RUNS > 1 && (row & 511) == 0 && useless(c64 + (dir ? min(r64, n64 - R) : r64 - (R - 1)), R)) {
                    skip[dir] = k0 + 512;
                    continue;
                }
                if ((row & 63) == 0 && useless(c64 + r64, 1)) {
                    skip[dir] = k0 + 64;
                    continue;
                }
            }
            const int r0 = dir ? min(b, n - R) : max(e - R, 0);  // n > R here
            int sa = EDT_FAR, si = EDT_FAR;
#pragma unroll
            for (int s = 0; s < R; ++s) {
                const int v = sum[r0 + s];
                sa = min(sa, max(v, 0));
                si = min(si, max(-v, 0));
            }
            if (!__any(ma > (uint32_t)sa + (uint32_t)(k0 * k0) || mi > (uint32_t)si + (uint32_t)(k0 * k0))) continue;
            EdtRows w;
            w.load(line, stride, n, dir ? b : e - R, x);
#pragma unroll
            for (int t = 0; t < R; ++t) {
                // nearest row of the window: k0 + t (below) or k0 + 7 - t (above) away
                const int kt = k0 + (dir ? R - 1 - t : t);
                if (!__any(best[t] > (uint32_t)(kt * kt))) continue;
#pragma unroll
                for (int s = 0; s < R; ++s) {
                    const int j = dir ? s : R - 1 - s;
                    best[t] = min(best[t], (uint32_t)(act[t] ? w.act[j] : w.ina[j]) + (uint32_t)((kt + s) * (kt + s)));
                }
            }
        }
        if constexpr (RUNS > 0) k0 = max(k0, min(e > 0 ? skip[0] : n, b < n ? skip[1] : n) - R);
    }
#pragma unroll
    for (int t = 0; t < R; ++t) out[t] = act[t] ? (int)best[t] : -(int)best[t];
}

// Summaries of the aligned runs of 64 rows of every line from those of its n rows, four per wave.
__global__ __launch_bounds__(256) void k_edt_runs(const int *__restrict__ sum, int n, int64_t nlines,
                                                  int *__restrict__ c64)
{
    const int n64 = (n + 63) / 64, n256 = (n + 255) / 256, lane = threadIdx.x & 63;
    const int64_t wave = ((int64_t)blockIdx.y * EDT_GRID_ROW + blockIdx.x) * 4 + (threadIdx.x >> 6), l = wave / n256;
    if (l >= nlines) return;
    const int r0 = (int)(wave % n256) * 4;
    int w[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) w[k] = (r0 + k) * 64 + lane < n ? sum[l * n + (r0 + k) * 64 + lane] : 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int v = edt_summary(w[k], (r0 + k) * 64 + lane < n);
        if (lane == 0 && r0 + k < n64) c64[l * n64 + r0 + k] = v;
    }
}

// Four tiles of one 64-voxel column block of a plane per workgroup.
template <int RUNS>
__global__ __launch_bounds__(256) void k_edt_y(const int *__restrict__ g, const int *__restrict__ gsum,
                                               const int *__restrict__ c64, int nx, int ny, int nz, int nc,
                                               int *__restrict__ h, int *__restrict__ hsum)
{
    const uint32_t wg = xcd_range(), nt = (uint32_t)(ny + 31) / 32;
    const int c = (int)(wg / nt % (uint32_t)nc), z = (int)(wg / nt / (uint32_t)nc);
    const int y0 = ((int)(wg % nt) * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6)) * EDT_ROWS;
    if (z >= nz || y0 >= ny) return;
    const int lane = threadIdx.x & 63;
    const bool in = c * 64 + lane < nx;
    const uint32_t x = (uint32_t)min(c * 64 + lane, nx - 1);
    int w[EDT_ROWS];
    const int64_t l = (int64_t)z * nc + c;
    edt_tile<RUNS>(g + (int64_t)z * ny * nx, nx, gsum + l * ny, c64 + l * ((ny + 63) / 64), y0, ny,
                   x, w);
    int *out = h + ((int64_t)z * ny + y0) * nx;
#pragma unroll
    for (int t = 0; t < EDT_ROWS; ++t) {
        if (y0 + t >= ny) break;
        if (in) out[(int64_t)t * nx + x] = w[t];
        const int s = edt_summary(w[t], in);
        if (lane == 0) hsum[((int64_t)(y0 + t) * nc + c) * nz + z] = s;  // [y][chunk][z]
    }
}

// Four tiles of one 64-voxel piece of a row through the planes per workgroup.
template <int RUNS>
__global__ __launch_bounds__(256) void k_edt_z(const int *__restrict__ h, const int *__restrict__ hsum,
                                               const int *__restrict__ c64, int nx, int ny, int nz, int nc,
                                               double dx, double diag, float *__restrict__ sdf)
{
    const uint32_t wg = xcd_range(), nt = (uint32_t)(nz + 31) / 32;
    const int c = (int)(wg / nt % (uint32_t)nc), y = (int)(wg / nt / (uint32_t)nc);
    const int z0 = ((int)(wg % nt) * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6)) * EDT_ROWS;
    if (y >= ny || z0 >= nz) return;
    const int lane = threadIdx.x & 63;
    const bool in = c * 64 + lane < nx;
    const uint32_t x = (uint32_t)min(c * 64 + lane, nx - 1);
    const int64_t plane = (int64_t)ny * nx;
    int w[EDT_ROWS];
    const int64_t l = (int64_t)y * nc + c;
    edt_tile<RUNS>(h + (int64_t)y * nx, plane, hsum + l * nz, c64 + l * ((nz + 63) / 64), z0, nz, x,
                   w);
    float *out = sdf + z0 * plane + (int64_t)y * nx;
#pragma unroll
    for (int t = 0; t < EDT_ROWS; ++t) {
        if (z0 + t >= nz) break;
        const int v = max(w[t], -w[t]);
        const double d = v == EDT_FAR ? diag : sqrt((double)v) - 0.5;
        if (in) out[t * plane + x] = (float)((w[t] > 0 ? d : -d) * dx);
    }
}

}  // namespace

static size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// Fixed scratch of rd_sdf_from_image_static: one array per GPU, resident until the
// process ends.  Host code uses only the device address fetched per device below; the
// array's name on the host is a stand-in, not a device address.
#define RD_SDF_STATIC_BYTES ((size_t)64 << 20)
static __device__ __align__(256) unsigned char scratch[RD_SDF_STATIC_BYTES];

namespace {
constexpr int MAX_DEVICES = 64;
std::mutex static_mu;
void *static_ptr[MAX_DEVICES];  // device address of `scratch` on each device, or NULL
}  // namespace

extern "C" rd_status rd_sdf_scratch_bytes(int64_t nx, int64_t ny, int64_t nz, size_t *bytes)
{
    if (!bytes) return rd_fail(RD_ERR_ARG, "bytes is NULL");
    if (nx < 1 || ny < 1 || nz < 1) return rd_fail(RD_ERR_SHAPE, "need nx, ny, nz >= 1");
    const size_t N = (size_t)nx * (size_t)ny * (size_t)nz;
    *bytes = align256(4 * N) + align256(4 * N) + align256(4 * N) + align256(8 * N);
    return RD_OK;
}

extern "C" rd_status rd_sdf_from_image_static(const uint8_t *dev_image, int64_t nx, int64_t ny, int64_t nz,
                                              double dx, float *dev_sdf, void *stream)
{
    if (!dev_image || !dev_sdf) return rd_fail(RD_ERR_ARG, "NULL pointer");
    if (nx < 1 || ny < 1 || nz < 1 || nx > 32768 || ny > 32768 || nz > 32768)
        return rd_fail(RD_ERR_SHAPE, "need 1 <= nx, ny, nz <= 32768");
    size_t need = 0;
    rd_sdf_scratch_bytes(nx, ny, nz, &need);
    if (need > RD_SDF_STATIC_BYTES)
        return rd_fail(RD_ERR_SHAPE, "volume needs " + std::to_string(need) + " scratch bytes; the fixed scratch holds " +
                                         std::to_string(RD_SDF_STATIC_BYTES) + " (20 bytes per voxel)");
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return rd_fail(RD_ERR_HIP, std::string("hipGetDevice: ") + hipGetErrorString(e));
    if (dev < 0 || dev >= MAX_DEVICES) return rd_fail(RD_ERR_HIP, "device id out of range");
    void *ptr = nullptr;
    {
        std::lock_guard<std::mutex> lock(static_mu);
        if (!static_ptr[dev]) {  // first call on this device (it is current)
            e = hipGetSymbolAddress(&static_ptr[dev], HIP_SYMBOL(scratch));
            if (e != hipSuccess) {
                static_ptr[dev] = nullptr;
                return rd_fail(RD_ERR_HIP, std::string("hipGetSymbolAddress: ") + hipGetErrorString(e));
            }
        }
        ptr = static_ptr[dev];
    }
    return rd_sdf_from_image(dev_image, nx, ny, nz, dx, dev_sdf, ptr, RD_SDF_STATIC_BYTES, stream);
}

extern "C" rd_status rd_sdf_from_image(const uint8_t *dev_image, int64_t nx, int64_t ny, int64_t nz, double dx,
                                       float *dev_sdf, void *dev_scratch, size_t scratch_bytes, void *stream)
{
    if (!dev_image || !dev_sdf || !dev_scratch) return rd_fail(RD_ERR_ARG, "NULL pointer");
    if (!(dx > 0.0)) return rd_fail(RD_ERR_ARG, "dx must be > 0");
    if (nx < 1 || ny < 1 || nz < 1 || nx > 32768 || ny > 32768 || nz > 32768)
        return rd_fail(RD_ERR_SHAPE, "need 1 <= nx, ny, nz <= 32768");
    size_t need = 0;
    rd_sdf_scratch_bytes(nx, ny, nz, &need);
    if (scratch_bytes < need)
        return rd_fail(RD_ERR_WORKSPACE, "scratch has " + std::to_string(scratch_bytes) + " bytes, needs " +
                                             std::to_string(need));
    const int64_t N = nx * ny * nz;
    // the words after the x and y passes and their summaries (at most one word per voxel)
    const size_t part = align256(4 * (size_t)N);
    char *p = (char *)dev_scratch;
    int *g = (int *)p, *h = (int *)(p + part);
    int *gsum = (int *)(p + 2 * part), *hsum = (int *)(p + 3 * part);
    hipStream_t st = (hipStream_t)stream;
    const double diag = sqrt((double)nx * nx + (double)ny * ny + (double)nz * nz);
    const int64_t nc = (nx + 63) / 64;
    hipLaunchKernelGGL(k_edt_x, edt_grid((ny * nz + 3) / 4), dim3(256), 32 * (size_t)nc, st, dev_image, (int)nx,
                       (int)ny, ny * nz, g, gsum);
    // the summaries of runs, behind those of the z pass's rows (their words are 2 % of these);
    // the y pass has read its own when the z pass's are written
    int *c64 = hsum + align256(4 * (size_t)(ny * nc * nz)) / 4;
    auto runs = [&](const int *sum, int64_t n, int64_t nlines) {  // the form of the line pass
        if (n <= EDT_LONG) return 0;
        hipLaunchKernelGGL(k_edt_runs, edt_grid((nlines * ((n + 255) / 256) + 3) / 4), dim3(256), 0, st, sum, (int)n,
                           nlines, c64);
        return n <= EDT_LONGER ? 1 : 2;
    };
    int form = runs(gsum, ny, nz * nc);
    hipLaunchKernelGGL((form == 0 ? k_edt_y<0> : form == 1 ? k_edt_y<1> : k_edt_y<2>),
                       edt_grid(nz * nc * ((ny + 31) / 32)), dim3(256), 0, st, g, gsum, c64, (int)nx, (int)ny, (int)nz,
                       (int)nc, h, hsum);
    form = runs(hsum, nz, ny * nc);
    hipLaunchKernelGGL((form == 0 ? k_edt_z<0> : form == 1 ? k_edt_z<1> : k_edt_z<2>),
                       edt_grid(ny * nc * ((nz + 31) / 32)), dim3(256), 0, st, h, hsum, c64, (int)nx, (int)ny, (int)nz,
                       (int)nc, dx, diag, dev_sdf);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return rd_fail(RD_ERR_HIP, std::string("EDT launch: ") + hipGetErrorString(e));
    return RD_OK;
}
