// Field preparation (sec. 3.2): Gladstone-Dale n = K rho + 1 (eq. 1) and the refractive-index
// gradient at the grid nodes (central differences inside, second-order one-sided differences on
// the faces), stored per cell as the coefficients of the trilinear interpolant of
// (n - 1, grad n) over the cell's eight corners (layout in pbr_internal.h), or per node.
//
// One block per brick of 8^3 cells; all arithmetic in FP64, rounded once to float32 on output.
#include "pbr_internal.h"

namespace pbr {
namespace {

constexpr int kHalo = kBrick + 3;   // density nodes of a brick: its 9 per axis and one beyond each side
constexpr int kSide = kBrick + 1;   // nodes of a brick per axis
constexpr int kNodes = kSide * kSide * kSide;

// Derivative with respect to the node index along one grid line through rho[q] (m: node index, n: nodes of
// the line): central difference inside, second-order one-sided difference on the first and last node,
// plain difference when the line has only two nodes.
__device__ __forceinline__ double index_derivative(const float *rho, int q, int stride, int m, int n)
{
    if (n == 2) {
        const int q0 = q - m * stride;
        return (double)rho[q0 + stride] - (double)rho[q0];
    }
    if (m == 0)
        return -1.5 * (double)rho[q] + 2.0 * (double)rho[q + stride] - 0.5 * (double)rho[q + 2 * stride];
    if (m == n - 1)
        return 1.5 * (double)rho[q] - 2.0 * (double)rho[q - stride] + 0.5 * (double)rho[q - 2 * stride];
    return 0.5 * ((double)rho[q + stride] - (double)rho[q - stride]);
}

// Between the LDS accesses of a wave's lanes and those of its other lanes to the same places.
__device__ __forceinline__ void wave_exchange()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// One brick: its density nodes through LDS once, the values of its 9^3 nodes computed once each (and not
// by each of the up to eight cells around a node), its steepness (largest |grad n| at its nodes) reduced in
// the block and written without atomics, then the cell records from the node values in LDS.  The 128-byte
// records go out through LDS too, so that a store instruction of a wave writes 1 KB in one piece.
// NODES: the node layout instead (each node written by the brick whose cells start at it).
// Bound by the 128 bytes per cell written; the one-thread-per-cell form computed every node eight times
// (24 derivatives and 8 square roots in FP64 per cell): 192^3 cells 1.17 -> 0.29 ms (3.1 TB/s written),
// 512^3 nodes 6.4 + 1.1 -> 1.25 ms (two kernels before).
template <bool NODES>
__global__ void __launch_bounds__(256)
k_field_prep(const float *__restrict__ rho, float4 *__restrict__ out, unsigned *__restrict__ brick_gmax, int nx, int ny,
             int nz, double kx, double ky, double kz, double K)
{
    __shared__ float sr[kHalo * kHalo * kHalo];
    __shared__ double sv[NODES ? 1 : kNodes][4];
    __shared__ double sg[4];
    __shared__ float4 stage[NODES ? 1 : 4][NODES ? 1 : 64 * kCellFloat4];
    const int i0 = (int)blockIdx.x * kBrick, j0 = (int)blockIdx.y * kBrick, k0 = (int)blockIdx.z * kBrick;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const size_t sy = (size_t)nx, sz = (size_t)nx * (size_t)ny;
    // (no planes beyond the grid: slices a few nodes deep along z)
    for (int t = threadIdx.x; t < kHalo * kHalo * min(kHalo, nz - k0 + 1); t += 256) {
        const int x = t % kHalo, y = (t / kHalo) % kHalo, z = t / (kHalo * kHalo);
        // nodes beyond the grid are not used
        const int i = min(max(i0 + x - 1, 0), nx - 1), j = min(max(j0 + y - 1, 0), ny - 1),
                  k = min(max(k0 + z - 1, 0), nz - 1);
        sr[t] = rho[(size_t)k * sz + (size_t)j * sy + (size_t)i];
    }
    __syncthreads();
    double gm = 0.0;
    for (int t = threadIdx.x; t < kSide * kSide * min(kSide, nz - k0); t += 256) {
        const int x = t % kSide, y = (t / kSide) % kSide, z = t / (kSide * kSide);
        const int i = i0 + x, j = j0 + y, k = k0 + z;
        if (i >= nx || j >= ny) continue;
        const int q = ((z + 1) * kHalo + y + 1) * kHalo + x + 1;
        const double d0 = (double)sr[q], v0 = K * d0, v1 = kx * index_derivative(sr, q, 1, i, nx),
                     v2 = ky * index_derivative(sr, q, kHalo, j, ny),
                     v3 = kz * index_derivative(sr, q, kHalo * kHalo, k, nz);
        gm = fmax(gm, v1 * v1 + v2 * v2 + v3 * v3);
        if (NODES) {
            if ((x < kBrick || i == nx - 1) && (y < kBrick || j == ny - 1) && (z < kBrick || k == nz - 1))
                out[(size_t)k * sz + (size_t)j * sy + (size_t)i] = make_float4((float)v0, (float)v1, (float)v2, (float)v3);
        } else {
            sv[t][0] = d0;  // the density itself (see below)
            sv[t][1] = v1;
            sv[t][2] = v2;
            sv[t][3] = v3;
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) gm = fmax(gm, __shfl_xor(gm, o, 64));
    if (lane == 0) sg[wave] = gm;
    __syncthreads();
    if (threadIdx.x == 0) {
        const float gf = (float)sqrt(fmax(fmax(sg[0], sg[1]), fmax(sg[2], sg[3])));
        brick_gmax[((size_t)blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x] = gf > 0.0f ? __float_as_uint(gf) : 0u;
    }
    if (NODES) return;
    for (int slab = wave; slab < kBrick; slab += 4) {  // 64 cells of one z per wave
        const int x = lane & 7, y = lane >> 3;
        const int k = k0 + slab;
        if (k >= nz - 1) break;
        const int t = (slab * kSide + y) * kSide + x;
        float4 rec[kCellFloat4];
        float *r = (float *)rec;
        {   // n - 1 = K rho: the sums take the products unrounded, one after the other; the gradients' sums take
            // the rounded values.  (The order and the roundings are part of the stored field: saved
            // surrogates carry its checksum.)
            const double *s0 = &sv[t][0], *s1 = &sv[t + kSide * kSide][0];
            const double d000 = s0[0], d100 = s0[4], d010 = s0[4 * kSide], d110 = s0[4 * (kSide + 1)];
            const double d001 = s1[0], d101 = s1[4], d011 = s1[4 * kSide], d111 = s1[4 * (kSide + 1)];
            const double f000 = K * d000, f100 = K * d100, f010 = K * d010, f110 = K * d110;
            auto plus = [&](double sum, double d) { return __builtin_fma(K, d, sum); };
            auto minus = [&](double sum, double d) { return __builtin_fma(-K, d, sum); };
            r[0] = (float)f000;
            r[4] = (float)plus(-f000, d100);
            r[8] = (float)plus(-f000, d010);
            r[12] = (float)plus(-f000, d001);
            r[16] = (float)plus(minus(plus(-f100, d110), d010), d000);
            r[20] = (float)plus(minus(plus(-f100, d101), d001), d000);
            r[24] = (float)plus(minus(plus(-f010, d011), d001), d000);
            r[28] = (float)minus(plus(plus(plus(minus(minus(plus(-f110, d111), d101), d011), d100), d010), d001), d000);
        }
#pragma unroll
        for (int m = 1; m < 4; ++m) {
            const double *s0 = &sv[t][m], *s1 = &sv[t + kSide * kSide][m];
            const double f000 = s0[0], f100 = s0[4], f010 = s0[4 * kSide], f110 = s0[4 * (kSide + 1)];
            const double f001 = s1[0], f101 = s1[4], f011 = s1[4 * kSide], f111 = s1[4 * (kSide + 1)];
            r[m] = (float)f000;
            r[4 + m] = (float)(f100 - f000);
            r[8 + m] = (float)(f010 - f000);
            r[12 + m] = (float)(f001 - f000);
            r[16 + m] = (float)(f110 - f100 - f010 + f000);
            r[20 + m] = (float)(f101 - f100 - f001 + f000);
            r[24 + m] = (float)(f011 - f010 - f001 + f000);
            r[28 + m] = (float)(f111 - f110 - f101 - f011 + f100 + f010 + f001 - f000);
        }
        // float4 e of cell `lane` at slot e ^ (lane & 7) of the cell: writes and reads spread over the banks
#pragma unroll
        for (int e = 0; e < kCellFloat4; ++e) stage[wave][lane * kCellFloat4 + (e ^ (lane & 7))] = rec[e];
        wave_exchange();
        const int cell = lane >> 3, e = lane & 7;  // this lane's cell of a row and part of its record
        if (i0 + cell < nx - 1) {
#pragma unroll
            for (int row = 0; row < kBrick; ++row) {
                if (j0 + row >= ny - 1) break;
                const float4 v = stage[wave][(row * 8 + cell) * kCellFloat4 + (e ^ cell)];
                out[((size_t)k * (size_t)(ny - 1) * (size_t)(nx - 1) + (size_t)(j0 + row) * (size_t)(nx - 1) + (size_t)(i0 + cell)) *
                        kCellFloat4 + e] = v;
            }
        }
        wave_exchange();
    }
}

// One axis of the distance map at brick q, the i-th of `len` along the axis: the least over r of
// max(r, distance so far at r bricks along the axis on either side).  Taken along x, then y, then z from
// 0 / kSkipMax this gives the largest-axis distance to the nearest marked brick.
template <typename At>
__device__ __forceinline__ int axis_distance(At at, int64_t q, int64_t stride, int i, int len)
{
    int best = at(q);
    for (int r = 1; r < best; ++r) {
        if (i - r < 0 && i + r >= len) break;
        if (i - r >= 0) best = min(best, max(r, at(q - r * stride)));
        if (i + r < len) best = min(best, max(r, at(q + r * stride)));
    }
    return best;
}

// The whole map of a grid of at most kSkipSmall bricks by one block, in LDS: one launch in place of the five
// below, which are most of what a small field waits for (pbr_set_density_field with 33^3 nodes 78 -> 39 us, 65^3
// 76 -> 45; 131 x 100 x 77, 2210 bricks, 98 -> 78).  With 4096 bricks it takes 64 us against 81 where the gradient is
// everywhere and 95 against 89 where the gas is uniform, with 5832 bricks 73 against 88 and 119 against 102.
constexpr int kSkipSmall = 4096;
__global__ void __launch_bounds__(1024) k_skip_small(unsigned *__restrict__ gmax, int nbx, int nby, int nbz)
{
    __shared__ unsigned char a[kSkipSmall], b[kSkipSmall];
    const int columns = nbx * nby, n = columns * nbz;
    for (int q = threadIdx.x; q < n; q += blockDim.x) a[q] = gmax[q] ? 0 : kSkipMax;
    __syncthreads();
    auto pass = [&](const unsigned char *from, unsigned char *to, int stride, int len) {
        for (int q = threadIdx.x; q < n; q += blockDim.x)
            to[q] = (unsigned char)axis_distance([&](int64_t k) { return (int)from[k]; }, q, stride, (q / stride) % len, len);
        __syncthreads();
    };
    pass(a, b, 1, nbx);
    pass(b, a, nbx, nby);
    pass(a, b, columns, nbz);
    for (int q = threadIdx.x; q < n; q += blockDim.x) {  // a: none of the brick and its neighbours in x and y has a gradient
        const int x = q % nbx, y = (q / nbx) % nby;
        bool open = true;
        for (int dy = -1; dy <= 1; ++dy)
            for (int dx = -1; dx <= 1; ++dx)
                if ((unsigned)(x + dx) < (unsigned)nbx && (unsigned)(y + dy) < (unsigned)nby) open = open && b[q + dy * nbx + dx];
        a[q] = open;
    }
    __syncthreads();
    for (int c = threadIdx.x; c < columns; c += blockDim.x) {
        int run = 0;
        for (int q = n - columns + c; q >= 0; q -= columns) {
            run = a[q] ? run + 1 : 0;
            if (b[q]) gmax[q] = kSkipBit | ((unsigned)run << 8) | b[q];
        }
    }
}

// One axis of the distance map of a larger grid.  FIRST reads the gradients themselves; WORDS: from the
// bytes of tmp into the words of gmax, otherwise from the words into the bytes.
template <bool FIRST, bool WORDS>
__global__ void __launch_bounds__(256) k_skip_pass(unsigned *__restrict__ gmax, unsigned char *__restrict__ tmp, int64_t n,
                                                   int64_t stride, int len)
{
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= n) return;
    const int i = (int)((q / stride) % len);
    auto at = [&](int64_t k) {
        if (WORDS) return (int)tmp[k];
        const unsigned v = gmax[k];
        return FIRST ? (v ? 0 : kSkipMax) : skip_distance(v);
    };
    const int best = axis_distance(at, q, stride, i, len);
    if (!WORDS) tmp[q] = (unsigned char)best;
    else if (best) gmax[q] = kSkipBit | (unsigned)best;
}

// The distances of the last pass back into gmax, marked kSkipSide where a neighbour in x or y has a
// gradient, and tmp zero again.  (Neighbours' words change under the reader; the tested bit does not.)
__global__ void __launch_bounds__(256) k_skip_finish(unsigned *__restrict__ gmax, unsigned char *__restrict__ tmp, int nbx,
                                                     int nby, int64_t n)
{
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= n) return;
    const unsigned d = tmp[q];
    tmp[q] = 0;
    if (!d) return;
    const int x = (int)(q % nbx), y = (int)((q / nbx) % nby);
    bool side = false;
    for (int dy = -1; dy <= 1; ++dy)
        for (int dx = -1; dx <= 1; ++dx) {
            if ((unsigned)(x + dx) >= (unsigned)nbx || (unsigned)(y + dy) >= (unsigned)nby) continue;
            const unsigned v = __hip_atomic_load(gmax + q + (int64_t)dy * nbx + dx, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            side = side || !(v & kSkipBit);
        }
    __hip_atomic_store(gmax + q, kSkipBit | (side ? kSkipSide : 0u) | d, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Runs towards +z, one thread per column of bricks.
__global__ void __launch_bounds__(64) k_skip_runs(unsigned *__restrict__ gmax, int64_t columns, int nbz)
{
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= columns) return;
    int run = 0;
#pragma unroll 8
    for (int z = nbz - 1; z >= 0; --z) {
        const unsigned v = gmax[(int64_t)z * columns + q];
        run = (v & (kSkipBit | kSkipSide)) == kSkipBit ? run + 1 : 0;
        if (v & kSkipBit) gmax[(int64_t)z * columns + q] = kSkipBit | ((unsigned)run << 8) | (v & 0xFFu);
    }
}

// Fingerprint of a field: sum over its 32-bit words w_k of SplitMix64's finaliser applied to
// (k << 32 | w_k), wrapping mod 2^64 (integer atomics: independent of the order of the blocks).
__global__ void __launch_bounds__(256) k_checksum(const unsigned *__restrict__ w, int64_t n,
                                                  unsigned long long *__restrict__ out)
{
    unsigned long long acc = 0ull;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < n; k += stride) {
        unsigned long long z = ((unsigned long long)k << 32) ^ (unsigned long long)w[k];
        z += 0x9E3779B97F4A7C15ull;
        z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
        z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
        acc += z ^ (z >> 31);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o, 64);
    if ((threadIdx.x & 63u) == 0)
        __hip_atomic_fetch_add(out, acc, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Integer that orders like the float x (any sign), above 0 for every number.
__device__ __forceinline__ unsigned ordered_bits(float x)
{
    const unsigned u = __float_as_uint(x);
    return (u >> 31) ? ~u : u | 0x80000000u;
}

// out[0]: waves that saw a value that is not finite; out[1], out[2]: largest ordered_bits of the
// values and of the negated values (the range of the density).
// Few, large blocks: the blocks' three atomics on one line are most of the time of a small grid (192^3: 56 us
// with 2048 blocks, 15 with 256 of 1024 threads).
__global__ void __launch_bounds__(1024) k_check_density(const float *__restrict__ rho, int64_t n,
                                                       unsigned long long *__restrict__ out)
{
    bool ok = true;
    float hi = -3.402823466e38f, lo = 3.402823466e38f;
    auto take = [&](float v) {
        ok = ok && isfinite(v);
        hi = fmaxf(hi, v);
        lo = fminf(lo, v);
    };
    const int64_t stride = (int64_t)gridDim.x * blockDim.x, at = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t n4 = ((uintptr_t)rho & 15u) == 0 ? n / 4 : 0;  // four at a time where the alignment allows
    for (int64_t k = at; k < n4; k += stride) {
        const float4 v = ((const float4 *)rho)[k];
        take(v.x);
        take(v.y);
        take(v.z);
        take(v.w);
    }
    for (int64_t k = 4 * n4 + at; k < n; k += stride) take(rho[k]);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        hi = fmaxf(hi, __shfl_xor(hi, o, 64));
        lo = fminf(lo, __shfl_xor(lo, o, 64));
    }
    const bool bad = __ballot(!ok) != 0ull;
    __shared__ float sh[2][16];
    __shared__ int sbad[16];
    if ((threadIdx.x & 63u) == 0) {
        sh[0][threadIdx.x >> 6] = hi;
        sh[1][threadIdx.x >> 6] = lo;
        sbad[threadIdx.x >> 6] = bad;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        int any = 0;
        for (int w = 0; w < (int)blockDim.x / 64; ++w) {
            hi = fmaxf(hi, sh[0][w]);
            lo = fminf(lo, sh[1][w]);
            any |= sbad[w];
        }
        if (any)
            __hip_atomic_fetch_add(out, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        atomicMax(out + 1, (unsigned long long)ordered_bits(hi));
        atomicMax(out + 2, (unsigned long long)ordered_bits(-lo));
    }
}

__global__ void __launch_bounds__(256) k_clear_u64(unsigned long long *p, int64_t n)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < n; q += stride) p[q] = 0ull;
}

}  // namespace

int launch_field_prep(const float *rho, float4 *cells, unsigned *brick_gmax, int nx, int ny, int nz,
                      const double spacing[3], double K, hipStream_t stream, bool nodes)
{
    const FieldLayout L = field_layout(nx, ny, nz, nodes);
    // one dimension per axis: a thin grid can have 2^24 bricks and more, whose threads no single one counts
    const dim3 grid((unsigned)L.nbx, (unsigned)L.nby, (unsigned)L.nbz), block(256);
    if (nodes)
        hipLaunchKernelGGL(k_field_prep<true>, grid, block, 0, stream, rho, cells, brick_gmax, nx, ny, nz, K / spacing[0],
                           K / spacing[1], K / spacing[2], K);
    else
        hipLaunchKernelGGL(k_field_prep<false>, grid, block, 0, stream, rho, cells, brick_gmax, nx, ny, nz, K / spacing[0],
                           K / spacing[1], K / spacing[2], K);
    return (int)hipGetLastError();
}

int launch_skip_map(unsigned *gmax, unsigned char *tmp, int nbx, int nby, int nbz, hipStream_t stream)
{
    const int64_t n = (int64_t)nbx * nby * nbz;
    if (n <= kSkipSmall) {
        hipLaunchKernelGGL(k_skip_small, dim3(1), dim3(1024), 0, stream, gmax, nbx, nby, nbz);
        return (int)hipGetLastError();
    }
    const dim3 grid((unsigned)((n + 255) / 256)), block(256);
    hipLaunchKernelGGL((k_skip_pass<true, false>), grid, block, 0, stream, gmax, tmp, n, (int64_t)1, nbx);
    hipLaunchKernelGGL((k_skip_pass<false, true>), grid, block, 0, stream, gmax, tmp, n, (int64_t)nbx, nby);
    hipLaunchKernelGGL((k_skip_pass<false, false>), grid, block, 0, stream, gmax, tmp, n, (int64_t)nbx * nby, nbz);
    hipLaunchKernelGGL(k_skip_finish, grid, block, 0, stream, gmax, tmp, nbx, nby, n);
    const int64_t columns = (int64_t)nbx * nby;
    hipLaunchKernelGGL(k_skip_runs, dim3((unsigned)((columns + 63) / 64)), dim3(64), 0, stream, gmax, columns, nbz);
    return (int)hipGetLastError();
}

int launch_field_checksum(const void *field, size_t bytes, unsigned long long *out, hipStream_t stream)
{
    const int64_t n = (int64_t)(bytes / 4);
    int e = launch_clear_u64(out, 1, stream);
    if (e || n == 0) return e;
    int64_t blocks = (n + 255) / 256;
    if (blocks > 8192) blocks = 8192;
    hipLaunchKernelGGL(k_checksum, dim3((unsigned)blocks), dim3(256), 0, stream, (const unsigned *)field, n, out);
    return (int)hipGetLastError();
}

int launch_check_density(const float *rho, int64_t n, unsigned long long *out, hipStream_t stream)
{
    int e = launch_clear_u64(out, 3, stream);
    if (e || n <= 0) return e;
    int64_t blocks = (n + 4095) / 4096;
    if (blocks > 256) blocks = 256;
    hipLaunchKernelGGL(k_check_density, dim3((unsigned)blocks), dim3(1024), 0, stream, rho, n, out);
    return (int)hipGetLastError();
}

int launch_clear_u64(unsigned long long *p, int64_t n, hipStream_t stream)
{
    if (n <= 0) return 0;
    int64_t blocks = (n + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    hipLaunchKernelGGL(k_clear_u64, dim3((unsigned)blocks), dim3(256), 0, stream, p, n);
    return (int)hipGetLastError();
}

}  // namespace pbr
