// Baking side of the method (Section 5.3, 5.4): which macroblocks of a
// densely evaluated field are stored, and their 8-bit values.
//
//  k_bake_block_max   largest density of every macroblock (HBM-bound
//                     streaming pass over the N^3 field); also resets the
//                     per-block visibility words.
//  k_bake_visibility  every training ray marched over the dense field on
//                     the render's sample lattice (step 1/N), one lane per
//                     ray and one wavefront per 8x8 pixel tile; the density
//                     prefix sum before the first sample of each macroblock
//                     the ray enters is folded into that block's minimum
//                     (64-bit atomic min on the bits of a non-negative
//                     double, which orders like the value).  The ray stops
//                     once the prefix sum passes the visibility threshold:
//                     later samples cannot make a block visible.
//  k_bake_cells,      the same two for macroblocks of 8^3 and more: the first
//  k_bake_visibility_cells
//                     pass also notes which 8^3 cells and whole macroblocks
//                     hold one value, and the march takes those in one step.
//  k_bake_choose      leaves fields with many mixed cells to k_bake_visibility.
//  k_bake_compact     the two culls and the atlas numbering in scan order
//                     (one workgroup: a ballot prefix per wavefront, then
//                     across wavefronts).
//  k_bake_quantize    8-bit quantisation of the kept blocks into the
//                     canonical atlas, four voxels per lane along x.
#include <type_traits>

#include "snerg_launch.h"

namespace snerg {

namespace {

constexpr uint64_t kInfBits = 0x7ff0000000000000ull;  // +inf as double bits

struct f32x4 {
    float v[4];
};
__device__ __forceinline__ f32x4 ld4(const float* p) {
    const float4 q = *reinterpret_cast<const float4*>(p);
    return {{q.x, q.y, q.z, q.w}};
}

__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) v = fmaxf(v, __shfl_xor(v, m));
    return v;
}

}  // namespace

// One workgroup per macroblock (grid.x = G^3).  V = voxels per load (4 when
// B >= 4, else 1).
template <int V>
__global__ __launch_bounds__(256) void k_bake_block_max(const float* __restrict__ sigma, int32_t N, int32_t logB,
                                                        int32_t G, float* __restrict__ bmax,
                                                        uint64_t* __restrict__ depth_bits) {
    __shared__ float part[4];
    const int64_t lin = blockIdx.x;
    const int32_t bx = int32_t(lin % G), by = int32_t((lin / G) % G), bz = int32_t(lin / (int64_t(G) * G));
    const int32_t B = 1 << logB;
    const int32_t rowq = B / V;  // loads per row
    const int32_t n_loads = B * B * rowq;
    float m = -INFINITY;
    for (int32_t e = threadIdx.x; e < n_loads; e += blockDim.x) {
        const int32_t q = e % rowq, r = e / rowq;
        const int32_t ly = r & (B - 1), lz = r >> logB;
        const int64_t base = (int64_t(bz * B + lz) * N + (by * B + ly)) * N + bx * B + q * V;
        if (V == 4) {
            const f32x4 x = ld4(sigma + base);
            m = fmaxf(m, fmaxf(fmaxf(x.v[0], x.v[1]), fmaxf(x.v[2], x.v[3])));
        } else {
            m = fmaxf(m, sigma[base]);
        }
    }
    m = wave_max(m);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
        float r = part[0];
        for (int w = 1; w < int(blockDim.x >> 6); ++w) r = fmaxf(r, part[w]);
        bmax[lin] = r;
        depth_bits[lin] = kInfBits;
    }
}

constexpr int kVisThreads = 256;  // of a visibility workgroup

struct BakeVisArgs {
    const float* sigma;
    const DevCamera* cams;
    int32_t n_cams;
    int32_t N, logB, G;
    int64_t total_tiles;
    int32_t tile_w, tile_h;
    double sum_thr;  // stop once the density prefix sum exceeds this
    uint64_t* depth_bits;
    const uint2* cells;     // k_bake_visibility_cells: the cell table and the field's statistics
    const uint32_t* stats;
};

// Per-workgroup cache of bounds on the blocks' minima: 2^LOG slots indexed by
// the low bits of the block index, each one 32-bit word (read and written
// whole, so no reader sees half an update): the block index's bits from 8 on,
// 10 of them, then a 22-bit code whose value is an upper bound of a prefix
// sum that some lane of the workgroup has folded, or is about to fold, into
// that block's minimum (the sum rounded up to float, then its bits rounded up
// to a multiple of 2^10).  A block entry whose prefix sum is at least that
// bound needs no global access.  A racing overwrite only costs a later global
// check.
// (Accessed by relaxed atomics: a volatile pointer argument would leave the LDS's
// address space unknown and every access a flat one.)
template <int LOG>
__device__ __forceinline__ void vis_cache_clear(uint32_t* vcache) {
#pragma unroll
    for (int i = threadIdx.x; i < (1 << LOG); i += kVisThreads)
        vcache[i] = (uint32_t(i >> 8) << 22) | (0x7f800000u >> 10);  // bound +inf: never skips
}
__device__ __forceinline__ uint32_t vis_cached(const uint32_t* slot) {
    return __hip_atomic_load(slot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ void vis_cache(uint32_t* slot, uint32_t key) {
    __hip_atomic_store(slot, key, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

__device__ __forceinline__ uint32_t vis_code(double sum) {
    float f = float(sum);
    if (double(f) < sum) f = __uint_as_float(__float_as_uint(f) + 1u);
    return (__float_as_uint(f) + 0x3ffu) >> 10;
}

// Folds a prefix sum into the minimum of the macroblock a ray enters with it,
// unless the cache of 2^LOG slots says that the minimum is no larger already.
// The lanes that enter a block together first agree in the cache on the
// smallest code; a lane with a larger one leaves the fold to that lane (its
// own sum is larger, and so is the bound it would have written).
// SCOPE: of the read of the global minimum.  It only ever falls, so an old value
// from a cache is a bound as good as any, and a read that waits for the other
// XCDs costs the ray several times a cached one; but the lanes that it does not
// stop go on to an atomic each, and with the 256 slots of the march by samples
// those are many: 100 views of 800x800 into 160^3 that varies in every voxel
// take 7.7 ms with cached reads and 6.65 without.
template <int LOG, int SCOPE>
__device__ __forceinline__ void vis_enter(uint32_t* vcache, uint64_t* depth_bits, uint32_t lin, double sum) {
    uint32_t* slot = vcache + (lin & ((1u << LOG) - 1u));
    const uint32_t tag = lin >> 8, key = vis_cached(slot);
    if ((key >> 22) == tag && double(__uint_as_float((key & 0x3fffffu) << 10)) <= sum) return;
    const uint32_t mine = (tag << 22) | vis_code(sum);
    if ((key >> 22) == tag) __hip_atomic_fetch_min(slot, mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    else vis_cache(slot, mine);
    const uint32_t now = vis_cached(slot);
    if ((now >> 22) == tag && now < mine) return;
    const uint64_t bits = uint64_t(__double_as_longlong(sum));
    uint64_t* w = depth_bits + lin;
    const uint64_t g = __hip_atomic_load(w, __ATOMIC_RELAXED, SCOPE);
    if (bits < g) atomicMin(reinterpret_cast<unsigned long long*>(w), (unsigned long long)bits);
    else vis_cache(slot, (tag << 22) | vis_code(__longlong_as_double((long long)g)));
}

// The ray of lane `lane` in tile t and its samples inside the grid: position
// of the first (Q16), step, count.  False: the pixel overhangs the image or
// the ray misses the grid.
__device__ __forceinline__ bool vis_ray(const BakeVisArgs& a, int64_t t, int lane, int32_t P[3], int32_t s[3],
                                        int32_t& n) {
    const int ci = find_camera_by_tile(a.cams, a.n_cams, t);
    const DevCamera& c = a.cams[ci];
    const int64_t tl = t - c.tile_offset;
    const int px = int(tl % c.tiles_x) * a.tile_w + lane % a.tile_w;
    const int py = int(tl / c.tiles_x) * a.tile_h + lane / a.tile_w;
    if (px >= c.W || py >= c.H) return false;
    int64_t o[3];
    float d[3];
    ray_setup(c, a.N, px, py, o, s, d);
    int64_t klo, khi;
    if (!entry_range(o, s, int64_t(a.N) << 16, klo, khi)) return false;
#pragma unroll
    for (int q = 0; q < 3; ++q) P[q] = int32_t(o[q] + klo * int64_t(s[q]));  // inside [0, N 2^16)
    n = int32_t(khi - klo + 1);
    return true;
}

// Samples loaded ahead of the sequential prefix sum.
constexpr int kVisAhead = 4;

// Voxel index arithmetic of the march: kIdx64 for any N, kIdx32 when
// N^3 < 2^32 (24-bit multiplies), kIdxPow2 when N is a power of two up to
// 1024 (bit fields: the voxel index is vx | vy << lg | vz << 2 lg, and the
// macroblock is that index with the low logB bits of each field masked off,
// one AND per sample).
enum { kIdx64 = 0, kIdx32 = 1, kIdxPow2 = 2 };

template <int IDX>
__global__ __launch_bounds__(256) void k_bake_visibility(BakeVisArgs a) {
    if (a.cells && a.stats[2] == 0) return;  // k_bake_visibility_cells takes the field
    __shared__ uint32_t vcache[256];
    vis_cache_clear<8>(vcache);
    __syncthreads();
    const int lane = threadIdx.x & 63;
    const int64_t t = int64_t(blockIdx.x) * (blockDim.x >> 6) + (threadIdx.x >> 6);
    if (t >= a.total_tiles) return;  // wave-uniform
    int32_t P[3], s[3], n;
    if (!vis_ray(a, t, lane, P, s, n)) return;
    const uint32_t N = uint32_t(a.N), G = uint32_t(a.G);
    const int bs = 16 + a.logB;
    int lg = 0;
    while ((1 << lg) < a.N) ++lg;
    const uint32_t fmask = (G - 1) << a.logB;  // block bits of one coordinate field
    const uint32_t bmask = fmask | (fmask << lg) | (fmask << (2 * lg));
    const double thr = a.sum_thr;
    double sum = 0.0;
    uint32_t prev = 0xffffffffu;
    // One chunk of kVisAhead samples: all loads first, then the sequential
    // prefix sum.  With FULL every sample of the chunk is inside the grid;
    // otherwise the ones past the last inside sample are clamped onto it, so
    // that every load stays in bounds.
    auto chunk = [&](auto full_tag, int32_t last) {
        constexpr bool FULL = decltype(full_tag)::value;
        float sv[kVisAhead];
        uint32_t bk[kVisAhead];
        uint32_t Q[3] = {uint32_t(P[0]), uint32_t(P[1]), uint32_t(P[2])};
#pragma unroll
        for (int u = 0; u < kVisAhead; ++u) {
            if (u > 0) {
                const uint32_t m = (FULL || u <= last) ? 0xffffffffu : 0u;
#pragma unroll
                for (int q = 0; q < 3; ++q) Q[q] += uint32_t(s[q]) & m;
            }
            if (IDX == kIdxPow2) {
                const uint32_t v = (Q[0] >> 16) | ((Q[1] >> 16) << lg) | ((Q[2] >> 16) << (2 * lg));
                sv[u] = a.sigma[v];
                bk[u] = v & bmask;
            } else {
                if (IDX == kIdx32) {  // every factor and partial sum below 2^24
                    const uint32_t v = __umul24(__umul24(Q[2] >> 16, N) + (Q[1] >> 16), N) + (Q[0] >> 16);
                    sv[u] = a.sigma[v];
                } else {
                    const uint64_t v = (uint64_t(Q[2] >> 16) * N + (Q[1] >> 16)) * N + (Q[0] >> 16);
                    sv[u] = a.sigma[v];
                }
                // macroblock coordinates packed 8 bits each (G <= 64)
                bk[u] = (Q[0] >> bs) | ((Q[1] >> bs) << 8) | ((Q[2] >> bs) << 16);
            }
        }
#pragma unroll
        for (int u = 0; u < kVisAhead; ++u) {
            if (FULL || u <= last) {
                // first sample of a macroblock: the ray's smallest prefix sum in
                // it; past the threshold no later block is visible from this ray
                if (bk[u] != prev) {
                    prev = bk[u];
                    if (sum <= thr) {
                        uint32_t bx, by, bz;
                        if (IDX == kIdxPow2) {
                            bx = (bk[u] >> a.logB) & (G - 1);
                            by = (bk[u] >> (lg + a.logB)) & (G - 1);
                            bz = bk[u] >> (2 * lg + a.logB);
                        } else {
                            bx = bk[u] & 0xff;
                            by = (bk[u] >> 8) & 0xff;
                            bz = bk[u] >> 16;
                        }
                        const uint32_t lin = __umul24(__umul24(bz, G) + by, G) + bx;
                        vis_enter<8, __HIP_MEMORY_SCOPE_AGENT>(vcache, a.depth_bits, lin, sum);
                    }
                }
                sum += double(sv[u]);
            }
        }
    };
    for (int32_t j = 0;; j += kVisAhead) {
        const int32_t last = n - 1 - j;
        if (__all(last >= kVisAhead - 1))
            chunk(std::true_type{}, last);
        else
            chunk(std::false_type{}, last);
        if (sum > thr || last < kVisAhead) break;
#pragma unroll
        for (int q = 0; q < 3; ++q) P[q] += kVisAhead * s[q];
    }
}

// Cells of one value.  Most of a baked field is empty or constant, yet the
// march above pays 21 instructions and a dependent add for each of its
// samples.  k_bake_cells reads the field once, as k_bake_block_max does, and
// notes for every 8^3 cell whether all its voxels hold the same bits: the
// entry is {value, edge shift}, the shift that of the whole macroblock where
// that holds one value, {kMixed, cell shift} where the cell does not.  It
// also collects the field's largest bits and smallest non-zero ones (stats,
// zero on entry: largest bits; complement of the smallest).
constexpr uint32_t kMixed = 0x7fc00000u;  // a NaN: no field value (one that is NaN reads as mixed)
constexpr int kCellLog = 3;
constexpr int kCell = 1 << kCellLog;

// One workgroup per macroblock, B >= 8.  A wavefront takes a slab of cells at
// a time, all cells along x of one (y, z): every step its lanes read whole
// rows of the block, 16 bytes each, `rows` of the slab's 64 rows at once.
__global__ __launch_bounds__(256) void k_bake_cells(const float* __restrict__ sigma, int32_t N, int32_t logB, int32_t G,
                                                    float* __restrict__ bmax, uint64_t* __restrict__ depth_bits,
                                                    uint2* __restrict__ cells, uint32_t* __restrict__ stats) {
    __shared__ uint32_t lo[512], hi[512];  // per cell: smallest and largest bits (B = 64: 8^3 cells)
    __shared__ float part[4];
    __shared__ uint32_t part_lo[4], part_hi[4], part_nz[4];
    const int64_t lin = blockIdx.x;
    const int32_t bx = int32_t(lin % G), by = int32_t((lin / G) % G), bz = int32_t(lin / (int64_t(G) * G));
    const int32_t B = 1 << logB, cb = B >> kCellLog, lrow = logB - 2, rowq = 1 << lrow;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, n_waves = blockDim.x >> 6;
    const int q = lane & (rowq - 1);
    float m = -INFINITY;
    uint32_t all_lo = 0xffffffffu, all_hi = 0, nz = 0xffffffffu;
    for (int slab = wave; slab < cb * cb; slab += n_waves) {
        const int cy = slab % cb, cz = slab / cb;
        uint32_t l = 0xffffffffu, h = 0;
#pragma unroll 8
        for (int st = 0; st < rowq; ++st) {
            const int row = (st << (6 - lrow)) + (lane >> lrow);
            const int ly = cy * kCell + (row & 7), lz = cz * kCell + (row >> 3);
            const int64_t at = (int64_t(bz * B + lz) * N + (by * B + ly)) * N + bx * B + 4 * q;
            float v[4];
            __builtin_memcpy(v, sigma + at, 16);  // one 16-byte load at any float alignment
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                m = fmaxf(m, v[i]);
                const uint32_t bits = v[i] == 0.0f ? 0u : __float_as_uint(v[i]);
                l = min(l, bits);
                h = max(h, bits);
                nz = min(nz, bits != 0 ? bits : 0xffffffffu);
            }
        }
        // lanes of one cell: all rows, and the two loads of a row that lie in it
        for (int x = 1; x < 64; x = x == 1 ? (rowq > 2 ? rowq : 2) : 2 * x) {
            l = min(l, uint32_t(__shfl_xor(int(l), x)));
            h = max(h, uint32_t(__shfl_xor(int(h), x)));
        }
        if (lane < rowq && (lane & 1) == 0) {
            lo[slab * cb + (q >> 1)] = l;
            hi[slab * cb + (q >> 1)] = h;
        }
        all_lo = min(all_lo, l);
        all_hi = max(all_hi, h);
    }
    m = wave_max(m);
#pragma unroll
    for (int x = 32; x >= 1; x >>= 1) {
        all_lo = min(all_lo, uint32_t(__shfl_xor(int(all_lo), x)));
        all_hi = max(all_hi, uint32_t(__shfl_xor(int(all_hi), x)));
        nz = min(nz, uint32_t(__shfl_xor(int(nz), x)));
    }
    if (lane == 0) {
        part[wave] = m;
        part_lo[wave] = all_lo;
        part_hi[wave] = all_hi;
        part_nz[wave] = nz;
    }
    __syncthreads();
    for (int w = 0; w < n_waves; ++w) {
        m = fmaxf(m, part[w]);
        all_lo = min(all_lo, part_lo[w]);
        all_hi = max(all_hi, part_hi[w]);
        nz = min(nz, part_nz[w]);
    }
    if (threadIdx.x == 0) {
        bmax[lin] = m;
        depth_bits[lin] = kInfBits;
        // reads first, from the caches, then behind them: after the first blocks
        // hardly any still has to write
        auto raise = [](uint32_t* p, uint32_t v) {
            if (__hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT) < v &&
                __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < v)
                atomicMax(p, v);
        };
        raise(stats, all_hi);
        raise(stats + 1, ~nz);
    }
    const bool whole = all_lo == all_hi;
    const int32_t M = N >> kCellLog;
    for (int c = threadIdx.x; c < cb * cb * cb; c += blockDim.x) {
        const int cx = c % cb, cy = c / cb % cb, cz = c / (cb * cb);
        uint2 e = make_uint2(kMixed, uint32_t(16 + kCellLog));
        if (lo[c] == hi[c]) e = make_uint2(lo[c], uint32_t(16 + (whole ? logB : kCellLog)));
        cells[(int64_t(bz * cb + cz) * M + (by * cb + cy)) * M + bx * cb + cx] = e;
    }
}

// Steps a ray at Q16 position P may take inside the aligned cube of edge
// 2^sh, at least 1.  up: all ones where s > 0, else 0; inv: just under 1/|s|
// (1e9 for s = 0).  The distance to the face in units of 2^-16, D =
// ((P ^ up) mod 2^sh) + 1, is left behind after ceil(D / |s|) steps; with inv
// low by 2^-22, more than the two roundings can add, the estimate is never
// above that.  Now and then it is one below, and the ray takes another step
// in the same cube.
__device__ __forceinline__ int32_t steps_in_cube(const int32_t P[3], const int32_t up[3], const float inv[3],
                                                 uint32_t sh) {
    const int32_t low = int32_t((1u << sh) - 1u);
    float f[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) f[a] = fmaf(float((P[a] ^ up[a]) & low), inv[a], inv[a]);
    return int32_t(__builtin_ceilf(fminf(fminf(f[0], f[1]), f[2])));
}

// The march of k_bake_visibility over the cell table: a step of a ray is a
// whole cell (or macroblock) of one value, whose samples add n times that
// value to the prefix sum, or the next eight samples of its macroblock.  The
// sums keep every bit of the sample-by-sample ones: a run of zeros changes
// nothing, and n c may stand for n additions of c where no addition rounds.
// That holds for all of the field when, with 2^e the last place of its smallest
// non-zero value (all values are multiples of it), no sum of interest reaches
// 2^(53+e); sums stop mattering past the threshold, so four times that plus twice
// the largest value bounds them.  Where the field does not satisfy this, only
// cells of zeros are skipped.
// Bound by instruction issue for many rays (VALUs 79% busy, five wavefronts per
// SIMD), by the chain of dependent loads for few (the next cell's entry is read
// before the current step's samples): 100 views of 800x800 into a 512^3 field take
// 5.6 ms, 30.2 sample by sample, 24 views of 200x150 into 160^3 0.2 and 0.33.  Lanes that sit through a mixed cell of up to 28
// samples together, as an earlier form had it, made fields with mixed cells twice
// as slow as the march by samples.  Every first look at a macroblock by a workgroup
// costs a global access (they took 40% of the time with 256 slots and one tile per
// wavefront): the cache has a slot for every macroblock up to 16^3, and large
// launches run resident workgroups over many tiles.
constexpr int kCellsCacheLog = 12;
constexpr int kCellAhead = 8;  // samples of a mixed cell's step; 12 and 16 are slower by up to 6 and 20%

// Which of the two marches takes the field: stats[2] is set, and it is the one by
// samples, where more than kMixedLine of 1024 cells, spread over the field, are
// mixed.  Time by samples over time by cells, 100 views of 800x800 into 512^3 in
// blocks of 32, cells mixed at random / in an outer layer: none 5.3, 30% 1.3 / 2.6,
// 50% 0.95 / 1.6, all 0.74; into 160^3 in blocks of 16 1.95, 1.1 / 1.1, 0.9 / 0.87,
// 0.7; 20 views of 300x300 into 512^3 in blocks of 8 2.4, 1.5 / 1.9, 1.05 / 1.5, 0.67.
constexpr int kMixedLine = 460;

__global__ __launch_bounds__(1024) void k_bake_choose(const uint2* __restrict__ cells, uint32_t M,
                                                      uint32_t* __restrict__ stats) {
    const uint32_t at = threadIdx.x << 22 | (threadIdx.x * 2654435761u) >> 10;  // a place in the thread's 1024th
    const uint64_t n = uint64_t(M * M) * M;
    const int mixed = __syncthreads_count(cells[(at * n) >> 32].x == kMixed);
    if (threadIdx.x == 0) stats[2] = mixed > kMixedLine ? 1 : 0;
}

template <int IDX>
__global__ __launch_bounds__(256) void k_bake_visibility_cells(BakeVisArgs a) {
    if (a.stats[2] != 0) return;  // k_bake_visibility takes the field
    __shared__ uint32_t vcache[1 << kCellsCacheLog];
    vis_cache_clear<kCellsCacheLog>(vcache);
    __syncthreads();
    const int lane = threadIdx.x & 63;
    const double thr = a.sum_thr;
    const uint32_t top = a.stats[0], least = ~a.stats[1];
    bool exact = top < 0x7f800000u;  // finite and none negative
    if (exact && top != 0) {
        const int e = int(max(least >> 23, 1u)) - 127 - 23;
        exact = 4.0 * thr + 2.0 * double(__uint_as_float(top)) < __builtin_ldexp(1.0, 53 + e);
    }
    const uint32_t N = uint32_t(a.N), G = uint32_t(a.G), M = N >> kCellLog;
    const int bs = 16 + a.logB;
    int lg = 0;
    while ((1 << lg) < a.N) ++lg;
    const int64_t stride = int64_t(gridDim.x) * (blockDim.x >> 6);
    for (int64_t t = int64_t(blockIdx.x) * (blockDim.x >> 6) + (threadIdx.x >> 6); t < a.total_tiles; t += stride) {
        int32_t P[3], s[3], left;
        if (!vis_ray(a, t, lane, P, s, left)) continue;
        int32_t up[3];
        float inv[3];
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            up[q] = s[q] > 0 ? -1 : 0;
            inv[q] = s[q] != 0 ? (1.0f / fabsf(float(s[q]))) * (1.0f - 0x1p-22f) : 1e9f;
        }
        auto entry = [&]() {
            return a.cells[((uint32_t(P[2]) >> (16 + kCellLog)) * M + (uint32_t(P[1]) >> (16 + kCellLog))) * M +
                           (uint32_t(P[0]) >> (16 + kCellLog))];
        };
        double sum = 0.0;
        uint32_t prev = 0xffffffffu;
        uint2 next = entry();
        while (left > 0 && sum <= thr) {
            const uint2 e = next;
            const uint32_t lin = __umul24(__umul24(uint32_t(P[2]) >> bs, G) + (uint32_t(P[1]) >> bs), G) +
                                 (uint32_t(P[0]) >> bs);
            if (lin != prev) {  // the ray's smallest prefix sum in this macroblock
                prev = lin;
                vis_enter<kCellsCacheLog, __HIP_MEMORY_SCOPE_WAVEFRONT>(vcache, a.depth_bits, lin, sum);
            }
            const float c = __uint_as_float(e.x);
            const bool run = c == 0.0f || (exact && e.x != kMixed);
            int32_t n = min(steps_in_cube(P, up, inv, run ? e.y : uint32_t(bs)), left);
            if (!run) n = min(n, kCellAhead);
            uint32_t Q[3] = {uint32_t(P[0]), uint32_t(P[1]), uint32_t(P[2])};
            left -= n;
#pragma unroll
            for (int q = 0; q < 3; ++q) P[q] += __mul24(n, s[q]);  // |n s| <= B 2^16 + 2^15
            if (left > 0) next = entry();  // in flight during the samples
            if (run) {
                sum = fma(double(n), double(c), sum);
            } else {
                // samples past the last are clamped onto it, so every load is in bounds
                float sv[kCellAhead];
#pragma unroll
                for (int u = 0; u < kCellAhead; ++u) {
                    if (u > 0) {
                        const uint32_t m = u < n ? 0xffffffffu : 0u;
#pragma unroll
                        for (int q = 0; q < 3; ++q) Q[q] += uint32_t(s[q]) & m;
                    }
                    if (IDX == kIdxPow2)
                        sv[u] = a.sigma[(Q[0] >> 16) | ((Q[1] >> 16) << lg) | ((Q[2] >> 16) << (2 * lg))];
                    else if (IDX == kIdx32)
                        sv[u] = a.sigma[__umul24(__umul24(Q[2] >> 16, N) + (Q[1] >> 16), N) + (Q[0] >> 16)];
                    else
                        sv[u] = a.sigma[(uint64_t(Q[2] >> 16) * N + (Q[1] >> 16)) * N + (Q[0] >> 16)];
                }
#pragma unroll
                for (int u = 0; u < kCellAhead; ++u) sum += u < n ? double(sv[u]) : 0.0;
            }
        }
    }
}

struct BakeCompactArgs {
    const float* bmax;
    const uint64_t* depth_bits;
    int64_t n_lin;        // G^3
    int32_t N;
    double sigma_thr;     // keep when max sigma >= this (alpha >= tau_alpha)
    double sum_thr;       // keep when min prefix sum <= this (T >= tau_vis)
    float* block_alpha;   // nullable
    float* block_vis;     // nullable
    int32_t* indirection;
    int32_t* n_blocks;    // device, one int
};

__global__ __launch_bounds__(1024) void k_bake_compact(BakeCompactArgs a) {
    __shared__ int32_t wtot[16];
    __shared__ int32_t base;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, n_waves = blockDim.x >> 6;
    if (threadIdx.x == 0) base = 0;
    __syncthreads();
    const double inv_n = 1.0 / double(a.N);
    for (int64_t c0 = 0; c0 < a.n_lin; c0 += blockDim.x) {
        const int64_t lin = c0 + threadIdx.x;
        bool keep = false;
        if (lin < a.n_lin) {
            const double sm = double(a.bmax[lin]);
            const double dm = __longlong_as_double((long long)a.depth_bits[lin]);
            keep = sm >= a.sigma_thr && dm <= a.sum_thr;
            if (a.block_alpha) a.block_alpha[lin] = float(1.0 - exp(-sm * inv_n));
            if (a.block_vis) a.block_vis[lin] = dm <= a.sum_thr ? float(exp(-dm * inv_n)) : 0.0f;
        }
        const uint64_t bal = __ballot(keep);
        const int32_t below = __popcll(bal & ((uint64_t(1) << lane) - 1));
        if (lane == 0) wtot[wave] = __popcll(bal);
        __syncthreads();
        int32_t off = base;
        for (int w = 0; w < wave; ++w) off += wtot[w];
        if (lin < a.n_lin) a.indirection[lin] = keep ? off + below : -1;
        __syncthreads();
        if (threadIdx.x == 0) {
            int32_t tot = 0;
            for (int w = 0; w < n_waves; ++w) tot += wtot[w];
            base += tot;
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) *a.n_blocks = base;
}

// lin_of[id] = indirection index of atlas id (ids outside [0, n_blocks) are
// ignored); lin_of holds -1 beforehand.
__global__ __launch_bounds__(256) void k_bake_invert(const int32_t* __restrict__ ind, int64_t n_lin, int32_t n_blocks,
                                                     int32_t* __restrict__ lin_of) {
    const int64_t lin = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (lin >= n_lin) return;
    const int32_t id = ind[lin];
    if (id >= 0 && id < n_blocks) lin_of[id] = int32_t(lin);
}

struct BakeQuantArgs {
    const float* sigma;
    const float* rgb;
    const float* feat;
    const int32_t* lin_of;
    int32_t N, logB, G;
    float k_sigma;  // 255 / sigma_scale, float32
    uint8_t* dens8;
    uint8_t* rgb8;
    uint8_t* feat8;
};

__device__ __forceinline__ uint32_t qbyte(float x, float k) {
    const float q = __builtin_rintf(__fmul_rn(x, k));
    return uint32_t(fminf(fmaxf(q, 0.0f), 255.0f));
}

// grid.x = atlas id, grid.y = chunk of 256 lanes x V voxels of the block.
template <int V>
__global__ __launch_bounds__(256) void k_bake_quantize(BakeQuantArgs a) {
    const int32_t id = blockIdx.x;
    const int32_t B = 1 << a.logB;
    const int64_t B3 = int64_t(B) * B * B;
    const int64_t e0 = (int64_t(blockIdx.y) * blockDim.x + threadIdx.x) * V;  // first voxel, canonical order
    if (e0 >= B3) return;
    const int32_t lx = int32_t(e0 & (B - 1)), ly = int32_t((e0 >> a.logB) & (B - 1)), lz = int32_t(e0 >> (2 * a.logB));
    const int64_t out = int64_t(id) * B3 + e0;
    const int32_t lin = a.lin_of[id];
    uint32_t dq[V], rq[3 * V], fq[4 * V];
    if (lin < 0) {
#pragma unroll
        for (int i = 0; i < V; ++i) dq[i] = 0;
#pragma unroll
        for (int i = 0; i < 3 * V; ++i) rq[i] = 0;
#pragma unroll
        for (int i = 0; i < 4 * V; ++i) fq[i] = 0;
    } else {
        const int32_t bx = lin % a.G, by = (lin / a.G) % a.G, bz = lin / (a.G * a.G);
        const int64_t v = (int64_t(bz * B + lz) * a.N + (by * B + ly)) * a.N + bx * B + lx;
        const float kr = 255.0f;
        if (V == 4) {
            const f32x4 sg = ld4(a.sigma + v);
#pragma unroll
            for (int i = 0; i < 4; ++i) dq[i] = qbyte(sg.v[i], a.k_sigma);
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const f32x4 x = ld4(a.rgb + 3 * v + 4 * c);
#pragma unroll
                for (int i = 0; i < 4; ++i) rq[4 * c + i] = qbyte(x.v[i], kr);
            }
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const f32x4 x = ld4(a.feat + 4 * v + 4 * c);
#pragma unroll
                for (int i = 0; i < 4; ++i) fq[4 * c + i] = qbyte(x.v[i], kr);
            }
        } else {
#pragma unroll
            for (int i = 0; i < V; ++i) {
                dq[i] = qbyte(a.sigma[v + i], a.k_sigma);
#pragma unroll
                for (int c = 0; c < 3; ++c) rq[3 * i + c] = qbyte(a.rgb[3 * (v + i) + c], kr);
#pragma unroll
                for (int c = 0; c < 4; ++c) fq[4 * i + c] = qbyte(a.feat[4 * (v + i) + c], kr);
            }
        }
    }
    if (V == 4) {
        *reinterpret_cast<uint32_t*>(a.dens8 + out) = dq[0] | (dq[1] << 8) | (dq[2] << 16) | (dq[3] << 24);
        uint32_t* r = reinterpret_cast<uint32_t*>(a.rgb8 + 3 * out);
#pragma unroll
        for (int w = 0; w < 3; ++w)
            r[w] = rq[4 * w] | (rq[4 * w + 1] << 8) | (rq[4 * w + 2] << 16) | (rq[4 * w + 3] << 24);
        uint32_t* f = reinterpret_cast<uint32_t*>(a.feat8 + 4 * out);
#pragma unroll
        for (int w = 0; w < 4; ++w)
            f[w] = fq[4 * w] | (fq[4 * w + 1] << 8) | (fq[4 * w + 2] << 16) | (fq[4 * w + 3] << 24);
    } else {
#pragma unroll
        for (int i = 0; i < V; ++i) {
            a.dens8[out + i] = uint8_t(dq[i]);
#pragma unroll
            for (int c = 0; c < 3; ++c) a.rgb8[3 * (out + i) + c] = uint8_t(rq[3 * i + c]);
#pragma unroll
            for (int c = 0; c < 4; ++c) a.feat8[4 * (out + i) + c] = uint8_t(fq[4 * i + c]);
        }
    }
}

hipError_t launch_bake_cull(const BakeCullPlan& p, hipStream_t s) {
    const int64_t G3 = int64_t(p.G) * p.G * p.G;
    hipError_t e;
    // Macroblocks of 8^3 and more on grids of up to 2048^3 (128 MB of cells)
    // go through the cell table; smaller ones would pay a step for every few
    // voxels, and past that the table would crowd a field of 275 GB.
    if (p.cells) {
        if ((e = launch_fill_i32(reinterpret_cast<int32_t*>(p.stats), 2, 0, s)) != hipSuccess) return e;
        hipLaunchKernelGGL(k_bake_cells, dim3(unsigned(G3)), dim3(p.logB == 3 ? 64 : 256), 0, s, p.sigma, p.N, p.logB,
                           p.G, p.bmax, p.depth_bits, p.cells, p.stats);
    } else if (p.vec4) {
        hipLaunchKernelGGL(k_bake_block_max<4>, dim3(unsigned(G3)), dim3(256), 0, s, p.sigma, p.N, p.logB, p.G,
                           p.bmax, p.depth_bits);
    } else {
        hipLaunchKernelGGL(k_bake_block_max<1>, dim3(unsigned(G3)), dim3(256), 0, s, p.sigma, p.N, p.logB, p.G,
                           p.bmax, p.depth_bits);
    }
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if (p.total_tiles > 0) {
        BakeVisArgs v;
        v.sigma = p.sigma;
        v.cams = p.cams;
        v.n_cams = p.n_cams;
        v.N = p.N;
        v.logB = p.logB;
        v.G = p.G;
        v.total_tiles = p.total_tiles;
        v.tile_w = p.tile_w;
        v.tile_h = p.tile_h;
        v.sum_thr = p.sum_thr;
        v.depth_bits = p.depth_bits;
        v.cells = p.cells;
        v.stats = p.stats;
        const dim3 blocks(unsigned((p.total_tiles + 3) / 4));
        const int idx = (p.N & (p.N - 1)) == 0 && p.N <= 1024
                            ? kIdxPow2
                            : (int64_t(p.N) * p.N * p.N <= int64_t(0xffffffffu) ? kIdx32 : kIdx64);
        if (p.cells) {
            hipLaunchKernelGGL(k_bake_choose, dim3(1), dim3(1024), 0, s, p.cells, uint32_t(p.N) >> kCellLog, p.stats);
            if ((e = hipGetLastError()) != hipSuccess) return e;
            // resident workgroups only, so that their caches of bounds serve many tiles
            const dim3 wgs(blocks.x > 4u * 2048u ? 2048u : blocks.x);
            if (idx == kIdxPow2) hipLaunchKernelGGL(k_bake_visibility_cells<kIdxPow2>, wgs, dim3(256), 0, s, v);
            else if (idx == kIdx32) hipLaunchKernelGGL(k_bake_visibility_cells<kIdx32>, wgs, dim3(256), 0, s, v);
            else hipLaunchKernelGGL(k_bake_visibility_cells<kIdx64>, wgs, dim3(256), 0, s, v);
            if ((e = hipGetLastError()) != hipSuccess) return e;
        }
        if (idx == kIdxPow2) hipLaunchKernelGGL(k_bake_visibility<kIdxPow2>, blocks, dim3(256), 0, s, v);
        else if (idx == kIdx32) hipLaunchKernelGGL(k_bake_visibility<kIdx32>, blocks, dim3(256), 0, s, v);
        else hipLaunchKernelGGL(k_bake_visibility<kIdx64>, blocks, dim3(256), 0, s, v);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    BakeCompactArgs c;
    c.bmax = p.bmax;
    c.depth_bits = p.depth_bits;
    c.n_lin = G3;
    c.N = p.N;
    c.sigma_thr = p.sigma_thr;
    c.sum_thr = p.sum_thr;
    c.block_alpha = p.block_alpha;
    c.block_vis = p.block_vis;
    c.indirection = p.indirection;
    c.n_blocks = p.n_blocks_dev;
    hipLaunchKernelGGL(k_bake_compact, dim3(1), dim3(1024), 0, s, c);
    return hipGetLastError();
}

hipError_t launch_bake_quantize(const BakeQuantPlan& p, hipStream_t s) {
    const int64_t G3 = int64_t(p.G) * p.G * p.G;
    hipError_t e = launch_fill_i32(p.lin_of, p.n_blocks, -1, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_bake_invert, dim3(unsigned((G3 + 255) / 256)), dim3(256), 0, s, p.indirection, G3,
                       p.n_blocks, p.lin_of);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    BakeQuantArgs q;
    q.sigma = p.sigma;
    q.rgb = p.rgb;
    q.feat = p.feat;
    q.lin_of = p.lin_of;
    q.N = p.N;
    q.logB = p.logB;
    q.G = p.G;
    q.k_sigma = p.k_sigma;
    q.dens8 = p.dens8;
    q.rgb8 = p.rgb8;
    q.feat8 = p.feat8;
    const int64_t B3 = int64_t(1) << (3 * p.logB);
    const int V = p.vec4 ? 4 : 1;
    const unsigned chunks = unsigned((B3 / V + 255) / 256);
    if (p.vec4)
        hipLaunchKernelGGL(k_bake_quantize<4>, dim3(unsigned(p.n_blocks), chunks), dim3(256), 0, s, q);
    else
        hipLaunchKernelGGL(k_bake_quantize<1>, dim3(unsigned(p.n_blocks), chunks), dim3(256), 0, s, q);
    return hipGetLastError();
}

}  // namespace snerg
