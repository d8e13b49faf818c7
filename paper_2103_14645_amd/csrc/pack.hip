// Packing of a canonical SNeRG atlas into the layout the render kernels read
// (described in snerg_dev.h).  Atlas ids outside [0, n_blocks) in the
// indirection grid count as empty macroblocks, and ranks beyond n_blocks
// (only possible when atlas ids repeat) are dropped, so no kernel can index
// past the packed buffer whatever the indirection holds.
#include "snerg_dev.h"
#include "snerg_launch.h"

namespace snerg {

__global__ void k_fill_i32(int32_t* p, int64_t n, int32_t v) {
    int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

__global__ void k_fill_f32(float* p, int64_t n, float v) {
    int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

// Occupancy table and rank maps.

// Occupancy bits of the words, 64 entries (two words) per wavefront and step,
// read coalesced: thread t of n, whole wavefronts.
__device__ __forceinline__ void pack_bits(const int32_t* __restrict__ ind, int64_t G3, int32_t n_blocks,
                                          int32_t n_words, uint2* occ, int64_t t, int64_t n) {
    const int lane = int(t & 63);
    for (int64_t base = t - lane; base < int64_t(n_words) * 32; base += n) {
        const int64_t lin = base + lane;
        const int32_t id = lin < G3 ? ind[lin] : -1;
        const uint64_t m = __ballot(id >= 0 && id < n_blocks);
        const int64_t w = (base >> 5) + (lane >> 5);
        if ((lane & 31) == 0 && w < n_words) occ[w].x = uint32_t(m >> (lane & 32));
    }
}

// Ranks of the words: an exclusive prefix sum of their popcounts by a workgroup of
// 1024 threads, each with `per` consecutive words.  Returns their total.
__device__ __forceinline__ int32_t pack_scan(int32_t n_words, uint2* occ) {
    __shared__ int32_t part[1024];
    const int t = threadIdx.x;
    const int per = (n_words + 1023) / 1024;
    const int w0 = t * per;
    int32_t sum = 0;
    for (int i = 0; i < per; ++i)
        if (w0 + i < n_words) sum += __popc(occ[w0 + i].x);
    part[t] = sum;
    __syncthreads();
    for (int off = 1; off < 1024; off <<= 1) {
        const int32_t v = t >= off ? part[t - off] : 0;
        __syncthreads();
        part[t] += v;
        __syncthreads();
    }
    int32_t run = part[t] - sum;
    for (int i = 0; i < per; ++i)
        if (w0 + i < n_words) {
            occ[w0 + i].y = uint32_t(run);
            run += __popc(occ[w0 + i].x);
        }
    return part[1023];
}

// The rank maps from the words, -1 past the last of `total` occupied macroblocks.
__device__ __forceinline__ void pack_ranks(const int32_t* __restrict__ ind, int64_t G3, int32_t n_blocks,
                                           int32_t total, const uint2* occ, int32_t* __restrict__ rank_lin,
                                           int32_t* __restrict__ rank_id, int64_t t, int64_t n) {
    for (int64_t lin = t; lin < G3; lin += n) {
        const uint2 e = occ[lin >> 5];
        const int j = int(lin & 31);
        if (!((e.x >> j) & 1u)) continue;
        const int32_t r = int32_t(e.y) + __popc(e.x & ((1u << j) - 1u));
        if (r < n_blocks) {  // beyond only when atlas ids repeat
            rank_lin[r] = int32_t(lin);
            rank_id[r] = ind[lin];
        }
    }
    for (int64_t r = total + t; r < n_blocks; r += n) {
        rank_lin[r] = -1;
        rank_id[r] = -1;
    }
}

// One launch for all three, while one workgroup's bandwidth does (5 launches and
// 23 us of kernels before, 7 us now, on a 16^3 indirection grid) ...
__global__ __launch_bounds__(1024) void k_pack_tables(const int32_t* __restrict__ ind, int64_t G3, int32_t n_blocks,
                                                      int32_t n_words, uint2* occ, int32_t* __restrict__ rank_lin,
                                                      int32_t* __restrict__ rank_id) {
    pack_bits(ind, G3, n_blocks, n_words, occ, threadIdx.x, 1024);
    __syncthreads();  // the workgroup's own global writes are visible to it
    const int32_t total = pack_scan(n_words, occ);
    __syncthreads();
    pack_ranks(ind, G3, n_blocks, total, occ, rank_lin, rank_id, threadIdx.x, 1024);
}

// ... and three for larger grids, the first and the last over the whole chip.
__global__ __launch_bounds__(256) void k_pack_bits(const int32_t* __restrict__ ind, int64_t G3, int32_t n_blocks,
                                                   int32_t n_words, uint2* __restrict__ occ) {
    pack_bits(ind, G3, n_blocks, n_words, occ, int64_t(blockIdx.x) * 256 + threadIdx.x, int64_t(gridDim.x) * 256);
}
__global__ __launch_bounds__(1024) void k_pack_scan(int32_t n_words, uint2* occ) { pack_scan(n_words, occ); }
__global__ __launch_bounds__(256) void k_pack_ranks(const int32_t* __restrict__ ind, int64_t G3, int32_t n_blocks,
                                                    int32_t n_words, const uint2* __restrict__ occ,
                                                    int32_t* __restrict__ rank_lin, int32_t* __restrict__ rank_id) {
    const uint2 last = occ[n_words - 1];
    pack_ranks(ind, G3, n_blocks, int32_t(last.y) + __popc(last.x), occ, rank_lin, rank_id,
               int64_t(blockIdx.x) * 256 + threadIdx.x, int64_t(gridDim.x) * 256);
}

// The eight channel values of canonical voxel vi.
__device__ __forceinline__ void load_voxel(const float* __restrict__ dens, const float* __restrict__ rgb,
                                           const float* __restrict__ feat, int64_t vi, float val[8]) {
    val[0] = dens[vi];
#pragma unroll
    for (int c = 0; c < 3; ++c) val[1 + c] = rgb[vi * 3 + c];
#pragma unroll
    for (int c = 0; c < 4; ++c) val[4 + c] = feat[vi * 4 + c];
}

// uint8: the colour and feature bytes as one dword each (at any alignment)
// instead of seven byte loads.  The colour dword ends with the voxel's last
// byte, so it never reaches past the array; voxel 0 has none before it and
// starts with its first.
__device__ __forceinline__ void load_voxel(const uint8_t* __restrict__ dens, const uint8_t* __restrict__ rgb,
                                           const uint8_t* __restrict__ feat, int64_t vi, uint8_t val[8]) {
    uint32_t c3, f4;
    if (vi > 0) {
        __builtin_memcpy(&c3, rgb + vi * 3 - 1, 4);
        c3 >>= 8;
    } else {
        c3 = uint32_t(rgb[0]) | (uint32_t(rgb[1]) << 8) | (uint32_t(rgb[2]) << 16);
    }
    __builtin_memcpy(&f4, feat + vi * 4, 4);
    val[0] = dens[vi];
#pragma unroll
    for (int c = 0; c < 3; ++c) val[1 + c] = uint8_t(c3 >> (8 * c));
#pragma unroll
    for (int c = 0; c < 4; ++c) val[4 + c] = uint8_t(f4 >> (8 * c));
}

// One thread per padded voxel, `chunks` workgroups per block record, of the records
// from `first` on.
template <typename T>
__global__ __launch_bounds__(256) void k_pack_vox(const int32_t* __restrict__ ind, const int32_t* __restrict__ rank_lin,
                                                  const T* __restrict__ dens, const T* __restrict__ rgb,
                                                  const T* __restrict__ feat, int32_t N, int32_t B, int32_t logB,
                                                  int32_t n_blocks, int32_t first, int32_t chunks,
                                                  int64_t rec_stride, int64_t dist_bytes, uint8_t* __restrict__ rec) {
    const uint32_t block = blockIdx.x / uint32_t(chunks);
    const int32_t r = first + int32_t(block);
    const uint32_t v = (blockIdx.x - block * uint32_t(chunks)) * 256u + threadIdx.x;
    const uint32_t Bp = uint32_t(B) + 2;
    if (v >= Bp * Bp * Bp) return;
    const int32_t pz = int32_t(v / (Bp * Bp)), py = int32_t(v / Bp - uint32_t(pz) * Bp), px = int32_t(v % Bp);
    const int32_t G = N >> logB;
    T val[8] = {T(0), T(0), T(0), T(0), T(0), T(0), T(0), T(0)};
    const int32_t lin = rank_lin[r];
    if (lin >= 0) {
        const int32_t bx = lin % G, by = (lin / G) % G, bz = lin / (G * G);
        const int32_t gx = bx * B + px - 1, gy = by * B + py - 1, gz = bz * B + pz - 1;
        if (gx >= 0 && gy >= 0 && gz >= 0 && gx < N && gy < N && gz < N) {
            const int32_t nb = ((gz >> logB) * G + (gy >> logB)) * G + (gx >> logB);
            const int32_t gid = ind[nb];
            if (gid >= 0 && gid < n_blocks) {
                const int32_t lx = gx & (B - 1), ly = gy & (B - 1), lz = gz & (B - 1);
                load_voxel(dens, rgb, feat, int64_t(gid) * B * B * B + (int64_t(lz) * B + ly) * B + lx, val);
            }
        }
    }
    T* out = reinterpret_cast<T*>(rec + int64_t(r) * rec_stride + dist_bytes + int64_t(v) * 8 * sizeof(T));
    __builtin_memcpy(__builtin_assume_aligned(out, 8 * sizeof(T) > 16 ? 16 : 8), val, 8 * sizeof(T));
}

// Distance bytes of a record, B <= 32, one workgroup per record.  Rows of
// cells are bit masks (B + 1 <= 33 bits in a 64-bit word), so the whole record
// lives in LDS and every step handles a row at once:
//  1. the non-zero bits of the padded voxels, straight from the canonical
//     densities (4 bytes a voxel instead of a 32-byte stride through the
//     packed ones), a ballot per row; a cell is active when any of its 8
//     corners is;
//  2. the Chebyshev distance by dilation: A_0 = active, A_{d+1} = the 3x3x3
//     dilation of A_d; a cell's distance is the number of A_d that do not
//     hold it, counted in bit planes kept in registers.  It ends when a pass
//     fills every row (at most B passes); a record without active cells gets
//     255 everywhere;
//  3. the planes go through LDS into coalesced 4-byte stores.
// Bound by the latency of the row loads.  The three byte-wise passes it
// replaces (a serial scan in x, then for each of y and z a minimum over all
// pairs of a line, from private arrays) took 5.86 ms for the 433 records of a
// float32 512^3 grid; this takes 0.15 ms.  At B = 64 a row does not fit the
// word and the planes do not fit LDS: k_dist_x and k_dist_line stay for it.
template <int LOGB>
struct DistShape {
    static constexpr int B = 1 << LOGB, Bp = B + 2, Bc = B + 1;
    static constexpr int kThreads = LOGB <= 3 ? 64 : (LOGB == 4 ? 256 : 512);
    static constexpr int kRows = Bc * Bc;                              // cell rows
    static constexpr int kOwn = (kRows + kThreads - 1) / kThreads;     // rows per thread
    static constexpr int kPlanes = LOGB + 1;                           // distances 0..B
    static constexpr int kWork = Bp * Bp + 2 * kRows;                  // voxel rows, two cell buffers
    static constexpr int kOut = kPlanes * kRows;
    static constexpr int kLds = kWork > kOut ? kWork : kOut;           // 64-bit words, the planes reuse the buffers
};

template <int LOGB, typename T>
__global__ __launch_bounds__(DistShape<LOGB>::kThreads) void k_dist(const int32_t* __restrict__ ind,
                                                                    const int32_t* __restrict__ rank_lin,
                                                                    const T* __restrict__ dens, int32_t N,
                                                                    int32_t n_blocks, int64_t rec_stride,
                                                                    uint8_t* __restrict__ rec) {
    using S = DistShape<LOGB>;
    constexpr int B = S::B, Bp = S::Bp, Bc = S::Bc;
    __shared__ uint64_t lds[S::kLds];
    uint64_t* nz = lds;                   // [Bp * Bp] non-zero voxels, bit x
    uint64_t* cur = lds + Bp * Bp;        // [kRows] cells within the current distance
    uint64_t* tmp = cur + S::kRows;       // [kRows] the same, dilated in x and y
    const int32_t r = blockIdx.x;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int32_t G = N >> LOGB;
    const int32_t lin = rank_lin[r];
    const int32_t bx = lin % G, by = (lin / G) % G, bz = lin / (G * G);

    // 1. voxel rows: 64 / Bp rows per wavefront and step, lane = x within a row
    constexpr int kPerWave = 64 / Bp, kWaves = S::kThreads / 64;
    constexpr int kAhead = 8;  // rows in flight per lane
    const int sub = lane / Bp, x = lane - sub * Bp;
    for (int row0 = wave * kPerWave; row0 < Bp * Bp; row0 += kAhead * kWaves * kPerWave) {
        T v[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            const int row = row0 + u * kWaves * kPerWave + sub;
            v[u] = T(0);
            if (lin >= 0 && sub < kPerWave && row < Bp * Bp) {
                const int32_t gx = bx * B + x - 1, gy = by * B + row % Bp - 1, gz = bz * B + row / Bp - 1;
                if (gx >= 0 && gy >= 0 && gz >= 0 && gx < N && gy < N && gz < N) {
                    const int32_t gid = ind[((gz >> LOGB) * G + (gy >> LOGB)) * G + (gx >> LOGB)];
                    if (gid >= 0 && gid < n_blocks)
                        v[u] = dens[(int64_t(gid) << (3 * LOGB)) + ((((gz & (B - 1)) << LOGB) + (gy & (B - 1))) << LOGB) +
                                    (gx & (B - 1))];
                }
            }
        }
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            const int row = row0 + u * kWaves * kPerWave + sub;
            const uint64_t m = __ballot(v[u] != T(0));
            if (x == 0 && sub < kPerWave && row < Bp * Bp) nz[row] = (m >> (sub * Bp)) & ((uint64_t(1) << Bp) - 1);
        }
    }
    __syncthreads();
    constexpr uint64_t kFull = (uint64_t(1) << Bc) - 1;
    uint64_t plane[S::kOwn][S::kPlanes];
    bool some = false;
#pragma unroll
    for (int i = 0; i < S::kOwn; ++i) {
#pragma unroll
        for (int p = 0; p < S::kPlanes; ++p) plane[i][p] = 0;
        const int row = threadIdx.x + i * S::kThreads;
        if (row < S::kRows) {
            const uint64_t* q = nz + (row / Bc) * Bp + row % Bc;
            uint64_t m = (q[0] | q[1]) | (q[Bp] | q[Bp + 1]);
            m = (m | (m >> 1)) & kFull;
            cur[row] = m;
            some |= m != 0;
        }
    }
    // 2. dilate until every row is full
    some = __syncthreads_or(some);
    if (some) {
        for (;;) {
            bool open = false;
#pragma unroll
            for (int i = 0; i < S::kOwn; ++i) {
                const int row = threadIdx.x + i * S::kThreads;
                if (row < S::kRows) {
                    const int cy = row % Bc;
                    const uint64_t own = cur[row];
                    uint64_t carry = ~own & kFull;  // one more for the cells not reached yet
                    open |= carry != 0;
#pragma unroll
                    for (int p = 0; p < S::kPlanes; ++p) {
                        const uint64_t t = plane[i][p];
                        plane[i][p] = t ^ carry;
                        carry &= t;
                    }
                    uint64_t m = own | (cy > 0 ? cur[row - 1] : 0) | (cy < Bc - 1 ? cur[row + 1] : 0);
                    tmp[row] = (m | (m << 1) | (m >> 1)) & kFull;
                }
            }
            if (!__syncthreads_or(open)) break;  // also: tmp complete, cur read
#pragma unroll
            for (int i = 0; i < S::kOwn; ++i) {
                const int row = threadIdx.x + i * S::kThreads;
                if (row < S::kRows)
                    cur[row] = tmp[row] | (row >= Bc ? tmp[row - Bc] : 0) | (row < S::kRows - Bc ? tmp[row + Bc] : 0);
            }
            __syncthreads();
        }
    }
    // 3. planes -> bytes (every thread has passed the barrier that ended the loop)
#pragma unroll
    for (int i = 0; i < S::kOwn; ++i) {
        const int row = threadIdx.x + i * S::kThreads;
        if (row < S::kRows)
#pragma unroll
            for (int p = 0; p < S::kPlanes; ++p) lds[p * S::kRows + row] = plane[i][p];
    }
    __syncthreads();
    constexpr int kCells = Bc * Bc * Bc;
    uint32_t* out = reinterpret_cast<uint32_t*>(rec + int64_t(r) * rec_stride);  // dist_bytes is a multiple of 16
    for (int w = threadIdx.x; w < (kCells + 3) / 4; w += S::kThreads) {
        uint32_t word = 0;
        int row = 4 * w / Bc, cx = 4 * w - row * Bc;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            uint32_t d = 255;
            if (some) {
                d = 0;
                const int rr = row < S::kRows ? row : S::kRows - 1;  // the last word's padding
#pragma unroll
                for (int p = 0; p < S::kPlanes; ++p) d |= uint32_t((lds[p * S::kRows + rr] >> cx) & 1u) << p;
            }
            word |= d << (8 * k);
            if (++cx == Bc) {
                cx = 0;
                ++row;
            }
        }
        out[w] = word;
    }
}

constexpr int kMaxLine = 65;  // B + 1 for B = 64

// Distance pass along x (B = 64): one thread per (record, cz, cy) line.  Computes
// each cell's activity from its 8 corner densities and the 1D distance to
// the nearest active cell of the line.
template <typename T>
__global__ void k_dist_x(int32_t B, int32_t n_blocks, int64_t rec_stride, int64_t dist_bytes,
                         uint8_t* __restrict__ rec) {
    const int32_t Bc = B + 1, Bp = B + 2;
    const int64_t t = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (t >= int64_t(n_blocks) * Bc * Bc) return;
    const int32_t r = int32_t(t / (Bc * Bc));
    const int32_t yz = int32_t(t - int64_t(r) * Bc * Bc);
    const int32_t cy = yz % Bc, cz = yz / Bc;
    uint8_t* dist = rec + int64_t(r) * rec_stride;
    const T* vox = reinterpret_cast<const T*>(dist + dist_bytes);
    int32_t last = -1000;
    for (int cx = 0; cx < Bc; ++cx) {
        bool any = false;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int32_t v = ((cz + (k >> 2)) * Bp + (cy + ((k >> 1) & 1))) * Bp + (cx + (k & 1));
            any |= vox[int64_t(v) * 8] != T(0);
        }
        if (any) last = cx;
        const int32_t d = cx - last;
        dist[(cz * Bc + cy) * Bc + cx] = uint8_t(d > 255 ? 255 : d);
    }
    last = 1000 + Bc;
    for (int cx = Bc - 1; cx >= 0; --cx) {
        uint8_t* q = &dist[(cz * Bc + cy) * Bc + cx];
        if (*q == 0) last = cx;
        const int32_t d = last - cx;
        if (d < *q) *q = uint8_t(d);
    }
}

// Distance pass along y (axis = 1) or z (axis = 2) (B = 64): one thread per line;
// out[i] = min_j max(|i - j|, in[j]) turns the distance to the nearest active
// cell in the lower dimensions into the Chebyshev distance in one more axis.
__global__ void k_dist_line(int32_t B, int32_t n_blocks, int32_t axis, int64_t rec_stride,
                            uint8_t* __restrict__ rec) {
    const int32_t Bc = B + 1;
    const int64_t t = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (t >= int64_t(n_blocks) * Bc * Bc) return;
    const int32_t r = int32_t(t / (Bc * Bc));
    const int32_t uv = int32_t(t - int64_t(r) * Bc * Bc);
    const int32_t u = uv % Bc, w = uv / Bc;
    uint8_t* dist = rec + int64_t(r) * rec_stride;
    // axis 1: cells (u, i, w) = x u, y i, z w; axis 2: (u, w, i) = x u, y w, z i
    const int32_t stride = axis == 1 ? Bc : Bc * Bc;
    const int32_t base = axis == 1 ? (w * Bc * Bc + u) : (w * Bc + u);
    uint8_t in[kMaxLine];
    for (int i = 0; i < Bc; ++i) in[i] = dist[base + i * stride];
    for (int i = 0; i < Bc; ++i) {
        int32_t best = 255;
        for (int j = 0; j < Bc; ++j) {
            const int32_t dj = i > j ? i - j : j - i;
            const int32_t m = dj > in[j] ? dj : in[j];
            best = m < best ? m : best;
        }
        dist[base + i * stride] = uint8_t(best);
    }
}

static inline unsigned nblk(int64_t n, int t) { return unsigned((n + t - 1) / t); }

hipError_t launch_fill_i32(int32_t* p, int64_t n, int32_t v, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_fill_i32, dim3(nblk(n, 256)), dim3(256), 0, s, p, n, v);
    return hipGetLastError();
}

hipError_t launch_fill_f32(float* p, int64_t n, float v, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_fill_f32, dim3(nblk(n, 256)), dim3(256), 0, s, p, n, v);
    return hipGetLastError();
}

template <typename T>
static hipError_t launch_pack_t(const PackedLayout& L, int32_t n_blocks, const int32_t* ind, const int32_t* rank_lin,
                                const T* dens, const T* rgb, const T* feat, uint8_t* rec, hipStream_t s) {
    hipError_t e;
    const int32_t chunks = (L.Bp * L.Bp * L.Bp + 255) / 256;
    // (a launch holds fewer than 2^32 threads: 108,942 records of blocks of 32)
    const int32_t most = ((1 << 24) - 1) / chunks;
    for (int32_t first = 0; first < n_blocks; first += most) {
        const int32_t n = n_blocks - first < most ? n_blocks - first : most;
        hipLaunchKernelGGL(k_pack_vox<T>, dim3(unsigned(n) * unsigned(chunks)), dim3(256), 0, s, ind, rank_lin, dens, rgb,
                           feat, L.N, L.B, L.logB, n_blocks, first, chunks, L.rec_stride, L.dist_bytes, rec);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
#define SNERG_DIST(LB)                                                                                               \
    case LB:                                                                                                         \
        hipLaunchKernelGGL((k_dist<LB, T>), dim3(unsigned(n_blocks)), dim3(DistShape<LB>::kThreads), 0, s, ind, rank_lin, \
                           dens, L.N, n_blocks, L.rec_stride, rec);                                                  \
        return hipGetLastError();
    switch (L.logB) {
        SNERG_DIST(1)
        SNERG_DIST(2)
        SNERG_DIST(3)
        SNERG_DIST(4)
        SNERG_DIST(5)
    }
#undef SNERG_DIST
    const int64_t lines = int64_t(n_blocks) * L.Bc * L.Bc;
    hipLaunchKernelGGL(k_dist_x<T>, dim3(nblk(lines, 256)), dim3(256), 0, s, L.B, n_blocks, L.rec_stride, L.dist_bytes,
                       rec);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    for (int axis = 1; axis <= 2; ++axis) {
        hipLaunchKernelGGL(k_dist_line, dim3(nblk(lines, 256)), dim3(256), 0, s, L.B, n_blocks, axis, L.rec_stride, rec);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    return hipSuccess;
}

// One workgroup for the tables up to 24^3 macroblocks: a call that packs little else
// takes 14.3 us with it and 18.0 with three launches at 20^3, 18.2 and 17.7 at 24^3,
// 31 and 18 at 32^3, 201 and 52 at 64^3.
constexpr int64_t kTablesOneGroup = 24 * 24 * 24;

hipError_t launch_pack(const PackedLayout& L, int32_t n_blocks, bool f32, const int32_t* ind,
                       const void* dens, const void* rgb, const void* feat, uint8_t* packed, hipStream_t s) {
    uint2* occ = reinterpret_cast<uint2*>(packed + L.off_occ);
    int32_t* rank_lin = reinterpret_cast<int32_t*>(packed + L.off_rank_lin);
    int32_t* rank_id = reinterpret_cast<int32_t*>(packed + L.off_rank_id);
    uint8_t* rec = packed + L.off_rec;
    const int64_t G3 = int64_t(L.G) * L.G * L.G;
    hipError_t e;
    if (G3 <= kTablesOneGroup) {
        hipLaunchKernelGGL(k_pack_tables, dim3(1), dim3(1024), 0, s, ind, G3, n_blocks, L.n_words, occ, rank_lin, rank_id);
    } else {
        const dim3 n(nblk(G3, 256));
        hipLaunchKernelGGL(k_pack_bits, n, dim3(256), 0, s, ind, G3, n_blocks, L.n_words, occ);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        hipLaunchKernelGGL(k_pack_scan, dim3(1), dim3(1024), 0, s, L.n_words, occ);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        hipLaunchKernelGGL(k_pack_ranks, n, dim3(256), 0, s, ind, G3, n_blocks, L.n_words, occ, rank_lin, rank_id);
    }
    if ((e = hipGetLastError()) != hipSuccess || n_blocks == 0) return e;
    if (f32)
        return launch_pack_t(L, n_blocks, ind, rank_lin, (const float*)dens, (const float*)rgb, (const float*)feat, rec, s);
    return launch_pack_t(L, n_blocks, ind, rank_lin, (const uint8_t*)dens, (const uint8_t*)rgb, (const uint8_t*)feat, rec,
                         s);
}

}  // namespace snerg
