// Adjoint of the render (fine-tuning by a pixel loss, Eq. 3, Section 5.5).
//
// For each ray with output gradient g = dL/d(rgb, alpha):
//  K1 (k_mlp_backward, only with the MLP on): MLP backward (Eq. 7):
//     g_C = g_rgb + (J_R^T g_rgb)[0:3], g_V = (J_R^T g_rgb)[3:7], written per
//     ray; the weight gradients of the wavefront's 64 rays are summed with
//     FP32 MFMA outer products (rays are the K dimension) into per-wavefront
//     partial rows, reduced afterwards.
//  K2 (k_adjoint): re-march the same samples (nothing per sample was
//     stored).  With E = g_C . C_d + g_V . V (from the forward's saved C_d,
//     V), the running prefix P_k = sum_{j<=k} w_j e_j, e_k = g_C . c_k +
//     g_V . v_k and dL/dT_N = g_rgb . bg - g_alpha, Eq. 2/5/6 give
//        dL/dsigma_k = delta [T_k e_k - (E - P_k) - T_N dL/dT_N],
//        dL/dc_k = w_k g_C,  dL/dv_k = w_k g_V,
//     (T_k: transmittance after sample k).  Through the trilinear weights
//     w_c(k) a corner voxel receives sum_k w_c(k) dL/dsigma_k (density) and
//     g_C, g_V times A = sum_k w_c(k) w_k (colour, features).  Along one ray
//     each cell coordinate is monotone, so the 8 corners of the current cell
//     are kept as running (A, D) sums and a voxel is handed over once, when
//     the ray's cell window leaves it: into an LDS table that sums the
//     hand-overs of 32 neighbouring rays (whole views in 64-pixel tiles,
//     patch lists, long lists) or an LDS log (scattered lists), either way
//     flushed to the gradient arrays with float atomics grouped by cache line.
#include <type_traits>

#include "march.h"
#include "mlp.h"
#include "snerg_launch.h"

namespace snerg {

typedef float float4v __attribute__((ext_vector_type(4)));

constexpr int kBwdWaves = 2;  // wavefronts per K1 workgroup
// K1 staging row per ray (floats): gh1 | x (34) 1 0 | gh2 | h1 | go (3) 0 | h2
constexpr int kSGh1 = 0, kSX = 16, kSGh2 = 52, kSH1 = 68, kSGo = 84, kSH2 = 88;
constexpr int kStageRow = 105;

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) v += __shfl_xor(v, m);
    return v;
}

__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) v = fmaxf(v, __shfl_xor(v, m));
    return v;
}

__device__ __forceinline__ void locate(const BackwardArgs& a, int64_t r, int& ci, int& px, int& py) {
    ci = find_camera_by_ray(a.cams, a.n_cams, r);
    const int64_t local = r - a.cams[ci].ray_offset;
    py = int(local / a.cams[ci].W);
    px = int(local - int64_t(py) * a.cams[ci].W);
}

// ------------------------------------------------------------------ K1: MLP

// A-operand fragment of the transpose of a row-major [rows][cols] matrix M
// (a 16x16 tile of M^T): lane l holds M^T[l%16][4(l/16) + j] = M[4(l/16) + j][l%16].
__device__ __forceinline__ half4_t a_frag_t(cfloat* M, int rows, int cols, int lane) {
    const int c = lane & 15;
    const int r = 4 * (lane >> 4);
    half4_t v;
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = (r + j < rows && c < cols) ? _Float16(M[(r + j) * cols + c]) : _Float16(0.0f);
    return v;
}

__device__ __forceinline__ half4_t to_half4(float4_t v) {
    half4_t h;
#pragma unroll
    for (int j = 0; j < 4; ++j) h[j] = _Float16(v[j]);
    return h;
}

// The MLP chain of 64 rays on FP16 MFMA tiles.  xs: the rays' inputs
// ([64][kXRow] halves), gsm: per ray g_rgb and the gate, stage: per-ray
// rows that receive h1, h2, go, gh2, gh1 (float).  Tile layouts (16x16x16):
// A lane l = [m = l%16][k = 4(l/16)+j], B lane l = [k = 4(l/16)+j][n = l%16],
// D lane l = [m = 4(l/16)+v][n = l%16]; hidden units are rows, rays columns,
// so every D tile (after its element-wise step) is the next B operand.
__device__ __forceinline__ void mlp_backward_f16_wave(const BackwardArgs& a, cfloat* W, const _Float16* xs,
                                                      const float* gsm, float* stage, int64_t base, int lane) {
    const half8_t w1[2] = {a_frag32(W + kOffW1, kMlpIn, 0, lane), a_frag32(W + kOffW1, kMlpIn, 1, lane)};
    const half4_t w2 = a_frag(W + kOffW2, kMlpH, kMlpH, 0, 0, lane);
    const half4_t w3 = a_frag(W + kOffW3, kMlpOut, kMlpH, 0, 0, lane);
    const half4_t w3t = a_frag_t(W + kOffW3, kMlpOut, kMlpH, lane);
    const half4_t w2t = a_frag_t(W + kOffW2, kMlpH, kMlpH, lane);
    const half4_t w1t = a_frag_t(W + kOffW1, kMlpH, kMlpIn, lane);  // input rows 0..15
    const float4_t bb1 = bias_frag(W + kOffB1, kMlpH, lane);
    const float4_t bb2 = bias_frag(W + kOffB2, kMlpH, lane);
    const float4_t bb3 = bias_frag(W + kOffB3, kMlpOut, lane);
    const float4_t zero = {0.f, 0.f, 0.f, 0.f};
    const int n = lane & 15, rq = 4 * (lane >> 4);
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        const int ray = 16 * g + n;  // this lane's column
        const _Float16 (*rows)[kXRow] = reinterpret_cast<const _Float16 (*)[kXRow]>(xs);
        float4_t h1 = __builtin_amdgcn_mfma_f32_16x16x32_f16(w1[0], x_frag32(rows, g, 0, lane), bb1, 0, 0, 0);
        h1 = __builtin_amdgcn_mfma_f32_16x16x32_f16(w1[1], x_frag32(rows, g, 1, lane), h1, 0, 0, 0);
#pragma unroll
        for (int v = 0; v < 4; ++v) h1[v] = fmaxf(h1[v], 0.0f);
        float4_t h2 = __builtin_amdgcn_mfma_f32_16x16x16f16(w2, to_half4(h1), bb2, 0, 0, 0);
#pragma unroll
        for (int v = 0; v < 4; ++v) h2[v] = fmaxf(h2[v], 0.0f);
        const float4_t o = __builtin_amdgcn_mfma_f32_16x16x16f16(w3, to_half4(h2), bb3, 0, 0, 0);
        const float use = gsm[ray * 4 + 3];
        float4_t go = zero;
#pragma unroll
        for (int v = 0; v < 3; ++v) {
            if (lane < 16) {
                const float R = sigmoid_f32(o[v]);
                go[v] = use * gsm[ray * 4 + v] * R * (1.0f - R);
            }
        }
        float4_t gh2 = __builtin_amdgcn_mfma_f32_16x16x16f16(w3t, to_half4(go), zero, 0, 0, 0);
#pragma unroll
        for (int v = 0; v < 4; ++v) gh2[v] = h2[v] > 0.0f ? gh2[v] : 0.0f;
        float4_t gh1 = __builtin_amdgcn_mfma_f32_16x16x16f16(w2t, to_half4(gh2), zero, 0, 0, 0);
#pragma unroll
        for (int v = 0; v < 4; ++v) gh1[v] = h1[v] > 0.0f ? gh1[v] : 0.0f;
        const float4_t gx = __builtin_amdgcn_mfma_f32_16x16x16f16(w1t, to_half4(gh1), zero, 0, 0, 0);
        float* sr = stage + ray * kStageRow;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            sr[kSH1 + rq + v] = use * h1[v];
            sr[kSH2 + rq + v] = use * h2[v];
            sr[kSGh2 + rq + v] = gh2[v];
            sr[kSGh1 + rq + v] = gh1[v];
            if (lane < 16) sr[kSGo + v] = go[v];
        }
        // g_C = g_rgb + gx[0:3], g_V = gx[3:7]: rows 0..3 sit in lanes 0..15,
        // rows 4..7 in lanes 16..31
        const int64_t i = base + ray;
        if (i < a.n_rays && lane < 32) {
            float4* gcv = reinterpret_cast<float4*>(a.gcv) + 2 * i;
            if (lane < 16)
                gcv[0] = make_float4(gsm[ray * 4 + 0] + gx[0], gsm[ray * 4 + 1] + gx[1], gsm[ray * 4 + 2] + gx[2], gx[3]);
            else
                gcv[1] = make_float4(gx[0], gx[1], gx[2], 0.0f);
        }
    }
}

// F16: the MLP chain (forward and backward through the three layers) runs as
// v_mfma_f32_16x16x16_f16 tiles over the wavefront's 64 rays (FP16 operands,
// FP32 accumulation); the per-ray activations and gradients land in the same
// staging rows as in the FP32 path, and the weight gradients are summed by
// the same FP32 MFMA outer products.
template <bool F16>
__global__ __launch_bounds__(64 * kBwdWaves) void k_mlp_backward(BackwardArgs a) {
    __shared__ float stage[kBwdWaves][64][kStageRow];
    __shared__ _Float16 xs[F16 ? kBwdWaves : 1][64][kXRow];
    __shared__ float gsm[F16 ? kBwdWaves : 1][64][4];  // g_rgb (3), gate
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    cfloat* W = as_const(a.mlp);
    float* me = &stage[wave][lane][0];
    const float* st = &stage[wave][0][0];
    const int li = lane & 15, lk = lane >> 4;

    float4v acc1[3] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
    float4v acc2 = {0.f, 0.f, 0.f, 0.f}, acc3 = {0.f, 0.f, 0.f, 0.f};
    float db2 = 0.f, db3 = 0.f;  // lane j < 16 / < 3 holds the sum

    const int64_t stride = int64_t(gridDim.x) * kBwdWaves * 64;
    for (int64_t base = (int64_t(blockIdx.x) * kBwdWaves + wave) * 64; base < a.n_rays; base += stride) {
        const int64_t i = base + lane;
        const bool valid = i < a.n_rays;
        float C[3] = {0.f, 0.f, 0.f}, V[4] = {0.f, 0.f, 0.f, 0.f}, d[3] = {0.f, 0.f, 1.f};
        float gr[4] = {0.f, 0.f, 0.f, 0.f};
        bool gate = false;
        if (valid) {
            const int64_t r = a.ray_ids ? a.ray_ids[i] : i;
            int ci, px, py;
            locate(a, r, ci, px, py);
            int64_t o[3];
            int32_t s[3];
            ray_setup(a.cams[ci], a.grid.N, px, py, o, s, d);
            const float4 a0 = reinterpret_cast<const float4*>(a.aux)[2 * i];
            const float4 a1 = reinterpret_cast<const float4*>(a.aux)[2 * i + 1];
            C[0] = a0.x; C[1] = a0.y; C[2] = a0.z; V[0] = a0.w;
            V[1] = a1.x; V[2] = a1.y; V[3] = a1.z;
            gate = a1.w >= 0.0f;
            const float4 gg = reinterpret_cast<const float4*>(a.grad_rgba)[i];
            gr[0] = gg.x; gr[1] = gg.y; gr[2] = gg.z; gr[3] = gg.w;
        }
        const bool use = valid && gate;

        // forward, staging x, h1, h2 for the weight gradients
        float x[kMlpIn];
        encode_x(C, V, d, x);
#pragma unroll
        for (int q = 0; q < kMlpIn; ++q) me[kSX + q] = x[q];
        me[kSX + 34] = use ? 1.0f : 0.0f;
        me[kSX + 35] = 0.0f;
        if (F16) {
#pragma unroll
            for (int q = 0; q < kXPad; ++q) xs[F16 ? wave : 0][lane][q] = _Float16(q < kMlpIn ? x[q] : 0.0f);
            gsm[F16 ? wave : 0][lane][0] = gr[0];
            gsm[F16 ? wave : 0][lane][1] = gr[1];
            gsm[F16 ? wave : 0][lane][2] = gr[2];
            gsm[F16 ? wave : 0][lane][3] = use ? 1.0f : 0.0f;
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            mlp_backward_f16_wave(a, W, &xs[F16 ? wave : 0][0][0], &gsm[F16 ? wave : 0][0][0],
                                  &stage[wave][0][0], base, lane);
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            if (lane < kMlpH) {
                float t = 0.f;
                for (int r = 0; r < 64; ++r) t += st[r * kStageRow + kSGh2 + lane];
                db2 += t;
            }
            if (lane < kMlpOut) {
                float t = 0.f;
                for (int r = 0; r < 64; ++r) t += st[r * kStageRow + kSGo + lane];
                db3 += t;
            }
        } else {
        float h2[kMlpH];
#pragma unroll
        for (int k = 0; k < kMlpH; ++k) h2[k] = W[kOffB2 + k];
#pragma nounroll
        for (int j = 0; j < kMlpH; ++j) {
            float t = W[kOffB1 + j];
#pragma unroll
            for (int q = 0; q < kMlpIn; ++q) t = fmaf(W[kOffW1 + j * kMlpIn + q], x[q], t);
            const float h1j = fmaxf(t, 0.0f);
            me[kSH1 + j] = use ? h1j : 0.0f;
#pragma unroll
            for (int k = 0; k < kMlpH; ++k) h2[k] = fmaf(W[kOffW2 + k * kMlpH + j], h1j, h2[k]);
        }
#pragma unroll
        for (int k = 0; k < kMlpH; ++k) {
            h2[k] = fmaxf(h2[k], 0.0f);
            me[kSH2 + k] = use ? h2[k] : 0.0f;
        }
        float go[kMlpOut];
#pragma unroll
        for (int j = 0; j < kMlpOut; ++j) {
            float t = W[kOffB3 + j];
#pragma unroll
            for (int q = 0; q < kMlpH; ++q) t = fmaf(W[kOffW3 + j * kMlpH + q], h2[q], t);
            const float R = sigmoid_f32(t);
            go[j] = use ? gr[j] * R * (1.0f - R) : 0.0f;
            me[kSGo + j] = go[j];
        }
        me[kSGo + 3] = 0.0f;
        // backward through layers 3 and 2 (the ReLU masks come from h2, h1)
#pragma unroll
        for (int q = 0; q < kMlpH; ++q) {
            float t = 0.f;
#pragma unroll
            for (int j = 0; j < kMlpOut; ++j) t = fmaf(W[kOffW3 + j * kMlpH + q], go[j], t);
            h2[q] = h2[q] > 0.0f ? t : 0.0f;  // h2 now holds gh2
            me[kSGh2 + q] = h2[q];
        }
        float gx[7] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma nounroll
        for (int j = 0; j < kMlpH; ++j) {
            float t = 0.f;
#pragma unroll
            for (int k = 0; k < kMlpH; ++k) t = fmaf(W[kOffW2 + k * kMlpH + j], h2[k], t);
            const float gh1j = me[kSH1 + j] > 0.0f ? t : 0.0f;
            me[kSGh1 + j] = gh1j;
#pragma unroll
            for (int q = 0; q < 7; ++q) gx[q] = fmaf(W[kOffW1 + j * kMlpIn + q], gh1j, gx[q]);
        }
        if (valid) {
            float4* gcv = reinterpret_cast<float4*>(a.gcv) + 2 * i;
            gcv[0] = make_float4(gr[0] + gx[0], gr[1] + gx[1], gr[2] + gx[2], gx[3]);
            gcv[1] = make_float4(gx[4], gx[5], gx[6], 0.0f);
        }
#pragma unroll
        for (int q = 0; q < kMlpH; ++q) {
            const float sq = wave_sum(h2[q]);
            if (lane == q) db2 += sq;
        }
#pragma unroll
        for (int q = 0; q < kMlpOut; ++q) {
            const float sq = wave_sum(go[q]);
            if (lane == q) db3 += sq;
        }
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        // dW = sum_r gA_r (x) act_r as 16x16x4 FP32 MFMAs: A = gradient rows
        // (16 x 4 rays), B = activations (4 rays x 16); D lane l holds row
        // 4(l/16) + v, column l % 16.
#pragma unroll
        for (int kk = 0; kk < 16; ++kk) {
            const float* rr = st + (4 * kk + lk) * kStageRow;
            const float a1v = rr[kSGh1 + li];
#pragma unroll
            for (int nt = 0; nt < 3; ++nt) {
                const int col = 16 * nt + li;
                const float bv = col < 36 ? rr[kSX + col] : 0.0f;
                acc1[nt] = __builtin_amdgcn_mfma_f32_16x16x4f32(a1v, bv, acc1[nt], 0, 0, 0);
            }
            acc2 = __builtin_amdgcn_mfma_f32_16x16x4f32(rr[kSGh2 + li], rr[kSH1 + li], acc2, 0, 0, 0);
            acc3 = __builtin_amdgcn_mfma_f32_16x16x4f32(li < 4 ? rr[kSGo + li] : 0.0f, rr[kSH2 + li], acc3, 0, 0, 0);
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }

    // this wavefront's partial MLP gradient, in parameter order
    float* out = a.g_mlp_partial + (int64_t(blockIdx.x) * kBwdWaves + wave) * kMlpParams;
    const int lr = 4 * (lane >> 4);
#pragma unroll
    for (int nt = 0; nt < 3; ++nt) {
        const int col = 16 * nt + li;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int row = lr + v;
            if (col < kMlpIn) out[kOffW1 + row * kMlpIn + col] = acc1[nt][v];
            else if (col == kMlpIn) out[kOffB1 + row] = acc1[nt][v];
        }
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        out[kOffW2 + (lr + v) * kMlpH + li] = acc2[v];
        if (lr + v < kMlpOut) out[kOffW3 + (lr + v) * kMlpH + li] = acc3[v];
    }
    if (lane < kMlpH) out[kOffB2 + lane] = db2;
    if (lane < kMlpOut) out[kOffB3 + lane] = db3;
}

// --------------------------------------------------------------- K2: march

// Canonical gradient slot of padded corner voxel (vx, vy, vz) (local
// coordinates in [-1, B]) of the block with atlas id `id` at block
// coordinates b (x | y << 8 | z << 16).  Voxels outside the grid or in empty
// blocks are structural zeros and have no slot (-1).  I: int32_t where all
// indices fit it (a 64-bit multiply costs several times a shift).
template <typename I>
__device__ __forceinline__ I canonical_voxel(const GridArgs& g, int32_t id, int32_t b, int vx, int vy, int vz,
                                             int32_t& nb_lin, int32_t& nb_id) {
    const int B = g.B;
    int32_t tid = id;
    if (tid < 0 || tid >= g.n_blocks) return -1;
    if ((vx | vy | vz) < 0 || max(max(vx, vy), vz) >= B) {
        const int nx = (b & 0xff) + (vx < 0 ? -1 : (vx >= B ? 1 : 0));
        const int ny = ((b >> 8) & 0xff) + (vy < 0 ? -1 : (vy >= B ? 1 : 0));
        const int nz = (b >> 16) + (vz < 0 ? -1 : (vz >= B ? 1 : 0));
        if ((nx | ny | nz) < 0 || max(max(nx, ny), nz) >= g.G) return -1;
        // the last neighbour looked up (a ray runs along a face for a while)
        const int32_t nlin = mul_s24(mul_s24(nz, g.G) + ny, g.G) + nx;
        if (nlin != nb_lin) {
            nb_lin = nlin;
            nb_id = g.ind[nlin];
        }
        tid = nb_id;
        if (tid < 0 || tid >= g.n_blocks) return -1;
        vx &= B - 1;
        vy &= B - 1;
        vz &= B - 1;
    }
    return (((((I(tid) << g.logB) | vz) << g.logB) | vy) << g.logB) | vx;
}

// Gradient aggregation in LDS.  Neighbouring rays share most of the voxels
// they touch, so each voxel's eight gradient values (density, RGB, features)
// are first summed in an open-addressed table of kAggSlots entries, one per
// workgroup, and reach device memory with one set of atomics per table flush
// instead of one per ray.  Keys are canonical voxel indices (< 2^31; the
// launch takes the log otherwise).
//
// The colour and feature sums are kept in 32-bit fixed point: on gfx950 an
// LDS float add (ds_add_f32) retires about one lane every three cycles, an
// LDS integer add (ds_add_u32) more than forty times faster.  A ray hands a
// voxel its colour gradient A g_C with A = sum_k w_c(k) w_k, and the A of all
// of a ray's hand-overs add up to at most sum_k w_k <= 1, so with M = max over
// the rays of the tile, or of 64 list entries, of |g_C|, |g_V| all that one ray
// hands to one voxel is at most M and a table entry (32 rays between flushes)
// at most 32 M.  Values are scaled by 2^S, the largest power of two with M 2^S < 2^24,
// and rounded to integers: an entry stays below 2^29 (plus its rounding),
// and each hand-over carries a rounding error of at most 2^-24 M.  The
// density sums, whose size depends on the grid values, stay in float.
constexpr int kAdjWaves = 4;  // wavefronts per workgroup: 32 rays, 8 lanes each
constexpr int kAggLog = 9;
constexpr int kAggSlots = 1 << kAggLog;
constexpr int kAggProbes = 16;
constexpr int kAggWords = kAggSlots * 9;  // keys, 8 value planes
// The workgroup looks at the table every kAggTrips trips of its rays and
// flushes it when it holds more than kAggFlushAt keys; what its rays add in
// four trips (up to 32 samples each) mostly fits above that, and a key that
// finds no free slot within kAggProbes probes goes to device memory directly.
constexpr int kAggFlushAt = kAggSlots * 9 / 16;
constexpr int kAggTrips = 4;

// The log of a wavefront whose rays share few voxels, in 16-byte entries.
constexpr int kLogEntries = 320;

struct AggTable {
    int32_t* key;  // [kAggSlots], -1 = free
    float* val;    // [8][kAggSlots]: plane 0 float (density), planes 1..7 int32 fixed point
    float q;       // 2^S: fixed-point scale of the colour and feature planes
    float dq;      // 2^-S
};

// Fixed-point scale for rays whose largest |g_C|, |g_V| is m (m >= 0, the
// same value in every lane): 2^S with m 2^S < 2^24 <= 2 m 2^S.
__device__ __forceinline__ void agg_scale(AggTable& t, float m) {
    int e = 0;
    (void)__builtin_frexpf(m, &e);  // 2^(e-1) <= m < 2^e
    int sh = 24 - e;
    sh = m > 0.0f ? (sh < 126 ? (sh > -126 ? sh : -126) : 126) : 0;
    t.q = __builtin_ldexpf(1.0f, sh);
    t.dq = __builtin_ldexpf(1.0f, -sh);
}

// The device address of channel c (0 density, 1..3 RGB, 4..7 features) of
// voxel vi.
__device__ __forceinline__ float* grad_channel(const BackwardArgs& a, int64_t vi, int c) {
    if (a.grad_packed) return a.grad_dens + 8 * vi + c;
    return c == 0 ? a.grad_dens + vi : (c < 4 ? a.grad_rgb + 3 * vi + (c - 1) : a.grad_feat + 4 * vi + (c - 4));
}

// The table slot of `key` (lanes may diverge), claimed if it has none; -1
// when no slot was found within kAggProbes probes.  `fresh` counts the lane's
// new keys.
__device__ __forceinline__ int agg_slot(const AggTable& t, int32_t key, int& fresh) {
    uint32_t sl = (uint32_t(key) * 2654435761u) >> (32 - kAggLog);
#pragma nounroll
    for (int pr = 0; pr < kAggProbes; ++pr) {
        // one round trip per probe: the compare-and-swap claims a free slot
        // and otherwise returns the key that holds it
        const int32_t k = atomicCAS(t.key + sl, -1, key);
        fresh += k == -1 ? 1 : 0;
        if (k == -1 || k == key) return int(sl);
        sl = (sl + 1) & (kAggSlots - 1);
    }
    return -1;
}

// The whole workgroup, between barriers: every used entry goes to device
// memory, the table is cleared.  gfx950 serves a wavefront's float atomics
// per 64-byte line (measured: about 21 G lines per second whether a line
// carries one lane's add or sixteen), so the lanes are laid across the
// entries' channels, not the entries: lane l takes entry l / 4 of a group of
// 16 and within it channels l % 4 and l % 4 + 4, so that one instruction adds
// an entry's density and colour (two lines) and the next its four features
// (one line), where one lane per entry would touch seven lines.  With packed
// gradients an entry's eight sums share one line: eight lanes per entry (four
// without features), one instruction per group.
template <bool FEAT>
__device__ __forceinline__ void agg_flush(const BackwardArgs& a, const AggTable& t) {
    int32_t* iv = reinterpret_cast<int32_t*>(t.val);
    auto take = [&](int sl, int c) {
        float v;
        if (c == 0) {
            v = t.val[sl];
            t.val[sl] = 0.0f;
        } else {
            v = float(iv[c * kAggSlots + sl]) * t.dq;
            iv[c * kAggSlots + sl] = 0;
        }
        return v;
    };
    // the lanes of an entry sit in one wavefront and read its key before any
    // of them frees it
    const int kC = a.grad_packed && FEAT ? 8 : 4;  // lanes per entry
    const int c = threadIdx.x & (kC - 1);
    for (int sl = threadIdx.x / kC; sl < kAggSlots; sl += blockDim.x / kC) {
        const int32_t key = t.key[sl];
        if (key >= 0) {
            const float v0 = take(sl, c);
            if (v0 != 0.0f) unsafeAtomicAdd(grad_channel(a, key, c), v0);
            if (FEAT && kC == 4) {
                const float v1 = take(sl, c + 4);
                if (v1 != 0.0f) unsafeAtomicAdd(grad_channel(a, key, c + 4), v1);
            }
            if (c == 0) t.key[sl] = -1;
        }
    }
}

template <int CTRL>
__device__ __forceinline__ int32_t dpp(int32_t v) {
    return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xf, 0xf, true);
}
template <int CTRL>
__device__ __forceinline__ float dpp(float v) {
    return __int_as_float(dpp<CTRL>(__float_as_int(v)));
}

// The 8 lanes of a ray.  Lane l holds corner (x, y, z) of the ray's cell with
// z = l / 4 and x, y the low bits of l, flipped where z = 1, so that the
// neighbour across each axis is one DPP step away: l ^ 1 in x, l ^ 2 in y and
// l ^ 7, the mirror of 8 lanes, in z.
constexpr int kFlipX = 0xB1, kFlipY = 0x4E, kFlipZ = 0x141;  // quad_perm 1,0,3,2; 2,3,0,1; row_half_mirror
// A value that lane a of every quad holds for axis a, of axis x, y, z.
constexpr int kAxisX = 0x00, kAxisY = 0x55, kAxisZ = 0xAA;

__device__ __forceinline__ float corner_sum(float v) {
    v += dpp<kFlipX>(v);
    v += dpp<kFlipY>(v);
    return v + dpp<kFlipZ>(v);
}

__device__ __forceinline__ uint32_t ray_bits(bool p, int lane) {
    return uint32_t(__ballot(p) >> (lane & ~7)) & 0xFFu;
}

// FlatWalk with its per-axis state dealt to the lanes: in every quad lane
// q % 4 = 0, 1, 2 holds axis x, y, z (lane 3 a copy of z), the rest is the
// same in all 8.  A third of the registers and of the work of a macroblock
// entry, and the registers are what bounds the number of resident wavefronts.
struct QuadWalk {
    int32_t kc, F, Q, s, q;  // own axis
    int32_t stride;          // change of lin across a face of the own axis (0 in lane 3)
    int32_t kend, k, lin, left, r, smax;
    float inv_smax;
    const uint8_t* __restrict__ dist;

    __device__ __forceinline__ bool init(const GridArgs& g, const int64_t o[3], const int32_t s3[3], int l) {
        FlatWalk w;
        if (!w.init(g, o, s3)) return false;
        const int a = l & 3;
        kc = a == 0 ? w.kc[0] : (a == 1 ? w.kc[1] : w.kc[2]);
        F = a == 0 ? w.F[0] : (a == 1 ? w.F[1] : w.F[2]);
        Q = a == 0 ? w.Q[0] : (a == 1 ? w.Q[1] : w.Q[2]);
        s = a == 0 ? s3[0] : (a == 1 ? s3[1] : s3[2]);
        stride = a == 0 ? 1 : (a == 1 ? g.G : (a == 2 ? g.G * g.G : 0));
        stride = s > 0 ? stride : -stride;
        q = 0;
        kend = w.kend;
        k = 0;
        lin = w.lin;
        left = 0;
        r = -1;
        smax = w.smax;
        inv_smax = w.inv_smax;
        dist = g.rec;
        return true;
    }

    // As FlatWalk::enter.
    __device__ __forceinline__ bool enter(const GridArgs& g, const uint2* occ) {
        const int bs = 16 + g.logB;
        const int32_t W = int32_t(1) << bs;
        const uint32_t G3 = uint32_t(g.G) * uint32_t(g.G) * uint32_t(g.G);
        if (k > kend || uint32_t(lin) >= G3) return false;
        int32_t kn = min(kc, dpp<kFlipX>(kc));
        kn = min(kn, dpp<kFlipY>(kn));
        kn = min(kn, kend + 1);
        r = block_rank(occ, lin, g.n_blocks);
        if (r >= 0) {
            // (records are multiples of 256 bytes)
            dist = g.rec + (uint64_t(uint32_t(r) * uint32_t(g.rec_stride >> 8)) << 8);
            q = (s > 0 ? W - F : F - 1) + mul_s24(k, s) + 32768;
            left = kn - k;
        }
        int32_t step = 0;
        if (kc == kn) {
            step = stride;
            F += W;
            const int32_t c = kc + Q;
            const int32_t cs = mul_s24(c, s);  // c |s| = sign(s) c s
            kc = (s > 0 ? cs : -cs) >= F ? c : c + 1;
        }
        step += dpp<kFlipX>(step);
        lin += step + dpp<kFlipY>(step);
        k = kn;
        return true;
    }
};

// One ray per 8 lanes.  A trip of the walk looks at the ray's next 8 lattice
// samples, one per lane (its distance byte), and then takes the active ones
// in order, all lanes together, lane by corner: each loads its corner's
// voxel, the two sums a sample needs (density and g . value) are three DPP
// additions each, and each lane keeps its corner's (A, D) and hands it over
// by itself.  One ray per lane, as this was before, paid for every sample
// with eight guarded hand-over passes and 256 bytes of loads per lane, at two
// wavefronts per SIMD (197 to 256 registers), and a list of 65,536 rays
// needed a separate walk to keep 64 rays of unequal length apart.
//   eight 800x800 views, 512^3, FP32 network   23.7 -> 18.1 ms
//   16,384 rays in 8x8 patches, 512^3           1.95 -> 0.41 ms
//   65,536 scattered rays, 1024^3, packed       2.35 -> 1.2 ms
// Bound by instruction issue with the table (VALUs 82% busy, half the lanes
// at work: about 270 instructions per sample of 8 rays), for scattered rays
// by latency and by rays of unequal length side by side.  Registers: 96 (five
// wavefronts per SIMD) with the table, where six or three cost 9 and 40%;
// scattered rays want the next sample's voxels in flight, which takes 118
// (20% slower squeezed into 96).
// Without a ray list the workgroups walk halves of the cameras'
// tile_w x tile_h pixel tiles, with one 32 consecutive list entries.  AGG:
// gradients go through the workgroup's LDS table, else through the
// wavefront's log.
template <bool FEAT, bool AGG>
__global__ __launch_bounds__(64 * kAdjWaves) __attribute__((amdgpu_waves_per_eu(AGG ? 5 : 4))) void k_adjoint(BackwardArgs a) {
    constexpr int kWaves = kAdjWaves;
    extern __shared__ uint2 s_occ[];
    __shared__ float s_max;
    __shared__ int32_t s_fresh[3], s_live[3];
    __shared__ float s_gch[AGG ? 1 : kWaves][8][8];  // the rays' gradients by channel
    const GridArgs& g = a.grid;
    for (int w = threadIdx.x; w < g.n_words; w += blockDim.x) s_occ[w] = g.occ[w];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int l = lane & 7;
    const int cz = l >> 2, cx = (l & 1) ^ cz, cy = ((l >> 1) & 1) ^ cz;
    AggTable tab = {nullptr, nullptr, 0.0f, 0.0f};
    if (AGG) {
        tab.key = reinterpret_cast<int32_t*>(s_occ + g.n_words);
        tab.val = reinterpret_cast<float*>(tab.key + kAggSlots);
        for (int sl = threadIdx.x; sl < kAggSlots; sl += blockDim.x) {
            tab.key[sl] = -1;
#pragma unroll
            for (int c = 0; c < 8; ++c) tab.val[c * kAggSlots + sl] = 0.0f;
        }
        if (threadIdx.x < 3) s_fresh[threadIdx.x] = s_live[threadIdx.x] = 0;
    }
    int4* log = reinterpret_cast<int4*>(s_occ + ((g.n_words + 1) & ~1)) + wave * kLogEntries;

    // Rays come in sets of 64 (a tile, or 64 list entries), a workgroup takes
    // half of one.  Ray idx of the set: list position i (indexes aux,
    // grad_rgba, gcv), pixel (px, py) of camera ci.
    // (of a view's tiles each XCD takes runs of 32 workgroups, as the render does)
    const uint32_t u = a.ray_ids ? blockIdx.x : xcd_grouped<32>(blockIdx.x, gridDim.x);
    const int64_t set = (a.first_group + u) >> 1;
    const int half = int(u & 1);
    auto ray_of = [&](int idx, int64_t& i, int& ci, int& px, int& py) {
        if (a.ray_ids) {
            i = set * 64 + idx;
            if (i >= a.n_rays) return false;
            locate(a, a.ray_ids[i], ci, px, py);
            return true;
        }
        ci = find_camera_by_tile(a.cams, a.n_cams, set);
        const DevCamera& c = a.cams[ci];
        const int64_t tl = set - c.tile_offset;
        px = int(tl % c.tiles_x) * a.tile_w + idx % a.tile_w;
        py = int(tl / c.tiles_x) * a.tile_h + idx / a.tile_w;
        i = c.ray_offset + int64_t(py) * c.W + px;
        return px < c.W && py < c.H;
    };
    if (AGG && threadIdx.x < 64) {  // the table's scale, from the whole set
        int64_t i;
        int ci, px, py;
        float m = 0.0f;
        if (ray_of(threadIdx.x, i, ci, px, py) && a.aux[8 * i + 7] >= 0.0f) {
            const float* v = FEAT ? a.gcv + 8 * i : a.grad_rgba + 4 * i;
#pragma unroll
            for (int c = 0; c < (FEAT ? 7 : 3); ++c) m = fmaxf(m, fabsf(v[c]));
        }
        m = wave_max(m);
        if (threadIdx.x == 0) s_max = m;
    }
    int64_t i = 0;
    int ci = 0, px = 0, py = 0;
    bool live = ray_of((half * kWaves + wave) * 8 + (lane >> 3), i, ci, px, py);
    QuadWalk w;
    if (live) {
        int64_t o[3];
        int32_t s[3];
        float d[3];
        ray_setup(a.cams[ci], g.N, px, py, o, s, d);
        live = w.init(g, o, s, l);
    }
    // its output gradient and what the forward saved
    float4 a0 = make_float4(0.f, 0.f, 0.f, 0.f), a1 = make_float4(0.f, 0.f, 0.f, -1.f);
    float4 gg = make_float4(0.f, 0.f, 0.f, 0.f);
    if (live) {
        a1 = reinterpret_cast<const float4*>(a.aux)[2 * i + 1];
        live = a1.w >= 0.0f;  // nothing was composited: no grid gradient
    }
    float gC[3] = {0.f, 0.f, 0.f}, gV[4] = {0.f, 0.f, 0.f, 0.f};
    if (live) {
        a0 = reinterpret_cast<const float4*>(a.aux)[2 * i];
        gg = reinterpret_cast<const float4*>(a.grad_rgba)[i];
        gC[0] = gg.x; gC[1] = gg.y; gC[2] = gg.z;
        if (FEAT) {
            const float4 c0 = reinterpret_cast<const float4*>(a.gcv)[2 * i];
            const float4 c1 = reinterpret_cast<const float4*>(a.gcv)[2 * i + 1];
            gC[0] = c0.x; gC[1] = c0.y; gC[2] = c0.z;
            gV[0] = c0.w; gV[1] = c1.x; gV[2] = c1.y; gV[3] = c1.z;
        }
    }
    const float E = gC[0] * a0.x + gC[1] * a0.y + gC[2] * a0.z +
                    (gV[0] * a0.w + gV[1] * a1.x + gV[2] * a1.y + gV[3] * a1.z);
    const float gTN = gg.x * a.opts.bg[0] + gg.y * a.opts.bg[1] + gg.z * a.opts.bg[2] - gg.w;
    const float tail = a1.w * gTN;  // T_N dL/dT_N
    const float inv_g = 1.0f / float(g.G);
    const float delta = 1.0f / float(g.N), kx = g.sigma_scale * delta;
    // Where the forward ended the ray early, at the sample that left it its
    // T_N < t_stop, the re-march ends there too: T is recomputed here with
    // other roundings (a few 2^-22), so it ends when T has come down to T_N,
    // give or take 2^-16, or is that clearly past the threshold.
    const float t_end = a.opts.early_stop && a1.w < a.opts.t_stop
                            ? fmaxf(a1.w * (1.0f + 0x1p-16f), a.opts.t_stop * (1.0f - 0x1p-16f))
                            : -1.0f;
    // direct atomics: this lane's channel and its gradient
    float gch = 0.0f;
#pragma unroll
    for (int c = 0; c < 3; ++c) gch = l == 1 + c ? gC[c] : gch;
#pragma unroll
    for (int c = 0; c < 4; ++c) gch = l == 4 + c ? gV[c] : gch;
    if (!AGG) s_gch[wave][lane >> 3][l] = gch;
    __syncthreads();
    if (AGG) agg_scale(tab, s_max);

    const uint32_t nb = uint32_t(g.Bp), nbb = nb * nb;
    const uint32_t nc = uint32_t(g.Bc), ncc = nc * nc;
    const uint32_t corner = (uint32_t(cz) * nbb + uint32_t(cy) * nb + uint32_t(cx)) * 32u;
    // weight of the corner on an axis: f = |0 - f| or 1 - f
    const float ox = cx ? 0.0f : 1.0f, oy = cy ? 0.0f : 1.0f, oz = cz ? 0.0f : 1.0f;

    float T = 1.0f, rest = E + tail;  // rest: E - P_k + T_N dL/dT_N
    float A = 0.0f, D = 0.0f;         // this corner's sums
    int32_t wc = 0;                      // the window's cell, own axis
    int32_t wrank = -1, wid = 0, wb = 0;  // its block's record, atlas id, coordinates (8 bits each)
    int32_t nb_lin = -1, nb_id = -1;
    int fresh = 0;
    int32_t* iv = reinterpret_cast<int32_t*>(tab.val);

    int4 out = make_int4(0, -1, 0, 0);  // without the table: what this lane hands over, out.y < 0: nothing

    // Hands this corner's sums over where `leave` is set (the same decision
    // rule in all lanes of the ray, not the same answer).
    auto hand_over = [&](bool leave) {
        const int vx = dpp<kAxisX>(wc) + cx - 1, vy = dpp<kAxisY>(wc) + cy - 1, vz = dpp<kAxisZ>(wc) + cz - 1;
        using Index = typename std::conditional<AGG, int32_t, int64_t>::type;  // the table's keys are int32
        Index vi = -1;
        if (leave && (A != 0.0f || D != 0.0f))
            vi = canonical_voxel<Index>(g, wid, wb, vx, vy, vz, nb_lin, nb_id);
        const float Ds = g.sigma_scale * D;
        if (AGG && vi >= 0) {
            const int sl = agg_slot(tab, vi, fresh);
            if (sl >= 0) {
                vi = -1;
                atomicAdd(tab.val + sl, Ds);
                const float Aq = A * tab.q;  // a power of two: exact, so the products round as A g would
#pragma unroll
                for (int c = 0; c < 3; ++c)
                    atomicAdd(iv + (1 + c) * kAggSlots + sl, int32_t(__builtin_rintf(Aq * gC[c])));
                if (FEAT) {
#pragma unroll
                    for (int c = 0; c < 4; ++c)
                        atomicAdd(iv + (4 + c) * kAggSlots + sl, int32_t(__builtin_rintf(Aq * gV[c])));
                }
            }
        }
        if (AGG) {  // no slot free: the ray's 8 lanes add a corner's 8 channels
            for (uint32_t m = ray_bits(vi >= 0, lane); m != 0; m &= m - 1) {
                const int from = (lane & ~7) | __builtin_ctz(m);
                const Index v = __shfl(vi, from);
                const float dv = __shfl(Ds, from), av = __shfl(A, from);
                const float x = l == 0 ? dv : av * gch;
                if (x != 0.0f) unsafeAtomicAdd(grad_channel(a, v, l), x);
            }
        } else {
            out = make_int4(int32_t(uint32_t(uint64_t(vi))), int32_t(vi >> 32), __float_as_int(A), __float_as_int(Ds));
        }
    };

    // Without the table: what the lanes hand over in a step goes, at the next
    // point where all 64 are together, to the wavefront's log (voxel, ray, A,
    // density sum), each to the place a ballot gives it, so the fill count is
    // the same in every lane.  A full log goes to device memory, 8 entries to
    // an instruction, the lanes of one across the voxel's channels.  Added
    // straight away, every atomic would stand in front of the next step's
    // loads, which wait for it (vector memory retires in order).
    int n_log = 0;
    auto log_flush = [&]() {
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
        for (int e = lane >> 3; e < n_log; e += 8) {
            const int4 h = log[e];
            const int64_t v = int64_t(uint64_t(uint32_t(h.x)) | (uint64_t(uint32_t(h.y & 0xffffff)) << 32));
            const float x = l == 0 ? __int_as_float(h.w) : __int_as_float(h.z) * s_gch[wave][h.y >> 24][l];
            if (x != 0.0f) unsafeAtomicAdd(grad_channel(a, v, l), x);
        }
        n_log = 0;
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
    };
    auto log_append = [&]() {
        const bool want = out.y >= 0;
        const uint64_t m = __ballot(want);
        if (m == 0) return;  // wave-uniform
        if (n_log > kLogEntries - 64) log_flush();
        if (want) {
            out.y |= (lane >> 3) << 24;
            log[n_log + int(__builtin_amdgcn_mbcnt_hi(uint32_t(m >> 32), __builtin_amdgcn_mbcnt_lo(uint32_t(m), 0u)))] =
                out;
        }
        n_log += __builtin_popcountll(m);
        out.y = -1;
    };

    int in_table = 0, phase = 0;  // AGG: keys in the table, the same in every lane of the workgroup
    for (int trip = 0;; ++trip) {
        if (AGG) {
            if (trip % kAggTrips == 0) {
                // Slot `phase` collects this phase's counts before the barrier
                // and is read after it; the slot of the phase after next was
                // last read before this barrier, and is cleared for it.
                int f = fresh;
#pragma unroll
                for (int sh = 32; sh >= 1; sh >>= 1) f += __shfl_xor(f, sh);
                const bool some = __any(live);
                if (lane == 0 && f != 0) atomicAdd(&s_fresh[phase], f);
                if (lane == 0 && some) s_live[phase] = 1;
                fresh = 0;
                __syncthreads();
                in_table += s_fresh[phase];
                const bool on = s_live[phase] != 0;
                const int clear = phase == 0 ? 2 : phase - 1;
                if (threadIdx.x == 0) s_fresh[clear] = s_live[clear] = 0;
                phase = phase == 2 ? 0 : phase + 1;
                if (!on || in_table > kAggFlushAt) {
                    if (!on) {  // the last windows
                        hand_over(wrank >= 0);
                        __syncthreads();
                    }
                    agg_flush<FEAT>(a, tab);
                    if (!on) break;
                    in_table = 0;
                    __syncthreads();
                }
            }
        } else if (!__any(live)) {
            break;
        }
        uint32_t todo = 0;
        int32_t reach = 0;
        if (live) {
            while (live && w.left <= 0) live = w.enter(g, s_occ);
        }
        if (live) {
            bool act = false;
            const int32_t p[3] = {(dpp<kAxisX>(w.q) + mul_s24(l, dpp<kAxisX>(w.s))) >> 16,
                                  (dpp<kAxisY>(w.q) + mul_s24(l, dpp<kAxisY>(w.s))) >> 16,
                                  (dpp<kAxisZ>(w.q) + mul_s24(l, dpp<kAxisZ>(w.s))) >> 16};
            if (l < w.left) {
                const int32_t db = w.dist[cell_index(p, nc, ncc)];
                act = db == 0;
                reach = l + (act ? 1 : skip_steps(db, w.smax, w.inv_smax));
            }
            todo = ray_bits(act, lane);
            reach = max(reach, dpp<kFlipX>(reach));
            reach = max(reach, dpp<kFlipY>(reach));
            reach = max(reach, dpp<kFlipZ>(reach));
            reach = min(reach, w.left);
        }
        // Reads this corner's voxel of the ray's next active sample.
        auto fetch = [&](int32_t& own, float4& va, float4& vb) {
            own = w.q + mul_s24(__builtin_ctz(todo), w.s);
            todo &= todo - 1;
            const int32_t p[3] = {dpp<kAxisX>(own) >> 16, dpp<kAxisY>(own) >> 16, dpp<kAxisZ>(own) >> 16};
            const uint8_t* at = w.dist + g.dist_bytes + (uint64_t(cell_index(p, nb, nbb)) * 32u + corner);
            va = reinterpret_cast<const float4*>(at)[0];
            if (FEAT) vb = reinterpret_cast<const float4*>(at)[1];
        };
        auto take = [&](int32_t own, const float4& va, const float4& vb) {
            const int32_t q[3] = {dpp<kAxisX>(own), dpp<kAxisY>(own), dpp<kAxisZ>(own)};
            const float fx = float(q[0] & 0xFFFF) * (1.0f / 65536.0f);
            const float fy = float(q[1] & 0xFFFF) * (1.0f / 65536.0f);
            const float fz = float(q[2] & 0xFFFF) * (1.0f / 65536.0f);
            const float wt = (fabsf(ox - fx) * fabsf(oy - fy)) * fabsf(oz - fz);
            // The exact active test: some corner of non-zero weight (every
            // product of non-zero fractions is at least 2^-48) has non-zero
            // density; or, the viewer's gate, the nearest corner has.
            bool dense = va.x != 0.0f && wt != 0.0f;
            if (a.opts.nn_gate)
                dense = va.x != 0.0f && cx == ((q[0] >> 15) & 1) && cy == ((q[1] >> 15) & 1) && cz == ((q[2] >> 15) & 1);
            float ev = gC[0] * va.y + gC[1] * va.z + gC[2] * va.w;
            if (FEAT) ev += gV[0] * vb.x + gV[1] * vb.y + gV[2] * vb.z + gV[3] * vb.w;
            const float sigma = corner_sum(wt * va.x);
            const float ek = corner_sum(wt * ev);
            if (ray_bits(dense, lane) == 0) return;
            const float e = __expf(-sigma * kx);
            const float ws = T * (1.0f - e);
            rest -= ws * ek;
            T *= e;
            const float gsig = delta * (T * ek - rest);
            // Slide the corner window to this sample's cell: corners on a
            // trailing face (or all of them after a jump) are handed over, the
            // survivors move to their new lane.
            const int32_t move = (own >> 16) - wc;
            const int32_t dd[3] = {dpp<kAxisX>(move), dpp<kAxisY>(move), dpp<kAxisZ>(move)};
            const bool jump = wrank != w.r || ray_bits(abs(move) > 1, lane) != 0;
            // the corner leaves on an axis the window moves along if it is on the trailing side
            const bool lx = dd[0] != 0 && (dd[0] > 0) == (cx == 0);
            const bool ly = dd[1] != 0 && (dd[1] > 0) == (cy == 0);
            const bool lz = dd[2] != 0 && (dd[2] > 0) == (cz == 0);
            hand_over(jump ? wrank >= 0 : lx || ly || lz);
            if (jump) {
                A = D = 0.0f;
                wrank = w.r;
                wid = g.rank_id[w.r];
                const int32_t lin = g.rank_lin[w.r];
                // lin < 2^18: the rounded product is never a half away from the quotient
                const int32_t yz = int32_t((float(lin) + 0.5f) * inv_g), z = int32_t((float(yz) + 0.5f) * inv_g);
                wb = (lin - mul_s24(yz, g.G)) | (yz - mul_s24(z, g.G)) << 8 | z << 16;
            } else {
                // a trailing corner takes its leading neighbour's sums, which start anew
                float An = dpp<kFlipX>(A), Dn = dpp<kFlipX>(D);
                A = dd[0] == 0 ? A : (lx ? An : 0.0f);
                D = dd[0] == 0 ? D : (lx ? Dn : 0.0f);
                An = dpp<kFlipY>(A), Dn = dpp<kFlipY>(D);
                A = dd[1] == 0 ? A : (ly ? An : 0.0f);
                D = dd[1] == 0 ? D : (ly ? Dn : 0.0f);
                An = dpp<kFlipZ>(A), Dn = dpp<kFlipZ>(D);
                A = dd[2] == 0 ? A : (lz ? An : 0.0f);
                D = dd[2] == 0 ? D : (lz ? Dn : 0.0f);
            }
            wc += move;
            A = fmaf(wt, ws, A);
            D = fmaf(wt, gsig, D);
            if (T <= t_end) live = false;
        };
        int32_t own = 0;
        float4 va = make_float4(0.f, 0.f, 0.f, 0.f), vb = va;
        if (AGG) {
            while (todo != 0) {
                fetch(own, va, vb);
                take(own, va, vb);
                if (!live) todo = 0;
            }
        } else {
            // the next sample's voxels are read before the current one's work
            bool more = todo != 0;
            if (more) fetch(own, va, vb);
            while (__any(more)) {
                if (more) {
                    const int32_t o1 = own;
                    const float4 a1v = va, b1v = vb;
                    more = todo != 0;
                    if (more) fetch(own, va, vb);
                    take(o1, a1v, b1v);
                    if (!live) {
                        todo = 0;
                        more = false;
                    }
                }
                log_append();
            }
        }
        if (live) {
            w.left -= reach;
            w.q += mul_s24(reach, w.s);
        }
    }
    if (!AGG) {
        hand_over(wrank >= 0);
        log_append();
        log_flush();
    }
}

// Column sums of the [rows][883] partial-gradient matrix into out (which
// holds zeros): each workgroup takes 64 columns x kReduceRows rows, four
// row phases of 64 threads, combines them in LDS and adds its sum to out.
constexpr int kReduceRows = 256;

__global__ __launch_bounds__(256) void k_reduce_rows(const float* __restrict__ partial, int rows,
                                                     float* __restrict__ out) {
    __shared__ float part[4][64];
    const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
    const int col = blockIdx.x * 64 + tx;
    const int r0 = blockIdx.y * kReduceRows;
    const int r1 = min(rows, r0 + kReduceRows);
    float acc = 0.f;
    if (col < kMlpParams)
        for (int r = r0 + ty; r < r1; r += 4) acc += partial[int64_t(r) * kMlpParams + col];
    part[ty][tx] = acc;
    __syncthreads();
    if (ty == 0 && col < kMlpParams) atomicAdd(out + col, (part[0][tx] + part[1][tx]) + (part[2][tx] + part[3][tx]));
}

// The longest list that is taken to be scattered.
constexpr int64_t kScatteredMaxRays = int64_t(1) << 18;

int backward_partial_rows(int n_groups) { return n_groups * kBwdWaves; }

bool backward_aggregates(const GridArgs& g) {
    return int64_t(g.n_blocks) * g.B * g.B * g.B < (int64_t(1) << 31);
}

hipError_t launch_backward(const BackwardArgs& a, int n_groups, hipStream_t s) {
    if (a.n_rays <= 0) return hipSuccess;
    hipError_t e;
    if (a.mlp_mode == kMlpF16) {
        hipLaunchKernelGGL(k_mlp_backward<true>, dim3(n_groups), dim3(64 * kBwdWaves), 0, s, a);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    } else if (a.mlp_mode == kMlpF32) {
        hipLaunchKernelGGL(k_mlp_backward<false>, dim3(n_groups), dim3(64 * kBwdWaves), 0, s, a);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    if (a.mlp_only) return hipSuccess;
    // Neighbouring rays share voxels and go through the table (half a tile to
    // a workgroup): whole views, patch lists, and lists so long that most of
    // the pixels must be in them.  Scattered rays share few and go through
    // the log, as do grids whose voxel indices exceed the table's int32 keys.
    const bool agg = backward_aggregates(a.grid) && (!a.ray_ids || a.patch_rays || a.n_rays > kScatteredMaxRays);
    const bool feat = a.mlp_mode != kMlpOff;
    static_assert(kAdjWaves * 8 == 32, "two workgroups to 64 rays");
    const int64_t wgs = 2 * (a.ray_ids ? (a.n_rays + 63) / 64 : a.total_tiles);
    const dim3 wg{64 * kAdjWaves};
    const size_t lds = (size_t(a.grid.n_words) + 1) / 2 * 16 +
                       (agg ? size_t(kAggWords) * 4 : size_t(kAdjWaves) * kLogEntries * sizeof(int4));
    // a launch holds fewer than 2^32 lanes
    constexpr int64_t kMaxGroups = int64_t(1) << 22;
    BackwardArgs b = a;
    for (b.first_group = 0; b.first_group < wgs; b.first_group += kMaxGroups) {
        const dim3 grid{unsigned(wgs - b.first_group < kMaxGroups ? wgs - b.first_group : kMaxGroups)};
        if (feat && agg) hipLaunchKernelGGL((k_adjoint<true, true>), grid, wg, lds, s, b);
        else if (feat) hipLaunchKernelGGL((k_adjoint<true, false>), grid, wg, lds, s, b);
        else if (agg) hipLaunchKernelGGL((k_adjoint<false, true>), grid, wg, lds, s, b);
        else hipLaunchKernelGGL((k_adjoint<false, false>), grid, wg, lds, s, b);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_reduce_mlp(const float* partial, int rows, float* out, hipStream_t s) {
    const dim3 grid((kMlpParams + 63) / 64, (rows + kReduceRows - 1) / kReduceRows);
    hipLaunchKernelGGL(k_reduce_rows, grid, dim3(256), 0, s, partial, rows, out);
    return hipGetLastError();
}

}  // namespace snerg
