// Adjoint of the render (fine-tuning by a pixel loss, Eq. 3, Section 5.5).
//
// For each ray with output gradient g = dL/d(rgb, alpha):
//  K1 (k_mlp_backward, only with the MLP on): MLP backward (Eq. 7):
//     g_C = g_rgb + (J_R^T g_rgb)[0:3], g_V = (J_R^T g_rgb)[3:7], written per
//     ray; the weight gradients of the wavefront's 64 rays are summed with
//     FP32 MFMA outer products (rays are the K dimension) into per-wavefront
//     partial rows, reduced afterwards.
//  K2: re-march the same samples (nothing per sample was stored).  With E = g_C . C_d + g_V . V (from the forward's saved C_d,
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
//     hand-overs of neighbouring rays (whole views, patch lists, long lists)
//     or an LDS log (scattered lists), either way flushed to the gradient
//     arrays with float atomics grouped by cache line.  launch_backward says
//     which of the kernels below runs when.
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

// Between LDS accesses of different lanes of one wavefront.
__device__ __forceinline__ void sync_wave() {
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Whether `p` holds in any thread of the workgroup; `word` is LDS that nothing
// else uses yet (__syncthreads_or takes LDS of its own, and at 512^3 in blocks
// of 16 two workgroups of k_march_backward fill a compute unit's to the byte:
// 7.0 ms against 10.8).
__device__ __forceinline__ bool any_in_group(int32_t* word, bool p) {
    if (threadIdx.x == 0) *word = 0;
    __syncthreads();
    if (p) *word = 1;
    __syncthreads();
    const bool any = *word != 0;
    __syncthreads();
    return any;
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

// Coordinates x | y << 8 | z << 16 of macroblock lin (< 2^18: the rounded
// product is never a half away from the quotient).
__device__ __forceinline__ int32_t block_coords(const GridArgs& g, int32_t lin) {
    const float inv_g = 1.0f / float(g.G);
    const int32_t yz = int32_t((float(lin) + 0.5f) * inv_g), z = int32_t((float(yz) + 0.5f) * inv_g);
    return (lin - mul_s24(yz, g.G)) | (yz - mul_s24(z, g.G)) << 8 | z << 16;
}

// Gradient aggregation in LDS.  Neighbouring rays share most of the voxels
// they touch, so each voxel's eight gradient values (density, RGB, features)
// are first summed in an open-addressed table of kAggSlots entries and reach
// device memory with one set of atomics per table flush instead of one per
// ray.  Keys are canonical voxel indices (< 2^31; the launch falls back to
// direct atomics otherwise).
//
// The colour and feature sums are kept in 32-bit fixed point: on gfx950 an
// LDS float add (ds_add_f32) retires about one lane every three cycles, an
// LDS integer add (ds_add_u32) more than forty times faster.  A ray hands a
// voxel its colour gradient A g_C with A = sum_k w_c(k) w_k, and the A of all
// of a ray's hand-overs add up to at most sum_k w_k <= 1, so with M = max over
// the rays of the tile, or of 64 list entries, of |g_C|, |g_V| all that one ray
// hands to one voxel is at most M and a table entry (64 rays between flushes)
// at most 64 M.  Values are scaled by 2^S, the largest power of two with
// M 2^S < 2^24, and rounded to integers: an entry stays below 2^30 (plus its
// rounding), and each hand-over carries a rounding error of at most 2^-24 M.
// The density sums, whose size depends on the grid values, stay in float.
constexpr int kAggLog = 9;
constexpr int kAggSlots = 1 << kAggLog;
constexpr int kAggProbes = 16;
constexpr int kAggWords = kAggSlots * 9;  // keys, 8 value planes
// A wavefront's own table is flushed once this many keys are in.  Every flush
// sends each held voxel's eight sums to device memory as float atomics, which
// gfx950 executes at the memory side, about 21 G cache lines per second, so
// the fewer flushes the better: at 7/8 full the adjoint frame ran 18% faster
// than at 1/2 (the table then holds most of a tile's voxels at once); a key
// that finds no free slot within kAggProbes probes goes to device memory
// directly.
constexpr int kAggFlushAt = kAggSlots * 7 / 8;

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

// The first of the kAggProbes consecutive slots in which `key` may be.
__device__ __forceinline__ uint32_t agg_hash(int32_t key) { return (uint32_t(key) * 2654435761u) >> (32 - kAggLog); }

// The table slot of `key` among `probes` from `sl` on (lanes may diverge),
// claimed if it has none; -1 when there is none free.  `fresh` counts the
// lane's new keys.  (Kept from unrolling, the loop cost the one-lane walk 10 to 17%:
// two sparse 160x160 views of 512^3 3.46 ms, 2.98 as it is.)
__device__ __forceinline__ int agg_slot(const AggTable& t, uint32_t sl, int probes, int32_t key, int& fresh) {
    for (; probes > 0; --probes) {
        // one round trip per probe: the compare-and-swap claims a free slot
        // and otherwise returns the key that holds it
        const int32_t k = atomicCAS(t.key + sl, -1, key);
        fresh += k == -1 ? 1 : 0;
        if (k == -1 || k == key) return int(sl);
        sl = (sl + 1) & (kAggSlots - 1);
    }
    return -1;
}

// Adds a ray's hand-over to the entry at slot sl.
template <bool FEAT>
__device__ __forceinline__ void agg_add(const AggTable& t, int sl, float Ds, float A, const float gC[3],
                                        const float gV[4]) {
    int32_t* iv = reinterpret_cast<int32_t*>(t.val);
    atomicAdd(t.val + sl, Ds);
    const float Aq = A * t.q;  // a power of two: exact, so the products round as A g would
#pragma unroll
    for (int c = 0; c < 3; ++c) atomicAdd(iv + (1 + c) * kAggSlots + sl, int32_t(__builtin_rintf(Aq * gC[c])));
    if (FEAT) {
#pragma unroll
        for (int c = 0; c < 4; ++c) atomicAdd(iv + (4 + c) * kAggSlots + sl, int32_t(__builtin_rintf(Aq * gV[c])));
    }
}

// Adds a voxel's hand-over to the table (lanes may diverge), or straight to
// device memory when it finds no slot.
template <bool FEAT>
__device__ __forceinline__ void agg_hand_over(const BackwardArgs& a, const AggTable& t, int32_t key, float Ds, float A,
                                              const float gC[3], const float gV[4], int& fresh) {
    const int sl = agg_slot(t, agg_hash(key), kAggProbes, key, fresh);
    if (sl >= 0) {
        agg_add<FEAT>(t, sl, Ds, A, gC, gV);
    } else {
        const float v[8] = {Ds, A * gC[0], A * gC[1], A * gC[2], A * gV[0], A * gV[1], A * gV[2], A * gV[3]};
        for (int c = 0; c < (FEAT ? 8 : 4); ++c) unsafeAtomicAdd(grad_channel(a, key, c), v[c]);
    }
}

// `threads` threads in whole wavefronts, with nobody else at the table: every
// used entry goes to device memory, the table is cleared.  gfx950 serves a
// wavefront's float atomics per 64-byte line (measured: about 21 G lines per
// second whether a line carries one lane's add or sixteen), so the lanes are
// laid across the entries' channels, not the entries: lane l takes entry l / 4
// of a group of 16 and within it channels l % 4 and l % 4 + 4, so that one
// instruction adds an entry's density and colour (two lines) and the next its
// four features (one line), where one lane per entry would touch seven lines.
// With packed gradients an entry's eight sums share one line: eight lanes per
// entry (four without features), one instruction per group.
// kC: lanes per entry; kBatch: entries of a lane whose keys and values are read
// together, 4 where one wavefront flushes alone, in a chain of LDS reads.
template <bool FEAT, int kC, int kBatch>
__device__ __forceinline__ void agg_flush_by(const BackwardArgs& a, const AggTable& t, int tid, int threads) {
    int32_t* iv = reinterpret_cast<int32_t*>(t.val);
    auto value = [&](int sl, int c) { return c == 0 ? t.val[sl] : float(iv[c * kAggSlots + sl]) * t.dq; };
    constexpr bool kTwo = FEAT && kC == 4;
    const int c = tid & (kC - 1), step = threads / kC;
    for (int s0 = tid / kC; s0 < kAggSlots; s0 += kBatch * step) {
        // the lanes of an entry sit in one wavefront and read its key before
        // any of them frees it
        int32_t key[kBatch];
        float v0[kBatch], v1[kBatch];
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            const int sl = s0 + u * step;
            key[u] = t.key[sl];
            v0[u] = value(sl, c);
            v1[u] = kTwo ? value(sl, c + 4) : 0.0f;
        }
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            const int sl = s0 + u * step;
            if (key[u] < 0) continue;
            if (v0[u] != 0.0f) unsafeAtomicAdd(grad_channel(a, key[u], c), v0[u]);
            iv[c * kAggSlots + sl] = 0;  // (zero bits are 0.0f too)
            if (kTwo) {
                if (v1[u] != 0.0f) unsafeAtomicAdd(grad_channel(a, key[u], c + 4), v1[u]);
                iv[(c + 4) * kAggSlots + sl] = 0;
            }
            if (c == 0) t.key[sl] = -1;
        }
    }
}

template <bool FEAT, int kBatch = 1>
__device__ __forceinline__ void agg_flush(const BackwardArgs& a, const AggTable& t, int tid, int threads) {
    if (FEAT && a.grad_packed) agg_flush_by<FEAT, 8, kBatch>(a, t, tid, threads);
    else agg_flush_by<FEAT, 4, kBatch>(a, t, tid, threads);
}

// ------------------------------------------------------ one lane to a ray

// Running gradient sums for the 8 corner voxels of the ray's current cell.
struct CellWindow {
    int32_t c[3];  // padded cell coordinates
    int32_t rank;  // block record, -1 when empty
    int32_t id;    // atlas id of the block
    int32_t b;     // block coordinates, x | y << 8 | z << 16
    float A[8], D[8];
};

__device__ __forceinline__ int wave_sum_i32(int v) {
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) v += __shfl_xor(v, m);
    return __builtin_amdgcn_readfirstlane(v);
}

template <bool FEAT>
__device__ __forceinline__ void flush_corner(const BackwardArgs& a, const AggTable& t, const CellWindow& w, int c,
                                             const float gC[3], const float gV[4], int& fresh, int32_t& nb_lin,
                                             int32_t& nb_id) {
    const float A = w.A[c], D = w.D[c];
    if (A == 0.0f && D == 0.0f) return;
    const int32_t vi = canonical_voxel<int32_t>(a.grid, w.id, w.b, w.c[0] + (c & 1) - 1, w.c[1] + ((c >> 1) & 1) - 1,
                                                w.c[2] + (c >> 2) - 1, nb_lin, nb_id);
    if (vi >= 0) agg_hand_over<FEAT>(a, t, vi, a.grid.sigma_scale * D, A, gC, gV, fresh);
}

// The T under which a ray's adjoint ends, so that it ends with the forward, whose
// last T is `t_last`.  The factor here is sigma_scale * (1 / N), the forward's
// sigma_scale / N.  Where they differ in the last place (sigma_scale 50: N = 48, 96,
// 192, 384, 768), T does by some 2^-20, and the line lies between the forward's last
// T and its T before, which was t_stop or more.  (With the forward's factor the
// gradients would be no nearer to those in 64 bits, 5e-5 of the features' norm either
// way, but patches of 768^3 would differ from these by up to 5e-3 of a value where
// the tables round the other way.)
__device__ __forceinline__ float stop_below(const BackwardArgs& a, float t_last) {
    const float t = a.opts.t_stop;
    if (!a.stop_by_t) return t;
    return t_last < t ? fmaxf(0.5f * (t_last + t), t_last * (1.0f + 0x1p-16f)) : -1.0f;
}

// The adjoint state of one ray's re-march: its output gradient and the
// forward's per-ray results (E, the T_N tail), the running transmittance T
// and prefix P_k, and the corner window.  sample() takes the samples in
// march order, as march_ray hands them over (inactive ones included), and
// returns true once the early-stop rule ends the ray; finish() hands over
// the last window.
template <bool FEAT>
struct AdjointRay {
    float gC[3], gV[4];
    float E, tail, T, Pk;
    float delta, kx, t_stop;
    bool nn_gate;
    CellWindow win;
    int fresh;  // this lane's new table keys since the last count
    int32_t nb_lin, nb_id;  // the last neighbouring block looked up: linear index, atlas id

    // Reads list position i's state; false when the ray composited nothing
    // (no grid gradient) or `live` is false.
    __device__ __forceinline__ bool setup(const BackwardArgs& a, int64_t i, bool live) {
        float4 a0 = make_float4(0.f, 0.f, 0.f, 0.f), a1 = make_float4(0.f, 0.f, 0.f, -1.f);
        float4 gg = make_float4(0.f, 0.f, 0.f, 0.f);
        if (live) {
            a1 = reinterpret_cast<const float4*>(a.aux)[2 * i + 1];
            live = a1.w >= 0.0f;  // nothing was composited: no grid gradient
        }
        gC[0] = gC[1] = gC[2] = 0.f;
        gV[0] = gV[1] = gV[2] = gV[3] = 0.f;
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
        E = gC[0] * a0.x + gC[1] * a0.y + gC[2] * a0.z + (gV[0] * a0.w + gV[1] * a1.x + gV[2] * a1.y + gV[3] * a1.z);
        const float gTN = gg.x * a.opts.bg[0] + gg.y * a.opts.bg[1] + gg.z * a.opts.bg[2] - gg.w;
        tail = a1.w * gTN;
        T = 1.0f;
        Pk = 0.0f;
        delta = 1.0f / float(a.grid.N);
        kx = a.grid.sigma_scale * delta;
        t_stop = stop_below(a, a1.w);
        nn_gate = a.opts.nn_gate != 0;
        win.rank = -1;
        win.id = 0;
        win.c[0] = win.c[1] = win.c[2] = 0;
        win.b = 0;
#pragma unroll
        for (int c = 0; c < 8; ++c) win.A[c] = win.D[c] = 0.0f;
        fresh = 0;
        nb_lin = -1;
        nb_id = -1;
        return live;
    }

    // Wavefront-wide (all 64 lanes, the same value in each): the largest
    // |g_C|, |g_V| sets the table's fixed-point scale.
    __device__ __forceinline__ void table_scale(AggTable& tab) const {
        float m = fmaxf(fmaxf(fabsf(gC[0]), fabsf(gC[1])), fmaxf(fabsf(gC[2]), fabsf(gV[0])));
        m = fmaxf(m, fmaxf(fmaxf(fabsf(gV[1]), fabsf(gV[2])), fabsf(gV[3])));
#pragma unroll
        for (int sh = 32; sh >= 1; sh >>= 1) m = fmaxf(m, __shfl_xor(m, sh));
        agg_scale(tab, m);  // the butterfly leaves the same maximum in every lane
    }

    __device__ __forceinline__ bool sample(const BackwardArgs& a, const AggTable& tab, int32_t rk, const uint8_t* vox,
                                           const int32_t p[3], const int32_t fr[3]) {
        Sample smp;
        gather_f32(vox, a.grid.Bp, p, fr, smp, nn_gate);
        const GridArgs& g = a.grid;
        if (!smp.active) return false;
        const float e = __expf(-smp.sigma_raw * kx);
        const float w = T * (1.0f - e);
        const float ek = gC[0] * smp.rgb[0] + gC[1] * smp.rgb[1] + gC[2] * smp.rgb[2] +
                         (gV[0] * smp.feat[0] + gV[1] * smp.feat[1] + gV[2] * smp.feat[2] + gV[3] * smp.feat[3]);
        Pk += w * ek;
        T *= e;
        const float gsig = delta * (T * ek - (E - Pk) - tail);
        // Slide the corner window to this sample's cell: corners on a
        // trailing face (or all of them after a jump) are flushed once, the
        // survivors shift to their new corner index.
        const bool jump = win.rank != rk || abs(p[0] - win.c[0]) > 1 || abs(p[1] - win.c[1]) > 1 ||
                          abs(p[2] - win.c[2]) > 1;
        int dd[3] = {p[0] - win.c[0], p[1] - win.c[1], p[2] - win.c[2]};
        uint32_t leave = 0;
        if (jump) {
            leave = win.rank >= 0 ? 0xFFu : 0u;
        } else {
#pragma unroll
            for (int ax = 0; ax < 3; ++ax) {
                // corners with bit ax clear: 0x55, 0x33, 0x0F for ax = 0, 1, 2
                const uint32_t clear = ax == 0 ? 0x55u : (ax == 1 ? 0x33u : 0x0Fu);
                if (dd[ax] > 0) leave |= clear;
                if (dd[ax] < 0) leave |= ~clear & 0xFFu;
            }
        }
#pragma unroll
        for (int c = 0; c < 8; ++c)
            if ((leave >> c) & 1u) flush_corner<FEAT>(a, tab, win, c, gC, gV, fresh, nb_lin, nb_id);
        if (jump) {
#pragma unroll
            for (int c = 0; c < 8; ++c) win.A[c] = win.D[c] = 0.0f;
            win.rank = rk;
            win.id = g.rank_id[rk];
            win.b = block_coords(g, g.rank_lin[rk]);
            win.c[0] = p[0]; win.c[1] = p[1]; win.c[2] = p[2];
        } else {
#pragma unroll
            for (int ax = 0; ax < 3; ++ax) {
                const int bit = 1 << ax;
#pragma unroll
                for (int c = 0; c < 8; ++c) {
                    if (c & bit) continue;
                    const int c1 = c | bit;
                    const float a0v = win.A[c], d0v = win.D[c], a1v = win.A[c1], d1v = win.D[c1];
                    win.A[c] = dd[ax] > 0 ? a1v : (dd[ax] < 0 ? 0.0f : a0v);
                    win.D[c] = dd[ax] > 0 ? d1v : (dd[ax] < 0 ? 0.0f : d0v);
                    win.A[c1] = dd[ax] < 0 ? a0v : (dd[ax] > 0 ? 0.0f : a1v);
                    win.D[c1] = dd[ax] < 0 ? d0v : (dd[ax] > 0 ? 0.0f : d1v);
                }
                win.c[ax] += dd[ax];
            }
        }
        float wc[8];
        corner_weights(fr, wc);
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            win.A[c] = fmaf(wc[c], w, win.A[c]);
            win.D[c] = fmaf(wc[c], gsig, win.D[c]);
        }
        return T < t_stop;
    }

    __device__ __forceinline__ void finish(const BackwardArgs& a, const AggTable& tab) {
        if (win.rank >= 0) {
#pragma unroll
            for (int c = 0; c < 8; ++c) flush_corner<FEAT>(a, tab, win, c, gC, gV, fresh, nb_lin, nb_id);
        }
    }
};

// The table of the calling wavefront in dynamic LDS (after the occupancy
// words), cleared.
__device__ __forceinline__ AggTable agg_table(uint2* s_occ, int n_words, int wave, int lane) {
    AggTable tab;
    int32_t* base = reinterpret_cast<int32_t*>(s_occ + n_words) + wave * kAggWords;
    tab.key = base;
    tab.val = reinterpret_cast<float*>(base + kAggSlots);
    for (int sl = lane; sl < kAggSlots; sl += 64) {
        tab.key[sl] = -1;
#pragma unroll
        for (int c = 0; c < 8; ++c) tab.val[c * kAggSlots + sl] = 0.0f;
    }
    return tab;
}

// agg_flush by one wavefront on its own table.
template <bool FEAT>
__device__ __forceinline__ void wave_flush(const BackwardArgs& a, const AggTable& t, int lane) {
    sync_wave();
    agg_flush<FEAT, 4>(a, t, lane, 64);
    sync_wave();
}

// Wavefront-wide, after each step of the lanes: counts the table's new keys
// and flushes it once it is full enough.
struct TableSync {
    int in_table = 0;  // wave-uniform: keys in the table
    template <bool FEAT>
    __device__ __forceinline__ void step(const BackwardArgs& a, const AggTable& tab, int lane, int& fresh) {
        if (__any(fresh != 0)) {
            in_table += wave_sum_i32(fresh);
            fresh = 0;
            if (in_table >= kAggFlushAt) {
                wave_flush<FEAT>(a, tab, lane);
                in_table = 0;
            }
        }
    }
};

// One lane per ray.  Without a ray list the wavefronts walk the cameras'
// tile_w x tile_h pixel tiles (neighbouring rays, shared voxels); with a list,
// 64 consecutive list entries.  Gradients go through the wavefront's LDS
// table.  Every lane stays to the end (the flushes need all 64).  backward_route
// says which calls come here.
constexpr int kAggWaves = 4;  // wavefronts per workgroup
constexpr int kAggLdsWords = kAggWaves * kAggWords;

template <bool FEAT>
__global__ __launch_bounds__(64 * kAggWaves) void k_march_backward(BackwardArgs a) {
    extern __shared__ uint2 s_occ[];
    const GridArgs& g = a.grid;
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    // this lane's ray: list position i (indexes aux, grad_rgba, gcv) and id r
    bool live;
    int64_t i, r;
    const int64_t wt = int64_t(a.ray_ids ? blockIdx.x : xcd_grouped(blockIdx.x, gridDim.x)) * kAggWaves + wave;
    if (a.ray_ids) {
        i = wt * 64 + lane;
        live = i < a.n_rays;
        // after a list launch: the rays whose samples it could not list
        if (a.list) live = live && a.list_count[i] > kBackwardListCap;
        r = live ? a.ray_ids[i] : 0;
    } else {
        live = wt < a.total_tiles;
        i = r = 0;
        if (live) {
            const int ci = find_camera_by_tile(a.cams, a.n_cams, wt);
            const DevCamera& c = a.cams[ci];
            const int64_t tl = wt - c.tile_offset;
            const int px = int(tl % c.tiles_x) * a.tile_w + lane % a.tile_w;
            const int py = int(tl / c.tiles_x) * a.tile_h + lane / a.tile_w;
            live = px < c.W && py < c.H;
            i = r = c.ray_offset + int64_t(py) * c.W + px;
        }
    }
    if (a.list && !any_in_group(reinterpret_cast<int32_t*>(s_occ), live)) return;
    for (int w = threadIdx.x; w < g.n_words; w += blockDim.x) s_occ[w] = g.occ[w];
    AggTable tab = agg_table(s_occ, g.n_words, wave, lane);
    __syncthreads();
    AdjointRay<FEAT> st;
    live = st.setup(a, i, live);
    st.table_scale(tab);

    int64_t o[3] = {0, 0, 0};
    int32_t s[3] = {0, 0, 1 << 15};
    if (live) {
        int ci, px, py;
        locate(a, r, ci, px, py);
        float d[3];
        ray_setup(a.cams[ci], g.N, px, py, o, s, d);
    }
    TableSync sync;
    march_ray_flat_sync(
        g, s_occ, live, o, s,
        [&](int64_t, int32_t rk, const uint8_t* vox, const int32_t p[3], const int32_t fr[3]) {
            return st.sample(a, tab, rk, vox, p, fr);
        },
        [&]() {
            sync.step<FEAT>(a, tab, lane, st.fresh);
            return false;
        });
    st.finish(a, tab);
    wave_flush<FEAT>(a, tab, lane);
}

// ------------------------------------------------------ eight lanes to a ray

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

// Where a lane stands in its ray's cell.
struct CornerLane {
    int l, cx, cy, cz;
    float ox, oy, oz;  // the corner's weight on an axis is f = |0 - f| or 1 - f
    uint32_t offset;   // of the corner's voxel from the cell's first, in bytes

    __device__ __forceinline__ CornerLane(const GridArgs& g, int lane) {
        l = lane & 7;
        cz = l >> 2;
        cx = (l & 1) ^ cz;
        cy = ((l >> 1) & 1) ^ cz;
        ox = cx ? 0.0f : 1.0f;
        oy = cy ? 0.0f : 1.0f;
        oz = cz ? 0.0f : 1.0f;
        offset = uint32_t((cz * g.Bp + cy) * g.Bp + cx) * 32u;
    }
};

// A sample as the lanes of its ray hold it: position in the block (Q16, own
// axis), record, corner voxel, exp(-sigma delta).
struct Fetched {
    int32_t own, rank;
    float4 rgb, feat;
    float e;

    // Reads this corner's voxel of the cell at `own`.
    template <bool FEAT>
    __device__ __forceinline__ void read(const GridArgs& g, const CornerLane& c, const uint8_t* vox) {
        const int32_t p[3] = {dpp<kAxisX>(own) >> 16, dpp<kAxisY>(own) >> 16, dpp<kAxisZ>(own) >> 16};
        const uint32_t nb = uint32_t(g.Bp);
        const uint8_t* at = vox + (uint64_t(cell_index(p, nb, nb * nb)) * 32u + c.offset);
        rgb = reinterpret_cast<const float4*>(at)[0];
        if (FEAT) feat = reinterpret_cast<const float4*>(at)[1];
    }
};

// The adjoint state of a ray in its 8 lanes: the same in all but A and D,
// the running sums of the lane's corner, and the window's cell, own axis.
template <bool FEAT>
struct CornerRay {
    float gC[3], gV[4];
    float T, rest;  // rest: E - P_k + T_N dL/dT_N
    float t_stop;
    float A, D;
    int32_t wc;              // the window's cell, own axis
    int32_t wrank, wid, wb;  // its block's record, atlas id, coordinates
    int32_t nb_lin, nb_id;

    // Reads list position i's state; false when the ray composited nothing
    // (no grid gradient) or `live` is false.
    __device__ __forceinline__ bool setup(const BackwardArgs& a, int64_t i, bool live) {
        float4 a0 = make_float4(0.f, 0.f, 0.f, 0.f), a1 = make_float4(0.f, 0.f, 0.f, -1.f);
        float4 gg = make_float4(0.f, 0.f, 0.f, 0.f);
        if (live) {
            a1 = reinterpret_cast<const float4*>(a.aux)[2 * i + 1];
            live = a1.w >= 0.0f;
        }
        gC[0] = gC[1] = gC[2] = 0.f;
        gV[0] = gV[1] = gV[2] = gV[3] = 0.f;
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
        rest = E + a1.w * gTN;
        T = 1.0f;
        t_stop = stop_below(a, a1.w);
        A = D = 0.0f;
        wc = 0;
        wrank = -1;
        wid = wb = 0;
        nb_lin = nb_id = -1;
        return live;
    }

    // The channel that lane l adds to device memory, where the lanes of a ray
    // stand for a voxel's channels.
    __device__ __forceinline__ float channel(int l) const {
        float v = 0.0f;
#pragma unroll
        for (int c = 0; c < 3; ++c) v = l == 1 + c ? gC[c] : v;
#pragma unroll
        for (int c = 0; c < 4; ++c) v = l == 4 + c ? gV[c] : v;
        return v;
    }

    // Slot of this lane's corner, -1 where `leave` is not set or it holds nothing.
    template <typename I>
    __device__ __forceinline__ I voxel(const GridArgs& g, const CornerLane& c, bool leave) {
        const int vx = dpp<kAxisX>(wc) + c.cx - 1, vy = dpp<kAxisY>(wc) + c.cy - 1, vz = dpp<kAxisZ>(wc) + c.cz - 1;
        I vi = -1;
        if (leave && (A != 0.0f || D != 0.0f)) vi = canonical_voxel<I>(g, wid, wb, vx, vy, vz, nb_lin, nb_id);
        return vi;
    }

    // What an active sample does to the window: the weights it brings, how
    // far the window's cell moves, whether this lane's corner leaves.
    struct Slide {
        float wt, ws, gsig;
        int32_t move;
        bool jump, lx, ly, lz, leave;
    };

    __device__ __forceinline__ Slide weigh(const BackwardArgs& a, const CornerLane& c, const Fetched& f, int lane) {
        Slide m;
        const int32_t q[3] = {dpp<kAxisX>(f.own), dpp<kAxisY>(f.own), dpp<kAxisZ>(f.own)};
        const float fx = float(q[0] & 0xFFFF) * (1.0f / 65536.0f);
        const float fy = float(q[1] & 0xFFFF) * (1.0f / 65536.0f);
        const float fz = float(q[2] & 0xFFFF) * (1.0f / 65536.0f);
        m.wt = (fabsf(c.ox - fx) * fabsf(c.oy - fy)) * fabsf(c.oz - fz);
        float ev = gC[0] * f.rgb.y + gC[1] * f.rgb.z + gC[2] * f.rgb.w;
        if (FEAT) ev += gV[0] * f.feat.x + gV[1] * f.feat.y + gV[2] * f.feat.z + gV[3] * f.feat.w;
        const float ek = corner_sum(m.wt * ev);
        m.ws = T * (1.0f - f.e);
        rest -= m.ws * ek;
        T *= f.e;
        m.gsig = (1.0f / float(a.grid.N)) * (T * ek - rest);
        // Corners on a trailing face (or all of them after a jump) leave: on
        // an axis the window moves along, those on the trailing side.
        m.move = (f.own >> 16) - wc;
        const int32_t dd[3] = {dpp<kAxisX>(m.move), dpp<kAxisY>(m.move), dpp<kAxisZ>(m.move)};
        m.jump = wrank != f.rank || ray_bits(abs(m.move) > 1, lane) != 0;
        m.lx = dd[0] != 0 && (dd[0] > 0) == (c.cx == 0);
        m.ly = dd[1] != 0 && (dd[1] > 0) == (c.cy == 0);
        m.lz = dd[2] != 0 && (dd[2] > 0) == (c.cz == 0);
        m.leave = m.jump ? wrank >= 0 : m.lx || m.ly || m.lz;
        return m;
    }

    // The corners that left have been handed over: the survivors move to their
    // new lane.  Returns true once the early-stop rule ends the ray.
    __device__ __forceinline__ bool slide(const BackwardArgs& a, const Fetched& f, const Slide& m) {
        if (m.jump) {
            A = D = 0.0f;
            wrank = f.rank;
            wid = a.grid.rank_id[f.rank];
            wb = block_coords(a.grid, a.grid.rank_lin[f.rank]);
        } else {
            // a trailing corner takes its leading neighbour's sums, which start anew
            const int32_t dd[3] = {dpp<kAxisX>(m.move), dpp<kAxisY>(m.move), dpp<kAxisZ>(m.move)};
            float An = dpp<kFlipX>(A), Dn = dpp<kFlipX>(D);
            A = dd[0] == 0 ? A : (m.lx ? An : 0.0f);
            D = dd[0] == 0 ? D : (m.lx ? Dn : 0.0f);
            An = dpp<kFlipY>(A), Dn = dpp<kFlipY>(D);
            A = dd[1] == 0 ? A : (m.ly ? An : 0.0f);
            D = dd[1] == 0 ? D : (m.ly ? Dn : 0.0f);
            An = dpp<kFlipZ>(A), Dn = dpp<kFlipZ>(D);
            A = dd[2] == 0 ? A : (m.lz ? An : 0.0f);
            D = dd[2] == 0 ? D : (m.lz ? Dn : 0.0f);
        }
        wc += m.move;
        A = fmaf(m.wt, m.ws, A);
        D = fmaf(m.wt, m.gsig, D);
        return T < t_stop;
    }

    // Takes an active sample.  hand_over(leave) is called once, by all lanes of
    // the ray, before the window moves: the lanes with `leave` hand over.
    template <typename HandOver>
    __device__ __forceinline__ bool take(const BackwardArgs& a, const CornerLane& c, const Fetched& f, int lane,
                                         HandOver&& hand_over) {
        const Slide m = weigh(a, c, f, lane);
        hand_over(m.leave);
        return slide(a, f, m);
    }
};

// The lanes of a ray add its corners with vi >= 0 to device memory, the 8
// channels of one after the other.  gch: own channel's gradient.
template <typename I>
__device__ __forceinline__ void add_direct(const BackwardArgs& a, int l, int lane, I vi, float Ds, float A, float gch) {
    for (uint32_t m = ray_bits(vi >= 0, lane); m != 0; m &= m - 1) {
        const int from = (lane & ~7) | __builtin_ctz(m);
        const I v = __shfl(vi, from);
        const float dv = __shfl(Ds, from), av = __shfl(A, from);
        const float x = l == 0 ? dv : av * gch;
        if (x != 0.0f) unsafeAtomicAdd(grad_channel(a, v, l), x);
    }
}

// exp(-sigma delta) of a sample in a float32 block at `vox` and whether it is
// active, with the forward's operations in their order (gather_f32) but for the
// factor (stop_below).
__device__ __forceinline__ bool sample_decay(const GridArgs& g, const uint8_t* vox, const int32_t p[3],
                                             const int32_t fr[3], bool nn_gate, float& e) {
    const uint32_t nb = uint32_t(g.Bp), nbb = nb * nb;
    const uint8_t* at = vox + uint64_t(cell_index(p, nb, nbb)) * 32u;
    float den[8], w[8];
#pragma unroll
    for (int c = 0; c < 8; ++c)
        den[c] = *reinterpret_cast<const float*>(at + ((c & 1 ? 32u : 0u) + (c & 2 ? nb * 32u : 0u) +
                                                       (c & 4 ? nbb * 32u : 0u)));
    corner_weights(fr, w);
    const int cnn = nearest_corner(fr);
    float sigma = 0.0f, dnn = 0.0f;
    bool act = false;
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        act |= den[c] != 0.0f && corner_live(c, fr);
        dnn = c == cnn ? den[c] : dnn;
        sigma = fmaf(w[c], den[c], sigma);
    }
    e = __expf(-sigma * (g.sigma_scale * (1.0f / float(g.N))));
    return nn_gate ? dnn != 0.0f : act;
}

// The log of a wavefront whose rays share few voxels: what the lanes hand
// over in a step (voxel, ray, A, density sum) goes, once all 64 are together,
// to the place a ballot gives it, so the fill count is the same in every lane.
// A full log goes to device memory, 8 entries to an instruction, the lanes of
// one across the voxel's channels.  Added straight away, every atomic would
// stand in front of the next step's loads, which wait for it (vector memory
// retires in order).
constexpr int kLogEntries = 320;  // 16 bytes each

template <int kEntries>
struct WaveLog {
    int4* at;           // [kEntries]: voxel (low word; ray << 24 | high), A, density sum
    float (*gch)[8];    // the rays' gradients by channel
    int n = 0;
    int64_t vi = -1;    // what this lane hands over, < 0: nothing
    float A = 0.0f, Ds = 0.0f;

    __device__ __forceinline__ void flush(const BackwardArgs& a, int lane) {
        sync_wave();
        const int l = lane & 7;
        for (int e = lane >> 3; e < n; e += 8) {
            const int4 h = at[e];
            const int64_t v = int64_t(uint64_t(uint32_t(h.x)) | (uint64_t(uint32_t(h.y & 0xffffff)) << 32));
            const float x = l == 0 ? __int_as_float(h.w) : __int_as_float(h.z) * gch[h.y >> 24][l];
            if (x != 0.0f) unsafeAtomicAdd(grad_channel(a, v, l), x);
        }
        n = 0;
        sync_wave();
    }

    __device__ __forceinline__ void append(const BackwardArgs& a, int lane) {
        const uint64_t m = __ballot(vi >= 0);
        if (m == 0) return;  // wave-uniform
        if (n > kEntries - 64) flush(a, lane);
        if (vi >= 0)
            at[n + int(__builtin_amdgcn_mbcnt_hi(uint32_t(m >> 32), __builtin_amdgcn_mbcnt_lo(uint32_t(m), 0u)))] =
                make_int4(int32_t(uint32_t(uint64_t(vi))), int32_t(vi >> 32) | (lane >> 3) << 24, __float_as_int(A),
                          __float_as_int(Ds));
        n += __builtin_popcountll(m);
        vi = -1;
    }
};

// Eight lanes to a ray.  A trip of the walk looks at the ray's
// next 8 lattice samples, one per lane (its distance byte and, in an active
// cell, its density), and then takes the active ones in order, all lanes
// together, lane by corner: each loads its corner's voxel, the sum g . value
// over the corners is three DPP additions, and each lane keeps its corner's
// (A, D) and hands it over by itself, into a table that the workgroup shares.
// One lane per ray pays for every sample with eight guarded hand-over passes
// and 256 bytes of loads per lane, at two wavefronts per SIMD (197 registers);
// this one runs five (96).
//   eight 800x800 views, 512^3, FP32 network   23.7 -> 17.0 ms
// Bound by instruction issue (VALUs 83% busy, half the lanes at work: about
// 270 instructions per sample of 8 rays).  Six wavefronts per SIMD cost 9%
// (spills), four 5%.
constexpr int kAdjWaves = 4;  // wavefronts per workgroup: half a tile, 8 lanes to a ray
// The workgroup looks at the table every kAdjTrips trips of its rays and
// flushes it when it holds more than kAdjFlushAt keys; what its rays add in
// four trips (up to 32 samples each) mostly fits above that.
constexpr int kAdjFlushAt = kAggSlots * 9 / 16;
constexpr int kAdjStaticLds = 512;  // at the most, beside the two tables
constexpr int kAdjTrips = 4;

// AGG: whole views and long lists of patches, half a tile (or 32 list entries) to
// a workgroup, gradients through the table.
// Else through the wavefronts' logs, with no limit on the voxel index: views
// and lists on grids beyond the table's keys, and of a scattered list the rays
// with too many samples to list.
template <bool FEAT, bool AGG>
__global__ __launch_bounds__(64 * kAdjWaves) __attribute__((amdgpu_waves_per_eu(AGG ? 5 : 4))) void k_adjoint(BackwardArgs a) {
    extern __shared__ int4 s_dyn[];  // the logs' entries set its alignment
    uint2* s_occ = reinterpret_cast<uint2*>(s_dyn);
    static_assert(alignof(decltype(s_dyn[0])) >= 16 && sizeof(uint2) == 8, "logs begin at an even uint2");
    __shared__ float s_max;
    __shared__ int32_t s_fresh[3], s_live[3];
    __shared__ float s_gch[AGG ? 1 : kAdjWaves][8][8];
    const GridArgs& g = a.grid;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    // Ray idx of the workgroup's 64: list position i (indexes aux, grad_rgba,
    // gcv), pixel (px, py) of camera ci.  Of a view's tiles each XCD takes
    // runs of 16.
    const uint32_t u = a.ray_ids ? blockIdx.x : xcd_grouped<32>(blockIdx.x, gridDim.x);
    const int64_t set = (a.first_group + u) >> 1;
    auto ray_of = [&](int idx, int64_t& i, int& ci, int& px, int& py) {
        if (a.ray_ids) {
            i = set * 64 + idx;
            if (i >= a.n_rays || (a.list && a.list_count[i] <= kBackwardListCap)) return false;
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
    int64_t i = 0;
    int ci = 0, px = 0, py = 0;
    if (AGG && threadIdx.x < 64) {  // the table's scale, from all 64 rays
        float m = 0.0f;
        if (ray_of(threadIdx.x, i, ci, px, py) && a.aux[8 * i + 7] >= 0.0f) {
            const float* v = FEAT ? a.gcv + 8 * i : a.grad_rgba + 4 * i;
#pragma unroll
            for (int ch = 0; ch < (FEAT ? 7 : 3); ++ch) m = fmaxf(m, fabsf(v[ch]));
        }
        m = wave_max(m);
        if (threadIdx.x == 0) s_max = m;
    }
    bool live = ray_of((int(u & 1) * kAdjWaves + wave) * 8 + (lane >> 3), i, ci, px, py);
    if (a.list && !any_in_group(reinterpret_cast<int32_t*>(s_occ), live)) return;
    for (int w = threadIdx.x; w < g.n_words; w += blockDim.x) s_occ[w] = g.occ[w];
    const CornerLane c(g, lane);
    AggTable tab = {nullptr, nullptr, 0.0f, 0.0f};
    if (AGG) {
        tab.key = reinterpret_cast<int32_t*>(s_occ + g.n_words);
        tab.val = reinterpret_cast<float*>(tab.key + kAggSlots);
        for (int sl = threadIdx.x; sl < kAggSlots; sl += blockDim.x) {
            tab.key[sl] = -1;
#pragma unroll
            for (int ch = 0; ch < 8; ++ch) tab.val[ch * kAggSlots + sl] = 0.0f;
        }
        if (threadIdx.x < 3) s_fresh[threadIdx.x] = s_live[threadIdx.x] = 0;
    }
    QuadWalk w;
    if (live) {
        int64_t o[3];
        int32_t s[3];
        float d[3];
        ray_setup(a.cams[ci], g.N, px, py, o, s, d);
        live = w.init(g, o, s, c.l);
    }
    CornerRay<FEAT> st;
    live = st.setup(a, i, live);
    const float gch = st.channel(c.l);
    WaveLog<kLogEntries> log = {reinterpret_cast<int4*>(s_occ + ((g.n_words + 1) & ~1)) + wave * kLogEntries, s_gch[AGG ? 0 : wave]};
    if (!AGG) s_gch[wave][lane >> 3][c.l] = gch;
    __syncthreads();
    if (AGG) agg_scale(tab, s_max);

    const uint32_t nc = uint32_t(g.Bc), ncc = nc * nc;
    int fresh = 0;
    auto hand_over = [&](bool leave) {
        using Index = typename std::conditional<AGG, int32_t, int64_t>::type;  // the table's keys are int32
        Index vi = st.template voxel<Index>(g, c, leave);
        const float Ds = g.sigma_scale * st.D;
        if (!AGG) {
            log.vi = vi;
            log.A = st.A;
            log.Ds = Ds;
            return;
        }
        if (vi >= 0) {
            const int sl = agg_slot(tab, agg_hash(int32_t(vi)), kAggProbes, int32_t(vi), fresh);
            if (sl >= 0) {
                vi = -1;
                agg_add<FEAT>(tab, sl, Ds, st.A, st.gC, st.gV);
            }
        }
        add_direct(a, c.l, lane, vi, Ds, st.A, gch);  // no slot free
    };

    int in_table = 0, phase = 0;  // keys in the table, the same in every lane of the workgroup
    for (int trip = 0;; ++trip) {
        if (!AGG) {
            if (!__any(live)) break;
        } else if (trip % kAdjTrips == 0) {
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
            if (!on || in_table > kAdjFlushAt) {
                if (!on) {  // the last windows
                    hand_over(st.wrank >= 0);
                    __syncthreads();
                }
                agg_flush<FEAT>(a, tab, threadIdx.x, blockDim.x);
                if (!on) break;
                in_table = 0;
                __syncthreads();
            }
        }
        uint32_t todo = 0;
        int32_t reach = 0;
        while (live && w.left <= 0) live = w.enter(g, s_occ);
        float my_e = 1.0f;  // exp(-sigma delta) of the sample this lane looks at
        if (live) {
            bool act = false;
            const int32_t q[3] = {dpp<kAxisX>(w.q) + mul_s24(c.l, dpp<kAxisX>(w.s)),
                                  dpp<kAxisY>(w.q) + mul_s24(c.l, dpp<kAxisY>(w.s)),
                                  dpp<kAxisZ>(w.q) + mul_s24(c.l, dpp<kAxisZ>(w.s))};
            if (c.l < w.left) {
                const int32_t p[3] = {q[0] >> 16, q[1] >> 16, q[2] >> 16};
                const int32_t db = w.dist[cell_index(p, nc, ncc)];
                reach = c.l + (db == 0 ? 1 : skip_steps(db, w.smax, w.inv_smax));
                if (db == 0) {  // (this also brings in the lines that the corners' lanes read next)
                    const int32_t fr[3] = {q[0] & 0xFFFF, q[1] & 0xFFFF, q[2] & 0xFFFF};
                    act = sample_decay(g, w.dist + g.dist_bytes, p, fr, a.opts.nn_gate != 0, my_e);
                }
            }
            todo = ray_bits(act, lane);
            reach = max(reach, dpp<kFlipX>(reach));
            reach = max(reach, dpp<kFlipY>(reach));
            reach = max(reach, dpp<kFlipZ>(reach));
            reach = min(reach, w.left);
        }
        while (AGG ? todo != 0 : __any(todo != 0)) {
            if (todo != 0) {
                const int32_t ahead = __builtin_ctz(todo);
                todo &= todo - 1;
                Fetched f;
                f.own = w.q + mul_s24(ahead, w.s);
                f.rank = w.r;
                f.e = __shfl(my_e, (lane & ~7) | ahead);
                f.template read<FEAT>(g, c, w.dist + g.dist_bytes);
                if (st.take(a, c, f, lane, hand_over)) {
                    live = false;
                    todo = 0;
                }
            }
            if (!AGG) log.append(a, lane);
        }
        if (live) {
            w.left -= reach;
            w.q += mul_s24(reach, w.s);
        }
    }
    if (!AGG) {
        hand_over(st.wrank >= 0);
        log.append(a, lane);
        log.flush(a, lane);
    }
}

// Ray lists of up to 2^18 rays, in two launches.  k_backward_record walks the
// rays, 16 lanes to each as the render does for few (with 4 the whole call
// takes 8% longer for 16,384 rays, 2% for 262,144), and lists the samples in cells
// with a zero distance byte: 16 bytes each, up to kBackwardListCap a ray; the
// gradient kernels then run over the lists, so that rays of unequal length
// and phase sit side by side without waiting for each other's walk.  A ray
// with more samples is left to the kernels that walk.  Every workgroup stages the
// occupancy table; where four of 256 lanes, 16 rays each, don't fit a compute
// unit, workgroups are of 1024 (200,000 rays, 64^3 macroblocks in blocks of 2:
// call 3.01 -> 2.18 ms).
// List entry: position in the block on x, y, z (p << 16 | fraction, 23 bits
// each) with the record's low 9 bits above x, its others above y, the active
// flag above z; exp(-sigma delta).
constexpr int kRecordLanes = 16;

__global__ __launch_bounds__(1024) void k_backward_record(BackwardArgs a) {
    constexpr int L = kRecordLanes;
    extern __shared__ uint2 s_occ[];
    const GridArgs& g = a.grid;
    for (int w = threadIdx.x; w < g.n_words; w += blockDim.x) s_occ[w] = g.occ[w];
    __syncthreads();
    const int lane = threadIdx.x & 63, me = lane & (L - 1);
    const int64_t i = (int64_t(blockIdx.x) * blockDim.x + threadIdx.x) / L;
    if (i >= a.n_rays) return;
    int32_t n = 0;
    // rays that composited nothing have no grid gradient
    if (a.aux[8 * i + 7] >= 0.0f) {
        int ci, px, py;
        locate(a, a.ray_ids[i], ci, px, py);
        int64_t o[3];
        int32_t s[3];
        float d[3];
        ray_setup(a.cams[ci], g.N, px, py, o, s, d);
        const uint32_t nc = uint32_t(g.Bc), ncc = nc * nc;
        const int32_t ahead[3] = {me * s[0], me * s[1], me * s[2]};
        int4* mine = a.list + i * kBackwardListCap;
        FlatWalk w;
        bool live = w.init(g, o, s);
        // The list may end where the gradient will stop.  Its T is the product
        // of the same factors in another order, so it differs by at most
        // 2 * 512 * 2^-24 in proportion: past a margin of 2^-10 there is no doubt.
        float T = 1.0f;
        const float t_end = a.opts.early_stop ? a.opts.t_stop * (1.0f - 0x1p-10f) : -1.0f;
        while (!(T < t_end)) {
            while (live && w.left <= 0) live = w.enter(g, s_occ, s);
            if (!live) break;
            bool hit = false;
            float decay = 1.0f;
            int32_t reach = 0;
            int4 e = make_int4(0, 0, 0, 0);
            if (me < w.left) {
                const int32_t q[3] = {w.q[0] + ahead[0], w.q[1] + ahead[1], w.q[2] + ahead[2]};
                const int32_t p[3] = {q[0] >> 16, q[1] >> 16, q[2] >> 16};
                const int32_t db = w.dist[cell_index(p, nc, ncc)];
                hit = db == 0;
                reach = me + (hit ? 1 : skip_steps(db, w.smax, w.inv_smax));
                if (hit) {
                    const int32_t fr[3] = {q[0] & 0xFFFF, q[1] & 0xFFFF, q[2] & 0xFFFF};
                    const bool act = sample_decay(g, w.dist + g.dist_bytes, p, fr, a.opts.nn_gate != 0, decay);
                    e = make_int4(q[0] | (w.r & 511) << 23, q[1] | (w.r >> 9) << 23, q[2] | int(act) << 23,
                                  __float_as_int(decay));
                    decay = act ? decay : 1.0f;
                }
            }
            const uint32_t hits = uint32_t(__ballot(hit) >> (lane & ~(L - 1))) & ((1u << L) - 1u);
            const int32_t at = n + __builtin_popcount(hits & ((1u << me) - 1u));
            if (hit && at < kBackwardListCap) mine[at] = e;
            n += __builtin_popcount(hits);
            if (hits != 0) T *= group_product<L>(decay);
            reach = min(group_max<L>(reach), w.left);
            w.left -= reach;
#pragma unroll
            for (int c = 0; c < 3; ++c) w.q[c] += mul_s24(reach, s[c]);
        }
    }
    if (me == 0) a.list_count[i] = n;
}

// A ray's list in its 8 lanes, read ahead: lane l of a quad holds word l % 4 of
// an entry.
template <bool FEAT>
struct ListReader {
    const int32_t* at;  // own word of entry 0
    int32_t n;          // listed samples to take (0: none, or left to the kernels that walk)
    int32_t word;       // own word of the entry after `f`
    Fetched f;
    bool active;

    __device__ __forceinline__ void init(const BackwardArgs& a, const CornerLane& c, int64_t i, bool live) {
        const int32_t count = live ? a.list_count[i] : 0;
        n = count <= kBackwardListCap ? count : 0;
        at = reinterpret_cast<const int32_t*>(a.list + i * kBackwardListCap) + (c.l & 3);
        word = n > 0 ? at[0] : 0;
        if (n > 0) load(a.grid, c, 0);
    }

    // Entry j (its words are in `word`) becomes f, and entry j + 1's are read.
    __device__ __forceinline__ void load(const GridArgs& g, const CornerLane& c, int32_t j) {
        const int32_t x = dpp<kAxisX>(word), y = dpp<kAxisY>(word), z = dpp<kAxisZ>(word);
        f.own = ((c.l & 3) == 3 ? z : word) & 0x7fffff;
        f.rank = int32_t(uint32_t(x) >> 23 | uint32_t(y) >> 23 << 9);
        f.e = __int_as_float(dpp<0xFF>(word));  // quad_perm 3, 3, 3, 3
        active = (uint32_t(z) >> 23) != 0;
        word = j + 1 < n ? at[4 * (j + 1)] : 0;
        f.template read<FEAT>(g, c, g.rec + (uint64_t(uint32_t(f.rank) * uint32_t(g.rec_stride >> 8)) << 8) + g.dist_bytes);
    }
};

// Scattered lists: gradients through the wavefronts' logs, the next sample's
// voxels read before the current one's work.  Bound by the latency of those
// loads and by the longest of 8 rays.  65,536 rays, 1024^3, packed, walk
// included: one lane to a ray 2.35 ms, this 1.15.
constexpr int kListWaves = 4;

template <bool FEAT>
__global__ __launch_bounds__(64 * kListWaves) void k_backward_scattered(BackwardArgs a) {
    __shared__ int4 s_log[kListWaves][kLogEntries];
    __shared__ float s_gch[kListWaves][8][8];
    const GridArgs& g = a.grid;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const CornerLane c(g, lane);
    const int64_t i = (int64_t(blockIdx.x) * kListWaves + wave) * 8 + (lane >> 3);
    CornerRay<FEAT> st;
    bool going = st.setup(a, i, i < a.n_rays);
    s_gch[wave][lane >> 3][c.l] = st.channel(c.l);
    WaveLog<kLogEntries> log = {s_log[wave], s_gch[wave]};
    auto hand_over = [&](bool leave) {
        log.vi = st.template voxel<int32_t>(g, c, leave);
        log.A = st.A;
        log.Ds = g.sigma_scale * st.D;
    };
    ListReader<FEAT> rd;
    rd.init(a, c, i, going);
    for (int32_t j = 0; __any(going && j < rd.n); ++j) {
        if (going && j < rd.n) {
            const Fetched now = rd.f;
            const bool act = rd.active;
            if (j + 1 < rd.n) rd.load(g, c, j + 1);
            if (act && st.take(a, c, now, lane, hand_over)) going = false;
        }
        log.append(a, lane);
    }
    hand_over(st.wrank >= 0);
    log.append(a, lane);
    log.flush(a, lane);
}

// Patch lists: 64 neighbouring rays to a workgroup, 8 lanes to each, one listed
// sample to a step, their gradients summed in one table.  The table's new
// voxels get their slots as one lane per ray with compare-and-swaps would give
// them out, corner by corner, probe by probe, ray by ray (k_march_backward), so
// that the same hand-overs find the table full; but in all lanes at once.  A
// voxel without an entry asks for its first free slot, the slot goes to the
// earliest of those that ask (atomic minimum of corner, probe, ray), who lost
// it asks for the next, until nobody has to.  What finds no slot goes to the
// wavefront's log.  Bound by the longest of the patches, some 200 steps where
// rays graze the surface, and there by the step's chain of loads, LDS round
// trips and barriers.
//   16,384 rays, 512^3       one lane to a ray  2.0 ms   this 0.75 (+ 0.05 for the list)
//   262,144 rays, 512^3, whole backward call    8.0 ms        2.5
constexpr int kPatchWaves = 8;
constexpr int kPatchLog = 160;

template <bool FEAT>
__global__ __launch_bounds__(64 * kPatchWaves) void k_backward_patches(BackwardArgs a) {
    __shared__ int32_t s_key[kAggSlots];
    __shared__ float s_val[8 * kAggSlots];
    __shared__ unsigned long long s_ask[kAggSlots];  // the earliest that asks for the slot: order << 32 | voxel
    __shared__ int4 s_log[kPatchWaves][kPatchLog];
    __shared__ float s_gch[kPatchWaves][8][8];
    __shared__ int32_t s_on[3], s_again[3], s_used;
    const GridArgs& g = a.grid;
    for (int sl = threadIdx.x; sl < kAggSlots; sl += blockDim.x) {
        s_key[sl] = -1;
        s_ask[sl] = ~0ull;
#pragma unroll
        for (int ch = 0; ch < 8; ++ch) s_val[ch * kAggSlots + sl] = 0.0f;
    }
    if (threadIdx.x < 3) s_on[threadIdx.x] = s_again[threadIdx.x] = 0;
    if (threadIdx.x == 3) s_used = 0;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t base = int64_t(blockIdx.x) * 64;
    AggTable tab = {s_key, s_val, 0.0f, 0.0f};
    {  // every wavefront finds the table's scale, from all 64 rays
        float m = 0.0f;
        const int64_t i = base + lane;
        if (i < a.n_rays && a.aux[8 * i + 7] >= 0.0f) {
            const float* v = FEAT ? a.gcv + 8 * i : a.grad_rgba + 4 * i;
#pragma unroll
            for (int ch = 0; ch < (FEAT ? 7 : 3); ++ch) m = fmaxf(m, fabsf(v[ch]));
        }
        agg_scale(tab, wave_max(m));
    }
    const CornerLane c(g, lane);
    const int corner = c.cx | c.cy << 1 | c.cz << 2, ray = wave * 8 + (lane >> 3);
    CornerRay<FEAT> st;
    bool going = st.setup(a, base + ray, base + ray < a.n_rays);
    s_gch[wave][lane >> 3][c.l] = st.channel(c.l);
    WaveLog<kPatchLog> log = {s_log[wave], s_gch[wave]};
    ListReader<FEAT> rd;
    rd.init(a, c, base + ray, going);
    __syncthreads();

    // All threads: adds what the lanes with vi >= 0 hand over.
    int round = 0;
    auto enter = [&](int32_t vi, float A, float Ds) {
        const uint32_t h = agg_hash(vi);
        int pr = kAggProbes;
        bool mine = false, asks = false;
        if (vi >= 0) {
#pragma nounroll
            for (int p0 = 0; p0 < kAggProbes; p0 += 4) {  // four slots to a round trip
                int32_t k[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) k[u] = s_key[(h + uint32_t(p0 + u)) & (kAggSlots - 1)];
#pragma unroll
                for (int u = 3; u >= 0; --u) {
                    const bool end = k[u] == vi || k[u] == -1;
                    pr = end ? p0 + u : pr;
                    mine = end ? k[u] == vi : mine;
                }
                if (pr < kAggProbes) break;
            }
            asks = pr < kAggProbes && !mine;
        }
        int sl = int((h + uint32_t(pr)) & (kAggSlots - 1));
        bool won = false;
        for (;;) {
            // slots are looked up and asked for up to this barrier, read up to
            // the next and taken after it
            const uint32_t order = uint32_t(corner << 10 | pr << 6 | ray);
            if (asks) atomicMin(&s_ask[sl], (unsigned long long)(order) << 32 | uint32_t(vi));
            __syncthreads();
            bool lost = false;
            if (asks) {
                const unsigned long long first = s_ask[sl];
                won = uint32_t(first >> 32) == order;
                lost = uint32_t(first) != uint32_t(vi);
            }
            if (__any(lost) && lane == 0) s_again[round] = 1;
            const int next = round == 2 ? 0 : round + 1;
            if (threadIdx.x == 0) s_again[next] = 0;  // last read a barrier ago
            __syncthreads();
            const bool again = s_again[round] != 0;
            round = next;
            if (!again) break;
            if (lost) {
                do {
                    ++pr;
                    sl = (sl + 1) & (kAggSlots - 1);
                } while (pr < kAggProbes && s_key[sl] != -1);
                asks = pr < kAggProbes;
            }
        }
        if (asks && won) {
            s_key[sl] = vi;
            s_ask[sl] = ~0ull;
        }
        const int fresh = __builtin_popcountll(__ballot(asks && won));
        if (lane == 0 && fresh != 0) atomicAdd(&s_used, fresh);
        if (mine || asks) {
            agg_add<FEAT>(tab, sl, Ds, A, st.gC, st.gV);
        } else if (vi >= 0) {
            log.vi = vi;
            log.A = A;
            log.Ds = Ds;
        }
        log.append(a, lane);
        __syncthreads();
    };

    for (int32_t j = 0;; ++j) {
        const bool more = going && j < rd.n;
        int32_t vi = -1;
        float A = 0.0f, Ds = 0.0f;
        if (more) {
            const Fetched now = rd.f;
            const bool act = rd.active;
            if (j + 1 < rd.n) rd.load(g, c, j + 1);
            if (act) going = !st.take(a, c, now, lane, [&](bool leave) {
                vi = st.template voxel<int32_t>(g, c, leave);
                A = st.A;
                Ds = g.sigma_scale * st.D;
            });
        }
        if (__any(going && j + 1 < rd.n) && lane == 0) s_on[j % 3] = 1;
        if (threadIdx.x == 0) s_on[(j + 1) % 3] = 0;  // last read a step ago
        enter(vi, A, Ds);
        if (s_used >= kAggFlushAt) {
            __syncthreads();
            agg_flush<FEAT>(a, tab, threadIdx.x, blockDim.x);
            if (threadIdx.x == 0) s_used = 0;
            __syncthreads();
        }
        if (s_on[j % 3] == 0) break;
    }
    enter(st.template voxel<int32_t>(g, c, st.wrank >= 0), st.A, g.sigma_scale * st.D);
    log.flush(a, lane);
    agg_flush<FEAT>(a, tab, threadIdx.x, blockDim.x);
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
    const bool feat = a.mlp_mode != kMlpOff;
    auto check = [] { return hipGetLastError(); };
    // Eight lanes to a ray, walking.
    auto walk8_lds = [&](bool agg) {
        return (size_t(a.grid.n_words) + 1) / 2 * 16 +
               (agg ? size_t(kAggWords) * 4 : size_t(kAdjWaves) * kLogEntries * sizeof(int4));
    };
    auto walk8 = [&](bool agg) {
        const int64_t wgs = 2 * (a.ray_ids ? (a.n_rays + 63) / 64 : a.total_tiles);
        const size_t lds = walk8_lds(agg);
        static_assert(kAdjWaves * 8 == 32, "two workgroups to 64 rays");
        constexpr int64_t kMaxGroups = int64_t(1) << 22;  // a launch holds fewer than 2^32 lanes
        BackwardArgs b = a;
        for (b.first_group = 0; b.first_group < wgs; b.first_group += kMaxGroups) {
            const dim3 n{unsigned(wgs - b.first_group < kMaxGroups ? wgs - b.first_group : kMaxGroups)};
            const dim3 wg{64 * kAdjWaves};
            if (feat && agg) hipLaunchKernelGGL((k_adjoint<true, true>), n, wg, lds, s, b);
            else if (feat) hipLaunchKernelGGL((k_adjoint<true, false>), n, wg, lds, s, b);
            else if (agg) hipLaunchKernelGGL((k_adjoint<false, true>), n, wg, lds, s, b);
            else hipLaunchKernelGGL((k_adjoint<false, false>), n, wg, lds, s, b);
            if ((e = check()) != hipSuccess) return e;
        }
        return hipSuccess;
    };
    // One lane to a ray, walking.
    auto walk1 = [&]() {
        const size_t lds = size_t(a.grid.n_words) * sizeof(uint2) + size_t(kAggLdsWords) * 4;
        const int64_t waves = a.ray_ids ? (a.n_rays + 63) / 64 : a.total_tiles;
        const dim3 n{unsigned((waves + kAggWaves - 1) / kAggWaves)}, wg{64 * kAggWaves};
        if (feat) hipLaunchKernelGGL(k_march_backward<true>, n, wg, lds, s, a);
        else hipLaunchKernelGGL(k_march_backward<false>, n, wg, lds, s, a);
        return check();
    };
    switch (backward_route(backward_aggregates(a.grid), a.list != nullptr, a.ray_ids != nullptr, a.patch_rays != 0,
                           a.dense_views != 0, int64_t(walk8_lds(true)) + kAdjStaticLds,
                           a.ray_ids ? a.n_rays : 64 * a.total_tiles)) {
        case BackwardRoute::kLogs: return walk8(false);
        case BackwardRoute::kEightLanes: return walk8(true);
        case BackwardRoute::kOneLane: return walk1();
        case BackwardRoute::kListed: break;
    }
    const size_t occ = size_t(a.grid.n_words) * sizeof(uint2);
    const unsigned threads = 4 * int64_t(occ) <= kCuLds ? 256 : 1024;
    const dim3 n{unsigned((a.n_rays * kRecordLanes + threads - 1) / threads)}, wg{threads};
    hipLaunchKernelGGL(k_backward_record, n, wg, occ, s, a);
    if ((e = check()) != hipSuccess) return e;
    if (a.patch_rays) {
        const dim3 n{unsigned((a.n_rays + 63) / 64)}, wg{64 * kPatchWaves};
        if (feat) hipLaunchKernelGGL(k_backward_patches<true>, n, wg, 0, s, a);
        else hipLaunchKernelGGL(k_backward_patches<false>, n, wg, 0, s, a);
    } else {
        const dim3 n{unsigned((a.n_rays + 8 * kListWaves - 1) / (8 * kListWaves))}, wg{64 * kListWaves};
        if (feat) hipLaunchKernelGGL(k_backward_scattered<true>, n, wg, 0, s, a);
        else hipLaunchKernelGGL(k_backward_scattered<false>, n, wg, 0, s, a);
    }
    if ((e = check()) != hipSuccess) return e;
    // the rays with more samples than the list holds
    return a.patch_rays ? walk1() : walk8(false);
}

hipError_t launch_reduce_mlp(const float* partial, int rows, float* out, hipStream_t s) {
    const dim3 grid((kMlpParams + 63) / 64, (rows + kReduceRows - 1) / kReduceRows);
    hipLaunchKernelGGL(k_reduce_rows, grid, dim3(256), 0, s, partial, rows, out);
    return hipGetLastError();
}

}  // namespace snerg
