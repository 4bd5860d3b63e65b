// Learned work estimator for the group walk: a multilayer perceptron
// 8 -> 64 -> 64 -> 1 (ReLU) mapping a group's geometry to
// log2(1 + n_pc + n_pp), the length of its interaction lists.  Weights are
// stored in float16, arithmetic accumulates in float32.  Training kernels
// (forward, backward, Adam) run on the GPU; the backward pass is
// deterministic (per-block outer products summed in a fixed order, then a
// fixed-order sum over blocks).  The prediction orders the walk's group
// queue, heaviest predicted work first.
#include "mibh_device.h"

#include <hip/hip_fp16.h>

namespace mibh {

// parameter layout: W1[64][8], b1[64], W2[64][64], b2[64], w3[64], b3
constexpr int OFF_W1 = 0, OFF_B1 = MLP_H * MLP_IN, OFF_W2 = OFF_B1 + MLP_H, OFF_B2 = OFF_W2 + MLP_H * MLP_H,
              OFF_W3 = OFF_B2 + MLP_H, OFF_B3 = OFF_W3 + MLP_H;
static_assert(OFF_B3 + 1 == MLP_NPARAM, "parameter layout");

// --------------------------------------------------------------------------
// Features of each group (one thread per group): particle count, bounding
// extent and distance to the system's centre of mass (in root-cube units),
// local density relative to the system's mean, theta, group level, system
// size.  All are O(1) by construction so that no data-dependent
// normalisation is needed.  The group's box is gathered 8 particles per round
// with the indices clamped to the group's last particle (a repeated particle
// leaves a minimum or maximum unchanged), so each round issues its 8 loads at
// once and a group of n particles takes ceil(n / 8) round trips.
// --------------------------------------------------------------------------

constexpr unsigned FEAT_BATCH = 8;

__global__ __launch_bounds__(256) void k_features(const Header *__restrict__ hdr, const SysCube *__restrict__ cube,
                                                  const uint2 *__restrict__ groups, const uint4 *__restrict__ topo,
                                                  const float4 *__restrict__ spos, const double *__restrict__ mp,
                                                  float theta, float *__restrict__ feat) {
    const unsigned ng = hdr->ngroups;
    for (unsigned g = blockIdx.x * 256u + threadIdx.x; g < ng; g += gridDim.x * 256u) {
        const uint2 gr = groups[g];
        const unsigned gf = gr.x, gn = gr.y & 255u, glev = (gr.y >> 8) & 255u, sys = gr.y >> 16;
        float3 bmin = make_float3(INFINITY, INFINITY, INFINITY), bmax = make_float3(-INFINITY, -INFINITY, -INFINITY);
        for (unsigned j0 = 0; j0 < gn; j0 += FEAT_BATCH) {
            float4 p[FEAT_BATCH];
#pragma unroll
            for (unsigned u = 0; u < FEAT_BATCH; u++) p[u] = spos[gf + min(j0 + u, gn - 1u)];
#pragma unroll
            for (unsigned u = 0; u < FEAT_BATCH; u++) {
                bmin.x = fminf(bmin.x, p[u].x); bmin.y = fminf(bmin.y, p[u].y); bmin.z = fminf(bmin.z, p[u].z);
                bmax.x = fmaxf(bmax.x, p[u].x); bmax.y = fmaxf(bmax.y, p[u].y); bmax.z = fmaxf(bmax.z, p[u].z);
            }
        }
        const float L = ldexpf(1.0f, cube[sys].k);
        const float ext = fmaxf(fmaxf(bmax.x - bmin.x, bmax.y - bmin.y), bmax.z - bmin.z);
        const double *root = mp + 10 * (size_t)sys;  // level-0 cell of system sys
        const float cx = 0.5f * (bmin.x + bmax.x) - (float)root[1];
        const float cy = 0.5f * (bmin.y + bmax.y) - (float)root[2];
        const float cz = 0.5f * (bmin.z + bmax.z) - (float)root[3];
        const float dist = sqrtf(cx * cx + cy * cy + cz * cz);
        const float nsys_particles = (float)topo[sys].y;
        const float e = fmaxf(ext, L * 9.5367431640625e-07f) / L;  // at least one finest cell
        float *f = feat + (size_t)g * MLP_IN;
        f[0] = log2f((float)gn) / 6.0f;
        f[1] = log2f(ext / L + 5.9604645e-08f) / 24.0f;
        f[2] = log2f(dist / L + 5.9604645e-08f) / 24.0f;
        f[3] = log2f(((float)gn / nsys_particles) / (e * e * e)) / 32.0f;
        f[4] = theta;
        f[5] = (float)glev / 20.0f;
        f[6] = log2f(nsys_particles) / 24.0f;
        f[7] = log2f(theta);
    }
}

// --------------------------------------------------------------------------
// Forward pass, one row per thread; weights converted once into LDS and read
// back as wave-uniform (broadcast) loads.  The hidden layers run as outer
// products: hidden unit j of the first layer is computed on its own, then
// added into the 64 second-layer sums, whose weights W2[.][j] sit transposed
// in LDS (16 broadcast loads of 4).  Each sum keeps the order of its dot
// product (bias first, then j = 0..63), so the predictions equal those of
// plain dot products bit for bit.  A fully unrolled first layer made the
// compiler keep 488 registers (one wave per SIMD); this form takes 221 (two
// waves per SIMD; bounds asking for three or four waves make it spill).
// --------------------------------------------------------------------------

// LDS image for the forward pass: W1, b1 as stored, W2 transposed, b2, w3, b3.
static_assert(OFF_W2 % 4 == 0, "float4 reads of the transposed second layer");
constexpr int FWD_W2T = OFF_W2;

__device__ __forceinline__ void load_weights_fwd(const __half *__restrict__ w16, float *s_w) {
    for (int i = threadIdx.x; i < MLP_NPARAM; i += blockDim.x) {
        int d = i;
        if (i >= OFF_W2 && i < OFF_B2) {  // W2[r][c] -> W2T[c][r]
            const int r = (i - OFF_W2) / MLP_H, c = (i - OFF_W2) % MLP_H;
            d = FWD_W2T + c * MLP_H + r;
        }
        s_w[d] = __half2float(w16[i]);
    }
    __syncthreads();
}

__global__ __launch_bounds__(256) void k_mlp_fwd(const __half *__restrict__ w16, const float *__restrict__ x,
                                                 unsigned rows, const Header *__restrict__ hdr,
                                                 float *__restrict__ y) {
    __shared__ __align__(16) float s_w[MLP_NPARAM];
    load_weights_fwd(w16, s_w);
    const unsigned nrows = hdr ? hdr->ngroups : rows;
    for (unsigned r = blockIdx.x * 256u + threadIdx.x; r < nrows; r += gridDim.x * 256u) {
        float xi[MLP_IN], h2[MLP_H];
#pragma unroll
        for (int k = 0; k < MLP_IN; k++) xi[k] = x[(size_t)r * MLP_IN + k];
#pragma unroll
        for (int i = 0; i < MLP_H; i++) h2[i] = s_w[OFF_B2 + i];
#pragma nounroll
        for (int j = 0; j < MLP_H; j++) {
            float a = s_w[OFF_B1 + j];
#pragma unroll
            for (int k = 0; k < MLP_IN; k++) a = fmaf(s_w[OFF_W1 + j * MLP_IN + k], xi[k], a);
            const float h1j = fmaxf(a, 0.0f);
            const float4 *col = reinterpret_cast<const float4 *>(s_w + FWD_W2T + j * MLP_H);
#pragma unroll
            for (int q = 0; q < MLP_H / 4; q++) {
                const float4 w = col[q];
                h2[4 * q] = fmaf(w.x, h1j, h2[4 * q]);
                h2[4 * q + 1] = fmaf(w.y, h1j, h2[4 * q + 1]);
                h2[4 * q + 2] = fmaf(w.z, h1j, h2[4 * q + 2]);
                h2[4 * q + 3] = fmaf(w.w, h1j, h2[4 * q + 3]);
            }
        }
        float out = s_w[OFF_B3];
#pragma unroll
        for (int i = 0; i < MLP_H; i++) out = fmaf(s_w[OFF_W3 + i], fmaxf(h2[i], 0.0f), out);
        y[r] = out;
    }
}

// --------------------------------------------------------------------------
// Backward pass of the mean squared error over a batch of sampled rows.  A
// workgroup of four waves takes tiles of 16 samples; the 64-wide products (second
// layer forward, its transpose backward, the second layer's weight gradient) run
// on the float32 matrix instruction (16 x 16 outputs, 4 terms), wave w for hidden
// units 16 w .. 16 w + 15, and the weight gradients stay in its accumulators over
// the workgroup's tiles.  Partial gradients per workgroup are then summed in a
// fixed order.
// What bounds it is latency: a batch of 1024 is 64 tiles, about ten dependent
// LDS and matrix steps each.  With one thread per sample and 64 samples per
// workgroup, 16 workgroups ran 64-term loops out of LDS for 84 us.
// The error of the gradient against float64 (l2, mean of 12 seeds) is a third of
// that form's: 4.9e-8 (1.5e-7) at a batch of 1024, 1.3e-7 (7.7e-7) at 64.
// --------------------------------------------------------------------------

constexpr int GT = 16;            // samples per tile
constexpr int GRAD_THREADS = 256;
constexpr unsigned GRAD_BLOCKS = 1024;  // workgroups at most: larger batches take several tiles each
constexpr int GP = MLP_H + 4;     // row pitch of the activations in LDS

typedef float f32x4 __attribute__((ext_vector_type(4)));

inline unsigned grad_blocks(unsigned batch) { return min((batch + GT - 1u) / GT, GRAD_BLOCKS); }

// acc += A B, one 16 x 16 tile over 64 terms: A row l & 15 from ap (stride 1 in
// the term), B column from bp (stride bs).  Lane l takes terms (l >> 4) * 16 + s
// in step s: any order of the terms will do as long as A and B agree.
template <typename T>
__device__ __forceinline__ f32x4 mfma_64(const float *ap, const T *bp, int bs, f32x4 acc) {
    const int k0 = (int)(threadIdx.x >> 4 & 3u) * 16;
#pragma unroll
    for (int s = 0; s < 16; s++)
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(ap[k0 + s], (float)bp[(k0 + s) * bs], acc, 0, 0, 0);
    return acc;
}

__global__ __launch_bounds__(GRAD_THREADS) void k_mlp_grad(const __half *__restrict__ w16, const float *__restrict__ x,
                                                           const float *__restrict__ target,
                                                           const int *__restrict__ idx, unsigned batch,
                                                           float *__restrict__ partial,
                                                           float *__restrict__ loss_part) {
    static_assert(MLP_H == 64 && MLP_IN == 8 && GRAD_THREADS == 256, "one wave per 16 hidden units");
    __shared__ _Float16 s_w[MLP_NPARAM + 1];
    __shared__ float s_x[GT][MLP_IN], s_h1[GT][GP], s_h2[GT][GP], s_d2[GT][GP], s_d1[GT][GP];
    __shared__ float s_dy[GT], s_e2[GT], s_t[GT];
    const int t = (int)threadIdx.x, w = t >> 6, ln = t & 63, col = ln & 15, quad = ln >> 4;
    const _Float16 *w16f = reinterpret_cast<const _Float16 *>(w16);
    for (int i = t; i < MLP_NPARAM; i += GRAD_THREADS) s_w[i] = w16f[i];
    const unsigned tiles = (batch + GT - 1u) / GT;
    f32x4 g2[4] = {};                 // dW2[16 w + 4 quad + r][16 c + col]
    float g1[2] = {0.0f, 0.0f};       // dW1 of parameters t, t + 256
    float gb = 0.0f, gl = 0.0f;       // t < 64 b1, < 128 b2, < 192 w3, 192 b3; 193 loss
    for (unsigned tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        if (t < GT * MLP_IN) {
            const unsigned s = tile * GT + (unsigned)t / MLP_IN;
            const bool valid = s < batch;
            const int row = valid ? idx[s] : 0;
            s_x[t / MLP_IN][t % MLP_IN] = valid ? x[(size_t)row * MLP_IN + t % MLP_IN] : 0.0f;
            if (t % MLP_IN == 0) s_t[t / MLP_IN] = valid ? target[row] : 0.0f;
        }
        __syncthreads();
        // first layer: unit ln of samples 4 w .. 4 w + 3
#pragma unroll
        for (int q = 0; q < 4; q++) {
            float a = (float)s_w[OFF_B1 + ln];
#pragma unroll
            for (int k = 0; k < MLP_IN; k++) a = fmaf((float)s_w[OFF_W1 + ln * MLP_IN + k], s_x[4 * w + q][k], a);
            s_h1[4 * w + q][ln] = fmaxf(a, 0.0f);
        }
        __syncthreads();
        // second layer: units 16 w + col; rows of the result are samples 4 quad + r
        const int u = 16 * w + col;
        {
            const float b = (float)s_w[OFF_B2 + u];
            f32x4 h = {b, b, b, b};
            h = mfma_64(s_h1[col], s_w + OFF_W2 + u * MLP_H, 1, h);
#pragma unroll
            for (int r = 0; r < 4; r++) s_h2[4 * quad + r][u] = fmaxf(h[r], 0.0f);
        }
        __syncthreads();
        // output, error and its derivative: sample t >> 4, 4 units per lane
        {
            const int q = t >> 4;
            float y = 0.0f;
#pragma unroll
            for (int k = 0; k < 4; k++) y = fmaf((float)s_w[OFF_W3 + col + 16 * k], s_h2[q][col + 16 * k], y);
#pragma unroll
            for (int o = 8; o > 0; o >>= 1) y += __shfl_xor(y, o, 16);
            y += (float)s_w[OFF_B3];
            const float err = tile * GT + (unsigned)q < batch ? y - s_t[q] : 0.0f;
            const float dy = 2.0f * err / (float)batch;
            s_dy[q] = dy;  // the same value from 16 lanes
            s_e2[q] = err * err;
#pragma unroll
            for (int k = 0; k < 4; k++) {
                const int i = col + 16 * k;
                s_d2[q][i] = s_h2[q][i] > 0.0f ? dy * (float)s_w[OFF_W3 + i] : 0.0f;
            }
        }
        __syncthreads();
        // deltas of the first layer, units u
        {
            f32x4 d = {};
            d = mfma_64(s_d2[col], s_w + OFF_W2 + u, MLP_H, d);
#pragma unroll
            for (int r = 0; r < 4; r++) s_d1[4 * quad + r][u] = s_h1[4 * quad + r][u] > 0.0f ? d[r] : 0.0f;
        }
        // second layer's weight gradient: rows 16 w .., over the tile's 16 samples
#pragma unroll
        for (int c = 0; c < 4; c++)
#pragma unroll
            for (int s = 0; s < 4; s++)
                g2[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(s_d2[4 * s + quad][16 * w + col],
                                                             s_h1[4 * s + quad][16 * c + col], g2[c], 0, 0, 0);
        __syncthreads();
        // the others, one or two parameters per thread
#pragma unroll
        for (int p = 0; p < 2; p++) {
            const int i = (t + 256 * p) / MLP_IN, k = t % MLP_IN;
#pragma unroll
            for (int q = 0; q < GT; q++) g1[p] = fmaf(s_d1[q][i], s_x[q][k], g1[p]);
        }
        if (t < 64) {
            for (int q = 0; q < GT; q++) gb += s_d1[q][t];
        } else if (t < 128) {
            for (int q = 0; q < GT; q++) gb += s_d2[q][t - 64];
        } else if (t < 192) {
            for (int q = 0; q < GT; q++) gb = fmaf(s_dy[q], s_h2[q][t - 128], gb);
        } else if (t == 192) {
            for (int q = 0; q < GT; q++) gb += s_dy[q];
        } else if (t == 193) {
            for (int q = 0; q < GT; q++) gl += s_e2[q];
        }
        __syncthreads();
    }
    float *out = partial + (size_t)blockIdx.x * MLP_NPARAM;
#pragma unroll
    for (int c = 0; c < 4; c++)
#pragma unroll
        for (int r = 0; r < 4; r++) out[OFF_W2 + (16 * w + 4 * quad + r) * MLP_H + 16 * c + col] = g2[c][r];
    out[OFF_W1 + t] = g1[0];
    out[OFF_W1 + 256 + t] = g1[1];
    if (t < 64) out[OFF_B1 + t] = gb;
    else if (t < 128) out[OFF_B2 + t - 64] = gb;
    else if (t < 192) out[OFF_W3 + t - 128] = gb;
    else if (t == 192) out[OFF_B3] = gb;
    else if (t == 193) loss_part[blockIdx.x] = gl;
}

// Sums the workgroups' partials: 16 parameters per workgroup, 16 threads per
// parameter over the partials 16 apart, then those 16 sums in a fixed tree.  The
// last workgroup sums the loss the same way.
__global__ __launch_bounds__(256) void k_mlp_reduce(const float *__restrict__ partial, unsigned nblk,
                                                    const float *__restrict__ loss_part, unsigned batch,
                                                    float *__restrict__ grad, float *__restrict__ loss) {
    __shared__ float s[16][17];
    const unsigned c = threadIdx.x & 15u, r = threadIdx.x >> 4;
    const bool is_loss = blockIdx.x == gridDim.x - 1u;
    const unsigned p = blockIdx.x * 16u + c;
    const float *src = is_loss ? loss_part : partial + p;
    const size_t stride = is_loss ? 1u : (size_t)MLP_NPARAM;
    float a = 0.0f;
    if (is_loss ? c == 0u : p < (unsigned)MLP_NPARAM) {
#pragma unroll 4
        for (unsigned b = r; b < nblk; b += 16u) a += src[b * stride];
    }
    s[r][c] = a;
    __syncthreads();
    a = s[c][r];  // lane c of a row of 16: partial sum c of parameter r
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) a += __shfl_xor(a, o, 16);
    if (c == 0u) {
        if (!is_loss && blockIdx.x * 16u + r < (unsigned)MLP_NPARAM) grad[blockIdx.x * 16u + r] = a;
        if (is_loss && r == 0u && loss) *loss = a / (float)batch;
    }
}

// Adam (Kingma & Ba 2015) on float32 master weights; float16 copies for the kernels.
__global__ __launch_bounds__(256) void k_adam(float *__restrict__ w32, __half *__restrict__ w16,
                                              const float *__restrict__ grad, float *__restrict__ m,
                                              float *__restrict__ v, float lr, float beta1, float beta2,
                                              float eps, float corr1, float corr2) {
    for (unsigned p = blockIdx.x * 256u + threadIdx.x; p < (unsigned)MLP_NPARAM; p += gridDim.x * 256u) {
        const float g = grad[p];
        const float mp = beta1 * m[p] + (1.0f - beta1) * g;
        const float vp = beta2 * v[p] + (1.0f - beta2) * g * g;
        m[p] = mp;
        v[p] = vp;
        const float w = w32[p] - lr * (mp / corr1) / (sqrtf(vp / corr2) + eps);
        w32[p] = w;
        w16[p] = __float2half(w);
    }
}

hipError_t launch_features(const Buffers &b, float theta, float *feat, hipStream_t s) {
    const unsigned grid = min((b.n_max + 255u) / 256u, 2048u);
    hipLaunchKernelGGL(k_features, dim3(grid), dim3(256), 0, s, b.hdr, b.cube, b.groups, b.topo, b.spos, b.mp, theta,
                       feat);
    return hipGetLastError();
}

hipError_t launch_mlp_forward(const void *w16, const float *x, unsigned rows, const Header *hdr, float *y,
                              hipStream_t s) {
    const unsigned grid = min(max((rows + 255u) / 256u, 1u), 1024u);
    hipLaunchKernelGGL(k_mlp_fwd, dim3(hdr ? 1024u : grid), dim3(256), 0, s, (const __half *)w16, x, rows, hdr, y);
    return hipGetLastError();
}

size_t mlp_scratch_bytes(unsigned batch) {
    const size_t nblk = grad_blocks(batch);
    return nblk * MLP_NPARAM * sizeof(float) + nblk * sizeof(float) + 256;
}

hipError_t launch_mlp_grad(const void *w16, const float *x, const float *target, const int *idx, unsigned batch,
                           float *grad, float *loss, void *scratch, hipStream_t s) {
    const unsigned nblk = grad_blocks(batch);
    float *partial = (float *)scratch;
    float *loss_part = partial + (size_t)nblk * MLP_NPARAM;
    hipLaunchKernelGGL(k_mlp_grad, dim3(nblk), dim3(GRAD_THREADS), 0, s, (const __half *)w16, x, target, idx, batch,
                       partial, loss_part);
    hipLaunchKernelGGL(k_mlp_reduce, dim3((MLP_NPARAM + 15) / 16 + 1), dim3(256), 0, s, partial, nblk, loss_part,
                       batch, grad, loss);
    return hipGetLastError();
}

hipError_t launch_adam(float *w32, void *w16, const float *grad, float *m, float *v, int step, float lr,
                       float beta1, float beta2, float eps, hipStream_t s) {
    const float corr1 = 1.0f - powf(beta1, (float)step), corr2 = 1.0f - powf(beta2, (float)step);
    hipLaunchKernelGGL(k_adam, dim3((MLP_NPARAM + 255) / 256), dim3(256), 0, s, w32, (__half *)w16, grad, m, v, lr,
                       beta1, beta2, eps, corr1, corr2);
    return hipGetLastError();
}

}  // namespace mibh
