// First convolution (Section 5.1: 32 filters of 4x8x8, stride 4, ReLU) on the
// raw uint8 frames, forward and weight gradient.  Bytes enter the products as
// exact integers; the 1/255 input scale is applied once in each epilogue.
#include "common.h"
#include "conv1_wgrad.h"
#include "kernels.h"
#include "planes.h"

#include <type_traits>

namespace gorila {

// The layer on v_mfma_f32_32x32x16_bf16 with exact products: the bytes
// (integers 0..255) are exact bf16 values, and W1 enters as WP bf16 planes
// whose sum is W1 exactly -- one plane for bf16 parameter sets; for fp32 sets
// three (w = hi + mid + lo, each the rounded remainder of the previous: 8 + 8
// + 8 significant bits cover fp32's 24; exact for |w| above ~2^-90), so every
// product is exact and only the fp32 accumulation rounds, as in an fp32 GEMM.  A workgroup of 13 waves
// keeps the planes in LDS and walks samples b = blockIdx.x, b + gridDim.x,
// ... of its parameter set: it converts a sample's 4 frames to bf16 once, into
// LDS, fetches the next sample's frames into registers while wave t computes
// pixel tile t (32 pixels x 32 filters; the 13th tile is half full).  One
// 16-wide MFMA step covers two filter rows (c, u) of 8 columns v: lane half h
// takes row 2 * step + h, so a lane's eight operands are eight consecutive
// bf16 pixels of one input row.
constexpr int C1F_WAVES = (P1 + 31) / 32;  // 13
constexpr int C1F_THREADS = 64 * C1F_WAVES;
constexpr int C1F_WLD = 256 + 8;           // W1 row stride in LDS (bf16): 528 bytes
constexpr int C1F_XV = STATE_BYTES / 16;   // 1764 16-byte vectors per sample
constexpr int C1F_XPT = (C1F_XV + C1F_THREADS - 1) / C1F_THREADS;
// resident workgroups: two per CU with one plane (73 KB of LDS), one with three
__host__ __device__ constexpr int c1f_target_wgs(int wp) { return wp == 1 ? 512 : 256; }

template <int WP>
__launch_bounds__(C1F_THREADS) __global__ void conv1_fwd_mfma16_kernel(
    const uint8_t* const* __restrict__ ftab, GroupPtrs theta, int n, float* __restrict__ h1) {
    __shared__ __attribute__((aligned(16))) __bf16 xs[STATE_BYTES];
    __shared__ __attribute__((aligned(16))) __bf16 ws[WP][C1 * C1F_WLD];
    __shared__ float bs[C1];
    const int g = blockIdx.y;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const float* W1 = theta.p[g];

    uint4 xv[C1F_XPT];
    unsigned okm = 0;  // bit k: xv[k] holds frame bytes (else zeros)
    // The sample's 16-byte vectors of this thread.  Branch-free, so all of
    // them are in flight together: the four frame pointers are read first (the
    // same for every thread), a null frame reads W1 instead and is zeroed when
    // converted (not here, which would wait for the loads).
    auto fetch = [&](int b) {
        const uint8_t* const* fr = ftab + ((int64_t)g * n + b) * 4;
        const uint8_t* f0 = fr[0];
        const uint8_t* f1 = fr[1];
        const uint8_t* f2 = fr[2];
        const uint8_t* f3 = fr[3];
#pragma unroll
        for (int k = 0; k < C1F_XPT; ++k) {
            const int e = tid + k * C1F_THREADS;  // vector e: frame e / 441
            const int fi = e / (FRAME_BYTES / 16);
            const uint8_t* f = fi == 0 ? f0 : fi == 1 ? f1 : fi == 2 ? f2 : f3;
            const bool ok = e < C1F_XV && f != nullptr;
            xv[k] = ldg_u4(ok ? (const uint4*)f + (e - fi * (FRAME_BYTES / 16))
                              : (const uint4*)(W1 + OFF_W1));
            okm = k == 0 ? (unsigned)ok : okm | ((unsigned)ok << k);
        }
    };
    fetch(blockIdx.x);

    constexpr int WQ = C1 * 256 / 4;  // 2048 weight quads
    for (int q = tid; q < WQ; q += C1F_THREADS) {
        f32x4 w = ld4(W1 + OFF_W1 + 4 * q);
#pragma unroll
        for (int pl = 0; pl < WP; ++pl) {
            bf16x4 v;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                v[i] = (__bf16)w[i];
                w[i] -= (float)v[i];  // exact: the remainder has at most 16 significant bits
            }
            *(bf16x4*)(ws[pl] + (q >> 6) * C1F_WLD + 4 * (q & 63)) = v;
        }
    }
    if (tid < C1) bs[tid] = W1[OFF_B1 + tid];
    const int col = lane & 31, h = lane >> 5;

    int m = wave * 32 + (lane & 31);
    if (m >= P1) m = 0;  // padding rows compute on a valid pixel, never stored
    const int i = m / H1, j = m - i * H1;
    const __bf16* xb = xs + (S1 * i) * IN_W + S1 * j;  // 8-byte aligned
    const int wofs = col * C1F_WLD + 8 * h;             // 16-byte aligned

    for (int b = blockIdx.x; b < n; b += gridDim.x) {
#pragma unroll
        for (int k = 0; k < C1F_XPT; ++k) {
            const int e = tid + k * C1F_THREADS;
            if (e < C1F_XV) {
                const uint4 v = (okm >> k) & 1u ? xv[k] : make_uint4(0, 0, 0, 0);
                const uint32_t d[4] = {v.x, v.y, v.z, v.w};
                bf16x8 lo, hi;
#pragma unroll
                for (int t = 0; t < 8; ++t) {
                    lo[t] = (__bf16)(float)((d[t >> 2] >> (8 * (t & 3))) & 255u);
                    hi[t] = (__bf16)(float)((d[2 + (t >> 2)] >> (8 * (t & 3))) & 255u);
                }
                *(bf16x8*)(xs + 16 * e) = lo;
                *(bf16x8*)(xs + 16 * e + 8) = hi;
            }
        }
        __syncthreads();
        if (b + (int)gridDim.x < n) fetch(b + gridDim.x);  // in flight during the products

        f32x16 acc = f32x16{};
#pragma unroll
        for (int st = 0; st < 16; ++st) {
            const int cb = 2 * st + h, c = cb >> 3, u = cb & 7;
            const __bf16* px = xb + c * FRAME_BYTES + u * IN_W;
            const bf16x4 x0 = *(const bf16x4*)px, x1 = *(const bf16x4*)(px + 4);
            const bf16x8 x = __builtin_shufflevector(x0, x1, 0, 1, 2, 3, 4, 5, 6, 7);
#pragma unroll
            for (int pl = 0; pl < WP; ++pl) {
                const bf16x8 w = *(const bf16x8*)(ws[pl] + wofs + 16 * st);
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x, w, acc, 0, 0, 0);
            }
        }
        float* out = h1 + ((int64_t)g * n + b) * P1 * C1 + (wave * 32 + 4 * h) * C1 + col;
        const float bias = bs[col];
        if (wave < C1F_WAVES - 1) {  // full tiles: no per-store conditions
#pragma unroll
            for (int r = 0; r < 16; ++r)
                out[(8 * (r >> 2) + (r & 3)) * C1] = fmaxf(acc[r] * (1.0f / 255.0f) + bias, 0.0f);
        } else {
#pragma unroll
            for (int r = 0; r < 16; ++r)
                if (wave * 32 + 8 * (r >> 2) + 4 * h + (r & 3) < P1)
                    out[(8 * (r >> 2) + (r & 3)) * C1] = fmaxf(acc[r] * (1.0f / 255.0f) + bias, 0.0f);
        }
        __syncthreads();  // every wave is done with xs before the next sample lands
    }
}

void launch_conv1_fwd(const uint8_t* const* ftab, const GroupPtrs& theta, int groups, int n,
                      float* h1, bool bf16, hipStream_t st) {
    if (n <= 0) return;
    // one round of resident workgroups, each walking its set's samples
    if (bf16) {
        const int per_group = max(1, min(n, c1f_target_wgs(1) / groups));
        conv1_fwd_mfma16_kernel<1><<<dim3(per_group, groups), C1F_THREADS, 0, st>>>(ftab, theta, n, h1);
    } else {
        const int per_group = max(1, min(n, c1f_target_wgs(3) / groups));
        conv1_fwd_mfma16_kernel<3><<<dim3(per_group, groups), C1F_THREADS, 0, st>>>(ftab, theta, n, h1);
    }
}
template <int WP>
__global__ __launch_bounds__(64 * C1W_WAVES) void conv1_wgrad_mfma16_kernel(
    const C1wDz<WP>* __restrict__ dz1, const uint8_t* const* __restrict__ ftab,
    const uint8_t* __restrict__ zero_frame, int n, int SP, float* __restrict__ partial,
    float* __restrict__ bias_part) {
    __shared__ __attribute__((aligned(16))) char smem[C1W_LDS];
    conv1_wgrad_run<WP>(smem, blockIdx.x, blockIdx.y, dz1, ftab, zero_frame, n, SP, partial, bias_part);
}

void launch_conv1_wgrad(const float* dz1, const uint8_t* const* ftab, const uint8_t* zero_frame,
                        int groups, int n, float* partial, float* bias_part, int max_splits,
                        int* splits_out, bool bf16, hipStream_t st) {
    if (n <= 0) {
        *splits_out = 0;
        return;
    }
    // workgroup pairs (one workgroup per channel pair) per group: one
    // workgroup per CU in all, each of whose waves gets at least one unit;
    // groups * pairs stays within max_splits (a pair writes one partial)
    const int splits = max(1, min((n * C1W_UNITS + C1W_WAVES - 1) / C1W_WAVES,
                                  min(C1W_WGS / 2, max_splits) / groups));
    *splits_out = splits;
    // the pairs in groups of eight: 16 blocks each, the kernel's block order
    const int blocks = 2 * pad_xcd(splits);
    if (bf16)
        conv1_wgrad_mfma16_kernel<1><<<dim3(blocks, groups), 64 * C1W_WAVES, 0, st>>>(
            (const uint16_t*)dz1, ftab, zero_frame, n, splits, partial, bias_part);
    else
        conv1_wgrad_mfma16_kernel<3><<<dim3(blocks, groups), 64 * C1W_WAVES, 0, st>>>(
            dz1, ftab, zero_frame, n, splits, partial, bias_part);
}

}  // namespace gorila
