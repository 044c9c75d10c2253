// The three convolutions forward (Section 5.1: 32@8x8 stride 4, 64@4x4 stride
// 2, 64@3x3 stride 1, ReLU after each) as one launch.  A workgroup takes one
// sample at a time from its four frames to h3 with every activation between in
// LDS, so h1 and h2 never reach memory, and a forward pass has two launches
// fewer than layer by layer.
//
// Products.  v_mfma_f32_16x16x32_bf16 with every operand as bf16 planes whose
// sum is the value: an fp32 weight or activation is hi + mid + lo, each the
// rounded remainder of the previous, 8 + 8 + 8 significant bits (exact above
// ~2^-110); the input bytes and bf16 weights are one plane, exact.  Of the nine
// plane products of two fp32 operands the three below 2^-24 of the value
// (mid*lo, lo*mid, lo*lo) are left out.  Each product is exact in fp32, so only
// the accumulation rounds; the leading product has an accumulator of its own
// and the others share a second, so the long sum takes one rounding per 32
// terms, not one per 2 as the fp32 instruction's does.  Against 64 bits the
// error of Q is below that of fp32 MFMA products.
//
// Why bf16 planes: the fp32 matrix instruction runs at 1/16 of the bf16 rate,
// so six products cost 3/8 of its time.  Why one sample a workgroup: the
// layers' patches overlap (an h1 value is read by four conv2 outputs, an h2
// value by up to nine of conv3), and three planes take 6 bytes a value, so
// tiles staged through LDS per layer would be bound by LDS and L2 traffic.
// Here an activation is stored to LDS once and the weights stream from the
// XCD's L2 straight into registers in operand order (prep_weights_part), 456
// KB a sample with three planes.
//
// Measured against the three layer launches: 1024 fp32 states 106 -> 70 us, one
// state 27 -> 17 us.  A sample takes 33.5 thousand cycles, 21.1 of them matrix
// instructions (six plane products); the rest is the epilogues' splits and
// stores and the waits at the layers' barriers, with one workgroup a unit (LDS).
#include "common.h"
#include "kernels.h"
#include "planes.h"

namespace gorila {

constexpr int TR_WAVES = 8, TR_THREADS = 64 * TR_WAVES;
constexpr int TR_XV = STATE_BYTES / 16;  // 1764 16-byte vectors of a sample
constexpr int TR_XPT = (TR_XV + TR_THREADS - 1) / TR_THREADS;
constexpr int TR_T2 = 3;  // conv2: pixel tiles of 16 per wave (6 in all, 81 pixels)
constexpr int TR_T3 = 2;  // conv3: 4 in all, 49 pixels

// h1 in LDS: 64 bytes a pixel and plane, two pixels to a 128-byte line whose
// eight 16-byte chunks are XOR-permuted by a key that runs on over the ends of
// conv2's rows (9 y / 2 + x / 2), so the stride-2 pixels that 8 lanes read at
// one chunk always fall into different banks.
__device__ inline int h1_at(int line, int odd, int key, int chunk) {
    return line * 128 + ((((odd << 2) | chunk) ^ (key & 7)) << 4);
}
__device__ inline int h1_off(int y, int x, int chunk) {
    return h1_at(y * (H1 / 2) + (x >> 1), x & 1, (y >> 1) * H2 + (x >> 1), chunk);
}
constexpr int H1_PLANE = P1 * 64;
// h2: 128 bytes a pixel and plane, chunks permuted by a key that runs on over
// the ends of conv3's rows.
__device__ inline int h2_at(int p, int key, int chunk) { return p * 128 + ((chunk ^ (key & 7)) << 4); }
__device__ inline int h2_off(int y, int x, int chunk) { return h2_at(y * H2 + x, y * H3 + x, chunk); }
constexpr int H2_PLANE = P2 * 128;

template <int AP>
struct TrunkLds {
    // h1 lives from conv1 to the end of conv2; conv3's exchange reuses it
    static constexpr int H1 = AP * H1_PLANE, XCHG3 = TR_WAVES * TR_T3 * 1024;
    // the frames as bf16 live until the end of conv1, then h2 and conv2's exchange
    static constexpr int X = STATE_BYTES * 2, H2 = AP * H2_PLANE, XCHG2 = TR_WAVES * TR_T2 * 1024;
    static constexpr int LO = cmax(H1, XCHG3), HI = cmax(X, H2 + XCHG2);
};

// WP planes of weights, AP of activations.  Samples r = blockIdx.x, +
// gridDim.x, ...
template <int WP, int AP>
__global__ __launch_bounds__(TR_THREADS) void trunk_fwd_kernel(
    const uint8_t* const* __restrict__ ftab, const uint16_t* __restrict__ frag,
    const float* __restrict__ th, int rows, float* __restrict__ h3) {
    using L = TrunkLds<AP>;
    __shared__ __attribute__((aligned(16))) char lds[L::LO + L::HI];
    char* const s1 = lds;                  // h1 planes / conv3 exchange
    __bf16* const xs = (__bf16*)(lds + L::LO);
    char* const s2 = lds + L::LO;          // h2 planes
    f32x4* const xch2 = (f32x4*)(s2 + L::H2);
    f32x4* const xch3 = (f32x4*)s1;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int q = lane >> 4, col = lane & 15;

    uint4 xv[TR_XPT];
    unsigned okm = 0;  // bit k: xv[k] holds frame bytes (else zeros)
    const uint8_t *f0, *f1, *f2, *f3;  // frames of the next sample to fetch
    auto point = [&](int r) {
        const uint8_t* const* fr = ftab + (int64_t)r * 4;
        f0 = fr[0];
        f1 = fr[1];
        f2 = fr[2];
        f3 = fr[3];
    };
    auto fetch = [&]() {
        okm = 0;
#pragma unroll
        for (int k = 0; k < TR_XPT; ++k) {
            const int e = tid + k * TR_THREADS;  // vector e: frame e / 441
            const int fi = e / (FRAME_BYTES / 16);
            const uint8_t* f = fi == 0 ? f0 : fi == 1 ? f1 : fi == 2 ? f2 : f3;
            const bool ok = e < TR_XV && f != nullptr;
            // a null frame reads the first weights instead and is zeroed when converted
            xv[k] = ldg_u4(ok ? (const uint4*)f + (e - fi * (FRAME_BYTES / 16)) : (const uint4*)frag);
            okm |= (unsigned)ok << k;
        }
    };
    point(blockIdx.x);
    fetch();

    // conv1: wave = (channel tile, pixel group); pixel tiles pg, pg + 4, ... of 25
    const int c1t = wave & 1, pg = wave >> 1;
    // conv2, conv3: wave = (reduction half kh, pixel half mh, channel half nh)
    const int kh = wave & 1, mh = (wave >> 1) & 1, nh = wave >> 2;
    // per pixel tile: LDS element of the frames; line of h1 and pixel of h2 at
    // tap (0, 0), and their keys (which are the output pixel's number)
    int x1[7], p2[TR_T2], k2[TR_T2], p3[TR_T3], k3[TR_T3];
#pragma unroll
    for (int k = 0; k < 7; ++k) {
        const int m = (pg + 4 * k < 25 ? pg + 4 * k : 0) * 16 + col, i = m / H1, j = m - i * H1;
        x1[k] = (S1 * i + q) * IN_W + S1 * j;
    }
#pragma unroll
    for (int k = 0; k < TR_T2; ++k) {
        const int m = min((mh * TR_T2 + k) * 16 + col, P2 - 1), i = m / H2, j = m - i * H2;
        p2[k] = i * H1 + j;
        k2[k] = m;
    }
#pragma unroll
    for (int k = 0; k < TR_T3; ++k) {
        const int m = min((mh * TR_T3 + k) * 16 + col, P3 - 1), i = m / H3, j = m - i * H3;
        p3[k] = i * H2 + j;
        k3[k] = m;
    }

    // Weight fragments of a layer's step s into w[s & 1].  Two steps are in
    // flight; a layer's first two are issued before the previous layer's
    // stores (loads and stores are counted in order, so a load issued after
    // them would be waited for together with them).
    bf16x8 w[2][2][WP];
    int zero = 0;
    auto wload = [&](int f0, int stride, int nc, int s) {
        const bf16x8* const wf = (const bf16x8*)(frag + zero) + lane;
#pragma unroll
        for (int i = 0; i < nc; ++i)
#pragma unroll
            for (int pl = 0; pl < WP; ++pl) w[s & 1][i][pl] = wf[((f0 + s * stride + i) * WP + pl) * 64];
    };
    const int wf1 = FRAG1 + c1t, wf2 = FRAG2 + kh * 32 + nh * 2, wf3 = FRAG3 + kh * 36 + nh * 2;
    wload(wf1, 2, 1, 0);
    wload(wf1, 2, 1, 1);

    for (int r = blockIdx.x; r < rows; r += gridDim.x) {
        const int next = r + (int)gridDim.x;
        // an offset of 0 that the compiler cannot see through: the weights and
        // biases are read again for every sample, not kept over the row loop
        asm volatile("" : "+s"(zero));
        point(min(next, rows - 1));

        // frames: bytes to bf16, exact
#pragma unroll
        for (int k = 0; k < TR_XPT; ++k) {
            const int e = tid + k * TR_THREADS;
            if (e < TR_XV) {
                const uint4 v = (okm >> k) & 1u ? xv[k] : make_uint4(0, 0, 0, 0);
                const uint32_t d[4] = {v.x, v.y, v.z, v.w};
                bf16x8 a, b;
#pragma unroll
                for (int t = 0; t < 8; ++t) {
                    a[t] = (__bf16)(float)((d[t >> 2] >> (8 * (t & 3))) & 255u);
                    b[t] = (__bf16)(float)((d[2 + (t >> 2)] >> (8 * (t & 3))) & 255u);
                }
                *(bf16x8*)(xs + 16 * e) = a;
                *(bf16x8*)(xs + 16 * e + 8) = b;
            }
        }
        __syncthreads();

        // ---- conv1: 8 steps of four filter rows (c, u) of 8 columns ----
        {
            f32x4 hi[7], lo[7];
#pragma unroll
            for (int k = 0; k < 7; ++k) hi[k] = lo[k] = f32x4{};
            auto run = [&](auto nt) {
                constexpr int NT = decltype(nt)::value;
                bf16x8 x[2][NT];
                int xo[NT];
#pragma unroll
                for (int k = 0; k < NT; ++k) xo[k] = opaque(x1[k]);
                auto xload = [&](int st) {
#pragma unroll
                    for (int k = 0; k < NT; ++k) {
                        const __bf16* px = xs + xo[k] + (st >> 1) * FRAME_BYTES + (st & 1) * 4 * IN_W;
                        const bf16x4 a = *(const bf16x4*)px, b = *(const bf16x4*)(px + 4);
                        x[st & 1][k] = __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7);
                    }
                };
                xload(0);
#pragma unroll
                for (int st = 0; st < 8; ++st) {
                    if (st + 1 < 8) xload(st + 1);
#pragma unroll
                    for (int pl = 0; pl < WP; ++pl)
#pragma unroll
                        for (int k = 0; k < NT; ++k) {
                            if (pl == 0) hi[k] = mfma16(w[st & 1][0][pl], x[st & 1][k], hi[k]);
                            else lo[k] = mfma16(w[st & 1][0][pl], x[st & 1][k], lo[k]);
                        }
                    if (st + 2 < 8) wload(wf1, 2, 1, st + 2);
                    __builtin_amdgcn_sched_barrier(0);
                }
                const f32x4 bias = ld4(th + zero + OFF_B1 + c1t * 16 + 4 * q);
                wload(wf2, 4, 2, 0);
                wload(wf2, 4, 2, 1);
                const int el = opaque(lane), c0 = c1t * 16 + 4 * (el >> 4);
#pragma unroll
                for (int k = 0; k < NT; ++k) {
                    const int p = (pg + 4 * k) * 16 + (el & 15);
                    f32x4 v;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float s = WP > 1 ? plane_sum<WP>(hi[k][e], lo[k][e]) : hi[k][e];
                        v[e] = fmaxf(s * (1.0f / 255.0f) + bias[e], 0.0f);
                    }
                    bf16x4 o[AP];
                    split4<AP>(v, o);
                    const int off = h1_off(p / H1, p % H1, c0 >> 3) + ((c0 & 4) << 1);
#pragma unroll
                    for (int pl = 0; pl < AP; ++pl) *(bf16x4*)(s1 + pl * H1_PLANE + off) = o[pl];
                }
            };
            if (pg == 0) run(std::integral_constant<int, 7>{});
            else run(std::integral_constant<int, 6>{});
        }
        __syncthreads();

        // ---- conv2: 16 steps (taps), 8 for each reduction half ----
        {
            f32x4 hi[2][TR_T2], lo[2][TR_T2];
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < TR_T2; ++j) hi[i][j] = lo[i][j] = f32x4{};
            int px[TR_T2], kx[TR_T2];
#pragma unroll
            for (int j = 0; j < TR_T2; ++j) {
                px[j] = opaque(p2[j]);
                kx[j] = opaque(k2[j]);
            }
            bf16x8 x[2][TR_T2][AP];
            auto xload = [&](int s) {
#pragma unroll
                for (int j = 0; j < TR_T2; ++j) {
                    const int u = 2 * kh + (s >> 2), v = s & 3;
                    const int off = h1_at(px[j] + u * (H1 / 2) + (v >> 1), v & 1, kx[j] + (u >> 1) * H2 + (v >> 1), q);
#pragma unroll
                    for (int pl = 0; pl < AP; ++pl)
                        x[s & 1][j][pl] = *(const bf16x8*)(s1 + pl * H1_PLANE + off);
                }
            };
            // the next step's operands are read beside this step's products;
            // the barriers keep the compiler from reading further ahead
            xload(0);
#pragma unroll
            for (int s = 0; s < 8; ++s) {
                if (s + 1 < 8) xload(s + 1);
                plane_products<0, false>(w[s & 1], x[s & 1], hi, lo);
                if (s + 2 < 8) wload(wf2, 4, 2, s + 2);
                __builtin_amdgcn_sched_barrier(0);
            }
            const int el = opaque(lane), c0 = (nh * 2 + kh) * 16 + 4 * (el >> 4);
            const f32x4 bias = ld4(th + zero + OFF_B2 + c0);
            wload(wf3, 4, 2, 0);
            wload(wf3, 4, 2, 1);
            // the reduction halves: a wave hands channel tile 1 - kh to its
            // partner and finishes channel tile kh
#pragma unroll
            for (int j = 0; j < TR_T2; ++j) {
                const f32x4 a = plane_sum<AP>(hi[0][j], lo[0][j]), b = plane_sum<AP>(hi[1][j], lo[1][j]);
                xch2[(wave * TR_T2 + j) * 64 + lane] = kh ? a : b;
                hi[0][j] = kh ? b : a;
            }
            __syncthreads();
#pragma unroll
            for (int j = 0; j < TR_T2; ++j) {
                const f32x4 part = xch2[((wave ^ 1) * TR_T2 + j) * 64 + lane];
                const int p = (mh * TR_T2 + j) * 16 + (el & 15);
                f32x4 v;
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = fmaxf((hi[0][j][e] + part[e]) + bias[e], 0.0f);
                if (p < P2) {
                    bf16x4 o[AP];
                    split4<AP>(v, o);
                    const int off = h2_off(p / H2, p % H2, c0 >> 3) + ((c0 & 4) << 1);
#pragma unroll
                    for (int pl = 0; pl < AP; ++pl) *(bf16x4*)(s2 + pl * H2_PLANE + off) = o[pl];
                }
            }
        }
        __syncthreads();

        // ---- conv3: 18 steps (tap, channel half), 9 for each reduction half ----
        {
            f32x4 hi[2][TR_T3], lo[2][TR_T3];
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < TR_T3; ++j) hi[i][j] = lo[i][j] = f32x4{};
            int px[TR_T3], kx[TR_T3];
#pragma unroll
            for (int j = 0; j < TR_T3; ++j) {
                px[j] = opaque(p3[j]);
                kx[j] = opaque(k3[j]);
            }
            const int el = opaque(lane), c0 = (nh * 2 + kh) * 16 + 4 * (el >> 4);
            const f32x4 bias = ld4(th + zero + OFF_B3 + c0);
            float* const out = h3 + (int64_t)r * FLAT;
            bf16x8 x[2][TR_T3][AP];
            auto xload = [&](int s) {
                const int st = kh * 9 + s, tap = st >> 1, u = tap / 3, v = tap - 3 * u;
#pragma unroll
                for (int j = 0; j < TR_T3; ++j) {
                    const int off = h2_at(px[j] + u * H2 + v, kx[j] + u * H3 + v, (st & 1) * 4 + q);
#pragma unroll
                    for (int pl = 0; pl < AP; ++pl)
                        x[s & 1][j][pl] = *(const bf16x8*)(s2 + pl * H2_PLANE + off);
                }
            };
            xload(0);
#pragma unroll
            for (int s = 0; s < 9; ++s) {
                if (s + 1 < 9) xload(s + 1);
                plane_products<0, false>(w[s & 1], x[s & 1], hi, lo);
                if (s + 2 < 9) wload(wf3, 4, 2, s + 2);
                // the next sample's frames come from memory: requested behind
                // this sample's last weights, they are waited for by no one
                // before they are staged
                if (s == 6) {
                    if (next < rows) {
                        fetch();
                    } else {  // nothing of this sample's frames stays in registers
#pragma unroll
                        for (int k = 0; k < TR_XPT; ++k) xv[k] = make_uint4(0, 0, 0, 0);
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            wload(wf1, 2, 1, 0);
            wload(wf1, 2, 1, 1);
#pragma unroll
            for (int j = 0; j < TR_T3; ++j) {
                const f32x4 a = plane_sum<AP>(hi[0][j], lo[0][j]), b = plane_sum<AP>(hi[1][j], lo[1][j]);
                xch3[(wave * TR_T3 + j) * 64 + lane] = kh ? a : b;
                hi[0][j] = kh ? b : a;
            }
            __syncthreads();
#pragma unroll
            for (int j = 0; j < TR_T3; ++j) {
                const f32x4 part = xch3[((wave ^ 1) * TR_T3 + j) * 64 + lane];
                const int p = (mh * TR_T3 + j) * 16 + (el & 15);
                if (p < P3)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        out[(c0 + e) * P3 + p] =
                            fmaxf((hi[0][j][e] + part[e]) + bias[e], 0.0f);
            }
        }
    }
}

void launch_trunk_fwd(const uint8_t* const* ftab, const uint16_t* frag, int planes,
                      const float* theta, int n, float* h3, int cus, hipStream_t st) {
    if (n <= 0) return;
    // one resident workgroup per compute unit (its LDS), each walking samples
    const int blocks = min(n, max(cus, 1));
    if (planes == 1) trunk_fwd_kernel<1, 3><<<blocks, TR_THREADS, 0, st>>>(ftab, frag, theta, n, h3);
    else trunk_fwd_kernel<3, 3><<<blocks, TR_THREADS, 0, st>>>(ftab, frag, theta, n, h3);
}

}  // namespace gorila
