// Data gradients of conv3 and conv2 (the exact gradient of Section 5.1's
// layers, eq. (2)) as one launch: a workgroup takes one sample from dz3 to dz1
// with dz3 and dz2 in LDS as bf16 planes (planes.h), so the layers' overlapping
// patches are read from LDS and one launch boundary is gone.
//   dz2[y][x][c] = [h2 > 0] sum_{u,v,o} W3[o][c][u][v] dz3[y-u][x-v][o]
//   dz1[2y'+py][2x'+px][c] = [h1 > 0] sum_{du,dv,o} W2[o][c][2du+py][2dv+px] dz2[y'-du][x'-dv][o]
// Both are stored with a border of zeros (11 x 11 pixels), so taps outside the
// image need no test (but see inside_sum); pixel tiles for which a whole tap is
// outside skip it.
//
// conv3: 6 tiles of 16 of the 81 pixels, 4 channel tiles, 9 taps x 64 o; a wave
// takes three pixel tiles (mh), two channel tiles (nh) and 32 of the 64 o (kh),
// and the kh pairs exchange halves through LDS.  conv2: for each of the four
// stride phases 7 tiles of the 100 positions and 2 channel tiles, 4 taps x 64
// o; a wave takes one phase and four or three tiles.  Weights stream from L2 in
// operand order (prep_weights_part).
//
// Bound by the matrix instructions and, with one workgroup a unit (LDS), the
// barriers between a sample's phases.  Measured, this launch and the weight
// gradients' (wgrad.hip) against one launch of both gradients a layer on fp32
// instructions (conv3, conv2): 512 rows 44 + 56 -> 37 + 35 us, 2001 rows 148 +
// 206 -> 148 + 124, four learners of 33 rows 24 + 31 -> 18 + 14, 32 rows 12.4 +
// 14.9 -> 18.3 + 9.1 (one sample's chain is then the whole launch), 16 bf16
// learners of 64 rows 34 + 53 -> 36.5 + 35.
#include "common.h"
#include "kernels.h"
#include "planes.h"

#include <type_traits>

namespace gorila {

constexpr int BD_WAVES = 8, BD_THREADS = 64 * BD_WAVES;
constexpr int BD_W = 11, BD_PIX = BD_W * BD_W;  // bordered images: dz3 by 2, dz2 by 1
constexpr int BD_PLANE = BD_PIX * 128;
// 128 bytes a pixel and plane, its eight 16-byte chunks permuted by a key that
// runs on over the ends of the output rows (9 wide for conv3, 10 for conv2), so
// that 8 consecutive outputs' pixels of a tap always fall into different banks.
__device__ inline int bd_off(int p, int key, int chunk) { return p * 128 + ((chunk ^ (key & 7)) << 4); }

template <int GP>
struct BdLds {
    static constexpr int Z3 = 0, Z2 = GP * BD_PLANE, XCHG = 2 * GP * BD_PLANE;
    static constexpr int M2 = XCHG + BD_WAVES * 3 * 1024, M1 = M2 + P2 * 16;
    static constexpr int BYTES = M1 + P1 * 8;  // masks: a nibble of four channels a byte
};

// conv3 pixel tile t (pixels 16 t .. of the 9 x 9 grid) has a pixel for which
// tap (u, v) reads inside the 7 x 7 image
constexpr bool bd3_active(int t, int u, int v) {
    for (int p = 16 * t; p < 16 * t + 16 && p < P2; ++p) {
        const int y = p / H2 - u, x = p % H2 - v;
        if (y >= 0 && y < H3 && x >= 0 && x < H3) return true;
    }
    return false;
}
// tiles of the two wave groups, chosen so that their active taps balance (19, 21)
constexpr int BD3_TILE[2][3] = {{1, 2, 5}, {0, 3, 4}};
__device__ inline int bd3_tile(int mh, int j) {  // the same for a j that is no constant
    constexpr auto pack = [](int m) { return BD3_TILE[m][0] | BD3_TILE[m][1] << 4 | BD3_TILE[m][2] << 8; };
    constexpr int T0 = pack(0), T1 = pack(1);
    return (mh ? T1 : T0) >> (4 * j) & 15;
}
constexpr unsigned bd3_mask(int mh, int tap) {
    unsigned m = 0;
    for (int j = 0; j < 3; ++j) m |= bd3_active(BD3_TILE[mh][j], tap / 3, tap % 3) ? 1u << j : 0u;
    return m;
}
constexpr bool bd2_active(int t, int du, int dv) {
    for (int p = 16 * t; p < 16 * t + 16 && p < 100; ++p) {
        const int y = p / 10 - du, x = p % 10 - dv;
        if (y >= 0 && y < H2 && x >= 0 && x < H2) return true;
    }
    return false;
}
constexpr unsigned bd2_mask(int mh, int tap) {
    unsigned m = 0;
    for (int j = 0; j < 4 && 4 * mh + j < 7; ++j) m |= bd2_active(4 * mh + j, tap / 2, tap % 2) ? 1u << j : 0u;
    return m;
}

template <int MH>
struct Bd3Masks {  // step = tap
    static constexpr unsigned at(int t) { return bd3_mask(MH, t); }
};
template <int MH>
struct Bd2Masks {  // step = (tap, half of o)
    static constexpr unsigned at(int s) { return bd2_mask(MH, s >> 1); }
};

// The active pixel tiles of one wave's steps, in order, one or two at a time
// (the active tiles of a step are neighbours).
template <class Masks, int STEPS, int NT>
struct TileSeq {
    int n = 0;
    unsigned char t[STEPS * NT] = {}, j[STEPS * NT] = {}, c[STEPS * NT] = {};  // step, first tile, count
    constexpr TileSeq() {
        for (int a = 0; a < STEPS; ++a)
            for (int b = 0; b < NT; ++b) {
                if (!(Masks::at(a) >> b & 1u)) continue;
                t[n] = (unsigned char)a;
                j[n] = (unsigned char)b;
                c[n] = b + 1 < NT && (Masks::at(a) >> (b + 1) & 1u) ? 2 : 1;
                b += c[n++] - 1;
            }
    }
};

// The reduction of one wave: steps t = 0 .. STEPS-1, each over the pixel tiles
// of Masks::at(t), two channel tiles w[t & 1] against one or two pixel tiles'
// operands at a time.  The next operands are read from LDS beside these
// products, and a step's weights are replaced by those of step t + 2 (wload)
// once it has used them.
template <class Masks, int STEPS, int NT, int GP, int NA, class XLoad, class WLoad>
__device__ __forceinline__ void tile_sequence(XLoad xload, bf16x8 (&w)[2][2][GP], f32x4 (&hi)[2][NA],
                                              f32x4 (&lo)[2][NA], WLoad wload) {
    using Seq = TileSeq<Masks, STEPS, NT>;
    bf16x8 x[2][2][GP];
    auto load = [&](auto ic) {
        constexpr Seq Q{};
        constexpr int i = decltype(ic)::value;
#pragma unroll
        for (int k = 0; k < Q.c[i]; ++k) xload(Q.t[i], Q.j[i] + k, x[i & 1][k]);
    };
    load(std::integral_constant<int, 0>{});
    static_for<0, Seq{}.n>([&](auto ic) {
        constexpr Seq Q{};
        constexpr int i = decltype(ic)::value, t = Q.t[i], j = Q.j[i];
        if constexpr (i + 1 < Q.n) load(std::integral_constant<int, i + 1>{});
        if constexpr (Q.c[i] == 2) plane_products<j>(w[t & 1], x[i & 1], hi, lo);
        else plane_products<j>(w[t & 1], *(bf16x8(*)[1][GP]) & x[i & 1], hi, lo);
        if constexpr (t + 2 < STEPS && (i + 1 == Q.n || Q.t[i + 1] != t)) wload(t + 2);
        __builtin_amdgcn_sched_barrier(0);
    });
}

// An infinite weight makes NaNs of the border's zeros (0 * inf), also in outputs
// of which its tap is no part.  So a lane that has stored a NaN (`check`, the sum
// of all it stored, is one too) forms such outputs again, one product at a time,
// over the taps inside the image; a NaN that is one of those ends the sum.  (The
// sums and the test: 90.5 -> 90.8 us of a step of 32 rows, 313.8 -> 314.8 of 512.)
// z(tap u, v, o): the gradient's planes there, or null; w(u, v, o): the weight.
template <int GP, int K, class Z, class W>
__device__ __forceinline__ float inside_sum(Z z, W w) {
    float t = 0.0f;
#pragma unroll 1
    for (int i = 0; i < K * K * 64 && t == t; ++i) {
        const int u = i / (K * 64), v = i / 64 % K, o = i & 63;
        const char* const p = z(u, v, o);
        if (!p) continue;
        float x = ldv((const uint16_t*)p);
        if (fabsf(x) < INFINITY)  // (an infinite value's other planes are NaNs)
#pragma unroll
            for (int pl = 1; pl < GP; ++pl) x += ldv((const uint16_t*)(p + pl * BD_PLANE));
        t = fmaf(w(u, v, o), x, t);
    }
    return t;
}

// Waves a SIMD: bf16 dz3 comes in steps of more than 128 rows, two workgroups a unit.
template <class T>
constexpr int BD_MIN_WAVES = std::is_same_v<T, float> ? 2 : 4;

// GP planes of gradients and of weights: 3 for fp32 steps, 1 for bf16 ones
// (gradients rounded to bf16).  dz3: `kp` partial planes [kp][rows][64][49] of
// type T, added in order, the sum of more than one left as plane kp; dz2 [rows][81][64], dz1 [rows][400][32] of type O.
template <int GP, class T, class O>
__global__ __launch_bounds__(BD_THREADS, BD_MIN_WAVES<T>) void bwd_data_kernel(
    T* dz3, int kp, const float* __restrict__ h2, const float* __restrict__ h1,
    GroupPtrs16 frags, GroupPtrs theta, int n, int rows, O* __restrict__ dz2, O* __restrict__ dz1) {
    using L = BdLds<GP>;
    __shared__ __attribute__((aligned(16))) char lds[L::BYTES];
    char* const z3 = lds + L::Z3;
    char* const z2 = lds + L::Z2;
    f32x4* const xch = (f32x4*)(lds + L::XCHG);
    unsigned char* const m2 = (unsigned char*)lds + L::M2;
    unsigned char* const m1 = (unsigned char*)lds + L::M1;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int q = lane >> 4, col = lane & 15;

    // one sample's inputs: quads of dz3 (784), h2 (1296) and h1 (3200)
    constexpr int N3 = FLAT / 4, N2 = P2 * C2 / 4, N1 = P1 * C1 / 4;
    constexpr int T3 = (N3 + BD_THREADS - 1) / BD_THREADS, T2 = (N2 + BD_THREADS - 1) / BD_THREADS,
                  T1 = (N1 + BD_THREADS - 1) / BD_THREADS;
    f32x4 v3[T3], v2[T2], v1[T1];
    // quad e of a sample of dz3 ([64][49]): channels 4 (e / 49) .. at pixel e % 49
    auto at3 = [](int e, int c) { return (e / P3 * 4 + c) * P3 + e % P3; };
    auto quad3 = [&](const T* z, int e) {
        return f32x4{ldv(z + at3(e, 0)), ldv(z + at3(e, 1)), ldv(z + at3(e, 2)), ldv(z + at3(e, 3))};
    };
    auto fetch = [&](int r) {
        const int et = opaque(tid);
#pragma unroll
        for (int k = 0; k < T3; ++k) v3[k] = quad3(dz3 + (int64_t)r * FLAT, min(et + k * BD_THREADS, N3 - 1));
#pragma unroll
        for (int k = 0; k < T2; ++k)
            v2[k] = ld4(h2 + (int64_t)r * P2 * C2 + 4 * min(et + k * BD_THREADS, N2 - 1));
#pragma unroll
        for (int k = 0; k < T1; ++k)
            v1[k] = ld4(h1 + (int64_t)r * P1 * C1 + 4 * min(et + k * BD_THREADS, N1 - 1));
    };
    fetch(blockIdx.x);
    for (int i = tid; i < L::XCHG / 16; i += BD_THREADS) ((uint4*)lds)[i] = make_uint4(0, 0, 0, 0);

    const int kh = wave & 1, nh = (wave >> 1) & 1, mh3 = wave >> 2;  // conv3 roles
    const int ph = wave & 3, mh2 = wave >> 2;                        // conv2 roles
    int p3[3], p2[4], k3[3], k2[4];  // bordered pixel of tap (0, 0), and its key
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        const int t = mh3 ? BD3_TILE[1][j] : BD3_TILE[0][j];
        const int m = min(t * 16 + col, P2 - 1), y = m / H2, x = m - y * H2;
        p3[j] = (y + 2) * BD_W + x + 2;
        k3[j] = (y + 2) * H2 + x + 2;
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int m = min((mh2 * 4 + j) * 16 + col, 99), y = m / 10, x = m - y * 10;
        p2[j] = (y + 1) * BD_W + x + 1;
        k2[j] = (y + 1) * 10 + x + 1;
    }

    bf16x8 w[2][2][GP];
    const uint16_t* frag = frags.p[blockIdx.x / n];
    int zero = 0;  // see below
    // fragments f0 + s * stride, + 1 into w[s & 1]
    auto wload = [&](int f0, int stride, int s) {
        const bf16x8* const wf = (const bf16x8*)(frag + zero) + lane;
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int pl = 0; pl < GP; ++pl) w[s & 1][i][pl] = wf[((f0 + s * stride + i) * GP + pl) * 64];
    };
    const int wf3 = FRAGD3 + kh * 4 + nh * 2, wf2 = FRAGD2 + ph * 16;
    __syncthreads();  // the borders' zeros before any interior

    for (int r = blockIdx.x; r < rows; r += gridDim.x) {
        const int next = r + (int)gridDim.x;
        const int g = r / n;
        frag = frags.p[g];
        const float* const th = theta.p[g];
        // an offset of 0 that the compiler cannot see through: the weights are
        // read again for every sample, not kept over the row loop
        asm volatile("" : "+s"(zero));
        wload(wf3, 8, 0);
        wload(wf3, 8, 1);
        {
            const int et = opaque(tid);
#pragma unroll
            for (int k = 0; k < T3; ++k) {
                const int e = et + k * BD_THREADS;
                if (e < N3) {
                    f32x4 v = v3[k];
                    if (kp > 1) {
                        for (int s = 1; s < kp; ++s) v += quad3(dz3 + ((int64_t)s * rows + r) * FLAT, e);
#pragma unroll
                        for (int c = 0; c < 4; ++c) stv(dz3 + ((int64_t)kp * rows + r) * FLAT + at3(e, c), v[c]);
                    }
                    bf16x4 o[GP];
                    split4<GP>(v, o);
                    const int cq = e / P3, p = e - cq * P3, y = p / H3, x = p - y * H3;
                    const int off = bd_off((y + 2) * BD_W + x + 2, (y + 2) * H2 + x + 2, cq >> 1) + ((cq & 1) << 3);
#pragma unroll
                    for (int pl = 0; pl < GP; ++pl) *(bf16x4*)(z3 + pl * BD_PLANE + off) = o[pl];
                }
            }
            auto nibble = [](f32x4 v) {
                return (unsigned char)((v[0] > 0.f) | (v[1] > 0.f) << 1 | (v[2] > 0.f) << 2 | (v[3] > 0.f) << 3);
            };
#pragma unroll
            for (int k = 0; k < T2; ++k)
                if (et + k * BD_THREADS < N2) m2[et + k * BD_THREADS] = nibble(v2[k]);
#pragma unroll
            for (int k = 0; k < T1; ++k)
                if (et + k * BD_THREADS < N1) m1[et + k * BD_THREADS] = nibble(v1[k]);
        }
        __syncthreads();

        // ---- conv3: 9 taps, this wave's half of the 64 o ----
        {
            f32x4 hi[2][3], lo[2][3];
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 3; ++j) hi[i][j] = lo[i][j] = f32x4{};
            auto run = [&](auto mhc) {
                constexpr int MH = decltype(mhc)::value;
                int px[3], kx[3];
#pragma unroll
                for (int j = 0; j < 3; ++j) {
                    px[j] = opaque(p3[j]);
                    kx[j] = opaque(k3[j]);
                }
                tile_sequence<Bd3Masks<MH>, 9, 3, GP>(
                    [&](int t, int j, bf16x8 (&x)[GP]) {
                        const int off = bd_off(px[j] - (t / 3) * BD_W - t % 3,
                                               kx[j] - (t / 3) * H2 - t % 3, kh * 4 + q);
#pragma unroll
                        for (int pl = 0; pl < GP; ++pl) x[pl] = *(const bf16x8*)(z3 + pl * BD_PLANE + off);
                    },
                    w, hi, lo, [&](int t) { wload(wf3, 8, t); });
            };
            if (mh3) run(std::integral_constant<int, 1>{});
            else run(std::integral_constant<int, 0>{});
            wload(wf2, 2, 0);
            wload(wf2, 2, 1);
            // a wave hands channel tile 1 - kh to its partner and finishes tile kh
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                const f32x4 a = plane_sum<GP>(hi[0][j], lo[0][j]), b = plane_sum<GP>(hi[1][j], lo[1][j]);
                xch[(wave * 3 + j) * 64 + lane] = kh ? a : b;
                hi[0][j] = kh ? b : a;
            }
            __syncthreads();
            const int el = opaque(lane), c0 = (nh * 2 + kh) * 16 + 4 * (el >> 4);
            O* const out = dz2 + (int64_t)r * P2 * C2;
            float check = 0.0f;
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                const f32x4 part = xch[((wave ^ 1) * 3 + j) * 64 + lane];
                const int p = (mh3 ? BD3_TILE[1][j] : BD3_TILE[0][j]) * 16 + (el & 15);
                if (p < P2) {
                    const unsigned m = m2[p * 16 + (c0 >> 2)];
                    f32x4 v;
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = m >> e & 1u ? hi[0][j][e] + part[e] : 0.0f;
                    const int y = p / H2, x = p - y * H2;
                    check += (v[0] + v[1]) + (v[2] + v[3]);
                    bf16x4 o[GP];
                    split4<GP>(v, o);
                    const int off = bd_off((y + 1) * BD_W + x + 1, (y + 1) * 10 + x + 1, c0 >> 3) + ((c0 & 4) << 1);
#pragma unroll
                    for (int pl = 0; pl < GP; ++pl) *(bf16x4*)(z2 + pl * BD_PLANE + off) = o[pl];
                    stq(out + p * C2 + c0, v);
                }
            }
            if (__builtin_expect(check != check, 0))
#pragma unroll 1
                for (int k = 0; k < 12; ++k) {  // channel c0 + k % 4 of the wave's tile k / 4
                    const int p = bd3_tile(mh3, k >> 2) * 16 + (el & 15), c = c0 + (k & 3);
                    if (p >= P2 || ldv(out + p * C2 + c) == ldv(out + p * C2 + c)) continue;
                    const int y = p / H2, x = p - y * H2;
                    const float t = inside_sum<GP, K3>(
                        [&](int u, int v, int o) -> const char* {
                            const int i = y - u, j = x - v;
                            if (i < 0 || i >= H3 || j < 0 || j >= H3) return nullptr;
                            return z3 + bd_off((i + 2) * BD_W + j + 2, (i + 2) * H2 + j + 2, o >> 3) + (o & 7) * 2;
                        },
                        [&](int u, int v, int o) { return th[OFF_W3 + ((o * C2 + c) * K3 + u) * K3 + v]; });
                    stv(out + p * C2 + c, t);
                    bf16x4 o[GP];
                    split4<GP>(f32x4{t, 0.f, 0.f, 0.f}, o);
                    char* const to = z2 + bd_off((y + 1) * BD_W + x + 1, (y + 1) * 10 + x + 1, c >> 3) + (c & 7) * 2;
#pragma unroll
                    for (int pl = 0; pl < GP; ++pl) *(__bf16*)(to + pl * BD_PLANE) = o[pl][0];
                }
        }
        __syncthreads();

        // ---- conv2: 8 steps (tap, half of o) of this wave's phase ----
        {
            f32x4 hi[2][4], lo[2][4];
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) hi[i][j] = lo[i][j] = f32x4{};
            auto run = [&](auto mhc) {
                constexpr int MH = decltype(mhc)::value, NT = MH ? 3 : 4;
                int px[4], kx[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    px[j] = opaque(p2[j]);
                    kx[j] = opaque(k2[j]);
                }
                tile_sequence<Bd2Masks<MH>, 8, NT, GP>(
                    [&](int t, int j, bf16x8 (&x)[GP]) {
                        const int off = bd_off(px[j] - (t >> 2) * BD_W - ((t >> 1) & 1),
                                               kx[j] - (t >> 2) * 10 - ((t >> 1) & 1), (t & 1) * 4 + q);
#pragma unroll
                        for (int pl = 0; pl < GP; ++pl) x[pl] = *(const bf16x8*)(z2 + pl * BD_PLANE + off);
                    },
                    w, hi, lo, [&](int t) { wload(wf2, 2, t); });
                if (next < rows) {
                    fetch(next);  // behind this sample's last weights
                } else {  // nothing of this sample's inputs stays in registers
#pragma unroll
                    for (int k = 0; k < T3; ++k) v3[k] = f32x4{};
#pragma unroll
                    for (int k = 0; k < T2; ++k) v2[k] = f32x4{};
#pragma unroll
                    for (int k = 0; k < T1; ++k) v1[k] = f32x4{};
                }
                const int el = opaque(lane), c0 = 4 * (el >> 4);
                O* const out = dz1 + (int64_t)r * P1 * C1;
                float check = 0.0f;
#pragma unroll
                for (int j = 0; j < NT; ++j) {
                    const int m = (MH * 4 + j) * 16 + (el & 15), y = m / 10, x0 = m - y * 10;
                    if (m < 100) {
                        const int p = (2 * y + (ph >> 1)) * H1 + 2 * x0 + (ph & 1);
#pragma unroll
                        for (int i = 0; i < 2; ++i) {
                            const unsigned b = m1[p * 8 + i * 4 + (c0 >> 2)];
                            f32x4 v;
#pragma unroll
                            for (int e = 0; e < 4; ++e) v[e] = b >> e & 1u ? plane_sum<GP>(hi[i][j][e], lo[i][j][e]) : 0.0f;
                            check += (v[0] + v[1]) + (v[2] + v[3]);
                            stq(out + p * C1 + i * 16 + c0, v);
                        }
                    }
                }
                if (__builtin_expect(check != check, 0))
#pragma unroll 1
                    for (int k = 0; k < 8 * NT; ++k) {  // channel of tile k / 8
                        const int m = (MH * 4 + (k >> 3)) * 16 + (el & 15), y = m / 10, x = m - y * 10;
                        const int p = (2 * y + (ph >> 1)) * H1 + 2 * x + (ph & 1), c = (k >> 2 & 1) * 16 + c0 + (k & 3);
                        if (m >= 100 || ldv(out + p * C1 + c) == ldv(out + p * C1 + c)) continue;
                        stv(out + p * C1 + c,
                            inside_sum<GP, 2>(
                                [&](int du, int dv, int o) -> const char* {
                                    const int i = y - du, j = x - dv;
                                    if (i < 0 || i >= H2 || j < 0 || j >= H2) return nullptr;
                                    return z2 + bd_off((i + 1) * BD_W + j + 1, (i + 1) * 10 + j + 1, o >> 3) + (o & 7) * 2;
                                },
                                [&](int du, int dv, int o) {
                                    return th[OFF_W2 + ((o * C1 + c) * K2 + 2 * du + (ph >> 1)) * K2 + 2 * dv + (ph & 1)];
                                }));
                    }
            };
            if (mh2) run(std::integral_constant<int, 1>{});
            else run(std::integral_constant<int, 0>{});
        }
        __syncthreads();  // the masks and dz3 are read before the next sample lands
    }
}

void launch_bwd_data(float* dz3, int kp, const float* h2, const float* h1,
                     const GroupPtrs16& frags, const GroupPtrs& theta, int groups, int n, float* dz2,
                     float* dz1, bool bf16, int cus, hipStream_t st) {
    const int rows = groups * n;
    if (rows <= 0) return;
    // resident workgroups per compute unit (LDS): one with three planes, two with one
    const int blocks = min(rows, max(cus, 1) * (bf16 ? 2 : 1));
    if (!bf16)
        bwd_data_kernel<3, float, float><<<blocks, BD_THREADS, 0, st>>>(dz3, kp, h2, h1, frags, theta, n, rows,
                                                                        dz2, dz1);
    else if (kp > 1)
        bwd_data_kernel<1, float, uint16_t><<<blocks, BD_THREADS, 0, st>>>(
            dz3, kp, h2, h1, frags, theta, n, rows, (uint16_t*)dz2, (uint16_t*)dz1);
    else  // dz3 as the fc1 backward rounded it
        bwd_data_kernel<1, uint16_t, uint16_t><<<blocks, BD_THREADS, 0, st>>>(
            (uint16_t*)dz3, kp, h2, h1, frags, theta, n, rows, (uint16_t*)dz2, (uint16_t*)dz1);
}

}  // namespace gorila
