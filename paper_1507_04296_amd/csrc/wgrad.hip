// Weight gradients of conv3 and conv2 (the exact gradient of Section 5.1's
// layers, eq. (2)) on bf16 planes (planes.h):
//   dW2[o][c][u][v] = sum_{b,i,j} dz2[b][i][j][o] h1[b][2i+u][2j+v][c]
//   dW3[o][c][u][v] = sum_{b,i,j} dz3[b][i][j][o] h2[b][i+u][j+v][c]
// The reduction runs over output pixels, the slow index of every operand.  The
// activations are staged in LDS as they lie in memory ([pixel][channel], split
// into planes) and read transposed (ds_read_b64_tr_b16: 16 lanes read four
// pixels of 16 channels and each receives one channel's four pixels), so one
// copy serves every tap; dz, which every column meets at the same pixels, is
// transposed as it is staged ([channel][pixel]) and read as whole vectors.
//
// A workgroup owns a slice of one layer's columns and a range of samples, and
// keeps its sums in registers over the range: conv2 in two slices (16 input
// channels x 16 taps), conv3 in three (one filter row u: 64 channels x 3
// taps).  A sample's dz is then staged once for all taps and an activation
// once for all the taps it meets, where tiles of a flattened GEMM read every
// activation four to nine times; samples are double buffered, one barrier
// each.  What bounds it is LDS: a transposed read moves 64 bytes a clock (a
// whole-vector one 128), so a conv2 wave takes all four row tiles of o against
// two column tiles.  db2 and db3 are summed from the staged values.
// A conv2 sample takes 7450 cycles, 4950 of them matrix instructions; whole-
// vector reads of the transposed dz (a third of the LDS bytes) and conflict-free
// pixel sets did not shorten it, nor did spreading the staging over the products.
// Times are given with the data gradients (bwd.hip).
#include "common.h"
#include "conv1_wgrad.h"
#include "kernels.h"
#include "planes.h"

namespace gorila {

constexpr int WG_THREADS = 512;
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

// Rows of 128 bytes whose four 32-byte granules (16 channels) are permuted by
// the row's number, so the four pixels that 16 lanes read fall into different
// banks.
__device__ inline int row_off(int p, int granule) { return p * 128 + ((granule ^ (p & 3)) << 5); }
// h1 slices hold one granule a pixel, four pixels a line.  conv2's pixels of a
// row are two apart and alternate between two granules of a line, so odd lines
// swap neighbours; its pixels of a column are 40 apart (p < 400: p / 40).
__device__ inline int h1s_off(int p) {
    return (p >> 2) * 128 + (((p ^ (p >> 2 & 1) ^ (p * 1639 >> 16)) & 3) << 5);
}

// The reduction's order: sets of four output pixels, each read by 16 lanes at
// once, that lie in one row (or, the ninth pixels of conv2's rows, one column)
// so that their granules differ; -1 is padding.  Sets 8 st + 2 q + half.
template <bool CONV2>
__device__ inline int set_pixel(int set, int r) {
    if (CONV2) {
        if (set < 18) return (set < 9 ? set : set - 9) * H2 + (set < 9 ? r : r + 4);
        const int i = (set - 18) * 4 + r;
        return i < H2 ? i * H2 + 8 : -1;
    }
    if (set < 7) return set * H3 + r;
    return set < 14 && r < 3 ? (set - 7) * H3 + 4 + r : -1;
}

// Operand of 16 rows (channels) x 32 pixels: the pixels' granules for this
// lane at a (first four of its eight) and b.
__device__ __forceinline__ bf16x8 tr_read(const char* a, const char* b) {
    const s16x4 x = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)a);
    const s16x4 y = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)b);
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(x, y, 0, 1, 2, 3, 4, 5, 6, 7));
}

// dz in LDS: [64 rows][reduction order], rows padded so that eight rows' 16-byte
// vectors fall into different banks (208 and 144 bytes: 13 and 9 x 16).  Row r
// is channel 4 (r % 16) + r / 16, so that threads of neighbouring channel quads
// store to neighbouring rows.
struct Wg2 {  // conv2, slice = 16 input channels; a wave: 4 row tiles x 2 taps
    static constexpr int SLICES = 2, PIX = P2, STEPS = 3, MT = 4, NT = 2, CG = 1;  // 81 pixels in 3 x 32
    static constexpr int XPIX = P1, XQ = 4;                                // h1 quads a pixel
    static constexpr int A_ROW = 208, A_PLANE = 64 * A_ROW;
    static constexpr int ZERO = XPIX * 32, X_PLANE = ZERO + 128;           // pixels 400 .. 403 are zeros
    static constexpr int LD = 16 * C1;                                     // columns of a partial
};
struct Wg3 {  // conv3, slice = one filter row; a wave: 2 row tiles x 3 taps of 16 channels
    static constexpr int SLICES = 3, PIX = P3, STEPS = 2, MT = 2, NT = 3, CG = 3;  // 49 pixels in 2 x 32
    static constexpr int XPIX = H3 * H2, XQ = 16;                          // 7 of the 9 rows of h2
    static constexpr int A_ROW = 144, A_PLANE = 64 * A_ROW;
    static constexpr int ZERO = 64 * 128, X_PLANE = ZERO + 6 * 128;        // pixels 64 .. 69 are zeros
    static constexpr int LD = 9 * C2;
};
template <int GP>
constexpr int WG_LDS = 2 * GP * (Wg2::A_PLANE + Wg2::X_PLANE);
static_assert(Wg3::A_PLANE + Wg3::X_PLANE <= Wg2::A_PLANE + Wg2::X_PLANE, "conv2 is the larger");

// One workgroup: samples [b0, b1) of one group.  dz: dz2 [b][81][64]
// or dz3 [b][64][49]; x: h1 [b][400][32] or h2 [b][81][64]; part
// [64][LD]; bias [64] (slice 0 only, else null).
template <class G, int GP, class T>
__device__ __forceinline__ void wgrad_run(char* lds, int slice, int b0, int b1, const T* __restrict__ dz,
                                          const float* __restrict__ x, float* __restrict__ part,
                                          float* __restrict__ bias) {
    constexpr bool CONV2 = std::is_same_v<G, Wg2>;
    constexpr int SETS = G::STEPS * 8, XN = G::XPIX * G::XQ;  // pixel sets; staged quads of x
    constexpr int TX = (XN + WG_THREADS - 1) / WG_THREADS;
    constexpr int BUF = GP * (G::A_PLANE + G::X_PLANE);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int q = lane >> 4, ri = (lane & 15) >> 2, ci = lane & 3;
    const int m0 = CONV2 ? 0 : (wave >> 2) * 2;  // first row tile
    // first column tile: conv2 tap (u, v) of 16 channels, conv3 channels 16 ng .. of tap v = 0
    const int tu = wave >> 1, tv = 2 * (wave & 1), ng = wave & 3;

    // Staging of dz: thread (set, channel quad) takes four pixels of four
    // channels, so that a channel's four pixels are stored together; padding
    // pixels (and sets: all, for the threads past the last) are zeros.
    static_assert(SETS * 16 <= WG_THREADS, "one set and channel quad a thread");
    const int set = tid >> 4, cq = tid & 15;
    int apix[4];
    bool aok[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int m = set_pixel<CONV2>(set, e);
        aok[e] = m >= 0;
        apix[e] = (m >= 0 ? m : 0) * 64 + cq * 4;
    }
    // dz2 is [81][64]: quad e is four channels of pixel e; dz3 is [64][49]: quad e
    // is the set's four pixels of channel e, one vector (a set's pixels follow
    // one another; a padding pixel reads what follows, the last three of the last
    // channel one value early)
    if constexpr (!CONV2) {
        const int p0 = max(0, set_pixel<false>(set, 0));
#pragma unroll
        for (int e = 0; e < 4; ++e) apix[e] = (cq * 4 + e) * P3 + p0;
    }
    const bool early = !CONV2 && apix[3] + 3 >= FLAT;
    if (early) apix[3] -= 1;
    f32x4 va[4], vx[TX], bsum = {};
    auto fetch_a = [&](int b) {
        const T* const z = dz + (int64_t)b * G::PIX * 64;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if constexpr (CONV2) va[e] = ldq(z + apix[e]);
            else va[e] = ldqa(z + apix[e]);
        }
        if (early) va[3] = f32x4{va[3][1], va[3][2], va[3][3], 0.0f};
    };
    auto stage_a = [&](char* buf, int c) {  // channel c of the four
        f32x4 v = va[c];
        if constexpr (CONV2) v = f32x4{va[0][c], va[1][c], va[2][c], va[3][c]};
        v = f32x4{aok[0] ? v[0] : 0.f, aok[1] ? v[1] : 0.f, aok[2] ? v[2] : 0.f, aok[3] ? v[3] : 0.f};
        bsum[c] += (v[0] + v[1]) + (v[2] + v[3]);
        bf16x4 o[GP];
        split4<GP>(v, o);
        if (set < SETS)
#pragma unroll
            for (int pl = 0; pl < GP; ++pl)
                *(bf16x4*)(buf + pl * G::A_PLANE + (c * 16 + cq) * G::A_ROW + set * 8) = o[pl];
    };
    // x: quad k of this thread (the last, incomplete round repeats the last
    // quad: the same bytes to the same place)
    auto fetch_x = [&](int b, int k) {
        const int e = min(tid + k * WG_THREADS, XN - 1);
        if (CONV2) vx[k] = ld4(x + (int64_t)b * P1 * C1 + slice * 16 + (e >> 2) * C1 + (e & 3) * 4);
        else vx[k] = ld4(x + ((int64_t)b * P2 + slice * H2) * C2 + 4 * e);
    };
    auto stage_x = [&](char* buf, int k) {
        const int e = opaque(min(tid + k * WG_THREADS, XN - 1));
        char* const p = buf + GP * G::A_PLANE +
                        (CONV2 ? h1s_off(e >> 2) + ((e & 3) << 3) : row_off(e >> 4, (e & 15) >> 2) + ((e & 3) << 3));
        bf16x4 o[GP];
        split4<GP>(vx[k], o);
#pragma unroll
        for (int pl = 0; pl < GP; ++pl) *(bf16x4*)(p + pl * G::X_PLANE) = o[pl];
    };
    // parts of staging one sample: channels of dz two at a time, then the quads of x
    constexpr int PARTS_N = 2 + TX;
    auto stage = [&](char* buf, int b2, auto kc) {
        constexpr int k = decltype(kc)::value;
        if constexpr (k < 2) {
            stage_a(buf, 2 * k);
            stage_a(buf, 2 * k + 1);
            if constexpr (k == 1) fetch_a(b2);
        } else {
            stage_x(buf, k - 2);
            fetch_x(b2, k - 2);
        }
    };

    // this lane's pixel of x at tap (0, 0), for its set of step st, half hf
    int px[G::STEPS * 2];
#pragma unroll
    for (int k = 0; k < G::STEPS * 2; ++k) {
        const int s = 8 * (k >> 1) + 2 * q + (k & 1), m = set_pixel<CONV2>(s, ri);
        if (CONV2) px[k] = 2 * (m / H2) * H1 + 2 * (m % H2) + tu * H1 + tv;
        else px[k] = (m / H3) * H2 + m % H3;
        // padding multiplies zeros with zeros (a real pixel's infinity would make
        // NaNs of them); conv3's of a pixel that shares no bank with its set's
        if (m < 0) px[k] = CONV2 ? P1 : 64 + (s & 3);
    }

    f32x4 hi[G::MT][G::NT], lo[G::MT][G::NT];
#pragma unroll
    for (int i = 0; i < G::MT; ++i)
#pragma unroll
        for (int j = 0; j < G::NT; ++j) hi[i][j] = lo[i][j] = f32x4{};

    auto aload = [&](const char* buf, int st, bf16x8 (&a)[G::MT][GP]) {
        const char* const p = buf + ((lane & 15) + m0 * 16) * G::A_ROW + q * 16 + st * 64;
#pragma unroll
        for (int pl = 0; pl < GP; ++pl)
#pragma unroll
            for (int i = 0; i < G::MT; ++i)
                a[i][pl] = *(const bf16x8*)(p + pl * G::A_PLANE + i * 16 * G::A_ROW);
    };
    auto xload = [&](const char* buf, int st, int j, bf16x8 (&b)[GP]) {
        const char* bx = buf + GP * G::A_PLANE + ci * 8;
        const int p0 = px[2 * st] + j, p1 = px[2 * st + 1] + j;
        const int o0 = CONV2 ? h1s_off(p0) : row_off(p0, ng), o1 = CONV2 ? h1s_off(p1) : row_off(p1, ng);
#pragma unroll
        for (int pl = 0; pl < GP; ++pl) b[pl] = tr_read(bx + pl * G::X_PLANE + o0, bx + pl * G::X_PLANE + o1);
    };

    // Column tiles go CG at a time, so that a round of products has at least
    // four independent accumulators.
    constexpr int GRP = G::NT / G::CG, TILES = G::STEPS * GRP;
    static_assert(TILES % 2 == 0, "a sample's first operands go where the last but one's were");
    bf16x8 xv[2][G::CG][GP];
    auto xgroup = [&](const char* buf, int i) {
#pragma unroll
        for (int c = 0; c < G::CG; ++c) xload(buf, i / GRP, (i % GRP) * G::CG + c, xv[i & 1][c]);
    };
    // One sample.  MORE: beside its products the next sample is converted into
    // the other buffer, part by part, a part's registers refilled with the
    // sample after that.  The barrier stands before the last products, when
    // their operands are in registers: after it no wave reads this buffer and
    // every wave's share of the next is there, whose first operands are read
    // beside the last products.
    auto sample = [&](int b, auto more) {
        constexpr bool MORE = decltype(more)::value;
        const char* const buf = lds + ((b - b0) & 1) * BUF;
        char* const nxt = lds + ((b - b0 + 1) & 1) * BUF;
        const int b2 = min(b + 2, b1 - 1);
        bf16x8 a[G::MT][GP];
        static_for<0, TILES>([&](auto ic) {
            constexpr int i = decltype(ic)::value;
            if constexpr (i % GRP == 0) aload(buf, i / GRP, a);
            if constexpr (i + 1 < TILES) xgroup(buf, i + 1);
            if constexpr (MORE && i + 1 == TILES) {
                __syncthreads();
                xgroup(nxt, 0);
            }
            plane_products<(i % GRP) * G::CG>(a, xv[i & 1], hi, lo);
            // parts [i PARTS_N / (TILES - 1), (i + 1) PARTS_N / (TILES - 1)), none beside the last
            constexpr int k0 = i * PARTS_N / (TILES - 1), k1 = (i + 1) * PARTS_N / (TILES - 1);
            if constexpr (MORE && i + 1 < TILES) static_for<k0, k1>([&](auto kc) { stage(nxt, b2, kc); });
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    if (b0 < b1) {
        const int bn = min(b0 + 1, b1 - 1);
        // the zero pixels of every plane of both buffers
        constexpr int ZV = (G::X_PLANE - G::ZERO) / 16;
        static_assert(2 * GP * ZV <= WG_THREADS, "one vector a thread");
        if (tid < 2 * GP * ZV) {
            const int pl = tid / ZV, half = pl / GP;  // plane pl % GP of buffer `half`
            *(uint4*)(lds + half * BUF + GP * G::A_PLANE + (pl - half * GP) * G::X_PLANE + G::ZERO + (tid - pl * ZV) * 16) =
                make_uint4(0, 0, 0, 0);
        }
        fetch_a(b0);
#pragma unroll
        for (int k = 0; k < TX; ++k) fetch_x(b0, k);
        static_for<0, PARTS_N>([&](auto kc) { stage(lds, bn, kc); });
        __syncthreads();
        xgroup(lds, 0);
        for (int b = b0; b < b1 - 1; ++b) sample(b, std::true_type{});
        sample(b1 - 1, std::false_type{});
        __syncthreads();
    }

#pragma unroll
    for (int i = 0; i < G::MT; ++i)
#pragma unroll
        for (int j = 0; j < G::NT; ++j) {
            const int o = 16 * q + m0 + i;  // of the tile's row 4 q (see A_ROW)
            const int c = CONV2 ? (tu * 4 + tv + j) * C1 + slice * 16 + (lane & 15)
                                : (slice * 3 + j) * C2 + ng * 16 + (lane & 15);
#pragma unroll
            for (int e = 0; e < 4; ++e) part[(o + 4 * e) * G::LD + c] = plane_sum<GP>(hi[i][j][e], lo[i][j][e]);
        }
    if (bias) {
        // 32 threads hold each channel quad; the buffers are free
        f32x4* const red = (f32x4*)lds;
        red[tid] = bsum;
        __syncthreads();
        if (tid < 64) {
            float t = 0.0f;
            for (int k = 0; k < WG_THREADS / 16; ++k) t += ((const float*)red)[k * 64 + tid];
            bias[tid] = t;
        }
    }
}

// conv1's part of a launch of all three layers: `blocks` workgroups a group (0: none).
struct C1wPart {
    int blocks = 0, splits = 0;
    const float* dz1 = nullptr;
    const uint8_t* const* ftab = nullptr;
    const uint8_t* zero_frame = nullptr;
    float* part = nullptr;
    float* bias = nullptr;
};

template <int GP, bool WITH1, class T3, class T2>
__global__ __launch_bounds__(WG_THREADS) void conv_wgrad_kernel(
    const T3* __restrict__ dz3, const float* __restrict__ h2, const T2* __restrict__ dz2,
    const float* __restrict__ h1, int groups, int n, int s3, int s2, float* __restrict__ part3,
    float* __restrict__ part2, float* __restrict__ bias3, float* __restrict__ bias2, C1wPart c1) {
    static_assert(!WITH1 || (C1W_LDS <= WG_LDS<GP> && WG_THREADS == 64 * C1W_WAVES), "conv1's workgroups fit");
    __shared__ __attribute__((aligned(16))) char lds[WG_LDS<GP>];
    int bid = blockIdx.x;
    if constexpr (WITH1) {
        const int n1 = c1.blocks * groups;  // a multiple of 16: the others keep their XCDs
        if (bid < n1) {
            conv1_wgrad_run<GP>(lds, bid % c1.blocks, bid / c1.blocks, c1.dz1, c1.ftab, c1.zero_frame, n,
                                c1.splits, c1.part, c1.bias);
            return;
        }
        bid -= n1;
    }
    // conv2 first (its samples cost more); the slices of one range, which read
    // the same dz, are neighbours and so share an XCD's L2
    const int n2 = Wg2::SLICES * s2 * groups, n3 = Wg3::SLICES * s3 * groups, pad2 = pad_xcd(n2);
    int t;
    if (bid < pad2) {
        t = xcd_tile(bid, pad2);
        if (t >= n2) return;
        const int slice = t % Wg2::SLICES, gs = t / Wg2::SLICES, g = gs / s2, ks = gs - g * s2;
        const int64_t row = (int64_t)g * n;
        wgrad_run<Wg2, GP>(lds, slice, (int)((int64_t)ks * n / s2), (int)((int64_t)(ks + 1) * n / s2),
                           dz2 + row * P2 * C2, h1 + row * P1 * C1,
                           part2 + (int64_t)gs * C2 * Wg2::LD, slice == 0 ? bias2 + gs * 64 : nullptr);
    } else {
        t = xcd_tile(bid - pad2, pad_xcd(n3));
        if (t >= n3) return;
        const int slice = t % Wg3::SLICES, gs = t / Wg3::SLICES, g = gs / s3, ks = gs - g * s3;
        const int64_t row = (int64_t)g * n;
        wgrad_run<Wg3, GP>(lds, slice, (int)((int64_t)ks * n / s3), (int)((int64_t)(ks + 1) * n / s3),
                           dz3 + row * FLAT, h2 + row * P2 * C2,
                           part3 + (int64_t)gs * C3 * Wg3::LD, slice == 0 ? bias3 + gs * 64 : nullptr);
    }
}

// Splits (sample ranges) per group: one workgroup per slot, shared between the
// layers so that the longer of the two kinds of workgroup is as short as it can
// be; the length is returned.  A conv2 sample costs about COST2 / COST3 of a
// conv3 sample.  The counts are taken as padded for the XCDs: one workgroup too
// many on an XCD would run as a second round (batch 512: 58 us with 148 + 108
// workgroups, 19 + 14 on an XCD's 32 units).
constexpr int COST2 = 9, COST3 = 5;  // 7500 and 4140 cycles
static int wgrad_splits(int slots, int groups, int n, int* s3, int* s2) {
    const int most = min(n, WG_MAX_SPLITS / groups);
    int best = COST2 * n;  // one split of each, also where that is more than one round
    for (int a = 1; a <= most; ++a) {
        const int left = slots - pad_xcd(Wg2::SLICES * a * groups);
        const int b = min(most, (left > 0 ? left / NUM_XCD * NUM_XCD : 0) / (Wg3::SLICES * groups));
        if (b < 1) break;
        best = min(best, max(COST2 * ((n + a - 1) / a), COST3 * ((n + b - 1) / b)));
    }
    // the fewest splits of that length (fewer partial sums to add)
    const int per2 = max(1, best / COST2), per3 = max(1, best / COST3);
    *s2 = (n + per2 - 1) / per2;
    *s3 = (n + per3 - 1) / per3;
    return best;
}
static int wgrad_blocks(int groups, int s3, int s2) {
    return pad_xcd(Wg2::SLICES * s2 * groups) + pad_xcd(Wg3::SLICES * s3 * groups);
}

// Pairs of conv1 workgroups a group for one launch of all three layers, or 0
// where conv1 keeps a launch of its own.  Beside the others conv1 costs them
// units of the chip (a workgroup a unit, all resident at once), and saves its
// own launch, 6.5 us at 32 rows, as long as a conv2 range is at most one sample
// (3.3 us) longer.  A conv1 wave's unit of work costs about COST1.  Ranges are
// whole samples, so beyond the smallest sizes that holds where the two-launch
// ranges had slack: on 256 units for one learner of 1 .. 132, 145 .. 153, 161 ..
// 182 and 229 .. 234 rows, for two of up to 64, 73 .. 76, 81 .. 89 and 115, for
// four of up to 32, 37, 38, 41 .. 44 and 57; never with more rows than units.
// Whole step, two launches -> one, us: 8 rows 92.9 -> 86.6, 32 97.3 -> 91.3, 64
// 103.8 -> 99.0, 96 116.6 -> 110.3, 128 128.6 -> 120.1, 150 146.2 -> 137.5, 176
// 153.7 -> 146.7, 230 185.0 -> 175.4, 2 x 16 107.5 -> 101.2, 2 x 85 158.4 -> 150.5,
// 4 x 42 164.1 -> 156.3, 5 x 44 203.1 -> 187.7, 8 x 6 154.4 -> 150.0.
// (bf16 steps keep two launches: with one plane the others take 52 KB of LDS, two
// workgroups a unit, and conv1's 133 KB in the same launch would leave one.)
static int conv1_beside(int groups, int n, int cus, int* s3, int* s2) {
    constexpr int COST1 = 5;
    int pairs = 0, best = wgrad_splits(cus, groups, n, s3, s2) + COST2;
    if (groups * n > cus) return 0;  // (the search would say so, after up to 100 us)
    const int units = n * C1W_UNITS;
    for (int k = 1; COST1 * k <= best; ++k) {  // units a wave
        const int p = (units + C1W_WAVES * k - 1) / (C1W_WAVES * k), n1 = 2 * pad_xcd(p) * groups;
        if (p > CONV1_WG_MAX_SPLITS / groups || n1 >= cus) continue;
        int a3, a2;
        const int len = max(COST1 * k, wgrad_splits(cus - n1, groups, n, &a3, &a2));
        if (len > best || (pairs && len == best) || n1 + wgrad_blocks(groups, a3, a2) > cus) continue;
        pairs = p;
        best = len;
        *s3 = a3;
        *s2 = a2;
    }
    return pairs;
}

int launch_conv_wgrad(const float* dz3, bool dz3_bf16, const float* h2, const float* dz2, const float* h1,
                      int groups, int n, float* part3, float* part2, float* bias3, float* bias2,
                      int* s3, int* s2, const float* dz1, const uint8_t* const* ftab,
                      const uint8_t* zero_frame, float* part1, float* bias1, bool bf16, int cus,
                      hipStream_t st) {
    *s3 = *s2 = 0;
    if (n <= 0) return 0;
    C1wPart c1;
    if (!bf16) {
        const int pairs = conv1_beside(groups, n, max(1, cus), s3, s2);
        if (pairs) c1 = C1wPart{2 * pad_xcd(pairs), pairs, dz1, ftab, zero_frame, part1, bias1};
    } else {  // one plane: two workgroups a unit
        wgrad_splits(max(1, cus) * 2, groups, n, s3, s2);
    }
    const int blocks = c1.blocks * groups + wgrad_blocks(groups, *s3, *s2);
    auto go = [&](auto gp, auto with1, auto* z3, auto* z2) {
        conv_wgrad_kernel<decltype(gp)::value, decltype(with1)::value><<<blocks, WG_THREADS, 0, st>>>(
            z3, h2, z2, h1, groups, n, *s3, *s2, part3, part2, bias3, bias2, c1);
    };
    constexpr std::integral_constant<int, 3> fp32{};
    constexpr std::integral_constant<int, 1> one{};
    if (c1.blocks) go(fp32, std::true_type{}, dz3, dz2);
    else if (!bf16) go(fp32, std::false_type{}, dz3, dz2);
    else if (!dz3_bf16) go(one, std::false_type{}, dz3, (const uint16_t*)dz2);
    else go(one, std::false_type{}, (const uint16_t*)dz3, (const uint16_t*)dz2);
    return c1.splits;
}

}  // namespace gorila
