// FC-512 (Section 5.1) on bf16 planes (planes.h): the forward product of the
// forward-only calls and both gradients of the layer (eq. (2)), as tiles
//   C[row][col] = sum_k A[row][k] B[col][k],   BM rows x BN columns,
// by one workgroup, in chunks of 32 reduction indices that are
// split into planes as they are staged in LDS (double buffered, one barrier a
// chunk).  Both operands lie in LDS as [row][32 k]: an operand whose rows are
// contiguous in k is stored as it is loaded; one whose k is the slow index is
// loaded as 4 k x 4 (or 2) row blocks and transposed in registers.
//
// A wave takes 32 (or 16) rows x 64 columns, so that a lane ends with four
// consecutive columns, stored as one vector, and with three planes LDS and
// matrix cores are about equally busy.  fp32 tiles are 128 x 128 (eight waves):
// the split of an operand, 5.5 vector instructions a value, is repeated in
// every tile that reads it, and 128 x 64 tiles, with half as many again per
// product, ran no faster than the fp32 matrix instructions (forward, 1024
// states: 25.8 us; both gradients at batch 512: 38.3 us).  One plane needs no
// such reuse and takes small tiles, for more of them a unit.  A second set of
// staging registers (values asked for two chunks ahead) moved nothing with
// three planes and cost a sixth with one (registers, so waves a unit).
//
// Measured, from the fp32 matrix instructions: forward, 1024 states, 33.5 ->
// 21.8 us; both gradients, 2001 rows, 122 -> 105 us, 512 rows, 36 -> 30 us; bf16,
// 16 learners x 64 rows, 54 -> 40 us (with dz3 stored in flatten order, which
// alone took 512 rows from 36 to 32 us).
#pragma once
#include "common.h"
#include "kernels.h"
#include "planes.h"

#include <type_traits>

namespace gorila {

typedef uint16_t u16x2a __attribute__((ext_vector_type(2), aligned(2)));

// 64 bytes a row and plane, two rows a 128-byte line, chunks of 8 k permuted so
// that eight neighbouring rows' chunks fall into different banks.
__device__ inline int pg_off(int row, int chunk) { return row * 64 + ((chunk ^ (row >> 1 & 3)) << 4); }

// LDS row of tile row r (N rows in all): rows 4 i + c lie at c N / 4 + i, so that
// threads that hold four neighbouring rows store to neighbouring LDS rows, and
// column tiles t = 0 .. 3 of 16 lanes hold columns 4 lane + t.
template <int N> __device__ inline int pg_slot(int r) { return (r & 3) * (N / 4) + (r >> 2); }
template <int N> __device__ inline int pg_row(int slot) { return (slot % (N / 4)) * 4 + slot / (N / 4); }

__device__ inline f32x2 pg_ld2(const float* p) {
    typedef float f32x2a __attribute__((ext_vector_type(2), aligned(4)));
    const f32x2a v = *(const f32x2a*)p;
    return f32x2{v[0], v[1]};
}
__device__ inline f32x2 pg_ld2(const uint16_t* p) {
    const u16x2a v = *(const u16x2a*)p;
    return f32x2{__uint_as_float((uint32_t)v[0] << 16), __uint_as_float((uint32_t)v[1] << 16)};
}

// An operand of N rows: ld elements between its slow index's steps.
//  KMAJ: element (row, k) at p[row * ld + k]; rows >= nrow read row 0
//  else: element (row, k) at p[k * ld + row]; k >= nk is zero (ZERO) or reads k
//        0, and row blocks past nrow (a multiple of 4) read the first
template <int N, int THREADS, bool KMAJ_, class T, bool ZERO = false>
struct PgOperand {
    static constexpr int Q = N * 32 / 4 / THREADS;          // quads a thread
    static constexpr bool KM = KMAJ_;
    static constexpr int W = KMAJ_ ? 4 : Q;                 // !KMAJ: rows of a thread's block
    static_assert(KMAJ_ || Q == 2 || Q == 4, "blocks of 4 k x 2 or 4 rows");
    const T* p;
    int64_t ld;
    int nrow, nk;
    f32x4 v[Q];
    // !KMAJ: thread = (k quad, row block); a wave's lanes run along the rows
    __device__ __forceinline__ static int kq(int tid) { return tid / (N / W); }
    __device__ __forceinline__ static int rb(int tid) { return tid % (N / W) * W; }
    __device__ __forceinline__ void fetch(int tid, int k0) {
        if constexpr (KMAJ_) {
#pragma unroll
            for (int j = 0; j < Q; ++j) {
                const int e = tid + THREADS * j, row = e >> 3;
                v[j] = ldqa(p + (row < nrow ? row : 0) * ld + k0 + (e & 7) * 4);
            }
        } else {
            const int k = k0 + 4 * kq(tid);
            f32x4 r[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const T* q = p + (int64_t)(k + j < nk ? k + j : 0) * ld + (rb(tid) < nrow ? rb(tid) : 0);
                if constexpr (W == 4) {
                    r[j] = ldqa(q);
                } else {
                    const f32x2 x = pg_ld2(q);
                    r[j] = f32x4{x[0], x[1], 0.f, 0.f};
                }
                if (ZERO) r[j] = sel4(k + j < nk, r[j]);
            }
#pragma unroll
            for (int c = 0; c < W; ++c) v[c] = f32x4{r[0][c], r[1][c], r[2][c], r[3][c]};
        }
    }
    template <int P>
    __device__ __forceinline__ void stage(int tid, char* s) const {
#pragma unroll
        for (int j = 0; j < Q; ++j) {
            int row, k;
            if constexpr (KMAJ_) {
                row = (tid + THREADS * j) >> 3;
                k = (tid & 7) * 4;
            } else {
                row = rb(tid) + j;
                k = 4 * kq(tid);
            }
            bf16x4 o[P];
            split4<P>(v[j], o);
            char* const d = s + pg_off(pg_slot<N>(row), k >> 3) + ((k & 4) << 1);
#pragma unroll
            for (int pl = 0; pl < P; ++pl) *(bf16x4*)(d + pl * N * 64) = o[pl];
        }
    }
};

// One tile: chunks [c0, c1).  epi(row, col, v): four consecutive columns.
// rowsum (or null): rowsum[row] = sum over the chunks of A's values (A not KMAJ).
template <int BM, int BN>
constexpr int PG_THREADS = 256 * (BN / 64);
template <int BM, int BN, int P, class OA, class OB, class Epi>
__device__ __forceinline__ void pg_tile(char* lds, int c0, int c1, OA& a, OB& b, Epi&& epi, float* rowsum) {
    constexpr int STAGE = P * (BM + BN) * 64, RT = BM / 64, CG = BN / 64;  // 16-row tiles a wave; column groups
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rg = wave >> (CG - 1), cg = wave & (CG - 1);  // CG is 1 or 2
    f32x4 hi[RT][4], lo[RT][4];
    float rs[OA::Q] = {};
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) hi[i][j] = lo[i][j] = f32x4{};
    auto fetch = [&](int c) {
        a.fetch(tid, c * 32);
        b.fetch(tid, c * 32);
    };
    auto stage = [&](char* s) {
        if (rowsum)
#pragma unroll
            for (int c = 0; c < OA::Q; ++c) rs[c] += (a.v[c][0] + a.v[c][1]) + (a.v[c][2] + a.v[c][3]);
        a.template stage<P>(tid, s);
        b.template stage<P>(tid, s + P * BM * 64);
    };
    auto compute = [&](const char* s) {
        bf16x8 av[RT][P], bv[4][P];
        const int off = pg_off(lane & 15, lane >> 4);  // rows 16 apart permute alike
#pragma unroll
        for (int pl = 0; pl < P; ++pl) {
#pragma unroll
            for (int i = 0; i < RT; ++i)
                av[i][pl] = *(const bf16x8*)(s + pl * BM * 64 + (rg * RT + i) * 1024 + off);
#pragma unroll
            for (int j = 0; j < 4; ++j)
                bv[j][pl] = *(const bf16x8*)(s + P * BM * 64 + pl * BN * 64 + (j * CG + cg) * 1024 + off);
        }
        plane_products<0>(av, bv, hi, lo);
    };
    fetch(c0);
    stage(lds);
    if (c0 + 1 < c1) fetch(c0 + 1);
    __syncthreads();
    for (int c = c0; c < c1; ++c) {
        compute(lds + ((c - c0) & 1) * STAGE);
        if (c + 1 < c1) {
            stage(lds + ((c + 1 - c0) & 1) * STAGE);
            if (c + 2 < c1) fetch(c + 2);
        }
        __syncthreads();
    }
    if constexpr (!OA::KM)
        if (rowsum) {  // the eight k quads of every row, in order
            float* const red = (float*)lds;
#pragma unroll
            for (int c = 0; c < OA::Q; ++c) red[OA::kq(tid) * BM + OA::rb(tid) + c] = rs[c];
            __syncthreads();
            if (tid < BM) {
                float t = 0.0f;
                for (int k = 0; k < 8; ++k) t += red[k * BM + tid];
                rowsum[tid] = t;
            }
        }
    int el = lane;
    asm volatile("" : "+v"(el));  // addresses are computed here, not held over the loop
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int row = pg_row<BM>((rg * RT + i) * 16 + 4 * (el >> 4) + e);
            epi(row, cg * 64 + 4 * (el & 15),
                plane_sum<P>(f32x4{hi[i][0][e], hi[i][1][e], hi[i][2][e], hi[i][3][e]},
                          f32x4{lo[i][0][e], lo[i][1][e], lo[i][2][e], lo[i][3][e]}));
        }
}
template <int BM, int BN, int P>
constexpr int PG_SMEM = 2 * P * (BM + BN) * 16;  // floats

// Forward: partial[s][row][512] over chunk ranges (as the fp32 launch).
struct PgFwdJob {
    const float* h3;
    const float* w4;
    float* partial;
    int n, splits, cps;
    static constexpr int BM = 128, BN = 128, THREADS = PG_THREADS<BM, BN>, SMEM = PG_SMEM<BM, BN, 3>;
    __host__ __device__ int mt() const { return (n + BM - 1) / BM; }
    __host__ __device__ int tiles() const { return mt() * (HID / BN) * splits; }
    __host__ __device__ int blocks() const { return pad_xcd(tiles()); }
    __device__ void run(int bid, float* smem) const {
        int t = xcd_tile(bid, blocks());
        if (t >= tiles()) return;
        const int r0 = t % mt() * BM;
        t /= mt();
        const int c0 = t % (HID / BN) * BN, s = t / (HID / BN);
        PgOperand<BM, THREADS, true, float> a{h3 + (int64_t)r0 * FLAT, FLAT, n - r0, 0, {}};
        PgOperand<BN, THREADS, true, float> b{w4 + (int64_t)c0 * FLAT, FLAT, BN, 0, {}};
        float* const out = partial + (int64_t)s * n * HID;
        pg_tile<BM, BN, 3>((char*)smem, s * cps, min(FLAT / 32, (s + 1) * cps), a, b,
                           [&](int row, int col, f32x4 v) {
                               if (r0 + row < n) *(f32x4*)(out + (int64_t)(r0 + row) * HID + c0 + col) = v;
                           },
                           nullptr);
    }
};

// Weight gradient: dW4[o][k] = sum_b dz4[b][o] h3[b][k], rows o, columns k; db4
// as the row sums.
template <int BM, int BN, int GP>
struct PgWgradJob {
    const float* dz4;
    const float* h3;
    float* grads;
    int64_t grads_stride;
    int n, groups;
    static constexpr int THREADS = PG_THREADS<BM, BN>, SMEM = PG_SMEM<BM, BN, GP>;
    static constexpr int NT = (FLAT + BN - 1) / BN;
    __host__ __device__ int tiles() const { return HID / BM * NT; }
    __host__ __device__ int blocks() const { return pad_xcd(tiles() * groups); }
    __device__ void run(int bid, float* smem) const {
        int t = xcd_tile(bid, blocks());
        if (t >= tiles() * groups) return;
        const int g = t / tiles();
        t -= g * tiles();
        const int r0 = t % (HID / BM) * BM, c0 = t / (HID / BM) * BN;
        const int64_t rows = (int64_t)g * n;
        float* const gr = grads + g * grads_stride;
        PgOperand<BM, THREADS, false, float, true> a{dz4 + rows * HID + r0, HID, BM, n, {}};
        PgOperand<BN, THREADS, false, float> b{h3 + rows * FLAT + c0, FLAT, FLAT - c0, n, {}};
        pg_tile<BM, BN, GP>((char*)smem, 0, (n + 31) / 32, a, b,
                            [&](int row, int col, f32x4 v) {
                                if (c0 + col < FLAT)
                                    *(f32x4a*)(gr + OFF_W4 + (int64_t)(r0 + row) * FLAT + c0 + col) = v;
                            },
                            c0 == 0 ? gr + OFF_B4 + r0 : nullptr);
    }
};

// Data gradient: dz3[b][k] = [h3 > 0] sum_o W4[o][k] dz4[b][o].
template <int BM, int BN, int GP, class TW>
struct PgDgradJob {
    const float* dz4;
    GroupPtrs theta;
    GroupPtrs16 w4b;  // TW = uint16_t: W4 of each set, read in place
    const float* h3;
    float* dz3;       // GP == 1: bf16 bit patterns
    int n, groups;
    static constexpr int THREADS = PG_THREADS<BM, BN>, SMEM = PG_SMEM<BM, BN, GP>;
    static constexpr int NT = (FLAT + BN - 1) / BN;
    __host__ __device__ int tiles() const { return (n + BM - 1) / BM * NT; }
    __host__ __device__ int blocks() const { return pad_xcd(tiles() * groups); }
    __device__ void run(int bid, float* smem) const {
        int t = xcd_tile(bid, blocks());
        if (t >= tiles() * groups) return;
        const int g = t / tiles();
        t -= g * tiles();
        const int mt = (n + BM - 1) / BM, r0 = t % mt * BM, c0 = t / mt * BN;
        const int64_t rows = (int64_t)g * n + r0;
        const TW* w4;
        if constexpr (std::is_same_v<TW, float>) w4 = theta.p[g] + OFF_W4;
        else w4 = w4b.p[g];
        PgOperand<BM, THREADS, true, float> a{dz4 + rows * HID, HID, n - r0, 0, {}};
        PgOperand<BN, THREADS, false, TW> b{w4 + c0, FLAT, FLAT - c0, HID, {}};
        pg_tile<BM, BN, GP>((char*)smem, 0, HID / 32, a, b,
                            [&](int row, int col, f32x4 v) {
                                if (r0 + row >= n || c0 + col >= FLAT) return;
                                const f32x4 h = ld4(h3 + (rows + row) * FLAT + c0 + col);
                                const f32x4 x{h[0] > 0.f ? v[0] : 0.f, h[1] > 0.f ? v[1] : 0.f,
                                              h[2] > 0.f ? v[2] : 0.f, h[3] > 0.f ? v[3] : 0.f};
                                const int64_t at = (rows + row) * FLAT + c0 + col;
                                if constexpr (GP == 1) stq((uint16_t*)dz3 + at, x);
                                else stq(dz3 + at, x);
                            },
                            nullptr);
    }
};

}  // namespace gorila
