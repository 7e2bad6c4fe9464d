// Full-state branch combine on matrix cores (Fig. 2, eq. (1); eqs. (6)-(7)):
//
//   Psi[x] = s(x) * sum_b A_b[x_A] B_b[x_B]
//
// for a circuit cut into sides A and B (circuit_split): x_A / x_B are the
// bits of x on the two sides, A_b / B_b the branch states of the halves and
// s(x) = (-1)^{sum over folded pairs x_a x_b}.  As matrices, Psi = Ahat Bhat^T
// with Ahat[x_A][b] = A_b[x_A], a complex GEMM of shape 2^nA x 2^nB x nb.
//
// It runs as two real GEMMs over an interleaved index k = 2b + part:
//   Mr = sum_k A1[k] B1[k],  A1 = (Ar, -Ai),  B1 = (Br, Bi)
//   Mi = sum_k A2[k] B1[k],  A2 = (Ai,  Ar)
// The default form widens the FP32 inputs and multiplies on
// v_mfma_f64_16x16x4f64: every product is exact and every partial sum an FP64
// sum, so a component is off by the roundings of its own sum alone; the result
// is rounded once, to the complex64 state or not at all for a complex128 one.
// (Three real products per complex one, re = P - Q, im = S - P - Q, take 104 ms
// where these take 135.6; but then a component is as far off as the larger one
// of its amplitude, and a sum of 1024 branches 1.06 times as far in the 2-norm.)
// The FP32 form (v_mfma_f32_16x16x4f32, FP32 accumulation) runs at twice the
// matrix-core rate and is selected explicitly.
//
// The matrix cores bound all of it (a complex64 state is written once, the
// branch tables are read from the caches), so a workgroup owns a large tile:
// 128 x 128 outputs, eight waves with a 64 x 32 part each in FP64: 135.6 ms for
// 2^15 x 2^15 x 1024, 64.9 TFLOP/s.  A small matrix has few such tiles (2^8 x
// 2^8: four); below a tile for every CU it is cut into 32 x 32 tiles of four
// waves (2^8 x 2^8 x 500: 265 us, now 29).  Branch chunks are staged in LDS as k-major planes whose rows are
// 16 banks apart (an operand read covers four rows at a time); the next chunk's
// global loads are issued before the current chunk's MFMA work so that they
// overlap it.  The epilogue applies s(x) and scatters the tile to the state's
// natural index order through per-tile tables of the rows' and columns' output
// bits.  A launch covers one block of rows and columns (CombineArgs): the whole
// matrix for a two-part split, one value of the selector qubits for a three-part
// partition.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <cstring>
#include <type_traits>

#include "kernels.h"

namespace qsv {
namespace {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef double v4d __attribute__((ext_vector_type(4)));


// WR x WC waves, each MB x NB blocks of 16 x 16 outputs; kBr branches per LDS
// chunk; WPE waves per SIMD (bounds the registers).
template <bool F64, int MB, int NB, int WR, int WC, int kBr, int WPE>
__global__ void __launch_bounds__(64 * WR * WC, WPE)
k_combine_gemm(const float2 *__restrict__ A, const float2 *__restrict__ B, uint64_t nbr,
               const CombineArgs P, void *__restrict__ out, int out_c128) {
    using Real = typename std::conditional<F64, double, float>::type;
    using Acc = typename std::conditional<F64, v4d, v4f>::type;
    constexpr int NTH = 64 * WR * WC, TM = 16 * MB * WR, TN = 16 * NB * WC;
    constexpr int kK = 2 * kBr;  // interleaved K per chunk
    __shared__ __attribute__((aligned(16))) float a1[kK][TM + 16];
    __shared__ float a2[kK][TM + 16], b1[kK][TN + 16];
    __shared__ uint64_t rowx[TM], rowf[TM], colx[TN];
    const uint32_t t = threadIdx.x, lane = t & 63u, w = t >> 6;
    const uint64_t i0 = uint64_t(blockIdx.x) * TM, j0 = uint64_t(blockIdx.y) * TN;
    // this wave's part: rows rw + [0, 16 MB), columns cw + [0, 16 NB)
    const uint32_t rw = (w % WR) * 16 * MB, cw = (w / WR) * 16 * NB;
    const uint32_t lr = lane & 15u, lk = lane >> 4;
    Acc acc[MB][NB][2];  // re, im
#pragma unroll
    for (int m = 0; m < MB; ++m)
#pragma unroll
        for (int c = 0; c < NB; ++c)
#pragma unroll
            for (int q = 0; q < 2; ++q) acc[m][c][q] = Acc{0, 0, 0, 0};
    // staging: thread t always loads one in-tile row of every BS-th branch
    constexpr int BA = NTH / TM, BB = NTH / TN;  // branches staged at once
    constexpr int PA = kBr / BA, PB = kBr / BB;  // staged elements per thread
    static_assert(BA * TM == NTH && BB * TN == NTH && PA * BA == kBr && PB * BB == kBr, "staging covers a chunk");
    const uint32_t ba = t / TM, ra = t % TM, bb = t / TN, rb = t % TN;
    const float2 *pa = A + P.a_off + ba * P.a_stride + i0 + ra;
    const float2 *pb = B + P.b_off + bb * P.b_stride + j0 + rb;
    const uint64_t sa = BA * P.a_stride, sb = BB * P.b_stride;
    float2 na_[PA], nb_[PB];
    auto fetch = [&](uint64_t b0) {
#pragma unroll
        for (int q = 0; q < PA; ++q) {
            na_[q] = make_float2(0.f, 0.f);
            if (b0 + ba + BA * q < nbr) na_[q] = pa[q * sa];
        }
#pragma unroll
        for (int q = 0; q < PB; ++q) {
            nb_[q] = make_float2(0.f, 0.f);
            if (b0 + bb + BB * q < nbr) nb_[q] = pb[q * sb];
        }
        pa += kBr * P.a_stride;
        pb += kBr * P.b_stride;
    };
    auto mfma = [](Real a, Real b, Acc c) {
        if constexpr (F64) return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
        else return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    };
    fetch(0);
    for (uint64_t b0 = 0; b0 < nbr; b0 += kBr) {
        __syncthreads();  // previous chunk's fragments are read
#pragma unroll
        for (int q = 0; q < PA; ++q) {
            const uint32_t b = ba + BA * q;
            a1[2 * b][ra] = na_[q].x;
            a1[2 * b + 1][ra] = -na_[q].y;
            a2[2 * b][ra] = na_[q].y;
            a2[2 * b + 1][ra] = na_[q].x;
        }
#pragma unroll
        for (int q = 0; q < PB; ++q) {
            const uint32_t b = bb + BB * q;
            b1[2 * b][rb] = nb_[q].x;
            b1[2 * b + 1][rb] = nb_[q].y;
        }
        __syncthreads();
        if (b0 + kBr < nbr) fetch(b0 + kBr);  // in flight during the MFMA work
#pragma unroll
        for (int ks = 0; ks < kK; ks += 4) {
            Real f1[MB], f2[MB], g[NB];
#pragma unroll
            for (int m = 0; m < MB; ++m) {
                f1[m] = Real(a1[ks + lk][rw + m * 16 + lr]);
                f2[m] = Real(a2[ks + lk][rw + m * 16 + lr]);
            }
#pragma unroll
            for (int c = 0; c < NB; ++c) g[c] = Real(b1[ks + lk][cw + c * 16 + lr]);
#pragma unroll
            for (int m = 0; m < MB; ++m)
#pragma unroll
                for (int c = 0; c < NB; ++c) {
                    acc[m][c][0] = mfma(f1[m], g[c], acc[m][c][0]);
                    acc[m][c][1] = mfma(f2[m], g[c], acc[m][c][1]);
                }
        }
    }
    // epilogue: block (m, c) element r of this lane is row 4*lk + r (FP32
    // accumulators) or row 4*r + lk (FP64 accumulators), column lr.  The
    // output bits of the tile's rows and columns and the sign mask of each
    // row are tabulated once.
    for (uint32_t k = t; k < uint32_t(TM + TN); k += NTH) {
        if (k < uint32_t(TM)) {
            const uint64_t i = P.row_base + i0 + k;
            uint64_t x = 0, f = 0;
            for (int q = 0; q < P.na; ++q)
                if ((i >> q) & 1ull) x |= 1ull << P.pos_a[q];
            for (int g = 0; g < P.n_fold; ++g)
                if ((i >> P.fold_a[g]) & 1ull) f ^= 1ull << P.fold_b[g];
            rowx[k] = x;
            rowf[k] = f;
        } else {
            const uint64_t j = P.col_base + j0 + (k - TM);
            uint64_t x = 0;
            for (int q = 0; q < P.nb; ++q)
                if ((j >> q) & 1ull) x |= 1ull << P.pos_b[q];
            colx[k - TM] = x;
        }
    }
    __syncthreads();
    uint64_t xb[NB];
#pragma unroll
    for (int c = 0; c < NB; ++c) xb[c] = colx[cw + c * 16 + lr];
#pragma unroll
    for (int m = 0; m < MB; ++m) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const uint32_t il = rw + m * 16 + (F64 ? 4 * r + lk : 4 * lk + r);
            const uint64_t xa = rowx[il], fm = rowf[il];
#pragma unroll
            for (int c = 0; c < NB; ++c) {
                const uint64_t j = P.col_base + j0 + cw + c * 16 + lr;
                double vr = double(acc[m][c][0][r]), vi = double(acc[m][c][1][r]);
                if (__popcll(fm & j) & 1) { vr = -vr; vi = -vi; }
                if (out_c128) static_cast<double2 *>(out)[xa | xb[c]] = make_double2(vr, vi);
                else static_cast<float2 *>(out)[xa | xb[c]] = make_float2(float(vr), float(vi));
            }
        }
    }
}

template <bool F64, int MB, int NB, int WR, int WC, int kBr, int WPE>
hipError_t launch_gemm(const float2 *X, const float2 *Y, uint64_t nbr, const CombineArgs &Q, void *out, bool out_c128,
                       hipStream_t s) {
    const dim3 grid(unsigned((1ull << Q.na_blk) / (16 * MB * WR)), unsigned((1ull << Q.nb_blk) / (16 * NB * WC)));
    hipLaunchKernelGGL((k_combine_gemm<F64, MB, NB, WR, WC, kBr, WPE>), grid, dim3(64 * WR * WC), 0, s, X, Y, nbr, Q, out,
                       out_c128 ? 1 : 0);
    return hipGetLastError();
}

// Leading local bits of a side that land on output bits 0, 1, 2, ... in order.
static int low_run(const uint8_t *pos, int n) {
    int k = 0;
    while (k < n && pos[k] == k) ++k;
    return k;
}

}  // namespace

// The 16 lanes of an accumulator row hold 16 consecutive columns, so the
// epilogue's stores are contiguous when the column side carries the lowest
// output bits: the product is symmetric in the two sides (A_b B_b = B_b A_b,
// the sign is symmetric), so the sides are exchanged when side A holds the
// longer run of low output bits.
hipError_t launch_combine_gemm(const float2 *A, const float2 *B, uint64_t nbr, const CombineArgs &P,
                               void *out, bool fp64, bool out_c128, hipStream_t s) {
    CombineArgs Q = P;
    const float2 *X = A, *Y = B;
    if (low_run(P.pos_a, P.na) > low_run(P.pos_b, P.nb) && P.na_blk <= 22) {
        X = B;
        Y = A;
        Q.na = P.nb; Q.nb = P.na;
        Q.na_blk = P.nb_blk; Q.nb_blk = P.na_blk;
        Q.a_off = P.b_off; Q.b_off = P.a_off;
        Q.a_stride = P.b_stride; Q.b_stride = P.a_stride;
        Q.row_base = P.col_base; Q.col_base = P.row_base;
        std::memcpy(Q.pos_a, P.pos_b, sizeof(Q.pos_a));
        std::memcpy(Q.pos_b, P.pos_a, sizeof(Q.pos_b));
        std::memcpy(Q.fold_a, P.fold_b, sizeof(Q.fold_a));
        std::memcpy(Q.fold_b, P.fold_a, sizeof(Q.fold_b));
    }
    // 128 x 128 tiles when there is one for every CU, else 32 x 32 (500
    // branches: 2^10 x 2^10 89 us against 269 on large tiles; 300 branches:
    // 2^12 x 2^12 680 us on large tiles).  The order of the products is the same
    // for every tile and chunk (FP64, 2^15 x 2^15 x 1024: chunks of 8 branches
    // 135.6 ms, of 16 135.2, 2^11 x 2^11 x 37 31 and 36 us).
    const bool large = Q.na_blk + Q.nb_blk >= 14 + 8;
    if (!fp64)
        return large ? launch_gemm<false, 4, 4, 2, 2, 16, 2>(X, Y, nbr, Q, out, out_c128, s)
                     : launch_gemm<false, 1, 1, 2, 2, 32, 1>(X, Y, nbr, Q, out, out_c128, s);
    return large ? launch_gemm<true, 4, 2, 2, 4, 8, 2>(X, Y, nbr, Q, out, out_c128, s)
                 : launch_gemm<true, 1, 1, 2, 2, 32, 1>(X, Y, nbr, Q, out, out_c128, s);
}

}  // namespace qsv
