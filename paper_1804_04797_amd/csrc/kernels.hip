// HIP kernels of the state-vector sweep for gfx950 (MI355X), and their
// host-side launchers.
//
// State: 2^n complex64 amplitudes, interleaved (re, im) float32, qubit k =
// index bit k (Section 2, preliminaries).  All kernels use 64-bit indices
// (2^34 amplitudes exceed 32 bits).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <cstring>

#include "kernels.h"

namespace qsv {
namespace {

__device__ __forceinline__ float2 f2(float x, float y) { return make_float2(x, y); }

typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v2f __attribute__((ext_vector_type(2)));

__device__ __forceinline__ float2 cmul(float2 a, float cr, float ci) {
    return f2(a.x * cr - a.y * ci, a.x * ci + a.y * cr);
}

// Gather for every entry of a batch: out[e*m + k] = amps_e[xs[e*m + k]].
__global__ void __launch_bounds__(256)
k_gather_batch(const BatchEntry *__restrict__ ents, uint64_t count, const uint64_t *__restrict__ xs,
               uint64_t m, float2 *__restrict__ out) {
    const uint64_t i = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i >= count * m) return;
    const BatchEntry en = ents[i / m];
    const uint64_t x = xs[i];
    const float2 *a = reinterpret_cast<const float2 *>(en.amps);
    out[i] = (x < (1ull << en.n)) ? a[x] : f2(__builtin_nanf(""), __builtin_nanf(""));
}


// ---------------------------------------------------------------------------
// Dense block on matrix cores: Y = M X for a 2^K x 2^K complex matrix M on K
// qubits.  A tile is 2^K rows (the block's qubits) x 64 columns (the six
// lowest other index bits); the remaining bits select the tile.  Persistent
// workgroups keep M^T (re, im) in LDS and loop over tiles: load the tile into
// LDS as separate re/im planes, form Yr = Mr Xr - Mi Xi and Yi = Mr Xi + Mi Xr
// with v_mfma_f32_16x16x4_f32 (four real products; wave w owns 16-row output
// blocks), write Y back through LDS and store it in place.
// ---------------------------------------------------------------------------
// 32-bit words only: the kernels read them with scalar loads.  (Read as bytes,
// the tile's origin was a chain of vector loads per tile, one per bit, whose
// waits also waited for the next tile's loads: 24 qubits, k = 4, 5, 6, 7: 63.8,
// 61.1, 96.5, 159.3 us per block, now 43.6, 51.7, 84.9, 144.4; k = 4 is bound by
// the state's traffic, 6.2 TB/s, k = 7 by the matrix cores, 119 TFLOP/s.)
struct DenseArgs {
    uint64_t tiles;
    uint32_t run[20];          // tile index -> origin: bits [src, src + len) to bit dst (src | len << 8 | dst << 16)
    uint32_t n_runs;
    uint32_t phys[16];         // tile local bit i -> physical bit
    uint32_t sub[16];          // position of local bit i within the row or column index
    uint32_t rowmask;          // local bits that belong to the row index
};

__device__ __forceinline__ uint64_t dense_origin(const DenseArgs &A, uint64_t tile) {
    uint64_t base = 0;
    for (uint32_t r = 0; r < A.n_runs; ++r) {
        const uint32_t x = A.run[r];
        base |= ((tile >> (x & 0xffu)) & ((1ull << ((x >> 8) & 0xffu)) - 1ull)) << (x >> 16);
    }
    return base;
}

template <int K>
__global__ void __launch_bounds__(256)
k_dense(float2 *__restrict__ amps, const float *__restrict__ mat_t, const DenseArgs A) {
    constexpr int DIM = 1 << K;
    constexpr int COLS = 64;
    constexpr int XS = COLS + 4;             // padded row stride of the X planes
    constexpr int PER = (DIM * COLS) / 256;  // elements per thread
    constexpr int NB = DIM / 16;             // 16x16 output blocks per wave
    __shared__ float mtr[DIM * DIM], mti[DIM * DIM];
    __shared__ float xr[DIM * XS], xi[DIM * XS];
    const uint32_t t = threadIdx.x, lane = t & 63u, w = t >> 6;
    for (uint32_t i = t; i < uint32_t(DIM * DIM); i += 256) {
        mtr[i] = mat_t[i];
        mti[i] = mat_t[DIM * DIM + i];
    }
    // thread part of the tile-local index: bits 0..7
    uint64_t poff_t = 0;
    uint32_t row_t = 0, col_t = 0;
#pragma unroll
    for (int b = 0; b < 8; ++b) {
        if (!((t >> b) & 1u)) continue;
        poff_t |= 1ull << A.phys[b];
        if ((A.rowmask >> b) & 1u) row_t |= 1u << A.sub[b];
        else col_t |= 1u << A.sub[b];
    }
    const uint32_t rb0 = (w * NB) / 4;       // row block of this wave
    const uint32_t cb0 = (w * NB) % 4;       // first column block
    for (uint64_t tile = blockIdx.x; tile < A.tiles; tile += gridDim.x) {
        const uint64_t base = dense_origin(A, tile);
        __syncthreads();  // previous tile's LDS reads are complete
#pragma unroll
        for (int it = 0; it < PER; ++it) {
            uint64_t poff = poff_t;
            uint32_t row = row_t, col = col_t;
#pragma unroll
            for (int b = 8; b < K + 6; ++b) {
                if (!((it >> (b - 8)) & 1)) continue;
                poff |= 1ull << A.phys[b];
                if ((A.rowmask >> b) & 1u) row |= 1u << A.sub[b];
                else col |= 1u << A.sub[b];
            }
            const float2 v = amps[base | poff];
            xr[row * XS + col] = v.x;
            xi[row * XS + col] = v.y;
        }
        __syncthreads();
        v4f ar[NB], ai[NB];
#pragma unroll
        for (int b = 0; b < NB; ++b) { ar[b] = v4f{0, 0, 0, 0}; ai[b] = v4f{0, 0, 0, 0}; }
        const uint32_t lr = lane & 15u, lk = lane >> 4;
#pragma unroll 4
        for (int kk = 0; kk < DIM; kk += 4) {
            const float a_r = mtr[(kk + lk) * DIM + rb0 * 16 + lr];
            const float a_i = mti[(kk + lk) * DIM + rb0 * 16 + lr];
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                const uint32_t cb = cb0 + b;
                const float b_r = xr[(kk + lk) * XS + cb * 16 + lr];
                const float b_i = xi[(kk + lk) * XS + cb * 16 + lr];
                ar[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(a_r, b_r, ar[b], 0, 0, 0);
                ar[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(-a_i, b_i, ar[b], 0, 0, 0);
                ai[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(a_r, b_i, ai[b], 0, 0, 0);
                ai[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(a_i, b_r, ai[b], 0, 0, 0);
            }
        }
        __syncthreads();  // all waves are done reading X
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const uint32_t cb = cb0 + b;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const uint32_t row = rb0 * 16 + 4 * lk + r, col = cb * 16 + lr;
                xr[row * XS + col] = ar[b][r];
                xi[row * XS + col] = ai[b][r];
            }
        }
        __syncthreads();
#pragma unroll
        for (int it = 0; it < PER; ++it) {
            uint64_t poff = poff_t;
            uint32_t row = row_t, col = col_t;
#pragma unroll
            for (int b = 8; b < K + 6; ++b) {
                if (!((it >> (b - 8)) & 1)) continue;
                poff |= 1ull << A.phys[b];
                if ((A.rowmask >> b) & 1u) row |= 1u << A.sub[b];
                else col |= 1u << A.sub[b];
            }
            amps[base | poff] = f2(xr[row * XS + col], xi[row * XS + col]);
        }
    }
}

// Dense block for k = 6, 7: Y = M X with the 2^k x 2^k matrix M held in
// registers.  Wave w of a workgroup owns output rows [16 w, 16 w + 16) (its
// strip of Mr and Mi, 2^k / 2 registers per lane, loaded once) and computes
// them for a tile of 64 columns: Yr = Mr Xr - Mi Xi and Yi = Mr Xi + Mi Xr on
// v_mfma_f32_16x16x4f32 (FP32 accumulation; the two products of Yi of a
// block are issued four instructions apart).  A tile is 2^(k+6) amplitudes whose
// local index bits are its physical bits from the lowest up (the block's k
// qubits and the 6 lowest other qubits; physical bit 0 is always among
// them), so thread t's 16-byte accesses at local indices 2 (i NT + t) are
// contiguous across a wave whatever the block's qubits.  Loads go to
// registers, then to LDS planes (re, im) at each element's (row, column):
// element (r, c) at 80 r + r / 4 + c (a stride of 80 puts the 4 rows one
// MFMA operand read covers on distinct bank groups; the extra r / 4 spreads
// rows that differ in their higher bits, as when the block holds the lowest
// qubits and a wave's lanes walk its rows, over distinct banks, and is a
// constant per operand read).  The results go back through the same planes
// and leave in the same physical order (16-byte stores from every lane:
// faster than storing the accumulators' 8-byte elements directly, even
// where 16 lanes would write 16 consecutive amplitudes).  Persistent workgroups walk the tiles;
// the next tile's loads are issued before the current tile's matrix-core work.
template <int K>
__global__ void __launch_bounds__(64 * (1 << K) / 16, K == 6 ? 2 : 1)
k_dense_strip(float2 *__restrict__ amps, const float *__restrict__ mat_t, const DenseArgs A) {
    constexpr int DIM = 1 << K;
    constexpr int WAVES = DIM / 16;
    constexpr int NT = 64 * WAVES;          // threads
    constexpr int COLS = 64;
    constexpr int XS = 80;                   // row stride of the X planes (floats)
    constexpr int KS = DIM / 4;              // k-steps of 4
    constexpr int PAIRS = DIM * COLS / 2;    // amplitude pairs of a tile
    constexpr int PER = PAIRS / NT;          // pairs per thread (8)
    static_assert(PER * NT == PAIRS, "tile split");
    constexpr int PLANE = DIM * XS + DIM / 4;
    __shared__ float xr[PLANE], xi[PLANE];
    const uint32_t t = threadIdx.x, lane = t & 63u, w = t >> 6;
    const uint32_t lr = lane & 15u, lk = lane >> 4;
    auto at = [](uint32_t row, uint32_t col) { return row * XS + (row >> 2) + col; };
    // this wave's strip of M: A operand of k-step ks, lane (k % 4) * 16 + i
    float mr[KS], mi[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
        const uint32_t k = uint32_t(ks) * 4u + lk, row = w * 16u + lr;
        mr[ks] = mat_t[k * DIM + row];
        mi[ks] = mat_t[DIM * DIM + k * DIM + row];
    }
    // pair it of this thread: local index l = 2 (it NT + t).  Bits 1..TB of
    // l come from t and the higher ones from it, so its physical offset and
    // its (row, column) are the OR of a per-thread part and a part common to
    // the workgroup; l + 1 is the next amplitude in memory and differs in
    // local bit 0 (a row or a column bit).
    constexpr int TB = K + 2;  // log2(NT)
    static_assert((1 << TB) == NT && (PER << TB) == PAIRS, "pair index split");
    uint64_t off_t = 0;
    uint32_t row_t = 0, col_t = 0;
#pragma unroll
    for (int b = 1; b <= TB; ++b) {
        if (!((t >> (b - 1)) & 1u)) continue;
        off_t |= 1ull << A.phys[b];
        if ((A.rowmask >> b) & 1u) row_t |= 1u << A.sub[b];
        else col_t |= 1u << A.sub[b];
    }
    auto off_it = [&](int it) {
        uint64_t o = 0;
#pragma unroll
        for (int b = TB + 1; b < K + 6; ++b)
            if ((it >> (b - TB - 1)) & 1) o |= 1ull << A.phys[b];
        return o;
    };
    auto rc_it = [&](int it, uint32_t &row, uint32_t &col) {
        row = row_t;
        col = col_t;
#pragma unroll
        for (int b = TB + 1; b < K + 6; ++b) {
            if (!((it >> (b - TB - 1)) & 1)) continue;
            if ((A.rowmask >> b) & 1u) row |= 1u << A.sub[b];
            else col |= 1u << A.sub[b];
        }
    };
    const bool b0row = (A.rowmask & 1u) != 0;
    const uint32_t b0 = 1u << A.sub[0];
    v4f nx[PER];
    auto fetch = [&](uint64_t base) {
#pragma unroll
        for (int it = 0; it < PER; ++it)
            nx[it] = __builtin_nontemporal_load(reinterpret_cast<const v4f *>(amps + (base | off_t | off_it(it))));
    };
    uint64_t tile = blockIdx.x;
    uint64_t next = dense_origin(A, tile);
    if (tile < A.tiles) fetch(next);
    for (; tile < A.tiles; tile += gridDim.x) {
        const uint64_t base = next;
        __syncthreads();  // the previous tile's LDS reads are complete
#pragma unroll
        for (int it = 0; it < PER; ++it) {
            uint32_t row, col;
            rc_it(it, row, col);
            const uint32_t p0 = at(row, col), p1 = b0row ? at(row | b0, col) : at(row, col | b0);
            xr[p0] = nx[it].x;
            xi[p0] = nx[it].y;
            xr[p1] = nx[it].z;
            xi[p1] = nx[it].w;
        }
        __syncthreads();
        next = dense_origin(A, tile + gridDim.x);
        if (tile + gridDim.x < A.tiles) fetch(next);  // in flight during the MFMA work
        v4f arr[4], aii[4], ai[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            arr[c] = v4f{0, 0, 0, 0};
            aii[c] = arr[c];
            ai[c] = arr[c];
        }
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const uint32_t krow = uint32_t(ks) * 4u + lk;
            float br[4], bi[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                br[c] = xr[at(krow, uint32_t(c) * 16u + lr)];
                bi[c] = xi[at(krow, uint32_t(c) * 16u + lr)];
            }
#pragma unroll
            for (int c = 0; c < 4; ++c) ai[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(mr[ks], bi[c], ai[c], 0, 0, 0);
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                arr[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(mr[ks], br[c], arr[c], 0, 0, 0);
                aii[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(mi[ks], bi[c], aii[c], 0, 0, 0);
                ai[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(mi[ks], br[c], ai[c], 0, 0, 0);
            }
        }
        // element r of block c: row 16 w + 4 lk + r, column 16 c + lr
        __syncthreads();  // every wave's operand reads of X are complete
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const uint32_t p = at(w * 16u + 4u * lk + uint32_t(r), uint32_t(c) * 16u + lr);
                xr[p] = arr[c][r] - aii[c][r];
                xi[p] = ai[c][r];
            }
        __syncthreads();
#pragma unroll
        for (int it = 0; it < PER; ++it) {
            uint32_t row, col;
            rc_it(it, row, col);
            const uint32_t p0 = at(row, col), p1 = b0row ? at(row | b0, col) : at(row, col | b0);
            const v4f y = {xr[p0], xi[p0], xr[p1], xi[p1]};
            __builtin_nontemporal_store(y, reinterpret_cast<v4f *>(amps + (base | off_t | off_it(it))));
        }
    }
}

template <int K>
hipError_t launch_dense_strip_t(float2 *amps, const float *mat_t, const DenseArgs &A, hipStream_t s) {
    constexpr int NT = 64 * (1 << K) / 16;
    int per_cu = 0, dev = 0, cus = 0;
    hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
        &per_cu, reinterpret_cast<const void *>(&k_dense_strip<K>), NT, 0);
    if (e == hipSuccess) e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e != hipSuccess) return e;
    const uint64_t resident = uint64_t(std::max(1, per_cu)) * uint64_t(std::max(1, cus));
    const uint64_t grid = A.tiles < resident ? A.tiles : resident;
    hipLaunchKernelGGL((k_dense_strip<K>), dim3(unsigned(grid)), dim3(NT), 0, s, amps, mat_t, A);
    return hipGetLastError();
}

template <int K>
hipError_t launch_dense_t(float2 *amps, int n, const int *qubits, const float *mat_t,
                          hipStream_t s) {
    DenseArgs A;
    std::memset(&A, 0, sizeof(A));
    uint64_t qmask = 0;
    for (int i = 0; i < K; ++i) qmask |= 1ull << qubits[i];
    // column bits: the six lowest bits outside the block
    uint64_t cmask = 0;
    for (int q = 0, c = 0; q < n && c < 6; ++q)
        if (!((qmask >> q) & 1)) { cmask |= 1ull << q; ++c; }
    const uint64_t res = qmask | cmask;
    int li = 0, ci = 0;
    for (int q = 0; q < n; ++q) {
        if (!((res >> q) & 1)) continue;
        A.phys[li] = uint32_t(q);
        if ((qmask >> q) & 1) {
            A.rowmask |= 1u << li;
            // row index bit = position of q in the block's qubit list
            int pos = 0;
            while (qubits[pos] != q) ++pos;
            A.sub[li] = uint32_t(pos);
        } else {
            A.sub[li] = uint32_t(ci++);
        }
        ++li;
    }
    for (int q = 0, src = 0; q < n;) {  // runs of non-resident bits
        if ((res >> q) & 1) { ++q; continue; }
        int e = q;
        while (e < n && !((res >> e) & 1)) ++e;
        A.run[A.n_runs++] = uint32_t(src) | uint32_t(e - q) << 8 | uint32_t(q) << 16;
        src += e - q;
        q = e;
    }
    A.tiles = 1ull << (n - K - 6);
    if constexpr (K >= 6) {
        return launch_dense_strip_t<K>(amps, mat_t, A, s);
    } else {
        const uint64_t grid = A.tiles < 1024 ? A.tiles : 1024;
        hipLaunchKernelGGL((k_dense<K>), dim3(unsigned(grid)), dim3(256), 0, s, amps, mat_t, A);
        return hipGetLastError();
    }
}

// ---------------------------------------------------------------------------
// Plain (unfused) gate kernels: one launch per gate.
// ---------------------------------------------------------------------------

__device__ __forceinline__ uint64_t insert_zero(uint64_t i, int q) {
    const uint64_t lo = i & ((1ull << q) - 1);
    return ((i >> q) << (q + 1)) | lo;
}

// General single-qubit gate, pair rule of Section 2 (preliminaries).
__global__ void __launch_bounds__(256)
k_plain_1q(float2 *__restrict__ a, uint64_t pairs, int q, float m0r, float m0i, float m1r,
           float m1i, float m2r, float m2i, float m3r, float m3i) {
    const uint64_t stride = uint64_t(gridDim.x) * blockDim.x;
    for (uint64_t i = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < pairs; i += stride) {
        const uint64_t lo = insert_zero(i, q), hi = lo | (1ull << q);
        const float2 x = a[lo], y = a[hi];
        a[lo] = f2(m0r * x.x - m0i * x.y + m1r * y.x - m1i * y.y,
                   m0r * x.y + m0i * x.x + m1r * y.y + m1i * y.x);
        a[hi] = f2(m2r * x.x - m2i * x.y + m3r * y.x - m3i * y.y,
                   m2r * x.y + m2i * x.x + m3r * y.y + m3i * y.x);
    }
}

// Multiply amplitudes with bit q = 1 by (cr, ci): touches half the state.
__global__ void __launch_bounds__(256)
k_plain_phase(float2 *__restrict__ a, uint64_t count, int q, float cr, float ci) {
    const uint64_t stride = uint64_t(gridDim.x) * blockDim.x;
    for (uint64_t i = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < count; i += stride) {
        const uint64_t k = insert_zero(i, q) | (1ull << q);
        a[k] = cmul(a[k], cr, ci);
    }
}

// Negate amplitudes with bits q0 and q1 set (q0 < q1): a quarter of the state.
__global__ void __launch_bounds__(256)
k_plain_cz(float2 *__restrict__ a, uint64_t count, int q0, int q1) {
    const uint64_t stride = uint64_t(gridDim.x) * blockDim.x;
    for (uint64_t i = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < count; i += stride) {
        const uint64_t k = insert_zero(insert_zero(i, q0), q1) | (1ull << q0) | (1ull << q1);
        const float2 x = a[k];
        a[k] = f2(-x.x, -x.y);
    }
}

// Zero amplitudes whose bit q is != l (projector P_l): write-only, half the state.
__global__ void __launch_bounds__(256)
k_plain_zero(float2 *__restrict__ a, uint64_t count, int q, int l) {
    const uint64_t stride = uint64_t(gridDim.x) * blockDim.x;
    for (uint64_t i = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < count; i += stride) {
        const uint64_t k = insert_zero(i, q) | (uint64_t(1 - l) << q);
        a[k] = f2(0.f, 0.f);
    }
}

// ---------------------------------------------------------------------------
// Initialisation, gather, norm, branch combine.
// ---------------------------------------------------------------------------

__global__ void __launch_bounds__(256)
k_init(v4f *__restrict__ a, uint64_t quads, float val, int kind, uint64_t basis) {
    const uint64_t stride = uint64_t(gridDim.x) * blockDim.x;
    for (uint64_t i = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < quads; i += stride) {
        v4f w;
        if (kind == 1) {
            w = v4f{val, 0.f, val, 0.f};
        } else {
            w = v4f{0.f, 0.f, 0.f, 0.f};
            if ((basis >> 1) == i) {
                if (basis & 1) w.z = 1.f; else w.x = 1.f;
            }
        }
        __builtin_nontemporal_store(w, a + i);
    }
}

__global__ void __launch_bounds__(256)
k_init_small(float2 *__restrict__ a, uint64_t dim, float val, int kind, uint64_t basis) {
    const uint64_t i = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i >= dim) return;
    if (kind == 1) a[i] = f2(val, 0.f);
    else a[i] = f2(i == basis ? 1.f : 0.f, 0.f);
}

// out[k] = amplitude of bitstring xs[k] (NaN beyond the state)
__device__ __forceinline__ void gather_one(const float2 *a, uint64_t dim, const uint64_t *xs, uint64_t m, void *out,
                                           int c128, uint64_t k) {
    if (k >= m) return;
    const uint64_t x = xs[k];
    float2 v;
    if (x < dim) v = a[x];
    else v = f2(__builtin_nanf(""), __builtin_nanf(""));
    if (c128) reinterpret_cast<double2 *>(out)[k] = make_double2(double(v.x), double(v.y));
    else reinterpret_cast<float2 *>(out)[k] = v;
}

__global__ void __launch_bounds__(256)
k_gather(const float2 *__restrict__ a, uint64_t dim, const uint64_t *__restrict__ xs, uint64_t m,
         void *__restrict__ out, int c128) {
    gather_one(a, dim, xs, m, out, c128, uint64_t(blockIdx.x) * blockDim.x + threadIdx.x);
}

// Range check of device bitstrings: raises *flag (mapped host memory) when
// some xs[k] >= dim.  Grid-stride; the flag is only ever set, never read here.
__global__ void __launch_bounds__(256)
k_check_range(const uint64_t *__restrict__ xs, uint64_t m, uint64_t dim, unsigned int *flag) {
    const uint64_t stride = uint64_t(gridDim.x) * blockDim.x;
    bool bad = false;
    for (uint64_t k = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x; k < m; k += stride) bad = bad || xs[k] >= dim;
    if (bad) __hip_atomic_fetch_or(flag, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

__global__ void __launch_bounds__(256)
k_gather_c128(const double2 *__restrict__ a, uint64_t dim, const uint64_t *__restrict__ xs,
              uint64_t m, double2 *__restrict__ out) {
    const uint64_t k = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (k >= m) return;
    const uint64_t x = xs[k];
    out[k] = (x < dim) ? a[x] : make_double2(__builtin_nan(""), __builtin_nan(""));
}

// Block b sums |a_i|^2 over its contiguous chunk in FP64 (products of FP32
// values are exact in FP64); fixed thread-then-tree order.  The read of the
// state bounds it: four nontemporal 16-byte loads in flight per thread and
// 2^13 blocks (the two states of k_dot_partial, 29 qubits: 7.1 TB/s, against
// 6.2 with one ordinary load at a time; 2^16 blocks are as fast, but their
// partials take one workgroup 13 us to add).  No sum is longer for that than with
// 2^16 blocks and a single sum per thread: 29 qubits, 16 additions in a row.
// Random states of norm 1, 28 qubits, 12 seeds, rms error: inner product 3.7e-17
// (4.1e-17 with 2^16 blocks), norm 7.9e-17 (9.8e-17).
__global__ void __launch_bounds__(256)
k_norm_partial(const v4f *__restrict__ a, uint64_t quads_per_block, double *__restrict__ part) {
    __shared__ double s[256];
    const uint64_t start = uint64_t(blockIdx.x) * quads_per_block;
    constexpr int U = 4;
    double acc = 0.0, other = 0.0;  // the loads of a round are added up first, rounds go to the two in turn
    for (uint64_t i = threadIdx.x; i < quads_per_block; i += 256 * U) {
        v4f w[U];
        double q[U];
#pragma unroll
        for (int u = 0; u < U; ++u) w[u] = __builtin_nontemporal_load(a + start + i + u * 256);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const double x0 = w[u].x, y0 = w[u].y, x1 = w[u].z, y1 = w[u].w;
            q[u] = (x0 * x0 + y0 * y0) + (x1 * x1 + y1 * y1);
        }
        const double sum = other + ((q[0] + q[1]) + (q[2] + q[3]));
        other = acc;
        acc = sum;
    }
    s[threadIdx.x] = acc + other;
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
        if (int(threadIdx.x) < h) s[threadIdx.x] += s[threadIdx.x + h];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = s[0];
}

// Sum of count partials by one block of 1024 threads: each thread keeps
// eight independent accumulators over a fixed strided subset, then a fixed
// tree over the threads.
__device__ __forceinline__ void sum_partials(const double *part, uint64_t count, double *out) {
    __shared__ double s[1024];
    double acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    uint64_t i = threadIdx.x;
    for (; i + 7 * 1024 < count; i += 8 * 1024) {
#pragma unroll
        for (int k = 0; k < 8; ++k) acc[k] += part[i + k * 1024];
    }
    for (int k = 0; i < count; i += 1024, ++k) acc[k & 7] += part[i];
    s[threadIdx.x] = ((acc[0] + acc[1]) + (acc[2] + acc[3])) + ((acc[4] + acc[5]) + (acc[6] + acc[7]));
    __syncthreads();
    for (int h = 512; h > 0; h >>= 1) {
        if (int(threadIdx.x) < h) s[threadIdx.x] += s[threadIdx.x + h];
        __syncthreads();
    }
    if (threadIdx.x == 0) *out = s[0];
}

// Block b sums the b-th run of count partials.
__global__ void __launch_bounds__(1024)
k_sum_partials(const double *__restrict__ part, uint64_t count, double *__restrict__ out) {
    sum_partials(part + blockIdx.x * count, count, out + blockIdx.x);
}

// What ends a simulation, in one launch: block 0 sums the norm's partials, the
// others gather the amplitudes.
__global__ void __launch_bounds__(1024)
k_finish(const double *__restrict__ part, uint64_t count, double *__restrict__ norm, const float2 *__restrict__ a,
         uint64_t dim, const uint64_t *__restrict__ xs, uint64_t m, void *__restrict__ out, int c128) {
    if (blockIdx.x == 0) sum_partials(part, count, norm);
    else gather_one(a, dim, xs, m, out, c128, uint64_t(blockIdx.x - 1) * 1024 + threadIdx.x);
}

// <a|b> = sum conj(a_i) b_i with FP64 products of the FP32 inputs (exact),
// same fixed-order tree as the norm: per-block partials (re at part[blk],
// im at part[nblk + blk]), then k_sum_partials on each half.
__global__ void __launch_bounds__(256)
k_dot_partial(const v4f *__restrict__ a, const v4f *__restrict__ b, uint64_t quads_per_block,
              double *__restrict__ part) {
    __shared__ double sr[256], si[256];
    const uint64_t start = uint64_t(blockIdx.x) * quads_per_block;
    constexpr int U = 4;  // 16-byte loads in flight per state
    double ar = 0.0, ai = 0.0, br = 0.0, bi = 0.0;  // two sums in turn, as in k_norm_partial
    for (uint64_t i = threadIdx.x; i < quads_per_block; i += 256 * U) {
        v4f x[U], y[U];
        double qr[U], qi[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            x[u] = __builtin_nontemporal_load(a + start + i + u * 256);
            y[u] = __builtin_nontemporal_load(b + start + i + u * 256);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const double x0 = x[u].x, x1 = x[u].y, x2 = x[u].z, x3 = x[u].w;
            const double y0 = y[u].x, y1 = y[u].y, y2 = y[u].z, y3 = y[u].w;
            qr[u] = (x0 * y0 + x1 * y1) + (x2 * y2 + x3 * y3);
            qi[u] = (x0 * y1 - x1 * y0) + (x2 * y3 - x3 * y2);
        }
        const double r = br + ((qr[0] + qr[1]) + (qr[2] + qr[3])), m = bi + ((qi[0] + qi[1]) + (qi[2] + qi[3]));
        br = ar;
        bi = ai;
        ar = r;
        ai = m;
    }
    sr[threadIdx.x] = ar + br;
    si[threadIdx.x] = ai + bi;
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
        if (int(threadIdx.x) < h) {
            sr[threadIdx.x] += sr[threadIdx.x + h];
            si[threadIdx.x] += si[threadIdx.x + h];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        part[blockIdx.x] = sr[0];
        part[gridDim.x + blockIdx.x] = si[0];
    }
}

__global__ void __launch_bounds__(256)
k_dot_small(const float2 *__restrict__ a, const float2 *__restrict__ b, uint64_t dim,
            double *__restrict__ out) {
    __shared__ double sr[256], si[256];
    double ar = 0.0, ai = 0.0;
    for (uint64_t i = threadIdx.x; i < dim; i += 256) {
        const double x0 = a[i].x, x1 = a[i].y, y0 = b[i].x, y1 = b[i].y;
        ar += x0 * y0 + x1 * y1;
        ai += x0 * y1 - x1 * y0;
    }
    sr[threadIdx.x] = ar;
    si[threadIdx.x] = ai;
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
        if (int(threadIdx.x) < h) {
            sr[threadIdx.x] += sr[threadIdx.x + h];
            si[threadIdx.x] += si[threadIdx.x + h];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        out[0] = sr[0];
        out[1] = si[0];
    }
}

__global__ void __launch_bounds__(256)
k_norm_small(const float2 *__restrict__ a, uint64_t dim, double *__restrict__ out) {
    __shared__ double s[256];
    double acc = 0.0;
    for (uint64_t i = threadIdx.x; i < dim; i += 256) {
        const double x = a[i].x, y = a[i].y;
        acc += x * x + y * y;
    }
    s[threadIdx.x] = acc;
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
        if (int(threadIdx.x) < h) s[threadIdx.x] += s[threadIdx.x + h];
        __syncthreads();
    }
    if (threadIdx.x == 0) *out = s[0];
}

// out[x] = sign[x] * sum_b A[b][x] * B[b][x]; FP64 products and sums, fixed
// order.  Both tables are read once, so the read is the bound (33.6 MB for
// 2048 branches of 1024 outputs); what it needs is loads in flight on every
// CU.  A workgroup sums 2^lc columns; its threads split the branches (thread
// t: column t mod 2^lc, branches t >> lc, + rows, ...), lanes of one column
// add up across the wave, the waves through LDS.  Groups of neighbouring
// columns go to one XCD (workgroups are dealt to the 8 XCDs in turn), so that
// the workgroups that share a cache line share an L2.  With 64 columns and
// four branch groups per workgroup, 16 workgroups in all, the table above
// took 173 us; with 4 columns and 256 branch groups 10.7 us
// with new tables each call (4096 x 4096 pairs: 38 us, 7.0 TB/s).
__global__ void __launch_bounds__(1024)
k_branch_combine(const float2 *__restrict__ A, const float2 *__restrict__ B, uint64_t nb,
                 uint64_t m, const int8_t *__restrict__ sign, double2 *__restrict__ out, int lc) {
    __shared__ double sr[1024], si[1024];  // [wave][column]
    const uint32_t t = threadIdx.x, cols = 1u << lc, col = t & (cols - 1u);
    const uint64_t rows = blockDim.x >> lc;
    const uint32_t g = gridDim.x, blk = blockIdx.x;
    const uint64_t group = (g % 8u == 0) ? uint64_t(blk % 8u) * (g / 8u) + blk / 8u : blk;
    const uint64_t x = (group << lc) + col;
    constexpr int U = 4;
    double ar = 0.0, ai = 0.0;
    if (x < m) {
        for (uint64_t b0 = t >> lc; b0 < nb; b0 += U * rows) {
            float2 p[U], q[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint64_t b = b0 + u * rows;
                p[u] = q[u] = f2(0.f, 0.f);
                if (b < nb) {
                    p[u] = A[b * m + x];
                    q[u] = B[b * m + x];
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (b0 + u * rows >= nb) break;
                const double pr = p[u].x, pi = p[u].y, qr = q[u].x, qi = q[u].y;
                ar += pr * qr - pi * qi;
                ai += pr * qi + pi * qr;
            }
        }
    }
    for (uint32_t off = 32; off >= cols; off >>= 1) {
        ar += __shfl_xor(ar, int(off), 64);
        ai += __shfl_xor(ai, int(off), 64);
    }
    // per wave one sum of each of its columns (a wave holds cols <= 64 of them)
    const uint32_t wave = t >> 6, lane = t & 63u;
    if (lane < cols) {
        sr[(wave << lc) + lane] = ar;
        si[(wave << lc) + lane] = ai;
    }
    __syncthreads();
    if (t < cols && x < m) {
        double r = 0.0, i = 0.0;
        for (uint32_t w = 0; w < blockDim.x >> 6; ++w) {
            r += sr[(w << lc) + t];
            i += si[(w << lc) + t];
        }
        if (sign && sign[x] < 0) { r = -r; i = -i; }
        out[x] = make_double2(r, i);
    }
}

// Streaming copy with the sweep's access pattern (16-byte nontemporal loads
// and stores, 8 in flight per thread): the HBM rate a pass that does no
// arithmetic would reach, the ceiling the fused passes are compared with.
__global__ void __launch_bounds__(256)
k_stream_copy(const v4f *__restrict__ src, v4f *__restrict__ dst, uint64_t count) {
    constexpr int U = 8;
    const uint64_t stride = uint64_t(gridDim.x) * 256u * U;
    for (uint64_t base = uint64_t(blockIdx.x) * 256u * U + threadIdx.x; base < count; base += stride) {
        v4f w[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint64_t i = base + uint64_t(u) * 256u;
            if (i < count) w[u] = __builtin_nontemporal_load(src + i);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint64_t i = base + uint64_t(u) * 256u;
            if (i < count) __builtin_nontemporal_store(w[u], dst + i);
        }
    }
}

unsigned grid_for(uint64_t work, unsigned per_block = 256, unsigned cap = 1u << 20) {
    uint64_t g = (work + per_block - 1) / per_block;
    if (g < 1) g = 1;
    if (g > cap) g = cap;
    return unsigned(g);
}

}  // namespace

hipError_t launch_gather_batch(const BatchEntry *ents, uint64_t count, const uint64_t *xs,
                               uint64_t m, float2 *out, hipStream_t s) {
    if (count * m == 0) return hipSuccess;
    hipLaunchKernelGGL(k_gather_batch, dim3(unsigned((count * m + 255) / 256)), dim3(256), 0, s,
                       ents, count, xs, m, out);
    return hipGetLastError();
}

hipError_t launch_dense(float2 *amps, int n, int k, const int *qubits, const float *mat_t,
                        hipStream_t s) {
    switch (k) {
    case 4: return launch_dense_t<4>(amps, n, qubits, mat_t, s);
    case 5: return launch_dense_t<5>(amps, n, qubits, mat_t, s);
    case 6: return launch_dense_t<6>(amps, n, qubits, mat_t, s);
    case 7: return launch_dense_t<7>(amps, n, qubits, mat_t, s);
    default: return hipErrorInvalidValue;
    }
}

bool fused_shape_supported(int R, int T) {
    switch (R * 16 + T) {
    case 5 * 16 + 8: case 5 * 16 + 7: case 4 * 16 + 7: case 4 * 16 + 6: case 3 * 16 + 6:
    case 3 * 16 + 4: case 2 * 16 + 3: case 4 * 16 + 8: case 6 * 16 + 8: case 5 * 16 + 9:
    case 4 * 16 + 9: case 6 * 16 + 7:
        return true;
    default:
        return false;
    }
}

bool compiled_shape_supported(int R, int T) { return fused_shape_supported(R, T) || (R == 6 && T == 9); }

hipError_t launch_plain_1q(float2 *amps, int n, int q, const float m[8], hipStream_t s) {
    const uint64_t pairs = 1ull << (n - 1);
    hipLaunchKernelGGL(k_plain_1q, dim3(grid_for(pairs)), dim3(256), 0, s, amps, pairs, q, m[0],
                       m[1], m[2], m[3], m[4], m[5], m[6], m[7]);
    return hipGetLastError();
}

hipError_t launch_plain_phase(float2 *amps, int n, int q, float cr, float ci, hipStream_t s) {
    const uint64_t cnt = 1ull << (n - 1);
    hipLaunchKernelGGL(k_plain_phase, dim3(grid_for(cnt)), dim3(256), 0, s, amps, cnt, q, cr, ci);
    return hipGetLastError();
}

hipError_t launch_plain_cz(float2 *amps, int n, int q0, int q1, hipStream_t s) {
    if (q0 > q1) { int t = q0; q0 = q1; q1 = t; }
    const uint64_t cnt = 1ull << (n - 2);
    hipLaunchKernelGGL(k_plain_cz, dim3(grid_for(cnt)), dim3(256), 0, s, amps, cnt, q0, q1);
    return hipGetLastError();
}

hipError_t launch_plain_zero(float2 *amps, int n, int q, int l, hipStream_t s) {
    const uint64_t cnt = 1ull << (n - 1);
    hipLaunchKernelGGL(k_plain_zero, dim3(grid_for(cnt)), dim3(256), 0, s, amps, cnt, q, l);
    return hipGetLastError();
}

hipError_t launch_init(float2 *amps, int n, int kind, uint64_t basis, hipStream_t s) {
    const uint64_t dim = 1ull << n;
    const float val = float(1.0 / __builtin_sqrt(double(dim)));
    if (n >= 1) {
        const uint64_t quads = dim / 2;
        hipLaunchKernelGGL(k_init, dim3(grid_for(quads)), dim3(256), 0, s,
                           reinterpret_cast<v4f *>(amps), quads, val, kind, basis);
    } else {
        hipLaunchKernelGGL(k_init_small, dim3(1), dim3(256), 0, s, amps, dim, val, kind, basis);
    }
    return hipGetLastError();
}

hipError_t launch_gather(const float2 *amps, int n, const uint64_t *xs, uint64_t m, void *out,
                         int c128, hipStream_t s) {
    if (m == 0) return hipSuccess;
    hipLaunchKernelGGL(k_gather, dim3(grid_for(m, 256, 1u << 30)), dim3(256), 0, s, amps,
                       1ull << n, xs, m, out, c128);
    return hipGetLastError();
}

hipError_t launch_check_range(const uint64_t *xs, uint64_t m, int n, unsigned int *flag, hipStream_t s) {
    if (m == 0) return hipSuccess;
    hipLaunchKernelGGL(k_check_range, dim3(grid_for(m, 256, 1024)), dim3(256), 0, s, xs, m, 1ull << n, flag);
    return hipGetLastError();
}

hipError_t launch_gather_c128(const void *amps, int n, const uint64_t *xs, uint64_t m, void *out,
                              hipStream_t s) {
    if (m == 0) return hipSuccess;
    hipLaunchKernelGGL(k_gather_c128, dim3(grid_for(m, 256, 1u << 30)), dim3(256), 0, s,
                       static_cast<const double2 *>(amps), 1ull << n, xs, m, static_cast<double2 *>(out));
    return hipGetLastError();
}

size_t norm_partial_count(int n) {
    if (n < 14) return 0;
    // log2(blocks) so that each block has 1024 quads, at most 8192 blocks
    const int lb = n - 1 - 10 > 13 ? 13 : n - 1 - 10;
    return size_t(1) << lb;
}

hipError_t launch_norm(const float2 *amps, int n, double *out, double *partials, hipStream_t s) {
    const uint64_t dim = 1ull << n;
    if (n < 14) {
        hipLaunchKernelGGL(k_norm_small, dim3(1), dim3(256), 0, s, amps, dim, out);
        return hipGetLastError();
    }
    // each block a contiguous chunk of >= 1024 quads
    const unsigned blocks = unsigned(norm_partial_count(n));
    const int lb = __builtin_ctz(blocks);
    const uint64_t qpb = (dim / 2) >> lb;
    hipLaunchKernelGGL(k_norm_partial, dim3(blocks), dim3(256), 0, s,
                       reinterpret_cast<const v4f *>(amps), qpb, partials);
    hipLaunchKernelGGL(k_sum_partials, dim3(1), dim3(1024), 0, s, partials, uint64_t(blocks), out);
    return hipGetLastError();
}

hipError_t launch_dot(const float2 *a, const float2 *b, int n, double *out, double *partials,
                      hipStream_t s) {
    const uint64_t dim = 1ull << n;
    if (n < 14) {
        hipLaunchKernelGGL(k_dot_small, dim3(1), dim3(256), 0, s, a, b, dim, out);
        return hipGetLastError();
    }
    const unsigned blocks = unsigned(norm_partial_count(n));
    const uint64_t qpb = (dim / 2) / blocks;
    hipLaunchKernelGGL(k_dot_partial, dim3(blocks), dim3(256), 0, s, reinterpret_cast<const v4f *>(a),
                       reinterpret_cast<const v4f *>(b), qpb, partials);
    hipLaunchKernelGGL(k_sum_partials, dim3(2), dim3(1024), 0, s, partials, uint64_t(blocks), out);
    return hipGetLastError();
}

hipError_t launch_stream_copy(const void *src, void *dst, uint64_t bytes, hipStream_t s) {
    const uint64_t count = bytes / 16;
    if (count == 0) return hipSuccess;
    // 8 workgroups of 256 threads per CU on 256 CUs, each thread 8 x 16 B in flight
    const uint64_t per_block = 256u * 8u;
    uint64_t grid = (count + per_block - 1) / per_block;
    if (grid > 2048) grid = 2048;
    hipLaunchKernelGGL(k_stream_copy, dim3(unsigned(grid)), dim3(256), 0, s, static_cast<const v4f *>(src),
                       static_cast<v4f *>(dst), count);
    return hipGetLastError();
}

hipError_t launch_sum_partials(const double *part, uint64_t count, double *out, hipStream_t s) {
    hipLaunchKernelGGL(k_sum_partials, dim3(1), dim3(1024), 0, s, part, count, out);
    return hipGetLastError();
}

hipError_t launch_finish(const double *part, uint64_t count, double *norm, const float2 *amps, int n,
                         const uint64_t *xs, uint64_t m, void *out, int c128, hipStream_t s) {
    if (m > (1ull << 30)) {
        const hipError_t e = launch_sum_partials(part, count, norm, s);
        return e == hipSuccess ? launch_gather(amps, n, xs, m, out, c128, s) : e;
    }
    hipLaunchKernelGGL(k_finish, dim3(1 + unsigned((m + 1023) / 1024)), dim3(1024), 0, s, part, count, norm, amps,
                       1ull << n, xs, m, out, c128);
    return hipGetLastError();
}

hipError_t launch_branch_combine(const float2 *A, const float2 *B, uint64_t nb, uint64_t m,
                                 const int8_t *sign, double2 *out, hipStream_t s) {
    if (m == 0) return hipSuccess;
    // fewer columns per workgroup until there is a workgroup per CU, as long
    // as the branches give the freed threads something to add
    int lc = 6;
    while (lc > 0 && ((m + (1ull << lc) - 1) >> lc) < 256 && (1024u >> lc) < nb) --lc;
    unsigned threads = 64;
    while (threads < 1024 && (threads >> lc) < nb) threads *= 2;
    hipLaunchKernelGGL(k_branch_combine, dim3(unsigned((m + (1ull << lc) - 1) >> lc)), dim3(threads), 0, s, A, B, nb,
                       m, sign, out, lc);
    return hipGetLastError();
}

}  // namespace qsv
