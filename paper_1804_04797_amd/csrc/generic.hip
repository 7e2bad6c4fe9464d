// Generic fused tile pass for gfx950: interprets a lowered pass program.
//
// One workgroup of 2^T threads owns one tile of 2^(R+T) amplitudes: slot
// coordinate x = j | t << R (j = register index, t = thread index) sits at
// physical index origin | sum_{s: x_s = 1} 2^{phys[s]}.  Loads and stores are
// 16-byte (register slot 0 is physical bit 0) and the thread slots 0..c-2 hold
// physical bits 1..c-1, so a wave access is made of runs of 2^c amplitudes.
//
// States of this path are small (below 2^24 amplitudes unless asked for): the
// caches hold them and a pass is bound by the instructions it issues, so the
// program has as few and as cheap ops as possible.  Diagonal gates are folded
// into the operands of the Hadamards after them; two Hadamards on different
// register slots are one op (four amplitudes in, four out); an exchange takes
// its addresses from the op.  The ops update the amplitude registers in place
// through asm: as plain C++ every case of the switch defines the whole array
// anew and the compiler joins the cases with 2^(R+1) copies (the file is also
// compiled with uniform regions left unstructurized, for the same reason).
// Before, every gate of the pass program was an op of its own: a 16-qubit
// sweep of 95 gates took 77 us, now 26 (tile (4, 8, 4)); the 20-qubit depth-10
// simulation 131, now 70, the 23-qubit depth-14 one 375, now 152 (both on
// (5, 8, 5), in gate order, with what run_tile and stage_halves say below).
#include <hip/hip_runtime.h>

#include <cstdint>

#include "genprog.h"
#include "kernels.h"

namespace qsv {
namespace {

typedef float v4f __attribute__((ext_vector_type(4)));

// x, y <- x + c y, x - c y
__device__ __forceinline__ void bf2(float &x, float &y, float c) {
    float t;
    asm("v_fma_f32 %2, %3, %1, %0\n\t"
        "v_fma_f32 %1, -%3, %1, %0\n\t"
        "v_mov_b32 %0, %2"
        : "+v"(x), "+v"(y), "=&v"(t)
        : "v"(c));
}
// the same on the slot of (a0, a1) with c, then on the slot of (a0, b0) with d
__device__ __forceinline__ void bf4(float &a0, float &a1, float &b0, float &b1, float c, float d) {
    float t0, t1, t2, t3;
    asm("v_fma_f32 %4, %8, %1, %0\n\t"
        "v_fma_f32 %5, -%8, %1, %0\n\t"
        "v_fma_f32 %6, %8, %3, %2\n\t"
        "v_fma_f32 %7, -%8, %3, %2\n\t"
        "v_fma_f32 %0, %9, %6, %4\n\t"
        "v_fma_f32 %2, -%9, %6, %4\n\t"
        "v_fma_f32 %1, %9, %7, %5\n\t"
        "v_fma_f32 %3, -%9, %7, %5"
        : "+v"(a0), "+v"(a1), "+v"(b0), "+v"(b1), "=&v"(t0), "=&v"(t1), "=&v"(t2), "=&v"(t3)
        : "v"(c), "v"(d));
}
// x, y <- x - i c y, c y - i x on the components (x.re, y.im) and (x.im, y.re)
__device__ __forceinline__ void bf_i(float &xr, float &xi, float &yr, float &yi, float c) {
    float t, u;
    asm("v_fma_f32 %4, %6, %3, %0\n\t"
        "v_fma_f32 %3, %6, %3, -%0\n\t"
        "v_fma_f32 %5, -%6, %2, %1\n\t"
        "v_fma_f32 %2, %6, %2, %1\n\t"
        "v_mov_b32 %0, %4\n\t"
        "v_mov_b32 %1, %5"
        : "+v"(xr), "+v"(xi), "+v"(yr), "+v"(yi), "=&v"(t), "=&v"(u)
        : "v"(c));
}
// (re, im) <- (cr + i ci) (re, im); the products with ci are rounded first
__device__ __forceinline__ void cmul(float &re, float &im, float cr, float ci) {
    float t, u;
    asm("v_mul_f32 %2, %5, %1\n\t"
        "v_mul_f32 %3, %5, %0\n\t"
        "v_fma_f32 %0, %0, %4, -%2\n\t"
        "v_fma_f32 %1, %1, %4, %3"
        : "+v"(re), "+v"(im), "=&v"(t), "=&v"(u)
        : "v"(cr), "v"(ci));
}
// the same for the closing scale: im rounds the product with cr first
__device__ __forceinline__ void cmul_scale(float &re, float &im, float cr, float ci) {
    float t, u;
    asm("v_mul_f32 %2, %5, %1\n\t"
        "v_mul_f32 %3, %4, %1\n\t"
        "v_fma_f32 %1, %0, %5, %3\n\t"
        "v_fma_f32 %0, %0, %4, -%2"
        : "+v"(re), "+v"(im), "=&v"(t), "=&v"(u)
        : "v"(cr), "v"(ci));
}
// (re, im) <- (1 + i) (re, im)
__device__ __forceinline__ void mul_1pi(float &re, float &im) {
    float t;
    asm("v_sub_f32 %2, %0, %1\n\t"
        "v_add_f32 %1, %0, %1\n\t"
        "v_mov_b32 %0, %2"
        : "+v"(re), "+v"(im), "=&v"(t));
}
// (re, im) <- i (re, im)
__device__ __forceinline__ void mul_i(float &re, float &im) {
    asm("v_swap_b32 %0, %1\n\t"
        "v_xor_b32 %0, 0x80000000, %0"
        : "+v"(re), "+v"(im));
}
__device__ __forceinline__ void flip(float &x, uint32_t m) { asm("v_xor_b32 %0, %1, %0" : "+v"(x) : "s"(m)); }
__device__ __forceinline__ void keep(float &x, uint32_t m) { asm("v_and_b32 %0, %1, %0" : "+v"(x) : "v"(m)); }
__device__ __forceinline__ void scale(float &x, float c) { asm("v_mul_f32 %0, %1, %0" : "+v"(x) : "v"(c)); }

// The amplitudes of one thread: register j is (re[j], im[j]).
template <int R> struct Amps {
    static constexpr int N = 1 << R;
    float re[N], im[N];

    // the pending diagonal of an operand on slot S: i^a (1 + i)^b and the
    // signs K of the registers with the slot's bit set
    template <int S> __device__ __forceinline__ void diagonal(uint32_t f, uint32_t K) {
        if (f & 8u) {
#pragma unroll
            for (int j = 0; j < N; ++j)
                if (j & (1 << S)) mul_1pi(re[j], im[j]);
        }
        if (f & 16u) {
#pragma unroll
            for (int j = 0; j < N; ++j)
                if (j & (1 << S)) mul_i(re[j], im[j]);
        }
        if (f & 64u) {
#pragma unroll
            for (int j = 0, i = 0; j < N; ++j) {
                if (!(j & (1 << S))) continue;
                const uint32_t m = (K << (31 - i)) & 0x80000000u;
                flip(re[j], m);
                flip(im[j], m);
                ++i;
            }
        }
    }
    __device__ __forceinline__ void diagonal(uint32_t f, uint32_t K) {
        switch (f & 7u) {
        case 0: diagonal<0>(f, K); break;
        case 1: if constexpr (R > 1) diagonal<1>(f, K); break;
        case 2: if constexpr (R > 2) diagonal<2>(f, K); break;
        case 3: if constexpr (R > 3) diagonal<3>(f, K); break;
        case 4: if constexpr (R > 4) diagonal<4>(f, K); break;
        default: if constexpr (R > 5) diagonal<5>(f, K); break;
        }
    }
    template <int S> __device__ __forceinline__ void h1(float c) {
        if constexpr (S < R) {
#pragma unroll
            for (int j = 0; j < N; ++j) {
                if (j & (1 << S)) continue;
                bf2(re[j], re[j | (1 << S)], c);
                bf2(im[j], im[j | (1 << S)], c);
            }
        }
    }
    template <int A, int B> __device__ __forceinline__ void h2(float c, float d) {
        if constexpr (B < R) {
#pragma unroll
            for (int j = 0; j < N; ++j) {
                if (j & ((1 << A) | (1 << B))) continue;
                bf4(re[j], re[j | (1 << A)], re[j | (1 << B)], re[j | (1 << A) | (1 << B)], c, d);
                bf4(im[j], im[j | (1 << A)], im[j | (1 << B)], im[j | (1 << A) | (1 << B)], c, d);
            }
        }
    }
    // the other order: the slot B of GEN_H2 first
    template <int A, int B> __device__ __forceinline__ void h2r(float c, float d) {
        if constexpr (B < R) {
#pragma unroll
            for (int j = 0; j < N; ++j) {
                if (j & ((1 << A) | (1 << B))) continue;
                bf4(re[j], re[j | (1 << B)], re[j | (1 << A)], re[j | (1 << A) | (1 << B)], d, c);
                bf4(im[j], im[j | (1 << B)], im[j | (1 << A)], im[j | (1 << A) | (1 << B)], d, c);
            }
        }
    }
    template <int S> __device__ __forceinline__ void hi(float c) {
        if constexpr (S < R) {
#pragma unroll
            for (int j = 0; j < N; ++j) {
                if (j & (1 << S)) continue;
                bf_i(re[j], im[j], re[j | (1 << S)], im[j | (1 << S)], c);
            }
        }
    }
    template <int S> __device__ __forceinline__ void t_gate(float ci) {
        if constexpr (S < R) {
#pragma unroll
            for (int j = 0; j < N; ++j)
                if (j & (1 << S)) cmul(re[j], im[j], 0.70710678118654752f, ci);
        }
    }
    __device__ __forceinline__ void all(float cr, float ci) {
#pragma unroll
        for (int j = 0; j < N; ++j) cmul(re[j], im[j], cr, ci);
    }
    template <int S> __device__ __forceinline__ void ph(float c) {
        if constexpr (S < R) {
#pragma unroll
            for (int j = 0; j < N; ++j) {
                if (!(j & (1 << S))) continue;
                scale(re[j], c);
                scale(im[j], c);
            }
        }
    }
    template <int S> __device__ __forceinline__ void proj(uint32_t l) {
        if constexpr (S < R) {
#pragma unroll
            for (int j = 0; j < N; ++j) {
                const uint32_t m = uint32_t((j >> S) & 1) == l ? ~0u : 0u;
                keep(re[j], m);
                keep(im[j], m);
            }
        }
    }
    // v_permlane16/32_swap exchange a register bit with lane bit 4 / 5
    template <int S, int LANE> __device__ __forceinline__ void lane_swap() {
        if constexpr (S < R) {
#pragma unroll
            for (int j = 0; j < N; ++j) {
                if (j & (1 << S)) continue;
                const int k = j | (1 << S);
                auto sw = [](float &x, float &y) {
                    const auto r = LANE == 4 ? __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(y), false, false)
                                             : __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false);
                    x = __uint_as_float(r[0]);
                    y = __uint_as_float(r[1]);
                };
                sw(re[j], re[k]);
                sw(im[j], im[k]);
            }
        }
    }
};

struct TileArgs {
    const float2 *src;  // the state to load (amps, or another one that stays as it is)
    float2 *amps;
    uint64_t branch, tile, basis;
    int init;  // -1: load the tile; 0 / 2: |basis>; 1: every amplitude init_val
    float init_val;
    double *norm;  // null, or the tiles' sums of |amp|^2
};

// e^{i pi k / 4}
__device__ __forceinline__ float2 omega(uint32_t k) {
    const float h = 0.70710678118654752f;
    float x = (k & 1u) ? h : 1.f, y = (k & 1u) ? h : 0.f;  // k = 0, 1
    if (k & 2u) { const float t = x; x = -y; y = t; }
    if (k & 4u) { x = -x; y = -y; }
    return make_float2(x, y);
}

// HALF: exchanges stage the real parts, then the imaginary parts: half the
// buffer, so twice the workgroups on a CU, for twice the barriers.
template <int R, int T, bool HALF>
__device__ __forceinline__ void run_tile(const GenProg &P, const TileArgs &A, float *lds) {
    constexpr int N = 1 << R;
    constexpr GenWeights W = gen_weights(R, T);
    const uint32_t t = threadIdx.x;
    const uint32_t tile = uint32_t(A.tile);

    uint64_t origin = 0;
    for (uint32_t r = 0; r < P.n_runs; ++r) {
        const uint32_t x = P.run[r];
        origin |= uint64_t((tile >> (x & 0xffu)) & ((1u << ((x >> 8) & 0xffu)) - 1u)) << (x >> 16);
    }
    auto thread_offset = [&](const uint32_t *phys) {
        uint64_t o = origin;
#pragma unroll
        for (int u = 0; u < T; ++u)
            o |= uint64_t((t >> u) & 1u) << gen_phys(phys, R + u);
        return o;
    };
    auto reg_offset = [&](const uint32_t *phys, int j) {
        uint64_t o = 0;
#pragma unroll
        for (int s = 1; s < R; ++s)
            if ((j >> s) & 1) o |= 1ull << gen_phys(phys, s);
        return o;
    };

    Amps<R> v;
    if (A.init < 0) {
        const float2 *src = A.src + thread_offset(P.ld_phys);
#pragma unroll
        for (int j = 0; j < N; j += 2) {
            const v4f w = *reinterpret_cast<const v4f *>(src + reg_offset(P.ld_phys, j));
            v.re[j] = w.x;
            v.im[j] = w.y;
            v.re[j + 1] = w.z;
            v.im[j + 1] = w.w;
        }
    } else {
        const uint64_t me = A.init == 1 ? 0 : thread_offset(P.ld_phys);
#pragma unroll
        for (int j = 0; j < N; ++j) {
            const uint64_t x = me | reg_offset(P.ld_phys, j) | uint64_t(j & 1);
            v.re[j] = A.init == 1 ? A.init_val : (x == A.basis ? 1.f : 0.f);
            v.im[j] = 0.f;
        }
    }

    uint32_t wt = 0;  // exchange buffer: this thread's first element
#pragma unroll
    for (int u = 0; u < T; ++u) wt += ((t >> u) & 1u) * W.w[R + u];
    uint32_t e = 0;

    auto parity = [](uint32_t x) { return uint32_t(__popc(x)) & 1u; };
    // coefficient of an operand: the sign from the thread and tile partners
    auto coef = [&](uint32_t bits, uint32_t tm, uint32_t gm) {
        const uint32_t uni = bits ^ (uint32_t(__popc(gm & tile)) << 31);
        return __uint_as_float(uni ^ (uint32_t(__popc(tm & t)) << 31));
    };
    uint32_t extra = 0;  // sign bit for the next op (GEN_ZB)
    GenOp nx = P.ops[0];
    for (uint32_t pc = 0;; ++pc) {
        const GenOp op = nx;
        const uint32_t code = op.w[0] & 0xffu;
        if (code == GEN_END) break;
        nx = P.ops[pc + 1];
        if (code < GEN_LSWAP4 || (code >= GEN_HI && code < GEN_T)) {
            const uint32_t f0 = (op.w[0] >> 8) & 0xffu, f1 = (op.w[0] >> 16) & 0xffu;
            if (f0 & 0x58u) v.diagonal(f0, op.w[1]);
            if (f1 & 0x58u) v.diagonal(f1, op.w[2]);
            const float c = coef(op.w[6] ^ extra, op.w[3] & 0xffffu, op.w[4]);
            const float d = coef(op.w[7], op.w[3] >> 16, op.w[5]);
            extra = 0;
            switch (code) {
#define QSV_H1(S) case GEN_H1 + S: v.template h1<S>(c); break;
            QSV_H1(0) QSV_H1(1) QSV_H1(2) QSV_H1(3) QSV_H1(4) QSV_H1(5)
#undef QSV_H1
#define QSV_H2(A, B) case GEN_H2 + gen_pair_index(A, B): v.template h2<A, B>(c, d); break;
            QSV_H2(0, 1) QSV_H2(0, 2) QSV_H2(1, 2) QSV_H2(0, 3) QSV_H2(1, 3) QSV_H2(2, 3)
            QSV_H2(0, 4) QSV_H2(1, 4) QSV_H2(2, 4) QSV_H2(3, 4)
            QSV_H2(0, 5) QSV_H2(1, 5) QSV_H2(2, 5) QSV_H2(3, 5) QSV_H2(4, 5)
#undef QSV_H2
#define QSV_HI(S) case GEN_HI + S: v.template hi<S>(c); break;
            QSV_HI(0) QSV_HI(1) QSV_HI(2) QSV_HI(3) QSV_HI(4) QSV_HI(5)
#undef QSV_HI
#define QSV_H2(A, B) case GEN_H2R + gen_pair_index(A, B): v.template h2r<A, B>(c, d); break;
            QSV_H2(0, 1) QSV_H2(0, 2) QSV_H2(1, 2) QSV_H2(0, 3) QSV_H2(1, 3) QSV_H2(2, 3)
            QSV_H2(0, 4) QSV_H2(1, 4) QSV_H2(2, 4) QSV_H2(3, 4)
            QSV_H2(0, 5) QSV_H2(1, 5) QSV_H2(2, 5) QSV_H2(3, 5) QSV_H2(4, 5)
#undef QSV_H2
#define QSV_PH(S) case GEN_PH + S: v.template ph<S>(c); break;
            QSV_PH(0) QSV_PH(1) QSV_PH(2) QSV_PH(3) QSV_PH(4) QSV_PH(5)
#undef QSV_PH
            default: break;
            }
            continue;
        }
        switch (code) {
        case GEN_XCHG: {
            // new slot s reads at weight h(s) of the old layout
            auto h = [&](int s) { return (op.w[1 + s / 2] >> (16 * (s % 2))) & 0xffffu; };
            uint32_t rt = 0;
#pragma unroll
            for (int u = 0; u < T; ++u) rt += ((t >> u) & 1u) * h(R + u);
            uint32_t off[N];
            off[0] = rt;
#pragma unroll
            for (int j = 1; j < N; ++j) off[j] = off[j & (j - 1)] + h(__builtin_ctz(j));
            __syncthreads();  // earlier reads of the buffer are complete
            if constexpr (HALF) {
#pragma unroll
                for (int j = 0; j < N; ++j) lds[wt + j] = v.re[j];
                __syncthreads();
#pragma unroll
                for (int j = 0; j < N; ++j) v.re[j] = lds[off[j]];
                __syncthreads();
#pragma unroll
                for (int j = 0; j < N; ++j) lds[wt + j] = v.im[j];
                __syncthreads();
#pragma unroll
                for (int j = 0; j < N; ++j) v.im[j] = lds[off[j]];
            } else {
                float2 *buf = reinterpret_cast<float2 *>(lds);
#pragma unroll
                for (int j = 0; j < N; ++j) buf[wt + j] = make_float2(v.re[j], v.im[j]);
                __syncthreads();
#pragma unroll
                for (int j = 0; j < N; ++j) {
                    const float2 x = buf[off[j]];
                    v.re[j] = x.x;
                    v.im[j] = x.y;
                }
            }
            break;
        }
#define QSV_SW(S)                                                         \
    case GEN_LSWAP4 + S: v.template lane_swap<S, 4>(); break;             \
    case GEN_LSWAP5 + S: v.template lane_swap<S, 5>(); break;
        QSV_SW(0) QSV_SW(1) QSV_SW(2) QSV_SW(3) QSV_SW(4) QSV_SW(5)
#undef QSV_SW
#define QSV_T(S) case GEN_T + S: v.template t_gate<S>(__uint_as_float(0x3f3504f3u | op.w[1])); break;
        QSV_T(0) QSV_T(1) QSV_T(2) QSV_T(3) QSV_T(4) QSV_T(5)
#undef QSV_T
        case GEN_ZB:
            extra = (parity(op.w[6] & uint32_t(A.branch)) ^ parity(op.w[7] & uint32_t(A.branch >> 32))) << 31;
            break;
        case GEN_W: {
            const float2 w = omega(e);
            v.all(w.x, w.y);
            e = 0;
            break;
        }
        case GEN_E: {
            const uint32_t loc = (op.w[0] >> 16) & 0xffu;
            const uint32_t bit = (loc & 0x80u) ? (tile >> (loc & 0x7fu)) & 1u : (t >> loc) & 1u;
            const uint32_t sg = (parity(op.w[3] & t) ^ parity(op.w[4] & tile) ^ (extra >> 31)) << 2;
            extra = 0;
            e += bit * (((op.w[0] >> 8) & 7u) + sg);
            break;
        }
        default: {  // projections
            const uint32_t l = (op.w[0] & 0x100u) ? uint32_t(A.branch >> op.w[1]) & 1u : op.w[1];
            if (code == GEN_PROJT) {
                const uint32_t loc = (op.w[0] >> 16) & 0xffu;
                const uint32_t bit = (loc & 0x80u) ? (tile >> (loc & 0x7fu)) & 1u : (t >> loc) & 1u;
                const uint32_t m = bit == l ? ~0u : 0u;
#pragma unroll
                for (int j = 0; j < N; ++j) {
                    keep(v.re[j], m);
                    keep(v.im[j], m);
                }
                break;
            }
            switch (code - GEN_PROJ) {
            case 0: v.template proj<0>(l); break;
            case 1: v.template proj<1>(l); break;
            case 2: v.template proj<2>(l); break;
            case 3: v.template proj<3>(l); break;
            case 4: v.template proj<4>(l); break;
            default: v.template proj<5>(l); break;
            }
            break;
        }
        }
    }

    if (P.scaled) {
        const float2 w = omega(e);
        const float cr = __builtin_fmaf(w.x, P.scale_re, -(P.scale_im * w.y));
        const float ci = __builtin_fmaf(w.y, P.scale_re, P.scale_im * w.x);
#pragma unroll
        for (int j = 0; j < N; ++j) cmul_scale(v.re[j], v.im[j], cr, ci);
    }
    float2 *dst = A.amps + thread_offset(P.st_phys);
#pragma unroll
    for (int j = 0; j < N; j += 2) {
        const v4f w = {v.re[j], v.im[j], v.re[j + 1], v.im[j + 1]};
        *reinterpret_cast<v4f *>(dst + reg_offset(P.st_phys, j)) = w;
    }
    if (A.norm) {
        // FP64 products of FP32 values are exact; fixed thread, lane, wave order.
        // Saves the norm's own read of the state and two launches (with the
        // gather in k_finish; 23 qubits: 164.5 -> 153.1 us, 20: 73.3 -> 69.9)
        // Four amplitudes to a sum, the sums in pairs: as short as in the norm's
        // own kernel.
        double q[N / 4];
#pragma unroll
        for (int j = 0; j < N; j += 4) {
            q[j / 4] = 0.0;
#pragma unroll
            for (int k = j; k < j + 4; ++k)
                q[j / 4] += double(v.re[k]) * double(v.re[k]) + double(v.im[k]) * double(v.im[k]);
        }
#pragma unroll
        for (int h = N / 8; h > 0; h >>= 1)
#pragma unroll
            for (int j = 0; j < h; ++j) q[j] += q[j + h];
        double acc = q[0];
        constexpr int kLanes = T < 6 ? 1 << T : 64;
        for (int h = kLanes / 2; h > 0; h >>= 1) acc += __shfl_down(acc, h, kLanes);
        if constexpr (T > 6) {
            double *s = reinterpret_cast<double *>(lds);
            __syncthreads();  // the last exchange has been read
            if ((t & 63u) == 0) s[t >> 6] = acc;
            __syncthreads();
            if (t == 0)
                for (int k = 1; k < (1 << (T - 6)); ++k) acc += s[k];
        }
        if (t == 0) A.norm[tile] = acc;
    }
}

template <int R, int T, bool HALF>
__global__ void __launch_bounds__(1 << T)
k_tile(const float2 *src, float2 *amps, const GenProg P, uint64_t branch, uint64_t tile0, int init, float init_val,
       uint64_t basis, double *norm) {
    extern __shared__ __attribute__((aligned(16))) float lds[];
    run_tile<R, T, HALF>(P, TileArgs{src, amps, branch, tile0 + blockIdx.x, basis, init, init_val, norm}, lds);
}

// One program round of a batch: block b belongs to the segment with the
// largest start <= b; the segment names the entry (state, branch, programs)
// and its first tile.  With init_plus an entry's first program starts from
// |+>^n.
template <int R, int T, bool HALF>
__global__ void __launch_bounds__(1 << T)
k_tile_batch(const BatchSeg *__restrict__ segs, int nseg, const BatchEntry *__restrict__ ents,
             const GenProg *__restrict__ progs, int round, int init_plus) {
    extern __shared__ __attribute__((aligned(16))) float lds[];
    const uint64_t blk = blockIdx.x;
    int lo = 0, hi = nseg - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (segs[mid].start <= blk) lo = mid; else hi = mid - 1;
    }
    const BatchSeg sg = segs[lo];
    const BatchEntry en = ents[sg.entry];
    float2 *a = reinterpret_cast<float2 *>(en.amps);
    run_tile<R, T, HALF>(
        progs[en.prog0 + round],
        TileArgs{a, a, en.branch, blk - sg.start, 0, (init_plus && round == 0) ? 1 : -1, en.init_val, nullptr}, lds);
}

// Exchanges staged in halves when the tiles are more than the CUs hold at once
// with whole buffers (160 KiB each on 256 CUs): then twice the workgroups on a
// CU hide each other's waits (23 qubits, tile (5, 8, 5): 137.6 -> 100.4 us,
// (4, 8, 4): 111.6 -> 101.2); with fewer tiles the extra barriers only cost (22
// qubits, (4, 8, 4): 71.7 -> 76.6).  Beside compiled passes, which fill the
// device anyway, a batch's rounds stay whole (32 circuits of 14..24 qubits: 835
// us, 852 in halves; 40 generic ones of 16..20 qubits: 220, 199 in halves).
bool stage_halves(int R, int T, uint64_t tiles) {
    const uint64_t whole = uint64_t(gen_weights(R, T).elems) * sizeof(float2);
    return tiles > 256 * ((160u << 10) / whole);
}

template <int R, int T> constexpr size_t tile_lds() { return size_t(gen_weights(R, T).elems) * sizeof(float2); }

template <class K> hipError_t allow_lds(K kernel, size_t bytes) {
    return hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                               int(bytes));
}

template <int R, int T, bool HALF>
hipError_t launch_tile_t(const float2 *src, float2 *amps, int n, const GenProg &p, uint64_t branch, int init,
                         uint64_t basis, double *norm, hipStream_t s) {
    constexpr size_t lds = tile_lds<R, T>() / (HALF ? 2 : 1);
    static const hipError_t attr = allow_lds(&k_tile<R, T, HALF>, lds);
    if (attr != hipSuccess) return attr;
    const uint64_t tiles = 1ull << (n - R - T);
    const uint64_t chunk = 1ull << 30;  // blocks per launch
    const float val = float(1.0 / __builtin_sqrt(double(1ull << n)));
    for (uint64_t t0 = 0; t0 < tiles; t0 += chunk) {
        const uint64_t cnt = (tiles - t0 < chunk) ? tiles - t0 : chunk;
        hipLaunchKernelGGL((k_tile<R, T, HALF>), dim3(unsigned(cnt)), dim3(1 << T), lds, s, src, amps, p, branch, t0,
                           init, val, basis, norm);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

template <int R, int T, bool HALF>
hipError_t launch_tile_batch_t(const BatchSeg *segs, int nseg, const BatchEntry *ents, const GenProg *progs, int round,
                               uint64_t blocks, int init_plus, hipStream_t s) {
    constexpr size_t lds = tile_lds<R, T>() / (HALF ? 2 : 1);
    static const hipError_t attr = allow_lds(&k_tile_batch<R, T, HALF>, lds);
    if (attr != hipSuccess) return attr;
    if (blocks == 0) return hipSuccess;
    if (blocks > kMaxBlocks) return hipErrorInvalidValue;
    hipLaunchKernelGGL((k_tile_batch<R, T, HALF>), dim3(unsigned(blocks)), dim3(1 << T), lds, s, segs, nseg, ents,
                       progs, round, init_plus);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_tile(const float2 *src, float2 *amps, int n, int R, int T, const GenProg &p, uint64_t branch,
                       int init, uint64_t basis, double *norm, hipStream_t s) {
    switch (R * 16 + T) {
#define QSV_SHAPE(RR, TT)                                                                                  \
    case RR * 16 + TT:                                                                                     \
        if (stage_halves(RR, TT, 1ull << (n - RR - TT)))                                                       \
            return launch_tile_t<RR, TT, true>(src, amps, n, p, branch, init, basis, norm, s);                 \
        return launch_tile_t<RR, TT, false>(src, amps, n, p, branch, init, basis, norm, s);
    QSV_SHAPE(5, 9) QSV_SHAPE(5, 8) QSV_SHAPE(5, 7) QSV_SHAPE(4, 9) QSV_SHAPE(4, 8) QSV_SHAPE(4, 7) QSV_SHAPE(4, 6)
    QSV_SHAPE(3, 6) QSV_SHAPE(3, 4) QSV_SHAPE(2, 3) QSV_SHAPE(6, 8) QSV_SHAPE(6, 7)
#undef QSV_SHAPE
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_tile_batch(int R, int T, const BatchSeg *segs, int nseg, const BatchEntry *ents,
                             const GenProg *progs, int round, uint64_t blocks, int init_plus, bool alone,
                             hipStream_t s) {
    switch (R * 16 + T) {
#define QSV_SHAPE(RR, TT)                                                                                            \
    case RR * 16 + TT: {                                                                                             \
        if (blocks == 0) { /* prepares both forms */                                                                 \
            const hipError_t e = launch_tile_batch_t<RR, TT, true>(segs, nseg, ents, progs, round, 0, init_plus, s); \
            if (e != hipSuccess) return e;                                                                           \
        }                                                                                                            \
        if (alone && stage_halves(RR, TT, blocks))                                                                   \
            return launch_tile_batch_t<RR, TT, true>(segs, nseg, ents, progs, round, blocks, init_plus, s);          \
        return launch_tile_batch_t<RR, TT, false>(segs, nseg, ents, progs, round, blocks, init_plus, s);             \
    }
    QSV_SHAPE(5, 9) QSV_SHAPE(5, 8) QSV_SHAPE(5, 7) QSV_SHAPE(4, 8) QSV_SHAPE(4, 7)
#undef QSV_SHAPE
    default: return hipErrorInvalidValue;
    }
}

}  // namespace qsv
