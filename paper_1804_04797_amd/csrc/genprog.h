// Program of the generic tile kernel: a pass program (PassProg) lowered to
// Hadamards with their pending diagonals, exchanges and a closing diagonal.
#pragma once

#include <cstdint>

#include "qsv_internal.h"

namespace qsv {

// Codes of a GenOp (low byte of w[0]); slot and pair numbers are part of the
// code so that one switch reaches straight-line code.
enum GenCode : uint32_t {
    GEN_END = 0,
    GEN_H1 = 1,       // + register slot s: (x, y) -> (x + c y, x - c y)
    GEN_H2 = 8,       // + pair_index(s1, s2): the same on s1, then on s2
    GEN_PH = 24,      // + register slot s: y -> c y (closing diagonal)
    GEN_LSWAP4 = 32,  // + register slot s: swap it with lane bit 4
    GEN_LSWAP5 = 40,  // + register slot s: swap it with lane bit 5
    GEN_PROJ = 48,    // + register slot s: zero the amplitudes whose bit differs from l
    GEN_XCHG = 56,    // slot permutation through LDS; w[1..7] = 14 16-bit element weights
    GEN_PROJT = 57,   // projection on a thread or tile-index bit
    GEN_E = 58,       // diagonal of a thread or tile-index bit: adds to the exponent e of w
    GEN_W = 59,       // multiply by w^e, e = 0
    GEN_ZB = 60,      // sign of the next op from branch bits
    // gate order (see lower_plan)
    GEN_HI = 64,      // + register slot s: (x, y) -> (x - i c y, c y - i x)
    GEN_H2R = 72,     // + pair_index(s1, s2): GEN_H1 on s2, then on s1
    GEN_T = 96,       // + register slot s: y -> e^{+-i pi/4} y, sign bit of the angle in w[1]
};

// The second half y of GEN_H1/H2/HI/PH is multiplied by w^l (-1)^{parity} first,
// l = 0..7 (w = e^{i pi/4}).  Operand k = 0, 1 of an op:
//   w[0] byte 1 + k: slot in bits 0-2, bit 3 T (l odd: (1 + i) y), bit 4 I
//                    (l & 2: i y), bit 6: the signs w[1 + k] are used
//   w[1 + k]: sign bit of pair p (the registers with bit `slot` set, in order)
//   w[3] half k: thread partners;  w[4 + k]: tile-index partners
//   w[6 + k]: bits of the FP32 coefficient: 1, or sqrt(1/2) after T; sign l & 4
// A GEN_ZB in front negates operand 0 by the parity of the branch bits w[6..7].
// GEN_PROJ / GEN_PROJT: bit 8 of w[0]: l is branch bit w[1], else l = w[1].
// GEN_PROJT / GEN_E: byte 2 of w[0]: locator (thread bit, or 0x80 | tile-index
// bit); GEN_E: byte 1 of w[0] = l, partners in w[3] and w[4].
struct alignas(32) GenOp {
    uint32_t w[8];
};

constexpr int kGenOps = 120;  // ops of one program, END included (a kernel argument: below 4 KiB)
constexpr int kGenRuns = 18;  // runs of consecutive tile-index bits

struct GenProg {
    GenOp ops[kGenOps];
    // 32-bit words only: the kernel reads them with scalar loads
    uint32_t ld_phys[kMaxSlots / 4];  // physical bit of each slot at load, a byte each
    uint32_t st_phys[kMaxSlots / 4];  // ... at store
    uint32_t run[kGenRuns];           // tile index -> origin: bits [src, src + len) to bit dst (src | len << 8 | dst << 16)
    uint32_t n_runs, scaled, n_ops;
    float scale_re, scale_im;
    uint32_t pad;
};

static_assert(sizeof(GenProg) <= 4032, "GenProg is a kernel argument");

QSV_HD inline uint32_t gen_phys(const uint32_t *phys, int s) { return (phys[s / 4] >> (8 * (s % 4))) & 0xffu; }

constexpr int gen_pair_index(int s1, int s2) {  // s1 < s2 < 6
    return s2 * (s2 - 1) / 2 + s1;
}

// Element weight of slot coordinate q in the exchange buffer: register slots
// 2^q, thread bit u (2^R + 1) 2^u + d_u.  Every weight exceeds the sum of the
// smaller ones, so an address names one element; d_u moves thread bits 4 and
// up off the bank pair of multiples of 16, so that a load whose lanes walk
// them does not serialise on one bank.
struct GenWeights {
    uint32_t w[kMaxSlots];
    uint32_t elems;
};
constexpr GenWeights gen_weights(int R, int T) {
    GenWeights g{};
    uint32_t sum = 0;
    for (int q = 0; q < R; ++q) {
        g.w[q] = 1u << q;
        sum += g.w[q];
    }
    const uint32_t residue[6] = {3, 6, 12, 9, 5, 10};
    for (int u = 0; u < T; ++u) {
        uint32_t x = (uint32_t(1 << R) + 1) << u;
        if (u >= 4) {
            if (x < sum + 1) x = sum + 1;
            while ((x & 15u) != residue[u - 4]) ++x;
        }
        g.w[R + u] = x;
        sum += x;
    }
    g.elems = sum + 1;
    return g;
}

// Lowers the passes of an in-place plan (natural qubit order).  A program
// longer than kGenOps is split: the tile is stored and loaded again.
// gate_order: T gates are multiplied in where the pass program has them (on a
// register slot at once, on other bits before the next exchange), so that
// every rounding is the one of the pass program run op by op; only signs,
// which round nothing, are folded into the butterflies.  Otherwise T gates
// and powers of i are folded too.
qsv_status lower_plan(const Plan &plan, bool gate_order, std::vector<GenProg> &out);
// The lowered programs of the plan, made on first use and kept with it.
qsv_status generic_programs(Plan &plan, bool gate_order, std::shared_ptr<const std::vector<GenProg>> &out);

// Host execution of one program (CPU checks of the lowering).
void emulate_gen(const GenProg &p, int n, int R, int T, uint64_t branch, float *amps);

}  // namespace qsv
