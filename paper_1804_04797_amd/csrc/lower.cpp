// Lowers pass programs for the generic tile kernel.
//
// Every non-diagonal gate is a Hadamard butterfly between two powers of i:
//   SX = g(-i) H b(-i), SY = H b(-1), SXDG = g(i) H b(i), SYDG = g(-1) H
// (b, g: diag(1, .) before and after; scalar factors are already removed).  A
// diagonal gate therefore never runs by itself: for every qubit the lowering
// keeps an exponent l of w = e^{i pi/4}, the set of qubits it shares a pending
// CZ with and the branch bits that negate it.  A Hadamard on a qubit applies
// what is pending on that qubit to its second half and clears it.  The pending
// diagonal is a function of the qubits, not of where they sit, so exchanges
// and pass boundaries leave it alone; the last pass of a call applies the rest.
// Consecutive Hadamards on two register slots become one op (four amplitudes
// in, four out, no copies).
#include <algorithm>
#include <cmath>
#include <cstring>
#include <memory>
#include <vector>

#include "genprog.h"

namespace qsv {

namespace {

constexpr uint8_t kT = 8, kI = 16, kK = 64;
constexpr uint32_t kOne = 0x3f800000u, kSqrtHalf = 0x3f3504f3u, kSign = 0x80000000u;  // FP32 bits

struct Pending {
    int l = 0;        // exponent of w
    uint64_t cz = 0;  // partners
    uint64_t zb = 0;  // branch bits
    bool any() const { return l || cz || zb; }
};

struct Lower {
    const Plan &plan;
    std::vector<GenProg> &out;
    const int R, T, L, n;
    const GenWeights W;
    Pending pend[64];
    int occ[kMaxSlots];      // qubit of each slot
    int slot_of[64];         // slot of a resident qubit, else -1
    int tile_bit[64];        // tile-index bit of a non-resident qubit
    const PassProg *P = nullptr;
    GenProg cur;
    int n_ops = 0;
    bool open_h1 = false;    // the last op is a Hadamard that another may join
    const bool gate_order;
    int ahead = 0;           // at most so many ops follow up to the next exchange
    bool e_dirty = false;    // e holds phases not multiplied in yet

    Lower(const Plan &p, bool ordered, std::vector<GenProg> &o)
        : plan(p), out(o), R(p.R), T(p.T), L(p.R + p.T), n(p.n), W(gen_weights(p.R, p.T)),
          gate_order(ordered) {}

    void open() {
        std::memset(&cur, 0, sizeof(cur));
        n_ops = 0;
        open_h1 = false;
        for (int s = 0; s < L; ++s) cur.ld_phys[s / 4] |= uint32_t(P->ld_phys[s]) << (8 * (s % 4));
        std::copy(cur.ld_phys, cur.ld_phys + kMaxSlots / 4, cur.st_phys);
        int r = 0;
        for (int i = 0, j; i < P->n_glob; i = j + 1) {
            for (j = i; j + 1 < P->n_glob && P->glob_bits[j + 1] == P->glob_bits[j] + 1;) ++j;
            cur.run[r++] = uint32_t(i) | uint32_t(j - i + 1) << 8 | uint32_t(P->glob_bits[i]) << 16;
        }
        cur.n_runs = uint32_t(r);
        cur.scale_re = 1.f;
        place(P->ld_phys);
    }
    void close() {
        cur.ops[n_ops].w[0] = GEN_END;
        cur.n_ops = uint32_t(n_ops + 1);
        out.push_back(cur);
    }
    template <class I> void place(const I *qubits) {
        for (int q = 0; q < 64; ++q) slot_of[q] = -1;
        for (int s = 0; s < L; ++s) {
            occ[s] = qubits[s];
            slot_of[occ[s]] = s;
        }
    }
    GenOp &push(uint32_t code) {
        if (n_ops >= kGenOps - 2) split();  // room for the exchange of a split and END
        open_h1 = false;
        GenOp &g = cur.ops[n_ops++];
        std::memset(&g, 0, sizeof(g));
        g.w[0] = code;
        return g;
    }
    // LDS exchange to the layout in which slot s holds qubit want[s]
    void exchange_op(const int *want) {
        GenOp &g = cur.ops[n_ops++];
        std::memset(&g, 0, sizeof(g));
        g.w[0] = GEN_XCHG;
        for (int s = 0; s < L; ++s) g.w[1 + s / 2] |= W.w[slot_of[want[s]]] << (16 * (s % 2));
        open_h1 = false;
        place(want);
    }
    // A full program stores the tile from the pass's load layout; the next
    // one loads it again and returns to the layout it had.
    void split() {
        int was[kMaxSlots], ld[kMaxSlots];
        std::copy(occ, occ + L, was);
        for (int s = 0; s < L; ++s) ld[s] = P->ld_phys[s];
        const bool moved = !std::equal(was, was + L, ld);
        if (moved) exchange_op(ld);
        cur.scaled = e_dirty ? 1u : 0u;  // e does not outlive a program
        e_dirty = false;
        close();
        open();
        if (moved) exchange_op(was);
    }
    void xchg(uint64_t pw) {
        int want[kMaxSlots], perm[kMaxSlots];
        bool lane = T >= 6, any = false;
        for (int s = 0; s < L; ++s) {
            perm[s] = int((pw >> (4 * s)) & 0xf);
            want[s] = occ[perm[s]];
        }
        // swaps of register slots with lane bits 4 and 5 only need no LDS
        for (int s = 0; s < L; ++s) {
            const int o = perm[s];
            if (o == s) continue;
            any = true;
            lane = lane && perm[o] == s &&
                   ((s < R && (o == R + 4 || o == R + 5)) || (o < R && (s == R + 4 || s == R + 5)));
        }
        if (e_dirty) push(GEN_W);
        e_dirty = false;
        // a program that cannot take the ops up to the next exchange ends
        // here, with nothing left in e
        if (n_ops + ahead + 3 > kGenOps - 2) split();
        if (!any) return;
        if (lane) {
            for (int s = 0; s < R; ++s) {
                if (perm[s] == s) continue;
                push((perm[s] == R + 4 ? GEN_LSWAP4 : GEN_LSWAP5) + uint32_t(s));
                std::swap(occ[s], occ[perm[s]]);
                place(std::vector<int>(occ, occ + L).data());
            }
            return;
        }
        exchange_op(want);
    }
    uint32_t reg_mask(uint64_t qs) const { return slot_mask(qs, 0, R); }
    uint32_t thread_mask(uint64_t qs) const { return slot_mask(qs, R, L); }
    uint32_t slot_mask(uint64_t qs, int lo, int hi) const {
        uint32_t m = 0;
        for (int s = lo; s < hi; ++s)
            if ((qs >> occ[s]) & 1) m |= 1u << (s - lo);
        return m;
    }
    uint32_t tile_mask(uint64_t qs) const {
        uint32_t m = 0;
        for (int i = 0; i < P->n_glob; ++i)
            if ((qs >> P->glob_bits[i]) & 1) m |= 1u << i;
        return m;
    }
    // operand k of an op on register slot s takes what is pending on its qubit
    void operand(GenOp &g, int k, int s) {
        const Pending &p = pend[occ[s]];
        uint32_t f = uint32_t(s) | (p.l & 1 ? kT : 0) | (p.l & 2 ? kI : 0);
        uint32_t K = 0;
        if (const uint32_t rm = reg_mask(p.cz)) {
            f |= kK;
            for (int j = 0, i = 0; j < (1 << R); ++j) {
                if (!((j >> s) & 1)) continue;
                K |= uint32_t(__builtin_popcount(uint32_t(j) & rm) & 1) << i++;
            }
        }
        g.w[0] |= f << (8 + 8 * k);
        g.w[1 + k] = K;
        g.w[3] |= thread_mask(p.cz) << (16 * k);
        g.w[4 + k] = tile_mask(p.cz);
        g.w[6 + k] = (p.l & 1 ? kSqrtHalf : kOne) | (p.l & 4 ? kSign : 0);
        clear(occ[s]);
    }
    // an op on register slot s; branch bits pending on it go in front
    GenOp &push_on(uint32_t code, int s) {
        if (n_ops >= kGenOps - 3) split();
        branch_sign(pend[occ[s]].zb);
        GenOp &g = push(code);
        operand(g, 0, s);
        return g;
    }
    void branch_sign(uint64_t zb) {
        if (!zb) return;
        GenOp &g = push(GEN_ZB);
        g.w[6] = uint32_t(zb);
        g.w[7] = uint32_t(zb >> 32);
    }
    void clear(int q) {
        for (int o = 0; o < 64; ++o)
            if ((pend[q].cz >> o) & 1) pend[o].cz &= ~(1ull << q);
        pend[q] = Pending{};
    }
    // phase i^{before/2} on the second half, the butterfly, phase after it
    void hadamard(int s, int before, int after) {
        Pending &p = pend[occ[s]];
        p.l = (p.l + before) & 7;
        GenOp *g = open_h1 ? &cur.ops[n_ops - 1] : nullptr;
        const int s1 = g ? int(g->w[0] & 0xff) - GEN_H1 : -1;
        // what the second gate applies must not depend on the first one's slot
        if (g && s1 != s && !((p.cz >> occ[s1]) & 1) && !p.zb) {
            operand(*g, 1, s);
            const bool reversed = s < s1;
            if (reversed) {  // operands in slot order
                g->w[0] = (g->w[0] & 0xff0000ffu) | ((g->w[0] >> 8) & 0xff00u) | ((g->w[0] & 0xff00u) << 8);
                std::swap(g->w[1], g->w[2]);
                std::swap(g->w[4], g->w[5]);
                std::swap(g->w[6], g->w[7]);
                g->w[3] = g->w[3] >> 16 | g->w[3] << 16;
            }
            g->w[0] = (g->w[0] & ~0xffu) | uint32_t((reversed && gate_order ? GEN_H2R : GEN_H2) +
                                                    gen_pair_index(std::min(s1, s), std::max(s1, s)));
            open_h1 = false;
        } else {
            const bool plain = !p.zb;
            push_on(uint32_t(GEN_H1 + s), s);
            open_h1 = plain;
        }
        pend[occ[s]].l = after;
    }
    // (x, y) -> (x - i y, y - i x) as such, signs before and after it pending
    void imaginary(int s, int before, int after) {
        Pending &p = pend[occ[s]];
        p.l = (p.l + before) & 7;
        push_on(uint32_t(GEN_HI + s), s);
        pend[occ[s]].l = after;
    }
    void phase(uint32_t loc, int k) {
        const int q = qubit(loc);
        if (!gate_order || k == 4) {
            pend[q].l = (pend[q].l + k) & 7;
            return;
        }
        const int s = slot_of[q];
        if (s >= 0 && s < R) {
            push(uint32_t(GEN_T + s)).w[1] = k == 7 ? 0x80000000u : 0u;
        } else {
            push(GEN_E).w[0] |= uint32_t(k) << 8 | locator(q) << 16;
            e_dirty = true;
        }
    }
    int qubit(uint32_t loc) const { return (loc & kLocGlobal) ? int(loc & 0x7f) : occ[loc]; }
    // locator byte of a thread or tile-index bit
    uint32_t locator(int q) const {
        return slot_of[q] >= 0 ? uint32_t(slot_of[q] - R) : uint32_t(kLocGlobal) | uint32_t(tile_bit[q]);
    }
    void projection(int q, uint32_t b, uint32_t c) {
        const int s = slot_of[q];
        const bool reg = s >= 0 && s < R;
        GenOp &g = push(reg ? uint32_t(GEN_PROJ + s) : uint32_t(GEN_PROJT));
        if (c) g.w[0] |= 1u << 8;
        if (!reg) g.w[0] |= locator(q) << 16;
        g.w[1] = b;
    }
    // the rest of the pending diagonal: register slots, then the other qubits
    void closing() {
        for (int s = 0; s < R; ++s)
            if (pend[occ[s]].any()) push_on(uint32_t(GEN_PH + s), s);
        for (int q = 0; q < n; ++q) {
            const Pending p = pend[q];
            if (!p.any()) continue;
            if (n_ops >= kGenOps - 3) split();
            branch_sign(p.zb);
            GenOp &g = push(GEN_E);
            g.w[0] |= uint32_t(p.l) << 8 | locator(q) << 16;
            g.w[3] = thread_mask(p.cz);
            g.w[4] = tile_mask(p.cz);
            e_dirty = true;  // a split before the next one multiplies it in
            clear(q);
        }
    }

    qsv_status run() {
        for (size_t pi = 0; pi < plan.passes.size(); ++pi) {
            const bool last = pi + 1 == plan.passes.size();
            P = &plan.passes[pi].prog;
            for (int i = 0; i < P->n_glob; ++i) {
                if (P->glob_bits[i] != P->glob_st[i]) return fail(QSV_EINTERNAL, "lower_plan: not an in-place plan");
                tile_bit[P->glob_bits[i]] = i;
            }
            open();
            for (int pc = 0; pc < P->n_ops; ++pc) {
                const uint64_t op = P->ops[pc];
                const uint32_t a = uint32_t((op >> 8) & 0xff), b = uint32_t((op >> 16) & 0xff);
                switch (uint32_t(op & 0xff)) {
                case OP_H: hadamard(int(a), 0, 0); break;
                case OP_SX: gate_order ? imaginary(int(a), 0, 0) : hadamard(int(a), 6, 6); break;
                case OP_SY: hadamard(int(a), 4, 0); break;
                case OP_SXDG: gate_order ? imaginary(int(a), 4, 4) : hadamard(int(a), 2, 2); break;
                case OP_SYDG: hadamard(int(a), 0, 4); break;
                case OP_PHASE: phase(a, int(b)); break;
                case OP_CZ:
                    pend[qubit(a)].cz ^= 1ull << qubit(b);
                    pend[qubit(b)].cz ^= 1ull << qubit(a);
                    break;
                case OP_ZB: pend[qubit(a)].zb ^= 1ull << b; break;
                case OP_PROJ: projection(qubit(a), b, uint32_t((op >> 24) & 0xff)); break;
                case OP_XCHG: {
                    const uint64_t perm = P->ops[++pc];
                    for (ahead = 1; pc + ahead < P->n_ops && (P->ops[pc + ahead] & 0xff) != OP_XCHG;) ++ahead;
                    if (last && pc + ahead >= P->n_ops) ahead += n;  // the closing diagonal
                    xchg(perm);
                    break;
                }
                default: break;  // OP_SCALE: the program's closing scale
                }
            }
            if (last) closing();
            std::fill(cur.st_phys, cur.st_phys + kMaxSlots / 4, 0u);
            for (int s = 0; s < L; ++s) cur.st_phys[s / 4] |= uint32_t(occ[s]) << (8 * (s % 4));
            cur.scale_re = P->scale_re;
            cur.scale_im = P->scale_im;
            cur.scaled = (last || e_dirty || P->scale_re != 1.f || P->scale_im != 0.f) ? 1u : 0u;
            e_dirty = false;  // the closing scale includes w^e
            close();
        }
        return QSV_OK;
    }
};

}  // namespace

qsv_status lower_plan(const Plan &plan, bool gate_order, std::vector<GenProg> &out) {
    out.clear();
    if (plan.oop) return fail(QSV_EINTERNAL, "lower_plan: not an in-place plan");
    auto l = std::make_unique<Lower>(plan, gate_order, out);
    return l->run();
}

qsv_status generic_programs(Plan &plan, bool gate_order, std::shared_ptr<const std::vector<GenProg>> &out) {
    std::lock_guard<std::mutex> g(plan.jit_mu);
    auto &kept = plan.gen[gate_order ? 1 : 0];
    if (!kept) {
        auto p = std::make_shared<std::vector<GenProg>>();
        const qsv_status st = lower_plan(plan, gate_order, *p);
        if (st != QSV_OK) return st;
        kept = p;
    }
    out = kept;
    return QSV_OK;
}

namespace {

unsigned parity(uint64_t x) { return unsigned(__builtin_popcountll(x) & 1); }

void mul(float *z, float cr, float ci) {
    const float re = std::fma(z[0], cr, -(z[1] * ci)), im = std::fma(z[1], cr, z[0] * ci);
    z[0] = re;
    z[1] = im;
}
void mul_omega(float *z, uint32_t e) {
    const float h = float(std::sqrt(0.5));
    const float wr[8] = {1.f, h, 0.f, -h, -1.f, -h, 0.f, h}, wi[8] = {0.f, h, 1.f, h, 0.f, -h, -1.f, -h};
    mul(z, wr[e & 7], wi[e & 7]);
}
// coefficient of operand k in thread t of a tile
float operand_coef(const uint32_t *w, int k, uint32_t t, uint64_t tile, unsigned extra) {
    const unsigned sg = parity((w[3] >> (16 * k)) & 0xffff & t) ^ parity(w[4 + k] & tile) ^ (k == 0 ? extra : 0u);
    float c;
    std::memcpy(&c, &w[6 + k], sizeof c);
    return sg ? -c : c;
}
// The ops that only gate-ordered programs have.
void emulate_ordered(const uint32_t *w, int R, int T, uint64_t tile, unsigned extra, float *v) {
    const int N = 1 << R;
    const uint32_t code = w[0] & 0xff;
    const float h = float(std::sqrt(0.5));
    auto signs = [&](int k) {  // signs K of the operand's registers
        const uint32_t f = (w[0] >> (8 + 8 * k)) & 0xff;
        if (!(f & kK)) return;
        for (uint32_t t = 0; t < (1u << T); ++t)
            for (int j = 0, i = 0; j < N; ++j) {
                if (!((j >> (f & 7)) & 1)) continue;
                if ((w[1 + k] >> i++) & 1) {
                    float *y = v + 2 * (uint32_t(j) | t << R);
                    y[0] = -y[0];
                    y[1] = -y[1];
                }
            }
    };
    auto pairs = [&](int s, auto fn) {
        for (uint32_t t = 0; t < (1u << T); ++t)
            for (int j = 0; j < N; ++j)
                if (!((j >> s) & 1)) fn(t, v + 2 * (uint32_t(j) | t << R), v + 2 * (uint32_t(j | 1 << s) | t << R));
    };
    if (code >= GEN_T) {
        pairs(int(code - GEN_T), [&](uint32_t, float *, float *y) { mul(y, h, w[1] ? -h : h); });
    } else if (code >= GEN_H2R) {
        signs(0);
        signs(1);
        for (int k = 1; k >= 0; --k)
            pairs(int((w[0] >> (8 + 8 * k)) & 7), [&](uint32_t t, float *x, float *y) {
                const float c = operand_coef(w, k, t, tile, extra);
                for (int q = 0; q < 2; ++q) {
                    const float a = x[q] + c * y[q];
                    y[q] = x[q] - c * y[q];
                    x[q] = a;
                }
            });
    } else {
        signs(0);
        pairs(int(code - GEN_HI), [&](uint32_t t, float *x, float *y) {
            const float c = operand_coef(w, 0, t, tile, extra);
            const float xr = x[0] + c * y[1], xi = x[1] - c * y[0], yr = x[1] + c * y[0], yi = c * y[1] - x[0];
            // c y - i x = (c yr + xi, c yi - xr)
            x[0] = xr; x[1] = xi; y[0] = yr; y[1] = yi;
        });
    }
}

}  // namespace

// The ops in the order and with the arithmetic of the device kernel.
void emulate_gen(const GenProg &p, int n, int R, int T, uint64_t branch, float *amps) {
    const int L = R + T, N = 1 << R;
    const GenWeights W = gen_weights(R, T);
    const float h = float(std::sqrt(0.5));
    std::vector<float> v(size_t(2) << L), buf(size_t(2) * W.elems);
    for (uint64_t tile = 0; tile < (1ull << (n - L)); ++tile) {
        uint64_t base = 0;
        for (uint32_t r = 0; r < p.n_runs; ++r)
            base |= ((tile >> (p.run[r] & 0xff)) & ((1ull << ((p.run[r] >> 8) & 0xff)) - 1)) << (p.run[r] >> 16);
        auto addr = [&](const uint32_t *phys, uint32_t x) {
            uint64_t a = base;
            for (int s = 0; s < L; ++s)
                if ((x >> s) & 1) a |= 1ull << gen_phys(phys, s);
            return a;
        };
        for (uint32_t x = 0; x < (1u << L); ++x)
            std::memcpy(&v[2 * x], amps + 2 * addr(p.ld_phys, x), 2 * sizeof(float));
        std::vector<uint32_t> e(size_t(1) << T, 0u);
        unsigned extra = 0;  // sign of the next op (GEN_ZB)
        for (uint32_t pc = 0; pc < p.n_ops; ++pc) {
            const uint32_t *w = p.ops[pc].w;
            const uint32_t code = w[0] & 0xff;
            if (code == GEN_END) break;
            if (code == GEN_ZB) {
                extra = parity((uint64_t(w[6]) | uint64_t(w[7]) << 32) & branch);
                continue;
            }
            if (code >= GEN_HI) {
                emulate_ordered(w, R, T, tile, extra, v.data());
            } else if (code == GEN_W) {
                for (uint32_t x = 0; x < (1u << L); ++x) {
                    mul_omega(&v[2 * x], e[x >> R]);
                }
                std::fill(e.begin(), e.end(), 0u);
            } else if (code < GEN_LSWAP4) {
                const int nop = (code >= GEN_H2 && code < GEN_PH) ? 2 : 1;
                for (int k = 0; k < nop; ++k)  // both operands' diagonals, then both butterflies
                    for (uint32_t t = 0; t < (1u << T); ++t)
                        for (int j = 0, i = 0; j < N; ++j) {
                            const uint32_t f = (w[0] >> (8 + 8 * k)) & 0xff;
                            if (!((j >> (f & 7)) & 1)) continue;
                            float *y = &v[2 * (uint32_t(j) | t << R)];
                            if (f & kT) { const float yr = y[0] - y[1]; y[1] = y[0] + y[1]; y[0] = yr; }
                            if (f & kI) { const float yr = -y[1]; y[1] = y[0]; y[0] = yr; }
                            if ((f & kK) && ((w[1 + k] >> i) & 1)) { y[0] = -y[0]; y[1] = -y[1]; }
                            ++i;
                        }
                for (int k = 0; k < nop; ++k)
                    for (uint32_t t = 0; t < (1u << T); ++t) {
                        const int s = int((w[0] >> (8 + 8 * k)) & 7);
                        const float c = operand_coef(w, k, t, tile, extra);
                        for (int j = 0; j < N; ++j) {
                            if ((j >> s) & 1) continue;
                            float *x = &v[2 * (uint32_t(j) | t << R)], *y = &v[2 * (uint32_t(j | 1 << s) | t << R)];
                            for (int q = 0; q < 2; ++q) {
                                if (code >= GEN_PH) { y[q] *= c; continue; }
                                const float a = std::fma(c, y[q], x[q]);
                                y[q] = std::fma(-c, y[q], x[q]);
                                x[q] = a;
                            }
                        }
                    }
            } else if (code < GEN_PROJ) {
                const int s = int(code & 7), u = code < GEN_LSWAP5 ? 4 : 5;
                for (uint32_t x = 0; x < (1u << L); ++x) {
                    if (!((x >> s) & 1) || ((x >> (R + u)) & 1)) continue;
                    const uint32_t o = (x ^ (1u << s)) | 1u << (R + u);
                    std::swap(v[2 * x], v[2 * o]);
                    std::swap(v[2 * x + 1], v[2 * o + 1]);
                }
            } else if (code == GEN_XCHG) {
                for (uint32_t x = 0; x < (1u << L); ++x) {
                    uint32_t a = 0;
                    for (int s = 0; s < L; ++s)
                        if ((x >> s) & 1) a += W.w[s];
                    buf[2 * a] = v[2 * x];
                    buf[2 * a + 1] = v[2 * x + 1];
                }
                for (uint32_t x = 0; x < (1u << L); ++x) {
                    uint32_t a = 0;
                    for (int s = 0; s < L; ++s)
                        if ((x >> s) & 1) a += (w[1 + s / 2] >> (16 * (s % 2))) & 0xffff;
                    v[2 * x] = buf[2 * a];
                    v[2 * x + 1] = buf[2 * a + 1];
                }
            } else if (code == GEN_E) {
                for (uint32_t t = 0; t < (1u << T); ++t) {
                    const uint32_t loc = (w[0] >> 16) & 0xff;
                    const uint32_t bit = (loc & kLocGlobal) ? uint32_t(tile >> (loc & 0x7f)) & 1 : (t >> loc) & 1;
                    e[t] += bit * (((w[0] >> 8) & 7) + 4 * (parity(w[3] & t) ^ parity(w[4] & tile) ^ extra));
                }
            } else {  // projections
                const uint32_t l = (w[0] >> 8) & 1 ? uint32_t(branch >> w[1]) & 1 : w[1], loc = (w[0] >> 16) & 0xff;
                for (uint32_t x = 0; x < (1u << L); ++x) {
                    const uint32_t bit = code != GEN_PROJT     ? (x >> (code & 7)) & 1
                                         : (loc & kLocGlobal) ? uint32_t(tile >> (loc & 0x7f)) & 1
                                                              : (x >> (R + loc)) & 1;
                    if (bit != l) v[2 * x] = v[2 * x + 1] = 0.f;
                }
            }
            extra = 0;
        }
        const float wr[8] = {1.f, h, 0.f, -h, -1.f, -h, 0.f, h}, wi[8] = {0.f, h, 1.f, h, 0.f, -h, -1.f, -h};
        for (uint32_t x = 0; x < (1u << L); ++x) {
            float a = v[2 * x], b = v[2 * x + 1];
            if (p.scaled) {
                const uint32_t k = e[x >> R] & 7;
                const float cr = std::fma(wr[k], p.scale_re, -(p.scale_im * wi[k]));
                const float ci = std::fma(wi[k], p.scale_re, p.scale_im * wr[k]);
                const float r = std::fma(a, cr, -(b * ci));
                b = std::fma(a, ci, b * cr);
                a = r;
            }
            float *o = amps + 2 * addr(p.st_phys, x);
            o[0] = a;
            o[1] = b;
        }
    }
}

}  // namespace qsv
