// Batched execution of many states (sv_batch_*).
//
// Many states - the branches of the halves of a cut circuit (Fig. 2, eq. (1))
// or independent circuits of uneven size - are swept together.  Every entry
// has its own state, branch index and pass plan; the pass programs of all
// plans live in one device array.  Entries fall into size classes:
//  - states of 2^14 amplitudes or fewer: one tile holds the whole state (the
//    whole circuit in one workgroup, registers and LDS: one read and one
//    write of the state per pass, usually one pass);
//  - larger states below 2^21 amplitudes: the batch's tile shape;
//  - states of 2^21 amplitudes or more: compiled kernels of their own plan
//    on the tile shape autotuned for their class (one launch per plan and
//    pass, all entries of the plan in its grid); a plan that kSharedPlan
//    entries or more share is compiled at any size, and states that its
//    entries share are computed once (share_passes).
// The generic-kernel classes run as one launch per tile shape and program
// round (a pass is one program, a very long one several), ordered by kernel
// boundaries.  The schedule of a persistent form (work items (pass round,
// entry, tile) taken in order from a device counter, BatchRound) is kept for
// its host check; its kernel did not finish on the device and is gone.  The
// launches and the closing gather of every entry's sampled amplitudes are
// captured once into a hipGraph and replayed: one graph launch per run.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <thread>
#include <atomic>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <map>
#include <memory>
#include <set>
#include <vector>

#include "jit.h"
#include "kernels.h"
#include "qsv_internal.h"

// Entries of the generic kernel that share one tile shape.
struct BatchShape {
    int R = 0, T = 0, c = 0;
    std::vector<uint32_t> entries;
    std::vector<int> round_seg_off, round_nseg;  // per-round launches: their segments
    std::vector<uint64_t> round_blocks;
    qsv::BatchSeg *d_segs = nullptr;             // into the batch's table block
};

// One launch of a compiled plan: a pass over count rows of the plan's table.
struct BatchStep {
    size_t pass, first, count;
};
// Row of that table: the pass reads state src and writes state dst for the
// branch of an entry (position in the plan's group).  States below the group's
// size are the entries' own, the others the plan's scratch.
struct BatchRow {
    uint32_t entry, dst, src;
};

struct qsv_batch {
    int R = 0, T = 0, c = 0;
    int low = 0;                // opts->low_qubits
    bool forced_shape = false;  // opts gave a tile shape: every generic entry uses it
    int jit_mode = 0;  // opts->jit: 1 always, -1 never, 0 for plans shared by >= 8 entries
    std::vector<std::vector<uint32_t>> group;       // entries of each plan
    std::vector<char> plan_jit;                     // plan runs as compiled kernels
    std::vector<char *> d_scratch;                  // states that a plan's entries share, or null
    std::vector<std::vector<BatchRow>> rows;        // per compiled plan: rows of its steps
    std::vector<std::vector<BatchStep>> steps;      // and its launches, in order
    std::vector<qsv::BatchEntry *> d_group_ents;    // per compiled plan: its rows' table
    std::vector<const qsv_circuit *> circs;
    std::vector<uint64_t> branches;
    // built for the layer range of the current run
    int built_lb = -1;
    std::vector<std::shared_ptr<qsv::Plan>> plans;
    std::vector<uint32_t> entry_plan;
    std::vector<BatchShape> shapes;
    qsv::GenProg *d_progs = nullptr;
    qsv::BatchEntry *d_ents = nullptr;
    void *d_tabs = nullptr;           // segments of every shape
    std::vector<qsv::BatchEntry> h_ents;
    // captured graph and the arguments it was captured for
    hipGraphExec_t exec = nullptr;
    hipStream_t cap = nullptr;
    // side streams of the capture: the chains of launches become parallel
    // branches of the graph (fork and join events)
    std::vector<hipStream_t> lanes;
    std::vector<hipEvent_t> lane_done;
    hipEvent_t fork = nullptr;
    std::vector<void *> g_ptrs;
    int g_init = -1;
    const void *g_bits = nullptr;
    size_t g_m = 0;
    void *g_table = nullptr;
};

namespace qsv {
namespace {

qsv_status hipfail(hipError_t e, const char *where) {
    return fail(QSV_EHIP, std::string(where) + ": " + hipGetErrorString(e));
}

void free_tables(qsv_batch *b) {
    for (auto *p : b->d_group_ents)
        if (p) hipFree(p);
    b->d_group_ents.clear();
    for (char *p : b->d_scratch)
        if (p) hipFree(p);
    b->d_scratch.clear();
    if (b->d_progs) hipFree(b->d_progs);
    if (b->d_ents) hipFree(b->d_ents);
    if (b->d_tabs) hipFree(b->d_tabs);
    b->d_progs = nullptr;
    b->d_ents = nullptr;
    b->d_tabs = nullptr;
    b->shapes.clear();
}

void drop_graph(qsv_batch *b) {
    if (b->exec) hipGraphExecDestroy(b->exec);
    b->exec = nullptr;
}

// Size classes: states of 2^21 amplitudes or more stream from HBM (or the
// last-level cache) and are swept by compiled kernels of their own plan
// (unless jit = -1); smaller ones run the generic kernel (or compiled kernels
// per plan shared by >= 8 entries): states of at most 2^14 amplitudes on a
// tile that holds the whole state, the others on the batch's tile shape.
constexpr int kBigState = 21;
// side streams of a batch's capture (512 uneven circuits: 53.2 ms with
// none, 47.2 with 2, 45.6 with 4, 45.8 with 8, 46.1 with 16)
constexpr int kLanes = 4;
constexpr int kLdsState = 14;
// entries that share a plan from which on its kernels are compiled
constexpr size_t kSharedPlan = 8;
bool big_state(const qsv_batch *b, int n) { return b->jit_mode >= 0 && n >= kBigState; }
// most scratch of a batch for states that entries share, and of one plan; more
// of them stay in the entries' own buffers, for one more launch where they are
// overwritten
constexpr size_t kShareScratch = size_t(128) << 20, kPlanScratch = size_t(64) << 20;
// entries of one launch of a compiled pass (grid rows)
constexpr size_t kGridRows = 65536;
// whether a plan of n qubits with count entries runs as compiled passes
bool compiled(const qsv_batch *b, int n, size_t count) {
    return (b->jit_mode > 0 || (b->jit_mode == 0 && (count >= kSharedPlan || big_state(b, n)))) && count < kGridRows;
}

// Tile shape (R, T) with R + T = n for a state held by one tile.
bool lds_shape(int n, int *R, int *T) {
    switch (n) {
    case 14: *R = 5; *T = 9; return true;
    case 13: *R = 5; *T = 8; return true;
    case 12: *R = 5; *T = 7; return true;
    case 11: *R = 4; *T = 7; return true;
    default: return false;
    }
}

// Schedule of one tile shape's entries (qubits n[i], pass count np[i],
// entry id ids[i]): per round, a segment per entry that has the pass, block
// offsets within the round, and the round's first work item.  A round is one
// launch: QSV_ERANGE above the blocks of one.
qsv_status make_schedule(const std::vector<int> &n, const std::vector<size_t> &np, const std::vector<uint32_t> &ids, int L,
                   std::vector<BatchRound> &rounds, std::vector<BatchSeg> &segs, std::vector<uint64_t> &round_blocks,
                   uint64_t &items) {
    size_t max_passes = 0;
    for (size_t x : np) max_passes = std::max(max_passes, x);
    items = 0;
    for (size_t r = 0; r < max_passes; ++r) {
        BatchRound rd{items, uint32_t(segs.size()), 0};
        uint64_t blocks = 0;
        for (size_t i = 0; i < n.size(); ++i) {
            if (np[i] <= r) continue;
            BatchSeg sg{};
            sg.start = blocks;
            sg.entry = ids[i];
            segs.push_back(sg);
            blocks += 1ull << (n[i] - L);
        }
        rd.nseg = uint32_t(segs.size()) - rd.seg_off;
        rounds.push_back(rd);
        if (blocks > kMaxBlocks) return fail(QSV_ERANGE, "sv_batch: too many tiles in one round");
        round_blocks.push_back(blocks);
        items += blocks;
    }
    return QSV_OK;
}

// Branch bits that a pass depends on.
uint64_t branch_bits(const PassProg &p) {
    uint64_t m = 0;
    for (int pc = 0; pc < p.n_ops; ++pc) {
        const uint64_t op = p.ops[pc];
        const uint32_t code = uint32_t(op & 0xff), b = uint32_t((op >> 16) & 0xff), c = uint32_t((op >> 24) & 0xff);
        if (code == OP_XCHG) ++pc;
        else if (code == OP_ZB || (code == OP_PROJ && c)) m |= 1ull << (b & 63);
    }
    return m;
}

// Values that the given bits take in the branches.
size_t distinct(const std::vector<uint64_t> &branches, uint64_t bits) {
    std::set<uint64_t> v;
    for (uint64_t x : branches) v.insert(x & bits);
    return v.size();
}

// Entries that differ in their branches only and start from the same state are
// the same state up to the first gate that takes the bits they differ in: it is
// computed once and read from there.  What bounds batched compiled passes is
// their arithmetic, so the gain is the gates not applied again; the cost are the
// launches added.  A plan that runs alone has to save a number of gates times
// tiles for that; beside other chains of launches, which fill the device as well,
// the batch needs tiles for three rounds of the workgroups that the CUs hold (two
// each).  Means of five processes, depth 14, us without and with:
//   alone         15 q x 66  16000 saved  36 / 32    18 q x 20  34000  42 / 47
//                 16 q x 66  40000        43 / 38    18 q x 33  66000  57 / 54
//                 15 q x 512 194000      100 / 78
//   side by side  2 x 130 of 15 q, 1040 tiles  87 / 96     2 x 16 of 18 q, 1024   77 / 82
//                 130 of 12 + 16 q, 1170       81 / 87     2 x 33 of 18 q, 2112  125 / 96
//                 2 x 100 of 16 q, 1600        95 / 91     2 x 512 of 15 q, 4096 193 / 162
// Not for states held by one tile: a pass over one of them is bound by the tile's
// own chain of ops, short enough already (14 q x 4096 393 / 388, 12 q x 4096 367 /
// 372, 2 x 1024 states of 12 q 221 / 228).
bool sharing_pays(double saved, uint64_t batch_tiles, bool alone) {
    return alone ? saved >= 40e3 : batch_tiles >= 3 * 512;
}

// Branch level at which the circuit is cut in two plans, so that the first one
// runs for few states: the cut with the fewest gates over all states, if that
// saves a quarter of them and pays; 0: none.
int shared_levels(const qsv_circuit &c, int lb, const std::vector<uint64_t> &branches, uint64_t tiles,
                  uint64_t batch_tiles, bool alone) {
    std::vector<int> lev;
    std::vector<uint64_t> bits;
    branch_levels(c, lev, bits);
    std::vector<double> gates(bits.size() + 1, 0.0);
    double total = 0, before = 0;
    for (size_t i = 0; i < lev.size(); ++i)
        if (c.gates[i].layer >= lb) ++gates[size_t(lev[i])], ++total;
    const double count = double(branches.size());
    double best = 0.75 * count * total;
    uint64_t known = 0;
    int cut = 0;
    for (size_t l = 1; l <= bits.size(); ++l) {
        before += gates[l - 1];
        if (l > 1) known |= bits[l - 2];
        if (before == 0 || before == total) continue;
        const double cost = double(distinct(branches, known)) * before + count * (total - before);
        if (cost < best) {
            best = cost;
            cut = int(l);
        }
    }
    return sharing_pays((count * total - best) * double(tiles), batch_tiles, alone) ? cut : 0;
}

// The launches of a compiled plan.  After pass p one state
// stands for the entries with the same values of the branch bits of passes 0..p:
// in scratch where max_scratch states are enough, otherwise that of the first
// entry.  Pass p + 1 reads it there for each of them, those that write elsewhere
// first, then those that overwrite what was read.  The last pass writes every
// entry.  A pass is shared when that halves its states or more.
void share_passes(const Plan &plan, const std::vector<uint64_t> &branches, bool share,
                  size_t max_scratch, std::vector<BatchRow> &rows, std::vector<BatchStep> &steps, size_t *scratch) {
    const size_t np = plan.passes.size(), count = branches.size();
    std::vector<std::vector<uint32_t>> first;  // per shared pass: the first entry with an entry's bits
    uint64_t bits = 0;
    size_t states = 0;
    for (size_t p = 0; share && p + 1 < np; ++p) {
        bits |= branch_bits(plan.passes[p].prog);
        std::map<uint64_t, uint32_t> rep;
        for (size_t i = 0; i < count; ++i) rep.emplace(branches[i] & bits, uint32_t(i));
        if (rep.size() * 2 > count) break;
        states = rep.size();
        first.emplace_back(count);
        for (size_t i = 0; i < count; ++i) first.back()[i] = rep[branches[i] & bits];
    }
    // where the first entries' states are (the last shared pass has them all)
    std::vector<uint32_t> slot(count);
    *scratch = states <= max_scratch ? states : 0;
    uint32_t used = 0;
    for (size_t i = 0; i < count; ++i)
        slot[i] = *scratch && first.back()[i] == i ? uint32_t(count) + used++ : uint32_t(i);
    std::vector<uint32_t> at(count), next(count);  // where an entry's state is, before and after the pass
    for (size_t i = 0; i < count; ++i) at[i] = first.empty() ? uint32_t(i) : slot[first[0][i]];
    for (size_t p = 0; p < np; ++p) {
        std::vector<BatchRow> away, in_place;
        for (size_t i = 0; i < count; ++i) {
            const bool shared = p < first.size();
            next[i] = shared ? slot[first[p][i]] : uint32_t(i);
            if (!shared || first[p][i] == i)
                (at[i] == next[i] ? in_place : away).push_back({uint32_t(i), next[i], at[i]});
        }
        // siblings side by side: they read the same tiles
        std::stable_sort(away.begin(), away.end(), [](const BatchRow &x, const BatchRow &y) { return x.src < y.src; });
        for (const auto *part : {&away, &in_place}) {
            if (part->empty()) continue;
            steps.push_back({p, rows.size(), part->size()});
            rows.insert(rows.end(), part->begin(), part->end());
        }
        at = next;
    }
}

// The circuit's plan from layer lb on in tile shape sh.  With cut > 0 the passes
// of the branch levels below it come before those of the others (each ends in
// the natural order of the qubits, so they follow one another); the plan's key
// then has a first layer of -cut (this only occurs with lb = 1).
qsv_status batch_plan(qsv_circuit *c, int lb, int cut, const TileShape &sh, std::shared_ptr<Plan> &p) {
    const PlanKey key{cut ? -cut : lb, -1, sh.R, sh.T, sh.c, false};
    {
        std::lock_guard<std::mutex> g(c->mu);
        auto pit = c->plans.find(key);
        if (pit != c->plans.end()) {
            p = pit->second;
            return QSV_OK;
        }
    }
    auto made = std::make_shared<Plan>();
    qsv_status st = QSV_OK;
    if (!cut) {
        st = build_plan(*c, lb, -1, sh, *made);
    } else {
        int levels = 0;
        st = circuit_branch_levels(c, &levels, nullptr, 0);
        for (int part = 0; part < 2 && st == QSV_OK; ++part) {
            qsv_circuit *out = nullptr;
            st = circuit_branch_stage(c, part ? cut : 0, part ? levels + 1 : cut, &out);
            if (st != QSV_OK) break;
            const std::unique_ptr<qsv_circuit, void (*)(qsv_circuit *)> stage(out, circuit_destroy);
            Plan half;
            st = build_plan(*stage, lb, -1, sh, part ? half : *made);
            for (Pass &pass : half.passes) made->passes.push_back(std::move(pass));
        }
    }
    if (st != QSV_OK) return st;
    std::lock_guard<std::mutex> g(c->mu);
    p = c->plans.emplace(key, made).first->second;
    return QSV_OK;
}

// Plans and device tables for layers [lb, end) of every entry.
qsv_status build_tables(qsv_batch *b, int lb) {
    drop_graph(b);
    free_tables(b);
    b->built_lb = -1;  // nothing is there until all of it is
    b->plans.clear();
    b->entry_plan.assign(b->circs.size(), 0);
    std::map<const qsv_circuit *, uint32_t> idx;
    std::map<const qsv_circuit *, std::vector<uint64_t>> sharers;  // the branches of each circuit
    for (size_t i = 0; i < b->circs.size(); ++i) sharers[b->circs[i]].push_back(b->branches[i]);
    std::vector<qsv_circuit *> circuits;  // of the plans
    std::vector<TileShape> plan_shape;
    for (size_t i = 0; i < b->circs.size(); ++i) {
        auto it = idx.find(b->circs[i]);
        if (it == idx.end()) {
            qsv_circuit *c = const_cast<qsv_circuit *>(b->circs[i]);
            TileShape sh{b->R, b->T, b->c};
            int lr = 0, lt = 0;
            if (big_state(b, c->n)) {
                // states of the HBM-streaming class get their own compiled
                // kernels with the single-state default tile shape
                sh = default_shape(c->n);
                const qsv_status shape_st = compiled_default_shape(c, lb, -1, 0, false, false, sh);
                if (shape_st != QSV_OK) return shape_st;
                // the autotuned shape of this circuit (sv_tune / sv_tune_set), if any
                qsv_fuse_opts t;
                if (tuned_opts(c, lb, -1, &t) && t.reg_qubits > 0 && t.thread_qubits > 0 &&
                    compiled_shape_supported(t.reg_qubits, t.thread_qubits) &&
                    t.reg_qubits + t.thread_qubits <= c->n) {
                    sh.R = t.reg_qubits;
                    sh.T = t.thread_qubits;
                    sh.c = t.low_qubits > 0 ? t.low_qubits : std::min(5, sh.T + 1);
                }
            } else if (!b->forced_shape && c->n <= kLdsState && lds_shape(c->n, &lr, &lt)) {
                sh = TileShape{lr, lt, std::min(5, lt + 1)};
            } else if (!b->forced_shape && b->jit_mode >= 0 &&
                       (b->jit_mode > 0 || sharers[c].size() >= kSharedPlan)) {
                // compiled passes over many states fill the device anyway, and
                // the larger tile has fewer exchanges (2 x 1024 branch states
                // of 15 qubits, nothing shared: 315 us against 387 us on (4, 8,
                // 4)).  A tile of 2^15 amplitudes, the whole state, is no faster
                // with shared prefixes (2 x 1024: 266 us, 258 on (5, 8, 5); 350
                // states: 85 and 63).
                sh = TileShape{5, 8, b->low ? b->low : 5};
            }
            it = idx.emplace(b->circs[i], uint32_t(circuits.size())).first;
            circuits.push_back(c);
            plan_shape.push_back(sh);
        }
        b->entry_plan[i] = it->second;
    }
    uint64_t batch_tiles = 0;
    for (size_t p = 0; p < circuits.size(); ++p)
        batch_tiles += uint64_t(sharers[circuits[p]].size()) << (circuits[p]->n - plan_shape[p].R - plan_shape[p].T);
    std::vector<int> plan_cut;
    for (size_t p = 0; p < circuits.size(); ++p) {
        qsv_circuit *c = circuits[p];
        const TileShape &sh = plan_shape[p];
        const std::vector<uint64_t> &branches = sharers[c];
        const uint64_t tiles = 1ull << (c->n - sh.R - sh.T);
        // from layer 1 on the run starts every entry from |+>^n
        const bool may = lb == 1 && tiles > 1 && compiled(b, c->n, branches.size());
        const int cut = may ? shared_levels(*c, lb, branches, tiles, batch_tiles, circuits.size() == 1) : 0;
        std::shared_ptr<Plan> plan;
        const qsv_status st = batch_plan(c, lb, cut, sh, plan);
        if (st != QSV_OK) return st;
        b->plans.push_back(plan);
        plan_cut.push_back(cut);
    }
    b->group.assign(b->plans.size(), {});
    for (size_t i = 0; i < b->circs.size(); ++i) b->group[b->entry_plan[i]].push_back(uint32_t(i));
    b->plan_jit.assign(b->plans.size(), 0);
    b->d_group_ents.assign(b->plans.size(), nullptr);
    b->d_scratch.assign(b->plans.size(), nullptr);
    b->rows.assign(b->plans.size(), {});
    b->steps.assign(b->plans.size(), {});
    size_t left = kShareScratch;
    for (size_t p = 0; p < b->plans.size(); ++p) {
        const Plan &plan = *b->plans[p];
        b->plan_jit[p] = !plan.passes.empty() && compiled(b, plan.n, b->group[p].size());
        if (b->plan_jit[p]) {
            std::vector<uint64_t> branches;
            for (uint32_t i : b->group[p]) branches.push_back(b->branches[i]);
            const bool share = plan_cut[p] > 0;
            const size_t bytes = sizeof(float2) << plan.n;
            size_t scratch = 0;
            share_passes(plan, branches, share, std::min(kPlanScratch, left) / bytes, b->rows[p], b->steps[p], &scratch);
            if (scratch && hipMalloc(reinterpret_cast<void **>(&b->d_scratch[p]), scratch * bytes) != hipSuccess) {
                (void)hipGetLastError();  // then in the entries' own states
                b->d_scratch[p] = nullptr;
                b->rows[p].clear();
                b->steps[p].clear();
                share_passes(plan, branches, share, 0, b->rows[p], b->steps[p], &scratch);
            }
            left -= scratch * bytes;
            hipError_t e = hipMalloc(reinterpret_cast<void **>(&b->d_group_ents[p]),
                                     b->rows[p].size() * sizeof(BatchEntry));
            if (e != hipSuccess) return fail(QSV_ENOMEM, "sv_batch: group entry table");
        }
    }
    // program array of the generic kernel's plans
    std::vector<GenProg> progs;
    std::vector<uint32_t> prog0(b->plans.size(), 0), prog_count(b->plans.size(), 0);
    for (size_t p = 0; p < b->plans.size(); ++p) {
        if (b->plan_jit[p]) continue;
        std::shared_ptr<const std::vector<GenProg>> g;
        const qsv_status st = generic_programs(*b->plans[p], false, g);
        if (st != QSV_OK) return st;
        prog0[p] = uint32_t(progs.size());
        prog_count[p] = uint32_t(g->size());
        progs.insert(progs.end(), g->begin(), g->end());
    }
    // entries
    b->h_ents.assign(b->circs.size(), BatchEntry{});
    for (size_t i = 0; i < b->circs.size(); ++i) {
        BatchEntry &e = b->h_ents[i];
        e.amps = nullptr;
        e.branch = b->branches[i];
        e.prog0 = prog0[b->entry_plan[i]];
        e.n = uint32_t(b->circs[i]->n);
        e.init_val = float(std::pow(2.0, -0.5 * e.n));
    }
    // generic-kernel entries by tile shape: segments of every program round
    std::map<std::pair<int, int>, size_t> shape_of;
    for (size_t i = 0; i < b->circs.size(); ++i) {
        const uint32_t p = b->entry_plan[i];
        if (b->plan_jit[p] || b->plans[p]->passes.empty()) continue;
        const auto key = std::make_pair(plan_shape[p].R, plan_shape[p].T);
        auto it = shape_of.find(key);
        if (it == shape_of.end()) {
            it = shape_of.emplace(key, b->shapes.size()).first;
            BatchShape bs;
            bs.R = plan_shape[p].R;
            bs.T = plan_shape[p].T;
            bs.c = plan_shape[p].c;
            b->shapes.push_back(bs);
        }
        b->shapes[it->second].entries.push_back(uint32_t(i));
    }
    std::vector<std::vector<BatchSeg>> shape_segs(b->shapes.size());
    for (size_t k = 0; k < b->shapes.size(); ++k) {
        BatchShape &bs = b->shapes[k];
        std::vector<int> nq;
        std::vector<size_t> np;
        for (uint32_t i : bs.entries) {
            nq.push_back(b->circs[i]->n);
            np.push_back(prog_count[b->entry_plan[i]]);
        }
        std::vector<BatchRound> rounds;
        uint64_t items = 0;
        const qsv_status st =
            make_schedule(nq, np, bs.entries, bs.R + bs.T, rounds, shape_segs[k], bs.round_blocks, items);
        if (st != QSV_OK) return st;
        for (const BatchRound &rd : rounds) {
            bs.round_seg_off.push_back(int(rd.seg_off));
            bs.round_nseg.push_back(int(rd.nseg));
        }
    }
    hipError_t e;
    if (!progs.empty()) {
        e = hipMalloc(reinterpret_cast<void **>(&b->d_progs), progs.size() * sizeof(GenProg));
        if (e != hipSuccess) return fail(QSV_ENOMEM, "sv_batch: program table");
        e = hipMemcpy(b->d_progs, progs.data(), progs.size() * sizeof(GenProg), hipMemcpyHostToDevice);
        if (e != hipSuccess) return hipfail(e, "sv_batch: program upload");
    }
    e = hipMalloc(reinterpret_cast<void **>(&b->d_ents), b->h_ents.size() * sizeof(BatchEntry));
    if (e != hipSuccess) return fail(QSV_ENOMEM, "sv_batch: entry table");
    // one block for the segments of every shape
    size_t bytes = 0;
    std::vector<size_t> off_s(b->shapes.size());
    for (size_t k = 0; k < b->shapes.size(); ++k) {
        off_s[k] = bytes;
        bytes += (shape_segs[k].size() * sizeof(BatchSeg) + 255) & ~size_t(255);
    }
    if (bytes) {
        e = hipMalloc(&b->d_tabs, bytes);
        if (e != hipSuccess) return fail(QSV_ENOMEM, "sv_batch: schedule tables");
        std::vector<char> h(bytes, 0);
        for (size_t k = 0; k < b->shapes.size(); ++k) {
            if (!shape_segs[k].empty())
                std::memcpy(h.data() + off_s[k], shape_segs[k].data(), shape_segs[k].size() * sizeof(BatchSeg));
            b->shapes[k].d_segs = reinterpret_cast<BatchSeg *>(static_cast<char *>(b->d_tabs) + off_s[k]);
        }
        e = hipMemcpy(b->d_tabs, h.data(), bytes, hipMemcpyHostToDevice);
        if (e != hipSuccess) return hipfail(e, "sv_batch: schedule upload");
    }
    b->built_lb = lb;
    b->g_ptrs.clear();
    return QSV_OK;
}

}  // namespace
}  // namespace qsv

using namespace qsv;

extern "C" {

qsv_status sv_batch_create(const qsv_circuit *const *circs, const uint64_t *branch_ids,
                           size_t count, const qsv_fuse_opts *opts, qsv_batch **out) {
    if (!out) return fail(QSV_EINVAL, "sv_batch_create: out is null");
    *out = nullptr;
    if (!circs || count == 0) return fail(QSV_EINVAL, "sv_batch_create: no entries");
    if (count > (1u << 24)) return fail(QSV_ERANGE, "sv_batch_create: too many entries");
    int nmin = 64;
    for (size_t i = 0; i < count; ++i) {
        if (!circs[i]) return fail(QSV_EINVAL, "sv_batch_create: null circuit");
        if (circs[i]->n > kMaxQubits) return fail(QSV_ERANGE, "sv_batch_create: n > 34");
        nmin = std::min(nmin, circs[i]->n);
    }
    auto b = std::unique_ptr<qsv_batch>(new qsv_batch);
    if (nmin < kBatchMinQubits) return fail(QSV_EUNSUPPORTED, "sv_batch_create: states need >= 11 qubits");
    // generic-kernel tile shape of the states that one tile cannot hold
    // (the LDS class has a shape per qubit count); opts may force one shape
    // for every generic entry
    b->R = 4;  // see default_shape
    b->T = 8;
    if (opts && opts->reg_qubits && opts->thread_qubits) {
        b->R = opts->reg_qubits;
        b->T = opts->thread_qubits;
        b->forced_shape = true;
        const bool ok = (b->R == 5 && (b->T == 9 || b->T == 8 || b->T == 7)) || (b->R == 4 && (b->T == 8 || b->T == 7));
        if (!ok) return fail(QSV_EUNSUPPORTED, "sv_batch_create: no batch kernel for this tile shape");
        if (b->R + b->T > nmin) return fail(QSV_EUNSUPPORTED, "sv_batch_create: tile larger than a state");
    }
    b->low = opts ? opts->low_qubits : 0;
    b->c = b->low ? b->low : b->forced_shape ? std::min(5, b->T + 1) : 4;
    b->jit_mode = opts ? opts->jit : 0;
    // There is no persistent launch (its kernel did not finish on the device):
    // asking for it is refused and every batch runs one launch per round.
    if (const char *v = std::getenv("QSV_BATCH_PERSISTENT"))
        if (v[0] != '0')
            return fail(QSV_EUNSUPPORTED, "sv_batch_create: the persistent batch launch is switched off");
    b->circs.assign(circs, circs + count);
    b->branches.assign(count, 0);
    if (branch_ids) b->branches.assign(branch_ids, branch_ids + count);
    // set kernel attributes outside any capture
    hipError_t e = hipSuccess;
    static const int kShapes[][2] = {{5, 9}, {5, 8}, {4, 8}, {5, 7}, {4, 7}};
    for (auto &sh : kShapes)
        if (e == hipSuccess) e = launch_tile_batch(sh[0], sh[1], nullptr, 0, nullptr, nullptr, 0, 0, 0, true, nullptr);
    if (e != hipSuccess) return fail(QSV_EHIP, std::string("sv_batch_create: ") + hipGetErrorString(e));
    e = hipStreamCreateWithFlags(&b->cap, hipStreamNonBlocking);
    if (e != hipSuccess) return fail(QSV_EHIP, "sv_batch_create: capture stream");
    *out = b.release();
    return QSV_OK;
}

qsv_status sv_batch_run(qsv_batch *b, void *const *amps_dev, int init_plus,
                        const uint64_t *bitstrings_dev, size_t m, void *amp_table_dev,
                        void *stream) {
    if (!b || !amps_dev) return fail(QSV_EINVAL, "sv_batch_run: null argument");
    if (m && (!bitstrings_dev || !amp_table_dev))
        return fail(QSV_EINVAL, "sv_batch_run: null gather buffer");
    const size_t count = b->circs.size();
    for (size_t i = 0; i < count; ++i) {
        if (!amps_dev[i]) return fail(QSV_EINVAL, "sv_batch_run: null state pointer");
        if (reinterpret_cast<uintptr_t>(amps_dev[i]) % 16)
            return fail(QSV_EINVAL, "sv_batch_run: state pointer not 16-byte aligned");
    }
    const int lb = init_plus ? 1 : 0;
    qsv_status st;
    if (b->built_lb != lb && (st = build_tables(b, lb)) != QSV_OK) return st;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const bool same = b->exec && b->g_init == (init_plus ? 1 : 0) && b->g_bits == bitstrings_dev &&
                      b->g_m == m && b->g_table == amp_table_dev && b->g_ptrs.size() == count &&
                      std::equal(b->g_ptrs.begin(), b->g_ptrs.end(), amps_dev);
    if (!same) {
        drop_graph(b);
        for (size_t i = 0; i < count; ++i) b->h_ents[i].src = b->h_ents[i].amps = amps_dev[i];
        // the previous graph may still read the entry table
        hipError_t e = hipStreamSynchronize(s);
        if (e != hipSuccess) return hipfail(e, "sv_batch_run");
        e = hipMemcpy(b->d_ents, b->h_ents.data(), count * sizeof(BatchEntry), hipMemcpyHostToDevice);
        if (e != hipSuccess) return hipfail(e, "sv_batch_run: entry upload");
        const int variant = kJitBatched | (init_plus ? (kJitInit | QSV_INIT_PLUS) : 0);
        std::vector<size_t> jp;
        for (size_t p = 0; p < b->plans.size(); ++p) {
            if (!b->plan_jit[p]) continue;
            std::vector<BatchEntry> ge;
            for (const BatchRow &r : b->rows[p]) {
                const auto state = [&](uint32_t k) -> void * {
                    const size_t own = b->group[p].size();
                    return k < own ? amps_dev[b->group[p][k]]
                                   : b->d_scratch[p] + ((k - own) * sizeof(float2) << b->plans[p]->n);
                };
                ge.push_back(b->h_ents[b->group[p][r.entry]]);
                ge.back().amps = state(r.dst);
                ge.back().src = state(r.src);
            }
            e = hipMemcpy(b->d_group_ents[p], ge.data(), ge.size() * sizeof(BatchEntry),
                          hipMemcpyHostToDevice);
            if (e != hipSuccess) return hipfail(e, "sv_batch_run: group entry upload");
            jp.push_back(p);
        }
        // compile the plans' kernels concurrently
        {
            int dev = 0;
            if ((e = hipGetDevice(&dev)) != hipSuccess) return hipfail(e, "sv_batch_run");
            const unsigned nth = std::max(1u, std::min<unsigned>(16, std::thread::hardware_concurrency()));
            std::atomic<size_t> next{0};
            std::vector<qsv_status> res(jp.size(), QSV_OK);
            std::vector<std::thread> pool;
            for (unsigned w = 0; w < std::min<size_t>(nth, jp.size()); ++w)
                pool.emplace_back([&, dev] {
                    (void)hipSetDevice(dev);
                    for (size_t k; (k = next++) < jp.size();) {
                        std::lock_guard<std::mutex> g(b->plans[jp[k]]->jit_mu);
                        res[k] = jit_prepare(*b->plans[jp[k]], variant);
                    }
                });
            for (auto &th : pool) th.join();
            for (qsv_status r : res)
                if (r != QSV_OK) return fail(r, "sv_batch_run: compiling pass kernels failed");
        }
        // chains of launches: the passes of a compiled plan, the rounds of a
        // tile shape; compiled ones first, then by work
        struct Chain {
            double work;
            size_t plan, shape;  // shape == ~0: compiled plan
        };
        std::vector<Chain> chains;
        for (size_t p : jp) chains.push_back({std::ldexp(double(b->rows[p].size()), b->plans[p]->n), p, ~size_t(0)});
        for (size_t k = 0; k < b->shapes.size(); ++k) {
            double blocks = 0;
            for (uint64_t x : b->shapes[k].round_blocks) blocks += double(x);
            // an interpreted pass costs about twice a compiled one
            chains.push_back({2.0 * std::ldexp(blocks, b->shapes[k].R + b->shapes[k].T), 0, k});
        }
        std::stable_sort(chains.begin(), chains.end(), [](const Chain &x, const Chain &y) {
            const bool xs = x.shape != ~size_t(0), ys = y.shape != ~size_t(0);
            return xs != ys ? ys : x.work > y.work;
        });
        // the side streams and their events (below), made before the first
        // capture that has two chains to run side by side
        if (chains.size() > 1 && b->lanes.empty()) {
            e = hipEventCreateWithFlags(&b->fork, hipEventDisableTiming);
            for (int k = 0; k < kLanes && e == hipSuccess; ++k) {
                hipStream_t ls = nullptr;
                hipEvent_t je = nullptr;
                if ((e = hipStreamCreateWithFlags(&ls, hipStreamNonBlocking)) != hipSuccess) break;
                if ((e = hipEventCreateWithFlags(&je, hipEventDisableTiming)) != hipSuccess) {
                    hipStreamDestroy(ls);
                    break;
                }
                b->lanes.push_back(ls);
                b->lane_done.push_back(je);
            }
            if (e != hipSuccess) return hipfail(e, "sv_batch_run: side streams");
        }
        e = hipStreamBeginCapture(b->cap, hipStreamCaptureModeThreadLocal);
        if (e != hipSuccess) return hipfail(e, "sv_batch_run: begin capture");
        hipError_t le = hipSuccess;
        // The chains go to the capture stream and the side streams, each to the
        // least loaded one, so the graph holds them as parallel branches and
        // small states do not leave the device idle one after another (40
        // circuits of 12..16 qubits, four tile shapes: 173 -> 79 us).
        size_t joined = 0;  // side streams that joined the capture
        if (chains.size() > 1 && !b->lanes.empty()) {
            le = hipEventRecord(b->fork, b->cap);
            while (le == hipSuccess && joined < b->lanes.size()) {
                le = hipStreamWaitEvent(b->lanes[joined], b->fork, 0);
                if (le == hipSuccess) ++joined;
            }
        }
        std::vector<double> load(joined + 1, 0.0);  // the last one: the capture stream
        for (const Chain &ch : chains) {
            if (le != hipSuccess) break;
            // beside compiled chains the capture stream is kept for the tile
            // shapes, whose launches are the many short ones (32 circuits of
            // 14..24 qubits: 835 us; spread over all streams 872)
            size_t k = size_t(std::min_element(load.begin(), load.end()) - load.begin());
            if (!jp.empty() && joined)
                k = ch.shape != ~size_t(0)
                        ? joined
                        : size_t(std::min_element(load.begin(), load.end() - 1) - load.begin());
            const hipStream_t ls = k < joined ? b->lanes[k] : b->cap;
            load[k] += ch.work;
            if (ch.shape == ~size_t(0)) {
                for (const BatchStep &sp : b->steps[ch.plan])
                    if (le == hipSuccess &&
                        jit_launch_batched(*b->plans[ch.plan], variant, sp.pass, b->d_group_ents[ch.plan] + sp.first,
                                           unsigned(sp.count), ls) != QSV_OK)
                        le = hipErrorLaunchFailure;
                continue;
            }
            const BatchShape &bs = b->shapes[ch.shape];
            for (size_t r = 0; r < bs.round_blocks.size() && le == hipSuccess; ++r)
                le = launch_tile_batch(bs.R, bs.T, bs.d_segs + bs.round_seg_off[r], bs.round_nseg[r], b->d_ents,
                                       b->d_progs, int(r), bs.round_blocks[r], init_plus ? 1 : 0, jp.empty(), ls);
        }
        // join every side stream back (also after an error: the capture
        // must end with all of them joined)
        for (size_t k = 0; k < joined; ++k) {
            hipError_t je = hipEventRecord(b->lane_done[k], b->lanes[k]);
            if (je == hipSuccess) je = hipStreamWaitEvent(b->cap, b->lane_done[k], 0);
            if (le == hipSuccess) le = je;
        }
        if (le == hipSuccess && m)
            le = launch_gather_batch(b->d_ents, count, bitstrings_dev, m,
                                     static_cast<float2 *>(amp_table_dev), b->cap);
        hipGraph_t g = nullptr;
        e = hipStreamEndCapture(b->cap, &g);
        if (le != hipSuccess) {
            if (g) hipGraphDestroy(g);
            return hipfail(le, "sv_batch_run: launch during capture");
        }
        if (e != hipSuccess) return hipfail(e, "sv_batch_run: end capture");
        e = hipGraphInstantiate(&b->exec, g, nullptr, nullptr, 0);
        hipGraphDestroy(g);
        if (e != hipSuccess) return hipfail(e, "sv_batch_run: instantiate");
        b->g_ptrs.assign(amps_dev, amps_dev + count);
        b->g_init = init_plus ? 1 : 0;
        b->g_bits = bitstrings_dev;
        b->g_m = m;
        b->g_table = amp_table_dev;
    }
    hipError_t e = hipGraphLaunch(b->exec, s);
    if (e != hipSuccess) return hipfail(e, "sv_batch_run: graph launch");
    return QSV_OK;
}

qsv_status sv_batch_status(qsv_batch *b, void *stream) {
    if (!b) return fail(QSV_EINVAL, "sv_batch_status: null batch");
    const hipError_t e = hipStreamSynchronize(static_cast<hipStream_t>(stream));
    return e == hipSuccess ? QSV_OK : hipfail(e, "sv_batch_status");
}

qsv_status sv_batch_abort(qsv_batch *b) {
    if (!b) return fail(QSV_EINVAL, "sv_batch_abort: null batch");
    return QSV_OK;  // no launch of a batch waits on another one
}

// Host emulation of a persistent launch's schedule (CPU check of the
// ordering rule; no product entry point calls it): `workers` virtual
// workgroups take the work items in order, an item of round r > 0 waits
// until its entry has completed r * tiles items, and a random running item
// completes at each step (planted_early_start != 0: a deliberately wrong
// rule that lets an item start one tile early, for the test that the check
// catches it).  Fails if the emulation stalls, if an item starts
// before every tile of its entry's earlier passes completed, or if some
// (entry, pass, tile) is not run exactly once.
qsv_status sv_debug_batch_schedule(const int *n_qubits, const int *passes, size_t count, int tile_qubits,
                                   int workers, uint64_t seed, int planted_early_start, uint64_t *items_out) {
    if (!n_qubits || !passes || count == 0 || workers <= 0 || tile_qubits <= 0)
        return fail(QSV_EINVAL, "sv_debug_batch_schedule: bad argument");
    std::vector<int> nq(n_qubits, n_qubits + count);
    std::vector<size_t> np(passes, passes + count);
    std::vector<uint32_t> ids(count);
    for (size_t i = 0; i < count; ++i) {
        if (nq[i] < tile_qubits || nq[i] > 30 || passes[i] < 0)
            return fail(QSV_EINVAL, "sv_debug_batch_schedule: state size out of range");
        ids[i] = uint32_t(i);
    }
    std::vector<BatchRound> rounds;
    std::vector<BatchSeg> segs;
    std::vector<uint64_t> blocks;
    uint64_t items = 0;
    const qsv_status st = make_schedule(nq, np, ids, tile_qubits, rounds, segs, blocks, items);
    if (st != QSV_OK) return st;
    if (items_out) *items_out = items;
    std::vector<uint64_t> done(count, 0);
    std::vector<std::vector<uint64_t>> runs(count);  // per entry: times each (pass, tile) ran
    for (size_t i = 0; i < count; ++i) runs[i].assign(np[i] << (nq[i] - tile_qubits), 0);
    struct W { bool busy = false, running = false; int r = 0; uint32_t e = 0; uint64_t t = 0; };
    std::vector<W> w(static_cast<size_t>(workers));
    uint64_t next = 0, rng = seed | 1;
    auto rnd = [&rng]() { rng ^= rng << 13; rng ^= rng >> 7; rng ^= rng << 17; return rng; };
    uint64_t finished = 0;
    while (finished < items) {
        bool progress = false;
        for (W &x : w) {  // take items, start those whose dependency holds
            if (!x.busy && next < items) {
                batch_decode(rounds.data(), int(rounds.size()), segs.data(), next++, &x.r, &x.e, &x.t);
                x.busy = true;
                x.running = false;
                progress = true;
            }
            const uint64_t need = uint64_t(x.r) << (nq[x.e] - tile_qubits);
            if (x.busy && !x.running && done[x.e] + (planted_early_start && need ? 1 : 0) >= need) {
                // every tile of the earlier passes has completed, none of this one yet started early
                for (int r2 = 0; r2 < x.r; ++r2)
                    for (uint64_t t2 = 0; t2 < (1ull << (nq[x.e] - tile_qubits)); ++t2)
                        if (runs[x.e][(uint64_t(r2) << (nq[x.e] - tile_qubits)) + t2] != 1)
                            return fail(QSV_EINTERNAL, "schedule: an item started before its dependency");
                x.running = true;
                progress = true;
            }
        }
        std::vector<size_t> run_idx;
        for (size_t k = 0; k < w.size(); ++k)
            if (w[k].running) run_idx.push_back(k);
        if (run_idx.empty()) {
            if (!progress) return fail(QSV_EINTERNAL, "schedule: the emulated launch stalls");
            continue;
        }
        W &x = w[run_idx[rnd() % run_idx.size()]];
        if (x.r >= int(np[x.e]) || x.t >= (1ull << (nq[x.e] - tile_qubits)))
            return fail(QSV_EINTERNAL, "schedule: decoded item out of range");
        ++runs[x.e][(uint64_t(x.r) << (nq[x.e] - tile_qubits)) + x.t];
        ++done[x.e];
        ++finished;
        x.busy = x.running = false;
    }
    for (size_t i = 0; i < count; ++i)
        for (uint64_t v : runs[i])
            if (v != 1) return fail(QSV_EINTERNAL, "schedule: an item ran other than once");
    return QSV_OK;
}

void sv_batch_destroy(qsv_batch *b) {
    if (!b) return;
    drop_graph(b);
    free_tables(b);
    if (b->cap) hipStreamDestroy(b->cap);
    for (hipStream_t ls : b->lanes) hipStreamDestroy(ls);
    for (hipEvent_t ev : b->lane_done) hipEventDestroy(ev);
    if (b->fork) hipEventDestroy(b->fork);
    delete b;
}

}  // extern "C"
