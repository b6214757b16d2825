// Planner of the tile passes (host only; kernel in tile.hip).
//
// Two levels. A pass takes T qubits of the state (the lowest ones always
// among them) and every gate that can be applied while only those are at
// hand; a stage of the pass takes four of them (the register qubits) and
// every gate of the pass that needs no others. Both levels scan the gates
// left in circuit order: a gate is taken if the qubits it needs are there and
// it commutes with every gate skipped so far. Two gates commute when on each
// qubit they share both are diagonal, as controls, phases and CZ are.
//
// A gate needs at hand only the qubits it is not diagonal on. Diagonal gates
// need none: their phases wait as terms (index mask, index values, phase)
// and are applied just before the next gate that does not commute with them,
// when one of their qubits is a register qubit anyway.
#include "tile.h"

#include <algorithm>
#include <cmath>
#include <complex>
#include <cstring>
#include <initializer_list>

#include "qs_internal.h"

namespace qs {
namespace {

enum Kind { kOne, kRotation, kTwo, kSwap, kDiagonal, kAlone, kNothing };

typedef std::complex<long double> Phase;

// Products and quotients as they are: the operators look for infinities in
// every one and scale every quotient, which took a third of the planning.
Phase times(const Phase &a, const Phase &b)
{
    return Phase(a.real() * b.real() - a.imag() * b.imag(), a.real() * b.imag() + a.imag() * b.real());
}
Phase over(const Phase &a, const Phase &b)
{
    const long double n = b.real() * b.real() + b.imag() * b.imag();
    return Phase((a.real() * b.real() + a.imag() * b.imag()) / n, (a.imag() * b.real() - a.real() * b.imag()) / n);
}

struct TGate {
    int kind = kAlone;
    bool x = false;            // kOne: exactly X
    uint64_t need = 0;         // qubits the gate is not diagonal on
    uint64_t diag = 0;         // qubits it is diagonal on
    uint64_t cvals = 0;        // kOne: control values (mask: diag)
    int target[2] = {0, 0};    // kOne, kRotation, kTwo, kSwap
    double m[8] = {0};         // kOne
    double r[4] = {0};         // kRotation: diag(a0, a0 after) r diag(1, before)
    Phase before, after, a0;
    const double *mat = nullptr;
    const int *targets = nullptr;
    int k = 0;
    uint64_t cmask = 0, cv = 0;
};

struct Term {
    uint64_t mask = 0, vals = 0;
    Phase p;
};

uint64_t word_of(double v)
{
    uint64_t w;
    std::memcpy(&w, &v, sizeof w);
    return w;
}

// A two-qubit matrix that is a one-qubit gate under a control (CNOT or CZ
// given as a 4 x 4 matrix): control bit t of the local index, value v, acts
// as the 2 x 2 matrix on the other bit and as the identity where the control
// differs.
bool as_controlled(const double *m, int &ctrl, int &val, double *u)
{
    auto at = [&](int r, int c) { return m + 2 * (4 * r + c); };
    for (ctrl = 0; ctrl < 2; ++ctrl)
        for (val = 0; val < 2; ++val) {
            bool ok = true;
            for (int r = 0; r < 4 && ok; ++r)
                for (int c = 0; c < 4 && ok; ++c) {
                    const int rb = (r >> ctrl) & 1, cb = (c >> ctrl) & 1;
                    const double *e = at(r, c);
                    if (rb != cb) ok = e[0] == 0.0 && e[1] == 0.0;
                    else if (rb != val) ok = e[0] == (r == c ? 1.0 : 0.0) && e[1] == 0.0;
                }
            if (!ok) continue;
            for (int r = 0; r < 2; ++r)
                for (int c = 0; c < 2; ++c) {
                    const int o = 1 - ctrl;
                    const double *e = at((val << ctrl) | (r << o), (val << ctrl) | (c << o));
                    u[2 * (2 * r + c)] = e[0];
                    u[2 * (2 * r + c) + 1] = e[1];
                }
            return true;
        }
    return false;
}

// A unitary one-qubit gate as a real matrix (all but a rotation) between
// phases. False where an entry is further from one than a few roundings of
// its own (it may be any matrix, of any scale): of random unitaries, whose
// entries have rounding errors of the whole matrix's size, 7 in 1000. Every
// entry keeps its own modulus, so that what rounding left of the gate's norms
// stays as given: over some hundred gates whose norms are off to the same
// side it would add up.
bool as_rotation(TGate &g)
{
    Phase u[4], a[4];
    for (int i = 0; i < 4; ++i) {
        u[i] = Phase(g.m[2 * i], g.m[2 * i + 1]);
        g.r[i] = std::hypot(g.m[2 * i], g.m[2 * i + 1]);
        if (g.r[i] == 0) return false;
        a[i] = u[i] / (long double)(g.r[i]);
    }
    g.r[1] = -g.r[1];
    g.a0 = a[0];
    g.after = over(a[2], a[0]);
    // the second column's phase, from both of its entries by their weight
    const Phase b = over(a[3], a[2]) * (long double)(g.r[3] * g.r[3]) -
                    over(a[1], a[0]) * (long double)(g.r[1] * g.r[1]);
    g.before = b / std::sqrt(std::norm(b));
    auto near = [&](const Phase &p, int i) {
        return std::norm(times(p, g.before) * (long double)(g.r[i]) - u[i]) <= 4e-30L * std::norm(u[i]);
    };
    return near(a[0], 1) && near(a[2], 3);
}

void read_gate(int k, const int *targets, const double *m, uint64_t cmask, uint64_t cvals, TGate &g)
{
    GateDesc d;
    classify(m, k, d);
    uint64_t tm = 0;
    for (int i = 0; i < k; ++i) tm |= 1ull << targets[i];
    g.mat = m;
    g.targets = targets;
    g.k = k;
    g.cmask = cmask;
    g.cv = cvals;
    if (d.cls == GC_IDENTITY) {
        g.kind = kNothing;
        return;
    }
    if (d.cls == GC_PHASE1 || d.cls == GC_DIAG) {
        g.kind = kDiagonal;
        g.diag = tm | cmask;
        return;
    }
    g.need = tm;
    g.diag = cmask;
    g.cvals = cvals;
    if (k == 1) {
        g.kind = kOne;
        g.target[0] = targets[0];
        std::copy_n(m, 8, g.m);
    } else if (k == 2 && cmask == 0) {
        int ctrl, val;
        g.target[0] = targets[0];
        g.target[1] = targets[1];
        if (as_controlled(m, ctrl, val, g.m)) {
            g.kind = kOne;
            g.target[0] = targets[1 - ctrl];
            g.need = 1ull << targets[1 - ctrl];
            g.diag = 1ull << targets[ctrl];
            g.cvals = val ? g.diag : 0;
        } else {
            static const double sw[32] = {1, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 1, 0, 0, 0,
                                          0, 0, 1, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 1, 0};
            g.kind = std::equal(m, m + 32, sw) ? kSwap : kTwo;
        }
    }
    if (g.kind == kOne) {
        static const double xm[8] = {0, 0, 1, 0, 1, 0, 0, 0};
        g.x = std::equal(g.m, g.m + 8, xm);
        if (!g.x && !g.diag && as_rotation(g)) g.kind = kRotation;
    }
}

void add_terms(const TGate &g, std::vector<Term> &out)
{
    const int D = 1 << g.k;
    uint64_t tm = 0;
    for (int i = 0; i < g.k; ++i) tm |= 1ull << g.targets[i];
    for (int j = 0; j < D; ++j) {
        const double pr = g.mat[2 * (size_t(j) * D + j)], pi = g.mat[2 * (size_t(j) * D + j) + 1];
        if (pr == 1.0 && pi == 0.0) continue;
        uint64_t v = g.cv;
        for (int i = 0; i < g.k; ++i)
            if ((j >> i) & 1) v |= 1ull << g.targets[i];
        out.push_back(Term{tm | g.cmask, v, Phase(pr, pi)});
    }
}

// Gates not applied yet, in circuit order from `front`. A scan of them ends
// where nothing behind can be taken any more, and what it took is closed up
// in the part it saw, so planning takes time in proportion to the gates
// (random layers, 25 qubits complex128, 9,472 and 75,776 gates: 17 and 139
// ms, a fifth less than before the phases' arithmetic was made lighter; scans
// to the end of the circuit took 33 and 2,015 ms).
struct GateList {
    std::vector<int> ids;
    size_t front = 0;
    uint64_t needs = 0;        // qubits that some gate is not diagonal on
    uint64_t phases = 0;       // qubits of the diagonal gates
    std::vector<int> taken;    // by the scan at hand
    bool empty() const { return front == ids.size(); }
    void add(int i, const TGate &g)
    {
        ids.push_back(i);
        needs |= g.need;
        if (!g.need) phases |= g.diag;
    }
    // Ends a scan that looked at the gates before place `end`.
    void close(size_t end, std::vector<char> &done)
    {
        for (int i : taken) done[size_t(i)] = 1;
        size_t w = end;
        for (size_t i = end; i-- > front;)
            if (!done[size_t(ids[i])]) ids[--w] = ids[i];
        front = w;
        for (int i : taken) done[size_t(i)] = 0;
        taken.clear();
    }
};

// Qubits of the gates skipped so far, by how those gates act on them.
struct Skipped {
    uint64_t diag = 0, other = 0;
    int count = 0;
    bool blocks(const TGate &g) const { return (g.need & (diag | other)) || (g.diag & other); }
    void add(const TGate &g)
    {
        diag |= g.diag;
        other |= g.need;
        ++count;
    }
    // Whether a scan ends here: every gate of the list is blocked, or so many
    // were that the rest (of a circuit some of whose qubits see diagonal gates
    // only) is not worth its time.
    bool ends(const GateList &l) const
    {
        return (!(l.needs & ~(diag | other)) && !(l.phases & ~other)) || count >= kSkips;
    }
    static constexpr int kSkips = 1024;
};

// Phases that wait at most, so that looking through them stays cheap.
constexpr size_t kWaiting = 4096;

int bits(uint64_t m) { return __builtin_popcountll(m); }

struct Planner {
    int n, T, low;                 // low: qubits inside a 128-byte line
    const std::vector<TGate> &gates;
    TilePlan &out;
    struct Placed {                // a phase as a stage sees it
        uint32_t amps;
        uint64_t om, ov;
        Phase p;
    };
    std::vector<Term> pending;     // phases not applied yet
    std::vector<Term> now;         // scratch of flush
    std::vector<Placed> sign, ph;
    struct Inside {                // phases that depend on register bits alone, by register mask
        uint32_t amps;
        Phase p;
    };
    std::vector<Inside> inside;
    Phase scale = 1.0L;            // and the one that all amplitudes share
    double flops = 0;              // multiply-adds per amplitude
    mutable size_t seen = 0;       // where the last closure ended
    std::vector<char> done;        // scratch of GateList::close

    Planner(int n_, int T_, int low_, const std::vector<TGate> &g, TilePlan &o)
        : n(n_), T(T_), low(low_), gates(g), out(o), done(g.size(), 0)
    {
    }

    // Gates of `left` that a pass with tile `S` takes; grow: take qubits of
    // skipped gates into S while there is room, and note what is taken.
    double closure(GateList &left, uint64_t &S, bool grow) const
    {
        Skipped sk;
        double score = 0;
        size_t i = left.front;
        for (; i < left.ids.size() && !sk.ends(left); ++i) {
            const TGate &g = gates[size_t(left.ids[i])];
            bool take = false;
            if (!sk.blocks(g) && g.kind != kAlone) {
                if (!(g.need & ~S)) take = true;
                else if (grow && bits(S | g.need) <= T) {
                    S |= g.need;
                    take = true;
                }
            }
            if (take) {
                score += g.need ? 1.0 : 0.3;
                if (grow) left.taken.push_back(left.ids[i]);
            } else {
                sk.add(g);
            }
        }
        seen = i;
        return score;
    }

    // The tile that takes most gates, grown by one frontier gate's qubits at
    // a time. About a fifth fewer passes than taking qubits in circuit
    // order, for some ten times the planning.
    uint64_t best_tile(GateList &left, uint64_t S) const
    {
        while (bits(S) < T) {
            const double now = closure(left, S, false);
            std::vector<uint64_t> cand;
            Skipped sk;
            for (size_t i = left.front; i < left.ids.size() && !sk.ends(left); ++i) {
                const TGate &g = gates[size_t(left.ids[i])];
                const bool free = !sk.blocks(g) && g.kind != kAlone;
                if (free && !(g.need & ~S)) continue;
                if (free && bits(S | g.need) <= T) {
                    const uint64_t a = g.need & ~S;
                    if (std::find(cand.begin(), cand.end(), a) == cand.end()) cand.push_back(a);
                }
                sk.add(g);
            }
            uint64_t pick = 0;
            double best = -1;
            for (uint64_t a : cand) {
                uint64_t s = S | a;
                const double gain = (closure(left, s, false) - now) / bits(a);
                if (gain > best) {
                    best = gain;
                    pick = a;
                }
            }
            if (!pick) break;
            S |= pick;
        }
        return S;
    }

    // ----- stages ---------------------------------------------------------
    struct Stage {
        uint64_t regs = 0;
        std::vector<int> gates;
    };

    // The tile's bits as a stage lays them out: thread bits, then registers.
    void layout(const TilePass &p, uint64_t regs, std::vector<uint64_t> &w, int *reg_bit) const
    {
        std::vector<int> thr, reg;
        for (int i = 0; i < T; ++i) ((regs >> p.pos[i]) & 1 ? reg : thr).push_back(i);
        // the low five lane bits on tile bits that differ modulo 5, lowest first
        std::vector<int> order;
        uint32_t cls = 0;
        for (int t : thr)
            if (!((cls >> (t % 5)) & 1) && order.size() < 5) {
                cls |= 1u << (t % 5);
                order.push_back(t);
            }
        for (int t : thr)
            if (std::find(order.begin(), order.end(), t) == order.end()) order.push_back(t);
        uint64_t w0 = 0, w1 = 0, w2 = 0;
        for (int i = 0; i < T - 4; ++i) {
            w0 |= uint64_t(order[size_t(i)]) << (4 * i);
            w1 |= uint64_t(p.pos[order[size_t(i)]]) << (6 * i);
        }
        for (int b = 0; b < 4; ++b) {
            w0 |= uint64_t(reg[size_t(b)]) << (4 * (T - 4 + b));
            w2 |= uint64_t(p.pos[reg[size_t(b)]]) << (6 * b);
            reg_bit[b] = p.pos[reg[size_t(b)]];
        }
        w.push_back(w0);
        w.push_back(w1);
        w.push_back(w2);
    }

    // Register mask of the registers whose bits match (mask, vals); the part
    // of both outside the registers is left in omask, ovals.
    static uint32_t registers(const int *reg_bit, uint64_t mask, uint64_t vals, uint64_t &omask, uint64_t &ovals)
    {
        static const uint32_t ones[4] = {0xaaaa, 0xcccc, 0xf0f0, 0xff00};   // registers j with bit b set
        uint32_t amps = 0xffff;
        uint64_t r = 0;
        for (int b = 0; b < 4; ++b) {
            r |= 1ull << reg_bit[b];
            if ((mask >> reg_bit[b]) & 1) amps &= (vals >> reg_bit[b]) & 1 ? ones[b] : ~ones[b];
        }
        omask = mask & ~r;
        ovals = vals & ~r;
        return amps;
    }

    // Applies the waiting terms that involve a qubit of `which` here; all:
    // every one, and the common phase.
    int flush(uint64_t which, bool all, const int *reg_bit, std::vector<uint64_t> &w)
    {
        now.clear();
        sign.clear();
        ph.clear();
        size_t kept = 0;
        for (size_t i = 0; i < pending.size(); ++i) {
            if (all || (pending[i].mask & which)) now.push_back(pending[i]);
            else pending[kept++] = pending[i];
        }
        pending.resize(kept);
        inside.clear();
        auto add_inside = [&](uint32_t amps, const Phase &f) {
            for (Inside &i : inside)
                if (i.amps == amps) {
                    i.p = times(i.p, f);
                    return;
                }
            inside.push_back(Inside{amps, f});
        };
        if (all && scale != Phase(1.0L)) add_inside(0xffff, scale);
        if (all) scale = 1.0L;
        for (const Term &t : now) {
            Placed q;
            q.amps = registers(reg_bit, t.mask, t.vals, q.om, q.ov);
            q.p = t.p;
            if (!q.om) {
                add_inside(q.amps, t.p);
            } else if (t.p == Phase(-1.0L) && sign.size() < 0xfff * kTileSigns) {
                sign.push_back(q);
            } else {
                ph.push_back(q);
            }
        }
        if (ph.size() > 1)
            std::stable_sort(ph.begin(), ph.end(), [](const Placed &a, const Placed &b) { return a.amps < b.amps; });
        // one set of registers: a group without conditions instead of a table
        const bool one = inside.size() == 1;
        const uint32_t set = one ? inside[0].amps : 0;
        const bool tab = inside.size() > 1;
        if (!one && !tab && sign.empty() && ph.empty()) return 0;
        const size_t head = w.size();
        w.push_back(0);
        auto put = [&](const Phase &f) {
            w.push_back(word_of(double(f.real())));
            w.push_back(word_of(double(f.imag())));
        };
        if (tab) {
            for (int j = 0; j < 16; ++j) {
                Phase f = 1.0L;
                for (const Inside &i : inside)
                    if ((i.amps >> j) & 1) f = times(f, i.p);
                put(f);
            }
            flops += 4;
        }
        flops += sign.empty() ? 0.0 : 2.0 + 0.25 * double(sign.size());
        while (sign.size() % kTileSigns) sign.push_back(Placed{0, 0, 0, Phase()});   // flips nothing
        for (const Placed &q : sign) {
            w.push_back(q.om);
            w.push_back(q.ov);
            w.push_back(q.amps);
        }
        uint64_t groups = 0;
        bool placed = !one;
        for (size_t i = 0; i < ph.size() || !placed;) {
            const bool lone = !placed && (i >= ph.size() || ph[i].amps > set);
            const uint32_t amps = lone ? set : ph[i].amps;
            size_t e = i;
            while (!lone && e < ph.size() && ph[e].amps == amps) ++e;
            w.push_back(uint64_t(amps) | uint64_t(e - i) << 16);
            const bool first = one && amps == set;
            put(first ? inside[0].p : Phase(1.0L));
            placed = placed || first;
            for (size_t j = i; j < e; ++j) {
                w.push_back(ph[j].om);
                w.push_back(ph[j].ov);
                put(ph[j].p);
            }
            ++groups;
            flops += 4.0 * bits(amps) / 16.0 + double(e - i);
            i = e;
        }
        ++out.ops[kTileDiag];
        w[head] = uint64_t(kTileDiag) | uint64_t(tab) << 6 | uint64_t(sign.size() / kTileSigns) << 8 | groups << 20 |
                  uint64_t(w.size() - head) << 32;
        return 1;
    }

    static int reg_of(const int *reg_bit, int q)
    {
        for (int b = 0; b < 4; ++b)
            if (reg_bit[b] == q) return b;
        return -1;
    }

    void emit(std::vector<uint64_t> &w, int kind, int arg, uint32_t amps, std::initializer_list<uint64_t> masks,
              const double *m, int count)
    {
        ++out.ops[kind];
        w.push_back(uint64_t(kind) | uint64_t(arg) << 3 | uint64_t(amps) << 8 |
                    uint64_t(1 + masks.size() + size_t(count)) << 32);
        w.insert(w.end(), masks);
        for (int i = 0; i < count; ++i) w.push_back(word_of(m[i]));
    }

    int emit_gate(const TGate &g, const int *reg_bit, std::vector<uint64_t> &w)
    {
        const int a = reg_of(reg_bit, g.target[0]);
        if (g.kind == kRotation) {
            emit(w, kTileRotate, a, 0, {}, g.r, 4);
            flops += 4;
            return 1;
        }
        if (g.kind == kOne) {
            uint64_t om = 0, ov = 0;
            const uint32_t amps = registers(reg_bit, g.diag, g.cvals, om, ov);
            // an X moves both words of its values by three logic instructions each
            flops += 8.0 * bits(amps) / 16.0;
            if (g.x) emit(w, kTileX, a, amps, {om, ov}, nullptr, 0);
            else if (g.diag) emit(w, kTileCDense1, a, amps, {om, ov}, g.m, 8);
            else emit(w, kTileDense1, a, 0, {}, g.m, 8);
            return 1;
        }
        const int b = reg_of(reg_bit, g.target[1]);
        if (g.kind == kSwap) {
            // X on one under the other, back, and again
            for (int i = 0; i < 3; ++i) {
                const int x = i & 1 ? b : a, ctl = i & 1 ? a : b;
                uint32_t amps = 0;
                for (int j = 0; j < 16; ++j) amps |= uint32_t((j >> ctl) & 1) << j;
                emit(w, kTileX, x, amps, {0, 0}, nullptr, 0);
            }
            flops += 12;
            return 3;
        }
        // local bit 0 = the lower register bit
        static const int pair_no[4][4] = {{0, 0, 1, 2}, {0, 0, 3, 4}, {0, 0, 0, 5}, {0, 0, 0, 0}};
        auto loc = [&](int i) { return a < b ? i : ((i & 1) << 1) | (i >> 1); };
        double m[32];
        for (int r = 0; r < 4; ++r)
            for (int c = 0; c < 4; ++c) std::copy_n(g.mat + 2 * (4 * loc(r) + loc(c)), 2, m + 2 * (4 * r + c));
        emit(w, kTileDense2, pair_no[std::min(a, b)][std::max(a, b)], 0, {}, m, 32);
        flops += 18;
        return 1;
    }

    // One pass over the gates ex (in order); last: apply every waiting term.
    void pass(uint64_t S, const std::vector<int> &ex, bool last)
    {
        const uint64_t lowmask = (1ull << low) - 1;
        for (int q = 0; bits(S) < T; ++q) S |= 1ull << q;   // room left: near qubits
        TilePass p;
        p.T = T;
        for (int q = 0, c = 0; q < n; ++q)
            if ((S >> q) & 1) p.pos[c++] = q;
        p.word0 = out.words.size();
        // stages; the first and the last keep the line qubits on the lanes,
        // so that global accesses move whole lines
        std::vector<Stage> st;
        GateList left;
        for (int i : ex) left.add(i, gates[size_t(i)]);
        while (!left.empty()) {
            Stage s;
            Skipped sk;
            size_t end = left.front;
            for (; end < left.ids.size() && !sk.ends(left); ++end) {
                const int i = left.ids[end];
                const TGate &g = gates[size_t(i)];
                bool take = !sk.blocks(g);
                if (take && g.need & ~s.regs) {
                    take = bits(s.regs | g.need) <= 4 && !(st.empty() && (g.need & lowmask));
                    if (take) s.regs |= g.need;
                }
                if (take) left.taken.push_back(i);
                else sk.add(g);
            }
            s.gates = left.taken;
            left.close(end, done);
            st.push_back(s);
        }
        if (st.empty() || (st.back().regs & lowmask)) st.push_back(Stage());
        for (size_t si = 0; si < st.size(); ++si) {
            Stage &s = st[si];
            // free register places: high tile bits, where lanes and lines are not
            for (int i = T - 1; bits(s.regs) < 4; --i)
                if (!((s.regs >> p.pos[i]) & 1)) s.regs |= 1ull << p.pos[i];
            int reg_bit[4];
            layout(p, s.regs, out.words, reg_bit);
            const size_t head = out.words.size() - 1;
            uint64_t ops = 0;
            // Rounds: the diagonal gates that come first, the phases in front
            // of the rotations, then at most one gate per qubit, so that one
            // diagonal operation serves up to four gates.
            GateList todo;
            for (int gi : s.gates) todo.add(gi, gates[size_t(gi)]);
            while (!todo.empty()) {
                std::vector<int> round;
                Skipped sk;
                size_t end = todo.front;
                for (; end < todo.ids.size() && !sk.ends(todo); ++end) {
                    const int gi = todo.ids[end];
                    const TGate &g = gates[size_t(gi)];
                    // a gate of this round is applied after its phases
                    if (sk.blocks(g)) {
                        sk.add(g);
                        continue;
                    }
                    todo.taken.push_back(gi);
                    if (g.kind == kDiagonal) {
                        add_terms(g, pending);
                    } else {
                        if (g.kind == kRotation && g.before != Phase(1.0L))
                            pending.push_back(Term{g.need, g.need, g.before});
                        sk.other |= g.need;     // one gate per qubit
                        round.push_back(gi);
                    }
                }
                todo.close(end, done);
                uint64_t need = 0;
                for (int gi : round) need |= gates[size_t(gi)].need;
                bool clash = false;
                for (const Term &t : pending) clash = clash || (t.mask & need);
                if (clash) ops += uint64_t(flush(s.regs, false, reg_bit, out.words));
                for (int gi : round) {
                    const TGate &g = gates[size_t(gi)];
                    ops += uint64_t(emit_gate(g, reg_bit, out.words));
                    if (g.kind != kRotation) continue;
                    scale = times(scale, g.a0);
                    if (g.after != Phase(1.0L)) pending.push_back(Term{g.need, g.need, g.after});
                }
                if (pending.size() > kWaiting) ops += uint64_t(flush(0, true, reg_bit, out.words));
            }
            if (last && si + 1 == st.size()) ops += uint64_t(flush(0, true, reg_bit, out.words));
            out.words[head] |= ops << 32;
        }
        p.n_stages = int(st.size());
        out.n_stages += p.n_stages;
        TileStep step;
        step.pass = int(out.passes.size());
        out.passes.push_back(p);
        out.steps.push_back(step);
    }
};

}  // namespace

// Estimated times, in microseconds. The choice between passes and blocks
// rests on them. Both ways were timed on 764 circuits of 10 to 27 qubits in
// both types and blocks of 2 to 6 (random layers, dense two-qubit gates in
// pairs and in rows, controlled one-qubit gates, Toffolis, Hadamards with
// CNOTs, QFTs, Ising steps, adders, mixtures, and gates left alone under one
// and four controls): the slower way is taken for 13 of them, by 16 % at most.

// Reading and writing the state once at 6 TB/s.
static double sweep_us(int n, size_t amp_bytes) { return std::ldexp(2.0 * double(amp_bytes), n) / 6e6; }

// One dense block of k qubits. A launch on a state too small to fill the chip
// takes the first term (fewer than 6 + k qubits leave a 5- or 6-qubit block
// to a few threads); the second is the sweep's (30 qubits, complex128: 5.7 ms
// for k <= 4, 6.6 and 21.3 ms for k = 5 and 6; complex64: 2.9, 3.5 and 4.5 ms).
double dense_us(int n, size_t amp_bytes, int k)
{
    const bool c128 = amp_bytes == 16;
    const double mem = sweep_us(n, amp_bytes);
    if (k <= 4) return (k <= 3 ? 4.0 : c128 ? 5.6 : 4.5) + mem;
    if (k == 5) return (n < 11 ? 22.0 : c128 ? 8.0 : 7.0) + 1.2 * mem;
    return (n < 12 ? (c128 ? 35.0 : 100.0) : c128 ? 18.0 : 9.0) + (c128 ? 3.7 : 1.55) * mem;
}

// A block of diagonal gates sweeps only what it changes, a quarter of the
// state for a CZ.
double diagonal_us(int n, size_t amp_bytes) { return 4.0 + 0.25 * sweep_us(n, amp_bytes); }

// The passes: per pass, stage and operation what a workgroup takes alone,
// which is all on a small state, and their memory and arithmetic (flops in
// multiply-adds per amplitude, 30 T of them a second) on a large one.
static double passes_us(int n, size_t amp_bytes, const TilePlan &p, double flops)
{
    const double mem = sweep_us(n, amp_bytes), fma = (30e12 / 6e12) * 2.0 * double(amp_bytes);
    const double moves = p.ops[kTileCDense1] + p.ops[kTileX] + p.ops[kTileDense2];
    return 4.2 * double(p.passes.size()) + 1.2 * p.n_stages + 0.28 * moves + 0.74 * p.ops[kTileDiag] +
           mem * (0.52 * double(p.passes.size()) + 0.79 * flops / fma);
}

bool plan_tiles(int n, size_t amp_bytes, const qs_circuit *c, double limit, TilePlan &out)
{
    out = TilePlan();
    if (n < kTileBitsMin) return false;
    // Twelve qubits: a larger tile needs fewer passes but leaves two large
    // workgroups per compute unit, a smaller one needs more (11, 12, 13: 28
    // qubits complex128 34.6, 32.5, 34.0 ms; 27 qubits complex64 14.5, 14.1,
    // 14.5 ms). A smaller state is one tile.
    const int T = std::min(n, kTileBitsMax), low = amp_bytes == 16 ? 3 : 4;
    std::vector<TGate> gates(size_t(std::max(0, c->n_gates)));
    const int *tp = c->targets;
    const double *mp = c->matrices;
    GateList left;
    double swept = 0;              // time of the gates left alone
    for (int g = 0; g < c->n_gates; ++g) {
        const uint64_t cm = c->ctrl_mask ? c->ctrl_mask[g] : 0;
        read_gate(c->k[g], tp, mp, cm, c->ctrl_vals ? c->ctrl_vals[g] & cm : 0, gates[size_t(g)]);
        tp += c->k[g];
        mp += size_t(2) << (2 * c->k[g]);
        if (gates[size_t(g)].kind == kAlone)   // a block over its targets and controls
            swept += dense_us(n, amp_bytes, bits(gates[size_t(g)].need | gates[size_t(g)].diag));
        if (gates[size_t(g)].kind != kNothing) left.add(g, gates[size_t(g)]);
    }
    Planner pl(n, T, low, gates, out);
    const uint64_t lowmask = (1ull << low) - 1;
    // Searching for tiles costs a millisecond for some hundred gates, a tenth
    // of one for each pass, and saves a fifth of the passes: worth it once a
    // pass takes as long.
    const bool search = (amp_bytes << n) >= (size_t(1) << 29);
    auto cost = [&]() { return passes_us(n, amp_bytes, out, pl.flops) + swept; };
    auto front_alone = [&]() { return !left.empty() && gates[size_t(left.ids[left.front])].kind == kAlone; };
    while (!left.empty()) {
        if (front_alone()) {
            TileStep s;
            s.gate = left.ids[left.front++];
            out.steps.push_back(s);
            continue;
        }
        if (cost() >= limit) break;
        uint64_t S = lowmask;
        if (search) S = pl.best_tile(left, S);
        pl.closure(left, S, true);
        const std::vector<int> ex = left.taken;
        left.close(pl.seen, pl.done);
        pl.pass(S, ex, left.empty() || front_alone());
    }
    out.words.insert(out.words.end(), size_t(kTileAhead), 0);
    out.cost = cost();
    if (out.cost < limit) return true;
    out = TilePlan();
    return false;
}

}  // namespace qs
