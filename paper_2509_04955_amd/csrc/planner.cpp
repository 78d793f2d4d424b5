// Host planner: dependency-aware gate contraction (Section 3.4) and the
// packing of fused blocks into streamed tile passes.
//
// DAG.  Gates that share a qubit (controls included) are ordered by program
// order; gates with no path between them commute (Section 3.4).  The DAG is
// never materialised: `last[q]` (the block holding the most recent gate on
// qubit q) carries exactly the information the merge needs.
//
// Merge.  The paper merges greedily without fixing the rule; this library's
// fixed-width greedy rule (width k_max) is: for gate g with qubit set Q,
// f = max_{q in Q} last[q]; g joins the lowest block j >= max(f, 1) with
// |Q_j u Q| <= k_max, else a new block.  Blocks after f hold no qubit of Q, so
// for j > f the test is |Q_j| + |Q| <= k_max; a segment tree over block widths
// finds that j in O(log blocks).  Block products compose the member gates in
// program order (Kronecker embedding of each gate into the block's qubits, the
// same-qubit product M2 M1 and the controlled merge being special cases).
//
// Passes.  Consecutive blocks are packed into one pass while the union of
// their qubits with the always-present low qubits {0..c-1} stays within t
// qubits; a pass is one read and one write of the state (one tile kernel).
#include <algorithm>
#include <cmath>
#include <cstring>
#include <limits>
#include <stdexcept>

#include "internal.h"

namespace qs {

namespace {

// Tile qubits and fixed low qubits where the caller leaves both open, for n
// qubits and blocks of up to k.  Geometric means over ansatz, random, UCC and
// Fourier circuits, us per plan, against tiles of 2^13 (complex64) or 2^12
// amplitudes with 6 low qubits:
//   * up to 16 qubits (complex128: 18): a pass is a few small workgroups in
//     flight, and smaller tiles spread it over more CUs; states of this size
//     stay in the caches, so short runs cost nothing (14 qubits complex64: 66
//     against 149 us for an ansatz of four layers; 16 qubits complex128: 126
//     against 239).  Exceptions are complex64 blocks of 4 and 6 qubits at 12
//     qubits (random gates, k 4: 35 us in one tile against 45; an ansatz of
//     six layers, k 6: 97 against 147) and of 4 at 13 (43 us in 2^11 tiles
//     against 61), where the matrix cores do more in larger tiles;
//   * to 22: the smallest tiles that still give every CU one or two (20 qubits
//     complex64: 200 against 260; complex128 as noted below);
//   * above: as many qubits as the LDS allows, fewest passes, and runs of a
//     cache line (24 qubits complex64: 1700 against 2000).  Complex128 blocks
//     of four and five qubits are held back by waves, not by passes: smaller
//     tiles (24 qubits, k 5: 4.1 against 6.3 ms, 26 qubits: 18.7 against 25.6;
//     k 3 is fastest at 2^12: 6.2 against 7.1 ms).  Single circuits can go the
//     other way by a pass more: random gates at 24 qubits, k 4, 1.34 against
//     1.17 ms, the Fourier transform at 26, k 5, 26.0 against 24.3.
// One tile holds states of up to 11 qubits (11 qubits: 44 us against 55 us in
// two tiles).
// A plan of single gates (k: its widest) has the least work per pass: 2^11
// tiles from 24 qubits complex128 (26 qubits: 17.3 against 18.2 ms at 2^12).
// rot: a plan of rotations with an X part.  They need few qubits in the tile
// and do little with them there, so passes decide.  One tile up to 13 qubits
// (complex128: 12; 40 exponentials on 12 qubits 42 us, in 2^10 tiles 67), and
// complex128 states from 23 qubits in 2^12 tiles with 3 low qubits (24 qubits:
// 1.66 ms, in 2^11 tiles with 5 2.19).
void auto_shape(int n, qs_dtype dt, int k, bool single, bool rot, int &t, int &low) {
    const bool c64 = dt == QS_C64;
    if (n <= 11 || (rot && n <= (c64 ? 13 : 12))) {
        t = std::max(n, 11);
        low = 6;
    } else if (c64 && !rot && ((n == 12 && (k == 4 || k == 6)) || (n == 13 && k == 4))) {
        t = n == 12 ? 12 : 11;
        low = 3;
    } else if (n <= (c64 ? 16 : 18)) {
        t = 10;
        low = 2;
    } else if (c64) {
        t = n <= 20 ? 11 : 13;
        low = n <= 20 ? 3 : 4;
    } else {
        // 20 qubits, k 5: 352 us at 2^12 against 390; k 2..4: 262..334 against 235..295 at 2^11
        const bool wide = k >= 4 && !rot;
        t = n == 19 || (n == 20 && k < 5) || (n >= 23 && wide) || (n >= 24 && single) ? 11 : 12;
        low = n >= 23 && wide && k >= 5 ? 5 : 3;
    }
}

// The same where only one of the two is open.  A given tile takes the low
// qubits of the rule above (five families of circuits, 10..26 qubits, tiles of
// 2^10..2^14, k 3 and 5: on average 0 to 30 % faster than six low qubits at
// every size, 12 of 576 plans slower, by 2 to 9 %).  Given low qubits keep the
// largest usual tile: the sizes above were chosen with their low qubits, and
// with others as many plans lost as won (12 qubits complex64, 4 low qubits, k
// 3: 53 against 67 us; 24 qubits complex128, 2 low, k 5: 4.0 against 5.5 ms).
constexpr int usual_tile(qs_dtype dt) { return dt == QS_C128 ? 12 : 13; }

}  // namespace

namespace {

// Segment tree over block widths: first index > f whose width <= s.
struct MinTree {
    int size = 1;
    std::vector<int> v;
    explicit MinTree(size_t cap) {
        while ((size_t)size < cap + 1) size <<= 1;
        v.assign(2 * size, std::numeric_limits<int>::max());
    }
    void set(int i, int val) {
        i += size;
        v[i] = val;
        for (i >>= 1; i; i >>= 1) v[i] = std::min(v[2 * i], v[2 * i + 1]);
    }
    // smallest index >= lo with value <= s, or -1
    int first_le(int lo, int s) const { return find(1, 0, size, lo, s); }
    int find(int node, int l, int r, int lo, int s) const {
        if (r <= lo || v[node] > s) return -1;
        if (r - l == 1) return l;
        int m = (l + r) / 2;
        int a = find(2 * node, l, m, lo, s);
        return a >= 0 ? a : find(2 * node + 1, m, r, lo, s);
    }
};

}  // namespace

uint64_t diagonal_qubits(const HGate &g) {
    if (g.m.empty()) return 0;
    const int d = 1 << g.nq;
    uint64_t out = 0;
    for (int j = 0; j < g.nq; ++j) {
        bool diag = true;
        for (int r = 0; r < d && diag; ++r)
            for (int c = 0; c < d; ++c)
                if (((r ^ c) >> j) & 1 && g.m[(size_t)r * d + c] != cd(0, 0)) {
                    diag = false;
                    break;
                }
        if (diag) out |= 1ull << g.q[j];
    }
    return out;
}

void greedy_blocks(const std::vector<HGate> &gates, int n, int kmax, std::vector<HBlock> &blocks,
                   const std::vector<char> *solo, bool commute) {
    blocks.clear();
    std::vector<int> last(n, 0);                 // 1-based block index, 0 = none
    std::vector<int> last_nd(n, 0);              // latest block acting non-diagonally on the qubit
    std::vector<uint64_t> qmask;                 // qubit mask per block
    std::vector<int> width;
    std::vector<char> closed;                    // blocks that take no further gates (solo units)
    MinTree tree(gates.size() + 1);
    for (size_t gi = 0; gi < gates.size(); ++gi) {
        const HGate &g = gates[gi];
        const uint64_t dq = commute ? diagonal_qubits(g) : 0;
        uint64_t gm = 0;
        int f = 0, L = 0;   // f: latest block g must follow; L: latest block touching g's qubits
        for (int j = 0; j < g.nq; ++j) {
            const int q = g.q[j];
            gm |= 1ull << q;
            f = std::max(f, ((dq >> q) & 1) ? last_nd[q] : last[q]);
            L = std::max(L, last[q]);
        }
        const int w = g.nq;
        const bool alone = solo && (*solo)[gi];
        int j = -1;  // 1-based
        if (w <= kmax && !alone) {
            // lowest block >= max(f, 1) whose qubits with g's stay within kmax:
            // blocks up to L may share qubits with g (only when it commutes
            // past them), blocks after L share none (width test in the tree)
            for (int b = std::max(f, 1); b <= L && j < 0; ++b)
                if (!closed[b - 1] && __builtin_popcountll(qmask[b - 1] | gm) <= kmax) j = b;
            if (j < 0) {
                int idx = tree.first_le(std::max(L + 1, 1), kmax - w);  // tree index = 1-based block id
                if (idx >= 1 && idx <= (int)blocks.size()) j = idx;
            }
        }
        if (j < 0) {
            blocks.emplace_back();
            qmask.push_back(0);
            width.push_back(0);
            closed.push_back(alone ? 1 : 0);
            j = (int)blocks.size();
        }
        blocks[j - 1].members.push_back((int64_t)gi);
        qmask[j - 1] |= gm;
        width[j - 1] = __builtin_popcountll(qmask[j - 1]);
        tree.set(j, closed[j - 1] ? 64 : width[j - 1]);
        for (int q = 0; q < g.nq; ++q) {
            const int qq = g.q[q];
            last[qq] = std::max(last[qq], j);
            if (!((dq >> qq) & 1)) last_nd[qq] = std::max(last_nd[qq], j);
        }
    }
    for (size_t b = 0; b < blocks.size(); ++b) {
        blocks[b].qubits.clear();
        for (int q = 0; q < 64; ++q)
            if ((qmask[b] >> q) & 1) blocks[b].qubits.push_back(q);
    }
}

// U_B = G_m ... G_1 with each gate embedded into the block's qubits.  A gate
// combines whole rows of U (left multiplication), real and imaginary parts in
// arrays of their own, so the inner loops run over contiguous columns and
// vectorise.  U grows with the qubits touched so far: their local bits are in
// order of first touch, so a new qubit doubles U by a copy of itself on the
// diagonal.  Zero entries of a gate are left out where every factor is finite
// (0 x would then add nothing).  192 gates in five-qubit blocks: 1.46 ms of
// host time per plan with full-width std::complex products column by column,
// 0.2 ms so.
void block_matrix(const std::vector<HGate> &gates, HBlock &b) {
    const int k = (int)b.qubits.size();
    const int d = 1 << k;
    bool finite = true;
    for (int64_t gi : b.members)
        for (const cd &v : gates[gi].m) finite &= std::isfinite(v.real()) && std::isfinite(v.imag());
    std::vector<double> buf((size_t)2 * d * d), tmp;
    double *ur = buf.data(), *ui = ur + (size_t)d * d;   // row stride d
    ur[0] = 1.0;
    int bit[64];      // local bit of a block qubit (by its place in b.qubits), -1: not touched yet
    std::fill(bit, bit + k, -1);
    int touched = 0;
    auto touch = [&](int place) {
        const int w = 1 << touched;
        for (int r = 0; r < w; ++r) {
            std::copy_n(ur + (size_t)r * d, w, ur + (size_t)(r + w) * d + w);
            std::copy_n(ui + (size_t)r * d, w, ui + (size_t)(r + w) * d + w);
        }
        bit[place] = touched++;
    };
    for (int64_t gi : b.members) {
        const HGate &g = gates[gi];
        const int gd = 1 << g.nq;
        int gmask = 0, off[64] = {0};   // gates have at most six qubits
        for (int j = 0; j < g.nq; ++j) {
            const int place = (int)(std::find(b.qubits.begin(), b.qubits.end(), g.q[j]) - b.qubits.begin());
            if (bit[place] < 0) touch(place);
            gmask |= 1 << bit[place];
            for (int a = 0; a < gd; ++a)
                if ((a >> j) & 1) off[a] |= 1 << bit[place];
        }
        const int w = 1 << touched;
        tmp.resize((size_t)2 * gd * w);
        for (int base = 0; base < w; ++base) {
            if (base & gmask) continue;
            std::fill(tmp.begin(), tmp.end(), 0.0);
            for (int a = 0; a < gd; ++a) {
                double *__restrict__ xr = tmp.data() + (size_t)2 * a * w, *__restrict__ xi = xr + w;
                for (int c = 0; c < gd; ++c) {
                    const double mr = g.m[(size_t)a * gd + c].real(), mi = g.m[(size_t)a * gd + c].imag();
                    const double *__restrict__ vr = ur + (size_t)(base | off[c]) * d;
                    const double *__restrict__ vi = ui + (size_t)(base | off[c]) * d;
                    if (finite && mi == 0.0) {
                        if (mr == 0.0) continue;
                        for (int col = 0; col < w; ++col) {
                            xr[col] += mr * vr[col];
                            xi[col] += mr * vi[col];
                        }
                    } else {
                        for (int col = 0; col < w; ++col) {
                            xr[col] += mr * vr[col] - mi * vi[col];
                            xi[col] += mr * vi[col] + mi * vr[col];
                        }
                    }
                }
            }
            for (int a = 0; a < gd; ++a) {
                std::copy_n(tmp.data() + (size_t)2 * a * w, w, ur + (size_t)(base | off[a]) * d);
                std::copy_n(tmp.data() + (size_t)2 * a * w + w, w, ui + (size_t)(base | off[a]) * d);
            }
        }
    }
    for (int place = 0; place < k; ++place)
        if (bit[place] < 0) touch(place);
    // back to ascending qubits
    std::vector<int> at(d, 0);
    for (int i = 0; i < d; ++i)
        for (int j = 0; j < k; ++j)
            if ((i >> j) & 1) at[i] |= 1 << bit[j];
    b.U.resize((size_t)d * d);
    for (int r = 0; r < d; ++r)
        for (int c = 0; c < d; ++c) b.U[(size_t)r * d + c] = cd(ur[(size_t)at[r] * d + at[c]], ui[(size_t)at[r] * d + at[c]]);
}

// Passes: list scheduling of the blocks over their dependence order (Section
// 3.4: blocks sharing a qubit keep their order; two Pauli-rotation blocks with
// commuting strings may swap).  A pass starts from the first
// pending block and its tile {0..c-1}; pending blocks are scanned in order and
// a block joins the pass if its qubits fit the tile (at most t qubits).  A block
// that does not fit is left for a later pass and its qubits are marked: no
// later block touching them may run ahead of it, but blocks on other qubits may
// still join.  The scan stops kLookahead blocks after the first one left out.
// The blocks are reordered into execution order (pass by pass), so a pass is a
// contiguous range; any order produced this way keeps every pair of blocks that
// share a qubit in program order, hence the same state in exact arithmetic.
constexpr size_t kLookahead = 64;

namespace {
// entries of a block product below this are rounding residue of exact zeros
// (the same threshold as the monomial test of the tile kernels)
constexpr double kDiagTol = 1e-14;

// qubits on which a (non-rotation) block acts diagonally, from its matrix
uint64_t block_diagonal(const HBlock &b) {
    const int k = (int)b.qubits.size(), d = 1 << k;
    if (b.U.size() != (size_t)d * d) return 0;
    uint64_t out = 0;
    for (int j = 0; j < k; ++j) {
        bool diag = true;
        for (int r = 0; r < d && diag; ++r)
            for (int c = 0; c < d; ++c)
                if (((r ^ c) >> j) & 1 && std::abs(b.U[(size_t)r * d + c]) > kDiagTol) {
                    diag = false;
                    break;
                }
        if (diag) out |= 1ull << b.qubits[j];
    }
    return out;
}
}  // namespace

void pack_passes(const qs_plan_s &p, std::vector<HBlock> &blocks, int t, int c, std::vector<HPass> &out) {
    out.clear();
    const int n = p.n;
    t = std::min(t, n);
    c = std::min(c, t);
    const uint64_t low = c >= 64 ? ~0ull : ((1ull << c) - 1);
    // dm: qubits a block depends on (its support); bm: qubits it needs in the
    // tile (the support, or the X part of a Pauli rotation: its Z part outside
    // the tile is a per-tile sign)
    std::vector<uint64_t> bm(blocks.size(), 0), dm(blocks.size(), 0);
    for (size_t b = 0; b < blocks.size(); ++b) {
        for (int q : blocks[b].qubits) dm[b] |= 1ull << q;
        bm[b] = blocks[b].pauli ? blocks[b].px : dm[b];
    }
    // Two Pauli-rotation blocks whose strings commute commute as operators
    // (each is c I + d P), so one may overtake the other although they share
    // qubits.  With the commute option, so may two blocks that are both
    // diagonal on every qubit they share (dg: qubits a block acts on
    // diagonally, from its matrix with entries below kDiagTol taken as the
    // rounding residue of exact zeros; a rotation is diagonal off its X
    // part).  Every other pair sharing a qubit keeps its order.
    const bool by_diag = p.opts.commute != 0;
    std::vector<uint64_t> dg(blocks.size(), 0);
    if (by_diag)
        for (size_t b = 0; b < blocks.size(); ++b) dg[b] = blocks[b].pauli ? dm[b] & ~blocks[b].px : block_diagonal(blocks[b]);
    auto commute = [&](size_t a, size_t b) {
        const HBlock &A = blocks[a], &B = blocks[b];
        if (A.pauli && B.pauli &&
            ((__builtin_popcountll(A.px & B.pz) + __builtin_popcountll(A.pz & B.px)) & 1) == 0)
            return true;
        const uint64_t shared = dm[a] & dm[b];
        return by_diag && (shared & ~(dg[a] & dg[b])) == 0;
    };
    std::vector<size_t> pending(blocks.size()), rest;
    for (size_t b = 0; b < blocks.size(); ++b) pending[b] = b;
    std::vector<HBlock> ordered;
    ordered.reserve(blocks.size());
    while (!pending.empty()) {
        HPass ps;
        ps.block0 = (int64_t)ordered.size();
        uint64_t cur = low, blocked = 0;
        size_t scanned_after_skip = 0, i = 0;
        bool skipped = false;
        rest.clear();
        for (; i < pending.size(); ++i) {
            if (skipped && scanned_after_skip++ >= kLookahead) break;
            const size_t b = pending[i];
            bool free = (dm[b] & blocked) == 0;
            if (!free && (blocks[b].pauli || by_diag)) {
                // overtaking is allowed past skipped blocks it commutes with
                free = true;
                for (size_t r : rest)
                    if ((dm[r] & dm[b]) && !commute(r, b)) {
                        free = false;
                        break;
                    }
            }
            if (free && __builtin_popcountll(cur | bm[b]) <= t) {
                cur |= bm[b];
                ordered.push_back(std::move(blocks[b]));
            } else {
                blocked |= dm[b];
                rest.push_back(b);
                skipped = true;
            }
        }
        rest.insert(rest.end(), pending.begin() + (int64_t)i, pending.end());
        ps.nblocks = (int64_t)ordered.size() - ps.block0;
        // the first pending block always fits (c is sized for the widest block)
        if (ps.nblocks == 0) throw std::logic_error("pass packing made no progress");
        // fill the tile up to t qubits with the lowest unused qubits
        uint64_t m = cur;
        for (int q = 0; q < n && __builtin_popcountll(m) < t; ++q) m |= 1ull << q;
        ps.t = t;
        for (int q = 0; q < n; ++q)
            if ((m >> q) & 1) ps.tile.push_back(q);
        int cc = 0;
        while (cc < (int)ps.tile.size() && ps.tile[cc] == cc) ++cc;
        ps.c = cc;
        // the planner sizes c so that every pass holds exactly t qubits and qubit 0
        if ((int)ps.tile.size() != t || cc < 1) throw std::logic_error("pass tile invariant broken");
        out.push_back(std::move(ps));
        pending.swap(rest);
    }
    blocks.swap(ordered);
}

std::vector<PauliWindow> pauli_windows(const std::vector<HGate> &gates, int k_max, int max_x_weight) {
    std::vector<PauliWindow> win = find_pauli_windows(gates, max_x_weight);
    // a diagonal rotation (no X part) no wider than k_max is left to the
    // greedy rule, which merges several of them (and their neighbours) into
    // one diagonal block: one block per rotation would cost a tile round trip
    // each (QAOA's ZZ terms)
    win.erase(std::remove_if(win.begin(), win.end(),
                             [&](const PauliWindow &w) { return w.x == 0 && (int)w.support.size() <= k_max; }),
              win.end());
    return win;
}

void pauli_contract(const std::vector<HGate> &gates, int n, int k_max, const std::vector<PauliWindow> &win,
                    std::vector<HBlock> &blocks, bool commute) {
    // units: each window, and every gate outside the windows, in program
    // order; a window is a block of its own, the gates merge greedily
    std::vector<HGate> units;
    std::vector<char> solo;
    std::vector<int64_t> first;   // window: its index; gate: its program index
    size_t wi = 0;
    for (int64_t gi = 0; gi < (int64_t)gates.size();) {
        if (wi < win.size() && win[wi].begin == gi) {
            HGate u;
            u.nq = (int)win[wi].support.size();
            for (int j = 0; j < u.nq; ++j) u.q[j] = win[wi].support[j];
            units.push_back(std::move(u));
            solo.push_back(1);
            first.push_back((int64_t)wi);
            gi = win[wi].end;
            ++wi;
        } else {
            units.push_back(gates[gi]);
            solo.push_back(0);
            first.push_back(gi);
            ++gi;
        }
    }
    greedy_blocks(units, n, k_max, blocks, &solo, commute);
    for (HBlock &b : blocks) {
        if (b.members.size() == 1 && solo[b.members[0]]) {
            const PauliWindow &w = win[first[b.members[0]]];
            b.pauli = true;
            b.px = w.x;
            b.pz = w.z;
            b.pc = w.c;
            b.pd = w.d;
            b.members.clear();
            for (int64_t gi = w.begin; gi < w.end; ++gi) b.members.push_back(gi);
        } else {
            for (int64_t &m : b.members) m = first[m];
        }
    }
}

qs_status build_plan(qs_plan_s &p) {
    qs_contract_opts &o = p.opts;
    const qs_dtype dt = o.dtype == QS_C128 ? QS_C128 : QS_C64;
    const int kcap = dt == QS_C128 ? kMaxK128 : kMaxK;
    if (o.k_max == 0) o.k_max = 5;
    QS_CHECK(o.k_max >= 1 && o.k_max <= kcap, QS_EINVAL, "k_max %d outside 1..%d", o.k_max, kcap);
    int gate_max = 1;
    for (const HGate &g : p.gates) gate_max = std::max(gate_max, g.nq);
    const bool single = o.strategy == QS_STRATEGY_NONE;
    // a plan of rotations: most gates lie in rotations that keep an X part
    // (where the tile is open it holds every X part of up to 8 qubits)
    std::vector<PauliWindow> win;
    const bool open = o.tile_qubits == 0 && o.strategy == QS_STRATEGY_PAULI;
    if (open) win = pauli_windows(p.gates, o.k_max, std::min(8, p.n - 1));
    size_t inside = 0;
    for (const PauliWindow &w : win) inside += (size_t)(w.end - w.begin);
    int auto_t, auto_low;
    auto_shape(p.n, dt, single ? gate_max : o.k_max, single, 2 * inside > p.gates.size(), auto_t, auto_low);
    if (o.tile_qubits == 0) o.tile_qubits = o.low_qubits ? usual_tile(dt) : auto_t;
    const int tcap = dt == QS_C128 ? kMaxTile128 : kMaxTile;
    QS_CHECK(o.tile_qubits >= 2 && o.tile_qubits <= tcap, QS_EINVAL, "tile_qubits %d outside 2..%d",
             o.tile_qubits, tcap);
    if (o.low_qubits == 0) o.low_qubits = std::min(auto_low, o.tile_qubits);
    QS_CHECK(o.low_qubits >= 1 && o.low_qubits <= o.tile_qubits, QS_EINVAL, "low_qubits %d invalid",
             o.low_qubits);
    const int t = std::min(o.tile_qubits, p.n);
    // Every block (a gate wider than k_max is a block of its own) must fit in a
    // tile next to at least one low qubit, so that qubit 0 is always in the
    // tile and tiles start with a contiguous run.
    QS_CHECK(o.strategy >= QS_STRATEGY_NONE && o.strategy <= QS_STRATEGY_PAULI, QS_EINVAL, "strategy %d unknown",
             o.strategy);
    QS_CHECK(o.commute == 0 || o.commute == 1, QS_EINVAL, "commute must be 0 or 1 (got %d)", o.commute);
    int wmax = std::max(o.k_max, gate_max);
    if (o.strategy == QS_STRATEGY_PAULI) {
        // X parts up to 8 qubits and below the tile (qubit 0 keeps a slot)
        if (!open) win = pauli_windows(p.gates, o.k_max, std::min(8, std::min(o.tile_qubits, p.n) - 1));
        for (const PauliWindow &w : win) wmax = std::max(wmax, __builtin_popcountll(w.x));
    }
    if (t < p.n)
        QS_CHECK(std::min(wmax, p.n) <= t - 1, QS_EINVAL,
                 "blocks of width %d need a tile of at least %d qubits (got %d)", wmax, wmax + 1, t);
    const int c = std::max(1, std::min(o.low_qubits, t - std::min(wmax, t)));

    if (o.strategy == QS_STRATEGY_NONE) {
        p.blocks.clear();
        for (size_t gi = 0; gi < p.gates.size(); ++gi) {
            HBlock b;
            b.members.push_back((int64_t)gi);
            for (int j = 0; j < p.gates[gi].nq; ++j) b.qubits.push_back(p.gates[gi].q[j]);
            std::sort(b.qubits.begin(), b.qubits.end());
            p.blocks.push_back(std::move(b));
        }
    } else if (o.strategy == QS_STRATEGY_LEARNED && costmodel_loaded()) {
        return learned_partition(p, t, c);
    } else if (o.strategy == QS_STRATEGY_PAULI) {
        pauli_contract(p.gates, p.n, o.k_max, win, p.blocks, o.commute != 0);
    } else {
        greedy_blocks(p.gates, p.n, o.k_max, p.blocks, nullptr, o.commute != 0);
    }
    for (HBlock &b : p.blocks)
        if (!b.pauli) block_matrix(p.gates, b);
    pack_passes(p, p.blocks, t, c, p.passes);
    return QS_OK;
}

}  // namespace qs
