// Gate lists applied as they come, many gates per read of the state.
//
// qs_apply_gates forms no products of gates: every gate acts as itself, in an
// order that keeps any two gates sharing a qubit in program order.  What a
// launch per gate costs is the sweep: at 25 qubits 75..91 us of memory time
// for 8 or fewer multiply-adds per amplitude, at 12 qubits a 2.5 us launch for
// 0.2 us of work.  So runs of gates share one launch: a workgroup stages a
// tile of 2^t amplitudes in LDS (t qubits that hold the run's targets; the
// lowest ones always, for contiguous runs in memory), applies the run's gates
// to it and writes it back.
//
// Inside a tile a run is cut into stages of at most four target qubits.  A
// thread takes the 16 amplitudes spanned by a stage's qubits into registers,
// applies all of the stage's gates there, and puts them back: one LDS round
// trip and one barrier per stage, no address work per gate.  Only targets need
// a tile qubit.  A control or a phase's qubit may be one of the stage's
// register qubits (a uniform choice per amplitude), another qubit of the tile
// (a choice per thread) or one outside the tile (uniform: a bit of the tile's
// base index).
//
// Measured on 25 qubits complex64 (hea, 437 gates): 35.7 ms as sweeps, 2.55 ms
// in 5 runs; on 12 qubits complex128 (360 gates) 0.91 and 0.14 ms.
//
// The run travels as a kernel argument (by value), as a layer does in
// kernels_smgp.hip: no device memory, no copy, and the launches can be
// captured.  What bounds it: vector issue, 8 multiply-adds per amplitude for
// a general gate, 4 when its matrix is real or real on and imaginary off the
// diagonal, 4 for a diagonal gate, none for a NOT or SWAP.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <utility>

#include "tile_device.h"

namespace qs {

namespace {
using namespace tiledev;

// G_SWAP is the host's: three controlled NOTs in the run
enum : uint8_t { G_DENSE = 0, G_REAL = 1, G_RX = 2, G_NOT = 3, G_PHASE = 4, G_DIAG = 5, G_SWAP = 6 };

constexpr int kMaxSlots = 4;           // register qubits of a stage, at most
constexpr int kMaxStages = 56;
constexpr int kMinQubits = 4;          // smaller states: sweeps
constexpr int kSweepQubits = 22;       // states beyond the L2s: two light gates are cheaper as sweeps (few_sweeps)
constexpr int kRunLookahead = 128;     // gates left out of a run before its search ends
constexpr uint64_t kMaxRunTiles = 1u << 20;   // tiles of one launch (a grid holds fewer than 2^32 threads)
constexpr int kNoQubit = 63;           // outside-qubit field of a gate without one (no state has such a qubit)

struct RunStage {
    uint32_t pos;                      // tile positions of the register qubits, ascending, a byte each
    uint16_t first, count;             // first word of the stage's gates, gates
};

// A gate is one 64-bit word and the values it needs, as many as its kind has:
// G_DENSE 8 (the 2x2, (re, im) row-major), G_REAL 4 (its real parts), G_RX 4
// (re 00, im 01, im 10, re 11), G_PHASE 2 (the factor), G_DIAG 4 (the factors
// for bit 0 and 1), G_NOT none.  The word: kind (4 bits), slot (4), then the
// controls (or a phase's qubits): a mask over the register qubits (8), over
// tile positions outside them (16), two global qubits outside the tile (8 each).
template <typename R>
struct GateRun {
    static constexpr int kWords = 424;
    PassArgs pa;                       // t, c, hi
    int32_t nstages;
    uint64_t tile0;                    // first tile of the launch
    uint32_t gpos[4];                  // global qubit of each tile position, a byte each
    RunStage st[kMaxStages];
    uint64_t w[kWords];
};
static_assert(sizeof(GateRun<double>) <= 4064 && sizeof(GateRun<float>) <= 4064, "a run must fit the kernel arguments");

constexpr int kGateValues[6] = {8, 4, 4, 0, 2, 4};
template <typename R>
__host__ __device__ constexpr int gate_words(int kind) {
    return 1 + kGateValues[kind] * (int)sizeof(R) / 8;
}

#define QS_INLINE __attribute__((always_inline))
#define QS_CONST __attribute__((address_space(4)))
template <int... I, typename F>
__device__ __forceinline__ void each_impl(std::integer_sequence<int, I...>, F &&f) {
    (f(std::integral_constant<int, I>()), ...);
}
template <int N, typename F>
__device__ __forceinline__ void each(F &&f) {
    each_impl(std::make_integer_sequence<int, N>(), f);
}

template <typename R, typename A>
__device__ __forceinline__ A cmul(A a, R fr, R fi) {
    A o;
    o.x = a.x * fr - a.y * fi;
    o.y = a.x * fi + a.y * fr;
    return o;
}

// (a, b) <- the 2x2 times (a, b)
template <int KIND, typename R, typename A>
__device__ __forceinline__ void pair_op(A &a, A &b, const R (&m)[8]) {
    const A x = a, y = b;
    if constexpr (KIND == G_NOT) {
        a = y;
        b = x;
    } else if constexpr (KIND == G_REAL) {
        a.x = m[0] * x.x + m[1] * y.x;
        a.y = m[0] * x.y + m[1] * y.y;
        b.x = m[2] * x.x + m[3] * y.x;
        b.y = m[2] * x.y + m[3] * y.y;
    } else if constexpr (KIND == G_RX) {
        a.x = m[0] * x.x - m[1] * y.y;
        a.y = m[0] * x.y + m[1] * y.x;
        b.x = m[3] * y.x - m[2] * x.y;
        b.y = m[3] * y.y + m[2] * x.x;
    } else {
        a.x = m[0] * x.x - m[1] * x.y + m[2] * y.x - m[3] * y.y;
        a.y = m[0] * x.y + m[1] * x.x + m[2] * y.y + m[3] * y.x;
        b.x = m[4] * x.x - m[5] * x.y + m[6] * y.x - m[7] * y.y;
        b.y = m[4] * x.y + m[5] * x.x + m[6] * y.y + m[7] * y.x;
    }
}

// The 2x2 on register qubit S, for the pairs whose other register bits hold
// every bit of rmask.
template <int KIND, int S, int NA, typename R, typename A>
__device__ __forceinline__ void slot_gate(A (&v)[NA], uint32_t rmask, const R (&m)[8]) {
    if (rmask == 0) {
        each<NA>([&](auto ic) QS_INLINE {
            constexpr int i = decltype(ic)::value;
            if constexpr (!(i & (1 << S))) pair_op<KIND, R>(v[i], v[i | (1 << S)], m);
        });
    } else {
        each<NA>([&](auto ic) QS_INLINE {
            constexpr int i = decltype(ic)::value;
            if constexpr (!(i & (1 << S)))
                if ((i & rmask) == rmask) pair_op<KIND, R>(v[i], v[i | (1 << S)], m);
        });
    }
}

// The same on register qubit `slot` (uniform).  The branches end in distinct
// markers: without them the compiler merges the ones that only differ in the
// amplitudes they move into one that indexes them by a variable, and the
// amplitudes go to scratch memory.
template <int KIND, int NA, typename R, typename A>
__device__ __forceinline__ void target_gate(A (&v)[NA], uint32_t slot, uint32_t rmask, const R (&m)[8]) {
    if (slot == 0) {
        slot_gate<KIND, 0, NA, R>(v, rmask, m);
        asm volatile("; slot 0");
        return;
    }
    if (NA == 4 || slot == 1) {
        slot_gate<KIND, 1, NA, R>(v, rmask, m);
        asm volatile("; slot 1");
        return;
    }
    if constexpr (NA >= 8) {
        if (NA == 8 || slot == 2) {
            slot_gate<KIND, 2, NA, R>(v, rmask, m);
            asm volatile("; slot 2");
            return;
        }
    }
    if constexpr (NA >= 16) {
        slot_gate<KIND, 3, NA, R>(v, rmask, m);
        asm volatile("; slot 3");
    }
}

// The run as the kernel reads it: its argument in the constant address space
// (through the by-value parameter, reads that the branches share were seen as
// reads of a private copy, and the whole table was copied to scratch memory).
template <typename R>
__device__ __forceinline__ const QS_CONST GateRun<R> *run_argument() {
    // second argument, behind one pointer
    static_assert(alignof(GateRun<R>) == 8, "argument offset");
    return (const QS_CONST GateRun<R> *)((const QS_CONST char *)__builtin_amdgcn_kernarg_segment_ptr() + 8);
}

// Applies the gate at w and returns its length in words.  base: the tile's
// first global index with bit kNoQubit set.
template <int NA, typename R, typename A>
__device__ __forceinline__ int apply_gate(A (&v)[NA], const QS_CONST uint64_t *w, uint32_t k0, uint64_t base) {
    const uint64_t code = w[0];
    const QS_CONST R *m = (const QS_CONST R *)(w + 1);
    const uint32_t kind = (uint32_t)code & 15u, slot = ((uint32_t)code >> 4) & 15u, rmask = ((uint32_t)code >> 8) & 255u;
    const uint32_t tmask = (uint32_t)code >> 16;
    const uint64_t omask = 1ull << ((code >> 32) & 63u) | 1ull << ((code >> 40) & 63u);
    if (kind == G_DIAG) {
        const R d0r = m[0], d0i = m[1], d1r = m[2], d1i = m[3];
        if (rmask) {
            each<NA>([&](auto ic) QS_INLINE {
                constexpr int i = decltype(ic)::value;
                const bool b = (i & rmask) != 0;   // uniform
                v[i] = cmul<R>(v[i], b ? d1r : d0r, b ? d1i : d0i);
            });
        } else {
            const bool b = tmask ? (k0 & tmask) != 0 : (base & omask) == omask;
            const R fr = b ? d1r : d0r, fi = b ? d1i : d0i;
            each<NA>([&](auto ic) QS_INLINE { v[ic.value] = cmul<R>(v[ic.value], fr, fi); });
        }
        return gate_words<R>(G_DIAG);
    }
    const bool on = (base & omask) == omask && (k0 & tmask) == tmask;   // per thread where tmask is set
    if (kind == G_PHASE) {
        if (on) {
            const R fr = m[0], fi = m[1];
            each<NA>([&](auto ic) QS_INLINE {
                constexpr int i = decltype(ic)::value;
                if ((i & rmask) == rmask) v[i] = cmul<R>(v[i], fr, fi);
            });
        }
        return gate_words<R>(G_PHASE);
    }
    // the values are read before the branches on slot and controls, once
    R mv[8] = {};
    if (kind == G_DENSE) {
#pragma unroll
        for (int i = 0; i < 8; ++i) mv[i] = m[i];
        if (on) target_gate<G_DENSE, NA, R>(v, slot, rmask, mv);
        return gate_words<R>(G_DENSE);
    }
    if (kind == G_REAL) {
#pragma unroll
        for (int i = 0; i < 4; ++i) mv[i] = m[i];
        if (on) target_gate<G_REAL, NA, R>(v, slot, rmask, mv);
        return gate_words<R>(G_REAL);
    }
    if (kind == G_RX) {
#pragma unroll
        for (int i = 0; i < 4; ++i) mv[i] = m[i];
        if (on) target_gate<G_RX, NA, R>(v, slot, rmask, mv);
        return gate_words<R>(G_RX);
    }
    if (on) target_gate<G_NOT, NA, R>(v, slot, rmask, mv);
    return gate_words<R>(G_NOT);
}

// One workgroup per tile; blockDim.x = max(64, 2^(t - NS)) threads, NS register
// qubits per stage.
template <typename R, int NS>
__global__ __launch_bounds__(NS == 4 ? 512 : 1024, 4) void k_gate_run(
    typename AmpOf<R>::A *__restrict__ psi, const GateRun<R> run) {
    const QS_CONST GateRun<R> *table = run_argument<R>();
    typedef R A __attribute__((ext_vector_type(2)));
    typedef R V __attribute__((ext_vector_type(16 / sizeof(R))));
    constexpr int NA = 1 << NS;                // amplitudes per thread
    constexpr uint32_t APV = 16 / sizeof(A);   // amplitudes per 16-byte vector
    constexpr int NJ = NA / APV;               // vectors per thread
    constexpr int LJ = NS - (APV == 2 ? 1 : 0);
    static_assert(NJ == 1 << LJ, "vectors per thread");
    extern __shared__ __align__(kTileAlign) unsigned char smem_raw[];
    const TileAligned tl{lds_addr(smem_raw)};
    const uint32_t tid = threadIdx.x;
    // the threads that hold the tile: all, but in tiles of fewer than 64 x 2^NS amplitudes
    const uint32_t lw = (uint32_t)run.pa.t - NS;
    const bool active = (tid >> lw) == 0;
    const uint64_t base = tile_base(run.tile0 + blockIdx.x, run.pa);
    // vector tid + j 2^lw of the tile: the thread's bits of its index and j's
    // bits, which sit at tile positions p0, p0 + 1, ...
    const uint32_t p0 = lw + (APV == 2 ? 1 : 0);
    const uint32_t my_li = (tid & ((1u << lw) - 1)) * APV;
    const uint64_t g_t = base | tile_offset(my_li, run.pa);
    const uint32_t h_t = tl.grp(sw(my_li) * (uint32_t)sizeof(A));
    uint64_t gb[LJ];
    uint32_t lb[LJ];
#pragma unroll
    for (int j = 0; j < LJ; ++j) {
        const uint32_t p = p0 + j;
        gb[j] = 1ull << ((run.gpos[p >> 2] >> (8 * (p & 3))) & 255u);
        lb[j] = sw(1u << p) * (uint32_t)sizeof(A);
    }
    auto vec_g = [&](int j) {
        uint64_t o = 0;
#pragma unroll
        for (int b = 0; b < LJ; ++b)
            if ((j >> b) & 1) o |= gb[b];
        return reinterpret_cast<V *>(psi + (g_t | o));
    };
    auto vec_l = [&](int j) {
        uint32_t o = 0;
#pragma unroll
        for (int b = 0; b < LJ; ++b)
            if ((j >> b) & 1) o ^= lb[b];
        return tl.template at<V>(h_t, o);
    };
    if (active) {
        V pre[NJ];
#pragma unroll
        for (int j = 0; j < NJ; ++j) pre[j] = *vec_g(j);
#pragma unroll
        for (int j = 0; j < NJ; ++j) *vec_l(j) = pre[j];
    }
    // The run's records reach the scalar cache with all of their misses in
    // flight at once; met one by one they are a good part of a short launch
    // (12 qubits: 97 -> 79 us for 200 gates).  Long launches hide them, and
    // pay 1..3 % for the extra reads.
    if (gridDim.x <= 128) {
        const QS_CONST uint32_t *w = (const QS_CONST uint32_t *)table;
        uint32_t touched = 0;
#pragma unroll
        for (uint32_t i = 0; i < sizeof(run) / 64; ++i) touched |= w[16 * i];
        asm volatile("" ::"s"(touched));
    }
    for (int s = 0; s < run.nstages; ++s) {
        const uint32_t sp = table->st[s].pos;
        const int ngates = table->st[s].count;
        __syncthreads();
        if (!active) continue;
        uint32_t k0 = tid, ob[NS];
#pragma unroll
        for (int j = 0; j < NS; ++j) {
            const int p = (sp >> (8 * j)) & 255u;
            k0 = ins0_32(k0, p);
            ob[j] = sw(1u << p) * (uint32_t)sizeof(A);
        }
        const uint32_t h = tl.grp(sw(k0) * (uint32_t)sizeof(A));
        auto slot = [&](int i) {
            uint32_t o = 0;
#pragma unroll
            for (int j = 0; j < NS; ++j)
                if ((i >> j) & 1) o ^= ob[j];
            return tl.template at<A>(h, o);
        };
        A v[NA];
        each<NA>([&](auto ic) QS_INLINE { v[ic.value] = *slot(ic.value); });
        const QS_CONST uint64_t *w = table->w + table->st[s].first;
        for (int gi = 0; gi < ngates; ++gi) w += apply_gate<NA, R>(v, w, k0, base | 1ull << kNoQubit);
        each<NA>([&](auto ic) QS_INLINE { *slot(ic.value) = v[ic.value]; });
    }
    __syncthreads();
    if (active) {
        V out[NJ];
#pragma unroll
        for (int j = 0; j < NJ; ++j) out[j] = *vec_l(j);
#pragma unroll
        for (int j = 0; j < NJ; ++j) *vec_g(j) = out[j];
    }
}

// ------------------------------------------------------------ host side
// A gate as a run sees it: targets (qubits a tile must hold), every qubit it
// touches, and the bytes its own sweep would move, in states.
struct RunItem {
    const HGate *src = nullptr;
    uint8_t kind = G_DENSE;
    uint64_t targets = 0, qubits = 0, mask = 0;   // mask: controls, or the qubits of a phase or diagonal
    cd m[4];
    double sweep = 2.0;
    bool alone = false;                           // dense gates of two or more qubits: a sweep of their own
};

uint8_t target_kind(const cd *m) {
    const cd zero(0, 0), one(1, 0);
    if (m[0] == zero && m[3] == zero && m[1] == one && m[2] == one) return G_NOT;
    bool real = true, rx = true;
    for (int i = 0; i < 4; ++i) {
        real &= m[i].imag() == 0.0;
        rx &= (i == 0 || i == 3) ? m[i].imag() == 0.0 : m[i].real() == 0.0;
    }
    return real ? G_REAL : rx ? G_RX : G_DENSE;
}

// false: the identity, nothing to do
bool run_item(const HGate &g, RunItem &it) {
    it.src = &g;
    for (int j = 0; j < g.nq; ++j) it.qubits |= 1ull << g.q[j];
    if (g.nq == 1) {
        for (int i = 0; i < 4; ++i) it.m[i] = g.m[i];
        if (g.m[1] == cd(0, 0) && g.m[2] == cd(0, 0)) {
            it.mask = it.qubits;
            if (g.m[0] == cd(1, 0)) {
                it.kind = G_PHASE;
                it.m[0] = g.m[3];
                it.sweep = 1.0;
                return g.m[3] != cd(1, 0);
            }
            it.kind = G_DIAG;
            it.m[1] = g.m[3];
            return true;
        }
        it.targets = it.qubits;
        it.kind = target_kind(it.m);
        return true;
    }
    switch (g.kind) {
    case QS_CZ:
    case QS_CP:
        it.kind = G_PHASE;
        it.mask = it.qubits;
        it.m[0] = g.m[3 * 4 + 3];
        it.sweep = 0.5;
        return true;
    case QS_CNOT:
    case QS_CU:
        // local index: bit 0 = control, bit 1 = target
        for (int a = 0; a < 2; ++a)
            for (int b = 0; b < 2; ++b) it.m[2 * a + b] = g.m[(1 + 2 * a) * 4 + (1 + 2 * b)];
        it.kind = target_kind(it.m);
        it.targets = 1ull << g.q[1];
        it.mask = 1ull << g.q[0];
        it.sweep = 1.0;
        return true;
    case QS_SWAP:
        it.kind = G_SWAP;
        it.targets = it.qubits;
        it.sweep = 1.0;
        return true;
    default:
        it.alone = true;
        it.targets = it.qubits;
        return true;
    }
}

// Tile and register qubits of a run on n qubits.  Below about 2^21 amplitudes
// the chip is not full and a run's time is the chain of its gates: small tiles
// spread it over more CUs, and four amplitudes per thread (two register
// qubits) give a tile four times the waves of sixteen and code that fits the
// instruction cache (14 qubits, hea of 5 layers: 87 us, 2^12-amplitude tiles
// 120 us, sixteen amplitudes 145 us or more; a quarter less on 12 qubits).
// Full chips are bound by vector issue and LDS round trips: complex64 then
// takes four register qubits (25 qubits: 2.57 ms against 4.38 ms with two),
// complex128 stays at two, whose registers allow twice the waves (24 qubits:
// 2.6 ms against 2.8 ms).
void run_shape(int n, qs_dtype dt, int &t, int &ns) {
    const int full = dt == QS_C64 ? 21 : 22;   // qubits from which on every CU has tiles enough
    ns = dt == QS_C64 && n >= full ? 4 : 2;
    t = n >= full ? (dt == QS_C64 ? 12 : 11) : n >= 20 ? 12 : 10;
    t = std::min(t, n);
}

// What a gate's own sweep reads and writes, in states, with whole 128-byte
// lines: a control, phase or SWAP qubit among the lowest leaves no line out.
double sweep_lines(const RunItem &it, int n, qs_dtype dt) {
    const uint64_t in_line = dt == QS_C64 ? 15 : 7;
    switch (it.kind) {
    case G_SWAP: return it.qubits & in_line ? 2.0 : 1.0;
    case G_DIAG: return 2.0;
    default: break;
    }
    if (!it.mask) return 2.0;   // an uncontrolled target
    double w = 2.0;
    for (uint64_t b = it.mask & ~in_line; b; b &= b - 1) w *= 0.5;
    // complex64 sweeps of controlled gates lose a quarter on states that the
    // memory-side cache holds (128 and 256 MiB)
    return it.targets && dt == QS_C64 && (n == 24 || n == 25) ? 1.25 * w : w;
}

// Whether the gates of a would-be run go as sweeps of their own.  A run moves
// 2 states; two sweeps that move one each take the same traffic with less work
// around it, and the second finds part of the first's output in a cache.
// Two SWAPs, far qubits: 26 qubits complex64 158 us as sweeps, 199 as a run,
// 23 qubits 18 and 28, 22 qubits complex128 18 and 27; two controlled gates on
// 25 qubits: complex128 156 and 206, complex64 96 and 70.
bool few_sweeps(const std::vector<const RunItem *> &taken, int n, qs_dtype dt) {
    double sweep = 0, lines = 0;
    bool swaps = true;
    for (const RunItem *it : taken) {
        sweep += it->sweep;
        lines += sweep_lines(*it, n, dt);
        swaps &= it->kind == G_SWAP;
    }
    // SWAPs alone, which only move amplitudes, from 32 MiB on (21 qubits
    // complex128: 10.3 us as sweeps, 13.7 as a run)
    if (swaps && lines <= 2.0 && n >= (dt == QS_C64 ? 22 : 21)) return true;
    if (n < kSweepQubits) return false;
    // more than two sweeps only on states that no cache holds (four CZ on 24
    // qubits complex64 47 us against 44, on 26 qubits 176 against 202)
    const bool far = n > (dt == QS_C64 ? 25 : 24);
    return sweep <= 1.5 || (lines <= 2.0 && (taken.size() == 2 || far) && (dt == QS_C128 || n > kSweepQubits));
}

int item_words(const RunItem &it, qs_dtype dt) {
    if (it.kind == G_SWAP) return 3 * gate_words<float>(G_NOT);
    return dt == QS_C64 ? gate_words<float>(it.kind) : gate_words<double>(it.kind);
}

// values of a gate record, see GateRun
template <typename R>
void put_values(const RunItem &it, R *m) {
    switch (it.kind) {
    case G_REAL:
        for (int i = 0; i < 4; ++i) m[i] = (R)it.m[i].real();
        break;
    case G_RX:
        for (int i = 0; i < 4; ++i) m[i] = (R)(i == 0 || i == 3 ? it.m[i].real() : it.m[i].imag());
        break;
    case G_NOT: break;
    default:   // G_DENSE, G_PHASE, G_DIAG: (re, im) of the first 4, 1 or 2
        for (int i = 0; i < kGateValues[it.kind] / 2; ++i) {
            m[2 * i] = (R)it.m[i].real();
            m[2 * i + 1] = (R)it.m[i].imag();
        }
    }
}

// Launches the items (whose targets with the lowest qubits make `targets`, at
// most t qubits) as one run.  Items beyond its stage table stay in `pending`.
template <typename R>
qs_status launch_run(qs_state_s &s, std::vector<const RunItem *> &pending, uint64_t targets, int t, int ns) {
    using A = typename AmpOf<R>::A;
    GateRun<R> run;
    std::memset(&run, 0, sizeof run);
    // tile: the targets (the lowest qubits among them), filled up with the lowest others
    uint64_t tile = targets;
    for (int q = 0; q < s.n && __builtin_popcountll(tile) < t; ++q) tile |= 1ull << q;
    int pos_of[64];
    int t_used = 0;
    run.pa.t = t;
    for (int q = 0; q < s.n; ++q) {
        if (!((tile >> q) & 1)) continue;
        if (q == run.pa.c) ++run.pa.c;
        else run.pa.hi[t_used - run.pa.c] = q;
        run.gpos[t_used >> 2] |= (uint32_t)q << (8 * (t_used & 3));
        pos_of[q] = t_used++;
    }
    QS_CHECK(t_used == t && run.pa.c >= 1, QS_EINVAL, "internal: gate run tile of %d qubits, want %d", t_used, t);
    // stages: gates in order; one that would need more register qubits than a
    // stage has, or shares a qubit with a gate left out, waits for a later stage
    std::vector<const RunItem *> taken, rest;
    int nw = 0;
    double flops = 0;
    while (!pending.empty() && run.nstages < kMaxStages) {
        RunStage &st = run.st[run.nstages++];
        uint64_t cur = 0, blocked = 0;
        taken.clear();
        rest.clear();
        for (const RunItem *it : pending) {
            if (!(it->qubits & blocked) && __builtin_popcountll(cur | it->targets) <= ns) {
                cur |= it->targets;
                taken.push_back(it);
            } else {
                blocked |= it->qubits;
                rest.push_back(it);
            }
        }
        // fill up with the highest tile qubits (their groups are contiguous runs of lanes)
        for (int q = s.n - 1; q >= 0 && __builtin_popcountll(cur) < ns; --q)
            if ((tile >> q) & 1) cur |= 1ull << q;
        int slot_of[64], k = 0;
        for (int q = 0; q < s.n; ++q)
            if ((cur >> q) & 1) {
                st.pos |= (uint32_t)pos_of[q] << (8 * k);
                slot_of[q] = k++;
            }
        st.first = (uint16_t)nw;
        auto put = [&](int kind, uint32_t slot, uint32_t rmask, uint32_t tmask, const int *out) {
            run.w[nw] = (uint64_t)((uint32_t)kind | slot << 4 | rmask << 8 | tmask << 16) | (uint64_t)out[0] << 32 |
                        (uint64_t)out[1] << 40;
            ++st.count;
        };
        for (const RunItem *it : taken) {
            int out[2] = {kNoQubit, kNoQubit}, nout = 0;
            if (it->kind == G_SWAP) {
                const uint32_t sa = (uint32_t)slot_of[__builtin_ctzll(it->targets)];
                const uint32_t sb = (uint32_t)slot_of[63 - __builtin_clzll(it->targets)];
                for (int i = 0; i < 3; ++i, ++nw) put(G_NOT, i == 1 ? sa : sb, 1u << (i == 1 ? sb : sa), 0, out);
                continue;
            }
            uint32_t rmask = 0, tmask = 0;
            for (uint64_t b = it->mask; b; b &= b - 1) {
                const int q = __builtin_ctzll(b);
                if ((cur >> q) & 1) rmask |= 1u << slot_of[q];
                else if ((tile >> q) & 1) tmask |= 1u << pos_of[q];
                else out[nout++] = q;   // at most two qubits in a mask
            }
            put(it->kind, it->targets ? (uint32_t)slot_of[__builtin_ctzll(it->targets)] : 0, rmask, tmask, out);
            put_values<R>(*it, reinterpret_cast<R *>(run.w + nw + 1));
            nw += gate_words<R>(it->kind);
            flops += (it->kind >= G_PHASE ? 3.0 : 7.0) * it->sweep * std::ldexp(1.0, s.n);
        }
        pending.swap(rest);
    }
    const uint64_t ntiles = 1ull << (s.n - t);
    const unsigned threads = std::max(64u, 1u << (t - ns));
    const size_t lds = sizeof(A) << t;
    void (*kernel)(A *, GateRun<R>) = k_gate_run<R, 2>;
    if constexpr (sizeof(R) == 4) {
        if (ns == 4) kernel = k_gate_run<R, 4>;
    }
    const void *fn = reinterpret_cast<const void *>(kernel);
    QS_CHECK(dynamic_tile_at_zero(fn), QS_EDEVICE, "gate run kernel declares static LDS");
    QS_HIP(set_dynamic_lds(fn, lds));
    prof_begin(s.stream, QS_PROF_PLAIN, 2 * std::ldexp((double)sizeof(A), s.n), flops);
    for (run.tile0 = 0; run.tile0 < ntiles; run.tile0 += kMaxRunTiles)
        hipLaunchKernelGGL(kernel, dim3((unsigned)std::min(ntiles - run.tile0, kMaxRunTiles)), dim3(threads), lds,
                           s.stream, (A *)s.amp, run);
    prof_end(s.stream);
    QS_HIP(hipGetLastError());
    return QS_OK;
}

}  // namespace

qs_status launch_gates(qs_state_s &s, const std::vector<HGate> &gates) {
    // states of a few amplitudes, a single gate: sweeps
    if (s.n < kMinQubits || gates.size() < 2) {
        for (const HGate &g : gates) {
            const qs_status st = launch_plain(s, g);
            if (st != QS_OK) return st;
        }
        return QS_OK;
    }
    std::vector<RunItem> all(gates.size());
    int t, ns;
    run_shape(s.n, s.dtype, t, ns);
    const int cap = GateRun<float>::kWords;
    const uint64_t low = (1ull << std::min(4, t - 2)) - 1;   // always in the tile: runs of 16 amplitudes
    std::vector<const RunItem *> carry, next, taken;
    size_t pos = 0;
    while (pos < gates.size() || !carry.empty()) {
        // list scheduling, as for passes of blocks: a gate that does not fit
        // waits, and so does every later gate that shares a qubit with it
        uint64_t cur = low, blocked = 0;
        int words = 0;
        taken.clear();
        next.clear();
        const RunItem *alone = nullptr;
        size_t ci = 0;
        while (next.size() < kRunLookahead) {
            const RunItem *it;
            if (ci < carry.size()) {
                it = carry[ci++];
            } else if (pos < gates.size()) {
                RunItem &n = all[pos];
                if (!run_item(gates[pos++], n)) continue;
                it = &n;
            } else {
                break;
            }
            if (it->alone && taken.empty() && next.empty()) {
                alone = it;
                break;
            }
            const int need = it->alone ? 0 : item_words(*it, s.dtype);
            if (words + need > cap) {
                next.push_back(it);
                break;
            }
            if (!it->alone && !(it->qubits & blocked) && __builtin_popcountll(cur | it->targets) <= t) {
                cur |= it->targets;
                words += need;
                taken.push_back(it);
            } else {
                blocked |= it->qubits;
                next.push_back(it);
            }
        }
        next.insert(next.end(), carry.begin() + (int64_t)ci, carry.end());
        qs_status st = QS_OK;
        if (alone) {
            st = launch_plain(s, *alone->src);
        } else if (taken.size() == 1 || few_sweeps(taken, s.n, s.dtype)) {
            for (const RunItem *it : taken) {
                st = launch_plain(s, *it->src);
                if (st != QS_OK) return st;
            }
            taken.clear();
        } else if (!taken.empty()) {
            st = s.dtype == QS_C64 ? launch_run<float>(s, taken, cur, t, ns) : launch_run<double>(s, taken, cur, t, ns);
        }
        if (st != QS_OK) return st;
        // what a run had no stages for goes before what was left out of it
        // (no gate left out shares a qubit with a later gate that was taken)
        carry.swap(taken);
        carry.insert(carry.end(), next.begin(), next.end());
    }
    return QS_OK;
}

}  // namespace qs
