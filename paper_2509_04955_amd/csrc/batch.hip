// Batches of independent states, run by one hipGraph launch.
//
// Each state (its own qubit count, circuit and Pauli-sum Hamiltonian) gets a
// contraction plan.  Level p of the graph is one launch that runs pass p of
// every state that has one: its items are runs of consecutive tiles of one
// state's pass, listed in a device table and started in order of falling cost
// (a state of one tile has all of its blocks in level 0, in one workgroup).
// Two more launches evaluate every state's Hamiltonian by groups of terms,
// one read of the state per group (kernels_expect.hip), and sum the energies.
// Kernel boundaries order the levels.  A single persistent kernel with a work
// queue and per-state counters in their place was measured slower: every item
// then pays a device-scope release and acquire, which write back and
// invalidate the XCD's L2, and waiting workgroups go on doing so.  64 states
// of 12..21 qubits (8 layers, 200 terms each, k_max 4, 12-qubit tiles) took 84
// ms for their passes and 8 ms for the energies, 4 states no less; as levels
// they take 4.2 ms (26 launches of 162 us on average) and 2.1 ms, 4 states 0.8 ms.
//
// The renormalisation scale of pass p is the fixed-order FP64 sum of pass
// p-1's item partials, recomputed by every consumer, so all of them see the
// same value.  Level 0 starts from |0...0> without reading the state: its
// tiles are zero but for amplitude 0, and every amplitude is written.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <map>
#include <memory>
#include <new>

#include "tile_device.h"

namespace qs {
const char *last_error();

namespace {
using namespace tiledev;

struct PassDev {
    PassArgs pa;             // block0 and the blocks' operands count from the batch's tables,
    uint64_t pool_off;       // the operands from here on (reals)
    uint64_t amp_off;        // bytes
    uint64_t prev_part_off;  // previous pass's partials
    uint32_t prev_nparts;    // 0 for the first pass
    uint32_t pad;
};

// one workgroup's work: tiles [tile0, tile0 + ntiles) of a pass
struct PassItem {
    uint32_t pass;
    uint32_t tile0;
    uint32_t ntiles;
    uint32_t part;           // the item's norm partial
};

// Norm slots behind the tile in the (dynamic) LDS region.
constexpr size_t kBatchRedBytes = TT / 64 * sizeof(double);

// Fixed-order FP64 sum of one value per thread over the workgroup.
__device__ __forceinline__ double wg_sum_values(double s, double *red) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) s += __shfl_xor(s, o);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
    __syncthreads();
    double t = 0;
#pragma unroll
    for (int w = 0; w < TT / 64; ++w) t += red[w];
    return t;
}

// Consecutive tiles of one pass of one state: each tile is loaded into LDS,
// every block of the pass is applied, and the tile is written back; the
// item's FP64 norm partial is the sum over its tiles.  The next tile's first
// kBatchPrefetch vectors per thread are loaded into registers while the
// current tile is processed (as in the single-state pass kernel); the rest
// follow in batches.
constexpr int kBatchPrefetch = 4;

template <typename R, bool WIDE>
__global__ __launch_bounds__(TT, WIDE ? 1 : 2) void k_batch_pass(const PassItem *__restrict__ items,
                                                                 const PassDev *__restrict__ passes,
                                                                 const BlockDev *__restrict__ blocks,
                                                                 const R *__restrict__ pools,
                                                                 unsigned char *__restrict__ amps,
                                                                 double *__restrict__ partials) {
    using A = typename AmpOf<R>::A;
    constexpr bool F32 = sizeof(R) == 4;
    constexpr uint32_t APV = F32 ? 2 : 1;
    constexpr int PF = kBatchPrefetch;
    extern __shared__ __align__(kTileAlign) unsigned char smem_raw[];
    const PassItem it = items[blockIdx.x];
    const PassDev &pd = passes[it.pass];
    const PassArgs &pa = pd.pa;
    A *psi = reinterpret_cast<A *>(amps + pd.amp_off);
    const TileAligned tl{lds_addr(smem_raw)};
    double *red = reinterpret_cast<double *>(smem_raw + (sizeof(A) << pa.t));
    const uint32_t nvec = (1u << pa.t) / APV;
    const uint32_t nj = (nvec + TT - 1) / TT;   // vectors per thread
    float4 pre[PF];
    auto gptr = [&](uint64_t base, uint32_t vi) {
        return reinterpret_cast<float4 *>(psi + (base | tile_offset(vi * APV, pa)));
    };
    auto slot = [&](uint32_t vi) {
        return tl.template at<float4>(tl.grp(sw(vi * APV) * (uint32_t)sizeof(A)), 0u);
    };
    const uint64_t t1 = (uint64_t)it.tile0 + it.ntiles;
    uint64_t tid = it.tile0;
    uint64_t base = tile_base(tid, pa);
    const bool first = pd.prev_nparts == 0;
    R sc = (R)1;
    auto load = [&](uint64_t b, uint32_t j0) {
#pragma unroll
        for (int i = 0; i < PF; ++i) {
            const uint32_t vi = threadIdx.x + (j0 + i) * TT;
            if (vi < nvec) pre[i] = *gptr(b, vi);
        }
    };
    auto put = [&](uint32_t j0) {
#pragma unroll
        for (int i = 0; i < PF; ++i) {
            const uint32_t vi = threadIdx.x + (j0 + i) * TT;
            if (vi >= nvec) continue;
            float4 v = pre[i];
            if constexpr (F32) {
                v.x *= sc;
                v.y *= sc;
                v.z *= sc;
                v.w *= sc;
            } else {
                double2 d = __builtin_bit_cast(double2, v);
                d.x *= sc;
                d.y *= sc;
                v = __builtin_bit_cast(float4, d);
            }
            *slot(vi) = v;
        }
    };
    // LDS <- the tile at b whose first PF vectors per thread are in registers
    auto stage = [&](uint64_t b) {
        put(0);
        for (uint32_t j0 = PF; j0 < nj; j0 += PF) {
            load(b, j0);
            put(j0);
        }
    };
    auto stage_basis = [&](uint64_t b) {
        for (uint32_t vi = threadIdx.x; vi < nvec; vi += TT) {
            float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
            if (b == 0 && vi == 0) {
                if constexpr (F32) v.x = 1.f;
                else v = __builtin_bit_cast(float4, make_double2(1.0, 0.0));
            }
            *slot(vi) = v;
        }
    };
    if (first) {
        stage_basis(base);
    } else {
        load(base, 0);
        double s = 0;
        for (uint32_t i = threadIdx.x; i < pd.prev_nparts; i += TT) s += partials[pd.prev_part_off + i];
        const double N = wg_sum_values(s, red);
        sc = (R)(N > 0 ? 1.0 / sqrt(N) : 1.0);
        stage(base);
    }
    const R *pool = pools + pd.pool_off;
    double nacc = 0;
    for (;;) {
        __syncthreads();
        const bool more = tid + 1 < t1;
        const uint64_t nbase = more ? tile_base(tid + 1, pa) : base;
        if (more && !first) load(nbase, 0);
        for (int b = 0; b < pa.nblocks; ++b) {
            apply_block<R, WIDE, false, TT, false>(tl, pa.t, blocks + pa.block0 + b, pool, base);
            __syncthreads();
        }
        for (uint32_t vi = threadIdx.x; vi < nvec; vi += TT) {
            const float4 v = *slot(vi);
            *gptr(base, vi) = v;
            if constexpr (F32) {
                nacc += (double)v.x * v.x + (double)v.y * v.y + (double)v.z * v.z + (double)v.w * v.w;
            } else {
                const double2 d = __builtin_bit_cast(double2, v);
                nacc += d.x * d.x + d.y * d.y;
            }
        }
        if (!more) break;
        __syncthreads();   // every read of this tile from LDS is done
        if (first) stage_basis(nbase);
        else stage(nbase);
        ++tid;
        base = nbase;
    }
    const double tot = wg_sum_values(nacc, red);
    if (threadIdx.x == 0) partials[it.part] = tot;
}

}  // namespace
}  // namespace qs

using namespace qs;

struct qs_batch_s {
    qs_dtype dtype = QS_C64;
    hipStream_t stream = nullptr;
    int nstates = 0;
    std::vector<qs_plan_s *> plans;
    std::vector<int> n;
    std::vector<uint64_t> amp_off;  // bytes
    void *d_amps = nullptr;
    uint64_t amp_bytes = 0;
    struct Level {
        uint32_t first, count;   // items
        size_t lds;
        bool wide;
    };
    std::vector<Level> levels;
    struct LastPass {
        uint64_t off;
        uint32_t n;
    };
    std::vector<LastPass> last;      // partials of each state's last pass (norm of the stored state)
    PassItem *d_items = nullptr;
    PassDev *d_passes = nullptr;
    BlockDev *d_blocks = nullptr;    // every plan's blocks
    void *d_pools = nullptr;         // and operands
    ExpectJob *d_jobs = nullptr;
    ExpectItem *d_eitems = nullptr;  // items of full cosets, then of small ones
    uint32_t n_full = 0, n_small = 0;
    ExpectGroup *d_groups = nullptr;
    ExpectTerm *d_terms = nullptr;
    double *d_coeff = nullptr, *d_partials = nullptr, *d_eparts = nullptr;
    double *h_energy = nullptr;      // pinned host memory the energy kernel writes
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
    ~qs_batch_s() {
        if (exec) hipGraphExecDestroy(exec);
        if (graph) hipGraphDestroy(graph);
        void *bufs[] = {d_amps, d_items, d_passes, d_blocks, d_pools, d_jobs, d_eitems, d_groups, d_terms, d_coeff, d_partials, d_eparts};
        for (void *b : bufs)
            if (b) hipFree(b);
        if (h_energy) hipHostFree(h_energy);
        for (qs_plan_s *p : plans) qs_plan_destroy(p);
    }
};

namespace {

template <typename T>
qs_status upload(T **dst, const std::vector<T> &src) {
    QS_HIP(hipMalloc((void **)dst, std::max<size_t>(1, src.size()) * sizeof(T)));
    if (!src.empty()) QS_HIP(hipMemcpy(*dst, src.data(), src.size() * sizeof(T), hipMemcpyHostToDevice));
    return QS_OK;
}

template <typename R>
using BatchKernel = void (*)(const PassItem *, const PassDev *, const BlockDev *, const R *, unsigned char *, double *);

template <typename R>
BatchKernel<R> batch_kernel(bool wide) {
    return wide ? k_batch_pass<R, true> : k_batch_pass<R, false>;
}

template <typename R>
void enqueue_levels(const qs_batch_s &b, hipStream_t st) {
    for (const qs_batch_s::Level &lv : b.levels)
        for (uint32_t i = 0, m; i < lv.count; i += m) {
            m = std::min(lv.count - i, kMaxBatchGrid);
            hipLaunchKernelGGL(batch_kernel<R>(lv.wide), dim3(m), dim3(TT), lv.lds, st, b.d_items + lv.first + i,
                               b.d_passes, b.d_blocks, (const R *)b.d_pools, (unsigned char *)b.d_amps, b.d_partials);
        }
}

qs_status enqueue_batch(qs_batch_s &b, hipStream_t st) {
    if (b.dtype == QS_C64) enqueue_levels<float>(b, st);
    else enqueue_levels<double>(b, st);
    launch_expect_jobs(st, b.dtype,
                       ExpectJobs{b.d_jobs, b.d_groups, b.d_terms, b.d_coeff, b.d_amps, b.d_eparts, b.nstates, b.d_eitems,
                                  b.n_full, b.n_small},
                       b.h_energy);
    QS_HIP(hipGetLastError());
    return QS_OK;
}

}  // namespace

extern "C" {

qs_status qs_batch_create(int n_states, const int *n_qubits, const qs_gate *const *circuits, const size_t *n_gates,
                          const uint64_t *const *x, const uint64_t *const *z, const double *const *coeff,
                          const size_t *n_terms, const qs_contract_opts *opts, void *stream, qs_batch *out) {
    QS_ABI_TRY
    QS_CHECK(out && n_qubits && circuits && n_gates && x && z && coeff && n_terms, QS_EINVAL, "null argument");
    QS_CHECK(n_states >= 1 && n_states <= 65536, QS_EINVAL, "n_states %d outside 1..65536", n_states);
    qs_contract_opts base{};
    if (opts) base = *opts;
    if (base.strategy == 0 && !opts) base.strategy = QS_STRATEGY_GREEDY;
    if (!opts) base.renorm = 1;
    const qs_dtype dt = base.dtype == QS_C128 ? QS_C128 : QS_C64;
    for (int i = 0; i < n_states; ++i) {
        QS_CHECK(n_qubits[i] >= 1 && n_qubits[i] <= 26, QS_EINVAL, "state %d: n=%d outside 1..26", i, n_qubits[i]);
        QS_CHECK(n_terms[i] >= 1 && n_terms[i] <= (1u << 16), QS_EINVAL, "state %d: n_terms outside 1..65536", i);
        const uint64_t lim = (1ull << n_qubits[i]) - 1;
        for (size_t k = 0; k < n_terms[i]; ++k)
            QS_CHECK((x[i][k] & ~lim) == 0 && (z[i][k] & ~lim) == 0, QS_EINVAL, "state %d term %zu out of range", i, k);
    }
    qs_batch_s *b = new (std::nothrow) qs_batch_s();
    QS_CHECK(b != nullptr, QS_ENOMEM, "host allocation failed");
    b->dtype = dt;
    b->stream = (hipStream_t)stream;
    b->nstates = n_states;
    std::unique_ptr<qs_batch_s> own(b);   // released to the caller at the end
    auto fail = [](qs_status s) { return s; };
    // ---- plans (autotuned per qubit count when k_max or tile is 0) ----
    std::map<int, qs_contract_opts> tuned;
    std::vector<unsigned char> pools, image;   // every plan's operands
    std::vector<size_t> pool0(n_states);
    const int di = dt == QS_C64 ? 0 : 1;
    for (int i = 0; i < n_states; ++i) {
        qs_contract_opts o = base;
        o.dtype = dt;
        if (base.k_max == 0 || base.tile_qubits == 0) {
            auto it = tuned.find(n_qubits[i]);
            if (it == tuned.end()) {
                qs_contract_opts best{};
                qs_status st = qs_autotune(n_qubits[i], dt, circuits[i], n_gates[i], &o, &best);
                if (st != QS_OK) return fail(st);
                it = tuned.emplace(n_qubits[i], best).first;
            }
            o = it->second;
        }
        // The batch kernel applies complex128 blocks wider than 3 qubits on the
        // vector ALU in its wide variant (no staged FP64 MFMA there), which the
        // single-state timings of the autotuner do not see: keep them narrow.
        if (dt == QS_C128 && (base.k_max == 0 || base.tile_qubits == 0)) o.k_max = std::min(o.k_max, 3);
        // The single-state pass kernel runs 2^13- and 2^14-amplitude tiles with
        // 512 and 1024 threads; the batch kernel has 256, where such tiles hold
        // a CU to one or two workgroups.  Tuned tiles stay at 2^12 here.
        if ((base.k_max == 0 || base.tile_qubits == 0) && o.tile_qubits > 12) o.tile_qubits = 12;
        qs_plan p = nullptr;
        qs_status st = qs_contract(n_qubits[i], circuits[i], n_gates[i], &o, &p);
        if (st != QS_OK) {
            std::string m = last_error();
            set_error("state %d: %s", i, m.c_str());
            return fail(st);
        }
        b->plans.push_back(p);
        b->n.push_back(n_qubits[i]);
        st = plan_image(*p, dt, false, image);
        if (st != QS_OK) return fail(st);
        pool0[i] = pools.size();
        pools.insert(pools.end(), image.begin(), image.begin() + (int64_t)p->pool_bytes[di]);
        pools.resize((pools.size() + 255) / 256 * 256);
    }
    // ---- device layout ----
    const size_t ab = dt == QS_C64 ? 8 : 16;
    uint64_t off = 0;
    for (int i = 0; i < n_states; ++i) {
        b->amp_off.push_back(off);
        off += ((ab << b->n[i]) + 255) / 256 * 256;
    }
    b->amp_bytes = off;
    hipError_t e = hipMalloc(&b->d_amps, off);
    if (e != hipSuccess) return fail(hip_fail(e, "hipMalloc(batch states)"));
    // ---- levels: pass p of every state that has one ----
    size_t maxpasses = 0;
    for (int i = 0; i < n_states; ++i) {
        if (b->plans[i]->passes.empty()) {
            set_error("state %d has an empty circuit", i);
            return fail(QS_EINVAL);
        }
        maxpasses = std::max(maxpasses, b->plans[i]->passes.size());
    }
    int dev = 0;
    hipDeviceProp_t prop;
    e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipGetDeviceProperties(&prop, dev);
    if (e != hipSuccess) return fail(hip_fail(e, "device properties"));
    const uint64_t cus = std::max(1, prop.multiProcessorCount);
    // one table of blocks and one of operands: kernel arguments, so that the
    // wave-uniform reads of block records and matrices are scalar loads
    std::vector<BlockDev> blocks;
    std::vector<size_t> block0(n_states);
    for (int i = 0; i < n_states; ++i) {
        const qs_plan_s &p = *b->plans[i];
        block0[i] = blocks.size();
        blocks.insert(blocks.end(), p.h_blocks[di].begin(), p.h_blocks[di].end());
    }
    QS_CHECK(blocks.size() <= 0x7fffffffu, QS_ERANGE, "batch has more than 2^31 blocks");
    qs_status st = upload(&b->d_blocks, blocks);
    if (st == QS_OK) st = upload((unsigned char **)&b->d_pools, pools);
    if (st != QS_OK) return fail(st);
    std::vector<PassDev> pdv;
    std::vector<PassItem> items;
    b->last.assign(n_states, qs_batch_s::LastPass{0, 0});
    uint64_t parts = 0;
    for (size_t pi = 0; pi < maxpasses; ++pi) {
        qs_batch_s::Level lv{(uint32_t)items.size(), 0, 0, false};
        uint64_t tiles = 0;
        for (int i = 0; i < n_states; ++i)
            if (pi < b->plans[i]->passes.size()) tiles += 1ull << (b->n[i] - b->plans[i]->passes[pi].t);
        // tiles per item: 1 until the level has 24 items per CU (six rounds of the
        // four workgroups a CU holds), then more, so that an item's next tile is
        // in flight during its current one; 16 at most, but enough that a pass
        // leaves at most 2^11 partials for its consumers to add.  Few long items
        // leave the last round nearly empty: with 6 per CU, 256 states took 16.6
        // ms for their passes, with 24 14.6 (64 states 4.3 and 4.2).
        uint64_t per_level = 1;
        while (per_level < 16 && tiles / (2 * per_level) >= 24 * cus) per_level *= 2;
        struct Cost {
            double c;
            PassItem it;
        };
        std::vector<Cost> level;
        for (int i = 0; i < n_states; ++i) {
            const qs_plan_s &p = *b->plans[i];
            if (pi >= p.passes.size()) continue;
            const HPass &ps = p.passes[pi];
            const uint64_t ntiles = 1ull << (b->n[i] - ps.t);
            uint64_t per = std::min(per_level, ntiles);
            while (ntiles / per > 2048) per *= 2;
            PassDev d;
            std::memset(&d, 0, sizeof d);
            d.pa.t = ps.t;
            d.pa.c = ps.c;
            d.pa.nblocks = (int32_t)ps.nblocks;
            d.pa.block0 = (int32_t)(block0[i] + ps.block0);
            for (int j = 0; j < ps.t - ps.c; ++j) d.pa.hi[j] = ps.tile[ps.c + j];
            d.pa.want_norm = 1;
            d.pool_off = pool0[i] / (dt == QS_C64 ? sizeof(float) : sizeof(double));
            d.amp_off = b->amp_off[i];
            d.prev_part_off = b->last[i].off;
            d.prev_nparts = b->last[i].n;
            b->last[i] = {parts, (uint32_t)(ntiles / per)};
            for (uint64_t t0 = 0; t0 < ntiles; t0 += per)
                level.push_back({(double)per * std::ldexp((double)(ps.nblocks + 2), ps.t),
                                 PassItem{(uint32_t)pdv.size(), (uint32_t)t0, (uint32_t)per, (uint32_t)parts++}});
            lv.lds = std::max(lv.lds, (ab << ps.t) + kBatchRedBytes);
            lv.wide |= p.pass_wide[di][pi] != 0;
            pdv.push_back(d);
        }
        QS_CHECK(items.size() + level.size() <= UINT32_MAX, QS_ERANGE, "batch has more than 2^32 pass items");
        std::stable_sort(level.begin(), level.end(), [](const Cost &x, const Cost &y) { return x.c > y.c; });
        for (const Cost &c : level) items.push_back(c.it);
        lv.count = (uint32_t)(items.size() - lv.first);
        b->levels.push_back(lv);
    }
    for (int w = 0; w < 2; ++w) {
        size_t lds = 0;
        for (const auto &lv : b->levels)
            if (lv.wide == (w != 0)) lds = std::max(lds, lv.lds);
        if (!lds) continue;
        const void *fn = dt == QS_C64 ? reinterpret_cast<const void *>(batch_kernel<float>(w != 0))
                                      : reinterpret_cast<const void *>(batch_kernel<double>(w != 0));
        if (!dynamic_tile_at_zero(fn)) {
            set_error("batch kernel declares static LDS: its tile would not sit at LDS address 0");
            return fail(QS_EDEVICE);
        }
        e = set_dynamic_lds(fn, lds);   // never lowered: other batches' graphs use the kernel too
        if (e != hipSuccess) return fail(hip_fail(e, "hipFuncSetAttribute(batch)"));
    }
    // ---- energies: one job per state, items = runs of cosets of a term group ----
    std::vector<ExpectPlan> eplans(n_states);
    std::vector<ExpectGroup> groups;
    std::vector<ExpectTerm> terms;
    std::vector<double> hc;
    std::vector<size_t> g0(n_states), t0(n_states), c0(n_states);
    uint64_t cosets = 0;
    for (int i = 0; i < n_states; ++i) {
        st = expect_plan(b->n[i], dt, x[i], z[i], n_terms[i], eplans[i]);
        if (st != QS_OK) return fail(st);
        ExpectPlan &ep = eplans[i];
        g0[i] = groups.size();
        t0[i] = terms.size();
        c0[i] = hc.size();
        groups.insert(groups.end(), ep.groups.begin(), ep.groups.end());
        terms.insert(terms.end(), ep.terms.begin(), ep.terms.end());
        hc.insert(hc.end(), coeff[i], coeff[i] + n_terms[i]);
        if (!ep.small) cosets += ep.items;
    }
    if ((st = upload(&b->d_groups, groups)) != QS_OK) return fail(st);
    if ((st = upload(&b->d_terms, terms)) != QS_OK) return fail(st);
    if ((st = upload(&b->d_coeff, hc)) != QS_OK) return fail(st);
    // consecutive cosets per item: 1 until every CU (one full coset's
    // workgroup each) has eight items, then more, 16 at most
    uint32_t per_item = 1;
    while (per_item < 16 && cosets / (2 * per_item) >= 8 * cus) per_item *= 2;
    std::vector<ExpectJob> jobs(n_states);
    std::vector<ExpectItem> full, small;
    uint64_t eparts = 0;
    for (int i = 0; i < n_states; ++i) {
        const ExpectPlan &ep = eplans[i];
        ExpectJob &j = jobs[i];
        std::memset(&j, 0, sizeof j);
        j.psi0 = b->amp_off[i];
        j.group0 = g0[i];
        j.term0 = t0[i];
        j.coeff0 = c0[i];
        j.part0 = eparts;
        j.l = ep.l;
        j.D = ep.D;
        j.b = ep.b;
        j.log_cosets = ep.log_cosets;
        j.per_item = ep.small ? 1 : std::min<uint32_t>(per_item, 1u << ep.log_cosets);
        j.chunks = (1u << ep.log_cosets) / j.per_item;
        j.n_terms = (uint32_t)ep.terms.size();
        eparts += (uint64_t)j.n_terms * j.chunks;
        for (uint32_t g = 0; g < ep.groups.size(); ++g)
            for (uint32_t c = 0; c < j.chunks; ++c)
                (ep.small ? small : full).push_back(ExpectItem{(uint32_t)i, g, c, 0});
    }
    QS_CHECK(full.size() + small.size() <= UINT32_MAX, QS_ERANGE, "batch has more than 2^32 energy items");
    b->n_full = (uint32_t)full.size();
    b->n_small = (uint32_t)small.size();
    full.insert(full.end(), small.begin(), small.end());
    if ((st = upload(&b->d_jobs, jobs)) != QS_OK) return fail(st);
    if ((st = upload(&b->d_eitems, full)) != QS_OK) return fail(st);
    if ((st = upload(&b->d_items, items)) != QS_OK) return fail(st);
    if ((st = upload(&b->d_passes, pdv)) != QS_OK) return fail(st);
    e = hipMalloc(&b->d_partials, std::max<uint64_t>(1, parts) * sizeof(double));
    if (e == hipSuccess) e = hipMalloc(&b->d_eparts, std::max<uint64_t>(1, eparts) * sizeof(double));
    if (e == hipSuccess) e = hipHostMalloc((void **)&b->h_energy, n_states * sizeof(double), hipHostMallocDefault);
    if (e != hipSuccess) return fail(hip_fail(e, "hipMalloc(batch)"));
    // ---- capture the whole batch in one graph ----
    hipStream_t cap = nullptr;
    e = hipStreamCreateWithFlags(&cap, hipStreamNonBlocking);
    if (e != hipSuccess) return fail(hip_fail(e, "hipStreamCreate"));
    e = hipStreamBeginCapture(cap, hipStreamCaptureModeThreadLocal);
    if (e == hipSuccess) {
        st = enqueue_batch(*b, cap);
        hipError_t e2 = hipStreamEndCapture(cap, &b->graph);
        if (st == QS_OK && e2 != hipSuccess) st = hip_fail(e2, "hipStreamEndCapture");
    } else {
        st = hip_fail(e, "hipStreamBeginCapture");
    }
    hipStreamDestroy(cap);
    if (st != QS_OK) return fail(st);
    e = hipGraphInstantiate(&b->exec, b->graph, nullptr, nullptr, 0);
    if (e != hipSuccess) return fail(hip_fail(e, "hipGraphInstantiate"));
    *out = own.release();
    return QS_OK;
    QS_ABI_CATCH
}

qs_status qs_batch_destroy(qs_batch b) {
    if (!b) return QS_OK;
    hipStreamSynchronize(b->stream);
    delete b;
    return QS_OK;
}

qs_status qs_batch_run(qs_batch b, double *energies) {
    QS_CHECK(b != nullptr, QS_EINVAL, "null batch");
    QS_HIP(hipGraphLaunch(b->exec, b->stream));
    QS_HIP(hipStreamSynchronize(b->stream));
    if (energies) std::memcpy(energies, b->h_energy, b->nstates * sizeof(double));
    return QS_OK;
}

qs_status qs_batch_state_copy_out(qs_batch b, int i, double *host) {
    QS_CHECK(b && host, QS_EINVAL, "null argument");
    QS_CHECK(i >= 0 && i < b->nstates, QS_EINVAL, "state index out of range");
    QS_HIP(hipStreamSynchronize(b->stream));
    const int n = b->n[i];
    const uint64_t cnt = 1ull << n;
    // the stored amplitudes carry the last pass's pending scale: read the partials back
    double N = 0;
    {
        // norm of the stored state = fixed-order sum of the last pass's partials
        std::vector<double> parts(b->last[i].n);
        QS_HIP(hipMemcpy(parts.data(), b->d_partials + b->last[i].off, parts.size() * sizeof(double),
                         hipMemcpyDeviceToHost));
        for (double v : parts) N += v;
    }
    const double scale = N > 0 ? 1.0 / std::sqrt(N) : 1.0;
    const unsigned char *src = (const unsigned char *)b->d_amps + b->amp_off[i];
    if (b->dtype == QS_C64) {
        std::vector<float> f(2 * cnt);
        QS_HIP(hipMemcpy(f.data(), src, f.size() * sizeof(float), hipMemcpyDeviceToHost));
        for (uint64_t k = 0; k < 2 * cnt; ++k) host[k] = f[k] * scale;
    } else {
        QS_HIP(hipMemcpy(host, src, 2 * cnt * sizeof(double), hipMemcpyDeviceToHost));
        for (uint64_t k = 0; k < 2 * cnt; ++k) host[k] *= scale;
    }
    return QS_OK;
}

}  // extern "C"
