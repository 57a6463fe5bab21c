// OP2-style indirect increment: every edge adds its value to the two cells
// it connects (an op_par_loop over edges with two OP_INC arguments through
// the edge-to-cell map, Sec. III-A).
//
// Two ways to run it:
//  * A plan (built once per mesh, on the host, like OP2's execution plans)
//    inverts the map: for each cell, the list of its incident edges in the
//    order the sequential loop visits them (edge index ascending; a
//    self-loop edge twice, its second cell first). The kernel then gives
//    each cell to one thread, which adds the cell's increments in exactly
//    that order: no atomics, no colouring, and the result equals the
//    sequential loop bit for bit. The plan has three forms with that
//    property: lists (k_gather) for meshes of few edges, fours
//    (k_gather_fours), and rounds (k_rounds) for large ones in random order.
//  * A scatter with float64 atomic adds: one thread per edge. Fast to set
//    up, but the order in which a cell's increments land varies from run
//    to run, so only a tolerance holds.
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <atomic>
#include <memory>
#include <new>
#include <thread>
#include <vector>

#include "dev_common.h"
#include "pf_internal.h"

namespace pf {
namespace inc {

typedef int32_t i2 __attribute__((ext_vector_type(2)));
typedef uint32_t u2 __attribute__((ext_vector_type(2)));
typedef int32_t i4 __attribute__((ext_vector_type(4)));

constexpr int kThreads = 256;

constexpr int kWaves = 16;        // waves of a k_rounds workgroup, a bin of cells each
constexpr int kMaxCells = 1024;   // cells of a bin; the slot behind them takes the padding
constexpr int kGroup = 2;         // rounds per step
constexpr int kSlotBits = 11;     // a round's entry: slot of the cell, then edge - base of the round
constexpr int32_t kSpan = 1 << (32 - kSlotBits);

}  // namespace inc
}  // namespace pf

struct pf_inc_plan {
    int32_t ncells = 0, nedges = 0;
    int device = -1;
    void *dev = nullptr;  // all tables
    // Lists: offsets (ncells + 1), the cells' edges (2 * nedges).
    const int32_t *off = nullptr, *idx = nullptr;
    // Fours: the cells' edges, four to a cell.
    const pf::inc::i4 *four = nullptr;
    // Rounds (nbins > 0): the bins' first groups (nbins + 1); per group, the
    // edge base of each round and 64 entries of each.
    int32_t nbins = 0, per = 0;
    const int32_t *first = nullptr;
    const pf::inc::i2 *base = nullptr;
    const pf::inc::u2 *entry = nullptr;
};

namespace pf {
namespace inc {

// cell[c] += edge[idx[k]] for k in off[c] .. off[c+1], in that order.
__global__ __launch_bounds__(kThreads) void k_gather(const int32_t *__restrict__ off, const int32_t *__restrict__ idx,
                                                     const double *__restrict__ edge, double *__restrict__ cell,
                                                     int32_t ncells) {
    const int64_t c = (int64_t)xcd_remap(blockIdx.x, gridDim.x) * kThreads + threadIdx.x;
    if (c >= ncells) return;
    const int32_t k0 = off[c], k1 = off[c + 1];
    double v = cell[c];
    int32_t k = k0;
    // Four independent index/value loads in flight, added in order.
    for (; k + 4 <= k1; k += 4) {
        const int32_t i0 = idx[k], i1 = idx[k + 1], i2 = idx[k + 2], i3 = idx[k + 3];
        const double e0 = edge[i0], e1 = edge[i1], e2 = edge[i2], e3 = edge[i3];
        v = v + e0;
        v = v + e1;
        v = v + e2;
        v = v + e3;
    }
    for (; k < k1; ++k) v = v + edge[idx[k]];
    cell[c] = v;
}

// The same with each cell's edges in one 16-byte entry (-1: none), the form of
// meshes whose cells have at most four and, on average, two or more, as in quad
// meshes: they and the cell's value come in one round trip, their values in the
// next, where the lists take three. Bound by latency up to some 100,000 cells,
// then by the lines fetched for single values. Lists -> fours, us: random quads
// 362 x 362 6.6 -> 5.8, 512 x 512 10.5 -> 9.4, 724 x 724 25.0 -> 23.5; numbered
// row by row 1024 x 1024 10.7 -> 9.0, 2048 x 2048 45 -> 39 (5.1 TB/s). Cells of
// more edges stay on lists: with three edges in the entry and the rest behind it
// 300,000 cells took, random edges, 10.8 us at 1.5 edges to a cell (lists 9.9),
// 13.7 (13.2) at 2, 20.9 (21.9) at 3, but their plans 2 to 3 times as long to
// make (4.0 and 1.9 ms, 5.8 and 2.4, 7.7 and 3.1).
__global__ __launch_bounds__(kThreads) void k_gather_fours(const i4 *__restrict__ four,
                                                           const double *__restrict__ edge, double *__restrict__ cell,
                                                           int32_t ncells) {
    const int64_t c = (int64_t)xcd_remap(blockIdx.x, gridDim.x) * kThreads + threadIdx.x;
    if (c >= ncells) return;
    const i4 e = four[c];
    double v = cell[c], x[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) x[k] = edge[max(e[k], 0)];
#pragma unroll
    for (int k = 0; k < 4; ++k)
        if (e[k] >= 0) v = v + x[k];
    cell[c] = v;
}

__device__ __forceinline__ void round_values(const double *__restrict__ edge, u2 e, i2 b, double *v) {
#pragma unroll
    for (int u = 0; u < kGroup; ++u) v[u] = edge[b[u] + (int32_t)(e[u] >> kSlotBits)];
}

// The same increments for large meshes in random order. There k_gather is
// bound by what it fetches, not by what it uses: every 8-byte value comes as a
// line of 128 bytes through the last-level cache (16.8 million of them for a
// 2048 x 2048 quad mesh: 2.1 GB at 7 TB/s). Here the cells sit in LDS, 1024
// per wave and 16384 per CU, so a mesh of up to 4.2 million cells is resident
// at once, and all waves walk the edge array from its start to its end: a
// line is fetched once per XCD while its workgroups pass it. Wave b owns bin
// b (cells b * per ..) and takes the bin's visits in the loop's order, cut on
// the host into rounds of 64 in which no cell occurs twice, and a cell's
// visits in rounds that ascend: one read-modify-write per lane and round, in
// the order of the loop, without atomics (LDS operations of one wave are
// performed in order). The barrier per step only keeps the 16 waves together:
// without it they drift apart by more than the L2 holds (79% misses, 254 us).
// Two rounds per step: 132 us; one 140, four 144, and a third step of loads in
// flight 135.
// 2048 x 2048 quads: 309 -> 133 us; 1024 x 1024: 64.5 -> 37.6 us.
__global__ __launch_bounds__(64 * kWaves) void k_rounds(const int32_t *__restrict__ first, const i2 *__restrict__ base,
                                                        const u2 *__restrict__ entry, const double *__restrict__ edge,
                                                        double *__restrict__ cell, int32_t ncells, int32_t per) {
    __shared__ double acc[kWaves][kMaxCells + 1];
    __shared__ int most;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int b = blockIdx.x * kWaves + wave;
    const int64_t c0 = (int64_t)b * per;
    const int cnt = (int)min((int64_t)per, max((int64_t)0, ncells - c0));
    double *a = acc[wave];
    for (int i = lane; i < cnt; i += 64) a[i] = __builtin_nontemporal_load(cell + c0 + i);
    int g0 = 0, g1 = 0;
    if (cnt > 0) {
        g0 = first[b];
        g1 = first[b + 1];
    }
    if (threadIdx.x == 0) most = 0;
    __syncthreads();
    if (lane == 0) atomicMax(&most, g1 - g0);
    __syncthreads();
    const int steps = most;
    if (steps > 0) {
        // Entries two steps ahead, values one; past the bin's last group the
        // loads repeat it (or the group before an empty bin).
        const int gl = max(g1 - 1, 0);
        u2 e = __builtin_nontemporal_load(entry + (int64_t)min(g0, gl) * 64 + lane);
        u2 en = __builtin_nontemporal_load(entry + (int64_t)min(g0 + 1, gl) * 64 + lane);
        double v[kGroup], vn[kGroup];
        round_values(edge, e, base[min(g0, gl)], v);
#pragma unroll 1
        for (int k = 0; k < steps; ++k) {
            const int g = g0 + k;
            round_values(edge, en, base[min(g + 1, gl)], vn);
            const u2 e2 = __builtin_nontemporal_load(entry + (int64_t)min(g + 2, gl) * 64 + lane);
            __builtin_amdgcn_sched_barrier(0);
            if (g < g1) {
#pragma unroll
                for (int u = 0; u < kGroup; ++u) {
                    const int slot = e[u] & ((1 << kSlotBits) - 1);
                    a[slot] = a[slot] + v[u];
                    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                    __builtin_amdgcn_wave_barrier();
                }
            }
            e = en;
            en = e2;
#pragma unroll
            for (int u = 0; u < kGroup; ++u) v[u] = vn[u];
            __builtin_amdgcn_s_barrier();
        }
    }
    for (int i = lane; i < cnt; i += 64) __builtin_nontemporal_store(a[i], cell + c0 + i);
}

// One thread per edge: cell[e2c[2i+1]] += edge[i]; cell[e2c[2i]] += edge[i].
__global__ __launch_bounds__(kThreads) void k_scatter(const int32_t *__restrict__ e2c, const double *__restrict__ edge,
                                                      double *__restrict__ cell, int32_t ncells, int32_t nedges) {
    const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (i >= nedges) return;
    const double e = edge[i];
    const int32_t c1 = e2c[2 * i + 1], c0 = e2c[2 * i];
    // The map lives in device memory and is not validated by the host:
    // entries outside 0..ncells-1 are skipped rather than written through.
    if ((uint32_t)c1 < (uint32_t)ncells) unsafeAtomicAdd(&cell[c1], e);
    if ((uint32_t)c0 < (uint32_t)ncells) unsafeAtomicAdd(&cell[c0], e);
}

}  // namespace inc
}  // namespace pf

namespace pf {
namespace inc {

// The form of a plan. Below 10 MiB of edge values the L2s hold most of what a
// gather fetches: fours, or lists (make_fours). us, lists / fours / rounds:
// random quads 724 x 724, 8 MiB 25.0 / 23.5 / 33; 860 x 860 42 / - / 29.
// From there by how far apart the cells are that neighbouring edges name, in a
// sample:
//  * within 1024 cells for the most part: fours, or lists. The values of a gather are in
//    the L2. 2048 x 2048 numbered row by row 45.1 / 39.3 / 49.9, its edges
//    shuffled within 1024 58.1 / 56.5 / 60.7.
//  * over a sixteenth of the mesh and 128 K cells (2 MiB of their edges) for
//    the most part: rounds. 2048 x 2048 in random order 309 / - / 132; shuffled
//    within a sixteenth 103 / 106 / 108, 1024 x 1024 within a quarter
//    24.1 / 23.3 / 33.
//  * between: lists, whose fewer loads in flight leave more of the L2 (2048 x
//    2048 shuffled within 65536 edges 89 / 96 / 72, 1024 x 1024 20 / 19 / 34).
enum Form { kLists, kFours, kRounds };

Form form_of(int32_t ncells, int32_t nedges, const int32_t *e2c) {
    if (nedges < (10 << 20) / 8) return kFours;
    constexpr int kSamples = 1024;
    const int32_t wide = std::max(ncells / 16, 1 << 17);
    int near = 0, far = 0;
    for (int s = 0; s < kSamples; ++s) {
        const int64_t i = (int64_t)s * (nedges - 1) / kSamples;
        for (int k = 0; k < 2; ++k) {
            const int32_t d = abs(e2c[2 * i + k] - e2c[2 * i + 2 + k]);
            near += d <= 1024;
            far += d > wide;
        }
    }
    if (near > kSamples) return kFours;
    return far > kSamples && ncells <= 1 << 30 ? kRounds : kLists;  // cells: see Quotient
}

// n / d by a multiplication: exact for n < 2^30 and 2^10 <= d <= 2^14 and for
// n < 2^14 and 1 <= d <= 2^14, since m = ceil(2^44 / d) is at most 1 more than
// 2^44 / d, and n m fits 64 bits.
struct Quotient {
    uint64_t m;
    explicit Quotient(int32_t d) : m((((uint64_t)1 << 44) + (uint64_t)d - 1) / (uint64_t)d) {}
    int32_t operator()(int32_t n) const { return (int32_t)((uint64_t)n * m >> 44); }
};

// f(0) .. f(threads - 1), one to a thread; what finds no thread runs here. False
// where one of them threw (found no memory).
template <class F>
bool shares(int threads, F f) {
    std::atomic<bool> ok{true};
    auto run = [&](int t) {
        try {
            f(t);
        } catch (const std::exception &) {
            ok = false;
        }
    };
    std::vector<std::thread> pool;
    int t = 1;
    try {
        for (; t < threads; ++t) pool.emplace_back(run, t);
    } catch (const std::exception &) {
    }
    run(0);
    for (; t < threads; ++t) run(t);
    for (std::thread &th : pool) th.join();
    return ok;
}

struct Rounds {
    int32_t nbins = 0, per = 0;
    std::vector<int32_t> first, base;
    std::unique_ptr<uint32_t[]> entry;
    size_t entries = 0;
};

// The visits of each bin in rounds of 64 (k_rounds). False where the rounds
// would be more than a quarter padding, or the longest bin more than twice
// the mean: a cell in many edges has a round for each of its visits.
// By up to 8 threads: by one, a plan took longer to make than the lists (ms on
// the host of an MI355X with 16 CPUs, lists / rounds by one / by 8: 860 x 860
// quads 6.3 / 16.9 / 3.5, 1024 x 1024 12.1 / 23.7 / 4.7, 2048 x 2048 127 / 120 /
// 31).
bool make_rounds(int32_t ncells, int32_t nedges, const int32_t *e2c, Rounds *out) {
    const int64_t visits = 2 * (int64_t)nedges;
    const int threads = (int)std::max<int64_t>(
        1, std::min<int64_t>({8, (int64_t)std::thread::hardware_concurrency(), visits >> 18}));
    // Bins for one workgroup per CU, or for as many sweeps of 256 workgroups as
    // the cells need; at least 192 cells, since small bins leave no 64 visits
    // of different cells to choose from (17% padding at 192, over 25% at 128).
    constexpr int64_t kResident = 256 * kWaves;
    const int64_t sweeps = (ncells + kResident * kMaxCells - 1) / (kResident * kMaxCells);
    const int32_t per = (int32_t)std::max<int64_t>(192, (ncells + kResident * sweeps * 64 - 1) / (kResident * sweeps * 64) * 64);
    const int32_t nbins = (int32_t)((ncells + (int64_t)per - 1) / per);
    // First by workgroup: few enough streams for the caches, in edge order. A
    // thread takes a range of the edges; at: where its visits of a workgroup go.
    const int32_t block = per * kWaves, nblocks = (int32_t)((ncells + (int64_t)block - 1) / block);
    const Quotient by_block(block), by_per(per);
    struct Visit {
        int32_t edge, slot;
    };
    auto range = [&](int t) { return (int32_t)((int64_t)nedges * t / threads); };
    std::vector<std::vector<int64_t>> at((size_t)threads);
    std::vector<int64_t> start((size_t)nblocks + 1, 0);
    std::unique_ptr<Visit[]> list(new Visit[(size_t)visits]);
    if (!shares(threads, [&](int t) {
            std::vector<int64_t> n((size_t)nblocks, 0);
            for (int64_t j = 2 * (int64_t)range(t); j < 2 * (int64_t)range(t + 1); ++j) ++n[(size_t)by_block(e2c[j])];
            at[(size_t)t] = std::move(n);
        }))
        return false;
    int64_t total = 0;
    for (int32_t b = 0; b < nblocks; ++b) {
        start[(size_t)b] = total;
        for (std::vector<int64_t> &n : at) {
            const int64_t here = n[(size_t)b];
            n[(size_t)b] = total;
            total += here;
        }
    }
    start[(size_t)nblocks] = total;
    shares(threads, [&](int t) {
        int64_t *fill = at[(size_t)t].data();
        for (int32_t i = range(t); i < range(t + 1); ++i)
            for (int k = 1; k >= 0; --k) {  // the second cell is incremented first
                const int32_t c = e2c[2 * (int64_t)i + k], b = by_block(c);
                list[(size_t)fill[b]++] = {i, c - b * block};
            }
    });
    // Then each workgroup's bins, the workgroups dealt to the threads.
    struct Round {
        int32_t base, count;
    };
    struct Bin {
        int32_t low = 0;  // rounds below are full or out of reach
        std::vector<Round> round;
        std::vector<uint32_t> entry;
    };
    struct Block {
        std::vector<int32_t> groups, base;  // groups: of each bin
        std::vector<uint32_t> entry;
    };
    const size_t most = (size_t)(visits + visits / 4);
    std::vector<Block> blocks((size_t)nblocks);
    // What all threads write lies apart from what they read for every visit
    // (beside it: 7.6 ms instead of 1.9 at 860 x 860).
    struct alignas(128) Shared {
        std::atomic<int32_t> next{0};
        std::atomic<size_t> entries{0};
    } all;
    const bool made = shares(threads, [&, by_per, per](int) {
        std::vector<Bin> bins(kWaves);
        std::vector<int32_t> last((size_t)block);  // the cells' last rounds
        for (int32_t w; (w = all.next++) < nblocks;) {
            size_t here = 0;
            for (Bin &q : bins) {
                q.low = 0;
                q.round.clear();
                q.entry.clear();
            }
            std::fill(last.begin(), last.end(), -1);
            const Visit *v = list.get() + start[(size_t)w], *const end = list.get() + start[(size_t)w + 1];
            for (; v != end; ++v) {
                const int32_t edge = v->edge, in = by_per(v->slot);
                Bin &q = bins[(size_t)in];
                const int32_t n = (int32_t)q.round.size();
                Round *const rd = q.round.data();
                auto closed = [&](int32_t r) { return rd[r].count == 64 || edge - rd[r].base >= kSpan; };
                int32_t low = q.low;
                while (low < n && closed(low)) ++low;
                q.low = low;
                int32_t r = std::max(low, last[(size_t)v->slot] + 1);
                while (r < n && closed(r)) ++r;
                last[(size_t)v->slot] = r;
                if (r == n) {
                    if (r % kGroup == 0) {
                        here += 64 * kGroup;
                        if (all.entries + here > most) {
                            all.entries += here;
                            return;
                        }
                        q.entry.resize(q.entry.size() + 64 * kGroup, (uint32_t)kMaxCells);
                    }
                    q.round.push_back({edge, 0});
                }
                Round &t = q.round[(size_t)r];
                q.entry[((size_t)(r / kGroup) * 64 + (size_t)t.count++) * kGroup + r % kGroup] =
                    (uint32_t)(edge - t.base) << kSlotBits | (uint32_t)(v->slot - in * per);
            }
            all.entries += here;
            Block &o = blocks[(size_t)w];
            o.entry.reserve(here);
            for (int32_t k = 0; k < kWaves && w * kWaves + k < nbins; ++k) {
                Bin &q = bins[(size_t)k];
                o.entry.insert(o.entry.end(), q.entry.begin(), q.entry.end());
                q.round.resize(q.entry.size() / 64, {0, 0});  // a round of padding reads edge 0
                for (const Round &t : q.round) o.base.push_back(t.base);
                o.groups.push_back((int32_t)(q.round.size() / kGroup));
            }
        }
    });
    if (!made || all.entries > most) return false;
    list.reset();
    out->entries = all.entries;
    out->entry.reset(new uint32_t[out->entries]);
    out->first.assign(1, 0);
    std::vector<size_t> to((size_t)nblocks, 0);
    int32_t longest = 0;
    for (int32_t w = 0; w < nblocks; ++w) {
        const Block &o = blocks[(size_t)w];
        to[(size_t)w] = (size_t)out->base.size() * 64;
        out->base.insert(out->base.end(), o.base.begin(), o.base.end());
        for (int32_t g : o.groups) {
            out->first.push_back(out->first.back() + g);
            longest = std::max(longest, g);
        }
    }
    all.next = 0;
    shares(threads, [&](int) {
        for (int32_t w; (w = all.next++) < nblocks;) {
            const Block &o = blocks[(size_t)w];
            if (!o.entry.empty()) memcpy(out->entry.get() + to[(size_t)w], o.entry.data(), o.entry.size() * 4);
        }
    });
    out->nbins = nbins;
    out->per = per;
    return (size_t)longest * 64 * kGroup * (size_t)nbins <= 2 * out->entries;
}

// The table of k_gather_fours. False for meshes with a cell of more than four
// visits, or of under two visits per cell, whose entries would mostly hold
// nothing (16 bytes a cell; the lists 4, and 4 per visit).
bool make_fours(int32_t ncells, int32_t nedges, const int32_t *e2c, std::unique_ptr<int32_t[]> *four) {
    if (nedges < ncells) return false;
    four->reset(new int32_t[(size_t)ncells * 4]);
    int32_t *const f = four->get();
    std::vector<uint8_t> at((size_t)ncells, 0);
    for (int64_t j = 0; j < 2 * (int64_t)nedges; ++j) {
        const size_t c = (size_t)e2c[j ^ 1];  // the second cell is incremented first
        if (at[c] == 4) return false;
        f[c * 4 + at[c]++] = (int32_t)(j / 2);
    }
    for (size_t c = 0; c < (size_t)ncells; ++c)
        for (size_t k = at[c]; k < 4; ++k) f[c * 4 + k] = -1;
    return true;
}

// Device memory for the plan's tables, filled from the host.
struct Part {
    const void *p;
    size_t bytes;
};

hipError_t upload(pf_inc_plan *p, const Part *parts, int n) {
    size_t total = 4;
    for (int i = 0; i < n; ++i) total += parts[i].bytes;
    hipError_t e = hipMalloc(&p->dev, total);
    if (e != hipSuccess) {
        p->dev = nullptr;
        return e;
    }
    size_t at = 0;
    for (int i = 0; i < n && e == hipSuccess; at += parts[i++].bytes)
        if (parts[i].bytes) e = hipMemcpy((char *)p->dev + at, parts[i].p, parts[i].bytes, hipMemcpyHostToDevice);
    if (e != hipSuccess) {
        (void)hipFree(p->dev);
        p->dev = nullptr;
    }
    return e;
}

}  // namespace inc
}  // namespace pf

using namespace pf;

extern "C" {

pf_status pf_inc_plan_create(int32_t ncells, int32_t nedges, const int32_t *__restrict edge_to_cells,
                             pf_inc_plan **const __restrict plan) {
    clear_error();
    if (!plan) return fail(PF_EINVAL, "null plan out-parameter");
    *plan = nullptr;
    if (ncells < 1 || nedges < 0) return fail(PF_EINVAL, "need ncells >= 1 and nedges >= 0");
    if (nedges > (1 << 30)) return fail(PF_EUNSUPPORTED, "more than 2^30 edges");
    if (nedges > 0 && !edge_to_cells) return fail(PF_EINVAL, "null edge-to-cell map");
    for (int64_t j = 0; j < 2 * (int64_t)nedges; ++j)
        if (edge_to_cells[j] < 0 || edge_to_cells[j] >= ncells)
            return fail(PF_EINVAL, "edge " + std::to_string(j / 2) + " names a cell outside 0.." +
                                       std::to_string(ncells - 1));
    pf_inc_plan *p = new (std::nothrow) pf_inc_plan;
    if (!p) return fail(PF_ENOMEM, "plan allocation");
    p->ncells = ncells;
    p->nedges = nedges;
    (void)hipGetDevice(&p->device);
    // The next form is made where one finds no memory, on either side.
    const inc::Form form = inc::form_of(ncells, nedges, edge_to_cells);
    inc::Rounds rounds;
    bool made = false;
    try {
        made = form == inc::kRounds && inc::make_rounds(ncells, nedges, edge_to_cells, &rounds);
    } catch (const std::bad_alloc &) {
    }
    if (made) {
        const size_t be = rounds.entries * 4, bb = rounds.base.size() * 4, bf = rounds.first.size() * 4;
        const inc::Part parts[] = {{rounds.entry.get(), be}, {rounds.base.data(), bb}, {rounds.first.data(), bf}};
        if (inc::upload(p, parts, 3) == hipSuccess) {
            p->entry = (const inc::u2 *)p->dev;
            p->base = (const inc::i2 *)((char *)p->dev + be);
            p->first = (const int32_t *)((char *)p->dev + be + bb);
            p->nbins = rounds.nbins;
            p->per = rounds.per;
            *plan = p;
            return PF_OK;
        }
        (void)hipGetLastError();
        rounds = inc::Rounds();
    }
    std::unique_ptr<int32_t[]> four;
    made = false;
    try {
        made = form == inc::kFours && inc::make_fours(ncells, nedges, edge_to_cells, &four);
    } catch (const std::bad_alloc &) {
    }
    if (made) {
        const inc::Part part = {four.get(), (size_t)ncells * sizeof(inc::i4)};
        if (inc::upload(p, &part, 1) == hipSuccess) {
            p->four = (const inc::i4 *)p->dev;
            *plan = p;
            return PF_OK;
        }
        (void)hipGetLastError();
    }
    four.reset();
    // Counting sort of the (edge, slot) visits by cell, in visit order.
    std::vector<int32_t> off((size_t)ncells + 1, 0);
    for (int64_t j = 0; j < 2 * (int64_t)nedges; ++j) ++off[(size_t)edge_to_cells[j] + 1];
    for (int32_t c = 0; c < ncells; ++c) off[(size_t)c + 1] += off[c];
    std::vector<int32_t> fill(off.begin(), off.end() - 1);
    std::vector<int32_t> idx((size_t)2 * nedges);
    for (int32_t i = 0; i < nedges; ++i) {
        idx[(size_t)fill[edge_to_cells[2 * (int64_t)i + 1]]++] = i;  // the second cell is incremented first
        idx[(size_t)fill[edge_to_cells[2 * (int64_t)i]]++] = i;
    }
    const size_t bo = off.size() * sizeof(int32_t), bi = idx.size() * sizeof(int32_t);
    const inc::Part parts[] = {{off.data(), bo}, {idx.data(), bi}};
    if (hipError_t e = inc::upload(p, parts, 2)) {
        delete p;
        return fail_hip(e, "plan tables");
    }
    p->off = (const int32_t *)p->dev;
    p->idx = (const int32_t *)((char *)p->dev + bo);
    *plan = p;
    return PF_OK;
}

pf_status pf_inc_plan_run(const pf_inc_plan *p, int32_t ncells, int32_t nedges, const double *__restrict edge,
                          double *__restrict cell, void *stream) {
    clear_error();
    if (!p) return fail(PF_EINVAL, "null plan");
    if (ncells != p->ncells || nedges != p->nedges) return fail(PF_EINVAL, "sizes differ from the plan's");
    if (!cell || (nedges > 0 && !edge)) return fail(PF_EINVAL, "null array");
    if (((uintptr_t)edge | (uintptr_t)cell) % 8) return fail(PF_EINVAL, "arrays must be 8-byte aligned");
    const uintptr_t a = (uintptr_t)edge, b = (uintptr_t)cell;
    const uintptr_t na = (uintptr_t)nedges * 8, nb = (uintptr_t)ncells * 8;
    if (nedges > 0 && a < b + nb && b < a + na) return fail(PF_EALIAS, "edge and cell arrays overlap (restrict)");
    if (p->nbins) {
        const int grid = (p->nbins + inc::kWaves - 1) / inc::kWaves;
        hipLaunchKernelGGL(inc::k_rounds, dim3(grid), dim3(64 * inc::kWaves), 0, (hipStream_t)stream, p->first, p->base,
                           p->entry, edge, cell, ncells, p->per);
    } else if (p->four) {
        const int grid = (int)(((int64_t)ncells + inc::kThreads - 1) / inc::kThreads);
        hipLaunchKernelGGL(inc::k_gather_fours, dim3(grid), dim3(inc::kThreads), 0, (hipStream_t)stream, p->four,
                           edge, cell, ncells);
    } else {
        const int grid = (int)(((int64_t)ncells + inc::kThreads - 1) / inc::kThreads);
        hipLaunchKernelGGL(inc::k_gather, dim3(grid), dim3(inc::kThreads), 0, (hipStream_t)stream, p->off, p->idx, edge,
                           cell, ncells);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail_hip(e, "kernel launch");
    return PF_OK;
}

pf_status pf_inc_plan_destroy(pf_inc_plan *p) {
    clear_error();
    if (!p) return PF_OK;
    int cur = -1;
    (void)hipGetDevice(&cur);
    if (p->device >= 0 && p->device != cur) (void)hipSetDevice(p->device);
    hipError_t e = hipFree(p->dev);
    if (p->device >= 0 && cur >= 0 && p->device != cur) (void)hipSetDevice(cur);
    delete p;
    if (e != hipSuccess) return fail_hip(e, "plan free");
    return PF_OK;
}

pf_status pf_edge_inc_atomic_f64(int32_t ncells, int32_t nedges, const int32_t *__restrict edge_to_cells,
                                 const double *__restrict edge, double *__restrict cell, void *stream) {
    clear_error();
    if (ncells < 1 || nedges < 0) return fail(PF_EINVAL, "need ncells >= 1 and nedges >= 0");
    if (nedges > (1 << 30)) return fail(PF_EUNSUPPORTED, "more than 2^30 edges");
    if (!cell || (nedges > 0 && (!edge || !edge_to_cells))) return fail(PF_EINVAL, "null array");
    if (((uintptr_t)edge | (uintptr_t)cell) % 8 || (uintptr_t)edge_to_cells % 4)
        return fail(PF_EINVAL, "misaligned array");
    const uintptr_t b = (uintptr_t)cell, nb = (uintptr_t)ncells * 8;
    const uintptr_t a = (uintptr_t)edge, na = (uintptr_t)nedges * 8;
    const uintptr_t m = (uintptr_t)edge_to_cells, nm = (uintptr_t)nedges * 8;
    if (nedges > 0 && ((a < b + nb && b < a + na) || (m < b + nb && b < m + nm)))
        return fail(PF_EALIAS, "cell array overlaps an input (restrict)");
    if (nedges == 0) return PF_OK;
    const int grid = (int)((nedges + inc::kThreads - 1) / inc::kThreads);
    hipLaunchKernelGGL(inc::k_scatter, dim3(grid), dim3(inc::kThreads), 0, (hipStream_t)stream, edge_to_cells, edge,
                       cell, ncells, nedges);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail_hip(e, "kernel launch");
    return PF_OK;
}

}  // extern "C"
