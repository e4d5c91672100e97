// Launch planning of the two-site H.psi (Eq. dgemm, Section 2.2.1): the owner-computes task list of
// a handle cut into balanced work items for each kernel path -- FP64 one-wavefront tiles, the FP64
// register-streamed kernel, the split row-mode and task-mode kernels, the two-pass large-block
// path in both precisions -- with ordered reductions of the partial tiles of cut items (no atomics),
// part tags for the part masks of merged handles, and the tiled operator copies these kernels read.
#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <map>
#include <string>
#include <unordered_map>
#include <vector>

#include "../../include/dmrg.h"
#include "host_common.h"
#include "internal.h"
#include "hop.h"
#include "plan.h"

namespace dmrg {

namespace {


// Merged problem (dmrg_hop_combine) that holds coefficient `off`.
int32_t part_of(const dmrg_hop& H, int64_t off) {
    return (int32_t)(std::upper_bound(H.part_coeff.begin(), H.part_coeff.end(), off) - H.part_coeff.begin()) - 1;
}
// Tag work records (items, reductions) with the merged problem of their target, for part masks.
template <class R>
void tag_parts(const dmrg_hop& H, std::vector<R>& recs) {
    for (auto& r : recs) r.part = H.n_parts > 1 ? part_of(H, r.y_off) : 0;
}

// Cost caps of work items. A plan cuts the task list of a tile into items of at most `cap` cost
// units, with cap = total / (target item count). A merged handle sets the cap of each problem from
// that problem's own total (tune_part_items), as its own handle would: when a part mask leaves only
// a few problems running, their items are as fine as in their own plans and still fill the GPU.
struct CostCaps {
    const dmrg_hop& H;
    std::vector<double> total;
    explicit CostCaps(const dmrg_hop& h) : H(h), total(h.n_parts > 1 && h.tune_part_items ? h.n_parts : 1, 0.0) {}
    size_t slot(int j) const { return total.size() > 1 ? (size_t)part_of(H, H.blk_off[j]) : 0; }
    void add(int j, double c) { total[slot(j)] += c; }
    double cap(int j, int items, double floor) const {
        return std::max(total[slot(j)] / std::max(1, items), floor);
    }
};

template <class T>
T* plan_alloc(dmrg_hop& H, size_t n) {
    void* p = nullptr;
    if (n == 0) n = 1;
    HIPCHK(hipMalloc(&p, n * sizeof(T)));
    H.plan_allocations.push_back(p);
    H.plan_bytes += (int64_t)(n * sizeof(T));
    return static_cast<T*>(p);
}

// Bytes of a matrix definition as stored in the pool (all its sector blocks, padded).
double mat_bytes(const dmrg_hop& H, int m) { return m < 0 ? 0.0 : H.mats[m].bytes; }

// Operand-pool offset of a task's factor: matrix m at ket sector `sec`, or the identity of `dim` states.
int64_t op64_of(const dmrg_hop& H, int m, int sec, int dim) {
    const int64_t off = m >= 0 ? H.mats[m].op64_of_in[sec] : H.ident64_off[dmrg::k4_of(dim)];
    if (off < 0) throw Error(DMRG_ERR_ARG, "internal: operator block missing from the operand pool");
    return off;
}

// Launch plan of H.psi: packed input layout, phases, work items, reductions (see internal.h).
//  * Phases: the distinct (left matrix, right matrix) pairs are sorted by (right, left) and cut into
//    groups of about kCacheBudget bytes of operators, so that the operators of one phase stay in
//    the last-level cache while all target tiles are updated.
//  * Items: in each phase every output tile (16 or 32 rows x up to 16 * tune_max_tq columns) gets
//    the phase's tasks of its target block, cut into chunks of bounded MFMA cost (about
//    tune_items items per matvec); a tile split over several chunks writes partial tiles that the
//    phase's reduction adds in order.
void build_plan_core(dmrg_hop& H, hipStream_t s, const std::vector<char>* only, bool split_bufs, dmrg::HpsiPlan& plan,
                     std::vector<dmrg::HpsiLaunch>& launches_out, std::vector<dmrg::HpsiPhase>& phases_out,
                     const std::vector<char>* task_only = nullptr) {
    // tasks of this plan: those of the targets in `only` (all without it) that `task_only` keeps
    auto keep = [&](size_t t) {
        return (!only || (*only)[H.tasks[t].j]) && (!task_only || (*task_only)[t]);
    };
    constexpr double kCacheBudget = 96.0 * 1024 * 1024;
    // packed input layout: every psi block padded to multiples of 32 in both directions
    std::vector<dmrg::PackBlock> packs;
    std::vector<int64_t> pk_off(H.blk.size());
    int64_t psize = 0;
    for (size_t i = 0; i < H.blk.size(); ++i) {
        int pa = dmrg::ld_of(H.blk_ma[i]), pd = dmrg::ld_of(H.blk_md[i]);
        pk_off[i] = psize;
        packs.push_back({H.blk_off[i], psize, H.blk_ma[i], H.blk_md[i], pa, pd});
        psize += (int64_t)pa * pd;
    }
    // phases over (left, right) matrix pairs
    std::map<std::pair<int, int>, int> pair_phase;
    {
        std::vector<std::pair<int, int>> pairs;
        for (size_t t = 0; t < H.tasks.size(); ++t)
            if (keep(t)) pairs.push_back({H.tasks[t].rm, H.tasks[t].lm});
        std::sort(pairs.begin(), pairs.end());
        pairs.erase(std::unique(pairs.begin(), pairs.end()), pairs.end());
        std::vector<double> pb(pairs.size());
        double total = 0.0;
        for (size_t k = 0; k < pairs.size(); ++k) { pb[k] = mat_bytes(H, pairs[k].first) + mat_bytes(H, pairs[k].second); total += pb[k]; }
        int np = H.tune_phases > 0 ? H.tune_phases : std::max(1, (int)std::ceil(total / kCacheBudget));
        np = std::min<int>(np, std::max<size_t>(1, pairs.size()));
        double cum = 0.0;
        for (size_t k = 0; k < pairs.size(); ++k) {
            int ph = std::min(np - 1, (int)(np * (cum + 0.5 * pb[k]) / std::max(total, 1.0)));
            pair_phase[{pairs[k].second, pairs[k].first}] = ph;
            cum += pb[k];
        }
        plan.n_phases = np;
    }
    const int np = plan.n_phases;
    // device tasks, grouped per target block and phase (stable: source order kept inside)
    std::vector<dmrg::Task> dtasks;
    dtasks.reserve(H.tasks.size());
    // trange[j * np + ph] = task range of target j in phase ph
    std::vector<std::pair<int32_t, int32_t>> trange(H.blk.size() * np, {0, 0});
    auto r16 = [](int m) { return (m + 15) / 16 * 16; };
    {
        size_t t = 0;
        std::vector<std::vector<size_t>> by_phase(np);
        for (size_t j = 0; j < H.blk.size(); ++j) {
            for (auto& v : by_phase) v.clear();
            while (t < H.tasks.size() && H.tasks[t].j == (int)j) {
                if (keep(t)) by_phase[pair_phase[{H.tasks[t].lm, H.tasks[t].rm}]].push_back(t);
                ++t;
            }
            for (int ph = 0; ph < np; ++ph) {
                int32_t tb = (int32_t)dtasks.size();
                for (size_t k : by_phase[ph]) {
                    const auto& ht = H.tasks[k];
                    int64_t ao = ht.lm >= 0 ? H.mats[ht.lm].pool_of_in[H.blk[ht.i][0]] : -1;
                    int64_t bo = ht.rm >= 0 ? H.mats[ht.rm].pool_of_in[H.blk[ht.i][3]] : -1;
                    const int ma = H.blk_ma[ht.i], md = H.blk_md[ht.i];
                    dtasks.push_back({pk_off[ht.i], ao, bo, ht.f, dmrg::ld_of(ma), dmrg::ld_of(md), r16(ma), r16(md)});
                }
                trange[j * np + ph] = {tb, (int32_t)dtasks.size()};
            }
        }
    }
    if (only && dtasks.empty()) {                // the other paths run everything: no packed copy of x either
        plan = dmrg::HpsiPlan{};
        launches_out.clear();
        phases_out.clear();
        return;
    }
    auto task_cost = [&](const dmrg::Task& T, int tp, int tq) -> double {
        double c = 8.0;                                   // per-task overhead
        if (T.a_off < 0 && T.b_off < 0) return c + 1.0;
        if (T.b_off < 0) return c + (double)(T.ka / 4) * tp * tq;
        if (T.a_off < 0) return c + (double)(T.kd / 4) * tp * tq;
        return c + (double)(T.kd / 16) * (tp * (T.ka / 4) + 4.0 * tp * tq);
    };
    struct Tile { int j, r0, c0, tp, tq; };
    std::vector<Tile> tiles;
    double max_task = 0.0;
    CostCaps caps(H);
    const int tile_cols = 16 * H.tune_max_tq;
    for (size_t j = 0; j < H.blk.size(); ++j) {
        if (only && !(*only)[j]) continue;
        if (trange[j * np].first == trange[j * np + np - 1].second) continue;   // no task kept
        int mj = H.blk_ma[j], nj = H.blk_md[j];
        for (int r0 = 0; r0 < mj; r0 += dmrg::kTileRows)
            for (int c0 = 0; c0 < nj; c0 += tile_cols) {
                int tp = mj - r0 <= 16 ? 1 : 2;
                int tq = (std::min(tile_cols, nj - c0) + 15) / 16;
                for (int32_t t = trange[j * np].first; t < trange[j * np + np - 1].second; ++t) {
                    double tc = task_cost(dtasks[t], tp, tq);
                    caps.add((int)j, tc);
                    max_task = std::max(max_task, tc);
                }
                tiles.push_back({(int)j, r0, c0, tp, tq});
            }
    }
    std::vector<dmrg::Item> all_items;
    std::vector<dmrg::Reduce> all_red;
    launches_out.clear();
    phases_out.clear();
    int64_t part_max = 0;
    for (int ph = 0; ph < np; ++ph) {
        std::vector<dmrg::Item> items;
        std::vector<double> icost;
        std::vector<int> iclass, igroup;
        std::vector<dmrg::Reduce> reduces;
        int64_t part_size = 0;
        for (const Tile& T : tiles) {
            const int j = T.j;
            const auto tr = trange[j * np + ph];
            if (tr.first == tr.second) continue;
            std::vector<std::pair<int32_t, int32_t>> chunks;
            std::vector<double> ccost;
            int32_t b = tr.first;
            double c = 0.0;
            const double cmax = std::max(caps.cap(j, H.tune_items, 256.0), max_task);
            for (int32_t t = tr.first; t < tr.second; ++t) {
                double tc = task_cost(dtasks[t], T.tp, T.tq);
                if (c + tc > cmax && t > b) { chunks.push_back({b, t}); ccost.push_back(c); b = t; c = 0.0; }
                c += tc;
            }
            chunks.push_back({b, tr.second});
            ccost.push_back(c);
            const int cls = (T.tp - 1) * 8 + (T.tq - 1);
            const int tm = 16 * T.tp, tn = 16 * T.tq;
            const int grp = H.blk[j][0];                     // target left sector: shares left operators
            if (chunks.size() == 1) {
                items.push_back({H.blk_off[j], -1, H.blk_ma[j], H.blk_md[j], T.r0, T.c0, chunks[0].first, chunks[0].second});
                icost.push_back(ccost[0]);
                iclass.push_back(cls);
                igroup.push_back(grp);
            } else {
                reduces.push_back({H.blk_off[j], part_size, H.blk_ma[j], H.blk_md[j], T.r0, T.c0, tm, tn,
                                   (int32_t)chunks.size(), 0});
                for (size_t k = 0; k < chunks.size(); ++k) {
                    items.push_back({H.blk_off[j], part_size, H.blk_ma[j], H.blk_md[j], T.r0, T.c0, chunks[k].first,
                                     chunks[k].second});
                    part_size += (int64_t)tm * tn;
                    icost.push_back(ccost[k]);
                    iclass.push_back(cls);
                    igroup.push_back(grp);
                }
            }
        }
        part_max = std::max(part_max, part_size);
        // Launch order inside a tile class. 0: heaviest first. 1: target order. 2: XCD-aware -- items
        // whose targets share the left sector (hence the left operators) are placed at positions of
        // the same residue mod 8, i.e. on the same XCD and its L2, groups balanced over the 8 XCDs.
        std::vector<int> perm(items.size());
        for (size_t i = 0; i < perm.size(); ++i) perm[i] = (int)i;
        std::stable_sort(perm.begin(), perm.end(), [&](int a, int b) {
            if (iclass[a] != iclass[b]) return iclass[a] < iclass[b];
            if (H.tune_order == 0) return icost[a] > icost[b];
            if (H.tune_order == 2 && igroup[a] != igroup[b]) return igroup[a] < igroup[b];
            return false;
        });
        if (H.tune_order == 2) {
            const int nx = 8;
            std::vector<int> out;
            out.reserve(perm.size());
            size_t c0 = 0;
            while (c0 < perm.size()) {
                size_t c1 = c0;
                while (c1 < perm.size() && iclass[perm[c1]] == iclass[perm[c0]]) ++c1;
                std::map<int, std::vector<int>> grp;
                std::map<int, double> gcost;
                for (size_t i = c0; i < c1; ++i) { grp[igroup[perm[i]]].push_back(perm[i]); gcost[igroup[perm[i]]] += icost[perm[i]]; }
                std::vector<std::pair<double, int>> order;
                for (auto& kv : gcost) order.push_back({-kv.second, kv.first});
                std::sort(order.begin(), order.end());
                std::vector<double> load(nx, 0.0);
                std::vector<std::vector<int>> lane(nx);
                for (auto& og : order) {
                    int x = (int)(std::min_element(load.begin(), load.end()) - load.begin());
                    load[x] -= og.first;
                    for (int it : grp[og.second]) lane[x].push_back(it);
                }
                std::vector<size_t> pos(nx, 0);
                size_t left = c1 - c0;
                for (size_t p = 0; left > 0; ++p) {
                    int x = (int)(p % nx);
                    if (pos[x] < lane[x].size()) { out.push_back(lane[x][pos[x]++]); --left; }
                    else {
                        int best = -1;
                        size_t rem = 0;
                        for (int y = 0; y < nx; ++y) if (lane[y].size() - pos[y] > rem) { rem = lane[y].size() - pos[y]; best = y; }
                        out.push_back(lane[best][pos[best]++]);
                        --left;
                    }
                }
                c0 = c1;
            }
            perm = out;
        }
        dmrg::HpsiPhase P;
        P.launch_begin = (int)launches_out.size();
        const int base = (int)all_items.size();
        for (size_t i = 0; i < perm.size(); ++i) {
            all_items.push_back(items[perm[i]]);
            const int cls = iclass[perm[i]];
            if (launches_out.size() == (size_t)P.launch_begin || launches_out.back().cls != cls)
                launches_out.push_back({cls, base + (int)i, 0});
            launches_out.back().item_count++;
        }
        P.launch_end = (int)launches_out.size();
        P.reduce_begin = (int)all_red.size();
        for (const auto& r : reduces) all_red.push_back(r);
        P.reduce_end = (int)all_red.size();
        phases_out.push_back(P);
    }
    if (!only) H.n_items = (int)all_items.size();
    H.n_dev_tasks = (int64_t)dtasks.size();
    if (const char* e = std::getenv("DMRG_PLAN_TRACE"))
        if (e[0] == '1')
            std::fprintf(stderr, "[dmrg plan] phases %d items %zu launches %zu reduces %zu partial %.1f MB packed %.1f MB\n",
                         np, all_items.size(), H.launches.size(), all_red.size(), part_max * 8e-6, psize * 8e-6);
    tag_parts(H, all_items);
    tag_parts(H, all_red);
    dmrg::Item* d_items = plan_alloc<dmrg::Item>(H, all_items.size());
    dmrg::Task* d_tasks = plan_alloc<dmrg::Task>(H, dtasks.size());
    dmrg::Reduce* d_red = plan_alloc<dmrg::Reduce>(H, all_red.size());
    dmrg::PackBlock* d_packs = plan_alloc<dmrg::PackBlock>(H, packs.size());
    HIPCHK(hipMemcpyAsync(d_items, all_items.data(), all_items.size() * sizeof(all_items[0]), hipMemcpyHostToDevice, s));
    HIPCHK(hipMemcpyAsync(d_tasks, dtasks.data(), dtasks.size() * sizeof(dtasks[0]), hipMemcpyHostToDevice, s));
    if (!all_red.empty())
        HIPCHK(hipMemcpyAsync(d_red, all_red.data(), all_red.size() * sizeof(all_red[0]), hipMemcpyHostToDevice, s));
    HIPCHK(hipMemcpyAsync(d_packs, packs.data(), packs.size() * sizeof(packs[0]), hipMemcpyHostToDevice, s));
    if (!only) H.d_tasks = d_tasks;
    plan.items = d_items;
    plan.reduces = d_red;
    plan.tasks = d_tasks;
    plan.partial = plan_alloc<double>(H, (size_t)std::max<int64_t>(part_max, 1) * H.vec_step);
    plan.partial_size = part_max;
    plan.launches = launches_out.data();
    plan.phases = phases_out.data();
    plan.packs = d_packs;
    plan.n_packs = (int)packs.size();
    plan.packed_size = psize;
    plan.xp = plan_alloc<double>(H, (size_t)psize * H.vec_step);
    if (split_bufs) {
        plan.xr_hi = plan_alloc<uint16_t>(H, (size_t)psize * H.vec_step);
        plan.xr_lo = plan_alloc<uint16_t>(H, (size_t)psize * H.vec_step);
        plan.xt_hi = plan_alloc<uint16_t>(H, (size_t)psize * H.vec_step);
        plan.xt_lo = plan_alloc<uint16_t>(H, (size_t)psize * H.vec_step);
    }
    HIPCHK(hipStreamSynchronize(s));
}

// Launch plan of the split kernels of hpsi_lds.hip. The tasks of every target block whose own and
// sources' padded dimensions are at most 96 are divided into small tasks (source one 32 x 32 tile)
// for the task-mode kernel and the others for the row-mode kernel; both lists keep the
// source order. Row-mode items cover the whole target (all rows and columns), task-mode items a row
// block of one or two row tiles; each list is cut into items of bounded cost, and a target row block
// covered by several items of one kind gets partial tiles that a reduction adds in item order.
// Targets with larger blocks (own, or every source with tune_split_task_route = 0) are flagged in
// `fallback`, and with them the tasks in `fb_task`: those the other paths (two-pass or one-wave) run.
// With tune_split_task_route, a target within 96 keeps its tasks whose source is within 96 too
// and only those with a larger source fall back, so one target can take both paths (each adds into y).
void build_lds_plan(dmrg_hop& H, hipStream_t s, std::vector<char>& fallback, std::vector<char>& fb_task) {
    const size_t nb = H.blk.size();
    fallback.assign(nb, 0);
    fb_task.assign(H.tasks.size(), 0);
    std::vector<int64_t> pk_off(nb);
    std::vector<dmrg::PackBlock> packs;
    int64_t psize = 0;
    for (size_t i = 0; i < nb; ++i) {
        int pa = dmrg::ld_of(H.blk_ma[i]), pd = dmrg::ld_of(H.blk_md[i]);
        pk_off[i] = psize;
        packs.push_back({H.blk_off[i], psize, H.blk_ma[i], H.blk_md[i], pa, pd});
        psize += (int64_t)pa * pd;
    }
    auto ident = [&](int p) -> int64_t {
        int k = p / 32 - 1;
        if (k < 0 || k >= (int)H.ident_off.size()) throw Error(DMRG_ERR_ARG, "internal: no tiled identity block");
        return H.ident_off[k];
    };
    // one run of tasks of one kernel kind for one target row block
    struct Run { int j, kind, cls, r0, c0, nr, tq; int32_t tb, te; };
    std::vector<dmrg::LTask> lt;
    lt.reserve(H.tasks.size());
    std::vector<Run> runs;
    auto row_cost = [](const dmrg::LTask& L, int tp, int tq, bool new_src) {
        return 3.0 * L.pd32 * (2.0 * L.pa32 * tp + tq * tp) + 24.0 + (new_src ? 2.0 * L.pd32 * L.pa32 : 0.0);
    };
    auto small_cost = [](int nr, int tq) { return 3.0 * (2.0 * nr + nr * tq) + 24.0; };
    CostCaps caps(H);
    size_t k = 0;
    for (size_t j = 0; j < nb; ++j) {
        size_t kb = k;
        while (k < H.tasks.size() && H.tasks[k].j == (int)j) ++k;
        if (k == kb) continue;
        const int own = std::max(dmrg::ld_of(H.blk_ma[j]), dmrg::ld_of(H.blk_md[j]));
        auto src_dim = [&](size_t t) {
            const int i = H.tasks[t].i;
            return std::max(dmrg::ld_of(H.blk_ma[i]), dmrg::ld_of(H.blk_md[i]));
        };
        int smax = own;
        for (size_t t = kb; t < k; ++t) smax = std::max(smax, src_dim(t));
        if (own > 96 || (smax > 96 && !H.tune_split_task_route)) {
            fallback[j] = 1;
            for (size_t t = kb; t < k; ++t) fb_task[t] = 1;
            continue;
        }
        if (smax > 96) {                              // per-task routing: the larger sources fall back
            fallback[j] = 1;
            for (size_t t = kb; t < k; ++t) fb_task[t] = src_dim(t) > 96;
        }
        const int nrt = dmrg::rows_of(H.blk_ma[j]) / 16, tq = dmrg::rows_of(H.blk_md[j]) / 16;
        std::vector<dmrg::LTask> big, small;
        std::vector<size_t> order;
        for (size_t t = kb; t < k; ++t)
            if (!fb_task[t]) order.push_back(t);
        if (H.tune_lds_task_order == 1)   // operator-pair order (same across targets) instead of source order
            std::stable_sort(order.begin(), order.end(), [&](size_t x, size_t y) {
                const auto &a = H.tasks[x], &b = H.tasks[y];
                if (a.lm != b.lm) return a.lm < b.lm;
                return a.rm < b.rm;
            });
        for (size_t t : order) {
            const auto& ht = H.tasks[t];
            const int a = H.blk[ht.i][0], d = H.blk[ht.i][3];
            const int pa = dmrg::ld_of(H.blk_ma[ht.i]), pd = dmrg::ld_of(H.blk_md[ht.i]);
            dmrg::LTask L;
            L.x_off = 2 * pk_off[ht.i];
            L.a_off = ht.lm >= 0 ? 2 * H.mats[ht.lm].pool_of_in[a] : ident(pa);
            L.b_off = ht.rm >= 0 ? 2 * H.mats[ht.rm].pool_of_in[d] : ident(pd);
            L.f = (float)ht.f;
            L.pa32 = (int16_t)(pa / 32);
            L.pd32 = (int16_t)(pd / 32);
            if (L.pa32 == 1 && L.pd32 == 1 && H.tune_small_mode) small.push_back(L);
            else big.push_back(L);
        }
        if (!big.empty()) {
            // source and target columns within 64 -> S = 64 run, rest -> S = 96
            const int tp = nrt > dmrg::kLdsRows ? 2 : 1;
            std::vector<dmrg::LTask> b64, b96;
            for (const auto& L : big)
                (L.pa32 <= 2 && L.pd32 <= 2 && tq <= 4 && H.tune_lds_split64 ? b64 : b96).push_back(L);
            for (int S : {64, 96}) {
                const auto& v = S == 64 ? b64 : b96;
                if (v.empty()) continue;
                Run R{(int)j, S == 64 ? 0 : 1, (S == 64 ? 0 : 2) + (tp - 1), 0, 0, nrt, tq, (int32_t)lt.size(), 0};
                int64_t px = -1;
                for (const auto& L : v) {
                    lt.push_back(L);
                    caps.add((int)j, row_cost(L, tp, tq, L.x_off != px));
                    px = L.x_off;
                }
                R.te = (int32_t)lt.size();
                runs.push_back(R);
            }
        }
        if (!small.empty()) {
            const int tb = (int32_t)lt.size();
            for (const auto& L : small) lt.push_back(L);
            const int te = (int32_t)lt.size();
            // classes (1,2) (2,2) (1,4); targets wider than 4 column tiles get column blocks
            const int NQ = tq <= 2 && H.tune_small_nq <= 2 ? 2 : 4;
            const int NR = NQ == 2 && nrt > 1 && H.tune_small_nr > 1 ? 2 : 1;
            const int cls = NQ == 4 ? 2 : NR - 1;
            for (int r = 0; r < nrt; r += NR)
                for (int c = 0; c < tq; c += NQ) {
                    const int nr = std::min(NR, nrt - r), nq = std::min(NQ, tq - c);
                    runs.push_back({(int)j, 2, cls, 16 * r, 16 * c, nr, nq, tb, te});
                    caps.add((int)j, (te - tb) * small_cost(nr, nq));
                }
        }
    }
    H.lplan = dmrg::LdsPlan{};
    struct It { dmrg::Item item; double cost; int kind, cls; };
    std::vector<It> its;
    std::vector<dmrg::Reduce> reds_k[dmrg::kReduceKinds];
    int64_t part = 0;
    for (const Run& R : runs) {
        const int tp = R.kind < 2 && R.nr > dmrg::kLdsRows ? 2 : 1;
        std::vector<std::pair<int32_t, int32_t>> chunks;
        std::vector<double> ccost;
        int32_t b = R.tb;
        double c = 0.0;
        int64_t px = -1;
        const double cmax = caps.cap(R.j, H.tune_lds_items, 600.0);
        for (int32_t t = R.tb; t < R.te; ++t) {
            const double tc = R.kind < 2 ? row_cost(lt[t], tp, R.tq, lt[t].x_off != px || t == b) : small_cost(R.nr, R.tq);
            px = lt[t].x_off;
            if (c + tc > cmax && t > b) { chunks.push_back({b, t}); ccost.push_back(c); b = t; c = 0.0; }
            c += tc;
        }
        chunks.push_back({b, R.te});
        ccost.push_back(c);
        const int j = R.j;
        const int tm = 16 * R.nr, tn = 16 * R.tq;
        if (chunks.size() == 1) {
            its.push_back({{H.blk_off[j], -1, H.blk_ma[j], H.blk_md[j], R.r0, R.c0, chunks[0].first, chunks[0].second},
                           ccost[0], R.kind, R.cls});
        } else {
            reds_k[R.kind].push_back({H.blk_off[j], part, H.blk_ma[j], H.blk_md[j], R.r0, R.c0, tm, tn,
                                      (int32_t)chunks.size(), 0});
            for (size_t q = 0; q < chunks.size(); ++q) {
                its.push_back({{H.blk_off[j], part, H.blk_ma[j], H.blk_md[j], R.r0, R.c0, chunks[q].first,
                                chunks[q].second},
                               ccost[q], R.kind, R.cls});
                part += (int64_t)tm * tn;
            }
        }
    }
    // launch order: row-mode classes, then task-mode classes; heaviest item first inside a class
    for (It& x : its) x.kind = x.kind < 2 ? 0 : 1;
    std::stable_sort(its.begin(), its.end(), [](const It& a, const It& b) {
        if (a.kind != b.kind) return a.kind < b.kind;
        if (a.cls != b.cls) return a.cls < b.cls;
        return a.cost > b.cost;
    });
    if (H.tune_lds_order == 2 && H.n_parts > 1) {
        // merged problems: inside a class, the items of one problem stay together (heaviest first),
        // so that the workgroups running at one time share that problem's operators in the caches
        auto part_of = [&](int64_t y_off) {
            return (int)(std::upper_bound(H.part_coeff.begin(), H.part_coeff.end(), y_off) - H.part_coeff.begin());
        };
        std::stable_sort(its.begin(), its.end(), [&](const It& a, const It& b) {
            if (a.kind != b.kind) return a.kind < b.kind;
            if (a.cls != b.cls) return a.cls < b.cls;
            const int pa = part_of(a.item.y_off), pb = part_of(b.item.y_off);
            if (pa != pb) return pa < pb;
            return a.cost > b.cost;
        });
    }
    if (H.tune_lds_order == 1) {
        // XCD-aware: workgroups are dealt to the 8 XCDs round-robin, so items at positions of one
        // residue mod 8 share an L2. Items of targets with the same left sector (which read the same
        // left operator blocks) are kept on one XCD; sectors are balanced over the XCDs by cost.
        constexpr int nx = 8;
        size_t c0 = 0;
        std::vector<It> out;
        out.reserve(its.size());
        while (c0 < its.size()) {
            size_t c1 = c0;
            while (c1 < its.size() && its[c1].kind == its[c0].kind && its[c1].cls == its[c0].cls) ++c1;
            std::map<int, std::vector<size_t>> grp;
            std::map<int, double> gcost;
            for (size_t i = c0; i < c1; ++i) {
                const int a = H.blk[std::lower_bound(H.blk_off.begin(), H.blk_off.end(), its[i].item.y_off) -
                                    H.blk_off.begin()][0];
                grp[a].push_back(i);
                gcost[a] += its[i].cost;
            }
            std::vector<std::pair<double, int>> gorder;
            for (auto& kv : gcost) gorder.push_back({-kv.second, kv.first});
            std::sort(gorder.begin(), gorder.end());
            std::vector<double> load(nx, 0.0);
            std::vector<std::vector<size_t>> lane(nx);
            for (auto& og : gorder) {
                const int x = (int)(std::min_element(load.begin(), load.end()) - load.begin());
                load[x] -= og.first;
                for (size_t i : grp[og.second]) lane[x].push_back(i);
            }
            std::vector<size_t> pos(nx, 0);
            for (size_t left = c1 - c0, p = 0; left > 0; ++p) {
                int x = (int)(p % nx);
                if (pos[x] >= lane[x].size()) {
                    size_t rem = 0;
                    for (int y2 = 0; y2 < nx; ++y2)
                        if (lane[y2].size() - pos[y2] > rem) { rem = lane[y2].size() - pos[y2]; x = y2; }
                }
                out.push_back(its[lane[x][pos[x]++]]);
                --left;
            }
            c0 = c1;
        }
        its.swap(out);
    }
    std::vector<dmrg::Item> items;
    items.reserve(its.size());
    int cnt_row[dmrg::kLdsClasses] = {0}, cnt_small[dmrg::kSmallClasses] = {0};
    for (const It& x : its) {
        items.push_back(x.item);
        if (x.kind == 0) cnt_row[x.cls]++; else cnt_small[x.cls]++;
    }
    H.lplan.cls_begin[0] = 0;
    for (int c = 0; c < dmrg::kLdsClasses; ++c) H.lplan.cls_begin[c + 1] = H.lplan.cls_begin[c] + cnt_row[c];
    H.lplan.small_begin[0] = H.lplan.cls_begin[dmrg::kLdsClasses];
    for (int c = 0; c < dmrg::kSmallClasses; ++c) H.lplan.small_begin[c + 1] = H.lplan.small_begin[c] + cnt_small[c];
    H.n_fallback_targets = 0;
    for (char f : fallback) H.n_fallback_targets += f;
    std::vector<dmrg::Reduce> reds;
    H.lplan.red_begin[0] = 0;
    for (int kk = 0; kk < dmrg::kReduceKinds; ++kk) {
        int mx = 1;
        for (const auto& r : reds_k[kk]) mx = std::max(mx, r.tm * r.tn);
        H.lplan.red_chunks[kk] = (mx + 255) / 256;
        reds.insert(reds.end(), reds_k[kk].begin(), reds_k[kk].end());
        H.lplan.red_begin[kk + 1] = (int)reds.size();
    }
    tag_parts(H, items);
    tag_parts(H, reds);
    dmrg::Item* d_items = plan_alloc<dmrg::Item>(H, items.size());
    dmrg::LTask* d_lt = plan_alloc<dmrg::LTask>(H, lt.size());
    dmrg::Reduce* d_red = plan_alloc<dmrg::Reduce>(H, reds.size());
    dmrg::PackBlock* d_packs = plan_alloc<dmrg::PackBlock>(H, packs.size());
    if (!items.empty())
        HIPCHK(hipMemcpyAsync(d_items, items.data(), items.size() * sizeof(items[0]), hipMemcpyHostToDevice, s));
    if (!lt.empty()) HIPCHK(hipMemcpyAsync(d_lt, lt.data(), lt.size() * sizeof(lt[0]), hipMemcpyHostToDevice, s));
    if (!reds.empty()) HIPCHK(hipMemcpyAsync(d_red, reds.data(), reds.size() * sizeof(reds[0]), hipMemcpyHostToDevice, s));
    HIPCHK(hipMemcpyAsync(d_packs, packs.data(), packs.size() * sizeof(packs[0]), hipMemcpyHostToDevice, s));
    H.lplan.items = d_items;
    H.lplan.tasks = d_lt;
    H.lplan.reduces = d_red;

    H.lplan.partial_size = part;
    H.lplan.partial = plan_alloc<double>(H, (size_t)std::max<int64_t>(part, 1) * H.vec_step);
    H.lplan.packs = d_packs;
    H.lplan.n_packs = (int)packs.size();
    H.lplan.xt_size = 2 * psize;
    H.lplan.xt = plan_alloc<uint16_t>(H, (size_t)2 * psize * H.vec_step + dmrg::kOperandSlack / sizeof(uint16_t));
    if (const char* e = std::getenv("DMRG_PLAN_TRACE"))
        if (e[0] == '1') {
            std::fprintf(stderr, "[dmrg lds plan] items %zu row classes", items.size());
            for (int c = 0; c < dmrg::kLdsClasses; ++c) std::fprintf(stderr, " %d", cnt_row[c]);
            std::fprintf(stderr, " small classes");
            for (int c = 0; c < dmrg::kSmallClasses; ++c) std::fprintf(stderr, " %d", cnt_small[c]);
            std::fprintf(stderr, " reduces %zu partial %.1f MB fallback %d\n", reds.size(), part * 8e-6,
                         H.n_fallback_targets);
        }
    HIPCHK(hipStreamSynchronize(s));
}

// Work dealt to the 8 XCDs (workgroups go to them in turn, so entries at positions of one residue modulo 8
// share an L2): the entries of a unit stay on one XCD, the least loaded when the unit opens.
template <class T>
struct XcdDeal {
    T none;                      // filler of the shorter lists
    std::vector<T> list[8];
    double load[8] = {0.0};
    int x = 0;
    void open(double cost) {
        x = (int)(std::min_element(load, load + 8) - load);
        load[x] += cost;
    }
    void add(const T& v) { list[x].push_back(v); }
    void take(std::vector<T>& out) {
        size_t n = 0;
        for (const auto& l : list) n = std::max(n, l.size());
        for (size_t i = 0; i < n; ++i)
            for (const auto& l : list) out.push_back(i < l.size() ? l[i] : none);
        for (auto& l : list) l.clear();
        std::fill(load, load + 8, 0.0);
    }
};

// f(first tile, tiles) of the parts of at most `most` tiles that n tiles are cut into
template <class F>
void for_parts(int n, int most, F&& f) {
    for (int t = 0; t < n; t += dmrg::part_len(n, t, most)) f(t, dmrg::part_len(n, t, most));
}

}  // namespace

void drop_graphs(dmrg_hop& H) {
    for (auto& g : H.graphs) {
        (void)hipGraphExecDestroy(g.exec);
        (void)hipGraphDestroy(g.graph);
    }
    H.graphs.clear();
}

namespace {

// Targets whose own or some source's dimension exceeds `limit` (96 for the split row-mode kernel,
// 128 for the FP64 register-streamed kernel).
std::vector<char> large_targets(const dmrg_hop& H, int limit = 96) {
    std::vector<int> smax(H.blk.size(), 0);
    for (size_t j = 0; j < H.blk.size(); ++j) smax[j] = std::max(H.blk_ma[j], H.blk_md[j]);
    for (const auto& t : H.tasks) smax[t.j] = std::max({smax[t.j], H.blk_ma[t.i], H.blk_md[t.i]});
    std::vector<char> big(H.blk.size(), 0);
    for (size_t j = 0; j < H.blk.size(); ++j) big[j] = smax[j] > limit;
    return big;
}

// Launch plan of the two-pass path, split (hpsi_big.hip) or FP64 (hpsi_big64.hip), for the targets flagged in
// `big`, without the tasks that run elsewhere. Targets are grouped into chunks whose T buffers (one per task:
// target rows x source columns, in tiles) stay below the T budget. A wavefront owns up to 64 x 64 elements:
// both extents are cut into equal parts, so that the parts of one block differ by a tile at most. Per
// chunk, pass 1 has one piece of work per task and part of its T; pass 2 one item per part of a target and
// task range, the task lists cut into ranges of about tune_big_stages T tiles whose partial sums a reduction
// adds in order. The pieces of one task, and those of one range of a target, read the same operands: they
// are dealt together to one XCD, the least loaded so far.
void build_big_plan(dmrg_hop& H, hipStream_t s, const std::vector<char>& big, bool fp64, const std::vector<char>& task_keep) {
    dmrg::BigPlan& plan = fp64 ? H.bplan64 : H.bplan;
    std::vector<dmrg::BigChunk>& chunks = fp64 ? H.big_chunks64 : H.big_chunks;
    plan = dmrg::BigPlan{};
    chunks.clear();
    const int tw = fp64 ? 16 : 32, j_most = 64 / tw;                  // width of a T tile; tile columns of a part
    const int64_t tile = fp64 ? 256 : dmrg::kTileU16;
    const int64_t t_budget = (int64_t)H.tune_big_tbudget_mb << (fp64 ? 18 : 19);   // T elements per chunk
    auto cols = [&](int i) { return (H.blk_md[i] + tw - 1) / tw; };
    // operands of a task (identity factors: identity blocks); < 0: none
    std::vector<int64_t> xt_off = H.xt64_off;
    if (!fp64) {
        xt_off.resize(H.blk.size());
        int64_t at = 0;
        for (size_t i = 0; i < H.blk.size(); ++i) {
            xt_off[i] = 2 * at;
            at += (int64_t)dmrg::ld_of(H.blk_ma[i]) * dmrg::ld_of(H.blk_md[i]);
        }
    }
    auto operand = [&](int m, int sector, int dim) -> int64_t {
        if (fp64) return op64_of(H, m, sector, dim);
        if (m >= 0) return 2 * H.mats[m].pool_of_in[sector];
        const int k = dmrg::ld_of(dim) / 32 - 1;
        return k < (int)H.ident_off.size() ? H.ident_off[k] : -1;
    };
    std::vector<dmrg::BigT> t1;
    std::vector<dmrg::BigT2> t2;
    std::vector<dmrg::Item> items;
    std::vector<dmrg::Reduce> reds;
    XcdDeal<dmrg::BigT> deal1{dmrg::BigT{}};
    dmrg::Item none{};
    none.part_off = -1;
    XcdDeal<dmrg::Item> deal2{none};
    int64_t part_max = 0, tbuf_max = 0, tsize = 0, part = 0;
    int red_max = 1;
    size_t pieces = 0, ranges = 0;
    dmrg::BigChunk cur{0, 0, 0, 0, 0, 0};
    bool open = false;
    auto close_chunk = [&]() {
        if (!open) return;
        cur.t1_begin = (int)t1.size();
        deal1.take(t1);
        cur.t1_end = (int)t1.size();
        cur.item_begin = (int)items.size();
        deal2.take(items);
        cur.item_end = (int)items.size();
        cur.red_end = (int)reds.size();
        chunks.push_back(cur);
        cur = dmrg::BigChunk{0, 0, 0, 0, (int)reds.size(), 0};
        part_max = std::max(part_max, part);
        tbuf_max = std::max(tbuf_max, tsize);
        tsize = part = 0;
        open = false;
    };
    size_t k = 0;
    for (size_t j = 0; j < H.blk.size(); ++j) {
        const size_t kb = k;
        while (k < H.tasks.size() && H.tasks[k].j == (int)j) ++k;
        if (!big[j]) continue;
        const int ma = H.blk_ma[j], md = H.blk_md[j], nrt = (ma + 15) / 16, nq = (md + 15) / 16;
        auto t_size = [&](const dmrg_hop::HTask& t) { return (int64_t)nrt * cols(t.i) * tile; };
        int64_t need = 0;
        for (size_t t = kb; t < k; ++t)
            if (task_keep[t]) need += t_size(H.tasks[t]);
        if (need == 0) continue;                  // every task of the target runs elsewhere
        if (tsize > 0 && tsize + need > t_budget) close_chunk();
        open = true;
        const int32_t part_j = H.n_parts > 1 ? part_of(H, H.blk_off[j]) : 0;
        std::vector<std::pair<int32_t, int32_t>> cuts;   // ranges of t2
        std::vector<double> cost;
        int32_t b0 = (int32_t)t2.size();
        int c = 0;
        for (size_t t = kb; t < k; ++t) {
            if (!task_keep[t]) continue;
            const auto& ht = H.tasks[t];
            const int sa = H.blk_ma[ht.i], sd = H.blk_md[ht.i], pd = cols(ht.i);
            const int64_t a = operand(ht.lm, H.blk[ht.i][0], sa), b = operand(ht.rm, H.blk[ht.i][3], sd);
            if (a < 0 || b < 0) throw Error(DMRG_ERR_ARG, "internal: no operand block");
            const int ka = fp64 ? dmrg::k4_of(sa) : (sa + 31) / 32, kd = fp64 ? dmrg::k4_of(sd) : pd;
            deal1.open((double)nrt * pd * ka);
            for_parts(nrt, 4, [&](int rb, int nr) {
                for_parts(pd, j_most, [&](int jb, int nj) {
                    deal1.add({xt_off[ht.i], a, tsize, ht.f, ka, kd, dmrg::k4_of(ma), pd, (int16_t)rb, (int16_t)nr,
                               (int16_t)jb, (int16_t)nj, part_j, 0});
                    ++pieces;
                });
            });
            if (c >= H.tune_big_stages) {
                cuts.push_back({b0, (int32_t)t2.size()});
                b0 = (int32_t)t2.size();
                c = 0;
            }
            if (c == 0) cost.push_back(0.0);
            c += pd;
            cost.back() += (double)nrt * nq * kd;
            t2.push_back({tsize, b, pd, kd});
            tsize += t_size(ht);
        }
        cuts.push_back({b0, (int32_t)t2.size()});
        const int64_t part0 = part;
        for (size_t q = 0; q < cuts.size(); ++q) {
            deal2.open(cost[q]);
            int64_t at = part0;                  // the records' partial tiles of this target, n_parts each
            for_parts(nrt, 4, [&](int rb, int nr) {
                for_parts(nq, 4, [&](int qb, int nqw) {
                    const int tm = 16 * nr, tn = 16 * nqw;
                    dmrg::Item it{H.blk_off[j], -1, ma, md, 16 * rb, 16 * qb, cuts[q].first, cuts[q].second};
                    if (cuts.size() > 1) {
                        it.part_off = at + (int64_t)q * tm * tn;
                        if (q == 0) {
                            reds.push_back({H.blk_off[j], at, ma, md, 16 * rb, 16 * qb, tm, tn, (int32_t)cuts.size(), 0});
                            red_max = std::max(red_max, tm * tn);
                        }
                        at += (int64_t)cuts.size() * tm * tn;
                    }
                    deal2.add(it);
                    ++ranges;
                });
            });
            part = std::max(part, at);
        }
    }
    close_chunk();
    if (t2.empty()) return;
    tag_parts(H, items);
    tag_parts(H, reds);
    auto upload = [&](const auto& v) {
        using T = typename std::decay_t<decltype(v)>::value_type;
        T* d = plan_alloc<T>(H, std::max<size_t>(v.size(), 1));
        if (!v.empty()) HIPCHK(hipMemcpyAsync(d, v.data(), v.size() * sizeof(T), hipMemcpyHostToDevice, s));
        return d;
    };
    plan.t1 = upload(t1);
    plan.t2 = upload(t2);
    plan.items = upload(items);
    plan.reduces = upload(reds);
    plan.chunks = chunks.data();
    plan.n_chunks = (int)chunks.size();
    plan.red_chunks = (red_max + 255) / 256;
    const size_t t_bytes = (size_t)std::max<int64_t>(tbuf_max, 4) * (fp64 ? sizeof(double) : sizeof(uint16_t));
    plan.tbuf = reinterpret_cast<uint16_t*>(plan_alloc<double>(H, t_bytes / sizeof(double)));
    plan.partial = plan_alloc<double>(H, (size_t)std::max<int64_t>(part_max, 1));
    plan.partial_size = part_max;
    if (const char* e = std::getenv("DMRG_PLAN_TRACE"))
        if (e[0] == '1')
            std::fprintf(stderr, "[dmrg big plan%s] chunks %zu pass-1 groups %zu pass-2 items %zu reduces %zu T %.1f MB "
                         "partial %.1f MB\n", fp64 ? " fp64" : "", chunks.size(), pieces, ranges, reds.size(), t_bytes * 1e-6, part_max * 8e-6);
    HIPCHK(hipStreamSynchronize(s));
}

// Operand pool of the FP64 MFMA kernels: every pool block in the operand form of internal.h (offsets per
// matrix and ket sector in MatDef::op64_of_in), identity blocks of the psi blocks' sizes (by 4-row
// groups), which stand in for identity factors. Made once. Also the places of the
// packed X^T of every psi block.
void make_op64(dmrg_hop& H, hipStream_t s) {
    if (H.d_op64) return;
    std::vector<dmrg::OpBlock64> ob;
    ob.reserve(H.pool_blocks.size());
    int64_t n = 0;
    for (const auto& pb : H.pool_blocks) {       // ascending pool offsets
        ob.push_back({pb.off, n, 32 * pb.k32, pb.rows, pb.cols, 0});
        n += dmrg::op64_size(pb.rows, pb.cols);
    }
    for (MatDef& m : H.mats) {
        m.op64_of_in.assign(m.pool_of_in.size(), -1);
        for (size_t q = 0; q < m.pool_of_in.size(); ++q) {
            if (m.pool_of_in[q] < 0) continue;
            // the last block at this offset: empty blocks take no room and share it with their successor
            auto it = std::upper_bound(ob.begin(), ob.end(), m.pool_of_in[q],
                                       [](int64_t off, const dmrg::OpBlock64& o) { return off < o.src; });
            if (it == ob.begin() || (it - 1)->src != m.pool_of_in[q]) throw Error(DMRG_ERR_ARG, "internal: not a pool block");
            m.op64_of_in[q] = (it - 1)->dst;
        }
    }
    int widest = 0;
    for (size_t i = 0; i < H.blk.size(); ++i) widest = std::max({widest, dmrg::k4_of(H.blk_ma[i]), dmrg::k4_of(H.blk_md[i])});
    H.ident64_off.assign(widest + 1, -1);
    std::vector<double> tail;                    // the identity blocks
    auto add_ident = [&](int m) {
        const int r4 = dmrg::k4_of(m);
        if (H.ident64_off[r4] >= 0) return;
        const size_t base = tail.size();
        H.ident64_off[r4] = n + (int64_t)base;
        tail.resize(base + (size_t)dmrg::op64_size(4 * r4, 4 * r4), 0.0);
        for (int i = 0; i < 4 * r4; ++i) {       // element (i, i): group p, row tile, g, li, u
            const int p = i / 8, rt = i / 16, w = std::min(16, 4 * r4 - 16 * rt), g = i % 4, u = (i % 8) / 4;
            tail[base + (size_t)p * r4 * 32 + rt * 128 + (g * w + i % 16) * 2 + u] = 1.0;
        }
    };
    for (const auto& t : H.tasks) {
        if (t.lm < 0) add_ident(H.blk_ma[t.i]);
        if (t.rm < 0) add_ident(H.blk_md[t.i]);
    }
    H.op64_len = n + (int64_t)tail.size() + dmrg::kOperandSlack / (int64_t)sizeof(double);
    H.d_op64 = dev_alloc<double>(H, H.op64_len);
    dmrg::OpBlock64* d_ob = dev_alloc<dmrg::OpBlock64>(H, ob.size());
    HIPCHK(hipMemcpyAsync(d_ob, ob.data(), ob.size() * sizeof(ob[0]), hipMemcpyHostToDevice, s));
    if (!tail.empty())
        HIPCHK(hipMemcpyAsync(H.d_op64 + n, tail.data(), tail.size() * sizeof(double), hipMemcpyHostToDevice, s));
    HIPCHK(dmrg::launch_op64(H.d_pool, d_ob, (int)ob.size(), H.d_op64, s));
    HIPCHK(hipStreamSynchronize(s));   // the staging vectors go out of scope
}

// Packing of X^T into operand form (every psi block).
void build_pack64(dmrg_hop& H, hipStream_t s) {
    std::vector<dmrg::PackBlock> packs;
    H.xt64_off.resize(H.blk.size());
    int64_t n = 0;
    for (size_t i = 0; i < H.blk.size(); ++i) {
        H.xt64_off[i] = n;
        packs.push_back({H.blk_off[i], n, H.blk_ma[i], H.blk_md[i], 0, 0});
        n += dmrg::op64_size(H.blk_md[i], H.blk_ma[i]);
    }
    dmrg::PackBlock* d = plan_alloc<dmrg::PackBlock>(H, packs.size());
    HIPCHK(hipMemcpyAsync(d, packs.data(), packs.size() * sizeof(packs[0]), hipMemcpyHostToDevice, s));
    H.xt64 = plan_alloc<double>(H, (size_t)n + dmrg::kOperandSlack / sizeof(double));
    H.packs64 = d;
    H.n_packs64 = (int)packs.size();
    HIPCHK(hipStreamSynchronize(s));
}

// Launch plan of the register-streamed FP64 kernel (hpsi_rs64.hip) for the targets and sources within its
// 128 x 128 (targets flagged in `large` are skipped, and so are tasks whose source is a single 32 x 32
// tile unless tune_lds64_small; `taken` marks the tasks taken). A target's tasks (source order) form up
// to three runs, sources of at most 32 rows, of more, and those of blocks above 96; each run is cut into
// items of bounded cost (the MFMAs of one wavefront over whole 16-wide tiles plus a per-step and per-task
// overhead), an item is run by one wavefront per row tile, its class the least that holds its tasks, and
// a target covered by several items gets partial tiles that a reduction adds in item order. Runs, cuts
// and orders fix the order of every sum: results do not depend on the classes.
void build_rs64_plan(dmrg_hop& H, hipStream_t s, const std::vector<char>& large, std::vector<char>& taken) {
    const size_t nb = H.blk.size();
    taken.assign(H.tasks.size(), 0);
    auto k16 = [](int k4) { return (k4 + 3) / 4; };
    auto cost = [&](const dmrg::LTask64& L, int tq) { return k16(L.kd4) * (4.0 * (k16(L.ka4) + tq) + 6.0) + 4.0; };
    struct Run { int j, bucket, tq; int32_t tb, te; };   // bucket: kind of source and target, for the plan trace alone
    std::vector<dmrg::LTask64> lt;
    lt.reserve(H.tasks.size());
    std::vector<Run> runs;
    CostCaps caps(H);
    constexpr int kMax = dmrg::kRsMaxTiles;
    std::vector<dmrg::LTask64> v[3];
    size_t k = 0;
    for (size_t j = 0; j < nb; ++j) {
        const size_t kb = k;
        while (k < H.tasks.size() && H.tasks[k].j == (int)j) ++k;
        if (k == kb || large[j]) continue;
        const int nrt = dmrg::rows_of(H.blk_ma[j]) / 16, tq = dmrg::rows_of(H.blk_md[j]) / 16;
        if (nrt > kMax || tq > kMax) throw Error(DMRG_ERR_ARG, "internal: FP64 target beyond 128 x 128");
        const bool wide = nrt > 6 || tq > 6;
        for (size_t t = kb; t < k; ++t) {
            const auto& ht = H.tasks[t];
            const int ma = H.blk_ma[ht.i], md = H.blk_md[ht.i];
            if (!H.tune_lds64_small && ma <= 32 && md <= 32) continue;   // single-tile source: one-wave kernel
            if (std::max(ma, md) > 16 * kMax) continue;                  // source above the tiles: other paths
            taken[t] = 1;
            const dmrg::LTask64 L{H.xt64_off[ht.i], op64_of(H, ht.lm, H.blk[ht.i][0], ma),
                                  op64_of(H, ht.rm, H.blk[ht.i][3], md), ht.f, dmrg::k4_of(ma), dmrg::k4_of(md)};
            v[wide || L.ka4 > 24 ? 2 : L.ka4 <= 8 ? 0 : 1].push_back(L);
        }
        for (int c = 0; c < 3; ++c) {
            if (v[c].empty()) continue;
            Run R{(int)j, c == 2 ? 4 : 2 * c + (tq > 3), tq, (int32_t)lt.size(), 0};
            for (const auto& L : v[c]) {
                lt.push_back(L);
                caps.add((int)j, cost(L, tq));
            }
            R.te = (int32_t)lt.size();
            runs.push_back(R);
            v[c].clear();
        }
    }
    H.rplan64 = dmrg::RsPlan64{};
    struct It { dmrg::Item item; double cost; int cls; };
    std::vector<It> its;
    std::vector<dmrg::Reduce> reds;
    int64_t part = 0;
    int most = 1, bucket[5] = {0};
    // the runs of one target are consecutive; all their chunks share one
    // reduction record, so that no two records of the one reduction launch add into the same tile
    for (size_t r0 = 0, r1; r0 < runs.size(); r0 = r1) {
        r1 = r0;
        while (r1 < runs.size() && runs[r1].j == runs[r0].j) ++r1;
        struct Chunk { int32_t b, e; double cost; int cls; };
        std::vector<Chunk> chunks;
        for (size_t r = r0; r < r1; ++r) {
            const Run& R = runs[r];
            int32_t b = R.tb;
            double c = 0.0;
            const double cmax = caps.cap(R.j, H.tune_lds64_items, 200.0);
            auto close = [&](int32_t e) {
                int ka4 = 0, kd4 = 0;
                for (int32_t t = b; t < e; ++t) { ka4 = std::max(ka4, lt[t].ka4); kd4 = std::max(kd4, lt[t].kd4); }
                chunks.push_back({b, e, c, 8 * dmrg::rs_kclass(ka4, kd4) + dmrg::rs_qclass(R.tq)});
                bucket[R.bucket]++;
            };
            for (int32_t t = R.tb; t < R.te; ++t) {
                const double tc = cost(lt[t], R.tq);
                if (c + tc > cmax && t > b) { close(t); b = t; c = 0.0; }
                c += tc;
            }
            close(R.te);
        }
        const int j = runs[r0].j, tm = dmrg::rows_of(H.blk_ma[j]), tn = 16 * runs[r0].tq;
        const bool cut = chunks.size() > 1;
        if (cut) {
            reds.push_back({H.blk_off[j], part, H.blk_ma[j], H.blk_md[j], 0, 0, tm, tn, (int32_t)chunks.size(), 0});
            most = std::max(most, tm * tn);
        }
        for (const Chunk& q : chunks) {
            its.push_back({{H.blk_off[j], cut ? part : -1, H.blk_ma[j], H.blk_md[j], 0, q.cls, q.b, q.e}, q.cost, q.cls});
            if (cut) part += (int64_t)tm * tn;
        }
    }
    // per launch group, the items (heaviest first) are dealt to the XCDs by load; an item's row tiles
    // follow one another in its XCD's workgroups and share the operands they read in that XCD's caches.
    // Workgroup b runs on XCD b % 8.
    std::stable_sort(its.begin(), its.end(), [](const It& a, const It& b) { return a.cost > b.cost; });
    std::vector<dmrg::Item> items;
    auto own_group = [](const It& x) { return dmrg::rs_group(x.cls / 8, x.cls % 8); };
    // A group with less than a quarter of the work joins the next one's launch: one launch less, and the last
    // wavefronts of both overlap, against fewer wavefronts per SIMD for the smaller classes (17 orbitals, 333
    // states: 228 us, 241 us with every group by itself; 24 orbitals, 1024 states: no difference).
    int group[dmrg::kRsGroups];
    {
        double work[dmrg::kRsGroups] = {0.0}, all = 0.0;
        int top = 0;
        for (const It& x : its) {
            const int g = own_group(x);
            work[g] += x.cost * (dmrg::rows_of(x.item.m_ap) / 16);
            all += x.cost * (dmrg::rows_of(x.item.m_ap) / 16);
            top = std::max(top, g);
        }
        for (int g = 0; g < dmrg::kRsGroups; ++g) group[g] = g;
        for (int g = 0; g < top; ++g)
            if (work[g] < 0.25 * all) {
                work[g + 1] += work[g];
                for (int i = 0; i <= g; ++i)
                    if (group[i] == g) group[i] = g + 1;
            }
    }
    for (int g = 0; g < dmrg::kRsGroups; ++g) {
        constexpr int kXcds = 8;
        std::vector<dmrg::Item> list[kXcds];
        double load[kXcds] = {0.0};
        for (const It& x : its) {
            if (group[own_group(x)] != g) continue;
            const int to = (int)(std::min_element(load, load + kXcds) - load);
            for (int rt = 0; rt < dmrg::rows_of(x.item.m_ap) / 16; ++rt) {
                list[to].push_back(x.item);
                list[to].back().r0 = 16 * rt;
                load[to] += x.cost;
            }
        }
        size_t wgs = 0;
        for (const auto& l : list) wgs = std::max(wgs, (l.size() + dmrg::kRsWaves - 1) / dmrg::kRsWaves);
        dmrg::Item none{};
        none.part_off = -1;                      // t_begin == t_end: no work
        for (size_t w = 0; w < wgs; ++w)
            for (const auto& l : list)
                for (size_t i = w * dmrg::kRsWaves; i < (w + 1) * dmrg::kRsWaves; ++i) items.push_back(i < l.size() ? l[i] : none);
        H.rplan64.begin[g + 1] = (int)items.size();
    }
    tag_parts(H, items);
    tag_parts(H, reds);
    dmrg::Item* d_items = plan_alloc<dmrg::Item>(H, items.size());
    dmrg::LTask64* d_lt = plan_alloc<dmrg::LTask64>(H, lt.size());
    dmrg::Reduce* d_red = plan_alloc<dmrg::Reduce>(H, reds.size());
    if (!items.empty())
        HIPCHK(hipMemcpyAsync(d_items, items.data(), items.size() * sizeof(items[0]), hipMemcpyHostToDevice, s));
    if (!lt.empty()) HIPCHK(hipMemcpyAsync(d_lt, lt.data(), lt.size() * sizeof(lt[0]), hipMemcpyHostToDevice, s));
    if (!reds.empty()) HIPCHK(hipMemcpyAsync(d_red, reds.data(), reds.size() * sizeof(reds[0]), hipMemcpyHostToDevice, s));
    H.rplan64.items = d_items;
    H.rplan64.tasks = d_lt;
    H.rplan64.reduces = d_red;
    H.rplan64.n_reduces = (int)reds.size();
    H.rplan64.red_chunks = (most + 255) / 256;
    H.rplan64.partial = plan_alloc<double>(H, (size_t)std::max<int64_t>(part, 1));
    H.rplan64.partial_size = part;
    H.rplan64.n_items = (int)its.size();
    if (const char* e = std::getenv("DMRG_PLAN_TRACE"))
        if (e[0] == '1') {
            std::fprintf(stderr, "[dmrg lds64 plan] items %zu classes", its.size());
            for (int c = 0; c < 5; ++c) std::fprintf(stderr, " %d", bucket[c]);
            std::fprintf(stderr, " reduces %zu partial %.1f MB\n", reds.size(), part * 8e-6);
            // what is launched: items by kernel class (8 k + q), wavefronts by launch group before and after joining
            int cls[56] = {0}, own[dmrg::kRsGroups] = {0}, run[dmrg::kRsGroups] = {0};
            for (const It& x : its) {
                const int w = dmrg::rows_of(x.item.m_ap) / 16, g = own_group(x);
                cls[x.cls]++;
                own[g] += w;
                run[group[g]] += w;
            }
            std::fprintf(stderr, "[dmrg rs64 plan] classes");
            for (int c = 0; c < 56; ++c)
                if (cls[c]) std::fprintf(stderr, " k%dq%d:%d", c / 8, c % 8, cls[c]);
            std::fprintf(stderr, " own");
            for (int n : own) std::fprintf(stderr, " %d", n);
            std::fprintf(stderr, " launched");
            for (int n : run) std::fprintf(stderr, " %d", n);
            std::fprintf(stderr, "\n");
        }
    HIPCHK(hipStreamSynchronize(s));
}

}  // namespace

// Every launch plan of the handle: FP64 (all targets) and, with split operators, the row-mode and task-mode
// plan plus the plans for the targets it does not cover.
void build_plan(dmrg_hop& H, hipStream_t s) {
    drop_graphs(H);
    for (void* p : H.plan_allocations) (void)hipFree(p);
    H.plan_allocations.clear();
    H.plan_bytes = 0;
    // FP64: targets and sources within 128 x 128 take the register-streamed kernel, larger ones the two-pass
    // path; what is switched off, and single-tile sources on request, the one-wave kernel
    H.bplan64 = dmrg::BigPlan{};
    H.big_chunks64.clear();
    H.rplan64 = dmrg::RsPlan64{};
    H.xt64 = nullptr;
    H.n_packs64 = 0;
    const size_t nb = H.blk.size();
    std::vector<char> big64(nb, 0), rs64;   // targets of the two-pass path; tasks of the register-streamed kernel
    bool any_big = false, any_rs = false;
    if (H.tune_big64) {
        // Every target above the limit: with tiles cut to the block no extent is too small for the two-pass
        // path. 76 orbitals at bond dimension 6000 (one share): 25.3 ms; 30.4 ms when the few percent of the
        // work in targets within 128 x 128 with a larger source ran on the one-wavefront kernel.
        big64 = large_targets(H, H.tune_lds64 ? 16 * dmrg::kRsMaxTiles : 96);
        for (char b : big64) any_big |= b != 0;
    }
    if (H.tune_lds64 || any_big) {
        make_op64(H, s);
        build_pack64(H, s);
    }
    if (H.tune_lds64) {
        // with task routing a target within 128 x 128 keeps its tasks whose source fits too, otherwise only
        // targets whose sources all fit are taken
        std::vector<char> large = large_targets(H, 16 * dmrg::kRsMaxTiles);
        if (H.tune_lds64_task_route)
            for (size_t j = 0; j < nb; ++j) large[j] = std::max(H.blk_ma[j], H.blk_md[j]) > 16 * dmrg::kRsMaxTiles;
        build_rs64_plan(H, s, large, rs64);
        for (char b : rs64) any_rs |= b != 0;
    }
    if (any_big || any_rs) {
        std::vector<char> rest(nb), rest_tasks(H.tasks.size(), 1);
        for (size_t j = 0; j < nb; ++j) rest[j] = !big64[j];
        for (size_t t = 0; t < rs64.size(); ++t) rest_tasks[t] = !rs64[t];
        build_plan_core(H, s, &rest, false, H.plan, H.launches, H.phases, &rest_tasks);
        if (any_big) build_big_plan(H, s, big64, true, rest_tasks);
    } else {
        build_plan_core(H, s, nullptr, false, H.plan, H.launches, H.phases);
    }
    H.plan_fb = dmrg::HpsiPlan{};
    H.launches_fb.clear();
    H.phases_fb.clear();
    H.n_fallback_targets = 0;
    if (!H.has_split) return;
    std::vector<char> fb, fb_task;
    build_lds_plan(H, s, fb, fb_task);
    H.bplan = dmrg::BigPlan{};
    if (H.n_fallback_targets > 0) {
        if (H.tune_big) {
            build_big_plan(H, s, fb, false, fb_task);
            H.n_fallback_targets = 0;
        } else {
            if (!H.d_hi) throw Error(DMRG_ERR_ARG, "internal: row-major split operators missing");
            build_plan_core(H, s, &fb, true, H.plan_fb, H.launches_fb, H.phases_fb, &fb_task);
        }
    }
}


// True when some target block (or one of its sources) has a dimension above the 96 of the split row-mode
// kernel.
bool needs_fallback(const dmrg_hop& H) {
    for (char b : large_targets(H)) if (b) return true;
    return false;
}


// Tiled hi/lo copy of the whole FP64 pool (internal.h) followed by tiled identity blocks of sizes
// 32, 64, ... up to the widest padded block (hi = 1 on the diagonal, lo = 0), which stand in for
// identity factors.
void make_tiled_split(dmrg_hop& H, hipStream_t s) {
    int64_t n = 2 * H.pool_size;
    int pmax = 96;
    for (size_t i = 0; i < H.blk.size(); ++i)
        pmax = std::max({pmax, dmrg::ld_of(H.blk_ma[i]), dmrg::ld_of(H.blk_md[i])});
    std::vector<uint16_t> id;
    H.ident_off.assign(pmax / 32, -1);
    for (int k = 0; k < pmax / 32; ++k) {
        const int p = 32 * (k + 1), r16 = p / 16, k32 = p / 32;
        H.ident_off[k] = n + (int64_t)id.size();
        const size_t base = id.size();
        id.resize(base + (size_t)r16 * k32 * dmrg::kTileU16, 0);
        for (int i = 0; i < p; ++i) {
            const int rt = i / 16, kt = i / 32, lane = (i % 16) + 16 * ((i % 32) / 8), u = i % 8;
            id[base + (size_t)(rt * k32 + kt) * dmrg::kTileU16 + lane * 8 + u] = 0x3F80;   // bf16 1.0
        }
    }
    H.tiled_size = n + (int64_t)id.size() + dmrg::kOperandSlack / (int64_t)sizeof(uint16_t);
    H.d_tiled = dev_alloc<uint16_t>(H, H.tiled_size);
    dmrg::PoolBlock* d_pb = dev_alloc<dmrg::PoolBlock>(H, H.pool_blocks.size());
    HIPCHK(hipMemcpyAsync(d_pb, H.pool_blocks.data(), H.pool_blocks.size() * sizeof(dmrg::PoolBlock),
                          hipMemcpyHostToDevice, s));
    HIPCHK(hipMemcpyAsync(H.d_tiled + n, id.data(), id.size() * sizeof(uint16_t), hipMemcpyHostToDevice, s));
    HIPCHK(dmrg::launch_split_tiled(H.d_pool, d_pb, (int)H.pool_blocks.size(), H.d_tiled, s));
    HIPCHK(hipStreamSynchronize(s));   // the staging vector goes out of scope
}


}  // namespace dmrg
