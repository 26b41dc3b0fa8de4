// Host planner of the resident loop (cfr_resident.h): team size, cut levels,
// which workgroup owns which decision points, and the order in which its
// payoff rows are streamed.
#include <algorithm>
#include <functional>
#include <limits>
#include <queue>
#include <utility>

#include "cfr.h"
#include "cfr_resident.h"

namespace cfr {

namespace {

constexpr int kMaxCut = 6;
constexpr int64_t kU16 = 65535;

// One barrier over a team (us), measured: 0.8 for 8 and 1.0 for 32
// workgroups of one XCD, 1.6 for 64, 2.0 for 128 and 2.4 for 256 over all.
double barrier_us(int blocks)
{
    return blocks <= 1 ? 0.1 : blocks <= 8 ? 0.8 : blocks <= 32 ? 1.0 : blocks <= 64 ? 1.6
           : blocks <= 128 ? 2.0 : 2.4;
}

// Units (subtrees) dealt to `blocks` workgroups, the heaviest first, each to
// the lightest workgroup so far.  owner[u]: unit u's workgroup.  Returns the
// heaviest workgroup's weight.
double deal(const std::vector<double> &w, int blocks, std::vector<int16_t> &owner)
{
    const int32_t n = (int32_t)w.size();
    owner.assign((size_t)n, 0);
    std::vector<int32_t> order((size_t)n);
    for (int32_t u = 0; u < n; ++u) order[(size_t)u] = u;
    std::stable_sort(order.begin(), order.end(),
                     [&](int32_t a, int32_t b) { return w[(size_t)a] > w[(size_t)b]; });
    using Load = std::pair<double, int>;
    std::priority_queue<Load, std::vector<Load>, std::greater<Load>> load;
    for (int k = 0; k < blocks; ++k) load.push({0.0, k});
    double most = 0;
    for (int32_t u : order) {
        Load l = load.top();
        load.pop();
        owner[(size_t)u] = (int16_t)l.second;
        l.first += w[(size_t)u];
        most = std::max(most, l.first);
        load.push(l);
    }
    return most;
}

struct Shape {
    int blocks, c[2];
    double cost;
};

}  // namespace

bool plan_resident(const ResSource &src, const ResRows rows[2], const int64_t seq_base[2], int prec,
                   int max_blocks, ResidentPlan &plan)
{
    const uint32_t V = (uint32_t)value_bytes(prec), R = (uint32_t)accum_bytes(prec),
                   C = (uint32_t)compute_bytes(prec);
    const bool quads[2] = {plan.team.quads[0] != 0, plan.team.quads[1] != 0};
    int32_t n_seq[2], n_inf[2], n_lev[2];
    std::vector<int32_t> seq_inf[2], inf_par[2];
    std::vector<double> weight[2];  // of the subtree at each decision point (us on one workgroup)
    std::vector<int32_t> below[2];  // sequences of that subtree
    double weight_all[2] = {0, 0};
    for (int p = 0; p < 2; ++p) {
        n_inf[p] = src.n_inf[p];
        n_seq[p] = (int32_t)src.child_ptr[p].size() - 1;
        n_lev[p] = (int32_t)src.lvl_inf[p].size() - 1;
        if (n_inf[p] < 1) return false;
        inf_par[p].resize((size_t)n_inf[p]);
        for (int32_t j = 0; j < n_inf[p]; ++j)
            inf_par[p][(size_t)j] = src.seq_par[p][(size_t)src.inf_first[p][(size_t)j]];
        const std::vector<int32_t> &rp = *rows[p].ptr;
        seq_inf[p].assign((size_t)n_seq[p], -1);
        weight[p].assign((size_t)n_inf[p], 0.0);
        below[p].assign((size_t)n_inf[p], 0);
        // measured: a quad 0.6 ns and an element 0.6 (double) or 0.45 ns of a
        // workgroup's time, a sequence's passes 1.2 ns
        const double el = quads[p] || V == 8 ? 0.6e-3 : 0.45e-3, sq = 1.2e-3;
        for (int32_t j = n_inf[p] - 1; j >= 0; --j) {
            // a group holds whole decision points
            if (src.inf_first[p][(size_t)j + 1] - src.inf_first[p][(size_t)j] > 64) return false;
            for (int32_t a = src.inf_first[p][(size_t)j]; a < src.inf_first[p][(size_t)j + 1]; ++a) {
                const int32_t len = rp[(size_t)a + 1] - rp[(size_t)a];
                if (len > kU16) return false;
                weight[p][(size_t)j] += sq + el * len;
                seq_inf[p][(size_t)a] = j;
            }
        }
        for (int32_t j = n_inf[p] - 1; j >= 0; --j) {
            const int32_t par = inf_par[p][(size_t)j];
            below[p][(size_t)j] += src.inf_first[p][(size_t)j + 1] - src.inf_first[p][(size_t)j];
            if (par > 0) {
                const size_t up = (size_t)seq_inf[p][(size_t)par];
                weight[p][up] += weight[p][(size_t)j];
                below[p][up] += below[p][(size_t)j];
            } else {
                weight_all[p] += weight[p][(size_t)j];
            }
        }
    }

    // candidate shapes, cheapest estimate first: for each team size (largest
    // first; one whose even share alone costs more than the best so far is
    // passed over) each player's cuts whose LDS can fit
    std::vector<Shape> shapes;
    std::vector<int16_t> dealt;
    const double total = weight_all[0] + weight_all[1];
    double best = std::numeric_limits<double>::infinity();
    struct Cut {
        int c;
        double cost, lds;
    };
    static const int kSizes[] = {256, 192, 128, 96, 64, 48, 32, 24, 16, 12, 8, 4, 2, 1};
    for (int blocks : kSizes) {
        if (blocks > std::min(max_blocks, kResCus)) continue;
        if (res_least_blocks((int64_t)n_seq[0] + n_seq[1], prec) > blocks) continue;
        if (total / blocks + 2 * barrier_us(blocks) > best + 2.0) continue;
        const bool lean = blocks > 1;
        const double per_seq = R + 2 * V + 12 + (lean ? 0 : R + V);
        std::vector<Cut> cuts[2];
        for (int p = 0; p < 2; ++p) {
            for (int c = 0; c < std::min(n_lev[p], kMaxCut) && (blocks > 1 || c == 0); ++c) {
                const int32_t lo = src.lvl_inf[p][(size_t)c], hi = src.lvl_inf[p][(size_t)c + 1];
                // the shallow part is in every workgroup's LDS
                const double shallow = per_seq * src.lvl_seq[p][(size_t)c] * (c > 0) + (double)C * hi;
                if (c > 0 && shallow > 0.6 * kResLds) break;
                const std::vector<double> w(weight[p].begin() + lo, weight[p].begin() + hi);
                const double most = deal(w, blocks, dealt);
                std::vector<int32_t> seqs((size_t)blocks, 0);
                for (int32_t u = 0; u < hi - lo; ++u)
                    seqs[(size_t)dealt[(size_t)u]] += below[p][(size_t)(lo + u)];
                const double own = *std::max_element(seqs.begin(), seqs.end());
                // barriers; 0.6 us for each level's chain of LDS accesses;
                // the shallow part's exchange
                const double cost = most + barrier_us(blocks) * (c > 0 ? 2 : 1) +
                                    0.6 * n_lev[p] + (c > 0 ? 0.6 + 3e-4 * hi : 0.0) + 1.0;
                cuts[p].push_back(Cut{c, cost, shallow + own * (per_seq + 0.4 * C)});
            }
        }
        for (const Cut &a : cuts[0])
            for (const Cut &b : cuts[1])
                if (a.lds + b.lds + kResWavesMax * kResStage <= 1.02 * kResLds) {
                    shapes.push_back(Shape{blocks, {a.c, b.c}, a.cost + b.cost});
                    best = std::min(best, a.cost + b.cost);
                }
    }
    std::stable_sort(shapes.begin(), shapes.end(),
                     [](const Shape &a, const Shape &b) { return a.cost < b.cost; });
    if (shapes.size() > 6) shapes.resize(6);

    for (const Shape &s : shapes) {
        plan.blocks = s.blocks;
        plan.cost_us = s.cost;
        plan.part.assign((size_t)s.blocks * 2, ResPart{});
        plan.i32.clear();
        plan.u16.clear();
        plan.chunk.clear();
        plan.row.clear();
        plan.src.clear();
        bool fits = true;
        int32_t longest = 0;
        for (int p = 0; p < 2 && fits; ++p) {
            const int c = s.c[p];
            const std::vector<int32_t> &inf_first = src.inf_first[p], &par = inf_par[p];
            const std::vector<int32_t> &cptr = src.child_ptr[p], &cidx = src.child_idx[p];
            const int32_t lo = src.lvl_inf[p][(size_t)c], hi = src.lvl_inf[p][(size_t)c + 1];
            ResShallow &h = plan.sh[p];
            h = ResShallow{};
            h.c = c;
            // owners: the cut level's decision points with their subtrees
            deal(std::vector<double>(weight[p].begin() + lo, weight[p].begin() + hi), s.blocks, dealt);
            std::vector<int16_t> owner((size_t)n_inf[p], -1);
            std::vector<int32_t> count((size_t)s.blocks + 1, 0);
            for (int32_t j = lo; j < n_inf[p]; ++j) {
                owner[(size_t)j] = j < hi ? dealt[(size_t)(j - lo)]
                                          : owner[(size_t)seq_inf[p][(size_t)par[(size_t)j]]];
                count[(size_t)owner[(size_t)j] + 1]++;
            }
            for (int k = 0; k < s.blocks; ++k) count[(size_t)k + 1] += count[(size_t)k];
            // Numbers a set of decision points level by level from `list`
            // (those of its first level): every level's are the children of
            // the sequences of the one above, in order.
            std::vector<int32_t> list, level_at;
            auto breadth_first = [&](int levels) {
                size_t from = 0;
                level_at.assign(1, 0);
                for (int L = 1; L <= levels; ++L) {
                    const size_t to = list.size();
                    level_at.push_back((int32_t)to);
                    if (L == levels) break;
                    for (size_t i = from; i < to; ++i) {
                        const int32_t j = list[i];
                        for (int32_t e = cptr[(size_t)inf_first[(size_t)j]];
                             e < cptr[(size_t)inf_first[(size_t)j + 1]]; ++e)
                            list.push_back(cidx[(size_t)e]);
                    }
                    from = to;
                }
            };
            std::vector<int32_t> local_q((size_t)n_seq[p], 0), cut_at((size_t)(hi - lo), 0);
            // The arrays of a numbered set (in breadth-first order a set's
            // children follow one another), its first n decision points in
            // `levels` levels.
            auto put = [&](int32_t n, int levels, auto &out) {
                int32_t nq = 1;
                out.ni = n;
                std::vector<int32_t> level_grp, group;
                int32_t i = 0;
                for (int L = 0; L < levels; ++L) {
                    level_grp.push_back((int32_t)group.size());
                    int32_t start = nq;
                    const int32_t end = level_at[(size_t)L + 1];
                    if (i < end) group.push_back(nq);
                    for (; i < end; ++i) {
                        const int32_t j = list[(size_t)i];
                        const int32_t m = inf_first[(size_t)j + 1] - inf_first[(size_t)j];
                        if (nq + m - start > 64) group.push_back(start = nq);
                        for (int32_t a = inf_first[(size_t)j]; a < inf_first[(size_t)j + 1]; ++a)
                            local_q[(size_t)a] = nq++;
                    }
                }
                level_grp.push_back((int32_t)group.size());
                group.push_back(nq);
                out.nq = nq;
                out.lev = (int32_t)plan.i32.size();
                plan.i32.insert(plan.i32.end(), level_grp.begin(), level_grp.end());
                out.grp = (int32_t)plan.i32.size();
                plan.i32.insert(plan.i32.end(), group.begin(), group.end());
                out.gs = (int32_t)plan.i32.size();
                plan.i32.push_back((int32_t)seq_base[p]);
                const int32_t first_kids = level_at[1];
                int32_t kids = first_kids;
                const size_t at = plan.u16.size(), sq = (size_t)nq;
                out.kn = (int32_t)at;
                out.in = (int32_t)(at + sq);
                out.cp = (int32_t)(at + 2 * sq);
                out.pq = (int32_t)(at + 3 * sq + 1);
                plan.u16.resize(at + 4 * sq + 1, 0);
                uint16_t *kn = &plan.u16[at], *in = kn + sq, *cp = in + sq, *pq = cp + sq + 1;
                kn[0] = 1 << 8;
                cp[0] = (uint16_t)first_kids;
                int32_t q = 1;
                for (i = 0; i < n; ++i) {
                    const int32_t j = list[(size_t)i];
                    const int32_t f = inf_first[(size_t)j], m = inf_first[(size_t)j + 1] - f;
                    for (int32_t k = 0; k < m; ++k, ++q) {
                        plan.i32.push_back((int32_t)seq_base[p] + f + k);
                        kn[q] = (uint16_t)(k | m << 8);
                        in[q] = (uint16_t)i;
                        cp[q] = (uint16_t)kids;
                        kids += cptr[(size_t)(f + k) + 1] - cptr[(size_t)(f + k)];
                        pq[q] = (uint16_t)local_q[(size_t)par[(size_t)j]];
                    }
                }
                cp[nq] = (uint16_t)kids;
            };
            if (c > 0) {
                if (src.lvl_seq[p][(size_t)c] > kU16 || hi > kU16) {
                    fits = false;
                    break;
                }
                list.clear();
                for (int32_t j = 0; j < src.lvl_inf[p][1]; ++j) list.push_back(j);
                breadth_first(c + 1);
                // the cut level's come last
                for (int32_t u = 0; u < hi - lo; ++u)
                    cut_at[(size_t)(list[(size_t)(lo + u)] - lo)] = u;
                h.ncut = hi - lo;
                put(lo, c, h);
            }
            // shallow rows with payoffs, dealt round over the workgroups
            std::vector<int32_t> shallow_rows;
            const std::vector<int32_t> &rp = *rows[p].ptr;
            for (int32_t a = 1; c > 0 && a < src.lvl_seq[p][(size_t)c]; ++a)
                if (rp[(size_t)a + 1] > rp[(size_t)a]) shallow_rows.push_back(a);
            plan.chunk0[p] = (int32_t)plan.chunk.size();
            plan.elements[p] = 0;
            struct Row {
                int32_t dest, src, len, lr;
            };
            std::vector<Row> order;
            for (int k = 0; k < s.blocks && fits; ++k) {
                ResPart &q = plan.part[(size_t)k * 2 + (size_t)p];
                const int32_t b0 = count[(size_t)k], b1 = count[(size_t)k + 1];
                q.nlev = n_lev[p] - c;
                list.clear();
                q.cut = (int32_t)plan.i32.size();
                for (int32_t u = 0; u < hi - lo; ++u)
                    if (dealt[(size_t)u] == k) list.push_back(lo + u);
                // the cut level in the shallow part's order
                if (c > 0)
                    std::sort(list.begin(), list.end(), [&](int32_t i, int32_t j) {
                        return cut_at[(size_t)(i - lo)] < cut_at[(size_t)(j - lo)];
                    });
                for (int32_t j : list) plan.i32.push_back(c > 0 ? cut_at[(size_t)(j - lo)] : j);
                breadth_first(q.nlev);
                if ((int32_t)list.size() != b1 - b0 || list.size() > (size_t)kU16) {
                    fits = false;
                    break;
                }
                int64_t own = 1;
                for (int32_t j : list) own += inf_first[(size_t)j + 1] - inf_first[(size_t)j];
                if (own + h.nq > kU16) {
                    fits = false;
                    break;
                }
                put(b1 - b0, q.nlev, q);
                q.first_q = 1;
                for (int32_t i = 0; i < level_at[1]; ++i)
                    q.first_q += inf_first[(size_t)list[(size_t)i] + 1] - inf_first[(size_t)list[(size_t)i]];
                const int32_t nq = q.nq;
                // the share's rows, in its own order (neighbouring rows gather
                // neighbouring entries), by lanes a row
                order.clear();
                int64_t total = 0;
                auto add = [&](int32_t a, int32_t dest) {
                    const int32_t len = rp[(size_t)a + 1] - rp[(size_t)a];
                    if (len <= 0) return;
                    order.push_back(Row{dest, rp[(size_t)a], len, rows[p].lr[(size_t)a]});
                    total += len;
                    longest = std::max(longest, len);
                };
                for (int32_t j : list)
                    for (int32_t a = inf_first[(size_t)j]; a < inf_first[(size_t)j + 1]; ++a)
                        add(a, local_q[(size_t)a]);
                for (size_t i = (size_t)k; i < shallow_rows.size(); i += (size_t)s.blocks)
                    add(shallow_rows[i], nq + local_q[(size_t)shallow_rows[i]]);
                std::stable_sort(order.begin(), order.end(),
                                 [](const Row &a, const Row &b) { return a.lr < b.lr; });
                // chunks of equal size, as many as fill the waves evenly
                const int64_t cap = res_chunk((int)V, quads[p]);
                const int64_t turns = (total + kResWavesMax * cap - 1) / (kResWavesMax * cap);
                const int64_t even = turns ? total / (kResWavesMax * turns) + 1 + longest / 2 : cap;
                const int64_t aim = std::max<int64_t>(64, std::min<int64_t>(cap, even));
                q.c0 = (int32_t)plan.chunk.size();
                for (size_t i = 0; i < order.size();) {
                    ResChunk ch{(int32_t)plan.elements[p], 0, 0, (int32_t)plan.row.size()};
                    size_t e = i;
                    while (e < order.size() && order[e].lr == order[i].lr &&
                           (e == i || ch.n + order[e].len <= aim)) {
                        plan.row.push_back((uint32_t)order[e].dest | (uint32_t)ch.n << 16);
                        plan.src.push_back(order[e].src);
                        ch.n += order[e].len;
                        ++e;
                    }
                    plan.row.push_back((uint32_t)ch.n << 16);
                    plan.src.push_back(0);
                    ch.rows_lr = (int32_t)(e - i) | order[i].lr << 16;
                    plan.chunk.push_back(ch);
                    plan.elements[p] += ch.n;
                    i = e;
                }
                q.nc = (int32_t)plan.chunk.size() - q.c0;
            }
            plan.n_chunk[p] = (int32_t)plan.chunk.size() - plan.chunk0[p];
            plan.local[p].clear();
            if (s.blocks == 1) plan.local[p] = local_q;
            if (plan.elements[p] > std::numeric_limits<int32_t>::max() - 4096) fits = false;
        }
        if (!fits) continue;
        // averages and own strategies in LDS too when that fits; a workgroup
        // alone gathers its strategies from there
        for (int lean = 0; lean < (s.blocks > 1 ? 2 : 1); ++lean) {
            ResOff o0, o1;
            plan.lds = 0;
            plan.team.lean = lean;
            for (int k = 0; k < s.blocks; ++k)
                plan.lds = std::max(plan.lds, res_layout(plan.sh, &plan.part[(size_t)k * 2], V, R, C,
                                                         lean, o0, o1));
            if (plan.lds + kResWavesMax * kResStage <= kResLds) return true;
        }
    }
    return false;
}

}  // namespace cfr
