// Grouped form of a recorded program (Program::group): dependency levels, separate arrays ("slabs")
// for contributions to one tensor, tile and split choice, and the work-item tables of the launches.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <unordered_set>

#include "elem.hpp"
#include "plan.hpp"

namespace lrcc {

namespace {

// One array holding a part of a tensor's value: the sum of a tensor's slabs (and of the slabs it takes
// over from copied or added tensors) is its value.
struct Slab {
    int tensor;
    int last = -1;                       // level of its last writer
    bool all = false;                    // a writer stores every element
    std::unordered_set<i64> cover;       // blocks (by offset) a writer stores completely
    std::unordered_set<i64> touched;     // blocks written by anybody
    std::vector<int> extra;              // further slabs of split products written at the same level
    void *p = nullptr;
};

struct Tensor {
    void *p;
    i64 count = 0;
    std::vector<int> own;                // slabs written for this tensor
    std::vector<int> parts;              // own slabs and slabs taken over, in order
    bool read = false;                   // no contribution may follow
    bool fixed = false;                  // written in its own buffer only
    bool real = false;                   // of real numbers: never summed or taken over
};

struct Prod {
    size_t node;
    int level, slab, beta;
    int tile = 0, ksplit = 1;
    int steps = 0;                       // largest number of reduction steps of a job
    i64 tiles = 0;
    bool full = false;
    bool alone = false;                  // fills the device by itself: a launch of its own
    std::vector<int> extra;              // slabs of its further splits
};

struct Other {
    size_t node;
    int level, slab = -1;
    bool acc = false, clear = false;     // clear: zero the slab (no op of its own)
};

i64 block_elems(const GemmArgs &g) {     // one past the largest offset inside an output block
    auto mx = [](int total, const Split &sp, const Strides &st) {
        const int e0 = total / (sp.d1 * sp.d2);
        const int m1 = sp.tri ? sp.tri - 2 : sp.d1 - 1, m2 = sp.tri ? sp.tri - 1 : sp.d2 - 1;
        return (i64)(e0 - 1) * st.s[0] + (i64)m1 * st.s[1] + (i64)m2 * st.s[2];
    };
    return mx(g.M, g.sm, g.Cm) + mx(g.N, g.sn, g.Cn) + 1;
}

i64 cdiv(i64 a, i64 b) { return (a + b - 1) / b; }

// Most slabs of a tensor: contributions that find no free slab wait for an earlier one instead.  Small
// tensors cost little to sum and every level costs a launch; a large one pays a write and a read of the
// whole array per slab, and its products fill the device one after another.  Measured per application:
// three-k chain, 33 MB doubles (complex128, 12 right-hand sides): 6 slabs 0.87 ms, 4 0.92 ms, 12 0.91 ms;
// Nk=5, o=8, v=40 transposed, 205 MB: 1 slab 19.4 ms, 2 20.3 ms, 3 20.5 ms.
int max_slabs(i64 bytes) {
    return bytes <= (1 << 20) ? 12 : bytes <= (16 << 20) ? 8 : bytes <= (64 << 20) ? 6 : 1;
}

// A product of this many 64x64 tiles (8 per compute unit) fills the device by itself and runs through its
// own launch, whose kernel has the larger tiles: wide transposed complex64 batch (Nk=3, o=10, v=60, 6
// right-hand sides) 35.4 ms at 2048, 34.9 at 4096; Nk=5 transposed complex128 vector 18.5 against 20.5 ms.
constexpr i64 kAloneTiles = 2048;

}  // namespace

template <typename T>
bool Program::group(size_t budget, bool keep) {
    const size_t had = owned.size();
    bool ok = false;
    try {
        ok = make_grouped<T>(budget, keep);
    } catch (const LrccError &e) {
        if (e.code != 4) throw;          // no room for the extra arrays: the program runs op by op
    }
    if (ok) {
        if (std::getenv("LRCC_PLAN_DUMP")) {
            std::fprintf(stderr, "grouped: %zu ops in %zu launches\n", ops.size(), grouped.size());
            for (const Launch &l : grouped) std::fprintf(stderr, "  %s\n", l.name.c_str());
        }
        return true;
    }
    grouped.clear();
    while (owned.size() > had) {
        dev_free(owned.back());
        owned.pop_back();
    }
    return false;
}

template <typename T>
bool Program::make_grouped(size_t budget, bool keep) {
    grouped.clear();
    group_tiles.clear();
    if (nodes.size() != ops.size()) return false;
    for (size_t i = 0; i < nodes.size(); ++i)
        if (nodes[i].op != i) return false;
    constexpr i64 esz = 2 * sizeof(T);
    std::map<const void *, int> ids;
    std::vector<Tensor> tens;
    std::vector<Slab> slabs;
    std::vector<Prod> prods;
    std::vector<Other> others, outs;
    std::unordered_set<const void *> constants;      // read, and not written by an earlier op
    auto last_of = [&](const Tensor &t) {
        int l = -1;
        for (int s : t.parts) l = std::max(l, slabs[s].last);
        return l;
    };
    auto new_slab = [&](int t) {
        Slab s;
        s.tensor = t;
        slabs.push_back(std::move(s));
        return (int)slabs.size() - 1;
    };
    // ---- levels and slabs, in program order
    for (size_t i = 0; i < nodes.size(); ++i) {
        const Node &nd = nodes[i];
        int lvl = 0;
        for (const void *r : nd.reads) {
            auto it = ids.find(r);
            if (it == ids.end()) {
                constants.insert(r);
                continue;
            }
            lvl = std::max(lvl, last_of(tens[it->second]) + 1);
            tens[it->second].read = true;
        }
        if (nd.kind == Node::OUT) {
            outs.push_back({i, lvl});
            continue;
        }
        for (const auto &x : nd.also) {      // stored by this op alone, in place
            if (constants.count(x.first) || !ids.emplace(x.first, (int)tens.size()).second) return false;
            Tensor xt;
            xt.p = x.first;
            xt.count = x.second;
            xt.fixed = true;
            Slab xs;
            xs.tensor = (int)tens.size();
            xs.last = lvl;
            xs.all = true;
            slabs.push_back(std::move(xs));
            xt.own.push_back((int)slabs.size() - 1);
            xt.parts = xt.own;
            tens.push_back(std::move(xt));
        }
        if (g_dry_run && (size_t)nd.count * (nd.real ? esz / 2 : esz) > dry_bytes(nd.write))
            throw LrccError(1, "a tensor of a grouped program is larger than its array");
        if (constants.count(nd.write)) return false;      // read before it is written
        auto ins = ids.emplace(nd.write, (int)tens.size());
        if (ins.second) {
            tens.push_back(Tensor{});
            tens.back().p = nd.write;
            tens.back().count = nd.count;
        }
        const int ti = ins.first->second;
        Tensor &t = tens[ti];
        const bool fresh = ins.second;
        if (t.count != nd.count || t.read || t.fixed) return false;
        if (!nd.also.empty() || nd.real) t.fixed = true;
        t.real = nd.real;
        if (nd.real && (nd.kind != Node::WRITE || nd.acc)) return false;
        if (nd.kind == Node::ZERO) {
            if (!t.parts.empty()) return false;
            continue;
        }
        if (!nd.acc && nd.kind != Node::ADD && !t.parts.empty()) return false;   // written twice
        if ((nd.acc || nd.kind == Node::ADD) && fresh) return false;             // adds to unknown contents
        if (nd.kind == Node::COPY || nd.kind == Node::ADD) {
            auto src = ids.find(nd.reads.at(0));
            if (src == ids.end()) {          // an array no op writes: one slab that is always there
                src = ids.emplace(nd.reads.at(0), (int)tens.size()).first;
                Slab xs;
                xs.tensor = (int)tens.size();
                xs.all = true;
                xs.p = const_cast<void *>(nd.reads.at(0));
                slabs.push_back(std::move(xs));
                Tensor xt;
                xt.p = const_cast<void *>(nd.reads.at(0));
                xt.count = nd.count;
                xt.read = xt.fixed = true;
                xt.own = xt.parts = {(int)slabs.size() - 1};
                tens.push_back(std::move(xt));
            }
            Tensor &t = tens[ti];            // (tens may have moved)
            const std::vector<int> &sp = tens[src->second].parts;
            if (sp.empty() || tens[src->second].count != t.count || tens[src->second].real) return false;
            t.parts.insert(t.parts.end(), sp.begin(), sp.end());
            continue;
        }
        const GemmOp *go = nullptr;
        if (nd.kind == Node::GEMM) {
            auto it = gemm_ops.find(i);
            if (it == gemm_ops.end() || it->second.sizeC != nd.count) return false;
            go = &it->second;
        }
        const bool bfull = go && !go->args->sm.tri && !go->args->sn.tri &&
                           (i64)go->args->M * go->args->N == block_elems(*go->args);
        // free slab: one whose written blocks hold these (added to later than its last writer) or
        // none of these (stored beside them)
        int pick = -1, beta = 0, best = -1;
        for (int s : t.own) {
            const Slab &sl = slabs[s];
            bool in = true, out = go != nullptr && !sl.all;
            if (go) {
                for (i64 o : go->offC) {
                    in = in && (sl.all || sl.cover.count(o));
                    out = out && !sl.touched.count(o);
                }
            } else
                in = sl.all;
            if (out) { pick = s; beta = 0; break; }
            if (in && sl.last < lvl) { pick = s; beta = 1; break; }
            if (in && (best < 0 || sl.last < slabs[best].last)) best = s;
        }
        if (pick < 0 && best >= 0 && (int)t.own.size() >= max_slabs(t.count * esz)) {
            pick = best;
            beta = 1;
            lvl = slabs[best].last + 1;
        }
        if (pick < 0) {
            pick = new_slab(ti);
            t.own.push_back(pick);
            t.parts.push_back(pick);
            if (go && !nd.full && nd.acc && max_slabs(t.count * esz) == 1) {
                // a large tensor whose contributions store parts of it: cleared once, then added to
                others.push_back({i, 0, pick, false, true});
                slabs[pick].all = true;
                lvl = std::max(lvl, 1);
                beta = 1;
            }
        }
        Slab &sl = slabs[pick];
        sl.last = std::max(sl.last, lvl);
        if (go) {
            for (i64 o : go->offC) {
                sl.touched.insert(o);
                if (bfull && !beta) sl.cover.insert(o);
            }
            if (nd.full && !beta) sl.all = true;
            Prod p;
            p.node = i;
            p.level = lvl;
            p.slab = pick;
            p.beta = beta;
            p.full = nd.full;
            prods.push_back(p);
        } else {
            if (!beta) sl.all = true;
            others.push_back({i, lvl, pick, beta != 0});
        }
    }
    // a tensor that others read and that nothing is added to: cleared in every run
    for (size_t t = 0; keep && t < tens.size(); ++t) {
        if (!tens[t].parts.empty()) continue;
        const int s = new_slab((int)t);
        slabs[s].all = true;
        slabs[s].last = 0;
        tens[t].own = tens[t].parts = {s};
        others.push_back({0, 0, s, false, true});
    }
    int nlev = 0;
    for (const Prod &p : prods) nlev = std::max(nlev, p.level + 1);
    for (const Other &p : others) nlev = std::max(nlev, p.level + 1);
    for (const Other &p : outs) nlev = std::max(nlev, p.level + 1);
    // ---- tiles and splits, level by level
    auto launch_of = [&](const Prod &p) {
        return std::make_pair(p.node < tags.size() ? tags[p.node] : (int)TAG_NONE, tile_class(p.tile));
    };
    std::vector<std::vector<int>> at(nlev);
    for (size_t q = 0; q < prods.size(); ++q) at[prods[q].level].push_back((int)q);
    size_t extra_bytes = 0;
    for (int l = 0; l < nlev; ++l) {
        // work per wave (GroupTile::frags) of each launch: (tag, launch class of the tile)
        std::map<std::pair<int, int>, double> units;
        for (int q : at[l]) {
            Prod &p = prods[q];
            const GemmOp &go = gemm_ops.at(p.node);
            const GemmArgs &g = *go.args;
            const i64 nj = (i64)go.offC.size();
            p.tile = best_tile(g.M, g.N, g.K, nj, sizeof(T) == 8, true);
            const i64 ks = cdiv(std::max(g.K, 1), kGroupTiles[p.tile].k);
            for (i64 j = 0; j < nj; ++j)
                p.steps = std::max<int>(p.steps, (int)std::min<i64>((go.segBeg[j + 1] - go.segBeg[j]) * ks, INT32_MAX));
            p.tiles = nj * cdiv(g.M, kGroupTiles[p.tile].m) * cdiv(g.N, kGroupTiles[p.tile].n);
            if (p.tiles * kGroupTiles[p.tile].m * kGroupTiles[p.tile].n >= kAloneTiles * 64 * 64 && tile_class(p.tile) > 0) {
                p.alone = true;
                continue;
            }
            group_tiles[p.node] = p.tile;
            units[launch_of(p)] += (double)p.tiles * kGroupTiles[p.tile].frags * p.steps;
        }
        // a workgroup runs at most about half of its launch's average work per compute unit in one
        // piece, and not less than 6 steps (a step of a small tile is shorter than starting one).  Pieces longer
        // than 48 steps are cut to a quarter of that, down to 48: with one or two pieces per compute unit the
        // last ones run alone (a level of Nk=3, o=10, v=60, transposed: 678 pieces 1.59 ms, 1725 1.13; of Nk=5,
        // o=8, v=40, complex128: 3.33 against 2.84).  Cut everywhere, Nk=3, o=4, v=20 takes 650 us against 583.
        for (int q : at[l]) {
            Prod &p = prods[q];
            if (p.alone) continue;
            const double all = units[launch_of(p)];
            const double most = std::max(6.0, std::min(all / 512, std::max(48.0, all / 2048)));
            const double mine = (double)p.steps * kGroupTiles[p.tile].frags;
            i64 ks = (i64)std::ceil(mine / most);
            const i64 bytes = tens[slabs[p.slab].tensor].count * esz;
            ks = std::min<i64>({ks, 256, std::max<i64>(1, p.steps / 2), 1 + ((i64)4 << 20) / std::max<i64>(bytes, 1)});
            p.ksplit = (int)std::max<i64>(1, ks);
            for (int s = 1; s < p.ksplit; ++s) {
                const int e = new_slab(slabs[p.slab].tensor);
                slabs[e].last = l;
                slabs[e].all = p.full;
                slabs[p.slab].extra.push_back(e);
                p.extra.push_back(e);
            }
        }
    }
    // ---- storage.  A tensor read as an operand needs its slabs summed into its buffer unless it is one
    // slab; the output steps read the slabs themselves.  The first slab lives in the tensor's buffer where its
    // writer stores every element again in each run and no sum goes there that another tensor does not count;
    // or, stored in part, where it is the tensor's only slab.  A run of the program op by op leaves the
    // tensor's whole value in that buffer: beside other slabs, elements that no writer of this one stores
    // would be counted twice by the next grouped run
    std::vector<std::vector<int>> parts(tens.size());
    for (size_t t = 0; t < tens.size(); ++t)
        for (int s : tens[t].parts) {
            parts[t].push_back(s);
            parts[t].insert(parts[t].end(), slabs[s].extra.begin(), slabs[s].extra.end());
        }
    std::vector<char> need_sum(tens.size(), 0), exposed(tens.size(), 0);
    auto single = [&](size_t t) { return parts[t].size() == 1 && slabs[parts[t][0]].tensor == (int)t; };
    for (size_t i = 0; i < nodes.size(); ++i) {
        if (nodes[i].kind == Node::COPY || nodes[i].kind == Node::ADD) continue;   // take slabs over
        for (const void *r : nodes[i].reads) {
            auto it = ids.find(r);
            if (it == ids.end()) continue;
            const int t = it->second;
            if (parts[t].empty()) return false;                                    // read before written
            if (nodes[i].kind != Node::OUT && !single(t)) need_sum[t] = 1;
        }
    }
    if (keep)
        for (size_t t = 0; t < tens.size(); ++t)
            if (!parts[t].empty() && !single(t)) need_sum[t] = 1;
    // what an output step reads: own slabs, and of tensors taken over their sum where there is one
    auto out_list = [&](int t) {
        std::vector<int> v;                 // slab, or -1 - tensor
        for (int s : parts[t]) {
            const int from = slabs[s].tensor;
            const int e = from != t && need_sum[from] ? -1 - from : s;
            if (std::find(v.begin(), v.end(), e) == v.end()) v.push_back(e);
        }
        return v;
    };
    for (const Other &o : outs) {
        for (const void *r : nodes[o.node].reads) {
            const int t = ids.at(r);
            if (!need_sum[t] && out_list(t).size() > (size_t)kMaxSlabs) need_sum[t] = 1;
        }
    }
    // a sum follows the level of its last writer: one of arrays that no op writes has none
    for (size_t t = 0; t < tens.size(); ++t)
        if (need_sum[t] && last_of(tens[t]) < 0) return false;
    for (size_t t = 0; t < tens.size(); ++t)
        if (need_sum[t])
            for (int s : parts[t])
                if (slabs[s].tensor != (int)t) exposed[slabs[s].tensor] = 1;
    for (size_t t = 0; t < tens.size(); ++t) {
        if (tens[t].own.empty()) continue;
        Slab &s0 = slabs[tens[t].own[0]];
        if (s0.all ? !need_sum[t] || !exposed[t] : !need_sum[t] && parts[t].size() == 1) s0.p = tens[t].p;
    }
    for (Slab &s : slabs)
        if (!s.p) extra_bytes += (size_t)(tens[s.tensor].count * esz);
    if (std::getenv("LRCC_PLAN_DUMP"))
        std::fprintf(stderr, "grouped form: %.1f MB of extra arrays, at most %.1f\n", extra_bytes / 1048576.0, budget / 1048576.0);
    if (extra_bytes > budget) return false;
    std::vector<std::pair<void *, i64>> clear;      // elements no writer stores stay zero from here on
    for (Slab &s : slabs) {
        const Tensor &t = tens[s.tensor];
        if (!s.p) s.p = alloc((size_t)(t.count * esz));
        if (!s.all) clear.push_back({s.p, t.count});
    }
    // ---- launch tables
    std::vector<GemmArgs> args;
    std::vector<GroupItem> items;
    std::vector<SumSeg> segs;
    std::vector<const void *> srcs;
    std::vector<int2> work;
    struct Range { int level, kind, cls, tag, begin, end; };   // kind 0: products, 1: sums
    std::vector<Range> ranges;
    std::map<size_t, int> argidx;
    for (const Prod &p : prods) {
        argidx[p.node] = (int)args.size();
        args.push_back(*gemm_ops.at(p.node).args);
    }
    std::vector<char> summed(tens.size(), 0);
    for (int l = 0; l < nlev; ++l) {
        std::map<std::pair<int, int>, std::vector<int>> by;
        for (int q : at[l])
            if (!prods[q].alone) by[launch_of(prods[q])].push_back(q);
        for (auto &kv : by) {
            const int begin = (int)items.size();
            // longest pieces first
            std::stable_sort(kv.second.begin(), kv.second.end(), [&](int a, int b) {
                return prods[a].steps / prods[a].ksplit > prods[b].steps / prods[b].ksplit;
            });
            for (int q : kv.second) {
                const Prod &p = prods[q];
                const GemmOp &go = gemm_ops.at(p.node);
                const GemmArgs &g = *go.args;
                const int tm = kGroupTiles[p.tile].m, tn = kGroupTiles[p.tile].n;
                const i64 ks = cdiv(std::max(g.K, 1), kGroupTiles[p.tile].k);
                for (size_t j = 0; j < go.offC.size(); ++j) {
                    const i64 nst = (i64)(go.segBeg[j + 1] - go.segBeg[j]) * (g.K > 0 ? ks : 0);
                    if (nst > INT32_MAX) return false;
                    for (int s = 0; s < p.ksplit; ++s)
                        for (int n0 = 0; n0 < g.N; n0 += tn)
                            for (int m0 = 0; m0 < g.M; m0 += tm) {
                                if (tile_skipped(g, (int)j, m0, n0, tm, tn)) continue;
                                GroupItem it{};
                                char *c = (char *)slabs[s == 0 ? p.slab : p.extra[s - 1]].p;
                                it.C = c + go.offC[j] * esz;
                                it.tile = p.tile;
                                it.op = argidx.at(p.node);
                                it.m0 = m0;
                                it.n0 = n0;
                                it.sb = go.segBeg[j];
                                it.t0 = (int)(nst * s / p.ksplit);
                                it.t1 = (int)(nst * (s + 1) / p.ksplit);
                                it.js = go.jscale.empty() ? 1.0f : go.jscale[j];
                                it.beta = s == 0 ? p.beta : 0;
                                items.push_back(it);
                            }
                }
            }
            if (items.size() > (1u << 21)) return false;
            ranges.push_back({l, 0, kv.first.second, kv.first.first, begin, (int)items.size()});
        }
        const int wb = (int)work.size();
        for (size_t t = 0; t < tens.size(); ++t) {
            if (!need_sum[t] || summed[t] || last_of(tens[t]) != l) continue;
            summed[t] = 1;
            SumSeg g{tens[t].p, tens[t].count, (int)srcs.size(), (int)parts[t].size()};
            for (int s : parts[t]) srcs.push_back(slabs[s].p);
            for (i64 ch = 0; ch * kSumChunk < g.n; ++ch) work.push_back(make_int2((int)segs.size(), (int)ch));
            segs.push_back(g);
        }
        if ((int)work.size() > wb) ranges.push_back({l, 1, 0, TAG_NONE, wb, (int)work.size()});
    }
    auto put = [&](const void *src, size_t bytes) {
        void *d = alloc(std::max<size_t>(bytes, 16));
        if (!g_dry_run && bytes && hipMemcpy(d, src, bytes, hipMemcpyHostToDevice) != hipSuccess)
            throw LrccError(5, "upload of launch tables failed");
        return d;
    };
    const GemmArgs *dargs = (const GemmArgs *)put(args.data(), args.size() * sizeof(GemmArgs));
    const GroupItem *ditems = (const GroupItem *)put(items.data(), items.size() * sizeof(GroupItem));
    const SumSeg *dsegs = (const SumSeg *)put(segs.data(), segs.size() * sizeof(SumSeg));
    const void *const *dsrc = (const void *const *)put(srcs.data(), srcs.size() * sizeof(void *));
    const int2 *dwork = (const int2 *)put(work.data(), work.size() * sizeof(int2));
    if (!g_dry_run) {
        for (auto &c : clear)
            if (zero_fill<T>(c.first, c.second, nullptr) != hipSuccess) throw LrccError(5, "clearing of slabs failed");
        if (hipStreamSynchronize(nullptr) != hipSuccess) throw LrccError(5, "clearing of slabs failed");
    }
    // ---- launches
    for (int l = 0; l < nlev; ++l) {
        for (const Other &o : others) {
            if (o.level != l) continue;
            void *dst = slabs[o.slab].p;
            if (o.clear) {
                const i64 n = tens[slabs[o.slab].tensor].count;
                grouped.push_back({[dst, n](hipStream_t s) { return zero_fill<T>(dst, n, s); }, TAG_NONE, "clear"});
                continue;
            }
            const auto fn = nodes[o.node].write_to;
            if (!fn) return false;
            const bool acc = o.acc;
            grouped.push_back({[fn, dst, acc](hipStream_t s) { return fn(s, dst, acc); }, TAG_NONE, "elementwise"});
        }
        for (int q : at[l]) {
            const Prod &p = prods[q];
            if (!p.alone) continue;
            const std::shared_ptr<GemmArgs> gp = gemm_ops.at(p.node).args;   // keeps its tuned tile
            void *dst = slabs[p.slab].p;
            const int beta = p.beta;
            grouped.push_back({[gp, dst, beta](hipStream_t s) {
                                   GemmArgs g = *gp;
                                   g.C = dst;
                                   g.beta = beta;
                                   return launch_gemm<T>(g, s);
                               },
                               launch_of(p).first, p.node < names.size() ? names[p.node] : std::string()});
        }
        for (const Range &r : ranges) {
            if (r.level != l) continue;
            if (r.kind == 0) {
                const GroupItem *it = ditems + r.begin;
                const int n = r.end - r.begin, cls = r.cls;
                grouped.push_back({[=](hipStream_t s) { return launch_gemm_group<T>(cls, dargs, it, n, s); }, r.tag,
                                   "level " + std::to_string(l) + " products, " + std::to_string(n) +
                                       (cls == 2 ? " bf16 tiles" : cls ? " large tiles" : " small tiles")});
            } else {
                const int2 *w = dwork + r.begin;
                const int n = r.end - r.begin;
                grouped.push_back({[=](hipStream_t s) { return launch_sums<T>(dsegs, dsrc, w, n, s); }, TAG_NONE,
                                   "level " + std::to_string(l) + " sums"});
            }
        }
        for (const Other &o : outs) {
            if (o.level != l) continue;
            const Node &nd = nodes[o.node];
            std::vector<SlabList> sl;
            for (const void *r : nd.reads) {
                const int t = ids.at(r);
                SlabList one{};
                if (need_sum[t]) one = one_slab(tens[t].p);
                else
                    for (int e : out_list(t)) one.p[one.n++] = e < 0 ? tens[-1 - e].p : slabs[e].p;
                sl.push_back(one);
            }
            const auto fn = nd.from;
            if (!fn) return false;
            grouped.push_back({[fn, sl](hipStream_t s) { return fn(s, sl); }, TAG_NONE, "output"});
        }
    }
    return true;
}

template bool Program::group<double>(size_t, bool);
template bool Program::group<float>(size_t, bool);

}  // namespace lrcc
