// Greedy fusion planner for the brickwork circuit (the gate fusion of Sec. II
// and the local-qubit remapping that the paper does with axis swaps, done here
// by choosing which high bits a tile spans).
//
// Dependencies.  Write a = 0 for bonds of the layer applied first in each
// period and a = 1 for the other layer (forward: first layer = odd b, Eq. (4);
// U_F^dagger: first layer = even b).  The k-th application of bond b sits in
// global layer 2k + a_b.  It may run once every neighbouring bond q = b +- 1
// (which touches one of its sites) has completed all of its applications in
// earlier layers, i.e. cnt[q] >= k + a_b, and no application of q in a later
// layer has run (guaranteed by q's own rule).  Ready bonds are never
// neighbours, so a whole round of ready bonds can be applied in any order.
//
// A pass picks the high window h whose tile bit set admits the most ready
// gates (repeating rounds inside the tile, which time-blocks several periods
// into one sweep), then packs the pass's gate list into register groups.
#include "planner.h"

#include <algorithm>
#include <cstring>

namespace fl {

fl_geom make_geom(int L, int kmax, int r, int lowbits) {
    fl_geom g;
    g.L = L;
    if (L <= kmax) {
        g.C = L;
        g.W = 0;
    } else {
        g.C = lowbits;
        g.W = kmax - lowbits;
    }
    g.K = g.C + g.W;
    g.R = std::min(r, g.K);
    return g;
}

namespace {

struct Gate {
    int bond;
    int u;     // tile-local bit (gate on u, u+1)
    int gidx;
    int slot;
};

// Progress of every bond.  In terms of the layer t_b = 2 cnt_b + a_b of a
// bond's next application the rule above reads: b may run when t_b is below
// both neighbours' layers, so neighbours' layers always differ by one and a
// run raises a local minimum of the profile by two.
struct Sched {
    int L, nb, n;
    std::vector<int> cnt, off;
    bool ready(int b) const {
        if (cnt[b] >= n) return false;
        const int need = cnt[b] + off[b];
        if (b > 0 && cnt[b - 1] < need) return false;
        if (b + 1 < nb && cnt[b + 1] < need) return false;
        return true;
    }
};

bool bond_in_tile(const fl_geom& g, int h, int b) {
    const int p = g.L - 2 - b;
    const int u = fl_local_bit(p, g.C, g.W, h);
    const int u1 = fl_local_bit(p + 1, g.C, g.W, h);
    return u >= 0 && u1 == u + 1;
}

// The bonds inside a tile of window h, as runs of consecutive bonds (the low
// bits' and the window's; one run where the window follows the low bits).
struct Window {
    int h = 0, nruns = 0;
    int lo[2] = {0, 0}, hi[2] = {-1, -1};
};

Window tile_window(const fl_geom& g, int h) {
    Window w;
    w.h = h;
    for (int b = 0; b < g.L - 1; ++b) {
        if (!bond_in_tile(g, h, b)) continue;
        if (w.nruns > 0 && w.hi[w.nruns - 1] == b - 1) {
            w.hi[w.nruns - 1] = b;
        } else {
            w.lo[w.nruns] = w.hi[w.nruns] = b;
            ++w.nruns;
        }
    }
    return w;
}

// Apply rounds of ready gates inside tile window w; returns the bonds in order.
std::vector<int> run_tile(const Window& w, Sched& s, int cap) {
    std::vector<int> out;
    int round[64];
    while ((int)out.size() < cap) {
        int nr = 0;
        for (int r = 0; r < w.nruns; ++r)
            for (int b = w.lo[r]; b <= w.hi[r]; ++b)
                if (s.ready(b)) round[nr++] = b;
        if (nr == 0) break;
        for (int k = 0; k < nr && (int)out.size() < cap; ++k) {
            s.cnt[round[k]]++;
            out.push_back(round[k]);
        }
    }
    return out;
}

// The layer profile of a schedule (t[b + 1] = t_b; the ends past the chain
// never hold a bond back) and its last layer n per bond.
struct Profile {
    int nb = 0;
    int t[66], last[66];
    explicit Profile(const Sched& s) : nb(s.nb) {
        t[0] = t[nb + 1] = 1 << 28;
        for (int b = 0; b < nb; ++b) {
            t[b + 1] = 2 * s.cnt[b] + s.off[b];
            last[b + 1] = 2 * s.n + s.off[b];
        }
    }
    // Where a tile's rounds end when none is cut short: every bond of a run goes
    // as far as the fixed layers beside the run allow (they bound it by their own
    // layer plus the distance) and no further than the circuit's end.
    // Writes the new layers to out[1 ..] of the runs and returns the gate count.
    int advance(const Window& w, int* out) const {
        int gates = 0;
        for (int r = 0; r < w.nruns; ++r) {
            const int l = w.lo[r], h = w.hi[r];
            int bound = t[l];   // the layer left of the run
            for (int b = l; b <= h; ++b) {
                bound = std::min(bound + 1, last[b + 1]);
                out[b + 1] = bound;
            }
            bound = t[h + 2];
            for (int b = h; b >= l; --b) {
                bound = std::min(bound + 1, out[b + 1]);
                out[b + 1] = bound;
                gates += (bound - t[b + 1]) / 2;
            }
        }
        return gates;
    }
};

// Pack an ordered gate list into register groups.  A gate may join the
// current group only if no earlier gate left for later shares one of its
// bits (then it commutes with everything it overtakes).  Returns the gates
// that did not fit into max_groups groups.
std::vector<Gate> pack_groups(const fl_geom& g, std::vector<Gate> rem, fl_pass& pd, int max_groups) {
    pd.ngroups = 0;
    while (!rem.empty() && pd.ngroups < max_groups) {
        const int nrem = (int)rem.size();
        int best_u0 = -1, nbest = 0;
        int best[FL_MAX_OPS], take[FL_MAX_OPS];
        for (int u0 = 0; u0 + g.R <= g.K; ++u0) {
            unsigned blocked = 0;
            const unsigned inside = ((1u << g.R) - 1u) << u0;   // once all of it is blocked no gate fits
            int n = 0;
            for (int i = 0; i < nrem && (blocked & inside) != inside; ++i) {
                const unsigned m = 3u << rem[i].u;
                const bool fits = rem[i].u >= u0 && rem[i].u + 1 < u0 + g.R;
                if ((m & blocked) == 0 && fits && n < FL_MAX_OPS)
                    take[n++] = i;
                else
                    blocked |= m;
            }
            if (n > nbest) {
                nbest = n;
                best_u0 = u0;
                std::copy(take, take + n, best);
            }
        }
        const int gi = pd.ngroups++;
        pd.u0[gi] = (int8_t)best_u0;
        pd.nops[gi] = (int8_t)nbest;
        for (int k = 0; k < nbest; ++k) {
            const Gate& q = rem[best[k]];
            pd.opi[gi][k] = (int8_t)(q.u - best_u0);
            pd.opg[gi][k] = (int16_t)q.gidx;
            pd.ops[gi][k] = (int16_t)q.slot;
        }
        // drop the taken gates (best is in increasing order)
        int out = 0, k = 0;
        for (int i = 0; i < nrem; ++i) {
            if (k < nbest && best[k] == i)
                ++k;
            else
                rem[out++] = rem[i];
        }
        rem.resize(out);
    }
    return rem;
}

// The kernels apply a group's ops two at a time; an odd count costs a copy of
// the register group after the last op.  Shift ops across the boundary of
// consecutive groups, which keeps the pass's op sequence unchanged, wherever
// the op's bits lie inside the other group's register bits, so that fewer
// groups have odd counts; groups left empty are dropped (one LDS exchange
// less).
void balance_groups(const fl_geom& g, fl_pass& pd) {
    auto fits = [&](int gi, int u) { return u >= pd.u0[gi] && u + 1 < pd.u0[gi] + g.R; };
    auto set_op = [&](int gi, int k, int u, int16_t gate, int16_t slot) {
        pd.opi[gi][k] = (int8_t)(u - pd.u0[gi]);
        pd.opg[gi][k] = gate;
        pd.ops[gi][k] = slot;
    };
    for (int gi = 0; gi + 1 < pd.ngroups; ++gi) {
        if (!(pd.nops[gi] & 1)) continue;
        const int a = gi, b = gi + 1;
        const int kl = pd.nops[a] - 1;
        const int ul = pd.u0[a] + pd.opi[a][kl];
        if (fits(b, ul) && pd.nops[b] < FL_MAX_OPS) {
            // the last op of a becomes the first op of b
            for (int k = pd.nops[b]; k > 0; --k) {
                pd.opi[b][k] = pd.opi[b][k - 1];
                pd.opg[b][k] = pd.opg[b][k - 1];
                pd.ops[b][k] = pd.ops[b][k - 1];
            }
            set_op(b, 0, ul, pd.opg[a][kl], pd.ops[a][kl]);
            pd.nops[b]++;
            pd.nops[a]--;
            continue;
        }
        if (pd.nops[b] == 0) continue;
        const int uf = pd.u0[b] + pd.opi[b][0];
        if (fits(a, uf) && pd.nops[a] < FL_MAX_OPS) {
            // the first op of b becomes the last op of a
            set_op(a, pd.nops[a], uf, pd.opg[b][0], pd.ops[b][0]);
            pd.nops[a]++;
            for (int k = 0; k + 1 < pd.nops[b]; ++k) {
                pd.opi[b][k] = pd.opi[b][k + 1];
                pd.opg[b][k] = pd.opg[b][k + 1];
                pd.ops[b][k] = pd.ops[b][k + 1];
            }
            pd.nops[b]--;
        }
    }
    int out = 0;
    for (int gi = 0; gi < pd.ngroups; ++gi) {
        if (pd.nops[gi] == 0) continue;
        if (out != gi) {
            pd.u0[out] = pd.u0[gi];
            pd.nops[out] = pd.nops[gi];
            for (int k = 0; k < pd.nops[gi]; ++k) {
                pd.opi[out][k] = pd.opi[gi][k];
                pd.opg[out][k] = pd.opg[gi][k];
                pd.ops[out][k] = pd.ops[gi][k];
            }
        }
        ++out;
    }
    for (int gi = out; gi < pd.ngroups; ++gi) pd.nops[gi] = 0;
    pd.ngroups = out;
}

// Passes the plain greedy rule (the window admitting the most gates) needs to
// finish the circuit from state s; gives up once `most` are not enough.
int greedy_passes(const std::vector<Window>& windows, const Sched& s0, int cap, int most) {
    long long left = 0;
    for (int b = 0; b < s0.nb; ++b) left += s0.n - s0.cnt[b];
    if (left == 0) return 0;
    Profile p(s0);
    Sched s;         // kept only once a tile's rounds are cut short by the cap
    bool exact = true;
    int passes = 0;
    int a[2][66];
    while (left > 0) {
        if (passes >= most) return most + 1;
        int best = 0, best_w = -1, cur = 0;
        for (int k = 0; k < (int)windows.size(); ++k) {
            const int got = std::min(p.advance(windows[k], a[cur]), cap);
            if (got > best) {
                best = got;
                best_w = k;
                cur ^= 1;   // keep this window's layers
            }
        }
        if (best == 0) return 1 << 20;   // cannot happen for a valid circuit
        const Window& w = windows[best_w];
        if (best == cap) {
            // the rounds may end at the cap: run them one by one
            if (exact) s = s0;
            for (int b = 0; b < s0.nb; ++b) s.cnt[b] = (p.t[b + 1] - s0.off[b]) / 2;
            exact = false;
            run_tile(w, s, cap);
            for (int b = 0; b < s0.nb; ++b) p.t[b + 1] = 2 * s.cnt[b] + s0.off[b];
        } else {
            for (int r = 0; r < w.nruns; ++r)
                for (int b = w.lo[r]; b <= w.hi[r]; ++b) p.t[b + 1] = a[cur ^ 1][b + 1];
        }
        left -= best;
        ++passes;
    }
    return passes;
}

}  // namespace

std::vector<fl_pass> plan_sweep(const fl_geom& g, int n, bool dagger, bool with_slots,
                                int max_gates_per_pass, PlanStats* st, int max_groups) {
    if (max_groups < 1 || max_groups > FL_MAX_GROUPS) max_groups = FL_MAX_GROUPS;
    std::vector<fl_pass> plan;
    const int L = g.L, nb = L - 1;
    Sched s;
    s.L = L;
    s.nb = nb;
    s.n = n;
    s.cnt.assign(nb, 0);
    s.off.resize(nb);
    for (int b = 0; b < nb; ++b) {
        const bool first = dagger ? (b % 2 == 0) : (b % 2 == 1);
        s.off[b] = first ? 0 : 1;
    }
    std::vector<Window> windows;
    if (g.W == 0)
        windows.push_back(tile_window(g, g.C));
    else
        for (int h = g.C; h + g.W <= L; ++h) windows.push_back(tile_window(g, h));

    long long total = (long long)n * nb, done = 0;
    while (done < total) {
        // One-step lookahead: take the window after which the greedy rule
        // finishes in the fewest passes; ties go to the window that applies
        // more gates now, then to the lower window.
        int best_h = -1, best_cost = 1 << 20;
        std::vector<int> best;
        for (const Window& w : windows) {
            Sched t = s;
            std::vector<int> got = run_tile(w, t, max_gates_per_pass);
            if (got.empty()) continue;
            const int cost = greedy_passes(windows, t, max_gates_per_pass, best_cost);
            if (cost < best_cost || (cost == best_cost && got.size() > best.size())) {
                best_cost = cost;
                best = std::move(got);
                best_h = w.h;
            }
        }
        if (best.empty()) break;  // cannot happen for a valid circuit
        std::vector<Gate> gl;
        for (int b : best) {
            Gate q;
            q.bond = b;
            q.u = fl_local_bit(L - 2 - b, g.C, g.W, best_h);
            q.gidx = dagger ? nb + b : b;
            q.slot = with_slots ? b : -1;
            gl.push_back(q);
        }
        fl_pass pd;
        std::memset(&pd, 0, sizeof(pd));
        pd.h = best_h;
        std::vector<Gate> left = pack_groups(g, gl, pd, max_groups);
#if !defined(FL_NO_BALANCE)
        balance_groups(g, pd);
#endif
        if (with_slots) {
            // map the bonds of this pass to local reduction slots
            int map[64];
            for (int b = 0; b < 64; ++b) map[b] = -1;
            pd.nslots = 0;
            for (int gi = 0; gi < pd.ngroups; ++gi)
                for (int k = 0; k < pd.nops[gi]; ++k) {
                    const int b = pd.ops[gi][k];
                    if (map[b] < 0) {
                        map[b] = pd.nslots++;
                        pd.sbond[map[b]] = (int8_t)b;
                    }
                    pd.ops[gi][k] = (int16_t)map[b];
                }
        }
        // gates that did not fit are not applied in this pass
        for (int b : best) s.cnt[b]++;
        for (const Gate& q : left) s.cnt[q.bond]--;
        const long long applied = (long long)best.size() - (long long)left.size();
        done += applied;
        plan.push_back(pd);
        if (st) {
            st->passes++;
            st->gates += applied;
            st->groups += pd.ngroups;
        }
    }
    return plan;
}

std::vector<fl_pass> plan_cover(const fl_geom& g) {
    std::vector<fl_pass> plan;
    const int L = g.L, nb = L - 1;
    std::vector<char> covered(nb, 0);
    int left = nb;
    std::vector<int> windows;
    if (g.W == 0)
        windows.push_back(g.C);
    else
        for (int h = g.C; h + g.W <= L; ++h) windows.push_back(h);
    bool first = true;
    while (left > 0 || first) {
        int best_h = windows[0], best_n = -1;
        for (int h : windows) {
            int c = 0;
            for (int b = 0; b < nb; ++b)
                if (!covered[b] && bond_in_tile(g, h, b)) ++c;
            if (c > best_n) {
                best_n = c;
                best_h = h;
            }
        }
        fl_pass pd;
        std::memset(&pd, 0, sizeof(pd));
        pd.h = best_h;
        pd.flags = first ? 1 : 0;
        first = false;
        for (int b = 0; b < nb && pd.ngroups < FL_MAX_GROUPS; ++b) {
            if (covered[b] || !bond_in_tile(g, best_h, b)) continue;
            const int gi = pd.ngroups++;
            pd.u0[gi] = (int8_t)fl_local_bit(L - 2 - b, g.C, g.W, best_h);
            pd.nops[gi] = 1;
            pd.opi[gi][0] = 0;
            pd.opg[gi][0] = -1;
            pd.ops[gi][0] = (int16_t)b;
            covered[b] = 1;
            --left;
        }
        plan.push_back(pd);
    }
    return plan;
}

std::vector<fl_pass> plan_cover_groups(const fl_geom& g) {
    std::vector<fl_pass> plan = plan_cover(g);
    for (fl_pass& pd : plan) {
        // (tile bit, bond) of every bond of the pass, by tile bit
        std::vector<std::pair<int, int>> bonds;
        for (int gi = 0; gi < pd.ngroups; ++gi) bonds.emplace_back((int)pd.u0[gi], (int)pd.ops[gi][0]);
        std::sort(bonds.begin(), bonds.end());
        fl_pass q;
        std::memset(&q, 0, sizeof(q));
        q.h = pd.h;
        q.flags = pd.flags;
        size_t k = 0;
        while (k < bonds.size()) {
            const int u0 = std::min(bonds[k].first, g.K - g.R);
            const int gi = q.ngroups++;
            q.u0[gi] = (int8_t)u0;
            int n = 0;
            while (k < bonds.size() && bonds[k].first + 1 < u0 + g.R) {
                q.opi[gi][n] = (int8_t)(bonds[k].first - u0);
                q.opg[gi][n] = -1;
                q.ops[gi][n] = (int16_t)bonds[k].second;
                ++n;
                ++k;
            }
            q.nops[gi] = (int8_t)n;
        }
        pd = q;
    }
    return plan;
}

std::vector<rdm_desc> cover_windows(const fl_geom& g) {
    std::vector<rdm_desc> out;
    for (const fl_pass& p : plan_cover(g)) {
        std::vector<std::pair<int, int>> bonds;   // (tile bit, bond)
        for (int k = 0; k < p.ngroups; ++k) bonds.emplace_back((int)p.u0[k], (int)p.ops[k][0]);
        std::sort(bonds.begin(), bonds.end());
        size_t done = 0;
        bool first = true;
        while (done < bonds.size()) {
            const size_t left = std::min<size_t>(bonds.size() - done, 12);
            rdm_desc d;
            std::memset(&d, 0, sizeof(d));
            d.h = p.h;
            d.flags = first ? p.flags : 0;
            d.nwin = left <= 3 ? 1 : left <= 6 ? 2 : 4;
            const size_t end = done + left;
            for (int w = 0; w < d.nwin; ++w) {
                const size_t share = (end - done + (size_t)(d.nwin - w) - 1) / (size_t)(d.nwin - w);
                if (share == 0) continue;   // an empty window: mask 0
                d.u0[w] = std::min(bonds[done].first, g.K - 4);
                for (size_t k = 0; k < share && bonds[done].first + 1 < d.u0[w] + 4; ++k) {
                    const int j = bonds[done].first - d.u0[w];
                    d.mask[w] |= 1 << j;
                    d.bond[w][j] = bonds[done].second;
                    if (++done == end) break;
                }
            }
            first = false;
            out.push_back(d);   // bonds that no window reached come in another pass
        }
    }
    return out;
}

void serialize_plan(const fl_geom& g, const std::vector<fl_pass>& plan, std::vector<int>& out) {
    out.clear();
    out.push_back(g.C);
    out.push_back(g.W);
    out.push_back(g.R);
    out.push_back((int)plan.size());
    for (const fl_pass& p : plan) {
        out.push_back(p.h);
        out.push_back(p.ngroups);
        out.push_back(p.flags);
        for (int gi = 0; gi < p.ngroups; ++gi) {
            out.push_back(p.u0[gi]);
            out.push_back(p.nops[gi]);
            for (int k = 0; k < p.nops[gi]; ++k) {
                out.push_back(p.opi[gi][k]);
                out.push_back(p.opg[gi][k]);
                const int sl = p.ops[gi][k];
                // report reduction slots as bond indices
                out.push_back((p.nslots > 0 && sl >= 0) ? (int)p.sbond[sl] : sl);
            }
        }
    }
}

}  // namespace fl
