// Plan of a tape's replay, shared by the two schedulers: liveness, activity,
// value numbering, multiply-add fusion, branch arms (Info), checkpoint
// segments, recomputation and resident values (Builder).
#pragma once
#include <algorithm>
#include <map>
#include <string>
#include <vector>

#include "common.h"

namespace ndvm {

enum Kind : uint8_t { K_COMP = 0, K_CONST = 1, K_OBS = 2, K_PARAM = 3 };

struct Info {
    const Tape &t;
    uint32_t N, P;
    std::vector<uint8_t> kind, nel, live, active, has_adj, need_rev;
    // Value numbering: rep[k] is the first slot that computes the same value
    // as slot k (same opcode, shape and immediate on the same operand values;
    // every op is a deterministic function of its operands, so the bits are
    // equal).  Only representatives are computed; every reader of a value
    // reads its representative's register.  Adjoints stay per slot, so each
    // slot keeps its own adjoint rule and the reverse sweep is unchanged.
    std::vector<uint32_t> rep;
    std::vector<uint8_t> vlive;      // representative whose value is needed
    std::vector<uint32_t> last_use;  // last forward reader of a value, or N for the loss
    // Multiply-add fusion: fmul[c] = 1 + m when the product m is folded into
    // the sum or difference c (c reads m's operands instead of m), else 0.
    // m's value is then never formed: its only reader is c and no adjoint
    // rule reads it.  x*y + z rounds the product and then the sum, so c
    // keeps the bits of the two separate operations.
    std::vector<uint32_t> fmul;
    // Differences take only a subtracted product one of whose factors is a
    // constant or a parameter (the wide kernel has no x*y - z; it computes
    // z - x*y as z + (-x)*y with a register holding the negated factor).
    bool fold_static_subtrahend = false;
    bool fold_scalars_only = false;

    explicit Info(const Tape &tape) : t(tape), N(uint32_t(tape.ops.size())), P(tape.n_params) {}

    // operand values of op k (as representatives; a fused sum reads the
    // product's operands, then its other operand)
    template <class F>
    void for_operands(uint32_t k, F f) const {
        if (!fmul.empty() && fmul[k]) {
            const uint32_t m = fmul[k] - 1;
            const TapeOp &o = t.ops[k];
            f(rep[t.ops[m].a]);
            f(rep[t.ops[m].b]);
            f(rep[rep[o.a] == m ? o.b : o.a]);
            return;
        }
        for_operands_raw(k, [&](uint32_t s) { f(rep[s]); });
    }
    // operand slots of op k as written in the tape
    template <class F>
    void for_operands_raw(uint32_t k, F f) const {
        const TapeOp &o = t.ops[k];
        switch (o.code) {
        case tp::CONST: case tp::PARAM: case tp::OBS:
            return;
        case tp::PACK:
            for (uint32_t i = 0; i < o.b; ++i) f(t.aux[o.a + i]);
            return;
        case tp::SELECT:
            f(o.a); f(o.b); f(o.c); f(o.d);
            return;
        case tp::ADD: case tp::SUB: case tp::MUL: case tp::DIV: case tp::POW: case tp::DOT:
        case tp::MATMUL: case tp::OUTER:
            f(o.a); f(o.b);
            return;
        default:
            f(o.a);
        }
    }
    // operands that receive an adjoint contribution from op k
    template <class F>
    void for_targets(uint32_t k, F f) const {
        const TapeOp &o = t.ops[k];
        switch (o.code) {
        case tp::CONST: case tp::PARAM: case tp::OBS:
            return;
        case tp::PACK:
            for (uint32_t i = 0; i < o.b; ++i) f(t.aux[o.a + i]);
            return;
        case tp::SELECT:
            f(o.c); f(o.d);
            return;
        case tp::ADD: case tp::SUB: case tp::MUL: case tp::DIV: case tp::POW: case tp::DOT:
        case tp::MATMUL: case tp::OUTER:
            f(o.a); f(o.b);
            return;
        default:
            f(o.a);
        }
    }
    // values the adjoint rule of op k reads (k itself = its output z), as
    // representatives
    template <class F>
    void for_revreads(uint32_t k, F f) const {
        for_revreads_raw(k, [&](uint32_t s) { f(rep[s]); });
    }
    // a slot that receives adjoint contributions
    bool takes_adjoint(uint32_t s) const { return kind[s] == K_PARAM || (kind[s] == K_COMP && active[s]); }
    // With exact_revreads, only what the contributions to the operands that
    // take them read.
    bool exact_revreads = false;
    template <class F>
    void for_revreads_raw(uint32_t k, F f) const {
        const TapeOp &o = t.ops[k];
        if (exact_revreads) {
            const bool ta = takes_adjoint(o.a), tb = takes_adjoint(o.b);
            switch (o.code) {
            case tp::MUL:
                if (tb) f(o.a);
                if (ta) f(o.b);
                return;
            case tp::DIV:
                f(o.b);
                if (tb) f(k);
                return;
            case tp::POW:
                f(o.a);
                if (ta) f(o.b);
                f(k);
                return;
            default: break;
            }
        }
        switch (o.code) {
        case tp::MUL: case tp::DOT: case tp::MATMUL: case tp::OUTER: case tp::SELECT:
            f(o.a); f(o.b);
            return;
        case tp::DIV: f(o.b); f(k); return;
        case tp::EXP: f(k); return;
        case tp::LOG: case tp::SIN: case tp::COS: case tp::ABS: case tp::LOGDET: f(o.a); return;
        case tp::SQRT: f(o.a); f(k); return;
        case tp::POW: f(o.a); f(o.b); f(k); return;
        case tp::INV: f(k); return;
        case tp::DET: f(o.a); f(k); return;
        default: return;
        }
    }

    bool is_static(uint32_t s) const { return kind[rep[s]] == K_CONST || kind[rep[s]] == K_PARAM; }

    // Fold a product into the sum or difference that is its only reader,
    // elementwise ops of one shape only (no broadcast operand).
    void fuse_products() {
        std::vector<uint32_t> readers(N, 0);
        std::vector<uint8_t> rule_reads(N, 0);
        for (uint32_t k = 0; k < N; ++k)
            if (vlive[k] && rep[k] == k) for_operands(k, [&](uint32_t s) { readers[s]++; });
        readers[rep[t.loss]]++;
        for (uint32_t k = 0; k < N; ++k)
            if (need_rev[k]) for_revreads(k, [&](uint32_t s) { rule_reads[s] = 1; });
        fmul.assign(N, 0);
        for (uint32_t c = 0; c < N; ++c) {
            const TapeOp &o = t.ops[c];
            if (!vlive[c] || rep[c] != c || kind[c] != K_COMP || (o.code != tp::ADD && o.code != tp::SUB)) continue;
            if (fold_scalars_only && nel[c] != 1) continue;
            const bool restricted = fold_static_subtrahend && o.code == tp::SUB;
            for (uint32_t side = restricted ? 1 : 0; side < 2; ++side) {
                const uint32_t m = rep[side == 0 ? o.a : o.b], other = rep[side == 0 ? o.b : o.a];
                if (restricted && !(kind[m] == K_COMP && t.ops[m].code == tp::MUL &&
                                    (is_static(t.ops[m].a) || is_static(t.ops[m].b))))
                    continue;
                if (kind[m] != K_COMP || t.ops[m].code != tp::MUL || rep[m] != m || !vlive[m]) continue;
                if (readers[m] != 1 || rule_reads[m] || m == rep[t.loss] || m == other) continue;
                const uint32_t n = nel[c];
                if (nel[m] != n || nel[other] != n || nel[t.ops[m].a] != n || nel[t.ops[m].b] != n) continue;
                fmul[c] = m + 1;
                vlive[m] = 0;
                break;
            }
        }
    }

    void number_values() {
        rep.assign(N, 0);
        std::map<std::vector<uint32_t>, uint32_t> first;
        std::vector<uint32_t> key;
        for (uint32_t k = 0; k < N; ++k) {
            const TapeOp &o = t.ops[k];
            key.assign({o.code, o.rows, o.cols, o.imm});
            for_operands_raw(k, [&](uint32_t s) { key.push_back(rep[s]); });
            auto it = first.emplace(key, k).first;
            rep[k] = it->second;
        }
    }

    void analyse() {
        kind.assign(N, K_COMP);
        nel.assign(N, 1);
        for (uint32_t k = 0; k < N; ++k) {
            uint16_t c = t.ops[k].code;
            kind[k] = c == tp::CONST ? K_CONST : c == tp::OBS ? K_OBS : c == tp::PARAM ? K_PARAM : K_COMP;
            nel[k] = uint8_t(t.nel(k));
        }
        number_values();
        // structure of the trace: slots the loss depends on (every one keeps
        // its adjoint rule, duplicates included)
        live.assign(N, 0);
        live[t.loss] = 1;
        for (uint32_t k = N; k-- > 0;)
            if (live[k]) for_operands_raw(k, [&](uint32_t s) { live[s] = 1; });
        active.assign(N, 0);
        for (uint32_t k = 0; k < N; ++k) {
            if (kind[k] == K_PARAM) { active[k] = 1; continue; }
            if (kind[k] != K_COMP) continue;
            bool a = false;
            for_targets(k, [&](uint32_t s) { a = a || active[s]; });
            active[k] = a;
        }
        has_adj.assign(N, 0);
        need_rev.assign(N, 0);
        has_adj[t.loss] = active[t.loss];
        for (uint32_t k = N; k-- > 0;) {
            if (!live[k] || kind[k] != K_COMP || !has_adj[k] || !active[k]) continue;
            need_rev[k] = 1;
            for_targets(k, [&](uint32_t s) {
                if (active[s]) has_adj[s] = 1;
            });
        }
        // values to compute: the loss, what the adjoint rules read, and what
        // those depend on
        vlive.assign(N, 0);
        vlive[rep[t.loss]] = 1;
        for (uint32_t k = N; k-- > 0;) {
            if (need_rev[k]) for_revreads(k, [&](uint32_t s) { vlive[s] = 1; });
            if (vlive[k] && rep[k] == k) for_operands(k, [&](uint32_t s) { vlive[s] = 1; });
        }
        fuse_products();
        last_use.assign(N, 0);
        for (uint32_t k = 0; k < N; ++k)
            if (vlive[k] && rep[k] == k) for_operands(k, [&](uint32_t s) { last_use[s] = k; });
        last_use[rep[t.loss]] = N;
        // no skippable arms unless find_arms finds them
        cone_of.assign(N, -1);
        sel_group.assign(N, -1);
        arm_of.assign(N, -1);
        hoist.assign(N, 0);
        groups.clear();
    }

    // ---- arms of numeric branches that a wave may skip (Section 6 lane
    // masking, taken per wave: when every lane of a wave decides a branch
    // the same way, the other arm's forward values and adjoint rules are not
    // run).  A group is one branch: a run of consecutive SELECT slots with the
    // same predicate operands.  Its cone on side 0 (then) / 1 (else) is the
    // set of values whose every reader is in that cone or is a select of the
    // group reading it through that side's input: values no lane needs when
    // the wave takes the other arm.  Groups inside another group's cone are
    // not skipped on their own (they are part of the outer arm).
    struct Group {
        std::vector<uint32_t> sel;       // SELECT slots, ascending
        uint32_t a = 0, b = 0;           // predicate operand slots
        std::vector<uint32_t> cone[2];   // representatives, ascending
        uint32_t lo = 0, hi = 0;         // tape range of its cones and selects
        std::vector<uint32_t> hoisted;   // observation loads laid out before the arms
    };
    std::vector<Group> groups;
    std::vector<int32_t> cone_of;        // representative -> 2 * group + side, or -1
    std::vector<int32_t> sel_group;      // SELECT slot -> group, or -1
    std::vector<int32_t> arm_of;         // slot -> 2 * group + side of the arm holding its rule, or -1
    std::vector<uint8_t> hoist;          // observation loads laid out with an earlier branch's arms

    void find_arms(uint32_t arm_min, uint32_t merge) {
        cone_of.assign(N, -1);
        sel_group.assign(N, -1);
        groups.clear();
        std::vector<uint32_t> readers(N, 0);
        for (uint32_t k = 0; k < N; ++k)
            if (vlive[k] && rep[k] == k) for_operands(k, [&](uint32_t s) { readers[s]++; });
        readers[rep[t.loss]]++;
        std::vector<Group> all;
        for (uint32_t k = 0; k < N;) {
            const TapeOp &o = t.ops[k];
            if (o.code != tp::SELECT) { ++k; continue; }
            Group g;
            g.a = o.a;
            g.b = o.b;
            uint32_t e = k;
            while (e < N && t.ops[e].code == tp::SELECT && rep[t.ops[e].a] == rep[o.a] && rep[t.ops[e].b] == rep[o.b])
                g.sel.push_back(e++);
            k = e;
            bool live = false;
            for (uint32_t q : g.sel) live = live || (vlive[q] && rep[q] == q);
            if (!live) continue;
            for (uint32_t side = 0; side < 2; ++side) {
                std::vector<uint32_t> cnt(N, 0);   // readers accounted for by the cone
                uint32_t top = 0;
                for (uint32_t q : g.sel) {
                    if (!(vlive[q] && rep[q] == q)) continue;
                    const TapeOp &so = t.ops[q];
                    const uint32_t in = rep[side == 0 ? so.c : so.d];
                    cnt[in]++;
                    top = std::max(top, in);
                }
                for (uint32_t v = top + 1; v-- > 0;) {
                    if (!cnt[v] || cnt[v] != readers[v] || rep[v] != v || !vlive[v] || kind[v] != K_COMP) continue;
                    // a select of the branch itself (one reading another) stays with the selects
                    if (std::find(g.sel.begin(), g.sel.end(), v) != g.sel.end()) continue;
                    g.cone[side].push_back(v);
                    for_operands(v, [&](uint32_t s2) { cnt[s2]++; });
                }
                std::reverse(g.cone[side].begin(), g.cone[side].end());
                // arms below arm_min elements stay unmarked
                uint32_t elems = 0;
                for (uint32_t v : g.cone[side]) elems += nel[v];
                if (elems < arm_min) g.cone[side].clear();
            }
            if (g.cone[0].empty() && g.cone[1].empty()) continue;
            all.push_back(std::move(g));
        }
        std::vector<int32_t> in_cone(N, -1);
        for (uint32_t gi = 0; gi < all.size(); ++gi)
            for (uint32_t side = 0; side < 2; ++side)
                for (uint32_t v : all[gi].cone[side]) in_cone[v] = int32_t(gi);
        std::vector<Group> kept;
        for (uint32_t gi = 0; gi < all.size(); ++gi) {
            bool nested = false;
            for (uint32_t q : all[gi].sel) nested = nested || (in_cone[rep[q]] >= 0 && in_cone[rep[q]] != int32_t(gi));
            if (!nested) kept.push_back(std::move(all[gi]));
        }
        // Branches on the same predicate value one after another (the trips
        // of a loop around a branch) share one skip test: the later arms'
        // values are computed with the first branch's, so the arms of up to
        // `merge` branches are independent chains the packer can put side
        // by side (one arm alone is mostly a dependent chain).  A later arm
        // qualifies when every value it reads from outside itself is a
        // constant, a parameter, an observation (its load moves up before
        // the skip test) or a value computed before the first branch's arm.
        hoist.assign(N, 0);
        for (size_t gi = 0; gi < kept.size();) {
            Group g = std::move(kept[gi]);
            const uint32_t at = g.sel.front();   // where the arms are laid out
            size_t e = gi + 1;
            std::vector<uint32_t> loads;
            for (uint32_t members = 1; e < kept.size() && members < merge; ++e, ++members) {
                const Group &h = kept[e];
                if (rep[h.a] != rep[g.a] || rep[h.b] != rep[g.b]) break;
                bool ok = true;
                std::vector<uint32_t> hl;
                for (uint32_t side = 0; side < 2 && ok; ++side)
                    for (uint32_t v : h.cone[side]) {
                        for_operands(v, [&](uint32_t u) {
                            if (std::binary_search(h.cone[side].begin(), h.cone[side].end(), u)) return;
                            if (kind[u] == K_CONST || kind[u] == K_PARAM) return;
                            if (kind[u] == K_OBS) {
                                if (u > at) hl.push_back(u);
                                return;
                            }
                            if (u >= at || cone_of[u] >= 0) ok = false;
                        });
                        // the arm's adjoint rules run after the first branch's
                        // select rules: every slot they add to outside the arm
                        // must have its own rule run later (lie before it)
                        const uint32_t fused = (!fmul.empty() && fmul[v]) ? fmul[v] - 1 : N;   // in the arm too
                        auto raw_ok = [&](uint32_t r) {
                            if (kind[r] != K_COMP) return;
                            if (std::binary_search(h.cone[side].begin(), h.cone[side].end(), rep[r])) return;
                            if (r >= at && r != fused) ok = false;
                        };
                        for_operands_raw(v, raw_ok);
                        if (!fmul.empty() && fmul[v]) for_operands_raw(fmul[v] - 1, raw_ok);
                    }
                if (!ok) break;
                for (uint32_t side = 0; side < 2; ++side) {
                    g.cone[side].insert(g.cone[side].end(), h.cone[side].begin(), h.cone[side].end());
                    std::sort(g.cone[side].begin(), g.cone[side].end());
                }
                g.sel.insert(g.sel.end(), h.sel.begin(), h.sel.end());
                loads.insert(loads.end(), hl.begin(), hl.end());
            }
            gi = e;
            std::sort(loads.begin(), loads.end());
            loads.erase(std::unique(loads.begin(), loads.end()), loads.end());
            for (uint32_t u : loads) hoist[u] = 1;
            g.hoisted = std::move(loads);
            const int32_t id = int32_t(groups.size());
            g.lo = g.sel.front();
            g.hi = g.sel.back();
            for (uint32_t side = 0; side < 2; ++side)
                for (uint32_t v : g.cone[side]) {
                    cone_of[v] = 2 * id + int32_t(side);
                    g.lo = std::min(g.lo, v);
                }
            for (uint32_t q : g.sel) sel_group[q] = id;
            groups.push_back(std::move(g));
        }
        // Slots whose adjoint rules lie in an arm: the cone's values; a
        // product folded into a cone value's sum (its value is never formed,
        // its rule is); duplicates of a cone value up to the branch's last
        // select (an adjoint rule there may contribute to a cone value, so it
        // must run before that value's rule).  A duplicate after the last
        // select is laid out before the arm as usual; when the wave skips the
        // arm its adjoint is exactly zero (only selects of the same predicate
        // and the arm's own values reach it), so its gated contributions are
        // nothing whatever stale values it reads.
        arm_of.assign(N, -1);
        for (uint32_t k = 0; k < N; ++k) {
            const int32_t c = cone_of[rep[k]];
            if (c >= 0 && k <= groups[uint32_t(c) / 2].hi) arm_of[k] = c;
        }
        for (uint32_t c = 0; c < N; ++c)
            if (!fmul.empty() && fmul[c] && arm_of[c] >= 0) {
                const uint32_t m = fmul[c] - 1;
                arm_of[m] = arm_of[c];
                Group &g = groups[uint32_t(arm_of[c]) / 2];
                g.lo = std::min(g.lo, m);
            }
    }
    // the cone (2 * group + side) a slot's adjoint rule or value belongs to, or -1
    int32_t cone_of_slot(uint32_t k) const { return arm_of[k]; }
};

struct Builder {
    const Info &I;
    const Tape &t;
    uint32_t N, P;
    // plan
    std::vector<uint32_t> cuts;       // segment starts, cuts[0] = 0
    std::vector<uint32_t> seg_of;
    std::vector<uint8_t> resident;
    std::vector<std::vector<uint32_t>> livein, recomp, revops;
    std::vector<uint32_t> res_off;    // resident slot -> offset in resident block
    uint32_t res_elems = 0;
    // save policy: values the adjoint rules read are stored in the forward
    // sweep (as segment inputs of their own segment) instead of recomputed
    bool save_reads = false;

    explicit Builder(const Info &info) : I(info), t(info.t), N(info.N), P(info.P) {}

    // a computed value the program needs (representatives only)
    bool comp_live(uint32_t s) const { return I.kind[s] == K_COMP && I.vlive[s]; }

    void set_cuts(const std::vector<uint32_t> &c) {
        cuts = c;
        seg_of.assign(N, 0);
        uint32_t j = 0;
        for (uint32_t k = 0; k < N; ++k) {
            while (j + 1 < cuts.size() && cuts[j + 1] <= k) ++j;
            seg_of[k] = j;
        }
    }

    void plan(bool with_residents) {
        uint32_t m = uint32_t(cuts.size());
        if (!with_residents) resident.assign(N, 0);
        livein.assign(m, {});
        recomp.assign(m, {});
        revops.assign(m, {});
        std::vector<uint32_t> mark(N, UINT32_MAX), inmark(N, UINT32_MAX), stack;
        for (uint32_t j = 0; j < m; ++j) {
            uint32_t lo = cuts[j], hi = j + 1 < m ? cuts[j + 1] : N;
            auto need = [&](uint32_t s) {
                if (I.kind[s] == K_OBS) {   // observations are reloaded, never checkpointed
                    if (mark[s] != j) { mark[s] = j; stack.push_back(s); }
                    return;
                }
                if (I.kind[s] != K_COMP || resident[s]) return;
                if (s >= lo && !save_reads) {
                    if (mark[s] != j) { mark[s] = j; stack.push_back(s); }
                } else if (inmark[s] != j) {
                    inmark[s] = j;
                    livein[j].push_back(s);
                }
            };
            for (uint32_t k = hi; k-- > lo;)
                if (I.need_rev[k]) {
                    revops[j].push_back(k);
                    I.for_revreads(k, need);
                }
            while (!stack.empty()) {
                uint32_t s = stack.back();
                stack.pop_back();
                recomp[j].push_back(s);
                I.for_operands(s, need);
            }
            std::sort(recomp[j].begin(), recomp[j].end());
            std::sort(livein[j].begin(), livein[j].end());
        }
    }

    void choose_residents(uint32_t K) {
        std::vector<uint32_t> cnt(N, 0);
        for (auto &v : livein)
            for (uint32_t s : v) cnt[s]++;
        resident.assign(N, 0);
        res_off.assign(N, 0);
        res_elems = 0;
        for (uint32_t s = 0; s < N; ++s)
            if (cnt[s] > K) {
                resident[s] = 1;
                res_off[s] = res_elems;
                res_elems += I.nel[s];
            }
    }

    std::vector<uint32_t> choose_cuts(uint64_t S) const {
        std::vector<int64_t> diff(N + 2, 0);
        for (uint32_t s = 0; s < N; ++s) {
            if (!comp_live(s) || resident[s]) continue;
            uint32_t lu = std::min(I.last_use[s], N);
            if (lu > s) {
                diff[s + 1] += I.nel[s];
                diff[lu + 1] -= I.nel[s];
            }
        }
        std::vector<int64_t> w(N + 1, 0);
        int64_t run = 0;
        for (uint32_t p = 0; p <= N; ++p) {
            run += diff[p];
            w[p] = run;
        }
        // no cut inside a skippable branch: its arms are laid out next to
        // its selects, after the positions their ops had in the tape
        std::vector<uint8_t> nocut(N + 1, 0);
        for (const auto &g : I.groups)
            for (uint32_t p = g.lo + 1; p <= g.hi; ++p) nocut[p] = 1;
        std::vector<uint32_t> c{0};
        uint64_t acc = 0;
        int64_t best = -1;
        uint32_t start = 0;
        for (uint32_t k = 0; k < N; ++k) {
            if (comp_live(k)) acc += I.nel[k];
            uint32_t p = k + 1;
            if (p >= N) break;
            if (acc * 2 >= S && p > start && !nocut[p]) {
                if (best < 0 || w[p] <= w[best]) best = p;
            }
            if (acc >= S && best > 0) {
                c.push_back(uint32_t(best));
                start = uint32_t(best);
                acc = 0;
                for (uint32_t q = start; q <= k; ++q)
                    if (comp_live(q)) acc += I.nel[q];
                best = -1;
            }
        }
        return c;
    }
};

}  // namespace ndvm
