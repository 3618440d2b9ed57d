#include "tables.hpp"

#include <algorithm>
#include <map>
#include <stdexcept>

namespace xg2 {

FlatTables flatten(const Grammar& g) {
    FlatTables t;
    t.state_info.resize((size_t)g.n_states);
    t.rule_info.resize(g.rules.size());
    {
        size_t nb = 0, nr = 0;
        for (const RuleFsm& f : g.rules) { nb += f.body->bedges.v.size(); nr += f.redges.v.size(); }
        t.byte_edges.reserve(nb); t.ref_edges.reserve(nr);
    }
    for (size_t r = 0; r < g.rules.size(); ++r) {
        const RuleFsm& f = g.rules[r];
        t.rule_info[r] = {(uint32_t)g.sid((int32_t)r, 0), f.nullable ? 1u : 0u};
        for (int q = 0; q < f.n_states(); ++q) {
            StateInfo si;
            si.byte_off = (uint32_t)t.byte_edges.size();
            si.ref_off = (uint32_t)t.ref_edges.size();
            for (auto& e : f.bedges(q)) t.byte_edges.push_back({(uint32_t)e.lo | ((uint32_t)e.hi << 8), (uint32_t)g.sid((int32_t)r, e.tgt)});
            for (auto& e : f.refs(q)) t.ref_edges.push_back({(uint32_t)e.rule, (uint32_t)g.sid((int32_t)r, e.tgt)});
            si.counts = (uint32_t)f.bedges(q).size() | ((uint32_t)f.refs(q).size() << 16);
            si.rule_final = (uint32_t)r | (f.is_final(q) ? 0x80000000u : 0u);
            t.state_info[(size_t)g.sid((int32_t)r, q)] = si;
        }
    }
    t.root_start = (uint32_t)g.sid(g.root, 0);
    // expansions: closure of prediction and of advancing over empty-deriving rules, per state with rule edges
    t.dev_state.resize(t.state_info.size());
    {
        std::vector<std::pair<uint32_t, uint32_t>> queue;            // (state, 1 = origin is the set being built)
        std::vector<uint32_t> items, triples;
        for (size_t sid = 0; sid < t.state_info.size(); ++sid) {
            const StateInfo& s0 = t.state_info[sid];
            DevState ds{s0.rule_final & 0x7FFFFFFFu, (uint32_t)t.exp_list.size(), 0, 0};
            if (s0.counts >> 16) {
                queue.assign(1, {(uint32_t)sid, 0u});
                items.clear(); triples.clear();
                auto enqueue = [&](uint32_t u, uint32_t cur) {
                    for (auto& q : queue) if (q.first == u && q.second == cur) return;
                    queue.emplace_back(u, cur);
                };
                for (size_t qi = 0; qi < queue.size(); ++qi) {
                    const uint32_t u = queue[qi].first, cur = queue[qi].second;
                    const StateInfo& su = t.state_info[u];
                    const uint32_t nb = su.counts & 0xFFFF, nr = su.counts >> 16;
                    const bool listed = nb > 0 || (su.rule_final >> 31) || nr == 0;   // scannable or completing
                    if (qi > 0 && listed) items.push_back(t.ref(u) | (cur ? kExpCurrent : 0u));
                    for (uint32_t k = 0; k < nr; ++k) {
                        const RefEdgeP& e = t.ref_edges[su.ref_off + k];
                        triples.push_back(e.rule);
                        triples.push_back(t.ref(e.tgt) | (cur ? kExpCurrent : 0u));
                        enqueue(t.rule_info[e.rule].start, 1u);
                        if (t.rule_info[e.rule].nullable) enqueue(e.tgt, cur);
                    }
                }
                ds.n_items = (uint32_t)items.size();
                ds.n_triples = (uint32_t)(triples.size() / 2);
                t.exp_list.insert(t.exp_list.end(), items.begin(), items.end());
                t.exp_list.insert(t.exp_list.end(), triples.begin(), triples.end());
            }
            t.dev_state[sid] = ds;
        }
    }
    // Byte classes: bytes that lead to the same target from every state are one class.  Every edge is a byte range, so
    // bytes between two consecutive range boundaries always behave alike: what follows runs over those intervals.
    // Every edge adds a 64-bit mix of (state, target) to the intervals it covers (as a difference at its two ends), so
    // intervals that behave alike have equal sums after one pass over the edges; that intervals with equal sums behave
    // alike is confirmed while the transitions are written below, and if it ever fails the mix is drawn anew.
    const size_t n = t.state_info.size();
    std::vector<uint8_t> is_bound(257, 0);
    is_bound[0] = 1;
    for (const ByteEdge& e : t.byte_edges) { is_bound[e.lohi & 0xFF] = 1; is_bound[((e.lohi >> 8) & 0xFF) + 1] = 1; }
    std::vector<uint32_t> iv_lo;                                    // first byte of every interval, ascending
    uint32_t iv_of[256];
    for (uint32_t b = 0; b < 256; ++b) {
        if (is_bound[b]) iv_lo.push_back(b);
        iv_of[b] = (uint32_t)iv_lo.size() - 1;
    }
    const uint32_t m = (uint32_t)iv_lo.size();
    t.sink = (uint32_t)n;
    std::vector<uint32_t> cls(m), cls_size;                         // interval -> class; intervals of each class
    std::vector<uint8_t> is_first(m);                               // the interval is the first of its class
    std::vector<uint64_t> sum(m + 1);
    for (uint64_t salt = 0x9E3779B97F4A7C15ull;; salt += 0x632BE59BD9B4E019ull) {
        std::fill(sum.begin(), sum.end(), 0);
        for (size_t sid = 0; sid < n; ++sid) {
            const StateInfo& si = t.state_info[sid];
            for (uint32_t k = 0; k < (si.counts & 0xFFFF); ++k) {
                const ByteEdge& e = t.byte_edges[si.byte_off + k];
                uint64_t x = (((uint64_t)sid << 32) | e.tgt) * 0xFF51AFD7ED558CCDull + salt;
                x ^= x >> 29; x *= 0xC4CEB9FE1A85EC53ull; x ^= x >> 32;
                sum[iv_of[e.lohi & 0xFF]] += x;
                sum[iv_of[(e.lohi >> 8) & 0xFF] + 1] -= x;
            }
        }
        uint32_t nc = 0;                                            // classes are numbered by their smallest byte
        cls_size.clear();
        std::vector<uint64_t> of_class;
        uint64_t run = 0;
        for (uint32_t j = 0; j < m; ++j) {
            run += sum[j];
            uint32_t c = 0;
            while (c < nc && of_class[c] != run) ++c;
            is_first[j] = c == nc;
            if (c == nc) { of_class.push_back(run); cls_size.push_back(0); ++nc; }
            cls[j] = c;
            ++cls_size[c];
        }
        if (nc > 256) throw std::logic_error("more byte classes than bytes");
        t.n_classes = nc;
        // one row more than there are states: the sink, which every missing edge leads to and which leads to itself, so
        // that an automaton walk needs no "is there an edge" branch (a dead run just stays in the sink)
        t.trans.assign((n + 1) * nc, t.sink);
        bool alike = true;
        for (size_t sid = 0; sid < n && alike; ++sid) {
            const StateInfo& si = t.state_info[sid];
            uint32_t* row = t.trans.data() + sid * nc;
            uint32_t covered = 0, expected = 0;                     // intervals with an edge; intervals of the classes seen
            for (uint32_t k = 0; k < (si.counts & 0xFFFF); ++k) {
                const ByteEdge& e = t.byte_edges[si.byte_off + k];
                const uint32_t ref = t.ref(e.tgt), j0 = iv_of[e.lohi & 0xFF], j1 = iv_of[(e.lohi >> 8) & 0xFF];
                covered += j1 - j0 + 1;
                for (uint32_t j = j0; j <= j1; ++j) {
                    if (is_first[j]) { row[cls[j]] = ref; expected += cls_size[cls[j]]; }
                    else alike &= row[cls[j]] == ref;
                }
            }
            alike &= covered == expected;
        }
        if (alike) break;
    }
    t.byte_class_words.assign(64, 0);
    for (int b = 0; b < 256; ++b) t.byte_class_words[(size_t)b >> 2] |= cls[iv_of[(size_t)b]] << ((b & 3) * 8);
    return t;
}

SiteTable site_table(const FlatTables& t, const std::function<uint32_t(const RefEdgeP&)>& number) {
    const size_t n = t.state_info.size();
    std::vector<uint32_t> edges(n, 0);
    for (const RefEdgeP& e : t.ref_edges) ++edges[e.tgt];
    SiteTable s;
    s.off.assign(n + 1, 0);
    for (size_t x = 0; x < n; ++x) {
        uint32_t size = edges[x] < 2 ? edges[x] : 4;
        while (size > 1 && size < 2 * edges[x]) size *= 2;
        s.off[x + 1] = s.off[x] + size;
    }
    s.slot.resize(2 * (size_t)s.off[n]);
    for (size_t k = 0; k < s.off[n]; ++k) { s.slot[2 * k] = kNoRule; s.slot[2 * k + 1] = 0; }
    for (const RefEdgeP& e : t.ref_edges) {
        const uint32_t size = s.off[(size_t)e.tgt + 1] - s.off[e.tgt];
        uint32_t k = site_home(e.rule, size);
        auto at = [&] { return s.slot.data() + 2 * (size_t)(s.off[e.tgt] + k); };
        while (at()[0] != kNoRule && at()[0] != e.rule) k = (k + 1) & (size - 1);
        if (at()[0] == kNoRule) { at()[0] = e.rule; at()[1] = number(e); }
    }
    return s;
}

namespace {
inline bool has(const std::vector<ChartItem>& v, ChartItem it) {
    for (auto& x : v) if (x.sid == it.sid && x.origin == it.origin) return true;
    return false;
}
}  // namespace

// Predictor and completer until nothing new.  A predicted rule that can derive the empty string
// also advances the predicting item at once, so completions with origin == index need no lookup.
void EarleyChart::close(ChartSet& set, int32_t index, std::vector<ChartItem>& pending) {
    while (!pending.empty()) {
        ChartItem it = pending.back();
        pending.pop_back();
        const StateInfo& si = t_->state_info[it.sid];
        uint32_t nb = si.counts & 0xFFFF, nr = si.counts >> 16;
        bool in_scan = nb > 0 || nr == 0, in_wait = nr > 0;
        if (in_scan) { if (has(set.scan, it)) continue; set.scan.push_back(it); }
        if (in_wait) { if (has(set.wait, it)) continue; set.wait.push_back(it); }
        for (uint32_t k = 0; k < nr; ++k) {
            const RefEdgeP& e = t_->ref_edges[si.ref_off + k];
            pending.push_back({t_->rule_info[e.rule].start, index});
            if (t_->rule_info[e.rule].nullable) pending.push_back({e.tgt, it.origin});
        }
        if (si.rule_final & 0x80000000u) {
            uint32_t rule = si.rule_final & 0x7FFFFFFFu;
            if (it.origin < 0) set.root_done = true;
            else if (it.origin != index)
                for (const ChartItem& w : chart_[(size_t)it.origin].wait) {
                    const StateInfo& wi = t_->state_info[w.sid];
                    for (uint32_t k = 0; k < (wi.counts >> 16); ++k) {
                        const RefEdgeP& e = t_->ref_edges[wi.ref_off + k];
                        if (e.rule == rule) pending.push_back({e.tgt, w.origin});
                    }
                }
        }
    }
}

void EarleyChart::start(uint32_t sid) {
    chart_.clear();
    chart_.emplace_back();
    std::vector<ChartItem> pending{{sid, -1}};
    close(chart_[0], 0, pending);
}

void EarleyChart::start_pair(uint32_t sid, uint32_t waiter_sid) {
    chart_.clear();
    chart_.emplace_back();
    chart_[0].wait.push_back({waiter_sid, -1});
    chart_.emplace_back();
    std::vector<ChartItem> pending{{sid, 0}};
    close(chart_[1], 1, pending);
}

bool EarleyChart::advance(const uint8_t* bytes, size_t n) {
    size_t keep = chart_.size();
    std::vector<ChartItem> pending;
    for (size_t i = 0; i < n; ++i) {
        uint8_t b = bytes[i];
        pending.clear();
        for (const ChartItem& it : chart_.back().scan) {
            const StateInfo& si = t_->state_info[it.sid];
            for (uint32_t k = 0; k < (si.counts & 0xFFFF); ++k) {
                const ByteEdge& e = t_->byte_edges[si.byte_off + k];
                if (b >= (e.lohi & 0xFF) && b <= ((e.lohi >> 8) & 0xFF)) { pending.push_back({e.tgt, it.origin}); break; }
            }
        }
        chart_.emplace_back();
        close(chart_.back(), (int32_t)chart_.size() - 1, pending);
        if (chart_.back().scan.empty() && chart_.back().wait.empty()) { chart_.resize(keep); return false; }
    }
    return true;
}

bool EarleyChart::context(ScanContext& out) const {
    out.items.clear(); out.wait.clear(); out.wait_off.clear();
    int32_t J = (int32_t)chart_.size() - 1;
    // sets reachable through origins, starting from the current set
    std::vector<int32_t> needed{J}, stack{J};
    std::map<int32_t, uint32_t> local;
    auto reach = [&](int32_t o) {
        if (o >= 0 && !std::binary_search(needed.begin(), needed.end(), o)) {
            needed.insert(std::upper_bound(needed.begin(), needed.end(), o), o);
            stack.push_back(o);
        }
    };
    for (const ChartItem& it : chart_[(size_t)J].scan) reach(it.origin);
    while (!stack.empty()) {
        int32_t s = stack.back(); stack.pop_back();
        for (const ChartItem& w : chart_[(size_t)s].wait) reach(w.origin);
    }
    if (needed.size() > kMaxLocalSets - 64) return false;
    for (size_t k = 0; k < needed.size(); ++k) local[needed[k]] = (uint32_t)k;
    out.H = (uint32_t)needed.size();
    auto loc = [&](int32_t o) { return o < 0 ? kRootOrigin : local.at(o); };
    for (const ChartItem& it : chart_[(size_t)J].scan) out.items.push_back(pack_item(t_->ref(it.sid), loc(it.origin)));
    for (size_t k = 0; k < needed.size(); ++k) {
        out.wait_off.push_back((uint32_t)(out.wait.size() / 2));
        for (const ChartItem& w : chart_[(size_t)needed[k]].wait) push_triples(w, loc(w.origin), out.wait);
    }
    out.wait_off.push_back((uint32_t)(out.wait.size() / 2));
    return true;
}

void EarleyChart::push_triples(const ChartItem& w, uint32_t local_origin, std::vector<uint32_t>& out) const {
    const StateInfo& wi = t_->state_info[w.sid];
    for (uint32_t k = 0; k < (wi.counts >> 16); ++k) {
        const RefEdgeP& e = t_->ref_edges[wi.ref_off + k];
        out.push_back(e.rule);
        out.push_back(pack_item(t_->ref(e.tgt), local_origin));
    }
}

}  // namespace xg2
