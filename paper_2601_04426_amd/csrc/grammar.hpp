// Host-side grammar lowering: EBNF text -> one canonical minimal byte-level automaton per rule
// (XGrammar-2 section 3.3: "structures are represented as multiple FSMs", edges are character
// ranges or references to other FSMs), plus the structural hashes of Algorithm 1 / Algorithm 2.
#pragma once
#include <cstdint>
#include <functional>
#include <memory>
#include <stdexcept>
#include <string>
#include <vector>

namespace xg2 {

struct ParseError : std::runtime_error { using std::runtime_error::runtime_error; };
struct GrammarError : std::runtime_error { using std::runtime_error::runtime_error; };

struct ByteRange { uint8_t lo, hi; int32_t tgt; };   // bytes lo..hi -> rule-local state tgt
struct RefEdge { int32_t rule; int32_t tgt; };       // reference to Grammar::rules[rule] -> state tgt

// Rows of T back to back: row i is v[off[i] .. off[i + 1]).  The automata of a grammar are thousands of short edge lists;
// kept this way a rule costs two allocations instead of one per state, and copying or dropping one is a block copy.
template <class T>
struct Span {
    const T* b; const T* e;
    const T* begin() const { return b; }
    const T* end() const { return e; }
    size_t size() const { return (size_t)(e - b); }
    bool empty() const { return b == e; }
    const T& operator[](size_t k) const { return b[k]; }
};
template <class T>
struct Rows {
    std::vector<uint32_t> off{0};
    std::vector<T> v;
    Span<T> operator[](size_t i) const { return {v.data() + off[i], v.data() + off[i + 1]}; }
    size_t size() const { return off.size() - 1; }
    void end_row() { off.push_back((uint32_t)v.size()); }
};

// The minimal automaton of a rule body, apart from the grammar it stands in: references are written as their rank among
// the body's references by declaration index.  Immutable and shared by every grammar that holds the same body.
struct RuleBody {
    std::vector<uint8_t> is_final;                    // [n_states]
    Rows<ByteRange> bedges;                           // sorted by lo; maximal runs per target
    Rows<RefEdge> redges;                             // sorted by rank
    bool single_refs = true;                          // no state has more than one reference
};

struct RuleFsm {
    std::string name;
    int32_t decl_index = 0;                           // position of the rule in the EBNF text
    std::shared_ptr<const RuleBody> body;
    Rows<RefEdge> redges;                             // sorted by referenced rule's decl_index
    bool nullable = false;
    int32_t min_len = 0;                              // length of the rule's shortest sentence, in bytes
    std::vector<int32_t> min_suf;                     // [state]: bytes of the shortest completion of the rule from the state
    // structural hash (Algorithm 1, refined by Algorithm 2 inside simple reference cycles)
    uint64_t hash = 0;
    bool shareable = true;                            // false: member of a non-simple cycle, never reused
    std::vector<int32_t> canon_id, by_canon;          // Algorithm 1 phase 1: state -> canonical id, and back
    Rows<RefEdge> redges_by_hash;                     // out-references in the order Algorithm 1 sorted them
    std::vector<int32_t> ring;                        // simple cycle through this rule, starting at it (else empty)
    int32_t n_states() const { return (int32_t)body->is_final.size(); }
    bool is_final(int q) const { return body->is_final[(size_t)q] != 0; }
    Span<ByteRange> bedges(int q) const { return body->bedges[(size_t)q]; }
    Span<RefEdge> refs(int q) const { return redges[(size_t)q]; }
};

struct Position { int32_t rule, state, sid; };

struct Grammar {
    std::vector<RuleFsm> rules;                       // rules reachable from the root, in declaration order
    int32_t root = 0;
    std::vector<int32_t> state_base;                  // global state id = state_base[rule] + state
    int32_t n_states = 0;
    std::vector<Position> positions;                  // states with at least one byte edge
    std::vector<int32_t> sid_to_pos;                  // [n_states] -> index into positions or -1
    std::vector<std::vector<int32_t>> hash_order;     // reference-graph components, referenced rules first
    int32_t sid(int32_t rule, int32_t state) const { return state_base[rule] + state; }
};

// Throws ParseError (syntax) or GrammarError (undefined rule, empty language, unproductive rule,
// ill-formed TagDispatch).
Grammar lower_grammar(const std::string& ebnf, const std::string& root_rule);

std::string describe_grammar(const Grammar& g);       // JSON

uint64_t hash_combine(uint64_t h, uint64_t v);        // the order-sensitive hash of Algorithms 1 and 2

// States of one rule that no string of at most `budget` bytes can tell apart (bounded bisimulation):
// returns, per state, the member of the state's class with the smallest canonical id.
// Rule edges are compared by ref_identity[rule] (rules known to be identical may share an identity).
// This is what makes planes independent of the bounds of a long repetition (section 3.6 observes
// that the states inside a repetition differ minimally): tokens are at most `budget` bytes long, so
// equivalent states have equal planes.
// The result depends only on the rule's structure and on the identities (and through them the
// shortest sentence and nullability) of the rules it references.
// near (optional): for the representative x of a class, near->base[x] is the representative of another class of the
// same rule that no string of at most near->depth[x] bytes tells apart from x (-1: none worth using), so the plane of
// x equals the plane of base[x] on every token of at most depth[x] bytes and only the longer tokens need checking.
// Bases are never derived themselves.
struct NearClasses { std::vector<int32_t> base, depth; };
constexpr int32_t kMinNearDepth = 3;       // shorter agreements save too few tokens to be worth a second pass
constexpr int32_t kMaxNearDepth = 32;
std::vector<int32_t> bounded_classes_rule(const Grammar& g, int32_t rule, int32_t budget, const std::vector<uint64_t>& ref_identity,
                                          NearClasses* near = nullptr);

// Exact numbering of descriptions: a list of words gets the number it got before, a list not met yet the next one (from 1).
// Nearly all lists have three words (a state with one byte run): those lie in the open-addressing table itself, so that a
// look-up is one cache line; longer ones lie back to back in one array behind a table of their own.
class NodeTable {
  public:
    uint32_t intern3(uint32_t a, uint32_t b, uint32_t c);
    uint32_t intern(const uint32_t* w, uint32_t n) { return n == 3 ? intern3(w[0], w[1], w[2]) : intern_long(w, n); }
    uint32_t fresh() { return ++count_; }               // a number no list ever gets
    uint32_t size() const { return count_; }

  private:
    struct Three { uint32_t id, a, b, c; };             // id 0: empty slot
    struct Long { uint32_t id, hash, at, n; };          // words_[at .. at + n)
    std::vector<Three> three_;
    std::vector<Long> long_;
    std::vector<uint32_t> words_;
    uint32_t count_ = 0, n_three_ = 0, n_long_ = 0;
    uint32_t intern_long(const uint32_t* w, uint32_t n);
    static uint32_t mix3(uint32_t a, uint32_t b, uint32_t c) {
        uint64_t h = (((uint64_t)a << 32 | b) ^ ((uint64_t)c * 0x9E3779B97F4A7C15ull)) * 0x9FB21C651E98DF25ull;
        return (uint32_t)(h ^ (h >> 32));
    }
};

// What one rule's states do on strings of at most d bytes, for every d up to the longest token, by canonical state number.
// level[d * n + c] is the class of state c among the rule's states: states of one class agree on whether they are final, on
// the byte runs with the classes they lead to on d - 1 bytes, and on the references, by identity, with what follows their
// shortest sentence.  rep and near are what bounded_classes_rule says.
struct RuleAnalysis {
    int32_t n = 0;
    bool acyclic = true;                               // no cycle of references to rules that derive the empty string
    std::vector<int32_t> level;
    std::vector<int32_t> rep;
    NearClasses near;
    // numbers of behaviours in the node table, worked out on demand (FollowSigs): [d * n + class] (by state instead of class
    // if not acyclic), 0 = not known yet.  Belongs to the pool whose table the numbers are from.
    mutable std::vector<uint32_t> number;
    std::vector<uint8_t> on_cycle;                     // [canonical state], if not acyclic: on or before such a cycle
};
// identity[r]: a number that identical rules share and different ones do not, for every rule that `rule` references
RuleAnalysis analyse_rule(const Grammar& g, int32_t rule, int32_t budget, const std::vector<uint64_t>& identity);

// What can follow an instance of a rule within d bytes in this grammar, as a number of the node table: the set of states
// referencing rules continue in (the number of their behaviour on the bytes that are left: equal numbers, equal behaviour,
// across rules and grammars that share the table), recursively through rules that can end within the budget, and whether
// the input may end (root rule).  States on or before a cycle of references to rules that derive the empty string get
// numbers of their own (never shared, always sound).  Two rules with equal numbers reject the same uncertain
// tokens by context expansion (section 2.2), so filtered planes can be shared across grammars (section 3.3: reuse needs
// matching lookahead).  A rule on a reference cycle through rule ends gets a number of its own.  Computed on demand.
class FollowSigs {
  public:
    // analysis[r] and rep[r] (by state number) of every rule; sites are taken at representatives, which leaves the follow
    // language as it is and the work independent of repetition bounds
    FollowSigs(const Grammar& g, int32_t budget, const std::vector<std::shared_ptr<const RuleAnalysis>>& analysis,
               const std::vector<std::vector<int32_t>>& rep, const std::vector<uint64_t>& identity, NodeTable& nodes);
    uint32_t sig(int rule, int d);

  private:
    struct Site { int32_t q, x; };
    const Grammar& g_;
    int32_t budget_;
    const std::vector<std::shared_ptr<const RuleAnalysis>>& analysis_;
    const std::vector<uint64_t>& identity_;
    NodeTable& nodes_;
    uint32_t behaviour(int rule, int c, int d);         // number of canonical state c's behaviour on at most d bytes
    Rows<Site> sites_;
    std::vector<uint32_t> memo_;                        // [rule * (budget + 1) + d]: 0 not known, kPending being computed
    static constexpr uint32_t kPending = 0xFFFFFFFFu;
};

// Exact serialisation of one rule in Algorithm 1's canonical order; a reference to rule r is
// written as ref_id[r].  Two rules with equal text and equal meaning of the ids are isomorphic.
std::string serialise_rule(const Grammar& g, int32_t rule, const std::vector<uint64_t>& ref_id);
constexpr uint64_t kInCycleRef = 0x5EEDF00DCAFEBEEFull;   // the shared placeholder X of Algorithm 2

}  // namespace xg2
