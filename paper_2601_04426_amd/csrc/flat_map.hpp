// A hash table in one array (linear probing, deletion by shifting back): what the compile path looks up per plane.
#pragma once
#include <cstddef>
#include <cstdint>
#include <utility>
#include <vector>

namespace xg2 {

// Key: equality-comparable, default-constructible; Hash: Key -> uint64_t with well-mixed low bits.
template <class Key, class Value, class Hash>
class FlatMap {
    struct Slot { Key key; Value value; bool used = false; };
    std::vector<Slot> slot_;
    size_t used_ = 0;
    size_t mask() const { return slot_.size() - 1; }
    size_t home(const Key& k) const { return (size_t)Hash()(k) & mask(); }
    void grow() {
        std::vector<Slot> old(slot_.empty() ? 64 : slot_.size() * 2);
        old.swap(slot_);
        for (Slot& s : old)
            if (s.used) {
                size_t at = home(s.key);
                while (slot_[at].used) at = (at + 1) & mask();
                slot_[at] = std::move(s);
            }
    }

  public:
    size_t size() const { return used_; }
    Value* find(const Key& k) {
        if (slot_.empty()) return nullptr;
        for (size_t at = home(k); slot_[at].used; at = (at + 1) & mask())
            if (slot_[at].key == k) return &slot_[at].value;
        return nullptr;
    }
    // the value under k and whether it was entered by this call (v is ignored if k is there already)
    std::pair<Value*, bool> emplace(const Key& k, Value v) {
        if ((used_ + 1) * 2 > slot_.size()) grow();
        size_t at = home(k);
        for (; slot_[at].used; at = (at + 1) & mask())
            if (slot_[at].key == k) return {&slot_[at].value, false};
        slot_[at].key = k; slot_[at].value = std::move(v); slot_[at].used = true;
        ++used_;
        return {&slot_[at].value, true};
    }
    void erase(const Key& k) {
        if (slot_.empty()) return;
        size_t at = home(k);
        while (slot_[at].used && !(slot_[at].key == k)) at = (at + 1) & mask();
        if (!slot_[at].used) return;
        for (size_t next = (at + 1) & mask(); slot_[next].used; next = (next + 1) & mask()) {
            // the entry at `next` may move to the hole unless its home lies after the hole
            if (((next - home(slot_[next].key)) & mask()) >= ((next - at) & mask())) { slot_[at] = std::move(slot_[next]); at = next; }
        }
        slot_[at] = Slot();
        --used_;
    }
};

}  // namespace xg2
