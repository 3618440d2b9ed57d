// Device blocks kept between the pools and caches of a vocabulary.  What touches the device goes through Memory, so that the
// rules of keeping and handing out can be run on the host.
#pragma once
#include <algorithm>
#include <cstddef>
#include <cstdint>
#include <mutex>
#include <new>
#include <vector>

namespace xg2 {

struct NoDeviceMemory : std::bad_alloc { const char* what() const noexcept override { return "device memory could not be allocated"; } };

// A request's planes and tables come and go, and allocating and freeing them in the driver costs 50 - 350 us a block (it maps
// and unmaps the memory), as much as building the planes of a small grammar.  Bounded (kMaxSpare bytes are kept, the rest is
// freed); what is kept goes back to the driver with the vocabulary that owns the list, or when an allocation fails, of this
// list or of anything else that asks through allocate().
// Work in flight may still use a block that is handed in, so it is handed out again only after a wait for its device, which is
// what freeing it would have done; where the wait fails (another thread is capturing a stream), the block is held until one
// succeeds.
//
// Memory: int device() (the current one), void* alloc(size_t) on it (null: none left), bool free(void*) (waits for the
// block's device, as hipFree does; false: the block is still allocated), bool wait(int device) (false: work may be in flight).
template <class Memory>
class BlockListOf {
  public:
    struct Block { void* p = nullptr; size_t n = 0; int device = 0; };
    static constexpr size_t kMaxSpare = (size_t)1 << 30;

    explicit BlockListOf(Memory mem = Memory()) : mem_(mem) {
        std::lock_guard<std::mutex> lk(lists().mu);
        lists().all.push_back(this);
    }
    BlockListOf(const BlockListOf&) = delete;
    BlockListOf& operator=(const BlockListOf&) = delete;
    ~BlockListOf() {
        {
            std::lock_guard<std::mutex> lk(lists().mu);
            lists().all.erase(std::find(lists().all.begin(), lists().all.end(), this));
        }
        drop_all();
    }

    // n bytes of device memory that no list looks after; what the lists keep spare makes room for them
    static void* allocate(Memory mem, size_t n) {
        void* p = mem.alloc(n);
        if (!p) {
            {
                std::lock_guard<std::mutex> lk(lists().mu);
                for (BlockListOf* list : lists().all) list->drop_all();
            }
            p = mem.alloc(n);
            if (!p) throw NoDeviceMemory();
        }
        return p;
    }

    // a block of n to `most` bytes, contents unspecified (Block::n: what it really holds); throws NoDeviceMemory
    Block get(size_t n, size_t most = ~(size_t)0) {
        n = std::max(n, std::min(most, (n + 0xFFFF) & ~(size_t)0xFFFF));
        Block b;
        b.device = mem_.device();
        if (take(n, most, b) || (release_held() && take(n, most, b))) return b;
        b.p = allocate(mem_, n);
        b.n = n;
        return b;
    }
    void put(const Block& b) {
        bool room;
        { std::lock_guard<std::mutex> lk(mu_); room = kept_bytes_ + b.n <= kMaxSpare; }
        if (!room && mem_.free(b.p)) return;
        const bool idle = mem_.wait(b.device);
        std::lock_guard<std::mutex> lk(mu_);
        kept_bytes_ += b.n;
        (idle ? spare_ : held_).push_back(b);
    }
    size_t spare_blocks() { std::lock_guard<std::mutex> lk(mu_); return spare_.size(); }
    size_t held_blocks() { std::lock_guard<std::mutex> lk(mu_); return held_.size(); }

  private:
    struct Lists { std::mutex mu; std::vector<BlockListOf*> all; };
    static Lists& lists() { static Lists* l = new Lists(); return *l; }      // of the process, until it ends

    Memory mem_;
    std::mutex mu_;                                  // not held while the device is waited for
    std::vector<Block> spare_, held_;                // nothing in flight uses them; work in flight may
    size_t kept_bytes_ = 0;                          // of both

    bool take(size_t n, size_t most, Block& b) {
        std::lock_guard<std::mutex> lk(mu_);
        most = std::min(most, 2 * n + ((size_t)1 << 20));
        size_t best = spare_.size();
        for (size_t k = 0; k < spare_.size(); ++k)                  // the smallest that fits, unless it is far too large
            if (spare_[k].device == b.device && spare_[k].n >= n && spare_[k].n <= most && (best == spare_.size() || spare_[k].n < spare_[best].n)) best = k;
        if (best == spare_.size()) return false;
        b = spare_[best];
        kept_bytes_ -= b.n;
        spare_[best] = spare_.back();
        spare_.pop_back();
        return true;
    }
    bool release_held() {                            // whether any of the held blocks is free to use now
        std::vector<Block> held;
        { std::lock_guard<std::mutex> lk(mu_); held.swap(held_); }
        bool any = false;
        for (const Block& b : held) {
            const bool idle = mem_.wait(b.device);
            any |= idle;
            std::lock_guard<std::mutex> lk(mu_);
            (idle ? spare_ : held_).push_back(b);
        }
        return any;
    }
    void drop_all() {
        std::vector<Block> all;
        {
            std::lock_guard<std::mutex> lk(mu_);
            all.swap(spare_);
            all.insert(all.end(), held_.begin(), held_.end());
            held_.clear();
        }
        for (const Block& b : all) {
            const bool freed = mem_.free(b.p);
            std::lock_guard<std::mutex> lk(mu_);
            if (freed) kept_bytes_ -= b.n;
            else held_.push_back(b);
        }
    }
};

// The memory a pool's rows lie in: slabs from the list, together never more than max_bytes (0: no bound).
template <class List>
struct SlabsOf {
    size_t max_bytes = 0;
    std::vector<typename List::Block> blocks;
    uint8_t* cur = nullptr; size_t left = 0;         // the part of the latest slab that no row has yet
    size_t device_bytes = 0;                         // of all slabs, as large as they really are

    // a new slab with room for a row at least, sized by the rows the caller is about to ask for; false: max_bytes is reached
    bool add(List& list, size_t row_bytes, size_t rows_ahead) {
        const size_t room = max_bytes ? max_bytes - device_bytes : ~(size_t)0;
        size_t want = std::min<size_t>(std::max<size_t>({row_bytes * 64, (size_t)8 << 20, rows_ahead * row_bytes}), (size_t)256 << 20);
        want = std::max(want, row_bytes);
        if (want > room) want = row_bytes * 16;
        if (want > room) want = row_bytes;
        if (want > room) return false;
        const typename List::Block b = list.get(want, room);
        blocks.push_back(b);
        cur = static_cast<uint8_t*>(b.p); left = b.n; device_bytes += b.n;
        return true;
    }
};

}  // namespace xg2
