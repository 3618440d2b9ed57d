// Test program (CPU only): the list of device blocks kept between requests, over memory that remembers what work may still use.
// Exits with 0 and "ok" if every check holds; built by tests/test_block_list.py with sanitizers.
#include <cstdio>
#include <cstdlib>
#include <map>

#include "../../paper_2601_04426_amd/csrc/block_list.hpp"

using namespace xg2;

#define CHECK(x) do { if (!(x)) { std::printf("%s:%d: %s\n", __FILE__, __LINE__, #x); std::exit(1); } } while (0)

namespace {

struct Device {                                       // what FakeMemory stands for
    int current = 0;
    bool refuses = false;                             // waiting and freeing fail (a capture elsewhere)
    size_t left = (size_t)8 << 30, taken = 0;
    std::map<void*, std::pair<size_t, int>> live;     // allocated blocks: size, device
    std::map<int, int> waits;                         // per device
};
struct FakeMemory {
    Device* d;
    int device() { return d->current; }
    void* alloc(size_t n) {
        if (n > d->left) return nullptr;
        void* p = std::malloc(1);
        d->left -= n; d->taken += n;
        d->live[p] = {n, d->current};
        return p;
    }
    bool free(void* p) {
        CHECK(d->live.count(p));
        if (d->refuses) return false;
        d->left += d->live[p].first; d->taken -= d->live[p].first;
        d->live.erase(p);
        std::free(p);
        return true;
    }
    bool wait(int device) { if (d->refuses) return false; ++d->waits[device]; return true; }
};
using List = BlockListOf<FakeMemory>;

void reuse() {
    Device d;
    {
        List list(FakeMemory{&d});
        const List::Block a = list.get(100000);
        CHECK(a.p && a.n >= 100000 && a.n < 200000);
        list.put(a);
        CHECK(d.waits[0] == 1);
        const List::Block b = list.get(90000);
        CHECK(b.p == a.p && b.n == a.n);
        const List::Block c = list.get(90000);
        CHECK(c.p != b.p);
        list.put(b); list.put(c);
        const List::Block big = list.get((size_t)64 << 20);     // far more than either
        CHECK(big.n >= (size_t)64 << 20);
        const List::Block tiny = list.get(1);
        CHECK(tiny.p == b.p || tiny.p == c.p);
        list.put(big); list.put(tiny);
    }
    CHECK(d.live.empty());
}

// a block whose wait failed may be in use by work in flight: nobody gets it before a wait succeeds
void failed_wait() {
    Device d;
    {
        List list(FakeMemory{&d});
        const List::Block a = list.get(1 << 20);
        d.refuses = true;
        list.put(a);
        CHECK(list.held_blocks() == 1 && list.spare_blocks() == 0);
        const List::Block b = list.get(1 << 20);
        CHECK(b.p && b.p != a.p);
        list.put(b);
        CHECK(list.held_blocks() == 2);
        d.refuses = false;
        const List::Block c = list.get(1 << 20);
        CHECK((c.p == a.p || c.p == b.p) && list.held_blocks() == 0 && list.spare_blocks() == 1);
        list.put(c);
    }
    CHECK(d.live.empty());
}

// blocks stay with their device, and that device is waited for whichever is current
void devices() {
    Device d;
    {
        List list(FakeMemory{&d});
        const List::Block a = list.get(1 << 20);
        d.current = 1;
        list.put(a);
        CHECK(d.waits[0] == 1 && d.waits[1] == 0);
        const List::Block b = list.get(1 << 20);
        CHECK(b.p != a.p && b.device == 1 && d.live[b.p].second == 1);
        d.current = 0;
        CHECK(list.get(1 << 20).p == a.p);
        list.put(a); list.put(b);
    }
    CHECK(d.live.empty());
}

// no more than kMaxSpare is kept, and a full device gets back what is
void bounds() {
    Device d;
    d.left = (size_t)3 << 30;
    {
        List list(FakeMemory{&d});
        std::vector<List::Block> v;
        for (int k = 0; k < 24; ++k) v.push_back(list.get((size_t)100 << 20));
        for (const List::Block& b : v) list.put(b);
        CHECK(d.taken <= List::kMaxSpare && d.taken >= (size_t)900 << 20);
        const List::Block all = list.get((size_t)3 << 30);
        CHECK(all.p && list.spare_blocks() == 0);
        bool none = false;
        try { list.get((size_t)1 << 20); } catch (const NoDeviceMemory&) { none = true; }
        CHECK(none);
        list.put(all);
        d.refuses = true;                             // nor does a block go amiss that can neither be kept nor freed
        const List::Block b = list.get((size_t)2 << 30);
        CHECK(b.p);
        list.put(b);
        CHECK(list.held_blocks() == 1);
        d.refuses = false;
        CHECK(list.get((size_t)2 << 30).p == b.p);
        list.put(b);
    }
    CHECK(d.live.empty());
}

// memory that other buffers need is not kept from them, by this vocabulary's list or another's
void makes_room() {
    Device d;
    d.left = (size_t)1 << 30;
    {
        List one(FakeMemory{&d}), other(FakeMemory{&d});
        const List::Block a = one.get((size_t)400 << 20), b = other.get((size_t)400 << 20);
        one.put(a); other.put(b);
        void* p = List::allocate(FakeMemory{&d}, (size_t)900 << 20);
        CHECK(p && one.spare_blocks() == 0 && other.spare_blocks() == 0);
        bool none = false;
        try { other.get((size_t)400 << 20); } catch (const NoDeviceMemory&) { none = true; }
        CHECK(none);
        CHECK(FakeMemory{&d}.free(p));
        one.put(one.get((size_t)800 << 20));
        other.put(other.get((size_t)800 << 20));     // from the other list's spare memory
    }
    CHECK(d.live.empty());
}

// a pool with a bound takes no more than that from the list, whatever sizes the list has to spare, and counts what it takes
void bounded_pool() {
    Device d;
    {
        List list(FakeMemory{&d});
        const size_t row = 57040;
        for (size_t max_bytes : {row, 3 * row, 10 * row, (size_t)1 << 20, (size_t)5 << 20, (size_t)9 << 20, (size_t)40 << 20, (size_t)0}) {
            std::vector<List::Block> spare;           // as the tables and planes of earlier requests leave them
            for (size_t n : {(size_t)100 << 10, (size_t)900 << 10, (size_t)1100 << 10, (size_t)9 << 20, (size_t)12 << 20, (size_t)70 << 20}) spare.push_back(list.get(n));
            for (const List::Block& b : spare) list.put(b);
            SlabsOf<List> pool;
            pool.max_bytes = max_bytes;
            size_t rows = 0, want = max_bytes ? max_bytes / row : 2000;
            for (;; ++rows) {
                if (pool.left < row && (rows == 2000 || !pool.add(list, row, want > rows ? want - rows : 1))) break;
                pool.cur += row; pool.left -= row;
                size_t taken = 0;
                for (const List::Block& b : pool.blocks) taken += d.live[b.p].first;
                CHECK(taken == pool.device_bytes && (!max_bytes || taken <= max_bytes));
            }
            CHECK(rows >= 1 && pool.device_bytes - rows * row < (pool.blocks.size() + 1) * row);   // and nothing of a slab is left unused but its remainder
            for (const List::Block& b : pool.blocks) list.put(b);
        }
    }
    CHECK(d.live.empty());
}

}  // namespace

int main() {
    reuse();
    failed_wait();
    devices();
    bounds();
    makes_room();
    bounded_pool();
    std::puts("ok");
    return 0;
}
