// The pool of result slots (host_slots.hpp) with an allocator that counts: exit status 0 if it behaves.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <set>
#include <thread>
#include <vector>

#include "../paper_1803_00437_amd/csrc/host_slots.hpp"

using fdlbm::HostSlots;

static int allocs = 0;
static double *counted(size_t bytes)
{
    ++allocs;
    return static_cast<double *>(std::calloc(1, bytes));
}
static double *refused(size_t)
{
    ++allocs;
    return nullptr;
}
#define CHECK(x)                                          \
    if (!(x)) {                                           \
        std::printf("line %d: %s\n", __LINE__, #x);       \
        return 1;                                         \
    }

int main()
{
    {  // contexts one after the other, six reads each: one page in all, at the twentieth read
        HostSlots pool(8, counted);
        int reads = 0;
        for (int c = 0; c < 10; ++c) {
            double *slot = nullptr;
            for (int r = 0; r < 6; ++r) {
                if (!slot) slot = pool.take();
                ++reads;
                CHECK((slot != nullptr) == (reads >= HostSlots::FIRST_READS));
            }
            pool.give(slot);
            CHECK(allocs == (reads >= HostSlots::FIRST_READS ? 1 : 0));
        }
    }
    {  // slots are distinct, bounded, and given back
        HostSlots pool(8, counted);
        for (int r = 1; r < HostSlots::FIRST_READS; ++r) CHECK(pool.take() == nullptr);
        std::vector<double *> s;
        for (int c = 0; c < HostSlots::SLOTS; ++c) s.push_back(pool.take());
        CHECK(std::set<double *>(s.begin(), s.end()).size() == size_t(HostSlots::SLOTS) && !std::set<double *>(s.begin(), s.end()).count(nullptr));
        for (double *a : s) CHECK(a >= s[0] && a + 8 <= s[0] + 8 * HostSlots::SLOTS);
        CHECK(pool.take() == nullptr);
        pool.give(s[17]);
        CHECK(pool.take() == s[17]);
    }
    {  // no page to be had: asked for once
        allocs = 0;
        HostSlots pool(8, refused);
        for (int r = 0; r < 100; ++r) CHECK(pool.take() == nullptr);
        CHECK(allocs == 1);
    }
    {  // threads
        allocs = 0;
        HostSlots pool(8, counted);
        std::vector<std::thread> t;
        for (int i = 0; i < 8; ++i)
            t.emplace_back([&pool, i] {
                for (int c = 0; c < 2000; ++c) {
                    double *slot = pool.take();
                    if (!slot) continue;
                    slot[0] = i;
                    if (slot[0] != i) std::abort();
                    pool.give(slot);
                }
            });
        for (auto &x : t) x.join();
        CHECK(allocs == 1);
    }
    return 0;
}
