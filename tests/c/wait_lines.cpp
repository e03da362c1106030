// The lines that waited extracts take: one page serves any number of threads
// that wait one after another, concurrent calls hold lines of their own, and a
// failed allocation hands out nothing.  Prints "ok".
#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <set>
#include <thread>
#include <vector>

#include "../../paper_0912_0947_amd/csrc/lsb_wait_lines.hpp"

static std::atomic<int> pages{0};
static void *page(size_t bytes) {
    ++pages;
    return aligned_alloc(4096, bytes);
}

#define CHECK(x) \
    if (!(x)) return std::printf("failed: %s (line %d)\n", #x, __LINE__), 1

int main() {
    lsb::WaitLines lines;
    CHECK(lines.take([](size_t) -> void * { return nullptr; }) == nullptr);
    for (int i = 0; i < 500; ++i)
        std::thread([&] { lines.give(lines.take(page)); }).join();
    CHECK(pages == 1);
    std::set<lsb::WaitLine *> held;
    for (int i = 0; i < 33; ++i) held.insert(lines.take(page));
    CHECK(held.size() == 33 && pages == 2);
    for (auto *l : held) lines.give(l);
    std::atomic<int> shared{0};
    std::vector<std::thread> threads;
    for (int t = 0; t < 8; ++t)
        threads.emplace_back([&, t] {
            for (int i = 0; i < 2000; ++i) {
                lsb::WaitLine *l = lines.take(page);
                l->len = (uint32_t)t;
                std::this_thread::yield();
                if (l->len != (uint32_t)t) ++shared;
                lines.give(l);
            }
        });
    for (auto &t : threads) t.join();
    CHECK(shared == 0 && pages == 2);
    std::printf("ok\n");
    return 0;
}
