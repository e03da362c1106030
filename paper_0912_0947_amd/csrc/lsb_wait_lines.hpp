// lsb_wait_lines.hpp -- result words of waited extracts: cache lines of pinned
// host memory that calls take and give back.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <mutex>

namespace lsb {

struct WaitLine {
    uint32_t len;
    int32_t status;
    WaitLine *next;
    uint8_t pad[112];
};
static_assert(sizeof(WaitLine) == 128, "one cache line each");

// A call takes a line and gives it back after its wait, so there are as many
// lines as calls have waited at once, whatever threads came and went (a line
// per thread would stay allocated for every thread that ever waited).  Lines
// come from pages of 32; nothing is freed before the process ends.
class WaitLines {
   public:
    static constexpr int kPerPage = 32;

    // A free line; `alloc(bytes)` brings a page, or null (then so is the line).
    template <typename Alloc>
    WaitLine *take(Alloc alloc) {
        std::lock_guard<std::mutex> g(mu_);
        if (!free_) {
            WaitLine *page = static_cast<WaitLine *>(alloc(kPerPage * sizeof(WaitLine)));
            if (!page) return nullptr;
            for (int i = 0; i < kPerPage; ++i) page[i].next = i + 1 < kPerPage ? page + i + 1 : nullptr;
            free_ = page;
        }
        WaitLine *line = free_;
        free_ = line->next;
        return line;
    }

    void give(WaitLine *line) {
        std::lock_guard<std::mutex> g(mu_);
        line->next = free_;
        free_ = line;
    }

   private:
    std::mutex mu_;
    WaitLine *free_ = nullptr;
};

}  // namespace lsb
