// Pinned host blocks handed from owner to owner.  Plain C++: the allocator is
// passed in.
//
// Blocks are for results of a few kilobytes that a kernel or a copy writes many
// times a second.  A block of more than kPinnedBlock bytes goes back to the system
// when it is freed, and no more than kPinnedKept bytes are kept in all, so one
// large hierarchy does not leave locked pages behind.
#pragma once

#include <cstddef>
#include <map>
#include <mutex>
#include <unordered_map>
#include <vector>

namespace pair {

constexpr size_t kPinnedBlock = 64 * 1024;
constexpr size_t kPinnedKept = 4 * 1024 * 1024;

class PinnedPool {
public:
    using Alloc = void* (*)(size_t);      // null: no memory
    using Free = void (*)(void*);
    PinnedPool(Alloc a, Free f) : alloc_(a), free_(f) {}

    // A block of at least `bytes`, or null.
    void* get(size_t bytes) {
        size_t sz = 4096;
        while (sz < bytes) sz <<= 1;
        std::lock_guard<std::mutex> g(mu_);
        void* p = nullptr;
        auto it = free_blocks_.find(sz);
        if (it != free_blocks_.end()) {
            p = it->second;
            free_blocks_.erase(it);
            kept_ -= sz;
        } else if (!(p = alloc_(sz))) {
            return nullptr;
        }
        live_[p] = sz;
        return p;
    }

    void put(void* p) {
        {
            std::lock_guard<std::mutex> g(mu_);
            auto it = live_.find(p);
            if (it == live_.end()) return;
            const size_t sz = it->second;
            live_.erase(it);
            if (sz <= kPinnedBlock && kept_ + sz <= kPinnedKept) {
                free_blocks_.emplace(sz, p);
                kept_ += sz;
                return;
            }
        }
        free_(p);
    }

    // Gives every kept block back.
    void release() {
        std::vector<void*> all;
        {
            std::lock_guard<std::mutex> g(mu_);
            for (auto& kv : free_blocks_) all.push_back(kv.second);
            free_blocks_.clear();
            kept_ = 0;
        }
        for (void* p : all) free_(p);
    }

    size_t kept() {
        std::lock_guard<std::mutex> g(mu_);
        return kept_;
    }

private:
    Alloc alloc_;
    Free free_;
    std::mutex mu_;
    std::multimap<size_t, void*> free_blocks_;     // size -> block
    std::unordered_map<void*, size_t> live_;
    size_t kept_ = 0;
};

}  // namespace pair
