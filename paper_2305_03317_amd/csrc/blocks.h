// Device arrays carved from few allocations.
#pragma once

#include <utility>
#include <vector>

#include "common.h"

namespace sp {

// Freed with the object unless given to someone who keeps them.  An allocation
// of under 2 MB takes 1 us, a larger one 250 to 490 (3 MB in one 284, in three of
// 1 MB 4): arrays below that share blocks that stay below it, the others one block.
struct DevBlocks {
    static constexpr size_t kLess = 2000 << 10;

    // An array of count T for *p.  beside: right behind the array before it.
    template <class T>
    void add(T **p, size_t count, bool beside = false) {
        parts_.push_back({(void **)p, (sizeof(T) * count + 255) & ~(size_t)255, beside});
    }

    sp_status alloc() {
        struct Block {
            size_t used;
            bool small;
        };
        std::vector<Block> plan;
        std::vector<std::pair<size_t, size_t>> place;  // block, offset
        for (size_t i = 0; i < parts_.size(); ++i) {
            size_t b = parts_[i].beside ? place.back().first : plan.size();
            if (!parts_[i].beside) {
                size_t need = parts_[i].bytes;
                for (size_t j = i + 1; j < parts_.size() && parts_[j].beside; ++j) need += parts_[j].bytes;
                const bool small = need <= kLess;
                for (size_t j = 0; j < plan.size(); ++j)
                    if (plan[j].small == small && (!small || plan[j].used + need <= kLess)) b = j;
                if (b == plan.size()) plan.push_back({0, small});
            }
            place.emplace_back(b, plan[b].used);
            plan[b].used += parts_[i].bytes;
        }
        blocks_.assign(plan.size(), nullptr);
        for (size_t b = 0; b < plan.size(); ++b) {
            SP_TRY(dev_alloc(&blocks_[b], plan[b].used));
            bytes_ += plan[b].used;
        }
        for (size_t i = 0; i < parts_.size(); ++i)
            *parts_[i].at = (char *)blocks_[place[i].first] + place[i].second;
        return SP_OK;
    }

    // Hands the blocks over; returns their bytes.
    size_t give_to(std::vector<void *> &keeper) {
        keeper.insert(keeper.end(), blocks_.begin(), blocks_.end());
        blocks_.clear();
        return bytes_;
    }

    DevBlocks() = default;
    DevBlocks(const DevBlocks &) = delete;
    DevBlocks &operator=(const DevBlocks &) = delete;
    ~DevBlocks() {
        for (void *b : blocks_) dev_free(b);
    }

  private:
    struct Part {
        void **at;
        size_t bytes;
        bool beside;
    };
    std::vector<Part> parts_;
    std::vector<void *> blocks_;
    size_t bytes_ = 0;
};

}  // namespace sp
