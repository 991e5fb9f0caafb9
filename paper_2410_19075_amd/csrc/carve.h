// Pieces of one allocation, host code only.
#pragma once

#include <cstddef>

namespace nd {

// Lays pieces out one after the other, each at a multiple of kAlign bytes (the base
// is aligned at least as much), so that a piece may be read in any vector width and
// starts on a cache line of its own.  Without a base it only counts: the same
// layout code run first without and then with one gives the size and the pieces.
class Carve {
public:
    static constexpr size_t kAlign = 128;
    explicit Carve(char* base = nullptr) : base_(base) {}

    template <class T>
    T* take(size_t count) {
        static_assert(kAlign % alignof(T) == 0, "piece alignment");
        off_ = (off_ + kAlign - 1) / kAlign * kAlign;
        char* q = base_ ? base_ + off_ : nullptr;
        off_ += count * sizeof(T);
        return reinterpret_cast<T*>(q);
    }
    size_t bytes() const { return off_; }

private:
    char* base_;
    size_t off_ = 0;
};

}  // namespace nd
