// jk_guard.h -- no C++ exception leaves the C entry points.
#pragma once
#include <exception>

// The body's status, or that of out_of_memory() where the body throws (the
// library itself throws nothing: host memory has run out).
template <typename F, typename G>
int guarded(F &&body, G &&out_of_memory) noexcept {
    try {
        return body();
    } catch (const std::exception &) {
        return out_of_memory();
    }
}
