// How a step shared over workgroups is cut into chunks (host and device).
#pragma once
#include <stdint.h>

namespace sgm {

// A step has at most this many chunks; unsuccessful claims raise the next
// field of its claim word past the chunk count by at most one per workgroup
// of the launch, so it never reaches the 20-bit chunk field.
constexpr int32_t kMaxChunks = 1 << 19;

constexpr int32_t chunk_count(int32_t n, int32_t items) { return n / items + (n % items != 0); }

// Items per chunk of a step over n items: an even share for the owner and its
// helpers within [lo, hi], and more than hi only where the step would have
// too many chunks (a root step's range is bounded by the graph's vertices
// alone).
constexpr int32_t chunk_items(int32_t n, int32_t helpers, int32_t lo, int32_t hi) {
    const int32_t even = chunk_count(n, helpers + 1), least = chunk_count(n, kMaxChunks);
    const int32_t k = even < lo ? lo : even > hi ? hi : even;
    return k < least ? least : k;
}

}  // namespace sgm
