// Sizes of the few-frames path (few.hip), as host arithmetic.
#pragma once

#include <algorithm>
#include <cstdint>

namespace ldpc {

// Words that the first launch sets: the channel values [n][W] and, with early
// stop, an unsatisfied mark per frame and iteration.  max_iter has no upper bound,
// so max_iter x W takes 64 bits (2^26 iterations of 32 frames pass 2^31).
struct FewInit {
    int64_t unsat_words, words;
    uint32_t blocks;  // of 256 threads, which stride over the words
};
inline FewInit few_init(int32_t n, int32_t W, int32_t max_iter, bool early_stop)
{
    constexpr int64_t kMostBlocks = 1 << 20;
    FewInit s;
    s.unsat_words = early_stop ? static_cast<int64_t>(max_iter) * W : 0;
    s.words = std::max<int64_t>(static_cast<int64_t>(n) * W, s.unsat_words);
    s.blocks = static_cast<uint32_t>(std::min<int64_t>((s.words + 255) / 256, kMostBlocks));
    return s;
}

}  // namespace ldpc
