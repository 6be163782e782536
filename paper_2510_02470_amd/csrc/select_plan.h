// Sizes of the top-m selection (select.hip) and of its work space.
//
// The last two kernels take the keys in blocks. Blocks of 4096 keys; four times as long where every work-group would read the
// counts, and with many equal scores the tables, of more than 1024 blocks before it (16 million keys of seven values, waiting
// included: 166 us with short blocks, 111 with long ones; 2 million distinct keys 37.3 with short ones, 42.8 with long ones).
// A block has a table of 2 KB, so the work space is counted in the blocks that a call uses: 2.1 MB up to 16.7 million keys (8.4
// if every 4096 of them had a table).
#pragma once
#include <stddef.h>
#include <stdint.h>

namespace sage {

constexpr int TOPM_HIST_WORDS = 4096 + 2 * 1024;
constexpr int SELECT_BLOCK = 4096;                // keys of a short block
constexpr int SELECT_LONG = 4 * SELECT_BLOCK;     // ... of a long one
constexpr int64_t SELECT_SHORT_MAX = 1024;        // short blocks up to this many
constexpr int SELECT_STATE_WORDS = 64;            // a 256-byte slot of its own
constexpr int SELECT_BLOCK_WORDS = 2 + 1024 / 2;  // counters and table of a block

constexpr bool topm_long(int64_t N) { return N > SELECT_SHORT_MAX * SELECT_BLOCK; }
// blocks of a call for N keys
constexpr int64_t topm_blocks(int64_t N) {
    const int64_t b = topm_long(N) ? SELECT_LONG : SELECT_BLOCK;
    return N > 0 ? (N + b - 1) / b : 1;
}
// the most that a call for N keys or fewer has
constexpr int64_t topm_work_blocks(int64_t N) {
    return !topm_long(N) || topm_blocks(N) > SELECT_SHORT_MAX ? topm_blocks(N) : SELECT_SHORT_MAX;
}
// words of a work space for them
constexpr size_t topm_work_words(int64_t blocks) {
    return (size_t)TOPM_HIST_WORDS + SELECT_STATE_WORDS + (size_t)SELECT_BLOCK_WORDS * (size_t)blocks;
}

}  // namespace sage
