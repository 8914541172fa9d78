// How a sequence's keys are cut into splits, plain C++ (the launchers' host code; a test compiles it by itself).
#pragma once

namespace poss {

constexpr int ATTN_MAX_BPS = 64;                         // blocks per split the kernels can address (one page-table entry per lane)
constexpr int ATTN_MAX_SPLITS = 256;
constexpr int ATTN_MAX_REGION = 128;                     // slots behind the prefix that a pass sees at most (a row's mask)

// Blocks of 32 keys per split.  A workgroup walks its blocks one after the other, each a dependent trip
// to memory, so a short context is still cut into about four pieces of >= 4 blocks (the merge kernel
// costs less than the serial walk it replaces); long contexts walk 32 blocks per workgroup.  The rule looks at the committed
// prefix only, never at the number of rows or the size of the tree region: a row's arithmetic (which keys
// meet in which split, in which order) is then the same whether it is verified alone or among 60 others,
// which is what makes the speculative stream reproduce the one-token-at-a-time stream bit for bit as long
// as only bonus tokens are committed.  keys_per_split > 0 overrides.
// keys_per_split < 0: the rule above with splits of at most -keys_per_split keys (the specialists' passes carry few
// rows, so that only a few dozen workgroups exist per split level: at long contexts they want shorter walks than the
// target's passes; the drafter's caches are its own, so its rule need not match the target's).
// At most ATTN_MAX_SPLITS splits, whatever the region (small splits on a very long context are doubled until they are that few);
// ATTN_MAX_SPLITS of ATTN_MAX_BPS blocks are 524288 keys, more than a context can hold.
static inline int attn_blocks_per_split(int n_prefix, int keys_per_split) {
    const int n_blocks = (n_prefix + ATTN_MAX_REGION + 31) / 32;
    int bps;
    if (keys_per_split > 0) {
        bps = keys_per_split >= 32 ? keys_per_split / 32 : 1;
    } else {
        bps = ((n_prefix + 31) / 32 + 3) / 4;
        if (bps < 4) bps = 4;
        const int cap = keys_per_split < 0 && -keys_per_split >= 128 ? -keys_per_split / 32 : 32;
        if (bps > cap) bps = cap;
    }
    while (bps < ATTN_MAX_BPS && (n_blocks + bps - 1) / bps > ATTN_MAX_SPLITS) bps *= 2;
    return bps < ATTN_MAX_BPS ? bps : ATTN_MAX_BPS;
}

}  // namespace poss
