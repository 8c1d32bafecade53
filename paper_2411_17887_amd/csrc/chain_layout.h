// What a workspace holds for a carry chain, and the tiles whose chains callers size it by.  Shared by the sources that check a
// workspace (tcuscan.hip asserts that its structures agree).
#ifndef TCUSCAN_CHAIN_LAYOUT_H
#define TCUSCAN_CHAIN_LAYOUT_H

#include <stddef.h>

namespace chain_layout {

constexpr size_t kHeaderBytes = 256;       // fault word, ticket counter
constexpr size_t kSlotBytes = 64;          // one status word per tile, alone in its slot
constexpr size_t kSmallTile = 8192;        // elements of the small workgroup tile, all input types
constexpr size_t kFlagTile = 16384;        // keys or mask entries of a workgroup of the fused split and compaction kernels

// Bytes for the chain of n elements in tiles of `tile` (none for one tile).
constexpr size_t bytes_for(size_t n, size_t tile) { return n > tile ? kHeaderBytes + kSlotBytes * ((n + tile - 1) / tile) : 0; }

}  // namespace chain_layout

#endif
