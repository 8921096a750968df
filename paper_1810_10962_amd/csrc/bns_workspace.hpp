// Where things lie in a workspace.  Plain C++ without HIP headers, so that a host compiler can check it alone.
#pragma once
#include <stddef.h>

namespace bns {

constexpr size_t kHeaderBytes = 256;        // in front of everything else: bns_expired_waits finds it without knowing the shape
// Exchange slots of the single-launch kernels.  N x H x W x C: one pair of 8-byte words per block and channel of its tile,
// at most one block per compute unit, 128 channels per tile and, for Eq. 4, two sets: 256 * 128 * 16 * 2 bytes.
// N x C x H x W: one pair per block, at most 8192 blocks, two sets or, for Eq. 4, four: half of that.
constexpr size_t kSlotBytes = size_t(1) << 20;
// What the N x C x H x W calls of bns_backward_builtin_workspace may need (3840 channels).
constexpr size_t kBuiltinNchwBytes = (size_t(4) << 20) + kHeaderBytes;

// Upper bound on blocks that share one channel's reduction in N x C x H x W, i.e. on partial sums per channel.  Workspaces of up
// to 3840 channels keep within kBuiltinNchwBytes: behind the slots that leaves room for 64 up to 3072 channels and
// for 48 up to 3840.  By itself the library takes one block per channel there (2048 blocks are enough), so only the overrides
// of "splits_stats", "splits_reduce" and "channel_group" ever meet the lower bound.
constexpr int kMaxSplits = 64;
inline int most_splits(int C) { return C > 3072 && C <= 3840 ? 48 : kMaxSplits; }

// [header][slots][sums S][sums V].
//
// A block that waits takes any slot word that carries the launch's stamp, and nothing clears the words between launches,
// so nothing but stamped words may ever be written there: the slots lie at the same place whatever the shape and the
// layout, and no partial sum -- arbitrary bits where a stamp is looked for -- lies below their end, also when
// calls of different shapes use the same memory one after the other.
struct WorkspaceLayout {
    size_t slots, slot_bytes;       // offset, size
    size_t sums, sum_bytes;         // offset of the first region, size of each of the two
    size_t total;
};

inline WorkspaceLayout workspace_layout(size_t sum_bytes) {
    WorkspaceLayout w;
    w.slots = kHeaderBytes;
    w.slot_bytes = kSlotBytes;
    w.sums = w.slots + w.slot_bytes;
    w.sum_bytes = sum_bytes;
    w.total = w.sums + 2 * sum_bytes;
    return w;
}

}  // namespace bns
