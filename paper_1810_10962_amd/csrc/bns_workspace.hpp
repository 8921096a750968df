// Where things lie in a workspace.  Plain C++ without HIP headers, so that a host compiler can check it alone.
#pragma once
#include <stddef.h>

#include "bns_validate.hpp"

namespace bns {

constexpr size_t kHeaderBytes = 256;        // in front of everything else: bns_expired_waits finds it without knowing the shape
// Exchange slots of the single-launch kernels.  N x H x W x C: one pair of 8-byte words per block and channel of its tile,
// at most one block per compute unit, 128 channels per tile and, for Eq. 4, two sets: 256 * 128 * 16 * 2 bytes.
constexpr size_t kSlotBytes = size_t(1) << 20;
// N x C x H x W: the slots of 8192 blocks in two sets (or 4096 in the four sets of Eq. 4) are the least it gets.
constexpr size_t kLeastSlotBytes = size_t(256) << 10;
// What the N x C x H x W calls of bns_backward_builtin_workspace may need (3840 channels).
constexpr size_t kBuiltinNchwBytes = (size_t(4) << 20) + kHeaderBytes;

// [header][slots][sums S][sums V].
//
// A block that waits takes any slot word that carries the launch's stamp, and nothing clears the words between launches,
// so nothing but stamped words may ever be written there: the slots begin at the same place whatever the shape and the
// layout, and no partial sum -- arbitrary bits where a stamp is looked for -- lies below the end of the slots, also when
// calls of different shapes use the same memory one after the other.
//
// One exception, so that workspaces of up to 3840 channels keep the size they have always had: from 3072 channels
// on the N x C x H x W layout gives up the upper part of the slots, down to kLeastSlotBytes, which its own kernels
// never need more of.  Only N x H x W x C calls of Eq. 4 or of more than 16384 pairs use that part.
struct WorkspaceLayout {
    size_t slots, slot_bytes;       // offset, size
    size_t sums, sum_bytes;         // offset of the first region, size of each of the two
    size_t total;
};

inline WorkspaceLayout workspace_layout(const Dims& d, size_t sum_bytes) {
    WorkspaceLayout w;
    w.slots = kHeaderBytes;
    w.slot_bytes = kSlotBytes;
    if (d.layout == BNS_NCHW) {
        const size_t room = kBuiltinNchwBytes - kHeaderBytes;
        const size_t left = room > 2 * sum_bytes ? room - 2 * sum_bytes : 0;
        w.slot_bytes = left < kLeastSlotBytes ? kLeastSlotBytes : left < kSlotBytes ? left : kSlotBytes;
    }
    w.sums = w.slots + w.slot_bytes;
    w.sum_bytes = sum_bytes;
    w.total = w.sums + 2 * sum_bytes;
    return w;
}

}  // namespace bns
