// copy_rule.hpp -- who waits for a chunk's last launch before a DMA copy-out:
// the host, which then queues the copy, or the device, by a stream wait.
#pragma once
#include <stddef.h>
#include <stdint.h>

namespace so2dr {

// `queued` host copies of at most `piece` bytes go to the device without the
// host waiting for any of them.  Queued that way a few large copies run as
// well as released ones, or better; many small ones collapse, from a count
// that falls with their size.  Measured on MI355X, ms with the host's wait and
// the device's: two slots, 13-point FP32, 512 MiB x 128 copies 739 and 721, 256
// MiB x 128 371 and 362, 128 MiB x 32 48.9 and 47.9; 7-point 128 MiB x 192 272
// and 276-435, 64 MiB x 64 46.3 and 45.9, x 128 91 and 98-189, 32 MiB x 64 47
// and 112.
constexpr bool queue_carries(size_t piece, int64_t queued) {
  return piece >= ((size_t)64 << 20) && (uint64_t)queued * 4 <= (uint64_t)(piece >> 20) * 3;
}

// A forward run, all of whose copies are queued at once.  With three slots the
// device always has a copy of each direction to go on with and the engines'
// higher rate counts: the host waits (13-point, 512 MiB: 356 against 363 ms).
// With two the launches lie between the copies, and beside the engines they
// take longer: the device waits where its queue carries that (2048^3, 1 GiB
// copies: 93.3 against 94.9 GCell/s).
constexpr bool host_waits_forward(int n_slots, size_t piece, int64_t queued) {
  return n_slots != 2 || !queue_carries(piece, queued);
}

// A pass of the reverse sweep over `chunks` chunks, two copies in and one out
// for each, drained at its end: the device waits wherever its queue carries
// that (gradient of 1024^3 in 28 chunks, 48 steps: 755 ms with the host's wait,
// 743; 1024 x 1024 x 512 in 16 chunks of 128 MiB and two slots 390 and 382, in
// 32 of 64 MiB 395 and 470-493).
constexpr bool host_waits_reverse(size_t piece, int chunks) { return !queue_carries(piece, 3 * (int64_t)chunks); }

}  // namespace so2dr
