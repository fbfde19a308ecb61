// copy_rule.hpp -- who waits for a chunk's last launch before a DMA copy-out in
// the reverse sweep: the host, which then queues the copy, or the device, by a
// stream wait.  Forward runs always leave it to the host: over two slots the
// device's wait is 2 % faster once a process is warm (13-point FP32 in 1 GiB
// copies 2885 against 2946 ms, 512 MiB 1444 and 1485, 256 MiB 363 and 371), but
// a process' first pass takes 3622 against 2947, 1772 and 1494, 535 and 383 ms;
// over three slots it is slower warm as well (512 MiB 363 against 356).
#pragma once
#include <stddef.h>
#include <stdint.h>

namespace so2dr {

// `queued` host copies of at most `piece` bytes go to the device without the
// host waiting for any of them.  Queued that way a few large copies run as
// well as released ones, or better; many small ones collapse, from a count
// that falls with their size.  Measured on MI355X, ms with the host's wait and
// the device's, 7-point forward runs over two slots: 128 MiB x 192 copies 272
// and 276-435, 64 MiB x 64 46.3 and 45.9, x 128 91 and 98-189, 32 MiB x 64 47
// and 112.
constexpr bool queue_carries(size_t piece, int64_t queued) {
  return piece >= ((size_t)64 << 20) && (uint64_t)queued * 4 <= (uint64_t)(piece >> 20) * 3;
}

// A pass of the reverse sweep over `chunks` chunks, two copies in and one out
// for each, drained at its end: the device waits wherever its queue carries
// that.  Gradients over 32 steps, first pass of a process and warm, host's wait
// and device's: 1024^3 in 28 chunks 1368 / 1348 and 1343 / 1322 ms, 1024 x 1024
// x 512 in 16 chunks of 128 MiB and two slots 714 / 698 and 706 / 685; in 32
// chunks of 64 MiB (16 steps, warm) 395 and 470-493, so the host waits there.
constexpr bool host_waits_reverse(size_t piece, int chunks) { return !queue_carries(piece, 3 * (int64_t)chunks); }

}  // namespace so2dr
