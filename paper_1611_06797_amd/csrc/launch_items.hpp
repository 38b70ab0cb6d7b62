// Work lists with one workgroup per item: what one launch can take, and which
// item a workgroup runs.
#pragma once

namespace ltmp2 {

// HIP takes no launch of 2^32 or more threads in x, so a list goes out in
// launches of at most this many items (a multiple of 8, the XCDs) for
// workgroups of nt threads: 8.4 million at 512 threads, a fraction of a second
// of any of these kernels.
constexpr long launch_items(int nt) { return ((1L << 32) - 1) / nt / 8 * 8; }

// Workgroups of a launch of count items.
constexpr unsigned launch_blocks(long count) { return unsigned((count + 7) / 8 * 8); }

// launch(first, count) for consecutive ranges of [0, total); the first status
// that is not 0 ends it.
template <class Fn>
auto launch_ranges(long total, int nt, Fn&& launch) {
  const long most = launch_items(nt);
  long first = 0;
  for (; total - first > most; first += most)
    if (const auto s = launch(first, most)) return s;
  return launch(first, total - first);
}

// Item of workgroup `block` of a launch of count items, or -1: workgroups are
// dispatched round-robin over the 8 XCDs, each XCD takes a contiguous range.
#ifdef __HIP__
__host__ __device__
#endif
constexpr long block_item(unsigned block, long count) {
  const long t = long(block % 8) * ((count + 7) / 8) + block / 8;
  return t < count ? t : -1;
}

}  // namespace ltmp2
