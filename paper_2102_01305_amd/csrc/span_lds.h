// Shape and local memory of an interpolation and span-solve block
// (markers.hip), the same for the host, which sizes the launch, and the kernel.
#pragma once

#include <cstddef>

namespace ibmk {

// Parts of the span range that a block of `threads` sums side by side.
__host__ __device__ inline int parts_at(int ns, int threads) {
  const int groups = (ns + 3) / 4;                   // threads per part
  const int parts = threads / groups;
  return parts < 1 ? 1 : (parts > 8 ? 8 : parts);
}

// Longest span whose interpolation blocks pull the moments of their marker's
// 16 nodes a layer themselves, with no band launch before them: a launch of
// the smallest chain is 4 us of latency.  Neighbouring markers then pull most
// nodes again, so it pays while half a block's threads take them in one turn.
// Step of clap & fling in us, band launch / pulled: 64x48x8 27.3 / 24.0,
// 96x80x16 28.9 / 27.5, 96x80x32 32.1 / 34.4, 96x80x48 36.0 / 41.3; 2D figure
// eight 1000x500 38.7 / 35.3.
constexpr int kPullSpan = 16;

// LDS of a block, in doubles: G (2 ns), B (3 ns), partial sums (parts x 3 ns),
// the xy sums R (4 ns) and, where it pulls them, the nodes' moments (32 ns) as
// records of 16 bytes, from an even double on.
__host__ __device__ inline size_t nodes_at(int ns, int parts) {
  const size_t d = (size_t)(9 + 3 * parts) * ns;
  return (d + 1) / 2 * 2;
}
__host__ __device__ inline size_t interp_span_doubles(int ns, int parts) {
  return nodes_at(ns, parts) + (ns <= kPullSpan ? 32 * (size_t)ns : 0);
}
__host__ __device__ inline size_t lds_at(int ns, int threads) {
  return interp_span_doubles(ns, parts_at(ns, threads)) * sizeof(double);
}

// Threads of an interp_span block for a span of ns layers: 512 (more parts
// of the span range in parallel) where its LDS fits, else 256.
__host__ __device__ inline int span_threads(int ns) { return lds_at(ns, 512) <= 150 * 1024 ? 512 : 256; }

// Parts of the span range and LDS of a block: fixed by ns alone, so a
// solve sums its span solve in the same order whatever block size a grouped
// launch runs it with (a smaller block takes the parts in turns).
__host__ __device__ inline int span_parts(int ns) { return parts_at(ns, span_threads(ns)); }
__host__ __device__ inline size_t interp_span_lds(int ns) { return lds_at(ns, span_threads(ns)); }

}  // namespace ibmk
