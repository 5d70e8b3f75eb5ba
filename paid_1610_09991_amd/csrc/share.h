// share.h -- how the evaluation's workgroups share the work items of a round:
// the integer arithmetic of it, plain functions for the kernels and for a host
// compiler.  Which workgroup evaluates an item changes nothing in its result.
#pragma once

namespace paid {

struct Span {  // items [i0, i1)
  int i0, i1;
};

__host__ __device__ inline int share_min(int a, int b) { return a < b ? a : b; }
__host__ __device__ inline int share_max(int a, int b) { return a > b ? a : b; }

// ---- one wave per parent (k_children)
// The round's work items in chunks: the grid is the workgroups resident at
// once; each takes a first chunk by its index and then further ones from one
// counter (zero at the start of a round) until the items are gone.  A chunk is
// half of an even share of the items that are left, in whole passes of the
// workgroup's waves, so chunks shrink towards the end and no workgroup is left
// with a long one; a round of few items is spread over all workgroups.
__host__ __device__ inline int chunk_items(int left, int waves, int grid) {
  const int half = left / (2 * grid);
  if (half >= waves) return half / waves * waves;
  const int even = (left - 1) / grid + 1;  // spread what is left
  return share_max(1, share_min(waves, even));
}
__host__ __device__ inline Span first_chunk(int total, int waves, int grid, int block) {
  const int c = chunk_items(total, waves, grid);
  const long i0 = (long)block * c;
  Span k;
  k.i0 = i0 < total ? (int)i0 : total;
  k.i1 = k.i0 + share_min(c, total - k.i0);
  return k;
}
// the items behind all first chunks start here (may lie past the end)
__host__ __device__ inline long chunk_base(int total, int waves, int grid) {
  return (long)chunk_items(total, waves, grid) * grid;
}

// ---- two lanes per child (k_children_lpc)
// An eighth of the round's items per XCD (the workgroups b = x mod 8; in a grid
// of fewer workgroups a share per workgroup), each workgroup of an XCD a first
// share by its index there and then shares from the XCD's own counter.
struct XcdShare {
  int x, first, last;  // the XCD, its items [first, last)
  int wgs, index;      // its workgroups, this one's place among them
};
__host__ __device__ inline XcdShare xcd_share(int total, int grid, int block, int xcds) {
  XcdShare s;
  const int nx = share_min(xcds, grid);
  s.x = block % nx;
  s.first = (int)((long)total * s.x / nx);
  s.last = (int)((long)total * (s.x + 1) / nx);
  s.wgs = (grid - s.x + nx - 1) / nx;
  s.index = block / nx;
  return s;
}
// share sizes: half of an even share of the XCD's items left, in whole groups
__host__ __device__ inline int share_items(int left, int group, int grid, int xcds) {
  const int wgs = (grid + xcds - 1) / xcds;  // (the XCD's workgroups, or one more)
  if (group == 1) return share_max(1, (left - 1) / wgs + 1);
  return share_max(group, left / (2 * wgs) / group * group);
}
// the first share of a workgroup, c = share_items of all of the XCD's items
__host__ __device__ inline Span first_share(const XcdShare &s, int c) {
  const long i0 = (long)s.first + (long)s.index * c;
  Span k;
  k.i0 = i0 < s.last ? (int)i0 : s.last;
  k.i1 = k.i0 + share_min(c, s.last - k.i0);
  return k;
}
// where the items behind the XCD's first shares start
__host__ __device__ inline int share_base(const XcdShare &s, int c) {
  const long b = (long)s.first + (long)s.wgs * c;
  return b < s.last ? (int)b : s.last;
}

// ---- both: the c items that the counter hands out at its value `count`, behind base
__host__ __device__ inline Span counted_span(int base, int total, int count, int c) {
  Span k;
  k.i0 = share_min(base + count, total);
  k.i1 = k.i0 + share_min(c, total - k.i0);
  return k;
}

// A workgroup's range in one word, end << 32 | next item: a wave takes `group`
// items by adding to it.
__host__ __device__ inline unsigned long long range_word(Span k) {
  return ((unsigned long long)(unsigned)k.i1 << 32) | (unsigned)k.i0;
}
__host__ __device__ inline int range_next(unsigned long long r) { return (int)(unsigned)r; }
__host__ __device__ inline int range_end(unsigned long long r) { return (int)(r >> 32); }
__host__ __device__ inline bool range_empty(unsigned long long r) { return (unsigned)r >= (unsigned)(r >> 32); }
// the group of a taker that found r there
__host__ __device__ inline Span range_group(unsigned long long r, int group) {
  Span k;
  k.i0 = range_next(r);
  k.i1 = k.i0 + share_min(range_end(r) - k.i0, group);
  return k;
}

}  // namespace paid
