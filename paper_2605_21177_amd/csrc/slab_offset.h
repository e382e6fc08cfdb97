// Where the loads of a slab of tokens lie: pure arithmetic, checked on the host over all tails.
#ifndef CHUNKFT_SLAB_OFFSET_H
#define CHUNKFT_SLAB_OFFSET_H

namespace chunkft {

// Byte offset of a lane's piece from the first token of its slab, as a buffer load takes it: a per-lane part
// and a scalar part.  The hardware adds the two without wrapping at 32 bits and checks the range of each load from
// them, so neither part may stand for a negative number.
struct LoadOffset {
  unsigned lane, scalar;
};

// The load covers the tokens first, first + 1, ...; the lane takes token first + k, `column` bytes into it.  `left`
// >= 1 tokens of the slab are there, `slab` is its full length.  In a complete slab the token of the load is the
// scalar part, so that the per-lane part is the same for every load; in the last one a token past the end becomes
// the last token, and the whole offset is the lane's.
constexpr LoadOffset slab_offset(unsigned column, unsigned token_bytes, int first, int k, int left, int slab) {
  if (left >= slab) return {column + (unsigned)k * token_bytes, (unsigned)first * token_bytes};
  const int t = first + k < left ? first + k : left - 1;
  return {column + (unsigned)t * token_bytes, 0u};
}

}  // namespace chunkft
#endif
