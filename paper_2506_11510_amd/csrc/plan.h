// plan.h -- sizes of a render's scratch: host arithmetic without HIP, so that
// it can be checked over whole ranges on a CPU.
#pragma once

#include <algorithm>
#include <cstdint>

namespace tv {

constexpr uint32_t kFirstBlock = 64;     // threads per block of k_first: entry records it walks
constexpr uint32_t kMostChunk = 16384;   // entry records of a chunk, at most

// The eight lists of colliding samples: entry records are dealt to them in
// chunks (at least 16 chunks per list where there are blocks enough).
struct ListPlan {
  uint32_t chunk_blocks;  // blocks of k_first per chunk
  uint32_t band_size;     // records per list
  uint64_t words() const { return 8 * (uint64_t)band_size; }
};

// The lists of a call whose largest pass has `most` entry records.  Every pass
// of the call uses this one plan: the room does not grow with the number of
// records (the chunk shrinks in steps and its count rounds up to eights), so a
// plan made for a shorter pass can need more than the largest one's.
inline ListPlan list_plan(uint64_t most) {
  ListPlan p;
  p.chunk_blocks = (uint32_t)std::max<uint64_t>(1, std::min<uint64_t>(kMostChunk, most / 128) / kFirstBlock);
  const uint64_t g = (uint64_t)p.chunk_blocks * kFirstBlock, chunks = (most + g - 1) / g;
  p.band_size = (uint32_t)((chunks + 7) / 8 * g);
  return p;
}

}  // namespace tv
