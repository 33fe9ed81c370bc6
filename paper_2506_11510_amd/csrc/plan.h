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

// Grid of k_first for its image blocks and the blocks of training paths before
// them: HIP launches fewer than 2^32 threads along x, so the largest batches
// (the lists' last round reaches past 2^32 records) take two rows.
struct FirstGrid {
  uint32_t x, y;
};

inline FirstGrid first_grid(const ListPlan& p, uint32_t train_blocks) {
  const uint64_t blocks = train_blocks + p.words() / kFirstBlock, most = (0xFFFFFFFFull / kFirstBlock) & ~7ull;
  const uint64_t rows = (blocks + most - 1) / most;
  return {(uint32_t)(((blocks + rows - 1) / rows + 7) / 8 * 8), (uint32_t)rows};
}

// Samples per pixel of a pass whose records, lists and light-ray queue share
// `bytes` of fixed scratch (at most `most`), with room for 1.25 light rays per
// sample; 0: not even one sample per pixel, the light rays are better walked by
// their own lanes.  A queue that fills leaves its paths to a second launch, as
// long as a whole one of lanes that walk their own (4.2 M samples of a 256^3
// cloud at 1.1 light rays each: room for 1.15 per sample 24.7 ms, no queue
// 16.9 ms; 3.7 M samples, room for 1.47: 9.2 ms, no queue 13.2 ms).
inline int64_t queued_pass(int64_t slots, int64_t most, int64_t bytes) {
  const int64_t fit = bytes / (slots * (32 + 4 + 40));
  return std::min(most, fit);
}

// The light-ray queue of a pass of `samples` samples traced by at most `waves`
// waves, which take it a chunk at a time: at most 4 rays per sample and 2^26 in
// all, and one more chunk for each wave (its last is partly used); no more
// than 2^27 records however many waves are asked for.
constexpr int64_t kMostQueued = 1ll << 27;

struct QueuePlan {
  uint32_t chunk, chunks;  // records per chunk, chunks
  int64_t waves;
  uint32_t records() const { return chunk * chunks; }
  // Rays that find room however the waves share the chunks.
  int64_t sure() const { return std::max<int64_t>(0, ((int64_t)chunks - waves) * chunk); }
};

inline QueuePlan queue_plan(int64_t samples, int64_t waves) {
  QueuePlan p;
  p.chunk = samples < (1 << 20) ? 64u : 256u;
  p.waves = std::min<int64_t>(waves, (samples + 63) / 64 + 4);
  p.chunks = (uint32_t)std::min<int64_t>(kMostQueued / p.chunk, std::min<int64_t>(1ll << 26, samples * 4) / p.chunk + p.waves);
  return p;
}

}  // namespace tv
