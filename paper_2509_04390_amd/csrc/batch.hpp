// batch.hpp -- how graph replay cuts a run of blocks into launches (host).
#pragma once

namespace rta {

constexpr int kBatch = 16;  // blocks that graph replay runs at once, at most (see graph_batch in rta.hip)

// Blocks that the next part of a run of `left` blocks takes: up to kBatch at
// once where the context can (`batched`), else one.  A batch is three
// launches, each waiting for the one before, so one and two blocks are faster
// one by one, three are even and more are not (us per replay, one by one / at
// once: 1 -> 1 x 65,536 taps, B = 256, of 1 / 2 / 3 / 4 blocks 18.0 / 21.1,
// 21.1 / 21.5, 24.1 / 21.9, 30.0 / 22.3; 1 -> 32 x 480,000, B = 128 18.3 / 24.3,
// 23.7 / 30.8, 32.1 / 34.7, 40.5 / 39.6).
inline int graph_run(bool batched, int left) {
  if (!batched || left < 3) return 1;
  return left < kBatch ? left : kBatch;
}

}  // namespace rta
