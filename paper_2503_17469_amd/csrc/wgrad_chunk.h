// How the weight-gradient kernels of the convolutions share out a worker's positions.
#pragma once

namespace omni {

// One chunk of one worker's positions, as a workgroup sees it.  In the second stage, which adds a worker's chunks, `row`
// is the worker's first chunk and idx is not used.
struct Chunk {
  int wk, idx, n;    // worker, chunk within the worker, the worker's chunks
  int row, total;    // chunk within the layer, the layer's chunks
  int beg, end;      // the worker's rows
};

}  // namespace omni
