// Which block's operands the inference kernels of bottleneck runs ask for ahead of their use.  Plain C++ (a constexpr function is compiled for both sides),
// so that it can be tested on the host.
#pragma once

namespace hpf {

// The block whose first matrix and tables block bi of a run of nblk asks for, `distance` blocks ahead.  Behind the last one: the last one's again, which nobody
// uses (no branch in the loop).  That block has to have the shape of those operands: a lead's first convolution and BatchNorm have half the
// channels of the others', so a run of the lead alone asks for none: -1.
constexpr int block_ahead(bool lead, int bi, int distance, int nblk) {
  return lead && nblk == 1 ? -1 : bi + distance < nblk ? bi + distance : nblk - 1;
}

}  // namespace hpf
