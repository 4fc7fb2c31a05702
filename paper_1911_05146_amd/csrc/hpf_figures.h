// Algorithmic figures of an image-resident run, for the profiling calls: per image, every tensor that a direction has to read or write once (elements), and the
// flop of its contractions (2*M*K*N each).  Plain C++, so that it can be tested on the host.
#pragma once

namespace hpf {

struct RunFigures {
  double forward = 0, inference = 0, backward = 0;   // elements
  double flops = 0;                                  // of one direction
  double wgrad = 0, wgrad_flops = 0;                 // of the run's own weight-gradient launch: the identity blocks
};
// kind 0: basic, 1: bottleneck, 2: post-activation; px: pixels of the run's output; count: blocks, lead: 1 if the first of them halves the image and doubles
// the channels (its weight gradients go with the grouped ones).
inline RunFigures run_figures(int kind, int C, int MID, double px, int count, int lead) {
  const double c = C, m = MID, n = count - lead;
  const double stash = px * (kind == 2 ? 3 * c : kind == 0 ? 2 * c : 2 * m + c);   // c1, [c2,] y of an identity block; the backward reads x, c1 [, c2] (2: y) ...
  const double flops = 2 * px * (kind == 1 ? 2 * c * m + 9 * m * m : 18 * c * c);
  const double in = lead ? 4 * px * c / 2 : px * c;
  RunFigures f;
  f.forward = in + n * stash;
  f.inference = in + px * c;
  f.backward = px * c + n * 2 * stash;                                             // ... and writes as many gradients
  f.flops = n * flops;
  f.wgrad = n * 2 * stash;
  f.wgrad_flops = n * flops;
  if (lead) {
    f.forward += kind == 2 ? px * 5 * c : stash;                                   // 2: c1, relu(bn1(c1)), c2, the shortcut, y
    f.backward += kind == 2 ? px * 6 * c + in                                      // y, c2, c1; dc2, dc1 and the shortcut's gradient, that of the input
                            : 2 * (in + stash - px * c);                           // x, c1 [, c2]; [dc2,] dc1, that of the input
    f.flops += 2 * px * (kind == 1 ? c / 2 * m + 9 * m * m + m * c + c / 2 * c : 9 * c / 2 * c + 9 * c * c + c / 2 * c);
  }
  return f;
}

}  // namespace hpf
