// The autotuner's choice of CG block sizes from its probes (host code only).
#pragma once

namespace tc {

// One probe step with `block` rows to a vertex block and threads to a product
// block: GPU time of its CG kernels, and its CG iterations.
struct CgProbe {
  int block;
  double spmv_ms, update_ms;   // launched iterations
  double small_ms;             // whole solves in one block
  long long its;
};

struct CgChoice {
  int vertex_block, spmv_block;
};

// Where every iteration was launched the two kernels are chosen each for
// itself, by its time per iteration.  A probe that ran solves in one block
// (blocks of 256, small pads) leaves its launched kernels only some of the
// iterations, or none, so their times are no measure of theirs: it is taken or
// left as a whole, by the time of all its CG kernels against the best launched
// pair.  A kernel without a time was not measured and is not chosen.
inline CgChoice choose_cg_blocks(const CgProbe* probe, int n, CgChoice now) {
  const double none = 1e300;
  double best_u = none, best_s = none, best_small = none;
  int small_block = 0;
  for (int i = 0; i < n; ++i) {
    const CgProbe& p = probe[i];
    if (p.its <= 0) continue;
    if (p.small_ms > 0.0) {
      const double t = (p.spmv_ms + p.update_ms + p.small_ms) / (double)p.its;
      if (t < best_small) { best_small = t; small_block = p.block; }
      continue;
    }
    const double u = p.update_ms / (double)p.its, s = p.spmv_ms / (double)p.its;
    if (u > 0.0 && u < best_u) { best_u = u; now.vertex_block = p.block; }
    if (s > 0.0 && s < best_s) { best_s = s; now.spmv_block = p.block; }
  }
  if (best_small < none && !(best_u < none && best_s < none && best_u + best_s < best_small))
    now.vertex_block = now.spmv_block = small_block;
  return now;
}

}  // namespace tc
