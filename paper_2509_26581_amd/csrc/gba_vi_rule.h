// The visual-inertial Schur solve's choice between explicit keyframe blocks and
// implicit products (host only).
#pragma once

namespace gba {
namespace vi {

// Whether a step's PCG pays for the explicit keyframe blocks: M observations,
// their pairs on one point, nnz blocks, far of the observations outside their
// workgroup's keyframe window.  Forming takes 20 ps a pair and 60 ps a block;
// an iteration reads a block in 80 ps where the implicit product takes 20 ps an
// observation, 300 ps more a far one (an atomic add of its own for each entry)
// and 15 us of launches.  2-trial solves of 200 iterations, blocks against
// implicit products: 300 keyframes 1.6 to 2.4 times as fast (0.03 to 0.56 blocks
// an observation), 1,000 keyframes 2.2 at 1.1 blocks an observation and 1.4 at
// 2.3, 3,000 keyframes seen at random 0.85 at 6.0 (1.1 GB of workspace where the
// products take 0.2).
inline bool vi_blocks_pay(long long M, long long pairs, long long nnz, long long far, int max_iters) {
    const double its = max_iters < 50 ? max_iters : 50;
    const double saved = 15.0 + 20e-6 * (double)M + 300e-6 * (double)far - 80e-6 * (double)nnz;
    return 20e-6 * (double)pairs + 60e-6 * (double)nnz <= its * saved;
}

}  // namespace vi
}  // namespace gba
