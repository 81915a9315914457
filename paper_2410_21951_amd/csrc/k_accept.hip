// Stand-alone top-k of the draft heads' logits (rows of more than 4096: slice by slice).
#include "accept_dev.h"

__global__ __launch_bounds__(256) void k_topk(Dims D, DevState s, int seq0) {
    dev_topk<true>(D, s, blockIdx.x, seq0 + blockIdx.y);
}
void launch_topk(const Dims& D, const DevState& s, int seq0, int nseq, hipStream_t st) {
    launch(k_topk, dim3(D.Hh, nseq), dim3(256), 0, st, D, s, seq0);
}
