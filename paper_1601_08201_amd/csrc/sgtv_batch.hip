// Elementwise kernels of the ADMM iteration for many scans in one launch.
// Block b works on scan blocks[b].scan starting at element blocks[b].start;
// the arithmetic per element is the single-scan kernels' own (shared device
// functions batch_*_elem / batch_split_block), so a scan of a batch
// reproduces its single-scan run bit for bit.
#include "sgtv_device.h"

namespace sgtv {

__global__ __launch_bounds__(kBlock) void k_ratio_batch(const BatchBlock *__restrict__ blocks,
                                                        const ScanDev *__restrict__ scans) {
    const BatchBlock bb = blocks[blockIdx.x];
    batch_ratio_elem(scans[bb.scan], bb.start + threadIdx.x);
}

__global__ __launch_bounds__(kBlock) void k_voxel_batch(const BatchBlock *__restrict__ blocks,
                                                        const ScanDev *__restrict__ scans,
                                                        int fcur, int vcur) {
    const BatchBlock bb = blocks[blockIdx.x];
    batch_voxel_elem(scans[bb.scan], bb.start + threadIdx.x, fcur, vcur);
}

__global__ __launch_bounds__(kBlock) void k_split_batch(const BatchBlock *__restrict__ blocks,
                                                        const ScanDev *__restrict__ scans,
                                                        int fcur, int vcur) {
    const BatchBlock bb = blocks[blockIdx.x];
    batch_split_block(scans[bb.scan], bb.start, threadIdx.x, fcur, vcur);
}

// Blocks [0, n_sblocks): the split update of the iteration before (image f[fcur],
// splits v[vcur] to v[vcur ^ 1]), then the ratio of this one; neither reads what
// the other writes.  us an iteration, apart / together: 16 scans of 9 x 41 x 54
// 56.4 / 54.2, 8 uneven scans of 48 to 96 a side 411 / 410.
__global__ __launch_bounds__(kBlock) void k_ratio_split_batch(const BatchBlock *__restrict__ rblocks,
                                                              const BatchBlock *__restrict__ sblocks,
                                                              unsigned n_sblocks, const ScanDev *__restrict__ scans,
                                                              int fcur, int vcur) {
    if (blockIdx.x < n_sblocks) {
        const BatchBlock bb = sblocks[blockIdx.x];
        batch_split_block(scans[bb.scan], bb.start, threadIdx.x, fcur, vcur);
        return;
    }
    const BatchBlock bb = rblocks[blockIdx.x - n_sblocks];
    batch_ratio_elem(scans[bb.scan], bb.start + threadIdx.x);
}

hipError_t launch_ratio_split_batch(const BatchBlock *rblocks, int64_t n_rblocks, const BatchBlock *sblocks,
                                    int64_t n_sblocks, const ScanDev *scans, int fcur, int vcur, hipStream_t st) {
    if (n_rblocks + n_sblocks == 0) return hipSuccess;
    hipLaunchKernelGGL(k_ratio_split_batch, dim3(static_cast<unsigned>(n_rblocks + n_sblocks)), dim3(kBlock), 0, st,
                       rblocks, sblocks, static_cast<unsigned>(n_sblocks), scans, fcur, vcur);
    return hipGetLastError();
}

hipError_t launch_ratio_batch(const BatchBlock *blocks, int64_t n_blocks, const ScanDev *scans,
                              hipStream_t st) {
    if (n_blocks == 0) return hipSuccess;
    hipLaunchKernelGGL(k_ratio_batch, dim3(static_cast<unsigned>(n_blocks)), dim3(kBlock), 0, st,
                       blocks, scans);
    return hipGetLastError();
}

hipError_t launch_voxel_batch(const BatchBlock *blocks, int64_t n_blocks, const ScanDev *scans,
                              int fcur, int vcur, hipStream_t st) {
    if (n_blocks == 0) return hipSuccess;
    hipLaunchKernelGGL(k_voxel_batch, dim3(static_cast<unsigned>(n_blocks)), dim3(kBlock), 0, st,
                       blocks, scans, fcur, vcur);
    return hipGetLastError();
}

hipError_t launch_split_batch(const BatchBlock *blocks, int64_t n_blocks, const ScanDev *scans,
                              int fcur, int vcur, hipStream_t st) {
    if (n_blocks == 0) return hipSuccess;
    hipLaunchKernelGGL(k_split_batch, dim3(static_cast<unsigned>(n_blocks)), dim3(kBlock), 0, st,
                       blocks, scans, fcur, vcur);
    return hipGetLastError();
}

}  // namespace sgtv
