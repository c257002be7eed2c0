// Copying tables into a block's LDS.
#pragma once

#include <hip/hip_runtime.h>

namespace qed {

constexpr int kStageBlock = 256;   // threads of every block that stages a table

// Element i < N of a table, for every thread of a block of kStageBlock: get(i) reads it,
// put(i, v) writes it to LDS.  The barrier before the first use is the caller's.
//
// What bounds a short launch here is the latency of the reads, a few hundred ns each,
// so all of a thread's reads are in flight before its first write, without a branch
// (a thread past the end reads the last element again), and the tables of a kernel follow
// each other without barriers: the network, the fits and the rate table (45 KB) in
// one trip instead of ten.  30,000 electrons and 7,500 photons of the laser field: k_lepton of
// the optical-depth path 20.6 to 19.2 us, k_photon 15.6 to 14.0.
template <int N, class Get, class Put>
__device__ __forceinline__ void stage_table(Get get, Put put) {
    constexpr int K = (N + kStageBlock - 1) / kStageBlock;
    decltype(get(0)) v[K];
#pragma unroll
    for (int q = 0; q < K; ++q) v[q] = get(min((int)threadIdx.x + q * kStageBlock, N - 1));
#pragma unroll
    for (int q = 0; q < K; ++q)
        if ((int)threadIdx.x + q * kStageBlock < N) put((int)threadIdx.x + q * kStageBlock, v[q]);
}

template <int N, class T>
__device__ __forceinline__ void stage_copy(T *dst, const T *src) {
    stage_table<N>([=](int i) { return src[i]; }, [=](int i, const T &v) { dst[i] = v; });
}

}  // namespace qed
