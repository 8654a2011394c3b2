// Sums of per-node values by community label (volumes), for kernels whose workgroups
// each hold many nodes: a small table in LDS gathers the values of the labels that came
// first to its slots (four probes each), and every slot leaves as one device atomic.
//
// What bounds such sums is the rate of device atomics on one address (about 12 ns each):
// a few giant communities hold most nodes of some streams, and one atomic per node then
// takes n * 12 ns.  A label that is frequent in a workgroup's nodes is almost surely among
// the first to reach one of its slots (with one probe, a rare label that came first to a
// giant one's slot cost that workgroup thousands of serial atomics: 1.8 or 16 ms per call
// of the volume rule, by the nodes' names); rare labels that find their slots taken go
// straight to memory, where they do not collide.  Integer sums: the order does not matter.
// One atomic per node -> this table: 11.7 ms -> 12 us on 1M nodes after three passes of
// the volume rule (97% of them in one community), 212 -> 28 us on the same nodes after
// the sequential rule, 224 -> 120 us on 3.2M nodes of 172,000 communities (there the
// rare labels' atomics, about 25 per ns, set the pace).
#pragma once
#include "common.h"

namespace bgv {

constexpr int kVsBits = 11;
constexpr int kVsSlots = 1 << kVsBits;
constexpr int kVsProbes = 4;

struct VolumeTable {
    unsigned long long sum[kVsSlots];
    int32_t key[kVsSlots];  // -1: free
};

__device__ __forceinline__ void vs_clear(VolumeTable &t) {
    for (int q = threadIdx.x; q < kVsSlots; q += blockDim.x) {
        t.key[q] = -1;
        t.sum[q] = 0ull;
    }
}

// Adds v at label lab (>= 0).
__device__ __forceinline__ void vs_add(VolumeTable &t, unsigned long long *vol, int32_t lab, unsigned long long v) {
    uint32_t q = ((uint32_t)lab * 2654435761u) >> (32 - kVsBits);
    for (int probe = 0; probe < kVsProbes; ++probe, q = (q + 1) & (kVsSlots - 1)) {
        int32_t k = __hip_atomic_load(&t.key[q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        if (k < 0) {
            k = atomicCAS(&t.key[q], -1, lab);
            if (k < 0) k = lab;
        }
        if (k == lab) {
            atomicAdd(&t.sum[q], v);
            return;
        }
    }
    atomicAdd(&vol[lab], v);
}

// Adds v at the label lab of node `node`.  The id a label is named after meets it once: that
// node's own value goes straight to memory, so that streams whose nodes mostly keep their own
// labels neither probe nor fill the table for them (683,000 nodes that all keep theirs: call
// 138 -> 113 us, 111 with one atomic per node).
__device__ __forceinline__ void vs_add_node(VolumeTable &t, unsigned long long *vol, int64_t node, int32_t lab,
                                            unsigned long long v) {
    if (lab == (int32_t)node) atomicAdd(&vol[lab], v);
    else vs_add(t, vol, lab, v);
}

// After a barrier behind the last vs_add.
__device__ __forceinline__ void vs_flush(const VolumeTable &t, unsigned long long *vol) {
    for (int q = threadIdx.x; q < kVsSlots; q += blockDim.x)
        if (t.sum[q]) atomicAdd(&vol[t.key[q]], t.sum[q]);
}

// Workgroups of 1024 threads that share n nodes out: two to a compute unit at most, so
// that a workgroup's table sees thousands of nodes when there are many.
inline unsigned vs_grid(int64_t n) { return grid_for(n, 1024, 512); }

}  // namespace bgv
