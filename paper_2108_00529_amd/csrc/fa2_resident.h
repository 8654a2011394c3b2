// Exact ForceAtlas2 iterations of one small supergraph by one workgroup, which keeps the
// whole state on chip: bodies, rows and (when they fit) neighbour ids in LDS, each node's
// mass, position and previous force in its thread's registers.  The same operations in the
// same order as the plain kernels (one repulsion segment, 256-node tiles), so the same bits.
//
// What bounds a small layout is the latency of its steps: three launches of a few us per
// iteration that together use two or three compute units.  Here an iteration is three
// barriers; the wavefronts that own nodes sum their repulsion (K terms one after the other
// per node, about 40 cycles each) while the others take the rows' attractions.  167
// supernodes of 2,700 superedges: 5.6 us per iteration instead of 12.9.
#pragma once
#include "common.h"
#include "fa2_math.h"

namespace bgv {

constexpr int32_t kResidentMax = kRepSegment;  // one segment: repulsion is one sum in order

template <int kIds>  // neighbour ids held in LDS
struct ResidentLds {
    float4 body[kResidentMax];
    float2 att[kResidentMax];
    uint32_t row[kResidentMax + 1];
    double2 ws[kResidentMax / kWave];
    uint32_t next;  // four rows that no wavefront has taken yet
    uint16_t ids[kIds];
};

struct ResidentPos {
    const float4 *body;
    __device__ __forceinline__ float2 operator[](int32_t i) const { return make_float2(body[i].x, body[i].y); }
};

// Whether the wavefronts that sum repulsion, one per 64 of K nodes, share in the rows: with
// fewer than three times as many others the rows are the longer part (512 threads: seven
// owners leave one wavefront to 448 rows), so they are taken from a counter, four at a time,
// and the owners join in when they are done; with more, or none, which leaves the same to
// all, the counter's trips cost what they save.  us per iteration with / without, 16 superedges per node: 1,024 threads 256 nodes
// 9.5 / 8.7, 320 12.7 / 13.2, 448 19.4 / 20.8; 512 threads 448 nodes 33 / 112.
template <int NT>
__host__ __device__ __forceinline__ bool resident_share(int32_t K) {
    const int owners = (K + kWave - 1) / kWave, others = NT / kWave - owners;
    return others > 0 && others < 3 * owners;
}

// `iters` iterations of K <= kResidentMax nodes by NT >= kResidentMax threads.  row[K+1]
// and cw: the supergraph's rows (kUnit: every weight is 1, so ids alone will do); kShare:
// resident_share<NT>(K), and true is right for any K; pos, fprev and *speed in and out.  Every thread of the workgroup calls it.
template <int NT, bool kUnit, bool kShare, int kIds, typename E>
__device__ __forceinline__ void fa2_resident(ResidentLds<kIds> &sh, int32_t K, int32_t iters, float2 *pos,
                                             float2 *fprev, const float *mass, const uint32_t *row, const E *cw,
                                             float *speed, float kr, float kg, float tau, float ks, float ksmax) {
    static_assert(NT >= kResidentMax && NT % 256 == 0, "one thread per node");
    constexpr int NW = NT / kWave;
    const int t = threadIdx.x, lane = t & (kWave - 1), w = t / kWave;
    const bool live = t < K;
    const uint32_t nent = row[K];
    const bool staged = kUnit && nent <= (uint32_t)kIds;
    float2 xi = live ? pos[t] : make_float2(0.f, 0.f), fp = live ? fprev[t] : make_float2(0.f, 0.f);
    const float mi = live ? mass[t] : 0.f;
    float s = *speed;
    if (t < kResidentMax) sh.body[t] = live ? fa2_body(xi, mi) : fa2_no_body();
    if (t <= K) sh.row[t] = row[t];
    if (t == 0) {
        sh.row[K] = nent;
        sh.next = 0u;
    }
    if (staged)
        for (uint32_t k = t; k < nent; k += NT) sh.ids[k] = (uint16_t)fa2_entry_id(cw[k]);
    __syncthreads();
    const int owners = (K + kWave - 1) / kWave, others = NW - owners;
    const int ntiles = (K + 255) / 256;
    const auto take = [&] {
        uint32_t g = 0u;
        if (lane == 0) g = atomicAdd(&sh.next, 1u);
        return 4 * (int32_t)__builtin_amdgcn_readfirstlane(g);
    };
    for (int32_t it = 0; it < iters; ++it) {
        float rx = 0.f, ry = 0.f;
        if (w < owners) fa2_rep_ahead(xi, sh.body, (K + 7) & ~7, rx, ry);
        if constexpr (kShare) {
            for (int32_t r = take(); r < K;) {
                const int32_t ahead = take(), n = min(4, K - r);
                if (staged) fa2_rows_attraction(ResidentPos{sh.body}, sh.ids, sh.row + r, r, n, sh.att + r, 0, 1, lane);
                else fa2_rows_attraction(ResidentPos{sh.body}, cw, sh.row + r, r, n, sh.att + r, 0, 1, lane);
                r = ahead;
            }
        } else if (others == 0 || w >= owners) {
            const int32_t first = others ? w - owners : w, step = others ? others : NW;
            if (staged) fa2_rows_attraction(ResidentPos{sh.body}, sh.ids, sh.row, 0, K, sh.att, first, step, lane);
            else fa2_rows_attraction(ResidentPos{sh.body}, cw, sh.row, 0, K, sh.att, first, step, lane);
        }
        __syncthreads();
        if (kShare && t == 0) sh.next = 0u;
        float2 f = make_float2(0.f, 0.f);
        if (w < kResidentMax / kWave) {
            double2 st = make_double2(0.0, 0.0);
            if (live) {
                f = fa2_net_force(xi, mi, kr, rx, ry, sh.att[t], kg);
                st = fa2_swing_traction(f, fp, mi);
            }
            st.x = fa2_wave_sum(st.x);
            st.y = fa2_wave_sum(st.y);
            if (lane == 0) sh.ws[w] = st;
        }
        __syncthreads();
        if (w < owners || it + 1 == iters) {
            double S = 0.0, T = 0.0;  // the tiles' sums, each of its four wavefronts' in order
            for (int b = 0; b < ntiles; ++b) {
                double x = 0.0, y = 0.0;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    x += sh.ws[4 * b + q].x;
                    y += sh.ws[4 * b + q].y;
                }
                S += x;
                T += y;
            }
            s = fa2_global_speed(S, T, s, tau);
            if (live) {
                xi = fa2_move(xi, f, fp, s, ks, ksmax);
                fp = f;
                sh.body[t] = fa2_body(xi, mi);
            }
        }
        __syncthreads();
    }
    if (live) {
        pos[t] = xi;
        fprev[t] = fp;
    }
    if (t == 0) *speed = s;
    // Before the LDS is used again, and before whatever thread 0 alone does next: without a
    // barrier in between, a caller's loop over graphs that starts with thread 0 taking the
    // next one is compiled into a loop of thread 0 around a loop of its wavefront's other
    // lanes, which then meet the barriers without it and never end.
    __syncthreads();
}

}  // namespace bgv
