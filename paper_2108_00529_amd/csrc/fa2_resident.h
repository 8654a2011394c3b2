// Exact ForceAtlas2 iterations of one small supergraph by one workgroup, which keeps the
// whole state on chip: bodies, rows and (when they fit) neighbour ids in LDS, each node's
// mass, position and previous force in its thread's registers.  The same operations in the
// same order as the plain kernels (one repulsion segment, 256-node tiles), so the same bits.
//
// What bounds a small layout is the latency of its steps: three launches of a few us per
// iteration that together use two or three compute units.  Here an iteration is three
// barriers; the wavefronts that own nodes sum their repulsion (the longest step: K terms
// one after the other per node, about 40 cycles each) while the others take the rows'
// attractions.  167 supernodes of 2,700 superedges: 5.6 us per iteration instead of 12.9.
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
    uint16_t ids[kIds];
};

struct ResidentPos {
    const float4 *body;
    __device__ __forceinline__ float2 operator[](int32_t i) const { return make_float2(body[i].x, body[i].y); }
};

// The attractions of rows first, first + step, ... by one wavefront, four rows at a time,
// so that their loads overlap and one packed reduction sums all four; rows cut into blocks
// (more than kAttBlock entries) go one by one.
template <typename E>
__device__ __forceinline__ void resident_attraction(const float4 *body, const E *cw, const uint32_t *row,
                                                    float2 *att, int32_t K, int32_t first, int32_t step, int lane) {
    const ResidentPos pos{body};
    for (int32_t r0 = first; r0 < K; r0 += 4 * step) {
        uint32_t b[4], len[4], longest = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int32_t r = min(r0 + q * step, K - 1);
            b[q] = row[r];
            len[q] = r0 + q * step < K ? row[r + 1] - b[q] : 0u;
            longest = max(longest, len[q]);
        }
        float ax[4], ay[4];
        if (longest <= (uint32_t)kWave) {  // uniform over the wavefront
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                ax[q] = ay[q] = 0.f;
                if ((uint32_t)lane < len[q]) {
                    const E e = cw[b[q] + lane];
                    fa2_entry_add(e, pos[fa2_entry_id(e)], pos[min(r0 + q * step, K - 1)], ax[q], ay[q]);
                }
            }
        } else if (longest <= kAttBlock) {
#pragma unroll
            for (int q = 0; q < 4; ++q)
                fa2_block_lane(pos, cw, b[q], b[q] + len[q], pos[min(r0 + q * step, K - 1)], lane, ax[q], ay[q]);
        } else {
            for (int q = 0; q < 4 && r0 + q * step < K; ++q) {
                const int32_t r = r0 + q * step;
                const float2 a = fa2_row_attraction(pos, cw, b[q], b[q] + len[q], pos[r], lane);
                if (lane == 0) att[r] = a;
            }
            continue;
        }
        const float sx = fa2_wave_sum4(ax), sy = fa2_wave_sum4(ay);
        const int32_t r = r0 + lane / 16 * step;
        if (lane % 16 == 0 && r < K) att[r] = make_float2(sx, sy);
    }
}

// `iters` iterations of K <= kResidentMax nodes by NT >= kResidentMax threads.  row[K+1]
// and cw: the supergraph's rows; pos, fprev and *speed in and out.  Every thread of the
// workgroup calls it.
template <int NT, int kIds, typename E>
__device__ __forceinline__ void fa2_resident(ResidentLds<kIds> &sh, int32_t K, int32_t iters, float2 *pos,
                                             float2 *fprev, const float *mass, const uint32_t *row, const E *cw,
                                             float *speed, float kr, float kg, float tau, float ks, float ksmax) {
    static_assert(NT >= kResidentMax && NT % 256 == 0, "one thread per node");
    constexpr int NW = NT / kWave;
    const int t = threadIdx.x, lane = t & (kWave - 1), w = t / kWave;
    const bool live = t < K;
    const uint32_t nent = row[K];
    const bool staged = !std::is_same<E, int2>::value && nent <= (uint32_t)kIds;
    float2 xi = live ? pos[t] : make_float2(0.f, 0.f), fp = live ? fprev[t] : make_float2(0.f, 0.f);
    const float mi = live ? mass[t] : 0.f;
    float s = *speed;
    if (t < kResidentMax) sh.body[t] = live ? fa2_body(xi, mi) : fa2_no_body();
    if (t <= K) sh.row[t] = row[t];
    if (t == 0) sh.row[K] = nent;
    if (staged)
        for (uint32_t k = t; k < nent; k += NT) sh.ids[k] = (uint16_t)fa2_entry_id(cw[k]);
    __syncthreads();
    // wavefronts [0, owners) sum repulsion; the rest, or all of them when there is no rest,
    // take the attractions
    const int owners = (K + kWave - 1) / kWave;
    const int helpers = NW - owners;
    const int ntiles = (K + 255) / 256;
    for (int32_t it = 0; it < iters; ++it) {
        float rx = 0.f, ry = 0.f;
        if (w < owners) fa2_rep_ahead(xi, sh.body, (K + 7) & ~7, rx, ry);
        if (helpers == 0 || w >= owners) {
            const int32_t first = helpers ? w - owners : w, step = helpers ? helpers : NW;
            if (staged) resident_attraction(sh.body, sh.ids, sh.row, sh.att, K, first, step, lane);
            else resident_attraction(sh.body, cw, sh.row, sh.att, K, first, step, lane);
        }
        __syncthreads();
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
}

}  // namespace bgv
