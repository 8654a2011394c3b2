// Batched form of the whole path: many independent graphs in one persistent launch.
// Each workgroup pops graphs from a queue (in the caller's order, e.g. largest first)
// and runs, with workgroup barriers only:
//   community passes (Section 3.2 rule, batch-synchronous chunks as in community.hip)
//   -> supernodes (ascending labels) -> sketch 1 in LDS -> inter-community keys ->
//   workgroup LSD radix sort -> superedges, sketch 2 in LDS, weights -> directed CSR ->
//   exact ForceAtlas2 iterations (Section 3.1 / Algorithm 1).
// The layout reproduces the plain exact path operation for operation: repulsion summed
// over j in order, the same per-row attraction wavefront, per-256-node partial sums of
// swing and traction in the plain kernels' fixed order, the same speed and move
// arithmetic (fa2_math.h).  Integer results equal the plain path's by construction.
#include <algorithm>

#include "block_scan.h"
#include "common.h"
#include "fa2_math.h"
#include "fa2_resident.h"
#include "sketch_hash.h"

namespace bgv {

constexpr int kBtMaxCells = 8192;  // rows*cols of a per-graph sketch, held in LDS
// Largest supergraph laid out by the multi-workgroup kernels after the persistent launch,
// and the repulsion segments it has at most (segment sums: that many per node).
constexpr int32_t kBtBigMax = 4096;
constexpr int32_t kBtMaxSeg = kBtBigMax / kRepSegment;

// An attraction item's workgroup holds the positions of a graph of up to this many nodes.
constexpr int32_t kBtAttPos = 2048;

constexpr int kBtIds = 8192;  // neighbour ids that a workgroup of the persistent launch holds on chip
static_assert(sizeof(ResidentLds<kBtIds>) <= sizeof(uint32_t) * kBtMaxCells, "fits where the sketch was");

struct BtArgs {
    int32_t G;
    const int64_t *node_off, *edge_off;  // device, G+1
    const int32_t *order;                // device, G, or null for 0..G-1
    const int2 *edges;                   // concatenated, local ids
    int32_t threshold, passes, growth, tie;
    int64_t chunk;
    int32_t rows;
    uint32_t cols;
    HashRows h1, h2;
    int32_t iters;
    float kr, kg, tau, ks, ksmax;
    // outputs (per-node arrays at node_off, per-edge arrays at edge_off)
    int32_t *labels, *degree, *K, *E, *super_label;
    uint32_t *super_size;
    int2 *superedges;
    uint32_t *se_weight;
    float2 *pos, *fprev;
    float *speed;
    // workspace
    int32_t *cnt, *lab, *prop, *row_base;
    unsigned long long *win;
    uint32_t *sid, *row;
    uint64_t *keyA, *keyB;  // 2 * m_total each
    uint32_t *cw;           // 2 * m_total neighbour ids (unit weights)
    float *mass;
    float2 *F, *att;
    double2 *vpart;         // floor(n_total/256) + G + 1
    unsigned int *queue;
    // graphs with more than big_k and at most kBtBigMax supernodes are listed in
    // big[0, *nbig) and laid out afterwards by the k_bt_* kernels; 0: none
    int32_t big_k;
    int32_t *big;
    unsigned int *nbig;
};

// Exclusive scan of in[0, n) into out (may alias); returns the total.
template <int NT>
__device__ uint32_t wg_scan(const uint32_t *in, uint32_t *out, int64_t n) {
    uint32_t carry = 0;
    for (int64_t t0 = 0; t0 < n; t0 += NT) {
        const int64_t i = t0 + threadIdx.x;
        const uint32_t v = i < n ? in[i] : 0u;
        uint32_t tot;
        const uint32_t e = block_excl_scan<uint32_t>(v, &tot);
        if (i < n) out[i] = carry + e;
        carry += tot;
    }
    return carry;
}

// Stable LSD radix sort of keys[0, n) on bits [0, nbits) by one workgroup, 8-bit digits.
// Returns the buffer holding the result (keys or alt).  A round takes kBtSortItems
// consecutive keys of each lane's wavefront: the wavefront ranks its keys by ballots into its
// own counters, one barrier, 256 threads turn the wavefronts' counts into places, one barrier,
// and the keys go out; the next round's keys are already on their way, and the next digit is
// counted on the way out.  What bounds it are the rounds' barriers: with one key per thread
// and round and a counting read per pass, the persistent launch of 512 planted graphs took
// 3.14 ms, so 2.88.
constexpr int kBtSortItems = 4;
template <int NT>
__device__ uint64_t *wg_radix_sort(uint64_t *keys, uint64_t *alt, int64_t n, int nbits, uint32_t (*hist)[256],
                                   uint32_t *running, uint32_t (*wcnt)[256]) {
    constexpr int NW = NT / kWave, R = kBtSortItems;
    const int t = threadIdx.x, lane = t & (kWave - 1), w = t / kWave;
    const uint64_t lt = lane ? (~0ull >> (64 - lane)) : 0ull;
    const int64_t mine = (int64_t)w * (R * kWave) + lane;  // of a round's keys, this thread's first
    uint64_t *src = keys, *dst = alt;
    for (int d = t; d < 2 * 256; d += NT) hist[0][d] = 0u;  // both rows
    __syncthreads();
    for (int64_t i = t; i < n; i += NT) atomicAdd(&hist[0][(uint32_t)src[i] & 255u], 1u);
    int cur = 0;
    for (int shift = 0; shift < nbits; shift += 8, cur ^= 1) {
        const bool more = shift + 8 < nbits;
        __syncthreads();
        uint32_t tot;
        const uint32_t e = block_excl_scan<uint32_t>(t < 256 ? hist[cur][t] : 0u, &tot);
        if (t < 256) {
            running[t] = e;
            hist[cur][t] = 0u;  // the pass after the next counts here
        }
        for (int d = t; d < NW * 256; d += NT) wcnt[0][d] = 0u;
        uint64_t key[R], next[R];
#pragma unroll
        for (int u = 0; u < R; ++u) next[u] = mine + u * kWave < n ? src[mine + u * kWave] : 0ull;
        __syncthreads();
        for (int64_t r0 = 0; r0 < n; r0 += (int64_t)NT * R) {
            uint32_t rank[R];
#pragma unroll
            for (int u = 0; u < R; ++u) {
                const int64_t ahead = r0 + (int64_t)NT * R + mine + u * kWave;
                key[u] = next[u];
                next[u] = ahead < n ? src[ahead] : 0ull;
            }
#pragma unroll
            for (int u = 0; u < R; ++u) {
                const bool valid = r0 + mine + u * kWave < n;
                const uint32_t d = (uint32_t)(key[u] >> shift) & 255u;
                uint64_t match = __ballot(valid);
#pragma unroll
                for (int b = 0; b < 8; ++b) {
                    const bool bit = (d >> b) & 1u;
                    const uint64_t bb = __ballot(bit);
                    match &= bit ? bb : ~bb;
                }
                rank[u] = 0u;
                if (valid) {
                    const uint32_t before = wcnt[w][d];
                    rank[u] = before + (uint32_t)__popcll(match & lt);
                    __builtin_amdgcn_wave_barrier();
                    if ((match & lt) == 0ull) wcnt[w][d] = before + (uint32_t)__popcll(match);
                }
                __builtin_amdgcn_wave_barrier();
            }
            __syncthreads();
            for (int d = t; d < 256; d += NT) {
                uint32_t c[NW], at = running[d];
#pragma unroll
                for (int q = 0; q < NW; ++q) c[q] = wcnt[q][d];
#pragma unroll
                for (int q = 0; q < NW; ++q) {
                    wcnt[q][d] = at;
                    at += c[q];
                }
                running[d] = at;
            }
            __syncthreads();
#pragma unroll
            for (int u = 0; u < R; ++u)
                if (r0 + mine + u * kWave < n) {
                    const uint32_t d = (uint32_t)(key[u] >> shift) & 255u;
                    dst[wcnt[w][d] + rank[u]] = key[u];
                    if (more) atomicAdd(&hist[cur ^ 1][(uint32_t)(key[u] >> (shift + 8)) & 255u], 1u);
                }
            __builtin_amdgcn_wave_barrier();
            for (int d = lane; d < 256; d += kWave) wcnt[w][d] = 0u;  // the wavefront's own
            __builtin_amdgcn_wave_barrier();
        }
        uint64_t *tmp = src;
        src = dst;
        dst = tmp;
    }
    __syncthreads();
    return src;
}

__device__ __forceinline__ int32_t bt_threshold(int32_t D1, int32_t growth, int32_t p) {
    int64_t D = D1;
    for (int32_t k = 0; k < p; ++k) {
        D *= growth;
        if (D > INT32_MAX) return INT32_MAX;
    }
    return (int32_t)D;
}

template <int NT>
__global__ void __launch_bounds__(NT) k_batched(BtArgs a) {
    constexpr int NW = NT / kWave;
    constexpr int NV = NT / 256;  // 256-node groups handled side by side in the layout
    static_assert(NT % 256 == 0 && NT <= 1024, "workgroup of 256, 512 or 1024 threads");
    static_assert(NT % kRepSegment == 0 || kRepSegment % NT == 0, "segment boundaries fall on LDS tile halves");
    __shared__ __align__(16) uint32_t sk[kBtMaxCells];
    __shared__ uint32_t hist[2][256], running[256];
    __shared__ uint32_t wcnt[NW][256];
    __shared__ float4 tile[NT];
    __shared__ double2 ws[NW];
    __shared__ int s_g;
    __shared__ uint32_t s_count;
    __shared__ float s_speed;
    const int t = threadIdx.x, lane = t & (kWave - 1), w = t / kWave;

    for (;;) {
        if (t == 0) s_g = (int)atomicAdd(a.queue, 1u);
        __syncthreads();
        const int qi = s_g;
        __syncthreads();
        if (qi >= a.G) break;
        const int g = a.order ? a.order[qi] : qi;
        const int64_t n0 = a.node_off[g], e0 = a.edge_off[g];
        const int32_t n = (int32_t)(a.node_off[g + 1] - n0);
        const int64_t m = a.edge_off[g + 1] - e0;
        const int2 *edges = a.edges + e0;
        int32_t *cnt = a.cnt + n0, *lab = a.lab + n0, *prop = a.prop + e0;
        unsigned long long *win = a.win + n0;
        uint32_t *sid = a.sid + n0;

        // ---- community passes, chunk by chunk -------------------------------------
        for (int32_t v = t; v < n; v += NT) {
            cnt[v] = 0;
            lab[v] = v;
            win[v] = ~0ull;
        }
        __syncthreads();
        // A chunk's steps are short and wait for each other, so where a thread has one edge
        // of it at most, the edge and its proposal stay in registers, a chunk's winners are
        // taken with the next one's increments (they touch different words), and labels are
        // read beside the counters: two barriers a chunk instead of three and half the chain
        // of reads (the persistent launch of 512 planted graphs, chunks of 256: 2.88 -> 2.70 ms).
        const bool one_each = a.chunk <= NT;
        for (int32_t pass = 0; one_each && pass < a.passes; ++pass) {
            const int32_t D = bt_threshold(a.threshold, a.growth, pass), chunk = (int32_t)a.chunk;
            int2 e = t < chunk && t < m ? edges[t] : make_int2(0, 0);
            int32_t x = -1;  // the chunk before's proposal of this thread, and its place in the stream
            uint32_t xi = 0;
            const auto take = [&] {
                if (x < 0) return;
                const unsigned long long wv = win[x];
                if ((uint32_t)(wv >> 32) == xi) {
                    lab[x] = (int32_t)(uint32_t)(wv & 0xffffffffull);
                    win[x] = ~0ull;
                }
            };
            for (int64_t cs = 0; cs < m; cs += chunk) {
                const bool edge = e.x != e.y;
                if (edge) {
                    __hip_atomic_fetch_add(&cnt[e.x], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                    __hip_atomic_fetch_add(&cnt[e.y], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                }
                take();
                __syncthreads();
                const int64_t ahead = cs + chunk + t;
                const int2 next = t < chunk && ahead < m ? edges[ahead] : make_int2(0, 0);
                x = -1;
                xi = (uint32_t)(cs + t);
                if (edge) {
                    const int32_t du = cnt[e.x], dv = cnt[e.y], lu = lab[e.x], lv = lab[e.y];
                    if (du <= D && dv <= D && (du != dv || a.tie)) {
                        const bool u_low = du <= dv;  // a tie (rule 1): the first endpoint joins
                        x = u_low ? e.x : e.y;
                        __hip_atomic_fetch_min(&win[x], ((unsigned long long)xi << 32) | (uint32_t)(u_low ? lv : lu),
                                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                    }
                }
                e = next;
                __syncthreads();
            }
            take();
            __syncthreads();
        }
        for (int32_t pass = 0; !one_each && pass < a.passes; ++pass) {
            const int32_t D = bt_threshold(a.threshold, a.growth, pass);
            for (int64_t cs = 0; cs < m; cs += a.chunk) {
                const int64_t ce = cs + a.chunk < m ? cs + a.chunk : m;
                for (int64_t i = cs + t; i < ce; i += NT) {
                    const int2 e = edges[i];
                    if (e.x != e.y) {
                        __hip_atomic_fetch_add(&cnt[e.x], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                        __hip_atomic_fetch_add(&cnt[e.y], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                    }
                }
                __syncthreads();
                for (int64_t i = cs + t; i < ce; i += NT) {
                    const int2 e = edges[i];
                    int32_t target = -1;
                    if (e.x != e.y) {
                        const int32_t du = cnt[e.x], dv = cnt[e.y];
                        if (du <= D && dv <= D && (du != dv || a.tie)) {
                            const bool u_low = du <= dv;  // a tie (rule 1): the first endpoint joins
                            target = u_low ? e.x : e.y;
                            const int32_t l = u_low ? lab[e.y] : lab[e.x];
                            __hip_atomic_fetch_min(&win[target], ((unsigned long long)i << 32) | (uint32_t)l,
                                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                        }
                    }
                    prop[i] = target;
                }
                __syncthreads();
                for (int64_t i = cs + t; i < ce; i += NT) {
                    const int32_t x = prop[i];
                    if (x >= 0) {
                        const unsigned long long wv = win[x];
                        if ((int64_t)(wv >> 32) == i) {
                            lab[x] = (int32_t)(uint32_t)(wv & 0xffffffffull);
                            win[x] = ~0ull;
                        }
                    }
                }
                __syncthreads();
            }
        }
        for (int32_t v = t; v < n; v += NT) {
            a.labels[n0 + v] = lab[v];
            a.degree[n0 + v] = cnt[v] / a.passes;
            sid[v] = 0u;
        }
        __syncthreads();

        // ---- supernodes: distinct labels in ascending order ---------------------
        for (int32_t v = t; v < n; v += NT) sid[lab[v]] = 1u;
        __syncthreads();
        uint32_t *flag = reinterpret_cast<uint32_t *>(win);  // free after the passes
        for (int32_t v = t; v < n; v += NT) flag[v] = sid[v];
        __syncthreads();
        const uint32_t K = wg_scan<NT>(sid, sid, n);
        int kb = 1;
        while (kb < 31 && (1u << kb) < K) ++kb;
        for (int32_t c = t; c < n; c += NT)
            if (flag[c]) a.super_label[n0 + sid[c]] = c;
        const int32_t cells = a.rows * (int32_t)a.cols;
        for (int32_t c = t; c < cells; c += NT) sk[c] = 0u;
        __syncthreads();

        // ---- sketch 1: community weights ------------------------------------------
        for (int32_t v = t; v < n; v += NT) {
            const uint32_t d = (uint32_t)(cnt[v] / a.passes);
            if (d == 0) continue;
            const uint32_t l = (uint32_t)lab[v];
            for (int r = 0; r < a.rows; ++r) atomicAdd(&sk[r * a.cols + col_key(a.h1.a[r], a.h1.b[r], l, a.cols)], d);
        }
        __syncthreads();
        for (uint32_t k = t; k < K; k += NT) {
            const uint32_t l = (uint32_t)a.super_label[n0 + k];
            uint32_t best = 0xffffffffu;
            for (int r = 0; r < a.rows; ++r) best = min(best, sk[r * a.cols + col_key(a.h1.a[r], a.h1.b[r], l, a.cols)]);
            a.super_size[n0 + k] = best;
        }
        __syncthreads();  // every read of sketch 1 is done before it is cleared for sketch 2
        if (t == 0) s_count = 0u;
        for (int32_t c = t; c < cells; c += NT) sk[c] = 0u;
        __syncthreads();

        // ---- inter-community keys, sorted -----------------------------------------
        uint64_t *keyA = a.keyA + 2 * e0, *keyB = a.keyB + 2 * e0;
        for (int64_t i = t; i < m; i += NT) {
            const int2 e = edges[i];
            if (e.x == e.y) continue;
            const int32_t la = lab[e.x], lb = lab[e.y];
            if (la == lb) continue;
            const uint32_t lo = (uint32_t)min(la, lb), hi = (uint32_t)max(la, lb);
            const uint32_t at = atomicAdd(&s_count, 1u);
            keyA[at] = ((uint64_t)sid[lo] << kb) | (uint64_t)sid[hi];
        }
        __syncthreads();
        const uint32_t nk = s_count;
        __syncthreads();
        const uint64_t *sorted = wg_radix_sort<NT>(keyA, keyB, nk, 2 * kb, hist, running, wcnt);

        // ---- superedges: distinct keys, multiplicities into sketch 2, weights -----
        const uint64_t lowmask = (1ull << kb) - 1ull;
        int2 *se = a.superedges + e0;
        uint32_t *run = reinterpret_cast<uint32_t *>(prop);  // run starts; prop is free now
        uint32_t E = 0;
        for (int64_t t0 = 0; t0 < nk; t0 += NT) {
            const int64_t i = t0 + t;
            const bool first = i < nk && (i == 0 || sorted[i] != sorted[i - 1]);
            uint32_t tot;
            const uint32_t j = E + block_excl_scan<uint32_t>(first ? 1u : 0u, &tot);
            if (first) {
                const uint64_t k = sorted[i];
                se[j] = make_int2((int32_t)(k >> kb), (int32_t)(k & lowmask));
                run[j] = (uint32_t)i;
            }
            E += tot;
        }
        __syncthreads();
        for (uint32_t j = t; j < E; j += NT) {
            const uint32_t c = (j + 1 < E ? run[j + 1] : nk) - run[j];
            const uint32_t la = (uint32_t)a.super_label[n0 + se[j].x], lb = (uint32_t)a.super_label[n0 + se[j].y];
            for (int r = 0; r < a.rows; ++r)
                atomicAdd(&sk[r * a.cols + col_pair(a.h2.a[r], a.h2.b[r], a.h2.c[r], la, lb, a.cols)], c);
        }
        __syncthreads();
        for (uint32_t j = t; j < E; j += NT) {
            const uint32_t la = (uint32_t)a.super_label[n0 + se[j].x], lb = (uint32_t)a.super_label[n0 + se[j].y];
            uint32_t best = 0xffffffffu;
            for (int r = 0; r < a.rows; ++r)
                best = min(best, sk[r * a.cols + col_pair(a.h2.a[r], a.h2.b[r], a.h2.c[r], la, lb, a.cols)]);
            a.se_weight[e0 + j] = best;
        }
        if (t == 0) {
            a.K[g] = (int32_t)K;
            a.E[g] = (int32_t)E;
        }

        // ---- directed CSR of the supergraph (neighbours ascending) ----------------
        for (uint32_t j = t; j < E; j += NT) {
            const int2 p = se[j];
            keyA[2 * j] = ((uint64_t)(uint32_t)p.x << kb) | (uint32_t)p.y;
            keyA[2 * j + 1] = ((uint64_t)(uint32_t)p.y << kb) | (uint32_t)p.x;
        }
        __syncthreads();
        const uint64_t *dk = wg_radix_sort<NT>(keyA, keyB, 2 * (int64_t)E, 2 * kb, hist, running, wcnt);
        uint32_t *row = a.row + n0 + g;
        uint32_t *cw = a.cw + 2 * e0;
        const int64_t nent = 2 * (int64_t)E;
        for (int64_t k = t; k < nent; k += NT) {
            const uint64_t key = dk[k];
            const int64_t src = (int64_t)(key >> kb);
            cw[k] = (uint32_t)(key & lowmask);
            const int64_t prev = k ? (int64_t)(dk[k - 1] >> kb) : -1;
            for (int64_t r = prev + 1; r <= src; ++r) row[r] = (uint32_t)k;
            if (k == nent - 1)
                for (int64_t r = src + 1; r <= (int64_t)K; ++r) row[r] = (uint32_t)nent;
        }
        if (nent == 0)
            for (uint32_t r = t; r <= K; r += NT) row[r] = 0u;
        __syncthreads();
        float *mass = a.mass + n0;
        for (uint32_t i = t; i < K; i += NT) mass[i] = (float)(row[i + 1] - row[i]) + 1.0f;
        if (a.big_k > 0 && a.iters > 0 && K > (uint32_t)a.big_k && K <= (uint32_t)kBtBigMax) {
            // a large supergraph is laid out by the multi-workgroup kernels afterwards,
            // so that it does not hold one compute unit for the whole layout
            if (t == 0) a.big[atomicAdd(a.nbig, 1u)] = g;
            __syncthreads();
            continue;
        }
        __syncthreads();
        if (NT >= kResidentMax && K <= (uint32_t)kResidentMax) {
            // the state on chip, where the sketch was
            constexpr int kThreads = NT >= kResidentMax ? NT : kResidentMax;
            ResidentLds<kBtIds> &lds = *reinterpret_cast<ResidentLds<kBtIds> *>(sk);
            if (resident_share<kThreads>((int32_t)K))
                fa2_resident<kThreads, true, true>(lds, (int32_t)K, a.iters, a.pos + n0, a.fprev + n0, mass, row, cw,
                                                   a.speed + g, a.kr, a.kg, a.tau, a.ks, a.ksmax);
            else
                fa2_resident<kThreads, true, false>(lds, (int32_t)K, a.iters, a.pos + n0, a.fprev + n0, mass, row, cw,
                                                    a.speed + g, a.kr, a.kg, a.tau, a.ks, a.ksmax);
            continue;
        }

        // ---- exact ForceAtlas2 iterations -------------------------------------------
        float2 *pos = a.pos + n0, *fprev = a.fprev + n0, *F = a.F + n0, *att = a.att + n0;
        double2 *vpart = a.vpart + (n0 / 256) + g;
        if (t == 0) s_speed = a.speed[g];
        __syncthreads();
        const int32_t nvb = (int32_t)((K + 255) / 256);
        for (int32_t it = 0; it < a.iters; ++it) {
            for (uint32_t i = w; i < K; i += NW) {
                const float2 f = fa2_row_attraction(pos, cw, row[i], row[i + 1], pos[i], lane);
                if (lane == 0) att[i] = f;
            }
            __syncthreads();
            for (int32_t vb0 = 0; vb0 < nvb; vb0 += NV) {
                const int32_t vb = vb0 + t / 256;
                const uint32_t i = (uint32_t)vb * 256u + (uint32_t)(t & 255);
                const bool live = vb < nvb && i < K;
                const float2 xi = live ? pos[i] : make_float2(0.f, 0.f);
                const float mi = live ? mass[i] : 0.f;
                // the plain kernels' order: segments of kRepSegment bodies, each summed
                // from zero, then added in order; a segment boundary can fall inside a tile
                float rx = 0.f, ry = 0.f, sx = 0.f, sy = 0.f;
                for (uint32_t j0 = 0; j0 < K; j0 += NT) {
                    const uint32_t j = j0 + t;
                    tile[t] = j < K ? fa2_body(pos[j], mass[j]) : fa2_no_body();
                    __syncthreads();
                    const uint32_t c = min((uint32_t)NT, K - j0);
                    for (uint32_t q0 = 0; q0 < c;) {
                        const uint32_t jj = j0 + q0;
                        if (jj != 0 && jj % (uint32_t)kRepSegment == 0) {
                            if (jj == (uint32_t)kRepSegment) {
                                rx = sx;
                                ry = sy;
                            } else {
                                rx += sx;
                                ry += sy;
                            }
                            sx = sy = 0.f;
                        }
                        const uint32_t q1 = min(c, (jj / (uint32_t)kRepSegment + 1u) * (uint32_t)kRepSegment - j0);
                        fa2_rep_run(xi, tile + q0, (int)((q1 - q0 + 7u) & ~7u), sx, sy);
                        q0 = q1;
                    }
                    __syncthreads();
                }
                if (K <= (uint32_t)kRepSegment) {
                    rx = sx;
                    ry = sy;
                } else {
                    rx += sx;
                    ry += sy;
                }
                double2 st = make_double2(0.0, 0.0);
                if (live) {
                    const float2 f = fa2_net_force(xi, mi, a.kr, rx, ry, att[i], a.kg);
                    F[i] = f;
                    st = fa2_swing_traction(f, fprev[i], mi);
                }
                st = fa2_sum256(st, ws);
                if ((t & 255) == 0 && vb < nvb) vpart[vb] = st;
            }
            __syncthreads();
            double2 acc = make_double2(0.0, 0.0);
            if (t < 256)
                for (int32_t p = t; p < nvb; p += 256) {
                    acc.x += vpart[p].x;
                    acc.y += vpart[p].y;
                }
            acc = fa2_sum256(acc, ws);
            if (t == 0) s_speed = fa2_global_speed(acc.x, acc.y, s_speed, a.tau);
            __syncthreads();
            const float s = s_speed;
            for (uint32_t i = t; i < K; i += NT) {
                const float2 f = F[i];
                pos[i] = fa2_move(pos[i], f, fprev[i], s, a.ks, a.ksmax);
                fprev[i] = f;
            }
            __syncthreads();
        }
        if (t == 0) a.speed[g] = s_speed;
        __syncthreads();
    }
}

// ---- layout of the listed large graphs, all of them per launch ------------------
// Work items are (64-node wave tile, repulsion segment) pairs for the repulsion and wave
// tiles for the attraction, in tables made once per call.  Each node's sums are those of
// the plain path in the same order, so a graph's result equals a plain layout of it bit
// for bit.
struct BtBig {
    const int64_t *node_off, *edge_off;
    const int32_t *K;
    const int32_t *big;
    const unsigned int *nbig;
    uint32_t *fitem_off, *aitem_off;  // G+1 each: prefix sums of the pairs / wave tiles over the list
    uint32_t *total;                  // (pairs, wave tiles, graphs)
    uint4 *graph;                     // per slot: first node, K, g, where its last segment's pairs start in fitem
    uint32_t *fpos;                   // per slot: where its whole segments' pairs start there
    uint4 *fitem;                     // (first node, K, wave tile, segment) of every pair, longest segments first
    uint4 *aitem;                     // (first node, K, wave tile, g) of every attraction item
    const uint32_t *row;
    const uint32_t *cw;
    const float *mass;
    float2 *pos, *fprev, *att;
    float2 *seg;  // segment sums: kBtMaxSeg per node from the graph's first node
    float *speed;
    float kr, kg, tau, ks, ksmax;
};

// Prefix sums of the items over the list, and the places of every graph's pairs in the
// order of falling segment length (32 classes; the order inside one does not matter).
__global__ void __launch_bounds__(1024) k_bt_plan(BtBig b) {
    const uint32_t nb = *b.nbig;
    uint32_t cf = 0, ca = 0;
    for (uint32_t s0 = 0; s0 < nb; s0 += 1024) {
        const uint32_t sl = s0 + threadIdx.x;
        uint32_t wt = 0, segs = 0;
        if (sl < nb) {
            const int32_t K = b.K[b.big[sl]];
            wt = (uint32_t)((K + kWave - 1) / kWave);
            segs = (uint32_t)fa2_rep_segments(K);
        }
        uint32_t tf, ta;
        const uint32_t ef = block_excl_scan<uint32_t>(wt * segs, &tf);
        const uint32_t ea = block_excl_scan<uint32_t>(wt, &ta);
        if (sl < nb) {
            b.fitem_off[sl] = cf + ef;
            b.aitem_off[sl] = ca + ea;
        }
        cf += tf;
        ca += ta;
    }
    if (threadIdx.x == 0) {
        b.fitem_off[nb] = cf;
        b.aitem_off[nb] = ca;
        b.total[0] = cf;
        b.total[1] = ca;
        b.total[2] = nb;
    }
    constexpr uint32_t kWidth = kRepSegment / 32;
    __shared__ uint32_t at[32];
    if (threadIdx.x < 32) at[threadIdx.x] = 0u;
    __syncthreads();
    for (uint32_t sl = threadIdx.x; sl < nb; sl += 1024) {
        const uint32_t K = (uint32_t)b.K[b.big[sl]], wt = (K + kWave - 1) / kWave, rest = K % kRepSegment;
        if (K >= (uint32_t)kRepSegment) atomicAdd(&at[0], wt * (K / kRepSegment));
        if (rest) atomicAdd(&at[(kRepSegment - rest) / kWidth], wt);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t run = 0;
        for (int c = 0; c < 32; ++c) {
            const uint32_t n = at[c];
            at[c] = run;
            run += n;
        }
    }
    __syncthreads();
    for (uint32_t sl = threadIdx.x; sl < nb; sl += 1024) {
        const int32_t g = b.big[sl];
        const uint32_t K = (uint32_t)b.K[g], wt = (K + kWave - 1) / kWave, rest = K % kRepSegment;
        b.fpos[sl] = K >= (uint32_t)kRepSegment ? atomicAdd(&at[0], wt * (K / kRepSegment)) : 0u;
        b.graph[sl] = make_uint4((uint32_t)b.node_off[g], K, (uint32_t)g,
                                 rest ? atomicAdd(&at[(kRepSegment - rest) / kWidth], wt) : 0u);
    }
}

// Largest slot s with off[s] <= x (off ascending, off[0] = 0, x < off[nb]).
__device__ __forceinline__ uint32_t bt_slot(const uint32_t *off, uint32_t nb, uint32_t x) {
    uint32_t lo = 0, hi = nb;  // off[lo] <= x < off[hi]
    while (hi - lo > 1) {
        const uint32_t mid = (lo + hi) / 2;
        if (off[mid] <= x) lo = mid;
        else hi = mid;
    }
    return lo;
}

// The items of both tables.
__global__ void __launch_bounds__(256) k_bt_maps(BtBig b) {
    const uint32_t FI = b.total[0], AI = b.total[1], nb = b.total[2];
    const uint32_t stride = gridDim.x * 256, t = blockIdx.x * 256 + threadIdx.x;
    for (uint32_t x = t; x < FI; x += stride) {
        const uint32_t sl = bt_slot(b.fitem_off, nb, x), q = x - b.fitem_off[sl];
        const uint4 d = b.graph[sl];
        const uint32_t wt = (d.y + kWave - 1) / kWave, whole = wt * (d.y / kRepSegment);
        b.fitem[q < whole ? b.fpos[sl] + q : d.w + (q - whole)] = make_uint4(d.x, d.y, q % wt, q / wt);
    }
    for (uint32_t x = t; x < AI; x += stride) {
        const uint32_t sl = bt_slot(b.aitem_off, nb, x);
        const uint4 d = b.graph[sl];
        b.aitem[x] = make_uint4(d.x, d.y, x - b.aitem_off[sl], d.z);
    }
}

// Repulsion of one (64-target wave tile, segment) item by one wavefront: the segment's
// bodies pass through the wavefront's own LDS slice 64 at a time and every lane adds
// them in ascending order, the same additions as the 256-target tiles of the plain path
// (a target's sum does not depend on which targets share its tile), into the segment
// sums seg[s * K + i].  Targets are grouped by 64 so that small supergraphs leave few
// lanes idle.
__device__ __forceinline__ void bt_wave_repulsion(int32_t wt, int32_t sgm, int32_t K, const float2 *__restrict__ pos,
                                                  const float *__restrict__ mass, float2 *__restrict__ seg,
                                                  float4 *slab) {
    const int lane = threadIdx.x & (kWave - 1);
    const int32_t i = wt * kWave + lane;
    const bool live = i < K;
    const float2 xi = live ? pos[i] : make_float2(0.f, 0.f);
    const int32_t jb = sgm * kRepSegment, je = min(K, jb + kRepSegment);
    float fx = 0.f, fy = 0.f;
    // the next bodies are loaded while these are used
    float4 next = jb + lane < je ? fa2_body(pos[jb + lane], mass[jb + lane]) : fa2_no_body();
    for (int32_t t0 = jb; t0 < je; t0 += kWave) {
        slab[lane] = next;
        const int32_t j = t0 + kWave + lane;
        next = j < je ? fa2_body(pos[j], mass[j]) : fa2_no_body();
        __builtin_amdgcn_wave_barrier();
        fa2_rep_run(xi, slab, min(kWave, (je - t0 + 7) & ~7), fx, fy);
        __builtin_amdgcn_wave_barrier();
    }
    if (live) seg[(int64_t)sgm * K + i] = make_float2(fx, fy);
}

// The first rep_blocks workgroups sum repulsion: their wavefronts share out the pairs,
// longest first, back and forth, so that each gets about the same number of terms whatever
// the graphs' sizes.  The others take the attraction of a wave tile's rows each, the
// graph's positions in LDS: read from memory for every entry, they took longer than the
// repulsion (47 against 31 us).  A graph of one segment takes the same path: its one
// segment sum is its repulsion.  Bound by the repulsion's vector issue: 512 planted graphs
// (74M pairs, 4.5M row entries per iteration) take 33.1 us, the repulsion alone 30.6; with
// entries of 8 bytes (id and weight) instead of 4, 40.6; a wavefront per item and then per
// row in one grid took 48.4.
__global__ void __launch_bounds__(kFa2Tile) k_bt_force(BtBig b, uint32_t rep_blocks) {
    __shared__ __align__(16) float2 xs[kBtAttPos];
    __shared__ uint32_t rows[kWave + 1];
    constexpr int NW = kFa2Tile / kWave;
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    if (blockIdx.x < rep_blocks) {
        float4 *slab = reinterpret_cast<float4 *>(xs) + w * kWave;
        const uint32_t FI = b.total[0], nw = rep_blocks * NW, x0 = blockIdx.x * NW + w;
        for (uint32_t base = 0, round = 0; base < FI; base += nw, ++round) {
            const uint32_t x = base + (round & 1u ? nw - 1u - x0 : x0);
            if (x >= FI) continue;
            const uint4 it = b.fitem[x];
            bt_wave_repulsion((int32_t)it.z, (int32_t)it.w, (int32_t)it.y, b.pos + it.x, b.mass + it.x,
                              b.seg + (int64_t)kBtMaxSeg * it.x, slab);
        }
        return;
    }
    const uint32_t AI = b.total[1];
    for (uint32_t x = blockIdx.x - rep_blocks; x < AI; x += gridDim.x - rep_blocks) {
        const uint4 it = b.aitem[x];
        const int64_t n0 = it.x;
        const int32_t g = (int32_t)it.w, K = (int32_t)it.y, r0 = (int32_t)it.z * kWave, nr = min(kWave, K - r0);
        const uint32_t *row = b.row + n0 + g + r0;
        const uint32_t *cw = b.cw + 2 * b.edge_off[g];
        const float2 *pos = b.pos + n0;
        if (threadIdx.x <= (uint32_t)nr) rows[threadIdx.x] = row[threadIdx.x];
        if (K <= kBtAttPos)
            for (int32_t i = threadIdx.x; i < K; i += kFa2Tile) xs[i] = pos[i];
        __syncthreads();
        if (K <= kBtAttPos)
            fa2_rows_attraction((const float2 *)xs, cw, rows, r0, nr, b.att + n0 + r0, w, NW, lane);
        else
            fa2_rows_attraction(pos, cw, rows, r0, nr, b.att + n0 + r0, w, NW, lane);
        __syncthreads();
    }
}

constexpr int kBtStep = 512;  // 256 threads 15.5 us, 1,024 10.0
// One workgroup per listed graph: segment sums added in order, the rest of every force, the
// 256-node tiles' partial sums, the global speed and the moves.  Two launches with a
// workgroup per tile took 10.9 us, this one 9.0: its chain of dependent loads.
__global__ void __launch_bounds__(kBtStep) k_bt_step(BtBig b) {
    constexpr int NW = kBtStep / kWave, kRounds = kBtBigMax / kBtStep;
    static_assert(kRounds * NW == kWave, "a lane per wavefront sum");
    __shared__ double2 ws[kWave];
    const int t = threadIdx.x, lane = t & (kWave - 1), w = t / kWave;
    const uint32_t nb = b.total[2];
    for (uint32_t sl = blockIdx.x; sl < nb; sl += gridDim.x) {
        const uint4 d = b.graph[sl];
        const int64_t n0 = d.x;
        const int32_t K = (int32_t)d.y, nseg = fa2_rep_segments(K);
        const float2 *seg = b.seg + kBtMaxSeg * n0;
        float s = b.speed[d.z];
        float2 xi[kRounds], fp[kRounds], f[kRounds];
#pragma unroll
        for (int q = 0; q < kRounds; ++q) {
            const int32_t i = q * kBtStep + t;
            double2 st = make_double2(0.0, 0.0);
            if (q * kBtStep + w * kWave < K) {  // whole wavefronts without a node add nothing
                if (i < K) {
                    const float mi = b.mass[n0 + i];
                    const float2 at = b.att[n0 + i];
                    xi[q] = b.pos[n0 + i];
                    fp[q] = b.fprev[n0 + i];
                    float2 v[kBtMaxSeg];  // all loads before the first sum
#pragma unroll
                    for (int32_t u = 0; u < kBtMaxSeg; ++u)
                        if (u < nseg) v[u] = seg[(int64_t)u * K + i];
                    float2 r = v[0];
#pragma unroll
                    for (int32_t u = 1; u < kBtMaxSeg; ++u)
                        if (u < nseg) {
                            r.x += v[u].x;
                            r.y += v[u].y;
                        }
                    f[q] = fa2_net_force(xi[q], mi, b.kr, r.x, r.y, at, b.kg);
                    st = fa2_swing_traction(f[q], fp[q], mi);
                }
                st.x = fa2_wave_sum(st.x);
                st.y = fa2_wave_sum(st.y);
            }
            if (lane == 0) ws[q * NW + w] = st;
        }
        __syncthreads();
        if (w * kWave < K) {
            // every wavefront for itself: a tile's four wavefront sums in order, then the tiles'
            // as one wavefront of the plain kernel sums them (its other three hold zeros)
            double2 acc = make_double2(0.0, 0.0);
            if (lane < kWave / 4)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    acc.x += ws[4 * lane + q].x;
                    acc.y += ws[4 * lane + q].y;
                }
            acc.x = fa2_wave_sum(acc.x);
            acc.y = fa2_wave_sum(acc.y);
            s = fa2_global_speed(acc.x, acc.y, s, b.tau);
#pragma unroll
            for (int q = 0; q < kRounds; ++q) {
                const int32_t i = q * kBtStep + t;
                if (i < K) {
                    b.pos[n0 + i] = fa2_move(xi[q], f[q], fp[q], s, b.ks, b.ksmax);
                    b.fprev[n0 + i] = f[q];
                }
            }
        }
        __syncthreads();  // LDS is reused by the next graph; every thread has read the speed
        if (t == 0) b.speed[d.z] = s;
    }
}

struct BtWs {
    int32_t *cnt, *lab, *prop;
    unsigned long long *win;
    uint32_t *sid, *row;
    uint64_t *keyA, *keyB;
    uint32_t *cw;
    float *mass;
    float2 *F, *att;
    double2 *vpart;
    unsigned int *queue;
    int32_t *big;
    unsigned int *nbig;
    uint32_t *fitem_off, *aitem_off;
    uint32_t *total, *fpos;
    uint4 *graph, *fitem, *aitem;
    float2 *seg;
};

static size_t bt_layout(Carver &c, int32_t G, int64_t n_total, int64_t m_total, BtWs *w) {
    const size_t n = (size_t)(n_total > 0 ? n_total : 1), m = (size_t)(m_total > 0 ? m_total : 1);
    w->cnt = c.take<int32_t>(n);
    w->lab = c.take<int32_t>(n);
    w->win = c.take<unsigned long long>(n);
    w->sid = c.take<uint32_t>(n);
    w->prop = c.take<int32_t>(m);
    w->keyA = c.take<uint64_t>(2 * m);
    w->keyB = c.take<uint64_t>(2 * m);
    w->cw = c.take<uint32_t>(2 * m);
    w->row = c.take<uint32_t>(n + (size_t)G);
    w->mass = c.take<float>(n);
    w->F = c.take<float2>(n);
    w->att = c.take<float2>(n);
    w->vpart = c.take<double2>(n / 256 + (size_t)G + 1);
    w->queue = c.take<unsigned int>(1);
    w->big = c.take<int32_t>((size_t)G);
    w->nbig = c.take<unsigned int>(1);
    w->fitem_off = c.take<uint32_t>((size_t)G + 1);
    w->aitem_off = c.take<uint32_t>((size_t)G + 1);
    // a listed graph has K <= kBtBigMax supernodes: at most kBtMaxSeg segments of K / 64 + 1 wave tiles
    w->fitem = c.take<uint4>((size_t)kBtMaxSeg * (n / kWave + (size_t)G + 1));
    w->aitem = c.take<uint4>(n / kWave + (size_t)G + 1);
    w->fpos = c.take<uint32_t>((size_t)G);
    w->graph = c.take<uint4>((size_t)G);
    w->total = c.take<uint32_t>(3);
    w->seg = c.take<float2>((size_t)kBtMaxSeg * n);
    return c.size();
}

static bool bt_valid(int32_t G, int64_t n_total, int64_t m_total, const bgv_cd_params *cd,
                     const bgv_sketch_params *sk, const bgv_fa2_params *fa) {
    return G >= 1 && n_total >= 0 && n_total <= INT32_MAX && m_total >= 0 && m_total <= INT32_MAX && cd && sk &&
           fa && cd->threshold >= 0 && cd->passes >= 1 && cd->growth >= 1 && cd->chunk >= 1 && cd->method == 0 &&
           (cd->tie == 0 || cd->tie == 1) && cd->rule == 0 &&
           sk->rows >= 1 && sk->rows <= kMaxRows && sk->cols >= 1 && (int64_t)sk->rows * sk->cols <= kBtMaxCells &&
           sk->coef1 && sk->coef2 && fa->iters >= 0 && fa->exact == 1 && fa->tau > 0.f && fa->ks >= 0.f &&
           fa->ksmax > 0.f;
}

}  // namespace bgv

using namespace bgv;

extern "C" size_t bgv_batched_workspace(int32_t G, int64_t n_total, int64_t m_total) {
    if (G < 1 || n_total < 0 || m_total < 0) return 0;
    Carver c(nullptr);
    BtWs w;
    return bt_layout(c, G, n_total, m_total, &w);
}

extern "C" bgv_status bgv_batched(int32_t G, int64_t n_total, int64_t m_total, const int64_t *node_off,
                                  const int64_t *edge_off, const int32_t *order, const int32_t *edges,
                                  const bgv_cd_params *cd, const bgv_sketch_params *sk, const bgv_fa2_params *fa,
                                  int32_t wg_threads, int32_t big_k, int32_t *labels, int32_t *degree, int32_t *K, int32_t *E_S,
                                  int32_t *super_label, uint32_t *super_size, int32_t *superedges,
                                  uint32_t *se_weight, float *pos, float *fprev, float *speed, void *ws,
                                  size_t ws_bytes, bgv_stream_t stream) {
    clear_error();
    if (!bt_valid(G, n_total, m_total, cd, sk, fa)) {
        set_error("bgv_batched: invalid arguments (G=%d n_total=%lld m_total=%lld)", G, (long long)n_total,
                  (long long)m_total);
        return BGV_E_INVALID;
    }
    if (big_k < 0) {
        set_error("bgv_batched: big_k must be >= 0 (got %d)", big_k);
        return BGV_E_INVALID;
    }
    if (wg_threads == 0) wg_threads = 512;
    if (wg_threads != 256 && wg_threads != 512 && wg_threads != 1024) {
        set_error("bgv_batched: wg_threads must be 0, 256, 512 or 1024 (got %d)", wg_threads);
        return BGV_E_INVALID;
    }
    if (!node_off || !edge_off || (m_total > 0 && (!edges || !superedges || !se_weight)) || !labels || !degree ||
        !K || !E_S || !super_label || !super_size || !pos || !fprev || !speed) {
        set_error("bgv_batched: null pointer");
        return BGV_E_INVALID;
    }
    BGV_TRY(check_ws(ws, ws_bytes, bgv_batched_workspace(G, n_total, m_total)));
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    if (range_check_on()) {  // K[0] holds the flag; it is written below
        BGV_TRY(check_batched_ids(G, n_total, m_total, node_off, edge_off, edges, K, s));
        if (order) BGV_TRY(check_id_list(G, order, G, K, s));
    }
    Carver c(ws);
    BtWs w;
    bt_layout(c, G, n_total, m_total, &w);

    BtArgs a{};
    a.G = G;
    a.node_off = node_off;
    a.edge_off = edge_off;
    a.order = order;
    a.edges = reinterpret_cast<const int2 *>(edges);
    a.threshold = cd->threshold;
    a.passes = cd->passes;
    a.growth = cd->growth;
    a.tie = cd->tie;
    a.chunk = cd->chunk;
    a.rows = sk->rows;
    a.cols = (uint32_t)sk->cols;
    a.h1 = make_hash_rows(sk->coef1, sk->rows);
    a.h2 = make_hash_rows(sk->coef2, sk->rows);
    a.iters = fa->iters;
    a.kr = fa->kr;
    a.kg = fa->kg;
    a.tau = fa->tau;
    a.ks = fa->ks;
    a.ksmax = fa->ksmax;
    a.labels = labels;
    a.degree = degree;
    a.K = K;
    a.E = E_S;
    a.super_label = super_label;
    a.super_size = super_size;
    a.superedges = reinterpret_cast<int2 *>(superedges);
    a.se_weight = se_weight;
    a.pos = reinterpret_cast<float2 *>(pos);
    a.fprev = reinterpret_cast<float2 *>(fprev);
    a.speed = speed;
    a.cnt = w.cnt;
    a.lab = w.lab;
    a.prop = w.prop;
    a.win = w.win;
    a.sid = w.sid;
    a.row = w.row;
    a.keyA = w.keyA;
    a.keyB = w.keyB;
    a.cw = w.cw;
    a.mass = w.mass;
    a.F = w.F;
    a.att = w.att;
    a.vpart = w.vpart;
    a.queue = w.queue;
    a.big_k = big_k;
    a.big = w.big;
    a.nbig = w.nbig;

    int cus = 1;
    BGV_TRY(device_cu_count(&cus));
    const int per_cu = wg_threads == 1024 ? 1 : 2;
    const int grid = G < cus * per_cu ? G : cus * per_cu;
    BGV_TRY(fill<uint32_t>(w.queue, 0u, 1, s));
    BGV_TRY(fill<uint32_t>(w.nbig, 0u, 1, s));
    switch (wg_threads) {
        case 256: BGV_LAUNCH(k_batched<256>, dim3(grid), dim3(256), 0, s, a); break;
        case 512: BGV_LAUNCH(k_batched<512>, dim3(grid), dim3(512), 0, s, a); break;
        default: BGV_LAUNCH(k_batched<1024>, dim3(grid), dim3(1024), 0, s, a); break;
    }
    if (big_k > 0 && fa->iters > 0) {
        // the listed large graphs: a fixed sequence of launches whose sizes are read on
        // the device, so the whole call can still be captured in a graph
        BtBig b{};
        b.node_off = node_off;
        b.edge_off = edge_off;
        b.K = K;
        b.big = w.big;
        b.nbig = w.nbig;
        b.fitem_off = w.fitem_off;
        b.aitem_off = w.aitem_off;
        b.fitem = w.fitem;
        b.aitem = w.aitem;
        b.fpos = w.fpos;
        b.graph = w.graph;
        b.total = w.total;
        b.seg = w.seg;
        b.row = w.row;
        b.cw = w.cw;
        b.mass = w.mass;
        b.pos = a.pos;
        b.fprev = a.fprev;
        b.att = w.att;
        b.speed = speed;
        b.kr = fa->kr;
        b.kg = fa->kg;
        b.tau = fa->tau;
        b.ks = fa->ks;
        b.ksmax = fa->ksmax;
        // Two wavefronts per SIMD for the repulsion, whose items are few and long (three:
        // 15.5 -> 16.6 ms for 300 iterations); as many attraction workgroups as it has items
        // or up to 14 per compute unit (eight are no slower).
        const unsigned rep_blocks = 2u * (unsigned)cus;
        const unsigned att_blocks = (unsigned)std::min<int64_t>(n_total / kWave + G, 14 * cus);
        BGV_LAUNCH(k_bt_plan, dim3(1), dim3(1024), 0, s, b);
        BGV_LAUNCH(k_bt_maps, dim3(grid_for(n_total > 0 ? n_total : 1, 256, 1024)), dim3(256), 0, s, b);
        for (int32_t it = 0; it < fa->iters; ++it) {
            BGV_LAUNCH(k_bt_force, dim3(rep_blocks + att_blocks), dim3(kFa2Tile), 0, s, b, rep_blocks);
            BGV_LAUNCH(k_bt_step, dim3((unsigned)std::min(G, 2048 / kBtStep * cus)), dim3(kBtStep), 0, s, b);
        }
    }
    return BGV_OK;
}
