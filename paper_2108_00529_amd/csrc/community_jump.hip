// Streaming community detection without a barrier per chunk (the rule of Section 3.2,
// the passes of Section 3.2.1 / Algorithm 3, batch-synchronous as in community.hip:
// the same integers for every chunk size, chunk = 1 being the sequential rule).
//
// Under the degree rule an edge's decision in a pass (whether it proposes, and which
// endpoint is the target) depends only on counters, and those follow in closed form
// from the stream: in pass p at the end of chunk k the counter of x is p d(x) + c(x, k),
// with c(x, k) the occurrences of x as an endpoint of a non-loop edge in chunks 0..k.
// Labels enter only as the value a proposal carries (its source's label when the chunk
// began).  So every pass's proposals are known up front; a target's winner in a chunk
// is its proposal of smallest stream index; and the label a winner carries is the one
// its source got from its own latest winner in an earlier chunk (the source's id if it
// had none).  Those links point strictly back in time, and pointer jumping over them
// labels every winner in O(log chunks) bulk steps:
//   1. endpoint occurrences sorted by node (stable): d(x) = run length, c(x, k) of each
//      occurrence by a binary search in its node's run;
//   2. the proposals of every (pass, edge), compacted in (pass, stream) order and sorted
//      stably by target: a proposal is its time t = pass * m + edge, so a target's
//      proposals come in time order and the first of each of its chunks is the winner;
//   3. winners compacted; each one's link = the last winner into its source with an
//      earlier chunk (a binary search in the source's run of winners: before its chunk's
//      first time);
//   4. pointer jumping along the links, in place on packed (link, label) words, several
//      links a round, each round skipped once a round has left nothing unresolved; a
//      node's label = its last winner's label.
// About 25 launches whatever the number of chunks, against two per chunk and pass for
// the chunk-by-chunk form: the choice for small chunks.
//
// What bounds it: the three passes over 8-byte (key, value) pairs of each sort (HBM), and
// the random accesses that no order avoids: each occurrence's count written to its edge,
// and per winner its edge, its source's run and the probes there.  Sorting by the target
// alone (20 bits of 45 for 1M nodes and chunk 1) halves the second sort, and 4-byte times
// in place of 8-byte (target, chunk) keys its traffic; proposals and winners are numbered
// by counting per 512 of them and again when they are written, so that no flag per (pass,
// edge) is stored or scanned.  1M nodes, 10M edges, 3 passes, chunk 1:
// 4.42 -> 2.54 ms against 8-byte keys sorted by all their bits and flags per (pass, edge).
#include <algorithm>

#include "common.h"
#include "community_jump.h"
#include "volume_sum.h"

namespace bgv {

constexpr int kSqThreads = 256;
constexpr int kSqMaxRounds = 66;  // ceil(log2 chunks) + 1 <= 34 for 32-bit proposal indices

static int bits_for(uint64_t x) {  // bits needed to hold values 0..x
    int b = 0;
    while (b < 64 && (x >> b) != 0) ++b;
    return b;
}

// D1 * growth^p, saturating at INT32_MAX (at most ~31 products before it saturates).
__host__ __device__ inline int32_t sq_threshold(int32_t D1, int32_t growth, int32_t p) {
    if (growth == 1 || D1 == 0) return D1;
    int64_t D = D1;
    for (int32_t k = 0; k < p; ++k) {
        D *= growth;
        if (D > INT32_MAX) return INT32_MAX;
    }
    return (int32_t)D;
}

bool sq_fits(int32_t n, int64_t m, const bgv_cd_params *p) {
    if (m < 1) return false;
    const int64_t nchunk = (m + p->chunk - 1) / p->chunk;
    if ((int64_t)p->passes * m > INT32_MAX) return false;  // proposals indexed in 32 bits
    const uint64_t G = (uint64_t)p->passes * (uint64_t)nchunk;
    return bits_for((uint64_t)(n - 1)) + bits_for(G - 1) <= 64;
}

constexpr int kSqRounds = 8;                       // edges or events per lane of a wavefront's tile
constexpr int64_t kSqTile = kWave * kSqRounds;     // consecutive edges or events per wavefront
constexpr int32_t kSqLeastPasses = 16;             // passes per wavefront at least
constexpr int kSqHops = 15;                        // links followed per pointer-jumping round

struct SqWs {
    uint32_t *okey, *okey_alt, *oval, *oval_alt;  // endpoint occurrences [2m]
    uint2 *run;                                   // run of each node in the sorted occurrences [n]
    uint2 *wrun;                                  // run of each node in the winners [n]
    int32_t *cc;                                  // c of each endpoint occurrence [2m]
    uint32_t *tally;                              // proposals per (pass, tile of edges), then per tile of events
    uint32_t *ekey, *ekey_alt;                    // proposals' targets [P m]; the unused one then holds the winners'
    uint32_t *etime, *etime_alt;                  // their times; likewise
    unsigned long long *jv;                       // per winner: label << 32 | link (link ~0: resolved) [P m]
    int32_t *go;                                  // [kSqMaxRounds + 1]: round r runs if go[r]
    uint32_t *tot;                                // [2]: winners
    unsigned long long *ne;                       // proposals
    void *osort, *esort, *scan_scratch;
};

static int64_t sq_tiles(int64_t count) { return (count + kSqTile - 1) / kSqTile; }

size_t sq_layout(Carver &c, int32_t n, int64_t m, const bgv_cd_params *p, void *out) {
    SqWs w{};
    const size_t no = 2 * (size_t)m, pm = (size_t)p->passes * (size_t)m;
    const int nbits = bits_for((uint64_t)n);
    const int64_t tally = std::max<int64_t>((int64_t)p->passes * sq_tiles(m), sq_tiles((int64_t)pm)) + 1;
    w.okey = c.take<uint32_t>(no);
    w.okey_alt = c.take<uint32_t>(no);
    w.oval = c.take<uint32_t>(no);
    w.oval_alt = c.take<uint32_t>(no);
    w.run = c.take<uint2>((size_t)n);
    w.wrun = c.take<uint2>((size_t)n);
    w.cc = c.take<int32_t>(no);
    w.tally = c.take<uint32_t>((size_t)tally);
    w.ekey = c.take<uint32_t>(pm);
    w.ekey_alt = c.take<uint32_t>(pm);
    w.etime = c.take<uint32_t>(pm);
    w.etime_alt = c.take<uint32_t>(pm);
    w.jv = c.take<unsigned long long>(pm);
    w.go = c.take<int32_t>(kSqMaxRounds + 1);
    w.tot = c.take<uint32_t>(2);
    w.ne = c.take<unsigned long long>(1);
    w.osort = c.take<char>(sort_workspace((int64_t)no, nbits));
    w.esort = c.take<char>(sort_workspace((int64_t)pm, nbits));
    w.scan_scratch = c.take<char>(scan_workspace(tally));
    if (out) *static_cast<SqWs *>(out) = w;
    // a caller may size its buffer by 48 bytes per edge and 40 per (pass, edge): the query
    // never asks for less
    return std::max(c.size(), 48 * (size_t)m + 40 * pm);
}

// ------------------------------------------------------------------ kernels ----
#define SQ_LOOP(i, count) \
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < (count); i += (int64_t)gridDim.x * blockDim.x)

// Occurrence 2i + s is endpoint s of edge i, keyed by its node (self-loops by n, past
// every node: they raise no counter).  Also clears the runs and the rounds' flags (round
// 0 runs).
__global__ void __launch_bounds__(kSqThreads) k_sq_occ(const int2 *__restrict__ edges, int64_t m, int32_t n,
                                                       uint2 *__restrict__ okey, uint2 *__restrict__ oval,
                                                       uint2 *__restrict__ run, uint2 *__restrict__ wrun,
                                                       int32_t *__restrict__ go, int32_t rounds) {
    SQ_LOOP(i, m) {
        const int2 e = edges[i];
        const bool loop = e.x == e.y;
        okey[i] = make_uint2(loop ? (uint32_t)n : (uint32_t)e.x, loop ? (uint32_t)n : (uint32_t)e.y);
        oval[i] = make_uint2((uint32_t)(2 * i), (uint32_t)(2 * i + 1));
    }
    SQ_LOOP(v, n) run[v] = wrun[v] = make_uint2(0u, 0u);
    SQ_LOOP(r, rounds + 1) go[r] = r == 0;
}

__global__ void __launch_bounds__(kSqThreads) k_sq_runs(const uint32_t *__restrict__ sk, int64_t no, int32_t n,
                                                        uint2 *__restrict__ run) {
    SQ_LOOP(j, no) {
        const uint32_t x = sk[j];
        if (x >= (uint32_t)n) continue;
        if (j == 0 || sk[j - 1] != x) run[x].x = (uint32_t)j;
        if (j + 1 == no || sk[j + 1] != x) run[x].y = (uint32_t)(j + 1);
    }
}

// c(x, k) of each occurrence: the occurrences of x before the end of its chunk, i.e.
// the first place in x's run (occurrences in stream order) at or past that end.
__global__ void __launch_bounds__(kSqThreads) k_sq_counts(const uint32_t *__restrict__ sk,
                                                          const uint32_t *__restrict__ sv, int64_t no, int32_t n,
                                                          const uint2 *__restrict__ run, uint32_t m, uint32_t B,
                                                          int32_t *__restrict__ cc) {
    SQ_LOOP(j, no) {
        const uint32_t x = sk[j];
        if (x >= (uint32_t)n) continue;
        const uint32_t o = sv[j];
        const uint64_t lim = 2 * (uint64_t)min((uint64_t)(o >> 1) / B * B + B, (uint64_t)m);
        // gallop from j (the chunk's run of x is usually short), then bisect
        const uint2 r = run[x];
        uint32_t lo = (uint32_t)j + 1, hi = r.y;
        uint64_t step = 1;
        while (true) {
            const uint64_t probe = (uint64_t)j + step;
            if (probe >= r.y || (uint64_t)sv[probe] >= lim) {
                hi = probe < r.y ? (uint32_t)probe : r.y;
                break;
            }
            lo = (uint32_t)probe + 1;
            step <<= 1;
        }
        while (lo < hi) {
            const uint32_t mid = lo + (hi - lo) / 2;
            if ((uint64_t)sv[mid] < lim) lo = mid + 1;
            else hi = mid;
        }
        cc[o] = (int32_t)(lo - r.x);
    }
}

__global__ void __launch_bounds__(kSqThreads) k_sq_init(int32_t n, int32_t rows, int32_t *__restrict__ pass_labels,
                                                        const uint2 *__restrict__ run, int32_t *__restrict__ degree) {
    SQ_LOOP(v, n) {
        degree[v] = (int32_t)(run[v].y - run[v].x);
        for (int32_t p = 0; p < rows; ++p) pass_labels[(int64_t)p * n + v] = (int32_t)v;
    }
}

// Target of an edge with endpoint counts c and degrees d in pass p (threshold D), or -1:
// both counters at most D and unequal, the endpoint with the smaller one is the target;
// equal ones with tie rule 1: e.x.
__device__ __forceinline__ int32_t sq_target(int2 e, int2 c, int2 d, int32_t p, int32_t D, int32_t tie) {
    if (e.x == e.y) return -1;
    const int32_t cu = p * d.x + c.x, cv = p * d.y + c.y;
    if (cu <= D && cv <= D && (cu != cv || tie)) return cu <= cv ? e.x : e.y;
    return -1;
}

// A wavefront takes kSqTile consecutive edges through `per` passes from per * blockIdx.y on
// (those below `first` propose nothing): all of them when there are enough edges to fill the
// chip, since the edges' counts and degrees are read once for all, otherwise at least
// kSqLeastPasses, so that many passes over a short stream are not one wavefront's chain (2,000
// edges: 1,000 passes 1.38 -> 0.15 ms, 10,000 13.1 -> 0.45; 20,000 edges, 100 passes 284 -> 160
// us).  Counting:
// its proposals per pass into tally[pass * tiles + tile].  Writing (tally now holds
// exclusive sums): proposal (p, i) at its place in (pass, stream) order: its target and
// its time p m + i.
template <bool kWrite>
__global__ void __launch_bounds__(kSqThreads) k_sq_proposals(const int2 *__restrict__ edges,
                                                             const int2 *__restrict__ cc,
                                                             const int32_t *__restrict__ degree, int64_t m, int32_t P,
                                                             int32_t D1, int32_t growth, int32_t tie, int32_t first,
                                                             int32_t per, int64_t tiles, uint32_t *__restrict__ tally,
                                                             uint32_t *__restrict__ ekey,
                                                             uint32_t *__restrict__ etime) {
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t tile = (blockIdx.x * (int64_t)kSqThreads + threadIdx.x) / kWave;
    if (tile >= tiles) return;
    const int64_t i0 = tile * kSqTile + lane;
    int2 e[kSqRounds], c[kSqRounds], d[kSqRounds];
#pragma unroll
    for (int u = 0; u < kSqRounds; ++u) {
        const int64_t i = i0 + u * kWave;
        e[u] = i < m ? edges[i] : make_int2(0, 0);
        c[u] = i < m ? cc[i] : make_int2(0, 0);  // a loop's is not set and not used
    }
#pragma unroll
    for (int u = 0; u < kSqRounds; ++u) d[u] = make_int2(degree[e[u].x], degree[e[u].y]);
    const uint64_t lt = lane ? ~0ull >> (64 - lane) : 0ull;
    const int32_t p0 = (int32_t)blockIdx.y * per, p1 = P - p0 < per ? P : p0 + per;
    for (int32_t p = p0; p < p1; ++p) {
        const int32_t D = sq_threshold(D1, growth, p);
        uint32_t at = kWrite ? tally[p * tiles + tile] : 0u;
#pragma unroll
        for (int u = 0; u < kSqRounds; ++u) {
            const int32_t v = p < first ? -1 : sq_target(e[u], c[u], d[u], p, D, tie);
            const uint64_t mask = __ballot(v >= 0);
            if (kWrite && v >= 0) {
                const uint32_t q = at + (uint32_t)__popcll(mask & lt);
                ekey[q] = (uint32_t)v;
                etime[q] = (uint32_t)(p * m + i0 + u * kWave);
            }
            at += (uint32_t)__popcll(mask);
        }
        if (!kWrite && lane == 0) tally[p * tiles + tile] = at;
    }
}

// The first time of time t's chunk (t = p m + i; chunks of B <= m edges within a pass).
__device__ __forceinline__ uint32_t sq_chunk_start(uint32_t t, uint32_t m, uint32_t B) {
    const uint32_t p = t / m, i = t - p * m;
    return p * m + i / B * B;
}

__global__ void k_sq_widen(const uint32_t *__restrict__ a, unsigned long long *b) { *b = *a; }

// A wavefront takes kSqTile consecutive sorted proposals.  A proposal wins if the one
// before it has another target or lies before its chunk.  Counting: its winners into
// tally[tile].  Writing (tally now holds exclusive sums): their targets and times, and the
// run of each node among them.
template <bool kWrite>
__global__ void __launch_bounds__(kSqThreads) k_sq_winners(const uint32_t *__restrict__ sk,
                                                           const uint32_t *__restrict__ st,
                                                           const unsigned long long *__restrict__ count, uint32_t m,
                                                           uint32_t B, int64_t tiles, uint32_t *__restrict__ tally,
                                                           uint32_t *__restrict__ wk, uint32_t *__restrict__ wt,
                                                           uint2 *__restrict__ wrun) {
    const int64_t E = (int64_t)*count;
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t tile = (blockIdx.x * (int64_t)kSqThreads + threadIdx.x) / kWave;
    if (tile >= tiles) return;
    const int64_t q0 = tile * kSqTile + lane;
    const uint64_t lt = lane ? ~0ull >> (64 - lane) : 0ull;
    uint32_t at = kWrite ? tally[tile] : 0u;
#pragma unroll
    for (int u = 0; u < kSqRounds; ++u) {
        const int64_t q = q0 + u * kWave;
        bool win = false, start = false;
        uint32_t k = 0, t = 0;
        if (q < E) {
            k = sk[q];
            t = st[q];
            start = q == 0 || sk[q - 1] != k;
            win = start || st[q - 1] < sq_chunk_start(t, m, B);
        }
        const uint64_t mask = __ballot(win);
        if (kWrite && q < E) {
            const uint32_t r = at + (uint32_t)__popcll(mask & lt);
            if (win) {
                wk[r] = k;
                wt[r] = t;
            }
            if (start) wrun[k].x = r;
            if (q + 1 == E || sk[q + 1] != k) wrun[k].y = r + (win ? 1u : 0u);
        }
        at += (uint32_t)__popcll(mask);
    }
    if (!kWrite && lane == 0) tally[tile] = at;
}

// Winner r's link: the last winner into its source with an earlier chunk, or none
// (~0); packed with the label it carries when it has no link: the source's starting
// label (its id, or lab0 of a resumed run).
__global__ void __launch_bounds__(kSqThreads) k_sq_links(const int2 *__restrict__ edges,
                                                         const uint32_t *__restrict__ wk,
                                                         const uint32_t *__restrict__ wt,
                                                         const uint32_t *__restrict__ wcount, uint32_t m, uint32_t B,
                                                         const uint2 *__restrict__ wrun,
                                                         const int32_t *__restrict__ lab0,
                                                         unsigned long long *__restrict__ jv) {
    const int64_t W = *wcount;
    SQ_LOOP(r, W) {
        const uint32_t t = wt[r];
        const int2 e = edges[t % m];
        const int32_t u = e.x == (int32_t)wk[r] ? e.y : e.x;
        const uint32_t want = sq_chunk_start(t, m, B);
        const uint2 b = wrun[u];  // u's winners (none: an empty run); the first time >= want
        uint32_t lo = b.x, hi = b.y;
        while (lo < hi) {
            const uint32_t mid = lo + (hi - lo) / 2;
            if (wt[mid] < want) lo = mid + 1;
            else hi = mid;
        }
        const uint32_t link = lo > b.x ? lo - 1 : 0xffffffffu;
        const int32_t l0 = lab0 ? lab0[u] : u;
        jv[r] = ((unsigned long long)(uint32_t)l0 << 32) | link;
    }
}

// One pointer-jumping round, in place: a winner follows up to kSqHops links; where it
// meets a resolved one it takes its label, else it keeps the last link it read.  Each
// 8-byte word is read and written by one instruction, so a concurrent reader sees a link
// and label that belong together (older or newer, both true of the chain: its label is
// that of its link's), and the final label is copied only from a resolved word; every
// word read is at least as new as the round's start, so each round shortens every
// remaining chain to at most a (kSqHops + 1)-th.  The round does nothing if the previous
// one left nothing unresolved (*go_in == 0), and sets *go_out when it did not resolve
// everything.
__global__ void __launch_bounds__(kSqThreads) k_sq_jump(unsigned long long *jv, const uint32_t *__restrict__ wcount,
                                                        const int32_t *go_in, int32_t *go_out) {
    if (*go_in == 0) return;  // the same value for every thread of the grid
    const int64_t W = *wcount;
    bool more = false;
    SQ_LOOP(r, W) {
        unsigned long long w = __hip_atomic_load(&jv[r], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        if ((uint32_t)w == 0xffffffffu) continue;
        const unsigned long long own = w & 0xffffffff00000000ull;
        for (int h = 0; h < kSqHops && (uint32_t)w != 0xffffffffu; ++h)
            w = __hip_atomic_load(&jv[(uint32_t)w], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        const bool done = (uint32_t)w == 0xffffffffu;
        more |= !done;
        __hip_atomic_store(&jv[r], done ? w : (own | (uint32_t)w), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    if (__syncthreads_or(more) && threadIdx.x == 0) *go_out = 1;
}

// A node's label after pass p: the label of its last winner in passes 0..p.
__global__ void __launch_bounds__(kSqThreads) k_sq_pass_labels(const uint32_t *__restrict__ wk,
                                                               const uint32_t *__restrict__ wt,
                                                               const uint32_t *__restrict__ wcount, uint32_t m,
                                                               int32_t P, const unsigned long long *__restrict__ jv,
                                                               int32_t n, int32_t *__restrict__ pass_labels) {
    const int64_t W = *wcount;
    SQ_LOOP(r, W) {
        const uint32_t v = wk[r];
        const int32_t lab = (int32_t)(jv[r] >> 32);
        const int32_t p0 = (int32_t)(wt[r] / m);
        const int32_t p1 = r + 1 < W && wk[r + 1] == v ? (int32_t)(wt[r + 1] / m) : P;
        for (int32_t p = p0; p < p1; ++p) pass_labels[(int64_t)p * n + v] = lab;
    }
}

// Final labels: of each node's last winner, or its starting one; and the volumes.
__global__ void __launch_bounds__(1024) k_sq_finish(const uint2 *__restrict__ wrun,
                                                    const unsigned long long *__restrict__ jv,
                                                    const int32_t *__restrict__ degree,
                                                    const int32_t *__restrict__ lab0, int32_t n,
                                                    int32_t *__restrict__ labels,
                                                    unsigned long long *__restrict__ volume) {
    __shared__ VolumeTable tab;
    if (volume) vs_clear(tab);
    __syncthreads();
    SQ_LOOP(v, n) {
        const uint2 b = wrun[v];
        const int32_t l = b.y > b.x ? (int32_t)(jv[b.y - 1] >> 32) : lab0 ? lab0[v] : (int32_t)v;
        labels[v] = l;
        const int32_t d = volume ? degree[v] : 0;
        if (d) vs_add_node(tab, volume, v, l, (unsigned long long)d);
    }
    __syncthreads();
    if (volume) vs_flush(tab, volume);
}

// ------------------------------------------------------------------- driver ----
bgv_status sq_run(int32_t n, int64_t m, const int32_t *edges, const bgv_cd_params *p, int32_t *labels,
                  int32_t *degree, int64_t *volume, int32_t *pass_labels, int32_t first, const int32_t *lab0,
                  void *ws, hipStream_t s) {
    Carver c(ws);
    SqWs w;
    sq_layout(c, n, m, p, &w);
    const int2 *e2 = reinterpret_cast<const int2 *>(edges);
    const int32_t P = p->passes;
    const int64_t no = 2 * m, pm = (int64_t)P * m, nchunk = (m + p->chunk - 1) / p->chunk;
    const uint32_t um = (uint32_t)m, B = (uint32_t)std::min<int64_t>(p->chunk, m);
    const unsigned go = grid_for(no, kSqThreads, 65536), gn = grid_for(n, kSqThreads, 65536);
    const unsigned gw = grid_for(pm, kSqThreads, 65536);
    // a chain of links visits at most one winner per chunk, and a round leaves at most a
    // (kSqHops + 1)-th of it
    int rounds = 2;
    for (uint64_t left = (uint64_t)P * (uint64_t)nchunk; left > 1; left = (left + kSqHops) / (kSqHops + 1)) ++rounds;
    BGV_LAUNCH(k_sq_occ, dim3(std::max(grid_for(m, kSqThreads, 65536), gn)), dim3(kSqThreads), 0, s, e2, m, n,
               reinterpret_cast<uint2 *>(w.okey), reinterpret_cast<uint2 *>(w.oval), w.run, w.wrun, w.go, rounds);
    const int nbits = bits_for((uint64_t)n);
    uint32_t *sk = nullptr, *sv = nullptr;
    BGV_TRY(sort_pairs<uint32_t>(w.okey, w.okey_alt, w.oval, w.oval_alt, no, nbits, &sk, &sv, w.osort, s));
    BGV_LAUNCH(k_sq_runs, dim3(go), dim3(kSqThreads), 0, s, sk, no, n, w.run);
    BGV_LAUNCH(k_sq_counts, dim3(go), dim3(kSqThreads), 0, s, sk, sv, no, n, w.run, um, B, w.cc);
    BGV_LAUNCH(k_sq_init, dim3(gn), dim3(kSqThreads), 0, s, n, pass_labels ? P : 0, pass_labels, w.run, degree);

    // proposals of every pass, in (pass, stream) order, then by target
    const int64_t ptiles = sq_tiles(m);
    // passes per wavefront: some 4,096 wavefronts, and at most 65,535 blocks in y
    const int64_t per = std::min<int64_t>(
        P, std::max<int64_t>({kSqLeastPasses, (P * ptiles + 4095) / 4096, ((int64_t)P + 65534) / 65535}));
    const dim3 gp((unsigned)((ptiles * kWave + kSqThreads - 1) / kSqThreads), (unsigned)((P + per - 1) / per));
    const int2 *cc = reinterpret_cast<const int2 *>(w.cc);
    BGV_LAUNCH(k_sq_proposals<false>, gp, dim3(kSqThreads), 0, s, e2, cc, degree, m, P, p->threshold, p->growth,
               p->tie, first, (int32_t)per, ptiles, w.tally, (uint32_t *)nullptr, (uint32_t *)nullptr);
    BGV_TRY(exclusive_scan_u32(w.tally, w.tally, P * ptiles, w.tot + 1, w.scan_scratch, s));
    BGV_LAUNCH(k_sq_widen, dim3(1), dim3(1), 0, s, w.tot + 1, w.ne);
    BGV_LAUNCH(k_sq_proposals<true>, gp, dim3(kSqThreads), 0, s, e2, cc, degree, m, P, p->threshold, p->growth,
               p->tie, first, (int32_t)per, ptiles, w.tally, w.ekey, w.etime);
    uint32_t *ek = nullptr, *et = nullptr;
    BGV_TRY(sort_pairs<uint32_t>(w.ekey, w.ekey_alt, w.etime, w.etime_alt, pm, nbits, &ek, &et, w.esort, s, w.ne));

    // winners, their links, the labels
    uint32_t *wk = ek == w.ekey ? w.ekey_alt : w.ekey, *wt = et == w.etime ? w.etime_alt : w.etime;
    const int64_t etiles = sq_tiles(pm);
    const dim3 ge((unsigned)((etiles * kWave + kSqThreads - 1) / kSqThreads));
    BGV_LAUNCH(k_sq_winners<false>, ge, dim3(kSqThreads), 0, s, ek, et, w.ne, um, B, etiles, w.tally, wk, wt, w.wrun);
    BGV_TRY(exclusive_scan_u32(w.tally, w.tally, etiles, w.tot, w.scan_scratch, s));
    BGV_LAUNCH(k_sq_winners<true>, ge, dim3(kSqThreads), 0, s, ek, et, w.ne, um, B, etiles, w.tally, wk, wt, w.wrun);
    BGV_LAUNCH(k_sq_links, dim3(gw), dim3(kSqThreads), 0, s, e2, wk, wt, w.tot, um, B, w.wrun, lab0, w.jv);
    for (int r = 0; r < rounds; ++r)
        BGV_LAUNCH(k_sq_jump, dim3(gw), dim3(kSqThreads), 0, s, w.jv, w.tot, w.go + r, w.go + r + 1);
    if (pass_labels)
        BGV_LAUNCH(k_sq_pass_labels, dim3(gw), dim3(kSqThreads), 0, s, wk, wt, w.tot, um, P, w.jv, n, pass_labels);
    BGV_LAUNCH(k_sq_finish, dim3(vs_grid(n)), dim3(1024), 0, s, w.wrun, w.jv, degree, lab0, n, labels,
               reinterpret_cast<unsigned long long *>(volume));
    return BGV_OK;
}

}  // namespace bgv
