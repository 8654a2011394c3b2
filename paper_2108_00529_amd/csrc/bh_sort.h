// Bodies in Morton order by one splitting pass and one sort per bucket, both on chip.
//
// A radix sort of 32-bit codes takes four passes, and for the 10^4 - 10^6 bodies of a
// Barnes-Hut layout each is bound by latency (its look-back chain and a launch's start), not
// by bytes.  Here the bodies are split once into up to kBhBuckets buckets between splitters
// sampled from the bodies themselves, and one workgroup per bucket sorts it in LDS.  What is
// compared is (code, body), so that equal codes are split and ordered by body, which is the
// order a stable sort of the codes gives: the result depends neither on the sample nor on the
// order within a bucket.  Both launches have one workgroup per tile or bucket and no look-back.
// 17,724 bodies: 16 us for codes, order and gathered bodies, 36 by the radix sort; 171,724:
// 38 us (beside the attraction) and 78.  What is left is chains of dependent loads: the
// frame, the samples' bodies and positions, a search; a bucket's parts, its keys, its bodies.
//
// Sample: the bodies that were at regular places of the previous iteration's order, at their
// present positions, since that order changes little from one iteration to the next; hashed
// places of the index order before there is one.
#pragma once
#include "block_scan.h"
#include "common.h"

namespace bgv {

constexpr int32_t kBhBuckets = 1024;
// From iteration kBhSettled on as many are enough up to kBhFewMax bodies, and a sample of
// that size is quicker to sort; before, the bodies move most, buckets of more than four
// times the average are common, and LDS should hold them (171,724 bodies: 200 iterations
// 33.9 ms, always 895 buckets 34.6; the first five 1.5 ms, with 512 buckets 1.7.  196,608:
// 100 iterations 17.7 ms, with 1,024 buckets 16.7).
constexpr int32_t kBhBucketsFew = 512;
constexpr int32_t kBhSettled = 16;
constexpr int32_t kBhFewMax = 184320;
constexpr int kBhBucketThreads = 512;
constexpr int32_t kBhTilesMax = 256;    // at most a thread of a bucket's workgroup per tile
constexpr int32_t kBhBucketLds = 1536;  // bodies of a bucket sorted in LDS; more: in memory
                                        // (two workgroups beside one of the attraction's)
constexpr int32_t kBhTileSmall = 256, kBhTileLarge = 1024;
constexpr int32_t kBhSplitSmall = kBhTilesMax * kBhTileSmall;
// Above this the radix sort (262,144 bodies, 100 iterations: 21.3 ms, with it 22.6).
constexpr int32_t kBhSplitMax = kBhTilesMax * kBhTileLarge;

struct BhSplit {
    int32_t tile, tiles, buckets;
};

__host__ __device__ __forceinline__ BhSplit bh_split_shape(int32_t K, int32_t it) {
    BhSplit p;
    p.tile = K <= kBhSplitSmall ? kBhTileSmall : kBhTileLarge;
    p.tiles = (K + p.tile - 1) / p.tile;
    p.buckets = (K + 191) / 192;  // most hold at most 256 bodies
    const int32_t most = it >= kBhSettled && K <= kBhFewMax ? kBhBucketsFew : kBhBuckets;
    if (p.buckets > most) p.buckets = most;
    return p;
}

// v of the lane whose number differs from this one's in the bits of kXor.
template <int kCtrl>
__device__ __forceinline__ uint32_t bh_dpp(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, kCtrl, 0xf, 0xf, true);
}
template <int kXor>
__device__ __forceinline__ uint32_t bh_partner(uint32_t v, int lane) {
    if constexpr (kXor == 1) return bh_dpp<0xB1>(v);   // within four lanes: 1 0 3 2
    if constexpr (kXor == 2) return bh_dpp<0x4E>(v);   // 2 3 0 1
    if constexpr (kXor == 3) return bh_dpp<0x1B>(v);   // 3 2 1 0
    if constexpr (kXor == 7) return bh_dpp<0x141>(v);  // half rows mirrored
    if constexpr (kXor == 4) return bh_dpp<0x141>(bh_dpp<0x1B>(v));
    if constexpr (kXor == 8) return bh_dpp<0x128>(v);  // rows of 16 rotated by 8
    if constexpr (kXor == 15) return bh_dpp<0x140>(v);  // rows mirrored
    if constexpr (kXor == 16) {
        const auto q = __builtin_amdgcn_permlane16_swap(v, v, false, false);
        return lane & 16 ? q[0] : q[1];
    }
    if constexpr (kXor == 32) {
        const auto q = __builtin_amdgcn_permlane32_swap(v, v, false, false);
        return lane & 32 ? q[0] : q[1];
    }
    if constexpr (kXor == 31) return bh_partner<16>(bh_dpp<0x140>(v), lane);
    if constexpr (kXor == 63) return bh_partner<32>(bh_partner<31>(v, lane), lane);
    return v;
}
template <int kXor, int kUpper>
__device__ __forceinline__ void bh_exchange(uint64_t &v, int lane) {
    const uint64_t o = (uint64_t)bh_partner<kXor>((uint32_t)(v >> 32), lane) << 32 | bh_partner<kXor>((uint32_t)v, lane);
    if ((v < o) == ((lane & kUpper) != 0)) v = o;
}

// One value per lane sorted over the wavefront, ascending: a bitonic network of ascending
// comparators in registers.  About 40 cycles a step; through LDS a step took 250 and more.
__device__ __forceinline__ uint64_t bh_sort_wave(uint64_t v, int lane) {
    bh_exchange<1, 1>(v, lane);
    bh_exchange<3, 2>(v, lane);
    bh_exchange<1, 1>(v, lane);
    bh_exchange<7, 4>(v, lane);
    bh_exchange<2, 2>(v, lane);
    bh_exchange<1, 1>(v, lane);
    bh_exchange<15, 8>(v, lane);
    bh_exchange<4, 4>(v, lane);
    bh_exchange<2, 2>(v, lane);
    bh_exchange<1, 1>(v, lane);
    bh_exchange<31, 16>(v, lane);
    bh_exchange<8, 8>(v, lane);
    bh_exchange<4, 4>(v, lane);
    bh_exchange<2, 2>(v, lane);
    bh_exchange<1, 1>(v, lane);
    bh_exchange<63, 32>(v, lane);
    bh_exchange<16, 16>(v, lane);
    bh_exchange<8, 8>(v, lane);
    bh_exchange<4, 4>(v, lane);
    bh_exchange<2, 2>(v, lane);
    bh_exchange<1, 1>(v, lane);
    return v;
}

// How many of a[0, n), ascending within runs of 64, are below key: a binary search in each
// run, four runs at a time.
__device__ __forceinline__ uint32_t bh_rank(const uint64_t *a, uint32_t n, uint64_t key) {
    uint32_t rank = 0;
    for (uint32_t r = 0; r < n; r += 4 * kWave) {
        uint32_t lo[4] = {0u, 0u, 0u, 0u};
#pragma unroll
        for (int b = 5; b >= -1; --b) {
            const uint32_t step = b >= 0 ? 1u << b : 1u;
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const uint32_t x = r + u * kWave + lo[u] + step - 1u;
                const uint64_t v = a[min(x, n - 1u)];
                if (x < n && v < key) lo[u] += step;
            }
        }
        rank += lo[0] + lo[1] + lo[2] + lo[3];
    }
    return rank;
}

// The bodies of one tile (NT ITEMS consecutive ones; code(position) encodes) grouped by
// bucket into keys[tile ..] as (code, body), and the buckets' starts there into
// off[tile (NB + 1) ..].
template <int NT, int ITEMS, typename Code>
__device__ __forceinline__ void bh_split_tile(int32_t K, const BhSplit sp, const float2 *__restrict__ pos, Code code,
                                              const float4 *__restrict__ before, uint64_t *__restrict__ keys,
                                              uint16_t *__restrict__ off) {
    __shared__ uint64_t runs[kBhBuckets], split[kBhBuckets];
    __shared__ uint32_t cnt[kBhBuckets];
    const int t = threadIdx.x, lane = t & (kWave - 1);
    const int32_t NB = sp.buckets, ns = NB - 1;
    const int32_t base = (int32_t)blockIdx.x * (NT * ITEMS);
    for (int32_t q = t; q < NB; q += NT) cnt[q] = 0u;
    for (int32_t q = t; q - lane < ns; q += NT) {  // whole wavefronts
        uint64_t v = ~0ull;
        if (q < ns) {
            uint32_t b;
            if (before)
                b = (uint32_t)__float_as_int(before[(int64_t)(q + 1) * K / NB].w);
            else
                b = (uint32_t)(((uint64_t)((uint32_t)(q + 1) * 2654435761u) * (uint32_t)K) >> 32);
            v = (uint64_t)code(pos[b]) << 32 | b;
        }
        runs[q] = bh_sort_wave(v, lane);
    }
    __syncthreads();
    // the samples are different bodies (hashed places lie at least 0.38 K / NB apart), so
    // every place of split is written
    for (int32_t q = t; q < ns; q += NT) {
        const uint64_t v = runs[q];
        split[bh_rank(runs, (uint32_t)ns, v)] = v;
    }
    __syncthreads();
    uint64_t key[ITEMS];
    int32_t lo[ITEMS];  // splitters not above the key
    uint32_t place[ITEMS];  // bucket << 16 | rank in the tile's part of it
#pragma unroll
    for (int u = 0; u < ITEMS; ++u) {
        const int32_t i = base + u * NT + t;
        key[u] = i < K ? (uint64_t)code(pos[i]) << 32 | (uint32_t)i : 0ull;
        lo[u] = 0;
    }
    for (int32_t step = kBhBuckets / 2; step > 0; step /= 2) {
        if (step > ns) continue;
#pragma unroll
        for (int u = 0; u < ITEMS; ++u) {
            const int32_t x = lo[u] + step;
            if (x <= ns && split[x - 1] <= key[u]) lo[u] = x;
        }
    }
#pragma unroll
    for (int u = 0; u < ITEMS; ++u)
        if (base + u * NT + t < K) place[u] = (uint32_t)lo[u] << 16 | atomicAdd(&cnt[lo[u]], 1u);
    __syncthreads();
    constexpr int BT = (kBhBuckets + NT - 1) / NT;  // buckets per thread
    uint32_t c[BT], sum = 0;
#pragma unroll
    for (int u = 0; u < BT; ++u) sum += c[u] = BT * t + u < NB ? cnt[BT * t + u] : 0u;
    uint32_t total;
    uint32_t e = block_excl_scan<uint32_t>(sum, &total);
    uint16_t *o = off + (int64_t)blockIdx.x * (NB + 1);
#pragma unroll
    for (int u = 0; u < BT; ++u) {
        if (BT * t + u < NB) {
            cnt[BT * t + u] = e;
            o[BT * t + u] = (uint16_t)e;
        }
        e += c[u];
    }
    if (t == 0) o[NB] = (uint16_t)total;
    __syncthreads();
#pragma unroll
    for (int u = 0; u < ITEMS; ++u)
        if (base + u * NT + t < K) keys[base + cnt[place[u] >> 16] + (place[u] & 0xffffu)] = key[u];
}

// One bucket: its parts of every tile collected, sorted, and the bodies written in order.
// spare and spare2: K words of memory each for buckets that LDS does not hold.
__global__ void __launch_bounds__(kBhBucketThreads) k_bh_bucket(int32_t K, int32_t it, const float2 *__restrict__ pos,
                                                               const float *__restrict__ mass,
                                                               const uint64_t *__restrict__ keys,
                                                               const uint16_t *__restrict__ off,
                                                               uint64_t *__restrict__ spare, uint64_t *__restrict__ spare2,
                                                               float4 *__restrict__ body,
                                                               uint32_t *__restrict__ code) {
    __shared__ uint64_t sh[kBhBucketLds];
    __shared__ uint32_t start[kBhTilesMax];  // of each tile's part in the bucket ...
    __shared__ uint32_t from[kBhTilesMax];   // ... and in keys, less that
    const BhSplit sp = bh_split_shape(K, it);
    const int t = threadIdx.x;
    uint32_t o0 = 0u, o1 = 0u;
    if (t < sp.tiles) {
        const uint16_t *o = off + (int64_t)t * (sp.buckets + 1) + blockIdx.x;
        o0 = o[0];
        o1 = o[1];
    }
    uint32_t first, n;
    block_excl_scan<uint32_t>(o0, &first);
    const uint32_t e = block_excl_scan<uint32_t>(o1 - o0, &n);
    if (t < kBhTilesMax) {
        start[t] = e;  // a thread without a tile: n
        from[t] = (uint32_t)t * (uint32_t)sp.tile + o0 - e;
    }
    static_assert(kBhBucketThreads >= kBhTilesMax, "a thread per tile");
    __syncthreads();
    const int lane = t & (kWave - 1);
    const auto sort_runs = [&](uint64_t *a) {  // the bucket into a[0, n), sorted in runs of 64
        for (uint32_t x = t; x - lane < n; x += kBhBucketThreads) {  // whole wavefronts
            uint64_t key = ~0ull;
            if (x < n) {
                int32_t lo = 0;  // parts that start at or before x: the last of them has it
#pragma unroll
                for (int32_t step = kBhTilesMax / 2; step > 0; step /= 2)
                    if (start[lo + step] <= x) lo += step;
                key = keys[from[lo] + x];
            }
            key = bh_sort_wave(key, lane);
            if (x < n) a[x] = key;
        }
        __syncthreads();
    };
    const auto write_body = [&](uint32_t place, uint64_t key) {
        const uint32_t b = (uint32_t)key, k = first + place;
        const float2 p = pos[b];
        body[k] = make_float4(p.x, p.y, mass[b], __int_as_float((int)b));
        code[k] = (uint32_t)(key >> 32);
    };
    if (n <= (uint32_t)kBhBucketLds) {
        sort_runs(sh);
        for (uint32_t x = t; x < n; x += kBhBucketThreads) {
            const uint64_t key = sh[x];
            write_body(bh_rank(sh, n, key), key);
        }
    } else {
        // runs merged in pairs, each body by a search in the other run of its pair, so that
        // a bucket of any size costs n log^2 n
        uint64_t *a = spare + first, *b = spare2 + first;
        sort_runs(a);
        for (uint32_t len = kWave; len < n; len *= 2) {
            for (uint32_t x = t; x < n; x += kBhBucketThreads) {
                const uint64_t key = a[x];
                const uint32_t run = x / len * len, pair = run / (2 * len) * (2 * len);
                const uint32_t o0 = run == pair ? min(run + len, n) : pair, o1 = run == pair ? min(run + 2 * len, n) : run;
                uint32_t lo = o0, hi = o1;
                while (lo < hi) {
                    const uint32_t mid = lo + (hi - lo) / 2;
                    if (a[mid] < key) lo = mid + 1;
                    else hi = mid;
                }
                b[pair + (x - run) + (lo - o0)] = key;
            }
            __syncthreads();
            uint64_t *const c = a;
            a = b;
            b = c;
        }
        for (uint32_t x = t; x < n; x += kBhBucketThreads) write_body(x, a[x]);
    }
}

}  // namespace bgv
