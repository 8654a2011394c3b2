// ForceAtlas2 per-pair and per-node arithmetic shared by the plain and batched layout
// kernels, so that both evaluate every force and speed with the same operation
// sequence (Section 3.1 / Algorithm 1, in the force and speed laws of the cited
// ForceAtlas2 publication).
#pragma once
#include "common.h"

namespace bgv {

// x^2 + y^2 with y^2 the product that is rounded on its own: written out, so that every
// kernel that inlines it gives the same bits.
__device__ __forceinline__ float fa2_norm2(float x, float y) { return __builtin_fmaf(x, x, y * y); }

// Repulsion from one body p = (x, y, mass): (x_i - x_j) * m_j / |x_i - x_j|^2, none if
// coincident.  The caller scales the sum by kr * m_i.  1/d^2 is the hardware reciprocal
// (within one ulp), the quotient's rounding being far below the layout's tolerance.
__device__ __forceinline__ void fa2_rep_term(float2 xi, float4 p, float &fx, float &fy) {
    const float dx = xi.x - p.x, dy = xi.y - p.y;
    const float d2 = fa2_norm2(dx, dy);
    const float f = d2 > 0.f ? p.z * __builtin_amdgcn_rcpf(d2) : 0.f;
    fx = __builtin_fmaf(f, dx, fx);
    fy = __builtin_fmaf(f, dy, fy);
}

// A body as the loops over all pairs stage it in LDS, and one that adds nothing to any force:
// without mass, and so far away that |x_i - x_j|^2 is large or zero for every x_i, since
// near a body the reciprocal is infinite and 0 times it NaN (a pad at the origin was near a
// body at (1e-20, 0)).  Its logarithm may be infinite: energies leave it out by its index.
__device__ __forceinline__ float4 fa2_body(float2 x, float m) { return make_float4(x.x, x.y, m, 0.f); }
__device__ __forceinline__ float4 fa2_no_body() { return make_float4(1e18f, 1e18f, 0.f, 0.f); }

// fa2_rep_term over n consecutive LDS bodies in ascending order, n a multiple of 8: each
// group of eight is read before any of it is used, so the reads overlap.
__device__ __forceinline__ void fa2_rep_run(float2 xi, const float4 *tile, int n, float &fx, float &fy) {
    for (int q = 0; q < n; q += 8) {
        float4 b[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) b[u] = tile[q + u];
#pragma unroll
        for (int u = 0; u < 8; ++u) fa2_rep_term(xi, b[u], fx, fy);
    }
}

// Whether a sum is not a number.  The loops below test groups of bodies for coincident ones,
// not each pair, so a pair whose |x_i - x_j|^2 is NaN (a body with one coordinate NaN or
// infinite), which the test of each pair drops along the other axis, reaches the sums there;
// such sums are made once more, pair by pair: at once by fa2_rep_ahead, by fa2_rep_again
// where the sums of the segments are added otherwise.
__device__ __forceinline__ bool fa2_nan(float fx, float fy) { return !(fx == fx && fy == fy); }

// The repulsion on a body at xi from all K, in segments of len: each summed from zero, then
// the segments in order.
__device__ __forceinline__ float2 fa2_rep_again(float2 xi, int32_t K, const float2 *__restrict__ pos,
                                                const float *__restrict__ mass, int32_t len) {
    float2 r = make_float2(0.f, 0.f);
    for (int32_t b = 0; b < K; b += len) {
        float sx = 0.f, sy = 0.f;
        const int32_t e = K - b < len ? K : b + len;
        for (int32_t j = b; j < e; ++j) fa2_rep_term(xi, fa2_body(pos[j], mass[j]), sx, sy);
        r.x = b ? r.x + sx : sx;
        r.y = b ? r.y + sy : sy;
        if (e == K) break;
    }
    return r;
}

// The same as fa2_rep_run for a wavefront that is alone on its SIMD, which waits for every result it uses
// at once: each group of eight is read while the one before it is used, and a group's
// steps are kept apart (eight differences, eight reciprocals, ..., eight additions), which
// the scheduler would interleave to save registers.
__device__ __forceinline__ void fa2_rep_steps(float2 xi, const float4 (&b)[8], float &fx, float &fy) {
    float dx[8], dy[8], d2[8], f[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
        dx[u] = xi.x - b[u].x;
        dy[u] = xi.y - b[u].y;
    }
    __builtin_amdgcn_sched_barrier(0);
    uint32_t least = ~0u;
#pragma unroll
    for (int u = 0; u < 8; ++u) d2[u] = fa2_norm2(dx[u], dy[u]);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < 8; ++u) f[u] = __builtin_amdgcn_rcpf(d2[u]);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < 8; ++u) least = min(least, __float_as_uint(d2[u]));
#pragma unroll
    for (int u = 0; u < 8; ++u) f[u] *= b[u].z;
    if (__any(least == 0u)) {
#pragma unroll
        for (int u = 0; u < 8; ++u) f[u] = d2[u] > 0.f ? f[u] : 0.f;
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < 8; ++u) {
        fx = __builtin_fmaf(f[u], dx[u], fx);
        fy = __builtin_fmaf(f[u], dy[u], fy);
    }
    __builtin_amdgcn_sched_barrier(0);
}
__device__ __forceinline__ void fa2_rep_load(const float4 *tile, float4 (&b)[8]) {
#pragma unroll
    for (int u = 0; u < 8; ++u) b[u] = tile[u];
    __builtin_amdgcn_sched_barrier(0);
}
__device__ __forceinline__ void fa2_rep_ahead(float2 xi, const float4 *tile, int n, float &fx, float &fy) {
    if (n <= 0) return;
    const float fx0 = fx, fy0 = fy;
    float4 b[8], c[8];
    fa2_rep_load(tile, b);
    int q = 8;
    for (; q + 8 < n; q += 16) {  // two groups a round, so that no group is moved
        fa2_rep_load(tile + q, c);
        fa2_rep_steps(xi, b, fx, fy);
        fa2_rep_load(tile + q + 8, b);
        fa2_rep_steps(xi, c, fx, fy);
    }
    if (q < n) {
        fa2_rep_load(tile + q, c);
        fa2_rep_steps(xi, b, fx, fy);
        fa2_rep_steps(xi, c, fx, fy);
    } else {
        fa2_rep_steps(xi, b, fx, fy);
    }
    if (__any(fa2_nan(fx, fy))) {
        fx = fx0;
        fy = fy0;
        fa2_rep_run(xi, tile, n, fx, fy);
    }
}

// The same sums on R bodies per lane, so that each LDS read serves R pairs.  With enough
// bodies the loop is bound by vector issue, so the test for coincident bodies is taken
// once per group: the smallest of its d^2 (as bit patterns: they are not negative) by
// three-operand minima, and the per-pair test and select only where some lane's is zero.
// That is 7.6 vector instructions per pair beside the reciprocal instead of 9 (50,000
// bodies, whole iteration: 613 -> 555 us).
template <int R>
__device__ __forceinline__ void fa2_rep_run(const float2 (&xi)[R], const float4 *tile, int n, float (&fx)[R],
                                            float (&fy)[R]) {
    for (int q = 0; q < n; q += 8) {
        float4 b[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) b[u] = tile[q + u];
        float dx[R][8], dy[R][8], d2[R][8];
        uint32_t least = ~0u;
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                dx[r][u] = xi[r].x - b[u].x;
                dy[r][u] = xi[r].y - b[u].y;
                d2[r][u] = fa2_norm2(dx[r][u], dy[r][u]);
                least = min(least, __float_as_uint(d2[r][u]));
            }
        if (__any(least == 0u)) {
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const float f = d2[r][u] > 0.f ? b[u].z * __builtin_amdgcn_rcpf(d2[r][u]) : 0.f;
                    fx[r] = __builtin_fmaf(f, dx[r][u], fx[r]);
                    fy[r] = __builtin_fmaf(f, dy[r][u], fy[r]);
                }
        } else {
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const float f = b[u].z * __builtin_amdgcn_rcpf(d2[r][u]);
                    fx[r] = __builtin_fmaf(f, dx[r][u], fx[r]);
                    fy[r] = __builtin_fmaf(f, dy[r][u], fy[r]);
                }
        }
    }
}
__device__ __forceinline__ void fa2_rep_run(const float2 (&xi)[1], const float4 *tile, int n, float (&fx)[1],
                                            float (&fy)[1]) {
    fa2_rep_run(xi[0], tile, n, fx[0], fy[0]);
}

// Exact repulsion on body i is summed over j in consecutive segments of kRepSegment
// bodies: each segment in ascending j starting from zero, then the segment sums in
// ascending order (the first one taken as is).  Segments let one body's sum be split
// over several workgroups while fixing the order of every addition, so any launch shape
// gives the same bits.  A multiple of the 256-body LDS tiles; short enough that a
// supergraph of a few thousand nodes spreads over many workgroups.
constexpr int32_t kRepSegment = 512;

// Bodies from which the gradient's repulsion gives each thread two bodies; with fewer, halving
// the wavefronts costs what the shared reads give.
constexpr int32_t kRepTwoMin = 16384;
// The same for the layout's exact forces, whose one body per thread reads ahead (us per
// iteration with one / two: 16,384 bodies 77 / 86, 30,000 218 / 224, 40,000 374 / 383, 50,000
// 570 / 563, 100,000 2,160 / 2,124).
constexpr int32_t kForceTwoMin = 45056;

__host__ __device__ __forceinline__ int32_t fa2_rep_segments(int32_t K) {
    return (K + kRepSegment - 1) / kRepSegment;
}

// CSR entries: (neighbour, weight bits) when edges are weighted, the bare neighbour id
// (32 or 16 bits) when every weight is 1.  Adding w * d with w = 1 rounds exactly like
// adding d (fused or not), so all three give the same bits for unit weights.
__device__ __forceinline__ int32_t fa2_entry_id(int2 e) { return e.x; }
__device__ __forceinline__ int32_t fa2_entry_id(uint32_t e) { return (int32_t)e; }
__device__ __forceinline__ int32_t fa2_entry_id(uint16_t e) { return (int32_t)e; }

__device__ __forceinline__ void fa2_entry_add(int2 e, float2 xj, float2 xi, float &ax, float &ay) {
    const float w = __int_as_float(e.y);
    ax += w * (xj.x - xi.x);
    ay += w * (xj.y - xi.y);
}
template <typename E>
__device__ __forceinline__ void fa2_entry_add(E, float2 xj, float2 xi, float &ax, float &ay) {
    ax += xj.x - xi.x;
    ay += xj.y - xi.y;
}

// Sum over a wavefront by the tree that adds lanes 32 apart, then 16, 8, 4, 2 and 1 (what
// a butterfly of __shfl_xor gives in every lane and one of __shfl_down in lane 0, bit for
// bit: an addition's operands may change places), without the LDS crossbar: the first two
// steps by lane swaps, the others by rotations within rows of 16, where the values
// already repeat every 16, 8, 4 or 2 lanes.
template <int kRor>
__device__ __forceinline__ uint32_t fa2_row_rotate(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x120 + kRor, 0xf, 0xf, true);
}
__device__ __forceinline__ float fa2_wave_sum(float v) {
    const uint32_t b = __float_as_uint(v);
    const auto h = __builtin_amdgcn_permlane32_swap(b, b, false, false);
    v = __uint_as_float(h[0]) + __uint_as_float(h[1]);
    const uint32_t c = __float_as_uint(v);
    const auto q = __builtin_amdgcn_permlane16_swap(c, c, false, false);
    v = __uint_as_float(q[0]) + __uint_as_float(q[1]);
    v += __uint_as_float(fa2_row_rotate<8>(__float_as_uint(v)));
    v += __uint_as_float(fa2_row_rotate<4>(__float_as_uint(v)));
    v += __uint_as_float(fa2_row_rotate<2>(__float_as_uint(v)));
    v += __uint_as_float(fa2_row_rotate<1>(__float_as_uint(v)));
    return v;
}
// Four such sums at once: lanes 16 q .. 16 q + 15 get the sum of v[q].  A swap exchanges
// the halves of two registers, so that one addition folds both: ten instructions for four
// sums instead of 64.
__device__ __forceinline__ float fa2_wave_sum4(const float (&v)[4]) {
    const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(v[0]), __float_as_uint(v[2]), false, false);
    const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v[1]), __float_as_uint(v[3]), false, false);
    const float s = __uint_as_float(a[0]) + __uint_as_float(a[1]);  // halves: v[0], v[2]
    const float t = __uint_as_float(b[0]) + __uint_as_float(b[1]);  // v[1], v[3]
    const auto c = __builtin_amdgcn_permlane16_swap(__float_as_uint(s), __float_as_uint(t), false, false);
    float r = __uint_as_float(c[0]) + __uint_as_float(c[1]);  // rows of 16: v[0], v[1], v[2], v[3]
    r += __uint_as_float(fa2_row_rotate<8>(__float_as_uint(r)));
    r += __uint_as_float(fa2_row_rotate<4>(__float_as_uint(r)));
    r += __uint_as_float(fa2_row_rotate<2>(__float_as_uint(r)));
    r += __uint_as_float(fa2_row_rotate<1>(__float_as_uint(r)));
    return r;
}
template <int kRor>
__device__ __forceinline__ double fa2_row_rotate(double v) {
    return __hiloint2double((int)fa2_row_rotate<kRor>((uint32_t)__double2hiint(v)),
                            (int)fa2_row_rotate<kRor>((uint32_t)__double2loint(v)));
}
__device__ __forceinline__ double fa2_wave_sum(double v) {
    uint32_t lo = (uint32_t)__double2loint(v), hi = (uint32_t)__double2hiint(v);
    const auto hl = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
    const auto hh = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
    v = __hiloint2double((int)hh[0], (int)hl[0]) + __hiloint2double((int)hh[1], (int)hl[1]);
    lo = (uint32_t)__double2loint(v);
    hi = (uint32_t)__double2hiint(v);
    const auto ql = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
    const auto qh = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
    v = __hiloint2double((int)qh[0], (int)ql[0]) + __hiloint2double((int)qh[1], (int)ql[1]);
    v += fa2_row_rotate<8>(v);
    v += fa2_row_rotate<4>(v);
    v += fa2_row_rotate<2>(v);
    v += fa2_row_rotate<1>(v);
    return v;
}

// Attraction over the CSR entries [b0, b1) of one block (at most kAttBlock entries), by
// one wavefront: lane l takes entries b0 + l, b0 + l + 64, ... in order (four loads in
// flight), then a fixed butterfly combines the lanes; every lane returns the total.
constexpr uint32_t kAttBlock = 16 * kWave;

template <typename P, typename E>  // P: positions by index (a pointer, or an accessor)
__device__ __forceinline__ void fa2_block_lane(P pos, const E *__restrict__ cw, uint32_t b0, uint32_t b1, float2 xi,
                                               int lane, float &ax, float &ay) {
    ax = ay = 0.f;
    uint32_t k = b0 + lane;
    // every lane adds its entries in ascending k; the unrolled loads only overlap
    for (; k + 7 * kWave < b1; k += 8 * kWave) {
        E e[8];
        float2 x[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) e[u] = cw[k + u * kWave];
#pragma unroll
        for (int u = 0; u < 8; ++u) x[u] = pos[fa2_entry_id(e[u])];
#pragma unroll
        for (int u = 0; u < 8; ++u) fa2_entry_add(e[u], x[u], xi, ax, ay);
    }
    for (; k + 3 * kWave < b1; k += 4 * kWave) {
        const E e0 = cw[k], e1 = cw[k + kWave], e2 = cw[k + 2 * kWave], e3 = cw[k + 3 * kWave];
        const float2 x0 = pos[fa2_entry_id(e0)], x1 = pos[fa2_entry_id(e1)], x2 = pos[fa2_entry_id(e2)],
                     x3 = pos[fa2_entry_id(e3)];
        fa2_entry_add(e0, x0, xi, ax, ay);
        fa2_entry_add(e1, x1, xi, ax, ay);
        fa2_entry_add(e2, x2, xi, ax, ay);
        fa2_entry_add(e3, x3, xi, ax, ay);
    }
    for (; k < b1; k += kWave) {
        const E e = cw[k];
        fa2_entry_add(e, pos[fa2_entry_id(e)], xi, ax, ay);
    }
}

template <typename P, typename E>
__device__ __forceinline__ float2 fa2_block_attraction(P pos, const E *__restrict__ cw,
                                                       uint32_t b0, uint32_t b1, float2 xi, int lane) {
    float ax, ay;
    fa2_block_lane(pos, cw, b0, b1, xi, lane, ax, ay);
    return make_float2(fa2_wave_sum(ax), fa2_wave_sum(ay));
}

// Attraction on node i = sum over its CSR entries [r0, r1) of w * (x_j - x_i): the row
// is cut into blocks of kAttBlock entries, each summed as above, and the block sums are
// added in order (the first taken as is).  A row of up to kAttBlock entries is a single
// block.  The blocks of a long (hub) row can then be summed by different wavefronts and
// combined afterwards with the same additions (fa2_att_combine).
template <typename P, typename E>
__device__ __forceinline__ float2 fa2_row_attraction(P pos, const E *__restrict__ cw,
                                                     uint32_t r0, uint32_t r1, float2 xi, int lane) {
    float2 t = fa2_block_attraction(pos, cw, r0, r1 - r0 > kAttBlock ? r0 + kAttBlock : r1, xi, lane);
    for (uint32_t b = r0 + kAttBlock; b < r1; b += kAttBlock) {
        const float2 v = fa2_block_attraction(pos, cw, b, r1 - b > kAttBlock ? b + kAttBlock : r1, xi, lane);
        t.x += v.x;
        t.y += v.y;
    }
    return t;
}

// The attractions of nodes base + first, base + first + step, ... below base + n by one
// wavefront into att[first], ...; row[0] is node base's row start.  Four rows at a time, so
// that their loads overlap and one packed reduction sums all four; rows cut into blocks
// (more than kAttBlock entries) go one by one.
template <typename P, typename E>
__device__ __forceinline__ void fa2_rows_attraction(P pos, const E *cw, const uint32_t *row, int32_t base, int32_t n,
                                                    float2 *att, int32_t first, int32_t step, int lane) {
    for (int32_t r0 = first; r0 < n; r0 += 4 * step) {
        uint32_t b[4], len[4], longest = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int32_t r = min(r0 + q * step, n - 1);
            b[q] = row[r];
            len[q] = r0 + q * step < n ? row[r + 1] - b[q] : 0u;
            longest = max(longest, len[q]);
        }
        float ax[4], ay[4];
        if (longest <= (uint32_t)kWave) {  // uniform over the wavefront
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                ax[q] = ay[q] = 0.f;
                if ((uint32_t)lane < len[q]) {
                    const E e = cw[b[q] + lane];
                    fa2_entry_add(e, pos[fa2_entry_id(e)], pos[base + min(r0 + q * step, n - 1)], ax[q], ay[q]);
                }
            }
        } else if (longest <= kAttBlock) {
#pragma unroll
            for (int q = 0; q < 4; ++q)
                fa2_block_lane(pos, cw, b[q], b[q] + len[q], pos[base + min(r0 + q * step, n - 1)], lane, ax[q], ay[q]);
        } else {
            for (int q = 0; q < 4 && r0 + q * step < n; ++q) {
                const int32_t r = r0 + q * step;
                const float2 a = fa2_row_attraction(pos, cw, b[q], b[q] + len[q], pos[base + r], lane);
                if (lane == 0) att[r] = a;
            }
            continue;
        }
        const float sx = fa2_wave_sum4(ax), sy = fa2_wave_sum4(ay);
        const int32_t r = r0 + lane / 16 * step;
        if (lane % 16 == 0 && r < n) att[r] = make_float2(sx, sy);
    }
}

// Node i's attraction from its block sums attb[item_of[i] .. item_of[i + 1]), added in
// block order exactly as fa2_row_attraction adds them.
__device__ __forceinline__ float2 fa2_att_combine(const float2 *__restrict__ attb, const uint32_t *__restrict__ item_of,
                                                  int32_t i) {
    const uint32_t a = item_of[i], b = item_of[i + 1];
    float2 t = attb[a];
    for (uint32_t q = a + 1; q < b; ++q) {
        const float2 v = attb[q];
        t.x += v.x;
        t.y += v.y;
    }
    return t;
}

// Fixed-pattern sum of one double2 per thread over a group of 256 threads (4
// wavefronts): the wavefront tree, then the 4 wavefront sums in order.
// ws must hold blockDim/64 entries; the result is valid in the group's first thread.
// Contains a barrier: every thread of the workgroup must call it.
__device__ __forceinline__ double2 fa2_sum256(double2 v, double2 *ws) {
    v.x = fa2_wave_sum(v.x);
    v.y = fa2_wave_sum(v.y);
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    if (lane == 0) ws[w] = v;
    __syncthreads();
    double2 r = make_double2(0.0, 0.0);
    if ((threadIdx.x & 255) == 0)
        for (int q = 0; q < 4; ++q) {
            r.x += ws[w + q].x;
            r.y += ws[w + q].y;
        }
    __syncthreads();
    return r;
}

// Net force: repulsion kr*m_i*sum + attraction + gravity (-kg m_i x / |x|, none at 0).
__device__ __forceinline__ float2 fa2_net_force(float2 xi, float mi, float kr, float rx, float ry, float2 att,
                                                float kg) {
    const float c = kr * mi;
    float fx = c * rx + att.x, fy = c * ry + att.y;
    const float r = sqrtf(fa2_norm2(xi.x, xi.y));
    if (r > 0.f) {
        const float g = kg * mi / r;
        fx -= g * xi.x;
        fy -= g * xi.y;
    }
    return make_float2(fx, fy);
}

// (m_i * swing_i, m_i * traction_i) with swing = |F - F'|, traction = |F + F'| / 2.
__device__ __forceinline__ double2 fa2_swing_traction(float2 F, float2 Fp, float mi) {
    const float sx = F.x - Fp.x, sy = F.y - Fp.y;
    const float tx = F.x + Fp.x, ty = F.y + Fp.y;
    const float sw = sqrtf(fa2_norm2(sx, sy));
    const float tr = 0.5f * sqrtf(fa2_norm2(tx, ty));
    return make_double2((double)mi * (double)sw, (double)mi * (double)tr);
}

// Global speed from the swing and traction sums: min(tau T / S, 1.5 s), kept if S = 0.
__device__ __forceinline__ float fa2_global_speed(double S, double T, float sp, float tau) {
    float s = sp;
    if (S > 0.0) s = (float)fmin((double)tau * T / S, 1.5 * (double)sp);
    return s;
}

// Local speed ks s / (1 + s sqrt(swing)), capped so the step is at most ksmax; moves p.
__device__ __forceinline__ float2 fa2_move(float2 p, float2 f, float2 fp, float s, float ks, float ksmax) {
    const float sx = f.x - fp.x, sy = f.y - fp.y;
    const float sw = sqrtf(fa2_norm2(sx, sy));
    float si = ks * s / (1.0f + s * sqrtf(sw));
    const float fn = sqrtf(fa2_norm2(f.x, f.y));
    if (fn > 0.f && si > ksmax / fn) si = ksmax / fn;
    p.x += si * f.x;
    p.y += si * f.y;
    return p;
}

// ---- whole-tile bodies of the plain kernels --------------------------------------------
// A tile is 256 consecutive nodes handled by one 256-thread workgroup.
constexpr int kFa2Tile = 256;

// Node i's attraction: its CSR block sums combined (item_of != null) or a final value.
__device__ __forceinline__ float2 fa2_att_value(const float2 *__restrict__ att, const uint32_t *__restrict__ item_of,
                                                int32_t i) {
    return item_of ? fa2_att_combine(att, item_of, i) : att[i];
}

// Exact repulsion of the nodes of tile bx (256 R nodes, R per thread) over the bodies of
// j segment by (all of [0, K) when kSegmented is false), bodies staged through LDS 256 at
// a time or, with one node per thread, the whole segment at once and each group read ahead
// (few wavefronts share a SIMD then: 27.2 -> 25.0 us an iteration at 4,001 bodies, 60.9 ->
// 57.6 at 12,000, 86.2 -> 82.1 at 16,000).  With one segment the tile's forces are finished (attraction, gravity, swing,
// traction and the tile's FP64 partial sums into part[bx]); with several, the segment
// sums go to seg.
template <bool kSegmented, int R = 1>
__device__ __forceinline__ void fa2_exact_force_tile(int32_t bx, int32_t by, int32_t K, const float2 *__restrict__ pos,
                                                     const float *__restrict__ mass, const float2 *__restrict__ att,
                                                     const uint32_t *__restrict__ item_of, float kr, float kg,
                                                     const float2 *__restrict__ fprev, float2 *__restrict__ F,
                                                     double2 *__restrict__ part, float2 *__restrict__ seg) {
    static_assert(kSegmented || R == 1, "finished tiles hold one node per thread");
    constexpr int kStage = R == 1 ? kRepSegment : kFa2Tile;
    __shared__ float4 tile[kStage];
    __shared__ double2 ws[kFa2Tile / kWave];
    const int32_t i = bx * (kFa2Tile * R) + threadIdx.x;
    float2 xi[R];
    float fx[R], fy[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        xi[r] = i + r * kFa2Tile < K ? pos[i + r * kFa2Tile] : make_float2(0.f, 0.f);
        fx[r] = fy[r] = 0.f;
    }
    const int32_t jb = kSegmented ? by * kRepSegment : 0;
    const int32_t je = kSegmented ? min(K, jb + kRepSegment) : K;
    for (int32_t t0 = jb; t0 < je; t0 += kStage) {
#pragma unroll
        for (int q = 0; q < kStage / kFa2Tile; ++q) {
            const int32_t j = t0 + q * kFa2Tile + threadIdx.x;
            tile[q * kFa2Tile + threadIdx.x] = j < je ? fa2_body(pos[j], mass[j]) : fa2_no_body();
        }
        __syncthreads();
        const int n = min(kStage, (je - t0 + 7) & ~7);
        if constexpr (R == 1) fa2_rep_ahead(xi[0], tile, n, fx[0], fy[0]);
        else fa2_rep_run(xi, tile, n, fx, fy);
        __syncthreads();
    }
    if (kSegmented) {
#pragma unroll
        for (int r = 0; r < R; ++r)
            if (i + r * kFa2Tile < K) seg[(int64_t)by * K + i + r * kFa2Tile] = make_float2(fx[r], fy[r]);
        return;
    }
    double2 st = make_double2(0.0, 0.0);
    if (i < K) {
        const float2 f = fa2_net_force(xi[0], mass[i], kr, fx[0], fy[0], fa2_att_value(att, item_of, i), kg);
        F[i] = f;
        st = fa2_swing_traction(f, fprev[i], mass[i]);
    }
    st = fa2_sum256(st, ws);
    if (threadIdx.x == 0) part[bx] = st;
}

// Segment sums of the nodes of tile bx added in ascending segment order, then the rest
// of the force as in fa2_exact_force_tile.
__device__ __forceinline__ void fa2_combine_tile(int32_t bx, int32_t K, int32_t nseg, const float2 *__restrict__ seg,
                                                 const float2 *__restrict__ pos, const float *__restrict__ mass,
                                                 const float2 *__restrict__ att, const uint32_t *__restrict__ item_of,
                                                 float kr, float kg, const float2 *__restrict__ fprev,
                                                 float2 *__restrict__ F, double2 *__restrict__ part) {
    __shared__ double2 ws[kFa2Tile / kWave];
    const int32_t i = bx * kFa2Tile + threadIdx.x;
    double2 st = make_double2(0.0, 0.0);
    if (i < K) {
        float2 r = seg[i];
        for (int32_t q = 1; q < nseg; ++q) {
            const float2 v = seg[(int64_t)q * K + i];
            r.x += v.x;
            r.y += v.y;
        }
        if (fa2_nan(r.x, r.y)) r = fa2_rep_again(pos[i], K, pos, mass, kRepSegment);
        const float f_mi = mass[i];
        const float2 f = fa2_net_force(pos[i], f_mi, kr, r.x, r.y, fa2_att_value(att, item_of, i), kg);
        F[i] = f;
        st = fa2_swing_traction(f, fprev[i], f_mi);
    }
    st = fa2_sum256(st, ws);
    if (threadIdx.x == 0) part[bx] = st;
}

// The global speed from part[0, nparts) by one 256-thread block (fixed order); every
// thread gets it.
__device__ __forceinline__ float fa2_speed_of_parts(const double2 *__restrict__ part, int32_t nparts,
                                                    const float *__restrict__ speed_in, float tau) {
    __shared__ float s_speed;
    __shared__ double2 ws[kFa2Tile / kWave];
    double2 acc = make_double2(0.0, 0.0);
    for (int p = threadIdx.x; p < nparts; p += kFa2Tile) {
        acc.x += part[p].x;
        acc.y += part[p].y;
    }
    acc = fa2_sum256(acc, ws);
    if (threadIdx.x == 0) s_speed = fa2_global_speed(acc.x, acc.y, *speed_in, tau);
    __syncthreads();
    return s_speed;
}

// Local speeds and displacement, at global speed s, of the nodes bx*256 + t + q*stride;
// returns the thread's bounding box (xmin, xmax, ymin, ymax) of the moved positions.
__device__ __forceinline__ float4 fa2_move_tile(int32_t bx, int32_t stride, int32_t K, float2 *__restrict__ pos,
                                                float2 *__restrict__ fprev, const float2 *__restrict__ F, float s,
                                                float ks, float ksmax) {
    const float inf = __builtin_huge_valf();
    float4 bb = make_float4(inf, -inf, inf, -inf);
    for (int32_t i = bx * kFa2Tile + threadIdx.x; i < K; i += stride * kFa2Tile) {
        const float2 f = F[i];
        const float2 p = fa2_move(pos[i], f, fprev[i], s, ks, ksmax);
        pos[i] = p;
        fprev[i] = f;
        bb = make_float4(fminf(bb.x, p.x), fmaxf(bb.y, p.x), fminf(bb.z, p.y), fmaxf(bb.w, p.y));
    }
    return bb;
}

__device__ __forceinline__ float4 fa2_update_tile(int32_t bx, int32_t stride, int32_t K, float2 *__restrict__ pos,
                                                  float2 *__restrict__ fprev, const float2 *__restrict__ F,
                                                  const double2 *__restrict__ part, int32_t nparts,
                                                  const float *__restrict__ speed_in, float *__restrict__ speed_out,
                                                  float tau, float ks, float ksmax) {
    const float s = fa2_speed_of_parts(part, nparts, speed_in, tau);
    if (bx == 0 && threadIdx.x == 0) *speed_out = s;
    return fa2_move_tile(bx, stride, K, pos, fprev, F, s, ks, ksmax);
}

}  // namespace bgv
