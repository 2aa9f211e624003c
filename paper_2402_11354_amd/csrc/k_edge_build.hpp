// PEOs steps (1)-(3) for every edge: one wave per unit of whole nodes (as many
// as make at most 64 edges), 16 edges of it at a time, on the matrix cores.
//
// For edge e = x_u - x_v (Sec. 4.2 of the paper):
//   (1) e = e_reg + e_res with e_reg the orthogonal projection of e on the
//       direction [e_i / (sqrt(L) |e_i|)]_i (a zero block contributes zero);
//       w_reg = |e_reg| / |e|, w_res = |e_res| / |e|;
//   (2) the projection vectors a^i_j, b_j are inputs;
//   (3) code e[i] = sign * argmax_j |e_i . a^i_j| per subspace, and e[0] the
//       same over e_res and b_j.
// The codes are integers decided by floating point, so they are computed in
// single precision with one fixed operation order, element for element:
//   e_k = x_u[k] - x_v[k]; s_i = sqrt(fma chain of e_k^2 over block i);
//   p_ij = fma chain over the block of e_k * a^i_j[k] (ascending, from 0);
//   j* = first j with the largest |p_ij|, negative sign iff p_ij* < 0;
//   c = (s_1 + ... + s_L) / L' (L' = nonzero blocks, sequential adds);
//   e_res_k = fma(-(c / s_i), e_k, e_k); p_0j = fma chain over all k.
// A code byte is j* + m * [sign < 0].
//
// Compact records (L <= 4; the experiments' compact form keeps w_reg = 1,
// w_res = 0 and two one-byte scalars per edge): the record starts with the
// node header {g_lo, g_step, i_lo, i_step}, then 4 code bytes per edge (byte
// i-1 = e[i]), then 2 scalar bytes per edge: cg = floor((gp - g_lo)/g_step)
// and ci = rint((ie - i_lo)/i_step) (255: zero-length edge), with gp =
// g_e/|e| (l2; 0 otherwise) and ie = 1/|e| in single precision:
//   ne2 = S_1 + ... + S_L (S_i the block's fma chain), ne = sqrt(ne2),
//   |x|^2 = fma chain over the original coordinates in order,
//   gp = (0.5 (|u|^2 - |v|^2)) / ne, ie = 1 / ne,
//   g_lo..g_hi, i_lo..i_hi over the node's edges of nonzero length,
//   g_step = (g_hi - g_lo)/255, i_step = (i_hi - i_lo)/254.
// The rounding directions make the search's A_r a lower bound of the exact
// one (g rounded down; 1/|e| decoded half a step towards the safe side).
//
// Where the time goes.  Per edge the projections are 4 d m flops (2 d m per
// step (2) family), 262 GFLOP for a million nodes of degree 32 at d = 128 and
// m = 16, and each neighbour's row is gathered once (16 GB).  The fp32
// v_mfma_f32_16x16x4f32 adds its four products to the accumulator one after
// another in ascending k, each fused, so a chain of them is bit for bit the
// fmaf chain above (checked over normal, integer, wide-range and denormal
// operands) and the codes can come from it: rows = 16 directions, columns =
// 16 edges, so a lane holds four directions of one edge and the argmax is
// three compares in the lane and two across the lanes.
// MFMA step t wants coordinate 4t + g in lane group g = lane/16, while memory
// gives a lane four consecutive ones: both operands are loaded 16 bytes a
// lane and turned with four lane-group swaps (transpose4); the edge vectors
// then wait in LDS in step order (each is used by the codes, the norms and
// the residual), kSegment coordinates at a time, longer vectors being
// gathered again for the residual.
// Measured: 400,000 nodes of degree 32 at d = 128, L = 8, m = 16 (no perm)
// 86.8 -> 3.1 ms (one fma per operand load before; now the vector ALUs are
// busy 51% of the time, the matrix cores 22%, and a wave waits 44% of its
// cycles at 2.9 waves a SIMD); 20,000 nodes at d = 960, L = 16 27.9 -> 2.2 ms
// (55% waiting: two passes over segments of 240 coordinates, 20 KB of LDS, at
// 1.8 waves a SIMD).  The general instantiations (MT = 8, blocks one at a time,
// a coordinate at a time with a permutation), 100,000 nodes of the first shape:
// with a permutation 21.3 -> 1.6 ms, with SimHash signatures 31.8 -> 2.4 ms;
// 50,000 at m = 128 89 -> 1.9 ms.
#pragma once

#include <type_traits>

#include "peos_device.hpp"

namespace peos {

struct EdgeBuildArgs {
    const float* base;
    const int32_t* graph;
    const float* dirs_a;  // L x m x dp
    const float* dirs_b;  // m x d
    uint8_t* rec;         // n x node_stride bytes
    int32_t* err;         // graph-validation flag (0 = ok)
    int64_t n;
    int64_t node_stride, codes_off, scal_off;
    int d, R, L, m, metric;
    int half_scalars;  // precision form: scalars as four halves per edge
    const int32_t* perm;  // optional dimension permutation: coordinate k of
                          // the test's vectors is original coordinate perm[k]
    const float* sdirs;   // 64 x d SimHash vectors, or null
    int64_t sig_off;      // SimHash signatures within a record
    int unit_nodes;       // nodes per wave: 1 .. max(1, 64 / R)
};

constexpr int kCompactZeroEdge = 255;
// Coordinates of the 16 edges' vectors held in LDS at a time (a multiple of 16,
// so that every coordinate keeps its place mod 16): vectors of up to 256 are
// held whole and gathered once (11.6 KB a wave at d = 128, L = 8, so 14 waves a
// CU; 20.3 KB at d = 256); longer ones go by whole groups of four blocks, as
// many as make 256 coordinates at most (20 KB, eight waves a CU, at d = 960,
// L = 16) or one of up to 512 (37 KB), else by 256 wherever the blocks lie.
constexpr int kSegment = 256;
constexpr int kMaxGroup = 512;
constexpr int kChunkWords = 4 * 64 + 16;  // LDS words of 16 coordinates: four steps of 64
                                          // lanes, padded so that lanes four steps apart
                                          // (the block norms) use different banks
constexpr int kCodeRow = 36;              // code bytes of one edge, at most

// the codes are taken four blocks at a time
__host__ __device__ inline bool edge_build_groups(int d, int L, int m)
{
    // (with more than two direction tiles a block's own chains fill the
    // matrix cores, and four blocks' would not fit the registers)
    return m <= 32 && (L < 4 ? d : 4 * (d / L)) <= kMaxGroup;
}

__host__ __device__ inline int edge_build_segment(int d, int L, bool groups)
{
    if (d <= kSegment || (groups && L < 4)) return (d + 15) / 16 * 16;
    if (!groups) return kSegment;
    const int group = 4 * (d / L);
    return group > kSegment ? group : kSegment / group * group;
}

inline size_t edge_build_lds(int d, int L, bool groups)
{
    const int seg = edge_build_segment(d, L, groups);
    return sizeof(float) * ((size_t)(seg / 16) * kChunkWords + 16 * (size_t)L + 7 * 64) + 16 * kCodeRow;
}

// row (16-lane group) swaps of two registers: the odd rows of a with the even
// rows of b, and the upper half of a with the lower half of b
template <typename T>
__device__ __forceinline__ void swap_rows(T& a, T& b)
{
    const auto r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(uint32_t, a), __builtin_bit_cast(uint32_t, b),
                                                    false, false);
    a = __builtin_bit_cast(T, (uint32_t)r[0]);
    b = __builtin_bit_cast(T, (uint32_t)r[1]);
}

template <typename T>
__device__ __forceinline__ void swap_halves(T& a, T& b)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, a), __builtin_bit_cast(uint32_t, b),
                                                    false, false);
    a = __builtin_bit_cast(T, (uint32_t)r[0]);
    b = __builtin_bit_cast(T, (uint32_t)r[1]);
}

// 4 x 4 transpose between the four groups of 16 lanes and four registers:
// afterwards register c of group g holds what register g of group c held
__device__ __forceinline__ void transpose4(float (&x)[4])
{
    swap_halves(x[0], x[2]);
    swap_halves(x[1], x[3]);
    swap_rows(x[0], x[1]);
    swap_rows(x[2], x[3]);
}

// LDS word of step t (coordinates 4t .. 4t + 3 of the segment)
__device__ __forceinline__ int step_word(int t) { return (t >> 2) * kChunkWords + (t & 3) * 64; }

// An extreme product and its direction.  A larger |p| wins, ties go to the
// smaller direction, and a NaN loses to any number.
struct Extreme {
    float p;
    int j;
};

__device__ __forceinline__ Extreme extreme_of(Extreme a, Extreme b)
{
    const bool second = (fabsf(b.p) > fabsf(a.p)) | ((fabsf(b.p) == fabsf(a.p)) & (b.j < a.j)) | (a.p != a.p);
    return Extreme{second ? b.p : a.p, second ? b.j : a.j};
}

// this lane's extreme of one edge: acc[t][r] is direction 16 t + 4 g + r
template <int MT>
__device__ __forceinline__ Extreme lane_extreme(const floatx4* acc, int mt, int g)
{
    Extreme x{acc[0][0], 4 * g};
#pragma unroll
    for (int t = 0; t < MT; ++t) {
        if (t >= mt) break;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            if (t == 0 && r == 0) continue;
            const float p = acc[t][r];
            const bool up = (fabsf(p) > fabsf(x.p)) | (x.p != x.p);  // (directions ascend: no ties to settle)
            x = Extreme{up ? p : x.p, up ? 16 * t + 4 * g + r : x.j};
        }
    }
    return x;
}

// the code byte: the direction, plus m if its product is negative
__device__ __forceinline__ int code_of(Extreme x, int m) { return x.p != x.p ? 0 : x.j + (x.p < 0.f ? m : 0); }

// the extreme over the four lane groups, in every lane
__device__ __forceinline__ Extreme group_extreme(Extreme x)
{
    Extreme y = x;
    swap_rows(x.p, y.p);
    swap_rows(x.j, y.j);
    x = y = extreme_of(x, y);
    swap_halves(x.p, y.p);
    swap_halves(x.j, y.j);
    return extreme_of(x, y);
}

// the same for four blocks at once: lane group g receives block g's
__device__ __forceinline__ Extreme group_extreme4(Extreme (&x)[4])
{
    auto fold = [](Extreme& a, Extreme& b, auto swap) {
        swap(a.p, b.p);
        swap(a.j, b.j);
        return extreme_of(a, b);
    };
    auto rows = [](auto& a, auto& b) { swap_rows(a, b); };
    auto halves = [](auto& a, auto& b) { swap_halves(a, b); };
    Extreme lo = fold(x[0], x[1], rows), hi = fold(x[2], x[3], rows);
    return fold(lo, hi, halves);
}

// MT: 16-direction tiles, at least m / 16 (exactly, up to 2).  FULL: blocks are
// whole groups of four steps (d / L a multiple of 16), so no chunk of a block
// or a vector is partly filled.  GROUP: codes four blocks at a time (see
// edge_build_groups).  PERM: with a dimension permutation.
template <int MT, bool COMPACT, bool SIM, bool FULL, bool PERM, bool GROUP>
__global__ __launch_bounds__(64, MT <= 2 ? 4 : 3) void k_edge_build(EdgeBuildArgs a)
{
#pragma clang fp contract(off)
    extern __shared__ __align__(16) float smem[];
    const int d = a.d, R = a.R, L = a.L, m = a.m;
    const int dp = d / L;
    const int mt = MT <= 2 ? MT : m >> 4;
    const int seg = edge_build_segment(d, L, GROUP);
    float* et = smem;                                // the tile's edge vectors, in step order
    float* sb = et + (seg / 16) * kChunkWords;       // 16 x L block norms (compact: squared)
    int32_t* row = reinterpret_cast<int32_t*>(sb + 16 * L);  // the unit's neighbour ids
    float* nvs = reinterpret_cast<float*>(row + 64);         // |v|^2 per node of the unit
    // per edge of the unit, for the scalars at the end.  Compact: g_e/|e|,
    // 1/|e| and the kind; full: |u|^2, |e|^2, |e_res|^2, c, L'
    float* ea = nvs + 64;
    float* eb = ea + 64;
    float* ecn = eb + 64;
    float* ed = ecn + 64;
    int32_t* ei = reinterpret_cast<int32_t*>(ed + 64);
    uint8_t* cb = reinterpret_cast<uint8_t*>(ei + 64);  // 16 x kCodeRow: the tile's codes
    const int lane = lane_id();
    const int g = lane >> 4;    // lane group: K offset within an MFMA step
    const int ec = lane & 15;   // edge of the tile (and direction row of the other operand)

    const int64_t v0 = (int64_t)blockIdx.x * a.unit_nodes;
    const int nn = (int)(a.n - v0 < a.unit_nodes ? a.n - v0 : a.unit_nodes);
    const int E = nn * R;
    const uint32_t inv_r = (65535u + (uint32_t)R) / (uint32_t)R;
    auto node_of = [&](int f) { return (int)(((uint32_t)f * inv_r) >> 16); };  // f / R for f < 64
    if (lane < E) row[lane] = a.graph[v0 * R + lane];
    wave_sync();
    // graph validation: id range, self loop, repeated id in the row
    if (lane < E) {
        const int b = node_of(lane);
        const int32_t u = row[lane];
        bool bad = (u < -1) || (u >= a.n) || (u == v0 + b);
        for (int jj = 0; jj < R; ++jj) bad |= b * R + jj < lane && u >= 0 && row[b * R + jj] == u;
        if (bad) atomicOr(a.err, 1);
    }
    auto coord = [&](int k) { return PERM ? a.perm[k] : k; };
    if (!COMPACT && a.metric == 0) {
        // |v|^2: lane partials over k = lane mod 64, then the wave's tree
        // (four nodes' loads in flight together)
        for (int b = 0; b < nn; b += 4) {
            float s[4] = {0.f, 0.f, 0.f, 0.f};
            for (int k = lane; k < d; k += kWave) {
                const int kc = coord(k);
                float x[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) x[q] = a.base[(v0 + (b + q < nn ? b + q : b)) * d + kc];
#pragma unroll
                for (int q = 0; q < 4; ++q) s[q] = fmaf(x[q], x[q], s[q]);
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                s[q] = wave_sum(s[q]);
                if (lane == 0 && b + q < nn) nvs[b + q] = s[q];
            }
        }
    }
    // full records: round_up(B + 1, 4) code bytes per edge with B the
    // search kernel's subspace bound (8, 16 or 32; zero past L), byte 0 the
    // residual code; compact: 4 bytes, byte i-1 = e[i]
    const int cbytes = COMPACT ? 4 : (((L <= 8 ? 8 : (L <= 16 ? 16 : 32)) + 4) & ~3);
    const int cfirst = COMPACT ? 0 : 1;

    // coordinates k .. k + 3 of a row in the test's order
    auto load4 = [&](const float* x, int k) {
        if (!PERM) return *reinterpret_cast<const float4*>(x + k);
        return make_float4(x[a.perm[k]], x[a.perm[k + 1]], x[a.perm[k + 2]], x[a.perm[k + 3]]);
    };
    // four steps (coordinates k .. k + 15) of a tile of 16 directions of
    // `len` coordinates each, in step order (zeros from len on).  The SimHash
    // directions may start at any float, so the load claims no more than that
    // (the same 16-byte instruction: device memory serves it at any dword)
    auto dirs4 = [&](const float* dirs, int k, int len, float (&x)[4]) {
        const bool in = FULL || k + 4 * g < len;
        const floatx4u v = *reinterpret_cast<const floatx4u*>(dirs + (uint32_t)(ec * len + (in ? k + 4 * g : 0)));
        x[0] = in ? v.x : 0.f;
        x[1] = in ? v.y : 0.f;
        x[2] = in ? v.z : 0.f;
        x[3] = in ? v.w : 0.f;
        transpose4(x);
    };
    // the edges' vectors at four steps from coordinate k of the segment
    auto edges4 = [&](int k, int ns, float (&e)[4]) {
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int w = FULL ? (k >> 4) * kChunkWords + 64 * c : step_word((k >> 2) + c);
            e[c] = c < ns ? et[w + lane] : 0.f;
        }
    };

    // tiles of 16 edges; one without an edge (sparse rows, small graphs) gets
    // its zero records here
    const uint64_t present = ballot(lane < E && (uint32_t)row[lane] < (uint64_t)a.n);
    if (lane < E && ((present >> (lane & 48)) & 0xFFFFu) == 0) {
        const int b = node_of(lane), j = lane - b * R;
        uint8_t* rv = a.rec + (v0 + b) * a.node_stride;
        uint32_t* codes = reinterpret_cast<uint32_t*>(rv + a.codes_off + (int64_t)j * cbytes);
        for (int w = 0; w < cbytes >> 2; ++w) codes[w] = 0u;
        if (SIM) *reinterpret_cast<uint2*>(rv + a.sig_off + 8 * j) = make_uint2(0u, 0u);
        ei[lane] = COMPACT ? 0 : -1;
    }
    const int ntile = (E + 15) >> 4;
    for (int T = 0; T < ntile; ++T) {
        if (((present >> (16 * T)) & 0xFFFFu) == 0) continue;
        const int f = 16 * T + ec;
        int32_t u = f < E ? row[f] : -1;
        if (u >= a.n) u = -1;  // never dereferenced (reported through err)
        const bool ok = u >= 0;
        const int b = f < E ? node_of(f) : 0;
        const float* xv = a.base + (v0 + b) * d;
        const float* xu = ok ? a.base + (int64_t)u * d : xv;  // no edge: e = 0

        float nu[4] = {0.f, 0.f, 0.f, 0.f}, ne[4] = {0.f, 0.f, 0.f, 0.f};
        // N chunks of 16 coordinates from k of the segment at k0: the edge
        // vectors to LDS in step order, all loads first (straight-line code,
        // so that they are in flight together); `first` also sums |u|^2 and
        // |e|^2
        auto chunks = [&](auto count, int k0, int k, int len, bool first) {
            constexpr int N = decltype(count)::value;
            float4 p[N], q[N];
#pragma unroll
            for (int j = 0; j < N; ++j) {
                const int kk = k + 16 * j + 4 * g;
                const bool in = FULL || kk < len;  // else the row's start, dropped below
                p[j] = load4(xu, in ? k0 + kk : 0);
                q[j] = load4(xv, in ? k0 + kk : 0);
            }
#pragma unroll
            for (int j = 0; j < N; ++j) {
                if (!FULL && k + 16 * j + 4 * g >= len) p[j] = q[j] = make_float4(0.f, 0.f, 0.f, 0.f);
                float e[4] = {p[j].x - q[j].x, p[j].y - q[j].y, p[j].z - q[j].z, p[j].w - q[j].w};
                if (first) {
                    nu[0] = fmaf(p[j].x, p[j].x, nu[0]);
                    nu[1] = fmaf(p[j].y, p[j].y, nu[1]);
                    nu[2] = fmaf(p[j].z, p[j].z, nu[2]);
                    nu[3] = fmaf(p[j].w, p[j].w, nu[3]);
                }
                transpose4(e);
                float* w = et + step_word((k >> 2) + 4 * j) + lane;
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    if (first) ne[c] = fmaf(e[c], e[c], ne[c]);
                    w[64 * c] = e[c];
                }
            }
        };
        auto stage = [&](int k0, int len, bool first) {
            int k = 0;
            if (PERM) {  // (a coordinate at a time: fewer in flight)
                for (; k < len; k += 16) chunks(std::integral_constant<int, 1>(), k0, k, len, first);
                return;
            }
            for (; k + 128 <= len; k += 128) chunks(std::integral_constant<int, 8>(), k0, k, len, first);
            if (len - k > 48) {
                chunks(std::integral_constant<int, 4>(), k0, k, len, first);
                k += 64;
            }
            if (len - k > 16) {
                chunks(std::integral_constant<int, 2>(), k0, k, len, first);
                k += 32;
            }
            if (len - k > 0) chunks(std::integral_constant<int, 1>(), k0, k, len, first);
            if (len - k > 16) chunks(std::integral_constant<int, 1>(), k0, k + 16, len, first);
        };

        floatx4 acc[MT], sacc[SIM ? 4 : 1];
#pragma unroll
        for (int t = 0; t < (SIM ? 4 : 1); ++t) sacc[t] = floatx4{0.f, 0.f, 0.f, 0.f};
        wave_sync();  // the last tile's reads of the LDS buffers
        for (int k0 = 0; k0 < d; k0 += seg) {
            const int len = d - k0 < seg ? d - k0 : seg;
            if (k0) wave_sync();
            stage(k0, len, true);
            wave_sync();
            const int i0 = k0 / dp, i1 = (k0 + len - 1) / dp;
            // block norms: lane group g takes every fourth block, a chain
            // over the block's coordinates in order (continued where the
            // last segment ended inside the block)
            for (int i = i0 + g; i <= i1; i += 4) {
                const int kb = i * dp > k0 ? i * dp : k0;
                const int ke = (i + 1) * dp < k0 + len ? (i + 1) * dp : k0 + len;
                float ss = kb == i * dp ? 0.f : sb[ec * L + i];
                constexpr int NT = FULL ? 4 : 1;  // steps read together
                for (int t = (kb - k0) >> 2; t < (ke - k0) >> 2; t += NT) {
                    const float* w = et + step_word(t) + ec;
                    float x[4 * NT];
#pragma unroll
                    for (int q = 0; q < 4 * NT; ++q) x[q] = w[16 * q];
#pragma unroll
                    for (int q = 0; q < 4 * NT; ++q) ss = fmaf(x[q], x[q], ss);
                }
                sb[ec * L + i] = (!COMPACT && ke == (i + 1) * dp) ? sqrtf(ss) : ss;
            }
            // subspace codes
            if (GROUP) {
                // segments hold whole groups: four blocks' chains side by
                // side, then one exchange for the four extremes
                for (int ig = i0; ig <= i1; ig += 4) {
                    Extreme x4[4];
                    constexpr int Q = MT == 1 ? 4 : 1;  // chains side by side in one tile
#pragma unroll
                    for (int q0 = 0; q0 < 4; q0 += Q) {
                        floatx4 ac[Q][MT];
#pragma unroll
                        for (int q = 0; q < Q; ++q)
#pragma unroll
                            for (int t = 0; t < MT; ++t) ac[q][t] = floatx4{0.f, 0.f, 0.f, 0.f};
                        for (int ks = 0; ks < dp; ks += 16) {
                            const int ns = !FULL && dp - ks < 16 ? (dp - ks) >> 2 : 4;
                            float e[Q][4], x[Q][MT][4];
#pragma unroll
                            for (int q = 0; q < Q; ++q) {
                                const int i = ig + q0 + q <= i1 ? ig + q0 + q : i1;
#pragma unroll
                                for (int t = 0; t < MT; ++t)
                                    if (t < mt) dirs4(a.dirs_a + ((int64_t)i * m + 16 * t) * dp, ks, dp, x[q][t]);
                                edges4(i * dp - k0 + ks, ns, e[q]);
                            }
#pragma unroll
                            for (int c = 0; c < 4; ++c) {
                                if (c >= ns) break;
#pragma unroll
                                for (int q = 0; q < Q; ++q)
#pragma unroll
                                    for (int t = 0; t < MT; ++t)
                                        if (t < mt)
                                            ac[q][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[q][t][c], e[q][c],
                                                                                            ac[q][t], 0, 0, 0);
                            }
                        }
#pragma unroll
                        for (int q = 0; q < Q; ++q) x4[q0 + q] = lane_extreme<MT>(ac[q], mt, g);
                    }
                    const int code = code_of(group_extreme4(x4), m);
                    if (ig + g <= i1) cb[ec * kCodeRow + cfirst + ig + g] = ok ? (uint8_t)code : 0;
                }
            } else {
                for (int i = i0; i <= i1; ++i) {
                    const int kb = i * dp > k0 ? i * dp : k0;
                    const int ke = (i + 1) * dp < k0 + len ? (i + 1) * dp : k0 + len;
                    if (kb == i * dp) {
#pragma unroll
                        for (int t = 0; t < MT; ++t) acc[t] = floatx4{0.f, 0.f, 0.f, 0.f};
                    }
                    for (int k = kb; k < ke; k += 16) {
                        const int ns = ke - k < 16 ? (ke - k) >> 2 : 4;
                        float e[4];
                        edges4(k - k0, ns, e);
#pragma unroll
                        for (int t = 0; t < MT; ++t) {
                            if (t >= mt) break;
                            float x[4];
                            dirs4(a.dirs_a + ((int64_t)i * m + 16 * t) * dp, k - i * dp, dp, x);
#pragma unroll
                            for (int c = 0; c < 4; ++c)
                                if (c < ns) acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[c], e[c], acc[t], 0, 0, 0);
                        }
                    }
                    if (ke == (i + 1) * dp) {
                        const int code = code_of(group_extreme(lane_extreme<MT>(acc, mt, g)), m);
                        if (g == 0) cb[ec * kCodeRow + cfirst + i] = ok ? (uint8_t)code : 0;
                    }
                }
            }
            if (SIM) {
                // SimHash signature of e: bit i = [e . c_i >= 0], chains over
                // the coordinates in order (64 directions, four tiles)
                for (int k = 0; k < len; k += 16) {
                    const int ns = !FULL && len - k < 16 ? (len - k) >> 2 : 4;
#pragma unroll
                    for (int t = 0; t < 4; ++t) {
                        float x[4];
                        dirs4(a.sdirs + (int64_t)(16 * t) * d, k0 + k, d, x);
#pragma unroll
                        for (int c = 0; c < 4; ++c)
                            if (c < ns)
                                sacc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(
                                    x[c], et[step_word((k >> 2) + c) + lane], sacc[t], 0, 0, 0);
                    }
                }
            }
        }
        wave_sync();  // block norms and codes in LDS

        uint8_t* rv = a.rec + (v0 + b) * a.node_stride;
        const int j = f - b * R;  // edge slot within its node
        if (COMPACT) {
            // compact scalars in the order stated above; |u|^2 and |v|^2 as
            // chains in the original coordinate order, lane group 0 and 1
            float x2 = 0.f;
            if (a.metric == 0 && g < 2) {
                const float* x = g == 0 ? xu : xv;
                for (int k = 0; k < d; k += 4) {
                    const float4 t = *reinterpret_cast<const float4*>(x + k);
                    x2 = fmaf(t.x, t.x, x2);
                    x2 = fmaf(t.y, t.y, x2);
                    x2 = fmaf(t.z, t.z, x2);
                    x2 = fmaf(t.w, t.w, x2);
                }
            }
            const float nv2 = __shfl_xor(x2, 16, kWave);
            if (g == 0 && f < E) {
                int kd = 0;
                float gp = 0.f, ie = 0.f;
                if (ok) {
                    float ne2 = 0.f;
                    for (int i = 0; i < L; ++i) ne2 = ne2 + sb[ec * L + i];
                    const float nrm = sqrtf(ne2);
                    kd = 2;
                    if (nrm > 0.f) {
                        kd = 1;
                        if (a.metric == 0) gp = (0.5f * (x2 - nv2)) / nrm;
                        ie = 1.f / nrm;
                    }
                }
                ea[f] = gp;
                eb[f] = ie;
                ei[f] = kd;
                uint32_t w = 0u;
                for (int i = 0; i < L; ++i) w |= (uint32_t)cb[ec * kCodeRow + i] << (8 * i);
                *reinterpret_cast<uint32_t*>(rv + a.codes_off + 4 * j) = w;
            }
            continue;
        }

        if (SIM) {
            uint32_t lo = 0u, hi = 0u;
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const uint32_t bit = sacc[t][r] >= 0.f ? 1u << ((16 * t + 4 * g + r) & 31) : 0u;
                    if (t < 2) lo |= bit;
                    else hi |= bit;
                }
            lo |= (uint32_t)__shfl_xor((int)lo, 16, kWave);
            lo |= (uint32_t)__shfl_xor((int)lo, 32, kWave);
            hi |= (uint32_t)__shfl_xor((int)hi, 16, kWave);
            hi |= (uint32_t)__shfl_xor((int)hi, 32, kWave);
            if (g == 0 && f < E)
                *reinterpret_cast<uint2*>(rv + a.sig_off + 8 * j) = ok ? make_uint2(lo, hi) : make_uint2(0u, 0u);
        }

        // regular part: c = sum(s_i) / L'
        float c = 0.f, ssum = 0.f;
        int nz = 0;
        for (int i = 0; i < L; ++i) {
            const float s = sb[ec * L + i];
            ssum = ssum + s;
            nz += s > 0.f;
        }
        c = nz > 0 ? ssum / (float)nz : 0.f;
        // c / s_i, each lane group every fourth block, in place of the norms
        wave_sync();
        for (int i = g; i < L; i += 4) {
            const float s = sb[ec * L + i];
            sb[ec * L + i] = s > 0.f ? c / s : 0.f;
        }
        wave_sync();

        // residual e - (c / s_i) e and its code, four steps at a time
        float nr[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int t = 0; t < MT; ++t) acc[t] = floatx4{0.f, 0.f, 0.f, 0.f};
        int bnd = 0, blk = 0;  // the next block and where it starts
        float ratio = 0.f;
        for (int k0 = 0; k0 < d; k0 += seg) {
            const int len = d - k0 < seg ? d - k0 : seg;
            if (d > seg) {
                wave_sync();
                stage(k0, len, false);
                wave_sync();
            }
            for (int k = 0; k < len; k += 16) {
                const int ns = !FULL && len - k < 16 ? (len - k) >> 2 : 4;
                float e[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    if (q >= ns) {
                        e[q] = 0.f;
                        continue;
                    }
                    if ((!FULL || q == 0) && k0 + k + 4 * q == bnd) {
                        ratio = sb[ec * L + blk];
                        ++blk;
                        bnd += dp;
                    }
                    const float x = et[step_word((k >> 2) + q) + lane];
                    e[q] = fmaf(-ratio, x, x);
                    nr[q] = fmaf(e[q], e[q], nr[q]);
                }
#pragma unroll
                for (int t = 0; t < MT; ++t) {
                    if (t >= mt) break;
                    float x[4];
                    dirs4(a.dirs_b + (int64_t)(16 * t) * d, k0 + k, d, x);
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        if (q < ns) acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[q], e[q], acc[t], 0, 0, 0);
                }
            }
        }
        const int rcode = code_of(group_extreme(lane_extreme<MT>(acc, mt, g)), m);
        if (g == 0) {
            cb[ec * kCodeRow] = ok ? (uint8_t)rcode : 0;
            for (int pz = L + 1; pz < cbytes; ++pz) cb[ec * kCodeRow + pz] = 0;
        }
        // sums over k mod 16 (register: k / 4 mod 4, lane group: k mod 4 in
        // step order; the other way round for |u|^2), then the tree over 8,
        // 4, 2, 1
        auto tree = [&](const float (&x)[4]) {
            float s = (x[0] + x[2]) + (x[1] + x[3]);
            s += xor_lane<32>(s);
            return s + xor_lane<16>(s);
        };
        const float ne2 = tree(ne), nr2 = tree(nr);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            nu[q] += xor_lane<32>(nu[q]);
            nu[q] += xor_lane<16>(nu[q]);
        }
        if (g == 0 && f < E) {
            ea[f] = (nu[0] + nu[2]) + (nu[1] + nu[3]);
            eb[f] = ne2;
            ecn[f] = nr2;
            ed[f] = c;
            ei[f] = ok ? nz : -1;
        }
        // the codes: lane group g stores every fourth dword of its edge
        wave_sync();
        if (f < E)
            for (int w = g; w < cbytes >> 2; w += 4)
                *reinterpret_cast<uint32_t*>(rv + a.codes_off + (int64_t)j * cbytes + 4 * w) =
                    *reinterpret_cast<const uint32_t*>(cb + ec * kCodeRow + 4 * w);
    }
    wave_sync();
    if (lane >= E) return;
    const int b = node_of(lane), j = lane - b * R;
    uint8_t* rv = a.rec + (v0 + b) * a.node_stride;
    if (!COMPACT) {
        // scalars of the unit's edges, one per lane: g_e, |e|, w_reg, sqrt(L)
        // w_res; in the precision form the halves of g_e/|e|, 1/|e| (infinite
        // for a zero edge), w_reg, sqrt(L) w_res
        float ge = 0.f, en = 0.f, wreg = 0.f, swres = 0.f;
        const int nz = ei[lane];
        const bool ok = nz >= 0;
        if (ok) {
            en = sqrtf(eb[lane]);
            if (en > 0.f) {
                wreg = fminf(1.f, ed[lane] * sqrtf((float)nz) / en);
                swres = sqrtf((float)L) * fminf(1.f, sqrtf(ecn[lane]) / en);
            } else {
                wreg = 1.f;
                swres = 0.f;
            }
            if (a.metric == 0) ge = 0.5f * (ea[lane] - nvs[b]);
        }
        if (a.half_scalars) {
            const float gp = en > 0.f ? ge / en : 0.f;
            const float ie = en > 0.f ? 1.f / en : INFINITY;
            _Float16* hs = reinterpret_cast<_Float16*>(rv + a.scal_off) + 4 * j;
            hs[0] = (_Float16)(ok ? gp : 0.f);
            hs[1] = (_Float16)(ok ? ie : 0.f);
            hs[2] = (_Float16)wreg;
            hs[3] = (_Float16)swres;
        } else {
            *reinterpret_cast<float4*>(reinterpret_cast<float*>(rv + a.scal_off) + 4 * j) =
                make_float4(ge, en, wreg, swres);
        }
        return;
    }
    // compact: node ranges (min / max are exact in any order) and the codes
    float glo = INFINITY, ghi = -INFINITY, ilo = INFINITY, ihi = -INFINITY;
    for (int t = b * R; t < (b + 1) * R; ++t) {
        if (ei[t] != 1) continue;
        glo = fminf(glo, ea[t]);
        ghi = fmaxf(ghi, ea[t]);
        ilo = fminf(ilo, eb[t]);
        ihi = fmaxf(ihi, eb[t]);
    }
    if (!(glo <= ghi)) glo = ghi = ilo = ihi = 0.f;  // no edge of nonzero length
    const float gstep = (ghi - glo) / 255.f;
    const float istep = (ihi - ilo) / 254.f;
    if (j == 0) *reinterpret_cast<float4*>(rv) = make_float4(glo, gstep, ilo, istep);
    uint32_t cg = 0u, ci = 0u;
    if (ei[lane] == 2) ci = kCompactZeroEdge;
    if (ei[lane] == 1) {
        if (gstep > 0.f) {
            const float c = floorf((ea[lane] - glo) / gstep);
            cg = (uint32_t)(c < 0.f ? 0.f : (c > 255.f ? 255.f : c));
        }
        if (istep > 0.f) {
            const float c = rintf((eb[lane] - ilo) / istep);
            ci = (uint32_t)(c < 0.f ? 0.f : (c > 254.f ? 254.f : c));
        }
    }
    reinterpret_cast<uint16_t*>(rv + a.scal_off)[j] = (uint16_t)(cg | (ci << 8));
}

// Energy of the edge coordinates for the optional dimension permutation:
// partial[b][j] = sum over the edges (v, u) of the nodes v = b, b + grid, ...
// of (x_u[j] - x_v[j])^2, in that fixed order (threads over coordinates).
__global__ __launch_bounds__(256) void k_edge_energy(const float* base, const int32_t* graph,
                                                     int64_t n, int d, int R, float* partial)
{
    for (int j = threadIdx.x; j < d; j += blockDim.x) {
        float acc = 0.f;
        for (int64_t v = blockIdx.x; v < n; v += gridDim.x) {
            const float xv = base[v * d + j];
            for (int r = 0; r < R; ++r) {
                const int32_t u = graph[v * R + r];
                if (u < 0 || u >= n) continue;
                const float t = base[(int64_t)u * d + j] - xv;
                acc = fmaf(t, t, acc);
            }
        }
        partial[(int64_t)blockIdx.x * d + j] = acc;
    }
}

// bfloat16 copy of the base (round to nearest even), the traversal copy of
// the precision form
__global__ void k_to_bf16(const float* x, uint16_t* y, int64_t count)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += stride) {
        uint32_t u = __float_as_uint(x[i]);
        if ((u & 0x7f800000u) != 0x7f800000u) u += 0x7fffu + ((u >> 16) & 1u);
        y[i] = (uint16_t)(u >> 16);
    }
}

}  // namespace peos
