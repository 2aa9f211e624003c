// PEOs step (5): the projection table of every query, on the matrix cores.
//
// tables[q][i][j] = q'_i . a^i_j (i = 1..L) and tables[q][0][j] = q' . b_j,
// with q' = q/|q| and q'_i its i-th block (Sec. 4.2; the table is built once
// per query, Alg. 2).  As a matrix product this is Q x [B^T | blockdiag(A^i)^T]
// scaled by 1/|q| per row; the block-diagonal structure is kept (each
// subspace contracts over its own d/L coordinates only).
//
// Each 16-query x 16-direction output tile is one chain of
// v_mfma_f32_16x16x4f32 (fp32 in, fp32 accumulate): per K step of 4, lane l
// feeds A[row = l%16][k = l/16] (queries) and B[k = l/16][col = l%16]
// (directions), and receives D[row = 4*(l/16) + r][col = l%16], r = 0..3.
// The precision form stores the table as halves.
#pragma once

#include <type_traits>

#include "peos_device.hpp"

namespace peos {

struct QueryTableArgs {
    const float* queries;  // nq x d
    const float* dirs_a;   // L x m x dp
    const float* dirs_b;   // m x d
    float* tables;         // nq x (L+1) x m floats, or halves when half_out
    float* qnorms;         // nq
    int64_t nq;
    int d, L, m;
    int half_out;          // store the table as IEEE halves (round to nearest even)
    int staged;            // the tile's rows are staged in LDS (16 (d + 4) floats fit)
    const int32_t* perm;   // optional dimension permutation of the test
};

// One workgroup of kTableWaves waves per tile of 16 queries (for m > 16 and few
// queries several of kWideWaves, see query_table_wide).  The tile's
// query rows are staged in LDS with coalesced 16-byte loads (row stride
// d + 4 floats, so the 16 rows x 4 consecutive k an MFMA step reads fall in
// 64 distinct banks; up to 61 KB at d = 960); the (L+1) x m/16 output tiles
// are dealt out to the waves.  With staged rows and no permutation both
// operands are read 16 bytes per lane: a group of four K steps per load.
constexpr int kTableWaves = 4;
constexpr int kWideWaves = 8;  // of the body for m > 16

// |q| of this lane's row (lane % 16) from the staged rows:
// sqrt((p0 + p1) + (p2 + p3)), p_j the fma chain of q_k^2 over k = j mod 4
// (one lane each, eight terms read together, then chained), combined by two
// xor shuffles, so that every lane of the row holds the same value.
__device__ __forceinline__ float staged_row_norm(const float* ql, int d, int kq)
{
    float ss = 0.f;
    int k = kq;
    for (; k + 28 < d; k += 32) {
        float v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = ql[k + 4 * j];
#pragma unroll
        for (int j = 0; j < 8; ++j) ss = fmaf(v[j], v[j], ss);
    }
    for (; k < d; k += 4) ss = fmaf(ql[k], ql[k], ss);
    ss += __shfl_xor(ss, 16, kWave);
    ss += __shfl_xor(ss, 32, kWave);
    return sqrtf(ss);
}

// N consecutive K groups j.. of one tile: all loads first, then the MFMAs
// (straight-line code, so that no load waits behind another's wait)
template <int N>
__device__ __forceinline__ floatx4 mfma_groups(floatx4 acc, const float* av, const float* bv, int j, int k4)
{
    float4 bq[N], aq[N];
#pragma unroll
    for (int u = 0; u < N; ++u) {
        bq[u] = *reinterpret_cast<const float4*>(bv + 16 * (j + u) + k4);
        aq[u] = *reinterpret_cast<const float4*>(av + 16 * (j + u) + k4);
    }
#pragma unroll
    for (int u = 0; u < N; ++u) {
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(aq[u].x, bq[u].x, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(aq[u].y, bq[u].y, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(aq[u].z, bq[u].z, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(aq[u].w, bq[u].w, acc, 0, 0, 0);
    }
    return acc;
}

// One round trip for a wave's whole work when it is at most 4 full-space
// groups (N of them, from group g0) and at most 4 subspace tiles of exactly
// one group each (d / L = 16; T tile slots, at least the wave's tiles): every
// load first, then the MFMAs in each accumulator's order.
template <int N, int T>
__device__ __forceinline__ void one_round(floatx4& part, floatx4 (&acc)[4], const float* ql,
                                          const float* brow, int g0, const float* const (&at)[4],
                                          const float* const (&bt)[4], int k4)
{
    float4 bq[N > 0 ? N : 1], aq[N > 0 ? N : 1], tb[T], ta[T];
#pragma unroll
    for (int u = 0; u < N; ++u) {
        bq[u] = *reinterpret_cast<const float4*>(brow + 16 * (g0 + u) + k4);
        aq[u] = *reinterpret_cast<const float4*>(ql + 16 * (g0 + u) + k4);
    }
#pragma unroll
    for (int u = 0; u < T; ++u) {
        tb[u] = *reinterpret_cast<const float4*>(bt[u] + k4);
        ta[u] = *reinterpret_cast<const float4*>(at[u] + k4);
    }
#pragma unroll
    for (int u = 0; u < N; ++u) {
        part = __builtin_amdgcn_mfma_f32_16x16x4f32(aq[u].x, bq[u].x, part, 0, 0, 0);
        part = __builtin_amdgcn_mfma_f32_16x16x4f32(aq[u].y, bq[u].y, part, 0, 0, 0);
        part = __builtin_amdgcn_mfma_f32_16x16x4f32(aq[u].z, bq[u].z, part, 0, 0, 0);
        part = __builtin_amdgcn_mfma_f32_16x16x4f32(aq[u].w, bq[u].w, part, 0, 0, 0);
    }
#pragma unroll
    for (int u = 0; u < T; ++u) {
        floatx4 c = {0.f, 0.f, 0.f, 0.f};
        c = __builtin_amdgcn_mfma_f32_16x16x4f32(ta[u].x, tb[u].x, c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_16x16x4f32(ta[u].y, tb[u].y, c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_16x16x4f32(ta[u].z, tb[u].z, c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_16x16x4f32(ta[u].w, tb[u].w, c, 0, 0, 0);
        acc[u] = c;
    }
}

template <int T>
__device__ __forceinline__ void one_round_n(int n0, floatx4& part, floatx4 (&acc)[4], const float* ql,
                                            const float* brow, int g0, const float* const (&at)[4],
                                            const float* const (&bt)[4], int k4)
{
    switch (n0) {
    case 4: one_round<4, T>(part, acc, ql, brow, g0, at, bt, k4); break;
    case 3: one_round<3, T>(part, acc, ql, brow, g0, at, bt, k4); break;
    case 2: one_round<2, T>(part, acc, ql, brow, g0, at, bt, k4); break;
    case 1: one_round<1, T>(part, acc, ql, brow, g0, at, bt, k4); break;
    default: one_round<0, T>(part, acc, ql, brow, g0, at, bt, k4); break;
    }
}

// m = 16, staged rows, no permutation (every workload's shape), a body of
// its own in which every wave takes the norms itself (no barrier between
// the norms and the products) and the loads of each round trip are issued
// together as straight-line code.
// The full-space tile (K = d, L times a subspace tile's K) is split over the
// waves, four K groups per round trip, and the parts summed at the end in
// the order (p0 + p1) + (p2 + p3); the subspace tiles go round robin (tile
// 1 + wv + 4 s to wave wv), four tiles per round trip, each taking its K
// groups, then its last dp mod 16 steps, in order.  When a wave's whole
// work fits one round trip (d / L = 16, at most 4 full-space groups and 4
// tiles per wave: d = 128, L = 8) it is requested at once.  A block of 16
// queries then takes as long as a kernel of the same grid that only reads
// its rows and writes its tables.  Rows past the batch are zero and not
// stored.
__device__ __forceinline__ void query_table16(const QueryTableArgs& a, float* qs, int nrows,
                                              int64_t q0, int wv, int lane)
{
#pragma clang fp contract(off)
    const int d = a.d, L = a.L;
    const int dp = d / L;
    const int ld = d + 4;
    const int row = lane & 15;  // A row, and B column (direction)
    const int kq = lane >> 4;   // K offset within a step
    const float* ql = qs + row * ld;

    const int ng = d >> 4;
    const int per = (ng + kTableWaves - 1) / kTableWaves;
    const int g0 = wv * per < ng ? wv * per : ng;
    const int g1 = g0 + per < ng ? g0 + per : ng;
    const float* brow = a.dirs_b + (int64_t)row * d;
    const int gpt = dp >> 4;
    const int ntw = L > wv ? (L - wv + kTableWaves - 1) / kTableWaves : 0;
    // operands of the wave's tiles sb .. sb + 3 (a slot past its last tile
    // repeats that tile: computed, not stored)
    auto tile_ptrs = [&](int sb, const float* (&at)[4], const float* (&bt)[4]) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int s = sb + u < ntw ? sb + u : ntw - 1;
            const int blk = wv + kTableWaves * s;  // subspace i - 1
            bt[u] = a.dirs_a + ((int64_t)blk * 16 + row) * dp;
            at[u] = ql + blk * dp;
        }
    };

    floatx4 part = {0.f, 0.f, 0.f, 0.f};
    floatx4 acc[4];
    const float* at[4];
    const float* bt[4];
    const int n0 = g1 - g0;
    const bool single = dp == 16 && n0 <= 4 && ntw >= 1 && ntw <= 4;
    if (single) {
        tile_ptrs(0, at, bt);
        if (ntw == 1) one_round_n<1>(n0, part, acc, ql, brow, g0, at, bt, 4 * kq);
        else if (ntw == 2) one_round_n<2>(n0, part, acc, ql, brow, g0, at, bt, 4 * kq);
        else one_round_n<4>(n0, part, acc, ql, brow, g0, at, bt, 4 * kq);
    } else {
        int j = g0;
        for (; j + 4 <= g1; j += 4) part = mfma_groups<4>(part, ql, brow, j, 4 * kq);
        switch (g1 - j) {
        case 3: part = mfma_groups<3>(part, ql, brow, j, 4 * kq); break;
        case 2: part = mfma_groups<2>(part, ql, brow, j, 4 * kq); break;
        case 1: part = mfma_groups<1>(part, ql, brow, j, 4 * kq); break;
        default: break;
        }
    }
    if (wv == kTableWaves - 1)
        for (int k0 = 16 * ng; k0 < d; k0 += 4)
            part = __builtin_amdgcn_mfma_f32_16x16x4f32(ql[k0 + kq], brow[k0 + kq], part, 0, 0, 0);

    const float nrm = staged_row_norm(ql, d, kq);
    const float inv = (nrm > 0.f && nrm < INFINITY) ? 1.f / nrm : 0.f;
    if (wv == 0 && kq == 0 && row < nrows) a.qnorms[q0 + row] = nrm;
    float invr[4];  // 1/|q| of output row 4 kq + r
#pragma unroll
    for (int r = 0; r < 4; ++r) invr[r] = __shfl(inv, 4 * kq + r, kWave);
    auto store = [&](const floatx4& v, int i) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int orow = 4 * kq + r;
            if (orow < nrows) {
                const float tv = v[r] * invr[r];
                const int64_t o = ((q0 + orow) * (L + 1) + i) * 16 + row;
                if (a.half_out) reinterpret_cast<_Float16*>(a.tables)[o] = (_Float16)tv;
                else a.tables[o] = tv;
            }
        }
    };

    if (single) {
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (u < ntw) store(acc[u], 1 + wv + kTableWaves * u);
    } else {
        for (int sb = 0; sb < ntw; sb += 4) {
            tile_ptrs(sb, at, bt);
#pragma unroll
            for (int u = 0; u < 4; ++u) acc[u] = floatx4{0.f, 0.f, 0.f, 0.f};
            for (int jg = 0; jg < gpt; ++jg) {
                float4 bq[4], aq[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    bq[u] = *reinterpret_cast<const float4*>(bt[u] + 16 * jg + 4 * kq);
                    aq[u] = *reinterpret_cast<const float4*>(at[u] + 16 * jg + 4 * kq);
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    acc[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(aq[u].x, bq[u].x, acc[u], 0, 0, 0);
                    acc[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(aq[u].y, bq[u].y, acc[u], 0, 0, 0);
                    acc[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(aq[u].z, bq[u].z, acc[u], 0, 0, 0);
                    acc[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(aq[u].w, bq[u].w, acc[u], 0, 0, 0);
                }
            }
            for (int k0 = 16 * gpt; k0 < dp; k0 += 4) {
                float bs[4], as[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    bs[u] = bt[u][k0 + kq];
                    as[u] = at[u][k0 + kq];
                }
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    acc[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(as[u], bs[u], acc[u], 0, 0, 0);
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (sb + u < ntw) store(acc[u], 1 + wv + kTableWaves * (sb + u));
        }
    }

    // the parts to LDS (the staged rows are dead once every wave is past its
    // MFMAs and norms), then wave 0 sums them
    __syncthreads();
    *reinterpret_cast<floatx4*>(qs + (wv * 64 + lane) * 4) = part;
    __syncthreads();
    if (wv == 0) {
        floatx4 p[kTableWaves];
#pragma unroll
        for (int w = 0; w < kTableWaves; ++w) p[w] = *reinterpret_cast<const floatx4*>(qs + (w * 64 + lane) * 4);
        floatx4 sum;
#pragma unroll
        for (int r = 0; r < 4; ++r) sum[r] = (p[0][r] + p[1][r]) + (p[2][r] + p[3][r]);
        store(sum, 0);
    }
}

// m > 16, staged rows, no permutation, few queries: the (L + 1) m / 16 output
// tiles of a block of 16 queries are dealt to the waves of gridDim.y workgroups by their
// number of K steps (a full-space tile counts as L subspace tiles: it is one
// chain and is not split), so that a few queries with many directions fill the
// chip.  Every tile keeps its chain of MFMAs in the order of K, so the table
// does not depend on the split.  Subspace tiles go four at a time, full-space
// tiles one at a time, the next group's operands loaded before a group's
// MFMAs; wave 0 takes the norms before its tiles, and the one barrier stands
// between the first tiles' MFMAs and their stores.
// What bounds it: the directions are read from L2 once per 16 queries, 1 MB
// at m = 128, d = 960 (2.1M requests of 64 bytes at 2,049 queries), and the
// latency of a full-space tile's 60 groups; the MFMAs take 6.5 us of it.
// 2,049 queries there: 65 us with one workgroup per 16 queries and a load's
// latency before every 16 MFMAs, 37 us with the tiles dealt out, 33 us with
// 64 bytes of a direction by four lanes.
// ROWS (m < 64, d >= 512): a direction by each lane of 16 instead, as the matrix
// cores take it.  With two or three direction tiles there are too few chains for
// the caches to bound them, and the permutes stand in each long one's way: 2,049
// queries at d = 960, L = 16, m = 32 19.8 -> 17.6 us, one query at L = 1 13.5 ->
// 12.1.  With more tiles it is the other way (m = 64, d = 512, L = 8: 15.1 with
// the permutes, 16.0 without), and with short rows too (m = 48, d = 32, L = 4, 300
// queries: 5.8 and 6.6).
template <bool ROWS>
__device__ __forceinline__ void query_table_wide(const QueryTableArgs& a, const float* qs, float* inv_norm,
                                                 int nrows, int64_t q0, int wv, int lane)
{
#pragma clang fp contract(off)
    const int d = a.d, L = a.L, m = a.m, mt = m >> 4;
    const int dp = d / L;
    const int row = lane & 15;
    const int kq = lane >> 4;
    const float* ql = qs + row * (d + 4);
    const int lrow = ROWS ? row : lane >> 2, lk = 4 * (ROWS ? kq : lane & 3);  // this lane's part of a load

    if (wv == 0) {
        const float nrm = staged_row_norm(ql, d, kq);
        if (kq == 0) {
            inv_norm[row] = (nrm > 0.f && nrm < INFINITY) ? 1.f / nrm : 0.f;
            if (blockIdx.y == 0 && row < nrows) a.qnorms[q0 + row] = nrm;
        }
    }
    // this wave's tiles: work units [u0, u1) of the 2 L mt of the block, the
    // full-space tiles' L units each first; a tile belongs to the wave that
    // holds its first unit
    const int nw = kWideWaves * (int)gridDim.y, w = (int)blockIdx.y * kWideWaves + wv;
    const int U = 2 * L * mt;
    const int u0 = (int)((int64_t)U * w / nw), u1 = (int)((int64_t)U * (w + 1) / nw);
    const int nf = L * mt;  // units of the full-space tiles
    const int f0 = ((u0 < nf ? u0 : nf) + L - 1) / L, f1 = ((u1 < nf ? u1 : nf) + L - 1) / L;
    const int s0 = u0 > nf ? u0 - nf : 0, s1 = u1 > nf ? u1 - nf : 0;  // subspace tiles (i - 1) mt + j

    auto store = [&](const floatx4& v, int i, int j) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int orow = 4 * kq + r;
            if (orow < nrows) {
                const float tv = v[r] * inv_norm[orow];
                const int64_t o = ((q0 + orow) * (L + 1) + i) * m + 16 * j + row;
                if (a.half_out) reinterpret_cast<_Float16*>(a.tables)[o] = (_Float16)tv;
                else a.tables[o] = tv;
            }
        }
    };
    // one chain over K = len of each of N tiles, in groups of 16 (step c of
    // group g: k = 16 g + 4 (lane / 16) + c for both operands), then the last
    // len mod 16 step by step.  G groups of every tile (N G = 4) are requested
    // while the G before them are multiplied, 64 bytes of a direction by four
    // lanes (by_row); the query operand comes from LDS as it is used.  bv: a
    // tile's first direction.
    auto chains = [&](auto tiles, const auto& av, const auto& bv, int len, auto& acc) __attribute__((always_inline)) {
        constexpr int N = decltype(tiles)::value, G = 4 / N;
        const int ng = len >> 4;
        auto load = [&](float4 (&b)[G][N], int g) __attribute__((always_inline)) {
#pragma unroll
            for (int j = 0; j < G; ++j)
#pragma unroll
                for (int u = 0; u < N; ++u)
                    b[j][u] = *reinterpret_cast<const float4*>(bv[u] + lrow * len +
                                                               16 * (g + j < ng ? g + j : ng - 1) + lk);
        };
        // n groups from g on (all operands first, then the MFMAs)
        auto mul = [&](float4 (&b)[G][N], int g, int n) __attribute__((always_inline)) {
            float4 aq[G][N];
#pragma unroll
            for (int j = 0; j < G; ++j)
#pragma unroll
                for (int u = 0; u < N; ++u) {
                    if (!ROWS) b[j][u] = by_row(b[j][u]);
                    aq[j][u] = *reinterpret_cast<const float4*>(av[u] + 16 * (g + j < ng ? g + j : ng - 1) + 4 * kq);
                }
#pragma unroll
            for (int j = 0; j < G; ++j) {
                if (j >= n) break;
#pragma unroll
                for (int u = 0; u < N; ++u) acc[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(aq[j][u].x, b[j][u].x, acc[u], 0, 0, 0);
#pragma unroll
                for (int u = 0; u < N; ++u) acc[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(aq[j][u].y, b[j][u].y, acc[u], 0, 0, 0);
#pragma unroll
                for (int u = 0; u < N; ++u) acc[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(aq[j][u].z, b[j][u].z, acc[u], 0, 0, 0);
#pragma unroll
                for (int u = 0; u < N; ++u) acc[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(aq[j][u].w, b[j][u].w, acc[u], 0, 0, 0);
            }
        };
        // the remainder's operands (at most three steps), requested first
        const int nr = (len - 16 * ng) >> 2;
        float br[3][N];
#pragma unroll
        for (int q = 0; q < 3; ++q)
#pragma unroll
            for (int u = 0; u < N; ++u) br[q][u] = q < nr ? bv[u][row * len + 16 * ng + 4 * q + kq] : 0.f;
        if (ng > 0) {
            float4 b0[G][N], b1[G][N];
            load(b0, 0);
            int g = 0;
            for (; g + 2 * G <= ng; g += 2 * G) {
                load(b1, g + G);
                mul(b0, g, G);
                load(b0, g + 2 * G);  // (past the end: the last group again, not used)
                mul(b1, g + G, G);
            }
            if (g < ng) {
                load(b1, g + G);
                mul(b0, g, ng - g);
                if (g + G < ng) mul(b1, g + G, ng - g - G);
            }
        }
#pragma unroll
        for (int q = 0; q < 3; ++q)
            if (q < nr)
#pragma unroll
                for (int u = 0; u < N; ++u)
                    acc[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[u][16 * ng + 4 * q + kq], br[q][u], acc[u], 0, 0, 0);
    };

    bool waited = false;
    auto wait_norms = [&]() {
        if (!waited) __syncthreads();
        waited = true;
    };
    for (int t = f0; t < f1; ++t) {
        floatx4 acc[1] = {floatx4{0.f, 0.f, 0.f, 0.f}};
        const float* av[1] = {ql};
        const float* bv[1] = {a.dirs_b + (int64_t)(16 * t) * d};
        chains(std::integral_constant<int, 1>(), av, bv, d, acc);
        wait_norms();
        store(acc[0], 0, t);
    }
    // subspace tiles t .. t + N - 1 side by side
    auto subspace = [&](auto tiles, int t) __attribute__((always_inline)) {
        constexpr int N = decltype(tiles)::value;
        floatx4 acc[N];
        const float* av[N];
        const float* bv[N];
        int ti[N], tj[N];
#pragma unroll
        for (int u = 0; u < N; ++u) {
            ti[u] = (t + u) / mt;
            tj[u] = (t + u) - ti[u] * mt;
            bv[u] = a.dirs_a + ((int64_t)ti[u] * m + 16 * tj[u]) * dp;
            av[u] = ql + ti[u] * dp;
            acc[u] = floatx4{0.f, 0.f, 0.f, 0.f};
        }
        chains(tiles, av, bv, dp, acc);
        wait_norms();
#pragma unroll
        for (int u = 0; u < N; ++u) store(acc[u], 1 + ti[u], tj[u]);
    };
    // (the last one to three tiles as they are: a slot that repeats a tile
    // costs its loads and MFMAs, three quarters of all at L = 1)
    int t = s0;
    for (; t + 4 <= s1; t += 4) subspace(std::integral_constant<int, 4>(), t);
    if (s1 - t >= 2) {
        subspace(std::integral_constant<int, 2>(), t);
        t += 2;
    }
    if (t < s1) subspace(std::integral_constant<int, 1>(), t);
    wait_norms();
}

// the bodies as kernels of their own (each with its own registers)
enum TableBody { kTable16, kTableWide, kTableMany, kTableGeneral };

template <int BODY>
__global__ __launch_bounds__((BODY == kTableWide ? kWideWaves : kTableWaves) * 64,
                             BODY == kTableWide ? 4 : 1) void k_query_table(QueryTableArgs a)
{
#pragma clang fp contract(off)
    extern __shared__ __align__(16) float qs[];  // 16 x (d + 4)
    __shared__ float inv_norm[16];
    const int tid = threadIdx.x;
    const int lane = lane_id();
    const int wv = wave_uniform(tid >> 6);  // (so that branches on it stay scalar)
    const int64_t q0 = (int64_t)blockIdx.x * 16;
    const int d = a.d, L = a.L, m = a.m;
    const int dp = d / L;
    const int ld = d + 4;
    const int nrows = (int)(a.nq - q0 < 16 ? a.nq - q0 : 16);

    // stage the tile in the original coordinate order (the norm is taken in
    // that order; a dimension permutation of the test is applied when the
    // operands are read).  Past 16 (d + 4) floats of LDS the rows are read
    // from global memory instead.
    const int nch = d >> 2;
    if constexpr (BODY == kTableWide) {
        // two rows a wave, their loads in flight together
        static_assert(2 * kWideWaves == 16, "two rows a wave");
        const int r0 = wv < nrows ? wv : 0, r1 = wv + kWideWaves < nrows ? wv + kWideWaves : 0;
        const float4* p0 = reinterpret_cast<const float4*>(a.queries + (q0 + r0) * (int64_t)d);
        const float4* p1 = reinterpret_cast<const float4*>(a.queries + (q0 + r1) * (int64_t)d);
        const bool in0 = wv < nrows, in1 = wv + kWideWaves < nrows;
        auto put = [](float4* w, float4 v, bool in) {
            *w = make_float4(in ? v.x : 0.f, in ? v.y : 0.f, in ? v.z : 0.f, in ? v.w : 0.f);
        };
        float4* w0 = reinterpret_cast<float4*>(qs + wv * ld);
        float4* w1 = reinterpret_cast<float4*>(qs + (wv + kWideWaves) * ld);
        for (int k = lane; k < nch; k += 2 * kWave) {
            const int k2 = k + kWave < nch ? k + kWave : k;
            const float4 v0 = p0[k], v1 = p1[k], v2 = p0[k2], v3 = p1[k2];
            put(w0 + k, v0, in0);
            put(w1 + k, v1, in1);
            put(w0 + k2, v2, in0);
            put(w1 + k2, v3, in1);
        }
    } else if (a.staged) {
        for (int c = tid; c < 16 * nch; c += kTableWaves * 64) {
            const int r = c / nch, k4 = (c - r * nch) * 4;
            float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
            if (r < nrows)
                v = *reinterpret_cast<const float4*>(a.queries + (q0 + r) * (int64_t)d + k4);
            *reinterpret_cast<float4*>(qs + r * ld + k4) = v;
        }
    }
    __syncthreads();
    if constexpr (BODY == kTable16) {
        query_table16(a, qs, nrows, q0, wv, lane);
        return;
    }
    if constexpr (BODY == kTableWide) {
        if (m < 64 && d >= 512) query_table_wide<true>(a, qs, inv_norm, nrows, q0, wv, lane);
        else query_table_wide<false>(a, qs, inv_norm, nrows, q0, wv, lane);
        return;
    }

    const int row = lane & 15;
    const int kq = lane >> 4;
    const bool rv = row < nrows;
    // this lane's row: in LDS, or in global memory (rows past the batch read
    // row 0 and contribute zeros)
    const bool staged = BODY == kTableMany || a.staged;
    const float* qglobal = a.queries + (q0 + (rv ? row : 0)) * (int64_t)d;
    if (wv == 0) {
        // |q| in the order of staged_row_norm, from LDS or global memory
        float nrm;
        if (staged) {
            nrm = staged_row_norm(qs + row * ld, d, kq);
        } else {
            float ss = 0.f;
            for (int k = kq; k < d; k += 4) {
                const float v = rv ? qglobal[k] : 0.f;
                ss = fmaf(v, v, ss);
            }
            ss += __shfl_xor(ss, 16, kWave);
            ss += __shfl_xor(ss, 32, kWave);
            nrm = sqrtf(ss);
        }
        if (kq == 0) {
            inv_norm[row] = (nrm > 0.f && nrm < INFINITY) ? 1.f / nrm : 0.f;
            if (row < nrows) a.qnorms[q0 + row] = nrm;
        }
    }
    __syncthreads();

    const int col = lane & 15;
    const int kb = lane >> 4;
    const int ntile = (L + 1) * (m >> 4);

    for (int t = wv; t < ntile; t += kTableWaves) {
        const int i = t / (m >> 4);
        const int jdir = (t - i * (m >> 4)) * 16 + col;
        const int k_begin = (i == 0) ? 0 : (i - 1) * dp;
        const int k_len = (i == 0) ? d : dp;
        const float* bv = (i == 0) ? a.dirs_b + (int64_t)jdir * d
                                   : a.dirs_a + ((int64_t)(i - 1) * m + jdir) * dp;
        floatx4 acc = {0.f, 0.f, 0.f, 0.f};
        int k0 = 0;
        if constexpr (BODY == kTableMany) {
            // staged rows, no permutation, m > 16 and blocks enough to fill the
            // chip: the wide form's order of K, four groups a round trip
            const float* ql = qs + row * ld + k_begin;
            const int ng = k_len >> 4;
            int j = 0;
            for (; j + 4 <= ng; j += 4) acc = mfma_groups<4>(acc, ql, bv, j, 4 * kq);
            switch (ng - j) {
            case 3: acc = mfma_groups<3>(acc, ql, bv, j, 4 * kq); break;
            case 2: acc = mfma_groups<2>(acc, ql, bv, j, 4 * kq); break;
            case 1: acc = mfma_groups<1>(acc, ql, bv, j, 4 * kq); break;
            default: break;
            }
            for (k0 = 16 * ng; k0 < k_len; k0 += 4)
                acc = __builtin_amdgcn_mfma_f32_16x16x4f32(ql[k0 + kq], bv[k0 + kb], acc, 0, 0, 0);
        } else {
            // N steps from k: every load of a kind before the next kind's, as
            // straight-line code (coordinate k_begin + k of the permuted row;
            // rows past the batch in global memory are dropped after the load).
            // What bounds this body is the latency of these loads: with a
            // branch around each it took 81 us for 17 queries at d = 1,024,
            // m = 16 (now 66) and 53 for 2,049 permuted ones at d = 960 (31)
            auto steps = [&](auto count, int k) {
                constexpr int N = decltype(count)::value;
                int kk[N];
                float bb[N], aa[N];
#pragma unroll
                for (int u = 0; u < N; ++u) bb[u] = bv[k + 4 * u + kb];
#pragma unroll
                for (int u = 0; u < N; ++u) kk[u] = k_begin + k + 4 * u + kq;
                if (a.perm) {
#pragma unroll
                    for (int u = 0; u < N; ++u) kk[u] = a.perm[kk[u]];
                }
                if (staged) {
                    const float* ql = qs + row * ld;  // (an LDS pointer, so LDS reads)
#pragma unroll
                    for (int u = 0; u < N; ++u) aa[u] = ql[kk[u]];
                } else {
#pragma unroll
                    for (int u = 0; u < N; ++u) aa[u] = qglobal[kk[u]];
#pragma unroll
                    for (int u = 0; u < N; ++u) aa[u] = rv ? aa[u] : 0.f;
                }
#pragma unroll
                for (int u = 0; u < N; ++u) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(aa[u], bb[u], acc, 0, 0, 0);
            };
            for (; k0 + 32 <= k_len; k0 += 32) steps(std::integral_constant<int, 8>(), k0);
            for (; k0 < k_len; k0 += 4) steps(std::integral_constant<int, 1>(), k0);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int orow = 4 * (lane >> 4) + r;
            if (orow < nrows) {
                const float tv = acc[r] * inv_norm[orow];
                const int64_t o = ((q0 + orow) * (L + 1) + i) * m + jdir;
                if (a.half_out) reinterpret_cast<_Float16*>(a.tables)[o] = (_Float16)tv;
                else a.tables[o] = tv;
            }
        }
    }
}

}  // namespace peos
