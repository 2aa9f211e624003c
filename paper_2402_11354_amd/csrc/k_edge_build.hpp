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
    int unit_nodes;       // nodes per wave: max(1, 64 / R)
};

constexpr int kCompactZeroEdge = 255;
// coordinates of the 16 edges' vectors held in LDS at a time (a multiple of
// 64, so that every coordinate keeps its place mod 16): 17 KB a wave at 256,
// eight waves a CU for long vectors; up to 256 coordinates are gathered once
constexpr int kSegment = 256;
constexpr int kChunkWords = 4 * 64 + 16;  // LDS words of 16 coordinates: four steps of 64
                                          // lanes, padded so that lanes four steps apart
                                          // (the block norms) use different banks
constexpr int kCodeRow = 36;              // code bytes of one edge, at most

inline size_t edge_build_lds(int d, int L)
{
    const int seg = d < kSegment ? (d + 15) / 16 * 16 : kSegment;
    return sizeof(float) * ((size_t)(seg / 16) * kChunkWords + 16 * (size_t)L + 5 * 64) + 16 * kCodeRow;
}

// 4 x 4 transpose between the four groups of 16 lanes and four registers:
// afterwards register c of group g holds what register g of group c held
__device__ __forceinline__ void transpose4(float (&x)[4])
{
    auto swap32 = [](float& a, float& b) {
        const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
        a = __uint_as_float(r[0]);
        b = __uint_as_float(r[1]);
    };
    auto swap16 = [](float& a, float& b) {
        const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
        a = __uint_as_float(r[0]);
        b = __uint_as_float(r[1]);
    };
    swap32(x[0], x[2]);
    swap32(x[1], x[3]);
    swap16(x[0], x[1]);
    swap16(x[2], x[3]);
}

// LDS word of step t (coordinates 4t .. 4t + 3 of the segment)
__device__ __forceinline__ int step_word(int t) { return (t >> 2) * kChunkWords + (t & 3) * 64; }

// The code of each edge (lane % 16) from its m products: the first largest
// |p|, plus m if that p is negative.  acc[t][r] is direction 16 t + 4 g + r.
template <int MT>
__device__ __forceinline__ int extreme_code(const floatx4 (&acc)[MT], int mt, int m, int g)
{
    float best = -1.f;
    int code = 0;  // direction, plus 256 if its product is negative
#pragma unroll
    for (int t = 0; t < MT; ++t) {
        if (t >= mt) break;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float p = acc[t][r];
            const bool up = fabsf(p) > best;
            best = up ? fabsf(p) : best;
            code = up ? 16 * t + 4 * g + r + (p < 0.f ? 256 : 0) : code;
        }
    }
    auto fold = [&](float b0, int c0, float b1, int c1) {
        const bool second = (b1 > b0) | ((b1 == b0) & ((c1 & 255) < (c0 & 255)));
        best = second ? b1 : b0;
        code = second ? c1 : c0;
    };
    {
        const auto b = __builtin_amdgcn_permlane16_swap(__float_as_uint(best), __float_as_uint(best), false, false);
        const auto c = __builtin_amdgcn_permlane16_swap((uint32_t)code, (uint32_t)code, false, false);
        fold(__uint_as_float(b[0]), (int)c[0], __uint_as_float(b[1]), (int)c[1]);
    }
    {
        const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(best), __float_as_uint(best), false, false);
        const auto c = __builtin_amdgcn_permlane32_swap((uint32_t)code, (uint32_t)code, false, false);
        fold(__uint_as_float(b[0]), (int)c[0], __uint_as_float(b[1]), (int)c[1]);
    }
    return (code & 255) + (code >= 256 ? m : 0);
}

// MT: 16-direction tiles, at least m / 16 (exactly, up to 2).  FULL: blocks are
// whole groups of four steps (d / L a multiple of 16), so no chunk of a block
// or a vector is partly filled.  PERM: with a dimension permutation.
template <int MT, bool COMPACT, bool SIM, bool FULL, bool PERM>
__global__ __launch_bounds__(64) void k_edge_build(EdgeBuildArgs a)
{
#pragma clang fp contract(off)
    extern __shared__ __align__(16) float smem[];
    const int d = a.d, R = a.R, L = a.L, m = a.m;
    const int dp = d / L;
    const int mt = MT <= 2 ? MT : m >> 4;
    const int seg = d < kSegment ? (d + 15) / 16 * 16 : kSegment;
    float* et = smem;                                // the tile's edge vectors, in step order
    float* sb = et + (seg / 16) * kChunkWords;       // 16 x L block norms (compact: squared)
    int32_t* row = reinterpret_cast<int32_t*>(sb + 16 * L);  // the unit's neighbour ids
    float* nvs = reinterpret_cast<float*>(row + 64);         // |v|^2 per node of the unit
    float* cgp = nvs + 64;                           // compact: scalars and kind per edge
    float* cie = cgp + 64;
    int32_t* ckd = reinterpret_cast<int32_t*>(cie + 64);
    uint8_t* cb = reinterpret_cast<uint8_t*>(ckd + 64);
    const int lane = lane_id();
    const int g = lane >> 4;    // lane group: K offset within an MFMA step
    const int ec = lane & 15;   // edge of the tile (and direction row of the other operand)

    const int64_t v0 = (int64_t)blockIdx.x * a.unit_nodes;
    const int nn = (int)(a.n - v0 < a.unit_nodes ? a.n - v0 : a.unit_nodes);
    const int E = nn * R;
    if (lane < E) row[lane] = a.graph[v0 * R + lane];
    wave_sync();
    // graph validation: id range, self loop, repeated id in the row
    if (lane < E) {
        const int b = lane / R;
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
    // four steps (coordinates k .. k + 15) of a direction tile, in step order
    // (zeros from kend on)
    auto dirs4 = [&](const float* p, int k, int kend, float (&x)[4]) {
        const bool in = FULL || k + 4 * g < kend;
        const float4 v = *reinterpret_cast<const float4*>(p + (in ? k + 4 * g : 0));
        x[0] = in ? v.x : 0.f;
        x[1] = in ? v.y : 0.f;
        x[2] = in ? v.z : 0.f;
        x[3] = in ? v.w : 0.f;
        transpose4(x);
    };

    const int ntile = (E + 15) >> 4;
    for (int T = 0; T < ntile; ++T) {
        const int f = 16 * T + ec;
        int32_t u = f < E ? row[f] : -1;
        if (u >= a.n) u = -1;  // never dereferenced (reported through err)
        const bool ok = u >= 0;
        const int b = f < E ? f / R : 0;
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
            for (int i = i0; i <= i1; ++i) {
                const int kb = i * dp > k0 ? i * dp : k0;
                const int ke = (i + 1) * dp < k0 + len ? (i + 1) * dp : k0 + len;
                if (kb == i * dp) {
#pragma unroll
                    for (int t = 0; t < MT; ++t) acc[t] = floatx4{0.f, 0.f, 0.f, 0.f};
                }
                const float* av = a.dirs_a + ((int64_t)i * m + ec) * dp;
                for (int k = kb; k < ke; k += 16) {
                    const int ns = !FULL && ke - k < 16 ? (ke - k) >> 2 : 4;
                    float e[4];
#pragma unroll
                    for (int c = 0; c < 4; ++c) e[c] = c < ns ? et[step_word(((k - k0) >> 2) + c) + lane] : 0.f;
#pragma unroll
                    for (int t = 0; t < MT; ++t) {
                        if (t >= mt) break;
                        float x[4];
                        dirs4(av + (int64_t)t * 16 * dp, k - i * dp, dp, x);
#pragma unroll
                        for (int c = 0; c < 4; ++c)
                            if (c < ns) acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[c], e[c], acc[t], 0, 0, 0);
                    }
                }
                if (ke == (i + 1) * dp) {
                    const int code = extreme_code<MT>(acc, mt, m, g);
                    if (g == 0) cb[ec * kCodeRow + cfirst + i] = ok ? (uint8_t)code : 0;
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
                        dirs4(a.sdirs + (int64_t)(16 * t + ec) * d, k0 + k, d, x);
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
                cgp[f] = gp;
                cie[f] = ie;
                ckd[f] = kd;
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
                        const float s = sb[ec * L + blk];
                        ratio = s > 0.f ? c / s : 0.f;
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
                    dirs4(a.dirs_b + (int64_t)(16 * t + ec) * d, k0 + k, d, x);
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        if (q < ns) acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[q], e[q], acc[t], 0, 0, 0);
                }
            }
        }
        const int rcode = extreme_code<MT>(acc, mt, m, g);
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
        const float nu2 = (nu[0] + nu[2]) + (nu[1] + nu[3]);
        // scalars: g_e, |e|, w_reg, sqrt(L) w_res; in the precision form
        // the halves of g_e/|e|, 1/|e| (infinite for a zero edge), w_reg,
        // sqrt(L) w_res
        if (g == 0 && f < E) {
            float ge = 0.f, en = 0.f, wreg = 0.f, swres = 0.f;
            if (ok) {
                en = sqrtf(ne2);
                if (en > 0.f) {
                    wreg = fminf(1.f, c * sqrtf((float)nz) / en);
                    swres = sqrtf((float)L) * fminf(1.f, sqrtf(nr2) / en);
                } else {
                    wreg = 1.f;
                    swres = 0.f;
                }
                if (a.metric == 0) ge = 0.5f * (nu2 - nvs[b]);
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
        }
        // the codes, a dword per lane
        wave_sync();
        const int cwords = cbytes >> 2;
        for (int w = lane; w < 16 * cwords; w += kWave) {
            const int e = w / cwords, o = w - e * cwords;
            const int fe = 16 * T + e;
            if (fe >= E) break;
            const int be = fe / R;
            *reinterpret_cast<uint32_t*>(a.rec + (v0 + be) * a.node_stride + a.codes_off +
                                         (int64_t)(fe - be * R) * cbytes + 4 * o) =
                *reinterpret_cast<const uint32_t*>(cb + e * kCodeRow + 4 * o);
        }
    }
    if (!COMPACT) return;
    // compact: node ranges (min / max are exact in any order) and the codes
    wave_sync();
    if (lane >= E) return;
    const int b = lane / R;
    float glo = INFINITY, ghi = -INFINITY, ilo = INFINITY, ihi = -INFINITY;
    for (int j = b * R; j < (b + 1) * R; ++j) {
        if (ckd[j] != 1) continue;
        glo = fminf(glo, cgp[j]);
        ghi = fmaxf(ghi, cgp[j]);
        ilo = fminf(ilo, cie[j]);
        ihi = fmaxf(ihi, cie[j]);
    }
    if (!(glo <= ghi)) glo = ghi = ilo = ihi = 0.f;  // no edge of nonzero length
    const float gstep = (ghi - glo) / 255.f;
    const float istep = (ihi - ilo) / 254.f;
    uint8_t* rv = a.rec + (v0 + b) * a.node_stride;
    if (lane == b * R) *reinterpret_cast<float4*>(rv) = make_float4(glo, gstep, ilo, istep);
    uint32_t cg = 0u, ci = 0u;
    if (ckd[lane] == 2) ci = kCompactZeroEdge;
    if (ckd[lane] == 1) {
        if (gstep > 0.f) {
            const float c = floorf((cgp[lane] - glo) / gstep);
            cg = (uint32_t)(c < 0.f ? 0.f : (c > 255.f ? 255.f : c));
        }
        if (istep > 0.f) {
            const float c = rintf((cie[lane] - ilo) / istep);
            ci = (uint32_t)(c < 0.f ? 0.f : (c > 254.f ? 254.f : c));
        }
    }
    reinterpret_cast<uint16_t*>(rv + a.scal_off)[lane - b * R] = (uint16_t)(cg | (ci << 8));
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
