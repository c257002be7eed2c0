// Training of the optical-depth paths' networks on the GPU: the inverse CDF of the
// emitted energy (target 0) and of the pair's energy split (target 1, the
// half-distribution of |d - 1/2|), same network shape and kernels.
//
//   k_cdf_table    the normalised CDF of the emitted energy, eq. (1) integrated over
//                  the candidate x (or of the split, eq. (2) integrated over d), on a
//                  grid of chi (double, from the double fits of the synchrotron
//                  functions);
//   k_cdf_index    the part of the table that every inversion reads, compactly;
//   k_mlp_data     training samples (chi, u) -> x = CDF_chi^{-1}(u) from the table;
//   k_train_pack   float parameters -> the matrix operands of k_mlp_train;
//   k_mlp_train    forward and backward passes on the matrix cores, gradients
//                  reduced per block;
//   k_mlp_reduce   sum of the block gradients and the Adam update (or only the sum,
//                  for gradient checks), and the next step's samples;
//   k_mlp_pack     float parameters -> the fragment layout the generator stages;
//   k_mlp_validate per chi bin, the largest CDF error |CDF_chi(x(chi, u)) - u| of
//                  the packed network over a grid of u;
//   k_mlp_infer    the packed network on given (chi, u) pairs.
#include "qed_device.hpp"
#include "qed_internal.hpp"
#include "qed_mlp.hpp"
#include "qed_synchro.hpp"

namespace qed {

namespace {

constexpr int kBlock = 256;

// Grid of the CDF table: x = 1 - (1 - xi)^2 with xi uniform, so points crowd
// towards x = 1, where the spectrum of large chi has its structure (1 - x ~ 1/b).
__device__ __forceinline__ double cdf_x_of_xi(double xi) { return 1.0 - (1.0 - xi) * (1.0 - xi); }
__device__ __forceinline__ double cdf_xi_of_x(double x) { return 1.0 - sqrt(fmax(1.0 - x, 0.0)); }

// ((1 - x^3) F(z) + x^6 G(z)) / x with z = x^3 / (b (1 - x^3)): eq. (1) over c b.
// x = 0 gives the limit 2^(2/3) Gamma(2/3) b^(-1/3).
__device__ __forceinline__ double emission_density(double x, double b, const SynTable<double> &tab) {
    if (x <= 0.0) return 2.1495282415344787 * cbrt(1.0 / b);
    const double x3 = x * x * x;
    const double omx3 = (1.0 - x) * (1.0 + x + x * x);
    if (omx3 <= 0.0) return 0.0;
    double F, G;
    syn_eval(x3 / (b * omx3), tab, F, G);
    return (omx3 * F + x3 * x3 * G) / x;
}

// Energy split of pair creation: the Baier-Katkov density (3/2) chi (G(z) - d(1-d) F(z)),
// z = 2/(3 chi d (1-d)), of the electron's fraction d (eq. (2) over its prefactor).
__device__ __forceinline__ double pair_density(double d, double chi, const SynTable<double> &tab) {
    const double dd = d * (1.0 - d);
    if (dd <= 0.0) return 0.0;
    double F, G;
    syn_eval(2.0 / (3.0 * chi * dd), tab, F, G);
    return 1.5 * chi * (G - dd * F);
}

// Density of the table's variable per unit of xi = k / nx at xi (kind 0: x(xi) with
// the grid's Jacobian; kind 1: D = xi / 2 of the half-distribution, d = 1/2 + D).
__device__ __forceinline__ double table_density(int kind, double xi, double l10, const SynTable<double> &tab) {
    if (kind == 0) return emission_density(cdf_x_of_xi(xi), 1.5 * exp10(l10), tab) * 2.0 * (1.0 - xi);
    return 0.5 * pair_density(0.5 + 0.5 * xi, exp10(l10), tab);
}

__global__ __launch_bounds__(kBlock) void k_cdf_table(CdfTableDev t) {
    __shared__ SynTable<double> tab;
    __shared__ double wsum[kBlock / 64];
    syn_stage(tab);
    __syncthreads();
    const int c = blockIdx.x;
    const double l10 = t.lo10 + (t.hi10 - t.lo10) * (double)c / (double)(t.nchi - 1);
    const int per = t.nx / kBlock;  // intervals per thread
    const double h = 1.0 / (double)t.nx;
    const int k0 = threadIdx.x * per;
    double part = 0.0;
    double dprev = table_density(t.kind, k0 * h, l10, tab);
    for (int k = k0; k < k0 + per; ++k) {
        const double xi = (k + 1) * h;
        const double d = table_density(t.kind, xi, l10, tab);
        part += 0.5 * h * (dprev + d);
        dprev = d;
    }
    // block exclusive prefix of the thread sums
    double incl = part;
    const int lane = __lane_id(), wv = threadIdx.x / 64;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const double v = __shfl_up(incl, o);
        if (lane >= o) incl += v;
    }
    if (lane == 63) wsum[wv] = incl;
    __syncthreads();
    double off = incl - part, total = 0.0;
    for (int w = 0; w < kBlock / 64; ++w) {
        if (w < wv) off += wsum[w];
        total += wsum[w];
    }
    double *row = t.cdf + (u64)c * (t.nx + 1);
    if (threadIdx.x == 0) {
        row[0] = 0.0;
        t.total[c] = total;
    }
    // second pass: the running sum (same order of additions as above)
    double acc = off;
    dprev = table_density(t.kind, k0 * h, l10, tab);
    for (int k = k0; k < k0 + per; ++k) {
        const double xi = (k + 1) * h;
        const double d = table_density(t.kind, xi, l10, tab);
        acc += 0.5 * h * (dprev + d);
        dprev = d;
        row[k + 1] = k + 1 == t.nx ? 1.0 : fmin(acc / total, 1.0);
    }
}

// Table CDF at (log10 chi, x), linear in xi and in log10 chi between nodes (x: the
// candidate for kind 0, the distance D from 1/2 for kind 1).
__device__ __forceinline__ double cdf_lookup(const CdfTableDev &t, double l10, double x) {
    const double cpos = (l10 - t.lo10) / (t.hi10 - t.lo10) * (double)(t.nchi - 1);
    const int j = min(max((int)floor(cpos), 0), t.nchi - 2);
    const double w = fmin(fmax(cpos - j, 0.0), 1.0);
    const double xi = (t.kind == 0 ? cdf_xi_of_x(fmin(fmax(x, 0.0), 1.0)) : fmin(fmax(2.0 * x, 0.0), 1.0)) *
                      (double)t.nx;
    const int k = min((int)xi, t.nx - 1);
    const double f = xi - k;
    const double *r0 = t.cdf + (u64)j * (t.nx + 1), *r1 = r0 + (t.nx + 1);
    const double c0 = r0[k] + f * (r0[k + 1] - r0[k]);
    const double c1 = r1[k] + f * (r1[k + 1] - r1[k]);
    return c0 + w * (c1 - c0);
}

// The index of a row: the values that the first eight levels of a bisection of the row
// read, in the order of the bisection's tree, four levels (15 values, the slots 1..15)
// to a line of 128 bytes: line 0, then one of the lines 1..16.
__global__ __launch_bounds__(kBlock) void k_cdf_index(CdfTableDev t) {
    for (int e = threadIdx.x; e < kCdfIndex; e += kBlock) {
        const int line = e / 16, slot = e % 16;
        if (slot == 0) continue;
        // the branches taken to the node, below a leading 1
        const int depth = 31 - __clz(slot);
        const int node = line == 0 ? slot : ((16 + line - 1) << depth) | (slot - (1 << depth));
        int lo = 0, hi = t.nx;
        for (int bit = 30 - __clz(node); bit >= 0; --bit) {
            const int mid = (lo + hi) >> 1;
            ((node >> bit) & 1 ? lo : hi) = mid;
        }
        t.index[(u64)blockIdx.x * kCdfIndex + e] = t.cdf[(u64)blockIdx.x * (t.nx + 1) + ((lo + hi) >> 1)];
    }
}

// Inverse of cdf_lookup at (log10 chi, u): x and the density dCDF/dx there.  A bisection:
// its first eight levels read the index (rows have at least 256 intervals), the others the
// rows.  Bound by the lines it reads: of the default table of 8,192 intervals, 2 + 2 from
// either row instead of 10, and the index (2.2 MB) stays in the L2 while the table (67 MB)
// does not: 65,536 samples 16.3 to 11.3 us.  (Reading both
// values that may follow along with each changes nothing: 11.5 us.)
__device__ __forceinline__ void cdf_invert(const CdfTableDev &t, double l10, double u, double &x,
                                           double &dens) {
    const double cpos = (l10 - t.lo10) / (t.hi10 - t.lo10) * (double)(t.nchi - 1);
    const int j = min(max((int)floor(cpos), 0), t.nchi - 2);
    const double w = fmin(fmax(cpos - j, 0.0), 1.0);
    int lo = 0, hi = t.nx;           // invariant: M(lo) <= u < M(hi)
    double m0 = 0.0, m1 = 1.0;       // M(lo), M(hi); every row runs from 0 to 1
    auto halve = [&](double a, double b) {
        const double m = a + w * (b - a);
        const int mid = (lo + hi) >> 1;
        const bool right = m <= u;
        (right ? lo : hi) = mid;
        (right ? m0 : m1) = m;
        return right;
    };
    const double *x0 = t.index + (u64)j * kCdfIndex, *x1 = x0 + kCdfIndex;
#pragma unroll
    for (int half = 0; half < 2; ++half) {
        uint32_t node = 1;
#pragma unroll
        for (int level = 0; level < 4; ++level) node = 2u * node + (halve(x0[node], x1[node]) ? 1u : 0u);
        x0 += 16u * (node - 15u);   // node is 16..31: the line below that leaf
        x1 += 16u * (node - 15u);
    }
    const double *r0 = t.cdf + (u64)j * (t.nx + 1), *r1 = r0 + (t.nx + 1);
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        halve(r0[mid], r1[mid]);
    }
    const double dm = m1 - m0;
    const double f = dm > 0.0 ? (u - m0) / dm : 0.5;
    const double xi = ((double)lo + f) / (double)t.nx;
    if (t.kind == 0) {
        x = cdf_x_of_xi(xi);
        dens = dm * (double)t.nx / fmax(2.0 * (1.0 - xi), 1e-300);
    } else {
        x = 0.5 * xi;
        dens = dm * (double)t.nx * 2.0;
    }
}

// Largest network input v: u = 1 - 2^-24, the largest float uniform, gives 1.55
// (emission) and 3.08 (pairs, v = sqrt(-ln(1 - u')) - 1).
constexpr double kVmax = 1.6;
constexpr double kVmaxPair = 3.1;

__device__ __forceinline__ void draw_samples(const DataArgs &da) {
    const CdfTableDev &t = da.t;
    const double lo10 = da.lo10, hi10 = da.hi10;
    const uint32_t klo = (uint32_t)da.seed ^ 0x7F4A7C15u, khi = (uint32_t)(da.seed >> 32) ^ 0xF39CC060u;
    for (u64 i = (u64)blockIdx.x * kBlock + threadIdx.x; i < da.n; i += (u64)da.blocks * kBlock) {
        const u32x4 w = philox10((uint32_t)i, (uint32_t)(i >> 32), da.step, 0u, klo, khi);
        const double tl = u53(w.x, w.y);  // position in the chi range
        // the network input v = (-ln(1 - u))^(1/3) - 1 is drawn uniformly on
        // [-1, kVmax] (u = 1 - exp(-(v + 1)^3)), so the tails of the spectrum are
        // sampled as densely as its bulk
        const double vmax = t.kind == 0 ? kVmax : kVmaxPair;
        const double v = -1.0 + (vmax + 1.0) * u53(w.z, w.w);
        const double u = t.kind == 0 ? -expm1(-(v + 1.0) * (v + 1.0) * (v + 1.0)) : -expm1(-(v + 1.0) * (v + 1.0));
        const double l10 = lo10 + (hi10 - lo10) * tl;
        double x, dens;
        cdf_invert(t, l10, u, x, dens);
        // output scale: (b / (1 + b))^(1/3) of x (emission), the split's width (pairs)
        const double xs = t.kind == 0 ? cbrt(1.5 * exp10(l10) / (1.0 + 1.5 * exp10(l10)))
                                      : (double)pair_width((float)exp10(l10));
        Sample s;
        s.s = (float)(2.0 * tl - 1.0);
        s.v = (float)v;
        s.y = (float)(x / xs);
        // weight: squared density in units of the network output, so the loss
        // approximates the squared CDF error (capped to keep the scale moderate,
        // with a small floor for the far tail)
        const double dy = fmin(dens * xs, 5.0);
        s.w = (float)(dy * dy + 1e-4);
        da.out[i] = s;
    }
}

__global__ __launch_bounds__(kBlock) void k_mlp_data(DataArgs da) { draw_samples(da); }

// ---------------------------------------------------------------------------
// Training step.
// ---------------------------------------------------------------------------
// Two waves share a tile of 16 samples, wave n the hidden units 32 n .. 32 n + 31 of
// every layer, and a block has four such groups, each with its own tiles.
constexpr int kTrainGroups = 4;
constexpr int kTrainBlock = kTrainGroups * 128;

// The waves of a group hand each other their units' values here: activations of layers
// 1 and 2 split into high parts and residuals (A operand: row = sample) and, for
// the weight gradients, the high parts with the samples of a unit side by side (B
// operand); the third layer's activations; the gradients dz of layers 3 and 2.  Every
// array has its own space, so a tile takes five barriers and no array is written
// before the barrier after its last reader.
struct alignas(16) TrainTile {
    uint16_t h[2][16][72], l[2][16][72], z[2][16][72];
    uint16_t ht[2][kHid][20];
    float h3[16][68];
    alignas(16) Sample sample[2][16];   // of this tile and the next
};

// The weights as B operands, 16 bytes per lane: tf[layer][n][kk][lane] holds
// W[16 n + r][32 kk + kidx(g, j)] (high parts; tl the residuals), and wt the transposed
// weights W[32 kk + kidx(g, j)][16 n + r] for dZ W.  k_mlp_reduce keeps it current.
struct TrainWeights {
    uint4 tf[2][4][2][64], tl[2][4][2][64], wt[2][4][2][64];
};
static_assert(sizeof(TrainWeights) == kTrainWeightBytes, "the buffer the host allocates");

// Weight p, value v, into its three places.
__device__ __forceinline__ void pack_weight(TrainWeights *t, int p, float v) {
    const int layer = p >= kOffW3, q = p - (layer ? kOffW3 : kOffW2);
    if (q < 0 || q >= kHid * kHid) return;
    const int o = q / kHid, i = q % kHid;
    uint16_t *tf = reinterpret_cast<uint16_t *>(&t->tf[layer][o >> 4][i >> 5][((i >> 3) & 3) * 16 + (o & 15)]);
    uint16_t *tl = reinterpret_cast<uint16_t *>(&t->tl[layer][o >> 4][i >> 5][((i >> 3) & 3) * 16 + (o & 15)]);
    uint16_t *wt = reinterpret_cast<uint16_t *>(&t->wt[layer][i >> 4][o >> 5][((o >> 3) & 3) * 16 + (i & 15)]);
    tf[i & 7] = bf_bits(v);
    tl[i & 7] = bf_bits(bf_res(v));
    wt[o & 7] = bf_bits(v);
}

__global__ __launch_bounds__(kBlock) void k_train_pack(const float *params, TrainWeights *t) {
    const int p = blockIdx.x * kBlock + threadIdx.x;
    if (p < kMlpParams) pack_weight(t, p, params[p]);
}

typedef short s16x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint2 pack4(const float *v) { return make_uint2(pack2(v[0], v[1]), pack2(v[2], v[3])); }

// Sum over the 16 lanes of a row, in every lane: the partners are lane ^ 1, ^ 2, ^ 4 and ^ 8
// (the mirrored lane holds what lane ^ 4 or ^ 8 does, as the lanes between are equal by then).
__device__ __forceinline__ float row_sum(float v) {
    auto add = [&](int other) { v += __builtin_bit_cast(float, other); };
    const auto bits = [&] { return __builtin_bit_cast(int, v); };
    add(__builtin_amdgcn_update_dpp(0, bits(), 0xB1, 0xF, 0xF, true));    // quad_perm 1 0 3 2
    add(__builtin_amdgcn_update_dpp(0, bits(), 0x4E, 0xF, 0xF, true));    // quad_perm 2 3 0 1
    add(__builtin_amdgcn_update_dpp(0, bits(), 0x141, 0xF, 0xF, true));   // row_half_mirror
    add(__builtin_amdgcn_update_dpp(0, bits(), 0x140, 0xF, 0xF, true));   // row_mirror
    return v;
}

// Forward and backward passes, a group's tiles one after the other.  Lane (r, g) of a wave
// holds the values of its units 32 n + r and 32 n + 16 + r for the samples 4 g .. 4 g + 3
// (the C layout of the matrix core).  Bound by latency and by the instructions of the
// activations: with one wave for all 64 units a SIMD held a single wave (340 registers),
// which issues at half the rate, and fetched every tile's samples only when it came to it:
// 65,536 samples took 31.2 us; two waves to a SIMD, with the forward weights in registers,
// the transposed ones in LDS (250 registers), take 19.7, 2.8 of them for each
// tile of 16 per wave pair.  Four waves (16 units each) leave no registers for
// weights, and reading these from the LDS in every tile then bounds: 21.4 us.  The
// operations on a value and their order are those of a wave that has all units.
__global__ __launch_bounds__(kTrainBlock) void k_mlp_train(TrainArgs ta) {
    constexpr int kRed = kMlpParams + 1;
    __shared__ union Lds {
        struct {
            TrainTile tile[kTrainGroups];
            float w4[kHid];
            uint4 wt[2][4][2][64];
        } t;
        float red[kTrainGroups][kRed];
    } L;
    const int lane = __lane_id(), r = lane & 15, g = lane >> 4;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), grp = wv >> 1, n = wv & 1;
    TrainTile &T = L.t.tile[grp];
    const float *P = ta.params;
    const TrainWeights &K = *reinterpret_cast<const TrainWeights *>(ta.weights);
    uint4 fh[2][2][2], fl[2][2][2];   // [layer][m][kk], m: the wave's first or second 16 units
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const int layer = k >> 2, m = (k >> 1) & 1, kk = k & 1;
        fh[layer][m][kk] = K.tf[layer][2 * n + m][kk][lane];
        fl[layer][m][kk] = K.tl[layer][2 * n + m][kk][lane];
    }
    const uint4 t0 = (&K.wt[0][0][0][0])[threadIdx.x], t1 = (&K.wt[0][0][0][0])[kTrainBlock + threadIdx.x];
    (&L.t.wt[0][0][0][0])[threadIdx.x] = t0;
    (&L.t.wt[0][0][0][0])[kTrainBlock + threadIdx.x] = t1;
    if (threadIdx.x < kHid) L.t.w4[threadIdx.x] = P[kOffW4 + threadIdx.x];   // a barrier follows in every tile
    const float b4 = P[kOffB4];
    float w10[2], w11[2], b1[2], b2[2], b3[2], w4[2];
    f32x4 gw2[2][4], gw3[2][4];
    float gw10[2], gw11[2], gb1[2], gb2[2], gb3[2], gw4[2], gb4 = 0.0f, loss = 0.0f;
#pragma unroll
    for (int m = 0; m < 2; ++m) {
        const int u = 32 * n + 16 * m + r;
        w10[m] = P[kOffW1 + 2 * u];
        w11[m] = P[kOffW1 + 2 * u + 1];
        b1[m] = P[kOffB1 + u];
        b2[m] = P[kOffB2 + u];
        b3[m] = P[kOffB3 + u];
        w4[m] = P[kOffW4 + u];
        gw10[m] = gw11[m] = gb1[m] = gb2[m] = gb3[m] = gw4[m] = 0.0f;
#pragma unroll
        for (int k = 0; k < 4; ++k) gw2[m][k] = gw3[m][k] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    }

    // this wave's units of layer k's activations, for the other wave
    auto share = [&](int k, const float (*v)[4]) {
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            const int u = 32 * n + 16 * m + r;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                T.h[k][4 * g + q][u] = bf_bits(v[m][q]);
                T.l[k][4 * g + q][u] = bf_bits(bf_res(v[m][q]));
            }
            *reinterpret_cast<uint2 *>(&T.ht[k][u][4 * g]) = pack4(v[m]);
        }
    };
    auto rows = [&](const uint16_t (*m)[72], int kk) {
        return as_bf8(*reinterpret_cast<const uint4 *>(&m[r][32 * kk + kidx(g, 0)]));
    };
    // [16 x 64] x [64 x 32] product of layer k's split activations with split weights:
    // hi*hi + hi*lo + lo*hi, small terms first
    auto forward = [&](int k, f32x4 *acc) {
        const bf16x8 h0 = rows(T.h[k], 0), h1 = rows(T.h[k], 1), l0 = rows(T.l[k], 0), l1 = rows(T.l[k], 1);
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            const bf16x8 p0 = as_bf8(fh[k][m][0]), p1 = as_bf8(fh[k][m][1]);
            f32x4 c = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
            c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(l0, p0, c, 0, 0, 0);
            c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(l1, p1, c, 0, 0, 0);
            c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(h0, as_bf8(fl[k][m][0]), c, 0, 0, 0);
            c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(h1, as_bf8(fl[k][m][1]), c, 0, 0, 0);
            c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(h0, p0, c, 0, 0, 0);
            acc[m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(h1, p1, c, 0, 0, 0);
        }
    };
    // dZ W of the dz in z[k] (0: layer 3, 1: layer 2)
    auto backward = [&](int k, f32x4 *acc) {
        const bf16x8 z0 = rows(T.z[k], 0), z1 = rows(T.z[k], 1);
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            f32x4 c = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
            c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(z0, as_bf8(L.t.wt[1 - k][2 * n + m][0][lane]), c, 0, 0, 0);
            acc[m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(z1, as_bf8(L.t.wt[1 - k][2 * n + m][1][lane]), c, 0, 0, 0);
        }
    };
    // dz for the other wave, and dW += dz^T h of layer k's activations (K = the 16 samples)
    auto weight_grad = [&](int z, const float (*dz)[4], int k, f32x4 (*acc)[4]) {
        s16x4 ad[2];
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            ad[m] = __builtin_bit_cast(s16x4, pack4(dz[m]));
#pragma unroll
            for (int q = 0; q < 4; ++q) T.z[z][4 * g + q][32 * n + 16 * m + r] = bf_bits(dz[m][q]);
        }
#pragma unroll
        for (int cj = 0; cj < 4; ++cj) {
            const s16x4 h = __builtin_bit_cast(s16x4, *reinterpret_cast<const uint2 *>(&T.ht[k][16 * cj + r][4 * g]));
#pragma unroll
            for (int m = 0; m < 2; ++m)
                acc[m][cj] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(ad[m], h, acc[m][cj], 0, 0, 0);
        }
    };

    const Sample *batch = ta.batch + ((u64)blockIdx.x * kTrainGroups + grp) * (u64)ta.tiles * 16;
    if (n == 0 && lane < 16) T.sample[0][lane] = batch[lane];
    __syncthreads();
    for (uint32_t tile = 0; tile < ta.tiles; ++tile) {
        const Sample *sm = &T.sample[tile & 1][4 * g];
        // the next tile's samples are under way while this one is worked on
        const bool fetch = n == 0 && lane < 16 && tile + 1 < ta.tiles;
        f32x4 next = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        if (fetch) next = *reinterpret_cast<const f32x4 *>(batch + 16ull * (tile + 1) + lane);
        float pre1[2][4], pre2[2][4], pre3[2][4], h[2][4];
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                pre1[m][q] = fmaf(w10[m], sm[q].s, fmaf(w11[m], sm[q].v, b1[m]));
                h[m][q] = mlp_act(pre1[m][q]);
            }
        share(0, h);
        __syncthreads();
        f32x4 acc[2];
        forward(0, acc);
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                pre2[m][q] = acc[m][q] + b2[m];
                h[m][q] = mlp_act(pre2[m][q]);
            }
        share(1, h);
        __syncthreads();
        forward(1, acc);
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                pre3[m][q] = acc[m][q] + b3[m];
                h[m][q] = mlp_act(pre3[m][q]);
                T.h3[4 * g + q][32 * n + 16 * m + r] = h[m][q];
            }
        __syncthreads();
        // the output, in both waves; loss and output gradient
        float dz[2][4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            float sacc = 0.0f;
#pragma unroll
            for (int k = 0; k < 4; ++k) sacc = fmaf(L.t.w4[16 * k + r], T.h3[4 * g + q][16 * k + r], sacc);
            const float y = row_sum(sacc);
            const float e = y + b4 - sm[q].y;
            const float wq = sm[q].w;
            const float dy = 2.0f * wq * e * ta.inv_batch;
            if (n == 0 && r == 0) {
                loss = fmaf(wq * e * e, ta.inv_batch, loss);
                gb4 += dy;
            }
#pragma unroll
            for (int m = 0; m < 2; ++m) {
                gw4[m] = fmaf(dy, h[m][q], gw4[m]);
                dz[m][q] = dy * w4[m] * mlp_dact(pre3[m][q]);
                gb3[m] += dz[m][q];
            }
        }
        weight_grad(0, dz, 1, gw3);
        __syncthreads();
        backward(0, acc);   // dh2 = dz3 W3
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                dz[m][q] = acc[m][q] * mlp_dact(pre2[m][q]);
                gb2[m] += dz[m][q];
            }
        if (fetch) *reinterpret_cast<f32x4 *>(&T.sample[(tile + 1) & 1][lane]) = next;
        weight_grad(1, dz, 0, gw2);
        __syncthreads();
        backward(1, acc);   // dh1 = dz2 W2
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float d1 = acc[m][q] * mlp_dact(pre1[m][q]);
                gw10[m] = fmaf(d1, sm[q].s, gw10[m]);
                gw11[m] = fmaf(d1, sm[q].v, gw11[m]);
                gb1[m] += d1;
            }
    }
    // per-unit sums over the four lane groups
#pragma unroll
    for (int o = 16; o < 64; o <<= 1)
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            gw10[m] += __shfl_xor(gw10[m], o);
            gw11[m] += __shfl_xor(gw11[m], o);
            gb1[m] += __shfl_xor(gb1[m], o);
            gb2[m] += __shfl_xor(gb2[m], o);
            gb3[m] += __shfl_xor(gb3[m], o);
            gw4[m] += __shfl_xor(gw4[m], o);
        }
    gb4 = wave_sum_f(gb4);
    loss = wave_sum_f(loss);
    // The block's sum: every group leaves its sums in the LDS (the tiles are done with),
    // and the threads add the four up in the order of the groups, so the float sums, and
    // with them a training run, are the same on every run.
    __syncthreads();
    float *red = L.red[grp];
#pragma unroll
    for (int m = 0; m < 2; ++m) {
        const int u = 32 * n + 16 * m;
        if (g == 0) {
            red[kOffW1 + 2 * (u + r)] = gw10[m];
            red[kOffW1 + 2 * (u + r) + 1] = gw11[m];
            red[kOffB1 + u + r] = gb1[m];
            red[kOffB2 + u + r] = gb2[m];
            red[kOffB3 + u + r] = gb3[m];
            red[kOffW4 + u + r] = gw4[m];
        }
#pragma unroll
        for (int cj = 0; cj < 4; ++cj)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int idx = (u + 4 * g + q) * kHid + 16 * cj + r;
                red[kOffW2 + idx] = gw2[m][cj][q];
                red[kOffW3 + idx] = gw3[m][cj][q];
            }
    }
    if (n == 0 && lane == 0) {
        red[kOffB4] = gb4;
        red[kMlpParams] = loss;
    }
    __syncthreads();
    float *dst = ta.partials + (u64)blockIdx.x * kRed;
    for (int i = threadIdx.x; i < kRed; i += kTrainBlock) {
        float sum = 0.0f;
#pragma unroll
        for (int k = 0; k < kTrainGroups; ++k) sum += L.red[k][i];
        dst[i] = sum;
    }
}

// Sum of the block gradients; then Adam (grad_out == nullptr) or a plain copy of
// the sum (gradient checks).  A block takes kRedParams parameters (the loss counts as
// one more): its 256 threads bring kRedRows blocks' partial sums into LDS, all loads in
// flight at once, and one thread per parameter adds them up in the order of the blocks,
// so the sum does not depend on the launch.  (One thread per parameter reading its 256
// partial sums from memory took 61.4 us a step at 256 blocks; this takes 6.0.)
//
// The first da.blocks blocks of the launch draw the samples of the next step, which do
// not depend on this one: both parts wait for memory rather than for each other,
// 13.3 us of a step instead of 11.3 + 6.7 and a launch between.
constexpr int kRedParams = 32, kRedRows = 256;

__global__ __launch_bounds__(kBlock) void k_mlp_reduce(ReduceArgs ra, DataArgs da) {
    if ((int)blockIdx.x < da.blocks) return draw_samples(da);
    __shared__ float part[kRedRows][kRedParams];
    const int p0 = ((int)blockIdx.x - da.blocks) * kRedParams;
    const int c = threadIdx.x % kRedParams, r0 = threadIdx.x / kRedParams;
    constexpr int kStep = kBlock / kRedParams, kLoads = kRedRows / kStep;
    const int p = p0 + c;
    const bool in = p <= kMlpParams;
    float gsum = 0.0f;
    for (int b0 = 0; b0 < ra.blocks; b0 += kRedRows) {
        const int rows = min(kRedRows, ra.blocks - b0);
        float v[kLoads];
#pragma unroll
        for (int k = 0; k < kLoads; ++k) {
            const int r = r0 + k * kStep;
            v[k] = in && r < rows ? ra.partials[(u64)(b0 + r) * (kMlpParams + 1) + p] : 0.0f;
        }
        __syncthreads();   // the previous rows have been added up
#pragma unroll
        for (int k = 0; k < kLoads; ++k) part[r0 + k * kStep][c] = v[k];
        __syncthreads();
        if (threadIdx.x < kRedParams) {
            if (rows == kRedRows) {
#pragma unroll 32
                for (int r = 0; r < kRedRows; ++r) gsum += part[r][c];
            } else {
                for (int r = 0; r < rows; ++r) gsum += part[r][c];
            }
        }
    }
    if (threadIdx.x >= kRedParams || !in) return;
    if (p == kMlpParams) {
        if (ra.loss_out) *ra.loss_out = gsum;
        return;
    }
    if (ra.grad_out) {
        ra.grad_out[p] = gsum;
        return;
    }
    const float m = ra.beta1 * ra.m[p] + (1.0f - ra.beta1) * gsum;
    const float v = ra.beta2 * ra.v[p] + (1.0f - ra.beta2) * gsum * gsum;
    ra.m[p] = m;
    ra.v[p] = v;
    const float next = ra.params[p] - ra.lr * (m * ra.c1) / (sqrtf(v * ra.c2) + ra.eps);
    ra.params[p] = next;
    pack_weight(reinterpret_cast<TrainWeights *>(ra.weights), p, next);
}

__global__ __launch_bounds__(kBlock) void k_mlp_pack(const float *params, MlpModel *out) {
    __shared__ MlpLds M;
    mlp_pack(params, M);
    __syncthreads();
    // weights only: lo, inv_span, nbins and the fallback flags are set by the host
    const uint4 *s = reinterpret_cast<const uint4 *>(&M);
    uint4 *d = reinterpret_cast<uint4 *>(out);
    constexpr int kHead = offsetof(MlpLds, b4) / 16;   // whole 16-byte words before b4
    for (int i = threadIdx.x; i < (int)(sizeof(MlpLds) / 16); i += kBlock) {
        if (i < kHead || (i >= (int)(offsetof(MlpLds, wf2) / 16) && i < (int)(offsetof(MlpLds, fallback) / 16)))
            d[i] = s[i];
    }
    if (threadIdx.x == 0) out->b4 = M.b4;
}

// x of the packed network for (chi, u) (kind 1: the electron's fraction d); NaN
// where the model does not sample.
__device__ __forceinline__ float infer_one(const MlpLds &M, MlpWave &W, bool valid, float chi, float u, int kind) {
    bool in_range;
    int bin;
    const float s = mlp_input_s(M, chi, in_range, bin);
    const bool use = valid && in_range && !M.fallback[bin];
    const float v = kind == 0 ? mlp_input_v(u) : mlp_input_v_pair(fabsf(2.0f * u - 1.0f));
    const float y = mlp_infer_wave(M, W, use, s, v);
    if (!use) return __builtin_nanf("");
    return kind == 0 ? mlp_x_of_y(y, chi) : pair_d_of_y(y, chi, u >= 0.5f);
}

__global__ __launch_bounds__(kBlock) void k_mlp_infer(const MlpModel *model, const float *chi, const float *u,
                                                      float *x, u64 n, int kind) {
    __shared__ MlpLds M;
    __shared__ MlpWave ws[kBlock / 64];
    mlp_stage(model, M);
    __syncthreads();
    MlpWave &W = ws[threadIdx.x / 64];
    // wave-uniform trip count: every lane takes part in the matrix-core passes
    for (u64 i0 = (u64)blockIdx.x * kBlock; i0 < n; i0 += (u64)gridDim.x * kBlock) {
        const u64 i = i0 + threadIdx.x;
        const bool valid = i < n;
        const float xi = infer_one(M, W, valid, valid ? chi[i] : 1.0f, valid ? u[i] : 0.5f, kind);
        if (valid) x[i] = xi;
    }
}

// One block per (bin, position in the bin); 1024 values of u per chi.
__global__ __launch_bounds__(kBlock) void k_mlp_validate(const MlpModel *model, CdfTableDev t, int per_bin,
                                                         float *bin_err) {
    __shared__ MlpLds M;
    __shared__ MlpWave ws[kBlock / 64];
    __shared__ float wmax[kBlock / 64];
    mlp_stage(model, M);
    __syncthreads();
    MlpWave &W = ws[threadIdx.x / 64];
    const int bin = blockIdx.x / per_bin, q = blockIdx.x % per_bin;
    const double span = 1.0 / (double)M.inv_span;
    const double l10 = (double)M.lo + span * ((double)bin + (double)q / (double)(per_bin - 1)) / (double)M.nbins;
    const double l10c = fmin(l10, (double)M.lo + span * (1.0 - 1e-7));   // stay inside [lo, hi)
    const float chi = (float)exp10(l10c);
    float emax = 0.0f;
    for (int k = threadIdx.x; k < 1024; k += kBlock) {
        const float u = ((float)k + 0.5f) / 1024.0f;
        bool in_range;
        int b;
        const float s = mlp_input_s(M, chi, in_range, b);
        const float y = mlp_infer_wave(M, W, true, s, t.kind == 0 ? mlp_input_v(u) : mlp_input_v_pair(u));
        // kind 1: u is u' of the half-distribution, the network gives D
        const float x = t.kind == 0 ? mlp_x_of_y(y, chi) : fminf(fmaxf(y * pair_width(chi), 0.0f), 0.5f);
        const double c = cdf_lookup(t, log10((double)chi), (double)x);
        emax = fmaxf(emax, (float)fabs(c - (double)u));
    }
    for (int o = 32; o > 0; o >>= 1) emax = fmaxf(emax, __shfl_xor(emax, o));
    if (__lane_id() == 0) wmax[threadIdx.x / 64] = emax;
    __syncthreads();
    if (threadIdx.x == 0) {
        float m = 0.0f;
        for (int w = 0; w < kBlock / 64; ++w) m = fmaxf(m, wmax[w]);
        atomicMax(reinterpret_cast<unsigned int *>(&bin_err[bin]), __float_as_uint(m));
    }
}

}  // namespace

hipError_t launch_cdf_table(const CdfTableDev &t, hipStream_t s) {
    if (t.nx % kBlock != 0 || t.nchi < 2) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_cdf_table, dim3(t.nchi), dim3(kBlock), 0, s, t);
    if (t.index) hipLaunchKernelGGL(k_cdf_index, dim3(t.nchi), dim3(kBlock), 0, s, t);
    return hipGetLastError();
}

hipError_t launch_mlp_data(const DataArgs &da, hipStream_t s) {
    hipLaunchKernelGGL(k_mlp_data, dim3(da.blocks), dim3(kBlock), 0, s, da);
    return hipGetLastError();
}

hipError_t launch_mlp_train(const TrainArgs &ta, int blocks, hipStream_t s) {
    hipLaunchKernelGGL(k_mlp_train, dim3(blocks), dim3(kTrainBlock), 0, s, ta);
    return hipGetLastError();
}

hipError_t launch_train_pack(const float *params, void *weights, hipStream_t s) {
    hipLaunchKernelGGL(k_train_pack, dim3((kMlpParams + kBlock - 1) / kBlock), dim3(kBlock), 0, s, params,
                       static_cast<TrainWeights *>(weights));
    return hipGetLastError();
}

hipError_t launch_mlp_reduce(const ReduceArgs &ra, const DataArgs *next, hipStream_t s) {
    DataArgs da{};
    if (next) da = *next;
    const int blocks = da.blocks + (kMlpParams + 1 + kRedParams - 1) / kRedParams;
    hipLaunchKernelGGL(k_mlp_reduce, dim3(blocks), dim3(kBlock), 0, s, ra, da);
    return hipGetLastError();
}

hipError_t launch_mlp_pack(const float *params, MlpModel *out, hipStream_t s) {
    hipLaunchKernelGGL(k_mlp_pack, dim3(1), dim3(kBlock), 0, s, params, out);
    return hipGetLastError();
}

hipError_t launch_mlp_validate(const MlpModel *model, const CdfTableDev &t, int nbins, int per_bin, float *bin_err,
                               hipStream_t s) {
    hipLaunchKernelGGL(k_mlp_validate, dim3(nbins * per_bin), dim3(kBlock), 0, s, model, t, per_bin, bin_err);
    return hipGetLastError();
}

hipError_t launch_mlp_infer(const MlpModel *model, const float *chi, const float *u, float *x, u64 n, int blocks,
                            hipStream_t s, int kind) {
    hipLaunchKernelGGL(k_mlp_infer, dim3(blocks), dim3(kBlock), 0, s, model, chi, u, x, n, kind);
    return hipGetLastError();
}

}  // namespace qed
