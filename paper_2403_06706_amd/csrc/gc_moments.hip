// gc_moments.hip -- snapshot statistics of the particle state (Sect. 3:
// <sin^2 alpha>(r), energy versus age near 1 AU, pitch-cosine distributions,
// and counts by status).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "gc_device.h"
#include "gc_launch.h"

namespace gc {

// ---------------------------------------------------------------------------
// Moments: per-block 64-bit histograms in LDS, merged with global atomics.
// Every contribution is an integer, so the result does not depend on order.
// ---------------------------------------------------------------------------
constexpr uint32_t kMomThreads = 512, kMomBlocks = 512;

__device__ __forceinline__ unsigned long long fixp(double x, double scale) {
    return (unsigned long long)(long long)floor(x * scale);
}

// Sum of v over the wavefront, modulo 2^64, in every lane: three limbs of at most
// 22 bits, so that 64 of them fit 32 bits, each reduced by six DPP additions.
// Every lane must be active.
__device__ __forceinline__ uint32_t wave_sum32(uint32_t x) {
    auto step = [&](auto ctrl, auto rows) {
        x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, decltype(ctrl)::value, decltype(rows)::value, 0xF, false);
    };
    using std::integral_constant;
    step(integral_constant<int, 0x111>(), integral_constant<int, 0xF>());   // row_shr 1, 2, 4, 8
    step(integral_constant<int, 0x112>(), integral_constant<int, 0xF>());
    step(integral_constant<int, 0x114>(), integral_constant<int, 0xF>());
    step(integral_constant<int, 0x118>(), integral_constant<int, 0xF>());
    step(integral_constant<int, 0x142>(), integral_constant<int, 0xA>());   // row_bcast 15: rows 1 and 3
    step(integral_constant<int, 0x143>(), integral_constant<int, 0xC>());   // row_bcast 31: rows 2 and 3
    return (uint32_t)__builtin_amdgcn_readlane((int)x, 63);
}
__device__ __forceinline__ unsigned long long wave_sum(unsigned long long v) {
    const unsigned long long a = wave_sum32((uint32_t)v & 0x3FFFFFu), b = wave_sum32((uint32_t)(v >> 22) & 0x3FFFFFu),
                             c = wave_sum32((uint32_t)(v >> 44));
    return a + (b << 22) + (c << 44);
}

// B at a point (g[0..2], the values of gather()); false where gather() is.  A tame
// field needs the nodes' first components only: a third of the loads for FP32 and
// FP64 fields, a quarter of the multiply-adds.
template <int FDT, bool TAME>
__device__ __forceinline__ bool field_b(const FieldDev &f, double r, double th, double ph, double g[12]) {
    if constexpr (!TAME) return gather<FDT, double>(f, r, th, ph, g);
    GatherPlan<double> gp;
    if (!gather_plan<FDT>(f, r, th, ph, gp)) return false;
    constexpr uint32_t W = Layout<FDT>::W, E = FDT == GC_F64 ? 8 : FDT == GC_F32 ? 4 : 2;
    constexpr int kLoads = W == 2 ? 2 : 1;
    using V = typename std::conditional<FDT == GC_F16, uint2, uint4>::type;
    V v[8][kLoads];
#pragma unroll
    for (int n = 0; n < 8; ++n)
#pragma unroll
        for (int c = 0; c < kLoads; ++c)
            v[n][c] = *reinterpret_cast<const V *>(static_cast<const char *>(f.data) + (size_t)(c * gp.cs) * E +
                                                   (gp.off[n / 2] + (n & 1) * gp.dk) * E);
    auto get = [&](int n, int c) -> double {
        if constexpr (FDT == GC_F64) {
            double d[2];
            __builtin_memcpy(d, &v[n][c / 2], 16);
            return d[c % 2];
        } else if constexpr (FDT == GC_F32) {
            float d[4];
            __builtin_memcpy(d, &v[n][0], 16);
            return (double)d[c];
        } else {
            __half d[4];
            __builtin_memcpy(d, &v[n][0], 8);
            return (double)(__half2float(d[c]) * f.scale[c]);
        }
    };
#pragma unroll
    for (int c = 0; c < 3; ++c) g[c] = 0.0;
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        const double wa = gp.w[p] * (1.0 - gp.wp), wb = gp.w[p] * gp.wp;
#pragma unroll
        for (int c = 0; c < 3; ++c) g[c] = fma(wb, get(2 * p + 1, c), fma(wa, get(2 * p, c), g[c]));
    }
    return true;
}

// Bound by latency and, before, by LDS atomics: cell-sorted particles of a
// wavefront share their radial bin, and 64 lanes adding to one address take turns.
// The wavefront now sums the bins of its first two distinct values itself
// (afterwards, in an unsorted set, the lanes add one by one); every load of a
// particle is issued at once; a tame field gives B alone.  2^20 electrons in cell
// order: 41 -> 28 us a call (71 MB: 15 us at the rate of a copy).
template <int FDT, bool TAME>
__global__ __launch_bounds__(kMomThreads) void k_moments(SoA st, FieldDev f, const EnsDev *ens, uint32_t n_all, MomDev m,
                                                         unsigned long long *out, const uint32_t *n_scan,
                                                         const unsigned long long *dead) {
    extern __shared__ unsigned long long h[];
    const uint32_t n = n_scan ? *n_scan : n_all;
    // consecutive particles: a workgroup of a cell-sorted set meets few radial bins,
    // and so merges few
    const uint32_t share = (n + gridDim.x - 1) / gridDim.x, per = (share + blockDim.x - 1) / blockDim.x * blockDim.x;
    const uint32_t begin = blockIdx.x * per, end = min(n, begin + per);
    if (blockIdx.x > 0 && begin >= n) return;                     // nothing to read (uniform)
    for (int i = threadIdx.x; i < m.total; i += blockDim.x) h[i] = 0ull;
    __syncthreads();
    unsigned long long *rb = h + 8;
    unsigned long long *mh = rb + 3 * m.n_rbins;
    unsigned long long *eh = mh + m.n_mubins;
    // the eight scalar moments are summed in registers, then once per wavefront
    unsigned long long acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    // (the trip count is uniform over the workgroup: the wavefront sums need every lane)
    for (uint32_t i0 = begin; i0 < end; i0 += blockDim.x) {
        const bool in = i0 + threadIdx.x < end;
        const uint32_t i = in ? i0 + threadIdx.x : n - 1;
        const uint32_t status = st.status[i], k = st.k[i], step = st.step[i], birth = st.birth[i];
        const uint32_t eidx = min(st.ens[i], (uint32_t)(kMaxEnsembles - 1));
        const double r = st.r[i], th = st.th[i], ph = st.ph[i], u = st.u[i], mu = st.mu[i], t = st.t[i];
        const double mass = ens[eidx].m;
        if (in) {
#pragma unroll
            for (uint32_t q = 0; q < 4; ++q) acc[q] += status == q ? 1 : 0;
            acc[4] += k;
            acc[5] += step;
        }
        bool live = in && status == GC_ACTIVE;
        if (live) {
            acc[6] += fixp(r / m.len_unit, 4294967296.0);
            if (k >= 1) acc[7] += 1;
        }
        double g[12];
        live = live && birth >= m.min_birth && field_b<FDT, TAME>(f, r, th, ph, g);
        double cosa = 0.0, ekin = 0.0;
        int bin = -1;
        unsigned long long vs = 0, ve = 0;
        if (live) {
            const double B = sqrt(g[0] * g[0] + g[1] * g[1] + g[2] * g[2]);
            const double p2 = u * u + 2.0 * mu * B;                // (|p|/m)^2
            const double pm = sqrt(p2);
            cosa = pm > 0.0 ? u / pm : 1.0;
            const double sin2 = 1.0 - cosa * cosa;
            const double gamma = sqrt(1.0 + p2 * kInvC2);
            ekin = (gamma - 1.0) * mass * kC * kC / m.e_unit;
            if (m.n_rbins > 0) {
                const double x = (r - m.r_lo) / (m.r_hi - m.r_lo) * m.n_rbins;
                if (x >= 0.0 && x < (double)m.n_rbins) {
                    bin = (int)floor(x);
                    vs = fixp(sin2, 4294967296.0);
                    ve = fixp(ekin, 65536.0);
                }
            }
        }
        uint64_t todo = __ballot(bin >= 0);
#pragma unroll 1
        for (int round = 0; round < 2 && todo; ++round) {
            const int b = __builtin_amdgcn_readlane(bin, __builtin_ctzll(todo));
            const bool mine = bin == b;
            const uint64_t same = __ballot(mine);
            const unsigned long long s1 = wave_sum(mine ? vs : 0ull), s2 = wave_sum(mine ? ve : 0ull);
            if ((threadIdx.x & 63u) == 0) {
                atomicAdd(&rb[3 * b + 0], (unsigned long long)__popcll(same));
                atomicAdd(&rb[3 * b + 1], s1);
                atomicAdd(&rb[3 * b + 2], s2);
            }
            if (mine) bin = -1;
            todo &= ~same;
        }
        if (bin >= 0) {
            atomicAdd(&rb[3 * bin + 0], 1ull);
            atomicAdd(&rb[3 * bin + 1], vs);
            atomicAdd(&rb[3 * bin + 2], ve);
        }
        if (!live || r < m.sel_r_lo || r >= m.sel_r_hi) continue;
        if (m.n_mubins > 0 && t >= m.age_lo && t < m.age_hi && (int64_t)k >= (int64_t)m.min_collisions) {
            const double x = (cosa + 1.0) * 0.5 * m.n_mubins;
            int bi = (int)floor(x);
            bi = bi < 0 ? 0 : (bi >= m.n_mubins ? m.n_mubins - 1 : bi);
            atomicAdd(&mh[bi], 1ull);
        }
        if (m.n_agebins > 0 && m.n_ebins > 0) {
            const double xa = t / m.age_max * m.n_agebins;
            const double xe = (ekin - m.e_lo) / (m.e_hi - m.e_lo) * m.n_ebins;
            if (xa >= 0.0 && xa < (double)m.n_agebins && xe >= 0.0 && xe < (double)m.n_ebins)
                atomicAdd(&eh[(int)floor(xa) * m.n_ebins + (int)floor(xe)], 1ull);
        }
    }
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const unsigned long long v = wave_sum(acc[q]);
        if ((threadIdx.x & 63u) == 0 && v) atomicAdd(&h[q], v);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < m.total; i += blockDim.x)
        if (h[i]) atomicAdd(&out[i], h[i]);
    // slots past the live prefix: their sums, kept by the reorders
    if (dead && blockIdx.x == 0 && threadIdx.x < 6 && dead[threadIdx.x]) atomicAdd(&out[threadIdx.x], dead[threadIdx.x]);
}

template <int FDT>
static void launch_moments_t(const SoA &st, const FieldDev &f, const EnsDev *ens, uint32_t n, const MomDev &m,
                             unsigned long long *out, const uint32_t *n_scan, const unsigned long long *dead,
                             hipStream_t s) {
    const dim3 grid(std::min<uint32_t>((n + kMomThreads - 1) / kMomThreads, kMomBlocks)), block(kMomThreads);
    const size_t lds = (size_t)m.total * sizeof(unsigned long long);
    if (f.tame) hipLaunchKernelGGL((k_moments<FDT, true>), grid, block, lds, s, st, f, ens, n, m, out, n_scan, dead);
    else hipLaunchKernelGGL((k_moments<FDT, false>), grid, block, lds, s, st, f, ens, n, m, out, n_scan, dead);
}

hipError_t launch_moments(const SoA &st, const FieldDev &f, const EnsDev *ens, uint32_t n, const MomDev &m,
                          unsigned long long *out, const uint32_t *n_scan, const unsigned long long *dead,
                          hipStream_t s) {
    hipError_t e = m.accumulate ? hipSuccess : launch_fill_u64(out, 0ull, (size_t)m.total, s);
    if (e != hipSuccess || n == 0) return e;
    switch (f.dtype) {
        case GC_F64: launch_moments_t<GC_F64>(st, f, ens, n, m, out, n_scan, dead, s); break;
        case GC_F32: launch_moments_t<GC_F32>(st, f, ens, n, m, out, n_scan, dead, s); break;
        default:     launch_moments_t<GC_F16>(st, f, ens, n, m, out, n_scan, dead, s); break;
    }
    return hipGetLastError();
}

}  // namespace gc
