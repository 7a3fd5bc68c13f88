// gc_kernels.hip -- injection, field packing, state copies, fills.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "gc_device.h"
#include "gc_launch.h"
#include "gc_step.h"

namespace gc {

// ---------------------------------------------------------------------------
// Field packing: [nr][nth][nph][12] float64 (staged on the device) -> the
// blocked layout of field_layout in the storage type (records == 0), or node
// records [nr][nth][nph+1][12] (records != 0); the extra phi node k = nph
// repeats node 0, padding nodes are zero.  FP16 stores v / scale rounded once
// from double to half.
// ---------------------------------------------------------------------------
__global__ void k_pack_field(const double *src, void *dst, int nr, int nth, int nph, int dtype, int records,
                             const float *inv_scale_in) {
    const FieldLayout L = field_layout(nr, nth, nph, dtype);
    const uint64_t nI = L.cs / (kLayB * L.W), nK = L.js / L.ks;
    const uint64_t total = records ? (uint64_t)nr * nth * (nph + 1) * 12 : L.total;
    for (uint64_t o = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; o < total;
         o += (uint64_t)gridDim.x * blockDim.x) {
        uint64_t i, j, k;
        int comp;
        if (records) {
            comp = (int)(o % 12);
            const uint64_t node = o / 12;
            k = node % (nph + 1);
            j = (node / (nph + 1)) % nth;
            i = node / ((uint64_t)(nph + 1) * nth);
        } else {
            uint64_t t = o / L.W;
            const uint64_t e = o % L.W;
            const uint64_t ii = t % kLayBr;
            t /= kLayBr;
            const uint64_t kk = t % kLayBk;
            t /= kLayBk;
            const uint64_t I = t % nI;
            t /= nI;
            const uint64_t c = t % L.nch;
            t /= L.nch;
            const uint64_t K = t % nK;
            j = t / nK;
            i = I * kLayBr + ii;
            k = K * kLayBk + kk;
            comp = (int)(c * L.W + e);
        }
        double v = 0.0;
        if (i < (uint64_t)nr && k <= (uint64_t)nph)
            v = src[((i * nth + j) * nph + (k == (uint64_t)nph ? 0 : k)) * 12 + comp];
        if (dtype == GC_F64) static_cast<double *>(dst)[o] = v;
        else if (dtype == GC_F32) static_cast<float *>(dst)[o] = (float)v;
        else   // one rounding, double -> half (to nearest even)
            static_cast<__half *>(dst)[o] = __half_raw{static_cast<_Float16>(v * (double)inv_scale_in[comp])};
    }
}

hipError_t launch_pack_field(const double *src, void *dst, int nr, int nth, int nph, int dtype, int records,
                             const float *inv_scale, hipStream_t s) {
    hipLaunchKernelGGL(k_pack_field, dim3(2048), dim3(256), 0, s, src, dst, nr, nth, nph, dtype, records, inv_scale);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Injection (Sect. 3): one particle per lane, FP64.
// ---------------------------------------------------------------------------
template <int FDT>
__global__ void k_inject(SoA st, FieldDev f, EnsDev e, uint32_t n0, uint32_t n, uint32_t first_id, uint32_t eidx) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const uint32_t slot = n0 + i, pid = first_id + i;
    const BirthState b = birth_state<FDT>(f, e, pid, 0);
    st.r[slot] = b.r; st.th[slot] = b.th; st.ph[slot] = b.ph; st.u[slot] = b.u; st.mu[slot] = b.mu;
    st.fr[slot] = 0.0; st.fth[slot] = 0.0; st.fph[slot] = 0.0; st.fu[slot] = 0.0;
    st.dtp[slot] = 0.0; st.s[slot] = 0.0; st.ell[slot] = b.ell; st.t[slot] = 0.0;
    st.cr[slot] = 0.0; st.cth[slot] = 0.0; st.cph[slot] = 0.0; st.cu[slot] = 0.0; st.ct[slot] = 0.0;
    st.k[slot] = 0; st.flags[slot] = GC_FLAG_BOOTSTRAP; st.status[slot] = b.status; st.step[slot] = 0;
    st.id[slot] = pid; st.ens[slot] = eidx; st.gid[slot] = slot; st.birth[slot] = 0;
}

hipError_t launch_inject(const SoA &st, const FieldDev &f, const EnsDev &e, uint32_t n0, uint32_t n,
                         uint32_t first_id, uint32_t eidx, hipStream_t s) {
    if (n == 0) return hipSuccess;
    const dim3 grid((n + 255) / 256), block(256);
    switch (f.dtype) {
        case GC_F64: hipLaunchKernelGGL(k_inject<GC_F64>, grid, block, 0, s, st, f, e, n0, n, first_id, eidx); break;
        case GC_F32: hipLaunchKernelGGL(k_inject<GC_F32>, grid, block, 0, s, st, f, e, n0, n, first_id, eidx); break;
        default:     hipLaunchKernelGGL(k_inject<GC_F16>, grid, block, 0, s, st, f, e, n0, n, first_id, eidx); break;
    }
    return hipGetLastError();
}

__global__ void k_fill_u64(unsigned long long *p, unsigned long long v, size_t n) {
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) p[i] = v;
}
__global__ void k_fill_u32(uint32_t *p, uint32_t v, size_t n) {
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) p[i] = v;
}

static unsigned grid_for(size_t n, unsigned block) {
    size_t g = (n + block - 1) / block;
    if (g > 4096) g = 4096;
    return g == 0 ? 1u : (unsigned)g;
}

hipError_t launch_fill_u64(unsigned long long *p, unsigned long long v, size_t n, hipStream_t s) {
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_fill_u64, dim3(grid_for(n, 256)), dim3(256), 0, s, p, v, n);
    return hipGetLastError();
}
hipError_t launch_fill_u32(uint32_t *p, uint32_t v, size_t n, hipStream_t s) {
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_fill_u32, dim3(grid_for(n, 256)), dim3(256), 0, s, p, v, n);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// State export / import in global injection order.
// ---------------------------------------------------------------------------
#define GC_FOR_DOUBLES(X) X(r) X(th) X(ph) X(u) X(mu) X(fr) X(fth) X(fph) X(fu) X(dtp) X(s) X(ell) X(t) \
                          X(cr) X(cth) X(cph) X(cu) X(ct)
#define GC_FOR_U32(X) X(k) X(flags) X(status) X(step) X(id) X(ens) X(birth)

// Slots to injection order.  Scattered stores of 25 arrays wrote whole lines for 4
// or 8 bytes each (2^20 particles: 0.42 ms for 172 bytes read and written a
// particle), so the order is inverted first and the arrays are gathered, four
// particles a thread.  Each XCD (workgroups go to them round-robin) takes two of the
// first sixteen FP64 arrays, one after the other, and one of the 32-bit arrays: read by
// one XCD, an array comes into one L2 (4 MB: 500,000 particles) once.  Gathered by all
// of them it came into eight: 300,007 particles 56 -> 34 us, 500,000 104 -> 75; the last
// two FP64 arrays still are.  Past kOutFits an array overflows the one L2 by so much
// that every XCD gathers from every array (2^20 particles: 160 us against 166).
__global__ void k_invert(const uint32_t *gid, uint32_t *inv, uint32_t n) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) inv[gid[i]] = i;
}

struct StateOut {
    const void *src[25];
    void *dst[25];        // NULL: skipped
};
constexpr int kOutDoubles = 18, kOutArrays = 25;

template <typename T>
__device__ __forceinline__ void gather4(const void *from, void *to, const uint32_t *inv, uint32_t chunk, uint32_t n) {
    const T *src = static_cast<const T *>(from);
    T *dst = static_cast<T *>(to);
    const uint32_t g0 = chunk * blockDim.x * 4 + threadIdx.x;
    uint32_t at[4];
    T v[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) at[q] = inv[min(g0 + q * blockDim.x, n - 1)];
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = src[at[q]];
#pragma unroll
    for (int q = 0; q < 4; ++q)
        if (g0 + q * blockDim.x < n) dst[g0 + q * blockDim.x] = v[q];
}

constexpr uint32_t kOutXcds = 8, kOutShared = 16;           // FP64 arrays [0, kOutShared): two per XCD
static_assert(2 * kOutXcds == kOutShared && kOutDoubles >= (int)kOutShared &&
              kOutArrays - kOutDoubles <= (int)kOutXcds, "array shares");

constexpr uint32_t kOutFits = 786432;                       // particles: 6 MB an FP64 array

// nb workgroups per array; the arrays from `shared` on (kOutShared, or 0: all) by all XCDs
__global__ __launch_bounds__(256) void k_state_out(StateOut a, const uint32_t *inv, uint32_t nb, uint32_t shared,
                                                   uint32_t n) {
    const uint32_t b = blockIdx.x, own = shared ? 3 * kOutXcds * nb : 0;
    uint32_t y, chunk;
    if (b < own) {
        const uint32_t xcd = b % kOutXcds, pos = b / kOutXcds, item = pos / nb;
        chunk = pos % nb;
        y = item < 2 ? 2 * xcd + item : kOutDoubles + xcd;
    } else {
        y = shared + (b - own) / nb;
        chunk = (b - own) % nb;
    }
    if (y >= (uint32_t)kOutArrays || !a.dst[y]) return;
    if (y < (uint32_t)kOutDoubles) gather4<uint64_t>(a.src[y], a.dst[y], inv, chunk, n);
    else gather4<uint32_t>(a.src[y], a.dst[y], inv, chunk, n);
}

__global__ void k_state_in(SoA st, gc_state_view src, uint32_t n) {
    const uint32_t g = blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= n) return;
#define IN_(name) st.name[g] = src.name[g];
    GC_FOR_DOUBLES(IN_)
    GC_FOR_U32(IN_)
#undef IN_
    st.gid[g] = g;
}

hipError_t launch_state_out(const SoA &st, const gc_state_view &dst, uint32_t n, uint32_t *inv, hipStream_t s) {
    if (n == 0) return hipSuccess;
    StateOut a{};
    int k = 0;
#define OUT_(name) a.src[k] = st.name; a.dst[k++] = dst.name;
    GC_FOR_DOUBLES(OUT_)
    GC_FOR_U32(OUT_)
#undef OUT_
    hipLaunchKernelGGL(k_invert, dim3((n + 255) / 256), dim3(256), 0, s, st.gid, inv, n);
    const uint32_t nb = (n + 1023) / 1024;
    const uint32_t shared = n <= kOutFits ? kOutShared : 0;
    const uint32_t arrays = shared ? 3 * kOutXcds + kOutDoubles - kOutShared : kOutArrays;
    hipLaunchKernelGGL(k_state_out, dim3(nb * arrays), dim3(256), 0, s, a, inv, nb, shared, n);
    return hipGetLastError();
}
hipError_t launch_state_in(const SoA &st, const gc_state_view &src, uint32_t n, hipStream_t s) {
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_state_in, dim3((n + 255) / 256), dim3(256), 0, s, st, src, n);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Plain streaming copy for counter calibration and the achievable HBM rate:
// each thread keeps four independent 16-byte loads in flight per iteration.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_copy_probe(uint4 *dst, const uint4 *src, size_t n16) {
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
    for (; i + 3 * stride < n16; i += 4 * stride) {
        const uint4 a = src[i], b = src[i + stride], c = src[i + 2 * stride], d = src[i + 3 * stride];
        dst[i] = a;
        dst[i + stride] = b;
        dst[i + 2 * stride] = c;
        dst[i + 3 * stride] = d;
    }
    for (; i < n16; i += stride) dst[i] = src[i];
}

hipError_t launch_copy_probe(void *dst, const void *src, size_t n_bytes, hipStream_t s) {
    const size_t n16 = n_bytes / 16;
    if (n16 == 0) return hipSuccess;
    const size_t want = (n16 + 4 * 256 - 1) / (4 * 256);           // four pieces per thread
    const unsigned grid = (unsigned)std::min<size_t>(std::max<size_t>(want, 1), 32768);
    hipLaunchKernelGGL(k_copy_probe, dim3(grid), dim3(256), 0, s, static_cast<uint4 *>(dst),
                       static_cast<const uint4 *>(src), n16);
    return hipGetLastError();
}

}  // namespace gc
