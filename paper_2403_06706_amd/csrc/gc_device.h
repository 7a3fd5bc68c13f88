// gc_device.h -- device building blocks of the push: counter-based random
// numbers, trilinear field gather, guiding-centre right-hand side.
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>
#include <hip/hip_fp16.h>
#include <stdint.h>

#include "gc_internal.h"

namespace gc {

constexpr double kC = 299792458.0;                    // speed of light (m/s)
constexpr double kInvC2 = 1.0 / (299792458.0 * 299792458.0);
constexpr double kPi = 3.14159265358979323846;

// A condition that seldom holds: its branch is laid out away from the path of
// the others.
__device__ __forceinline__ bool rare(bool c) { return __builtin_expect(c, 0); }

// ---------------------------------------------------------------------------
// Philox4x64-10 (Salmon, Moraes, Dror & Shaw, SC'11): ten rounds of the
// 64x64->128-bit multiply-xor bijection, key advanced by two Weyl constants.
// ---------------------------------------------------------------------------
struct U64x4 { uint64_t v[4]; };

__device__ __forceinline__ U64x4 philox4x64_10(uint64_t c0, uint64_t c1, uint64_t c2, uint64_t c3,
                                               uint64_t k0, uint64_t k1) {
#pragma unroll
    for (int round = 0; round < 10; ++round) {
        if (round) { k0 += 0x9E3779B97F4A7C15ULL; k1 += 0xBB67AE8584CAA73BULL; }
        const uint64_t m0 = 0xD2E7470EE14C6C93ULL, m1 = 0xCA5A826395121157ULL;
        uint64_t hi0 = __umul64hi(m0, c0), lo0 = m0 * c0;
        uint64_t hi1 = __umul64hi(m1, c2), lo1 = m1 * c2;
        uint64_t n0 = hi1 ^ c1 ^ k0, n2 = hi0 ^ c3 ^ k1;
        c0 = n0; c1 = lo1; c2 = n2; c3 = lo0;
    }
    U64x4 o; o.v[0] = c0; o.v[1] = c1; o.v[2] = c2; o.v[3] = c3;
    return o;
}

// uniform double on [0, 1) from the top 53 bits
__device__ __forceinline__ double u01(uint64_t x) { return (double)(x >> 11) * 0x1.0p-53; }

// counter word 2: what the block is drawn for
enum : uint64_t { kPurposePath = 0, kPurposeInject = 1 };

// ---------------------------------------------------------------------------
// Trilinear interpolation of the packed grid in index space: r nodes from
// r_min with spacing dr, theta nodes at (j + 1/2) dth, phi periodic.  The
// stencil is clamped to the grid in floating point before any conversion to
// an integer, so every load stays inside the buffer for any input.
// Returns false if the input or any interpolated value is not finite.
//
// The packed layout (chunks of W components, 4 x 2 node blocks) is described
// with field_layout in gc_internal.h.  Loads address the field as its base
// (uniform, or plus a uniform chunk offset) and a 32-bit byte offset per lane,
// the form of the SGPR-base global load; the packed field is at most 4 GiB.
// ---------------------------------------------------------------------------
template <typename R>
__device__ __forceinline__ R clampr(R x, R lo, R hi) { return fmin(fmax(x, lo), hi); }

// Chunk width and count per node of each storage type (as field_layout).
template <int FDT> struct Layout { static constexpr uint32_t W = 4, nch = 3; };   // FP32, FP16
template <> struct Layout<GC_F64> { static constexpr uint32_t W = 2, nch = 6; };

template <int FDT> struct Pair;   // 24 values of two phi-adjacent nodes, 12 components each

// Each load(): off = element offset of chunk 0 of the pair's first node, dk =
// offset of the second node from the first, cs = element stride between
// chunks; chunk c of node h is at off + h dk + c cs.
template <> struct Pair<GC_F32> {
    float v[24];
    __device__ __forceinline__ void load(const void *base, uint32_t off, uint32_t dk, uint32_t cs) {
        const char *b = static_cast<const char *>(base);
#pragma unroll
        for (int q = 0; q < 6; ++q) {
            const float4 x = *reinterpret_cast<const float4 *>(b + (size_t)((q % 3) * cs) * 4u +
                                                               (off + (q / 3) * dk) * 4u);
            v[4 * q + 0] = x.x; v[4 * q + 1] = x.y; v[4 * q + 2] = x.z; v[4 * q + 3] = x.w;
        }
    }
    __device__ __forceinline__ float get(int c, const FieldDev &) const { return v[c]; }
};

template <> struct Pair<GC_F64> {
    double v[24];
    __device__ __forceinline__ void load(const void *base, uint32_t off, uint32_t dk, uint32_t cs) {
        const char *b = static_cast<const char *>(base);
#pragma unroll
        for (int q = 0; q < 12; ++q) {
            const double2 x = *reinterpret_cast<const double2 *>(b + (size_t)((q % 6) * cs) * 8u +
                                                                (off + (q / 6) * dk) * 8u);
            v[2 * q + 0] = x.x; v[2 * q + 1] = x.y;
        }
    }
    __device__ __forceinline__ double get(int c, const FieldDev &) const { return v[c]; }
};

template <> struct Pair<GC_F16> {
    __half v[24];
    __device__ __forceinline__ void load(const void *base, uint32_t off, uint32_t dk, uint32_t cs) {
        const char *b = static_cast<const char *>(base);
#pragma unroll
        for (int q = 0; q < 6; ++q) {
            const uint2 x = *reinterpret_cast<const uint2 *>(b + (size_t)((q % 3) * cs) * 2u +
                                                             (off + (q / 3) * dk) * 2u);
            __half h[4];
            __builtin_memcpy(h, &x, 8);
            v[4 * q + 0] = h[0]; v[4 * q + 1] = h[1]; v[4 * q + 2] = h[2]; v[4 * q + 3] = h[3];
        }
    }
    __device__ __forceinline__ float get(int c, const FieldDev &f) const {
        return __half2float(v[c]) * f.scale[c % 12];
    }
};

// Stencil of a trilinear gather: the four node pairs (r, theta corners, each
// with its two phi nodes) and their weights.
template <typename R>
struct GatherPlan {
    R w[4];              // (r, theta) weight of each node pair
    R wp;                // phi weight of the second node of a pair
    uint32_t off[4];     // element offset of chunk 0 of each pair's first node
    uint32_t dk;         // offset of a pair's second (phi) node from its first
    uint32_t cs;         // element stride between chunks
    uint32_t rec;        // element offset of the first node of pair 0 in the node records
};

template <int FDT, typename R>
__device__ __forceinline__ bool gather_plan(const FieldDev &f, R r, R th, R ph, GatherPlan<R> &gp) {
    R x = (r - (R)f.r_min) * (R)f.inv_dr;
    R y = th * (R)f.inv_dth - (R)0.5;
    R z = ph * (R)f.inv_dph;
    if (!(isfinite(x) && isfinite(y) && isfinite(z))) return false;
    const R nph = (R)f.nph;
    R fi = clampr(floor(x), (R)0, (R)(f.nr - 2));
    R fj = clampr(floor(y), (R)0, (R)(f.nth - 2));
    R wr = clampr(x - fi, (R)0, (R)1);
    R wt = clampr(y - fj, (R)0, (R)1);
    R zf = floor(z);
    gp.wp = z - zf;
    R km = zf - nph * floor(zf * (R)f.inv_nph);
    km = km < (R)0 ? km + nph : km;
    km = km >= nph ? km - nph : km;
    km = clampr(km, (R)0, nph - (R)1);
    const uint32_t i = (uint32_t)fi, j = (uint32_t)fj, k = (uint32_t)km;
    constexpr uint32_t W = Layout<FDT>::W;
    // separable offsets of the blocked layout (field_layout)
    const uint32_t i1 = i + 1u;
    const uint32_t gi0 = (i >> 2) * (kLayB * W) + (i & 3u) * W;
    const uint32_t gi1 = (i1 >> 2) * (kLayB * W) + (i1 & 3u) * W;
    const uint32_t gk0 = (k >> 1) * f.ks + (k & 1u) * (kLayBr * W);
    gp.dk = (k & 1u) ? f.ks - kLayBr * W : kLayBr * W;          // gK(k + 1) - gK(k)
    const uint32_t gj0 = j * f.js;
    gp.cs = f.cs;
    gp.rec = ((i * (uint32_t)f.nth + j) * (uint32_t)(f.nph + 1) + k) * 12u;
    gp.w[0] = ((R)1 - wr) * ((R)1 - wt);
    gp.w[1] = ((R)1 - wr) * wt;
    gp.w[2] = wr * ((R)1 - wt);
    gp.w[3] = wr * wt;
    gp.off[0] = gj0 + gk0 + gi0;
    gp.off[1] = gj0 + f.js + gk0 + gi0;
    gp.off[2] = gj0 + gk0 + gi1;
    gp.off[3] = gj0 + f.js + gk0 + gi1;
    return true;
}

// Add node pair p (index q of the stencil) to out: for each component,
// out = fma(wb, B, fma(wa, A, out)) with wa = w_q (1 - w_ph), wb = w_q w_ph.
template <int FDT, typename R>
__device__ __forceinline__ void gather_add(const FieldDev &f, const GatherPlan<R> &gp, int q, const Pair<FDT> &p,
                                           R out[12]) {
    const R wa = gp.w[q] * ((R)1 - gp.wp), wb = gp.w[q] * gp.wp;
#pragma unroll
    for (int c = 0; c < 12; ++c) out[c] = fma(wb, (R)p.get(c + 12, f), fma(wa, (R)p.get(c, f), out[c]));
}

template <int N, typename R>
__device__ __forceinline__ bool finite_sum(const R out[N]) {
    R sum = (R)0;
#pragma unroll
    for (int c = 0; c < N; ++c) sum += out[c];
    return isfinite(sum);
}
template <typename R>
__device__ __forceinline__ bool finite12(const R out[12]) { return finite_sum<12>(out); }

// One lane: the four node pairs added in order, at most two of them in registers
// at a time.  kTame: the caller knows the field is tame (FieldDev::tame): no
// finiteness test.
template <int FDT, typename R, bool kTame = false>
__device__ __forceinline__ bool gather(const FieldDev &f, R r, R th, R ph, R out[12]) {
    GatherPlan<R> gp;
    if (!gather_plan<FDT>(f, r, th, ph, gp)) return false;
#pragma unroll
    for (int c = 0; c < 12; ++c) out[c] = (R)0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        Pair<FDT> p;
        p.load(f.data, gp.off[q], gp.dk, gp.cs);
        gather_add<FDT, R>(f, gp, q, p, out);
        if (q & 1) __builtin_amdgcn_sched_barrier(0);   // at most two node pairs in registers
    }
    if constexpr (kTame) return true;
    else return finite12(out);
}

// ---------------------------------------------------------------------------
// Cell-resident gathers: a lane keeps the 8 nodes of the cell it evaluated last
// in registers, as stored, with the cell's origin in index space.  An
// evaluation in the same cell takes them from there, without the stencil's
// index arithmetic and without a load: nearly every evaluation at X^{n+1}, which
// differs from X* of the step before by the corrector's last order, and the
// X* of a lane that stays in its cell.  The values, their weights and the order
// of the multiply-adds are those of gather().
//
// cell_seek moves to the cell of a point (loading its nodes if it is another
// one) and leaves the weights of the point; false for a non-finite point.
// ---------------------------------------------------------------------------
template <typename R>
struct CellPos {
    R fi, fj, zf;        // lower node in index space (zf: phi, not wrapped); NaN: no cell
    R wr, wt, wp;        // weights of the upper nodes at the point sought last
    __device__ __forceinline__ CellPos() : fi((R)__builtin_nan("")), fj(fi), zf(fi) {}
};

// Every weight in [0, 1): as unsigned integers such bit patterns are below that
// of 1, and those of negative, larger and non-finite values are not.
__device__ __forceinline__ bool in_unit(double a, double b, double c) {
    const uint32_t m = max(max((uint32_t)__double2hiint(a), (uint32_t)__double2hiint(b)), (uint32_t)__double2hiint(c));
    return m < 0x3FF00000u;
}
__device__ __forceinline__ bool in_unit(float a, float b, float c) {
    return max(max(__float_as_uint(a), __float_as_uint(b)), __float_as_uint(c)) < 0x3F800000u;
}

// A value the compiler knows nothing about: a register it need not keep alive
// before this point.
template <typename T>
__device__ __forceinline__ void forget(T &x) { asm volatile("" : "=v"(x)); }

// The nodes of a cell, one lane per particle: chunk c of node h of pair p at
// q[(2 p + h) kWhole + c].  NC = 9: the extra array of the full equations (9
// components and 3 zeros a node), the ninth alone in last (FP16: whole chunks).
template <int FDT, int NC = 12>
struct LaneCell {
    static constexpr int W = Layout<FDT>::W, kChunks = Layout<FDT>::nch;
    static constexpr int kWhole = FDT == GC_F16 ? kChunks : NC / W;          // chunks loaded whole
    static constexpr bool kLast = kWhole * W < NC;
    using T = typename std::conditional<FDT == GC_F64, double, float>::type;
    using V = typename std::conditional<FDT == GC_F64, double __attribute__((ext_vector_type(2))),
              typename std::conditional<FDT == GC_F32, float __attribute__((ext_vector_type(4))),
                                        uint32_t __attribute__((ext_vector_type(2)))>::type>::type;
    V q[8 * kWhole];
    T last[kLast ? 8 : 1];
    template <typename R>
    __device__ __forceinline__ void load(const FieldDev &f, const GatherPlan<R> &gp, uint32_t) {
        constexpr uint32_t E = sizeof(V) / W;             // bytes of a component
        const char *b = static_cast<const char *>(f.data);
#pragma unroll
        for (int n = 0; n < 8; ++n)
#pragma unroll
            for (int c = 0; c < kWhole + (kLast ? 1 : 0); ++c) {
                const char *a = b + (size_t)(c * gp.cs) * E + (gp.off[n / 2] + (n & 1) * gp.dk) * E;
                if (c < kWhole) q[n * kWhole + c] = *reinterpret_cast<const V *>(a);
                else last[n] = *reinterpret_cast<const T *>(a);
            }
    }
    __device__ __forceinline__ T get(int p, int h, int c, const FieldDev &f) const {
        if (kLast && c == NC - 1) return last[2 * p + h];
        const V v = q[(2 * p + h) * kWhole + c / W];
        if constexpr (FDT != GC_F16) return v[c % W];
        else return __half2float(__ushort_as_half((unsigned short)(v[(c % 4) / 2] >> (16 * (c % 2))))) * f.scale[c];
    }
    __device__ __forceinline__ void drop() {
#pragma unroll
        for (int i = 0; i < 8 * kWhole; ++i) forget(q[i]);
        if (kLast)
#pragma unroll
            for (int i = 0; i < 8; ++i) forget(last[i]);
    }
    // components [c0, c1) at the weights of at
    template <int c0, int c1, typename R>
    __device__ __forceinline__ void value(const FieldDev &f, const CellPos<R> &at, uint32_t, R out[]) const {
        const R w[4] = {((R)1 - at.wr) * ((R)1 - at.wt), ((R)1 - at.wr) * at.wt, at.wr * ((R)1 - at.wt), at.wr * at.wt};
#pragma unroll
        for (int c = c0; c < c1; ++c) out[c] = (R)0;
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            const R wa = w[p] * ((R)1 - at.wp), wb = w[p] * at.wp;
#pragma unroll
            for (int c = c0; c < c1; ++c) out[c] = fma(wb, (R)get(p, 1, c, f), fma(wa, (R)get(p, 0, c, f), out[c]));
        }
    }
};

// A value of lane J of an aligned group of G = 2 or 4 lanes, to every lane of the
// group (DPP quad permutations [J, J, J, J], or [J, J, J + 2, J + 2]).
template <int G, int J, typename R>
__device__ __forceinline__ R group_bcast(R x) {
    static_assert(sizeof(R) % 4 == 0 && (G == 2 || G == 4) && J < G, "whole words, lanes of the group");
    constexpr int kPerm = G == 4 ? J * 0x55 : J | J << 2 | (J + 2) << 4 | (J + 2) << 6;
    uint32_t w[sizeof(R) / 4];
    __builtin_memcpy(w, &x, sizeof w);
#pragma unroll
    for (int i = 0; i < (int)(sizeof(R) / 4); ++i)
        w[i] = (uint32_t)__builtin_amdgcn_mov_dpp((int)w[i], kPerm, 0xF, 0xF, true);
    R y;
    __builtin_memcpy(&y, w, sizeof w);
    return y;
}

// The nodes of a cell, an aligned group of G = 2 or 4 lanes per particle (FP32 and
// FP64 fields): lane gl keeps the N = 12 / G components from N gl on (node h of
// pair p at v[p][N h + c], from the node records, whose phi pairs are adjacent, 48
// or 96 bytes each), runs their chains with the operations and order of gather_add,
// and the group exchanges the finished components, so all its lanes hold the bits
// of gather().  Each lane converts and multiplies its share of the values.  All
// lanes of the group must call value together.
template <int FDT, int G>
struct GroupCell {
    using T = typename std::conditional<FDT == GC_F64, double, float>::type;
    static constexpr int N = 12 / G;
    T v[4][2 * N];
    template <typename R>
    __device__ __forceinline__ void load(const FieldDev &f, const GatherPlan<R> &gp, uint32_t gl) {
        const uint32_t row = (uint32_t)(f.nph + 1) * 12u;             // theta stride of the records
        const uint32_t o[4] = {gp.rec, gp.rec + row, gp.rec + (uint32_t)f.nth * row, gp.rec + (uint32_t)f.nth * row + row};
        // per-lane 64-bit addresses: the components of a node merge into wide loads
        // and the second node is a constant offset from the first
        const T *base = static_cast<const T *>(f.rec) + N * gl;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const T *p = base + o[q];
#pragma unroll
            for (int c = 0; c < N; ++c) {
                v[q][c] = p[c];            // node k
                v[q][N + c] = p[12 + c];   // node k + 1
            }
        }
    }
    __device__ __forceinline__ void drop() {
#pragma unroll
        for (int i = 0; i < 8 * N; ++i) forget(v[i / (2 * N)][i % (2 * N)]);
    }
    template <int c0, int c1, typename R>
    __device__ __forceinline__ void value(const FieldDev &, const CellPos<R> &at, uint32_t, R out[]) const {
        const R w[4] = {((R)1 - at.wr) * ((R)1 - at.wt), ((R)1 - at.wr) * at.wt, at.wr * ((R)1 - at.wt), at.wr * at.wt};
        R acc[N] = {};
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const R wa = w[q] * ((R)1 - at.wp), wb = w[q] * at.wp;
#pragma unroll
            for (int c = 0; c < N; ++c) acc[c] = fma(wb, (R)v[q][N + c], fma(wa, (R)v[q][c], acc[c]));
        }
#pragma unroll
        for (int c = 0; c < N; ++c) {
            if (c0 <= c && c < c1) out[c] = group_bcast<G, 0>(acc[c]);
            if (c0 <= N + c && N + c < c1) out[N + c] = group_bcast<G, 1>(acc[c]);
            if constexpr (G == 4) {
                if (c0 <= 6 + c && 6 + c < c1) out[6 + c] = group_bcast<G, 2>(acc[c]);
                if (c0 <= 9 + c && 9 + c < c1) out[9 + c] = group_bcast<G, 3>(acc[c]);
            }
        }
    }
};

// more: null, or the extra array's cell (description fx) moved along with it.
struct NoCell {
    template <typename R> __device__ __forceinline__ void load(const FieldDev &, const GatherPlan<R> &, uint32_t) {}
};
template <int FDT, typename R, typename Cell, typename More = NoCell>
__device__ __forceinline__ bool cell_seek(const FieldDev &f, R r, R th, R ph, uint32_t gl, CellPos<R> &at, Cell &cell,
                                          const FieldDev &fx, More &more) {
    const R x = (r - (R)f.r_min) * (R)f.inv_dr;
    const R y = th * (R)f.inv_dth - (R)0.5;
    const R z = ph * (R)f.inv_dph;
    // x - fi is exact when fi = floor(x), unless it rounds to 1, and then, as for
    // a clamped stencil, the test fails and gather_plan's own weights are taken
    at.wr = x - at.fi;
    at.wt = y - at.fj;
    at.wp = z - at.zf;
    if (rare(!in_unit(at.wr, at.wt, at.wp))) {
        GatherPlan<R> gp;
        if (!gather_plan<FDT>(f, r, th, ph, gp)) return false;
        at.fi = clampr(floor(x), (R)0, (R)(f.nr - 2));
        at.fj = clampr(floor(y), (R)0, (R)(f.nth - 2));
        at.zf = floor(z);
        at.wr = clampr(x - at.fi, (R)0, (R)1);
        at.wt = clampr(y - at.fj, (R)0, (R)1);
        at.wp = z - at.zf;
        cell.load(f, gp, gl);
        more.load(fx, gp, gl);
    }
    return true;
}

// ---------------------------------------------------------------------------
// Reciprocal, inverse square root and sine for the right-hand side.
// Hardware estimates refined by Newton steps (two in double, one in float:
// each step doubles the correct bits), faithful to about one ulp for the
// normal, finite arguments met here.  sin on [0, pi] (theta of a particle
// inside the grid) folds to [0, pi/4] and sums the Taylor series of sin or
// cos up to the z^17 / z^16 term (truncation below 1e-19).
// ---------------------------------------------------------------------------
__device__ __forceinline__ double rcp_nr(double x) {
    double r = __builtin_amdgcn_rcp(x);
    double e = fma(-x, r, 1.0);
    r = fma(r, e, r);
    e = fma(-x, r, 1.0);
    return fma(r, e, r);
}
__device__ __forceinline__ float rcp_nr(float x) {
    const float r = __builtin_amdgcn_rcpf(x);
    return fmaf(r, fmaf(-x, r, 1.0f), r);
}
__device__ __forceinline__ double rsqrt_nr(double x) {
    double y = __builtin_amdgcn_rsq(x);
    const double hx = 0.5 * x;
    y = y * fma(-hx, y * y, 1.5);
    return y * fma(-hx, y * y, 1.5);
}
__device__ __forceinline__ float rsqrt_nr(float x) {
    const float y = __builtin_amdgcn_rsqf(x);
    return y * fmaf(-0.5f * x, y * y, 1.5f);
}

// A constant held in scalar registers (an FP64 multiply-add takes no literal,
// and the compiler would keep the series coefficients in vector registers).
__device__ __forceinline__ double scalar_const(double c) {
    asm("" : "+s"(c));
    return c;
}
__device__ __forceinline__ float scalar_const(float c) { return c; }

template <typename R>
__device__ __forceinline__ R sin_0_pi(R x) {
    const R half_pi = (R)1.5707963267948966, pi = (R)3.141592653589793, quarter_pi = (R)0.7853981633974483;
    const R y = x > half_pi ? pi - x : x;            // sin(x) = sin(pi - x)
    const bool use_cos = y > quarter_pi;
    const R z = use_cos ? half_pi - y : y;           // sin(y) = cos(pi/2 - y)
    const R z2 = z * z;
    // One series per lane, behind a branch: the particles of a wavefront are
    // binned by cell, so nearly always all of its lanes take the same one.
    if (!rare(!use_cos)) {
        // cos z = 1 - z^2/2! + z^4/4! - ... + z^16/16!
        R pc = scalar_const((R)(1.0 / 20922789888000.0));
        pc = fma(pc, -z2, scalar_const((R)(1.0 / 87178291200.0)));
        pc = fma(pc, -z2, scalar_const((R)(1.0 / 479001600.0)));
        pc = fma(pc, -z2, scalar_const((R)(1.0 / 3628800.0)));
        pc = fma(pc, -z2, scalar_const((R)(1.0 / 40320.0)));
        pc = fma(pc, -z2, scalar_const((R)(1.0 / 720.0)));
        pc = fma(pc, -z2, scalar_const((R)(1.0 / 24.0)));
        pc = fma(pc, -z2, (R)0.5);
        return fma(pc, -z2, (R)1);
    }
    // sin z = z (1 - z^2/3! + z^4/5! - ... + z^16/17!)
    R ps = scalar_const((R)(1.0 / 355687428096000.0));
    ps = fma(ps, -z2, scalar_const((R)(1.0 / 1307674368000.0)));
    ps = fma(ps, -z2, scalar_const((R)(1.0 / 6227020800.0)));
    ps = fma(ps, -z2, scalar_const((R)(1.0 / 39916800.0)));
    ps = fma(ps, -z2, scalar_const((R)(1.0 / 362880.0)));
    ps = fma(ps, -z2, scalar_const((R)(1.0 / 5040.0)));
    ps = fma(ps, -z2, scalar_const((R)(1.0 / 120.0)));
    ps = fma(ps, -z2, scalar_const((R)(1.0 / 6.0)));
    ps = fma(ps, -z2, (R)1);
    return z * ps;
}

// ---------------------------------------------------------------------------
// Guiding-centre right-hand side, Eqs. (1)-(2), reduced to the terms the
// twelve gridded components determine (b, E, grad|B|, (b.grad)b):
//   gamma = sqrt(1 + (u^2 + 2 mu B)/c^2)      (mu = mu_B / m, u = gamma v_par)
//   dR/dt = v_par b + v_E + (gamma/(q/m B)) b x a,
//   a     = (mu/gamma^2) grad B + ((q/m) v_par E_par/(gamma c^2)) v_E + v_par^2 (b.grad)b
//   du/dt = (q/m) E_par - (mu/gamma) b.grad B + gamma v_par v_E.(b.grad)b
// drift-free form (only v_par b kept): dR/dt = v_par b, du/dt without the v_E term.
// Output: coordinate rates (dr/dt, dth/dt, dph/dt, du/dt) and v_par.
// kFull: the full Eqs. 1-2, x = (v_E.grad)b, (b.grad)v_E, (v_E.grad)v_E at the
// point: v_par (x0..2 + x3..5) + x6..8 joins the bracket of dR/dt and
// gamma v_E.x0..2 joins du/dt.
// ---------------------------------------------------------------------------
// ir, is: 1/r and 1/sin(th), which the caller may compute while the field at the
// point is still on its way.
template <typename R, bool kFull = false>
__device__ __forceinline__ void gc_rhs_at(R ir, R is, R u, R mu, R qm, R iqm, bool drift_free,
                                          const R g[12], R F[4], R &vpar, const R *x = nullptr) {
    const R Bx = g[0], By = g[1], Bz = g[2];
    const R Ex = g[3], Ey = g[4], Ez = g[5];
    const R Gx = g[6], Gy = g[7], Gz = g[8];
    const R Kx = g[9], Ky = g[10], Kz = g[11];
    const R B2 = Bx * Bx + By * By + Bz * Bz;
    const R iB = rsqrt_nr(B2);
    const R B = B2 * iB;
    const R bx = Bx * iB, by = By * iB, bz = Bz * iB;
    const R g2 = (R)1 + (u * u + (R)2 * mu * B) * (R)kInvC2;
    const R ig = rsqrt_nr(g2);
    const R gamma = g2 * ig;
    vpar = u * ig;
    const R Epar = Ex * bx + Ey * by + Ez * bz;
    const R vEx = (Ey * bz - Ez * by) * iB;
    const R vEy = (Ez * bx - Ex * bz) * iB;
    const R vEz = (Ex * by - Ey * bx) * iB;
    const R bG = bx * Gx + by * Gy + bz * Gz;
    const R cG = mu * ig * ig;
    const R cE = qm * vpar * Epar * ig * (R)kInvC2;
    const R cK = vpar * vpar;
    R ax = cG * Gx + cE * vEx + cK * Kx;
    R ay = cG * Gy + cE * vEy + cK * Ky;
    R az = cG * Gz + cE * vEz + cK * Kz;
    if (kFull) {
        ax += vpar * (x[0] + x[3]) + x[6];
        ay += vpar * (x[1] + x[4]) + x[7];
        az += vpar * (x[2] + x[5]) + x[8];
    }
    const R pref = gamma * iqm * iB;
    R Vx = vpar * bx + vEx + pref * (by * az - bz * ay);
    R Vy = vpar * by + vEy + pref * (bz * ax - bx * az);
    R Vz = vpar * bz + vEz + pref * (bx * ay - by * ax);
    R udot = qm * Epar - mu * ig * bG + gamma * vpar * (vEx * Kx + vEy * Ky + vEz * Kz);
    if (kFull) udot += gamma * (vEx * x[0] + vEy * x[1] + vEz * x[2]);
    if (rare(drift_free)) {
        Vx = vpar * bx; Vy = vpar * by; Vz = vpar * bz;
        udot = qm * Epar - mu * ig * bG;
    }
    F[0] = Vx;
    F[1] = Vy * ir;
    F[2] = Vz * ir * is;
    F[3] = udot;
}
template <typename R>
__device__ __forceinline__ void gc_rhs(R r, R th, R u, R mu, R qm, R iqm, bool drift_free, const R g[12], R F[4],
                                       R &vpar) {
    gc_rhs_at<R>(rcp_nr(r), rcp_nr(sin_0_pi(th)), u, mu, qm, iqm, drift_free, g, F, vpar);
}

}  // namespace gc
