// gc_order.hip -- particle reordering between chunks of steps.
//
//  * cell binning: key = field cell of the particle (optionally coarsened),
//    inactive particles get the largest key; LSD radix sort of (key, slot)
//    pairs; permute the state (for the grid push, only the particles stopped
//    since the last reorder, by the sort's last pass: the push applies the
//    permutation to the others as it reads them).  Particles of one cell then
//    sit in consecutive lanes, so their trilinear gathers hit the same cache
//    lines.
//    Up to a tile one workgroup does it all.  Past that the key kernel also
//    counts the digits of every pass; each pass is then one kernel that ranks
//    its tile, finds the tile's offset per digit by looking back over the
//    tiles before it, and scatters.
//  * compaction: stable partition active-first from wavefront ballots.
// Both produce perm[dst] = src and leave the active count on the device.
#include <hip/hip_runtime.h>

#include "gc_device.h"
#include "gc_launch.h"

namespace gc {

// A sort tile is one workgroup of sixteen wavefronts, 4,096 particles: four
// items per lane keep each wavefront's serial part (the rank of one item waits
// for the counts of the one before) short, and halve the tiles a look-back
// passes against 2,048.
constexpr int kRsThreads = 1024;
constexpr int kRsItems = kSortTile / kRsThreads;   // items per thread per tile
constexpr int kWaves = kRsThreads / 64;
constexpr int kLook = 8;                           // look-back words in flight

__device__ __forceinline__ uint64_t lanemask_lt() {
    const uint32_t lane = threadIdx.x & 63u;
    return lane == 0 ? 0ull : (~0ull >> (64 - lane));
}

__device__ __forceinline__ uint32_t cell_key(const FieldDev &f, double r, double th, double ph, int coarsen) {
    const double x = (r - f.r_min) * f.inv_dr;
    const double y = th * f.inv_dth - 0.5;
    const double z = ph * f.inv_dph;
    double fi = clampr(floor(x), 0.0, (double)(f.nr - 2));
    double fj = clampr(floor(y), 0.0, (double)(f.nth - 2));
    double zf = floor(z);
    double km = zf - (double)f.nph * floor(zf * f.inv_nph);
    km = km < 0.0 ? km + f.nph : km;
    km = km >= f.nph ? km - f.nph : km;
    km = clampr(km, 0.0, (double)(f.nph - 1));
    if (!(isfinite(x) && isfinite(y) && isfinite(z))) { fi = 0.0; fj = 0.0; km = 0.0; }
    const uint32_t nthc = ((uint32_t)f.nth + (1u << coarsen) - 1) >> coarsen;
    const uint32_t nphc = ((uint32_t)f.nph + (1u << coarsen) - 1) >> coarsen;
    return (((uint32_t)fi >> coarsen) * nthc + ((uint32_t)fj >> coarsen)) * nphc + ((uint32_t)km >> coarsen);
}

// lanes of the wavefront whose valid digit of kBits equals this lane's
template <int kBits>
__device__ __forceinline__ uint64_t same_digit(uint32_t d, bool valid) {
    uint64_t same = __ballot(valid);
#pragma unroll
    for (int b = 0; b < kBits; ++b) {
        const uint64_t bb = __ballot((d >> b) & 1u);
        same &= ((d >> b) & 1u) ? bb : ~bb;
    }
    return same;
}

// Keys of a lane's items first + 64 * it (it < items, slots below n <= n_max,
// n_max > 0 slots exist), all ones past n, and the wavefront's active particles.
// Every load is in flight before the first is used, and none waits for n: item
// after item the kernel waited for memory eight times (16 us for 300,000
// particles, now 8).
__device__ __forceinline__ uint32_t item_keys(const SoA &st, const FieldDev &f, uint32_t first, uint32_t n,
                                              uint32_t n_max, int items, int coarsen, uint32_t dead_key,
                                              uint32_t *key) {
    uint32_t status[kRsItems];
    double r[kRsItems], th[kRsItems], ph[kRsItems];
#pragma unroll
    for (int it = 0; it < kRsItems; ++it) {
        const uint32_t i = first + 64u * it;
        const uint32_t j = it < items && i < n_max ? i : 0u;
        status[it] = st.status[j];
        r[it] = st.r[j];
        th[it] = st.th[j];
        ph[it] = st.ph[j];
    }
    uint32_t alive_n = 0;
#pragma unroll
    for (int it = 0; it < kRsItems; ++it) {
        const bool valid = it < items && first + 64u * it < n, alive = valid && status[it] == GC_ACTIVE;
        const uint32_t k = cell_key(f, r[it], th[it], ph[it], coarsen);
        key[it] = alive ? k : valid ? dead_key : 0xFFFFFFFFu;
        alive_n += (uint32_t)__popcll(__ballot(alive));
    }
    return alive_n;
}

// Keys of the live prefix, one sort tile per workgroup; the digit counts of
// every pass and the number of active particles are added to the sort state
// (which the end of the previous reorder left at zero).  Neighbouring slots
// mostly share their digits (the order decays slowly), so a run of equal
// digits adds its length once.
__global__ __launch_bounds__(kRsThreads) void k_cell_keys(SoA st, FieldDev f, const uint32_t *np, uint32_t n_max,
                                                         int coarsen, uint32_t dead_key, int passes, uint32_t *keys,
                                                         uint32_t *state, uint32_t *sorted_n) {
    __shared__ uint32_t h[kMaxPasses][256];
    __shared__ uint32_t s_alive;
    const uint32_t n = *np, tid = threadIdx.x, lane = tid & 63u;
    if (blockIdx.x == 0 && tid == 0) *sorted_n = n;
    if (blockIdx.x * kSortTile >= n) return;   // tile past the live prefix (uniform)
    h[tid >> 8][tid & 255u] = 0;
    if (tid == 0) s_alive = 0;
    static_assert(kMaxPasses * 256 == kRsThreads, "one digit count per thread");
    __syncthreads();
    const uint32_t first = blockIdx.x * kSortTile + (tid >> 6) * (64u * kRsItems) + lane;
    uint32_t key[kRsItems];
    const uint32_t alive_n = item_keys(st, f, first, n, n_max, kRsItems, coarsen, dead_key, key);
#pragma unroll
    for (int it = 0; it < kRsItems; ++it) {
        const uint32_t i = first + 64u * it;
        const bool valid = i < n;
        if (valid) keys[i] = key[it];
        const uint32_t nvalid = (uint32_t)__popcll(__ballot(valid));   // (the first lanes)
        const uint32_t before = __shfl_up(key[it], 1);
        for (int p = 0; p < passes; ++p) {
            const uint32_t d = (key[it] >> (8 * p)) & 255u;
            const bool head = lane == 0 || d != ((before >> (8 * p)) & 255u);
            const uint64_t heads = __ballot(head);
            const uint64_t later = heads & ~(lanemask_lt() | 1ull << lane);
            const uint32_t end = later ? (uint32_t)__builtin_ctzll(later) : 64u;
            if (valid && head) atomicAdd(&h[p][d], (end < nvalid ? end : nvalid) - lane);
        }
    }
    if (lane == 0 && alive_n) atomicAdd(&s_alive, alive_n);
    __syncthreads();
    const uint32_t c = h[tid >> 8][tid & 255u];
    if (c) atomicAdd(&state[kStHist + tid], c);
    if (tid == 0 && s_alive) atomicAdd(&state[kStAlive], s_alive);
}

// Ranks of a lane's items among the equal digits before them in the wavefront's
// items (item after item, lane after lane), with cnt[1 << kBits], this
// wavefront's counts, zero before and the totals after.
template <int kBits>
__device__ __forceinline__ void wave_ranks(const uint32_t *key, int shift, int items, uint32_t first, uint32_t n,
                                           uint32_t *cnt, uint32_t *rank) {
    const uint64_t lt = lanemask_lt();
    uint64_t same[kRsItems];
#pragma unroll
    for (int it = 0; it < kRsItems; ++it)
        if (it < items) same[it] = same_digit<kBits>((key[it] >> shift) & ((1u << kBits) - 1u), first + 64u * it < n);
#pragma unroll
    for (int it = 0; it < kRsItems; ++it) {
        if (it >= items) break;
        const uint32_t d = (key[it] >> shift) & ((1u << kBits) - 1u);
        const uint32_t seen = cnt[d];
        rank[it] = seen + (uint32_t)__popcll(same[it] & lt);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        if (first + 64u * it < n && (same[it] & lt) == 0) cnt[d] = seen + (uint32_t)__popcll(same[it]);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
}

// inclusive sum over the lanes of the wavefront
__device__ __forceinline__ uint32_t wave_scan(uint32_t v) {
    const uint32_t lane = threadIdx.x & 63u;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t t = __shfl_up(v, off);
        v += lane >= (uint32_t)off ? t : 0u;
    }
    return v;
}

// offsets of each wavefront's items of one digit, in place of their counts;
// returns the tile's count
template <int kBins>
__device__ __forceinline__ uint32_t wave_offsets(uint32_t (*wcnt)[kBins], uint32_t digit) {
    uint32_t c[kWaves], count = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) c[w] = wcnt[w][digit];
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        wcnt[w][digit] = count;
        count += c[w];
    }
    return count;
}

// one particle from slot j of src to slot i of dst: every load before the first
// store (the arrays may alias as far as the compiler knows, and copied one
// after the other each would wait for the one before)
__device__ __forceinline__ void move_particle(const SoA &src, const SoA &dst, uint32_t j, uint32_t i, bool comp) {
#define EACH_(X) X(r) X(th) X(ph) X(u) X(mu) X(fr) X(fth) X(fph) X(fu) X(dtp) X(s) X(ell) X(t) \
    X(k) X(flags) X(status) X(step) X(id) X(ens) X(gid) X(birth)
#define LOAD_(name) const auto v_##name = src.name[j];
#define STORE_(name) dst.name[i] = v_##name;
    EACH_(LOAD_)
    EACH_(STORE_)
    if (comp) {
#define COMP_(X) X(cr) X(cth) X(cph) X(cu) X(ct)
        COMP_(LOAD_)
        COMP_(STORE_)
    }
#undef COMP_
#undef STORE_
#undef LOAD_
#undef EACH_
}

// ---------------------------------------------------------------------------
// At most one tile: keys, every pass and the move of the stopped particles in
// one workgroup, the pairs in LDS between the passes.  Small sets are bound by
// the round trips of each kernel and the launches between them, not by work:
// 9 us for 1,000 particles against 34 of the key kernel, three passes and the
// move below.  Past a tile one workgroup has more than four items per lane to
// rank in turn, and the kernels below take 34 us at 20,000.
// ---------------------------------------------------------------------------
template <int kBits>
__global__ __launch_bounds__(kRsThreads) void k_sort_one(SoA st, FieldDev f, const uint32_t *np, uint32_t n_max,
                                                        int coarsen, uint32_t dead_key, int passes,
                                                        uint32_t *keys_out, uint32_t *vals_out, uint32_t *n_active,
                                                        uint32_t *sorted_n, bool move, bool comp, SoA dst) {
    constexpr uint32_t kBins = 1u << kBits, kMask = kBins - 1u;
    __shared__ uint32_t wcnt[kWaves][kBins];
    __shared__ uint32_t s_key[kSortTile], s_val[kSortTile];
    __shared__ uint32_t s_base[kBins], s_wave[kBins / 64], s_alive;
    const uint32_t tid = threadIdx.x, wave = tid >> 6, lane = tid & 63u;
    const int items = (int)((n_max + kRsThreads - 1) / kRsThreads);   // (n_max <= kSortTile)
    const uint32_t first = wave * 64u * (uint32_t)items + lane;
    const uint32_t n = *np;                                            // (<= n_max)
    if (tid == 0) s_alive = 0;
    __syncthreads();
    uint32_t key[kRsItems], val[kRsItems], rank[kRsItems];
    const uint32_t alive_n = item_keys(st, f, first, n, n_max, items, coarsen, dead_key, key);
    if (lane == 0 && alive_n) atomicAdd(&s_alive, alive_n);
#pragma unroll
    for (int it = 0; it < kRsItems; ++it) val[it] = first + 64u * it;
    for (int p = 0; p < passes; ++p) {
        const int shift = kBits * p;
#pragma unroll
        for (uint32_t q = 0; q < kBins; q += 64) wcnt[wave][q + lane] = 0;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        wave_ranks<kBits>(key, shift, items, first, n, wcnt[wave], rank);
        __syncthreads();
        if (tid < kBins) {
            const uint32_t count = wave_offsets<kBins>(wcnt, tid), upto = wave_scan(count);
            if (lane == 63u) s_wave[wave] = upto;
            s_base[tid] = upto - count;
        }
        __syncthreads();
        uint32_t tot[kBins / 64];
#pragma unroll
        for (uint32_t w = 0; w < kBins / 64; ++w) tot[w] = s_wave[w];
#pragma unroll
        for (int it = 0; it < kRsItems; ++it) {
            if (it < items && first + 64u * it < n) {
                const uint32_t d = (key[it] >> shift) & kMask;
                uint32_t pos = s_base[d] + wcnt[wave][d] + rank[it];   // (a permutation of [0, n))
#pragma unroll
                for (uint32_t w = 0; w < kBins / 64 - 1; ++w) pos += (d >> 6) > w ? tot[w] : 0u;
                s_key[pos] = key[it];
                s_val[pos] = val[it];
            }
        }
        __syncthreads();
#pragma unroll
        for (int it = 0; it < kRsItems; ++it) {
            if (it < items && first + 64u * it < n) {
                key[it] = s_key[first + 64u * it];
                val[it] = s_val[first + 64u * it];
            }
        }
    }
    const uint32_t alive = s_alive;
    if (tid == 0) {
        *n_active = alive;
        *sorted_n = n;
    }
#pragma unroll
    for (int it = 0; it < kRsItems; ++it) {
        const uint32_t i = first + 64u * it;
        if (it < items && i < n) {
            keys_out[i] = key[it];
            vals_out[i] = val[it];
            if (move && i >= alive) move_particle(st, dst, val[it], i, comp);
        }
    }
}

// ---------------------------------------------------------------------------
// More than one tile: LSD radix sort, one 8-bit digit per pass, one kernel per
// pass.  A workgroup takes the next tile in start order from a ticket counter,
// ranks its items stably (per wavefront by ballots, then across wavefronts in
// LDS) and publishes its count per digit.  Its offset per digit among the
// tiles before it comes from looking back over their published words, kLook of
// them in flight: an inclusive prefix ends the walk, an aggregate adds to it
// and the walk goes on.  A tile waits only for tiles that took their tickets
// before it and so are already running; each publishes its aggregate before it
// waits itself, so every wait ends.  Look-back words carry a tag (reorder epoch
// and pass), so words of earlier passes read as not yet published and the array
// never needs clearing; the tag repeats after 2^28 reorders.
// The last pass also moves the stopped particles (move set): they end in the
// slots past the active ones.  A pass is a chain of round trips (count,
// ticket, look-back) more than traffic: with the items loaded before the ticket
// is known, 1,024 threads a tile and eight look-back words in flight it takes
// 9 us at 20,000 particles, 13 at 300,000 and 25 at 2^20 (11, 17 and 30 with
// tiles of 2,048 by 256 threads and one word in flight; sixteen words: 10, 13
// and 26).
// ---------------------------------------------------------------------------
constexpr uint32_t kFlagAgg = 1, kFlagPrefix = 2;
constexpr uint32_t kSpinLimit = 1u << 22;

__device__ __forceinline__ unsigned long long look_word(uint32_t tag, uint32_t flag, uint32_t v) {
    return ((unsigned long long)(tag & 0x3FFFFFFFu) << 34) | ((unsigned long long)flag << 32) | v;
}

// sum of one digit's counts over the tiles before `tile`
__device__ __forceinline__ uint32_t look_back(const unsigned long long *look, uint32_t tile, uint32_t digit,
                                              uint32_t tag, uint32_t *state) {
    const unsigned long long want = (unsigned long long)(tag & 0x3FFFFFFFu);
    uint32_t prefix = 0, spins = 0;
    uint32_t left = tile;                          // tiles [0, left) not added yet
    while (left > 0) {
        unsigned long long w[kLook];
#pragma unroll
        for (int q = 0; q < kLook; ++q) {
            const uint32_t j = left > (uint32_t)q ? left - 1 - q : 0u;
            w[q] = __hip_atomic_load(look + (size_t)j * 256 + digit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        uint32_t got = 0;
        bool open = true;                          // no prefix and no unpublished word yet
#pragma unroll
        for (int q = 0; q < kLook; ++q) {
            const uint32_t flag = (uint32_t)(w[q] >> 32) & 3u;
            const bool ready = (w[q] >> 34) == want && flag != 0;
            if (open && ready && left > (uint32_t)q) {
                prefix += (uint32_t)w[q];
                ++got;
                if (flag == kFlagPrefix) {
                    got = left;
                    open = false;
                }
            } else {
                open = false;
            }
        }
        left -= got;
        if (got == 0) {
            if (++spins > kSpinLimit) {
                atomicOr(&state[kStError], 1u);    // reported by the next synchronizing call
                break;
            }
            __builtin_amdgcn_s_sleep(1);
        }
    }
    return prefix;
}

__global__ __launch_bounds__(kRsThreads) void k_rs_pass(const uint32_t *keys_in, const uint32_t *vals_in,
                                                       uint32_t *keys_out, uint32_t *vals_out, const uint32_t *np,
                                                       uint32_t n_max, int pass, uint32_t *state,
                                                       unsigned long long *look, uint32_t *n_active, bool move,
                                                       bool comp, SoA src, SoA dst) {
    __shared__ uint32_t s_tile;
    __shared__ uint32_t wcnt[kWaves][256];   // per (wave, digit): count, then offset in the tile
    __shared__ uint32_t s_base[256], s_wave[4];
    const uint32_t tid = threadIdx.x, wave = tid >> 6, lane = tid & 63u;
    const uint32_t n = *np;
    // the items of tile blockIdx.x, which mostly is the one its ticket gives:
    // their loads wait for neither the count nor the ticket
    uint32_t key[kRsItems], val[kRsItems], rank[kRsItems];
    uint32_t first = blockIdx.x * kSortTile + wave * (64u * kRsItems) + lane;
#pragma unroll
    for (int it = 0; it < kRsItems; ++it) {
        const uint32_t j = first + 64u * it < n_max ? first + 64u * it : 0u;
        key[it] = keys_in[j];
        val[it] = vals_in ? vals_in[j] : j;
    }
    // Only the first ceil(n / kSortTile) workgroups take tickets, so the tiles
    // of the live prefix are taken once each, in start order; the others leave
    // at once (workgroup 0 then publishes the active count of an empty prefix).
    if (blockIdx.x * kSortTile >= n) {
        if (pass == 0 && blockIdx.x == 0 && tid == 0) *n_active = state[kStAlive];
        return;
    }
    const uint32_t alive = state[kStAlive];
    const uint32_t tag = (state[kStEpoch] + 1u) * 4u + (uint32_t)pass;
    if (tid == 0) {
        s_tile = n > (uint32_t)kSortTile ? atomicAdd(&state[kStTicket + pass], 1u) : 0u;
        if (pass == 0 && s_tile == 0) *n_active = alive;
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) wcnt[wave][64 * q + lane] = 0;
    __syncthreads();
    const uint32_t tile = s_tile;
    const int shift = 8 * pass;
    if (tile != blockIdx.x) {
        first = tile * kSortTile + wave * (64u * kRsItems) + lane;
#pragma unroll
        for (int it = 0; it < kRsItems; ++it) {
            const uint32_t j = first + 64u * it < n ? first + 64u * it : 0u;
            key[it] = keys_in[j];
            val[it] = vals_in ? vals_in[j] : j;
        }
    }
    // global start of each digit: exclusive sums of this pass's digit totals,
    // by the four wavefronts that own no digit of the look-back
    if (tid >= 256 && tid < 512) {
        const uint32_t tot = state[kStHist + pass * 256 + (tid - 256)], upto = wave_scan(tot);
        if (lane == 63u) s_wave[wave - 4] = upto;
        s_base[tid - 256] = upto - tot;
    }
    wave_ranks<8>(key, shift, kRsItems, first, n, wcnt[wave], rank);
    __syncthreads();
    if (tid < 256) {   // thread tid owns digit tid
        const uint32_t count = wave_offsets<256>(wcnt, tid);
        unsigned long long *mine = look + (size_t)tile * 256 + tid;
        __hip_atomic_store(mine, look_word(tag, tile == 0 ? kFlagPrefix : kFlagAgg, count), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
        uint32_t start = s_base[tid];
        for (uint32_t w = 0; w < wave; ++w) start += s_wave[w];
        if (tile > 0) {
            const uint32_t prefix = look_back(look, tile, tid, tag, state);
            __hip_atomic_store(mine, look_word(tag, kFlagPrefix, prefix + count), __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
            start += prefix;
        }
        s_base[tid] = start;
    }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < kRsItems; ++it) {
        if (first + 64u * it < n) {
            const uint32_t d = (key[it] >> shift) & 255u;
            const uint32_t pos = s_base[d] + wcnt[wave][d] + rank[it];
            if (pos < n) {   // always, with digit counts of these keys
                keys_out[pos] = key[it];
                vals_out[pos] = val[it];
                if (move && pos >= alive) move_particle(src, dst, val[it], pos, comp);
            }
        }
    }
}

hipError_t launch_cell_sort(const SoA &st, const FieldDev &f, const uint32_t *np, uint32_t n_max, int coarsen,
                            uint32_t dead_key, int bits, OrderScratch &sc, uint32_t *n_active, uint32_t *sorted_n,
                            const SoA *stopped, bool with_comp, uint32_t **perm_out, hipStream_t s,
                            hipEvent_t start) {
    const int passes = (bits + 7) / 8;
    const uint32_t nb = (n_max + kSortTile - 1) / kSortTile;
    if (passes > kMaxPasses || nb > sc.max_blocks) return hipErrorInvalidValue;
    int cur = 0;
    const SoA dst = stopped ? *stopped : st;
    if (n_max == 0) {
        if (start) (void)hipEventRecord(start, s);
        const hipError_t e = launch_fill_u32(n_active, 0u, 1, s);
        if (e != hipSuccess) return e;
        const hipError_t e2 = launch_fill_u32(sorted_n, 0u, 1, s);
        if (e2 != hipSuccess) return e2;
    } else if (nb == 1) {
        cur = 1;
        // nine bits a pass where they save one (a grid of 2^16 cells: 17 bits)
        const int wide = (bits + 8) / 9;
        launch_timed(wide < passes ? k_sort_one<9> : k_sort_one<8>, dim3(1), dim3(kRsThreads), s, start, nullptr, st,
                     f, np, n_max, coarsen, dead_key, wide < passes ? wide : passes, sc.keys[1], sc.vals[1], n_active,
                     sorted_n, stopped != nullptr, with_comp, dst);
    } else {
        launch_timed(k_cell_keys, dim3(nb), dim3(kRsThreads), s, start, nullptr, st, f, np, n_max, coarsen, dead_key,
                     passes, sc.keys[0], sc.state, sorted_n);
        const uint32_t *vals_in = nullptr;
        for (int p = 0; p < passes; ++p) {
            hipLaunchKernelGGL(k_rs_pass, dim3(nb), dim3(kRsThreads), 0, s, sc.keys[cur], vals_in, sc.keys[cur ^ 1],
                               sc.vals[cur ^ 1], np, n_max, p, sc.state, sc.look, n_active,
                               stopped != nullptr && p == passes - 1, with_comp, st, dst);
            vals_in = sc.vals[cur ^ 1];
            cur ^= 1;
        }
    }
    *perm_out = sc.vals[cur];
    sc.sorted_keys = sc.keys[cur];
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Compaction: stable partition (active first) from wavefront ballots.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_compact_count(const uint32_t *status, const uint32_t *np,
                                                       uint32_t *block_alive) {
    __shared__ uint32_t wsum[4];
    const uint32_t n = *np;
    const uint32_t i = blockIdx.x * 256 + threadIdx.x;
    const bool alive = i < n && status[i] == GC_ACTIVE;
    const uint64_t b = __ballot(alive);
    if ((threadIdx.x & 63u) == 0) wsum[threadIdx.x >> 6] = (uint32_t)__popcll(b);
    __syncthreads();
    if (threadIdx.x == 0) block_alive[blockIdx.x] = wsum[0] + wsum[1] + wsum[2] + wsum[3];
}

// single workgroup: exclusive scan of the per-block counts, total -> n_active
__global__ __launch_bounds__(1024) void k_scan_blocks(uint32_t *v, uint32_t nb, const uint32_t *np, uint32_t *n_active,
                                                      uint32_t *sorted_n) {
    __shared__ uint32_t sh[1024];
    uint32_t carry = 0;
    for (uint32_t base = 0; base < nb; base += 1024) {
        const uint32_t i = base + threadIdx.x;
        const uint32_t x = i < nb ? v[i] : 0u;
        sh[threadIdx.x] = x;
        __syncthreads();
        for (int off = 1; off < 1024; off <<= 1) {
            const uint32_t t = threadIdx.x >= (uint32_t)off ? sh[threadIdx.x - off] : 0u;
            __syncthreads();
            sh[threadIdx.x] += t;
            __syncthreads();
        }
        if (i < nb) v[i] = carry + sh[threadIdx.x] - x;
        carry += sh[1023];
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        *n_active = carry;
        *sorted_n = *np;
    }
}

__global__ __launch_bounds__(256) void k_compact_scatter(const uint32_t *status, const uint32_t *np,
                                                         const uint32_t *block_off, const uint32_t *n_active,
                                                         uint32_t *perm) {
    __shared__ uint32_t wsum[4];
    const uint32_t n = *np;
    const uint32_t i = blockIdx.x * 256 + threadIdx.x;
    const bool valid = i < n;
    const bool alive = valid && status[i] == GC_ACTIVE;
    const uint64_t b = __ballot(alive);
    const uint32_t w = threadIdx.x >> 6;
    if ((threadIdx.x & 63u) == 0) wsum[w] = (uint32_t)__popcll(b);
    __syncthreads();
    uint32_t before = block_off[blockIdx.x];
    for (uint32_t q = 0; q < w; ++q) before += wsum[q];
    before += (uint32_t)__popcll(b & lanemask_lt());     // active slots before i
    if (valid) {
        const uint32_t pos = alive ? before : *n_active + (i - before);
        perm[pos] = i;
    }
}

hipError_t launch_compact(const SoA &st, const uint32_t *np, uint32_t n_max, OrderScratch &sc, uint32_t *n_active,
                          uint32_t *sorted_n, uint32_t **perm_out, hipStream_t s, hipEvent_t start) {
    const uint32_t nb = (n_max + 255) / 256;
    if (nb == 0) {
        if (start) (void)hipEventRecord(start, s);
        const hipError_t e = launch_fill_u32(n_active, 0u, 1, s);
        return e != hipSuccess ? e : launch_fill_u32(sorted_n, 0u, 1, s);
    }
    if (nb > 256u * sc.max_blocks) return hipErrorInvalidValue;
    launch_timed(k_compact_count, dim3(nb), dim3(256), s, start, nullptr, st.status, np, sc.counts);
    hipLaunchKernelGGL(k_scan_blocks, dim3(1), dim3(1024), 0, s, sc.counts, nb, np, n_active,
                       sorted_n);
    hipLaunchKernelGGL(k_compact_scatter, dim3(nb), dim3(256), 0, s, st.status, np, sc.counts, n_active, sc.vals[0]);
    *perm_out = sc.vals[0];
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
__global__ void k_permute(SoA src, SoA dst, const uint32_t *perm, const uint32_t *lo, const uint32_t *hi,
                          bool with_comp) {
    const uint32_t i = (lo ? *lo : 0u) + blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= *hi) return;
    move_particle(src, dst, perm[i], i, with_comp);
}

hipError_t launch_permute(const SoA &src, const SoA &dst, const uint32_t *perm, const uint32_t *lo,
                          const uint32_t *hi, uint32_t n_max, bool with_comp, hipStream_t s) {
    if (n_max == 0) return hipSuccess;
    hipLaunchKernelGGL(k_permute, dim3((n_max + 255) / 256), dim3(256), 0, s, src, dst, perm, lo, hi, with_comp);
    return hipGetLastError();
}

// The sort state for the next reorder: no counts, no tickets, a new epoch (by
// one workgroup, after every kernel that reads it).
__device__ __forceinline__ void reset_sort(uint32_t *state) {
    const uint32_t tid = threadIdx.x;
    for (uint32_t i = tid; i < kMaxPasses * 256; i += blockDim.x) state[kStHist + i] = 0;
    if (tid < kMaxPasses) state[kStTicket + tid] = 0;
    if (tid == 0) {
        state[kStAlive] = 0;
        state[kStEpoch] += 1u;
    }
}

// The end of a reorder.  Both state buffers hold identical data for the dead
// tail: slots past the live prefix are never permuted again.  The particles
// that died since the last reorder (slots [*n_active, *sorted_n) of the new
// buffer) are copied back into the other buffer, which keeps the two in
// agreement on the tail, and workgroup 0 takes *n_active over as the live
// prefix (no workgroup of this kernel reads *n_bound) and resets the sort.
// Mostly few particles died, and the kernel is its launch and the word to the
// host (4 us; 9 when the count had a kernel of its own); with many, 1,024
// workgroups fill the machine.
__global__ __launch_bounds__(256) void k_end_reorder(SoA src, SoA dst, const uint32_t *n_active,
                                                     const uint32_t *sorted_n, bool with_comp,
                                                     unsigned long long *dead, uint32_t *n_bound,
                                                     volatile uint32_t *host_mirror, uint32_t *state) {
    __shared__ unsigned long long part[4][6];
    const uint32_t lo = *n_active, end = *sorted_n;
    if (blockIdx.x == 0) {
        reset_sort(state);
        if (threadIdx.x == 0) {
            *n_bound = lo;
            if (host_mirror) *host_mirror = lo;
        }
    }
    if (end <= lo || blockIdx.x * 256u >= end - lo) return;   // workgroup past the range (uniform)
    unsigned long long v[6] = {0, 0, 0, 0, 0, 0};
    for (uint32_t b0 = lo + blockIdx.x * 256u; b0 < end; b0 += gridDim.x * 256u) {
        const uint32_t i = b0 + threadIdx.x;
        const bool in = i < end;
        uint32_t status = 0xFFFFFFFFu;
        if (in) {
            move_particle(src, dst, i, i, with_comp);
            status = src.status[i];
            v[4] += src.k[i];
            v[5] += src.step[i];
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] += (unsigned long long)__popcll(__ballot(in && status == (uint32_t)q));
    }
    // the slots leave the live prefix for good: their sums join dead[], one
    // atomic per sum and workgroup
    for (int off = 32; off > 0; off >>= 1) {
        v[4] += __shfl_xor(v[4], off);
        v[5] += __shfl_xor(v[5], off);
    }
    const uint32_t wave = threadIdx.x >> 6;
    if ((threadIdx.x & 63u) == 0)
        for (int q = 0; q < 6; ++q) part[wave][q] = v[q];
    __syncthreads();
    if (threadIdx.x < 6) {
        const unsigned long long t = part[0][threadIdx.x] + part[1][threadIdx.x] + part[2][threadIdx.x] +
                                     part[3][threadIdx.x];
        if (t) atomicAdd(&dead[threadIdx.x], t);
    }
}

hipError_t launch_end_reorder(const SoA &src, const SoA &dst, const uint32_t *n_active, const uint32_t *sorted_n,
                              uint32_t n_max, bool with_comp, unsigned long long *dead, uint32_t *n_bound,
                              volatile uint32_t *host_mirror, uint32_t *state, hipStream_t s, hipEvent_t stop) {
    uint32_t nb = (n_max + 255) / 256;
    nb = nb < 1u ? 1u : nb > 1024u ? 1024u : nb;
    launch_timed(k_end_reorder, dim3(nb), dim3(256), s, nullptr, stop, src, dst, n_active, sorted_n, with_comp, dead,
                 n_bound, host_mirror, state);
    return hipGetLastError();
}

__global__ __launch_bounds__(256) void k_reset_sort(uint32_t *state) { reset_sort(state); }

hipError_t launch_reset_sort(uint32_t *state, hipStream_t s) {
    hipLaunchKernelGGL(k_reset_sort, dim3(1), dim3(256), 0, s, state);
    return hipGetLastError();
}

// Cell keys of the last sort in slot order: the sorted keys over the sorted
// prefix [0, *sorted_n), the inactive key past it.
__global__ void k_keys_out(const uint32_t *sorted_keys, const uint32_t *sorted_n, uint32_t dead_key, uint32_t n,
                           uint32_t *out) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    out[i] = i < *sorted_n ? sorted_keys[i] : dead_key;
}

hipError_t launch_keys_out(const uint32_t *sorted_keys, const uint32_t *sorted_n, uint32_t dead_key, uint32_t n,
                           uint32_t *out, hipStream_t s) {
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_keys_out, dim3((n + 255) / 256), dim3(256), 0, s, sorted_keys, sorted_n, dead_key, n, out);
    return hipGetLastError();
}

__global__ void k_set_count(uint32_t *p, uint32_t v) { *p = v; }

__global__ void k_reset_bound(uint32_t *n_bound, uint32_t n, unsigned long long *dead) {
    if (threadIdx.x == 0) *n_bound = n;
    if (threadIdx.x < 6) dead[threadIdx.x] = 0;
}

hipError_t launch_reset_bound(uint32_t *n_bound, uint32_t n, unsigned long long *dead, hipStream_t s) {
    hipLaunchKernelGGL(k_reset_bound, dim3(1), dim3(64), 0, s, n_bound, n, dead);
    return hipGetLastError();
}

hipError_t launch_set_count(uint32_t *n_active, uint32_t n, hipStream_t s) {
    hipLaunchKernelGGL(k_set_count, dim3(1), dim3(1), 0, s, n_active, n);
    return hipGetLastError();
}

}  // namespace gc
