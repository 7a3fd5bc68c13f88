// gc_mlp.hip -- neural field: training (forward, loss, backward, Adam) with
// BF16 MFMA matrix products and FP32 accumulation/master weights; point
// evaluation of the neural field and of the trilinear grid (its judge).
#include <hip/hip_runtime.h>

#include "gc_device.h"
#include "gc_launch.h"
#include "gc_mlp.h"
#include "gc_mlp_launch.h"

namespace gc {

// ---------------------------------------------------------------------------
// Training step in four kernels:
//   k_mlp_train<false>  features and forward of a block of 64 rows: the outputs;
//   k_mlp_train<true>   loss and output gradient, the forward again (its
//                       pre-activations stay in registers) and the backward pass
//                       to every dZ, with the block's bias and output-layer sums;
//   k_mlp_wgrad         the hidden layers' weight gradients;
//   k_mlp_update        the remaining sums, Adam, the BF16 copies, the loss.
// The loss couples rows i and n + i of different blocks, hence two forward
// passes: the second costs less than writing the pre-activations and reading
// them back (50 MB at 16,384 rows).  A step of that size is 10 GFLOP, 8 us at the
// rate of a large BF16 product; as one kernel per layer and pass (43 launches,
// every activation, pre-activation and gradient through memory) it took 0.78 ms,
// of which 0.66 ms in kernels; now 15 + 34 + 17 + 5 us.
//
// Activations H_0..H_5 and gradients dZ_1..dZ_6 go to memory once, in BF16,
// transposed in tiles [block][layer][64 rows / 8][128 columns][8]: k_mlp_wgrad sums over
// rows and reads its operands, eight rows of a column, straight from there.  Rows
// past the last repeat it with a zero gradient.  Every FP32 sum over rows is taken
// in one order (blocks of 64 rows: even rows, odd rows; four interleaved chains
// over the blocks; weight gradients: groups of mlp_train_chunk rows, four
// interleaved chains over the groups), whatever the launch shapes.
// ---------------------------------------------------------------------------
constexpr int kTrainThreads = 512;
constexpr int kTrainPitch = kMlpWidth + 8;      // LDS row of a 64 x 128 BF16 matrix: 272 bytes, four banks a row
constexpr size_t kTileT = (size_t)kMlpWidth * kTrainRows;   // elements of a transposed tile
// Operand order of a matrix of n rows in memory: eight elements k of a row are 16
// bytes, and rows follow each other, so that a wavefront's operand loads (32 rows,
// 16 elements of each) are two runs of 512 bytes, and so are the stores of the
// transposed tiles (whose rows are columns here).  Row after row, every load touched
// 32 lines and used 32 bytes of each: at 16,384 rows k_mlp_wgrad 35 -> 17 us,
// k_mlp_train 24 -> 15 and 48 -> 34.
__host__ __device__ constexpr int operand_at(int n, int row, int k) { return ((k >> 3) * n + row) * 8 + (k & 7); }
__device__ __forceinline__ int tile_at(int r, int c) { return operand_at(kMlpWidth, c, r); }

// A wavefront owns one 32 x 32 tile of every 64 x 128 matrix (row half w / 4,
// columns 32 (w % 4)..): its slice of the weights comes from L2 straight into
// registers, one layer ahead; the pre-activations of its tile stay there (96
// registers) until the backward pass needs their slopes; the matrix itself goes
// round through LDS for the next product's rows.  v_mfma_f32_32x32x16_bf16, K in
// order.  Bound by the chain of 11 products, each an LDS round trip, eight
// dependent matrix instructions and a barrier.
template <bool kBack>
__global__ __launch_bounds__(kTrainThreads) __attribute__((amdgpu_waves_per_eu(2)))
void k_mlp_train(MlpArgs m, TrainNet net, const double *pts, const double *tgt, int npair, MlpLoss L, float *Y,
                 __bf16 *HT, __bf16 *DT, float *sums, double *loss_part) {
    __shared__ __bf16 X[2][kTrainRows * kTrainPitch];
    __shared__ float dYs[kBack ? kTrainRows : 1][8];
    __shared__ float Gs[kBack ? kTrainRows * kMlpWidth : 1], Ss[kBack ? kTrainRows * kMlpWidth : 1];   // dH, silu'(Z)
    __shared__ double red[kBack ? kTrainRows * kMlpOut : 1];
    __shared__ float odd[kBack ? kMlpOut * kMlpWidth + kMlpOut : 1];
    const int tid = threadIdx.x, l = tid & 63, w = tid >> 6, blk = blockIdx.x;
    const int half = l >> 5, lane = l & 31, rt = w >> 2, col = 32 * (w & 3) + lane;
    const int rows = 2 * npair, row0 = blk * kTrainRows;
    // operand fragment s of a matrix (row r, elements 16 s + 8 half ..): in LDS by rows
    // of `pitch`, in memory in operand order, n rows
    auto frag = [&](const __bf16 *base, size_t pitch, int r, int s) {
        return *reinterpret_cast<const bf16x8 *>(base + (size_t)r * pitch + 16 * s + 8 * half);
    };
    auto wfrag = [&](const __bf16 *base, int n, int r, int s) {
        return *reinterpret_cast<const bf16x8 *>(base + operand_at(n, r, 16 * s + 8 * half));
    };
    // row of accumulator element j within the block
    auto row_of = [&](int j) { return 32 * rt + (j / 4) * 8 + half * 4 + (j % 4); };
    auto tile_t = [&](__bf16 *base, int layer) { return base + ((size_t)blk * kMlpDepth + layer) * kTileT; };
    // a tile in BF16: into LDS by rows, and into its transposed tile
    auto put = [&](const float v[16], __bf16 *lds, __bf16 *T) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            __bf16 b[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) b[e] = (__bf16)v[4 * q + e];
            if (lds)
#pragma unroll
                for (int e = 0; e < 4; ++e) lds[row_of(4 * q + e) * kTrainPitch + col] = b[e];
            if (T) __builtin_memcpy(T + tile_at(row_of(4 * q), col), b, 8);
        }
    };
    bf16x8 bw[8];
#pragma unroll
    for (int s = 0; s < 8; ++s) bw[s] = wfrag(net.W, kMlpWidth, col, s);
    if constexpr (kBack) {
        if (tid < kTrainRows * kMlpOut) {               // loss and dY: one (row, output) each
            const int rl = tid / kMlpOut, c = tid % kMlpOut, r = row0 + rl, i = r < npair ? r : r - npair;
            double part = 0.0;
            float d = 0.0f;
            if (r < rows) {
                const double e1 = (double)m.scale[c] * pow((double)m.r_ref / pts[i], (double)m.power[c]);
                const double e2 = (double)m.scale[c] * pow((double)m.r_ref / pts[npair + i], (double)m.power[c]);
                const double t1 = tgt[(size_t)i * kMlpOut + c] / e1, t2 = tgt[(size_t)(npair + i) * kMlpOut + c] / e2;
                const double y1 = Y[(size_t)i * kMlpOut + c], y2 = Y[(size_t)(npair + i) * kMlpOut + c];
                const double d1 = y1 - t1, d12 = (y2 - y1) - (t2 - t1);
                if (r < npair) {
                    part = L.wc[c] * (d1 * d1 + L.beta * d12 * d12);
                    d = (float)((2.0 * L.wc[c] * d1 - 2.0 * L.beta * L.wc[c] * d12) / npair);
                } else {
                    d = (float)(2.0 * L.beta * L.wc[c] * d12 / npair);
                }
            }
            dYs[rl][c] = d;
            red[tid] = part;
        }
    }
    {   // features: phase tid % 64, eight rows
        const int j = l, r0 = 8 * w;
        __bf16 sc[2][8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int r = r0 + e, row = min(row0 + r, rows - 1);
            const float rt_ = (float)((pts[row] - (double)m.r_min) * (double)m.inv_rspan);
            const float tt = (float)(pts[(size_t)rows + row] * 0.3183098861837907);
            const float ph = (float)pts[2 * (size_t)rows + row];
            const float psi = 6.283185307179586f * (m.fa[j] * rt_ + m.fb[j] * tt) + m.fn[j] * ph;
            float sn, cs;
            __sincosf(psi, &sn, &cs);
            sc[0][e] = (__bf16)sn;
            sc[1][e] = (__bf16)cs;
            X[0][r * kTrainPitch + 2 * j] = sc[0][e];
            X[0][r * kTrainPitch + 2 * j + 1] = sc[1][e];
        }
        if constexpr (kBack) {
            __bf16 *T = tile_t(HT, 0);
            __builtin_memcpy(T + tile_at(r0, 2 * j), sc[0], 16);
            __builtin_memcpy(T + tile_at(r0, 2 * j + 1), sc[1], 16);
        }
    }
    float Z[kBack ? kMlpDepth : 1][16];
#pragma unroll
    for (int k = 0; k < kMlpDepth; ++k) {
        __syncthreads();                                // X[k & 1] holds H_k
        floatx16 acc = {};
#pragma unroll
        for (int s = 0; s < 8; ++s)
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag(X[k & 1], kTrainPitch, 32 * rt + lane, s), bw[s], acc, 0, 0, 0);
        const float bias = net.c[k * kMlpWidth + col];
        // the next product's weights: the next layer's; then the output layer's (one
        // 32-row tile), or the first of the backward pass
        const __bf16 *nw = k + 1 < kMlpDepth ? net.W + (size_t)(k + 1) * kMlpWidth * kMlpWidth
                           : kBack           ? net.WT + (size_t)k * kMlpWidth * kMlpWidth
                                             : net.Wo;
#pragma unroll
        for (int s = 0; s < 8; ++s)
            bw[s] = k + 1 < kMlpDepth || kBack ? wfrag(nw, kMlpWidth, col, s) : wfrag(nw, kMlpOutPad, lane, s);
        float h[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const float z = acc[j] + bias;
            if constexpr (kBack) Z[k][j] = z;
            h[j] = silu_f(z);
        }
        put(h, X[(k + 1) & 1], kBack && k + 1 < kMlpDepth ? tile_t(HT, k + 1) : nullptr);
    }
    __syncthreads();                                    // X[0] holds H_6
    if constexpr (!kBack) {
        if ((w & 3) == 0) {                             // outputs: 32 padded columns, two wavefronts
            floatx16 acc = {};
#pragma unroll
            for (int s = 0; s < 8; ++s)
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag(X[0], kTrainPitch, 32 * rt + lane, s), bw[s], acc, 0, 0, 0);
            if (lane < kMlpOut) {
                const float co = net.co[lane];
#pragma unroll
                for (int j = 0; j < 16; ++j)
                    if (row0 + row_of(j) < rows) Y[(size_t)(row0 + row_of(j)) * kMlpOut + lane] = acc[j] + co;
            }
        }
        return;
    }
    // column sums: thread (parity, k) adds the rows of its parity in order
    const int par = tid >> 7, kk = tid & (kMlpWidth - 1);
    float *out = sums + (size_t)blk * kTrainSums;       // bias gradients [6][128], dWo [6][128], dco [6]
    float ws[kMlpOut] = {}, wb[kMlpOut] = {};
    if (par < 2) {                                      // output layer: dWo[c][k] = sum_r dY[r][c] H6[r][k], dco
        for (int r = par; r < kTrainRows; r += 2) {
            const float h = (float)X[0][r * kTrainPitch + kk];
#pragma unroll
            for (int c = 0; c < kMlpOut; ++c) {
                ws[c] = fmaf(dYs[r][c], h, ws[c]);
                wb[c] += dYs[r][c];
            }
        }
        if (par == 1) {
#pragma unroll
            for (int c = 0; c < kMlpOut; ++c) {
                odd[c * kMlpWidth + kk] = ws[c];
                if (kk == 0) odd[kMlpOut * kMlpWidth + c] = wb[c];
            }
        }
    } else if (w == 7) {                                // the block's loss
        double v = 0.0;
        for (int q = l; q < kTrainRows * kMlpOut; q += 64) v += red[q];
        for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
        if (l == 0) loss_part[blk] = v / npair;
    }
    float dH[16];
    {   // dH6 = dY Wo (K = 6: plain FP32)
        float wo[kMlpOut];
#pragma unroll
        for (int c = 0; c < kMlpOut; ++c) wo[c] = net.Wo_master[c * kMlpWidth + col];
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            dH[j] = 0.0f;
#pragma unroll
            for (int c = 0; c < kMlpOut; ++c) dH[j] = fmaf(dYs[row_of(j)][c], wo[c], dH[j]);
        }
    }
    __syncthreads();
    if (par == 0) {
        constexpr int o = kMlpDepth * kMlpWidth;
#pragma unroll
        for (int c = 0; c < kMlpOut; ++c) {
            out[o + c * kMlpWidth + kk] = ws[c] + odd[c * kMlpWidth + kk];
            if (kk == 0) out[o + kMlpOut * kMlpWidth + c] = wb[c] + odd[kMlpOut * kMlpWidth + c];
        }
    }
#pragma unroll
    for (int k = kMlpDepth - 1; k >= 0; --k) {
        // X[(k + 1) & 1], Gs and Ss are free: their last readers passed a barrier
        float dz[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const float slope = dsilu_f(Z[k][j]);
            dz[j] = dH[j] * slope;
            Gs[row_of(j) * kMlpWidth + col] = dH[j];
            Ss[row_of(j) * kMlpWidth + col] = slope;
        }
        put(dz, k > 0 ? X[(k + 1) & 1] : nullptr, tile_t(DT, k));
        __syncthreads();
        if (k > 0) {
            floatx16 acc = {};
#pragma unroll
            for (int s = 0; s < 8; ++s)
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag(X[(k + 1) & 1], kTrainPitch, 32 * rt + lane, s), bw[s], acc, 0, 0, 0);
            if (k > 1) {
#pragma unroll
                for (int s = 0; s < 8; ++s) bw[s] = wfrag(net.WT + (size_t)(k - 1) * kMlpWidth * kMlpWidth, kMlpWidth, col, s);
            }
#pragma unroll
            for (int j = 0; j < 16; ++j) dH[j] = acc[j];
        }
        float bsum = 0.0f;                              // bias gradient, the slope product unrounded
        if (par < 2) {
#pragma unroll 8
            for (int r = par; r < kTrainRows; r += 2) bsum = fmaf(Gs[r * kMlpWidth + kk], Ss[r * kMlpWidth + kk], bsum);
            if (par == 1) odd[kk] = bsum;
        }
        __syncthreads();
        if (par == 0) out[k * kMlpWidth + kk] = bsum + odd[kk];
    }
}

// Weight gradients of the hidden layers: chain u of layer y (blockIdx) sums the
// groups u, u + 4, .. (the last groups % 4 join chain 0), each group's product
// from zero: part[layer][u][n][k].  A workgroup takes one 32 x 32 tile of a
// chain; its eight wavefronts take eight groups at a time and the sums follow in
// order from LDS.  Operands are 16-byte loads of transposed tiles.  Workgroups go
// to the XCDs round-robin: the 16 tiles of a chain, which share its operands,
// have one id modulo 8.
__global__ __launch_bounds__(512) void k_mlp_wgrad(const __bf16 *HT, const __bf16 *DT, int rows, int chunk, int groups,
                                                   float *part) {
    __shared__ float P[8][32 * 32];
    const int chain = (blockIdx.x & 7) + 8 * (blockIdx.x >> 7), tile = (blockIdx.x >> 3) & 15;
    const int layer = chain >> 2, u = chain & 3, n0 = 32 * (tile >> 2), k0 = 32 * (tile & 3);
    const int l = threadIdx.x & 63, w = threadIdx.x >> 6, half = l >> 5, lane = l & 31;
    const int quads = groups >> 2;
    const int len = quads + (u == 0 ? groups & 3 : 0);      // groups of this chain
    float s[2] = {0.0f, 0.0f};                              // elements threadIdx.x and threadIdx.x + 512
    auto load = [&](const __bf16 *T, int c0, int r0) {      // column c0 + lane, rows r0 + 8 half ..
        const __bf16 *t = T + ((size_t)(r0 >> 6) * kMlpDepth + layer) * kTileT;
        return *reinterpret_cast<const bf16x8 *>(t + tile_at((r0 & 63) + 8 * half, c0 + lane));
    };
    for (int j0 = 0; j0 < len; j0 += 8) {
        const int j = j0 + w;
        floatx16 acc = {};
        if (j < len) {
            const int g = j < quads ? 4 * j + u : 4 * quads + (j - quads);
            const int r_end = min(rows, (g + 1) * chunk);
            for (int r0 = g * chunk; r0 < r_end; r0 += 128) {
                bf16x8 a[8], b[8];
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    const int r = min(r0 + 16 * q, (r_end - 1) & ~15);   // (past the end: loaded, not used)
                    a[q] = load(DT, n0, r);
                    b[q] = load(HT, k0, r);
                }
#pragma unroll
                for (int q = 0; q < 8; ++q)
                    if (r0 + 16 * q < r_end) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[q], b[q], acc, 0, 0, 0);
            }
        }
#pragma unroll
        for (int e = 0; e < 16; ++e) P[w][((e / 4) * 8 + half * 4 + (e % 4)) * 32 + lane] = acc[e];
        __syncthreads();
        const int cnt = min(8, len - j0);
        for (int q = 0; q < cnt; ++q) {
            s[0] += P[q][threadIdx.x];
            s[1] += P[q][threadIdx.x + 512];
        }
        __syncthreads();
    }
    float *out = part + ((size_t)layer * 4 + u) * kMlpWidth * kMlpWidth;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int e = threadIdx.x + 512 * q;
        out[(n0 + (e >> 5)) * kMlpWidth + k0 + (e & 31)] = s[q];
    }
}

// Slot of evaluation column k within its 32-block: the inverse of mlp_perm.
__device__ __forceinline__ int mlp_perm_slot(int k) { return 8 * ((k >> 2) & 3) + 4 * (k >> 4) + (k & 3); }

// One parameter's gradient g: stored, and with apply its Adam step taken on the
// FP32 master.  Returns the parameter.
__device__ __forceinline__ float adam_step(const TrainNet &net, const AdamArgs &a, int i, float g) {
    net.g[i] = g;
    float p = net.p[i];
    if (a.apply) {
        const float mi = a.b1 * net.mo[i] + (1.0f - a.b1) * g;
        const float vi = a.b2 * net.ve[i] + (1.0f - a.b2) * g * g;
        net.mo[i] = mi;
        net.ve[i] = vi;
        p -= a.lr * (mi / a.c1) / (sqrtf(vi / a.c2) + a.eps);
        net.p[i] = p;
    }
    return p;
}

// Blocks [0, kUpdateW): 256 hidden weights each, the four chains of their gradient;
// then 64 of the other sums each, over the blocks of k_mlp_train, one thread a
// chain; the last: the loss.  With apply the BF16 copies are rewritten too.
constexpr int kUpdateW = kMlpDepth * kMlpWidth * kMlpWidth / 256;
constexpr int kUpdateS = (kTrainSums + 63) / 64;

__global__ __launch_bounds__(256) void k_mlp_update(TrainNet net, AdamArgs a, const float *part, const float *sums,
                                                    const double *loss_part, int nblk, volatile double *loss_host) {
    const int tid = threadIdx.x, blk = blockIdx.x;
    if (blk < kUpdateW) {
        constexpr int WW = kMlpWidth * kMlpWidth;
        const int i = blk * 256 + tid, layer = i / WW, e = i % WW;
        const float *P = part + (size_t)layer * 4 * WW + e;
        const float p = adam_step(net, a, kMlpOffW + i, (P[0] + P[WW]) + (P[2 * WW] + P[3 * WW]));
        if (a.apply) {
            const int n = e / kMlpWidth, k = e % kMlpWidth;
            const __bf16 v = (__bf16)p;
            net.W[(size_t)layer * WW + operand_at(kMlpWidth, n, k)] = v;
            net.WT[(size_t)layer * WW + operand_at(kMlpWidth, k, n)] = v;
            net.We[(size_t)layer * WW + n * kMlpWidth + (layer == 0 ? k : (k & ~31) + mlp_perm_slot(k & 31))] = v;
        }
        return;
    }
    if (blk < kUpdateW + kUpdateS) {
        __shared__ float red[4][64];
        const int o = (blk - kUpdateW) * 64 + (tid & 63), u = tid >> 6;
        float s = 0.0f;
        if (o < kTrainSums) {
            const float *S = sums + o;
            const int quads = nblk >> 2;
            int q = 0;
            for (; q + 16 <= quads; q += 16) {          // sixteen loads in flight, added in order
                float v[16];
#pragma unroll
                for (int x = 0; x < 16; ++x) v[x] = S[(size_t)(4 * (q + x) + u) * kTrainSums];
#pragma unroll
                for (int x = 0; x < 16; ++x) s += v[x];
            }
            for (; q < quads; ++q) s += S[(size_t)(4 * q + u) * kTrainSums];
            if (u == 0)
                for (int g = 4 * quads; g < nblk; ++g) s += S[(size_t)g * kTrainSums];
        }
        red[u][tid & 63] = s;
        __syncthreads();
        if (u != 0 || o >= kTrainSums) return;
        const float g = (red[0][tid] + red[1][tid]) + (red[2][tid] + red[3][tid]);
        constexpr int nc = kMlpDepth * kMlpWidth, nw = kMlpOut * kMlpWidth;
        const int i = o < nc ? kMlpOffC + o : o < nc + nw ? kMlpOffWo + (o - nc) : kMlpOffCo + (o - nc - nw);
        const float p = adam_step(net, a, i, g);
        if (a.apply && o >= nc && o < nc + nw) {
            const int e = o - nc, n = e / kMlpWidth, k = e % kMlpWidth;
            net.Wo[operand_at(kMlpOutPad, n, k)] = (__bf16)p;
            net.Woe[n * kMlpWidth + (k & ~31) + mlp_perm_slot(k & 31)] = (__bf16)p;
        }
        return;
    }
    __shared__ double sum[256];
    double v = 0.0;
    for (int g = tid; g < nblk; g += 256) v += loss_part[g];
    sum[tid] = v;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (tid < s) sum[tid] += sum[tid + s];
        __syncthreads();
    }
    if (tid == 0) *loss_host = sum[0];
}

// W, WT, Wo: operand order (training products); We, Woe: evaluation order
// (columns of layers 2..6 and of the output layer permuted by mlp_perm).
__global__ void k_mlp_refresh(const float *p, __bf16 *W, __bf16 *WT, __bf16 *Wo, __bf16 *We, __bf16 *Woe) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < kMlpDepth * kMlpWidth * kMlpWidth) {
        const int layer = i / (kMlpWidth * kMlpWidth), e = i % (kMlpWidth * kMlpWidth);
        const int n = e / kMlpWidth, k = e % kMlpWidth;
        const __bf16 v = (__bf16)p[kMlpOffW + i];
        W[(size_t)layer * kMlpWidth * kMlpWidth + operand_at(kMlpWidth, n, k)] = v;
        WT[(size_t)layer * kMlpWidth * kMlpWidth + operand_at(kMlpWidth, k, n)] = v;
        const int ks = layer == 0 ? k : (k & ~31) + mlp_perm(k & 31);
        We[i] = (__bf16)p[kMlpOffW + (size_t)layer * kMlpWidth * kMlpWidth + n * kMlpWidth + ks];
    }
    if (i < kMlpOutPad * kMlpWidth) Wo[operand_at(kMlpOutPad, i / kMlpWidth, i % kMlpWidth)] = (__bf16)p[kMlpOffWo + i];
    if (i < kMlpEvalRows * kMlpWidth) {
        const int n = i / kMlpWidth, k = i % kMlpWidth;
        Woe[i] = n < kMlpOut ? (__bf16)p[kMlpOffWo + n * kMlpWidth + (k & ~31) + mlp_perm(k & 31)] : (__bf16)0.0f;
    }
}

// ---------------------------------------------------------------------------
// Point evaluation: neural field (64 points per wavefront) and trilinear grid.
// pts SoA: r[n], th[n], ph[n]; out: [n][12].
// ---------------------------------------------------------------------------
// The twelve components of point i, or NaN, in 16-byte stores (96 bytes a point;
// the caller's array is aligned to its doubles only).
__device__ __forceinline__ void store12(double *out, int i, const double g[12], bool ok) {
    typedef double pair __attribute__((ext_vector_type(2), aligned(8)));
    const double nan = __builtin_nan("");
    pair *o = reinterpret_cast<pair *>(out + (size_t)i * 12);
#pragma unroll
    for (int c = 0; c < 6; ++c) {
        pair v;
        v.x = ok ? g[2 * c] : nan;
        v.y = ok ? g[2 * c + 1] : nan;
        o[c] = v;
    }
}

// NT = 512: 8 wavefronts (2 per SIMD) share the staged weights; 256 for so few
// points that one wavefront per SIMD holds them.
// kHalves: 8, or 0 for the argument's number (a constant count is 1 % faster).
template <int NT, int kHalves>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(NT / 256)))
void k_mlp_eval(MlpArgs m, int n_halves, const double *pts, int n, double *out) {
    __shared__ MlpLds<NT> L;
    mlp_lds_init(m, L);
    const int halves = kHalves ? kHalves : n_halves;
    const MlpShare share = mlp_share(halves, NT / 64);
    const int lane = threadIdx.x & 63;
    const int i = blockIdx.x * (NT / 8 * halves) + (int)share.first + lane;
    const bool in = lane < 16 * share.passes && i < n;
    const int ii = in ? i : n - 1;                    // idle lanes evaluate a valid point
    const double r = pts[ii], th = pts[(size_t)n + ii], ph = pts[2 * (size_t)n + ii];
    float y[kMlpOut], dy[3][kMlpOut];
    mlp_block<NT>(m, halves, (float)r, (float)th, (float)ph, L, y, dy);
    double g[12];
    const bool ok = mlp_assemble<double>(m, r, th, y, dy, g);
    if (in) store12(out, i, g, ok);
}

// One point per lane, the eight nodes of its cell in flight at once; workgroups of
// one wavefront, so that a training batch (16,384 points) spreads over every
// compute unit: 16.3 -> 6.9 us.
template <int FDT>
__global__ __launch_bounds__(64) void k_field_sample(FieldDev f, const double *pts, int n, double *out) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    CellPos<double> at;
    LaneCell<FDT> cell;
    NoCell none;
    double g[12];
    bool ok = cell_seek<FDT, double>(f, pts[i], pts[(size_t)n + i], pts[2 * (size_t)n + i], 0u, at, cell, f, none);
    if (ok) {
        cell.template value<0, 12, double>(f, at, 0u, g);
        ok = finite12(g);
    }
    store12(out, i, g, ok);
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
hipError_t mlp_launch_train(const MlpArgs &m, const TrainNet &net, const double *pts, const double *tgt, int npair,
                            const MlpLoss &L, const AdamArgs &adam, const TrainBufs &w, volatile double *loss_host,
                            hipStream_t s) {
    const int rows = 2 * npair, nblk = mlp_train_blocks(npair);
    const int chunk = mlp_train_chunk(rows), groups = (rows + chunk - 1) / chunk;
    hipLaunchKernelGGL(k_mlp_train<false>, dim3(nblk), dim3(kTrainThreads), 0, s, m, net, pts, tgt, npair, L, w.Y, w.HT,
                       w.DT, w.sums, w.loss);
    hipLaunchKernelGGL(k_mlp_train<true>, dim3(nblk), dim3(kTrainThreads), 0, s, m, net, pts, tgt, npair, L, w.Y, w.HT,
                       w.DT, w.sums, w.loss);
    hipLaunchKernelGGL(k_mlp_wgrad, dim3(16 * 4 * kMlpDepth), dim3(512), 0, s, w.HT, w.DT, rows, chunk, groups, w.part);
    hipLaunchKernelGGL(k_mlp_update, dim3(kUpdateW + kUpdateS + 1), dim3(256), 0, s, net, adam, w.part, w.sums, w.loss,
                       nblk, loss_host);
    return hipGetLastError();
}

hipError_t mlp_launch_refresh(const float *p, __bf16 *W, __bf16 *WT, __bf16 *Wo, __bf16 *We, __bf16 *Woe,
                              hipStream_t s) {
    const int n = kMlpDepth * kMlpWidth * kMlpWidth;
    hipLaunchKernelGGL(k_mlp_refresh, dim3((n + 255) / 256), dim3(256), 0, s, p, W, WT, Wo, We, Woe);
    return hipGetLastError();
}

hipError_t mlp_launch_eval(const MlpArgs &m, const double *pts, int n, double *out, int cus, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    const int waves = mlp_waves(n, cus), halves = mlp_halves(n, waves, cus), per = 8 * halves * waves;
    const dim3 grid((n + per - 1) / per);
    if (waves == 4) hipLaunchKernelGGL((k_mlp_eval<256, 0>), grid, dim3(256), 0, s, m, halves, pts, n, out);
    else if (halves == 8) hipLaunchKernelGGL((k_mlp_eval<512, 8>), grid, dim3(512), 0, s, m, halves, pts, n, out);
    else hipLaunchKernelGGL((k_mlp_eval<512, 0>), grid, dim3(512), 0, s, m, halves, pts, n, out);
    return hipGetLastError();
}

hipError_t launch_field_sample(const FieldDev &f, const double *pts, int n, double *out, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    const dim3 grid((n + 63) / 64), block(64);
    switch (f.dtype) {
        case GC_F64: hipLaunchKernelGGL(k_field_sample<GC_F64>, grid, block, 0, s, f, pts, n, out); break;
        case GC_F32: hipLaunchKernelGGL(k_field_sample<GC_F32>, grid, block, 0, s, f, pts, n, out); break;
        default:     hipLaunchKernelGGL(k_field_sample<GC_F16>, grid, block, 0, s, f, pts, n, out); break;
    }
    return hipGetLastError();
}

}  // namespace gc
