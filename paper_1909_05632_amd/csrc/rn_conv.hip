// Dirty-tile convolution kernels (Sec. 1: recompute only where the change can
// reach and reuse the cached activations elsewhere).
//
// A conv layer is bias and ReLU after a k x k cross-correlation with stride s
// and zero padding p:
//   out[y][x][co] = ReLU(b[co] + sum_{ky,kx,ci} w[co][ci][ky][kx] * in[s y-p+ky][s x-p+kx][ci]).
// Most kernels here are for 3x3, stride 1, pad 1 (6x6 input halo per tile); the
// general-layer kernel k_conv_gen takes other k and s.  Each work-list entry
// names one 4x4 output tile of one stream; the kernels compute its 16 pixels x
// cout outputs and write them in place into the stream's cache (scatter fused
// with bias and ReLU).
// Pixels of a ragged edge tile that fall outside the image are written as 0:
// they are the next layer's zero padding and carry zero dense weights.
//
// Cache layout ("tiled NHWC"): per slot [TH][TW][16][C], a tile's 16 pixels in
// row-major order, channels innermost; one tile is 16 * C contiguous elements.
//
// The kernels are persistent: the grid is sized to the chip and the blocks walk
// the device-side work list until the device-side count is exhausted, so no
// host synchronisation is needed to size a launch.  In dense mode (the
// comparison path) they walk every tile of every stream instead of a list;
// the arithmetic per tile is the same code, so a dense pass and a reuse pass
// give the same bits.
//
// Tile-partial head (last layer only): the dense head is linear, so the logits
// are a sum over tiles of each tile's own contribution.  The epilogue computes
// that contribution for the tiles it recomputes and stores it per (stream,
// tile); clean tiles keep theirs.  The head then only adds partials.
#include "rn_split.hpp"

namespace rn {
namespace {

using namespace dev;

// ------------------------------------------------------------------ first layer

// Direct conv for a few input channels (1, or 4 stacked frames): 9 * CIN FMAs
// per output, too few for a matrix core to pay off; the layer is HBM-bound on
// its output writes.  One wave per tile: lane l owns output channels l, l + 64
// (its 9 CIN weights in registers for the kernel's life); the 6x6 x CIN halo
// goes to LDS channel-innermost and from there, by broadcast reads, into every
// lane's registers, so the 16 x 9 CIN FMAs of a lane touch registers only.
// Each output is accumulated with fmaf over (c, ky, kx) in that order, then the
// bias is added (the order the folded layer-1 staging of the layer-2 kernel
// uses, so both give the same bits).  Stores: the lanes of one pixel write
// consecutive channels.  VAR: the tiles of variants (input from the base slot
// and the variant's frame, output to the overlay row of the work item).
template <int CIN, int COUT, bool DENSE, bool VAR>
__global__ __launch_bounds__(256) void k_conv_first_f32(ConvArgs a) {
    constexpr int CPL = (COUT + 63) / 64;         // channels per lane
    constexpr int HN = 36 * CIN;                  // halo values
    __shared__ float s_halo[4][HN];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const float *wg = static_cast<const float *>(a.w);
    float wr[CPL][CIN * 9], br[CPL];
#pragma unroll
    for (int j = 0; j < CPL; ++j) {
        const int co = min(lane + 64 * j, COUT - 1);
#pragma unroll
        for (int k = 0; k < CIN * 9; ++k) wr[j][k] = wg[k * COUT + co];
        br[j] = a.bias[co];
    }

    const int cnt = work_count<DENSE>(a);
    const size_t HW = (size_t)a.H * a.W;
    const int cin1 = CIN / a.stack;               // channels per frame
    float *halo = s_halo[wave];
    const float *xin = static_cast<const float *>(a.in);
    float *outp = static_cast<float *>(a.out);

    // The halo values of the next tile (past the end: the last tile again,
    // never used) are loaded into registers, HPL per lane, before this tile's
    // FMAs, so their latency overlaps the arithmetic.
    constexpr int HPL = (HN + 63) / 64;
    const XcdRange xr = xcd_range(cnt, 4);
    auto load_tile = [&](int t, float *pv) __attribute__((always_inline)) {
        const TileRef r = decode<DENSE>(a, t);
        int head = 0;
        if (!VAR && a.stack != 1) head = a.ring_head[r.slot];
#pragma unroll
        for (int k = 0; k < HPL; ++k) {
            const int h = lane + 64 * k;
            const int c = h / 36, pos = h - c * 36;
            const int hy = pos / 6, hx = pos - hy * 6;
            const int y = r.ty * kTile - 1 + hy, x = r.tx * kTile - 1 + hx;
            float v = 0.0f;
            if (h < HN && y >= 0 && y < a.H && x >= 0 && x < a.W) {
                if constexpr (VAR) {
                    v = var_input(a, r.slot, c, y, x);
                } else {
                    const float *plane;
                    if (a.stack == 1) {
                        plane = xin + ((size_t)r.slot * CIN + c) * HW;
                    } else {
                        // Channel c = frame j (oldest first) of the ring, channel c1 of it.
                        const int j = c / cin1, c1 = c - j * cin1;
                        const int rp = (head - (a.stack - 1) + j + 4 * a.stack) & 3;
                        plane = xin + (((size_t)r.slot * 4 + rp) * cin1 + c1) * HW;
                    }
                    v = plane[(size_t)y * a.W + x];
                }
            }
            pv[k] = v;
        }
    };
    int t = xr.first + wave;
    if (t >= xr.end) return;
    float pv[HPL];
    load_tile(t, pv);
    for (; t < xr.end; t += xr.stride) {
        const TileRef r = decode<DENSE>(a, t);
#pragma unroll
        for (int k = 0; k < HPL; ++k) {
            const int h = lane + 64 * k;
            if (h < HN) {
                const int c = h / 36, pos = h - c * 36;
                halo[pos * CIN + c] = pv[k];
            }
        }
        wave_sync();
        // One output row at a time: its three halo rows (18 pixels x CIN,
        // contiguous in LDS) go to registers by broadcast reads.
        float hr[18 * CIN];
        load_tile(min(t + xr.stride, xr.end - 1), pv);
        float *dst = VAR ? static_cast<float *>(a.vov_out) + (size_t)t * kTilePx * COUT
                         : outp + (size_t)r.slot * a.out_stride + (size_t)r.tile * kTilePx * COUT;
#pragma unroll
        for (int py = 0; py < kTile; ++py) {
            if constexpr (CIN % 4 == 0) {
#pragma unroll
                for (int q = 0; q < 18 * CIN / 4; ++q) {
                    const float4 v4 = reinterpret_cast<const float4 *>(halo + py * 6 * CIN)[q];
                    hr[4 * q] = v4.x;
                    hr[4 * q + 1] = v4.y;
                    hr[4 * q + 2] = v4.z;
                    hr[4 * q + 3] = v4.w;
                }
            } else {
#pragma unroll
                for (int q = 0; q < 18 * CIN; ++q) hr[q] = halo[py * 6 * CIN + q];
            }
#pragma unroll
            for (int j = 0; j < CPL; ++j) {
                const int co = lane + 64 * j;
                if (co >= COUT) continue;
#pragma unroll
                for (int px = 0; px < kTile; ++px) {
                    const int m = py * kTile + px;
                    float acc = 0.0f;
#pragma unroll
                    for (int c = 0; c < CIN; ++c)
#pragma unroll
                        for (int ky = 0; ky < 3; ++ky)
#pragma unroll
                            for (int kx = 0; kx < 3; ++kx)
                                acc = fmaf(wr[j][c * 9 + ky * 3 + kx], hr[(ky * 6 + px + kx) * CIN + c], acc);
                    float v = acc + br[j];
                    v = v > 0.0f ? v : 0.0f;
                    if (r.ty * kTile + py >= a.H || r.tx * kTile + px >= a.W) v = 0.0f;
                    dst[m * COUT + co] = v;
                }
            }
        }
        wave_sync();                                   // halo reads done before the next tile's writes
    }
}

// Layer 1 with four input channels (stacked frames, or a 4-channel input) on
// the matrix cores: for every output channel count a lane-per-channel kernel
// leaves lanes idle (40 channels use 40 of 64 lanes) and runs its FMAs at the
// VALU rate.  Per tile an implicit GEMM on v_mfma_f32_16x16x4_f32: M = 16
// pixels (row m = pixel (m / 4, m % 4)), N = COUT in blocks of 16 (padded with
// zero weights), K = 36 in (c, ky, kx) order, nine k-steps; step s gives lane
// group kq the K index 4 s + kq, a halo value gathered from LDS (offsets fixed
// per lane), and the B fragments stay in registers for the kernel's life.
// D: lane (n, kq) holds pixels 4 kq + i (row kq, column i) of channel
// 16 nb + n.  The halo prefetch and the VAR handling are those of
// k_conv_first_f32.
template <int COUT, bool DENSE, bool VAR>
__global__ __launch_bounds__(256) void k_conv_first4_mfma(ConvArgs a) {
    constexpr int CIN = 4, KS = 9, NB = (COUT + 15) / 16;
    constexpr int HN = 36 * CIN;                  // halo values
    constexpr int HPL = (HN + 63) / 64;
    __shared__ float s_halo[4][HN];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int mrow = lane & 15, kq = lane >> 4;
    const float *wg = static_cast<const float *>(a.w);
    float bw[KS][NB], bias[NB];
    int aoff[KS];
#pragma unroll
    for (int s = 0; s < KS; ++s) {
        const int k = 4 * s + kq, c = k / 9, r = k - 9 * c, ky = r / 3, kx = r - 3 * ky;
        aoff[s] = (((mrow >> 2) + ky) * 6 + (mrow & 3) + kx) * CIN + c;
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            const int n = 16 * nb + mrow;
            bw[s][nb] = n < COUT ? wg[k * COUT + n] : 0.f;
        }
    }
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) bias[nb] = 16 * nb + mrow < COUT ? a.bias[16 * nb + mrow] : 0.f;

    const int cnt = work_count<DENSE>(a);
    const size_t HW = (size_t)a.H * a.W;
    const int cin1 = CIN / a.stack;               // channels per frame
    float *halo = s_halo[wave];
    const float *xin = static_cast<const float *>(a.in);
    float *outp = static_cast<float *>(a.out);
    const XcdRange xr = xcd_range(cnt, 4);
    auto load_tile = [&](int t, float *pv) __attribute__((always_inline)) {
        const TileRef r = decode<DENSE>(a, t);
        int head = 0;
        if (!VAR && a.stack != 1) head = a.ring_head[r.slot];
#pragma unroll
        for (int k = 0; k < HPL; ++k) {
            const int h = lane + 64 * k;
            const int c = h / 36, pos = h - c * 36;
            const int hy = pos / 6, hx = pos - hy * 6;
            const int y = r.ty * kTile - 1 + hy, x = r.tx * kTile - 1 + hx;
            float v = 0.0f;
            if (h < HN && y >= 0 && y < a.H && x >= 0 && x < a.W) {
                if constexpr (VAR) {
                    v = var_input(a, r.slot, c, y, x);
                } else {
                    const float *plane;
                    if (a.stack == 1) {
                        plane = xin + ((size_t)r.slot * CIN + c) * HW;
                    } else {
                        const int j = c / cin1, c1 = c - j * cin1;
                        const int rp = (head - (a.stack - 1) + j + 4 * a.stack) & 3;
                        plane = xin + (((size_t)r.slot * 4 + rp) * cin1 + c1) * HW;
                    }
                    v = plane[(size_t)y * a.W + x];
                }
            }
            pv[k] = v;
        }
    };
    int t = xr.first + wave;
    if (t >= xr.end) return;
    float pv[HPL];
    load_tile(t, pv);
    for (; t < xr.end; t += xr.stride) {
        const TileRef r = decode<DENSE>(a, t);
#pragma unroll
        for (int k = 0; k < HPL; ++k) {
            const int h = lane + 64 * k;
            if (h < HN) {
                const int c = h / 36, pos = h - c * 36;
                halo[pos * CIN + c] = pv[k];
            }
        }
        wave_sync();
        float av[KS];
#pragma unroll
        for (int s = 0; s < KS; ++s) av[s] = halo[aoff[s]];
        load_tile(min(t + xr.stride, xr.end - 1), pv);
        floatx4 acc[NB];
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) acc[nb] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < KS; ++s)
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) acc[nb] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[s], bw[s][nb], acc[nb], 0, 0, 0);
        float *dst = VAR ? static_cast<float *>(a.vov_out) + (size_t)t * kTilePx * COUT
                         : outp + (size_t)r.slot * a.out_stride + (size_t)r.tile * kTilePx * COUT;
        const bool row_in = r.ty * kTile + kq < a.H;
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            const int n = 16 * nb + mrow;
            if (n >= COUT) continue;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                float v = acc[nb][i] + bias[nb];
                v = v > 0.0f ? v : 0.0f;
                if (!row_in || r.tx * kTile + i >= a.W) v = 0.0f;
                dst[(4 * kq + i) * COUT + n] = v;
            }
        }
        wave_sync();                                   // halo reads done before the next tile's writes
    }
}

// ------------------------------------------------------------------ MFMA layers

// v_mfma_f32_16x16x4_f32 operand layout (lane l, kq = l / 16):
//   A: row l % 16, k-row kq;  B: k-row kq, column l % 16;
//   D: rows 4 kq + i, column l % 16, i = 0..3.
// Rows are tile pixels in column-major order, row m = pixel (m % 4, m / 4), so
// lane l of D holds pixels (i, kq), i = 0..3, of channel l % 16 + 16 nb (D is
// the same for v_mfma_f32_16x16x32_bf16, whose lanes hold eight K values each).

// Layer 1 folded into layer 2 (one input channel): the 8x8 input patch around
// a tile, one pixel a lane; pixels outside the image are 0.
template <bool VAR>
__device__ inline float fetch_patch(const ConvArgs &a, const TileRef &r, int lane) {
    const int y = r.ty * kTile - 2 + (lane >> 3), x = r.tx * kTile - 2 + (lane & 7);
    const bool in = y >= 0 && y < a.H && x >= 0 && x < a.W;
    if constexpr (VAR) return in ? var_input(a, r.slot, 0, y, x) : 0.f;
    const float *plane = static_cast<const float *>(a.in) + (size_t)r.slot * a.in_stride;
    return in ? plane[(size_t)y * a.W + x] : 0.f;
}

// Bias, ReLU, zero outside the image, coalesced store of the 16 x COUT tile
// through LDS (the halo area is free by now), and the tile's head partials.
template <int COUT>
struct Epi {
    static constexpr int NB = COUT / 16;      // 16-column blocks of the 16x16x4 product
    static constexpr int SR = COUT + 4;       // row stride of the output staging area
};

template <int COUT>
__device__ inline void epilogue(const ConvArgs &a, const TileRef &r, floatx4 *acc, const float *s_bias,
                                float *stage, int lane) {
    using M = Epi<COUT>;
    const int mrow = lane & 15, kq = lane >> 4;       // D holds pixels (py = i, px = kq)
    // Bias, then ReLU and the zero outside the image on the bit patterns, with
    // no per-value compare into a lane mask: a float above zero has a positive
    // int pattern (zeros, negatives go to +0 under the int max), and pixels
    // outside the image are masked to +0 (all-ones / all-zero row masks; the
    // row bound is the same for the whole wave).
    const int col_keep = ~((a.W - 1 - (r.tx * kTile + kq)) >> 31);
    int keep[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) keep[i] = col_keep & ~((a.H - 1 - (r.ty * kTile + i)) >> 31);
#pragma unroll
    for (int nb = 0; nb < M::NB; ++nb) {
        const float b = s_bias[nb * 16 + mrow];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            acc[nb][i] = __int_as_float(max(__float_as_int(acc[nb][i] + b), 0) & keep[i]);
            stage[(i * 4 + kq) * M::SR + nb * 16 + mrow] = acc[nb][i];
        }
    }
    wave_sync();
    const int n_out = a.n_out;
    if (n_out > 0) {
        // Tile contribution to each logit: per-lane partial dot products, then
        // the lane sums, 8 logits at a time (lane_sums8).
        const int ntiles = a.TH * a.TW;
        for (int o0 = 0; o0 < n_out; o0 += 8) {
            float p[8];
#pragma unroll
            for (int q = 0; q < 8; q += 2) {
                // Two logits per batch: their 2 x NB weight loads are issued
                // together (indices clamped, results of absent logits dropped).
                const int oa = min(o0 + q, n_out - 1), ob = min(o0 + q + 1, n_out - 1);
                const float4 *wa = reinterpret_cast<const float4 *>(
                                       a.hw + ((size_t)oa * ntiles + r.tile) * kTilePx * COUT) + lane;
                const float4 *wb = reinterpret_cast<const float4 *>(
                                       a.hw + ((size_t)ob * ntiles + r.tile) * kTilePx * COUT) + lane;
                float4 va[M::NB], vb[M::NB];
#pragma unroll
                for (int nb = 0; nb < M::NB; ++nb) {
                    va[nb] = wa[nb * 64];
                    vb[nb] = wb[nb * 64];
                }
                float pa = 0.f, pb = 0.f;
#pragma unroll
                for (int nb = 0; nb < M::NB; ++nb) {
                    pa = fmaf(acc[nb][0], va[nb].x, pa);
                    pa = fmaf(acc[nb][1], va[nb].y, pa);
                    pa = fmaf(acc[nb][2], va[nb].z, pa);
                    pa = fmaf(acc[nb][3], va[nb].w, pa);
                    pb = fmaf(acc[nb][0], vb[nb].x, pb);
                    pb = fmaf(acc[nb][1], vb[nb].y, pb);
                    pb = fmaf(acc[nb][2], vb[nb].z, pb);
                    pb = fmaf(acc[nb][3], vb[nb].w, pb);
                }
                p[q] = pa;
                p[q + 1] = pb;
                if (o0 + q + 2 >= n_out) {
                    for (int z = q + 2; z < 8; ++z) p[z] = 0.f;
                    break;
                }
            }
            const float v = lane_sums8(p, lane);
            const int q = (lane >> 5) * 4 + ((lane >> 4) & 1) * 2 + ((lane >> 3) & 1);
            if ((lane & 7) == 0 && o0 + q < n_out) {
                a.hpart[((size_t)r.slot * ntiles + r.tile) * n_out + o0 + q] = v;
            }
        }
    }
    // The tile's stores go last: the next tile's waits on its own loads then
    // never have to drain them.
    float4 *d4 = reinterpret_cast<float4 *>(static_cast<float *>(a.out) + (size_t)r.slot * a.out_stride + (size_t)r.tile * kTilePx * COUT);
#pragma unroll
    for (int j = 0; j < M::NB; ++j) {                  // 16 * COUT / 4 float4 = 64 * NB
        const int o4 = lane + 64 * j;
        const int e = 4 * o4, m = e / COUT, n = e - m * COUT;
        d4[o4] = *reinterpret_cast<const float4 *>(stage + m * M::SR + n);
    }
    wave_sync();
}

// Item words of a wave's items (the block's items t, t + G, ..), 64 at a time:
// lane j of chunk c holds the word of the wave's item 64 c + j (past the last:
// the block's last item's word, so every load reads a valid entry).  The words
// of a whole chunk arrive in one load, long before they are read with
// readlane, so no per-tile word load is waited for.
template <bool DENSE>
__device__ inline uint32_t word_chunk(const ConvArgs &a, const RunRange &rr, int t, int G, int c, int lane) {
    return item_word<DENSE>(a, rr.at(min(t + (64 * c + lane) * G, rr.count - 1)));
}

// Word of item j, held in chunk c0 (w0) or c0 + 1 (w1); j is wave-uniform.
__device__ inline TileRef item_of(const ConvArgs &a, uint32_t w0, uint32_t w1, int c0, int j) {
    const uint32_t src = (j >> 6) == c0 ? w0 : w1;
    return item_ref(a, (uint32_t)__builtin_amdgcn_readlane((int)src, j & 63));
}

// ---- 40 -> 80: weights in registers, bf16 matrix cores with split operands
//
// Bound: matrix issue.  A tile is 2 * 16 * 80 * 360 flops six times over on
// v_mfma_f32_16x16x32_bf16 (rn_split.hpp): 360 ops with K padded from 360 to
// 384, 1440 cycles a tile when one wave of each SIMD issues nothing else (the
// float32 instruction: 450 ops of 32 cycles, 3600).  Measured, about twice that
// (256 105x80 streams all dirty, 540 tiles a CU: 640 us, the matrix pipe busy
// 55% of the cycles; 44% in a step's 73 tiles a CU), whatever form the halo
// takes: the other roles' vector work sets the period as well.  Split, the weights take
// 184 KB: more than LDS, but they fit the registers of four waves that each
// hold a quarter of K (three k-steps x 80 channels x three planes, 180
// registers).  So a block of eight waves splits the work by role, two waves a
// SIMD, and the vector work runs beside the matrix ops:
//   waves 0-3 (one per SIMD) read the pixels of both tiles of a group from LDS
//     and sum their quarter of K into partial products in LDS;
//   waves 4, 5 add a tile's four partial products (in wave order) and run the
//     epilogue;
//   waves 6, 7 build a tile's halo: the 6 x 6 x 40 layer-1 activations, loaded
//     or (FUSE) computed from the 8 x 8 input patch, split into three bf16
//     planes.  Lane c4 + 10 hy has four channels of a halo row, so the folded
//     layer's weights stay in its registers too.
// The roles work on consecutive groups: in a period groups i (halo), i - 1
// (products) and i - 2 (epilogue), one block barrier a period.
//
// K is walked in octets of channels, octet g = position g / 5, channels
// 8 (g % 5): k-step s of 32 gives lane group kq octet 4 s + kq (octets 45 to 47
// have zero weights).  A plane's halo pixel (hy, hx) starts at 16-byte slot
// 36 hy + 5 hx, so the 16 pixels of a 16-lane read lie in 16 distinct bank
// groups at every octet.
//
// A result that is not finite: an infinity or a NaN among its operands makes it
// NaN (split4_any), and the sum of its leading terms alone, formed then, has the
// class of the float32 sum; a NaN weight makes its channel's results NaN by the
// bias (flagged when packed), so that a net full of NaN takes no second look.
// What overflows from finite operands is taken from the plain float32 sum.
//
// So is a result next to 0: within 2^-19 of the largest of its channel's first
// and last partial products over the 4 pixels of its tile column.  ReLU
// decisions, which the gradient depends on, are then those of the float32 sums.
// (Of 168 K results next to 0, the float32 sums' errors relative to that scale
// are below 2^-19.2 but for 1 in 10 K; 1 or 2 tiles in 1000 hold such a result,
// whatever the sizes of the channels.  A scale taken over all 80 channels made
// every tile of an uneven net sum again, 10 times the time.)  More than four of
// them in a tile come from inputs that cancel by structure, an edge filter over
// a flat patch: their float32 sums are rounding noise as well, and they stay as
// they are, so that a tile's time is bounded whatever its values.  Variants, of
// which no gradient is taken, go without: they share the base's results, so one
// of its results next to 0 is met by every variant that reaches its tile, one
// after the other (4096 occlusion variants of a 105x80 frame 273 -> 349 us).
constexpr float kNearZero = 0x1p-19f;
constexpr int kMostSingle = 4;            // results of a tile taken one by one

struct Res {
    static constexpr int CIN = 40, COUT = 80, NB = COUT / 16, KS = 12, KW = KS / 4;
    static constexpr int OCT = 45;                    // octets of K
    static constexpr int ROW = 36 * 16;               // bytes of a halo row
    static constexpr int PLANE = 6 * ROW;
    static constexpr int HALO = 3 * PLANE;            // one tile
    static constexpr int PART = 4 * NB * 64 * 16;     // partial products of one tile
    // Two tiles a group: three halo buffers (built, read, kept for the check
    // of the sums), two of partial products.
    static constexpr int OPART = 3 * 2 * HALO, OSMALL = OPART + 2 * 2 * PART;
    static constexpr int PAIRS = 2 * 9 * CIN, OPAIRS = OSMALL + 2 * 64 * 4 + COUT * 4;   // floats a wave; bytes
    static constexpr size_t lds_bytes = (size_t)OPAIRS + 2 * PAIRS * 4;
    static_assert(lds_bytes <= 160 * 1024, "LDS of a CU");
    static constexpr size_t w_bytes = (size_t)KS * NB * 3 * 1024;   // then [COUT] floats: NaN where a weight of the channel is
};

// The plain float32 product of a tile from its halo planes (their sum is the
// float32 value), in the order of v_mfma_f32_16x16x4_f32 over (position,
// 16-channel block, k-step): float32 weights as pack_conv_mfma lays them out.
__device__ inline void res_plain(const float *w, const unsigned char *halo, floatx4 (&acc)[Res::NB], int lane) {
    using R = Res;
    const int m = lane & 15, kq = lane >> 4;
    const unsigned char *px = halo + (m & 3) * R::ROW + (m >> 2) * 80;
    auto value = [&](int off) {
        const unsigned char *p = px + off;
        return (float)*reinterpret_cast<const __bf16 *>(p) + (float)*reinterpret_cast<const __bf16 *>(p + R::PLANE) +
               (float)*reinterpret_cast<const __bf16 *>(p + 2 * R::PLANE);
    };
#pragma unroll
    for (int nb = 0; nb < R::NB; ++nb) acc[nb] = floatx4{0.f, 0.f, 0.f, 0.f};
    // Blocks u = 3 kpos + blk of 16, 16 and 8 channels.
    auto load = [&](floatx4 (&b)[R::NB], int u) __attribute__((always_inline)) {
        const int kpos = u / 3, blk = u - 3 * kpos;
        const float *p = w + kpos * R::CIN * R::COUT + blk * 16 * R::COUT;
#pragma unroll
        for (int nb = 0; nb < R::NB; ++nb) {
            if (blk < 2) {
                b[nb] = *reinterpret_cast<const floatx4 *>(p + (nb * 64 + lane) * 4);
            } else {
                const float2 v = *reinterpret_cast<const float2 *>(p + (nb * 64 + lane) * 2);
                b[nb] = floatx4{v.x, v.y, 0.f, 0.f};
            }
        }
    };
#pragma unroll 1
    for (int u = 0; u < 27; ++u) {
        floatx4 b[R::NB];
        load(b, u);
        const int kpos = u / 3, blk = u - 3 * kpos, steps = blk < 2 ? 4 : 2;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (j >= steps) break;                        // uniform
            const float av = value(kpos / 3 * R::ROW + kpos % 3 * 80 + 2 * (16 * blk + steps * kq + j));
#pragma unroll
            for (int nb = 0; nb < R::NB; ++nb) acc[nb] = __builtin_amdgcn_mfma_f32_16x16x4f32(av, b[nb][j], acc[nb], 0, 0, 0);
        }
        // NaN stays NaN: a net that has diverged ends here after one block.
        bool open = false;
#pragma unroll
        for (int nb = 0; nb < R::NB; ++nb)
#pragma unroll
            for (int e = 0; e < 4; ++e) open |= !__builtin_isnan(acc[nb][e]);
        if (!__any(open)) break;                          // uniform
    }
}

// The sum of the leading terms, hh, of a tile.
__device__ inline void res_lead(const bf16x8 *w, const unsigned char *halo, floatx4 (&acc)[Res::NB], int lane) {
    using R = Res;
    const int m = lane & 15, kq = lane >> 4;
#pragma unroll
    for (int nb = 0; nb < R::NB; ++nb) acc[nb] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 3
    for (int s = 0; s < R::KS; ++s) {
        const int g = 4 * s + kq, pos = g / 5;
        bf16x8 x{};                                       // octets past the last: 0, where 0 times an infinity would be NaN
        if (g < R::OCT)
            x = *reinterpret_cast<const bf16x8 *>(halo + ((m & 3) + pos / 3) * R::ROW + ((m >> 2) + pos % 3) * 80 + (g - 5 * pos) * 16);
#pragma unroll
        for (int nb = 0; nb < R::NB; ++nb)
            acc[nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x, w[(s * R::NB + nb) * 3 * 64 + lane], acc[nb], 0, 0, 0);
    }
}

// One output of it: channel n, pixel (row, column) of the tile.  The wave lays
// the 360 pairs of factors out in `pairs` in the order of the sum, one memory
// round trip, and then runs the chain, every lane the same: about 2 us, where
// the whole tile's product takes some 14.
__device__ inline float res_plain_one(const float *w, const unsigned char *halo, float *pairs, int n, int row, int col, int lane) {
    using R = Res;
    constexpr int K = 9 * R::CIN, V = (K + 63) / 64;
    float x[V], y[V];
#pragma unroll
    for (int v = 0; v < V; ++v) {
        const int k = min(lane + 64 * v, K - 1), kpos = k / 40, r = k - 40 * kpos;
        const int blk = r / 16, steps = blk < 2 ? 4 : 2, j = (r - 16 * blk) / 4, kq = r & 3;
        const unsigned char *p = halo + (row + kpos / 3) * R::ROW + (col + kpos % 3) * 80 + 2 * (16 * blk + steps * kq + j);
        y[v] = w[kpos * R::CIN * R::COUT + blk * 16 * R::COUT + ((n / 16) * 64 + kq * 16 + n % 16) * steps + j];
        x[v] = (float)*reinterpret_cast<const __bf16 *>(p) + (float)*reinterpret_cast<const __bf16 *>(p + R::PLANE) +
               (float)*reinterpret_cast<const __bf16 *>(p + 2 * R::PLANE);
    }
#pragma unroll
    for (int v = 0; v < V; ++v)
        if (lane + 64 * v < K) reinterpret_cast<float2 *>(pairs)[lane + 64 * v] = make_float2(x[v], y[v]);
    wave_sync();
    // Two pairs a read, B reads in flight while the chain takes the B before.
    constexpr int B = 5, N = K / 2 / B;
    static_assert(N * B * 2 == K, "whole batches");
    const floatx4 *src = reinterpret_cast<const floatx4 *>(pairs);
    floatx4 cur[B], next[B];
#pragma unroll
    for (int i = 0; i < B; ++i) cur[i] = src[i];
    float acc = 0.f;
#pragma unroll 2
    for (int n = 0; n < N; ++n) {
        const floatx4 *s = src + min(n + 1, N - 1) * B;
#pragma unroll
        for (int i = 0; i < B; ++i) next[i] = s[i];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < B; ++i) {
            acc = fmaf(cur[i][0], cur[i][1], acc);
            acc = fmaf(cur[i][2], cur[i][3], acc);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < B; ++i) cur[i] = next[i];
    }
    wave_sync();
    return acc;
}

// Largest magnitude of a channel's first and last partial products over a tile column.
__device__ inline float column_size(const floatx4 q0, const floatx4 q3) {
    float m = 0.f;
#pragma unroll
    for (int e = 0; e < 4; ++e) m = fmaxf(fmaxf(fabsf(q0[e]), fabsf(q3[e])), m);
    return m;
}

template <bool DENSE, bool FUSE, int NO, bool VAR>
__global__ __launch_bounds__(512, 2) void k_conv_mfma_res(ConvArgs a) {
    using R = Res;
    extern __shared__ __align__(16) unsigned char lds[];
    float *s_patch = reinterpret_cast<float *>(lds + R::OSMALL);
    float *s_bias = s_patch + 128;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int cnt = work_count<DENSE>(a);
    const RunRange rr = run_range(cnt);
    if (rr.count <= 0) return;                            // uniform per block
    const int G = rr.count > 1 ? 2 : 1;                   // tiles a group
    const int groups = (rr.count + G - 1) / G;
    auto halo_of = [&](int i, int t) { return lds + (2 * (i % 3) + t) * R::HALO; };
    auto part_of = [&](int i, int t) { return reinterpret_cast<floatx4 *>(lds + R::OPART + (2 * (i & 1) + t) * R::PART); };
    if (tid < R::COUT)
        s_bias[tid] = a.bias[tid] +
                      reinterpret_cast<const float *>(static_cast<const unsigned char *>(a.w_split) + R::w_bytes)[tid];

    if (wave < 4) {
        bf16x8 w[R::KW][R::NB][3];
        const bf16x8 *wg = static_cast<const bf16x8 *>(a.w_split) + (size_t)wave * R::KW * R::NB * 3 * 64 + lane;
#pragma unroll
        for (int s = 0; s < R::KW; ++s)
#pragma unroll
            for (int nb = 0; nb < R::NB; ++nb)
#pragma unroll
                for (int pl = 0; pl < 3; ++pl) w[s][nb][pl] = wg[((s * R::NB + nb) * 3 + pl) * 64];
        const int m = lane & 15, kq = lane >> 4;
        int off[R::KW];
#pragma unroll
        for (int s = 0; s < R::KW; ++s) {
            const int g = min(4 * (wave * R::KW + s) + kq, R::OCT - 1), pos = g / 5;
            off[s] = ((m & 3) + pos / 3) * R::ROW + ((m >> 2) + pos % 3) * 80 + (g - 5 * pos) * 16;
        }
        for (int i = 0; i < groups + 2; ++i) {
            if (i >= 1 && i <= groups) {
                bf16x8 x[R::KW][3];
                auto load_x = [&](int s, int t) __attribute__((always_inline)) {
                    const unsigned char *h = halo_of(i - 1, t) + off[s];
#pragma unroll
                    for (int pl = 0; pl < 3; ++pl) x[s][pl] = *reinterpret_cast<const bf16x8 *>(h + pl * R::PLANE);
                };
#pragma unroll
                for (int s = 0; s < R::KW; ++s) load_x(s, 0);
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    if (t >= G) break;                    // uniform
                    floatx4 acc[R::NB];
#pragma unroll
                    for (int nb = 0; nb < R::NB; ++nb) acc[nb] = floatx4{0.f, 0.f, 0.f, 0.f};
                    // (pixel plane, weight plane), small terms first
                    constexpr int px[6] = {2, 0, 1, 1, 0, 0}, pw[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
                    for (int s = 0; s < R::KW; ++s) {
#pragma unroll
                        for (int k = 0; k < 6; ++k)
#pragma unroll
                            for (int nb = 0; nb < R::NB; ++nb)
                                acc[nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x[s][px[k]], w[s][nb][pw[k]], acc[nb], 0, 0, 0);
                        __builtin_amdgcn_sched_barrier(0);
                        if (t == 0) load_x(s, 1);         // (one tile a group: read, not used)
                    }
                    floatx4 *p = part_of(i - 1, t) + wave * R::NB * 64 + lane;
#pragma unroll
                    for (int nb = 0; nb < R::NB; ++nb) p[nb * 64] = acc[nb];
                }
            }
            lds_barrier();
        }
    } else if (wave < 6) {
        const int t = wave - 4;
        const int mine = t < G ? (rr.count - t + G - 1) / G : 0;
        const int mrow = lane & 15, kq = lane >> 4;
        int c0 = 0;
        uint32_t w0 = word_chunk<DENSE>(a, rr, t, G, 0, lane);
        uint32_t w1 = word_chunk<DENSE>(a, rr, t, G, 1, lane);
        // Head weights of a position for NQ logits from o0 on (indices clamped).
        // The first ones stay in registers while the position is the same, and
        // are loaded at the previous tile's end when it changes.
        const int n_out = NO >= 0 ? NO : a.n_out, ntiles = a.TH * a.TW;
        constexpr int NQ = NO == 6 ? 6 : 4;
        floatx4 hw[NO == 0 ? 1 : NQ][R::NB];
        auto load_hw = [&](int tile, int o0) __attribute__((always_inline)) {
            if constexpr (NO != 0) {
#pragma unroll
                for (int q = 0; q < NQ; ++q) {
                    const floatx4 *src = reinterpret_cast<const floatx4 *>(
                                             a.hw + ((size_t)min(o0 + q, n_out - 1) * ntiles + tile) * kTilePx * R::COUT) + lane;
#pragma unroll
                    for (int nb = 0; nb < R::NB; ++nb) hw[q][nb] = src[nb * 64];
                }
            }
        };
        int held = -1;                                    // position of the weights in hw, o0 = 0
        if (mine > 0) load_hw(held = item_of(a, w0, w1, 0, 0).tile, 0);
        for (int i = 0; i < groups + 2; ++i) {
            const int k = i - 2;
            if (k >= 0 && k < mine) {
                if (k >= 64 * (c0 + 1)) {
                    w0 = w1;
                    ++c0;
                    w1 = word_chunk<DENSE>(a, rr, t, G, c0 + 1, lane);
                }
                floatx4 *p = part_of(k, t) + lane;
                // Sums and bias; `least` is below 0 where a result is near 0,
                // `most` is not finite where one is not.
                floatx4 acc[R::NB];
                float least = 0.f, most = 0.f;
#pragma unroll
                for (int nb = 0; nb < R::NB; ++nb) {
                    const floatx4 q0 = p[nb * 64], q3 = p[(3 * R::NB + nb) * 64];
                    acc[nb] = q0 + p[(R::NB + nb) * 64] + p[(2 * R::NB + nb) * 64] + q3;
                    acc[nb] += s_bias[nb * 16 + mrow];
                    float small = fabsf(acc[nb][0]);
#pragma unroll
                    for (int e = 1; e < 4; ++e) small = fminf(small, fabsf(acc[nb][e]));
                    if constexpr (!VAR) least = fminf(least, fmaf(column_size(q0, q3), -kNearZero, small));
#pragma unroll
                    for (int e = 0; e < 4; ++e) most = __builtin_elementwise_maximum(most, fabsf(acc[nb][e]));
                }
                const TileRef r = item_of(a, w0, w1, c0, k);
                const int col_keep = ~((a.W - 1 - (r.tx * kTile + kq)) >> 31);
                if (__builtin_expect(__any(!is_finite(most) || least < 0.f), 0)) {
                    // Results inside the image to be taken again, bit 4 nb + e.
                    uint32_t lost = 0, near = 0;
                    int ln = lane;
                    asm volatile("" : "+v"(ln));          // what follows is computed here, not kept in registers throughout
                    const float *bias = s_bias + (ln & 15);
#pragma unroll
                    for (int nb = 0; nb < R::NB; ++nb) {
                        __builtin_amdgcn_sched_barrier(0);   // one block's partial products in registers at a time
                        const float size = column_size(p[nb * 64], p[(3 * R::NB + nb) * 64]);
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const uint32_t bit = (col_keep & ~((a.H - 1 - (r.ty * kTile + e)) >> 31)) & (1 << (4 * nb + e));
                            if (!is_finite(acc[nb][e])) lost |= bit;
                            acc[nb][e] = __builtin_isnan(acc[nb][e]) ? __uint_as_float(0x7fc00000u) : acc[nb][e];   // of either sign
                            if (!VAR && is_finite(acc[nb][e]) && fmaf(size, -kNearZero, fabsf(acc[nb][e])) < 0.f) near |= bit;
                        }
                    }
                    __builtin_amdgcn_sched_barrier(0);
                    asm volatile("" : "+v"(lost), "+v"(near));
#pragma unroll
                    for (int nb = 0; nb < R::NB; ++nb) lost &= __builtin_isnan(bias[nb * 16]) ? ~(15u << (4 * nb)) : ~0u;
                    if (__any((lost | near) != 0)) {      // not so where every such channel has a NaN weight
                        // The results wait in LDS, in place of the first partial
                        // products (head weights and plain sums fill the registers).
#pragma unroll
                        for (int nb = 0; nb < R::NB; ++nb) p[nb * 64] = acc[nb];
                        float *z = reinterpret_cast<float *>(p);
                        if (__any(lost != 0)) {
                            floatx4 lead[R::NB];
                            res_lead(static_cast<const bf16x8 *>(a.w_split), halo_of(k, t), lead, ln);
#pragma unroll
                            for (int nb = 0; nb < R::NB; ++nb)
#pragma unroll
                                for (int e = 0; e < 4; ++e) {
                                    const float b = bias[nb * 16], v = lead[nb][e] + b;
                                    if ((lost >> (4 * nb + e) & 1) && !(is_finite(lead[nb][e]) && is_finite(b))) {
                                        z[nb * 256 + e] = __builtin_isnan(v) ? __uint_as_float(0x7fc00000u) : v;
                                        lost &= ~(1u << (4 * nb + e));
                                    }
                                }
                        }
                        int n_lost = 0, n_near = 0;
#pragma unroll
                        for (int j = 0; j < 4 * R::NB; ++j) {
                            n_lost += __popcll(__ballot(lost >> j & 1));
                            n_near += __popcll(__ballot(near >> j & 1));
                        }
                        if (n_near <= kMostSingle) lost |= near;
                        if (n_lost > kMostSingle) {
                            floatx4 plain[R::NB];
                            res_plain(static_cast<const float *>(a.w), halo_of(k, t), plain, ln);
#pragma unroll
                            for (int nb = 0; nb < R::NB; ++nb)
#pragma unroll
                                for (int e = 0; e < 4; ++e)
                                    if (lost >> (4 * nb + e) & 1) z[nb * 256 + e] = plain[nb][e] + bias[nb * 16];
                        } else {
                            float *pairs = reinterpret_cast<float *>(lds + R::OPAIRS) + t * R::PAIRS;
#pragma unroll 1
                            for (int j = 0; j < 4 * R::NB; ++j) {
                                uint64_t which = __ballot(lost >> j & 1);
                                const int nb = j >> 2, e = j & 3;
                                while (which) {               // lane i: channel nb * 16 + i % 16, pixel (e, i / 16)
                                    const int i = __ffsll((long long)which) - 1;
                                    which &= which - 1;
                                    const float f = res_plain_one(static_cast<const float *>(a.w), halo_of(k, t), pairs,
                                                                  nb * 16 + (i & 15), e, i >> 4, ln);
                                    if (lane == i) z[nb * 256 + e] = f + bias[nb * 16];
                                }
                            }
                        }
                        wave_sync();
#pragma unroll
                        for (int nb = 0; nb < R::NB; ++nb) acc[nb] = p[nb * 64];
                    }
                }
                // As epilogue(), with the head weights in registers already.
                const int widx = rr.at(t + k * G);
#pragma unroll
                for (int nb = 0; nb < R::NB; ++nb)
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[nb][e] = __int_as_float(max(__float_as_int(acc[nb][e]), 0));
                if ((r.ty + 1) * kTile > a.H || (r.tx + 1) * kTile > a.W) {   // uniform: pixels outside the image
#pragma unroll
                    for (int nb = 0; nb < R::NB; ++nb)
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const int keep = col_keep & ~((a.H - 1 - (r.ty * kTile + e)) >> 31);
                            acc[nb][e] = __int_as_float(__float_as_int(acc[nb][e]) & keep);
                        }
                }
                if constexpr (NO != 0) {
                    for (int o0 = 0; o0 < n_out; o0 += NQ) {
                        if (o0 > 0) {
                            load_hw(r.tile, o0);
                            held = -1;
                        }
                        float d[8];
#pragma unroll
                        for (int q = 0; q < 8; ++q) {
                            d[q] = 0.f;
                            if (q >= NQ) continue;
#pragma unroll
                            for (int nb = 0; nb < R::NB; ++nb)
#pragma unroll
                                for (int e = 0; e < 4; ++e) d[q] = fmaf(acc[nb][e], hw[q][nb][e], d[q]);
                        }
                        const float v = lane_sums8(d, lane);
                        const int q = (lane >> 5) * 4 + ((lane >> 4) & 1) * 2 + ((lane >> 3) & 1);
                        if ((lane & 7) == 0 && q < NQ && o0 + q < n_out) {
                            float *hp = VAR ? a.vhpart + (size_t)widx * n_out
                                            : a.hpart + ((size_t)r.slot * ntiles + r.tile) * n_out;
                            hp[o0 + q] = v;
                        }
                    }
                    if (k + 1 < mine) {
                        const int next = item_of(a, w0, w1, c0, k + 1).tile;
                        if (next != held) load_hw(held = next, 0);
                    }
                }
                if (!VAR || n_out == 0) {
                    // 16 channels (64 bytes) of four pixels a store, straight
                    // from the registers.
                    float *dst = (VAR ? static_cast<float *>(a.vov_out) + (size_t)widx * kTilePx * R::COUT
                                      : static_cast<float *>(a.out) + (size_t)r.slot * a.out_stride +
                                            (size_t)r.tile * kTilePx * R::COUT) + kq * R::COUT + mrow;
#pragma unroll
                    for (int nb = 0; nb < R::NB; ++nb)
#pragma unroll
                        for (int e = 0; e < 4; ++e) dst[e * 4 * R::COUT + nb * 16] = acc[nb][e];
                }
            }
            lds_barrier();
        }
    } else {
        const int t = wave - 6;
        const int c4 = lane % 10, hy = lane / 10;         // lanes 60 to 63: none
        int c0 = 0;
        uint32_t w0 = word_chunk<DENSE>(a, rr, t, G, 0, lane);
        uint32_t w1 = word_chunk<DENSE>(a, rr, t, G, 1, lane);
        auto has = [&](int k) { return t < G && t + k * G < rr.count; };
        float wr[FUSE ? 9 : 1][4], br[4], pin = 0.f;
        float *patch = s_patch + t * 64;
        if constexpr (FUSE) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
#pragma unroll
                for (int q = 0; q < 9; ++q) wr[q][e] = a.w1[q * R::CIN + 4 * c4 + e];
                br[e] = a.b1[4 * c4 + e];
            }
        }
        floatx4 pre[6];
        // Input of group k's tile into registers: the patch, or the halo row.
        auto fetch = [&](const TileRef &r) __attribute__((always_inline)) {
            if constexpr (FUSE) {
                pin = fetch_patch<VAR>(a, r, lane);
            } else {
                const int y = r.ty * kTile - 1 + hy;
#pragma unroll
                for (int hx = 0; hx < 6; ++hx) {
                    const int x = r.tx * kTile - 1 + hx;
                    pre[hx] = floatx4{0.f, 0.f, 0.f, 0.f};
                    if (hy < 6 && y >= 0 && y < a.H && x >= 0 && x < a.W) {
                        const float *src =
                            VAR ? var_src<float>(a, r.slot, y, x, R::CIN)
                                : static_cast<const float *>(a.in) + (size_t)r.slot * a.in_stride +
                                      ((size_t)((y >> 2) * a.TW + (x >> 2)) * kTilePx + (y & 3) * 4 + (x & 3)) * R::CIN;
                        pre[hx] = *reinterpret_cast<const floatx4 *>(src + 4 * c4);
                    }
                }
            }
        };
        if (has(0)) fetch(item_of(a, w0, w1, c0, 0));
        for (int i = 0; i < groups + 2; ++i) {
            if (has(i)) {
                if (i >= 64 * (c0 + 1)) {
                    w0 = w1;
                    ++c0;
                    w1 = word_chunk<DENSE>(a, rr, t, G, c0 + 1, lane);
                }
                const TileRef r = item_of(a, w0, w1, c0, i);
                unsigned char *h = halo_of(i, t) + hy * R::ROW + c4 * 8;
                floatx4 v[6];
                if constexpr (FUSE) {
                    patch[lane] = pin;
                    wave_sync();
                    if (has(i + 1)) fetch(item_of(a, w0, w1, c0, i + 1));
                    float p[3][8];
#pragma unroll
                    for (int ky = 0; ky < 3; ++ky)
#pragma unroll
                        for (int x = 0; x < 8; ++x) p[ky][x] = patch[min(hy + ky, 7) * 8 + x];
#pragma unroll
                    for (int hx = 0; hx < 6; ++hx)
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            float acc = 0.0f;
#pragma unroll
                            for (int ky = 0; ky < 3; ++ky)
#pragma unroll
                                for (int kx = 0; kx < 3; ++kx) acc = fmaf(wr[ky * 3 + kx][e], p[ky][hx + kx], acc);
                            const float z = acc + br[e];
                            v[hx][e] = z > 0.0f ? z : 0.0f;
                        }
                    // The halo's pixels outside the image (edge tiles only) are 0.
                    const int y0 = r.ty * kTile - 1, x0 = r.tx * kTile - 1;
                    if (y0 < 0 || x0 < 0 || y0 + 6 > a.H || x0 + 6 > a.W) {
#pragma unroll
                        for (int hx = 0; hx < 6; ++hx)
                            if (y0 + hy < 0 || y0 + hy >= a.H || x0 + hx < 0 || x0 + hx >= a.W)
                                v[hx] = floatx4{0.f, 0.f, 0.f, 0.f};
                    }
                    wave_sync();                          // patch reads done before the next tile's write
                } else {
#pragma unroll
                    for (int hx = 0; hx < 6; ++hx) v[hx] = pre[hx];
                    if (has(i + 1)) fetch(item_of(a, w0, w1, c0, i + 1));
                }
                float big = 0.f;
#pragma unroll
                for (int hx = 0; hx < 6; ++hx)
#pragma unroll
                    for (int e = 0; e < 4; e += 2) big = fmaxf(fmaxf(fabsf(v[hx][e]), fabsf(v[hx][e + 1])), big);
                const bool wide = __any(big >= kWide);
                if (hy < 6) {
#pragma unroll
                    for (int hx = 0; hx < 6; ++hx) {
                        bf16x4 q[3];
                        if (wide) split4_any(v[hx], q[0], q[1], q[2]);
                        else split4(v[hx], q[0], q[1], q[2]);
#pragma unroll
                        for (int pl = 0; pl < 3; ++pl) *reinterpret_cast<bf16x4 *>(h + pl * R::PLANE + hx * 80) = q[pl];
                    }
                }
            }
            lds_barrier();
        }
    }
}

// The split weights in the order the waves hold them, [k-step][16-channel
// block][plane][lane][8], from the float32 packing.
// The waves past those take a channel each: NaN if one of its weights is, else 0.
__global__ void k_pack_res(const float *w, __bf16 *dst) {
    using R = Res;
    const int u = blockIdx.x * blockDim.x + threadIdx.x;  // (k-step, block, lane)
    const int n = (u - R::KS * R::NB * 64) / 64, ln = u & 63;
    if (n >= R::COUT) return;
    if (u >= R::KS * R::NB * 64) {                        // uniform per wave
        float nan = 0.f;
        for (int kpos = 0; kpos < 9; ++kpos)
            if (ln < R::CIN) {
                const int blk = ln / 16, steps = blk < 2 ? 4 : 2, c = ln - 16 * blk;
                const float v = w[kpos * R::CIN * R::COUT + blk * 16 * R::COUT + (n / 16 * 64 + c / steps * 16 + n % 16) * steps + c % steps];
                nan = __builtin_isnan(v) ? v : nan;
            }
        const bool any = __any(__builtin_isnan(nan));
        if (ln == 0) reinterpret_cast<float *>(reinterpret_cast<unsigned char *>(dst) + R::w_bytes)[n] = any ? __uint_as_float(0x7fc00000u) : 0.f;
        return;
    }
    const int l = u & 63, nb = u / 64 % R::NB, s = u / 64 / R::NB;
    const int g = 4 * s + (l >> 4), kpos = g / 5;
    for (int q = 0; q < 2; ++q) {
        floatx4 v{0.f, 0.f, 0.f, 0.f};
        for (int e = 0; e < 4; ++e) {
            const int c = 8 * (g - 5 * kpos) + 4 * q + e, blk = c / 16, steps = blk < 2 ? 4 : 2;
            const int lw = (c - 16 * blk) / steps * 16 + (l & 15);
            if (g < R::OCT)
                v[e] = w[kpos * R::CIN * R::COUT + blk * 16 * R::COUT + (nb * 64 + lw) * steps + c % steps];
        }
        bf16x4 p[3];
        split4_any(v, p[0], p[1], p[2]);
        for (int pl = 0; pl < 3; ++pl)
            *reinterpret_cast<bf16x4 *>(dst + ((size_t)((s * R::NB + nb) * 3 + pl) * 64 + l) * 8 + 4 * q) = p[pl];
    }
}

// Operands of one 16-channel block: the A fragments of the T tiles and the B
// fragments of the wave's NBW output blocks.
template <int T, int NBW>
struct SplitOps {
    float4 a[T];
    float4 b[NBW];
};

// ---- weights too large for LDS (64->128, 128->128) on the float32 matrix instructions
//
// The form of nets with RN_OPT_SEPARATE_FIRST, the option training uses: the
// gradient depends on which side of 0 each pre-activation lies, so training
// keeps the plain float32 sums (the split form of rn_conv_split.hip rounds
// differently, and in layers that feed another a decision can then fall the
// other way); a training step of 24 106x92 streams spends about 12% of its time
// here.  Variants (VAR) take the same sums as the net's steps.
//
// A block of four waves computes a group of T tiles, each wave COUT / 4 output
// channels of all of them, walking K one 16-channel chunk at a time and, within
// a chunk, the nine kernel positions (a stage = one position of one chunk:
// 4 k-steps x T x COUT / 64 matrix ops per wave).  Only three chunks of the
// group's halos are in LDS at once: chunk K is read, K + 1 is ready, K + 2 is
// in flight, each loaded straight from global memory into LDS with
// global_load_lds_dwordx4 (lane i writes 16 bytes at base + 16 i, so the
// lanes' source addresses lay out the buffer: tile t's 6 x 6 pixels x 4
// channel quads at 16-byte slot 144 t + 24 hy + 4 hx + quad; pixels outside
// the image and tiles past the end load from a zero page).  Rows padded to
// 25 or 27 slots, which put the 16 pixels of a 16-lane read in 16 distinct
// bank groups, measured no faster and with the same bank-conflict count.
// The stage sequence runs on across groups: when a chunk's last stage starts,
// the waves have read all of it, so after one block barrier it is refilled
// with the chunk three ahead (the next group's when the group runs out), 18
// stages before it is read.  Weights stream per stage through a ring of five
// LDS slots per wave (stage q + 4 loaded at the start of stage q) and each
// stage's operands are read during the previous stage's matrix ops.  The
// memory counter the waits use retires loads and stores in issue order, so
// every wait names how many later operations it may leave in flight; the work
// items are loaded into LDS the same way, and the only loads the compiler
// issues (the bias) are waited for before the first ring load.  The epilogue
// applies bias, ReLU and the zero outside the image, transposes each lane
// quad's 4 x 4 values with DPP moves so a lane holds four channels of one
// pixel, and stores 16 bytes a lane straight to the cache.  The order of the
// sums over K (chunk, then position, then channel) is the same for every T,
// so a tile's outputs do not depend on the group size a launch picks.
template <int CIN, int COUT, int T>
struct Chunked {
    static constexpr int NCH = CIN / 16;             // 16-channel chunks
    static constexpr int NQ = 9 * NCH;               // stages per group
    static constexpr int NB = COUT / 16;             // 16-output blocks
    static constexpr int NBW = COUT / 64;            // 16-output blocks per wave
    static constexpr int CW = 16 * NBW;              // output channels per wave
    static constexpr int WSW = 16 * CW;              // weight floats per stage and wave
    static constexpr int NWB = 5;                    // weight ring slots per wave
    static constexpr int WL = NWB - 2;               // stages between a weight load and its wait
    static constexpr int RS = 24;                    // 16-byte slots per halo row
    static constexpr int HT = 6 * RS;                // slots per tile of a chunk buffer
    static constexpr int HD = (T * HT * 16 + 1023) / 1024;   // 1 KB loads per chunk buffer
    static constexpr int HB = HD * 1024;             // bytes per chunk buffer
    static constexpr int HDW = (HD + 3) / 4;         // most loads of one wave per chunk
    static constexpr int HDMIN = HD / 4;             // fewest
    static constexpr int NS = T * NBW;               // 16-byte-a-lane stores per group and wave
    static constexpr size_t lds_bytes = 3 * (size_t)HB + (size_t)4 * NWB * WSW * sizeof(float) + 4 * 256;
    static_assert(CIN % 16 == 0 && COUT % 64 == 0 && NCH >= 4, "whole chunks, at least four per group");
    static_assert(WSW == 256 * NBW, "one 1 KB load per output block and stage");
    static_assert(T <= 16 && T % 4 == 0, "group size");
    static_assert(WL >= 2 && WL <= 8 && WL * NBW + HDMIN + NS <= 63, "the stage waits below assume these");
};

// Zero page (512 bytes): the source of every halo slot that holds no input
// value (chunk c reads 16 c floats further on).
__device__ __align__(16) float g_zero_page[128];

// Work items of a group, staged per wave in LDS: lane u loads the word of
// tile g + u (clamped to the last item) straight into the wave's item slot
// (global_load_lds_dword), so no register is written behind the compiler's
// back and the load is counted with the ring loads; in dense mode the words
// loaded are the stream ids and the positions are computed on reading.
template <bool DENSE>
__device__ inline const uint32_t *item_src(const ConvArgs &a, int t) {
    if constexpr (DENSE) {
        constexpr int CH = 32;                            // as item_word<true>
        const int per_chunk = CH * a.TH * a.TW;
        const int c = t / per_chunk, rr = t - c * per_chunk;
        const int nc = min(CH, a.dense_n - c * CH);
        const int tile = rr / nc;
        return reinterpret_cast<const uint32_t *>(a.ids) + c * CH + (rr - tile * nc);
    } else {
        return a.wl + t;
    }
}

template <bool DENSE>
__device__ inline uint32_t item_from(const ConvArgs &a, int t, uint32_t raw) {
    if constexpr (DENSE) {
        constexpr int CH = 32;
        const int per_chunk = CH * a.TH * a.TW;
        const int c = t / per_chunk, rr = t - c * per_chunk;
        const int nc = min(CH, a.dense_n - c * CH);
        const int tile = rr / nc;
        const int ty = tile / a.TW;
        return (raw << 16) | ((uint32_t)ty << 8) | (uint32_t)(tile - ty * a.TW);
    } else {
        return raw;
    }
}

template <bool DENSE, int T>
__device__ inline void dma_items(const ConvArgs &a, int g, int end, uint32_t dst, int lane) {
    lds_dma4(item_src<DENSE>(a, min(g + min(lane, T - 1), end - 1)), dst);
}

// Source of each of this wave's halo loads for chunk 0 of the group at g.  (The
// loads that VAR's look-ups take are waited for here, so the counts above hold.)
template <int CIN, int COUT, int T, bool DENSE, bool VAR>
__device__ inline void chunk_sources(const ConvArgs &a, int g, int end, const uint32_t *items,
                                     const float *(&src)[Chunked<CIN, COUT, T>::HDW], int wave, int lane) {
    using C = Chunked<CIN, COUT, T>;
    const float *in = static_cast<const float *>(a.in);
#pragma unroll
    for (int k = 0; k < C::HDW; ++k) {
        const int s = 64 * (wave + 4 * k) + lane;
        const int t = s / C::HT, rem = s - t * C::HT;
        const int hy = rem / C::RS, r2 = rem - hy * C::RS;
        const int hx = r2 >> 2, kq = r2 & 3;
        const int tc = min(t, T - 1);
        const TileRef r = item_ref(a, item_from<DENSE>(a, min(g + tc, end - 1), items[tc]));
        const int y = r.ty * kTile - 1 + hy, x = r.tx * kTile - 1 + hx;
        const bool ok = t < T && g + t < end && r2 < 24 && y >= 0 && y < a.H && x >= 0 && x < a.W;
        if constexpr (VAR)
            src[k] = (ok ? var_src<float>(a, r.slot, y, x, CIN) : g_zero_page) + 4 * kq;
        else
            src[k] = ok ? in + (size_t)r.slot * a.in_stride +
                              ((size_t)((y >> 2) * a.TW + (x >> 2)) * kTilePx + (y & 3) * 4 + (x & 3)) * CIN + 4 * kq
                        : g_zero_page + 4 * kq;
    }
}

// Chunk c of the halos into the chunk buffer at LDS byte address dst.
template <int CIN, int COUT, int T>
__device__ inline void dma_chunk(const float *const (&src)[Chunked<CIN, COUT, T>::HDW], int c, uint32_t dst,
                                 int wave) {
    using C = Chunked<CIN, COUT, T>;
#pragma unroll
    for (int k = 0; k < C::HDW; ++k) {
        const int j = wave + 4 * k;
        if (k + 1 < C::HDW || j < C::HD) lds_dma16(src[k] + 16 * c, dst + 1024u * j);
    }
}

// Stage s (chunk s / 9, position s % 9) of this wave's weights into the ring
// slot at LDS byte address dst, [output block][lane][4].
template <int CIN, int COUT, int T>
__device__ inline void dma_wchunk(const float *wg, int s, uint32_t dst, int wave, int lane) {
    using C = Chunked<CIN, COUT, T>;
    const int c = s / 9, kpos = s - 9 * c;
#pragma unroll
    for (int nb = 0; nb < C::NBW; ++nb)
        lds_dma16(wg + ((size_t)(kpos * C::NCH + c) * C::NB + wave * C::NBW + nb) * 256 + 4 * lane,
                  dst + 1024u * nb);
}

// A fragments of the T tiles at kernel position kpos from the chunk buffer
// (hb: this lane's slot of tile 0, position 0) and the B fragments of the
// stage's ring slot (wb: this lane's 16 bytes of output block 0).
template <int CIN, int COUT, int T>
__device__ inline void chunk_ops(SplitOps<T, Chunked<CIN, COUT, T>::NBW> &o, const float *hb, const float *wb,
                                 int kpos) {
    using C = Chunked<CIN, COUT, T>;
    const int ky = kpos / 3, kx = kpos - 3 * ky;
#pragma unroll
    for (int t = 0; t < T; ++t)
        o.a[t] = *reinterpret_cast<const float4 *>(hb + 4 * (t * C::HT + ky * C::RS + kx * 4));
#pragma unroll
    for (int nb = 0; nb < C::NBW; ++nb) o.b[nb] = *reinterpret_cast<const float4 *>(wb + 256 * nb);
}

// Parts of a stage, issued interleaved: A fragments of tiles [t0, t1), the
// B fragments, and the matrix ops of one k-step (the order of the matrix ops
// over a stage is that of split_mma).
template <int CIN, int COUT, int T, int T0, int T1>
__device__ inline void chunk_ops_a(SplitOps<T, Chunked<CIN, COUT, T>::NBW> &o, const float *hb, int kpos) {
    using C = Chunked<CIN, COUT, T>;
    const int ky = kpos / 3, kx = kpos - 3 * ky;
#pragma unroll
    for (int t = T0; t < T1; ++t)
        o.a[t] = *reinterpret_cast<const float4 *>(hb + 4 * (t * C::HT + ky * C::RS + kx * 4));
}

template <int CIN, int COUT, int T>
__device__ inline void chunk_ops_b(SplitOps<T, Chunked<CIN, COUT, T>::NBW> &o, const float *wb) {
#pragma unroll
    for (int nb = 0; nb < Chunked<CIN, COUT, T>::NBW; ++nb) o.b[nb] = *reinterpret_cast<const float4 *>(wb + 256 * nb);
}

template <int T, int NBW, int J>
__device__ inline void mma_kstep(floatx4 (&acc)[T][NBW], const SplitOps<T, NBW> &o) {
#pragma unroll
    for (int t = 0; t < T; ++t) {
        const float av = J == 0 ? o.a[t].x : J == 1 ? o.a[t].y : J == 2 ? o.a[t].z : o.a[t].w;
#pragma unroll
        for (int nb = 0; nb < NBW; ++nb) {
            const float bv = J == 0 ? o.b[nb].x : J == 1 ? o.b[nb].y : J == 2 ? o.b[nb].z : o.b[nb].w;
            acc[t][nb] = __builtin_amdgcn_mfma_f32_16x16x4f32(av, bv, acc[t][nb], 0, 0, 0);
        }
    }
}

// 4 x 4 transpose inside each lane quad: lane 4 m + b holds v[i] = X[i][b] on
// entry and X[b][i] on return (two exchanges, over lane bit 0 with element
// bit 0, then over lane bit 1 with element bit 1).
__device__ inline void quad_transpose(float (&v)[4], int b) {
    {
        const bool hi = b & 1;
        const float s0 = hi ? v[0] : v[1], s1 = hi ? v[2] : v[3];
        const float r0 = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(s0), 0xb1, 0xf, 0xf, false));
        const float r1 = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(s1), 0xb1, 0xf, 0xf, false));
        if (hi) {
            v[0] = r0;
            v[2] = r1;
        } else {
            v[1] = r0;
            v[3] = r1;
        }
    }
    {
        const bool hi = b & 2;
        const float s0 = hi ? v[0] : v[2], s1 = hi ? v[1] : v[3];
        const float r0 = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(s0), 0x4e, 0xf, 0xf, false));
        const float r1 = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(s1), 0x4e, 0xf, 0xf, false));
        if (hi) {
            v[0] = r0;
            v[1] = r1;
        } else {
            v[2] = r0;
            v[3] = r1;
        }
    }
}

template <int CIN, int COUT, bool DENSE, bool VAR, int T>
__device__ void chunk_path(const ConvArgs &a, int cnt, float *smem) {
    using C = Chunked<CIN, COUT, T>;
    constexpr int NBW = C::NBW;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const XcdRange xr = xcd_range(cnt, T);
    if (xr.first >= xr.end) return;                       // uniform per block
    const int mrow = lane & 15, kq = lane >> 4;
    unsigned char *lds = reinterpret_cast<unsigned char *>(smem);
    float *wring = reinterpret_cast<float *>(lds + 3 * C::HB) + wave * C::NWB * C::WSW;
    const uint32_t *items = reinterpret_cast<const uint32_t *>(lds + 3 * C::HB + 4 * C::NWB * C::WSW * 4) + 64 * wave;
    const uint32_t hlds = lds_addr(lds), wlds = lds_addr(wring), ilds = lds_addr(items);
    const float *wg = static_cast<const float *>(a.w);
    // this lane's A slot (halo pixel (mrow & 3, mrow >> 2), channel quad kq) and B slot
    const float *ha = reinterpret_cast<const float *>(lds) + 4 * ((mrow & 3) * C::RS + (mrow >> 2) * 4 + kq);
    const float *wa = wring + 4 * lane;

    // Bias of the lane's output channels, waited for before any ring load.
    float bias[NBW];
#pragma unroll
    for (int nb = 0; nb < NBW; ++nb) bias[nb] = a.bias[wave * C::CW + nb * 16 + mrow];
    asm volatile("" ::"v"(bias[0]), "v"(bias[NBW - 1]));

    // Prologue: halo chunks 0-2 and weight stages 0 .. NWB - 2 of the first group.
    const float *src[C::HDW];
    dma_items<DENSE, T>(a, xr.first, xr.end, ilds, lane);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    chunk_sources<CIN, COUT, T, DENSE, VAR>(a, xr.first, xr.end, items, src, wave, lane);
#pragma unroll
    for (int k = 0; k < 3; ++k) dma_chunk<CIN, COUT, T>(src, k, hlds + k * C::HB, wave);
#pragma unroll
    for (int q = 0; q < C::NWB - 1; ++q) dma_wchunk<CIN, COUT, T>(wg, q, wlds + q * C::WSW * 4, wave, lane);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    lds_barrier();

    int hk = 0;                                           // chunk buffer of the current chunk
    int qs = 0;                                           // ring slot of the current stage
    int dc = 3;                                           // next chunk to load (of the group at g, or, once
                                                          // past NCH, of the next group)
    SplitOps<T, NBW> cur;
    chunk_ops<CIN, COUT, T>(cur, ha, wa, 0);
    for (int g = xr.first; g < xr.end; g += xr.stride) {   // uniform per block
        const bool stores_before = g != xr.first;         // the previous group's stores are in flight
        floatx4 acc[T][NBW];
#pragma unroll
        for (int t = 0; t < T; ++t)
#pragma unroll
            for (int nb = 0; nb < NBW; ++nb) acc[t][nb] = floatx4{0.f, 0.f, 0.f, 0.f};
        for (int c = 0; c < C::NCH; ++c) {
#pragma unroll
            for (int kp = 0; kp < 9; ++kp) {
                if (kp == 8) {
                    // This chunk's reads are done in every wave, chunk + 1 is
                    // in LDS: its loads (issued two chunks ago) are followed
                    // by 17 stages' weight loads and one chunk's halo loads.
                    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(17 * NBW + C::HDMIN) : "memory");
                    lds_barrier();
                }
                // Matrix ops of this stage, one k-step at a time, with the
                // rest of the stage's work in between so the matrix pipe is
                // never left waiting on a burst of other instructions: stage
                // q + NWB - 1's weights into the slot stage q - 1 used (its
                // reads fed matrix ops that have issued), at a chunk boundary
                // the item and halo loads, and the next stage's operands,
                // its weights once they are in: they were loaded WL stages
                // ago and are followed by WL stages' weight loads, plus a
                // chunk's halo loads when a chunk boundary is that close,
                // plus the previous group's stores at a group's start.
                SplitOps<T, NBW> nxt;
                const int qn = qs + 1 == C::NWB ? 0 : qs + 1;
                const int hn = kp == 8 ? (hk + 1 == 3 ? 0 : hk + 1) : hk;
                const int kn = kp == 8 ? 0 : kp + 1;
                mma_kstep<T, NBW, 0>(acc, cur);
                __builtin_amdgcn_sched_barrier(0);
                const int s4 = c * 9 + kp + C::NWB - 1;
                dma_wchunk<CIN, COUT, T>(wg, s4 >= C::NQ ? s4 - C::NQ : s4,
                                         wlds + ((qs + C::NWB - 1) % C::NWB) * C::WSW * 4, wave, lane);
                if (kp == 8) {
                    // The wave's item slot: the next group's items a chunk
                    // before its halo sources are needed, then this group's
                    // for the epilogue (each followed by this boundary's halo
                    // loads and the next nine stages' weight loads).
                    const int gn = min(g + xr.stride, xr.end - 1);
                    if (c == C::NCH - 4) dma_items<DENSE, T>(a, gn, xr.end, ilds, lane);
                    if (c == C::NCH - 2) dma_items<DENSE, T>(a, g, xr.end, ilds, lane);
                    // Refill this chunk's buffer with the chunk three ahead.
                    if (dc == C::NCH) {                       // on to the next group
                        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(9 * NBW + C::HDMIN) : "memory");
                        chunk_sources<CIN, COUT, T, DENSE, VAR>(a, g + xr.stride, xr.end, items, src, wave, lane);
                        dc = 0;
                    }
                    dma_chunk<CIN, COUT, T>(src, dc, hlds + hk * C::HB, wave);
                    ++dc;
                }
                chunk_ops_a<CIN, COUT, T, 0, T / 2>(nxt, ha + hn * (C::HB / 4), kn);
                __builtin_amdgcn_sched_barrier(0);
                mma_kstep<T, NBW, 1>(acc, cur);
                __builtin_amdgcn_sched_barrier(0);
                chunk_ops_a<CIN, COUT, T, T / 2, T>(nxt, ha + hn * (C::HB / 4), kn);
                __builtin_amdgcn_sched_barrier(0);
                mma_kstep<T, NBW, 2>(acc, cur);
                __builtin_amdgcn_sched_barrier(0);
                if (kp >= C::WL && kp <= 7) {
                    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(C::WL * NBW) : "memory");
                } else if (c == 0 && kp <= C::WL - 1 && stores_before) {
                    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(C::WL * NBW + C::HDMIN + C::NS) : "memory");
                } else {
                    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(C::WL * NBW + C::HDMIN) : "memory");
                }
                chunk_ops_b<CIN, COUT, T>(nxt, wa + qn * C::WSW);
                __builtin_amdgcn_sched_barrier(0);
                mma_kstep<T, NBW, 3>(acc, cur);
                __builtin_amdgcn_sched_barrier(0);
                cur = nxt;
                qs = qn;
                hk = hn;
            }
        }
        // Epilogue: bias, ReLU and the zero outside the image on the bit
        // patterns (a float above zero has a positive int pattern), the quad
        // transpose, 16 bytes a lane: pixel (b, kq) of the tile, channels
        // 16 nb + 4 m .. + 3 of the wave's, for lane 16 kq + 4 m + b.
        const int qb = lane & 3, qm = (lane >> 2) & 3;
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(9 * NBW + 2 * C::HDMIN) : "memory");
#pragma unroll
        for (int t = 0; t < T; ++t) {
            if (g + t >= xr.end) break;                   // uniform
            const TileRef r = item_ref(a, item_from<DENSE>(a, g + t, items[t]));
            const int col_keep = ~((a.W - 1 - (r.tx * kTile + kq)) >> 31);
            float *dst = (VAR ? static_cast<float *>(a.vov_out) + (size_t)(g + t) * kTilePx * COUT
                              : static_cast<float *>(a.out) + (size_t)r.slot * a.out_stride + (size_t)r.tile * kTilePx * COUT) +
                         (qb * 4 + kq) * COUT + wave * C::CW + 4 * qm;
#pragma unroll
            for (int nb = 0; nb < NBW; ++nb) {
                float v[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int keep = col_keep & ~((a.H - 1 - (r.ty * kTile + i)) >> 31);
                    v[i] = __int_as_float(max(__float_as_int(acc[t][nb][i] + bias[nb]), 0) & keep);
                }
                quad_transpose(v, qb);
                *reinterpret_cast<float4 *>(dst + 16 * nb) = make_float4(v[0], v[1], v[2], v[3]);
            }
        }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // loads issued for a group that does not come
}

template <int CIN, int COUT, bool DENSE, bool VAR>
__global__ __launch_bounds__(256) void k_conv_mfma_staged(ConvArgs a) {
    extern __shared__ float smem[];
    // Groups of 8 tiles when every block has at least 16 of them to do, else of 4.
    const int cnt = work_count<DENSE>(a);
    if (cnt >= 16 * 8 * (int)gridDim.x) chunk_path<CIN, COUT, DENSE, VAR, 8>(a, cnt, smem);
    else chunk_path<CIN, COUT, DENSE, VAR, 4>(a, cnt, smem);
}

// ------------------------------------------------------------------ general layers

// Any k x k kernel with stride s and zero padding p <= (k - 1) / 2 (the growth
// rule of Fig. 1 for general k and s; DQN-style trunks: 8x8/4, 4x4/2, 3x3/1
// without padding).  A 4x4 output tile reads an E x E input patch, E = 3 s + k,
// whose corner is input pixel (4 s ty - p, 4 s tx - p); out-of-grid pixels are
// zero.  Implicit GEMM on v_mfma_f32_16x16x4_f32 (operand layout above):
// M = 16 tile pixels (column-major rows), N = COUT, K = k k CIN in (ky, kx, c)
// order, walked in blocks of 16 K values: in block b, k-step j gives lane group
// kq the K index 16 b + 4 kq + j, so a lane's four k-steps are consecutive K
// values (four consecutive channels of one input pixel when CIN % 4 = 0: one
// 16-byte LDS read).  K is padded to a multiple of 16 with zero weights and
// zero A values.  The patch sits in LDS channel-innermost; the weights,
// packed [block][n-block][lane][j], stream from global memory (the same few
// hundred KB for every wave, served by L1/L2), one 16-byte load per lane and
// n-block, three blocks ahead of their use (a ring of three register sets
// with fixed roles, the loop unrolled by three).  A block of four waves works
// on one tile at a time and splits its K blocks four ways (these layers have
// few tiles on their small grids, so a launch lasts about one tile's latency);
// the four partial products are added in LDS in wave order and wave 0 runs
// the epilogue; the next tile's patch is fetched into registers during this
// tile's matrix work;
// the epilogue is the one of the 3x3 kernels (bias, ReLU, zero outside the
// output grid, tile head partials on the last layer, cache store).
// FIRST: the input is the float32 input cache (planar, a ring of 4 frames when
// stacking) instead of a tiled layer cache.
template <int KS, int ST, int CIN, int COUT>
struct Gen {
    static constexpr int E = 3 * ST + KS;
    static constexpr int KT = KS * KS * CIN;
    static constexpr int KSPLIT = 4;                             // waves per tile, each a quarter of K
    static constexpr int NBLK = ((KT + 15) / 16 + 11) / 12 * 12;  // 16-K blocks, padded to 4 x whole triples
    static constexpr int NBW = NBLK / KSPLIT;                    // blocks per wave
    static constexpr int NB = COUT / 16;
    static constexpr int HALO = E * E * CIN;
    static constexpr int STAGE = 16 * Epi<COUT>::SR;
    static constexpr int AREA = HALO > STAGE ? HALO : STAGE;   // floats per wave
    static constexpr int PART = (KSPLIT - 1) * NB * 64 * 4;     // partial products of waves 1..3
    static constexpr size_t lds_bytes = (size_t)(AREA + PART) * sizeof(float);
    static_assert(COUT % 16 == 0, "16-column blocks");
};

// The patch of tile r, thread idx's share (elements idx, idx + 256, ...), in
// registers: PF values per thread (scalars from the input frames, FIRST), or
// PF 16-byte channel groups (cache layers).  Every load is issued before any
// is used; out-of-image elements are zero.
template <int KS, int ST, int CIN, int COUT, bool FIRST>
struct GenPatch {
    using G = Gen<KS, ST, CIN, COUT>;
    static constexpr int N = FIRST ? G::HALO : G::E * G::E * (CIN / 4);   // elements
    static constexpr int PF = (N + 255) / 256;                            // per thread
    using T = typename std::conditional<FIRST, float, float4>::type;
};

template <int KS, int ST, int CIN, int COUT, bool FIRST>
__device__ inline void gen_fetch_patch(const ConvArgs &a, const TileRef &r,
                                       typename GenPatch<KS, ST, CIN, COUT, FIRST>::T *v, int idx) {
    using G = Gen<KS, ST, CIN, COUT>;
    using P = GenPatch<KS, ST, CIN, COUT, FIRST>;
    const int y0 = 4 * ST * r.ty - a.pad, x0 = 4 * ST * r.tx - a.pad;
    if constexpr (FIRST) {
        const float *xin = static_cast<const float *>(a.in);
        const size_t HW = (size_t)a.Hin * a.Win;
        const int cin1 = CIN / a.stack;
        const int head = a.stack != 1 ? a.ring_head[r.slot] : 0;
#pragma unroll
        for (int k = 0; k < P::PF; ++k) {
            const int h = idx + 256 * k;
            const int c = h / (G::E * G::E), pos = h - c * (G::E * G::E);
            const int hy = pos / G::E, hx = pos - hy * G::E;
            const int y = y0 + hy, x = x0 + hx;
            float val = 0.0f;
            if (h < P::N && y >= 0 && y < a.Hin && x >= 0 && x < a.Win) {
                const float *plane;
                if (a.stack == 1) {
                    plane = xin + ((size_t)r.slot * CIN + c) * HW;
                } else {
                    const int j = c / cin1, c1 = c - j * cin1;
                    const int rp = (head - (a.stack - 1) + j + 4 * a.stack) & 3;
                    plane = xin + (((size_t)r.slot * 4 + rp) * cin1 + c1) * HW;
                }
                val = plane[(size_t)y * a.Win + x];
            }
            v[k] = val;
        }
    } else {
        static_assert(CIN % 4 == 0, "cache layers carry whole 16-byte channel groups");
        constexpr int C4 = CIN / 4;
        const float *src = static_cast<const float *>(a.in) + (size_t)r.slot * a.in_stride;
#pragma unroll
        for (int k = 0; k < P::PF; ++k) {
            const int h = idx + 256 * k;
            const int pos = h / C4, c4 = h - pos * C4;
            const int hy = pos / G::E, hx = pos - hy * G::E;
            const int y = y0 + hy, x = x0 + hx;
            float4 val = make_float4(0.f, 0.f, 0.f, 0.f);
            if (h < P::N && y >= 0 && y < a.Hin && x >= 0 && x < a.Win)
                val = *reinterpret_cast<const float4 *>(
                    src + ((size_t)((y >> 2) * a.TWin + (x >> 2)) * kTilePx + (y & 3) * 4 + (x & 3)) * CIN + 4 * c4);
            v[k] = val;
        }
    }
}

// The fetched patch into LDS, channel-innermost.
template <int KS, int ST, int CIN, int COUT, bool FIRST>
__device__ inline void gen_store_patch(float *halo, const typename GenPatch<KS, ST, CIN, COUT, FIRST>::T *v, int idx) {
    using G = Gen<KS, ST, CIN, COUT>;
    using P = GenPatch<KS, ST, CIN, COUT, FIRST>;
#pragma unroll
    for (int k = 0; k < P::PF; ++k) {
        const int h = idx + 256 * k;
        if (h >= P::N) break;
        if constexpr (FIRST) {
            const int c = h / (G::E * G::E), pos = h - c * (G::E * G::E);
            halo[pos * CIN + c] = v[k];
        } else {
            constexpr int C4 = CIN / 4;
            const int pos = h / C4, c4 = h - pos * C4;
            *reinterpret_cast<float4 *>(halo + pos * CIN + 4 * c4) = v[k];
        }
    }
}


// A values of block b for this lane: K = 16 b + 4 kq + j, j = 0..3, of tile
// pixel (py, px).
template <int KS, int ST, int CIN, int COUT>
__device__ inline float4 gen_a(const float *halo, int b, int kq, int py, int px) {
    using G = Gen<KS, ST, CIN, COUT>;
    const int K0 = 16 * b + 4 * kq;
    if constexpr (CIN % 4 == 0) {
        if (K0 >= G::KT) return make_float4(0.f, 0.f, 0.f, 0.f);
        const int kpos = K0 / CIN, c = K0 - kpos * CIN;
        const int ky = kpos / KS, kx = kpos - ky * KS;
        return *reinterpret_cast<const float4 *>(halo + ((py * ST + ky) * G::E + px * ST + kx) * CIN + c);
    } else {
        float v[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int K = K0 + j < G::KT ? K0 + j : G::KT - 1;   // padded K: an in-patch address, value 0
            const int kpos = K / CIN, c = K - kpos * CIN;
            const int ky = kpos / KS, kx = kpos - ky * KS;
            const float hv = halo[((py * ST + ky) * G::E + px * ST + kx) * CIN + c];
            v[j] = K0 + j < G::KT ? hv : 0.f;
        }
        return make_float4(v[0], v[1], v[2], v[3]);
    }
}

template <int KS, int ST, int CIN, int COUT, bool DENSE, bool FIRST>
__global__ __launch_bounds__(256) void k_conv_gen(ConvArgs a) {
    using G = Gen<KS, ST, CIN, COUT>;
    extern __shared__ float smem[];
    __shared__ float s_bias[COUT];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    for (int j = tid; j < COUT; j += blockDim.x) s_bias[j] = a.bias[j];
    float *halo = smem;                                   // patch, then the epilogue's staging
    floatx4 *part = reinterpret_cast<floatx4 *>(smem + G::AREA);
    const floatx4 *wg = static_cast<const floatx4 *>(a.w);
    const int cnt = work_count<DENSE>(a);
    const XcdRange xr = xcd_range(cnt, 1);
    const int m = lane & 15, kq = lane >> 4;
    const int py = m & 3, px = m >> 2;
    const int b0 = wave * G::NBW;                         // this wave's K blocks [b0, b0 + NBW)
    // The next tile's patch is fetched into registers while this tile's
    // matrix work runs (past the end: the last tile again, never used).
    using P = GenPatch<KS, ST, CIN, COUT, FIRST>;
    typename P::T pv[P::PF];
    if (xr.first < xr.end) gen_fetch_patch<KS, ST, CIN, COUT, FIRST>(a, decode<DENSE>(a, xr.first), pv, tid);
    for (int t = xr.first; t < xr.end; t += xr.stride) {  // uniform per block
        const TileRef r = decode<DENSE>(a, t);
        lds_barrier();                                    // the previous tile's epilogue is done with the area
        gen_store_patch<KS, ST, CIN, COUT, FIRST>(halo, pv, tid);
        gen_fetch_patch<KS, ST, CIN, COUT, FIRST>(a, decode<DENSE>(a, min(t + xr.stride, xr.end - 1)), pv, tid);
        lds_barrier();
        floatx4 acc[G::NB];
#pragma unroll
        for (int nb = 0; nb < G::NB; ++nb) acc[nb] = floatx4{0.f, 0.f, 0.f, 0.f};
        // Weight ring: block b's fragments live in set (b - b0) % 3 (ext-vector arrays stay in registers).
        floatx4 w0[G::NB], w1[G::NB], w2[G::NB];
        auto fetch = [&](floatx4 *dst, int b) __attribute__((always_inline)) {
            const int bb = b < b0 + G::NBW ? b : b0 + G::NBW - 1;   // past this wave's range: unused
#pragma unroll
            for (int nb = 0; nb < G::NB; ++nb) dst[nb] = wg[(bb * G::NB + nb) * 64 + lane];
        };
        auto block = [&](floatx4 *w, int b) __attribute__((always_inline)) {
            const float4 av = gen_a<KS, ST, CIN, COUT>(halo, b, kq, py, px);
            const float al[4] = {av.x, av.y, av.z, av.w};
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int nb = 0; nb < G::NB; ++nb)
                    acc[nb] = __builtin_amdgcn_mfma_f32_16x16x4f32(al[j], w[nb][j], acc[nb], 0, 0, 0);
        };
        fetch(w0, b0);
        fetch(w1, b0 + 1);
        fetch(w2, b0 + 2);
#pragma unroll 1
        for (int b = b0; b < b0 + G::NBW; b += 3) {
            block(w0, b);
            fetch(w0, b + 3);
            block(w1, b + 1);
            fetch(w1, b + 4);
            block(w2, b + 2);
            fetch(w2, b + 5);
        }
        if (wave > 0) {
#pragma unroll
            for (int nb = 0; nb < G::NB; ++nb) part[((wave - 1) * G::NB + nb) * 64 + lane] = acc[nb];
        }
        lds_barrier();
        if (wave == 0) {
#pragma unroll
            for (int w = 0; w < G::KSPLIT - 1; ++w)
#pragma unroll
                for (int nb = 0; nb < G::NB; ++nb) acc[nb] += part[(w * G::NB + nb) * 64 + lane];
            epilogue<COUT>(a, r, acc, s_bias, halo, lane);
        }
    }
}

// ------------------------------------------------------------------ dispatch

template <bool DENSE, bool FUSE, int NO, bool VAR>
hipError_t run_resident_no(const ConvArgs &a, int cus, hipStream_t s) {
    auto kern = k_conv_mfma_res<DENSE, FUSE, NO, VAR>;
    static hipError_t attr = set_lds(kern, Res::lds_bytes);
    if (attr != hipSuccess) return attr;
    hipLaunchKernelGGL(kern, dim3(persistent_grid(cus, a.max_tiles)), dim3(512), Res::lds_bytes, s, a);
    return hipGetLastError();
}

// Logit count as a template argument where it is a common one.
template <bool DENSE, bool FUSE, bool VAR>
hipError_t run_resident(const ConvArgs &a, int cus, hipStream_t s) {
    if (a.n_out == 0) return run_resident_no<DENSE, FUSE, 0, VAR>(a, cus, s);
    if (a.n_out == 6) return run_resident_no<DENSE, FUSE, 6, VAR>(a, cus, s);
    return run_resident_no<DENSE, FUSE, -1, VAR>(a, cus, s);
}

template <bool DENSE, bool VAR>
hipError_t run_mfma(const ConvArgs &a, int cus, hipStream_t s) {
    return a.fuse_first ? run_resident<DENSE, true, VAR>(a, cus, s) : run_resident<DENSE, false, VAR>(a, cus, s);
}

template <int CIN, int COUT, bool DENSE, bool VAR>
hipError_t run_staged(const ConvArgs &a, int cus, hipStream_t s) {
    // Head partials come from their own kernel, which reads the overlays.
    if (a.fuse_first || a.n_out > 0 || (VAR && a.vov_out == nullptr)) return hipErrorInvalidValue;
    constexpr size_t lds = std::max(Chunked<CIN, COUT, 8>::lds_bytes, Chunked<CIN, COUT, 4>::lds_bytes);
    static_assert(lds <= 160 * 1024, "staged layer exceeds LDS");
    auto kern = k_conv_mfma_staged<CIN, COUT, DENSE, VAR>;
    static hipError_t attr = set_lds(kern, lds);
    if (attr != hipSuccess) return attr;
    hipLaunchKernelGGL(kern, dim3(persistent_grid(cus, (a.max_tiles + 3) / 4)), dim3(256), lds, s, a);
    return hipGetLastError();
}

template <int CIN, int COUT, bool DENSE, bool VAR>
hipError_t run_first(const ConvArgs &a, int cus, hipStream_t s) {
    const int total_max = a.max_tiles;
    if constexpr (CIN == 4) {
        // about 100-150 registers: four blocks of four waves are resident per CU
        const int grid = persistent_grid(cus * 4, (total_max + 3) / 4);
        hipLaunchKernelGGL((k_conv_first4_mfma<COUT, DENSE, VAR>), dim3(grid), dim3(256), 0, s, a);
    } else {
        const int grid = persistent_grid(cus * 8, (total_max + 3) / 4);
        hipLaunchKernelGGL((k_conv_first_f32<CIN, COUT, DENSE, VAR>), dim3(grid), dim3(256), 0, s, a);
    }
    return hipGetLastError();
}

#define RN_STAGED_SHAPES(X) X(64, 128) X(128, 128)
// General layers: (k, stride, cin, cout); first layers read the input frames.
#define RN_GEN_FIRST_SHAPES(X) X(8, 4, 4, 32) X(8, 4, 1, 32) X(5, 1, 1, 32) X(7, 2, 1, 32) X(5, 2, 4, 32)
#define RN_GEN_SHAPES(X) X(4, 2, 32, 64) X(3, 1, 64, 64) X(3, 1, 32, 64) X(3, 2, 32, 64) X(5, 2, 32, 64) X(5, 1, 32, 32)

template <int KS, int ST, int CIN, int COUT, bool FIRST>
hipError_t run_gen(const ConvArgs &a, int cus, hipStream_t s) {
    using G = Gen<KS, ST, CIN, COUT>;
    const bool dense = a.wl == nullptr;
    auto kern = dense ? k_conv_gen<KS, ST, CIN, COUT, true, FIRST> : k_conv_gen<KS, ST, CIN, COUT, false, FIRST>;
    static hipError_t attr = set_lds(k_conv_gen<KS, ST, CIN, COUT, true, FIRST>, G::lds_bytes);
    static hipError_t attr2 = set_lds(k_conv_gen<KS, ST, CIN, COUT, false, FIRST>, G::lds_bytes);
    if (attr != hipSuccess) return attr;
    if (attr2 != hipSuccess) return attr2;
    // As many blocks as the CUs hold at once (registers and LDS decide), so
    // every block starts in the first generation and walks several tiles.
    static int occ = [] {
        int b = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&b, k_conv_gen<KS, ST, CIN, COUT, false, FIRST>,
                                                         64 * G::KSPLIT, G::lds_bytes) != hipSuccess || b < 1)
            b = 2;
        return b;
    }();
    const int grid = persistent_grid(cus * occ, a.max_tiles);
    hipLaunchKernelGGL(kern, dim3(grid), dim3(64 * G::KSPLIT), G::lds_bytes, s, a);
    return hipGetLastError();
}
#define RN_FIRST_SHAPES(X) X(1, 20) X(1, 40) X(1, 64) X(1, 80) X(4, 20) X(4, 40) X(4, 64) X(4, 80)

}  // namespace

bool conv_gen_supported(int k, int s, int cin, int cout, bool first) {
#define X(kk, ss, ci, co) if (k == kk && s == ss && cin == ci && cout == co) return true;
    if (first) {
        RN_GEN_FIRST_SHAPES(X)
    } else {
        RN_GEN_SHAPES(X)
    }
#undef X
    return false;
}

hipError_t launch_conv_gen(const ConvArgs &a, int k, int s, bool first, int cus, hipStream_t st) {
#define X(kk, ss, ci, co) \
    if (k == kk && s == ss && a.cin == ci && a.cout == co) return run_gen<kk, ss, ci, co, FIRSTV>(a, cus, st);
    if (first) {
#define FIRSTV true
        RN_GEN_FIRST_SHAPES(X)
#undef FIRSTV
    } else {
#define FIRSTV false
        RN_GEN_SHAPES(X)
#undef FIRSTV
    }
#undef X
    return hipErrorInvalidValue;
}

// 16-K blocks of a general layer, padded like Gen::NBLK (four waves x whole
// triples of the kernel's weight ring).
static int gen_blocks(int k, int cin) { return ((k * k * cin + 15) / 16 + 11) / 12 * 12; }

size_t conv_gen_packed_elems(int k, int cin, int cout) { return (size_t)gen_blocks(k, cin) * 16 * cout; }
#define X(kk, ss, ci, co) static_assert(Gen<kk, ss, ci, co>::NBLK == ((kk * kk * ci + 15) / 16 + 11) / 12 * 12, "padding");
RN_GEN_FIRST_SHAPES(X)
RN_GEN_SHAPES(X)
#undef X

void pack_conv_gen(const float *oihw, int k, int cin, int cout, float *dst) {
    // [block][n-block][lane][j]: K = 16 block + 4 (lane / 16) + j in (ky, kx, c)
    // order, n = 16 n-block + lane % 16; zero past K = k k cin.
    const int kt = k * k * cin, nblk = gen_blocks(k, cin), nbn = cout / 16;
    size_t o = 0;
    for (int b = 0; b < nblk; ++b)
        for (int nb = 0; nb < nbn; ++nb)
            for (int l = 0; l < 64; ++l)
                for (int j = 0; j < 4; ++j) {
                    const int K = 16 * b + 4 * (l / 16) + j, n = nb * 16 + l % 16;
                    float v = 0.f;
                    if (K < kt) {
                        const int kpos = K / cin, c = K % cin, ky = kpos / k, kx = kpos % k;
                        v = oihw[(((size_t)n * cin + c) * k + ky) * k + kx];
                    }
                    dst[o++] = v;
                }
}

static bool is_resident(int cin, int cout) { return cin == Res::CIN && cout == Res::COUT; }

bool conv_mfma_supported(int cin, int cout, rn_dtype dt) {
    return dt == RN_F32 && (is_resident(cin, cout) || conv_split_supported(cin, cout));
}

bool conv_fused_first_supported(int c1, int c2, rn_dtype dt) { return dt == RN_F32 && is_resident(c1, c2); }

size_t conv_res_bytes(int cin, int cout) { return is_resident(cin, cout) ? Res::w_bytes + Res::COUT * sizeof(float) : 0; }

hipError_t launch_pack_res(const float *w, void *dst, hipStream_t s) {
    const int units = (Res::KS * Res::NB + Res::COUT) * 64;
    hipLaunchKernelGGL(k_pack_res, dim3((units + 255) / 256), dim3(256), 0, s, w, static_cast<__bf16 *>(dst));
    return hipGetLastError();
}

bool conv_first_supported(int cin, int cout, rn_dtype dt) {
    if (dt != RN_F32) return false;
#define X(ci, co) if (cin == ci && cout == co) return true;
    RN_FIRST_SHAPES(X)
#undef X
    return false;
}

// cus: compute units of the device; the persistent grid is at most one block
// (resident MFMA kernel) or eight blocks (first layer) per CU.
hipError_t launch_conv_mfma(const ConvArgs &a, int cus, hipStream_t s, bool var) {
    const bool dense = a.wl == nullptr;
    if ((var && dense) || !is_resident(a.cin, a.cout)) return hipErrorInvalidValue;
    return var ? run_mfma<false, true>(a, cus, s) : dense ? run_mfma<true, false>(a, cus, s) : run_mfma<false, false>(a, cus, s);
}

hipError_t launch_conv_staged(const ConvArgs &a, int cus, hipStream_t s, bool var) {
    const bool dense = a.wl == nullptr;
    if (var && dense) return hipErrorInvalidValue;
#define X(ci, co)                                                      \
    if (a.cin == ci && a.cout == co)                                   \
        return var ? run_staged<ci, co, false, true>(a, cus, s)        \
                   : dense ? run_staged<ci, co, true, false>(a, cus, s) : run_staged<ci, co, false, false>(a, cus, s);
    RN_STAGED_SHAPES(X)
#undef X
    return hipErrorInvalidValue;
}

hipError_t launch_conv_first(const ConvArgs &a, rn_dtype dt, int cus, hipStream_t s, bool var) {
    (void)dt;
    const bool dense = a.wl == nullptr;
    if (var && dense) return hipErrorInvalidValue;
#define X(ci, co)                                                                          \
    if (a.cin == ci && a.cout == co)                                                       \
        return var ? run_first<ci, co, false, true>(a, cus, s)                             \
                   : dense ? run_first<ci, co, true, false>(a, cus, s) : run_first<ci, co, false, false>(a, cus, s);
    RN_FIRST_SHAPES(X)
#undef X
    return hipErrorInvalidValue;
}

size_t conv_first_packed_elems(int cin, int cout) { return (size_t)cin * 9 * cout; }

size_t conv_mfma_packed_elems(int cin, int cout, rn_dtype dt) {
    (void)dt;
    return (size_t)9 * cin * cout;
}

void pack_conv_first(const float *oihw, int cin, int cout, rn_dtype dt, void *dst) {
    // [ci * 9 + ky * 3 + kx][co]
    (void)dt;
    float *d = static_cast<float *>(dst);
    for (int co = 0; co < cout; ++co)
        for (int ci = 0; ci < cin; ++ci)
            for (int k = 0; k < 9; ++k) d[(ci * 9 + k) * cout + co] = oihw[((size_t)co * cin + ci) * 9 + k];
}

void pack_conv_mfma(const float *oihw, int cin, int cout, rn_dtype dt, void *dst) {
    // [kpos][block][nb][lane][j]: block b of a kernel position covers channels
    // [16 b, 16 b + 16) (the last block [16 nf, 16 nf + 8) when cin % 16 = 8);
    // element j of lane l is B[channel][n] with n = nb * 16 + l % 16 and
    // channel = 16 b + 4 (l / 16) + j (block of 8: 16 nf + 2 (l / 16) + j).
    (void)dt;
    float *d = static_cast<float *>(dst);
    const int nb_n = cout / 16, nf = cin / 16;
    size_t o = 0;
    for (int kpos = 0; kpos < 9; ++kpos) {
        for (int b = 0; b < nf + (cin % 16 ? 1 : 0); ++b) {
            const bool full = b < nf;
            const int steps = full ? 4 : 2;
            for (int nb = 0; nb < nb_n; ++nb)
                for (int l = 0; l < 64; ++l)
                    for (int j = 0; j < steps; ++j) {
                        const int ci = 16 * b + (full ? 4 : 2) * (l / 16) + j;
                        const int n = nb * 16 + l % 16;
                        d[o++] = oihw[((size_t)n * cin + ci) * 9 + kpos];
                    }
        }
    }
}

size_t tile_head_w_elems(int ntiles, int cout, int n_out) { return (size_t)n_out * ntiles * kTilePx * cout; }

void pack_tile_head(const float *dense_w, int n_out, int C, int H, int W, int TH, int TW, float *dst) {
    // [o][tile][nb][lane][i]: the weight of the output the MFMA epilogue holds
    // in lane `lane`, register i of block nb: channel nb * 16 + lane % 16,
    // tile pixel (row i, column lane / 16).  Zero outside the image.
    const int NB = C / 16, ntiles = TH * TW;
    for (int o = 0; o < n_out; ++o)
        for (int t = 0; t < ntiles; ++t) {
            const int ty = t / TW, tx = t % TW;
            for (int nb = 0; nb < NB; ++nb)
                for (int l = 0; l < 64; ++l)
                    for (int i = 0; i < 4; ++i) {
                        const int c = nb * 16 + l % 16, y = ty * kTile + i, x = tx * kTile + l / 16;
                        const size_t di = ((((size_t)o * ntiles + t) * NB + nb) * 64 + l) * 4 + i;
                        dst[di] = (y < H && x < W) ? dense_w[(size_t)o * C * H * W + ((size_t)c * H + y) * W + x]
                                                   : 0.f;
                    }
        }
}

}  // namespace rn
