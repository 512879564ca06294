// Float32 3x3 layers of many channels (64->128, 128->128), and the input
// gradients of training, on the bf16 matrix cores with operands split three
// ways (rn_split.hpp).
//
// Bound: matrix issue.  A tile is 2 * 16 * COUT * 9 CIN flops six times over on
// v_mfma_f32_32x32x16_bf16 (~2.06 PFLOP/s from one wave per SIMD in a bare loop,
// 344 TFLOP/s of float32 work; the float32 instruction gives 150).  Counters of
// layers 3 and 2 of 1024 210x160 streams: matrix pipe busy 81% and 72% of the
// cycles, at 1.7 and 1.9 GHz, which this load brings the clock down to; input
// gradients 80->40 58% at 2.2 GHz (40 channels fill 5/8 of the rows).
//
// A block of four waves computes a group of T tiles x all COUT channels, a wave
// 32 channels of all tiles (of half of them where COUT has two such blocks): T /
// 2 tile pairs (32 pixels), twice (large and small sums), 256 accumulator
// registers at T = 16, so one block per CU.  (Two waves along the channels, two
// along the tiles: the weights of a stage are read twice, 3824 against 3579 us
// at T = 8, layer 3 of 1024 210x160 streams; T = 16 then 3370, where the
// float32 instructions took 6233.)  The product
// is transposed (rows = channels, columns = pixels): a lane ends with four
// neighbouring channels of one pixel and stores 16 bytes.
// K runs over chunks of 16 input channels and, within one, the nine kernel
// positions (a stage = one position of one chunk, one k-step of 16).
//   Halos: the chunk's 6 x 6 x 16 values of each tile sit in LDS as three bf16
//   planes, two chunk buffers.  Every value is split once per group: a thread
//   loads its 16-byte units (pixel, channel quad) of a chunk into registers
//   two chunks ahead and, one unit per stage, splits them and writes
//   them to the buffer of the next chunk, so the staging (about 30 vector
//   instructions a stage) runs between the matrix ops; one barrier per chunk.
//   Plane layout: 16-byte slot (8 channels of a pixel) 12 hy + 6 half + hx; the
//   16 pixels of a 16-lane read then lie in 16 distinct bank groups at every
//   kernel position.
//   Weights: packed in fragment order (pack below) and read straight into
//   registers two stages ahead (one stage: T = 4 alone on its CU 30 instead of
//   24 us).  Larger groups read fewer weight bytes per tile: 12 KB a stage.
// The sums over K of an output run in one order whatever T is, so a tile's
// outputs do not depend on the group size a launch picks, and a dense pass, a
// reuse step and a variant give the same bits.
//   A result that is not finite: an infinity or a NaN among its operands makes
// the sum of the small terms NaN, and the leading sum alone has the class that
// float32 arithmetic gives.  Where the sum of the small terms is finite, finite
// operands overflowed, and where a halo holds a finite value that rounds up to
// infinity in bf16 (watched while staging; clamping each of them instead cost
// 1.2% of the step) the leading sum says nothing: such results are summed again
// in plain float32.  The weights' leading planes are clamped when packed.
#include "rn_split.hpp"

namespace rn {
namespace {

using namespace dev;

// Source of halo values that lie outside the image or past the work list.
__device__ __align__(16) float g_zero_halo[128];

// What a launch computes: a layer's outputs for a work list, for every tile, or
// for variants; or the gradient at a layer's input (INPUT_GRAD): a convolution
// of dJ/dz (CIN channels) with the transposed, flipped weights, kept where the
// layer's input (COUT channels, the layer before's activations) is above 0.
enum { LIST = 0, DENSE_PASS = 1, VARIANTS = 2, INPUT_GRAD = 3 };

template <int CIN, int COUT, int T>
struct SplitConv {
    static constexpr int NCH = CIN / 16;             // chunks of 16 channels
    static constexpr int C16 = (COUT + 15) / 16 * 16;   // columns of the float32 packing
    static constexpr int NN = (COUT + 31) / 32;      // blocks of 32 channels, one per wave
    static constexpr int WM = 4 / NN;                // waves along the tiles
    static constexpr int MB = T / 2 / WM;            // tile pairs per wave
    static constexpr int PLANE = 72 * 16;            // bytes of one plane of one tile's chunk
    static constexpr int TILE = 3 * PLANE;
    static constexpr int BUF = T * TILE;             // bytes of a chunk buffer
    // 16-byte units of a chunk, (tile, pixel, channel quad): a tile's 256 / T
    // threads are RY x RX x 4 (those past that: idle), each with the JY x JX
    // pixels at (JY ry, JX rx) of one quad.
    static constexpr int TPT = 256 / T;
    static constexpr int RY = T == 16 ? 2 : 6, RX = T == 4 ? 2 : T == 8 ? 1 : 2;
    static constexpr int JY = 6 / RY, JX = 6 / RX;
    static constexpr int UPT = JY * JX;
    static constexpr size_t WSTAGE = (size_t)3 * NN * 512;   // bf16 weights per stage
    static constexpr size_t lds_bytes = 2 * (size_t)BUF + COUT * sizeof(float) + T * sizeof(int);
    static_assert(CIN % 16 == 0 && NCH >= 3 && COUT % 4 == 0 && NN * WM == 4 && T % 4 == 0, "chunks in flight, waves");
    static_assert(UPT <= 9 && RY * RX * 4 <= TPT, "at most one unit per stage, all of them covered");
    static_assert(CIN <= 128, "zero source");
};

// Float32 weight of (kernel position, input channel ci, output channel n) in
// the packing of pack_conv_mfma.
__device__ inline size_t f32_weight(int kpos, int ci, int n, int cin, int cout) {
    return ((size_t)(kpos * (cin / 16) + ci / 16) * (cout / 16) + n / 16) * 256 + ((ci % 16) / 4 * 16 + n % 16) * 4 +
           ci % 4;
}

// Address of channel 0 of pixel (y, x) of layer l - 1 as tile r's stream sees
// it, or of zeros outside the image or where `listed` is false.  Without
// branches also for variants (loads at clamped positions, the address selected).
template <int CIN, bool VAR>
__device__ inline const float *halo_src(const ConvArgs &a, const TileRef &r, int y, int x, bool listed) {
    const bool in = listed && y >= 0 && y < a.H && x >= 0 && x < a.W;
    y = min(max(y, 0), a.H - 1);
    x = min(max(x, 0), a.W - 1);
    const int t = (y >> 2) * a.TW + (x >> 2);
    const size_t off = (size_t)t * kTilePx * CIN;
    const float *src = static_cast<const float *>(a.in) + (size_t)(VAR ? a.vbase : r.slot) * a.in_stride + off;
    if constexpr (VAR) {
        const int ntiles = a.TH * a.TW;
        const uint64_t own = a.vtm_in[(size_t)r.slot * ((ntiles + 63) >> 6) + (t >> 6)] >> (t & 63);
        const size_t row = (uint32_t)a.vmap_in[(size_t)r.slot * ntiles + t];    // listed tiles only
        src = own & 1 ? static_cast<const float *>(a.vov_in) + row * kTilePx * CIN : src;
    }
    return in ? src + ((y & 3) * 4 + (x & 3)) * CIN : g_zero_halo;
}

// Outputs n, n + 8, n + 16 and n + 24 of pixel p before bias in plain float32
// (C16: columns of the float32 packing), those with a bit in `want`.  A sum
// that has become NaN stays NaN: it ends there.
template <int CIN, int C16, bool VAR>
__device__ __attribute__((always_inline)) inline void plain_outputs(const ConvArgs &a, const TileRef &r, int p, int n, int want, float (&acc)[4]) {
    const float *w = static_cast<const float *>(a.w);
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[j] = 0.f;
    for (int ci0 = 0; ci0 < CIN; ci0 += 16)
        for (int kpos = 0; kpos < 9; ++kpos) {
            const int y = r.ty * kTile + (p >> 2) + kpos / 3 - 1, x = r.tx * kTile + (p & 3) + kpos % 3 - 1;
            const float *src = halo_src<CIN, VAR>(a, r, y, x, true);
#pragma unroll 4
            for (int ci = ci0; ci < ci0 + 16; ++ci)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    acc[j] = fmaf(src[ci], w[f32_weight(kpos, ci, min(n + 8 * j, C16 - 1), CIN, C16)], acc[j]);
            bool open = false;
#pragma unroll
            for (int j = 0; j < 4; ++j) open |= (want >> j & 1) && !__builtin_isnan(acc[j]);
            if (!open) return;
        }
}
constexpr uint32_t kNan = 0x7fc00000u, kAgain = 0x7fc00001u;   // a NaN result; one to be summed again

// Row of the output a tile is written to.
template <int COUT, bool VAR>
__device__ inline float *out_tile(const ConvArgs &a, const TileRef &r, int t) {
    return VAR ? static_cast<float *>(a.vov_out) + (size_t)t * kTilePx * COUT
               : static_cast<float *>(a.out) + (size_t)r.slot * a.out_stride + (size_t)r.tile * kTilePx * COUT;
}

template <int CIN, int COUT, int MODE, int T>
__device__ __attribute__((always_inline)) inline void split_path(const ConvArgs &a, int cnt, unsigned char *lds) {
    using C = SplitConv<CIN, COUT, T>;
    constexpr bool DENSE = MODE == DENSE_PASS || MODE == INPUT_GRAD, VAR = MODE == VARIANTS, GRAD = MODE == INPUT_GRAD;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wn = wave % C::NN, wm = wave / C::NN;       // the wave's channel block and share of the tiles
    const XcdRange xr = xcd_range(cnt, T);
    if (xr.first >= xr.end) return;                       // uniform per block
    float *s_bias = reinterpret_cast<float *>(lds + 2 * C::BUF);
    if constexpr (!GRAD)
        for (int j = tid; j < COUT; j += 256) s_bias[j] = a.bias[j];
    // The last group whose halo of tile t holds a finite value that rounds to infinity.
    int *s_wide = reinterpret_cast<int *>(s_bias + COUT);
    if (tid < T) s_wide[tid] = -1;
    float rest = 0.f;                                     // split4, over this thread's values of the group being staged

    // Item word of tile lane % T of a group (past the end: the last item).
    auto items = [&](int g) __attribute__((always_inline)) {
        return item_word<DENSE>(a, min(g + lane % T, xr.end - 1));
    };
    // This thread's units, and their sources in chunk 0 of the group at g.
    const int ut = tid % C::TPT, utile = tid / C::TPT, uq = ut & 3;
    const bool unit = (ut >> 2) < C::RY * C::RX;
    const int uy = (ut >> 2) / C::RX * C::JY, ux = (ut >> 2) % C::RX * C::JX;
    const float *src[C::UPT];
    auto sources = [&](int g, uint32_t words) __attribute__((always_inline)) {
        const TileRef r = item_ref(a, (uint32_t)__shfl((int)words, utile));
        const bool listed = unit && g + utile < xr.end;
#pragma unroll
        for (int j = 0; j < C::UPT; ++j) {
            const int y = r.ty * kTile - 1 + uy + j / C::JX, x = r.tx * kTile - 1 + ux + j % C::JX;
            src[j] = halo_src<CIN, VAR>(a, r, y, x, listed) + 4 * uq;
        }
    };
    floatx4 pre[C::UPT];
    auto load_unit = [&](int j, int c) __attribute__((always_inline)) {
        pre[j] = *reinterpret_cast<const floatx4 *>(src[j] + 16 * c);
    };
    unsigned char *ulds = lds + utile * C::TILE + (uy * 12 + (uq >> 1) * 6 + ux) * 16 + (uq & 1) * 8;
    auto store_unit = [&](int j, int buf) __attribute__((always_inline)) {
        unsigned char *d = ulds + buf * C::BUF + (j / C::JX * 12 + j % C::JX) * 16;
        bf16x4 h, m, l;
        split4(pre[j], h, m, l, rest);
        if (unit) {
            *reinterpret_cast<bf16x4 *>(d) = h;
            *reinterpret_cast<bf16x4 *>(d + C::PLANE) = m;
            *reinterpret_cast<bf16x4 *>(d + 2 * C::PLANE) = l;
        }
    };
    // Weight fragments of a stage: [plane][channel block][lane] 16 bytes.
    const bf16x8 *wg = reinterpret_cast<const bf16x8 *>(a.w_split) + wn * 64 + lane;
    auto load_w = [&](bf16x8 (&w)[3], int s) __attribute__((always_inline)) {
        const bf16x8 *p = wg + (size_t)s * (C::WSTAGE / 8);
#pragma unroll
        for (int pl = 0; pl < 3; ++pl) w[pl] = p[pl * C::NN * 64];
    };
    // Pixel fragments of tile pair m at kernel position kpos.
    const int pix = lane & 15;
    const unsigned char *xa = lds + (2 * wm * C::MB + ((lane >> 4) & 1)) * C::TILE +
                              ((pix >> 2) * 12 + (lane >> 5) * 6 + (pix & 3)) * 16;
    auto load_x = [&](bf16x8 (&x)[3], int buf, int m, int kpos) __attribute__((always_inline)) {
        const unsigned char *p = xa + buf * C::BUF + 2 * m * C::TILE + (kpos / 3 * 12 + kpos % 3) * 16;
#pragma unroll
        for (int pl = 0; pl < 3; ++pl) x[pl] = *reinterpret_cast<const bf16x8 *>(p + pl * C::PLANE);
    };

    // Prologue: chunk 0 split into buffer 0, chunk 1 in registers.
    uint32_t it = items(xr.first), it_next = 0;
    sources(xr.first, it);
#pragma unroll
    for (int j = 0; j < C::UPT; ++j) load_unit(j, 0);
    bf16x8 w[3][3];                                       // stage s in slot s % 3 (nine stages a chunk)
    load_w(w[0], 0);
    load_w(w[1], 1);
#pragma unroll
    for (int j = 0; j < C::UPT; ++j) {
        store_unit(j, 0);
        load_unit(j, 1);
    }
    lds_barrier();

    int buf = 0;                                          // buffer of the current chunk
    for (int g = xr.first; g < xr.end; g += xr.stride) {   // uniform per block
        floatx16 hi[C::MB], lo[C::MB];
#pragma unroll
        for (int m = 0; m < C::MB; ++m)
#pragma unroll
            for (int e = 0; e < 16; ++e) hi[m][e] = lo[m][e] = 0.f;
        it_next = items(min(g + xr.stride, xr.end - 1));
#pragma unroll 1
        for (int c = 0; c < C::NCH; ++c) {
            // From here on the loads are the next group's (chunk c + 2).
            if (c == C::NCH - 2) sources(g + xr.stride, it_next);
            const int cl = c + 2 < C::NCH ? c + 2 : c + 2 - C::NCH;
            if (c == C::NCH - 1) {                        // staged in full; what follows is the next group's
                if (rest == __builtin_inff()) s_wide[utile] = g;
                rest = 0.f;
            }
            bf16x8 x[3];
            load_x(x, buf, 0, 0);
#pragma unroll
            for (int kp = 0; kp < 9; ++kp) {
                const int s = c * 9 + kp + 2;
#pragma unroll
                for (int m = 0; m < C::MB; ++m) {
                    // Beside the six matrix ops of a tile pair: the next
                    // operands, and a part of the stage's staging.
                    bf16x8 xn[3];
                    __builtin_amdgcn_sched_barrier(0);
                    if (m == 0) load_w(w[(kp + 2) % 3], s >= 9 * C::NCH ? s - 9 * C::NCH : s);
                    if (m + 1 < C::MB) load_x(xn, buf, m + 1, kp);
                    else if (kp < 8) load_x(xn, buf, 0, kp + 1);
                    if (m == (C::MB > 1 ? 1 : 0) && kp < C::UPT) {
                        store_unit(kp, buf ^ 1);
                        load_unit(kp, cl);
                    }
                    // (weight plane, pixel plane): the leading term, the five small ones
                    constexpr int pw[6] = {0, 2, 0, 1, 1, 0}, px[6] = {0, 0, 2, 1, 0, 1};
#pragma unroll
                    for (int k = 0; k < 6; ++k) {
                        floatx16 &acc = k == 0 ? hi[m] : lo[m];
                        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w[kp % 3][pw[k]], x[px[k]], acc, 0, 0, 0);
                    }
#pragma unroll
                    for (int k = 0; k < 6; ++k) {
                        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);      // a matrix op
                        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);      // an LDS read
                        __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);      // a load
                        __builtin_amdgcn_sched_group_barrier(0x002, 6, 0);      // vector instructions
                        __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);      // an LDS write
                    }
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int pl = 0; pl < 3; ++pl) x[pl] = xn[pl];
                }
            }
            lds_barrier();                                // chunk c read, chunk c + 1 written by every wave
            buf ^= 1;
        }
        // Epilogue: bias, ReLU and the zero outside the image on the bit
        // patterns (a float above zero has a positive int pattern), 16 bytes
        // a lane.  A result to be summed again is marked, and taken below.
        bool bad = false;
#pragma unroll
        for (int m = 0; m < C::MB; ++m) asm volatile("" : "+a"(hi[m]), "+a"(lo[m]));
#pragma unroll
        for (int m = 0; m < C::MB; ++m) {
            // Each pair's sums leave the accumulator registers on their own
            // (all at once they would push everything else to scratch).
            asm volatile("" : "+a"(hi[m]), "+a"(lo[m]));
            const int t = 2 * (wm * C::MB + m) + ((lane >> 4) & 1);
            const TileRef r = item_ref(a, (uint32_t)__shfl((int)it, t));
            const int keep = ~((a.W - 1 - (r.tx * kTile + (pix & 3))) >> 31) & ~((a.H - 1 - (r.ty * kTile + (pix >> 2))) >> 31);
            const int ch = wn * 32 + 4 * (lane >> 5);
            float *dst = out_tile<COUT, VAR>(a, r, min(g + t, xr.end - 1)) + pix * COUT + ch;
            floatx4 mask[4];
            if constexpr (GRAD) {
                const float *src = a.mask + (size_t)a.mask_ids[r.slot] * a.mask_stride + ((size_t)r.tile * kTilePx + pix) * COUT;
#pragma unroll
                for (int q = 0; q < 4; ++q) mask[q] = *reinterpret_cast<const floatx4 *>(src + min(ch + 8 * q, COUT - 4));
            }
            float seen = 0.f;
            floatx16 v;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                floatx4 b{0.f, 0.f, 0.f, 0.f};
                if constexpr (!GRAD) b = *reinterpret_cast<const floatx4 *>(s_bias + ch + 8 * q);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    v[4 * q + e] = (hi[m][4 * q + e] + lo[m][4 * q + e]) + b[e];
                    seen = nonfinite(v[4 * q + e], seen);
                }
            }
            if (__builtin_expect(__any(seen != 0.f), 0)) {   // NaN: some result is not finite
                const bool wide = s_wide[t] == g;
                bool again = false;
#pragma unroll
                for (int q = 0; q < 4; ++q)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int i = 4 * q + e;
                        const float bias = GRAD ? 0.f : s_bias[ch + 8 * q + e];
                        const bool lost = !is_finite(v[i]), plain = wide || (is_finite(lo[m][i]) && is_finite(bias));
                        float lead = hi[m][i] + bias;
                        lead = plain ? __uint_as_float(kAgain) : __builtin_isnan(lead) ? __uint_as_float(kNan) : lead;
                        v[i] = lost ? lead : v[i];
                        again |= lost && plain && (GRAD ? mask[q][e] > 0.f : keep != 0);
                    }
                bad |= __any(again);
            }
            if (g + t < xr.end && (!VAR || a.vov_out != nullptr)) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    if (ch + 8 * q >= COUT) continue;
                    floatx4 o;
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        o[e] = GRAD ? (mask[q][e] > 0.f ? v[4 * q + e] : 0.f)
                                    : __int_as_float(max(__float_as_int(v[4 * q + e]), 0) & keep);
                    *reinterpret_cast<floatx4 *>(dst + 8 * q) = o;
                }
            }
        }
        if (__builtin_expect(bad, 0)) {                   // uniform per wave
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            for (int k = 4 * wm * C::MB; k < 4 * (wm + 1) * C::MB; ++k) {   // 8 pixels x 8 lanes x 4 channels a pass
                const int t = k >> 1, p = (k & 1) * 8 + (lane >> 3);
                if (g + t >= xr.end || (VAR && a.vov_out == nullptr)) continue;
                const TileRef r = item_ref(a, (uint32_t)__shfl((int)it, t));
                float *dst = out_tile<COUT, VAR>(a, r, g + t) + p * COUT;
                const int n = wn * 32 + (lane & 7);
                int want = 0;
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    want |= n + 8 * j < COUT && __float_as_uint(dst[min(n + 8 * j, COUT - 1)]) == kAgain ? 1 << j : 0;
                if (want == 0) continue;
                float f[4];
                plain_outputs<CIN, C::C16, VAR>(a, r, p, n, want, f);
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (want >> j & 1)
                        dst[n + 8 * j] = GRAD ? f[j] : __int_as_float(max(__float_as_int(f[j] + s_bias[n + 8 * j]), 0));
            }
        }
        it = it_next;
    }
}

// The group size by the rounds a launch takes: a group of 16, 8 or 4 tiles of a
// 128 -> 128 layer takes 69, 41 or 26 us with every CU busy (an MI355X; the
// other layers in proportion).
template <int CIN, int COUT, int MODE>
__global__ __launch_bounds__(256, 1) void k_conv_mfma_split(ConvArgs a) {
    extern __shared__ __align__(16) unsigned char lds[];
    const int cnt = work_count<MODE == DENSE_PASS || MODE == INPUT_GRAD>(a);
    auto rounds = [&](int T) { return (cnt + T * (int)gridDim.x - 1) / (T * (int)gridDim.x); };
    const int c16 = rounds(16) * 69, c8 = rounds(8) * 41, c4 = rounds(4) * 26;
    if (c16 <= c8 && c16 <= c4) split_path<CIN, COUT, MODE, 16>(a, cnt, lds);
    else if (c8 <= c4) split_path<CIN, COUT, MODE, 8>(a, cnt, lds);
    else split_path<CIN, COUT, MODE, 4>(a, cnt, lds);
}

// Split weights in fragment order, [chunk][kernel position][plane][32-channel
// block][lane][8]: element i of lane l is input channel 16 chunk + 8 (l / 32) + i
// of output channel 32 block + l % 32, from the float32 packing of c16 columns
// (zero past them).
__global__ void k_pack_split(const float *w, int cin, int c16, int NN, __bf16 *dst) {
    const size_t u = (size_t)blockIdx.x * blockDim.x + threadIdx.x;      // (chunk, position, block, lane)
    if (u >= (size_t)9 * (cin / 16) * NN * 64) return;
    const int l = u % 64, n0 = u / 64 % NN, kpos = u / 64 / NN % 9, c = (int)(u / 64 / NN / 9);
    const int n = 32 * n0 + l % 32, ci = 16 * c + 8 * (l / 32);
    __bf16 *d = dst + ((size_t)(c * 9 + kpos) * 3 * NN + n0) * 512 + l * 8;
    for (int q = 0; q < 2; ++q) {
        floatx4 v{0.f, 0.f, 0.f, 0.f};
        if (n < c16) v = *reinterpret_cast<const floatx4 *>(w + f32_weight(kpos, ci + 4 * q, n, cin, c16));
        bf16x4 p[3];
        split4_any(v, p[0], p[1], p[2]);
        for (int pl = 0; pl < 3; ++pl) *reinterpret_cast<bf16x4 *>(d + (size_t)pl * NN * 512 + 4 * q) = p[pl];
    }
}

template <int CIN, int COUT, int MODE>
hipError_t run_split(const ConvArgs &a, int cus, hipStream_t s) {
    constexpr size_t lds = SplitConv<CIN, COUT, 16>::lds_bytes;
    static_assert(lds <= 160 * 1024, "chunk buffers exceed LDS");
    auto kern = k_conv_mfma_split<CIN, COUT, MODE>;
    static hipError_t attr = set_lds(kern, lds);
    if (attr != hipSuccess) return attr;
    hipLaunchKernelGGL(kern, dim3(persistent_grid(cus, (a.max_tiles + 3) / 4)), dim3(256), lds, s, a);
    return hipGetLastError();
}

#define RN_SPLIT_SHAPES(X) X(64, 128) X(128, 128)
// Input gradients: channels of dJ/dz, of the layer's input.
#define RN_DX_SHAPES(X) X(80, 40) X(128, 64) X(128, 128)

}  // namespace

bool conv_split_supported(int cin, int cout) {
#define X(ci, co) if (cin == ci && cout == co) return true;
    RN_SPLIT_SHAPES(X)
#undef X
    return false;
}

bool train_dx_supported(int cz, int ca) {
#define X(ci, co) if (cz == ci && ca == co) return true;
    RN_DX_SHAPES(X)
#undef X
    return false;
}

size_t conv_split_bytes(int cin, int cout) { return (size_t)9 * cin * ((cout + 31) / 32 * 32) * 6; }

hipError_t launch_pack_split(const float *w, int cin, int cout, void *dst, hipStream_t s) {
    const int NN = (cout + 31) / 32, units = 9 * (cin / 16) * NN * 64;
    hipLaunchKernelGGL(k_pack_split, dim3((units + 255) / 256), dim3(256), 0, s, w, cin, (cout + 15) / 16 * 16, NN,
                       static_cast<__bf16 *>(dst));
    return hipGetLastError();
}

hipError_t launch_conv_split(const ConvArgs &a, int cus, hipStream_t s, bool var) {
    const bool dense = a.wl == nullptr;
    if (var && dense) return hipErrorInvalidValue;
    if (a.fuse_first || a.n_out > 0) return hipErrorInvalidValue;   // head partials come from their own kernel
#define X(ci, co)                                                      \
    if (a.cin == ci && a.cout == co)                                   \
        return var ? run_split<ci, co, VARIANTS>(a, cus, s)            \
                   : dense ? run_split<ci, co, DENSE_PASS>(a, cus, s) : run_split<ci, co, LIST>(a, cus, s);
    RN_SPLIT_SHAPES(X)
#undef X
    return hipErrorInvalidValue;
}

hipError_t launch_bwd_dx(const ConvArgs &a, int cus, hipStream_t s) {
    if (a.wl != nullptr || a.mask == nullptr) return hipErrorInvalidValue;
#define X(ci, co) \
    if (a.cin == ci && a.cout == co) return run_split<ci, co, INPUT_GRAD>(a, cus, s);
    RN_DX_SHAPES(X)
#undef X
    return hipErrorInvalidValue;
}

}  // namespace rn
