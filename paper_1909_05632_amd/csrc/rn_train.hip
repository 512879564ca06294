// Training kernels (Sec. 2: the policy is trained with REINFORCE; within a
// rollout the weights are fixed, so the forward steps reuse activations as in
// inference, and the gradient of a step is taken from the activations the
// caches then hold).
//
// For a batch of streams and given dJ/dlogits g, backpropagation through
// logits = Wd a_L + bd and a_l = ReLU(conv(a_{l-1}, W_l) + b_l):
//   head:   dWd (+)= sum_i g_i a_L,i^T,  dbd (+)= sum_i g_i,
//           dz_L = (Wd^T g_i) where a_L > 0 (the ReLU derivative, 0 at the kink);
//   layer l: dW_l (+)= sum over pixels of dz_l x im2col(a_{l-1}), db_l (+)= sum dz_l,
//           dz_{l-1} = (transposed conv of dz_l with W_l) where a_{l-1} > 0.
// The conv products run on the matrix cores, those of layers 2..L on the bf16
// ones with operands split three ways (rn_split.hpp), layer 1's dW on the
// float32 ones:
//   dx: per 4x4 tile of layer l-1 an implicit GEMM, M = 16 pixels, N = C_{l-1},
//       K = 9 C_l, i.e. a forward 3x3 conv of dz_l with the weights transposed
//       (input <-> output channels) and flipped (kernel position 8 - k), in
//       rn_conv_split.hip;
//   dW: M = C_l, N = 9 C_{l-1} + 1 (the last column, all ones, gives the bias
//       gradient), K = every pixel of every stream, split over teams of blocks
//       whose partial sums are added in team order (no atomics, so the result
//       is deterministic).
// The SGD step updates every packed copy of a weight in place.
#include "rn_split.hpp"
#include "rn_train.hpp"

namespace rn {
namespace {

using dev::floatx4;

// ------------------------------------------------------------------ REINFORCE

// g[i][o] = G_i (softmax(z_i)[o] - [o == a_i]): the derivative of
// -G_i log softmax(z_i)[a_i] with respect to z_i (one thread per stream).
__global__ __launch_bounds__(256) void k_reinforce(int n, int n_out, const float *z, const int32_t *act,
                                                   const float *ret, float *g) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float *zi = z + (size_t)i * n_out;
    float m = zi[0];
    for (int o = 1; o < n_out; ++o) m = fmaxf(m, zi[o]);
    float den = 0.f;
    for (int o = 0; o < n_out; ++o) den += expf(zi[o] - m);
    const float G = ret[i];
    const int a = act[i];
    for (int o = 0; o < n_out; ++o) {
        const float p = expf(zi[o] - m) / den;
        g[(size_t)i * n_out + o] = G * (p - (o == a ? 1.f : 0.f));
    }
}

// ------------------------------------------------------------------ dense head

// Up to NO logits.  Block (t, c) takes 4 blockDim.x of the 16 C head inputs of
// tile position t of the last layer (chunk c); a thread owns four consecutive
// inputs j (one 16-byte access per stream), keeps their NO weights and NO
// gradient sums in registers and walks the streams (their g rows staged in
// LDS).  Each input's sums run over o and over the streams in order.
template <int NO>
__global__ __launch_bounds__(512) void k_bwd_head(HeadBwdArgs a) {
    constexpr int V = 4;
    constexpr int kHeadStreams = 256;                     // streams per LDS stage of g
    __shared__ float s_g[kHeadStreams * NO];
    __shared__ int32_t s_slot[kHeadStreams];
    const int t = blockIdx.x;
    const int E = kTilePx * a.C;                          // a multiple of V
    const int ty = t / a.TW, tx = t - ty * a.TW;
    {
        const int j0 = (blockIdx.y * blockDim.x + threadIdx.x) * V;
        const bool ok = j0 < E;
        float w[V][NO], acc[V][NO];
#pragma unroll
        for (int v = 0; v < V; ++v)
#pragma unroll
            for (int o = 0; o < NO; ++o) {
                w[v][o] = ok && o < a.n_out ? a.wd[(size_t)o * a.K + (size_t)t * E + j0 + v] : 0.f;
                acc[v][o] = 0.f;
            }
        for (int i0 = 0; i0 < a.n; i0 += kHeadStreams) {
            const int nc = min(kHeadStreams, a.n - i0);
            __syncthreads();                      // the previous stage's readers are done
            for (int k = threadIdx.x; k < nc * NO; k += blockDim.x) {
                const int ii = k / NO, o = k - ii * NO;
                s_g[k] = o < a.n_out ? a.g[(size_t)(i0 + ii) * a.n_out + o] : 0.f;
            }
            for (int k = threadIdx.x; k < nc; k += blockDim.x) s_slot[k] = a.ids[i0 + k];
            __syncthreads();
            if (ok) {
#pragma unroll 4
                for (int ii = 0; ii < nc; ++ii) {
                    const float4 in = *reinterpret_cast<const float4 *>(a.act + (size_t)s_slot[ii] * a.act_stride + (size_t)t * E + j0);
                    const float *vin = reinterpret_cast<const float *>(&in);
                    float4 out;
                    float *vout = reinterpret_cast<float *>(&out);
#pragma unroll
                    for (int v = 0; v < V; ++v) {
                        float da = 0.f;
#pragma unroll
                        for (int o = 0; o < NO; ++o) {
                            const float gv = s_g[ii * NO + o];
                            da = fmaf(w[v][o], gv, da);
                            acc[v][o] = fmaf(gv, vin[v], acc[v][o]);
                        }
                        vout[v] = vin[v] > 0.f ? da : 0.f;
                    }
                    *reinterpret_cast<float4 *>(a.dz + ((size_t)(i0 + ii) * a.ntiles + t) * E + j0) = out;
                }
            }
        }
        if (ok) {
#pragma unroll
            for (int v = 0; v < V; ++v) {
                const int j = j0 + v, m = j / a.C, c = j - m * a.C;
                const int y = ty * kTile + (m >> 2), x = tx * kTile + (m & 3);
                if (y < a.H && x < a.W) {
#pragma unroll
                    for (int o = 0; o < NO; ++o) {
                        if (o >= a.n_out) break;
                        float *d = a.gwd + (size_t)o * a.C * a.H * a.W + ((size_t)c * a.H + y) * a.W + x;
                        *d = a.accumulate ? *d + acc[v][o] : acc[v][o];
                    }
                }
            }
        }
    }
    if (t == 0 && blockIdx.y == 0 && (int)threadIdx.x < a.n_out) {
        float s = 0.f;
        for (int i = 0; i < a.n; ++i) s += a.g[(size_t)i * a.n_out + threadIdx.x];
        a.gbd[threadIdx.x] = a.accumulate ? a.gbd[threadIdx.x] + s : s;
    }
}

// The same for more logits or few streams: block (t, r) takes row r of tile
// position t, a thread one input.  The weight gradients are [o][c][y][x], so a
// thread's sums go out through LDS and leave as the four pixels of a row
// (16 bytes), eight logits a round, and the tiles of one XCD are neighbours, so
// its L2 completes the lines: stored as they lie (4 bytes at H W apart a lane)
// they took most of the time (18 logits, 24 streams of 106x92: 408 us).
// vec: gwd is 16-byte aligned.
template <int NO>
__global__ __launch_bounds__(512) void k_bwd_head_row(HeadBwdArgs a, int vec) {
    constexpr int kStreams = NO <= 32 ? 128 : 64;         // streams per LDS stage of g
    constexpr int kRound = 8;
    __shared__ float s_g[kStreams * NO];
    __shared__ int32_t s_slot[kStreams];
    __shared__ float s_out[kRound * 512];
    const int per = (a.ntiles + 7) / 8, t = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
    if (t >= a.ntiles) return;                            // uniform per block
    const int E = kTilePx * a.C, n = 4 * a.C, tid = threadIdx.x;
    const int ty = t / a.TW, tx = t - ty * a.TW, y = ty * kTile + blockIdx.y;
    const bool ok = tid < n;
    const int j = blockIdx.y * n + (ok ? tid : 0);
    float w[NO], acc[NO];
#pragma unroll
    for (int o = 0; o < NO; ++o) {
        w[o] = ok && o < a.n_out ? a.wd[(size_t)o * a.K + (size_t)t * E + j] : 0.f;
        acc[o] = 0.f;
    }
    for (int i0 = 0; i0 < a.n; i0 += kStreams) {
        const int nc = min(kStreams, a.n - i0);
        __syncthreads();                                  // the previous stage's readers are done
        for (int k = tid; k < nc * NO; k += blockDim.x) {
            const int ii = k / NO, o = k - ii * NO;
            s_g[k] = o < a.n_out ? a.g[(size_t)(i0 + ii) * a.n_out + o] : 0.f;
        }
        for (int k = tid; k < nc; k += blockDim.x) s_slot[k] = a.ids[i0 + k];
        __syncthreads();
        if (ok) {
#pragma unroll 4
            for (int ii = 0; ii < nc; ++ii) {
                const float in = a.act[(size_t)s_slot[ii] * a.act_stride + (size_t)t * E + j];
                float da = 0.f;
#pragma unroll
                for (int o = 0; o < NO; ++o) {
                    const float gv = s_g[ii * NO + o];
                    da = fmaf(w[o], gv, da);
                    acc[o] = fmaf(gv, in, acc[o]);
                }
                a.dz[((size_t)(i0 + ii) * a.ntiles + t) * E + j] = in > 0.f ? da : 0.f;
            }
        }
    }
    if (y < a.H) {                                        // uniform per block; four whole pixels (W % 4 = 0)
#pragma unroll
        for (int o0 = 0; o0 < NO; o0 += kRound) {
            __syncthreads();
#pragma unroll
            for (int o = 0; o < kRound; ++o)
                if (o0 + o < NO) s_out[o * 512 + tid] = acc[o0 + o];
            __syncthreads();
            for (int k = tid; k < kRound * a.C; k += blockDim.x) {
                const int o = k / a.C, c = k - o * a.C;
                if (o0 + o >= a.n_out) break;
                float v[4];
#pragma unroll
                for (int p = 0; p < 4; ++p) v[p] = s_out[o * 512 + p * a.C + c];
                float *d = a.gwd + ((size_t)(o0 + o) * a.C + c) * a.H * a.W + (size_t)y * a.W + tx * kTile;
                if (vec) {
                    float4 *d4 = reinterpret_cast<float4 *>(d);
                    float4 q = make_float4(v[0], v[1], v[2], v[3]);
                    if (a.accumulate) {
                        const float4 b = *d4;
                        q = make_float4(b.x + v[0], b.y + v[1], b.z + v[2], b.w + v[3]);
                    }
                    *d4 = q;
                } else {
#pragma unroll
                    for (int p = 0; p < 4; ++p) d[p] = a.accumulate ? d[p] + v[p] : v[p];
                }
            }
        }
    }
    if (t == 0 && blockIdx.y == 0 && tid < a.n_out) {
        float s = 0.f;
        for (int i = 0; i < a.n; ++i) s += a.g[(size_t)i * a.n_out + tid];
        a.gbd[tid] = a.accumulate ? a.gbd[tid] + s : s;
    }
}

// ------------------------------------------------------------------ dW

// dW and db of layers 2..L on the bf16 matrix cores with operands split three
// ways (rn_split.hpp): a GEMM with M = output channels, N = (kernel position,
// input channel), K = pixels, on v_mfma_f32_16x16x32_bf16, two tiles (32
// pixels) a step.
//
// Bound: matrix issue, 6 x 2 * 16 * CZ * 9 CA flops a tile (the float32
// instruction needs 16/6 of that time), but the pipe is busy only 50% of the
// cycles at 40->80: three waves hold four column blocks, five three, and 40
// columns a kernel position are padded to 48.  A block of eight waves (two per SIMD)
// sums CZB output channels x CAB input channels of a team's tiles: the waves
// share out the 9 x CAB / 16 column blocks, each with all CZB / 16 row blocks
// in registers (80 accumulator registers).  A team has CA / CAB x CZ / CZB
// blocks, on one XCD where the teams allow it, since they read the same tiles.
// The tiles' dz and a_{l-1} halos sit in LDS as bf16 planes, pixel by pixel as
// in the caches (32 bytes of padding a pixel keep the banks apart); the matrix
// operands want consecutive pixels of one channel, which ds_read_b64_tr_b16
// gives: 16 lanes address 16 channels of four pixels and each receives its
// channel's four.  So a value is split and written once, and a kernel position
// is an address offset.  (The float32 kernels kept a transposed dz and three
// column-shifted halo copies in LDS.)  Two buffers of two tiles: while the
// matrix ops read one, the next step's tiles, loaded a step earlier, are split
// into the other between them; one barrier a step.
// A sum that is not finite is summed again in plain float32 by
// k_bwd_reduce_rows.
template <int CAB, int CZB>
struct DwSplit {
    static constexpr int MB = CZB / 16;                   // row blocks
    static constexpr int NBC = (CAB + 15) / 16;           // column blocks per kernel position
    static constexpr int NBT = 9 * NBC;
    static constexpr int NW = NBT / 8, EXTRA = NBT % 8;   // column blocks per wave; the first EXTRA waves have one more
    static constexpr int HS = CAB * 2 + 32, HP = 36 * HS; // bytes of a halo pixel, of a plane
    static constexpr int DS = CZB * 2 + 32, DP = 16 * DS;
    static constexpr int TILE = 3 * (HP + DP);
    static constexpr int BUF = 2 * TILE;
    static constexpr size_t lds_bytes = 2 * (size_t)BUF;
    static constexpr int HU = 36 * CAB / 4, DU = 16 * CZB / 4;   // 16-byte units of a tile
    static constexpr int UPT = (2 * (HU + DU) + 511) / 512;      // per thread
    static_assert(CZB % 16 == 0 && CAB % 8 == 0 && lds_bytes <= 160 * 1024, "block shape");
    static_assert(EXTRA < 8 && UPT <= NW, "a staging unit beside each column block");
};

__device__ __align__(16) float g_zero_unit[4];

typedef short shortx4 __attribute__((ext_vector_type(4)));
typedef short shortx8 __attribute__((ext_vector_type(8)));

// Two transposed reads: pixels of the halves' first and second row of four.
__device__ inline dev::bf16x8 tr_frag(const unsigned char *p, int second) {
    const shortx4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) shortx4 *)p);
    const shortx4 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) shortx4 *)(p + second));
    return __builtin_bit_cast(dev::bf16x8, __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7));
}

template <int CAB, int CZB, int NW, bool BIAS, typename Fetch, typename Stage>
__device__ inline void dw_split_wave(const BwdArgs &a, const unsigned char *lds, int q0, int steps, int team, int ci0, int co0,
                                     Fetch fetch, Stage stage) {
    using D = DwSplit<CAB, CZB>;
    using dev::bf16x8;
    const int lane = threadIdx.x & 63, kq = lane >> 4, col = lane & 15;
    // Lane group kq takes tile kq / 2, pixel rows 2 (kq % 2) and the next; its
    // lane i addresses pixel i / 4 of a row, channels 4 (i % 4) ..
    const int tile = (kq >> 1) * D::TILE, row = 2 * (kq & 1), px = col >> 2, c4 = (col & 3) * 8;
    const unsigned char *ab = lds + tile + 3 * D::HP + (row * 4 + px) * D::DS + c4;
    const unsigned char *bb = lds + tile + (row * 6 + px) * D::HS + c4;
    int boff[NW];
#pragma unroll
    for (int k = 0; k < NW; ++k) {
        const int pos = (q0 + k) / D::NBC, nb = (q0 + k) - pos * D::NBC;
        boff[k] = (pos / 3 * 6 + pos % 3) * D::HS + nb * 32;
    }
    floatx4 acc[D::MB][NW], accb[BIAS ? D::MB : 1];
#pragma unroll
    for (int m = 0; m < D::MB; ++m) {
        if constexpr (BIAS) accb[m] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < NW; ++k) acc[m][k] = floatx4{0.f, 0.f, 0.f, 0.f};
    }
    bf16x8 ones;
#pragma unroll
    for (int i = 0; i < 8; ++i) ones[i] = (__bf16)1.0f;
    int buf = 0;
    for (int s = 0; s < steps; ++s) {
        bf16x8 x[D::MB][3];
#pragma unroll
        for (int m = 0; m < D::MB; ++m)
#pragma unroll
            for (int pl = 0; pl < 3; ++pl) x[m][pl] = tr_frag(ab + buf * D::BUF + pl * D::DP + m * 32, 4 * D::DS);
        bf16x8 y[3];
#pragma unroll
        for (int pl = 0; pl < 3; ++pl) y[pl] = tr_frag(bb + buf * D::BUF + boff[0] + pl * D::HP, 6 * D::HS);
#pragma unroll
        for (int k = 0; k < NW; ++k) {
            bf16x8 yn[3];
            if (k + 1 < NW) {
#pragma unroll
                for (int pl = 0; pl < 3; ++pl) yn[pl] = tr_frag(bb + buf * D::BUF + boff[k + 1] + pl * D::HP, 6 * D::HS);
            }
            __builtin_amdgcn_sched_barrier(0);
            // (dz plane, a plane), small terms first
            constexpr int px_[6] = {2, 0, 1, 1, 0, 0}, py_[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
            for (int p = 0; p < 6; ++p)
#pragma unroll
                for (int m = 0; m < D::MB; ++m)
                    acc[m][k] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x[m][px_[p]], y[py_[p]], acc[m][k], 0, 0, 0);
            if (k < D::UPT) stage(k, buf ^ 1);            // the next step's tiles
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int pl = 0; pl < 3; ++pl) y[pl] = yn[pl];
        }
        if constexpr (BIAS) {
#pragma unroll
            for (int pl = 2; pl >= 0; --pl)
#pragma unroll
                for (int m = 0; m < D::MB; ++m)
                    accb[m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x[m][pl], ones, accb[m], 0, 0, 0);
        }
        fetch(s + 2);
        dev::lds_barrier();                               // the other buffer staged, this one read
        buf ^= 1;
    }
    const int NQ = 9 * a.ca + 1;
    float *part = a.part + (size_t)team * a.cz * NQ;      // [team][co][column]: 16 lanes write 64 bytes
#pragma unroll
    for (int m = 0; m < D::MB; ++m) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const size_t base = (size_t)(co0 + 16 * m + 4 * kq + r) * NQ;
#pragma unroll
            for (int k = 0; k < NW; ++k) {
                const int pos = (q0 + k) / D::NBC, ci = 16 * ((q0 + k) - pos * D::NBC) + col;
                if (ci < CAB) part[base + pos * a.ca + ci0 + ci] = acc[m][k][r];
            }
            if constexpr (BIAS)
                if (ci0 == 0 && col == 0) part[base + 9 * a.ca] = accb[m][r];
        }
    }
}

template <int CA, int CZ, int CAB, int CZB>
__global__ __launch_bounds__(512, 2) void k_bwd_dw_split(BwdArgs a) {
    using D = DwSplit<CAB, CZB>;
    using dev::bf16x4;
    constexpr int PZ = CZ / CZB, BPT = CA / CAB * PZ;     // blocks per team
    extern __shared__ __align__(16) unsigned char lds[];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // Blocks go round robin over the 8 XCDs: a team's blocks 8 apart.
    const int b = blockIdx.x, j8 = b >> 3;
    const bool whole = a.teams % 8 == 0;
    const int team = whole ? j8 / BPT * 8 + (b & 7) : b / BPT, part = whole ? j8 % BPT : b % BPT;
    const int co0 = part % PZ * CZB, ci0 = part / PZ * CAB;
    const long long NT = (long long)a.n * a.ntiles;
    const int t0 = (int)(NT * team / a.teams), t1 = (int)(NT * (team + 1) / a.teams);
    const int steps = (t1 - t0 + 1) / 2;
    int fi = t0 / a.ntiles, ft = t0 - fi * a.ntiles;      // the next tile to load
    const __attribute__((address_space(4))) int32_t *ids = (const __attribute__((address_space(4))) int32_t *)a.ids;
    floatx4 pre[D::UPT];
    // This thread's units of step s's two tiles (past the team's last: zeros).
    auto fetch = [&](int s) __attribute__((always_inline)) {
        bool ok[2];
        int ty[2], tx[2];
        const float *act[2], *dz[2];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            ok[t] = t0 + 2 * s + t < t1;
            const int i = __builtin_amdgcn_readfirstlane(ok[t] ? fi : 0), tl = ok[t] ? ft : 0;
            if (++ft == a.ntiles) {
                ft = 0;
                ++fi;
            }
            ty[t] = tl / a.TW;
            tx[t] = tl - ty[t] * a.TW;
            act[t] = a.act_prev + (size_t)ids[i] * a.prev_stride + ci0;
            dz[t] = a.dz_in + ((size_t)i * a.ntiles + tl) * kTilePx * CZ + co0;
        }
#pragma unroll
        for (int k = 0; k < D::UPT; ++k) {
            const int u = threadIdx.x + 512 * k;
            const int hu = u < D::HU ? u : u - D::HU, t = u < 2 * D::HU ? (u >= D::HU) : (u - 2 * D::HU >= D::DU);
            const float *src = g_zero_unit;
            if (u < 2 * D::HU) {
                const int pos = hu / (CAB / 4), c = hu - pos * (CAB / 4);
                const int y = ty[t] * kTile - 1 + pos / 6, x = tx[t] * kTile - 1 + pos % 6;
                if (ok[t] && y >= 0 && y < a.H && x >= 0 && x < a.W)
                    src = act[t] + ((size_t)((y >> 2) * a.TW + (x >> 2)) * kTilePx + (y & 3) * 4 + (x & 3)) * CA + 4 * c;
            } else if (u < 2 * (D::HU + D::DU)) {
                const int v = u - 2 * D::HU - (t ? D::DU : 0), p = v / (CZB / 4), c = v - p * (CZB / 4);
                if (ok[t]) src = dz[t] + p * CZ + 4 * c;
            }
            pre[k] = *reinterpret_cast<const floatx4 *>(src);
        }
    };
    auto stage = [&](int k, int buf) __attribute__((always_inline)) {
        const int u = threadIdx.x + 512 * k;
        int off, plane;
        if (u < 2 * D::HU) {
            const int t = u >= D::HU, v = u - (t ? D::HU : 0), pos = v / (CAB / 4), c = v - pos * (CAB / 4);
            off = t * D::TILE + pos * D::HS + 8 * c;
            plane = D::HP;
        } else {
            const int w = u - 2 * D::HU, t = w >= D::DU, v = w - (t ? D::DU : 0), p = v / (CZB / 4), c = v - p * (CZB / 4);
            off = t * D::TILE + 3 * D::HP + p * D::DS + 8 * c;
            plane = D::DP;
        }
        if (u < 2 * (D::HU + D::DU)) {
            unsigned char *d = lds + buf * D::BUF + off;
            bf16x4 h, m, l;
            dev::split4(pre[k], h, m, l);
            *reinterpret_cast<bf16x4 *>(d) = h;
            *reinterpret_cast<bf16x4 *>(d + plane) = m;
            *reinterpret_cast<bf16x4 *>(d + 2 * plane) = l;
        }
    };
    fetch(0);
#pragma unroll
    for (int k = 0; k < D::UPT; ++k) stage(k, 0);
    fetch(1);
    dev::lds_barrier();
    const int q0 = wave * D::NW + min(wave, D::EXTRA);
    if (wave < D::EXTRA)
        dw_split_wave<CAB, CZB, D::NW + 1, false>(a, lds, q0, steps, team, ci0, co0, fetch, stage);
    else if (wave < 7)
        dw_split_wave<CAB, CZB, D::NW, false>(a, lds, q0, steps, team, ci0, co0, fetch, stage);
    else
        dw_split_wave<CAB, CZB, D::NW, true>(a, lds, q0, steps, team, ci0, co0, fetch, stage);
}

// dW for layer 1 (a_0 the float32 input planes, 1 or 4 channels): so few
// columns (9 cin + 1) that staging a tile through LDS for a handful of matrix
// ops costs more than the ops.  Each wave is a team of its own and walks its
// tiles with the operands loaded straight into the matrix layout (lane
// (m, kq), k-step j: A = dz at pixel (row kq, column j), channel 16 mb + m;
// B = the input at that pixel shifted by the column's kernel position, or 1
// for the bias column), the next tile's loads issued before this tile's
// matrix ops.  Memory-bound: each tile's dz (16 x CZ floats) is read once.
template <int CA, int CZ>
struct DwFirst {
    static constexpr int NQ = 9 * CA + 1;
    static constexpr int NBQ = (NQ + 15) / 16;            // 16-column blocks
    static constexpr int MB = (CZ + 15) / 16;             // 16-row blocks
};

template <int CA, int CZ>
__global__ __launch_bounds__(256) void k_bwd_dw_first(BwdArgs a) {
    using D = DwFirst<CA, CZ>;
    const int lane = threadIdx.x & 63;
    const int team = blockIdx.x * 4 + (threadIdx.x >> 6);
    const int kq = lane >> 4, col = lane & 15;
    const long long NT = (long long)a.n * a.ntiles;
    const int t0 = (int)(NT * team / a.teams), t1 = (int)(NT * (team + 1) / a.teams);
    if (team >= a.teams) return;                           // uniform per wave
    // This lane's column per block: kernel position offset (ky, kx) and input
    // channel, or the bias / padding column.
    int qky[D::NBQ], qkx[D::NBQ], qci[D::NBQ], qkind[D::NBQ];   // kind 0: input, 1: bias, 2: zero
#pragma unroll
    for (int k = 0; k < D::NBQ; ++k) {
        const int q = 16 * k + col;
        const int kpos = q / CA;
        qci[k] = q - kpos * CA;
        qky[k] = kpos / 3;
        qkx[k] = kpos - 3 * (kpos / 3);
        qkind[k] = q < 9 * CA ? 0 : q == 9 * CA ? 1 : 2;
    }
    floatx4 acc[D::MB][D::NBQ];
#pragma unroll
    for (int m = 0; m < D::MB; ++m)
#pragma unroll
        for (int k = 0; k < D::NBQ; ++k) acc[m][k] = floatx4{0.f, 0.f, 0.f, 0.f};
    const size_t HW = (size_t)a.H * a.W;
    float av[2][D::MB][4], bv[2][D::NBQ][4];
    int fi = t0 / a.ntiles, ft = t0 - fi * a.ntiles;
    auto fetch = [&](int slot_buf) __attribute__((always_inline)) {
        const int i = fi, t = ft;
        if (++ft == a.ntiles) {
            ft = 0;
            ++fi;
        }
        const int ty = t / a.TW, tx = t - ty * a.TW;
        const int slot = a.ids[i];
        const float *dz = a.dz_in + ((size_t)i * a.ntiles + t) * kTilePx * CZ;
#pragma unroll
        for (int m = 0; m < D::MB; ++m) {
            const int co = 16 * m + col;
#pragma unroll
            for (int j = 0; j < 4; ++j) av[slot_buf][m][j] = co < CZ ? dz[(4 * kq + j) * CZ + co] : 0.f;
        }
        const int head = a.stack != 1 ? a.ring_head[slot] : 0;
#pragma unroll
        for (int k = 0; k < D::NBQ; ++k) {
            const float *plane;
            if (a.stack == 1) {
                plane = a.act_prev + ((size_t)slot * CA + qci[k]) * HW;
            } else {
                const int jj = qci[k] / a.cin0, c1 = qci[k] - jj * a.cin0;
                const int rp = (head - (a.stack - 1) + jj + 4 * a.stack) & 3;
                plane = a.act_prev + (((size_t)slot * 4 + rp) * a.cin0 + c1) * HW;
            }
            const int y = ty * kTile - 1 + kq + qky[k];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int x = tx * kTile - 1 + j + qkx[k];
                const bool in = qkind[k] == 0 && y >= 0 && y < a.H && x >= 0 && x < a.W;
                bv[slot_buf][k][j] = in ? plane[(size_t)y * a.W + x] : (qkind[k] == 1 ? 1.f : 0.f);
            }
        }
    };
    if (t0 < t1) fetch(0);
    for (int tt = t0; tt < t1; tt += 2) {
        if (tt + 1 < t1) fetch(1);                         // in flight during tile tt's matrix ops
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int m = 0; m < D::MB; ++m)
#pragma unroll
                for (int k = 0; k < D::NBQ; ++k)
                    acc[m][k] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[0][m][j], bv[0][k][j], acc[m][k], 0, 0, 0);
        if (tt + 1 >= t1) break;
        if (tt + 2 < t1) fetch(0);
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int m = 0; m < D::MB; ++m)
#pragma unroll
                for (int k = 0; k < D::NBQ; ++k)
                    acc[m][k] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[1][m][j], bv[1][k][j], acc[m][k], 0, 0, 0);
    }
#pragma unroll
    for (int m = 0; m < D::MB; ++m)
#pragma unroll
        for (int k = 0; k < D::NBQ; ++k) {
            const int q = 16 * k + col;
            if (q >= D::NQ) continue;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int co = 16 * m + 4 * kq + r;
                if (co < CZ) a.part[((size_t)co * D::NQ + q) * a.teams + team] = acc[m][k][r];
            }
        }
}

// Where the gradient of weight e = (co, column) of a layer goes.
__device__ inline float *dw_dest(const BwdArgs &a, int e) {
    const int NQ = 9 * a.ca + 1, co = e / NQ, q = e - co * NQ;
    if (q == 9 * a.ca) return a.gb + co;
    const int kpos = q / a.ca, ci = q - kpos * a.ca;
    return a.gw + ((size_t)co * a.ca + ci) * 9 + kpos;
}

// Layer 1's dW and db from the teams' partial sums ([co][column][team]): one
// wave per weight, lane j adding teams j, j + 64, ... in order, then the lanes'
// sums by a fixed butterfly, so the order never changes.
__global__ __launch_bounds__(256) void k_bwd_reduce(BwdArgs a) {
    const int NQ = 9 * a.ca + 1;
    const int e = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (e >= a.cz * NQ) return;                            // uniform per wave
    const float *p = a.part + (size_t)e * a.teams;
    float s = 0.f;
    for (int team = lane; team < a.teams; team += 64) s += p[team];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
    if (lane != 0) return;
    float *d = dw_dest(a, e);
    *d = a.accumulate ? *d + s : s;
}

// A team's share of the gradient of weight e in plain float32 products, one
// lane of 64 taking every 64th pixel of its tiles (the whole wave's sum is
// returned, NaN as soon as it must be).
__device__ inline float dw_plain(const BwdArgs &a, int e, int team, int lane) {
    constexpr int U = 4;                                   // tiles a lane loads at once
    const int NQ = 9 * a.ca + 1, co = e / NQ, q = e - co * NQ, kpos = q / a.ca, ci = q - kpos * a.ca;
    const bool bias = q == 9 * a.ca;
    const int dy = bias ? 0 : kpos / 3 - 1, dx = bias ? 0 : kpos % 3 - 1;
    const long long NT = (long long)a.n * a.ntiles;
    const int t0 = (int)(NT * team / a.teams), t1 = (int)(NT * (team + 1) / a.teams), m = lane & 15;
    float s = 0.f;
    for (int b = t0; b < t1; b += 4 * U) {                 // four tiles of 16 pixels a wave, U times
        float d[U], v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int T = b + 4 * u + (lane >> 4), Tc = min(T, t1 - 1), i = Tc / a.ntiles, t = Tc - i * a.ntiles, ty = t / a.TW;
            const int y = ty * kTile + (m >> 2) + dy, x = (t - ty * a.TW) * kTile + (m & 3) + dx;
            const int yc = min(max(y, 0), a.H - 1), xc = min(max(x, 0), a.W - 1);
            const float act = bias ? 1.f : a.act_prev[(size_t)a.ids[i] * a.prev_stride +
                                                      ((size_t)((yc >> 2) * a.TW + (xc >> 2)) * kTilePx + (yc & 3) * 4 + (xc & 3)) * a.ca + ci];
            const float dz = a.dz_in[((size_t)Tc * kTilePx + m) * a.cz + co];
            d[u] = T < t1 ? dz : 0.f;
            v[u] = T < t1 && (bias || (y == yc && x == xc)) ? act : 0.f;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) s = fmaf(d[u], v[u], s);
        if (__any(__builtin_isnan(s)) || (__any(s == __builtin_inff()) && __any(s == -__builtin_inff())))
            return __uint_as_float(0x7fc00000u);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
    return s;
}

// dW_l and db_l of layers 2..L from partial sums [team][co][column]: a block
// takes 64 weights, wave w the w-th quarter of the teams in order (four sums,
// teams mod 4), then the quarters in order.  Loads and the kernel's stores are
// contiguous; with the team fastest every store was 4 bytes on a line of its
// own (28880 weights of 256 teams, 4 streams of 105x80: 135 us in all).  Where
// the sum is not finite, the partial sums that are not are taken again from
// plain float32 products, the block's waves taking such weights in turn, team
// by team until the sum is NaN (whatever follows); a team ends there too.
__global__ __launch_bounds__(256) void k_bwd_reduce_rows(BwdArgs a) {
    __shared__ float s_sum[4][64];
    const int total = a.cz * (9 * a.ca + 1);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, e = blockIdx.x * 64 + lane;
    const int t0 = a.teams * wave / 4, t1 = a.teams * (wave + 1) / 4;
    float s[4] = {0.f, 0.f, 0.f, 0.f};
    if (e < total) {
        const float *p = a.part + e;
#pragma unroll 4
        for (int t = t0; t < t1; t += 4)
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (t + k < t1) s[k] += p[(size_t)(t + k) * total];
    }
    s_sum[wave][lane] = (s[0] + s[1]) + (s[2] + s[3]);
    __syncthreads();
    float v = (s_sum[0][lane] + s_sum[1][lane]) + (s_sum[2][lane] + s_sum[3][lane]);
    const uint64_t plain = __ballot(e < total && !dev::is_finite(v));      // the same in every wave
    if (plain) {                                           // rare: one weight at a time, by a whole wave
        __syncthreads();                                   // every wave has read the sums
        int turn = 0;
        for (uint64_t left = plain; left; left &= left - 1, ++turn) {
            if ((turn & 3) != wave) continue;              // uniform per wave
            const int j = __ffsll((long long)left) - 1, ej = blockIdx.x * 64 + j;
            float f = 0.f;
            for (int b = 0; b < a.teams && !__builtin_isnan(f); b += 64) {     // uniform: every lane has the sum
                const float pt = b + lane < a.teams ? a.part[(size_t)(b + lane) * total + ej] : 0.f;
                const bool fin = dev::is_finite(pt);
                float good = fin ? pt : 0.f;
#pragma unroll
                for (int o = 32; o > 0; o >>= 1) good += __shfl_xor(good, o, 64);
                f += good;
                for (uint64_t bad = __ballot(!fin); bad && !__builtin_isnan(f); bad &= bad - 1)
                    f += dw_plain(a, ej, b + __ffsll((long long)bad) - 1, lane);
            }
            if (lane == 0) s_sum[0][j] = f;
        }
        __syncthreads();
        if (plain >> lane & 1) v = s_sum[0][lane];
    }
    if (wave > 0) return;
    if (e >= total) return;
    float *d = dw_dest(a, e);
    *d = a.accumulate ? *d + v : v;
}

// ------------------------------------------------------------------ SGD

// Natural-layout index of packed element d (or -1 for a padding zero).
__device__ inline long long sgd_src(const SgdArgs &a, size_t d) {
    switch (a.kind) {
    case SGD_FIRST: {                                         // [ci * 9 + k][co]
        const int co = (int)(d % a.cout);
        const size_t r = d / a.cout;
        const int ci = (int)(r / 9), k = (int)(r % 9);
        return ((long long)co * a.cin + ci) * 9 + k;
    }
    case SGD_MFMA: {                                          // [kpos][block][nb][lane][j]
        const size_t per = (size_t)a.cin * a.cout;
        const int kpos = (int)(d / per);
        size_t r = d - (size_t)kpos * per;
        const int nf = a.cin / 16;
        const size_t full = (size_t)nf * 16 * a.cout;
        int ci, n;
        if (r < full) {
            const int b = (int)(r / (16 * a.cout));
            const int rb = (int)(r - (size_t)b * 16 * a.cout);
            const int nb = rb / 256, l = (rb / 4) % 64, j = rb % 4;
            ci = 16 * b + 4 * (l / 16) + j;
            n = nb * 16 + l % 16;
        } else {
            const int rt = (int)(r - full);
            const int nb = rt / 128, l = (rt / 2) % 64, j = rt % 2;
            ci = 16 * nf + 2 * (l / 16) + j;
            n = nb * 16 + l % 16;
        }
        return ((long long)n * a.cin + ci) * 9 + kpos;
    }
    case SGD_DENSE: {                                         // [o][tile][16][C], 0 outside the image
        const int o = (int)(d / a.K);
        const size_t e = d - (size_t)o * a.K;
        const int c = (int)(e % a.C), m = (int)((e / a.C) % kTilePx), tile = (int)(e / ((size_t)kTilePx * a.C));
        const int ty = tile / a.TW, tx = tile - ty * a.TW;
        const int y = ty * kTile + m / 4, x = tx * kTile + m % 4;
        if (y >= a.H || x >= a.W) return -1;
        return (long long)o * a.C * a.H * a.W + ((long long)c * a.H + y) * a.W + x;
    }
    case SGD_TILE_HEAD: {                                     // [o][tile][nb][lane][i]
        const int NB = a.C / 16;
        const int i = (int)(d % 4), l = (int)((d / 4) % 64), nb = (int)((d / 256) % NB);
        const size_t r = d / (256 * (size_t)NB);
        const int tile = (int)(r % a.ntiles), o = (int)(r / a.ntiles);
        const int ty = tile / a.TW, tx = tile - ty * a.TW;
        const int c = nb * 16 + l % 16, y = ty * kTile + i, x = tx * kTile + l / 16;
        if (y >= a.H || x >= a.W) return -1;
        return (long long)o * a.C * a.H * a.W + ((long long)c * a.H + y) * a.W + x;
    }
    case SGD_TILE_PART: {                                     // [tile][b][kq][o][j], b < C
        const int j = (int)(d % 4);
        size_t r = d / 4;
        const int o = (int)(r % a.n_out);
        r /= a.n_out;
        const int kq = (int)(r % 4);
        r /= 4;
        const int b = (int)(r % a.C), tile = (int)(r / a.C);
        const int k = 16 * b + 4 * kq + j, m = k / a.C, c = k - m * a.C;
        const int ty = tile / a.TW, tx = tile - ty * a.TW;
        const int y = ty * kTile + m / 4, x = tx * kTile + m % 4;
        if (y >= a.H || x >= a.W) return -1;
        return (long long)o * a.C * a.H * a.W + ((long long)c * a.H + y) * a.W + x;
    }
    case SGD_DX: {                                            // [b][nb][lane][j], cin = ca, cout = cz
        const int NB = (a.cin + 15) / 16;
        const int j = (int)(d % 4), l = (int)((d / 4) % 64), nb = (int)((d / 256) % NB);
        const int b = (int)(d / (256 * (size_t)NB));
        const int K = 16 * b + 4 * (l / 16) + j, n = nb * 16 + l % 16;
        if (n >= a.cin) return -1;
        const int kpos = K / a.cout, co = K - kpos * a.cout;
        return ((long long)co * a.cin + n) * 9 + (8 - kpos);
    }
    default:
        return (long long)d;
    }
}

// Two roundings, fl(w - fl(lr g)), as a host computing the same update in
// float32 does: contraction into one fused multiply-add is switched off.
// assign: a plain gather into the packed layout (padding elements 0).
__global__ __launch_bounds__(256) void k_sgd(SgdArgs a) {
#pragma clang fp contract(off)
    for (size_t d = (size_t)blockIdx.x * blockDim.x + threadIdx.x; d < a.count; d += (size_t)gridDim.x * blockDim.x) {
        const long long s = sgd_src(a, d);
        if (a.assign) {
            a.dst[d] = s >= 0 ? a.g[s] : 0.f;
        } else if (s >= 0) {
            const float step = a.lr * a.g[s];
            a.dst[d] = a.dst[d] - step;
        }
    }
}

__global__ __launch_bounds__(256) void k_unprime(int32_t *primed, int S) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < S) primed[i] = 0;
}

// ------------------------------------------------------------------ launchers

#define RN_DW_FIRST_SHAPES(X) X(1, 20) X(1, 40) X(1, 64) X(1, 80) X(4, 20) X(4, 40) X(4, 64) X(4, 80)
// (input, output channels, those of a block)
#define RN_DW_SHAPES(X) X(40, 80, 40, 80) X(64, 128, 64, 64) X(128, 128, 64, 64)

int dw_blocks_per_team(int ca, int cz, bool first) {
#define X(a_, z_) \
    if (first && ca == a_ && cz == z_) return 1;
    RN_DW_FIRST_SHAPES(X)
#undef X
#define X(a_, z_, ab, zb) \
    if (!first && ca == a_ && cz == z_) return a_ / ab * (z_ / zb);
    RN_DW_SHAPES(X)
#undef X
    return 0;
}

template <int CA, int CZ>
hipError_t run_dw_first(const BwdArgs &a, hipStream_t s) {
    hipLaunchKernelGGL((k_bwd_dw_first<CA, CZ>), dim3((a.teams + 3) / 4), dim3(256), 0, s, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int total = CZ * DwFirst<CA, CZ>::NQ;
    hipLaunchKernelGGL(k_bwd_reduce, dim3((total + 3) / 4), dim3(256), 0, s, a);
    return hipGetLastError();
}

template <int CA, int CZ, int CAB, int CZB>
hipError_t run_dw_split(const BwdArgs &a, hipStream_t s) {
    auto kern = k_bwd_dw_split<CA, CZ, CAB, CZB>;
    constexpr size_t lds = DwSplit<CAB, CZB>::lds_bytes;
    static hipError_t attr = dev::set_lds(kern, lds);
    if (attr != hipSuccess) return attr;
    hipLaunchKernelGGL(kern, dim3(CA / CAB * (CZ / CZB) * a.teams), dim3(512), lds, s, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int total = CZ * (9 * CA + 1);
    hipLaunchKernelGGL(k_bwd_reduce_rows, dim3((total + 63) / 64), dim3(256), 0, s, a);
    return hipGetLastError();
}

}  // namespace

bool train_shapes_supported(int ca, int cz, bool first) { return dw_blocks_per_team(ca, cz, first) > 0; }

size_t dx_weights_elems(int cz, int ca) { return (size_t)9 * cz * ((ca + 15) / 16) * 16; }

void pack_dx_weights(const float *oihw, int ca, int cz, float *dst) {
    // [b][nb][lane][j]: K = 16 b + 4 (lane / 16) + j is (kernel position
    // K / cz, channel K % cz of layer l), column n = 16 nb + lane % 16 is
    // channel n of layer l-1; the value is W_l[K % cz][n] at the flipped
    // position 8 - K / cz, 0 for padding columns.
    const int NB = (ca + 15) / 16, KB = 9 * cz / 16;
    size_t d = 0;
    for (int b = 0; b < KB; ++b)
        for (int nb = 0; nb < NB; ++nb)
            for (int l = 0; l < 64; ++l)
                for (int j = 0; j < 4; ++j) {
                    const int K = 16 * b + 4 * (l / 16) + j, n = nb * 16 + l % 16;
                    const int kpos = K / cz, co = K % cz;
                    dst[d++] = n < ca ? oihw[((size_t)co * ca + n) * 9 + (8 - kpos)] : 0.f;
                }
}

int bwd_dw_teams(int ca, int cz, bool first, int n, int ntiles, int cus) {
    if (first) {
        // a team per wave, 16 waves per CU, at least 8 tiles each
        const long long tiles = (long long)n * ntiles;
        return (int)std::max(1LL, std::min(16LL * cus, (tiles + 7) / 8));
    }
    const int bpt = std::max(1, dw_blocks_per_team(ca, cz, first));
    const long long tiles = (long long)n * ntiles;
    // One block per CU, one round: its two buffers take most of LDS, and equal
    // tile ranges finish together (more, shorter teams each add a partial to
    // reduce).
    const long long want = std::max(1, cus / bpt);
    return (int)std::max(1LL, std::min(want, (tiles + 7) / 8));
}

size_t bwd_dw_part_elems(int ca, int cz, int teams) { return (size_t)teams * cz * (9 * ca + 1); }

hipError_t launch_reinforce(int n, int n_out, const float *logits, const int32_t *actions, const float *returns,
                            float *g, hipStream_t s) {
    hipLaunchKernelGGL(k_reinforce, dim3((n + 255) / 256), dim3(256), 0, s, n, n_out, logits, actions, returns, g);
    return hipGetLastError();
}

hipError_t launch_bwd_head(const HeadBwdArgs &a, hipStream_t s) {
    if (a.W % 4 != 0 || a.C > 128) return hipErrorInvalidValue;
    if (a.n_out <= 8 && a.n >= 48) {
        // A float4 of inputs per thread, one block per tile up to 512 threads:
        // the caches' bytes bound it (64 streams of 105x80, 6 logits: 105 us
        // against 113 by rows, 256: 341 against 420).  With few streams the
        // weight gradients' stores do (16 streams: 33 us by rows against 47,
        // 24 of 106x92 with 128 channels: 83 against 108).
        const int q = kTilePx * a.C / 4, th = std::min(512, (q + 63) / 64 * 64);
        hipLaunchKernelGGL((k_bwd_head<8>), dim3(a.ntiles, (q + th - 1) / th), dim3(th), 0, s, a);
        return hipGetLastError();
    }
    const dim3 grid((a.ntiles + 7) / 8 * 8, 4), block((4 * a.C + 63) / 64 * 64);
    const int vec = reinterpret_cast<uintptr_t>(a.gwd) % 16 == 0;
    if (a.n_out <= 8) hipLaunchKernelGGL((k_bwd_head_row<8>), grid, block, 0, s, a, vec);
    else if (a.n_out <= 18) hipLaunchKernelGGL((k_bwd_head_row<18>), grid, block, 0, s, a, vec);
    else if (a.n_out <= 32) hipLaunchKernelGGL((k_bwd_head_row<32>), grid, block, 0, s, a, vec);
    else hipLaunchKernelGGL((k_bwd_head_row<64>), grid, block, 0, s, a, vec);
    return hipGetLastError();
}

hipError_t launch_bwd_dw(const BwdArgs &a, int cus, hipStream_t s) {
    (void)cus;
    const bool first = a.first != 0;
#define X(a_, z_) \
    if (first && a.ca == a_ && a.cz == z_) return run_dw_first<a_, z_>(a, s);
    RN_DW_FIRST_SHAPES(X)
#undef X
#define X(a_, z_, ab, zb) \
    if (!first && a.ca == a_ && a.cz == z_) return run_dw_split<a_, z_, ab, zb>(a, s);
    RN_DW_SHAPES(X)
#undef X
    return hipErrorInvalidValue;
}

hipError_t launch_sgd(const SgdArgs &a, hipStream_t s) {
    if (a.count == 0) return hipSuccess;
    const size_t blocks = std::min<size_t>((a.count + 255) / 256, 65536);
    hipLaunchKernelGGL(k_sgd, dim3((unsigned)blocks), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_unprime(int32_t *primed, int S, hipStream_t s) {
    hipLaunchKernelGGL(k_unprime, dim3((S + 255) / 256), dim3(256), 0, s, primed, S);
    return hipGetLastError();
}

}  // namespace rn
