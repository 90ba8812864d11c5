// lb_mlp: the restoring-force surrogate's forward, backward and Adam kernels for gfx950, and the
// C ABI declared in include/lb_mlp.h.
//
// Products run on the matrix cores: v_mfma_f32_16x16x16_bf16 with BF16 operands rounded (nearest
// even) from FP32 as they are staged, FP32 accumulation in the order of k, and fused epilogues (bias,
// tanh, tanh derivative).  Master weights, gradients and Adam moments are FP32.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <memory>
#include <mutex>
#include <string>
#include <type_traits>
#include <vector>

#include "lb.h"
#include "lb_launch.h"
#include "lb_mlp.h"

namespace {

typedef short bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 hw_bf16x4 __attribute__((ext_vector_type(4)));

// four values rounded to BF16 (nearest even; the conversion instruction of the target)
__device__ __forceinline__ bf16x4 bf16_rne4(f32x4 v) {
    return __builtin_bit_cast(bf16x4, __builtin_convertvector(v, hw_bf16x4));
}

enum Epi { EPI_STORE = 0, EPI_BIAS = 1, EPI_BIAS_TANH = 2, EPI_TANH_GRAD = 3 };

constexpr int TM = 64, TN = 64, TK = 64;
constexpr int lds_row(int KT) { return KT + 8; }   // LDS row stride in BF16 values: 36 words for 64 of k, so the
                                                   // 16 rows of an operand read start at 16 different
                                                   // multiples of four banks
constexpr int LDK = lds_row(TK);

// Loads through a buffer resource return zero for an offset beyond its range, so what lies outside an
// operand is loaded with kOut as its offset instead of being branched around: the loads of a trip
// then issue back to back and stay in flight until their own values are used.
constexpr unsigned kOut = 0xfffffff0u;
__device__ __forceinline__ __amdgpu_buffer_rsrc_t operand_rsrc(const float *p) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(p), (short)0, 0x7fffffff, 0x00020000);
}
__device__ __forceinline__ float load1(__amdgpu_buffer_rsrc_t r, unsigned off) {
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, (int)off, 0, 0));
}
__device__ __forceinline__ f32x4 load4(__amdgpu_buffer_rsrc_t r, unsigned off) {
    return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, 0, 0));
}

// One thread's share of a 64 x KT operand tile (KT 64, or 16 with KC), as the KT / 16 float4 it loads.  KC: the
// operand is contiguous along k (element (r, k) at p[r * ld + k]) and the thread takes k4 .. k4+3 of rows
// r0, r0+16, r0+32, r0+48 (one row of 64 for KT 16).  Otherwise it is contiguous along the rows (element at
// p[k * ld + r]) and the thread takes the 4 x 4 block of rows r0 .. r0+3 and k4 .. k4+3, v[i] holding k4 + i.
// VEC: p and ld, and with ld the extent along the contiguous direction, are multiples of four
// floats.  Values outside R x K are zero.
// Buffer offsets are taken from the tile's corner and hold 63 rows (or k) of up to kLongRow floats: any
// network's, whose widths are at most 4096.  LONG: rows beyond that (lb_mlp_gemm_bf16 only), 64-bit
// addresses and a branch around what lies outside.
constexpr long kLongRow = 1l << 23;
static_assert(4 * (63 * kLongRow + 64) <= 0x7fffffff, "a tile's offsets stay within its buffer resource");
template <bool KC, bool VEC, bool LONG, int KT>
__device__ __forceinline__ void tile_load(f32x4 v[KT / 16], const float *__restrict__ p, long ld, int R, int K, int row, int k0) {
    static_assert(KC || KT == 64, "a short tile is contiguous along k");
    constexpr int Q = KT / 4, ROWS = 256 / Q;   // float4 of a row's k, rows of one load of the block
    const int t = threadIdx.x;
    const __amdgpu_buffer_rsrc_t src = operand_rsrc(KC ? p + (long)row * ld + k0 : p + (long)k0 * ld + row);
    const unsigned l = (unsigned)ld;
#pragma unroll
    for (int i = 0; i < KT / 16; ++i) {
        const int r = KC ? t / Q + ROWS * i : (t & 15) * 4;
        const int k = KC ? t % Q * 4 : (t >> 4) * 4 + i;
        const int n = KC ? (row + r < R ? K - k0 - k : 0) : (k0 + k < K ? R - row - r : 0);   // values left
        if (LONG) {
            const float *q = p + (KC ? (long)(row + r) * ld + k0 + k : (long)(k0 + k) * ld + row + r);
            v[i] = f32x4{0.f, 0.f, 0.f, 0.f};
            if (VEC) {
                if (n > 0) v[i] = *reinterpret_cast<const f32x4 *>(q);
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (j < n) v[i][j] = q[j];
            }
            continue;
        }
        const unsigned o = 4u * (KC ? (unsigned)r * l + (unsigned)k : (unsigned)k * l + (unsigned)r);
        if (VEC) {
            v[i] = load4(src, n > 0 ? o : kOut);
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) v[i][j] = load1(src, j < n ? o + 4u * j : kOut);
        }
    }
}
template <bool KC, int KT> __device__ __forceinline__ void tile_store(short (*S)[lds_row(KT)], const f32x4 v[KT / 16]) {
    constexpr int Q = KT / 4, ROWS = 256 / Q;
    const int t = threadIdx.x;
    if (KC) {
#pragma unroll
        for (int i = 0; i < KT / 16; ++i) *reinterpret_cast<bf16x4 *>(&S[t / Q + ROWS * i][t % Q * 4]) = bf16_rne4(v[i]);
    } else {
#pragma unroll
        for (int j = 0; j < 4; ++j)
            *reinterpret_cast<bf16x4 *>(&S[(t & 15) * 4 + j][(t >> 4) * 4]) =
                bf16_rne4(f32x4{v[0][j], v[1][j], v[2][j], v[3][j]});
    }
}

template <int KT> struct Stage {   // the two LDS buffers of both operands' tiles
    short a[2][TM][lds_row(KT)], b[2][TN][lds_row(KT)];
};

// acc = this wave's 32 x 32 part of the 64 x 64 tile at (m0, n0) of sum_k A(m, k) B(k, n), operands
// rounded to BF16 while staged through LDS, FP32 accumulation in steps of 16 in the order of k.
// AK / BK: A / B is contiguous along k (leading dimension lda / ldb between rows m / columns n), else
// along m / n (leading dimension between k).
// Block: 256 threads = 4 waves, each with 2 x 2 MFMA tiles of 16 x 16.
// These products are small (K of a few hundred, some tens of blocks), so a block's time is its chain
// of dependent loads, not arithmetic or bandwidth: a trip takes 64 of k with eight 16-byte loads per
// thread, issued before the previous trip's products, and one barrier (two LDS buffers).  Against a
// trip of 16 of k with scalar loads and two barriers, same results bit for bit: the four products of
// a 512-row forward pass of the 256-wide network 104 -> 31 us, one of 1000 x 1000 x 1000 78-152 -> about
// 30 us.
// KT 16: products of K <= 16 (a network's few inputs), whose tile of 64 would be mostly zeros to convert and
// store, and leave room for four blocks a unit instead of eight: 65 536 x 512 x 5
// 58.5 -> 31.0 us (34.5 in trips of 16 with scalar loads), 262 144 rows of 2-16-16-2 53.0 -> 30.2 (44.0).
template <bool AK, bool BK, bool VEC, bool LONG, int KT>
__device__ __forceinline__ void product_tile(Stage<KT> &S, f32x4 acc[2][2], const float *__restrict__ A, long lda,
                                             const float *__restrict__ B, long ldb, int M, int N, int K, int m0,
                                             int n0) {
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int wm = (wv >> 1) * 32, wn = (wv & 1) * 32;
    for (int i = 0; i < 2; ++i)
        for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    f32x4 va[KT / 16], vb[KT / 16];
    tile_load<AK, VEC, LONG, KT>(va, A, lda, M, K, m0, 0);
    tile_load<BK, VEC, LONG, KT>(vb, B, ldb, N, K, n0, 0);
    for (int k0 = 0, s = 0; k0 < K; k0 += KT, s ^= 1) {
        // buffer s was last read two trips ago, before the previous trip's barrier
        tile_store<AK, KT>(S.a[s], va);
        tile_store<BK, KT>(S.b[s], vb);
        __syncthreads();
        if (k0 + KT < K) {
            tile_load<AK, VEC, LONG, KT>(va, A, lda, M, K, m0, k0 + KT);
            tile_load<BK, VEC, LONG, KT>(vb, B, ldb, N, K, n0, k0 + KT);
        }
        // operand layout of the 16x16x16 BF16 MFMA: lane l holds A(l%16, 4*(l/16)+0..3) and
        // B(4*(l/16)+0..3, l%16)
        const int r = lane & 15, kq = (lane >> 4) * 4;
#pragma unroll
        for (int kk = 0; kk < KT; kk += 16) {
            if (k0 + kk >= K) break;
            bf16x4 a[2], b[2];
            for (int i = 0; i < 2; ++i) a[i] = *reinterpret_cast<const bf16x4 *>(&S.a[s][wm + 16 * i + r][kk + kq]);
            for (int j = 0; j < 2; ++j) b[j] = *reinterpret_cast<const bf16x4 *>(&S.b[s][wn + 16 * j + r][kk + kq]);
            for (int i = 0; i < 2; ++i)
                for (int j = 0; j < 2; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a[i], b[j], acc[i][j], 0, 0, 0);
        }
    }
}

// D(m, n) = epilogue(product).  Epilogues: + bias[n]; tanh(+ bias); times (1 - aux(m, n)^2) with aux
// row-major M x N (the tanh derivative from stored activations).
template <int EPI, bool AK, bool BK, bool VEC, bool LONG = false, int KT = TK>
__global__ __launch_bounds__(256) void k_gemm(const float *__restrict__ A, long lda, const float *__restrict__ B, long ldb,
                                              float *__restrict__ D, int M, int N, int K,
                                              const float *__restrict__ bias, const float *__restrict__ aux) {
    __shared__ __align__(16) Stage<KT> S;
    const int m0 = blockIdx.y * TM, n0 = blockIdx.x * TN;
    f32x4 acc[2][2];
    product_tile<AK, BK, VEC, LONG, KT>(S, acc, A, lda, B, ldb, M, N, K, m0, n0);
    // result layout: lane l holds D(4*(l/16)+q, l%16), q = 0..3
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int c = n0 + (wv & 1) * 32 + (lane & 15), rq = m0 + (wv >> 1) * 32 + (lane >> 4) * 4;
    for (int i = 0; i < 2; ++i)
        for (int j = 0; j < 2; ++j) {
            const int n = c + 16 * j;
            if (n >= N) continue;
            for (int q = 0; q < 4; ++q) {
                const int m = rq + 16 * i + q;
                if (m >= M) continue;
                float v = acc[i][j][q];
                if (EPI == EPI_BIAS || EPI == EPI_BIAS_TANH) v += bias[n];
                if (EPI == EPI_BIAS_TANH) v = tanhf(v);
                if (EPI == EPI_TANH_GRAD) {
                    const float a = aux[(long)m * N + n];
                    v *= 1.0f - a * a;
                }
                D[(long)m * N + n] = v;
            }
        }
}

// ---- weight gradients -----------------------------------------------------------------------
// One layer's share of k_weights: dW = dZ^T A over the batch and db = column sums of dZ.
struct LayerGrad {
    const float *dZ, *A;   // batch x N, batch x K
    long oW;               // of W and then b in the parameter-shaped arrays
    int N, K, vec;
    int tile0, tn;         // first block, and blocks along K
};
struct Grads {
    LayerGrad l[8];
    int n, blocks, bias;   // layers; blocks of all their tiles, and of all their biases (64 columns each)
};
struct Adam {
    float *p, *m1, *m2;
    float lr, b1, b2, eps, c1, c2;
};

__device__ __forceinline__ void adam_update(const Adam &o, float gi, float &p, float &m1, float &m2) {
    const float a = fmaf(1.0f - o.b1, gi, o.b1 * m1);   // written out: the same bits wherever it is inlined
    const float b = fmaf(gi, (1.0f - o.b2) * gi, o.b2 * m2);
    m1 = a;
    m2 = b;
    p -= o.lr * (a / o.c1) / (sqrtf(b / o.c2) + o.eps);
}

// Every layer's weight and bias gradients in one launch, a 32 x 32 tile of one layer per block, and
// with STEP the Adam update of the parameters on the spot (the gradients then need no memory); else
// they go to G.  Half the threads load 4 x 4 blocks of dZ, the other half of A, 64 rows of the batch
// a trip, transposed in registers; each of the four waves multiplies 16 x 16 in the order of the
// rows.  Further blocks take the mean of the rows' losses and the biases: 64 columns of dZ, every fourth
// row by one wave in order, 16 loads in flight, beside the tiles (the order of k_colsum: Adam's first steps
// turn the last bit of a sum that cancels into a step of either sign).
// Bounded by the chain of loads over the batch and the fetch of its code: hence one small tile a wave
// (a 64 x 64 tile's 16 values a lane cost 15 KB of unrolled update), and more blocks than units.
// A training step of 256 rows of the 256-wide network: 390 us in 19 launches -> 39 us in three
// (k_forward 16.2, k_backward 14.5, this 8.2).
constexpr int WT = 32;
template <bool STEP>
__global__ __launch_bounds__(256) void k_weights(Grads gr, int batch, float *__restrict__ G, Adam adam,
                                                 const float *__restrict__ rows, float *__restrict__ loss) {
    __shared__ __align__(16) short S[2][2][WT][LDK];   // [buffer][dZ, A]
    __shared__ float part[256];
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    if ((int)blockIdx.x > gr.blocks) {
        int q = 0, t = (int)blockIdx.x - gr.blocks - 1;
#pragma unroll 1
        for (; t >= (gr.l[q].N + 63) / 64; ++q) t -= (gr.l[q].N + 63) / 64;
        const LayerGrad &l = gr.l[q];
        const int N = l.N, n = t * 64 + lane;
        float s = 0.f;
#pragma unroll 1
        for (int k = wv; k < batch; k += 64) {
            const __amdgpu_buffer_rsrc_t b = operand_rsrc(l.dZ + (long)k * N);
            float v[16];
#pragma unroll
            for (int i = 0; i < 16; ++i) v[i] = load1(b, n < N && k + 4 * i < batch ? 4u * (unsigned)(4 * i * N + n) : kOut);
#pragma unroll
            for (int i = 0; i < 16; ++i) s += v[i];
        }
        part[tid] = s;
        __syncthreads();
        if (wv != 0 || n >= N) return;
        const float g = (part[lane] + part[64 + lane]) + (part[128 + lane] + part[192 + lane]);
        const long at = l.oW + (long)N * l.K + n;
        if (STEP)
            adam_update(adam, g, adam.p[at], adam.m1[at], adam.m2[at]);
        else
            G[at] = g;
        return;
    }
    if ((int)blockIdx.x == gr.blocks) {
        float s = 0.f;
        for (int i = tid; i < batch; i += 256) s += rows[i];
        part[tid] = s;
        __syncthreads();
#pragma unroll 1
        for (int w = 128; w > 0; w >>= 1) {
            if (tid < w) part[tid] += part[tid + w];
            __syncthreads();
        }
        if (tid == 0) *loss = part[0] / (float)batch;
        return;
    }
    int q = 0;
#pragma unroll 1
    while (q + 1 < gr.n && (int)blockIdx.x >= gr.l[q + 1].tile0) ++q;
    const LayerGrad &l = gr.l[q];
    const int t = blockIdx.x - l.tile0, N = l.N, K = l.K, m0 = (t / l.tn) * WT, n0 = (t % l.tn) * WT;

    // this wave's operand: dZ (columns from m0) or A (columns from n0)
    const int half = wv >> 1, u = tid & 127, c4 = (u & 7) * 4, k4 = (u >> 3) * 4;
    const int ld = half ? K : N, left = ld - (half ? n0 : m0) - c4;
    const float *src = (half ? l.A + n0 : l.dZ + m0);
    const int wm = (wv >> 1) * 16, wn = (wv & 1) * 16, r = lane & 15, g4 = (lane >> 4) * 4;
    f32x4 acc{0.f, 0.f, 0.f, 0.f};
    auto products = [&](auto vec) {
        f32x4 v[4];
        auto load = [&](int k0) {
            const __amdgpu_buffer_rsrc_t b = operand_rsrc(src + (long)k0 * ld);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const unsigned o = 4u * ((unsigned)(k4 + i) * (unsigned)ld + (unsigned)c4);
                const int n = k0 + k4 + i < batch ? left : 0;
                if (vec) {
                    v[i] = load4(b, n > 0 ? o : kOut);
                } else {
#pragma unroll
                    for (int j = 0; j < 4; ++j) v[i][j] = load1(b, j < n ? o + 4u * j : kOut);
                }
            }
        };
        load(0);
#pragma unroll 1
        for (int k0 = 0, s = 0; k0 < batch; k0 += TK, s ^= 1) {
            // buffer s was last read two trips ago, before the previous trip's barrier
#pragma unroll
            for (int j = 0; j < 4; ++j)
                *reinterpret_cast<bf16x4 *>(&S[s][half][c4 + j][k4]) = bf16_rne4(f32x4{v[0][j], v[1][j], v[2][j], v[3][j]});
            __syncthreads();
            if (k0 + TK < batch) load(k0 + TK);
#pragma unroll
            for (int kk = 0; kk < TK; kk += 16) {
                if (k0 + kk >= batch) break;
                const bf16x4 a = *reinterpret_cast<const bf16x4 *>(&S[s][0][wm + r][kk + g4]);
                const bf16x4 b = *reinterpret_cast<const bf16x4 *>(&S[s][1][wn + r][kk + g4]);
                acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, acc, 0, 0, 0);
            }
        }
    };
    if (l.vec)
        products(std::true_type{});
    else
        products(std::false_type{});
    bool in[4];
    long at[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int m = m0 + wm + g4 + i, n = n0 + wn + r;
        in[i] = m < N && n < K;
        at[i] = l.oW + (long)m * K + n;
    }
    if (!STEP) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (in[i]) G[at[i]] = acc[i];
        return;
    }
    float p[4], m1[4], m2[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const long o = in[i] ? at[i] : 0;
        p[i] = adam.p[o];
        m1[i] = adam.m1[o];
        m2[i] = adam.m2[o];
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        adam_update(adam, acc[i], p[i], m1[i], m2[i]);
        if (in[i]) {
            adam.p[at[i]] = p[i];
            adam.m1[at[i]] = m1[i];
            adam.m2[at[i]] = m2[i];
        }
    }
}

// ---- narrow networks: the whole pass in one launch --------------------------------------------
// Networks whose layers are all at most kNarrow wide keep a block of rows' activations in LDS from
// the first layer to the last.
constexpr int kNarrow = 512;

// LDS row stride in BF16 values for rows of n: 4 words more than a multiple of 64, so that the 16 rows
// of an operand read spread over all banks (a training step of 256 rows 43.0 us; with 2 words 43.3, 8 words 44.4)
constexpr __host__ __device__ int row_stride(int n) { return ((n + 127) & ~127) + 8; }

constexpr int kWaves = 16;      // waves of a narrow-network block
constexpr int kPanel = 128;     // k of the weights that a wave stages at a time

// Between a wave's stores to its own panel and the reads of it by other lanes, and between those and the
// next panel's stores.  A wave's LDS accesses are performed in the order of the code, so nothing is
// waited for; what the fence holds is the compiler, to which the lanes are threads of their own.
__device__ __forceinline__ void order_wave_lds() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
}

struct Net {
    int L;
    int w[9];
    int oW[8];      // offset of W_l in the parameters (b_l follows it)
    int stride;     // LDS row stride of the activations in BF16 values (row_stride of the widest layer)
};

// Y = network(X) for 16 * RT rows per block.  Each of the 16 waves owns every 16th column tile of a
// layer and stages that tile's weights itself: 16 rows x 128 of k at a time, loaded with 512
// contiguous bytes per row and put into its own part of LDS as BF16 (the operand layout of the
// product, 16 rows side by side in consecutive lanes, loaded directly costs four times the cache
// lookups).  The next panel's loads (also across layers: weights wait for no activation) are in flight
// during this one's products, and no barrier is needed but one a layer, for the activations, which
// are handed on through two LDS buffers.  The first layer, whose few inputs need no 16-byte rows, takes
// single loads.  The products, their order and the epilogues are those of k_gemm, so the results are
// the same bits.
// What bounds it: at a few hundred rows a chain of dependent steps (one round of loads per panel, some
// eight cycles for each instruction of a wave; deeper unrolled forms were slower, 16-27 us for 512 rows
// against 13), at tens of thousands the vector instructions, most of them the tanh (about 30 a value: 50
// of the 94 us for 65 536 rows, the products 16).
// 512 rows of 5-256-256-256-64: 31 -> 12.9 us against a launch per layer; 65 536 rows 172 -> 94 us.
// KEEP: every hidden layer's activations are also stored, in FP32, for the backward pass.
struct Kept {
    float *act[8];
};
template <int RT, bool KEEP>
__global__ __launch_bounds__(64 * kWaves) void k_forward(Net net, const float *__restrict__ P, const float *__restrict__ X,
                                                         int B, float *__restrict__ Y, Kept kept) {
    constexpr int LD = row_stride(kPanel), NL = kPanel / 16;   // loads per lane and panel
    extern __shared__ __align__(16) short sAct[];   // [2][16 RT][stride], then [kWaves][16][LD]
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 15, g4 = (lane >> 4) * 4;
    const int m0 = blockIdx.x * (16 * RT), L = net.L, S = net.stride;
    short *const sW = sAct + 2 * (16 * RT) * S + wave * (16 * LD);

    // the panels in the order this wave takes them (l == L: none left)
    struct Panel {
        int l, nt, kc, K, N;
        const float *W;
    };
    auto first = [&](int l) {
        while (l < L && 16 * wave >= net.w[l + 1]) ++l;
        return l < L ? Panel{l, wave, 0, net.w[l], net.w[l + 1], P + net.oW[l]} : Panel{L, 0, 0, 0, 0, P};
    };
    auto after = [&](Panel p) {
        if (p.kc + kPanel < p.K)
            p.kc += kPanel;
        else if (16 * (p.nt + kWaves) < p.N)
            p.nt += kWaves, p.kc = 0;
        else
            p = first(p.l + 1);
        return p;
    };
    // a panel of a layer after the first, zero outside it: a wave's load i covers whole rows of the
    // panel; and the bias of the panel's tile
    struct Weights {
        float bias;
        f32x4 w[NL];
    };
    const int row = lane / (kPanel / 4), quad = (lane % (kPanel / 4)) * 4;
    auto issue = [&](const Panel &p) {
        Weights b;
        const __amdgpu_buffer_rsrc_t src = operand_rsrc(p.W + (long)p.nt * 16 * p.K + p.kc);
        const int rows = p.kc + quad < p.K ? p.N - 16 * p.nt : 0;
        b.bias = load1(operand_rsrc(p.W + (long)p.N * p.K), 16 * p.nt + r < p.N ? 4u * (unsigned)(16 * p.nt + r) : kOut);
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            const int n = (256 / kPanel) * i + row;
            b.w[i] = load4(src, n < rows ? 4u * (unsigned)(n * p.K + quad) : kOut);
        }
        return b;
    };
    Panel now = first(0);             // the panel to multiply next
    Weights b = issue(first(1));      // in flight: that panel, or the first one after layer 0

    {   // the rows of X as BF16, zero beyond the batch and up to the next multiple of 16 columns
        const int K = net.w[0], KP = (K + 15) & ~15;
#pragma unroll 1
        for (int m = wave * 4 + (lane >> 4); m < 16 * RT; m += 4 * kWaves)
#pragma unroll 1
            for (int k = r; k < KP; k += 16) {
                const float v = m0 + m < B && k < K ? X[(long)(m0 + m) * K + k] : 0.f;
                sAct[m * S + k] = bf16_rne4(f32x4{v, v, v, v})[0];
            }
    }
    f32x4 acc[RT];
    int layer = -1;   // every wave has begun this layer
    while (now.l < L) {
        const Panel p = now;
        now = after(p);
#pragma unroll 1
        for (; layer < p.l; ++layer) __syncthreads();
        const short *in = sAct + (p.l & 1) * (16 * RT) * S + p.kc;
        const int n = p.nt * 16 + r, steps = min(kPanel, p.K - p.kc);
        float bias;
        if (p.l == 0) {   // few inputs: single loads
            const __amdgpu_buffer_rsrc_t src = operand_rsrc(p.W);
            bias = load1(src, n < p.N ? 4u * (unsigned)(p.N * p.K + n) : kOut);
#pragma unroll 1
            for (int j = 0; j < steps; j += 16) {
                f32x4 w;
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    w[q] = load1(src, n < p.N && p.kc + j + g4 + q < p.K ? 4u * (unsigned)(n * p.K + p.kc + j + g4 + q) : kOut);
                *reinterpret_cast<bf16x4 *>(sW + r * LD + j + g4) = bf16_rne4(w);
            }
        } else {
#pragma unroll
            for (int i = 0; i < NL; ++i)
                *reinterpret_cast<bf16x4 *>(sW + ((256 / kPanel) * i + row) * LD + quad) = bf16_rne4(b.w[i]);
            bias = b.bias;
            b = issue(now);
        }
        order_wave_lds();
        if (p.kc == 0)
#pragma unroll
            for (int t = 0; t < RT; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 2
        for (int j = 0; j < steps; j += 16) {
            const bf16x4 w = *reinterpret_cast<const bf16x4 *>(sW + r * LD + j + g4);
#pragma unroll
            for (int t = 0; t < RT; ++t) {
                const bf16x4 a = *reinterpret_cast<const bf16x4 *>(in + (16 * t + r) * S + j + g4);
                acc[t] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, w, acc[t], 0, 0, 0);
            }
        }
        order_wave_lds();
        if (p.kc + kPanel < p.K) continue;
        if (p.l + 1 == L) {
            if (n < p.N)
#pragma unroll
                for (int t = 0; t < RT; ++t)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int m = m0 + 16 * t + g4 + q;
                        if (m < B) Y[(long)m * p.N + n] = acc[t][q] + bias;
                    }
            continue;
        }
        short *out = sAct + ((p.l + 1) & 1) * (16 * RT) * S;
#pragma unroll
        for (int t = 0; t < RT; ++t) {
            f32x4 v;
#pragma unroll
            for (int q = 0; q < 4; ++q) v[q] = n < p.N ? tanhf(acc[t][q] + bias) : 0.f;
            const bf16x4 o = bf16_rne4(v);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int m = 16 * t + g4 + q;
                out[m * S + n] = o[q];
                if (KEEP && n < p.N && m0 + m < B) kept.act[p.l][(long)(m0 + m) * p.N + n] = v[q];
            }
        }
    }
#pragma unroll 1
    for (; layer < L - 1; ++layer) __syncthreads();   // every wave meets every layer's barrier
}

// zero n bytes (n a multiple of 4, 4-byte aligned): a kernel rather than a memset node, so a caller
// may capture the calls that clear state into a graph
__global__ __launch_bounds__(256) void k_zero(unsigned *__restrict__ p, size_t n_words) {
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n_words; i += (size_t)gridDim.x * 256) p[i] = 0u;
}

static hipError_t zero_async(void *p, size_t bytes, hipStream_t st) {
    const size_t words = bytes / 4;
    if (words == 0) return hipSuccess;
    const unsigned blocks = (unsigned)std::min<size_t>((words + 255) / 256, 4096);
    k_zero<<<blocks, 256, 0, st>>>(static_cast<unsigned *>(p), words);
    return hipGetLastError();
}

// one wave, row i: returns r_i = |yhat_i - y_i|^2 / |y_i|^2 and hands put(n, dYhat) the gradient
// dYhat = 2 (yhat - y) / (|y|^2 batch)
template <typename Put>
__device__ __forceinline__ float rel_loss_row(const float *Yh, const float *__restrict__ Y, int i, int B, int N, Put put) {
    const int l = threadIdx.x & 63;
    float e2 = 0.f, y2 = 0.f;
    for (int n = l; n < N; n += 64) {
        float d = Yh[(long)i * N + n] - Y[(long)i * N + n];
        float y = Y[(long)i * N + n];
        e2 += d * d;
        y2 += y * y;
    }
    for (int o = 32; o > 0; o >>= 1) {
        e2 += __shfl_xor(e2, o);
        y2 += __shfl_xor(y2, o);
    }
    const float inv = 1.0f / fmaxf(y2, 1e-30f);
    for (int n = l; n < N; n += 64) put(n, 2.0f * (Yh[(long)i * N + n] - Y[(long)i * N + n]) * inv / (float)B);
    return e2 * inv;
}

// dY may be Yh itself
__global__ __launch_bounds__(64) void k_rel_loss(const float *Yh, const float *__restrict__ Y, int B, int N, float *dY,
                                                 float *__restrict__ row_loss) {
    const int i = blockIdx.x;
    const float r = rel_loss_row(Yh, Y, i, B, N, [&](int n, float v) { dY[(long)i * N + n] = v; });
    if (threadIdx.x == 0) row_loss[i] = r;
}

// The gradients of every layer's pre-activations for 16 rows per block, from the stored activations:
// dZ of the last layer from the loss, then dZ_{l-1} = (dZ_l W_l) (1 - A_{l-1}^2) down to the first,
// each stored in FP32 for k_weights and handed on in LDS as the next product's BF16 operand.  Built
// like k_forward (waves, panels, prefetch, barriers); W_l is read along its rows (64 bytes of 16
// columns per k) and transposed 4 x 4 in registers.
struct Chain {
    const float *act[8];   // A_l (batch x w[l+1]), l < L - 1
    float *dz[8];          // dZ_l (batch x w[l+1]); dz[L-1] holds the network's output on entry
};
__global__ __launch_bounds__(64 * kWaves) void k_backward(Net net, Chain ch, const float *__restrict__ P,
                                                          const float *__restrict__ Y, int B, float *__restrict__ rows) {
    constexpr int LD = row_stride(kPanel);
    extern __shared__ __align__(16) short sAct[];   // [2][16][stride], then [kWaves][16][LD]
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 15, g4 = (lane >> 4) * 4;
    const int m0 = blockIdx.x * 16, L = net.L, S = net.stride;
    short *const sW = sAct + 2 * 16 * S + wave * (16 * LD);

    // the panels in the order this wave takes them: layer l from L-1 down to 1, column tile nt of its
    // K inputs, 128 of its N outputs (l == 0: none left)
    struct Panel {
        int l, nt, kc, K, N;
        const float *W;
    };
    auto first = [&](int l) {
        while (l > 0 && 16 * wave >= net.w[l]) --l;
        return l > 0 ? Panel{l, wave, 0, net.w[l], net.w[l + 1], P + net.oW[l]} : Panel{0, 0, 0, 0, 0, P};
    };
    auto after = [&](Panel p) {
        if (p.kc + kPanel < p.N)
            p.kc += kPanel;
        else if (16 * (p.nt + kWaves) < p.K)
            p.nt += kWaves, p.kc = 0;
        else
            p = first(p.l - 1);
        return p;
    };
    struct Weights {
        f32x4 w[8];   // two 4 x 4 blocks: w[4 h + i] row kc + 64 h + 4 (lane / 4) + i, columns 4 (lane % 4) ..
    };
    const int k4 = (lane >> 2) * 4, c4 = (lane & 3) * 4;
    auto issue = [&](const Panel &p) {
        Weights b;
        const __amdgpu_buffer_rsrc_t src = operand_rsrc(p.W + (long)p.kc * p.K + 16 * p.nt);
        const int rowsLeft = 16 * p.nt + c4 < p.K ? p.N - p.kc : 0;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int k = 64 * (i >> 2) + k4 + (i & 3);
            b.w[i] = load4(src, k < rowsLeft ? 4u * (unsigned)(k * p.K + c4) : kOut);
        }
        return b;
    };
    Panel now = first(L - 1);
    Weights b = issue(now);

    {   // one wave a row: the loss and dZ of the last layer, zero beyond the batch and the layer
        const int N = net.w[L], NP = (N + 15) & ~15, i = m0 + wave;
        short *o = sAct + ((L - 1) & 1) * 16 * S + wave * S;
#pragma unroll 1
        for (int n = lane; n < NP; n += 64) o[n] = 0;
        if (i < B) {
            float *dz = ch.dz[L - 1];
            const float v = rel_loss_row(dz, Y, i, B, N, [&](int n, float g) {
                dz[(long)i * N + n] = g;
                o[n] = bf16_rne4(f32x4{g, g, g, g})[0];
            });
            if (lane == 0) rows[i] = v;
        }
    }
    f32x4 acc;
    int layer = L;   // every wave has begun this layer
    while (now.l > 0) {
        const Panel p = now;
        now = after(p);
#pragma unroll 1
        for (; layer > p.l; --layer) __syncthreads();
        const short *in = sAct + (p.l & 1) * 16 * S + p.kc;
        const int n = 16 * p.nt + r, steps = min(kPanel, p.N - p.kc);
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int j = 0; j < 4; ++j)
                *reinterpret_cast<bf16x4 *>(sW + (c4 + j) * LD + 64 * h + k4) =
                    bf16_rne4(f32x4{b.w[4 * h][j], b.w[4 * h + 1][j], b.w[4 * h + 2][j], b.w[4 * h + 3][j]});
        float a[4];
        {
            const __amdgpu_buffer_rsrc_t src = operand_rsrc(ch.act[p.l - 1] + (long)m0 * p.K);
#pragma unroll
            for (int q = 0; q < 4; ++q)
                a[q] = load1(src, n < p.K && m0 + g4 + q < B ? 4u * (unsigned)((g4 + q) * p.K + n) : kOut);
        }
        b = issue(now);
        order_wave_lds();
        if (p.kc == 0) acc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 2
        for (int j = 0; j < steps; j += 16) {
            const bf16x4 w = *reinterpret_cast<const bf16x4 *>(sW + r * LD + j + g4);
            const bf16x4 d = *reinterpret_cast<const bf16x4 *>(in + r * S + j + g4);
            acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(d, w, acc, 0, 0, 0);
        }
        order_wave_lds();
        if (p.kc + kPanel < p.N) continue;
        f32x4 v;
        float *dz = ch.dz[p.l - 1];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            v[q] = acc[q] * (1.0f - a[q] * a[q]);
            if (n >= p.K) v[q] = 0.f;
            if (n < p.K && m0 + g4 + q < B) dz[(long)(m0 + g4 + q) * p.K + n] = v[q];
        }
        short *out = sAct + ((p.l - 1) & 1) * 16 * S;
        const bf16x4 o = bf16_rne4(v);
#pragma unroll
        for (int q = 0; q < 4; ++q) out[(g4 + q) * S + n] = o[q];
    }
#pragma unroll 1
    for (; layer > 1; --layer) __syncthreads();   // every wave meets every layer's barrier
}

__global__ __launch_bounds__(256) void k_adam(Adam o, const float *__restrict__ g, long n) {
    const long i = (long)blockIdx.x * 256 + threadIdx.x;
    if (i < n) adam_update(o, g[i], o.p[i], o.m1[i], o.m2[i]);
}

int fail(int code, const char *fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    lbk::set_last_error(buf);
    return code;
}
#define HIPCHK(expr)                                                                            \
    do {                                                                                        \
        hipError_t e_ = (expr);                                                                 \
        if (e_ != hipSuccess) return fail(LB_EDEVICE, "%s: %s", #expr, hipGetErrorString(e_)); \
    } while (0)

struct Layout {
    int L = 0;
    std::vector<int> w;
    std::vector<size_t> oW, oB;   // offsets (floats) of W_l and b_l in the parameter array
    size_t n_params = 0, acts = 0;
    size_t bytes = 0;       // of the arena
    size_t least = 0;       // what an arena needs to be usable at all: two gradient buffers instead of
                            // one per hidden layer, and so a launch per layer in the backward pass
    size_t oP = 0, oG = 0, oM1 = 0, oM2 = 0, oAct = 0, oGrad = 0, oRow = 0, oLoss = 0;
};

int layout(const lb_mlp_config *c, Layout &lo) {
    if (!c) return fail(LB_EINVAL, "config is NULL");
    if (c->n_layers < 1 || c->n_layers > 8) return fail(LB_EINVAL, "n_layers must be 1..8");
    if (c->max_batch < 1 || c->max_batch > (1 << 20)) return fail(LB_EINVAL, "max_batch out of range");
    lo.L = c->n_layers;
    lo.w.assign(c->widths, c->widths + c->n_layers + 1);
    for (int x : lo.w)
        if (x < 1 || x > 4096) return fail(LB_EINVAL, "layer widths must be 1..4096");
    size_t off = 0, acts = 0;
    for (int l = 0; l < lo.L; ++l) {
        lo.oW.push_back(off);
        off += (size_t)lo.w[l + 1] * lo.w[l];
        lo.oB.push_back(off);
        off += (size_t)lo.w[l + 1];
        acts += (size_t)lo.w[l + 1];
    }
    lo.n_params = off;
    lo.acts = acts;
    auto al = [](size_t b) { return (b + 255) & ~(size_t)255; };
    size_t o = 0;
    lo.oP = o;  o += al(4 * off);
    lo.oG = o;  o += al(4 * off);
    lo.oM1 = o; o += al(4 * off);
    lo.oM2 = o; o += al(4 * off);
    lo.oAct = o; o += al(4 * acts * (size_t)c->max_batch);           // activations of every layer
    size_t wmax = *std::max_element(lo.w.begin(), lo.w.end());
    lo.oRow = o; o += al(4 * (size_t)c->max_batch);
    lo.oLoss = o; o += al(4);
    const size_t hidden = acts - (size_t)lo.w[lo.L];
    lo.oGrad = o;                                                    // gradient buffers
    lo.least = o + al(4 * 2 * wmax * (size_t)c->max_batch) + 256;
    lo.bytes = o + al(4 * std::max(2 * wmax, hidden) * (size_t)c->max_batch) + 256;
    return LB_OK;
}

}  // namespace

struct lb_mlp {
    lb_mlp_config cfg;
    Layout lo;
    char *base = nullptr;
    hipStream_t stream = nullptr;
    bool own_stream = false;
    long step = 0;
    bool room = true;   // a gradient buffer per layer
    // waits for the stream and releases it if the library created it (also when lb_mlp_create
    // fails part way); the arena belongs to the caller
    ~lb_mlp() {
        if (stream) (void)hipStreamSynchronize(stream);
        if (own_stream && stream) (void)hipStreamDestroy(stream);
    }
    float *P() { return reinterpret_cast<float *>(base + lo.oP); }
    float *G() { return reinterpret_cast<float *>(base + lo.oG); }
    float *M1() { return reinterpret_cast<float *>(base + lo.oM1); }
    float *M2() { return reinterpret_cast<float *>(base + lo.oM2); }
    float *act(int l) {   // output of layer l (batch x w[l+1]) at max_batch stride
        size_t off = 0;
        for (int i = 0; i < l; ++i) off += (size_t)lo.w[i + 1];
        return reinterpret_cast<float *>(base + lo.oAct) + off * (size_t)cfg.max_batch;
    }
    float *grad(int i) {
        size_t wmax = *std::max_element(lo.w.begin(), lo.w.end());
        return reinterpret_cast<float *>(base + lo.oGrad) + (size_t)i * wmax * cfg.max_batch;
    }
    // gradient of layer l's pre-activations, with room for one per layer: the last one's takes the place
    // of the network's output
    float *dz(int l) {
        if (l + 1 == lo.L) return act(l);
        return reinterpret_cast<float *>(base + lo.oGrad) + (act(l) - act(0));
    }
    float *rows() { return reinterpret_cast<float *>(base + lo.oRow); }
    float *loss() { return reinterpret_cast<float *>(base + lo.oLoss); }
};

namespace {

template <int EPI, bool AK, bool BK>
hipError_t gemm(const float *A, long lda, const float *B, long ldb, float *D, int M, int N, int K, const float *bias,
                const float *aux, hipStream_t st) {
    // 16-byte loads where every row (or k) of the operand starts on 16 bytes
    auto vec = [](const float *p, long ld) { return ((uintptr_t)p & 15) == 0 && (ld & 3) == 0; };
    dim3 grid((N + TN - 1) / TN, (M + TM - 1) / TM);
    if constexpr (EPI == EPI_STORE)
        if (std::max(lda, ldb) > kLongRow) {
            if (vec(A, lda) && vec(B, ldb))
                k_gemm<EPI, AK, BK, true, true><<<grid, 256, 0, st>>>(A, lda, B, ldb, D, M, N, K, bias, aux);
            else
                k_gemm<EPI, AK, BK, false, true><<<grid, 256, 0, st>>>(A, lda, B, ldb, D, M, N, K, bias, aux);
            return hipGetLastError();
        }
    if constexpr (EPI == EPI_BIAS || EPI == EPI_BIAS_TANH)
        if (K <= 16) {
            if (vec(A, lda) && vec(B, ldb))
                k_gemm<EPI, AK, BK, true, false, 16><<<grid, 256, 0, st>>>(A, lda, B, ldb, D, M, N, K, bias, aux);
            else
                k_gemm<EPI, AK, BK, false, false, 16><<<grid, 256, 0, st>>>(A, lda, B, ldb, D, M, N, K, bias, aux);
            return hipGetLastError();
        }
    if (vec(A, lda) && vec(B, ldb))
        k_gemm<EPI, AK, BK, true><<<grid, 256, 0, st>>>(A, lda, B, ldb, D, M, N, K, bias, aux);
    else
        k_gemm<EPI, AK, BK, false><<<grid, 256, 0, st>>>(A, lda, B, ldb, D, M, N, K, bias, aux);
    return hipGetLastError();
}

// Z = in W^T + b over a batch (in: B x K, W: N x K, both row-major), tanh unless it is the last layer
hipError_t layer_forward(bool last, const float *in, const float *W, const float *b, float *out, int B, int N, int K,
                         hipStream_t st) {
    return last ? gemm<EPI_BIAS, true, true>(in, K, W, K, out, B, N, K, b, nullptr, st)
                : gemm<EPI_BIAS_TANH, true, true>(in, K, W, K, out, B, N, K, b, nullptr, st);
}

// The network as the narrow kernels take it; false if it is not one for them: a layer too wide; rows of a
// weight matrix after the first that do not start on 16 bytes; one layer, which is one launch anyway; or a
// first layer, whose weights come in single loads, of more than 32 768 of them.  Forward passes layer by layer and
// in one launch, us: 256 rows of 64-256-256-64 26 and 18, of 128-256-256-64 26.3 and 26.0, of 256-256-256-256 26 and
// 40, of 384-384-384 20 and 75; widths up to the limit of LDS, 1000 rows of 16-384-384-16 26 and 16, of
// 5-512-512-512-64 44 and 31, 65 536 of them 450 and 308 (one row 28 and 29).
bool narrow_net(int L, const int *w, const float *P, Net &net) {
    if (*std::max_element(w, w + L + 1) > kNarrow || L < 2 || w[0] * w[1] > 32768) return false;
    int o = 0;
    net.L = L;
    for (int l = 0; l < L; ++l) {
        if (l > 0 && ((w[l] & 3) != 0 || ((uintptr_t)(P + o) & 15) != 0)) return false;
        net.w[l] = w[l];
        net.oW[l] = o;
        o += w[l + 1] * w[l] + w[l + 1];
    }
    net.w[L] = w[L];
    net.stride = row_stride(*std::max_element(w, w + L + 1));
    return true;
}

bool overlap(const void *a, size_t na, const void *b, size_t nb) {
    const uintptr_t x = (uintptr_t)a, y = (uintptr_t)b;
    return x < y + nb && y < x + na;
}

// Whether a forward pass of B rows goes in one launch.  A net of up to 64 columns leaves most of a block's 16
// waves idle, so over many rows the layers win: 5-16-16-8, 16 384 rows 10.4 us in one launch, 13.0 by layers,
// 24 576 rows 18.2 and 13.8; 5-64-64-8, 32 768 rows 20.1 and 20.7, 49 152 rows 31 and 25.
bool narrow_forward(const Net &net, int B) {
    const int widest = *std::max_element(net.w, net.w + net.L + 1);
    return widest > 64 || B <= std::min(std::max(1024 * widest, 16384), 32768);
}

// Whether gradients of B rows go through k_forward and k_backward, 16 rows a block.  Each block reads every weight, so
// beyond a block or two a unit the layers win, the earlier the wider: a training step of 8192 rows of 5-256-256-256-64
// 211 us, 224 by layers, of 16 384 rows 406 and 401; of 5-512-512-512-64, 2000 rows 112 and 121, 4100 rows 223 and 180.
bool narrow_gradients(const Net &net, int B) {
    return B <= (*std::max_element(net.w, net.w + net.L + 1) <= 256 ? 8192 : 4096);
}

template <int RT> size_t narrow_lds(const Net &net) {
    return (2 * (16 * RT) * (size_t)net.stride + kWaves * 16 * row_stride(kPanel)) * sizeof(short);
}
template <int RT> hipError_t forward_narrow(const Net &net, const float *P, const float *X, int B, float *Y, hipStream_t st) {
    k_forward<RT, false><<<(B + 16 * RT - 1) / (16 * RT), 64 * kWaves, narrow_lds<RT>(net), st>>>(net, P, X, B, Y, Kept{});
    return hipGetLastError();
}

// Y = network(X) in one launch.  Rows per block: 16 while the blocks are at most one per compute
// unit of the whole device, 256 (each block reads every weight, so fewer rows a block only help while units are idle), then 32
// and, where 64 rows' activations fit the 160 KB of LDS, 64, which halve and quarter the weight
// traffic: 4096 rows take 14.5 us with 16 rows a block, 8192 rows 19 with 32 (22 with 64), 65 536 rows
// 94 with 64 (124 with 32).
hipError_t forward_narrow(const Net &net, const float *P, const float *X, int B, float *Y, hipStream_t st) {
    if (B <= 16 * 256) return forward_narrow<1>(net, P, X, B, Y, st);
    if (B <= 32 * 256 || narrow_lds<4>(net) > 160 * 1024) return forward_narrow<2>(net, P, X, B, Y, st);
    return forward_narrow<4>(net, P, X, B, Y, st);
}

// ---- forward pass without allocation ------------------------------------------------------
// The hidden activations of lb_mlp_forward_noalloc live in this file-scope device array, two
// ping-pong halves of kScratchFloats / 2 floats.  Host code never passes the array's name to a
// kernel (on the host it is only a stand-in for the symbol): each device's copy is looked up once
// with hipGetSymbolAddress and its address kept per device.
constexpr size_t kScratchFloats = size_t(1) << 20;   // 4 MiB per GPU, held until the process ends
constexpr int kMaxDevices = 64;
__device__ __align__(256) float scratch[kScratchFloats];
std::mutex g_scratch_mu;
float *g_scratch_ptr[kMaxDevices] = {};

int scratch_on_current_device(float **out) {
    int dev = 0;
    HIPCHK(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) return fail(LB_EINVAL, "device index %d beyond %d", dev, kMaxDevices);
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        HIPCHK(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (!p) return fail(LB_EDEVICE, "no device address for the scratch array");
        g_scratch_ptr[dev] = static_cast<float *>(p);
    }
    *out = g_scratch_ptr[dev];
    return LB_OK;
}

// forward into the activation buffers, a launch per layer, the last layer into `out`
int forward(lb_mlp *m, const float *X, int B, float *out) {
    const Layout &lo = m->lo;
    const float *in = X;
    for (int l = 0; l < lo.L; ++l) {
        const int K = lo.w[l], N = lo.w[l + 1];
        const float *W = m->P() + lo.oW[l], *b = m->P() + lo.oB[l];
        float *Z = l + 1 == lo.L ? out : m->act(l);
        HIPCHK(layer_forward(l + 1 == lo.L, in, W, b, Z, B, N, K, m->stream));
        in = Z;
    }
    return LB_OK;
}

// one layer's entry of k_weights' work, its blocks after those already there
void add_layer(Grads &g, lb_mlp *m, int l, const float *dZ, const float *A) {
    const int N = m->lo.w[l + 1], K = m->lo.w[l];
    auto vec = [](const float *p, int ld) { return ((uintptr_t)p & 15) == 0 && (ld & 3) == 0; };
    const int tn = (K + WT - 1) / WT;
    g.l[g.n++] = LayerGrad{dZ, A, (long)m->lo.oW[l], N, K, vec(dZ, N) && vec(A, K), g.blocks, tn};
    g.blocks += tn * ((N + WT - 1) / WT);
    g.bias += (N + 63) / 64;
}

// Forward pass, loss and gradients of the mean squared relative error: with `adam` the update of the
// parameters, else the gradients in G().  The mean loss goes to `loss`.
// Narrow networks: three launches (k_forward, k_backward, k_weights).  Others: a launch per layer and
// direction, then k_weights.  An arena with two gradient buffers only: each layer's weight gradients as
// soon as its dZ is there, and the update at the end.
int gradients(lb_mlp *m, const float *X, const float *Y, int B, const Adam *adam, float *loss) {
    const Layout &lo = m->lo;
    const int L = lo.L, NL = lo.w[L];
    Net net;
    Grads g{};
    if (m->room) {
        if (narrow_net(L, lo.w.data(), m->P(), net) && narrow_gradients(net, B)) {
            Kept kept{};
            Chain ch{};
            for (int l = 0; l < L; ++l) {
                kept.act[l] = m->act(l);
                ch.act[l] = m->act(l);
                ch.dz[l] = m->dz(l);
            }
            k_forward<1, true><<<(B + 15) / 16, 64 * kWaves, narrow_lds<1>(net), m->stream>>>(net, m->P(), X, B, m->act(L - 1),
                                                                                            kept);
            HIPCHK(hipGetLastError());
            k_backward<<<(B + 15) / 16, 64 * kWaves, narrow_lds<1>(net), m->stream>>>(net, ch, m->P(), Y, B, m->rows());
            HIPCHK(hipGetLastError());
        } else {
            int rc = forward(m, X, B, m->act(L - 1));
            if (rc) return rc;
            k_rel_loss<<<B, 64, 0, m->stream>>>(m->act(L - 1), Y, B, NL, m->dz(L - 1), m->rows());
            HIPCHK(hipGetLastError());
            for (int l = L - 1; l > 0; --l) {
                // dZ_prev = (dZ W) * (1 - A_prev^2): A(m=row, k=out) = dZ[row*N + out], B(k=out, n=in) = W[out*K + in]
                const int K = lo.w[l], N = lo.w[l + 1];
                HIPCHK((gemm<EPI_TANH_GRAD, true, false>(m->dz(l), N, m->P() + lo.oW[l], K, m->dz(l - 1), B, K, N, nullptr,
                                                         m->act(l - 1), m->stream)));
            }
        }
        for (int l = 0; l < L; ++l) add_layer(g, m, l, m->dz(l), l > 0 ? m->act(l - 1) : X);
        if (adam)
            k_weights<true><<<g.blocks + 1 + g.bias, 256, 0, m->stream>>>(g, B, nullptr, *adam, m->rows(), loss);
        else
            k_weights<false><<<g.blocks + 1 + g.bias, 256, 0, m->stream>>>(g, B, m->G(), Adam{}, m->rows(), loss);
        HIPCHK(hipGetLastError());
        return LB_OK;
    }
    int rc = forward(m, X, B, m->act(L - 1));
    if (rc) return rc;
    float *dA = m->grad(0), *dZ = m->grad(1);
    k_rel_loss<<<B, 64, 0, m->stream>>>(m->act(L - 1), Y, B, NL, dZ, m->rows());
    HIPCHK(hipGetLastError());
    for (int l = L - 1; l >= 0; --l) {
        const int K = lo.w[l], N = lo.w[l + 1];
        const float *Aprev = l > 0 ? m->act(l - 1) : X;
        g = Grads{};
        add_layer(g, m, l, dZ, Aprev);
        k_weights<false><<<g.blocks + 1 + g.bias, 256, 0, m->stream>>>(g, B, m->G(), Adam{}, m->rows(), loss);
        HIPCHK(hipGetLastError());
        if (l > 0) {
            HIPCHK((gemm<EPI_TANH_GRAD, true, false>(dZ, N, m->P() + lo.oW[l], K, dA, B, K, N, nullptr, Aprev, m->stream)));
            std::swap(dA, dZ);
        }
    }
    if (adam) {
        const long n = (long)lo.n_params;
        k_adam<<<(unsigned)((n + 255) / 256), 256, 0, m->stream>>>(*adam, m->G(), n);
        HIPCHK(hipGetLastError());
    }
    return LB_OK;
}

}  // namespace

extern "C" {

int lb_mlp_query_bytes(const lb_mlp_config *cfg, size_t *bytes) {
    if (!bytes) return fail(LB_EINVAL, "bytes is NULL");
    Layout lo;
    int rc = layout(cfg, lo);
    if (rc) return rc;
    *bytes = lo.bytes;
    return LB_OK;
}

int lb_mlp_n_params(const lb_mlp_config *cfg, size_t *n) {
    if (!n) return fail(LB_EINVAL, "n is NULL");
    Layout lo;
    int rc = layout(cfg, lo);
    if (rc) return rc;
    *n = lo.n_params;
    return LB_OK;
}

int lb_mlp_create(const lb_mlp_config *cfg, void *arena, size_t arena_bytes, void *stream, lb_mlp **out) {
    if (!out || !arena) return fail(LB_EINVAL, "NULL argument");
    if ((uintptr_t)arena & 255) return fail(LB_EINVAL, "arena must be 256-byte aligned");
    try {
        std::unique_ptr<lb_mlp> m(new lb_mlp());
        int rc = layout(cfg, m->lo);
        if (rc) return rc;
        if (arena_bytes < m->lo.least) return fail(LB_ENOMEM, "arena too small: %zu < %zu", arena_bytes, m->lo.bytes);
        m->room = arena_bytes >= m->lo.bytes;
        m->cfg = *cfg;
        if (m->cfg.beta1 == 0.f) m->cfg.beta1 = 0.9f;
        if (m->cfg.beta2 == 0.f) m->cfg.beta2 = 0.999f;
        if (m->cfg.eps == 0.f) m->cfg.eps = 1e-8f;
        m->base = static_cast<char *>(arena);
        if (stream) {
            m->stream = static_cast<hipStream_t>(stream);
        } else {
            HIPCHK(hipStreamCreateWithFlags(&m->stream, hipStreamNonBlocking));
            m->own_stream = true;
        }
        HIPCHK(zero_async(m->base, m->lo.oAct, m->stream));
        HIPCHK(hipStreamSynchronize(m->stream));
        *out = m.release();
        return LB_OK;
    } catch (...) {
        return fail(LB_ENOMEM, "host allocation failed");
    }
}

int lb_mlp_set_params(lb_mlp *m, const float *host) {
    if (!m || !host) return fail(LB_EINVAL, "NULL argument");
    HIPCHK(hipMemcpyAsync(m->P(), host, 4 * m->lo.n_params, hipMemcpyHostToDevice, m->stream));
    HIPCHK(zero_async(m->M1(), 4 * m->lo.n_params, m->stream));
    HIPCHK(zero_async(m->M2(), 4 * m->lo.n_params, m->stream));
    HIPCHK(hipStreamSynchronize(m->stream));
    m->step = 0;
    return LB_OK;
}

int lb_mlp_get_params(lb_mlp *m, float *host) {
    if (!m || !host) return fail(LB_EINVAL, "NULL argument");
    HIPCHK(hipMemcpyAsync(host, m->P(), 4 * m->lo.n_params, hipMemcpyDeviceToHost, m->stream));
    HIPCHK(hipStreamSynchronize(m->stream));
    return LB_OK;
}

int lb_mlp_forward(lb_mlp *m, const float *X, int32_t batch, float *Y) {
    if (!m || !X || !Y) return fail(LB_EINVAL, "NULL argument");
    if (batch < 1 || batch > m->cfg.max_batch) return fail(LB_ERANGE, "batch out of range");
    const int NL = m->lo.w[m->lo.L];
    Net net;
    // overlapping X and Y: layer by layer, where X has been read when the last layer is written (a single
    // layer goes through its own buffer)
    const bool apart = !overlap(X, 4 * (size_t)batch * m->lo.w[0], Y, 4 * (size_t)batch * NL);
    if (apart && narrow_net(m->lo.L, m->lo.w.data(), m->P(), net) && narrow_forward(net, batch)) {
        HIPCHK(forward_narrow(net, m->P(), X, batch, Y, m->stream));
        return LB_OK;
    }
    const bool direct = apart || m->lo.L > 1;
    int rc = forward(m, X, batch, direct ? Y : m->act(m->lo.L - 1));
    if (rc || direct) return rc;
    HIPCHK(hipMemcpyAsync(Y, m->act(m->lo.L - 1), 4 * (size_t)batch * NL, hipMemcpyDeviceToDevice, m->stream));
    return LB_OK;
}

int lb_mlp_gradients(lb_mlp *m, const float *X, const float *Y, int32_t batch, float *host_loss, float *host_grads) {
    if (!m || !X || !Y) return fail(LB_EINVAL, "NULL argument");
    if (batch < 1 || batch > m->cfg.max_batch) return fail(LB_ERANGE, "batch out of range");
    int rc = gradients(m, X, Y, batch, nullptr, m->loss());
    if (rc) return rc;
    if (host_loss) HIPCHK(hipMemcpyAsync(host_loss, m->loss(), 4, hipMemcpyDeviceToHost, m->stream));
    if (host_grads) HIPCHK(hipMemcpyAsync(host_grads, m->G(), 4 * m->lo.n_params, hipMemcpyDeviceToHost, m->stream));
    HIPCHK(hipStreamSynchronize(m->stream));
    return LB_OK;
}

int lb_mlp_train_step(lb_mlp *m, const float *X, const float *Y, int32_t batch, float lr, float *device_loss) {
    if (!m || !X || !Y) return fail(LB_EINVAL, "NULL argument");
    if (batch < 1 || batch > m->cfg.max_batch) return fail(LB_ERANGE, "batch out of range");
    const float step = (float)(m->step + 1);
    const Adam adam{m->P(), m->M1(), m->M2(), lr, m->cfg.beta1, m->cfg.beta2, m->cfg.eps,
                    1.0f - std::pow(m->cfg.beta1, step), 1.0f - std::pow(m->cfg.beta2, step)};
    int rc = gradients(m, X, Y, batch, &adam, device_loss ? device_loss : m->loss());
    if (rc) return rc;
    m->step += 1;
    return LB_OK;
}

int lb_mlp_destroy(lb_mlp *m) {
    if (!m) return fail(LB_EINVAL, "NULL argument");
    delete m;
    return LB_OK;
}

int lb_mlp_forward_noalloc(const lb_mlp_config *cfg, const float *params, const float *X, int32_t batch, float *Y,
                           void *hip_stream) {
    if (!cfg || !params || !X || !Y) return fail(LB_EINVAL, "NULL argument");
    const int L = cfg->n_layers;
    if (L < 1 || L > 8) return fail(LB_EINVAL, "n_layers must be 1..8");
    int wmax_hidden = 0;
    for (int l = 0; l <= L; ++l) {
        if (cfg->widths[l] < 1 || cfg->widths[l] > 4096) return fail(LB_EINVAL, "layer widths must be 1..4096");
        if (l > 0 && l < L) wmax_hidden = std::max(wmax_hidden, cfg->widths[l]);
    }
    if (batch < 1) return fail(LB_ERANGE, "batch must be positive");
    if ((size_t)batch * (size_t)wmax_hidden > kScratchFloats / 2)
        return fail(LB_ERANGE, "batch %d x hidden width %d exceeds the scratch limit of %zu values", batch, wmax_hidden,
                    kScratchFloats / 2);
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    Net net;
    size_t n_params = 0;
    for (int l = 0; l < L; ++l) n_params += (size_t)cfg->widths[l + 1] * (cfg->widths[l] + 1);
    const size_t nY = 4 * (size_t)batch * cfg->widths[L];
    if (narrow_net(L, cfg->widths, params, net) && narrow_forward(net, batch) && !overlap(X, 4 * (size_t)batch * cfg->widths[0], Y, nY) &&
        !overlap(params, 4 * n_params, Y, nY)) {
        HIPCHK(forward_narrow(net, params, X, batch, Y, st));
        return LB_OK;
    }
    float *buf = nullptr;
    int rc = scratch_on_current_device(&buf);
    if (rc) return rc;
    const float *in = X;
    size_t off = 0;   // parameter offset of W_l
    for (int l = 0; l < L; ++l) {
        const int K = cfg->widths[l], N = cfg->widths[l + 1];
        const float *W = params + off, *b = params + off + (size_t)N * K;
        off += (size_t)N * K + N;
        float *out = l + 1 < L ? buf + (size_t)(l & 1) * (kScratchFloats / 2) : Y;
        HIPCHK(layer_forward(l + 1 == L, in, W, b, out, batch, N, K, st));
        in = out;
    }
    return LB_OK;
}

int lb_mlp_gemm_bf16(const float *A, const float *B, float *D, int32_t M, int32_t N, int32_t K, void *stream) {
    if (!A || !B || !D) return fail(LB_EINVAL, "NULL argument");
    if (M < 1 || N < 1 || K < 1) return fail(LB_EINVAL, "sizes must be positive");
    HIPCHK((gemm<EPI_STORE, true, false>(A, K, B, N, D, M, N, K, nullptr, nullptr, static_cast<hipStream_t>(stream))));
    return LB_OK;
}

}  // extern "C"
