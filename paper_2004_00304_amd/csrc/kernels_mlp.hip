// kernels_mlp.hip -- the learned closure's network on gfx950 matrix cores.
//
// The dense layers of a small MLP (271 -> 128 -> 128 -> 128 -> 9, GELU) run as
// BF16 x BF16 -> FP32 products on the MFMA units (v_mfma_f32_32x32x16_bf16).
// k_net takes a tile of rows through the whole network in one workgroup; in
// training it goes on through the loss and back to the gradient of the first
// layer's pre-activation, k_dw forms the weight gradients as a contraction
// over the rows, split so that it fills the chip, and k_reduce sums the
// splits and applies Adam: three launches per optimiser step.  k_gemm is the
// plain product on its own.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "common.hpp"
#include "gelu.hpp"
#include "launch.hpp"
#include "mlp.hpp"

namespace lbmpcd {

typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

// BF16 with round-to-nearest-even: gfx950's conversion instruction
// (v_cvt_pk_bf16_f32); NaN stays NaN.
__device__ __forceinline__ uint16_t to_bf16(float x) { return __builtin_bit_cast(uint16_t, (__bf16)x); }

__device__ __forceinline__ f32x16 mfma16(const uint4& a, const uint4& b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0,
                                                   0);
}

constexpr int GT = 64;   // output tile side
constexpr int GK = 32;   // K step
constexpr int GKP = GK + 8;  // LDS row pitch (bf16), breaks bank conflicts

// C[M][N] = A[M][K] B[N][K]^T: one 64x64 output tile per workgroup, each of
// its four waves owning a 32x32 quarter.
__global__ void __launch_bounds__(256) k_gemm(GemmArgs g) {
    __shared__ uint16_t As[GT][GKP];  // [m][k]
    __shared__ uint16_t Bs[GT][GKP];  // [n][k]
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    const long long m0 = (long long)blockIdx.y * GT, n0 = (long long)blockIdx.x * GT;
    f32x16 acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.0f;

    for (long long k0 = 0; k0 < g.K; k0 += GK) {
        for (int e = tid; e < GT * GK; e += 256) {
            const int m = e / GK, k = e % GK;
            const long long gm = m0 + m, gn = n0 + m, gk = k0 + k;
            As[m][k] = (gm < g.M && gk < g.K) ? g.A[gm * g.K + gk] : (uint16_t)0;
            Bs[m][k] = (gn < g.N && gk < g.K) ? g.B[gn * g.K + gk] : (uint16_t)0;
        }
        __syncthreads();
#pragma unroll
        for (int kk = 0; kk < GK; kk += 16) {
            // v_mfma_f32_32x32x16_bf16: lane l holds row (column) l % 32 and
            // the 8 k values 8 (l / 32) .. 8 (l / 32) + 7 of the step
            s16x8 a, b;
            const int ar = wm * 32 + (lane & 31), br = wn * 32 + (lane & 31);
            const int kc = kk + 8 * (lane >> 5);
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                a[j] = (short)As[ar][kc + j];
                b[j] = (short)Bs[br][kc + j];
            }
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b),
                                                          acc, 0, 0, 0);
        }
        __syncthreads();
    }

    // lane holds column (lane & 31) of its quarter, rows
    // 8 (r / 4) + 4 (lane / 32) + r % 4 for r = 0..15
    const long long col = n0 + wn * 32 + (lane & 31);
    if (col >= g.N) return;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const long long row = m0 + wm * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
        if (row < g.M) g.C[row * g.N + col] = acc[r];
    }
}

hipError_t launch_gemm(const GemmArgs& g, hipStream_t s) {
    if (g.M <= 0 || g.N <= 0) return hipSuccess;
    dim3 grid((unsigned)((g.N + GT - 1) / GT), (unsigned)((g.M + GT - 1) / GT));
    hipLaunchKernelGGL(k_gemm, grid, dim3(256), 0, s, g);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// weights in fragment order
// ---------------------------------------------------------------------------
static inline unsigned nblk(long long n, int t = 256) { return (unsigned)((n + t - 1) / t); }

// Place of element (k, n) of a B operand of ncb 32-column blocks in fragment
// order: lane t of a wave holds column t % 32 and k values 8 (t / 32) + j.
__device__ __forceinline__ long long frag_pos(int ncb, int k, int n) {
    return ((((long long)(k >> 4) * ncb + (n >> 5)) * 64 + (n & 31) + 32 * ((k >> 3) & 1)) << 3) + (k & 7);
}

// Writes parameter i's BF16 value to its places in the fragment arrays (none
// for a bias).
__device__ __forceinline__ void frag_store(uint16_t* Pf, long long i, uint16_t v) {
    if (i < OFF_B1) {
        const int o = (int)(i / NFP), c = (int)(i % NFP);
        Pf[FRAG_L1 + frag_pos(4, c, o)] = v;
    } else if (i >= OFF_W2 && i < OFF_B2) {
        const int o = (int)((i - OFF_W2) / NH), c = (int)((i - OFF_W2) % NH);
        Pf[FRAG_L2 + frag_pos(4, c, o)] = v;
        Pf[TFRAG_L2 + frag_pos(4, o, c)] = v;
    } else if (i >= OFF_W3 && i < OFF_B3) {
        const int o = (int)((i - OFF_W3) / NH), c = (int)((i - OFF_W3) % NH);
        Pf[FRAG_L3 + frag_pos(4, c, o)] = v;
        Pf[TFRAG_L3 + frag_pos(4, o, c)] = v;
    } else if (i >= OFF_W4 && i < OFF_B4) {
        const int o = (int)((i - OFF_W4) / NH), c = (int)((i - OFF_W4) % NH);
        Pf[FRAG_L4 + frag_pos(1, c, o)] = v;
        Pf[TFRAG_L4 + frag_pos(4, o, c)] = v;
    }
}

// ---------------------------------------------------------------------------
// the network, forward and backward, on tiles of rows
// ---------------------------------------------------------------------------
constexpr int XPITCH = NFP + 8;  // LDS row pitch of the feature block (BF16; 16-byte rows, 20 banks apart)
constexpr int HPITCH = NH + 8;   // LDS row pitch of a hidden block
constexpr int YPITCH = 24;       // LDS row pitch of the output gradients (16 columns)

struct NetArgs {
    const float* X;          // [.][NF] raw features
    const float* Y;          // [.][NOUT] raw targets (training)
    const float* st;         // standardisation
    const uint16_t* Pf;      // weights in fragment order
    const float* P32;        // FP32 parameters (biases)
    long long n, rows;       // rows of X, rows of the batch
    int draw;                // batch rows drawn from X with Philox, else row r is r
    uint32_t k0, k1, step;
    float* out;              // [rows][NOUT] physical outputs (forward)
    uint16_t *Xt, *Ht[3], *dZt[3], *dYt;  // training: k_dw's operands, [rows / 16][column][16]
    float* db;               // [row tiles][NBIAS] column sums of the pre-activation gradients
    double* loss;
};

// Products of the wave's 32-column block for RB blocks of 32 rows: NS k steps
// of 16, inputs from LDS, weight fragments in registers.
template <int NS, int RB>
__device__ __forceinline__ void mfma_cols(const uint16_t* act, int pitch, const uint4 (&w)[NS], f32x16 (&acc)[RB]) {
    const int lane = threadIdx.x & 63, lr = lane & 31, h = lane >> 5;
#pragma unroll
    for (int b = 0; b < RB; ++b)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[b][r] = 0.0f;
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
        for (int b = 0; b < RB; ++b)
            acc[b] = mfma16(*(const uint4*)(act + (32 * b + lr) * pitch + s * 16 + 8 * h), w[s], acc[b]);
}

template <int NS>
__device__ __forceinline__ void load_frags(const uint16_t* Pf, int ncb, int blk, uint4 (&w)[NS]) {
    const uint4* p = (const uint4*)Pf + (threadIdx.x & 63);
#pragma unroll
    for (int s = 0; s < NS; ++s) w[s] = p[(s * ncb + blk) * 64];
}

// A 32-row column block (lane: column col, rows 8 q + 4 h + j in v[4 q + j])
// as BF16 into LDS rows of `pitch` and, four rows per store, into the
// row-blocked transpose g ([rows / 16][cols][16]) that k_dw reads.
template <bool TR>
__device__ __forceinline__ void put_cols(const float (&v)[16], int col, uint16_t* act, int pitch, uint16_t* g,
                                         long long kb0, int cols) {
    const int h = (threadIdx.x & 63) >> 5;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        uint16_t b[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            b[j] = to_bf16(v[4 * q + j]);
            if (act) act[(8 * q + 4 * h + j) * pitch + col] = b[j];
        }
        if constexpr (TR) {
            const uint2 pk = {(uint32_t)b[0] | ((uint32_t)b[1] << 16), (uint32_t)b[2] | ((uint32_t)b[3] << 16)};
            *(uint2*)(g + ((kb0 + (q >> 1)) * cols + col) * 16 + 8 * (q & 1) + 4 * h) = pk;
        }
    }
}

// Sum over the tile's 32 rows of a column block, on every lane of the column.
__device__ __forceinline__ float col_sum(const float (&v)[16]) {
    float s = 0.0f;
#pragma unroll
    for (int r = 0; r < 16; ++r) s += v[r];
    return s + __shfl_xor(s, 32);
}

// One workgroup of four waves per tile of 32 RB rows; wave w owns columns
// 32 w .. 32 w + 31 of every hidden layer, and its weight fragments of all
// layers are loaded at the start, while the rows are gathered.  Forward: the
// workgroup walks over tiles with its weights in registers.  The products run
// their k steps in the order of the plain product, the hidden activations are
// rounded to BF16 between layers and the accumulation is FP32.
//
// What bounds it: at the sizes of a request or a training batch (1,000 to
// 4,096 rows, 32 to 128 workgroups) the latency of one tile's chain of four
// (seven with the backward pass) short products.  Separate launches per layer
// with their activations in memory took 93 us for a forward pass of 1,000
// rows and 2.6 ms for an optimiser step of 4,096.
template <int RB, bool TRAIN>
__global__ void __launch_bounds__(256, RB) k_net(NetArgs a) {
    constexpr int TR = 32 * RB;
    static_assert(!TRAIN || RB == 1, "training tiles have 32 rows");
    __shared__ __align__(16) uint16_t xs[TR * XPITCH];  // features, then the second hidden block
    __shared__ __align__(16) uint16_t ha[TR * HPITCH];  // first and third hidden block
    __shared__ __align__(16) uint16_t dys[TRAIN ? 32 * YPITCH : 8];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, lr = lane & 31, h = lane >> 5;
    const int col = 32 * wave + lr;

    uint4 w1[NFP / 16], w2[NH / 16], w3[NH / 16], w4[NH / 16];
    load_frags(a.Pf + FRAG_L1, 4, wave, w1);
    load_frags(a.Pf + FRAG_L2, 4, wave, w2);
    load_frags(a.Pf + FRAG_L3, 4, wave, w3);
    load_frags(a.Pf + FRAG_L4, 1, 0, w4);
    [[maybe_unused]] uint4 t4[1], t3[NH / 16], t2[NH / 16];
    const float b1 = a.P32[OFF_B1 + col], b2 = a.P32[OFF_B2 + col], b3 = a.P32[OFF_B3 + col];
    const int oc = lr < NOUT ? lr : 0;
    const float b4 = a.P32[OFF_B4 + oc], ym = a.st[2 * NF + oc], ysd = a.st[2 * NF + NOUT + oc];
    constexpr int NC = (NFP + 63) / 64;  // columns per lane of a gathered row
    float mean[NC], inv[NC];
#pragma unroll
    for (int j = 0; j < NC; ++j) {
        const int c = lane + 64 * j;
        mean[j] = c < NF ? a.st[c] : 0.0f;
        // the binary32 reciprocal, as every kernel that standardises uses it
        inv[j] = c < NF ? 1.0f / a.st[NF + c] : 0.0f;
    }

    for (long long tile = blockIdx.x; tile * TR < a.rows; tile += gridDim.x) {
        const long long r0 = tile * TR;
        // source row of tile row `lane % TR`
        long long src = r0 + (lane & (TR - 1));
        const bool in = src < a.rows;
        if (TRAIN && a.draw) {
            const U4 w = rng_block(Key{a.k0, a.k1}, (uint32_t)src, a.step, 0u, P_MLP_BATCH, 0u);
            const uint64_t v = ((uint64_t)w.y << 32) | w.x;
            src = (long long)(v % (uint64_t)a.n);
        }
        if (!in) src = -1;
        // standardised features of the wave's rows (zero past the batch)
#pragma unroll 1
        for (int g = 0; g < RB; ++g) {
            float x[8][NC];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const long long sr = __shfl(src, (g * 4 + wave) * 8 + i);
#pragma unroll
                for (int j = 0; j < NC; ++j) {
                    const int c = lane + 64 * j;
                    x[i][j] = (sr >= 0 && c < NF) ? a.X[sr * NF + c] : mean[j];
                }
            }
#pragma unroll
            for (int i = 0; i < 8; ++i)
#pragma unroll
                for (int j = 0; j < NC; ++j) {
                    const int c = lane + 64 * j;
                    if (c < NFP) xs[((g * 4 + wave) * 8 + i) * XPITCH + c] = to_bf16((x[i][j] - mean[j]) * inv[j]);
                }
        }
        // the targets (training), or the LB velocities the outputs are
        // relative to, of the rows this wave finishes, in flight until then
        float uc[16];
        [[maybe_unused]] float yt[16];
        if (wave < RB) {
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const long long sr = __shfl(src, 32 * wave + 8 * (r >> 2) + 4 * h + (r & 3));
                uc[r] = (sr >= 0 && lr < 3) ? a.X[sr * NF + UC + lr] : 0.0f;
                if constexpr (TRAIN) yt[r] = (sr >= 0 && lr < NOUT) ? a.Y[sr * NOUT + lr] : 0.0f;
            }
        }
        __syncthreads();
        const long long kb0 = 2 * tile;
        if constexpr (TRAIN) {
            for (int c = threadIdx.x; c < NFP; c += 256)
#pragma unroll
                for (int b = 0; b < 2; ++b) {
                    uint32_t pk[8];
#pragma unroll
                    for (int i = 0; i < 8; ++i)
                        pk[i] = (uint32_t)xs[(16 * b + 2 * i) * XPITCH + c] |
                                ((uint32_t)xs[(16 * b + 2 * i + 1) * XPITCH + c] << 16);
                    uint4* o = (uint4*)(a.Xt + ((kb0 + b) * NFP + c) * 16);
                    o[0] = uint4{pk[0], pk[1], pk[2], pk[3]};
                    o[1] = uint4{pk[4], pk[5], pk[6], pk[7]};
                }
        }
        f32x16 acc[RB];
        float z1[16], z2[16], z3[16], v[16];
        auto hidden = [&](float bias, float (&z)[16], uint16_t* act, uint16_t* g) {
#pragma unroll
            for (int b = 0; b < RB; ++b) {
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    z[r] = acc[b][r] + bias;
                    v[r] = gelu(z[r]);
                }
                put_cols<TRAIN>(v, col, act + 32 * b * HPITCH, HPITCH, g, kb0, NH);
            }
        };
        mfma_cols<NFP / 16, RB>(xs, XPITCH, w1, acc);
        if constexpr (TRAIN) {
            // the backward pass's weights take the place of the first layer's
            load_frags(a.Pf + TFRAG_L4, 4, wave, t4);
            load_frags(a.Pf + TFRAG_L3, 4, wave, t3);
            load_frags(a.Pf + TFRAG_L2, 4, wave, t2);
        }
        hidden(b1, z1, ha, a.Ht[0]);
        __syncthreads();
        mfma_cols<NH / 16, RB>(ha, HPITCH, w2, acc);
        hidden(b2, z2, xs, a.Ht[1]);
        __syncthreads();
        mfma_cols<NH / 16, RB>(xs, HPITCH, w3, acc);
        hidden(b3, z3, ha, a.Ht[2]);
        __syncthreads();
        if (wave < RB) {
            f32x16 y[1];
            mfma_cols<NH / 16, 1>(ha + 32 * wave * HPITCH, HPITCH, w4, y);
            if constexpr (!TRAIN) {
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const long long row = r0 + 32 * wave + 8 * (r >> 2) + 4 * h + (r & 3);
                    if (lr < NOUT && row < a.rows) a.out[row * NOUT + lr] = (y[0][r] + b4) * ysd + ym + uc[r];
                }
            } else {
                const float nn = (float)(a.rows * NOUT);
                double l = 0.0;
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const bool ok = lr < NOUT && r0 + 8 * (r >> 2) + 4 * h + (r & 3) < a.rows;
                    const float dd = ok ? (y[0][r] + b4) - ((yt[r] - uc[r]) - ym) / ysd : 0.0f;
                    v[r] = 2.0f * dd / nn;
                    l += (double)dd * (double)dd / (double)(a.rows * NOUT);
                }
                if (lr < 16) put_cols<true>(v, lr, dys, YPITCH, a.dYt, kb0, 16);
                const float s = col_sum(v);
                if (lane < NOUT) a.db[tile * NBIAS + 3 * NH + lane] = s;
#pragma unroll
                for (int o = 32; o > 0; o >>= 1) l += __shfl_xor(l, o);
                if (lane == 0) atomicAdd(a.loss, l);
            }
        }
        if constexpr (TRAIN) {
            __syncthreads();
            auto back = [&](const float (&z)[16], uint16_t* act, uint16_t* g, int layer) {
#pragma unroll
                for (int r = 0; r < 16; ++r) v[r] = acc[0][r] * gelu_grad(z[r]);
                put_cols<true>(v, col, act, HPITCH, g, kb0, NH);
                const float s = col_sum(v);
                if (h == 0) a.db[tile * NBIAS + layer * NH + col] = s;
            };
            mfma_cols<1, 1>(dys, YPITCH, t4, acc);
            back(z3, ha, a.dZt[2], 2);
            __syncthreads();
            mfma_cols<NH / 16, 1>(ha, HPITCH, t3, acc);
            back(z2, xs, a.dZt[1], 1);
            __syncthreads();
            mfma_cols<NH / 16, 1>(xs, HPITCH, t2, acc);
            back(z1, nullptr, a.dZt[0], 0);
            break;  // one tile per workgroup
        }
    }
}

// Rows of physical outputs.  Up to 8,192 rows every 32-row tile has a CU of its
// own and the call takes one tile's latency (11.7 us); beyond, 64-row tiles read
// each weight fragment's operands once per two products, and two workgroups per
// CU walk over what is left (us, 64 rows / 32 rows: 8,193 rows 15.5 / 18.9,
// 16,384 16.3 / 21.9, 65,536 38.0 / 76.5, 524,288 270 / 633; one workgroup per
// CU 38.0 -> 55.2), although that form spills 16 of its 256 registers.
hipError_t net_forward(const float* X, long long rows, const float* st, const uint16_t* Pf, const float* P32, float* out,
                       hipStream_t s) {
    NetArgs a{};
    a.X = X; a.st = st; a.Pf = Pf; a.P32 = P32; a.n = rows; a.rows = rows; a.out = out;
    const long long most = 512;
    if (rows <= 8192) {
        hipLaunchKernelGGL((k_net<1, false>), dim3((unsigned)((rows + 31) / 32)), dim3(256), 0, s, a);
    } else {
        const long long tiles = (rows + 63) / 64;
        hipLaunchKernelGGL((k_net<2, false>), dim3((unsigned)(tiles < most ? tiles : most)), dim3(256), 0, s, a);
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// training
// ---------------------------------------------------------------------------
// Weight gradients dW[o][i] = sum over rows of dZ[row][o] In[row][i].  The
// operands lie in blocks of 16 rows, [rows / 16][column][16], so that a k
// step's fragment of 32 columns is one contiguous KiB, read straight into
// registers.  Workgroup (j, s) takes input block j of one layer (waves: the
// four output blocks) over split s of the rows and writes its own partial, so
// that the 18 x S workgroups fill the chip and no order depends on atomics;
// job 18 sums the bias gradients of the split's tiles.  With one split per
// 128 rows (at most 64 splits) a batch of 4,096 has 608 workgroups; as one
// product per layer over all rows it had 10, and took 0.64 ms.
struct DwArgs {
    const uint16_t *Xt, *Ht[3], *dZt[3], *dYt;
    const float* db;
    float* part;             // [S][NPARAM]
    long long nkb, chunk;    // 16-row blocks in all, per split
};

__global__ void __launch_bounds__(256) k_dw(DwArgs a) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, lr = lane & 31, h = lane >> 5;
    const int j = blockIdx.x;
    const long long kb0 = blockIdx.y * a.chunk;
    const long long kb1 = kb0 + a.chunk < a.nkb ? kb0 + a.chunk : a.nkb;
    float* part = a.part + blockIdx.y * NPARAM;
    if (j == 18) {
        // chunk is even and nkb is even: a tile of 32 rows is two blocks
        for (int c = threadIdx.x; c < NBIAS; c += 256) {
            float s = 0.0f;
            for (long long t = kb0 / 2; t < kb1 / 2; ++t) s += a.db[t * NBIAS + c];
            const long long o = c < NH ? OFF_B1 + c
                                       : (c < 2 * NH ? OFF_B2 + c - NH : (c < 3 * NH ? OFF_B3 + c - 2 * NH : OFF_B4 + c - 3 * NH));
            part[o] = s;
        }
        return;
    }
    const uint16_t *A, *B;
    int ca = NH, cb = NH, ib, ob = wave, om = NH;
    long long off;
    if (j < 9) { A = a.dZt[0]; B = a.Xt; cb = NFP; ib = j; off = OFF_W1; }
    else if (j < 13) { A = a.dZt[1]; B = a.Ht[0]; ib = j - 9; off = OFF_W2; }
    else if (j < 17) { A = a.dZt[2]; B = a.Ht[1]; ib = j - 13; off = OFF_W3; }
    else { A = a.dYt; B = a.Ht[2]; ca = 16; ib = wave; ob = 0; om = NOUT; off = OFF_W4; }
    const int ac = 32 * ob + lr;
    const uint16_t* pa = A + (kb0 * ca + (ac < ca ? ac : 0)) * 16 + 8 * h;
    const uint16_t* pb = B + (kb0 * cb + 32 * ib + lr) * 16 + 8 * h;
    const bool az = ac >= ca;
    f32x16 acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
    for (long long kb = kb0; kb < kb1; ++kb) {
        uint4 x = *(const uint4*)pa;
        const uint4 y = *(const uint4*)pb;
        if (az) x = uint4{0u, 0u, 0u, 0u};
        acc = mfma16(x, y, acc);
        pa += ca * 16;
        pb += cb * 16;
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int m = 32 * ob + 8 * (r >> 2) + 4 * h + (r & 3);
        if (m < om) part[off + (long long)m * cb + 32 * ib + lr] = acc[r];
    }
}

// The gradient as the sum of the splits, in their order; with ADAM it goes
// through Adam (Kingma & Ba) on the FP32 parameters, with the bias-corrected
// moment estimates, and the BF16 copies follow; else it is written to G.
struct ReduceArgs {
    const float* part;
    int S;
    float *G, *P, *m, *v;
    uint16_t* Pf;
    float lr, b1, b2, eps, c1, c2;
};

template <bool ADAM>
__global__ void __launch_bounds__(256) k_reduce(ReduceArgs a) {
    const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
    if (i >= NPARAM) return;
    float g = 0.0f;
#pragma unroll 8
    for (int s = 0; s < a.S; ++s) g += a.part[s * NPARAM + i];
    if constexpr (!ADAM) {
        a.G[i] = g;
    } else {
        const float mi = a.b1 * a.m[i] + (1.0f - a.b1) * g;
        const float vi = a.b2 * a.v[i] + (1.0f - a.b2) * g * g;
        a.m[i] = mi;
        a.v[i] = vi;
        const float p = a.P[i] - a.lr * (mi / a.c1) / (sqrtf(vi / a.c2) + a.eps);
        a.P[i] = p;
        frag_store(a.Pf, i, to_bf16(p));
    }
}

// Carve-up of the training scratch for a batch.
struct TrainBufs {
    uint16_t *Xt, *Ht[3], *dZt[3], *dYt;
    float *db, *part;
    long long nkb, chunk;
    int S;
};

static size_t train_carve(unsigned char* base, long long rows, TrainBufs& b) {
    size_t o = 0;
    auto take = [&](size_t bytes) { unsigned char* p = base + o; o += (bytes + 255) & ~(size_t)255; return p; };
    const long long tiles = (rows + 31) / 32;
    b.nkb = 2 * tiles;
    b.chunk = std::max(8LL, 2 * ((b.nkb + 127) / 128));  // at most 64 splits
    b.S = (int)((b.nkb + b.chunk - 1) / b.chunk);
    // longer chunks make fewer splits (64 at 8,192 rows, 52 just above): room
    // for as many as any smaller batch has, so that scratch serves fewer rows too
    const long long splits = std::min(64LL, (b.nkb + 7) / 8);
    b.Xt = (uint16_t*)take((size_t)b.nkb * NFP * 32);
    for (int l = 0; l < 3; ++l) {
        b.Ht[l] = (uint16_t*)take((size_t)b.nkb * NH * 32);
        b.dZt[l] = (uint16_t*)take((size_t)b.nkb * NH * 32);
    }
    b.dYt = (uint16_t*)take((size_t)b.nkb * 16 * 32);
    b.db = (float*)take((size_t)tiles * NBIAS * 4);
    b.part = (float*)take((size_t)splits * NPARAM * 4);
    return o;
}

size_t train_bytes(long long rows) {
    TrainBufs b;
    return train_carve(nullptr, rows, b);
}

hipError_t net_gradient(const NetBatch& q, void* scratch, float* G, const AdamState* adam, double* loss, hipStream_t s) {
    TrainBufs b;
    train_carve((unsigned char*)scratch, q.rows, b);
    NetArgs a{};
    a.X = q.X; a.Y = q.Y; a.st = q.st; a.Pf = q.Pf; a.P32 = q.P32; a.n = q.n; a.rows = q.rows; a.draw = q.draw ? 1 : 0;
    a.k0 = q.k0; a.k1 = q.k1; a.step = q.step; a.Xt = b.Xt; a.dYt = b.dYt; a.db = b.db; a.loss = loss;
    DwArgs d{};
    d.Xt = b.Xt; d.dYt = b.dYt; d.db = b.db; d.part = b.part; d.nkb = b.nkb; d.chunk = b.chunk;
    for (int l = 0; l < 3; ++l) {
        d.Ht[l] = a.Ht[l] = b.Ht[l];
        d.dZt[l] = a.dZt[l] = b.dZt[l];
    }
    hipLaunchKernelGGL((k_net<1, true>), dim3((unsigned)(b.nkb / 2)), dim3(256), 0, s, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_dw, dim3(19, (unsigned)b.S), dim3(256), 0, s, d);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    ReduceArgs r{};
    r.part = b.part; r.S = b.S; r.G = G;
    if (!adam) {
        hipLaunchKernelGGL(k_reduce<false>, dim3(nblk(NPARAM)), dim3(256), 0, s, r);
        return hipGetLastError();
    }
    r.P = adam->P32; r.Pf = adam->Pf; r.m = adam->m; r.v = adam->v;
    r.lr = adam->lr; r.b1 = adam->beta1; r.b2 = adam->beta2; r.eps = adam->eps;
    r.c1 = 1.0f - powf(adam->beta1, (float)adam->t);
    r.c2 = 1.0f - powf(adam->beta2, (float)adam->t);
    hipLaunchKernelGGL(k_reduce<true>, dim3(nblk(NPARAM)), dim3(256), 0, s, r);
    return hipGetLastError();
}

// Uniform(-a, a) weights with a = sqrt(6 / (fan_in + fan_out)) over the real
// inputs (Glorot), zero biases, zero padding columns, zero Adam moments.
__global__ void __launch_bounds__(256) k_mlp_init(float* P, float* m, float* v, uint32_t k0, uint32_t k1) {
    const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
    if (i >= NPARAM) return;
    float w = 0.0f;
    long long off = 0;
    int fin = 0, fout = 0, K = 0;
    bool weight = false;
    if (i < OFF_B1) { off = OFF_W1; fin = NF; fout = NH; K = NFP; weight = true; }
    else if (i >= OFF_W2 && i < OFF_B2) { off = OFF_W2; fin = NH; fout = NH; K = NH; weight = true; }
    else if (i >= OFF_W3 && i < OFF_B3) { off = OFF_W3; fin = NH; fout = NH; K = NH; weight = true; }
    else if (i >= OFF_W4 && i < OFF_B4) { off = OFF_W4; fin = NH; fout = NOUT; K = NH; weight = true; }
    if (weight && (int)((i - off) % K) < fin) {
        const U4 r = rng_block(Key{k0, k1}, (uint32_t)i, 0u, 0u, P_MLP_INIT, 0u);
        const double a = sqrt(6.0 / (double)(fin + fout));
        w = (float)((2.0 * u01(r.x, r.y) - 1.0) * a);
    }
    P[i] = w;
    m[i] = 0.0f;
    v[i] = 0.0f;
}

// Every element of the fragment arrays from the parameters, the padding zero:
// the inverse of frag_store's places.
__global__ void __launch_bounds__(256) k_frag_fill(const float* P, uint16_t* Pf) {
    const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
    if (i >= NFRAG) return;
    struct Part { long long at, w; int ncb, outs, ins; bool t; };
    constexpr Part parts[7] = {{FRAG_L1, OFF_W1, 4, NH, NFP, false},  {FRAG_L2, OFF_W2, 4, NH, NH, false},
                               {FRAG_L3, OFF_W3, 4, NH, NH, false},   {FRAG_L4, OFF_W4, 1, NOUT, NH, false},
                               {TFRAG_L2, OFF_W2, 4, NH, NH, true},   {TFRAG_L3, OFF_W3, 4, NH, NH, true},
                               {TFRAG_L4, OFF_W4, 4, NOUT, NH, true}};
    Part q = parts[0];
#pragma unroll
    for (int l = 1; l < 7; ++l)
        if (i >= parts[l].at) q = parts[l];
    const int e = (int)(i - q.at), lane = (e >> 3) & 63, sb = e >> 9;
    const int k = 16 * (sb / q.ncb) + 8 * (lane >> 5) + (e & 7), n = 32 * (sb % q.ncb) + (lane & 31);
    const int o = q.t ? k : n, c = q.t ? n : k;
    Pf[i] = o < q.outs ? to_bf16(P[q.w + (long long)o * q.ins + c]) : (uint16_t)0;
}

hipError_t mlp_refresh(const float* P32, uint16_t* Pf, hipStream_t s) {
    hipLaunchKernelGGL(k_frag_fill, dim3(nblk(NFRAG)), dim3(256), 0, s, P32, Pf);
    return hipGetLastError();
}

hipError_t mlp_init(float* P32, uint16_t* Pf, float* m, float* v, uint32_t k0, uint32_t k1, hipStream_t s) {
    hipLaunchKernelGGL(k_mlp_init, dim3(nblk(NPARAM)), dim3(256), 0, s, P32, m, v, k0, k1);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? mlp_refresh(P32, Pf, s) : e;
}

// ---------------------------------------------------------------------------
// data
// ---------------------------------------------------------------------------
// Column sums of x and x^2 (FP64), one thread per column, rows in blocks.
__global__ void __launch_bounds__(256) k_colstats(const float* X, long long n, int cols, long long rows_per,
                                                  double* sums) {
    const int c = blockIdx.y * 256 + threadIdx.x;
    if (c >= cols) return;
    const long long r0 = (long long)blockIdx.x * rows_per;
    const long long r1 = r0 + rows_per < n ? r0 + rows_per : n;
    double s1 = 0.0, s2 = 0.0;
    for (long long r = r0; r < r1; ++r) {
        const double x = X[r * cols + c];
        s1 += x;
        s2 += x * x;
    }
    atomicAdd(&sums[2 * c], s1);
    atomicAdd(&sums[2 * c + 1], s2);
}

__global__ void k_stats_final(const double* sx, const double* sy, long long n, float* stats) {
    const int c = threadIdx.x + blockIdx.x * blockDim.x;
    // The scale never drops below 1e-3 of the column's mean magnitude (nor
    // below 1e-12): columns that barely vary, such as the density of a
    // nearly incompressible flow, are not blown up to unit spread.
    auto fin = [&](const double* s, int col, float* mean, float* sd) {
        const double mu = s[2 * col] / (double)n;
        const double var = s[2 * col + 1] / (double)n - mu * mu;
        const double st = var > 0.0 ? sqrt(var) : 0.0;
        mean[col] = (float)mu;
        sd[col] = (float)fmax(fmax(st, 1e-3 * fabs(mu)), 1e-12);
    };
    if (c < NF) fin(sx, c, stats, stats + NF);
    if (c < NOUT) fin(sy, c, stats + 2 * NF, stats + 2 * NF + NOUT);
}

// Column sums of the network targets: velocity relative to the node's LB
// velocity, stress as is.
__global__ void __launch_bounds__(256) k_colstats_y(const float* Y, const float* X, long long n, long long rows_per,
                                                    double* sums) {
    const int c = threadIdx.x;
    if (c >= NOUT) return;
    const long long r0 = (long long)blockIdx.x * rows_per;
    const long long r1 = r0 + rows_per < n ? r0 + rows_per : n;
    double s1 = 0.0, s2 = 0.0;
    for (long long r = r0; r < r1; ++r) {
        const double y = (double)Y[r * NOUT + c] - (c < 3 ? (double)X[r * NF + UC + c] : 0.0);
        s1 += y;
        s2 += y * y;
    }
    atomicAdd(&sums[2 * c], s1);
    atomicAdd(&sums[2 * c + 1], s2);
}

hipError_t mlp_stats(const float* X, const float* Y, long long n, double* sums, float* stats, hipStream_t s) {
    hipError_t e = hipMemsetAsync(sums, 0, sizeof(double) * 2 * (NF + NOUT), s);
    if (e != hipSuccess) return e;
    const long long rows_per = 1024;
    const unsigned gx = (unsigned)((n + rows_per - 1) / rows_per);
    hipLaunchKernelGGL(k_colstats, dim3(gx, (NF + 255) / 256), dim3(256), 0, s, X, n, NF, rows_per, sums);
    hipLaunchKernelGGL(k_colstats_y, dim3(gx, 1), dim3(64), 0, s, Y, X, n, rows_per, sums + 2 * NF);
    hipLaunchKernelGGL(k_stats_final, dim3(2), dim3(256), 0, s, sums, sums + 2 * NF, n, stats);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// coupling
// ---------------------------------------------------------------------------
// Moments of node (x, y, z): rho, u = j / rho + g / 2, Pi_ab = sum f (c_a c_b
// - delta_ab / 3) in the order xx yy zz xy xz yz.
template <typename LT>
__device__ __forceinline__ void node_moments(const LT* fp, long long N, long long n, const double g[3],
                                             double m[10]) {
    using L = Lat<3>;
    double rho = 0.0, j[3] = {0.0, 0.0, 0.0}, P[6] = {0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int i = 0; i < L::Q; ++i) {
        const double fi = (double)fp[i * N + n];
        const double c0 = L::cx[i], c1 = L::cy[i], c2 = L::cz[i];
        rho += fi;
        j[0] += fi * c0; j[1] += fi * c1; j[2] += fi * c2;
        P[0] += fi * (c0 * c0 - 1.0 / 3.0);
        P[1] += fi * (c1 * c1 - 1.0 / 3.0);
        P[2] += fi * (c2 * c2 - 1.0 / 3.0);
        P[3] += fi * c0 * c1;
        P[4] += fi * c0 * c2;
        P[5] += fi * c1 * c2;
    }
    m[0] = rho;
    for (int a = 0; a < 3; ++a) m[1 + a] = j[a] / rho + 0.5 * g[a];
    for (int a = 0; a < 6; ++a) m[4 + a] = P[a];
}

// The 10 moments and the shear rate sqrt(2 S:S), S = -(Pi - rho u u) /
// (2 rho c_s^2 tau), of a node.
template <typename LT>
__device__ __forceinline__ void node_features(const LT* fp, const InstDesc& d, long long n, double m[11]) {
    node_moments<LT>(fp, d.N, n, d.g, m);
    const double rho = m[0], u[3] = {m[1], m[2], m[3]};
    const int A[6] = {0, 1, 2, 0, 0, 1}, B[6] = {0, 1, 2, 1, 2, 2};
    double ss = 0.0;
    for (int q = 0; q < 6; ++q) {
        const double Sab = -(m[4 + q] - rho * u[A[q]] * u[B[q]]) / (2.0 * rho * (1.0 / 3.0) * d.tau);
        ss += (q < 3 ? 1.0 : 2.0) * Sab * Sab;
    }
    m[10] = sqrt(2.0 * ss);
}

// Collection window: adds the moments and the shear rate of every band node
// (the rows [by0, by0 + nyb) that the slab's 3x3x3 stencils reach) to its
// FP64 sums facc[11][band nodes].  A slab node's 271 features are those of
// its 27 neighbours, so the window's sums are kept per band node and spread
// over the stencils once, at its end (k_collect_finish): summed per slab
// node, with every neighbour's moments formed 27 times, a step of 16,384 slab
// nodes took 216 us instead of 7.9, and the end of a window 132 us
// instead of 20.7.
template <typename LT>
__global__ void __launch_bounds__(256) k_features(const InstDesc* __restrict__ D, int inst, long long nband,
                                                  const LT* __restrict__ f, double* facc) {
    const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
    if (i >= nband) return;
    const InstDesc& d = D[inst];
    const int x = (int)(i % d.nx), yb = (int)((i / d.nx) % d.nyb), z = (int)(i / ((long long)d.nx * d.nyb));
    double m[11];
    node_features<LT>(f + d.node_off * Lat<3>::Q, d, ((long long)z * d.ny + (d.by0 + yb)) * d.nx + x, m);
#pragma unroll
    for (int q = 0; q < 11; ++q) facc[q * nband + i] += m[q];
}

hipError_t closure_features(int lb_fp, const InstDesc* D, int inst, long long nband, const void* f, double* facc,
                            hipStream_t s) {
    if (lb_fp == 64)
        hipLaunchKernelGGL(k_features<double>, dim3(nblk(nband)), dim3(256), 0, s, D, inst, nband, (const double*)f,
                           facc);
    else
        hipLaunchKernelGGL(k_features<float>, dim3(nblk(nband)), dim3(256), 0, s, D, inst, nband, (const float*)f, facc);
    return hipGetLastError();
}

// Network output -> the sample sums of every slab node (acc, when the
// feedback reads them) and, with do_prof, the profile: each of a node's r fine
// rows takes one sample at the predicted velocity.  A workgroup takes up to
// ACC_NODES nodes of one node row, sums them in FP64 and adds its sum to each
// fine row once (524,288 nodes: 2048 workgroups, 33 thousand FP64 atomics; one
// add per node, fine row and component were 8.4 million on 64 replicas of 64
// rows, 450 us).
constexpr int ACC_NODES = 1024;

__global__ void __launch_bounds__(256) k_to_acc(const InstDesc* __restrict__ D, int inst, const float* __restrict__ Y,
                                                const float* __restrict__ st, const float* __restrict__ uc, double* acc,
                                                double* prof, int do_prof) {
    __shared__ double red[4][4];
    const InstDesc& d = D[inst];
    const int nsy = d.yhi - d.ylo, yy = blockIdx.y;
    const long long nrow = (long long)d.nx * d.nz;  // nodes of one node row
    const long long i0 = (long long)blockIdx.x * ACC_NODES;
    double s[4] = {0.0, 0.0, 0.0, 0.0};
    for (int k = threadIdx.x; k < ACC_NODES; k += 256) {
        const long long i = i0 + k;
        if (i >= nrow) break;
        const long long z = i / d.nx, sn = (z * nsy + yy) * d.nx + (i - z * d.nx);
        double u[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            u[a] = (double)Y[sn * NOUT + a] * (double)st[2 * NF + NOUT + a] + (double)st[2 * NF + a] +
                   (double)uc[sn * 3 + a];
            s[1 + a] += u[a];
        }
        s[0] += 1.0;
        if (acc) {
            double* o = acc + (d.acc_off + sn) * 4;
            o[0] = 1.0; o[1] = u[0]; o[2] = u[1]; o[3] = u[2];
        }
    }
    if (!do_prof) return;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) s[q] += __shfl_xor(s[q], o);
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6][q] = s[q];
    }
    __syncthreads();
    const int q = threadIdx.x & 3;
    const double sum = red[0][q] + red[1][q] + red[2][q] + red[3][q];
    const int copy = (int)((blockIdx.x + blockIdx.y) % NCOPY);
    for (int i = threadIdx.x >> 2; i < d.r; i += 64)
        atomicAdd(&prof[(d.prof_off + (long long)copy * d.R + (long long)yy * d.r + i) * 4 + q], sum);
}

hipError_t closure_to_acc(const InstDesc* D, int inst, long long nslab, int nsy, const float* Y, const float* stats,
                          const float* uc, double* acc, double* prof, int do_prof, hipStream_t s) {
    if (!acc && !do_prof) return hipSuccess;
    hipLaunchKernelGGL(k_to_acc, dim3(nblk(nslab / nsy, ACC_NODES), (unsigned)nsy), dim3(256), 0, s, D, inst, Y, stats,
                       uc, acc, prof, do_prof);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// fused inference: features and the four layers in one kernel
// ---------------------------------------------------------------------------
// The 10 moments and the shear rate of every node of the rows [y0, y0 + nyb)
// that the slab's 3x3x3 stencils reach, computed exactly as the per-node
// feature kernel computes them.
template <typename LT>
__global__ void __launch_bounds__(256) k_band_moments(const InstDesc* __restrict__ D, int inst,
                                                      const LT* __restrict__ f, int y0, int nyb, float* M) {
    const InstDesc& d = D[inst];
    const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
    if (i >= (long long)d.nx * nyb * d.nz) return;
    const int x = (int)(i % d.nx), yb = (int)((i / d.nx) % nyb), z = (int)(i / ((long long)d.nx * nyb));
    const long long n = ((long long)z * d.ny + (y0 + yb)) * d.nx + x;
    double m[11];
    node_features<LT>(f + d.node_off * Lat<3>::Q, d, n, m);
    // binary32 is what the features use of them: (float)m - mean, then / std
    float* o = M + i * BMS;
    for (int q = 0; q < 10; ++q) o[q] = (float)m[q];
    o[10] = (float)m[10];
    o[11] = 0.0f;
}

// The network on every slab node: one wave takes 32 nodes through all layers
// on its own rows of LDS, with no barrier, so that the waves of a SIMD overlap
// one's gathers and products with another's GELUs.  The 271 features are
// gathered, standardised, rounded and multiplied in chunks of eight stencil
// entries (80 features, five k steps), which keeps a wave's LDS to one hidden
// block (8.5 KB) and lets three waves share a SIMD.  The k steps run in the
// order of k_net's, so the two agree bit for bit.  Outputs: the standardised
// network output Y and the centre node's LB velocity uc.
//
// What bounds it: the vector work of 384 GELUs and 271 features per node (the
// matrix cores are busy a tenth of the time) and the loads' latency.  524,288
// nodes: 194 us (370 TFLOP/s of network arithmetic); 334 us with all features
// of 32 rows in LDS (two waves per SIMD, a barrier per layer), 370 us with a
// wave per 32 columns and its weights in registers (two waves per SIMD, five
// barriers per tile).  Three waves per SIMD: at four 21 registers spill (235
// against 227 us before the chunks' loads moved ahead of the products).
constexpr int FTAB = 24;            // floats per stencil entry of the statistics table
constexpr int SWAVES = 4;           // waves per workgroup

// NB column blocks of one layer for the wave's 32 rows, NS k steps; weight
// fragments from the caches, one k step ahead.
template <int NS, int NB>
__device__ __forceinline__ void mfma_rows(const uint16_t* act, const uint4* wf, f32x16 (&acc)[NB]) {
    const int lane = threadIdx.x & 63, lr = lane & 31, h = lane >> 5;
    const uint16_t* ap = act + lr * HPITCH + 8 * h;
    uint4 w[2][NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) w[0][nb] = wf[nb * 64];
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        if (s + 1 < NS) {
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) w[(s + 1) & 1][nb] = wf[((s + 1) * NB + nb) * 64];
        }
        const uint4 x = *(const uint4*)(ap + 16 * s);
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) acc[nb] = mfma16(x, w[s & 1][nb], acc[nb]);
    }
}

// Orders the wave's LDS accesses (the LDS serves a wave's accesses in their
// order; this keeps the compiler from moving them).
__device__ __forceinline__ void wave_order() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

__global__ void __launch_bounds__(64 * SWAVES, 3) k_net_slab(const InstDesc* __restrict__ D, int inst, long long nslab,
                                                             int y0, int nyb, const float* __restrict__ M,
                                                             const float* __restrict__ st,
                                                             const uint16_t* __restrict__ Pf,
                                                             const float* __restrict__ P32, float* __restrict__ Y,
                                                             float* __restrict__ uc) {
    __shared__ __align__(16) uint16_t rows[SWAVES * 32 * HPITCH];
    __shared__ __align__(16) float tab[28 * FTAB];  // per stencil entry: 10 means (pad 2), 10 reciprocal deviations (pad 2)
    const InstDesc& d = D[inst];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, lr = lane & 31, h = lane >> 5;
    for (int k = threadIdx.x; k < NF; k += 64 * SWAVES) {
        tab[(k / 10) * FTAB + k % 10] = st[k];
        tab[(k / 10) * FTAB + 12 + k % 10] = 1.0f / st[NF + k];
    }
    __syncthreads();
    const long long r0 = ((long long)blockIdx.x * SWAVES + wave) * 32;
    if (r0 >= nslab) return;
    const long long sn = r0 + lr;
    const bool in = sn < nslab;
    const int nsy = d.yhi - d.ylo, nx = d.nx, ny = d.ny, nz = d.nz;
    const long long sc = in ? sn : 0, rw = sc / nx;
    const int x = (int)(sc - rw * nx), y = d.ylo + (int)(rw % nsy), z = (int)(rw / nsy);
    uint16_t* act = rows + wave * 32 * HPITCH;
    const uint4* wf = (const uint4*)Pf + lane;
    f32x16 acc[4];
    auto clear = [&] {
#pragma unroll
        for (int nb = 0; nb < 4; ++nb)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[nb][r] = 0.0f;
    };
    clear();
    // stencil entry e of the lane's node into columns c..c + 9 of its row
    auto node = [&](int e) {
        const int dx = e % 3 - 1, dy = (e / 3) % 3 - 1, dz = e / 9 - 1;
        int xx = x + dx; if (xx < 0) xx += nx; else if (xx >= nx) xx -= nx;
        int zz = z + dz; if (zz < 0) zz += nz; else if (zz >= nz) zz -= nz;
        int yy = y + dy; yy = yy < 0 ? 0 : (yy >= ny ? ny - 1 : yy);
        return (const float4*)(M + (((long long)zz * nyb + (yy - y0)) * nx + xx) * BMS);
    };
    auto put = [&](const float4& m0, const float4& m1, const float4& m2, int e, int c) {
        const float m[10] = {m0.x, m0.y, m0.z, m0.w, m1.x, m1.y, m1.z, m1.w, m2.x, m2.y};
        const float* t = tab + FTAB * e;
        uint32_t* o = (uint32_t*)(act + lr * HPITCH + c);
#pragma unroll
        for (int q = 0; q < 10; q += 2) {
            const uint32_t lo = to_bf16((m[q] - t[q]) * t[12 + q]);
            const uint32_t hi = to_bf16((m[q + 1] - t[q + 1]) * t[13 + q]);
            o[q / 2] = in ? lo | (hi << 16) : 0u;
        }
    };
    // three chunks of eight entries, then the last three, the shear rate of
    // the node itself and zeros; lane half h takes the entries of its parity.
    // Each chunk's nodes are loaded before the products of the chunk before.
    float4 m[4][3];
    auto load = [&](int ch) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int e = 8 * ch + 2 * i + h;
            const float4* p = node(e < 27 ? e : 13);
            m[i][0] = p[0]; m[i][1] = p[1]; m[i][2] = p[2];
        }
    };
    load(0);
#pragma unroll 1
    for (int ch = 0; ch < 3; ++ch) {
        wave_order();
#pragma unroll
        for (int i = 0; i < 4; ++i) put(m[i][0], m[i][1], m[i][2], 8 * ch + 2 * i + h, 10 * (2 * i + h));
        wave_order();
        load(ch + 1);
        mfma_rows<5, 4>(act, wf + (FRAG_L1 / 8 + ch * 5 * 4 * 64), acc);
    }
    wave_order();
    put(m[0][0], m[0][1], m[0][2], 24 + h, 10 * h);
    if (h == 0) {
        put(m[1][0], m[1][1], m[1][2], 26, 20);
    } else {
        uint32_t* o = (uint32_t*)(act + lr * HPITCH + 30);
        const float* t = tab + FTAB * 27;
        o[0] = in ? (uint32_t)to_bf16((m[1][2].z - t[0]) * t[12]) : 0u;
#pragma unroll
        for (int q = 1; q < 9; ++q) o[q] = 0u;
        if (in) {
            uc[sn * 3] = m[1][0].y;
            uc[sn * 3 + 1] = m[1][0].z;
            uc[sn * 3 + 2] = m[1][0].w;
        }
    }
    wave_order();
    mfma_rows<3, 4>(act, wf + (FRAG_L1 / 8 + 15 * 4 * 64), acc);
    auto hidden = [&](long long ob) {
        wave_order();
#pragma unroll
        for (int nb = 0; nb < 4; ++nb) {
            const float bias = P32[ob + 32 * nb + lr];
            float v[16];
#pragma unroll
            for (int r = 0; r < 16; ++r) v[r] = gelu(acc[nb][r] + bias);
            put_cols<false>(v, 32 * nb + lr, act, HPITCH, nullptr, 0, NH);
        }
        wave_order();
        clear();
    };
    hidden(OFF_B1);
    mfma_rows<NH / 16, 4>(act, wf + FRAG_L2 / 8, acc);
    hidden(OFF_B2);
    mfma_rows<NH / 16, 4>(act, wf + FRAG_L3 / 8, acc);
    hidden(OFF_B3);
    f32x16 yo[1];
#pragma unroll
    for (int r = 0; r < 16; ++r) yo[0][r] = 0.0f;
    mfma_rows<NH / 16, 1>(act, wf + FRAG_L4 / 8, yo);
    if (lr >= NOUT) return;
    const float b4 = P32[OFF_B4 + lr];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const long long row = r0 + 8 * (r >> 2) + 4 * h + (r & 3);
        if (row < nslab) Y[row * NOUT + lr] = yo[0][r] + b4;
    }
}

hipError_t closure_predict(int lb_fp, const InstDesc* D, int inst, long long nslab, long long nband, int y0,
                           int nyb, const void* f, float* M, const float* stats, const uint16_t* Pf,
                           const float* P32, float* Y, float* uc, hipStream_t s) {
    if (lb_fp == 64)
        hipLaunchKernelGGL(k_band_moments<double>, dim3(nblk(nband)), dim3(256), 0, s, D, inst, (const double*)f,
                           y0, nyb, M);
    else
        hipLaunchKernelGGL(k_band_moments<float>, dim3(nblk(nband)), dim3(256), 0, s, D, inst, (const float*)f,
                           y0, nyb, M);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_net_slab, dim3(nblk(nslab, 32 * SWAVES)), dim3(64 * SWAVES), 0, s, D, inst, nslab, y0, nyb, M,
                       stats, Pf, P32, Y, uc);
    return hipGetLastError();
}

__global__ void __launch_bounds__(256) k_destd_uc(const float* Y, const float* st, const float* uc, long long n,
                                                  float* out) {
    const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const int c = (int)(i % NOUT);
    const long long r = i / NOUT;
    out[i] = Y[i] * st[2 * NF + NOUT + c] + st[2 * NF + c] + (c < 3 ? uc[r * 3 + c] : 0.0f);
}

hipError_t mlp_destandardize_uc(const float* Y, const float* stats, const float* uc, long long rows, float* out,
                                hipStream_t s) {
    hipLaunchKernelGGL(k_destd_uc, dim3(nblk(rows * NOUT)), dim3(256), 0, s, Y, stats, uc, rows * NOUT, out);
    return hipGetLastError();
}

// One workgroup per particle tile: count, sum v and sum v v of every
// particle's LB node (all particles of the slab lie in slab nodes).  A tile
// of the shifted grid covers few nodes, so the sums go through an LDS window
// of those nodes (NMREP interleaved replicas of each, lane l adding into
// replica l mod NMREP) and reach memory with one global atomic per node and
// moment; a particle outside the window adds to memory directly.
constexpr int NMREP = 8;    // 40 KB of LDS with 10 FP64 sums per node and replica

template <typename PT>
__global__ void __launch_bounds__(256) k_node_moments(const InstDesc* __restrict__ D, int inst,
                                                      PartBuf P, const uint32_t* fill, double* nm) {
    __shared__ double win[NM_WIN * NMREP * 10];
    const InstDesc& d = D[inst];
    const uint32_t T = blockIdx.x;  // tile within the channel
    const uint32_t nxy = (uint32_t)d.ntx * (uint32_t)d.nty;
    const int tz = (int)(T / nxy), rem = (int)(T - (uint32_t)tz * nxy);
    const int ty = rem / d.ntx, tx = rem - ty * d.ntx;
    const int r = d.r, nsy = d.yhi - d.ylo;
    // nodes that particles binned in this tile can occupy (one cell of margin per side)
    const int wx0 = (tx * d.Tx) / r - 1, wy0 = (ty * d.Ty) / r - 1, wz0 = (tz * d.Tz) / r - 1;
    const int wnx = (d.Tx + r - 1) / r + 2, wny = (d.Ty + r - 1) / r + 2, wnz = (d.Tz + r - 1) / r + 2;
    const bool win_ok = wnx * wny * wnz <= NM_WIN;
    const int nwin = win_ok ? wnx * wny * wnz : 0;
    for (int i = threadIdx.x; i < nwin * NMREP * 10; i += 256) win[i] = 0.0;
    __syncthreads();
    const uint32_t n = min(fill[d.tile_off + T], (uint32_t)d.cap);
    const int A[6] = {0, 1, 2, 0, 0, 1}, B[6] = {0, 1, 2, 1, 2, 2};
    const int rep = (threadIdx.x & 63) & (NMREP - 1);
    for (uint32_t k = threadIdx.x; k < n; k += 256) {
        PT px[3], pv[3];
        uint32_t id;
        load_part<3, PT>(P, d.slot_off + (long long)T * d.cap, k, px, pv, id);
        const int x = min(max((int)floor((double)px[0]), 0), d.nx - 1);
        const int y = min(max((int)floor((double)px[1]), d.ylo), d.yhi - 1);
        const int z = min(max((int)floor((double)px[2]), 0), d.nz - 1);
        const double v[3] = {(double)pv[0], (double)pv[1], (double)pv[2]};
        double m[10];
        m[0] = 1.0;
        for (int a = 0; a < 3; ++a) m[1 + a] = v[a];
        for (int q = 0; q < 6; ++q) m[4 + q] = v[A[q]] * v[B[q]];
        int ax = x - wx0; if (ax < 0) ax += d.nx; else if (ax >= d.nx) ax -= d.nx;
        int az = z - wz0; if (az < 0) az += d.nz; else if (az >= d.nz) az -= d.nz;
        const int ay = (y - d.ylo) - wy0;
        double* o;
        if (win_ok && ax < wnx && ay >= 0 && ay < wny && az < wnz)
            o = win + 10 * (NMREP * (ax + wnx * (ay + wny * az)) + rep);
        else
            o = nm + (((long long)z * nsy + (y - d.ylo)) * d.nx + x) * 10;
        for (int q = 0; q < 10; ++q) atomicAdd(&o[q], m[q]);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < nwin * 10; i += 256) {
        const int w = i / 10, q = i - 10 * w;
        double sum = 0.0, cnt = 0.0;
        for (int rr = 0; rr < NMREP; ++rr) {
            sum += win[10 * (NMREP * w + rr) + q];
            cnt += win[10 * (NMREP * w + rr)];
        }
        if (cnt == 0.0) continue;  // no particle in this node
        const int ax = w % wnx, ay = (w / wnx) % wny, az = w / (wnx * wny);
        int x = wx0 + ax; if (x < 0) x += d.nx; else if (x >= d.nx) x -= d.nx;
        int z = wz0 + az; if (z < 0) z += d.nz; else if (z >= d.nz) z -= d.nz;
        const int yl = wy0 + ay;
        if (yl < 0 || yl >= nsy) continue;
        atomicAdd(&nm[(((long long)z * nsy + yl) * d.nx + x) * 10 + q], sum);
    }
}

hipError_t closure_node_moments(int part_fp, const InstDesc* D, int inst, long long ntiles, const PartBuf& buf,
                                const uint32_t* fill, double* nm, hipStream_t s) {
    if (part_fp == 64)
        hipLaunchKernelGGL(k_node_moments<double>, dim3((unsigned)ntiles), dim3(256), 0, s, D, inst,
                           buf, fill, nm);
    else
        hipLaunchKernelGGL(k_node_moments<float>, dim3((unsigned)ntiles), dim3(256), 0, s, D, inst,
                           buf, fill, nm);
    return hipGetLastError();
}

// Averages of the window: one wave per slab node, lane: features lane, lane +
// 64, ... (feature 10 e + q is moment q of stencil entry e = dz, dy, dx in
// -1..1, x and z periodic, y clamped to the channel; the last is the node's
// shear rate), then the targets.
__global__ void __launch_bounds__(256) k_collect_finish(const InstDesc* __restrict__ D, int inst, long long nslab,
                                                        long long nband, int K, double mass,
                                                        const double* __restrict__ facc, const double* __restrict__ nm,
                                                        float* X, float* Y) {
    const long long sn = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (sn >= nslab) return;
    const InstDesc& d = D[inst];
    const int lane = threadIdx.x & 63, nsy = d.yhi - d.ylo;
    const long long rw = sn / d.nx;
    const int x = (int)(sn - rw * d.nx), y = d.ylo + (int)(rw % nsy), z = (int)(rw / nsy);
    for (int k = lane; k < NF; k += 64) {
        const int e = k < NF - 1 ? k / 10 : 13, q = k < NF - 1 ? k - 10 * e : 10;
        int xx = x + e % 3 - 1; if (xx < 0) xx += d.nx; else if (xx >= d.nx) xx -= d.nx;
        int zz = z + e / 9 - 1; if (zz < 0) zz += d.nz; else if (zz >= d.nz) zz -= d.nz;
        int yy = y + (e / 3) % 3 - 1; yy = yy < 0 ? 0 : (yy >= d.ny ? d.ny - 1 : yy);
        X[sn * NF + k] = (float)(facc[q * nband + ((long long)zz * d.nyb + (yy - d.by0)) * d.nx + xx] / K);
    }
    if (!Y || lane >= NOUT) return;
    const double* o = nm + sn * 10;
    const double cnt = o[0];
    auto mean = [&](int a) { return cnt > 0.0 ? o[1 + a] / cnt : 0.0; };
    if (lane < 3) {
        Y[sn * NOUT + lane] = (float)mean(lane);
    } else {
        const int A[6] = {0, 1, 2, 0, 0, 1}, B[6] = {0, 1, 2, 1, 2, 2}, q = lane - 3;
        Y[sn * NOUT + lane] = (float)(mass * (o[4 + q] - cnt * mean(A[q]) * mean(B[q])) / K);
    }
}

hipError_t closure_collect_finish(const InstDesc* D, int inst, long long nslab, long long nband, int K, double mass,
                                  const double* facc, const double* nm, float* X, float* Y, hipStream_t s) {
    hipLaunchKernelGGL(k_collect_finish, dim3(nblk(nslab, 4)), dim3(256), 0, s, D, inst, nslab, nband, K, mass, facc, nm,
                       X, Y);
    return hipGetLastError();
}

}  // namespace lbmpcd
