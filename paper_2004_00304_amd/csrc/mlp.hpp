// mlp.hpp -- launchers of the learned closure's kernels (host side).
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

#include "common.hpp"
#include "launch.hpp"

namespace lbmpcd {

// The closure network: 271 features (the 3x3x3 stencil of rho, u(3) and
// Pi(6) around a slab node, plus the node's shear rate) -> 128 -> 128 -> 128
// -> 9 outputs (the node's MPCD mean velocity (3) and kinetic stress (6)),
// GELU between layers.  The first layer's inputs are padded to 288.
constexpr int NF = 271, NFP = 288, NH = 128, NOUT = 9;
// Flat FP32 parameter block: W1[NH][NFP] b1[NH] W2[NH][NH] b2 W3[NH][NH] b3
// W4[NOUT][NH] b4[NOUT] (each weight matrix is [out][in]).
constexpr long long OFF_W1 = 0;
constexpr long long OFF_B1 = OFF_W1 + (long long)NH * NFP;
constexpr long long OFF_W2 = OFF_B1 + NH;
constexpr long long OFF_B2 = OFF_W2 + (long long)NH * NH;
constexpr long long OFF_W3 = OFF_B2 + NH;
constexpr long long OFF_B3 = OFF_W3 + (long long)NH * NH;
constexpr long long OFF_W4 = OFF_B3 + NH;
constexpr long long OFF_B4 = OFF_W4 + (long long)NOUT * NH;
constexpr long long NPARAM = OFF_B4 + NOUT;
constexpr int NBIAS = 3 * NH + NOUT;
// The BF16 weights in the order the matrix cores read them as the B operand of
// a product: for layer l, k step s (16 inputs), 32-column block b and lane t of
// a wave, the 8 values W[32 b + t % 32][16 s + 8 (t / 32) + j], j = 0..7 (zero
// past the last output), so that every lane's 16 bytes of a (step, block) are
// contiguous.  TFRAG: the transposes of layers 2 to 4, the B operand of the
// input gradients (k runs over the layer's outputs, 9 padded to 16 in the
// last).
constexpr long long FRAG_L1 = 0;
constexpr long long FRAG_L2 = FRAG_L1 + (long long)(NFP / 16) * 4 * 512;
constexpr long long FRAG_L3 = FRAG_L2 + (long long)(NH / 16) * 4 * 512;
constexpr long long FRAG_L4 = FRAG_L3 + (long long)(NH / 16) * 4 * 512;
constexpr long long TFRAG_L2 = FRAG_L4 + (long long)(NH / 16) * 1 * 512;
constexpr long long TFRAG_L3 = TFRAG_L2 + (long long)(NH / 16) * 4 * 512;
constexpr long long TFRAG_L4 = TFRAG_L3 + (long long)(NH / 16) * 4 * 512;
constexpr long long NFRAG = TFRAG_L4 + 4 * 512;
// Standardisation: feature mean[NF], std[NF], target mean[NOUT], std[NOUT].
constexpr long long NSTATS = 2 * NF + 2 * NOUT;
// The network's velocity outputs are relative to the LB velocity of the node
// itself: the centre entry (dz = dy = dx = 0, the 14th of 27) of the
// stencil, features UC..UC+2.  Targets and forward outputs in physical units
// are absolute.
constexpr int UC = 13 * 10 + 1;
constexpr int BMS = 12;  // floats per band node of the fused inference: 10 moments, shear rate, pad

// C[M][N] = A[M][K] B[N][K]^T, row-major BF16 operands, FP32 accumulation and result.
struct GemmArgs {
    long long M, N, K;
    const uint16_t* A;
    const uint16_t* B;
    float* C;
};

hipError_t launch_gemm(const GemmArgs& g, hipStream_t s);

// Network on rows of raw features [rows][NF]: physical outputs [rows][NOUT].
// st: standardisation, Pf: BF16 weights in fragment order, P32: FP32
// parameters (biases).
hipError_t net_forward(const float* X, long long rows, const float* st, const uint16_t* Pf, const float* P32, float* out,
                       hipStream_t s);

// One batch of raw features and targets: `rows` rows, drawn uniformly from
// the n rows of X, Y with Philox when `draw`, else the first ones.
struct NetBatch {
    const float *X, *Y, *st;
    const uint16_t* Pf;
    const float* P32;
    long long n, rows;
    bool draw;
    uint32_t k0, k1, step;
};
// Adam's state and the step number t >= 1 of the update.
struct AdamState {
    float *P32, *m, *v;
    uint16_t* Pf;
    long long t;
    float lr, beta1, beta2, eps;
};
// Scratch bytes of a batch of `rows` rows.
size_t train_bytes(long long rows);
// Loss (mean squared error over rows x NOUT, accumulated into *loss) and the
// parameter gradient of a batch: into G (layout of the parameter block), or
// with `adam` straight through an Adam step.
hipError_t net_gradient(const NetBatch& q, void* scratch, float* G, const AdamState* adam, double* loss, hipStream_t s);

hipError_t mlp_init(float* P32, uint16_t* Pf, float* m, float* v, uint32_t k0, uint32_t k1, hipStream_t s);
// The fragment arrays from the FP32 parameters.
hipError_t mlp_refresh(const float* P32, uint16_t* Pf, hipStream_t s);

// Column statistics of raw features / targets.
hipError_t mlp_stats(const float* X, const float* Y, long long n, double* sums, float* stats, hipStream_t s);

// Collection window: adds moments and shear rate of one channel's band nodes
// to the FP64 sums facc, [11][nband].
hipError_t closure_features(int lb_fp, const InstDesc* D, int inst, long long nband, const void* f, double* facc,
                            hipStream_t s);
// Network output -> feedback sums (count 1, predicted velocity) of every slab
// node (unless acc is null); with do_prof also into the profile accumulators.
// nsy: node rows of the slab.
hipError_t closure_to_acc(const InstDesc* D, int inst, long long nslab, int nsy, const float* Y, const float* stats,
                          const float* uc, double* acc, double* prof, int do_prof, hipStream_t s);
// Fused inference of every slab node of the current populations: the moments
// and shear rate of the band rows [y0, y0 + nyb) into M (nband x 12 floats),
// then features and the four layers in one kernel.  Y: standardised output
// [nslab][NOUT]; uc: the node's LB velocity [nslab][3].
hipError_t closure_predict(int lb_fp, const InstDesc* D, int inst, long long nslab, long long nband, int y0,
                           int nyb, const void* f, float* M, const float* stats, const uint16_t* Pf,
                           const float* P32, float* Y, float* uc, hipStream_t s);
// Physical units from a standardised output and the nodes' LB velocities.
hipError_t mlp_destandardize_uc(const float* Y, const float* stats, const float* uc, long long rows, float* out,
                                hipStream_t s);
// Particle moments per slab node (count, sum v, sum v v) of one channel;
// one workgroup per particle tile.
hipError_t closure_node_moments(int part_fp, const InstDesc* D, int inst, long long ntiles, const PartBuf& buf,
                                const uint32_t* fill, double* nm, hipStream_t s);
// Averages of a collection window of K LB steps: features X [nslab][NF] from
// the band nodes' sums and, unless Y is null, targets Y [nslab][NOUT] (mean
// velocity, kinetic stress per unit volume).
hipError_t closure_collect_finish(const InstDesc* D, int inst, long long nslab, long long nband, int K, double mass,
                                  const double* facc, const double* nm, float* X, float* Y, hipStream_t s);

}  // namespace lbmpcd
