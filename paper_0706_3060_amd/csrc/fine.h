// Internal interface between the host runtime (api.cpp) and the fine pair tiles (fine.inl).
// Not part of the public ABI (include/nbody.h).
#pragma once
#include "kernels.h"

namespace nbk {

// ---- fine pair tiles: every unordered pair of one whole system once, in work units small enough
// to fill the chip from a few thousand particles on ----
// The pair operators.  Forces: the law's records and NC = 4 (3 without the potential) sums per
// particle, FP32 or FP64 pair arithmetic.  The others: FP32 pair arithmetic; the position adjoint
// of gravity (3 sums), the adjoint of LJC(linear) (6) and gravity's acceleration and jerk (7, 6
// without the potential).
enum FineOp { FINE_FORCE = 0, FINE_HVP = 1, FINE_LJC_ADJ = 2, FINE_JERK = 3 };
constexpr int kFineWaves = 4;                            // waves per workgroup
constexpr int kFineIch = 2, kFineIch4 = 4;               // i chunks of 64 records per wave: 2 or 4
constexpr int kFineMaxWgs = 1024;                        // workgroups of a launch, at most: four on each of 256 CUs
constexpr int64_t kFineMaxN = int64_t(1) << 18;

// Columns of a slot row: the operator's sums rounded up to 4 or 8.
__host__ __device__ inline int fine_cols(int op) { return op == FINE_LJC_ADJ || op == FINE_JERK ? 8 : 4; }

// The work of n particles: nch chunks of 64 records, nb blocks of ch = kFineWaves ich chunks.  Block b
// meets chunks b ch .. nch - 1, one sweep of 64 steps each, cut into four quarters of 16 steps;
// the quarters of all blocks, block after block and chunk after chunk, form one line of
// fine_begin(nb, nch, ch) quarters that the workgroups share out in equal contiguous pieces.
__host__ __device__ inline int fine_begin(int b, int nch, int ch) { return 4 * (b * nch - ch * (b * (b - 1) / 2)); }

// The j slots of the blocks follow one another, block b's from its own first row on (it meets no
// row before): row r (of nb blocks of `rows`) of block b lies at slot row fine_jslot(b, nb, rows) + r, of
// fine_jslot_rows(nb, rows) in all.
// (At most 2^25.1 rows, 2^18 particles in blocks of 1,024.)
__host__ __device__ inline int fine_jslot(int b, int nb, int rows) { return rows * (b * nb - b * (b + 1) / 2); }
__host__ __device__ inline int fine_jslot_rows(int nb, int rows) { return rows * (nb * (nb + 1) / 2); }

struct FineLaunch {
    int op, law, prec, pot;
    int64_t n;
    int ich;                       // i chunks of a wave, 2 or 4
    int nch, nb;                   // chunks and blocks of the n particles
    int per, nwg;                  // quarters per workgroup (>= 4), workgroups
    int wide, wide_i;              // FP32 pair arithmetic: the j slots and carries, and the i slots, are FP64
    double eps2;
    double zeta[4];
    const void *rec;               // records, padded to whole blocks
    void *jslot;                   // [fine_jslot_rows][cols] j sums of the blocks' sweeps
    void *islot;                   // [nwg + nb][rows of a block][cols] i sums of workgroup w in block b: w + b
    void *carry;                   // [nwg][64][cols] j sums of a sweep that began in the workgroup before
    Epilogue epi;                  // FINE_FORCE
    StepNext next;
    double G, qscale;              // the adjoints and the jerk
    const double *params;
    double *grad_pos, *grad_params;
    double *out_acc, *out_jerk, *out_pot;
};
bool fine_supported(int op, int law, int prec);
bool fine_has4(int op, int law, int prec);               // with four i chunks a wave too
hipError_t launch_fine(const FineLaunch &a, hipStream_t s);
hipError_t launch_fine_reduce(const FineLaunch &a, hipStream_t s);

}  // namespace nbk
