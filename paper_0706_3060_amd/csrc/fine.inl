// Fine pair tiles: every unordered pair {i, j} of one whole system once, its terms applied to both
// particles (Newton's third law), in work units of a block's rows by 16 steps, for systems whose coarser
// tiles would leave much of the chip idle and for FP64 pair arithmetic.
//
// Decomposition.  The rows form blocks of 8 or 16 chunks of 64 (512 or 1,024 rows); a workgroup of four waves holds one
// block in registers, two or four chunks a wave, and sweeps j chunks from the block's own onwards.
// A sweep takes 64 steps: at step s lane l pairs its i particles with particle j = l + s (mod
// 64) of the chunk, which is staged twice in LDS so that each lane reads its record at a constant
// offset.  The j sums travel with their particle from lane to lane (most through the LDS crossbar,
// the last on the VALU by a DPP rotation: the two units share the moves); after the sweep the four
// waves' j sums meet in LDS, are added in wave order, and leave as one row of the block's j slot.
// Inside the block's own chunks, chunk k meets chunk q symmetrically when q > k, one-sidedly (i side
// only, the own pair neutralised) when q == k, and not at all when q < k.
//
// Balance.  The sweeps of all blocks, in quarters of 16 steps, form one line that the launch cuts
// into equal contiguous pieces, one per workgroup, so that every SIMD gets the same number of steps
// (8,192 particles: 1,088 sweeps for 256 CUs, which whole sweeps would fill to 85 % and quarters
// fill to 94 %).  A piece may begin inside a sweep: the j sums of such a sweep's rest go to the
// workgroup's carry row.  A piece that crosses into the next block writes the i sums of the block it
// leaves and loads the next.
//
// Sums.  i sums: FP32 partials of a sweep (64 terms) folded into Kahan or FP64 sums (FP64: plain FP64
// partials folded with compensation).  j sums: a wave's terms of a sweep in the law's type, 128 with
// two i chunks and 256 with four, and the four waves' sums in FP64.  FP32 chains of at most 256 are what
// the one-sided kernels add before they fold, and like theirs the slots are FP64 (`wide`) below the
// coarser tiles' sizes; from there on FP32 as those tiles' are.  The i slots of pieces of at most 16
// quarters hold no more than such a chain, 256 terms, and are FP32 at every size (8,192 LJC(linear) atoms
// with energies: 12 MB of FP64 i slots, all stored at the launch's end, cost 3 us of 45).  Every slot row is written once;
// k_fine_reduce adds a row's j slots, carries and i sums in a fixed order in FP64 with compensation, so
// results repeat bit for bit.
#include "allpairs.h"
#include "fine.h"

namespace nbk {
namespace {

constexpr int kQuarter = 16;                             // steps of a quarter sweep

// ------------------------------------------------------------------ moves
__device__ __forceinline__ float next_cross(int byte_addr, float v) { return from_next_lane(byte_addr, v); }
__device__ __forceinline__ double next_cross(int byte_addr, double v)
{
    const int2 w = __builtin_bit_cast(int2, v);
    return __builtin_bit_cast(double, int2{__builtin_amdgcn_ds_bpermute(byte_addr, w.x),
                                           __builtin_amdgcn_ds_bpermute(byte_addr, w.y)});
}
__device__ __forceinline__ float next_dpp(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0x134, 0xF, 0xF, false));
}
__device__ __forceinline__ double next_dpp(double v)
{
    const int2 w = __builtin_bit_cast(int2, v);
    return __builtin_bit_cast(double, int2{__builtin_amdgcn_mov_dpp(w.x, 0x134, 0xF, 0xF, false),
                                           __builtin_amdgcn_mov_dpp(w.y, 0x134, 0xF, 0xF, false)});
}

// -------------------------------------------------------------- operators
// Each: record type Rec (kCols values of T, of which the pair reads the first kStage), the sums NC per
// particle, how many of them move through the crossbar, and the pair.  own marks the particle's own
// pair, which contributes nothing; JS: add the j side.
// FAR: m / s^3 as (m / s) / s^2, the one-sided kernels' order, whose range holds FP32 masses and
// distances in SI units; otherwise m times s^-3, the coarser tiles', a multiplication less for the two
// particles and out of FP32's range for distances above 4e12 or below 2e-13.
template <typename PT, bool POT, bool FAR = false> struct GravOp {
    using T = PT;
    struct alignas(16) Rec { T x, y, z, m; };
    static constexpr int kCols = 4, kStage = 4, NC = POT ? 4 : 3, kCross = sizeof(T) == 8 ? 0 : 3;
    template <bool JS>
    static __device__ __forceinline__ void pair(const Rec &I, const Rec &J, const PairK<T> &k, bool own, T (&p)[NC],
                                                T (&jv)[NC])
    {
        const T dx = J.x - I.x, dy = J.y - I.y, dz = J.z - I.z;
        T r2 = fma_(dx, dx, k.eps2);
        r2 = fma_(dy, dy, r2);
        r2 = fma_(dz, dz, r2);
        T mj = J.m;
        r2 = own ? T(1) : r2;
        mj = own ? T(0) : mj;
        const T ri = rsqrt_(r2);
        const T ri2 = ri * ri;
        const T ri3 = ri2 * ri;
        const T cj = FAR ? (mj * ri) * ri2 : mj * ri3;
        p[0] = fma_(cj, dx, p[0]);
        p[1] = fma_(cj, dy, p[1]);
        p[2] = fma_(cj, dz, p[2]);
        if constexpr (POT) p[3] = fma_(mj, ri, p[3]);
        if constexpr (JS) {
            const T ci = FAR ? (I.m * ri) * ri2 : I.m * ri3;
            jv[0] = fma_(-ci, dx, jv[0]);
            jv[1] = fma_(-ci, dy, jv[1]);
            jv[2] = fma_(-ci, dz, jv[2]);
            if constexpr (POT) jv[3] = fma_(I.m, ri, jv[3]);
        }
    }
};

template <typename PT, bool POT, int LAW> struct LjcOp {
    using T = PT;
    struct alignas(16) Rec { T x, y, z, qs, sh, se, p0, p1; };
    static constexpr int kCols = 8, kStage = sizeof(T) == 8 ? 6 : 8, NC = POT ? 4 : 3, kCross = sizeof(T) == 8 ? 0 : 3;
    template <bool JS>
    static __device__ __forceinline__ void pair(const Rec &I, const Rec &J, const PairK<T> &k, bool own, T (&p)[NC],
                                                T (&jv)[NC])
    {
        const T dx = J.x - I.x, dy = J.y - I.y, dz = J.z - I.z;
        T r2 = dx * dx;
        r2 = fma_(dy, dy, r2);
        r2 = fma_(dz, dz, r2);
        T qq = I.qs * J.qs;
        T e = I.se * J.se;
        r2 = own ? T(1) : r2;
        qq = own ? T(0) : qq;
        e = own ? T(0) : e;
        T W, u = T(0);
        ljc_terms<POT, LAW>(r2, qq, e, I.sh + J.sh, k, W, u);
        p[0] = fma_(-W, dx, p[0]);
        p[1] = fma_(-W, dy, p[1]);
        p[2] = fma_(-W, dz, p[2]);
        if constexpr (POT) p[3] += u;
        if constexpr (JS) {
            jv[0] = fma_(W, dx, jv[0]);
            jv[1] = fma_(W, dy, jv[1]);
            jv[2] = fma_(W, dz, jv[2]);
            if constexpr (POT) jv[3] += u;
        }
    }
};

// Gravity's position adjoint: with w = m_i g_j - m_j g_i the term t = s^-3 (w - 3 s^-2 (d.w) d) of i
// is minus that of j.
struct HvpOp {
    using T = float;
    struct alignas(16) Rec { T x, y, z, m, gx, gy, gz, p0; };
    static constexpr int kCols = 8, kStage = 8, NC = 3, kCross = 2;
    template <bool JS>
    static __device__ __forceinline__ void pair(const Rec &I, const Rec &J, const PairK<T> &k, bool own, T (&p)[NC],
                                                T (&jv)[NC])
    {
        const T dx = J.x - I.x, dy = J.y - I.y, dz = J.z - I.z;
        T r2 = fma_(dx, dx, k.eps2);
        r2 = fma_(dy, dy, r2);
        r2 = fma_(dz, dz, r2);
        r2 = own ? 1.0f : r2;
        T ri = rsqrt_(r2);
        ri = own ? 0.0f : ri;
        const T ri2 = ri * ri;
        const T ri3 = ri2 * ri;
        const T wx = fma_(-J.m, I.gx, I.m * J.gx);
        const T wy = fma_(-J.m, I.gy, I.m * J.gy);
        const T wz = fma_(-J.m, I.gz, I.m * J.gz);
        T dw = dx * wx;
        dw = fma_(dy, wy, dw);
        dw = fma_(dz, wz, dw);
        const T u = (ri2 * 3.0f) * dw;
        const T t[3] = {fma_(-u, dx, wx), fma_(-u, dy, wy), fma_(-u, dz, wz)};
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            p[c] = fma_(ri3, t[c], p[c]);
            if constexpr (JS) jv[c] = fma_(-ri3, t[c], jv[c]);
        }
    }
};

// LJC(linear)'s adjoint: with u = g_j - g_i the position terms are opposite, and the charge, sigma
// and epsilon terms share x (d.u); the derivatives are those of the one-sided adjoint kernel.
struct LjcAdjOp {
    using T = float;
    struct alignas(16) Rec { T x, y, z, qs, sh, se, gx, gy, gz, p0, p1, p2; };
    static constexpr int kCols = 16, kStage = 12, NC = 6, kCross = 5;
    template <bool JS>
    static __device__ __forceinline__ void pair(const Rec &I, const Rec &J, const PairK<T> &, bool own, T (&p)[NC],
                                                T (&jv)[NC])
    {
        const T dx = J.x - I.x, dy = J.y - I.y, dz = J.z - I.z;
        T r2 = dx * dx;
        r2 = fma_(dy, dy, r2);
        r2 = fma_(dz, dz, r2);
        T qq = I.qs * J.qs;
        T e = I.se * J.se;
        r2 = own ? 1.0f : r2;
        qq = own ? 0.0f : qq;
        e = own ? 0.0f : e;
        const T x = rcp_(r2);
        const T sg = I.sh + J.sh;
        const T sgx = sg * x;
        const T s2 = sg * sgx;
        const T s4 = s2 * s2;
        const T s6 = s4 * s2;
        const T lj = e * s6;
        const T t = fma_(s6, 2.0f, -1.0f);
        const T cx = qq * x;
        const T W = fma_(lj, t, cx) * x;
        const T wpr = fma_(lj, fma_(s6, 28.0f, -8.0f), cx * 4.0f) * (x * x);
        const T ux = J.gx - I.gx, uy = J.gy - I.gy, uz = J.gz - I.gz;
        T du = dx * ux;
        du = fma_(dy, uy, du);
        du = fma_(dz, uz, du);
        du = own ? 0.0f : du;
        const T tt = wpr * du;
        const T v[3] = {fma_(tt, dx, -W * ux), fma_(tt, dy, -W * uy), fma_(tt, dz, -W * uz)};
        const T xdu = x * du;
        const T A = x * xdu;
        const T B = ((e * (s4 * sgx)) * fma_(s6, 4.0f, -1.0f)) * xdu;
        const T C = (s6 * t) * xdu;
#pragma unroll
        for (int c = 0; c < 3; ++c) p[c] += v[c];
        p[3] = fma_(J.qs, A, p[3]);
        p[4] += B;
        p[5] = fma_(J.se, C, p[5]);
        if constexpr (JS) {
#pragma unroll
            for (int c = 0; c < 3; ++c) jv[c] -= v[c];
            jv[3] = fma_(I.qs, A, jv[3]);
            jv[4] += B;
            jv[5] = fma_(I.se, C, jv[5]);
        }
    }
};

// Acceleration and jerk: with w = v_j - v_i and u = w - 3 (d.w) d / s^2, i gets m_j d / s^3 and
// m_j u / s^3, j the same with -m_i (m / s^3 as (m / s) / s^2, as in GravOp).
template <bool POT> struct JerkOp {
    using T = float;
    struct alignas(16) Rec { T x, y, z, m, vx, vy, vz, p0; };
    static constexpr int kCols = 8, kStage = 8, NC = POT ? 7 : 6, kCross = 4;
    template <bool JS>
    static __device__ __forceinline__ void pair(const Rec &I, const Rec &J, const PairK<T> &k, bool own, T (&p)[NC],
                                                T (&jv)[NC])
    {
        const T dx = J.x - I.x, dy = J.y - I.y, dz = J.z - I.z;
        const T wx = J.vx - I.vx, wy = J.vy - I.vy, wz = J.vz - I.vz;
        T r2 = fma_(dx, dx, k.eps2);
        r2 = fma_(dy, dy, r2);
        r2 = fma_(dz, dz, r2);
        T mj = J.m;
        r2 = own ? 1.0f : r2;
        mj = own ? 0.0f : mj;
        const T ri = rsqrt_(r2);
        const T ri2 = ri * ri;
        T dw = dx * wx;
        dw = fma_(dy, wy, dw);
        dw = fma_(dz, wz, dw);
        const T q = (dw * ri2) * -3.0f;
        const T ux = fma_(q, dx, wx), uy = fma_(q, dy, wy), uz = fma_(q, dz, wz);
        const T cj = (mj * ri) * ri2;
        p[0] = fma_(cj, dx, p[0]);
        p[1] = fma_(cj, dy, p[1]);
        p[2] = fma_(cj, dz, p[2]);
        p[3] = fma_(cj, ux, p[3]);
        p[4] = fma_(cj, uy, p[4]);
        p[5] = fma_(cj, uz, p[5]);
        if constexpr (POT) p[6] = fma_(mj, ri, p[6]);
        if constexpr (JS) {
            const T ci = (I.m * ri) * ri2;
            jv[0] = fma_(-ci, dx, jv[0]);
            jv[1] = fma_(-ci, dy, jv[1]);
            jv[2] = fma_(-ci, dz, jv[2]);
            jv[3] = fma_(-ci, ux, jv[3]);
            jv[4] = fma_(-ci, uy, jv[4]);
            jv[5] = fma_(-ci, uz, jv[5]);
            if constexpr (POT) jv[6] = fma_(I.m, ri, jv[6]);
        }
    }
};

// 128-bit vectors of a staged record
template <class Op> constexpr int kVecs = Op::kStage * (int)sizeof(typename Op::T) / 16;

template <class Op>
__device__ __forceinline__ typename Op::Rec rec_from(const float4 *v, int stride)
{
    typename Op::Rec r;
    float4 *o = (float4 *)&r;
#pragma unroll
    for (int k = 0; k < kVecs<Op>; ++k) o[k] = v[k * stride];
    return r;
}

template <class Op, int NC = Op::NC, typename T = typename Op::T>
__device__ __forceinline__ void move_on(int addr, T (&jv)[NC])
{
#pragma unroll
    for (int c = 0; c < NC; ++c) jv[c] = c < Op::kCross ? next_cross(addr, jv[c]) : next_dpp(jv[c]);
}

// Steps s0 .. s1 - 1 of a sweep: the wave's i chunks before OWN against the chunk in `st`
// symmetrically, i chunk OWN (when the wave has it: the chunk itself) one-sidedly.
template <class Op, int OWN, int I>
__device__ __forceinline__ void fine_sweep(const float4 (&st)[kVecs<Op>][2 * kWave], int s0, int s1,
                                           const typename Op::Rec (&iv)[I], const PairK<typename Op::T> &kc,
                                           int addr, typename Op::T (&p)[I][Op::NC], typename Op::T (&jv)[Op::NC])
{
    using R = typename Op::Rec;
    const int lane = lane_id();
    R J = rec_from<Op>(&st[0][lane + s0], 2 * kWave);
    for (int s = s0; s < s1; s += kQuarter) {
        const float4 *at = &st[0][lane + s + 1];
#pragma unroll(16 / I)
        for (int u = 0; u < kQuarter; ++u) {
            // the next step's record, a step ahead (at most record 127 of the chunk staged twice)
            const R next = rec_from<Op>(at + u, 2 * kWave);
#pragma unroll
            for (int k = 0; k < OWN; ++k) Op::template pair<true>(iv[k], J, kc, false, p[k], jv);
            if constexpr (OWN < I) Op::template pair<false>(iv[OWN], J, kc, s + u == 0, p[OWN], jv);
            if constexpr (OWN > 0) move_on<Op>(addr, jv);
            J = next;
        }
    }
}

// the block of the quarter q: the last whose first quarter is at or before q
__device__ __forceinline__ int fine_block(int q, int nb, int nch, int ch)
{
    int lo = 0, hi = nb - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) / 2;
        if (fine_begin(mid, nch, ch) <= q) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// waves per SIMD the register allocation aims at (FP64 with four i chunks holds 190 to 250 registers)
template <class Op, int I> constexpr int fine_waves_per_eu()
{
    if (sizeof(typename Op::T) == 8) return I == 2 ? 3 : 2;
    return Op::NC >= 6 ? 3 : 4;
}

// the i sums of a wave's chunks, one slot row a lane and chunk
template <typename S, int NC, int NCP, int PREC, int I>
__device__ __forceinline__ void put_sums(S *dst, const RunSum<PREC> (&acc)[I][NC])
{
#pragma unroll
    for (int k = 0; k < I; ++k)
#pragma unroll
        for (int c = 0; c < NCP; ++c) dst[k * kWave * NCP + c] = c < NC ? (S)acc[k][c < NC ? c : 0].value() : S(0);
}

}  // namespace

template <class Op, int PREC, int I>
__global__ __launch_bounds__(kFineWaves * kWave) __attribute__((amdgpu_waves_per_eu(fine_waves_per_eu<Op, I>())))
void k_fine(FineLaunch a)
{
    using T = typename Op::T;
    using R = typename Op::Rec;
    constexpr int NC = Op::NC, NCP = NC > 4 ? 8 : 4, V = kVecs<Op>;
    constexpr int RV = Op::kCols * (int)sizeof(T) / 16;         // vectors from record to record
    constexpr int kChunks = kFineWaves * I, kRows = kChunks * kWave;   // of a block
    __shared__ float4 st[2][V][2 * kWave];                      // the j chunk, staged twice, two buffers
    __shared__ T jr[2][kFineWaves][kWave][NCP];                 // the waves' j sums of a sweep, two buffers
    const int lane = lane_id();
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nch = a.nch, nb = a.nb;
    // the workgroups reach the XCDs in turn: each XCD takes a contiguous run of pieces
    const int wg = (int)(blockIdx.x % kSymXcds) * (int)(gridDim.x / kSymXcds) + (int)(blockIdx.x / kSymXcds);
    const int total = fine_begin(nb, nch, kChunks);
    if (wg >= a.nwg || (int64_t)wg * a.per >= total) return;    // whole workgroup
    int q = wg * a.per;
    const int qe = q + a.per < total ? q + a.per : total;
    int b = fine_block(q, nb, nch, kChunks);
    int jc = b * kChunks + (q - fine_begin(b, nch, kChunks)) / 4;
    int s0 = (q % 4) * kQuarter;                                // fine_begin is a multiple of 4
    const float4 *__restrict__ rec4 = (const float4 *)a.rec;
    PairK<T> kc;
    kc.eps2 = (T)a.eps2;
    kc.za = (T)a.zeta[0];
    kc.zb = (T)a.zeta[1];
    kc.zc = (T)a.zeta[2];
    kc.zd = (T)a.zeta[3];
    kc.za3 = (T)(3.0 * a.zeta[0]);
    kc.zb2 = (T)(2.0 * a.zeta[1]);
    const int addr = ((lane + 1) & (kWave - 1)) * 4;

    R iv[I];
    RunSum<PREC> acc[I][NC];
    T p[I][NC];
    auto load_block = [&]() {
#pragma unroll
        for (int k = 0; k < I; ++k) {
            iv[k] = rec_from<Op>(rec4 + ((int64_t)(b * kChunks + w * I + k) * kWave + lane) * RV, 1);
#pragma unroll
            for (int c = 0; c < NC; ++c) acc[k][c] = RunSum<PREC>{};
        }
    };
    load_block();
    // the first chunk: wave w stages vectors w, w + 4, ... of its 64 records
    constexpr int VW = (V + kFineWaves - 1) / kFineWaves;
    float4 g[VW];
    auto fetch = [&](int c) {
#pragma unroll
        for (int k = 0; k < VW; ++k)
            if (w + k * kFineWaves < V) g[k] = rec4[((int64_t)c * kWave + lane) * RV + w + k * kFineWaves];
    };
    auto stage = [&](int buf) {
#pragma unroll
        for (int k = 0; k < VW; ++k)
            if (w + k * kFineWaves < V) {
                st[buf][w + k * kFineWaves][lane] = g[k];
                st[buf][w + k * kFineWaves][lane + kWave] = g[k];
            }
    };
    fetch(jc);
    stage(0);
    __syncthreads();
    int buf = 0;
    for (;;) {
        const int s1 = s0 + (qe - q) * kQuarter < kWave ? s0 + (qe - q) * kQuarter : kWave;
        q += (s1 - s0) / kQuarter;
        // the sweep after this one
        const bool more = q < qe;
        const bool over = jc + 1 >= nch;                        // it begins the next block
        const int jn = over ? (b + 1) * kChunks : jc + 1;
        if (more) fetch(jn);
        T jv[NC];
#pragma unroll
        for (int c = 0; c < NC; ++c) jv[c] = T(0);
        const int rel = jc - (b * kChunks + w * I);         // chunk jc against i chunk k of the wave: rel - k
        if (rel >= 0) {
#pragma unroll
            for (int k = 0; k < I; ++k)
#pragma unroll
                for (int c = 0; c < NC; ++c) p[k][c] = T(0);
            // rel >= I: the chunk after all of the wave's i chunks; otherwise the chunk is i chunk rel,
            // and only the i chunks up to it meet it
            if (rel >= I) fine_sweep<Op, I>(st[buf], s0, s1, iv, kc, addr, p, jv);
            else if (rel == 0) fine_sweep<Op, 0>(st[buf], s0, s1, iv, kc, addr, p, jv);
            else if (rel == 1) fine_sweep<Op, 1>(st[buf], s0, s1, iv, kc, addr, p, jv);
            else if constexpr (I > 2) {
                if (rel == 2) fine_sweep<Op, 2>(st[buf], s0, s1, iv, kc, addr, p, jv);
                else fine_sweep<Op, 3>(st[buf], s0, s1, iv, kc, addr, p, jv);
            }
#pragma unroll
            for (int k = 0; k < I; ++k)
#pragma unroll
                for (int c = 0; c < NC; ++c) acc[k][c].fold(p[k][c]);
        }
        // lane l holds the sums of j = l + s1
#pragma unroll
        for (int c = 0; c < NCP; ++c) jr[buf][w][(lane + s1) & (kWave - 1)][c] = c < NC ? jv[c < NC ? c : 0] : T(0);
        if (more) stage(buf ^ 1);
        // One barrier a sweep: the other buffers were last read in the sweep before, by waves that
        // have all reached this barrier's predecessor.
        __syncthreads();
        {
            void *dst = s0 == 0 ? a.jslot : a.carry;
            const int64_t at = s0 == 0 ? (int64_t)(fine_jslot(b, nb, kRows) + jc * kWave) * NCP : (int64_t)wg * kWave * NCP;
            for (int e = threadIdx.x; e < kWave * NCP; e += kFineWaves * kWave) {
                double v = (double)(&jr[buf][0][0][0])[e];
#pragma unroll
                for (int x = 1; x < kFineWaves; ++x) v += (double)(&jr[buf][x][0][0])[e];
                if (sizeof(T) == 8 || a.wide) ((double *)dst)[at + e] = v;
                else ((float *)dst)[at + e] = (float)v;
            }
        }
        if (!more || over) {
            const int64_t at = ((int64_t)(wg + b) * kRows + w * I * kWave + lane) * NCP;
            if (sizeof(T) == 8 || a.wide_i) put_sums<double, NC, NCP>((double *)a.islot + at, acc);
            else put_sums<float, NC, NCP>((float *)a.islot + at, acc);
            if (!more) return;
            ++b;
            load_block();
        }
        jc = jn;
        s0 = 0;
        buf ^= 1;
    }
}

// Column c of row r for each of 64 consecutive (row, column) pairs of a workgroup: the j slots of
// blocks 0 .. r's own (with the carry of a sweep that two workgroups shared), then the i sums of r's
// block by workgroup, the terms dealt out to the workgroup's eight waves (the smallest systems have
// few rows and up to a hundred terms a row), each wave adding its own in order, and the waves' sums
// merged in wave order, all in FP64 with compensation.  The operator's epilogue is separate for each
// column.
template <typename T, typename SJ, typename SI, int NCP>
__global__ __launch_bounds__(kRedWaves * kWave) void k_fine_reduce(FineLaunch a)
{
    __shared__ double part[kRedWaves][2][kWave];
    const int lane = lane_id();
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t t = (int64_t)blockIdx.x * kWave + lane;
    const int64_t r = t / NCP;
    const int c = (int)(t % NCP);
    const int jc = (int)(blockIdx.x / NCP);                     // 64 (row, column) pairs lie in one chunk
    const int ch = kFineWaves * a.ich, rows = ch * kWave;        // of a block
    const int b = jc / ch, nch = a.nch, per = a.per;
    const SJ *__restrict__ jslot = (const SJ *)a.jslot + t;
    const SJ *__restrict__ carry = (const SJ *)a.carry + (t - (int64_t)jc * kWave * NCP);
    const SI *__restrict__ islot = (const SI *)a.islot + (t - (int64_t)b * rows * NCP);
    NSum v;
    // fine_jslot(k), kRedWaves blocks a time
    int at = fine_jslot(w, a.nb, rows), step = rows * kRedWaves * (2 * (a.nb - w) - kRedWaves - 1) / 2;
    for (int k = w; k <= b; k += kRedWaves) {
        const int q = fine_begin(k, nch, ch) + 4 * (jc - k * ch);
        const int last = (q + 3) / per;
        v.add((double)jslot[(int64_t)at * NCP]);
        at += step;
        step -= rows * kRedWaves * kRedWaves;
        if (q / per != last) v.add((double)carry[(int64_t)last * kWave * NCP]);
    }
    const int w1 = (fine_begin(b + 1, nch, ch) - 1) / per;
#pragma unroll 4
    for (int u = fine_begin(b, nch, ch) / per + w; u <= w1; u += kRedWaves)
        v.add((double)islot[(int64_t)(u + b) * rows * NCP]);
    part[w][0][lane] = v.s;
    part[w][1][lane] = v.c;
    __syncthreads();
    if (w != 0) return;
#pragma unroll
    for (int u = 1; u < kRedWaves; ++u) v.merge(part[u][0][lane], part[u][1][lane]);
    if (r >= a.n) return;
    const double x = v.value();
    switch (a.op) {
    case FINE_FORCE: finish_column<T>(a.epi, a.next, r, c, x, a.pot != 0); return;
    case FINE_HVP:
        if (c < 3 && a.grad_pos) a.grad_pos[3 * r + c] = a.G * x;
        return;
    case FINE_LJC_ADJ:
        if (c < 3) {
            if (a.grad_pos) a.grad_pos[3 * r + c] = x;
        } else if (c < 6 && a.grad_params) {
            // the sums carry the records' factor 24 in eps (sigma) and sqrt(24) in se_j (epsilon)
            const double k = c == 3 ? a.qscale : (c == 4 ? 3.0 : 12.0 / __builtin_sqrt(24.0 * a.params[3 * r + 2]));
            a.grad_params[3 * r + c - 3] = k * x;
        }
        return;
    default:
        if (c < 3) a.out_acc[3 * r + c] = a.G * x;
        else if (c < 6) a.out_jerk[3 * r + c - 3] = a.G * x;
        else if (c == 6 && a.pot && a.out_pot) a.out_pot[r] = -a.G * x;
    }
}

static dim3 fine_grid(const FineLaunch &a) { return dim3((unsigned)((a.nwg + kSymXcds - 1) / kSymXcds * kSymXcds)); }
template <class Op, int PREC> static void fine_go4(const FineLaunch &a, hipStream_t s)
{
    hipLaunchKernelGGL((k_fine<Op, PREC, kFineIch4>), fine_grid(a), dim3(kFineWaves * kWave), 0, s, a);
}
template <class Op, int PREC, bool FOUR> static void fine_go(const FineLaunch &a, hipStream_t s)
{
    const dim3 grid = fine_grid(a), block(kFineWaves * kWave);
    if constexpr (FOUR)
        if (a.ich == kFineIch4) {
            fine_go4<Op, PREC>(a, s);
            return;
        }
    hipLaunchKernelGGL((k_fine<Op, PREC, kFineIch>), grid, block, 0, s, a);
}
template <class Op, bool FOUR> static void fine_go32(const FineLaunch &a, hipStream_t s)
{
    if (a.prec == P_KAHAN) fine_go<Op, P_KAHAN, FOUR>(a, s);
    else fine_go<Op, P_FP64ACC, FOUR>(a, s);
}
template <template <typename, bool> class Op, bool POT> static void fine_go_law(const FineLaunch &a, hipStream_t s)
{
    if (a.prec == P_FP64) fine_go<Op<double, POT>, P_FP64, true>(a, s);
    else fine_go32<Op<float, POT>, false>(a, s);
}
// FP32: the one-sided kernels' order of factors (and FP64 slots) where those would run, the coarser tiles'
// (FP32 slots, four i chunks) from their sizes on
template <bool POT> static void fine_go_gravity(const FineLaunch &a, hipStream_t s)
{
    if (a.prec == P_FP64) fine_go<GravOp<double, POT>, P_FP64, true>(a, s);
    else if (a.wide) fine_go32<GravOp<float, POT, true>, true>(a, s);
    else if (a.prec == P_KAHAN) fine_go4<GravOp<float, POT>, P_KAHAN>(a, s);
    else fine_go4<GravOp<float, POT>, P_FP64ACC>(a, s);
}
template <typename T, bool POT> using LjcLinOp = LjcOp<T, POT, LJC>;
template <typename T, bool POT> using LjcConstOp = LjcOp<T, POT, LJC_CONST>;
template <typename T, bool POT> using LjcSigOp = LjcOp<T, POT, LJC_SIG>;
template <bool POT> static void fine_go_force(const FineLaunch &a, hipStream_t s)
{
    switch (a.law) {
    case GRAVITY: return fine_go_gravity<POT>(a, s);
    case LJC: return fine_go_law<LjcLinOp, POT>(a, s);
    case LJC_CONST: return fine_go_law<LjcConstOp, POT>(a, s);
    default: return fine_go_law<LjcSigOp, POT>(a, s);
    }
}

bool fine_supported(int op, int law, int prec)
{
    const bool f32 = prec == P_KAHAN || prec == P_FP64ACC;
    switch (op) {
    case FINE_FORCE: return f32 || prec == P_FP64;
    case FINE_LJC_ADJ: return f32 && law == LJC;
    default: return f32 && law == GRAVITY;
    }
}

// FP64 forces and FP32 gravity's: elsewhere four chunks a wave cost more in balance than their moves
// save (FP32, 30,011 particles: LJC(linear) with energies 317 us with two chunks against 342, gravity's
// adjoint 314 against 319)
bool fine_has4(int op, int law, int prec)
{
    return fine_supported(op, law, prec) && op == FINE_FORCE && (prec == P_FP64 || law == GRAVITY);
}

// a launch description that does not match the work of n particles is refused, never launched
static bool fine_valid(const FineLaunch &a)
{
    if (!fine_supported(a.op, a.law, a.prec) || a.n <= 0 || a.n > kFineMaxN || (a.wide_i && !a.wide)) return false;
    if (a.ich != kFineIch && !(a.ich == kFineIch4 && fine_has4(a.op, a.law, a.prec))) return false;
    if (a.op == FINE_FORCE && a.law == GRAVITY && a.prec != P_FP64 && !a.wide && a.ich != kFineIch4) return false;
    const int ch = kFineWaves * a.ich;
    if (a.nch != (int)((a.n + kWave - 1) / kWave) || a.nb != (a.nch + ch - 1) / ch) return false;
    const int total = fine_begin(a.nb, a.nch, ch);
    return a.per >= 4 && a.nwg == (total + a.per - 1) / a.per && a.nwg <= kFineMaxWgs && a.rec && a.jslot &&
           a.islot && a.carry;
}

hipError_t launch_fine(const FineLaunch &a, hipStream_t s)
{
    if (!fine_valid(a)) return hipErrorInvalidValue;
    switch (a.op) {
    case FINE_FORCE: a.pot ? fine_go_force<true>(a, s) : fine_go_force<false>(a, s); break;
    case FINE_HVP: fine_go32<HvpOp, false>(a, s); break;
    case FINE_LJC_ADJ: fine_go32<LjcAdjOp, false>(a, s); break;
    default: a.pot ? fine_go32<JerkOp<true>, false>(a, s) : fine_go32<JerkOp<false>, false>(a, s);
    }
    return hipGetLastError();
}

template <int NCP> static void fine_reduce_go(const FineLaunch &a, dim3 grid, dim3 block, hipStream_t s)
{
    if (a.wide_i) hipLaunchKernelGGL((k_fine_reduce<float, double, double, NCP>), grid, block, 0, s, a);
    else if (a.wide) hipLaunchKernelGGL((k_fine_reduce<float, double, float, NCP>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((k_fine_reduce<float, float, float, NCP>), grid, block, 0, s, a);
}

hipError_t launch_fine_reduce(const FineLaunch &a, hipStream_t s)
{
    if (!fine_valid(a)) return hipErrorInvalidValue;
    const int cols = fine_cols(a.op);
    const dim3 grid((unsigned)(a.nch * cols)), block(kRedWaves * kWave);
    if (a.prec == P_FP64) hipLaunchKernelGGL((k_fine_reduce<double, double, double, 4>), grid, block, 0, s, a);
    else if (cols == 4) fine_reduce_go<4>(a, grid, block, s);
    else fine_reduce_go<8>(a, grid, block, s);
    return hipGetLastError();
}

}  // namespace nbk
