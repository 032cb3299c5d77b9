// Row groups: the forces of a small system in one launch (part of forward.hip).
//
// A few thousand particles are a few microseconds of arithmetic; the pack, the all-pairs kernel over
// j parts and the reduction of the parts then cost more in launches and in waiting for one another
// than in work.  Here one workgroup of 1,024 threads finishes R rows on its own: thread t takes row
// t mod R against the particles t / R, t / R + G, ... (G = 1024 / R), the records pass through LDS in
// tiles of 1,024, made from the caller's FP64 arrays as they are staged (or taken from packed records:
// a leapfrog step's), and the G partial sums of a row meet at the end, by lane exchange in a wave and
// through LDS across the sixteen waves.  R follows the size, so that n / R workgroups fill the 256 CUs;
// each reads all n particles, which L2 holds.  Bound by launch and memory latency: 7 us a leapfrog step
// of 1,280 LJC(linear) atoms (15 with three launches), 11 us for 4,096 stars (19), 13-14 us a call of
// nbody_forces from Python (20-21), most of it the caller's.
//
// Sums: a thread's terms (at most 128) are added in the law's type, everything after in FP64 over a
// tree of ten levels, in a fixed order.  (Compensation there brought nothing, 1.5e-16 either way in
// FP64 at 4,096 particles, and cost a microsecond.)
//
// A leapfrog step is one launch too: the finished row is kicked, drifted for the next step and written
// to the other of two record buffers, which the next launch reads.
namespace nbk {
namespace {

constexpr int kRowThreads = 1024;
constexpr int kRowTile = 1024;                           // records of an LDS tile, one a thread
constexpr int kRowMost = 32;                             // rows of a workgroup, at most

// The particle's record from the caller's arrays (pads past n)
template <typename R>
__device__ __forceinline__ void row_stage(const RowLaunch &a, int64_t i, R *to)
{
    constexpr int P = std::is_same<R, GravRec<decltype(R::x)>>::value ? 1 : 3;
    if (i < a.n) {
        const double *x = a.pos + 3 * i;
        store_rec(to, 0, x[0], x[1], x[2], a.params + P * i, a.qscale);
    } else {
        store_pad(to, 0);
    }
}

}  // namespace

template <int LAW, int PREC, bool POT, bool PACKED>
__global__ __launch_bounds__(kRowThreads) void k_rows(RowLaunch a)
{
    using T = typename RealOf<PREC>::type;
    using R = typename RecOf<T, LAW>::type;
    using IS = typename IStateOf<R>::type;
    // the tile, and after the last one the waves' row sums [16][rows][4]
    constexpr size_t kSums = (kRowThreads / kWave) * kRowMost * 4 * sizeof(double);
    __shared__ __align__(16) unsigned char lds[sizeof(R) * kRowTile > kSums ? sizeof(R) * kRowTile : kSums];
    R *tile = (R *)lds;
    const int tid = threadIdx.x, lane = lane_id(), wave = tid >> 6;
    const int rows = a.rows, groups = kRowThreads / rows, n = (int)a.n;
    const int row0 = blockIdx.x * rows;
    const int g = tid / rows;
    const int row = row0 + tid % rows;
    const int mine = row < n ? row : n - 1;
    const R *__restrict__ rec = (const R *)a.rec;
    const PairK<T> kc = PairK<T>{(T)a.eps2, (T)a.zeta[0], (T)a.zeta[1], (T)a.zeta[2], (T)a.zeta[3],
                                 (T)(3.0 * a.zeta[0]), (T)(2.0 * a.zeta[1])};
    IS is;
    R own, next;
    if constexpr (PACKED) {
        own = rec[mine];
        if (tid < n) next = rec[tid];
        else store_pad(&next, 0);
    } else {
        row_stage(a, mine, &own);
        row_stage(a, tid, &next);
    }
    load_i(&own, 0, is);
    T p[4] = {T(0), T(0), T(0), T(0)};
    for (int t0 = 0; t0 < n; t0 += kRowTile) {
        if (t0 > 0) __syncthreads();                     // the tile before has been read
        tile[tid] = next;
        const int64_t nx = t0 + kRowTile + tid;
        if (t0 + kRowTile < n) {
            if constexpr (PACKED) {
                if (nx < n) next = rec[nx];
                else store_pad(&next, 0);
            } else {
                row_stage(a, nx, &next);
            }
        }
        __syncthreads();
        const int count = n - t0 < kRowTile ? n - t0 : kRowTile;
        // the own pair is looked for only in the tile that holds the workgroup's rows (a multiple of
        // the row count, so they lie in one)
        if (row0 >= t0 && row0 < t0 + kRowTile) {
#pragma unroll 4
            for (int j = g; j < count; j += groups) pair<true, POT, LAW>(is, tile[j], kc, t0 + j == row, p);
        } else {
#pragma unroll 4
            for (int j = g; j < count; j += groups) pair<false, POT, LAW>(is, tile[j], kc, false, p);
        }
    }
    // lanes of a row: rows, 2 rows, ... apart
    double v[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) v[c] = (double)p[c];
    for (int m = rows; m < kWave; m <<= 1)
#pragma unroll
        for (int c = 0; c < (POT ? 4 : 3); ++c) v[c] += __shfl_xor(v[c], m);
    __syncthreads();
    double *sums = (double *)lds;                        // [16][rows][4]
    if (lane < rows)
#pragma unroll
        for (int c = 0; c < 4; ++c) sums[(wave * rows + lane) * 4 + c] = v[c];
    __syncthreads();
    // column c of row k, a thread each
    if (tid >= rows * 4) return;
    const int k = tid / 4, c = tid % 4;
    const int64_t r = row0 + k;
    if (r >= n) return;
    double x[kRowThreads / kWave];
#pragma unroll
    for (int w = 0; w < kRowThreads / kWave; ++w) x[w] = sums[w * rows * 4 + tid];
#pragma unroll
    for (int h = kRowThreads / kWave / 2; h > 0; h /= 2)
#pragma unroll
        for (int w = 0; w < h; ++w) x[w] += x[w + h];
    if constexpr (PACKED) {
        // the rest of the next step's record (its position is written column by column)
        if (a.next.on && c == 3) {
            R m = rec[r];
            T *to = (T *)((R *)a.next.rec + r);
            const T *from = (const T *)&m;
#pragma unroll
            for (int u = 3; u < (int)(sizeof(R) / sizeof(T)); ++u) to[u] = from[u];
        }
    }
    finish_column<T>(a.epi, a.next, r, c, x[0], POT);
}

template <int LAW, int PREC, bool POT> static void rows_go(const RowLaunch &a, dim3 grid, hipStream_t s)
{
    if (a.rec) hipLaunchKernelGGL((k_rows<LAW, PREC, POT, true>), grid, dim3(kRowThreads), 0, s, a);
    else hipLaunchKernelGGL((k_rows<LAW, PREC, POT, false>), grid, dim3(kRowThreads), 0, s, a);
}
template <int LAW, bool POT> static void rows_prec(const RowLaunch &a, dim3 grid, hipStream_t s)
{
    // FP32 terms are carried in FP64 from the thread's sum on, under either of the FP32 sums' names
    if (a.prec == P_FP64) rows_go<LAW, P_FP64, POT>(a, grid, s);
    else rows_go<LAW, P_FP64ACC, POT>(a, grid, s);
}
template <bool POT> static void rows_law(const RowLaunch &a, dim3 grid, hipStream_t s)
{
    switch (a.law) {
    case GRAVITY: return rows_prec<GRAVITY, POT>(a, grid, s);
    case LJC: return rows_prec<LJC, POT>(a, grid, s);
    case LJC_CONST: return rows_prec<LJC_CONST, POT>(a, grid, s);
    default: return rows_prec<LJC_SIG, POT>(a, grid, s);
    }
}

hipError_t launch_rows(const RowLaunch &a, hipStream_t s)
{
    if (a.n <= 0) return hipSuccess;
    // a power of two of rows, and no more terms a thread than its FP32 sum is meant for
    if (a.n > kRowsMaxN || a.rows < 1 || a.rows > kRowMost || (a.rows & (a.rows - 1)) != 0 || a.prec == P_PLAIN ||
        (!a.rec && (!a.pos || !a.params)) || (a.next.on && (!a.rec || a.next.rec == a.rec)))
        return hipErrorInvalidValue;
    const dim3 grid((unsigned)((a.n + a.rows - 1) / a.rows));
    if (a.pot) rows_law<true>(a, grid, s);
    else rows_law<false>(a, grid, s);
    return hipGetLastError();
}

}  // namespace nbk
