// Matrix-core variant of the resident Lloyd kernel: one workgroup runs the whole iteration of
// one (task, k) unit (paper Algorithm 1, K-means.run(s_Theta, k); Sec. 3.3), with the squared
// distance screened by v_mfma_f32_32x32x16_f16.
//
// Screen:  score(c, i) = |mu'_c|^2 - 2 x'_i . mu'_c   (x', mu' centred by an integer offset)
//   A (32 centroids x K) = [ hi(w) | lo(w) ],  w = fl32(-2 mu'),  hi = f16(w), lo = f16(w - hi)
//   B (K x 32 rows)      = [ x' ; x' ]        (x' is a small integer: exact in f16)
//   the last knob slot (unused when d < DK) carries the bias: B = 256 (16384 for two-byte knobs), A = hi/lo of |mu'_c|^2 / B;
//   with d = DK = 32 (SEP) the bias is a step of its own at the head of the chain, slots 0 and 1 of
//   sixteen: one instruction in five more, against twice the row registers and steps of 64-wide rows
// so every product is exact and only the fp32 accumulation and the 22-bit splits round.
//
// Centroid c sits in fragment row 8 (i / 4) + 4 (c & 1) + (i & 3), i = (c & 31) / 2, of m-tile c / 32,
// so that accumulator register i of lane half hh holds centroid 2 i + hh: a unit with k centroids
// has live scores in its first ceil(k / 2) registers only, and the epilogue walks live groups of
// four registers, not all sixteen.  Per 32-row tile: minimum over the live registers (v_min3),
// threshold = minimum + error bound of the row (a constant of the row for the whole unit: the
// bound uses the largest squared norm that a centroid can have, that of the farthest row), one
// subtract and one v_alignbit per score for the mask of centroids within the threshold.  If every
// row's mask is that of its label alone (rows in registers: the mask it had when the tile was last decided, and none of its rows was
// undecided then), every row keeps its label and nothing else happens for the tile.  Otherwise a
// row with a single centroid inside the threshold takes it; the others are queued per wave and
// their marked centroids are re-evaluated in double in the oracle's operation order.
// The matrix instructions of the next tile are issued between the epilogue pieces of the current
// one.  Centroids, labels, integer sums and counts stay in LDS; a row touches the sums only when its label changes (exact: the
// sums are integers), through a dense per-wave queue.  The rows (f16 B fragments) stay in registers for all passes
// (run_unit: tasks of at most 1024 rows, and where few units run also larger ones) or are fetched from packed tiles in every pass (run_unit_fetched), which lets two
// workgroups share a compute unit whatever the size of the task: 256 tasks x 4096 x 24, k = 1..64: 16.9 -> 12.7 ms a step.
//
// A pass that changes no label leaves the sums, hence the centroids, hence every later pass as
// they are: the iteration stops there and reports the state it has, which is what the remaining
// passes of the fixed-length iteration would reproduce.  The number of passes run is recorded.
#include <type_traits>

#include "cham_device.h"
#include "cham_internal.h"
#include "mfma_common.h"
#include "fetched_tiles.h"

namespace cham {

namespace {

// Rows a wave's queue holds (a tile fills at most 32): with few tiles per wave, 40 let two workgroups of
// 32-wide rows and 64 centroids share a compute unit (32 tasks x 1000 rows x 24 knobs, k = 2..48: 551 -> 458 us).
__host__ __device__ constexpr int rec_cap(int DK, int ntw) { return DK == 32 && ntw <= 4 ? 40 : kRecCap; }

// The variant that launch_mfma_sweep_t prefers to the one with twice the tiles per wave by the number of units alone: it
// sums the loss in its order.
constexpr bool paired_loss(int DK, int ntw) { return DK == 16 && ntw == 2; }

// A loss is summed by equal parts of the task's rows where the number of units chooses between rows in registers and rows fetched.
constexpr int kParts = 16;
__device__ __forceinline__ int rows_of_part(int nrows) { return nrows > 64 * kParts ? (nrows + 64 * kParts - 1) / (64 * kParts) * 64 : 64; }

// Total of the parts' sums, neighbours first: four roundings of full size, not fifteen (mean error of a loss of
// values in two parts against 80-bit sums, 1536 losses, 6.4e-17 / 8.5e-17; the vector kernel 7.3e-17).
__device__ __forceinline__ double sum_of_parts(const double *red, int n)
{
    double v[kParts];
#pragma unroll
    for (int p = 0; p < kParts; ++p) v[p] = p < n ? red[p] : 0.0;
#pragma unroll
    for (int step = 1; step < kParts; step *= 2)
#pragma unroll
        for (int p = 0; p < kParts; p += 2 * step) v[p] = v[p] + v[p + step];
    return v[0];
}

// LDS carve-up.  DK = padded knob count (16, 32, 48 or 64), KP = padded centroid count (32 or 64); SEP: the
// bias has fragments of its own.
template <int DK, bool SEP = false>
struct MfmaLds {
    double *mu64T;      // [DK][KP]   exact centroids, transposed
    double *red;        // [32]       partial sums of the loss
    float *bias;        // [KP]       upper bound of |mu - o|^2 per centroid (0 for padding rows)
    float *start;       // [KP]       initial scores in the order of the accumulator's registers (values in two parts)
    half8 *afrag;       // [KP/32][2*DK/16][64]  A fragments: hi parts then lo parts
    half8 *abias;       // [KP/32][64] A fragments of the bias step (SEP only; directly behind afrag)
    int *S;             // [KP][DK+1] integer cluster sums (row stride DK + 1: rows of different clusters fall into different banks)
    int *n;             // [KP]       cluster sizes
    int *dirty;         // [KP]       pass in which the cluster last changed
    float *ojf;         // [DK]       centring offsets
    unsigned long long *acc64;  // [2]  sum over the task's rows of |x|^2; sum over the clusters of floor(|S|^2 / n)
    int *stamp;         // [4]        [1] float bits of the largest squared row norm, [2], [3] rows that changed in an even / odd pass
    unsigned char *wave_base;   // per-wave regions follow
    __host__ __device__ static size_t wave_bytes(int ntw)
    {
        return ((size_t)rec_cap(DK, ntw) * (DK * 2 + 8 + 2) + 4 * 32 * 8 + (size_t)ntw * 32 * 6 + (size_t)ntw * 64 * 4 + 15) / 16 * 16;
    }
    // without the per-wave regions
    __host__ __device__ static size_t base_bytes(int KP)
    {
        size_t b = sizeof(double) * DK * KP + sizeof(double) * 32 + sizeof(float) * KP * 2;
        b += 16 * (size_t)(KP / 32) * (2 * DK / 16 + (SEP ? 1 : 0)) * 64;
        b += sizeof(int) * (size_t)KP * (DK + 1) + sizeof(int) * KP * 2 + sizeof(float) * DK + 32;
        return (b + 15) & ~(size_t)15;
    }
    __host__ __device__ static size_t bytes(int KP, int nwaves, int ntw) { return base_bytes(KP) + wave_bytes(ntw) * nwaves; }
    __device__ MfmaLds(unsigned char *base, int KP)
    {
        // plain offset arithmetic from the LDS base keeps every pointer provably in LDS
        size_t o = 0;
        mu64T = reinterpret_cast<double *>(base + o);  o += sizeof(double) * DK * KP;
        red = reinterpret_cast<double *>(base + o);    o += sizeof(double) * 32;
        bias = reinterpret_cast<float *>(base + o);    o += sizeof(float) * KP;
        start = reinterpret_cast<float *>(base + o);   o += sizeof(float) * KP;
        afrag = reinterpret_cast<half8 *>(base + o);   o += 16 * (size_t)(KP / 32) * (2 * DK / 16) * 64;
        abias = reinterpret_cast<half8 *>(base + o);   o += SEP ? 16 * (size_t)(KP / 32) * 64 : 0;
        S = reinterpret_cast<int *>(base + o);         o += sizeof(int) * (size_t)KP * (DK + 1);
        n = reinterpret_cast<int *>(base + o);         o += sizeof(int) * KP;
        dirty = reinterpret_cast<int *>(base + o);     o += sizeof(int) * KP;
        ojf = reinterpret_cast<float *>(base + o);     o += sizeof(float) * DK;
        stamp = reinterpret_cast<int *>(base + o);     o += 16;
        acc64 = reinterpret_cast<unsigned long long *>(base + o);  o += 16;
        o = (o + 15) & ~(size_t)15;
        wave_base = base + o;
    }
};

// Per-wave LDS region.  A queue of at most kCap rows (their centred knob values as f16, the
// candidate masks of both lane halves, the row index), used first for the rows the screen could
// not decide and then for the label changes of the pass, in batches; behind it the current label of
// every row, the labels the pass arrives at, the error bound of every row and, per (tile, lane),
// the mask the lane had when its tile was last decided.
template <int DK, int NTW>
struct WaveQueue {
    static constexpr int kPlanes = 1;
    static constexpr int kRows = NTW * 32;                  // rows a wave owns at most
    static constexpr int kCap = rec_cap(DK, NTW);
    static constexpr size_t kOffMask = (size_t)kCap * DK * 2;
    static constexpr size_t kOffPid = kOffMask + (size_t)kCap * 8;
    static constexpr size_t kOffFew = kOffPid + (size_t)kCap * 2;
    static constexpr size_t kOffLab = kOffFew + 4 * 32 * 8;
    static constexpr size_t kOffNew = kOffLab + (size_t)kRows;
    static constexpr size_t kOffEb = kOffNew + (size_t)kRows;
    static constexpr size_t kOffSeen = kOffEb + (size_t)kRows * 4;
    unsigned char *base;
    __device__ explicit WaveQueue(unsigned char *wb) : base(wb) {}
    __device__ _Float16 *rec_x() const { return reinterpret_cast<_Float16 *>(base); }                    // [kCap][DK]
    __device__ unsigned *rec_mask() const { return reinterpret_cast<unsigned *>(base + kOffMask); }      // [kCap][2]
    __device__ unsigned short *rec_pid() const { return reinterpret_cast<unsigned short *>(base + kOffPid); }
    __device__ double *few() const { return reinterpret_cast<double *>(base + kOffFew); }                 // [4][32] squares of one (row, centroid)
    __device__ unsigned char *lab() const { return base + kOffLab; }                                      // [kRows] current labels (0xFF: none)
    __device__ unsigned char *lab_new() const { return base + kOffNew; }                                  // [kRows] labels of the pass under way
    static __device__ __forceinline__ unsigned stored(unsigned c) { return c; }                           // centroid -> entry of the label tables
    static __device__ __forceinline__ unsigned centroid(unsigned v) { return v; }
    __device__ float *eb() const { return reinterpret_cast<float *>(base + kOffEb); }                     // [kRows] screen bound of the row
    __device__ unsigned *seen() const { return reinterpret_cast<unsigned *>(base + kOffSeen); }           // [tiles][64] mask at the last decision
};

// Row-major f16 copy of X (one row = DK halfs, padded knobs zero): a lane fetches the eight knobs
// of a B fragment with one 16-byte load.
// Two-byte knobs take this path only when every value is below 2048 (integers up to 2048 are
// exact in f16): a larger value sets *too_large, which makes the sweep kernel report status 4.
template <int DK, typename XT>
__global__ void pack_rows_kernel(const XT *__restrict__ X, int64_t ld, int d, int64_t n_rows,
                                 _Float16 *__restrict__ xh, int *too_large)
{
    const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= n_rows) return;
    unsigned top = 0;
#pragma unroll
    for (int g = 0; g < DK / 8; ++g) {
        half8 v;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int j = 8 * g + i;
            const unsigned xv = j < d ? (unsigned)X[(int64_t)j * ld + r] : 0u;
            top = xv > top ? xv : top;
            v[i] = (_Float16)(float)xv;
        }
        *reinterpret_cast<half8 *>(xh + r * DK + 8 * g) = v;
    }
    if (sizeof(XT) == 2 && top >= 2048u) *too_large = 1;
}

// Apply queued label changes of this wave to the integer sums and counts: 256 / DK queued rows
// per step, one lane per (row, group of 4 knobs).  Entry word: cur | prev << 8, prev = 0xFF for a
// row that had no label yet.
template <int DK, typename Queue>
__device__ __forceinline__ void apply_changes(const Queue &Q, int cnt, int *S, int *n, int *dirty,
                                              const float *ojf, int d, int stamp)
{
    constexpr int LPR = DK / 4;              // lanes per row
    constexpr int EPI = 64 / LPR;            // rows per step
    const int lane = threadIdx.x & 63;
    const int j0 = 4 * (lane % LPR);
    const float4 o4 = *reinterpret_cast<const float4 *>(ojf + j0);
    const float of[4] = {o4.x, o4.y, o4.z, o4.w};
    const bool on = j0 < d && lane < LPR * EPI;      // (twelve lanes per row leave four idle)
#pragma unroll 2
    for (int e0 = 0; e0 < cnt; e0 += EPI) {
        const int e = e0 + lane / LPR;
        if (e < cnt && on) {
            const unsigned w = Q.rec_mask()[e];
            typedef _Float16 half4 __attribute__((ext_vector_type(4)));
            const half4 xq = *reinterpret_cast<const half4 *>(Q.rec_x() + (size_t)e * DK + j0);
            const int cur = w & 0xFF, prev = (w >> 8) & 0xFF;
            const bool first = prev == 0xFF;
            int *sc = S + cur * (DK + 1) + j0;
            int *sp = S + (first ? cur : prev) * (DK + 1) + j0;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (j0 + i < d) {
                    const int xi = (int)((float)xq[i] + of[i]);
                    atomicAdd(sc + i, xi);
                    if (!first) atomicSub(sp + i, xi);
                }
            }
            if (j0 == 0) {
                atomicAdd(&n[cur], 1);
                dirty[cur] = stamp;
                if (!first) {
                    atomicSub(&n[prev], 1);
                    dirty[prev] = stamp;
                }
            }
        }
    }
    __builtin_amdgcn_wave_barrier();
}

// As packed_sums, from the knob-major byte matrix: 64 consecutive rows = 64 bytes per lane and group of 128 rows, so that a wave uses
// up the lines it touches (the labels are taken in the same order).  Needs 16-byte aligned rows (xw, ld) and reads whole runs of 64
// rows: the caller makes sure that the last run of the task still lies inside the matrix (rows of other tasks or padding read
// there meet the label 0xFF, which matches no centroid).  NG = runs of 64 rows a wave owns at most; the loads of 256 rows are
// under way at any time.  SEP: every knob row is in use, so the sizes are counted from the labels.
template <int DK, int NG, bool SEP, typename Queue>
__device__ __forceinline__ void full_sums(const Queue &Q, int *S, int *n, const uint8_t *xw, int64_t ld,
                                          int d, int k, int rows_here, int lane)
{
    constexpr int W = NG % 2 == 0 ? 2 : 1;                  // a lane's 32-row pieces per group of 64 * W rows
    constexpr int kGroups = NG / W;
    constexpr int kDepth = kGroups < 4 / W ? kGroups : 4 / W;
    const int m32 = lane & 31, kh = lane >> 5;
    const bool two = k > 32;
    const bool knob = m32 < d;
    const uint8_t *xp = xw + (int64_t)(knob ? m32 : 0) * ld + 32 * W * kh;
    const unsigned char *lp = Q.lab() + 32 * W * kh;
    const int c4a = (int)(Queue::stored(m32) * 0x01010101u), c4b = (int)(Queue::stored(m32 + 32) * 0x01010101u);
    int16v acc0, acc1;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        acc0[i] = 0;
        acc1[i] = 0;
    }
    const int runs = (rows_here + 63) >> 6;

    // this lane's bytes of group g (zero where the knob or the run of 64 rows does not exist)
    auto fetch = [&](int g, int4v (&w)[2 * W]) {
#pragma unroll
        for (int i = 0; i < 2 * W; ++i) w[i] = int4v{0, 0, 0, 0};
        if (knob && W * g + (W == 2 ? kh : 0) < runs) {
#pragma unroll
            for (int i = 0; i < 2 * W; ++i) w[i] = *reinterpret_cast<const int4v *>(xp + 64 * W * g + 16 * i);
        }
    };
    int4v w[kDepth][2 * W];
#pragma unroll
    for (int g = 0; g < kDepth; ++g) fetch(g, w[g]);
#pragma unroll
    for (int g = 0; g < kGroups; ++g) {
        if (W * g < runs) {
#pragma unroll
            for (int i = 0; i < 2 * W; ++i) {
                const int4v A = w[g % kDepth][i] ^ (int)0x80808080;
                const int4v l = *reinterpret_cast<const int4v *>(lp + 64 * W * g + 16 * i);
                acc0 = __builtin_amdgcn_mfma_i32_32x32x32_i8(A, members<false>(l, c4a), acc0, 0, 0, 0);
                if (two) acc1 = __builtin_amdgcn_mfma_i32_32x32x32_i8(A, members<false>(l, c4b), acc1, 0, 0, 0);
            }
            if (g + kDepth < kGroups) fetch(g + kDepth, w[g % kDepth]);
        }
    }
    // accumulator register i of lane (c, kh) = knob (i & 3) + 8 (i >> 2) + 4 kh of centroid c (or 32 + c)
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int m = (i & 3) + 8 * (i >> 2) + 4 * kh;
        if (m < d) {
            if (m32 < k) atomicAdd(&S[m32 * (DK + 1) + m], -(acc0[i] >> 7));
            if (two && m32 + 32 < k) atomicAdd(&S[(m32 + 32) * (DK + 1) + m], -(acc1[i] >> 7));
        }
        if (!SEP && i == 15 && kh == 1) {                              // knob row 31: 2^14 per row of the cluster
            if (m32 < k) atomicAdd(&n[m32], acc0[i] >> 14);
            if (two && m32 + 32 < k) atomicAdd(&n[m32 + 32], acc1[i] >> 14);
        }
    }
    if (SEP) {
        for (int e = lane; e < rows_here; e += 64) {
            const unsigned v = Q.lab()[e];
            if (v < 64u) atomicAdd(&n[Queue::centroid(v)], 1);       // (k <= 64)
        }
    }
}

// Centroid update for the clusters touched in this pass, all threads: item (c, q) owns knobs
// 4q..4q+3 of centroid c: mean = (double)S / (double)n, then the f16 hi/lo fragments of
// w = -2 (mu - o) (one 8-byte store each).  The DK/4 items of a centroid sit in adjacent lanes and
// add up |mu - o|^2 among themselves; the last of them owns the bias slot (knob slot DK - 1, or with
// SEP slots 0 and 1 of the bias step) and stores the sum / 256 there as hi/lo, and its rounded-up value for the error bound.
// all: fragments from the centroids as they are (no sums yet); starts from the caller may lie anywhere, so the
// operands are clamped (a mean of rows is always in range).  raw: the sums were rebuilt by
// full_sums or packed_sums for every cluster (each still off by raw_offset n): every cluster is updated, and the sums
// are left either corrected (the next pass applies label changes to them) or, with zero_after,
// cleared together with the sizes (the next pass rebuilds them).
// PL = 2 (knob values in two parts, below): operands and scores are a quarter of the full ones, so that w fits f16 for any
// two-byte value, and the bias is an initial score in fp32.
constexpr float kTwoPartScale = 0.25f;
template <int DK, bool BYTE_KNOBS, bool SEP, int PL = 1>
__device__ __forceinline__ void update_centroids(const MfmaLds<DK, SEP> &U, int k, int KP, int d, int stamp, bool all,
                                                 bool raw = false, bool zero_after = false)
{
    constexpr int NS = DK / 16, NS2 = 2 * NS, QN = DK / 4;
    constexpr float kBiasScale = bias_scale(BYTE_KNOBS);
    constexpr int LQ = QN == 12 ? 16 : QN;              // lanes per centroid: a power of two for the exchanges
    typedef _Float16 half4 __attribute__((ext_vector_type(4)));
    const int items = k * LQ;
    for (int base = 0; base < items; base += blockDim.x) {      // uniform trip count: every lane shuffles
        const int item = base + (int)threadIdx.x;
        const int c = item / LQ, q = item % LQ;
        bool act = item < items && q < QN;
        int cnt = 0;
        if (act) {
            cnt = U.n[c];
            if (!all && ((!raw && U.dirty[c] != stamp) || cnt == 0)) act = false;   // an empty cluster keeps its centroid
        }
        if (!zero_after && !__any(act)) continue;           // none of this wave's clusters was touched
        half4 hi4 = {(_Float16)0.0f, (_Float16)0.0f, (_Float16)0.0f, (_Float16)0.0f};
        half4 lo4 = hi4;
        double b = 0.0;
        bool clamped = false;
        // The mean S / n with one division per item instead of one per knob: r = fl(1 / n), then
        // q0 = fl(S r), rem = S - q0 n (exact in one fused operation), fl(q0 + rem r).  That this
        // equals the correctly rounded quotient fl(S / n) for every count 1 <= n <= 4096 and every
        // integer sum 0 <= S <= 255 n (the whole domain of this kernel: byte knobs, tasks of at most
        // 4096 rows) is checked exhaustively on the CPU (quotient_check.c, run by the test suite).
        const double dn = (double)(cnt > 0 ? cnt : 1);
        const double rn = 1.0 / dn;
        if (act && 4 * q < d) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int j = 4 * q + i;
                double mu = U.mu64T[(size_t)j * KP + c];
                if (!all && j < d) {
                    int sv = U.S[c * (DK + 1) + j];
                    if (raw) {
                        sv -= raw_offset(BYTE_KNOBS) * cnt;
                        U.S[c * (DK + 1) + j] = sv;
                    }
                    const double sd = (double)sv;
                    if (BYTE_KNOBS) {
                        const double q0 = sd * rn;
                        const double rem = __builtin_fma(-q0, dn, sd);
                        mu = __builtin_fma(rem, rn, q0);
                    } else {
                        mu = sd / dn;             // (sums of two-byte knobs lie outside the checked domain)
                    }
                    U.mu64T[(size_t)j * KP + c] = mu;
                }
                const double m = j < d ? mu - (double)U.ojf[j] : 0.0;
                b = __builtin_fma(m, m, b);
                float w = (float)((PL == 2 ? -2.0 * kTwoPartScale : -2.0) * m);
                if (PL == 2 && all && !(__builtin_fabsf(w) <= kHalfMax)) clamped = true;
                if (all) w = __builtin_amdgcn_fmed3f(w, -kHalfMax, kHalfMax);
                const _Float16 hi = (_Float16)w;
                hi4[i] = hi;
                lo4[i] = (_Float16)(w - (float)hi);
            }
        }
        b = b + dpp_xor_f64<1>(b);
        b = b + dpp_xor_f64<2>(b);
        if (LQ >= 8) b = b + dpp_xor_f64<4>(b);
        if (LQ == 16) b = b + dpp_xor_f64<8>(b);
        if (act && (4 * q < d || q == QN - 1)) {
            if (q == QN - 1) {
                float bs = (float)b * (1.0f / kBiasScale);
                if (all) bs = __builtin_fminf(bs, kHalfMax);
                const _Float16 bhi = (_Float16)bs;
                const _Float16 blo = (_Float16)(bs - (float)bhi);
                if constexpr (PL == 2) {
                    float st = (float)b * kTwoPartScale;
                    if (all) st = __builtin_fminf(st, kFarScore);
                    U.start[(c >> 5) * 32 + 16 * (c & 1) + ((c & 31) >> 1)] = st;
                } else if constexpr (SEP) {
                    typedef _Float16 half2v __attribute__((ext_vector_type(2)));
                    *reinterpret_cast<half2v *>(U.abias + (c >> 5) * 64 + frag_row(c)) = half2v{bhi, blo};
                } else {
                    hi4[3] = bhi;
                    lo4[3] = blo;
                }
                U.bias[c] = __double2float_ru(b) * 1.0000005f;
            }
            const int mt = c >> 5, m32 = frag_row(c);
            const int g = q >> 1, kh = g & 1, fstep = g >> 1, sub = q & 1;
            half4 *fh = reinterpret_cast<half4 *>(U.afrag + (mt * NS2 + fstep) * 64 + 32 * kh + m32) + sub;
            half4 *fl = reinterpret_cast<half4 *>(U.afrag + (mt * NS2 + NS + fstep) * 64 + 32 * kh + m32) + sub;
            *fh = hi4;
            *fl = lo4;
            // (beyond the range of the operands: behind the bound's own value, which a lane of this wave has stored)
            if (PL == 2 && clamped) atomicMax(reinterpret_cast<int *>(U.bias + c), __float_as_int(kFarNorm));
        }
        if (zero_after && item < items) {
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (4 * q + i < d) U.S[c * (DK + 1) + 4 * q + i] = 0;
            // every item of a cluster sits in this wave and has read the size by now
            __builtin_amdgcn_wave_barrier();
            if (q == 0) U.n[c] = 0;
        }
    }
}

// Everything one workgroup does for its unit.  Units with more than 32 centroids use two 32-row
// m-tiles per row tile; otherwise the two accumulators alternate between row tiles.
template <int DK, int NTW, typename XT, bool SEP>
__device__ __forceinline__ void run_unit(const SweepArgs &a, unsigned char *smem, int ki, int t, int k)
{
    constexpr bool kByteKnobs = sizeof(XT) == 1;
    constexpr double kMaxValue = kByteKnobs ? 255.0 : 2047.0;
    constexpr float kBiasScale = bias_scale(kByteKnobs);
    // 48- and 64-wide rows: k <= 32
    constexpr bool kAllowTwo = DK <= 32;
    const XT *X = reinterpret_cast<const XT *>(a.X);
    const bool two = kAllowTwo && k > 32;
    constexpr int NS = DK / 16;          // distinct B fragments per row
    constexpr int NS2 = 2 * NS;          // chained instructions per 32x32 tile, without the bias step
    constexpr int NSA = NS2 + (SEP ? 1 : 0);   // ... with it
    constexpr int CH = NS2 == 6 ? 4 : 16 / NS2;   // scores handled between two matrix instructions
    const int KP = a.kmax > 32 ? 64 : 32;
    MfmaLds<DK, SEP> U(smem, KP);

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nwaves = blockDim.x >> 6;
    const int n32 = lane & 31;           // row within a 32-row tile
    const int h = lane >> 5;             // which half of the knob slots / centroid rows this lane holds
    // The phases of a pass take the lane index through this: values derived from it (addresses into
    // the wave's tables) are then computed where they are used instead of living, or being spilled,
    // across the whole iteration next to the 128 registers of rows.
    const int lane_id = lane;
    auto opaque = [](int v) {
        asm volatile("" : "+v"(v));
        return v;
    };

    const int d = a.d;
    const int64_t r0 = a.task_off[t], r1 = a.task_off[t + 1];
    const int nrows = (int)(r1 - r0);
    const int64_t slot = (int64_t)t * a.n_k + ki;
    const int64_t crow = (int64_t)t * a.Ksum + a.koff[ki];
    uint8_t *labrow = a.labbuf + (int64_t)ki * a.ld;

    constexpr bool kShortQueue = WaveQueue<DK, NTW>::kCap < kRecCap;     // filled up to the row, at the price of some registers
    WaveQueue<DK, NTW> Q(U.wave_base + MfmaLds<DK, SEP>::wave_bytes(NTW) * wave);
    const int wave_row0 = wave * NTW * 32;                 // first row (task-relative) of this wave
    const bool wave_live = wave_row0 < nrows;              // the wave owns at least one row

    // Live accumulator registers: centroids 2 i + hh sit in register i, so a tile of kk centroids has
    // scores in its first ceil(kk / 2) registers; they are walked in groups of four.
    const int kk_last = two ? k - 32 : k;                  // centroids in the last (or only) m-tile
    const int lregs = ((kk_last + 1) / 2 + 3) & ~3;        // 4, 8, 12 or 16

    // Without SEP the last knob slot of the fragments is reserved (d <= DK - 1): it carries the bias (256
    // in B, |mu'|^2 / 256 as hi/lo in A).
    constexpr int bstep = NS - 1, bhalf = 1, belem = 7;
    constexpr int kFullDivisor = 8;

    // ---- this lane's rows as B fragments (kept in registers for every pass).  The loads are issued
    // first (raw knob values; they are centred once the offsets are known) so that they are under way
    // during the set-up of the unit's state.
    const _Float16 *xh_wave = reinterpret_cast<const _Float16 *>(a.xh) + (r0 + (wave_live ? wave_row0 : 0)) * DK;
    half8 B[NTW][NS];
#pragma unroll
    for (int nt = 0; nt < NTW; ++nt) {
        const bool live = wave_live && (wave_row0 + nt * 32 + n32) < nrows;
        const int64_t prow = live ? (int64_t)(nt * 32 + n32) : 0;         // always a row of this task
#pragma unroll
        for (int f = 0; f < NS; ++f) {
            half8 v;
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] = (_Float16)0.0f;
            if (nrows > 0) v = *reinterpret_cast<const half8 *>(xh_wave + prow * DK + 16 * f + 8 * h);
            B[nt][f] = v;
        }
    }

    // ---- set-up
    for (int e = tid; e < DK * KP; e += blockDim.x) U.mu64T[e] = 0.0;
    for (int e = tid; e < KP * (DK + 1); e += blockDim.x) U.S[e] = 0;
    for (int c = tid; c < KP; c += blockDim.x) {
        U.n[c] = 0;
        U.dirty[c] = -1;
    }
    for (int c = tid; c < KP; c += blockDim.x) U.bias[c] = 0.0f;
    {
        half8 z;
#pragma unroll
        for (int i = 0; i < 8; ++i) z[i] = (_Float16)0.0f;
        for (int e = tid; e < (KP / 32) * NSA * 64; e += blockDim.x) U.afrag[e] = z;      // (abias included)
    }
    __syncthreads();
    // padding centroid rows (beyond k) carry a huge bias so that they never win
    for (int c = k + tid; c < KP; c += blockDim.x) {
        _Float16 *bslot = SEP ? reinterpret_cast<_Float16 *>(U.abias + (c >> 5) * 64 + frag_row(c))
                              : reinterpret_cast<_Float16 *>(U.afrag + ((c >> 5) * NS2 + bstep) * 64 + 32 * bhalf + frag_row(c)) + belem;
        bslot[0] = (_Float16)kHalfMax;
    }
    if (tid == 0) {
        U.stamp[0] = 0;           // (unused)
        U.stamp[1] = 0;           // float bits of the largest squared norm of a centred row
        U.stamp[2] = 0;           // rows that changed their label in an even pass
        U.stamp[3] = 0;           // ... in an odd pass
        U.acc64[0] = 0ull;
        U.acc64[1] = 0ull;
    }
    for (int e = tid; e < k * d; e += blockDim.x) {
        const int c = e / d, j = e % d;
        double v;
        if (a.init_mode == 0) {
            const int row = a.init_rows[(int64_t)t * a.kmax + c];
            v = (double)X[(int64_t)j * a.ld + r0 + row];
        } else {
            v = a.init_centroids[(crow + c) * d + j];
        }
        U.mu64T[(size_t)j * KP + c] = v;
    }
    __syncthreads();
    {
        // centring offset of knob j: the rounded mean of the starting centroids (any integer would do:
        // it only keeps the centred magnitudes small); eight lanes per knob
        const int part = tid & 7;
        for (int j = tid >> 3; j < DK; j += blockDim.x >> 3) {       // (uniform within a wave: every lane shuffles)
            double s = 0.0;
            if (j < d)
                for (int c = part; c < k; c += 8) s += U.mu64T[(size_t)j * KP + c];
            s = s + dpp_xor_f64<1>(s);
            s = s + dpp_xor_f64<2>(s);
            s = s + dpp_xor_f64<4>(s);
            if (part == 0) {
                float o = 0.0f;
                if (j < d) {
                    double m = rint(s / (double)k);
                    m = m < 0.0 ? 0.0 : (m > kMaxValue ? kMaxValue : m);
                    o = (float)m;
                }
                U.ojf[j] = o;
            }
        }
    }
    __syncthreads();
    update_centroids<DK, kByteKnobs, SEP>(U, k, KP, d, 0, true);

    // ---- centre the rows; on the way, the sum of |x|^2 over the task's rows as an integer (for the loss
    // at a fixed point, see the end) and the squared norm of every centred row (for the error bound).
    // Squares are summed two at a time into fp32 (v_dot2): the raw values are integers below 256, so
    // a lane's sum per tile stays below 16 * 255^2 < 2^24 and is exact.
    {
        typedef _Float16 half2v __attribute__((ext_vector_type(2)));
        typedef unsigned uint4v __attribute__((ext_vector_type(4)));
        auto sumsq = [](const half8 &v, float acc) {
            const uint4v w = __builtin_bit_cast(uint4v, v);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const unsigned we = w[e];
                const half2v p = __builtin_bit_cast(half2v, we);
                acc = __builtin_amdgcn_fdot2(p, p, acc, false);
            }
            return acc;
        };
        float x2row[NTW];                // squared norm of this lane's centred row of every tile
        half8 off8[NS];
        uint4v keep[NS];                 // all ones in the halves of the knobs that exist
#pragma unroll
        for (int f = 0; f < NS; ++f) {
#pragma unroll
            for (int i = 0; i < 8; ++i) off8[f][i] = (_Float16)U.ojf[16 * f + 8 * h + i];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int j = 16 * f + 8 * h + 2 * e;
                keep[f][e] = (j < d ? 0x0000FFFFu : 0u) | (j + 1 < d ? 0xFFFF0000u : 0u);
            }
        }
        unsigned q2 = 0;
        float xmax = 0.0f;
#pragma unroll
        for (int nt = 0; nt < NTW; ++nt) {
            const bool live = wave_live && (wave_row0 + nt * 32 + n32) < nrows;
            float raw = 0.0f, part = 0.0f;
#pragma unroll
            for (int f = 0; f < NS; ++f) {
                if (kByteKnobs) raw = sumsq(B[nt][f], raw);
                const half8 c8 = B[nt][f] - off8[f];
                uint4v w = __builtin_bit_cast(uint4v, c8) & keep[f];
#pragma unroll
                for (int e = 0; e < 4; ++e) w[e] = live ? w[e] : 0u;
                half8 cv = __builtin_bit_cast(half8, w);
                part = sumsq(cv, part);
                // the bias slot: a constant for every live row (after the norm, which excludes it)
                if (!SEP && f == bstep && live && h == bhalf) cv[belem] = (_Float16)kBiasScale;
                B[nt][f] = cv;
            }
            if (kByteKnobs) q2 += live ? (unsigned)raw : 0u;
            part = part + __shfl_xor(part, 32, 64);
            x2row[nt] = part;
            xmax = __builtin_fmaxf(xmax, part);
        }
        // the wave's sum of |x|^2 (at most 512 rows * 31 * 255^2 < 2^31) -> the unit's 64-bit sum
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) q2 += (unsigned)__shfl_xor((int)q2, off, 64);
        if (lane_id == 0 && q2) atomicAdd(&U.acc64[0], (unsigned long long)q2);
        xmax = wave_max_nonneg(xmax);
        if (lane == 0) atomicMax(&U.stamp[1], __float_as_int(xmax));     // non-negative floats order like integers
        __syncthreads();
        // Largest squared norm a centred centroid can take during the iteration: every later centroid
        // is a mean of rows (inside their convex hull) or stays where it started.
        float m2 = wave_max_nonneg(lane < k ? U.bias[lane] : 0.0f);
        m2 = __builtin_fmaxf(m2, __int_as_float(U.stamp[1])) * 1.000001f;
        // starts beyond the range of the screen (their operands are clamped): every centroid is a candidate of every row
        if (!(m2 <= max_screened(kByteKnobs))) m2 = kFarNorm;
#pragma unroll
        for (int nt = 0; nt < NTW; ++nt)
            if (h == 0) Q.eb()[nt * 32 + n32] = mfma_bound<NSA, kByteKnobs>(x2row[nt], m2);
    }
    __builtin_amdgcn_wave_barrier();

    // no row has a label yet
    for (int e = lane; e < WaveQueue<DK, NTW>::kRows; e += 64) Q.lab()[e] = 0xFF;
    __builtin_amdgcn_wave_barrier();

    const int rows_wave = __builtin_amdgcn_readfirstlane(nrows - wave_row0);   // rows from this wave's first row to the task's end
    uint32_t force_tiles = 0xFFFFFFFFu;  // tiles to decide whatever their masks say: all at first, later those with undecided rows
    int passes_run = 0;
    bool at_fixed_point = false;         // the last pass run moved no row: every centroid is the mean of its cluster
    // A pass after one that moved many rows rebuilds the sums from the labels on the matrix cores
    // instead of applying the changes one by one; the first pass (every row is new) always does.
    const uint8_t *xw = a.X + r0 + (wave_live ? wave_row0 : 0);
    const bool x_aligned = kByteKnobs &&                              // (the rebuild reads the byte matrix)
                           ((reinterpret_cast<uintptr_t>(a.X) | (uintptr_t)a.ld | (uintptr_t)r0) & 15) == 0 &&
                           r0 + ((nrows + 63) & ~63) <= a.ld;       // ... and its last group of 64 rows lies inside the matrix
    bool full_mode = x_aligned;
    const int full_above = nrows / kFullDivisor;      // changed rows of a pass above which the next one rebuilds
    bool traced_last = false;

    // lanes of tile nt (as a 32-bit mask over the row index within the tile) whose row belongs to the task
    auto live_rows = [&](int nt) -> uint32_t {
        int left = rows_wave - 32 * nt;
        left = left < 0 ? 0 : (left > 32 ? 32 : left);
        return left == 32 ? 0xFFFFFFFFu : ((1u << left) - 1u);
    };
    // This lane's B fragments of tile nt, nt known at run time only (the same for the whole wave): one
    // branch per tile around a register copy, so that the code that follows exists once, not per tile.
    auto rows_of_tile = [&](int nt, half8 (&bt)[NS]) {
#pragma unroll
        for (int n = 0; n < NTW; ++n) {
            if (nt == n) {
#pragma unroll
                for (int f = 0; f < NS; ++f) {
                    bt[f] = B[n][f];
                    asm volatile("" : "+v"(bt[f]));      // keeps the copy under its branch
                }
            }
        }
    };

    // Exact loss of the current labels from the rows in registers: (x - mu)^2 in double over the knobs
    // a lane holds (x = centred value + offset, exact), the two lanes of a row and all rows added up
    // afterwards; the sums of the waves land in U.red[slot8 .. slot8 + n_parts).
    // kPaired: the number of units chose this number of tiles per wave over twice it.  A loss is the same in
    // a whole sweep and in a chunk of it, which have different numbers of units: the terms of an odd wave go
    // through its idle queue to the wave before it, whose lanes add up what they would with twice the tiles.
    constexpr bool kPaired = paired_loss(DK, NTW);
    static_assert(!kPaired || (size_t)NTW * 64 * sizeof(double) <= WaveQueue<DK, NTW>::kOffMask, "the terms fit the queue's rows");
    // kCanPart: the sums of the task's parts (kParts, of 64 or 128 rows, so that a wave has whole ones), as run_unit_fetched adds them up.
    constexpr bool kCanPart = NTW == 8 || (DK > 32 && NTW == 4);
    const bool parted = kCanPart && (NTW == 8 || a.loss_parts != 0);
    const int part_rows = parted ? rows_of_part(nrows) : NTW * 32;
    const int all_parts = parted ? nwaves * NTW * 32 / part_rows : (kPaired ? (nwaves + 1) / 2 : nwaves);
    const int n_parts = all_parts < kParts ? all_parts : kParts;
    auto wave_loss = [&](int first_slot) {
        double part = 0.0;
        const bool handed_over = kPaired && (wave & 1) != 0;
        const int lane = opaque(lane_id), n32 = lane & 31, h = lane >> 5;
        // a total in the fixed order lane ^ 32, 16, ..., 1 (partner indices from the local lane index)
        auto put = [&](double ws, int place) {
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) {
                const long long b = __double_as_longlong(ws);
                const int plo = __builtin_amdgcn_ds_bpermute((lane ^ off) << 2, (int)(b & 0xFFFFFFFFll));
                const int phi = __builtin_amdgcn_ds_bpermute((lane ^ off) << 2, (int)(b >> 32));
                ws = ws + __longlong_as_double(((long long)phi << 32) | (unsigned int)plo);
            }
            if (lane == 0 && place < kParts) U.red[first_slot + place] = ws;
        };
        double ends[NTW / 2] = {};                                  // sums up to every second tile
        auto ends_part = [&](int nt) { return ((nt + 1) * 32 & (part_rows - 1)) == 0; };
        if (wave_live) {
            float of[NS][8];
#pragma unroll
            for (int f = 0; f < NS; ++f)
#pragma unroll
                for (int i = 0; i < 8; ++i) of[f][i] = U.ojf[16 * f + 8 * h + i];
            // (unrolled over the tiles: runs once per unit, and the loads of several tiles overlap)
#pragma unroll
            for (int nt = 0; nt < NTW; ++nt) {
                const half8 (&bt)[NS] = B[nt];
                const uint32_t lab = Q.lab()[nt * 32 + n32];
                const bool live = lab != 0xFFu;
                const double *mc = U.mu64T + (live ? lab : 0u) + (size_t)(8 * h) * KP;
                // the centroid's knobs first, all loads under way together, then the sum in knob order
                double mu[NS][8];
#pragma unroll
                for (int f = 0; f < NS; ++f)
#pragma unroll
                    for (int i = 0; i < 8; ++i) mu[f][i] = mc[(size_t)(16 * f + i) * KP];
                double s = 0.0;
#pragma unroll
                for (int f = 0; f < NS; ++f)
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        float xf = (float)bt[f][i] + of[f][i];
                        if (!SEP && f == bstep && i == belem) xf = h == bhalf ? 0.0f : xf;     // the bias slot is no knob
                        const double tq = (double)xf - mu[f][i];
                        s = s + tq * tq;
                    }
                if (handed_over) reinterpret_cast<double *>(Q.rec_x())[nt * 64 + lane] = live ? s : 0.0;
                else part = part + (live ? s : 0.0);
                if (kCanPart && (nt & 1)) {
                    ends[nt / 2] = part;
                    part = ends_part(nt) ? 0.0 : part;
                }
            }
        }
        if constexpr (kPaired) {
            __syncthreads();
            if (!handed_over && wave_row0 + NTW * 32 < nrows) {          // the next wave owns rows
                const double *terms = reinterpret_cast<const double *>(U.wave_base + MfmaLds<DK, SEP>::wave_bytes(NTW) * (wave + 1));
#pragma unroll
                for (int nt = 0; nt < NTW; ++nt) part = part + terms[nt * 64 + lane];
            }
        }
        if constexpr (kCanPart) {
#pragma unroll
            for (int q = 0; q < NTW / 2; ++q)
                if (ends_part(2 * q + 1)) put(ends[q], (wave_row0 + q * 64) / part_rows);
        } else if (!handed_over) {
            put(part, kPaired ? wave >> 1 : wave);
        }
    };

    for (int it = 0; it <= a.n_iter; ++it) {
        const bool last_pass = (it == a.n_iter);
        passes_run = it + 1;
        uint32_t flagged_tiles = 0;      // tiles with rows that the screen could not decide
        uint32_t changed_tiles = 0;      // tiles in which a label may differ from the current one

        // The tile loop, compiled once per number of live registers of the last m-tile (4, 8, 12 or 16),
        // so that the epilogue has no branches.
        auto tile_pass = [&](auto live_tag) {
            constexpr int LREGS = decltype(live_tag)::value;
            const int lane = opaque(lane_id), n32 = lane & 31;
            // A fragments of this pass (the bias slot included)
            half8 A0[NSA], A1[NSA];
#pragma unroll
            for (int s = 0; s < NS2; ++s) {
                A0[s] = U.afrag[s * 64 + lane];
                A1[s] = two ? U.afrag[(NS2 + s) * 64 + lane] : A0[s];
            }
            // the bias step: 256 against hi (slot 0) and lo (slot 1), the same for every row
            half8 bias_b;
            if constexpr (SEP) {
                A0[NS2] = U.abias[lane];
                A1[NS2] = two ? U.abias[64 + lane] : A0[NS2];
#pragma unroll
                for (int i = 0; i < 8; ++i) bias_b[i] = (_Float16)(i < 2 && lane < 32 ? kBiasScale : 0.0f);
            }

            float16v accA, accB;
            const float16v zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};

            // one matrix instruction of the chain of a 32x32 tile (the first one behind the bias step)
            auto mma = [&](float16v &acc, const half8 (&Af)[NSA], const half8 (&Bt)[NS], int s) {
                if constexpr (SEP) {
                    if (s == 0) acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(Af[NS2], bias_b, zero16, 0, 0, 0);
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(Af[s], Bt[s % NS], acc, 0, 0, 0);
                    return;
                }
                acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(Af[s], Bt[s % NS], s == 0 ? zero16 : acc, 0, 0, 0);
            };
            // mark scores [i0, i0 + CH): bit set = above the threshold (or padding)
            auto mark = [&](uint32_t &far, const float16v &acc, float thr, int i0) {
#pragma unroll
                for (int i = 0; i < CH; ++i)
                    if (i0 + i < 16) far = __builtin_amdgcn_alignbit(far, __float_as_uint(thr - acc[i0 + i]), 31);
            };
            // minimum over the first nreg registers (nreg = 4, 8, 12 or 16)
            auto min_live = [&](const float16v &acc, auto nreg_tag) {
                constexpr int nreg = decltype(nreg_tag)::value;
                float b = vmin(vmin3(acc[0], acc[1], acc[2]), acc[3]);
                if (nreg > 4) b = vmin3(vmin3(b, acc[4], acc[5]), acc[6], acc[7]);
                if (nreg > 8) b = vmin3(vmin3(b, acc[8], acc[9]), acc[10], acc[11]);
                if (nreg > 12) b = vmin3(vmin3(b, acc[12], acc[13]), acc[14], acc[15]);
                return b;
            };
            // both lane halves' minima of a row -> the row's minimum
            auto row_min = [&](float v) {
                unsigned lo, hi;
                both_halves(__float_as_uint(v), lo, hi);
                return vmin(__uint_as_float(lo), __uint_as_float(hi));
            };
            // After the masks of tile nt: if any row's mask differs from the remembered one (or the tile is
            // forced), remember the new masks and decide the tile's rows: a row with exactly one
            // candidate takes it, any other row is left to the exact evaluation after the tile loop
            // (label 0xFE until then).  Tiles with such rows and tiles in which a label differs from
            // the current one are listed.  (The matrix instructions of the next tile are under way
            // meanwhile.)
            auto settle = [&](uint32_t far, uint32_t seen, int nt) {
                const uint64_t diff = __ballot(far != seen);
                const uint32_t live32 = live_rows(nt);
                uint32_t dirty32 = ((uint32_t)diff | (uint32_t)(diff >> 32)) & live32;
                if ((force_tiles >> nt) & 1u) dirty32 = live32;
                if (dirty32) {
                    Q.seen()[nt * 64 + lane] = far;
                    const uint32_t prev = Q.lab()[nt * 32 + n32];
                    const uint32_t cand = ~far;                          // bit 31 = position 0
                    uint32_t cand_lo, cand_hi;
                    both_halves(cand, cand_lo, cand_hi);
                    const int total = __popc(cand_lo) + __popc(cand_hi);
                    const bool live = (live32 >> n32) & 1u;
                    const bool flagged = live && total != 1;
                    const int hh = cand_lo ? 0 : 1;
                    const int q = __clz((int)(cand_lo ? cand_lo : cand_hi));
                    const uint32_t lab = (uint32_t)slot_centroid(q & 31, hh);
                    const uint32_t now = !live ? 0xFFu : (flagged ? 0xFEu : lab);
                    if (__ballot(flagged)) flagged_tiles |= 1u << nt;
                    if (__ballot(now != prev)) {
                        changed_tiles |= 1u << nt;
                        if (lane < 32) Q.lab_new()[nt * 32 + n32] = (unsigned char)now;
                    }
                }
            };

            // bound and remembered mask of the tile under way; those of the next tile are fetched a tile ahead
            float eb_cur = Q.eb()[n32];
            uint32_t seen_cur = Q.seen()[lane];
            if (kAllowTwo && two) {
                // accA = centroids 0..31 (all sixteen registers live), accB = centroids 32..k-1 of the current tile
#pragma unroll
                for (int s = 0; s < NS2; ++s) mma(accA, A0, B[0], s);
#pragma unroll
                for (int s = 0; s < NS2; ++s) mma(accB, A1, B[0], s);
#pragma unroll
                for (int nt = 0; nt < NTW; ++nt) {
                    constexpr int kLast = NTW - 1;
                    const int nx = nt < kLast ? nt + 1 : nt;
                    const float eb_nxt = Q.eb()[nx * 32 + n32];
                    const uint32_t seen_nxt = Q.seen()[nx * 64 + lane];
                    const float best = row_min(vmin(min_live(accA, std::integral_constant<int, 16>{}), min_live(accB, live_tag)));
                    const float thr = best + eb_cur;
                    uint32_t far = 0;
#pragma unroll
                    for (int s = 0; s < NS2; ++s) mark(far, accA, thr, s * CH);
                    // accA is consumed: its next chain runs under the marking of accB
#pragma unroll
                    for (int s = 0; s < NS2; ++s) {
                        __builtin_amdgcn_sched_barrier(0);
                        if (nt < kLast) mma(accA, A0, B[nx], s);
                        __builtin_amdgcn_sched_barrier(0);
                        if (s * CH < LREGS) mark(far, accB, thr, s * CH);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                    if (nt < kLast) {
#pragma unroll
                        for (int s = 0; s < NS2; ++s) mma(accB, A1, B[nx], s);
                    }
                    // registers of accB that were not walked hold padding only: far
                    constexpr int live_marks = CH * ((LREGS + CH - 1) / CH);
                    far = (far << (16 - live_marks)) | ((1u << (16 - live_marks)) - 1u);
                    settle(far, seen_cur, nt);
                    eb_cur = eb_nxt;
                    seen_cur = seen_nxt;
                    __builtin_amdgcn_sched_barrier(0);
                }
            } else {
                // one m-tile: the accumulators alternate, the next tile's chain runs under this epilogue
#pragma unroll
                for (int s = 0; s < NS2; ++s) mma(accA, A0, B[0], s);
#pragma unroll
                for (int nt = 0; nt < NTW; ++nt) {
                    constexpr int kLast = NTW - 1;
                    const int nx = nt < kLast ? nt + 1 : nt;
                    float16v &cur = (nt & 1) ? accB : accA;
                    float16v &nxt = (nt & 1) ? accA : accB;
                    const float eb_nxt = Q.eb()[nx * 32 + n32];
                    const uint32_t seen_nxt = Q.seen()[nx * 64 + lane];
                    const float best = row_min(min_live(cur, live_tag));
                    const float thr = best + eb_cur;
                    uint32_t far = 0;
#pragma unroll
                    for (int s = 0; s < NS2; ++s) {
                        __builtin_amdgcn_sched_barrier(0);
                        if (nt < kLast) mma(nxt, A0, B[nx], s);
                        __builtin_amdgcn_sched_barrier(0);
                        if (s * CH < LREGS) mark(far, cur, thr, s * CH);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                    constexpr int live_marks = CH * ((LREGS + CH - 1) / CH);
                    far = (far << (32 - live_marks)) | (0xFFFFFFFFu >> live_marks);
                    settle(far, seen_cur, nt);
                    eb_cur = eb_nxt;
                    seen_cur = seen_nxt;
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        };
        if (wave_live) {
            switch (lregs) {
            case 4: tile_pass(std::integral_constant<int, 4>{}); break;
            case 8: tile_pass(std::integral_constant<int, 8>{}); break;
            case 12: tile_pass(std::integral_constant<int, 12>{}); break;
            default: tile_pass(std::integral_constant<int, 16>{}); break;
            }
        }

        // ---- the undecided rows: exact evaluation, through the queue (this code exists once; the tile
        // index is a run-time value)
        int nrec = 0;
        {
            const int lane = opaque(lane_id), n32 = lane & 31, h = lane >> 5;
            uint32_t todo = flagged_tiles;
            while (todo) {
                const int nt = __builtin_ctz(todo);
                todo &= todo - 1;
                // a batch of queued rows that may not fit one more tile is resolved first
                if constexpr (!kShortQueue) {
                    if (nrec + 32 > kRecCap) {
                        resolve_queue<DK>(Q, nrec, U.mu64T, U.ojf, KP, k, d);
                        nrec = 0;
                    }
                }
                const uint32_t live32 = live_rows(nt);
                const uint32_t cand = ~Q.seen()[nt * 64 + lane];       // bit 31 = position 0
                uint32_t cand_lo, cand_hi;
                both_halves(cand, cand_lo, cand_hi);
                const int total = __popc(cand_lo) + __popc(cand_hi);
                const bool live = (live32 >> n32) & 1u;
                const bool flagged = live && total != 1;
                const uint64_t fm = __ballot(flagged) & 0xFFFFFFFFull;
                if (fm) {
                    if constexpr (kShortQueue) {
                        if (nrec + __popcll(fm) > WaveQueue<DK, NTW>::kCap) {
                            resolve_queue<DK>(Q, nrec, U.mu64T, U.ojf, KP, k, d);
                            nrec = 0;
                        }
                    }
                    half8 bt[NS];
                    rows_of_tile(nt, bt);
                    if (flagged) {
                        const int rs = nrec + __popcll(fm & ((1ull << n32) - 1ull));
#pragma unroll
                        for (int f = 0; f < NS; ++f)
                            *reinterpret_cast<half8 *>(Q.rec_x() + (size_t)rs * DK + 16 * f + 8 * h) = bt[f];
                        // no candidate at all cannot happen (the smallest score is always one); if it does, every centroid is one
                        Q.rec_mask()[rs * 2 + h] = total ? cand : 0xFFFFFFFFu;
                        if (h == 0) Q.rec_pid()[rs] = (unsigned short)(nt * 32 + n32);
                    }
                    nrec += __popcll(fm);
                }
            }
            if (nrec) resolve_queue<DK>(Q, nrec, U.mu64T, U.ojf, KP, k, d);
        }
        force_tiles = flagged_tiles;

        // ---- label changes of the decided tiles -> integer sums and counts.
        // A row without a label yet has previous = 0xFF; rows outside the task keep 0xFF and never change.
        int wave_changed = 0;
        if (full_mode) {
            // the new labels become the current ones; the sums are rebuilt from all of them
            const int lane = opaque(lane_id), n32 = lane & 31, h = lane >> 5;
            uint32_t todo = changed_tiles;
            while (todo) {
                const int nt = __builtin_ctz(todo);
                todo &= todo - 1;
                const uint32_t cur = Q.lab_new()[nt * 32 + n32];
                const uint32_t prev = Q.lab()[nt * 32 + n32];
                const bool changed = cur != prev;
                wave_changed += __popcll(__ballot(changed) & 0xFFFFFFFFull);
                if (changed && h == 0) Q.lab()[nt * 32 + n32] = (unsigned char)cur;
            }
            __builtin_amdgcn_wave_barrier();
            if (wave_live) {
                const int left = nrows - wave_row0;
                full_sums<DK, NTW / 2, SEP>(Q, U.S, U.n, xw, a.ld, d, k, left < NTW * 32 ? left : NTW * 32, lane);
            }
        } else {
            // a dense queue of (previous, new, knob values), applied with one lane per (row, group of four
            // knobs), in batches of at most kCap rows
            const int lane = opaque(lane_id), n32 = lane & 31, h = lane >> 5;
            (void)lane;
            uint32_t todo = changed_tiles;
            int cnt = 0;
            while (todo) {
                const int nt = __builtin_ctz(todo);
                todo &= todo - 1;
                const uint32_t cur = Q.lab_new()[nt * 32 + n32];
                const uint32_t prev = Q.lab()[nt * 32 + n32];
                const bool changed = cur != prev;
                const uint64_t cm = __ballot(changed) & 0xFFFFFFFFull;
                if (cm) {
                    int add = 32;
                    if constexpr (kShortQueue) add = __popcll(cm);
                    if (cnt + add > WaveQueue<DK, NTW>::kCap) {
                        apply_changes<DK>(Q, cnt, U.S, U.n, U.dirty, U.ojf, d, it);
                        cnt = 0;
                    }
                    half8 bt[NS];
                    rows_of_tile(nt, bt);
                    if (changed) {
                        const int rs = cnt + __popcll(cm & ((1ull << n32) - 1ull));
#pragma unroll
                        for (int f = 0; f < NS; ++f)
                            *reinterpret_cast<half8 *>(Q.rec_x() + (size_t)rs * DK + 16 * f + 8 * h) = bt[f];
                        if (h == 0) {
                            Q.rec_mask()[rs] = cur | (prev << 8);
                            Q.lab()[nt * 32 + n32] = (unsigned char)cur;
                        }
                    }
                    cnt += __popcll(cm);
                    wave_changed += __popcll(cm);
                }
            }
            if (cnt) apply_changes<DK>(Q, cnt, U.S, U.n, U.dirty, U.ojf, d, it);
        }
        if (wave_changed && lane_id == 0) atomicAdd(&U.stamp[2 + (it & 1)], wave_changed);
        traced_last = false;
        if (a.trace) {
            wave_loss((it & 1) * kParts);
            traced_last = true;
        }
        __syncthreads();
        if (a.trace && tid == 0) {
            double s = 0.0;
            if (parted) s = sum_of_parts(U.red + (it & 1) * kParts, n_parts);
            else for (int w = 0; w < n_parts; ++w) s = s + U.red[(it & 1) * kParts + w];
            a.trace[slot * (a.n_iter + 1) + it] = s;
        }
        // A pass that moved no row leaves every sum, hence every centroid, as it was: the labels are
        // final.  (The count is read between this pass's two barriers, or after its only one when the
        // loop ends here; no wave adds to it in between.)
        const int rows_changed = __builtin_amdgcn_readfirstlane(U.stamp[2 + (it & 1)]);
        at_fixed_point = rows_changed == 0;
        if (last_pass || rows_changed == 0) break;
        if (tid == 0) U.stamp[2 + ((it + 1) & 1)] = 0;      // the next pass counts from zero (nobody adds before the barrier below)
        const bool full_next = x_aligned && rows_changed > full_above;
        update_centroids<DK, kByteKnobs, SEP>(U, k, KP, d, it, false, full_mode, full_next);
        full_mode = full_next;
        __syncthreads();
    }

    // ---- results: labels, loss, centroids, counts
    if (wave_live) {
        for (int e = lane; e < NTW * 32; e += 64) {
            const int pid = wave_row0 + e;
            if (pid < nrows) labrow[r0 + pid] = Q.lab()[e];
        }
    }
    // the loss of the final labels: the per-wave sums of the last traced pass are still in place
    int loss_slot = ((passes_run - 1) & 1) * kParts;
    double loss = 0.0;
    if (kByteKnobs && !traced_last && at_fixed_point) {
        // At a fixed point every non-empty centroid is the mean S / n of its cluster, so the loss is
        // sum_rows |x|^2 - sum_c |S_c|^2 / n_c, all integers but the last division: with
        // |S_c|^2 = q_c n_c + r_c it is the integer (sum |x|^2 - sum q_c) minus the sum of the fractions
        // r_c / n_c, which is exact up to the rounding of those k fractions and of the final
        // subtraction (and exactly zero when every cluster's rows coincide).  The sums left by a
        // pass that rebuilt them on the matrix cores are still off by raw_offset n.
        double *frac0 = WaveQueue<DK, NTW>(U.wave_base).few();     // the queues are idle: [k] doubles of the first wave's region
        for (int c = tid; c < k; c += blockDim.x) {
            const int nc = U.n[c];
            double fr = 0.0;
            if (nc > 0) {
                unsigned long long ss = 0;
                for (int j = 0; j < d; ++j) {
                    const long long sv = (long long)U.S[c * (DK + 1) + j] - (full_mode ? (long long)raw_offset(true) * nc : 0ll);
                    ss += (unsigned long long)(sv * sv);
                }
                const unsigned long long qc = ss / (unsigned long long)nc;
                const unsigned long long rc = ss - qc * (unsigned long long)nc;
                atomicAdd(&U.acc64[1], qc);
                fr = (double)rc / (double)nc;
            }
            frac0[c] = fr;
        }
        __syncthreads();
        if (tid == 0) {
            double fsum = 0.0;
            for (int c = 0; c < k; ++c) fsum = fsum + frac0[c];
            loss = (double)(U.acc64[0] - U.acc64[1]) - fsum;
        }
    } else {
        if (!traced_last) {
            loss_slot = 0;
            wave_loss(0);
            __syncthreads();
        }
        if (tid == 0) {
            if (parted) loss = sum_of_parts(U.red + loss_slot, n_parts);
            else for (int w = 0; w < n_parts; ++w) loss = loss + U.red[loss_slot + w];
        }
    }
    if (a.trace && tid == 0) {
        // the passes that were not run would have seen the same labels and centroids
        for (int it = passes_run; it <= a.n_iter; ++it) a.trace[slot * (a.n_iter + 1) + it] = loss;
    }
    for (int e = tid; e < k * d; e += blockDim.x) {
        const int c = e / d, j = e % d;
        a.centroids[(crow + c) * d + j] = U.mu64T[(size_t)j * KP + c];
    }
    for (int c = tid; c < k; c += blockDim.x) a.counts[crow + c] = U.n[c];
    if (tid == 0) {
        a.status[slot] = 0;
        a.inertia[slot] = loss;
        a.passes[slot] = passes_run;
    }
}

// ---- the variant that fetches its rows in every pass ----
//
// Rows of this many make up one workgroup of the packing kernel and one entry of the tasks' tables of norms.
constexpr int kPackRows = 256;

__device__ __forceinline__ const unsigned char *packed_task(const SweepArgs &a, int t, int DK)
{
    return reinterpret_cast<const unsigned char *>(a.xh) + ((a.task_off[t] >> 5) + t) * (32 * DK * 2);
}

// Centred f16 copy of X: knob j less the task's offset, absent knobs zero, the bias slot
// (last one, not with SEP) holding its constant, so that a lane's 16 bytes are a B fragment as they stand.  Offset of a
// knob: the rounded mean over eight runs of eight rows spread over the task (any integer would do: it keeps the magnitudes
// small).  Beside the rows, per workgroup: the largest squared norm of a centred row (for the error bound) and
// the sum of the raw squared norms (for the loss at a fixed point; byte knobs).
// PL = 2: any two-byte value, in two parts that are exact in f16, the multiple of 256 below its magnitude and the rest; there
// is no bias slot.
// Bound by its chain of latencies (task, offsets, rows, LDS) in small calls, so the row's knobs are asked for first, and by bank conflicts of
// the byte copy, whose lanes read 256 bytes apart but for the padding.  Us, with both / with neither: 32 tasks of 2000 x 32
// bytes 10.9 / 13.5, one of 2000 x 24 8.8 / 10.4, 64 of up to 600 x 48 two-byte knobs 12.6 / 20.0, of up to 2048 x 32 13.7 / 19.8, values in
// two parts 13.4 / 15.5.
template <int DK, typename XT, bool SEP, int PL>
__global__ __launch_bounds__(kPackRows) void pack_centred_kernel(const SweepArgs a, int per_task, int first_task)
{
    constexpr bool kByteKnobs = sizeof(XT) == 1;
    constexpr int NM = DK > 32 ? 2 : 1, NP = (int)sizeof(XT);
    __shared__ int off[DK];
    __shared__ unsigned top_sq, sum_sq;
    __shared__ __align__(16) unsigned char raw[NP][32 * NM][kPackRows + 16];      // (16: the lanes of a fragment read different banks)
    const int t = first_task + (int)(blockIdx.x / (unsigned)per_task), b = (int)(blockIdx.x % (unsigned)per_task);
    const int64_t r0 = a.task_off[t];
    const int nrows = (int)(a.task_off[t + 1] - r0);
    if (b * kPackRows >= nrows) return;
    const XT *X = reinterpret_cast<const XT *>(a.X);
    const int tid = threadIdx.x, d = a.d;
    const int row = b * kPackRows + tid;
    if (tid == 0) {
        top_sq = 0u;
        sum_sq = 0u;
    }
    // the row's knobs are on their way while the offsets are found
    XT x[DK];
#pragma unroll
    for (int j = 0; j < DK; ++j) x[j] = j < d && row < nrows ? X[(int64_t)j * a.ld + r0 + row] : (XT)0;
    for (int e = tid; e < DK * 8; e += kPackRows) {          // (uniform within a wave: every lane exchanges)
        const int j = e >> 3, part = e & 7;
        int sum = 0;
        if (j < d) {
            const int first = (int)((int64_t)nrows * part / 8);
            for (int i = 0; i < 8; ++i) sum += (int)X[(int64_t)j * a.ld + r0 + (first + i < nrows ? first + i : nrows - 1)];
        }
        sum += dpp_xor_i32<1>(sum);
        sum += dpp_xor_i32<2>(sum);
        sum += dpp_xor_i32<4>(sum);
        if (part == 0) {
            const int o = (sum + 32) >> 6;
            off[j] = o;
            if (b == 0) a.ojf[t * 64 + j] = (float)o;
        }
    }
    __syncthreads();
    float c2 = 0.0f;                                         // (byte knobs and values below 2048: within 2^-20 of exact)
    unsigned raw2 = 0, top = 0;
    if (row < nrows) {
        unsigned char *out = const_cast<unsigned char *>(packed_task(a, t, DK * PL));
#pragma unroll
        for (int g = 0; g < DK / 8; ++g) {
            half8 v, rest;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int j = 8 * g + i;
                const int xv = (int)x[j];
                const int cv = j < d ? xv - off[j] : 0;
                top = (unsigned)xv > top ? (unsigned)xv : top;
                raw[0][j][tid] = (unsigned char)xv;
                if (NP == 2) raw[NP - 1][j][tid] = (unsigned char)(xv >> 8);
                if (kByteKnobs) raw2 += (unsigned)(xv * xv);
                c2 = __builtin_fmaf((float)cv, (float)cv, c2);
                const int high = PL == 2 ? (cv < 0 ? -(-cv & ~255) : cv & ~255) : cv;
                v[i] = (_Float16)(float)high;
                rest[i] = (_Float16)(float)(cv - high);
            }
            if (!SEP && PL == 1 && g == DK / 8 - 1) v[7] = (_Float16)bias_scale(kByteKnobs);
            *reinterpret_cast<half8 *>(out + packed_at(row, g, DK * PL)) = v;
            if (PL == 2) *reinterpret_cast<half8 *>(out + packed_at(row, DK / 8 + g, DK * PL)) = rest;
        }
        if (!kByteKnobs && PL == 1 && top >= 2048u) *a.too_large = 1;
    }
    atomicMax(&top_sq, (unsigned)__float_as_int(c2));        // (non-negative floats order like integers)
    if (kByteKnobs) atomicAdd(&sum_sq, raw2);                // (at most 256 * 32 * 255^2 < 2^32)
    __syncthreads();
    // the bytes of 32 rows in the order of A fragments (packed_sums): sixteen rows of a knob at a time
    {
        unsigned char *out = reinterpret_cast<unsigned char *>(a.xk) + ((r0 >> 5) + t + b * (kPackRows / 32)) * (int64_t)(1024 * NM * NP);
        const int tiles = ((nrows - b * kPackRows < kPackRows ? nrows - b * kPackRows : kPackRows) + 31) >> 5;
        for (int e = tid; e < tiles * 64 * NM * NP; e += kPackRows) {
            const int f = e >> 6, kh = (e >> 5) & 1, m = e & 31;         // fragment of the workgroup's tiles, lane within it
            const int tile = f / (NM * NP), q = f / NP % NM, p = f % NP;
            typedef unsigned uint4v __attribute__((ext_vector_type(4)));
            uint4v v = {0u, 0u, 0u, 0u};
            if (32 * q + m < d) v = *reinterpret_cast<const uint4v *>(&raw[p][32 * q + m][32 * tile + 16 * kh]);
            *reinterpret_cast<uint4v *>(out + (size_t)e * 16) = v;
        }
    }
    if (tid == 0) {
        a.norms[t * 32 + b] = __float_as_int(__int_as_float((int)top_sq) * 1.00001f);
        a.norms[t * 32 + 16 + b] = (int)sum_sq;
    }
}

// Centroid rows LDS holds (KP).
template <bool MANY>
__host__ __device__ constexpr int centroid_rows(int kmax) { return MANY ? (kmax + 31) / 32 * 32 : (kmax > 32 ? 64 : 32); }

// One unit, its rows fetched from the packed copy in every pass (L2 holds the rows of the tasks under way) instead of kept
// in registers: 128 registers a wave and 80 KiB of LDS then let two workgroups share a compute unit whatever the size of the
// task, and one's barriers and chains of dependent LDS accesses run under the other's tiles.
// MANY: k up to kManyCentroids, a tile against 64 centroids at a time.  A chunk of 64 leaves its minimum and the marks within the
// bound of it; the marks of a chunk count iff its minimum is within the bound of the overall one (that keeps every centroid
// within the bound of the overall minimum, and some up to two bounds away).  LDS holds one workgroup per compute unit, of
// sixteen waves up to k = 192.  16 tasks of up to 2500 x 24, k = 72, 96, 128, 20 steps: the streaming kernels' 43
// launches 645 us a step, one launch of this 450 us.
template <int DK, typename XT, bool SEP, bool MANY, int PL>
__device__ __forceinline__ void run_unit_fetched(const SweepArgs &a, unsigned char *smem, int ki, int t, int k)
{
    constexpr bool kByteKnobs = sizeof(XT) == 1;
    constexpr float kBiasScale = bias_scale(kByteKnobs);
    constexpr bool kAllowTwo = DK <= 32;      // (k <= 32 with wider rows)
    typedef typename std::conditional<MANY, ManyQueue<DK>, FetchedQueue<DK, PL>>::type Queue;
    const XT *X = reinterpret_cast<const XT *>(a.X);
    const bool two = kAllowTwo && k > 32;
    constexpr int NS = DK / 16;          // distinct B fragments per row
    constexpr int NS2 = 2 * NS;          // chained instructions per 32x32 tile, without the bias step
    constexpr int NSA = NS2 + (SEP ? 1 : 0);   // ... with it
    const int KP = centroid_rows<MANY>(a.kmax);
    MfmaLds<DK, SEP> U(smem, KP);

    const int tid = threadIdx.x;
    const int lane_id = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nwaves = blockDim.x >> 6;
    // the phases of a pass take the lane index through this: values derived from it are then computed where they are used
    auto opaque = [](int v) {
        asm volatile("" : "+v"(v));
        return v;
    };

    const int d = a.d;
    const int64_t r0 = a.task_off[t], r1 = a.task_off[t + 1];
    const int nrows = (int)(r1 - r0);
    const int64_t slot = (int64_t)t * a.n_k + ki;
    const int64_t crow = (int64_t)t * a.Ksum + a.koff[ki];
    uint8_t *labrow = a.labbuf + (int64_t)ki * a.ld;

    auto region = [&]() {
        if constexpr (MANY) return Queue(U.wave_base + Queue::bytes(nwaves) * wave, nwaves);
        else return Queue(U.wave_base + Queue::kBytes * wave);
    };
    const Queue Q = region();
    const int lab_rows = nwaves == 16 && MANY ? Queue::kRows / 2 : Queue::kRows;       // rows the label tables hold
    // Rows of the task in kParts equal parts of whole groups of 64; a wave has one, or two in a row.  The loss is summed part by
    // part, so that its order does not depend on the number of waves.
    const int part_rows = rows_of_part(nrows);
    const int run = part_rows * (kParts / nwaves);
    const int wave_row0 = wave * run;
    const int rows_wave = nrows - wave_row0 < run ? (nrows - wave_row0 > 0 ? nrows - wave_row0 : 0) : run;
    const bool wave_live = rows_wave > 0;
    const int ntiles = (rows_wave + 31) >> 5;
    const unsigned char *packed = packed_task(a, t, DK * PL) + (size_t)(wave_live ? wave_row0 : 0) * (DK * PL * 2);      // (whole tiles)

    const int kk_last = two ? k - 32 : k;                  // centroids in the last (or only) m-tile
    const int lregs = ((kk_last + 1) / 2 + 3) & ~3;        // live accumulator registers, in groups of four
    constexpr int bstep = NS - 1, bhalf = 1, belem = 7;
    // (the rebuild against changes applied one by one after a pass that moved more than 1/3, 1/8, 1/16, 1/32 of the rows: the full model
    // 12.68 / 12.99 / 13.2 / 13.6 ms a step, 16 x 1900 x 27 two-byte knobs 479 / 510 / 525 / 569 us)
    constexpr int kFullDivisor = 3;

    // ---- set-up
    for (int e = tid; e < DK * KP; e += blockDim.x) U.mu64T[e] = 0.0;
    for (int e = tid; e < KP * (DK + 1); e += blockDim.x) U.S[e] = 0;
    for (int c = tid; c < KP; c += blockDim.x) {
        U.n[c] = 0;
        U.dirty[c] = -1;
        U.bias[c] = 0.0f;
    }
    if (tid < DK) U.ojf[tid] = a.ojf[t * 64 + tid];
    {
        half8 z;
#pragma unroll
        for (int i = 0; i < 8; ++i) z[i] = (_Float16)0.0f;
        for (int e = tid; e < (KP / 32) * NSA * 64; e += blockDim.x) U.afrag[e] = z;      // (abias included)
    }
    if (tid == 0) {
        U.stamp[1] = 0;           // float bits of the largest squared norm of a centred row
        U.stamp[2] = 0;           // rows that changed their label in an even pass
        U.stamp[3] = 0;           // ... in an odd pass
        U.acc64[0] = 0ull;
        U.acc64[1] = 0ull;
    }
    for (int e = lane_id; e < 2 * lab_rows / 4; e += 64) reinterpret_cast<unsigned *>(Q.lab())[e] = 0xFFFFFFFFu;      // no row has a label yet
    __syncthreads();
    // padding centroid rows (beyond k) carry a huge bias so that they never win
    if (PL == 2) {
        for (int c = k + tid; c < KP; c += blockDim.x) U.start[(c >> 5) * 32 + 16 * (c & 1) + ((c & 31) >> 1)] = kPadScore;
    } else for (int c = k + tid; c < KP; c += blockDim.x) {
        _Float16 *bslot = SEP ? reinterpret_cast<_Float16 *>(U.abias + (c >> 5) * 64 + frag_row(c))
                              : reinterpret_cast<_Float16 *>(U.afrag + ((c >> 5) * NS2 + bstep) * 64 + 32 * bhalf + frag_row(c)) + belem;
        bslot[0] = (_Float16)kHalfMax;
    }
    if (tid < (nrows + kPackRows - 1) / kPackRows) {
        atomicMax(&U.stamp[1], a.norms[t * 32 + tid]);           // non-negative floats order like integers
        if (kByteKnobs && !MANY) atomicAdd(&U.acc64[0], (unsigned long long)(unsigned)a.norms[t * 32 + 16 + tid]);
    }
    for (int e = tid; e < k * d; e += blockDim.x) {
        const int c = e / d, j = e % d;
        double v;
        if (a.init_mode == 0) {
            const int row = a.init_rows[(int64_t)t * a.kmax + c];
            v = (double)X[(int64_t)j * a.ld + r0 + row];
        } else {
            v = a.init_centroids[(crow + c) * d + j];
        }
        U.mu64T[(size_t)j * KP + c] = v;
    }
    __syncthreads();
    update_centroids<DK, kByteKnobs, SEP, PL>(U, k, KP, d, 0, true);
    __syncthreads();
    if constexpr (MANY) {
        // Starts that no row can be nearest to take no part in the screen.  Some centroid always lies within reach = max(farthest row, nearest
        // start) of the origin (it stays, or becomes a mean of rows), hence within 2 reach of every row; a start beyond 3 reach is farther off
        // than that, keeps no rows and so stays there.  It gets the score of a padding row: one such start widened the bound for all
        // rows, beyond the operands' range without end.  A quarter of the starts 0 / 1500 / 3000 from the rows, 8 tasks of 2500 x 24, k = 72 and
        // 128, 20 steps: 408 / 419 / 418 us a sweep, without this 404 / 493 / 21 200.
        const unsigned inf = 0x7F800000u;                  // (norms are not negative: they order like integers)
        unsigned nearest = inf, farthest = 0u;
        for (int c = lane_id; c < k; c += 64) {
            const unsigned b = __float_as_uint(U.bias[c]);
            nearest = b < nearest ? b : nearest;
            farthest = b <= inf && b > farthest ? b : farthest;
        }
        for (int off = 32; off >= 1; off >>= 1) {
            const unsigned o = __shfl_xor(nearest, off, 64), f = __shfl_xor(farthest, off, 64);
            nearest = o < nearest ? o : nearest;
            farthest = f > farthest ? f : farthest;
        }
        const unsigned reach = nearest > (unsigned)U.stamp[1] ? nearest : (unsigned)U.stamp[1];
        const unsigned limit = __float_as_uint(10.0f * __uint_as_float(reach));      // 3^2, and room for the roundings
        if (farthest > limit) {
            __syncthreads();
            half8 z;
#pragma unroll
            for (int i = 0; i < 8; ++i) z[i] = (_Float16)0.0f;
            for (int c = tid; c < k; c += blockDim.x) {
                const unsigned b = __float_as_uint(U.bias[c]);
                if (b <= limit || b > inf) continue;
                half8 *frag = U.afrag + (c >> 5) * NS2 * 64 + frag_row(c);
                for (int f = 0; f < 2 * NS2; ++f) frag[32 * f] = z;
                reinterpret_cast<_Float16 *>(frag + bstep * 64 + 32 * bhalf)[belem] = (_Float16)kHalfMax;
                U.bias[c] = 0.0f;
            }
            __syncthreads();
        }
    }
    // Screen bound of the unit: that of its farthest row, half as much again as the origin's at most (m2 counts twice).  Largest squared norm a centred centroid can take during the iteration: every
    // later centroid is a mean of rows (inside their convex hull) or stays where it started.
    float bound;
    {
        const float x2 = __int_as_float(U.stamp[1]);
        float m2 = lane_id < k ? U.bias[lane_id] : 0.0f;
        if (MANY)
            for (int c = lane_id + 64; c < k; c += 64) m2 = __builtin_fmaxf(m2, U.bias[c]);
        m2 = wave_max_nonneg(m2);
        m2 = __builtin_fmaxf(m2, x2) * 1.000001f;
        // starts beyond the range of the screen (their operands are clamped): every centroid is a candidate of every row
        if (!(m2 <= (PL == 2 ? 1.0e13f : max_screened(kByteKnobs)))) m2 = kFarNorm;
        // Values in two parts: twice the instructions, a quarter of the score; the absolute term is half the spacing of the low
        // operands' subnormal values times the sum of the parts' magnitudes, at most sqrt(48) |x'| + 48 * 255.
        if (PL == 2) bound = kTwoPartScale * mfma_bound_slope<NS2 * PL>() * (x2 + 2.0f * m2) + 7.5e-8f * (7.0f * __builtin_sqrtf(x2) + 12288.0f);
        else bound = mfma_bound<NSA, kByteKnobs>(x2, m2);
    }

    int passes_run = 0;
    bool at_fixed_point = false;         // the last pass run moved no row: every centroid is the mean of its cluster
    // A pass after one that moved many rows rebuilds the sums from the labels on the matrix cores
    // instead of applying the changes one by one; the first pass (every row is new) always does.
    constexpr int NM = DK > 32 ? 2 : 1, NP = (int)sizeof(XT);
    const unsigned char *bytes_w = reinterpret_cast<const unsigned char *>(a.xk) + ((r0 >> 5) + t + (wave_live ? wave_row0 >> 5 : 0)) * (int64_t)(1024 * NM * NP);
    bool full_mode = true;
    const int full_above = nrows / kFullDivisor;      // changed rows of a pass above which the next one rebuilds
    bool traced_last = false;

    // Exact loss of the current labels: (x - mu)^2 in double over the knobs a lane holds (x = centred value + offset, exact), the two
    // lanes of a row and all rows of a part added up afterwards; the sums of the parts land in U.red[at .. at + kParts).
    auto wave_loss = [&](int at) {
        const int lane = opaque(lane_id), n32 = lane & 31, h = lane >> 5;
        float of[NS][8];
#pragma unroll
        for (int f = 0; f < NS; ++f)
#pragma unroll
            for (int i = 0; i < 8; ++i) of[f][i] = U.ojf[16 * f + 8 * h + i];
        for (int first = 0; first < run; first += part_rows) {
            double part = 0.0;
            const int last = first + part_rows < rows_wave ? first + part_rows : rows_wave;
            for (int nt = first >> 5; 32 * nt < last; ++nt) {
                half8 bt[NS * PL];
                fetch_tile<DK * PL>(bt, packed + nt * (32 * DK * PL * 2), (unsigned)(16 * lane));
                const uint32_t lab = Q.lab()[nt * 32 + n32];
                const bool live = lab != 0xFFu;
                const double *mc = U.mu64T + (live ? Queue::centroid(lab) : 0u) + (size_t)(8 * h) * KP;
                double s = 0.0;
#pragma unroll
                for (int f = 0; f < NS; ++f) {
                    // the centroid's knobs first, all loads under way together, then the sum in knob order
                    double mu[8];
#pragma unroll
                    for (int i = 0; i < 8; ++i) mu[i] = mc[(size_t)(16 * f + i) * KP];
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        float xf = (float)bt[f][i] + of[f][i];
                        if (PL == 2) xf += (float)bt[NS + f][i];
                        else if (!SEP && f == bstep && i == belem) xf = h == bhalf ? 0.0f : xf;     // the bias slot is no knob
                        const double tq = (double)xf - mu[i];
                        s = s + tq * tq;
                    }
                }
                part = part + (live ? s : 0.0);
            }
            // the part's total in the fixed order lane ^ 32, 16, ..., 1 (partner indices from the local lane index)
            double ws = part;
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) {
                const long long b = __double_as_longlong(ws);
                const int plo = __builtin_amdgcn_ds_bpermute((lane ^ off) << 2, (int)(b & 0xFFFFFFFFll));
                const int phi = __builtin_amdgcn_ds_bpermute((lane ^ off) << 2, (int)(b >> 32));
                ws = ws + __longlong_as_double(((long long)phi << 32) | (unsigned int)plo);
            }
            if (lane == 0) U.red[at + (wave_row0 + first) / part_rows] = ws;
        }
    };

    // MANY: the same terms in the order of the streaming kernels (stream_loss_kernel, tasks of one block of 4096 rows), which run such
    // lists of k when a task of the batch is larger: a loss does not depend on the form.  Every wave leaves the terms of its rows in its
    // queue's place; four waves add up, their sums land in U.red[at .. at + 4).
    auto many_loss = [&](int at) {
        const int lane = opaque(lane_id);
        double *term = reinterpret_cast<double *>(Q.base);
        for (int r = lane; r < rows_wave; r += 64) {
            const double *mc = U.mu64T + Queue::centroid(Q.lab()[r]);
            const unsigned char *x = packed + packed_at(r, 0, DK);
            double s = 0.0;
            for (int j0 = 0; j0 < d; j0 += 8) {
                const half8 xq = *reinterpret_cast<const half8 *>(x + packed_at(0, j0 >> 3, DK));
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    if (j0 + i < d) {
                        const double tq = (double)((float)xq[i] + U.ojf[j0 + i]) - mc[(size_t)(j0 + i) * KP];
                        s = s + tq * tq;
                    }
                }
            }
            term[r] = s;
        }
        __syncthreads();
        if (wave < kLossWaves) {
            const int consecutive = loss_run(d, k);
            double part = 0.0;
            for (int base = wave * consecutive; base < nrows; base += kLossWaves * consecutive)
                for (int first = base; first < base + consecutive && first < nrows; first += 64) {
                    const int owner = first / run;                 // (whole groups of 64 rows a wave)
                    if (first + lane < nrows)
                        part = part + reinterpret_cast<const double *>(U.wave_base + ManyQueue<DK>::bytes(nwaves) * owner)[first - owner * run + lane];
                }
            const double ws = wave_sum(part);
            if (lane == 0) U.red[at + wave] = ws;
        }
    };
    auto sum_losses = [&](int at) {
        if constexpr (MANY) many_loss(at);
        else wave_loss(at);
    };

    for (int it = 0; it <= a.n_iter; ++it) {
        const bool last_pass = (it == a.n_iter);
        passes_run = it + 1;
        int nrec = 0;                    // queued rows that the screen could not decide
        const Tiles tiles = {packed, U.afrag, U.abias, U.start, nullptr, bound, 0.0f, kBiasScale, ntiles, rows_wave, it == 0 ? ~0ull : 0ull};

        if constexpr (MANY) {
            decide_tiles_many<DK, false, false>(Q, tiles, nrec, U.mu64T, U.ojf, KP, k, d, opaque(lane_id));
        } else {
        if (wave_live) {
            int nt = 0;
            do {
                auto live_pass = [&](auto two_tag) {
                    switch (lregs) {
                    case 4: nt = decide_tiles<DK, SEP, PL == 2, false, 4, decltype(two_tag)::value>(Q, tiles, nt, nrec, opaque(lane_id)); break;
                    case 8: nt = decide_tiles<DK, SEP, PL == 2, false, 8, decltype(two_tag)::value>(Q, tiles, nt, nrec, opaque(lane_id)); break;
                    case 12: nt = decide_tiles<DK, SEP, PL == 2, false, 12, decltype(two_tag)::value>(Q, tiles, nt, nrec, opaque(lane_id)); break;
                    default: nt = decide_tiles<DK, SEP, PL == 2, false, 16, decltype(two_tag)::value>(Q, tiles, nt, nrec, opaque(lane_id)); break;
                    }
                };
                if constexpr (kAllowTwo) {
                    if (two) live_pass(std::true_type{});
                    else live_pass(std::false_type{});
                } else {
                    live_pass(std::false_type{});
                }
                if (nrec) resolve_batches<DK, PL>(Q, nrec, packed, U.mu64T, U.ojf, KP, k, d, opaque(lane_id));
                nrec = 0;
            } while (nt < ntiles);
        }
        }

        // ---- label changes -> integer sums and sizes.  Both label tables agree but for this pass's changes (a row without a label
        // yet has previous = 0xFF; rows outside the task keep 0xFF): a lane compares four rows at a time.
        int wave_changed = 0;
        {
            const int lane = opaque(lane_id);
            const uint64_t below = (1ull << lane) - 1ull;
            int cnt = 0;
            __builtin_amdgcn_wave_barrier();
            for (int first = 0; first < rows_wave; first += 256) {
                const unsigned at = first + 4 * lane;
                unsigned *oldp = reinterpret_cast<unsigned *>(Q.lab() + at);
                const unsigned cur4 = at < (unsigned)lab_rows ? *reinterpret_cast<const unsigned *>(Q.lab_new() + at) : 0u;
                const unsigned prev4 = at < (unsigned)lab_rows ? *oldp : 0u;
                const unsigned diff = cur4 ^ prev4;
                if (!__ballot(diff != 0u)) continue;
                if (diff) *oldp = cur4;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const bool changed = ((diff >> (8 * i)) & 0xFFu) != 0u;
                    const uint64_t cm = __ballot(changed);
                    if (!cm) continue;
                    const int add = __popcll(cm);
                    wave_changed += add;
                    if (full_mode) continue;                     // (the sums are rebuilt from all labels)
                    if (cnt + add > Queue::kChanges) {
                        apply_listed<DK>(Q, cnt, packed, U.S, U.n, U.dirty, U.ojf, d, it);
                        cnt = 0;
                    }
                    if (changed) {
                        const unsigned cur = (cur4 >> (8 * i)) & 0xFFu, prev = (prev4 >> (8 * i)) & 0xFFu;
                        Q.changes()[cnt + __popcll(cm & below)] =
                            Queue::centroid(cur) | (prev == 0xFFu ? 0x80000000u : Queue::centroid(prev) << 8) | (at + i) << 16;
                    }
                    cnt += add;
                }
            }
            if (full_mode) {
                __builtin_amdgcn_wave_barrier();
                if (wave_live) {
                    for (int first = 0; first < (MANY ? k : 1); first += 64)
                        packed_sums<DK, NM, NP, MANY>(Q, U.S, U.n, bytes_w, d, k, rows_wave, lane_id, first);
                }
            } else if (cnt) {
                apply_listed<DK>(Q, cnt, packed, U.S, U.n, U.dirty, U.ojf, d, it);
            }
        }
        if (wave_changed && lane_id == 0) atomicAdd(&U.stamp[2 + (it & 1)], wave_changed);
        traced_last = false;
        if (a.trace) {
            sum_losses((it & 1) * kParts);
            traced_last = true;
        }
        __syncthreads();
        if (a.trace && tid == 0) {
            double s = 0.0;
            if constexpr (MANY) for (int w = 0; w < kLossWaves; ++w) s = s + U.red[(it & 1) * kParts + w];
            else s = sum_of_parts(U.red + (it & 1) * kParts, kParts);
            a.trace[slot * (a.n_iter + 1) + it] = s;
        }
        // A pass that moved no row leaves every sum, hence every centroid, as it was: the labels are
        // final.  (The count is read between this pass's two barriers, or after its only one when the
        // loop ends here; no wave adds to it in between.)
        const int rows_changed = __builtin_amdgcn_readfirstlane(U.stamp[2 + (it & 1)]);
        at_fixed_point = rows_changed == 0;
        if (last_pass || rows_changed == 0) break;
        if (tid == 0) U.stamp[2 + ((it + 1) & 1)] = 0;      // the next pass counts from zero (nobody adds before the barrier below)
        const bool full_next = rows_changed > full_above;
        update_centroids<DK, kByteKnobs, SEP, PL>(U, k, KP, d, it, false, full_mode, full_next);
        full_mode = full_next;
        __syncthreads();
    }

    // ---- results: labels, loss, centroids, counts
    for (int e = lane_id; e < rows_wave; e += 64) labrow[r0 + wave_row0 + e] = (uint8_t)Queue::centroid(Q.lab()[e]);
    // the loss of the final labels: the per-wave sums of the last traced pass are still in place
    int loss_slot = ((passes_run - 1) & 1) * kParts;
    double loss = 0.0;
    if (kByteKnobs && !MANY && !traced_last && at_fixed_point) {
        // At a fixed point every non-empty centroid is the mean S / n of its cluster: the loss in integers, as in run_unit
        double *frac0 = reinterpret_cast<double *>(U.wave_base);     // the queues are idle: [k] doubles of the first wave's region
        for (int c = tid; c < k; c += blockDim.x) {
            const int nc = U.n[c];
            double fr = 0.0;
            if (nc > 0) {
                unsigned long long ss = 0;
                for (int j = 0; j < d; ++j) {
                    const long long sv = (long long)U.S[c * (DK + 1) + j] - (full_mode ? (long long)raw_offset(true) * nc : 0ll);
                    ss += (unsigned long long)(sv * sv);
                }
                const unsigned long long qc = ss / (unsigned long long)nc;
                const unsigned long long rc = ss - qc * (unsigned long long)nc;
                atomicAdd(&U.acc64[1], qc);
                fr = (double)rc / (double)nc;
            }
            frac0[c] = fr;
        }
        __syncthreads();
        if (tid == 0) {
            double fsum = 0.0;
            for (int c = 0; c < k; ++c) fsum = fsum + frac0[c];
            loss = (double)(U.acc64[0] - U.acc64[1]) - fsum;
        }
    } else {
        if (!traced_last) {
            loss_slot = 0;
            sum_losses(0);
            __syncthreads();
        }
        if (tid == 0) {
            if constexpr (MANY) for (int w = 0; w < kLossWaves; ++w) loss = loss + U.red[loss_slot + w];
            else loss = sum_of_parts(U.red + loss_slot, kParts);
        }
    }
    if (a.trace && tid == 0) {
        // the passes that were not run would have seen the same labels and centroids
        for (int it = passes_run; it <= a.n_iter; ++it) a.trace[slot * (a.n_iter + 1) + it] = loss;
    }
    for (int e = tid; e < k * d; e += blockDim.x) {
        const int c = e / d, j = e % d;
        a.centroids[(crow + c) * d + j] = U.mu64T[(size_t)j * KP + c];
    }
    for (int c = tid; c < k; c += blockDim.x) a.counts[crow + c] = U.n[c];
    if (tid == 0) {
        a.status[slot] = 0;
        a.inertia[slot] = loss;
        a.passes[slot] = passes_run;
    }
}

// Persistent workgroups (one or two per compute unit) take units from a counter until none is left: the
// next unit starts as soon as the last one ends, without a new dispatch of a workgroup of this size.
// Units are handed out in descending-k order so that the longest ones start first.
// Few tiles per wave leave registers to spare: held to 128 of them, two workgroups share a compute unit, and one's barriers and dependent LDS accesses run
// under the other's tiles.  64 tasks x 1024 rows x 12 knobs, k = 2..32: 632 -> 452 us a step; 64 tasks x
// 1000 rows x 24 knobs: 650 -> 532 us.  The price is scratch memory, in the tile loop too: with four tiles of 32-wide rows
// some single words.
constexpr bool two_workgroups(int DK, int NTW, bool SEP) { return NTW == 0 || DK == 16 || (DK == 32 && !SEP); }

// Rows that are fetched in every pass have to come from the L2 of the XCD that runs the unit (4 MiB; workgroups go to XCDs in turn),
// so tasks belong to queues, one per XCD, once the packed rows of a call exceed 3 MiB, and the units of kQueueGroup tasks (1 MiB at
// most for 32-wide rows) are handed out together.  256 tasks x 4096 x 24: one queue 17.5 ms a step, eight 14.3 ms.  A workgroup
// whose queue is empty goes on with the next one.
constexpr int kQueueGroup = 4;

// NTW = 0: rows fetched per pass (run_unit_fetched), otherwise tiles of rows a wave keeps in registers (run_unit).
template <int DK, int NTW, typename XT, bool SEP, bool MANY, int PL>
__global__ __launch_bounds__(NTW == 0 ? 1024 : 512, two_workgroups(DK, NTW, SEP) ? 4 : 2) void resident_mfma_kernel(const SweepArgs a)
{
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ int next_unit;
    const int tid = threadIdx.x;
    const int nk = a.ki_end - a.ki_begin;

    if (a.done && a.T <= 4096) {
        // a chunk in which every task has stopped: nothing to do (with very many tasks the look itself costs)
        int live = 0;
        for (int t = tid; t < a.T; t += blockDim.x) live |= a.done[t] == 0 ? 1 : 0;
        if (!__syncthreads_or(live)) return;
    }
    // (thread 0) place in a queue -> unit, moving on to the next queue when this one is empty; -1: all are
    int q = (int)blockIdx.x % a.n_queues, hops = 0;
    auto unit_of = [&](int v) -> int {
        if constexpr (NTW != 0) return v < a.T * nk ? a.T * nk - 1 - v : -1;       // one queue
        for (;;) {
            const int tasks = (a.T - q + a.n_queues - 1) / a.n_queues;
            if (v < tasks * nk) {
                const int first = v / (a.queue_group * nk) * a.queue_group;
                const int group = tasks - first < a.queue_group ? tasks - first : a.queue_group;
                const int w = v - first * nk;
                return (nk - 1 - w / group) * a.T + q + a.n_queues * (first + w % group);
            }
            if (++hops >= a.n_queues) return -1;
            q = q + 1 < a.n_queues ? q + 1 : 0;
            v = atomicAdd(a.unit_counter + q, 1);
        }
    };
    if (tid == 0) next_unit = unit_of(atomicAdd(a.unit_counter + q, 1));
    for (;;) {
        __syncthreads();
        const int u = __builtin_amdgcn_readfirstlane(next_unit);     // uniform: what derives from it lives in scalar registers
        __syncthreads();                           // everyone has read it before it is written again
        if (u < 0) break;
        // the unit after this one is asked for now; the answer is needed when this one is done
        int after = 0;
        if (tid == 0) after = atomicAdd(a.unit_counter + q, 1);
        const int ki = a.ki_begin + u / a.T;
        const int t = u % a.T;
        const int k = a.ks[ki];
        const bool skipped = a.done && a.done[t];     // the task's sweep stopped at a smaller k
        const bool too_large = a.too_large && *a.too_large != 0;     // a two-byte value the f16 rows cannot hold

        if (skipped) {
            // (its outputs were written when the task was marked)
        } else if (too_large || (a.init_mode == 0 && a.ndist[t] < k)) {
            // fewer than k distinct rows or unusable input: all outputs zero, status says which
            const int d = a.d;
            const int64_t r0 = a.task_off[t], r1 = a.task_off[t + 1];
            const int64_t slot = (int64_t)t * a.n_k + ki;
            const int64_t crow = (int64_t)t * a.Ksum + a.koff[ki];
            uint8_t *labrow = a.labbuf + (int64_t)ki * a.ld;
            for (int e = tid; e < k * d; e += blockDim.x) a.centroids[crow * d + e] = 0.0;
            for (int c = tid; c < k; c += blockDim.x) a.counts[crow + c] = 0;
            for (int64_t r = r0 + tid; r < r1; r += blockDim.x) labrow[r] = 0;
            if (tid == 0) {
                a.status[slot] = too_large ? 4 : 1;
                a.passes[slot] = 0;
                a.inertia[slot] = 0.0;
            }
            if (a.trace)
                for (int e = tid; e <= a.n_iter; e += blockDim.x) a.trace[slot * (a.n_iter + 1) + e] = 0.0;
        } else {
            if constexpr (NTW == 0) run_unit_fetched<DK, XT, SEP, MANY, PL>(a, smem, ki, t, k);
            else run_unit<DK, NTW, XT, SEP>(a, smem, ki, t, k);
        }
        if (tid == 0) next_unit = unit_of(after);   // (read by everyone after the barrier at the loop's head)
        // The compiler leaves out the wait for this write across the loop's back edge: without it a wave may
        // pass the barrier and still read the unit before (LDS requests of different SIMDs are not ordered).
        __builtin_amdgcn_s_waitcnt(0xC07F);         // lgkmcnt(0)
    }
}

template <int DK, int NTW, typename XT, bool SEP = false, bool MANY = false, int PL = 1>
hipError_t launch_mfma_t(const SweepArgs &a, int nwaves, int64_t n_max, int64_t n_total, int cus, hipStream_t s)
{
    const int KP = centroid_rows<MANY>(a.kmax);
    size_t lds;
    if constexpr (NTW == 0) {
        const unsigned per_task = (unsigned)((n_max + kPackRows - 1) / kPackRows);
        if (per_task && a.ki_begin == 0) {
            // (a launch takes less than 2^32 threads: 2^20 tasks of sixteen workgroups and more go in parts)
            const int tasks = (int)((1u << 23) / per_task);
            for (int first = 0; first < a.T; first += tasks) {
                const unsigned here = (unsigned)(a.T - first < tasks ? a.T - first : tasks);
                hipLaunchKernelGGL((pack_centred_kernel<DK, XT, SEP, PL>), dim3(per_task * here), dim3(kPackRows), 0, s, a, (int)per_task, first);
                const hipError_t e = hipGetLastError();
                if (e != hipSuccess) return e;
            }
        }
        lds = MfmaLds<DK, SEP>::base_bytes(KP) + (MANY ? ManyQueue<DK>::bytes(nwaves) : FetchedQueue<DK, PL>::kBytes) * nwaves;
    } else {
        const unsigned pb = (unsigned)((n_total + 255) / 256);
        if (pb && a.ki_begin == 0)
            hipLaunchKernelGGL((pack_rows_kernel<DK, XT>), dim3(pb), dim3(256), 0, s, reinterpret_cast<const XT *>(a.X), a.ld, a.d,
                               n_total, reinterpret_cast<_Float16 *>(a.xh), a.too_large);
        lds = MfmaLds<DK, SEP>::bytes(KP, nwaves, NTW);
    }
    SweepArgs b = a;
    b.n_queues = NTW == 0 && n_total * DK * PL * 2 > 3 * 1024 * 1024 ? kUnitQueues : 1;
    b.queue_group = b.n_queues == 1 ? a.T : kQueueGroup;
    b.loss_parts = mfma_fetches_rows(a.d, n_max) ? 1 : 0;
    auto kern = resident_mfma_kernel<DK, NTW, XT, SEP, MANY, PL>;
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    // as many workgroups as can be resident at once
    int per_cu = 0;
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, nwaves * 64, lds);
    if (e != hipSuccess) return e;
    if (per_cu < 1) per_cu = 1;
    const unsigned units = (unsigned)a.T * (unsigned)(a.ki_end - a.ki_begin);
    unsigned grid = (unsigned)cus * (unsigned)per_cu;
    if (grid > units) grid = units;
    if (grid < 1) grid = 1;
    hipLaunchKernelGGL(kern, dim3(grid), dim3(nwaves * 64), lds, s, b);
    return hipGetLastError();
}

}  // namespace

// One knob slot stays free for the bias.  Byte knobs: d <= 31, k <= 64, tasks of at most 4096 rows.
bool mfma_path_fits(int d, int kmax, int64_t n_max)
{
    return d >= 1 && d <= 31 && kmax <= 64 && n_max <= 4096;
}

// All 32 byte knobs: the bias takes a step of its own, which 4096 rows leave registers for up to k = 32
// only (one m-tile) and 2048 rows up to k = 64.
bool mfma_path_fits_d32(int d, int kmax, int64_t n_max)
{
    return d == 32 && ((kmax <= 32 && n_max <= 4096) || (kmax <= 64 && n_max <= 2048));
}

// Two-byte knobs whose values the caller promises to be below 2048: the same limits up to 31 knobs;
// up to 63 knobs in 64-wide rows, which leave registers for 2048 rows and one tile of 32 centroids.
bool mfma_path_fits_u16(int d, int kmax, int64_t n_max)
{
    if (mfma_path_fits(d, kmax, n_max)) return true;
    return d >= 1 && d <= 63 && kmax <= 32 && n_max <= 2048;
}

hipError_t compute_units(int &cus)
{
    int dev = 0;
    const hipError_t e = hipGetDevice(&dev);
    return e != hipSuccess ? e : hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
}

bool mfma_fetches_rows(int d, int64_t n_max) { return n_max > (d > 32 ? 512 : 1024); }

template <typename XT>
static hipError_t launch_mfma_sweep_t(const SweepArgs &a, int64_t n_max, int64_t n_total, hipStream_t s)
{
    const bool sep = sizeof(XT) == 1 && a.d == 32;
    // Row width: the next multiple of 16 with a slot to spare.  48 against 64 (64 tasks x 2048 rows x 40 knobs, k = 2..32):
    // six instructions per tile instead of eight and rows that fit the registers (8 spilled, not 112): 1815 -> 1530 us a step.
    const int DK = a.d <= 15 ? 16 : (a.d <= 31 || sep ? 32 : (a.d <= 47 ? 48 : 64));
    int cus = 0;
    const hipError_t e = compute_units(cus);
    if (e != hipSuccess) return e;
    const int64_t units = (int64_t)a.T * a.n_k;            // of the whole list of k: a chunk of it is run the same way
    // Few units (at most one on every second compute unit) of rows that fit the registers beside them: a sweep is then the latency of its
    // passes, and fetching pays only from there on.  us a sweep, registers / fetched, 20 steps: 16 tasks of 2048 x 32 bytes, k = 16, 167 / 200;
    // 32 tasks, k = 8, 32, 196 / 222; 64 tasks of 1536, k = 8, 32, 60 (192 units), 285 / 265; two-byte knobs: 64 tasks of up to 600 x 48, k = 2, 8,
    // 140 / 169, 8 of 600 x 40, k = 4, 16, 32, 119 / 138, but 32 of 900 x 40, k = 2..32 (992 units), 536 / 493.
    const bool few = units <= cus / 2 && ((sep && n_max <= 2048) || (a.d > 32 && n_max <= 1024));
    if (mfma_fetches_rows(a.d, n_max) && !few) {
        // One workgroup per compute unit at most: sixteen waves hide what two workgroups of eight would, if each has work enough.
        // 8 / 16 waves, us a step: one task of 4096 x 12, k = 2..64, 519 / 483, of 4096 x 24 524 / 494, of 2000 x 14 239 / 232; 4 tasks of
        // 1100 x 12 191 / 182, 6 of 2000 x 24 360 / 363.  At 32 byte knobs from more than 2048 rows on: 4 tasks of 3000 rows 390 / 375,
        // but 7 of 2000 292 / 309, 10 of up to 1200 191 / 216.
        const int nwaves = units <= cus && !(sep && n_max <= 2048) ? 16 : 8;
        if (sep) return launch_mfma_t<32, 0, uint8_t, true>(a, nwaves, n_max, n_total, cus, s);
        if (DK == 16) return launch_mfma_t<16, 0, XT>(a, nwaves, n_max, n_total, cus, s);
        if (DK == 32) return launch_mfma_t<32, 0, XT>(a, nwaves, n_max, n_total, cus, s);
        if constexpr (sizeof(XT) == 2) {
            if (DK == 48) return launch_mfma_t<48, 0, XT>(a, nwaves, n_max, n_total, cus, s);
            return launch_mfma_t<64, 0, XT>(a, nwaves, n_max, n_total, cus, s);
        }
        return hipErrorInvalidValue;        // (byte knobs never come with more than 32 knobs)
    }
    // Rows in registers: four tiles per wave hold 1024 rows in eight waves, eight 2048 (32 byte knobs, few units).  Two where one task's latency counts (no more units than
    // compute units), DK = 16, up to 512 rows: 256 rows 121 / 102 us a step, 500 rows 137 / 109 us; with many
    // units four are as good (64 tasks x 500 rows 271 / 277 us).
    const int ntw = n_max <= 512 && DK == 16 && (int64_t)a.T * (a.ki_end - a.ki_begin) <= cus ? 2 : (few && sep && n_max > 1024 ? 8 : 4);
    int nwaves = (int)((n_max + 32 * ntw - 1) / (32 * ntw));
    if (nwaves < 1) nwaves = 1;
    if (sep)
        return ntw == 8 ? launch_mfma_t<32, 8, uint8_t, true>(a, nwaves, n_max, n_total, cus, s) : launch_mfma_t<32, 4, uint8_t, true>(a, nwaves, n_max, n_total, cus, s);
    if (DK == 16)
        return ntw == 2 ? launch_mfma_t<16, 2, XT>(a, nwaves, n_max, n_total, cus, s) : launch_mfma_t<16, 4, XT>(a, nwaves, n_max, n_total, cus, s);
    if (DK == 32) return launch_mfma_t<32, 4, XT>(a, nwaves, n_max, n_total, cus, s);
    if constexpr (sizeof(XT) == 2) {
        if (DK == 48) return launch_mfma_t<48, 4, XT>(a, nwaves, n_max, n_total, cus, s);
        return launch_mfma_t<64, 4, XT>(a, nwaves, n_max, n_total, cus, s);
    }
    return hipErrorInvalidValue;
}

// k beyond 64 (byte knobs, d <= 31): within what LDS holds beside a wave's labels, and up to 7000 rows x chunks of 64 centroids. One
// compute unit has a unit's rows to itself here, the streaming kernels spread them over the chip at two launches a pass.
// us a sweep, this / streaming, 20 steps, 24 knobs, 2 and 16 tasks: k = 72, 96, 128: 1500 rows 230 / 379 and 244 / 444, 2500 rows 360 / 450 and
// 387 / 508, 4096 rows 552 / 485 and 557 / 580; k = 100, 200: 1500 rows 264 / 345 and 350 / 484, 2000 rows 363 / 397 and 448 / 459.  At the limit,
// one task of 3500 rows, k = 66: 451 / 431; 100 tasks of up to 3400, k = 65: 503 / 764.  (With 96 units of 4096 rows and k up to 128 this would be
// ahead again, 567 / 799.)
bool mfma_many_fits(int d, int kmax, int64_t n_max)
{
    return d >= 1 && d <= 31 && kmax > 64 && kmax <= kManyCentroids && n_max * ((kmax + 63) / 64) <= 7000;
}

hipError_t launch_mfma_many(const SweepArgs &a, int64_t n_max, int64_t n_total, hipStream_t s)
{
    int cus = 0;
    const hipError_t e = compute_units(cus);
    if (e != hipSuccess) return e;
    const int nwaves = a.kmax <= 192 ? 16 : 8;             // 160 KiB of LDS hold sixteen waves' regions beside 192 centroids
    if (a.d <= 15) return launch_mfma_t<16, 0, uint8_t, false, true>(a, nwaves, n_max, n_total, cus, s);
    return launch_mfma_t<32, 0, uint8_t, false, true>(a, nwaves, n_max, n_total, cus, s);
}

// Two-byte values without the promise, in two parts: rows of 64 slots up to 32 knobs, of 96 up to 48 (registers for one tile of 32
// centroids then).  The matrix kernel works for 32 (48) knobs whatever their number, the vector kernel for the next multiple of eight,
// and with 1025 to 2048 rows every lane of it has its four rows of the one step there is.  So up to 16 knobs a longer list is asked for;
// time of the vector kernel over this one's (one task and 64, cardinalities up to 32, 600 and 6000): 4 to 8 knobs, largest k 8, 0.90 at 260
// rows, 0.82 at 700, 0.68 at 2048, 0.77 at 4096; k 24, 1.1 to 1.2 up to 700 rows, 1.0 at 1100, 0.92 at 2048, 1.1 to 1.3 above; k 48, 1.15 at
// 1500.  9 to 16 knobs, k 8: 1.05 to 1.1 up to 700 rows, 0.92 to 1.03 at 1100, 0.85 to 0.94 at 2048, 1.05 to 1.25 above; k 16, 1.02 at 2048.
// 17 to 48 knobs, k 8: 1.15 to 1.9 everywhere.  (Up to 256 rows and below k = 8 calls stay where they are, on the vector kernel: even or behind up
// to 16 knobs, 1.05 to 1.4 could be had above.)
int mfma_two_part_halfs(int d, int kmax, int64_t n_max)
{
    const bool one_step = n_max > 1024 && n_max <= 2048;
    const int least = d <= 8 ? (one_step ? 33 : 24) : (d <= 16 && one_step ? 16 : 8);
    if (kmax < least || n_max <= 256) return 0;
    if (d <= 32) return kmax <= 64 && n_max <= 4096 ? 64 : 0;
    return d <= 48 && kmax <= 32 && n_max <= 2048 ? 96 : 0;
}

hipError_t launch_mfma_two_part(const SweepArgs &a, int64_t n_max, int64_t n_total, hipStream_t s)
{
    int cus = 0;
    const hipError_t e = compute_units(cus);
    if (e != hipSuccess) return e;
    // Few units, 8 / 16 waves, us a step: 4 tasks of 1500 x 31, k = 2..40, 431 / 411; above 32 knobs, with at most 2048 rows and 32
    // centroids, 4 of 1900 x 40 475 / 518, 2 of 2000 x 45 457 / 496.
    if (a.d > 32) return launch_mfma_t<48, 0, uint16_t, false, false, 2>(a, 8, n_max, n_total, cus, s);
    const int nwaves = (int64_t)a.T * a.n_k <= cus ? 16 : 8;
    return launch_mfma_t<32, 0, uint16_t, false, false, 2>(a, nwaves, n_max, n_total, cus, s);
}

hipError_t launch_mfma_sweep(const SweepArgs &a, int64_t n_max, int64_t n_total, hipStream_t s)
{
    if (a.xbytes == 2) return launch_mfma_sweep_t<uint16_t>(a, n_max, n_total, s);
    return launch_mfma_sweep_t<uint8_t>(a, n_max, n_total, s);
}

}  // namespace cham
