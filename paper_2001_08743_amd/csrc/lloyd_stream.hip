// Streaming variant of the sweep for tasks too large to stay on one compute unit
// (paper Algorithm 1, K-means.run(s_Theta, k); Sec. 3.3): every Lloyd pass is one launch of
// stream_assign_kernel over (unit, row chunk) workgroups followed by one launch of
// stream_update_kernel over units.  Labels, integer sums and counts live in global memory and are
// updated incrementally (a row touches the sums only when its label changes: exact, integers).
//
// The assignment is a pass of the resident kernel that fetches its rows (fetched_tiles.h), for up to 256
// centroids.  With at most 16 knobs every slot of the fragments holds a knob (one 16-wide
// step per part) and |mu'|^2 enters as the initial value of the accumulator, in fp32; otherwise it takes the last slot.  Up to 64
// centroids are swept at once; more are taken in chunks of 64: every chunk leaves the
// minimum score of every row and the scores within the error bound of that minimum, and the chunks
// whose minimum lies within the bound of the overall minimum contribute their marks.  A row with
// exactly one marked score is decided; any other row is re-evaluated in double against its marked
// centroids (knobs ascending, no fused multiply-add, lowest index on ties).
#include "cham_device.h"
#include "cham_internal.h"
#include "mfma_common.h"
#include "fetched_tiles.h"

namespace cham {

namespace {

constexpr int kWavesPerWg = 8;
constexpr int kLossRows = 4096;      // rows of a partial sum of the loss, whatever an assigning workgroup walks

// Knobs in 16-wide rows may fill every slot: |mu'|^2 starts the accumulator (fp32), which 32-wide rows have no registers for; those
// have a slot to spare (d <= 31) and carry it there.
template <int DK>
constexpr bool starts_from_bias() { return DK == 16; }

// Per-unit state in global memory.  KPM = kmax rounded up to 32.
struct UnitState {
    int *S;            // [KPM][32]      integer sums
    int *n;            // [KPM]          counts
    double *mu;        // [32][KPM]      exact centroids, transposed
    half8 *afrag;      // [KPM/32][4][64] A fragments (hi steps then lo steps; NS2 <= 4), centroid c in row frag_row(c)
    float *bias;       // [KPM]          |mu'|^2 (fp32), huge for padding rows, in the order of the accumulator's registers
};

__device__ __forceinline__ UnitState unit_state(const StreamArgs &a, int u)
{
    UnitState s;
    const size_t kpm = (size_t)a.kpm;
    s.S = a.Sg + (size_t)u * kpm * 32;
    s.n = a.ng + (size_t)u * kpm;
    s.mu = a.mu + (size_t)u * 32 * kpm;
    s.afrag = reinterpret_cast<half8 *>(a.afrag) + (size_t)u * (kpm / 32) * 4 * 64;
    s.bias = a.biasf + (size_t)u * kpm;
    return s;
}

// Centring offsets per task: rounded mean of the starting centroids of the largest k (any integer
// would do: it only keeps the centred magnitudes small).  Eight lanes per knob, four loads of a lane
// under way at a time: one lane per knob walked up to 256 dependent pairs of loads (28 us at k = 256).
__global__ __launch_bounds__(256) void stream_offsets_kernel(const StreamArgs a)
{
    const int t = blockIdx.x;
    const int j = threadIdx.x >> 3, part = threadIdx.x & 7;
    double s = 0.0;
    int cnt = a.kmax;
    if (a.init_mode == 0) cnt = a.ndist[t] < a.kmax ? a.ndist[t] : a.kmax;
    if (j < a.d) {
        if (a.init_mode == 0) {
            const uint8_t *col = a.X + (int64_t)j * a.ld + a.task_off[t];
            const int *rows = a.init_rows + (int64_t)t * a.kmax;
#pragma unroll 4
            for (int c = part; c < cnt; c += 8) s += (double)col[rows[c]];
        } else {
            const int64_t crow = (int64_t)t * a.Ksum + a.koff[a.n_k - 1];
#pragma unroll 4
            for (int c = part; c < cnt; c += 8) s += a.init_centroids[(crow + c) * a.d + j];
        }
    }
#pragma unroll
    for (int off = 4; off >= 1; off >>= 1) s = s + __shfl_xor(s, off, 64);
    if (part == 0) {
        double m = j < a.d && cnt > 0 ? rint(s / (double)cnt) : 0.0;
        m = m < 0.0 ? 0.0 : (m > 255.0 ? 255.0 : m);
        a.ojf[t * 32 + j] = (float)m;
    }
}

// Centred f16 copy of the rows in tiles (packed_at; absent knobs zero, 32-wide rows with the bias slot's constant) and the squared
// norm of every centred row.
template <int DK>
__global__ void stream_pack_kernel(const StreamArgs a, int64_t n_rows)
{
    const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= n_rows || r < a.task_off[0]) return;        // (rows before the first task have no place among the tiles)
    int lo = 0, hi = a.T;                      // task of row r: last t with task_off[t] <= r
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (a.task_off[mid] <= r) lo = mid; else hi = mid;
    }
    const float *o = a.ojf + lo * 32;
    float x2 = 0.0f;
    unsigned char *dst = reinterpret_cast<unsigned char *>(a.xh) + ((a.task_off[lo] >> 5) + lo) * (32 * DK * 2);
    const int in_task = (int)(r - a.task_off[lo]);
#pragma unroll
    for (int g = 0; g < DK / 8; ++g) {
        half8 v;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int j = 8 * g + i;
            float f = 0.0f;
            if (j < a.d) f = (float)a.X[(int64_t)j * a.ld + r] - o[j];
            x2 = __builtin_fmaf(f, f, x2);
            v[i] = (_Float16)f;
        }
        if (!starts_from_bias<DK>() && g == DK / 8 - 1) v[7] = (_Float16)bias_scale(true);
        *reinterpret_cast<half8 *>(dst + packed_at(in_task, g, DK)) = v;
    }
    a.x2[r] = x2;
}

// mode 0: start of the sweep (centroids from the first distinct rows or from the caller);
// mode 1: centroid update after pass a.it; mode 2: outputs after the final pass.
// Grid: (unit, tile of 32 centroids); a thread per (centroid of the tile, group of 8 knobs).  The
// bound on max |mu'|^2 is kept per tile: m2[unit][tile], tile 0 negative = unit unusable.
constexpr int kM2Tiles = 8;            // k <= 256
template <int DK>
__global__ __launch_bounds__(32 * (DK / 8)) void stream_update_kernel(const StreamArgs a, int mode)
{
    constexpr int NS = DK / 16, G = DK / 8;
    __shared__ float red[32 * G / 64 + 1];
    const int ul = blockIdx.x;                 // unit within this launch
    const int mt = blockIdx.y;                 // tile of 32 centroids
    const int u = a.u_begin + ul;
    const int ki = a.n_k - 1 - u / a.T;
    const int t = u % a.T;
    const int k = a.ks[ki];
    const int d = a.d;
    const int tid = threadIdx.x;
    const int64_t slot = (int64_t)t * a.n_k + ki;
    const int64_t crow = (int64_t)t * a.Ksum + a.koff[ki];
    const int64_t r0 = a.task_off[t], r1 = a.task_off[t + 1];
    const UnitState st = unit_state(a, u);
    const int kpm = a.kpm;
    const bool skipped = a.done && a.done[t];  // the task's sweep stopped at a smaller k
    const bool unusable = skipped || (a.init_mode == 0 && a.ndist[t] < k);

    if (unusable) {
        if (mt != 0) return;
        if (mode == 0 && tid == 0) a.m2[u * kM2Tiles] = -1.0f;
        if (mode == 2 && !skipped) {           // (the outputs of a skipped unit were written when its task was marked)
            for (int e = tid; e < k * d; e += blockDim.x) a.centroids[crow * d + e] = 0.0;
            for (int c = tid; c < k; c += blockDim.x) a.counts[crow + c] = 0;
            uint8_t *labrow = a.labbuf + (int64_t)ki * a.ld;
            for (int64_t r = r0 + tid; r < r1; r += blockDim.x) labrow[r] = 0;
            if (tid == 0) {
                a.status[slot] = 1;
                a.passes[slot] = 0;
                a.inertia[slot] = 0.0;
            }
            if (a.trace)
                for (int e = tid; e <= a.n_iter; e += blockDim.x) a.trace[slot * (a.n_iter + 1) + e] = 0.0;
        }
        return;
    }

    // loss of the pass that just ran: partials in row order
    if (mt == 0 && mode != 0 && tid == 0 && (mode == 2 || a.trace)) {
        const int np = (int)((r1 - r0 + kLossRows - 1) / kLossRows);
        double s = 0.0;
        const double *part = a.rows_per_wg < kLossRows ? reinterpret_cast<const double *>(st.S) : a.loss_part + a.wg_off[ul];
#pragma unroll 8
        for (int b = 0; b < np; ++b) s = s + part[b];
        if (a.trace) a.trace[slot * (a.n_iter + 1) + a.it] = s;
        if (mode == 2) {
            a.inertia[slot] = s;
            a.status[slot] = 0;
            // up to and including the first pass that moved no row (a pass launched after it returns at once)
            a.passes[slot] = a.trace ? a.n_iter + 1 : a.passes[slot] + 1;
        }
    }
    if (mode == 0 && mt == 0 && tid == 0) a.passes[slot] = 0;
    // the pass moved no row of the unit: every sum, hence every centroid, is what it was
    if (mode == 1 && !a.trace && a.passes[slot] <= a.it) return;
    const int kpu = (k + 31) & ~31;
    if (mt * 32 >= kpu) return;                // no such tile in this unit
    if (mode == 2) {
        for (int e = tid; e < 32 * d; e += blockDim.x) {
            const int c = mt * 32 + e / d, j = e % d;
            if (c < k) a.centroids[(crow + c) * d + j] = st.mu[(size_t)j * kpm + c];
        }
        for (int c = mt * 32 + tid; c < k && c < mt * 32 + 32; c += blockDim.x) a.counts[crow + c] = st.n[c];
        return;
    }

    const float *o = a.ojf + t * 32;
    const int m32 = tid / G, g = tid % G;
    const int c = mt * 32 + m32;
    if (mode == 0) {
        if (g == 0) st.n[c] = 0;
#pragma unroll
        for (int i = 0; i < 8; ++i) st.S[c * 32 + 8 * g + i] = 0;
        if (DK == 16) {
#pragma unroll
            for (int i = 0; i < 8; ++i) st.S[c * 32 + 16 + 8 * g + i] = 0;
        }
    }
    const int cnt = (mode == 1 && c < k) ? st.n[c] : 0;
    double b = 0.0;
    half8 hi8, lo8;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int j = 8 * g + i;
        double m = 0.0;
        if (c < k && j < d) {
            double mu;
            if (mode == 0) {
                if (a.init_mode == 0) mu = (double)a.X[(int64_t)j * a.ld + r0 + a.init_rows[(int64_t)t * a.kmax + c]];
                else mu = a.init_centroids[(crow + c) * d + j];
                st.mu[(size_t)j * kpm + c] = mu;
            } else if (cnt > 0) {
                mu = (double)st.S[c * 32 + j] / (double)cnt;      // an empty cluster keeps its centroid
                st.mu[(size_t)j * kpm + c] = mu;
            } else {
                mu = st.mu[(size_t)j * kpm + c];
            }
            m = mu - (double)o[j];
        } else if (mode == 0 && c < k) {
            st.mu[(size_t)j * kpm + c] = 0.0;
        }
        b = __builtin_fma(m, m, b);
        const float w = __builtin_amdgcn_fmed3f((float)(-2.0 * m), -kHalfMax, kHalfMax);
        const _Float16 hi = (_Float16)w;
        hi8[i] = hi;
        lo8[i] = (_Float16)(w - (float)hi);
    }
    // |mu'|^2 over all knob groups of the centroid (the G lanes of a centroid are neighbours)
#pragma unroll
    for (int off = G / 2; off >= 1; off >>= 1) b = b + __shfl_xor(b, off, 64);
    // padding centroid rows get a score above all others
    if (starts_from_bias<DK>()) {
        if (g == G - 1) st.bias[mt * 32 + 16 * (c & 1) + (m32 >> 1)] = c < k ? __builtin_fminf((float)b, kFarScore) : kPadScore;
    } else if (g == G - 1) {
        const float bs = c < k ? __builtin_fminf((float)b * (1.0f / bias_scale(true)), kHalfMax) : kHalfMax;
        hi8[7] = (_Float16)bs;
        lo8[7] = (_Float16)(bs - (float)hi8[7]);
    }
    const int hh = g & 1, fstep = g >> 1;
    st.afrag[(mt * 4 + fstep) * 64 + 32 * hh + frag_row(m32)] = hi8;
    st.afrag[(mt * 4 + NS + fstep) * 64 + 32 * hh + frag_row(m32)] = lo8;

    float bmax = c < k ? __double2float_ru(b) * 1.0000005f : 0.0f;
    // a start (or an empty cluster still there) so far off that an operand may have been clamped: every centroid
    // is a candidate of every row
    if (!(bmax <= (starts_from_bias<DK>() ? kHalfMax * kHalfMax / 4.0f : max_screened(true)))) bmax = kFarNorm;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) bmax = __builtin_fmaxf(bmax, __shfl_xor(bmax, off, 64));
    if ((tid & 63) == 0) red[tid >> 6] = bmax;
    __syncthreads();
    if (tid == 0) {
        float m = 0.0f;
        for (int i = 0; i < (int)(blockDim.x + 63) / 64; ++i) m = __builtin_fmaxf(m, red[i]);
        a.m2[u * kM2Tiles + mt] = m;
    }
}

template <int DK>
struct StreamLds {
    half8 *afrag;        // [KPM/32][2*DK/16][64]
    float *bias;         // [KPM]
    int *S;              // [KPM][DK+1] changes of the sums made by this workgroup
    int *n;              // [KPM]
    int *dirty;          // [KPM] (written beside the sizes; not used here)
    float *ojf;          // [DK]
    unsigned char *wave_base;
    static __host__ __device__ size_t wave_bytes(bool many) { return many ? ManyQueue<DK>::bytes(kWavesPerWg) : FetchedQueue<DK>::kBytes; }
    __host__ __device__ static size_t bytes(int kpm)
    {
        size_t b = 16 * (size_t)(kpm / 32) * (2 * DK / 16) * 64 + sizeof(float) * kpm + sizeof(int) * (size_t)kpm * (DK + 1) +
                   sizeof(int) * kpm * 2 + sizeof(float) * DK;
        b = (b + 15) & ~(size_t)15;
        const size_t wave = wave_bytes(false);
        return b + (kpm > 64 && wave_bytes(true) > wave ? wave_bytes(true) : wave) * kWavesPerWg;      // (units of either form)
    }
    __device__ StreamLds(unsigned char *base, int kpm)
    {
        size_t o = 0;
        afrag = reinterpret_cast<half8 *>(base + o);  o += 16 * (size_t)(kpm / 32) * (2 * DK / 16) * 64;
        bias = reinterpret_cast<float *>(base + o);   o += sizeof(float) * kpm;
        S = reinterpret_cast<int *>(base + o);        o += sizeof(int) * (size_t)kpm * (DK + 1);
        n = reinterpret_cast<int *>(base + o);        o += sizeof(int) * kpm;
        dirty = reinterpret_cast<int *>(base + o);    o += sizeof(int) * kpm;
        ojf = reinterpret_cast<float *>(base + o);    o += sizeof(float) * DK;
        o = (o + 15) & ~(size_t)15;
        wave_base = base + o;
    }
};

// One (unit, row chunk) workgroup of the assignment: a pass of the resident kernel that fetches its rows, over at most 512 rows
// per wave, with the unit's state in global memory.  128 registers a wave let two workgroups of eight waves share a compute unit
// where LDS holds them (k <= 192, or d <= 16): with four waves of 256 registers, steps of four or eight tiles and every row
// decided afresh in every pass, the vector ALU was busy less than half of the time.  MANY: k > 64.
template <int DK, bool MANY>
__device__ __forceinline__ void assign_unit(const StreamArgs &a, int unit_idx)
{
    constexpr int NS2 = 2 * DK / 16;
    constexpr bool CIN = starts_from_bias<DK>();
    typedef typename std::conditional<MANY, ManyQueue<DK>, FetchedQueue<DK>>::type Queue;
    extern __shared__ __align__(16) unsigned char smem[];
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wgi = blockIdx.x - a.wg_off[unit_idx];
    const int u = a.u_begin + unit_idx;
    const int ki = a.n_k - 1 - u / a.T;
    const int t = u % a.T;
    const int k = a.ks[ki];
    const int d = a.d;
    const int kpm = a.kpm;
    const int kpu = (k + 31) & ~31;
    float m2 = a.m2[u * kM2Tiles];
    if (m2 < 0.0f) return;                     // unusable unit (fewer than k distinct rows)
    // The pass before moved no row: sums and centroids are what that pass used, so this one would move
    // none either.  (passes holds 1 + the last pass that moved a row; a workgroup of this pass may
    // raise it to it + 1 meanwhile, but only in a unit that none of them skips.)  A traced sweep runs
    // every pass.
    int *moved_at = a.passes + (int64_t)t * a.n_k + ki;
    if (a.it > 0 && !a.trace && *moved_at < a.it) return;
    for (int i = 1; i < kpu / 32; ++i) m2 = __builtin_fmaxf(m2, a.m2[u * kM2Tiles + i]);
    const UnitState st = unit_state(a, u);
    StreamLds<DK> L(smem, kpm);
    auto region = [&]() {
        if constexpr (MANY) return Queue(L.wave_base + Queue::bytes(kWavesPerWg) * wave, kWavesPerWg);
        else return Queue(L.wave_base + Queue::kBytes * wave);
    };
    const Queue Q = region();

    const int64_t t0 = a.task_off[t], t1 = a.task_off[t + 1];
    const int first_row = wgi * a.rows_per_wg;                     // of the chunk, within the task
    const int left = (int)(t1 - t0) - first_row;
    const int run = a.rows_per_wg / kWavesPerWg;                   // rows of a wave: whole groups of 64
    const int wave_row0 = first_row + wave * run;
    const int here = (left < a.rows_per_wg ? left : a.rows_per_wg) - wave * run;
    const int rows_wave = here < 0 ? 0 : (here < run ? here : run);
    const bool first = a.it == 0;
    uint8_t *labrow = a.labbuf + (int64_t)ki * a.ld + t0 + wave_row0;
    const unsigned char *packed = reinterpret_cast<const unsigned char *>(a.xh) + ((t0 >> 5) + t) * (32 * DK * 2) +
                                  (size_t)(rows_wave ? wave_row0 : 0) * (DK * 2);

    // the labels so far (0xFF: none): both tables, in their stored form
    {
        unsigned char c[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) c[i] = !first && 64 * i + lane < rows_wave ? labrow[64 * i + lane] : 0;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int r = 64 * i + lane;
            const unsigned char v = !first && r < rows_wave ? (unsigned char)Queue::stored(c[i]) : 0xFFu;
            Q.lab()[r] = v;
            Q.lab_new()[r] = v;
        }
    }
    for (int e = tid; e < (kpu / 32) * NS2 * 64; e += blockDim.x)        // the NS2 slots in use of every m-tile
        L.afrag[e] = st.afrag[(e / (NS2 * 64)) * 4 * 64 + e % (NS2 * 64)];
    if (CIN)
        for (int e = tid; e < kpu; e += blockDim.x) L.bias[e] = st.bias[e];
    for (int e = tid; e < k * (DK + 1); e += blockDim.x) L.S[e] = 0;
    for (int c = tid; c < k; c += blockDim.x) L.n[c] = 0;
    if (tid < DK) L.ojf[tid] = a.ojf[t * 32 + tid];
    __syncthreads();

    // the bound of a row, as a constant and a multiple of its squared norm
    constexpr float kPerNorm = mfma_bound_slope<NS2>();
    const Tiles tiles = {packed, L.afrag, nullptr, L.bias, a.x2 + t0 + wave_row0, mfma_bound<NS2>(0.0f, m2), kPerNorm, bias_scale(true),
                         (rows_wave + 31) >> 5, rows_wave, first ? ~0ull : 0ull};
    int nrec = 0;
    if constexpr (MANY) {
        decide_tiles_many<DK, CIN, true>(Q, tiles, nrec, st.mu, L.ojf, kpm, k, d, lane);
    } else if (rows_wave) {
        const bool two = k > 32;
        const int lregs = (((two ? k - 32 : k) + 1) / 2 + 3) & ~3;       // live accumulator registers of the last m-tile
        int nt = 0;
        do {
            auto live_pass = [&](auto two_tag) {
                constexpr bool TWO = decltype(two_tag)::value;
                switch (lregs) {
                case 4: nt = decide_tiles<DK, false, CIN, true, 4, TWO>(Q, tiles, nt, nrec, lane); break;
                case 8: nt = decide_tiles<DK, false, CIN, true, 8, TWO>(Q, tiles, nt, nrec, lane); break;
                case 12: nt = decide_tiles<DK, false, CIN, true, 12, TWO>(Q, tiles, nt, nrec, lane); break;
                default: nt = decide_tiles<DK, false, CIN, true, 16, TWO>(Q, tiles, nt, nrec, lane); break;
                }
            };
            if (two) live_pass(std::true_type{});
            else live_pass(std::false_type{});
            resolve_batches<DK, 1>(Q, nrec, packed, st.mu, L.ojf, kpm, k, d, lane);
            nrec = 0;
        } while (nt < tiles.ntiles);
    }

    // ---- label changes -> labels in memory, changes of the sums in LDS; a lane compares four rows at a time
    bool moved = false;
    {
        const uint64_t below = (1ull << lane) - 1ull;
        int cnt = 0;
        __builtin_amdgcn_wave_barrier();
        for (int base = 0; base < rows_wave; base += 256) {
            const int at = base + 4 * lane;
            const unsigned cur4 = *reinterpret_cast<const unsigned *>(Q.lab_new() + at);
            const unsigned prev4 = *reinterpret_cast<const unsigned *>(Q.lab() + at);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const unsigned cur = (cur4 >> (8 * i)) & 0xFFu, prev = (prev4 >> (8 * i)) & 0xFFu;
                const bool changed = first ? at + i < rows_wave : cur != prev;
                const uint64_t cm = __ballot(changed);
                if (!cm) continue;
                const int add = __popcll(cm);
                moved = true;
                if (cnt + add > Queue::kChanges) {
                    apply_listed<DK>(Q, cnt, packed, L.S, L.n, L.dirty, L.ojf, d, 0);
                    cnt = 0;
                }
                if (changed) {
                    const unsigned c = Queue::centroid(cur);
                    labrow[at + i] = (uint8_t)c;
                    // (a first label is told by a place of its own: the number 255 is a centroid here)
                    Q.changes()[cnt + __popcll(cm & below)] = c | (first ? 0u : Queue::centroid(prev)) << 8 | (unsigned)(at + i) << 16 | (first ? 0x80000000u : 0u);
                }
                cnt += add;
            }
        }
        if (cnt) apply_listed<DK>(Q, cnt, packed, L.S, L.n, L.dirty, L.ojf, d, 0);
    }

    const bool any_moved = __syncthreads_or(moved ? 1 : 0) != 0;
    // changes of this workgroup -> the unit's sums (which nothing reads after the final pass)
    if (any_moved && !a.final_pass) {
        if (tid == 0) *moved_at = a.it + 1;
        for (int e = tid; e < k * DK; e += blockDim.x) {
            const int v = L.S[(e / DK) * (DK + 1) + e % DK];
            if (v != 0) atomicAdd(&st.S[(e / DK) * 32 + (e % DK)], v);
        }
    }
    if (any_moved) for (int c = tid; c < k; c += blockDim.x) {
        const int v = L.n[c];
        if (v != 0) atomicAdd(&st.n[c], v);
    }
}

// Unit of this workgroup: the last one with wg_off[unit] <= blockIdx.x, by a 64-way search of the first
// wave (one or two rounds of independent loads instead of a chain of dependent ones).
__device__ __forceinline__ int unit_of_block(const StreamArgs &a, int *unit_sh)
{
    const int tid = threadIdx.x;
    if (tid < 64) {
        int lo = 0, hi = a.n_units;
        while (hi - lo > 1) {
            const int span = hi - lo;
            const int stride = (span + 63) / 64;
            const int probe = lo + tid * stride;
            const bool le = probe < hi && a.wg_off[probe] <= (int)blockIdx.x;     // true for a prefix of the lanes
            const int cntle = __popcll(__ballot(le));                              // >= 1: wg_off[lo] <= blockIdx.x
            const int nlo = lo + (cntle - 1) * stride;
            const int nhi = nlo + stride < hi ? nlo + stride : hi;
            lo = nlo;
            hi = nhi;
        }
        if (tid == 0) *unit_sh = lo;
    }
    __syncthreads();
    return __builtin_amdgcn_readfirstlane(*unit_sh);
}

template <int DK>
__global__ __launch_bounds__(kWavesPerWg * 64, 4) void stream_assign_kernel(const StreamArgs a)
{
    __shared__ int unit_sh;
    const int unit_idx = unit_of_block(a, &unit_sh);
    const int u = a.u_begin + unit_idx;
    const int k = a.ks[a.n_k - 1 - u / a.T];
    // the unit index goes through an opaque copy per variant: what a variant derives from it stays inside
    // its branch instead of being computed for both ahead of the branch (scalar registers)
    int ui = unit_idx;
    if (k <= 64) {
        asm volatile("" : "+s"(ui));
        assign_unit<DK, false>(a, ui);
    } else {
        asm volatile("" : "+s"(ui));
        assign_unit<DK, true>(a, ui);
    }
}

// Loss of the labels of the pass that just ran (the final one, or every one of a traced sweep): one
// workgroup per kLossRows rows of a unit, whatever the assigning workgroups walk.  How the rows are split
// among those depends on the batch and on the chunk of the list of k, and the knee rule compares the losses,
// so the order of the sum must not: the terms of all rows go to LDS, then lane l of four waves adds up rows l,
// l + 64, ... of its wave's runs of consecutive rows (128, or 256 with at most 16 knobs and k <= 64), then
// the lanes, the waves and, in the update kernel, the blocks of kLossRows.  Bound by the latency of the
// centroids' gathers, hence from LDS: a step of 171 256 x 14, k = 64 and 128 (84 workgroups), takes 529 us, 545 us
// with gathers from memory and 536 us with the loss inside the assignment, where it cost registers.
// Not unrolled over all knobs: the addresses of 32 loads in scalar registers cost more than their overlap gains
// (pools of 21 000 to 60 000 x 23 1356 / 1343 us a step); 512 or 256 threads and more rows under way are slower.
template <int DK>
__global__ __launch_bounds__(1024) void stream_loss_kernel(const StreamArgs a)
{
    extern __shared__ __align__(16) unsigned char smem[];
    double *term = reinterpret_cast<double *>(smem);               // [kLossRows]
    double *mu_sh = term + kLossRows;                              // [d][KPM] centroids
    __shared__ double red[kLossWaves];
    __shared__ int unit_sh;
    const int tid = threadIdx.x;
    const int unit_idx = unit_of_block(a, &unit_sh);
    const int first = ((int)blockIdx.x - a.wg_off[unit_idx]) * a.rows_per_wg;     // of the assigning workgroup of this index
    const int u = a.u_begin + unit_idx;
    if (first % kLossRows != 0 || a.m2[u * kM2Tiles] < 0.0f) return;              // inside another block, or an unusable unit
    const int ki = a.n_k - 1 - u / a.T;
    const int t = u % a.T;
    const int64_t r0 = a.task_off[t] + first, t1 = a.task_off[t + 1];
    const int n = (int)(t1 - r0 < kLossRows ? t1 - r0 : kLossRows);
    const int k = a.ks[ki], d = a.d, kpm = a.kpm;
    const UnitState st = unit_state(a, u);
    const uint8_t *lab = a.labbuf + (int64_t)ki * a.ld + r0;
    for (int e = tid; e < d * kpm; e += blockDim.x) mu_sh[e] = st.mu[e];
    __syncthreads();
    for (int r = tid; r < n; r += blockDim.x) {
        const int c = lab[r];
        double s = 0.0;
        for (int j0 = 0; j0 < d; j0 += 8) {                        // eight knob values under way at a time
            uint8_t xv[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) xv[i] = a.X[(int64_t)(j0 + i < d ? j0 + i : 0) * a.ld + r0 + r];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                if (j0 + i < d) {
                    const double tq = (double)xv[i] - mu_sh[(j0 + i) * kpm + c];
                    s = s + tq * tq;
                }
            }
        }
        term[r] = s;
    }
    __syncthreads();
    if (tid < kLossWaves * 64) {
        const int run = loss_run(d, k);
        double part = 0.0;
        for (int base = (tid >> 6) * run; base < n; base += kLossWaves * run)
            for (int r = base + (tid & 63); r < base + run; r += 64)
                if (r < n) part = part + term[r];
        const double ws = wave_sum(part);
        if ((tid & 63) == 0) red[tid >> 6] = ws;
    }
    __syncthreads();
    if (tid == 0) {
        double s = 0.0;
        for (int w = 0; w < kLossWaves; ++w) s = s + red[w];
        // with fewer rows per workgroup the partials stand in the unit's sums, which nothing reads any more
        if (a.rows_per_wg < kLossRows) reinterpret_cast<double *>(st.S)[first / kLossRows] = s;
        else a.loss_part[blockIdx.x] = s;
    }
}

template <int DK>
hipError_t run_stream(StreamArgs a, int64_t n_total, int total_wgs, hipStream_t s)
{
    const size_t lds = StreamLds<DK>::bytes(a.kpm);
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(stream_assign_kernel<DK>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    const size_t lds_loss = sizeof(double) * ((size_t)kLossRows + (size_t)a.d * a.kpm);      // at most 96 KiB
    e = hipFuncSetAttribute(reinterpret_cast<const void *>(stream_loss_kernel<DK>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_loss);
    if (e != hipSuccess) return e;
    if (a.prepare) {
        hipLaunchKernelGGL(stream_offsets_kernel, dim3(a.T), dim3(256), 0, s, a);
        const unsigned pb = (unsigned)((n_total + 255) / 256);
        if (pb) hipLaunchKernelGGL(stream_pack_kernel<DK>, dim3(pb), dim3(256), 0, s, a, n_total);
    }
    a.it = 0;
    a.final_pass = 0;
    const dim3 ugrid(a.n_units, a.kpm / 32), ublock(32 * (DK / 8));
    hipLaunchKernelGGL(stream_update_kernel<DK>, ugrid, ublock, 0, s, a, 0);
    for (int it = 0; it <= a.n_iter; ++it) {
        a.it = it;
        a.final_pass = it == a.n_iter ? 1 : 0;
        hipLaunchKernelGGL(stream_assign_kernel<DK>, dim3(total_wgs), dim3(kWavesPerWg * 64), lds, s, a);
        if (a.final_pass || a.trace) hipLaunchKernelGGL(stream_loss_kernel<DK>, dim3(total_wgs), dim3(1024), lds_loss, s, a);
        hipLaunchKernelGGL(stream_update_kernel<DK>, ugrid, ublock, 0, s, a, a.final_pass ? 2 : 1);
    }
    return hipGetLastError();
}

}  // namespace

int64_t stream_lds_bytes(int d, int kpm)
{
    return d <= 16 ? (int64_t)StreamLds<16>::bytes(kpm) : (int64_t)StreamLds<32>::bytes(kpm);
}

hipError_t launch_stream_sweep(const StreamArgs &a, int64_t n_total, int total_wgs, hipStream_t s)
{
    if (a.d <= 16) return run_stream<16>(a, n_total, total_wgs, s);
    return run_stream<32>(a, n_total, total_wgs, s);
}

}  // namespace cham
