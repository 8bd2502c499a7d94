// Pieces shared by the matrix-core kernels that fetch their rows from packed tiles in every pass: the whole iteration of a unit in
// one workgroup (lloyd_mfma.hip) and one pass over a run of rows (lloyd_stream.hip).  Lane exchanges, the layout of scores and
// packed rows, the tables of a wave, the tile loops, the exact evaluation of undecided rows, label changes and the rebuild of
// sums.  The files are compiled with -fno-honor-nans.
#pragma once
#include <type_traits>

#include "cham_device.h"
#include "mfma_common.h"

namespace cham {

namespace {

// Cross-lane exchanges done in the vector ALU (DPP), no LDS round trip.
// xor_lanes<1|2|4|8>: the value held by lane ^ 1, 2, 4 or 8.
template <int XOR>
__device__ __forceinline__ int dpp_xor_i32(int v)
{
    if (XOR == 8) return __builtin_amdgcn_update_dpp(0, v, 0x128, 0xF, 0xF, false);     // row_ror:8 = lane ^ 8 within a row of 16
    if (XOR == 1) return __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xF, 0xF, false);      // quad_perm [1,0,3,2]
    if (XOR == 2) return __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xF, 0xF, false);      // quad_perm [2,3,0,1]
    // lane ^ 4 = mirror within each group of eight lanes, then reverse within each quad
    const int m = __builtin_amdgcn_update_dpp(0, v, 0x141, 0xF, 0xF, false);            // row_half_mirror
    return __builtin_amdgcn_update_dpp(0, m, 0x1B, 0xF, 0xF, false);                    // quad_perm [3,2,1,0]
}
template <int XOR>
__device__ __forceinline__ double dpp_xor_f64(double v)
{
    const long long b = __double_as_longlong(v);
    const int lo = dpp_xor_i32<XOR>((int)(b & 0xFFFFFFFFll));
    const int hi = dpp_xor_i32<XOR>((int)(b >> 32));
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
// maximum of a non-negative float over the wave: rotations within the 16-lane rows, then the four
// row results through scalar registers
__device__ __forceinline__ float wave_max_nonneg(float v)
{
    int b = __float_as_int(v);          // non-negative floats order like integers
    int o = __builtin_amdgcn_update_dpp(0, b, 0x128, 0xF, 0xF, false);    // row_ror:8
    b = b > o ? b : o;
    o = __builtin_amdgcn_update_dpp(0, b, 0x124, 0xF, 0xF, false);        // row_ror:4
    b = b > o ? b : o;
    o = __builtin_amdgcn_update_dpp(0, b, 0x122, 0xF, 0xF, false);        // row_ror:2
    b = b > o ? b : o;
    o = __builtin_amdgcn_update_dpp(0, b, 0x121, 0xF, 0xF, false);        // row_ror:1
    b = b > o ? b : o;
    const int r0 = __builtin_amdgcn_readlane(b, 0), r1 = __builtin_amdgcn_readlane(b, 16);
    const int r2 = __builtin_amdgcn_readlane(b, 32), r3 = __builtin_amdgcn_readlane(b, 48);
    const int m01 = r0 > r1 ? r0 : r1, m23 = r2 > r3 ? r2 : r3;
    return __int_as_float(m01 > m23 ? m01 : m23);
}

// Minimum of two / three scores.  This file is compiled with -fno-honor-nans (every score is a finite
// sum of finite products), which spares the instruction that would otherwise quiet a possible NaN in
// each operand coming out of a matrix instruction.  (Not inline assembly: the compiler has to see
// these reads to keep the wait states between a matrix instruction and the use of its result.)
__device__ __forceinline__ float vmin(float a, float b) { return __builtin_fminf(a, b); }
__device__ __forceinline__ float vmin3(float a, float b, float c) { return __builtin_fminf(__builtin_fminf(a, b), c); }

// Score position -> centroid.  Position q = 16 * m-tile + accumulator register (the order in which
// the mask bits are collected, most significant first), hh = lane half.
__device__ __forceinline__ int slot_centroid(int q, int hh) { return 2 * q + hh; }
// Mask of the positions (bit 31 = position 0) of lane half hh that hold centroids below kk.
__device__ __forceinline__ uint32_t marks_below(int kk, int hh)
{
    const int n = (kk + 1 - hh) >> 1;
    return n <= 0 ? 0u : (n >= 32 ? 0xFFFFFFFFu : ~(0xFFFFFFFFu >> n));
}
// Row of the 32-row A fragment that holds centroid c of its m-tile.
__device__ __forceinline__ int frag_row(int c)
{
    const int i = (c & 31) >> 1;
    return 8 * (i >> 2) + 4 * (c & 1) + (i & 3);
}

// The packed copy holds tiles of 32 rows in the order of B fragments: eight knobs (16 bytes) of row n, knob group g of a tile stand at
// byte 1024 (g / 2) + 512 (g & 1) + 16 n, so that one load of a fragment reads 1024 bytes in a row.  (One row after the
// other a load touched 16 lines of 128 bytes and half of each: 56 accesses to the vector cache per load instead of 16, which
// kept it busy two thirds of the sweep.)  Task t starts at tile task_off[t] / 32 + t, which leaves every task room for its last tile.
__device__ __forceinline__ size_t packed_at(int row, int g, int DK)
{
    return (size_t)(row >> 5) * (32 * DK * 2) + (g >> 1) * 1024 + (g & 1) * 512 + (row & 31) * 16;
}
// Resolve the queued rows of this wave: four lanes per row, each lane takes every fourth marked
// centroid of its row and evaluates the exact double distance (knobs ascending, no fused
// multiply-add); the four lanes then agree on the smallest distance, lowest index on ties.  The
// result goes to the row's entry of the labels of the pass under way.
template <int DK, typename Queue>
__device__ __forceinline__ void resolve_rows(const Queue &Q, int nrec, const double *mu64T,
                                             const float *ojf, int KP, int k, int d)
{
    const int lane = threadIdx.x & 63;
    const int q = lane & 3;
    __builtin_amdgcn_wave_barrier();
    for (int r0 = 0; r0 < nrec; r0 += 16) {
        const int r = r0 + (lane >> 2);
        const bool have = r < nrec;
        const int rr = have ? r : 0;
        unsigned rem0 = 0, rem1 = 0;
        if (have) {
            rem0 = Q.rec_mask()[r * 2 + 0];
            rem1 = Q.rec_mask()[r * 2 + 1];
        }
        const int pid = Q.rec_pid()[rr];
        // next marked centroid of the row, -1 when none is left
        auto pop = [&]() -> int {
            int c = -1;
            if (rem0) {
                const int b = __clz((int)rem0);
                rem0 &= ~(0x80000000u >> b);
                c = slot_centroid(b, 0);
            } else if (rem1) {
                const int b = __clz((int)rem1);
                rem1 &= ~(0x80000000u >> b);
                c = slot_centroid(b, 1);
            }
            return c;
        };
        for (int i = 0; i < q; ++i) pop();
        double bs = __builtin_inf();
        int bc = 0x7fffffff;
        while (__ballot((rem0 | rem1) != 0u)) {
            const int cc = pop();
            const int ci = (cc < 0 || cc >= k) ? 0 : cc;
            double ss = 0.0;
            // knobs in groups of 8; the loads of a group are independent and overlap
            for (int j0 = 0; j0 < d; j0 += 8) {
                const _Float16 *xr = Q.rec_x() + (size_t)rr * (DK * Queue::kPlanes) + j0;
                const half8 xq = *reinterpret_cast<const half8 *>(xr);
                half8 xs = xq;                   // (the second part of a value, where there is one)
                if (Queue::kPlanes == 2) xs = *reinterpret_cast<const half8 *>(xr + DK);
                const float4 oa = *reinterpret_cast<const float4 *>(ojf + j0);
                const float4 ob = *reinterpret_cast<const float4 *>(ojf + j0 + 4);
                const float of[8] = {oa.x, oa.y, oa.z, oa.w, ob.x, ob.y, ob.z, ob.w};
                double mu[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) mu[i] = mu64T[(size_t)(j0 + i) * KP + ci];
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    // queued copies are centred; padded knobs are skipped (the last one carries the bias)
                    float xf = (float)xq[i] + of[i];
                    if (Queue::kPlanes == 2) xf += (float)xs[i];
                    if (j0 + i >= d) xf = 0.0f;
                    const double tq = (double)xf - mu[i];
                    ss = ss + tq * tq;
                }
            }
            if (cc >= 0 && cc < k && (ss < bs || (ss == bs && cc < bc))) {
                bs = ss;
                bc = cc;
            }
            pop();
            pop();
            pop();
        }
        {
            const double os = dpp_xor_f64<1>(bs);
            const int oc = dpp_xor_i32<1>(bc);
            if (os < bs || (os == bs && oc < bc)) {
                bs = os;
                bc = oc;
            }
        }
        {
            const double os = dpp_xor_f64<2>(bs);
            const int oc = dpp_xor_i32<2>(bc);
            if (os < bs || (os == bs && oc < bc)) {
                bs = os;
                bc = oc;
            }
        }
        if (have && q == 0) Q.lab_new()[pid] = (unsigned char)Queue::stored(bc < k ? bc : 0);
    }
    __builtin_amdgcn_wave_barrier();
}

// A few queued rows (the usual case): two rows at a time, two marked centroids per row at a time,
// sixteen lanes per (row, centroid): every lane squares the differences of its one or two knobs,
// then one lane adds the d squares up in knob order (the only part that has to be serial) and the
// lanes of a row agree on the smallest distance, lowest index on ties.
template <int DK, typename Queue>
__device__ __forceinline__ void resolve_few(const Queue &Q, int nrec, const double *mu64T,
                                            const float *ojf, int KP, int k, int d)
{
    const int lane = threadIdx.x & 63;
    const int slot = lane >> 4, jl = lane & 15;
    double *sc = Q.few() + slot * 32;      // squares of one (row, centroid)
    __builtin_amdgcn_wave_barrier();
    for (int r0 = 0; r0 < nrec; r0 += 2) {
        const int r = r0 + (slot >> 1);
        const bool have = r < nrec;
        const int rr = have ? r : 0;
        unsigned rem0 = 0, rem1 = 0;
        if (have) {
            rem0 = Q.rec_mask()[r * 2 + 0];
            rem1 = Q.rec_mask()[r * 2 + 1];
        }
        const int pid = Q.rec_pid()[rr];
        // this lane's knobs of the row (the queued copy is centred; the bias slot and padded slots count as zero)
        float xa = 0.0f, xb = 0.0f;
        const _Float16 *xr = Q.rec_x() + (size_t)rr * (DK * Queue::kPlanes) + jl;
        if (jl < d) xa = (float)xr[0] + ojf[jl] + (Queue::kPlanes == 2 ? (float)xr[DK] : 0.0f);
        if (DK == 32 && jl + 16 < d) xb = (float)xr[16] + ojf[jl + 16] + (Queue::kPlanes == 2 ? (float)xr[DK + 16] : 0.0f);
        auto pop = [&]() -> int {
            int c = -1;
            if (rem0) {
                const int b = __clz((int)rem0);
                rem0 &= ~(0x80000000u >> b);
                c = slot_centroid(b, 0);
            } else if (rem1) {
                const int b = __clz((int)rem1);
                rem1 &= ~(0x80000000u >> b);
                c = slot_centroid(b, 1);
            }
            return c;
        };
        if (slot & 1) pop();
        double bs = __builtin_inf();
        int bc = 0x7fffffff;
        while (__ballot((rem0 | rem1) != 0u)) {
            const int cc = pop();
            const int ci = (cc < 0 || cc >= k) ? 0 : cc;
            const double ta = (double)xa - mu64T[(size_t)jl * KP + ci];
            sc[jl] = ta * ta;
            if (DK == 32) {
                const double tb = (double)xb - mu64T[(size_t)(jl + 16) * KP + ci];
                sc[jl + 16] = tb * tb;
            }
            __builtin_amdgcn_wave_barrier();
            if (jl == 0) {
                // eight loads in flight at a time; slots from d on hold exact zeros
                double ss = 0.0;
                for (int j0 = 0; j0 < d; j0 += 8) {
                    double v[8];
#pragma unroll
                    for (int i = 0; i < 8; ++i) v[i] = sc[j0 + i];
#pragma unroll
                    for (int i = 0; i < 8; ++i) ss = ss + v[i];
                }
                if (cc >= 0 && cc < k && (ss < bs || (ss == bs && cc < bc))) {
                    bs = ss;
                    bc = cc;
                }
            }
            __builtin_amdgcn_wave_barrier();
            pop();
        }
        const double os = __shfl_xor(bs, 16, 64);
        const int oc = __shfl_xor(bc, 16, 64);
        if (os < bs || (os == bs && oc < bc)) {
            bs = os;
            bc = oc;
        }
        if (have && (lane & 31) == 0) Q.lab_new()[pid] = (unsigned char)Queue::stored(bc < k ? bc : 0);
    }
    __builtin_amdgcn_wave_barrier();
}

template <int DK, typename Queue>
__device__ __forceinline__ void resolve_queue(const Queue &Q, int nrec, const double *mu64T,
                                              const float *ojf, int KP, int k, int d)
{
    if constexpr (DK <= 32) {
        if (nrec <= 8) {
            resolve_few<DK>(Q, nrec, mu64T, ojf, KP, k, d);
            return;
        }
    }
    resolve_rows<DK>(Q, nrec, mu64T, ojf, KP, k, d);
}

// Sums and sizes of every cluster over this wave's rows, from the current labels, on the matrix
// cores: S^T (knob x centroid) = X^T (knob x row) * onehot (row x centroid), 32 rows per instruction, all in bytes.
// Lane (m, kh) of the A fragment holds knob m of sixteen consecutive rows.  A knob (of two-byte knobs, either of its bytes) enters as the
// signed byte x - 128 (x ^ 0x80), a row of the cluster as -128, any other as 0: with t = label ^ centroid, bit 7 of t + 127 is clear
// where t is zero (labels below 128; otherwise two more operations).  The sums come out as -128 (S - 128 n), |.| <= 2^26, and the knob
// rows of absent knobs (all bytes zero) as 2^14 n, of which the last serves as the cluster size; with all knob rows in use the sizes are
// counted from the labels.  They are added to the sums of the workgroup off by raw_offset n (the centroid update takes that off)
// and to the sizes.  In bytes a step of 32 rows takes 20 (k > 32: 32) vector instructions; in f16 (bytes widened by
// placement, one-hot by a clamped difference) it was 44 (80).
typedef int int4v __attribute__((ext_vector_type(4)));
typedef int int16v __attribute__((ext_vector_type(16)));
constexpr int raw_offset(bool byte_knobs) { return byte_knobs ? -128 : -128 * 257; }
// labels -> -128 for the rows of the centroid, 0 for others
template <bool MANY>
__device__ __forceinline__ int4v members(const int4v &l, int c4)
{
    int4v o;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int t = MANY ? l[e] ^ c4 : (l[e] & 0x7F7F7F7F) ^ c4;
        o[e] = MANY ? ~(((t & 0x7F7F7F7F) + 0x7F7F7F7F) | t) & (int)0x80808080 : ~(t + 0x7F7F7F7F) & (int)0x80808080;
    }
    return o;
}
// From the packed byte copy: per 32 rows, NM blocks of 32 knobs, NP bytes of a value (low, high), the 1024 bytes of an A fragment in lane
// order.  bytes_w: the wave's first tile.  first: the 64 centroids [first, first + 64) are summed; MANY: there are more than those.
template <int DK, int NM, int NP, bool MANY, typename Queue>
__device__ __forceinline__ void packed_sums(const Queue &Q, int *S, int *n, const unsigned char *bytes_w, int d, int k_all, int rows_here,
                                            int lane, int first)
{
    constexpr int NF = NM * NP;                    // fragments per 32 rows
    constexpr int U = NF == 1 ? 4 : (NF == 2 ? 2 : 1);      // steps under way
    const int m32 = lane & 31, kh = lane >> 5;
    const int k = k_all - first;
    S += first * (DK + 1);
    n += first;
    const bool two = k > 32 && NM == 1;            // (k <= 32 with more than 32 knobs)
    const unsigned char *lp = Q.lab() + 16 * kh;
    const int c4a = (int)(Queue::stored(first + m32) * 0x01010101u), c4b = (int)(Queue::stored(first + m32 + 32) * 0x01010101u);
    int16v acc0[NF], acc1[NF];
#pragma unroll
    for (int f = 0; f < NF; ++f)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            acc0[f][i] = 0;
            acc1[f][i] = 0;
        }
    const int steps = (rows_here + 31) >> 5;
    const unsigned char *xp = bytes_w + 16 * lane;
    int4v w[U][NF];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
        for (int f = 0; f < NF; ++f) w[u][f] = *reinterpret_cast<const int4v *>(xp + (size_t)((u < steps ? u : 0) * NF + f) * 1024);
    for (int s0 = 0; s0 < steps; s0 += U) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int s = s0 + u;
            if (s < steps) {
                const int4v l = *reinterpret_cast<const int4v *>(lp + 32 * s);
                const int4v oa = members<MANY>(l, c4a);
                int4v ob = oa;
                if (two) ob = members<MANY>(l, c4b);
#pragma unroll
                for (int f = 0; f < NF; ++f) {
                    const int4v A = w[u][f] ^ (int)0x80808080;
                    acc0[f] = __builtin_amdgcn_mfma_i32_32x32x32_i8(A, oa, acc0[f], 0, 0, 0);
                    if (two) acc1[f] = __builtin_amdgcn_mfma_i32_32x32x32_i8(A, ob, acc1[f], 0, 0, 0);
                }
                const int ahead = s + U < steps ? s + U : s;
#pragma unroll
                for (int f = 0; f < NF; ++f) w[u][f] = *reinterpret_cast<const int4v *>(xp + (size_t)(ahead * NF + f) * 1024);
            }
        }
    }
    // accumulator register i of lane (c, kh) = knob (i & 3) + 8 (i >> 2) + 4 kh of centroid c (or 32 + c)
    const bool count_labels = (d & 31) == 0;
#pragma unroll
    for (int q = 0; q < NM; ++q) {
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int m = 32 * q + (i & 3) + 8 * (i >> 2) + 4 * kh;
            if (m < d) {
                int a = -(acc0[q * NP][i] >> 7), b = -(acc1[q * NP][i] >> 7);
                if (NP == 2) {
                    a -= 256 * (acc0[q * NP + NP - 1][i] >> 7);
                    b -= 256 * (acc1[q * NP + NP - 1][i] >> 7);
                }
                if (m32 < k) atomicAdd(&S[m32 * (DK + 1) + m], a);
                if (two && m32 + 32 < k) atomicAdd(&S[(m32 + 32) * (DK + 1) + m], b);
            }
            if (q == NM - 1 && !count_labels && i == 15 && kh == 1) {     // the last knob row: 2^14 per row of the cluster
                if (m32 < k) atomicAdd(&n[m32], acc0[q * NP][i] >> 14);
                if (two && m32 + 32 < k) atomicAdd(&n[m32 + 32], acc1[q * NP][i] >> 14);
            }
        }
    }
    if (count_labels) {
        for (int e = lane; e < rows_here; e += 64) {
            const unsigned v = Q.lab()[e];
            if (v != 0xFFu && (int)Queue::centroid(v) >= first && (int)Queue::centroid(v) < first + 64) atomicAdd(&n[Queue::centroid(v) - first], 1);
        }
    }
}

// Per-wave LDS region of this variant: the undecided rows of the tiles seen so far (candidate masks and row index), later the
// label changes of the pass; the knobs of the rows being resolved, a batch at a time, from the packed copy; the labels.  A label is
// stored as its position among the mask bits of a row (32 * lane half + position in that half's word), so that the mask of a
// decided row is one shift away.
// PL: f16 parts a knob value is split into (packed rows of PL * DK halfs).
template <int DK, int PL = 1>
struct FetchedQueue {
    static constexpr int kPlanes = PL;
    static constexpr int kRows = DK <= 32 ? 512 : 256;      // rows a wave owns at most
    static constexpr int kCap = 96;                         // (a tile adds at most 32)
    static constexpr int kBatch = 16;
    static constexpr int kChanges = 64;
    static constexpr size_t kOffFew = (size_t)8 * DK * PL * 2;   // (behind the eight rows there are then at most; up to 32-wide rows)
    static constexpr size_t kOffMask = DK <= 32 ? (kOffFew + 4 * 32 * 8 > (size_t)kBatch * DK * PL * 2 ? kOffFew + 4 * 32 * 8 : (size_t)kBatch * DK * PL * 2) : (size_t)kBatch * DK * PL * 2;
    static constexpr size_t kOffPid = kOffMask + (size_t)kCap * 8;
    static constexpr size_t kOffLab = kOffPid + (size_t)kCap * 2;
    static constexpr size_t kOffNew = kOffLab + (size_t)kRows;
    static constexpr size_t kBytes = kOffNew + (size_t)kRows;
    static_assert(kBytes % 16 == 0 && kOffLab % 16 == 0, "regions of a wave stay 16-byte aligned");
    static_assert(kCap * 8 >= kChanges * 4 && kOffMask >= (size_t)kBatch * DK * PL * 2 && kOffMask >= 64 * sizeof(double), "what shares a place fits it");
    unsigned char *base;
    int first;                                              // first row of the batch being resolved
    __device__ explicit FetchedQueue(unsigned char *wb) : base(wb), first(0) {}
    __device__ _Float16 *rec_x() const { return reinterpret_cast<_Float16 *>(base); }                    // [kBatch][PL * DK]
    __device__ unsigned *rec_mask() const { return reinterpret_cast<unsigned *>(base + kOffMask) + 2 * first; }      // [kCap][2]
    __device__ unsigned short *rec_pid() const { return reinterpret_cast<unsigned short *>(base + kOffPid) + first; }
    __device__ double *few() const { return reinterpret_cast<double *>(base + kOffFew); }                 // [4][32]
    __device__ unsigned *changes() const { return reinterpret_cast<unsigned *>(base + kOffMask); }         // [kChanges] new label | previous << 8 | row << 16, top bit: no label before
    __device__ unsigned char *lab() const { return base + kOffLab; }                                      // [kRows] current labels (0xFF: none)
    __device__ unsigned char *lab_new() const { return base + kOffNew; }                                  // [kRows] labels of the pass under way
    static __device__ __forceinline__ unsigned stored(unsigned c) { return (c >> 1) | ((c & 1u) << 5); }
    static __device__ __forceinline__ unsigned centroid(unsigned v) { return ((v & 31u) << 1) | (v >> 5); }
};

// ... of the form for more than 64 centroids: undecided rows with (row, candidate) pairs instead of masks, and what the evaluation of
// the pairs leaves per row.  Chunk c / 64 of a centroid is bits 6 and 7 of its stored label.
constexpr int kManyCentroids = 224;                         // (labels 0xFE and 0xFF mean undecided and none; LDS)
template <int DK>
struct ManyQueue {
    static constexpr int kPlanes = 1;
    static constexpr int kRows = 512;
    static constexpr int kCap = 96;                         // (a tile adds at most 32)
    static constexpr int kPairs = 256;
    static constexpr int kChanges = 64;
    static constexpr size_t kOffBestC = (size_t)kCap * 8;
    static constexpr size_t kOffPid = kOffBestC + (size_t)kCap * 4;
    static constexpr size_t kOffPairs = kOffPid + (size_t)kCap * 2;
    static constexpr size_t kOffCount = kOffPairs + (size_t)kPairs * 4;
    static constexpr size_t kOffLab = kOffCount + 16;
    static_assert(kPairs >= kChanges && kOffLab % 16 == 0 && kOffLab >= 256 * sizeof(double), "the label changes fit the pairs' place, the terms of a loss the queue's");
    static __host__ __device__ size_t bytes(int nwaves) { return kOffLab + 2 * (size_t)(nwaves == 16 ? kRows / 2 : kRows); }
    unsigned char *base;
    int rows;                                               // rows a wave owns at most
    __device__ ManyQueue(unsigned char *wb, int nwaves) : base(wb), rows(nwaves == 16 ? kRows / 2 : kRows) {}
    __device__ unsigned long long *best() const { return reinterpret_cast<unsigned long long *>(base); }            // [kCap] smallest distance (bits)
    __device__ int *best_c() const { return reinterpret_cast<int *>(base + kOffBestC); }                            // [kCap] lowest centroid attaining it
    __device__ unsigned short *rec_pid() const { return reinterpret_cast<unsigned short *>(base + kOffPid); }       // [kCap]
    __device__ unsigned *pairs() const { return reinterpret_cast<unsigned *>(base + kOffPairs); }                   // [kPairs] queued row << 8 | centroid
    __device__ unsigned *changes() const { return pairs(); }                                                         // [kChanges] new label | previous << 8 | row << 16, top bit: no label before
    __device__ unsigned *n_pairs() const { return reinterpret_cast<unsigned *>(base + kOffCount); }
    __device__ unsigned char *lab() const { return base + kOffLab; }
    __device__ unsigned char *lab_new() const { return base + kOffLab + rows; }
    static __device__ __forceinline__ unsigned stored(unsigned c) { return (c & 0xC0u) | ((c & 63u) >> 1) | ((c & 1u) << 5); }
    static __device__ __forceinline__ unsigned centroid(unsigned v) { return (v & 0xC0u) | ((v & 31u) << 1) | ((v >> 5) & 1u); }
};

// Exact evaluation of the queued rows against their candidates, one lane per (row, centroid) pair: the distance as
// sum_j ((double)x_j - mu_j)^2 with j ascending, no fused multiply-add; per row the smallest distance, then the lowest centroid
// attaining it.  all: every centroid of every queued row instead of the listed pairs (they found no room).
template <int DK>
__device__ __forceinline__ void resolve_pairs(const ManyQueue<DK> &Q, int nrec, bool all, const unsigned char *packed, const double *mu64T,
                                              const float *ojf, int KP, int k, int d, int lane)
{
    for (int r = lane; r < nrec; r += 64) {
        Q.best()[r] = ~0ull;
        Q.best_c()[r] = 0x7fffffff;
    }
    __builtin_amdgcn_wave_barrier();
    const unsigned np = all ? (unsigned)(nrec * k) : *Q.n_pairs();
    auto distance = [&](unsigned p, int &r, int &c) {
        if (all) {
            r = (int)(p / (unsigned)k);
            c = (int)(p % (unsigned)k);
        } else {
            const unsigned w = Q.pairs()[p];
            r = (int)(w >> 8);
            c = (int)(w & 0xFFu);
        }
        const unsigned char *x = packed + packed_at(Q.rec_pid()[r], 0, DK);
        double s = 0.0;
        for (int j0 = 0; j0 < d; j0 += 8) {
            const half8 xq = *reinterpret_cast<const half8 *>(x + packed_at(0, j0 >> 3, DK));
            double mu[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) mu[i] = mu64T[(size_t)(j0 + i) * KP + c];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                if (j0 + i < d) {
                    const double tq = (double)((float)xq[i] + ojf[j0 + i]) - mu[i];
                    s = s + tq * tq;
                }
            }
        }
        return (unsigned long long)__double_as_longlong(s);
    };
    // 64 pairs at a time: where they lower a row's smallest distance, the centroids that attained the one before no longer count
    // (A distance is evaluated once.  With a second walk for the centroids behind one for the distances, and full lists more often (below):
    // starts 3000 from the rows, streaming, 60 000 x 24, k = 64 and 128, 5110 / 2890 us a sweep; few values per knob, 84 shapes, 8 % more.)
    for (unsigned p0 = 0; p0 < np; p0 += 64) {
        const bool have = p0 + lane < np;
        int r = 0, c = 0;
        unsigned long long mine = ~0ull, before = ~0ull;
        if (have) {
            mine = distance(p0 + lane, r, c);
            before = Q.best()[r];
        }
        __builtin_amdgcn_wave_barrier();
        if (have) atomicMin(&Q.best()[r], mine);
        __builtin_amdgcn_wave_barrier();
        const unsigned long long now = Q.best()[r];
        if (have && now != before) Q.best_c()[r] = 0x7fffffff;
        __builtin_amdgcn_wave_barrier();
        if (have && now == mine) atomicMin(&Q.best_c()[r], c);
        __builtin_amdgcn_wave_barrier();
    }
    __builtin_amdgcn_wave_barrier();
    for (int r = lane; r < nrec; r += 64) {
        const int c = Q.best_c()[r];
        Q.lab_new()[Q.rec_pid()[r]] = (unsigned char)ManyQueue<DK>::stored(c < k ? c : 0);
    }
    __builtin_amdgcn_wave_barrier();
}

// Listed label changes of this wave (centroids, not stored labels) -> integer sums and sizes: 256 / DK rows per step, one lane per
// (row, four knobs), the knobs from the packed copy, those of four steps under way together.
template <int DK, typename Queue>
__device__ __forceinline__ void apply_listed(const Queue &Q, int cnt, const unsigned char *packed, int *S, int *n, int *dirty,
                                             const float *ojf, int d, int stamp)
{
    typedef _Float16 half4 __attribute__((ext_vector_type(4)));
    constexpr int LPR = DK / 4;              // lanes per row
    constexpr int EPI = 64 / LPR;            // rows per step
    constexpr int U = 4, PL = Queue::kPlanes;
    const int lane = threadIdx.x & 63;
    const int j0 = 4 * (lane % LPR);
    const float4 o4 = *reinterpret_cast<const float4 *>(ojf + j0);
    const float of[4] = {o4.x, o4.y, o4.z, o4.w};
    const bool on = j0 < d && lane < LPR * EPI;      // (twelve lanes per row leave four idle)
    __builtin_amdgcn_wave_barrier();
    for (int e0 = 0; e0 < cnt; e0 += U * EPI) {
        unsigned w[U];
        half4 xq[U], xs[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int e = e0 + u * EPI + lane / LPR;
            w[u] = Q.changes()[e < cnt ? e : 0];
            xq[u] = *reinterpret_cast<const half4 *>(packed + packed_at((w[u] >> 16) & 0x7FFF, j0 >> 3, DK * PL) + 2 * (j0 & 4));
            if (PL == 2) xs[u] = *reinterpret_cast<const half4 *>(packed + packed_at((w[u] >> 16) & 0x7FFF, (DK + j0) >> 3, DK * PL) + 2 * (j0 & 4));
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int e = e0 + u * EPI + lane / LPR;
            if (e < cnt && on) {
                const int cur = w[u] & 0xFF, prev = (w[u] >> 8) & 0xFF;
                const bool first = (w[u] >> 31) != 0u;
                int *sc = S + cur * (DK + 1) + j0;
                int *sp = S + (first ? cur : prev) * (DK + 1) + j0;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    if (j0 + i < d) {
                        const int xi = (int)((float)xq[u][i] + of[i] + (PL == 2 ? (float)xs[u][i] : 0.0f));
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
    }
    __builtin_amdgcn_wave_barrier();
}

// Tiles whose rows are fetched ahead (even: the accumulators alternate).
constexpr int rows_ahead(int W, bool two, bool CIN) { return (W == 16 && !CIN) || (W == 32 && !two) ? 4 : 2; }

// The undecided rows of a wave: their knobs from the packed copy, a batch at a time, then the exact evaluation.
template <int DK, int PL>
__device__ __forceinline__ void resolve_batches(const FetchedQueue<DK, PL> &Q, int nrec, const unsigned char *packed, const double *mu64T,
                                                const float *ojf, int KP, int k, int d, int lane)
{
    typedef FetchedQueue<DK, PL> Queue;
    constexpr int LPR = DK * PL / 8;              // lanes per row, 16 bytes each
    Queue part = Q;
    for (part.first = 0; part.first < nrec; part.first += Queue::kBatch) {
        const int left = nrec - part.first, rows = left < Queue::kBatch ? left : Queue::kBatch;
        __builtin_amdgcn_wave_barrier();
        for (int e = lane; e < rows * LPR; e += 64)
            *reinterpret_cast<half8 *>(part.rec_x() + 8 * e) =
                *reinterpret_cast<const half8 *>(packed + packed_at(part.rec_pid()[e / LPR], e % LPR, DK * PL));
        resolve_queue<DK>(part, rows, mu64T, ojf, KP, k, d);
    }
}

// What the tile loops work on: the wave's packed tiles, the centroids' fragments in LDS (with SEP those of the bias step, with CIN the
// initial scores in fragment order instead of a bias slot), the screen bound (of every row, or with ROW_BOUND bound + x2_scale |x'|^2) and
// all ones where every tile is to be decided whatever its masks say.
struct Tiles {
    const unsigned char *packed;
    const half8 *afrag, *abias;
    const float *bias;
    const float *x2;
    float bound, x2_scale, bias_scale;
    int ntiles, rows_wave;
    uint64_t undecided;
};

// rows of tile nt that the wave owns, as a mask
__device__ __forceinline__ uint32_t live_rows(int rows_wave, int nt)
{
    const int left = rows_wave - 32 * nt;
    return left >= 32 ? 0xFFFFFFFFu : (left <= 0 ? 0u : ((1u << left) - 1u));
}

// this lane's B fragments of a tile (rows behind the task's last are read, from inside the workspace, and ignored)
template <int DK>
__device__ __forceinline__ void fetch_tile(half8 (&Bt)[DK / 16], const unsigned char *p, unsigned lane_off)
{
    // a scalar base in global memory: a lane's part of the address is one 32-bit register
    uint64_t at = reinterpret_cast<uint64_t>(p);
    asm volatile("" : "+s"(at));
    typedef const __attribute__((address_space(1))) unsigned char gbyte;
    typedef const __attribute__((address_space(1))) half8 ghalf8;
#pragma unroll
    for (int f = 0; f < DK / 16; ++f) Bt[f] = *reinterpret_cast<ghalf8 *>(reinterpret_cast<gbyte *>(at) + lane_off + 1024 * f);
}

// initial scores of an m-tile: [lane half][16], the order of the accumulator's registers
__device__ __forceinline__ void start_scores(float16v &acc, const float *bias, int lane)
{
    const float4 *p = reinterpret_cast<const float4 *>(bias + 16 * (lane >> 5));
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        const float4 b = p[g];
        acc[4 * g + 0] = b.x; acc[4 * g + 1] = b.y; acc[4 * g + 2] = b.z; acc[4 * g + 3] = b.w;
    }
}

// The tile loop from tile nt on, for up to 64 centroids; compiled once per number of live registers of the last m-tile (4, 8, 12 or
// 16), so that the epilogue has no branches.  Returns the tile to go on with: ntiles, or an earlier one when the queue has to be
// emptied.
template <int DK, bool SEP, bool CIN, bool ROW_BOUND, int LREGS, bool TWO, typename Queue>
__device__ __forceinline__ int decide_tiles(const Queue &Q, const Tiles &T, int nt, int &nrec, int lane)
{
    constexpr int NS = DK / 16, NS2 = 2 * NS, NSA = NS2 + (SEP ? 1 : 0);
    constexpr int PL = Queue::kPlanes, NB = NS * PL, NC = NS2 * PL;      // B fragments of a row, instructions of a chain
    constexpr int CH = NC == 6 ? 4 : (NC == 12 ? 2 : 16 / NC);           // scores handled between two matrix instructions
    constexpr unsigned kTileBytes = 32 * DK * PL * 2;
    constexpr int kAhead = rows_ahead(DK * PL, TWO, CIN);
    const std::integral_constant<int, LREGS> live_tag;
    const int n32 = lane & 31;
    const unsigned char *packed = T.packed;
    const bool upper = lane >= 32;
    const unsigned lane_off = (unsigned)(16 * lane);
    const float16v zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    half8 Bq[kAhead][NB];                // rows of tiles nt .. nt + kAhead - 1
#pragma unroll
    for (int u = 0; u < kAhead; ++u) fetch_tile<DK * PL>(Bq[u], packed + (nt + u) * kTileBytes, lane_off);
    // squared norms of the rows, as far ahead
    float x2q[kAhead];
    const float *norms = T.x2 + 32 * nt + n32;
    if (ROW_BOUND) {
#pragma unroll
        for (int u = 0; u < kAhead; ++u) x2q[u] = norms[32 * u];
        norms += 32 * kAhead;
    }
    const unsigned char *ahead = packed + (nt + kAhead) * kTileBytes;
    int end = T.ntiles;                    // where this call stops
    const unsigned char *labs = Q.lab() + nt * 32 + n32;
    // A fragments of this pass (the bias slot included)
    half8 A0[NSA], A1[NSA];
#pragma unroll
    for (int s = 0; s < NS2; ++s) {
        A0[s] = T.afrag[s * 64 + lane];
        A1[s] = TWO ? T.afrag[(NS2 + s) * 64 + lane] : A0[s];
    }
    // the bias step: 256 against hi (slot 0) and lo (slot 1), the same for every row
    half8 bias_b;
    if constexpr (SEP) {
        A0[NS2] = T.abias[lane];
        A1[NS2] = TWO ? T.abias[64 + lane] : A0[NS2];
#pragma unroll
        for (int i = 0; i < 8; ++i) bias_b[i] = (_Float16)(i < 2 && lane < 32 ? T.bias_scale : 0.0f);
    }

    // the chain starts from zero (the bias is in the operands), or from the bias in fp32
    float16v startA = zero16, startB = zero16;
    if constexpr (CIN && PL == 1) {
        start_scores(startA, T.bias, lane);
        if (TWO) start_scores(startB, T.bias + 32, lane);
    }
    float16v accA, accB;
    // one matrix instruction of the chain of a 32x32 tile (the first one behind the bias step)
    auto mma = [&](float16v &acc, const half8 (&Af)[NSA], const half8 (&Bt)[NB], const float16v &start, int s) {
        if constexpr (SEP) {
            if (s == 0) acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(Af[NS2], bias_b, zero16, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(Af[s], Bt[s % NS], acc, 0, 0, 0);
            return;
        }
        if constexpr (CIN && PL == 2) {
            // (no registers to keep the initial scores in: fetched where the chain starts)
            if (s == 0) start_scores(acc, T.bias + (&Af == &A1 ? 32 : 0), lane);
            acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(Af[s / PL], Bt[(s / PL) % NS + NS * (s % PL)], acc, 0, 0, 0);
            return;
        }
        acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(Af[s], Bt[s % NS], s == 0 ? start : acc, 0, 0, 0);
    };
    // mark scores [i0, i0 + CH): bit set = below the threshold
    auto mark = [&](uint32_t &near, const float16v &acc, float thr, int i0) {
#pragma unroll
        for (int i = 0; i < CH; ++i)
            if (i0 + i < 16) near = __builtin_amdgcn_alignbit(near, __float_as_uint(acc[i0 + i] - thr), 31);
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
    // After the masks of tile nt: a tile whose rows all have exactly their current label marked is done (but in the first
    // pass).  Otherwise the tile's rows are decided: a row with exactly one candidate takes it, any other row is queued
    // for the exact evaluation after the tile loop (label 0xFE until then).  (The matrix instructions of the next tile are under way meanwhile.)
    auto settle = [&](uint32_t cand, uint32_t prev, int nt) {       // cand: bit 31 = position 0
        const uint64_t place = 0x8000000000000000ull >> (prev & 63u);
        const uint32_t own = upper ? (uint32_t)place : (uint32_t)(place >> 32);
        if ((__ballot(cand != own) | T.undecided) == 0) return;
        const uint32_t live32 = live_rows(T.rows_wave, nt);
        uint32_t cand_lo, cand_hi;
        both_halves(cand, cand_lo, cand_hi);
        const int total = __popc(cand_lo) + __popc(cand_hi);
        const bool live = (live32 >> n32) & 1u;
        const bool flagged = live && total != 1;
        const uint32_t fm = (uint32_t)__ballot(flagged);
        if (fm) {
            if (flagged) {
                const int rs = nrec + __popc(fm & ((1u << n32) - 1u));
                // no candidate at all cannot happen (the smallest score is always one); if it does, every centroid is one
                Q.rec_mask()[rs * 2 + (upper ? 1 : 0)] = total ? cand : 0xFFFFFFFFu;
                if (!upper) Q.rec_pid()[rs] = (unsigned short)(nt * 32 + n32);
            }
            nrec += __popc(fm);
            if (nrec > Queue::kCap - 32) end = nt + 1;      // the next tile might not fit
        }
        const uint32_t lab = cand_lo ? (uint32_t)__clz((int)cand_lo) : 32u + ((uint32_t)__clz((int)cand_hi) & 31u);
        const uint32_t now = !live ? 0xFFu : (flagged ? 0xFEu : lab);
        if (!upper) Q.lab_new()[nt * 32 + n32] = (unsigned char)now;
    };

    if constexpr (TWO) {
        // accA = centroids 0..31 (all sixteen registers live), accB = centroids 32..k-1 of the current tile; Bn = rows of
        // the next tile, Bf = free for those of the tile kAhead further on
        auto step = [&](half8 (&Bn)[NB], half8 (&Bf)[NB], float &x2f) {
            fetch_tile<DK * PL>(Bf, ahead, lane_off);
            ahead += kTileBytes;
            const float x2 = x2f;
            if (ROW_BOUND) {
                x2f = *norms;
                norms += 32;
            }
            const uint32_t prev = *labs;
            labs += 32;
            const float best = row_min(vmin(min_live(accA, std::integral_constant<int, 16>{}), min_live(accB, live_tag)));
            const float thr = best + T.bound + (ROW_BOUND ? T.x2_scale * x2 : 0.0f);
            uint32_t near = 0;
#pragma unroll
            for (int s = 0; s < NC; ++s) mark(near, accA, thr, s * CH);
            // accA is consumed: its next chain runs under the marking of accB
#pragma unroll
            for (int s = 0; s < NC; ++s) {
                __builtin_amdgcn_sched_barrier(0);
                mma(accA, A0, Bn, startA, s);
                __builtin_amdgcn_sched_barrier(0);
                if (s * CH < LREGS) mark(near, accB, thr, s * CH);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int s = 0; s < NC; ++s) mma(accB, A1, Bn, startB, s);
            // (registers of accB that were not walked hold padding only)
            constexpr int live_marks = CH * ((LREGS + CH - 1) / CH);
            settle(near << (16 - live_marks), prev, nt);
            __builtin_amdgcn_sched_barrier(0);
            asm volatile("" : "+v"(accB));      // (as below)
        };
#pragma unroll
        for (int s = 0; s < NC; ++s) mma(accA, A0, Bq[0], startA, s);
#pragma unroll
        for (int s = 0; s < NC; ++s) mma(accB, A1, Bq[0], startB, s);
        for (;;) {
#pragma unroll
            for (int u = 0; u < kAhead; ++u) {
                step(Bq[(u + 1) % kAhead], Bq[u], x2q[u]);
                if (++nt >= end) return nt;
            }
        }
    } else {
        // one m-tile: the accumulators alternate, the next tile's chain runs under this epilogue
        auto step = [&](float16v &cur, float16v &nxt, half8 (&Bn)[NB], half8 (&Bf)[NB], float &x2f) {
            fetch_tile<DK * PL>(Bf, ahead, lane_off);
            ahead += kTileBytes;
            const float x2 = x2f;
            if (ROW_BOUND) {
                x2f = *norms;
                norms += 32;
            }
            const uint32_t prev = *labs;
            labs += 32;
            const float best = row_min(min_live(cur, live_tag));
            const float thr = best + T.bound + (ROW_BOUND ? T.x2_scale * x2 : 0.0f);
            uint32_t near = 0;
#pragma unroll
            for (int s = 0; s < NC; ++s) {
                __builtin_amdgcn_sched_barrier(0);
                mma(nxt, A0, Bn, startA, s);
                __builtin_amdgcn_sched_barrier(0);
                if (s * CH < LREGS) mark(near, cur, thr, s * CH);
            }
            __builtin_amdgcn_sched_barrier(0);
            constexpr int live_marks = CH * ((LREGS + CH - 1) / CH);
            settle(near << (32 - live_marks), prev, nt);
            __builtin_amdgcn_sched_barrier(0);
            // registers of dead scores are not used for anything else meanwhile: that would wait for the chain's end
            asm volatile("" : "+v"(nxt));
        };
#pragma unroll
        for (int s = 0; s < NC; ++s) mma(accA, A0, Bq[0], startA, s);
        for (;;) {
#pragma unroll
            for (int u = 0; u < kAhead; ++u) {
                step(u & 1 ? accB : accA, u & 1 ? accA : accB, Bq[(u + 1) % kAhead], Bq[u], x2q[u]);
                if (++nt >= end) return nt;
            }
        }
    }
}

// All tiles, for any number of centroids, 64 at a time: a chunk leaves its minimum and the marks within the bound of it; the marks
// of a chunk count iff its minimum is within the bound of the overall one.
template <int DK, bool CIN, bool ROW_BOUND>
__device__ __forceinline__ void decide_tiles_many(const ManyQueue<DK> &Q, const Tiles &T, int &nrec, const double *mu, const float *ojf,
                                                  int KP, int k, int d, int lane)
{
    typedef ManyQueue<DK> Queue;
    constexpr int kChunks = 4;                     // k <= 256
    constexpr int NS = DK / 16, NS2 = 2 * NS;
    constexpr unsigned kTileBytes = 32 * DK * 2;
    const unsigned char *packed = T.packed;
    const int n32 = lane & 31;
    bool all_pairs = false;          // the list of pairs is not complete
    const bool upper = lane >= 32;
    const unsigned lane_off = (unsigned)(16 * lane);
    const int nch = (k + 63) >> 6, kpu = (k + 31) & ~31;
    const float16v zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    half8 Bn[NS];
    if (lane == 0) *Q.n_pairs() = 0u;
    const float *norms = T.x2 + n32;
    float x2n = 0.0f;
    if (T.ntiles > 0) {
        fetch_tile<DK>(Bn, packed, lane_off);
        if (ROW_BOUND) x2n = norms[0];
    }
    for (int nt = 0; nt < T.ntiles; ++nt) {
        half8 Bt[NS];
#pragma unroll
        for (int f = 0; f < NS; ++f) Bt[f] = Bn[f];
        fetch_tile<DK>(Bn, packed + (nt + 1) * kTileBytes, lane_off);
        const float bound = T.bound + (ROW_BOUND ? T.x2_scale * x2n : 0.0f);
        if (ROW_BOUND) x2n = norms[32 * (nt + 1)];
        const uint32_t prev = Q.lab()[nt * 32 + n32];
        uint32_t near[kChunks];
        float least[kChunks];
        float best = __builtin_inff();
#pragma unroll
        for (int ch = 0; ch < kChunks; ++ch) {
            near[ch] = 0u;
            least[ch] = __builtin_inff();
            if (ch < nch) {
                const bool has1 = (2 * ch + 1) * 32 < kpu;
                float16v accA = zero16, accB = zero16;
                if (CIN) {
                    start_scores(accA, T.bias + 64 * ch, lane);
                    if (has1) start_scores(accB, T.bias + 64 * ch + 32, lane);
                }
#pragma unroll
                for (int s = 0; s < NS2; ++s)
                    accA = __builtin_amdgcn_mfma_f32_32x32x16_f16(T.afrag[((2 * ch) * NS2 + s) * 64 + lane], Bt[s % NS], accA, 0, 0, 0);
                if (has1) {
#pragma unroll
                    for (int s = 0; s < NS2; ++s)
                        accB = __builtin_amdgcn_mfma_f32_32x32x16_f16(T.afrag[((2 * ch + 1) * NS2 + s) * 64 + lane], Bt[s % NS], accB, 0, 0, 0);
                }
                auto min16 = [](const float16v &acc) {
                    float m = vmin3(acc[0], acc[1], acc[2]);
#pragma unroll
                    for (int i = 3; i < 15; i += 2) m = vmin3(m, acc[i], acc[i + 1]);
                    return vmin(m, acc[15]);
                };
                float m = min16(accA);
                if (has1) m = vmin(m, min16(accB));
                unsigned lo, hi;
                both_halves(__float_as_uint(m), lo, hi);
                m = vmin(__uint_as_float(lo), __uint_as_float(hi));
                const float thr = m + bound;
                uint32_t bits = 0;
#pragma unroll
                for (int i = 0; i < 16; ++i) bits = __builtin_amdgcn_alignbit(bits, __float_as_uint(accA[i] - thr), 31);
                if (has1) {
#pragma unroll
                    for (int i = 0; i < 16; ++i) bits = __builtin_amdgcn_alignbit(bits, __float_as_uint(accB[i] - thr), 31);
                } else {
                    bits <<= 16;
                }
                near[ch] = bits;
                least[ch] = m;
                best = vmin(best, m);
            }
        }
        // a tile whose rows all have exactly their current label marked is done (but in the first pass)
        const float lim = best + bound;
        const uint64_t place = 0x8000000000000000ull >> (prev & 63u);
        const uint32_t own = upper ? (uint32_t)place : (uint32_t)(place >> 32);
        uint32_t diff = 0u;
#pragma unroll
        for (int ch = 0; ch < kChunks; ++ch) {
            near[ch] = least[ch] <= lim ? near[ch] : 0u;
            diff |= near[ch] ^ ((prev >> 6) == (uint32_t)ch ? own : 0u);
        }
        if ((__ballot(diff != 0u) | T.undecided) == 0) continue;
        const uint32_t live32 = live_rows(T.rows_wave, nt);
        int cnt = 0, at = 0;                       // marks of this lane half, stored label of one of them
#pragma unroll
        for (int ch = 0; ch < kChunks; ++ch) {
            cnt += __popc(near[ch]);
            at = near[ch] ? 64 * ch + (upper ? 32 : 0) + __clz((int)near[ch]) : at;
        }
        unsigned c_lo, c_hi, at_lo, at_hi;
        both_halves((unsigned)cnt, c_lo, c_hi);
        both_halves((unsigned)at, at_lo, at_hi);
        const bool live = (live32 >> n32) & 1u;
        const bool flagged = live && c_lo + c_hi != 1u;
        const uint32_t fm = (uint32_t)__ballot(flagged);
        if (fm) {
            if (flagged) {
                const int rs = nrec + __popc(fm & ((1u << n32) - 1u));
                if (!upper) Q.rec_pid()[rs] = (unsigned short)(nt * 32 + n32);
                // Starts beyond the range of the operands have every score within the bound, those of the padding rows
                // k .. 32 ceil(k / 32) - 1 too: no candidates (their centroids are zero, or whatever memory held).
                cnt = 0;
#pragma unroll
                for (int ch = 0; ch < kChunks; ++ch) {
                    near[ch] &= marks_below(k - 64 * ch, upper ? 1 : 0);
                    cnt += __popc(near[ch]);
                }
                unsigned pos = atomicAdd(Q.n_pairs(), (unsigned)cnt);
#pragma unroll
                for (int ch = 0; ch < kChunks; ++ch) {
                    uint32_t m = near[ch];
                    while (m) {
                        const int q = __clz((int)m);
                        m &= ~(0x80000000u >> q);
                        const int c = 64 * ch + slot_centroid(q, upper ? 1 : 0);
                        if (pos < (unsigned)Queue::kPairs) Q.pairs()[pos] = (unsigned)(rs << 8 | c);
                        ++pos;
                    }
                }
                if (pos > (unsigned)Queue::kPairs) all_pairs = true;
            }
            // no candidate at all cannot happen (the smallest score is always one); if it does, every centroid is one
            if (flagged && c_lo + c_hi == 0u) all_pairs = true;
            nrec += __popc(fm);
            // the next tile might not fit; nor would its pairs, at three a row or more
            if (nrec > Queue::kCap - 32 || *Q.n_pairs() > (unsigned)Queue::kPairs - 96u) {
                resolve_pairs<DK>(Q, nrec, __any(all_pairs), packed, mu, ojf, KP, k, d, lane);
                nrec = 0;
                all_pairs = false;
                if (lane == 0) *Q.n_pairs() = 0u;
                __builtin_amdgcn_wave_barrier();
            }
        }
        const uint32_t now = !live ? 0xFFu : (c_lo ? at_lo : at_hi);
        // (a row resolved just now has its label already)
        if (!upper && !flagged) Q.lab_new()[nt * 32 + n32] = (unsigned char)now;
    }
    if (nrec) resolve_pairs<DK>(Q, nrec, __any(all_pairs), packed, mu, ojf, KP, k, d, lane);
}

}  // namespace

}  // namespace cham
