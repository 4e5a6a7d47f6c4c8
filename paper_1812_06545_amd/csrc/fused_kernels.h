// Fused frame-resident decoder: one workgroup decodes one frame through all
// of its iterations with the frame's messages held in LDS, on the flooding
// schedule or (jobs with LDPC_LAYERED) the layered one.
//
// Schedule (arxiv 1812.06545, Section II; Algorithm 1): the same flooding
// two-phase iteration as the plain path, but the global barrier between the
// check-node and variable-node phases becomes a workgroup barrier, because
// the frames are independent (the frame-level parallelism of Section III-A)
// and one workgroup owns a whole frame.  HBM traffic per frame is the channel
// LLRs (read once per iteration, from L2 after the first) and the outputs; the
// code's address tables stream from L2.
//
// One launch decodes a batch of jobs of different codes, lengths and rates, in
// items of one (job, frame) each; a frame that stops early frees its workgroup
// for the next item.
//
// Lanes and tables.  Every code runs from address tables that its handle
// carries (FusedTables, code.cpp), so that no kernel derives an address:
//   flooding   a group is 32 check rows of like degree (rows sorted by
//              descending degree); lane l takes the first half of row l mod 32
//              for l < 32, the second half for l >= 32.  Slot k of every lane
//              has its posterior's LDS address in the table, four slots to a
//              16-byte load.  The messages lie in the same order, slot by slot
//              and lane by lane, so a message's address is the group's plus a
//              constant, and no two lanes meet in an LDS bank.
//   columns    a group is 64 variables; the table holds the addresses of each
//              one's messages in ascending row order.
//   layered    a group is up to 16 rows of one layer; lanes l, l + 16, l + 32
//              and l + 48 take a row's quarters.  Messages lie in CSR order and
//              have table addresses too, since a layer may hold few rows and
//              the padded order would not be bounded.
// A lane with fewer slots than its group's longest is padded with dummies:
// their posterior is a word holding +inf, whose term is exactly the identity
// of the row's combination and whose sign is +, so every real message is
// computed with exactly the operations and rounding of the plain path
// (bit-identical results); a column's dummies add a word holding -0, which
// changes no sum.
//
// What this layout is for: the flooding kernel is bound by VALU issue.  With
// addresses formed from the circulants' shifts in the kernel (one table word
// per block in LDS) a slot cost 7 of its 44 instructions, a column's message
// 3, and the parked terms two LDS accesses; codes without circulants read
// their indices uncoalesced, a cache line per lane.  The tables cost 4 bytes
// of L2 traffic per edge and phase, about 3 TB/s over the device.
#pragma once

#include <algorithm>
#include <mutex>
#include <type_traits>
#include <vector>

#include "ldpc_internal.h"
#include "minsum_kernels.h"
#include "spa_math.h"

namespace ldpc {
namespace fused {

constexpr int kMaxCodes = 16;
constexpr int kMaxJobs = 24;

// Kernel-argument copy of a code's tables (device pointers; see FusedTables).
struct Code {
    int32_t n, E;
    int32_t row_groups, nlayers;
    int32_t r_words;  // message words of a flooding frame (E with an explicit order)
    int32_t m, layer_rows;  // rows; rows of the largest layer
    int32_t row_words, col_words, lay_words;  // sizes of the tables
    const int32_t *row_grp, *row_tab, *row_pos, *col_grp, *col_tab, *lay_ptr, *lay_grp, *lay_tab;
};

struct Job {
    int32_t code, frames, max_iter;
    uint32_t flags;
    float ms_scale, ms_offset;  // min-sum correction (LDPC_MIN_SUM), natural LLR units
    const void *llr;
    uint8_t *bits;
    int32_t *iters;
    void *post;
};

// One launch's jobs, passed to the kernel by value.  Item i (a frame, or
// frames_per_item of them) belongs to the last job j with begin[j] <= i; the
// entries past njobs hold INT32_MAX.
struct Batch {
    int32_t njobs, ncodes;
    int32_t nitems, frames_per_item;
    uint32_t flags_at;   // LDS address of the workgroup's flag words
    uint32_t tables_at;  // and of its code's tables (kernels that copy them)
    int32_t layer_turn;  // by what the wavefronts' places in a layer change from each to the next
    int32_t begin[kMaxJobs];
    Code codes[kMaxCodes];
    Job jobs[kMaxJobs];
};
static_assert(sizeof(Batch) <= 4080, "a launch's kernel arguments are limited to 4 KiB");

__device__ __forceinline__ int32_t job_of_item(const Batch &b, int32_t item)
{
    int32_t j = 0;
#pragma unroll
    for (int32_t k = 1; k < kMaxJobs; ++k)
        j += b.begin[k] <= item;
    return j;
}

// Workgroups have up to kMaxThreads threads in FP32 and kBaseThreads in FP64,
// whose bodies need the registers of two wavefronts per SIMD.  kBaseThreads is
// also the size the callers' settings end at; a launch left at it takes the
// size workgroup_threads() picks.
constexpr int kBaseThreads = 512, kMaxThreads = 1024;

// LDS of a workgroup, in words of the message type: the posteriors, then at
// n + kInfWord .. the constants dummies use, then from first_message(n) the
// messages; the flag words follow the launch's largest frame.  All of it is
// dynamic and starts at address 0 (the kernels have no static LDS).  The
// tables hold byte addresses of 4-byte words.
constexpr int kInfWord = 0, kMinusZeroWord = 1, kJunkWord = 2;  // junk: a dummy's message (any finite value)
constexpr int kFlagWords = 4, kItemFlag = 3;                    // three vote words, then the workgroup's next item

// Bytes for the flag words and a frame of n variables and `r_words` messages
// (cleared by fours).
inline size_t lds_bytes(int32_t n, int64_t r_words, size_t tsize)
{
    return (static_cast<size_t>(fused_first_message(n)) + align_up(static_cast<size_t>(r_words), 4)) * tsize +
           kFlagWords * sizeof(int32_t);
}

// LDS is addressed by integers: a workgroup's LDS starts at address 0, and an
// array symbol for it would be resolved too late for the compiler to fold its
// address into an access (one addition per slot of every row).
template <class T>
using Lds = __attribute__((address_space(3))) T;
template <class T>
__device__ __forceinline__ Lds<T> *lds_at(uint32_t addr)
{
    return (Lds<T> *)addr;
}
template <class T>
__device__ __forceinline__ T lds_ld(uint32_t addr)
{
    return *lds_at<T>(addr);
}
template <class T>
__device__ __forceinline__ void lds_st(uint32_t addr, T v)
{
    *lds_at<T>(addr) = v;
}

// Workgroup-wide OR at a barrier, through an LDS word per use: any(v) is
// nonzero on every thread if v (uniform in each wavefront) was on some
// wavefront.  Three words take turns.  After the barrier of use u thread 0
// clears the word of use u + 2: every thread has read it (for use u - 1)
// before that barrier, and use u + 2 sets it after the barrier of use u + 1,
// which thread 0 reaches after the clear.  One barrier and one LDS word per
// use, where __syncthreads_or takes several barriers and static LDS.
struct Vote {
    Lds<int32_t> *w;  // three words, zero at the start
    uint32_t k = 0;   // uses so far, mod 3
    __device__ __forceinline__ int32_t any(bool v)
    {
        if (v && (threadIdx.x & 63) == 0)
            w[k] = 1;
        __syncthreads();
        const int32_t r = __builtin_amdgcn_readfirstlane(w[k]);
        if (threadIdx.x == 0)
            w[k == 0 ? 2 : k - 1] = 0;
        k = k == 2 ? 0 : k + 1;
        return r;
    }
};

// Value of the partner lane (lane ^ 32: the other half of the row) and of the
// sibling lane (lane ^ 16: the other quarter of the half), by the lane-group
// swaps: after a swap of x with itself one result holds x's even lane groups
// in every group, the other its odd ones.
template <int M>
__device__ __forceinline__ uint32_t lane_swap(uint32_t v)
{
    static_assert(M == 16 || M == 32, "lane groups of 16 or 32");
    const bool odd = (threadIdx.x & M) != 0;
    if constexpr (M == 32) {
        const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
        return odd ? r[0] : r[1];
    } else {
        const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
        return odd ? r[0] : r[1];
    }
}
// The same of a lane mask.
template <int M>
__device__ __forceinline__ Lanes lane_swap(Lanes m)
{
    constexpr Lanes even = M == 32 ? 0x00000000ffffffffull : 0x0000ffff0000ffffull;
    return (m & even) << M | (m >> M & even);
}
template <int M>
__device__ __forceinline__ float lane_swap(float v)
{
    return __uint_as_float(lane_swap<M>(__float_as_uint(v)));
}
template <int M>
__device__ __forceinline__ double lane_swap(double v)
{
    const uint64_t u = static_cast<uint64_t>(__double_as_longlong(v));
    const uint64_t lo = lane_swap<M>(static_cast<uint32_t>(u)), hi = lane_swap<M>(static_cast<uint32_t>(u >> 32));
    return __longlong_as_double(static_cast<long long>(hi << 32 | lo));
}
template <int M>
__device__ __forceinline__ ArithF32::Acc lane_swap(const ArithF32::Acc &v)
{
    return ArithF32::Acc{lane_swap<M>(v.P), lane_swap<M>(v.Q)};
}
template <int M>
__device__ __forceinline__ ArithF64::Acc lane_swap(const ArithF64::Acc &v)
{
    return ArithF64::Acc{lane_swap<M>(v.P), lane_swap<M>(v.Q)};
}

// Slots 4i .. 4i + 3 of a lane.
typedef int32_t Quad __attribute__((ext_vector_type(4)));
constexpr int quads(int d) { return (d + 3) / 4; }

// A table: in device memory, or (LT) the workgroup's copy in LDS.  Where every
// frame has a CU to itself, nothing hides the L2 latency that starts each
// group's work, and the CU's LDS is mostly free: the frame's workgroup copies
// its code's tables there first, if they fit.  us per call of 10 iterations,
// tables in L2 and in LDS: 24 layered frames of qc n = 1296, rate 2/3, early stop
// 104 and 92; a plan of 64 frames of four codes 48.8 and 45.6; one frame of
// (3,6)-regular n = 2040 40 and 36; of qc n = 648 34 and 33.
template <bool LT>
using Table = typename std::conditional<LT, const Lds<Quad> *, const Quad *>::type;
template <bool LT>
__device__ __forceinline__ Table<LT> table_at(const int32_t *tab, uint32_t copy)
{
    if constexpr (LT)
        return lds_at<Quad>(copy);
    else
        return reinterpret_cast<const Quad *>(tab);
}

// Table addresses of D slots, from this lane's first quad, quads `stride` apart.
template <class T, int D>
struct Addresses {
    Quad q[quads(D)];
    template <class Tab>
    __device__ __forceinline__ void load(Tab tab, int stride)
    {
#pragma unroll
        for (int i = 0; i < quads(D); ++i)
            q[i] = tab[i * stride];
    }
    __device__ __forceinline__ uint32_t operator[](int k) const
    {
        return static_cast<uint32_t>(q[k / 4][k % 4]) * static_cast<uint32_t>(sizeof(T) / 4);
    }
};

// Where a flooding lane's messages lie: slot by slot (ra: slot 0's address),
// or, where the padded order did not fit, at table addresses.
template <class T, int D, bool POS>
struct Messages {
    uint32_t ra;
    Addresses<T, POS ? D : 1> pos;
    __device__ __forceinline__ uint32_t operator[](int k) const
    {
        if constexpr (POS)
            return pos[k];
        else
            return ra + static_cast<uint32_t>(k * 64 * static_cast<int>(sizeof(T)));
    }
};

// Parity of a row whose two halves lie 32 lanes apart, over the wavefront:
// some row is odd.
__device__ __forceinline__ bool some_odd(uint64_t half_parity)
{
    return (static_cast<uint32_t>(half_parity) ^ static_cast<uint32_t>(half_parity >> 32)) != 0u;
}

// One half of a check row of each lane, D slots.  All loads are issued before
// the arithmetic.  PAR: `odd` is set if a row of the wavefront is unsatisfied
// by the decision [L < 0] that the gathered posteriors hold (one comparison
// per slot; the parities are lane masks in scalar registers).
template <class A, int D, bool PAR, bool POS, class Tab>
__device__ __forceinline__ void half_row(Tab tab, const Messages<typename A::T, D, POS> &msg, bool &odd)
{
    using T = typename A::T;
    Addresses<T, D> ci;
    ci.load(tab, 64);
    T lv[D], rv[D];
#pragma unroll
    for (int j = 0; j < D; ++j)
        rv[j] = lds_ld<T>(msg[j]);
#pragma unroll
    for (int j = 0; j < D; ++j)
        lv[j] = lds_ld<T>(ci[j]);
    typename A::Term a[D];
    typename A::Acc p[D];
    typename A::Acc acc = A::identity();
    Lanes sign = 0;
    uint64_t par = 0;
#pragma unroll
    for (int j = 0; j < D; ++j) {
        if constexpr (PAR)
            par ^= __ballot(lv[j] < T(0));
        check_forward<A>(lv[j] - rv[j], a[j], p[j], acc, sign);
    }
    typename A::Acc sx = A::seed(lane_swap<32>(acc));
    const Lanes sign_total = sign ^ lane_swap<32>(sign);
    if constexpr (PAR)
        odd |= some_odd(par);
#pragma unroll
    for (int j = D - 1; j >= 0; --j)
        lds_st<T>(msg[j], check_backward<A>(a[j], p[j], sx, sign_total));
}

// Minimum state of part of a row: its two smallest magnitudes and the parity
// of its negative messages.  Which edge holds the smallest needs no index: an
// edge whose magnitude equals m1 takes m2, and if another edge equals it too,
// m2 is that value.  NaN magnitudes count as +inf (the comparisons of
// min_add pass them over).
template <class T>
struct Min2 {
    T m1, m2;
    Lanes neg;
};
__device__ __forceinline__ float min_of(float a, float b) { return __builtin_fminf(a, b); }
__device__ __forceinline__ float max_of(float a, float b) { return __builtin_fmaxf(a, b); }
__device__ __forceinline__ double min_of(double a, double b) { return __builtin_fmin(a, b); }
__device__ __forceinline__ double max_of(double a, double b) { return __builtin_fmax(a, b); }
// The second smallest of m1 <= m2 and a (no NaN among them).
__device__ __forceinline__ float second_of(float m1, float m2, float a)
{
    return __builtin_amdgcn_fmed3f(m1, m2, a);
}
__device__ __forceinline__ double second_of(double m1, double m2, double a) { return min_of(m2, max_of(m1, a)); }
template <int M, class T>
__device__ __forceinline__ void min_merge(Min2<T> &s)
{
    const T o1 = lane_swap<M>(s.m1), o2 = lane_swap<M>(s.m2);
    s.neg ^= lane_swap<M>(s.neg);
    s.m2 = min_of(max_of(s.m1, o1), min_of(s.m2, o2));
    s.m1 = min_of(s.m1, o1);
}

// Messages of D slots of a min-sum row under min_message's rule, spread over
// two lanes (QUARTERS: four), from q: the correction and the clamp are applied
// to the row's two minima, and each edge selects one.
template <class A, int D, bool QUARTERS, class Store>
__device__ __forceinline__ void min_row(const typename A::T (&q)[D], typename A::T scale, typename A::T offset,
                                        const Store &store)
{
    using T = typename A::T;
    const T inf = T(__builtin_huge_val());
    Min2<T> s{inf, inf, 0};
    T a[D];
    Lanes neg[D];
#pragma unroll
    for (int j = 0; j < D; ++j) {
        a[j] = min_of(fabs(q[j]), inf);  // NaN: inf
        s.m2 = second_of(s.m1, s.m2, a[j]);
        s.m1 = min_of(s.m1, a[j]);
        neg[j] = __ballot(q[j] < T(0));
        s.neg ^= neg[j];
    }
    if constexpr (QUARTERS)
        min_merge<16>(s);
    min_merge<32>(s);
    auto corrected = [&](T m) {
        T mag = scale * m - offset;
        mag = mag > T(0) ? mag : T(0);
        return mag < T(A::kRmax) ? mag : T(A::kRmax);
    };
    const T r1 = corrected(s.m1), r2 = corrected(s.m2);
#pragma unroll
    for (int j = 0; j < D; ++j) {
        const T mag = a[j] == s.m1 ? r2 : r1;
        store(j, lane_of(s.neg ^ neg[j]) ? -mag : mag);
    }
}

// half_row under the min-sum rule.
template <class A, int D, bool PAR, bool POS, class Tab>
__device__ __forceinline__ void ms_half_row(Tab tab, const Messages<typename A::T, D, POS> &msg, bool &odd,
                                            typename A::T scale, typename A::T offset)
{
    using T = typename A::T;
    Addresses<T, D> ci;
    ci.load(tab, 64);
    T lv[D], q[D];
#pragma unroll
    for (int j = 0; j < D; ++j)
        q[j] = lds_ld<T>(msg[j]);
#pragma unroll
    for (int j = 0; j < D; ++j)
        lv[j] = lds_ld<T>(ci[j]);
    uint64_t par = 0;
#pragma unroll
    for (int j = 0; j < D; ++j) {
        if constexpr (PAR)
            par ^= __ballot(lv[j] < T(0));
        q[j] = lv[j] - q[j];
    }
    if constexpr (PAR)
        odd |= some_odd(par);
    min_row<A, D, false>(q, scale, offset, [&](int j, T r) { lds_st<T>(msg[j], r); });
}

// One quarter of a layered row of each lane (Section II, Algorithm 2, with the
// layered combination order of spa_math.h), D slots: the quarter combinations
// are exchanged in two steps, with the sibling quarter and then between the
// halves, which gives every lane O_i in the same association as the streaming
// layer kernel; new posteriors are stored at once.  `stride`: quads of one
// slot quad of the group (4 lanes per row).
template <class A, int D, class Tab>
__device__ __forceinline__ void layered_quarter(Tab tab, int stride, bool ms, typename A::T scale,
                                                typename A::T offset)
{
    using T = typename A::T;
    Addresses<T, D> ci, ri;
    ci.load(tab, stride);
    ri.load(tab + quads(D) * stride, stride);
    T q[D], rv[D];
#pragma unroll
    for (int j = 0; j < D; ++j) {
        q[j] = lds_ld<T>(ci[j]);
        rv[j] = lds_ld<T>(ri[j]);
    }
#pragma unroll
    for (int j = 0; j < D; ++j)
        q[j] = q[j] - rv[j];  // +inf for a dummy
    if (ms) {
        min_row<A, D, true>(q, scale, offset, [&](int j, T r) {
            lds_st<T>(ri[j], r);
            lds_st<T>(ci[j], q[j] + r);
        });
        return;
    }
    typename A::Term a[D];
    typename A::Acc p[D];
    typename A::Acc acc = A::identity();
    Lanes sign = 0;
#pragma unroll
    for (int j = 0; j < D; ++j)
        check_forward<A>(q[j], a[j], p[j], acc, sign);
    const typename A::Acc c_sib = lane_swap<16>(acc);
    const typename A::Acc c_other = lane_swap<32>(A::merge(acc, c_sib));  // the other half's combination
    typename A::Acc sx = A::seed(A::merge(c_sib, c_other));
    const Lanes sign_half = sign ^ lane_swap<16>(sign);
    const Lanes sign_total = sign_half ^ lane_swap<32>(sign_half);
#pragma unroll
    for (int j = D - 1; j >= 0; --j) {
        const T r = check_backward<A>(a[j], p[j], sx, sign_total);
        lds_st<T>(ri[j], r);
        lds_st<T>(ci[j], q[j] + r);
    }
}

// Exact-length bodies for D in [D, DB], by the group's longest part.
template <class A, int D, int DB, bool PAR, bool POS, bool MS, class Tab>
__device__ __forceinline__ void half_row_dispatch(int d, Tab tab, const Quad *pos, uint32_t ra, bool &odd,
                                                  typename A::T scale, typename A::T offset)
{
    if constexpr (D < DB) {
        if (d != D) {
            half_row_dispatch<A, D + 1, DB, PAR, POS, MS>(d, tab, pos, ra, odd, scale, offset);
            return;
        }
    }
    Messages<typename A::T, D, POS> msg;
    msg.ra = ra;
    if constexpr (POS)
        msg.pos.load(pos, 64);
    if constexpr (MS)
        ms_half_row<A, D, PAR, POS>(tab, msg, odd, scale, offset);
    else
        half_row<A, D, PAR, POS>(tab, msg, odd);
}

template <class A, int D, int DB, class Tab>
__device__ __forceinline__ void layered_dispatch(int d, Tab tab, int stride, bool ms, typename A::T scale,
                                                 typename A::T offset)
{
    if constexpr (D < DB) {
        if (d != D) {
            layered_dispatch<A, D + 1, DB>(d, tab, stride, ms, scale, offset);
            return;
        }
    }
    layered_quarter<A, D>(tab, stride, ms, scale, offset);
}

// acc plus a column's messages in ascending row order, D slots (dummies add -0).
template <class A, int D, class Tab>
__device__ __forceinline__ typename A::T column_sum(Tab tab, typename A::T acc)
{
    using T = typename A::T;
    if constexpr (D > 0) {
        Addresses<T, D> ad;
        ad.load(tab, 64);
        T rv[D];
#pragma unroll
        for (int k = 0; k < D; ++k)
            rv[k] = lds_ld<T>(ad[k]);
#pragma unroll
        for (int k = 0; k < D; ++k)
            acc += rv[k];
    }
    return acc;
}
constexpr int kColExact = 16;  // longer columns run in steps of four slots
template <class A, int D, class Tab>
__device__ __forceinline__ typename A::T column_dispatch(int d, Tab tab, typename A::T acc)
{
    if constexpr (D <= kColExact) {
        if (d == D)
            return column_sum<A, D>(tab, acc);
        return column_dispatch<A, D + 1>(d, tab, acc);
    } else {
        for (int i = 0; i < quads(d); ++i)
            acc = column_sum<A, 4>(tab + i * 64, acc);
        return acc;
    }
}

// Kernel instances: one for any batch, and three compiled with one schedule
// and rule only, in the padded message order, for batches whose jobs all allow
// it (FP32).
enum Instance { kAnyJob = 0, kFlood = 1, kLayered = 2, kMinSum = 3 };

// Four consecutive values of a frame's arrays.  Frames are moved by fours
// where n and the caller's pointers allow it (frame f starts f n values in).
template <class T>
using Four = T __attribute__((ext_vector_type(4)));
template <class T>
__device__ __forceinline__ bool by_four(int32_t n, const void *p)
{
    return (n & 3) == 0 && (reinterpret_cast<uintptr_t>(p) & (4 * sizeof(T) - 1)) == 0;
}

// A frame's posteriors (the channel values), the dummies' constants and its
// messages, which start at 0: the first iteration then forms q = L - 0 = L
// exactly, as the streaming kernels' first iteration, with the same code as
// every later one.
template <class A>
__device__ __forceinline__ void start_frame(const Code &c, const typename A::T *llr, int32_t r_words)
{
    using T = typename A::T;
    const int tid = static_cast<int>(threadIdx.x), NT = static_cast<int>(blockDim.x);
    const int32_t n = c.n;
    Lds<T> *sL = lds_at<T>(0);
    if (by_four<T>(n, llr)) {
        for (int j = 4 * tid; j < n; j += 4 * NT) {
            Four<T> v = *reinterpret_cast<const Four<T> *>(llr + j);
            v *= T(A::kIn);
            *reinterpret_cast<Lds<Four<T>> *>(sL + j) = v;
        }
    } else {
        for (int j = tid; j < n; j += NT)
            sL[j] = llr[j] * T(A::kIn);
    }
    if (tid == 0) {
        sL[n + kInfWord] = T(__builtin_huge_val());
        sL[n + kMinusZeroWord] = T(-0.0);
        sL[n + kJunkWord] = T(0);
    }
    // whole fours: the messages start at a multiple of four words, and
    // lds_bytes counts their last four
    Lds<Four<T>> *sR = reinterpret_cast<Lds<Four<T>> *>(sL + fused_first_message(n));
    for (int e = tid; 4 * e < r_words; e += NT)
        sR[e] = Four<T>(T(0));
    __syncthreads();
}

// One frame on the flooding schedule; returns the iterations it ran.
template <class A, int DB, Instance INST, bool LT>
__device__ __forceinline__ int32_t decode_frame(const Code &c, const Job &job, int64_t f, uint32_t tables, Vote &vote)
{
    using T = typename A::T;
    constexpr uint32_t TS = sizeof(T);
    const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
    const int lane = static_cast<int>(threadIdx.x & 63), nwaves = static_cast<int>(blockDim.x >> 6);
    const int32_t n = c.n, col_groups = (n + 63) / 64;
    const T *llr = static_cast<const T *>(job.llr) + f * n;
    Lds<T> *sL = lds_at<T>(0);
    const Table<LT> row_tab = table_at<LT>(c.row_tab, tables) + lane;
    const Quad *row_pos = reinterpret_cast<const Quad *>(c.row_pos) + lane;
    const Table<LT> col_tab =
        table_at<LT>(c.col_tab, tables + 4u * static_cast<uint32_t>(c.row_words)) + lane;
    const uint32_t r0 = TS * static_cast<uint32_t>(fused_first_message(n) + lane);
    start_frame<A>(c, llr, c.r_words);

    const bool es = (job.flags & LDPC_EARLY_STOP) != 0;
    const bool ms = INST == kMinSum || (INST == kAnyJob && (job.flags & LDPC_MIN_SUM) != 0);
    const bool pos = INST == kAnyJob && !LT && c.row_pos != nullptr;
    const T scale = static_cast<T>(job.ms_scale), offset = static_cast<T>(job.ms_offset * A::kIn);
    // Alone on its CU (LT), a wavefront keeps the words of its first groups: a
    // scalar load less in every phase.  Where others hide it, the selects cost more.
    const int32_t row0 = min(wave, c.row_groups - 1), col0 = min(wave, col_groups - 1);
    const int32_t row_w0 = LT && row0 >= 0 ? c.row_grp[2 * row0] : 0;
    const int32_t row_first0 = LT && row0 >= 0 ? c.row_grp[2 * row0 + 1] : 0;
    const int32_t col_w0 = LT ? c.col_grp[2 * col0] : 0, col_first0 = LT ? c.col_grp[2 * col0 + 1] : 0;
    for (int32_t t = 1; t <= job.max_iter; ++t) {
        bool odd = false;
        for (int g = wave; g < c.row_groups; g += nwaves) {
            // group word 0: message slots before the group (16 bits), its longest half; word 1: first quad
            const int32_t w = LT && g == wave ? row_w0 : c.row_grp[2 * g];
            const int32_t first = LT && g == wave ? row_first0 : c.row_grp[2 * g + 1];
            const int d = w >> 16;
            const uint32_t ra = r0 + TS * 64u * static_cast<uint32_t>(w & 0xffff);
            const Table<LT> tab = row_tab + first * 64;
            const Quad *pt = row_pos + static_cast<int64_t>(first) * 64;
            if (d == 0)
                continue;
            if (ms) {
                if constexpr (INST == kMinSum || INST == kAnyJob) {
                    if (INST == kAnyJob && !LT && pos)
                        half_row_dispatch<A, DB / 2, DB / 2, true, true, true>(d, tab, pt, ra, odd, scale, offset);
                    else
                        half_row_dispatch<A, 1, DB / 2, true, false, true>(d, tab, pt, ra, odd, scale, offset);
                }
            } else if constexpr (INST != kMinSum) {
                if (INST == kAnyJob && !LT && pos)
                    half_row_dispatch<A, DB / 2, DB / 2, true, true, false>(d, tab, pt, ra, odd, scale, offset);
                else if (es)
                    half_row_dispatch<A, 1, DB / 2, true, false, false>(d, tab, pt, ra, odd, scale, offset);
                else
                    half_row_dispatch<A, 1, DB / 2, false, false, false>(d, tab, pt, ra, odd, scale, offset);
            }
        }
        // The syndrome of x^(t-1), formed by the rows just run.
        if (es) {
            if (!vote.any(odd))  // a codeword: stop at t-1, keep L^(t-1)
                return t - 1;
        } else {
            __syncthreads();
        }
        for (int g = wave; g < col_groups; g += nwaves) {
            const int j = g * 64 + lane;
            T acc = T(0);
            if (j < n)
                acc = llr[j] * T(A::kIn);
            // longest column, first quad
            const int32_t d = LT && g == wave ? col_w0 : c.col_grp[2 * g];
            const int32_t first = LT && g == wave ? col_first0 : c.col_grp[2 * g + 1];
            const T v = column_dispatch<A, 0>(d, col_tab + first * 64, acc);
            if (j < n)
                sL[j] = v;
        }
        __syncthreads();
    }
    return job.max_iter;
}

// One frame on the layered schedule: the layers in order, the rows of a layer
// in parallel with four lanes each and a workgroup barrier between layers.
// With early stop the syndrome of [L < 0] is tested before the first pass and
// after every pass but the last.  Each row's arithmetic is the plain layered
// path's, bit for bit.  Returns the passes run.
template <class A, int DB, Instance INST, bool LT>
__device__ __forceinline__ int32_t decode_frame_layered(const Code &c, const Job &job, int64_t f, uint32_t tables,
                                                        int32_t turn, Vote &vote)
{
    using T = typename A::T;
    const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
    const int lane = static_cast<int>(threadIdx.x & 63), nwaves = static_cast<int>(blockDim.x >> 6);
    const T *llr = static_cast<const T *>(job.llr) + f * c.n;
    const Table<LT> row_tab = table_at<LT>(c.row_tab, tables) + lane;
    const Table<LT> lay_tab = table_at<LT>(c.lay_tab, tables + 4u * static_cast<uint32_t>(c.row_words));
    start_frame<A>(c, llr, c.E);

    // Whether some row is unsatisfied by the decision [L < 0], from the
    // flooding table.  A wavefront stops at its first group of 32 rows holding
    // one (the answer is then known; in most passes that is the first group).
    // That group's addresses are loaded at once; alone on its CU (LT), a wavefront
    // keeps them in registers from pass to pass (24 frames of qc n = 1296, rate
    // 2/3: 84.5 us per call without and 82.3 with), where frames share a CU, holding
    // 8 to 16 registers through every layer would cost resident wavefronts
    // (kFusedWavesPerEU).
    const bool es = (job.flags & LDPC_EARLY_STOP) != 0;
    constexpr int kFirstQuads = quads(DB / 2);
    struct First {
        Quad quad[kFirstQuads];
        int slots = 0;
    };
    auto load_first = [&]() {
        First f;
        if (wave < c.row_groups) {
            f.slots = c.row_grp[2 * wave] >> 16;
            const Table<LT> tab = row_tab + c.row_grp[2 * wave + 1] * 64;
#pragma unroll
            for (int i = 0; i < kFirstQuads; ++i)
                if (4 * i < f.slots)
                    f.quad[i] = tab[i * 64];
        }
        return f;
    };
    First kept;
    if (LT && es)
        kept = load_first();
    auto parity_of = [&](const Quad &q, uint64_t &par) {
#pragma unroll
        for (int k = 0; k < 4; ++k)
            par ^= __ballot(lds_ld<T>(static_cast<uint32_t>(q[k]) * static_cast<uint32_t>(sizeof(T) / 4)) < T(0));
    };
    auto unsatisfied = [&]() -> int32_t {
        const First first_group = LT ? kept : load_first();
        uint64_t par = 0;
#pragma unroll
        for (int i = 0; i < kFirstQuads; ++i)
            if (4 * i < first_group.slots)
                parity_of(first_group.quad[i], par);
        bool odd = some_odd(par);
        for (int g = wave + nwaves; g < c.row_groups && !odd; g += nwaves) {
            const int32_t w = c.row_grp[2 * g], first = c.row_grp[2 * g + 1];
            const Table<LT> tab = row_tab + first * 64;
            par = 0;
            for (int i = 0; i < quads(w >> 16); ++i) {
                const Quad q = tab[i * 64];
                parity_of(q, par);
            }
            odd = some_odd(par);
        }
        return vote.any(odd);
    };

    const bool ms = INST == kAnyJob && (job.flags & LDPC_MIN_SUM) != 0;
    const T scale = static_cast<T>(job.ms_scale), offset = static_cast<T>(job.ms_offset * A::kIn);
    if (es && !unsatisfied())
        return 0;
    // The group a wavefront takes first in a layer, and where the layer after
    // it ends, are read a layer ahead, by vector loads (scalar ones return out
    // of order, so that every LDS wait would wait for them too): the two reads
    // depend on each other and would start every layer with both latencies.
    int lane0 = 0;
    asm("" : "+v"(lane0));  // the same in every lane, which the compiler does not know
    const int32_t nlayers = c.nlayers, ngroups = c.lay_ptr[nlayers];
    auto group_words = [&](int32_t g, int32_t &w, int32_t &first) {
        const int32_t *at = c.lay_grp + 2 * min(g, ngroups - 1) + lane0;
        w = at[0];
        first = at[1];
    };
    auto layer_after = [&](int32_t l) { return l + 1 == nlayers ? 0 : l + 1; };
    // This wavefront's first group of the layer; `turn` swaps pairs of
    // wavefronts from layer to layer (layer_turn).
    int mine = wave;
    int32_t begin = 0, end = c.lay_ptr[1], w_ahead, first_ahead;
    int32_t end_ahead = c.lay_ptr[layer_after(0) + 1 + lane0];
    group_words(mine, w_ahead, first_ahead);
    for (int32_t t = 1; t <= job.max_iter; ++t) {
        for (int32_t l = 0; l < nlayers; ++l) {
            const int32_t next = layer_after(l), next_begin = next == 0 ? 0 : end;
            const int32_t next_end = __builtin_amdgcn_readfirstlane(end_ahead);
            int32_t w = __builtin_amdgcn_readfirstlane(w_ahead), first = __builtin_amdgcn_readfirstlane(first_ahead);
            int g = begin + mine;
            if (!LT)
                mine ^= turn;
            group_words(next_begin + mine, w_ahead, first_ahead);
            end_ahead = c.lay_ptr[layer_after(next) + 1 + lane0];
            while (g < end) {
                const int rows = w & 0xff, d = w >> 8;  // first: the group's first quad
                if ((lane & 15) < rows && d > 0)
                    layered_dispatch<A, 1, DB / 4>(
                        d, lay_tab + (first + (lane >> 4) * rows + (lane & 15)), 4 * rows, ms, scale, offset);
                g += nwaves;
                if (g < end) {
                    w = c.lay_grp[2 * g];
                    first = c.lay_grp[2 * g + 1];
                }
            }
            begin = next_begin;
            end = next_end;
            __syncthreads();
        }
        if (es && t < job.max_iter && !unsatisfied())
            return t;
    }
    return job.max_iter;
}

// Bits, iteration count and posterior of a decoded frame (stopped after `it`
// iterations; one that ran none reports the caller's LLRs bit-exactly).
template <class A>
__device__ __forceinline__ void write_frame(const Code &c, const Job &job, int64_t f, int32_t it)
{
    using T = typename A::T;
    const int tid = static_cast<int>(threadIdx.x), NT = static_cast<int>(blockDim.x);
    const int32_t n = c.n;
    const Lds<T> *sL = lds_at<T>(0);
    const T *llr = static_cast<const T *>(job.llr) + f * n;
    uint8_t *bits = job.bits + f * n;
    T *post = job.post ? static_cast<T *>(job.post) + f * n : nullptr;
    if (by_four<T>(n, llr) && by_four<T>(n, post) && by_four<uint8_t>(n, bits)) {
        for (int j = 4 * tid; j < n; j += 4 * NT) {
            Four<T> v = *reinterpret_cast<const Lds<Four<T>> *>(sL + j);
            uint32_t four = 0;
#pragma unroll
            for (int k = 0; k < 4; ++k)
                four |= static_cast<uint32_t>(v[k] < T(0)) << (8 * k);
            *reinterpret_cast<uint32_t *>(bits + j) = four;
            if (post) {
                if (it == 0)
                    v = *reinterpret_cast<const Four<T> *>(llr + j);
                else
                    v *= T(A::kOut);
                *reinterpret_cast<Four<T> *>(post + j) = v;
            }
        }
        if (tid == 0)
            job.iters[f] = it;
        return;
    }
    for (int j = tid; j < n; j += NT) {
        const T v = sL[j];
        bits[j] = static_cast<uint8_t>(v < T(0));
        if (post)
            post[j] = it == 0 ? llr[j] : v * T(A::kOut);
    }
    if (tid == 0)
        job.iters[f] = it;
}

// A launch's items are handed out in one of two ways.  Up to as many items as
// the device holds workgroups at once (counter null): one workgroup each, and
// the launch, whose job table arrives by value, is the whole call (a kernel
// that first wrote the table and a counter to memory cost a 64-frame batch 10
// of its 75 us).  More items: resident workgroups that draw their next item
// from *counter, which starts at 0.  There the hardware's own dispatch of one
// workgroup per item is slower where frames run different numbers of
// iterations, since it deals the items to the XCDs in turn whatever their
// load (4096 layered frames of n = 1944 with early stop: 1463 against 1358
// us; a static stride over the items: 2045 us).
// Workgroup b's first item is b; the next is counted from the grid's end on.
// Called by all threads; `drawn` is thread 0's draw, issued before the frame's
// outputs are written, so that the writes cover its latency.
__device__ __forceinline__ uint32_t draw_item(uint32_t *counter)
{
    return counter != nullptr && threadIdx.x == 0 ? atomicAdd(counter, 1u) : 0u;
}
__device__ __forceinline__ int32_t next_item(const uint32_t *counter, uint32_t drawn, int32_t nitems,
                                             Lds<int32_t> *flags)
{
    if (counter == nullptr)
        return nitems;
    if (threadIdx.x == 0)
        flags[kItemFlag] = static_cast<int32_t>(min(drawn + gridDim.x, static_cast<uint32_t>(nitems)));
    __syncthreads();
    return __builtin_amdgcn_readfirstlane(flags[kItemFlag]);
}

// Batch kernel.  FP32 bodies are held to 128 VGPRs, so that a CU holds 16
// wavefronts (4 per SIMD): two 512-thread workgroups for n = 1944, whose LDS
// admits no third, or one of 1024.  FP64 bodies get 256 VGPRs.  The layered
// instance is bound by the latency of a layer (gather, exchange, scatter,
// barrier), which a CU's other frames hide, and its frames are small: where
// frames share a CU it is held to the registers of 6 wavefronts per SIMD (5 for
// rows longer than 24; both spill one pair, once per frame).  us per call of 6
// passes, 4000 frames of qc n = 1584 at rates 2/3, 3/4 and 5/6 with 4 and 6
// wavefronts per SIMD (and 8, with 61 registers and the terms parked in LDS): 588
// and 460 (511), 440 and 349 (388), 303 and 241 (275); n = 648 at rate 1/2 358 and
// 303 (545).
template <class A, int DB, Instance INST, bool LT>
constexpr int kFusedWavesPerEU =
    !std::is_same<A, ArithF32>::value ? 2 : INST == kLayered && !LT ? (DB <= 24 ? 6 : 5) : 4;
template <class A>
constexpr int kFusedMaxThreads = std::is_same<A, ArithF32>::value ? kMaxThreads : kBaseThreads;

// The code's tables for a job, copied into LDS at b.tables_at (published by the
// barrier of start_frame).
__device__ __forceinline__ void copy_tables(const Batch &b, const Code &c, const Job &job)
{
    Lds<Quad> *to = lds_at<Quad>(b.tables_at);
    const int32_t rows = c.row_words / 4, rest = ((job.flags & LDPC_LAYERED) ? c.lay_words : c.col_words) / 4;
    const Quad *row_tab = reinterpret_cast<const Quad *>(c.row_tab);
    const Quad *tab = reinterpret_cast<const Quad *>((job.flags & LDPC_LAYERED) ? c.lay_tab : c.col_tab);
    for (int i = static_cast<int>(threadIdx.x); i < rows; i += static_cast<int>(blockDim.x))
        to[i] = row_tab[i];
    for (int i = static_cast<int>(threadIdx.x); i < rest; i += static_cast<int>(blockDim.x))
        to[rows + i] = tab[i];
}

template <class A, int DB, Instance INST = kAnyJob, bool LT = false>
__global__ __launch_bounds__(kFusedMaxThreads<A>) __attribute__((amdgpu_waves_per_eu(kFusedWavesPerEU<A, DB, INST, LT>))) void k_fused(const Batch b, uint32_t *counter)
{
    Lds<int32_t> *flags = lds_at<int32_t>(b.flags_at);
    if (threadIdx.x < kFlagWords)
        flags[threadIdx.x] = 0;  // published by the barrier of start_frame
    Vote vote{flags};
    for (int32_t item = static_cast<int32_t>(blockIdx.x); item < b.nitems;) {
        const int32_t j = job_of_item(b, item);
        const Job &job = b.jobs[j];
        const Code &c = b.codes[job.code];
        const int32_t f0 = (item - b.begin[j]) * b.frames_per_item;
        uint32_t drawn = 0;
        if constexpr (LT)
            copy_tables(b, c, job);
        for (int32_t f = f0; f < f0 + b.frames_per_item && f < job.frames; ++f) {
            if (f > f0)
                __syncthreads();  // the last frame's posteriors have been read
            int32_t it;
            if (INST == kLayered || (INST == kAnyJob && (job.flags & LDPC_LAYERED)))
                it = decode_frame_layered<A, DB, INST, LT>(c, job, f, b.tables_at, b.layer_turn, vote);
            else
                it = decode_frame<A, DB, INST, LT>(c, job, f, b.tables_at, vote);
            if (f == f0)
                drawn = draw_item(counter);
            write_frame<A>(c, job, f, it);
        }
        item = next_item(counter, drawn, b.nitems, flags);
    }
}

// The instance of k_fused that runs every job of the batch.
inline Instance batch_instance(const Batch &b)
{
    for (int32_t k = 0; k < b.ncodes; ++k)
        if (b.codes[k].row_pos != nullptr)
            return kAnyJob;
    const uint32_t first = b.jobs[0].flags & (LDPC_LAYERED | LDPC_MIN_SUM);
    for (int32_t k = 0; k < b.njobs; ++k)
        if ((b.jobs[k].flags & (LDPC_LAYERED | LDPC_MIN_SUM)) != first)
            return kAnyJob;
    if (first == 0)
        return kFlood;
    return first == LDPC_LAYERED ? kLayered : first == LDPC_MIN_SUM ? kMinSum : kAnyJob;
}

}  // namespace fused

namespace fused {

// Workgroups per CU and CU count for a launch of kernel fn with this LDS size
// and block size on the current device.  The runtime calls behind them (the
// kernel's LDS limit, the occupancy query, the device attribute) run once per
// (kernel, device, LDS bytes, threads) and are cached, not repeated on every
// launch; the LDS limit is only ever raised.  The caches are fixed-size
// tables (no heap allocation on any call): when the shape table is full it
// starts over, and a kernel missing from the full limit table has its limit
// set on every launch of a new shape.
inline ldpc_status launch_shape(const void *fn, size_t lds, int threads, int &per_cu, int &cus)
{
    struct Shape {
        const void *fn;
        int dev;
        size_t lds;
        int threads, per_cu, cus;
    };
    struct Limit {
        const void *fn;
        int dev;
        size_t lds;
    };
    constexpr int kShapes = 256, kLimits = 512;  // (38 kernels, on up to 13 devices)
    static std::mutex mu;
    static Shape shapes[kShapes];
    static Limit limits[kLimits];
    static int nshapes = 0, nlimits = 0;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess)
        return LDPC_EDEVICE;
    std::lock_guard<std::mutex> lk(mu);
    for (int i = 0; i < nshapes; ++i) {
        const Shape &e = shapes[i];
        if (e.fn == fn && e.dev == dev && e.lds == lds && e.threads == threads) {
            per_cu = e.per_cu;
            cus = e.cus;
            return LDPC_OK;
        }
    }
    Limit *lim = nullptr;
    for (int i = 0; i < nlimits; ++i)
        if (limits[i].fn == fn && limits[i].dev == dev)
            lim = &limits[i];
    if (lim == nullptr || lim->lds < lds) {
        if (hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds)) != hipSuccess)
            return LDPC_EUNSUPPORTED;
        if (lim != nullptr)
            lim->lds = lds;
        else if (nlimits < kLimits)
            limits[nlimits++] = Limit{fn, dev, lds};
    }
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, threads, lds) != hipSuccess || per_cu < 1)
        return LDPC_EUNSUPPORTED;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
        return LDPC_EDEVICE;
    if (nshapes == kShapes)  // batches of many different code mixes: start over
        nshapes = 0;
    shapes[nshapes++] = Shape{fn, dev, lds, threads, per_cu, cus};
    return LDPC_OK;
}

}  // namespace fused

namespace fused {

// LDS bytes of a launch, up to and with its flag words.
inline size_t batch_lds_bytes(const Batch &b, size_t tsize)
{
    size_t bytes = 0;
    for (int32_t i = 0; i < b.njobs; ++i) {
        const Code &c = b.codes[b.jobs[i].code];
        bytes = std::max(bytes, lds_bytes(c.n, (b.jobs[i].flags & LDPC_LAYERED) ? c.E : c.r_words, tsize));
    }
    return bytes;
}

// LDS bytes of a launch whose workgroups hold their code's tables too, or 0 if
// a job's tables lie in CSR order; sets where they start.
inline size_t batch_table_lds_bytes(const Batch &b, size_t tsize, uint32_t &tables_at)
{
    const size_t frame = batch_lds_bytes(b, tsize) - kFlagWords * sizeof(int32_t);
    size_t words = 0;
    for (int32_t i = 0; i < b.njobs; ++i) {
        const Code &c = b.codes[b.jobs[i].code];
        if (c.row_pos != nullptr)
            return 0;
        const bool layered = (b.jobs[i].flags & LDPC_LAYERED) != 0;
        words = std::max(words, static_cast<size_t>(c.row_words) + static_cast<size_t>(layered ? c.lay_words : c.col_words));
    }
    tables_at = static_cast<uint32_t>(frame);
    return frame + words * sizeof(int32_t) + kFlagWords * sizeof(int32_t);
}

// Workgroup size of a launch whose caller left it at kBaseThreads, for the job
// with the most rows to run.  Measured on MI355X over eleven codes, 64 to 4000
// frames and 64 to 1024 threads; the figures are us per call of 10 iterations
// by wavefronts per workgroup.
//
// Every frame has a CU to itself: the size with the shortest chain of rounds.
// A wavefront takes 32 check rows at a time and 64 columns; the unit is a
// group's VALU time on a whole CU (a wavefront alone on its SIMD takes 4), a
// round's latency 11 of them in FP32 and 5 in FP64, a column round's 2.  (64
// frames of qc n = 1944: 4, 8, 12, 16 wavefronts 133, 86, 72, 70; n = 648,
// eleven groups: 4, 8, 11, 16 55, 40, 34, 34.)  A layer's rows, 16 to a
// wavefront, are one round, and wider workgroups wait at its barriers.
//
// Frames share the CUs: the fewest wavefronts per frame, in fours (one to each
// SIMD: sizes between place unevenly), with which the resident frames hold 16
// on a CU, 24 for min-sum, whose rounds are mostly latency; but 8 for more than
// twelve groups.  (4000 frames: qc n = 648 4, 5, 8, 11 wavefronts 270, 357,
// 357, 506; n = 1944 4, 8, 12, 16 1221, 851, 1104, 1069; (3,6)-regular n =
// 2040 462, 382, 395, 595; min-sum n = 1944 861, 565, 466, 647.)  Workgroups
// that would fill a CU's 32 wavefronts in one pass did not all start at once
// (1024 min-sum frames of n = 648: 4 and 8 wavefronts 56 and 73), and a size
// that needs a second pass where a smaller one does not is no gain.  FP64
// sum-product takes the wider of equals (1024 frames of n = 648: 4 and 8
// wavefronts 325 and 299), and with early stop the wider always, which ends the
// last pass's long frames sooner.  Layered frames: a layer's rows in one round, at
// most 8 wavefronts where a CU holds two frames (4000 frames of qc n = 1944: 4,
// 6, 7, 8 wavefronts 2210, 1651, 1651, 1517), and one to spare for the layers of two
// wavefronts or less (n = 648: 1, 2, 3, 6 wavefronts 723, 489, 492, 796).
template <class K>
ldpc_status workgroup_threads(K kern, const Batch &b, size_t tsize, size_t lds, int max_threads, int &threads)
{
    const bool f32 = tsize == sizeof(float);
    const Job *main_job = &b.jobs[0];
    int64_t most = -1;
    bool stops = false;
    for (int32_t i = 0; i < b.njobs; ++i) {
        const Job &j = b.jobs[i];
        stops |= (j.flags & LDPC_EARLY_STOP) != 0;
        const int64_t work = static_cast<int64_t>(j.frames) * b.codes[j.code].m;
        if (work > most) {
            most = work;
            main_job = &j;
        }
    }
    const Code &c = b.codes[main_job->code];
    const bool layered = (main_job->flags & LDPC_LAYERED) != 0, ms = (main_job->flags & LDPC_MIN_SUM) != 0;
    const int max_waves = max_threads / 64, g = (c.m + 31) / 32, cols = (c.n + 63) / 64;
    int per_cu = 0, cus = 0;
    const auto shape = [&](int w) {
        return launch_shape(reinterpret_cast<const void *>(kern), lds, w * 64, per_cu, cus);
    };
    ldpc_status rc = shape(4);
    if (rc != LDPC_OK)
        return rc;
    const int64_t share = (b.nitems + cus - 1) / cus;  // frames per CU
    int best = 4;
    if (layered) {
        const int most_rows = (c.layer_rows + 15) / 16;
        const int mean_rows = (c.m / std::max(c.nlayers, 1) + 15) / 16;
        if (share <= 1)
            best = std::max({most_rows, c.n / 256 + 1, 2});
        else if (mean_rows <= 2)
            best = std::max(mean_rows, 1) + 1;
        else {
            rc = shape(8);
            if (rc != LDPC_OK)
                return rc;
            best = std::min((most_rows + 3) / 4 * 4, per_cu >= 2 ? 8 : max_waves);
        }
        best = std::min(best, max_waves);
    } else if (share <= 1) {
        const int unit = ms ? 1 : 3, round = 3 * (f32 ? 11 : 5);  // in thirds
        int least = 0;
        for (int w = 2; w <= max_waves; ++w) {
            const int rest = (g % w + 3) / 4 * 4;
            const int time = std::max(unit * g, g / w * std::max(round, unit * ((w + 3) / 4 * 4)) +
                                                    (rest > 0 ? std::max(round, unit * rest) : 0) +
                                                    (cols + w - 1) / w * 6);
            if (least == 0 || time < least) {
                least = time;
                best = w;
            }
        }
    } else {
        const int64_t enough = f32 ? (ms ? 24 : 16) : stops ? 24 : 16;
        int64_t held = 0;
        bool one_pass = false;
        for (int w = g <= 12 ? 4 : 8; w <= max_waves && held < enough; w += 4) {
            rc = shape(w);
            if (rc != LDPC_OK)
                return rc;
            const int64_t waves = std::min<int64_t>(per_cu, share) * w;
            if ((f32 && waves > 28 && share <= per_cu) || (one_pass && share > per_cu))
                continue;
            if (waves > held || (waves == held && !f32 && !ms)) {
                held = waves;
                best = w;
                one_pass = f32 && share <= per_cu;
            }
        }
    }
    threads = best * 64;
    return LDPC_OK;
}

}  // namespace fused

namespace fused {

// By what a wavefront's place in a layer changes (^) from each layer to the next.
// Five to seven groups on the first of eight wavefronts give some of the four
// SIMDs twice the work of the others, in both frames of a CU that holds two;
// swapping the first two wavefronts with the next two, and the last, evens that
// out.  us per call of 6 passes, 4000 frames, fixed and swapping: qc n = 1944 at
// rate 1/2 992 and 920, n = 2304 at rate 2/3 669 and 617.  With any other share
// there is nothing to even out, and a changing first wavefront costs up to 10%
// (fixed and changing: one frame of ten groups to a CU, qc n = 3840 at rate 3/4
// 715 and 753; one of eight groups, qc n = 3072, 64 frames 69 and 76; 700 frames of
// n = 648 at rate 1/2, two groups, 91 and 95).
inline int32_t layer_turn(const Batch &b, int threads, int per_cu, int cus)
{
    int32_t rows = 0;
    for (int32_t i = 0; i < b.njobs; ++i)
        if (b.jobs[i].flags & LDPC_LAYERED)
            rows = std::max(rows, b.codes[b.jobs[i].code].layer_rows);
    const int32_t groups = (rows + 15) / 16;
    return threads == 512 && per_cu == 2 && b.nitems > cus && groups > 4 && groups < 8 ? 2 : 0;
}

}  // namespace fused

// Sets a launch's item counter to 0.
void launch_zero_counter(uint32_t *counter, hipStream_t s, bool profile);

// Launcher of the fused kernel for codes of row degree <= DB (one
// translation unit per dtype and bucket).
// counter: a device word of the launch's own (its items' queue when they
// exceed the resident workgroups).
// profile = false keeps the launch out of ldpc_profile_* timing (whose event
// pool may create events).
template <class A, int DB>
ldpc_status launch_fused_bucket(fused::Batch &batch, uint32_t *counter, int threads, hipStream_t s, bool profile);

// lds_bytes: the launch's LDS, its flag words last.
template <class A, class K>
ldpc_status launch_fused_kernel(K kern, fused::Batch &batch, size_t lds_bytes, uint32_t *counter, int threads,
                                hipStream_t s, bool profile)
{
    batch.flags_at = static_cast<uint32_t>(lds_bytes - fused::kFlagWords * sizeof(int32_t));
    if (threads == fused::kBaseThreads) {
        const ldpc_status rc = fused::workgroup_threads(kern, batch, sizeof(typename A::T), lds_bytes,
                                                        fused::kFusedMaxThreads<A>, threads);
        if (rc != LDPC_OK)
            return rc;
    }
    int per_cu = 0, cus = 0;
    const ldpc_status shape_rc =
        fused::launch_shape(reinterpret_cast<const void *>(kern), lds_bytes, threads, per_cu, cus);
    if (shape_rc != LDPC_OK)
        return shape_rc;
    batch.layer_turn = fused::layer_turn(batch, threads, per_cu, cus);
    const int32_t resident = per_cu * cus;
    if (batch.nitems <= resident)
        counter = nullptr;  // one workgroup per item
    else
        launch_zero_counter(counter, s, profile);
    ProfScope ps(LDPC_KERNEL_FUSED, s, profile);
    LDPC_LAUNCH(ps, kern, dim3(static_cast<unsigned>(std::min(batch.nitems, resident))), dim3(threads),
                static_cast<uint32_t>(lds_bytes), s, batch, counter);
    return hipGetLastError() == hipSuccess ? LDPC_OK : LDPC_EDEVICE;
}

// Launches an instance: with the tables copied to LDS where every item has a CU
// to itself and they fit, else with the tables in L2.
template <class A, int DB, fused::Instance INST>
ldpc_status launch_fused_instance(fused::Batch &batch, uint32_t *counter, int threads, hipStream_t s, bool profile)
{
    constexpr size_t tsize = sizeof(typename A::T);
    int dev = 0, cus = 0, limit = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        hipDeviceGetAttribute(&limit, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess)
        return LDPC_EDEVICE;
    if (batch.nitems <= cus) {
        const size_t bytes = fused::batch_table_lds_bytes(batch, tsize, batch.tables_at);
        if (bytes != 0 && bytes <= static_cast<size_t>(limit))
            return launch_fused_kernel<A>(fused::k_fused<A, DB, INST, true>, batch, bytes, counter, threads, s,
                                          profile);
    }
    return launch_fused_kernel<A>(fused::k_fused<A, DB, INST, false>, batch, fused::batch_lds_bytes(batch, tsize),
                                  counter, threads, s, profile);
}

#define LDPC_DEFINE_FUSED_BUCKET(A_, DB_)                                                                        \
    template <>                                                                                                  \
    ldpc_status launch_fused_bucket<A_, DB_>(fused::Batch & batch, uint32_t *counter, int threads,               \
                                             hipStream_t s, bool profile)                                        \
    {                                                                                                            \
        if constexpr (std::is_same<A_, ArithF32>::value) {                                                       \
            switch (fused::batch_instance(batch)) {                                                              \
            case fused::kFlood:                                                                                  \
                return launch_fused_instance<A_, DB_, fused::kFlood>(batch, counter, threads, s, profile);       \
            case fused::kLayered:                                                                                \
                return launch_fused_instance<A_, DB_, fused::kLayered>(batch, counter, threads, s, profile);     \
            case fused::kMinSum:                                                                                 \
                return launch_fused_instance<A_, DB_, fused::kMinSum>(batch, counter, threads, s, profile);      \
            default: break;                                                                                      \
            }                                                                                                    \
        }                                                                                                        \
        return launch_fused_instance<A_, DB_, fused::kAnyJob>(batch, counter, threads, s, profile);              \
    }

}  // namespace ldpc
