// Flooding for a few frames of a code too long for the frame-resident kernel:
// one launch per iteration instead of two.
//
// With up to kFewFrames frames the streaming kernels are bound by their
// launches (about 5 us each at any size below that): a chunk's 64 lanes are
// mostly padding, and a check and a variable launch follow each other for
// every iteration, also after the last frame has stopped.  Here one launch is
// a whole iteration (arxiv 1812.06545, Section II, Algorithm 1): the check rows
// form the posteriors they need, L_n = Lch_n + sum of r_mn in ascending row
// order, from the messages of the iteration before, so no variable launch has
// to come first.  A column's sum is formed once per row that holds it, which
// multiplies the reads of r by the mean column degree; the rule that picks
// this path (few_frames_groups) bounds that product.  The messages alternate
// between two buffers; nothing else passes from launch to launch.
//
// One wavefront is one check row of FW frames: lane k FW + f holds edge k of
// frame f.  The lanes sum their columns, exchange their edges' terms through
// LDS, and each forms its own exclusive combination in the order of the other
// paths (spa_math.h), so that every message has their bits.
//
// Early stop: launch t forms the syndrome of x^(t-1) and marks unsatisfied
// frames.  Launch t + 1 finds a frame that launch t left unmarked stopped at
// t - 1 and leaves its messages alone from then on: those of iteration t - 1
// stay in their buffer, from which the output launch forms its posteriors.
#include <algorithm>
#include <type_traits>

#include "few_layout.h"
#include "flood_kernels.h"
#include "minsum_kernels.h"

namespace ldpc {
namespace {

// Two message buffers of up to 32 frames take the place of a 64-frame chunk's one.
constexpr int kFewFrames = 32;
// Frames per wavefront for rows of degree d.
constexpr int few_width(int d) { return d <= 8 ? 8 : d <= 16 ? 4 : 2; }

template <class A>
struct FewArgs {
    using T = typename A::T;
    const int32_t *row_ptr, *col_idx, *col_ptr, *col_edge;
    int32_t m, n, W, groups;    // W: frames of storage (a multiple of FW); groups: frame groups of FW
    const T *Lch;               // [n][W]
    const T *Rold;              // [E][W]: the messages of iteration t - 1
    T *Rnew;
    int32_t *done;              // [W]: iteration a frame stopped at, or -1
    const int32_t *unsat_prev;  // [W] of launch t - 1 (null for t = 1)
    int32_t *unsat;             // [W] of this launch
    int32_t t;
    T scale, offset;
};

// Scaled channel values [n][W] (padding frames get LLR 1) and the frames' state.
template <class A>
__global__ __launch_bounds__(256) void k_few_ingest(const typename A::T *__restrict__ llr, int32_t F, int32_t n,
                                                    int32_t W, typename A::T *__restrict__ Lch,
                                                    int32_t *__restrict__ done, int32_t *__restrict__ unsat,
                                                    int64_t unsat_words, int64_t words)
{
    using T = typename A::T;
    const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < words; i += stride) {
        if (i < W)
            done[i] = -1;
        if (i < unsat_words)
            unsat[i] = 0;
        if (i < static_cast<int64_t>(n) * W) {
            const int32_t f = static_cast<int32_t>(i) % W, c = static_cast<int32_t>(i) / W;
            const T v = f < F ? llr[static_cast<int64_t>(f) * n + c] : T(1);
            Lch[i] = v * T(A::kIn);
        }
    }
}

// Byte offset of frame f of item i in an array [items][W]: 24-bit factors and a
// 32-bit product (few_frames_groups bounds them).
template <class T>
__device__ __forceinline__ uint32_t frame_offset(uint32_t i, uint32_t W, uint32_t f)
{
    return (__umul24(i, W) + f) * static_cast<uint32_t>(sizeof(T));
}

// L of a column: the channel value and its messages in ascending row order, the
// loads of eight edges issued before their sum.  Past the column's end the last
// edge is read again and not added.
template <class T>
__device__ __forceinline__ T few_column(T acc, const int32_t *__restrict__ edges, int32_t dv, const T *__restrict__ R,
                                        int32_t W, int32_t f)
{
    constexpr int kStep = 8;
    for (int32_t j0 = 0; j0 < dv; j0 += kStep) {
        T v[kStep];
#pragma unroll
        for (int j = 0; j < kStep; ++j) {
            const uint32_t e = static_cast<uint32_t>(edges[min(j0 + j, dv - 1)]);
            v[j] = flood::ld_lane(R, frame_offset<T>(e, static_cast<uint32_t>(W), static_cast<uint32_t>(f)));
        }
#pragma unroll
        for (int j = 0; j < kStep; ++j)
            acc = j0 + j < dv ? acc + v[j] : acc;
    }
    return acc;
}

// Orders a wavefront's LDS writes before its lanes' reads of each other's.
__device__ __forceinline__ void wave_exchange()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <class A, int KL, bool FIRST, bool ES, bool MS>
__global__ __launch_bounds__(256) void k_few(FewArgs<A> a)
{
    using T = typename A::T;
    constexpr int FW = few_width(KL);
    static_assert(FW * KL == 64, "a wavefront is KL edges of FW frames");
    __shared__ T s_t[4][64], s_u[4][64];  // sum-product: an edge's t and u, by slot; min-sum: its |q| (in s_t)
    const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
    const int lane = static_cast<int>(threadIdx.x & 63), k = lane / FW;
    const int64_t item = static_cast<int64_t>(blockIdx.x) * 4 + wave;
    const int32_t row = static_cast<int32_t>(item / a.groups), f = static_cast<int32_t>(item % a.groups) * FW + lane % FW;
    if (row >= a.m)
        return;
    bool stopped = false;
    if constexpr (ES && !FIRST) {
        const int32_t dn = a.done[f];
        const bool stops = dn < 0 && a.unsat_prev[f] == 0;
        stopped = dn >= 0 || stops;
        if (row == 0 && k == 0 && stops)
            a.done[f] = a.t - 2;
        if (__all(stopped))
            return;
    }
    const int32_t e0 = a.row_ptr[row], d = a.row_ptr[row + 1] - e0;
    const bool real = k < d;
    T L = T(0), q = T(0);
    if (real) {
        const int32_t c = a.col_idx[e0 + k];
        L = flood::ld_lane(a.Lch, frame_offset<T>(static_cast<uint32_t>(c), a.W, f));
        if constexpr (FIRST) {
            q = L;
        } else {
            const T own = flood::ld_lane(a.Rold, frame_offset<T>(static_cast<uint32_t>(e0 + k), a.W, f));
            const int32_t b = a.col_ptr[c];
            L = few_column(L, a.col_edge + b, a.col_ptr[c + 1] - b, a.Rold, a.W, f);
            q = L - own;
        }
    }
    // lanes of one frame: bits f, f + FW, ..
    constexpr uint64_t kFrameLanes = ~0ull / ((1ull << FW) - 1);
    if constexpr (ES) {
        const uint64_t ones = __ballot(real && L < T(0)) >> (lane % FW) & kFrameLanes;
        if (k == 0 && (__popcll(ones) & 1) != 0)
            a.unsat[f] = 1;
    }
    T r;
    if constexpr (MS) {
        const uint64_t negs = __ballot(real && q < T(0)) >> (lane % FW) & kFrameLanes;
        s_t[wave][lane] = fabs(q);
        wave_exchange();
        T low = T(__builtin_huge_val());
        for (int j = 0; j < d; ++j) {
            const T x = s_t[wave][j * FW + lane % FW];
            low = j != k && x < low ? x : low;
        }
        T mag = a.scale * low - a.offset;
        mag = mag > T(0) ? mag : T(0);
        mag = mag < T(A::kRmax) ? mag : T(A::kRmax);
        r = ((__popcll(negs) & 1) != 0) != (q < T(0)) ? -mag : mag;
    } else {
        const typename A::Term own = A::term(q);
        const uint64_t neg_all = own.neg & __ballot(real);
        const uint64_t negs = neg_all >> (lane % FW) & kFrameLanes;
        // The halves lie in slots 0 .. KH - 1 and KH .. 2 KH - 1, each from its
        // first edge on; the lanes past the row's end fill the other slots with
        // identities (t = 1, u = 0), which change no bit of a combination, so
        // that every lane runs the same straight code over its own half and the
        // other.
        constexpr int KH = KL / 2;
        const int h = (d + 1) / 2, spare = k - d;
        const int own_lo = k < h ? 0 : KH, at = k < h ? k : k - h;  // this edge's half, its place there
        const int slot = real ? own_lo + at : spare < KH - h ? h + spare : d - h + KH + spare - (KH - h);
        s_t[wave][slot * FW + lane % FW] = real ? own.t : T(1);
        s_u[wave][slot * FW + lane % FW] = real ? own.u : T(0);
        wave_exchange();
        auto term_at = [&](int j, bool use) {
            typename A::Term x;
            const T t = s_t[wave][j * FW + lane % FW], u = s_u[wave][j * FW + lane % FW];
            x.t = use ? t : T(1);
            x.u = use ? u : T(0);
            return x;
        };
        typename A::Acc p = A::identity(), other = A::identity();
#pragma unroll
        for (int j = 0; j < KH - 1; ++j)
            p = A::add(p, term_at(own_lo + j, j < at));
#pragma unroll
        for (int j = 0; j < KH; ++j)
            other = A::add(other, term_at(KH - own_lo + j, true));
        typename A::Acc s = A::seed(other);
#pragma unroll
        for (int j = KH - 1; j > 0; --j)
            s = A::add(s, term_at(own_lo + j, j > at));
        const T mag = A::message(A::merge(p, s));
        r = ((__popcll(negs) & 1) != 0) != ((neg_all >> lane & 1) != 0) ? -mag : mag;
    }
    if (real && !stopped)
        flood::st_lane(a.Rnew, frame_offset<T>(static_cast<uint32_t>(e0 + k), a.W, f), r);
}

// Bits, iteration counts and posteriors: a frame's posteriors are those of the
// iteration it stopped at, formed from that iteration's messages.
template <class A>
__global__ __launch_bounds__(256) void k_few_output(const int32_t *__restrict__ col_ptr,
                                                    const int32_t *__restrict__ col_edge,
                                                    const typename A::T *__restrict__ llr, int32_t F, int32_t n,
                                                    int32_t W, const typename A::T *__restrict__ Lch,
                                                    const typename A::T *__restrict__ R0,
                                                    const typename A::T *__restrict__ R1,
                                                    const int32_t *__restrict__ done,
                                                    const int32_t *__restrict__ unsat_last, int32_t max_iter,
                                                    uint8_t *__restrict__ bits, int32_t *__restrict__ iters,
                                                    typename A::T *__restrict__ posterior)
{
    using T = typename A::T;
    const int32_t i = static_cast<int32_t>(blockIdx.x * blockDim.x + threadIdx.x);
    const int32_t f = i % W, c = i / W;
    if (c >= n || f >= F)
        return;
    int32_t it = max_iter;
    if (unsat_last != nullptr) {  // early stop
        const int32_t dn = done[f];
        it = dn >= 0 ? dn : unsat_last[f] == 0 ? max_iter - 1 : max_iter;
    }
    T v = Lch[i];
    if (it > 0)
        v = few_column(v, col_edge + col_ptr[c], col_ptr[c + 1] - col_ptr[c], (it & 1) ? R1 : R0, W, f);
    const int64_t o = static_cast<int64_t>(f) * n + c;
    bits[o] = static_cast<uint8_t>(v < T(0));
    if (posterior)
        posterior[o] = it == 0 ? llr[o] : v * T(A::kOut);
    if (c == 0)
        iters[f] = it;
}

template <class A, int KL, bool MS>
ldpc_status run_few(const ldpc_code_s *c, int32_t frames, int32_t max_iter, bool es, const typename A::T *llr,
                    uint8_t *bits, int32_t *iters, typename A::T *post, typename A::T *R, typename A::T *Lch,
                    int32_t *done, int32_t *unsat, hipStream_t s, typename A::T scale, typename A::T offset)
{
    using T = typename A::T;
    constexpr int32_t FW = few_width(KL);
    const int32_t W = (frames + FW - 1) / FW * FW;
    T *buffer[2] = {R, R + c->E * W};
    const FewInit init = few_init(c->n, W, max_iter, es);
    const dim3 vgrid(init.blocks), ogrid(static_cast<unsigned>((c->n * W + 255) / 256));
    {
        ProfScope ps(LDPC_KERNEL_INGEST, s);
        LDPC_LAUNCH(ps, (k_few_ingest<A>), vgrid, dim3(256), 0, s, llr, frames, c->n, W, Lch, done, unsat,
                    init.unsat_words, init.words);
    }
    FewArgs<A> a{c->row_ptr, c->col_idx, c->col_ptr, c->col_edge, c->m, c->n, W, W / FW, Lch, nullptr, nullptr, done,
                 nullptr, nullptr, 0, scale, offset};
    const dim3 grid(static_cast<unsigned>((static_cast<int64_t>(c->m) * a.groups + 3) / 4));
    for (int32_t t = 1; t <= max_iter; ++t) {
        a.t = t;
        a.Rold = buffer[(t - 1) & 1];
        a.Rnew = buffer[t & 1];
        a.unsat = unsat + static_cast<int64_t>(t - 1) * W;
        a.unsat_prev = t > 1 ? a.unsat - W : nullptr;
        ProfScope ps(LDPC_KERNEL_CHECK, s);
        if (t == 1 && es)
            LDPC_LAUNCH(ps, (k_few<A, KL, true, true, MS>), grid, dim3(256), 0, s, a);
        else if (t == 1)
            LDPC_LAUNCH(ps, (k_few<A, KL, true, false, MS>), grid, dim3(256), 0, s, a);
        else if (es)
            LDPC_LAUNCH(ps, (k_few<A, KL, false, true, MS>), grid, dim3(256), 0, s, a);
        else
            LDPC_LAUNCH(ps, (k_few<A, KL, false, false, MS>), grid, dim3(256), 0, s, a);
    }
    ProfScope ps(LDPC_KERNEL_OUTPUT, s);
    LDPC_LAUNCH(ps, (k_few_output<A>), ogrid, dim3(256), 0, s, c->col_ptr, c->col_edge, llr, frames, c->n, W, Lch,
                buffer[0], buffer[1], done, es && max_iter > 0 ? unsat + static_cast<int64_t>(max_iter - 1) * W : nullptr,
                max_iter, bits, iters, post);
    return hipGetLastError() == hipSuccess ? LDPC_OK : LDPC_EDEVICE;
}

}  // namespace

// The streaming kernels cost the same from 1 to 64 frames; a launch here costs
// in proportion to its wavefronts, m x (frame groups), beyond its latency, and
// more for long rows, whose lanes gather more.  Measured on MI355X, us per call,
// streaming kernels and 1, 2, 3, 4 groups, 20 iterations: n = 16200 of degree 7 FP32
// 335 and 161, 223, 307, -, FP64 600 and 207, 300, 420, 512; n = 64800 FP32 905 and
// 414, 688, FP64 1840 and 550, 928, 1396; n = 12007 of degree 16 FP32 350 and 147, 213,
// -, 338 (four groups: left to the streaming kernels), FP64 730 and 199, 286, -, 450.
// The third group in FP32, 8 iterations, streaming and here, sum-product with early
// stop and min-sum: degree 7, 14000 rows 197 and 196, 199 and 162; 20000 rows 250 and 265,
// - ; degree 9 to 16, 14000 rows 285 and 241, 277 and 220; degree 20 to 32, 6000 rows 297
// and 252, 243 and 238; 9000 rows 406 and 375, 336 and 355; 18000 rows 716 and 778, 630 and
// 749.  The bound on the reads keeps out codes whose dense columns would be summed by
// very many rows (near it: a column of degree 2503, 19.3 and 3.3 to 17.5 ms).
int32_t few_frames_groups(const ldpc_code_s *c, bool f64, int32_t frames)
{
    if (frames > kFewFrames || c->max_row_deg > 32)
        return 0;
    const int32_t width = few_width(c->max_row_deg), groups = (frames + width - 1) / width;
    if (std::max<int64_t>(c->E, c->n) * groups * width >= 1 << 24)  // 24-bit factors, 32-bit byte offsets
        return 0;
    const int32_t third = c->max_row_deg <= 16 ? 14000 : 6000;  // rows up to which FP32 takes three groups
    const int32_t most = f64 ? (c->m <= 20000 ? 4 : 3) : c->m <= third ? 3 : 2;
    return groups <= most && c->column_reads * groups * width <= 1 << 26 ? groups : 0;
}

template <class A>
ldpc_status decode_few(const ldpc_code_s *c, int32_t frames, int32_t max_iter, uint32_t flags,
                       const typename A::T *llr, uint8_t *bits, int32_t *iters, typename A::T *post,
                       typename A::T *R, typename A::T *Lch, int32_t *done, int32_t *unsat, hipStream_t s,
                       typename A::T scale, typename A::T offset)
{
    const bool es = (flags & LDPC_EARLY_STOP) != 0;
    const auto run = [&](auto lanes) {
        constexpr int KL = decltype(lanes)::value;
        if (flags & LDPC_MIN_SUM)
            return run_few<A, KL, true>(c, frames, max_iter, es, llr, bits, iters, post, R, Lch, done, unsat, s, scale,
                                        offset);
        return run_few<A, KL, false>(c, frames, max_iter, es, llr, bits, iters, post, R, Lch, done, unsat, s, scale,
                                     offset);
    };
    if (c->max_row_deg <= 8)
        return run(std::integral_constant<int, 8>());
    if (c->max_row_deg <= 16)
        return run(std::integral_constant<int, 16>());
    return run(std::integral_constant<int, 32>());
}

template ldpc_status decode_few<ArithF32>(const ldpc_code_s *, int32_t, int32_t, uint32_t, const float *, uint8_t *,
                                          int32_t *, float *, float *, float *, int32_t *, int32_t *, hipStream_t,
                                          float, float);
template ldpc_status decode_few<ArithF64>(const ldpc_code_s *, int32_t, int32_t, uint32_t, const double *, uint8_t *,
                                          int32_t *, double *, double *, double *, int32_t *, int32_t *, hipStream_t,
                                          double, double);

}  // namespace ldpc
