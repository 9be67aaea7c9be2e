// Interaction loops: steps e (local-local) and f (local x received boundary
// particles) of Section II, FORCE and GRADIENT passes, FP64 and FP32-split.
//
// Neighbour search (Section I): the 27 buckets around a target are 9 rows of
// up to 3 buckets that are contiguous in hash order (the hash runs
// x-fastest), so each row is one contiguous range of the sorted sources.
//
// Work mapping (k_pairs): a workgroup of four wavefronts takes 64
// consecutive targets (32 or 16 where the call is small), in groups that share
// a bucket row (cy, cz); consecutive sorted targets often do.
//   * Up to four groups are taken together where their windows are short enough:
//     one after the other, each would go through the chain of loads and barriers
//     below for its few targets.  (One by one and together, in us: FORCE of a gas
//     of 30,000 particles at one a bucket FP32 43 and 25, FP64 70 and 33; at 0.05 a
//     bucket 66 and 34, 118 and 52; of a shuffled list of 30,000 particles 222 and
//     158; the step of a lattice of 101,306 FP32 particles 98.7 and 88.3.)
//   * The window of a group is the 9 neighbour rows over the union of its
//     targets' buckets, about 800 sources on a lattice.  The workgroup first
//     reads their positions and culls those that are farther than 2h from the
//     box of its targets (435 remain of a lattice's, 600 of a disordered
//     fluid's), then loads the others once, straight from the particle fields,
//     and keeps the whole records in LDS (in pages when they fill more than one).
//   * Each wavefront takes 16 (8, 4) of the targets.  The candidate test of 16
//     sources against 16 targets is one matrix product (K = 4) on the matrix
//     cores, with the test's bound as its initial value, so the sign of each
//     result is the answer and one instruction per result collects the signs
//     in a bit mask per lane.
//   * The hits of a target go to its list in LDS, and four (8, 16) lanes share
//     the list evenly: only ~1 candidate in 6 is a neighbour, so the cheap test
//     and the pair body (about a hundred operations) are kept apart, and the
//     body runs dense.  (One lane per target would leave the chip idle below
//     some 60,000 particles, and wait for its busiest lane.)
// The lanes' sums are added at the end.  The order of summation depends on
// the number of targets (which sets the lanes per target), on what other targets a
// workgroup has and on all positions (which set what a page holds), so a target
// listed and the same target in a pass over its whole array may differ by
// rounding; calls with the same arrays, counts and list agree bit for bit.  A pair
// with r = 0 (the target itself, or a coincident particle) adds nothing: its
// terms all carry F(0) = 0.
//
// A candidate outside a target's own 27 buckets is farther than one bucket
// side >= 2h on some axis and fails the pair body's distance test, so testing
// the group's whole window changes no neighbour set.
//
// What bounds it: vector-instruction issue.  On the 810,448-particle column
// (FP32) a wavefront issues about 3,600 vector instructions, 2,100 of them in
// the pair body, and the vector units are busy for three quarters of the
// pass.  Hits read from L1 instead of LDS (one lane per target, three to ten
// 16-byte reads per hit that touch a line each) held the vector units back: L1
// lookups took 76 % (FP32) to 100 % (FP64) of such a kernel's cycles.  Culling
// brings the records of a group down to one page or two, so that fewer targets
// wait for the one with the most hits in a page (22 rounds of the body per
// wavefront instead of 26; 20.25 if no lane ever waited).  Measured per pass,
// reads from L1 with their staging kernel first, whole windows in LDS second,
// culled ones third, several rows together fourth: column FORCE FP32 401, 391,
// 350, 330 us, FP64 675, 572, 520, 500; 4.0 M cylinder (FP32) FORCE 2.89, 2.59,
// 2.23, 2.07 ms, GRADIENT 1.62, 1.50, 1.29, 1.27; 6.7 M impact (FP64) FORCE 8.83,
// 6.53, 5.70, 5.58 ms, GRADIENT 4.02, 3.04, 2.71, 2.74; 250,047-particle FORCE
// reverse FP32 260, 248, 228, 207 us; 27,000 ones FP64 FORCE 54, 43, 39, 31 us;
// 8,000 ones FP32 63, 33, 17 and 14 us (the last two with 16 targets per
// workgroup).  Culling and loading in one sweep instead of two was slower (441 us
// for the column's 373): each source's fields then wait for its position.
//
// Where it is slower than one wavefront per 64 targets and records read from L1
// (us, with that kernel's staging second): FP32 FORCE of a uniform gas of some
// 200,000 particles and more, at 0.3 to 4 a bucket, so fewer than 20 neighbours
// each (1 M particles at 0.3, 1 and 4 a bucket 222 and 157, 224 and 149, 256 and
// 199; FP64 295 and 302, 302 and 304, 356 and 368): 64 targets then lie in 16 and
// more buckets, share little of their window, and use few of its records.
//
// In the FP32-split form the position difference is rebuilt from bucket
// indices and float offsets, d = (c_j - c_i) L + (off_j - off_i), which is
// exactly odd under i <-> j and never cancels the way a difference of large
// float positions would; its pair sums accumulate in FP64 (full rate on
// gfx950: a convert and an add per term) and are stored as a float (hi, lo)
// pair.
#include <atomic>
#include <cmath>

#include "pair.hpp"

namespace sph {

namespace {

// Events recorded around every pair-kernel launch when set (sph_set_pair_events).
std::atomic<void *> g_pair_events[2] = {nullptr, nullptr};

constexpr int kPairWaves = 4;                     // wavefronts per workgroup
constexpr int kPairBlock = kPairWaves * kWave;    // threads per workgroup
constexpr uint32_t kCUs = 256;
// Sources in flight per lane while the window is culled (column FP32: 1 364,
// 2 362, 4 368 us).
constexpr int kAhead = 2;
constexpr int kBatch = 1536;                      // window entries culled at a time (a lattice's windows: 800 to 1,450)
constexpr int kEntryBits = 11;                    // of a kept entry's code: its place in the batch, then its row
static_assert(kBatch <= 1 << kEntryBits, "a batch's entries");
constexpr int kPassAdjoint = 2;            // reverse mode of the FORCE pass
constexpr int kPassGradAdjoint = 4;        // reverse mode of the GRADIENT pass

// Census outputs: per target, the number of sources the pass evaluates
// (r^2 < (2h)^2 on the rebuilt d, the pairs at r = 0 included) and the sum,
// modulo 2^64, of mix64 of their ids; sid is the sources' id array.
struct Census {
    uint32_t *count;
    unsigned long long *sum;
    const uint32_t *sid;
};

// SplitMix64 output function (Steele, Lea and Flood, "Fast splittable
// pseudorandom number generators", 2014): a bijection of 64-bit words whose
// sums over two different id sets differ with overwhelming probability.
__device__ inline unsigned long long mix64(uint32_t id)
{
    unsigned long long z = (unsigned long long)id + 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

// A source's record in LDS: its position (FP32 split: offsets and bucket x
// index; FP64: x), the fields that the pass reads, and in the split form the
// (c_j - c_i) L of its row in y and z.  Held in planes of 16 bytes per source,
// the last one of 8 bytes where that is enough, so that a hit costs a few wide
// LDS reads.
template <typename real, int PASS, bool SOLID, int TILE = 16>
struct Pass {
    static constexpr int kGroup = kPairWaves * TILE;   // targets per workgroup
    static constexpr int kShare = kWave / TILE;        // lanes that share a target
    static_assert(TILE <= 16 && kGroup <= kWave, "lane l of every wavefront looks at target l of the workgroup");
    static constexpr bool SPLIT = sizeof(real) == 4;
    static constexpr bool ADJ = PASS == kPassAdjoint, GADJ = PASS == kPassGradAdjoint;
    static constexpr bool FORCE = PASS == SPH_PASS_FORCE, GRAD = PASS == SPH_PASS_GRADIENT;
    static constexpr int NOUT = FORCE ? 6 : (ADJ ? (SOLID ? 17 : 11) : (GADJ ? 7 : 9));
    static constexpr int NPOS = SPLIT ? 4 : 3;
    static constexpr int NF = FORCE ? (SOLID ? 14 : 8) : (ADJ ? (SOLID ? 20 : 14) : (GADJ ? 13 : 4));
    static constexpr int NR = NPOS + NF + (SPLIT ? 2 : 0);   // reals of a record
    static constexpr int C = 16 / (int)sizeof(real);          // reals per 16 bytes
    static constexpr int REST = NR % C;
    static constexpr bool HALF = REST > 0 && 2 * REST <= C;
    static constexpr int NV = NR / C + (REST > 0 && !HALF ? 1 : 0);
    // Wavefronts per SIMD: caps the registers at 512 / that and the LDS of a
    // workgroup at 160 KB / that (LDS is given out in 1,280 bytes).  The most
    // at which little is spilled (ten registers at most, outside the loop over
    // hits): one more is slower by 20 to 80 % (FP32 adjoint 278 -> 502 us), one
    // fewer by 2 to 30 %, as a page holds more but fewer wavefronts hide each
    // other's waits.  Small calls of the solid FORCE pass, whose workgroups are
    // all resident anyway, have one fewer and the larger page (13,824 FP64
    // particles 27.3 us, 29.3 with three).
    static constexpr bool FEW = FORCE && SOLID && TILE < 16;
    static constexpr int waves_f32 = ADJ ? (SOLID ? 2 : 3) : (GADJ || FEW ? 3 : 4);
    static constexpr int waves_f64 = ADJ ? (SOLID ? 1 : 2) : (GADJ || FEW ? 2 : 3);
    static constexpr int waves = SPLIT ? waves_f32 : waves_f64;
    // Records in flight while hits are evaluated: a second one costs registers
    // and is worth them where a page's hits are few instructions apart or where
    // it costs no wavefront (GRADIENT FP32 1,498 us with two, 1,537 with one;
    // fluid FORCE FP32 420 and 397, FP64 598 and 563, FP32 adjoint 277 and 250;
    // solid FORCE 4 M FP32 2,406 with two and three wavefronts per SIMD, 2,225
    // with one and four, 6.7 M FP64 6,160 with two and two, 5,950 with one and
    // three).
    static constexpr bool kTwoAhead = GRAD || GADJ || FEW;
    // Listed hits per target and round: above the 81 (and near misses) of a
    // lattice at h = 1.3 dx, since all may be in one page and a second round
    // lists them by a slower loop (64: column FP64 523 us, 8,000 FP32 particles
    // 32; 96: 515 and 28; 112 leaves less room for the page: 536 and 29.5).
    static constexpr int kCap = 96;
    // A page is laid out as kRows rows of up to kPlaces sources, as many as the
    // LDS has room for (up to 20 rows: a page of 16 held GRADIENT at 1.38 ms for
    // 1.31; with 24 its lists and words cost more than the page gains).  The
    // hit lists take the place of the candidate operands once these have been
    // read, which is worth a barrier: one page holds 432 sources instead of 336
    // (column FP32 352 -> 344 us).  Rows start in different LDS banks (odd
    // pitch), and so do the candidate operands that 16 lanes read together
    // (pitch 4 or 12 modulo 16).
    static constexpr int kBudget = 128 / waves * 1280 - kBatch * 2 - 128;
    static constexpr int kListPitch = kCap + 2;   // (+ 2: the rows start in different banks)
    static constexpr int kListBytes = (kGroup * kListPitch + 6 * kShare) * 2;   // (a lane reads up to six ahead)
    static constexpr int most_of(int a, int b) { return a > b ? a : b; }
    static constexpr int REC = 16 * NV + (HALF ? 8 : 0);
    static constexpr int up4(int places) { return (places + 3) / 4 * 4; }
    static constexpr int pitch_of(int places) { return places | 1; }
    static constexpr int cand_pitch_of(int places) { return up4(places) % 8 ? up4(places) : up4(places) + 4; }
    static constexpr int places_of(int rows)
    {
        int p = 32;   // a row's hits fit one word
        while (p > 0 && rows * pitch_of(p) * REC + most_of(rows * cand_pitch_of(p) * 16, kListBytes) > kBudget) --p;
        return p;
    }
    static constexpr int best_rows()
    {
        int best = 4;
        for (int r = 4; r <= 20; r += 4)
            if (r * places_of(r) > best * places_of(best)) best = r;
        return best;
    }
    static constexpr int kRows = best_rows(), kPlaces = places_of(kRows);
    static constexpr int kPitch = pitch_of(kPlaces), kCandPitch = cand_pitch_of(kPlaces);
    static constexpr int kPage = kRows * kPlaces;
    static constexpr int kShared = most_of(kRows * kCandPitch * 16, kListBytes);
    static_assert(kPage >= 128, "a page");
};

// (2h)^2 predicate on FP64 differences without FMA contraction, identical
// to a left-to-right IEEE evaluation of ((dx dx + dy dy) + dz dz).
__device__ inline double r2_exact(double a, double b, double c)
{
#pragma clang fp contract(off)
    return (a * a + b * b) + c * c;
}

template <typename real>
__device__ inline real r2_of(const real d[3]);
template <>
__device__ inline double r2_of<double>(const double d[3])
{
    return r2_exact(d[0], d[1], d[2]);
}
template <>
__device__ inline float r2_of<float>(const float d[3])
{
    return d[0] * d[0] + d[1] * d[1] + d[2] * d[2];
}

// Orders this wavefront's LDS writes before its following LDS reads.
__device__ inline void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The lanes where b holds (a lane mask as the compare leaves it: __ballot's int
// costs two more vector instructions).
__device__ inline uint64_t ballot(bool b) { return __builtin_amdgcn_ballot_w64(b); }

// a / d, where inv is (1 + 2^-50) / d: the product exceeds a / d by up to
// 2^-17 / d, and a / d is at least 1 / d below the next integer.
__device__ inline uint32_t udiv(uint32_t a, double inv) { return (uint32_t)((double)a * inv); }

// A wave-uniform double held in scalar registers (it is an operand of
// vector instructions, so it takes no vector registers of its own).
__device__ inline double uniform_double(double v)
{
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)b);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(b >> 32));
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// v of the lane that a data-parallel move CTRL names, `own` where it names none.
template <int CTRL, int ROWS = 0xF>
__device__ inline int dpp(int own, int v)
{
    return __builtin_amdgcn_update_dpp(own, v, CTRL, ROWS, 0xF, false);
}

// Largest value over the wavefront of a v in [0, 128), by seven ballots (no
// cross-lane data movement).
__device__ inline int wave_max_u7(int v)
{
    int r = 0;
#pragma unroll
    for (int b = 6; b >= 0; --b) {
        const int c = r | (1 << b);
        if (ballot(v >= c)) r = c;
    }
    return r;
}

// The largest values over the wavefront of four unsigned numbers, in place:
// two exchanges of half wavefronts and one of rows of 16 lanes leave one
// number to a row, whose lanes then fold towards the last.
__device__ inline void wave_max4(uint32_t v[4])
{
    uint32_t m[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const auto s = __builtin_amdgcn_permlane32_swap(v[k], v[k + 2], false, false);
        m[k] = max(s[0], s[1]);   // v[k] in the lower half, v[k + 2] in the upper one
    }
    const auto s = __builtin_amdgcn_permlane16_swap(m[0], m[1], false, false);
    uint32_t a = max(s[0], s[1]);   // rows: v[0], v[1], v[2], v[3]
    a = max(a, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)a, 0x111, 0xF, 0xF, true));
    a = max(a, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)a, 0x112, 0xF, 0xF, true));
    a = max(a, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)a, 0x114, 0xF, 0xF, true));
    a = max(a, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)a, 0x118, 0xF, 0xF, true));
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = __builtin_amdgcn_readlane(a, 16 * k + 15);
}

// Floats as unsigned integers of the same order, and back.
__device__ inline uint32_t ordered(float v)
{
    const uint32_t b = __builtin_bit_cast(uint32_t, v);
    return b ^ ((uint32_t)((int)b >> 31) | 0x80000000u);
}
__device__ inline float unordered(uint32_t u)
{
    return __builtin_bit_cast(float, u ^ (~(uint32_t)((int)u >> 31) | 0x80000000u));
}

// v of another lane of the row of 16, as the data-parallel move CTRL names it.
template <int CTRL>
__device__ inline double lane_other(double v)
{
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, CTRL, 0xF, 0xF, true);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), CTRL, 0xF, 0xF, true);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
// The sum of v over the N lanes N k .. N k + N - 1, in each of them.
template <int N>
__device__ inline double share_sum(double v)
{
    v += lane_other<0xB1>(v);   // lanes 1 0 3 2
    v += lane_other<0x4E>(v);   // lanes 2 3 0 1
    if constexpr (N > 4) v += lane_other<0x141>(v);   // lanes 7 .. 0 of 8: the other four
    if constexpr (N > 8) v += lane_other<0x140>(v);   // lanes 15 .. 0 of 16: the other eight
    return v;
}

// Target position: bucket offsets and bucket x index (split), or x (FP64).
template <typename real>
struct TargetPos {
    real o[3];
    double x[3];
    real cxf;
    real Lf;
};

// Pair-sum accumulator: FP64 in both forms.
struct Acc {
    double s;
    __device__ inline void add(float x) { s += (double)x; }
    __device__ inline void add(double x) { s += x; }
};

typedef float f32x4 __attribute__((ext_vector_type(4)));
template <typename real>
struct Chunk;
template <>
struct Chunk<float> {
    using full = float __attribute__((ext_vector_type(4)));
    using half = float __attribute__((ext_vector_type(2)));
};
template <>
struct Chunk<double> {
    using full = double __attribute__((ext_vector_type(2)));
    using half = double __attribute__((ext_vector_type(1)));
};

// Constants of a pass, made on the host so that they are scalar operands.
template <typename real>
struct PairArgs {
    PairK<real> K;
    real R2;    // (2h)^2
    float h2;   // 2h
};

// Arguments of a call.
template <typename real>
struct PairCall {
    PairArgs<real> A;
    Grid g;
    PV<real> tg;
    const uint32_t *tidx, *ntdev;
    PV<real> src;
    const uint32_t *sstart;
    double nx_inv, ny_inv;   // for udiv by the grid's nx and ny
    real Linv;               // 1 / L, no number where L is not between 2^-60 and 2^45
    int zero_first;
    RV<real> R, Rsrc;
    AV<real> B;
    Census cz;
};
template <typename real>
using CallArgs = const __attribute__((address_space(4))) PairCall<real> *;

// The kernel's arguments, read again where they are used.  Some 40 pointers and
// constants that stay in scalar registers from one use to the next push the loops'
// own scalars out into vector registers (50 to 120 of them, and up to 23 vector
// registers out into scratch, against 0 to 16 and up to 10: column FORCE FP32 356
// and 339 us, a share's sort and two passes 1,393 and 1,305).
template <typename real>
__device__ inline CallArgs<real> call_args()
{
    auto a = (CallArgs<real>)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(a));
    return a;
}

// Entry j of a field, by a 32-bit byte offset from its base (sources are fewer
// than 2^27), so that the loads of all fields share one address register.
template <typename T>
__device__ inline T field(const T *base, uint32_t j)
{
    using Byte = const __attribute__((address_space(1))) char *;
    using Entry = const __attribute__((address_space(1))) T *;
    return *(Entry)((Byte)base + j * (uint32_t)sizeof(T));
}

// Entry j of a field of any length, through a pointer read by call_args (of
// which the compiler would not know that it points to global memory).
template <typename T>
__device__ inline __attribute__((address_space(1))) T &entry(T *base, uint32_t j)
{
    return ((__attribute__((address_space(1))) T *)base)[j];
}

// The fields of source j that a pass reads, in record order.
template <typename real, int PASS, bool SOLID, bool CENSUS>
__device__ inline void load_fields(CallArgs<real> a, uint32_t j, real *f)
{
    using W = Pass<real, PASS, SOLID>;
    if constexpr (CENSUS) {   // the id in place of the first
#pragma unroll
        for (int k = 1; k < W::NF; ++k) f[k] = real(0);
        if constexpr (W::SPLIT)
            f[0] = __builtin_bit_cast(float, field(a->cz.sid, j));
        else
            f[0] = __builtin_bit_cast(double, (uint64_t)field(a->cz.sid, j));
    } else {
#pragma unroll
        for (int d = 0; d < 3; ++d) f[d] = field(a->src.v[d], j);
        f[3] = field(a->src.w, j);
        if constexpr (W::FORCE || W::ADJ) {
            f[4] = field(a->src.rho, j);
            f[5] = field(a->src.p, j);
            f[6] = field(a->src.c, j);
            f[7] = field(a->src.e, j);
            if constexpr (SOLID) {
#pragma unroll
                for (int k = 0; k < 6; ++k) f[8 + k] = field(a->src.S[k], j);
            }
        }
        // cotangents of the sources' rates or velocity gradients (none: zero)
        if constexpr (W::ADJ) {
#pragma unroll
            for (int k = 0; k < 6; ++k) f[(SOLID ? 14 : 8) + k] = a->Rsrc.hi[0] ? field(a->Rsrc.hi[k], j) : real(0);
        }
        if constexpr (W::GADJ) {
#pragma unroll
            for (int k = 0; k < 9; ++k) f[4 + k] = a->Rsrc.Lhi[0] ? field(a->Rsrc.Lhi[k], j) : real(0);
        }
    }
}

// (CENSUS: the pass's neighbour sets instead of its sums, by the same pages,
// lists and launches.)
template <typename real, int PASS, bool SOLID, int TILE, bool CENSUS>
__global__ __launch_bounds__(kPairBlock)
__attribute__((amdgpu_waves_per_eu(Pass<real, PASS, SOLID, TILE>::waves)))
void k_pairs(PairCall<real> call)
{
    using W = Pass<real, PASS, SOLID, TILE>;
    constexpr bool SPLIT = W::SPLIT, ADJ = W::ADJ, GADJ = W::GADJ, FORCE = W::FORCE;
    constexpr int NOUT = W::NOUT, kPage = W::kPage, kCap = W::kCap, C = W::C;
    constexpr int kGroup = W::kGroup, kShare = W::kShare;
    constexpr int kRows = W::kRows, kPitch = W::kPitch, kCandPitch = W::kCandPitch;
    constexpr int kWords = kRows / 4;   // bit-mask words of a lane per page
    using full = typename Chunk<real>::full;
    using half = typename Chunk<real>::half;
    __shared__ full plane[W::NV][kRows * kPitch];
    __shared__ half plane_h[W::HALF ? kRows * kPitch : 1];
    // the candidate operands (q, |q|^2) of the page's sources, then the hit
    // lists, at the end the targets' sums
    __shared__ alignas(16) unsigned char shared[W::kShared];
    f32x4 *const cand = reinterpret_cast<f32x4 *>(shared);
    uint16_t *const list = reinterpret_cast<uint16_t *>(shared);
    __shared__ uint16_t kept_of[kBatch];      // the window's entries near the group, a segment per wavefront
    __shared__ uint32_t kept_n[kPairWaves];   // and how many each holds, and of how many looked at
    __shared__ double corner_of[SPLIT ? 1 : kPairWaves][3];   // the frames of groups taken together (FP64 form)
    constexpr int kListPitch = W::kListPitch;

    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave0 = __builtin_amdgcn_readfirstlane(tid / kWave);
    const PV<real> &tg = call.tg;
    const uint32_t *const tidx = call.tidx;
    const bool listed = tidx != nullptr;
    uint32_t nt = tg.n, tile;
    if (listed) {
        // a target list's count is on the device and the grid is sized for the
        // whole array: the list's tiles shared evenly by the XCDs
        const uint32_t c = *call.ntdev;
        nt = c < nt ? c : nt;
        if (!xcd_tile_active(blockIdx.x, (nt + kGroup - 1) / kGroup, tile)) return;
    } else {
        tile = xcd_tile(blockIdx.x, gridDim.x);   // neighbouring tiles share sources
    }
    // lane l of every wavefront looks at target l of the workgroup
    const uint32_t t = tile * (uint32_t)kGroup + (uint32_t)lane;
    uint32_t ti = lane < kGroup && t < nt ? (listed ? tidx[t] : t) : tg.n;
    const bool tvalid = ti < tg.n;   // a listed index outside the target array names no target
    ti = tvalid ? ti : 0u;
    const uint32_t th = tg.hash[ti];
    uint32_t trow = udiv(th, call.nx_inv);   // cy + ny cz
    const int tcx = (int)(th - trow * (uint32_t)call.g.nx);
    trow = tvalid ? trow : ~0u;   // no target's row: there are fewer buckets than 2^32 - 1
    // the lane's target in the candidate test, and the one whose pairs it evaluates
    // (of a test's 16 columns, the first TILE hold targets)
    const int lf = wave0 * TILE + (lane & (TILE - 1)), le = wave0 * TILE + lane / kShare;
    const int sub = lane & (kShare - 1);
    const uint32_t i = __shfl(ti, le, kWave);
    const int ecx = __shfl(tcx, le, kWave);
    uint64_t pending = ballot(tvalid);
    const bool valid = (pending >> le) & 1ull;

    PairK<real> K;
    real R2;

    // The position of the lane's target for the culling is kept in the FP32 fluid FORCE
    // pass and read again in each round in the others, which are short of its three
    // registers (FP64: six): 4 M cylinder GRADIENT FP32 1,310 us kept and 1,268 read
    // again, 6.7 M impact FORCE FP32 3,490 and 3,420, FP64 5,690 and 5,580,
    // 250,047-particle FORCE reverse FP32 215 and 207, but column step FP32 382 and 384.
    constexpr bool KEPT = SPLIT && FORCE && !SOLID;
    real tpos[3];
    TargetPos<real> T;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        if constexpr (KEPT) tpos[d] = tg.off[d][ti];
        if constexpr (SPLIT) {
            T.o[d] = tg.off[d][i];
            T.x[d] = 0.0;
        } else {
            T.x[d] = tg.x[d][i];
            T.o[d] = real(0);
        }
    }
    // Listed targets need not ascend; where they do, a group's outer buckets are
    // those of its first and last target.  (All lanes' hashes are looked at, those of
    // indices outside the array too: no descent can hide behind one.)
    const uint32_t before = __shfl_up(th, 1, kWave);
    const bool ascend = !ballot(lane > 0 && lane < kGroup && t < nt && th < before);
    Part<real, SOLID> I;
    real rbi[GADJ ? 9 : 6];   // adjoint: the target's rate (or velocity-gradient) cotangents
    if constexpr (CENSUS) {
    } else if constexpr (FORCE || ADJ) {
        load_part<real, SOLID>(tg, i, I);
    } else {
#pragma unroll
        for (int d = 0; d < 3; ++d) I.v[d] = tg.v[d][i];
        if constexpr (GADJ) I.w = tg.w[i];
    }
    if constexpr (ADJ) {
#pragma unroll
        for (int k = 0; k < 6; ++k) rbi[k] = call.R.hi[0] ? call.R.hi[k][i] : real(0);
    }
    if constexpr (GADJ) {
#pragma unroll
        for (int k = 0; k < 9; ++k) rbi[k] = call.R.Lhi[0] ? call.R.Lhi[k][i] : real(0);
    }

    Acc acc[NOUT];
#pragma unroll
    for (int k = 0; k < NOUT; ++k) acc[k].s = 0.0;
    uint32_t ncen = 0;             // census: pairs evaluated
    unsigned long long scen = 0;   // census: sum of mix64 of their ids

    // the pair terms of one hit, whose record is q, added to the lane's sums
    auto eval = [&](const real *q) {
        const real *f = q + W::NPOS;
        real d[3];
        if constexpr (SPLIT) {
            d[0] = (q[3] - T.cxf) * T.Lf + (q[0] - T.o[0]);
            d[1] = q[W::NR - 2] + (q[1] - T.o[1]);
            d[2] = q[W::NR - 1] + (q[2] - T.o[2]);
        } else {
#pragma unroll
            for (int a = 0; a < 3; ++a) d[a] = q[a] - T.x[a];
        }
        const real r2 = r2_of<real>(d);
        // the neighbour predicate, on the exact and odd d (so a pair is in or
        // out for both of its particles); the candidate test's bound is wider
        if (!(r2 < R2)) return;   // outside the support: nothing to add
        if constexpr (CENSUS) {
            uint32_t id;
            if constexpr (SPLIT)
                id = __builtin_bit_cast(uint32_t, f[0]);
            else
                id = (uint32_t)__builtin_bit_cast(uint64_t, f[0]);
            ++ncen;
            scen += mix64(id);
        } else if constexpr (FORCE || ADJ) {
            Part<real, SOLID> J;
#pragma unroll
            for (int a = 0; a < 3; ++a) J.v[a] = f[a];
            J.w = f[3];
            J.rho = f[4];
            J.p = f[5];
            J.c = f[6];
            J.e = f[7];
            if constexpr (SOLID) {
#pragma unroll
                for (int a = 0; a < 6; ++a) J.S[a] = f[8 + a];
            }
            if constexpr (FORCE) {
                real o[6];
                pair_force<real, SOLID>(d, r2, I, J, K, o);
#pragma unroll
                for (int k = 0; k < 6; ++k) acc[k].add(o[k]);
            } else {
                // T(s_j, s_i) = sigma T(s_i, s_j): mass, momentum and energy terms
                // are odd (sigma = -1), the volume term even (+1)
                const real *rbj = f + (SOLID ? 14 : 8);
                real wb[6];
#pragma unroll
                for (int k = 0; k < 5; ++k) wb[k] = rbi[k] - rbj[k];
                wb[5] = rbi[5] + rbj[5];
                real o[NOUT];
#pragma unroll
                for (int k = 0; k < NOUT; ++k) o[k] = real(0);
                pair_force_vjp<real, SOLID>(d, r2, I, J, K, wb, o);
#pragma unroll
                for (int k = 0; k < NOUT; ++k) acc[k].add(o[k]);
            }
        } else if constexpr (GADJ) {
            real o[7] = {0, 0, 0, 0, 0, 0, 0};
            pair_grad_vjp<real>(d, r2, I.v, f, I.w, f[3], rbi, f + 4, K, o);
#pragma unroll
            for (int k = 0; k < 7; ++k) acc[k].add(o[k]);
        } else {
            real o[9];
            pair_grad<real>(d, r2, I.v, f, f[3], K, o);
#pragma unroll
            for (int k = 0; k < 9; ++k) acc[k].add(o[k]);
        }
    };
    // the record of the page's source in slot `k`
    auto fetch = [&](uint32_t k, real *q) {
#pragma unroll
        for (int c = 0; c < W::NV; ++c) {
            const full v = plane[c][k];
#pragma unroll
            for (int a = 0; a < C; ++a) q[c * C + a] = v[a];
        }
        if constexpr (W::HALF) {
            const half v = plane_h[k];
#pragma unroll
            for (int a = 0; a < C / 2; ++a) q[W::NV * C + a] = v[a];
        }
    };
    constexpr int kRec = W::NV * C + (W::HALF ? C / 2 : 0);
    const float kFar = __builtin_inff();   // of no source, and of no target: above any bound, in any unit of length

    while (pending) {
        // (What depends on these alone is made anew in each round, not kept.)
        int quarter = lane / 16, wave = wave0;
        asm volatile("" : "+v"(quarter));
        asm volatile("" : "+s"(wave));
        const CallArgs<real> at_round = call_args<real>();
        const auto &g = at_round->g;
        T.Lf = SPLIT ? (real)g.Lf : real(0);
        if constexpr (!KEPT) {
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                if constexpr (SPLIT)
                    tpos[d] = entry(at_round->tg.off[d], ti);
                else
                    tpos[d] = entry(at_round->tg.x[d], ti);
            }
        }
        // The next groups, of targets that share a bucket row: the first pending
        // target's and up to three more.  Lanes 16 k .. 16 k + 15 keep what
        // concerns group k: its row, the bucket its frame starts at, its buckets.
        uint64_t in64[kPairWaves];
        uint32_t ng = 0, wkey = 0;
        int wcx = 0, wx1 = 0;
        uint64_t rest = pending;
#pragma unroll
        for (int k = 0; k < kPairWaves; ++k) {
            in64[k] = 0;
            if (rest) {
                const int first = __ffsll((unsigned long long)rest) - 1;
                const uint32_t key = __builtin_amdgcn_readlane(trow, first);
                in64[k] = ballot(trow == key);
                rest &= ~in64[k];
                const int c0 = __builtin_amdgcn_readlane(tcx, first);
                const int c1 = __builtin_amdgcn_readlane(tcx, 63 - __clzll((long long)in64[k]));
                wkey = quarter == k ? key : wkey;
                wcx = quarter == k ? c0 : wcx;
                wx1 = quarter == k ? c1 : wx1;
                ng = (uint32_t)k + 1u;
            }
        }
        int wx0 = wcx;
        if (!ascend) {
            uint32_t most[kPairWaves], least[kPairWaves];
#pragma unroll
            for (int k = 0; k < kPairWaves; ++k) {
                const bool in = (in64[k] >> lane) & 1ull;
                most[k] = in ? (uint32_t)tcx : 0u;
                least[k] = in ? ~(uint32_t)tcx : 0u;
            }
            wave_max4(most);
            wave_max4(least);
#pragma unroll
            for (int k = 0; k < kPairWaves; ++k) {
                wx0 = quarter == k ? (int)~least[k] : wx0;
                wx1 = quarter == k ? (int)most[k] : wx1;
            }
        }
        if (ng > 1) {
            // Frames that lie apart along x, so that no source of one group passes the
            // candidate test of another's target: its d would be meaningless.  The groups
            // are taken together only if their targets are at most half a bucket outside
            // their own buckets; what culling keeps is at most 2h beyond those, but for
            // the margins, 2^-16 of the square of the frames' length T (1.2 sum W + 50
            // buckets, W their widths) and in FP64 less than T / 64 squared buckets.  The
            // gap of 8 + sum W / 32 buckets leaves room for these and for the test's.
            uint32_t w[kPairWaves], sum = 0, from = 0;
#pragma unroll
            for (int k = 0; k < kPairWaves; ++k) {
                w[k] = (uint32_t)__builtin_amdgcn_readlane(wx1 - wx0, 16 * k) + 1u;
                sum += (uint32_t)k < ng ? w[k] : 0u;
            }
#pragma unroll
            for (int k = 0; k < kPairWaves; ++k) {
                wcx = quarter == k ? wx0 - (int)from : wcx;
                from += w[k] + 8u + sum / 32u;
            }
            if (sum > 4096u) ng = 1;   // (squares of the frame's lengths stay finite)
        }
        // Their windows: lane 16 k + r, r < 9, keeps row r of group k's, which holds
        // entries [off, off + n) of it; entry u is source u + del
        const int wgz = (int)udiv(wkey, at_round->ny_inv), wgy = (int)(wkey - (uint32_t)wgz * (uint32_t)g.ny);
        const int wr = lane & 15, wrz = (wr * 11) >> 5;
        uint32_t wub = 0, wn = 0;
        {
            const int xa = wx0 > 0 ? wx0 - 1 : 0, xb = wx1 + 1 < g.nx ? wx1 + 1 : g.nx - 1;
            const int z = wgz + wrz - 1, y = wgy + (wr - 3 * wrz) - 1;
            if (wr < 9 && (uint32_t)quarter < ng && z >= 0 && z < g.nz && y >= 0 && y < g.ny) {
                const uint32_t row = (uint32_t)g.nx * ((uint32_t)y + (uint32_t)g.ny * (uint32_t)z);
                wub = entry(at_round->sstart, row + (uint32_t)xa);
                wn = entry(at_round->sstart, row + (uint32_t)xb + 1u) - wub;
            }
        }
        uint32_t woff = wn;   // sums over rows 0 .. r of the window
        woff += (uint32_t)dpp<0x111>(0, (int)woff);
        woff += (uint32_t)dpp<0x112>(0, (int)woff);
        woff += (uint32_t)dpp<0x114>(0, (int)woff);
        woff += (uint32_t)dpp<0x118>(0, (int)woff);
        uint32_t tot[kPairWaves];
#pragma unroll
        for (int k = 0; k < kPairWaves; ++k) tot[k] = __builtin_amdgcn_readlane(woff, 16 * k + 8);
        woff -= wn;
        const uint32_t wdel = wub - woff;
        // hash of bucket wcx of the lane's row of the window
        const uint32_t rhash = wkey * (uint32_t)g.nx + (uint32_t)wcx +
                               (uint32_t)g.nx * ((uint32_t)(wr - 3 * wrz - 1) + (uint32_t)g.ny * (uint32_t)(wrz - 1));
        // Groups whose windows fit one batch are taken together; otherwise the
        // first alone.  The wavefronts that cull a group's window: two for the
        // largest of three, or those of two that share the work best; gm holds
        // each wavefront's group, two bits of it.
        uint32_t all = tot[0], gm = 0;
        uint64_t act = in64[0];
        if (ng > 1) {
            // With targets that are outside their buckets (beyond the grid, whose
            // outer buckets hold what is), or a grid too far from the origin, or a bucket
            // side near the ends of the floats' range (Linv is no number), one alone.
            bool astray = false;
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                if constexpr (SPLIT) {
                    const float q = tpos[d] * at_round->Linv;
                    astray = astray || !(q > -0.5f && q < 1.5f);
                } else {
                    const uint32_t y = udiv(trow, at_round->ny_inv);
                    const uint32_t c = d == 0 ? (uint32_t)tcx : (d == 1 ? trow - y * (uint32_t)g.ny : y);
                    const double o = g.o[d] + (double)c * g.L, q = (tpos[d] - o) * at_round->Linv;
                    astray = astray || !(q > -0.5 && q < 1.5 && fabs(o) * at_round->Linv < 0x1p38);
                }
            }
            uint32_t taken = 1;
            bool fit = !ballot(tvalid && astray);
#pragma unroll
            for (int k = 1; k < kPairWaves; ++k) {
                fit = fit && (uint32_t)k < ng && all + tot[k] <= (uint32_t)kBatch;
                if (fit) {
                    all += tot[k];
                    act |= in64[k];
                    ++taken;
                }
            }
            if (taken == 4)
                gm = 0xE4;   // 3 2 1 0
            else if (taken == 3)
                gm = tot[0] >= max(tot[1], tot[2]) ? 0x90 : (tot[1] >= tot[2] ? 0x94 : 0xA4);   // 2 1 0 0, 2 1 1 0, 2 2 1 0
            else if (taken == 2)
                gm = tot[0] > 2 * tot[1] ? 0x40 : (tot[1] > 2 * tot[0] ? 0x54 : 0x50);   // 1 0 0 0, 1 1 1 0, 1 1 0 0
        }
        const bool multi = gm != 0;
        pending &= ~act;
        // This wavefront's group, how many share it and which of them it is, the
        // entries of its window, and the place of the first in the batch
        int gs = 0;
        uint32_t nw = kPairWaves, iw = (uint32_t)wave, total = tot[0], place0 = 0;
        uint64_t ins = in64[0];
        if (multi) {
            gs = (int)(gm >> (2 * wave)) & 3;
            nw = iw = 0;
#pragma unroll
            for (int k = 0; k < kPairWaves; ++k) {
                const bool same = (int)(gm >> (2 * k) & 3u) == gs;
                nw += same ? 1u : 0u;
                iw += same && k < wave ? 1u : 0u;
                place0 += k < gs ? tot[k] : 0u;
                total = k == gs ? tot[k] : total;
                ins = k == gs ? in64[k] : ins;
            }
        }
        const bool tin = (ins >> lane) & 1ull;
        const int lcx = __builtin_amdgcn_readlane(wcx, 16 * gs);   // origin of the group's frame along x
        const int gy = __builtin_amdgcn_readlane(wgy, 16 * gs), gz = __builtin_amdgcn_readlane(wgz, 16 * gs);
        const bool fin = (lane & 15) < TILE && (act >> lf) & 1ull;
        const uint32_t in_tile = (uint32_t)(act >> (wave * TILE)) & ((1u << TILE) - 1u);
        int og = 0, ocx = lcx;   // the group of the lane's target, and its frame's origin along x
        if (multi) {
#pragma unroll
            for (int k = 1; k < kPairWaves; ++k) og = (in64[k] >> lane) & 1ull ? k : og;
            ocx = __shfl(wcx, 16 * og, kWave);
            T.cxf = (real)(ecx - __shfl(ocx, le, kWave));
        } else {
            T.cxf = (real)(ecx - lcx);
        }
        // Frame of the candidate test, in FP32 in both forms: positions relative
        // to the corner of bucket (lcx, gy, gz); split form ((c - lcx) L + off)
        // in x and (dy L + off) in y, z; FP64 form (x - corner) in FP64, rounded
        // once to float.  The test is the expanded form
        // |q|^2 - 2 q.f < R2 - |f|^2.  For a candidate within 2h of the target
        // (|q| <= |f| + 2h) its rounding, with that of the frame, stays below
        // 2^-18 (|f| + 2h)^2; the bound is widened by four times that, and in
        // FP64 also by 2^-46 X (|f| + 2h) with X = |corner|_1 + |f| + 2h, over
        // ten times the rounding of the FP64 differences.  So the listed
        // candidates hold every neighbour.  The pair body applies the neighbour
        // predicate itself, on the exact, odd d.
        uint32_t ext[8];
        float lo[3], hi[3], fo[3];   // the box of the group's targets, and the lane's target of the test
        double corner[3] = {0.0, 0.0, 0.0}, ocorner[3] = {0.0, 0.0, 0.0};   // of the group, of the lane's target's group
        if constexpr (!SPLIT) {
            corner[0] = uniform_double(g.o[0] + (double)lcx * g.L);
            corner[1] = uniform_double(g.o[1] + (double)gy * g.L);
            corner[2] = uniform_double(g.o[2] + (double)gz * g.L);
#pragma unroll
            for (int d = 0; d < 3; ++d) ocorner[d] = corner[d];
            if (multi) {
                ocorner[0] = g.o[0] + (double)ocx * g.L;
                ocorner[1] = g.o[1] + (double)__shfl(wgy, 16 * og, kWave) * g.L;
                ocorner[2] = g.o[2] + (double)__shfl(wgz, 16 * og, kWave) * g.L;
                if (lane < 3) corner_of[gs][lane] = lane == 0 ? corner[0] : (lane == 1 ? corner[1] : corner[2]);
            }
        }
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            float at;
            if constexpr (SPLIT)
                at = d == 0 ? (real)(tcx - ocx) * T.Lf + tpos[d] : tpos[d];
            else
                at = (float)(tpos[d] - ocorner[d]);
            const uint32_t o = ordered(at);
            ext[2 * d] = tin ? o : 0u;
            ext[2 * d + 1] = tin ? ~o : 0u;
            fo[d] = __shfl(at, lf, kWave);
        }
        ext[6] = ext[7] = 0u;
        wave_max4(ext);
        wave_max4(ext + 4);
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            hi[d] = unordered(ext[2 * d]);
            lo[d] = unordered(~ext[2 * d + 1]);
        }
        const float f2 = fo[0] * fo[0] + fo[1] * fo[1] + fo[2] * fo[2];
        const float fl = __builtin_amdgcn_sqrtf(f2) + at_round->A.h2;
        float margin = 0x1p-16f * fl * fl;
        if constexpr (!SPLIT) {
            float X = (float)(fabs(ocorner[0]) + fabs(ocorner[1]) + fabs(ocorner[2]));
            if (multi) X = __shfl(X, lf, kWave);
            X += fl;
            margin += 0x1p-46f * X * fl;
        }
        // Sources within 2h of a target lie within 2h of the targets' box, up to
        // the same rounding (a NaN keeps every source).
        float b2 = 0.0f;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            const float m = fmaxf(fabsf(lo[d]), fabsf(hi[d]));
            b2 += m * m;
        }
        const float bl = __builtin_amdgcn_sqrtf(b2) + at_round->A.h2;
        float bmargin = 0x1p-16f * bl * bl;
        if constexpr (!SPLIT) {
            const float X = (float)(fabs(corner[0]) + fabs(corner[1]) + fabs(corner[2])) + bl;
            bmargin += 0x1p-46f * X * bl;
        }
        R2 = at_round->A.R2;
        const float bbound = (float)R2 + bmargin;
        // the product starts at minus the bound: its sign bit is the answer
        const float c0 = fin ? -(((float)R2 - f2) + margin) : kFar;
        const f32x4 cinit = {c0, c0, c0, c0};
        // operand B: component lane / 16 of (-2 f, 1) of target lane % 16
        const float bop = quarter == 3 ? 1.0f : -2.0f * (quarter == 0 ? fo[0] : (quarter == 1 ? fo[1] : fo[2]));

        // a source's position in the frame of the candidate test
        auto framed = [&](const real *q, real dcx, real ddy, real ddz, const double *corner) {
            f32x4 a;
            if constexpr (SPLIT) {
                a.x = dcx * T.Lf + q[0];
                a.y = ddy + q[1];
                a.z = ddz + q[2];
            } else {
                a.x = (float)(q[0] - corner[0]);
                a.y = (float)(q[1] - corner[1]);
                a.z = (float)(q[2] - corner[2]);
            }
            return a;
        };
        uint32_t off[9];   // of the rows, in scalar registers
#pragma unroll
        for (int r = 1; r < 9; ++r) off[r] = __builtin_amdgcn_readlane(woff, 16 * gs + r);
        for (uint32_t batch = 0; batch < all; batch += kBatch) {
            // The batch's sources that are near no target are culled before their
            // records are read.  Each wavefront looks at its share of its group's
            // entries, whole pieces of 64 of them, several pieces in flight, and
            // lists what it keeps.
            const CallArgs<real> at_cull = call_args<real>();
            const uint32_t here = min(total - batch, (uint32_t)kBatch);
            const uint32_t piece = ((nw == 4 ? (here + 3) / 4 : (nw == 3 ? (here + 2) / 3 : (nw == 2 ? (here + 1) / 2 : here))) +
                                    (kWave - 1)) & ~(uint32_t)(kWave - 1);
            const uint32_t from = min(iw * piece, here), len = min(piece, here - from);
            const uint32_t seg = place0 + from, bend = batch + from + len;
            uint32_t n = 0;
            for (uint32_t w0 = batch + from; w0 < bend; w0 += kAhead * kWave) {
                real q[kAhead][3];
                uint32_t row[kAhead], hs[kAhead];
#pragma unroll
                for (int a = 0; a < kAhead; ++a) {
                    const uint32_t u = min(w0 + (uint32_t)(a * kWave + lane), bend - 1);
                    int r = 0;
#pragma unroll
                    for (int k = 1; k < 9; ++k) r += u >= off[k] ? 1 : 0;
                    const uint32_t j = u + __shfl(wdel, 16 * gs + r, kWave);
                    row[a] = r;
#pragma unroll
                    for (int d = 0; d < 3; ++d) q[a][d] = SPLIT ? field(at_cull->src.off[d], j) : (real)field(at_cull->src.x[d], j);
                    if constexpr (SPLIT) hs[a] = field(at_cull->src.hash, j);
                }
#pragma unroll
                for (int a = 0; a < kAhead; ++a) {
                    if (a && w0 + a * kWave >= bend) break;
                    real dcx = 0, ddy = 0, ddz = 0;
                    if constexpr (SPLIT) {
                        dcx = (real)(int)(hs[a] - __shfl(rhash, 16 * gs + (int)row[a], kWave));
                        const int z = (int)(row[a] * 11) >> 5;
                        ddy = (real)((int)row[a] - 3 * z - 1) * T.Lf;
                        ddz = (real)(z - 1) * T.Lf;
                    }
                    const f32x4 at = framed(q[a], dcx, ddy, ddz, corner);
                    // distances from the box along each axis
                    const float ex = fmaxf(fmaxf(lo[0] - at.x, at.x - hi[0]), 0.0f);
                    const float ey = fmaxf(fmaxf(lo[1] - at.y, at.y - hi[1]), 0.0f);
                    const float ez = fmaxf(fmaxf(lo[2] - at.z, at.z - hi[2]), 0.0f);
                    const uint32_t u = w0 + (uint32_t)(a * kWave + lane);
                    const bool keep = u < bend && !(ex * ex + ey * ey + ez * ez > bbound);
                    const uint64_t mask = ballot(keep);
                    const uint32_t rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                                                    __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
                    if (keep) kept_of[seg + n + rank] = (uint16_t)(row[a] << kEntryBits | (u - batch));
                    n += (uint32_t)__popcll(mask);
                }
            }
            if (lane == 0) kept_n[wave] = n | len << 16;
            __syncthreads();   // the kept entries are listed, and every read of the page before is done
            uint32_t kept = 0, seg0[kPairWaves], jump[kPairWaves];
#pragma unroll
            for (int w = 0; w < kPairWaves; ++w) {
                const uint32_t c = __builtin_amdgcn_readfirstlane(kept_n[w]), n = c & 0xFFFFu;
                seg0[w] = kept;
                kept += n;
                jump[w] = (c >> 16) - n;   // from the end of the segment to the next one
            }
            // page p takes the kept entries p, p + npages, ..., so that every page
            // holds an even share of each target's hits
            const uint32_t npages = (kept + kPage - 1) / kPage;
            if (npages == 0) __syncthreads();   // every read of kept_n is done
            for (uint32_t page = 0; page < npages; ++page) {
                const uint32_t len = (kept - page + npages - 1) / npages;
                const uint32_t blocks = (len + 4 * kRows - 1) / (4 * kRows);   // of four places of every row
                if (page) __syncthreads();   // every read of the page before is done
                // Entry u of the page goes to place u / kRows of row u % kRows: a row,
                // which one lane's word of hit bits covers, samples the page
                // evenly, so that the words of a target hold similar numbers of hits.
                // One source per thread at a time (two or three in flight cost
                // spills: impact FORCE 6.5 -> 8.9 ms, FP32 adjoint 278 -> 366 us).
                // Blocks need not end where 64 lanes do: what lies past the last
                // one has no place.
                const uint32_t ends = blocks * (4 * kRows);
                const CallArgs<real> at_load = call_args<real>();
#pragma unroll 1
                for (uint32_t w0 = (uint32_t)(wave * kWave); w0 < ends; w0 += kPairBlock) {
                    const uint32_t u = w0 + (uint32_t)lane;
                    const uint32_t v = min(u, len - 1) * npages + page;   // of the kept entries
                    uint32_t at = v, sv = 0;   // its place, and its segment
#pragma unroll
                    for (int w = 1; w < kPairWaves; ++w) {
                        at += v >= seg0[w] ? jump[w - 1] : 0u;
                        sv += v >= seg0[w] ? 1u : 0u;
                    }
                    const uint32_t code = kept_of[at];
                    const uint32_t gv = gm >> (2 * sv) & 3u;   // its group
                    const int r = (int)(code >> kEntryBits), wl = (int)gv * 16 + r;
                    const uint32_t j = batch + (code & ((1u << kEntryBits) - 1u)) + __shfl(wdel, wl, kWave);
                    const uint32_t hr = SPLIT ? __shfl(rhash, wl, kWave) : 0u;
                    const uint32_t place = u / (uint32_t)kRows, row = u % (uint32_t)kRows;
                    f32x4 a = {0.0f, 0.0f, 0.0f, kFar};   // past the page's end: no target takes it
                    if (u < len) {
                        real q[W::NR];
                        if constexpr (SPLIT) {
#pragma unroll
                            for (int d = 0; d < 3; ++d) q[d] = field(at_load->src.off[d], j);
                            q[3] = (real)(int)(field(at_load->src.hash, j) - hr);
                            const int z = (r * 11) >> 5;
                            q[W::NR - 2] = (real)(r - 3 * z - 1) * T.Lf;
                            q[W::NR - 1] = (real)(z - 1) * T.Lf;
                        } else {
#pragma unroll
                            for (int d = 0; d < 3; ++d) q[d] = field(at_load->src.x[d], j);
                        }
                        load_fields<real, PASS, SOLID, CENSUS>(at_load, j, q + W::NPOS);
                        if (SPLIT || !multi)
                            a = framed(q, q[3], q[W::NR - 2], q[W::NR - 1], corner);
                        else
                            a = framed(q, 0, 0, 0, corner_of[gv]);
                        a.w = a.x * a.x + a.y * a.y + a.z * a.z;
                        const uint32_t k = row * (uint32_t)kPitch + place;
#pragma unroll
                        for (int c = 0; c < W::NV; ++c) {
                            full v;
#pragma unroll
                            for (int e = 0; e < C; ++e) v[e] = c * C + e < W::NR ? q[c * C + e] : real(0);
                            plane[c][k] = v;
                        }
                        if constexpr (W::HALF) {
                            half v;
#pragma unroll
                            for (int e = 0; e < C / 2; ++e) v[e] = W::NV * C + e < W::NR ? q[W::NV * C + e] : real(0);
                            plane_h[k] = v;
                        }
                    }
                    if (u < ends) cand[row * (uint32_t)kCandPitch + place] = a;
                }
                __syncthreads();

                // The candidate test, 16 entries x 16 targets at a time: block m of
                // rows 4 k .. 4 k + 3 takes their places 4 m .. 4 m + 3, lane l
                // receives the values of row 4 k + l / 16 for target l % 16 and
                // shifts their signs into word k, place 0 highest.
                uint32_t word[kWords];
                const float *pa = reinterpret_cast<const float *>(cand + ((lane & 15) >> 2) * kCandPitch + (lane & 3)) + quarter;
#pragma unroll
                for (int k = 0; k < kWords; ++k) word[k] = 0;
                float aop[kWords];
#pragma unroll
                for (int k = 0; k < kWords; ++k) aop[k] = pa[k * 4 * kCandPitch * 4];
                for (uint32_t m = in_tile ? 1 : blocks + 1; m <= blocks; ++m) {
                    f32x4 c[kWords];
#pragma unroll
                    for (int k = 0; k < kWords; ++k) c[k] = __builtin_amdgcn_mfma_f32_16x16x4f32(aop[k], bop, cinit, 0, 0, 0);
                    if (m < blocks) {   // the next block's operands
                        pa += 16;
#pragma unroll
                        for (int k = 0; k < kWords; ++k) aop[k] = pa[k * 4 * kCandPitch * 4];
                    }
#pragma unroll
                    for (int k = 0; k < kWords; ++k)
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const float v = c[k][e];
                            word[k] = __builtin_amdgcn_alignbit(word[k], __builtin_bit_cast(uint32_t, v), 31);
                        }
                }
                __syncthreads();   // every read of the operands is done: the lists take their place
                if (!in_tile) continue;
                const uint32_t top = 4 * blocks - 1;   // place 0's bit
                {
                    const CallArgs<real> at_eval = call_args<real>();
                    K.hinv = at_eval->A.K.hinv, K.Fc = at_eval->A.K.Fc, K.beta = at_eval->A.K.beta;
                    K.half_beta = at_eval->A.K.half_beta, K.F3 = at_eval->A.K.F3, K.F225 = at_eval->A.K.F225;
                    K.F075 = at_eval->A.K.F075, K.hb4 = at_eval->A.K.hb4, K.hbq = at_eval->A.K.hbq;
                    R2 = at_eval->A.R2;
                }
                int own = 0;
#pragma unroll
                for (int k = 0; k < kWords; ++k) own += __popc(word[k]);
                // the four lanes that tested a target list its hits one after the other
                const int own16 = __shfl_xor(own, 16, kWave);
                const int two = own + own16, two32 = __shfl_xor(two, 32, kWave);
                const int before = ((quarter & 1) ? own16 : 0) + ((quarter & 2) ? two32 : 0);
                const int all = two + two32;
                const int mine = __shfl(all, lane / kShare, kWave);   // of the target the lane evaluates
                // rounds of up to kCap listed hits per target (one, unless the
                // particles are far denser than a lattice)
                const bool fits = !ballot(all > kCap);
                for (int done = 0; ballot(all > done); done += kCap) {
                    uint16_t *to = list + lf * kListPitch;
                    int pos = before - done;
#pragma unroll
                    for (int k = 0; k < kWords; ++k) {
                        // a bit b stands for the source in slot last - b
                        const uint32_t last = (uint32_t)((4 * k + quarter) * kPitch) + top;
                        uint32_t w = word[k];
                        if (fits) {
                            // a word's hits from both ends at once; the last of an
                            // odd number is written twice, to the same place
                            uint16_t *lo = to + pos, *hi = to + (pos += __popc(w)) - 1;
                            while (w) {
                                const int a = __builtin_clz(w), z = __builtin_ctz(w);
                                *lo++ = (uint16_t)(last - 31u + (uint32_t)a);
                                *hi-- = (uint16_t)(last - (uint32_t)z);
                                w &= 0x7FFFFFFFu >> a;
                                w &= w - 1u;
                            }
                        } else {
                            while (w) {
                                const int z = __builtin_ctz(w);
                                w &= w - 1u;
                                if ((uint32_t)pos < (uint32_t)kCap) to[pos] = (uint16_t)(last - (uint32_t)z);
                                ++pos;
                            }
                        }
                    }
                    wave_lds_sync();   // the lists are written
                    const int left = mine - done;
                    const int cnt = left < 0 ? 0 : (left < kCap ? left : kCap);
                    const int most = wave_max_u7(cnt);
                    // a target's lanes take its hits in turn (what a lane reads
                    // past the list's end is not evaluated)
                    const uint16_t *hits = list + le * kListPitch;
                    auto slot = [&](int s) { return min((uint32_t)hits[s], (uint32_t)(kRows * kPitch - 1)); };
                    if constexpr (W::kTwoAhead) {
                        // while a pair is evaluated the next hit's record is read,
                        // and the slot of the one after it
                        real qa[kRec], qb[kRec];
                        uint32_t ka = slot(sub), kb = slot(sub + kShare);
                        fetch(ka, qa);
                        ka = slot(sub + 2 * kShare);
                        fetch(kb, qb);
                        kb = slot(sub + 3 * kShare);
                        for (int s = sub; s - sub < most; s += 2 * kShare) {
                            if (s < cnt) eval(qa);
                            fetch(ka, qa);
                            ka = slot(s + 4 * kShare);
                            if (s + kShare < cnt) eval(qb);
                            fetch(kb, qb);
                            kb = slot(s + 5 * kShare);
                        }
                    } else {
                        real q[kRec];
                        uint32_t k = slot(sub);   // the slot of the next hit is read ahead
#pragma unroll 2
                        for (int s = sub; s - sub < most; s += kShare) {
                            fetch(k, q);
                            k = slot(s + kShare);
                            if (s < cnt) eval(q);
                        }
                    }
                    wave_lds_sync();   // the lists are read
                }
            }
        }
    }

    if constexpr (CENSUS) {
#pragma unroll
        for (int off = 1; off < kShare; off <<= 1) {
            ncen += __shfl_xor(ncen, off, kWave);
            scen += __shfl_xor(scen, off, kWave);
        }
        if (valid && sub == 0) {
            call.cz.count[i] = ncen;
            call.cz.sum[i] = scen;
        }
    } else {
        // The workgroup's sums go through LDS, so that a wavefront reads and
        // stores every fourth output of all targets, 64 lanes at a time, instead
        // of every output of its 16 (2 M targets with half a million sources
        // among them, two passes: 1,152 -> 1,100 us; FP32 reverse 232 -> 227).
        __syncthreads();   // every read of the lists is done
        double *const sums = reinterpret_cast<double *>(shared);
        static_assert(NOUT * kGroup * 8 <= W::kShared, "the sums fit");
#pragma unroll
        for (int k = 0; k < NOUT; ++k) {
            acc[k].s = share_sum<kShare>(acc[k].s);
            if (sub == (k & (kShare - 1))) sums[k * kGroup + le] = acc[k].s;
        }
        __syncthreads();
        if (!tvalid) return;
        const CallArgs<real> at_end = call_args<real>();
        const auto &B = at_end->B;
        real *const adj[17] = {B.x[0], B.x[1], B.x[2], B.v[0], B.v[1], B.v[2], B.w, B.rho, B.p, B.c, B.e,
                               B.S[0], B.S[1], B.S[2], B.S[3], B.S[4], B.S[5]};
#pragma unroll
        for (int k = 0; k < NOUT; ++k) {
            if ((k & (kPairWaves - 1)) != wave0) continue;
            double sum = sums[k * kGroup + lane];
            if constexpr (ADJ || GADJ) {
                // accumulate the cotangents of x, v, omega (FORCE: rho, p, c, e and S too)
                auto &to = entry(adj[k], ti);
                to = (real)((double)to + sum);
            } else {
                auto &hi = entry(FORCE ? at_end->R.hi[k] : at_end->R.Lhi[k], ti);
                auto &lo = entry(SPLIT ? (FORCE ? at_end->R.lo[k] : at_end->R.Llo[k]) : (real *)nullptr, SPLIT ? ti : 0u);
                if (!at_end->zero_first) sum += SPLIT ? (double)hi + (double)lo : (double)hi;
                const real hv = (real)sum;
                hi = hv;
                if constexpr (SPLIT) lo = (real)(sum - (double)hv);
            }
        }
    }
}

// Candidates and hits of one pass, with the predicate of the pair kernel.
template <typename real, bool SELF>
__global__ __launch_bounds__(kBlock) void k_count(Params P, Grid g, PV<real> tg, const uint32_t *__restrict__ tidx,
                                                  const uint32_t *__restrict__ ntdev, PV<real> sr,
                                                  const uint32_t *__restrict__ sstart,
                                                  unsigned long long *__restrict__ counts)
{
    constexpr bool SPLIT = sizeof(real) == 4;
    uint32_t t = blockIdx.x * kBlock + threadIdx.x;
    uint32_t nt = tg.n;
    if (tidx) {
        uint32_t c = *ntdev;
        nt = c < nt ? c : nt;
    }
    unsigned long long cand = 0, hits = 0;
    const uint32_t i = t < nt ? (tidx ? tidx[t] : t) : tg.n;
    if (i < tg.n) {   // a listed index outside the target array names no target
        const real R2 = (real)P.R2;
        const real Lf = SPLIT ? (real)g.Lf : real(0);
        const uint32_t h = tg.hash[i];
        const int cx = (int)(h % (uint32_t)g.nx);
        const int cy = (int)((h / (uint32_t)g.nx) % (uint32_t)g.ny);
        const int cz = (int)(h / ((uint32_t)g.nx * (uint32_t)g.ny));
        const int x0 = cx > 0 ? cx - 1 : 0;
        const int x1 = cx + 1 < g.nx ? cx + 1 : g.nx - 1;
        double xi[3];
        real oi[3];
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            if constexpr (SPLIT)
                oi[d] = tg.off[d][i];
            else
                xi[d] = tg.x[d][i];
        }
        for (int dz = -1; dz <= 1; ++dz) {
            const int z = cz + dz;
            if (z < 0 || z >= g.nz) continue;
            for (int dy = -1; dy <= 1; ++dy) {
                const int y = cy + dy;
                if (y < 0 || y >= g.ny) continue;
                const uint32_t row = (uint32_t)g.nx * ((uint32_t)y + (uint32_t)g.ny * (uint32_t)z);
                const uint32_t jb = sstart[row + x0], je = sstart[row + x1 + 1];
                const uint32_t sA = sstart[row + cx], sB = sstart[row + cx + 1];
                const real ddy = (real)dy * Lf, ddz = (real)dz * Lf;
                for (uint32_t j = jb; j < je; ++j) {
                    if (SELF && j == i) continue;
                    real d[3];
                    if constexpr (SPLIT) {
                        const int dcx = (int)(j >= sB) - (int)(j < sA);
                        d[0] = (real)dcx * Lf + (sr.off[0][j] - oi[0]);
                        d[1] = ddy + (sr.off[1][j] - oi[1]);
                        d[2] = ddz + (sr.off[2][j] - oi[2]);
                    } else {
                        d[0] = sr.x[0][j] - xi[0];
                        d[1] = sr.x[1][j] - xi[1];
                        d[2] = sr.x[2][j] - xi[2];
                    }
                    ++cand;
                    const real r2 = r2_of<real>(d);
                    hits += (r2 < R2 && r2 > real(0)) ? 1u : 0u;
                }
            }
        }
    }
    // wavefront sums, one atomic per wavefront (integer: order-independent)
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) {
        cand += __shfl_down(cand, off, kWave);
        hits += __shfl_down(hits, off, kWave);
    }
    if ((threadIdx.x & (kWave - 1)) == 0) {
        atomicAdd(&counts[0], cand);
        atomicAdd(&counts[1], hits);
    }
}

// One pass, or its census.
template <typename real, int PASS, bool SOLID, bool CENSUS = false>
hipError_t go(const Params &P, const Grid &g, const sph_particles &tg, const uint32_t *tidx,
              const uint32_t *nt, const sph_particles &sr, const uint32_t *sstart, int zero_first,
              const sph_rates &r, const sph_adjoint &bar, hipStream_t s, const Census cz = Census{},
              const sph_rates *rsrc = nullptr)
{
    if (tg.n == 0) return hipSuccess;
    const sph_rates none{};
    hipEvent_t ev_begin = static_cast<hipEvent_t>(g_pair_events[0].load());
    hipEvent_t ev_end = static_cast<hipEvent_t>(g_pair_events[1].load());
    if (ev_begin && ev_end) {
        const hipError_t e = hipEventRecord(ev_begin, s);
        if (e != hipSuccess) return e;
    }
    const real linv = g.L > 0x1p-60 && g.L < 0x1p45 ? (real)(1.0 / g.L) : (real)NAN;
    auto above = [](int d) { return (1.0 + 0x1p-50) / d; };
    const PairCall<real> call{{make_pair_k<real>(P), (real)P.R2, (float)(2.0 * P.h)}, g, view<real>(tg), tidx, nt,
                              view<real>(sr), sstart, above(g.nx), above(g.ny), linv, zero_first, view<real>(r), view<real>(rsrc ? *rsrc : none),
                              view<real>(bar), cz};
    auto launch = [&](auto kernel, int group) { kernel<<<div_up(tg.n, group), kPairBlock, 0, s>>>(call); };
    // The fewest targets per wavefront whose workgroups are all resident at
    // once (one per SIMD's wavefront on each CU): below that a call is bound by
    // the latency of one workgroup's chain of loads and barriers, which fewer
    // targets shorten; above it their windows overlap more and the chip is full.
    // 16, 8 and 4 targets, in us a call (12 of them the launch): FORCE FP32 of
    // 1,728 particles 20, 14, 12; 8,000 20, 14, 13; 27,000 22, 21, 27; 46,656 29,
    // 31, 42; 64,000 33, 36, 52; solid FP64 FORCE of 4,096 25, 16, 14; 13,824 28,
    // 21, 28; its reverse (one workgroup per CU) 35, 24, 20 and 41, 44, 64.
    using W4 = Pass<real, PASS, SOLID, 4>;
    using W8 = Pass<real, PASS, SOLID, 8>;
    if (div_up(tg.n, W4::kGroup) <= kCUs * W4::waves)
        launch(k_pairs<real, PASS, SOLID, 4, CENSUS>, W4::kGroup);
    else if (div_up(tg.n, W8::kGroup) <= kCUs * W8::waves)
        launch(k_pairs<real, PASS, SOLID, 8, CENSUS>, W8::kGroup);
    else
        launch(k_pairs<real, PASS, SOLID, 16, CENSUS>, Pass<real, PASS, SOLID, 16>::kGroup);
    const hipError_t le = hipGetLastError();
    if (le != hipSuccess) return le;
    if (ev_begin && ev_end) return hipEventRecord(ev_end, s);
    return hipSuccess;
}

template <typename real>
hipError_t go_prec(const Params &P, const Grid &g, int pass, const sph_particles &tg, const uint32_t *tidx,
                   const uint32_t *nt, const sph_particles &sr, const uint32_t *sstart, int zero_first,
                   const sph_rates &r, hipStream_t s)
{
    const sph_adjoint none{};
    if (pass == SPH_PASS_GRADIENT)
        return go<real, SPH_PASS_GRADIENT, false>(P, g, tg, tidx, nt, sr, sstart, zero_first, r, none, s);
    if (P.material == SPH_SOLID_J2)
        return go<real, SPH_PASS_FORCE, true>(P, g, tg, tidx, nt, sr, sstart, zero_first, r, none, s);
    return go<real, SPH_PASS_FORCE, false>(P, g, tg, tidx, nt, sr, sstart, zero_first, r, none, s);
}

template <typename real>
hipError_t go_adjoint(const Params &P, const Grid &g, int pass, const sph_particles &tg, const uint32_t *tidx,
                      const uint32_t *nt, const sph_particles &sr, const uint32_t *sstart, const sph_rates &rbar_t,
                      const sph_rates &rbar_s, const sph_adjoint &bar, hipStream_t s)
{
    if (pass == SPH_PASS_GRADIENT)
        return go<real, kPassGradAdjoint, false>(P, g, tg, tidx, nt, sr, sstart, 0, rbar_t, bar, s, Census{}, &rbar_s);
    if (P.material == SPH_SOLID_J2)
        return go<real, kPassAdjoint, true>(P, g, tg, tidx, nt, sr, sstart, 0, rbar_t, bar, s, Census{}, &rbar_s);
    return go<real, kPassAdjoint, false>(P, g, tg, tidx, nt, sr, sstart, 0, rbar_t, bar, s, Census{}, &rbar_s);
}

}  // namespace

hipError_t launch_count_pairs(const Params &P, const Grid &g, int prec, const sph_particles &tg,
                              const uint32_t *tidx, const uint32_t *nt, const sph_particles &sr,
                              const uint32_t *sstart, bool self, uint64_t *counts, hipStream_t s)
{
    uint32_t blocks = div_up(tg.n, kBlock);
    if (blocks == 0) return hipSuccess;
    auto *c = reinterpret_cast<unsigned long long *>(counts);
    if (prec == SPH_FP64) {
        if (self)
            k_count<double, true><<<blocks, kBlock, 0, s>>>(P, g, view<double>(tg), tidx, nt, view<double>(sr),
                                                            sstart, c);
        else
            k_count<double, false><<<blocks, kBlock, 0, s>>>(P, g, view<double>(tg), tidx, nt, view<double>(sr),
                                                             sstart, c);
    } else {
        if (self)
            k_count<float, true><<<blocks, kBlock, 0, s>>>(P, g, view<float>(tg), tidx, nt, view<float>(sr),
                                                           sstart, c);
        else
            k_count<float, false><<<blocks, kBlock, 0, s>>>(P, g, view<float>(tg), tidx, nt, view<float>(sr),
                                                            sstart, c);
    }
    return hipGetLastError();
}

hipError_t launch_census(const Params &P, const Grid &g, int prec, int pass, const sph_particles &tg,
                         const uint32_t *tidx, const uint32_t *nt, const sph_particles &sr, const uint32_t *sstart,
                         uint32_t *count, uint64_t *sum, hipStream_t s)
{
    const sph_rates none{};
    const sph_adjoint nobar{};
    const Census cz{count, reinterpret_cast<unsigned long long *>(sum), sr.id};
    auto run = [&](auto real_v) {
        using real = decltype(real_v);
        if (pass == SPH_PASS_GRADIENT)
            return go<real, SPH_PASS_GRADIENT, false, true>(P, g, tg, tidx, nt, sr, sstart, 1, none, nobar, s, cz);
        if (P.material == SPH_SOLID_J2)
            return go<real, SPH_PASS_FORCE, true, true>(P, g, tg, tidx, nt, sr, sstart, 1, none, nobar, s, cz);
        return go<real, SPH_PASS_FORCE, false, true>(P, g, tg, tidx, nt, sr, sstart, 1, none, nobar, s, cz);
    };
    return prec == SPH_FP64 ? run(double()) : run(float());
}

hipError_t launch_interact_adjoint(const Params &P, const Grid &g, int prec, int pass, const sph_particles &tg,
                                   const uint32_t *tidx, const uint32_t *nt, const sph_particles &sr,
                                   const uint32_t *sstart, const sph_rates &rbar_t, const sph_rates &rbar_s,
                                   const sph_adjoint &bar, hipStream_t s)
{
    if (prec == SPH_FP64) return go_adjoint<double>(P, g, pass, tg, tidx, nt, sr, sstart, rbar_t, rbar_s, bar, s);
    return go_adjoint<float>(P, g, pass, tg, tidx, nt, sr, sstart, rbar_t, rbar_s, bar, s);
}

hipError_t launch_interact(const Params &P, const Grid &g, int prec, int pass, const sph_particles &tg,
                           const uint32_t *tidx, const uint32_t *nt, const sph_particles &sr, const uint32_t *sstart,
                           int zero_first, const sph_rates &r, hipStream_t s)
{
    if (prec == SPH_FP64) return go_prec<double>(P, g, pass, tg, tidx, nt, sr, sstart, zero_first, r, s);
    return go_prec<float>(P, g, pass, tg, tidx, nt, sr, sstart, zero_first, r, s);
}

void set_pair_events(void *begin, void *end)
{
    g_pair_events[0].store(begin);
    g_pair_events[1].store(end);
}

}  // namespace sph
