// Exact per-KV-head top-k of alpha[h, 0..L) for gfx950 (Alg. 1 "S <- Top-k(alpha)", Eq. 5):
// the k positions with the largest fp32 value, equal values to the smaller index, indices
// emitted in ascending order.  alpha >= 0, so the order of the fp32 bit patterns as unsigned
// integers is the order of the values.
//
// One workgroup of 1024 threads per KV head.  The work is one chain of short dependent phases on a single
// workgroup, so its time is the number of phases (a barrier each, 16 wavefronts on 4 SIMDs: every instruction of a
// phase costs 16 issue cycles) plus the round trips to memory.  Hence ONE histogram instead of a radix select: alpha is a
// probability, so its useful range is known beforehand and a bin is a fixed interval of the fp32 bit pattern
// (value_bin: 64 octaves below 1.0, 64 bins per octave).  Everything above the bin that holds rank k is in, and only
// the few elements of that bin (1.6 % of a value, typically 5 .. 50 elements) are ranked exactly, all pairs at once.  Two routes:
//   direct route: the row is binned element by element, then classified.  For rows that one sweep of registers
//     holds (L <= 16384), and for large k, where a filter would let most of the row through.
//   filter route (long rows, k up to three quarters of the groups): the k-th largest of the maxima of disjoint groups of elements is a lower bound
//     of the k-th largest element.  The column-sum pass leaves one maximum per kGroupKeys consecutive keys; they are
//     binned first and only the groups at or above the bound (about k of them) are read at all.
// Membership is kept as a bitmap in LDS; walking it gives the positions in ascending order.
// Measured (profiler) at k = 512: Hkv = 4, L = 8192: 19.7 us with the radix select that stood here (a filter in front of it
// at every length, two digits for the bound and three for the k-th value), 6.2 us now; Hkv = 8, L = 131072: 18.4 us
// before, 12.3 us now.  The row is read by a straight line of code that is fetched once, at about 13 cycles per
// instruction, so what is not executed in the usual case (ragged ends, second sweeps, near-ties) sits behind branches.
//   radix route (the exit for everything else: more ties around rank k than TK_LIST, more groups at
//     or above the bound than TK_HITS, a k-th value below 2^-64, k > 2048 in a row longer than TK_BITMAP): three MSB-first radix-select steps over the whole row find the k-th value and the
//     number of ties to keep, then an ordered sweep emits the set.
// Near-ties at rank k: alpha is an fp32 result whose relative error (a few 1e-6 from the
// fp32 dot products, exponentials and sums) is of the order of typical gaps between neighbouring values
// at rank k, so the fp32 ranking can differ from the ranking of the exactly computed averages.  The
// candidates within `eps` (relative) of the k-th value -- usually none, a handful at most -- are therefore
// scored again from the inputs in fp64 (exact dot products, fp64 exponentials, the row normalisers
// merged in fp64 from the per-split statistics), rounded to fp32 once, and ranked among themselves by
// (value, smaller index first); as many of them enter the set as the fp32 ranking had admitted.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "combine.hpp"
#include "ids.hpp"
#include "plan.hpp"

namespace mage {

constexpr int TK_THREADS = 1024;
constexpr int TK_WAVES = TK_THREADS / 64;
constexpr int TK_BINS = 4096;
constexpr int TK_EPT = 16;                           // elements per thread in a sweep of the row
constexpr int TK_SWEEP = TK_THREADS * TK_EPT;        // elements one sweep covers
constexpr int TK_HITS = 4096;                        // filter route: groups at or above the bound, at most
constexpr int TK_NX = 4;                             // filter route: 16-byte pieces of those groups that a thread keeps in registers
constexpr int TK_FILTER_MAX_K = 2048;
constexpr int TK_LIST = 512;                         // elements around rank k that are ranked all pairs
constexpr uint32_t TK_MARGIN = 256;                  // the list reaches this many bit patterns past the bin of rank k: more than
                                                     // the near-tie band on either side (a pattern is at least 2^-24 of a value)
constexpr int TK_BITMAP = 262144;                    // positions whose membership bits LDS holds
constexpr int TK_NEAR_MAX = 32;                      // candidates re-scored at most; more of them (massive ties) keep the fp32 ranking

// Inclusive prefix sum over the 64 lanes of a wavefront with data-parallel-primitive moves
// (row shifts inside rows of 16 lanes, then the row broadcasts of the gfx9 family): eight
// vector-ALU instructions instead of six trips through the LDS crossbar.
__device__ __forceinline__ uint32_t wave_scan_incl(uint32_t x)
{
    constexpr int ROW_SHR = 0x110, ROW_BCAST15 = 0x142, ROW_BCAST31 = 0x143;
    uint32_t v = x;
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, ROW_SHR + 1, 0xf, 0xf, true);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, ROW_SHR + 2, 0xf, 0xf, true);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, ROW_SHR + 3, 0xf, 0xf, true);      // x[l-3..l] inside the row
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, ROW_SHR + 4, 0xf, 0xe, true);      // lanes 4..15 of a row: 8 terms
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, ROW_SHR + 8, 0xf, 0xc, true);      // lanes 8..15: the whole row prefix
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, ROW_BCAST15, 0xa, 0xf, true);      // rows 1 and 3 take the row before
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, ROW_BCAST31, 0xc, 0xf, true);      // rows 2 and 3 take lane 31
    return v;
}

// value of a wavefront-uniform lane
__device__ __forceinline__ uint32_t lane_value(uint32_t v, int lane_uniform)
{
    return (uint32_t)__builtin_amdgcn_readlane((int)v, __builtin_amdgcn_readfirstlane(lane_uniform));
}

// inclusive scan of one value per thread over the workgroup; returns this thread's inclusive
// prefix and the workgroup total.  `tmp` holds TK_WAVES entries.  Every wavefront adds up the
// per-wavefront totals itself (TK_WAVES <= 64 lanes), so nothing runs on a single thread.
__device__ __forceinline__ uint32_t block_scan_incl(uint32_t v, uint32_t *tmp, uint32_t &total)
{
    const int lane = tid_x() & 63, wave = tid_x() >> 6;
    const uint32_t x = wave_scan_incl(v);
    __syncthreads();                      // tmp may still be read from a previous call
    if (lane == 63) tmp[wave] = x;
    __syncthreads();
    const uint32_t w = lane < TK_WAVES ? tmp[lane] : 0u;
    const uint32_t wi = wave_scan_incl(w);
    total = lane_value(wi, TK_WAVES - 1);
    return x + lane_value(wi - w, wave);
}

// Histogram bin of a value, larger values first: 64 bins per octave from 1.0 (bin 0) down to 2^-64.  What lies outside
// (smaller values, the zeros behind the end of a row) has a bin number, taken as unsigned, beyond TK_BIN_LAST.
// bin_floor: the smallest bit pattern in a bin -- value_bin(x) <= b exactly if x >= bin_floor(b).
constexpr int TK_BIN_SHIFT = 17, TK_BIN_ONE = 0x3f800000 >> TK_BIN_SHIFT;
constexpr uint32_t TK_BIN_LAST = TK_BINS - 2;
__device__ __forceinline__ uint32_t value_bin(uint32_t x) { return (uint32_t)TK_BIN_ONE - (x >> TK_BIN_SHIFT); }
__device__ __forceinline__ uint32_t bin_floor(int b) { return (uint32_t)(TK_BIN_ONE - b) << TK_BIN_SHIFT; }

// Four consecutive elements of a row; rows start at any multiple of four bytes (the hardware loads 16 bytes from there in
// one go).
struct __attribute__((packed, aligned(4))) Piece { uint32_t v[4]; };

// piece at element j (zeros past the end)
__device__ __forceinline__ void load_piece_tail(const uint32_t *row, long long j, long long len, uint32_t (&x)[4])
{
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const uint32_t v = row[j + c < len ? j + c : len - 1];
        x[c] = j + c < len ? v : 0u;
    }
}

// The bin in which the `want`-th largest element falls, the number of elements in the bins before it and its own
// count.  Two barriers: after the histogram, and after every wavefront has published the running sums of its threads'
// bins; from those every wavefront works out the answer itself.  Fewer than `want` elements in all: the last bin.
__device__ __forceinline__ void pick_bin(const uint32_t *hist, uint32_t want, uint32_t *lscan, uint32_t *wtot, int &bin, uint32_t &before)
{
    constexpr int PER = TK_BINS / TK_THREADS;
    static_assert(PER == 4, "a thread reads its bins as one 16-byte load");
    const int lane = tid_x() & 63, wave = tid_x() >> 6;
    __syncthreads();
    const uint4 c = *reinterpret_cast<const uint4 *>(hist + tid_x() * PER);
    const uint32_t incl = wave_scan_incl(c.x + c.y + c.z + c.w);
    lscan[tid_x()] = incl;
    if (lane == 63) wtot[wave] = incl;
    __syncthreads();
    // the wavefront, then the thread, in whose bins the running count reaches `want`
    const uint32_t w = lane < TK_WAVES ? wtot[lane] : 0u;
    const uint32_t wi = wave_scan_incl(w);
    const unsigned long long wmask = __ballot(lane < TK_WAVES && wi >= want);
    const int wsel = wmask ? __ffsll((long long)wmask) - 1 : TK_WAVES - 1;
    const uint32_t wbase = lane_value(wi - w, wsel);                       // elements in the wavefronts before it
    const uint32_t v = lscan[wsel * 64 + lane];
    const unsigned long long lmask = __ballot(wbase + v >= want);
    const int lsel = lmask ? __ffsll((long long)lmask) - 1 : 63;
    const int tsel = wsel * 64 + lsel;
    uint32_t run = wbase + (lsel > 0 ? lane_value(v, lsel > 0 ? lsel - 1 : 0) : 0u);   // elements in the bins before that thread's
    const uint4 d = *reinterpret_cast<const uint4 *>(hist + tsel * PER);
    int i = 0;
    if (run + d.x < want) { run += d.x; i = 1;
        if (run + d.y < want) { run += d.y; i = 2;
            if (run + d.z < want) { run += d.z; i = 3; } } }
    bin = tsel * PER + i;
    before = run;
}

// One radix step over n elements of u (global or LDS): histogram the `bits`-wide digit at
// `shift` of every element whose higher bits equal `prefix`, then pick the digit in which the
// `want`-th largest element falls.  On return prefix has that digit appended and want is the
// rank inside the digit's bucket.
__device__ __forceinline__ void radix_step(const uint32_t *u, long long n, int shift, int bits,
                                           uint32_t &prefix, uint32_t &want,
                                           uint32_t *hist, uint32_t *tmp, uint32_t *bcast)
{
    const int nb = 1 << bits;
    const uint32_t hi_mask = (shift + bits >= 32) ? 0u : (0xffffffffu << (shift + bits));
    for (int b = tid_x(); b < nb; b += TK_THREADS) hist[b] = 0;
    __syncthreads();
    constexpr int UNR = 8;      // independent loads in flight per thread
    for (long long j0 = tid_x(); j0 < n; j0 += (long long)TK_THREADS * UNR) {
        uint32_t x[UNR];
#pragma unroll
        for (int i = 0; i < UNR; ++i) {
            const long long j = j0 + (long long)i * TK_THREADS;
            x[i] = j < n ? u[j] : 0xffffffffu;
        }
#pragma unroll
        for (int i = 0; i < UNR; ++i) {
            const long long j = j0 + (long long)i * TK_THREADS;
            if (j < n && (x[i] & hi_mask) == prefix) atomicAdd(&hist[(x[i] >> shift) & (nb - 1)], 1u);
        }
    }
    __syncthreads();
    // thread t owns bins [t*per, (t+1)*per) counted from the TOP digit downwards
    const int per = (nb + TK_THREADS - 1) / TK_THREADS;
    uint32_t mine = 0;
    for (int i = 0; i < per; ++i) {
        const int b = nb - 1 - (tid_x() * per + i);
        if (b >= 0) mine += hist[b];
    }
    uint32_t total;
    const uint32_t incl = block_scan_incl(mine, tmp, total);
    const uint32_t excl = incl - mine;
    if (excl < want && want <= incl) {     // exactly one thread: the bucket lies in its bins
        uint32_t run = excl;
        for (int i = 0; i < per; ++i) {
            const int b = nb - 1 - (tid_x() * per + i);
            if (b < 0) break;
            const uint32_t c = hist[b];
            if (run < want && want <= run + c) {
                bcast[0] = (uint32_t)b;
                bcast[1] = want - run;
                bcast[2] = c;
                break;
            }
            run += c;
        }
    }
    __syncthreads();
    prefix |= bcast[0] << shift;
    want = bcast[1];
    __syncthreads();
}

// 2^x in fp64 for x <= 0 or a little above: Taylor series of 2^f, |f| <= 1/2, up to the term below 2^-52
__device__ __forceinline__ double exp2_f64(double x)
{
    x = fmax(x, -1100.0);                                // (zero, as far as fp64 goes)
    const double n = __builtin_rint(x), f = x - n;
    constexpr double C[13] = {1.0, 0.6931471805599453, 0.24022650695910072, 0.05550410866482158, 0.009618129107628477,      // ln2^k / k!
                              0.0013333558146428443, 0.0001540353039338161, 1.5252733804059841e-05, 1.321548679014431e-06,
                              1.01780860092397e-07, 7.054911620801123e-09, 4.4455382718708116e-10, 2.5678435993488206e-11};
    double p = C[12];
#pragma unroll
    for (int k = 11; k >= 0; --k) p = fma(p, f, C[k]);
    return __builtin_amdgcn_ldexp(p, (int)n);
}

// sum of q[e] * k[e] over the values of a 16-byte piece (8 bf16 or 4 fp32), in order; the product of two bf16 values is exact in
// fp32 (underflow below 2^-126 and overflow aside), which saves a conversion
__device__ __forceinline__ double dot_piece(const uint4 &q, const uint4 &k, int esz, double p)
{
    const uint32_t a[4] = {q.x, q.y, q.z, q.w}, b[4] = {k.x, k.y, k.z, k.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if (esz == 4) {
            p = fma((double)__uint_as_float(a[i]), (double)__uint_as_float(b[i]), p);
            continue;
        }
        p += (double)(__uint_as_float(a[i] << 16) * __uint_as_float(b[i] << 16));
        p += (double)(__uint_as_float(a[i] & 0xffff0000u) * __uint_as_float(b[i] & 0xffff0000u));
    }
    return p;
}

// the positive (neg = false) or negative part of the bf16 values of a piece
__device__ __forceinline__ uint4 signed_part(const uint4 &x, bool neg)
{
    auto part = [&](uint32_t v) {
        const uint32_t m = ((v >> 15) & 0x00010001u) * 0xffffu;                // all ones where the value is negative
        return neg ? v & m : v & ~m;
    };
    return make_uint4(part(x.x), part(x.y), part(x.z), part(x.w));
}

// x * 2^e for a whole number e <= 0 (far below -1100 too)
__device__ __forceinline__ double scale_pow2(double x, float e) { return __builtin_amdgcn_ldexp(x, (int)fmaxf(e, -1100.f)); }

// x of lane (l ^ 1) or (l ^ 2): a quad permutation, no trip through the LDS crossbar
template <int X>
__device__ __forceinline__ double quad_xor(double x)
{
    constexpr int PERM = X == 1 ? 0xb1 : 0x4e;
    return __hiloint2double(__builtin_amdgcn_update_dpp(0, __double2hiint(x), PERM, 0xf, 0xf, true),
                            __builtin_amdgcn_update_dpp(0, __double2loint(x), PERM, 0xf, 0xf, true));
}

// alpha[h, j] in fp64 from the inputs (Eq. 5) for n of the listed elements, j = list[slot[c]].y:
//   1/(G*B) * sum over the R rows of exp2(q_r.k_j * scale - M_r) / L_r,
// with (M_r, L_r) the row's softmax statistics merged in fp64 over the key splits.  Four threads per
// row (a quarter of the channels and of the splits each), 256 rows per pass.  Taken by one head in a few dozen, and then
// as a tail of the whole selection, bound by the instructions that sixteen wavefronts issue on one CU and by the dependent loads.  So
// the references of the statistics are whole numbers (the passes that write them see to it) and their merge needs no exponentials;
// the first query and key pieces are requested before the statistics, every piece after them one step ahead; and the
// wavefronts' sums of all candidates meet in LDS once, at the end.  Two candidates, 224 rows: 42 us with element-by-element loads and the
// library's exp2, 14 us with 16-byte loads and an exp2 of its own, 8 us now.  Every thread of the workgroup calls; out[c] receives the results rounded to fp32 (valid after the final barrier).
__device__ __forceinline__ void rescore_candidates(const RescoreArgs &rs, int h, const uint2 *list, const uint32_t *slot, int n, float *out,
                                   double *acc, double (*red)[TK_WAVES])
{
    constexpr int ROWS = TK_THREADS / 4;
    const int lane = tid_x() & 63, wave = tid_x() >> 6;
    const int part = tid_x() & 3, rl = tid_x() >> 2;
    const int cpt = rs.d / 4;
    const int pieces = cpt * rs.esz / 16;                  // 2, 4 or 8
    if (tid_x() < n) acc[tid_x()] = 0.0;
    auto key = [&](int c) {
        const long long ko = ((long long)list[slot[c]].y * rs.Hkv + h) * rs.d + part * cpt;
        return reinterpret_cast<const uint4 *>(static_cast<const char *>(rs.kc) + ko * rs.esz);
    };
    for (int r0 = 0; r0 < rs.R; r0 += ROWS) {              // uniform trip count (one pass unless R > 256)
        const int r = r0 + rl;
        const bool live = r < rs.R;
        // split_q: the queries are rows of d / 2 channels, to be taken as [max(q, 0) | min(q, 0)]  (rows past the last read row 0)
        const int gl = live ? r / rs.B : 0, qi = live ? r - gl * rs.B : 0;
        const long long qo = ((long long)qi * rs.Hq + (long long)h * rs.G + gl) * (rs.split_q ? rs.d / 2 : rs.d) + (rs.split_q ? (part & 1) : part) * cpt;
        const uint4 *qp = reinterpret_cast<const uint4 *>(static_cast<const char *>(rs.q) + qo * rs.esz);
        const uint4 *kp = key(0);
        uint4 q0 = qp[0], q1 = qp[1], k0 = kp[0], k1 = kp[1];

        // this row's statistics, merged over the key splits, eight in flight per thread
        constexpr int SF = 8;
        float M = -3.0e38f;
        double Lr = 0.0;
        const long long base = (long long)h * rs.n_split * rs.rpad + (live ? r : 0);
        for (int s0 = part; s0 < rs.n_split; s0 += 4 * SF) {
            float m[SF], l[SF], top = M;
#pragma unroll
            for (int i = 0; i < SF; ++i) {
                const int s = s0 + 4 * i;
                const long long pi = base + (long long)(s < rs.n_split ? s : s0) * rs.rpad;
                m[i] = rs.stat_m[pi];
                l[i] = s < rs.n_split ? rs.stat_l[pi] : 0.f;
            }
#pragma unroll
            for (int i = 0; i < SF; ++i) top = fmaxf(top, m[i]);
            Lr = scale_pow2(Lr, M - top);
            M = top;
#pragma unroll
            for (int i = 0; i < SF; ++i) Lr += scale_pow2((double)l[i], m[i] - M);
        }
        // the four threads of the row: one common reference, then plain sums
        float top = fmaxf(M, __shfl_xor(M, 1));
        top = fmaxf(top, __shfl_xor(top, 2));
        Lr = scale_pow2(Lr, M - top);
        Lr += quad_xor<1>(Lr);
        Lr += quad_xor<2>(Lr);
        M = top;
        const double inv = live && part == 0 ? 1.0 / Lr : 0.0;

        for (int c = 0; c < n; ++c) {
            double p = 0.0;
#pragma unroll 1
            for (int i = 0; i < pieces; i += 2) {
                uint4 qa = q0, qb = q1;
                const uint4 ka = k0, kb = k1;
                const bool last = i + 2 == pieces;           // then the next candidate's first pieces (after the last one: its own again)
                if (last && c + 1 < n) kp = key(c + 1);
                const int e = last ? 0 : i + 2;
                q0 = qp[e], q1 = qp[e + 1], k0 = kp[e], k1 = kp[e + 1];
                if (rs.split_q) {
                    qa = signed_part(qa, part >= 2);
                    qb = signed_part(qb, part >= 2);
                }
                p = dot_piece(qa, ka, rs.esz, p);
                p = dot_piece(qb, kb, rs.esz, p);
            }
            p += quad_xor<1>(p);
            p += quad_xor<2>(p);
            double t = exp2_f64(p * (double)rs.scale_log2 - (double)M) * inv;
#pragma unroll
            for (int d = 32; d >= 4; d >>= 1) t += __shfl_xor(t, d);           // (rows sit four lanes apart)
            if (lane == 0) red[c][wave] = t;
        }
        __syncthreads();
        if (tid_x() < n) {
            double tot = 0.0;
            for (int w = 0; w < TK_WAVES; ++w) tot += red[tid_x()][w];      // fixed order
            acc[tid_x()] += tot;
        }
        __syncthreads();                                   // the next pass writes red
    }
    if (tid_x() < n) out[tid_x()] = (float)(acc[tid_x()] * rs.inv_rows);
    __syncthreads();
}

// Bits [0, n) of the bitmap in ascending order (bits from n to the next multiple of 128 are zero): emit(rank, position)
// for every set bit, rank counted from `first`; returns the number of set bits.  The caller has put a barrier between
// the last change of the bitmap and this.
template <class Emit>
__device__ __forceinline__ uint32_t walk_bitmap(const uint32_t *bits, int n, uint32_t first, uint32_t *tmp, Emit emit)
{
    // Short bitmaps: 16 positions per thread.  Longer ones: whole words, four at a time where there are that many.
    const int words = (n + 31) >> 5;
    uint32_t w[4] = {0u, 0u, 0u, 0u};
    uint32_t total, mine = 0;
    int at, per;                                          // first word (half word) of this thread, words per thread
    if (words <= TK_THREADS / 2) {
        at = tid_x();
        per = 0;
        if (at < 2 * words) w[0] = reinterpret_cast<const uint16_t *>(bits)[at];
        mine = __popc(w[0]);
    } else {
        per = (words + TK_THREADS - 1) / TK_THREADS;
        per = per > 2 ? (per + 3) & ~3 : per;
        at = tid_x() * per;
        for (int i = 0; i < per; i += 4) {
            if (per >= 4) {
                const uint4 v = at + i < words ? *reinterpret_cast<const uint4 *>(bits + at + i) : make_uint4(0, 0, 0, 0);
                w[0] = v.x; w[1] = v.y; w[2] = v.z; w[3] = v.w;
            } else {
                if (at < words) w[0] = bits[at];
                if (per == 2 && at + 1 < words) w[1] = bits[at + 1];
            }
            mine += __popc(w[0]) + __popc(w[1]) + __popc(w[2]) + __popc(w[3]);
        }
    }
    uint32_t rank = first + block_scan_incl(mine, tmp, total) - mine;
    if (mine == 0) return total;
    if (per <= 1) {
        for (uint32_t b = w[0]; b; b &= b - 1) emit(rank++, at * (per ? 32 : 16) + __ffs(b) - 1);
        return total;
    }
    for (int i = 0; i < per; ++i)
        for (uint32_t b = at + i < words ? bits[at + i] : 0u; b; b &= b - 1) emit(rank++, (at + i) * 32 + __ffs(b) - 1);
    return total;
}

// DC: head dimension of attention partials that the workgroups from n_heads on merge (four query rows each), 0 = none.
// In the fused step 1 that merge (5 to 8 us as a launch of its own) depends on nothing but the attention pass and runs
// beside the top-k's few workgroups.
// PAGED: every selected element stands for `page` consecutive positions, which are what is written.
template <int DC, bool PAGED>
__global__ __launch_bounds__(TK_THREADS) void topk_kernel(const float *alpha, const float *group_max, long long L, int k, int32_t *idx_out,
                                                          const RescoreArgs rs, int page, int n_heads, const KernelArgs comb)
{
    if constexpr (DC > 0) {
        __shared__ CombineLds<DC> comb_lds[TK_THREADS / 256];
        if ((int)wg_x() >= n_heads) {                    // uniform
            const int sub = tid_x() >> 8;
            const int item = ((int)wg_x() - n_heads) * (TK_THREADS / 256) + sub, ch = item / comb.R;
            combine_row<DC>(comb, item - ch * comb.R, ch, tid_x() & 255, ch < comb.Hkv, comb_lds[sub]);
            return;
        }
    }
    __shared__ __attribute__((aligned(16))) uint32_t hist[TK_BINS + 64], hist2[TK_BINS];      // (the last 64 of hist: elements outside the bins)
    __shared__ __attribute__((aligned(16))) uint32_t bits[TK_BITMAP / 32];                    // membership by position
    __shared__ uint32_t lscan[TK_THREADS];
    __shared__ uint32_t tmp[TK_WAVES + 1];
    __shared__ uint32_t tmp2[TK_WAVES + 1];
    __shared__ uint32_t bcast[3];                        // radix route: chosen digit, rank inside its bucket, bucket size
    __shared__ uint32_t glist[TK_HITS];                  // filter route: groups at or above the bound
    __shared__ uint32_t winners[TK_FILTER_MAX_K];        // the set: for rows longer than the bitmap (unordered), or to be expanded to positions (ascending)
    __shared__ uint2 list[TK_LIST];                      // (value, position) around rank k
    __shared__ uint32_t ltake[TK_LIST];
    __shared__ uint32_t n_hit, n_cand, n_win, n_list, n_near, n_near_in, thr_bits, next_bits;
    __shared__ uint32_t near_slot[TK_NEAR_MAX];          // list entries within eps of the k-th value
    __shared__ float near_val[TK_NEAR_MAX];              // their fp64 score, rounded to fp32
    __shared__ double near_red[TK_NEAR_MAX][TK_WAVES], near_acc[TK_NEAR_MAX];

    const int h = wg_x();
    const uint32_t *u = reinterpret_cast<const uint32_t *>(alpha) + (long long)h * L;
    int32_t *out = idx_out + (long long)h * k * (PAGED ? page : 1);
    auto put = [&](uint32_t rank, int j) {
        if (PAGED) winners[rank] = (uint32_t)j;
        else out[rank] = j;
    };
    // a set of pages: every position of each of them (the caller keeps k <= TK_FILTER_MAX_K and L <= TK_BITMAP then)
    auto expand = [&] {
        if (!PAGED) return;
        __syncthreads();
        for (int i = tid_x(); i < k * page; i += TK_THREADS) {
            const int r = i / page;
            out[i] = (int32_t)winners[r] * page + (i - r * page);
        }
    };
    const int ng = (int)((L + kGroupKeys - 1) / kGroupKeys);          // group maxima of the row
    // a row of one sweep is binned directly; so is a longer one whose groups would mostly pass the filter
    const bool filter = L > TK_SWEEP && k <= ng - ng / 4 && k <= TK_FILTER_MAX_K;

    if (filter || L <= TK_BITMAP) {
        const int t = tid_x(), lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
        const uint32_t *row = filter ? reinterpret_cast<const uint32_t *>(group_max) + (long long)h * ng : u;
        const int len = filter ? ng : (int)L;
        // This thread's elements of a sweep: `per` consecutive ones (8 if that covers the row: then every wavefront has
        // work), in 16-byte pieces.
        const int per = len <= TK_SWEEP / 2 ? TK_EPT / 2 : TK_EPT;
        uint32_t x[TK_EPT / 4][4];
        auto sweep = [&](int j0) {
            const int j = j0 + t * per;
            if (j0 + (wave + 1) * 64 * per <= len) {      // uniform: nothing of this wavefront is past the end
#pragma unroll
                for (int i = 0; i < TK_EPT / 4; ++i)
                    if (4 * i < per) {                    // uniform
                        const Piece p = *reinterpret_cast<const Piece *>(row + j + 4 * i);
#pragma unroll
                        for (int c = 0; c < 4; ++c) x[i][c] = p.v[c];
                    }
            } else {
#pragma unroll
                for (int i = 0; i < TK_EPT / 4; ++i)
                    if (4 * i < per) load_piece_tail(row, j + 4 * i, len, x[i]);
            }
        };
        sweep(0);
        // while the loads travel
        reinterpret_cast<uint4 *>(hist)[t] = make_uint4(0, 0, 0, 0);
        if (filter) {
            reinterpret_cast<uint4 *>(hist2)[t] = make_uint4(0, 0, 0, 0);
            const int zero = (int)((L < TK_BITMAP ? L : TK_BITMAP) + 127) / 128;
            for (int i = t; i < zero; i += TK_THREADS) reinterpret_cast<uint4 *>(bits)[i] = make_uint4(0, 0, 0, 0);
        }
        if (t == 0) {
            n_hit = 0;
            n_cand = 0;
            n_win = 0;
            n_list = 0;
            next_bits = 0;
        }
        __syncthreads();

        for (int j0 = 0; j0 < len; j0 += TK_SWEEP) {
            if (j0 > 0) sweep(j0);
            if (j0 + wave * 64 * per < len) {             // uniform
#pragma unroll
                for (int i = 0; i < TK_EPT / 4; ++i)
                    if (4 * i < per)
#pragma unroll
                        for (int c = 0; c < 4; ++c) {
                            const uint32_t b = value_bin(x[i][c]);
                            atomicAdd(&hist[b <= TK_BIN_LAST ? b : (uint32_t)(TK_BINS + lane)], 1u);
                        }
            }
        }
        int bin;
        uint32_t before;
        pick_bin(hist, (uint32_t)k, lscan, tmp, bin, before);
        bool give_up = bin > (int)TK_BIN_LAST - 1;        // uniform: leave for the radix route

        // one bit per element of x that is at least `floor`
        auto at_least = [&](uint32_t floor) {
            uint32_t m = 0;
#pragma unroll
            for (int i = 0; i < TK_EPT / 4; ++i)
                if (4 * i < per)
#pragma unroll
                    for (int c = 0; c < 4; ++c) m |= (x[i][c] >= floor ? 1u : 0u) << (4 * i + c);
            return m;
        };
        // elements around rank k: bit e of `m` = position j + e
        auto append = [&](uint32_t m, int j) {
            if (m == 0) return;
            uint32_t p = atomicAdd(&n_list, (uint32_t)__popc(m));
            while (m) {
                const int e = __ffs(m) - 1;
                if (p < TK_LIST) list[p] = make_uint2(u[j + e], (uint32_t)(j + e));
                ++p;
                m &= m - 1;
            }
        };
        if (!filter) {
            // in: everything above `bin` and its margin; listed: `bin` and the margins
            const uint32_t in_floor = bin_floor(bin - 1) + TK_MARGIN, list_floor = bin_floor(bin) - TK_MARGIN;
            for (int j0 = 0; j0 < len && !give_up; j0 += TK_SWEEP) {
                if (len > TK_SWEEP) sweep(j0);
                if (j0 + wave * 64 * per < len) {
                    const uint32_t in = at_least(in_floor);
                    append(at_least(list_floor) & ~in, j0 + t * per);
                    if (per == 8) reinterpret_cast<uint8_t *>(bits)[t] = (uint8_t)in;
                    else reinterpret_cast<uint16_t *>(bits)[(j0 >> 4) + t] = (uint16_t)in;
                }
            }
        } else {
            // ---- groups at or above the bound (and its margin)
            const uint32_t floor = bin_floor(bin) - TK_MARGIN;
            for (int j0 = 0; j0 < len && !give_up; j0 += TK_SWEEP) {
                if (len > TK_SWEEP) sweep(j0);
                uint32_t m = j0 + wave * 64 * per < len ? at_least(floor) : 0u;
                const uint32_t cnt = __popc(m), incl = wave_scan_incl(cnt), all = lane_value(incl, 63);
                if (all == 0) continue;                   // uniform per wavefront
                uint32_t base = 0;
                if (lane == 0) base = atomicAdd(&n_hit, all);
                uint32_t p = lane_value(base, 0) + incl - cnt;
                while (m) {
                    if (p < TK_HITS) glist[p] = (uint32_t)(j0 + t * per + __ffs(m) - 1);
                    ++p;
                    m &= m - 1;
                }
            }
            __syncthreads();
            // ---- their elements, 16 bytes per thread: kept in registers while TK_NX pieces per thread cover them
            const uint32_t nh = n_hit;
            give_up = give_up || nh > TK_HITS;
            constexpr int QPG = kGroupKeys / 4;           // pieces per group
            const int items = give_up ? 0 : (int)nh * QPG;
            int jp[TK_NX];
            auto fetch = [&](int i0) {
#pragma unroll
                for (int i = 0; i < TK_NX; ++i)
                    if (i0 + i * TK_THREADS < items) {    // uniform
                        const int it = i0 + i * TK_THREADS + t;
                        jp[i] = (int)glist[it < items ? it / QPG : 0] * kGroupKeys + 4 * (it % QPG);
                        if (it >= items) {
                            x[i][0] = x[i][1] = x[i][2] = x[i][3] = 0u;
                        } else if (jp[i] + 4 <= L) {
                            const Piece pc = *reinterpret_cast<const Piece *>(u + jp[i]);
#pragma unroll
                            for (int c = 0; c < 4; ++c) x[i][c] = pc.v[c];
                        } else {
                            load_piece_tail(u, jp[i], L, x[i]);
                        }
                    }
            };
            for (int i0 = 0; i0 < items; i0 += TK_NX * TK_THREADS) {
                fetch(i0);
                uint32_t cnt = 0;
#pragma unroll
                for (int i = 0; i < TK_NX; ++i)
                    if (i0 + i * TK_THREADS < items)
#pragma unroll
                        for (int c = 0; c < 4; ++c)
                            if (x[i][c] >= floor) {
                                atomicAdd(&hist2[value_bin(x[i][c])], 1u);
                                ++cnt;
                            }
                cnt = lane_value(wave_scan_incl(cnt), 63);
                if (lane == 0 && cnt) atomicAdd(&n_cand, cnt);
            }
            __syncthreads();
            // ---- the bin of rank k, counted from below: usually within an octave of the bound (groups hold few
            // elements of the set each), which one read of the histogram per wavefront covers
            const uint32_t nc = n_cand;
            const uint32_t c = bin + 1 - lane >= 0 ? hist2[bin + 1 - lane] : 0u;
            const uint32_t low = wave_scan_incl(c);                       // elements in this lane's bin and below
            const unsigned long long mask = __ballot(low > nc - (uint32_t)k);
            if (mask) {                                   // uniform
                const int d = __ffsll((long long)mask) - 1;
                bin = bin + 1 - d;
                before = nc - lane_value(low, d);
            } else {
                pick_bin(hist2, (uint32_t)k, lscan, tmp2, bin, before);
            }
            const uint32_t in_floor = bin_floor(bin - 1) + TK_MARGIN, list_floor = bin_floor(bin) - TK_MARGIN;
            for (int i0 = 0; i0 < items; i0 += TK_NX * TK_THREADS) {
                if (items > TK_NX * TK_THREADS) fetch(i0);
#pragma unroll
                for (int i = 0; i < TK_NX; ++i)
                    if (i0 + i * TK_THREADS < items) {
                        uint32_t in = 0, near = 0;
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            in |= (x[i][e] >= in_floor ? 1u : 0u) << e;
                            near |= (x[i][e] >= list_floor ? 1u : 0u) << e;
                        }
                        append(near & ~in, jp[i]);
                        if (in == 0) continue;
                        if (L <= TK_BITMAP) {
                            atomicOr(&bits[jp[i] >> 5], in << (jp[i] & 31));
                        } else {
                            for (; in; in &= in - 1) {
                                const uint32_t p = atomicAdd(&n_win, 1u);
                                if (p < TK_FILTER_MAX_K) winners[p] = (uint32_t)(jp[i] + __ffs(in) - 1);
                            }
                        }
                    }
            }
        }
        __syncthreads();
        const uint32_t nl = n_list;
        if (!give_up && nl <= TK_LIST) {
            // ---- rank of every listed element (value, then smaller position), 16 threads per element
            for (uint32_t i0 = 0; i0 < nl; i0 += TK_THREADS / 16) {
                const uint32_t i = i0 + (t >> 4);
                const uint2 me = list[i < nl ? i : 0];
                // counted together: the rank (low half) and the listed elements above the bin, which `before` has counted
                uint32_t rank = 0;
                for (uint32_t o = t & 15; o < nl; o += 16) {
                    const uint2 other = list[o];
                    rank += other.x > me.x || (other.x == me.x && other.y < me.y);
                    rank += other.x >= bin_floor(bin - 1) ? 0x10000u : 0u;
                }
                constexpr int ROW_ROR = 0x120;            // rotation inside a row of 16 lanes
                rank += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)rank, ROW_ROR + 1, 0xf, 0xf, true);
                rank += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)rank, ROW_ROR + 2, 0xf, 0xf, true);
                rank += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)rank, ROW_ROR + 4, 0xf, 0xf, true);
                rank += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)rank, ROW_ROR + 8, 0xf, 0xf, true);
                const uint32_t want = (uint32_t)k - before + (rank >> 16);      // how many of the listed elements belong to the set
                rank &= 0xffffu;
                if ((t & 15) == 0 && i < nl) {
                    ltake[i] = rank < want;
                    if (rank + 1 == want) thr_bits = me.x;
                    if (rank == want) next_bits = me.x;
                    if (rank < want && L <= TK_BITMAP) atomicOr(&bits[me.y >> 5], 1u << (me.y & 31));
                }
            }
            __syncthreads();
            // ---- near-ties: the first element left out is within eps of the k-th value
            const float thr_f = __uint_as_float(thr_bits);
            const uint32_t near_lo = __float_as_uint(thr_f * (1.f - rs.eps)), near_hi = __float_as_uint(thr_f * (1.f + rs.eps));
            if (next_bits >= near_lo) {                   // uniform; rare
                if (t == 0) {
                    n_near = 0;
                    n_near_in = 0;
                }
                __syncthreads();
                if (t < (int)nl && list[t].x >= near_lo && list[t].x <= near_hi) {
                    const uint32_t slot = atomicAdd(&n_near, 1u);
                    if (slot < TK_NEAR_MAX) near_slot[slot] = t;
                    if (ltake[t]) atomicAdd(&n_near_in, 1u);
                }
                __syncthreads();
                const uint32_t nn = n_near, nin = n_near_in;
                if (nn <= TK_NEAR_MAX) {                 // more of them (massive ties) keep the fp32 ranking
                    rescore_candidates(rs, h, list, near_slot, (int)nn, near_val, near_acc, near_red);
                    if (t < (int)nn) {                   // rank among the near elements: value, then smaller position
                        const uint32_t me = near_slot[t], j = list[me].y;
                        const float v = near_val[t];
                        uint32_t rank = 0;
                        for (uint32_t c = 0; c < nn; ++c) rank += (near_val[c] > v) || (near_val[c] == v && list[near_slot[c]].y < j);
                        ltake[me] = rank < nin;
                        if (L <= TK_BITMAP) {
                            if (rank < nin) atomicOr(&bits[j >> 5], 1u << (j & 31));
                            else atomicAnd(&bits[j >> 5], ~(1u << (j & 31)));
                        }
                    }
                }
                __syncthreads();
            }
            if (L <= TK_BITMAP) {
                walk_bitmap(bits, (int)L, 0u, tmp2, [&](uint32_t rank, int j) {
                    if (rank < (uint32_t)k) put(rank, j);
                });
                expand();
                return;
            }
            // rows longer than the bitmap: one stretch of positions after the other
            if (t < (int)nl && ltake[t]) {
                const uint32_t p = atomicAdd(&n_win, 1u);
                if (p < TK_FILTER_MAX_K) winners[p] = list[t].y;
            }
            uint32_t done = 0;
            for (long long j0 = 0; j0 < L; j0 += TK_BITMAP) {
                __syncthreads();
                for (int i = t; i < k; i += TK_THREADS) {
                    const long long j = (long long)winners[i] - j0;
                    if (j >= 0 && j < TK_BITMAP) atomicOr(&bits[j >> 5], 1u << (j & 31));
                }
                __syncthreads();
                done += walk_bitmap(bits, TK_BITMAP, done, tmp2, [&](uint32_t rank, int j) {
                    if (rank < (uint32_t)k) out[rank] = (int32_t)(j0 + j);
                });
                __syncthreads();
                for (int i = t; i < k; i += TK_THREADS) {                // leave the bitmap empty
                    const long long j = (long long)winners[i] - j0;
                    if (j >= 0 && j < TK_BITMAP) bits[j >> 5] = 0u;
                }
            }
            return;
        }
        __syncthreads();                                  // the radix route reuses the histogram
    }

    // ---- radix route: threshold = bit pattern of the k-th largest value; want = how many
    // elements equal to it belong to the set (those with the smallest indices) ----
    uint32_t prefix = 0, want = (uint32_t)k;
    radix_step(u, L, 20, 12, prefix, want, hist, tmp, bcast);
    radix_step(u, L, 10, 10, prefix, want, hist, tmp, bcast);
    radix_step(u, L, 0, 10, prefix, want, hist, tmp, bcast);
    const uint32_t thr = prefix;

    // ordered sweep: element j goes to slot (#greater before j) + min(#equal before j, want)
    uint32_t base_gt = 0, base_eq = 0;
    for (long long c0 = 0; c0 < L; c0 += TK_SWEEP) {
        const long long j0 = c0 + (long long)tid_x() * TK_EPT;
        uint32_t x[TK_EPT];
        uint32_t ngt = 0, neq = 0;
#pragma unroll
        for (int i = 0; i < TK_EPT; ++i) {
            x[i] = (j0 + i < L) ? u[j0 + i] : 0u;
            const bool in = j0 + i < L;
            ngt += (in && x[i] > thr) ? 1u : 0u;
            neq += (in && x[i] == thr) ? 1u : 0u;
        }
        uint32_t tot_gt, tot_eq;
        const uint32_t pre_gt = block_scan_incl(ngt, tmp, tot_gt) - ngt + base_gt;
        const uint32_t pre_eq = block_scan_incl(neq, tmp2, tot_eq) - neq + base_eq;
        uint32_t g = pre_gt, e = pre_eq;
#pragma unroll
        for (int i = 0; i < TK_EPT; ++i) {
            if (j0 + i < L) {
                if (x[i] > thr) {
                    put(g + (e < want ? e : want), (int)(j0 + i));
                    ++g;
                } else if (x[i] == thr) {
                    if (e < want) put(g + e, (int)(j0 + i));
                    ++e;
                }
            }
        }
        base_gt += tot_gt;
        base_eq += tot_eq;
    }
    expand();
}

// group_max: [Hkv][ceil(L / kGroupKeys)] maxima of alpha over groups of kGroupKeys consecutive positions
// Can the top-k expand a set of k pages out of L to positions itself?
bool topk_expands(long long L, int k) { return k <= TK_FILTER_MAX_K && L <= TK_BITMAP; }

// page: 1, or the number of consecutive positions every selected element stands for: idx_out is then [Hkv][k * page].
// comb: nullptr, or the arguments of an attention call (head dimension d) whose split partials are merged in the same launch
hipError_t launch_topk(const float *alpha, const float *group_max, int Hkv, long long L, int k, int32_t *idx_out, const RescoreArgs &rs,
                       int page, const KernelArgs *comb, int d, hipStream_t stream)
{
    dim3 grid(Hkv), block(TK_THREADS);
    if (!comb) {
        if (page > 1) hipLaunchKernelGGL((topk_kernel<0, true>), grid, block, 0, stream, alpha, group_max, L, k, idx_out, rs, page, Hkv, KernelArgs{});
        else hipLaunchKernelGGL((topk_kernel<0, false>), grid, block, 0, stream, alpha, group_max, L, k, idx_out, rs, 1, Hkv, KernelArgs{});
        return hipGetLastError();
    }
    const long long rows = (long long)comb->R * Hkv, per = TK_THREADS / 256;
    if ((rows + per - 1) / per + Hkv > 0x7fffffff) return hipErrorInvalidValue;
    grid.x = Hkv + (unsigned)((rows + per - 1) / per);
    if (d == 128) hipLaunchKernelGGL((topk_kernel<128, false>), grid, block, 0, stream, alpha, group_max, L, k, idx_out, rs, 1, Hkv, *comb);
    else if (d == 64) hipLaunchKernelGGL((topk_kernel<64, false>), grid, block, 0, stream, alpha, group_max, L, k, idx_out, rs, 1, Hkv, *comb);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

}  // namespace mage
