// Host side of the matrix kernel (matrix_kernel.h): the weight table, the tiles of a geometry and which split of them to take.
#include <algorithm>
#include <climits>
#include <cmath>
#include <cstring>

#include "internal.h"

namespace sc {

namespace {

constexpr int kMatrixGroups = 8;      // groups of 16 channels a chunk holds at most (eight wavefronts that share them: twice as many)
int waves(int KS) { return std::max(4, KS); }
int most_groups(int KS) { return KS > 4 ? 2 * kMatrixGroups : kMatrixGroups; }
// Bytes where the sums of wavefronts that share the channels meet.
int meeting_bytes(int MK, int NP, int KS) { return KS * MK * NP * 4096; }
constexpr int kMaxLds = 160 * 1024;   // LDS per CU
constexpr int kCUs = 256;

// Place of weight (k, col) in the image, first piece.
size_t image_at(const MatrixWeights& m, int RS, int k, int col)
{
    const int c = col / RS, tap = col % RS;
    const size_t step = (size_t)(c / 16) * RS + tap, lane = (size_t)((c % 16) / 8) * 32 + k % 32;
    return (((size_t)(k / 32) * m.steps + step) * m.pieces) * 512 + lane * 8 + c % 8;
}

// The exponent that puts a row's largest weight in [2^14, 2^15).
int row_exponent(const Csr& csr, int k)
{
    float top = 0.f;
    for (int i = csr.rowptr[k]; i < csr.rowptr[k + 1]; ++i) top = std::max(top, std::fabs(csr.val32[i]));
    int ex = 0;
    if (top > 0.f) (void)std::frexp(top, &ex), ex = 15 - ex;
    return ex;
}

// A weight, scaled, of which two binary16 pieces keep less than 2^-23 of it, or the high one 2^-12 times as large less than
// all its bits.
bool small_weight(float scaled) { return scaled != 0.f && std::fabs(scaled) < 0.25f; }
// Small weights a block of 32 rows may have: the first four are added at no cost that shows, eight more in about 2 us a tile.
// Normally distributed weights have 4 in a block of 147456.
constexpr int kMaxSmall = 32;

// Weights of the rows but zeros, which add no rounding.
std::vector<int> row_weights(const Csr& csr)
{
    std::vector<int> n(csr.K, 0);
    for (int k = 0; k < csr.K; ++k)
        for (int i = csr.rowptr[k]; i < csr.rowptr[k + 1]; ++i) n[k] += csr.val32[i] != 0.f;
    return n;
}

// fp32 rows of few weights are the less exact in two pieces: all of their weights stand in the list, where they are multiplied as
// fp32, each row a sum of its own as in the tile kernel (33 rows of 3 to 54 weights: the tile kernel's error to the digit).  A sum
// of two pieces' products is rounded with every tap, so the two meet at some 35, 65 and 130 weights under 1 x 1, 3 x 3 and 5 x 5
// taps: a layer that has a row below that and not in the list takes the tile kernel.
int short_row(int RS) { return 32 + 4 * RS; }
// Weights of short rows a block of 32 rows may have, at 2.2 us a tile for eight (estimate_matrix counts them).  A layer with more
// has none in the list: one whose rows are mostly short is the tile kernel's.
constexpr int kMaxShort = 160;

// Whether the rows' weights stand in the list, by their numbers.
std::vector<char> listed_rows(const std::vector<int>& n, int RS)
{
    const int K = (int)n.size();
    std::vector<char> listed(K, 0);
    for (int k0 = 0; k0 < K; k0 += 32) {
        int weights = 0;
        for (int k = k0; k < std::min(K, k0 + 32); ++k) {
            if (n[k] > short_row(RS)) continue;
            listed[k] = 1;
            weights += n[k];
        }
        if (weights > kMaxShort) return std::vector<char>(K, 0);
    }
    return listed;
}

// Halves of the image: behind the last stream, the groups of its last chunk that are not there (they meet zeros of the input)
// and what its last steps ask for ahead.
size_t image_halves(int K, int C, int RS, int pieces)
{
    return ((size_t)((K + 31) / 32) * ((C + 15) / 16 * RS) + (size_t)kMatrixGroups * RS + 3) * pieces * 512;
}

}  // namespace

size_t matrix_bytes_at_least(int K, int C, int R, int S, bool split)
{
    return image_halves(K, C, R * S, split ? 2 : 1) * sizeof(uint16_t) + (size_t)K * ((C * R * S + 31) / 32) * sizeof(unsigned);
}

bool matrix_holds(const Csr& csr, bool split)
{
    for (int k0 = 0; k0 < csr.K; k0 += 32) {
        int small = 0;
        for (int k = k0; k < std::min(csr.K, k0 + 32); ++k) {
            for (int i = csr.rowptr[k]; i < csr.rowptr[k + 1]; ++i)
                if (!std::isfinite(csr.val32[i])) return false;
            if (!split) continue;
            const int ex = row_exponent(csr, k);
            for (int i = csr.rowptr[k]; i < csr.rowptr[k + 1]; ++i) small += small_weight(std::ldexp(csr.val32[i], ex));
        }
        if (small > kMaxSmall) return false;
    }
    return true;
}

void pack_matrix_weights(const Csr& csr, int C, int R, int S, bool split, MatrixWeights& m)
{
    const int K = csr.K, RS = R * S;
    m.pieces = split ? 2 : 1;
    m.KF = (K + 31) / 32;
    m.steps = (C + 15) / 16 * RS;
    m.image.assign(image_halves(K, C, RS, m.pieces), 0);
    m.mask_words = (C * RS + 31) / 32;
    m.mask.assign((size_t)K * m.mask_words, 0u);
    m.row_exp.assign((size_t)m.KF * 32, 0);
    m.small_first.assign(split ? (size_t)m.KF + 1 : 0, 0);
    m.slots.assign(split ? (size_t)m.KF * m.kSlots : 0, {-1, 0, 0, 0.f});
    const std::vector<char> listed = split ? listed_rows(row_weights(csr), RS) : std::vector<char>();
    for (int k = 0; k < K; ++k) {
        m.longest = std::max(m.longest, csr.rowptr[k + 1] - csr.rowptr[k]);
        if (split) m.row_exp[k] = row_exponent(csr, k);
        for (int i = csr.rowptr[k]; i < csr.rowptr[k + 1]; ++i) {
            const int col = csr.colidx[i];
            const float w = split ? std::ldexp(csr.val32[i], m.row_exp[k]) : csr.val32[i];
            if (split && (small_weight(w) || (listed[k] && w != 0.f))) {
                const MatrixWeights::Small s{k % 32, col / RS, col % RS, w};
                MatrixWeights::Small *slot = &m.slots[(size_t)(k / 32) * m.kSlots], *end = slot + m.kSlots;
                while (slot < end && slot->row >= 0) ++slot;
                if (slot < end) {
                    *slot = s;
                } else {
                    m.small.push_back(s);
                    ++m.small_first[k / 32 + 1];
                }
                continue;
            }
            m.mask[(size_t)k * m.mask_words + col / 32] |= 1u << (col % 32);
            uint16_t* to = &m.image[image_at(m, RS, k, col)];
            to[0] = float_to_half_rne(w);
            if (split) to[512] = float_to_half_rne(w - half_to_float(to[0]));
        }
    }
    for (int b = 0; split && b < m.KF; ++b) m.small_first[b + 1] += m.small_first[b];
}

int check_matrix(const Csr& csr, int C, int R, int S, const MatrixWeights& m)
{
    const int RS = R * S;
    if (m.KF != (csr.K + 31) / 32 || m.steps != (C + 15) / 16 * RS || m.mask_words != (C * RS + 31) / 32) return 10;
    if (m.image.size() != image_halves(csr.K, C, RS, m.pieces)) return 10;
    // 11: every stored weight is in its place; 12: and nothing else is in the table or the mask
    size_t marked = 0, small = 0, listed = m.small.size();
    for (const auto& s : m.slots) listed += s.row >= 0;
    std::vector<int> used(m.KF, 0);
    std::vector<uint16_t> rest = m.image;
    const std::vector<char> in_list = m.pieces == 2 ? listed_rows(row_weights(csr), RS) : std::vector<char>();
    for (int k = 0; k < csr.K; ++k)
        for (int i = csr.rowptr[k]; i < csr.rowptr[k + 1]; ++i) {
            const int col = csr.colidx[i];
            const size_t at = image_at(m, RS, k, col);
            const float scaled = std::ldexp(csr.val32[i], m.pieces == 2 ? m.row_exp[k] : 0);
            // 13: every small weight and those of short rows are in a slot or in their block's part of the list
            if (m.pieces == 2 && (small_weight(scaled) || (in_list[k] && scaled != 0.f))) {
                const int n = used[k / 32]++, at = m.small_first[k / 32] + n - m.kSlots;
                if (n >= m.kSlots && at >= m.small_first[k / 32 + 1]) return 13;
                const MatrixWeights::Small& s = n < m.kSlots ? m.slots[(size_t)(k / 32) * m.kSlots + n] : m.small[at];
                ++small;
                if (s.row != k % 32 || s.c * RS + s.tap != col || s.weight != scaled) return 13;
                continue;
            }
            if (!(m.mask[(size_t)k * m.mask_words + col / 32] >> (col % 32) & 1u)) return 11;
            const float is = half_to_float(m.image[at]) + (m.pieces == 2 ? half_to_float(m.image[at + 512]) : 0.f);
            // two pieces: 22 bits and a sign
            if (!(std::fabs(is - scaled) <= (m.pieces == 2 ? std::fabs(scaled) * 0x1p-23f : 0.f))) return 11;
            rest[at] = 0;
            if (m.pieces == 2) rest[at + 512] = 0;
        }
    for (uint16_t h : rest)
        if (h) return 12;
    for (unsigned w : m.mask) marked += (size_t)__builtin_popcount(w);
    return marked + small == csr.colidx.size() && small == listed ? 0 : 12;
}

// fp32: the blocks' first small weights, the images' windows, a bit per lattice element
int matrix_extra_lds(const MatrixPlan& p)
{
    return p.MK * p.WK * MatrixWeights::kSlots * (int)sizeof(MatrixWeights::Small) + p.images * kImageWindowBytes + p.EB * 8;
}

// What the wavefronts' rows of outputs take on their way to memory.
int out_runs_lds(const MatrixPlan& p, int elem_bytes) { return 4 * 32 * ((p.KS > 1 ? 1 : p.NP) * 32 * elem_bytes + 16); }

// Whether the kernel stages runs.  Where a wavefront has but one block of single
// pixels to stage (binary16: two), runs would leave wavefronts without one: of 506 splits of 27 layers those with one are 2 to
// 4 % slower with runs in the mean, up to 24 % (64 -> 256, 56 x 56, binary16: 65 -> 80 us); with two (three) and more, 6 to 40 %
// faster, two in a hundred of them slower, by 5 % at most.
bool stages_runs(const MatrixPlan& p, int elem_bytes) { return p.quads && p.fly > (elem_bytes == 4 ? 1 : 2); }

// Whether planes that are not whole runs are staged in runs, the last of a plane overlapping the one before it; `blocks`: of single
// pixels, a wavefront and chunk.  Every split of 1693 layers with such planes timed both ways, those within 30 % of their layer's best:
// binary16 4463 that stage runs by this rule, 0.87 of the time in the mean, two slower by 3 % (173 -> 354 channels, 25 x 25: 17.2 ->
// 13.8 us); fp32 904, 0.89, none slower by 3 %.  With four blocks or fewer under 1 x 1 taps half of binary16 splits lose, up to 37 %, and three
// quarters of fp32 ones, up to 59 %; under larger taps fp32 would gain 7 %, but one in 23 loses 3 to 11 %.
// (`late`: binary16 variants of 2 x 4 fragments have one block of runs in flight and six of single pixels.  Where that is all of the single
// pixels and not all of the runs, and the layer's tensors exceed the 256 MB of the last cache, 16 of 40 splits lose 3 to 9 % by runs and the
// mean 1 %; below 256 MB 166 gain 4 %.)
// (Fewer than 16 channels, a network's first layers: 83 that take the matrix kernel anyway gain 10 %, but by its lower estimate 11 others leave
// the tile kernel for it, six of which lose 6 to 43 %: 1 -> 217, 207 x 207, batch 8: 44.4 and 63.4 us.)
bool ragged_runs(int C, int RS, int blocks, bool late, long long bytes, int elem_bytes)
{
    if (C < 16 || (late && blocks <= 6 && bytes > 256ll << 20)) return false;
    return blocks > (RS == 1 || elem_bytes == 4 ? 4 : 2);
}

bool plan_matrix(int K, int C, int R, int S, int elem_bytes, const Geometry& g, bool pool, int MK, int NP, int WK, int KS,
                 int CG, MatrixPlan& p)
{
    p = MatrixPlan{};
    p.MK = MK; p.NP = NP; p.WK = WK; p.KS = KS; p.WP = waves(KS) / (WK * KS);
    p.E = (g.H + 2 * g.pad - R) / g.stride + 1;
    p.F = (g.W + 2 * g.pad - S) / g.stride + 1;
    const long long EF = (long long)p.E * p.F, nout = g.N * EF;
    p.PT = 32 * NP * p.WP;
    // 2 x 2 maximum in the store step: a wavefront's outputs hold whole pairs of rows, a pair in 2, 4 ... 32 lanes of one
    // fragment or in the same lanes of fragments 1 or 2 apart
    if (pool) {
        if (((p.E | p.F) & 1) || (p.F & (p.F - 1)) || g.stride != 1) return false;
        if ((KS == 1 ? 32 * NP : 32) % (2 * p.F) != 0 || p.F > 64) return false;
    }
    p.Wp = std::max(g.W + g.pad, (p.F - 1) * g.stride + 1);
    p.Hs = std::max(g.H + g.pad, (p.E - 1) * g.stride + 1);
    if (nout >= (1ll << 31) - 4096 || (long long)g.N * p.Hs * p.Wp + (long long)(R + 1) * p.Wp + 4096 >= (1ll << 31)) return false;
    p.nout = (int)nout;
    p.ntiles = (int)((nout + p.PT - 1) / p.PT);
    // the lattice elements a tile spans depend only on its first output's place in its image, which repeats after
    // EF / gcd(PT, EF) tiles
    long long gcd = EF;
    for (long long r = p.PT % EF; r;) { const long long t = gcd % r; gcd = r; r = t; }
    auto lattice = [&](long long o) { return (o / EF * p.Hs + o % EF / p.F * g.stride) * (long long)p.Wp + o % p.F * g.stride; };
    // The runs of pixels before a lattice element, images one behind the other: those a tile needs are consecutive.
    const int px = 8 / elem_bytes;
    const long long plane = (long long)g.H * g.W, plane_quads = (plane + px - 1) / px;
    auto runs_before = [&](long long L, int begun) {       // begun: px - 1 to count one that it is in the middle of
        const long long Y = L / p.Wp, u = Y / p.Hs, y = Y % p.Hs - g.pad, x = L % p.Wp - g.pad;
        const long long before = y < 0 ? 0 : y >= g.H ? plane : y * g.W + std::min<long long>(std::max<long long>(x, 0), g.W);
        return u * plane_quads + (before + begun) / px;
    };
    long long span = 0, quads = 0;
    for (long long t = 0; t < std::min<long long>(p.ntiles, EF / gcd); ++t) {
        const long long a = t * p.PT, b = std::min<long long>(nout, a + p.PT) - 1;
        span = std::max(span, lattice(b) - lattice(a));
        quads = std::max(quads, runs_before(lattice(b) + (long long)(R - 1) * p.Wp + S, px - 1) - runs_before(lattice(a), 0));
    }
    const long long elems = span + (long long)(R - 1) * p.Wp + S;
    if (elems > kMaxLds / 16) return false;
    p.EB = (int)((elems + 63) / 64);
    // source offsets are 31-bit byte offsets from the tile's first image
    const long long images = ((long long)p.EB * 64 / p.Wp + 1) / p.Hs + 2;
    p.images = (int)images;
    if (images * C * g.H * g.W * elem_bytes >= (1ll << 31)) return false;
    if (CG / 2 > most_groups(KS) || CG / 2 % KS) return false;
    // Eight wavefronts: above 64 channels, and where there are more than 32 outputs.  (With 64 channels or fewer half of the wavefronts and
    // more have none to multiply: 163 layers of 33 to 64 channels that would take it, of 6 to 12 us, gain 5 % in the mean, where those above
    // gain 20, and 11 of them lose 3 to 24 %.  Launches of 32 outputs or fewer are bound by their issue where their sums are short: 17 of 276 that
    // would take it, of 6 to 10 us, lose 3 to 13 %; where they are long they would halve, 941 -> 621, 3 x 3, one output: 31.7 and 13.5 us.)
    if (KS > 4 && (C <= 64 || nout <= 32)) return false;
    p.CG = CG;
    const int own = CG / 2 / KS * R * S;
    if (own % 3 && own % 2) return false;           // the kernel walks a chunk two or three steps at a time
    const int pieces = elem_bytes == 4 ? 2 : 1, groups = 2 * ((C + 15) / 16);
    p.nchunks = (groups + CG - 1) / CG;
    // (two binary16 pieces: three steps of weights ahead are more registers than there are, unless it has to be three)
    p.ahead = own % 3 == 0 && !(pieces == 2 && own % 2 == 0) ? 3 : 2;
    const int unit = pieces == 2 ? 1 : 2, blocks = (CG * p.EB + waves(KS) - 1) / waves(KS);   // a chunk's staging blocks of a wavefront
    p.fly = blocks <= unit ? unit : blocks < 3 * unit ? 2 * unit : 3 * unit;
    p.odd_planes = plane % px != 0;
    p.wide_fly = 1;
    if (g.W >= 2 && quads > 0) {
        const long long run_blocks = (CG * quads + 64 * waves(KS) - 1) / (64 * waves(KS));
        const int wide_fly = run_blocks > 1 && MK * NP * pieces < 8 ? 2 : 1;
        const bool late = pieces == 1 && MK * NP == 8 && run_blocks > wide_fly;
        const long long bytes = g.N * (C * plane + K * EF / (pool ? 4 : 1)) * elem_bytes;
        if (!p.odd_planes || (plane > px && ragged_runs(C, R * S, blocks, late, bytes, elem_bytes))) {
            p.quads = (int)quads;
            p.wide_fly = wide_fly;
        }
    }
    long long lds = (long long)(p.nchunks > 1 ? 2 : 1) * CG * p.EB * 64 * 16 * pieces;
    if (KS > 1) lds = std::max(lds, (long long)meeting_bytes(MK, NP, KS));   // where the sums of a pair meet
    // outputs in runs, where a plane is whole ones: 32 rows of a wavefront's outputs at a time go through LDS (pooled: rows of
    // four at least, whose windows begin at whole words)
    const long long plane_bytes = (pool ? EF / 4 : EF) * elem_bytes;
    p.out_runs = (pool && p.F < 4) || plane_bytes % 8 ? 0 : plane_bytes % 16 ? 8 : 16;
    if (p.out_runs) lds = std::max(lds, (long long)out_runs_lds(p, elem_bytes));
    lds += 64 + 8 * 32 * MK * WK;             // what the wavefronts tell each other, bias and scale of the rows
    if (pieces == 2) lds += matrix_extra_lds(p);
    if (lds > kMaxLds) return false;
    p.lds_bytes = (int)lds;
    p.kblocks = (K + 32 * MK * WK - 1) / (32 * MK * WK);
    const long long grid = ((long long)p.ntiles * p.kblocks + 7) / 8 * 8;   // a multiple of the XCD count
    if (grid > INT_MAX - 8) return false;
    p.grid = (int)grid;
    return true;
}

int matrix_resident(int MK, int NP, int KS, int ahead, int fly, int runs, bool split)
{
    const int unit = split ? 1 : 2, pieces = split ? 2 : 1;
    // eight wavefronts are two a SIMD: 71 to 80 registers hold three such workgroups, 86 to 128 two, 133 one
    if (KS > 4) {
        if (MK * NP == 1) return runs == 1 || (!runs && fly == unit) ? 3 : 2;
        return !runs && ahead == 3 && fly == 3 * unit ? 1 : 2;
    }
    // four are one: two, three of the small variants (fp32 with three steps of weights ahead and two blocks in flight: 169 registers, two),
    // four of the smallest
    if (MK * NP * pieces > 4) return 2;
    if (runs) return split && runs == 2 ? 2 : 3;
    if (!split && ahead == 2 && fly == unit && KS == 1) return 4;
    return fly == 3 * unit || (split && ahead == 3 && fly == 2) ? 2 : 3;
}

namespace {

// Rough time of one launch in microseconds.  Structure and constants are fitted to the measured times of every split (3278 of
// them) of 186 layers (the 32-pixel VGG-16's, those of larger networks, and random ones: 1 x 1, 1-D, 3 x 3, 5 x 5, stride 2,
// batches of 1 to 256): 10 % rms of the logarithm, the cheapest by estimate 2 % slower than the fastest measured in the mean.
// (The fit is from before outputs left in runs, which it does not price: it is high where stores bound a layer, most for wide 1 x 1 layers in
// binary16, of which 64 -> 256, 56 x 56 takes two thirds of what it did.)  In clocks of 2.1 GHz:
//  * A step costs its matrix instructions (39 to 41 clocks each over the workgroups resident on the CU; 32 at the nominal rate)
//    and its reads, but never less than a wavefront's own chain of loads and instructions.
//  * A chunk's staging blocks cost 59 to 299 clocks each by kind (single pixels or runs, half or two pieces); multiplying and
//    staging hide each other little.  What a wavefront does not have in flight costs most of a memory latency a block.
//  * Workgroups run in rounds of what is resident.
// (A launch of few products is mostly the fixed part: 51 fp32 and 44 binary16 layers of fewer than 4e8, zeros counted, are
// within 2.4 and 1.4 % of their fastest split in the mean as well.)
//  * Eight wavefronts that share the channels have constants of their own: 864 splits of 429 layers, 9 % rms beside the 1.06 of their
//    time that the others' estimate has on those layers.  By it the fastest split of all is missed by 2.4 % in the mean; what was
//    taken without them by 16 %.  (Of 296 others that take them the mean is 20 % faster than by four, one is slower, by 16 %.  In more
//    than two rounds of workgroups only rows of 32 channels or fewer take them: seven of 126 such layers, six 3 to 25 % faster, one
//    8 % slower, as 127 -> 29, 54 x 54, batch 45, is: 31.0 -> 33.4 us.)
//  * Weights in the list (but for a block's first ones) take 4700 clocks for eight, in a wavefront's own chain: `listed`.
double estimate_matrix(const MatrixPlan& p, int RS, bool split, double listed, double lone = 1.0)
{
    struct Clocks { double fixed, chain, chain_mf, mf, read, chunk, stage_chunk, stage, run_chunk, run, both, late, pair, tail; };
    static const Clocks k16 = {11300, 172, 17.2, 40.9, 9.2, 482, 13, 58.5, 2, 197, 1.24, 659, 993, 1.0},
                        k32 = {11800, 7, 49.0, 38.9, 1.5, 306, 45, 139, 6, 290, 1.19, 676, 2110, 1.09},
                        k16_8 = {7190, 230, 0, 28, 0, 1100, 0, 56.4, 0, 190, 1.77, 0, 4700, 1.05};
    const Clocks& k = split ? k32 : p.KS > 4 ? k16_8 : k16;
    const int pieces = split ? 2 : 1;
    const bool runs = stages_runs(p, split ? 4 : 2);
    const int blocks = runs ? (p.CG * p.quads + 63) / 64 : p.CG * p.EB, fly = runs ? p.wide_fly : p.fly;
    const int conc_max = std::min(matrix_resident(p.MK, p.NP, p.KS, p.ahead, p.fly, runs ? p.wide_fly : 0, split), kMaxLds / p.lds_bytes);
    const double mf = p.MK * p.NP * (split ? 3 : 1), own = (double)(p.CG / 2 / p.KS) * RS;
    const double late = std::max(0, (blocks + waves(p.KS) - 1) / waves(p.KS) - fly) * k.late, begin = runs ? k.run_chunk : k.stage_chunk;
    const double pair = p.KS > 4 && !p.out_runs ? 1.35 * k.pair : k.pair;
    auto round = [&](double conc) {
        const double multiply = own * std::max(k.chain + k.chain_mf * mf, conc * waves(p.KS) / 4 * (mf * k.mf + p.NP * pieces * k.read));
        const double stage = conc * blocks * (runs ? k.run : k.stage);
        return p.nchunks * (std::max(multiply, stage + begin) + k.both * std::min(multiply, stage) + k.chunk + late) + 0.6 * stage + begin +
               conc * pair * p.MK * p.NP / (p.KS > 1 ? 4 : 1) + listed;
    };
    const long long slots = (long long)kCUs * conc_max, wgs = (long long)p.ntiles * p.kblocks;
    const long long full = wgs / slots, rest = wgs % slots;
    double t = k.fixed + (double)full * round(conc_max) * lone;
    if (rest) t += round((double)((rest + kCUs - 1) / kCUs)) * (full ? k.tail * lone : 1.0);
    return t / 2100.0;
}

// Splits whose wavefronts share the tile out are ranked with a full round of a launch taking so much longer than the estimate says.  Runs of
// odd planes start off a word, and where few workgroups of a CU hide their loads from one another the estimate, fitted to whole planes, is
// low: of 1142 binary16 layers with such planes 16 are 3 to 9 % slower with this than by the split that was taken when odd planes were
// staged pixel by pixel, the mean is 13 % faster; without, 26, by up to 20 % (301 -> 45, 71 x 71, batch 158: 296 us by single pixels, 354
// and, with this, 319).  In fp32 (150 layers, 12 % faster in the mean, 15 3 to 20 % slower) it picks wrong as often as right, and so it does
// beside splits whose wavefronts share the channels (102 -> 24, 47 x 47, stride 2, batch 246: 53.7 and 68.0 us).  There and beside the tile
// kernel, which was compared with the estimate as it is, it does not count.
double lone_rounds(const MatrixPlan& p, bool split)
{
    if (split || p.KS > 1 || !p.odd_planes || !stages_runs(p, 2)) return 1.0;
    const int resident = std::min(matrix_resident(p.MK, p.NP, p.KS, p.ahead, p.fly, p.wide_fly, split), kMaxLds / p.lds_bytes);
    return resident == 1 ? 1.25 : resident == 2 && p.MK * p.NP == 4 ? 1.1 : 1.0;
}

}  // namespace

namespace {

// The splits an automatic choice looks at: MK, NP, WK, KS.
constexpr int kShapes16[][4] = {{2, 4, 1, 1}, {2, 4, 2, 1}, {2, 4, 4, 1}, {2, 2, 1, 1}, {2, 2, 2, 1}, {2, 2, 4, 1}, {2, 2, 1, 4}, {1, 2, 1, 8}, {1, 1, 1, 8}};
constexpr int kShapes32[][4] = {{2, 2, 1, 1}, {2, 2, 2, 1}, {2, 2, 4, 1}, {1, 2, 1, 1}, {1, 2, 2, 1}, {1, 2, 4, 1}, {2, 2, 1, 4}};
struct Shapes {
    const int (*first)[4], (*last)[4];
    const int (*begin() const)[4] { return first; }
    const int (*end() const)[4] { return last; }
};
Shapes shapes(bool split)
{
    return split ? Shapes{std::begin(kShapes32), std::end(kShapes32)} : Shapes{std::begin(kShapes16), std::end(kShapes16)};
}

int check_matrix_plan(int K, int C, int R, int S, int elem_bytes, const Geometry& g, bool pool, const MatrixPlan& p)
{
    const int pieces = elem_bytes == 4 ? 2 : 1, RS = R * S, own = p.CG / 2 / p.KS * RS;
    // 14: the channels are covered, the steps come out, the table holds what the last block asks for (last steps' weights ahead)
    // (eight wavefronts: one whose groups are past the last starts right behind it)
    const long long steps = (C + 15) / 16 * RS, last = (p.KS > 4 ? steps + own : (long long)p.nchunks * (p.CG / 2) * RS) + p.ahead;
    if ((long long)p.nchunks * p.CG * 8 < C || own % p.ahead || p.CG / 2 % p.KS) return 14;
    if (((long long)(K + 31) / 32 - 1) * steps + last > (long long)image_halves(K, C, RS, 1) / 512) return 14;
    // 15: LDS holds the buffers (and the sums that meet there) and what lies behind them; every block of rows and outputs is there
    const long long buffers = (long long)(p.nchunks > 1 ? 2 : 1) * p.CG * p.EB * 1024 * pieces, rows = 32ll * p.MK * p.WK;
    const long long behind = 64 + 8 * rows + (pieces == 2 ? matrix_extra_lds(p) : 0);
    if (p.lds_bytes > kMaxLds || buffers + behind > p.lds_bytes || (p.KS > 1 && meeting_bytes(p.MK, p.NP, p.KS) + behind > p.lds_bytes)) return 15;
    if (p.out_runs && (out_runs_lds(p, elem_bytes) + behind > p.lds_bytes || (long long)p.E * p.F / (pool ? 4 : 1) * elem_bytes % p.out_runs)) return 15;
    if (p.kblocks * rows < K || (long long)p.ntiles * p.PT < p.nout || p.WK * p.WP * p.KS != waves(p.KS) || p.PT != 32 * p.NP * p.WP) return 15;
    if (p.grid % 8 || p.grid < (long long)p.ntiles * p.kblocks) return 15;
    // 17: (wide staging) the tile's runs of pixels hold every input that its taps read
    const int px = 8 / elem_bytes, plane = g.H * g.W, run = (plane + px - 1) / px;
    if (p.quads && (plane < px || g.W < 2)) return 17;
    // 16: each tap of each output of a tile is inside the tile, at the element of its input or at one that reads as zero
    const int EF = p.E * p.F, look = std::min(p.ntiles, 48);
    auto lattice = [&](int o) { return (o / EF * p.Hs + o % EF / p.F * g.stride) * p.Wp + o % p.F * g.stride; };
    for (int t = 0; t < look; ++t) {
        const int tile = t == look - 1 ? p.ntiles - 1 : t, o0 = tile * p.PT, q0 = lattice(o0), u0 = o0 / EF;
        if ((q0 + p.EB * 64 - 1) / p.Wp / p.Hs - u0 >= p.images) return 16;
        const int Y0 = q0 / p.Wp % p.Hs - g.pad, X0 = q0 % p.Wp - g.pad;      // as the kernel finds the first run
        const int first = p.quads ? u0 * run + (Y0 < 0 ? 0 : std::min(Y0 * g.W + std::min(std::max(X0, 0), g.W), plane)) / px : 0;
        for (int o = o0; o < std::min(p.nout, o0 + p.PT); ++o)
            for (int r = 0; r < R; ++r)
                for (int s = 0; s < S; ++s) {
                    const int L = lattice(o) + r * p.Wp + s, Y = L / p.Wp, X = L % p.Wp - g.pad, u = Y / p.Hs, y = Y % p.Hs - g.pad;
                    const int yy = o % EF / p.F * g.stride + r - g.pad, xx = o % p.F * g.stride + s - g.pad;
                    if (L - q0 >= p.EB * 64) return 16;
                    const bool reads = u < g.N && y >= 0 && y < g.H && X >= 0 && X < g.W;
                    const bool wants = yy >= 0 && yy < g.H && xx >= 0 && xx < g.W;
                    if (reads != wants || (wants && (u != o / EF || y != yy || X != xx))) return 16;
                    const int quad = p.quads && wants ? u * run + (y * g.W + X) / px - first : 0;
                    if (quad < 0 || (p.quads && quad >= p.quads)) return 17;
                }
    }
    return 0;
}

}  // namespace

int check_matrix_plans(int K, int C, int R, int S, int elem_bytes, const Geometry& g, bool pool)
{
    for (const auto& sh : shapes(elem_bytes == 4))
        for (int CG = 2; CG <= 2 * most_groups(sh[3]); CG *= 2) {
            MatrixPlan p;
            if (!plan_matrix(K, C, R, S, elem_bytes, g, pool, sh[0], sh[1], sh[2], sh[3], CG, p)) continue;
            const int bad = check_matrix_plan(K, C, R, S, elem_bytes, g, pool, p);
            if (bad) return bad;
        }
    return 0;
}

bool choose_matrix(const Csr& csr, int C, int R, int S, int elem_bytes, const Geometry& g, bool pool, int tile_parts,
                   MatrixPlan& best, double* us)
{
    const bool split = elem_bytes == 4;
    const int RS = R * S;
    const int E = (g.H + 2 * g.pad - R) / g.stride + 1, F = (g.W + 2 * g.pad - S) / g.stride + 1;
    // fp32 sums: the share of an output's terms that do not fall on padding, and the terms, both in the mean
    double inside = 0.0, terms = 0.0;
    std::vector<int> before;       // [K][C + 1]: a row's weights (but zeros, which add no rounding) before a channel
    int shortest = INT_MAX;        // weights of the shortest row that has any, but for those in the list
    std::vector<char> in_list;     // [K]
    bool lists = false;            // it has rows with weights
    std::vector<int> trips;        // [blocks of 32 rows]: turns of eight weights in the list, behind the first ones
    if (split) {
        double rows = 0, cols = 0;
        for (int i = 0; i < E; ++i)
            for (int r = 0; r < R; ++r) rows += (unsigned)(i * g.stride + r - g.pad) < (unsigned)g.H;
        for (int j = 0; j < F; ++j)
            for (int s = 0; s < S; ++s) cols += (unsigned)(j * g.stride + s - g.pad) < (unsigned)g.W;
        inside = rows * cols / ((double)E * F * RS);
        terms = (double)csr.colidx.size() / csr.K * inside;
        const std::vector<int> weights = row_weights(csr);
        in_list = listed_rows(weights, RS);
        for (int k = 0; k < csr.K; ++k) {
            if (k % 32 == 0) trips.push_back(0);
            const int n = weights[k];
            if (in_list[k]) trips.back() += n, lists |= n > 0;
            else if (n) shortest = std::min(shortest, n);
        }
        for (int& t : trips) t = (std::max(0, t - MatrixWeights::kSlots) + 7) / 8;
    }
    const int parts = std::max(1, tile_parts);
    // Terms that a term of row k is summed with, in the mean, itself included, where every `width` channels have a sum.
    auto company = [&](int k, int width) {
        const int* n = &before[(size_t)k * (C + 1)];
        double squares = 0.0;
        for (int c = 0; c < C; c += width) {
            const double here = n[std::min(C, c + width)] - n[c];
            squares += here * here;
        }
        return squares / n[C] * inside;
    };
    // Whether no row is less exact under the split than in the tile kernel.  Units and numbers as below, but a row of few weights
    // has no term in some steps and chunks: then the pieces' own error is most of it (10 terms: 9e-8 to 1.0e-7, the tile kernel
    // 5e-8 to 6e-8).  Those in the list aside, 5026 rows of 36 layers that pass have 0.99 of the tile kernel's error or less,
    // 0.43 in the mean.
    auto rows_as_exact = [&](const MatrixPlan& p, double steps) {
        if (0.81 + 0.047 * 3 * steps + 0.04 * p.nchunks <= 0.0335 * shortest * inside / parts) return true;   // the least they can be
        if (before.empty()) {
            before.assign((size_t)csr.K * (C + 1), 0);
            for (int k = 0; k < csr.K; ++k) {
                int* n = &before[(size_t)k * (C + 1)];
                for (int i = csr.rowptr[k]; i < csr.rowptr[k + 1]; ++i) n[csr.colidx[i] / RS + 1] += csr.val32[i] != 0.f;
                for (int c = 0; c < C; ++c) n[c + 1] += n[c];
            }
        }
        const int own = p.CG / 2 / p.KS * 16, part = (C + parts - 1) / parts;
        for (int k = 0; k < csr.K; ++k) {
            const int n = before[(size_t)(k + 1) * (C + 1) - 1];
            if (!n || in_list[k]) continue;
            const double met = steps * (1.0 - std::exp(-company(k, own) / steps)), chunks = p.nchunks * (1.0 - std::exp(-n * inside / p.nchunks));
            if (0.81 + 0.047 * 3 * met + 0.04 * chunks > 0.0335 * company(k, part)) return false;
        }
        return true;
    };
    // (a row in the list is one sum of its terms, as in the tile kernel where that does not deal the channels over parts)
    if (lists && parts > 1) return false;
    struct Choice {
        double rank = -1.0, us = 0.0;
        MatrixPlan plan{};
    } choices[2];                  // the wavefronts share the tile out, or the channels
    double cheapest = -1.0;        // of all, by the estimate as it is
    for (const auto& sh : shapes(split))
        for (int CG = 2; CG <= 2 * most_groups(sh[3]); CG *= 2) {
            MatrixPlan p;
            if (CG > 2 && CG / 2 >= 2 * ((C + 15) / 16)) break;   // a smaller chunk holds them all (eight wavefronts': 128 of more than 64 channels)
            if (!plan_matrix(csr.K, C, R, S, elem_bytes, g, pool, sh[0], sh[1], sh[2], sh[3], CG, p)) continue;
            if (split) {
                // Squared relative error of an output, in units of 1e-14, fitted to the measured ones: the tile kernel rounds
                // its sum at every term (1.8e-7 at 100); here the pieces' own error, three roundings a step of a chunk's
                // sum, one a chunk.  What is as exact by this measure, with 15 % to spare, may run.
                const double steps = RS * (CG / 2.0 / sh[3]);
                if ((0.81 + 0.047 * 3 * steps + 0.04 * p.nchunks) * 1.3 > 0.0335 * terms / parts) continue;
            }
            int turns = 0;                 // of the wavefront with most of the list
            for (int b = 0; b < (int)trips.size(); b += sh[0]) {
                int mine = 0;
                for (int q = b; q < std::min((int)trips.size(), b + sh[0]); ++q) mine += trips[q];
                turns = std::max(turns, mine);
            }
            const double t = estimate_matrix(p, RS, split, 4700.0 * turns), rank = estimate_matrix(p, RS, split, 4700.0 * turns, lone_rounds(p, split));
            Choice& of_kind = choices[p.KS > 1];
            const bool first = of_kind.rank < 0 || rank < of_kind.rank;
            if ((first || t < cheapest) && (!split || rows_as_exact(p, RS * (CG / 2.0 / sh[3])))) {
                if (first) of_kind = {rank, t, p};
                cheapest = cheapest < 0 ? t : std::min(cheapest, t);
            }
        }
    const Choice& choice = choices[choices[0].rank < 0 || (choices[1].rank >= 0 && choices[1].us < choices[0].us)];
    if (choice.rank < 0) return false;
    best = choice.plan;
    *us = cheapest;
    return true;
}

// binary16: taken where it is estimated 0.7 us faster.  Of 504 layers of every size timed in turn, four that take it so are 4 to
// 8 % slower, and the mean loses 2.2 % to the better kernel of each.  (The 0.7 us are for launches of 8 to 10 us, most of which
// both kernels have alike: without, 16 are slower, by up to 20 %.  Below 0.95 of the tile kernel's estimate instead: six, by up
// to 14 %, the mean loses 2.3 %, and VGG-16's last layer takes 26 us by the tile kernel for 18.7.  Of 95 others whose kernel
// or split this and the one estimate for all sizes changed, the mean is 13 % faster, and three of 8 to 9 us are 8 to 21 % slower.)
// fp32: taken below 0.85 of the cheapest tile launch by the estimate for kernels by rows.  Of 71 layers, timed over blocks of a tenth of a
// second, which heat the chip as a pass does, all below gain 6 % or more; between 0.85 and 0.9 lie 256 -> 256, 14 x 14, batch 256 at 90 %
// (169 us; tile kernel 167 then, 153 since its rows share a stream) and its like.  (Of 36 others with ragged rows, all below, two are
// slower, by 1 and 8 %; the mean takes 0.53 of the tile kernel's time.)  Not below all of the estimate that tile launches are chosen by (estimate_f32): of 113 drawn layers that
// it adds, 25 are 3 to 31 % slower by the matrix kernel, and its products hold 21 bits where the tile kernel's hold 24: with inputs that
// went through a ReLU, whose sums cancel less, 13 of 48 are less exact by it, up to 1.15 of the tile kernel's error against 64 bits.
bool matrix_pays(double us, double tile_us, bool split) { return us < (split ? 0.85 * tile_us : tile_us - 0.7); }

void fill_matrix_args(const MatrixWeights& m, const MatrixPlan& p, int K, int C, int R, int S, const Geometry& g, MatrixArgs& a)
{
    a.N = g.N; a.C = C; a.H = g.H; a.W = g.W; a.K = K; a.E = p.E; a.F = p.F; a.EF = p.E * p.F;
    a.stride = g.stride; a.pad = g.pad; a.R = R; a.S = S; a.RS = R * S;
    a.Wp = p.Wp; a.Hs = p.Hs;
    a.PT = p.PT; a.nout = p.nout; a.ntiles = p.ntiles; a.kblocks = p.kblocks;
    a.WK = p.WK;
    a.logWK = p.WK == 4 ? 2 : p.WK == 2 ? 1 : 0;
    a.mask_words = m.mask_words;
    a.meet_at = p.lds_bytes - 64 - 8 * 32 * p.MK * p.WK - (m.pieces == 2 ? matrix_extra_lds(p) : 0);
    a.images = p.images;
    a.longest = m.longest;
    a.CG = p.CG; a.EB = p.EB; a.nchunks = p.nchunks;
    a.own_groups = p.CG / 2 / p.KS;
    a.own_steps = a.own_groups * a.RS;
    a.stream_steps = m.steps; a.KF = m.KF;
    a.block_major = m.image.size() * 2 > (size_t)g.N * C * g.H * g.W * (m.pieces == 2 ? 4 : 2);
    a.fd_EF = make_fastdiv(a.EF);
    a.fd_F = make_fastdiv(p.F);
    a.fd_Wp = make_fastdiv(p.Wp);
    a.fd_Hs = make_fastdiv(p.Hs);
    a.fd_EB = make_fastdiv(p.EB);
    const int px = m.pieces == 2 ? 2 : 4;
    a.groups = (C + 15) / 16;
    a.quads = p.quads;
    a.last_run = g.H * g.W - px;
    a.padded = p.Wp != g.W || p.Hs != g.H;
    a.plane_quads = (g.H * g.W + px - 1) / px;
    a.fd_W = make_fastdiv(g.W);
    a.fd_quads = make_fastdiv(std::max(1, a.quads));
    a.fd_plane_quads = make_fastdiv(std::max(1, a.plane_quads));
}

}  // namespace sc
