// Legendre contractions whose recursion feeds the matrix cores from registers
// (HIP, gfx950).  Same operands, layouts and sums as k_leg.hip (all of E and B).
//
// An MFMA's 16 rows and 4 K slots need not be neighbours in l or in theta: a wave's
// lane (i = lane & 15, k = lane >> 4) runs the recursion of one ring over one run of
// l, and its current value is the A operand of that row and K slot as it stands.
//  * map2alm: row i is an 8-row segment of l, slot k a ring; step t of the recursion
//    contracts row t of 16 segments against 4 rings, into accumulator t.
//  * alm2map: row i is a ring, slot k a quarter of the l range; each lane follows one
//    long chain from a single seed pair, so no seed table is read on the way.
// No LDS tile, no barrier, and every wave works alone on its column tiles, so a
// batch is padded to 4 map sets (spin 2) or 8 (spin 0) instead of 32, small batches
// fill the chip with independent waves, and the recursion coefficients stay in
// registers (map2alm).  A wave repeats the recursion for its own columns: 7 FP64
// operations a row (spin 2), beside 2 MFMAs (32 of them) per column tile.
//
// Spin 2 packs one 16-column tile from both components of 4 map sets:
//   map2alm  [E | B'] += F+ [Q | Y] + F- [Y | Q]       (Y = iU, B' = i a_B)
//   alm2map  in the basis P, M = lambda_{+2}, lambda_{-2} with S = E + B', D = E - B'
//            and the mirror signs s_l = (-1)^{l+m}: P_S = s M_N, M_S = s P_N, so
//            P [S | s D] = [G_N | H_S],  M [s S | D] = [G_S | H_N],
//            Q = -(G + H)/2, Y = -(G - H)/2 on either hemisphere.
// The long chains run in P, M: each function then grows by its own recursion, where
// F+- would carry a small one as the difference of two large ones.
//
// Bound by the FP64 pipe, which MFMAs and every other vector instruction share (see
// k_m2a_reg64); one-wave blocks, since a block of four waits with its registers for the
// longest (10-14% slower).  Measured (us per launch, LDS kernels of k_leg.hip -> these;
// spin 2, spin 0):
//   nside 512, 1 map set    alm2map 4507 -> 654, 1839 -> 410; map2alm 5211 -> 840, 1837 -> 530
//   nside 256, 16 map sets  alm2map 1444 -> 622, 487 -> 178; map2alm 1368 -> 690, 429 -> 216
//   nside 512, 125 map sets alm2map 37.2 -> 30.9 ms, 11.1 -> 8.5; map2alm 36.8 -> 31.3, 10.2 -> 8.5
//   FP32, 125 map sets      map2alm 20.8 -> 19.4 ms, 5.9 -> 5.4
#include "leg_rec.h"

namespace sht {
namespace {

constexpr int RWAVES = 4;    // waves of a block that splits its rings
constexpr int RTL = 128;     // map2alm, FP32: l per tile (16 segments)
constexpr unsigned SGN = 0x80000000u;

// value of the lane NC / 2 further on within each group of NC lanes
template <int NC>
__device__ __forceinline__ int swap_half(int v)
{
    static_assert(NC == 16 || NC == 4, "row_ror:8, quad_perm:[2,3,0,1]");
    return __builtin_amdgcn_mov_dpp(v, NC == 16 ? 0x128 : 0x4e, 0xf, 0xf, true);
}
template <int NC>
__device__ __forceinline__ float swap_half(float v)
{
    return __int_as_float(swap_half<NC>(__float_as_int(v)));
}
template <int NC>
__device__ __forceinline__ double swap_half(double v)
{
    return __hiloint2double(swap_half<NC>(__double2hiint(v)), swap_half<NC>(__double2loint(v)));
}

// FP64 MFMA of 16 rows x 4 K slots x NC columns: 16x16x4, or four 4x4x4 blocks whose
// B operands repeat the same 4 columns (same rate, a quarter of the work).  A: row
// lane & 15, slot lane >> 4 in both; B: column lane & (NC - 1), slot lane >> 4.
template <int NC>
struct Mf64;
template <>
struct Mf64<16> {
    using acc = v4d;
    static constexpr int AR = 4;
    __device__ static __forceinline__ acc zero() { return acc{0, 0, 0, 0}; }
    __device__ static __forceinline__ acc run(double a, double b, acc c) { return Mfma<double>::run(a, b, c); }
    __device__ static __forceinline__ double get(const acc& c, int q) { return c[q]; }
    __device__ static __forceinline__ int row(int lane, int q) { return 4 * q + (lane >> 4); }
};
template <>
struct Mf64<4> {
    using acc = double;
    static constexpr int AR = 1;
    __device__ static __forceinline__ acc zero() { return 0.0; }
    __device__ static __forceinline__ acc run(double a, double b, acc c)
    {
        return __builtin_amdgcn_mfma_f64_4x4x4f64(a, b, c, 0, 0, 0);
    }
    __device__ static __forceinline__ double get(const acc& c, int) { return c; }
    __device__ static __forceinline__ int row(int lane, int) { return (lane & 12) + (lane >> 4); }
};

// l tiles of rtl rows of order m (none if the plan does not own it)
__device__ __forceinline__ int ntl(const LegArgs& a, int m, int rtl)
{
    if (a.rowoff[m + 1] == a.rowoff[m]) return 0;
    return (a.lmax - lbase(a.spin, m) + rtl) / rtl;
}

// Work order: block b runs on XCD b mod 8.  The m are dealt to the XCDs in turn (the
// tiles of an m then share an L2) and start in order of m, longest chains first, so
// that a launch ends on short ones.  With few m (short lists, small lmax) the blocks of
// one m are spread over the XCDs, which would otherwise stand idle.
constexpr int FEW_M = 128;
__host__ __device__ inline int m_group(const LegArgs& a) { return nm_rows(a) < FEW_M ? 1 : 8; }

// the same number of blocks per m (alm2map): m index and block of it
__device__ __forceinline__ void unit_of(const LegArgs& a, int b, int per, int& unit, int& slot)
{
    const int g = m_group(a), pos = g == 8 ? b >> 3 : b, q = pos / per;
    unit = q * g + (g == 8 ? b & 7 : 0);
    slot = pos - q * per;
}
int blocks_for(const LegArgs& a, int per)
{
    const int g = m_group(a), n = nm_rows(a);
    return (n + g - 1) / g * g * per;
}

// map2alm: l tiles of rtl rows, fewer toward high m.  The m, or the m that a part plan
// owns, are dealt in groups of g consecutive positions, which all get as many blocks as
// the first of them can have tiles.  (By the position, not by m itself: a part owns one or
// two residues of m modulo the number of parts, so its work lay on one or two XCDs.  Nside
// 2048, 2 IQU sets, part 0 or 3 of 8: spin 2 49.7 -> 10.2 ms, spin 0 13.7 -> 2.9; of 4:
// 49.9 -> 20.2, 13.7 -> 5.9.)  Other lists, the few m of a level, give every m the same
// number of blocks.
__host__ __device__ inline int most_tiles(const LegArgs& a, int rtl) { return (a.lmax + rtl) / rtl; }
__host__ __device__ inline int deal_log(const LegArgs& a) { return m_group(a) == 1 ? 0 : 3; }
// number of deals whose first m can have more than nt tiles: whose lower bound (position
// i: m = i, owned m: mstep (i - 1)) lies below lmax + 1 - nt rtl
__host__ __device__ inline int deals_above(const LegArgs& a, int rtl, int nt)
{
    const int x = a.lmax + 1 - nt * rtl, lg = deal_log(a), up = (1 << lg) - 1;
    if (x <= 0) return 0;
    if (!a.mstep) return (x + up) >> lg;
    const int e = ((x + a.mstep - 1) / a.mstep + 1 + up) >> lg;  // positions i < x / mstep + 1
    const int all = (nm_rows(a) + up) >> lg;
    return e < all ? e : all;
}
int blocks_m2a(const LegArgs& a, int rtl, int ncg)
{
    if (a.mlist && !a.mstep) return a.nlist * most_tiles(a, rtl) * ncg;
    int n = 0;
    for (int nt = most_tiles(a, rtl); nt > 0; --nt) n += deals_above(a, rtl, nt - 1);
    return (n << deal_log(a)) * ncg;
}
// the (m, l tile, column group) of this block; false past the m's tiles
__device__ __forceinline__ bool m2a_task(const LegArgs& a, int b, int rtl, int ncg, int& m, int& lt, int& cg)
{
    int slot;
    if (a.mlist && !a.mstep) {
        const int per = most_tiles(a, rtl) * ncg, u = b / per;
        if (u >= a.nlist) return false;
        m = a.mlist[u];
        slot = b - u * per;
    } else {
        const int lg = deal_log(a);
        int rem = b >> lg, q = 0, nt = most_tiles(a, rtl);
        while (nt > 1) {  // deals q .. e - 1 have nt tiles per m
            const int e = deals_above(a, rtl, nt - 1), n = (e - q) * nt * ncg;
            if (rem < n) break;
            rem -= n;
            q = e;
            --nt;
        }
        const int d = rem / (nt * ncg);
        slot = rem - d * nt * ncg;
        m = ((q + d) << lg) + (b & ((1 << lg) - 1));
        if (m >= nm_rows(a)) return false;
        if (a.mlist) m = a.mlist[m];
    }
    m = __builtin_amdgcn_readfirstlane(m);
    lt = __builtin_amdgcn_readfirstlane(slot / ncg);
    cg = slot - lt * ncg;
    return lt < ntl(a, m, rtl);
}

// FP32: emitter of one recursion row, whose values are A operands at once
template <int C>
struct RowToMfma {
    using MF = Mfma<float>;
    typename MF::acc (&acc)[C];
    const float (&b)[2][C];   // T_N + T_S, T_N - T_S (spin 2: [Q | Y])
    const float (&bs)[2][C];  // spin 2: the same of [Y | Q]
    template <int R>
    __device__ __forceinline__ void put(float v)
    {
#pragma unroll
        for (int c = 0; c < C; ++c) acc[c] = MF::run(v, b[R & 1][c], acc[c]);
    }
    template <int R>
    __device__ __forceinline__ void put(float p, float q)
    {
#pragma unroll
        for (int c = 0; c < C; ++c) acc[c] = MF::run(p, b[R & 1][c], acc[c]);
#pragma unroll
        for (int c = 0; c < C; ++c) acc[c] = MF::run(q, bs[(R & 1) ^ 1][c], acc[c]);
    }
};

// A value that counts as zero: its upper word cleared (what is left, a denormal
// below 2^-1042, vanishes in any sum), one select instead of two.
__device__ __forceinline__ double zero_unless(bool live, double v)
{
    return __hiloint2double(live ? __double2hiint(v) : 0, __double2loint(v));
}
// FP32 A operand from a recursion value
__device__ __forceinline__ float operand32(bool live, double v) { return live ? (float)v : 0.0f; }

// rec_row (same recursion, same values) with the row masked in the operand's format;
// rows past lmax need no mask: their coefficients are zero
template <int R, int C>
__device__ __forceinline__ void rec_row_reg(Rec<0>& f, const double (&c)[3], RowToMfma<C>& em)
{
    if constexpr (R > 1) {
        double v = fma(-c[0], f.t, c[0]) * f.v1 - c[1] * f.v0;
        if (__builtin_expect(f.any, 0)) {
            if (f.k > 0 && fabs(v) > RESCALE_AT) {
                v *= SCALE_DOWN;
                f.v1 *= SCALE_DOWN;
                --f.k;
            }
        }
        f.v0 = f.v1;
        f.v1 = v;
    }
    em.template put<R>(operand32(f.k == 0, R == 0 ? f.v0 : f.v1));
}
template <int R, int C>
__device__ __forceinline__ void rec_row_reg(Rec<2>& f, const double (&c)[3], RowToMfma<C>& em)
{
    if constexpr (R > 1) {
        const double ax = fma(-c[0], f.t, c[0]), be = c[1], ga = c[2];
        double fp = fma(ax, f.a1, fma(be, f.b1, -ga * f.a0));
        double fm = fma(ax, f.b1, fma(be, f.a1, -ga * f.b0));
        if (__builtin_expect(f.any, 0)) {
            if (f.k > 0 && fmax(fabs(fp), fabs(fm)) > RESCALE_AT) {
                fp *= SCALE_DOWN;
                fm *= SCALE_DOWN;
                f.a1 *= SCALE_DOWN;
                f.b1 *= SCALE_DOWN;
                --f.k;
            }
        }
        f.a0 = f.a1;
        f.a1 = fp;
        f.b0 = f.b1;
        f.b1 = fm;
    }
    em.template put<R>(operand32(f.k == 0, R == 0 ? f.a0 : f.a1), operand32(f.k == 0, R == 0 ? f.b0 : f.b1));
}

// ============================================================================
// map2alm, FP32: A_l = sum over north rings of lambda_l (T_N +- T_S), or the block form of
// spin 2.  Wave: 128 l x C column tiles, all rings from the equator to the first
// significant chunk.  The sum over rings runs in the order of k_leg.hip's kernels
// (chunks of 32 rings from the equator, groups of 4 within a chunk): same bits.
// ============================================================================
template <int SPIN, int C>
__global__ __launch_bounds__(64, 2) void k_m2a_reg32(LegArgs a, int ncg)
{
    using T = float;
    constexpr int MS = SPIN == 2 ? 8 : 16;  // columns of one component per tile
    constexpr int CS = SPIN == 0 ? 2 : 4, NCF = SPIN == 0 ? 2 : 3;
    const int lane = threadIdx.x;
    const int i = lane & 15, k = lane >> 4;
    const int L = a.lmax;

    int m, lt, cg;
    if (!m2a_task(a, blockIdx.x, RTL, ncg, m, lt, cg)) return;
    const int lb = lbase(SPIN, m);
    const int l0 = lb + lt * RTL, lend = min(L, l0 + RTL - 1);
    const int ls = l0 + SEG * i, cnt = L - ls + 1;  // this lane's segment; rows in range
    const int64_t row0 = a.rowoff[m];

    // coefficients of the segment's rows (zero past lmax: those rows stay zero)
    double cf[SEG][3];
#pragma unroll
    for (int t = 2; t < SEG; ++t)
#pragma unroll
        for (int q = 0; q < NCF; ++q)
            cf[t][q] = t < cnt ? a.coef[(row0 + (ls - lb) + t) * CS + q] : 0.0;

    // columns
    const int j = SPIN == 2 ? (i & 7) : i;
    const int col = cg * (C * MS) + j;  // tile c of the wave: col + MS c; C MS divides ldx
    const bool second = SPIN == 2 && i >= 8;  // lane holds Y columns (outputs B')
    const unsigned ysg = second ? ((j & 1) ? 0u : SGN) : 0u;  // Y_re = -U_im, Y_im = U_re
    const unsigned pos = SPIN == 2 && ((lb - m) & 1) ? SGN : 0u;
    const T* X = xptr<T>(a, SPIN == 2 ? (second ? 2 : 1) : 0) + (int64_t)m * a.nring * a.ldx + (second ? (col ^ 1) : col);
    // seed arrays of this m: one scalar base each, one 32-bit offset per lane
    const double* mu = a.mu + a.seedoff[m];
    const int* kk = a.kk + a.seedoff[m];
    const unsigned sofs = (unsigned)(min(16 * lt + i, (L - lb) / SEG) * a.rn);

    using MF = Mfma<T>;
    typename MF::acc acc[SEG][C];
#pragma unroll
    for (int t = 0; t < SEG; ++t)
#pragma unroll
        for (int c = 0; c < C; ++c) acc[t][c] = typename MF::acc{0, 0, 0, 0};

    const int nchunk = (a.rn + RCHUNK - 1) / RCHUNK;
    const int rc0 = first_chunk(a, m, nchunk, lend);
    if (rc0 < nchunk) {
        // eight rings at a time, as two MFMA groups of 4 (n0 eights in the equator
        // chunk, 4 in every other)
        const int n0 = (a.rn - (nchunk - 1) * RCHUNK + 7) / 8;
        const int g1 = n0 + 4 * (nchunk - 1 - rc0);
        constexpr int NV = SPIN == 0 ? 2 : 4;
        struct Stage {
            double v[NV][2], t[2];  // seed values and 1 - x of the two rings
            int k[2], r;
            T x[2][2][C];           // [ring][north, south][column tile]
        };
        auto load = [&](Stage& s, int g) {
            const int h = g - n0;
            const int r8 = g < n0 ? (nchunk - 1) * RCHUNK + 8 * g : (nchunk - 2 - (h >> 2)) * RCHUNK + 8 * (h & 3);
            s.r = r8 + k;
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int rr = min(s.r + 4 * u, a.rn - 1);
                const unsigned o = sofs + (unsigned)rr;
#pragma unroll
                for (int q = 0; q < NV; ++q) s.v[q][u] = (mu + q * a.seedstride)[o];
                s.k[u] = kk[o];
                s.t[u] = a.rings[(unsigned)rr].omz;
                const T* pn = X + (int64_t)rr * a.ldx;
                const T* ps = X + (int64_t)(a.nring - 1 - rr) * a.ldx;
#pragma unroll
                for (int c = 0; c < C; ++c) {
                    s.x[u][0][c] = pn[MS * c];
                    s.x[u][1][c] = ps[MS * c];
                }
            }
        };
        auto run = [&](Stage& s, auto ui, int gnext) {
            constexpr int u = decltype(ui)::v;
            Seed<SPIN> sd;
            if constexpr (SPIN == 0) {
                sd.v0 = s.v[0][u];
                sd.v1 = s.v[1][u];
            } else {
                sd.p0 = s.v[0][u];
                sd.p1 = s.v[1][u];
                sd.q0 = s.v[2][u];
                sd.q1 = s.v[3][u];
            }
            sd.t = s.t[u];
            sd.k = s.k[u];
            double w = m2a_weight(a, s.r + 4 * u);
            if (cnt < 1) w = 0.0;
            Rec<SPIN> f;
            f.start(sd, w);
            if constexpr (SPIN == 0) {
                if (cnt < 2) f.v1 = 0.0;
            } else {
                if (cnt < 2) f.a1 = f.b1 = 0.0;
            }
            T b[2][C], bs[2][C];  // sums and differences: own component, the other one
#pragma unroll
            for (int c = 0; c < C; ++c) {
                const T n = flip(s.x[u][0][c], ysg), so = flip(s.x[u][1][c], ysg ^ pos);
                b[0][c] = n + so;
                b[1][c] = n - so;
                if constexpr (SPIN == 2) {
                    bs[0][c] = swap_half<16>(b[0][c]);
                    bs[1][c] = swap_half<16>(b[1][c]);
                }
            }
            if constexpr (u == 1) load(s, gnext);
            __builtin_amdgcn_sched_barrier(0);
            static_for<0, SEG>([&](auto ti) {
                constexpr int t = decltype(ti)::v;
                RowToMfma<C> em{acc[t], b, bs};
                rec_row_reg<t>(f, cf[t], em);
            });
        };
        Stage s;
        load(s, 0);
        for (int g = 0; g < g1; ++g) {
            run(s, IC<0>{}, 0);
            run(s, IC<1>{}, min(g + 1, g1 - 1));
        }
    }

    T* A = aptr<T>(a, SPIN == 2 ? (second ? 2 : 1) : 0) + row0 * a.ldx;
#pragma unroll
    for (int t = 0; t < SEG; ++t)
#pragma unroll
        for (int c = 0; c < C; ++c)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int l = l0 + SEG * MF::row(lane, q) + t;
                if (l <= L) A[(int64_t)(l - lb) * a.ldx + col + MS * c] = acc[t][c][q];
            }
}

// ============================================================================
// map2alm, FP64.  Wave: 16 runs of TS rows of l (one per MFMA row) x C tiles of NC
// columns; rings eight at a time from the equator to the first significant chunk, slot
// k taking rings 2k, 2k + 1 of the eight (one 16-byte load per seed array).  Split: the
// four waves of a block share one tile and take a quarter of its rings each (grids too
// small to fill the chip); their sums meet in LDS in a fixed order.
//
// While an FP64 MFMA runs, no other vector instruction of the SIMD does: one costs about 3
// cycles of it, an FP64 one 5 (measured beside 8 MFMAs of 64).  So the loop is kept to the
// recursion and one operation per operand:
//  * The recursion runs on p_l = P_l / N_l (N of a run's first two rows 1, N_l =
//    gamma_l N_{l-2}), which makes it p_l = (a_l x + b_l) p_{l-1} - p_{l-2}: four FP64
//    operations a row for P and M together, not seven; N_l multiplies the sums.
//  * Spin 2 in the basis P, M (see the head of the file): with S = Q + Y, D = Q - Y of
//    either hemisphere, P [S_N | s D_S] + M [s S_S | D_N] = [g | h],
//    E = -(g + h)/2, B' = -(g - h)/2.  The mirror signs s_l alternate with l: they go into
//    the recursion of s M and, for the second half, into the sums, so that every row
//    takes the same operands [S_N | D_S], [S_S | D_N].
//  * Waves mask and rescale only where a lane carries an exponent (toward the poles); the
//    equator's group (counted half) and a last one reaching past the first ring run the
//    masked form too.
//  * TS = 16 reads every second seed of the table: half the traffic, which bounds one or
//    two map sets.  Rows past lmax go on harmlessly and are not stored.
// ============================================================================
template <int SPIN, int NC, int C, int TS, bool SPLIT>
__device__ __forceinline__ void m2a_reg64(const LegArgs& a, int block, int ncg, double* lds)
{
    using MF = Mf64<NC>;
    constexpr int MS = SPIN == 2 ? NC / 2 : NC;  // columns of one component per tile
    constexpr int CS = SPIN == 0 ? 2 : 4, NV = SPIN == 0 ? 2 : 4;
    constexpr int RTL64 = 16 * TS;
    const int lane = threadIdx.x & 63, wave = SPLIT ? wave_index() : 0;
    const int i = lane & 15, k = lane >> 4;
    const int L = a.lmax;

    int m, lt, cg;
    if (!m2a_task(a, block, RTL64, ncg, m, lt, cg)) return;
    const int lb = lbase(SPIN, m);
    const int l0 = lb + lt * RTL64, lend = min(L, l0 + RTL64 - 1);
    const int ls = l0 + TS * i;  // first row of this lane's run
    const int64_t row0 = a.rowoff[m];
    auto gamma = [&](int t) { return a.coef[(row0 + min(ls + t, L) - lb) * CS + (SPIN == 0 ? 1 : 2)]; };

    // the normalised recursion: spin 0 a; spin 2 a, b + a, b - a (of s M)
    double cf[TS][SPIN == 0 ? 1 : 3];
    {
        double n1 = 1.0, n0 = 1.0;  // N of rows t - 1, t - 2
#pragma unroll
        for (int t = 2; t < TS; ++t) {
            const double* c = a.coef + (row0 + min(ls + t, L) - lb) * CS;
            const bool in = ls + t <= L;
            const double n = in ? c[SPIN == 0 ? 1 : 2] * n0 : 1.0;
            const double f = in ? n1 / n : 0.0;
            cf[t][0] = c[0] * f;
            if constexpr (SPIN == 2) {
                cf[t][1] = (c[1] + c[0]) * f;
                cf[t][2] = (c[1] - c[0]) * f;
            }
            n0 = n1;
            n1 = n;
        }
    }

    // columns
    const int jc = lane & (NC - 1), j = jc & (MS - 1);
    const bool second = SPIN == 2 && jc >= MS;  // lane holds the D half (outputs B')
    const int col = cg * (C * MS) + j;          // tile c of the wave: col + MS c; C MS divides ldx
    const unsigned po = SPIN == 2 && ((lb - m) & 1) ? SGN : 0u;
    const double one = second ? -1.0 : 1.0;
    const double yw = (j & 1) ? one : -one;     // Q +- Y: Y_re = -U_im, Y_im = U_re

    typename MF::acc acc[TS][C];
#pragma unroll
    for (int t = 0; t < TS; ++t)
#pragma unroll
        for (int c = 0; c < C; ++c) acc[t][c] = MF::zero();

    const int nchunk = (a.rn + RCHUNK - 1) / RCHUNK;
    const int rlo = first_chunk(a, m, nchunk, lend) * RCHUNK;  // first ring
    // groups of eight rings, group g = rings rn - 8 (g + 1) ..
    int g = 0, gend = max(0, (a.rn - rlo + 7) / 8);
    const int partial = (a.rn - rlo) & 7 ? gend - 1 : -1;      // reaches below rlo
    if constexpr (SPLIT) {
        const int len = (gend + RWAVES - 1) / RWAVES;
        g = min(gend, len * wave);
        gend = min(gend, g + len);
    }
    if (g < gend) {
        // addresses: one scalar base per array and one 32-bit byte offset per lane
        const char* mu = reinterpret_cast<const char*>(a.mu + a.seedoff[m]);
        const char* kk = reinterpret_cast<const char*>(a.kk + a.seedoff[m]);
        const int64_t mstride = a.seedstride * 8;
        const char* rg = reinterpret_cast<const char*>(&a.rings[0].omz);
        const int64_t xm = (int64_t)m * a.nring * a.ldx;
        const char* X0 = reinterpret_cast<const char*>(xptr<double>(a, SPIN == 2 ? 1 : 0) + xm);
        const char* X1 = reinterpret_cast<const char*>(xptr<double>(a, SPIN == 2 ? 2 : 0) + xm);
        const unsigned sofs = (unsigned)(min((TS / SEG) * (16 * lt + i), (L - lb) / SEG) * a.rn);
        // hemisphere a of a ring is the north for the S half, the south for the D half
        const unsigned row = (unsigned)a.ldx * 8u, south = (unsigned)(a.nring - 1) * row, cb = (unsigned)col * 8u;
        const unsigned rowa = second ? 0u - row : row;
        const unsigned basea = cb + (second ? south : 0u), baseb = cb + (second ? 0u : south);
        const int pc = (j & 1) ? -8 : 8;  // partner column of U

        double sv[NV][2], st[2], x[2][SPIN == 2 ? 4 : 2][C];  // seeds, 1 - x; X rows of the two rings
        int sk[2], sr = 0;
        auto at = [](const char* base, unsigned o) { return *reinterpret_cast<const double*>(base + o); };
        auto load = [&](int gg) {
            sr = a.rn - 8 * (gg + 1) + 2 * k;
            const int rr = max(sr, rlo);
            const unsigned o = (sofs + (unsigned)rr) * 4u;
#pragma unroll
            for (int q = 0; q < NV; ++q) {
                const double2 d = *reinterpret_cast<const double2*>(mu + q * mstride + 2u * o);
                sv[q][0] = d.x;
                sv[q][1] = d.y;
            }
            const int2 kd = *reinterpret_cast<const int2*>(kk + o);
            sk[0] = kd.x;
            sk[1] = kd.y;
            const unsigned ro = (unsigned)rr * (unsigned)sizeof(RingDev), xo = (unsigned)rr * rowa;
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                st[u] = at(rg + u * sizeof(RingDev), ro);
                const unsigned oa = basea + xo + (u ? rowa : 0u), ob = baseb - xo - (u ? rowa : 0u);
#pragma unroll
                for (int c = 0; c < C; ++c) {
                    x[u][0][c] = at(X0 + 8 * MS * c, oa);
                    x[u][1][c] = at(X0 + 8 * MS * c, ob);
                    if constexpr (SPIN == 2) {
                        x[u][2][c] = at(X1 + 8 * MS * c, oa + pc);
                        x[u][3][c] = at(X1 + 8 * MS * c, ob + pc);
                    }
                }
            }
        };
        auto run = [&](auto masked, auto ui, int gnext) {
            constexpr bool MASK = decltype(masked)::v != 0;
            constexpr int u = decltype(ui)::v;
            double p0 = sv[0][u], p1 = sv[1][u], q0 = 0.0, q1 = 0.0;
            if constexpr (SPIN == 2) {  // s M
                q0 = flip(sv[2][u], po);
                q1 = flip(sv[3][u], SGN ^ po);
            }
            const double tt = st[u];
            int e = 0;
            if constexpr (MASK) {
                // the equator ring counts half, rings below the first one nothing
                const double w = sr < rlo ? 0.0 : (2 * (sr + u) + 1 == a.nring ? 0.5 : 1.0);
                p0 *= w;
                p1 *= w;
                q0 *= w;
                q1 *= w;
                e = sk[u];
            }
            bool mk[2] = {true, true};
            // spin 0: even rows T_N + T_S, odd rows T_N - T_S; spin 2: operands of P and of s M
            double b[C], d[C];
#pragma unroll
            for (int c = 0; c < C; ++c) {
                if constexpr (SPIN == 0) {
                    b[c] = x[u][0][c] + x[u][1][c];
                    d[c] = x[u][0][c] - x[u][1][c];
                } else {
                    b[c] = fma(x[u][2][c], yw, x[u][0][c]);
                    d[c] = fma(x[u][3][c], yw, x[u][1][c]);
                }
            }
            if constexpr (u == 1) load(gnext);
            __builtin_amdgcn_sched_barrier(0);
            static_for<0, TS / 2>([&](auto hi) {
                constexpr int t = 2 * decltype(hi)::v;
                // rows t, t + 1
                if constexpr (t > 0) {
#pragma unroll
                    for (int v = 0; v < 2; ++v) {
                        double pn, qn = 0.0;
                        if constexpr (SPIN == 0) {
                            const double c0 = cf[t + v][0];
                            pn = fma(fma(-c0, tt, c0), v ? p0 : p1, v ? -p1 : -p0);
                        } else {
                            const double c0 = cf[t + v][0];
                            pn = fma(fma(-c0, tt, cf[t + v][1]), v ? p0 : p1, v ? -p1 : -p0);
                            qn = fma(fma(c0, tt, cf[t + v][2]), v ? q0 : q1, v ? -q1 : -q0);
                        }
                        if constexpr (MASK) {
                            const double big = SPIN == 0 ? fabs(pn) : fmax(fabs(pn), fabs(qn));
                            if (e > 0 && big > RESCALE_AT) {
                                pn *= SCALE_DOWN;
                                qn *= SCALE_DOWN;
                                if (v) {
                                    p0 *= SCALE_DOWN;
                                    q0 *= SCALE_DOWN;
                                } else {
                                    p1 *= SCALE_DOWN;
                                    q1 *= SCALE_DOWN;
                                }
                                --e;
                            }
                        }
                        if (v) {
                            p1 = pn;
                            q1 = qn;
                        } else {
                            p0 = pn;
                            q0 = qn;
                        }
                        if constexpr (MASK) mk[v] = e == 0;
                    }
                } else if constexpr (MASK) {
                    mk[0] = mk[1] = e == 0;
                }
                const double po0 = MASK ? zero_unless(mk[0], p0) : p0, po1 = MASK ? zero_unless(mk[1], p1) : p1;
#pragma unroll
                for (int c = 0; c < C; ++c) acc[t][c] = MF::run(po0, b[c], acc[t][c]);
#pragma unroll
                for (int c = 0; c < C; ++c) acc[t + 1][c] = MF::run(po1, SPIN == 0 ? d[c] : b[c], acc[t + 1][c]);
                if constexpr (SPIN == 2) {
                    const double qo0 = MASK ? zero_unless(mk[0], q0) : q0, qo1 = MASK ? zero_unless(mk[1], q1) : q1;
#pragma unroll
                    for (int c = 0; c < C; ++c) acc[t][c] = MF::run(qo0, d[c], acc[t][c]);
#pragma unroll
                    for (int c = 0; c < C; ++c) acc[t + 1][c] = MF::run(qo1, d[c], acc[t + 1][c]);
                }
            });
        };
        load(g);
        // three loops in a row, not a choice per group: the compiler would keep two sets
        // of accumulators for the two forms
        const int plain_end = partial < 0 ? gend : min(gend, partial);
        if constexpr (!SPLIT) {
            run(IC<1>{}, IC<0>{}, 0);
            run(IC<1>{}, IC<1>{}, min(g + 1, gend - 1));
            ++g;
        }
        for (; !SPLIT && g < plain_end && !__any((sk[0] | sk[1]) > 0); ++g) {
            run(IC<0>{}, IC<0>{}, 0);
            run(IC<0>{}, IC<1>{}, min(g + 1, gend - 1));
        }
        for (; g < gend; ++g) {
            run(IC<1>{}, IC<0>{}, 0);
            run(IC<1>{}, IC<1>{}, min(g + 1, gend - 1));
        }
    }

    double* A = aptr<double>(a, SPIN == 2 ? (second ? 2 : 1) : 0) + row0 * a.ldx;
    // row t of every run: undo the normalisation, form E and B', store
    auto store = [&](int t, double nt, const typename MF::acc (&v)[C]) {
#pragma unroll
        for (int q = 0; q < MF::AR; ++q) {
            const int s = MF::row(lane, q), l = l0 + TS * s + t;
            const double f = __shfl(nt, s);  // N of run s
#pragma unroll
            for (int c = 0; c < C; ++c) {
                double y = MF::get(v[c], q);
                if constexpr (SPIN == 2) {
                    if (second) y = flip(y, t & 1 ? SGN ^ po : po);  // the D half's mirror sign
                    y = -0.5 * fma(y, one, swap_half<NC>(y));
                }
                if (l <= L) A[(int64_t)(l - lb) * a.ldx + col + MS * c] = f * y;
            }
        }
    };
    // partial sums [wave][row][tile][lane]
    typename MF::acc* part = reinterpret_cast<typename MF::acc*>(lds) + lane;
    if constexpr (SPLIT) {
#pragma unroll
        for (int t = 0; t < TS; ++t)
#pragma unroll
            for (int c = 0; c < C; ++c) part[((wave * TS + t) * C + c) * 64] = acc[t][c];
        __syncthreads();
    }
    double n1 = 1.0, n0 = 1.0;
#pragma unroll
    for (int t = 0; t < TS; ++t) {
        const double n = t < 2 ? 1.0 : gamma(t) * n0;
        n0 = n1;
        n1 = n;
        if constexpr (!SPLIT) {
            store(t, n, acc[t]);
        } else if (t / (TS / RWAVES) == wave) {  // each wave adds and stores its share of the rows
            typename MF::acc v[C];
#pragma unroll
            for (int c = 0; c < C; ++c) {
                v[c] = part[(t * C + c) * 64];
#pragma unroll
                for (int w = 1; w < RWAVES; ++w) v[c] += part[((w * TS + t) * C + c) * 64];
            }
            store(t, n, v);
        }
    }
}

// doubles of LDS of a split block
template <int NC, int C, int TS>
constexpr int split_lds() { return RWAVES * TS * C * 64 * Mf64<NC>::AR; }

template <int SPIN, int NC, int C, int TS, bool SPLIT>
__global__ __launch_bounds__(SPLIT ? 64 * RWAVES : 64, 2) void k_m2a_reg64(LegArgs a, int ncg)
{
    __shared__ alignas(32) double lds[SPLIT ? split_lds<NC, C, TS>() : 4];
    m2a_reg64<SPIN, NC, C, TS, SPLIT>(a, blockIdx.x, ncg, lds);
}

// Both spins of a small call in one launch: blocks below n2 are spin 2, the others spin
// 0.  Launched apart, each ends on a half-empty chip and pays its own start.
template <int NC2, int NC0>
__global__ __launch_bounds__(64 * RWAVES, 2) void k_m2a_pair(LegArgs a2, int ncg2, int n2, LegArgs a0, int ncg0)
{
    __shared__ alignas(32) double lds[split_lds<(NC2 > NC0 ? NC2 : NC0), 1, SEG>()];
    if ((int)blockIdx.x < n2) m2a_reg64<2, NC2, 1, SEG, true>(a2, blockIdx.x, ncg2, lds);
    else m2a_reg64<0, NC0, 1, SEG, true>(a0, (int)blockIdx.x - n2, ncg0, lds);
}

// ============================================================================
// alm2map: T_r = sum over l of lambda_l A_l.  Wave: R x 16 rings x C column tiles;
// slot k takes the k-th quarter of the l range (whole 8-row segments), row i a ring.
// Each step needs one row of coefficients and of A per quarter, read PD steps ahead.
// ============================================================================
constexpr int A2M_LDS = 2 * 4 * (SEG * 4 + 4);  // doubles: two blocks of coefficients of four quarters
// EB = 1 (E only), 2 (B only): plain columns as in spin 0 (tiles of 8 map sets), even
// and odd rows of P and M apart; the other component is neither read nor multiplied.
template <int SPIN, int EB, int NC, int R, int C>
__device__ __forceinline__ void a2m_reg(const LegArgs& a, int block, int per, int nrt, double* lds)
{
    constexpr bool PACK = SPIN == 2 && EB == 0;  // S and D columns in one tile
    using MF = Mf64<NC>;
    constexpr int MS = PACK ? NC / 2 : NC;
    constexpr int NA = SPIN == 2 && EB ? 4 : 2;
    constexpr int CS = SPIN == 0 ? 2 : 4;
    constexpr int PD = PACK && C == 4 ? 2 : 4;  // rows of A read ahead
    static_assert(SEG % PD == 0, "the operand buffers cycle within a segment");
    constexpr int CQ = SEG * CS + 4;  // doubles per quarter of a coefficient block (padded)
    static_assert(8 * CQ <= A2M_LDS);
    const int lane = threadIdx.x;
    const int i = lane & 15, k = lane >> 4;
    const int L = a.lmax;

    int unit, slot;
    unit_of(a, block, per, unit, slot);
    if (unit >= nm_rows(a)) return;
    const int m = a.mlist ? __builtin_amdgcn_readfirstlane(a.mlist[unit]) : unit;
    const int cg = slot / nrt, rt = slot - cg * nrt;
    if (cg * C * MS >= a.ncols) return;
    const int lb = lbase(SPIN, m);
    const int r0 = rt * 16 * R;

    const int jc = lane & (NC - 1), j = jc & (MS - 1);
    const int col = cg * (C * MS) + j;  // tile c of the wave: col + MS c; C MS divides ldx
    const bool second = PACK && jc >= MS;

    // first segment with a significant value on these rings
    int lsig = L + 1;
    if (lb <= L)
        for (int c = r0 / RCHUNK; c < min(a.nrc, (r0 + 16 * R + RCHUNK - 1) / RCHUNK); ++c)
            lsig = min(lsig, a.lsig[(int64_t)m * a.nrc + c]);
    lsig = __builtin_amdgcn_readfirstlane(lsig);

    using acc_t = typename MF::acc;
    acc_t acc[NA][R][C];  // spin 0: even, odd rows; spin 2: P and M products; EB: P even, odd, M even, odd
#pragma unroll
    for (int h = 0; h < NA; ++h)
#pragma unroll
        for (int q = 0; q < R; ++q)
#pragma unroll
            for (int c = 0; c < C; ++c) acc[h][q][c] = MF::zero();

    if (lsig <= L) {
        const int s0 = (lsig - lb) / SEG, nseg = (L - lb) / SEG - s0 + 1;
        const int nrow = L - lb;                        // last row of this m
        // quarter k: segments s0 + k nseg / 4 .. s0 + (k + 1) nseg / 4 - 1
        const int nb = (nseg + 3) / 4, nmin = nseg / 4;  // longest and shortest quarter
        const int sk = s0 + k * nseg / 4;
        const int t0 = SEG * sk, lim = min(nrow, SEG * (s0 + (k + 1) * nseg / 4) - 1);  // first, last row
        const int64_t row0 = a.rowoff[m];
        double v0[R], v1[R], w0[R], w1[R], x[R];        // rows t, t + 1: lambda; spin 2: P and s M
        int e[R];
#pragma unroll
        for (int q = 0; q < R; ++q) {
            const int r = min(r0 + 16 * q + i, a.rn - 1);
            const int64_t s = a.seedoff[m] + (int64_t)sk * a.rn + r;
            v0[q] = a.mu[s];
            v1[q] = a.mu[a.seedstride + s];
            if constexpr (SPIN == 2) {
                w0[q] = a.mu[2 * a.seedstride + s];
                w1[q] = -a.mu[3 * a.seedstride + s];
            }
            e[q] = a.kk[s];
            x[q] = a.rings[r].omz;
        }
        // rows t .. t + PD - 1 of A: spin 2 S = A0 + A1, D = A0 - A1 (E and B'); the last
        // row of the m repeats past its end
        constexpr int NS = PACK ? 2 : 1;
        double st[PD][NS][C];
        const char* A0 = reinterpret_cast<const char*>(aptr<double>(a, SPIN == 2 ? (EB == 2 ? 2 : 1) : 0) + row0 * a.ldx);
        const char* A1 = reinterpret_cast<const char*>(aptr<double>(a, SPIN == 2 ? 2 : 0) + row0 * a.ldx);
        const unsigned rowb = (unsigned)a.ldx * 8u, cb = (unsigned)col * 8u;
        auto fetch = [&](double (&s)[NS][C], unsigned o) {  // one 32-bit byte offset per lane
#pragma unroll
            for (int c = 0; c < C; ++c) {
                s[0][c] = *reinterpret_cast<const double*>(A0 + 8 * MS * c + o);
                if constexpr (PACK) s[NS - 1][c] = *reinterpret_cast<const double*>(A1 + 8 * MS * c + o);
            }
        };
        unsigned ahead = 0;  // plain blocks: offset of the next row to read
        // coefficients of the 8 rows a block of steps produces, per quarter: one
        // 16-byte load per lane and block, handed round through the wave's own LDS
        double2* cw = reinterpret_cast<double2*>(lds) + k * (CQ / 2) + (CS == 4 ? i : (i & 7));
        const double* cr = lds + k * CQ;
        const double2* cg2 = reinterpret_cast<const double2*>(a.coef + row0 * CS);
        auto load_coef = [&](int t) {
            const int row = min(t + 2 + (CS == 4 ? (i >> 1) : (i & 7)), nrow);
            return cg2[CS == 4 ? 2 * row + (i & 1) : row];
        };
        double2 cnext = load_coef(t0);
        const double one = second ? -1.0 : 1.0;
        // Block n of 8 steps.  Packed operand of row t, for P and for s M: [S | s D] with
        // s_l = (-1)^t (the sign of the first row enters the southern sums at the end).
        // MASK: a lane carries an exponent or is near the end of its quarter.
        auto block = [&](auto masked, int n) {
            constexpr bool MASK = decltype(masked)::v != 0;
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            cw[(n & 1) * 2 * CQ] = cnext;
            cnext = load_coef(t0 + SEG * (n + 1));
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            const double* cb_ = cr + (n & 1) * 4 * CQ;
            static_for<0, SEG>([&](auto ti) {
                constexpr int t = decltype(ti)::v;
                double (&s)[NS][C] = st[t % PD];
                const double c0 = cb_[CS * t], c1 = cb_[CS * t + 1], c2 = SPIN == 2 ? cb_[CS * t + 2] : 0.0;
                double b[C];
#pragma unroll
                for (int c = 0; c < C; ++c)
                    b[c] = !PACK ? s[0][c] : t & 1 ? fma(s[0][c], one, s[NS - 1][c]) : fma(s[NS - 1][c], one, s[0][c]);
                fetch(s, MASK ? (unsigned)min(t0 + SEG * n + t + PD, nrow) * rowb + cb : ahead);
                if constexpr (!MASK) ahead += rowb;
                const bool in = !MASK || t0 + SEG * n + t <= lim;
#pragma unroll
                for (int q = 0; q < R; ++q) {
                    const bool live = !MASK || (in && e[q] == 0);
                    const double p = MASK ? zero_unless(live, v0[q]) : v0[q];
#pragma unroll
                    for (int c = 0; c < C; ++c) {
                        acc_t& d = acc[PACK ? 0 : (t & 1)][q][c];
                        d = MF::run(p, b[c], d);
                    }
                    if constexpr (SPIN == 2) {
                        const double g = MASK ? zero_unless(live, w0[q]) : w0[q];
#pragma unroll
                        for (int c = 0; c < C; ++c) {
                            acc_t& d = acc[PACK ? 1 : 2 + (t & 1)][q][c];
                            d = MF::run(g, b[c], d);
                        }
                    }
                    // row t + 2
                    const double ax = fma(-c0, x[q], c0);
                    double v, w = 0.0;
                    if constexpr (SPIN == 0) {
                        v = ax * v1[q] - c1 * v0[q];
                    } else {
                        v = (c1 + ax) * v1[q] - c2 * v0[q];
                        w = (c1 - ax) * w1[q] - c2 * w0[q];
                    }
                    if constexpr (MASK) {
                        const double big = SPIN == 0 ? fabs(v) : fmax(fabs(v), fabs(w));
                        if (e[q] > 0 && big > RESCALE_AT) {
                            v *= SCALE_DOWN;
                            v1[q] *= SCALE_DOWN;
                            if constexpr (SPIN == 2) {
                                w *= SCALE_DOWN;
                                w1[q] *= SCALE_DOWN;
                            }
                            --e[q];
                        }
                    }
                    v0[q] = v1[q];
                    v1[q] = v;
                    if constexpr (SPIN == 2) {
                        w0[q] = w1[q];
                        w1[q] = w;
                    }
                }
            });
        };
        auto scaled = [&] {
            bool any = false;
#pragma unroll
            for (int q = 0; q < R; ++q) any |= e[q] > 0;
            return __any(any) != 0;
        };
#pragma unroll
        for (int t = 0; t < PD; ++t) fetch(st[t], (unsigned)min(t0 + t, nrow) * rowb + cb);
        // exponents only shrink along a chain: masked blocks, plain ones, and the last ones
        // (loops in a row: a choice per block would keep two sets of accumulators)
        int n = 0;
        for (; n < nb && scaled(); ++n) block(IC<1>{}, n);
        ahead = (unsigned)(t0 + SEG * n + PD) * rowb + cb;
        for (; n + 2 < nmin; ++n) block(IC<0>{}, n);
        for (; n < nb; ++n) block(IC<1>{}, n);
    }

    const int64_t xm = (int64_t)m * a.nring * a.ldx;
    const unsigned po = SPIN == 2 && ((lb - m) & 1) ? SGN : 0u;
    // U = -i Y: U_re = Y_im, U_im = -Y_re, this lane's Y goes to the partner column
    const unsigned usg = (j & 1) ? 0u : SGN;
    double* X0 = xptr<double>(a, SPIN == 2 ? (second ? 2 : 1) : 0) + xm + (second ? (col ^ 1) : col);
    double* X1 = xptr<double>(a, SPIN == 2 && EB ? 2 : 0) + xm + (col ^ 1);
#pragma unroll
    for (int c = 0; c < C; ++c)
#pragma unroll
        for (int q = 0; q < R; ++q)
#pragma unroll
            for (int v = 0; v < MF::AR; ++v) {
                const int r = r0 + 16 * q + MF::row(lane, v);
                const double g = MF::get(acc[0][q][c], v), h = MF::get(acc[1][q][c], v);
                double n, s, yn = 0.0, ys = 0.0;
                if constexpr (SPIN == 0) {
                    n = g + h;
                    s = g - h;
                } else if constexpr (PACK) {
                    // lanes of S columns hold (G_N, G_S), lanes of D columns (H_S, H_N)
                    const double go = swap_half<NC>(g), ho = swap_half<NC>(h);
                    n = flip(second ? -0.5 * (go - h) : -0.5 * (g + ho), second ? usg : 0u);
                    s = flip(second ? -0.5 * (ho - g) : -0.5 * (h + go), (second ? usg : 0u) ^ po);
                } else {
                    const double u = MF::get(acc[NA - 2][q][c], v), w = MF::get(acc[NA - 1][q][c], v);
                    // odd rows hold -M; P_S = s M_N, M_S = s P_N
                    const double pn = g + h, mn = u - w, ps = u + w, ms = g - h;
                    const double a0 = -0.5 * (pn + mn), a1 = -0.5 * (pn - mn);
                    const double b0 = -0.5 * (ps + ms), b1 = -0.5 * (ps - ms);
                    n = EB == 1 ? a0 : a1;
                    s = flip(EB == 1 ? b0 : b1, po);
                    yn = flip(EB == 1 ? a1 : a0, usg);
                    ys = flip(EB == 1 ? b1 : b0, usg ^ po);
                }
                if (r >= a.rn) continue;
                const int rs = a.nring - 1 - r;
                X0[(int64_t)r * a.ldx + MS * c] = n;
                if (rs != r) X0[(int64_t)rs * a.ldx + MS * c] = s;
                if constexpr (PACK && NC == 4) {
                    // a tile is one map set: the last of an odd count clears the columns of the
                    // padding map it shares a ring FFT with
                    if ((a.ncols & 2) && col - j + MS * (c + 1) == a.ncols) {
                        X0[(int64_t)r * a.ldx + MS * (c + 1)] = 0.0;
                        X0[(int64_t)rs * a.ldx + MS * (c + 1)] = 0.0;
                    }
                }
                if constexpr (SPIN == 2 && EB) {
                    X1[(int64_t)r * a.ldx + MS * c] = yn;
                    if (rs != r) X1[(int64_t)rs * a.ldx + MS * c] = ys;
                }
            }
}

template <int SPIN, int EB, int NC, int R, int C>
__global__ __launch_bounds__(64, 2) void k_a2m_reg(LegArgs a, int per, int nrt)
{
    __shared__ alignas(16) double lds[A2M_LDS];
    a2m_reg<SPIN, EB, NC, R, C>(a, blockIdx.x, per, nrt, lds);
}

// both spins of a small call in one launch, as k_m2a_pair
template <int NC, int R>
__global__ __launch_bounds__(64, 2) void k_a2m_pair(LegArgs a2, int per2, int n2, LegArgs a0, int per0, int nrt)
{
    __shared__ alignas(16) double lds[A2M_LDS];
    if ((int)blockIdx.x < n2) a2m_reg<2, 0, NC, R, 1>(a2, blockIdx.x, per2, nrt, lds);
    else a2m_reg<0, 0, NC, R, 1>(a0, (int)blockIdx.x - n2, per0, nrt, lds);
}

// ----------------------------------------------------------------------------
// Choice of kernel and tile
// ----------------------------------------------------------------------------
// Times below are in units of the MFMAs of one 16-column tile (of one wave's rows),
// fitted on one MI355X at nside 64..512 with 1 to 1000 map sets.

int tiles_of(const LegArgs& a, int ms) { return (a.ncols + ms - 1) / ms; }

// l tiles of `tl` rows over all m (of a list approximately)
double l_tiles(const LegArgs& a, int tl)
{
    const double n = a.lmax + 1;
    return nm_rows(a) * 0.5 * (n / tl + 1.0);
}

// alm2map: R x 16 rings and C tiles of NC columns per wave.  Beside its MFMAs a wave
// spends about 0.5 (R = 1) or 0.3 (R = 2) of a tile on recursion and operands; the last waves
// of a launch run alone for about one more wave (chains of the first m are twice the
// mean).  One or two 4-column tiles (spin 2: 1 or 2 map sets, spin 0: up to 4) take the
// 4-column form: us per launch at nside 512, spin 2, 1 set 1228 -> 654, 2 sets 1233 ->
// 946; a third tile costs more than 16 columns.
struct A2mPick { int nc, r, c; };
A2mPick pick_a2m(const LegArgs& a)
{
    const bool pack = a.spin == 2 && !a.eb;
    auto waves = [&](int r, int ncg) { return (double)nm_rows(a) * ((a.rn + 16 * r - 1) / (16 * r)) * ncg; };
    A2mPick best{16, 1, 1};
    double least = 1e300;
    const int t4 = a.eb ? 3 : tiles_of(a, pack ? 2 : 4), t = tiles_of(a, pack ? 8 : 16);
    if (t4 <= 2) {
        // per 16 rings, relative: more rings per wave share the reads and the chain's latency
        const double k[2][3] = {{1.1, 0.7, 0.62}, {1.88, 1.09, 0.95}};
        for (int i = 0; i < 3; ++i) {
            const double cost = k[t4 - 1][i] * (1 << i) * (waves(1 << i, 1) / 1024.0 + 1.5);
            if (cost < least) {
                least = cost;
                best = {4, 1 << i, t4};
            }
        }
        return best;
    }
    for (int r = 1; r <= 2; ++r)
        for (int c = 1; c <= (a.eb && r == 2 ? 2 : 4); c *= 2) {
            const int ncg = (t + c - 1) / c;
            const double cost = r * (c + (r == 1 ? 0.38 + 0.05 * c : 0.3)) * (waves(r, ncg) / 1024.0 + 1.0);
            if (cost < least) {
                least = cost;
                best = {16, r, c};
            }
        }
    return best;
}

// The same counted row by row: chains below two tiles are mostly remainders.
double l_tiles_exact(const LegArgs& a, int tl)
{
    const double n = a.lmax + 1, q = (a.lmax + 1) / tl;
    return nm_rows(a) / n * (q + 1.0) * (n - 0.5 * q * tl);
}

// map2alm: C tiles of NC columns per wave and TS rows per run, rings split over a
// block's waves or not; c = 0: the LDS kernels of k_leg.hip, which share a recursion tile
// between 64 to 256 columns, pad the batch to their width and the l range to 64 rows
// instead of 128 (narrow lmax, wide batches; FP32 batches that leave the chip idle here).
//  * Few waves: split or the LDS kernels.  Split while its blocks (128 rows x 16 columns)
//    leave the chip room, and past that while it does less work than the LDS kernels, which
//    pad 64-row tiles to 64 or 128 columns but share the recursion.  The lines are those of
//    least regret over 1090 shapes of nside 2 to 512, 5 to 1500 maps (0.3% of the call's time
//    on average; always split 3.4%, always LDS 16%).  Whole calls, split / LDS us: nside 16,
//    lmax 16, 800 IQU sets 131 / 91; nside 16, lmax 47, 300 T maps 49 / 36; nside 64, lmax
//    191, 16 IQU sets 81 / 99; nside 128, lmax 383, 8 IQU sets 168 / 350.
//  * One or two 4-column tiles: runs of 16 rows where that leaves 1024 waves (nside 512, 1
//    IQU set: 830 us against 1385 for 8-row runs and 1400 for 16 columns).
struct M2aPick { int nc, c, ts; bool split; };
M2aPick pick_m2a(const LegArgs& a, int prec)
{
    if (prec == 2 || a.eb) return {16, 0, 8, false};
    const bool f64 = prec == 0;
    const int t = tiles_of(a, a.spin == 2 ? 8 : 16), t4 = tiles_of(a, a.spin == 2 ? 2 : 4);
    if (f64 && t4 <= 2) {
        if (l_tiles(a, 256) >= 1024.0) return {4, 1, 16, false};
        return {4, 1, 8, l_tiles(a, 128) * t4 < 2048.0};
    }
    const double lt = l_tiles(a, 128);
    if (f64 && lt * t < 2048.0) {
        const double blocks = l_tiles_exact(a, 128) * t;
        // 256-column tiles (spin 0) take the LDS kernel longer
        const double room = a.spin == 2 ? 1400.0 : a.ldx % 256 == 0 ? 950.0 : 550.0;
        const double wide = a.ldx == 64 ? 64.0 : (a.ncols + 127) / 128 * 128.0;
        const double lds = l_tiles_exact(a, 64) * 0.5 * wide / (a.spin == 2 ? 8 : 16);
        // the few orders of a level: the LDS kernels split their rings too, with a pass to clear
        // the sums (nside 8, lmax 23, 3000 T maps, immediate iteration: 538 us split, 575 not)
        const bool level = a.mlist && !a.mstep;
        if (level || blocks < room || (0.88 + 14.0 / a.rn) * blocks < lds) return {16, 1, 8, true};
        return {16, 0, 8, false};
    }
    if (!f64 && lt * t < 4096.0) return {16, 0, 8, false};
    // per tile: MFMAs, and the recursion of a wave (FP32 halves only the MFMAs); a wave's
    // set-up costs about eight of its groups of 8 rings
    const double rec = f64 ? 0.35 : (a.spin == 2 ? 1.35 : 1.5), setup = 1.0 + 64.0 / a.rn;
    const double lds = f64 ? 1.53 : (a.spin == 2 ? 1.58 : 1.7);  // per tile of the LDS kernels
    // columns the LDS kernels compute; their narrow forms (FP32) take 0.45 (16 columns) and
    // 0.7 (32) of a full tile's time
    const int nw = f64 ? 0 : narrow(a);
    const double wide = nw == 1 ? 29.0 : nw == 2 ? 45.0 : a.ldx == 64 ? 64.0 : (a.ncols + 127) / 128 * 128.0;
    double least = lds * (wide / (a.spin == 2 ? 8 : 16)) * l_tiles(a, 64) * 0.5;
    M2aPick best{16, 0, 8, false};
    for (int c = 1; c <= (f64 ? 2 : 4); c *= 2) {
        const double cost = (t + c - 1) / c * (c + rec) * lt * setup;
        if (cost < least) {
            least = cost;
            best.c = c;
        }
    }
    return best;
}

template <int SPIN, int C>
hipError_t go_m2a32(const LegArgs& a, hipStream_t st)
{
    const int ncg = (tiles_of(a, SPIN == 2 ? 8 : 16) + C - 1) / C;
    hipLaunchKernelGGL((k_m2a_reg32<SPIN, C>), dim3(blocks_m2a(a, RTL, ncg)), dim3(64), 0, st, a, ncg);
    return hipGetLastError();
}

template <int SPIN, int NC, int C, int TS, bool SPLIT>
hipError_t go_m2a64(const LegArgs& a, hipStream_t st)
{
    const int ncg = (tiles_of(a, SPIN == 2 ? NC / 2 : NC) + C - 1) / C;
    hipLaunchKernelGGL((k_m2a_reg64<SPIN, NC, C, TS, SPLIT>), dim3(blocks_m2a(a, 16 * TS, ncg)),
                       dim3(SPLIT ? 64 * RWAVES : 64), 0, st, a, ncg);
    return hipGetLastError();
}

template <int SPIN, int EB, int NC, int R, int C>
hipError_t go_a2m(const LegArgs& a, hipStream_t st)
{
    const int ncg = (tiles_of(a, SPIN == 2 && EB == 0 ? NC / 2 : NC) + C - 1) / C;
    const int nrt = (a.rn + 16 * R - 1) / (16 * R);
    const int per = nrt * ncg;
    hipLaunchKernelGGL((k_a2m_reg<SPIN, EB, NC, R, C>), dim3(blocks_for(a, per)), dim3(64), 0, st, a, per, nrt);
    return hipGetLastError();
}

template <int SPIN, int EB>
hipError_t a2m_tile(const LegArgs& a, hipStream_t st)
{
    const A2mPick k = pick_a2m(a);
    if constexpr (EB == 0) {
        if (k.nc == 4) {
            if (k.c == 1) return k.r == 1 ? go_a2m<SPIN, EB, 4, 1, 1>(a, st) : k.r == 2 ? go_a2m<SPIN, EB, 4, 2, 1>(a, st) : go_a2m<SPIN, EB, 4, 4, 1>(a, st);
            return k.r == 1 ? go_a2m<SPIN, EB, 4, 1, 2>(a, st) : k.r == 2 ? go_a2m<SPIN, EB, 4, 2, 2>(a, st) : go_a2m<SPIN, EB, 4, 4, 2>(a, st);
        }
        if (k.r == 2 && k.c == 4) return go_a2m<SPIN, EB, 16, 2, 4>(a, st);
    }
    if (k.r == 1) return k.c == 1 ? go_a2m<SPIN, EB, 16, 1, 1>(a, st) : k.c == 2 ? go_a2m<SPIN, EB, 16, 1, 2>(a, st) : go_a2m<SPIN, EB, 16, 1, 4>(a, st);
    return k.c == 1 ? go_a2m<SPIN, EB, 16, 2, 1>(a, st) : go_a2m<SPIN, EB, 16, 2, 2>(a, st);
}

template <int SPIN>
hipError_t m2a_tile(const LegArgs& a, const M2aPick& k, int prec, hipStream_t st)
{
    if (prec == 1) return k.c == 1 ? go_m2a32<SPIN, 1>(a, st) : k.c == 2 ? go_m2a32<SPIN, 2>(a, st) : go_m2a32<SPIN, 4>(a, st);
    if (k.nc == 4) {
        if (k.ts == 16) return go_m2a64<SPIN, 4, 1, 16, false>(a, st);
        return k.split ? go_m2a64<SPIN, 4, 1, 8, true>(a, st) : go_m2a64<SPIN, 4, 1, 8, false>(a, st);
    }
    if (k.split) return go_m2a64<SPIN, 16, 1, 8, true>(a, st);
    return k.c == 1 ? go_m2a64<SPIN, 16, 1, 8, false>(a, st) : go_m2a64<SPIN, 16, 2, 8, false>(a, st);
}

template <int NC2, int NC0>
void go_m2a_pair(const LegArgs& a0, const LegArgs& a2, int spins, hipStream_t st)
{
    const int ncg2 = tiles_of(a2, NC2 / 2), ncg0 = tiles_of(a0, NC0);
    const PairGrid pg(blocks_m2a(a2, 16 * SEG, ncg2), blocks_m2a(a0, 16 * SEG, ncg0), spins);
    hipLaunchKernelGGL((k_m2a_pair<NC2, NC0>), dim3(pg.total), dim3(64 * RWAVES), 0, st, a2, ncg2, pg.first0, a0, ncg0);
}

template <int NC, int R>
void go_a2m_pair(const LegArgs& a0, const LegArgs& a2, int spins, hipStream_t st)
{
    const int nrt = (a2.rn + 16 * R - 1) / (16 * R);
    const int per2 = nrt * tiles_of(a2, NC / 2), per0 = nrt * tiles_of(a0, NC);
    const PairGrid pg(blocks_for(a2, per2), blocks_for(a0, per0), spins);
    hipLaunchKernelGGL((k_a2m_pair<NC, R>), dim3(pg.total), dim3(64), 0, st, a2, per2, pg.first0, a0, per0, nrt);
}

}  // namespace

// A part plan takes these kernels where its own m and all m both ask for them: where the
// whole plan runs the LDS kernels (short chains, wide batches) a part's few waves would pick
// the split form, 12 us more (nside 64, lmax 128, 400 T maps, part 0 of 4: 161 -> 173 us).
bool leg_m2a_reg(const LegArgs& a, int prec)
{
    return pick_m2a(a, prec).c != 0 && (!a.mstep || pick_m2a(by_tiles(a), prec).c != 0);
}

hipError_t launch_leg_m2a_reg(const LegArgs& a, int prec, hipStream_t st)
{
    const M2aPick k = pick_m2a(a, prec);
    return a.spin == 0 ? m2a_tile<0>(a, k, prec, st) : m2a_tile<2>(a, k, prec, st);
}

// Pairing pays while one spin alone leaves the chip part empty: map2alm where spin 2 splits
// its rings (spin 0 then splits too, also where it would not by itself: nside 32, lmax 95, 48
// IQU sets, 75 us with spin 0 in the LDS kernel, 68 as a pair), alm2map up to 8192 waves
// (nside 64, 16 IQU sets).
bool launch_leg_m2a_pair(const LegArgs& a0, const LegArgs& a2, int prec, int spins, hipStream_t st)
{
    if (prec == 2) return launch_leg_m2a_pair_bf16(a0, a2, spins, st);
    if (prec == 1) return !leg_m2a_reg(a0, prec) && !leg_m2a_reg(a2, prec) && launch_leg_m2a_pair_f32(a0, a2, spins, st);
    const M2aPick k0 = pick_m2a(a0, prec), k2 = pick_m2a(a2, prec);
    if (!k2.split || !leg_m2a_reg(a2, prec) || (k0.c != 0 && !k0.split)) return false;
    if (k2.nc == 4) go_m2a_pair<4, 4>(a0, a2, spins, st);
    else if (k0.nc == 4) go_m2a_pair<16, 4>(a0, a2, spins, st);
    else go_m2a_pair<16, 16>(a0, a2, spins, st);
    return true;
}

bool launch_leg_a2m_pair(const LegArgs& a0, const LegArgs& a2, int prec, int spins, hipStream_t st)
{
    if (prec == 2) return launch_leg_a2m_pair_bf16(a0, a2, spins, st);
    if (prec == 1) return launch_leg_a2m_pair_f32(a0, a2, spins, st);
    if (a2.eb) return false;
    const double waves = (double)nm_rows(a2) * ((a2.rn + 15) / 16);
    if (a2.ncols == 2) {
        if (waves > 8192.0) return false;
        if (waves > 4096.0) go_a2m_pair<4, 2>(a0, a2, spins, st);
        else go_a2m_pair<4, 1>(a0, a2, spins, st);
        return true;
    }
    if (waves * tiles_of(a2, 8) > 8192.0) return false;
    go_a2m_pair<16, 1>(a0, a2, spins, st);
    return true;
}

hipError_t launch_leg_a2m_reg(const LegArgs& a, hipStream_t st)
{
    if (a.spin == 0) return a2m_tile<0, 0>(a, st);
    return a.eb == 0 ? a2m_tile<2, 0>(a, st) : a.eb == 1 ? a2m_tile<2, 1>(a, st) : a2m_tile<2, 2>(a, st);
}

}  // namespace sht
