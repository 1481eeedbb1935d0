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
// Bound by the FP64 pipe, which MFMAs and the recursion share; one-wave blocks, since
// a block of four waits with its registers for the longest (10-14% slower).  Measured
// (us per launch, LDS kernels of k_leg.hip -> these):
//   nside 512, 1 map set    alm2map 4507 -> 1355 (spin 2), 1839 -> 726 (spin 0)
//                           map2alm 5211 -> 1665,          1837 -> 876
//   nside 256, 16 map sets  alm2map 1444 -> 627, 487 -> 187; map2alm 1368 -> 773, 429 -> 270
//   nside 512, 125 map sets alm2map 37.2 -> 33.2 ms, 11.1 -> 9.2; map2alm 36.8 -> 35.9, 10.2 -> 9.7
//   FP32, 125 map sets      map2alm 20.8 -> 19.6 ms, 5.9 -> 5.4
#include "leg_rec.h"

namespace sht {
namespace {

constexpr int RWAVES = 4;    // waves of a block that splits its rings
constexpr int RTL = 128;     // map2alm: l per tile (16 segments)
constexpr unsigned SGN = 0x80000000u;

// value of lane ^ 8 within each row of 16 lanes
__device__ __forceinline__ int swap8(int v) { return __builtin_amdgcn_mov_dpp(v, 0x128, 0xf, 0xf, true); }
__device__ __forceinline__ float swap8(float v) { return __int_as_float(swap8(__float_as_int(v))); }
__device__ __forceinline__ double swap8(double v)
{
    return __hiloint2double(swap8(__double2hiint(v)), swap8(__double2loint(v)));
}

// l tiles of RTL rows of order m (none if the plan does not own it)
__device__ __forceinline__ int ntl(const LegArgs& a, int m)
{
    if (m < 0 || m > a.lmax || a.rowoff[m + 1] == a.rowoff[m]) return 0;
    return (a.lmax - lbase(a.spin, m) + RTL) / RTL;
}

// Work order: block b runs on XCD b mod 8; a unit of work (an m, or the pair m,
// lmax - m in map2alm, whose l tiles add up to the same number for every pair) is
// kept on one XCD, units are dealt to the XCDs in turn and start in order of m,
// longest chains first.  With few units (short lists, small lmax) the blocks of one
// unit are spread over the XCDs instead, which would otherwise stand idle.
constexpr int FEW_UNITS = 64;
__host__ __device__ inline int units_m2a(const LegArgs& a) { return a.mlist ? a.nlist : (a.lmax + 2) / 2; }
__device__ __forceinline__ void unit_of(int units, int per, int& unit, int& slot)
{
    const int b = blockIdx.x;
    if (units < FEW_UNITS) {
        unit = b / per;
        slot = b - unit * per;
        return;
    }
    const int pos = b >> 3;
    unit = (pos / per) * 8 + (b & 7);
    slot = pos - (pos / per) * per;
}
int blocks_for(int units, int per) { return (units < FEW_UNITS ? units : (units + 7) / 8 * 8) * per; }

// emitter of one recursion row: its values are A operands at once
template <typename T, int C>
struct RowToMfma {
    using MF = Mfma<T>;
    typename MF::acc (&acc)[C];
    const T (&b)[2][C];   // T_N + T_S, T_N - T_S (spin 2: [Q | Y])
    const T (&bs)[2][C];  // spin 2: the same of [Y | Q]
    template <int R>
    __device__ __forceinline__ void put(T v)
    {
#pragma unroll
        for (int c = 0; c < C; ++c) acc[c] = MF::run(v, b[R & 1][c], acc[c]);
    }
    template <int R>
    __device__ __forceinline__ void put(T p, T q)
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
// A operand from a recursion value
__device__ __forceinline__ void operand(double& o, bool live, double v) { o = zero_unless(live, v); }
__device__ __forceinline__ void operand(float& o, bool live, double v) { o = live ? (float)v : 0.0f; }

// rec_row (same recursion, same values) with the row masked in the operand's format;
// rows past lmax need no mask: their coefficients are zero
template <int R, typename T, int C>
__device__ __forceinline__ void rec_row_reg(Rec<0>& f, const double (&c)[3], RowToMfma<T, C>& em)
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
    T o;
    operand(o, f.k == 0, R == 0 ? f.v0 : f.v1);
    em.template put<R>(o);
}
template <int R, typename T, int C>
__device__ __forceinline__ void rec_row_reg(Rec<2>& f, const double (&c)[3], RowToMfma<T, C>& em)
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
    T p, q;
    operand(p, f.k == 0, R == 0 ? f.a0 : f.a1);
    operand(q, f.k == 0, R == 0 ? f.b0 : f.b1);
    em.template put<R>(p, q);
}

// ============================================================================
// map2alm: A_l = sum over north rings of lambda_l (T_N +- T_S), or the block form of
// spin 2.  Wave: 128 l x C column tiles, all rings from the equator to the first
// significant chunk.  Split: the four waves of a block share one tile and take a
// quarter of its rings each (grids too small to fill the chip); their sums meet in
// LDS in a fixed order.
// The sum over rings runs in the order of k_leg.hip's kernels (chunks of 32 rings
// from the equator, groups of 4 within a chunk), so FP32 results are the same bits.
// ============================================================================
template <typename T, int SPIN, int C, bool SPLIT>
__global__ __launch_bounds__(SPLIT ? 64 * RWAVES : 64, 2) void k_m2a_reg(LegArgs a, int per, int ncg)
{
    constexpr int MS = SPIN == 2 ? 8 : 16;  // columns of one component per tile
    constexpr int CS = SPIN == 0 ? 2 : 4, NCF = SPIN == 0 ? 2 : 3;
    const int lane = threadIdx.x & 63, wave = wave_index();
    const int i = lane & 15, k = lane >> 4;
    const int L = a.lmax;

    int unit, slot;
    unit_of(units_m2a(a), per, unit, slot);
    int lt = slot / ncg;
    const int cg = slot - lt * ncg;
    int m;
    if (a.mlist) {
        if (unit >= a.nlist) return;
        m = a.mlist[unit];
    } else {
        if (2 * unit > L) return;
        const int n0 = ntl(a, unit);
        m = unit;
        if (lt >= n0) {
            lt -= n0;
            m = L - unit;
            if (m == unit) return;
        }
    }
    m = __builtin_amdgcn_readfirstlane(m);
    lt = __builtin_amdgcn_readfirstlane(lt);
    if (lt >= ntl(a, m)) return;
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
        // Rings are taken eight at a time, as two MFMA groups of 4 (n0 eights in the
        // equator chunk, 4 in every other).  FP64: slot k takes rings 2k, 2k + 1 of the
        // eight, so its seeds come as one 16-byte load per array.  FP32: 4u + k, the
        // order of k_leg.hip.
        constexpr bool PAIR = sizeof(T) == 8;
        const int n0 = (a.rn - (nchunk - 1) * RCHUNK + 7) / 8;
        int g0 = 0, g1 = n0 + 4 * (nchunk - 1 - rc0);
        if constexpr (SPLIT) {
            const int len = (g1 + RWAVES - 1) / RWAVES;
            g0 = min(g1, len * wave);
            g1 = min(g1, g0 + len);
        }
        constexpr int NV = SPIN == 0 ? 2 : 4;
        struct Stage {
            double v[NV][2], t[2];  // seed values and 1 - x of the two rings
            int k[2], r;
            T x[2][2][C];           // [ring][north, south][column tile]
        };
        auto load = [&](Stage& s, int g) {
            const int h = g - n0;
            const int r8 = g < n0 ? (nchunk - 1) * RCHUNK + 8 * g : (nchunk - 2 - (h >> 2)) * RCHUNK + 8 * (h & 3);
            s.r = r8 + (PAIR ? 2 * k : k);
            if constexpr (PAIR) {
                const unsigned o = sofs + (unsigned)min(s.r, a.rn - 2);  // rn is even
#pragma unroll
                for (int q = 0; q < NV; ++q) {
                    const double2 d = *reinterpret_cast<const double2*>(mu + q * a.seedstride + o);
                    s.v[q][0] = d.x;
                    s.v[q][1] = d.y;
                }
                const int2 kd = *reinterpret_cast<const int2*>(kk + o);
                s.k[0] = kd.x;
                s.k[1] = kd.y;
            }
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int rr = PAIR ? min(s.r, a.rn - 2) + u : min(s.r + 4 * u, a.rn - 1);
                if constexpr (!PAIR) {
                    const unsigned o = sofs + (unsigned)rr;
#pragma unroll
                    for (int q = 0; q < NV; ++q) s.v[q][u] = (mu + q * a.seedstride)[o];
                    s.k[u] = kk[o];
                }
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
            double w = m2a_weight(a, s.r + (PAIR ? u : 4 * u));
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
                    bs[0][c] = swap8(b[0][c]);
                    bs[1][c] = swap8(b[1][c]);
                }
            }
            if constexpr (u == 1) load(s, gnext);
            __builtin_amdgcn_sched_barrier(0);
            static_for<0, SEG>([&](auto ti) {
                constexpr int t = decltype(ti)::v;
                RowToMfma<T, C> em{acc[t], b, bs};
                rec_row_reg<t>(f, cf[t], em);
            });
        };
        if (g0 < g1) {
            Stage s;
            load(s, g0);
            for (int g = g0; g < g1; ++g) {
                run(s, IC<0>{}, 0);
                run(s, IC<1>{}, min(g + 1, g1 - 1));
            }
        }
    }

    T* A = aptr<T>(a, SPIN == 2 ? (second ? 2 : 1) : 0) + row0 * a.ldx;
    auto store = [&](int t, int c, const typename MF::acc& v) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int l = l0 + SEG * MF::row(lane, q) + t;
            if (l <= L) A[(int64_t)(l - lb) * a.ldx + col + MS * c] = v[q];
        }
    };
    if constexpr (!SPLIT) {
#pragma unroll
        for (int t = 0; t < SEG; ++t)
#pragma unroll
            for (int c = 0; c < C; ++c) store(t, c, acc[t][c]);
    } else {
        // partial sums [wave][row][lane]; wave w adds and stores rows 2w, 2w + 1
        static_assert(C == 1, "LDS holds the partial sums of one column tile");
        __shared__ typename MF::acc part[RWAVES][SEG][64];
#pragma unroll
        for (int t = 0; t < SEG; ++t) part[wave][t][lane] = acc[t][0];
        __syncthreads();
#pragma unroll
        for (int q = 0; q < SEG / RWAVES; ++q) {
            const int t = wave * (SEG / RWAVES) + q;
            typename MF::acc v = part[0][t][lane];
#pragma unroll
            for (int w = 1; w < RWAVES; ++w) v += part[w][t][lane];
            store(t, 0, v);
        }
    }
}

// ============================================================================
// alm2map: T_r = sum over l of lambda_l A_l.  Wave: R x 16 rings x C column tiles;
// slot k takes the k-th quarter of the l range (whole 8-row segments), row i a ring.
// Each step needs one row of coefficients and of A per quarter, read PD steps ahead.
// ============================================================================
// EB = 1 (E only), 2 (B only): plain columns as in spin 0 (tiles of 8 map sets), even
// and odd rows of P and M apart; the other component is neither read nor multiplied.
template <int SPIN, int EB, int R, int C>
__global__ __launch_bounds__(64, 2) void k_a2m_reg(LegArgs a, int per, int nrt)
{
    constexpr bool PACK = SPIN == 2 && EB == 0;  // S and D columns in one tile
    constexpr int MS = PACK ? 8 : 16;
    constexpr int NA = SPIN == 2 && EB ? 4 : 2;
    constexpr int CS = SPIN == 0 ? 2 : 4;
    constexpr int PD = 4;
    static_assert(SEG % PD == 0, "the operand buffers cycle within a segment");
    constexpr int CQ = SEG * CS + 4;  // doubles per quarter of a coefficient block (padded)
    __shared__ alignas(16) double ctab[2][4 * CQ];
    const int lane = threadIdx.x;
    const int i = lane & 15, k = lane >> 4;
    const int L = a.lmax;

    int unit, slot;
    unit_of(nm_rows(a), per, unit, slot);
    if (unit >= nm_rows(a)) return;
    const int m = a.mlist ? __builtin_amdgcn_readfirstlane(a.mlist[unit]) : unit;
    const int cg = slot / nrt, rt = slot - cg * nrt;
    if (cg * C * MS >= a.ncols) return;
    const int lb = lbase(SPIN, m);
    const int r0 = rt * 16 * R;

    const int j = PACK ? (i & 7) : i;
    const int col = cg * (C * MS) + j;  // tile c of the wave: col + MS c; C MS divides ldx
    const bool second = PACK && i >= 8;

    // first segment with a significant value on these rings
    int lsig = L + 1;
    if (lb <= L)
        for (int c = r0 / RCHUNK; c < min(a.nrc, (r0 + 16 * R + RCHUNK - 1) / RCHUNK); ++c)
            lsig = min(lsig, a.lsig[(int64_t)m * a.nrc + c]);
    lsig = __builtin_amdgcn_readfirstlane(lsig);

    typedef v4d acc_t;
    acc_t acc[NA][R][C];  // spin 0: even, odd rows; spin 2: P and M products; EB: P even, odd, M even, odd
#pragma unroll
    for (int h = 0; h < NA; ++h)
#pragma unroll
        for (int q = 0; q < R; ++q)
#pragma unroll
            for (int c = 0; c < C; ++c) acc[h][q][c] = acc_t{0, 0, 0, 0};

    if (lsig <= L) {
        const int s0 = (lsig - lb) / SEG, nseg = (L - lb) / SEG - s0 + 1;
        const int nb = (nseg + 3) / 4;               // segments per quarter
        const int nrow = L - lb;                      // last row of this m
        const int64_t row0 = a.rowoff[m];
        int t0 = SEG * (s0 + nb * k);                 // this lane's current row
        double v0[R], v1[R], w0[R], w1[R], x[R];      // spin 2: P and M at rows t, t + 1
        int e[R];
#pragma unroll
        for (int q = 0; q < R; ++q) {
            const int r = min(r0 + 16 * q + i, a.rn - 1);
            const int64_t s = a.seedoff[m] + (int64_t)min(s0 + nb * k, nrow / SEG) * a.rn + r;
            v0[q] = a.mu[s];
            v1[q] = a.mu[a.seedstride + s];
            if constexpr (SPIN == 2) {
                w0[q] = a.mu[2 * a.seedstride + s];
                w1[q] = a.mu[3 * a.seedstride + s];
            }
            e[q] = a.kk[s];
            x[q] = a.rings[r].omz;
            // rows past lmax stay exactly zero: they start so here, and the coefficients
            // of later ones are zero
            if (t0 + 1 > nrow) v1[q] = w1[q] = 0.0;
            if (t0 > nrow) {
                v0[q] = w0[q] = 0.0;
                e[q] = 0;
            }
        }
        // rows t .. t + PD - 1 of A (spin 2: E in one half of the lanes, B' in the other)
        double st[PD][C];
        int tl = t0;                    // row the next load takes; the last row repeats
        const int64_t ldx = a.ldx;
        const double* pa = aptr<double>(a, SPIN == 2 ? (second || EB == 2 ? 2 : 1) : 0) + (row0 + min(t0, nrow)) * ldx + col;
        auto load = [&](double (&s)[C]) {
#pragma unroll
            for (int c = 0; c < C; ++c) s[c] = pa[MS * c];
            pa += tl < nrow ? ldx : 0;
            ++tl;
        };
        // coefficients of the 8 rows a block of steps produces, per quarter: one
        // 16-byte load per lane and block, handed round through the wave's own LDS
        double2* cw = reinterpret_cast<double2*>(ctab[0]) + k * (CQ / 2) + (CS == 4 ? i : (i & 7));
        const double* cr = ctab[0] + k * CQ;
        const double2* cg2 = reinterpret_cast<const double2*>(a.coef + row0 * CS);
        auto load_coef = [&](int t) {
            const int row = t + 2 + (CS == 4 ? (i >> 1) : (i & 7)), rr = min(row, nrow);
            double2 c = cg2[CS == 4 ? 2 * rr + (i & 1) : rr];
            if (row > nrow) c = make_double2(0.0, 0.0);
            return c;
        };
        double2 cnext = load_coef(t0);
        // Packed operands of row t: d = S or D; the mirror sign s_l = (-1)^t (up to the
        // sign of the first row, applied to the southern sums at the end) goes to the D
        // half of P's operand and the S half of M's.
        const double one = second ? -1.0 : 1.0;
        const unsigned sg0 = second ? SGN : 0u, sg1 = second ? 0u : SGN;
#pragma unroll
        for (int t = 0; t < PD; ++t) load(st[t]);
        for (int n = 0; n < nb; ++n, t0 += SEG) {
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            cw[(n & 1) * 2 * CQ] = cnext;
            cnext = load_coef(t0 + SEG);
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            const double* cb = cr + (n & 1) * 4 * CQ;
            bool any = false;  // a lane carries an exponent (they never grow)
#pragma unroll
            for (int q = 0; q < R; ++q) any |= e[q] > 0;
            any = __any(any);
            static_for<0, SEG>([&](auto ti) {
                constexpr int t = decltype(ti)::v;
                const double(&s)[C] = st[t % PD];
                const double c0 = cb[CS * t], c1 = cb[CS * t + 1], c2 = SPIN == 2 ? cb[CS * t + 2] : 0.0;
                double b0[C], b1[C];
#pragma unroll
                for (int c = 0; c < C; ++c) {
                    if constexpr (PACK) {
                        const double d = fma(s[c], one, swap8(s[c]));  // S = E + B', D = E - B'
                        b0[c] = t & 1 ? flip(d, sg0) : d;
                        b1[c] = t & 1 ? flip(d, sg1) : d;
                    } else {
                        b0[c] = s[c];
                    }
                }
                load(st[t % PD]);
                double vn[R], wn[R];  // row t + 2
#pragma unroll
                for (int q = 0; q < R; ++q) {
                    const double p = zero_unless(e[q] == 0, v0[q]);
#pragma unroll
                    for (int c = 0; c < C; ++c) {
                        acc_t& d = acc[PACK ? 0 : (t & 1)][q][c];
                        d = Mfma<double>::run(p, b0[c], d);
                    }
                    if constexpr (SPIN == 2) {
                        const double g = zero_unless(e[q] == 0, w0[q]);
#pragma unroll
                        for (int c = 0; c < C; ++c) {
                            acc_t& d = acc[PACK ? 1 : 2 + (t & 1)][q][c];
                            d = Mfma<double>::run(g, PACK ? b1[c] : b0[c], d);
                        }
                    }
                    const double ax = fma(-c0, x[q], c0);
                    if constexpr (SPIN == 0) {
                        vn[q] = ax * v1[q] - c1 * v0[q];
                    } else {
                        vn[q] = (ax + c1) * v1[q] - c2 * v0[q];
                        wn[q] = (ax - c1) * w1[q] - c2 * w0[q];
                    }
                }
                if (__builtin_expect(any, 0)) {
#pragma unroll
                    for (int q = 0; q < R; ++q) {
                        const double big = SPIN == 0 ? fabs(vn[q]) : fmax(fabs(vn[q]), fabs(wn[q]));
                        if (e[q] > 0 && big > RESCALE_AT) {
                            vn[q] *= SCALE_DOWN;
                            v1[q] *= SCALE_DOWN;
                            if constexpr (SPIN == 2) {
                                wn[q] *= SCALE_DOWN;
                                w1[q] *= SCALE_DOWN;
                            }
                            --e[q];
                        }
                    }
                }
#pragma unroll
                for (int q = 0; q < R; ++q) {
                    v0[q] = v1[q];
                    v1[q] = vn[q];
                    if constexpr (SPIN == 2) {
                        w0[q] = w1[q];
                        w1[q] = wn[q];
                    }
                }
            });
        }
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
            for (int v = 0; v < 4; ++v) {
                const int r = r0 + 16 * q + Mfma<double>::row(lane, v);
                const double g = acc[0][q][c][v], h = acc[1][q][c][v];
                double n, s, yn = 0.0, ys = 0.0;
                if constexpr (SPIN == 0) {
                    n = g + h;
                    s = g - h;
                } else if constexpr (PACK) {
                    // lanes of S columns hold (G_N, G_S), lanes of D columns (H_S, H_N)
                    const double go = swap8(g), ho = swap8(h);
                    n = flip(second ? -0.5 * (go - h) : -0.5 * (g + ho), second ? usg : 0u);
                    s = flip(second ? -0.5 * (ho - g) : -0.5 * (h + go), (second ? usg : 0u) ^ po);
                } else {
                    const double u = acc[NA - 2][q][c][v], w = acc[NA - 1][q][c][v];
                    const double pn = g + h, mn = u + w, ps = u - w, ms = g - h;  // P_S = s M_N, M_S = s P_N
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
                if constexpr (SPIN == 2 && EB) {
                    X1[(int64_t)r * a.ldx + MS * c] = yn;
                    if (rs != r) X1[(int64_t)rs * a.ldx + MS * c] = ys;
                }
            }
}

// ----------------------------------------------------------------------------
// Choice of kernel and tile
// ----------------------------------------------------------------------------
// Times below are in units of the MFMAs of one column tile (of one wave's rows) and
// fitted on one MI355X at nside 64..512 with 1 to 1000 map sets.

int tiles_of(const LegArgs& a, int ms) { return (a.ncols + ms - 1) / ms; }

// m values and their l tiles of `tl` rows, the owned m only approximately (parts)
double l_tiles(const LegArgs& a, int tl)
{
    const double n = a.lmax + 1;
    return (a.mlist ? a.nlist / n : 1.0) * n * 0.5 * (n / tl + 1.0);
}

// alm2map: R x 16 rings and C tiles per wave; the recursion and the coefficient reads
// of a wave cost as much as 0.5 (R = 1) or 0.37 (R = 2) of a tile's MFMAs, and the
// last waves of a launch run alone for about one more wave (chains of the first m are
// twice the mean).
struct A2mPick { int r, c; };
A2mPick pick_a2m(const LegArgs& a)
{
    const int t = tiles_of(a, a.spin == 2 && !a.eb ? 8 : 16);
    A2mPick best{1, 1};
    double least = 1e300;
    for (int r = 1; r <= 2; ++r)
        for (int c = 1; c <= (a.eb && r == 2 ? 2 : 4); c *= 2) {
            const int ncg = (t + c - 1) / c;
            const double waves = (double)nm_rows(a) * ((a.rn + 16 * r - 1) / (16 * r)) * ncg;
            const double cost = r * (c + (r == 1 ? 0.5 : 0.37)) * (waves / 1024.0 + 1.0);
            if (cost < least) {
                least = cost;
                best = {r, c};
            }
        }
    return best;
}

// map2alm: C tiles per wave, or 9: one tile, rings split over the block's waves;
// 0: the LDS kernels of k_leg.hip, which share a recursion tile between 64 to 256
// columns, pad the batch to their width and the l range to 64 rows instead of 128.
int pick_m2a(const LegArgs& a, int prec)
{
    if (prec == 2 || a.eb) return 0;
    const bool f64 = prec == 0;
    const int t = tiles_of(a, a.spin == 2 ? 8 : 16);
    const double lt = l_tiles(a, 128);
    if (lt * t < 4096.0) return f64 ? 9 : 0;
    // per tile: MFMAs, and the recursion of a wave; FP32 halves only the MFMAs
    const double rec = f64 ? 0.5 : (a.spin == 2 ? 1.35 : 1.7);
    const double lds = (f64 ? 1.28 : 1.4) * (a.ldx / (a.spin == 2 ? 8 : 16)) * l_tiles(a, 64) * 0.5;
    int best = 0;
    double least = lds;
    for (int c = 1; c <= (f64 ? 2 : 4); c *= 2) {
        const double cost = (t + c - 1) / c * (c + rec) * lt;
        if (cost < least) {
            least = cost;
            best = c;
        }
    }
    return best;
}

template <typename T, int SPIN, int C, bool SPLIT>
hipError_t go_m2a(const LegArgs& a, hipStream_t st)
{
    constexpr int MS = SPIN == 2 ? 8 : 16;
    const int ncg = (tiles_of(a, MS) + C - 1) / C;
    // l tiles per unit: of one m (list), or of a pair m, lmax - m: ceil(x / n) + ceil(y / n)
    // with x + y <= lmax + 2 rows
    const int tiles = a.mlist ? (a.lmax + RTL) / RTL : (a.lmax + 2 + 2 * (RTL - 1)) / RTL;
    const int per = tiles * ncg;
    const dim3 grid((unsigned)blocks_for(units_m2a(a), per));
    hipLaunchKernelGGL((k_m2a_reg<T, SPIN, C, SPLIT>), grid, dim3(SPLIT ? 64 * RWAVES : 64), 0, st, a, per, ncg);
    return hipGetLastError();
}

template <int SPIN, int EB, int R, int C>
hipError_t go_a2m(const LegArgs& a, hipStream_t st)
{
    constexpr int MS = SPIN == 2 && EB == 0 ? 8 : 16;
    const int ncg = (tiles_of(a, MS) + C - 1) / C;
    const int nrt = (a.rn + 16 * R - 1) / (16 * R);
    const int per = nrt * ncg;
    const dim3 grid((unsigned)blocks_for(nm_rows(a), per));
    hipLaunchKernelGGL((k_a2m_reg<SPIN, EB, R, C>), grid, dim3(64), 0, st, a, per, nrt);
    return hipGetLastError();
}

template <int SPIN, int EB>
hipError_t a2m_tile(const LegArgs& a, hipStream_t st)
{
    const A2mPick k = pick_a2m(a);
    if (k.r == 1) return k.c == 1 ? go_a2m<SPIN, EB, 1, 1>(a, st) : k.c == 2 ? go_a2m<SPIN, EB, 1, 2>(a, st) : go_a2m<SPIN, EB, 1, 4>(a, st);
    if constexpr (EB == 0)
        if (k.c == 4) return go_a2m<SPIN, EB, 2, 4>(a, st);
    return k.c == 1 ? go_a2m<SPIN, EB, 2, 1>(a, st) : go_a2m<SPIN, EB, 2, 2>(a, st);
}

template <int SPIN>
hipError_t m2a_tile(const LegArgs& a, int prec, int c, hipStream_t st)
{
    if (prec == 1)
        return c == 1 ? go_m2a<float, SPIN, 1, false>(a, st) : c == 2 ? go_m2a<float, SPIN, 2, false>(a, st) : go_m2a<float, SPIN, 4, false>(a, st);
    return c == 9 ? go_m2a<double, SPIN, 1, true>(a, st) : c == 1 ? go_m2a<double, SPIN, 1, false>(a, st) : go_m2a<double, SPIN, 2, false>(a, st);
}

}  // namespace

bool leg_m2a_reg(const LegArgs& a, int prec) { return pick_m2a(a, prec) != 0; }

hipError_t launch_leg_m2a_reg(const LegArgs& a, int prec, hipStream_t st)
{
    const int c = pick_m2a(a, prec);
    return a.spin == 0 ? m2a_tile<0>(a, prec, c, st) : m2a_tile<2>(a, prec, c, st);
}

hipError_t launch_leg_a2m_reg(const LegArgs& a, hipStream_t st)
{
    if (a.spin == 0) return a2m_tile<0, 0>(a, st);
    return a.eb == 0 ? a2m_tile<2, 0>(a, st) : a.eb == 1 ? a2m_tile<2, 1>(a, st) : a2m_tile<2, 2>(a, st);
}

}  // namespace sht
