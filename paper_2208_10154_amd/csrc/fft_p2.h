// Ring FFTs of compile-time lengths: power-of-two rings and Bluestein convolutions,
// run by k_fft.hip's shared launch; the passes, the Bluestein step and the fold /
// unfold also serve the four-step kernels (k_fft_four.hip).  Each translation unit
// gets its own copy (internal linkage).
//
// Every equatorial-belt ring of a HEALPix grid has N = 4 nside pixels, a power of
// two for the usual resolutions, and those rings hold two thirds of the pixels.
// For them the length is a template parameter, so every stride, pass count and
// LDS offset below is a compile-time constant: the index arithmetic that the
// runtime-length kernels (k_fft.hip) spend most of their instructions on folds
// into immediate offsets, and what remains is the butterflies themselves.
//
// Transform: two real maps are packed as z = a + i b (forward) and the length-N
// DFT is a Stockham autosort FFT of radix-8 passes with one final radix-2, -4 or
// -8 pass.  Each thread owns 8 values of one sequence: the first pass reads them
// straight from global memory (forward) or gathers them from the m-major
// coefficients (inverse), later passes exchange through LDS, and the last pass
// leaves its outputs in natural order.  The FFT mapping is that of the paper
// (Sec. 2.1 eq. "mm", Appendix A.1): T_m = e^{-i m phi0} F_{m mod N} forward, and
// C_j = sum_{m = j} c_m + sum_{m >= 1, -m = j} conj(c_m), c_m = e^{i m phi0} T_m,
// backward (mod N), with the inverse DFT taken as conj(DFT(conj C)).
#pragma once
#include "fft_internal.h"

namespace sht {
namespace {

__device__ __forceinline__ double2 cmul(double2 a, double2 b)
{
    return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ double2 cadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ double2 csub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }

// forward DFTs (e^{-2 pi i jk/R}) of R values in registers, natural order out
__device__ __forceinline__ void dft2(double2* v)
{
    const double2 t = v[0];
    v[0] = cadd(t, v[1]);
    v[1] = csub(t, v[1]);
}
__device__ __forceinline__ void dft4(double2* v)
{
    const double2 a0 = cadd(v[0], v[2]), a1 = csub(v[0], v[2]);
    const double2 a2 = cadd(v[1], v[3]), a3 = csub(v[1], v[3]);
    v[0] = cadd(a0, a2);
    v[2] = csub(a0, a2);
    v[1] = make_double2(a1.x + a3.y, a1.y - a3.x);  // a1 - i a3
    v[3] = make_double2(a1.x - a3.y, a1.y + a3.x);  // a1 + i a3
}
// radix 8 by decimation in frequency: X_{2q} = DFT4(x_n + x_{n+4}),
// X_{2q+1} = DFT4((x_n - x_{n+4}) W^n), W = e^{-2 pi i/8}
__device__ __forceinline__ void dft8(double2* v)
{
    constexpr double H = 0.7071067811865476;  // 1/sqrt(2), correctly rounded
    double2 a[4], b[4];
#pragma unroll
    for (int n = 0; n < 4; ++n) {
        a[n] = cadd(v[n], v[n + 4]);
        b[n] = csub(v[n], v[n + 4]);
    }
    b[1] = make_double2(H * (b[1].x + b[1].y), H * (b[1].y - b[1].x));    // * (1 - i)/sqrt(2)
    b[2] = make_double2(b[2].y, -b[2].x);                                  // * -i
    b[3] = make_double2(H * (b[3].y - b[3].x), -H * (b[3].x + b[3].y));   // * (-1 - i)/sqrt(2)
    dft4(a);
    dft4(b);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        v[2 * q] = a[q];
        v[2 * q + 1] = b[q];
    }
}
// the same with v[4..7] = 0 (zero padding of the chirp transform)
__device__ __forceinline__ void dft8_low(double2* v)
{
    constexpr double H = 0.70710678118654752440;
    double2 a[4], b[4];
#pragma unroll
    for (int n = 0; n < 4; ++n) a[n] = v[n];
    b[0] = v[0];
    b[1] = make_double2(H * (v[1].x + v[1].y), H * (v[1].y - v[1].x));    // * (1 - i)/sqrt(2)
    b[2] = make_double2(v[2].y, -v[2].x);                                  // * -i
    b[3] = make_double2(H * (v[3].y - v[3].x), -H * (v[3].x + v[3].y));   // * (-1 - i)/sqrt(2)
    dft4(a);
    dft4(b);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        v[2 * q] = a[q];
        v[2 * q + 1] = b[q];
    }
}
template <int R>
__device__ __forceinline__ void dftr(double2* v)
{
    if constexpr (R == 2) dft2(v);
    else if constexpr (R == 4) dft4(v);
    else dft8(v);
}

template <int LOGN>
struct P2 {
    static constexpr int N = 1 << LOGN;
    static constexpr int E = 8;                      // values per thread
    static constexpr int T = N / E;                  // threads per sequence
    // sequences (map pairs) per workgroup: 4096 values (two rings of 2048) per
    // workgroup, at most 16 pairs (the map pairs of the narrowest chunk, 32 map
    // sets).  Two or more pairs give every coefficient row access 64 contiguous
    // bytes or more (a single pair's 32 bytes per row leave every access its own
    // partial line and page translation).
    static constexpr int S = (4096 / N) < 1 ? 1 : ((4096 / N) > 16 ? 16 : 4096 / N);
    static constexpr int LOGS = S == 1 ? 0 : (S == 2 ? 1 : (S == 4 ? 2 : (S == 8 ? 3 : 4)));
    static constexpr int NTH = S * T;                // threads per workgroup
    static constexpr int NP = (LOGN + 2) / 3;        // passes
    static constexpr int LOGRL = LOGN - 3 * (NP - 1);  // log2 of the last radix (1..3)
    static constexpr int SEQ = N + N / 8;            // LDS slots per sequence
    static constexpr int LDS_BYTES = S * SEQ * 16;
};

// LDS position of element pos at the boundary after pass P (radix 8, stride
// 8^P between the values of one butterfly).  After the first pass a thread's
// outputs are 8 consecutive slots, after the second 8 runs of 8 lanes, 64
// slots apart: one pad slot per 8 (resp. 8 per 64) spreads those over the
// banks.  Later boundaries are written in runs of >= 64 lanes and need none.
template <int P>
__device__ __forceinline__ int padp(int pos)
{
    if constexpr (P == 0) return pos + (pos >> 3);
    else if constexpr (P == 1) return pos + ((pos >> 6) << 3);
    else return pos;
}

template <int LOGN, int PASS>
struct Pass {
    using C = P2<LOGN>;
    static constexpr bool LAST = (PASS == C::NP - 1);
    static constexpr int LOGR = LAST ? C::LOGRL : 3;
    static constexpr int R = 1 << LOGR;
    static constexpr int B = 8 / R;                  // butterflies per thread
    static constexpr int LOGNS = 3 * PASS;
    static constexpr int NS = 1 << LOGNS;            // product of the earlier radices
    static constexpr int TWS = 2 * (C::N >> (LOGNS + LOGR));  // twiddle index step in e^{-i pi t/N}
};

// twiddles of pass PASS (>= 1): w^{r k}, w = e^{-2 pi i/(NS R)}, k = j mod NS.
// One table load per butterfly (w^k); the other powers are products.  The
// gathers, not the arithmetic, were the latency of a pass: one load instead of
// seven cut the ring FFT time by a fifth to a quarter, and the products add a few
// ulp to twiddles used once.
template <int LOGN, int PASS>
__device__ __forceinline__ void load_twiddles(double2 (&w)[8], int tl, const double2* tw)
{
    using Q = Pass<LOGN, PASS>;
#pragma unroll
    for (int b = 0; b < Q::B; ++b) {
        const int k = (tl + P2<LOGN>::T * b) & (Q::NS - 1);
#pragma unroll
        for (int r = 1; r < Q::R; ++r)
            w[b * Q::R + r] = r == 1 ? tw[Q::TWS * k] : cmul(w[b * Q::R + r - 1], w[b * Q::R + 1]);
    }
}

// Runs passes PASS..NP-1 on the values in v (inputs of pass PASS, twiddles w
// already loaded).  On return v holds the last pass's outputs: value b*R + r is
// element tl + T*b + r*N/R of the transform.  LOW: the inputs v[4..7] are zero.
template <int LOGN, int PASS, bool LOW = false>
__device__ __forceinline__ void run_passes(double2 (&v)[8], double2 (&w)[8], double2* sb, int tl, const double2* tw)
{
    using C = P2<LOGN>;
    using Q = Pass<LOGN, PASS>;
    if constexpr (PASS > 0) {
#pragma unroll
        for (int b = 0; b < Q::B; ++b) {
#pragma unroll
            for (int r = 1; r < Q::R; ++r) v[b * Q::R + r] = cmul(v[b * Q::R + r], w[b * Q::R + r]);
        }
    }
#pragma unroll
    for (int b = 0; b < Q::B; ++b) {
        if constexpr (LOW) dft8_low(v);
        else dftr<Q::R>(v + b * Q::R);
    }
    if constexpr (!Q::LAST) {
        using Q2 = Pass<LOGN, PASS + 1>;
        load_twiddles<LOGN, PASS + 1>(w, tl, tw);  // in flight across the exchange
        if constexpr (PASS > 0) __syncthreads();    // earlier readers of sb are done
        // outputs y[(j - k) R + k + r NS] (radix 8, one butterfly per thread)
        {
            const int j = tl, k = j & (Q::NS - 1);
            const int pos = (j - k) * 8 + k;
#pragma unroll
            for (int r = 0; r < 8; ++r) sb[padp<PASS>(pos + r * Q::NS)] = v[r];
        }
        __syncthreads();
#pragma unroll
        for (int b = 0; b < Q2::B; ++b) {
#pragma unroll
            for (int r = 0; r < Q2::R; ++r)
                v[b * Q2::R + r] = sb[padp<PASS>(tl + C::T * b + r * (C::N / Q2::R))];
        }
        run_passes<LOGN, PASS + 1>(v, w, sb, tl, tw);
    }
}

// Work item of workgroup pos of the cnt workgroups of a class (cnt = components x
// ring groups x pair groups): workgroups are dealt to the 8 XCDs round-robin, so pos is
// remapped to give each XCD one contiguous range (neighbouring pair groups of a
// ring, which write adjacent columns of the same m-major rows, then share an L2).
// Only groups holding map sets of the chunk are launched: the ring coefficient
// columns of the padding are never read into a result (every later step treats the
// columns of a map set on their own, and pairs the two map sets of one FFT sequence
// only with each other).
struct Item {
    int ring, pair0, comp;
    // workgroups of several rings: the group's rings (left of them) and log2 of the
    // sequences per ring
    const int* rings;
    int left, lgp;
    int direct;  // every ring of the class: cut below its length
};
__device__ __forceinline__ bool work_item(const FftWork& w, int cnt, int pos, int comp0, Item& it)
{
    const int q = cnt >> 3, r = cnt & 7, x = pos & 7, y = pos >> 3;
    if (y >= q + (x < r ? 1 : 0)) return false;  // a class starts on a multiple of 8
    const int idx = x * q + min(x, r) + y;
    const int ngr = (w.nrings + w.rpw - 1) / w.rpw, per = ngr * w.groups;
    const int comp = idx / per, rem = idx - comp * per;
    const int gi = rem / w.groups, ri = gi * w.rpw;
    it = Item{w.rings[ri], (rem - gi * w.groups) << w.lgp, comp0 + comp, w.rings + ri, w.nrings - ri, w.lgp, w.direct};
    return true;
}
__host__ __device__ inline int work_count(const FftWork& w, int ncompl)
{
    return (w.nrings + w.rpw - 1) / w.rpw * w.groups * ncompl;
}
// minlg: least log2 of the sequences per ring of the compile-time kinds (ONE_RING:
// every workgroup serves one ring)
constexpr int ONE_RING = 31;
inline FftWork work_of(const FftArgs& a, const FftClass& c, int minlg = ONE_RING)
{
    const int used = (a.nmaps + 1) / 2;
    int lgs = 0, lgp = c.kind < FFT_P2 ? ONE_RING : minlg;
    while ((1 << lgs) < c.nseq) ++lgs;
    while (lgp < lgs && (1 << lgp) < used) ++lgp;
    lgp = std::min(lgp, lgs);
    const int per = 1 << lgp;
    return FftWork{c.rings, c.nrings, (used + per - 1) / per, c.nseq >> lgp, lgp, c.direct};
}
// Sequence seq of a workgroup: its ring and map pair.  dead: past the class's rings
// (the last ring stands in for the loads, nothing is stored).
struct Seq {
    int ring, pair;
    bool dead;
};
template <bool MULTI>
__device__ __forceinline__ Seq seq_of(const Item& it, int seq)
{
    if constexpr (MULTI) {
        const int slot = seq >> it.lgp;
        return Seq{it.rings[min(slot, it.left - 1)], it.pair0 + (seq & ((1 << it.lgp) - 1)), slot >= it.left};
    } else {
        return Seq{it.ring, it.pair0 + seq, false};
    }
}

// m values per thread and batch in the unfolding (loads of a batch issued first)
constexpr int MB = 8;

template <typename XT>
__device__ __forceinline__ void store4(XT* p, double2 ta, double2 tb)
{
    if constexpr (sizeof(XT) == 4) {
        *reinterpret_cast<float4*>(p) = make_float4((float)ta.x, (float)ta.y, (float)tb.x, (float)tb.y);
    } else {
        reinterpret_cast<double2*>(p)[0] = ta;
        reinterpret_cast<double2*>(p)[1] = tb;
    }
}
template <typename XT>
__device__ __forceinline__ void load4(const XT* p, double2& ta, double2& tb)
{
    if constexpr (sizeof(XT) == 4) {
        const float4 f = *reinterpret_cast<const float4*>(p);
        ta = make_double2(f.x, f.y);
        tb = make_double2(f.z, f.w);
    } else {
        ta = reinterpret_cast<const double2*>(p)[0];
        tb = reinterpret_cast<const double2*>(p)[1];
    }
}

// ----------------------------------------------------------------------------
// Rings whose length n has a prime factor above 7 (most polar-cap rings):
// Bluestein's chirp-z form, y_j = w_j sum_i (x_i w_i) conj(w_{j-i}) with
// w_i = e^{-i pi i^2/n}, the circular convolution taken through a power-of-two
// length M >= 2n - 1 with the compile-time passes above.  The kernel spectrum
// bhat (FFT of conj(w) placed circularly, times 1/M) is precomputed per length.
// The last pass of a length-M transform leaves element tl + T k in register
// slot b R + r with k = b + r B, exactly the pass-0 inputs of the next
// transform: the two transforms are chained in registers.
// ----------------------------------------------------------------------------

// m = m0, m0 + dm, ...: keeps j = m mod n and ph = (m s) mod 2n (s is 0 or 1; m0, dm < 2^16)
struct MStep {
    int j, ph, dj, dph, n, two_n;
    // m mod n and m mod 2n through the quotient in single precision, off by one at most
    __device__ __forceinline__ void mod(int m, int& r, int& r2) const
    {
        int q = (int)((float)m * __builtin_amdgcn_rcpf((float)n));
        r = m - q * n;
        if (r < 0) { r += n; --q; }
        if (r >= n) { r -= n; ++q; }
        r2 = r + ((q & 1) ? n : 0);
    }
    __device__ __forceinline__ MStep(int m0, int dm, int n_, int s)
    {
        n = n_;
        two_n = 2 * n_;
        mod(m0, j, ph);
        mod(dm, dj, dph);
        if (!s) ph = dph = 0;
    }
    __device__ __forceinline__ void next()
    {
        j += dj;
        if (j >= n) j -= n;
        ph += dph;
        if (ph >= two_n) ph -= two_n;
    }
};

// Fold of one map pair's rows m <= lmax < n onto the bins of a ring: with
// c_m = e^{+i m phi0} T_m of both maps, d_m = c^a_m + i c^b_m and e_m = conj(c^a_m) +
// i conj(c^b_m), bin j takes d_j and, for j >= 1, e_{n-j}.  The rows j and n - j give the
// bins j and n - j, so a thread that holds both writes each bin once, with no clearing,
// no atomics and no barrier between terms (bin 0 goes with bin n/2).  The phase of row
// n - j is (-1)^s times the conjugate of that of row j: one table load for both.  FP32
// rows load both, as the table's rounding of the second decides the last bit of the maps,
// and these maps are rounded to FP32 again by the next map2alm.
// Against cleared bins and four FP64 LDS atomics per row and pair, inverse transforms of
// FP64 IQU, us: nside 128 x 16 93 -> 70, 256 x 16 307 -> 247, 512 x 16 1143 -> 952,
// 512 x 125 9240 -> 7470.
// conj(p) t, with the rounding of each part stated: it must not depend on the code around
__device__ __forceinline__ double2 cmul_conj(double2 p, double2 t)
{
    return make_double2(fma(p.x, t.x, p.y * t.y), fma(p.x, t.y, -(p.y * t.x)));
}
constexpr int FB = 2;  // bin pairs whose rows are loaded together
template <typename XT, typename Put>
__device__ __forceinline__ void fold_direct(const FftArgs& a, const XT* X, int64_t mrow, const double2* twn, int n, int s,
                                            int lmax, int j0, int dj, const Put& put)
{
    const int nh = n >> 1;
    const double2 zero = make_double2(0.0, 0.0);
    const double fl = s ? -1.0 : 1.0;
    for (int jb = j0; jb < nh; jb += FB * dj) {
        double2 ta[FB], tb[FB], ua[FB], ub[FB], p[FB], pm[FB];
#pragma unroll
        for (int u = 0; u < FB; ++u) {
            const int j = min(jb + u * dj, nh - 1), m = j ? n - j : nh;
            load4<XT>(X + min(j, lmax) * mrow, ta[u], tb[u]);
            p[u] = twn[s * j];
            if constexpr (sizeof(XT) == 4) pm[u] = twn[s * m];
            ua[u] = ub[u] = zero;
            if (m <= lmax) load4<XT>(X + m * mrow, ua[u], ub[u]);
        }
#pragma unroll
        for (int u = 0; u < FB; ++u) {
            const int j = jb + u * dj, m = j ? n - j : nh;
            if (j >= nh) break;
            bool l1 = j <= lmax, l2 = m <= lmax;
            if (a.mown) {
                l1 = l1 && a.mown[min(j, lmax)];
                l2 = l2 && a.mown[min(m, lmax)];
            }
            const double2 p2 = sizeof(XT) == 4 ? pm[u]
                               : j             ? make_double2(fl * p[u].x, -fl * p[u].y)
                                               : make_double2(s ? 0.0 : 1.0, s ? -1.0 : 0.0);
            const double2 ca = l1 ? cmul_conj(p[u], ta[u]) : zero, cb = l1 ? cmul_conj(p[u], tb[u]) : zero;
            const double2 ga = l2 ? cmul_conj(p2, ua[u]) : zero, gb = l2 ? cmul_conj(p2, ub[u]) : zero;
            const double2 e1 = make_double2(ca.x + cb.y, cb.x - ca.y), e2 = make_double2(ga.x + gb.y, gb.x - ga.y);
            const double2 d1 = make_double2(ca.x - cb.y, ca.y + cb.x), d2 = make_double2(ga.x - gb.y, ga.y + gb.x);
            put(j, j ? cadd(d1, e2) : d1);
            put(m, cadd(d2, j ? e1 : e2));
        }
    }
}

// the registers after a transform, reordered to the pass-0 layout
template <int LOGM>
__device__ __forceinline__ void to_pass0(const double2 (&v)[8], double2 (&u)[8])
{
    using QL = Pass<LOGM, P2<LOGM>::NP - 1>;
#pragma unroll
    for (int b = 0; b < QL::B; ++b) {
#pragma unroll
        for (int r = 0; r < QL::R; ++r) u[b + r * QL::B] = v[b * QL::R + r];
    }
}

// Convolution step of Bluestein on the pass-0 values u (x_i w_i at i = tl + k T, k < 4,
// zero for i >= n; n <= M/2 = 4 T): on return y_j = w_j u[k] for j = tl + k T < n, k < 4.
// CUT: the first transform skips the zero half of its inputs, the second the outputs past
// 4 T.  The compiler then fuses other products of the butterflies, which moves the last
// bit of the results: chunks with FP32 rows, whose rounding to FP32 would turn such a bit
// into 6e-8 of a coefficient now and then, keep the whole transforms.
template <typename XT>
constexpr bool CUT = sizeof(XT) == 8;
template <typename XT>
constexpr int NU = CUT<XT> ? 4 : 8;
// scale of the pixels taken into a forward transform: the halves of Z +- conj Z' go in
// with them for FP64 rows
template <typename XT>
constexpr double PIXS = CUT<XT> ? 0.5 : 1.0;
template <int LOGM, bool CUT>
__device__ __forceinline__ void blue_core(double2 (&u)[CUT ? 4 : 8], double2* sb, int tl, const double2* twM, const double2* bhat)
{
    constexpr int T = P2<LOGM>::T;
    double2 v[8], z[8], w[8];
#pragma unroll
    for (int k = 0; k < (CUT ? 4 : 8); ++k) v[k] = u[k];
    run_passes<LOGM, 0, CUT>(v, w, sb, tl, twM);
    to_pass0<LOGM>(v, z);
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const double2 y = cmul(z[k], bhat[tl + k * T]);
        z[k] = make_double2(y.x, -y.y);
    }
    __syncthreads();  // the first transform's last readers of sb are done
    run_passes<LOGM, 0>(z, w, sb, tl, twM);
    to_pass0<LOGM>(z, v);
#pragma unroll
    for (int k = 0; k < (CUT ? 4 : 8); ++k) u[k] = make_double2(v[k].x, -v[k].y);
}

// Output of one ring's forward transform, the spectrum Z of each map pair times PIXS in
// LDS (natural order, n values at lds + seq * SEQ): the unfold T_m = e^{-i m phi0} F_{m mod n}
// into the X rows.  Lanes run over (m, pair, part): FP64 rows take two 16-byte parts per
// pair (map k, map k+1), FP32 rows one, so the lanes of a wave store contiguous row
// segments of all S pairs.  The FP64 lane of map k forms Z + conj Z', that of map k+1
// -i (Z - conj Z'), with the -i in its phase.  Constructed before the barrier that
// completes Z, so that the first phases load across it; a batch's phases load behind the
// stores of the one before.  Forward transforms of FP64 IQU, us, with the changes to the
// zero half of the chirp transforms: nside 256 x 16 257 -> 247, 512 x 16 1048 -> 1002,
// 512 x 125 9000 -> 8140 (25 GB moved; 5.0 ms at the rate of a copy).
template <int LOGM, typename XT, bool MULTI, bool POW2>
struct Unfold {
    using C = P2<LOGM>;
    static constexpr int LP = sizeof(XT) == 8 ? 1 : 0;  // log2 parts per pair
    static constexpr int MSTEP = C::NTH >> (LP + C::LOGS);
    const double2 *zs, *tw;
    XT* X;
    int64_t mrow;
    int part, m0, mtop, n, s;
    MStep ws;
    double2 ph[MB];
    int jj[MB];

    __device__ __forceinline__ Unfold(const FftArgs& a, const Item& it, const double2* lds)
        : Unfold(a, it, lds, ((int)threadIdx.x >> LP) & (C::S - 1))
    {
    }
    __device__ __forceinline__ Unfold(const FftArgs& a, const Item& it, const double2* lds, int sq)
        : Unfold(a, it, lds, sq, seq_of<MULTI>(it, sq))
    {
    }
    __device__ __forceinline__ Unfold(const FftArgs& a, const Item& it, const double2* lds, int sq, Seq sr)
        : Unfold(a, it, lds, sq, sr, a.rings[sr.ring])
    {
    }
    __device__ __forceinline__ Unfold(const FftArgs& a, const Item& it, const double2* lds, int sq, Seq sr, const RingDev& rg)
        : zs(lds + sq * C::SEQ), tw(a.tw + a.lens[rg.len].tw), mrow((int64_t)a.nring * a.ldx),
          part((int)threadIdx.x & ((1 << LP) - 1)), m0((int)threadIdx.x >> (LP + C::LOGS)),
          mtop(sr.dead ? -1 : min(a.lmax, rg.mcut)), n(rg.n), s(rg.s), ws(m0, MSTEP, rg.n, rg.s)
    {
        X = static_cast<XT*>(a.X) + (int64_t)it.comp * a.xcomp + (int64_t)sr.ring * a.ldx + 4 * sr.pair + 2 * part;
        fetch();
    }
    __device__ __forceinline__ void fetch()
    {
#pragma unroll
        for (int u = 0; u < MB; ++u) {
            if constexpr (POW2) {
                const int m = m0 + u * MSTEP;
                ph[u] = tw[(m * s) & (2 * C::N - 1)];
                jj[u] = m & (C::N - 1);
            } else {
                ph[u] = tw[ws.ph];
                jj[u] = ws.j;
                ws.next();
            }
        }
    }
    __device__ __forceinline__ void run()
    {
        const double sg = part ? -1.0 : 1.0;
        while (m0 <= mtop) {
#pragma unroll
            for (int u = 0; u < MB; ++u) {
                const int m = m0 + u * MSTEP;
                if (m <= mtop) {
                    const int j = jj[u], jn = POW2 ? (C::N - j) & (C::N - 1) : (j ? n - j : 0);
                    const double2 z = zs[j], y = zs[jn];
                    if constexpr (sizeof(XT) == 8) {
                        const double2 Fp = make_double2(fma(sg, y.x, z.x), fma(-sg, y.y, z.y));
                        *reinterpret_cast<double2*>(X + m * mrow) = cmul(part ? make_double2(ph[u].y, -ph[u].x) : ph[u], Fp);
                    } else {
                        const double2 Fa = make_double2(0.5 * (z.x + y.x), 0.5 * (z.y - y.y));
                        const double2 Fb = make_double2(0.5 * (z.y + y.y), 0.5 * (y.x - z.x));
                        store4<XT>(X + m * mrow, cmul(ph[u], Fa), cmul(ph[u], Fb));
                    }
                }
            }
            m0 += MB * MSTEP;
            if (m0 <= mtop) fetch();
        }
    }
};

// data spectra of both maps (iterative map2alm), halfcomplex, all threads past the
// barrier that completes Z
template <int LOGM, typename XT, bool MULTI>
__device__ __forceinline__ void keep_spectra(const FftArgs& a, const Item& it, const double2* lds)
{
    using C = P2<LOGM>;
    constexpr int T = C::T;
    const int seq = (int)threadIdx.x / T, tl = (int)threadIdx.x % T;
    const double2* sb = lds + seq * C::SEQ;
    const Seq sr = seq_of<MULTI>(it, seq);
    const RingDev rg = a.rings[sr.ring];
    const int n = rg.n, k = sr.dead ? a.nmaps : 2 * sr.pair;
    for (int pos = tl; pos < n; pos += T) {
        const int j = (pos == 0) ? 0 : (pos == n - 1 ? n / 2 : (pos + 1) / 2);
        const int jn = j ? n - j : 0;
        const double2 z = sb[j], y = sb[jn];
        constexpr double h = 0.5 / PIXS<XT>;
        const double2 Fa = make_double2(h * (z.x + y.x), h * (z.y - y.y));
        const double2 Fb = make_double2(h * (z.y + y.y), h * (y.x - z.x));
        const bool im = (pos != 0) && (pos != n - 1) && ((pos & 1) == 0);
        if (k < a.nmaps) a.F[((int64_t)k * a.ncomp + it.comp) * a.npix + rg.first + pos] = im ? Fa.y : Fa.x;
        if (k + 1 < a.nmaps) a.F[((int64_t)(k + 1) * a.ncomp + it.comp) * a.npix + rg.first + pos] = im ? Fb.y : Fb.x;
    }
}

// Fold of one ring's X rows into conj(Z_j), j < n, at lds + seq * SEQ.  Rings whose
// cut lies below n take one direct and one mirror term per bin at most (fold_direct,
// lanes over (bin, pair)).  On the others (short rings near the poles) every m up to
// the cut lands on bin m mod n and its mirror, several terms per bin: the first nclear
// slots are cleared and the terms added atomically, lanes over (m, pair, part), the
// map-b lane handing its term to the map-a lane.  Ends with a barrier.
template <int LOGM, typename XT, bool MULTI = false>
__device__ __forceinline__ void fold(const FftArgs& a, const Item it, double2* lds, int nclear)
{
    using C = P2<LOGM>;
    constexpr int S = C::S;
    const int64_t mrow = (int64_t)a.nring * a.ldx;
    {
        const int sq = (int)threadIdx.x & (S - 1);
        const Seq sr = seq_of<MULTI>(it, sq);
        const RingDev rg = a.rings[sr.ring];
        const int lmax = min(a.lmax, rg.mcut);  // rows past the ring's cutoff are zero
        if (MULTI ? it.direct : lmax < rg.n) {
            double2* zs = lds + sq * C::SEQ;
            const XT* X = static_cast<const XT*>(a.X) + (int64_t)it.comp * a.xcomp + (int64_t)sr.ring * a.ldx + 4 * sr.pair;
            fold_direct<XT>(a, X, mrow, a.tw + a.lens[rg.len].tw, rg.n, rg.s, lmax, (int)threadIdx.x >> C::LOGS,
                            C::NTH >> C::LOGS, [zs](int j, double2 z) { zs[j] = make_double2(z.x, -z.y); });
            __syncthreads();
            return;
        }
    }
    for (int e = (int)threadIdx.x; e < nclear; e += C::NTH) lds[e] = make_double2(0.0, 0.0);
    __syncthreads();
    const int part = (int)threadIdx.x & 1;
    const int sq = ((int)threadIdx.x >> 1) & (S - 1);
    const int mi = (int)threadIdx.x >> (1 + C::LOGS);
    constexpr int MSTEP = C::NTH >> (1 + C::LOGS);
    double2* zs = lds + sq * C::SEQ;
    const Seq sr = seq_of<MULTI>(it, sq);
    const RingDev rg = a.rings[sr.ring];
    const double2* twn = a.tw + a.lens[rg.len].tw;  // e^{-i pi t/n}, t < 2n
    const int n = rg.n, lmax = min(a.lmax, rg.mcut);  // rows past the ring's cutoff are zero
    const XT* X = static_cast<const XT*>(a.X) + (int64_t)it.comp * a.xcomp + (int64_t)sr.ring * a.ldx +
                  4 * sr.pair + 2 * part;
    MStep ws(mi, MSTEP, n, rg.s);
    for (int m0 = mi; m0 <= lmax; m0 += MB * MSTEP) {
        double2 tv[MB], p[MB];
        int jj[MB];
#pragma unroll
        for (int q = 0; q < MB; ++q) {
            const XT* xr = X + min(m0 + q * MSTEP, lmax) * mrow;
            if constexpr (sizeof(XT) == 8) {
                tv[q] = *reinterpret_cast<const double2*>(xr);
            } else {
                const float2 f = *reinterpret_cast<const float2*>(xr);
                tv[q] = make_double2(f.x, f.y);
            }
            p[q] = twn[ws.ph];
            jj[q] = ws.j;
            ws.next();
        }
#pragma unroll
        for (int q = 0; q < MB; ++q) {
            const int m = m0 + q * MSTEP;
            const double2 c = cmul(make_double2(p[q].x, -p[q].y), tv[q]);  // c_m of this lane's map
            const double cbx = __shfl_xor(c.x, 1), cby = __shfl_xor(c.y, 1);
            if (part == 0 && m <= lmax && (!a.mown || a.mown[m])) {
                const double2 ca = c, cb = make_double2(cbx, cby);
                double* z1 = reinterpret_cast<double*>(zs + jj[q]);
                atomicAdd(z1, ca.x - cb.y);
                atomicAdd(z1 + 1, -(ca.y + cb.x));
                if (m >= 1) {
                    double* z2 = reinterpret_cast<double*>(zs + (jj[q] ? n - jj[q] : 0));
                    atomicAdd(z2, ca.x + cb.y);
                    atomicAdd(z2 + 1, -(cb.x - ca.y));
                }
            }
        }
    }
    __syncthreads();
}

template <int LOGN, typename XT, bool MULTI>
__device__ __forceinline__ void fwd_item(const FftArgs& a, const Item it, double2* lds)
{
    using C = P2<LOGN>;
    constexpr int N = C::N, T = C::T;
    const double2* tw = a.tw + a.lens[a.rings[it.ring].len].tw;  // e^{-i pi t/N}, t < 2N
    const int seq = (int)threadIdx.x / T, tl = (int)threadIdx.x % T;
    double2* sb = lds + seq * C::SEQ;
    const Seq sr = seq_of<MULTI>(it, seq);
    const int64_t first = a.rings[sr.ring].first;
    const int k = sr.dead ? a.nmaps : 2 * sr.pair;

    // pass-0 inputs x[tl + r T] of map pair (k, k+1), straight from global memory
    double2 v[8], w[8];
    {
        const int64_t ms = (int64_t)a.ncomp * a.npix;
        const double* pa = a.maps_in + (int64_t)it.comp * a.npix + first + min(k, a.nmaps - 1) * ms;
        const double* pb = a.maps_in + (int64_t)it.comp * a.npix + first + min(k + 1, a.nmaps - 1) * ms;
#pragma unroll
        for (int r = 0; r < 8; ++r) v[r] = make_double2(pa[tl + r * T], pb[tl + r * T]);
#pragma unroll
        for (int r = 0; r < 8; ++r)
            v[r] = make_double2(k < a.nmaps ? PIXS<XT> * v[r].x : 0.0, k + 1 < a.nmaps ? PIXS<XT> * v[r].y : 0.0);
    }
    run_passes<LOGN, 0>(v, w, sb, tl, tw);

    // the spectrum Z in natural order into LDS
    using QL = Pass<LOGN, C::NP - 1>;
    __syncthreads();
#pragma unroll
    for (int b = 0; b < QL::B; ++b) {
#pragma unroll
        for (int r = 0; r < QL::R; ++r) sb[tl + T * b + r * (N / QL::R)] = v[b * QL::R + r];
    }
    Unfold<LOGN, XT, MULTI, true> out(a, it, lds);
    __syncthreads();

    if (a.F) keep_spectra<LOGN, XT, MULTI>(a, it, lds);
    out.run();
}

template <int LOGN, typename XT, bool MULTI>
__device__ __forceinline__ void inv_item(const FftArgs& a, const Item it, double2* lds)
{
    using C = P2<LOGN>;
    constexpr int N = C::N, T = C::T, S = C::S;
    const double2* tw = a.tw + a.lens[a.rings[it.ring].len].tw;
    fold<LOGN, XT, MULTI>(a, it, lds, S * C::SEQ);

    // pass-0 inputs conj(Z_j) at bins j = tl + r T: the inverse DFT is conj(DFT(conj Z))
    const int seq = (int)threadIdx.x / T, tl = (int)threadIdx.x % T;
    double2* sb = lds + seq * C::SEQ;
    double2 v[8], w[8];
#pragma unroll
    for (int r = 0; r < 8; ++r) v[r] = sb[tl + r * T];
    __syncthreads();  // pass 0 overwrites the buffer
    run_passes<LOGN, 0>(v, w, sb, tl, tw);

    // natural-order outputs: map k = Re, map k+1 = -Im (conjugate of the DFT)
    using QL = Pass<LOGN, C::NP - 1>;
    const Seq so = seq_of<MULTI>(it, seq);
    const int k = so.dead ? a.nmaps : 2 * so.pair;
    const int64_t ms = (int64_t)a.ncomp * a.npix;
    double* oa = a.maps_out + (int64_t)it.comp * a.npix + a.rings[so.ring].first + (int64_t)k * ms;
    if (k < a.nmaps) {
#pragma unroll
        for (int b = 0; b < QL::B; ++b) {
#pragma unroll
            for (int r = 0; r < QL::R; ++r) oa[tl + T * b + r * (N / QL::R)] = v[b * QL::R + r].x;
        }
    }
    if (k + 1 < a.nmaps) {
#pragma unroll
        for (int b = 0; b < QL::B; ++b) {
#pragma unroll
            for (int r = 0; r < QL::R; ++r) oa[ms + tl + T * b + r * (N / QL::R)] = -v[b * QL::R + r].y;
        }
    }
}

template <int LOGM, typename XT, bool MULTI>
__device__ __forceinline__ void fwd_item_blue(const FftArgs& a, const Item it, double2* lds)
{
    using C = P2<LOGM>;
    constexpr int T = C::T;
    const int seq = (int)threadIdx.x / T, tl = (int)threadIdx.x % T;
    const Seq sr = seq_of<MULTI>(it, seq);
    const RingDev rg = a.rings[sr.ring];
    const FftLen* L = a.lens + rg.len;
    const int n = rg.n;
    const double2* twM = a.tw + L->twm;     // e^{-i pi t/M}, t < 2M
    const double2* chirp = a.tw + L->chirp;
    const double2* bhat = a.bhat + L->bhat;
    double2* sb = lds + seq * C::SEQ;
    const int k = sr.dead ? a.nmaps : 2 * sr.pair;

    double2 u[NU<XT>];
    {
        const int64_t ms = (int64_t)a.ncomp * a.npix;
        const double* pa = a.maps_in + (int64_t)it.comp * a.npix + rg.first + min(k, a.nmaps - 1) * ms;
        const double* pb = a.maps_in + (int64_t)it.comp * a.npix + rg.first + min(k + 1, a.nmaps - 1) * ms;
        double2 c[NU<XT>];
#pragma unroll
        for (int q = 0; q < NU<XT>; ++q) {
            const int i = min(tl + q * T, n - 1);
            u[q] = make_double2(pa[i], pb[i]);
            c[q] = chirp[i];
        }
#pragma unroll
        for (int q = 0; q < NU<XT>; ++q) {
            const bool live = tl + q * T < n;
            const double2 x = make_double2(k < a.nmaps ? PIXS<XT> * u[q].x : 0.0, k + 1 < a.nmaps ? PIXS<XT> * u[q].y : 0.0);
            u[q] = live ? cmul(x, c[q]) : make_double2(0.0, 0.0);
        }
    }
    blue_core<LOGM, CUT<XT>>(u, sb, tl, twM, bhat);

    // the spectrum, y_j = w_j u[k] (j = tl + k T < n), into LDS in natural order
    __syncthreads();
#pragma unroll
    for (int q = 0; q < NU<XT>; ++q) {
        const int j = tl + q * T;
        if (j < n) sb[j] = cmul(chirp[j], u[q]);
    }
    Unfold<LOGM, XT, MULTI, false> out(a, it, lds);
    __syncthreads();
    if (a.F) keep_spectra<LOGM, XT, MULTI>(a, it, lds);
    out.run();
}

template <int LOGM, typename XT, bool MULTI>
__device__ __forceinline__ void inv_item_blue(const FftArgs& a, const Item it, double2* lds)
{
    using C = P2<LOGM>;
    constexpr int T = C::T, S = C::S;
    fold<LOGM, XT, MULTI>(a, it, lds, S * C::SEQ);

    const int seq = (int)threadIdx.x / T, tl = (int)threadIdx.x % T;
    const Seq sr = seq_of<MULTI>(it, seq);
    const RingDev rg = a.rings[sr.ring];
    const FftLen* L = a.lens + rg.len;
    const int n = rg.n;
    const double2* twM = a.tw + L->twm;
    const double2* chirp = a.tw + L->chirp;
    const double2* bhat = a.bhat + L->bhat;

    // Bluestein on conj(Z): pass-0 values conj(Z_i) w_i
    double2* sb = lds + seq * C::SEQ;
    double2 u[NU<XT>];
    {
        double2 c[NU<XT>];
#pragma unroll
        for (int q = 0; q < NU<XT>; ++q) c[q] = chirp[min(tl + q * T, n - 1)];
#pragma unroll
        for (int q = 0; q < NU<XT>; ++q) {
            const int i = tl + q * T;
            u[q] = i < n ? cmul(sb[i], c[q]) : make_double2(0.0, 0.0);
        }
    }
    __syncthreads();  // pass 0 overwrites the buffer
    blue_core<LOGM, CUT<XT>>(u, sb, tl, twM, bhat);

    // pixels: y_j = w_j u[k] = DFT(conj Z)_j; map k = Re(conj y), map k+1 = Im(conj y)
    const int k = sr.dead ? a.nmaps : 2 * sr.pair;
    const int64_t ms = (int64_t)a.ncomp * a.npix;
    double* oa = a.maps_out + (int64_t)it.comp * a.npix + rg.first + (int64_t)k * ms;
    double2 c[NU<XT>];
#pragma unroll
    for (int q = 0; q < NU<XT>; ++q) c[q] = chirp[min(tl + q * T, n - 1)];
#pragma unroll
    for (int q = 0; q < NU<XT>; ++q) {
        const int j = tl + q * T;
        const double2 y = cmul(c[q], u[q]);
        if (j < n) {
            if (k < a.nmaps) oa[j] = y.x;
            if (k + 1 < a.nmaps) oa[ms + j] = -y.y;
        }
    }
}

}  // namespace
}  // namespace sht
