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
// element tl + T*b + r*N/R of the transform.
template <int LOGN, int PASS>
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
    for (int b = 0; b < Q::B; ++b) dftr<Q::R>(v + b * Q::R);
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
};
__device__ __forceinline__ bool work_item(const FftWork& w, int cnt, int pos, int comp0, Item& it)
{
    const int q = cnt >> 3, r = cnt & 7, x = pos & 7, y = pos >> 3;
    if (y >= q + (x < r ? 1 : 0)) return false;  // a class starts on a multiple of 8
    const int idx = x * q + min(x, r) + y;
    const int ngr = (w.nrings + w.rpw - 1) / w.rpw, per = ngr * w.groups;
    const int comp = idx / per, rem = idx - comp * per;
    const int gi = rem / w.groups, ri = gi * w.rpw;
    it = Item{w.rings[ri], (rem - gi * w.groups) << w.lgp, comp0 + comp, w.rings + ri, w.nrings - ri, w.lgp};
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
    return FftWork{c.rings, c.nrings, (used + per - 1) / per, c.nseq >> lgp, lgp};
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

// m = m0, m0 + dm, ...: keeps j = m mod n and ph = (m s) mod 2n
struct MStep {
    int j, ph, dj, dph, n, two_n;
    __device__ __forceinline__ MStep(int m0, int dm, int n_, int s)
    {
        n = n_;
        two_n = 2 * n_;
        j = m0 % n;
        ph = (int)(((int64_t)m0 * s) % two_n);
        dj = dm % n;
        dph = (int)(((int64_t)dm * s) % two_n);
    }
    __device__ __forceinline__ void next()
    {
        j += dj;
        if (j >= n) j -= n;
        ph += dph;
        if (ph >= two_n) ph -= two_n;
    }
};

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

// Convolution step of Bluestein on the pass-0 values u (x_i w_i at i = tl + k T,
// zero for i >= n): on return y_j = w_j u[k] for j = tl + k T < n.
template <int LOGM>
__device__ __forceinline__ void blue_core(double2 (&u)[8], double2* sb, int tl, const double2* twM, const double2* bhat)
{
    constexpr int T = P2<LOGM>::T;
    double2 v[8], w[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = u[k];
    run_passes<LOGM, 0>(v, w, sb, tl, twM);
    to_pass0<LOGM>(v, u);
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const double2 z = cmul(u[k], bhat[tl + k * T]);
        u[k] = make_double2(z.x, -z.y);
    }
    __syncthreads();  // the first transform's last readers of sb are done
    run_passes<LOGM, 0>(u, w, sb, tl, twM);
    to_pass0<LOGM>(u, v);
#pragma unroll
    for (int k = 0; k < 8; ++k) u[k] = make_double2(v[k].x, -v[k].y);
}

// Output of one ring's forward transform, the spectrum Z of each map pair in LDS
// (natural order, n values at lds + seq * SEQ, all threads past a barrier): the
// data spectra F of the iterative map2alm (halfcomplex, when kept) and the unfold
// T_m = e^{-i m phi0} F_{m mod n} into the X rows, lanes over (m, pair, part).
template <int LOGM, typename XT, bool MULTI = false>
__device__ __forceinline__ void blue_spectrum_out(const FftArgs& a, const Item it, const double2* lds)
{
    using C = P2<LOGM>;
    constexpr int T = C::T, S = C::S;
    if (a.F) {  // data spectra of both maps (iterative map2alm), halfcomplex
        const int seq = (int)threadIdx.x / T, tl = (int)threadIdx.x % T;
        const double2* sb = lds + seq * C::SEQ;
        const Seq sr = seq_of<MULTI>(it, seq);
        const RingDev rg = a.rings[sr.ring];
        const int n = rg.n, k = sr.dead ? a.nmaps : 2 * sr.pair;
        for (int pos = tl; pos < n; pos += T) {
            const int j = (pos == 0) ? 0 : (pos == n - 1 ? n / 2 : (pos + 1) / 2);
            const int jn = j ? n - j : 0;
            const double2 z = sb[j], y = sb[jn];
            const double2 Fa = make_double2(0.5 * (z.x + y.x), 0.5 * (z.y - y.y));
            const double2 Fb = make_double2(0.5 * (z.y + y.y), 0.5 * (y.x - z.x));
            const bool im = (pos != 0) && (pos != n - 1) && ((pos & 1) == 0);
            if (k < a.nmaps) a.F[((int64_t)k * a.ncomp + it.comp) * a.npix + rg.first + pos] = im ? Fa.y : Fa.x;
            if (k + 1 < a.nmaps)
                a.F[((int64_t)(k + 1) * a.ncomp + it.comp) * a.npix + rg.first + pos] = im ? Fb.y : Fb.x;
        }
    }

    constexpr int LP = sizeof(XT) == 8 ? 1 : 0;
    constexpr int MSTEP = C::NTH >> (LP + C::LOGS);
    const int part = (int)threadIdx.x & ((1 << LP) - 1);
    const int sq = ((int)threadIdx.x >> LP) & (S - 1);
    const int mi = (int)threadIdx.x >> (LP + C::LOGS);
    const double2* zs = lds + sq * C::SEQ;
    const Seq sr = seq_of<MULTI>(it, sq);
    const RingDev rg = a.rings[sr.ring];
    const double2* twn = a.tw + a.lens[rg.len].tw;  // e^{-i pi t/n}, t < 2n
    XT* X = static_cast<XT*>(a.X) + (int64_t)it.comp * a.xcomp + (int64_t)sr.ring * a.ldx + 4 * sr.pair + 2 * part;
    const int64_t mrow = (int64_t)a.nring * a.ldx;
    const int n = rg.n;
    MStep ws(mi, MSTEP, n, rg.s);
    const int mtop = sr.dead ? -1 : min(a.lmax, rg.mcut);
    for (int m0 = mi; m0 <= mtop; m0 += MB * MSTEP) {
        double2 ph[MB];
        int jj[MB];
#pragma unroll
        for (int q = 0; q < MB; ++q) {
            ph[q] = twn[ws.ph];
            jj[q] = ws.j;
            ws.next();
        }
#pragma unroll
        for (int q = 0; q < MB; ++q) {
            const int m = m0 + q * MSTEP;
            if (m <= mtop) {
                const int j = jj[q], jn = j ? n - j : 0;
                const double2 z = zs[j], y = zs[jn];
                const double2 Fa = make_double2(0.5 * (z.x + y.x), 0.5 * (z.y - y.y));
                const double2 Fb = make_double2(0.5 * (z.y + y.y), 0.5 * (y.x - z.x));
                if constexpr (sizeof(XT) == 8) {
                    *reinterpret_cast<double2*>(X + m * mrow) = cmul(ph[q], part ? Fb : Fa);
                } else {
                    store4<XT>(X + m * mrow, cmul(ph[q], Fa), cmul(ph[q], Fb));
                }
            }
        }
    }
}

// Fold of one ring's X rows into conj(Z_j), j < n, at lds + seq * SEQ after
// clearing the first nclear LDS slots: every m up to the ring's cut lands on bin
// m mod n and its mirror, several terms per bin, so added atomically; lanes over
// (m, pair, part), the map-b lane handing its term to the map-a lane.  Ends with
// a barrier.
template <int LOGM, typename XT, bool MULTI = false>
__device__ __forceinline__ void blue_fold(const FftArgs& a, const Item it, double2* lds, int nclear)
{
    using C = P2<LOGM>;
    constexpr int S = C::S;
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
    const int64_t mrow = (int64_t)a.nring * a.ldx;
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
    constexpr int N = C::N, T = C::T, S = C::S;
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
            v[r] = make_double2(k < a.nmaps ? v[r].x : 0.0, k + 1 < a.nmaps ? v[r].y : 0.0);
    }
    run_passes<LOGN, 0>(v, w, sb, tl, tw);

    // spectrum Z in natural order into LDS
    using QL = Pass<LOGN, C::NP - 1>;
    __syncthreads();
#pragma unroll
    for (int b = 0; b < QL::B; ++b) {
#pragma unroll
        for (int r = 0; r < QL::R; ++r) sb[tl + T * b + r * (N / QL::R)] = v[b * QL::R + r];
    }
    __syncthreads();

    if (a.F) {  // keep the data spectra of both maps (iterative map2alm), halfcomplex
        for (int pos = tl; pos < N; pos += T) {
            const int j = (pos == 0) ? 0 : (pos == N - 1 ? N / 2 : (pos + 1) / 2);
            const int jn = (N - j) & (N - 1);
            const double2 z = sb[j], y = sb[jn];
            const double2 Fa = make_double2(0.5 * (z.x + y.x), 0.5 * (z.y - y.y));
            const double2 Fb = make_double2(0.5 * (z.y + y.y), 0.5 * (y.x - z.x));
            const bool im = (pos != 0) && (pos != N - 1) && ((pos & 1) == 0);
            if (k < a.nmaps) a.F[((int64_t)k * a.ncomp + it.comp) * a.npix + first + pos] = im ? Fa.y : Fa.x;
            if (k + 1 < a.nmaps)
                a.F[((int64_t)(k + 1) * a.ncomp + it.comp) * a.npix + first + pos] = im ? Fb.y : Fb.x;
        }
    }

    // unfold T_m = e^{-i m phi0} F_{m mod N}.  Lanes run over (m, pair, part):
    // FP64 rows take two 16-byte parts per pair (map k, map k+1), FP32 rows one,
    // so the lanes of a wave store contiguous row segments of all S pairs.
    constexpr int LP = sizeof(XT) == 8 ? 1 : 0;  // log2 parts per pair
    constexpr int MSTEP = C::NTH >> (LP + C::LOGS);
    const int part = (int)threadIdx.x & ((1 << LP) - 1);
    const int sq = ((int)threadIdx.x >> LP) & (S - 1);
    const int mi = (int)threadIdx.x >> (LP + C::LOGS);
    const double2* zs = lds + sq * C::SEQ;
    const Seq so = seq_of<MULTI>(it, sq);
    const RingDev rg = a.rings[so.ring];
    XT* X = static_cast<XT*>(a.X) + (int64_t)it.comp * a.xcomp + (int64_t)so.ring * a.ldx + 4 * so.pair + 2 * part;
    const int64_t mrow = (int64_t)a.nring * a.ldx;
    const int s = rg.s, mtop = so.dead ? -1 : min(a.lmax, rg.mcut);
    for (int m0 = mi; m0 <= mtop; m0 += MB * MSTEP) {
        double2 ph[MB];
#pragma unroll
        for (int u = 0; u < MB; ++u) ph[u] = tw[((m0 + u * MSTEP) * s) & (2 * N - 1)];
#pragma unroll
        for (int u = 0; u < MB; ++u) {
            const int m = m0 + u * MSTEP;
            if (m <= mtop) {
                const int j = m & (N - 1), jn = (N - j) & (N - 1);
                const double2 z = zs[j], y = zs[jn];
                const double2 Fa = make_double2(0.5 * (z.x + y.x), 0.5 * (z.y - y.y));
                const double2 Fb = make_double2(0.5 * (z.y + y.y), 0.5 * (y.x - z.x));
                if constexpr (sizeof(XT) == 8) {
                    *reinterpret_cast<double2*>(X + m * mrow) = cmul(ph[u], part ? Fb : Fa);
                } else {
                    store4<XT>(X + m * mrow, cmul(ph[u], Fa), cmul(ph[u], Fb));
                }
            }
        }
    }
}

template <int LOGN, typename XT, bool MULTI>
__device__ __forceinline__ void inv_item(const FftArgs& a, const Item it, double2* lds)
{
    using C = P2<LOGN>;
    constexpr int N = C::N, T = C::T, S = C::S;
    constexpr int MSTEP = C::NTH >> C::LOGS;  // = T
    const double2* tw = a.tw + a.lens[a.rings[it.ring].len].tw;

    // Fold: C_j = sum_{m = j} c_m + sum_{m >= 1, -m = j} conj(c_m) of both maps,
    // Z = C^a + i C^b, into LDS in natural order.  Lanes run over (m, pair) so a
    // wave reads contiguous row segments of all S pairs.  d_m = c^a_m + i c^b_m is
    // the direct term, e_m = conj(c^a_m) + i conj(c^b_m) the mirror term.
    {
        const int sq = (int)threadIdx.x & (S - 1);
        const int mi = (int)threadIdx.x >> C::LOGS;
        double2* zs = lds + sq * C::SEQ;
        const Seq sr = seq_of<MULTI>(it, sq);
        const RingDev rg = a.rings[sr.ring];
        const int s = rg.s, lmax = min(a.lmax, rg.mcut);  // rows past the ring's cutoff are zero
        const XT* X = static_cast<const XT*>(a.X) + (int64_t)it.comp * a.xcomp + (int64_t)sr.ring * a.ldx + 4 * sr.pair;
        const int64_t mrow = (int64_t)a.nring * a.ldx;
        if ((MULTI ? a.lmax : lmax) < N) {  // the same for every ring of the workgroup
            // every bin has at most one direct and one mirror term: bins j = m
            // take d_m (zero beyond lmax), then bins N - m add e_m
            double2 e[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {  // m = mi + u T covers 0..N-1
                const int m = mi + u * MSTEP;
                double2 ta, tb;
                load4<XT>(X + min(m, lmax) * mrow, ta, tb);
                const double2 p = tw[(m * s) & (2 * N - 1)];
                const double2 ph = make_double2(p.x, -p.y);  // e^{+i m phi0}
                const double2 ca = cmul(ph, ta), cb = cmul(ph, tb);
                const bool live = m <= lmax && (!a.mown || a.mown[min(m, lmax)]);
                zs[m] = live ? make_double2(ca.x - cb.y, ca.y + cb.x) : make_double2(0.0, 0.0);
                e[u] = (live && m >= 1) ? make_double2(ca.x + cb.y, cb.x - ca.y) : make_double2(0.0, 0.0);
            }
            __syncthreads();
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int m = mi + u * MSTEP;
                if (m >= 1 && m <= lmax && (!a.mown || a.mown[m])) {
                    double2& z = zs[N - m];
                    z = make_double2(z.x + e[u].x, z.y + e[u].y);
                }
            }
        } else {
            // aliased rows (lmax >= N): several terms per bin, added atomically
            for (int e = (int)threadIdx.x; e < S * C::SEQ; e += C::NTH) lds[e] = make_double2(0.0, 0.0);
            __syncthreads();
            for (int m0 = mi; m0 <= lmax; m0 += MB * MSTEP) {
                double2 ta[MB], tb[MB], p[MB];
#pragma unroll
                for (int u = 0; u < MB; ++u) {
                    const int m = m0 + u * MSTEP;
                    load4<XT>(X + min(m, lmax) * mrow, ta[u], tb[u]);
                    p[u] = tw[(m * s) & (2 * N - 1)];
                }
#pragma unroll
                for (int u = 0; u < MB; ++u) {
                    const int m = m0 + u * MSTEP;
                    if (m <= lmax && (!a.mown || a.mown[m])) {
                        const double2 ph = make_double2(p[u].x, -p[u].y);
                        const double2 ca = cmul(ph, ta[u]), cb = cmul(ph, tb[u]);
                        double* z1 = reinterpret_cast<double*>(zs + (m & (N - 1)));
                        atomicAdd(z1, ca.x - cb.y);
                        atomicAdd(z1 + 1, ca.y + cb.x);
                        if (m >= 1) {
                            double* z2 = reinterpret_cast<double*>(zs + ((N - (m & (N - 1))) & (N - 1)));
                            atomicAdd(z2, ca.x + cb.y);
                            atomicAdd(z2 + 1, cb.x - ca.y);
                        }
                    }
                }
            }
        }
        __syncthreads();
    }

    // pass-0 inputs conj(Z_j) at bins j = tl + r T; the inverse DFT is conj(DFT(conj Z))
    const int seq = (int)threadIdx.x / T, tl = (int)threadIdx.x % T;
    double2* sb = lds + seq * C::SEQ;
    double2 v[8], w[8];
#pragma unroll
    for (int r = 0; r < 8; ++r) {
        const double2 z = sb[tl + r * T];
        v[r] = make_double2(z.x, -z.y);
    }
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

    double2 u[8];
    {
        const int64_t ms = (int64_t)a.ncomp * a.npix;
        const double* pa = a.maps_in + (int64_t)it.comp * a.npix + rg.first + min(k, a.nmaps - 1) * ms;
        const double* pb = a.maps_in + (int64_t)it.comp * a.npix + rg.first + min(k + 1, a.nmaps - 1) * ms;
        double2 c[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int i = min(tl + q * T, n - 1);
            u[q] = make_double2(pa[i], pb[i]);
            c[q] = chirp[i];
        }
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const bool live = tl + q * T < n;
            const double2 x = make_double2(k < a.nmaps ? u[q].x : 0.0, k + 1 < a.nmaps ? u[q].y : 0.0);
            u[q] = live ? cmul(x, c[q]) : make_double2(0.0, 0.0);
        }
    }
    blue_core<LOGM>(u, sb, tl, twM, bhat);

    // spectrum y_j = w_j u[k] (j = tl + k T < n) into LDS in natural order
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const int j = tl + q * T;
        if (j < n) sb[j] = cmul(chirp[j], u[q]);
    }
    __syncthreads();

    blue_spectrum_out<LOGM, XT, MULTI>(a, it, lds);
}

template <int LOGM, typename XT, bool MULTI>
__device__ __forceinline__ void inv_item_blue(const FftArgs& a, const Item it, double2* lds)
{
    using C = P2<LOGM>;
    constexpr int T = C::T, S = C::S;
    blue_fold<LOGM, XT, MULTI>(a, it, lds, S * C::SEQ);

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
    double2 u[8];
    {
        double2 c[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) c[q] = chirp[min(tl + q * T, n - 1)];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int i = tl + q * T;
            u[q] = i < n ? cmul(sb[i], c[q]) : make_double2(0.0, 0.0);
        }
    }
    __syncthreads();  // pass 0 overwrites the buffer
    blue_core<LOGM>(u, sb, tl, twM, bhat);

    // pixels: y_j = w_j u[k] = DFT(conj Z)_j; map k = Re(conj y), map k+1 = Im(conj y)
    const int k = sr.dead ? a.nmaps : 2 * sr.pair;
    const int64_t ms = (int64_t)a.ncomp * a.npix;
    double* oa = a.maps_out + (int64_t)it.comp * a.npix + rg.first + (int64_t)k * ms;
    double2 c[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) c[q] = chirp[min(tl + q * T, n - 1)];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
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
