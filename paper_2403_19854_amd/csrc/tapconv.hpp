// tapconv.hpp -- the operators of Alg 2-4 in one launch, for short supports.
//
// A convolving array of the method is a monomial times a tensor-product kernel
// of compact support (Eq 6, 44, 77): along an axis it has 2R + 1 taps,
// t_e(o) = o^e phi(o / a~) for |o| <= R = ceil(a~) - 1.  The circular
// convolutions of Eq 34 can then be summed directly, axis by axis; with R <= 3
// that is 5 to 7 multiply-adds per value, and because a direct sum needs only
// R neighbours, both halves of a product and the pointwise stage between them
// fit one kernel that reads d and writes f once:
//
//   part 1   u -> z-convolutions -> y-convolutions -> D_q (x-convolutions)
//   point    E = M D, M = V B^T B   (rows of b^a; Eq 90-91, Alg 2)
//   part 2   E_p -> x -> y -> z with the reflected taps (Eq 55, 91)
//
// A workgroup owns TX x TY columns of the result and marches through a chunk
// of planes.  z is the first axis of part 1 and the last of part 2, so both z
// convolutions run in registers: an incoming plane is kept for 2R
// more steps, a plane of part 2 is added to the 2R + 1 pending sums of its
// column, and only the x and y convolutions exchange values through LDS.  The work of one
// plane is cut into five phases that run as a software pipeline over three
// planes, in two halves per step:
//
//   half A   Z -> sZ (plane p)     sY -> D, E -> sE (p - 1)   sF -> y, z, store (p - 2)
//   half B   sZ -> sY (plane p)    sE -> sF (p - 1)
//
// Every buffer is written in one half and read in the other, so one copy of
// each and two barriers per plane suffice.
//
// What bounds it: the vector pipes on large boxes (256^3 FP32: 219 lane
// operations per node issued, 71% of the issue slots; about 145 of them are taps
// with the halo of a 32 x 16 tile and the run-in of a chunk; LDS active 49% of
// the time; 208 MB fetched, a third more than what is unique), the chain of steps
// on small ones (32^3: 7 steps of about 0.6 us after 2-3 us of launch and first
// loads).  K products back to back, linear basis, R = 2, against the five FFT
// passes: 32^3 FP32 9.4 us (28.8), 128^3 FP32 30 (55) and FP64 46 (107), 256^3
// FP32 131 (362), 32 right-hand sides of 96^3 211 (552); quadratic ball of 128^3,
// R = 2, FP32 60 (181).
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>

#include "fcrkpm_impl.hpp"

namespace fcrkpm {

constexpr int kTapR = 3;          // largest tap radius

constexpr int kTapMint = kMaxNodeConst + 1;  // interior record: rows and V (wider row sets have no interior class)

// K products; u^h; the loads f^r, f^q and N^T y; the gradient force.  TAP_GRAD
// is u^h with the rows b^a (one field, its dim components nn apart).  TAP_MOM
// writes the D_q of the domain mask: the moments of Eq 49, Alg 1 (its basis has
// twice the degree).
enum { TAP_K = SEP_PW_K, TAP_UH = SEP_PW_UH, TAP_LOAD = SEP_PW_LOAD, TAP_KN = SEP_PW_KN, TAP_GRAD = kTapGrad, TAP_CG = kTapCg, TAP_MOM = 6 };

// Monomials of degree <= DEG in DIM variables (the library's basis order), as
// the tree the passes walk: fields after z (exponent ez), after y (ey, ez),
// and the basis itself (ex on y field yf).
template <int DIM_, int DEG_>
struct TapBasis {
    static constexpr int DIM = DIM_, DEG = DEG_;
    static constexpr int NZ = DIM > 2 ? DEG + 1 : 1;
    static constexpr int NY = DIM > 2 ? (DEG + 1) * (DEG + 2) / 2 : DIM > 1 ? DEG + 1 : 1;
    static constexpr int S = DIM == 1   ? DEG + 1
                             : DIM == 2 ? (DEG + 1) * (DEG + 2) / 2
                                        : (DEG + 1) * (DEG + 2) * (DEG + 3) / 6;
    struct Tab {
        int yey[NY], yez[NY];
        int xex[S], xyf[S];
    };
    static constexpr Tab make()
    {
        Tab t{};
        int n = 0;
        for (int d = 0; d <= DEG; ++d)
            for (int b = d; b >= 0; --b) {
                const int c = d - b;
                if (DIM < 2 && b != 0) continue;
                if (DIM < 3 && c != 0) continue;
                t.yey[n] = b;
                t.yez[n] = c;
                ++n;
            }
        int k = 0;
        for (int d = 0; d <= DEG; ++d)
            for (int a = d; a >= 0; --a)
                for (int b = d - a; b >= 0; --b) {
                    const int c = d - a - b;
                    if (DIM < 2 && b != 0) continue;
                    if (DIM < 3 && c != 0) continue;
                    t.xex[k] = a;
                    for (int f = 0; f < NY; ++f)
                        if (t.yey[f] == b && t.yez[f] == c) t.xyf[k] = f;
                    ++k;
                }
        return t;
    }
    static constexpr Tab tab = make();
};

template <typename T>
struct TapArgs {
    const void* in;            // field (Tio)
    void* out;                 // field (Tio)
    const uint8_t* mask_in;
    const uint8_t* mask_out;
    T t[3][kTapE][kTapR + 1];  // t[axis][e][o], o = 0..R
    int n[3];
    int ntx, nty;              // tiles along x and y
    int cz;                    // planes per chunk (one workgroup), a multiple of cu
    int cu;                    // planes per dot partial
    const int2* zr;            // per tile column: first and last plane with a domain node
    const uint32_t* words;     // [nz][ny][gx]: classes and first record of two nodes
    int gx;                    // words per row (the row starts R nodes before x = 0)
    const T* rec;              // records of the class-2 nodes
    T mint[kTapMint];          // record of the interior nodes
    const T* rows;             // UH, LOAD: b^0 [s][nn] (UH also b^a, [dim][s][nn]); KN: b^a
    const T* vol;              // UH, LOAD: weight [nn] or NULL; KN: V [nn]
    T kappa;                   // KN
    // TAP_CG: K p after the pending update p = r + beta p of CG (pend = 0: none),
    // with the partials of p . K p; in holds the old p, pnew takes the new one
    // (another array, as neighbours still read the old)
    const void* r;
    void* pnew;
    double* dot_part;          // partials of p . K p per tile and cu planes
    long dot_stride;           // their slots between right-hand sides
    const double* rr_part;     // partials of the new r.r, nrr of them
    int pend, nrr, parity;           // scal[parity] = old r.r; scal[1 - parity] takes the new
    double* scal;
    const int* act;            // right-hand sides still iterating
    long nn;
    long rb;                   // bytes between right-hand sides of in and out
};

// A record holds M = V B^T B (upper triangle) for the linear bases, where the
// product with M costs no more than the two with B; the others keep the rows
// of B and V.  Padded to whole 16-byte loads.
template <class B, int MODE>
constexpr bool tap_mform() { return B::DEG == 1 && MODE != TAP_KN; }
constexpr int tap_rec_values(bool mform, int s, int rows) { return mform ? s * (s + 1) / 2 : rows * s + 1; }
constexpr int tap_rec_pitch(bool mform, int s, int rows, int elem)
{
    const int per = 16 / elem;
    return (tap_rec_values(mform, s, rows) + per - 1) / per * per;
}

// LDS traffic alone is ordered here: global loads in flight stay in flight.
__device__ __forceinline__ void tap_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

template <typename T>
struct alignas(2 * sizeof(T)) TapPair {
    T x, y;
};

// f(0), f(1), ... with the index as a constant: the basis tables and the taps
// they pick are resolved when the kernel is compiled
template <int N, int I = 0, typename F>
__device__ __forceinline__ void tap_for(F&& f)
{
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        tap_for<N, I + 1>(f);
    }
}

// sum over the taps of exponent E at the window centre w[R]: the convolution
// sum_o t_e(o) u(I - o), or with REFL its reflection sum_o t_e(o) u(I + o).
// t_e is even or odd with e, so two neighbours share a tap.
template <int R, bool REFL, int E, typename T, typename TP>
__device__ __forceinline__ T tap_conv(const T* w, const TP& t)
{
    if constexpr (R == 0) {
        return w[0];
    } else {
        T acc = (E == 0) ? t[0] * w[R] : T(0);
#pragma unroll
        for (int o = 1; o <= R; ++o) {
            const T lo = w[R - o], hi = w[R + o];
            const T v = (E & 1) ? (REFL ? hi - lo : lo - hi) : lo + hi;
            acc = (E > 0 && o == 1) ? t[o] * v : acc + t[o] * v;
        }
        return acc;
    }
}

__device__ __forceinline__ int tap_wrap(int i, int n)
{
    i %= n;
    return i < 0 ? i + n : i;
}

// Workgroup b runs on XCD b % 8: neighbouring tiles go to one XCD, whose L2 then
// serves most of their halos (K in FP32, bytes fetched past the L2 and time,
// without and with this order: 128^3 152 -> 34 MB, 37 -> 30 us; 256^3 597 -> 208 MB,
// 140 -> 131 us; 32 right-hand sides of 96^3 784 -> 217 MB, 257 -> 211 us).
__device__ __forceinline__ long tap_xcd(long b, long nblocks)
{
    if (nblocks % 8 != 0) return b;
    return (b & 7) * (nblocks >> 3) + (b >> 3);
}

// Sizes of one variant.
template <class B, int R, int MODE, int TX, int TY>
struct TapGeom {
    static constexpr bool P1 = MODE != TAP_LOAD, P2 = MODE != TAP_UH && MODE != TAP_MOM;
    static constexpr int RX = R, RY = B::DIM > 1 ? R : 0, RZ = B::DIM > 2 ? R : 0;
    static constexpr int HX = P2 ? RX : 0, HY = P2 ? RY : 0, HZ = P2 ? RZ : 0;
    static constexpr int XE = TX + 2 * HX, YE = TY + 2 * HY;  // where D and E are formed
    static constexpr int XL = XE + 2 * RX, YL = YE + 2 * RY;  // where u is read
    static constexpr int NSZ = P1 ? B::NZ * YL * XL : 0, NSY = P1 ? B::NY * YE * XL : 0;
    static constexpr int NSE = P2 ? B::S * YE * XE : 0, NSF = P2 ? B::NY * YE * TX : 0;
    static constexpr int LDS = NSZ + NSY + NSE + NSF;
};

template <class B, int R, int MODE, int TX, int TY>
constexpr int tap_lds_of = TapGeom<B, R, MODE, TX, TY>::LDS;
// Workgroups that a CU is meant to hold: as many as the LDS (160 KB) takes, but
// no more than leave every thread the registers it needs (about 80 of 4 bytes
// for the small bases in FP32 at R <= 2, 128 in FP64 and for larger ones, 256
// for ten monomials in FP64 or at R = 3).
constexpr int tap_residents(int elem, int lds, int nt, int s, int r)
{
    const int waves = elem == 4 && s <= 4 && r <= 2 ? 24 : elem == 8 && (s == 10 || r == 3) ? 8 : s == 10 && r == 3 ? 8 : 16;
    const int byregs = waves / (nt / 64), bylds = 160 * 1024 / (elem * lds + 64);
    const int n = byregs < bylds ? byregs : bylds;
    return n < 1 ? 1 : n;
}
constexpr int tap_min_waves(int elem, int lds, int nt, int s, int r)
{
    const int w = tap_residents(elem, lds, nt, s, r) * (nt / 64) / 4;
    return w < 1 ? 1 : w;
}

// The arguments live in the kernel-argument segment.  The taps and the interior
// record of a small basis stay in scalar registers; those of a large one would
// not fit, so every phase reads what it needs again (scalar loads that hit the
// constant cache; 1.5% slower where both work).
template <typename T>
using TapArgPtr = const __attribute__((address_space(4))) TapArgs<T>*;

template <bool HOLD, typename P>
__device__ __forceinline__ P tap_fresh(P p)
{
    if constexpr (!HOLD) asm volatile("" : "+s"(p));
    return p;
}

// Threads of one variant.  Half A gives D and E to the first NA threads and
// the y and z reflections to the other NB; half B gives the y convolutions to
// the first N2 threads and the x reflections to the rest.  SPLIT = false (1D)
// lets every thread do everything.
template <int DIM, int NT>
struct TapRoles {
    static constexpr bool SPLIT = DIM > 1;
    // TAP_CG asks for the first planes before it forms beta: not in the large 3D
    // tile, whose registers do not hold both (128^3 FP32 67 us an iteration
    // against 56; 32^3 18.5 -> 17.9, 300^2 14.4 -> 13.9 with it)
    static constexpr bool EARLY = DIM < 3 || NT < 512;
    static constexpr int NA = SPLIT ? NT * 3 / 4 : NT, NB = SPLIT ? NT - NA : NT;
    static constexpr int N2 = SPLIT ? NT / 2 : NT, N4 = SPLIT ? NT - N2 : NT;
};

// What TAP_CG adds to a march.  beta comes from the partials of r.r, summed as
// the stand-alone update sums them; every load that it needs is issued by load(),
// and the first planes are asked for before settle() waits for them.
template <typename T, typename Tio, int NT>
struct TapUpdate {
    const Tio* r = nullptr;
    Tio* pnew = nullptr;
    T alpha = T(0), beta = T(1);  // p = alpha r + beta p
    double* dpart = nullptr;
    double* dsum = nullptr;       // LDS, a slot per wave
    double* sum = nullptr;        // LDS, a slot per wave
    double part[kRedBlocks / NT], old = 0.0;

    __device__ __forceinline__ void load(TapArgPtr<T> kp)
    {
        const double* q = kp->rr_part + (long)blockIdx.y * kRedBlocks;
#pragma unroll
        for (int k = 0; k < kRedBlocks / NT; ++k) part[k] = q[threadIdx.x + k * NT];
        old = (kp->scal + (long)blockIdx.y * kScal)[kp->parity];
    }
    // all threads of the workgroup
    __device__ __forceinline__ void settle(TapArgPtr<T> kp)
    {
        double v = 0.0;
#pragma unroll
        for (int k = 0; k < kRedBlocks / NT; ++k)
            if ((int)threadIdx.x + k * NT < kp->nrr) v += part[k];
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
        if ((threadIdx.x & 63) == 0) sum[threadIdx.x >> 6] = v;
        tap_barrier();
        double rr = 0.0;
#pragma unroll
        for (int i = 0; i < NT / 64; ++i) rr += sum[i];
        alpha = T(1);
        beta = old > 0.0 ? T(rr / old) : T(0);
        if (blockIdx.x == 0 && threadIdx.x == 0) (kp->scal + (long)blockIdx.y * kScal)[1 - kp->parity] = rr;
    }
};

// One workgroup's march; ROLE bit 0: D and E, bit 1: the reflections along y and z.
template <typename T, typename Tio, class B, int R, int MODE, int ROWS, int TX, int TY, int NT, int ROLE>
struct TapMarch {
    using G = TapGeom<B, R, MODE, TX, TY>;
    using RO = TapRoles<B::DIM, NT>;
    using KP = TapArgPtr<T>;
    static constexpr bool EARLY = RO::EARLY;
    static constexpr int S = B::S, NZ = B::NZ, NY = B::NY;
    static constexpr int RY = G::RY, RZ = G::RZ, HX = G::HX, HY = G::HY, HZ = G::HZ;
    static constexpr int XE = G::XE, YE = G::YE, XL = G::XL, YL = G::YL;
    static constexpr bool CG = MODE == TAP_CG, KMODE = MODE == TAP_K || MODE == TAP_KN || CG;
    static constexpr int NC = G::P1 ? (XL * YL + NT - 1) / NT : 1;          // input columns per thread
    static constexpr int NB2 = YE % 4 == 0 ? 4 : YE % 2 == 0 ? 2 : 1;       // rows per item, y convolution
    static constexpr int XB4 = 4;                                           // nodes per item, x reflection
    static constexpr int NB5 = TY % 4 ? 1 : TX * TY >= 256 ? 4 : 2;         // rows per item, y reflection
    static constexpr int N3 = XE / 2 * YE, NP3 = (N3 + RO::NA - 1) / RO::NA;
    static constexpr int N5 = TX * (TY / NB5);
    static_assert((!G::P2 || (N5 <= RO::NB && N5 % 64 == 0)) && XE % 2 == 0 && TX % XB4 == 0);
    static constexpr bool MF = tap_mform<B, MODE>();
    static constexpr int RP = tap_rec_pitch(MF, S, ROWS, sizeof(T));
    static constexpr bool ICONST = ROWS * S <= kMaxNodeConst;  // wider row sets have no classes
    static constexpr bool A = (ROLE & 1) != 0, Bq = (ROLE & 2) != 0 && G::P2;

    // x convolutions of two nodes: put(i, q, D_q of node i) from the y-level fields
    template <typename F>
    static __device__ __forceinline__ void x_conv(const T* sY, int yy, int gi, KP k, F&& put)
    {
        tap_for<NY>([&](auto fc) {
            constexpr int f = decltype(fc)::value;
            T w[2 + 2 * R];
            const TapPair<T>* src = reinterpret_cast<const TapPair<T>*>(sY + (f * YE + yy) * XL + 2 * gi);
#pragma unroll
            for (int j = 0; j <= R; ++j) {
                const TapPair<T> v = src[j];
                w[2 * j] = v.x;
                w[2 * j + 1] = v.y;
            }
            tap_for<S>([&](auto qc) {
                constexpr int q = decltype(qc)::value;
                if constexpr (B::tab.xyf[q] == f) {
                    constexpr int e = B::tab.xex[q];
                    put(0, q, tap_conv<R, false, e>(w, k->t[0][e]));
                    put(1, q, tap_conv<R, false, e>(w + 1, k->t[0][e]));
                }
            });
        });
    }

    // E = M D, or V B^T (f B D) with the rows of B (f = 1 but for KN)
    template <typename M>
    static __device__ __forceinline__ void point(const M& m, KP k, const T (&D)[S], T (&E)[S])
    {
        if constexpr (MF) {
#pragma unroll
            for (int p = 0; p < S; ++p) {
                T acc = T(0);
#pragma unroll
                for (int q = 0; q < S; ++q) {
                    const int lo = p < q ? p : q, hi = p < q ? q : p;
                    acc += m[lo * S - lo * (lo - 1) / 2 + hi - lo] * D[q];
                }
                E[p] = acc;
            }
        } else {
            T v = m[ROWS * S];
            T Ar[ROWS];
#pragma unroll
            for (int r = 0; r < ROWS; ++r) {
                T acc = T(0);
#pragma unroll
                for (int q = 0; q < S; ++q) acc += m[r * S + q] * D[q];
                Ar[r] = acc;
            }
            if constexpr (MODE == TAP_KN) {
                T s2 = T(0);
#pragma unroll
                for (int r = 0; r < ROWS; ++r) s2 += Ar[r] * Ar[r];
                v *= T(1) + k->kappa * s2;
            }
#pragma unroll
            for (int r = 0; r < ROWS; ++r) Ar[r] *= v;
#pragma unroll
            for (int p = 0; p < S; ++p) {
                T acc = T(0);
#pragma unroll
                for (int r = 0; r < ROWS; ++r) acc += m[r * S + p] * Ar[r];
                E[p] = acc;
            }
        }
    }

    static __device__ __forceinline__ uint32_t rec_at(uint32_t w, int i)
    {
        const uint32_t c = (w >> (2 * i)) & 3;
        return c == 2 ? (w >> 4) + ((i && (w & 3) == 2) ? 1u : 0u) : c;
    }

    static __device__ __forceinline__ void run(KP kp, T* smem, const Tio* in, Tio* out, int tile, int ntiles,
                                               int x0, int y0, int zlo, int zhi, TapUpdate<T, Tio, NT> up)
    {
        T* const sZ = smem;
        T* const sY = sZ + G::NSZ;
        T* const sE = sY + G::NSY;
        T* const sF = sE + G::NSE;
        const int tid = threadIdx.x;
        const int nx = kp->n[0], ny = kp->n[1], nz = kp->n[2], nxy = nx * ny, gx = kp->gx;
        const uint8_t* const mask_in = kp->mask_in;
        const uint8_t* const mask_out = kp->mask_out;
        double dacc = 0.0;
        bool flush = false;  // the wave sums of a partial wait in up.dsum
        int left = 0;        // planes up to the partial's end
        double* dpart = nullptr;
        if constexpr (CG) {
            left = kp->cu - zlo % kp->cu;
            dpart = up.dpart + (long)(zlo / kp->cu) * ntiles + tile;
        }

        // input columns of this thread
        uint32_t col[NC];
        bool own[NC];
        if constexpr (G::P1) {
#pragma unroll
            for (int k = 0; k < NC; ++k) {
                const int c = min(tid + k * NT, XL * YL - 1);
                col[k] = (uint32_t)(tap_wrap(y0 - HY - RY + c / XL, ny) * nx + tap_wrap(x0 - HX - R + c % XL, nx));
                if constexpr (CG) {
                    // columns of this tile: their new p is stored
                    const int lx = c % XL - HX - R, ly = c / XL - HY - RY;
                    own[k] = lx >= 0 && lx < TX && x0 + lx < nx && ly >= 0 && ly < TY && y0 + ly < ny &&
                             tid + k * NT < XL * YL;
                }
            }
        }
        // E-level items: two nodes along x; word offset in a plane (K, KN) and
        // offsets of the two nodes (the modes that read node arrays)
        uint32_t wt3[NP3], it3[NP3], jt3[NP3];
        if constexpr (A) {
#pragma unroll
            for (int k = 0; k < NP3; ++k) {
                const int it = min(tid + k * RO::NA, N3 - 1);
                const int gi = it % (XE / 2), gy = tap_wrap(y0 - HY + it / (XE / 2), ny);
                if constexpr (KMODE) wt3[k] = (uint32_t)(gy * gx + x0 / 2 + gi);
                if constexpr (MODE != TAP_K && !CG) {
                    it3[k] = (uint32_t)(gy * nx + tap_wrap(x0 - HX + 2 * gi, nx));
                    jt3[k] = (uint32_t)(gy * nx + tap_wrap(x0 - HX + 2 * gi + 1, nx));
                }
            }
        }
        const int i5 = RO::SPLIT ? tid - RO::NA : tid;
        const bool do5 = Bq && i5 >= 0 && i5 < N5;
        const int x5 = i5 % TX, y5 = i5 / TX * NB5;
        T zout[NB5][2 * RZ + 1];
        uint8_t mk5[NB5];
        bool ok5[NB5];
        uint32_t o5 = 0;
        if constexpr (Bq) {
#pragma unroll
            for (int k = 0; k < NB5; ++k) {
#pragma unroll
                for (int j = 0; j <= 2 * RZ; ++j) zout[k][j] = T(0);
                ok5[k] = do5 && x0 + x5 < nx && y0 + y5 + k < ny;
                mk5[k] = 0;
            }
            o5 = (uint32_t)((y0 + y5) * nx + x0 + x5);
        }
        const int nE = zhi - zlo + 2 * HZ;               // E-level planes
        int pin = tap_wrap(zlo - HZ - RZ, nz);           // next plane to load
        int pe = tap_wrap(zlo - HZ, nz);                 // next plane of the E level
        // the last planes of each column: the first 2 RZ are loaded here, all at
        // once; from then on values are loaded a step ahead and masked when they
        // are used
        T zin[NC][2 * RZ + 1];
        // (CG vectors are zero off the free nodes: r comes in place of the mask)
        Tio nxt[NC];
        std::conditional_t<CG, Tio, uint8_t> nmk[NC];
        const auto value = [&](int k) -> T {
            if constexpr (CG) return up.alpha * T(nmk[k]) + up.beta * T(nxt[k]);
            else if constexpr (MODE == TAP_MOM) return T(nmk[k] != 0);
            else return nmk[k] ? T(nxt[k]) : T(0);
        };
        const auto fetch = [&](int z) {
            const Tio* pi = in + (long)z * nxy;
#pragma unroll
            for (int k = 0; k < NC; ++k) {
                if constexpr (MODE != TAP_MOM) nxt[k] = pi[col[k]];
                if constexpr (CG) nmk[k] = (up.r + (long)z * nxy)[col[k]];
                else nmk[k] = (mask_in + (long)z * nxy)[col[k]];
            }
        };
        if constexpr (CG && EARLY) {
            Tio p0[NC][2 * RZ + 1], r0[NC][2 * RZ + 1];
#pragma unroll
            for (int j = 0; j <= 2 * RZ; ++j) {
                fetch(pin);
#pragma unroll
                for (int k = 0; k < NC; ++k) {
                    p0[k][j] = nxt[k];
                    r0[k][j] = nmk[k];
                }
                if (j < 2 * RZ) pin = (pin + 1 == nz) ? 0 : pin + 1;
            }
            if (kp->pend) up.settle(kp);
#pragma unroll
            for (int j = 0; j < 2 * RZ; ++j)
#pragma unroll
                for (int k = 0; k < NC; ++k) zin[k][j + 1] = up.alpha * T(r0[k][j]) + up.beta * T(p0[k][j]);
        } else if constexpr (G::P1) {
#pragma unroll
            for (int j = 0; j <= 2 * RZ; ++j) {
                fetch(pin);
#pragma unroll
                for (int k = 0; k < NC; ++k)
                    if (j < 2 * RZ) zin[k][j + 1] = value(k);
                if (j < 2 * RZ) pin = (pin + 1 == nz) ? 0 : pin + 1;
            }
        }
        uint32_t word[NP3];
        if constexpr (A && KMODE) {
            const uint32_t* pw = kp->words + (long)pe * ny * gx;
#pragma unroll
            for (int k = 0; k < NP3; ++k) word[k] = pw[wt3[k]];
        }
        const int s0 = G::P1 ? 2 * RZ : 2 * RZ + 1, s1 = nE + 2 * RZ + (G::P2 ? 2 : 1);
        for (int s = s0; s < s1; ++s) {
            // ---------------------------------------------------------- half A
            if constexpr (G::P1) {
                if (s < nE + 2 * RZ) {
                    const KP k_ = tap_fresh<(S <= 4)>(kp);
                    T cur[NC];
#pragma unroll
                    for (int k = 0; k < NC; ++k) cur[k] = value(k);
                    if constexpr (CG) {
                        // the planes of the chunk itself
                        if (s < zhi - zlo + 2 * RZ) {
                            Tio* po = up.pnew + (long)pin * nxy;
#pragma unroll
                            for (int k = 0; k < NC; ++k)
                                if (own[k]) po[col[k]] = Tio(cur[k]);
                        }
                    }
                    if (s + 1 < nE + 2 * RZ) {
                        pin = (pin + 1 == nz) ? 0 : pin + 1;
                        fetch(pin);
                    }
#pragma unroll
                    for (int k = 0; k < NC; ++k) {
#pragma unroll
                        for (int j = 0; j < 2 * RZ; ++j) zin[k][j] = zin[k][j + 1];
                        zin[k][2 * RZ] = cur[k];
                    }
#pragma unroll
                    for (int k = 0; k < NC; ++k)
                        if ((k + 1) * NT <= XL * YL || tid + k * NT < XL * YL)
                            tap_for<NZ>([&](auto ec) {
                                constexpr int e = decltype(ec)::value;
                                sZ[e * YL * XL + tid + k * NT] = tap_conv<RZ, false, e>(zin[k], k_->t[2][e]);
                            });
                }
            }
            if constexpr (A) {
                if (s >= 2 * RZ + 1 && s < nE + 2 * RZ + 1) {
                    const KP k_ = tap_fresh<(S <= 4)>(kp);
#pragma unroll
                    for (int k = 0; k < NP3; ++k) {
                        const int it = tid + k * RO::NA;
                        if (it < N3) {
                            const int gi = it % (XE / 2), yy = it / (XE / 2);
                            T D[2][S];
                            if constexpr (G::P1 && MODE != TAP_MOM)
                                x_conv(sY, yy, gi, k_, [&](int i, int q, T v) { D[i][q] = v; });
                            if constexpr (MODE == TAP_MOM) {
                                // pairs of monomials, as the moment solves read them; each
                                // value leaves as it is formed (35 of them would not fit)
                                T* o = reinterpret_cast<T*>(out) + (long)pe * nxy * 2;
                                const bool row = y0 + yy < ny, ok[2] = {row && x0 + 2 * gi < nx, row && x0 + 2 * gi + 1 < nx};
                                x_conv(sY, yy, gi, k_, [&](int i, int q, T v) {
                                    if (ok[i]) (o + (long)(q / 2) * k_->nn * 2 + (q & 1))[2 * (i ? jt3[k] : it3[k])] = v;
                                });
                            } else if constexpr (MODE == TAP_UH) {
                                // u = sum_p b0_p D_p (times V for V o N; Eq 94), or with
                                // the rows b^a the implicit gradient, a field per row
                                const T* vol = k_->vol ? k_->vol + (long)pe * nxy : nullptr;
#pragma unroll
                                for (int r = 0; r < ROWS; ++r) {
                                    const T* b = k_->rows + (long)r * S * k_->nn + (long)pe * nxy;
                                    Tio* o = out + r * k_->nn + (long)pe * nxy;
#pragma unroll
                                    for (int i = 0; i < 2; ++i) {
                                        if (x0 + 2 * gi + i < nx && y0 + yy < ny) {
                                            const uint32_t g = i ? jt3[k] : it3[k];
                                            T acc = T(0);
#pragma unroll
                                            for (int p = 0; p < S; ++p) acc += (b + p * k_->nn)[g] * D[i][p];
                                            o[g] = Tio(vol ? acc * vol[g] : acc);
                                        }
                                    }
                                }
                            } else {
                                T E[2][S];
                                if constexpr (MODE == TAP_LOAD) {
                                    // E_p = (V) b0_p r  (Eq 92, Alg 4)
                                    const T* b = k_->rows + (long)pe * nxy;
                                    const T* vol = k_->vol ? k_->vol + (long)pe * nxy : nullptr;
                                    const Tio* pi = in + (long)pe * nxy;
#pragma unroll
                                    for (int i = 0; i < 2; ++i) {
                                        const uint32_t g = i ? jt3[k] : it3[k];
                                        const T x = vol ? T(pi[g]) * vol[g] : T(pi[g]);
#pragma unroll
                                        for (int p = 0; p < S; ++p) E[i][p] = (b + p * k_->nn)[g] * x;
                                    }
                                } else if (ICONST && __all((word[k] & 15) == 5)) {
                                    // interior nodes throughout the wave: the shared record
#pragma unroll
                                    for (int i = 0; i < 2; ++i)
                                        if constexpr (ICONST) point(k_->mint, k_, D[i], E[i]);
                                } else if constexpr (MODE == TAP_KN) {
                                    // rows and V from the node arrays (zero outside the domain)
                                    const T* b = k_->rows + (long)pe * nxy;
#pragma unroll
                                    for (int i = 0; i < 2; ++i) {
                                        const uint32_t g = i ? jt3[k] : it3[k];
                                        T m[ROWS * S + 1];
#pragma unroll
                                        for (int j = 0; j < ROWS * S; ++j) m[j] = (b + j * k_->nn)[g];
                                        m[ROWS * S] = (k_->vol + (long)pe * nxy)[g];
                                        point(m, k_, D[i], E[i]);
                                    }
                                } else {
#pragma unroll
                                    for (int i = 0; i < 2; ++i)
                                        point(k_->rec + (size_t)rec_at(word[k], i) * RP, k_, D[i], E[i]);
                                }
#pragma unroll
                                for (int p = 0; p < S; ++p)
                                    *reinterpret_cast<TapPair<T>*>(sE + (p * YE + yy) * XE + 2 * gi) =
                                        TapPair<T>{E[0][p], E[1][p]};
                            }
                        }
                    }
                    if constexpr (!KMODE) pe = (pe + 1 == nz) ? 0 : pe + 1;
                }
            }
            if constexpr (Bq) {
                if (s >= 2 * RZ + 2 && do5) {
                    const KP k_ = tap_fresh<(S <= 4)>(kp);
                    T g[NZ][NB5];
#pragma unroll
                    for (int e = 0; e < NZ; ++e)
#pragma unroll
                        for (int j = 0; j < NB5; ++j) g[e][j] = T(0);
                    tap_for<NY>([&](auto fc) {
                        constexpr int f = decltype(fc)::value, e = B::tab.yey[f];
                        T w[NB5 + 2 * RY];
#pragma unroll
                        for (int j = 0; j < NB5 + 2 * RY; ++j) w[j] = sF[(f * YE + y5 + j) * TX + x5];
#pragma unroll
                        for (int j = 0; j < NB5; ++j)
                            g[B::tab.yez[f]][j] += tap_conv<RY, true, e>(w + j, k_->t[1][e]);
                    });
#pragma unroll
                    for (int k = 0; k < NB5; ++k)
#pragma unroll
                        for (int j = 0; j <= 2 * RZ; ++j) {
                            const int o = RZ - j, ao = o < 0 ? -o : o;
                            T acc = j < 2 * RZ ? zout[k][j < 2 * RZ ? j + 1 : j] : T(0);
#pragma unroll
                            for (int e = 0; e < NZ; ++e) {
                                if (RZ == 0) acc += g[e][k];
                                else if (!(e > 0 && o == 0))
                                    acc = (o < 0 && (e & 1)) ? acc - k_->t[2][e][ao] * g[e][k]
                                                             : acc + k_->t[2][e][ao] * g[e][k];
                            }
                            zout[k][j] = acc;
                        }
                    if (s >= 4 * RZ + 2) {
                        const int z = zlo + s - (4 * RZ + 2);
                        const long zo = (long)z * nxy;
#pragma unroll
                        for (int k = 0; k < NB5; ++k) {
                            if (ok5[k]) {
                                const Tio v = mk5[k] ? Tio(zout[k][0]) : Tio(0);
                                (out + zo)[o5 + (uint32_t)(k * nx)] = v;
                                if constexpr (CG) {
                                    // the new p here (asked for a step ahead it cost the third
                                    // workgroup of a CU its registers: 256^3 FP32 359 us an
                                    // iteration against 283)
                                    const uint32_t g = o5 + (uint32_t)(k * nx);
                                    const T pv = up.alpha * T((up.r + zo)[g]) + up.beta * T((in + zo)[g]);
                                    dacc += (double)v * (double)pv;
                                }
                            }
                        }
                        if constexpr (CG) {
                            if (--left == 0 || z + 1 == zhi) {
                                // the partial of these planes is complete
#pragma unroll
                                for (int o = 32; o > 0; o >>= 1) dacc += __shfl_xor(dacc, o, 64);
                                if ((tid & 63) == 0) up.dsum[i5 >> 6] = dacc;
                                dacc = 0.0;
                                left = kp->cu;
                                flush = true;
                            }
                        }
                    }
                }
            }
            tap_barrier();
            // ---------------------------------------------------------- half B
            if constexpr (A && KMODE) {
                // the classes of the next plane, asked for ahead of their use
                if (s >= 2 * RZ + 1 && s + 1 < nE + 2 * RZ + 1) {
                    pe = (pe + 1 == nz) ? 0 : pe + 1;
                    const uint32_t* pw = tap_fresh<(S <= 4)>(kp)->words + (long)pe * ny * gx;
#pragma unroll
                    for (int k = 0; k < NP3; ++k) word[k] = pw[wt3[k]];
                }
            }
            if constexpr (Bq) {
                if (CG && flush) {
                    if (i5 == 0) {
                        double r = 0.0;
#pragma unroll
                        for (int w = 0; w < N5 / 64; ++w) r += up.dsum[w];
                        *dpart = r;
                    }
                    dpart += ntiles;
                    flush = false;
                }
                // the mask of the next result plane
                if (s + 1 >= 4 * RZ + 2 && s + 1 < s1) {
                    const uint8_t* pm = mask_out + (long)(zlo + s + 1 - (4 * RZ + 2)) * nxy;
#pragma unroll
                    for (int k = 0; k < NB5; ++k)
                        if (ok5[k]) mk5[k] = pm[o5 + (uint32_t)(k * nx)];
                }
            }
            if constexpr (G::P1) {
                if (s < nE + 2 * RZ && (!RO::SPLIT || !G::P2 || tid < RO::N2)) {
                    const KP k_ = tap_fresh<(S <= 4)>(kp);
                    for (int it = tid; it < XL * (YE / NB2); it += G::P2 ? RO::N2 : NT) {
                        const int x = it % XL, yb = it / XL * NB2;
                        T w[NZ][NB2 + 2 * RY];
#pragma unroll
                        for (int e = 0; e < NZ; ++e)
#pragma unroll
                            for (int j = 0; j < NB2 + 2 * RY; ++j) w[e][j] = sZ[(e * YL + yb + j) * XL + x];
                        tap_for<NY>([&](auto fc) {
                            constexpr int f = decltype(fc)::value, e = B::tab.yey[f];
#pragma unroll
                            for (int j = 0; j < NB2; ++j)
                                sY[(f * YE + yb + j) * XL + x] =
                                    tap_conv<RY, false, e>(w[B::tab.yez[f]] + j, k_->t[1][e]);
                        });
                    }
                }
            }
            if constexpr (G::P2) {
                if (s >= 2 * RZ + 1 && s < nE + 2 * RZ + 1 && (!RO::SPLIT || tid >= RO::N2)) {
                    const KP k_ = tap_fresh<(S <= 4)>(kp);
                    for (int it = RO::SPLIT ? tid - RO::N2 : tid; it < TX / XB4 * YE; it += RO::N4) {
                        const int xb = it % (TX / XB4) * XB4, yy = it / (TX / XB4);
                        T f_[NY][XB4];
#pragma unroll
                        for (int f = 0; f < NY; ++f)
#pragma unroll
                            for (int j = 0; j < XB4; ++j) f_[f][j] = T(0);
                        tap_for<S>([&](auto qc) {
                            constexpr int q = decltype(qc)::value, e = B::tab.xex[q];
                            T w[XB4 + 2 * R];
                            const TapPair<T>* src =
                                reinterpret_cast<const TapPair<T>*>(sE + (q * YE + yy) * XE + xb);
#pragma unroll
                            for (int j = 0; j < XB4 / 2 + R; ++j) {
                                const TapPair<T> v = src[j];
                                w[2 * j] = v.x;
                                w[2 * j + 1] = v.y;
                            }
#pragma unroll
                            for (int j = 0; j < XB4; ++j)
                                f_[B::tab.xyf[q]][j] += tap_conv<R, true, e>(w + j, k_->t[0][e]);
                        });
#pragma unroll
                        for (int f = 0; f < NY; ++f)
#pragma unroll
                            for (int j = 0; j < XB4 / 2; ++j)
                                reinterpret_cast<TapPair<T>*>(sF + (f * YE + yy) * TX + xb)[j] =
                                    TapPair<T>{f_[f][2 * j], f_[f][2 * j + 1]};
                    }
                }
            }
            tap_barrier();
        }
    }
};

template <typename T, typename Tio, class B, int R, int MODE, int ROWS, int TX, int TY, int NT>
__global__ __launch_bounds__(NT, tap_min_waves(sizeof(T), tap_lds_of<B, R, MODE, TX, TY>, NT, B::S, R)) void k_tap(const TapArgs<T>)
{
    using G = TapGeom<B, R, MODE, TX, TY>;
    using RO = TapRoles<B::DIM, NT>;
    __shared__ __align__(16) T smem[G::LDS > 0 ? G::LDS : 1];
    const TapArgPtr<T> kp = (TapArgPtr<T>)__builtin_amdgcn_kernarg_segment_ptr();

    const int tid = threadIdx.x;
    const int nx = kp->n[0], ny = kp->n[1], nxy = nx * ny, ntx = kp->ntx, nty = kp->nty;
    const long rj = (long)blockIdx.y * kp->rb;
    const Tio* const in = reinterpret_cast<const Tio*>((const char*)kp->in + rj);
    Tio* const out = reinterpret_cast<Tio*>((char*)kp->out + rj);
    TapUpdate<T, Tio, NT> up;
    if constexpr (MODE == TAP_CG) {
        if (!((const __attribute__((address_space(4))) int*)kp->act)[blockIdx.y]) return;
        __shared__ double sh[2][NT / 64];
        up.dsum = sh[1];
        up.sum = sh[0];
        up.r = reinterpret_cast<const Tio*>((const char*)kp->r + rj);
        up.pnew = reinterpret_cast<Tio*>((char*)kp->pnew + rj);
        up.dpart = kp->dot_part + (long)blockIdx.y * kp->dot_stride;
        if (kp->pend) {
            up.load(kp);
            if constexpr (!RO::EARLY) up.settle(kp);
        }
    }
    int b = (int)tap_xcd(blockIdx.x, gridDim.x);
    const int tx = b % ntx;
    b /= ntx;
    const int ty = b % nty;
    const int x0 = tx * TX, y0 = ty * TY;
    const int za = (b / nty) * kp->cz, ze = min(za + kp->cz, kp->n[2]);
    // planes of the chunk outside the domain's extent in this tile column are
    // zero, in every field of the result (the implicit gradient has ROWS of them)
    constexpr int NF = MODE == TAP_UH ? ROWS : 1;
    const int2 zr = kp->zr[ty * ntx + tx];
    const int zlo = min(max(za, zr.x), ze), zhi = max(zlo, min(ze, zr.y + 1));
    if (MODE != TAP_MOM && (za < zlo || zhi < ze)) {
        for (int i = tid; i < TX * TY; i += NT) {
            const int x = x0 + i % TX, y = y0 + i / TX;
            if (x < nx && y < ny) {
#pragma unroll
                for (int f = 0; f < NF; ++f) {
                    Tio* o = out + f * kp->nn + (long)y * nx + x;
                    for (int z = za; z < zlo; ++z) o[(long)z * nxy] = Tio(0);
                    for (int z = zhi; z < ze; ++z) o[(long)z * nxy] = Tio(0);
                }
            }
        }
    }
    const int ntiles = ntx * nty, tile = ty * ntx + tx;
    if constexpr (MODE == TAP_CG) {
        if (tid == 0)
            for (int u = za / kp->cu; u * kp->cu < ze; ++u)
                if (zlo >= zhi || (u + 1) * kp->cu <= zlo || u * kp->cu >= zhi)
                    up.dpart[(long)u * ntiles + tile] = 0.0;
        if (RO::EARLY && zlo >= zhi && blockIdx.x == 0 && kp->pend) up.settle(kp);  // it keeps the new r.r
    }
    if (zlo < zhi) {
        // the roles hold different state: each gets its own copy of the march
        // (both meet at the same number of barriers)
#define FC_TAP_RUN(ROLE)                                                                                          \
    TapMarch<T, Tio, B, R, MODE, ROWS, TX, TY, NT, ROLE>::run(kp, smem, in, out, tile, ntiles, x0, y0, zlo, zhi, up)
        if constexpr (!RO::SPLIT) {
            FC_TAP_RUN(3);
        } else {
            if (__builtin_amdgcn_readfirstlane(tid) < RO::NA) FC_TAP_RUN(1);
            else FC_TAP_RUN(2);
        }
#undef FC_TAP_RUN
    }
}

// Tile of a variant: the columns of one workgroup and its threads.  32 x 16
// columns over 8 waves: 64 x 16 and 32 x 32 over 16 waves overlap less but
// measured slower (256^3 FP32: 189 and 188 us against 175), 32 x 8 over 4 waves
// too (197).  The quadratic basis in 3D at R = 3 takes half the columns, so
// that its FP64 fields fit the LDS.
// SMALL: 16 x 8 columns over 4 waves, for 3D boxes that leave the chip idle.
constexpr int tap_tile_x(int dim, int degree, int r, bool small)
{
    return dim == 1 ? 256 : small || (dim == 3 && degree == 2 && r == 3) ? 16 : 32;
}
constexpr int tap_tile_y(int dim, bool small) { return dim == 1 ? 1 : small ? 8 : 16; }
constexpr int tap_threads(int dim, bool small) { return dim == 1 || small ? 256 : 512; }

// instantiated in the tap_*.hip files, a list of tap_list.hpp each
template <typename T, typename Tio, class B, int R, int MODE, int ROWS>
void tap_go(const TapArgs<T>& a, dim3 grid, bool small, hipStream_t st)
{
    if constexpr (B::DIM == 3 && (MODE == TAP_K || MODE == TAP_CG)) {
        if (small) {
            constexpr int TX = tap_tile_x(3, B::DEG, R, true), TY = tap_tile_y(3, true), NT = tap_threads(3, true);
            hipLaunchKernelGGL((k_tap<T, Tio, B, R, MODE, ROWS, TX, TY, NT>), grid, dim3(NT), 0, st, a);
            return;
        }
    }
    constexpr int TX = tap_tile_x(B::DIM, MODE == TAP_MOM ? B::DEG / 2 : B::DEG, R, false), TY = tap_tile_y(B::DIM, false);
    constexpr int NT = tap_threads(B::DIM, false);
    hipLaunchKernelGGL((k_tap<T, Tio, B, R, MODE, ROWS, TX, TY, NT>), grid, dim3(NT), 0, st, a);
}

}  // namespace fcrkpm
