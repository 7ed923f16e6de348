// tapconv.hip -- setup and dispatch of the direct tap kernels (tapconv.hpp).
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <math.h>
#include <string.h>

#include <algorithm>

#include "tap_list.hpp"

namespace fcrkpm {

namespace {

struct TapSet {
    uint32_t* words = nullptr;
    float* rec32 = nullptr;
    double* rec64 = nullptr;
    float m32[kTapMint] = {};
    double m64[kTapMint] = {};
    double words_bytes = 0.0, rec_bytes[2] = {};  // of the arrays (records: FP32, FP64)
};

void tap_check(hipError_t e)
{
    if (e != hipSuccess) raise_hip(e, "direct tap records");
}

template <typename U>
U* tap_alloc(size_t n)
{
    void* p = nullptr;
    tap_check(hipMalloc(&p, std::max<size_t>(n, 1) * sizeof(U)));
    return reinterpret_cast<U*>(p);
}

void tap_free(TapSet* s)
{
    if (!s) return;
    if (s->words) (void)hipFree(s->words);
    if (s->rec32) (void)hipFree(s->rec32);
    if (s->rec64) (void)hipFree(s->rec64);
    delete s;
}

int tile_x(const Ctx& c, bool small = false) { return tap_tile_x(c.dim, c.degree, c.tap_r, small); }
int tile_y(const Ctx& c, bool small = false) { return tap_tile_y(c.dim, small); }
int tap_gx(const Ctx& c)
{
    const int tx = tile_x(c);
    return (c.n[0] + tx - 1) / tx * (tx / 2) + c.tap_r;
}

// First and last plane with a domain node per tile column, from (nz, -1): a
// block looks at eight planes of a column.
constexpr int kExtentPlanes = 8;

__global__ void k_tap_extent_clear(int2* __restrict__ zr, int n, int nz)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) zr[i] = int2{nz, -1};
}

__global__ __launch_bounds__(256) void k_tap_extent(const uint8_t* __restrict__ chi, int nx, int ny, int nz,
                                                    int ntx, int tx, int ty, int2* __restrict__ zr)
{
    const int x0 = (blockIdx.x % ntx) * tx, y0 = (blockIdx.x / ntx) * ty;
    const int w = min(tx, nx - x0), h = min(ty, ny - y0), z0 = blockIdx.y * kExtentPlanes;
    const int np = min(kExtentPlanes, nz - z0);
    int l = nz, u = -1;
    for (int i = threadIdx.x; i < w * h * np; i += blockDim.x) {
        const int z = z0 + i / (w * h), k = i % (w * h);
        if (chi[((long)z * ny + y0 + k / w) * nx + x0 + k % w]) {
            l = min(l, z);
            u = max(u, z);
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        l = min(l, __shfl_xor(l, o, 64));
        u = max(u, __shfl_xor(u, o, 64));
    }
    if ((threadIdx.x & 63) == 0 && u >= 0) {
        atomicMin(&zr[blockIdx.x].x, l);
        atomicMax(&zr[blockIdx.x].y, u);
    }
}

// Class words and records.  A word covers two nodes along x: two bits of class
// each (0 outside the domain, 1 interior, 2 with a record of its own) and the
// index of the first record.  FILL = false counts the records, FILL = true
// hands out their places block by block and writes them, a record's values all
// read before the first is used (80^3 linear, FP64: 235 -> 155 us).
template <bool FILL>
__global__ __launch_bounds__(256) void k_tap_words(const uint8_t* __restrict__ cls,
                                                   const uint8_t* __restrict__ chi, int nx, int ny, int nz,
                                                   int gx, int r, const double* __restrict__ ba,
                                                   const double* __restrict__ vol, int rows, int s, int mform,
                                                   int rp32, int rp64, unsigned long long* __restrict__ count,
                                                   uint32_t* __restrict__ words, float* __restrict__ rec32,
                                                   double* __restrict__ rec64)
{
    const long total = (long)nz * ny * gx, nn = (long)nx * ny * nz;
    __shared__ unsigned int wsum[4];
    __shared__ unsigned long long base;
    for (long b0 = (long)blockIdx.x * 256; b0 < total; b0 += (long)gridDim.x * 256) {
        const long i = b0 + threadIdx.x;
        int k[2] = {0, 0};
        long g[2] = {0, 0};
        if (i < total) {
            const uint32_t line = (uint32_t)i / (uint32_t)gx;  // (fewer than 2^31 words)
            const int gi = (int)((uint32_t)i - line * gx);
            const long row = (long)line * nx;
            for (int j = 0; j < 2; ++j) {
                const int x = tap_wrap(2 * gi - r + j, nx);
                g[j] = row + x;
                k[j] = cls ? cls[g[j]] : (chi[g[j]] ? 2 : 0);
            }
        }
        const unsigned int n2 = (k[0] == 2) + (k[1] == 2);
        unsigned int scan = n2;
        for (int o = 1; o < 64; o <<= 1) {
            const unsigned int v = __shfl_up(scan, o, 64);
            if ((threadIdx.x & 63) >= (unsigned)o) scan += v;
        }
        if ((threadIdx.x & 63) == 63) wsum[threadIdx.x >> 6] = scan;
        __syncthreads();
        if (threadIdx.x == 0) base = atomicAdd(count, (unsigned long long)(wsum[0] + wsum[1] + wsum[2] + wsum[3]));
        __syncthreads();
        if constexpr (FILL) {
            unsigned long long at = base + scan - n2;
            for (unsigned w = 0; w < threadIdx.x >> 6; ++w) at += wsum[w];
            if (i < total) {
                words[i] = (uint32_t)k[0] | (uint32_t)k[1] << 2 | (uint32_t)at << 4;
                for (int j = 0; j < 2; ++j) {
                    if (k[j] != 2) continue;
                    float* f = rec32 + (size_t)at * rp32;
                    double* d = rec64 + (size_t)at * rp64;
                    int n = 0;
                    const auto put = [&](double v) {
                        d[n] = v;
                        f[n++] = (float)v;
                    };
                    if (mform) {
                        // at most four rows of four (the linear bases), all read
                        // before the first is used
                        double b[4][4], v = vol[g[j]];
#pragma unroll
                        for (int a = 0; a < 4; ++a)
#pragma unroll
                            for (int p = 0; p < 4; ++p)
                                b[a][p] = a < rows && p < s ? ba[(long)(a * s + p) * nn + g[j]] : 0.0;
#pragma unroll
                        for (int p = 0; p < 4; ++p)
#pragma unroll
                            for (int q = p; q < 4; ++q) {
                                double acc = 0.0;
#pragma unroll
                                for (int a = 0; a < 4; ++a) acc += b[a][p] * b[a][q];
                                if (q < s) put(v * acc);
                            }
                    } else {
#pragma unroll 8
                        for (int q = 0; q < rows * s; ++q) put(ba[(long)q * nn + g[j]]);
                        put(vol[g[j]]);
                    }
                    for (int q = n; q < rp32; ++q) f[q] = 0.0f;
                    for (int q = n; q < rp64; ++q) d[q] = 0.0;
                    ++at;
                }
            }
        }
        __syncthreads();
    }
}

// values one workgroup keeps in LDS (TapGeom of a K product)
int tap_lds(const Ctx& c, bool small)
{
    const int r = c.tap_r, d = c.degree, dim = c.dim, tx = tile_x(c, small), ty = tile_y(c, small);
    const int ry = dim > 1 ? r : 0;
    const int nz = dim > 2 ? d + 1 : 1;
    const int ny = dim > 2 ? (d + 1) * (d + 2) / 2 : dim > 1 ? d + 1 : 1;
    const int xe = tx + 2 * r, ye = ty + 2 * ry, xl = xe + 2 * r, yl = ye + 2 * ry;
    return nz * yl * xl + ny * ye * xl + c.s * ye * xe + ny * ye * tx;
}

// Tile and planes per chunk.  A chunk of cz planes takes cz + 2R + 2 steps, so
// few long chunks do the least work, but the workgroups have to fill the chip
// evenly: a step with r workgroups on a CU takes about s0 + s1 r, and a last
// round that fills a few CUs takes as long as a full one.  Measured at R = 2 in
// FP32, us a step: large tile 1.45-1.8, 1.9-2.05, 2.4-2.5 for r = 1, 2, 3; small
// tile 1.15-1.25, 1.2-1.5, 1.3-1.6, 1.5-1.7 for r = 1 to 4 (a quarter of the
// columns, so it pays only where the large tile leaves CUs idle: 32^3 10.1 us
// against 11.9, 48^3 FP64 15.9 against 17.5; 128^3 39.7 against 32.1).  In FP64:
// 1.9-2.4, 2.8-3.1; 1.35-1.8, 1.55-2.0, 1.85-2.2, 2.2-2.4.  The other radii and
// bases take the same constants: of 56 products on 3D boxes (radii 1 to 3, linear
// and quadratic, both types) 46 are within 5% of the best of all cuts; the
// quadratic basis is the furthest off (R = 3 FP32, 128^3 143 us where the best is
// 111; R = 2 FP64, 64^3 44 and 37).
struct TapCut {
    bool small;
    int cz;
    double cost;
};

// unit: the chunk has to be a multiple of so many planes.
TapCut tap_cut_tile(const Ctx& c, bool small, int nrhs, int elem, int unit)
{
    const int nz = c.n[2];
    if (c.dim < 3) return {false, 1, 0.0};
    const long tiles = (long)c.tap_nt[small][0] * c.tap_nt[small][1] * nrhs;
    const bool f64 = elem == 8;
    const int occ = tap_residents(elem, tap_lds(c, small), tap_threads(c.dim, small), c.s, c.tap_r);
    const double slots = (double)c.tap_cus * occ, s0 = f64 ? (small ? 1.25 : 1.4) : (small ? 1.0 : 1.1),
                 s1 = f64 ? (small ? 0.3 : 0.85) : (small ? 0.16 : 0.47);
    TapCut best{small, unit, 1e300};
    for (int k = (nz + unit - 1) / unit; k >= 1; --k) {
        const int cz = ((nz + k - 1) / k + unit - 1) / unit * unit;
        const double wg = (double)tiles * ((nz + cz - 1) / cz), full = floor(wg / slots), rem = wg - full * slots;
        const double t = (std::min(cz, nz) + 2 * c.tap_r + 2) *
                         (full * (s0 + s1 * occ) + (rem > 0.0 ? s0 + s1 * ceil(rem / c.tap_cus) : 0.0));
        if (t <= best.cost) best = {small, cz, t};
    }
    return best;
}

// the cheaper tile
TapCut tap_cut_best(const Ctx& c, int nrhs, int elem)
{
    const TapCut a = tap_cut_tile(c, false, nrhs, elem, 1);
    if (c.dim < 3) return a;
    const TapCut b = tap_cut_tile(c, true, nrhs, elem, 1);
    return b.cost < a.cost ? b : a;
}

// The cut of a launch over nrhs right-hand sides.  In CG it is a multiple of
// one right-hand side's, so that a batch adds up the same dot partials as
// single products.
TapCut tap_cut(const Ctx& c, int mode, int nrhs, int elem)
{
    if (mode == TAP_K) return tap_cut_best(c, nrhs, elem);
    if (mode != TAP_CG) return tap_cut_tile(c, false, nrhs, elem, 1);
    const TapCut one = tap_cut_best(c, 1, elem);
    return nrhs == 1 ? one : tap_cut_tile(c, one.small, nrhs, elem, one.cz);
}

}  // namespace

// Bases and radii with a kernel (tap_list.hpp).
bool tap_served(const Ctx& c) { return c.tap_r >= c.degree && c.tap_r >= 1 && c.tap_r <= kTapR; }

bool tap_active(const Ctx& c) { return c.use_taps && !c.fft_pins && c.tap; }

long tap_dots(const Ctx& c, int elem)
{
    const TapCut u = tap_cut_best(c, 1, elem);
    return (long)c.tap_nt[u.small][0] * c.tap_nt[u.small][1] * ((c.n[2] + u.cz - 1) / u.cz);
}

// (a rule on the geometry, the same for every operator set of a context)
long tap_dot_slots(const Ctx& c) { return tap_served(c) ? std::max(tap_dots(c, 4), tap_dots(c, 8)) : 0; }

double tap_word_bytes(const Ctx& c) { return ((const TapSet*)c.tap)->words_bytes; }
double tap_rec_bytes(const Ctx& c, int elem) { return ((const TapSet*)c.tap)->rec_bytes[elem == 8]; }

void tap_release_set(void*& s)
{
    tap_free((TapSet*)s);
    s = nullptr;
}

void tap_release(Ctx& c)
{
    tap_release_set(c.tap);
    for (auto& z : c.tap_zr) {
        if (z) (void)hipFree(z);
        z = nullptr;
    }
}

// taps and the domain's extent per tile column (once per context)
void tap_setup(Ctx& c, const double (*taps)[kTapE][4], hipStream_t st)
{
    memcpy(c.tap_t, taps, sizeof(c.tap_t));
    int dev = 0;
    tap_check(hipGetDevice(&dev));
    tap_check(hipDeviceGetAttribute(&c.tap_cus, hipDeviceAttributeMultiprocessorCount, dev));
    for (int small = 0; small < (c.dim == 3 ? 2 : 1); ++small) {
        const int tx = tile_x(c, small), ty = tile_y(c, small);
        const int nx = c.tap_nt[small][0] = (c.n[0] + tx - 1) / tx;
        const int ny = c.tap_nt[small][1] = (c.n[1] + ty - 1) / ty;
        c.tap_zr[small] = tap_alloc<int2>((size_t)nx * ny);
        hipLaunchKernelGGL(k_tap_extent_clear, dim3((nx * ny + 255) / 256), dim3(256), 0, st, c.tap_zr[small], nx * ny,
                           c.n[2]);
        hipLaunchKernelGGL(k_tap_extent, dim3(nx * ny, (c.n[2] + kExtentPlanes - 1) / kExtentPlanes), dim3(256), 0, st, c.chi, c.n[0], c.n[1], c.n[2], nx, tx,
                           ty, c.tap_zr[small]);
    }
    tap_check(hipGetLastError());
}

// words and records of the coefficient rows in use (c.ba_64, c.krows, c.cls)
void tap_build(Ctx& c, hipStream_t st)
{
    if (!tap_served(c)) return;
    TapSet* s = new TapSet();
    c.tap = s;
    const bool mf = c.degree == 1;
    const int nv = tap_rec_values(mf, c.s, c.krows);
    const int rp32 = tap_rec_pitch(mf, c.s, c.krows, 4), rp64 = tap_rec_pitch(mf, c.s, c.krows, 8);
    if (c.cls && c.nconst.bmax >= 0.0) {
        const NodeConst& nc = c.nconst;
        int n = 0;
        if (mf) {
            for (int p = 0; p < c.s; ++p)
                for (int q = p; q < c.s; ++q) {
                    double acc = 0.0;
                    for (int a = 0; a < c.krows; ++a) acc += nc.b[a * c.s + p] * nc.b[a * c.s + q];
                    s->m64[n++] = nc.v * acc;
                }
        } else {
            for (int q = 0; q < c.krows * c.s; ++q) s->m64[n++] = nc.b[q];
            s->m64[n++] = nc.v;
        }
        for (int q = 0; q < n; ++q) s->m32[q] = (float)s->m64[q];
    }
    const int gx = tap_gx(c);
    const size_t total = (size_t)c.n[2] * c.n[1] * gx;
    s->words = tap_alloc<uint32_t>(total);
    unsigned long long* cnt = reinterpret_cast<unsigned long long*>(c.dflag + 4);
    const unsigned blocks = (unsigned)std::min<size_t>((total + 255) / 256, 4096);
    const unsigned long long zero = 0;
    unsigned long long n = 0;
    tap_check(hipMemcpyAsync(cnt, &zero, sizeof(zero), hipMemcpyHostToDevice, st));
    hipLaunchKernelGGL(k_tap_words<false>, dim3(blocks), dim3(256), 0, st, c.cls, c.chi, c.n[0], c.n[1], c.n[2],
                       gx, c.tap_r, c.ba_64, c.vol64, c.krows, c.s, mf ? 1 : 0, rp32, rp64, cnt, s->words,
                       (float*)nullptr, (double*)nullptr);
    tap_check(hipMemcpyAsync(&n, cnt, sizeof(n), hipMemcpyDeviceToHost, st));
    tap_check(hipStreamSynchronize(st));
    if (n + 2 >= (1ull << 28)) {  // a word holds 28 bits of record index
        tap_release_set(c.tap);
        return;
    }
    n += 2;  // records 0 and 1: a node outside the domain (zero) and the interior nodes'
    s->words_bytes = (double)total * sizeof(uint32_t);
    s->rec_bytes[0] = (double)n * rp32 * sizeof(float);
    s->rec_bytes[1] = (double)n * rp64 * sizeof(double);
    s->rec32 = tap_alloc<float>((size_t)n * rp32);
    s->rec64 = tap_alloc<double>((size_t)n * rp64);
    std::vector<float> h32((size_t)2 * rp32, 0.0f);
    std::vector<double> h64((size_t)2 * rp64, 0.0);
    const int ni = std::min(nv, kTapMint);  // wider records have no interior class
    std::copy(s->m32, s->m32 + ni, h32.begin() + rp32);
    std::copy(s->m64, s->m64 + ni, h64.begin() + rp64);
    tap_check(hipMemcpyAsync(s->rec32, h32.data(), h32.size() * sizeof(float), hipMemcpyHostToDevice, st));
    tap_check(hipMemcpyAsync(s->rec64, h64.data(), h64.size() * sizeof(double), hipMemcpyHostToDevice, st));
    const unsigned long long first = 2;
    tap_check(hipMemcpyAsync(cnt, &first, sizeof(first), hipMemcpyHostToDevice, st));
    hipLaunchKernelGGL(k_tap_words<true>, dim3(blocks), dim3(256), 0, st, c.cls, c.chi, c.n[0], c.n[1], c.n[2],
                       gx, c.tap_r, c.ba_64, c.vol64, c.krows, c.s, mf ? 1 : 0, rp32, rp64, cnt, s->words,
                       s->rec32, s->rec64);
    tap_check(hipGetLastError());
    tap_check(hipStreamSynchronize(st));
}

// Workgroups of a row of the grid, a multiple of eight so that tap_xcd orders
// every grid: those beyond the last chunk start past the last plane and find
// nothing to do (without: 8 right-hand sides of 80^3 FP32 56.1 us against 51.4, of
// 48^3 FP64 34.7 against 30.4, 32 of 96^3 FP64 455 against 434).
static unsigned tap_grid(const Ctx& c, int ntx, int nty, int cz)
{
    const long n = (long)ntx * nty * ((c.n[2] + cz - 1) / cz);
    return (unsigned)((n + 7) / 8 * 8);
}

// what every launch passes
template <typename T>
static TapArgs<T> tap_args(const Ctx& c)
{
    TapArgs<T> a = {};
    for (int k = 0; k < 3; ++k) {
        a.n[k] = c.n[k];
        for (int e = 0; e < kTapE; ++e)
            for (int o = 0; o <= kTapR; ++o) a.t[k][e][o] = (T)c.tap_t[k][e][o];
    }
    a.nn = c.nn;
    return a;
}

void launch_tap_moments(const Ctx& c, cplx<double>* G, hipStream_t st)
{
    TapArgs<double> a = tap_args<double>(c);
    a.out = G;
    a.mask_in = c.chi;
    const TapCut cut = tap_cut_tile(c, false, 1, 8, 1);
    a.ntx = c.tap_nt[0][0];
    a.nty = c.tap_nt[0][1];
    a.cz = a.cu = cut.cz;
    a.zr = c.tap_zr[0];
    const dim3 grid(tap_grid(c, a.ntx, a.nty, a.cz));
    bool done = false;
#define FC_TAP_CASE(T_, TIO_, DIM, DEG, R, MODE, ROWS)                            \
    if (!done && c.dim == DIM && 2 * c.degree == DEG && c.tap_r == R) {           \
        tap_go<T_, TIO_, TapBasis<DIM, DEG>, R, MODE, ROWS>(a, grid, false, st);  \
        done = true;                                                              \
    }
    FC_TAP_MOM(FC_TAP_CASE)
#undef FC_TAP_CASE
    if (!done) raise_unsupported("internal: no moment kernel for this basis");
    tap_check(hipGetLastError());
}

template <typename T, typename Tio>
void launch_tap(const Ctx& c, int mode, const Tio* in, Tio* out, const uint8_t* mask_in,
                const uint8_t* mask_out, const T* rows_in, const T* vol, int nrhs, hipStream_t st, const TapCg* cg)
{
    const TapSet& s = *(const TapSet*)c.tap;
    TapArgs<T> a = tap_args<T>(c);
    a.in = in;
    a.out = out;
    a.mask_in = mask_in;
    a.mask_out = mask_out;
    const TapCut cut = tap_cut(c, mode, nrhs, sizeof(T));
    a.ntx = c.tap_nt[cut.small][0];
    a.nty = c.tap_nt[cut.small][1];
    a.cu = cg ? tap_cut_best(c, 1, sizeof(T)).cz : cut.cz;
    a.cz = cut.cz;
    a.zr = c.tap_zr[cut.small];
    a.words = s.words;
    a.gx = tap_gx(c);
    if constexpr (sizeof(T) == 8) {
        a.rec = s.rec64;
        memcpy(a.mint, s.m64, sizeof(a.mint));
        if (mode == TAP_KN) memcpy(a.mint, c.cint64, sizeof(double) * (c.dim * c.s + 1));
    } else {
        a.rec = s.rec32;
        memcpy(a.mint, s.m32, sizeof(a.mint));
    }
    a.rows = rows_in;
    if (cg) {
        a.r = cg->r;
        a.pnew = cg->pnew;
        a.dot_part = cg->dot_part;
        a.dot_stride = cg->dot_stride;
        a.pend = cg->pend;
        a.rr_part = cg->rr_part;
        a.nrr = cg->nrr;
        a.parity = cg->parity;
        a.scal = cg->scal;
        a.act = cg->act;
    }
    a.vol = vol;
    a.kappa = (T)c.pw_kappa;
    a.rb = c.nn * (long)sizeof(Tio) * (mode == TAP_GRAD ? c.dim : 1);
    const dim3 grid(tap_grid(c, a.ntx, a.nty, a.cz), (unsigned)nrhs);
    // the linear bases keep M, whatever the rows it was made of
    const int rows = mode == TAP_K || mode == TAP_CG ? (c.degree > 1 ? c.krows : c.dim) : mode == TAP_KN || mode == TAP_GRAD ? c.dim : 1;
    const int kmode = mode == TAP_GRAD ? TAP_UH : mode;
    bool done = false;
#define FC_TAP_CASE(T_, TIO_, DIM, DEG, R, MODE, ROWS)                                              \
    if (!done && c.dim == DIM && c.degree == DEG && c.tap_r == R && kmode == MODE && rows == ROWS) { \
        tap_go<T_, TIO_, TapBasis<DIM, DEG>, R, MODE, ROWS>(a, grid, cut.small, st);                       \
        done = true;                                                                                \
    }
    if constexpr (sizeof(T) == 8) {
        FC_TAP_F64(FC_TAP_CASE)
        FC_TAP_F64N(FC_TAP_CASE)
        FC_TAP_CG64(FC_TAP_CASE)
    } else if constexpr (sizeof(Tio) == 4) {
        FC_TAP_F32(FC_TAP_CASE)
        FC_TAP_CG32(FC_TAP_CASE)
    } else {
        FC_TAP_MIX(FC_TAP_CASE)
    }
#undef FC_TAP_CASE
    if (!done) raise_unsupported("internal: no direct kernel for this basis");
}

template void launch_tap<float, float>(const Ctx&, int, const float*, float*, const uint8_t*, const uint8_t*,
                                       const float*, const float*, int, hipStream_t, const TapCg*);
template void launch_tap<double, double>(const Ctx&, int, const double*, double*, const uint8_t*,
                                         const uint8_t*, const double*, const double*, int, hipStream_t,
                                         const TapCg*);
template void launch_tap<float, double>(const Ctx&, int, const double*, double*, const uint8_t*,
                                        const uint8_t*, const float*, const float*, int, hipStream_t,
                                        const TapCg*);

}  // namespace fcrkpm
