// spectral.hip -- second-derivative tensors of a periodic grid field, for the tidal-tensor and
// Hessian analysis the paper lists as future grid outputs (section 4):
//   tidal:   T_ij = d_i d_j phi,  laplacian(phi) = delta,  delta = f / mean(f) - 1
//            -> T_ij(k) = k_i k_j / |k|^2 * f(k) / mean(f)   (k != 0; 0 at k = 0)
//   Hessian: H_ij = d_i d_j f  ->  H_ij(k) = -k_i k_j f(k)
// with k_a = 2 pi m / L_a, m the signed frequency index.  A mixed component (i != j) is set to
// zero on the Nyquist plane of either of its axes, where the sign of k is ambiguous; this keeps
// every multiplier even in k, so every component is real.
//
// The transforms are bound by HBM, so the work is ordered to move few bytes.  The field is real:
// a row of n2 values becomes n2/2 + 1 complex ones, and with the last of them (the Nyquist plane,
// kept apart) the rest fills exactly the row's own bytes.  A multiplier k_i k_j g(k) is a product
// of per-axis factors, so the six components share transforms as long as they agree on the axes
// done so far:
//   k_fft_rows   rows of f along z, real to half-complex        8 B read,  8 B written a point
//   k_fft_y      y, in place                                     8          8
//   k_fft_x      x forward, g(k) = f(k) / |k|^2 (or -f(k)), and back by three inverse
//                transforms: g, k_x g and k_x^2 g                8         24
//   k_fft_y      back along y: k_x^2 g -> xx; k_x g -> xy, xz;
//                g -> yy, yz, zz (times k_y^2, k_y, 1)          48         48
//   k_unfft_rows the factors of k_z, back to real rows          48         48
// in all 256 B a point.  The intermediate arrays are the six output arrays themselves (each pass
// of a line is done in place or into a component not yet used), so scratch is the planes of Nyquist
// values only, 96 / n2 B a point.  At 256^3 this took 2.16 ms when the field was widened to
// complex, every component had its own three inverse passes and multiply and unpack passes stood
// between them (600 B a point, 4.7 TB/s, the rate of a large copy); now 1.00 ms, 4.3 TB/s: the y
// passes at 4.4-4.9 TB/s, the row passes at 3-3.9 (their three exchanges through LDS leave less in
// flight) and k_fft_x at 2.6 (its g beside the transform's values leaves three waves per SIMD;
// capped to four it spills and the whole takes 1.06 ms).  Measured and not kept: y and z passes by
// slabs of x planes, whose intermediates stay in the memory-side cache (1.07-1.66 ms for 4M to 1M
// points a slab: shorter launches, with more of each spent filling and draining the chip).
//
// A block takes B lines of N complex values, eight per thread (2048 per block of 256 threads,
// lines of 4096 by 512 threads).  A transform is Stockham's: radix-8 passes and a last one of 8, 4
// or 2, each from and to registers, with an exchange through LDS between two passes.  In every
// pass a thread's eight values are those at j + q N / 8, so the first pass takes what the thread
// loaded from HBM and the last leaves what it stores there, both with consecutive threads on
// consecutive addresses (along a row, across the lines of the other axes).  LDS lines are padded
// by one value in eight and to an odd pitch, which keeps the exchanges free of bank conflicts.
// The twiddles are one table per block, computed with sincospi in FP64.
#include <mutex>

#include "vt_internal.h"

// a complex value at the alignment of the caller's doubles
struct cd {
    double x, y;
};

__device__ __forceinline__ cd cmul(cd a, cd b) { return {fma(a.x, b.x, -(a.y * b.y)), fma(a.x, b.y, a.y * b.x)}; }
__device__ __forceinline__ cd cadd(cd a, cd b) { return {a.x + b.x, a.y + b.y}; }
__device__ __forceinline__ cd csub(cd a, cd b) { return {a.x - b.x, a.y - b.y}; }
__device__ __forceinline__ cd cscale(cd a, double s) { return {a.x * s, a.y * s}; }
// i s a
template <int SIGN>
__device__ __forceinline__ cd crot(cd a) {
    return SIGN > 0 ? cd{-a.y, a.x} : cd{a.y, -a.x};
}

template <int SIGN>
__device__ __forceinline__ void dft2(cd &a, cd &b) {
    const cd t = a;
    a = cadd(t, b);
    b = csub(t, b);
}
template <int SIGN>
__device__ __forceinline__ void dft4(cd &a, cd &b, cd &c, cd &d) {
    const cd p = cadd(a, c), q = csub(a, c), r = cadd(b, d), s = crot<SIGN>(csub(b, d));
    a = cadd(p, r);
    b = cadd(q, s);
    c = csub(p, r);
    d = csub(q, s);
}
template <int SIGN>
__device__ __forceinline__ void dft8(cd v[8]) {
    dft4<SIGN>(v[0], v[2], v[4], v[6]);
    dft4<SIGN>(v[1], v[3], v[5], v[7]);
    const double h = 0.70710678118654752440;
    // times exp(SIGN i pi q / 4)
    const cd o1 = {h * (v[3].x - SIGN * v[3].y), h * (v[3].y + SIGN * v[3].x)};
    const cd o2 = crot<SIGN>(v[5]);
    const cd o3 = {-h * (v[7].x + SIGN * v[7].y), -h * (v[7].y - SIGN * v[7].x)};
    const cd e0 = v[0], e1 = v[2], e2 = v[4], e3 = v[6], o0 = v[1];
    v[0] = cadd(e0, o0);
    v[4] = csub(e0, o0);
    v[1] = cadd(e1, o1);
    v[5] = csub(e1, o1);
    v[2] = cadd(e2, o2);
    v[6] = csub(e2, o2);
    v[3] = cadd(e3, o3);
    v[7] = csub(e3, o3);
}

// A block's lines and the thread's place in them.  Rows (contiguous lines) give consecutive
// threads consecutive values of a line, the other axes consecutive lines.
struct Lines {
    int logn, N, B, pitch;
    int l, j;         // N >= 8: the thread's line and its first value; value q is j + q N / 8
    __device__ __forceinline__ void init(int logn_, bool rows) {
        logn = logn_;
        N = 1 << logn;
        pitch = (N + (N >> 3)) | 1;
        B = (8 * (int)blockDim.x) >> logn;
        const int t = threadIdx.x;
        if (N >= 8) {
            const int tl = N >> 3;
            l = rows ? t / tl : t % B;
            j = rows ? t % tl : t / B;
        } else {
            l = j = 0;
        }
    }
    // line and index of the thread's value q (lines shorter than eight: 8 / N whole lines a thread)
    __device__ __forceinline__ int line(int q) const { return N >= 8 ? l : (int)threadIdx.x * (8 >> logn) + (q >> logn); }
    __device__ __forceinline__ int elem(int q) const { return N >= 8 ? j + q * (N >> 3) : q & (N - 1); }
    __device__ __forceinline__ int at(int l_, int i) const { return l_ * pitch + i + (i >> 3); }
};

// exp(2 pi i m / n) for m < n / 2 into tw (n >= 2)
__device__ __forceinline__ void twiddles(cd *tw, int n) {
    for (int m = threadIdx.x; m < n / 2; m += blockDim.x) {
        double s, c;
        sincospi(2.0 * (double)m / (double)n, &s, &c);
        tw[m] = {c, s};
    }
}
// exp(SIGN 2 pi i m / n), m < n, from the half table
template <int SIGN>
__device__ __forceinline__ cd twiddle(const cd *tw, int n, int m) {
    const cd t = tw[m & (n / 2 - 1)];
    const double s = m >= n / 2 ? -1.0 : 1.0;
    return {s * t.x, SIGN * s * t.y};
}

// The transform of the block's lines, value q of each thread in v[q] before and after; tw holds
// the half table for n = N << twshift.  Every thread of the block takes part; the LDS is free for
// other use after the barrier at the start and must not be read by others afterwards without one.
template <int SIGN>
__device__ __forceinline__ void fft(const Lines &Z, cd v[8], cd *lds, const cd *tw, int twshift) {
    const int N = Z.N, logn = Z.logn;
    if (logn < 3) {
        if (logn == 2) {
            dft4<SIGN>(v[0], v[1], v[2], v[3]);
            dft4<SIGN>(v[4], v[5], v[6], v[7]);
        } else if (logn == 1) {
#pragma unroll
            for (int q = 0; q < 8; q += 2) dft2<SIGN>(v[q], v[q + 1]);
        }
        return;
    }
    const int nt = N << twshift;
    int ls = 0;  // log2 of the product of the radices done
    while (logn - ls >= 3) {
        const int k = Z.j & ((1 << ls) - 1);
        if (ls > 0) {
            const int step = (k << (logn - 3 - ls)) << twshift;
#pragma unroll
            for (int q = 1; q < 8; ++q) v[q] = cmul(v[q], twiddle<SIGN>(tw, nt, q * step));
        }
        dft8<SIGN>(v);
        const int base = ((Z.j >> ls) << (ls + 3)) + k;
        ls += 3;
        if (ls == logn) return;  // the last pass leaves value q at j + q N / 8
        __syncthreads();
#pragma unroll
        for (int q = 0; q < 8; ++q) lds[Z.at(Z.l, base + (q << (ls - 3)))] = v[q];
        __syncthreads();
#pragma unroll
        for (int q = 0; q < 8; ++q) v[q] = lds[Z.at(Z.l, Z.elem(q))];
    }
    // the last pass: butterflies j + p N / 8, whose values are v[p + r (8 / R)]
    if (logn - ls == 2) {
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            const int k = (Z.j + p * (N >> 3)) << twshift;
#pragma unroll
            for (int r = 1; r < 4; ++r) v[p + 2 * r] = cmul(v[p + 2 * r], twiddle<SIGN>(tw, nt, r * k));
            dft4<SIGN>(v[p], v[p + 2], v[p + 4], v[p + 6]);
        }
    } else {
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            const int k = (Z.j + p * (N >> 3)) << twshift;
            v[p + 4] = cmul(v[p + 4], twiddle<SIGN>(tw, nt, k));
            dft2<SIGN>(v[p], v[p + 4]);
        }
    }
}

// Half-complex arrays of a grid n0 x n1 x n2: `main` holds k_z = 0 .. n2/2 - 1 (pitch n2/2), `nyq`
// the plane k_z = n2/2 as n0 x n1.
struct Half {
    cd *main, *nyq;
};

struct TensorGeo {
    int n[3], logn[3];
    double k1[3];   // wave number per index: 2 pi / L (Hessian), L_0 / L (tidal, where only ratios count)
    int tidal;
    double *dc;     // the field's sum, written by k_fft_x and read by k_unfft_rows
};

// signed wave number of index m along axis a; zero_nyq: the factor of a mixed component
__device__ __forceinline__ double wavenumber(const TensorGeo &G, int a, int m, bool zero_nyq) {
    const int h = G.n[a] / 2;
    if (zero_nyq && m == h) return 0.0;
    return (double)(m < h ? m : m - G.n[a]) * G.k1[a];
}

// Lines along axis 0 or 1 of a half-complex array with `no` planes along the other of the two: the
// main part's lines, B to a block, then the Nyquist plane's.  Gives the line's first value, the
// stride along it and its (other axis, k_z).
struct HalfLine {
    bool valid, nyq;
    int64_t first, stride;
    int other, kz;
};
__device__ __forceinline__ HalfLine half_line(const TensorGeo &G, int axis, int no, int64_t main_tiles, int B, int l) {
    const int logm = G.logn[2] - 1, M = 1 << logm;
    const int64_t tile = blockIdx.x;
    HalfLine h;
    h.nyq = tile >= main_tiles;
    const int64_t line = (tile - (h.nyq ? main_tiles : 0)) * B + l;
    h.valid = line < (h.nyq ? (int64_t)no : (int64_t)no * M);
    const int64_t o = h.nyq ? line : line >> logm;
    h.kz = h.nyq ? M : (int)(line & (M - 1));
    h.other = (int)o;
    const int64_t row = h.nyq ? 1 : M, z = h.nyq ? 0 : h.kz;
    if (axis == 1) {
        h.first = o * G.n[1] * row + z;
        h.stride = row;
    } else {
        h.first = o * row + z;
        h.stride = G.n[1] * row;
    }
    return h;
}

extern __shared__ cd fft_lds[];

// z: rows of reals to half-complex rows.  A row of n2 = 2 M reals is transformed as M complex
// values z_m = f_2m + i f_2m+1; with w = exp(-2 pi i k / n2), X_k = (Z_k + conj Z_M-k) / 2
// - i w (Z_k - conj Z_M-k) / 2.
__global__ void __launch_bounds__(256) k_fft_rows(TensorGeo G, const cd *f, Half S, int64_t rows) {
    Lines Z;
    const int M = G.n[2] / 2;
    Z.init(G.logn[2] - 1, true);
    const int64_t r0 = (int64_t)blockIdx.x * Z.B;
    cd *tw = fft_lds + Z.B * Z.pitch;
    cd v[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const int64_t r = r0 + Z.line(q);
        v[q] = r < rows ? f[r * M + Z.elem(q)] : cd{0.0, 0.0};
    }
    twiddles(tw, 2 * M);
    __syncthreads();
    fft<-1>(Z, v, fft_lds, tw, 1);
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 8; ++q) fft_lds[Z.at(Z.line(q), Z.elem(q))] = v[q];
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const int l = Z.line(q), k = Z.elem(q);
        const int64_t r = r0 + l;
        if (r >= rows) continue;
        if (k == 0) {
            S.main[r * M] = {v[q].x + v[q].y, 0.0};
            S.nyq[r] = {v[q].x - v[q].y, 0.0};
        } else {
            const cd m = fft_lds[Z.at(l, M - k)];
            const cd e = {0.5 * (v[q].x + m.x), 0.5 * (v[q].y - m.y)};
            const cd o = cmul({0.5 * (v[q].x - m.x), 0.5 * (v[q].y + m.y)}, twiddle<-1>(tw, 2 * M, k));
            S.main[r * M + k] = {e.x + o.y, e.y - o.x};
        }
    }
}

// z back: half-complex rows, times the component's factor of k_z and the scale, to rows of reals in
// place (with w as above, Z_k = X_k + conj X_M-k + i conj(w) (X_k - conj X_M-k)).  Component
// blockIdx.y takes k_z to the power pow (0, 1 or 2).
struct ZJobs {
    Half h[6];
    int pow[6];
};
__global__ void __launch_bounds__(256) k_unfft_rows(TensorGeo G, ZJobs J, int64_t rows) {
    Lines Z;
    const int M = G.n[2] / 2;
    Z.init(G.logn[2] - 1, true);
    const Half S = J.h[blockIdx.y];
    const int kzpow = J.pow[blockIdx.y];
    const int64_t r0 = (int64_t)blockIdx.x * Z.B;
    // room for M + 1 values a row
    cd *tw = fft_lds + Z.B * (Z.pitch + 1);
    cd *nyq = fft_lds + Z.B * Z.pitch;
    cd v[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const int64_t r = r0 + Z.line(q);
        v[q] = r < rows ? S.main[r * M + Z.elem(q)] : cd{0.0, 0.0};
    }
    const double total = *G.dc;
    twiddles(tw, 2 * M);
    const double scale = 1.0 / (G.tidal ? total : -(double)G.n[0] * (double)G.n[1] * (double)G.n[2]);
    auto factor = [&](int k) {
        const double kz = wavenumber(G, 2, k, kzpow == 1);
        return kzpow == 0 ? scale : kzpow == 1 ? kz * scale : kz * kz * scale;
    };
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const int l = Z.line(q), k = Z.elem(q);
        const int64_t r = r0 + l;
        v[q] = cscale(v[q], factor(k));
        if (k == 0) nyq[l] = r < rows ? cscale(S.nyq[r], factor(M)) : cd{0.0, 0.0};
        fft_lds[Z.at(l, k)] = v[q];
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const int l = Z.line(q), k = Z.elem(q);
        const cd m = k == 0 ? nyq[l] : fft_lds[Z.at(l, M - k)];
        const cd e = {v[q].x + m.x, v[q].y - m.y};
        const cd o = cmul({v[q].x - m.x, v[q].y + m.y}, twiddle<1>(tw, 2 * M, k));
        v[q] = {e.x - o.y, e.y + o.x};
    }
    fft<1>(Z, v, fft_lds, tw, 1);
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const int64_t r = r0 + Z.line(q);
        if (r < rows) S.main[r * M + Z.elem(q)] = v[q];
    }
}

// y, forward (SIGN -1) or back (SIGN 1): job blockIdx.y transforms S times k_y to the power pow into
// O, which may be S.
struct YJobs {
    Half S[4], O[4];
    int pow[4];
};
template <int SIGN>
__global__ void __launch_bounds__(512) k_fft_y(TensorGeo G, YJobs J, int nx, int64_t main_tiles) {
    const Half S = J.S[blockIdx.y], O = J.O[blockIdx.y];
    const int pw = J.pow[blockIdx.y];
    Lines Z;
    Z.init(G.logn[1], false);
    const HalfLine h0 = half_line(G, 1, nx, main_tiles, Z.B, Z.line(0));
    cd *tw = fft_lds + Z.B * Z.pitch;
    cd v[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const HalfLine h = Z.N >= 8 ? h0 : half_line(G, 1, nx, main_tiles, Z.B, Z.line(q));
        const cd *p = h.nyq ? S.nyq : S.main;
        v[q] = h.valid ? p[h.first + Z.elem(q) * h.stride] : cd{0.0, 0.0};
    }
    twiddles(tw, Z.N);
    if (pw != 0) {
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const double ky = wavenumber(G, 1, Z.elem(q), pw == 1);
            v[q] = cscale(v[q], pw == 1 ? ky : ky * ky);
        }
    }
    __syncthreads();
    fft<SIGN>(Z, v, fft_lds, tw, 0);
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const HalfLine h = Z.N >= 8 ? h0 : half_line(G, 1, nx, main_tiles, Z.B, Z.line(q));
        cd *p = h.nyq ? O.nyq : O.main;
        if (h.valid) p[h.first + Z.elem(q) * h.stride] = v[q];
    }
}

// x forward, the shared multiplier g(k), and back: O0 = g, O1 = k_x g, O2 = k_x^2 g.  S may be any
// of the three (every line is read whole before it is written).
__global__ void __launch_bounds__(512) k_fft_x(TensorGeo G, Half S, Half O0, Half O1, Half O2, int64_t main_tiles) {
    Lines Z;
    Z.init(G.logn[0], false);
    const HalfLine h0 = half_line(G, 0, G.n[1], main_tiles, Z.B, Z.line(0));
    cd *tw = fft_lds + Z.B * Z.pitch;
    cd g[8], v[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const HalfLine h = Z.N >= 8 ? h0 : half_line(G, 0, G.n[1], main_tiles, Z.B, Z.line(q));
        const cd *p = h.nyq ? S.nyq : S.main;
        g[q] = h.valid ? p[h.first + Z.elem(q) * h.stride] : cd{0.0, 0.0};
    }
    twiddles(tw, Z.N);
    __syncthreads();
    fft<-1>(Z, g, fft_lds, tw, 0);
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const HalfLine h = Z.N >= 8 ? h0 : half_line(G, 0, G.n[1], main_tiles, Z.B, Z.line(q));
        const int kx = Z.elem(q);
        if (h.valid && !h.nyq && kx == 0 && h.other == 0 && h.kz == 0) *G.dc = g[q].x;
        if (G.tidal) {
            const double a = wavenumber(G, 0, kx, false), b = wavenumber(G, 1, h.other, false),
                         c = wavenumber(G, 2, h.kz, false);
            const double k2 = a * a + b * b + c * c;
            g[q] = k2 > 0.0 ? cscale(g[q], 1.0 / k2) : cd{0.0, 0.0};
        }
    }
#pragma unroll 1
    for (int o = 0; o < 3; ++o) {
        const Half O = o == 0 ? O0 : o == 1 ? O1 : O2;
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const double kx = wavenumber(G, 0, Z.elem(q), o == 1);
            v[q] = o == 0 ? g[q] : cscale(g[q], o == 1 ? kx : kx * kx);
        }
        fft<1>(Z, v, fft_lds, tw, 0);
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const HalfLine h = Z.N >= 8 ? h0 : half_line(G, 0, G.n[1], main_tiles, Z.B, Z.line(q));
            cd *p = h.nyq ? O.nyq : O.main;
            if (h.valid) p[h.first + Z.elem(q) * h.stride] = v[q];
        }
    }
}

// threads per block for lines of N = 2^logn values, lines per block, and the block's LDS
static int fft_threads(int logn) { return logn > 11 ? 512 : 256; }
static int fft_lines(int logn) { return (8 * fft_threads(logn)) >> logn; }
static size_t fft_lds_bytes(int logn, int ntw, bool extra) {
    const int N = 1 << logn, pitch = ((N + (N >> 3)) | 1) + (extra ? 1 : 0);
    return sizeof(cd) * ((size_t)fft_lines(logn) * pitch + (ntw > 1 ? ntw / 2 : 1));
}

template <typename K, typename... A>
static hipError_t fft_launch(K kern, dim3 blocks, int threads, size_t lds, hipStream_t s, A... args) {
    hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    kern<<<blocks, dim3((unsigned)threads), lds, s>>>(args...);
    return hipGetLastError();
}

// Scratch values (complex) a call needs: Nyquist planes (see grid_tensor_into) and the field's sum.
static int tensor_planes(int nz) { return nz >= 4 ? 6 : 3; }
static int64_t tensor_scratch(int nx, int ny, int nz) { return tensor_planes(nz) * (int64_t)nx * ny + 1; }

static hipError_t grid_tensor_into(vt_ctx *c, const double *grid, int nx, int ny, int nz, int kind, double *out,
                                   cd *scratch_) {
    const int64_t ntot = (int64_t)nx * ny * nz, plane = (int64_t)nx * ny;
    hipStream_t s = c->stream;
    TensorGeo G;
    G.n[0] = nx;
    G.n[1] = ny;
    G.n[2] = nz;
    G.tidal = kind == VT_TENSOR_TIDAL ? 1 : 0;
    const double *L = c->h_items[0].L;
    for (int a = 0; a < 3; ++a) {
        G.logn[a] = 0;
        while ((1 << G.logn[a]) < G.n[a]) ++G.logn[a];
        G.k1[a] = G.tidal ? L[0] / L[a] : 2.0 * M_PI / L[a];
    }
    G.dc = (double *)(scratch_ + tensor_planes(nz) * plane);
    enum { XX, YY, ZZ, XY, XZ, YZ };
    // component comp's array with Nyquist plane p
    auto half = [&](int comp, int p) { return Half{(cd *)(out + comp * ntot), scratch_ + p * plane}; };
    // The field's spectrum is made in ZZ's array; a field that overlaps it other than exactly
    // (rows would be written before they are read) has it made in XX's, which it cannot reach too.
    const double *z0 = out + ZZ * ntot;
    const bool clash = grid != z0 && grid < z0 + ntot && grid + ntot > z0;
    const Half S = half(clash ? XX : ZZ, 0);
    const int lz = G.logn[2] - 1, ly = G.logn[1], lx = G.logn[0], M = nz / 2;
    const unsigned bz = (unsigned)((plane + fft_lines(lz) - 1) / fft_lines(lz));
    const size_t mz = fft_lds_bytes(lz, nz, true), my = fft_lds_bytes(ly, ny, false), mx = fft_lds_bytes(lx, nx, false);
    auto tiles = [&](int lg, int other, int64_t *main_tiles) {
        const int B = fft_lines(lg);
        *main_tiles = ((int64_t)other * M + B - 1) / B;
        return (unsigned)(*main_tiles + (other + B - 1) / B);
    };
    int64_t ty, tx;
    const unsigned by = tiles(ly, nx, &ty), bx = tiles(lx, ny, &tx);
    hipError_t e = fft_launch(k_fft_rows, dim3(bz), fft_threads(lz), mz, s, G, (const cd *)grid, S, plane);
    if (e == hipSuccess) e = fft_launch(k_fft_y<-1>, dim3(by), fft_threads(ly), my, s, G, YJobs{{S}, {S}, {0}}, nx, ty);
    const Half A0 = half(ZZ, 0), A1 = half(XZ, 1), A2 = half(XX, 2);
    if (e == hipSuccess) e = fft_launch(k_fft_x, dim3(bx), fft_threads(lx), mx, s, G, S, A0, A1, A2, tx);
    auto along_y = [&](unsigned njobs, const YJobs &J) {
        if (e == hipSuccess) e = fft_launch(k_fft_y<1>, dim3(by, njobs), fft_threads(ly), my, s, G, J, nx, ty);
    };
    auto along_z = [&](unsigned njobs, const ZJobs &J) {
        if (e == hipSuccess) e = fft_launch(k_unfft_rows, dim3(bz, njobs), fft_threads(lz), mz, s, G, J, plane);
    };
    // the components made in place of a field follow the others made from it
    if (nz >= 4) {
        const Half xy = half(XY, 3), yy = half(YY, 4), yz = half(YZ, 5);
        along_y(4, YJobs{{A0, A0, A1, A2}, {yy, yz, xy, A2}, {2, 1, 1, 0}});
        along_y(2, YJobs{{A0, A1}, {A0, A1}, {0, 0}});
        along_z(6, ZJobs{{A2, yy, A0, xy, A1, yz}, {0, 0, 2, 0, 1, 1}});
    } else {
        // rows of two: a Nyquist plane is half a component, and three of them (48 bytes a row) are
        // all the allocation-free scratch holds; a plane is used again when its component is done
        along_y(1, YJobs{{A2}, {A2}, {0}});
        along_z(1, ZJobs{{A2}, {0}});
        const Half xy = half(XY, 2);
        along_y(1, YJobs{{A1}, {xy}, {1}});
        along_y(1, YJobs{{A1}, {A1}, {0}});
        along_z(2, ZJobs{{xy, A1}, {0, 1}});
        const Half yy = half(YY, 1), yz = half(YZ, 2);
        along_y(2, YJobs{{A0, A0}, {yy, yz}, {2, 1}});
        along_y(1, YJobs{{A0}, {A0}, {0}});
        along_z(3, ZJobs{{yy, A0, yz}, {0, 2, 1}});
    }
    return e;
}

hipError_t vt_launch_grid_tensor(vt_ctx *c, const double *grid, int nx, int ny, int nz, int kind, double *out) {
    const int64_t need = tensor_scratch(nx, ny, nz);
    if (c->cap_spec < need) {
        (void)hipFree(c->spec_buf);
        c->spec_buf = nullptr;
        c->cap_spec = 0;
        hipError_t e = hipMalloc(&c->spec_buf, sizeof(cd) * (size_t)need);
        if (e != hipSuccess) return e;
        c->cap_spec = need;
    }
    return grid_tensor_into(c, grid, nx, ny, nz, kind, out, (cd *)c->spec_buf);
}

// ---------------------------------------------------------------- allocation-free variant
// Scratch for vt_grid_tensor_noalloc: the Nyquist planes of a grid of at most
// VT_NOALLOC_TENSOR_POINTS points (64 MiB: three planes of rows of two, or six of rows of four, take
// 48), one copy per device, held until the process ends.
// In host code `scratch` names a host-side stand-in; kernels get the device address that
// hipGetSymbolAddress returns for the current device.
static __device__ __align__(256) double2 scratch[2 * (size_t)VT_NOALLOC_TENSOR_POINTS];

#define VT_MAX_DEVICES 64
static void *g_scratch_ptr[VT_MAX_DEVICES];
static std::mutex g_scratch_mu;

// the calling thread's current device's copy of `scratch` (looked up once per device)
static hipError_t scratch_address(cd **ptr) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= VT_MAX_DEVICES) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        g_scratch_ptr[dev] = p;
    }
    *ptr = (cd *)g_scratch_ptr[dev];
    return hipSuccess;
}

hipError_t vt_launch_grid_tensor_noalloc(vt_ctx *c, const double *grid, int nx, int ny, int nz, int kind,
                                         double *out) {
    const int64_t ntot = (int64_t)nx * ny * nz;
    if (ntot > VT_NOALLOC_TENSOR_POINTS) return hipErrorInvalidValue;
    cd *F = nullptr;
    hipError_t e = scratch_address(&F);
    if (e != hipSuccess) return e;
    return grid_tensor_into(c, grid, nx, ny, nz, kind, out, F);
}

void vt_spec_free(vt_ctx *c) {
    (void)hipFree(c->spec_buf);
    c->spec_buf = nullptr;
    c->cap_spec = 0;
}
