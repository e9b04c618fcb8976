// Small planes: the x and y transforms of one z plane in one kernel, and the
// z-systems solved in one pass over the spectra.
//
// A plane of nx x ny values that fits in LDS (128 x 128 in double, about 181 x
// 181 in float) needs no trip to memory between its x and y transforms, and
// once the y transforms are done the z-systems of the (slot, entry) columns are
// independent of one another.  So such grids take three kernels, each one pass
// over the data (6 real values moved per point against 8 of the x kernels and
// the z march), none of them bound to one workgroup per spectral slot:
//   k_plane_fwd  f -> x and y transforms of a plane -> S,
//   k_zscan      z-systems, a few columns by all of z per workgroup,
//   k_plane_inv  S -> inverse y and x transforms of a plane -> u.
// The transforms are those of the x kernels and the z march (same packing of
// two real rows in one complex line, same pre- and post-processing, same
// spectral layout S[b][z][slot][y] and tables); only the work is split
// differently: a workgroup transforms all lines of its plane at once (a line of
// 64 by itself keeps 8 of a wavefront's lanes busy in a radix-8 stage).

#include <type_traits>

#include "pp_kernels.hpp"

namespace pp {

// Index arithmetic of these kernels: products below 2^24 (24-bit multiplies run
// at full rate, 32-bit ones at a quarter).
__device__ __forceinline__ int mul24(int a, int b) { return (int)__umul24((unsigned)a, (unsigned)b); }
// fdiv with the half folded into the multiply-add: floor(i / n), inv = 1.0f / n.
__device__ __forceinline__ int qdiv(int i, float inv) { return (int)fmaf((float)i, inv, 0.5f * inv); }

// One Stockham stage (see wfft_stage) of all `nl` lines of a plane by the whole
// workgroup.  Consecutive lanes take the same butterfly of consecutive lines,
// whose stride is odd: no bank conflicts at any stage without padding inside
// the lines, so the elements of a butterfly are at one address plus multiples
// of a stride, and the lanes share their twiddles.  (One wavefront per group
// of padded lines, no barriers between stages, spent most of its instructions
// on LDS addresses: 101 x 96 x 144 in double, forward 28 us.)
template <int R, int MAXB, int NTH, bool INV, typename T>
__device__ __forceinline__ void plane_stage(cplx<T>* buf, int ld, int nl, float inv_nl, int N, int Ls,
                                            const cplx<T>* tw, int tid) {
    const int nbf = N / R, total = nl * nbf;
    const float inv_ls = 1.0f / (float)Ls;
    cplx<T> v[MAXB][R];
    int dst[MAXB];
#pragma unroll
    for (int i = 0; i < MAXB; ++i) {
        const int q = tid + NTH * i;
        dst[i] = -1;
        if (q < total) {
            const int j = qdiv(q, inv_nl), l = q - mul24(j, nl);
            const int row = mul24(l, ld);
#pragma unroll
            for (int t = 0; t < R; ++t) v[i][t] = buf[row + j + t * nbf];
            int k = 0;
            if (Ls > 1) {
                k = j - mul24(qdiv(j, inv_ls), Ls);
#pragma unroll
                for (int t = 1; t < R; ++t) {
                    const cplx<T> w = tw[k + (t * Ls - 1)];
                    v[i][t] = INV ? cmulc(v[i][t], w) : cmul(v[i][t], w);
                }
            }
            rbfly<R, INV, T>(v[i]);
            dst[i] = row + (j - k) * R + k;
        }
    }
    lds_barrier();
#pragma unroll
    for (int i = 0; i < MAXB; ++i) {
        if (dst[i] >= 0) {
#pragma unroll
            for (int t = 0; t < R; ++t) buf[dst[i] + t * Ls] = v[i][t];
        }
    }
    lds_barrier();
}

// Transform nl lines of d.n values, ld apart (nl d.n <= EPT NTH).  Radices up
// to 16 (plane_radices()): a stage costs a pass through LDS and two barriers.
template <int EPT, int NTH, bool INV, typename T, bool BIG = (NTH > kPlaneSmallThreads)>
__device__ __forceinline__ void plane_fft(cplx<T>* buf, int ld, int nl, const FftDesc& d, const cplx<T>* tw) {
    const float inv_nl = 1.0f / (float)nl;
    int Ls = 1, tid = threadIdx.x;
    for (int s = 0; s < d.nstages; ++s) {
        const int R = d.radix[s];
        // (opaque, so that the addresses of all four radices are not kept in
        // registers across the stages)
        asm volatile("" : "+v"(tid));
        // (small planes, 256 threads, are launch-bound: more code than radix 8
        // costs them more than the stages it saves, 32^3 forward 7.6 -> 8.8 us)
        if (BIG && R == 16) plane_stage<16, cdiv(EPT, 16), NTH, INV, T>(buf, ld, nl, inv_nl, d.n, Ls, tw, tid);
        else if (BIG && R == 12) plane_stage<12, cdiv(EPT, 12), NTH, INV, T>(buf, ld, nl, inv_nl, d.n, Ls, tw, tid);
        else if (BIG && R == 9) plane_stage<9, cdiv(EPT, 9), NTH, INV, T>(buf, ld, nl, inv_nl, d.n, Ls, tw, tid);
        else if (BIG && R == 6) plane_stage<6, cdiv(EPT, 6), NTH, INV, T>(buf, ld, nl, inv_nl, d.n, Ls, tw, tid);
        else if (R == 8) plane_stage<8, cdiv(EPT, 8), NTH, INV, T>(buf, ld, nl, inv_nl, d.n, Ls, tw, tid);
        else if (R == 4) plane_stage<4, cdiv(EPT, 4), NTH, INV, T>(buf, ld, nl, inv_nl, d.n, Ls, tw, tid);
        else if (R == 3) plane_stage<3, cdiv(EPT, 3), NTH, INV, T>(buf, ld, nl, inv_nl, d.n, Ls, tw, tid);
        else plane_stage<2, cdiv(EPT, 2), NTH, INV, T>(buf, ld, nl, inv_nl, d.n, Ls, tw, tid);
        Ls *= R;
    }
}

// Complex values of a plane one thread holds while the plane is transposed
// (32 registers' worth of double or float pairs per direction).
template <typename T> constexpr int kPlaneVals = sizeof(T) == 8 ? 8 : 16;
constexpr int kPlaneMaxThreads = 1024;

// LDS of a plane kernel: the packed lines (rows in pairs, or slots; the larger),
// then the twiddles of x and y and, where those transforms need them, the DCT twiddles.
template <typename T> struct PlaneLds {
    cplx<T>*buf, *twx, *mkx, *twy, *mky;
};
template <typename T> __device__ __forceinline__ PlaneLds<T> plane_lds(unsigned char* smem, const PlaneArgs<T>& a) {
    PlaneLds<T> l;
    l.buf = reinterpret_cast<cplx<T>*>(smem);
    l.twx = l.buf + a.bufn;
    l.twy = l.twx + a.nx;
    l.mkx = l.twy + a.ny;
    l.mky = l.mkx + (a.bx != BC_P ? a.nx : 0);
    return l;
}
template <typename T, int NTH>
__device__ __forceinline__ void plane_tables(const PlaneLds<T>& l, const PlaneArgs<T>& a) {
    for (int i = threadIdx.x; i < a.nx; i += NTH) {
        l.twx[i] = a.twx[i];
        if (a.bx != BC_P) l.mkx[i] = a.mkx[i];
    }
    for (int i = threadIdx.x; i < a.ny; i += NTH) {
        l.twy[i] = a.twy[i];
        if (a.by != BC_P) l.mky[i] = a.mky[i];
    }
}

// DCT-II bin k of a packed line (see the x kernels): 1/2 (e^{-i pi k/2N} V_k + e^{+i pi k/2N} V_{N-k}).
template <typename T>
__device__ __forceinline__ cplx<T> plane_dct_bin(const cplx<T>* line, const cplx<T>* mk_, int k, int N) {
    const cplx<T> vk = line[k];
    const cplx<T> vr = line[k == 0 ? 0 : N - k];
    const cplx<T> w = mk_[k];
    return cscale(cadd(cmul(w, vk), cmulc(vr, w)), T(0.5));
}

// Entry e of a transformed y line: its DCT bin, or its DFT bin; with `pair`, two
// real x spectra share the line: A_k -> entry k, B_k -> entry N-k (k < N/2).
template <typename T>
__device__ __forceinline__ cplx<T> plane_bin(const cplx<T>* line, int e, int N, bool dct, bool pair,
                                             const cplx<T>* mk_) {
    if (dct) return plane_dct_bin<T>(line, mk_, e, N);
    const cplx<T> v = line[e];
    if (!pair || e == 0 || 2 * e == N) return v;
    const cplx<T> w = line[N - e];
    return 2 * e < N ? mk<T>(T(0.5) * (v.x + w.x), T(0.5) * (v.y - w.y))
                     : mk<T>(T(0.5) * (w.y + v.y), T(0.5) * (v.x - w.x));
}

template <int NW> __device__ __forceinline__ void plane_partial(double acc, double* red, double* out) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) acc += __shfl_down(acc, off, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
    lds_barrier();
    if (threadIdx.x == 0) {
        double s = 0.0;
        for (int w = 0; w < NW; ++w) s += red[w];
        *out = s;
    }
}

// Forward: one workgroup per plane (blockIdx.x = z, blockIdx.y = batch entry).
// The sum of its source values goes to partial[b nz + z].
template <typename T, int NTH, bool FACES>
__global__ __launch_bounds__(NTH) void k_plane_fwd(const T* __restrict__ f, cplx<T>* __restrict__ S,
                                                   double* __restrict__ partial, PlaneArgs<T> a, FaceArgs<T> fa) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ double red[NTH / 64];
    constexpr int V = kPlaneVals<T>, NW = NTH / 64;
    const PlaneLds<T> L = plane_lds<T>(smem, a);
    const int nx = a.nx, ny = a.ny, nyp = (ny + 1) >> 1;
    const int z = blockIdx.x, b = blockIdx.y, tid = threadIdx.x;
    const T* src = f + ((size_t)b * a.nz + z) * (size_t)ny * nx;
    const float inv_nx = 1.0f / (float)nx, inv_slots = 1.0f / (float)a.slots, inv_ny = 1.0f / (float)ny;

    // 1. rows -> packed lines (row 2j real part, row 2j+1 imaginary part), reordered for the x transform
    T ra[V], rb[V];
    const int nin = nyp * nx;
#pragma unroll
    for (int k = 0; k < V; ++k) {
        const int i = tid + k * NTH;
        ra[k] = T(0);
        rb[k] = T(0);
        if (i < nin) {
            // row 2j, column n: element 2 j nx + n = i + j nx
            const int j = qdiv(i, inv_nx), at = i + mul24(j, nx);
            ra[k] = ld_stream(src + at);
            if (2 * j + 1 < ny) rb[k] = ld_stream(src + at + nx);
        }
    }
    plane_tables<T, NTH>(L, a);
    double acc = 0.0;
#pragma unroll
    for (int k = 0; k < V; ++k) {
        const int i = tid + k * NTH;
        if (i < nin) {
            const int j = qdiv(i, inv_nx), n = i - mul24(j, nx);
            double fa_ = (double)ra[k], fb_ = (double)rb[k];
            if constexpr (FACES) {
                fa_ -= face_lift(fa, b, n, 2 * j, z, nx, ny, a.nz);
                if (2 * j + 1 < ny) fb_ -= face_lift(fa, b, n, 2 * j + 1, z, nx, ny, a.nz);
            }
            acc += fa_ + fb_;
            T va = (T)fa_, vb = (T)fb_;
            int pos = n;
            if (a.bx != BC_P) {
                pos = makhoul_pos(n, nx);
                if (a.bx == BC_D && (n & 1)) {
                    va = -va;
                    vb = -vb;
                }
            }
            L.buf[mul24(j, a.ldx) + pos] = mk<T>(va, vb);
        }
    }
    plane_partial<NW>(acc, red, partial + (size_t)b * a.nz + z);   // (barrier: lines and tables in)

    // 2. x transforms
    plane_fft<V, NTH, false, T>(L.buf, a.ldx, nyp, a.fx, L.twx);

    // 3. post-processed spectra of row pairs, transposed into lines of y (one per slot) through registers
    constexpr int VP = (V + 1) / 2;
    cplx<T> oa[VP], ob[VP];
    const int nit = a.slots * nyp;
#pragma unroll
    for (int k = 0; k < VP; ++k) {
        const int i = tid + k * NTH;
        oa[k] = mk<T>(T(0), T(0));
        ob[k] = oa[k];
        if (i < nit) {
            const int j = qdiv(i, inv_slots), m = i - mul24(j, a.slots);
            const cplx<T>* line = L.buf + mul24(j, a.ldx);
            if (a.bx == BC_P) {
                if (m == 0) {
                    const cplx<T> z0 = line[0];
                    cplx<T> zn = mk<T>(T(0), T(0));
                    if (!(nx & 1)) zn = line[nx >> 1];
                    oa[k] = mk<T>(z0.x, zn.x);
                    ob[k] = mk<T>(z0.y, zn.y);
                } else {
                    const cplx<T> zk = line[m], zr = line[nx - m];
                    oa[k] = mk<T>(T(0.5) * (zk.x + zr.x), T(0.5) * (zk.y - zr.y));
                    ob[k] = mk<T>(T(0.5) * (zk.y + zr.y), T(0.5) * (zr.x - zk.x));
                }
            } else {
                const cplx<T> c0 = plane_dct_bin<T>(line, L.mkx, 2 * m, nx);
                const cplx<T> c1 = (2 * m + 1 < nx) ? plane_dct_bin<T>(line, L.mkx, 2 * m + 1, nx) : mk<T>(T(0), T(0));
                oa[k] = mk<T>(c0.x, c1.x);
                ob[k] = mk<T>(c0.y, c1.y);
            }
        }
    }
    lds_barrier();
#pragma unroll
    for (int k = 0; k < VP; ++k) {
        const int i = tid + k * NTH;
        if (i < nit) {
            const int j = qdiv(i, inv_slots), m = i - mul24(j, a.slots);
            cplx<T>* line = L.buf + mul24(m, a.ldy);
            int pa = 2 * j, pb = 2 * j + 1;
            cplx<T> vb = ob[k];
            if (a.by != BC_P) {
                pa = makhoul_pos(pa, ny);
                pb = makhoul_pos(pb, ny);
                if (a.by == BC_D) vb = mk<T>(-vb.x, -vb.y);
            }
            line[pa] = oa[k];
            if (2 * j + 1 < ny) line[pb] = vb;
        }
    }
    lds_barrier();

    // 4. y transforms
    plane_fft<V, NTH, false, T>(L.buf, a.ldy, a.slots, a.fy, L.twy);

    // 5. post-processed columns of the plane
    cplx<T>* dst = S + ((size_t)b * a.nz + z) * (size_t)a.slots * ny;
    for (int i = tid; i < a.slots * ny; i += NTH) {
        const int m = qdiv(i, inv_ny), e = i - mul24(m, ny);
        const cplx<T>* line = L.buf + mul24(m, a.ldy);
        dst[i] = plane_bin<T>(line, e, ny, a.by != BC_P, a.by == BC_P && (a.bx != BC_P || m == 0), L.mky);
    }
}

// Pre-processing of one pair (k, N-k), k > 0, of a line for the inverse transform.
template <typename T>
__device__ __forceinline__ void plane_pre_pair(cplx<T>* line, int k, int N, bool dct, const cplx<T>* mk_) {
    if (2 * k > N) return;
    const cplx<T> a = line[k];
    if (2 * k == N) {
        if (dct) line[k] = cmulc(mk<T>(a.x + a.y, a.y - a.x), mk_[k]);
        return;
    }
    const cplx<T> b = line[N - k];
    if (dct) {
        line[k] = cmulc(mk<T>(a.x + b.y, a.y - b.x), mk_[k]);
        line[N - k] = cmulc(mk<T>(b.x + a.y, b.y - a.x), mk_[N - k]);
    } else {
        line[k] = mk<T>(a.x - b.y, a.y + b.x);
        line[N - k] = mk<T>(a.x + b.y, b.x - a.y);
    }
}

// Pre-processing of the inverse transforms of nl lines of N values, in place
// over the pairs (k, N-k): `dct`, W_k = e^{+i pi k/2N} (X_k - i X_{N-k}); otherwise
// the two real spectra of a line packed again, A + i B and conj(A) + i conj(B).
template <int NTH, typename T>
__device__ __forceinline__ void plane_pre(cplx<T>* buf, int ld, int nl, int N, bool dct, const cplx<T>* mk_) {
    const int hn = (N >> 1) + 1;
    const float inv_hn = 1.0f / (float)hn;
    for (int q = threadIdx.x; q < nl * hn; q += NTH) {
        const int l = qdiv(q, inv_hn), k = q - mul24(l, hn);
        cplx<T>* line = buf + mul24(l, ld);
        if (k != 0) plane_pre_pair<T>(line, k, N, dct, mk_);
    }
    lds_barrier();
}

// Inverse: one workgroup per plane.
template <typename T, int NTH>
__global__ __launch_bounds__(NTH) void k_plane_inv(const cplx<T>* __restrict__ S, T* __restrict__ u, PlaneArgs<T> a,
                                                   const double* __restrict__ shift) {
    extern __shared__ __align__(16) unsigned char smem[];
    constexpr int V = kPlaneVals<T>;
    const PlaneLds<T> L = plane_lds<T>(smem, a);
    const int nx = a.nx, ny = a.ny, nyp = (ny + 1) >> 1;
    const int z = blockIdx.x, b = blockIdx.y, tid = threadIdx.x;
    const cplx<T>* src = S + ((size_t)b * a.nz + z) * (size_t)a.slots * ny;
    const float inv_nx = 1.0f / (float)nx, inv_slots = 1.0f / (float)a.slots;
    const float inv_ny = 1.0f / (float)ny;

    // 1. columns -> lines of y
    cplx<T> v[V];
    const int nin = a.slots * ny;
#pragma unroll
    for (int k = 0; k < V; ++k) {
        const int i = tid + k * NTH;
        v[k] = i < nin ? src[i] : mk<T>(T(0), T(0));
    }
    plane_tables<T, NTH>(L, a);
    const double sh = shift[b];
#pragma unroll
    for (int k = 0; k < V; ++k) {
        const int i = tid + k * NTH;
        if (i < nin) {
            const int m = qdiv(i, inv_ny), e = i - mul24(m, ny);
            L.buf[mul24(m, a.ldy) + e] = v[k];
        }
    }
    lds_barrier();

    // 2. pre-processing (pairs k, ny-k) and inverse transforms along y
    if (a.by != BC_P || a.bx != BC_P) plane_pre<NTH, T>(L.buf, a.ldy, a.slots, ny, a.by != BC_P, L.mky);
    else plane_pre<NTH, T>(L.buf, a.ldy, 1, ny, false, L.mky);
    plane_fft<V, NTH, true, T>(L.buf, a.ldy, a.slots, a.fy, L.twy);

    // 3. row pairs of every slot -> packed lines of x, through registers
    constexpr int VP = (V + 1) / 2;
    cplx<T> sa[VP], sb[VP];
    const int nit = a.slots * nyp;
#pragma unroll
    for (int k = 0; k < VP; ++k) {
        const int i = tid + k * NTH;
        sa[k] = mk<T>(T(0), T(0));
        sb[k] = sa[k];
        if (i < nit) {
            const int j = qdiv(i, inv_slots), m = i - mul24(j, a.slots);
            const cplx<T>* line = L.buf + mul24(m, a.ldy);
            int pa = 2 * j, pb = 2 * j + 1;
            const bool two = pb < ny;
            if (a.by != BC_P) {
                pa = makhoul_pos(pa, ny);
                pb = makhoul_pos(pb, ny);
            }
            sa[k] = line[pa];
            if (two) {
                sb[k] = line[pb];
                if (a.by == BC_D) sb[k] = mk<T>(-sb[k].x, -sb[k].y);
            }
        }
    }
    lds_barrier();
#pragma unroll
    for (int k = 0; k < VP; ++k) {
        const int i = tid + k * NTH;
        if (i < nit) {
            const int j = qdiv(i, inv_slots), m = i - mul24(j, a.slots);
            cplx<T>* line = L.buf + mul24(j, a.ldx);
            const cplx<T> va = sa[k], vb = sb[k];
            if (a.bx == BC_P) {
                if (m == 0) {
                    line[0] = mk<T>(va.x, vb.x);
                    if (!(nx & 1)) line[nx >> 1] = mk<T>(va.y, vb.y);
                } else {
                    line[m] = mk<T>(va.x - vb.y, va.y + vb.x);        // X_a + i X_b
                    line[nx - m] = mk<T>(va.x + vb.y, vb.x - va.y);   // conj(X_a) + i conj(X_b)
                }
            } else {
                line[2 * m] = mk<T>(va.x, vb.x);
                if (2 * m + 1 < nx) line[2 * m + 1] = mk<T>(va.y, vb.y);
            }
        }
    }
    lds_barrier();

    // 4. inverse transforms along x
    if (a.bx != BC_P) plane_pre<NTH, T>(L.buf, a.ldx, nyp, nx, true, L.mkx);
    plane_fft<V, NTH, true, T>(L.buf, a.ldx, nyp, a.fx, L.twx);

    // 5. rows
    T* dst = u + ((size_t)b * a.nz + z) * (size_t)ny * nx;
    for (int i = tid; i < nyp * nx; i += NTH) {
        const int j = qdiv(i, inv_nx), n = i - mul24(j, nx);
        int pos = n;
        if (a.bx != BC_P) pos = makhoul_pos(n, nx);
        cplx<T> c = L.buf[mul24(j, a.ldx) + pos];
        if (a.bx == BC_D && (n & 1)) c = mk<T>(-c.x, -c.y);
        const int at = i + mul24(j, nx);
        st_stream(dst + at, (T)((double)c.x - sh));
        if (2 * j + 1 < ny) st_stream(dst + at + nx, (T)((double)c.y - sh));
    }
}

// ---------------------------------------------------------------------------
// The y transforms of spectral lines by themselves, in place (grids whose planes
// do not fit in LDS and whose columns are too few for the z march): a workgroup
// takes a group of whole lines (b, z, slot), kPlaneVals values per thread.
// ---------------------------------------------------------------------------
template <typename T, int NTH, bool INV>
__global__ __launch_bounds__(NTH) void k_ylines(cplx<T>* __restrict__ S, LineArgs<T> a) {
    extern __shared__ __align__(16) unsigned char smem[];
    constexpr int V = kPlaneVals<T>;
    const int ny = a.ny, ld = a.ld, tid = threadIdx.x;
    const size_t first = (size_t)blockIdx.x * a.group;
    const int nl = (int)(a.nlines - first < (size_t)a.group ? a.nlines - first : (size_t)a.group);
    cplx<T>* buf = reinterpret_cast<cplx<T>*>(smem);
    cplx<T>* tw = buf + a.group * ld;
    cplx<T>* mk_ = tw + ny;
    cplx<T>* col = S + first * ny;
    const float inv_ny = 1.0f / (float)ny;
    const int n = nl * ny;
    cplx<T> v[V];
#pragma unroll
    for (int k = 0; k < V; ++k) {
        const int i = tid + k * NTH;
        v[k] = i < n ? col[i] : mk<T>(T(0), T(0));
    }
    for (int i = tid; i < ny; i += NTH) {
        tw[i] = a.twy[i];
        if (a.by != BC_P) mk_[i] = a.mky[i];
    }
    // the slot of a line decides whether its two parts are separate real spectra
    const float inv_slots = 1.0f / (float)a.slots;
    const int slot0 = (int)(first % (size_t)a.slots);
    auto paired = [&](int l) {
        if (a.bx != BC_P) return true;
        const int q = slot0 + l;
        return q - mul24(qdiv(q, inv_slots), a.slots) == 0;
    };
#pragma unroll
    for (int k = 0; k < V; ++k) {
        const int i = tid + k * NTH;
        if (i < n) {
            const int l = qdiv(i, inv_ny), y = i - mul24(l, ny);
            int pos = y;
            cplx<T> x = v[k];
            if (!INV && a.by != BC_P) {
                pos = makhoul_pos(y, ny);
                if (a.by == BC_D && (y & 1)) x = mk<T>(-x.x, -x.y);
            }
            buf[mul24(l, ld) + pos] = x;
        }
    }
    lds_barrier();
    if constexpr (INV) {
        // pairs (k, ny-k) of every line; periodic y: only of lines that hold two real spectra
        const int hn = (ny >> 1) + 1;
        const float inv_hn = 1.0f / (float)hn;
        for (int q = tid; q < nl * hn; q += NTH) {
            const int l = qdiv(q, inv_hn), k = q - mul24(l, hn);
            if (k == 0 || (a.by == BC_P && !paired(l))) continue;
            plane_pre_pair<T>(buf + mul24(l, ld), k, ny, a.by != BC_P, mk_);
        }
        lds_barrier();
    }
    plane_fft<V, NTH, INV, T, true>(buf, ld, nl, a.fy, tw);
    for (int i = tid; i < n; i += NTH) {
        const int l = qdiv(i, inv_ny), y = i - mul24(l, ny);
        const cplx<T>* line = buf + mul24(l, ld);
        cplx<T> x;
        if constexpr (INV) {
            x = line[a.by != BC_P ? makhoul_pos(y, ny) : y];
            if (a.by == BC_D && (y & 1)) x = mk<T>(-x.x, -x.y);
        } else {
            x = plane_bin<T>(line, y, ny, a.by != BC_P, a.by == BC_P && paired(l), mk_);
        }
        col[i] = x;
    }
}

// ---------------------------------------------------------------------------
// z-systems in one pass.  Both sweeps of the Thomas algorithm are first-order
// recurrences with tabulated factors,
//     y_z = (d_z - y_{z-1}) w_z,      u_z = y_z - w_z u_{z+1},
// so a stretch of rows maps its incoming value c to its outgoing one as B + A c,
// A = prod(-w_z) and B its result from c = 0.  A workgroup owns `ct` adjacent
// columns (128 bytes of every plane: whole lines) and all of z (or chunks of
// P L rows): thread (column, segment) keeps L rows and their pivots in
// registers, runs the recurrence from zero, and adds the incoming value's part
// once the P segments' (A, B) have been chained.  The pivots are those of the whole column, so the
// rounding is that of one march (|A| <= 1; no reduced system, nothing divided).
// Periodic z: as in the z march, the value y_0 = sum alpha_z d_z and the last
// y give the Sherman-Morrison factor before the sweep back, which then starts
// from y - c qp.
// ---------------------------------------------------------------------------
//
// Float spectra whose march would be split (Ts float, T double): one recurrence
// over the whole column in float carries its rounding, and that of the float
// pivots, which is the same in every row past their table, further than the
// pieces of a split or segmented march do.  There the pivots are in two floats
// (MidArgs::wrowsl) and the recurrences in double, which leaves the rounding of
// the spectra themselves (rms error from the f64 solve of one float recurrence,
// of the split march and of this: 1000 x 128 x 64 DDDDDN x 16 1.2e-6, 5.3e-7 and
// 2.1e-7; 2048 x 32 x 128 x 6 2.0e-6, 8.1e-7 and 1.9e-7; 64 x 64 x 64 x 16 gradient
// 104 us either way).
template <typename Ts, typename T, int L, bool PERZ, bool ONE>
__global__ __launch_bounds__(kScanThreads) void k_zscan(cplx<Ts>* __restrict__ S, MidArgs<Ts> a, ScanArgs g) {
    constexpr bool LOW = !std::is_same_v<Ts, T>;
    static_assert(!(LOW && PERZ), "periodic z is never split");
    extern __shared__ __align__(16) unsigned char smem[];
    const int ct = 1 << g.lct, P = g.segs, ny = a.ny, nz = a.nz;
    cplx<T>* sA = reinterpret_cast<cplx<T>*>(smem);   // a value per (wavefront, column) each
    cplx<T>* sB = sA + (blockDim.x >> 6) * ct;
    double* red = reinterpret_cast<double*>(sB + (blockDim.x >> 6) * ct);   // one per wavefront
    const int tid = threadIdx.x, nth = blockDim.x;
    const int b = blockIdx.y, tile = blockIdx.x;
    const int cl = tid & (ct - 1), seg = tid >> g.lct;
    const int c = tile * ct + cl;
    const bool on = seg < P && c < a.slots * ny;
    const int cc = on ? c : 0;
    const int m = cc / ny, e = cc - m * ny;
    cplx<Ts>* col = S + (size_t)b * a.slots * nz * ny + (size_t)m * a.sstride + e;
    const size_t zs = (size_t)a.zstride;
    const bool sing = a.singular && c == 0;
    const cplx<T> zero = mk<T>(T(0), T(0));

    // rows of this thread's segment in the chunk at z0 (past the end: the last
    // row), issued before anything else is waited for
    cplx<T> y[L], w[L];
    auto rows = [&](int z0) __attribute__((always_inline)) {
        const int zb = z0 + seg * L;
#pragma unroll
        for (int r = 0; r < L; ++r) y[r] = cvt<T>(col[(size_t)(zb + r < nz ? zb + r : nz - 1) * zs]);
    };
    rows(0);
    cplx<T> winf = zero, wlast = zero;
    int elen = 0, roff = 0;
    if (on) {
        winf = cvt<T>(a.winf[(size_t)m * ny + e]);
        wlast = cvt<T>(a.wlast[(size_t)m * ny + e]);
        if constexpr (LOW) {
            winf = cadd(winf, cvt<T>(a.winfl[(size_t)m * ny + e]));
            wlast = cadd(wlast, cvt<T>(a.wlastl[(size_t)m * ny + e]));
        }
        elen = a.elen[(size_t)m * ny + e];
        roff = a.rowoff[m];
    }
    int alen = 0, qlen = 0, aoff = 0, qoff = 0;   // periodic z: this column's rows of alpha and qp
    cplx<T> qlast = zero, ig = zero, id = zero;
    if constexpr (PERZ) {
        if (on) {
            alen = a.aelen[(size_t)m * ny + e];
            qlen = a.qelen[(size_t)m * ny + e];
            aoff = a.aoff[m];
            qoff = a.qoff[m];
            qlast = cvt<T>(a.qlast[(size_t)m * ny + e]);
            ig = cvt<T>(a.inv_gamma[(size_t)m * ny + e]);
            id = cvt<T>(a.inv_den[(size_t)m * ny + e]);
        }
    }

    // the planes' sums of the source (k_plane_fwd), by the first column's
    // workgroup; a source with an Inf or NaN gives a mean that is not finite
    T proj = T(0);
    if (!g.partial) {
        if (sing && a.project) proj = (T)(a.hz2 * a.mu[b]);
    } else if (tile == 0) {
        double s = 0.0;
        for (int i = tid; i < nz; i += nth) s += g.partial[(size_t)b * nz + i];
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) s += __shfl_down(s, off, 64);
        if ((tid & 63) == 0) red[tid >> 6] = s;
        lds_barrier();
        s = 0.0;
        for (int w = 0; w < nth / 64; ++w) s += red[w];
        const double mu = s / g.npts;
        if (tid == 0) {
            g.mu[b] = mu;
            if (b == 0) *g.maxf = fabs(mu);
        }
        if (sing && a.project) proj = (T)(a.hz2 * mu);
        lds_barrier();
    }

    // Eight rows from zb of a table that holds `len` of them from row `off` (`low`:
    // their low parts, or null); past them the value `past`.  One branch for the eight (skipped by a wavefront
    // whose columns have none left): a branch per row waits for each load by
    // itself (200 x 192 x 256 f32 periodic: 45 -> 31 us).
    constexpr int H = 8;
    static_assert(L % H == 0, "rows in groups of eight");
    auto table = [&](const cplx<Ts>* rows_, const cplx<Ts>* low, int off, int len, int zb, cplx<T> past,
                     cplx<T>* t) __attribute__((always_inline)) {
#pragma unroll
        for (int r = 0; r < H; ++r) t[r] = past;
        if (__builtin_amdgcn_ballot_w64(zb < len)) {
            cplx<T> q[H];
#pragma unroll
            for (int r = 0; r < H; ++r) {
                const size_t at = zb + r < len ? (size_t)(off + zb + r) * ny + e : 0;
                q[r] = cvt<T>(rows_[at]);
                if constexpr (LOW) q[r] = cadd(q[r], cvt<T>(low[at]));
            }
#pragma unroll
            for (int r = 0; r < H; ++r) {
                const bool tab = zb + r < len;
                t[r] = mk<T>(tab ? q[r].x : past.x, tab ? q[r].y : past.y);
            }
        }
    };
    // pivots of the thread's rows in the chunk at z0, and rows past the end made inert
    auto pivots = [&](int z0) __attribute__((always_inline)) {
        const int zb = z0 + seg * L;
#pragma unroll
        for (int h = 0; h < L; h += H) table(a.wrows, a.wrowsl, roff, elen, zb + h, winf, w + h);
#pragma unroll
        for (int r = 0; r < L; ++r) {
            const int z = zb + r;
            const bool last = z == nz - 1, in = on && z < nz;
            w[r] = mk<T>(in ? (last ? wlast.x : w[r].x) : T(0), in ? (last ? wlast.y : w[r].y) : T(0));
        }
#pragma unroll
        for (int r = 0; r < L; ++r) {
            const bool in = on && zb + r < nz;
            y[r] = mk<T>(in ? y[r].x : T(0), in ? y[r].y : T(0));
        }
    };
    // Chain the segments' maps from `carry`, the value entering the chunk (at
    // its first row for DIR 1, past its last for DIR -1): returns the value
    // entering this thread's segment and leaves in `carry` the one that leaves
    // the chunk.  Scan over the segments of a wavefront by lane shifts, then
    // over the wavefronts' totals from LDS.  (A serial chain over LDS by one
    // thread per column part took 2.3 us for 64 segments, twice per solve.)
    const int wave = tid >> 6, nw = nth >> 6;
    cplx<T> carry = zero;
    auto chain = [&](auto dirc, cplx<T> A, cplx<T> B) __attribute__((always_inline)) -> cplx<T> {
        constexpr int DIR = decltype(dirc)::value;
        const int lane = tid & 63, ls = DIR > 0 ? lane >> g.lct : (63 - lane) >> g.lct;   // place in the wavefront's chain
        auto shift = [&](T v, int d) { return DIR > 0 ? __shfl_up(v, d, 64) : __shfl_down(v, d, 64); };
        for (int d = 1; d < (64 >> g.lct); d <<= 1) {
            const int dl = d << g.lct;
            const cplx<T> pA = mk<T>(shift(A.x, dl), shift(A.y, dl)), pB = mk<T>(shift(B.x, dl), shift(B.y, dl));
            if (ls >= d) {
                B = mk<T>(B.x + A.x * pB.x, B.y + A.y * pB.y);
                A = mk<T>(A.x * pA.x, A.y * pA.y);
            }
        }
        // exclusive within the wavefront
        cplx<T> eA = mk<T>(shift(A.x, ct), shift(A.y, ct)), eB = mk<T>(shift(B.x, ct), shift(B.y, ct));
        if (ls == 0) {
            eA = mk<T>(T(1), T(1));
            eB = zero;
        }
        if (DIR > 0 ? lane >= 64 - ct : lane < ct) {
            sA[wave * ct + cl] = A;
            sB[wave * ct + cl] = B;
        }
        lds_barrier();
        cplx<T> c = carry, in = carry;
        for (int q = 0; q < nw; ++q) {
            const int wq = DIR > 0 ? q : nw - 1 - q;
            if (wq == wave) in = c;
            const cplx<T> tA = sA[wq * ct + cl], tB = sB[wq * ct + cl];
            c = mk<T>(tB.x + tA.x * c.x, tB.y + tA.y * c.y);
        }
        carry = c;
        lds_barrier();   // the totals are read before they are written again
        return mk<T>(eB.x + eA.x * in.x, eB.y + eA.y * in.y);
    };
    cplx<T> y0 = zero;   // periodic z: this segment's share of sum alpha_z d_z
    cplx<T> corr = zero;
    double csum = 0.0;
    const int nch = ONE ? 1 : g.chunks;
    for (int ch = 0; ch < nch; ++ch) {
        const int z0 = ch * P * L;
        if (ch > 0) rows(z0);
        pivots(z0);
#pragma unroll
        for (int r = 0; r < L; ++r) {
            y[r] = cscale(y[r], (T)a.scale);
            if (sing && z0 + seg * L + r < nz) y[r].x -= proj;
        }
        if constexpr (PERZ) {
#pragma unroll
            for (int h = 0; h < L; h += H) {
                cplx<T> al[H];
                table(a.arows, nullptr, aoff, alen, z0 + seg * L + h, zero, al);
#pragma unroll
                for (int r = 0; r < H; ++r) {
                    y0.x += al[r].x * y[h + r].x;
                    y0.y += al[r].y * y[h + r].y;
                }
            }
        }
        cplx<T> A = mk<T>(T(1), T(1)), prev = zero;
#pragma unroll
        for (int r = 0; r < L; ++r) {
            prev = mk<T>((y[r].x - prev.x) * w[r].x, (y[r].y - prev.y) * w[r].y);
            y[r] = prev;
            A = mk<T>(-w[r].x * A.x, -w[r].y * A.y);
        }
        cplx<T> p = chain(std::integral_constant<int, 1>{}, A, prev);
#pragma unroll
        for (int r = 0; r < L; ++r) {
            p = mk<T>(-w[r].x * p.x, -w[r].y * p.y);
            y[r] = cadd(y[r], p);
        }
        if constexpr (!ONE) {
#pragma unroll
            for (int r = 0; r < L; ++r) {
                const int z = z0 + seg * L + r;
                if (on && z < nz) col[(size_t)z * zs] = cvt<Ts>(y[r]);
            }
        }
    }
    if constexpr (PERZ) {
        // y_0 over the segments, y_{n-1} from its owner, then the factor
#pragma unroll
        for (int d = 32; d > 0; d >>= 1) {
            if (d >= ct) {
                y0.x += __shfl_xor(y0.x, d, 64);
                y0.y += __shfl_xor(y0.y, d, 64);
            }
        }
        if ((tid & 63) < ct) sB[wave * ct + cl] = y0;
        const int zl = (nz - 1) - (nch - 1) * P * L;
#pragma unroll
        for (int r = 0; r < L; ++r)
            if (seg < P && seg * L + r == zl) sA[cl] = y[r];
        lds_barrier();
        cplx<T> s = zero;
        for (int q = 0; q < nw; ++q) s = cadd(s, sB[q * ct + cl]);
        if (on) {
            const cplx<T> yl = sA[cl];
            corr = mk<T>((s.x + yl.x * ig.x) * id.x, (s.y + yl.y * ig.y) * id.y);
        }
        lds_barrier();
    }
    carry = zero;
    for (int ch = nch - 1; ch >= 0; --ch) {
        const int z0 = ch * P * L;
        if constexpr (!ONE) {
            rows(z0);
            pivots(z0);
        }
        if constexpr (PERZ) {
#pragma unroll
            for (int h = 0; h < L; h += H) {
                cplx<T> q[H];
                table(a.qrows, nullptr, qoff, qlen, z0 + seg * L + h, zero, q);
#pragma unroll
                for (int r = 0; r < H; ++r) {
                    if (z0 + seg * L + h + r == nz - 1) q[r] = qlast;
                    y[h + r] = mk<T>(y[h + r].x - corr.x * q[r].x, y[h + r].y - corr.y * q[r].y);
                }
            }
        }
        cplx<T> A = mk<T>(T(1), T(1)), nxt = zero;
#pragma unroll
        for (int r = L - 1; r >= 0; --r) {
            nxt = mk<T>(y[r].x - w[r].x * nxt.x, y[r].y - w[r].y * nxt.y);
            y[r] = nxt;
            A = mk<T>(-w[r].x * A.x, -w[r].y * A.y);
        }
        cplx<T> p = chain(std::integral_constant<int, -1>{}, A, nxt);
#pragma unroll
        for (int r = L - 1; r >= 0; --r) {
            const int z = z0 + seg * L + r;
            p = mk<T>(-w[r].x * p.x, -w[r].y * p.y);
            const cplx<T> u = cadd(y[r], p);
            if (on && z < nz) {
                col[(size_t)z * zs] = cvt<Ts>(u);
                csum += (double)u.x;
            }
        }
    }
    if (tile == 0) {
        // mean of the zero-mode solution (subtracted by the inverse kernel)
        double s = (sing && on && a.demean) ? csum : 0.0;
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) s += __shfl_down(s, off, 64);
        if ((tid & 63) == 0) red[tid >> 6] = s;
        lds_barrier();
        if (tid == 0) {
            s = 0.0;
            for (int w_ = 0; w_ < nth / 64; ++w_) s += red[w_];
            a.cmean[b] = s / (double)nz;
        }
    }
}

// ------------------------------------------------------------------ launchers
template <typename T> static int plane_threads(int nx, int ny, int slots) {
    const int nyp = (ny + 1) / 2;
    for (int nth = 256; nth <= kPlaneMaxThreads; nth *= 2)
        if (nyp * nx <= kPlaneVals<T> * nth && slots * ny <= kPlaneVals<T> * nth &&
            slots * nyp <= (kPlaneVals<T> + 1) / 2 * nth)
            return nth;
    return 0;
}
template <typename T> static size_t plane_lds_bytes(const PlaneArgs<T>& a) {
    return ((size_t)a.bufn + (size_t)(a.bx != BC_P ? 2 : 1) * a.nx + (size_t)(a.by != BC_P ? 2 : 1) * a.ny) *
           sizeof(cplx<T>);
}

template <typename T> bool plane_shape(PlaneArgs<T>& a) {
    if (a.nx > kPlaneMaxLine || a.ny > kPlaneMaxLine) return false;
    const int nyp = (a.ny + 1) / 2;
    a.ldx = a.nx | 1;
    a.ldy = a.ny | 1;
    a.bufn = nyp * a.ldx > a.slots * a.ldy ? nyp * a.ldx : a.slots * a.ldy;
    const int nth = plane_threads<T>(a.nx, a.ny, a.slots);
    if (nth == 0 || plane_lds_bytes(a) + 1024 > (size_t)kXLdsMax) return false;
    a.nth = nth;
    return true;
}
template bool plane_shape<double>(PlaneArgs<double>&);
template bool plane_shape<float>(PlaneArgs<float>&);

template <auto K> static hipError_t plane_allow() {
    return allow_dynamic_lds(reinterpret_cast<const void*>(K), kXLdsMax - 1024);
}

template <typename T, int NTH, bool FACES>
static hipError_t run_plane_fwd(const T* f, cplx<T>* S, double* partial, const PlaneArgs<T>& a, int batch,
                                const FaceArgs<T>& fa, hipStream_t s) {
    const hipError_t e = plane_allow<k_plane_fwd<T, NTH, FACES>>();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_plane_fwd<T, NTH, FACES>), dim3(a.nz, batch), dim3(NTH), plane_lds_bytes(a), s, f, S, partial,
                       a, fa);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_plane_fwd(const T* f, cplx<T>* S, double* partial, const PlaneArgs<T>& a, int batch,
                            const FaceArgs<T>* faces, hipStream_t s) {
    const FaceArgs<T> none{};
    if (faces) {
        if (a.nth == 256) return run_plane_fwd<T, 256, true>(f, S, partial, a, batch, *faces, s);
        if (a.nth == 512) return run_plane_fwd<T, 512, true>(f, S, partial, a, batch, *faces, s);
        return run_plane_fwd<T, 1024, true>(f, S, partial, a, batch, *faces, s);
    }
    if (a.nth == 256) return run_plane_fwd<T, 256, false>(f, S, partial, a, batch, none, s);
    if (a.nth == 512) return run_plane_fwd<T, 512, false>(f, S, partial, a, batch, none, s);
    return run_plane_fwd<T, 1024, false>(f, S, partial, a, batch, none, s);
}

template <typename T, int NTH>
static hipError_t run_plane_inv(const cplx<T>* S, T* u, const PlaneArgs<T>& a, int batch, const double* shift,
                                hipStream_t s) {
    const hipError_t e = plane_allow<k_plane_inv<T, NTH>>();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_plane_inv<T, NTH>), dim3(a.nz, batch), dim3(NTH), plane_lds_bytes(a), s, S, u, a, shift);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_plane_inv(const cplx<T>* S, T* u, const PlaneArgs<T>& a, int batch, const double* shift,
                            hipStream_t s) {
    if (a.nth == 256) return run_plane_inv<T, 256>(S, u, a, batch, shift, s);
    if (a.nth == 512) return run_plane_inv<T, 512>(S, u, a, batch, shift, s);
    return run_plane_inv<T, 1024>(S, u, a, batch, shift, s);
}

template <typename T, int NTH>
static hipError_t run_ylines(cplx<T>* S, LineArgs<T> a, bool inverse, hipStream_t s) {
    a.ld = a.ny | 1;
    a.group = kPlaneVals<T> * NTH / a.ny;
    if ((size_t)a.group > a.nlines) a.group = (int)a.nlines;
    const size_t lds = ((size_t)a.group * a.ld + (size_t)(a.by != BC_P ? 2 : 1) * a.ny) * sizeof(cplx<T>);
    const dim3 grid((unsigned)((a.nlines + a.group - 1) / a.group));
    const hipError_t e = inverse ? plane_allow<k_ylines<T, NTH, true>>() : plane_allow<k_ylines<T, NTH, false>>();
    if (e != hipSuccess) return e;
    if (inverse) hipLaunchKernelGGL((k_ylines<T, NTH, true>), grid, dim3(NTH), lds, s, S, a);
    else hipLaunchKernelGGL((k_ylines<T, NTH, false>), grid, dim3(NTH), lds, s, S, a);
    return hipGetLastError();
}

// Groups of 2048 (double) or 4096 (float) values: four lines of 512 and up.
template <typename T> hipError_t launch_ylines(cplx<T>* S, const LineArgs<T>& a, bool inverse, hipStream_t s) {
    return run_ylines<T, 256>(S, a, inverse, s);
}

template <typename Ts, typename T, int L, bool PERZ, bool ONE>
static hipError_t run_zscan(cplx<Ts>* S, const MidArgs<Ts>& a, const ScanArgs& g, int batch, hipStream_t s) {
    const int ct = 1 << g.lct;
    const int nth = (ct * g.segs + 63) / 64 * 64;
    const size_t lds = (size_t)(nth / 64) * (2 * ct * sizeof(cplx<T>) + sizeof(double));
    const int tiles = (a.slots * a.ny + ct - 1) / ct;
    hipLaunchKernelGGL((k_zscan<Ts, T, L, PERZ, ONE>), dim3(tiles, batch), dim3(nth), lds, s, S, a, g);
    return hipGetLastError();
}

// Columns per workgroup: 128 bytes of every plane (whole lines), twice that
// where the segments of so few would not fill a wavefront; small workgroups,
// since a CU holds 12 to 16 wavefronts of these kernels (200 x 192 x 256 f32
// periodic, 13 segments: 60 us with 32 columns, one workgroup of 7 wavefronts per
// CU).  Rows per thread: 8 up to 128 planes (more threads per column, shorter
// recurrences) and in double with periodic z (16 spill), else 16; longer columns than a workgroup holds go in chunks.
template <typename T> hipError_t launch_zscan(cplx<T>* S, const MidArgs<T>& a, ScanArgs g, int batch, hipStream_t s) {
    const int base = sizeof(T) == 8 ? 3 : 4;
    const int L = (a.nz <= 128 || (a.zper && sizeof(T) == 8)) ? 8 : 16;
    int P = (a.nz + L - 1) / L;
    g.lct = (P << base) >= 64 ? base : base + 1;
    const int pmax = kScanThreads >> g.lct;
    g.chunks = (P + pmax - 1) / pmax;
    if (g.chunks > 1) P = pmax;
    g.segs = P;
    if (a.zper) {
        if (L == 8 && g.chunks == 1) return run_zscan<T, T, 8, true, true>(S, a, g, batch, s);
        constexpr int LP = sizeof(T) == 8 ? 8 : 16;
        if (g.chunks == 1) return run_zscan<T, T, LP, true, true>(S, a, g, batch, s);
        return run_zscan<T, T, LP, true, false>(S, a, g, batch, s);
    }
    if constexpr (sizeof(T) == 4) {
        if (a.wrowsl) {
            if (L == 8) return run_zscan<T, double, 8, false, true>(S, a, g, batch, s);
            if (g.chunks == 1) return run_zscan<T, double, 16, false, true>(S, a, g, batch, s);
            return run_zscan<T, double, 16, false, false>(S, a, g, batch, s);
        }
    }
    if (L == 8) return run_zscan<T, T, 8, false, true>(S, a, g, batch, s);
    if (g.chunks == 1) return run_zscan<T, T, 16, false, true>(S, a, g, batch, s);
    return run_zscan<T, T, 16, false, false>(S, a, g, batch, s);
}

#define PP_PLANE_INST(T)                                                                                           \
    template hipError_t launch_plane_fwd<T>(const T*, cplx<T>*, double*, const PlaneArgs<T>&, int,                 \
                                            const FaceArgs<T>*, hipStream_t);                                      \
    template hipError_t launch_plane_inv<T>(const cplx<T>*, T*, const PlaneArgs<T>&, int, const double*,           \
                                            hipStream_t);                                                          \
    template hipError_t launch_ylines<T>(cplx<T>*, const LineArgs<T>&, bool, hipStream_t);                         \
    template hipError_t launch_zscan<T>(cplx<T>*, const MidArgs<T>&, ScanArgs, int, hipStream_t);
PP_PLANE_INST(double)
PP_PLANE_INST(float)

}  // namespace pp
