// Two-kernel field evaluation for small and mid-sized grids.
//
// k_slab takes the rows of one y over all layers (one work-group per instance
// and y) through the inverse z and x transforms of the electrostatic field,
// the local terms and the time step of its cells, and the forward x and z
// transforms of the new state; k_ymul does the y transforms and the tensor
// multiply between two of them.  Against the path of four kernels (y, z with
// the tensor, y, update) two launches and the two y passes' traffic go: per
// evaluation of an open grid with S bytes of unpadded x spectra, 8 S instead of
// 12 S.  What bounds it: at these sizes the latency of each kernel's chain
// (global load, exchange stages, store), so fewer and longer chains win
// (slab_fits has the figures).
//
// The spectra S hold x- and z-transformed rows in tiles of 8 kx: element (c, kx,
// kz, y) of instance b at ((((kx/8) nb + b) 3 + c) mz + kz) ny + y) 8 + kx%8 for
// kx < mx/2, and the column kx = mx/2 behind them in tiles of 8 kz, at
// (((b 3 + c) (mz/8) + kz/8) ny + y) 8 + kz%8: no tile is padded.
// These 3 nb mz ny hx values fit into S1 and S2 together, 3 nb nz (ny + my) times
// the hx of whole blocks: my >= 2 ny for a power of two, and slab_fits asks for
// 3 nz >= mz.
#include "cell.h"
#include "fft_core.h"
#include "internal.h"

namespace tdgl {

constexpr int SLAB_KX = 8;
constexpr int SLAB_THREADS = 512;     // 256 and 1024 were slower

__host__ __device__ __forceinline__ long long slab_main(const Geom &g)
{
    return (long long)3 * g.nb * g.mz * g.ny * (g.mx / 2);
}

// z transforms of the slab's 3 (M2 + 1) columns (c, kx): INV from S into the
// rows U[(c nz + z)(M2 + 1) + kx], forward back.  Eight columns of a tile sit in
// adjacent lanes, the MZ/8 threads of a column in steps of 8 lanes, all within
// one wave; the three columns kx = M2 form the last group.
template <typename T, int M2, int MZ, bool INV>
__device__ __forceinline__ void slab_z(cpx<T> *S, cpx<T> *U, cpx<T> *scr,
                                       const cpx<T> *__restrict__ tw, const Geom &g, int b, int y)
{
    constexpr int TPL = MZ / 8, GT = 8 * TPL, TILES = M2 / SLAB_KX, NGR = 3 * TILES + 1;
    constexpr int HS = M2 + 1;
    const int tid = threadIdx.x, cc = tid & 7, t = (tid >> 3) & (TPL - 1), gl = tid / GT;
    const int per = blockDim.x / GT, ny = g.ny, nz = g.nz;
    TwReg<T, MZ> tr;
    twiddle_load(tr, tw + tw_off(MZ), t);
    cpx<T> *L = scr + gl * (LinePad<MZ>::len * 8) + cc;
    const IdxStridePad ip{8};
    for (int g0 = 0; g0 < NGR; g0 += per) {
        const int gi = g0 + gl;
        const bool last = gi == NGR - 1;
        const int c = last ? cc : gi / TILES, tile = gi - c * TILES;
        const bool act = gi < NGR && (!last || cc < 3);
        const int kx = last ? M2 : tile * SLAB_KX + cc;
        cpx<T> *src = last ? S + slab_main(g) + ((long long)(b * 3 + c) * (MZ / 8) * ny + y) * 8
                           : S + (((long long)(tile * g.nb + b) * 3 + c) * MZ * ny + y) * 8 + cc;
        auto at = [&](int kz) {
            return last ? (kz >> 3) * ny * 8 + (kz & 7) : kz * ny * 8;
        };
        cpx<T> *row = U + (act ? c : 0) * nz * HS + kx;
        cpx<T> v[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int k = t + q * TPL;
            v[q] = {T(0), T(0)};
            if (act && INV) v[q] = src[at(k)];
            if (act && !INV && k < nz) v[q] = row[k * HS];
        }
        fft_line<T, MZ, INV, IdxStridePad, true>(v, L, ip, t, tr, act);
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int k = t + q * TPL;
            if (act && INV && k < nz) row[k * HS] = v[q];
            if (act && !INV) src[at(k)] = v[q];
        }
        line_sync<true>();                         // the line's scratch is free again
    }
}

template <typename T, int M2, bool INV>
__device__ __forceinline__ void slab_z_any(cpx<T> *S, cpx<T> *U, cpx<T> *scr,
                                           const cpx<T> *__restrict__ tw, const Geom &g, int b,
                                           int y)
{
    switch (g.mz) {                                // uniform
    case 8: slab_z<T, M2, 8, INV>(S, U, scr, tw, g, b, y); break;
    case 16: slab_z<T, M2, 16, INV>(S, U, scr, tw, g, b, y); break;
    case 32: slab_z<T, M2, 32, INV>(S, U, scr, tw, g, b, y); break;
    default: slab_z<T, M2, 64, INV>(S, U, scr, tw, g, b, y); break;
    }
}

// x transforms of the slab's 3 nz rows in place: the half spectrum X[0..M2] of
// a row <-> its reals as M2 complex pairs (real_merge, real_split)
template <typename T, int M, bool INV>
__device__ __forceinline__ void slab_x(cpx<T> *U, cpx<T> *scr, const cpx<T> *__restrict__ tw,
                                       int nx, int nz)
{
    constexpr int M2 = M / 2, HS = M2 + 1;
    constexpr int PPT = HalfLine<M2>::PPT, TPL = HalfLine<M2>::TPL, LEN = LinePad<M2>::len;
    static_assert(64 % TPL == 0, "a line must not straddle waves");
    const int tid = threadIdx.x, lane = tid & 63, ll = tid / TPL, t = tid - ll * TPL;
    const int partner = (lane - t) + ((TPL - t) & (TPL - 1));
    const int per = blockDim.x / TPL, rows = 3 * nz;
    TwReg<T, M2> tr;
    twiddle_load(tr, tw + tw_off(M2), t);
    cpx<T> wk[PPT];
#pragma unroll
    for (int q = 0; q < PPT; ++q) wk[q] = tw[tw_off(M) + t + q * TPL];
    cpx<T> *L = scr + ll * LEN;
    for (int l0 = 0; l0 < rows; l0 += per) {
        const int l = l0 + ll;
        const bool act = l < rows;
        cpx<T> *row = U + (act ? l : 0) * HS;
        cpx<T> v[PPT];
        if constexpr (INV) {
#pragma unroll
            for (int q = 0; q < PPT; ++q) {
                const int k = t + q * TPL;
                cpx<T> p = row[k], m = row[M2 - k];
                if (k == 0) p.y = m.y = T(0);      // X[0], X[M/2] are real
                v[q] = real_merge(p, m, wk[q]);
            }
            half_fft<T, M2, true, true>(v, L, t, tr, act);
            line_sync<true>();
#pragma unroll
            for (int q = 0; q < PPT; ++q)
                if (act && 2 * (t + q * TPL) < nx) row[t + q * TPL] = v[q];
        } else {
#pragma unroll
            for (int q = 0; q < PPT; ++q) {
                const int n = t + q * TPL;
                v[q] = {T(0), T(0)};
                if (2 * n < nx) v[q] = row[n];
                if (2 * n + 1 >= nx) v[q].y = T(0);
            }
            half_fft<T, M2, false, true>(v, L, t, tr, act);
            line_sync<true>();
#pragma unroll
            for (int q = 0; q < PPT; ++q) {
                // Z[M2 - k]: lane TPL - t, point PPT-1-q; for t = 0 this lane's
                const int qs = PPT - 1 - q;
                cpx<T> zm = {__shfl(v[qs].x, partner, 64), __shfl(v[qs].y, partner, 64)};
                if (t == 0) zm = v[(PPT - q) % PPT];
                cpx<T> xh;
                const cpx<T> xk = real_split(v[q], zm, wk[q], xh);
                if (act) row[t + q * TPL] = xk;
                if (act && t == 0 && q == 0) row[M2] = xh;
            }
        }
        line_sync<true>();
    }
}

// The values a cell's local terms need: centre, neighbours (-x +x -y +y -z +z; a
// missing one is the centre), old state (two-stage schemes)
template <typename T>
struct SlabCell {
    T p[3], n[6][3], old[3];
};

template <typename T, int M, int MODE>
__global__ void __launch_bounds__(SLAB_THREADS)
    k_slab(UpdArgs a, Geom g, const cpx<T> *__restrict__ tw)
{
    constexpr int M2 = M / 2, HS = M2 + 1;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    const int nx = g.nx, ny = g.ny, nz = g.nz, tid = threadIdx.x, nthr = blockDim.x;
    cpx<T> *U = reinterpret_cast<cpx<T> *>(smem_raw);            // [3 nz][HS]
    cpx<T> *scr = U + 3 * nz * HS;                                // transform exchanges
    T *lc = reinterpret_cast<T *>(scr + nthr * (HalfLine<M2>::PPT * 9) / 8);   // [nz][NCOEF]
    const unsigned tile = xcd_tile(blockIdx.x, gridDim.x);        // (instance, y)
    const int b = (int)udiv(tile, (unsigned)ny, a.mgx), y = (int)tile - b * ny;
    const int plane = nx * ny, ncell = nz * nx;
    const long long comp = (long long)nz * plane;
    const T *Pin = reinterpret_cast<const T *>(a.P_in) + 3LL * b * comp;
    T *Pout = reinterpret_cast<T *>(a.P_out) + 3LL * b * comp;
    const unsigned nx_div = 0xffffffffu / (unsigned)nx + 1u;      // e / nx for e < 2^16
    if (g.frozen && g.frozen[b]) {                                // a retired instance
        if constexpr (MODE == UPD_STEP) {                         // carried over unchanged
            for (int e = tid; e < 3 * ncell; e += nthr) {
                const int l = e / nx, x = e - l * nx;
                const long long o = (long long)l * plane + y * nx + x;
                Pout[o] = Pin[o];
            }
        } else if (MODE == UPD_ENERGY && tid < 8) {
            a.partials[(long long)tile * 8 + tid] = 0.0;
        }
        return;
    }
    cpx<T> *S = reinterpret_cast<cpx<T> *>(a.S1);
    const KParams<T> *kp = reinterpret_cast<const KParams<T> *>(a.kp);
    const T *Pold = reinterpret_cast<const T *>(a.P_old);
    const unsigned terms = a.terms;
    const bool need_nb = (terms & T_GRAD) != 0;
    const bool need_old =
        (MODE == UPD_STEP && a.stage == 1) || (MODE == UPD_STEP_MS && a.stage == 3);
    constexpr unsigned SZ = sizeof(T);
    auto load = [&](int e, SlabCell<T> &s) {       // cell e = (z, x) of this y; all loads
        const int z = nx == 1 ? e : (int)__umulhi((unsigned)e, nx_div), x = e - z * nx;
        const unsigned o = (unsigned)(z * plane + y * nx + x) * SZ;
        const unsigned cb = (unsigned)comp * SZ;
#pragma unroll
        for (int c = 0; c < 3; ++c) s.p[c] = ld_at(Pin, o + c * cb);
        if (need_nb) {
            const int d[6] = {x > 0 ? -1 : 0,       x < nx - 1 ? 1 : 0,  y > 0 ? -nx : 0,
                              y < ny - 1 ? nx : 0,  z > 0 ? -plane : 0,  z < nz - 1 ? plane : 0};
#pragma unroll
            for (int k = 0; k < 6; ++k)
#pragma unroll
                for (int c = 0; c < 3; ++c) s.n[k][c] = ld_at(Pin, o + c * cb + (unsigned)(d[k] * (int)SZ));
        }
        if (need_old) {
#pragma unroll
            for (int c = 0; c < 3; ++c) s.old[c] = ld_at(Pold + 3LL * b * comp, o + c * cb);
        }
    };

    // the first cell of every thread travels while the field is transformed
    SlabCell<T> cell;
    if (tid < ncell) load(tid, cell);
    if constexpr (MODE != UPD_FX) {
        const T *coef = reinterpret_cast<const T *>(a.coef) + (long long)b * nz * NCOEF;
        for (int e = tid; e < nz * NCOEF; e += nthr) lc[e] = coef[e];
        slab_z_any<T, M2, true>(S, U, scr, tw, g, b, y);
        __syncthreads();
        slab_x<T, M, true>(U, scr, tw, nx, nz);
        __syncthreads();
    }

    double acc[7] = {0, 0, 0, 0, 0, 0, 0};
    T rkerr = T(0);
    const T dtau = kp->dtau;
    for (int e = tid; e < ncell; e += nthr) {
        if (e != tid) load(e, cell);
        const int z = nx == 1 ? e : (int)__umulhi((unsigned)e, nx_div), x = e - z * nx;
        const T *p = cell.p;
        const unsigned off = (unsigned)(z * plane + y * nx + x);
        auto real = [&](int c) -> T & {            // this cell in the slab's real rows
            return reinterpret_cast<T *>(U + (c * nz + z) * HS)[x];
        };
        if constexpr (MODE == UPD_FX) {
#pragma unroll
            for (int c = 0; c < 3; ++c) real(c) = p[c];
            continue;
        }
        const T *cf = lc + z * NCOEF;
        const bool material = cf[8] != T(0);
        T E[3] = {T(0), T(0), T(0)}, hel[3], sq[3], fg = T(0);
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            hel[c] = real(c);
            sq[c] = p[c] * p[c];
        }
        if (material) {
            if (terms & T_LANDAU) {
#pragma unroll
                for (int c = 0; c < 3; ++c) E[c] -= landau_dfdp(p, sq, cf, c);
            }
            if (terms & T_GRAD) {
                // z neighbours in vacuum layers are dropped (they read as the centre)
                const bool hzm = z > 0 && lc[(z - 1) * NCOEF + 8] != T(0);
                const bool hzp = z < nz - 1 && lc[(z + 1) * NCOEF + 8] != T(0);
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    if (!hzm) cell.n[4][c] = p[c];
                    if (!hzp) cell.n[5][c] = p[c];
                }
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    const T pc = p[c];
                    const T lx = (cell.n[0][c] - pc) + (cell.n[1][c] - pc);
                    const T ly = (cell.n[2][c] - pc) + (cell.n[3][c] - pc);
                    const T lz = (cell.n[4][c] - pc) + (cell.n[5][c] - pc);
                    E[c] += kp->gh2[c][0] * lx + kp->gh2[c][1] * ly + kp->gh2[c][2] * lz;
                    if (MODE == UPD_ENERGY) {      // edges towards +x, +y, +z, each once
                        const T dx = cell.n[1][c] - pc, dy = cell.n[3][c] - pc,
                                dz = cell.n[5][c] - pc;
                        fg += T(0.5) * (kp->gh2[c][0] * dx * dx + kp->gh2[c][1] * dy * dy +
                                        kp->gh2[c][2] * dz * dz);
                    }
                }
                if (MODE == UPD_ENERGY && (kp->g12 != T(0) || kp->gm != T(0))) {
                    T D[3][3];                     // D[i][d] = D_d P_i (see k_cross)
#pragma unroll
                    for (int i = 0; i < 3; ++i)
#pragma unroll
                        for (int d = 0; d < 3; ++d)
                            D[i][d] = (cell.n[2 * d + 1][i] - cell.n[2 * d][i]) * kp->inv2h[d];
                    fg += kp->g12 * (D[0][0] * D[1][1] + D[1][1] * D[2][2] + D[2][2] * D[0][0]) +
                          kp->gm * (D[0][1] * D[1][0] + D[1][2] * D[2][1] + D[2][0] * D[0][2]);
                }
                if (a.cross) {                     // the cross terms' field, from k_cross
                    const T *hx = reinterpret_cast<const T *>(a.cross) + 3LL * b * comp;
#pragma unroll
                    for (int c = 0; c < 3; ++c) E[c] += hx[c * comp + off];
                }
            }
#pragma unroll
            for (int c = 0; c < 3; ++c) E[c] += hel[c];
            if (terms & T_EXT) {
#pragma unroll
                for (int c = 0; c < 3; ++c) E[c] += kp->eext[c];
            }
        }
        if constexpr (MODE == UPD_ENERGY) {
            if (material) {
                if (terms & T_LANDAU) acc[0] += (double)landau_f(sq, cf);
                acc[1] += (double)fg;
                acc[2] += -0.5 * ((double)p[0] * hel[0] + (double)p[1] * hel[1] +
                                  (double)p[2] * hel[2]);
                if (terms & T_EXT)
                    acc[3] += -((double)p[0] * kp->eext[0] + (double)p[1] * kp->eext[1] +
                                (double)p[2] * kp->eext[2]);
#pragma unroll
                for (int c = 0; c < 3; ++c) acc[4 + c] += (double)p[c];
            }
        } else if constexpr (MODE == UPD_FIELD) {
#pragma unroll
            for (int c = 0; c < 3; ++c)
                Pout[c * comp + off] = material ? kp->out_scale * E[c] : T(0);
        } else {
            T o[3];
            bool bad = false;
            const bool store = !(MODE == UPD_STEP_RK && a.stage == 7);
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const T e1 = material ? E[c] : T(0);
                const long long ho = 3LL * b * comp + c * comp + off;   // history, RK buffers
                if constexpr (MODE == UPD_STEP) {
                    if (a.stage == 0) o[c] = p[c] + dtau * e1;
                    else o[c] = T(0.5) * (cell.old[c] + p[c]) + T(0.5) * dtau * e1;
                    if (!material) o[c] = T(0);
                } else if constexpr (MODE == UPD_STEP_MS) {
                    const T *ha = reinterpret_cast<const T *>(a.hist_a);
                    const T *hb = reinterpret_cast<const T *>(a.hist_b);
                    const T k12 = dtau / T(12);
                    if (a.stage == 0) o[c] = p[c] + dtau * e1;           // Heun predictor
                    else if (a.stage == 2)                               // AB3 predictor
                        o[c] = p[c] + k12 * (T(23) * e1 - T(16) * ha[ho] + T(5) * hb[ho]);
                    else                                                 // AM2 corrector
                        o[c] = cell.old[c] + k12 * (T(5) * e1 + T(8) * ha[ho] - hb[ho]);
                    if (!material) o[c] = T(0);
                    if (a.stage != 3) reinterpret_cast<T *>(a.hist_w)[ho] = e1;
                } else {                                                 // UPD_STEP_RK
                    const int st = a.stage;
                    const long long ko = 3LL * g.nb * comp;              // one k buffer
                    T *K = reinterpret_cast<T *>(a.rk_k);
                    const T pn = reinterpret_cast<const T *>(a.rk_base)[ho];
                    const T h = (T)a.rk->h;
                    K[(st - 1) * ko + ho] = e1;
                    if (st < 7) {
                        T s = T(RK_A[st - 1][st - 1]) * e1;
                        for (int j = 0; j < st - 1; ++j) s += T(RK_A[st - 1][j]) * K[j * ko + ho];
                        o[c] = material ? pn + h * s : T(0);
                    } else {
                        T s = T(RK_E[6]) * e1;
                        for (int j = 0; j < 6; ++j) s += T(RK_E[j]) * K[j * ko + ho];
                        const T m = fabs(pn) > fabs(p[c]) ? fabs(pn) : fabs(p[c]);
                        const T r = rk_scaled(h * s, T(a.rk->atol) + T(a.rk->rtol) * m);
                        rkerr = r > rkerr ? r : rkerr;
                        o[c] = p[c];               // P5 itself (for the spectrum)
                    }
                }
                if (store) Pout[c * comp + off] = o[c];
                bad = bad || !isfinite(o[c]);
                real(c) = o[c];
            }
            if (bad) atomicOr(a.flag, 1);
        }
    }

    if constexpr (MODE == UPD_ENERGY || MODE == UPD_STEP_RK) {
        if (MODE == UPD_ENERGY || a.stage == 7) {
            // sums (energies) or the maximum (scaled error, entry 0) of the group
            constexpr int NV = MODE == UPD_ENERGY ? 7 : 1;
            __syncthreads();
            double *red = reinterpret_cast<double *>(scr);
            if (MODE == UPD_STEP_RK) acc[0] = (double)rkerr;
#pragma unroll
            for (int k = 0; k < NV; ++k) {
                double v = acc[k];
                for (int o = 32; o > 0; o >>= 1) {
                    const double w = __shfl_xor(v, o, 64);
                    v = MODE == UPD_ENERGY ? v + w : (w > v ? w : v);
                }
                if ((tid & 63) == 0) red[(tid >> 6) * 8 + k] = v;
            }
            __syncthreads();
            if (tid < NV) {
                double v = red[tid];
                for (int w = 1; w < (nthr + 63) / 64; ++w) {
                    const double u = red[w * 8 + tid];
                    v = MODE == UPD_ENERGY ? v + u : (u > v ? u : v);
                }
                a.partials[(long long)tile * 8 + tid] = v;
            }
        }
    }
    if constexpr (MODE != UPD_ENERGY && MODE != UPD_FIELD) {
        __syncthreads();
        slab_x<T, M, false>(U, scr, tw, nx, nz);
        __syncthreads();
        slab_z_any<T, M2, false>(S, U, scr, tw, g, b, y);
    }
}

// y transforms and tensor multiply: G tiles of 8 columns (kx of one kz, or kz
// of kx = mx/2) x 3 components per work-group, in place.  As the z pass with the
// tensor (k_zmul), with y as the transformed dimension.
template <typename T, int MY>
struct YmulCfg {
    static constexpr int PPT = Plan<MY>::PPT, TPL = Plan<MY>::TPL;
    static constexpr int G = TPL >= 8 ? 1 : 8 / TPL;             // at least 192 threads
    static constexpr int NTHR = G * 24 * TPL;
    static constexpr size_t LDS = (size_t)G * 24 * LinePad<MY>::len * sizeof(cpx<T>);
};

template <typename T, int MY>
__global__ void __launch_bounds__((YmulCfg<T, MY>::NTHR))
    k_ymul(cpx<T> *S, const T *__restrict__ Nt, Geom g, const cpx<T> *__restrict__ tw,
           unsigned ntile)
{
    using C = YmulCfg<T, MY>;
    constexpr int PPT = C::PPT, TPL = C::TPL, LEN = LinePad<MY>::len;
    constexpr bool WAVE = 8 * TPL <= 64;           // a line's lanes lie within one wave
    extern __shared__ __align__(16) unsigned char smem_raw[];
    const int tid = threadIdx.x, cc = tid & 7, t = (tid >> 3) & (TPL - 1);
    const int cs = tid / (8 * TPL), sub = cs / 3, c = cs - 3 * sub;
    const int ny = g.ny, mz = g.mz, nb = g.nb, M2 = g.mx / 2;
    const unsigned tile = xcd_tile(blockIdx.x, gridDim.x) * C::G + sub;
    const unsigned nmain = (unsigned)(M2 / SLAB_KX) * nb * mz;
    const bool last = tile >= nmain;               // a tile of the column kx = mx/2
    const unsigned r = last ? tile - nmain : tile, dz = last ? mz / 8 : mz;
    const int kb = (int)(r / dz), kzt = (int)(r - kb * dz);      // (kx tile, instance), kz or its tile
    const int b = last ? kb : kb % nb, kx = last ? M2 : kb / nb * SLAB_KX + cc;
    const int kz = last ? kzt * 8 + cc : kzt;
    bool act = tile < ntile;
    if (act && g.frozen && g.frozen[b]) act = false;
    cpx<T> *base = S + (last ? slab_main(g) : 0) +
                   (act ? (((long long)kb * 3 + c) * dz + kzt) * ny * 8 + cc : 0);
    cpx<T> v[PPT];
#pragma unroll
    for (int q = 0; q < PPT; ++q) {
        const int y = t + q * TPL;
        v[q] = (act && y < ny) ? base[y * 8] : cpx<T>{T(0), T(0)};
    }
    // row c of the tensor (octant store in blocks of KB kx, as in k_zmul): xy is
    // odd in ky, xz odd in kz, yz odd in both
    const int hy = MY / 2 + 1, hz = mz / 2 + 1;
    const bool zneg = kz > mz / 2;
    const unsigned qs = (unsigned)hz * hy * KB;
    const unsigned o0 = ((unsigned)(kx >> KBS) * 6 * qs + (unsigned)(zneg ? mz - kz : kz) * hy * KB +
                         (kx & (KB - 1)));
    const int i0 = c == 0 ? 0 : (c == 1 ? 3 : 4), i1 = c == 0 ? 3 : (c == 1 ? 1 : 5),
              i2 = c == 0 ? 4 : (c == 1 ? 5 : 2);
    T n[PPT][3];
#pragma unroll
    for (int q = 0; q < PPT; ++q) {
        const int ky = t + q * TPL;
        const bool yneg = ky > MY / 2;
        const T *p = Nt + (act ? o0 + (unsigned)(yneg ? MY - ky : ky) * KB : 0u);
        auto sign = [&](int i) {
            return ((i == 3 && yneg) || (i == 4 && zneg) || (i == 5 && yneg != zneg)) ? T(-1) : T(1);
        };
        n[q][0] = p[i0 * qs] * sign(i0);
        n[q][1] = p[i1 * qs] * sign(i1);
        n[q][2] = p[i2 * qs] * sign(i2);
    }
    TwReg<T, MY> tr;
    twiddle_load(tr, tw + tw_off(MY), t);
    const IdxStridePad ip{8};
    cpx<T> *lds = reinterpret_cast<cpx<T> *>(smem_raw) + sub * 24 * LEN;
    cpx<T> *L = lds + c * LEN * 8 + cc;
    fft_line<T, MY, false, IdxStridePad, WAVE>(v, L, ip, t, tr, act);
    __syncthreads();
    if (act) {
#pragma unroll
        for (int q = 0; q < PPT; ++q) lds_put(&L[ip(t + q * TPL)], v[q]);
    }
    __syncthreads();
    if (act) {
#pragma unroll
        for (int q = 0; q < PPT; ++q) {
            const int o = ip(t + q * TPL) + cc;
            const cpx<T> p0 = lds[o], p1 = lds[LEN * 8 + o], p2 = lds[2 * LEN * 8 + o];
            v[q] = {n[q][0] * p0.x + n[q][1] * p1.x + n[q][2] * p2.x,
                    n[q][0] * p0.y + n[q][1] * p1.y + n[q][2] * p2.y};
        }
    }
    __syncthreads();
    fft_line<T, MY, true, IdxStridePad, WAVE>(v, L, ip, t, tr, act);
#pragma unroll
    for (int q = 0; q < PPT; ++q) {
        const int y = t + q * TPL;
        if (act && y < ny) base[y * 8] = v[q];
    }
}

// -------------------------------------------------------------- launchers
// threads of k_slab: enough for the widest of its phases, at most 512
template <typename T, int M>
static int slab_threads(const Geom &g)
{
    constexpr int M2 = M / 2;
    int n = 3 * g.nz * HalfLine<M2>::TPL;                        // x rows
    const int z = (3 * (M2 / SLAB_KX) + 1) * g.mz;               // z columns
    if (z > n) n = z;
    if (g.nz * g.nx > n) n = g.nz * g.nx;                        // cells
    n = (n + 63) / 64 * 64;
    return n > SLAB_THREADS ? SLAB_THREADS : n;
}

template <typename T, int M>
static size_t slab_lds(const Geom &g)
{
    constexpr int M2 = M / 2;
    const size_t c = (size_t)3 * g.nz * (M2 + 1) + (size_t)slab_threads<T, M>(g) * HalfLine<M2>::PPT * 9 / 8;
    return c * sizeof(cpx<T>) + (size_t)g.nz * NCOEF * sizeof(T);
}

#define TDGL_SLAB_MX(CALL)                             \
    switch (g.mx) {                                    \
    case 16: { constexpr int LEN_ = 16; CALL; }        \
    case 32: { constexpr int LEN_ = 32; CALL; }        \
    case 64: { constexpr int LEN_ = 64; CALL; }        \
    case 128: { constexpr int LEN_ = 128; CALL; }      \
    default: return hipErrorInvalidValue;              \
    }

#define TDGL_SLAB_MY(CALL)                             \
    switch (g.my) {                                    \
    case 8: { constexpr int LEN_ = 8; CALL; }          \
    case 16: { constexpr int LEN_ = 16; CALL; }        \
    case 32: { constexpr int LEN_ = 32; CALL; }        \
    case 64: { constexpr int LEN_ = 64; CALL; }        \
    default: return hipErrorInvalidValue;              \
    }

template <typename T, int M, int MODE>
static hipError_t slab_one(const Geom &g, const UpdArgs &a, const void *tw, hipStream_t s,
                           bool prepare, size_t lds_max)
{
    const size_t shm = slab_lds<T, M>(g);
    if (prepare) {
        // the limit belongs to the kernel, which contexts of other heights share:
        // the device's, not this grid's
        if (shm > lds_max) return hipErrorInvalidConfiguration;
        return lds_max <= 65536 ? hipSuccess
                                : hipFuncSetAttribute((const void *)k_slab<T, M, MODE>,
                                                      hipFuncAttributeMaxDynamicSharedMemorySize,
                                                      (int)lds_max);
    }
    UpdArgs am = a;
    const unsigned n = (unsigned)(g.ny * g.nb);
    am.mgx = div_magic((unsigned)g.ny, n);
    hipLaunchKernelGGL((k_slab<T, M, MODE>), dim3(n), dim3(slab_threads<T, M>(g)), shm, s, am, g,
                       (const cpx<T> *)tw);
    return hipGetLastError();
}

template <typename T, int M>
static hipError_t slab_mode(int mode, const Geom &g, const UpdArgs &a, const void *tw,
                            hipStream_t s, bool prepare, size_t lds_max)
{
    switch (mode) {
    case UPD_STEP: return slab_one<T, M, UPD_STEP>(g, a, tw, s, prepare, lds_max);
    case UPD_FIELD: return slab_one<T, M, UPD_FIELD>(g, a, tw, s, prepare, lds_max);
    case UPD_ENERGY: return slab_one<T, M, UPD_ENERGY>(g, a, tw, s, prepare, lds_max);
    case UPD_STEP_MS: return slab_one<T, M, UPD_STEP_MS>(g, a, tw, s, prepare, lds_max);
    case UPD_STEP_RK: return slab_one<T, M, UPD_STEP_RK>(g, a, tw, s, prepare, lds_max);
    default: return slab_one<T, M, UPD_FX>(g, a, tw, s, prepare, lds_max);
    }
}

static hipError_t slab_any(int prec, int mode, const Geom &g, const UpdArgs &a, const void *tw,
                           hipStream_t s, bool prepare, size_t lds_max)
{
    if (prec == PREC_F32) {
        TDGL_SLAB_MX(return (slab_mode<float, LEN_>(mode, g, a, tw, s, prepare, lds_max)))
    } else {
        TDGL_SLAB_MX(return (slab_mode<double, LEN_>(mode, g, a, tw, s, prepare, lds_max)))
    }
}

hipError_t launch_slab(int prec, int mode, const Geom &g, const UpdArgs &a, const void *tw,
                       hipStream_t s)
{
    return slab_any(prec, mode, g, a, tw, s, false, 0);
}

template <typename T, int MY>
static hipError_t ymul_impl(const Geom &g, void *S, const void *Nt, const void *tw, hipStream_t s)
{
    using C = YmulCfg<T, MY>;
    static_assert(C::LDS <= 65536, "above the default limit");
    const unsigned n = (unsigned)((g.mx / 2 / SLAB_KX) * g.nb * g.mz + g.nb * (g.mz / 8));
    hipLaunchKernelGGL((k_ymul<T, MY>), dim3((n + C::G - 1) / C::G), dim3(C::NTHR), C::LDS, s,
                       (cpx<T> *)S, (const T *)Nt, g, (const cpx<T> *)tw, n);
    return hipGetLastError();
}

hipError_t launch_ymul(int prec, const Geom &g, void *S, const void *Nt, const void *tw,
                       hipStream_t s)
{
    if (prec == PREC_F32) {
        TDGL_SLAB_MY(return (ymul_impl<float, LEN_>(g, S, Nt, tw, s)))
    } else {
        TDGL_SLAB_MY(return (ymul_impl<double, LEN_>(g, S, Nt, tw, s)))
    }
}

hipError_t prepare_slab(int prec, const Geom &g, size_t lds_max)
{
    const int modes[6] = {UPD_STEP, UPD_FIELD, UPD_ENERGY, UPD_STEP_MS, UPD_STEP_RK, UPD_FX};
    for (int m : modes) {
        const hipError_t e = slab_any(prec, m, g, UpdArgs{}, nullptr, nullptr, true, lds_max);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// Open boxes of powers of two.  Heun steps in us, this path against the fused
// plane or three passes, one box / 8 / 64 of them:
//   8x8x8      FP32 20.9/23.1  20.8/21.2  23.6/27.3    FP64 22.6/25.4  22.5/23.2  29.0/35.0
//   16x16x8    FP32 23.3/26.7  23.7/24.3  40.7/44.9    FP64 25.8/29.5  27.6/27.3  65.8/66.5
//   32x32x8    FP32 24.9/30.6  32.2/34.7  93.2/126     FP64 28.5/33.4  43.4/49.2  149/209
//   32x32x16   FP32 28.0/31.6  42.9/56.0  158/172      FP64 34.7/37.7  65.7/75.5  288/319
//   62x32x8    FP32 27.5/32.3  40.9/41.9  152/148      FP64 34.3/36.3  66.2/70.2  282/274
//   15x32x32   FP32 30.0/31.0  43.4/58.7  175/187      FP64 35.9/37.9  64.3/73.1  305/344
//   16x30x24   FP32 27.6/33.9  39.9/54.7  168/158      FP64 34.0/39.8  62.3/83.0  289/305
// Wider slabs (w, the values of one y's spectra) wait longer than the launches
// cost, sooner where few rows of y share the tensor pass: my = 32 at w = 1584,
// 30x16x8, FP64 27.9/30.6 33.9/31.7 89.2/99.1, and at 3120 47.5/37.3 for 8 of
// 60x16x8.  Thin boxes have cheap planes (nz my points) and a slab that is half
// padding: 30x30x2 FP32 22.6/24.2 25.3/23.7 62.0/43.4; 64 of 32x8x3 FP64 40.4/38.3,
// 256 FP32 60.6/49.3 (but 32x3x3 20.1/23.2 21.8/25.4 for 1 and 64, 16x8x3 37.3/35.7 only
// for 256); 16x32x20 (mz = 64) FP64
// 33.5/38.2 -/- 436/414 (100 of them).  Periodic films have no padding in x and
// y to leave out: 32x32x8 FP32 24.1/27.4 -/- 72.3/57.4.  Lengths 3 * 2^a hold
// 12 points a thread: 40x40x10, 8 of them, 0.82 of the three passes' speed.
// The rule does not look at the number of instances, so that a batch and
// separate contexts add up energies in the same order.
static bool pow2(int n) { return (n & (n - 1)) == 0; }

bool slab_fits(const Geom &g)
{
    if (g.px || g.py || g.pz || g.mx < 16 || g.my > 64 || g.mz > 64) return false;
    if (!pow2(g.mx) || !pow2(g.my) || !pow2(g.mz) || 3 * g.nz < g.mz) return false;
    const int w = 3 * (g.mx / 2 + 1) * g.mz;       // mx <= 128 by the limits
    if (g.my <= 16) return w <= (g.nz > 3 || g.my == 8 ? 900 : 500);
    return g.nz >= 7 && w <= (g.my == 64 ? 3300 : 900);
}

}  // namespace tdgl
