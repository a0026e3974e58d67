// Electrostatic interaction tensor, built once per geometry in FP64.
//
// For P uniform inside each box cell (paper section 3), the bound charges of
// eq 6 sit on cell faces and the field averaged over a target cell is
//   E(target) = -1/(eps0 epsB) * sum_src N(r_t - r_s) P(src),
//   N_ij(R)   = -1/(4 pi V) Int_tgt Int_src d_i d_j |x - x'|^-1,
// the cell-averaged dipolar ("demagnetising") tensor of two boxes.
//
// Evaluation:
//  * touching or overlapping cells (every |o_k| <= 1): Newell's closed form,
//    N_xx = -(1/(4 pi V)) * (triple second difference of f), N_xy likewise
//    with g, where d_y^2 d_z^2 f = 1/r and d_x d_y d_z^2 g = 1/r;
//  * all other offsets: the double cell integral is one integral of
//    (delta_ij r^2 - 3 r_i r_j)/r^5 against the tent weight prod(d_k - |u_k|)
//    over [-d, d]^3, done with the n-point Gauss rule of the tent weight in
//    every dimension, or n Gauss-Legendre nodes on each of its halves where that
//    needs more points than the tables hold (host tables, quadrature_tables);
//    n from the Bernstein-ellipse bound of the nearest complex singularity
//    (error target 1e-17 relative to the entry).
// Every entry is even or odd in each offset component, so only the offsets of
// one octant are evaluated (k_tensor_octant_real); periodic dimensions sum
// lattice images o + m N with |o + m N| <= (mimg + 1/2) N, weight 1/2 on the
// window edge.  Placement (k_tensor_expand): open dimensions use wrap-around
// order on the padded grid (offset o at o mod M, the gap N..M-N is zero).  k_tensor_k0 then sets the in-plane k = 0
// mode of an x-y periodic film to its infinite-lattice value (a uniformly
// polarised infinite sheet: zz sum 1 in its own layer, every other sum 0).
#include <cmath>

#include "fft_core.h"
#include "internal.h"

namespace tdgl {

__device__ static double newell_fd(double x, double y, double z)
{
    x = fabs(x);
    y = fabs(y);
    z = fabs(z);
    const double x2 = x * x, y2 = y * y, z2 = z * z;
    const double R = sqrt(x2 + y2 + z2);
    if (R == 0.0) return 0.0;
    double r = (2.0 * x2 - y2 - z2) * R / 6.0;
    if (y > 0.0 && x2 + z2 > 0.0) r += 0.5 * y * (z2 - x2) * asinh(y / sqrt(x2 + z2));
    if (z > 0.0 && x2 + y2 > 0.0) r += 0.5 * z * (y2 - x2) * asinh(z / sqrt(x2 + y2));
    if (x > 0.0 && y > 0.0 && z > 0.0) r -= x * y * z * atan(y * z / (x * R));
    return r;
}

__device__ static double newell_gd(double x, double y, double z)
{
    double sgn = 1.0;
    if (x < 0.0) { sgn = -sgn; x = -x; }
    if (y < 0.0) { sgn = -sgn; y = -y; }
    z = fabs(z);
    const double x2 = x * x, y2 = y * y, z2 = z * z;
    const double R = sqrt(x2 + y2 + z2);
    if (R == 0.0) return 0.0;
    double r = -x * y * R / 3.0;
    if (z > 0.0 && x2 + y2 > 0.0) r += x * y * z * asinh(z / sqrt(x2 + y2));
    if (x > 0.0 && y2 + z2 > 0.0) r += y / 6.0 * (3.0 * z2 - y2) * asinh(x / sqrt(y2 + z2));
    if (y > 0.0 && x2 + z2 > 0.0) r += x / 6.0 * (3.0 * z2 - x2) * asinh(y / sqrt(x2 + z2));
    if (z > 0.0) r -= z2 * z / 6.0 * atan(x * y / (z * R));
    if (y > 0.0) r -= z * y2 / 2.0 * atan(x * z / (y * R));
    if (x > 0.0) r -= z * x2 / 2.0 * atan(y * z / (x * R));
    return sgn * r;
}

// Term e (0..161) of the closed form: component q = e / 27 (xx yy zz from f, xy
// xz yz from g, with the coordinates permuted), term e % 27 = (i + 1, j + 1,
// k + 1) in base 3 of its triple second difference sum_{i,j,k in -1..1}
// w_i w_j w_k fn(X+i a, Y+j b, Z+k c), w = (1,-2,1)
__device__ static double newell_term(int e, const double (&R)[3], const double (&d)[3])
{
    const int q = e / 27, f = e - q * 27;
    const int p0 = q == 1 ? 1 : (q == 2 ? 2 : (q == 5 ? 1 : 0));
    const int p1 = q == 1 ? 0 : (q == 4 || q == 5 ? 2 : 1);
    const int p2 = 3 - p0 - p1;
    const int i = f / 9 - 1, j = f / 3 % 3 - 1, k = f % 3 - 1;
    const double w = (i == 0 ? -2.0 : 1.0) * (j == 0 ? -2.0 : 1.0) * (k == 0 ? -2.0 : 1.0);
    auto at = [](const double (&v)[3], int n) { return n == 0 ? v[0] : (n == 1 ? v[1] : v[2]); };
    const double x = at(R, p0) + i * at(d, p0), y = at(R, p1) + j * at(d, p1),
                 z = at(R, p2) + k * at(d, p2);
    return w * (q < 3 ? newell_fd(x, y, z) : newell_gd(x, y, z));
}

// The quadrature rule (nodes and weights, n of them in every dimension) for
// the entry at integer offset (ox, oy, oz).  In the variable of one dimension the
// integrand is singular where r^2 = 0, at a distance of at least gap from
// [-d, d], which for an offset of 0 in that dimension lies beside its centre,
// the normalised point i gap/d.  The Gauss rule of the tent weight on the whole
// of [-d, d] converges as rho^-2n, rho = g + sqrt(1 + g^2), g = gap / dmax;
// two Gauss-Legendre rules, one on each half, see the singularity at 1 + 2 i g and
// converge as rho'^-2n with 2 n nodes.  The first needs fewer nodes but next to
// the origin (5 against 8 per dimension at 64 cells, 3 against 6 at 1000);
// cells far from cubes leave a small g beside the origin, where its order
// passes the tables' and the second is taken.  Error target 1e-17.
struct Rule {
    int n;
    const double *t, *w;
};
__device__ static Rule rule_for(double ox, double oy, double oz, double a, double b, double c,
                                const double *gl)
{
    const double gx = fabs(ox) > 1.0 ? (fabs(ox) - 1.0) * a : 0.0;
    const double gy = fabs(oy) > 1.0 ? (fabs(oy) - 1.0) * b : 0.0;
    const double gz = fabs(oz) > 1.0 ? (fabs(oz) - 1.0) * c : 0.0;
    const double g = sqrt(gx * gx + gy * gy + gz * gz) / fmax(a, fmax(b, c));
    const double m = ceil(39.14 / (2.0 * log(g + sqrt(1.0 + g * g))));
    if (m < (double)GL_MAXN) {
        const int n = m < 3.0 ? 3 : (int)m;
        return {n, gl + n * GL_MAXN, gl + (GL_MAXN + n) * GL_MAXN};
    }
    // rho' = |z + sqrt(z^2 - 1)|, z = 1 + 2 i g
    const double wr = -4.0 * g * g, wi = 4.0 * g;
    const double mod = sqrt(sqrt(wr * wr + wi * wi)), ang = 0.5 * atan2(wi, wr);
    const double sr = mod * cos(ang), si = mod * sin(ang);
    const double rho = fmax(hypot(1.0 + sr, 2.0 * g + si), hypot(1.0 - sr, 2.0 * g - si));
    const double h = ceil(39.14 / (2.0 * log(rho)));
    const int n = h > GL_MAXN - 1.0 ? GL_MAXN - 1 : (int)h;
    const double *half = gl + GL_HALF + n * 2 * GL_MAXN;
    return {2 * n, half, half + GL_MAXN * 2 * GL_MAXN};
}

// Nodes (ia, ib) x all z nodes of an n-point rule, added to the six sums:
// with w3, w5, z1, z2 = sum over the z nodes of w r^-3, w r^-5, w z r^-5 and
// w z^2 r^-5, the entries of the column are w3 - 3 x^2 w5, -3 x y w5, ...
__device__ __forceinline__ void tent_column(double rx, double ry, double wxy, double Z, double c,
                                            int n, const double *__restrict__ t,
                                            const double *__restrict__ w, double (&acc)[6])
{
    const double rxy = rx * rx + ry * ry;
    double w3 = 0.0, w5 = 0.0, z1 = 0.0, z2 = 0.0;
    for (int ic = 0; ic < n; ++ic) {
        const double rz = Z + c * t[ic];
        const double r2 = rxy + rz * rz;
        const double ir = rsqrt(r2), ir2 = ir * ir;
        const double u3 = w[ic] * ir * ir2, u5 = u3 * ir2;
        w3 += u3;
        w5 += u5;
        z1 += u5 * rz;
        z2 += u5 * rz * rz;
    }
    acc[0] += wxy * (w3 - 3.0 * rx * rx * w5);
    acc[1] += wxy * (w3 - 3.0 * ry * ry * w5);
    acc[2] += wxy * (w3 - 3.0 * z2);
    acc[3] -= wxy * 3.0 * rx * ry * w5;
    acc[4] -= wxy * 3.0 * rx * z1;
    acc[5] -= wxy * 3.0 * ry * z1;
}

struct DimImages {
    int periodic, N, M, mimg;
    int K;              // offsets of the octant: N (open), N / 2 + 1 (periodic)
    int nimg;           // images of one offset: 1 (open), 2 mimg + 2 (periodic)
};

// offset of image m (0 .. nimg - 1) of octant position p, and its weight
// (0: outside the window)
__device__ __forceinline__ double dim_offset(const DimImages &d, int p, int m, double &wgt)
{
    wgt = 1.0;
    if (!d.periodic) return (double)p;
    const double o = (double)p + (double)(m - d.mimg - 1) * d.N;
    const double lim = (d.mimg + 0.5) * d.N, ao = fabs(o);
    if (ao > lim) wgt = 0.0;
    else if (ao == lim) wgt = 0.5;
    return o;
}

// One octant position per thread (PER = 1: a single image) or per wave (PER =
// 64: the lanes share its images).  A lane evaluates the entries that need at
// most SERIAL nodes per dimension by itself; the whole wave shares the nodes
// of every larger one and the closed form's 27 terms of six components, one
// entry after the other.  Without that split the entries next to the origin
// (12,167 nodes, or 162 closed-form terms) are a serial chain in one thread,
// which alone took 6 to 9 ms however small the grid.  Measured with the
// octant and the tent rule against one thread per padded position: 64x64x16
// film with 81 images 21.7 -> 0.43 ms, 128x128x32 film with 1089 images
// 698 -> 10.6 ms, 256x256x64 box 43.6 -> 0.61 ms.
template <int PER>
__global__ void __launch_bounds__(256)
    k_tensor_octant_real(DimImages dx_, DimImages dy_, DimImages dz_, double a, double b,
                         double c, const double *__restrict__ gl, double *__restrict__ O)
{
    constexpr int SERIAL = 6;
    const long long total = (long long)dx_.K * dy_.K * dz_.K;
    const int lane = threadIdx.x & 63;
    const long long gid = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const long long pos = PER == 1 ? gid : gid / 64;
    const bool act = pos < total;
    const long long pc = act ? pos : 0;
    const int ix = (int)(pc % dx_.K);
    const int iy = (int)((pc / dx_.K) % dy_.K);
    const int iz = (int)(pc / ((long long)dx_.K * dy_.K));
    const int nimg = dx_.nimg * dy_.nimg * dz_.nimg;
    double acc[6] = {0, 0, 0, 0, 0, 0};
    for (int i0 = 0; i0 < nimg; i0 += PER) {
        const int img = PER == 1 ? i0 : i0 + lane;
        const int jx = img % dx_.nimg, jy = img / dx_.nimg % dy_.nimg;
        const int jz = img / (dx_.nimg * dy_.nimg);
        double wx = 0.0, wy = 0.0, wz = 0.0, ox = 0.0, oy = 0.0, oz = 0.0;
        if (act && img < nimg) {
            ox = dim_offset(dx_, ix, jx, wx);
            oy = dim_offset(dy_, iy, jy, wy);
            oz = dim_offset(dz_, iz, jz, wz);
        }
        const double wgt = wx * wy * wz;
        const bool near = fabs(ox) <= 1.0 && fabs(oy) <= 1.0 && fabs(oz) <= 1.0;
        const Rule r = near ? Rule{0, gl, gl} : rule_for(ox, oy, oz, a, b, c, gl);
        const int n = r.n;
        const double pref = wgt * a * b * c / (4.0 * M_PI);
        if (wgt != 0.0 && !near && n <= SERIAL) {
            const double *t = r.t, *w = r.w;
            double s[6] = {0, 0, 0, 0, 0, 0};
            for (int ia = 0; ia < n; ++ia)
                for (int ib = 0; ib < n; ++ib)
                    tent_column(ox * a + a * t[ia], oy * b + b * t[ib], w[ia] * w[ib], oz * c, c,
                                n, t, w, s);
            for (int q = 0; q < 6; ++q) acc[q] += pref * s[q];
        }
        // the entries left over, one at a time with the whole wave
        unsigned long long todo = __ballot(wgt != 0.0 && (near || n > SERIAL));
        while (todo) {
            const int src = __ffsll(todo) - 1;
            todo &= todo - 1;
            const double X = __shfl(ox, src, 64) * a, Y = __shfl(oy, src, 64) * b,
                         Z = __shfl(oz, src, 64) * c;
            const int ns = __shfl(n, src, 64);
            double s[6] = {0, 0, 0, 0, 0, 0};
            if (ns == 0) {
                const double R[3] = {X, Y, Z}, d[3] = {a, b, c};
                for (int e = lane; e < 162; e += 64) {
                    const double v = newell_term(e, R, d);
                    for (int k = 0; k < 6; ++k) s[k] += k == e / 27 ? v : 0.0;
                }
            } else {
                const double *t = gl + __shfl((int)(r.t - gl), src, 64);
                const double *w = gl + __shfl((int)(r.w - gl), src, 64);
                for (int e = lane; e < ns * ns; e += 64) {
                    const int ia = e / ns, ib = e - ia * ns;
                    tent_column(X + a * t[ia], Y + b * t[ib], w[ia] * w[ib], Z, c, ns, t, w, s);
                }
            }
            const double scale = ns == 0 ? __shfl(wgt, src, 64) * -1.0 / (4.0 * M_PI * a * b * c)
                                         : __shfl(pref, src, 64);
            for (int q = 0; q < 6; ++q) {
                double v = s[q];
                for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
                if (lane == src) acc[q] += scale * v;
            }
        }
    }
    for (int q = 0; q < 6; ++q) {
        double v = acc[q];
        if (PER == 64) {
            for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
        }
        if (act && (PER == 1 || lane == 0)) O[q * total + pos] = v;
    }
}

// octant index of padded position p along one dimension (-1 in the zero gap of
// an open one) and whether it is a mirror image
__device__ __forceinline__ int octant_index(const DimImages &d, int p, bool &mirror)
{
    mirror = false;
    if (p < d.K) return p;
    const int o = d.M - p;
    mirror = true;
    return o < d.K ? o : -1;
}

// R[q][iz][iy][ix] on the padded grid from the octant: xy is odd in x and y,
// xz in x and z, yz in y and z
__global__ void k_tensor_expand(Geom g, DimImages dx_, DimImages dy_, DimImages dz_,
                                const double *__restrict__ O, double *__restrict__ R)
{
    const long long total = (long long)g.mx * g.my * g.mz;
    const long long octant = (long long)dx_.K * dy_.K * dz_.K;
    const long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= total) return;
    bool fx, fy, fz;
    const int ix = octant_index(dx_, (int)(idx % g.mx), fx);
    const int iy = octant_index(dy_, (int)((idx / g.mx) % g.my), fy);
    const int iz = octant_index(dz_, (int)(idx / ((long long)g.mx * g.my)), fz);
    const bool in = ix >= 0 && iy >= 0 && iz >= 0;
    const long long src = in ? ((long long)iz * dy_.K + iy) * dx_.K + ix : 0;
    for (int q = 0; q < 6; ++q) {
        const bool neg = q == 3 ? fx != fy : (q == 4 ? fx != fz : (q == 5 ? fy != fz : false));
        const double v = in ? O[q * octant + src] : 0.0;
        R[q * total + idx] = neg ? -v : v;
    }
}

size_t tensor_octant_bytes(const Geom &g)
{
    const size_t kx = g.px ? g.nx / 2 + 1 : g.nx, ky = g.py ? g.ny / 2 + 1 : g.ny,
                 kz = g.pz ? g.nz / 2 + 1 : g.nz;
    return 6 * kx * ky * kz * sizeof(double);
}

hipError_t launch_tensor_real(const Geom &g, int mimg, double dx, double dy, double dz,
                              const double *gl, double *octant, double *R, hipStream_t s)
{
    auto dim = [&](int per, int N, int M) {
        return DimImages{per, N, M, mimg, per ? N / 2 + 1 : N, per ? 2 * mimg + 2 : 1};
    };
    const DimImages ix = dim(g.px, g.nx, g.mx), iy = dim(g.py, g.ny, g.my),
                    iz = dim(g.pz, g.nz, g.mz);
    const long long noct = (long long)ix.K * iy.K * iz.K;
    const long long total = (long long)g.mx * g.my * g.mz;
    const bool images = ix.nimg * iy.nimg * iz.nimg > 1;
    const long long blocks = images ? (noct + 3) / 4 : (noct + 255) / 256;
    if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    if (images)
        hipLaunchKernelGGL((k_tensor_octant_real<64>), dim3((unsigned)blocks), dim3(256), 0, s,
                           ix, iy, iz, dx, dy, dz, gl, octant);
    else
        hipLaunchKernelGGL((k_tensor_octant_real<1>), dim3((unsigned)blocks), dim3(256), 0, s,
                           ix, iy, iz, dx, dy, dz, gl, octant);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_tensor_expand, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, g,
                       ix, iy, iz, octant, R);
    return hipGetLastError();
}

// In-plane k = 0 correction.  Film (pmask 3): one block per (component, z
// position); fully periodic (pmask 7): one block per component.
__global__ void k_tensor_k0(Geom g, int full, double *R)
{
    __shared__ double red[256];
    const int q = blockIdx.y;
    const long long total = (long long)g.mx * g.my * g.mz;
    const int tid = threadIdx.x;
    long long start, count;
    double target;
    if (full) {
        start = 0;
        count = total;
        target = 0.0;
    } else {
        const int iz = blockIdx.x;
        // open z: positions in the zero gap hold no offset
        if (iz >= g.nz && iz <= g.mz - g.nz) return;
        const int dz = iz < g.nz ? iz : iz - g.mz;
        start = (long long)iz * g.mx * g.my;
        count = (long long)g.mx * g.my;
        target = (q == 2 && dz == 0) ? 1.0 : 0.0;
    }
    double *p = R + q * total + start;
    double s = 0.0;
    for (long long i = tid; i < count; i += 256) s += p[i];
    red[tid] = s;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (tid < w) red[tid] += red[tid + w];
        __syncthreads();
    }
    const double corr = (target - red[0]) / (double)count;
    for (long long i = tid; i < count; i += 256) p[i] += corr;
}

hipError_t launch_tensor_k0(const Geom &g, unsigned pmask, double *R, double *sums,
                            hipStream_t s)
{
    (void)sums;
    if (pmask == 3u)
        hipLaunchKernelGGL(k_tensor_k0, dim3(g.mz, 6), dim3(256), 0, s, g, 0, R);
    else if (pmask == 7u)
        hipLaunchKernelGGL(k_tensor_k0, dim3(1, 6), dim3(256), 0, s, g, 1, R);
    else
        return hipSuccess;
    return hipGetLastError();
}

// Octant of the real spectrum, scaled:
//   Nt(kx, q, kz, ky) = scale * Re C[kx][q][kz][ky],  kz <= mz/2, ky <= my/2,
// from the full spectrum C[kx][q][mz][my], stored in blocks of KB kx:
// Nt(kx, q, kz, ky) at (((kx/KB)*6 + q)*(mz/2+1) + kz)*(my/2+1) + ky)*KB + kx%KB.
template <typename T>
__global__ void k_tensor_octant(Geom g, const cpx<double> *__restrict__ C, double scale,
                                T *__restrict__ Nt)
{
    const int hy = g.my / 2 + 1, hz = g.mz / 2 + 1;
    const long long total = (long long)g.hx * 6 * hz * hy;
    const long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= total) return;
    const int ky = (int)(idx % hy);
    const int kz = (int)((idx / hy) % hz);
    const long long kq = idx / ((long long)hy * hz);      // kx*6 + q
    const long long src = (kq * g.mz + kz) * g.my + ky;
    // stored in blocks of KB kx, as the spectra that it multiplies
    const long long kx = kq / 6, q = kq - kx * 6;
    const long long dst = ((((kx >> KBS) * 6 + q) * hz + kz) * hy + ky) * KB + (kx & (KB - 1));
    Nt[dst] = (T)(scale * C[src].x);
}

hipError_t launch_tensor_octant(int prec, const Geom &g, const void *C, double scale, void *Nt,
                                hipStream_t s)
{
    const long long total = (long long)g.hx * 6 * (g.mz / 2 + 1) * (g.my / 2 + 1);
    const long long blocks = (total + 255) / 256;
    if (prec == PREC_F32)
        hipLaunchKernelGGL((k_tensor_octant<float>), dim3((unsigned)blocks), dim3(256), 0, s, g,
                           (const cpx<double> *)C, scale, (float *)Nt);
    else
        hipLaunchKernelGGL((k_tensor_octant<double>), dim3((unsigned)blocks), dim3(256), 0, s,
                           g, (const cpx<double> *)C, scale, (double *)Nt);
    return hipGetLastError();
}

}  // namespace tdgl
