// One colour sweep of the Schwarz alternating procedure: every Schwarz block
// of the given colour computes its residual r = (rho - D psi)|_Lambda with the
// full operator, runs nmr minimal-residual steps on the block operator
// D_Lambda (Dirichlet walls) and adds the block solution to psi.
//
// Mapping: one workgroup per Schwarz block. The residual reads the neighbour
// spinors across the block faces directly from global memory; those sites
// belong to blocks of the other colour, which no workgroup of this launch
// writes, so there is no race. Inside the MR loop the current residue r is
// exchanged through LDS (12 planes x |block|), and the block reductions of a
// step use DPP wavefront sums plus one LDS pass. Every kernel keeps the links on
// the chip for the MR steps (spare lanes of the last wavefront only join the
// reductions), the first three as the residue has read them:
//   k_sap_rl    FP32, one lane per site
//   k_sap_cl    the same with the clover term or antiperiodic time
//   k_sap_pair  two lanes per site: FP64 blocks of up to 256 sites, and FP32
//               single fields on lattices with few blocks
//   k_sap_big   FP64 blocks of 257..512 sites, one lane per site and link
//
// init (first cycle, where psi starts at zero): 2 = psi is zero everywhere
// (colour 0: the residue is rho, no hops, no reads of psi), 1 = psi is zero on
// the sweep's own blocks (colour 1: only the neighbours' values are read).
// out64 (optional, last cycle of an FP32 sweep): the block's new psi is also
// written in FP64 there, so no conversion pass follows.
#include <type_traits>

#include "hop.h"

namespace dfl {

namespace {

// factor of field b's rho when it enters scaled: 1 / sqrt(nrm2[2 b]) (0 for
// a zero field), 1 without nrm2
template <typename T> __device__ inline T rho_scale(const double* nrm2, int b)
{
    if (!nrm2)
        return T(1);
    const double q = nrm2[2 * b];
    return q > 0.0 ? (T)(1.0 / sqrt(q)) : T(0);
}
template <typename T> __device__ inline void scale_spinor(spinor<T>& p, T f)
{
#pragma unroll
    for (int al = 0; al < 4; ++al)
#pragma unroll
        for (int a = 0; a < 3; ++a)
            p.s[al].c[a] = cpx<T>{p.s[al].c[a].re * f, p.s[al].c[a].im * f};
}

// (q, r) and ||q||^2 of the block from every lane's shares, in a fixed order;
// NW: wavefronts of the workgroup (0: nw, at run time). red: LDS.
template <int NW>
__device__ inline void block_products(double& re, double& im, double& qq, double (*red)[8], int lane, int wid, int nw)
{
    re = wave_sum(re);
    im = wave_sum(im);
    qq = wave_sum(qq);
    if (lane == 0) {
        red[0][wid] = re;
        red[1][wid] = im;
        red[2][wid] = qq;
    }
    __syncthreads();
    re = im = qq = 0.0;
    if (NW > 0) {
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            re += red[0][w];
            im += red[1][w];
            qq += red[2][w];
        }
    } else {
        for (int w = 0; w < nw; ++w) {
            re += red[0][w];
            im += red[1][w];
            qq += red[2][w];
        }
    }
}

template <typename T> __device__ inline void store_spinor_f64(c64* __restrict__ f, long V, long s, const spinor<T>& p)
{
    spinor<double> d;
#pragma unroll
    for (int al = 0; al < 4; ++al)
#pragma unroll
        for (int a = 0; a < 3; ++a)
            d.s[al].c[a] = c64{(double)p.s[al].c[a].re, (double)p.s[al].c[a].im};
    store_spinor(f, V, s, d);
}

// the eight hops of the full operator at one site, neighbours from global
// memory; with outside_only, only the hops that leave the Schwarz block (the
// block's own psi is zero in the first cycle's colour-1 sweep)
template <typename T, typename L>
__device__ inline void full_hops(const Geom& g, const SapGeom& sg, const L& U, const cpx<T>* __restrict__ psi, long s,
                                 const int n[4], const int y[4], const int yl[4], bool outside_only, spinor<T>& acc)
{
#pragma unroll 1
    for (int h = 0; h < 8; ++h) {
        const int mu = h >> 1;
        const int step = (h & 1) ? -1 : +1;
        if (outside_only && (step > 0 ? yl[mu] + 1 < sg.sb[mu] : yl[mu] > 0))
            continue;
        long tn = site_step(g, s, n, y, mu, step);
        spinor<T> p = load_spinor(psi, g.V, tn);
        if (crosses_time(g, n, y, mu, step))
            negate(p);
        if (step > 0)
            hop_fwd_rt(mu, load_link(U, mu, s), p, acc);
        else
            hop_bwd_rt(mu, load_link(U, mu, tn), p, acc);
    }
}

// FP32 sweep for several fields with the site's eight links kept for the MR
// steps: the first two rows in registers (96 VGPRs), the third row, formed
// once during the residual, in LDS (24 planes x block). The MR steps then read
// only LDS, and two blocks of up to 256 sites share a CU (2 x 72 KB of LDS).
template <typename L> struct Link2 {
    c32 e[6];
};

template <typename L> __device__ inline Link2<L> load_link2(const L& U, int mu, long s);
template <> __device__ inline Link2<Links32> load_link2(const Links32& U, int mu, long s)
{
    Link2<Links32> r;
#pragma unroll
    for (int k = 0; k < 6; ++k)
        r.e[k] = ld(U.u, toff<c32>(s, mu * 6 + k, 24));
    return r;
}
template <> __device__ inline Link2<LinksBF16> load_link2(const LinksBF16& U, int mu, long s)
{
    Link2<LinksBF16> r;
#pragma unroll
    for (int k = 0; k < 6; ++k) {
        uint32_t w = ld(U.u, toff<uint32_t>(s, mu * 6 + k, 24));
        r.e[k] = c32{bf16_to_f(w & 0xffffu), bf16_to_f(w >> 16)};
    }
    return r;
}
template <typename L> __device__ inline su3<float> expand(const Link2<L>& l)
{
    su3<float> u;
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 3; ++b)
            u.m[a][b] = l.e[a * 3 + b];
    complete_third_row(u);
    return u;
}

// Makes v's value unknown to the compiler at this point, so that what is computed
// from it inside a loop is not moved out of the loop (and then spilled).
template <typename T> __device__ inline void pin(cpx<T>& v) { asm volatile("" : "+v"(v.re), "+v"(v.im)); }

// the link from its two register rows and its third row in LDS (entry b at l3[b * stride])
template <typename L> __device__ inline su3<float> expand_lds(const Link2<L>& l, const c32* l3, int stride)
{
    su3<float> u;
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 3; ++b)
            u.m[a][b] = l.e[a * 3 + b];
#pragma unroll
    for (int b = 0; b < 3; ++b)
        u.m[2][b] = l3[b * stride];
    return u;
}

// B4: 4^4 blocks, whose extents, in-block strides and LDS plane size are
// compile-time constants (every LDS access of a hop is then an immediate
// offset from the thread's own address). WIDE: antiperiodic time, blocks of
// 257..512 sites (one per CU); the lanes' products are summed in FP64, the block
// hops by themselves.
template <typename L, bool B4, bool WIDE>
__global__ __launch_bounds__(WIDE && !B4 ? 512 : 256, 2) void k_sap_rl(Geom g, SapGeom sg, L U, const c32* __restrict__ rho,
                                                                      const double* __restrict__ rho_nrm2,
                                                                      c32* __restrict__ psi, float diag, int nmr,
                                                                      int colour, int nrhs, int init,
                                                                      c64* __restrict__ out64)
{
    const int Vsb = B4 ? 256 : sg.Vsb;
    int sbl[4], lst[4];
#pragma unroll
    for (int mu = 0; mu < 4; ++mu) {
        sbl[mu] = B4 ? 4 : sg.sb[mu];
        lst[mu] = B4 ? (64 >> (2 * mu)) : sg.lstr[mu];
    }
    // workgroup -> (block of this colour, right-hand side), right-hand sides fastest
    const float rs = rho_scale<float>(rho_nrm2, blockIdx.x % nrhs);
    rho += (long)(blockIdx.x % nrhs) * 12 * g.V;
    psi += (long)(blockIdx.x % nrhs) * 12 * g.V;
    if (out64)
        out64 += (long)(blockIdx.x % nrhs) * 12 * g.V;
    extern __shared__ char smem_raw[];
    c32* lr = reinterpret_cast<c32*>(smem_raw);
    c32* l3 = lr + 12 * Vsb;  // third link rows: entry (3 h + b) * Vsb + site
    __shared__ double red[3][8];

    const int t = threadIdx.x;
    const bool active = t < Vsb;
    const int lane = t & 63, wid = t >> 6, nw = blockDim.x >> 6;

    int k = blockIdx.x / nrhs;
    int half = sg.nsb[3] / 2;
    int m[4];
    int j = k % half;
    int rest = k / half;
    m[2] = rest % sg.nsb[2];
    rest /= sg.nsb[2];
    m[1] = rest % sg.nsb[1];
    m[0] = rest / sg.nsb[1];
    m[3] = 2 * j + ((colour + m[0] + m[1] + m[2]) & 1);

    int yl[4] = {0, 0, 0, 0};
    int n[4] = {0, 0, 0, 0}, y[4] = {0, 0, 0, 0};
    long s = 0;
    if (active) {
        int tt = t;
        yl[3] = tt % sbl[3];
        tt /= sbl[3];
        yl[2] = tt % sbl[2];
        tt /= sbl[2];
        yl[1] = tt % sbl[1];
        yl[0] = tt / sbl[1];
        for (int mu = 0; mu < 4; ++mu) {
            int x = m[mu] * sbl[mu] + yl[mu];
            n[mu] = x / g.b[mu];
            y[mu] = x - n[mu] * g.b[mu];
        }
        s = site_compose(g, n, y);
    }

    // residual with the full operator; the links are kept for the MR steps
    Link2<L> lk[8];
    spinor<float> r, xs;
    zero(r);
    zero(xs);
    if (active) {
        spinor<float> acc, self;
        zero(acc);
        zero(self);
#pragma unroll
        for (int h = 0; h < 8; ++h) {
            const int mu = h >> 1;
            const int step = (h & 1) ? -1 : +1;
            long tn = site_step(g, s, n, y, mu, step);
            lk[h] = load_link2(U, mu, step > 0 ? s : tn);
            const su3<float> u = expand(lk[h]);
#pragma unroll
            for (int b = 0; b < 3; ++b)
                l3[(3 * h + b) * Vsb + t] = u.m[2][b];
            const bool inside = step > 0 ? yl[mu] + 1 < sbl[mu] : yl[mu] > 0;
            if (init == 0 || (init == 1 && !inside)) {
                spinor<float> p = load_spinor(psi, g.V, tn);
                if (WIDE && mu == 0 && crosses_time(g, n, y, mu, step))
                    negate(p);
                if (step > 0)
                    hop_fwd_rt(mu, u, p, acc);
                else
                    hop_bwd_rt(mu, u, p, acc);
            }
            if (h & 1)
                asm volatile("" ::: "memory");  // two hops' loads in flight at a time
        }
        if (init == 0)
            self = load_spinor(psi, g.V, s);
        spinor<float> d = finish(self, acc, diag);
        spinor<float> b = load_spinor(rho, g.V, s);
        if (rho_nrm2)
            scale_spinor(b, rs);
#pragma unroll
        for (int al = 0; al < 4; ++al)
            r.s[al] = b.s[al] - d.s[al];
    }

    for (int stp = 0; stp < nmr; ++stp) {
        if (active) {
#pragma unroll
            for (int al = 0; al < 4; ++al)
#pragma unroll
                for (int a = 0; a < 3; ++a)
                    lr[(3 * al + a) * Vsb + t] = r.s[al].c[a];
        }
        // acc = -2 D_Lambda r: it starts at -2 diag r (WIDE: ends with it, the hops are
        // summed by themselves) and collects the inside hops, so the MR coefficient
        // follows from it without forming D_Lambda r
        spinor<float> acc;
        zero(acc);
        auto add_diag = [&] {
#pragma unroll
            for (int al = 0; al < 4; ++al)
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    acc.s[al].c[a].re = fmadd(-2.0f * diag, r.s[al].c[a].re, acc.s[al].c[a].re);
                    acc.s[al].c[a].im = fmadd(-2.0f * diag, r.s[al].c[a].im, acc.s[al].c[a].im);
                }
        };
        if (active && !WIDE)
            add_diag();
        __syncthreads();
        // the lane's products, then the block sums in FP64
        using S = std::conditional_t<WIDE, double, float>;
        S fr_re = 0, fr_im = 0, fqq = 0;
        if (active) {
#pragma unroll
            for (int h = 0; h < 8; ++h) {
                const int mu = h >> 1;
                const int step = (h & 1) ? -1 : +1;
                if (step > 0 ? yl[mu] + 1 < sbl[mu] : yl[mu] > 0) {
                    const int tn = t + step * lst[mu];
                    spinor<float> p;
#pragma unroll
                    for (int al = 0; al < 4; ++al)
#pragma unroll
                        for (int a = 0; a < 3; ++a)
                            p.s[al].c[a] = lr[(3 * al + a) * Vsb + tn];
                    const su3<float> u = expand_lds(lk[h], l3 + 3 * h * Vsb + t, Vsb);
                    if (step > 0)
                        hop_fwd_rt(mu, u, p, acc);
                    else
                        hop_bwd_rt(mu, u, p, acc);
                }
                if (h & 1)
                    asm volatile("" ::: "memory");
            }
            if (WIDE)
                add_diag();
#pragma unroll
            for (int al = 0; al < 4; ++al)
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    const S qa = acc.s[al].c[a].re, qb = acc.s[al].c[a].im;
                    const S ra = r.s[al].c[a].re, rb = r.s[al].c[a].im;
                    fr_re = fmadd(qb, rb, fmadd(qa, ra, fr_re));
                    fr_im = fmadd(-qb, ra, fmadd(qa, rb, fr_im));
                    fqq = fmadd(qb, qb, fmadd(qa, qa, fqq));
                }
        }
        double sre = fr_re, sim = fr_im, sqq = fqq;
        block_products<B4 ? 4 : 0>(sre, sim, sqq, red, lane, wid, nw);
        if (!(sqq > 0.0))
            break;  // zero residue on this block: uniform across the workgroup
        // with q = D_Lambda r = -acc / 2: alpha = (q, r) / ||q||^2 = -2 (acc, r) / ||acc||^2,
        // x += alpha r, r -= alpha q = r + (alpha / 2) acc
        const c32 alpha{(float)(-2.0 * sre / sqq), (float)(-2.0 * sim / sqq)};
        const c32 half{0.5f * alpha.re, 0.5f * alpha.im};
#pragma unroll
        for (int al = 0; al < 4; ++al)
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                xs.s[al].c[a] = cfma(alpha, r.s[al].c[a], xs.s[al].c[a]);
                r.s[al].c[a] = cfma(half, acc.s[al].c[a], r.s[al].c[a]);
            }
    }

    if (active) {
        spinor<float> p;
        zero(p);
        if (init == 0)
            p = load_spinor(psi, g.V, s);
#pragma unroll
        for (int al = 0; al < 4; ++al)
            p.s[al] += xs.s[al];
        store_spinor(psi, g.V, s, p);
        if (out64)
            store_spinor_f64(out64, g.V, s, p);
    }
}

// The same with the clover term. Beside the links the 36
// clover entries of a site fit neither registers nor LDS, and re-reading them
// at every MR step is paid in exposed latency (192 us per sweep of one field on
// 48 x 24^3, 95 without the term). So the residue lives in LDS alone, the block
// solution too, the third link rows are rebuilt for every use, and of every
// chirality block's entries kLC are in LDS, the others in registers: one read
// of everything per sweep, two blocks of 256 sites per CU: 145 us.
constexpr int kLC = 5;  // LDS entries of a chirality block (of 18)
template <typename L, bool B4>
__global__ __launch_bounds__(B4 ? 256 : 512, 2) void k_sap_cl(Geom g, SapGeom sg, L U, const c32* __restrict__ rho,
                                                              const double* __restrict__ rho_nrm2,
                                                              c32* __restrict__ psi, float diag, int nmr, int colour,
                                                              int nrhs, int init, c64* __restrict__ out64,
                                                              Clover<float> C)
{
    const int Vsb = B4 ? 256 : sg.Vsb;
    int sbl[4], lst[4];
#pragma unroll
    for (int mu = 0; mu < 4; ++mu) {
        sbl[mu] = B4 ? 4 : sg.sb[mu];
        lst[mu] = B4 ? (64 >> (2 * mu)) : sg.lstr[mu];
    }
    // workgroup -> (block of this colour, right-hand side), right-hand sides fastest
    const float rs = rho_scale<float>(rho_nrm2, blockIdx.x % nrhs);
    rho += (long)(blockIdx.x % nrhs) * 12 * g.V;
    psi += (long)(blockIdx.x % nrhs) * 12 * g.V;
    if (out64)
        out64 += (long)(blockIdx.x % nrhs) * 12 * g.V;
    extern __shared__ char smem_raw[];
    c32* lr = reinterpret_cast<c32*>(smem_raw);  // residue
    c32* lx = lr + 12 * Vsb;                     // block solution
    c32* lc = lx + 12 * Vsb;                     // clover entries, (kLC h + q) * Vsb + site
    __shared__ double red[3][8];

    const int t = threadIdx.x;
    const bool active = t < Vsb;
    const int lane = t & 63, wid = t >> 6, nw = blockDim.x >> 6;

    int k = blockIdx.x / nrhs;
    int half = sg.nsb[3] / 2;
    int m[4];
    int j = k % half;
    int rest = k / half;
    m[2] = rest % sg.nsb[2];
    rest /= sg.nsb[2];
    m[1] = rest % sg.nsb[1];
    m[0] = rest / sg.nsb[1];
    m[3] = 2 * j + ((colour + m[0] + m[1] + m[2]) & 1);

    int yl[4] = {0, 0, 0, 0};
    int n[4] = {0, 0, 0, 0}, y[4] = {0, 0, 0, 0};
    long s = 0;
    if (active) {
        int tt = t;
        yl[3] = tt % sbl[3];
        tt /= sbl[3];
        yl[2] = tt % sbl[2];
        tt /= sbl[2];
        yl[1] = tt % sbl[1];
        yl[0] = tt / sbl[1];
        for (int mu = 0; mu < 4; ++mu) {
            int x = m[mu] * sbl[mu] + yl[mu];
            n[mu] = x / g.b[mu];
            y[mu] = x - n[mu] * g.b[mu];
        }
        s = site_compose(g, n, y);
    }
    c32 cl[2][18 - kLC];
    // o += f C p at this site for the p with component (3 * spin + colour) p(c); C p
    // is summed by itself (o is the larger part)
    auto site_clover = [&](int Vsb, float f, const auto& p, spinor<float>& o) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            c32 e[18], v[6], w[6];
#pragma unroll
            for (int q = 0; q < 18; ++q)
                e[q] = q < kLC ? lc[(kLC * h + q) * Vsb + t] : cl[h][q < kLC ? 0 : q - kLC];
#pragma unroll
            for (int i = 0; i < 6; ++i) {
                v[i] = f * p(6 * h + i);
                w[i] = c32{0.0f, 0.0f};
            }
            clover_mul(e, v, w);
#pragma unroll
            for (int i = 0; i < 6; ++i)
                o.s[2 * h + i / 3].c[i % 3] += w[i];
            asm volatile("" ::: "memory");
        }
    };

    // residual with the full operator; the links are kept for the MR steps
    Link2<L> lk[8];
    if (active) {
        spinor<float> acc, self;
        zero(acc);
        zero(self);
#pragma unroll
        for (int h = 0; h < 8; ++h) {
            const int mu = h >> 1;
            const int step = (h & 1) ? -1 : +1;
            long tn = site_step(g, s, n, y, mu, step);
            lk[h] = load_link2(U, mu, step > 0 ? s : tn);
            const bool inside = step > 0 ? yl[mu] + 1 < sbl[mu] : yl[mu] > 0;
            if (init == 0 || (init == 1 && !inside)) {
                spinor<float> p = load_spinor(psi, g.V, tn);
                if (mu == 0 && crosses_time(g, n, y, mu, step))
                    negate(p);
                if (step > 0)
                    hop_fwd_rt(mu, expand(lk[h]), p, acc);
                else
                    hop_bwd_rt(mu, expand(lk[h]), p, acc);
            }
            if (h & 1)
                asm volatile("" ::: "memory");  // two hops' loads in flight at a time
        }
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int q = 0; q < 18; ++q) {
                const c32 e = ld(C.c, toff<c32>(s, 18 * h + q, kCloverComp));
                if (q < kLC)
                    lc[(kLC * h + q) * Vsb + t] = e;
                else
                    cl[h][q < kLC ? 0 : q - kLC] = e;
            }
        if (init == 0)
            self = load_spinor(psi, g.V, s);
        spinor<float> d = finish(self, acc, diag);
        if (init == 0)
            site_clover(Vsb, 1.0f, [&](int c) { return self.s[c / 3].c[c % 3]; }, d);
        spinor<float> b = load_spinor(rho, g.V, s);
        if (rho_nrm2)
            scale_spinor(b, rs);
#pragma unroll
        for (int al = 0; al < 4; ++al)
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                lr[(3 * al + a) * Vsb + t] = b.s[al].c[a] - d.s[al].c[a];
                lx[(3 * al + a) * Vsb + t] = c32{0.0f, 0.0f};
            }
    }

    const int V0 = Vsb;
    for (int stp = 0; stp < nmr; ++stp) {
        // (unknown to the compiler here: addresses are formed in the step, not kept over all of them)
        int Vsb = V0;
        if (!B4)
            asm volatile("" : "+s"(Vsb));
        // acc = -2 D_Lambda r: the inside hops, then -2 (diag + C) r; the MR
        // coefficient follows from it without forming D_Lambda r
        spinor<float> acc;
        zero(acc);
        __syncthreads();
        double sre = 0.0, sim = 0.0, sqq = 0.0;  // (squares of FP32 entries would leave FP32's range)
        if (active) {
#pragma unroll
            for (int h = 0; h < 8; ++h) {
                const int mu = h >> 1;
                const int step = (h & 1) ? -1 : +1;
                if (step > 0 ? yl[mu] + 1 < sbl[mu] : yl[mu] > 0) {
                    const int tn = t + step * lst[mu];
                    spinor<float> p;
#pragma unroll
                    for (int al = 0; al < 4; ++al)
#pragma unroll
                        for (int a = 0; a < 3; ++a)
                            p.s[al].c[a] = lr[(3 * al + a) * Vsb + tn];
                    pin(lk[h].e[0]);
                    pin(lk[h].e[1]);
                    pin(lk[h].e[2]);
                    if (step > 0)
                        hop_fwd_rt(mu, expand(lk[h]), p, acc);
                    else
                        hop_bwd_rt(mu, expand(lk[h]), p, acc);
                }
                asm volatile("" ::: "memory");
            }
            const c32* own = lr + t;
#pragma unroll
            for (int al = 0; al < 4; ++al)
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    const c32 r = own[(3 * al + a) * Vsb];
                    acc.s[al].c[a].re = fmadd(-2.0f * diag, r.re, acc.s[al].c[a].re);
                    acc.s[al].c[a].im = fmadd(-2.0f * diag, r.im, acc.s[al].c[a].im);
                }
            site_clover(Vsb, -2.0f, [&](int c) { return own[c * Vsb]; }, acc);
#pragma unroll
            for (int al = 0; al < 4; ++al)
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    const double qa = acc.s[al].c[a].re, qb = acc.s[al].c[a].im;
                    const c32 r = lr[(3 * al + a) * Vsb + t];
                    const double ra = r.re, rb = r.im;
                    sre = fmadd(qb, rb, fmadd(qa, ra, sre));
                    sim = fmadd(-qb, ra, fmadd(qa, rb, sim));
                    sqq = fmadd(qb, qb, fmadd(qa, qa, sqq));
                }
        }
        block_products<B4 ? 4 : 0>(sre, sim, sqq, red, lane, wid, nw);
        if (!(sqq > 0.0))
            break;  // zero residue on this block: uniform across the workgroup
        // with q = D_Lambda r = -acc / 2: alpha = (q, r) / ||q||^2 = -2 (acc, r) / ||acc||^2,
        // x += alpha r, r -= alpha q = r + (alpha / 2) acc
        const c32 alpha{(float)(-2.0 * sre / sqq), (float)(-2.0 * sim / sqq)};
        const c32 half{0.5f * alpha.re, 0.5f * alpha.im};
        if (active) {
#pragma unroll
            for (int al = 0; al < 4; ++al)
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    const int e = (3 * al + a) * Vsb + t;
                    const c32 r = lr[e];
                    lx[e] = cfma(alpha, r, lx[e]);
                    lr[e] = cfma(half, acc.s[al].c[a], r);
                }
        }
    }

    if (active) {
#pragma unroll
        for (int al = 0; al < 4; ++al)
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                const uint32_t at = toff<c32>(s, 3 * al + a, 12);
                c32 p = lx[(3 * al + a) * Vsb + t];
                if (init == 0)
                    p += ld(psi, at);
                st(psi, at, p);
                if (out64)
                    st(out64, 2 * at, c64{(double)p.re, (double)p.im});
            }
    }
}

// ---------------------------------------------------------------- lane pairs
//
// Sweep with two lanes per site (lanes i and i + 32 of a wavefront). The lower
// lane takes the four forward hops, (1 - g_mu) U_mu(x) psi(x + mu), the upper
// lane the four backward ones, (1 + g_mu) U_mu(x - mu)^+ psi(x - mu). The upper
// lane holds the adjoint of its link, and its spin projection and reconstruction
// equal the forward ones with the sign of every e_mu term flipped (see the
// projector identities in hop.h), so both lanes run one instruction stream with
// the sign as an FMA operand. The pair's partial sums are combined by one swap
// of wavefront halves and one add per real, which leaves each lane the two spin
// components that it owns of the residue, the MR direction and the block
// solution (lower: spins 0 and 1, upper: 2 and 3, which is also one chirality
// block of the clover term each). Neighbouring lanes are neighbouring sites of
// one kind of hop, so the LDS reads have no bank conflicts.
// FP32: four links of 3x3 per lane (72 VGPRs). FP64: the links' first two rows
// (96 VGPRs), the third ones rebuilt for every use; the residue and the block
// solution live in LDS alone, and so do kPC of the lane's 18 clover entries.
// Both leave room for two wavefronts per SIMD, one block of 256 sites per CU.
// FP64, 4^4 blocks: 20 fields on 16^4 360 us per sweep (links re-read at every
// step: 579), one field on 8^4 29 us (61), with the clover term on 32 x 16^3
// 55 us (138). The vector units are busy half of the time, the rest is the latency of
// the LDS reads, barriers and first loads at two wavefronts per SIMD.

// x + s*y, x + s*i*y and x - s*i*y with the lane's sign s
template <typename T> __device__ inline cpx<T> add_s(cpx<T> x, T sg, cpx<T> y)
{
    return {fmadd(sg, y.re, x.re), fmadd(sg, y.im, x.im)};
}
template <typename T> __device__ inline cpx<T> add_si(cpx<T> x, T sg, cpx<T> y)
{
    return {fmadd(-sg, y.im, x.re), fmadd(sg, y.re, x.im)};
}
template <typename T> __device__ inline cpx<T> add_smi(cpx<T> x, T sg, cpx<T> y)
{
    return {fmadd(sg, y.im, x.re), fmadd(-sg, y.re, x.im)};
}

// the projected colour vector K (h_K of hop.h with the lane's sign) of the
// neighbour whose component (spin, colour) is p(3 * spin + colour)
template <int MU, int K, typename T, typename P> __device__ inline cvec3<T> pair_project(const P& p, T sg)
{
    cvec3<T> h;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const cpx<T> x = p(3 * K + a);
        if (MU == 0)
            h.c[a] = add_s(x, sg, p(3 * (2 + K) + a));
        else if (MU == 1)
            h.c[a] = add_si(x, sg, p(3 * (3 - K) + a));
        else if (MU == 2)
            h.c[a] = add_s(x, K == 0 ? sg : -sg, p(3 * (3 - K) + a));
        else
            h.c[a] = K == 0 ? add_si(x, sg, p(3 * 2 + a)) : add_smi(x, sg, p(3 * 3 + a));
    }
    return h;
}
// acc += the contribution of w = W h_K to all four spins
template <int MU, int K, typename T> __device__ inline void pair_add(const cvec3<T>& w, T sg, spinor<T>& acc)
{
    acc.s[K] += w;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        if (MU == 0)
            acc.s[2 + K].c[a] = add_s(acc.s[2 + K].c[a], sg, w.c[a]);
        else if (MU == 1)
            acc.s[3 - K].c[a] = add_smi(acc.s[3 - K].c[a], sg, w.c[a]);
        else if (MU == 2)
            acc.s[3 - K].c[a] = add_s(acc.s[3 - K].c[a], K == 0 ? sg : -sg, w.c[a]);
        else
            acc.s[2 + K].c[a] = K == 0 ? add_smi(acc.s[2].c[a], sg, w.c[a]) : add_si(acc.s[3].c[a], sg, w.c[a]);
    }
}
// acc += forward (sg = +1, w = U_mu(x)) or backward (sg = -1, w = U_mu(x-mu)^+)
// hop. FP64 takes the two colour vectors one after the other, which keeps the
// live registers below 256.
template <int MU, typename T, typename P>
__device__ inline void hop_pair(const su3<T>& w, const P& p, T sg, spinor<T>& acc)
{
    if constexpr (sizeof(T) == 8) {
        pair_add<MU, 0>(mul(w, pair_project<MU, 0, T>(p, sg)), sg, acc);
        asm volatile("" ::: "memory");
        pair_add<MU, 1>(mul(w, pair_project<MU, 1, T>(p, sg)), sg, acc);
        return;
    }
    const cvec3<T> h0 = pair_project<MU, 0, T>(p, sg), h1 = pair_project<MU, 1, T>(p, sg);
    const cvec3<T> w0 = mul(w, h0), w1 = mul(w, h1);
    pair_add<MU, 0>(w0, sg, acc);
    pair_add<MU, 1>(w1, sg, acc);
}
template <typename T, typename P>
__device__ inline void hop_pair_rt(int mu, const su3<T>& w, const P& p, T sg, spinor<T>& acc)
{
    if (mu == 0) hop_pair<0>(w, p, sg, acc);
    else if (mu == 1) hop_pair<1>(w, p, sg, acc);
    else if (mu == 2) hop_pair<2>(w, p, sg, acc);
    else hop_pair<3>(w, p, sg, acc);
}

// lo + (lo of the upper lane of the pair) in the lower lanes, hi + (hi of the
// lower lane) in the upper ones; every lane of the wavefront must take part
__device__ inline float pair_sum(float lo, float hi)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(lo), __float_as_uint(hi), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ inline double pair_sum(double lo, double hi)
{
    const unsigned long long a = (unsigned long long)__double_as_longlong(lo), b = (unsigned long long)__double_as_longlong(hi);
    const auto l = __builtin_amdgcn_permlane32_swap((unsigned)a, (unsigned)b, false, false);
    const auto h = __builtin_amdgcn_permlane32_swap((unsigned)(a >> 32), (unsigned)(b >> 32), false, false);
    return __longlong_as_double((long long)(((unsigned long long)h[0] << 32) | l[0])) +
           __longlong_as_double((long long)(((unsigned long long)h[1] << 32) | l[1]));
}

// the lane's link for direction mu: U_mu(x) (forward lane) or U_mu(x - mu)^+ (backward lane)
template <typename L> __device__ inline auto pair_link(const L& U, int mu, long site, bool bwd)
{
    auto u = to_link(load_rows(U, mu, site));
    decltype(u) w;
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int b = 0; b < 3; ++b) {
            const auto x = u.m[a][b], y = u.m[b][a];
            w.m[a][b] = bwd ? conjg(y) : x;
        }
    return w;
}

// IMP: clover term (C.c non-null); FP32: or antiperiodic time, and the lanes'
// products summed in FP64
constexpr int kPC = 7;
template <typename T, typename L, bool B4, bool IMP>
__global__ __launch_bounds__(512, 1) void k_sap_pair(Geom g, SapGeom sg, L U, const cpx<T>* __restrict__ rho,
                                                     const double* __restrict__ rho_nrm2, cpx<T>* __restrict__ psi,
                                                     T diag, int nmr, int colour, int nrhs, int init,
                                                     c64* __restrict__ out64, Clover<T> C)
{
    constexpr bool F64 = sizeof(T) == 8;
    const int Vsb = B4 ? 256 : sg.Vsb, NT = B4 ? 512 : (int)blockDim.x;
    int sbl[4], lst[4];
#pragma unroll
    for (int mu = 0; mu < 4; ++mu) {
        sbl[mu] = B4 ? 4 : sg.sb[mu];
        lst[mu] = B4 ? (64 >> (2 * mu)) : sg.lstr[mu];
    }
    const T rs = rho_scale<T>(rho_nrm2, blockIdx.x % nrhs);
    rho += (long)(blockIdx.x % nrhs) * 12 * g.V;
    psi += (long)(blockIdx.x % nrhs) * 12 * g.V;
    if (out64)
        out64 += (long)(blockIdx.x % nrhs) * 12 * g.V;
    extern __shared__ char smem_raw[];
    cpx<T>* lr = reinterpret_cast<cpx<T>*>(smem_raw);
    cpx<T>* lx = lr + 12 * Vsb;  // FP64: block solution
    cpx<T>* lc = lx + 12 * Vsb;  // FP64: clover entries, q * blockDim.x + thread
    __shared__ double red[3][8];

    const int t = threadIdx.x;
    const int ts = (t >> 6) * 32 + (t & 31);  // site in the block
    const int hb = (t >> 5) & 1;     // 0: forward hops, spins 0-1; 1: backward hops, spins 2-3
    const T sgn = hb ? T(-1) : T(1);
    const bool active = ts < Vsb;  // both lanes of a pair agree
    const int lane = t & 63, wid = t >> 6, nw = blockDim.x >> 6;

    int k = blockIdx.x / nrhs;
    int half = sg.nsb[3] / 2;
    int m[4];
    int j = k % half;
    int rest = k / half;
    m[2] = rest % sg.nsb[2];
    rest /= sg.nsb[2];
    m[1] = rest % sg.nsb[1];
    m[0] = rest / sg.nsb[1];
    m[3] = 2 * j + ((colour + m[0] + m[1] + m[2]) & 1);

    int yl[4] = {0, 0, 0, 0};
    int n[4] = {0, 0, 0, 0}, y[4] = {0, 0, 0, 0};
    long s = 0;
    if (active) {
        int tt = ts;
        yl[3] = tt % sbl[3];
        tt /= sbl[3];
        yl[2] = tt % sbl[2];
        tt /= sbl[2];
        yl[1] = tt % sbl[1];
        yl[0] = tt / sbl[1];
        for (int mu = 0; mu < 4; ++mu) {
            int x = m[mu] * sbl[mu] + yl[mu];
            n[mu] = x / g.b[mu];
            y[mu] = x - n[mu] * g.b[mu];
        }
        s = site_compose(g, n, y);
    }
    // neighbour of this lane's hop inside the block
    bool inside[4];
#pragma unroll
    for (int mu = 0; mu < 4; ++mu)
        inside[mu] = hb ? yl[mu] > 0 : yl[mu] + 1 < sbl[mu];
    const int c0 = 6 * hb;  // first owned component (3 * spin + colour)

    // residual with the full operator; the links are kept for the MR steps
    cpx<T> lk[4][F64 ? 6 : 9];
    auto link = [&](int mu) {
        su3<T> w;
#pragma unroll
        for (int q = 0; q < (F64 ? 6 : 9); ++q)
            w.m[q / 3][q % 3] = lk[mu][q];
        if constexpr (F64) {
            pin(w.m[0][0]);
            pin(w.m[0][1]);
            pin(w.m[0][2]);
            complete_third_row(w);
        }
        return w;
    };
    spinor<T> acc;
    zero(acc);
    if (active) {
#pragma unroll
        for (int mu = 0; mu < 4; ++mu) {
            long tn = site_step(g, s, n, y, mu, hb ? -1 : +1);
            const su3<T> w = pair_link(U, mu, hb ? tn : s, hb != 0);
#pragma unroll
            for (int q = 0; q < (F64 ? 6 : 9); ++q)
                lk[mu][q] = w.m[q / 3][q % 3];
            if (init == 0 || (init == 1 && !inside[mu])) {
                spinor<T> p = load_spinor(psi, g.V, tn);
                if ((F64 || IMP) && mu == 0 && crosses_time(g, n, y, mu, hb ? -1 : +1))
                    negate(p);
                hop_pair_rt(mu, w, [&](int c) { return p.s[c / 3].c[c % 3]; }, sgn, acc);
            }
            if (F64 || (mu & 1))
                asm volatile("" ::: "memory");  // two hops' loads in flight at a time (FP64: one)
        }
    }
    // this lane's components of the residue and of the block solution
    cpx<T> rr[F64 ? 1 : 6], xx[F64 ? 1 : 6], q[6];
    auto r_of = [&](int i) { return F64 ? lr[(c0 + i) * Vsb + ts] : rr[F64 ? 0 : i]; };
    // the lane's clover block
    cpx<T> cl[18];
    const bool clv = IMP && (F64 || C.c) && active;
    if (clv) {
        clover_load(C, s, hb, cl);
        if (F64)
#pragma unroll
            for (int e = 0; e < kPC; ++e)
                lc[e * NT + t] = cl[e];
    }
    auto clover = [&](const cpx<T> (&v)[6], cpx<T> (&w)[6]) {
        cpx<T> e[18];
#pragma unroll
        for (int i = 0; i < 18; ++i)
            e[i] = F64 && i < kPC ? lc[i * NT + t] : cl[i];
        clover_mul(e, v, w);
    };
#pragma unroll
    for (int i = 0; i < 6; ++i)
        q[i] = cpx<T>{0, 0};
    if (clv && init == 0) {
        cpx<T> self[6];
#pragma unroll
        for (int i = 0; i < 6; ++i)
            self[i] = ld(psi, toff<cpx<T>>(s, c0 + i, 12));
        clover(self, q);
    }
#pragma unroll
    for (int i = 0; i < 6; ++i) {
        // pair sum, then the owned half (spins 0-1 or 2-3)
        const int al = i / 3, a = i % 3;
        const cpx<T> ao{pair_sum(acc.s[al].c[a].re, acc.s[al + 2].c[a].re),
                        pair_sum(acc.s[al].c[a].im, acc.s[al + 2].c[a].im)};
        cpx<T> r = cpx<T>{0, 0};
        if (active) {
            cpx<T> self = cpx<T>{0, 0};
            if (init == 0)
                self = ld(psi, toff<cpx<T>>(s, c0 + i, 12));
            cpx<T> b = ld(rho, toff<cpx<T>>(s, c0 + i, 12));
            if (rho_nrm2)
                b = cpx<T>{b.re * rs, b.im * rs};
            if (IMP)
                b -= q[i];
            r = cpx<T>{b.re - (diag * self.re - T(0.5) * ao.re), b.im - (diag * self.im - T(0.5) * ao.im)};
            if (F64) {
                lr[(c0 + i) * Vsb + ts] = r;
                lx[(c0 + i) * Vsb + ts] = cpx<T>{0, 0};
            }
        }
        if (!F64) {
            rr[F64 ? 0 : i] = r;
            xx[F64 ? 0 : i] = cpx<T>{0, 0};
        }
    }

    for (int stp = 0; stp < nmr; ++stp) {
        // q = (diag + C) r, then - 1/2 of the inside hops
        if (active) {
            cpx<T> r[6];
#pragma unroll
            for (int i = 0; i < 6; ++i) {
                r[i] = r_of(i);
                if (!F64)
                    lr[(c0 + i) * Vsb + ts] = r[i];
                q[i] = cpx<T>{diag * r[i].re, diag * r[i].im};
            }
            if (clv)
                clover(r, q);
        }
        __syncthreads();
        zero(acc);
        if (active) {
#pragma unroll
            for (int mu = 0; mu < 4; ++mu) {
                if (inside[mu]) {
                    const cpx<T>* pn = lr + ts + (hb ? -lst[mu] : lst[mu]);
                    hop_pair_rt(mu, link(mu), [&](int c) { return pn[c * Vsb]; }, sgn, acc);
                }
                if (F64 || (mu & 1))
                    asm volatile("" ::: "memory");
            }
        }
        // (spare lanes only join the reductions)
        if (!active)
#pragma unroll
            for (int i = 0; i < 6; ++i)
                q[i] = cpx<T>{0, 0};
        // the lane's products, then the block sums in FP64
        using S = std::conditional_t<F64 || IMP, double, float>;
        S fr_re = 0, fr_im = 0, fqq = 0;
#pragma unroll
        for (int i = 0; i < 6; ++i) {
            const int al = i / 3, a = i % 3;
            const cpx<T> ao{pair_sum(acc.s[al].c[a].re, acc.s[al + 2].c[a].re),
                            pair_sum(acc.s[al].c[a].im, acc.s[al + 2].c[a].im)};
            q[i] = cpx<T>{q[i].re - T(0.5) * ao.re, q[i].im - T(0.5) * ao.im};
            const S qa = q[i].re, qb = q[i].im;
            const cpx<T> r = active ? r_of(i) : cpx<T>{0, 0};
            const S ra = r.re, rb = r.im;
            fr_re = fmadd(qb, rb, fmadd(qa, ra, fr_re));
            fr_im = fmadd(-qb, ra, fmadd(qa, rb, fr_im));
            fqq = fmadd(qb, qb, fmadd(qa, qa, fqq));
        }
        double sre = fr_re, sim = fr_im, sqq = fqq;
        block_products<B4 ? 8 : 0>(sre, sim, sqq, red, lane, wid, nw);
        if (!(sqq > 0.0))
            break;  // zero residue on this block: uniform across the workgroup
        const cpx<T> alpha{(T)(sre / sqq), (T)(sim / sqq)};
        if (F64 ? active : true) {
#pragma unroll
            for (int i = 0; i < 6; ++i) {
                const int e = (c0 + i) * Vsb + ts, v = F64 ? 0 : i;
                const cpx<T> r = r_of(i);
                if (F64) {
                    lx[e] = cfma(alpha, r, lx[e]);
                    lr[e] = cfma(-alpha, q[i], r);
                } else {
                    xx[v] = cfma(alpha, r, xx[v]);
                    rr[v] = cfma(-alpha, q[i], r);
                }
            }
        }
    }

    if (active) {
#pragma unroll
        for (int i = 0; i < 6; ++i) {
            cpx<T> p = F64 ? lx[(c0 + i) * Vsb + ts] : xx[F64 ? 0 : i];
            if (init == 0)
                p += ld(psi, toff<cpx<T>>(s, c0 + i, 12));
            st(psi, toff<cpx<T>>(s, c0 + i, 12), p);
            if (out64)
                st(out64, toff<c64>(s, c0 + i, 12), c64{(double)p.re, (double)p.im});
        }
    }
}

// o = f (dg + C(x)) p, the entries read nine at a time and the chirality blocks
// one after the other (few live registers)
template <typename T>
__device__ inline void clover_set_low(const Clover<T>& C, int s, T f, T dg, const spinor<T>& p, spinor<T>& o)
{
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        cpx<T> e[9], w[6];
        auto v = [&](int i) { return f * p.s[2 * h + i / 3].c[i % 3]; };
#pragma unroll
        for (int i = 0; i < 6; ++i)
            w[i] = dg * v(i);
#pragma unroll
        for (int part = 0; part < 2; ++part) {
#pragma unroll
            for (int q = 0; q < 9; ++q)
                e[q] = ld(C.c, toff<cpx<T>>(s, 18 * h + 9 * part + q, kCloverComp));
            if (part == 0) {
#pragma unroll
                for (int i = 0; i < 6; ++i) {
                    const T d = (i & 1) ? e[i / 2].im : e[i / 2].re;
                    w[i] = cpx<T>{fmadd(d, v(i).re, w[i].re), fmadd(d, v(i).im, w[i].im)};
                }
            }
            int q = 3;
#pragma unroll
            for (int i = 0; i < 6; ++i)
#pragma unroll
                for (int j = i + 1; j < 6; ++j, ++q)
                    if (q / 9 == part) {
                        w[i] = cfma(e[q % 9], v(j), w[i]);
                        w[j] = cfma(conjg(e[q % 9]), v(i), w[j]);
                    }
            // the next entries' address waits for these products
            asm volatile("" : "+v"(s), "+v"(w[0].re), "+v"(w[3].re), "+v"(w[5].im));
        }
#pragma unroll
        for (int i = 0; i < 6; ++i)
            o.s[2 * h + i / 3].c[i % 3] = w[i];
    }
}

// FP64 sweep for blocks of more than 256 sites, one lane per site, one block
// per CU. A site holds its four forward links only (two rows, 96 registers) and
// works on both ends of each: U_mu(x) times the projected neighbour x + mu for
// itself, and U_mu(x)^+ times its own projected residue for x + mu, which takes
// it from LDS; so the MR steps read no link. (The residue before them reads the
// eight links of a site, and the clover entries are read again in every step:
// they fit neither registers nor LDS.) The residue lives in LDS alone, the block
// solution in registers, and psi is read and written once. Bound by latency: one
// block fills a CU's registers, and its eight wavefronts meet at ten barriers a
// step.
// 8 x 4^3 blocks on 32 x 16^3: with the clover term 102 us per sweep where the
// links re-read at every step took 168; three fields without it 146 (238). With
// the residue in registers too, and psi updated in every step, 125 and 150.
template <bool IMP>
__global__ __launch_bounds__(512, 2) void k_sap_big(Geom g, SapGeom sg, Links64 U, const c64* __restrict__ rho,
                                                    c64* __restrict__ psi, double diag, int nmr, int colour, int nrhs,
                                                    int init, Clover<double> C)
{
    // workgroup -> (block of this colour, right-hand side), right-hand sides fastest
    rho += (long)(blockIdx.x % nrhs) * 12 * g.V;
    psi += (long)(blockIdx.x % nrhs) * 12 * g.V;
    extern __shared__ char smem_raw[];
    c64* lr = reinterpret_cast<c64*>(smem_raw);  // [12][Vsb] residue
    c64* ex = lr + 12 * sg.Vsb;                  // [6][Vsb] backward hops on their way to x + mu
    __shared__ double red[3][8];

    const int t = threadIdx.x;
    const bool active = t < sg.Vsb;
    const int lane = t & 63, wid = t >> 6, nw = blockDim.x >> 6;

    // k-th block of this colour -> block coordinates m
    int k = blockIdx.x / nrhs;
    int half = sg.nsb[3] / 2;
    int m[4];
    int j = k % half;
    int rest = k / half;
    m[2] = rest % sg.nsb[2];
    rest /= sg.nsb[2];
    m[1] = rest % sg.nsb[1];
    m[0] = rest / sg.nsb[1];
    m[3] = 2 * j + ((colour + m[0] + m[1] + m[2]) & 1);

    int yl[4] = {0, 0, 0, 0};
    int n[4] = {0, 0, 0, 0}, y[4] = {0, 0, 0, 0};
    long s = 0;
    if (active) {
        int tt = t;
        yl[3] = tt % sg.sb[3];
        tt /= sg.sb[3];
        yl[2] = tt % sg.sb[2];
        tt /= sg.sb[2];
        yl[1] = tt % sg.sb[1];
        yl[0] = tt / sg.sb[1];
        for (int mu = 0; mu < 4; ++mu) {
            int x = m[mu] * sg.sb[mu] + yl[mu];
            n[mu] = x / g.b[mu];
            y[mu] = x - n[mu] * g.b[mu];
        }
        s = site_compose(g, n, y);
    }
    const bool clv = IMP && C.c != nullptr;

    // residual with the full operator
    spinor<double> xs;
    zero(xs);
    if (active) {
        spinor<double> acc, self;
        zero(acc);
        zero(self);
        if (init < 2)
            full_hops(g, sg, U, psi, s, n, y, yl, init == 1, acc);
        if (init == 0)
            self = load_spinor(psi, g.V, s);
        spinor<double> d = finish(self, acc, diag);
        if (clv && init == 0)
            clover_add(C, s, self, d);
        const spinor<double> b = load_spinor(rho, g.V, s);
#pragma unroll
        for (int al = 0; al < 4; ++al)
#pragma unroll
            for (int a = 0; a < 3; ++a)
                lr[(3 * al + a) * sg.Vsb + t] = b.s[al].c[a] - d.s[al].c[a];
    }
    LinkRows<Links64> lk[4];
    if (active)
#pragma unroll
        for (int mu = 0; mu < 4; ++mu)
            lk[mu] = load_rows(U, mu, s);

    for (int step = 0; step < nmr; ++step) {
        // (unknown to the compiler here: addresses are formed in the step, not kept over all of them)
        int Vsb = sg.Vsb, sc = (int)s;
        asm volatile("" : "+s"(Vsb), "+v"(sc));
        // acc = -2 D_Lambda r: it starts at -2 (diag + C) r and collects the inside
        // hops, so the MR coefficient follows from it without forming D_Lambda r
        spinor<double> acc;
        if (active) {
            spinor<double> r;
#pragma unroll
            for (int al = 0; al < 4; ++al)
#pragma unroll
                for (int a = 0; a < 3; ++a)
                    r.s[al].c[a] = lr[(3 * al + a) * Vsb + t];
            if (clv) {
                clover_set_low(C, sc, -2.0, diag, r, acc);
            } else {
#pragma unroll
                for (int al = 0; al < 4; ++al)
#pragma unroll
                    for (int a = 0; a < 3; ++a)
                        acc.s[al].c[a] = -2.0 * diag * r.s[al].c[a];
            }
        } else {
            zero(acc);
        }
        __syncthreads();
        auto direction = [&](auto mu_c) {
            constexpr int MU = decltype(mu_c)::value;
            const int lst = sg.lstr[MU];
            if (active && yl[MU] + 1 < sg.sb[MU]) {
                pin(lk[MU].e[0]);
                pin(lk[MU].e[1]);
                pin(lk[MU].e[2]);
                const su3<double> u = to_link(lk[MU]);
#pragma unroll
                for (int K = 0; K < 2; ++K) {
                    // (1 + g_mu) r(x) and (1 - g_mu) r(x + mu), their colour vector K
                    const c64 *po = lr + t, *pn = po + lst;
                    const auto own = [&](int c) { return po[c * Vsb]; };
                    const cvec3<double> v = mul_dag(u, K == 0 ? pair_project<MU, 0, double>(own, -1.0)
                                                              : pair_project<MU, 1, double>(own, -1.0));
#pragma unroll
                    for (int a = 0; a < 3; ++a)
                        ex[(3 * K + a) * Vsb + t] = v.c[a];
                    const auto p = [&](int c) { return pn[c * Vsb]; };
                    if (K == 0)
                        pair_add<MU, 0>(mul(u, pair_project<MU, 0, double>(p, 1.0)), 1.0, acc);
                    else
                        pair_add<MU, 1>(mul(u, pair_project<MU, 1, double>(p, 1.0)), 1.0, acc);
                    asm volatile("" ::: "memory");
                }
            }
            __syncthreads();
            if (active && yl[MU] > 0) {
                cvec3<double> v0, v1;
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    v0.c[a] = ex[a * Vsb + t - lst];
                    v1.c[a] = ex[(3 + a) * Vsb + t - lst];
                }
                bwd_add<MU>(v0, v1, acc);
            }
            if (MU < 3)
                __syncthreads();
        };
        direction(std::integral_constant<int, 0>());
        direction(std::integral_constant<int, 1>());
        direction(std::integral_constant<int, 2>());
        direction(std::integral_constant<int, 3>());
        double sre = 0.0, sim = 0.0, sqq = 0.0;
        if (active) {
#pragma unroll
            for (int al = 0; al < 4; ++al)
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    const double qa = acc.s[al].c[a].re, qb = acc.s[al].c[a].im;
                    const c64 r = lr[(3 * al + a) * Vsb + t];
                    const double ra = r.re, rb = r.im;
                    sre = fmadd(qb, rb, fmadd(qa, ra, sre));
                    sim = fmadd(-qb, ra, fmadd(qa, rb, sim));
                    sqq = fmadd(qb, qb, fmadd(qa, qa, sqq));
                }
        }
        block_products<0>(sre, sim, sqq, red, lane, wid, nw);
        if (!(sqq > 0.0))
            break;  // zero residue on this block: uniform across the workgroup
        // with q = D_Lambda r = -acc / 2: alpha = (q, r) / ||q||^2 = -2 (acc, r) / ||acc||^2,
        // x += alpha r, r -= alpha q = r + (alpha / 2) acc
        const c64 alpha{-2.0 * sre / sqq, -2.0 * sim / sqq};
        const c64 ha{0.5 * alpha.re, 0.5 * alpha.im};
        if (active) {
#pragma unroll
            for (int al = 0; al < 4; ++al)
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    const int e = (3 * al + a) * Vsb + t;
                    const c64 r = lr[e];
                    xs.s[al].c[a] = cfma(alpha, r, xs.s[al].c[a]);
                    lr[e] = cfma(ha, acc.s[al].c[a], r);
                }
        }
    }

    if (active) {
#pragma unroll
        for (int al = 0; al < 4; ++al)
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                const uint32_t at = toff<c64>(s, 3 * al + a, 12);
                c64 p = xs.s[al].c[a];
                if (init == 0)
                    p += ld(psi, at);
                st(psi, at, p);
            }
    }
}

inline bool is_b4(const SapGeom& sg) { return sg.sb[0] == 4 && sg.sb[1] == 4 && sg.sb[2] == 4 && sg.sb[3] == 4; }

template <typename T, typename L, bool IMP>
void launch_pair(const Geom& g, const SapGeom& sg, L U, const cpx<T>* rho, const double* rho_nrm2, cpx<T>* psi, T m0,
                 int nmr, int colour, int nrhs, int init, c64* out64, hipStream_t s, const cpx<T>* clov)
{
    const int threads = (sg.Vsb + 31) / 32 * 64;
    size_t lds = (size_t)12 * sg.Vsb * sizeof(cpx<T>);
    if (sizeof(T) == 8)
        lds += lds + (IMP ? (size_t)kPC * threads * sizeof(cpx<T>) : 0);
    static std::once_flag attr[2];  // per kernel instantiation
    auto go = [&](std::once_flag& f, auto* kernel) {
        set_max_lds_once(f, reinterpret_cast<const void*>(kernel), 160 * 1024 - 1024);
        hipLaunchKernelGGL(kernel, dim3(sg.n_per_colour * nrhs), dim3(threads), lds, s, g, sg, U, rho, rho_nrm2, psi,
                           T(4) + m0, nmr, colour, nrhs, init, out64, Clover<T>{clov});
    };
    if (is_b4(sg))
        go(attr[0], &k_sap_pair<T, L, true, IMP>);
    else
        go(attr[1], &k_sap_pair<T, L, false, IMP>);
}

// one lane per site: with the clover term (CLV), else k_sap_rl
template <typename L, bool B4, bool CLV, bool WIDE>
void launch_rl_kernel(const Geom& g, const SapGeom& sg, L U, const c32* rho, const double* rho_nrm2, c32* psi,
                      float m0, int nmr, int colour, int nrhs, int init, c64* out64, hipStream_t s, const c32* clov)
{
    const dim3 grid(sg.n_per_colour * nrhs), threads(((sg.Vsb + 63) / 64) * 64);
    static std::once_flag attr;  // one per kernel instantiation
    if constexpr (CLV) {
        set_max_lds_once(attr, reinterpret_cast<const void*>(&k_sap_cl<L, B4>), 160 * 1024 - 1024);
        hipLaunchKernelGGL((k_sap_cl<L, B4>), grid, threads, (size_t)(24 + 2 * kLC) * sg.Vsb * sizeof(c32), s, g, sg,
                           U, rho, rho_nrm2, psi, 4.0f + m0, nmr, colour, nrhs, init, out64, Clover<float>{clov});
    } else {
        set_max_lds_once(attr, reinterpret_cast<const void*>(&k_sap_rl<L, B4, WIDE>), 160 * 1024 - 1024);
        hipLaunchKernelGGL((k_sap_rl<L, B4, WIDE>), grid, threads, (size_t)36 * sg.Vsb * sizeof(c32), s, g, sg, U, rho,
                           rho_nrm2, psi, 4.0f + m0, nmr, colour, nrhs, init, out64);
    }
}

// FP32: links in registers. One field on lattices whose colours hold few blocks
// per CU (sg.one_rl == 0), blocks of up to 256 sites: lane pairs, one block per
// CU at two wavefronts per SIMD (16^4 and 32 x 16^3 with 4^4 blocks: 11% faster
// than one lane per site). Several fields, one field with many blocks per
// colour, or larger blocks: one lane per site, two blocks of up to 256 sites
// per CU (16 fields on 16^4: 12% faster than three blocks per CU with the links
// re-read at every MR step, and 28% faster than lane pairs; one field on 64 x
// 32^3: 346 against 475 us per sweep with lane pairs).
template <typename L>
void launch32(const Geom& g, const SapGeom& sg, L U, const c32* rho, const double* rho_nrm2, c32* psi, float m0,
              int nmr, int colour, int nrhs, int init, c64* out64, hipStream_t s, const c32* clov)
{
    auto go = [&](auto launch) { launch(g, sg, U, rho, rho_nrm2, psi, m0, nmr, colour, nrhs, init, out64, s, clov); };
    const bool b4 = is_b4(sg), anti = g.tsign < 0;
    if (nrhs == 1 && !sg.one_rl && sg.Vsb <= 256)
        clov || anti ? go(&launch_pair<float, L, true>) : go(&launch_pair<float, L, false>);
    else if (clov)
        b4 ? go(&launch_rl_kernel<L, true, true, true>) : go(&launch_rl_kernel<L, false, true, true>);
    else if (anti || sg.Vsb > 256)
        b4 ? go(&launch_rl_kernel<L, true, false, true>) : go(&launch_rl_kernel<L, false, false, true>);
    else
        b4 ? go(&launch_rl_kernel<L, true, false, false>) : go(&launch_rl_kernel<L, false, false, false>);
}

// FP64: lane pairs for blocks of up to 256 sites (55 us per sweep of one improved
// field on 32 x 16^3, with one lane per site and links re-read 138). Pairs of
// larger blocks would need twice a CU's registers: one lane per site and link.
void launch64(const Geom& g, const SapGeom& sg, Links64 U, const c64* rho, c64* psi, double m0, int nmr, int colour,
              int nrhs, int init, hipStream_t s, const c64* clov)
{
    if (sg.Vsb <= 256) {
        if (clov)
            launch_pair<double, Links64, true>(g, sg, U, rho, nullptr, psi, m0, nmr, colour, nrhs, init, nullptr, s,
                                               clov);
        else
            launch_pair<double, Links64, false>(g, sg, U, rho, nullptr, psi, m0, nmr, colour, nrhs, init, nullptr, s,
                                                clov);
        return;
    }
    const int threads = ((sg.Vsb + 63) / 64) * 64;
    const size_t lds = (size_t)18 * sg.Vsb * sizeof(c64);
    static std::once_flag attr[2];
    auto go = [&](std::once_flag& f, auto* kernel) {
        set_max_lds_once(f, reinterpret_cast<const void*>(kernel), 160 * 1024 - 1024);
        hipLaunchKernelGGL(kernel, dim3(sg.n_per_colour * nrhs), dim3(threads), lds, s, g, sg, U, rho, psi, 4.0 + m0,
                           nmr, colour, nrhs, init, Clover<double>{clov});
    };
    if (clov)
        go(attr[0], &k_sap_big<true>);
    else
        go(attr[1], &k_sap_big<false>);
}

}  // namespace

void launch_sap_colour64(const Geom& g, const SapGeom& sg, Links64 U, const c64* rho, c64* psi, double m0, int nmr,
                         int colour, int nrhs, int init, hipStream_t s, const c64* clov)
{
    launch64(g, sg, U, rho, psi, m0, nmr, colour, nrhs, init, s, clov);
}
void launch_sap_colour32(const Geom& g, const SapGeom& sg, Links32 U, const c32* rho, c32* psi, float m0, int nmr,
                         int colour, int nrhs, int init, c64* out64, hipStream_t s, const c32* clov,
                         const double* rho_nrm2)
{
    launch32(g, sg, U, rho, rho_nrm2, psi, m0, nmr, colour, nrhs, init, out64, s, clov);
}
void launch_sap_colour_bf16(const Geom& g, const SapGeom& sg, LinksBF16 U, const c32* rho, c32* psi, float m0,
                            int nmr, int colour, int nrhs, int init, c64* out64, hipStream_t s, const c32* clov,
                            const double* rho_nrm2)
{
    launch32(g, sg, U, rho, rho_nrm2, psi, m0, nmr, colour, nrhs, init, out64, s, clov);
}

}  // namespace dfl
