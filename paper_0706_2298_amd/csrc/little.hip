// GCR for the little system A v = w (eq. (6.1), appendix A.4) in a single
// cooperative launch.
//
// The little vector has Nb*Ns entries; workgroup g owns the block pairs
// g, g + G, g + 2G, ... (G = grid size; pair p = blocks 2p and 2p + 1) and all
// entries of those blocks. A pair are neighbours along x3, one block of either
// colour, so both halves of the even-odd operator occupy every workgroup (with
// single blocks g, g + G, ... a workgroup's blocks often had one colour and
// half of the workgroups idled in either half). One GCR step normally needs two grid-wide barriers (one more inside the
// even-odd operator):
//   S1  xi_k = r is complete everywhere: apply chi_k = A xi_k (rows of the
//       owned blocks; the nine neighbour blocks' entries are read from global
//       memory). Convergence is tested before it on ||r_k||^2 =
//       ||r_{k-1}||^2 - |c_k|^2, which needs no reduction;
//   S2  reduce (chi_j, chi_k), (chi_j, r) for j < k, ||chi_k||^2 and
//       (chi_k, r) in one pass; classical Gram-Schmidt then gives the
//       normalised chi_k, its coefficient c_k = (chi_k, r) and the new residue
//       without another reduction (||chi_k - sum a_j chi_j||^2 =
//       ||chi_k||^2 - sum |a_j|^2).
// If that single pass cancels more than 99% of ||chi_k||^2 (orthogonality
// would suffer), a second pass with its own barrier S3 repeats it.
// Partial sums are written per workgroup, summed in a fixed order by one
// workgroup per slot and published, so all workgroups take identical decisions
// and the result is bit-reproducible. After nkv steps (or convergence) the
// solution is updated from the triangular system and the residue recomputed as
// w - A x (two more barriers); convergence is decided on that true residue. The
// barriers are this file's own (flag_barrier, grid_barrier); the launch is
// cooperative so all workgroups are resident.
#include <algorithm>

#include "internal.h"

namespace dfl {

namespace {

constexpr int LT = 1024;            // threads per workgroup of the many-source solver (16 wavefronts)
constexpr int LT1 = 512;            // threads per workgroup of the single-source solver: a few blocks per
                                    // workgroup need no more, and 512 threads leave 256 VGPRs per lane
constexpr long kSpinLimit = 1L << 24;  // ~0.5 s of polling before a barrier gives up
using namespace little;              // the partial-sum slots
static_assert(NK + NQ <= 64, "the coefficient step gives each projection one lane of a wavefront");

template <typename T> struct LittleArgs {
    Geom g;
    int Ns, nkv, maxiter;
    double tol2;           // stop at ||r||^2 <= tol2 * ||w||^2
    const double* tol_dev; // if set: the relative tolerance is read from here at entry
    const cpx<T>* At;      // [Nb][9][Ns(l)][Ns(k)]: transposed blocks
    const cpx<T>* Mt;      // even-odd: [Nb][0] = D^-1, [Nb][d] = D^-1 A_d, transposed likewise
    const cpx<T>* w;
    cpx<T>* x;
    cpx<T>* r;
    cpx<T>* xi;            // nkv * N
    cpx<T>* chi;           // nkv * N
    cpx<T>* w1;            // even-odd workspaces (N each)
    cpx<T>* w2;
    const cpx<T>* Q;       // global deflation (appendix A.3), minimal-residual form: nq orthonormal
    const cpx<T>* Z;       //   images Q = A_hat Z and their preimages Z, little vectors (even blocks);
                           //   oblique form: Q holds W = A_hat Z, Z is orthonormal
    int nq;
    int oblique;           // 1: the oblique projectors of section 3 on the even-odd system, with
    const double* Ainv;    //   Ainv = (Z^+ W)^-1 (nq x nq complex, row-major) and
    const double* Gw;      //   Gw = W^+ W (nq x nq complex)
    double* part;          // NSLOT * G complex partial sums, then NSLOT published sums
    int* stats;            // [0] += iterations, [1] += solves, [2] |= 1 not converged, |= 4 barrier timeout
    int ucap, tab;         // blocks whose neighbour vectors fit LDS; whether the neighbour table does
    unsigned long long* bar_gen;  // flags of the workgroups, two each (flag_barrier)
};

// Grid-wide barrier for a cooperative launch (all workgroups co-resident).
// Thread 0 of each workgroup publishes the workgroup's writes with one
// agent-scope release fence, counts in with a relaxed atomic, and (unless it
// is the last to arrive) polls the generation word with relaxed coherent
// loads; one agent-scope acquire fence follows. The last arrival resets the
// counter and publishes the next generation. Acquire/release semantics on
// every poll would make each poll an L2 invalidation, which serialises
// across the device; this form costs one cache write-back and one
// invalidation per workgroup and barrier. The generation word is never
// reset: a launch continues from the value the previous one left (read once
// at entry). Polling is bounded; on timeout the workgroup records a failure
// and continues, so every wave reaches the end.
__device__ inline void grid_barrier(unsigned* count, unsigned long long* gen, unsigned long long& target, int* stats)
{
    __syncthreads();
    if (threadIdx.x == 0) {
        ++target;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
        unsigned old = __hip_atomic_fetch_add(count, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (old == gridDim.x - 1) {
            __hip_atomic_store(count, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(gen, target, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
        } else {
            long spin = 0;
            while (__hip_atomic_load(gen, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < target) {
                __builtin_amdgcn_s_sleep(1);
                if (++spin > kSpinLimit) {
                    atomicOr(&stats[2], 4);
                    break;
                }
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    }
    __syncthreads();
}

// What workgroups of the single-source solvers exchange (the operator's
// argument and intermediate, partial and reduced sums) is written and read with
// agent-scope relaxed atomics, which are coherent by themselves: their barriers
// need no cache write-back or invalidation, only that a thread's stores have
// completed before its workgroup raises its flag, and what a workgroup keeps to
// itself (matrices, Krylov vectors) stays in its caches.
template <typename T> __device__ inline cpx<T> ld_agent(const cpx<T>* p)
{
    if constexpr (sizeof(T) == 4) {
        const unsigned long long b = __hip_atomic_load(reinterpret_cast<const unsigned long long*>(p), __ATOMIC_RELAXED,
                                                       __HIP_MEMORY_SCOPE_AGENT);
        return cpx<T>{(T)__uint_as_float((unsigned)b), (T)__uint_as_float((unsigned)(b >> 32))};
    } else {
        const double* q = reinterpret_cast<const double*>(p);
        const double re = __hip_atomic_load(q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const double im = __hip_atomic_load(q + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return cpx<T>{(T)re, (T)im};
    }
}
template <typename T> __device__ inline void st_agent(cpx<T>* p, cpx<T> v)
{
    if constexpr (sizeof(T) == 4) {
        const unsigned long long b = (unsigned long long)__float_as_uint((float)v.re) |
                                     ((unsigned long long)__float_as_uint((float)v.im) << 32);
        __hip_atomic_store(reinterpret_cast<unsigned long long*>(p), b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    } else {
        double* q = reinterpret_cast<double*>(p);
        __hip_atomic_store(q, (double)v.re, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(q + 1, (double)v.im, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// With `raise`, sets this workgroup's flag to `target` once all its threads'
// stores have completed; then every thread with wait >= 0 waits until the flag
// of workgroup `wait` has reached it (the count may wrap). Polling is bounded;
// on timeout a failure is recorded and the thread goes on.
__device__ inline void flag_barrier(unsigned* flags, unsigned target, int g, bool raise, int wait, int* stats)
{
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0 && raise)
        __hip_atomic_store(flags + g, target, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (wait >= 0) {
        long spin = 0;
        while ((int)(__hip_atomic_load(flags + wait, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) - target) < 0) {
            __builtin_amdgcn_s_sleep(1);
            if (++spin > kSpinLimit) {
                atomicOr(&stats[2], 4);
                break;
            }
        }
    }
    __syncthreads();
}

__device__ inline double2 cfma_conj(double2 acc, double ar, double ai, double br, double bi)
{
    // acc += conj(a) * b
    acc.x += ar * br + ai * bi;
    acc.y += ar * bi - ai * br;
    return acc;
}

constexpr int kMaxOwned = 1024;  // blocks one workgroup of the even-odd solver may own
constexpr int kLittleStage = 52 * 1024;              // LDS for staged neighbour vectors
constexpr int kLittleDynLds = kLittleStage + 36 * 1024 + 1024;  // and the tables of kMaxOwned blocks

// colour (sum of block coordinates mod 2) of block blk
__device__ inline int block_colour(const Geom& g, int blk)
{
    int sum = 0, rest = blk;
    for (int mu = 3; mu >= 0; --mu) {
        sum += rest % g.nb[mu];
        rest /= g.nb[mu];
    }
    return sum & 1;
}

__device__ inline int nbr_block(const Geom& g, int blk, int d)
{
    if (d == 0)
        return blk;
    const int mu = (d - 1) >> 1;
    int rest = blk;
    for (int nu = 3; nu > mu; --nu)
        rest /= g.nb[nu];
    const int n_mu = rest % g.nb[mu];
    int nn = n_mu + ((d & 1) ? 1 : -1);
    if (nn < 0)
        nn += g.nb[mu];
    if (nn >= g.nb[mu])
        nn -= g.nb[mu];
    return blk + (nn - n_mu) * g.bstr[mu];
}

// The i-th owned block of workgroup g of G, and how many it owns (Nb is even)
__device__ inline int owned_block(int g, int G, int i) { return 2 * (g + (i >> 1) * G) + (i & 1); }
__device__ inline int owned_count(int Nb, int g, int G) { return 2 * ((Nb / 2 - g + G - 1) / G); }

// The workgroup's view: it owns owned_block(i) (i = owned position); its
// vector entries are those of the owned positions listed in vb (all of them
// when vb is null). nbr (LDS, may be null): nbr[8 i + d - 1] = neighbour d of
// owned position i.
template <typename T> struct LittleCtx {
    const LittleArgs<T>& a;
    int G, g, t;
    long N;
    const int* vb;
    int nvb;
    const int* nbr;
    cpx<T>* us;  // LDS: the neighbour vectors of up to ucap blocks
    int ucap;
    __device__ int block(int i) const { return owned_block(g, G, vb ? vb[i] : i); }
    __device__ long entry(int e) const
    {
        int i = e / a.Ns;
        int k = e - i * a.Ns;
        return (long)block(i) * a.Ns + k;
    }
    __device__ int R() const { return nvb * a.Ns; }
    // this workgroup's share of a partial-sum slot
    __device__ void put(int slot, double re, double im) const
    {
        st_agent(reinterpret_cast<cpx<double>*>(a.part) + (long)slot * G + g, cpx<double>{re, im});
    }
};

// Slots of one Gram-Schmidt pass that a wavefront sums at a time, their loads
// in flight together
constexpr int kSlotUnroll = 4;

// red[0 .. ns) = the sums over the G workgroups of the partial-sum slots s0 ..,
// the same in all of them: workgroup g sums the slots g, g + G, ..., one
// wavefront each, and publishes them in pub, and everyone reads those. Ends a
// flag_barrier of all workgroups. red: 2 ns doubles in LDS.
__device__ inline void reduce_slots(unsigned* flags, unsigned* rflags, unsigned& target, int* stats, double* part,
                                    double* pub, int G, int g, int s0, int ns, double* red)
{
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
    const int owners = ns < G ? ns : G;
    flag_barrier(flags, ++target, g, true, t < G && g < owners ? t : -1, stats);
    const cpx<double>* pp = reinterpret_cast<const cpx<double>*>(part);
    cpx<double>* pb = reinterpret_cast<cpx<double>*>(pub);
    for (int s = g + wv * G; s < ns; s += G * (LT1 / 64)) {
        cpx<double> v[kLittleMaxGrid / 64];
#pragma unroll
        for (int i = 0; i < kLittleMaxGrid / 64; ++i) {
            const int q = lane + 64 * i;
            v[i] = q < G ? ld_agent(pp + (long)(s0 + s) * G + q) : cpx<double>{0.0, 0.0};
        }
        double re = 0.0, im = 0.0;
#pragma unroll
        for (int i = 0; i < kLittleMaxGrid / 64; ++i) {
            re += v[i].re;
            im += v[i].im;
        }
        re = wave_sum(re);
        im = wave_sum(im);
        if (lane == 0)
            st_agent(pb + s, cpx<double>{re, im});
    }
    flag_barrier(rflags, target, g, g < owners, t < owners ? t : -1, stats);
    for (int s = t; s < ns; s += LT1) {
        const cpx<double> v = ld_agent(pb + s);
        red[2 * s] = v.re;
        red[2 * s + 1] = v.im;
    }
    __syncthreads();
}

// y_blk = alpha s_blk + beta sum_{d0 <= d < d1} Mat[blk][d] u_{nbr_d(blk)} for
// the blocks at the listed owned positions (list null: positions 0..nlist-1).
// u is an exchanged vector: the neighbours' entries are fetched into LDS, ucap
// blocks at a time. Mat is stored transposed, Mat[blk][d][l][k] = (block d of
// blk)[k][l], so the threads of a block's rows k read Mat coalesced in k. A
// thread sums all terms of one row (or, when the rows do not fill the
// workgroup, those of a contiguous range of d, the ranges meeting in lds in a
// fixed order), with kApplyChunk matrix loads of kApplyD neighbour blocks in
// flight at a time, and writes its row without waiting for the others: y may
// alias u where the rows written and the entries read lie on different blocks
// (the even-odd updates). y is written for exchange. Ends with a workgroup
// barrier.
constexpr int kApplyChunk = 8;
template <typename T>
__device__ inline void apply_blocks(const LittleCtx<T>& c, const int* list, int nlist, const cpx<T>* __restrict__ Mat,
                                    int d0, int d1, const cpx<T>* u, const cpx<T>* s, double alpha, double beta,
                                    cpx<T>* y, double* lds)
{
    constexpr int kApplyD = 2;
    const Geom& g = c.a.g;
    const int Ns = c.a.Ns;
    const int nd = d1 - d0;
    for (int b0 = 0; b0 < nlist; b0 += c.ucap) {
        const int nb = min(c.ucap, nlist - b0);
        const int rows = nb * Ns;
        for (int q = c.t; q < rows * nd; q += LT1) {
            const int l = q % Ns, bd = q / Ns;
            const int ib = bd / nd, d = d0 + bd - ib * nd;
            const int own = list ? list[b0 + ib] : b0 + ib;
            const int blk = owned_block(c.g, c.G, own);
            const int nbr = d == 0 ? blk : (c.nbr ? c.nbr[8 * own + d - 1] : nbr_block(g, blk, d));
            c.us[q] = ld_agent(u + (long)nbr * Ns + l);
        }
        __syncthreads();
        const int ng = max(1, min(LT1 / rows, nd));
        const int per = (nd + ng - 1) / ng;
        for (int t0 = 0; t0 < ng * rows; t0 += LT1) {
            const int task = t0 + c.t;
            if (task < ng * rows) {
                const int gq = task / rows, row = task - gq * rows;
                const int ib = row / Ns, k = row - ib * Ns;
                const int blk = owned_block(c.g, c.G, list ? list[b0 + ib] : b0 + ib);
                const int da = d0 + gq * per, dz = min(d1, da + per);
                double re = 0.0, im = 0.0;
                for (int db = da; db < dz; db += kApplyD) {
                    const cpx<T>* M[kApplyD];
                    const cpx<T>* uu[kApplyD];
#pragma unroll
                    for (int v = 0; v < kApplyD; ++v) {
                        const int d = min(db + v, dz - 1);  // past dz: a valid block, dropped below
                        M[v] = Mat + ((long)blk * 9 + d) * Ns * Ns + k;
                        uu[v] = c.us + (ib * nd + d - d0) * Ns;
                    }
                    for (int l0 = 0; l0 < Ns; l0 += kApplyChunk) {
                        cpx<T> mv[kApplyD][kApplyChunk];
#pragma unroll
                        for (int v = 0; v < kApplyD; ++v)
#pragma unroll
                            for (int q = 0; q < kApplyChunk; ++q)
                                mv[v][q] = M[v][(long)min(l0 + q, Ns - 1) * Ns];  // past Ns: re-read, dropped below
#pragma unroll
                        for (int v = 0; v < kApplyD; ++v)
#pragma unroll
                            for (int q = 0; q < kApplyChunk; ++q)
                                if (db + v < dz && l0 + q < Ns) {
                                    const cpx<T> p = mv[v][q], w = uu[v][l0 + q];
                                    re += (double)p.re * (double)w.re - (double)p.im * (double)w.im;
                                    im += (double)p.re * (double)w.im + (double)p.im * (double)w.re;
                                }
                    }
                }
                if (ng == 1) {
                    const long i = (long)blk * Ns + k;
                    double yr = beta * re, yi = beta * im;
                    if (alpha != 0.0) {
                        yr += alpha * (double)s[i].re;
                        yi += alpha * (double)s[i].im;
                    }
                    st_agent(y + i, cpx<T>{(T)yr, (T)yi});
                } else {
                    lds[2 * task] = re;
                    lds[2 * task + 1] = im;
                }
            }
        }
        __syncthreads();
        if (ng > 1) {
            for (int row = c.t; row < rows; row += LT1) {
                double sr = 0.0, si = 0.0;
                for (int gq = 0; gq < ng; ++gq) {
                    sr += lds[2 * (gq * rows + row)];
                    si += lds[2 * (gq * rows + row) + 1];
                }
                const int ib = row / Ns, k = row - ib * Ns;
                const int blk = owned_block(c.g, c.G, list ? list[b0 + ib] : b0 + ib);
                const long i = (long)blk * Ns + k;
                double yr = beta * sr, yi = beta * si;
                if (alpha != 0.0) {
                    yr += alpha * (double)s[i].re;
                    yi += alpha * (double)s[i].im;
                }
                st_agent(y + i, cpx<T>{(T)yr, (T)yi});
            }
            __syncthreads();
        }
    }
    __syncthreads();
}

// ||v||^2 over the workgroup's vector entries -> part[slot][g]
template <typename T>
__device__ inline void partial_norm2(const LittleCtx<T>& c, const cpx<T>* __restrict__ v, int slot, double* sh)
{
    double s = 0.0;
    const int R = c.R();
    for (int e = c.t; e < R; e += LT1) {
        cpx<T> z = v[c.entry(e)];
        s += (double)z.re * (double)z.re + (double)z.im * (double)z.im;
    }
    s = block_sum(s, sh);
    if (c.t == 0)
        c.put(slot, s, 0.0);
}

// Partial sums of one Gram-Schmidt pass over the vector entries, one
// wavefront per slot: (chi_j, y) and (chi_j, r) for j < k, ||y||^2, (y, r)
// and (Q_l, y) for the nq global deflation directions, written to
// part[slot0 ...][g].
template <typename T>
__device__ inline void partial_pass(const LittleCtx<T>& c, const cpx<T>* chi, int k, const cpx<T>* __restrict__ y,
                                    const cpx<T>* __restrict__ r, int slot0, int nqg)
{
    constexpr int NW = LT1 / 64;
    const int lane = c.t & 63, w = c.t >> 6;
    const int ns = 2 * k + 2 + nqg;
    const int R = c.R();
    // kSlotUnroll slots per wavefront at a time, their loads in flight together
    for (int sb = w; sb < ns; sb += NW * kSlotUnroll) {
        double2 acc[kSlotUnroll];
        const cpx<T>* p[kSlotUnroll];
        const cpx<T>* q[kSlotUnroll];
#pragma unroll
        for (int u = 0; u < kSlotUnroll; ++u) {
            acc[u] = make_double2(0.0, 0.0);
            const int s = sb + u * NW;  // slots past ns read y (result dropped)
            if (s < k) {
                p[u] = chi + (long)s * c.N;
                q[u] = y;
            } else if (s < 2 * k) {
                p[u] = chi + (long)(s - k) * c.N;
                q[u] = r;
            } else if (s < 2 * k + 2) {
                p[u] = y;
                q[u] = (s == 2 * k) ? y : r;
            } else if (s < ns) {
                p[u] = c.a.Q + (long)(s - 2 * k - 2) * c.N;
                q[u] = y;
            } else {
                p[u] = y;
                q[u] = y;
            }
        }
        for (int e = lane; e < R; e += 64) {
            const long i = c.entry(e);
            cpx<T> pv[kSlotUnroll], qv[kSlotUnroll];
#pragma unroll
            for (int u = 0; u < kSlotUnroll; ++u) {
                pv[u] = p[u][i];
                qv[u] = q[u][i];
            }
#pragma unroll
            for (int u = 0; u < kSlotUnroll; ++u)
                acc[u] = cfma_conj(acc[u], (double)pv[u].re, (double)pv[u].im, (double)qv[u].re, (double)qv[u].im);
        }
#pragma unroll
        for (int u = 0; u < kSlotUnroll; ++u) {
            const int s = sb + u * NW;
            const double sr = wave_sum(acc[u].x), si = wave_sum(acc[u].y);
            if (s < ns && lane == 0)
                c.put(slot0 + s, sr, si);
        }
    }
}

// ||v||^2 into slot sn and (Q_l, v), l < nq, into slots SQ + l (one wavefront per slot)
template <typename T>
__device__ inline void partial_norm2_q(const LittleCtx<T>& c, const cpx<T>* __restrict__ v, int sn)
{
    const int lane = c.t & 63, w = c.t >> 6;
    const int R = c.R();
    // minimal-residual form: (Q_l, v); oblique form: (Z_l, v) and (W_l, v)
    const int nd = c.a.oblique ? 2 * c.a.nq : c.a.nq;
    for (int s = w; s < 1 + nd; s += LT1 / 64) {
        const cpx<T>* u = s == 0 ? v
                          : (c.a.oblique && s <= c.a.nq) ? c.a.Z + (long)(s - 1) * c.N
                                                          : c.a.Q + (long)((s - 1) % c.a.nq) * c.N;
        double2 acc = make_double2(0.0, 0.0);
        for (int e = lane; e < R; e += 64) {
            long i = c.entry(e);
            cpx<T> p = u[i], q = v[i];
            acc = cfma_conj(acc, (double)p.re, (double)p.im, (double)q.re, (double)q.im);
        }
        acc.x = wave_sum(acc.x);
        acc.y = wave_sum(acc.y);
        if (lane == 0) {
            const int slot = s == 0 ? sn : SQ + s - 1;  // (W_l, v) follow the nq (Z_l, v)
            c.put(slot, acc.x, acc.y);
        }
    }
}

// (Z_l, y), l < nq, into slots SQ + l (oblique deflation of a new Krylov image)
template <typename T>
__device__ inline void partial_zdots(const LittleCtx<T>& c, const cpx<T>* __restrict__ y)
{
    const int lane = c.t & 63, w = c.t >> 6;
    const int R = c.R();
    for (int s = w; s < c.a.nq; s += LT1 / 64) {
        const cpx<T>* u = c.a.Z + (long)s * c.N;
        double2 acc = make_double2(0.0, 0.0);
        for (int e = lane; e < R; e += 64) {
            long i = c.entry(e);
            cpx<T> p = u[i], q = y[i];
            acc = cfma_conj(acc, (double)p.re, (double)p.im, (double)q.re, (double)q.im);
        }
        acc.x = wave_sum(acc.x);
        acc.y = wave_sum(acc.y);
        if (lane == 0)
            c.put(SQ + s, acc.x, acc.y);
    }
}

// For each of the workgroup's entries e (entry index i): out(e, i, sr, si)
// with sr + i si = sum_{j < nterm} cf(j) v(j)[i], cf(j) a complex coefficient
// (double2) and v(j) a little vector. When the workgroup has few entries the
// terms of an entry are split over thread groups whose partial sums meet in
// lds (2 LT1 doubles, summed in a fixed order); loads are issued four terms
// at a time. Ends with a workgroup barrier.
constexpr int kTermChunk = 4;
template <typename T, typename CF, typename VF, typename OUT>
__device__ inline void combine_terms(const LittleCtx<T>& c, int nterm, CF cf, VF vf, double* lds, OUT out)
{
    const int R = c.R();
    const int ng = R > 0 ? max(1, min(LT1 / R, (nterm + kTermChunk - 1) / kTermChunk)) : 1;
    const int per = (nterm + ng - 1) / ng;
    for (int t = c.t; t < ng * R; t += LT1) {
        const int gq = t / R, e = t - gq * R;
        const long i = c.entry(e);
        double sr = 0.0, si = 0.0;
        const int ja = gq * per, jz = min(nterm, ja + per);
        for (int jb = ja; jb < jz; jb += kTermChunk) {
            cpx<T> zv[kTermChunk];
            double2 cv[kTermChunk];
#pragma unroll
            for (int u = 0; u < kTermChunk; ++u) {
                const int j = min(jb + u, jz - 1);  // past jz: a valid term with coefficient 0
                cv[u] = jb + u < jz ? cf(j) : make_double2(0.0, 0.0);
                zv[u] = vf(j)[i];
            }
#pragma unroll
            for (int u = 0; u < kTermChunk; ++u) {
                sr += cv[u].x * (double)zv[u].re - cv[u].y * (double)zv[u].im;
                si += cv[u].x * (double)zv[u].im + cv[u].y * (double)zv[u].re;
            }
        }
        if (ng > 1) {
            lds[2 * t] = sr;
            lds[2 * t + 1] = si;
        } else {
            out(e, i, sr, si);
        }
    }
    if (ng > 1) {
        __syncthreads();
        for (int e = c.t; e < R; e += LT1) {
            double sr = 0.0, si = 0.0;
            for (int gq = 0; gq < ng; ++gq) {
                sr += lds[2 * (gq * R + e)];
                si += lds[2 * (gq * R + e) + 1];
            }
            out(e, c.entry(e), sr, si);
        }
    }
    __syncthreads();
}

// GCR on A v = w (EO = false) or on the even-odd reduced system (EO = true,
// appendix A.2): with D the block diagonal of A and M_d = D^-1 A_d,
//   v_e solves (1 - M_eo M_oe) v_e = (D^-1 w)_e - M_eo (D^-1 w)_o,
//   v_o = (D^-1 w)_o - M_oe v_e.
// Even-odd workspaces: w1 = D^-1 w (all blocks); w2 holds the reduced source
// on even blocks and the intermediate M_oe u on odd blocks.
//
// What bounds it: the matrices, 16 Nb Ns^2 entries a step, where they exceed
// the caches (64 x 32^3, Ns = 24: 302 MB in FP32, 604 in FP64), else the latency of
// its exchanges. Those go through agent-scope atomics and flags without cache
// maintenance, so the Krylov vectors, and matrices that fit, are read from the
// workgroup's own L2 instead of beyond it after each barrier; a workgroup waits
// for its neighbours only before it applies A. MI355X, with fenced barriers
// before and now: 48 x 24^3 (Ns = 20) 55 and 41 us a step in FP32, 2.91 and
// 2.27 ms a solve in FP64; 64 x 32^3 1.82 and 1.46 ms a solve in FP32, 7.05 and
// 6.36 in FP64.
template <typename T, bool EO> __global__ __launch_bounds__(LT1) void k_little_gcr(LittleArgs<T> a)
{
    // FP64: the residue norm inside a cycle follows from the coefficients
    // while it is more than kNormFloor ||w||^2 above the tolerance
    constexpr bool kTrackNorm = sizeof(T) == sizeof(double);
    constexpr double kNormFloor = 1e-12;
    // FP64 solves to a relative tolerance of 1e-8 or looser end on the
    // measured recursive residue (its drift from the true one is ~1e-15);
    // tighter ones, and FP32 solves, confirm it by recomputing w - A x
    constexpr double kLooseTol2 = 1e-16;
    __shared__ double red[2 * (2 * NK + 2 + NQ)];
    __shared__ double acoef[NK][NK][2];
    __shared__ double qcoef[NQ][NK][2];  // components of each direction's image along Q
    __shared__ double zc[NQ][2];
    __shared__ double cq_s[NQ][2];       // coefficients of the current projection along W (or Q) and Z
    __shared__ double pn2_s;             // ||r||^2 after a projection
    __shared__ double bcoef[NK];
    __shared__ double ccoef[NK][2];
    __shared__ double alpha[NK][2];
    __shared__ double sh[16];
    __shared__ double wn2_s, rn2_s;
    __shared__ int second_s;
    __shared__ double lds[2 * LT1];
    // neighbour vectors of ucap blocks, the owned positions by colour (a pair has one of either),
    // and the neighbours of the owned blocks where they fit (tab)
    extern __shared__ char dyn[];
    const int G = (int)gridDim.x, gi = (int)blockIdx.x, t = (int)threadIdx.x;
    const int nbg = owned_count(a.g.Nb, gi, G);
    const bool tab = a.tab != 0;
    cpx<T>* us = reinterpret_cast<cpx<T>*>(dyn);
    int* l_even = reinterpret_cast<int*>(us + (size_t)a.ucap * (EO ? 8 : 9) * a.Ns);
    int* l_odd = l_even + nbg / 2;
    int* nbr_tab = l_odd + nbg / 2;
    if (tab)
        for (int q = t; q < 8 * nbg; q += LT1)
            nbr_tab[q] = nbr_block(a.g, owned_block(gi, G, q >> 3), 1 + (q & 7));
    if (EO)
        for (int q = t; q < nbg / 2; q += LT1) {
            const int odd = block_colour(a.g, owned_block(gi, G, 2 * q));
            l_even[q] = 2 * q + odd;
            l_odd[q] = 2 * q + 1 - odd;
        }
    __syncthreads();
    const int n_even = EO ? nbg / 2 : 0, n_odd = n_even;
    LittleCtx<T> c{a, G, gi, t, (long)a.g.Nb * a.Ns, EO ? l_even : nullptr, EO ? n_even : nbg, tab ? nbr_tab : nullptr,
                   us, a.ucap};
    const double tol2 = a.tol_dev ? (*a.tol_dev) * (*a.tol_dev) : a.tol2;
    unsigned* const flags = reinterpret_cast<unsigned*>(a.bar_gen);
    unsigned* const rflags = flags + kLittleMaxGrid;
    unsigned target = __hip_atomic_load(flags + gi, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (t == 0)  // raised by some reductions only: not to fall behind by more than a launch
        __hip_atomic_store(rflags + gi, target, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    // Barriers after which a workgroup reads its neighbours' blocks wait for their owners only: what they
    // read is not overwritten before the next reduction, which every workgroup takes part in
    const bool few = 8 * nbg <= LT1 && tab;
    auto owner = [&](int own) { return (nbr_tab[8 * own + (t & 7)] >> 1) % G; };
    auto wait_for = [&](const int* list, int n) {
        return few ? ((t >> 3) < n ? owner(list ? list[t >> 3] : t >> 3) : -1) : t < G ? t : -1;
    };
    const int wait_1 = wait_for(EO ? l_odd : nullptr, EO ? n_odd : nbg), wait_2 = EO ? wait_for(l_even, n_even) : -1;
    auto sync_1 = [&]() { flag_barrier(flags, ++target, gi, true, wait_1, a.stats); };  // before op's first half
    auto sync_2 = [&]() { flag_barrier(flags, ++target, gi, true, wait_2, a.stats); };  // before its second
    const long N = c.N;
    const int R = c.R();
    // op: y = A u (plain) or y = u - M_eo M_oe u on even blocks (one more barrier)
    auto op = [&](const cpx<T>* u, cpx<T>* y) {
        if (EO) {
            apply_blocks(c, l_odd, n_odd, a.Mt, 1, 9, u, (const cpx<T>*)nullptr, 0.0, 1.0, a.w2, lds);
            sync_2();
            apply_blocks(c, l_even, n_even, a.Mt, 1, 9, (const cpx<T>*)a.w2, u, 1.0, -1.0, y, lds);
        } else {
            apply_blocks(c, (const int*)nullptr, nbg, a.At, 0, 9, u, (const cpx<T>*)nullptr, 0.0, 1.0, y, lds);
        }
    };
    // a barrier of all workgroups that reduces slots [s0, s0 + ns) into red for everyone
    double* const pub = a.part + (long)NSLOT * G * 2;
    auto barrier_reduce = [&](int s0, int ns) {
        reduce_slots(flags, rflags, target, a.stats, a.part, pub, G, gi, s0, ns, red);
    };
    // red[q] = red[from + q], q < n (then a workgroup barrier)
    auto shift_red = [&](int from, int n) {
        const double v = c.t < n ? red[from + c.t] : 0.0;
        __syncthreads();
        if (c.t < n)
            red[c.t] = v;
        __syncthreads();
    };
    const cpx<T>* rhs = a.w;
    if (EO) {
        apply_blocks(c, (const int*)nullptr, nbg, a.Mt, 0, 1, a.w, (const cpx<T>*)nullptr, 0.0, 1.0, a.w1, lds);
        sync_2();
        apply_blocks(c, l_even, n_even, a.Mt, 1, 9, (const cpx<T>*)a.w1, (const cpx<T>*)a.w1, 1.0, -1.0, a.w2, lds);
        rhs = a.w2;
    }

    const int nq = a.nq;
    const bool obl = a.oblique && nq > 0;
    const int nqg = obl ? 0 : nq;  // deflation directions inside the Gram-Schmidt pass (minimal-residual form)
    // Coefficients of the projection of a vector v whose dots sit in red
    // ((Q_l, v) or (Z_l, v) at 0.., (W_l, v) at 2 nq.. in the oblique form):
    // c = (Q_l, v) (Q orthonormal), or c = Ainv Z^+ v (section 3's P_L on the
    // even-odd system, Ainv the inverse of the little little operator Z^+ A_hat Z).
    // Returns ||v - Q c||^2 given ||v||^2 (thread 0's value is authoritative).
    auto proj_coef = [&](double vn2) {
        if (c.t < nq) {
            double cr = red[2 * c.t], ci = red[2 * c.t + 1];
            if (obl) {
                cr = 0.0;
                ci = 0.0;
                for (int m = 0; m < nq; ++m) {
                    const double ar = a.Ainv[2 * (c.t * nq + m)], ai = a.Ainv[2 * (c.t * nq + m) + 1];
                    cr += ar * red[2 * m] - ai * red[2 * m + 1];
                    ci += ar * red[2 * m + 1] + ai * red[2 * m];
                }
            }
            cq_s[c.t][0] = cr;
            cq_s[c.t][1] = ci;
        }
        __syncthreads();
        double rn = vn2;
        if (c.t == 0) {
            if (!obl) {
                for (int l = 0; l < nq; ++l)
                    rn -= cq_s[l][0] * cq_s[l][0] + cq_s[l][1] * cq_s[l][1];
            } else {
                // ||v - W c||^2 = ||v||^2 - 2 Re sum conj(c_l) (W_l, v) + c^+ Gw c
                for (int l = 0; l < nq; ++l) {
                    const double cr = cq_s[l][0], ci = cq_s[l][1];
                    const double wr = red[2 * (nq + l)], wi = red[2 * (nq + l) + 1];
                    rn -= 2.0 * (cr * wr + ci * wi);
                    for (int m = 0; m < nq; ++m) {
                        const double gr = a.Gw[2 * (l * nq + m)], gi = a.Gw[2 * (l * nq + m) + 1];
                        const double dr = cq_s[m][0], di = cq_s[m][1];
                        // conj(c_l) G_lm c_m
                        const double tr = gr * dr - gi * di, ti = gr * di + gi * dr;
                        rn += cr * tr + ci * ti;
                    }
                }
            }
        }
        return rn;
    };
    // r -= Q c (or W c), x += Z c with c = cq_s: the residue leaves span Q (minimal-residual
    // form) or range(A_hat Z) along the oblique projector (section 3)
    auto project_q = [&]() {
        auto cq = [&](int l) { return make_double2(cq_s[l][0], cq_s[l][1]); };
        combine_terms(c, nq, cq, [&](int l) { return a.Q + (long)l * N; }, lds, [&](int, long i, double sr, double si) {
            a.r[i] = cpx<T>{(T)((double)a.r[i].re - sr), (T)((double)a.r[i].im - si)};
        });
        combine_terms(c, nq, cq, [&](int l) { return a.Z + (long)l * N; }, lds, [&](int, long i, double sr, double si) {
            st_agent(a.x + i, cpx<T>{(T)((double)a.x[i].re + sr), (T)((double)a.x[i].im + si)});
        });
    };

    // x = 0, r = rhs, ||rhs||^2 and (Q, rhs); then r leaves span Q
    for (int e = c.t; e < R; e += LT1) {
        long i = c.entry(e);
        st_agent(a.x + i, cpx<T>{0, 0});
        a.r[i] = rhs[i];
    }
    partial_norm2_q(c, rhs, SW);
    // SW and the SQ slots are adjacent: one reduction, then the (Q_l, rhs) moved to red[0..]
    const int nqd = nq > 0 ? (obl ? 2 * nq : nq) : 0;
    barrier_reduce(SW, 1 + nqd);
    if (c.t == 0)
        wn2_s = red[0];
    shift_red(2, 2 * nqd);
    const double wn2 = wn2_s;
    double rn2_0 = wn2;  // ||r||^2 after the projection below (thread 0)
    if (nq > 0) {
        rn2_0 = proj_coef(wn2);
        project_q();
    }
    if (c.t == 0)
        rn2_s = rn2_0;
    __syncthreads();
    int iters = 0;
    bool converged = !(wn2 > 0.0);
    bool broke = false;
    bool hit = false;      // the last cycle ended on the measured ||r||^2 <= tol^2 ||w||^2
    bool skipped = false;  // ... and the solve ended there without recomputing the residue

    // Every branch below depends only on values reduced identically by all
    // workgroups, so all of them pass the same sequence of grid barriers.
    while (!converged && !broke && iters < a.maxiter) {
        int k = 0;
        hit = false;
        for (; k < a.nkv && iters < a.maxiter; ++k) {
            cpx<T>* xk = a.xi + (long)k * N;
            cpx<T>* ck = a.chi + (long)k * N;
            cpx<T>* xnext = a.xi + (long)(k + 1) * N;  // used only while k + 1 < nkv
            // ||r||^2 inside a cycle: in FP64 it follows from the coefficients
            // (||r_k||^2 = ||r_{k-1}||^2 - |c_k|^2, chi_k a unit vector
            // orthogonal to r_k), but that difference carries an absolute
            // error of a few ulp of ||w||^2. While the estimate lies well
            // above the tolerance it only says "not converged" and the
            // reduction is skipped; near the tolerance, and always in single
            // precision, ||r||^2 is measured. The true residue is recomputed
            // and tested at every restart.
            const bool far = k > 0 && kTrackNorm && rn2_s > (tol2 + kNormFloor) * wn2;
            if (k == 0 || far) {
                if (k == 0)
                    for (int e = c.t; e < R; e += LT1) {
                        long i = c.entry(e);
                        st_agent(xk + i, a.r[i]);  // xi_k = r (else written by the previous step's update)
                    }
                sync_1();  // S1: xi_k complete where it is read
            } else {
                for (int e = c.t; e < R; e += LT1) {
                    long i = c.entry(e);
                    st_agent(xk + i, a.r[i]);
                }
                partial_norm2(c, a.r, SC, sh);
                barrier_reduce(SC, 1);  // S1: r complete everywhere
                if (c.t == 0)
                    rn2_s = red[0];
                __syncthreads();
                if (rn2_s <= tol2 * wn2) {
                    hit = true;
                    break;  // converged with k directions
                }
            }
            op(xk, ck);
            if (obl) {
                // oblique form: chi_k = P_L A_hat xi_k = A_hat xi_k - W Ainv Z^+ A_hat xi_k
                // before the Gram-Schmidt pass (one more reduction); the
                // preimage of chi_k is xi_k - Z c_k
                __syncthreads();
                partial_zdots(c, ck);
                barrier_reduce(SQ, nq);
                proj_coef(0.0);
                if (c.t < nq) {
                    qcoef[c.t][k][0] = cq_s[c.t][0];
                    qcoef[c.t][k][1] = cq_s[c.t][1];
                }
                combine_terms(c, nq, [&](int l) { return make_double2(cq_s[l][0], cq_s[l][1]); },
                              [&](int l) { return a.Q + (long)l * N; }, lds, [&](int, long i, double sr, double si) {
                                  ck[i] = cpx<T>{(T)((double)ck[i].re - sr), (T)((double)ck[i].im - si)};
                              });
            }
            // one Gram-Schmidt pass: everything needed for chi_k, c_k and the new r
            partial_pass(c, a.chi, k, ck, a.r, SA, nqg);
            barrier_reduce(SA, 2 * k + 2 + nqg);  // S2
            // red: [0,k) a_j; [k,2k) (chi_j, r); 2k: ||chi_k||^2; 2k+1: (chi_k, r); [2k+2, 2k+2+nq) (Q_l, chi_k)
            const int q0 = 2 * k + 2;
            // the k + nq <= 64 projections are spread over the lanes of wavefront 0
            if (c.t < 64) {
                const int ri = c.t < k ? 2 * c.t : 2 * (q0 + c.t - k);
                const double m2 = c.t < k + nqg ? red[ri] * red[ri] + red[ri + 1] * red[ri + 1] : 0.0;
                const double p2 = wave_sum(m2);
                if (c.t == 0) {
                    const double n2 = red[4 * k];
                    second_s = ((k > 0 || nqg > 0) && !(n2 - p2 >= 0.01 * n2)) ? 1 : 0;
                }
            }
            __syncthreads();
            if (second_s) {
                // heavy cancellation: subtract the first projections, then a second pass
                for (int e = c.t; e < R; e += LT1) {
                    long i = c.entry(e);
                    double yr = (double)ck[i].re, yi = (double)ck[i].im;
#pragma unroll 8
                    for (int j = 0; j < k; ++j) {
                        cpx<T> z = a.chi[(long)j * N + i];
                        yr -= red[2 * j] * (double)z.re - red[2 * j + 1] * (double)z.im;
                        yi -= red[2 * j] * (double)z.im + red[2 * j + 1] * (double)z.re;
                    }
                    for (int l = 0; l < nqg; ++l) {
                        const double qr = red[2 * (q0 + l)], qi = red[2 * (q0 + l) + 1];
                        const cpx<T> z = a.Q[(long)l * N + i];
                        yr -= qr * (double)z.re - qi * (double)z.im;
                        yi -= qr * (double)z.im + qi * (double)z.re;
                    }
                    ck[i] = cpx<T>{(T)yr, (T)yi};
                }
                if (c.t < k) {
                    acoef[c.t][k][0] = red[2 * c.t];
                    acoef[c.t][k][1] = red[2 * c.t + 1];
                }
                if (c.t < nqg) {
                    qcoef[c.t][k][0] = red[2 * (q0 + c.t)];
                    qcoef[c.t][k][1] = red[2 * (q0 + c.t) + 1];
                }
                __syncthreads();
                partial_pass(c, a.chi, k, ck, a.r, SB, nqg);
                barrier_reduce(SB, 2 * k + 2 + nqg);  // S3
            } else {
                if (c.t < k) {
                    acoef[c.t][k][0] = 0.0;
                    acoef[c.t][k][1] = 0.0;
                }
                if (c.t < nqg) {
                    qcoef[c.t][k][0] = 0.0;
                    qcoef[c.t][k][1] = 0.0;
                }
            }
            // red now holds the (last) pass: a_j, (chi_j, r), ||chi||^2, (chi, r)
            if (c.t < 64) {
                // lane j < k: chi_j; lane k + l: Q_l
                double m2 = 0.0, dr = 0.0, di = 0.0;
                if (c.t < k) {
                    const int j = c.t;
                    const double ar = red[2 * j], ai = red[2 * j + 1];
                    const double qr = red[2 * (k + j)], qi = red[2 * (k + j) + 1];
                    m2 = ar * ar + ai * ai;
                    // (chi - sum a_j chi_j, r) = (chi, r) - sum conj(a_j) (chi_j, r)
                    dr = ar * qr + ai * qi;
                    di = ar * qi - ai * qr;
                    acoef[j][k][0] += ar;
                    acoef[j][k][1] += ai;
                } else if (c.t < k + nqg) {
                    const int l = c.t - k;
                    const double qr = red[2 * (q0 + l)], qi = red[2 * (q0 + l) + 1];
                    m2 = qr * qr + qi * qi;
                    qcoef[l][k][0] += qr;
                    qcoef[l][k][1] += qi;
                }
                m2 = wave_sum(m2);
                dr = wave_sum(dr);
                di = wave_sum(di);
                if (c.t == 0) {
                    const double b2 = red[4 * k] - m2;
                    const double crr = red[4 * k + 2] - dr, cri = red[4 * k + 3] - di;
                    const double b = b2 > 0.0 ? sqrt(b2) : 0.0;
                    bcoef[k] = b;
                    ccoef[k][0] = b > 0.0 ? crr / b : 0.0;
                    ccoef[k][1] = b > 0.0 ? cri / b : 0.0;
                    if (kTrackNorm)
                        rn2_s -= ccoef[k][0] * ccoef[k][0] + ccoef[k][1] * ccoef[k][1];
                }
            }
            __syncthreads();
            const double b = bcoef[k];
            if (!(b > 0.0)) {
                broke = true;  // the new direction lies in the span: end the cycle without it
                break;
            }
            const double inv = 1.0 / b, cr0 = ccoef[k][0], ci0 = ccoef[k][1];
            // chi_k -= sum_j a_j chi_j + sum_l q_l Q_l, then normalise; r -= c_k chi_k
            combine_terms(
                c, k + nqg,
                [&](int j) {
                    const int ri = j < k ? 2 * j : 2 * (q0 + j - k);
                    return make_double2(red[ri], red[ri + 1]);
                },
                [&](int j) { return j < k ? a.chi + (long)j * N : a.Q + (long)(j - k) * N; }, lds,
                [&](int, long i, double sr, double si) {
                    double yr = ((double)ck[i].re - sr) * inv, yi = ((double)ck[i].im - si) * inv;
                    ck[i] = cpx<T>{(T)yr, (T)yi};
                    double rr = (double)a.r[i].re - (cr0 * yr - ci0 * yi);
                    double ri = (double)a.r[i].im - (cr0 * yi + ci0 * yr);
                    a.r[i] = cpx<T>{(T)rr, (T)ri};
                    if (kTrackNorm && k + 1 < a.nkv)
                        st_agent(xnext + i, cpx<T>{(T)rr, (T)ri});  // xi_{k+1} = r
                });
            ++iters;
            __syncthreads();
        }
        // x += sum alpha_k xi_k, alpha from the triangular system
        if (c.t == 0) {
            for (int i = k - 1; i >= 0; --i) {
                double sr = ccoef[i][0], si = ccoef[i][1];
                for (int j = i + 1; j < k; ++j) {
                    double ar = acoef[i][j][0], ai = acoef[i][j][1];
                    sr -= ar * alpha[j][0] - ai * alpha[j][1];
                    si -= ar * alpha[j][1] + ai * alpha[j][0];
                }
                alpha[i][0] = sr / bcoef[i];
                alpha[i][1] = si / bcoef[i];
            }
        }
        __syncthreads();
        // the direction preimages are xi_k - Z q_k: zc = sum_k q_k alpha_k
        if (c.t < nq) {
            double zr = 0.0, zi = 0.0;
            for (int j = 0; j < k; ++j) {
                zr += qcoef[c.t][j][0] * alpha[j][0] - qcoef[c.t][j][1] * alpha[j][1];
                zi += qcoef[c.t][j][0] * alpha[j][1] + qcoef[c.t][j][1] * alpha[j][0];
            }
            zc[c.t][0] = zr;
            zc[c.t][1] = zi;
        }
        __syncthreads();
        // x += sum_j alpha_j xi_j - sum_l zc_l Z_l
        combine_terms(
            c, k + nq,
            [&](int j) {
                return j < k ? make_double2(alpha[j][0], alpha[j][1]) : make_double2(-zc[j - k][0], -zc[j - k][1]);
            },
            [&](int j) { return j < k ? a.xi + (long)j * N : a.Z + (long)(j - k) * N; }, lds,
            [&](int, long i, double sr, double si) {
                st_agent(a.x + i, cpx<T>{(T)((double)a.x[i].re + sr), (T)((double)a.x[i].im + si)});
            });
        if (kTrackNorm && hit && tol2 >= kLooseTol2) {
            converged = true;
            skipped = true;
            break;
        }
        // recompute r = rhs - op(x)
        sync_1();
        op(a.x, a.r);
        __syncthreads();
        for (int e = c.t; e < R; e += LT1) {
            long i = c.entry(e);
            a.r[i] = cpx<T>{(T)((double)rhs[i].re - (double)a.r[i].re), (T)((double)rhs[i].im - (double)a.r[i].im)};
        }
        // partial_norm2_q reads each entry from another thread than the one that wrote it
        __syncthreads();
        partial_norm2_q(c, a.r, SR);
        // slots SR, SW (not used here) and SQ.. in one reduction; the (Q_l, r) then moved to red[0..]
        barrier_reduce(SR, 2 + nqd);
        if (c.t == 0)
            rn2_s = red[0];
        shift_red(4, 2 * nqd);
        double rn2 = rn2_s;
        if (nq > 0) {
            // project the residue (x moves along Z); ||r||^2 as it is afterwards
            rn2 = proj_coef(rn2);
            if (c.t == 0)
                pn2_s = rn2;  // thread 0's value, shared below
            project_q();
            __syncthreads();
            rn2 = pn2_s;
        }
        converged = rn2 <= tol2 * wn2;
        __syncthreads();  // every thread has read rn2_s
        if (c.t == 0)
            rn2_s = rn2;  // start of the next cycle's norm updates
        __syncthreads();
    }
    if (EO) {
        // x_e must be complete everywhere: a barrier followed its last GCR
        // update unless the solve ended without the residue recomputation,
        // and none followed the projection along Z that may come after it
        if (nq > 0 || skipped)
            sync_1();
        apply_blocks(c, l_odd, n_odd, a.Mt, 1, 9, (const cpx<T>*)a.x, (const cpx<T>*)a.w1, 1.0, -1.0, a.x, lds);
    }
    if (c.g == 0 && c.t == 0) {
        atomicAdd(&a.stats[0], iters);
        atomicAdd(&a.stats[1], 1);
        if (!converged)
            atomicOr(&a.stats[2], 1);
    }
}

// -------------------------------------------------- one block pair per workgroup
//
// The even-odd GCR for lattices of at most 512 blocks, where a step is all
// latency: one workgroup per block pair, its eight-neighbour matrices in
// registers (a thread holds one row of one neighbour term), the pair's Krylov
// and deflation vectors in LDS, and every dot product and combination spread
// over groups of 8 or 16 lanes, so that a step has three exchanges between
// workgroups and otherwise no memory access. What workgroups exchange (the
// operator's argument and intermediate, partial and reduced sums) is written
// and read with agent-scope relaxed atomics, which are coherent by themselves:
// the barrier needs no cache write-back or invalidation, only that a thread's
// stores have completed before its workgroup raises its flag. The flags rise by
// one per barrier and are never reset; a launch continues from their value.
// Same algorithm, decisions and precisions as k_little_gcr with the
// minimal-residual deflation; its comments explain the steps.
// MI355X: a little solve of P_L on 32 x 16^3 (Ns = 20, FP64 to 1e-12, 27 steps)
// takes 0.58 ms (k_little_gcr: 1.20), 18 us a step of which 8 are the reduction
// over 256 workgroups; on 8^4 9 us a step (30). P_L of five fields on 8^4 0.26 ms
// (one batched solve: 2.5).

// sums over aligned groups of 8 and 16 lanes, in every lane
__device__ inline double sum8(double v)
{
    using wave_detail::row;
    v += row<0xB1>(v);
    v += row<0x4E>(v);
    return v + row<0x141>(v);
}
__device__ inline double sum16(double v)
{
    v = sum8(v);
    return v + wave_detail::row<0x140>(v);
}

template <typename T, int NL> __global__ __launch_bounds__(LT1) void k_little_gcr_pair(LittleArgs<T> a)
{
    constexpr bool kTrackNorm = sizeof(T) == sizeof(double);
    constexpr double kNormFloor = 1e-12;
    constexpr double kLooseTol2 = 1e-16;
    constexpr int NP = NL + 1;  // LDS stride of a staged neighbour vector (odd: the eight neighbours' banks differ)
    __shared__ cpx<T> chi_s[NK][NL], xi_s[NK][NL], q_s[NQ][NL], z_s[NQ][NL];
    __shared__ cpx<T> su[8 * NP];
    __shared__ cpx<T> w1e_s[NL], w1o_s[NL], rhs_s[NL], r_s[NL], x_s[NL], y_s[NL];
    __shared__ double red[2 * (2 * NK + 2 + NQ)];
    __shared__ double acoef[NK][NK][2], qcoef[NQ][NK][2];
    __shared__ double zc[NQ][2], cq_s[NQ][2], ccoef[NK][2], alpha[NK][2], bcoef[NK];
    __shared__ double rn2_s;
    __shared__ int second_s;

    // several sources are so many independent solves side by side
    const int G = a.g.Nb / 2, src = (int)blockIdx.x / G, g = (int)blockIdx.x - src * G, t = (int)threadIdx.x;
    const int Ns = a.Ns, nq = a.nq;
    a.w += (long)src * a.g.Nb * Ns;
    a.x += (long)src * a.g.Nb * Ns;
    a.w1 += (long)src * a.g.Nb * Ns;
    a.part += (long)src * NSLOT_PAIR * (G + 1) * 2;
    const int lane = t & 63, wv = t >> 6;
    const int first_even = block_colour(a.g, 2 * g) == 0;
    const int be = 2 * g + (first_even ? 0 : 1), bo = 2 * g + (first_even ? 1 : 0);
    const double tol2 = a.tol_dev ? (*a.tol_dev) * (*a.tol_dev) : a.tol2;
    unsigned* const flags = reinterpret_cast<unsigned*>(a.bar_gen) + (long)src * 2 * kLittleMaxGrid;  // one per workgroup
    unsigned* const rflags = flags + kLittleMaxGrid;                 // of the reductions
    unsigned target = __hip_atomic_load(flags + g, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (t == 0)  // raised by some reductions only: not to fall behind by more than a launch
        __hip_atomic_store(rflags + g, target, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    cpx<T>* const ex = a.w1;  // exchanged vectors: the operator's argument (even) and intermediate (odd blocks)
    double* const pub = a.part + (long)NSLOT_PAIR * G * 2;

    // waits for the owners of the odd (even) block's neighbours only: the exchanged vectors that they read are
    // not overwritten before the next reduction, which every workgroup takes part in
    const int wait_o = t < 8 ? nbr_block(a.g, bo, t + 1) >> 1 : -1, wait_e = t < 8 ? nbr_block(a.g, be, t + 1) >> 1 : -1;
    auto sync_odd = [&]() { flag_barrier(flags, ++target, g, true, wait_o, a.stats); };
    auto sync_even = [&]() { flag_barrier(flags, ++target, g, true, wait_e, a.stats); };

    // operator rows in registers: threads 0 .. 8 Ns - 1 the odd block, the next 8 Ns the even one;
    // lane group of eight = one row, lane d of it the term of neighbour d + 1
    const int half = t < 8 * Ns ? 0 : 1;
    const int task = t - half * 8 * Ns;
    const bool has = task < 8 * Ns;
    const int row = task >> 3, d = task & 7;
    cpx<T> m[NL];
    {
        const cpx<T>* M = a.Mt + ((long)(half ? be : bo) * 9 + 1 + d) * Ns * Ns + row;
#pragma unroll
        for (int l = 0; l < NL; ++l)
            m[l] = has && l < Ns ? M[(long)l * Ns] : cpx<T>{0, 0};
    }
    for (int q = t; q < 8 * NP; q += LT1)
        su[q] = cpx<T>{0, 0};
    for (int q = t; q < nq * Ns; q += LT1) {
        q_s[q / Ns][q % Ns] = a.Q[(long)(q / Ns) * a.g.Nb * Ns + (long)be * Ns + q % Ns];
        z_s[q / Ns][q % Ns] = a.Z[(long)(q / Ns) * a.g.Nb * Ns + (long)be * Ns + q % Ns];
    }
    // staging: thread t < 8 Ns fetches entry t % Ns of neighbour t / Ns + 1 of either block
    const int sd = t / Ns, sl = t - sd * Ns;
    const long nb_o = t < 8 * Ns ? (long)nbr_block(a.g, bo, sd + 1) * Ns + sl : 0;
    const long nb_e = t < 8 * Ns ? (long)nbr_block(a.g, be, sd + 1) * Ns + sl : 0;
    auto stage = [&](long from) {
        if (t < 8 * Ns)
            su[sd * NP + sl] = ld_agent(ex + from);
        __syncthreads();
    };
    // sum_d M_d u_d of this thread's row group over the staged vectors, in every lane of the group
    auto rows = [&](double& re, double& im) {
        re = im = 0.0;
        const cpx<T>* u = su + d * NP;
#pragma unroll
        for (int l = 0; l < NL; ++l) {
            const cpx<T> w = u[l];
            re += (double)m[l].re * (double)w.re - (double)m[l].im * (double)w.im;
            im += (double)m[l].re * (double)w.im + (double)m[l].im * (double)w.re;
        }
        re = sum8(re);
        im = sum8(im);
    };
    // the odd half: ex_o = M_oe ex_e
    auto odd_half = [&]() {
        stage(nb_o);
        double re, im;
        rows(re, im);
        if (has && half == 0 && d == 0)
            st_agent(ex + (long)bo * Ns + row, cpx<T>{(T)re, (T)im});
    };
    // the even half: y = u - M_eo ex_o for this block's u
    auto even_half = [&](const cpx<T>* u, cpx<T>* y) {
        stage(nb_e);
        double re, im;
        rows(re, im);
        if (has && half == 1 && d == 0)
            y[row] = cpx<T>{(T)((double)u[row].re - re), (T)((double)u[row].im - im)};
        __syncthreads();
    };
    auto publish = [&](const cpx<T>* v) {
        if (t < Ns)
            st_agent(ex + (long)be * Ns + t, v[t]);
    };
    // dot product of one slot over this block, the first of eight lanes writes the partial sum
    auto slot_dot = [&](const cpx<T>* p, const cpx<T>* q, int slot, bool on) {
        double re = 0.0, im = 0.0;
        if (on)
            for (int e = t & 7; e < Ns; e += 8) {
                const cpx<T> x = p[e], y = q[e];
                re += (double)x.re * (double)y.re + (double)x.im * (double)y.im;
                im += (double)x.re * (double)y.im - (double)x.im * (double)y.re;
            }
        re = sum8(re);
        im = sum8(im);
        if (on && (t & 7) == 0)
            st_agent(reinterpret_cast<cpx<double>*>(a.part) + (long)slot * G + g, cpx<double>{re, im});
    };
    // red[0 .. ns) = the sums of slots s0 .. over the workgroups, the same in all of them
    auto reduce = [&](int s0, int ns) {
        const cpx<double>* part = reinterpret_cast<const cpx<double>*>(a.part);
        const int owners = ns < G ? ns : G;
        flag_barrier(flags, ++target, g, true, t < G && (g < owners || G <= kPairAllRead) ? t : -1, a.stats);
        if (G <= kPairAllRead) {
            constexpr int kRounds = (2 * NK + 2 + NQ + LT1 / 16 - 1) / (LT1 / 16);
            cpx<double> v[kRounds];
            const int q = t & 15;
#pragma unroll
            for (int i = 0; i < kRounds; ++i) {
                const int s = (t >> 4) + i * (LT1 / 16);
                v[i] = s < ns && q < G ? ld_agent(part + (long)(s0 + s) * G + q) : cpx<double>{0.0, 0.0};
            }
#pragma unroll
            for (int i = 0; i < kRounds; ++i) {
                const int s = (t >> 4) + i * (LT1 / 16);
                const double re = sum16(v[i].re), im = sum16(v[i].im);
                if (s < ns && q == 0) {
                    red[2 * s] = re;
                    red[2 * s + 1] = im;
                }
            }
            __syncthreads();
            return;
        }
        // workgroup g sums the slots g, g + G, ..., one wavefront each, and publishes them
        for (int s = g + wv * G; s < ns; s += G * (LT1 / 64)) {
            cpx<double> v[kLittleMaxGrid / 64];
#pragma unroll
            for (int i = 0; i < kLittleMaxGrid / 64; ++i) {
                const int q = lane + 64 * i;
                v[i] = q < G ? ld_agent(part + (long)(s0 + s) * G + q) : cpx<double>{0.0, 0.0};
            }
            double re = 0.0, im = 0.0;
#pragma unroll
            for (int i = 0; i < kLittleMaxGrid / 64; ++i) {
                re += v[i].re;
                im += v[i].im;
            }
            re = wave_sum(re);
            im = wave_sum(im);
            if (lane == 0)
                st_agent(reinterpret_cast<cpx<double>*>(pub) + s, cpx<double>{re, im});
        }
        flag_barrier(rflags, target, g, g < owners, t < owners ? t : -1, a.stats);
        for (int s = t; s < ns; s += LT1) {
            const cpx<double> v = ld_agent(reinterpret_cast<const cpx<double>*>(pub) + s);
            red[2 * s] = v.re;
            red[2 * s + 1] = v.im;
        }
        __syncthreads();
    };
    // sum over the terms of entry e = t / 16 in every lane of its group of 16
    const int ce = t >> 4;
    auto combine = [&](int nterm, auto term, double& re, double& im) {
        re = im = 0.0;
        if (ce < Ns)
            for (int j = t & 15; j < nterm; j += 16) {
                cpx<T> v;
                double2 c;
                term(j, c, v);
                re += c.x * (double)v.re - c.y * (double)v.im;
                im += c.x * (double)v.im + c.y * (double)v.re;
            }
        re = sum16(re);
        im = sum16(im);
    };
    const bool writer = ce < Ns && (t & 15) == 0;
    // (Q_l, v) in red[2 from ..]: c = (Q_l, v); r -= Q c, x += Z c; ||r||^2 afterwards from vn2
    auto project = [&](int from, double vn2) {
        if (t < nq) {
            cq_s[t][0] = red[2 * (from + t)];
            cq_s[t][1] = red[2 * (from + t) + 1];
        }
        __syncthreads();
        double qr, qi, zr, zi;
        combine(nq, [&](int j, double2& c, cpx<T>& v) { c = make_double2(cq_s[j][0], cq_s[j][1]); v = q_s[j][ce]; }, qr, qi);
        combine(nq, [&](int j, double2& c, cpx<T>& v) { c = make_double2(cq_s[j][0], cq_s[j][1]); v = z_s[j][ce]; }, zr, zi);
        if (writer) {
            r_s[ce] = cpx<T>{(T)((double)r_s[ce].re - qr), (T)((double)r_s[ce].im - qi)};
            x_s[ce] = cpx<T>{(T)((double)x_s[ce].re + zr), (T)((double)x_s[ce].im + zi)};
        }
        for (int l = 0; l < nq; ++l)
            vn2 -= cq_s[l][0] * cq_s[l][0] + cq_s[l][1] * cq_s[l][1];
        __syncthreads();
        return vn2;
    };

    // w1 = D^-1 w on both blocks (eight lanes per row), the odd part published; the reduced source on the even block
    {
        const int blk = half ? be : bo;
        double re = 0.0, im = 0.0;
        if (has)
            for (int l = d; l < Ns; l += 8) {
                const cpx<T> p = a.Mt[((long)blk * 9 * Ns + l) * Ns + row], w = a.w[(long)blk * Ns + l];
                re += (double)p.re * (double)w.re - (double)p.im * (double)w.im;
                im += (double)p.re * (double)w.im + (double)p.im * (double)w.re;
            }
        re = sum8(re);
        im = sum8(im);
        if (has && d == 0) {
            const cpx<T> v{(T)re, (T)im};
            if (half) {
                w1e_s[row] = v;
            } else {
                w1o_s[row] = v;
                st_agent(ex + (long)bo * Ns + row, v);
            }
        }
    }
    sync_even();
    even_half(w1e_s, rhs_s);
    if (t < Ns) {
        x_s[t] = cpx<T>{0, 0};
        r_s[t] = rhs_s[t];
    }
    __syncthreads();
    // ||rhs||^2 and (Q, rhs); then r leaves span Q
    slot_dot((t >> 3) == 0 ? rhs_s : q_s[((t >> 3) - 1) & (NQ - 1)], rhs_s, SW + (t >> 3), (t >> 3) < 1 + nq);
    reduce(SW, 1 + nq);
    const double wn2 = red[0];
    double rn2 = project(1, wn2);
    if (t == 0)
        rn2_s = rn2;
    __syncthreads();

    int iters = 0;
    bool converged = !(wn2 > 0.0), broke = false, hit = false;
    while (!converged && !broke && iters < a.maxiter) {
        int k = 0;
        hit = false;
        for (; k < a.nkv && iters < a.maxiter; ++k) {
            if (t < Ns)
                xi_s[k][t] = r_s[t];
            publish(r_s);
            const bool far = k > 0 && kTrackNorm && rn2_s > (tol2 + kNormFloor) * wn2;
            if (k == 0 || far) {
                sync_odd();
            } else {
                slot_dot(r_s, r_s, SC, t < 8);
                reduce(SC, 1);
                if (t == 0)
                    rn2_s = red[0];
                const double rr = red[0];
                __syncthreads();
                if (rr <= tol2 * wn2) {
                    hit = true;
                    break;  // converged with k directions
                }
            }
            odd_half();
            sync_even();
            even_half(xi_s[k], y_s);
            // one Gram-Schmidt pass: (chi_j, y), (chi_j, r), ||y||^2, (y, r), (Q_l, y)
            auto pass = [&](int slot0) {
                const int ns = 2 * k + 2 + nq;
                for (int s = t >> 3; s < (ns + 7) / 8 * 8; s += LT1 / 8) {
                    const cpx<T>* p = s < k ? chi_s[s] : s < 2 * k ? chi_s[s - k] : s < 2 * k + 2 ? y_s
                                      : q_s[(s - 2 * k - 2) & (NQ - 1)];
                    slot_dot(p, (s >= k && s < 2 * k) || s == 2 * k + 1 ? r_s : y_s, slot0 + s, s < ns);
                }
                reduce(slot0, ns);
            };
            pass(pair_first_slot(k));
            const int q0 = 2 * k + 2;
            if (t < 64) {
                const int ri = t < k ? 2 * t : 2 * (q0 + t - k);
                const double m2 = t < k + nq ? red[ri] * red[ri] + red[ri + 1] * red[ri + 1] : 0.0;
                const double p2 = wave_sum(m2);
                if (t == 0) {
                    const double n2 = red[4 * k];
                    second_s = ((k > 0 || nq > 0) && !(n2 - p2 >= 0.01 * n2)) ? 1 : 0;
                }
            }
            __syncthreads();
            auto gs_term = [&](int j, double2& c, cpx<T>& v) {
                const int ri = j < k ? 2 * j : 2 * (q0 + j - k);
                c = make_double2(red[ri], red[ri + 1]);
                v = j < k ? chi_s[j][ce] : q_s[j - k][ce];
            };
            const bool second = second_s != 0;
            if (second) {
                // heavy cancellation: subtract the first projections, then a second pass
                double sr, si;
                combine(k + nq, gs_term, sr, si);
                if (writer)
                    y_s[ce] = cpx<T>{(T)((double)y_s[ce].re - sr), (T)((double)y_s[ce].im - si)};
            }
            if (t < k) {
                acoef[t][k][0] = second ? red[2 * t] : 0.0;
                acoef[t][k][1] = second ? red[2 * t + 1] : 0.0;
            }
            if (t < nq) {
                qcoef[t][k][0] = second ? red[2 * (q0 + t)] : 0.0;
                qcoef[t][k][1] = second ? red[2 * (q0 + t) + 1] : 0.0;
            }
            if (second) {
                __syncthreads();
                pass(SB);
            }
            // red now holds the (last) pass: a_j, (chi_j, r), ||chi||^2, (chi, r)
            if (t < 64) {
                double m2 = 0.0, dr = 0.0, di = 0.0;
                if (t < k) {
                    const double ar = red[2 * t], ai = red[2 * t + 1];
                    const double qr = red[2 * (k + t)], qi = red[2 * (k + t) + 1];
                    m2 = ar * ar + ai * ai;
                    dr = ar * qr + ai * qi;
                    di = ar * qi - ai * qr;
                    acoef[t][k][0] += ar;
                    acoef[t][k][1] += ai;
                } else if (t < k + nq) {
                    const int l = t - k;
                    const double qr = red[2 * (q0 + l)], qi = red[2 * (q0 + l) + 1];
                    m2 = qr * qr + qi * qi;
                }
                m2 = wave_sum(m2);
                dr = wave_sum(dr);
                di = wave_sum(di);
                if (t == 0) {
                    const double b2 = red[4 * k] - m2;
                    const double crr = red[4 * k + 2] - dr, cri = red[4 * k + 3] - di;
                    const double b = b2 > 0.0 ? sqrt(b2) : 0.0;
                    bcoef[k] = b;
                    ccoef[k][0] = b > 0.0 ? crr / b : 0.0;
                    ccoef[k][1] = b > 0.0 ? cri / b : 0.0;
                    if (kTrackNorm)
                        rn2_s -= ccoef[k][0] * ccoef[k][0] + ccoef[k][1] * ccoef[k][1];
                }
            }
            if (t < nq) {
                qcoef[t][k][0] += red[2 * (q0 + t)];
                qcoef[t][k][1] += red[2 * (q0 + t) + 1];
            }
            __syncthreads();
            const double b = bcoef[k];
            if (!(b > 0.0)) {
                broke = true;  // the new direction lies in the span: end the cycle without it
                break;
            }
            // chi_k = (y - sum_j a_j chi_j - sum_l q_l Q_l) / b; r -= c_k chi_k
            double sr, si;
            combine(k + nq, gs_term, sr, si);
            if (writer) {
                const double inv = 1.0 / b, cr0 = ccoef[k][0], ci0 = ccoef[k][1];
                const double yr = ((double)y_s[ce].re - sr) * inv, yi = ((double)y_s[ce].im - si) * inv;
                chi_s[k][ce] = cpx<T>{(T)yr, (T)yi};
                r_s[ce] = cpx<T>{(T)((double)r_s[ce].re - (cr0 * yr - ci0 * yi)),
                                 (T)((double)r_s[ce].im - (cr0 * yi + ci0 * yr))};
            }
            ++iters;
            __syncthreads();
        }
        // x += sum_j alpha_j xi_j - sum_l zc_l Z_l, alpha from the triangular system
        if (t == 0) {
            for (int i = k - 1; i >= 0; --i) {
                double sr = ccoef[i][0], si = ccoef[i][1];
                for (int j = i + 1; j < k; ++j) {
                    const double ar = acoef[i][j][0], ai = acoef[i][j][1];
                    sr -= ar * alpha[j][0] - ai * alpha[j][1];
                    si -= ar * alpha[j][1] + ai * alpha[j][0];
                }
                alpha[i][0] = sr / bcoef[i];
                alpha[i][1] = si / bcoef[i];
            }
        }
        __syncthreads();
        if (t < nq) {
            double zr = 0.0, zi = 0.0;
            for (int j = 0; j < k; ++j) {
                zr += qcoef[t][j][0] * alpha[j][0] - qcoef[t][j][1] * alpha[j][1];
                zi += qcoef[t][j][0] * alpha[j][1] + qcoef[t][j][1] * alpha[j][0];
            }
            zc[t][0] = zr;
            zc[t][1] = zi;
        }
        __syncthreads();
        {
            double sr, si;
            combine(k + nq, [&](int j, double2& c, cpx<T>& v) {
                c = j < k ? make_double2(alpha[j][0], alpha[j][1]) : make_double2(-zc[j - k][0], -zc[j - k][1]);
                v = j < k ? xi_s[j][ce] : z_s[j - k][ce];
            }, sr, si);
            if (writer)
                x_s[ce] = cpx<T>{(T)((double)x_s[ce].re + sr), (T)((double)x_s[ce].im + si)};
            __syncthreads();
        }
        if (kTrackNorm && hit && tol2 >= kLooseTol2) {
            converged = true;
            break;
        }
        // recompute r = rhs - op(x)
        publish(x_s);
        sync_odd();
        odd_half();
        sync_even();
        even_half(x_s, y_s);
        if (t < Ns)
            r_s[t] = cpx<T>{(T)((double)rhs_s[t].re - (double)y_s[t].re), (T)((double)rhs_s[t].im - (double)y_s[t].im)};
        __syncthreads();
        slot_dot((t >> 3) == 0 ? r_s : q_s[((t >> 3) - 1) & (NQ - 1)], r_s, SW + (t >> 3), (t >> 3) < 1 + nq);
        reduce(SW, 1 + nq);
        rn2 = project(1, red[0]);
        converged = rn2 <= tol2 * wn2;
        if (t == 0)
            rn2_s = rn2;  // start of the next cycle's norm updates
        __syncthreads();
    }
    // x_o = w1_o - M_oe x_e
    publish(x_s);
    sync_odd();
    {
        stage(nb_o);
        double re, im;
        rows(re, im);
        if (has && half == 0 && d == 0)
            a.x[(long)bo * Ns + row] = cpx<T>{(T)((double)w1o_s[row].re - re), (T)((double)w1o_s[row].im - im)};
        if (t < Ns)
            a.x[(long)be * Ns + t] = x_s[t];
    }
    if (g == 0 && t == 0) {
        atomicAdd(&a.stats[0], iters);
        atomicAdd(&a.stats[1], 1);
        if (!converged)
            atomicOr(&a.stats[2], 1);
    }
}

// ------------------------------------------------------------ many sources
//
// The same GCR for nrhs little systems A v_b = w_b at once: the right-hand
// sides share the launch, the grid barriers and the reads of A, and each has
// its own Krylov space, coefficients and convergence test. Vectors of RHS b
// sit at b * N (w, x, r) and at (k * nrhs + b) * N (xi_k, chi_k).
// Reductions over the workgroups are two-level: partial sums, a barrier,
// workgroup g sums the slots t = g mod G into fin, a barrier, everyone reads
// fin. A RHS leaves the cycle when it converges or its new direction falls
// in the span; the cycle ends when no RHS is left in it. With EO the systems
// are the even-odd reduced ones of appendix A.2, as in the single-source
// solver: the Krylov vectors live on the even blocks, w1 = M_0 w holds each
// source's block-diagonally scaled right-hand side, w2 the reduced one on the
// even blocks and the operator's intermediate on the odd ones, and the odd
// part of each solution follows from the even part at the end.

constexpr int RS = 2 * NK + 2;  // slots of one pass per RHS

template <typename T> struct LittleMultiArgs {
    Geom g;
    int Ns, nkv, maxiter, nrhs;
    double tol2;
    const double* tol_dev;
    const cpx<T>* At;
    const cpx<T>* Mt;  // even-odd matrices (even-odd kernel only)
    cpx<T>* w1;        // M_0 w, nrhs vectors (even-odd kernel only)
    cpx<T>* w2;        // the reduced right-hand sides on even blocks, the odd-block intermediate of the operator
    const cpx<T>* w;
    cpx<T>* x;
    cpx<T>* r;
    cpx<T>* xi;
    cpx<T>* chi;
    double* part;   // [NSLOT][nrhs][G] complex
    double* fin;    // [nrhs][RS] complex
    double* acoef;  // [G][nrhs][NK][NK] complex (each workgroup's own copy)
    int* stats;
    unsigned* bar_count;
    unsigned long long* bar_gen;
};

template <typename T> struct MultiCtx {
    const LittleMultiArgs<T>& a;
    int G, g, t, nbg, R;
    long N;
    const int* vb;  // positions of the blocks the vectors live on (even-odd: the even ones), null: all owned
    __device__ long entry(int e) const
    {
        int i = e / a.Ns;
        int k = e - i * a.Ns;
        return (long)owned_block(g, G, vb ? vb[i] : i) * a.Ns + k;
    }
    __device__ double* pslot(int slot, int b) const { return a.part + (((long)slot * a.nrhs + b) * G + g) * 2; }
};

// y_b = alpha s_b + beta sum_{d0 <= d < d1} M_d v_b on owned blocks for the
// listed sources, on the matrix cores: for an owned block the terms
// sum_d M_d V_d (V_d: the listed sources' entries on the d-th neighbour, Ns x
// nlist) form one real GEMM of the 2Ns x 2(d1-d0)Ns matrix [[ar, -ai], [ai, ar]]
// (rows and columns interleaved re/im) with the 2(d1-d0)Ns x nlist matrix of
// the V_d entries read as reals, in 16x16x4 tiles (FP32 or FP64 MFMA). Wave w
// takes (block, row tile) tasks w, w + 16, ...; the sources (<= 16) are the
// 16 columns. M (A or the even-odd matrices) is read from transposed blocks,
// coalesced in the row. pos lists the npos owned positions to apply on (null:
// positions 0..npos-1); s is read only when alpha is not zero.
template <typename T> struct Mfma;
// Operands: lane l holds A[l % 16][l / 16] and B[l / 16][l % 16]; result
// element i of lane l is D[row(l / 16, i)][l % 16], with the row order of
// the FP32 and FP64 instructions differing.
template <> struct Mfma<float> {
    using acc_t = __attribute__((ext_vector_type(4))) float;
    static __device__ inline acc_t step(float a, float b, acc_t c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
    static __device__ inline int row(int kq, int i) { return 4 * kq + i; }
};
template <> struct Mfma<double> {
    using acc_t = __attribute__((ext_vector_type(4))) double;
    static __device__ inline acc_t step(double a, double b, acc_t c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }
    static __device__ inline int row(int kq, int i) { return 4 * i + kq; }
};

constexpr int kMfmaBatch = 6;  // MFMA steps whose operands are in flight together (2 Ns = 48: two batches)
template <typename T>
__device__ inline void apply_multi_mfma(const MultiCtx<T>& c, const cpx<T>* __restrict__ Mat, int d0, int d1,
                                        const int* pos, int npos, const cpx<T>* __restrict__ v, const cpx<T>* s,
                                        double alpha, double beta, cpx<T>* y, const int* list, int nlist)
{
    const Geom& g = c.a.g;
    const int Ns = c.a.Ns;
    const int mt = (2 * Ns + 15) / 16;
    const int lane = c.t & 63, wave = c.t >> 6;
    const int n = lane & 15, kq = lane >> 4;
    const int b_n = n < nlist ? list[n] : 0;
    for (int task = wave; task < npos * mt; task += LT / 64) {
        const int ib = task / mt, tt = task - ib * mt;
        const int blk = owned_block(c.g, c.G, pos ? pos[ib] : ib);
        const int rr = 16 * tt + n;
        const int m = rr >> 1, cr = rr & 1;
        typename Mfma<T>::acc_t acc = {0, 0, 0, 0};
#pragma unroll 1
        for (int d = d0; d < d1; ++d) {
            const int nbr = nbr_block(g, blk, d);
            const cpx<T>* Ad = Mat + ((long)blk * 9 + d) * Ns * Ns;
            const cpx<T>* vb = v + b_n * c.N + (long)nbr * Ns;
            // the operands of kMfmaBatch steps loaded together, then their products
#pragma unroll 1
            for (int kc0 = 0; kc0 < 2 * Ns; kc0 += 4 * kMfmaBatch) {
                T av[kMfmaBatch], bw[kMfmaBatch];
                // clamped indices: every load is issued (no branch between them), the
                // out-of-range operands are zeroed afterwards
                cpx<T> za[kMfmaBatch], qa[kMfmaBatch];
#pragma unroll
                for (int st = 0; st < kMfmaBatch; ++st) {
                    const int kk = min(kc0 + 4 * st + kq, 2 * Ns - 1);
                    const int l = kk >> 1;
                    za[st] = Ad[(long)l * Ns + min(m, Ns - 1)];
                    qa[st] = vb[l];
                }
#pragma unroll
                for (int st = 0; st < kMfmaBatch; ++st) {
                    const int kk = kc0 + 4 * st + kq;
                    const int ck = kk & 1;
                    const bool in = kk < 2 * Ns;
                    const cpx<T> z = za[st], q = qa[st];
                    av[st] = (in && m < Ns) ? (cr == 0 ? (ck == 0 ? z.re : -z.im) : (ck == 0 ? z.im : z.re)) : T(0);
                    bw[st] = (in && n < nlist) ? (ck == 0 ? q.re : q.im) : T(0);
                }
#pragma unroll
                for (int st = 0; st < kMfmaBatch; ++st)
                    if (kc0 + 4 * st < 2 * Ns)
                        acc = Mfma<T>::step(av[st], bw[st], acc);
            }
        }
        if (n < nlist) {
            const long o = b_n * c.N + (long)blk * Ns;
            T* yb = reinterpret_cast<T*>(y + o);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int ro = 16 * tt + Mfma<T>::row(kq, i);
                if (ro < 2 * Ns) {
                    double val = beta * (double)acc[i];
                    if (alpha != 0.0)
                        val += alpha * (double)reinterpret_cast<const T*>(s + o)[ro];
                    yb[ro] = (T)val;
                }
            }
        }
    }
    __syncthreads();
}

// part[slot][b][g] = ||v_b||^2 over the owned entries, one wavefront per listed RHS
template <typename T>
__device__ inline void multi_norm2(const MultiCtx<T>& c, const cpx<T>* v, const int* list, int nlist, int slot)
{
    const int lane = c.t & 63, wv = c.t >> 6;
    for (int bi = wv; bi < nlist; bi += LT / 64) {
        const int b = list[bi];
        const cpx<T>* vb = v + b * c.N;
        double s = 0.0;
        for (int e = lane; e < c.R; e += 64) {
            cpx<T> z = vb[c.entry(e)];
            s += (double)z.re * (double)z.re + (double)z.im * (double)z.im;
        }
        s = wave_sum(s);
        if (lane == 0) {
            double* p = c.pslot(slot, b);
            p[0] = s;
            p[1] = 0.0;
        }
    }
}

// every workgroup: out[b] = sum over workgroups of part[slot][b] (real part), listed RHS
__device__ inline void multi_reduce_real(const double* part, int nrhs, int G, int slot, const int* list, int nlist,
                                         double* out)
{
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    for (int bi = wv; bi < nlist; bi += LT / 64) {
        const int b = list[bi];
        double s = 0.0;
        for (int q = lane; q < G; q += 64)
            s += part[(((long)slot * nrhs + b) * G + q) * 2];
        s = wave_sum(s);
        if (lane == 0)
            out[b] = s;
    }
    __syncthreads();
}

// Gram-Schmidt partial sums for the listed RHS into slots slot0 + s, s < 2k+2
// (same layout as partial_pass). One wavefront per (RHS, group of 8 slots):
// the lanes run over the workgroup's entries, y and r are read once for the
// group, and the 8 complex sums are reduced across the wavefront at the end.
constexpr int kSlotGroup = 8;

template <typename T>
__device__ inline void multi_pass(const MultiCtx<T>& c, int k, const int* list, int nlist, int slot0)
{
    const int ns = 2 * k + 2;
    const int ngrp = (ns + kSlotGroup - 1) / kSlotGroup;
    const int lane = c.t & 63, wv = c.t >> 6;
    const long N = c.N;
    const int nr = c.a.nrhs;
    for (int task = wv; task < nlist * ngrp; task += LT / 64) {
        const int bi = task / ngrp, s0 = (task - bi * ngrp) * kSlotGroup;
        const int b = list[bi];
        const cpx<T>* y = c.a.chi + ((long)k * nr + b) * N;
        const cpx<T>* r = c.a.r + b * N;
        double2 acc[kSlotGroup];
#pragma unroll
        for (int q = 0; q < kSlotGroup; ++q)
            acc[q] = make_double2(0.0, 0.0);
        for (int e = lane; e < c.R; e += 64) {
            const long i = c.entry(e);
            const cpx<T> yv = y[i], rv = r[i];
#pragma unroll
            for (int q = 0; q < kSlotGroup; ++q) {
                const int sl = s0 + q;
                if (sl < ns) {
                    cpx<T> u, v;
                    if (sl < 2 * k) {
                        u = c.a.chi[((long)(sl < k ? sl : sl - k) * nr + b) * N + i];
                        v = sl < k ? yv : rv;
                    } else {
                        u = yv;
                        v = sl == 2 * k ? yv : rv;
                    }
                    acc[q] = cfma_conj(acc[q], (double)u.re, (double)u.im, (double)v.re, (double)v.im);
                }
            }
        }
#pragma unroll
        for (int q = 0; q < kSlotGroup; ++q) {
            if (s0 + q >= ns)
                break;
            const double re = wave_sum(acc[q].x), im = wave_sum(acc[q].y);
            if (lane == 0) {
                double* p = c.pslot(slot0 + s0 + q, b);
                p[0] = re;
                p[1] = im;
            }
        }
    }
}

// workgroup g: fin[b][s] = sum over workgroups of part[slot0 + s][b], for the
// (listed RHS, s < ns) tasks t with t mod G == g
__device__ inline void multi_fin(const double* part, double* fin, int nrhs, int G, int g, int slot0, int ns,
                                 const int* list, int nlist)
{
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int ntask = nlist * ns;
    int j = 0;
    for (int task = g; task < ntask; task += G, ++j) {
        if ((j % (LT / 64)) != wv)
            continue;
        const int bi = task / ns, s = task - bi * ns;
        const int b = list[bi];
        double re = 0.0, im = 0.0;
        for (int q = lane; q < G; q += 64) {
            re += part[((((long)slot0 + s) * nrhs + b) * G + q) * 2];
            im += part[((((long)slot0 + s) * nrhs + b) * G + q) * 2 + 1];
        }
        re = wave_sum(re);
        im = wave_sum(im);
        if (lane == 0) {
            fin[((long)b * RS + s) * 2] = re;
            fin[((long)b * RS + s) * 2 + 1] = im;
        }
    }
}

template <typename T, bool EO> __global__ __launch_bounds__(LT) void k_little_gcr_multi(LittleMultiArgs<T> a)
{
    __shared__ double red[kMaxLittleRhs][2 * RS];
    __shared__ double bcoef[kMaxLittleRhs][NK];
    __shared__ double ccoef[kMaxLittleRhs][NK][2];
    __shared__ double alpha[kMaxLittleRhs][NK][2];
    __shared__ double wn2[kMaxLittleRhs], rn2[kMaxLittleRhs];
    __shared__ int act[kMaxLittleRhs], stop[kMaxLittleRhs], conv[kMaxLittleRhs], kb[kMaxLittleRhs];
    __shared__ int second[kMaxLittleRhs];
    __shared__ int list[kMaxLittleRhs], nlist_s, list2[kMaxLittleRhs], nlist2_s;
    __shared__ int l_even[EO ? kMaxOwned : 1], l_odd[EO ? kMaxOwned : 1];  // owned positions by colour
    __shared__ int n_even_s, n_odd_s;

    MultiCtx<T> c{a, (int)gridDim.x, (int)blockIdx.x, (int)threadIdx.x, 0, 0, (long)a.g.Nb * a.Ns, nullptr};
    const double tol2 = a.tol_dev ? (*a.tol_dev) * (*a.tol_dev) : a.tol2;
    const int nr = a.nrhs;
    const long N = c.N;
    unsigned long long bar_target = 0;
    if (c.t == 0)
        bar_target = __hip_atomic_load(a.bar_gen, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    c.nbg = owned_count(a.g.Nb, c.g, c.G);
    if (EO && c.t == 0) {
        int ne = 0, no = 0;
        for (int i = 0; i < c.nbg; ++i) {
            if (block_colour(a.g, owned_block(c.g, c.G, i)))
                l_odd[no++] = i;
            else
                l_even[ne++] = i;
        }
        n_even_s = ne;
        n_odd_s = no;
    }
    if (c.t < nr)
        list[c.t] = c.t;
    if (c.t == 0)
        nlist_s = nr;
    __syncthreads();
    const int n_even = EO ? n_even_s : 0, n_odd = EO ? n_odd_s : 0;
    if (EO)
        c.vb = l_even;
    c.R = (EO ? n_even : c.nbg) * a.Ns;
    double* acoef = a.acoef + (long)c.g * nr * NK * NK * 2;
    auto AC = [&](int b, int i, int j) -> double* { return acoef + (((long)b * NK + i) * NK + j) * 2; };
    // y = A u (plain) or y = u - M_eo M_oe u on even blocks, the odd-block
    // intermediate in w2 (one more grid barrier), for the listed sources
    auto op = [&](const cpx<T>* u, cpx<T>* y, const int* lst, int nl) {
        if (EO) {
            apply_multi_mfma(c, a.Mt, 1, 9, l_odd, n_odd, u, (const cpx<T>*)nullptr, 0.0, 1.0, a.w2, lst, nl);
            grid_barrier(a.bar_count, a.bar_gen, bar_target, a.stats);
            apply_multi_mfma(c, a.Mt, 1, 9, l_even, n_even, (const cpx<T>*)a.w2, u, 1.0, -1.0, y, lst, nl);
        } else {
            apply_multi_mfma(c, a.At, 0, 9, (const int*)nullptr, c.nbg, u, (const cpx<T>*)nullptr, 0.0, 1.0, y, lst,
                             nl);
        }
    };
    // the system's right-hand sides: w, or w1_e - M_eo w1_o (w1 = M_0 w) on even blocks
    const cpx<T>* rhs = a.w;
    if (EO) {
        apply_multi_mfma(c, a.Mt, 0, 1, (const int*)nullptr, c.nbg, a.w, (const cpx<T>*)nullptr, 0.0, 1.0, a.w1,
                         list, nr);
        grid_barrier(a.bar_count, a.bar_gen, bar_target, a.stats);
        apply_multi_mfma(c, a.Mt, 1, 9, l_even, n_even, (const cpx<T>*)a.w1, (const cpx<T>*)a.w1, 1.0, -1.0, a.w2,
                         list, nr);
        rhs = a.w2;
    }

    // x = 0, r = rhs, ||rhs_b||^2
    for (long q = c.t; q < (long)c.R * nr; q += LT) {
        const int b = (int)(q / c.R), e = (int)(q - (long)b * c.R);
        const long i = c.entry(e) + b * N;
        a.x[i] = cpx<T>{0, 0};
        a.r[i] = rhs[i];
    }
    __syncthreads();
    multi_norm2(c, rhs, list, nr, SW);
    grid_barrier(a.bar_count, a.bar_gen, bar_target, a.stats);
    multi_reduce_real(a.part, nr, c.G, SW, list, nr, wn2);
    if (c.t < nr) {
        conv[c.t] = !(wn2[c.t] > 0.0);
        stop[c.t] = conv[c.t];
    }
    __syncthreads();
    int iters = 0;

    // every branch depends on values all workgroups reduce identically
    while (iters < a.maxiter) {
        if (c.t == 0) {
            int n = 0;
            for (int b = 0; b < nr; ++b) {
                act[b] = !stop[b];
                kb[b] = 0;
                if (act[b])
                    list[n++] = b;
            }
            nlist_s = n;
        }
        __syncthreads();
        if (nlist_s == 0)
            break;
        int k = 0;
        for (; k < a.nkv && iters < a.maxiter; ++k) {
            const int nl = nlist_s;
            // xi_k = r and the partial ||r||^2 for the RHS still in the cycle
            for (long q = c.t; q < (long)c.R * nl; q += LT) {
                const int bi = (int)(q / c.R), e = (int)(q - (long)bi * c.R);
                const int b = list[bi];
                const long i = c.entry(e);
                a.xi[((long)k * nr + b) * N + i] = a.r[b * N + i];
            }
            multi_norm2(c, a.r, list, nl, SC);
            grid_barrier(a.bar_count, a.bar_gen, bar_target, a.stats);  // S1
            multi_reduce_real(a.part, nr, c.G, SC, list, nl, rn2);
            if (c.t == 0) {
                int n = 0;
                for (int bi = 0; bi < nl; ++bi) {
                    const int b = list[bi];
                    if (k > 0 && rn2[b] <= tol2 * wn2[b])
                        act[b] = 0;  // converged with k directions
                    else
                        list[n++] = b;
                }
                nlist_s = n;
            }
            __syncthreads();
            const int na = nlist_s;
            if (na == 0)
                break;
            op(a.xi + (long)k * nr * N, a.chi + (long)k * nr * N, list, na);
            multi_pass(c, k, list, na, SA);
            grid_barrier(a.bar_count, a.bar_gen, bar_target, a.stats);  // S2
            multi_fin(a.part, a.fin, nr, c.G, c.g, SA, 2 * k + 2, list, na);
            grid_barrier(a.bar_count, a.bar_gen, bar_target, a.stats);  // S2b
            for (int q = c.t; q < na * (2 * k + 2) * 2; q += LT) {
                const int bi = q / ((2 * k + 2) * 2), rem = q - bi * (2 * k + 2) * 2;
                const int b = list[bi];
                red[b][rem] = a.fin[(long)b * RS * 2 + rem];
            }
            __syncthreads();
            if (c.t < na) {
                const int b = list[c.t];
                double n2 = red[b][4 * k];
                double b2 = n2;
                for (int j = 0; j < k; ++j)
                    b2 -= red[b][2 * j] * red[b][2 * j] + red[b][2 * j + 1] * red[b][2 * j + 1];
                second[b] = (k > 0 && !(b2 >= 0.01 * n2)) ? 1 : 0;
                for (int j = 0; j < k; ++j) {
                    double* p = AC(b, j, k);
                    p[0] = 0.0;
                    p[1] = 0.0;
                }
            }
            __syncthreads();
            if (c.t == 0) {
                int n = 0;
                for (int bi = 0; bi < na; ++bi)
                    if (second[list[bi]])
                        list2[n++] = list[bi];
                nlist2_s = n;
            }
            __syncthreads();
            const int n2l = nlist2_s;
            if (n2l > 0) {
                // heavy cancellation for some RHS: subtract the first projections, then a second pass
                for (long q = c.t; q < (long)c.R * n2l; q += LT) {
                    const int bi = (int)(q / c.R), e = (int)(q - (long)bi * c.R);
                    const int b = list2[bi];
                    const long i = c.entry(e);
                    cpx<T>* ck = a.chi + ((long)k * nr + b) * N;
                    double yr = (double)ck[i].re, yi = (double)ck[i].im;
                    for (int j = 0; j < k; ++j) {
                        cpx<T> z = a.chi[((long)j * nr + b) * N + i];
                        yr -= red[b][2 * j] * (double)z.re - red[b][2 * j + 1] * (double)z.im;
                        yi -= red[b][2 * j] * (double)z.im + red[b][2 * j + 1] * (double)z.re;
                    }
                    ck[i] = cpx<T>{(T)yr, (T)yi};
                }
                if (c.t < n2l) {
                    const int b = list2[c.t];
                    for (int j = 0; j < k; ++j) {
                        double* p = AC(b, j, k);
                        p[0] = red[b][2 * j];
                        p[1] = red[b][2 * j + 1];
                    }
                }
                __syncthreads();
                multi_pass(c, k, list2, n2l, SB);
                grid_barrier(a.bar_count, a.bar_gen, bar_target, a.stats);  // S3
                multi_fin(a.part, a.fin, nr, c.G, c.g, SB, 2 * k + 2, list2, n2l);
                grid_barrier(a.bar_count, a.bar_gen, bar_target, a.stats);  // S3b
                for (int q = c.t; q < n2l * (2 * k + 2) * 2; q += LT) {
                    const int bi = q / ((2 * k + 2) * 2), rem = q - bi * (2 * k + 2) * 2;
                    const int b = list2[bi];
                    red[b][rem] = a.fin[(long)b * RS * 2 + rem];
                }
                __syncthreads();
            }
            if (c.t < na) {
                const int b = list[c.t];
                double b2 = red[b][4 * k];
                double crr = red[b][4 * k + 2], cri = red[b][4 * k + 3];
                for (int j = 0; j < k; ++j) {
                    double ar = red[b][2 * j], ai = red[b][2 * j + 1];
                    double qr = red[b][2 * (k + j)], qi = red[b][2 * (k + j) + 1];
                    b2 -= ar * ar + ai * ai;
                    crr -= ar * qr + ai * qi;
                    cri -= ar * qi - ai * qr;
                    double* p = AC(b, j, k);
                    p[0] += ar;
                    p[1] += ai;
                }
                double bb = b2 > 0.0 ? sqrt(b2) : 0.0;
                bcoef[b][k] = bb;
                ccoef[b][k][0] = bb > 0.0 ? crr / bb : 0.0;
                ccoef[b][k][1] = bb > 0.0 ? cri / bb : 0.0;
            }
            __syncthreads();
            if (c.t == 0) {
                int n = 0;
                for (int bi = 0; bi < na; ++bi) {
                    const int b = list[bi];
                    if (!(bcoef[b][k] > 0.0)) {
                        act[b] = 0;  // new direction in the span: the RHS ends its cycle without it
                        stop[b] = 1;
                    } else {
                        kb[b] = k + 1;
                        list[n++] = b;
                    }
                }
                nlist_s = n;
            }
            __syncthreads();
            const int nu = nlist_s;
            for (long q = c.t; q < (long)c.R * nu; q += LT) {
                const int bi = (int)(q / c.R), e = (int)(q - (long)bi * c.R);
                const int b = list[bi];
                const long i = c.entry(e);
                cpx<T>* ck = a.chi + ((long)k * nr + b) * N;
                const double inv = 1.0 / bcoef[b][k], cr0 = ccoef[b][k][0], ci0 = ccoef[b][k][1];
                double yr = (double)ck[i].re, yi = (double)ck[i].im;
                for (int j = 0; j < k; ++j) {
                    cpx<T> z = a.chi[((long)j * nr + b) * N + i];
                    yr -= red[b][2 * j] * (double)z.re - red[b][2 * j + 1] * (double)z.im;
                    yi -= red[b][2 * j] * (double)z.im + red[b][2 * j + 1] * (double)z.re;
                }
                yr *= inv;
                yi *= inv;
                ck[i] = cpx<T>{(T)yr, (T)yi};
                cpx<T>* rb = a.r + b * N;
                double rr = (double)rb[i].re - (cr0 * yr - ci0 * yi);
                double ri = (double)rb[i].im - (cr0 * yi + ci0 * yr);
                rb[i] = cpx<T>{(T)rr, (T)ri};
            }
            ++iters;
            __syncthreads();
            if (nu == 0)
                break;
        }
        // x_b += sum alpha_j xi_j for the RHS that took directions in this cycle
        if (c.t < nr) {
            const int b = c.t;
            for (int i = kb[b] - 1; i >= 0; --i) {
                double sr = ccoef[b][i][0], si = ccoef[b][i][1];
                for (int j = i + 1; j < kb[b]; ++j) {
                    const double* p = AC(b, i, j);
                    sr -= p[0] * alpha[b][j][0] - p[1] * alpha[b][j][1];
                    si -= p[0] * alpha[b][j][1] + p[1] * alpha[b][j][0];
                }
                alpha[b][i][0] = sr / bcoef[b][i];
                alpha[b][i][1] = si / bcoef[b][i];
            }
        }
        if (c.t == 0) {
            int n = 0;
            for (int b = 0; b < nr; ++b)
                if (kb[b] > 0)
                    list[n++] = b;
            nlist_s = n;
        }
        __syncthreads();
        const int nx = nlist_s;
        for (long q = c.t; q < (long)c.R * nx; q += LT) {
            const int bi = (int)(q / c.R), e = (int)(q - (long)bi * c.R);
            const int b = list[bi];
            const long i = c.entry(e);
            double yr = (double)a.x[b * N + i].re, yi = (double)a.x[b * N + i].im;
            for (int j = 0; j < kb[b]; ++j) {
                cpx<T> z = a.xi[((long)j * nr + b) * N + i];
                yr += alpha[b][j][0] * (double)z.re - alpha[b][j][1] * (double)z.im;
                yi += alpha[b][j][0] * (double)z.im + alpha[b][j][1] * (double)z.re;
            }
            a.x[b * N + i] = cpx<T>{(T)yr, (T)yi};
        }
        // recompute r_b = w_b - A x_b for those RHS
        grid_barrier(a.bar_count, a.bar_gen, bar_target, a.stats);
        op(a.x, a.r, list, nx);
        for (long q = c.t; q < (long)c.R * nx; q += LT) {
            const int bi = (int)(q / c.R), e = (int)(q - (long)bi * c.R);
            const int b = list[bi];
            const long i = c.entry(e) + b * N;
            a.r[i] = cpx<T>{(T)((double)rhs[i].re - (double)a.r[i].re), (T)((double)rhs[i].im - (double)a.r[i].im)};
        }
        __syncthreads();
        multi_norm2(c, a.r, list, nx, SR);
        grid_barrier(a.bar_count, a.bar_gen, bar_target, a.stats);
        multi_reduce_real(a.part, nr, c.G, SR, list, nx, rn2);
        if (c.t < nx) {
            const int b = list[c.t];
            conv[b] = rn2[b] <= tol2 * wn2[b];
            if (conv[b])
                stop[b] = 1;
        }
        __syncthreads();
        if (nx == 0)
            break;  // no RHS made progress: all stopped
    }
    if (EO) {
        // x_o = w1_o - M_oe x_e for every source: a grid barrier followed the
        // last update of x_e (the zero start or the update before the residue
        // recomputation), so the neighbours' entries are complete
        __syncthreads();
        if (c.t < nr)
            list[c.t] = c.t;
        __syncthreads();
        apply_multi_mfma(c, a.Mt, 1, 9, l_odd, n_odd, (const cpx<T>*)a.x, (const cpx<T>*)a.w1, 1.0, -1.0, a.x, list,
                         nr);
    }
    if (c.g == 0 && c.t == 0) {
        int nc = 0;
        for (int b = 0; b < nr; ++b)
            nc += conv[b] ? 0 : 1;
        atomicAdd(&a.stats[0], iters);
        atomicAdd(&a.stats[1], nr);
        if (nc)
            atomicOr(&a.stats[2], 1);
    }
}

template <typename T>
void launch_impl(const Geom& g, int Ns, int nkv, int maxiter, double tol, const double* tol_dev, const cpx<T>* At,
                 const cpx<T>* Mt, const cpx<T>* Q, const cpx<T>* Z, int nq, int oblique, const double* Ainv,
                 const double* Gw, const cpx<T>* w, cpx<T>* x, cpx<T>* r,
                 cpx<T>* xi, cpx<T>* chi, cpx<T>* w1, cpx<T>* w2, double* part, int* stats,
                 unsigned long long* bar_gen, int grid_size, hipStream_t s, bool cooperative)
{
    LittleArgs<T> a;
    a.g = g;
    a.Ns = Ns;
    a.nkv = nkv;
    a.maxiter = maxiter;
    a.tol2 = tol * tol;
    a.tol_dev = tol_dev;
    a.At = At;
    a.Mt = Mt;
    a.w = w;
    a.x = x;
    a.r = r;
    a.xi = xi;
    a.chi = chi;
    a.w1 = w1;
    a.w2 = w2;
    a.Q = Mt ? Q : nullptr;
    a.Z = Mt ? Z : nullptr;
    a.nq = (Mt && Q && Z) ? nq : 0;
    a.oblique = oblique && a.nq > 0 && Ainv && Gw;
    a.Ainv = Ainv;
    a.Gw = Gw;
    if (oblique && a.nq > 0 && !a.oblique)
        fail(DFL_EINVAL, "oblique little deflation needs the inverse and Gram matrices");
    a.part = part;
    a.stats = stats;
    a.bar_gen = bar_gen + kLittleFlags;
    // dynamic LDS: the neighbour vectors of up to kLittleStage bytes, the block lists and, where it fits, the
    // neighbour table
    const int nbg = 2 * ((g.Nb / 2 + grid_size - 1) / grid_size);
    const size_t per_block = (size_t)(Mt ? 8 : 9) * Ns * sizeof(cpx<T>);
    a.ucap = std::max(1, std::min(Mt ? nbg / 2 : nbg, (int)(kLittleStage / per_block)));
    a.tab = nbg <= kMaxOwned;
    const size_t lds = a.ucap * per_block + sizeof(int) * (size_t)(Mt || a.tab ? nbg * (a.tab ? 9 : 1) : 0);
    const void* fn = Mt ? reinterpret_cast<const void*>(&k_little_gcr<T, true>)
                        : reinterpret_cast<const void*>(&k_little_gcr<T, false>);
    static std::once_flag attr[2];
    set_max_lds_once(attr[Mt ? 1 : 0], fn, kLittleDynLds);
    if (!cooperative) {
        if (Mt)
            hipLaunchKernelGGL((k_little_gcr<T, true>), dim3(grid_size), dim3(LT1), lds, s, a);
        else
            hipLaunchKernelGGL((k_little_gcr<T, false>), dim3(grid_size), dim3(LT1), lds, s, a);
        HIPCHECK(hipGetLastError());
        return;
    }
    void* args[] = {&a};
    HIPCHECK(hipLaunchCooperativeKernel(fn, dim3(grid_size), dim3(LT1), args, (unsigned)lds, s));
}

}  // namespace

// The barrier and reduction costs grow with the workgroup count, the apply's
// bandwidth with it. Default four blocks per workgroup: with the even-odd
// operator each apply covers two blocks, one round of the 512 threads for Ns
// up to 32. At most kLittleMaxGrid workgroups. Even-odd solves of up to 512
// blocks: one block pair per workgroup, which for Ns up to 32 the kernel with
// the matrices in registers takes; beyond, in this kernel, 16^4 with Ns = 40
// (256 blocks) 562 us a solve with 128 workgroups, 638 with 64; but oblique
// deflation (Ns = 20) 560 and 544, and the plain operator 643 and 658.
int little_gcr_grid(const Geom& g, int requested, bool eo)
{
    int G = requested > 0 ? requested : eo && g.Nb <= 2 * kLittleMaxGrid ? g.Nb / 2 : g.Nb / 4;
    if (G > kLittleMaxGrid)
        G = kLittleMaxGrid;
    if (G > g.Nb / 2)
        G = g.Nb / 2;
    if (G < 1)
        G = 1;
    return G;
}

int little_gcr_multi_grid(const Geom& g, int requested)
{
    int G = requested > 0 ? 2 * requested : g.Nb / 4;
    if (G > kLittleMaxGridMulti)
        G = kLittleMaxGridMulti;
    if (G > g.Nb / 2)
        G = g.Nb / 2;
    if (G < 1)
        G = 1;
    return G;
}

int little_gcr_resident_limit(bool multi)
{
    int dev = 0, cus = 0;
    HIPCHECK(hipGetDevice(&dev));
    HIPCHECK(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
    int per_cu = 1 << 30;
    auto occ = [&](const void* fn, int threads, size_t lds = 0) {
        int n = 0;
        if (lds)
            HIPCHECK(hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
        HIPCHECK(hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, fn, threads, lds));
        per_cu = n < per_cu ? n : per_cu;
    };
    if (multi) {
        occ(reinterpret_cast<const void*>(&k_little_gcr_multi<double, false>), LT);
        occ(reinterpret_cast<const void*>(&k_little_gcr_multi<float, false>), LT);
        occ(reinterpret_cast<const void*>(&k_little_gcr_multi<double, true>), LT);
        occ(reinterpret_cast<const void*>(&k_little_gcr_multi<float, true>), LT);
    } else {
        occ(reinterpret_cast<const void*>(&k_little_gcr<double, true>), LT1, kLittleDynLds);
        occ(reinterpret_cast<const void*>(&k_little_gcr<double, false>), LT1, kLittleDynLds);
        occ(reinterpret_cast<const void*>(&k_little_gcr<float, true>), LT1, kLittleDynLds);
        occ(reinterpret_cast<const void*>(&k_little_gcr<float, false>), LT1, kLittleDynLds);
        occ(reinterpret_cast<const void*>(&k_little_gcr_pair<double, 24>), LT1);
        occ(reinterpret_cast<const void*>(&k_little_gcr_pair<double, 32>), LT1);
        occ(reinterpret_cast<const void*>(&k_little_gcr_pair<float, 24>), LT1);
        occ(reinterpret_cast<const void*>(&k_little_gcr_pair<float, 32>), LT1);
    }
    return per_cu * cus;
}

bool little_eo_fits(const Geom& g, int grid)
{
    return 2 * ((g.Nb / 2 + grid - 1) / grid) <= kMaxOwned;
}

size_t little_gcr_partial_doubles(int grid_size) { return (size_t)NSLOT * (grid_size + 1) * 2; }

template <typename T>
void launch_little_gcr(const Geom& g, int Ns, int nkv, int maxiter, double tol, const double* tol_dev, const cpx<T>* At,
                       const cpx<T>* Mt, cpx<T>* w1, cpx<T>* w2, const cpx<T>* Q, const cpx<T>* Z, int nq, int oblique,
                       const double* Ainv, const double* Gw, const cpx<T>* w,
                       cpx<T>* x, cpx<T>* r, cpx<T>* xi, cpx<T>* chi, double* part, int* stats,
                       unsigned long long* bar_gen, int grid, hipStream_t s, bool cooperative)
{
    launch_impl<T>(g, Ns, nkv, maxiter, tol, tol_dev, At, Mt, Q, Z, nq, oblique, Ainv, Gw, w, x, r, xi, chi, w1, w2, part,
                   stats, bar_gen, grid, s, cooperative);
}

int little_pair_sources(const Geom& g, int Ns, int grid, int resident)
{
    return 2 * grid == g.Nb && Ns <= 32 ? std::max(1, resident / grid) : 0;
}

size_t little_pair_partial_doubles(int grid) { return (size_t)NSLOT_PAIR * (grid + 1) * 2; }

template <typename T>
void launch_little_gcr_pair(const Geom& g, int Ns, int nkv, int maxiter, double tol, const double* tol_dev,
                            const cpx<T>* Mt, cpx<T>* w1, const cpx<T>* Q, const cpx<T>* Z, int nq, const cpx<T>* w,
                            cpx<T>* x, double* part, int* stats, unsigned long long* bar, int nsrc, hipStream_t s,
                            bool cooperative)
{
    LittleArgs<T> a{};
    a.g = g;
    a.Ns = Ns;
    a.nkv = nkv;
    a.maxiter = maxiter;
    a.tol2 = tol * tol;
    a.tol_dev = tol_dev;
    a.Mt = Mt;
    a.w = w;
    a.x = x;
    a.w1 = w1;
    a.Q = Q;
    a.Z = Z;
    a.nq = Q && Z ? nq : 0;
    a.part = part;
    a.stats = stats;
    a.bar_gen = bar + kLittleFlags;
    const auto pair = Ns <= 24 ? &k_little_gcr_pair<T, 24> : &k_little_gcr_pair<T, 32>;
    const dim3 grid(g.Nb / 2 * nsrc);
    if (!cooperative) {
        hipLaunchKernelGGL(pair, grid, dim3(LT1), 0, s, a);
        HIPCHECK(hipGetLastError());
        return;
    }
    void* args[] = {&a};
    HIPCHECK(hipLaunchCooperativeKernel(reinterpret_cast<const void*>(pair), grid, dim3(LT1), args, 0, s));
}
template void launch_little_gcr_pair<double>(const Geom&, int, int, int, double, const double*, const c64*, c64*,
                                             const c64*, const c64*, int, const c64*, c64*, double*, int*,
                                             unsigned long long*, int, hipStream_t, bool);
template void launch_little_gcr_pair<float>(const Geom&, int, int, int, double, const double*, const c32*, c32*,
                                            const c32*, const c32*, int, const c32*, c32*, double*, int*,
                                            unsigned long long*, int, hipStream_t, bool);

template <typename T>
void launch_little_gcr_multi(const Geom& g, int Ns, int nkv, int maxiter, double tol, const double* tol_dev, int nrhs,
                             const cpx<T>* At, const cpx<T>* Mt, cpx<T>* w1, cpx<T>* w2,
                             const cpx<T>* w, cpx<T>* x, cpx<T>* r, cpx<T>* xi, cpx<T>* chi, double* part, double* fin,
                             double* acoef, int* stats, unsigned* bar_count, unsigned long long* bar_gen, int grid,
                             hipStream_t s, bool cooperative)
{
    if (Mt && !(w1 && w2 && little_eo_fits(g, grid)))
        fail(DFL_EINVAL, "even-odd little solve: missing work vectors or too many blocks per workgroup");
    LittleMultiArgs<T> a;
    a.g = g;
    a.Ns = Ns;
    a.nkv = nkv;
    a.maxiter = maxiter;
    a.nrhs = nrhs;
    a.tol2 = tol * tol;
    a.tol_dev = tol_dev;
    a.At = At;
    a.Mt = Mt;
    a.w1 = w1;
    a.w2 = w2;
    a.w = w;
    a.x = x;
    a.r = r;
    a.xi = xi;
    a.chi = chi;
    a.part = part;
    a.fin = fin;
    a.acoef = acoef;
    a.stats = stats;
    a.bar_count = bar_count;
    a.bar_gen = bar_gen;
    if (!cooperative) {
        if (Mt)
            hipLaunchKernelGGL((k_little_gcr_multi<T, true>), dim3(grid), dim3(LT), 0, s, a);
        else
            hipLaunchKernelGGL((k_little_gcr_multi<T, false>), dim3(grid), dim3(LT), 0, s, a);
        HIPCHECK(hipGetLastError());
        return;
    }
    void* args[] = {&a};
    const void* fn = Mt ? reinterpret_cast<const void*>(&k_little_gcr_multi<T, true>)
                        : reinterpret_cast<const void*>(&k_little_gcr_multi<T, false>);
    HIPCHECK(hipLaunchCooperativeKernel(fn, dim3(grid), dim3(LT), args, 0, s));
}

size_t little_gcr_multi_doubles(int grid_size, int nrhs, size_t* fin, size_t* acoef)
{
    *fin = (size_t)nrhs * RS * 2;
    *acoef = (size_t)grid_size * nrhs * NK * NK * 2;
    return (size_t)NSLOT * nrhs * grid_size * 2;
}

#define INST_MULTI(T)                                                                                               \
    template void launch_little_gcr_multi<T>(const Geom&, int, int, int, double, const double*, int, const cpx<T>*,  \
                                             const cpx<T>*, cpx<T>*, cpx<T>*, const cpx<T>*,                        \
                                             cpx<T>*, cpx<T>*, cpx<T>*, cpx<T>*, double*, double*, double*, int*,    \
                                             unsigned*, unsigned long long*, int, hipStream_t, bool);
INST_MULTI(double)
INST_MULTI(float)
#undef INST_MULTI

template void launch_little_gcr<double>(const Geom&, int, int, int, double, const double*, const c64*, const c64*,
                                        c64*, c64*, const c64*, const c64*, int, int, const double*, const double*,
                                        const c64*, c64*, c64*, c64*, c64*, double*, int*,
                                        unsigned long long*, int, hipStream_t, bool);
template void launch_little_gcr<float>(const Geom&, int, int, int, double, const double*, const c32*, const c32*,
                                       c32*, c32*, const c32*, const c32*, int, int, const double*, const double*,
                                       const c32*, c32*, c32*, c32*, c32*, double*, int*,
                                       unsigned long long*, int, hipStream_t, bool);

}  // namespace dfl
