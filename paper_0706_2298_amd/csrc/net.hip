// Kernels of the start-field network and its training: periodic 3^4
// convolutions (forward, backward to the input, backward to the weights),
// the maps between output channels and quark fields, the block deficit loss
// of eq. (3.15) with its gradient, and the Adam update.
//
// Activations are FP32 planes [C][V] in canonical site order (x0 slowest),
// so a tap's neighbour is a fixed shift of the site index up to the periodic
// wrap. Weights are [81][Cin][Cout], tap t = sum_mu (o_mu + 1) 3^(3 - mu) for
// the offset o in {-1,0,1}^4. Quark fields are native FP64 fields (common.h).
#include <algorithm>
#include <mutex>

#include "internal.h"

namespace dfl {

namespace {

constexpr int kCO = 16;        // output channels per workgroup of the vector convolution
constexpr int kCN = 8;         // its most input channels
constexpr int kWT = 64;        // output channels per workgroup of the weight gradient
constexpr int kWS = 64;        // sites per LDS tile of the weight gradient
constexpr int kMaxCin = 96;

struct Lat {
    int L[4];
    long str[4];  // canonical strides (x3 fastest)
    long V;
    int W3;       // x3 extent of a staged row: L[3], or that of a segment (see Tile)
    int nseg;     // segments of a row, 0: tiles are runs of whole rows' sites
};

// delta[mu][o+1]: index shift of the neighbour x + o mu_hat of site i
__device__ inline void tap_shifts(const Lat& lt, long i, int sign, long delta[4][3])
{
    long rest = i;
    int x[4];
    for (int mu = 3; mu >= 0; --mu) {
        x[mu] = (int)(rest % lt.L[mu]);
        rest /= lt.L[mu];
    }
#pragma unroll
    for (int mu = 0; mu < 4; ++mu) {
#pragma unroll
        for (int o = -1; o <= 1; ++o) {
            int y = x[mu] + sign * o;
            if (y < 0)
                y += lt.L[mu];
            if (y >= lt.L[mu])
                y -= lt.L[mu];
            delta[mu][o + 1] = (long)(y - x[mu]) * lt.str[mu];
        }
    }
}

// canonical index of site x3 on the x3 line `line` = (x0 L1 + x1) L2 + x2
__device__ inline long base_site(const Lat& lt, long line, int x3) { return line * lt.L[3] + x3; }

__device__ inline float silu_f(float z) { return z / (1.0f + __expf(-z)); }
__device__ inline float silu_grad_f(float z)
{
    const float s = 1.0f / (1.0f + __expf(-z));
    return s * (1.0f + z * (1.0f - s));
}

// out[oc][i] = bias[oc] + sum_t sum_ic Wt(t, ic, oc) in[ic][i + s o_t]
//   forward (TRANS = false, s = +1): Wt(t, ic, oc) = W[t][ic][oc], nic = Cin
//   input gradient (TRANS = true, s = -1): Wt(t, ic, oc) = W[t][oc][ic], nic = Cout of W
// Epilogue: forward stores z and optionally a = silu(z); the input gradient
// is optionally multiplied by silu'(zprev[oc][i]).
// The vector kernel, for few input channels on many sites (launch_conv), where
// the matrix-core kernel spends its time on staging 32 channels that are not there.
template <bool TRANS>
__global__ __launch_bounds__(256) void k_conv(Lat lt, const float* __restrict__ in, int nic,
                                              const float* __restrict__ W, int w_cin, int w_cout,
                                              const float* __restrict__ bias, int noc, float* __restrict__ out,
                                              float* __restrict__ act, const float* __restrict__ zprev)
{
    __shared__ float4 ws[576 * kCO / 4];  // (with room for kCN channels only the channel loop compiles to a slower form)
    const long V = lt.V;
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    const int oc0 = blockIdx.y * kCO;
    long dl[4][3];
    if (i < V)
        tap_shifts(lt, i, TRANS ? -1 : 1, dl);
    float acc[kCO];
#pragma unroll
    for (int j = 0; j < kCO; ++j)
        acc[j] = (bias && oc0 + j < noc) ? bias[oc0 + j] : 0.f;
    float* wsf = reinterpret_cast<float*>(ws);
    for (int t = 0; t < 81; ++t) {
        __syncthreads();
        for (int e = threadIdx.x; e < nic * kCO; e += blockDim.x) {
            int ic, j;
            if (TRANS) {
                ic = e % nic;
                j = e / nic;
            } else {
                ic = e / kCO;
                j = e % kCO;
            }
            float w = 0.f;
            if (oc0 + j < noc)
                w = TRANS ? W[((long)t * w_cin + oc0 + j) * w_cout + ic] : W[((long)t * w_cin + ic) * w_cout + oc0 + j];
            wsf[ic * kCO + j] = w;
        }
        __syncthreads();
        if (i < V) {
            const int o0 = t / 27, o1 = (t / 9) % 3, o2 = (t / 3) % 3, o3 = t % 3;
            const long nb = i + dl[0][o0] + dl[1][o1] + dl[2][o2] + dl[3][o3];
            const float* src = in + nb;
            for (int ic = 0; ic < nic; ++ic) {
                const float x = src[(long)ic * V];
#pragma unroll
                for (int q = 0; q < kCO / 4; ++q) {
                    const float4 w = ws[ic * (kCO / 4) + q];
                    acc[4 * q] += x * w.x;
                    acc[4 * q + 1] += x * w.y;
                    acc[4 * q + 2] += x * w.z;
                    acc[4 * q + 3] += x * w.w;
                }
            }
        }
    }
    if (i >= V)
        return;
#pragma unroll
    for (int j = 0; j < kCO; ++j) {
        if (oc0 + j >= noc)
            continue;
        float v = acc[j];
        if (TRANS && zprev)
            v *= silu_grad_f(zprev[(long)(oc0 + j) * V + i]);
        out[(long)(oc0 + j) * V + i] = v;
        if (!TRANS && act)
            act[(long)(oc0 + j) * V + i] = silu_f(v);
    }
}

// ------------------------------------------------------- staged site tiles
//
// The matrix-core convolutions work on tiles of T consecutive canonical sites.
// For a pair of offsets (o0, o1) the tile's rows along x3, each with its two
// neighbours along x3, and the rows x2 - 1 and x2 + 1 around every run of rows
// of one (x0, x1) plane are staged in LDS ("slots" of L3 + 2 positions); all
// nine taps (o2, o3) then read the same staged values at a constant shift of
// o2 (L3 + 2) + o3 positions. Any lattice works: a tile may start inside a
// row and cross planes. Where long rows make that halo too large (more than
// kCPos positions), a tile is a segment of one row instead, the shortest of
// equal parts of at most T sites, staged with its neighbours only (slots of
// W3 + 2 positions).
struct Tile {
    long site0;   // first site
    int n;        // sites (T, fewer at the end of the lattice or in segments)
    int x3_0;     // x3 of the slots' first site
    int x2_0;     // x2 of the first row
    int plane0;   // its plane x0 L1 + x1
    int slots;    // staged rows
};
__device__ inline Tile make_tile(const Lat& lt, long tile, int T)
{
    Tile t;
    t.x3_0 = 0;
    if (lt.nseg) {
        const long row = tile / lt.nseg;
        t.x3_0 = (int)(tile - row * lt.nseg) * lt.W3;
        t.site0 = row * lt.L[3] + t.x3_0;
        t.n = lt.L[3] - t.x3_0 < lt.W3 ? lt.L[3] - t.x3_0 : lt.W3;
    } else {
        t.site0 = tile * T;
        t.n = (int)(lt.V - t.site0 < T ? lt.V - t.site0 : T);
    }
    const long r0 = t.site0 / lt.L[3], r1 = (t.site0 + t.n - 1) / lt.L[3];
    t.plane0 = (int)(r0 / lt.L[2]);
    t.x2_0 = (int)(r0 - (long)t.plane0 * lt.L[2]);
    const int pl1 = (int)(r1 / lt.L[2]);
    const int x2_1 = (int)(r1 - (long)pl1 * lt.L[2]);
    t.slots = (pl1 - t.plane0) * (lt.L[2] + 2) + x2_1 - t.x2_0 + 3;
    return t;
}
// staged position of site i of the tile
__device__ inline int tile_pos(const Lat& lt, const Tile& t, int i)
{
    const long s = t.site0 + i;
    const long r = s / lt.L[3];
    const int x3 = (int)(s - r * lt.L[3]) - t.x3_0;
    const int pl = (int)(r / lt.L[2]);
    const int x2 = (int)(r - (long)pl * lt.L[2]);
    return ((pl - t.plane0) * (lt.L[2] + 2) + x2 + 1 - t.x2_0) * (lt.W3 + 2) + x3 + 1;
}
// a staged position's source: x0, x1 of its plane and the index in the plane
struct Src {
    int x0, x1, in_plane;
};
__device__ inline Src pos_source(const Lat& lt, const Tile& t, int p)
{
    const int w3 = lt.W3 + 2, w2 = lt.L[2] + 2;
    const int slot = p / w3;
    int x3 = t.x3_0 + p - slot * w3 - 1;
    x3 = x3 < 0 ? x3 + lt.L[3] : (x3 >= lt.L[3] ? x3 - lt.L[3] : x3);
    const int u = slot + t.x2_0;
    const int seg = u / w2;
    int x2 = u - seg * w2 - 1;
    x2 = x2 < 0 ? x2 + lt.L[2] : (x2 >= lt.L[2] ? x2 - lt.L[2] : x2);
    const int pl = t.plane0 + seg;
    Src r;
    r.x0 = pl / lt.L[1];
    r.x1 = pl - r.x0 * lt.L[1];
    r.in_plane = x2 * lt.L[3] + x3;
    return r;
}
// canonical index of the source in the plane (x0 + d0, x1 + d1)
__device__ inline long src_site(const Lat& lt, const Src& r, int d0, int d1)
{
    int y0 = r.x0 + d0, y1 = r.x1 + d1;
    y0 = y0 < 0 ? y0 + lt.L[0] : (y0 >= lt.L[0] ? y0 - lt.L[0] : y0);
    y1 = y1 < 0 ? y1 + lt.L[1] : (y1 >= lt.L[1] ? y1 - lt.L[1] : y1);
    return (long)y0 * lt.str[0] + (long)y1 * lt.str[1] + r.in_plane;
}

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// k_conv's map on the matrix cores (v_mfma_f32_32x32x2f32, FP32 products and sums), one GEMM
// per tap: out[oc][x] += sum_ic Wt(t, ic, oc) in[ic][x + s o_t].
// Workgroup: a tile of 128 sites and 32 OT output channels, wavefront w the
// sites 32 w .. 32 w + 31 of all of them. For each (o0, o1) and each chunk of
// 32 input channels the tile is staged as [position][channel], and the weights
// of three taps at a time as [tap][output channel][channel], both with a row of
// 36 floats: a lane's four consecutive channels are one 16-byte LDS read that
// feeds four instructions, and eight neighbouring rows cover all banks. Of the
// instruction's two contraction steps the lower lanes take the first and the
// upper lanes the second four of eight channels, for both operands alike.
// Lane l supplies A[l % 32][l / 32] and B[l / 32][l % 32] and holds
// C[8 (i / 4) + 4 (l / 32) + i % 4][l % 32], i < 16.
// Bound by the matrix cores: a workgroup step of nine taps is 9216 OT matrix
// cycles against some 60 staged values per thread, and two or three workgroups
// per CU cover each other's staging. The next three taps' weights are loaded
// into registers while three are multiplied (32 -> 32 channels 10% faster).
// MI355X, 16^4: 32 -> 576 channels 1.88 ms = 104 TFLOP/s (vector kernel 4.14
// ms), 576 -> 32 (input gradient) 2.06 ms = 95 TFLOP/s (8.97 ms), 32 -> 32
// 0.12 ms (0.31 ms); a large FP32 matrix product reaches 154 TFLOP/s.
constexpr int kCT = 128;  // sites per tile
constexpr int kCPos = 512;  // most staged positions (two per thread)
constexpr int kCK = 32;   // input channels per LDS chunk
constexpr int kCP = 36;   // LDS row stride in floats
template <bool TRANS, int OT>
__global__ __launch_bounds__(256, 2) void k_conv_mfma(Lat lt, int ntiles, const float* __restrict__ in, int nic,
                                                      const float* __restrict__ W, int w_cin, int w_cout,
                                                      const float* __restrict__ bias, int noc, int npos,
                                                      float* __restrict__ out, float* __restrict__ act,
                                                      const float* __restrict__ zprev)
{
    constexpr int OCT = 32 * OT;
    extern __shared__ float4 conv_lds[];
    float* xs = reinterpret_cast<float*>(conv_lds);  // [npos][kCP]
    float* ws = xs + npos * kCP;                     // [3][OCT][kCP]
    const int tile_id = xcd_remap(blockIdx.x, gridDim.x);
    if (tile_id >= ntiles)
        return;
    const int sgn = TRANS ? -1 : 1;
    const Tile tl = make_tile(lt, tile_id, kCT);
    const int w3 = lt.W3 + 2;
    const int np = tl.slots * w3;
    const int oc0 = blockIdx.y * OCT;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int col = lane & 31, kh = lane >> 5;
    // this thread's staged positions (npos <= kCPos)
    Src src[2];
#pragma unroll
    for (int k = 0; k < 2; ++k)
        src[k] = pos_source(lt, tl, tid + 256 * k < np ? tid + 256 * k : 0);
    const int my = w * 32 + col;  // this lane's site in the tile
    const float* xb = xs + tile_pos(lt, tl, my < tl.n ? my : 0) * kCP + 4 * kh;
    const float* wb = ws + col * kCP + 4 * kh;
    f32x16 acc[OT];
#pragma unroll
    for (int ot = 0; ot < OT; ++ot)
#pragma unroll
        for (int i = 0; i < 16; ++i)
            acc[ot][i] = 0.f;
    // the weights of three taps (from tap t0 on) and a channel chunk, four channels a piece: loaded into
    // registers while the previous taps are multiplied, then stored to LDS
    constexpr int NW = 3 * OT;
    f32x4 wr[NW];
    auto w_place = [&](int k, int& c, int& j, int& q) {  // first channel, output channel, tap of piece k
        const int e = tid + 256 * k;
        if (TRANS) {  // channels are contiguous in W
            c = (e % (kCK / 4)) * 4;
            j = (e / (kCK / 4)) % OCT;
            q = e / (kCK / 4 * OCT);
        } else {  // output channels are
            j = e % OCT;
            c = (e / OCT) % (kCK / 4) * 4;
            q = e / (OCT * (kCK / 4));
        }
    };
    int woff[NW];  // of its first channel, from the chunk's first entry
#pragma unroll
    for (int k = 0; k < NW; ++k) {
        int c, j, q;
        w_place(k, c, j, q);
        woff[k] = TRANS ? (q * w_cin + j) * w_cout + c : (q * w_cin + c) * w_cout + j;
    }
    const int wstep = TRANS ? 1 : w_cout;
    auto load_weights = [&](int t0, int c0) {
        const float* wp = W + (TRANS ? ((long)t0 * w_cin + oc0) * w_cout + c0 : ((long)t0 * w_cin + c0) * w_cout + oc0);
        if (c0 + kCK <= nic && oc0 + OCT <= noc) {
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int k = 0; k < NW; ++k)
                    wr[k][i] = (wp + i * wstep)[woff[k]];
        } else {
#pragma unroll
            for (int k = 0; k < NW; ++k) {
                int c, j, q;
                w_place(k, c, j, q);
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    wr[k][i] = c0 + c + i < nic && oc0 + j < noc ? (wp + i * wstep)[woff[k]] : 0.f;
            }
        }
    };
    load_weights(0, 0);
    for (int l01 = 0; l01 < 9; ++l01) {
        const int o0 = l01 / 3 - 1, o1 = l01 % 3 - 1;
        for (int c0 = 0; c0 < nic; c0 += kCK) {
            const int nc = nic - c0 < kCK ? nic - c0 : kCK;
            const int nj = (nc + 7) / 8;  // groups of eight channels
            __syncthreads();              // the previous chunk's operands are consumed
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const int p = tid + 256 * k;
                if (p < np) {
                    const float* q = in + (long)c0 * lt.V + src_site(lt, src[k], sgn * o0, sgn * o1);
                    if (nc == kCK) {
#pragma unroll
                        for (int c = 0; c < kCK; c += 4) {
                            const f32x4 v = {q[(long)c * lt.V], q[(long)(c + 1) * lt.V], q[(long)(c + 2) * lt.V],
                                             q[(long)(c + 3) * lt.V]};
                            *reinterpret_cast<f32x4*>(xs + p * kCP + c) = v;
                        }
                    } else {
                        for (int c = 0; c < 8 * nj; c += 4) {
                            f32x4 v;
#pragma unroll
                            for (int e = 0; e < 4; ++e)
                                v[e] = c + e < nc ? q[(long)(c + e) * lt.V] : 0.f;
                            *reinterpret_cast<f32x4*>(xs + p * kCP + c) = v;
                        }
                    }
                }
            }
            for (int o2 = -1; o2 <= 1; ++o2) {
                if (o2 > -1)
                    __syncthreads();  // the previous taps' weights are consumed
#pragma unroll
                for (int k = 0; k < NW; ++k) {
                    int c, j, q;
                    w_place(k, c, j, q);
                    *reinterpret_cast<f32x4*>(ws + (q * OCT + j) * kCP + c) = wr[k];
                }
                __syncthreads();
                const int t0 = l01 * 9 + (o2 + 1) * 3;
                if (o2 < 1)
                    load_weights(t0 + 3, c0);
                else if (c0 + kCK < nic)
                    load_weights(l01 * 9, c0 + kCK);
                else if (l01 < 8)
                    load_weights(t0 + 3, 0);
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                    const float* xt = xb + sgn * (o2 * w3 + q - 1) * kCP;
                    const float* wt = wb + q * OCT * kCP;
                    auto step = [&](int j) {
                        const f32x4 b = *reinterpret_cast<const f32x4*>(xt + 8 * j);
                        f32x4 a[OT];
#pragma unroll
                        for (int ot = 0; ot < OT; ++ot)
                            a[ot] = *reinterpret_cast<const f32x4*>(wt + ot * 32 * kCP + 8 * j);
#pragma unroll
                        for (int k = 0; k < 4; ++k)
#pragma unroll
                            for (int ot = 0; ot < OT; ++ot)
                                acc[ot] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[ot][k], b[k], acc[ot], 0, 0, 0);
                    };
                    if (nj == kCK / 8) {
#pragma unroll
                        for (int j = 0; j < kCK / 8; ++j)
                            step(j);
                    } else {
                        for (int j = 0; j < nj; ++j)
                            step(j);
                    }
                }
            }
        }
    }
    if (my >= tl.n)
        return;
    const long site = tl.site0 + my;
#pragma unroll
    for (int ot = 0; ot < OT; ++ot)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int oc = oc0 + ot * 32 + 8 * (i / 4) + 4 * kh + i % 4;
            if (oc >= noc)
                continue;
            float v = acc[ot][i] + (bias ? bias[oc] : 0.f);
            if (TRANS && zprev)
                v *= silu_grad_f(zprev[(long)oc * lt.V + site]);
            out[(long)oc * lt.V + site] = v;
            if (!TRANS && act)
                act[(long)oc * lt.V + site] = silu_f(v);
        }
}

// Forward map with BF16 operands on the matrix cores, for lattices whose rows are
// too long for the staged tiles of k_conv_bf16_tile or where its rounded input
// finds no room: inputs and weights
// rounded to BF16 (nearest even), products summed in FP32
// (v_mfma_f32_16x16x32_bf16), bias and activation in FP32. The weights come
// pre-converted as Wb[t][oc][ic] (ic padded to a multiple of 32 and oc to
// the channel tile with zeros), so a tap's 32-channel chunk is a straight
// 16-byte copy into LDS. Workgroup: kBNL consecutive x2 lines of kBTS sites
// along x3 (one line per wavefront) and 16 OT output channels; every
// wavefront keeps OT x 2 tiles of 16 x 16 accumulators, so one staged
// operand row feeds two (weights) or OT (inputs) instructions. For each of
// the 27 neighbour line offsets (o0, o1, o2) and each 32-channel chunk the
// four lines' segments with their +-1 halo along x3 and the three taps'
// weights (o3 = -1, 0, 1) are staged; the taps read the segments at shifts
// of one site. Lane l supplies A[l % 16][8 (l / 16) + j] and
// B[8 (l / 16) + j][l % 16], j < 8 (the contraction index is summed, so
// only its being the same for A and B matters) and holds
// C[4 (l / 16) + i][l % 16], i < 4.
// round-to-nearest-even float -> bfloat16 bits (finite inputs)
__device__ inline uint32_t bf16_bits(float f)
{
    uint32_t u = __float_as_uint(f);
    u += 0x7fffu + ((u >> 16) & 1u);
    return u >> 16;
}

constexpr int kBTS = 32;       // sites per line segment
constexpr int kBNL = 4;        // x2 lines per workgroup (one per wavefront)
constexpr int kBK = 32;        // input channels per chunk (the instruction's K)
constexpr int kBRow = kBK + 8; // LDS row stride in BF16 elements (80 bytes)
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned short u16x8 __attribute__((ext_vector_type(8)));

template <int OT>
__global__ __launch_bounds__(256) void k_conv_bf16(Lat lt, const float* __restrict__ in, int cin, int cinP,
                                                   const uint16_t* __restrict__ Wb, int coutP,
                                                   const float* __restrict__ bias, int cout, float* __restrict__ out,
                                                   float* __restrict__ act)
{
    constexpr int OCT = 16 * OT;
    __shared__ __attribute__((aligned(16))) uint16_t xs[kBNL][kBTS + 2][kBRow];
    __shared__ __attribute__((aligned(16))) uint16_t ws[3][OCT][kBRow];
    typedef float f4 __attribute__((ext_vector_type(4)));
    const long V = lt.V;
    const int n_oct = coutP / OCT;
    const long grp = blockIdx.x / n_oct;  // channel tiles of one site group are adjacent
    const int oc0 = (int)(blockIdx.x - grp * n_oct) * OCT;
    const int nseg = lt.L[3] / kBTS, ngx2 = lt.L[2] / kBNL;
    long r = grp;
    const int seg = (int)(r % nseg);
    r /= nseg;
    const int x2g = (int)(r % ngx2) * kBNL;
    r /= ngx2;
    const int x1 = (int)(r % lt.L[1]);
    const int x0 = (int)(r / lt.L[1]);
    const int x3_0 = seg * kBTS;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int kr = lane >> 4, kc = lane & 15;
    f4 acc[OT][2];
#pragma unroll
    for (int ot = 0; ot < OT; ++ot)
        acc[ot][0] = acc[ot][1] = f4{0.f, 0.f, 0.f, 0.f};
    for (int l = 0; l < 27; ++l) {
        const int o0 = l / 9 - 1, o1 = (l / 3) % 3 - 1, o2 = l % 3 - 1;
        int y0 = x0 + o0, y1 = x1 + o1;
        y0 = y0 < 0 ? y0 + lt.L[0] : (y0 >= lt.L[0] ? y0 - lt.L[0] : y0);
        y1 = y1 < 0 ? y1 + lt.L[1] : (y1 >= lt.L[1] ? y1 - lt.L[1] : y1);
        const long base01 = (long)y0 * lt.str[0] + (long)y1 * lt.str[1];
        for (int c0 = 0; c0 < cinP; c0 += kBK) {
            __syncthreads();  // the previous chunk's operands are consumed
            for (int e = threadIdx.x; e < kBNL * kBK * (kBTS + 2); e += 256) {
                const int j = e % (kBTS + 2);
                const int rest = e / (kBTS + 2);
                const int ic = rest % kBK, ln = rest / kBK;
                int y2 = x2g + ln + o2;
                y2 = y2 < 0 ? y2 + lt.L[2] : (y2 >= lt.L[2] ? y2 - lt.L[2] : y2);
                int y3 = x3_0 - 1 + j;
                y3 = y3 < 0 ? y3 + lt.L[3] : (y3 >= lt.L[3] ? y3 - lt.L[3] : y3);
                const float v = c0 + ic < cin ? in[(long)(c0 + ic) * V + base01 + (long)y2 * lt.str[2] + y3] : 0.f;
                xs[ln][j][ic] = (uint16_t)bf16_bits(v);
            }
            for (int e = threadIdx.x; e < 3 * OCT * (kBK / 8); e += 256) {
                const int v8 = e % (kBK / 8);
                const int rest = e / (kBK / 8);
                const int oc = rest % OCT, q = rest / OCT;
                const long t = l * 3 + q;  // tap of (o0, o1, o2, o3 = q - 1)
                *reinterpret_cast<u16x8*>(&ws[q][oc][8 * v8]) =
                    *reinterpret_cast<const u16x8*>(Wb + (t * coutP + oc0 + oc) * cinP + c0 + 8 * v8);
            }
            __syncthreads();
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                // the neighbour x3 + (q - 1) of segment site i sits in staged column i + q
                bf16x8 b[2];
#pragma unroll
                for (int st = 0; st < 2; ++st)
                    b[st] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u16x8*>(&xs[w][st * 16 + kc + q][8 * kr]));
#pragma unroll
                for (int ot = 0; ot < OT; ++ot) {
                    const bf16x8 a = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u16x8*>(&ws[q][ot * 16 + kc][8 * kr]));
#pragma unroll
                    for (int st = 0; st < 2; ++st)
                        acc[ot][st] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b[st], acc[ot][st], 0, 0, 0);
                }
            }
        }
    }
    const long line = ((long)x0 * lt.L[1] + x1) * lt.L[2] + x2g + w;
#pragma unroll
    for (int ot = 0; ot < OT; ++ot)
#pragma unroll
        for (int st = 0; st < 2; ++st) {
            const long site = base_site(lt, line, x3_0 + st * 16 + kc);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int oc = oc0 + ot * 16 + 4 * kr + i;
                if (oc >= cout)
                    continue;
                const float v = acc[ot][st][i] + (bias ? bias[oc] : 0.f);
                out[(long)oc * V + site] = v;
                if (act)
                    act[(long)oc * V + site] = silu_f(v);
            }
        }
}

// The BF16 forward map on staged site tiles (see make_tile), with
// v_mfma_f32_32x32x16_bf16. The input comes rounded and site-major, Xb[site][ic]
// (k_planes_bf16), the weights rounded and in operand order (k_weights_frag):
// 64 lanes of eight channels per (tap, sixteen input channels, 32 output
// channels), which the wavefronts read straight into registers, one tap ahead
// of their use. Workgroup: a tile of 128 NS sites and 32 OT output channels,
// wavefront w the sites 32 NS w .. of all of them, so that an operand read
// feeds OT or NS instructions. Staged rows have 40 entries (80 bytes): eight
// neighbouring positions' 16-byte reads cover all banks.
// With NS = 4 and OT = 2 a tap and 32 channels are 16 instructions of 32 cycles
// per wavefront against 8 KB of LDS reads, half of the LDS's time. MI355X, 32 ->
// 576 channels on 64 x 32^3: 7.9 ms = 790 TFLOP/s with the rounding pass
// (k_conv_bf16: 23.4 ms); a large BF16 matrix product reaches 1180.
template <int OT, int NS>
__global__ __launch_bounds__(256, 2) void k_conv_bf16_tile(Lat lt, int ntiles, const uint16_t* __restrict__ Xb,
                                                           int cinP, const u16x8* __restrict__ Wf, int noct,
                                                           const float* __restrict__ bias, int cout, int npos,
                                                           float* __restrict__ out, float* __restrict__ act)
{
    constexpr int T = 128 * NS;
    extern __shared__ float4 conv_lds[];
    uint16_t* xs = reinterpret_cast<uint16_t*>(conv_lds);        // [npos][kBRow]
    int2* tab = reinterpret_cast<int2*>(xs + (size_t)npos * kBRow);  // source of every position
    const int tile_id = xcd_remap(blockIdx.x, gridDim.x);
    if (tile_id >= ntiles)
        return;
    const Tile tl = make_tile(lt, tile_id, T);
    const int w3 = lt.W3 + 2;
    const int np = tl.slots * w3;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int col = lane & 31, kh = lane >> 5;
    const int oct0 = blockIdx.y * OT;
    for (int p = tid; p < np; p += 256) {
        const Src r = pos_source(lt, tl, p);
        tab[p] = make_int2(r.x0 << 16 | r.x1, r.in_plane);
    }
    const uint16_t* xb[NS];
#pragma unroll
    for (int st = 0; st < NS; ++st) {
        const int i = (w * NS + st) * 32 + col;
        xb[st] = xs + tile_pos(lt, tl, i < tl.n ? i : 0) * kBRow + 8 * kh;
    }
    const int nk = cinP / 16;
    u16x8 a[2][OT], an[2][OT];  // weights of this tap and of the next one
    auto load_a = [&](int t, int c0) {
        const u16x8* q = Wf + (((long)t * nk + c0 / 16) * noct + oct0) * 64 + lane;
#pragma unroll
        for (int kk = 0; kk < 2; ++kk)
#pragma unroll
            for (int ot = 0; ot < OT; ++ot)
                an[kk][ot] = q[(kk * noct + ot) * 64];
    };
    load_a(0, 0);
    f32x16 acc[OT][NS];
#pragma unroll
    for (int ot = 0; ot < OT; ++ot)
#pragma unroll
        for (int st = 0; st < NS; ++st)
#pragma unroll
            for (int i = 0; i < 16; ++i)
                acc[ot][st][i] = 0.f;
    for (int c0 = 0; c0 < cinP; c0 += kBK)
        for (int l01 = 0; l01 < 9; ++l01) {
            const int o0 = l01 / 3 - 1, o1 = l01 % 3 - 1;
            __syncthreads();  // the table is written, the previous operands are consumed
            for (int e = tid; e < np * 4; e += 256) {
                const int2 s = tab[e >> 2];
                const Src r{s.x >> 16, s.x & 0xffff, s.y};
                *reinterpret_cast<u16x8*>(xs + (e >> 2) * kBRow + (e & 3) * 8) =
                    *reinterpret_cast<const u16x8*>(Xb + src_site(lt, r, o0, o1) * cinP + c0 + (e & 3) * 8);
            }
            __syncthreads();
            for (int o2 = -1; o2 <= 1; ++o2) {
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                    const int t = l01 * 9 + (o2 + 1) * 3 + q;
#pragma unroll
                    for (int kk = 0; kk < 2; ++kk)
#pragma unroll
                        for (int ot = 0; ot < OT; ++ot)
                            a[kk][ot] = an[kk][ot];
                    if (t < 80)
                        load_a(t + 1, c0);
                    else if (c0 + kBK < cinP)
                        load_a(0, c0 + kBK);
#pragma unroll
                    for (int kk = 0; kk < 2; ++kk)
#pragma unroll
                        for (int st = 0; st < NS; ++st) {
                            const bf16x8 b = __builtin_bit_cast(
                                bf16x8, *reinterpret_cast<const u16x8*>(xb[st] + (o2 * w3 + q - 1) * kBRow + 16 * kk));
#pragma unroll
                            for (int ot = 0; ot < OT; ++ot)
                                acc[ot][st] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                                    __builtin_bit_cast(bf16x8, a[kk][ot]), b, acc[ot][st], 0, 0, 0);
                        }
                }
            }
        }
#pragma unroll
    for (int ot = 0; ot < OT; ++ot)
#pragma unroll
        for (int st = 0; st < NS; ++st) {
            const int k = (w * NS + st) * 32 + col;
            if (k >= tl.n)
                continue;
            const long site = tl.site0 + k;
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int oc = (oct0 + ot) * 32 + 8 * (i / 4) + 4 * kh + i % 4;
                if (oc >= cout)
                    continue;
                const float v = acc[ot][st][i] + (bias ? bias[oc] : 0.f);
                out[(long)oc * lt.V + site] = v;
                if (act)
                    act[(long)oc * lt.V + site] = silu_f(v);
            }
        }
}

// Xb[site][ic] = bf16(in[ic][site]), ic padded to cinP with zeros: one thread
// per site and eight channels (grid: 64 sites x cinP / 32)
__global__ __launch_bounds__(256) void k_planes_bf16(const float* __restrict__ in, int cin, int cinP, long V,
                                                     uint16_t* __restrict__ Xb)
{
    const long site = (long)blockIdx.x * 64 + (threadIdx.x & 63);
    const int c0 = blockIdx.y * 32 + (threadIdx.x >> 6) * 8;
    if (site >= V)
        return;
    u16x8 v;
#pragma unroll
    for (int j = 0; j < 8; ++j)
        v[j] = (uint16_t)bf16_bits(c0 + j < cin ? in[(long)(c0 + j) * V + site] : 0.f);
    *reinterpret_cast<u16x8*>(Xb + site * cinP + c0) = v;
}

// Wf[((t nk + k) noct + o) 64 + lane][j] = bf16(W[t][16 k + 8 (lane / 32) + j][32 o + lane % 32]),
// zero beyond the channels: the weights in the operand order of k_conv_bf16_tile
__global__ __launch_bounds__(256) void k_weights_frag(const float* __restrict__ W, int cin, int cout, int nk, int noct,
                                                      u16x8* __restrict__ Wf)
{
    const long e = (long)blockIdx.x * 256 + threadIdx.x;
    if (e >= 81L * nk * noct * 64)
        return;
    const int lane = (int)(e & 63);
    long r = e >> 6;
    const int oc = (int)(r % noct) * 32 + (lane & 31);
    r /= noct;
    const int ic = (int)(r % nk) * 16 + 8 * (lane >> 5);
    const long t = r / nk;
    u16x8 v;
#pragma unroll
    for (int j = 0; j < 8; ++j)
        v[j] = (uint16_t)bf16_bits(ic + j < cin && oc < cout ? W[(t * cin + ic + j) * cout + oc] : 0.f);
    Wf[e] = v;
}

// Wb[t][oc][ic] = bf16(W[t][ic][oc]) on the padded [81][coutP][cinP] grid (zeros outside)
__global__ __launch_bounds__(256) void k_weights_bf16(const float* __restrict__ W, int cin, int cout, int cinP,
                                                      int coutP, uint16_t* __restrict__ Wb)
{
    const long e = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= 81L * coutP * cinP)
        return;
    const int ic = (int)(e % cinP);
    const long rest = e / cinP;
    const int oc = (int)(rest % coutP);
    const long t = rest / coutP;
    const float v = (ic < cin && oc < cout) ? W[(t * cin + ic) * cout + oc] : 0.f;
    Wb[e] = (uint16_t)bf16_bits(v);
}

// Weight gradient on the matrix cores (v_mfma_f32_32x32x2f32), partial over a
// range of tiles: part[r][t][ci][co] = sum_y in[ci][y + o_t] g[co][y].
// Workgroup (o0, o1; 32 input channels; 32 or, PAIR, 64 output channels; range
// of tiles): per tile the input is staged with its halo as for the forward map
// and g as [site][output channel]. Six wavefronts: o2 = w % 3 - 1, each with
// the accumulators of the three taps o3; w / 3 selects the output channels
// 32 (w / 3) .. or, without PAIR, half of the sites of every tile, whose sums
// are a partial of their own (r = 2 range + w / 3). The contraction runs over
// the sites, two per instruction; lanes are channels, so every LDS read is a
// run of 32 consecutive floats. Sums run over at most kWF tiles before they are
// added to the range's, which keeps the rounding error below that of one long
// chain (32 -> 576 channels on 16^4: 1.9e-6 of the gradient with one chain).
// Bound by the matrix cores: five LDS reads of two cycles feed three
// instructions of 64. MI355X, 16^4: 32 -> 576 channels 2.50 ms = 78 TFLOP/s
// where the vector kernel took 42.9 ms, 96 -> 32 0.48 ms (14.4 ms). At most 128
// registers, so that twelve wavefronts share a CU (136: 25% slower).
constexpr int kWF = 8;
template <bool PAIR>
__global__ __launch_bounds__(384, 4) void k_conv_wgrad_mfma(Lat lt, const float* __restrict__ in, int cin,
                                                            const float* __restrict__ g, int cout, int tiles,
                                                            int npos, float* __restrict__ part)
{
    constexpr int CO = PAIR ? 64 : 32;
    constexpr int GP = CO + 4;                       // LDS row stride of g
    constexpr int NK = (PAIR ? kCT : kCT / 2) / 2;   // instructions per tap and tile
    extern __shared__ float4 conv_lds[];
    float* xs = reinterpret_cast<float*>(conv_lds);  // [npos][kCP]
    float* gs = xs + npos * kCP;                     // [kCT][GP]
    int* ptab = reinterpret_cast<int*>(gs + kCT * GP);  // [kCT] staged offset of every site
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int col = lane & 31, kh = lane >> 5;
    const int nct = (cin + 31) / 32;
    const int l01 = blockIdx.x % 9, ci0 = blockIdx.x / 9 % nct * 32, co0 = blockIdx.x / 9 / nct * CO;
    const int o0 = l01 / 3 - 1, o1 = l01 % 3 - 1;
    const int o2 = w % 3 - 1, half = w / 3;
    const int w3 = lt.W3 + 2;
    const int nc = cin - ci0 < 32 ? cin - ci0 : 32;
    const int ntiles = (int)((lt.V + kCT - 1) / kCT);
    const int tile1 = min(ntiles, (int)(blockIdx.y + 1) * tiles);
    f32x16 acc[3], sum[3];
#pragma unroll
    for (int q = 0; q < 3; ++q)
#pragma unroll
        for (int i = 0; i < 16; ++i)
            acc[q][i] = sum[q][i] = 0.f;
    const int it0 = blockIdx.y * tiles;
    for (int it = it0; it < tile1; ++it) {
        if (it > it0 && (it - it0) % kWF == 0) {
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                sum[q] += acc[q];
#pragma unroll
                for (int i = 0; i < 16; ++i)
                    acc[q][i] = 0.f;
            }
        }
        const Tile tl = make_tile(lt, it, kCT);
        const int np = tl.slots * w3;
        __syncthreads();  // the previous tile's operands are consumed
        for (int p = tid; p < np; p += 384) {
            const float* q = in + (long)ci0 * lt.V + src_site(lt, pos_source(lt, tl, p), o0, o1);
            if (nc == 32) {
#pragma unroll
                for (int c = 0; c < 32; c += 4) {
                    const f32x4 v = {q[(long)c * lt.V], q[(long)(c + 1) * lt.V], q[(long)(c + 2) * lt.V],
                                     q[(long)(c + 3) * lt.V]};
                    *reinterpret_cast<f32x4*>(xs + p * kCP + c) = v;
                }
            } else {
                for (int c = 0; c < 32; c += 4) {
                    f32x4 v;
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        v[e] = c + e < nc ? q[(long)(c + e) * lt.V] : 0.f;
                    *reinterpret_cast<f32x4*>(xs + p * kCP + c) = v;
                }
            }
        }
        for (int e = tid; e < kCT * (CO / 4); e += 384) {
            const int i = e % kCT, c = e / kCT * 4;
            f32x4 v;
#pragma unroll
            for (int k = 0; k < 4; ++k)
                v[k] = i < tl.n && co0 + c + k < cout ? g[(long)(co0 + c + k) * lt.V + tl.site0 + i] : 0.f;
            *reinterpret_cast<f32x4*>(gs + i * GP + c) = v;
        }
        if (tid < kCT)
            ptab[tid] = tile_pos(lt, tl, tid < tl.n ? tid : 0) * kCP;
        __syncthreads();
        const float* xb = xs + o2 * w3 * kCP + col;
        const float* gb = gs + (PAIR ? half * 32 : 0) + col;
        const int s0 = PAIR ? 0 : half * (kCT / 2), k0 = s0 + kh;  // first site of this lane
        const int nk = min(NK, (tl.n - s0) / 2);  // (V, hence tl.n, is a multiple of 64)
#pragma unroll 4
        for (int k = 0; k < nk; ++k) {
            const int i = k0 + 2 * k;
            const float* xp = xb + ptab[i];
            const float b = gb[i * GP];
#pragma unroll
            for (int q = 0; q < 3; ++q)
                acc[q] = __builtin_amdgcn_mfma_f32_32x32x2f32(xp[(q - 1) * kCP], b, acc[q], 0, 0, 0);
        }
    }
    const int co = co0 + (PAIR ? half * 32 : 0) + col;
    if (co >= cout)
        return;
    const long r = PAIR ? blockIdx.y : 2 * blockIdx.y + half;
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        float* dst = part + (r * 81 + l01 * 9 + (o2 + 1) * 3 + q) * cin * cout;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int c = 8 * (i / 4) + 4 * kh + i % 4;
            if (c < nc)
                dst[(long)(ci0 + c) * cout + co] = sum[q][i] + acc[q][i];
        }
    }
}

// The same with vector instructions, where the rows are too long for tiles of
// whole rows, partial over a
// chunk of sites:
// part[chunk][t][ci][co] = sum_{y in chunk} in[ci][y + o_t] g[co][y].
// Workgroup (t, co tile of kWT, site chunk); thread (ci group, co), the
// tiles of g and of the shifted input staged in LDS kWS sites at a time.
__global__ __launch_bounds__(256) void k_conv_wgrad(Lat lt, const float* __restrict__ in, int cin,
                                                    const float* __restrict__ g, int cout, long chunk,
                                                    float* __restrict__ part)
{
    __shared__ float gs[kWS][kWT + 1];
    __shared__ float xs[kWS][kMaxCin + 1];
    const long V = lt.V;
    const int t = blockIdx.x;
    const int co0 = blockIdx.y * kWT;
    const long y0 = (long)blockIdx.z * chunk;
    const long y1 = y0 + chunk < V ? y0 + chunk : V;
    const int col = threadIdx.x % kWT, cg = threadIdx.x / kWT;  // 4 groups of ci
    const int cpt = (cin + 3) / 4;
    const int o0 = t / 27, o1 = (t / 9) % 3, o2 = (t / 3) % 3, o3 = t % 3;
    float acc[kMaxCin / 4];
#pragma unroll
    for (int c = 0; c < kMaxCin / 4; ++c)
        acc[c] = 0.f;
    for (long ys = y0; ys < y1; ys += kWS) {
        __syncthreads();
        for (int e = threadIdx.x; e < kWS * kWT; e += blockDim.x) {
            const int yy = e % kWS, cc = e / kWS;
            const long y = ys + yy;
            gs[yy][cc] = (y < y1 && co0 + cc < cout) ? g[(long)(co0 + cc) * V + y] : 0.f;
        }
        for (int e = threadIdx.x; e < kWS * cin; e += blockDim.x) {
            const int yy = e % kWS, ci = e / kWS;
            const long y = ys + yy;
            float v = 0.f;
            if (y < y1) {
                long dl[4][3];
                tap_shifts(lt, y, 1, dl);
                v = in[(long)ci * V + y + dl[0][o0] + dl[1][o1] + dl[2][o2] + dl[3][o3]];
            }
            xs[yy][ci] = v;
        }
        __syncthreads();
        for (int yy = 0; yy < kWS; ++yy) {
            const float gv = gs[yy][col];
#pragma unroll
            for (int c = 0; c < kMaxCin / 4; ++c)
                if (c < cpt && cg * cpt + c < cin)
                    acc[c] += xs[yy][cg * cpt + c] * gv;
        }
    }
    if (co0 + col >= cout)
        return;
    float* dst = part + ((long)blockIdx.z * 81 + t) * cin * cout;
#pragma unroll
    for (int c = 0; c < kMaxCin / 4; ++c) {
        const int ci = cg * cpt + c;
        if (c < cpt && ci < cin)
            dst[(long)ci * cout + co0 + col] = acc[c];
    }
}

// dW[e] = sum over chunks of part[chunk][e] (fixed order)
__global__ __launch_bounds__(256) void k_sum_chunks(const float* __restrict__ part, long n, int nchunk,
                                                    float* __restrict__ dW)
{
    const long e = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n)
        return;
    float s = 0.f;
    for (int q = 0; q < nchunk; ++q)
        s += part[(long)q * n + e];
    dW[e] = s;
}

// db[co] = sum_y g[co][y] in FP64, rounded once, one workgroup per channel;
// sixteen loads in flight per thread (V is a multiple of 64), summed in pairs in
// a fixed order
__global__ __launch_bounds__(1024) void k_bias_grad(const float* __restrict__ g, long V, float* __restrict__ db)
{
    __shared__ double sh[16];
    const float* gc = g + (long)blockIdx.x * V;
    double a[16];
#pragma unroll
    for (int k = 0; k < 16; ++k)
        a[k] = 0.0;
    for (long y = threadIdx.x; y < V; y += 16 * 1024) {
        float v[16];
#pragma unroll
        for (int k = 0; k < 16; ++k)
            v[k] = y + 1024 * k < V ? gc[y + 1024 * k] : 0.f;
#pragma unroll
        for (int k = 0; k < 16; ++k)
            a[k] += (double)v[k];
    }
#pragma unroll
    for (int h = 8; h > 0; h >>= 1)
#pragma unroll
        for (int k = 0; k < h; ++k)
            a[k] += a[k + h];
    const double s = block_sum(a[0], sh);
    if (threadIdx.x == 0)
        db[blockIdx.x] = (float)s;
}

// canonical site index of native site s
__device__ inline long canon_of(const Geom& g, long s)
{
    int n[4], y[4], x[4];
    site_decompose(g, s, n, y);
    for (int mu = 0; mu < 4; ++mu)
        x[mu] = n[mu] * g.b[mu] + y[mu];
    return canon_index(g, x);
}

// x[c][i]: Re/Im of U_mu(x)[a][b] at channel ((mu*3 + a)*3 + b)*2 + r, then
// the 24 noise channels (noise [V][24], canonical)
__global__ __launch_bounds__(256) void k_features(Geom g, const c64* __restrict__ U64, const float* __restrict__ noise,
                                                  float* __restrict__ x)
{
    const long s = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= g.V)
        return;
    const long i = canon_of(g, s);
    for (int mu = 0; mu < 4; ++mu) {
        c64 u[9];
        for (int k = 0; k < 6; ++k)
            u[k] = U64[tidx(s, mu * 6 + k, 24)];
        for (int b = 0; b < 3; ++b)
            u[6 + b] = conjg(u[(b + 1) % 3] * u[3 + (b + 2) % 3] - u[(b + 2) % 3] * u[3 + (b + 1) % 3]);
        for (int k = 0; k < 9; ++k) {
            const int ch = 2 * (mu * 9 + k);
            x[(long)ch * g.V + i] = (float)u[k].re;
            x[(long)(ch + 1) * g.V + i] = (float)u[k].im;
        }
    }
    for (int k = 0; k < 24; ++k)
        x[(long)(72 + k) * g.V + i] = noise[i * 24 + k];
}

// field_l(x)[c] = out[(l*12 + c)*2][i] + i out[(l*12 + c)*2 + 1][i]
__global__ __launch_bounds__(256) void k_out_to_fields(Geom g, const float* __restrict__ out, int Ns,
                                                       c64* __restrict__ f)
{
    const long s = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= g.V)
        return;
    const long i = canon_of(g, s);
    const long F = 12 * g.V;
    for (int l = 0; l < Ns; ++l)
        for (int c = 0; c < 12; ++c) {
            const long ch = (long)(l * 12 + c) * 2;
            f[l * F + tidx(s, c, 12)] = c64{(double)out[ch * g.V + i], (double)out[(ch + 1) * g.V + i]};
        }
}

// dout[(l*12 + c)*2 + r][i] = 2 Re / 2 Im of grad_l(x)[c]  (real gradient of a
// real loss from its derivative with respect to conj(field))
__global__ __launch_bounds__(256) void k_fields_to_out(Geom g, const c64* __restrict__ gr, int Ns,
                                                       float* __restrict__ dout)
{
    const long s = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= g.V)
        return;
    const long i = canon_of(g, s);
    const long F = 12 * g.V;
    for (int l = 0; l < Ns; ++l)
        for (int c = 0; c < 12; ++c) {
            const long ch = (long)(l * 12 + c) * 2;
            const c64 v = gr[l * F + tidx(s, c, 12)];
            dout[ch * g.V + i] = (float)(2.0 * v.re);
            dout[(ch + 1) * g.V + i] = (float)(2.0 * v.im);
        }
}

// Per deflation block: G = Psi^+ Psi, C = Psi^+ T, Cholesky G = L L^+,
// Y = G^-1 C; writes Y[blk][l][k], tb2[blk][k] = ||t_k on the block||^2 and
// proj[blk][k] = Re(c_k^+ y_k). Entries are staged through LDS 64 at a time.
constexpr int kMaxLossN = 32;
constexpr int kLT = 64;  // staged entries

__global__ __launch_bounds__(256) void k_deficit_block(Geom g, const c64* __restrict__ Psi, int Ns,
                                                       const c64* __restrict__ T, int K, c64* __restrict__ Y,
                                                       double* __restrict__ tb2, double* __restrict__ proj,
                                                       int* __restrict__ flag)
{
    extern __shared__ double dyn[];
    c64* ps = reinterpret_cast<c64*>(dyn);              // [Ns][kLT + 1]
    c64* ts = ps + Ns * (kLT + 1);                      // [K][kLT + 1]
    c64* Gm = ts + K * (kLT + 1);                       // [Ns][Ns]
    c64* Cm = Gm + Ns * Ns;                             // [Ns][K]
    double* tn = reinterpret_cast<double*>(Cm + Ns * K);  // [K]
    const int blk = blockIdx.x;
    const long F = 12 * g.V;
    const int ne = 12 * g.Vb;
    // products: G (l <= m), C (l, k), ||t_k||^2
    const int nG = Ns * (Ns + 1) / 2, nC = Ns * K, np = nG + nC + K;
    c64 acc[8];
    int pid[8];
    int nmine = 0;
    for (int p = threadIdx.x; p < np && nmine < 8; p += blockDim.x)
        pid[nmine++] = p;
    for (int q = 0; q < 8; ++q)
        acc[q] = c64{0.0, 0.0};
    for (int e0 = 0; e0 < ne; e0 += kLT) {
        __syncthreads();
        for (int q = threadIdx.x; q < (Ns + K) * kLT; q += blockDim.x) {
            const int r = q / kLT, e = q % kLT;
            c64 v{0.0, 0.0};
            if (e0 + e < ne) {
                long idx;
                if ((g.Vb & (kTile - 1)) == 0)
                    idx = (long)blk * ne + e0 + e;
                else
                    idx = tidx((long)blk * g.Vb + (e0 + e) % g.Vb, (e0 + e) / g.Vb, 12);
                v = r < Ns ? Psi[(long)r * F + idx] : T[(long)(r - Ns) * F + idx];
            }
            if (r < Ns)
                ps[r * (kLT + 1) + e] = v;
            else
                ts[(r - Ns) * (kLT + 1) + e] = v;
        }
        __syncthreads();
        for (int q = 0; q < nmine; ++q) {
            const int p = pid[q];
            const c64 *u, *v;
            if (p < nG) {
                int l = 0, rem = p;
                while (rem >= Ns - l) {
                    rem -= Ns - l;
                    ++l;
                }
                u = ps + l * (kLT + 1);
                v = ps + (l + rem) * (kLT + 1);
            } else if (p < nG + nC) {
                const int l = (p - nG) / K, k = (p - nG) % K;
                u = ps + l * (kLT + 1);
                v = ts + k * (kLT + 1);
            } else {
                u = ts + (p - nG - nC) * (kLT + 1);
                v = u;
            }
            double re = acc[q].re, im = acc[q].im;
            for (int e = 0; e < kLT; ++e) {
                const c64 a = u[e], b = v[e];
                re += a.re * b.re + a.im * b.im;
                im += a.re * b.im - a.im * b.re;
            }
            acc[q] = c64{re, im};
        }
    }
    __syncthreads();
    for (int q = 0; q < nmine; ++q) {
        const int p = pid[q];
        if (p < nG) {
            int l = 0, rem = p;
            while (rem >= Ns - l) {
                rem -= Ns - l;
                ++l;
            }
            const int m = l + rem;
            Gm[l * Ns + m] = acc[q];
            Gm[m * Ns + l] = c64{acc[q].re, -acc[q].im};
        } else if (p < nG + nC) {
            Cm[p - nG] = acc[q];
        } else {
            tn[p - nG - nC] = acc[q].re;
        }
    }
    __syncthreads();
    // Cholesky in place (lower triangle): G = L L^+
    if (threadIdx.x == 0) {
        for (int j = 0; j < Ns; ++j) {
            double d = Gm[j * Ns + j].re;
            for (int k = 0; k < j; ++k)
                d -= Gm[j * Ns + k].re * Gm[j * Ns + k].re + Gm[j * Ns + k].im * Gm[j * Ns + k].im;
            if (!(d > 0.0)) {
                atomicOr(flag, 1);
                d = 1.0;
            }
            const double ljj = sqrt(d);
            Gm[j * Ns + j] = c64{ljj, 0.0};
            for (int i = j + 1; i < Ns; ++i) {
                c64 s = Gm[i * Ns + j];
                for (int k = 0; k < j; ++k) {
                    const c64 a = Gm[i * Ns + k], b = Gm[j * Ns + k];  // s -= L_ik conj(L_jk)
                    s.re -= a.re * b.re + a.im * b.im;
                    s.im -= a.im * b.re - a.re * b.im;
                }
                Gm[i * Ns + j] = c64{s.re / ljj, s.im / ljj};
            }
        }
    }
    __syncthreads();
    // columns of Y: L z = c, L^+ y = z
    for (int k = threadIdx.x; k < K; k += blockDim.x) {
        c64 z[kMaxLossN];
        for (int i = 0; i < Ns; ++i) {
            c64 s = Cm[i * K + k];
            for (int j = 0; j < i; ++j) {
                const c64 a = Gm[i * Ns + j];
                s.re -= a.re * z[j].re - a.im * z[j].im;
                s.im -= a.re * z[j].im + a.im * z[j].re;
            }
            const double d = Gm[i * Ns + i].re;
            z[i] = c64{s.re / d, s.im / d};
        }
        for (int i = Ns - 1; i >= 0; --i) {
            c64 s = z[i];
            for (int j = i + 1; j < Ns; ++j) {
                const c64 a = Gm[j * Ns + i];  // (L^+)_ij = conj(L_ji)
                s.re -= a.re * z[j].re + a.im * z[j].im;
                s.im -= a.re * z[j].im - a.im * z[j].re;
            }
            const double d = Gm[i * Ns + i].re;
            z[i] = c64{s.re / d, s.im / d};
        }
        double pr = 0.0;
        for (int i = 0; i < Ns; ++i) {
            const c64 cc = Cm[i * K + k];
            pr += cc.re * z[i].re + cc.im * z[i].im;
            Y[((long)blk * Ns + i) * K + k] = z[i];
        }
        tb2[(long)blk * K + k] = tn[k];
        proj[(long)blk * K + k] = pr;
    }
}

// grad_l(x) = -sum_k (t_k(x) - sum_m Psi_m(x) Y_mk) conj(Y_lk) wk[k]
// (wk = 1 / (K ||t_k||^2)). Workgroup = kLT entries of one block: first the
// residuals r_k(x) into LDS (task (k, x)), then the gradient (task (l, x)).
__global__ __launch_bounds__(256) void k_deficit_grad(Geom g, const c64* __restrict__ Psi, int Ns,
                                                      const c64* __restrict__ T, int K, const c64* __restrict__ Y,
                                                      const double* __restrict__ wk, c64* __restrict__ grad)
{
    __shared__ c64 ys[kMaxLossN * kMaxLossN];
    __shared__ c64 rs[kMaxLossN * kLT];
    __shared__ double ws[kMaxLossN];
    const int blk = blockIdx.y;
    const long F = 12 * g.V;
    const int ne = 12 * g.Vb;
    const int e0 = blockIdx.x * kLT;
    for (int q = threadIdx.x; q < Ns * K; q += blockDim.x)
        ys[q] = Y[(long)blk * Ns * K + q];
    for (int q = threadIdx.x; q < K; q += blockDim.x)
        ws[q] = wk[q];
    __syncthreads();
    auto index = [&](int e) -> long {
        if ((g.Vb & (kTile - 1)) == 0)
            return (long)blk * ne + e;
        return tidx((long)blk * g.Vb + e % g.Vb, e / g.Vb, 12);
    };
    for (int q = threadIdx.x; q < K * kLT; q += blockDim.x) {
        const int k = q / kLT, e = q % kLT;
        c64 r{0.0, 0.0};
        if (e0 + e < ne) {
            const long idx = index(e0 + e);
            r = T[(long)k * F + idx];
            for (int m = 0; m < Ns; ++m) {
                const c64 p = Psi[(long)m * F + idx], y = ys[m * K + k];
                r.re -= p.re * y.re - p.im * y.im;
                r.im -= p.re * y.im + p.im * y.re;
            }
        }
        rs[k * kLT + e] = r;
    }
    __syncthreads();
    for (int q = threadIdx.x; q < Ns * kLT; q += blockDim.x) {
        const int l = q / kLT, e = q % kLT;
        if (e0 + e >= ne)
            continue;
        double gr = 0.0, gi = 0.0;
        for (int k = 0; k < K; ++k) {
            const c64 r = rs[k * kLT + e], y = ys[l * K + k];  // r conj(y)
            gr -= ws[k] * (r.re * y.re + r.im * y.im);
            gi -= ws[k] * (r.im * y.re - r.re * y.im);
        }
        grad[(long)l * F + index(e0 + e)] = c64{gr, gi};
    }
}

__global__ __launch_bounds__(256) void k_adam(float* __restrict__ th, const float* __restrict__ gr,
                                              float* __restrict__ m, float* __restrict__ v, long n, float lr,
                                              float b1, float b2, float eps, float c1, float c2)
{
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n)
        return;
    const float gi = gr[i];
    const float mi = b1 * m[i] + (1.f - b1) * gi;
    const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    th[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

Lat make_lat(const Geom& g)
{
    Lat lt;
    for (int mu = 0; mu < 4; ++mu)
        lt.L[mu] = g.L[mu];
    lt.str[3] = 1;
    for (int mu = 2; mu >= 0; --mu)
        lt.str[mu] = lt.str[mu + 1] * lt.L[mu + 1];
    lt.V = g.V;
    lt.W3 = lt.L[3];
    lt.nseg = 0;
    return lt;
}

inline unsigned site_blocks(long n) { return (unsigned)((n + 255) / 256); }

}  // namespace

// Positions staged for a tile of T sites, the largest over all tiles: a tile
// covers at most rows = (T - 1) / L3 + 2 rows (exactly T / L3 when tiles start
// at row boundaries) and each run of rows of one plane adds two.
int conv_tile_positions(const Geom& g, int T)
{
    const int L3 = g.L[3], L2 = g.L[2];
    int rows = T % L3 == 0 ? T / L3 : L3 % T == 0 ? 1 : (T - 1) / L3 + 2;
    const long total = g.V / L3;
    if (rows > total)
        rows = (int)total;
    int planes = rows % L2 == 0 && T % L3 == 0 ? rows / L2 : L2 % rows == 0 && T % L3 == 0 ? 1 : (rows - 1) / L2 + 2;
    if (L3 % T == 0)
        planes = 1;
    return (rows + 2 * planes) * (L3 + 2);
}

// LDS of the FP32 weight-gradient tiles, in bytes; 0 if the lattice's rows are
// too long for them (more than kCPos staged positions): the vector kernel serves those.
size_t wgrad_lds_bytes(const Geom& g, bool pair)
{
    const int np = conv_tile_positions(g, kCT);
    return np > kCPos ? 0 : sizeof(float) * ((size_t)np * kCP + (size_t)kCT * ((pair ? 64 : 32) + 4) + kCT);
}

// Two workgroups of the matrix-core weight gradient fit a CU, so the ranges of
// tiles are cut to give at most 512 workgroups (one full round of 256 CUs; a
// few more would run alone afterwards). cap: most floats of partial sums.
bool conv_wgrad_plan(const Geom& g, int cin, int cout, size_t cap, WgradPlan* p)
{
    const size_t per = (size_t)81 * cin * cout;
    p->mfma = wgrad_lds_bytes(g, true) != 0;
    if (p->mfma) {
        p->pair = cout > 32;
        const int tiles = (int)((g.V + kCT - 1) / kCT);
        const int groups = 9 * ((cin + 31) / 32) * ((cout + (p->pair ? 63 : 31)) / (p->pair ? 64 : 32));
        const int per_range = p->pair ? 1 : 2;  // partials written per range
        long n = std::max(1, std::min(tiles, 512 / groups));
        n = std::min<long>(n, (long)(cap / per) / per_range);
        if (n < 1)
            return false;
        p->chunk = (tiles + n - 1) / n;
        p->nchunk = (int)((tiles + p->chunk - 1) / p->chunk);
        p->nparts = p->nchunk * per_range;
    } else {
        // at most 32 ranges of at least 4096 sites
        long c = std::max<long>(4096, (g.V + 31) / 32);
        const long most = (long)(cap / per);
        if (most < 1)
            return false;
        c = std::max(c, (g.V + most - 1) / most);
        c = ((c + kWS - 1) / kWS) * kWS;
        p->chunk = c;
        p->pair = false;
        p->nparts = p->nchunk = (int)((g.V + c - 1) / c);
    }
    p->floats = (size_t)p->nparts * per;
    return p->floats <= cap;
}

// ------------------------------------- allocation-free weight gradient
//
// Partial sums of the weight gradient for callers that cannot allocate
// (conv4d_backward_noalloc): a file-scope device array of kNoAllocFloats
// floats, which every device the library runs on holds until the process
// ends. Host code takes its device address from hipGetSymbolAddress, once per
// device, and passes that to the kernels (the array's name is no device
// address on the host). Every call overwrites the part it uses before reading
// it; calls that overlap on one device race on it.
static __device__ __align__(256) float scratch[kNoAllocFloats];

float* noalloc_scratch()
{
    static std::mutex mu;
    static float* ptr[kMaxDevices] = {};
    int dev = 0;
    HIPCHECK(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices)
        fail(DFL_EINVAL, "device index beyond the allocation-free scratch table");
    std::lock_guard<std::mutex> lock(mu);
    if (!ptr[dev]) {
        void* p = nullptr;
        HIPCHECK(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (!p)
            fail(DFL_EHIP, "hipGetSymbolAddress returned no address for the scratch array");
        ptr[dev] = static_cast<float*>(p);
    }
    return ptr[dev];
}

void launch_net_features(const Geom& g, const c64* U64, const float* noise, float* x, hipStream_t s)
{
    hipLaunchKernelGGL(k_features, dim3(site_blocks(g.V)), dim3(256), 0, s, g, U64, noise, x);
}

namespace {

template <bool TRANS>
void launch_conv(const Geom& g, const float* in, int nic, const float* W, int w_cin, int w_cout, const float* bias,
                 int noc, float* out, float* act, const float* zprev, hipStream_t s)
{
    Lat lt = make_lat(g);
    int np = conv_tile_positions(g, kCT);
    long ntiles = (g.V + kCT - 1) / kCT;
    if (np > kCPos) {
        // Tiles of whole rows' sites stage up to three rows and their halo; from
        // about L3 = 72 on they pass kCPos, and a tile becomes a segment of one
        // row. MI355X, forward on 8^3 x 160, 32 -> 32 channels 256 us and 32 -> 288
        // 2.00 ms, with vector instructions 489 us and 3.17 ms.
        lt.nseg = (lt.L[3] + kCT - 1) / kCT;
        lt.W3 = (lt.L[3] + lt.nseg - 1) / lt.nseg;
        lt.nseg = (lt.L[3] + lt.W3 - 1) / lt.W3;  // none of them empty
        np = 3 * (lt.W3 + 2);
        ntiles = g.V / lt.L[3] * lt.nseg;
    }
    // 64 output channels a workgroup, or 32 where that would leave CUs idle (4^3 x 32, 32 -> 96 channels: 133 us with
    // 64, 73 with 32)
    const long groups = (noc + 63) / 64;
    const int ot = noc <= 32 || ntiles * groups < 256 ? 1 : 2;
    // Few input channels and enough workgroups for every CU (more than two rounds of 32 output channels for five to
    // eight channels): the vector kernel. 32 x 16^3, 1 -> 1 channels 47 us (matrix cores 94), 4 -> 16 64 (116), 8 -> 16
    // 90 (118); 16^4, 1 -> 1 40 (51), 5 -> 40 86 (92), 8 -> 16 86 (57); 8^4, 1 -> 1 42 (39).
    if ((nic <= 4 && ntiles * groups >= 256) || (nic <= kCN && ntiles * ((noc + 31) / 32) > 512)) {
        hipLaunchKernelGGL(k_conv<TRANS>, dim3(site_blocks(g.V), (noc + kCO - 1) / kCO), dim3(256), 0, s, lt, in, nic,
                           W, w_cin, w_cout, bias, noc, out, act, zprev);
        return;
    }
    const size_t lds = sizeof(float) * ((size_t)np * kCP + (size_t)3 * 32 * ot * kCP);
    const dim3 grid((unsigned)pad_grid(ntiles), (noc + 32 * ot - 1) / (32 * ot));
    static std::once_flag attr[2];  // per instantiation
    auto launch = [&](std::once_flag& f, auto* kernel) {
        set_max_lds_once(f, reinterpret_cast<const void*>(kernel), 128 * 1024);
        hipLaunchKernelGGL(kernel, grid, dim3(256), lds, s, lt, (int)ntiles, in, nic, W, w_cin, w_cout, bias, noc, np,
                           out, act, zprev);
    };
    if (ot == 1)
        launch(attr[0], &k_conv_mfma<TRANS, 1>);
    else
        launch(attr[1], &k_conv_mfma<TRANS, 2>);
}

}  // namespace

void launch_conv_forward(const Geom& g, const float* in, int cin, const float* W, const float* b, int cout, float* z,
                         float* a, hipStream_t s)
{
    launch_conv<false>(g, in, cin, W, cin, cout, b, cout, z, a, nullptr, s);
}

bool conv_bf16_fits(const Geom& g) { return g.L[3] % kBTS == 0 && g.L[2] % kBNL == 0; }

namespace {

size_t bf16_lds_bytes(const Geom& g, int ns)
{
    return (size_t)conv_tile_positions(g, 128 * ns) * (kBRow * sizeof(uint16_t) + sizeof(int2));
}

// Sites per tile of the BF16 map: 512 where that gives two workgroups per CU
// and two of them share a CU's LDS (32 -> 576 on 16^2 x 24 x 64: 1.55 ms, the
// segment kernel 4.41), 128 where the lattice is too small for that (32 -> 32
// on 4 x 8^2 x 32: 34 us against 136), 0 (segment kernel) where the rows are
// too long for a tile. Returned in units of 128 sites.
int bf16_tile_ns(const Geom& g, int cout)
{
    constexpr size_t half = 80 * 1024;
    const long nco = (cout + 63) / 64;
    if (bf16_lds_bytes(g, 4) <= half && g.V / 512 * nco >= 512)
        return 4;
    return bf16_lds_bytes(g, 1) <= half ? 1 : 0;
}

}  // namespace

size_t conv_bf16_weight_elems(int cin, int cout)
{
    const int ot = cout <= 32 ? 2 : 4;
    const int cinP = (cin + kBK - 1) / kBK * kBK, coutP = (cout + 16 * ot - 1) / (16 * ot) * (16 * ot);
    return 81ul * (size_t)cinP * (size_t)coutP;
}

size_t conv_bf16_input_elems(const Geom& g)
{
    return bf16_tile_ns(g, 1) ? (size_t)((kNetMaxCin + kBK - 1) / kBK * kBK) * (size_t)g.V : 0;
}

void launch_conv_forward_bf16(const Geom& g, const float* in, int cin, const float* W, const float* b, int cout,
                              float* z, float* a, uint16_t* Wb, uint16_t* Xb, hipStream_t s)
{
    const Lat lt = make_lat(g);
    const int cinP = (cin + kBK - 1) / kBK * kBK;
    const int ns = bf16_tile_ns(g, cout);
    if (ns && Xb) {
        const int ot = cout <= 32 ? 1 : 2;
        const int noct = (cout + 32 * ot - 1) / (32 * ot) * ot, nk = cinP / 16;
        u16x8* Wf = reinterpret_cast<u16x8*>(Wb);
        hipLaunchKernelGGL(k_weights_frag, dim3(site_blocks(81L * nk * noct * 64)), dim3(256), 0, s, W, cin, cout, nk,
                           noct, Wf);
        hipLaunchKernelGGL(k_planes_bf16, dim3((unsigned)(g.V / 64), cinP / 32), dim3(256), 0, s, in, cin, cinP, g.V,
                           Xb);
        const int ntiles = (int)((g.V + 128 * ns - 1) / (128 * ns));
        const int np = conv_tile_positions(g, 128 * ns);
        const size_t lds = bf16_lds_bytes(g, ns);
        const dim3 grid((unsigned)pad_grid(ntiles), noct / ot);
        static std::once_flag attr[4];
        auto launch = [&](std::once_flag& f, auto* kernel) {
            set_max_lds_once(f, reinterpret_cast<const void*>(kernel), 80 * 1024);
            hipLaunchKernelGGL(kernel, grid, dim3(256), lds, s, lt, ntiles, Xb, cinP, Wf, noct, b, cout, np, z, a);
        };
        if (ot == 1)
            ns == 1 ? launch(attr[0], &k_conv_bf16_tile<1, 1>) : launch(attr[1], &k_conv_bf16_tile<1, 4>);
        else
            ns == 1 ? launch(attr[2], &k_conv_bf16_tile<2, 1>) : launch(attr[3], &k_conv_bf16_tile<2, 4>);
        return;
    }
    const int ot = cout <= 32 ? 2 : 4;
    const int coutP = (cout + 16 * ot - 1) / (16 * ot) * (16 * ot);
    const long nw = 81L * cinP * coutP;
    hipLaunchKernelGGL(k_weights_bf16, dim3(site_blocks(nw)), dim3(256), 0, s, W, cin, cout, cinP, coutP, Wb);
    const unsigned ngrp = (unsigned)(g.V / (kBTS * kBNL));
    if (ot == 2)
        hipLaunchKernelGGL(k_conv_bf16<2>, dim3(ngrp * (unsigned)(coutP / 32)), dim3(256), 0, s, lt, in, cin, cinP,
                           Wb, coutP, b, cout, z, a);
    else
        hipLaunchKernelGGL(k_conv_bf16<4>, dim3(ngrp * (unsigned)(coutP / 64)), dim3(256), 0, s, lt, in, cin, cinP,
                           Wb, coutP, b, cout, z, a);
}

void launch_conv_backward(const Geom& g, const float* in, int cin, const float* W, int cout, const float* gr,
                          float* dW, float* db, float* din, const float* zprev, float* part, const WgradPlan& p,
                          hipStream_t s)
{
    const Lat lt = make_lat(g);
    static std::once_flag attr[2];
    const int np = conv_tile_positions(g, kCT);
    const unsigned nct = (cin + 31) / 32;
    if (p.mfma && p.pair) {
        set_max_lds_once(attr[0], reinterpret_cast<const void*>(&k_conv_wgrad_mfma<true>), 128 * 1024);
        hipLaunchKernelGGL(k_conv_wgrad_mfma<true>, dim3(9 * nct * ((cout + 63) / 64), p.nchunk), dim3(384),
                           wgrad_lds_bytes(g, true), s, lt, in, cin, gr, cout, (int)p.chunk, np, part);
    } else if (p.mfma) {
        set_max_lds_once(attr[1], reinterpret_cast<const void*>(&k_conv_wgrad_mfma<false>), 128 * 1024);
        hipLaunchKernelGGL(k_conv_wgrad_mfma<false>, dim3(9 * nct * ((cout + 31) / 32), p.nchunk), dim3(384),
                           wgrad_lds_bytes(g, false), s, lt, in, cin, gr, cout, (int)p.chunk, np, part);
    } else {
        hipLaunchKernelGGL(k_conv_wgrad, dim3(81, (cout + kWT - 1) / kWT, p.nchunk), dim3(256), 0, s, lt, in, cin,
                           gr, cout, p.chunk, part);
    }
    const long n = 81L * cin * cout;
    hipLaunchKernelGGL(k_sum_chunks, dim3(site_blocks(n)), dim3(256), 0, s, part, n, p.nparts, dW);
    hipLaunchKernelGGL(k_bias_grad, dim3(cout), dim3(1024), 0, s, gr, g.V, db);
    if (din)
        launch_conv<true>(g, gr, cout, W, cin, cout, nullptr, cin, din, nullptr, zprev, s);
}

void launch_out_to_fields(const Geom& g, const float* out, int Ns, c64* f, hipStream_t s)
{
    hipLaunchKernelGGL(k_out_to_fields, dim3(site_blocks(g.V)), dim3(256), 0, s, g, out, Ns, f);
}

void launch_fields_to_out(const Geom& g, const c64* gr, int Ns, float* dout, hipStream_t s)
{
    hipLaunchKernelGGL(k_fields_to_out, dim3(site_blocks(g.V)), dim3(256), 0, s, g, gr, Ns, dout);
}

size_t deficit_lds_bytes(int Ns, int K)
{
    return sizeof(c64) * ((size_t)(Ns + K) * (kLT + 1) + (size_t)Ns * Ns + (size_t)Ns * K) + sizeof(double) * K;
}

void launch_deficit_block(const Geom& g, const c64* Psi, int Ns, const c64* T, int K, c64* Y, double* tb2,
                          double* proj, int* flag, hipStream_t s)
{
    const size_t lds = deficit_lds_bytes(Ns, K);
    static std::once_flag attr;
    set_max_lds_once(attr, reinterpret_cast<const void*>(&k_deficit_block), (int)deficit_lds_bytes(kMaxLossN, kMaxLossN));
    hipLaunchKernelGGL(k_deficit_block, dim3(g.Nb), dim3(256), lds, s, g, Psi, Ns, T, K, Y, tb2, proj, flag);
}

void launch_deficit_grad(const Geom& g, const c64* Psi, int Ns, const c64* T, int K, const c64* Y, const double* wk,
                         c64* grad, hipStream_t s)
{
    const int ne = 12 * (int)g.Vb;
    hipLaunchKernelGGL(k_deficit_grad, dim3((ne + kLT - 1) / kLT, g.Nb), dim3(256), 0, s, g, Psi, Ns, T, K, Y, wk,
                       grad);
}

void launch_adam(float* th, const float* gr, float* m, float* v, long n, float lr, float b1, float b2, float eps,
                 float c1, float c2, hipStream_t s)
{
    if (n > 0)
        hipLaunchKernelGGL(k_adam, dim3(site_blocks(n)), dim3(256), 0, s, th, gr, m, v, n, lr, b1, b2, eps, c1, c2);
}

}  // namespace dfl
