// Energy-test pair sums on gfx950 (Sect. 2.2 eq. (2), Sect. 3 eq. (3)).
//
// For coordinates y_i (D <= 8 per event), psi_ij = exp(-|y_i - y_j|^2 / 2 sigma^2)
// for i != j (0 on the diagonal) and a 0/1 column matrix G [n][C], the kernel
// accumulates for every column c
//   sums[c][0]     = sum_i sum_{j != i} G[i][c] psi_ij G[j][c]
//   sums[c][1 + q] = sum_i sum_{j != i} G[i][q] psi_ij G[j][c],   q < R,
// i.e. the leading R columns double as row weights.  Every within-sample and
// cross-sample sum of eq. (2) and eq. (3) -- for the observed split and every
// permutation at once -- is a combination of these.
//
// psi is symmetric, so only pairs j > i are formed: the first sum is twice its
// upper-triangle part, and the second is the upper-triangle part of
// sum w_i psi_ij G_jc plus the transposed term sum_i G_ic (Psi_upper w_q)_i,
// where (Psi_upper w_q) is column q of the same product.
//
// Both steps run on the matrix cores.  Distances: with the scaled coordinates
// centred on the mean c of the first 256 events, v = y yscale - c, the vectors
// x_j = (v_j, |v_j|^2, 1) and x_i = (-2 v_i, 1, |v_i|^2) give
// x_i . x_j = |v_i - v_j|^2.  Each vector is split into two float16 terms
// (hi, lo: 2^-22 relative) and laid out so that one float16 contraction over
// 32 slots forms hi.hi + hi.lo + lo.hi - 14 (the -14, the psi scale, is an
// exact extra slot): two v_mfma_f32_32x32x16_f16 per 32 x 32 pairs, with exact
// products and float32 accumulation.  Then psi * 2^14 = 2^-(that) costs one
// exp2 per pair on the vector ALU.  The rounding of the squared distance is
// about 2^-22 (2 |v_i|^2 + 2 |v_j|^2) plus the float32 accumulation; centring
// keeps |v|^2 small (a few units for invariant masses at sigma ~ 0.3 GeV, ~100
// at 0.05 GeV), and the errors are of random sign, so sums over many pairs
// keep ~1e-8.  An event with |v|^2 > VMAX2 (or a non-finite one) is outside
// that range.  A range check over all events runs first and sets a device
// flag; the kernel is launched in two instantiations, of which only one does
// the work: without the flag the matrix-core form above, with it the SAFE form,
// in which every chunk of pairs that holds such an event as a row or as a
// column forms its distances as direct float32 differences of the raw
// coordinates, (y_i - y_j) yscale, squared and summed on the vector ALU
// (accurate at any distance from the centre), the matrix-core operands of
// those events being finite placeholders.
// V = Psi G is then a dense contraction over j in half precision with float32
// accumulation (v_mfma_f32_32x32x16_f16): psi * 2^14 is split into two float16
// terms hi = rtz(psi), lo = rtz(psi - hi): the difference is exact in float32
// and hi + lo is within 2^-20 (relative, from below) of the float32 psi; the
// scale keeps both terms clear of the float16 subnormals for every psi above
// 2^-17.  The 0/1 columns are exact in float16, so each product is exact and
// only the float32 accumulation rounds.  The distance tile of 32 rows x 32 j
// leaves each lane 16 psi of its row, which are the lane's half of two 32 x 16
// operand tiles; columns are staged in LDS transposed ([c][j], float16, in the
// j order those tiles use), so a lane's 8 values of one column are one 16-byte
// read.  The next chunk's columns and coordinates are loaded into registers
// while the current one is multiplied.  Every FL chunks the float32 tiles are
// reduced per column into float64 partials, so float32 only sums 2 * FL * JC
// products.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "tp_energy.h"
#include "tp_launch.h"
#define TP_HD __host__ __device__
#include "tp_exact.h"

namespace tpe {
using tpk::launch;
namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int ROWS = 128;     // rows i per workgroup (4 waves x 32)
constexpr int JC = 128;       // j per LDS chunk
constexpr int KS = 16;        // j per matrix-core step
constexpr int FL = 8;         // chunks per float32 -> float64 reduction
constexpr int XCDS = 8;       // dies with an L2 each; workgroups go to them in turn
constexpr int RESIDENT = 512; // workgroups that run at a time (two per compute unit at 128 columns)
constexpr int64_t L2_BYTES = 3 << 20;   // a sample that stays in each 4 MiB L2
constexpr int GPAD = 8;       // float16 padding per staged column (spreads LDS banks)
constexpr int XS = 40;        // float16 slots per staged j vector: 32 used, 8 padding (spreads LDS banks)
constexpr float PSI_LOG2 = 14.0f;             // psi is formed scaled by 2^14
// Largest |v|^2 (squared scaled distance from the centre) of an event whose
// distances go through the matrix cores: their rounding grows as 2^-22 |v|^2,
// and float16 holds |v|^2 only below 65504.
constexpr float VMAX2 = 1024.0f;
constexpr double PSI_UNSCALE = 1.0 / 16384.0;

template <int NT, bool SAFE>
struct Smem {
    static constexpr int C = 32 * NT;
    uint16_t xh[2][JC][XS];             // distance operands of this chunk and the next, float16 slots (see slot())
    uint16_t gs[C][JC + GPAD];          // columns of the chunk, [32 t + col][j], float16 0 or 1
    float cw[4][MAXD];                  // per-wave coordinate sums for the centre c
    float cen[MAXD];                    // the centre c
    double red[C][1 + MAXR];            // workgroup totals
    // SAFE: raw coordinates of the two chunks (direct distances), and whether an event of
    // the first / second 64 of each is outside the matrix-core range
    alignas(16) float yc[2][SAFE ? MAXD : 1][SAFE ? JC : 1];
    uint32_t far[2][2];
};

// The centre's scratch of the range check (same fields as Smem).
struct CentreSmem {
    float cw[4][MAXD];
    float cen[MAXD];
};

// Coordinates 0 .. KD - 1 of event i, read without a branch (past either end the
// last one's), so that the loads are all in flight together.
template <int KD>
__device__ __forceinline__ void load_coords(const EParams &p, int64_t i, float (&y)[KD])
{
    i = i < p.n ? i : p.n - 1;
#pragma unroll
    for (int d = 0; d < KD; ++d) y[d] = p.Y[(d < p.D ? d : p.D - 1) * p.ldY + i];
}

// x + the x of the lane whose number differs in bit O (a mirrored lane for
// O = 4, 8: equal, since lanes that differ only in lower bits hold the same sum)
template <int O>
__device__ __forceinline__ float add_xor(float x)
{
    if constexpr (O >= 16) return x + __shfl_xor(x, O);
    constexpr int ctrl = O == 1 ? 0xB1 : O == 2 ? 0x4E : O == 4 ? 0x141 : 0x140;
    return x + __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), ctrl, 0xf, 0xf, false));
}

// Centre c of the scaled coordinates: the mean of the first min(n, 256)
// events, formed in a fixed order so that every workgroup gets the same bits.
// y: thread tid's event, coordinates 0 .. KD - 1 (KD >= D).
template <int KD, class SM>
__device__ __forceinline__ void centre(const EParams &p, SM &sm, const float (&y)[KD])
{
    const int tid = threadIdx.x;
    const int64_t m = p.n < 256 ? p.n : 256;
    float x[KD];
#pragma unroll
    for (int d = 0; d < KD; ++d) x[d] = (d < p.D && tid < m) ? y[d] * p.yscale : 0.0f;
#pragma unroll
    for (int d = 0; d < KD; ++d) x[d] = add_xor<8>(add_xor<4>(add_xor<2>(add_xor<1>(x[d]))));
#pragma unroll
    for (int d = 0; d < KD; ++d) x[d] = add_xor<16>(x[d]);
#pragma unroll
    for (int d = 0; d < KD; ++d) {
        x[d] = add_xor<32>(x[d]);
        if ((tid & 63) == 0) sm.cw[tid >> 6][d] = x[d];
    }
    __syncthreads();
    if (tid < KD)
        sm.cen[tid] = ((sm.cw[0][tid] + sm.cw[1][tid]) + (sm.cw[2][tid] + sm.cw[3][tid])) / (float)(m > 0 ? m : 1);
    __syncthreads();
}

// Distance operands in float16.  A float32 vector x of KA <= 10 components is
// split into hi = f16(x) and lo = f16(x - hi) (the difference exact in
// float32, hi + lo within 2^-22 |x|); a row vector takes the 32 slots
// [hi | lo | hi | -14 | 0] and a column vector [hi | hi | lo | 1 | 0], so that
// their float16 dot product over the 32 slots, with exact products and float32
// accumulation, is hi.hi + lo.hi + hi.lo - 14: x_i . x_j - 14 up to the lo.lo
// term (2^-22 relative).
// Slot s of the row (COL = false) or column (COL = true) pattern:
template <int KA, bool COL>
__device__ __forceinline__ uint16_t slot(const uint16_t (&hi)[KA], const uint16_t (&lo)[KA], int s)
{
    if (s < KA) return hi[s];
    if (s < 2 * KA) return COL ? hi[s - KA] : lo[s - KA];
    if (s < 3 * KA) return COL ? lo[s - 2 * KA] : hi[s - 2 * KA];
    // the scale of psi, exact in float16: 1 x (-14) in the first free slot
    if (s == 3 * KA) return __builtin_bit_cast(uint16_t, COL ? (_Float16)1.0f : (_Float16)(-PSI_LOG2));
    return 0;
}

template <int KA>
__device__ __forceinline__ void split16(const float (&x)[KA], uint16_t (&hi)[KA], uint16_t (&lo)[KA])
{
#pragma unroll
    for (int k = 0; k < KA; ++k) {
        const _Float16 a = (_Float16)x[k];
        const _Float16 b = (_Float16)(x[k] - (float)a);
        hi[k] = __builtin_bit_cast(uint16_t, a);
        lo[k] = __builtin_bit_cast(uint16_t, b);
    }
}

template <int N> struct Bytes;
template <> struct Bytes<1> { typedef uint8_t t; };
template <> struct Bytes<2> { typedef uint16_t t; };
template <> struct Bytes<4> { typedef uint32_t t; };

// Columns and lanes.  Lane col (0..31) of product tile t holds column NT col + t,
// so that a lane's columns are neighbours in G: one load of NT bytes per row.
// What a lane keeps of its wave's 32 rows of a row block: its row's operand
// halves, its row's raw coordinates (SAFE), and for the flush the column values
// G[row][NT col + t] in byte t of g[r], row = 8 (r / 4) + 4 h + r % 4 (the lane's
// rows in a product tile).
template <int NT, int NS, bool SAFE>
struct Rows {
    u32x4 xi[2];
    float y[SAFE ? 2 * NS - 2 : 1];
    uint32_t g[16];
    bool far;           // SAFE: a row of the block is outside the matrix-core range
};

// Row block setup, each wave for itself: rows ib .. ib + 31, the wave's share of
// the block of ROWS rows that starts at block0.  The loads first; rows past the
// end read the last row and count as 0 (a branch per row would have each row's
// load waited for in turn, some 10 us).
template <int NT, int NS>
struct RowLoads {
    float y[2 * NS - 2];
    uint32_t g[16];
};

template <int NT, int NS>
__device__ __forceinline__ void load_rows(const EParams &p, int64_t ib, RowLoads<NT, NS> &rl)
{
    constexpr int C = 32 * NT;
    const int lane = threadIdx.x & 63;
    const int h = lane >> 5;
    const int col = lane & 31;
    load_coords<2 * NS - 2>(p, ib + col, rl.y);
    const uint8_t *G = p.G + ib * C + NT * col;
    const int last = p.n - ib < 32 ? (int)(p.n - ib) - 1 : 31;      // the wave's last row (< 0: none)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int row = 8 * (r >> 2) + 4 * h + (r & 3);
        typename Bytes<NT>::t w = 0;
        if (last >= 0) w = *reinterpret_cast<const typename Bytes<NT>::t *>(G + (row < last ? row : last) * C);
        rl.g[r] = w;
    }
}

// This lane's row vector is x_i = (-2 (y_i - c), 1, |y_i - c|^2) (scaled
// coordinates, so psi = 2^-(scaled distance)^2): x_i . x_j = |y_i - y_j|^2 for
// the chunk vectors x_j.  Lane half h holds slots 16 m + 8 h .. + 7 of the row
// pattern for the two distance steps m.
template <int NT, int NS, bool SAFE>
__device__ __forceinline__ void setup_rows(const EParams &p, const Smem<NT, SAFE> &sm, int64_t block0, int64_t ib,
                                           const RowLoads<NT, NS> &rl, Rows<NT, NS, SAFE> &rb)
{
    constexpr int KA = 2 * NS;
    const int lane = threadIdx.x & 63;
    const int h = lane >> 5;
    const int col = lane & 31;
    const int64_t i = ib + col;
    const int rows = p.n - ib < 32 ? (int)(p.n - ib) : 32;      // of the wave's that exist
#pragma unroll
    for (int r = 0; r < 16; ++r) rb.g[r] = 8 * (r >> 2) + 4 * h + (r & 3) < rows ? rl.g[r] : 0u;
    float x[KA];
    float nrm = 0.0f;
#pragma unroll
    for (int k = 0; k < KA; ++k) x[k] = 0.0f;
#pragma unroll
    for (int d = 0; d < KA - 2; ++d) {
        const bool real = d < p.D && i < p.n;
        const float v = real ? rl.y[d] * p.yscale - sm.cen[d] : 0.0f;
        nrm = fmaf(v, v, nrm);
        if (d < p.D) x[d] = -2.0f * v;
        if constexpr (SAFE) rb.y[d] = real ? rl.y[d] : 0.0f;
    }
    rb.far = false;
    if constexpr (SAFE) {
        // outside the matrix-core range: finite placeholders; the chunks of the
        // whole row block take the direct distances
        if (!(nrm <= VMAX2)) {
            nrm = 0.0f;
#pragma unroll
            for (int k = 0; k < KA; ++k) x[k] = 0.0f;
        }
        bool far = false;
#pragma unroll
        for (int e = 0; e < ROWS; e += 64) {
            const int64_t j = block0 + e + lane;
            float nj = 0.0f;
            for (int d = 0; d < p.D; ++d) {
                const float v = j < p.n ? p.Y[d * p.ldY + j] * p.yscale - sm.cen[d] : 0.0f;
                nj = fmaf(v, v, nj);
            }
            far = far || !(nj <= VMAX2);
        }
        rb.far = __any(far) != 0;
    }
#pragma unroll
    for (int k = 0; k < KA; ++k) {
        if (k == p.D) x[k] = 1.0f;
        if (k == p.D + 1) x[k] = nrm;
    }
    uint16_t hi[KA], lo[KA];
    split16<KA>(x, hi, lo);
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const int s0 = 16 * m + 8 * h + 2 * w;
            rb.xi[m][w] = (uint32_t)slot<KA, false>(hi, lo, s0) | ((uint32_t)slot<KA, false>(hi, lo, s0 + 1) << 16);
        }
}

// Position of local j in a staged column: bits 2 and 3 swapped, the order in
// which the distance tiles deliver psi to the matrix-core operand (see
// chunk_products).
__device__ __forceinline__ int swap23(int j) { return (j & ~12) | ((j & 4) << 1) | ((j & 8) >> 1); }

// Load element i (32-bit index) from a uniform base pointer: the byte offset is
// formed in 32 bits, so the load takes the scalar-base + vector-offset form.
template <typename T>
__device__ __forceinline__ T ld(const void *base, uint32_t byte)
{
    typedef const T __attribute__((address_space(1))) *gptr;
    return *(gptr)((const char *)base + byte);
}

template <int N> struct Words;
template <> struct Words<1> { typedef uint32_t t; };
template <> struct Words<2> { typedef u32x2 t; };
template <> struct Words<4> { typedef u32x4 t; };

// Staging.  Columns of chunk j0 .. j0 + JC - 1 go to LDS transposed, [32 t + col][swap23(j)],
// as float16 (events j >= n: 0).  A thread takes 4 rows x 4 NT columns, one load of
// 4 NT bytes per row, and writes, per column, its 4 rows as one 8-byte word.  A dword
// of four 0/1 bytes times 60, in two 16-bit lanes, holds 0x3C for each 1, the high byte
// of float16 1.0; a byte permute then places the column's bytes of two rows in the high
// bytes of the two halves of a word.
// A chunk wholly inside the sample (``full``, uniform) takes unconditional loads off
// scalar bases, which cost no vector instructions.
template <int NT>
struct Columns {
    typename Words<NT>::t w[4];
};

template <int NT>
__device__ __forceinline__ void load_columns(const EParams &p, int64_t j0, Columns<NT> &pd)
{
    typedef typename Words<NT>::t W;
    constexpr int C = 32 * NT;
    const int tid = threadIdx.x;
    const uint32_t item = (uint32_t)((tid & 31) * 4 * C + (tid >> 5) * 4 * NT);
    const uint8_t *G = p.G + j0 * C;
    if (j0 + JC <= p.n) {
#pragma unroll
        for (int rr = 0; rr < 4; ++rr) pd.w[rr] = ld<W>(G, item + rr * C);
    } else {
#pragma unroll
        for (int rr = 0; rr < 4; ++rr) {
            W z;
            __builtin_memset(&z, 0, sizeof z);
            pd.w[rr] = j0 + (tid & 31) * 4 + rr < p.n ? ld<W>(G, item + rr * C) : z;
        }
    }
}

template <int NT>
__device__ __forceinline__ void expand_columns(const Columns<NT> &pd, u32x2 (&o)[4 * NT])
{
    typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
    uint32_t w[4][NT];
#pragma unroll
    for (int rr = 0; rr < 4; ++rr) {
        __builtin_memcpy(w[rr], &pd.w[rr], sizeof w[rr]);
#pragma unroll
        for (int e = 0; e < NT; ++e)
            w[rr][e] = __builtin_bit_cast(uint32_t, (u16x2)(__builtin_bit_cast(u16x2, w[rr][e]) * (uint16_t)60));
    }
#pragma unroll
    for (int q = 0; q < 4 * NT; ++q) {
        const int m = q & 3, e = q >> 2;
        // zero, byte m of the second source (first row of the pair), zero, byte m of the first source
        const uint32_t sel = 0x0cu | ((uint32_t)m << 8) | (0x0cu << 16) | ((uint32_t)(4 + m) << 24);
        o[q] = u32x2{ __builtin_amdgcn_perm(w[1][e], w[0][e], sel), __builtin_amdgcn_perm(w[3][e], w[2][e], sel) };
    }
}

template <int NT, bool SAFE>
__device__ __forceinline__ void store_columns(Smem<NT, SAFE> &sm, const u32x2 (&o)[4 * NT])
{
    const int tid = threadIdx.x;
    const int jq = swap23((tid & 31) * 4);
    const int c0 = (tid >> 5) * 4;       // column NT (c0 + q / NT) + q % NT
#pragma unroll
    for (int q = 0; q < 4 * NT; ++q) *reinterpret_cast<u32x2 *>(&sm.gs[32 * (q % NT) + c0 + q / NT][jq]) = o[q];
}

// The vectors x_j = (y_j - c, |y_j - c|^2, 1) go to LDS as [j][slot], one event per
// thread of the first two waves (padding events j >= n get y_j = c, so every psi stays
// finite).  The groups of 8 slots past the last term are the same for every event.
template <int KA>
struct Event {
    float y[KA - 2];
};

template <int KA>
__device__ __forceinline__ void load_events(const EParams &p, int64_t j0, Event<KA> &pd)
{
    const int tid = threadIdx.x;
    if (tid >= JC) return;
    if (j0 + JC <= p.n) {
#pragma unroll
        for (int d = 0; d < KA - 2; ++d)
            pd.y[d] = d < KA - 3 || d < p.D ? ld<float>(p.Y + d * p.ldY + j0, 4u * tid) : 0.0f;
    } else {
#pragma unroll
        for (int d = 0; d < KA - 2; ++d) pd.y[d] = (d < p.D && j0 + tid < p.n) ? p.Y[d * p.ldY + j0 + tid] : 0.0f;
    }
}

template <int KA>
constexpr int slot_groups() { return (3 * KA + 7) / 8; }

template <int NT, int KA, bool SAFE>
__device__ __forceinline__ void fill_slots(Smem<NT, SAFE> &sm)
{
    const uint16_t none[KA] = {};
    const int tid = threadIdx.x;
#pragma unroll
    for (int q = slot_groups<KA>(); q < 4; ++q) {
        u32x4 w;
#pragma unroll
        for (int e = 0; e < 4; ++e)
            w[e] = (uint32_t)slot<KA, true>(none, none, 8 * q + 2 * e) |
                   ((uint32_t)slot<KA, true>(none, none, 8 * q + 2 * e + 1) << 16);
        *reinterpret_cast<u32x4 *>(&sm.xh[tid / JC][tid % JC][8 * q]) = w;
    }
}

template <int NT, int KA, bool SAFE>
__device__ __forceinline__ void store_events(const EParams &p, Smem<NT, SAFE> &sm, int b, int64_t j0, const Event<KA> &pd)
{
    const int tid = threadIdx.x;
    if (tid >= JC) return;
    const bool real = j0 + JC <= p.n || j0 + tid < p.n;
    const bool all = p.D == KA - 2;             // else D = KA - 3
    float x[KA];
    float nrm = 0.0f;
#pragma unroll
    for (int d = 0; d < KA - 2; ++d) {
        const float v = (d < KA - 3 || all) && real ? pd.y[d] * p.yscale - sm.cen[d] : 0.0f;
        nrm = fmaf(v, v, nrm);
        x[d] = v;
        if constexpr (SAFE) sm.yc[b][d][tid] = real ? pd.y[d] : 0.0f;
    }
    if constexpr (SAFE) {
        const bool far = !(nrm <= VMAX2);
        const bool any = __any(far) != 0;
        if ((tid & 63) == 0) sm.far[b][tid >> 6] = any;
        if (far) {
            nrm = 0.0f;
#pragma unroll
            for (int k = 0; k < KA - 2; ++k) x[k] = 0.0f;
        }
    }
    x[KA - 3] = all ? x[KA - 3] : nrm;
    x[KA - 2] = all ? nrm : 1.0f;
    x[KA - 1] = all ? 1.0f : 0.0f;
    uint16_t hi[KA], lo[KA];
    split16<KA>(x, hi, lo);
#pragma unroll
    for (int q = 0; q < slot_groups<KA>(); ++q) {
        u32x4 w;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int s0 = 8 * q + 2 * e;
            w[e] = (uint32_t)slot<KA, true>(hi, lo, s0) | ((uint32_t)slot<KA, true>(hi, lo, s0 + 1) << 16);
        }
        *reinterpret_cast<u32x4 *>(&sm.xh[b][tid][8 * q]) = w;
    }
}

// Squared distances (minus 14) of local j = jb .. jb + 31 against the wave's 32
// rows, 32 float16 slots of the column and row vectors (two
// v_mfma_f32_32x32x16_f16): lane (col, h) gets row col and the 16 j =
// jb + 8 (r / 4) + 4 h + r % 4, r < 16.  DIRECT (SAFE form only): as direct
// float32 differences of the raw coordinates instead, |(y_i - y_j) yscale|^2 - 14,
// in the same lane layout.
template <int NT, int NS, bool SAFE, bool DIRECT>
__device__ __forceinline__ f32x16 distances(const Smem<NT, SAFE> &sm, int b, const Rows<NT, NS, SAFE> &rb, int jb, int D,
                                            float yscale)
{
    const int lane = threadIdx.x & 63;
    const int h = lane >> 5;
    const int col = lane & 31;
    f32x16 dd = f32x16{};
    if constexpr (DIRECT) {
        // Coordinate by coordinate, so that a read gives it for 4 rows and only 16
        // values are held beside the sums (read row by row, the rows' coordinates
        // filled the registers).  No branch: a coordinate beyond D is 0 on both
        // sides and adds (0 x 0)^2; with one per row, each row's reads were waited
        // for in turn (5e4 events x 32 columns, 3 coordinates, all out of range: 733
        // against 680 us).
#pragma unroll
        for (int d = 0; d < 2 * NS - 2; ++d) {
            const float scale = d < 2 * NS - 3 || D == 2 * NS - 2 ? yscale : 0.0f;
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const f32x4 y = *reinterpret_cast<const f32x4 *>(&sm.yc[b][d][jb + 8 * g + 4 * h]);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float t = (rb.y[d] - y[e]) * scale;
                    dd[4 * g + e] = fmaf(t, t, dd[4 * g + e]);
                }
            }
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) dd[r] -= PSI_LOG2;
    } else {
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            const f16x8 A = *reinterpret_cast<const f16x8 *>(&sm.xh[b][jb + col][16 * m + 8 * h]);
            dd = __builtin_amdgcn_mfma_f32_32x32x16_f16(A, __builtin_bit_cast(f16x8, rb.xi[m]), dd, 0, 0, 0);
        }
    }
    return dd;
}

// psi * 2^14 = 2^-dd of one step, split into float16 hi and lo: the operand
// tiles of the contraction.  Taken in pairs k of r = 2 k, 2 k + 1, the values
// for r < 8 are the lane's 8 consecutive k of the first 32 x 16 psi tile and
// r >= 8 those of the second; k = 8 h + (r % 8) stands for local
// j = 8 (r % 8 / 4) + 4 h + r % 4 (+16 for the second tile), which is k with
// bits 2 and 3 swapped, the order in which the columns are staged.
struct Psi {
    u32x4 hi[2], lo[2];
};

// Pair k of a step at local j = jb.  MASK keeps only j > rel (rel = i - j0),
// needed only in the chunk that holds the diagonal.
template <bool MASK>
__device__ __forceinline__ void psi_pair(const f32x16 &dd, int k, int jb, int rel, Psi &o)
{
    const int h = (threadIdx.x >> 5) & 1;
    const int r = 2 * k;
    float a = __builtin_amdgcn_exp2f(-dd[r]);
    float b = __builtin_amdgcn_exp2f(-dd[r + 1]);
    if (MASK) {
        const int ja = jb + 8 * (r >> 2) + 4 * h + (r & 3);
        a = (ja > rel) ? a : 0.0f;
        b = (ja + 1 > rel) ? b : 0.0f;
    }
    const uint32_t hw = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(a, b));
    // residuals a - hi_a, b - hi_b, each one mixed-precision multiply-add
    // reading its float16 half of hw directly (exact: hi is a truncation of a)
    float ra, rb;
    asm("v_fma_mix_f32 %0, -%1, 1.0, %2 op_sel_hi:[1,0,0]" : "=v"(ra) : "v"(hw), "v"(a));
    asm("v_fma_mix_f32 %0, -%1, 1.0, %2 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(rb) : "v"(hw), "v"(b));
    o.hi[k >> 2][k & 3] = hw;
    o.lo[k >> 2][k & 3] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(ra, rb));
}

// psi of a chunk's first step.
template <int NT, int NS>
__device__ __forceinline__ void first_psi(const Smem<NT, false> &sm, int b, const Rows<NT, NS, false> &rb, Psi &cur)
{
    const f32x16 dd = distances<NT, NS, false, false>(sm, b, rb, 0, 0, 0.0f);
#pragma unroll
    for (int k = 0; k < 8; ++k) psi_pair<false>(dd, k, 0, 0, cur);
}

// psi products of one staged chunk into the float32 tiles, 32 j per step, the
// steps pipelined in each wave: while the matrix cores contract step s (4 NT
// MFMAs), the vector ALU forms psi of step s + 1 from the distances issued just
// ahead.  An MFMA holds the matrix core for 32 cycles and the wave's issue for
// 4, so the psi instructions (16 exp2 and 32 conversions and residuals, about
// 270 cycles a step) fit between the MFMAs (512 cycles a step at 128 columns);
// the fences keep the interleaving, which the scheduler would undo.  The
// pipeline runs on into the next chunk: ``cur`` enters holding psi of this
// chunk's first step and leaves with that of the next one's, which is of use
// when that is the row block's next chunk.  The SAFE form goes step by step
// instead (step_products): its time is the direct distances on the vector ALU,
// and with their coordinates the pipelined form spilled 50 to 110 registers (9e3
// events x 64 columns, 8 coordinates, out of range: 112 us with it, 97 us
// without; 2e4 x 128, 4 coordinates: 239 and 225 us).
template <int NT, int NS>
__device__ __forceinline__ void chunk_products(const Smem<NT, false> &sm, int b, const Rows<NT, NS, false> &rb,
                                               f32x16 (&acc)[NT], Psi &cur)
{
    const int lane = threadIdx.x & 63;
    const int h = lane >> 5;
    const int col = lane & 31;
    constexpr int Q = 2 * NT;             // (psi tile, column tile) items per step
    constexpr int STEPS = JC / (2 * KS);
    // operand of item e (counted over the chunk's steps), read one item ahead of its use
    auto column = [&](int e) {
        const int jb = e / Q * 2 * KS, q = e % Q;
        return *reinterpret_cast<const f16x8 *>(&sm.gs[32 * (q % NT) + col][jb + KS * (q / NT) + 8 * h]);
    };
    f16x8 B0 = column(0);
#pragma unroll
    for (int st = 0; st < STEPS; ++st) {
        const bool last = st + 1 == STEPS;
        const f32x16 dd = last ? distances<NT, NS, false, false>(sm, b ^ 1, rb, 0, 0, 0.0f)
                               : distances<NT, NS, false, false>(sm, b, rb, (st + 1) * 2 * KS, 0, 0.0f);
        Psi next;
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const int e = st * Q + q, m = q / NT, t = q % NT;
            const f16x8 B = B0;
            if (e + 1 < STEPS * Q) B0 = column(e + 1);
            acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, cur.hi[m]), B, acc[t], 0, 0, 0);
            acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, cur.lo[m]), B, acc[t], 0, 0, 0);
#pragma unroll
            for (int k = 8 * q / Q; k < 8 * (q + 1) / Q; ++k)
                psi_pair<false>(dd, k, 0, 0, next);
            __builtin_amdgcn_sched_barrier(0);
        }
        cur = next;
    }
}

// A chunk step by step: the one that holds the diagonal of the wave's rows
// (MASK: psi only for j > rel), which is its row block's first, and every chunk
// of the SAFE form.
template <int NT, int NS, bool SAFE, bool DIRECT, bool MASK>
__device__ __forceinline__ void step_products(const Smem<NT, SAFE> &sm, int b, const Rows<NT, NS, SAFE> &rb, int rel,
                                              f32x16 (&acc)[NT], int D, float yscale)
{
    const int lane = threadIdx.x & 63;
    const int h = lane >> 5;
    const int col = lane & 31;
#pragma unroll 1
    for (int jb = 0; jb < JC; jb += 2 * KS) {
        const f32x16 dd = distances<NT, NS, SAFE, DIRECT>(sm, b, rb, jb, D, yscale);
        Psi psi;
#pragma unroll
        for (int k = 0; k < 8; ++k) psi_pair<MASK>(dd, k, jb, rel, psi);
#pragma unroll
        for (int q = 0; q < 2 * NT; ++q) {
            const int m = q / NT, t = q % NT;
            const f16x8 B = *reinterpret_cast<const f16x8 *>(&sm.gs[32 * t + col][jb + KS * m + 8 * h]);
            acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, psi.hi[m]), B, acc[t], 0, 0, 0);
            acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, psi.lo[m]), B, acc[t], 0, 0, 0);
        }
    }
}

// Value of lane Q < 16 of each half of the wave, in all its lanes: broadcast in
// the rows of 16 lanes, then from the last lane of the first and third row to the
// second and fourth (two moves on the vector ALU, no trip through LDS).
template <int Q>
__device__ __forceinline__ uint32_t half_lane(uint32_t x)
{
    const int t = __builtin_amdgcn_update_dpp((int)x, (int)x, 0x150 + Q, 0xf, 0xf, false);
    return (uint32_t)__builtin_amdgcn_update_dpp(t, t, 0x142, 0xa, 0xf, false);
}

// Row weight q of row r, and (Psi_upper w_q) of it: column q of G and of the tiles.
template <int NT, int Q>
__device__ __forceinline__ void weight(const uint32_t (&g)[16], const f32x16 (&acc)[NT], int r, float &w, float &u)
{
    w = (float)((half_lane<Q / NT>(g[r]) >> (8 * (Q % NT))) & 255u);
    const float a = acc[Q % NT][r];     // bits are taken from a scalar: of an element in place they are element 0's
    u = __builtin_bit_cast(float, half_lane<Q / NT>(__builtin_bit_cast(uint32_t, a)));
}

// Reduce the float32 tiles into the float64 partials and clear them.  The
// leading R columns are the row weights; their values (Psi_upper w_q)_i come
// from the lane that holds them, so that every column can take the transposed
// term sum_i G_ic (Psi_upper w_q)_i.
template <int NT, int NS, int RR, bool SAFE>
__device__ __forceinline__ void flush(const Rows<NT, NS, SAFE> &rb, f32x16 (&acc)[NT], double (&part)[NT][1 + RR])
{
    float s0[NT], s1[NT], s2[NT], s3[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) s0[t] = s1[t] = s2[t] = s3[t] = 0.0f;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        float w[3], u[3];
        weight<NT, 0>(rb.g, acc, r, w[0], u[0]);
        if constexpr (RR > 1) weight<NT, 1>(rb.g, acc, r, w[1], u[1]);
        if constexpr (RR > 2) weight<NT, 2>(rb.g, acc, r, w[2], u[2]);
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const float v = acc[t][r];
            const float g = (float)((rb.g[r] >> (8 * t)) & 255u);
            s0[t] = fmaf(g, v, s0[t]);
            s1[t] = fmaf(w[0], v, fmaf(g, u[0], s1[t]));
            if constexpr (RR > 1) s2[t] = fmaf(w[1], v, fmaf(g, u[1], s2[t]));
            if constexpr (RR > 2) s3[t] = fmaf(w[2], v, fmaf(g, u[2], s3[t]));
        }
    }
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        part[t][0] += 2.0 * (double)s0[t];       // diagonal-type sums are symmetric
        part[t][1] += (double)s1[t];
        if (RR > 1) part[t][RR > 1 ? 2 : 1] += (double)s2[t];
        if (RR > 2) part[t][RR > 2 ? 3 : 1] += (double)s3[t];
        acc[t] = f32x16{};
    }
}

// Work split.  Row blocks g and nb - 1 - g pair up (together nb + 1 chunks);
// their chunks, block g's first, form one list, and the lists of all pairs in
// turn one sequence of chunks.  Float32 accumulation runs over segments of
// this sequence: a pair's list is cut into K equal pieces, a piece at the row
// block's end, and the rest every FL chunks.  A workgroup takes a contiguous
// share of the sequence, rounded to segments, so a share costs one set-up and
// one reduction however small the pieces are, and the float32 sums do not
// depend on how many workgroups there are or which share each takes.  (One
// workgroup per piece instead: at 3e4 events pieces of two chunks, 13.8 k
// workgroups, each with its centre, its rows' columns, and 256 float64 atomics
// on the same addresses as the others': 0.533 ms against 0.353 ms, 128 columns.)
// All positions fit 32 bits: nb < 2^26 for any sample that fits in memory, and
// K (nb + 1) < 2^15 + 2 nb.
struct Seq {
    uint32_t nb, K;
    __device__ __forceinline__ uint32_t len1(uint32_t g) const { return nb - g; }            // chunks of block g's row
    __device__ __forceinline__ uint32_t len(uint32_t g) const                                 // of the pair's list
    {
        return 2 * g + 1 == nb ? nb - g : nb + 1;
    }
    // the run of segments (a piece, cut at the row block's end) of pair g that
    // holds list position v: its first position, end
    __device__ __forceinline__ void run(uint32_t g, uint32_t v, uint32_t &a, uint32_t &b) const
    {
        const uint32_t L1 = len1(g), L = len(g);
        const uint32_t k = ((v + 1) * K - 1) / L;
        a = k * L / K;
        b = (k + 1) * L / K;
        if (v < L1) b = b < L1 ? b : L1;
        else a = a > L1 ? a : L1;
    }
    // list position v of pair g, rounded down to a segment's start
    __device__ __forceinline__ uint32_t round(uint32_t g, uint32_t v) const
    {
        if (v >= len(g)) return v;
        uint32_t a, b;
        run(g, v, a, b);
        return a + (v - a) / FL * FL;
    }
};

// RR: row-weight columns the reduction carries (RR covers R <= RR).
//
// What bounds it: the 18 MFMAs per 32 x 32 pairs (128 columns, 576 cycles), and
// the power they draw: products alone, on data that stays in LDS, run at 1.8 GHz
// with the matrix cores 86 % busy.  The vector ALU's psi work, staging and
// flush (about 350 instructions per wave and chunk beside 72 MFMAs) share the
// issue, so the loop over the chunks of a segment holds nothing else: the
// diagonal, the row set-up and the flush stand outside it, which also keeps the
// accumulators in place and everything in registers (with the diagonal's mask
// as a variant inside it the loop carried 70 moves and scratch reloads, and
// the reloads waited for the loads of the next chunk).  At 3e5 events x 128
// columns: 23.6 ms with the products unpipelined, 20.2 ms with them pipelined
// inside a chunk, 18.5 ms in this form.
//
// At 3e4 events a share is 54 chunks and the flushes count: a lane holds its
// columns' bytes of its 16 rows (Rows), converts them one byte at a time, and
// takes the row weights' values by lane broadcasts on the vector ALU.  With
// the bytes reread as eight selects per row and the weights through LDS
// permutes: 0.316 ms against 0.290 ms (128 columns), 0.203 against 0.177 ms
// (32).  Below 1e4 a workgroup has two chunks and the time is the latency of
// its set-up, so the loads of that are issued together: 5e3 events x 128
// columns, 5 coordinates, 33.5 us a call with them in turn, 28.1 us so.
template <int NT, int NS, int RR, bool SAFE>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(NT == 4 ? 2 : 3)))
void tp_pairsum_kernel(const EParams p, const uint32_t K, const uint32_t S, const uint32_t total)
{
    constexpr int C = 32 * NT;
    constexpr int KA = 2 * NS;
    // the range check's flag selects the one instantiation that works
    const bool flagged = __atomic_load_n(p.flag, __ATOMIC_RELAXED) != 0u;
    if (flagged != SAFE) return;
    __shared__ __align__(16) Smem<NT, SAFE> sm;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int h = lane >> 5;
    const int col = lane & 31;
    const Seq sq = { (uint32_t)((p.n + ROWS - 1) / ROWS), K };
    // this workgroup's share of the sequence of chunks, ``todo`` of them from
    // list position v0 of pair g0 on: with S > 0 one of S parts of a pair's list
    // (part r of every pair before part r + 1 of any, and each die given a run
    // of this order, so that the workgroups of a die read the same chunks at
    // about the same time), else an equal part of it all (``total`` < 2^32)
    uint32_t g0, v0, todo;
    if (S > 0) {
        const uint32_t pairs = (sq.nb + 1) / 2, units = gridDim.x;
        const uint32_t xcd = blockIdx.x % XCDS, slot = blockIdx.x / XCDS;
        const uint32_t u = xcd * (units / XCDS) + (xcd < units % XCDS ? xcd : units % XCDS) + slot;
        const uint32_t r = u / pairs;
        g0 = u - r * pairs;
        const uint32_t L = sq.len(g0);
        v0 = sq.round(g0, r * L / S);
        todo = sq.round(g0, r + 1 < S ? (r + 1) * L / S : L) - v0;
    } else {
        const uint32_t share = total / gridDim.x, extra = total % gridDim.x, wg = blockIdx.x;
        const uint32_t p0 = wg * share + (wg < extra ? wg : extra), p1 = p0 + share + (wg < extra ? 1 : 0);
        g0 = p0 / (sq.nb + 1);
        const uint32_t g1 = p1 / (sq.nb + 1), at0 = g0 * (sq.nb + 1), at1 = g1 * (sq.nb + 1);
        v0 = sq.round(g0, p0 - at0);
        todo = (p1 < total ? at1 + sq.round(g1, p1 - at1) : total) - (at0 + v0);
    }
    if (todo > 0) {
        // the loads of the set-up, all in flight together: a small sample's time is
        // made of such latencies
        float cy[KA - 2];
        load_coords<KA - 2>(p, tid, cy);
        double part[NT][1 + RR];
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int q = 0; q <= RR; ++q) part[t][q] = 0.0;
        f32x16 acc[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[t] = f32x16{};
        // cursors of the sequence: this chunk, the next, the one after
        struct Cursor { uint32_t g, v; };
        auto after = [&](Cursor c) { return c.v + 1 < sq.len(c.g) ? Cursor{ c.g, c.v + 1 } : Cursor{ c.g + 1, 0u }; };
        // ROWS == JC: a row block starts a chunk, and its first chunk holds the diagonal
        auto chunk_j0 = [&](Cursor c) {
            const uint32_t L1 = sq.len1(c.g);
            return (int64_t)(c.v < L1 ? c.g + c.v : sq.nb - 1 - c.g + (c.v - L1)) * JC;
        };
        Cursor at = { g0, v0 }, at1 = after(at);
        Columns<NT> cols;
        Event<KA> ev;
        Rows<NT, NS, SAFE> rb;
        uint32_t blk;       // the row block of rb
        {
            const int64_t j0 = chunk_j0(at);
            load_columns<NT>(p, j0, cols);
            load_events<KA>(p, j0, ev);
            RowLoads<NT, NS> rl;
            blk = at.v < sq.len1(at.g) ? at.g : sq.nb - 1 - at.g;
            load_rows<NT, NS>(p, (int64_t)blk * ROWS + wave * 32, rl);
            for (int e = tid; e < C * (1 + MAXR); e += 256) (&sm.red[0][0])[e] = 0.0;
            fill_slots<NT, KA, SAFE>(sm);
            centre<KA - 2>(p, sm, cy);
            store_events<NT, KA, SAFE>(p, sm, 0, j0, ev);
            if (todo > 1) load_events<KA>(p, chunk_j0(at1), ev);
            setup_rows<NT, NS, SAFE>(p, sm, (int64_t)blk * ROWS, (int64_t)blk * ROWS + wave * 32, rl, rb);
        }
        __syncthreads();
        Psi cur;
        bool primed = false;
        int b = 0;
        const int rel = wave * 32 + col;
        // this chunk's columns and the next one's vectors to LDS, the loads after them issued
        auto stage = [&]() {
            u32x2 o[4 * NT];
            expand_columns<NT>(cols, o);
            __syncthreads();                    // the last chunk's columns have been read
            store_columns<NT, SAFE>(sm, o);
            if (todo > 1) store_events<NT, KA, SAFE>(p, sm, b ^ 1, chunk_j0(at1), ev);
            __syncthreads();
            const Cursor at2 = after(at1);
            if (todo > 1) load_columns<NT>(p, chunk_j0(at1), cols);
            if (todo > 2) load_events<KA>(p, chunk_j0(at2), ev);
            at = at1;
            at1 = at2;
            --todo;
        };
        uint32_t run_end = 0;
        while (todo > 0) {
            const uint32_t L1 = sq.len1(at.g), L = sq.len(at.g);
            const uint32_t row = at.v < L1 ? at.g : sq.nb - 1 - at.g;
            if (at.v == 0 || run_end == 0 || at.v == run_end) {
                uint32_t a;
                sq.run(at.g, at.v, a, run_end);
            }
            uint32_t left = run_end - at.v < FL ? run_end - at.v : FL;      // chunks of this segment
            const uint32_t s1 = at.v + left;
            const bool diag = at.v == 0 || at.v == L1, more = s1 != L1 && s1 != L && left < todo;
            if (row != blk) {
                RowLoads<NT, NS> rl;
                load_rows<NT, NS>(p, (int64_t)row * ROWS + wave * 32, rl);
                setup_rows<NT, NS, SAFE>(p, sm, (int64_t)row * ROWS, (int64_t)row * ROWS + wave * 32, rl, rb);
                blk = row;
                primed = false;
            }
            if (diag) {
                stage();
                if (SAFE && (rb.far || (sm.far[b][0] | sm.far[b][1]) != 0u))
                    step_products<NT, NS, SAFE, SAFE, true>(sm, b, rb, rel, acc, p.D, p.yscale);
                else step_products<NT, NS, SAFE, false, true>(sm, b, rb, rel, acc, p.D, p.yscale);
                b ^= 1;
                --left;
            }
            if (left > 0) {
                if constexpr (!SAFE)
                    if (!primed) first_psi<NT, NS>(sm, b, rb, cur);
                do {
                    stage();
                    if constexpr (!SAFE) chunk_products<NT, NS>(sm, b, rb, acc, cur);
                    else if (rb.far || (sm.far[b][0] | sm.far[b][1]) != 0u)
                        step_products<NT, NS, SAFE, true, false>(sm, b, rb, rel, acc, p.D, p.yscale);
                    else step_products<NT, NS, SAFE, false, false>(sm, b, rb, rel, acc, p.D, p.yscale);
                    b ^= 1;
                } while (--left > 0);
                primed = more;
            }
            flush<NT, NS, RR, SAFE>(rb, acc, part);
        }
        // combine the two row halves of each column, then the four waves, then workgroups
        const int R = p.R;
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int q = 0; q <= RR; ++q) {
                double x = part[t][q];
                x += __shfl_xor(x, 32);
                if (h == 0 && q <= R) atomicAdd(&sm.red[NT * col + t][q], x);
            }
        __syncthreads();
        for (int e = tid; e < C * (1 + R); e += 256) {
            const int c = e / (1 + R), q = e % (1 + R);
            if (c < p.C) atomicAdd(&p.sums[(int64_t)c * (1 + R) + q], sm.red[c][q] * PSI_UNSCALE);
        }
    }
    if constexpr (SAFE) {
        // the last workgroup clears the flag and the count for the next launch
        __shared__ bool last;
        __syncthreads();
        if (tid == 0) {
            __threadfence();
            last = atomicAdd(p.flag + 1, 1u) == gridDim.x - 1;
        }
        __syncthreads();
        if (last && tid == 0) {
            p.flag[0] = 0u;
            p.flag[1] = 0u;
            __threadfence();
        }
    }
}

// Range check: sets p.flag[0] when any event lies outside the matrix-core
// range of the centre (|v|^2 > VMAX2, or not finite), with the same centre
// and the same arithmetic as the pair-sum kernels.
__global__ __launch_bounds__(256) void tp_range_kernel(const EParams p)
{
    __shared__ CentreSmem sm;
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    float cy[MAXD], y[MAXD];
    load_coords<MAXD>(p, threadIdx.x, cy);
    load_coords<MAXD>(p, i, y);
    centre<MAXD>(p, sm, cy);
    if (i >= p.n) return;
    float nrm = 0.0f;
#pragma unroll
    for (int d = 0; d < MAXD; ++d) {
        const float v = y[d] * p.yscale - sm.cen[d];
        nrm = d < p.D ? fmaf(v, v, nrm) : nrm;
    }
    if (!(nrm <= VMAX2)) atomicOr(p.flag, 1u);
}

template <int NT, int NS, int RR>
hipError_t launch_ntd(const EParams &p, hipStream_t st)
{
    const int64_t nb = (p.n + ROWS - 1) / ROWS;
    const int64_t pairs = (nb + 1) / 2;
    // pieces per block pair: about 16 k in all, none shorter than two chunks
    int64_t K = (16384 + pairs - 1) / pairs;
    K = K > nb / 2 ? nb / 2 : K;
    K = K < 1 ? 1 : K;
    // Shares of at least about 64 chunks keep a workgroup's set-up and reduction
    // below a few percent.  A sample that does not fit an L2 is split by pairs
    // and parts (S), the number of parts chosen for full rounds of resident
    // workgroups: at 3e5 events the L2 misses fall from 72 to 2 % of the
    // requests, the time from 19.9 to 19.5 ms.  A smaller one (or one with too
    // few pairs for that) is split evenly, in up to 16 full rounds.  The rounds of
    // a split by parts are of RESIDENT workgroups at every width (measured at 128
    // columns only; three fit a compute unit at 32 and 64, see below).
    const int64_t total = nb * (nb + 1) / 2;
    int64_t S = 0, grid = total / 64;
    if (p.n * (p.C + 4 * p.D) > L2_BYTES && pairs * 2 > RESIDENT) {
        double best = 0.0;      // full rounds, times the share of a part that is not its set-up
        for (int64_t s = 1; s <= 64; ++s) {
            const int64_t u = pairs * s, len = (nb + 1) / s;
            if (s > 1 && (len < 48 || u > 32 * RESIDENT)) break;
            const double rounds = (double)u / RESIDENT, full = (double)((u + RESIDENT - 1) / RESIDENT);
            const double score = rounds / full * (double)len / (double)(len + 2);
            if (score > best) {
                best = score;
                S = s;
            }
        }
        grid = pairs * S;
    } else {
        // With 32 or 64 columns three workgroups fit a compute unit.  From 6
        // chunks a share on all three are used: 4e4 events x 32 columns 273 us
        // with two, 240 with three; x 64 330 and 303; 12345 x 64 52 and 49; at
        // 9000 (3 chunks a share) 38 and 41.  (Out-of-range samples: 5e4 x 32
        // 899 and 721, 3e4 x 64 432 and 407.)
        const int64_t resident = NT < 4 && total >= 6 * (RESIDENT + RESIDENT / 2) ? RESIDENT + RESIDENT / 2 : RESIDENT;
        grid = grid < resident ? resident : grid > 16 * resident ? 16 * resident : grid / resident * resident;
        if (grid > (total + 1) / 2) grid = (total + 1) / 2;
    }
    // one of the two instantiations works (the range check's flag), the other exits
    const hipError_t e = launch(tp_pairsum_kernel<NT, NS, RR, false>, (unsigned)grid, 256, 0, st, p, (uint32_t)K,
                                (uint32_t)S, (uint32_t)total);
    if (e != hipSuccess) return e;
    return launch(tp_pairsum_kernel<NT, NS, RR, true>, (unsigned)grid, 256, 0, st, p, (uint32_t)K, (uint32_t)S,
                  (uint32_t)total);
}

template <int NT, int RR>
hipError_t launch_ntr(const EParams &p, hipStream_t st)
{
    switch (p.D) {   // distance-vector components D + 2, in pairs
    case 1: case 2: return launch_ntd<NT, 2, RR>(p, st);
    case 3: case 4: return launch_ntd<NT, 3, RR>(p, st);
    case 5: case 6: return launch_ntd<NT, 4, RR>(p, st);
    default: return launch_ntd<NT, 5, RR>(p, st);
    }
}

template <int NT>
hipError_t launch_nt(const EParams &p, hipStream_t st)
{
    if (p.R <= 1) return launch_ntr<NT, 1>(p, st);
    if (p.R == 2) return launch_ntr<NT, 2>(p, st);
    return launch_ntr<NT, 3>(p, st);
}

// Certified order of two pair masses m^2(a, b) against m^2(c, d): +1 if
// larger, -1 if smaller, 0 if equal.  float64 with the magnitude bound
// |m^2_computed - m^2| <= 8u (sum_q |x_aq| + |x_bq|)^2 (one rounding for each
// component sum, four for the squares and their sum), exact integers when the
// two intervals overlap.
template <typename Tin>
__device__ int pair_cmp(const double (&x)[4][4], int a, int b, int c, int d)
{
    double m2[2], mag[2];
    const int sl[2][2] = { { a, b }, { c, d } };
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        double S[4], A = 0.0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            S[q] = x[sl[k][0]][q] + x[sl[k][1]][q];
            A += __builtin_fabs(x[sl[k][0]][q]) + __builtin_fabs(x[sl[k][1]][q]);
        }
        m2[k] = fma(-S[3], S[3], fma(-S[2], S[2], fma(-S[1], S[1], S[0] * S[0])));
        mag[k] = fma(8.0 * 0x1p-53 * A, A, 0x1p-1000);
    }
    const double diff = m2[0] - m2[1];
    const double err = (mag[0] + mag[1]) * (1.0 + 0x1p-50);
    if (diff > err) return 1;
    if (diff < -err) return -1;
    int64_t mant[4][4];
    int ex[4][4];
    for (int s = 0; s < 4; ++s)
        for (int q = 0; q < 4; ++q) {
            if constexpr (sizeof(Tin) == 4) tpx::decode_f32((float)x[s][q], mant[s][q], ex[s][q]);
            else tpx::decode_f64(x[s][q], mant[s][q], ex[s][q]);
        }
    const int r = tpx::pair_mass2_cmp(mant, ex, sizeof(Tin) == 4 ? 136 : 107, a, b, c, d);
    return r == 2 ? 0 : r;
}

// Invariant mass of the slots in a mask, per event (Sect. 4.2 coordinates).
// With relabel 1 (D0 -> pi+ pi- pi+ pi-, slots in charge order + - + -) the
// event is first relabelled as Sect. 4.2 prescribes: of the four pi+ pi- pairs
// the one of largest invariant mass becomes pi3 pi4 (slots 2, 3), which fixes
// the order of all four pions.  Ties go to the first pair in the order
// (2,3), (0,1), (0,3), (2,1) (the stored labelling, then the swap of both
// pairs, of the pi+, of the pi-).
template <typename Tin>
__global__ void tp_coords_kernel(CParams c)
{
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= c.n) return;
    const Tin *const *P = reinterpret_cast<const Tin *const *>(c.p);
    double x[4][4];
    for (int s = 0; s < 4; ++s)
        for (int q = 0; q < 4; ++q) x[s][q] = (double)P[s * 4 + q][e];
    int perm[4] = { 0, 1, 2, 3 };   // new slot t holds stored slot perm[t]
    if (c.relabel == 1) {
        const int pa[4][2] = { { 2, 3 }, { 0, 1 }, { 0, 3 }, { 2, 1 } };
        const int pm[4][4] = { { 0, 1, 2, 3 }, { 2, 3, 0, 1 }, { 2, 1, 0, 3 }, { 0, 3, 2, 1 } };
        int best = 0;
        for (int k = 1; k < 4; ++k)
            if (pair_cmp<Tin>(x, pa[k][0], pa[k][1], pa[best][0], pa[best][1]) > 0) best = k;
        for (int t = 0; t < 4; ++t) perm[t] = pm[best][t];
    }
    for (int k = 0; k < c.ncoord; ++k) {
        double S[4] = { 0.0, 0.0, 0.0, 0.0 };
        for (int s = 0; s < 4; ++s)
            if (c.masks[k] & (1 << s))
                for (int q = 0; q < 4; ++q) S[q] += x[perm[s]][q];
        const double m2 = S[0] * S[0] - S[1] * S[1] - S[2] * S[2] - S[3] * S[3];
        c.out[(int64_t)k * c.ldo + e] = (float)(m2 > 0.0 ? sqrt(m2) * c.scale : 0.0);
    }
}

}  // namespace

hipError_t launch_pairsums(const EParams &p, hipStream_t st)
{
    if (p.C != 32 && p.C != 64 && p.C != 128) return hipErrorInvalidValue;
    const hipError_t e = launch(tp_range_kernel, (unsigned)((p.n + 255) / 256), 256, 0, st, p);
    if (e != hipSuccess) return e;
    return p.C == 32 ? launch_nt<1>(p, st) : p.C == 64 ? launch_nt<2>(p, st) : launch_nt<4>(p, st);
}

hipError_t launch_coords(const CParams &c, int dtype, hipStream_t st)
{
    const int64_t grid = (c.n + 255) / 256;
    return dtype == 0 ? launch(tp_coords_kernel<float>, (unsigned)grid, 256, 0, st, c)
                      : launch(tp_coords_kernel<double>, (unsigned)grid, 256, 0, st, c);
}

}  // namespace tpe
