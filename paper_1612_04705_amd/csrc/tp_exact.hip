// Last tiers of the T-odd pass: the events the float64 tier could not decide,
// taken from the work list and decided first in certified double-word
// arithmetic (tp_dword.h) and, if that does not settle them, in exact integer
// arithmetic (tp_exact.h): validity, sign of the triple product (Sect. 5,
// eq. (4)) and every bin-edge comparison.  Results are added to the sample's counters with
// device-scope atomics; the last workgroup clears the list for the next launch.
#include <hip/hip_runtime.h>

#define TP_HD __host__ __device__
#include "tp_dword.h"
#include "tp_exact.h"
#include "tp_kernel.h"
#include "tp_launch.h"

namespace tpk {
namespace {

__device__ __forceinline__ double dabs(double x) { return __builtin_fabs(x); }

// Rest-frame energy order of kernel slots lo, lo + 2 in float64 (the pass's
// test: s = P.(p_lo - p_hi) against 8.1u W (w_lo + w_hi)): +1 if p_lo is
// faster, -1 if slower, 0 if the bound does not settle it.
__device__ __forceinline__ int order_f64(const double (&x)[4][4], int lo)
{
    const int hi = lo + 2;
    double P[4], w[4], W = 0.0;
    for (int c = 0; c < 4; ++c) P[c] = (x[0][c] + x[1][c]) + (x[2][c] + x[3][c]);
    for (int k = 0; k < 4; ++k) {
        w[k] = (dabs(x[k][0]) + dabs(x[k][1])) + (dabs(x[k][2]) + dabs(x[k][3]));
        W += w[k];
    }
    double d[4];
    for (int c = 0; c < 4; ++c) d[c] = x[lo][c] - x[hi][c];
    const double sv = fma(-P[3], d[3], fma(-P[2], d[2], fma(-P[1], d[1], P[0] * d[0])));
    const double bound = fma((8.2 * 0x1p-53) * W, w[lo] + w[hi], 0x1p-1000);
    if (!(dabs(sv) > bound)) return 0;
    return sv > 0.0 ? 1 : -1;
}

// ------------------------------------------------- double words on 16 lanes
// tpw::decide_dw of one event by a group of 16 lanes.  A listed event's
// decisions are a chain of some 7,700 dependent float64 instructions on one lane,
// about 20 us however few events there are, and a launch that lists any waits
// for it.  Here lane l = 4 a + b of the group forms the quantities of its own
// index -- P_b, the products p_a.p_b, G_ab, one Laplace term, one square, every
// 16th edge -- and the lanes exchange them, which leaves about a seventh of the
// chain.  The values are the same invariants with the same running bounds (only
// the order of some sums differs, and each sum carries its own bound), so every
// decision it certifies is the exact one.
using tpw::V;

__device__ __forceinline__ V vget(const V &x, int src)      // x of lane src of the wave
{
    return V{ { __shfl(x.v.hi, src), __shfl(x.v.lo, src) }, __shfl(x.e, src) };
}

__device__ __forceinline__ V vsum(V x, int lanes)            // sum over aligned runs of ``lanes`` lanes
{
    for (int o = 1; o < lanes; o <<= 1)
        x = tpw::add(x, V{ { __shfl_xor(x.v.hi, o), __shfl_xor(x.v.lo, o) }, __shfl_xor(x.e, o) });
    return x;
}

__device__ __forceinline__ double pick(const double (&r)[4], int c)
{
    const double lo = c & 1 ? r[1] : r[0], hi = c & 1 ? r[3] : r[2];
    return c & 2 ? hi : lo;
}

// The lanes of one group must enter together; ``base`` is its first lane.
__device__ __forceinline__ int decide_lanes(const double (&x)[4][4], int tag, const KSample &S, int nax,
                                         const double *const (&edges)[2], int base, int &bin)
{
    using namespace tpw;
    bin = -1;
    const int l = (int)(threadIdx.x & 15), a = l >> 2, b = l & 3;
    auto any = [&](bool p) { return ((__ballot(p) >> base) & 0xffffull) != 0; };
    auto count = [&](bool p) { return __popcll((__ballot(p) >> base) & 0xffffull); };
    if (tag != 0 && tag != 1) return W_INVALID;
    double xa[4], xb[4], col[4];                 // rows a and b, column b
    bool small = true;
    for (int s = 0; s < 4; ++s) {
        col[s] = pick(x[s], b);
        for (int c = 0; c < 4; ++c) {
            const double m = dabs(x[s][c]);
            small = small && (m == 0.0 || (m >= 0x1p-30 && m <= 0x1p40));
        }
    }
    if (!small) return W_UNCERTAIN;
    for (int c = 0; c < 4; ++c) {
        const double r[4] = { x[0][c], x[1][c], x[2][c], x[3][c] };
        xa[c] = pick(r, a);
        xb[c] = pick(r, b);
    }
    // P_b; M^2 = P_0^2 - P_1^2 - P_2^2 - P_3^2
    const V Pb = add(add(add(exact(col[0]), exact(col[1])), exact(col[2])), exact(col[3]));
    const V Pb2 = mul(Pb, Pb);
    const V M2 = vsum(b == 0 ? Pb2 : neg(Pb2), 4);
    const V P0 = vget(Pb, base), P02 = vget(Pb2, base);
    const int sE = csign(P0), sM = csign(M2);
    if (any(sE < 0 || sM < 0)) return W_INVALID;
    if (any(sE == 0 || sM == 0)) return W_UNCERTAIN;
    // Laplace term l & 7 (6 and 7: none) of det[x0; x1; x2; x3] on row pairs (0,1) | (2,3)
    V term = exact(0.0);
    {
        const int k = l & 7;
        const int i = k < 3 ? 0 : k < 5 ? 1 : 2, j = k < 3 ? k + 1 : k < 5 ? k - 1 : 3;      // its columns
        const int m = k < 1 ? 2 : k < 3 ? 1 : 0, n = k == 5 ? 1 : k == 2 || k == 4 ? 2 : 3;       // the other two, in order
        const V top = sub(prod(pick(x[0], i), pick(x[1], j)), prod(pick(x[0], j), pick(x[1], i)));
        const V bot = sub(prod(pick(x[2], m), pick(x[3], n)), prod(pick(x[2], n), pick(x[3], m)));
        const V t = mul(top, bot);
        if (k < 6) term = (k == 1 || k == 4) ? neg(t) : t;
    }
    const int sd = csign(vsum(term, 8)) * S.sigma;
    if (any(sd == 0)) return W_UNCERTAIN;
    const int cls = tag == 0 ? (sd > 0 ? W_I : W_II) : (sd < 0 ? W_III : W_IV);
    if (nax <= 0) return cls;

    const V d = mink(xa, xb);
    const V PPa = vsum(d, 4);
    const V PPb = vget(PPa, base + 4 * b);
    const V G = sub(mul(PPa, PPb), mul(M2, d));
    int bsum = 0;
    bool oor = false;
    for (int ax = 0; ax < nax; ++ax) {
        const int nb = S.nbins[ax];
        const double *e = edges[ax];
        int j = 0;
        bool bad = false;
        if (S.kind[ax] == AX_ABSPHI) {
            // lane b: X = G02 G13 - G03 G12, N1 = G00 G11 - G01^2, N2 = G22 G33 - G23^2
            const int i0 = b == 0 ? 2 : b == 1 ? 0 : 10, i1 = b == 0 ? 7 : b == 1 ? 5 : 15;
            const int i2 = b == 0 ? 3 : b == 1 ? 1 : 11, i3 = b == 0 ? 6 : b == 1 ? 1 : 11;
            const V Z = sub(mul(vget(G, base + i0), vget(G, base + i1)), mul(vget(G, base + i2), vget(G, base + i3)));
            const V X = vget(Z, base), D = mul(vget(Z, base + 1), vget(Z, base + 2)), X2 = mul(X, X);
            const int sX = csign(X);
            for (int k0 = 1; k0 < nb; k0 += 16) {
                const int k = k0 + l;
                int le = 0;
                if (k < nb) le = cos_le(sX, csign(sub(X2, mul(prod(e[k], e[k]), D))), e[k]);
                bad = bad || any(le < 0);
                j += count(le > 0);
            }
        } else if (S.kind[ax] == AX_ABSCOS) {
            const int s = S.slots[ax];
            const double r[4] = { x[0][0], x[1][0], x[2][0], x[3][0] };
            const V Nn = sub(mul(vget(PPa, base + 4 * s), P0), mul(M2, exact(pick(r, s))));
            const V AB = mul(vget(G, base + 5 * s), sub(P02, M2)), Nn2 = mul(Nn, Nn);
            for (int k0 = 1; k0 < nb; k0 += 16) {
                const int k = k0 + l;
                int sF = -1;
                if (k < nb) sF = csign(sub(Nn2, mul(prod(e[k], e[k]), AB)));
                bad = bad || any(sF == 0);
                j += count(sF > 0);
            }
        } else {
            V Sb = exact(0.0);
            for (int t = 0; t < 4; ++t)
                if (S.slots[ax] & (1 << t)) Sb = add(Sb, exact(col[t]));
            const V Sb2 = mul(Sb, Sb);
            const V m2 = vsum(b == 0 ? Sb2 : neg(Sb2), 4);
            for (int k0 = 0; k0 <= nb; k0 += 16) {
                const int k = k0 + l;
                int sF = -1;
                if (k <= nb) sF = csign(sub(m2, prod(e[k], e[k])));
                bad = bad || any(sF == 0);
                j += count(k > 0 && k < nb && sF > 0);
                oor = oor || any((k == 0 && sF < 0) || (k == nb && sF > 0));
            }
        }
        if (bad) return W_UNCERTAIN;
        bsum = bsum * nb + j;
    }
    bin = oor ? -1 : bsum;
    return cls;
}

// ------------------------------------------------------------------ exact tier
template <typename Tin, int MODE>
__global__ __launch_bounds__(64) void tp_exact_kernel(const KParams kp)
{
    const uint32_t cnt = __atomic_load_n(kp.xcount, __ATOMIC_RELAXED);
    const uint32_t n = cnt < kp.xcap ? cnt : kp.xcap;
    // fold the pass's replicated counters into the samples' and clear them
    for (int f = blockIdx.x; f < kp.nfold; f += gridDim.x) {
        const uint32_t item = kp.fold ? kp.fold[f] : (uint32_t)f;
        const KSample &S = kp.samples[kp.fold ? item >> 8 : 0];
        const int nrow = (S.nbtot + 1) * 4;
        const int w = (int)(item & 255u) * FOLD + (int)threadIdx.x;
        if (S.rep_off < 0 || w >= rep_words(S.nbtot)) continue;
        uint64_t *copy = kp.rep + S.rep_off + w;
        const int stride = rep_stride(S.nbtot), n = S.rep_mask + 1;
        uint64_t v[MAXREP], sum = 0;   // every copy's load in flight at once
#pragma unroll
        for (int r = 0; r < MAXREP; ++r) v[r] = r < n ? copy[(int64_t)r * stride] : 0;
#pragma unroll
        for (int r = 0; r < MAXREP; ++r) {
            sum += v[r];
            if (v[r]) copy[(int64_t)r * stride] = 0;
        }
        uint64_t *to = w < nrow ? (S.counts ? S.counts + w : nullptr) : S.stats + (w - nrow);
        if (sum && to) atomicAdd((unsigned long long *)to, (unsigned long long)sum);
    }
    // a list that the launch's groups of 16 lanes take in one go is decided by
    // groups (3e6 float32 events of a |cos theta| scheme, about 25 listed: the
    // launch 27 us by lanes, 16 by groups; 64-sample batch, 417 listed: 35 and
    // 22), a longer one by lanes, which spend half as many instructions per event
    const bool grouped = n <= gridDim.x * blockDim.x / 16;
    const uint32_t me = blockIdx.x * blockDim.x + threadIdx.x;
    for (uint32_t it = grouped ? me / 16 : me; it < n; it += gridDim.x * blockDim.x) {
        const uint64_t ent = kp.xlist[it];
        const int s = (int)((ent >> 40) & 0xfffff);
        const int64_t i = (int64_t)(ent & ((1ull << 40) - 1));
        const KSample &S = kp.samples[s];
        const int tag = S.tag[i];
        double xv[4][4];
        bool finite = true;
        for (int k = 0; k < 4; ++k)
            for (int c = 0; c < 4; ++c) {
                xv[k][c] = (double)reinterpret_cast<const Tin *>(S.p[k * 4 + c])[i];
                if (!isfinite(xv[k][c])) finite = false;
            }
        const double *eds[2] = { nullptr, nullptr };
        for (int a = 0; a < S.naxes && a < 2; ++a)
            eds[a] = kp.edges + S.eoff[a] + (S.kind[a] == AX_MASS ? 2 * (S.nbins[a] + 1) : 0);
        const int nax = MODE == 0 ? S.naxes : 0;
        const int span = sizeof(Tin) == 4 ? 136 : 107;
        // identical particles: exact rest-frame energy order first (an exact
        // tie keeps the stored order), then every decision on the ordered rows
        bool order_unres = false;
        int osg = (finite && S.olo >= 0) ? order_f64(xv, S.olo) : 0;
        if (osg != 0 && osg * S.odir < 0) {
            for (int c = 0; c < 4; ++c) {
                const double t = xv[S.olo][c];
                xv[S.olo][c] = xv[S.olo + 2][c];
                xv[S.olo + 2][c] = t;
            }
        }
        if (finite && S.olo >= 0 && osg == 0) {
            int64_t om[4][4];
            int oe[4][4];
            for (int k = 0; k < 4; ++k)
                for (int c = 0; c < 4; ++c) {
                    if constexpr (sizeof(Tin) == 4) tpx::decode_f32((float)xv[k][c], om[k][c], oe[k][c]);
                    else tpx::decode_f64(xv[k][c], om[k][c], oe[k][c]);
                }
            const int sg = tpx::order_sign(om, oe, span, S.olo, S.olo + 2);
            if (sg == 2) {
                order_unres = true;
            } else if (sg * S.odir < 0) {
                for (int c = 0; c < 4; ++c) {
                    const double t = xv[S.olo][c];
                    xv[S.olo][c] = xv[S.olo + 2][c];
                    xv[S.olo + 2][c] = t;
                }
            }
        }
        int bin = -1;
        int cls;
        if (order_unres) cls = (int)CLS_UNRESOLVED;
        else if (!finite) cls = (int)tpw::W_UNCERTAIN;
        else if (grouped) cls = decide_lanes(xv, tag, S, nax, eds, (int)(threadIdx.x & 48), bin);
        else cls = tpw::decide_dw(xv, tag, S.sigma, nax, S.kind, S.nbins, S.slots, eds, bin);
        if (grouped && (threadIdx.x & 15) != 0) continue;      // the group's first lane goes on
        if (cls == tpw::W_UNCERTAIN) {
            int64_t mant[4][4];
            int ex[4][4];
            for (int k = 0; k < 4; ++k)
                for (int c = 0; c < 4; ++c) {
                    if constexpr (sizeof(Tin) == 4) tpx::decode_f32((float)xv[k][c], mant[k][c], ex[k][c]);
                    else tpx::decode_f64(xv[k][c], mant[k][c], ex[k][c]);
                }
            cls = tpx::decide(mant, ex, finite, tag, span, S.sigma, nax, S.kind,
                              S.nbins, S.slots, eds, bin);
        }
        const bool unres = cls == CLS_UNRESOLVED;
        if (MODE == 1) {
            S.cls_out[i] = (int8_t)cls;
            if (S.ct_out) {
                const double est = S.ct_out[i];
                double mag = dabs(est);
                if (mag == 0.0 || !(mag < 1e308)) mag = 0x1p-1074;
                S.ct_out[i] = cls == CLS_ZERO ? 0.0
                            : (cls < 4 ? (((cls == CLS_I) || (cls == CLS_IV)) ? mag : -mag) : est);
            }
        }
        unsigned long long *st = (unsigned long long *)S.stats;
        if (cls == CLS_UNRESOLVED) {
            atomicAdd(st + ST_UNRESOLVED, 1ull);
        } else if (cls == CLS_ZERO) {
            atomicAdd(st + ST_ZERO, 1ull);
        } else if (cls == CLS_INVALID) {
            atomicAdd(st + ST_INVALID, 1ull);
        } else if (MODE == 0) {
            if (S.counts) {
                atomicAdd((unsigned long long *)S.counts + cls, 1ull);
                if (S.naxes > 0 && bin >= 0)
                    atomicAdd((unsigned long long *)S.counts + (1 + bin) * 4 + cls, 1ull);
            }
            if (S.naxes > 0 && bin < 0) atomicAdd(st + ST_OOR, 1ull);
        }
    }
    // the last workgroup to finish clears the list for the next launch
    __shared__ bool last;
    __syncthreads();
    if (threadIdx.x == 0) {
        __threadfence();
        const uint32_t t = atomicAdd(kp.xdone, 1u);
        last = (t == gridDim.x - 1);
    }
    __syncthreads();
    if (last && threadIdx.x == 0) {
        *kp.xcount = 0u;
        *kp.xdone = 0u;
        if (kp.mail) {
            const uint64_t u = __hip_atomic_load(kp.samples[0].stats + ST_UNRESOLVED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(kp.mail, u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        }
        __threadfence();
    }
}

}  // namespace

hipError_t launch_exact(int dtype, int mode, const KParams &kp, int grid, hipStream_t st)
{
    if (dtype == 0)
        return mode == 0 ? launch(tp_exact_kernel<float, 0>, grid, 64, 0, st, kp)
                         : launch(tp_exact_kernel<float, 1>, grid, 64, 0, st, kp);
    return mode == 0 ? launch(tp_exact_kernel<double, 0>, grid, 64, 0, st, kp)
                     : launch(tp_exact_kernel<double, 1>, grid, 64, 0, st, kp);
}

}  // namespace tpk
