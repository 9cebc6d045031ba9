// Register-resident window kernel for models with general B-dependency lists
// (VMP and MMP; lists of one or two factors).  Likelihood and states as in
// resident_kernel.h; the transitions are contracted the same way.
//
// B_j at the action of step t (log B_j for VMP) is a tensor over the next
// state i of factor j and the states of its list at t, and each of its
// leave-one-out contractions is a message: to i, the forward message to
// (t + 1, j), to a listed factor, the backward message from child j to (t, g).
// One lane therefore forms shares of all of them at once: its roles are an
// outer one (walked by the lane; absent for a list of one factor), an inner
// row and an inner column, 4 x 4 states of these at a time, read from the
// tables in LDS (one copy per action, shared by all steps).  Per (step, child)
// there are na x nb x parts lanes, the outer states divided among the parts.
// A sweep has four phases with a barrier after each: transition shares,
// transition messages (kept by the state's lane), likelihood shares, states.
// The two kinds of shares take turns in the same LDS, so their lines have no
// zero padding and are summed exactly.
//
// What bounds it: the four phases' latencies and vector instructions.  A step
// of three factors of 12, 10 and 8 states with lists of two takes 3008 table
// values, each converted and used in two products, against 960 of the
// likelihood.  4096 agents, 20 steps, MMP (2.7 ms): one workgroup of 8 waves to
// a compute unit, vector instructions in 47% of a SIMD's cycles, waves wait in
// 55% of theirs, LDS works in 34% of the cycles, 45% of these bank conflicts.
#pragma once

#include "resident_kernel.h"

namespace bi {
namespace res {

constexpr int kTA = 4, kTB = 4;   // states of the inner roles per lane
enum { kO, kA, kB, kTRoles };   // roles of a transition tensor: outer, inner row, inner column

struct Trans {
    int32_t n[kTRoles];       // states per role (outer absent: 1)
    int32_t na, nb, parts, per;   // blocks of kTA and kTB states, parts of the outer states, states per part
    int32_t lane0;            // first lane of the child in a step
    int32_t q[kTRoles];       // marginal offset of the role, from step t's marginals (0: absent, the constant 1)
    int32_t line[kTRoles], pitch[kTRoles];   // shares: offset of state 0 from step t's block of lines, distance
    int32_t tb, us, os, rs;   // table in LDS: first element, strides of action, outer state, row
    int32_t s[kTRoles], i;    // strides in the packed table [u][i][list], and of the action
    int64_t packed, agent;    // the packed table: byte offset, elements per agent
};

// Transition messages of a factor: its forward line and those from its children.
struct TFac {
    int32_t line, pitch, fwd, nch;        // a state's lines: first, distance; values of the forward one, children
    int32_t off[kMaxF], len[kMaxF];       // the children's lines behind it
};

struct CoupledArgs {
    Args a;
    int LP, steps, plt;        // lanes per step, steps side by side in the workgroup, line values per context
    int lds_tab;               // tables in LDS (else read from the packed buffer)
    int o_x, o_s;              // LDS: TFac table, the state lanes' transition messages (several states per lane)
    Trans tr[kMaxF];
    TFac tf[kMaxF];
};

// sum of n values without padding behind them
__device__ inline double exact_sum(const double *v, int n)
{
    double sum = 0.0;
    int k = 0;
    for (; k + 8 <= n; k += 8) {
        const Four f(v + k), g(v + k + 4);
        sum += f.sum() + g.sum();
    }
    if (k + 4 <= n) {
        sum += Four(v + k).sum();
        k += 4;
    }
    if (k < n) {   // 1 to 3 values: reads past them repeat the last one, left out
        const double x = v[k], y = v[min(k + 1, n - 1)], z = v[n - 1];
        double t = x;
        t = k + 1 < n ? t + y : t;
        sum += k + 2 < n ? t + z : t;
    }
    return sum;
}

// log(x) of a positive normal number: x = 2^e m, sqrt(1/2) <= m < sqrt(2),
// log m = 2 atanh(s), s = (m - 1) / (m + 1), by its series in s^2 <= 0.0295
// (the first term left out is below 1e-18 of the sum).
__device__ inline double log_of(double x)
{
    int e = __builtin_amdgcn_frexp_exp(x);
    double m = __builtin_amdgcn_frexp_mant(x);   // [1/2, 1)
    const bool low = m < 0.70710678118654752;
    m = low ? m + m : m;
    e -= low;
    const double s = (m - 1.0) * reciprocal(m + 1.0), z = s * s;
    double y = scalar(1.0 / 23.0);
    y = fma(y, z, scalar(1.0 / 21.0));
    y = fma(y, z, scalar(1.0 / 19.0));
    y = fma(y, z, scalar(1.0 / 17.0));
    y = fma(y, z, scalar(1.0 / 15.0));
    y = fma(y, z, scalar(1.0 / 13.0));
    y = fma(y, z, scalar(1.0 / 11.0));
    y = fma(y, z, scalar(1.0 / 9.0));
    y = fma(y, z, scalar(1.0 / 7.0));
    y = fma(y, z, scalar(1.0 / 5.0));
    y = fma(y, z, scalar(1.0 / 3.0));
    y = fma(y, z, 1.0);
    const double n = (double)e, t = s + s;
    return fma(n, scalar(0x1.62e42fefa0000p-1), fma(t, y, n * scalar(0x1.cf79abc9e3b3ap-40)));
}

// A lane's place in the transition phase: its tensor and blocks, fixed, and
// the first step it takes; offsets from step t's marginals and lines, two to
// a word.
struct Place {
    bool on;
    int t0, ju;              // first step; child | table elements per action << 8
    int qab, qoc;            // marginals of the inner roles; of the outer one | its states to walk
    int lab, lo;             // shares of the inner roles; of the outer one (-1: absent)
    int pab, po;             // between the shares of consecutive states: inner roles; outer role | row stride
    int x, os;               // table in LDS: first value at action 0, outer stride

    __device__ void here()   // (see Tile::here)
    {
        asm volatile("" : "+v"(ju), "+v"(qab), "+v"(qoc), "+v"(lab), "+v"(lo));
        asm volatile("" : "+v"(pab), "+v"(po), "+v"(x), "+v"(os));
    }
    __device__ int j() const { return ju & 0xff; }
};

__device__ inline Place place_of(const CoupledArgs &c)
{
    Place p;
    const int l = (int)threadIdx.x;
    p.t0 = l / c.LP;
    int rem = l - p.t0 * c.LP;
    p.on = p.t0 < c.steps;
    int j = 0;
    for (int k = 1; k < c.a.F; ++k)
        if (rem >= c.tr[k].lane0) j = k;
    const Trans &tr = c.tr[j];
    rem -= tr.lane0;
    const int parts = tr.parts, part = rem % parts;
    rem /= parts;
    const int bb = rem % tr.nb, ab = rem / tr.nb;
    const int a = kTA * ab, b = kTB * bb, o = part * tr.per;
    const int pa = tr.pitch[kA], pb = tr.pitch[kB], po = tr.pitch[kO];
    p.ju = j | tr.us << 8;
    p.qab = (tr.q[kA] + a) | (tr.q[kB] + b) << 16;
    p.qoc = (tr.q[kO] + o) | min(tr.per, tr.n[kO] - o) << 16;
    p.lab = (tr.line[kA] + a * pa + bb * parts + part) | (tr.line[kB] + b * pb + ab * parts + part) << 16;
    p.lo = tr.q[kO] ? tr.line[kO] + o * po + ab * tr.nb + bb : -1;
    p.pab = pa | pb << 16;
    p.po = po | tr.rs << 16;
    p.os = tr.os;
    p.x = tr.tb + o * tr.os + a * tr.rs + b;
    return p;
}

// The block of a table that lies in the packed buffer (states past the last
// one repeat it: their weights are 0).
template <class BT>
__device__ inline void read_packed(const CoupledArgs &c, int64_t am, int u, int j, int o, int a, int b, BT (&x)[kTA][kTB])
{
    const Trans &tr = c.tr[j];
    const BT *src = at<BT>(c.a.base, tr.packed) + am * tr.agent + (int64_t)u * tr.i + o * tr.s[kO];
#pragma unroll
    for (int i = 0; i < kTA; ++i)
#pragma unroll
        for (int k = 0; k < kTB; ++k)
            x[i][k] = src[min(a + i, tr.n[kA] - 1) * tr.s[kA] + min(b + k, tr.n[kB] - 1) * tr.s[kB]];
}

// Shares of the messages of B_j (action u) between steps t and t + 1.  LT:
// tables in LDS.
template <class BT, bool LT>
__device__ inline void contract_trans(const CoupledArgs &c, const Place &p, const BT *tab, int64_t am, double *smem,
                                      int cur, int t, int u)
{
    const Args &a = c.a;
    // (offsets into LDS, not pointers: these would become generic)
    const int q = cur + t * a.pq, lines = a.o_p + t * c.plt;
    double wa[kTA], wb[kTB], z[kTA], v[kTB];
#pragma unroll
    for (int i = 0; i < kTA; ++i) {
        wa[i] = smem[q + (p.qab & 0xffff) + i];
        z[i] = 0.0;
    }
#pragma unroll
    for (int k = 0; k < kTB; ++k) {
        wb[k] = smem[q + (p.qab >> 16) + k];
        v[k] = 0.0;
    }
    const int rs = p.po >> 16, po = p.po & 0xffff, count = p.qoc >> 16;
    int x = p.x + u * (p.ju >> 8), lo = lines + p.lo;
    const int qo = q + (p.qoc & 0xffff);
    for (int o = 0; o < count; ++o) {
        const double w = smem[qo + o];
        double y = 0.0;
        BT b[kTA][kTB];
        if constexpr (LT) {
#pragma unroll
            for (int i = 0; i < kTA; ++i) __builtin_memcpy(b[i], __builtin_assume_aligned(tab + x + i * rs, 16), sizeof(b[i]));
        } else {
            const Trans &tr = c.tr[p.j()];
            read_packed<BT>(c, am, u, p.j(), (p.qoc & 0xffff) - tr.q[kO] + o, (p.qab & 0xffff) - tr.q[kA],
                            (p.qab >> 16) - tr.q[kB], b);
        }
#pragma unroll
        for (int i = 0; i < kTA; ++i) {
            const double wo = wa[i] * w;
            double r = 0.0;
#pragma unroll
            for (int k = 0; k < kTB; ++k) {
                const double bk = b[i][k];
                r = fma(bk, wb[k], r);
                v[k] = fma(wo, bk, v[k]);
            }
            y = fma(wa[i], r, y);
            z[i] = fma(w, r, z[i]);
        }
        if (p.lo >= 0) smem[lo] = y;
        x += p.os;
        lo += po;
    }
    const int la = lines + (p.lab & 0xffff), lb = lines + (p.lab >> 16);
#pragma unroll
    for (int i = 0; i < kTA; ++i) smem[la + i * (p.pab & 0xffff)] = z[i];
#pragma unroll
    for (int k = 0; k < kTB; ++k) smem[lb + k * (p.pab >> 16)] = v[k];
}

// The agent's tables in LDS, inner rows and columns padded to whole blocks
// with zeros.
template <class BT>
__device__ inline void stage_trans(const CoupledArgs &c, int64_t am, int total, BT *tab)
{
    const Args &a = c.a;
    const int nt = (int)blockDim.x;
    for (int i = threadIdx.x; i < total; i += nt) tab[i] = BT(0);
    __syncthreads();
    for (int j = 0; j < a.F; ++j) {
        const Trans &tr = c.tr[j];
        const BT *src = at<BT>(a.base, tr.packed) + am * tr.agent;
        const int rows = tr.n[kO] * tr.n[kA], cnt = a.fac[j].U * rows * tr.n[kB];
        for (int e = threadIdx.x; e < cnt; e += nt) {
            int k = e;
            const int cb = k % tr.n[kB];
            k /= tr.n[kB];
            const int ra = k % tr.n[kA];
            k /= tr.n[kA];
            const int o = k % tr.n[kO], u = k / tr.n[kO];
            tab[tr.tb + u * tr.us + o * tr.os + ra * tr.rs + cb] =
                src[u * tr.i + o * tr.s[kO] + ra * tr.s[kA] + cb * tr.s[kB]];
        }
    }
}

// Transition messages of one state: VMP their sum (in *add), MMP their
// geometric mean over the messages present, as a weight (*mult) where it is a
// product or its square root, else as a logarithm (*add).
template <int ALGO>
__device__ inline void trans_messages(const CoupledArgs &c, const double *smem, const State &st, int f, double first,
                                      double *add, double *mult)
{
    const Args &a = c.a;
    const int *tf = reinterpret_cast<const int *>(smem + c.o_x) + f * (int)(sizeof(TFac) / 4);
    const double *line = smem + a.o_p + st.t() * c.plt + tf[0] + st.s() * tf[1];
    double sum = 0.0, prod = 1.0, logs = 0.0;
    int messages = 1, held = 0;   // (held: messages multiplied into prod)
    auto take = [&](double d) {
        if (ALGO == BI_ALGO_VMP) {
            sum += d;
        } else {
            if (held == 6) {   // (unnormalised tables: keep the product in range)
                logs += log_of(prod);
                prod = 1.0;
                held = 0;
            }
            prod *= fmax(d, kEps);
            ++held;
        }
    };
    if (st.prev())
        take(exact_sum(line, tf[2]));
    else if (a.prior && ALGO == BI_ALGO_MMP)
        take(first);
    if (st.next()) {
        const int nch = tf[3];
        messages += nch;
        for (int k = 0; k < nch; ++k) take(exact_sum(line + tf[4 + k], tf[4 + kMaxF + k]));
    }
    if (ALGO == BI_ALGO_VMP) {
        *add = st.prev() || a.prior ? sum : sum + first;
        *mult = !st.prev() && a.prior ? first : 1.0;
        return;
    }
    // the first step's log D takes the forward message's place in the mean
    const double ld = st.prev() || a.prior ? 0.0 : first, w = 1.0 / messages;
    if (messages <= 2) {
        *mult = messages == 2 ? root(prod) : prod;
        *add = messages == 2 ? 0.5 * ld : ld;
    } else {
        *mult = 1.0;
        *add = (ld + logs + log_of(prod)) * w;
    }
}

template <int ALGO, int RB, int CB, bool ONE, bool LT>
__global__ __launch_bounds__(max_threads(RB, CB, true)) void coupled_kernel(CoupledArgs c)
{
    using BT = std::conditional_t<ALGO == BI_ALGO_VMP, double, float>;
    extern __shared__ double smem[];
    const Args &a = c.a;
    const int agent = blockIdx.x, waves = (int)blockDim.x >> 6;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = (int)threadIdx.x & 63;
    const int64_t am = a.shared ? 0 : agent;
    stage_window<BT>(a, smem, agent, am, ALGO == BI_ALGO_VMP, waves);   // (a.tab is kGlobal: no tables yet)
    const int *acts = reinterpret_cast<const int *>(smem + a.o_a), *obs = acts + (a.T - 1) * a.F;
    int *tf = reinterpret_cast<int *>(smem + c.o_x);
    for (int i = threadIdx.x; i < (int)(a.F * sizeof(TFac) / 4); i += blockDim.x)
        tf[i] = reinterpret_cast<const int *>(c.tf)[i];
    BT *tab = reinterpret_cast<BT *>(smem + a.o_b);
    if (LT) stage_trans<BT>(c, am, a.btot, tab);
    Tile tl = tile_of<RB, CB>(a, a.T);
    Place pl = place_of(c);
    __syncthreads();
    double x[RB][CB];
    if (tl.on) load_mod<RB, CB>(a, tl, a.mod[a.grp[tl.g].m0], obs, agent, tl.c, x);
    const int units = a.units;
    State one{};
    double first_shift = __builtin_nan("");
    int2 *roles = reinterpret_cast<int2 *>(smem + a.o_r);
    for (int u = wave; u < units; u += waves) {
        const Where h = where_of(a, u, a.T);
        one = state_of(a, h, acts, a.T, am);
        one.fwd = factor_of(a, h.j);   // (in place of the transition row)
        if (!ONE) put_role(roles, u * 64 + lane, one);
        if (one.on()) smem[a.o_q + one.t() * a.pq + one.po() + one.s()] = 1.0 / one.states();   // uniform start
    }
    const int slots = wave * a.sv + (a.nchunk == 1 && lane < a.cpw * a.ntot ? lane / a.ntot * a.pq : 0);
    if (tl.on) add_mods<RB, CB>(a, tl, 1, obs, agent, tl.c, x);
    __syncthreads();
    int cur = a.o_q, nxt = a.o_q + a.T * a.pq;
    const int tq = tl.c * a.pq, tp = a.o_p + tl.c * a.pl;
    auto role = [&](int u, double &shift) {
        if (ONE) {
            shift = first_shift;
            return one;
        }
        return get_role(roles, u * 64 + lane, shift);
    };
    for (int k = 0; k < a.iters; ++k) {
        pl.here();
        if (pl.on)
            for (int t = pl.t0; t + 1 < a.T; t += c.steps)
                contract_trans<BT, LT>(c, pl, tab, am, smem, cur, t, acts[t * a.F + pl.j()]);
        __syncthreads();
        double add = 0.0, mult = 1.0;
        for (int u = wave; u < units; u += waves) {
            double shift;
            State st = role(u, shift);
            st.here();
            trans_messages<ALGO>(c, smem, st, st.fwd, smem[a.o_f + st.po() + st.s()], &add, &mult);
            if (!ONE) {
                smem[c.o_s + 2 * (u * 64 + lane)] = add;
                smem[c.o_s + 2 * (u * 64 + lane) + 1] = mult;
            }
        }
        __syncthreads();
        tl.here();
        if (tl.on) contract<RB, CB>(tl, x, smem, cur + tq, tp);
        __syncthreads();
        for (int u = wave; u < units; u += waves) {
            double shift;
            State st = role(u, shift);
            st.here();
            if (!ONE) {
                add = smem[c.o_s + 2 * (u * 64 + lane)];
                mult = smem[c.o_s + 2 * (u * 64 + lane) + 1];
            }
            const double lam = exact_sum(smem + a.o_p + st.t() * a.pl + st.line(), st.len());
            double qn = softmax(a, smem, st, slots, lam + add, mult, shift);
            if (ONE)
                first_shift = shift;
            else
                roles[3 * (u * 64 + lane) + 2].y = __float_as_int((float)shift);
            if (st.on()) {
                const int own = st.t() * a.pq + st.po() + st.s();
                if (a.tau != 1.0) qn = (1.0 - a.tau) * smem[cur + own] + a.tau * qn;
                if (k + 1 < a.iters) {
                    smem[nxt + own] = qn;
                } else {
                    const Where h = where_of(a, u, a.T);
                    a.q[((int64_t)agent * a.T + h.t) * a.ntot + h.j] = (float)qn;
                }
            }
        }
        __syncthreads();
        const int tmp = cur;
        cur = nxt;
        nxt = tmp;
    }
}

// The tile shapes this kernel is built for (indices into kShapes), with the
// tables in LDS and, the second list, in the packed buffer.  Times without a
// shape over those with it, as in resident_kernel.h: 1 x 1 1.10, 2 x 2 0.96 (at
// most 1.4), 4 x 2 1.07, 4 x 4 1.03 (at most 5.7), 6 x 4 1.01 (at most 1.1),
// 12 x 4 5.0, 12 x 5 1.5 (at most 7.3, where no other plan fits).
#define BI_RES_COUPLED(X) X(0, 1, 1) X(4, 2, 2) X(5, 4, 2) X(7, 4, 4) X(8, 6, 4) X(11, 12, 4) X(12, 12, 5)
#define BI_RES_COUPLED_PACKED(X) X(4, 2, 2) X(5, 4, 2) X(11, 12, 4)

template <int ALGO, int I, int R, int C, bool LT>
const void *coupled_passes(bool one)
{
    static_assert(kShapes[I].rb == R && kShapes[I].cb == C, "shape");
    return one ? (const void *)coupled_kernel<ALGO, R, C, true, LT> : (const void *)coupled_kernel<ALGO, R, C, false, LT>;
}

template <int ALGO>
const void *coupled_of(int shape, bool one, bool lds_tab)
{
    if (lds_tab) {
        switch (shape) {
#define BI_X(i, r, c) \
    case i: return coupled_passes<ALGO, i, r, c, true>(one);
            BI_RES_COUPLED(BI_X)
#undef BI_X
        }
    } else {
        switch (shape) {
#define BI_X(i, r, c) \
    case i: return coupled_passes<ALGO, i, r, c, false>(one);
            BI_RES_COUPLED_PACKED(BI_X)
#undef BI_X
        }
    }
    return nullptr;
}

// nullptr: not built for this shape.
const void *vmp_coupled(int shape, bool one, bool lds_tab);
const void *mmp_coupled(int shape, bool one, bool lds_tab);

}  // namespace res
}  // namespace bi
