// Register-resident agent kernels: device code shared by the instantiations
// (resident_fpi.hip, resident_vmp.hip, resident_mmp.hip).
//
// One workgroup per agent runs every iteration, like the kernels of
// agent.hip, but the likelihood is merged and kept in registers:
//
//  - Merging.  The likelihood message is linear in the slices, and a modality
//    whose dependency list is contained in another's adds a tensor that is
//    constant along the missing factors (their marginals sum to 1).  So the
//    observed slices of all modalities inside one maximal list are added
//    into one tensor per context and group, once per call (FPI: per step),
//    and every sweep contracts that one tensor (the paper's merging of
//    A-arrays, Sec. III-C, here of the observed slices).
//  - Registers.  The factors of a group take up to four roles: outer row a0,
//    inner row a1, outer column b0, inner column b1 (an absent role has one
//    state).  A lane holds RB x CB values, RB states of a1 by CB of b1, at one
//    state of a0 and b0; a sweep reads no slice from memory or LDS.
//
// A sweep has two phases with a barrier after each:
//  1. contraction: every lane contracts its tile with the marginals of a1 and
//     of b1, which gives its share of the messages to b1 and a1, and folds
//     those once more into its share of the messages to a0 and b0.  Every
//     share goes to LDS, to the line of the state it is for: a state's line
//     holds its shares from all lanes and groups side by side;
//  2. states: a lane per (step, state) adds its line, forms the transition
//     messages (B from LDS, the table and its transpose both stored by rows)
//     and takes the softmax over its factor, whose states lie in one wave,
//     through LDS.
// No logarithm is taken: softmax(lam + log p) has the weights exp(lam) p (the
// priors of FPI and of the first step), softmax(lam + (log f + log b) / 2) the
// weights exp(lam) sqrt(f b) (MMP).  p, f and b are clamped to 1e-16 as their
// logarithms would be, so the largest weight of a factor is at least 1e-16 and
// nothing that could reach an fp32 result underflows.  All arithmetic is fp64,
// in a fixed order.
//
// What bounds them: the latency of a sweep's two phases.  One agent's filter of
// 4 states (79 us for 128 sweeps) issues vector instructions in 27% of the
// cycles; 4096 agents of 12 x 10 x 8 states, 20 steps, MMP (1.12 ms; 6 x 4
// tiles, one workgroup of 13 waves to a compute unit) in 44%, with LDS at work in
// 27% and waves waiting in 61% of their cycles.  Its tiles spill: 116 bytes a
// lane, 0.4 GB a call.
#pragma once

#include <hip/hip_runtime.h>

#include "internal.h"
#include "transition.h"

namespace bi {
namespace res {

constexpr int kMaxG = 4;    // groups (maximal dependency lists)
constexpr int kMaxF = 8;    // factors
constexpr int kMaxM = 16;   // modalities
constexpr int kMaxN = 64;   // states of a factor (a softmax segment lies in one wave)
// A context's marginals: the constant 1 (the marginal of an absent role),
// then every factor's states followed by zeros.
constexpr int kFirst = 4;

// Threads a workgroup may have: tiles of more than 24 values need more than the
// 128 registers that 1024 threads leave each.
// (more: the filter, whose next step's slices are in flight too, and the
// kernel with a transition phase: of 8)
constexpr int max_threads(int rb, int cb, bool more) { return rb * cb >= (more ? 8 : 25) ? 512 : 1024; }

enum { kGlobal, kOnce, kBoth };

// Roles of a group's factors.
enum { kA0, kA1, kB0, kB1, kRoles };

struct Mod {
    int64_t la, la_agent, ll;   // byte offset of the slices, elements per agent, offset in the soft tensors
    int32_t slice, m;           // elements per outcome, modality index
    int32_t s[kRoles];          // element stride of every role's factor (0: not on the list)
};

struct Group {
    int32_t lane0, m0, m1;      // first lane of the group in a context; its modalities
    int32_t n[kRoles];          // states per role
    int32_t na, nb;             // lanes along a1 and b1 (blocks of RB and CB states)
    int32_t q[kRoles];          // marginal offset of the role (0: absent, the constant 1)
    int32_t line[kRoles];       // offset of state 0's shares in the context's lines (absent: the spare line)
    int32_t pitch[kRoles];      // between the lines of the role's states
};

struct Fac {
    int32_t n, U, qo, po;       // states, actions, offset in a marginal vector: packed, padded
    int32_t line, pitch, len;   // the states' lines in a context: first, distance, values
    int32_t bt, bs;             // transition table: first element and row stride (see Args::tab)
    int64_t b, lb, ld, b_agent, ld_agent;
};

struct Args {
    const char *base;
    int F, G, M, shared, T, iters, ntot;
    int pq, pl, LT;             // per context: marginals, line values, lanes
    int nchunk, cpw, sv;        // state lanes: chunks of factors per context, contexts per wave, slots per wave
    int units;                  // passes of one wave over the window's states
    int chunk0[kMaxF + 1];      // first state of every chunk
    // Transition tables: kBoth: in LDS twice, the table and btot elements behind
    // its transpose, rows padded with zeros; kOnce: in LDS, rows padded; kGlobal: read
    // from the packed buffer, fac.bt counting elements from its start.
    int tab, btot;
    // LDS offsets in doubles: marginals, lines, softmax slots, transition tables, actions, first-step terms, roles
    int o_q, o_p, o_e, o_b, o_a, o_f, o_r;
    const int32_t *obs;
    const double *ll;
    int64_t llpc;
    const int32_t *act;
    const float *prior;
    double tau;
    float *q;
    Group grp[kMaxG];
    Mod mod[kMaxM];
    Fac fac[kMaxF];
};

template <class T>
__device__ inline const T *at(const char *base, int64_t byte_off)
{
    return reinterpret_cast<const T *>(base + byte_off);
}

// Reads and writes of one wave through LDS: the hardware keeps a wave's LDS
// operations in order, so only the compiler has to be held.
__device__ inline void wave_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// ---------------------------------------------------------------------------
// contraction
// ---------------------------------------------------------------------------
// A lane's tile: its place, and packed into a few words what every sweep
// needs of it.
struct Tile {
    bool on;
    int c, g;                // context of the window, group
    int a0, a1, b0, b1;      // states: of the outer roles, first of the inner ones
    int qa, qb;              // marginal offsets: outer | inner << 16
    int wa, wb;              // line offsets of its shares: outer | inner << 16
    int pitch;               // between the lines of a1's | b1's states << 16

    // Keeps what is derived from the words out of the registers between
    // sweeps: without it every unpacked offset and address of a sweep is
    // hoisted out of the loop (60 registers and more, spilled).
    __device__ void here()
    {
        asm volatile("" : "+v"(qa), "+v"(qb), "+v"(wa), "+v"(wb), "+v"(pitch));
    }
};

template <int RB, int CB>
__device__ inline Tile tile_of(const Args &a, int contexts)
{
    Tile t;
    const int l = (int)threadIdx.x;
    t.c = l / a.LT;
    int rem = l - t.c * a.LT;
    t.on = t.c < contexts;
    t.g = 0;
    for (int g = 1; g < a.G; ++g)
        if (rem >= a.grp[g].lane0) t.g = g;
    const Group &g = a.grp[t.g];
    rem -= g.lane0;
    // lanes of a line's shares side by side: b1 blocks fastest, then b0, a1 blocks, a0
    const int nb = g.nb, nb0 = g.n[kB0], na = g.na;
    const int bb = rem % nb;
    rem /= nb;
    t.b0 = rem % nb0;
    rem /= nb0;
    const int ab = rem % na;
    t.a0 = rem / na;
    t.a1 = ab * RB;
    t.b1 = bb * CB;
    // (the coordinate of an absent role is 0)
    t.qa = (g.q[kA0] + t.a0) | (g.q[kA1] + t.a1) << 16;
    t.qb = (g.q[kB0] + t.b0) | (g.q[kB1] + t.b1) << 16;
    // a share's place in its state's line: the lane's number without that role
    const int la1 = (t.a0 * nb0 + t.b0) * nb + bb, lb1 = (t.a0 * na + ab) * nb0 + t.b0;
    const int la0 = (ab * nb0 + t.b0) * nb + bb, lb0 = (t.a0 * na + ab) * nb + bb;
    t.wa = (g.line[kA0] + t.a0 * g.pitch[kA0] + (g.q[kA0] ? la0 : 0)) |
           (g.line[kA1] + t.a1 * g.pitch[kA1] + (g.q[kA1] ? la1 : 0)) << 16;
    t.wb = (g.line[kB0] + t.b0 * g.pitch[kB0] + (g.q[kB0] ? lb0 : 0)) |
           (g.line[kB1] + t.b1 * g.pitch[kB1] + lb1) << 16;
    t.pitch = g.pitch[kA1] | g.pitch[kB1] << 16;
    return t;
}

// Values of one modality's observed slice under a lane's tile (step t).  obs:
// the agent's outcomes [T][M] (LDS).  Reads past the states of a1 and b1
// repeat the last one; a modality that depends on neither, or on one of the
// two only, reads the same few values for every row or column.
template <int RB, int CB>
__device__ inline void load_mod(const Args &a, const Tile &tl, const Mod &md, const int *obs, int agent, int t,
                                double (&y)[RB][CB])
{
    const Group &g = a.grp[tl.g];
    const int ia = g.n[kA1] - 1 - tl.a1, jb = g.n[kB1] - 1 - tl.b1;   // last row and column inside
    // one base for the agent, 32-bit offsets (checked by the plan)
    const char *X = a.ll ? reinterpret_cast<const char *>(a.ll + (int64_t)agent * a.T * a.llpc + md.ll)
                         : a.base + md.la + (a.shared ? 0 : (int64_t)agent * md.la_agent * 8);
    const int sa = md.s[kA1], sb = md.s[kB1];
    const uint32_t at0 = (a.ll ? (uint32_t)t * (uint32_t)a.llpc : (uint32_t)obs[t * a.M + md.m] * (uint32_t)md.slice) +
                         (uint32_t)(tl.a0 * md.s[kA0] + tl.a1 * sa + tl.b0 * md.s[kB0] + tl.b1 * sb);
    auto load = [&](int o) { return *reinterpret_cast<const double *>(X + ((at0 + (uint32_t)o) << 3)); };
    if (sa == 0) {
        double v[CB];
#pragma unroll
        for (int j = 0; j < CB; ++j) v[j] = load(min(j, jb) * sb);
#pragma unroll
        for (int i = 0; i < RB; ++i)
#pragma unroll
            for (int j = 0; j < CB; ++j) y[i][j] = v[j];
    } else if (sb == 0) {
        double v[RB];
#pragma unroll
        for (int i = 0; i < RB; ++i) v[i] = load(min(i, ia) * sa);
#pragma unroll
        for (int i = 0; i < RB; ++i)
#pragma unroll
            for (int j = 0; j < CB; ++j) y[i][j] = v[i];
    } else {
#pragma unroll
        for (int i = 0; i < RB; ++i)
#pragma unroll
            for (int j = 0; j < CB; ++j) y[i][j] = load(min(i, ia) * sa + min(j, jb) * sb);
    }
}

// Adds the group's modalities from number k0 on to the tile, and clears what
// lies past the states of a1 and b1.  A few rows are in flight at a time.
template <int RB, int CB>
__device__ inline void add_mods(const Args &a, const Tile &tl, int k0, const int *obs, int agent, int t,
                                double (&x)[RB][CB])
{
    constexpr int kRows = RB * CB <= 8 ? RB : CB >= 4 ? 2 : CB >= 2 ? 4 : 8;
    const Group &g = a.grp[tl.g];
    for (int k = g.m0 + k0; k < g.m1; ++k) {
        const Mod md = a.mod[k];
#pragma unroll
        for (int i0 = 0; i0 < RB; i0 += kRows) {
            Tile part = tl;
            part.a1 = min(tl.a1 + i0, g.n[kA1] - 1);
            double y[kRows][CB];
            load_mod<kRows, CB>(a, part, md, obs, agent, t, y);
#pragma unroll
            for (int i = 0; i < kRows; ++i)
                if (i0 + i < RB)
#pragma unroll
                    for (int j = 0; j < CB; ++j) x[i0 + i][j] += y[i][j];
        }
    }
    const int ia = g.n[kA1] - 1 - tl.a1, jb = g.n[kB1] - 1 - tl.b1;
#pragma unroll
    for (int i = 0; i < RB; ++i)
#pragma unroll
        for (int j = 0; j < CB; ++j)
            if (i > ia || j > jb) x[i][j] = 0.0;
}

// Phase 1 of a sweep: q, p: LDS offsets of the context's marginals and lines.
template <int RB, int CB>
__device__ inline void contract(const Tile &tl, const double (&x)[RB][CB], double *smem, int q, int p)
{
    const double *qa = smem + q + (tl.qa >> 16), *qb = smem + q + (tl.qb >> 16);
    const double oa = smem[q + (tl.qa & 0xffff)], ob = smem[q + (tl.qb & 0xffff)];
    double wb[CB], v[CB];
#pragma unroll
    for (int j = 0; j < CB; ++j) {
        wb[j] = qb[j];
        v[j] = 0.0;
    }
    const double o = oa * ob;
    double *za = smem + p + (tl.wa >> 16), *vb = smem + p + (tl.wb >> 16);
    const int pa = tl.pitch & 0xffff, pb = tl.pitch >> 16;
    double y = 0.0;
#pragma unroll
    for (int i = 0; i < RB; ++i) {
        const double wa = qa[i];
        double z = x[i][0] * wb[0];
        v[0] = fma(wa, x[i][0], v[0]);
#pragma unroll
        for (int j = 1; j < CB; ++j) {
            z = fma(x[i][j], wb[j], z);
            v[j] = fma(wa, x[i][j], v[j]);
        }
        y = fma(wa, z, y);
        za[i * pa] = z * o;
    }
#pragma unroll
    for (int j = 0; j < CB; ++j) vb[j * pb] = v[j] * o;
    smem[p + (tl.wa & 0xffff)] = y * ob;
    smem[p + (tl.wb & 0xffff)] = y * oa;
}

// ---------------------------------------------------------------------------
// states
// ---------------------------------------------------------------------------
// Loops over n values, padded to whole groups of 4 with zeros: two groups at a
// time, then one.
struct Four {
    double2 p, r;
    __device__ Four(const double *v)
        : p(reinterpret_cast<const double2 *>(v)[0]), r(reinterpret_cast<const double2 *>(v)[1])
    {
    }
    __device__ double sum() const { return (p.x + p.y) + (r.x + r.y); }
};

// (maximum: what lies past the end is repeated, not read)
__device__ inline double line_max(const double *v, int n)
{
    double mx = -INFINITY;
    for (int k = 0; k < n; k += 4) {
        const int l = n - 1;
        const double x = v[k], y = v[min(k + 1, l)], z = v[min(k + 2, l)], w = v[min(k + 3, l)];
        mx = fmax(fmax(mx, fmax(x, y)), fmax(z, w));
    }
    return mx;
}

__device__ inline double line_sum(const double *v, int n)
{
    double sum = 0.0;
    int k = 0;
    for (; k + 4 < n; k += 8) {
        const Four f(v + k), g(v + k + 4);
        sum += f.sum() + g.sum();
    }
    if (k < n) sum += Four(v + k).sum();
    return sum;
}

// Dot product of a padded transition row and a padded marginal vector.
template <class BT>
struct Row4 {
    BT b[4];
    __device__ Row4(const BT *row) { __builtin_memcpy(b, __builtin_assume_aligned(row, 16), sizeof(b)); }
    __device__ double dot(const Four &q, double acc) const
    {
        acc = fma((double)b[0], q.p.x, acc);
        acc = fma((double)b[1], q.p.y, acc);
        acc = fma((double)b[2], q.r.x, acc);
        return fma((double)b[3], q.r.y, acc);
    }
};

template <class BT>
__device__ inline double row_dot(const BT *row, const double *q, int n)
{
    double acc = 0.0;
    int k = 0;
    for (; k + 4 < n; k += 8) {
        const Row4<BT> r0(row + k), r1(row + k + 4);
        const Four q0(q + k), q1(q + k + 4);
        acc = r1.dot(q1, r0.dot(q0, acc));
    }
    if (k < n) {
        const Row4<BT> r0(row + k);
        acc = r0.dot(Four(q + k), acc);
    }
    return acc;
}

// sum_{k < n} load(k) q[k], 8 reads in flight at a time (rows and columns that
// are not padded).
template <class Load>
__device__ inline double plain_dot(Load load, const double *q, int n)
{
    double acc = 0.0;
    int k = 0;
    for (; k + 8 <= n; k += 8) {
        double b[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) b[i] = (double)load(k + i);
#pragma unroll
        for (int i = 0; i < 8; ++i) acc = fma(b[i], q[k + i], acc);
    }
    if (k + 4 <= n) {
        double b[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) b[i] = (double)load(k + i);
#pragma unroll
        for (int i = 0; i < 4; ++i) acc = fma(b[i], q[k + i], acc);
        k += 4;
    }
    for (; k < n; ++k) acc = fma((double)load(k), q[k], acc);
    return acc;
}

// The transition products of a state: its row of the table before the step
// with the marginals before, its column of the table after with those after.
template <class BT>
__device__ inline double forward(const Args &a, const BT *tab, int at_row, const double *q, int n)
{
    if (a.tab != kGlobal) return row_dot(tab + at_row, q, n);
    return plain_dot([&](int k) { return *reinterpret_cast<const BT *>(a.base + (uint32_t)(at_row + k) * (uint32_t)sizeof(BT)); }, q, n);
}

template <class BT>
__device__ inline double backward(const Args &a, const BT *tab, int at_col, int bs, const double *q, int n)
{
    if (a.tab == kBoth) return row_dot(tab + at_col, q, n);
    if (a.tab == kOnce) return plain_dot([&](int k) { return tab[at_col + k * bs]; }, q, n);
    return plain_dot([&](int k) { return *reinterpret_cast<const BT *>(a.base + (uint32_t)(at_col + k * n) * (uint32_t)sizeof(BT)); }, q, n);
}

// A constant in scalar registers at the place of its use: hoisted out of the
// sweeps, the constants of the functions below would take the vector
// registers that the tiles need.
__device__ inline double scalar(double c)
{
    asm volatile("" : "+s"(c));
    return c;
}

// exp(x) (NaN stays NaN, +inf gives NaN): 2^n exp(r), n = x / ln 2 rounded,
// |r| <= ln 2 / 2, exp(r) by its Taylor series (the first term left out,
// r^14 / 14!, is below 5e-18).  ln 2 is split so that n times its high part
// is exact.
__device__ inline double exp_of(double x)
{
    x = x < -800.0 ? -800.0 : x;   // (exp is 0; also for -inf)
    const double n = __builtin_rint(x * scalar(1.4426950408889634));
    double r = fma(n, scalar(-0x1.62e42fefa0000p-1), x);
    r = fma(n, scalar(-0x1.cf79abc9e3b3ap-40), r);
    double y = scalar(1.0 / 6227020800.0);
    y = fma(y, r, scalar(1.0 / 479001600.0));
    y = fma(y, r, scalar(1.0 / 39916800.0));
    y = fma(y, r, scalar(1.0 / 3628800.0));
    y = fma(y, r, scalar(1.0 / 362880.0));
    y = fma(y, r, scalar(1.0 / 40320.0));
    y = fma(y, r, scalar(1.0 / 5040.0));
    y = fma(y, r, scalar(1.0 / 720.0));
    y = fma(y, r, scalar(1.0 / 120.0));
    y = fma(y, r, scalar(1.0 / 24.0));
    y = fma(y, r, scalar(1.0 / 6.0));
    y = fma(y, r, 0.5);
    y = fma(y, r, 1.0);
    y = fma(y, r, 1.0);
    return __builtin_ldexp(y, (int)n);
}

// sqrt(x) of a positive normal number: Goldschmidt's iteration from the
// hardware's reciprocal square root, corrected by the residual.
__device__ inline double root(double x)
{
    const double y = __builtin_amdgcn_rsq(x);
    double g = x * y, h = 0.5 * y;
    double r = fma(-h, g, 0.5);
    g = fma(g, r, g);
    h = fma(h, r, h);
    r = fma(-g, g, x);
    g = fma(r, h, g);
    r = fma(-g, g, x);
    return fma(r, h, g);
}

// 1 / x of a normal number: the hardware's reciprocal refined twice.
__device__ inline double reciprocal(double x)
{
    double r = __builtin_amdgcn_rcp(x);
    r = fma(fma(-x, r, 1.0), r, r);
    return fma(fma(-x, r, 1.0), r, r);
}

// A lane's role in the state phase, packed (the window kernel keeps those of
// all its states in LDS when a lane has several).
struct State {
    int js;         // marginal offset of the factor | state << 15 | row stride of its table << 21
    int info;       // states | kOn, kPrev, kNext | values of its line << 16
    int tp;         // offset of its line in the context's lines | step << 16
    int fwd, bwd;   // transition row and column (kBoth: row of the transpose)

    static constexpr int kOn = 1 << 8, kPrev = 1 << 9, kNext = 1 << 10;
    __device__ void here()   // (see Tile::here)
    {
        asm volatile("" : "+v"(js), "+v"(info), "+v"(tp), "+v"(fwd), "+v"(bwd));
    }
    __device__ bool on() const { return info & kOn; }
    __device__ bool prev() const { return info & kPrev; }
    __device__ bool next() const { return info & kNext; }
    __device__ int states() const { return info & 0xff; }
    __device__ int len() const { return info >> 16; }
    __device__ int po() const { return js & 0x7fff; }
    __device__ int s() const { return js >> 15 & 0x3f; }
    __device__ int bs() const { return js >> 21; }
    __device__ int t() const { return tp >> 16; }
    __device__ int line() const { return tp & 0xffff; }
};

// Which state of the window a lane of unit `unit` has: step, state of the
// packed marginal vector.
struct Where {
    bool on;
    int t, j;
};

__device__ inline Where where_of(const Args &a, int unit, int contexts)
{
    Where r;
    const int lane = (int)threadIdx.x & 63;
    if (a.nchunk == 1) {
        const int c = lane / a.ntot;
        r.t = unit * a.cpw + c;
        r.j = lane - c * a.ntot;
        r.on = c < a.cpw && r.t < contexts;
    } else {
        r.t = unit / a.nchunk;
        const int ch = unit - r.t * a.nchunk;
        r.j = a.chunk0[ch] + lane;
        r.on = r.t < contexts && r.j < a.chunk0[ch + 1];
    }
    if (!r.on) r.t = r.j = 0;
    return r;
}

// The factor of state j of the packed vector.
__device__ inline int factor_of(const Args &a, int j)
{
    int f = 0;
    for (int k = 1; k < a.F; ++k) f = j >= a.fac[k].qo ? k : f;
    return f;
}

// act: the agent's actions [T-1][F] (LDS), not read for a window of one step
__device__ inline State state_of(const Args &a, const Where &h, const int *act, int contexts, int64_t am)
{
    // (selected factor by factor: indexed by the lane, the descriptors would
    // be loaded through vector memory)
    int f = 0, n = a.fac[0].n, qo = 0, po = a.fac[0].po, line = a.fac[0].line, pitch = a.fac[0].pitch;
    int len = a.fac[0].len, bt = a.fac[0].bt, bs = a.fac[0].bs, own = (int)(am * a.fac[0].b_agent);
    for (int k = 1; k < a.F; ++k) {
        const Fac &fd = a.fac[k];
        const bool in = h.j >= fd.qo;
        f = in ? k : f;
        n = in ? fd.n : n;
        qo = in ? fd.qo : qo;
        po = in ? fd.po : po;
        line = in ? fd.line : line;
        pitch = in ? fd.pitch : pitch;
        len = in ? fd.len : len;
        bt = in ? fd.bt : bt;
        bs = in ? fd.bs : bs;
        own = in ? (int)(am * fd.b_agent) : own;
    }
    State st;
    const int s = h.j - qo;
    const bool prev = h.t > 0, next = h.t + 1 < contexts;
    st.js = po | s << 15 | bs << 21;
    st.info = n | (h.on ? State::kOn : 0) | (prev ? State::kPrev : 0) | (next ? State::kNext : 0) | len << 16;
    st.tp = (line + s * pitch) | h.t << 16;
    const int up = prev ? act[(h.t - 1) * a.F + f] : 0, un = next ? act[h.t * a.F + f] : 0;
    if (a.tab == kGlobal) bt += own;
    st.fwd = bt + (up * n + s) * bs;
    st.bwd = a.tab == kBoth ? a.btot + bt + (un * n + s) * bs : bt + un * n * bs + s;
    return st;
}

// Softmax over the lane's factor: e = exp(v - shift) mult over the sum of e.
// base: the lane's context in the softmax slots.  shift (the same for every
// state of a factor): the maximum of v in an earlier sweep is as good as this
// sweep's while the sum stays far from overflow and underflow (what is lost
// below it is 1e-200 of the sum); else, and first of all (shift NaN), the
// maximum is taken.
__device__ inline double softmax(const Args &a, double *smem, const State &st, int base, double v, double mult,
                                 double &shift)
{
    const int seg = base + st.po(), n = st.states();
    double *eb = smem + a.o_e + seg;
    double e = exp_of(v - shift) * mult;
    if (st.on()) eb[st.s()] = e;
    wave_fence();
    double sum = line_sum(eb, n);
    wave_fence();
    if (__builtin_amdgcn_ballot_w64(!(sum > 1e-100 && sum < 1e100) && st.on())) {
        if (st.on()) eb[st.s()] = v;
        wave_fence();
        shift = line_max(eb, n);
        wave_fence();
        e = exp_of(v - shift) * mult;
        if (st.on()) eb[st.s()] = e;
        wave_fence();
        sum = line_sum(eb, n);
        wave_fence();
    }
    return e * reciprocal(sum);
}

// LDS start: marginals 0 behind the constant 1 (the padding stays 0; uniform
// values are written over the states), lines 0, softmax slots.
__device__ inline void init_lds(const Args &a, double *smem, int vectors, int waves)
{
    const int nt = (int)blockDim.x;
    for (int i = threadIdx.x; i < vectors * a.pq; i += nt) smem[a.o_q + i] = i % a.pq == 0 ? 1.0 : 0.0;
    for (int i = a.o_p + (int)threadIdx.x; i < a.o_e + waves * a.sv; i += nt) smem[i] = 0.0;   // (o_e follows o_p)
}

// Transition tables of the agent in LDS (Args::tab).
template <class BT>
__device__ inline void stage_tables(const Args &a, int64_t am, bool lb, BT *tab)
{
    const int nt = (int)blockDim.x;
    const bool both = a.tab == kBoth;
    for (int i = threadIdx.x; i < (both ? 2 : 1) * a.btot; i += nt) tab[i] = BT(0);
    __syncthreads();
    for (int f = 0; f < a.F; ++f) {
        const Fac &fd = a.fac[f];
        const BT *src = at<BT>(a.base, lb ? fd.lb : fd.b) + am * fd.b_agent;
        const int nn = fd.n * fd.n, cnt = fd.U * nn;
        for (int i = threadIdx.x; i < cnt; i += nt) {
            const int u = i / nn, ij = i - u * nn, r = ij / fd.n, c = ij - r * fd.n;
            const BT v = src[i];
            tab[fd.bt + (u * fd.n + r) * fd.bs + c] = v;
            if (both) tab[a.btot + fd.bt + (u * fd.n + c) * fd.bs + r] = v;
        }
    }
}

// Outcomes, actions, transition tables and first-step terms in LDS.  First
// step: log D is added to the message, the caller's prior (clamped) multiplies
// the weight.
template <class BT>
__device__ inline void stage_window(const Args &a, double *smem, int agent, int64_t am, bool lb, int waves)
{
    int *acts = reinterpret_cast<int *>(smem + a.o_a), *obs = acts + (a.T - 1) * a.F;
    if (!a.ll)
        for (int i = threadIdx.x; i < a.T * a.M; i += blockDim.x) obs[i] = a.obs[(int64_t)agent * a.T * a.M + i];
    for (int i = threadIdx.x; i < (a.T - 1) * a.F; i += blockDim.x)
        acts[i] = a.act[(int64_t)agent * (a.T - 1) * a.F + i];
    init_lds(a, smem, 2 * a.T, waves);
    if (a.T > 1 && a.tab != kGlobal) stage_tables<BT>(a, am, lb, reinterpret_cast<BT *>(smem + a.o_b));
    for (int f = 0; f < a.F; ++f)
        for (int s = threadIdx.x; s < a.fac[f].n; s += blockDim.x)
            smem[a.o_f + a.fac[f].po + s] =
                a.prior ? fmax((double)a.prior[(int64_t)agent * a.ntot + a.fac[f].qo + s], kEps)
                        : at<double>(a.base, a.fac[f].ld)[am * a.fac[f].ld_agent + s];
}

// A lane's roles in LDS: 5 words of State and the softmax shift (fp32: any
// value near the maximum serves, as long as a factor's states share it).
__device__ inline void put_role(int2 *roles, int i, const State &st)
{
    int2 *r = roles + 3 * i;
    r[0] = make_int2(st.js, st.info);
    r[1] = make_int2(st.tp, st.fwd);
    r[2] = make_int2(st.bwd, __float_as_int(__builtin_nanf("")));
}

__device__ inline State get_role(const int2 *roles, int i, double &shift)
{
    const int2 *r = roles + 3 * i;
    const int2 r0 = r[0], r1 = r[1], r2 = r[2];
    shift = __int_as_float(r2.y);
    return State{r0.x, r0.y, r1.x, r1.y, r2.x};
}

// The new marginal of a state, lam its likelihood message: transition messages
// from the neighbouring steps, softmax.  Written to the other buffer, or in
// the last sweep to the output.
template <int ALGO, class BT>
__device__ inline void update_state(const Args &a, double *smem, const BT *tab, const State &st, int agent, int unit,
                                    int slots, int cur, int nxt, bool last, double lam, double &shift)
{
    double v = lam, mult = 1.0;
    const int own = st.t() * a.pq + st.po();
    const double *q = smem + cur + own;
    const int n = st.states();
    double fwd = 1.0, bwd = 1.0;   // MMP
    if (st.prev()) {
        const double d = forward<BT>(a, tab, st.fwd, q - a.pq, n);
        if (ALGO == BI_ALGO_VMP)
            v += d;
        else
            fwd = fmax(d, kEps);
    } else {
        const double d = smem[a.o_f + st.po() + st.s()];
        if (a.prior)
            (ALGO == BI_ALGO_VMP ? mult : fwd) = d;
        else
            v += ALGO == BI_ALGO_MMP && st.next() ? 0.5 * d : d;
    }
    if (st.next()) {
        const double d = backward<BT>(a, tab, st.bwd, st.bs(), q + a.pq, n);
        if (ALGO == BI_ALGO_VMP)
            v += d;
        else
            bwd = fmax(d, kEps);
    }
    if (ALGO == BI_ALGO_MMP) mult = st.next() ? root(fwd * bwd) : fwd;
    double qn = softmax(a, smem, st, slots, v, mult, shift);
    if (st.on()) {
        if (a.tau != 1.0) qn = (1.0 - a.tau) * q[st.s()] + a.tau * qn;
        if (!last) {
            smem[nxt + own + st.s()] = qn;
        } else {
            const Where h = where_of(a, unit, a.T);
            a.q[((int64_t)agent * a.T + h.t) * a.ntot + h.j] = (float)qn;
        }
    }
}

// VMP and MMP.  ONE: every state has a lane (one pass of the state phase);
// otherwise a lane's roles are kept in LDS.
template <int ALGO, int RB, int CB, bool ONE>
__global__ __launch_bounds__(max_threads(RB, CB, false)) void window_kernel(Args a)
{
    using BT = std::conditional_t<ALGO == BI_ALGO_VMP, double, float>;
    extern __shared__ double smem[];
    const int agent = blockIdx.x, waves = (int)blockDim.x >> 6;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = (int)threadIdx.x & 63;
    const int64_t am = a.shared ? 0 : agent;
    // outcomes, actions and transition tables first, then, while the tiles'
    // loads are in flight, the roles of the state phase
    stage_window<BT>(a, smem, agent, am, ALGO == BI_ALGO_VMP, waves);
    const BT *tab = reinterpret_cast<const BT *>(smem + a.o_b);
    const int *acts = reinterpret_cast<const int *>(smem + a.o_a), *obs = acts + (a.T - 1) * a.F;
    Tile tl = tile_of<RB, CB>(a, a.T);
    __syncthreads();
    double x[RB][CB];
    if (tl.on) load_mod<RB, CB>(a, tl, a.mod[a.grp[tl.g].m0], obs, agent, tl.c, x);
    const int units = a.units;
    State one{};
    double first_shift = __builtin_nan("");
    int2 *roles = reinterpret_cast<int2 *>(smem + a.o_r);
    for (int u = wave; u < units; u += waves) {
        one = state_of(a, where_of(a, u, a.T), acts, a.T, am);
        if (!ONE) put_role(roles, u * 64 + lane, one);
        if (one.on()) smem[a.o_q + one.t() * a.pq + one.po() + one.s()] = 1.0 / one.states();   // uniform start
    }
    const int slots = wave * a.sv + (a.nchunk == 1 && lane < a.cpw * a.ntot ? lane / a.ntot * a.pq : 0);
    if (tl.on) add_mods<RB, CB>(a, tl, 1, obs, agent, tl.c, x);
    __syncthreads();
    int cur = a.o_q, nxt = a.o_q + a.T * a.pq;
    const int tq = tl.c * a.pq, tp = a.o_p + tl.c * a.pl;
    for (int k = 0; k < a.iters; ++k) {
        tl.here();
        if (tl.on) contract<RB, CB>(tl, x, smem, cur + tq, tp);
        __syncthreads();
        for (int u = wave; u < units; u += waves) {
            State st = one;
            double shift = first_shift;
            if (!ONE) st = get_role(roles, u * 64 + lane, shift);
            st.here();
            const double lam = line_sum(smem + a.o_p + st.t() * a.pl + st.line(), st.len());
            update_state<ALGO, BT>(a, smem, tab, st, agent, u, slots, cur, nxt, k + 1 == a.iters, lam, shift);
            if (ONE)
                first_shift = shift;
            else
                roles[3 * (u * 64 + lane) + 2].y = __float_as_int((float)shift);
        }
        __syncthreads();
        const int tmp = cur;
        cur = nxt;
        nxt = tmp;
    }
}

// FPI: one step at a time, its merged tensor in registers for all its
// iterations.  A wave per chunk of factors in the state phase.  TB: every
// B-dependency list is {f}.
template <int RB, int CB, bool TB>
__global__ __launch_bounds__(max_threads(RB, CB, true)) void filter_kernel(Args a)
{
    extern __shared__ double smem[];
    const int agent = blockIdx.x, waves = (int)blockDim.x >> 6;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int64_t am = a.shared ? 0 : agent;
    int *acts = reinterpret_cast<int *>(smem + a.o_a), *obs = acts + (a.T - 1) * a.F;
    if (!a.ll)
        for (int i = threadIdx.x; i < a.T * a.M; i += blockDim.x) obs[i] = a.obs[(int64_t)agent * a.T * a.M + i];
    for (int i = threadIdx.x; i < (a.T - 1) * a.F; i += blockDim.x)
        acts[i] = a.act[(int64_t)agent * (a.T - 1) * a.F + i];
    init_lds(a, smem, 2, waves);
    Tile tl = tile_of<RB, CB>(a, 1);
    const bool states = wave < a.nchunk;
    const Where h = where_of(a, wave, 1);
    State st = state_of(a, h, nullptr, 1, 0);
    const int f = factor_of(a, h.j);
    const int slots = wave * a.sv, own = st.po() + st.s();
    // this lane's row of B at action 0, its first-step term
    int64_t row0 = 0, frow = 0;
    double lp = 0.0, mult = 1.0;
    for (int k = 0; k < a.F; ++k)
        if (k == f) {
            const Fac &fd = a.fac[k];
            row0 = fd.b + 4 * (am * fd.b_agent + (int64_t)st.s() * fd.n);
            frow = 4 * (int64_t)fd.n * fd.n;
            if (a.prior)
                mult = fmax((double)a.prior[(int64_t)agent * a.ntot + h.j], kEps);
            else
                lp = at<double>(a.base, fd.ld)[am * fd.ld_agent + st.s()];
        }
    __syncthreads();
    // the next step's slices are fetched while a step is iterated: the first
    // kPre modalities of a group, where the tile leaves registers for them
    constexpr int kPre = RB * CB <= 4 ? 3 : RB * CB <= 8 ? 2 : RB * CB <= 16 ? 1 : 0;
    double x[RB][CB], y[kPre > 0 ? kPre : 1][RB][CB];
    const Group &g = a.grp[tl.g];
    auto fetch = [&](int t) {
#pragma unroll
        for (int k = 0; k < kPre; ++k)
            if (g.m0 + k < g.m1) load_mod<RB, CB>(a, tl, a.mod[g.m0 + k], obs, agent, t, y[k]);
    };
    if (tl.on) fetch(0);
    int cur = a.o_q, nxt = a.o_q + a.pq;
    for (int t = 0; t < a.T; ++t) {
        if (tl.on) {
            if (kPre > 0) {
#pragma unroll
                for (int i = 0; i < RB; ++i)
#pragma unroll
                    for (int j = 0; j < CB; ++j) {
                        x[i][j] = y[0][i][j];
#pragma unroll
                        for (int k = 1; k < kPre; ++k)
                            if (g.m0 + k < g.m1) x[i][j] += y[k][i][j];
                    }
                add_mods<RB, CB>(a, tl, kPre, obs, agent, t, x);
                if (t + 1 < a.T) fetch(t + 1);
            } else {
                load_mod<RB, CB>(a, tl, a.mod[g.m0], obs, agent, t, x);
                add_mods<RB, CB>(a, tl, 1, obs, agent, t, x);
            }
        }
        // predictive prior of the step: a weight, or log D at the first step
        if (states) {
            const int n = st.states();
            if (t > 0) {
                // (cur: the marginals of the step before)
                double acc = 0.0;
                if constexpr (!TB) {   // the predictive marginal under the factorised marginals
                    const FacDesc *facs = reinterpret_cast<const FacDesc *>(
                        a.base + (sizeof(ModDesc) * a.M + kAlign - 1) / kAlign * kAlign);
                    const FacDesc &fd = facs[f];
                    BDep d = bdep_of(facs, fd);
#pragma unroll
                    for (int p = 0; p < kMaxBDep; ++p)
                        for (int k = 0; k < a.F; ++k)
                            if (p < d.k && fd.bd[p] == k) d.off[p] = a.fac[k].po;
                    const float *B = at<float>(a.base, fd.b_off) + am * fd.b_agent;
                    acc = bdep_row(d, B + ((int64_t)acts[(t - 1) * a.F + f] * n + st.s()) * d.bs, smem + cur, -1, 0);
                } else {
                    const float *row = at<float>(a.base, row0 + acts[(t - 1) * a.F + f] * frow);
                    acc = plain_dot([&](int k) { return row[k]; }, smem + cur + st.po(), n);
                }
                mult = fmax(acc, kEps);
                lp = 0.0;
            }
            if (st.on()) smem[nxt + own] = 1.0 / n;
        }
        const int tmp = cur;
        cur = nxt;
        nxt = tmp;
        __syncthreads();
        double shift = __builtin_nan("");
        for (int k = 0; k < a.iters; ++k) {
            tl.here();
            if (tl.on) contract<RB, CB>(tl, x, smem, cur, a.o_p);
            __syncthreads();
            st.here();
            if (states) {
                const double lam = line_sum(smem + a.o_p + st.line(), st.len());
                double qn = softmax(a, smem, st, slots, lam + lp, mult, shift);
                if (st.on()) {
                    if (a.tau != 1.0) qn = (1.0 - a.tau) * smem[cur + own] + a.tau * qn;
                    smem[nxt + own] = qn;
                    if (k + 1 == a.iters) a.q[((int64_t)agent * a.T + t) * a.ntot + h.j] = (float)qn;
                }
            }
            __syncthreads();
            const int tm = cur;
            cur = nxt;
            nxt = tm;
        }
    }
}

// Tile shapes (rows x columns per lane) the kernels are built for; F: the
// filter only.  What a shape gives: the time of the calls that plan it (up to
// 28 each, drawn from 1 to 8 factors of 2 to 64 states, 1 to 200 steps, 1 to
// 2048 agents) when they have to do without it, in the geometric mean.
// Windows: 1 x 1 to 4 x 2 1.01 to 1.02, 8 x 1 1.04 (at most 1.9), 8 x 2 1.04,
// 4 x 4 1.04, 6 x 4 1.01 (at most 2.9), 8 x 4 1.08, 12 x 4 1.11, 12 x 5 1.75
// and 8 x 8 1.85 (both up to 12, where no other plan fits); 12 x 2 0.94 (0.80
// to 1.03: with 1024 threads it spills), so windows are not built for it.
// Filter: 0.97 to 1.06 up to 8 x 2 and 6 x 4, 12 x 2 1.01 (at most 1.9), 8 x 4
// 1.11, 12 x 4 1.15, 8 x 8 1.10 and 12 x 5 1.47 (both up to 13).
#define BI_RES_SHAPES(X, F) \
    X(1, 1) X(2, 1) X(4, 1) X(8, 1) X(2, 2) X(4, 2) X(8, 2) X(4, 4) X(6, 4) F(12, 2) X(8, 4) X(12, 4) X(12, 5) X(8, 8)

struct Shape {
    int rb, cb;
};
constexpr Shape kShapes[] = {
#define BI_X(r, c) {r, c},
    BI_RES_SHAPES(BI_X, BI_X)
#undef BI_X
};
constexpr int kNumShapes = sizeof(kShapes) / sizeof(kShapes[0]);

// Kernels by shape (the files named above).
const void *fpi_kernel(int shape);
const void *fpi_coupled(int shape);   // general B-dependency lists
// nullptr: not built for this shape
const void *vmp_kernel(int shape, bool one);
const void *mmp_kernel(int shape, bool one);

}  // namespace res
}  // namespace bi
