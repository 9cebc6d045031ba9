// Plan and launch of the register-resident agent kernels (resident_kernel.h).
#include "resident.h"

#include <algorithm>
#include <cstdio>
#include <cstring>

#include "profile.h"
#include "resident_coupled.h"
#include "resident_kernel.h"
#include "resident_streamed.h"

namespace bi {

namespace {

using namespace res;

constexpr size_t kLds = 160 * 1024;
constexpr int kCus = 256;
static_assert(sizeof(CoupledArgs) <= 4096 && sizeof(StreamedArgs) <= 4096, "kernel arguments");

struct Plan {
    CoupledArgs c;   // c.a: every kernel's arguments; the rest: general B-dependency lists
    int shape = -1, threads = 0;
    bool one = false, coupled = false;
    size_t lds = 0;
    double cost = 0.0;
};

// A group: factors of a maximal dependency list and the modalities inside it.
struct GroupSet {
    std::vector<int> fac, mods;
};

int div_up(int x, int y) { return (x + y - 1) / y; }
int pad4(int x) { return (x + 3) & ~3; }

// Modalities by falling rank, each into the first group that holds its list.
std::vector<GroupSet> groups_of(const bi_model *m)
{
    std::vector<int> order(m->M);
    for (int i = 0; i < m->M; ++i) order[i] = i;
    std::stable_sort(order.begin(), order.end(), [&](int x, int y) { return m->mods[x].rank > m->mods[y].rank; });
    std::vector<GroupSet> out;
    for (int i : order) {
        const int32_t *d = m->dep.data() + m->dep_off[i];
        const int k = m->dep_off[i + 1] - m->dep_off[i];
        GroupSet *in = nullptr;
        for (GroupSet &g : out)
            if (std::includes(g.fac.begin(), g.fac.end(), d, d + k)) {
                in = &g;
                break;
            }
        if (!in) {
            out.push_back({std::vector<int>(d, d + k), {}});
            in = &out.back();
        }
        in->mods.push_back(i);
    }
    return out;
}

// Element stride of factor f in a slice of modality md (0: not on its list).
int stride_of(const ModDesc &md, int f)
{
    int s = 1;
    for (int i = md.ncol - 1; i >= 0; --i) {
        if (md.cf[i] == f) return s;
        s *= md.cn[i];
    }
    s = md.Cp;
    for (int i = md.nrow - 1; i >= 0; --i) {
        if (md.rf[i] == f) return s;
        s *= md.rn[i];
    }
    return 0;
}

// Everything that does not depend on the tile shape.
bool plan_base(const bi_model *m, int algo, int T, Args &a)
{
    if (m->F > kMaxF || m->M > kMaxM) return false;
    for (const FacDesc &fd : m->facs) {
        if (fd.n > kMaxN) return false;
        // the transition phase for general lists takes lists of up to two factors
        if (!m->trivial_b && algo != BI_ALGO_FPI && T > 1 && fd.nbd > 2) return false;
    }
    for (const ModDesc &md : m->mods)
        if (md.rank > kRoles) return false;
    std::memset(&a, 0, sizeof(a));
    a.F = m->F;
    a.M = m->M;
    a.shared = m->mb == 1;
    a.T = T;
    a.ntot = m->ntot;
    int64_t bt = 0;
    const int es = algo == BI_ALGO_VMP ? 8 : 4;
    for (int f = 0; f < m->F; ++f) {
        const FacDesc &fd = m->facs[f];
        Fac &o = a.fac[f];
        o.n = fd.n;
        o.U = fd.U;
        o.qo = fd.q_off;
        o.b = fd.b_off;
        o.lb = fd.lb_off;
        o.ld = fd.ld_off;
        o.b_agent = fd.b_agent;
        o.ld_agent = fd.ld_agent;
        // rows an odd number of 16-byte units apart: the lanes' 16-byte reads
        // of consecutive rows fall on different banks
        o.bs = pad4(fd.n);
        if (o.bs * es / 16 % 2 == 0) o.bs += 16 / es;
        o.bt = (int)bt;
        bt += (int64_t)fd.U * fd.n * o.bs;
        if (bt > (int64_t)kLds) return false;
    }
    a.btot = (int)((bt * es + 15) / 16 * 16 / es);
    // state lanes: contexts side by side in a wave, or chunks of whole factors
    a.nchunk = 1;
    a.cpw = 64 / std::min(m->ntot, 64);
    if (m->ntot > 64) {
        a.cpw = 1;
        a.nchunk = 0;
        int start = 0, used = 0;
        for (int f = 0; f < m->F; ++f) {
            if (used + m->n[f] > 64) {
                a.chunk0[a.nchunk++] = start;
                start = a.fac[f].qo;
                used = 0;
            }
            used += m->n[f];
        }
        a.chunk0[a.nchunk++] = start;
        a.chunk0[a.nchunk] = m->ntot;
    }
    // 32-bit byte offsets into an agent's slices and soft tensors
    for (const ModDesc &md : m->mods) {
        a.llpc += md.slice;
        if ((int64_t)md.K * md.slice * 8 > UINT32_MAX) return false;
    }
    return a.llpc * 8 * T <= (int64_t)UINT32_MAX;
}

// The roles of a group's factors on tiles of rb x cb: the assignment with the
// least work per context (lanes, and values per line for the state phase).
// role[r]: factor of role r, or -1.
void choose_roles(const bi_model *m, const std::vector<int> &fac, int rb, int cb, int role[kRoles])
{
    const int k = (int)fac.size();
    double best = -1.0;
    std::vector<int> perm(fac);
    std::sort(perm.begin(), perm.end());
    do {
        // rank 1: b1; 2: a1 b1; 3: a1 b0 b1; 4: all
        int r[kRoles] = {-1, -1, -1, -1};
        r[kB1] = perm[0];
        if (k > 1) r[kA1] = perm[1];
        if (k > 2) r[kB0] = perm[2];
        if (k > 3) r[kA0] = perm[3];
        auto n = [&](int i) { return r[i] < 0 ? 1 : m->n[r[i]]; };
        const int na = div_up(n(kA1), rb), nb = div_up(n(kB1), cb), outer = n(kA0) * n(kB0);
        const double lanes = (double)outer * na * nb;
        double line = 0.0;
        for (int i = 0; i < kRoles; ++i)
            if (r[i] >= 0) {
                const double len = i == kA1 ? (double)outer * nb : i == kB1 ? (double)outer * na : lanes / n(i);
                line = std::max(line, len);
            }
        const double c = lanes * (2 * rb * cb + 4 * (rb + cb) + 20) / 64 + 2.0 * line;
        if (best < 0.0 || c < best) {
            best = c;
            std::copy(r, r + kRoles, role);
        }
    } while (std::next_permutation(perm.begin(), perm.end()));
}

// Transition tables read from the packed buffer, at 32-bit byte offsets.
bool tables_in_place(const bi_model *m, int algo, Args &a)
{
    if (m->bytes > (int64_t)UINT32_MAX) return false;
    for (int f = 0; f < a.F; ++f) {
        Fac &fd = a.fac[f];
        fd.bt = (int)(algo == BI_ALGO_VMP ? fd.lb / 8 : fd.b / 4);
        fd.bs = fd.n;
    }
    return true;
}

// Transition phase for general B-dependency lists (resident_coupled.h) in a
// workgroup of `threads`.  Returns the wave instructions of a sweep's
// transition phases.
double plan_trans(const bi_model *m, int algo, int T, int threads, CoupledArgs &c)
{
    const Args &a = c.a;
    const int es = algo == BI_ALGO_VMP ? 8 : 4;
    int role[kMaxF][kTRoles];   // factor of the role; kNext: the next state i
    constexpr int kNext = 100, kNone = -1;
    int lanes = 0;
    for (int j = 0; j < a.F; ++j) {
        const FacDesc &fd = m->facs[j];
        Trans &tr = c.tr[j];
        std::vector<int> dim = {kNext};
        for (int k = 0; k < fd.nbd; ++k) dim.push_back(fd.bd[k]);
        auto n = [&](int d) { return d == kNone ? 1 : d == kNext ? fd.n : m->n[d]; };
        // the roles with the fewest padded values
        std::sort(dim.begin(), dim.end());
        int64_t best = -1;
        do {
            const int r[kTRoles] = {dim.size() > 2 ? dim[2] : kNone, dim[0], dim[1]};
            const int64_t v = (int64_t)n(r[kO]) * div_up(n(r[kA]), kTA) * div_up(n(r[kB]), kTB);
            if (best < 0 || v < best) {
                best = v;
                std::copy(r, r + kTRoles, role[j]);
            }
        } while (std::next_permutation(dim.begin(), dim.end()));
        for (int r = 0; r < kTRoles; ++r) tr.n[r] = n(role[j][r]);
        tr.na = div_up(tr.n[kA], kTA);
        tr.nb = div_up(tr.n[kB], kTB);
        lanes += tr.na * tr.nb;
    }
    // spare threads divide the outer states
    const int spare = std::max(1, threads / std::max(1, lanes * (T - 1)));
    c.LP = 0;
    int64_t bt = 0;
    double work = 0.0;
    for (int j = 0; j < a.F; ++j) {
        Trans &tr = c.tr[j];
        tr.per = div_up(tr.n[kO], std::min(spare, tr.n[kO]));
        tr.parts = div_up(tr.n[kO], tr.per);
        tr.lane0 = c.LP;
        c.LP += tr.na * tr.nb * tr.parts;
        work = std::max(work, tr.per * 45.0 + 50.0);
        // strides of the packed table [u][i][list], and of the copy in LDS
        const FacDesc &fd = m->facs[j];
        tr.packed = algo == BI_ALGO_VMP ? fd.lb_off : fd.b_off;
        tr.agent = fd.b_agent;
        tr.i = fd.n * fd.bstates;
        for (int r = 0; r < kTRoles; ++r) {
            int s = role[j][r] == kNext ? fd.bstates : 0;
            for (int k = 0, low = fd.bstates; k < fd.nbd; ++k) {
                low /= fd.bdn[k];
                if (role[j][r] == fd.bd[k]) s = low;
            }
            tr.s[r] = s;
        }
        tr.rs = kTB * tr.nb;   // (rows an odd number of 16-byte units apart)
        if (tr.rs * es / 16 % 2 == 0) tr.rs += 16 / es;
        tr.os = kTA * tr.na * tr.rs;
        tr.us = tr.n[kO] * tr.os;
        tr.tb = (int)bt;
        bt = std::min<int64_t>(bt + (int64_t)fd.U * tr.us, kLds);
    }
    c.steps = std::max(1, std::min(T - 1, threads / c.LP));
    c.a.btot = (int)bt;
    // lines: per factor the forward message's shares, then each child's
    int off = 0;
    auto shares = [&](int j, int r) {
        const Trans &tr = c.tr[j];
        return r == kO ? tr.na * tr.nb : r == kA ? tr.nb * tr.parts : tr.na * tr.parts;
    };
    auto role_of = [&](int j, int f) { return (int)(std::find(role[j], role[j] + kTRoles, f) - role[j]); };
    for (int f = 0; f < a.F; ++f) {
        const FacDesc &fd = m->facs[f];
        TFac &tf = c.tf[f];
        tf.line = off;
        tf.fwd = shares(f, role_of(f, kNext));
        int len = (tf.fwd + 1) / 2 * 2;
        tf.nch = fd.nch;
        for (int k = 0; k < fd.nch; ++k) {
            tf.off[k] = len;
            tf.len[k] = shares(fd.ch[k], role_of(fd.ch[k], f));
            len += (tf.len[k] + 1) / 2 * 2;
        }
        tf.pitch = len / 2 % 2 ? len : len + 2;
        off += std::max(div_up(fd.n, kTA) * kTA, div_up(fd.n, kTB) * kTB) * tf.pitch;
    }
    c.plt = off;   // (even: the pitches are)
    if (2 * (int64_t)off > 0x7fff) c.LP = INT32_MAX;   // (packed offsets, see Place)
    for (int j = 0; j < a.F; ++j) {
        Trans &tr = c.tr[j];
        for (int r = 0; r < kTRoles; ++r) {
            const int d = role[j][r], f = d == kNext ? j : d;
            if (d == kNone) {
                tr.q[r] = tr.line[r] = tr.pitch[r] = 0;
                continue;
            }
            const TFac &tf = c.tf[f];
            int at = 0;
            if (d != kNext)
                for (int k = 0; k < tf.nch; ++k)
                    if (m->facs[f].ch[k] == j) at = tf.off[k];
            // the next state's marginals and lines are those of step t + 1
            tr.q[r] = a.fac[f].po + (d == kNext ? a.pq : 0);
            tr.line[r] = tf.line + at + (d == kNext ? c.plt : 0);
            tr.pitch[r] = tf.pitch;
        }
    }
    return work * div_up(T - 1, c.steps) * threads / 64;
}

bool plan_shape(const bi_model *m, int algo, int b, int T, const Args &base, const std::vector<GroupSet> &gs,
                int shape, Plan &out)
{
    const int rb = kShapes[shape].rb, cb = kShapes[shape].cb;
    Args &a = out.c.a;
    a = base;
    const bool coupled = !m->trivial_b && algo != BI_ALGO_FPI && T > 1;
    out.coupled = coupled;
    const bool fpi = algo == BI_ALGO_FPI;
    if (!fpi && !coupled && !vmp_kernel(shape, false)) return false;
    const int contexts = fpi ? 1 : T, maxthreads = max_threads(rb, cb, fpi || coupled);
    int role[kMaxG][kRoles];
    int room[kMaxF];   // marginals of a factor that a tile may read (its states and padding)
    for (int f = 0; f < a.F; ++f) room[f] = pad4(coupled ? div_up(a.fac[f].n, kTA) * kTA : a.fac[f].n);
    int64_t lanes = 0;
    for (int gi = 0; gi < a.G; ++gi) {
        choose_roles(m, gs[gi].fac, rb, cb, role[gi]);
        Group &g = a.grp[gi];
        for (int r = 0; r < kRoles; ++r) g.n[r] = role[gi][r] < 0 ? 1 : m->n[role[gi][r]];
        g.na = div_up(g.n[kA1], rb);
        g.nb = div_up(g.n[kB1], cb);
        g.lane0 = (int)lanes;
        lanes += (int64_t)g.n[kA0] * g.na * g.n[kB0] * g.nb;
        if (lanes * contexts > maxthreads) return false;
        if (role[gi][kA1] >= 0) room[role[gi][kA1]] = std::max(room[role[gi][kA1]], pad4(g.na * rb));
        room[role[gi][kB1]] = std::max(room[role[gi][kB1]], pad4(g.nb * cb));
    }
    a.LT = (int)lanes;
    // marginals of a context; the states' lines.  Values of a group in a line:
    // one from every lane of the same state.  A tile's rows and columns past
    // the last state write into lines behind it (pad), which nothing reads; the
    // shares for an absent role go to the spare line at the end.
    a.pq = std::max(kFirst, pad4(rb));   // (an absent a1 reads rb values)
    int64_t off = 0;
    int longest = 0, pad[kMaxF] = {};
    for (int gi = 0; gi < a.G; ++gi) {
        const Group &g = a.grp[gi];
        if (role[gi][kA1] >= 0) pad[role[gi][kA1]] = std::max(pad[role[gi][kA1]], g.na * rb - g.n[kA1]);
        pad[role[gi][kB1]] = std::max(pad[role[gi][kB1]], g.nb * cb - g.n[kB1]);
    }
    for (int f = 0; f < a.F; ++f) {
        Fac &fd = a.fac[f];
        fd.po = a.pq;
        a.pq += room[f];
        fd.len = 0;
        for (int gi = 0; gi < a.G; ++gi) {
            Group &g = a.grp[gi];
            const int all = g.n[kA0] * g.na * g.n[kB0] * g.nb;
            for (int r = 0; r < kRoles; ++r)
                if (role[gi][r] == f) {
                    g.q[r] = fd.po;
                    g.line[r] = (int)off + fd.len;   // (base added below: off is the factor's first line)
                    fd.len += r == kA1 ? all / g.na : r == kB1 ? all / g.nb : all / g.n[r];
                }
        }
        fd.line = (int)off;
        // lines of whole groups of 4 values, an odd number of 16-byte units apart
        // (a factor on no list has none)
        fd.pitch = fd.len ? pad4(fd.len) + 2 : 0;
        off += (int64_t)(fd.n + pad[f]) * fd.pitch;
        longest = std::max(longest, fd.len);
        if (off > (int64_t)kLds / 8 || fd.len > 0x7fff) return false;
    }
    const int spare = (int)off;
    a.pl = spare + 2 * rb;   // (an absent a1 writes rb values)
    a.pl = (a.pl + 1) / 2 * 2;
    for (int gi = 0; gi < a.G; ++gi) {
        Group &g = a.grp[gi];
        for (int r = 0; r < kRoles; ++r) {
            const int f = role[gi][r];
            g.pitch[r] = f < 0 ? (r == kA1 ? 1 : 0) : a.fac[f].pitch;
            if (f < 0) {
                g.q[r] = 0;
                g.line[r] = spare;
            }
        }
        g.m0 = gi ? a.grp[gi - 1].m1 : 0;
        g.m1 = g.m0;
        for (int i : gs[gi].mods) {
            const ModDesc &md = m->mods[i];
            Mod &o = a.mod[g.m1++];
            o.la = md.la_off;
            o.la_agent = md.la_agent;
            o.ll = 0;
            for (int k = 0; k < i; ++k) o.ll += m->mods[k].slice;
            o.slice = md.slice;
            o.m = i;
            for (int r = 0; r < kRoles; ++r) o.s[r] = role[gi][r] < 0 ? 0 : stride_of(md, role[gi][r]);
        }
    }
    if (a.pl > 0x7fff || a.pq > 0x7fff || T > 0x7fff) return false;   // (packed offsets, see State)
    a.sv = a.cpw * a.pq;
    const int cw = div_up(a.LT * contexts, 64);
    const int units = a.nchunk == 1 ? div_up(contexts, a.cpw) : contexts * a.nchunk;
    const int waves = fpi ? std::max(cw, units) : std::max(cw, std::min(units, maxthreads / 64));
    if (waves * 64 > maxthreads) return false;
    out.one = units <= waves;
    out.threads = 64 * waves;
    a.units = units;
    // LDS, in doubles
    const int64_t es = algo == BI_ALGO_VMP ? 8 : 4;
    double trans = 0.0;
    if (coupled) trans = plan_trans(m, algo, T, out.threads, out.c);
    if (coupled && out.c.LP > out.threads) return false;
    int64_t o = 0;
    auto take = [&](int64_t n) {
        const int64_t at = o;
        o += (n + 1) / 2 * 2;
        return (int)at;
    };
    a.o_q = take((fpi ? 2 : 2 * (int64_t)T) * a.pq);
    a.o_p = take((int64_t)contexts * std::max(a.pl, coupled ? out.c.plt : 0));
    a.o_e = take((int64_t)waves * a.sv);
    a.o_a = take(((int64_t)(T - 1) * a.F + (int64_t)T * a.M + 1) / 2);
    a.o_f = take(fpi ? 0 : a.pq);
    a.o_r = take(fpi || out.one ? 0 : 3 * 64 * (int64_t)units);
    if (o * 8 > (int64_t)kLds) return false;
    // the transition tables take the form that fits behind the rest
    a.tab = kGlobal;
    if (coupled) {
        out.c.o_x = take((int64_t)a.F * sizeof(TFac) / 8);
        out.c.o_s = take(out.one ? 0 : 2 * 64 * (int64_t)units);
        const int64_t once = ((int64_t)a.btot * es + 7) / 8;
        out.c.lds_tab = (o + once) * 8 <= (int64_t)kLds;
        if (!mmp_coupled(shape, out.one, out.c.lds_tab)) return false;
        a.o_b = take(out.c.lds_tab ? once : 0);
        for (int f = 0; f < a.F; ++f) a.fac[f].bt = a.fac[f].bs = 0;
    } else if (!fpi && T > 1) {
        const int64_t room = (int64_t)kLds / 8 - o, once = ((int64_t)a.btot * es + 7) / 8;
        a.tab = 2 * once <= room ? kBoth : once <= room ? kOnce : kGlobal;
        a.o_b = take(a.tab * once);
        if (a.tab == kGlobal && !tables_in_place(m, algo, a)) return false;
    }
    if (o * 8 > (int64_t)kLds) return false;
    out.lds = (size_t)o * 8;
    out.shape = shape;
    // Estimated cycles of a sweep.  A workgroup's instructions keep its compute
    // unit busy for 5 / 4 cycles each (4 SIMDs, 4 cycles for a wave's fp64
    // instruction, some of them idle), one wave's chain of them takes 10 each and
    // the barriers and LDS round trips 1000; as many workgroups as fit share
    // a compute unit (8 x 6 states, 1024 agents, VMP: 4 x 2 tiles 36 us, 1 x 1
    // 59 us; 12 x 10 x 8 states, 4096 agents, MMP: 6 x 4 tiles 1.11 ms, 12 x 4
    // 1.26 ms, 12 x 5 1.48 ms).  The order of the estimates is not always that
    // of the times: on 785 drawn calls the next shape was more than 5% faster
    // 117 times, more than 20% 14 times, 0.38 of the time at the extreme (a
    // filter on 2 x 2 tiles that 4 x 4 suit better).
    const int nmax = *std::max_element(m->n.begin(), m->n.end()), p = rb * cb;
    const double ic = 2.0 * p + 4.0 * (rb + cb) + 20.0;
    const double is = 160.0 + 2.0 * longest + (fpi ? 0.0 : (a.tab == kBoth ? 5.0 : a.tab == kOnce ? 8.0 : 16.0) * nmax) + 2.0 * nmax;
    const int regs = p <= 4 ? 80 : p <= 8 ? 96 : p <= 24 ? 128 : p <= 32 ? 200 : 256;
    const int fit = std::max(1, std::min(4 * (512 / regs) / waves, (int)(kLds / out.lds)));
    const int side = std::min(fit, div_up(b, kCus));   // workgroups side by side on a compute unit
    // (12 x 5 and 8 x 8 spill 58 to 74 registers; 6 x 4, with 25 to 29, is not charged)
    const double issue = 1.25 * (cw * ic + units * is + trans) * (p > 48 ? 1.2 : 1.0);
    const double chain = 10.0 * (ic + div_up(units, waves) * is + trans / waves) + (coupled ? 2000.0 : 1000.0);
    out.cost = std::max(side * issue, chain) * div_up(b, kCus * side);
    return true;
}

bool make_plan(const bi_model *m, int algo, int b, int T, Plan &best)
{
    Args base;
    if (!plan_base(m, algo, T, base)) return false;
    best.shape = -1;
    const std::vector<GroupSet> gs = groups_of(m);
    base.G = (int)gs.size();
    if (base.G > kMaxG) return false;
    Plan p;
    for (int s = 0; s < kNumShapes; ++s)
        if (plan_shape(m, algo, b, T, base, gs, s, p) && (best.shape < 0 || p.cost < best.cost)) best = p;
    return best.shape >= 0;
}

// Plan of the streamed window kernel for at most `blocks` blocks of a slice
// per lane and step (resident_streamed.h).
bool plan_streamed(const bi_model *m, int algo, int T, const Args &base, int blocks, int tab, StreamedArgs &c, size_t &lds,
                   int &threads, double &cost)
{
    Args &a = c.a;
    a = base;
    int role[kStreamM][kSRoles];
    int64_t lanes = 0, values = 0;
    int longest = 0;   // blocks of a lane
    for (int i = 0; i < a.M; ++i) {
        const ModDesc &md = m->mods[i];
        SMod &s = c.mod[i];
        const int32_t *d = m->dep.data() + m->dep_off[i];
        std::vector<int> rest(d, d + md.rank);
        int *r = role[i];
        std::fill(r, r + kSRoles, -1);
        // columns: the factor with stride 1; where it has one or two states,
        // and for the rows, the one that fills its blocks best; of the others
        // the larger is divided among lanes.  (Windows of 256 agents, 16
        // sweeps: 31 x 11 x 26 x 2 states with the last as columns 2.45 ms,
        // with the third 1.54 ms; 30 x 30 x 19 x 3 1.56 ms, with the first
        // 1.89 ms, as its loads then touch three times the lines.)
        const int inner = md.cf[md.ncol - 1];
        auto fills = [&](int x, int y) { return (int64_t)pad4(m->n[x]) * m->n[y] < (int64_t)pad4(m->n[y]) * m->n[x]; };
        r[kCol] = m->n[inner] < 3 ? *std::min_element(rest.begin(), rest.end(), fills) : inner;
        rest.erase(std::find(rest.begin(), rest.end(), r[kCol]));
        auto pick = [&](auto better) {
            if (rest.empty()) return -1;
            const auto it = std::min_element(rest.begin(), rest.end(), better);
            const int f = *it;
            rest.erase(it);
            return f;
        };
        r[kRow] = pick(fills);
        r[kP] = pick([&](int x, int y) { return m->n[x] > m->n[y]; });
        r[kO2] = pick([](int, int) { return false; });
        for (int k = 0; k < kSRoles; ++k) {
            s.n[k] = r[k] < 0 ? 1 : m->n[r[k]];
            s.s[k] = r[k] < 0 ? 0 : stride_of(md, r[k]);
        }
        s.na = div_up(s.n[kRow], kBlk);
        s.nb = div_up(s.n[kCol], kBlk);
        s.per = std::min(s.n[kP], std::max(1, blocks / s.n[kO2]));
        // The walked states whose values lie closer together go innermost: a
        // cache line that a lane's block takes in part is then finished in the
        // next steps of the walk, while it is still in the compute unit's cache
        // (a second outer role walked in between brings up to 1 MB past it).
        // Of 524 streamed calls 48 became 1.02 to 1.28 times as fast, none less
        // than 0.97; 256 agents, 15 x 32 x 24 x 6 states, 8 steps, VMP: 4.52 ->
        // 3.58 ms (4.09 by the kernels of agent.hip).
        s.flip = s.per > 1 && s.n[kO2] > 1 && s.s[kP] < s.s[kO2];
        s.parts = div_up(s.n[kP], s.per);
        s.lane0 = (int)lanes;
        lanes += (int64_t)s.na * s.nb * s.parts;
        if (lanes > kStreamThreads) return false;
        longest = std::max(longest, s.per * s.n[kO2]);
        values += md.slice;
        s.slice = md.slice;
        s.m = i;
        s.la = md.la_off;
        s.la_agent = md.la_agent;
        s.ll = i ? c.mod[i - 1].ll + m->mods[i - 1].slice : 0;
    }
    c.LP = (int)lanes;
    a.pq = kFirst;
    int64_t off = 0;
    for (int f = 0; f < a.F; ++f) {
        Fac &fd = a.fac[f];
        fd.po = a.pq;
        a.pq += pad4(fd.n);
        fd.line = (int)off;
        fd.len = 0;
        for (int i = 0; i < a.M; ++i) {
            SMod &s = c.mod[i];
            const int64_t blk = (int64_t)s.na * s.nb;
            for (int k = 0; k < kSRoles; ++k)
                if (role[i][k] == f) {
                    s.q[k] = fd.po;
                    s.line[k] = (int)off + fd.len;
                    fd.len += (int)(k == kP ? blk : k == kO2 ? blk * s.parts : k == kRow ? s.nb * s.parts : s.na * s.parts);
                }
        }
        fd.pitch = fd.len ? pad4(fd.len) + 2 : 0;
        off += (int64_t)pad4(fd.n) * fd.pitch;
        if (off > (int64_t)kLds / 8 || fd.len > 0x7fff) return false;
    }
    a.pl = (int)off + 2;   // (shares of absent roles go to the spare value behind the lines)
    for (int i = 0; i < a.M; ++i)
        for (int k = 0; k < kSRoles; ++k) {
            SMod &s = c.mod[i];
            s.pitch[k] = role[i][k] < 0 ? 0 : a.fac[role[i][k]].pitch;
            if (role[i][k] < 0) {
                s.q[k] = 0;
                s.line[k] = (int)off;
            }
        }
    if (a.pl > 0x7fff || T > 0x7fff) return false;   // (packed offsets, see State)
    a.sv = a.cpw * a.pq;
    a.units = a.nchunk == 1 ? div_up(T, a.cpw) : T * a.nchunk;
    const int waves = std::min(kStreamThreads / 64, std::max(div_up((int)std::min<int64_t>(lanes * T, kStreamThreads), 64), a.units));
    threads = 64 * waves;
    c.steps = std::min(T, threads / c.LP);
    if (c.steps < 1) return false;
    int64_t o = 0;
    auto take = [&](int64_t n) {
        const int64_t at = o;
        o += (n + 1) / 2 * 2;
        return (int)at;
    };
    const int64_t once = T > 1 ? ((int64_t)a.btot * (algo == BI_ALGO_VMP ? 8 : 4) + 7) / 8 : 0;
    const int64_t fixed = 2 * (int64_t)T * a.pq + (int64_t)waves * a.sv + ((int64_t)(T - 1) * a.F + (int64_t)T * a.M + 1) / 2 +
                          a.pq + 3 * 64 * (int64_t)a.units + (int64_t)T * a.pq + 16;
    a.tab = tab;
    const int64_t room = (int64_t)kLds / 8 - fixed - a.tab * once;
    c.chunk = (int)std::min<int64_t>(T, std::max<int64_t>(0, room / a.pl));
    if (c.chunk < 1) return false;
    c.steps = std::min(c.steps, c.chunk);
    if (a.tab == kGlobal && T > 1 && !tables_in_place(m, algo, a)) return false;
    a.o_q = take(2 * (int64_t)T * a.pq);
    a.o_p = take((int64_t)c.chunk * a.pl);
    a.o_e = take((int64_t)waves * a.sv);
    a.o_a = take(((int64_t)(T - 1) * a.F + (int64_t)T * a.M + 1) / 2);
    a.o_f = take(a.pq);
    a.o_r = take(3 * 64 * (int64_t)a.units);
    a.o_b = take(a.tab * once);
    c.o_l = take((int64_t)T * a.pq);
    if (o * 8 > (int64_t)kLds) return false;
    lds = (size_t)o * 8;
    // cycles of a sweep: the lanes' blocks (85 instructions each, 5 cycles on a
    // SIMD's share of the waves) or the slices' way from L2, then the sums of the
    // chunks' lines and their barriers, then the state phase, whose reads of a
    // table outside LDS wait for one another (75 states, 20 steps, 1925 states'
    // transitions: MMP 662 us with 9 steps to a chunk and the tables in memory)
    const double rounds = (double)(T / c.chunk) * div_up(c.chunk, c.steps) +
                          (T % c.chunk ? div_up(T % c.chunk, c.steps) : 0);
    const double work = rounds * (longest * 85.0 + 100.0) * 5.0 * waves / 4.0;
    int longest_line = 0;
    for (int f = 0; f < a.F; ++f) longest_line = std::max(longest_line, a.fac[f].len);
    const double sums = std::max(longest_line / 32.0 * 130.0, a.pl * (double)c.chunk / 16.0);
    int n = 0;
    for (int f = 0; f < a.F; ++f) n = std::max(n, a.fac[f].n);
    const double states = T > 1 ? (double)div_up(a.units, waves) * n * (tab == kBoth ? 16.0 : tab == kOnce ? 30.0 : 400.0) : 0.0;
    cost = std::max(work, (double)T * values * 8.0 / 64.0) + (800.0 + sums) * div_up(T, c.chunk) + states;
    return true;
}

bool make_streamed(const bi_model *m, int algo, int T, StreamedArgs &best, size_t &lds, int &threads)
{
    Args base;
    if (algo == BI_ALGO_FPI || !m->trivial_b || m->M > kStreamM || !plan_base(m, algo, T, base)) return false;
    static const int kBlocks[] = {1, 2, 3, 4, 6, 8, 11, 16, 24, 32, 64, 128, 512, 4096};
    double cost = -1.0;
    StreamedArgs c;
    for (int i = 0; i < 3 * (int)(sizeof(kBlocks) / sizeof(kBlocks[0])); ++i) {
        const int blocks = kBlocks[i / 3], tab = kBoth - i % 3;
        size_t l = 0;
        int th = 0;
        double co = 0.0;
        if (!plan_streamed(m, algo, T, base, blocks, tab, c, l, th, co) || (cost >= 0.0 && co >= cost)) continue;
        best = c;
        lds = l;
        threads = th;
        cost = co;
    }
    return cost >= 0.0;
}

// Whether a window that the kernels of agent.hip would hold in LDS (staged)
// runs better there than streamed.  Their workgroups of 4 waves share a compute
// unit by fours and more; the streamed kernel's 209 registers leave a unit 8
// waves, so where its workgroups do not all fit at once they take turns.  On
// 596 staged windows of 5 to 8 maximal lists (2 to 9 states a factor, 1 to 20
// steps, 1 to 2048 agents, 16 sweeps) the streamed kernel was 1.00 to 5.0 times
// as fast on all 526 that fit, and 0.42 to 1.84 times (0.93 in the geometric
// mean) on the other 70: 1438 agents, 5 steps, VMP 226 us staged, 542 us streamed.
bool staged_is_better(int b, int threads, bool staged)
{
    constexpr int kWavesFit = 8;
    return staged && div_up(b, kCus) * (threads / 64) > kWavesFit;
}

// Whether some modality's walk is flipped.
bool flips(const StreamedArgs &c)
{
    return std::any_of(c.mod, c.mod + c.a.M, [](const SMod &s) { return s.flip != 0; });
}

// The kernel and arguments of a call.
struct Choice {
    Plan p;           // (streamed: lds and threads of it)
    StreamedArgs sa;
    const void *fn;
    const char *name;   // profile class
    Args *a;
    void *args;
};

bool choose(const bi_model *m, int algo, int b, int T, bool staged, Choice &c)
{
    const bool fpi = algo == BI_ALGO_FPI, vmp = algo == BI_ALGO_VMP;
    Plan &p = c.p;
    if (make_plan(m, algo, b, T, p)) {
        c.a = &p.c.a;
        c.args = p.coupled ? (void *)&p.c : (void *)c.a;
        c.fn = fpi ? (m->trivial_b ? fpi_kernel(p.shape) : fpi_coupled(p.shape))
             : p.coupled ? (vmp ? vmp_coupled(p.shape, p.one, p.c.lds_tab) : mmp_coupled(p.shape, p.one, p.c.lds_tab))
                         : (vmp ? vmp_kernel(p.shape, p.one) : mmp_kernel(p.shape, p.one));
        c.name = fpi ? "agent_filter_resident" : p.coupled ? "agent_window_coupled" : "agent_window_resident";
        return true;
    }
    if (make_streamed(m, algo, T, c.sa, p.lds, p.threads) && !staged_is_better(b, p.threads, staged)) {
        c.a = &c.sa.a;
        c.args = &c.sa;
        c.fn = vmp ? vmp_streamed(flips(c.sa)) : mmp_streamed(flips(c.sa));
        c.name = "agent_window_streamed";
        return true;
    }
    return false;
}

}  // namespace

bool describe_resident(const bi_model *m, int algo, int b, int T, bool staged, char *buf, size_t cap)
{
    Choice c;
    if (!choose(m, algo, b, T, staged, c)) return false;
    static const char *tabs[] = {"packed", "once", "twice"};
    const Plan &p = c.p;
    if (c.a == &c.sa.a)
        std::snprintf(buf, cap, "%s chunk=%d steps=%d flip=%d tables=%s threads=%d lds=%zu", c.name, c.sa.chunk,
                      c.sa.steps, (int)flips(c.sa), tabs[c.a->tab], p.threads, p.lds);
    else
        std::snprintf(buf, cap, "%s tile=%dx%d tables=%s passes=%s groups=%d threads=%d lds=%zu", c.name,
                      kShapes[p.shape].rb, kShapes[p.shape].cb,
                      p.coupled ? (p.c.lds_tab ? "lds" : "packed") : tabs[c.a->tab], p.one ? "one" : "several", c.a->G,
                      p.threads, p.lds);
    return true;
}

int launch_resident(const bi_model *m, int algo, int b, int T, bool staged, const int32_t *obs, const double *ll,
                    const int32_t *act, const float *prior, double tau, int iters, float *q, hipStream_t stream)
{
    Choice c;
    if (!choose(m, algo, b, T, staged, c)) return kNoPlan;
    Args *a = c.a;
    a->base = m->dev;
    a->iters = iters;
    a->obs = obs;
    a->ll = ll;
    a->act = act;
    a->prior = prior;
    a->tau = tau;
    a->q = q;
    void *args[1] = {c.args};
    hipError_t e = func_max_lds(c.fn, (int)kLds);
    if (e == hipSuccess) {
        ProfScope ps(c.name, stream);
        e = hipLaunchKernel(c.fn, dim3(b), dim3(c.p.threads), args, c.p.lds, stream);
    }
    if (e != hipSuccess) return fail(BI_ERR_DEVICE, "kernel launch failed: %s", hipGetErrorString(e));
    return BI_OK;
}

}  // namespace bi
