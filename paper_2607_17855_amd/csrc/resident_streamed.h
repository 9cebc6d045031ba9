// Window kernel (VMP and MMP, trivial B-dependency lists) for agents whose
// likelihood tensors do not fit a workgroup's registers: states and shares as
// in resident_kernel.h, the observed slices read from memory in every sweep.
//
// A modality's slice is contracted like a transition tensor of
// resident_coupled.h: its factors take the roles of an inner column (the
// factor with stride 1), an inner row and up to two outer ones; a lane has 4
// x 4 states of the inner roles and walks the outer ones, loading the next
// block while it works on one, and leaves one share per inner state, per
// outer state that it walked and, for a second outer role, per state of that.
// So every value is read once per sweep for all of its messages, a wave reads
// whole rows, and a lane's 8 loads of 16 bytes are in flight for the 16 values
// before them.
//
// Lanes: per step LP places (modality, blocks, part of the outer states), as
// many steps side by side as fit the workgroup, the other steps after them.
// Where the lines of the whole window do not fit LDS, steps are taken in
// chunks; each chunk's messages are added up before the next one starts.
//
// What bounds it: latency.  256 agents sharing a model of 17 x 11 x 5 x 26
// states in lists of up to three, 11 steps, 16 sweeps, VMP: 894 -> 388 us
// against the kernels of agent.hip, which read the slices twice per sweep.  Of
// the 388 us, leaving out the loads saves 90, the sums of the lines 74, the
// state phase 68, the share writes nothing; the rest is the products with the
// barriers between a sweep's rounds.  One workgroup of 8 waves to a compute unit
// (158 KB of LDS, 209 registers): vector instructions issue in 32% of a SIMD's
// cycles, waves wait in 46% of theirs, LDS works in 21% of the cycles, and the
// slices take 9 of the 64 bytes a cycle that L2 gives a compute unit.
#pragma once

#include "resident_kernel.h"

namespace bi {
namespace res {

constexpr int kBlk = 4;   // states of the inner roles per lane
// 512 threads: two blocks of 16 values, the sums and the offsets take 150
// registers (1024 threads, 128 registers: 98 spilled).
constexpr int kStreamThreads = 512;
constexpr int kStreamM = 8;   // modalities

enum { kP, kO2, kRow, kCol, kSRoles };   // outer (divided among lanes), second outer, inner row, inner column

struct SMod {
    int32_t n[kSRoles];        // states per role (1: absent)
    int32_t q[kSRoles];        // marginal offset (0: absent, the constant 1)
    int32_t line[kSRoles], pitch[kSRoles];   // shares: offset of state 0, distance (absent: the spare line)
    int32_t s[kSRoles];        // element strides in the slice
    int32_t na, nb, parts, per, lane0;       // blocks along row and column, parts of the outer states, first lane
    int32_t slice, m;
    int32_t flip;              // the lane's own outer states are walked innermost, not the second ones
    int64_t la, la_agent, ll;
};

struct StreamedArgs {
    Args a;
    int LP, steps, chunk;      // lanes per step, steps side by side, steps per chunk
    int o_l;                   // LDS: messages of the window
    SMod mod[kStreamM];
};

struct Block {
    double x[kBlk][kBlk];
};

// FLIP: some modality's walk is flipped.
template <int ALGO, bool FLIP>
__global__ __launch_bounds__(kStreamThreads) void streamed_kernel(StreamedArgs c)
{
    using BT = std::conditional_t<ALGO == BI_ALGO_VMP, double, float>;
    extern __shared__ double smem[];
    const Args &a = c.a;
    const int agent = blockIdx.x, waves = (int)blockDim.x >> 6;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = (int)threadIdx.x & 63;
    const int64_t am = a.shared ? 0 : agent;
    stage_window<BT>(a, smem, agent, am, ALGO == BI_ALGO_VMP, waves);
    const BT *tab = reinterpret_cast<const BT *>(smem + a.o_b);
    const int *acts = reinterpret_cast<const int *>(smem + a.o_a), *obs = acts + (a.T - 1) * a.F;
    __syncthreads();
    const int units = a.units;
    int2 *roles = reinterpret_cast<int2 *>(smem + a.o_r);
    for (int u = wave; u < units; u += waves) {
        const State st = state_of(a, where_of(a, u, a.T), acts, a.T, am);
        put_role(roles, u * 64 + lane, st);
        if (st.on()) smem[a.o_q + st.t() * a.pq + st.po() + st.s()] = 1.0 / st.states();   // uniform start
    }
    const int slots = wave * a.sv + (a.nchunk == 1 && lane < a.cpw * a.ntot ? lane / a.ntot * a.pq : 0);

    // this lane's place: modality, blocks, outer part; the first step it takes
    const int t0 = (int)threadIdx.x / c.LP;
    int rem = (int)threadIdx.x - t0 * c.LP, mi = 0;
    for (int k = 1; k < a.M; ++k)
        if (rem >= c.mod[k].lane0) mi = k;
    const bool on = t0 < c.steps;
    const SMod &md = c.mod[mi];
    rem -= md.lane0;
    const int nb = md.nb, na = md.na;
    const int bb = rem % nb;
    rem /= nb;
    const int ab = rem % na, part = rem / na;
    // outer states walked: o_count of its own (the names in _p), each with the n2
    // second ones (_2), or flipped the other way round
    const int row = kBlk * ab, o_first = part * md.per;
    int o_count = min(md.per, md.n[kP] - o_first), n2 = md.n[kO2];
    // the last column block reaches back over states of the one before (skip
    // of them, left out) so that its loads stay inside the row
    const int ncol = md.n[kCol], col = max(0, min(kBlk * bb, ncol - kBlk)), skip = kBlk * bb - col;
    int ro[kBlk];
#pragma unroll
    for (int i = 0; i < kBlk; ++i) ro[i] = min(row + i, md.n[kRow] - 1) * md.s[kRow] + col * md.s[kCol];
    const int s_col = md.s[kCol], last_col = ncol - 1 - col;   // (fewer than 4 columns: the last one repeats, at weight 0)
    const bool rows4 = ncol >= kBlk && s_col == 1;
    int sp = md.s[kP], s2 = md.s[kO2];
    const int m_obs = md.m, slice = md.slice;
    const int first = o_first * sp;   // element offset of its first outer state
    const char *X = a.ll ? reinterpret_cast<const char *>(a.ll + (int64_t)agent * a.T * a.llpc + md.ll)
                         : a.base + md.la + (a.shared ? 0 : (int64_t)agent * md.la_agent * 8);
    const int q_row = md.q[kRow] + row, q_col = md.q[kCol] + col;
    int q_p = md.q[kP] + o_first, q_2 = md.q[kO2];
    const int parts = md.parts, pitch_row = md.pitch[kRow], pitch_col = md.pitch[kCol];
    int pitch_p = md.pitch[kP], pitch_2 = md.pitch[kO2];
    const int l_row = md.line[kRow] + row * pitch_row + (md.q[kRow] ? bb * parts + part : 0);
    const int l_col = md.line[kCol] + col * pitch_col + ab * parts + part;
    int l_p = md.line[kP] + o_first * pitch_p + (md.q[kP] ? ab * nb + bb : 0);
    int l_2 = md.line[kO2] + (md.q[kO2] ? (ab * nb + bb) * parts + part : 0);
    bool share_2 = n2 > 1;   // (an absent second outer role has no share)
    if (FLIP && md.flip) {
        auto swap = [](int &x, int &y) {
            const int t = x;
            x = y;
            y = t;
        };
        swap(o_count, n2);
        swap(sp, s2);
        swap(q_p, q_2);
        swap(pitch_p, pitch_2);
        swap(l_p, l_2);
        share_2 = true;
    }

    auto load = [&](Block &b, uint32_t at0) {
        if (rows4) {
#pragma unroll
            for (int i = 0; i < kBlk; ++i)
                __builtin_memcpy(b.x[i], __builtin_assume_aligned(X + ((at0 + (uint32_t)ro[i]) << 3), 8), sizeof(b.x[i]));
        } else {
#pragma unroll
            for (int i = 0; i < kBlk; ++i)
#pragma unroll
                for (int k = 0; k < kBlk; ++k)
                    b.x[i][k] = *reinterpret_cast<const double *>(X + ((at0 + (uint32_t)(ro[i] + min(k, last_col) * s_col)) << 3));
        }
    };
    __syncthreads();
    int cur = a.o_q, nxt = a.o_q + a.T * a.pq;
    for (int it = 0; it < a.iters; ++it) {
        for (int c0 = 0; c0 < a.T; c0 += c.chunk) {
            const int c1 = min(c0 + c.chunk, a.T);
            for (int t = c0 + t0; on && t < c1; t += c.steps) {
                const int q = cur + t * a.pq, p = a.o_p + (t - c0) * a.pl;
                const uint32_t at0 = (a.ll ? (uint32_t)t * (uint32_t)a.llpc
                                           : (uint32_t)obs[t * a.M + m_obs] * (uint32_t)slice) +
                                     (uint32_t)first;
                double wa[kBlk], wb[kBlk], z[kBlk], v[kBlk];
#pragma unroll
                for (int i = 0; i < kBlk; ++i) {
                    wa[i] = smem[q + q_row + i];
                    wb[i] = smem[q + q_col + i];
                    wb[i] = i < skip ? 0.0 : wb[i];
                    z[i] = v[i] = 0.0;
                }
                const int total = o_count * n2;
                int o = 0, o2 = 0;        // outer states of the block at hand
                int op = 0, op2 = 0;      // of the next one to load
                auto next = [&](Block &b) {
                    load(b, at0 + (uint32_t)(op * sp + op2 * s2));
                    if (++op2 == n2) {
                        op2 = 0;
                        ++op;
                    }
                };
                double yp = 0.0;          // share of the outer state, over the second one's
                auto work = [&](const Block &b) {
                    const double w2 = smem[q + q_2 + o2], wp = smem[q + q_p + o], w = w2 * wp;
                    double y = 0.0;
#pragma unroll
                    for (int i = 0; i < kBlk; ++i) {
                        const double wo = wa[i] * w;
                        double r = 0.0;
#pragma unroll
                        for (int k = 0; k < kBlk; ++k) {
                            r = fma(b.x[i][k], wb[k], r);
                            v[k] = fma(wo, b.x[i][k], v[k]);
                        }
                        y = fma(wa[i], r, y);
                        z[i] = fma(w, r, z[i]);
                    }
                    yp = fma(y, w2, yp);
                    if (share_2) {
                        const int l = p + l_2 + o2 * pitch_2;
                        smem[l] = o ? fma(y, wp, smem[l]) : y * wp;
                    }
                    if (++o2 == n2) {
                        smem[p + l_p + o * pitch_p] = yp;
                        yp = 0.0;
                        o2 = 0;
                        ++o;
                    }
                };
                Block b0, b1;
                next(b0);
                for (int k = 0; k < total; k += 2) {
                    if (k + 1 < total) next(b1);
                    work(b0);
                    if (k + 2 < total) next(b0);
                    if (k + 1 < total) work(b1);
                }
#pragma unroll
                for (int i = 0; i < kBlk; ++i) {
                    smem[p + l_row + i * pitch_row] = z[i];
                    if (i >= skip) smem[p + l_col + i * pitch_col] = v[i];
                }
            }
            __syncthreads();
            // the chunk's messages, four lanes to a line (a lane alone would
            // wait for every eighth of its values)
            const int sub = (int)threadIdx.x & 3;
            for (int i = (int)threadIdx.x >> 2; i < (c1 - c0) * a.ntot; i += (int)blockDim.x >> 2) {
                const int t = c0 + i / a.ntot, j = i - (t - c0) * a.ntot;
                int n = 0, line = 0, at = 0;
                for (int f = 0; f < a.F; ++f) {
                    const Fac &fd = a.fac[f];
                    if (j >= fd.qo) {
                        n = fd.len;
                        line = fd.line + (j - fd.qo) * fd.pitch;
                        at = fd.po + j - fd.qo;
                    }
                }
                const double *l = smem + a.o_p + (t - c0) * a.pl + line;
                double sum = 0.0;
                int k = 4 * sub;
                for (; k + 16 < n; k += 32) {
                    const Four f(l + k), g(l + k + 16);
                    sum += f.sum() + g.sum();
                }
                if (k < n) sum += Four(l + k).sum();
                sum += __shfl_xor(sum, 1, 64);
                sum += __shfl_xor(sum, 2, 64);
                if (sub == 0) smem[c.o_l + t * a.pq + at] = sum;
            }
            __syncthreads();
        }
        for (int u = wave; u < units; u += waves) {
            double shift;
            State st = get_role(roles, u * 64 + lane, shift);
            st.here();
            const double lam = smem[c.o_l + st.t() * a.pq + st.po() + st.s()];
            update_state<ALGO, BT>(a, smem, tab, st, agent, u, slots, cur, nxt, it + 1 == a.iters, lam, shift);
            roles[3 * (u * 64 + lane) + 2].y = __float_as_int((float)shift);
        }
        __syncthreads();
        const int tmp = cur;
        cur = nxt;
        nxt = tmp;
    }
}

const void *vmp_streamed(bool flip);
const void *mmp_streamed(bool flip);

}  // namespace res
}  // namespace bi
