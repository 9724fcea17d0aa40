// HIP kernels of libbcinc for gfx950 (64-lane wavefronts).
//
// Update pipeline for a batch of jobs (one update on each of several graphs):
//   k_prep        affected sources A and Alg 4 scalars (Eq.6, Eq.7); row v''
//                 of the Out phase (Alg 4 on the reverse graph) and the
//                 candidate targets; E* (by head) plus the updated arcs (YC)
//   k_rows        the affected sources' changed targets (Lemma 2 / Lemma 4)
//   k_source      per affected source: old and new partial dependencies over
//                 its changed targets, BC difference (k_source_wide and
//                 k_wide_apply: sources with many)
//   k_es_*        E*' = arcs of YC whose weight equals their new distance, and
//                 BC += difference (compensated), counters reset
// Static pass (initial state and full recompute, Alg 7):
//   k_sssp        distances of every source (near/far search in LDS)
//   k_es_*        E* = arcs with w(a,b) = d(a,b), by head (XC)
//   k_static      per source: path counts in DAG order, dependencies, BC
#include <type_traits>

#include "bc_device.h"

namespace bcinc {

// ------------------------------------------------------------ arithmetic ---

__device__ __forceinline__ uint64_t mul_chk(uint64_t a, uint64_t b, bool &ovf) {
    ovf |= (__umul64hi(a, b) != 0);
    return a * b;
}

__device__ __forceinline__ uint64_t add_chk(uint64_t a, uint64_t b, bool &ovf) {
    uint64_t r = a + b;
    ovf |= (r < a);
    return r;
}

// Lemma 4 (In phase) for one pair (s,t), with D(s,t) = d'(s,v) + d(v,t):
// case 1 keeps (d, sigma); case 2 adds sigma-hat'_sv * sigma_vt when
// d'(s,v) = d(s,v); case 3 adds sigma'_sv * sigma_vt when d'(s,v) < d(s,v);
// case 4 replaces both.  The arc update is the special case E_i = {(u,v)}:
// it reproduces the three cases of Lemma 2.  For t = v it returns Alg 4's
// d'(s,v), sigma'_sv.  An unreachable pair (d0 = INF32) with a finite c is
// always taken, so that a c of 2^31-1 or more reaches the caller's distance
// overflow check.
__device__ __forceinline__ bool in_rule(int32_t d0, int32_t dv, int32_t dvt, int64_t &c) {
    if (dv == INF32 || dvt == INF32) return false;
    c = (int64_t)dv + (int64_t)dvt;
    return c <= (int64_t)d0 || d0 == INF32;
}

// A graph whose E* outgrew its buffers is dead until reloaded: every kernel
// that walks E* row pointers skips it, so no access can leave the buffers.
__device__ __forceinline__ bool job_dead(const UpdateJob &J) {
    return (*(volatile int32_t *)&J.g.ctl->status & ST_ESTAR_CAP) != 0;
}

// A graph with any sticky error holds no valid state until it is recomputed:
// the update kernels after the scan skip it (the bits only ever get set
// during a step, so a kernel that skips a job is never followed by one that
// runs it).
__device__ __forceinline__ bool job_halted(const UpdateJob &J) {
    return *(volatile int32_t *)&J.g.ctl->status != 0;
}

// Unreachable in the 64-bit sums of the scan kernels: far above every sum of
// two finite 31-bit distances, so a finite candidate never equals it.
constexpr int64_t INF64 = INT64_MAX / 4;

// ------------------------------------------------------------ wave tools ---

__device__ __forceinline__ int lane_id() { return __lane_id(); }

__device__ __forceinline__ uint32_t popc_below(uint64_t mask, int lane) {
    return (uint32_t)__popcll(mask & ((lane == 0) ? 0ull : (~0ull >> (64 - lane))));
}

// Wave-wide inclusive scans by data-parallel moves (one VALU instruction per
// step; a shuffle goes through LDS): shifts by 1, 2, 4 and 8 within rows of 16
// lanes, then the last lane of a row, and of the first two rows, to those above.
template <int CTRL, int ROWS>
__device__ __forceinline__ int32_t dpp_or_zero(const int32_t x) {
    return __builtin_amdgcn_update_dpp(0, x, CTRL, ROWS, 0xf, false);
}
__device__ __forceinline__ int32_t wave_incl_add(int32_t x) {
    x += dpp_or_zero<0x111, 0xf>(x);
    x += dpp_or_zero<0x112, 0xf>(x);
    x += dpp_or_zero<0x114, 0xf>(x);
    x += dpp_or_zero<0x118, 0xf>(x);
    x += dpp_or_zero<0x142, 0xa>(x);
    x += dpp_or_zero<0x143, 0xc>(x);
    return x;
}
// of values >= 0
__device__ __forceinline__ int32_t wave_incl_max(int32_t x) {
    x = max(x, dpp_or_zero<0x111, 0xf>(x));
    x = max(x, dpp_or_zero<0x112, 0xf>(x));
    x = max(x, dpp_or_zero<0x114, 0xf>(x));
    x = max(x, dpp_or_zero<0x118, 0xf>(x));
    x = max(x, dpp_or_zero<0x142, 0xa>(x));
    x = max(x, dpp_or_zero<0x143, 0xc>(x));
    return x;
}

// Block-wide exclusive scan of one int per thread (blockDim.x <= 1024).
__device__ int32_t block_excl_scan(int32_t x, int32_t *sh /* >= 32 */, int32_t &total) {
    const int lane = lane_id(), wid = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
    int32_t incl = x;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        int32_t y = __shfl_up(incl, d, 64);
        if (lane >= d) incl += y;
    }
    if (lane == 63) sh[wid] = incl;
    __syncthreads();
    if (wid == 0) {
        int32_t v = (lane < nw) ? sh[lane] : 0;
        int32_t vi = v;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            int32_t y = __shfl_up(vi, d, 64);
            if (lane >= d) vi += y;
        }
        if (lane < nw) sh[lane] = vi - v;
        if (lane == nw - 1) sh[32] = vi;
    }
    __syncthreads();
    int32_t res = sh[wid] + incl - x;
    total = sh[32];
    __syncthreads();
    return res;
}

// ------------------------------------------------------------ k_prep -------
//
// The first launch of a step: three roles side by side, told apart by
// blockIdx.x (scan, targets, merge), a row of blocks per job.  None needs
// another's output (the few scalars the targets role wants it forms itself),
// and at small sizes a launch costs as much as its work: with the fused tail
// (k_es_place) and the wide kernel left out where no source can be deferred, an
// update takes 5 or 7 launches instead of a copy and 12.  16 updates of a
// 64-vertex graph went from 1.61 to 1.02 ms, 8 vertex updates of 32 edges on a
// complete graph of 2048 from 9.7 to 2.4 (the column reads besides), 64 arc
// updates at n = 4096 from 13.5 to 12.3.

// Alg 4 over E_i for source s (Eq.6 d'(s,v), Eq.7 sigma-hat'_sv, sigma'_sv).
// cur is d'(s,v) in 64 bits with INF64 for unreachable: a candidate of 2^31-1
// or more is compared like any other and is an overflow only if it wins (it is
// then the new finite d'(s,v)).  Distances and counts into column u are read
// from row u where the graph is undirected (the state is symmetric between
// updates): coalesced over the sources, against a cache line per source.
// `one` is the winning in-arc's place + 1 where d'(s,v) fell and one arc
// attains it, else 0.
struct ScanOut {
    int64_t d0, cur;
    uint64_t sig, hat;
    int32_t one;
};

__device__ __forceinline__ ScanOut scan_source(const UpdateJob &J, const int32_t s, bool &ovf_s, bool &ovf_d) {
    const int32_t n = J.g.n, v = J.v, n_in = J.n_in;
    const size_t rs = J.g.directed ? (size_t)n : 1, cs = J.g.directed ? 1 : (size_t)n;
    const int32_t *D = J.g.D + s * rs;
    const uint64_t *S = J.g.S + s * rs;
    const int32_t dsv = D[v * cs];
    ScanOut o;
    o.d0 = dsv == INF32 ? INF64 : (int64_t)dsv;
    o.cur = o.d0;
    o.sig = S[v * cs];
    o.hat = 0;
    constexpr int U = 8;  // column loads in flight
    uint64_t win = 0;     // the arcs that attain cur (at most KMAX)
    for (int k0 = 0; k0 < n_in; k0 += U) {
        int32_t du[U];
#pragma unroll
        for (int k = 0; k < U; ++k) du[k] = k0 + k < n_in ? D[J.in_tail[k0 + k] * cs] : INF32;
#pragma unroll
        for (int k = 0; k < U; ++k) {
            if (du[k] == INF32) continue;
            const int64_t c = (int64_t)du[k] + J.in_w[k0 + k];
            if (c > o.cur) continue;
            win = (c < o.cur ? 0 : win) | 1ull << (k0 + k);
            o.cur = c;
        }
    }
    // the counts of those alone (one round trip each; rarely more than one)
    bool strict = o.cur < o.d0;
    o.one = strict && (win & (win - 1)) == 0 ? __ffsll((unsigned long long)win) : 0;
    for (; win; win &= win - 1) {
        const uint64_t su = S[J.in_tail[__ffsll((unsigned long long)win) - 1] * cs];
        if (strict) {
            o.sig = su;
            strict = false;
        } else {
            o.sig = add_chk(o.sig, su, ovf_s);
            o.hat = add_chk(o.hat, su, ovf_s);
        }
    }
    if (o.cur != INF64 && o.cur >= INF32) {
        // d'(s,v) does not fit the distance matrix: the graph is halted
        // (sticky), s is left out
        ovf_d = true;
        o.cur = o.d0;
        o.hat = 0;
    }
    return o;
}

__device__ __forceinline__ SrcScal scan_scal(const ScanOut &o, const bool aff) {
    SrcScal sc;
    sc.dv = o.cur == INF64 ? INF32 : (int32_t)o.cur;
    sc.flags = (o.cur == o.d0 ? 1 : 0) | (aff ? 2 : 0) | (o.one << 8);
    sc.sv = o.sig;
    sc.hv = o.hat;
    return sc;
}

// Scan role: per source s its Alg 4 scalars, then the affected test.  s
// changes in the In phase iff d'(s,v) < d(s,v) or sigma-hat'_sv > 0 (Lemma 4
// cases 2-4 need one of them; for an arc update this is Lemma 2 case 1 failing
// at t = v).  s changes in the Out phase iff d'(s,v) + w'(v,x) <= d'(s,x) for
// some (v,x) in E_o.  Affected sources are compacted with a wave ballot and one
// atomic per wave.
__device__ __forceinline__ void prep_scan(const UpdateJob &J, const int64_t first, const int64_t stride) {
    const int32_t n = J.g.n, v = J.v, n_out = J.n_out;
    const size_t rs = J.g.directed ? (size_t)n : 1, cs = J.g.directed ? 1 : (size_t)n;
    const int32_t *Dv = J.g.D + (size_t)v * n;
    bool ovf_s = false, ovf_d = false;
    for (int64_t base = first; base < n; base += stride) {
        const int32_t s = (int32_t)(base + threadIdx.x);
        bool aff = false;
        if (s < n) {
            const ScanOut o = scan_source(J, s, ovf_s, ovf_d);
            aff = (o.cur < o.d0) || (o.hat != 0);
            if (!aff && o.cur != INF64) {
                const int32_t *Ds = J.g.D + s * rs;
                constexpr int U = 8;
                for (int k0 = 0; k0 < n_out && !aff; k0 += U) {
                    int32_t dx[U];
#pragma unroll
                    for (int k = 0; k < U; ++k) dx[k] = k0 + k < n_out ? Ds[J.out_head[k0 + k] * cs] : 0;
#pragma unroll
                    for (int k = 0; k < U; ++k) {
                        if (k0 + k >= n_out) continue;
                        int64_t d1 = dx[k] == INF32 ? INF64 : (int64_t)dx[k];
                        const int32_t dvx = Dv[J.out_head[k0 + k]];
                        if (dvx != INF32 && o.cur + dvx < d1) d1 = o.cur + dvx;
                        // a candidate of 2^31-1 or more also marks s: the row
                        // kernel's pair update decides with row v'' whether it
                        // wins, and only then raises the overflow
                        aff |= o.cur + J.out_w[k0 + k] <= d1;
                    }
                }
            }
            J.g.scal[s] = scan_scal(o, aff);
        }
        const uint64_t mask = __ballot(aff);
        if (mask) {
            const int lane = lane_id();
            const int leader = __ffsll((unsigned long long)mask) - 1;
            int32_t b0 = 0;
            if (lane == leader) b0 = atomicAdd(&J.g.ctl->a_count, (int32_t)__popcll(mask));
            b0 = __shfl(b0, leader, 64);
            if (aff) J.g.alist[b0 + popc_below(mask, lane)] = s;
        }
    }
    if (ovf_s) atomicOr(&J.g.ctl->status, ST_SIGMA_OVF);
    if (ovf_d) atomicOr(&J.g.ctl->status, ST_DIST_OVF);
}

// Stored predecessor of a vertex whose DAG in-arcs are those of a and of b.
__device__ __forceinline__ int32_t pred_union(const int32_t a, const int32_t b) {
    return a == PRED_NONE ? b : b == PRED_NONE || a == b ? a : PRED_MULTI;
}

// Targets role: row v'' and the candidate targets of an update, one thread per
// target t.
//
// Row v'' (Section 4, Out phase): with E_o = {(v, x_j)}, Alg 4 on G'_R gives
// d''(v,t) = min(d'(v,t), min_j w'(v,x_j) + d'(x_j,t)) and the counts
// sigma''_vt, sigma-hat''_vt.  The rows x_j of G' are formed on the fly by
// the In-phase rule from the old rows and the scalars of the sources x_j
// (formed here once per workgroup: the scan role writes them in the same
// launch).  The old row v is snapshotted, since the source v itself rewrites
// it during the update.  rvv_pred is the stored-predecessor row of v'': the
// DAG''(v) in-arcs of t are those of DAG(v) where d''(v,t) = d(v,t), and those
// of every DAG(x_j) whose arc attains d''(v,t) ((v,x_j) itself at t = x_j); a
// path from x_j that enters v again attains nothing.
//
// Candidates: a pair (s,t) can change in the In phase only if
// d'(s,v) + d(v,t) <= d(s,t) with d'(s,v) = d(s,u_j) + w'_j for some in-arc,
// and d(s,t) <= d(s,u_j) + d(u_j,t), hence only if w'_j + d(v,t) <= d(u_j,t)
// (for an arc update this is the target set of the tail u).  It can change in
// the Out phase only if row v'' changed at t (d''(v,t) < d'(v,t), or a tie
// with new paths).  The union T is listed once per update, with row v and
// row v'' at t copied next to it, so each affected source scans T instead of
// its whole row when T is short.  For whole-row scans the two tests are kept
// per target as filter rows: f_out = d''(v,t) on Out candidates, INF32
// elsewhere, and f_any = min(f_in, f_out) with f_in = d(v,t) on In
// candidates, INF32 elsewhere.
__device__ __forceinline__ void prep_targets(const UpdateJob &J, const int64_t first, const int64_t stride,
                                             SrcScal *xs) {
    const int32_t n = J.g.n, v = J.v;
    const int32_t *D = J.g.D;
    const uint64_t *S = J.g.S;
    bool ovf_s = false, ovf_d = false;
    for (int j = threadIdx.x; j < J.n_out; j += blockDim.x) {
        bool os = false, od = false;  // raised by the scan role
        xs[j] = scan_scal(scan_source(J, J.out_head[j], os, od), false);
    }
    __syncthreads();
    constexpr int U = 8;  // row loads in flight
    for (int64_t base = first; base < n; base += stride) {
        const int32_t t = (int32_t)(base + threadIdx.x);
        bool cand = false, cand_out = false;
        int32_t dvt = INF32, cur = INF32;
        if (t < n) {
            dvt = D[(size_t)v * n + t];
            if (dvt != INF32) {
                for (int k0 = 0; k0 < J.n_in && !cand; k0 += U) {
                    int32_t dut[U];
#pragma unroll
                    for (int k = 0; k < U; ++k) dut[k] = k0 + k < J.n_in ? D[(size_t)J.in_tail[k0 + k] * n + t] : 0;
#pragma unroll
                    for (int k = 0; k < U; ++k)
                        cand |= k0 + k < J.n_in && (int64_t)J.in_w[k0 + k] + dvt <= (int64_t)dut[k];
                }
            }
            const int32_t f_in = cand ? dvt : INF32;
            cur = dvt;
            if (J.n_out > 0) {
                const uint64_t svt = S[(size_t)v * n + t];
                const int32_t pvt = J.g.pred[(size_t)v * n + t];
                J.g.rv_D[t] = dvt;
                J.g.rv_S[t] = svt;
                // 64-bit sums with INF64 for unreachable, as in scan_source:
                // only a winning candidate of 2^31-1 or more overflows
                int64_t c64 = dvt == INF32 ? INF64 : (int64_t)dvt;
                const int64_t v64 = c64;
                uint64_t sig = svt, hat = 0, win = 0;  // win: the arcs that attain c64
                for (int k0 = 0; k0 < J.n_out; k0 += U) {
                    int32_t dx[U];
#pragma unroll
                    for (int k = 0; k < U; ++k) dx[k] = k0 + k < J.n_out ? D[(size_t)J.out_head[k0 + k] * n + t] : INF32;
#pragma unroll
                    for (int k = 0; k < U; ++k) {
                        if (k0 + k >= J.n_out) continue;
                        int32_t d1 = dx[k];
                        int64_t c;
                        if (in_rule(d1, xs[k0 + k].dv, dvt, c)) {
                            // in_rule takes c only where it is shortest: a
                            // c of 2^31-1 or more is a real overflow of (x,t)
                            if (c >= INF32) ovf_d = true;
                            else d1 = (int32_t)c;
                        }
                        if (d1 == INF32) continue;
                        const int64_t cc = (int64_t)J.out_w[k0 + k] + d1;
                        if (cc > c64) continue;
                        win = (cc < c64 ? 0 : win) | 1ull << (k0 + k);
                        c64 = cc;
                    }
                }
                // sigma'_(x,t) of those alone, by the In rule
                bool strict = c64 < v64;
                int32_t pr = strict ? PRED_NONE : pvt;
                for (; win; win &= win - 1) {
                    const int32_t k = __ffsll((unsigned long long)win) - 1, x = J.out_head[k];
                    const SrcScal sc = xs[k];
                    const int32_t d1 = D[(size_t)x * n + t];
                    const uint64_t sxt = S[(size_t)x * n + t];
                    const int32_t pxt = J.g.pred[(size_t)x * n + t];
                    pr = pred_union(pr, t == x ? v : pxt);
                    int64_t c;
                    uint64_t s1;
                    const bool in = in_rule(d1, sc.dv, dvt, c) && c < INF32;
                    if (in && c < d1) {
                        s1 = mul_chk(sc.sv, svt, ovf_s);
                    } else {
                        s1 = sxt;
                        if (in) s1 = add_chk(s1, mul_chk((sc.flags & 1) ? sc.hv : sc.sv, svt, ovf_s), ovf_s);
                    }
                    if (strict) {
                        sig = s1;
                        strict = false;
                    } else {
                        sig = add_chk(sig, s1, ovf_s);
                        hat = add_chk(hat, s1, ovf_s);
                    }
                }
                if (c64 != INF64 && c64 >= INF32) {
                    // d''(v,t) does not fit: the graph is halted (sticky)
                    ovf_d = true;
                    c64 = INF64;
                    hat = 0;
                }
                cur = c64 == INF64 ? INF32 : (int32_t)c64;
                J.g.rvv_D[t] = cur;
                J.g.rvv_S[t] = sig;
                J.g.rvv_H[t] = hat;
                J.g.rvv_pred[t] = pr;
                cand_out = cur < dvt || hat != 0;
                cand = cand || cand_out;
            }
            const int32_t f_out = cand_out ? cur : INF32;
            J.g.f_out[t] = f_out;
            J.g.f_any[t] = min(f_in, f_out);
        }
        const uint64_t mask = __ballot(cand);
        if (mask) {
            const int lane = lane_id();
            const int leader = __ffsll((unsigned long long)mask) - 1;
            int32_t b0 = 0;
            if (lane == leader) b0 = atomicAdd(&J.g.ctl->t_count, (int32_t)__popcll(mask));
            b0 = __shfl(b0, leader, 64);
            if (cand) {
                const int32_t pos = b0 + (int32_t)popc_below(mask, lane);
                J.g.tlist[pos] = t;
                J.g.tl_rvD[pos] = dvt;
                J.g.tl_rvvD[pos] = cur;
            }
        }
    }
    if (ovf_s) atomicOr(&J.g.ctl->status, ST_SIGMA_OVF);
    if (ovf_d) atomicOr(&J.g.ctl->status, ST_DIST_OVF);
}

// Merge role: YC keeps every XC arc and adds the update's arcs behind their
// head's XC arcs, so head h's segment starts before(h) entries later than in
// XC, before(h) = the update arcs into heads below h; every arc is placed
// directly.  An XC arc that the update lowers stays beside its new copy: its
// old weight satisfies Eq.1 for no source, and the filter drops it.
__device__ __forceinline__ void prep_merge(const UpdateJob &J, const int64_t gid, const int64_t nthreads) {
    if (job_halted(J)) return;
    const int32_t n = J.g.n, nu = J.n_u;
    const int32_t *__restrict__ ptr = J.g.xc_ptr;
    const int32_t m = ptr[n];
    const int64_t total = (int64_t)m + nu;
    if (total > J.g.es_cap) {
        if (gid == 0) atomicOr(&J.g.ctl->status, ST_ESTAR_CAP);
        return;
    }
    if (gid == 0) J.g.ctl->esc_m_tmp = (int32_t)total;
    for (int64_t h = gid; h <= n; h += nthreads) {
        int32_t before = 0;
        for (int k = 0; k < nu; ++k) before += J.u_head[k] < h;
        J.g.yc_ptr[h] = ptr[h] + before;
    }
    for (int64_t i = gid; i < m; i += nthreads) {
        const int32_t h = J.g.xc_dst[i];
        int32_t before = 0;
        for (int k = 0; k < nu; ++k) before += J.u_head[k] < h;
        const int64_t o = i + before;
        J.g.yc_src[o] = J.g.xc_src[i];
        J.g.yc_dst[o] = h;
        J.g.yc_w[o] = J.g.xc_w[i];
    }
    for (int64_t k = gid; k < nu; k += nthreads) {
        const int32_t h = J.u_head[k];
        int32_t before = 0;
        for (int q = 0; q < nu; ++q) before += J.u_head[q] < h || (J.u_head[q] == h && q < k);
        const int64_t o = (int64_t)ptr[h + 1] + before;
        J.g.yc_src[o] = J.u_tail[k];
        J.g.yc_dst[o] = h;
        J.g.yc_w[o] = J.u_w[k];
    }
}

// `elem` blocks of the scan role, as many of the targets role, the others
// merge.
__device__ __forceinline__ void prep_roles(const UpdateJob &J, const int32_t elem, SrcScal *xs) {
    const int32_t b = (int32_t)blockIdx.x;
    if (b < elem) {
        prep_scan(J, (int64_t)b * blockDim.x, (int64_t)elem * blockDim.x);
    } else if (b < 2 * elem) {
        prep_targets(J, (int64_t)(b - elem) * blockDim.x, (int64_t)elem * blockDim.x, xs);
    } else {
        prep_merge(J, (int64_t)(b - 2 * elem) * blockDim.x + threadIdx.x, (int64_t)((int32_t)gridDim.x - 2 * elem) * blockDim.x);
    }
}

__global__ void __launch_bounds__(256) k_prep(const UpdateJob *__restrict__ jobs, const int32_t *__restrict__ njobs_p,
                                              int32_t elem) {
    __shared__ SrcScal xs[KMAX];
    const int njobs = *njobs_p;
    for (int j = blockIdx.y; j < njobs; j += gridDim.y) {  // a row of blocks per job
        prep_roles(jobs[j], elem, xs);
        __syncthreads();
    }
}

// The same for a step of one job that is not captured: the job comes with the
// launch, and block 0 stages it for the kernels behind.
__global__ void __launch_bounds__(256) k_prep_one(const UpdateJob J, UpdateJob *__restrict__ jobs,
                                                  int32_t *__restrict__ njobs_p, int32_t elem) {
    __shared__ SrcScal xs[KMAX];
    static_assert(sizeof(UpdateJob) % 4 == 0 && sizeof(UpdateJob) < 4000, "a job fits the kernel arguments");
    if (blockIdx.x == gridDim.x - 1) {
        for (uint32_t i = threadIdx.x; i < sizeof(UpdateJob) / 4; i += blockDim.x)
            ((uint32_t *)jobs)[i] = ((const uint32_t *)&J)[i];
        if (threadIdx.x == 0) *njobs_p = 1;
    }
    prep_roles(J, elem, xs);
}

// ------------------------------------------------------------ E* rebuild ---
//
// E* is kept as segments of arcs keyed by head (XC; the static pass and the
// updates walk DAG predecessors).  A wave-per-segment compaction of the arcs
// by head builds it in the static pass (k_es_count / k_es_scan /
// k_es_scatter); an update's merge (k_prep) and filter (k_es_keep / k_es_place) are
// arc-parallel.  An arc whose
// weight exceeds its distance lies on no
// shortest path and is dropped; distances only decrease under incremental
// updates, so E*' is contained in E* plus the updated arcs (Section 1
// definition of E*; Alg 6 steps 2-4 use the same test w(u,v) = d(u,v)).

__device__ __forceinline__ bool es_keep(const UpdateJob &J, int32_t a, int32_t b, int32_t w) {
    return J.g.D[(size_t)a * J.g.n + b] == w;
}

__global__ void __launch_bounds__(256) k_es_count(const UpdateJob *__restrict__ jobs) {
    const int lane = lane_id();
    const int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const int64_t nwaves = ((int64_t)gridDim.x * blockDim.x) >> 6;
    const UpdateJob &J = jobs[0];
    const int32_t n = J.g.n;
    for (int64_t key = wave; key < n; key += nwaves) {
        const int32_t p0 = J.g.arcin_ptr[key], p1 = J.g.arcin_ptr[key + 1];
        int32_t cnt = 0;
        for (int32_t base = p0; base < p1; base += 64) {
            const int32_t i = base + lane;
            const bool keep = i < p1 && es_keep(J, J.g.arcin[i].v, (int32_t)key, J.g.arcin[i].w);
            cnt += (int32_t)__popcll(__ballot(keep));
        }
        if (lane == 0) J.g.es_cnt[key] = cnt;
    }
}

// One workgroup: exclusive scan of the per-segment counts into the
// output segment pointers; the total goes to the control block.  A total
// above the capacity sets the sticky E* capacity error and the scatter is
// skipped.
__global__ void __launch_bounds__(1024) k_es_scan(const UpdateJob *__restrict__ jobs) {
    __shared__ int32_t sh[40];
    const UpdateJob &J = jobs[0];
    int32_t *const optr = J.g.xc_ptr;
    const int32_t n = J.g.n;
    const int32_t *cnt = J.g.es_cnt;
    // tiles of 8 consecutive counts per thread (two 16-byte loads), one block
    // scan per tile, a running carry between tiles
    int32_t carry = 0;
    for (int32_t base = 0; base < n; base += 8 * (int32_t)blockDim.x) {
        const int32_t i0 = base + 8 * (int32_t)threadIdx.x;
        int32_t v[8];
        const bool whole = i0 + 8 <= n;
        if (whole) {
            const int4 a = *(const int4 *)(cnt + i0), b = *(const int4 *)(cnt + i0 + 4);
            v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
            v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
        } else {
#pragma unroll
            for (int k = 0; k < 8; ++k) v[k] = (i0 + k < n) ? cnt[i0 + k] : 0;
        }
        int32_t local = 0;
#pragma unroll
        for (int k = 0; k < 8; ++k) local += v[k];
        int32_t total;
        int32_t off = block_excl_scan(local, sh, total) + carry;
        int32_t o[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            o[k] = off;
            off += v[k];
        }
        if (whole) {
            *(int4 *)(optr + i0) = make_int4(o[0], o[1], o[2], o[3]);
            *(int4 *)(optr + i0 + 4) = make_int4(o[4], o[5], o[6], o[7]);
        } else {
#pragma unroll
            for (int k = 0; k < 8; ++k)
                if (i0 + k < n) optr[i0 + k] = o[k];
        }
        carry += total;
    }
    if (threadIdx.x == 0) {
        const int32_t total = carry;
        optr[n] = total;
        if ((int64_t)total > J.g.es_cap) {
            atomicOr(&J.g.ctl->status, ST_ESTAR_CAP);
        } else {
            J.g.ctl->esc_m = total;
        }
    }
}

__global__ void __launch_bounds__(256) k_es_scatter(const UpdateJob *__restrict__ jobs) {
    const int lane = lane_id();
    const int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const int64_t nwaves = ((int64_t)gridDim.x * blockDim.x) >> 6;
    const UpdateJob &J = jobs[0];
    const int32_t n = J.g.n;
    if ((int64_t)J.g.xc_ptr[n] > J.g.es_cap) return;
    for (int64_t key = wave; key < n; key += nwaves) {
        const int32_t p0 = J.g.arcin_ptr[key], p1 = J.g.arcin_ptr[key + 1];
        int32_t out = J.g.xc_ptr[key];
        for (int32_t base = p0; base < p1; base += 64) {
            const int32_t i = base + lane;
            int32_t a = 0, w = 0;
            bool keep = false;
            if (i < p1) {
                a = J.g.arcin[i].v;
                w = J.g.arcin[i].w;
                keep = es_keep(J, a, (int32_t)key, w);
            }
            const uint64_t mask = __ballot(keep);
            if (keep) {
                const int32_t o = out + (int32_t)popc_below(mask, lane);
                J.g.xc_src[o] = a;
                J.g.xc_dst[o] = (int32_t)key;
                J.g.xc_w[o] = w;
            }
            out += (int32_t)__popcll(mask);
        }
    }
}

// E* filter, arc-parallel: XC = the arcs of YC with w = d'(a,b), in YC
// order.  One gather per arc sets a bit of a 64-bit keep mask per 64 arcs;
// then every kept arc and every head's segment start is placed directly
// (k_es_place; the masks' popcounts are summed by each of its workgroups for
// itself, or scanned before by one workgroup per job where an E* may hold more
// than ES_LONG arcs: at that size the last workgroups read 128 KiB of masks, 512
// bytes per thread).
__device__ __forceinline__ uint64_t *es_mask(const UpdateJob &J) { return (uint64_t *)J.g.x_src; }
__device__ __forceinline__ int32_t *es_wpre(const UpdateJob &J) { return J.g.x_dst; }

__global__ void __launch_bounds__(256) k_es_keep(const UpdateJob *__restrict__ jobs, const int32_t *__restrict__ njobs_p) {
    const int njobs = *njobs_p;
    const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t nthreads = (int64_t)gridDim.x * blockDim.x;
    for (int j = blockIdx.y; j < njobs; j += gridDim.y) {  // a row of blocks per job
        const UpdateJob &J = jobs[j];
        if (job_halted(J)) continue;
        const int32_t n = J.g.n;
        const int64_t m = J.g.yc_ptr[n];
        const int64_t m64 = (m + 63) & ~(int64_t)63;
        uint64_t *const mask = es_mask(J);
        // a wave covers 64 consecutive arcs (the stride is a multiple of 64).
        // A tail outside the affected sources kept its row, so an arc of XC
        // (the front of its head's YC segment: XC's pointers still hold the
        // previous E*) stays without a test; the update's arcs, and the old
        // copy of a lowered arc (whose tail's row did change), are tested.
        for (int64_t i = gid; i < m64; i += nthreads) {
            bool keep = false;
            if (i < m) {
                const int32_t a = J.g.yc_src[i], b = J.g.yc_dst[i];
                const bool affected = (J.g.scal[a].flags & 2) != 0;
                const bool from_xc = i - J.g.yc_ptr[b] < J.g.xc_ptr[b + 1] - J.g.xc_ptr[b];
                keep = (!affected && from_xc) || J.g.D[(size_t)a * n + b] == J.g.yc_w[i];
            }
            const uint64_t word = __ballot(keep);
            if (lane_id() == 0) mask[i >> 6] = word;
        }
    }
}

__global__ void __launch_bounds__(1024) k_es_wscan(const UpdateJob *__restrict__ jobs, const int32_t *__restrict__ njobs_p) {
    __shared__ int32_t sh[40];
    const int j = blockIdx.x;
    if (j >= *njobs_p) return;
    const UpdateJob &J = jobs[j];
    if (job_halted(J)) return;
    const int64_t m = J.g.yc_ptr[J.g.n];
    const int32_t words = (int32_t)((m + 63) >> 6);
    const uint64_t *const mask = es_mask(J);
    int32_t *const wpre = es_wpre(J);
    int32_t carry = 0;
    for (int32_t base = 0; base < words; base += 4 * (int32_t)blockDim.x) {
        const int32_t w0 = base + 4 * (int32_t)threadIdx.x;
        int32_t c[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) c[k] = w0 + k < words ? __popcll(mask[w0 + k]) : 0;
        int32_t total;
        int32_t off = block_excl_scan(c[0] + c[1] + c[2] + c[3], sh, total) + carry;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (w0 + k < words) wpre[w0 + k] = off;
            off += c[k];
        }
        carry += total;
    }
    if (threadIdx.x == 0) {
        wpre[words] = carry;
        J.g.ctl->esc_m = carry;
    }
}

// The last launch of a step: the kept arcs of YC and the segment starts are
// placed in XC (PLACE arcs per workgroup at a time; the kept arcs before them
// are counted from the masks, or come from k_es_wscan where the masks are
// long), the BC difference is folded in (commit_job) and the counters go back
// to zero.  The first arc of a segment places the starts of its head and of
// the empty heads before it; long runs of empty heads are shared by the
// workgroup.  What bounds it is the chain of dependent reads of one chunk:
// searching the heads of a chunk of 2048 and reading arc by arc took 15.0 us at
// n = 4096 and 19.6 us at n = 32768, this takes 6.9 and 12.4 us.
constexpr int32_t PLACE = 1024;  // four arcs per thread, all loads out at once
constexpr int RUNS = 64;       // runs of more than RUN_LONG empty heads per chunk
constexpr int RUN_LONG = 16;

__device__ __forceinline__ void commit_job(const UpdateJob &J, const StepPool &pool, const bool replace);

__global__ void __launch_bounds__(256) k_es_place(const UpdateJob *__restrict__ jobs, const int32_t *__restrict__ njobs_p,
                                                  int32_t scanned, StepPool pool) {
    __shared__ int32_t sh[40];
    __shared__ int32_t pre[PLACE / 64 + 1];
    __shared__ uint64_t word[PLACE / 64];
    __shared__ int32_t runs, run_from[RUNS], run_to[RUNS], run_start[RUNS];
    const int njobs = *njobs_p;
    const int tid = threadIdx.x;
    for (int j = blockIdx.y; j < njobs; j += gridDim.y) {  // a row of blocks per job
        const UpdateJob &J = jobs[j];
        // (the flag is read once per workgroup: a job is halted before this launch)
        if (!job_halted(J)) {
            const int32_t n = J.g.n, m = J.g.yc_ptr[n];
            const uint64_t *const mask = es_mask(J);
            for (int64_t c0 = (int64_t)blockIdx.x * PLACE; c0 <= m; c0 += (int64_t)gridDim.x * PLACE) {
                const int32_t w0 = (int32_t)(c0 >> 6), words = (m + 63) >> 6;
                const int32_t c1 = (int32_t)min((int64_t)m, c0 + PLACE);
                const bool last = c0 + PLACE > m;
                int32_t av[PLACE / 256], hv[PLACE / 256], pv[PLACE / 256], wv[PLACE / 256];
#pragma unroll
                for (int k = 0; k < PLACE / 256; ++k) {
                    const int32_t i = (int32_t)c0 + tid + 256 * k;
                    hv[k] = pv[k] = -1;
                    if (i < c1) {
                        hv[k] = J.g.yc_dst[i];
                        if (i > 0) pv[k] = J.g.yc_dst[i - 1];
                        av[k] = J.g.yc_src[i];
                        wv[k] = J.g.yc_w[i];
                    }
                }
                // kept arcs before the chunk, then before each of its words
                int32_t kept = 0, base;
                if (!scanned)
                    for (int32_t w = tid; w < w0; w += blockDim.x) kept += __popcll(mask[w]);
                (void)block_excl_scan(kept, sh, base);
                if (scanned) base = es_wpre(J)[w0];
                if (tid < 64) {
                    const uint64_t x = tid < PLACE / 64 && w0 + tid < words ? mask[w0 + tid] : 0ull;
                    int32_t incl = __popcll(x);
#pragma unroll
                    for (int d = 1; d < 64; d <<= 1) {
                        const int32_t y = __shfl_up(incl, d, 64);
                        if (tid >= d) incl += y;
                    }
                    if (tid < PLACE / 64) {
                        word[tid] = x;
                        pre[tid + 1] = base + incl;
                    }
                    if (tid == 0) {
                        pre[0] = base;
                        runs = 0;
                    }
                }
                __syncthreads();
                auto before = [&](const int32_t p) {
                    const int32_t w = (p >> 6) - w0;
                    const int r = p & 63;
                    return pre[w] + (r ? (int32_t)__popcll(word[w] & ((1ull << r) - 1)) : 0);
                };
                // heads from .. to (inclusive) start at `start`
                auto starts = [&](const int32_t from, const int32_t to, const int32_t start) {
                    if (to - from >= RUN_LONG) {
                        const int32_t r = atomicAdd(&runs, 1);
                        if (r < RUNS) {
                            run_from[r] = from;
                            run_to[r] = to;
                            run_start[r] = start;
                            return;
                        }
                    }
                    for (int32_t h = from; h <= to; ++h) J.g.xc_ptr[h] = start;
                };
#pragma unroll
                for (int k = 0; k < PLACE / 256; ++k) {
                    const int32_t i = (int32_t)c0 + tid + 256 * k;
                    if (i >= c1) continue;
                    const bool keep = (word[(i >> 6) - w0] >> (i & 63)) & 1;
                    if (!keep && hv[k] == pv[k]) continue;
                    const int32_t o = before(i);
                    if (keep) {
                        J.g.xc_src[o] = av[k];
                        J.g.xc_dst[o] = hv[k];
                        J.g.xc_w[o] = wv[k];
                    }
                    if (hv[k] != pv[k]) starts(pv[k] + 1, hv[k], o);
                }
                if (last && tid == 0) {
                    // the heads past the last arc, and the end of E*
                    const int32_t total = before(m);
                    starts(m > 0 ? J.g.yc_dst[m - 1] + 1 : 0, n, total);
                    J.g.ctl->esc_m = total;
                }
                __syncthreads();
                for (int32_t r = 0; r < min(runs, RUNS); ++r)
                    for (int32_t h = run_from[r] + tid; h <= run_to[r]; h += blockDim.x) J.g.xc_ptr[h] = run_start[r];
                __syncthreads();
            }
        }
        commit_job(J, pool, false);
    }
}

// ------------------------------------------------------------ DAG passes ---

struct BlockShared {
    int32_t head, tail, next, nlev;
    int32_t item, seg, source, role;
    int32_t wl_total, wl_seg, wl_lo, wl_hi, wl_first;  // WorkList
    int32_t nb, nf;
    int32_t ovf, progress;
    int32_t nk, kpos;
    int32_t scan[40];
    unsigned long long counter;
};

// A workgroup's slot.  Slots of the DAG kernel have no B list and no new
// row (null pointers) and an arc record of n arcs; wide-kernel slots have
// all of them, with a record of KARC_PER_VERTEX * n arcs.
struct USlot {
    int32_t *outdeg, *sub, *q1, *q2, *bl_t, *bl_d;
    double *acc;
    uint64_t *bl_s;
    int32_t *kcnt, *kend, *ka, *kb, *kr, *dnew;
    uint64_t *snew;
    int64_t kcap;
};

__device__ __forceinline__ USlot uslot_at(char *base, int32_t n) {
    const UpdateLayout L = update_layout(n);
    USlot u;
    u.outdeg = (int32_t *)(base + L.outdeg);
    u.acc = (double *)(base + L.acc);
    u.sub = (int32_t *)(base + L.sub);
    u.q1 = (int32_t *)(base + L.q1);
    u.q2 = (int32_t *)(base + L.q2);
    u.bl_t = u.bl_d = nullptr;
    u.bl_s = nullptr;
    u.kcnt = (int32_t *)(base + L.kcnt);
    u.kend = (int32_t *)(base + L.kend);
    u.ka = (int32_t *)(base + L.ka);
    u.kb = (int32_t *)(base + L.kb);
    u.kr = (int32_t *)(base + L.kr);
    u.dnew = nullptr;
    u.snew = nullptr;
    u.kcap = L.kcap;
    return u;
}

__device__ __forceinline__ USlot wslot_at(char *base, int32_t n) {
    const WideLayout L = wide_layout(n);
    USlot u;
    u.outdeg = (int32_t *)(base + L.outdeg);
    u.acc = (double *)(base + L.acc);
    u.sub = (int32_t *)(base + L.sub);
    u.q1 = (int32_t *)(base + L.q1);
    u.q2 = (int32_t *)(base + L.q2);
    u.bl_t = (int32_t *)(base + L.bl_t);
    u.bl_d = (int32_t *)(base + L.bl_d);
    u.bl_s = (uint64_t *)(base + L.bl_s);
    u.kcnt = (int32_t *)(base + L.kcnt);
    u.kend = (int32_t *)(base + L.kend);
    u.ka = (int32_t *)(base + L.ka);
    u.kb = (int32_t *)(base + L.kb);
    u.kr = (int32_t *)(base + L.kr);
    u.dnew = (int32_t *)(base + L.dnew);
    u.snew = (uint64_t *)(base + L.snew);
    u.kcap = L.kcap;
    return u;
}

// A row copy with U loads in flight per lane (a plain loop waits for each
// load before the next one).
template <int U, typename T>
__device__ __forceinline__ void copy_row(T *dst, const T *__restrict__ src, const int32_t n) {
    const int tid = threadIdx.x, bs = blockDim.x;
    for (int32_t t0 = tid; t0 < n; t0 += U * bs) {
        T v[U];
#pragma unroll
        for (int k = 0; k < U; ++k) v[k] = t0 + k * bs < n ? src[t0 + k * bs] : T(0);
#pragma unroll
        for (int k = 0; k < U; ++k)
            if (t0 + k * bs < n) dst[t0 + k * bs] = v[k];
    }
}

// A value other lanes of the workgroup change by atomics: in global memory
// those act in L2, so it is read there too.
template <bool LDS, typename T>
__device__ __forceinline__ T shared_value(const T *p) {
    if (LDS) return *p;
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Arc-parallel expansion helpers: the in-arcs of a list of vertices are
// flattened with a block-wide scan of their in-degrees; each lane takes XU
// consecutive arcs and issues their loads together.  Two keep the DAG kernel
// within its 96 registers without spills (four cost six spilled registers
// and were slower).
constexpr int XU = 2;

struct ExpandShared {
    int32_t *off, *vtx, *beg, *dx;
    double *val;
};

// Bytes of expansion arrays per thread (val, off, vtx, beg, dx).
constexpr size_t XB = 24;

// Dynamic LDS of the per-source kernels: the staged row (4 * lds_cap bytes),
// the expansion arrays (XB bytes per thread), then the small-DAG table.
__device__ __forceinline__ ExpandShared expand_at(char *dyn, int32_t lds_cap) {
    ExpandShared es;
    char *p = dyn + align256((size_t)lds_cap * 4);
    es.val = (double *)p;
    es.off = (int32_t *)(p + 8 * blockDim.x);
    es.vtx = es.off + blockDim.x;
    es.beg = es.vtx + blockDim.x;
    es.dx = es.beg + blockDim.x;
    return es;
}

__device__ __forceinline__ int32_t find_owner(const ExpandShared &es, int32_t nv, int32_t j) {
    int32_t lo = 0, hi = nv - 1;
    while (lo < hi) {
        const int32_t mid = (lo + hi + 1) >> 1;
        if (es.off[mid] <= j) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// Arcs jb .. jb+XU-1 of an expansion chunk of nv vertices and total arcs:
// for each, the owning chunk entry iv and the arc id ev (ok false past the
// end).  One binary search, then a forward walk (the arcs are consecutive).
template <int U>
__device__ __forceinline__ void chunk_arcs(const ExpandShared &es, const int32_t nv, const int32_t total,
                                           const int32_t jb, int32_t (&iv)[U], int32_t (&ev)[U], bool (&ok)[U]) {
    int32_t i = find_owner(es, nv, jb);
#pragma unroll
    for (int k = 0; k < U; ++k) {
        const int32_t j = jb + k;
        ok[k] = j < total;
        iv[k] = 0;
        ev[k] = 0;
        if (ok[k]) {
            while (i + 1 < nv && es.off[i + 1] <= j) ++i;
            iv[k] = i;
            ev[k] = es.beg[i] + (j - es.off[i]);
        }
    }
}

// The accumulation of a restricted pass over a recorded sub-DAG of nsub
// vertices and nk arcs in LDS: the vertices are renumbered in the order they
// were found, the arcs grouped by head, and Kahn runs as in dual_kahn (the
// lane whose push completes a vertex carries on with it).  The slot's arrays
// are cleared for the next use as they are read.  Fits when lds_kahn_bytes
// does.  In the slot a round of the accumulation is two or three L2 round
// trips, and the few heavy sources end an update last: 64 arc updates at n = 4096
// take 11.9 ms this way against 13.6, 16 unit-weight insertions at n = 8191 17.0
// against 17.9.
__host__ __device__ constexpr inline size_t lds_kahn_bytes(const size_t nsub, const size_t nk, const bool counts) {
    return nsub * ((counts ? 8 : 0) + 8 + 4 + 4 + 2) + nk * 2 + 16;
}

__device__ __forceinline__ void kahn_in_lds(const int32_t s, const int32_t nsub, const int32_t nk, const USlot &u,
                                            const uint64_t *__restrict__ Srow, const bool counts, const double sign,
                                            double *out, BlockShared &sh, char *buf) {
    const int tid = threadIdx.x, bs = blockDim.x;
    double *const acc = (double *)buf;
    uint64_t *const sig = (uint64_t *)(acc + nsub);  // with counts
    int32_t *const left = (int32_t *)(sig + (counts ? nsub : 0));  // successors to come, and W_B
    uint32_t *const range = (uint32_t *)(left + nsub);             // end of the in-arcs | their number << 16
    uint16_t *const list = (uint16_t *)(range + nsub), *const tails = list + nsub;
    if (tid == 0) {
        sh.kpos = 0;
        sh.tail = 0;
    }
    __syncthreads();
    for (int32_t i = tid; i < nsub; i += bs) {
        const int32_t x = u.sub[i];
        const int32_t o = u.outdeg[x], c = u.kcnt[x];
        if (counts) sig[i] = Srow[x];
        u.kend[x] = i;
        u.outdeg[x] = 0;
        u.kcnt[x] = 0;
        acc[i] = 0.0;
        left[i] = o & (W_COUNT | W_B);
        const int32_t beg = atomicAdd(&sh.kpos, c);
        range[i] = (uint32_t)beg | (uint32_t)c << 16;  // (the start; the scatter moves it to the end)
        if ((o & W_COUNT) == 0) list[atomicAdd(&sh.tail, 1)] = (uint16_t)i;
    }
    __syncthreads();
    for (int32_t p = tid; p < nk; p += bs) {
        const int32_t h = u.kend[u.kb[p]], a = u.kend[u.ka[p]];
        tails[atomicAdd(&range[h], 1u) & 0xffffu] = (uint16_t)a;
    }
    __syncthreads();
    int32_t lo = 0, hi = sh.tail;
    __syncthreads();
    while (lo < hi) {
        for (int32_t idx = lo + tid; idx < hi; idx += bs) {
            int32_t x = list[idx];
            for (;;) {
                const uint32_t r = range[x];
                const int32_t e1 = (int32_t)(r & 0xffffu), deg = (int32_t)(r >> 16);
                double c = ((left[x] & W_B) ? 1.0 : 0.0) + acc[x];
                // one in-arc: the tail has the vertex's path count
                if (deg > 1) c /= (double)(counts ? sig[x] : Srow[u.sub[x]]);
                int32_t next = -1;
                for (int32_t e = e1 - deg; e < e1; ++e) {
                    const int32_t a = tails[e];
                    const double share = deg > 1 ? c * (double)(counts ? sig[a] : Srow[u.sub[a]]) : c;
                    if (share != 0.0) atomicAdd(&acc[a], share);
                    // release: the share lands before the count drops;
                    // acquire: the last pusher sees every other share
                    const int32_t was = __hip_atomic_fetch_sub(&left[a], 1, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_WORKGROUP);
                    if ((was & W_COUNT) == 1) {
                        if (next < 0) next = a;
                        else list[atomicAdd(&sh.tail, 1)] = (uint16_t)a;
                    }
                }
                if (next < 0) break;
                x = next;
            }
        }
        __syncthreads();
        lo = hi;
        hi = sh.tail;
        __syncthreads();
    }
    for (int32_t i = tid; i < nsub; i += bs) {
        const int32_t x = u.sub[i];
        const double ax = acc[i];
        if (x != s && ax != 0.0) atomicAdd(&out[x], sign * ax);
    }
    __syncthreads();
}

// Partial dependency of source s over a target set B (one workgroup):
//   delta_B(x) = sum_{t in B} delta_st(x)
//              = sum_{w : x in P_s(w)} sigma_sx / sigma_sw * ([w in B] + delta_B(w)),
// Eq.4 with the indicator of B in place of 1.  It is non-zero only on the
// ancestors of B in DAG(s):
//   1. the vertices to visit and their successor counts: either a backward
//      BFS from B over DAG predecessor arcs (E* by head, Eq.1), counting each
//      sub-DAG vertex's successors inside the sub-DAG, or (full) one sweep
//      over all of E* counting every reachable vertex's DAG successors, for
//      large B where the sub-DAG is most of DAG(s) (vertices outside it get
//      delta_B = 0 and change nothing); with OUT_ROW, in a slot with an arc
//      record, it also keeps the DAG(s) arcs it finds, grouped by head,
//   2. Kahn from the sinks (a reverse topological order, which serves the
//      accumulation, Section 2.1): each vertex pushes its term to its
//      predecessors once all its successors have pushed to it, over the
//      recorded arcs when there are any, else over its E* in-arcs with the
//      Eq.1 test.
// Targets whose d(s,t) and sigma_st do not change keep the same set of
// shortest paths, so delta_st is unchanged for them and the BC difference of
// source s is delta'_B - delta_B with B the changed targets (Alg 3 re-runs
// the whole accumulation; both give the same BC).
// OUT_ROW: delta_B goes to out[x] (introspection); otherwise
// out[x] += sign * delta_B(x) for x != s (out = the BC difference).
// RU: arcs in flight per lane in the arc-parallel loops (the E* sweep
// included); LU: vertices or recorded arcs in flight per lane in the loops
// over the row, the changed targets and the arc record (each lane issues LU
// independent loads or atomics before it uses any).
// kbuf: kbytes of LDS for the accumulation of a sub-DAG that fits (0: none).
template <bool OUT_ROW, int RU, int LU = 1>
__device__ void restricted_pass(const int32_t s, const int32_t n, const int32_t *__restrict__ Drow,
                                const uint64_t *__restrict__ Srow, const int32_t *__restrict__ cptr,
                                const int32_t *__restrict__ csrc, const int32_t *__restrict__ cdst,
                                const int32_t *__restrict__ cw, const int32_t *__restrict__ Bt, const int32_t nB,
                                const bool full, const USlot &u, const double sign, double *out,
                                const int32_t *__restrict__ pred, BlockShared &sh, const ExpandShared &es,
                                char *kbuf = nullptr, const size_t kbytes = 0) {
    const int tid = threadIdx.x, bs = blockDim.x;
    const int32_t kcap = (int32_t)u.kcap;
    if (tid == 0) {
        sh.next = 0;
        sh.tail = 0;
        sh.nk = 0;
        sh.kpos = 0;
    }
    __syncthreads();
    for (int32_t i0 = tid; i0 < nB; i0 += LU * bs) {
        int32_t tv[LU];
#pragma unroll
        for (int k = 0; k < LU; ++k) tv[k] = i0 + k * bs < nB ? Bt[i0 + k * bs] : s;
        bool live[LU];
#pragma unroll
        for (int k = 0; k < LU; ++k) live[k] = tv[k] != s && Drow[tv[k]] != INF32;
#pragma unroll
        for (int k = 0; k < LU; ++k) {
            if (!live[k]) continue;
            if (full) {
                u.outdeg[tv[k]] = W_B;
            } else {
                u.outdeg[tv[k]] = W_VIS | W_B;
                u.sub[atomicAdd(&sh.next, 1)] = tv[k];
            }
        }
    }
    __syncthreads();
    int32_t nsub;
    bool rec = false;  // Kahn walks recorded arcs
    // a sweep records for the dependency row only: in an update it runs where the
    // arcs have outgrown the record already (full_pass)
    const bool sweep_rec = OUT_ROW && kcap > 0;
    if (full) {
        // 1. every DAG(s) arc: one more successor of its tail, and (with an
        //    arc record) the arc itself with one more arc into its head
        const int32_t m = cptr[n];
        for (int32_t e0 = tid; e0 < m; e0 += RU * bs) {
            int32_t av[RU], bv[RU], wv[RU];
#pragma unroll
            for (int k = 0; k < RU; ++k) {
                const int32_t e = e0 + k * bs;
                av[k] = 0;
                bv[k] = 0;
                wv[k] = 0;
                if (e < m) {
                    av[k] = csrc[e];
                    bv[k] = cdst[e];
                    wv[k] = cw[e];
                }
            }
#pragma unroll
            for (int k = 0; k < RU; ++k) {
                if (e0 + k * bs >= m) continue;
                const int32_t da = Drow[av[k]];
                if (da != INF32 && (int64_t)da + wv[k] == (int64_t)Drow[bv[k]]) {
                    atomicAdd(&u.outdeg[av[k]], 1);
                    if (sweep_rec) {
                        const int32_t p = atomicAdd(&sh.nk, 1);
                        if (p < kcap) {
                            u.ka[p] = av[k];
                            u.kb[p] = bv[k];
                            atomicAdd(&u.kcnt[bv[k]], 1);
                        }
                    }
                }
            }
        }
    }
    __syncthreads();
    if (!full) {
        // 1. backward walk from B.  A lane follows a chain of stored
        //    predecessors itself (a vertex's one DAG in-arc, then its tail's,
        //    and so on) until it reaches a vertex already in the sub-DAG, or
        //    s, or a vertex with two or more DAG in-arcs.  Those vertices test
        //    their E* in-arcs by Eq.1 in a round of their own, arc-parallel,
        //    and the tails first found there start the next round's walks.
        //    So the rounds follow the vertices with two or more in-arcs along
        //    a path, not its levels.
        int32_t wlo = 0, whi = sh.next;
        for (;;) {
            if (tid == 0) sh.head = 0;
            __syncthreads();
            for (int32_t idx = wlo + tid; idx < whi; idx += bs) {
                int32_t x = u.sub[idx];
                int32_t p = PRED_MULTI;
                if (pred) p = pred[x];
                for (;;) {
                    if (p < 0) {
                        // s has no DAG in-arc; any other vertex tests E*
                        if (p == PRED_MULTI || x != s) u.q1[atomicAdd(&sh.head, 1)] = x;
                        break;
                    }
                    // p's own predecessor, loaded before the count returns (unused
                    // when p is already in the sub-DAG, as every B vertex is)
                    const int32_t pp = pred[p];
                    const int32_t old = atomicAdd(&u.outdeg[p], 1);
                    if (kcap > 0) {
                        const int32_t k = atomicAdd(&sh.nk, 1);
                        if (k < kcap) {
                            u.ka[k] = p;
                            u.kb[k] = x;
                            atomicAdd(&u.kcnt[x], 1);
                        }
                    }
                    if (old & (W_COUNT | W_VIS)) break;
                    u.sub[atomicAdd(&sh.next, 1)] = p;
                    x = p;
                    p = pp;
                }
            }
            __syncthreads();
            const int32_t nslow = sh.head;
            if (nslow == 0) break;
            wlo = sh.next;
            for (int32_t c = 0; c < nslow; c += bs) {
                const int32_t idx = c + tid;
                int32_t x = 0, b0 = 0, deg = 0, dx = 0;
                if (idx < nslow) {
                    x = u.q1[idx];
                    b0 = cptr[x];
                    deg = cptr[x + 1] - b0;
                    dx = Drow[x];
                }
                int32_t total;
                const int32_t off = block_excl_scan(deg, sh.scan, total);
                es.off[tid] = off;
                es.vtx[tid] = x;
                es.beg[tid] = b0;
                es.dx[tid] = dx;
                __syncthreads();
                const int32_t nv = min(bs, nslow - c);
                for (int32_t jb = tid * RU; jb < total; jb += bs * RU) {
                    int32_t iv[RU], ev[RU], av[RU], wv[RU];
                    bool ok[RU];
                    chunk_arcs(es, nv, total, jb, iv, ev, ok);
#pragma unroll
                    for (int k = 0; k < RU; ++k) {
                        av[k] = ok[k] ? csrc[ev[k]] : 0;
                        wv[k] = ok[k] ? cw[ev[k]] : 0;
                    }
#pragma unroll
                    for (int k = 0; k < RU; ++k) {
                        if (!ok[k]) continue;
                        const int32_t a = av[k];
                        const int32_t da = Drow[a];
                        if (da == INF32 || (int64_t)da + wv[k] != (int64_t)es.dx[iv[k]]) continue;
                        if ((atomicAdd(&u.outdeg[a], 1) & (W_COUNT | W_VIS)) == 0)
                            u.sub[atomicAdd(&sh.next, 1)] = a;
                        if (kcap > 0) {
                            const int32_t p = atomicAdd(&sh.nk, 1);
                            if (p < kcap) {
                                const int32_t x = es.vtx[iv[k]];
                                u.ka[p] = a;
                                u.kb[p] = x;
                                atomicAdd(&u.kcnt[x], 1);
                            }
                        }
                    }
                }
                __syncthreads();
            }
            whi = sh.next;
        }
    }
    if (full) {
        const int32_t nk = sh.nk;
        rec = sweep_rec && nk <= kcap;
        if (rec) {
            // group the arcs by head: each head with arcs gets a range
            // [kend - kcnt, kend); the scatter advances kend from its start
            for (int32_t x0 = tid; x0 < n; x0 += LU * bs) {
                int32_t cv[LU];
#pragma unroll
                for (int k = 0; k < LU; ++k) cv[k] = x0 + k * bs < n ? u.kcnt[x0 + k * bs] : 0;
#pragma unroll
                for (int k = 0; k < LU; ++k)
                    if (cv[k]) u.kend[x0 + k * bs] = atomicAdd(&sh.kpos, cv[k]);
            }
            __syncthreads();
            for (int32_t p0 = tid; p0 < nk; p0 += LU * bs) {
                int32_t hv[LU], tv[LU], pos[LU];
#pragma unroll
                for (int k = 0; k < LU; ++k) {
                    const int32_t q = p0 + k * bs;
                    hv[k] = q < nk ? u.kb[q] : -1;
                    tv[k] = q < nk ? u.ka[q] : 0;
                }
#pragma unroll
                for (int k = 0; k < LU; ++k) pos[k] = hv[k] >= 0 ? atomicAdd(&u.kend[hv[k]], 1) : 0;
#pragma unroll
                for (int k = 0; k < LU; ++k)
                    if (hv[k] >= 0) u.kr[pos[k]] = tv[k];
            }
        } else if (sweep_rec) {
            // too many arcs to record: Kahn tests E*; undo the counts
            for (int32_t p = tid; p < kcap; p += bs) u.kcnt[u.kb[p]] = 0;
        }
        __syncthreads();
        if (tid == 0) sh.tail = 0;
        __syncthreads();
        for (int32_t x0 = tid; x0 < n; x0 += LU * bs) {
            bool sink[LU];
#pragma unroll
            for (int k = 0; k < LU; ++k) {
                const int32_t x = x0 + k * bs;
                sink[k] = false;
                if (x < n) {
                    const int32_t dx = Drow[x], o = u.outdeg[x];
                    sink[k] = dx != INF32 && (o & W_COUNT) == 0;
                }
            }
#pragma unroll
            for (int k = 0; k < LU; ++k)
                if (sink[k]) u.q1[atomicAdd(&sh.tail, 1)] = x0 + k * bs;
        }
        nsub = n;
    } else {
        nsub = sh.next;
        const int32_t nk = sh.nk;
        rec = kcap > 0 && nk <= kcap;
        if (!OUT_ROW && rec && nk < 0xffff && nsub < 0xffff && lds_kahn_bytes(nsub, nk, false) <= kbytes) {
            kahn_in_lds(s, nsub, nk, u, Srow, lds_kahn_bytes(nsub, nk, true) <= kbytes, sign, out, sh, kbuf);
            return;
        }
        if (rec) {
            // group the recorded arcs by head (the sub-DAG vertices)
            for (int32_t i = tid; i < nsub; i += bs) {
                const int32_t x = u.sub[i];
                const int32_t c = u.kcnt[x];
                if (c) u.kend[x] = atomicAdd(&sh.kpos, c);
            }
            __syncthreads();
            for (int32_t p = tid; p < nk; p += bs) u.kr[atomicAdd(&u.kend[u.kb[p]], 1)] = u.ka[p];
        } else if (kcap > 0) {
            for (int32_t p = tid; p < kcap; p += bs) u.kcnt[u.kb[p]] = 0;
        }
        __syncthreads();
        if (tid == 0) sh.tail = 0;
        __syncthreads();
        for (int32_t i = tid; i < nsub; i += bs) {
            const int32_t x = u.sub[i];
            if ((u.outdeg[x] & W_COUNT) == 0) u.q1[atomicAdd(&sh.tail, 1)] = x;
        }
    }
    __syncthreads();
    // 2. Kahn from the sinks
    int32_t qn = sh.tail;
    int32_t *qa = u.q1, *qb = u.q2;
    __syncthreads();
    while (qn > 0) {
        if (tid == 0) {
            sh.tail = 0;
            sh.kpos = 0;
        }
        __syncthreads();
        int32_t nslow = qn;
        const int32_t *slow = qa;
        if (pred || rec) {
            // a vertex with one DAG in-arc (a, x): sigma_sx = sigma_sa, so a
            // receives [x in B] + acc(x) itself (no count, no scan).  Its
            // tail is the stored predecessor, or the one recorded arc where
            // none are stored.  The others go to the back of the next
            // round's queue (the two never meet: a vertex queued for the
            // next round is not in this one) for the general step.
            for (int32_t idx = tid; idx < qn; idx += bs) {
                const int32_t x = qa[idx];
                const bool in_b = (u.outdeg[x] & W_B) != 0;
                int32_t p = PRED_MULTI;
                if (pred) p = pred[x];
                else if (u.kcnt[x] == 1) p = u.kr[u.kend[x] - 1];
                if (p < 0) {
                    qb[n - 1 - atomicAdd(&sh.kpos, 1)] = x;
                    continue;
                }
                const double ax = u.acc[x];
                if (x != s && ax != 0.0) {
                    if (OUT_ROW) out[x] = ax;
                    else atomicAdd(&out[x], sign * ax);
                }
                const double push = (in_b ? 1.0 : 0.0) + ax;
                if (push != 0.0) atomicAdd(&u.acc[p], push);
                if ((atomicSub(&u.outdeg[p], 1) & W_COUNT) == 1) qb[atomicAdd(&sh.tail, 1)] = p;
            }
            __syncthreads();
            nslow = sh.kpos;
            slow = qb + n - nslow;
        }
        for (int32_t c = 0; c < nslow; c += bs) {
            const int32_t idx = c + tid;
            int32_t x = 0, b0 = 0, deg = 0, dx = 0;
            double coef = 0.0;
            if (idx < nslow) {
                x = slow[idx];
                const double ax = u.acc[x];
                if (x != s && ax != 0.0) {
                    if (OUT_ROW) out[x] = ax;
                    else atomicAdd(&out[x], sign * ax);
                }
                // each predecessor a receives sigma_sa * coef
                coef = (((u.outdeg[x] & W_B) ? 1.0 : 0.0) + ax) / (double)Srow[x];
                if (rec) {
                    deg = u.kcnt[x];
                    b0 = deg ? u.kend[x] - deg : 0;
                } else {
                    b0 = cptr[x];
                    deg = cptr[x + 1] - b0;
                }
                dx = Drow[x];
            }
            int32_t total;
            const int32_t off = block_excl_scan(deg, sh.scan, total);
            es.off[tid] = off;
            es.vtx[tid] = x;
            es.beg[tid] = b0;
            es.dx[tid] = dx;
            es.val[tid] = coef;
            __syncthreads();
            const int32_t nv = min(bs, nslow - c);
            for (int32_t jb = tid * RU; jb < total; jb += bs * RU) {
                int32_t iv[RU], ev[RU], av[RU], wv[RU];
                bool ok[RU];
                chunk_arcs(es, nv, total, jb, iv, ev, ok);
#pragma unroll
                for (int k = 0; k < RU; ++k) {
                    av[k] = ok[k] ? (rec ? u.kr[ev[k]] : csrc[ev[k]]) : 0;
                    wv[k] = (ok[k] && !rec) ? cw[ev[k]] : 0;
                }
                double cf[RU];
#pragma unroll
                for (int k = 0; k < RU; ++k) {
                    cf[k] = 0.0;
                    if (!ok[k]) continue;
                    if (!rec) {
                        const int32_t da = Drow[av[k]];
                        ok[k] = da != INF32 && (int64_t)da + wv[k] == (int64_t)es.dx[iv[k]];
                    }
                    if (ok[k]) cf[k] = es.val[iv[k]];
                }
                uint64_t sa[RU];
#pragma unroll
                for (int k = 0; k < RU; ++k) sa[k] = (ok[k] && cf[k] != 0.0) ? Srow[av[k]] : 0;
#pragma unroll
                for (int k = 0; k < RU; ++k) {
                    if (!ok[k]) continue;
                    const int32_t a = av[k];
                    if (cf[k] != 0.0) atomicAdd(&u.acc[a], (double)sa[k] * cf[k]);
                    if ((atomicSub(&u.outdeg[a], 1) & W_COUNT) == 1) qb[atomicAdd(&sh.tail, 1)] = a;
                }
            }
            __syncthreads();
        }
        qn = sh.tail;
        int32_t *tmp = qa;
        qa = qb;
        qb = tmp;
        __syncthreads();
    }
    if (full) {
        for (int32_t x = tid; x < n; x += bs) {
            u.outdeg[x] = 0;
            u.acc[x] = 0.0;
            if (rec) u.kcnt[x] = 0;
        }
    } else {
        for (int32_t i = tid; i < nsub; i += bs) {
            const int32_t x = u.sub[i];
            u.outdeg[x] = 0;
            u.acc[x] = 0.0;
            if (rec) u.kcnt[x] = 0;
        }
    }
    __syncthreads();
}

// Partial dependency of source s over a target set B that is most of the row,
// from the stored predecessors (one workgroup): the pass of restricted_pass
// over all of DAG(s) instead of the ancestors of B.  The vertices with two or
// more DAG in-arcs test their E* in-arcs by Eq.1 and record them grouped by
// head; every other vertex has its tail in pred.  Then, with the successor
// counts in LDS over the staged row (lcnt; the row is not needed any more) and,
// where it fits, the accumulated dependency too (lacc), the leaves push first
// (several per lane in flight), and each lane carries on with the vertex that
// its push completes, along single in-arcs; a vertex with more of them waits
// for the workgroup's next arc-parallel step.  The share lands before the count
// drops (release), and the last pusher sees the others' (acquire).
// A pass is bound by the dependent accesses of one workgroup: rounds over the
// levels with counts and the record of all arcs in L2, after a sweep over all
// of E*, took 680 us at n = 32768, this takes 245 (half of it along the single
// in-arcs, with the dependency in L2); at n = 8192 255 and 56.
// Returns false, with nothing written but the slot's scratch, when the arcs
// outgrow the record (or a sample says that they would).
__device__ bool full_pass(const int32_t s, const int32_t n, const int32_t *Drow, const uint64_t *__restrict__ Srow,
                          const int32_t *__restrict__ cptr, const int32_t *__restrict__ csrc,
                          const int32_t *__restrict__ cw, const int32_t *__restrict__ Bt, const int32_t nB,
                          const USlot &u, const double sign, double *out, const int32_t *__restrict__ pred,
                          BlockShared &sh, const ExpandShared &es, int32_t *lcnt, double *lacc) {
    constexpr int RU = 4, LU = 4;
    const int tid = threadIdx.x, bs = blockDim.x;
    const int32_t kcap = (int32_t)u.kcap;
    auto cnt_at = [&](const int32_t x) -> int32_t { return lcnt ? lcnt[x] : shared_value<false>(&u.outdeg[x]); };
    auto cnt_inc = [&](const int32_t x) {
        if (lcnt) atomicAdd(&lcnt[x], 1);
        else atomicAdd(&u.outdeg[x], 1);
    };
    auto cnt_dec = [&](const int32_t x) -> int32_t {
        return lcnt ? __hip_atomic_fetch_sub(&lcnt[x], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)
                    : __hip_atomic_fetch_sub(&u.outdeg[x], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    };
    auto acc_at = [&](const int32_t x) -> double { return lacc ? lacc[x] : shared_value<false>(&u.acc[x]); };
    auto acc_add = [&](const int32_t x, const double v) {
        if (lacc) atomicAdd(&lacc[x], v);
        else atomicAdd(&u.acc[x], v);
    };
    if (tid == 0) {
        sh.next = 0;
        sh.nk = 0;
        sh.kpos = 0;
        sh.tail = 0;
        sh.head = 0;
    }
    __syncthreads();
    // the vertices with two or more DAG in-arcs, and those arcs
    for (int32_t x0 = tid; x0 < n; x0 += LU * bs) {
        int32_t pv[LU];
#pragma unroll
        for (int k = 0; k < LU; ++k) pv[k] = x0 + k * bs < n ? pred[x0 + k * bs] : PRED_NONE;
#pragma unroll
        for (int k = 0; k < LU; ++k)
            if (pv[k] == PRED_MULTI) u.sub[atomicAdd(&sh.next, 1)] = x0 + k * bs;
    }
    __syncthreads();
    const int32_t nmulti = sh.next;
    // the DAG in-arcs of one vertex per thread (-1: none), arc-parallel
    auto dag_in_arcs = [&](const int32_t x, auto &&f) {
        const int32_t b0 = x >= 0 ? cptr[x] : 0, deg = x >= 0 ? cptr[x + 1] - b0 : 0;
        int32_t total;
        const int32_t off = block_excl_scan(deg, sh.scan, total);
        es.off[tid] = off;
        es.vtx[tid] = x;
        es.beg[tid] = b0;
        es.dx[tid] = x >= 0 ? Drow[x] : 0;
        __syncthreads();
        for (int32_t jb = tid * RU; jb < total; jb += bs * RU) {
            int32_t iv[RU], ev[RU], av[RU], wv[RU];
            bool ok[RU];
            chunk_arcs(es, bs, total, jb, iv, ev, ok);
#pragma unroll
            for (int k = 0; k < RU; ++k) {
                av[k] = ok[k] ? csrc[ev[k]] : 0;
                wv[k] = ok[k] ? cw[ev[k]] : 0;
            }
#pragma unroll
            for (int k = 0; k < RU; ++k) {
                if (!ok[k]) continue;
                const int32_t da = Drow[av[k]];
                if (da != INF32 && (int64_t)da + wv[k] == (int64_t)es.dx[iv[k]]) f(av[k], es.vtx[iv[k]]);
            }
        }
        __syncthreads();
    };
    // where E* has many arcs per vertex, a sample first (a vertex for one thread in
    // eight; one for each costs 7% where the record fits): a record that these
    // would overfill is not begun, nor, below half of the row, one that they would
    // nearly fill (8 updates, 100 sources, 6001 changed targets of a row of 26101,
    // a record filled to the brim: 11.2 ms with it, 6.5 to 7.4 without)
    if (cptr[n] > 4 * kcap && nmulti > bs) {
        dag_in_arcs(tid & 7 ? -1 : u.sub[(int64_t)tid * nmulti / bs], [&](int32_t, int32_t) { atomicAdd(&sh.nk, 1); });
        const bool over = (int64_t)sh.nk * nmulti > (int64_t)(2 * (int64_t)nB >= n ? kcap : kcap / 4 * 3) * (bs / 8);
        __syncthreads();
        if (over) return false;
        if (tid == 0) sh.nk = 0;
        __syncthreads();
    }
    for (int32_t c = 0; c < nmulti; c += bs) {
        dag_in_arcs(c + tid < nmulti ? u.sub[c + tid] : -1, [&](const int32_t a, const int32_t h) {
            const int32_t p = atomicAdd(&sh.nk, 1);
            if (p < kcap) {
                u.ka[p] = a;
                u.kb[p] = h;
                atomicAdd(&u.kcnt[h], 1);
            }
        });
        if (sh.nk > kcap) break;  // (nothing adds to it before the next chunk's barriers)
    }
    const int32_t nk = sh.nk;
    if (nk > kcap) {
        for (int32_t i = tid; i < nmulti; i += bs) u.kcnt[u.sub[i]] = 0;
        __syncthreads();
        return false;
    }
    for (int32_t i = tid; i < nmulti; i += bs) {
        const int32_t x = u.sub[i];
        u.kend[x] = atomicAdd(&sh.kpos, shared_value<false>(&u.kcnt[x]));
    }
    // (the staged row ends here)
    if (lcnt)
        for (int32_t x = tid; x < n; x += bs) lcnt[x] = 0;
    if (lacc)
        for (int32_t x = tid; x < n; x += bs) lacc[x] = 0.0;
    __syncthreads();
    for (int32_t i = tid; i < nB; i += bs) {
        const int32_t t = Bt[i];
        if (t == s) continue;
        if (lcnt) lcnt[t] = W_B;
        else u.outdeg[t] = W_B;
    }
    for (int32_t p = tid; p < nk; p += bs) u.kr[atomicAdd(&u.kend[u.kb[p]], 1)] = u.ka[p];
    __syncthreads();
    // successor counts
    for (int32_t x0 = tid; x0 < n; x0 += LU * bs) {
        int32_t pv[LU];
#pragma unroll
        for (int k = 0; k < LU; ++k) pv[k] = x0 + k * bs < n ? pred[x0 + k * bs] : PRED_NONE;
#pragma unroll
        for (int k = 0; k < LU; ++k)
            if (pv[k] >= 0) cnt_inc(pv[k]);
    }
    for (int32_t p = tid; p < nk; p += bs) cnt_inc(u.ka[p]);
    __syncthreads();
    // the leaves (marked before any count drops; q1: vertices completed, q2:
    // those with two or more in-arcs)
    for (int32_t x = tid; x < n; x += bs) {
        const int32_t c = cnt_at(x);
        if (c & W_COUNT) continue;
        if (lcnt) lcnt[x] = c | W_VIS;
        else u.outdeg[x] = c | W_VIS;
    }
    __syncthreads();
    for (int32_t x0 = tid; x0 < n; x0 += LU * bs) {
        int32_t pv[LU];
#pragma unroll
        for (int k = 0; k < LU; ++k) pv[k] = x0 + k * bs < n ? pred[x0 + k * bs] : PRED_NONE;
#pragma unroll
        for (int k = 0; k < LU; ++k) {
            if (pv[k] == PRED_NONE) continue;
            const int32_t x = x0 + k * bs, c = cnt_at(x);
            if (!(c & W_VIS)) pv[k] = PRED_NONE;
            else if (pv[k] < 0) u.q2[atomicAdd(&sh.head, 1)] = x;
            else if (c & W_B) acc_add(pv[k], 1.0);
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        int32_t was[LU];
#pragma unroll
        for (int k = 0; k < LU; ++k) was[k] = pv[k] >= 0 ? cnt_dec(pv[k]) : 0;
#pragma unroll
        for (int k = 0; k < LU; ++k)
            if ((was[k] & W_COUNT) == 1) u.q1[atomicAdd(&sh.tail, 1)] = pv[k];
    }
    __syncthreads();
    int32_t lo = 0, hi = sh.tail;
    for (;;) {
        // along single in-arcs
        for (int32_t idx = lo + tid; idx < hi; idx += bs) {
            int32_t x = u.q1[idx], p = pred[x];
            for (;;) {
                if (p < 0) {
                    if (p == PRED_MULTI) u.q2[atomicAdd(&sh.head, 1)] = x;
                    break;
                }
                const int32_t pp = pred[p];
                const double push = ((cnt_at(x) & W_B) ? 1.0 : 0.0) + acc_at(x);
                if (push != 0.0) acc_add(p, push);
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
                if ((cnt_dec(p) & W_COUNT) != 1) break;
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
                x = p;
                p = pp;
            }
        }
        __syncthreads();
        const int32_t nslow = sh.head;
        lo = hi;
        __syncthreads();
        if (nslow == 0) break;
        if (tid == 0) sh.head = 0;
        for (int32_t c = 0; c < nslow; c += bs) {
            const int32_t idx = c + tid;
            int32_t b0 = 0, deg = 0;
            double coef = 0.0;
            if (idx < nslow) {
                const int32_t x = u.q2[idx];
                // each predecessor a receives sigma_sa * coef
                coef = (((cnt_at(x) & W_B) ? 1.0 : 0.0) + acc_at(x)) / (double)Srow[x];
                deg = shared_value<false>(&u.kcnt[x]);
                b0 = shared_value<false>(&u.kend[x]) - deg;
            }
            int32_t total;
            const int32_t off = block_excl_scan(deg, sh.scan, total);
            es.off[tid] = off;
            es.beg[tid] = b0;
            es.val[tid] = coef;
            __syncthreads();
            const int32_t nv = min(bs, nslow - c);
            for (int32_t jb = tid * RU; jb < total; jb += bs * RU) {
                int32_t iv[RU], ev[RU], av[RU];
                bool ok[RU];
                chunk_arcs(es, nv, total, jb, iv, ev, ok);
#pragma unroll
                for (int k = 0; k < RU; ++k) av[k] = ok[k] ? u.kr[ev[k]] : 0;
#pragma unroll
                for (int k = 0; k < RU; ++k) {
                    if (!ok[k]) continue;
                    const double cf = es.val[iv[k]];
                    if (cf != 0.0) acc_add(av[k], (double)Srow[av[k]] * cf);
                }
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
#pragma unroll
                for (int k = 0; k < RU; ++k)
                    if (ok[k] && (cnt_dec(av[k]) & W_COUNT) == 1) u.q1[atomicAdd(&sh.tail, 1)] = av[k];
            }
            __syncthreads();
        }
        hi = sh.tail;
    }
    for (int32_t x0 = tid; x0 < n; x0 += LU * bs) {
        double av[LU];
#pragma unroll
        for (int k = 0; k < LU; ++k) av[k] = x0 + k * bs < n ? acc_at(x0 + k * bs) : 0.0;
#pragma unroll
        for (int k = 0; k < LU; ++k) {
            const int32_t x = x0 + k * bs;
            if (x >= n) continue;
            if (av[k] != 0.0) {
                if (x != s) atomicAdd(&out[x], sign * av[k]);
                if (!lacc) u.acc[x] = 0.0;
            }
            if (!lcnt) u.outdeg[x] = 0;
        }
    }
    for (int32_t i = tid; i < nmulti; i += bs) u.kcnt[u.sub[i]] = 0;
    __syncthreads();
    return true;
}

// Small sub-DAGs in LDS.  Most sources' sub-DAGs hold a few dozen vertices,
// so the partial-dependency pass keeps their per-vertex state in an
// open-addressing hash table in LDS (with d(s,x) and sigma_sx cached), records
// the sub-DAG's arcs while discovering it, and runs the Kahn rounds over that
// arc list without touching global memory.  Only the E* in-arcs and the
// predecessors' distances are read from global memory.  A sub-DAG that
// outgrows the table is redone by restricted_pass (nothing global has been
// written by then).
// Table sizes of the LDS passes are a template parameter TS (a power of two
// of at most 256, so a slot fits a byte): TS hash slots, 3/4 of them admitted
// as vertices (load factor 3/4), 2 TS sub-DAG arcs.  Smaller tables let more
// workgroups share a CU; larger ones fall back to global memory less often.
#define SD_CONSTS                          \
    constexpr int SD_SLOTS = TS;           \
    constexpr int SD_CAP = TS * 3 / 4;     \
    constexpr int SD_ARCS = 2 * TS;

struct SmallDag {
    int32_t *key, *flags, *outdeg, *dval, *round;
    double *acc, *coef;
    uint64_t *sval;
    int16_t *sub, *arc_a, *arc_x;
};

template <int TS>
__host__ __device__ constexpr size_t small_dag_bytes() {
    SD_CONSTS
    return (size_t)SD_SLOTS * (5 * 4 + 3 * 8 + 2) + (size_t)SD_ARCS * 4 + 256;
}

template <int TS>
__device__ __forceinline__ SmallDag small_dag_at(char *p) {
    SD_CONSTS
    SmallDag d;
    d.acc = (double *)p;             p += 8 * SD_SLOTS;
    d.coef = (double *)p;            p += 8 * SD_SLOTS;
    d.sval = (uint64_t *)p;          p += 8 * SD_SLOTS;
    d.key = (int32_t *)p;            p += 4 * SD_SLOTS;
    d.flags = (int32_t *)p;          p += 4 * SD_SLOTS;
    d.outdeg = (int32_t *)p;         p += 4 * SD_SLOTS;
    d.dval = (int32_t *)p;           p += 4 * SD_SLOTS;
    d.round = (int32_t *)p;          p += 4 * SD_SLOTS;
    d.sub = (int16_t *)p;            p += 2 * SD_SLOTS;
    d.arc_a = (int16_t *)p;          p += 2 * SD_ARCS;
    d.arc_x = (int16_t *)p;
    return d;
}

// Slot of vertex x, inserting it if absent; -1 if the table is full.
template <int TS>
__device__ __forceinline__ int32_t sd_slot(const SmallDag &d, int32_t x, bool &inserted) {
    SD_CONSTS
    uint32_t h = ((uint32_t)x * 2654435761u) >> 24;
    inserted = false;
    for (int p = 0; p < SD_SLOTS; ++p) {
        const int32_t slot = (int32_t)((h + (uint32_t)p) & (SD_SLOTS - 1));
        const int32_t prev = atomicCAS(&d.key[slot], -1, x);
        if (prev == -1) {
            inserted = true;
            return slot;
        }
        if (prev == x) return slot;
    }
    return -1;
}

// The partial dependency of restricted_pass with all per-vertex state in
// LDS.  Returns false (and leaves global memory untouched) if the sub-DAG
// does not fit.
// One arc (a, x) of the LDS walk (x in slot sxv, da = d(s,a)): recorded,
// a's successor count raised, and a queued at its first sight.
template <int TS>
__device__ __forceinline__ void sd_add_arc(const SmallDag &d, BlockShared &sh, const int32_t a, const int32_t sxv,
                                           const int32_t da, const uint64_t *__restrict__ Srow) {
    SD_CONSTS
    bool ins;
    const int32_t sa = sd_slot<TS>(d, a, ins);
    const int32_t k = atomicAdd(&sh.tail, 1);
    if (sa < 0 || k >= SD_ARCS) {
        sh.ovf = 1;
        return;
    }
    d.arc_a[k] = (int16_t)sa;
    d.arc_x[k] = (int16_t)sxv;
    atomicAdd(&d.outdeg[sa], 1);
    if ((atomicOr(&d.flags[sa], F_VIS) & F_VIS) == 0) {
        d.dval[sa] = da;
        d.sval[sa] = Srow[a];
        const int32_t pos = atomicAdd(&sh.next, 1);
        if (pos >= SD_CAP) sh.ovf = 1;
        else d.sub[pos] = (int16_t)sa;
    }
}

template <int TS>
__device__ bool small_pass(const int32_t s, const int32_t *__restrict__ Drow, const uint64_t *__restrict__ Srow,
                           const int32_t *__restrict__ cptr, const int32_t *__restrict__ csrc,
                           const int32_t *__restrict__ cw, const int32_t *__restrict__ Bt, const int32_t nB,
                           const double sign, double *out, const int32_t *__restrict__ pred, BlockShared &sh, const ExpandShared &es, const SmallDag &d) {
    SD_CONSTS
    const int tid = threadIdx.x, bs = blockDim.x;
    for (int32_t i = tid; i < SD_SLOTS; i += bs) {
        d.key[i] = -1;
        d.flags[i] = 0;
        d.outdeg[i] = 0;
        d.acc[i] = 0.0;
        d.round[i] = -1;
    }
    if (tid == 0) {
        sh.next = 0;
        sh.tail = 0;  // arcs
        sh.ovf = 0; // overflow
    }
    __syncthreads();
    for (int32_t i = tid; i < nB; i += bs) {
        const int32_t t = Bt[i];
        const int32_t dt = Drow[t];
        if (t == s || dt == INF32) continue;
        bool ins;
        const int32_t slot = sd_slot<TS>(d, t, ins);
        const int32_t pos = atomicAdd(&sh.next, 1);
        if (slot < 0 || pos >= SD_CAP) {
            sh.ovf = 1;
            continue;
        }
        d.flags[slot] = F_VIS | F_B;
        d.dval[slot] = dt;
        d.sval[slot] = Srow[t];
        d.sub[pos] = (int16_t)slot;
    }
    __syncthreads();
    if (sh.ovf) return false;
    int32_t lo = 0, hi = sh.next;
    __syncthreads();
    while (lo < hi) {
        if (tid == 0) sh.head = 0;
        __syncthreads();
        // a vertex with one stored predecessor: that arc, at once; the others
        // (their E* in-arcs tested) listed in d.round, idle until the
        // accumulation
        for (int32_t idx = lo + tid; idx < hi; idx += bs) {
            const int32_t sx = d.sub[idx];
            const int32_t x = d.key[sx];
            const int32_t p = pred[x];
            if (p < 0) {
                d.round[atomicAdd(&sh.head, 1)] = sx;
                continue;
            }
            sd_add_arc<TS>(d, sh, p, sx, Drow[p], Srow);
        }
        __syncthreads();
        const int32_t nslow = sh.head;
        for (int32_t c = 0; c < nslow; c += bs) {
            const int32_t idx = c + tid;
            int32_t sx = 0, b0 = 0, deg = 0;
            if (idx < nslow) {
                sx = d.round[idx];
                const int32_t x = d.key[sx];
                b0 = cptr[x];
                deg = cptr[x + 1] - b0;
            }
            int32_t total;
            const int32_t off = block_excl_scan(deg, sh.scan, total);
            es.off[tid] = off;
            es.vtx[tid] = sx;
            es.beg[tid] = b0;
            __syncthreads();
            const int32_t nv = min(bs, nslow - c);
            for (int32_t j = tid; j < total; j += bs) {
                const int32_t i = find_owner(es, nv, j);
                const int32_t sxv = es.vtx[i];
                const int32_t e = es.beg[i] + (j - es.off[i]);
                const int32_t a = csrc[e];
                const int32_t da = Drow[a];
                if (da != INF32 && (int64_t)da + cw[e] == (int64_t)d.dval[sxv]) sd_add_arc<TS>(d, sh, a, sxv, da, Srow);
            }
            __syncthreads();
        }
        const bool ovf = sh.ovf != 0;
        lo = hi;
        hi = sh.next;
        __syncthreads();
        if (ovf) return false;
    }
    const int32_t nsub = hi, narcs = sh.tail;
    for (int32_t i = tid; i < SD_SLOTS; i += bs) d.round[i] = -1;
    __syncthreads();
    // Kahn from the sinks over the recorded arcs, all in LDS.  Round r makes
    // final the vertices whose successors all became final before r.
    for (int32_t i = tid; i < nsub; i += bs) {
        const int32_t sx = d.sub[i];
        if (d.outdeg[sx] == 0) d.round[sx] = 0;
    }
    __syncthreads();
    for (int32_t r = 0;; ++r) {
        if (tid == 0) sh.progress = 0;
        __syncthreads();
        // the vertices final in round r publish their coefficient and BC term
        for (int32_t i = tid; i < nsub; i += bs) {
            const int32_t sx = d.sub[i];
            if (d.round[sx] != r) continue;
            const double ax = d.acc[sx];
            const int32_t x = d.key[sx];
            if (x != s && ax != 0.0) atomicAdd(&out[x], sign * ax);
            d.coef[sx] = (((d.flags[sx] & F_B) ? 1.0 : 0.0) + ax) / (double)d.sval[sx];
            sh.progress = 1;
        }
        __syncthreads();
        if (sh.progress == 0) break;
        // and push to their predecessors
        for (int32_t k = tid; k < narcs; k += bs) {
            const int32_t sx = d.arc_x[k];
            if (d.round[sx] != r) continue;
            const int32_t sa = d.arc_a[k];
            atomicAdd(&d.acc[sa], (double)d.sval[sa] * d.coef[sx]);
            if (atomicSub(&d.outdeg[sa], 1) == 1) d.round[sa] = r + 1;
        }
        __syncthreads();
    }
    return true;
}

// Alg 2 (Update-DAG) on the stored predecessors: the new one of a changed
// target t of source s.  A target whose distance fell has exactly its DAG''(v)
// in-arcs as DAG'(s) in-arcs (at t = v: the in-arcs of the update that attain
// d'(s,v)); one whose distance stayed keeps its old in-arcs and gains those (at
// v: gains an arc, so it has two or more).  The row of v'' is that of v itself
// without out-arcs (no shortest path from v enters v again, so that row stands
// while others change), else the one the targets role formed.
// Testing the E* in-arcs of every changed target by Eq.1 instead (which any
// update but that of one arc did) is a round of gathers per pass and a record
// of all arcs per changed target: a submitted batch at n = 32768 took 34.4 ms
// that way and takes 32.0, a served queue of three Chung-Lu graphs 16.6 and 14.9.
__device__ __forceinline__ int32_t new_pred(const UpdateJob &J, const int32_t s, const int32_t t,
                                            const int32_t old_pred, const bool fell) {
    if (t == J.v) {
        const int32_t one = fell ? J.g.scal[s].flags >> 8 : 0;
        return one ? J.in_tail[one - 1] : PRED_MULTI;
    }
    const int32_t pv = J.row_v_pred[t];
    return fell ? pv : pred_union(old_pred, pv);
}

// Old and new partial dependency of one source in one traversal (LDS only).
// The vertices to visit are the union of the old sub-DAG (ancestors of B in
// DAG(s)) and the new one (ancestors of B in DAG'(s)); both are walked back
// from B at once.  The new distances and path counts are those of the B list
// for targets in B and the old ones elsewhere, so D and sigma are not written
// before the new pass.  Over the merged E* segment of a head x (E* by head,
// with the update's arcs appended), the first |E*(x)| arcs are the old E*
// arcs with their old weights: the old Eq.1 test looks at those only, the new
// test at all of them (an old-weight copy of a lowered arc cannot pass it).
// The two Kahn accumulations then run over the recorded arcs, and BC gets the
// difference delta'_B - delta_B once per vertex.  Returns false, before
// anything global is written, when the union does not fit.
//
// The walk is bound by its dependent loads.  A lane follows a chain of single
// in-arcs by itself (dd_follow), one load of the stored predecessors' row per
// vertex: a vertex with one DAG in-arc has its tail's path count, and its
// distance is needed only where Eq.1 is tested.  The changed targets' new
// in-arcs come from Alg 2 like stored ones.  Only vertices with two or more
// in-arcs test their E* in-arcs, in rounds of the whole workgroup; a tail's
// count and predecessor are read when it has passed the test.  A listed source of the
// n = 32768 Chung-Lu updates takes 28 us, one of a 64-vertex graph 14.6; level by
// level, with distance, count and predecessor read for every vertex and every
// tested arc, 35 and 17.6.
#define DD_CONSTS                          \
    constexpr int DD_SLOTS = TS;           \
    constexpr int DD_CAP = TS * 3 / 4;     \
    constexpr int DD_ARCS = 2 * TS;        \
    constexpr int DD_ROOTS = TS * 3 / 8;   \
    constexpr int DD_SLOW = 2 * DD_CAP;
enum : int32_t { DF_O = 1, DF_N = 2, DF_B = 4 };

struct DualDag {
    int32_t *key, *flags, *cnt, *dold, *dnew, *pr, *ybeg, *ydeg, *xdeg, *front, *slow, *arcs;
    double *acc_o, *acc_n, *coef;
    uint64_t *sold, *snew;
    // after the walk: the recorded arcs grouped by head (harc over ybeg and
    // ydeg, 2 * TS entries), each head's range end (hend over slow) and
    // in-arc count (hdeg over xdeg), and the Kahn work list (over coef, 2 * TS
    // entries of slot | kind << 8)
    int32_t *harc, *hend, *hdeg, *klist;
};

template <int TS>
__host__ __device__ constexpr size_t dual_dag_bytes() {
    DD_CONSTS
    return (size_t)DD_SLOTS * (9 * 4 + 5 * 8) + (size_t)(DD_ROOTS + DD_SLOW) * 4 + (size_t)DD_ARCS * 4 + 256;
}

template <int TS>
__device__ __forceinline__ DualDag dual_dag_at(char *p) {
    DD_CONSTS
    DualDag d;
    d.acc_o = (double *)p;    p += 8 * DD_SLOTS;
    d.acc_n = (double *)p;    p += 8 * DD_SLOTS;
    d.coef = (double *)p;     p += 8 * DD_SLOTS;
    d.sold = (uint64_t *)p;   p += 8 * DD_SLOTS;
    d.snew = (uint64_t *)p;   p += 8 * DD_SLOTS;
    d.key = (int32_t *)p;     p += 4 * DD_SLOTS;
    d.flags = (int32_t *)p;   p += 4 * DD_SLOTS;
    d.cnt = (int32_t *)p;     p += 4 * DD_SLOTS;  // successors: old in bits 0-15, new in 16-31
    d.dold = (int32_t *)p;    p += 4 * DD_SLOTS;
    d.dnew = (int32_t *)p;    p += 4 * DD_SLOTS;
    d.pr = (int32_t *)p;      p += 4 * DD_SLOTS;  // changed targets: stored (old) predecessor
    d.ybeg = (int32_t *)p;    p += 4 * DD_SLOTS;  // changed targets: merged E* in-arcs (start,
    d.ydeg = (int32_t *)p;    p += 4 * DD_SLOTS;  // count,
    d.xdeg = (int32_t *)p;    p += 4 * DD_SLOTS;  // and how many are old E* arcs), or with a
                                                  // count of -1 their one new in-arc's tail
    d.front = (int32_t *)p;   p += 4 * DD_ROOTS;  // the changed targets' slots
    d.slow = (int32_t *)p;    p += 4 * DD_SLOW;   // slot | memberships << 16 whose E* in-arcs are tested
    d.arcs = (int32_t *)p;                        // tail slot | head slot << 8 | kinds << 16
    d.harc = d.ybeg;
    d.hend = d.slow;
    d.hdeg = d.xdeg;
    d.klist = (int32_t *)d.coef;
    return d;
}

template <int TS>
__device__ __forceinline__ int32_t dd_find(const DualDag &d, int32_t x) {
    DD_CONSTS
    uint32_t h = ((uint32_t)x * 2654435761u) >> 24;
    for (int p = 0; p < DD_SLOTS; ++p) {
        const int32_t slot = (int32_t)((h + (uint32_t)p) & (DD_SLOTS - 1));
        const int32_t k = d.key[slot];
        if (k == x) return slot;
        if (k == -1) return -1;
    }
    return -1;
}

template <int TS>
__device__ __forceinline__ int32_t dd_slot(const DualDag &d, int32_t x) {
    DD_CONSTS
    uint32_t h = ((uint32_t)x * 2654435761u) >> 24;
    for (int p = 0; p < DD_SLOTS; ++p) {
        const int32_t slot = (int32_t)((h + (uint32_t)p) & (DD_SLOTS - 1));
        const int32_t prev = atomicCAS(&d.key[slot], -1, x);
        if (prev == -1 || prev == x) return slot;
    }
    return -1;
}

// One arc (a, x) of the union walk (x in slot sx; kinds: the sub-DAGs it is
// in; sa: a's slot, or -1 and then found): recorded, a's successor counts and
// memberships raised.  sg: sigma_sa, kept at a's first sight (a not in B: its
// new values are its old ones).  Returns the memberships a gains, 0 when the
// tables are full.
template <int TS>
__device__ __forceinline__ int32_t dd_add_arc(const DualDag &d, BlockShared &sh, const int32_t a, int32_t &sa,
                                              const int32_t sx, const int32_t kinds, const uint64_t sg) {
    DD_CONSTS
    if (sa < 0) sa = dd_slot<TS>(d, a);
    const int32_t k = atomicAdd(&sh.tail, 1);
    if (sa < 0 || k >= DD_ARCS) {
        sh.ovf = 1;
        return 0;
    }
    d.arcs[k] = sa | (sx << 8) | (kinds << 16);
    atomicAdd(&d.cnt[sa], ((kinds & DF_O) ? 1 : 0) + ((kinds & DF_N) ? 1 << 16 : 0));
    const int32_t old = atomicOr(&d.flags[sa], kinds);
    if (!(old & (DF_O | DF_N | DF_B))) {
        if (atomicAdd(&sh.nk, 1) >= DD_CAP) {
            sh.ovf = 1;
            return 0;
        }
        d.sold[sa] = sg;
        d.snew[sa] = sg;
    }
    return kinds & ~old;
}

// Slot sl, newly a member of the sub-DAGs `kinds`, has two or more in-arcs.
template <int TS>
__device__ __forceinline__ void dd_push_slow(const DualDag &d, BlockShared &sh, const int32_t sl, const int32_t kinds) {
    DD_CONSTS
    const int32_t pos = atomicAdd(&sh.kpos, 1);
    if (pos >= DD_SLOW) sh.ovf = 1;
    else d.slow[pos] = sl | (kinds << 16);
}

// From the vertex in slot x, whose one in-arc in the sub-DAGs `kinds` comes
// from p (with path count sg), back along single in-arcs: to s, to a vertex
// that has the memberships already (a changed target always has), or to one
// with two or more in-arcs.
template <int TS>
__device__ __forceinline__ void dd_follow(const DualDag &d, BlockShared &sh, const int32_t s,
                                          const int32_t *__restrict__ pred, int32_t x, int32_t p, int32_t kinds,
                                          const uint64_t sg) {
    for (;;) {
        const int32_t pp = pred[p];  // (on its way while the arc is recorded)
        int32_t sp = -1;
        kinds = dd_add_arc<TS>(d, sh, p, sp, x, kinds, sg);
        if (!kinds || p == s) break;
        if (pp < 0) {
            dd_push_slow<TS>(d, sh, sp, kinds);
            break;
        }
        x = sp;
        p = pp;
    }
}

// The recorded arcs grouped by head (a counting sort in LDS), for the Kahn
// walks of both sub-DAGs.
template <int TS>
__device__ __forceinline__ void dual_group_arcs(const DualDag &d, const int32_t narcs, BlockShared &sh) {
    DD_CONSTS
    const int tid = threadIdx.x, bs = blockDim.x;
    for (int32_t i = tid; i < DD_SLOTS; i += bs) d.hdeg[i] = 0;
    __syncthreads();
    for (int32_t k = tid; k < narcs; k += bs) atomicAdd(&d.hdeg[(d.arcs[k] >> 8) & 0xff], 1);
    __syncthreads();
    // exclusive scan over the slots, a run of consecutive slots per thread
    const int32_t per = (DD_SLOTS + bs - 1) / bs, i0 = min(tid * per, DD_SLOTS), i1 = min(i0 + per, DD_SLOTS);
    int32_t run = 0;
    for (int32_t i = i0; i < i1; ++i) run += d.hdeg[i];
    int32_t total;
    int32_t off = block_excl_scan(run, sh.scan, total);
    for (int32_t i = i0; i < i1; ++i) {
        d.hend[i] = off;
        off += d.hdeg[i];
    }
    __syncthreads();
    // the scatter leaves hend[h] at the end of h's range
    for (int32_t k = tid; k < narcs; k += bs) {
        const int32_t e = d.arcs[k];
        d.harc[atomicAdd(&d.hend[(e >> 8) & 0xff], 1)] = e;
    }
    __syncthreads();
}

// Dependency accumulation over both sub-DAGs at once from their sinks: a member
// x of one, once every successor has pushed, gives each DAG predecessor a the
// share sigma_sa * ([x in B] + acc(x)) / sigma_sx.  The lane whose push
// completes a carries on with a at once, so a chain takes no rounds; a vertex
// completing two or more waits for the next round.
template <int TS>
__device__ __forceinline__ void dual_kahn(const DualDag &d, BlockShared &sh) {
    DD_CONSTS
    const int tid = threadIdx.x, bs = blockDim.x;
    if (tid == 0) sh.kpos = 0;
    __syncthreads();
    for (int32_t i = tid; i < DD_SLOTS; i += bs) {
        if (d.key[i] < 0) continue;
        const int32_t f = d.flags[i], c = d.cnt[i];
        if ((f & DF_O) && (c & 0xffff) == 0) d.klist[atomicAdd(&sh.kpos, 1)] = i | (DF_O << 8);
        if ((f & DF_N) && ((c >> 16) & 0xffff) == 0) d.klist[atomicAdd(&sh.kpos, 1)] = i | (DF_N << 8);
    }
    __syncthreads();
    int32_t lo = 0, hi = sh.kpos;
    // (every wave has read the end of the first round before one lists more)
    __syncthreads();
    while (lo < hi) {
        for (int32_t idx = lo + tid; idx < hi; idx += bs) {
            int32_t x = d.klist[idx] & 0xff;
            const int32_t kind = d.klist[idx] >> 8, shift = kind == DF_O ? 0 : 16;
            double *const acc = kind == DF_O ? d.acc_o : d.acc_n;
            const uint64_t *const sv = kind == DF_O ? d.sold : d.snew;
            for (;;) {
                const double c = (((d.flags[x] & DF_B) ? 1.0 : 0.0) + acc[x]) / (double)sv[x];
                int32_t next = -1;
                const int32_t e1 = d.hend[x];
                for (int32_t e = e1 - d.hdeg[x]; e < e1; ++e) {
                    const int32_t arc = d.harc[e];
                    if (!((arc >> 16) & kind)) continue;
                    const int32_t a = arc & 0xff;
                    if (c != 0.0) atomicAdd(&acc[a], (double)sv[a] * c);
                    // release: the share lands before the count drops;
                    // acquire: the last pusher sees every other share
                    const int32_t left = __hip_atomic_fetch_sub(&d.cnt[a], 1 << shift, __ATOMIC_ACQ_REL,
                                                                 __HIP_MEMORY_SCOPE_WORKGROUP);
                    if (((left >> shift) & 0xffff) == 1) {
                        if (next < 0) next = a;
                        else d.klist[atomicAdd(&sh.kpos, 1)] = a | (kind << 8);
                    }
                }
                if (next < 0) break;
                x = next;
            }
        }
        __syncthreads();
        lo = hi;
        hi = sh.kpos;
        __syncthreads();
    }
}

template <int TS>
__device__ bool dual_pass(const UpdateJob &J, const int32_t s, const int32_t *__restrict__ Dold,
                          const uint64_t *__restrict__ Sold, const int32_t *__restrict__ xcp,
                          const int32_t *__restrict__ ycp, const int32_t *__restrict__ ycs,
                          const int32_t *__restrict__ ycw, const int32_t *__restrict__ Bt,
                          const int32_t *__restrict__ Bd, const uint64_t *__restrict__ Bs,
                          const int32_t *__restrict__ pred, const int32_t nb, double *out, BlockShared &sh,
                          const ExpandShared &es, const DualDag &d) {
    DD_CONSTS
    const int tid = threadIdx.x, bs = blockDim.x;
    for (int32_t i = tid; i < DD_SLOTS; i += bs) {
        d.key[i] = -1;
        d.flags[i] = 0;
        d.cnt[i] = 0;
        d.acc_o[i] = 0.0;
        d.acc_n[i] = 0.0;
    }
    if (tid == 0) {
        sh.next = 0;   // changed targets
        sh.tail = 0;   // recorded arcs
        sh.nk = 0;     // vertices
        sh.kpos = 0;   // slow list
        sh.ovf = 0;
    }
    __syncthreads();
    // B: roots of both sub-DAGs (of the old one only if t was reachable)
    for (int32_t i = tid; i < nb; i += bs) {
        const int32_t t = Bt[i];
        if (t == s) continue;
        const int32_t slot = dd_slot<TS>(d, t);
        const int32_t v = atomicAdd(&sh.nk, 1);
        const int32_t pos = atomicAdd(&sh.next, 1);
        if (slot < 0 || v >= DD_CAP || pos >= DD_ROOTS) {
            sh.ovf = 1;
            continue;
        }
        // what the walk reads of t, in one round trip
        const int32_t dt = Dold[t], dn = Bd[i];
        const uint64_t st = Sold[t];
        const int32_t pt = pred[t];
        int32_t yb = new_pred(J, s, t, pt, dn < dt), deg = -1, olen = 0;
        const int32_t mem = DF_N | (dt != INF32 ? DF_O : 0);
        d.flags[slot] = DF_B | mem;
        d.dold[slot] = dt;
        d.dnew[slot] = dn;
        d.sold[slot] = dt != INF32 ? st : 0;
        d.snew[slot] = Bs[i];
        d.pr[slot] = pt;
        if (yb < 0) {
            // two or more new in-arcs
            yb = ycp[t];
            deg = ycp[t + 1] - yb;
            olen = xcp[t + 1] - xcp[t];
        }
        d.ybeg[slot] = yb;
        d.ydeg[slot] = deg;
        d.xdeg[slot] = olen;
        d.front[pos] = slot;
    }
    __syncthreads();
    if (sh.ovf) return false;
    // back from every changed target, a lane for its old in-arcs and one for
    // its new ones (an in-arc that is both goes with the old ones)
    const int32_t nroot = sh.next;
    for (int32_t idx = tid; idx < 2 * nroot; idx += bs) {
        const int32_t sl = d.front[idx >> 1];
        const int32_t pr = (d.flags[sl] & DF_O) ? d.pr[sl] : PRED_NONE, pn = d.ydeg[sl] < 0 ? d.ybeg[sl] : PRED_MULTI;
        const bool one = pr >= 0 && pr == pn;
        // (one walk for both kinds of lane: two would run one after the other)
        const bool odd = (idx & 1) != 0;
        const int32_t slow = (pr == PRED_MULTI ? DF_O : 0) | (pn < 0 ? DF_N : 0);
        if (odd && slow) dd_push_slow<TS>(d, sh, sl, slow);
        const int32_t p = odd ? (one ? PRED_NONE : pn) : pr;
        if (p >= 0)
            dd_follow<TS>(d, sh, s, pred, sl, p, odd ? DF_N : one ? DF_O | DF_N : DF_O, odd ? d.snew[sl] : d.sold[sl]);
    }
    __syncthreads();
    // the vertices whose E* in-arcs are tested: arc-parallel, and back from
    // every tail found
    int32_t lo = 0, hi = sh.kpos;
    bool ovf = sh.ovf != 0;
    __syncthreads();
    while (lo < hi && !ovf) {
        for (int32_t c = lo; c < hi; c += bs) {
            const int32_t idx = c + tid;
            int32_t entry = 0, b0 = 0, cnt = 0, olen = 0;
            if (idx < hi) {
                entry = d.slow[idx];
                const int32_t sl = entry & 0xffff, mem = entry >> 16;
                const int32_t x = d.key[sl];
                if ((d.flags[sl] & DF_B) && d.ydeg[sl] >= 0) {
                    b0 = d.ybeg[sl];
                    cnt = d.ydeg[sl];
                    olen = d.xdeg[sl];
                } else {
                    b0 = ycp[x];
                    cnt = ycp[x + 1] - b0;
                    olen = xcp[x + 1] - xcp[x];
                    if (!(d.flags[sl] & DF_B)) {
                        const int32_t dx = Dold[x];
                        d.dold[sl] = dx;
                        d.dnew[sl] = dx;
                    }
                }
                // old in-arcs alone: the old E* arcs alone are tested
                if (mem == DF_O) cnt = olen;
            }
            int32_t total;
            const int32_t off = block_excl_scan(cnt, sh.scan, total);
            es.off[tid] = off;
            es.vtx[tid] = entry;
            es.beg[tid] = b0;
            es.dx[tid] = olen;
            __syncthreads();
            const int32_t nv = min(bs, hi - c);
            for (int32_t j = tid; j < total; j += bs) {
                if (*(volatile int32_t *)&sh.ovf) break;
                const int32_t i = find_owner(es, nv, j);
                const int32_t ent = es.vtx[i];
                const int32_t sx = ent & 0xffff, mem = ent >> 16;
                const int32_t rel = j - es.off[i];
                const int32_t e = es.beg[i] + rel;
                const int32_t a = ycs[e], w = ycw[e];
                const int32_t da_o = Dold[a];
                int32_t sa = dd_find<TS>(d, a);
                const int32_t da_n = (sa >= 0 && (d.flags[sa] & DF_B)) ? d.dnew[sa] : da_o;
                const bool po = (mem & DF_O) && rel < es.dx[i] && da_o != INF32 &&
                                (int64_t)da_o + w == (int64_t)d.dold[sx];
                const bool pn = (mem & DF_N) && da_n != INF32 && (int64_t)da_n + w == (int64_t)d.dnew[sx];
                if (!po && !pn) continue;
                const uint64_t sg = Sold[a];
                const int32_t pa = pred[a];
                const int32_t gained = dd_add_arc<TS>(d, sh, a, sa, sx, (po ? DF_O : 0) | (pn ? DF_N : 0), sg);
                if (!gained || a == s) continue;
                if (pa < 0) dd_push_slow<TS>(d, sh, sa, gained);
                else dd_follow<TS>(d, sh, s, pred, sa, pa, gained, sg);
            }
            __syncthreads();
        }
        lo = hi;
        hi = sh.kpos;
        ovf = sh.ovf != 0;
        __syncthreads();
    }
    if (ovf) return false;
    const int32_t narcs = sh.tail;
    dual_group_arcs<TS>(d, narcs, sh);
    dual_kahn<TS>(d, sh);
    for (int32_t i = tid; i < DD_SLOTS; i += bs) {
        const int32_t x = d.key[i];
        if (x < 0 || x == s) continue;
        const double diff = d.acc_n[i] - d.acc_o[i];
        if (diff != 0.0) atomicAdd(&out[x], diff);
    }
    __syncthreads();
    return true;
}

// Row-v data an update reads for every pair (s,t) of an affected row.
struct RowV {
    const int32_t *rvD;   // d(v,t)  (= d'(v,t))
    const uint64_t *rvS;  // sigma_vt
    const int32_t *rvvD;  // d''(v,t)           (Out phase only)
    const uint64_t *rvvS; // sigma''_vt
    const uint64_t *rvvH; // sigma-hat''_vt
    bool has_out;
};

// New (d, sigma) of pair (s,t) by Lemma 4 In phase (D = d'(s,v) + d(v,t)),
// then, if E_o is not empty, Lemma 4 on G'_R (D = d'(s,v) + d''(v,t)).  sigma
// is read only where a distance test says the pair may change.  Returns true
// if the pair changes.
__device__ __forceinline__ bool pair_update(const RowV &R, const SrcScal &sc, const bool same, const int32_t t,
                                            const int32_t d0, const int32_t rvd, const int32_t dvv,
                                            const uint64_t *Sg, int32_t &d_out, uint64_t &s_out, bool &ovf_s,
                                            bool &ovf_d) {
    int32_t d = d0;
    uint64_t sg = 0;
    bool sg_known = false;
    int64_t c;
    if (in_rule(d0, sc.dv, rvd, c)) {
        if (c >= INF32) {
            ovf_d = true;
        } else if (c < d0) {
            d = (int32_t)c;
            sg = mul_chk(sc.sv, R.rvS[t], ovf_s);
            sg_known = true;
        } else {
            const uint64_t add = mul_chk(same ? sc.hv : sc.sv, R.rvS[t], ovf_s);
            if (add != 0) {
                sg = add_chk(Sg[t], add, ovf_s);
                sg_known = true;
            }
        }
    }
    if (R.has_out) {
        int64_t c2;
        if (in_rule(d, sc.dv, dvv, c2)) {
            if (c2 >= INF32) {
                ovf_d = true;
            } else if (c2 < d) {
                d = (int32_t)c2;
                sg = mul_chk(sc.sv, R.rvvS[t], ovf_s);
                sg_known = true;
            } else {
                const uint64_t mult = (dvv == rvd) ? R.rvvH[t] : R.rvvS[t];
                const uint64_t add = mul_chk(sc.sv, mult, ovf_s);
                if (add != 0) {
                    sg = add_chk(sg_known ? sg : Sg[t], add, ovf_s);
                    sg_known = true;
                }
            }
        }
    }
    d_out = d;
    s_out = sg;
    return sg_known;
}

// Quick reject: neither phase can reach pair (s,t) unless d'(s,v) plus the
// row-v distance is at most the current d(s,t) (Lemma 4 case 1 otherwise).
// in_on is false for a source whose In phase is void: d'(s,v) = d(s,v) with
// no new paths into v (sigma-hat'_sv = 0), where a tie adds 0 paths and a
// strict gain would break the triangle inequality of the old distances.
__device__ __forceinline__ bool may_change(int32_t d0, int32_t dv, int32_t rvd, int32_t dvv, bool in_on) {
    if (dv == INF32) return false;
    const bool in = in_on && rvd != INF32 && ((int64_t)dv + rvd <= (int64_t)d0 || d0 == INF32);
    const bool out = dvv != INF32 && ((int64_t)dv + dvv <= (int64_t)d0 || d0 == INF32);
    return in || out;
}

// The same test against one filter row f (f_any, or f_out when the In phase
// is void) for a finite d'(s,v): d'(s,v) + f(t) <= d(s,t), or t unreachable.
// Finite distances are below 2^31-1, so the sum of two fits in 32 unsigned
// bits.
__device__ __forceinline__ bool may_change1(int32_t d0, int32_t dv, int32_t f) {
    return f != INF32 && ((uint32_t)dv + (uint32_t)f <= (uint32_t)d0 || d0 == INF32);
}

// Changed-target list a row scan fills: entries go to (t, d, s) up to cap;
// the count (BlockShared::nb) keeps going past cap, and then the list is
// incomplete.
struct BList {
    int32_t *t, *d;
    uint64_t *s;
    int32_t cap;
};

// A streamed row quad.  Each affected row is read once per update, so its
// loads are nontemporal: they do not displace the filter row, which every
// row of the update reads again, from the caches.
__device__ __forceinline__ int4 load_stream(const int4 *p) {
    typedef int v4i __attribute__((ext_vector_type(4)));
    const v4i t = __builtin_nontemporal_load((const v4i *)p);
    return make_int4(t.x, t.y, t.z, t.w);
}

// Bit mask of the pairs of one quad that may change (dv finite).
__device__ __forceinline__ uint32_t quad_mask(const int4 d, const int4 f, const int32_t dv) {
    return (may_change1(d.x, dv, f.x) ? 1u : 0u) | (may_change1(d.y, dv, f.y) ? 2u : 0u) |
           (may_change1(d.z, dv, f.z) ? 4u : 0u) | (may_change1(d.w, dv, f.w) ? 8u : 0u);
}

// Row scan of affected source s (the all-pairs step of Alg 3, restricted to
// row s), in two phases:
//   1. the distance filter (may_change) over the candidate targets when that
//      list is short, else over the whole row against the filter rows; the
//      targets that pass go to F (up to fcap; the count in sh.nf goes on),
//   2. after a barrier, all lanes share the flagged targets: the full
//      Lemma 4 update of each (from the rows themselves), and the pairs that
//      change go to the B list L with their new values (count in sh.nb).
// Keeping the second phase out of the streaming loop keeps that loop small
// and spreads the flagged pairs over the workgroup.  The caller zeroes sh.nf
// and sh.nb before; if sh.nf > fcap after the call, the B list is incomplete.
// QU quads per lane are in flight in the streaming loop.
template <int QU>
__device__ __forceinline__ void scan_row(const UpdateJob &J, const RowV &R, const SrcScal &sc, const bool same,
                                         const int32_t *__restrict__ Drow, const uint64_t *__restrict__ Sg,
                                         const bool use_tlist, const int32_t t_count, int32_t *F, const int32_t fcap,
                                         const BList &L, BlockShared &sh, bool &ovf_s, bool &ovf_d) {
    const int tid = threadIdx.x, bs = blockDim.x;
    const int32_t n = J.g.n;
    const bool in_on = !same || sc.hv != 0;
    auto flag = [&](int32_t t) {
        const int32_t pos = atomicAdd(&sh.nf, 1);
        if (pos < fcap) F[pos] = t;
    };
    if (use_tlist) {
        const int32_t *const tlist = J.g.tlist, *const tl_rvD = J.g.tl_rvD, *const tl_rvvD = J.g.tl_rvvD;
        for (int32_t i = tid; i < t_count; i += bs) {
            const int32_t t = tlist[i];
            if (may_change(Drow[t], sc.dv, tl_rvD[i], R.has_out ? tl_rvvD[i] : INF32, in_on)) flag(t);
        }
    } else if (sc.dv == INF32) {
        // v unreachable from s: no pair of the row can change
    } else if ((n & 3) == 0) {
        // QU quads (4 QU pairs) per lane in flight, tested against one
        // filter row
        const int32_t nq = n >> 2;
        const int4 *D4 = (const int4 *)Drow;
        const int4 *F4 = (const int4 *)(in_on ? J.g.f_any : J.g.f_out);
        for (int32_t q0 = tid; q0 < nq; q0 += QU * bs) {
            int4 dq[QU], fq[QU];
#pragma unroll
            for (int k = 0; k < QU; ++k) {
                const int32_t q = q0 + k * bs;
                dq[k] = (q < nq) ? load_stream(D4 + q) : make_int4(0, 0, 0, 0);
                fq[k] = (q < nq) ? F4[q] : make_int4(INF32, INF32, INF32, INF32);
            }
            uint32_t m = 0;
#pragma unroll
            for (int k = 0; k < QU; ++k) m |= quad_mask(dq[k], fq[k], sc.dv) << (4 * k);
            while (m) {
                const int b = __ffs(m) - 1;
                m &= m - 1;
                flag(((q0 + (b >> 2) * bs) << 2) + (b & 3));
            }
        }
    } else {
        const int32_t *f = in_on ? J.g.f_any : J.g.f_out;
        // rows that start at any vertex: one pair per load, as many loads in
        // flight as keep the memory busy (one at a time, the row kernel took
        // 94 us an update at n = 8191, with them 63)
        constexpr int U = 2 * QU;
        for (int32_t t0 = tid; t0 < n; t0 += U * bs) {
            int32_t dv[U], fv[U];
#pragma unroll
            for (int k = 0; k < U; ++k) {
                const int32_t t = t0 + k * bs;
                dv[k] = t < n ? __builtin_nontemporal_load(Drow + t) : 0;
                fv[k] = t < n ? f[t] : INF32;
            }
            uint32_t m = 0;
#pragma unroll
            for (int k = 0; k < U; ++k) m |= (may_change1(dv[k], sc.dv, fv[k]) ? 1u : 0u) << k;
            for (; m; m &= m - 1) flag(t0 + (__ffs(m) - 1) * bs);
        }
    }
    __syncthreads();
    const int32_t nf = min(sh.nf, fcap);
    for (int32_t i = tid; i < nf; i += bs) {
        const int32_t t = F[i];
        int32_t d;
        uint64_t sg;
        if (pair_update(R, sc, same, t, Drow[t], R.rvD[t], R.has_out ? R.rvvD[t] : INF32, Sg, d, sg, ovf_s, ovf_d)) {
            const int32_t pos = atomicAdd(&sh.nb, 1);
            if (pos < L.cap) {
                L.t[pos] = t;
                L.d[pos] = d;
                L.s[pos] = sg;
            }
        }
    }
}

__device__ __forceinline__ RowV row_v_of(const UpdateJob &J) {
    RowV R;
    R.rvD = J.row_v_D;
    R.rvS = J.row_v_S;
    R.rvvD = J.g.rvv_D;
    R.rvvS = J.g.rvv_S;
    R.rvvH = J.g.rvv_H;
    R.has_out = J.n_out > 0;
    return R;
}

// Rows of an update with at most 64 candidate targets (the candidate list is
// scanned instead of the rows): each wave takes 64 / lpr rows at once, a
// group of lpr lanes per row (lpr = the candidate count rounded up to a power
// of two), one candidate per lane, with no workgroup barriers.  The changed pairs of a
// row are compacted with a ballot and written to the step's target pool
// straight from the lanes; the listing rules are those of k_rows, with the
// pool and list reservations of a wave's rows taken in one atomic each.
__device__ void rows_few_targets(const UpdateJob &J, const RowV &R, const int32_t count, const int32_t t_count,
                                 const int32_t cap, const StepPool &pool, const int32_t turn) {
    GraphCtl *ctl = J.g.ctl;
    const int32_t n = J.g.n;
    const int lane = lane_id();
    int lpr = 1;
    while (lpr < t_count) lpr <<= 1;
    const int rpw = 64 / lpr;
    const int g = lane / lpr, r = lane - g * lpr;
    const uint64_t gmask = lpr == 64 ? ~0ull : ((1ull << lpr) - 1);
    // this lane's candidate and its row-v data, the same for every row
    const bool has_t = r < t_count;
    const int32_t t = has_t ? J.g.tlist[r] : 0;
    const int32_t f_rvd = has_t ? J.g.tl_rvD[r] : INF32;
    const int32_t f_rvvd = has_t && R.has_out ? J.g.tl_rvvD[r] : INF32;
    const int32_t rvd = has_t ? R.rvD[t] : INF32;
    const int32_t rvvd = has_t && R.has_out ? R.rvvD[t] : INF32;
    bool ovf_s = false, ovf_d = false;
    int32_t listed_pairs = 0;
    // the wave's first rows by its turn, the others from the counter (see k_rows)
    const int32_t wpb = (int32_t)blockDim.x >> 6, dealt = (int32_t)gridDim.x * wpb * rpw;
    int32_t base = (turn * wpb + ((int32_t)threadIdx.x >> 6)) * rpw;
    for (;;) {
        if (base >= count) break;
        const int32_t item = base + g;
        const bool row_ok = item < count;
        int32_t s = 0, d = 0;
        uint64_t sg = 0;
        bool chg = false;
        if (row_ok && has_t) {
            s = J.g.alist[item];
            const SrcScal sc = J.g.scal[s];
            const bool same = (sc.flags & 1) != 0;
            const int32_t *Drow = J.g.D + (size_t)s * n;
            const int32_t d0 = Drow[t];
            if (may_change(d0, sc.dv, f_rvd, f_rvvd, !same || sc.hv != 0))
                chg = pair_update(R, sc, same, t, d0, rvd, rvvd, J.g.S + (size_t)s * n, d, sg, ovf_s, ovf_d);
        }
        const uint64_t gm = (__ballot(chg) >> (g * lpr)) & gmask;
        const int32_t nb = (int32_t)__popcll(gm);
        // the groups' first lanes (each holds a candidate, so it read s) list
        // their sources, with one reservation per wave in the pool and in
        // each end of the list: a wave prefix sum of the pool entries wanted
        const bool lead = row_ok && r == 0 && nb > 0;
        const int32_t want = lead && nb <= cap ? nb : 0;
        int32_t incl = want;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int32_t v = __shfl_up(incl, o, 64);
            if (lane >= o) incl += v;
        }
        const int32_t total = __shfl(incl, 63, 64);
        int32_t pb_lo = 0, pb_hi = 0;
        if (lane == 0 && total > 0) {
            const unsigned long long o = atomicAdd(pool.next, (unsigned long long)total);
            pb_lo = (int32_t)(o & 0xffffffffull);
            pb_hi = (int32_t)(o >> 32);
        }
        pb_lo = __shfl(pb_lo, 0, 64);
        pb_hi = __shfl(pb_hi, 0, 64);
        const unsigned long long pbase = ((unsigned long long)(uint32_t)pb_hi << 32) | (uint32_t)pb_lo;
        const unsigned long long mine = pbase + (unsigned long long)(incl - want);
        const bool listed = want > 0 && mine + (unsigned long long)nb <= (unsigned long long)pool.cap;
        const uint64_t hm = __ballot(listed && nb >= HEAVY_NB), lm = __ballot(listed && nb < HEAVY_NB);
        const uint64_t dm = __ballot(lead && !listed);
        int32_t hb = 0, lb = 0, db = 0;
        if (lane == 0) {
            if (hm) hb = atomicAdd(&ctl->dag_count, (int32_t)__popcll(hm));
            if (lm) lb = atomicAdd(&ctl->dag_back, (int32_t)__popcll(lm));
            if (dm) db = atomicAdd(&ctl->big_count, (int32_t)__popcll(dm));
        }
        hb = __shfl(hb, 0, 64);
        lb = __shfl(lb, 0, 64);
        db = __shfl(db, 0, 64);
        if (listed) {
            DItem it;
            it.s = s;
            it.nb = nb;
            it.off = (int64_t)mine;
            if (nb >= HEAVY_NB) J.g.dlist[hb + (int32_t)popc_below(hm, lane)] = it;
            else J.g.dlist[n - 1 - (lb + (int32_t)popc_below(lm, lane))] = it;
            listed_pairs += nb;
        } else if (lead) {
            J.g.biglist[db + (int32_t)popc_below(dm, lane)] = s;
        }
        // the group's changed pairs go to its pool entries
        const int src_lane = g * lpr;
        const bool g_listed = __shfl((int32_t)listed, src_lane, 64) != 0;
        const int32_t off_lo = __shfl((int32_t)(mine & 0xffffffffull), src_lane, 64);
        const int32_t off_hi = __shfl((int32_t)(mine >> 32), src_lane, 64);
        if (chg && g_listed) {
            const unsigned long long p = (((unsigned long long)(uint32_t)off_hi << 32) | (uint32_t)off_lo) +
                                         (unsigned long long)__popcll(gm & ((1ull << r) - 1));
            pool.t[p] = t;
            pool.d[p] = d;
            pool.s[p] = sg;
        }
        if (count <= dealt) break;
        if (lane == 0) base = dealt + atomicAdd(&ctl->work_next, rpw);
        base = __shfl(base, 0, 64);
    }
    if (ovf_s) atomicOr(&ctl->status, ST_SIGMA_OVF);
    if (ovf_d) atomicOr(&ctl->status, ST_DIST_OVF);
    // one statistic update per wave
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) listed_pairs += __shfl_xor(listed_pairs, o, 64);
    if (lane == 0 && listed_pairs) atomicAdd(&ctl->changed_pairs, (unsigned long long)listed_pairs);
}

// Row kernel (persistent): each workgroup's first affected source of a job is
// its turn in a deal over the grid (the deal goes on from job to job), the
// others come from a device counter; it scans their rows (scan_row).  With
// the first one dealt, a job with no more sources than workgroups makes no
// claim at all: 1024 workgroups' claims on one counter are serialized where
// it lives (with WorkList in the other two kernels, 16 updates of a 64-vertex
// graph went from 2.12 to 1.61 ms, 64 of an n = 4096 one from 15.4 to 13.5).  A source's changed targets are
// collected in LDS; up to big_b of them are copied to the step's target pool
// and the source is listed for the DAG kernel, more (or a full pool) defer
// the source to the wide kernel, which scans the row again; so do more than
// soon_b while the step has places for them (see SOON_NB).  Nothing in D or sigma is written here: the old partial dependency still needs the old row.
__global__ void __launch_bounds__(256) k_rows(const UpdateJob *__restrict__ jobs, const int32_t *__restrict__ njobs_p,
                                              int32_t big_b, int32_t soon_b, StepPool pool) {
    __shared__ int32_t lt[LCAP], ld[LCAP], lf[LCAP];
    __shared__ uint64_t ls[LCAP];
    __shared__ BlockShared sh;
    __shared__ long long sh_off;
    const int tid = threadIdx.x, bs = blockDim.x;
    const int njobs = *njobs_p;
    const BList L{lt, ld, ls, min(big_b, LCAP)};
    const int32_t grid = (int32_t)gridDim.x;
    int32_t dealt = 0;  // sources dealt by the jobs before this one, modulo the grid
    for (int j = 0; j < njobs; ++j) {
        const UpdateJob &J = jobs[j];
        // another workgroup may halt the job meanwhile: one answer per workgroup
        if (__syncthreads_or(job_halted(J))) continue;
        GraphCtl *ctl = J.g.ctl;
        const int32_t n = J.g.n;
        const int32_t count = *(volatile int32_t *)&ctl->a_count;
        int32_t turn = (int32_t)blockIdx.x - dealt;
        if (turn < 0) turn += grid;
        const RowV R = row_v_of(J);
        const int32_t t_count = *(volatile int32_t *)&ctl->t_count;
        const bool use_tlist = (int64_t)t_count * 8 <= (int64_t)n;
        if (use_tlist && t_count <= 64) {
            // a row without candidates cannot change
            if (t_count > 0) rows_few_targets(J, R, count, t_count, L.cap, pool, turn);
            continue;
        }
        dealt = (int32_t)(((int64_t)dealt + min(count, grid)) % grid);
        if (turn >= count) continue;
        if (tid == 0) sh.counter = 0;
        bool ovf_s = false, ovf_d = false;
        for (bool first = true;; first = false) {
            if (!first && count <= grid) break;
            __syncthreads();
            if (tid == 0) {
                sh.item = first ? turn : grid + atomicAdd(&ctl->work_next, 1);
                sh.nb = 0;
                sh.nf = 0;
            }
            __syncthreads();
            const int32_t item = sh.item;
            if (item >= count) break;
            const int32_t s = J.g.alist[item];
            const SrcScal sc = J.g.scal[s];
            const int32_t *Drow = J.g.D + (size_t)s * n;
            const uint64_t *Sg = J.g.S + (size_t)s * n;
            scan_row<8>(J, R, sc, (sc.flags & 1) != 0, Drow, Sg, use_tlist, t_count, lf, LCAP, L, sh, ovf_s, ovf_d);
            __syncthreads();
            const int32_t nb = sh.nb;
            if (nb == 0 && sh.nf <= LCAP) continue;
            if (tid == 0) {
                long long off = -1;
                if (nb <= L.cap && sh.nf <= LCAP && !(nb > soon_b && atomicAdd(pool.soon, 1) < SOON_MAX)) {
                    const unsigned long long o = atomicAdd(pool.next, (unsigned long long)nb);
                    if (o + (unsigned long long)nb <= (unsigned long long)pool.cap) off = (long long)o;
                }
                if (off >= 0) {
                    DItem it;
                    it.s = s;
                    it.nb = nb;
                    it.off = off;
                    if (nb >= HEAVY_NB) J.g.dlist[atomicAdd(&ctl->dag_count, 1)] = it;
                    else J.g.dlist[n - 1 - atomicAdd(&ctl->dag_back, 1)] = it;
                    sh.counter += (unsigned long long)nb;
                } else {
                    J.g.biglist[atomicAdd(&ctl->big_count, 1)] = s;
                }
                sh_off = off;
            }
            __syncthreads();
            const long long off = sh_off;
            if (off >= 0) {
                for (int32_t i = tid; i < nb; i += bs) {
                    pool.t[off + i] = lt[i];
                    pool.d[off + i] = ld[i];
                    pool.s[off + i] = ls[i];
                }
            }
        }
        if (ovf_s) atomicOr(&ctl->status, ST_SIGMA_OVF);
        if (ovf_d) atomicOr(&ctl->status, ST_DIST_OVF);
        __syncthreads();
        if (tid == 0 && sh.counter) atomicAdd(&ctl->changed_pairs, sh.counter);
    }
}

// Bytes of LDS the DAG kernel's tables share.
template <int TS>
__host__ __device__ constexpr size_t dag_table_bytes() {
    return small_dag_bytes<TS>() > dual_dag_bytes<TS>() ? small_dag_bytes<TS>() : dual_dag_bytes<TS>();
}

// One listed source with its changed targets B (Bt, Bd, Bs; nb of them):
// both partial dependencies in one traversal in LDS (dual_pass) and then the
// changed pairs written to D and sigma; or, when the two sub-DAGs do not fit
// together:
//   1. old partial dependency over B (E* by head, old row), sign -1,
//   2. write the changed pairs (only those) to D and sigma,
//   3. new partial dependency over B (merged E*, new row), sign +1,
// each in LDS (small_pass) when it fits, else in the workgroup's slot.
template <int TS>
__device__ __forceinline__ void update_source(const UpdateJob &J, const int32_t s, const int32_t *__restrict__ Bt,
                                              const int32_t *__restrict__ Bd, const uint64_t *__restrict__ Bs,
                                              const int32_t nb, const USlot &u, BlockShared &sh, const ExpandShared &es, const SmallDag &sd,
                                              const DualDag &dd, char *table) {
    const int tid = threadIdx.x, bs = blockDim.x;
    const int32_t n = J.g.n;
    int32_t *const Dg = J.g.D + (size_t)s * n;
    uint64_t *const Sg = J.g.S + (size_t)s * n;
    double *const bc_delta = J.g.bc_delta;
    // an LDS table holds at most 3/4 of its slots in vertices: larger B sets
    // go straight to the slot passes.  The union of both sub-DAGs with a B of
    // half that many or more almost never fits (on the Chung-Lu headline
    // window, 120 of 20 600 such sources fit with the 128-slot table), so
    // those skip the union walk; the new sub-DAG alone often fits
    const bool fits = nb < TS * 3 / 4;
    const bool dual_fits = nb < TS * 3 / 8;  // (DD_ROOTS)
    int32_t *const pred_row = J.g.pred + (size_t)s * n;
    const bool dual = dual_fits && dual_pass<TS>(J, s, Dg, Sg, J.g.xc_ptr, J.g.yc_ptr, J.g.yc_src, J.g.yc_w, Bt, Bd,
                                                 Bs, pred_row, nb, bc_delta, sh, es, dd);
    // when the union outgrew the table it is mostly the old sub-DAG that did:
    // the old pass goes straight to the slot (it follows stored
    // predecessors), the new one tries the LDS table first
    if (!dual)
        restricted_pass<false, XU>(s, n, Dg, Sg, J.g.xc_ptr, J.g.xc_src, J.g.xc_dst, J.g.xc_w, Bt, nb, false, u,
                                   -1.0, bc_delta, pred_row, sh, es, table, dag_table_bytes<TS>());
    const int32_t old_sub = sh.next;  // (of the old pass; read before the barrier below)
    // the changed targets' new predecessors by Alg 2 (before the old distances
    // are overwritten); the new pass follows them like any stored predecessor
    for (int32_t i = tid; i < nb; i += bs) {
        const int32_t t = Bt[i];
        const int32_t d = Bd[i];
        pred_row[t] = new_pred(J, s, t, pred_row[t], d < Dg[t]);
        Sg[t] = Bs[i];
        Dg[t] = d;
    }
    __syncthreads();
    if (dual) return;
    // a sub-DAG of twice the table's capacity before the update rarely fits now
    // (with unit weights at n = 8191 the attempt cost 47 of a source's 264 us)
    const bool small = fits && old_sub <= TS * 3 / 2;
    if (!small || !small_pass<TS>(s, Dg, Sg, J.g.yc_ptr, J.g.yc_src, J.g.yc_w, Bt, nb, 1.0, bc_delta, pred_row, sh, es,
                                  sd))
        restricted_pass<false, XU>(s, n, Dg, Sg, J.g.yc_ptr, J.g.yc_src, J.g.yc_dst, J.g.yc_w, Bt, nb, false, u, 1.0,
                                   bc_delta, pred_row, sh, es, table, dag_table_bytes<TS>());
}

// The sources of a step's segments (one list per job, or two), numbered
// through in segment order and shared out over the persistent workgroups in
// units: the first max_pairs sources are two units each, the others one.
// Workgroup b takes unit b first and then units past the grid from a device
// counter, and makes no claim where there are no more units than workgroups.
// Claims on one counter are serialized where it lives, and 2560 workgroups with
// a claim per list took 48 us in a 64-vertex update (see k_rows).  Wave 0 keeps the segment of its last source and looks 64 segments
// up at a time when it moves on; it alone reads the halted flags, so that a
// job halted in between stops whole workgroups.
// Its state is in LDS (the DAG kernel has no register to spare for it).
template <typename F, typename H>
struct WorkList {
    const int32_t segs, max_pairs;
    int32_t *const counter;
    const F count;
    const H halted;
    BlockShared &sh;
    __device__ __forceinline__ WorkList(const int32_t nseg, const int32_t pairs, int32_t *next_unit, const F &f,
                                        const H &h, BlockShared &s)
        : segs(nseg), max_pairs(pairs), counter(next_unit), count(f), halted(h), sh(s) {
        if (threadIdx.x >= 64) return;
        int32_t total = 0;
        for (int32_t q = lane_id(); q < segs; q += 64) total += count(q);
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) total += __shfl_xor(total, o, 64);
        if (lane_id() == 0) {
            sh.wl_total = total;
            sh.wl_seg = -1;
            sh.wl_lo = sh.wl_hi = 0;
            sh.wl_first = 1;
        }
    }
    // The workgroup's next unit: sh.seg, sh.item (its source's place in the
    // segment), sh.source (its number) and sh.role (0 and 1 of a pair, else
    // 2); false when all are taken.  Every thread of the workgroup calls it.
    __device__ __forceinline__ bool next() {
        __syncthreads();
        if (threadIdx.x < 64) {
            const int32_t total = sh.wl_total, pairs = min(max_pairs, total), units = total + pairs;
            const int32_t grid = (int32_t)gridDim.x;
            int32_t seg = sh.wl_seg, lo = sh.wl_lo, hi = sh.wl_hi, unit, src = -1;
            bool first = sh.wl_first != 0;
            do {
                unit = first ? (int32_t)blockIdx.x : units;
                if (!first && units > grid) {
                    if (lane_id() == 0) unit = grid + atomicAdd(counter, 1);
                    unit = __shfl(unit, 0, 64);
                }
                first = false;
                if (unit >= units) break;
                src = unit < 2 * pairs ? unit >> 1 : unit - pairs;
                while (src >= hi) {
                    const int32_t q = seg + 1 + lane_id();
                    const int32_t c = q < segs ? count(q) : 0;
                    int32_t incl = c;
#pragma unroll
                    for (int o = 1; o < 64; o <<= 1) {
                        const int32_t v = __shfl_up(incl, o, 64);
                        if (lane_id() >= o) incl += v;
                    }
                    const uint64_t past = __ballot(hi + incl > src);
                    const int at = past ? __ffsll((unsigned long long)past) - 1 : 63;
                    const int32_t end = hi + __shfl(incl, at, 64), mine = __shfl(c, at, 64);
                    seg += 1 + at;
                    lo = end - mine;
                    hi = end;
                }
            } while (halted(seg));
            if (lane_id() == 0) {
                sh.item = unit < units ? src - lo : -1;
                sh.seg = seg;
                sh.source = src;
                sh.role = unit < 2 * pairs ? (unit & 1) : 2;
                sh.wl_seg = seg;
                sh.wl_lo = lo;
                sh.wl_hi = hi;
                sh.wl_first = 0;
            }
        }
        __syncthreads();
        return sh.item >= 0;
    }
};

// DAG kernel (persistent): workgroups take the sources the row kernel listed
// (WorkList) and run update_source on each.  Every workgroup's slot is laid out
// for the context-wide n_layout (the largest graph), so the zero-kept arrays sit
// at the same place for every job.  The work is bound by dependent gathers, so
// what counts is the sources in flight: the register budget is held to five
// waves per SIMD (ten 128-thread workgroups per CU), 96 registers with no
// spills, and the source's row is read from memory.  Staged in LDS (up to
// n = 8192) it left room for two or three workgroups per CU: 16 unit-weight
// insertions at n = 8191 took 16.4 ms with it and take 13.9, 64 arc updates at
// n = 4096 9.6 and 9.0; at n = 2048 and below both are the same.
template <int TS>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(5, 8))) k_source(const UpdateJob *__restrict__ jobs, const int32_t *__restrict__ njobs_p,
                                                char *__restrict__ scratch, size_t slot_bytes, int32_t n_layout,
                                                StepPool pool) {
    extern __shared__ __align__(16) char dyn_lds[];
    const ExpandShared es = expand_at(dyn_lds, 0);
    char *const table = dyn_lds + align256(XB * (size_t)blockDim.x);
    const SmallDag sd = small_dag_at<TS>(table);
    const DualDag dd = dual_dag_at<TS>(table);
    __shared__ BlockShared sh;
    const int njobs = *njobs_p;
    const USlot u = uslot_at(scratch + (size_t)blockIdx.x * slot_bytes, n_layout);
    // the heavy sources of every job first (the front of each job's list),
    // then the light ones (the back): a step's long sub-DAG passes start
    // early whatever job they belong to, and the light sources fill the tail
    auto seg_count = [&](const int32_t q) {
        const GraphCtl *c = jobs[q < njobs ? q : q - njobs].g.ctl;
        return q < njobs ? *(const volatile int32_t *)&c->dag_count : *(const volatile int32_t *)&c->dag_back;
    };
    auto seg_halted = [&](const int32_t q) { return job_halted(jobs[q < njobs ? q : q - njobs]); };
    WorkList wl(2 * njobs, 0, pool.src_next, seg_count, seg_halted, sh);
    while (wl.next()) {
        const int32_t seg = sh.seg, item = sh.item;
        const UpdateJob &J = jobs[seg < njobs ? seg : seg - njobs];
        const DItem it = J.g.dlist[seg < njobs ? item : J.g.n - 1 - item];
        update_source<TS>(J, it.s, pool.t + it.off, pool.d + it.off, pool.s + it.off, it.nb, u, sh, es, sd, dd, table);
    }
}

// Wide kernel (persistent, beside the DAG kernel): the deferred sources,
// one workgroup of up to 1024 threads per unit of work.  The first
// item_regions deferred sources (over the jobs in order) run as two units on
// two workgroups at once: the old pass (it also stores the changed pairs in
// the source's item region) and the new pass (it forms the new row, path counts
// and stored predecessors in its slot from the old ones and the changed pairs).
// Neither writes D, sigma or the predecessors; k_wide_apply does afterwards.  Further deferred sources
// run as one unit each: scan, old pass, write the changed pairs, new pass.
// Every unit scans its row again into the slot's full-length list.
__global__ void __launch_bounds__(1024) k_source_wide(const UpdateJob *__restrict__ jobs,
                                                      const int32_t *__restrict__ njobs_p, char *__restrict__ scratch,
                                                      size_t slot_bytes, int32_t lds_cap, int32_t n_layout,
                                                      char *__restrict__ items, int32_t item_regions, StepPool pool,
                                                      size_t lds_bytes) {
    extern __shared__ __align__(16) char dyn_lds[];
    int32_t *const lds_row = (int32_t *)dyn_lds;
    const ExpandShared es = expand_at(dyn_lds, lds_cap);
    __shared__ BlockShared sh;
    const int tid = threadIdx.x, bs = blockDim.x;
    const int njobs = *njobs_p;
    const USlot u = wslot_at(scratch + (size_t)blockIdx.x * slot_bytes, n_layout);
    const size_t region_bytes = item_region_bytes(n_layout);
    // the deferred sources of the jobs in order; source k of the first
    // item_regions has item region k (k_wide_apply counts them the same way)
    auto seg_count = [&](const int32_t q) { return *(const volatile int32_t *)&jobs[q].g.ctl->big_count; };
    auto seg_halted = [&](const int32_t q) { return job_halted(jobs[q]); };
    WorkList wl(njobs, item_regions, pool.wide_next, seg_count, seg_halted, sh);
    while (wl.next()) {
        const UpdateJob &J = jobs[sh.seg];
        GraphCtl *ctl = J.g.ctl;
        const int32_t n = J.g.n;
        const bool lds = n <= lds_cap;
        const RowV R = row_v_of(J);
        const int32_t t_count = *(volatile int32_t *)&ctl->t_count;
        const bool use_tlist = (int64_t)t_count * 8 <= (int64_t)n;
        const BList L{u.bl_t, u.bl_d, u.bl_s, n};
        bool ovf_s = false, ovf_d = false;
        if (tid == 0) {
            sh.nb = 0;
            sh.nf = 0;
        }
        // role 0: old pass, 1: new pass, 2: the whole update of the source
        const int role = sh.role;
        const int32_t region = sh.source;
        const int32_t s = J.g.biglist[sh.item];
        const SrcScal sc = J.g.scal[s];
        int32_t *const pred_row = J.g.pred + (size_t)s * n;
        const int32_t *Dg = J.g.D + (size_t)s * n;
        const uint64_t *Sg = J.g.S + (size_t)s * n;
        __syncthreads();
        if (lds) {
            copy_row<4>(lds_row, Dg, n);
            __syncthreads();
        }
        scan_row<4>(J, R, sc, (sc.flags & 1) != 0, lds ? lds_row : Dg, Sg, use_tlist, t_count, u.q1, n, L, sh,
                    ovf_s, ovf_d);
        if (ovf_s) atomicOr(&ctl->status, ST_SIGMA_OVF);
        if (ovf_d) atomicOr(&ctl->status, ST_DIST_OVF);
        __syncthreads();
        const int32_t nb = sh.nb;
        if (role == 0) {
            const ItemRegion ir = item_region_at(items + (size_t)region * region_bytes, n_layout);
            copy_row<4>(ir.t, u.bl_t, nb);
            copy_row<4>(ir.d, u.bl_d, nb);
            copy_row<4>(ir.s, u.bl_s, nb);
            if (tid == 0) *ir.nb = nb;
        }
        if (nb == 0) continue;
        if (role != 1 && tid == 0) atomicAdd(&ctl->changed_pairs, (unsigned long long)nb);
        // a pass over all of DAG(s) instead of walking back from B where B is
        // an eighth of the row or more: at n = 32768 it takes 245 us whatever
        // B is, a walk 190 from 3000 changed targets and 500 from 10 000; at
        // n = 8192 (with the dependency in LDS too) 56 against 72 from 1400
        const bool full = (int64_t)nb * 8 >= (int64_t)n;
        // where ties outgrow its record the other pass sweeps all of E* and tests
        // it again: that pays only where B is half of the row or more.  Eight
        // updates of 300 sources with 601, 1025 and 2501 changed targets of a row
        // of 3901, 4325 and 5801, 22 DAG arcs per vertex, take 7.7, 8.2 and 10.1 ms;
        // with the sweep from an eighth on and a record filled to the end 46.6,
        // 49.2 and 56.0; with no whole-DAG pass below half of the row 14.7, 15.9
        // and 19.8 (an earlier build)
        const bool sweep = (int64_t)nb * 2 >= (int64_t)n;
        // where the passes use the staged row's LDS: full ones for the counts
        // and (past the expansion arrays) the dependency, walks for their
        // accumulation
        int32_t *const lcnt = lds ? lds_row : nullptr;
        const size_t acc_off = align256((size_t)lds_cap * 4) + align256(XB * (size_t)bs);
        double *const lacc = acc_off + 8 * (size_t)n <= lds_bytes ? (double *)(dyn_lds + acc_off) : nullptr;
        // phase 0: old pass (roles 0 and 2); phase 1: new pass (roles 1 and 2)
        for (int ph = role == 1 ? 1 : 0; ph <= (role == 0 ? 0 : 1); ++ph) {
            const int32_t *Dr = lds ? lds_row : Dg;
            const uint64_t *Sr = Sg;
            const int32_t *Pr = pred_row;
            if (ph == 1) {
                if (role == 1) {
                    // the new row, counts and predecessors: the old ones with the
                    // changed pairs in (the predecessors over the list's counts,
                    // which are in the row by then)
                    int32_t *Dn = lds ? lds_row : u.dnew;
                    if (!lds)
                        for (int32_t t = tid; t < n; t += bs) u.dnew[t] = Dg[t];
                    copy_row<4>(u.snew, Sg, n);
                    __syncthreads();
                    for (int32_t i0 = tid; i0 < nb; i0 += 4 * bs) {
                        int32_t tv[4], pv[4];
#pragma unroll
                        for (int k = 0; k < 4; ++k) tv[k] = i0 + k * bs < nb ? u.bl_t[i0 + k * bs] : -1;
#pragma unroll
                        for (int k = 0; k < 4; ++k) pv[k] = tv[k] >= 0 ? pred_row[tv[k]] : 0;
#pragma unroll
                        for (int k = 0; k < 4; ++k) {
                            const int32_t i = i0 + k * bs, t = tv[k];
                            if (t < 0) continue;
                            const int32_t d = u.bl_d[i];
                            u.snew[t] = u.bl_s[i];
                            u.bl_d[i] = new_pred(J, s, t, pv[k], d < Dn[t]);
                            Dn[t] = d;
                        }
                    }
                    __syncthreads();
                    int32_t *const Pn = (int32_t *)u.bl_s;
                    copy_row<4>(Pn, pred_row, n);
                    __syncthreads();
                    for (int32_t i = tid; i < nb; i += bs) Pn[u.bl_t[i]] = u.bl_d[i];
                    Dr = Dn;
                    Sr = u.snew;
                    Pr = Pn;
                } else {
                    int32_t *Dw = J.g.D + (size_t)s * n;
                    uint64_t *Sw = J.g.S + (size_t)s * n;
                    if (lds) {  // (the old pass used it)
                        copy_row<4>(lds_row, Dg, n);
                        __syncthreads();
                    }
                    for (int32_t i = tid; i < nb; i += bs) {
                        const int32_t t = u.bl_t[i];
                        const int32_t d = u.bl_d[i];
                        pred_row[t] = new_pred(J, s, t, pred_row[t], d < (lds ? lds_row[t] : Dw[t]));
                        Sw[t] = u.bl_s[i];
                        Dw[t] = d;
                        if (lds) lds_row[t] = d;
                    }
                }
                __syncthreads();
            }
            const int32_t *const cp = ph ? J.g.yc_ptr : J.g.xc_ptr, *const ca = ph ? J.g.yc_src : J.g.xc_src,
                          *const cb = ph ? J.g.yc_dst : J.g.xc_dst, *const cw = ph ? J.g.yc_w : J.g.xc_w;
            const double sign = ph ? 1.0 : -1.0;
            if (!full || !full_pass(s, n, Dr, Sr, cp, ca, cw, u.bl_t, nb, u, sign, J.g.bc_delta, Pr, sh, es, lcnt, lacc))
                restricted_pass<false, 2, 4>(s, n, Dr, Sr, cp, ca, cb, cw, u.bl_t, nb, sweep, u, sign, J.g.bc_delta,
                                             Pr, sh, es, dyn_lds, lds_bytes);
        }
    }
}

// Writes the changed pairs (and, by Alg 2, their predecessors) of the deferred
// sources whose two passes ran apart (same item-region assignment as k_source_wide).
__global__ void __launch_bounds__(256) k_wide_apply(const UpdateJob *__restrict__ jobs,
                                                    const int32_t *__restrict__ njobs_p, char *__restrict__ items,
                                                    int32_t item_regions, int32_t n_layout) {
    const int njobs = *njobs_p;
    const size_t region_bytes = item_region_bytes(n_layout);
    int32_t region0 = 0;
    for (int j = 0; j < njobs; ++j) {
        const UpdateJob &J = jobs[j];
        const int32_t n = J.g.n;
        const int32_t count = *(volatile int32_t *)&J.g.ctl->big_count;
        const int32_t paired = min(count, item_regions - region0);
        // a job halted since (or before) the wide kernel ran gets no writes;
        // its regions are still counted, as in k_source_wide
        if (job_halted(J)) {
            region0 += paired;
            continue;
        }
        // a group of gridDim / paired workgroups (at least one) per source,
        // sharing its changed pairs (a few sources can hold tens of thousands
        // each), four in flight per lane
        constexpr int U = 4;
        const int32_t per = paired > 0 ? max(1, (int32_t)gridDim.x / paired) : 1;
        for (int32_t w = blockIdx.x; w < paired * per; w += gridDim.x) {
            const int32_t item = w / per, slice = w % per;
            const ItemRegion ir = item_region_at(items + (size_t)(region0 + item) * region_bytes, n_layout);
            const int32_t s = J.g.biglist[item];
            const int32_t nb = *ir.nb;
            int32_t *Dg = J.g.D + (size_t)s * n;
            uint64_t *Sg = J.g.S + (size_t)s * n;
            int32_t *pred_row = J.g.pred + (size_t)s * n;
            const int32_t stride = per * (int32_t)blockDim.x;
            for (int32_t i0 = slice * (int32_t)blockDim.x + (int32_t)threadIdx.x; i0 < nb; i0 += U * stride) {
                int32_t tv[U], dv[U], od[U], op[U];
                uint64_t sv[U];
#pragma unroll
                for (int k = 0; k < U; ++k) {
                    const int32_t i = i0 + k * stride;
                    tv[k] = -1;
                    if (i < nb) {
                        tv[k] = ir.t[i];
                        dv[k] = ir.d[i];
                        sv[k] = ir.s[i];
                    }
                }
#pragma unroll
                for (int k = 0; k < U; ++k)
                    if (tv[k] >= 0) {
                        od[k] = Dg[tv[k]];
                        op[k] = pred_row[tv[k]];
                    }
#pragma unroll
                for (int k = 0; k < U; ++k)
                    if (tv[k] >= 0) {
                        Dg[tv[k]] = dv[k];
                        Sg[tv[k]] = sv[k];
                        pred_row[tv[k]] = new_pred(J, s, tv[k], op[k], dv[k] < od[k]);
                    }
            }
        }
        region0 += paired;
    }
}

// ------------------------------------------------------------ commit -------

// BC(x) += bc_delta(x) as a compensated (hi, lo) pair (Knuth's two-sum),
// then clears bc_delta, the per-update counters and the step's pool.  Every
// counter is at zero between steps.
__device__ __forceinline__ void commit_job(const UpdateJob &J, const StepPool &pool, const bool replace) {
    const int32_t n = J.g.n;
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < n; t += (int64_t)gridDim.x * blockDim.x) {
        const double d = J.g.bc_delta[t];
        if (replace) {
            J.g.bc_hi[t] = d;
            J.g.bc_lo[t] = 0.0;
        } else if (d != 0.0) {
            const double hi = J.g.bc_hi[t];
            const double s = hi + d;
            const double bp = s - hi;
            double e = (hi - (s - bp)) + (d - bp);
            e += J.g.bc_lo[t];
            const double h2 = s + e;
            J.g.bc_hi[t] = h2;
            J.g.bc_lo[t] = e - (h2 - s);
        }
        J.g.bc_delta[t] = 0.0;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        GraphCtl *c = J.g.ctl;
        c->affected_last = (unsigned long long)c->a_count;
        c->big_last = c->big_count;
        c->changed_last = c->changed_pairs;
        // algorithmic bytes of the row scans: per affected source its
        // distance row (4n) or, with the candidate list, the distances at
        // the candidates (4|T|); sigma is read for the changed pairs only
        const unsigned long long a = (unsigned long long)c->a_count, t = (unsigned long long)c->t_count;
        const bool tl = (int64_t)c->t_count * 8 <= (int64_t)n;
        c->scan_bytes_last = a * 4ull * (tl ? t : (unsigned long long)n) + 8ull * c->changed_pairs;
        if (!replace) {
            c->updates += 1;
            c->affected_total += (unsigned long long)c->a_count;
            c->changed_total += c->changed_pairs;
            c->scan_bytes_total += c->scan_bytes_last;
        }
        c->changed_pairs = 0;
        c->a_count = 0;
        c->t_count = 0;
        c->work_next = 0;
        c->big_count = 0;
        c->dag_count = 0;
        c->dag_back = 0;
        *pool.next = 0;
        *pool.src_next = 0;
        *pool.wide_next = 0;
        *pool.soon = 0;
        if (*(volatile int32_t *)&c->status) *pool.errors = 1;
    }
}

// The static pass's commit: BC = bc_delta.
__global__ void __launch_bounds__(256) k_commit(const UpdateJob *__restrict__ jobs, StepPool pool) {
    commit_job(jobs[0], pool, true);
}

// ------------------------------------------------------------ static pass --

// Distances from every source: a near/far search with the row in LDS
// (Dijkstra's order up to a width `delta` in distance, as in the delta-stepping
// of Meyer and Sanders, 2003, with one near and one far set as in Davidson,
// Baxter, Garland and Owens, 2014; positive weights make any order converge to
// d(s,.)).  A vertex whose distance has fallen since its
// out-arcs were last relaxed has its bit set; a round relaxes the out-arcs of
// the marked vertices below a bound, and when none is left the bound moves to
// the nearest marked vertex plus delta.  With delta three quarters of the mean
// weight the rounds relax 1.27 arcs per arc of an n = 16384 Chung-Lu graph
// (1.15 of an out-degree-8 one) against 4.15 (3.06) for a frontier of all
// improved vertices, in 33 rounds against 20.5.
// The search relaxes the arcs of the set given by tail (ptr, arc): every arc
// of the graph, or a set known or checked to contain E* (Section 6: any arc
// set containing E* gives the same distances).
//
// The marks are two bit sets, near (below the bound) and far; a relaxation that
// lowers a distance sets a bit without waiting for anything.  A round collects
// the near vertices into a queue, a thread per 32 of them, and relaxes their
// out-arcs: a wave takes an equal share of the queue, 64 vertices at most at a
// time, their arc ranges come in one round trip, a prefix sum lays the arcs end
// to end, and a lane finds the owner of its arc by a running maximum over marks
// at the owners' first arcs; so hub and leaf fill the lanes alike (vertices of
// more than SG_DEG arcs are listed in chunks, a wave per chunk).  When no near
// vertex is left the bound moves and far vertices below it become near.
// Distances, marks and queue are in LDS.  All sources of the Chung-Lu graph take
// 9.0 ms, of the n = 4096 out-degree-8 graph 0.41 ms.  What bounds it are VALU
// instructions (busy three quarters of the time): 8 lanes per vertex, or an
// owner search by shuffles with a queue filled by returning atomics, issue
// about 90 per 64 arcs, twice as many, and took 18.7 and 0.75 ms.
constexpr int SG_DEG = 256;       // most arcs of a vertex taken with others'
constexpr int SCHUNK = 256;       // arcs per chunk of a heavier one
constexpr int SHEAVY = 256;       // chunks listed per round (more are relaxed in place)
constexpr int SV_BITS = 18;       // vertex number in a chunk entry
constexpr int SU = 4;             // batches of 64 arcs in flight per wave

// Static LDS (the heavy list and a few words) and dynamic LDS of a search.
constexpr size_t SSSP_STATIC = 4 * SHEAVY + 64;
__host__ __device__ constexpr inline size_t sssp_lds(const size_t n, const size_t qcap, const size_t block, const bool lds) {
    return 2 * 8 * ((n + 63) / 64) + (lds ? 4 * n + 2 * qcap : 4 * qcap) + SU * block;
}

template <bool LDS>
__global__ void __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(6, 8))) k_sssp(
    const GraphPtrs G, const int32_t *__restrict__ ptr, const ArcW *__restrict__ arc, const int32_t delta,
    const int32_t qcap) {
    typedef typename std::conditional<LDS, uint16_t, int32_t>::type Q;
    extern __shared__ __align__(16) char dyn_lds[];
    __shared__ int32_t sh_q[3], sh_heavy[3], sh_min, sh_item;
    __shared__ uint32_t heavy[SHEAVY];
    const int32_t n = G.n;
    const int32_t words = 2 * ((n + 63) >> 6);  // of 32 marks
    uint32_t *const near = (uint32_t *)dyn_lds, *const far = near + words;
    int32_t *const lds_row = (int32_t *)(far + words);
    Q *const queue = (Q *)(lds_row + (LDS ? n : 0));
    GraphCtl *const ctl = G.ctl;
    const int tid = threadIdx.x, bs = blockDim.x, lane = lane_id(), wid = tid >> 6, nw = bs >> 6;
    // this wave's owner marks, one byte per arc of SU batches, kept at zero
    volatile uint8_t *const own_at = (volatile uint8_t *)(queue + qcap) + wid * 64 * SU;
#pragma unroll
    for (int k = 0; k < SU; ++k) own_at[64 * k + lane] = 0;
    bool ovf = false;
    for (int32_t s = (int32_t)blockIdx.x; s < n;) {
        int32_t *const Dg = G.D + (size_t)s * n;
        int32_t *const row = LDS ? lds_row : Dg;
        auto dist = [&](const int32_t v) {
            return LDS ? row[v] : __hip_atomic_load(&row[v], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        };
        int32_t bound = delta;
        // a relaxation whose sum reaches 2^31-1 is dropped; it overflows only
        // if nothing shorter ever reaches its head, which the check after the
        // search settles (long candidates that lose are no error)
        bool long_cand = false;
        auto relax = [&](const ArcW e, const int32_t da) {
            const uint32_t nd = (uint32_t)da + (uint32_t)e.w;
            long_cand |= nd >= (uint32_t)INF32;
            if (nd < (uint32_t)dist(e.v)) {
                // (a distance is at most INF32, so a dropped sum never passes)
                atomicMin(&row[e.v], (int32_t)nd);
                atomicOr(&near[((int32_t)nd < bound ? 0 : words) + (e.v >> 5)], 1u << (e.v & 31));
            }
        };
        for (int32_t i = tid; i < n; i += bs) row[i] = i == s ? 0 : INF32;
        for (int32_t i = tid; i < 2 * words; i += bs) near[i] = i == (s >> 5) ? 1u << (s & 31) : 0u;
        if (tid < 3) {
            sh_q[tid] = 0;
            sh_heavy[tid] = 0;
        }
        __syncthreads();
        for (int32_t r = 0;;) {
            // the near vertices go to the queue, as many as it holds (the
            // others keep their mark)
            for (int32_t w0 = tid - lane; w0 < words; w0 += bs) {
                const int32_t w = w0 + lane;
                uint32_t m = w < words ? near[w] : 0u;
                const int32_t cnt = (int32_t)__popc(m);
                const int32_t incl = wave_incl_add(cnt);
                const int32_t total = __builtin_amdgcn_readlane(incl, 63);
                if (total == 0) continue;
                int32_t base = 0;
                if (lane == 0) base = atomicAdd(&sh_q[r], total);
                base = __builtin_amdgcn_readfirstlane(base);
                if (m) {
                    far[w] &= ~m;
                    int32_t pos = base + incl - cnt;
                    for (; m && pos < qcap; ++pos, m &= m - 1) queue[pos] = (Q)((w << 5) + __ffs(m) - 1);
                    near[w] = m;
                }
            }
            __syncthreads();
            const int32_t q = min(sh_q[r], qcap);
            const int32_t rn = r == 2 ? 0 : r + 1;
            if (tid == 0) {
                sh_q[rn] = 0;
                sh_heavy[rn] = 0;
                sh_min = INF32;
            }
            if (q == 0) {
                // none: the nearest far vertex moves the bound, and those
                // below it become near (a thread keeps to its own words)
                __syncthreads();
                int32_t low = INF32;
                for (int32_t w = tid; w < words; w += bs)
                    for (uint32_t m = far[w]; m; m &= m - 1) low = min(low, dist((w << 5) + __ffs(m) - 1));
                if (low != INF32) atomicMin(&sh_min, low);
                __syncthreads();
                low = sh_min;
                if (low == INF32) break;
                bound = (int32_t)min((uint32_t)low + (uint32_t)delta, (uint32_t)INF32);
                for (int32_t w = tid; w < words; w += bs) {
                    const uint32_t all = far[w];
                    uint32_t below = 0;
                    for (uint32_t m = all; m; m &= m - 1)
                        if (dist((w << 5) + __ffs(m) - 1) < bound) below |= m & (0u - m);
                    if (below) near[w] = below;
                }
                __syncthreads();
                continue;
            }
            // an equal share of the queue per wave, at most a lane per vertex
            const int32_t share = min(64, (q + nw - 1) / nw);
            for (int32_t i0 = wid * share; i0 < q; i0 += nw * share) {
                int32_t e0 = 0, deg = 0, da = 0;
                if (lane < share && i0 + lane < q) {
                    const int32_t a = (int32_t)queue[i0 + lane];
                    e0 = ptr[a];
                    deg = ptr[a + 1] - e0;
                    da = dist(a);
                    if (deg > SG_DEG) {
                        // hubs: listed in chunks, or taken here where the list is full
                        const int32_t chunks = (deg + SCHUNK - 1) / SCHUNK;
                        const int32_t pos = atomicAdd(&sh_heavy[r], chunks);
                        const bool room = pos + chunks <= SHEAVY;
                        for (int32_t c = 0; c < chunks; ++c)
                            if (pos + c < SHEAVY) heavy[pos + c] = room ? (uint32_t)a | (uint32_t)c << SV_BITS : ~0u;
                        if (room) deg = 0;
                    }
                }
                const int32_t incl = wave_incl_add(deg), excl = incl - deg;
                const int32_t total = __builtin_amdgcn_readlane(incl, 63);
                const int32_t first = e0 - excl;  // arc j of the share is arc first + j of its owner
                int32_t last = 0;                 // owner (lane + 1) of the arc before the batch
                for (int32_t j0 = 0; j0 < total; j0 += 64 * SU) {
                    if (deg > 0 && excl >= j0 && excl < j0 + 64 * SU) own_at[excl - j0] = (uint8_t)(lane + 1);
                    ArcW x[SU];
                    int32_t d[SU];
#pragma unroll
                    for (int k = 0; k < SU; ++k) {
                        x[k].w = 0;
                        if (j0 + 64 * k >= total) continue;
                        const int32_t j = j0 + 64 * k + lane;
                        const int32_t own = max(last, wave_incl_max((int32_t)own_at[64 * k + lane]));
                        own_at[64 * k + lane] = 0;
                        last = __builtin_amdgcn_readlane(own, 63);
                        const int32_t at = __builtin_amdgcn_ds_bpermute(4 * (own - 1), first) + j;
                        d[k] = __builtin_amdgcn_ds_bpermute(4 * (own - 1), da);
                        if (j < total) x[k] = arc[at];
                    }
#pragma unroll
                    for (int k = 0; k < SU; ++k)
                        if (x[k].w) relax(x[k], d[k]);
                }
            }
            __syncthreads();
            const int32_t nh = min(sh_heavy[r], SHEAVY);
            if (nh) {
                for (int32_t h = wid; h < nh; h += nw) {
                    const uint32_t c = heavy[h];
                    if (c == ~0u) continue;
                    const int32_t a = (int32_t)(c & ((1u << SV_BITS) - 1));
                    const int32_t e0 = ptr[a] + (int32_t)(c >> SV_BITS) * SCHUNK, e1 = min(ptr[a + 1], e0 + SCHUNK);
                    const int32_t da = dist(a);
                    ArcW x[SCHUNK / 64];
#pragma unroll
                    for (int k = 0; k < SCHUNK / 64; ++k) {
                        const int32_t at = e0 + k * 64 + lane;
                        x[k].w = 0;
                        if (at < e1) x[k] = arc[at];
                    }
#pragma unroll
                    for (int k = 0; k < SCHUNK / 64; ++k)
                        if (x[k].w) relax(x[k], da);
                }
                __syncthreads();
            }
            r = rn;
        }
        if (__syncthreads_or(long_cand)) {
            // converged: a vertex still unreached that has an arc from a
            // reached one is reachable, and every path to it is 2^31-1 or
            // longer
            for (int32_t a = tid; a < n; a += bs) {
                if (dist(a) == INF32) continue;
                const int32_t e1 = ptr[a + 1];
                for (int32_t e = ptr[a]; e < e1; ++e)
                    if (dist(arc[e].v) == INF32) ovf = true;
            }
        }
        if (LDS)
            for (int32_t i = tid; i < n; i += bs) Dg[i] = row[i];
        if (tid == 0) sh_item = (int32_t)gridDim.x + atomicAdd(&ctl->work_next, 1);
        __syncthreads();
        s = sh_item;
        __syncthreads();
    }
    if (ovf) atomicOr(&ctl->status, ST_DIST_OVF);
}

// Check of a searched arc set H against every arc of the graph (by tail in
// arc_ptr / arc), with D the distances the search over H found:
// the arcs (a,b) with w(a,b) <= D(a,b) go to the out list (up to cap; *cnt
// counts them all).  An arc of E* has w(a,b) = d(a,b) <= D(a,b), so it is
// listed unless H holds it; and when every listed arc is in H, no path can
// be shortened by an arc outside H (its weight exceeds the H-distance of its
// ends), so D is the graph's distance matrix and H contains E*.  One wave
// per tail (the tail's arcs and its distance row are contiguous).
__global__ void __launch_bounds__(256) k_search_check(const UpdateJob *__restrict__ jobs, int32_t *__restrict__ out_a,
                                                      int32_t *__restrict__ out_b, int32_t *__restrict__ out_w,
                                                      int64_t cap, unsigned long long *__restrict__ cnt) {
    const UpdateJob &J = jobs[0];
    const int32_t n = J.g.n;
    const int lane = lane_id();
    const int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const int64_t nwaves = ((int64_t)gridDim.x * blockDim.x) >> 6;
    for (int64_t a = wave; a < n; a += nwaves) {
        const int32_t *Da = J.g.D + (size_t)a * n;
        const int32_t p0 = J.g.arc_ptr[a], p1 = J.g.arc_ptr[a + 1];
        for (int32_t base = p0; base < p1; base += 64) {
            const int32_t i = base + lane;
            bool keep = false;
            int32_t b = 0, w = 0;
            if (i < p1) {
                b = J.g.arc[i].v;
                w = J.g.arc[i].w;
                const int32_t d = Da[b];
                keep = d == INF32 || w <= d;
            }
            const uint64_t mask = __ballot(keep);
            if (!mask) continue;
            unsigned long long b0 = 0;
            const int leader = __ffsll((unsigned long long)mask) - 1;
            if (lane == leader) b0 = atomicAdd(cnt, (unsigned long long)__popcll(mask));
            b0 = __shfl(b0, leader, 64);
            if (keep) {
                const unsigned long long o = b0 + popc_below(mask, lane);
                if ((int64_t)o < cap) {
                    out_a[o] = (int32_t)a;
                    out_b[o] = b;
                    out_w[o] = w;
                }
            }
        }
    }
}

// ---------------------------------------------------- static DAG pass ------
//
// Path counts, stored predecessors and dependencies of one source from its
// distance row and E* (one workgroup; Alg 6 step 7 and Alg 1).  An arc (a,b)
// of E* is in DAG(s) iff d(s,a) is finite and d(s,a) + w(a,b) = d(s,b) (Eq.1).
//   1. one coalesced sweep over E* lists the DAG arcs (about one per vertex on
//      weighted graphs), the distance row in LDS;
//   2. the level of every vertex, the longest DAG path from s: relaxations
//      lev(b) >= lev(a) + 1 over the list in LDS until none changes;
//   3. the list sorted by the level of its heads (a counting sort), and the
//      stored predecessors from it;
//   4. levels upwards: sigma_sb = sum of sigma_sa over the DAG arcs (a,b);
//   5. levels downwards: acc(a) = sum of 1/sigma_sb + acc(b), so that
//      delta(a) = sigma_sa * acc(a), and BC(a) gets delta(a) for a != s.
// Every phase is arc-parallel over the list, so a level costs one round trip
// whatever the degrees: all sources of an n = 16384 Chung-Lu graph take 10.3
// ms and those of an n = 4096 out-degree-8 one 0.77 ms, against 108.7 and 4.74
// with a lane per vertex walking its E* out-arcs (up to 32 one after the
// other, per level and direction).
//
// Where the values live: up to ST_VALS vertices counts and accumulators are in
// LDS (8 bytes per vertex, over the distance row's place, which the list
// replaces); up to LDS_ROW_MAX the row and the levels are (4 bytes), counts in
// the state's row and accumulators in the workgroup's slot; above, nothing is.
// The unsorted list sits in the output rows of sigma and the predecessors,
// which are written after the sort.
enum { ST_VAL_LDS = 0, ST_ROW_LDS = 1, ST_GLOBAL = 2 };

// Levels counted in LDS (more are counted in the slot).
constexpr int32_t ST_HIST = 2048;
// Most vertices with 8 bytes each in LDS beside the level counts.
constexpr int32_t ST_VALS = 18432;

// A listed DAG arc: tail and head in one word where vertex numbers fit 16
// bits, else in two.
template <int MODE>
struct DagArc {
    typedef uint32_t T;
    static constexpr int32_t WORDS = 1;
    static __device__ __forceinline__ T make(uint32_t a, uint32_t b) { return a | (b << 16); }
    static __device__ __forceinline__ int32_t tail(T e) { return (int32_t)(e & 0xffffu); }
    static __device__ __forceinline__ int32_t head(T e) { return (int32_t)(e >> 16); }
};
template <>
struct DagArc<ST_GLOBAL> {
    typedef uint2 T;
    static constexpr int32_t WORDS = 2;
    static __device__ __forceinline__ T make(uint32_t a, uint32_t b) { return make_uint2(a, b); }
    static __device__ __forceinline__ int32_t tail(T e) { return (int32_t)e.x; }
    static __device__ __forceinline__ int32_t head(T e) { return (int32_t)e.y; }
};

// The workgroup's slot as the static pass uses it: of the arrays the update
// kernels keep at zero, `bc` (BC terms of all the workgroup's sources) and
// `lev` are handed back at zero; the others need not be.
struct SSlot {
    double *bc, *acc;
    int32_t *lev, *hist;
    void *list;  // 16 n bytes
};

__device__ __forceinline__ SSlot sslot_at(char *base, int32_t n_layout) {
    const UpdateLayout L = update_layout(n_layout);
    SSlot s;
    s.bc = (double *)(base + L.acc);
    s.lev = (int32_t *)(base + L.outdeg);
    s.acc = (double *)(base + L.sub);  // sub and q1
    s.hist = (int32_t *)(base + L.q2);
    s.list = (void *)(base + L.kend);  // kend, ka, kb, kr
    return s;
}

// A source with more DAG arcs than the list holds (three per vertex, 1.5 above
// LDS_ROW_MAX): ties nearly everywhere.  No list: a group of lanes per vertex
// walks its in-arcs in E* or its out-arcs in the searched set (every DAG arc is
// in both) with the Eq.1 test, the distance row in LDS.
//   1. in-arcs of every vertex: their number and the stored predecessor;
//   2. Kahn from s: a frontier's vertices add up their predecessors' path counts
//      and take one off their successors' counts; those that reach zero are the
//      next frontier (the one at the length of the longest path from s);
//   3. the frontiers backwards: acc(a) = sum of 1/sigma_sb + acc(b) over the
//      out-arcs, as in the list's levels.
// So an arc is tested five times whatever the number of levels, and no sum is
// made by atomics.  All sources at n = 2048, out-degree 64, weights 1 and 2 take
// 4.2 ms, at n = 8192 of mean degree 64, weights 1, 61; sweeps over all of E* per
// round and level took 21.9 and 294, a lane per vertex over its out-arcs 7.1 and
// 112.  A chain of 1000 behind 1024 vertices of out-degree 64: 13.7 ms against 653
// and 41 for the recomputation.
// indeg: n words, in LDS (VAL) or the slot's zero-kept ones.
template <int MODE>
__device__ __forceinline__ void static_dense(const GraphPtrs &G, const int32_t s, const int32_t m, const int32_t *Drow,
                                             int32_t *indeg, const SSlot &sl, int32_t *pred, uint64_t *Srow,
                                             BlockShared &sh) {
    constexpr bool VAL = MODE == ST_VAL_LDS;
    const int tid = threadIdx.x, bs = blockDim.x;
    const int32_t n = G.n;
    // lanes per vertex: a quarter of its mean E* in-degree (at least three here),
    // each with U arcs in flight
    constexpr int U = 4;
    int w = 4;
    while (w < 64 && (int64_t)U * w * n < m) w <<= 1;
    const int lane = tid & (w - 1), per = bs / w, mine = tid / w;
    int32_t *const ord = (int32_t *)sl.list, *const ends = sl.hist;
    double *const coef = sl.acc;
    // f gets the other ends of U arcs, -1 for one that is no DAG arc
    auto in_arcs = [&](const int32_t b, auto &&f) {
        const int32_t db = Drow[b], e1 = G.xc_ptr[b + 1];
        for (int32_t e0 = G.xc_ptr[b] + lane; e0 < e1; e0 += U * w) {
            int32_t a[U], wt[U];
#pragma unroll
            for (int k = 0; k < U; ++k) {
                const int32_t e = e0 + k * w;
                a[k] = e < e1 ? G.xc_src[e] : s;
                wt[k] = e < e1 ? G.xc_w[e] : -1;
            }
#pragma unroll
            for (int k = 0; k < U; ++k) {
                const int32_t da = Drow[a[k]];
                if (wt[k] < 0 || da == INF32 || (int64_t)da + wt[k] != (int64_t)db) a[k] = -1;
            }
            f(a);
        }
    };
    auto out_arcs = [&](const int32_t a, auto &&f) {
        const int64_t da = Drow[a];
        const int32_t e1 = G.arc_ptr[a + 1];
        for (int32_t e0 = G.arc_ptr[a] + lane; e0 < e1; e0 += U * w) {
            ArcW x[U];
            int32_t b[U];
#pragma unroll
            for (int k = 0; k < U; ++k) {
                x[k].v = s;
                x[k].w = 0;
                if (e0 + k * w < e1) x[k] = G.arc[e0 + k * w];
            }
#pragma unroll
            for (int k = 0; k < U; ++k) b[k] = x[k].w && da + x[k].w == (int64_t)Drow[x[k].v] ? x[k].v : -1;
            f(b);
        }
    };
    for (int32_t b0 = 0; b0 < n; b0 += per) {
        const int32_t b = b0 + mine;
        int32_t cnt = 0, tail = PRED_NONE;
        if (b < n && Drow[b] != INF32)
            in_arcs(b, [&](const int32_t (&a)[U]) {
#pragma unroll
                for (int k = 0; k < U; ++k) {
                    cnt += a[k] >= 0;
                    tail = max(tail, a[k]);
                }
            });
        for (int o = w >> 1; o >= 1; o >>= 1) {
            cnt += __shfl_xor(cnt, o, 64);
            tail = max(tail, __shfl_xor(tail, o, 64));
        }
        if (b < n && lane == 0) {
            indeg[b] = cnt;
            pred[b] = cnt > 1 ? PRED_MULTI : tail;
            Srow[b] = b == s ? 1ull : 0ull;
        }
    }
    if (tid == 0) {
        ord[0] = s;
        sh.next = 1;
    }
    __syncthreads();
    bool ovf = false;
    int32_t nlev = 0;
    for (int32_t lo = 0, hi = 1; lo < hi; ++nlev) {
        for (int32_t i0 = lo; i0 < hi; i0 += per) {
            const bool on = i0 + mine < hi;
            const int32_t x = on ? ord[i0 + mine] : s;
            uint64_t sum = 0;
            if (on && x != s)
                in_arcs(x, [&](const int32_t (&a)[U]) {
                    uint64_t sg[U];
#pragma unroll
                    for (int k = 0; k < U; ++k) sg[k] = a[k] >= 0 ? Srow[a[k]] : 0;
#pragma unroll
                    for (int k = 0; k < U; ++k) sum = add_chk(sum, sg[k], ovf);
                });
            for (int o = w >> 1; o >= 1; o >>= 1)
                sum = add_chk(sum, (uint64_t)__shfl_xor((unsigned long long)sum, o, 64), ovf);
            if (on && x != s && lane == 0) Srow[x] = sum;
            if (on)
                out_arcs(x, [&](const int32_t (&b)[U]) {
                    int32_t left[U];
#pragma unroll
                    for (int k = 0; k < U; ++k) left[k] = b[k] >= 0 ? atomicSub(&indeg[b[k]], 1) : 0;
#pragma unroll
                    for (int k = 0; k < U; ++k)
                        if (left[k] == 1) ord[atomicAdd(&sh.next, 1)] = b[k];
                });
        }
        if (tid == 0) ends[nlev] = hi;
        __syncthreads();
        lo = hi;
        hi = sh.next;
        __syncthreads();
    }
    if (ovf) atomicOr(&G.ctl->status, ST_SIGMA_OVF);
    for (int32_t f = nlev - 1; f >= 1; --f) {
        const int32_t lo = ends[f - 1], hi = ends[f];
        for (int32_t i0 = lo; i0 < hi; i0 += per) {
            const bool on = i0 + mine < hi;
            const int32_t x = on ? ord[i0 + mine] : s;
            double acc = 0.0;
            if (on)
                out_arcs(x, [&](const int32_t (&b)[U]) {
                    double c[U];
#pragma unroll
                    for (int k = 0; k < U; ++k) c[k] = b[k] >= 0 ? coef[b[k]] : 0.0;
#pragma unroll
                    for (int k = 0; k < U; ++k) acc += c[k];
                });
            for (int o = w >> 1; o >= 1; o >>= 1) acc += __shfl_xor(acc, o, 64);
            if (on && lane == 0) {
                const double sg = (double)Srow[x];
                coef[x] = 1.0 / sg + acc;
                if (acc != 0.0) sl.bc[x] += sg * acc;
            }
        }
        __syncthreads();
    }
    if (!VAL)
        for (int32_t i = tid; i < n; i += bs) indeg[i] = 0;
    if (tid == 0) sh.nlev = nlev;
    __syncthreads();
}

// One source; sh.nlev gets its number of levels.  region: LDS of 8 (ST_VAL_LDS)
// or 4 (ST_ROW_LDS) bytes per vertex; lhist: LDS of lhist_n level counts.
template <int MODE>
__device__ void static_source(const GraphPtrs &G, const int32_t s, const int32_t m, const SSlot &sl, char *region,
                              int32_t *lhist, const int32_t lhist_n, BlockShared &sh) {
    typedef DagArc<MODE> A;
    typedef typename A::T Arc;
    constexpr bool ROW = MODE != ST_GLOBAL, VAL = MODE == ST_VAL_LDS;
    constexpr int U = 4;
    const int tid = threadIdx.x, bs = blockDim.x, lane = lane_id();
    const int32_t n = G.n;
    const int32_t *const Dg = G.D + (size_t)s * n;
    uint64_t *const Srow = G.S + (size_t)s * n;
    int32_t *const pred = G.pred + (size_t)s * n;
    int32_t *const row = (int32_t *)region;
    // the unsorted list, 3 n words: the sigma row's 2 n, then the predecessor row's
    const int32_t cap = 3 * n / A::WORDS;
    auto word = [&](const int32_t p) -> uint32_t & {
        return *(p < 2 * n ? (uint32_t *)Srow + p : (uint32_t *)pred + (p - 2 * n));
    };
    auto put = [&](const int32_t p, const Arc e) {
        if constexpr (A::WORDS == 1) word(p) = e;
        else word(p) = e.x, word(cap + p) = e.y;
    };
    auto get = [&](const int32_t p) {
        if constexpr (A::WORDS == 1) return word(p);
        else return make_uint2(word(p), word(cap + p));
    };
    if (tid == 0) sh.nk = 0;
    if (ROW) copy_row<U>(row, Dg, n);
    __syncthreads();
    // 1. the DAG arcs, four consecutive E* arcs per load, two loads of each kind per
    // lane in flight (one: 20.03 ms for a recompute at n = 16384, two 19.75, three
    // spill and take 20.03)
    auto tight = [&](const int32_t a, const int32_t b, const int32_t w) {
        const int32_t da = ROW ? row[a] : Dg[a], db = ROW ? row[b] : Dg[b];
        return da != INF32 && (int64_t)da + w == (int64_t)db;
    };
    const int4 *const src4 = (const int4 *)G.xc_src, *const dst4 = (const int4 *)G.xc_dst, *const w4 = (const int4 *)G.xc_w;
    const int32_t m4 = (m + 3) >> 2;
    constexpr int Q = 2;
    for (int32_t i0 = tid - lane; i0 < m4; i0 += Q * bs) {
        int av[4 * Q] = {}, bv[4 * Q] = {}, wv[4 * Q] = {};
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const int32_t i = i0 + q * bs + lane;
            if (4 * i + 3 < m) {
                const int4 a = src4[i], b = dst4[i], w = w4[i];
                av[4 * q] = a.x, av[4 * q + 1] = a.y, av[4 * q + 2] = a.z, av[4 * q + 3] = a.w;
                bv[4 * q] = b.x, bv[4 * q + 1] = b.y, bv[4 * q + 2] = b.z, bv[4 * q + 3] = b.w;
                wv[4 * q] = w.x, wv[4 * q + 1] = w.y, wv[4 * q + 2] = w.z, wv[4 * q + 3] = w.w;
            } else if (i < m4) {
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    if (4 * i + k < m) {
                        av[4 * q + k] = G.xc_src[4 * i + k];
                        bv[4 * q + k] = G.xc_dst[4 * i + k];
                        wv[4 * q + k] = G.xc_w[4 * i + k];
                    }
            }
        }
        // (an entry past the end is the arc (0,0) of weight 0: not counted)
        uint32_t mine = 0;
        int32_t before[4 * Q], cnt = 0;
#pragma unroll
        for (int k = 0; k < 4 * Q; ++k) {
            const bool t = wv[k] != 0 && tight(av[k], bv[k], wv[k]);
            const uint64_t mask = __ballot(t);
            mine |= (t ? 1u : 0u) << k;
            before[k] = cnt + (int32_t)popc_below(mask, lane);
            cnt += (int32_t)__popcll(mask);
        }
        if (cnt == 0) continue;
        int32_t base = 0;
        if (lane == 0) base = atomicAdd(&sh.nk, cnt);
        base = __shfl(base, 0, 64);
#pragma unroll
        for (int k = 0; k < 4 * Q; ++k)
            if ((mine >> k) & 1) {
                const int32_t p = base + before[k];
                if (p < cap) put(p, A::make((uint32_t)av[k], (uint32_t)bv[k]));
            }
    }
    __syncthreads();
    const int32_t nt = sh.nk;
    if (nt > cap) {
        static_dense<MODE>(G, s, m, ROW ? row : Dg, VAL ? row + n : sl.lev, sl, pred, Srow, sh);
        return;
    }
    // 2. levels (rounds until none changes; with as many levels as vertices that
    // costs about what a frontier per level does: a recomputation of a chain of
    // 16384 vertices takes 2.15 s against 2.41, of 20000 4.2 against 3.8)
    int32_t *const lev = ROW ? row : sl.lev;
    if (ROW) {
        for (int32_t i = tid; i < n; i += bs) lev[i] = 0;
        __syncthreads();
    }
    auto arcs = [&](auto &&f) {  // the unsorted list, U arcs per lane in flight
        for (int32_t p0 = tid; p0 < nt; p0 += U * bs) {
            Arc e[U];
#pragma unroll
            for (int k = 0; k < U; ++k) e[k] = p0 + k * bs < nt ? get(p0 + k * bs) : A::make(0, 0);
#pragma unroll
            for (int k = 0; k < U; ++k)
                if (p0 + k * bs < nt) f(A::tail(e[k]), A::head(e[k]), e[k]);
        }
    };
    bool changed;
    int32_t top;
    do {
        changed = false;
        top = 0;
        arcs([&](const int32_t a, const int32_t b, const Arc) {
            const int32_t la = shared_value<ROW>(&lev[a]), lb = shared_value<ROW>(&lev[b]);
            top = max(top, max(la + 1, lb));
            if (la >= lb) {
                atomicMax(&lev[b], la + 1);
                changed = true;
            }
        });
        if (tid == 0) sh.nlev = 0;
    } while (__syncthreads_or(changed));
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) top = max(top, __shfl_xor(top, o, 64));
    if (lane == 0) atomicMax(&sh.nlev, top);
    __syncthreads();
    top = sh.nlev;
    // 3. sorted by level: hist[L] counts, then starts, then (after the
    //    placement) ends of level L's arcs; level 0 has none
    Arc *const list = (Arc *)sl.list;
    auto sort = [&](int32_t *hist, auto lds_hist) {
        constexpr bool LH = decltype(lds_hist)::value;
        for (int32_t i = tid; i <= top; i += bs) hist[i] = 0;
        __syncthreads();
        arcs([&](const int32_t, const int32_t b, const Arc) { atomicAdd(&hist[shared_value<ROW>(&lev[b])], 1); });
        __syncthreads();
        int32_t carry = 0;
        for (int32_t c = 0; c <= top; c += bs) {
            const int32_t i = c + tid;
            int32_t total;
            const int32_t off = block_excl_scan(i <= top ? shared_value<LH>(&hist[i]) : 0, sh.scan, total);
            if (i <= top) hist[i] = carry + off;
            carry += total;
        }
        __syncthreads();
        arcs([&](const int32_t, const int32_t b, const Arc e) {
            list[atomicAdd(&hist[shared_value<ROW>(&lev[b])], 1)] = e;
        });
        __syncthreads();
    };
    const bool small = top < lhist_n;
    if (small) sort(lhist, std::true_type{});
    else sort(sl.hist, std::false_type{});
    auto level_end = [&](const int32_t L) { return small ? lhist[L] : shared_value<false>(&sl.hist[L]); };
    // the stored predecessors, built where the levels were
    int32_t *const pt = ROW ? row : pred;
    for (int32_t i = tid; i < n; i += bs) {
        pt[i] = PRED_NONE;
        if (!ROW) lev[i] = 0;
    }
    __syncthreads();
    for (int32_t p = tid; p < nt; p += bs) {
        const Arc e = list[p];
        const int32_t b = A::head(e);
        if (atomicCAS(&pt[b], PRED_NONE, A::tail(e)) != PRED_NONE) pt[b] = PRED_MULTI;
    }
    __syncthreads();
    if (ROW) {
        for (int32_t i = tid; i < n; i += bs) pred[i] = pt[i];
        __syncthreads();
    }
    // 4. path counts
    uint64_t *const sig = VAL ? (uint64_t *)region : Srow;
    for (int32_t i = tid; i < n; i += bs) sig[i] = i == s ? 1ull : 0ull;
    __syncthreads();
    bool ovf = false;
    for (int32_t L = 1; L <= top; ++L) {
        const int32_t p1 = level_end(L);
        for (int32_t p = level_end(L - 1) + tid; p < p1; p += bs) {
            const Arc e = list[p];
            const uint64_t sa = shared_value<VAL>(&sig[A::tail(e)]);
            const uint64_t old = atomicAdd((unsigned long long *)&sig[A::head(e)], (unsigned long long)sa);
            if (old + sa < old) ovf = true;
        }
        __syncthreads();
    }
    if (ovf) atomicOr(&G.ctl->status, ST_SIGMA_OVF);
    // 5. dependencies
    double *const acc = VAL ? (double *)region : sl.acc;
    for (int32_t i = tid; i < n; i += bs) {
        if (VAL) Srow[i] = sig[i];
        acc[i] = 0.0;
    }
    __syncthreads();
    for (int32_t L = top; L >= 1; --L) {
        const int32_t p1 = level_end(L);
        for (int32_t p = level_end(L - 1) + tid; p < p1; p += bs) {
            const Arc e = list[p];
            const int32_t b = A::head(e);
            const uint64_t sb = VAL ? Srow[b] : shared_value<false>(&Srow[b]);
            atomicAdd(&acc[A::tail(e)], 1.0 / (double)sb + shared_value<VAL>(&acc[b]));
        }
        __syncthreads();
    }
    for (int32_t i = tid; i < n; i += bs) {
        const double ax = shared_value<VAL>(&acc[i]);
        if (ax != 0.0 && i != s) sl.bc[i] += (double)(VAL ? Srow[i] : shared_value<false>(&Srow[i])) * ax;
    }
    if (tid == 0) sh.nlev = top + 1;
    __syncthreads();
}

// Every source after the distances and E* exist (static_source); persistent
// workgroups, BC terms summed per workgroup in its slot and added up at the end.
template <int MODE>
__global__ void __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(5, 8))) k_static(const GraphPtrs G, char *__restrict__ scratch, size_t slot_bytes,
                                                 int32_t lhist_n, int32_t n_layout) {
    extern __shared__ __align__(16) char dyn_lds[];
    __shared__ BlockShared sh;
    GraphCtl *const ctl = G.ctl;
    if ((*(volatile int32_t *)&ctl->status & ST_ESTAR_CAP) != 0) return;
    const SSlot sl = sslot_at(scratch + (size_t)blockIdx.x * slot_bytes, n_layout);
    const int32_t n = G.n, m = ctl->esc_m;
    int32_t *const lhist = (int32_t *)dyn_lds;
    char *const region = dyn_lds + align256(4 * (size_t)lhist_n);
    int32_t nlev = 0;
    for (int32_t s = (int32_t)blockIdx.x; s < n;) {
        static_source<MODE>(G, s, m, sl, region, lhist, lhist_n, sh);
        nlev = max(nlev, sh.nlev);
        if (threadIdx.x == 0) sh.item = (int32_t)gridDim.x + atomicAdd(&ctl->work_next, 1);
        __syncthreads();
        s = sh.item;
    }
    for (int32_t i = threadIdx.x; i < n; i += blockDim.x) {
        const double v = sl.bc[i];
        if (v != 0.0) {
            atomicAdd(&G.bc_delta[i], v);
            sl.bc[i] = 0.0;
        }
    }
    if (threadIdx.x == 0) atomicMax(&ctl->max_levels, nlev);
}

__global__ void k_reset_work(GraphCtl *ctl) {
    ctl->work_next = 0;
    ctl->a_count = 0;
}

// ------------------------------------------------------------ introspection

// Dependency row of one source, delta_s.(x) = sum over all reachable t of
// delta_st(x), by the same restricted pass with B = every reachable t != s.
// Writes the row to out_row (n values, 0 at s and at unreachable x).  One
// workgroup; `scratch` is one wide-kernel slot laid out for n_layout >= n.
__device__ __forceinline__ void delta_row(const GraphPtrs &G, int32_t s, char *__restrict__ scratch, int32_t lds_cap,
                                          int32_t n_layout, double *out_row) {
    extern __shared__ __align__(16) char dyn_lds[];
    int32_t *const lds_row = (int32_t *)dyn_lds;
    const ExpandShared es = expand_at(dyn_lds, lds_cap);
    __shared__ BlockShared sh;
    const int32_t n = G.n;
    const bool lds = n <= lds_cap;
    const USlot u = wslot_at(scratch, n_layout);
    if ((*(volatile int32_t *)&G.ctl->status & ST_ESTAR_CAP) != 0) return;
    const int32_t *Dg = G.D + (size_t)s * n;
    const int32_t *Drow = Dg;
    if (threadIdx.x == 0) sh.nb = 0;
    __syncthreads();
    for (int32_t t = threadIdx.x; t < n; t += blockDim.x) {
        out_row[t] = 0.0;
        if (lds) lds_row[t] = Dg[t];
        if (t != s && Dg[t] != INF32) u.bl_t[atomicAdd(&sh.nb, 1)] = t;
    }
    if (lds) Drow = lds_row;
    __syncthreads();
    restricted_pass<true, XU>(s, n, Drow, G.S + (size_t)s * n, G.xc_ptr, G.xc_src, G.xc_dst, G.xc_w, u.bl_t, sh.nb,
                              true, u, 1.0, out_row, nullptr, sh, es);
}

__global__ void __launch_bounds__(1024) k_delta_row(const UpdateJob *__restrict__ jobs, int32_t s, char *__restrict__ scratch,
                                                    int32_t lds_cap, int32_t n_layout, double *out_row) {
    delta_row(jobs[0].g, s, scratch, lds_cap, n_layout, out_row);
}

// The same with the graph's pointers passed by value (no staged job) and the
// slot in the caller-supplied scratch address (the library's fixed array).
__global__ void __launch_bounds__(1024) k_delta_row_byval(const GraphPtrs G, int32_t s, char *__restrict__ scratch,
                                                          int32_t lds_cap, int32_t n_layout, double *out_row) {
    delta_row(G, s, scratch, lds_cap, n_layout, out_row);
}

// The ranges of a graph's arena that a clone takes over, each of 256-byte
// pieces, at the same place in both arenas.  Bound by HBM: four 16-byte loads
// per thread in flight, with STREAM past the caches (the runtime's copy of all of
// the arena took 8.3 ms at n = 32768, 4.15 TB/s; this takes 7.0, 4.95 TB/s).
struct CopyRanges {
    int32_t count;
    size_t off[5], bytes[5];
};
template <bool STREAM>
__global__ void __launch_bounds__(256) k_copy_ranges(char *__restrict__ dst, const char *__restrict__ src,
                                                     const CopyRanges c) {
    typedef int v4i __attribute__((ext_vector_type(4)));
    constexpr int U = 4;
    for (int r = 0; r < c.count; ++r) {
        const v4i *const from = (const v4i *)(src + c.off[r]);
        v4i *const to = (v4i *)(dst + c.off[r]);
        const size_t words = c.bytes[r] / 16, step = (size_t)gridDim.x * blockDim.x * U;
        for (size_t i0 = (size_t)blockIdx.x * blockDim.x * U + threadIdx.x; i0 < words; i0 += step) {
            v4i v[U];
#pragma unroll
            for (int k = 0; k < U; ++k)
                if (i0 + k * blockDim.x < words)
                    v[k] = STREAM ? __builtin_nontemporal_load(from + i0 + k * blockDim.x) : from[i0 + k * blockDim.x];
#pragma unroll
            for (int k = 0; k < U; ++k)
                if (i0 + k * blockDim.x < words) {
                    if (STREAM) __builtin_nontemporal_store(v[k], to + i0 + k * blockDim.x);
                    else to[i0 + k * blockDim.x] = v[k];
                }
        }
    }
}

// Zero fill of a byte range (the fixed scratch array at set-up).
__global__ void __launch_bounds__(256) k_zero_fill(char *__restrict__ p, size_t bytes) {
    const size_t words = bytes / 8;
    uint64_t *q = (uint64_t *)p;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < words; i += (size_t)gridDim.x * blockDim.x)
        q[i] = 0;
}

// Sticky status words of up to STATUS_GATHER graphs gathered into one device
// array by one launch, so that reading back many graphs' errors costs one
// launch and one copy instead of a copy per graph.
constexpr int STATUS_GATHER = 64;
struct StatusPtrs {
    const int32_t *p[STATUS_GATHER];
};
__global__ void __launch_bounds__(STATUS_GATHER) k_gather_status(const StatusPtrs a, int32_t count,
                                                                 int32_t *__restrict__ out) {
    const int i = threadIdx.x;
    if (i < count) out[i] = *(const volatile int32_t *)a.p[i];
}

// Arcs of DAG(s): the predicate of Eq.1 over E*.
__global__ void k_dag_arcs(const UpdateJob *__restrict__ jobs, int32_t s, int32_t *out_a, int32_t *out_b, int64_t cap,
                           unsigned long long *cnt) {
    const UpdateJob &J = jobs[0];
    if (job_dead(J)) return;
    const int32_t n = J.g.n, m = J.g.ctl->esc_m;
    const int32_t *Drow = J.g.D + (size_t)s * n;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < m; i += (int64_t)gridDim.x * blockDim.x) {
        const int32_t a = J.g.xc_src[i], b = J.g.xc_dst[i];
        const int32_t da = Drow[a], db = Drow[b];
        if (da != INF32 && db != INF32 && (int64_t)da + J.g.xc_w[i] == (int64_t)db) {
            const unsigned long long k = atomicAdd(cnt, 1ull);
            if ((int64_t)k < cap) {
                out_a[k] = a;
                out_b[k] = b;
            }
        }
    }
}

__device__ __forceinline__ uint64_t mix64(uint64_t z) {
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

// Order-independent 2 x 64-bit hash of (D, sigma): sums of mixed
// (index, value) words, which commute, so the result is bit-exact.
__global__ void k_hash(const UpdateJob *__restrict__ jobs, unsigned long long *out) {
    const UpdateJob &J = jobs[0];
    const int64_t nn = (int64_t)J.g.n * J.g.n;
    uint64_t h0 = 0, h1 = 0;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nn; i += (int64_t)gridDim.x * blockDim.x) {
        h0 += mix64(((uint64_t)i << 32) ^ (uint32_t)J.g.D[i] ^ 0x5bd1e995ull);
        h1 += mix64((uint64_t)i * 0x9E3779B97F4A7C15ull + J.g.S[i]);
    }
    for (int d = 32; d >= 1; d >>= 1) {
        h0 += (uint64_t)__shfl_down((unsigned long long)h0, d, 64);
        h1 += (uint64_t)__shfl_down((unsigned long long)h1, d, 64);
    }
    if (lane_id() == 0) {
        atomicAdd(&out[0], (unsigned long long)h0);
        atomicAdd(&out[1], (unsigned long long)h1);
    }
}

}  // namespace bcinc
