// pg_edges.hip -- aggregation operators (edge weights, direct terms) and the
// per-path pass (successors, predecessors, path-traced initial estimate).
//
// Paper Sec. "Path Graph Operators": each neighbour of a receiver is a
// sampling technique; its continuation sample is combined with the balance
// heuristic over all techniques of the receiver's neighbourhood (eqs.
// indirect-weight, ag-indirect), and the direct-light records form 2K samples
// from K+1 strategies (eq. ag-direct).  The pdfs of the techniques are HG
// with parameter g_s about each neighbour's arriving direction; the receiver
// evaluates its own phase function (HG with g about its arriving direction).
#include "pg_internal.h"

namespace pg {

// One group of KP lanes per receiver, lane j = j-th neighbour.  The
// neighbours' arriving directions (the techniques) are staged in LDS; every
// lane sums the K technique pdfs at its own two samples (continuation and
// environment) to get the marginals, then forms its three weights; the
// direct term is a group reduction, which one thread a row turns into the
// vertex's terms.
//
// Bound by the vector instructions: K pairs of densities a lane and what is done
// once a row.  With the row's terms in its group (instructions for one lane of
// 16) and sums by way of the LDS, 20M rows (K = 16) took 5.45 ms, now 4.60; 3.8M in
// path order (K = 13), where the gathers come in between, 1.18 and 1.12 ms.
template <int KP>
__global__ __launch_bounds__(kBlock) void k_edges(int64_t N, Consts c, const int32_t* __restrict__ col,
                                                  const VRec* __restrict__ rec, EdgeOut o, int32_t* flag) {
    constexpr int GR = kBlock / KP;
    __shared__ f3 tsh[GR][KP];
    __shared__ f3 csum[GR], ssum[GR], qsum[GR];
    __shared__ int own[GR];
    const int64_t tile = xcd_tile(blockIdx.x, gridDim.x);
    const int lane = threadIdx.x % KP, grp = threadIdx.x / KP;
    const int64_t i = tile * GR + grp;
    const int K = c.K;
    const bool row_ok = i < N;
    bool act = row_ok && lane < K;

    RecRegs n;   // of the neighbour
    f3 dpl{0.f, 0.f, 0.f}, lpl{0.f, 0.f, 0.f};   // point light sample of the neighbour
    const int64_t e = o.ell ? eidx(i, lane, K) : i * K + lane;
    if (act) {
        int64_t j = col[e];
        if (j < 0 || j >= N || (lane == 0 && j != i)) {
            set_flag(flag, kFlagIndex);
            act = false;
        } else {
            n.load(rec + j);
            if (o.dir_pl) {
                const int64_t cj = o.canon_row ? (int64_t)o.canon_row[j] : j;
                dpl = ld3(o.dir_pl, cj);
                lpl = ld3(o.l_pl, cj);
            }
        }
    }
    tsh[grp][lane] = n.t;
    __syncthreads();
    const f3 ti = tsh[grp][0];

    float mplus = 0.0f, menv = 0.0f;
    for (int l = 0; l < K; ++l) {
        const f3 tl = tsh[grp][l];
        mplus += c.pdf.between(tl, n.w);
        menv += c.pdf.between(tl, n.we);
    }
    const float Kpe = (float)K * c.env_pdf;
    const float u_w = one_minus_cos(ti, n.w), u_e = one_minus_cos(ti, n.we);
    const float rho = c.rho(u_w), rho_e = c.rho(u_e);
    const float wi = rho / mplus;
    const float wp = rho / (mplus + Kpe);
    const float wev = rho_e / (menv + Kpe);

    float cx = act ? wev * n.le.x + wp * n.lp.x : 0.0f;
    float cy = act ? wev * n.le.y + wp * n.lp.y : 0.0f;
    float cz = act ? wev * n.le.z + wp * n.lp.z : 0.0f;
    float sx = act ? n.ls.x : 0.0f, sy = act ? n.ls.y : 0.0f, sz = act ? n.ls.z : 0.0f;
    cx = group_sum<KP>(cx);
    cy = group_sum<KP>(cy);
    cz = group_sum<KP>(cz);
    sx = group_sum<KP>(sx);
    sy = group_sum<KP>(sy);
    sz = group_sum<KP>(sz);
    // point light: a delta light per neighbour sample, weight 1/K
    const float rho_pl = (act && o.dir_pl) ? c.rho(one_minus_cos(ti, dpl)) : 0.0f;
    float qx = rho_pl * lpl.x, qy = rho_pl * lpl.y, qz = rho_pl * lpl.z;
    if (o.dir_pl) {
        qx = group_sum<KP>(qx);
        qy = group_sum<KP>(qy);
        qz = group_sum<KP>(qz);
    }

    if (o.ell && row_ok && lane == 0) {   // padding slots of the last quad: weight 0
        for (int l = K; l < ell_k4(K); ++l) {
            o.w[eidx(i, l, K)] = 0.0f;
            if (o.gw) o.gw[eidx(i, l, K)] = 0.0f;
        }
    }
    if (act) {
        o.w[e] = wi;
        if (o.gw) o.gw[e] = wi * hg_dlog(c.g, u_w);
        if (o.canon_row || o.w_ind || o.w_ph || o.w_env) {
            const int64_t ce = (o.canon_row ? (int64_t)o.canon_row[i] : i) * K + lane;
            if (o.w_ind) o.w_ind[ce] = wi;
            if (o.w_ph) o.w_ph[ce] = wp;
            if (o.w_env) o.w_env[ce] = wev;
        }
    }
    if (lane == 0) {
        csum[grp] = f3{cx, cy, cz};
        ssum[grp] = f3{sx, sy, sz};
        if (o.dir_pl) qsum[grp] = f3{qx, qy, qz};
        own[grp] = act;
    }
    __syncthreads();
    const int f = finished_row<GR>();
    const int64_t v = tile * GR + f;
    if (f < 0 || v >= N) return;
    const f3 tv = tsh[f][0], cs = csum[f], ss = ssum[f];
    RecRegs m;   // the vertex's own
    if (own[f]) m.load(rec + v);
    if (o.succ) o.succ[v] = -1;
    if (o.pred) o.pred[v] = -1;
    if (o.x0) st3(o.x0, v, f3{0.f, 0.f, 0.f});
    const int64_t cv = o.canon_row ? (int64_t)o.canon_row[v] : v;
    // aggregated direct: sun (delta light, weight 1/K per neighbour) + MIS'd records
    const float rho_sun = c.rho(one_minus_cos(tv, c.sun));
    const float invK = 1.0f / (float)K;
    f3 dagg{fmaf(rho_sun * invK, ss.x, cs.x), fmaf(rho_sun * invK, ss.y, cs.y), fmaf(rho_sun * invK, ss.z, cs.z)};
    if (o.dir_pl) {
        const f3 qs = qsum[f];
        dagg = f3{fmaf(invK, qs.x, dagg.x), fmaf(invK, qs.y, dagg.y), fmaf(invK, qs.z, dagg.z)};
    }
    // constant of the row: the vertex's own volume emission (not scattered) + alpha d_agg
    f3 em{0.f, 0.f, 0.f};
    if (o.emit) em = ld3(o.emit, cv);
    const f3 b{fmaf(m.alpha, dagg.x, em.x), fmaf(m.alpha, dagg.y, em.y), fmaf(m.alpha, dagg.z, em.z)};
    // own (path-traced) direct: one sun sample, environment and phase samples by the balance heuristic
    const float o_w = one_minus_cos(tv, m.w), o_e = one_minus_cos(tv, m.we);
    const float rho_w = c.rho(o_w), p_w = c.pdf(o_w), p_e = c.pdf(o_e);
    const float f_env = c.rho(o_e) / (p_e + c.env_pdf), f_out = rho_w / (p_w + c.env_pdf);
    f3 dpt{rho_sun * m.ls.x + f_env * m.le.x + f_out * m.lp.x, rho_sun * m.ls.y + f_env * m.le.y + f_out * m.lp.y,
           rho_sun * m.ls.z + f_env * m.le.z + f_out * m.lp.z};
    if (o.dir_pl && own[f]) {   // the receiver's own sample
        const float rp = c.rho(one_minus_cos(tv, ld3(o.dir_pl, cv)));
        const f3 lq = ld3(o.l_pl, cv);
        dpt = f3{fmaf(rp, lq.x, dpt.x), fmaf(rp, lq.y, dpt.y), fmaf(rp, lq.z, dpt.z)};
    }
    if (o.b) st3(o.b, v, b);
    if (o.dpt) st3(o.dpt, v, dpt);
    const float r = rho_w / p_w;
    if (o.r) o.r[v] = r;
    if (o.alpha) o.alpha[v] = m.alpha;
    if (o.step)
        o.step[v] = make_float4(fmaf(m.alpha, dpt.x, em.x), fmaf(m.alpha, dpt.y, em.y), fmaf(m.alpha, dpt.z, em.z),
                                m.alpha * r);
    if (o.b_canon) st3(o.b_canon, cv, b);
    if (o.dpt_canon) st3(o.dpt_canon, cv, dpt);
}

hipError_t launch_edges(int64_t N, const Consts& c, const int32_t* col, const VRec* rec, const EdgeOut& o,
                        int32_t* flag, hipStream_t s) {
    if (N == 0) return hipSuccess;
    dispatch_kp(c.K, [&](auto kp) {
        constexpr int KP = decltype(kp)::value;
        hipLaunchKernelGGL(k_edges<KP>, dim3((unsigned)div_up(N, kBlock / KP)), dim3(kBlock), 0, s, N, c, col,
                           rec, o, flag);
    });
    return hipGetLastError();
}

// One wave per path.  Writes, in local ids, succ(v) / pred(v) (-1 at the
// ends) and the initial radiance arriving from the successor u along the
// continuation: 0 at the last vertex, else e_u + albedo_u (d_pt_u + r_u L(u))
// -- the path tracer's own estimate (init PT) -- or e_u alone (init zero: the
// indirect part starts at 0), e_u being the volume emission collected at u
// (emit, path order, nullable: 0).  The recurrence L(v) = F_u(L(u)), F_u an
// affine map, is taken 64 vertices at a time from the path's end: lane c
// holds vertex hi - c, a wave-level inclusive scan composes the lanes' maps
// (F(L) = A + B L; F2 o F1 = (A2 + B2 A1, B2 B1)), and each lane applies
// the composition of the lanes above it to the value arriving at the chunk.
// succ, pred and x0 must hold -1, -1, 0 (k_edges or fills).
//
// Bound by its scattered accesses, a memory line each: the vertex's map comes in one
// 16-byte piece (step) instead of from albedo, d_pt and r, 20M vertices 1.50 ->
// 0.94 ms.
__global__ __launch_bounds__(kBlock) void k_paths(int64_t P, int64_t N, const int64_t* __restrict__ off,
                                                  const int32_t* __restrict__ inv, const float4* __restrict__ step,
                                                  const float* __restrict__ emit, int init,
                                                  int32_t* __restrict__ succ, int32_t* __restrict__ pred,
                                                  float* __restrict__ x0, int32_t* flag) {
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t p = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / kWave;   // uniform over the wave
    if (p == 0 && lane == 0 && (off[0] != 0 || off[P] != N)) set_flag(flag, kFlagOffsets);
    if (p >= P) return;
    const int64_t a = off[p], e = off[p + 1];
    if (a < 0 || e < a || e > N) {
        if (lane == 0) set_flag(flag, kFlagOffsets);
        return;
    }
    const bool pt = init == PG_INIT_PT && x0;
    const bool ez = !pt && emit && x0;   // init zero with emission
    auto sid = [&](int64_t u) { return inv ? inv[u] : (int32_t)u; };
    f3 carry{0.f, 0.f, 0.f};   // the value arriving at the chunk's highest vertex
    for (int64_t hi = e - 1; hi >= a; hi -= kWave) {
        const int64_t v = hi - lane;
        const bool valid = v >= a;
        const int32_t s = valid ? sid(v) : -1;
        if (valid) {
            if (succ) succ[s] = v + 1 < e ? sid(v + 1) : -1;
            if (pred) pred[s] = v > a ? sid(v - 1) : -1;
        }
        if (!pt && !ez) continue;
        // this vertex's map: the value arriving at its predecessor from the
        // value arriving at it (identity on the lanes past the path's start)
        float B = 1.0f;
        f3 A{0.f, 0.f, 0.f};
        if (valid) {
            if (pt) {
                const float4 m = step[s];
                A = f3{m.x, m.y, m.z};
                B = m.w;
            } else {
                A = ld3(emit, v);
                B = 0.0f;
            }
        }
        // inclusive scan: lane c composes the maps of lanes 0..c (lane c's
        // applied last)
#pragma unroll
        for (int o = 1; o < kWave; o <<= 1) {
            const float Bo = __shfl_up(B, o, kWave);
            const float Ax = __shfl_up(A.x, o, kWave), Ay = __shfl_up(A.y, o, kWave), Az = __shfl_up(A.z, o, kWave);
            if (lane >= o) {
                A = f3{fmaf(B, Ax, A.x), fmaf(B, Ay, A.y), fmaf(B, Az, A.z)};
                B *= Bo;
            }
        }
        // exclusive: the lanes above this one, applied to the carry
        // every lane takes part in the shuffles (a lane inactive in one
        // gives no data to its neighbour), then lane 0 takes the identity
        const float Bsh = __shfl_up(B, 1, kWave);
        const float Be = lane > 0 ? Bsh : 1.0f;
        const float Aex = __shfl_up(A.x, 1, kWave), Aey = __shfl_up(A.y, 1, kWave), Aez = __shfl_up(A.z, 1, kWave);
        const f3 Ae = lane > 0 ? f3{Aex, Aey, Aez} : f3{0.f, 0.f, 0.f};
        if (valid) st3(x0, s, f3{fmaf(Be, carry.x, Ae.x), fmaf(Be, carry.y, Ae.y), fmaf(Be, carry.z, Ae.z)});
        // the value arriving at the next chunk's highest vertex (the whole
        // chunk's composition, held by lane 63)
        const float Bl = __shfl(B, kWave - 1, kWave);
        const f3 Al{__shfl(A.x, kWave - 1, kWave), __shfl(A.y, kWave - 1, kWave), __shfl(A.z, kWave - 1, kWave)};
        carry = f3{fmaf(Bl, carry.x, Al.x), fmaf(Bl, carry.y, Al.y), fmaf(Bl, carry.z, Al.z)};
    }
}

hipError_t launch_paths(int64_t P, int64_t N, const int64_t* off, const int32_t* inv, const float4* step,
                        const float* emit, int init, int32_t* succ, int32_t* pred, float* x0, int32_t* flag,
                        hipStream_t s) {
    const int64_t n = P > 0 ? P : 1;
    hipLaunchKernelGGL(k_paths, dim3((unsigned)div_up(n * kWave, kBlock)), dim3(kBlock), 0, s, P, N, off, inv, step,
                       emit, init, succ, pred, x0, flag);
    return hipGetLastError();
}

}  // namespace pg
