// pg_trace.hip -- the instrumented delta-tracking volume path tracer on the
// GPU: the upstream step that produces the path-ordered vertex records (paper
// Sec. "Volume Path Tracing"; Sec. "Rendering System", instrumented path
// tracer: per shading point the emitter-sampling and phase-sampling data and
// the radiance of its continuation), written straight into HBM.
//
// Medium: a grid of extinction coefficients over the unit cube (nearest
// voxel, x fastest), vacuum outside; albedo per voxel or constant.  Lights:
// a directional (delta) sun and a constant environment.  Per path: a camera
// ray through the pixel (jittered), analog delta tracking against the grid
// majorant; at every real collision a sun shadow ray and one uniform-sphere
// environment shadow ray, both with ratio-tracking transmittance, and a
// continuation sampled from Henyey-Greenstein about the arriving direction;
// at most max_depth vertices, the last without continuation; no Russian
// roulette.  Random numbers: PCG32 (O'Neill 2014), one stream per pixel of
// the full image, seeded from (seed, sample index) through splitmix64, so a
// crop traces the paths the full image traces there.
//
// Double precision without contraction, one path per lane at a time; a lane
// whose path has ended takes the next one from a queue.  The counting pass
// traces each path into max_depth record slots of its own in the workspace; a
// scan gives the offsets, and the record pass copies each path's records to its
// offsets.
#include <algorithm>
#include <cmath>

#include "pg_api_common.h"
#include "pg_quotient.h"

#pragma clang fp contract(off)

namespace pg {

namespace {

struct Rng {
    uint64_t state, inc;
    __device__ uint32_t next() {
        const uint64_t old = state;
        state = old * 6364136223846793005ull + inc;
        const uint32_t xs = (uint32_t)(((old >> 18u) ^ old) >> 27u);
        const uint32_t rot = (uint32_t)(old >> 59u);
        return (xs >> rot) | (xs << ((0u - rot) & 31u));
    }
    __device__ void seed(uint64_t initstate, uint64_t initseq) {
        state = 0u;
        inc = (initseq << 1u) | 1u;
        (void)next();
        state += initstate;
        (void)next();
    }
    __device__ double uniform() { return (double)next() * (1.0 / 4294967296.0); }   // [0, 1), 32 bits
};

__device__ inline uint64_t splitmix64(uint64_t x) {
    x += 0x9E3779B97F4A7C15ull;
    x = (x ^ (x >> 30)) * 0xBF58476D1CE4E5B9ull;
    x = (x ^ (x >> 27)) * 0x94D049BB133111EBull;
    return x ^ (x >> 31);
}

struct D3 {
    double x, y, z;
};
__device__ inline D3 d3(double x, double y, double z) { return D3{x, y, z}; }
__device__ inline double comp(const D3& v, int a) { return a == 0 ? v.x : (a == 1 ? v.y : v.z); }

__device__ inline D3 normalized(D3 v) {
    const double l = sqrt(v.x * v.x + v.y * v.y + v.z * v.z);
    return d3(v.x / l, v.y / l, v.z / l);
}

struct Tracer {
    pg_tracer t;
    int cw, ch, cx0, cy0;
    int point_light;
    // camera frame
    D3 f, r, up;
    double th, aspect;
    double inv_maj;   // 1 / t.majorant, correctly rounded
};

__device__ inline size_t voxel_of(const pg_tracer& t, const D3& p) {
    int i[3];
    for (int a = 0; a < 3; ++a) {
        const int v = (int)floor(comp(p, a) * t.R);
        i[a] = v < 0 ? 0 : (v >= t.R ? t.R - 1 : v);
    }
    return ((size_t)i[2] * t.R + i[1]) * t.R + i[0];
}

__device__ inline double sigma_at(const pg_tracer& t, const D3& p) { return (double)t.sigma[voxel_of(t, p)]; }

__device__ inline double albedo_at(const pg_tracer& t, const D3& p) {
    return t.albedo ? (double)t.albedo[voxel_of(t, p)] : t.albedo_const;
}

// Ray / unit-cube slab test: 1 and [t0, t1] (t0 may be < 0) on a hit.
__device__ inline int box_hit(const D3& o, const D3& d, double& t0, double& t1) {
    double lo = -INFINITY, hi = INFINITY;
    for (int a = 0; a < 3; ++a) {
        const double oa = comp(o, a), da = comp(d, a);
        if (da == 0.0) {
            if (oa < 0.0 || oa > 1.0) return 0;
            continue;
        }
        const double inv = 1.0 / da;
        double ta = (0.0 - oa) * inv, tb = (1.0 - oa) * inv;
        if (ta > tb) {
            const double tt = ta;
            ta = tb;
            tb = tt;
        }
        if (ta > lo) lo = ta;
        if (tb < hi) hi = tb;
    }
    if (hi < lo || hi <= 0.0) return 0;
    t0 = lo;
    t1 = hi;
    return 1;
}

__device__ inline double exit_distance(const D3& o, const D3& d) {
    double t0 = 0.0, t1 = 0.0;
    if (!box_hit(o, d, t0, t1)) return 0.0;
    return t1 > 0.0 ? t1 : 0.0;
}

// Orthonormal basis around unit n (Duff et al. 2017).
__device__ inline void onb(const D3& n, D3& b1, D3& b2) {
    const double s = n.z >= 0.0 ? 1.0 : -1.0;
    const double a = -1.0 / (s + n.z);
    const double b = n.x * n.y * a;
    b1 = d3(1.0 + s * n.x * n.x * a, s * b, -s * n.x);
    b2 = d3(b, s + n.y * n.y * a, -n.y);
}

// Direction whose cosine with the travel direction t follows HG(g) (inversion).
__device__ inline D3 sample_hg(const D3& t, double g, double u1, double u2) {
    double mu;
    if (fabs(g) < 1e-3) {
        mu = 1.0 - 2.0 * u1;
    } else {
        const double s = (1.0 - g * g) / (1.0 - g + 2.0 * g * u1);
        mu = (1.0 + g * g - s * s) / (2.0 * g);
    }
    if (mu > 1.0) mu = 1.0;
    if (mu < -1.0) mu = -1.0;
    const double st = sqrt(fmax(0.0, 1.0 - mu * mu));
    const double phi = 2.0 * M_PI * u2;
    D3 b1, b2;
    onb(t, b1, b2);
    double c, sn;
    sincos(phi, &sn, &c);
    return normalized(d3(mu * t.x + st * (c * b1.x + sn * b2.x), mu * t.y + st * (c * b1.y + sn * b2.y),
                         mu * t.z + st * (c * b1.z + sn * b2.z)));
}

__device__ inline D3 sample_sphere(double u1, double u2) {
    const double z = 1.0 - 2.0 * u1;
    const double r = sqrt(fmax(0.0, 1.0 - z * z));
    const double phi = 2.0 * M_PI * u2;
    double c, sn;
    sincos(phi, &sn, &c);
    return normalized(d3(r * c, r * sn, z));
}

// Ratio-tracking transmittance estimate on [0, t1).
__device__ inline double ratio_track(const Tracer& tr, Rng& rng, const D3& o, const D3& d, double t1) {
    const pg_tracer& t = tr.t;
    const double maj = t.majorant;
    if (maj <= 0.0) return 1.0;
    double T = 1.0, s = 0.0;
    for (;;) {
        s -= div_by(log(1.0 - rng.uniform()), maj, tr.inv_maj);
        if (s >= t1) return T;
        const D3 p = d3(o.x + s * d.x, o.y + s * d.y, o.z + s * d.z);
        T *= 1.0 - div_by(sigma_at(t, p), maj, tr.inv_maj);
        if (T == 0.0) return 0.0;
    }
}

struct Out {
    float *pos, *dir_in, *dir_out, *albedo, *l_sun, *dir_env, *l_env, *l_phase;
    float *fb_l_sun, *fb_dir_env, *fb_l_env;   // [P][M][3]
    float *dir_pl, *l_pl;
};

// One traced vertex in the slab, stored by its lane in 16-byte pieces of its own
// lines: 88 bytes (112 with a point light).
//   pos albedo | dir_in l_phase.x | l_sun dir_env.x | dir_env.yz l_env.xy | l_env.z dir_out
//   then l_phase.yz: 8 bytes in an array of their own, or the point light's
//   l_phase.yz dir_pl.xy | dir_pl.z l_pl
struct Slab {
    float4* rec;
    float2* tail;   // without a point light
};
constexpr int kRec = 5, kRecPl = 7;

// The M extra emitter samples at a path's first vertex pt (paper, handling
// direct light): sun and uniform-sphere environment shadow rays from a
// second stream of the pixel, so the path itself does not depend on M.
__device__ void extra_samples(const Tracer& tr, uint64_t pixel, int s, const D3& pt, int64_t p, const Out& o) {
    const pg_tracer& t = tr.t;
    Rng rng;
    rng.seed(splitmix64(t.seed * 0x100000001B3ull + (uint64_t)s) ^ 0x5851F42D4C957F2Dull, pixel);
    const D3 sun = d3(t.sun_dir[0], t.sun_dir[1], t.sun_dir[2]);
    for (int k = 0; k < t.extra_samples; ++k) {
        const double Ts = ratio_track(tr, rng, pt, sun, exit_distance(pt, sun));
        const double v2 = rng.uniform();   // azimuth number first
        const double v1 = rng.uniform();
        const D3 we = sample_sphere(v1, v2);
        const double Te = ratio_track(tr, rng, pt, we, exit_distance(pt, we));
        const int64_t b = ((int64_t)p * t.extra_samples + k) * 3;
        for (int a = 0; a < 3; ++a) {
            o.fb_l_sun[b + a] = (float)(t.sun_E[a] * Ts);
            o.fb_dir_env[b + a] = (float)comp(we, a);
            o.fb_l_env[b + a] = (float)(t.env_L[a] * Te);
        }
    }
}

// A lane's path and the ray it is on.  Rays are tracked one tentative collision
// (step) at a time; a ray that has ended waits (kEnd) until its event is
// handled, which starts the path's next ray.
enum State : int { kIdle, kStep, kEnd };
enum Ray : int { kSun, kEnv, kPoint, kFlight };   // shadow rays, and the flight to the next vertex
struct Walk {
    int state = kIdle, ray = kFlight;
    bool hit = false;    // the flight ended in a collision
    uint32_t p = 0;      // path id
    int nv = -1;         // vertices so far; -1: on the camera ray
    Rng rng;
    D3 o, d, dir;        // ray origin, the path's arriving direction at it, ray direction
    double s, t1, T;     // distance along the ray, its end, transmittance
    double Ts, Te;       // of the sun and the environment ray

    __device__ __forceinline__ void cast(int kind, const D3& direction, double end) {
        ray = kind;
        dir = direction;
        s = 0.0;
        t1 = end;
        T = 1.0;
        state = kStep;
    }
};

// Takes path w.p: its camera ray.
__device__ __forceinline__ void start_path(const Tracer& tr, Walk& w) {
    const pg_tracer& t = tr.t;
    const int64_t p = w.p, pix = p / t.spp;
    const int s = (int)(p % t.spp);
    const int X = tr.cx0 + (int)(pix % tr.cw), Y = tr.cy0 + (int)(pix / tr.cw);
    w.rng.seed(splitmix64(t.seed * 0x100000001B3ull + (uint64_t)s), (uint64_t)Y * (uint64_t)t.width + (uint64_t)X);
    const double u2 = w.rng.uniform();   // the jitter: y first, then x
    const double u1 = w.rng.uniform();
    const double sx = ((X + u1) / t.width * 2.0 - 1.0) * tr.th * tr.aspect;
    const double sy = (1.0 - (Y + u2) / t.height * 2.0) * tr.th;
    const D3 d = normalized(d3(tr.f.x + sx * tr.r.x + sy * tr.up.x, tr.f.y + sx * tr.r.y + sy * tr.up.y,
                               tr.f.z + sx * tr.r.z + sy * tr.up.z));
    w.o = d3(t.cam_pos[0], t.cam_pos[1], t.cam_pos[2]);
    w.nv = -1;
    double t0 = 0.0, t1 = 0.0;
    const bool in = box_hit(w.o, d, t0, t1) && t.majorant > 0.0;
    w.cast(kFlight, d, t1);
    w.s = fmax(t0, 0.0);
    w.hit = false;
    if (!in) w.state = kEnd;
}

// One tentative collision: analog delta tracking on a flight, ratio tracking on
// a shadow ray.
template <bool FLIGHT>
__device__ __forceinline__ void step(const Tracer& tr, Walk& w) {
    const pg_tracer& t = tr.t;
    const double maj = t.majorant;
    w.s -= div_by(log(1.0 - w.rng.uniform()), maj, tr.inv_maj);
    if (w.s >= w.t1) {
        w.hit = false;
        w.state = kEnd;
        return;
    }
    const double sg = sigma_at(t, d3(w.o.x + w.s * w.dir.x, w.o.y + w.s * w.dir.y, w.o.z + w.s * w.dir.z));
    if (FLIGHT) {
        w.hit = w.rng.uniform() * maj < sg;
        if (w.hit) w.state = kEnd;
    } else {
        w.T *= 1.0 - div_by(sg, maj, tr.inv_maj);
        if (w.T == 0.0) {
            w.T = 0.0;
            w.state = kEnd;
        }
    }
}

// Steps the lanes on rays of kind RAY until at most `behind` of them are left;
// those go on when the wave comes back to this kind of ray.
template <int RAY>
__device__ __forceinline__ void track(const Tracer& tr, Walk& w, int behind) {
    for (;;) {
        const bool on = w.state == kStep && w.ray == RAY;
        if (__popcll(__ballot(on)) <= behind) return;
        if (on) step<RAY == kFlight>(tr, w);
    }
}

// The radiance that arrives along the continuation if it escapes.
template <bool PL>
__device__ __forceinline__ void store_phase(const Slab& slab, int64_t slot, float x, float y, float z) {
    float4* r = slab.rec + slot * (PL ? kRecPl : kRec);
    r[1].w = x;
    *(PL ? reinterpret_cast<float2*>(r + 5) : slab.tail + slot) = make_float2(y, z);
}

// The flight has ended: at the path's next vertex, whose sun ray starts, or
// outside, which ends the path.
template <bool PL>
__device__ __forceinline__ void flight_ended(const Tracer& tr, Walk& w, const Slab& slab,
                                             uint32_t* __restrict__ count, float* __restrict__ ecam) {
    const pg_tracer& t = tr.t;
    const int64_t slot = (int64_t)w.p * t.max_depth + w.nv;
    const float ex = w.hit ? 0.0f : (float)t.env_L[0], ey = w.hit ? 0.0f : (float)t.env_L[1],
                ez = w.hit ? 0.0f : (float)t.env_L[2];
    if (w.nv < 0) {
        ecam[3 * (int64_t)w.p] = ex;
        ecam[3 * (int64_t)w.p + 1] = ey;
        ecam[3 * (int64_t)w.p + 2] = ez;
    } else {
        store_phase<PL>(slab, slot, ex, ey, ez);
    }
    if (w.hit) w.o = d3(w.o.x + w.s * w.dir.x, w.o.y + w.s * w.dir.y, w.o.z + w.s * w.dir.z);
    ++w.nv;
    if (!w.hit) {
        count[w.p] = (uint32_t)w.nv;
        w.state = kIdle;
        return;
    }
    w.d = w.dir;
    float4* r = slab.rec + (slot + 1) * (PL ? kRecPl : kRec);
    r[0] = make_float4((float)w.o.x, (float)w.o.y, (float)w.o.z, (float)albedo_at(t, w.o));
    r[1] = make_float4((float)w.d.x, (float)w.d.y, (float)w.d.z, 0.0f);   // l_phase.x when the flight has ended
    const D3 sun = d3(t.sun_dir[0], t.sun_dir[1], t.sun_dir[2]);
    w.cast(kSun, sun, exit_distance(w.o, sun));
}

__device__ __forceinline__ void sun_ended(Walk& w) {
    w.Ts = w.T;
    const double e2 = w.rng.uniform();   // azimuth number first
    const double e1 = w.rng.uniform();
    const D3 we = sample_sphere(e1, e2);
    w.cast(kEnv, we, exit_distance(w.o, we));
}

// The environment ray (with a point light: its ray) has ended: the
// continuation is sampled and the record's emitter samples are stored.
template <bool PL>
__device__ __forceinline__ void shadow_ended(const Tracer& tr, Walk& w, const Slab& slab,
                                             uint32_t* __restrict__ count) {
    const pg_tracer& t = tr.t;
    const int64_t slot = (int64_t)w.p * t.max_depth + w.nv;
    float4* r = slab.rec + slot * (PL ? kRecPl : kRec);
    if (w.ray == kEnv) {
        w.Te = w.T;
        r[2] = make_float4((float)(t.sun_E[0] * w.Ts), (float)(t.sun_E[1] * w.Ts), (float)(t.sun_E[2] * w.Ts),
                           (float)w.dir.x);
        r[3] = make_float4((float)w.dir.y, (float)w.dir.z, (float)(t.env_L[0] * w.Te), (float)(t.env_L[1] * w.Te));
    }
    if (PL) {   // point light shadow ray (delta light): irradiance I T / r^2
        const D3 v = d3(t.pl_pos[0] - w.o.x, t.pl_pos[1] - w.o.y, t.pl_pos[2] - w.o.z);
        const double r2 = v.x * v.x + v.y * v.y + v.z * v.z;
        if (w.ray == kEnv) {
            const double dist = sqrt(r2);
            const D3 dl = d3(v.x / dist, v.y / dist, v.z / dist);
            double tmax = exit_distance(w.o, dl);
            if (dist < tmax) tmax = dist;
            w.cast(kPoint, dl, tmax);
            return;
        }
        reinterpret_cast<float2*>(r + 5)[1] = make_float2((float)w.dir.x, (float)w.dir.y);
        r[6] = make_float4((float)w.dir.z, (float)(t.pl_I[0] * w.T / r2), (float)(t.pl_I[1] * w.T / r2),
                           (float)(t.pl_I[2] * w.T / r2));
    }
    const double h2 = w.rng.uniform();   // azimuth number first
    const double h1 = w.rng.uniform();
    const D3 wo = sample_hg(w.d, t.g, h1, h2);
    r[4] = make_float4((float)(t.env_L[2] * w.Te), (float)wo.x, (float)wo.y, (float)wo.z);
    if (w.nv == t.max_depth - 1) {   // the last vertex has no continuation
        store_phase<PL>(slab, slot, 0.0f, 0.0f, 0.0f);
        count[w.p] = (uint32_t)t.max_depth;
        w.state = kIdle;
        return;
    }
    w.cast(kFlight, wo, exit_distance(w.o, wo));
}

// Pass 1: traces every path into its max_depth slots of the workspace slab
// (slot p * max_depth + k), with its extra samples and camera term, and counts
// its vertices.  Bound by the double-precision instructions a wave issues.  A
// wave that keeps its 64 paths and walks them vertex by vertex runs each ray as
// long as the lanes' longest, and all of it as long as the longest path, with a
// fifth of its lanes working.  So
//  * lanes without a path take the next ones from a queue (one atomic a wave),
//    kRefill or more at a time, since a few camera rays cost as much as many;
//  * the wave goes round the kinds of rays (flight, sun, environment), starting
//    the rays of all lanes that have come to a kind together, but leaves a kind
//    once at most 1 / kBehind of its lanes are still on such a ray: those miss
//    the round and go on with the next one's.
// 20M vertices on a ball (21 a path, depth 64), with the copy below: 14.5 -> 6.7
// ms (queue and wider records alone 9.0); a dense cloud whose rays mostly end at
// the first step 4.7 -> 3.6 ms.  Refilling at 16 lanes or leaving at 1/5 and 1/16
// changes at most 8%.  Without rounds (an event handled once enough lanes wait
// for it) the ball takes 7.7 ms, the cloud 5.8.
// A path draws its numbers in its own order whatever the lanes around it do, so
// the records do not depend on any of this.  Every round moves a lane on: the
// kinds of rays are fewer than kBehind, so not all lanes can be left behind; and
// the queue's counter only grows: the wave leaves when it is empty and no lane
// has a path.
//
// Few paths leave the chip to single waves, whose time is that of their slowest
// lanes in turn: then fewer lanes a wave take paths (width).  64 / 16 / 8 lanes: 16
// thousand paths of the small cube 0.348 / 0.337 / 0.362 ms, 4 thousand 0.341 / 0.331 /
// 0.293, 4 thousand on the ball 1.44 / 1.32 / 1.05; 66 thousand of the cube 0.354 / 0.402.
constexpr int kRefill = 8, kBehind = 8;
constexpr int kTraceBlocks = 2048;
constexpr int kMinWidth = kRefill, kNarrowWaves = 512;
template <bool PL>
__global__ __launch_bounds__(kBlock) void k_trace(Tracer tr, uint32_t P, int width, uint32_t* __restrict__ next,
                                                  uint32_t* __restrict__ count, Slab slab,
                                                  float* __restrict__ ecam) {
    Walk w;
    const int lane = threadIdx.x & (kWave - 1);
    const uint64_t lanes = ~0ull >> (kWave - width);
    bool dry = false;   // the queue is empty (uniform over the wave)
    for (;;) {
        const uint64_t idle = __ballot(w.state == kIdle) & lanes;
        const int n = __popcll(idle);
        if (!dry && n >= kRefill) {
            uint32_t base = 0;
            if (lane == 0) base = atomicAdd(next, (uint32_t)n);
            base = (uint32_t)__shfl((int)base, 0, kWave);
            dry = (uint64_t)base + (uint32_t)n >= P;
            const uint64_t p = (uint64_t)base + __popcll(idle & ((1ull << lane) - 1ull));
            if (w.state == kIdle && lane < width && p < P) {
                w.p = (uint32_t)p;
                start_path(tr, w);
            }
        } else if (n == width) {
            break;   // dry, and no path left
        }
        const int behind = __popcll(__ballot(w.state != kIdle)) / kBehind;
        track<kFlight>(tr, w, behind);
        if (w.state == kEnd && w.ray == kFlight) flight_ended<PL>(tr, w, slab, count, ecam);
        track<kSun>(tr, w, behind);
        if (w.state == kEnd && w.ray == kSun) sun_ended(w);
        track<kEnv>(tr, w, behind);
        if (w.state == kEnd && w.ray == kEnv) shadow_ended<PL>(tr, w, slab, count);
        if (PL) {
            track<kPoint>(tr, w, behind);
            if (w.state == kEnd && w.ray == kPoint) shadow_ended<PL>(tr, w, slab, count);
        }
    }
}

// The extra samples of every path's first vertex, one thread a path: it walks the
// camera ray again, which is short beside the samples' rays, and all lanes of a wave
// have their samples to do together.  In k_trace, where few lanes come to a first
// vertex at a time, 64 samples a path took the wave three times as long (256 x 256 at
// 4 samples on a ball: 28.9 ms with the paths, 7.2 so).
__global__ __launch_bounds__(kBlock) void k_trace_extra(Tracer tr, uint32_t P, Out o) {
    const pg_tracer& t = tr.t;
    const uint32_t p = blockIdx.x * kBlock + threadIdx.x;
    if (p >= P) return;
    Walk w;
    w.p = p;
    start_path(tr, w);
    while (w.state == kStep) step<true>(tr, w);
    if (w.hit) {
        const int64_t pix = (int64_t)p / t.spp;
        const int X = tr.cx0 + (int)(pix % tr.cw), Y = tr.cy0 + (int)(pix / tr.cw);
        const D3 pt = d3(w.o.x + w.s * w.dir.x, w.o.y + w.s * w.dir.y, w.o.z + w.s * w.dir.z);
        extra_samples(tr, (uint64_t)Y * (uint64_t)t.width + (uint64_t)X, (int)(p % (uint32_t)t.spp), pt, p, o);
    } else {   // no first vertex: zero samples
        for (int64_t b = (int64_t)p * t.extra_samples * 3; b < ((int64_t)p + 1) * t.extra_samples * 3; ++b)
            o.fb_l_sun[b] = o.fb_dir_env[b] = o.fb_l_env[b] = 0.0f;
    }
}

// Pass 2: one thread per slab slot (p, k) copies the k-th record of path p
// to path_offsets[p] + k.  A path whose offsets do not span exactly its
// traced vertex count (offsets not from this trace) is not written and is
// reported.
template <bool PL>
__global__ __launch_bounds__(kBlock) void k_trace_compact(int64_t P, int64_t maxd, const int64_t* __restrict__ off,
                                                          const uint32_t* __restrict__ start,
                                                          Slab slab, Out o, int32_t* flag) {
    const int64_t slot = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (slot >= P * maxd) return;
    const int64_t p = slot / maxd, k = slot - p * maxd;
    const int64_t c = (int64_t)start[p + 1] - (int64_t)start[p];
    const int64_t a = off[p], n = off[p + 1] - a;
    if (n != c || a < 0) {
        if (k == 0) set_flag(flag, kFlagOffsets);   // offsets not from this tracer
        return;
    }
    if (k >= c) return;
    const int64_t v = a + k;
    float f[4 * kRecPl];
    const float4* r = slab.rec + slot * (PL ? kRecPl : kRec);
#pragma unroll
    for (int q = 0; q < (PL ? kRecPl : kRec); ++q) {
        const float4 x = r[q];
        f[4 * q] = x.x;
        f[4 * q + 1] = x.y;
        f[4 * q + 2] = x.z;
        f[4 * q + 3] = x.w;
    }
    if (!PL) {
        const float2 x = slab.tail[slot];
        f[20] = x.x;
        f[21] = x.y;
    }
    o.albedo[v] = f[3];
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        o.pos[3 * v + q] = f[q];
        o.dir_in[3 * v + q] = f[4 + q];
        o.l_sun[3 * v + q] = f[8 + q];
        o.dir_env[3 * v + q] = f[11 + q];
        o.l_env[3 * v + q] = f[14 + q];
        o.dir_out[3 * v + q] = f[17 + q];
        o.l_phase[3 * v + q] = f[q == 0 ? 7 : 19 + q];
        if (PL) {
            o.dir_pl[3 * v + q] = f[22 + q];
            o.l_pl[3 * v + q] = f[25 + q];
        }
    }
}

// offsets (int64) from the scanned counts (uint32, P+1 entries)
__global__ __launch_bounds__(kBlock) void k_widen(int64_t n, const uint32_t* __restrict__ in, int64_t* __restrict__ out) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) out[i] = in[i];
}

}  // namespace

static Tracer make_tracer(const pg_tracer* t) {
    Tracer tr;
    tr.t = *t;
    tr.cw = t->crop_w ? t->crop_w : t->width;
    tr.ch = t->crop_w ? t->crop_h : t->height;
    tr.cx0 = t->crop_w ? t->crop_x0 : 0;
    tr.cy0 = t->crop_w ? t->crop_y0 : 0;
    tr.point_light = t->pl_I[0] != 0.0 || t->pl_I[1] != 0.0 || t->pl_I[2] != 0.0;
    // camera frame, as the device would compute it (host double, same order)
    double f[3], r[3], up[3];
    const double wup[3] = {0.0, 1.0, 0.0};
    for (int a = 0; a < 3; ++a) f[a] = t->look_at[a] - t->cam_pos[a];
    double l = std::sqrt(f[0] * f[0] + f[1] * f[1] + f[2] * f[2]);
    for (int a = 0; a < 3; ++a) f[a] /= l;
    r[0] = f[1] * wup[2] - f[2] * wup[1];
    r[1] = f[2] * wup[0] - f[0] * wup[2];
    r[2] = f[0] * wup[1] - f[1] * wup[0];
    l = std::sqrt(r[0] * r[0] + r[1] * r[1] + r[2] * r[2]);
    for (int a = 0; a < 3; ++a) r[a] /= l;
    up[0] = r[1] * f[2] - r[2] * f[1];
    up[1] = r[2] * f[0] - r[0] * f[2];
    up[2] = r[0] * f[1] - r[1] * f[0];
    tr.f = D3{f[0], f[1], f[2]};
    tr.r = D3{r[0], r[1], r[2]};
    tr.up = D3{up[0], up[1], up[2]};
    tr.th = std::tan(0.5 * t->vfov_deg * M_PI / 180.0);
    tr.aspect = (double)t->width / (double)t->height;
    tr.t.majorant = walked_majorant(t->majorant);
    tr.inv_maj = tr.t.majorant > 0.0 ? 1.0 / tr.t.majorant : 0.0;
    return tr;
}

int64_t tracer_paths(const pg_tracer* t) {
    const int64_t cw = t->crop_w ? t->crop_w : t->width, ch = t->crop_w ? t->crop_h : t->height;
    return cw * ch * t->spp;
}

// Workspace: flags, the vertex counts (scanned in place to offsets), and the
// slab the count pass traces into: max_depth record slots per path, the
// paths' extra samples and camera terms.  Pass 2 copies from the slab, so
// both passes must use the same workspace, unchanged in between.
struct TraceWs {
    int32_t* flag;
    uint32_t* next;    // the path queue's counter
    uint32_t* count;
    uint32_t* part;
    Slab slab;
    Out fb;            // the extra samples' arrays
    float* ecam;
};

static TraceWs carve_trace(Carver& cv, const pg_tracer* t) {
    const int64_t P = tracer_paths(t);
    const int64_t S = P * (int64_t)t->max_depth;
    const bool pl = t->pl_I[0] != 0.0 || t->pl_I[1] != 0.0 || t->pl_I[2] != 0.0;
    const int64_t F = t->extra_samples > 0 ? P * (int64_t)t->extra_samples * 3 : 0;
    TraceWs w;
    w.flag = cv.take<int32_t>(64);
    w.next = cv.take<uint32_t>(64);
    w.count = cv.take<uint32_t>(P + 1);
    w.part = cv.take<uint32_t>(scan_partials_bytes(P + 1) / 4);
    w.slab.rec = cv.take<float4>(S * (pl ? kRecPl : kRec));
    w.slab.tail = pl ? nullptr : cv.take<float2>(S);
    w.fb = Out{};
    w.fb.fb_l_sun = F ? cv.take<float>(F) : nullptr;
    w.fb.fb_dir_env = F ? cv.take<float>(F) : nullptr;
    w.fb.fb_l_env = F ? cv.take<float>(F) : nullptr;
    w.ecam = cv.take<float>(3 * P + 3);
    return w;
}

size_t trace_ws_size(const pg_tracer* t) {
    Carver cv(nullptr);
    (void)carve_trace(cv, t);
    return cv.size();
}

hipError_t run_trace_count(const pg_tracer* t, int64_t* path_offsets, float* e_cam, void* ws, hipStream_t s) {
    (void)e_cam;   // kept in the slab; pass 2 writes it
    const int64_t P = tracer_paths(t);
    Carver cv(ws);
    const TraceWs w = carve_trace(cv, t);
    hipError_t e;
    if ((e = launch_fill(w.count, (size_t)P * 4, s)) != hipSuccess) return e;
    if ((e = launch_fill(w.next, 4, s)) != hipSuccess) return e;
    const Tracer tr = make_tracer(t);
    if (P > 0) {
        ProfScope ps(s, "trace_count");
        int width = kWave;
        while (width > kMinWidth && P <= (int64_t)width * kNarrowWaves) width /= 2;
        const dim3 grid((unsigned)std::min<int64_t>(kTraceBlocks, div_up(P, width * (kBlock / kWave))));
        if (tr.point_light)
            hipLaunchKernelGGL(k_trace<true>, grid, dim3(kBlock), 0, s, tr, (uint32_t)P, width, w.next, w.count, w.slab,
                               w.ecam);
        else
            hipLaunchKernelGGL(k_trace<false>, grid, dim3(kBlock), 0, s, tr, (uint32_t)P, width, w.next, w.count,
                               w.slab, w.ecam);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        if (t->extra_samples > 0)
            hipLaunchKernelGGL(k_trace_extra, dim3((unsigned)div_up(P, kBlock)), dim3(kBlock), 0, s, tr, (uint32_t)P,
                               w.fb);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    if ((e = launch_scan_exclusive(w.count, w.count, P, w.part, s)) != hipSuccess) return e;
    hipLaunchKernelGGL(k_widen, dim3((unsigned)div_up(P + 1, kBlock)), dim3(kBlock), 0, s, P + 1, w.count,
                       path_offsets);
    return hipGetLastError();
}

hipError_t run_trace_write(const pg_tracer* t, const int64_t* path_offsets, const pg_records& o, void* ws,
                           hipStream_t s, int32_t** flag_out) {
    const int64_t P = tracer_paths(t);
    Carver cv(ws);
    const TraceWs w = carve_trace(cv, t);
    *flag_out = w.flag;
    hipError_t e;
    if ((e = launch_fill(w.flag, 64 * 4, s)) != hipSuccess) return e;
    if (P == 0) return hipSuccess;
    const Tracer tr = make_tracer(t);
    Out out{o.pos, o.dir_in, o.dir_out, o.albedo, o.l_sun, o.dir_env, o.l_env, o.l_phase,
            o.fb_l_sun, o.fb_dir_env, o.fb_l_env, o.dir_pl, o.l_pl};
    ProfScope ps(s, "trace_write");
    const int64_t maxd = t->max_depth;
    const dim3 grid((unsigned)div_up(P * maxd, kBlock));
    if (tr.point_light)
        hipLaunchKernelGGL(k_trace_compact<true>, grid, dim3(kBlock), 0, s, P, maxd, path_offsets,
                           (const uint32_t*)w.count, w.slab, out, w.flag);
    else
        hipLaunchKernelGGL(k_trace_compact<false>, grid, dim3(kBlock), 0, s, P, maxd, path_offsets,
                           (const uint32_t*)w.count, w.slab, out, w.flag);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if ((e = hipMemcpyAsync(o.e_cam, w.ecam, (size_t)P * 12, hipMemcpyDeviceToDevice, s)) != hipSuccess) return e;
    if (t->extra_samples > 0) {
        const size_t F = (size_t)P * (size_t)t->extra_samples * 12;
        if ((e = hipMemcpyAsync(o.fb_l_sun, w.fb.fb_l_sun, F, hipMemcpyDeviceToDevice, s)) != hipSuccess) return e;
        if ((e = hipMemcpyAsync(o.fb_dir_env, w.fb.fb_dir_env, F, hipMemcpyDeviceToDevice, s)) != hipSuccess)
            return e;
        if ((e = hipMemcpyAsync(o.fb_l_env, w.fb.fb_l_env, F, hipMemcpyDeviceToDevice, s)) != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace pg
