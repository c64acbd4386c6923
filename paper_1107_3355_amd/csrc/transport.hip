// Transport kernels of libgdpm for gfx950 (CDNA4, 64-wide wavefronts).
//
// The paper separates photon and electron transport into different kernel
// launches so that threads of a warp follow the same physics (section 2.2.1,
// Fig. 1): particles live in a particle array and two secondary stacks, and the
// host alternates source generation, photon kernels and electron kernels.
// Here the same separation is kept (one queue per particle type, one kernel per
// type) but the launch shape is built for CDNA:
//   - a kernel is a persistent grid of wavefronts; each lane holds one
//     particle and advances it by one event per iteration (one Woodcock flight
//     for a photon, one condensed-history step for an electron); a lane whose
//     particle ends takes the next one from the queue (or starts a new source
//     history), so lanes stay busy instead of idling until the slowest particle
//     of the wave finishes;
//   - queue traffic is per wavefront: a ballot + mbcnt prefix gives each lane
//     its slot, one atomic per 32 to 256 records reserves ring space and one
//     per 32 to 2048 claims input;
//   - dose goes into double-precision tallies with hardware FP64 atomics; a
//     charged particle's deposits are merged per voxel, and added for several
//     voxels of one line of memory at a time (see Brick).
// Random numbers: Philox4x32-10 (Salmon et al., SC'11); a particle owns the
// stream (history id, path id) and the draw order of each event is fixed, so
// results do not depend on scheduling.
// Energy is conserved exactly in single precision: when an energy X splits in
// two, the larger part L >= X/2 is computed and the smaller is X - L, which is
// exact (Sterbenz).  This unit is therefore compiled without floating-point
// contraction; fused multiply-adds are written out with fmaf.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "dev_types.h"

namespace gdpm {

#define GDPM_DEV __device__ __forceinline__
#define GDPM_HD __host__ __device__ inline

constexpr float kMec2f = 0.51099895f;
constexpr float kTwoMec2f = 1.0219979f;
constexpr float kLn2f = 0.693147180559945f;
constexpr float kMwIsoF = 20.0f;

// ---------------------------------------------------------------------------
// hardware math (v_log_f32 is log2, v_exp_f32 is 2^x, v_sin/v_cos take turns)
// ---------------------------------------------------------------------------
GDPM_DEV float hlog2(float x) { return __builtin_amdgcn_logf(x); }
GDPM_DEV float hexp2(float x) { return __builtin_amdgcn_exp2f(x); }
GDPM_DEV float hsqrt(float x) { return __builtin_amdgcn_sqrtf(x); }
GDPM_DEV float hrsq(float x) { return __builtin_amdgcn_rsqf(x); }
GDPM_DEV float hrcp(float x) { return __builtin_amdgcn_rcpf(x); }
GDPM_DEV float sin_turns(float t) { return __builtin_amdgcn_sinf(t); }
GDPM_DEV float cos_turns(float t) { return __builtin_amdgcn_cosf(t); }
GDPM_DEV float neg_ln(float u) { return -kLn2f * hlog2(u); }

// ---------------------------------------------------------------------------
// wavefront helpers
// ---------------------------------------------------------------------------
GDPM_DEV uint32_t lane_id() { return __lane_id(); }
GDPM_DEV uint32_t mbcnt(uint64_t m) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}
GDPM_DEV uint64_t ballot(bool p) { return __ballot(p); }
GDPM_DEV uint32_t first_lane(uint64_t m) { return (uint32_t)(__ffsll((unsigned long long)m) - 1); }
GDPM_DEV uint32_t bcast(uint32_t v, uint32_t lane) { return __builtin_amdgcn_readlane(v, lane); }

GDPM_DEV double wave_sum(double v) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

// ---------------------------------------------------------------------------
// address spaces: pointers that come out of structures in memory are generic to
// the compiler, and a generic access is a FLAT instruction, which waits for every
// outstanding vector-memory operation and for LDS.  The transport therefore
// names the space of each access.
// ---------------------------------------------------------------------------
#define GDPM_GLOBAL __attribute__((address_space(1)))
#define GDPM_LDS __attribute__((address_space(3)))
#define GDPM_CONST __attribute__((address_space(4)))
typedef float f2 __attribute__((ext_vector_type(2)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef uint32_t u4 __attribute__((ext_vector_type(4)));

template <class T>
GDPM_DEV GDPM_GLOBAL T* global_ptr(T* p) { return (GDPM_GLOBAL T*)p; }
// vector view of a table of float4
GDPM_DEV const GDPM_GLOBAL f4* global_f4(const float4* p) { return (const GDPM_GLOBAL f4*)p; }

// A wave-uniform pointer the compiler cannot see through: what is read from it
// afterwards is read here (by scalar loads, from the scalar cache) instead of
// being kept in scalar registers over the whole loop, where the job's data, the
// tables' parameters and the generator's round keys were spilled to lanes of
// vector registers and fetched back one v_readlane each.
template <class T>
GDPM_DEV T* reread(T* p) {
    asm volatile("" : "+s"(p));
    return p;
}

// A wave-uniform value (32 bits, or a pointer) that stays in scalar registers: without
// it the compiler reads a kernel argument or a field of the job again inside the loop,
// and each of those scalar loads is waited for.
template <class T>
GDPM_DEV T pin(T v) {
    asm volatile("" : "+s"(v));
    return v;
}

// ---------------------------------------------------------------------------
// Philox4x32-10
// ---------------------------------------------------------------------------
GDPM_DEV uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) { return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96); }

GDPM_DEV void philox(uint32_t k0, uint32_t k1, uint32_t& x0, uint32_t& x1, uint32_t& x2,
                     uint32_t& x3) {
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        // one 32x32 -> 64-bit product per multiplier
        const uint64_t p0 = (uint64_t)0xD2511F53u * (uint64_t)x0;
        const uint64_t p1 = (uint64_t)0xCD9E8D57u * (uint64_t)x2;
        const uint32_t y0 = xor3((uint32_t)(p1 >> 32), x1, k0);
        const uint32_t y2 = xor3((uint32_t)(p0 >> 32), x3, k1);
        x0 = y0;
        x1 = (uint32_t)p1;
        x2 = y2;
        x3 = (uint32_t)p0;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
}

// (2 (x >> 9) + 1) 2^-24: exact in single and double precision, inside (0, 1).
// The fused product and sum are exact, like the two operations apart.
GDPM_DEV float unit_float(uint32_t x) { return fmaf((float)(x >> 9), 0x1p-23f, 0x1p-24f); }

// A lane's stream: key (k0, k1), counter (hist lo, hist hi, path, draw >> 2);
// draw d is word d & 3 of its block.  Blocks are only ever generated in counter
// order, so the draws are the same whatever is buffered.
//
// The transport's generator keeps up to two blocks of a lane in LDS, already
// converted to uniforms: draw d in word d & 7 of the lane's column (the words of
// a wavefront are 64 lanes apart, so no access has a bank conflict).  Held in
// registers, the two blocks took 8 vector registers and every draw a chain of
// divergent branches to pick its word.  Blocks are generated with the wavefront
// converged, and only once some lane is short of draws for its next event: then
// every lane with room gets its next block (rng_topup), so nearly all lanes of
// the wavefront take part, where generating each lane's block as it came due ran
// the generator in every iteration for about half of them.
constexpr uint32_t kRngWords = 8;    // draws buffered per lane
template <uint32_t kCols>
struct Rng {
    uint32_t hlo, hhi, path;
    uint32_t ctr;                    // next draw
    uint32_t nb;                     // blocks up to nb are generated: draws below 4 nb are buffered
    GDPM_LDS float* buf;             // the lane's column of the wavefront's LDS slice
    // draws buffered (negative in a fresh stream that starts inside a block)
    GDPM_DEV int left() const { return (int)(4u * nb - ctr); }
    GDPM_DEV float peek(uint32_t ahead) const { return buf[((ctr + ahead) & (kRngWords - 1u)) * kCols]; }
    // the next draw; the caller has made sure that it is buffered
    GDPM_DEV float draw() {
        const float u = peek(0u);
        ctr += 1u;
        return u;
    }
    GDPM_DEV void fill(uint32_t k0, uint32_t k1) {
        uint32_t x0 = hlo, x1 = hhi, x2 = path, x3 = nb;
        // the round keys are formed here, not kept in 18 scalar registers
        asm volatile("" : "+s"(k0), "+s"(k1));
        philox(k0, k1, x0, x1, x2, x3);
        GDPM_LDS float* b = buf + (nb & 1u) * (4u * kCols);
        b[0] = unit_float(x0);
        b[kCols] = unit_float(x1);
        b[2u * kCols] = unit_float(x2);
        b[3u * kCols] = unit_float(x3);
        nb += 1u;
    }
    // at least n <= 4 draws buffered (in the lanes that call it: a divergent branch)
    GDPM_DEV void ensure(uint32_t n, uint32_t k0, uint32_t k1) {
        while (left() < (int)n) fill(k0, k1);
    }
};

// counter of the next draw
template <uint32_t kCols>
GDPM_DEV uint32_t rng_ctr(const Rng<kCols>& r) { return r.ctr; }

// position the stream at draw `ctr` (no block generated yet)
template <uint32_t kCols>
GDPM_DEV void rng_start(Rng<kCols>& r, uint32_t hlo, uint32_t hhi, uint32_t path, uint32_t ctr) {
    r.hlo = hlo;
    r.hhi = hhi;
    r.path = path;
    r.ctr = ctr;
    r.nb = ctr >> 2;
}

// The wavefront's lanes exchange data in LDS here: no LDS access moves across (they
// complete in order).
GDPM_DEV void wave_fence() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// with the wavefront converged: n <= 4 draws in the lanes of `want`; every lane
// of `live` that holds fewer than two blocks gets one in each turn (a fresh
// stream may need two)
template <uint32_t kCols>
GDPM_DEV void rng_topup(Rng<kCols>& r, bool want, bool live, uint32_t n, uint32_t k0, uint32_t k1) {
    while (ballot(want && r.left() < (int)n)) {
        if (live && r.nb - (r.ctr >> 2) < 2u) r.fill(k0, k1);
    }
}

// path id of the secondary created in role `word` at the parent's current counter
template <class R>
GDPM_DEV uint32_t spawn_path(const R& r, uint32_t k0, uint32_t k1, int word) {
    uint32_t x0 = r.hlo, x1 = r.hhi, x2 = r.path, x3 = 0x80000000u | rng_ctr(r);
    asm volatile("" : "+s"(k0), "+s"(k1));
    philox(k0, k1, x0, x1, x2, x3);
    return word == 0 ? x0 : (word == 1 ? x1 : (word == 2 ? x2 : x3));
}

// a stream held in registers, for the kernels outside the transport loops (the
// samplers' and the source's tests)
struct RegRng {
    uint32_t hlo, hhi, path, ctr;
    u4 w;
    GDPM_DEV RegRng(uint32_t lo, uint32_t hi, uint32_t p) : hlo(lo), hhi(hi), path(p), ctr(0u), w(0u) {}
    GDPM_DEV void ensure(uint32_t, uint32_t, uint32_t) {}
    GDPM_DEV float draw(uint32_t k0, uint32_t k1) {
        const uint32_t i = ctr & 3u;
        if (i == 0u) {
            uint32_t x0 = hlo, x1 = hhi, x2 = path, x3 = ctr >> 2;
            philox(k0, k1, x0, x1, x2, x3);
            w = u4{x0, x1, x2, x3};
        }
        ctr += 1u;
        return unit_float(i == 0u ? w.x : (i == 1u ? w.y : (i == 2u ? w.z : w.w)));
    }
};
// the samplers draw from either
template <uint32_t kCols>
GDPM_DEV float uniform(Rng<kCols>& r, uint32_t, uint32_t) { return r.draw(); }
GDPM_DEV float uniform(RegRng& r, uint32_t k0, uint32_t k1) { return r.draw(k0, k1); }

// device-coherent load of a counter, made wave-uniform
GDPM_DEV uint32_t load_agent(const GDPM_GLOBAL uint32_t* p) {
    return __builtin_amdgcn_readfirstlane(
        __hip_atomic_load(const_cast<GDPM_GLOBAL uint32_t*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}
template <class T>
GDPM_DEV T atomic_add(GDPM_GLOBAL T* p, T v) {
    return __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
GDPM_DEV void atomic_or(GDPM_GLOBAL uint32_t* p, uint32_t v) {
    (void)__hip_atomic_fetch_or(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
GDPM_DEV void atomic_add_f64(GDPM_GLOBAL double* p, double v) { (void)__builtin_amdgcn_global_atomic_fadd_f64(p, v); }

// non-exact division through the hardware reciprocal (about 1 ulp)
GDPM_DEV float fdiv(float a, float b) { return a * hrcp(b); }

// ---------------------------------------------------------------------------
// table lookups (linear in log2 E); a table is given by a pointer into LDS or
// global memory
// ---------------------------------------------------------------------------
GDPM_DEV void grid(float lg, float lo, float inv, int n, int& i, float& t) {
    float f = (lg - lo) * inv;
    f = fminf(fmaxf(f, 0.0f), (float)(n - 1));
    i = min((int)f, n - 2);
    t = f - (float)i;
}

template <class P>
GDPM_DEV f4 lerp4(P tab, int i, float t) {
    const f4 a = tab[i], b = tab[i + 1];
    return f4{fmaf(t, b.x - a.x, a.x), fmaf(t, b.y - a.y, a.y), fmaf(t, b.z - a.z, a.z), fmaf(t, b.w - a.w, a.w)};
}

template <class P>
GDPM_DEV float lerp1(P tab, int i, float t) {
    const float a = tab[i], b = tab[i + 1];
    return fmaf(t, b - a, a);
}

// What a flight needs of the photon table, the total cross section, and what a
// step needs of the electron table: in LDS the columns lie apart (a pass reads
// one or two of the four, and neighbouring rows fall on different banks), in
// global memory they are the table's float4 rows.  The columns that only an
// interaction needs are read from global memory in either case.
struct PhotLds {
    const GDPM_LDS float* tot;                  // [mat][pg_n]
    GDPM_DEV float total(int i, float t) const { return lerp1(tot, i, t); }
};
struct PhotGlobal {
    const GDPM_GLOBAL f4* tab;
    GDPM_DEV float total(int i, float t) const {
        const float a = tab[i].w, b = tab[i + 1].w;
        return fmaf(t, b - a, a);
    }
};
struct ElecLds {
    const GDPM_LDS f2* rh;                      // [mat][eg_n] range, mu_hard
    const GDPM_LDS float* lam;                  // [mat][eg_n] 1/lambda_1
    const GDPM_LDS float* rinv;                 // [mat][nr], then the scales [mat]
    const GDPM_LDS float* aw;                   // [aw_n] (a global load in a step would wait for
                                                // the wavefront's tally additions before it)
    GDPM_DEV f2 range_hard(int i, float t) const {
        const f2 a = rh[i], b = rh[i + 1];
        return f2{fmaf(t, b.x - a.x, a.x), fmaf(t, b.y - a.y, a.y)};
    }
    GDPM_DEV float range(int i, float t) const {
        const float a = rh[i].x, b = rh[i + 1].x;
        return fmaf(t, b - a, a);
    }
    GDPM_DEV float inv_lambda(int i, float t) const { return lerp1(lam, i, t); }
};
struct ElecGlobal {
    const GDPM_GLOBAL f4* tab;
    const GDPM_GLOBAL float* rinv;
    const GDPM_GLOBAL float* rscale;
    const GDPM_GLOBAL float* aw;
    GDPM_DEV f2 range_hard(int i, float t) const {
        const f4 a = tab[i], b = tab[i + 1];
        return f2{fmaf(t, b.x - a.x, a.x), fmaf(t, b.y - a.y, a.y)};
    }
    GDPM_DEV float range(int i, float t) const {
        const float a = tab[i].x, b = tab[i + 1].x;
        return fmaf(t, b - a, a);
    }
    GDPM_DEV float inv_lambda(int i, float t) const {
        const float a = tab[i].w, b = tab[i + 1].w;
        return fmaf(t, b - a, a);
    }
};

// the electron tables' parameters, in scalar registers for a whole pass
struct ElecGrid {
    float lo, inv, aw_lo, aw_inv;
    int n, nr, aw_n;
    template <class TT>
    GDPM_DEV explicit ElecGrid(const TT& T)
        : lo(pin(T.eg_lo)), inv(pin(T.eg_inv)), aw_lo(pin(T.aw_lo)), aw_inv(pin(T.aw_inv)), n(pin(T.eg_n)),
          nr(pin(T.nr)), aw_n(pin(T.aw_n)) {}
    // cell of energy e of material m
    GDPM_DEV void cell(int m, float e, int& i, float& t) const {
        grid(hlog2(e), lo, inv, n, i, t);
        i += m * n;
    }
};

// energy whose residual range is r (g/cm^2): the inverse range on sqrt(r)
template <class P>
GDPM_DEV float range_inv(P rtab, float scale, int nr, int m, float r) {
    const float f = fminf(hsqrt(fmaxf(r, 0.0f)) * scale, (float)(nr - 1));
    const int i = min((int)f, nr - 2);
    return lerp1(rtab + m * nr, i, f - (float)i);
}
GDPM_DEV float rinv_scale(const ElecLds& E, const ElecGrid& g, int n_mat, int m) { return E.rinv[n_mat * g.nr + m]; }
GDPM_DEV float rinv_scale(const ElecGlobal& E, const ElecGrid&, int, int m) { return E.rscale[m]; }

// screening A of the modified-Wentzel law for t = s / lambda_1 (t < t_iso)
template <class P>
GDPM_DEV float mw_screening(const ElecGrid& g, P aw, float tt) {
    const float f = fminf((hlog2(tt) - g.aw_lo) * g.aw_inv, (float)(g.aw_n - 1));
    const int i = min(max((int)f, 0), g.aw_n - 2);  // f < 0 extrapolates the first cell
    return hexp2(lerp1(aw, i, f - (float)i));
}

// modified-Wentzel deflection mu = (1 - cos)/2 for t = s / lambda_1
template <class P>
GDPM_DEV float mw_mu(const ElecGrid& g, P aw, float tt, float u) {
    if (!(tt < kMwIsoF)) return u;
    const float a = mw_screening(g, aw, tt);
    return fdiv(a * u, 1.0f + a - u);
}

// ---------------------------------------------------------------------------
// geometry
// ---------------------------------------------------------------------------
GDPM_DEV void rotate(float& u, float& v, float& w, float ct, float st, float turns) {
    const float cp = cos_turns(turns), sp = sin_turns(turns);
    const float r2 = u * u + v * v;
    float nu, nv, nw;
    if (r2 > 1e-12f) {
        const float ir = hrsq(r2), r = r2 * ir;
        nu = u * ct + st * (u * w * cp - v * sp) * ir;
        nv = v * ct + st * (v * w * cp + u * sp) * ir;
        nw = w * ct - st * cp * r;
    } else {
        nu = st * cp;
        nv = st * sp;
        nw = (w >= 0.0f ? ct : -ct);
    }
    const float n = hrsq(nu * nu + nv * nv + nw * nw);
    u = nu * n;
    v = nv * n;
    w = nw * n;
}

GDPM_DEV int clampi(int x, int n) { return min(max(x, 0), n - 1); }

GDPM_DEV int voxel_of(float idx, float idy, float idz, int nx, int ny, int nz, float x, float y, float z, int& ix,
                      int& iy, int& iz) {
    ix = clampi((int)floorf(x * idx), nx);
    iy = clampi((int)floorf(y * idy), ny);
    iz = clampi((int)floorf(z * idz), nz);
    return ix + nx * (iy + ny * iz);
}
// GG: Geom, in any address space
template <class GG>
GDPM_DEV int voxel_of(const GG& G, float x, float y, float z, int& ix, int& iy, int& iz) {
    return voxel_of(G.idx, G.idy, G.idz, G.nx, G.ny, G.nz, x, y, z, ix, iy, iz);
}

GDPM_DEV uint32_t pack_vox(int ix, int iy, int iz) {
    return (uint32_t)ix | ((uint32_t)iy << 11) | ((uint32_t)iz << 22);
}

// x in [0, lx) and so on (lx: the extent's bits).  For non-negative floats the order of the values is
// the order of their bits; a negative number's sign bit and a NaN's exponent make
// it larger than any extent.  (A position of -0 counts as outside; a position is
// set to a face as +0 or as a product with a non-negative index, and a sum that
// cancels is +0.)
GDPM_DEV bool inside(uint32_t lx, uint32_t ly, uint32_t lz, float x, float y, float z) {
    const bool ix = __float_as_uint(x) < lx;
    const bool iy = __float_as_uint(y) < ly;
    const bool iz = __float_as_uint(z) < lz;
    return ix && iy && iz;
}

struct Spacing {
    float dx, dy, dz;   // voxel size
};

// distance to the exit face of voxel (ix, iy, iz) along the direction; axis of that face
template <class GG>
GDPM_DEV float face_dist(const GG& G, float x, float y, float z, float u, float v, float w,
                         int ix, int iy, int iz, int& ax) {
    const float du = fdiv((float)(u > 0.0f ? ix + 1 : ix) * G.dx - x, u);
    const float dv = fdiv((float)(v > 0.0f ? iy + 1 : iy) * G.dy - y, v);
    const float dw = fdiv((float)(w > 0.0f ? iz + 1 : iz) * G.dz - z, w);
    float best = u != 0.0f ? du : 3.0e38f;
    ax = 0;
    const bool by = v != 0.0f && dv < best;
    best = by ? dv : best;
    ax = by ? 1 : ax;
    const bool bz = w != 0.0f && dw < best;
    best = bz ? dw : best;
    ax = bz ? 2 : ax;
    return fmaxf(best, 0.0f);
}

// ---------------------------------------------------------------------------
// source: history h -> primary particle (section 2.3)
// ---------------------------------------------------------------------------
// SS, GG: SourceDev and Geom in any address space
template <class SS>
GDPM_DEV float spectrum_energy(const SS& S, float u) {
    if (S.spec_kind == 0) return S.e_mono;
    const GDPM_GLOBAL float* sc = global_ptr(S.spec_c);
    const GDPM_GLOBAL float* se = global_ptr(S.spec_e);
    const GDPM_GLOBAL float* sp = global_ptr(S.spec_p);
    const int n = S.spec_n;
    const float r = u * sc[n - 1];
    int j = 0;
    while (j < n - 2 && sc[j + 1] <= r) ++j;
    const float e0 = se[j], e1 = se[j + 1];
    const float p0 = sp[j], sl = (sp[j + 1] - p0) / (e1 - e0);
    const float d = r - sc[j];
    const float den = p0 + hsqrt(fmaxf(0.0f, p0 * p0 + 2.0f * sl * d));
    const float x = den > 0.0f ? 2.0f * d / den : 0.0f;
    return fminf(fmaxf(e0 + x, e0), e1);
}

// beamlet I with P(I) <= r < P(I+1); start from the guide table, walk both ways
template <class SS>
GDPM_DEV int beamlet_of(const SS& S, float u) {
    const GDPM_GLOBAL double* cdf = global_ptr(S.cdf);
    const double r = (double)u;
    int k = (int)(r * (double)S.n_guide);
    k = min(k, S.n_guide - 1);
    int i = (int)global_ptr(S.guide)[k];
    while (i > 0 && cdf[i] > r) --i;
    while (i < S.nf - 1 && cdf[i + 1] <= r) ++i;
    return i;
}

struct Primary {
    float x, y, z, u, v, w, e;
    int beamlet;
    uint32_t draws;   // of the history's stream, taken by the source
    bool in;
};

// Metropolis chains (Algorithm A1, section 2.3.1): at each step a trial beamlet J
// is drawn with equal probability among those of nonzero intensity, then r; the
// chain moves to J when r < f_J / f_prev, tested as r f_prev < f_J in double
// precision (exact for single-precision r and f)
template <class SS>
GDPM_DEV uint32_t metropolis_trial(const SS& S, float uj) {
    return global_ptr(S.nz)[min((int)((double)uj * (double)S.n_nz), S.n_nz - 1)];
}
GDPM_DEV bool metropolis_moves(float r, float f_prev, float f_j) { return (double)r * (double)f_prev < (double)f_j; }

// chain start: a beamlet drawn with equal probability among those of nonzero
// intensity, from the chain's own stream (history id (2^32-1) 2^32 + chain)
template <class SS>
GDPM_DEV uint32_t metropolis_start(const SS& S, uint32_t chain, uint32_t k0, uint32_t k1) {
    uint32_t x0 = chain, x1 = 0xFFFFFFFFu, x2 = 0u, x3 = 0u;
    philox(k0, k1, x0, x1, x2, x3);
    return metropolis_trial(S, unit_float(x0));
}

// section 2.3.2: energy of the history at position i of a round of `size`:
// interval k with C_k <= i < C_{k+1}, C_k = floor(size F_k + 1/2); inside it
// the energy is uniform (strata_shape 0) or the spectrum's inverse CDF at
// F_k + u (F_{k+1} - F_k) (strata_shape 1)
template <class SS>
GDPM_DEV float stratified_energy(const SS& S, uint32_t i, uint32_t size, float u) {
    const GDPM_GLOBAL double* F = global_ptr(S.strata_F);
    // the first k that is the last interval or has C_{k+1} > i (C never falls)
    int k = 0, hi = S.strata - 1;
    while (k < hi) {
        const int mid = (k + hi) >> 1;
        if (floor((double)size * F[mid + 1] + 0.5) <= (double)i) k = mid + 1;
        else hi = mid;
    }
    if (S.strata_shape == 0) return fmaf(u, S.strata_w, fmaf((float)k, S.strata_w, S.strata_lo));
    const double f0 = F[k], f1 = F[k + 1];
    return spectrum_energy(S, (float)(f0 + (double)u * (f1 - f0)));
}

// section 2.3.3: history h starts as phase-space record h mod n: inside the phantom where it is, outside where its forward ray
// enters (else it escapes); the record number stands in for the beamlet
template <class SS, class GG>
GDPM_DEV Primary phase_space_primary(const SS& S, const GG& G, unsigned long long h) {
    const unsigned long long k = h % S.n_phsp;
    const GDPM_GLOBAL float* rec = global_ptr(S.phsp) + 7 * k;
    Primary p;
    p.draws = 0u;
    p.beamlet = (int)k;
    p.e = rec[6];
    p.u = rec[3];
    p.v = rec[4];
    p.w = rec[5];
    const float o[3] = {rec[0], rec[1], rec[2]}, d[3] = {p.u, p.v, p.w}, L[3] = {G.lx, G.ly, G.lz};
    p.x = o[0];
    p.y = o[1];
    p.z = o[2];
    p.in = true;
    if (o[0] >= 0.0f && o[0] < G.lx && o[1] >= 0.0f && o[1] < G.ly && o[2] >= 0.0f && o[2] < G.lz) return p;
    float tmin = 0.0f, tmax = 3.0e38f;
    int ax = -1;
    bool miss = false;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        if (d[i] != 0.0f) {
            const float ta = (0.0f - o[i]) / d[i], tb = (L[i] - o[i]) / d[i];
            const float tn = fminf(ta, tb), tf = fmaxf(ta, tb);
            if (tn > tmin) {
                tmin = tn;
                ax = i;
            }
            tmax = fminf(tmax, tf);
        } else if (o[i] < 0.0f || o[i] > L[i]) {
            miss = true;
        }
    }
    p.in = !miss && tmax > tmin;
    p.x = o[0] + tmin * p.u;
    p.y = o[1] + tmin * p.v;
    p.z = o[2] + tmin * p.w;
    if (ax == 0) p.x = p.u > 0.0f ? 0.0f : G.lx;
    if (ax == 1) p.y = p.v > 0.0f ? 0.0f : G.ly;
    if (ax == 2) p.z = p.w > 0.0f ? 0.0f : G.lz;
    return p;
}

// draws 0-3 of history h's stream, path 0
GDPM_DEV f4 source_draws(unsigned long long h, uint32_t k0, uint32_t k1) {
    uint32_t x0 = (uint32_t)h, x1 = (uint32_t)(h >> 32), x2 = 0u, x3 = 0u;
    philox(k0, k1, x0, x1, x2, x3);
    return f4{unit_float(x0), unit_float(x1), unit_float(x2), unit_float(x3)};
}

// The primary of history h, whose first draws are d.  chain_beamlet >= 0: the
// beamlet of its Metropolis chain (draws 1 and 2 are then the chain's, and a
// fifth draw is taken), else the beamlet is searched for.  rpos and rsize
// (stratified spectra only) place the history in its round.
template <class SS, class GG>
GDPM_DEV Primary make_primary(const SS& S, const GG& G, unsigned long long h, f4 d, uint32_t k0, uint32_t k1,
                              int chain_beamlet, uint32_t rpos, uint32_t rsize) {
    Primary p;
    p.e = S.strata ? stratified_energy(S, rpos, rsize, d.x) : spectrum_energy(S, d.x);
    int gi = chain_beamlet;
    float ux = d.z, uy = d.w;
    p.draws = 4u;
    if (S.metro) {
        uint32_t w0 = (uint32_t)h, w1 = (uint32_t)(h >> 32), w2 = 0u, w3 = 1u;
        philox(k0, k1, w0, w1, w2, w3);
        ux = d.w;
        uy = unit_float(w0);
        p.draws = 5u;
    } else {
        gi = beamlet_of(S, d.y);
    }
    p.beamlet = gi;
    const GDPM_GLOBAL BeamDev& b = global_ptr(S.beams)[global_ptr(S.beam_of)[gi]];
    const int j = gi - b.off;
    const int jx = j % b.nbx, jy = j / b.nbx;
    const float px = ((float)jx + ux) * b.bw - b.hx;
    const float py = ((float)jy + uy) * b.bh - b.hy;
    const float qx = b.iso[0] + px * b.e1[0] + py * b.e2[0];
    const float qy = b.iso[1] + px * b.e1[1] + py * b.e2[1];
    const float qz = b.iso[2] + px * b.e1[2] + py * b.e2[2];
    float ox, oy, oz, tlo;
    if (b.sad > 0.0f) {
        ox = b.iso[0] - b.sad * b.dir[0];
        oy = b.iso[1] - b.sad * b.dir[1];
        oz = b.iso[2] - b.sad * b.dir[2];
        const float dx = qx - ox, dy = qy - oy, dz = qz - oz;
        const float n = hrsq(dx * dx + dy * dy + dz * dz);
        p.u = dx * n;
        p.v = dy * n;
        p.w = dz * n;
        tlo = 0.0f;
    } else {
        ox = qx;
        oy = qy;
        oz = qz;
        p.u = b.dir[0];
        p.v = b.dir[1];
        p.w = b.dir[2];
        tlo = -3.0e38f;
    }
    // slab-method ray-box entry
    float tmin = tlo, tmax = 3.0e38f;
    int ax = -1;
    bool miss = false;
    const float o[3] = {ox, oy, oz}, dir[3] = {p.u, p.v, p.w}, L[3] = {G.lx, G.ly, G.lz};
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        if (dir[i] != 0.0f) {
            const float ta = (0.0f - o[i]) / dir[i], tb = (L[i] - o[i]) / dir[i];
            const float tn = fminf(ta, tb), tf = fmaxf(ta, tb);
            if (tn > tmin) {
                tmin = tn;
                ax = i;
            }
            tmax = fminf(tmax, tf);
        } else if (o[i] < 0.0f || o[i] > L[i]) {
            miss = true;
        }
    }
    p.in = !miss && tmax > tmin;
    p.x = ox + tmin * p.u;
    p.y = oy + tmin * p.v;
    p.z = oz + tmin * p.w;
    if (ax == 0) p.x = p.u > 0.0f ? 0.0f : G.lx;
    if (ax == 1) p.y = p.v > 0.0f ? 0.0f : G.ly;
    if (ax == 2) p.z = p.w > 0.0f ? 0.0f : G.lz;
    return p;
}
// ---------------------------------------------------------------------------
// arguments of the transport kernels, read from the kernel-argument segment
// where they are needed (see reread)
// ---------------------------------------------------------------------------
typedef const GDPM_CONST PassArgs* Args;
typedef const GDPM_CONST JobDev* JobPtr;
GDPM_DEV Args pass_args() { return (Args)__builtin_amdgcn_kernarg_segment_ptr(); }
// queue control fields that no one writes during a transport pass
GDPM_DEV const GDPM_CONST RingCtl* ring_const(Args A, int ri) {
    return &((const GDPM_CONST Ctl*)A->ctl)->ring[ri];
}

// the wavefronts that work in the pass (the first group_waves of each workgroup)
GDPM_DEV uint32_t pass_waves(Args A, int ri) { return gridDim.x * ring_const(A, ri)->group_waves; }

// ---------------------------------------------------------------------------
// queue reservation and claiming (wave-uniform state)
// ---------------------------------------------------------------------------
struct PushState {
    uint32_t next, end;  // reserved, unused ring slots [next, end)
    uint32_t chunk;      // slots reserved at a time
};

// Reserve `n` consecutive logical positions for this wave; item j of the wave
// lands in slot slot_of(j).  Returns false if the ring would exceed its hard
// limit (the run is then marked overflowed and the items are dropped).
struct Reservation {
    uint32_t old_next, old_avail, new_base;
    bool ok;
};

GDPM_DEV Reservation reserve(PushState& ps, Args A, int ri, uint32_t n) {
    Reservation r;
    r.old_next = ps.next;
    r.old_avail = ps.end - ps.next;
    r.new_base = 0;
    r.ok = true;
    if (n <= r.old_avail) {
        ps.next += n;
        return r;
    }
    GDPM_GLOBAL Ctl* ctl = global_ptr(A->ctl);
    const uint32_t chunk = max(ps.chunk, n - r.old_avail);
    const uint32_t leader = first_lane(ballot(true));
    uint32_t base = 0;
    if (lane_id() == leader) base = atomic_add(&ctl->ring[ri].tail, chunk);
    base = bcast(base, leader);
    if (base + chunk - ring_const(A, ri)->head > A->R.hard[ri]) {
        if (lane_id() == leader) atomic_or(&ctl->overflow, 1u);
        r.ok = false;
        ps.next = ps.end;
        return r;
    }
    r.new_base = base;
    ps.next = base + (n - r.old_avail);
    ps.end = base + chunk;
    return r;
}

GDPM_DEV uint32_t slot_of(const Reservation& r, uint32_t j) {
    return j < r.old_avail ? r.old_next + j : r.new_base + (j - r.old_avail);
}

GDPM_DEV GDPM_GLOBAL f4* record_ptr(Args A, int ri, uint32_t slot) {
    return (GDPM_GLOBAL f4*)(global_ptr(A->R.buf[ri]) + (slot & A->R.mask[ri]));
}

// mark the unused tail of this wave's reservation as empty slots
GDPM_DEV void release(PushState& ps, Args A, int ri) {
    // by offset from ps.next: queue positions run modulo 2^32, and a reserved
    // run may straddle the wrap (then ps.end < ps.next as numbers)
    const uint32_t n = ps.end - ps.next;
    for (uint32_t o = lane_id(); o < n; o += 64u)
        ((GDPM_GLOBAL float*)record_ptr(A, ri, ps.next + o))[3] = kEmptyEnergy;
    ps.next = ps.end;
}

// Counters kept per wavefront (scalar registers): updated only where the
// wavefront is converged, from ballots of the lanes concerned.
struct WaveTally {
    uint32_t events;      // flights (photon pass) or steps (electron pass)
    uint32_t real[2];     // photons: real interactions; electrons: hard-event
                          // candidates, hard events
    uint32_t dep;         // FP64 tally additions
    uint32_t pushes;      // secondaries written, all jobs
    uint32_t ld, rq;      // records loaded from the queue, records handed on
    uint32_t born, died;  // records created and particles ended, current job
    uint32_t bad;         // particles ended by the iteration bound of a wavefront
    uint32_t it[2];       // real interactions by type (photons: photoelectric,
                          // pair; electrons: Moller); Compton and bremsstrahlung
                          // are the rest of the real interactions and hard events
};
GDPM_DEV uint32_t count(bool p) { return (uint32_t)__popcll(ballot(p)); }

// a queue record as loaded: the four vectors of Particle
struct Rec {
    f4 a, b;   // x y z e; u v w nh
    u4 c, d;   // hlo hhi path ctr; vox a flags job
};

GDPM_DEV void write_record(GDPM_GLOBAL f4* q, const Rec& p) {
    q[0] = p.a;
    q[1] = p.b;
    ((GDPM_GLOBAL u4*)q)[2] = p.c;
    ((GDPM_GLOBAL u4*)q)[3] = p.d;
}

// Hand particles to the next pass of the same type (the record keeps the whole
// state, random stream position included, so nothing physical changes).
GDPM_DEV void requeue(bool active, PushState& ps, Args A, int ri, const Rec& p, WaveTally& c) {
    const uint64_t b = ballot(active);
    const uint32_t n = (uint32_t)__popcll(b);
    if (n == 0) return;
    const Reservation res = reserve(ps, A, ri, n);
    if (!res.ok) return;
    c.rq += n;
    if (active) write_record(record_ptr(A, ri, slot_of(res, mbcnt(b))), p);
}

// ---------------------------------------------------------------------------
// the job a wavefront works on (a wavefront only ever holds one job's
// particles).  Its data are read from the job table by scalar loads where they
// are used.
// ---------------------------------------------------------------------------
struct WJob {
    JobPtr p;
    int j;
    uint32_t tag;                    // slot | generation << 8: low half of the records' job word
    uint32_t seg_begin, seg_count;   // the job's records in the running pass
};

GDPM_DEV void load_job(WJob& w, Args A, int j, int ri) {
    j = __builtin_amdgcn_readfirstlane(j);
    w.p = (JobPtr)A->R.jobs + j;
    w.j = j;
    w.tag = (uint32_t)j | ((w.p->gen & 0xFFu) << 8);
    const GDPM_CONST JobCtl* jc = (const GDPM_CONST JobCtl*)A->R.jc;
    w.seg_begin = jc->seg_begin[ri][j];
    w.seg_count = jc->seg_count[ri][j];
}

// first job of a wavefront: the pass input is split over the wavefronts of the
// grid in proportion to the jobs' record counts; -1 if the pass is empty
GDPM_DEV int first_job(Args A, uint32_t total, int ri) {
    if (total == 0) return -1;
    const GDPM_CONST JobCtl* jc = (const GDPM_CONST JobCtl*)A->R.jc;
    const uint32_t waves = pass_waves(A, ri);
    const uint32_t w =
        __builtin_amdgcn_readfirstlane(blockIdx.x * ring_const(A, ri)->group_waves + (threadIdx.x >> 6));
    const uint32_t pos = (uint32_t)(((unsigned long long)w * total + total / 2) / waves);
    int lo = 0, hi = A->R.n_jobs - 1;   // last job whose segment starts at or before pos
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (jc->seg_begin[ri][mid] <= pos) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

GDPM_DEV unsigned long long load_agent64(const GDPM_GLOBAL unsigned long long* p) {
    const unsigned long long v = __hip_atomic_load(const_cast<GDPM_GLOBAL unsigned long long*>(p),
                                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return (unsigned long long)hi << 32 | lo;
}

// the next job after j (cyclically) with unclaimed records in this pass, or -1
GDPM_DEV int next_job(const GDPM_GLOBAL JobCtl* jc, int j, int n_jobs, int ri) {
    if (n_jobs <= 1) return -1;
    const int nw = (n_jobs + 63) >> 6;
    for (int k = 0; k <= nw; ++k) {
        const int wi = ((j >> 6) + k) % nw;
        unsigned long long m = load_agent64(&jc->left[ri][wi]);
        if (k == 0) {
            const int b = j & 63;   // only jobs after j in j's own word
            m = b == 63 ? 0ull : m & (~0ull << (b + 1));
        } else if (k == nw) {
            m &= (1ull << (j & 63)) - 1ull;   // jobs before j in j's word, last
        }
        if (m) {
            const int c = wi * 64 + (__ffsll(m) - 1);
            if (c < n_jobs && c != j) return c;
        }
    }
    return -1;
}

struct ClaimState {
    uint32_t next, end;  // claimed positions of the job's segment not yet handed out
    uint32_t seen;       // the job's claim counter as this wave last saw it
    bool done;           // the job's segment has nothing left to claim
};

// ---------------------------------------------------------------------------
// tallies
// ---------------------------------------------------------------------------
// deposits go to the batch slot `pb` of the particle's history; a split job's
// particles are tallied at weight 1 and the host scales the sums by 2^-split
// (exact: a power of two commutes with every rounding of the sum)
template <class R>
GDPM_DEV void add_history(JobPtr J, double de, const R& r) {
    if (J->hist) {
        const unsigned long long h = ((unsigned long long)r.hhi << 32 | r.hlo) - J->hist0;
        atomic_add_f64(global_ptr(J->hist) + 2 * h, de);
    }
}
template <class R>
GDPM_DEV void add_dose(JobPtr J, uint32_t pb, uint32_t pos, double de, const R& r) {
    atomic_add_f64(global_ptr(J->tally) + ((unsigned long long)pb * J->nv + pos), de);
    add_history(J, de, r);
}

// positions in a tally (see Brick)
struct TallyOrder {
    int mx, my, mz, sy, sz, s;   // widths less one; the voxel's bit positions; log2 of the brick's size
    int nbx, nby;                // bricks along x and y
    GDPM_DEV TallyOrder(int x, int y, int z, int nx, int ny)
        : mx(x), my(y), mz(z), sy(x), sz(x + y), s(x + y + z), nbx(nx >> x), nby(ny >> y) {}
    GDPM_DEV uint32_t brick(int ix, int iy, int iz) const {
        return (uint32_t)((ix >> mx) + nbx * ((iy >> my) + nby * (iz >> mz)));
    }
    GDPM_DEV uint32_t voxel(int ix, int iy, int iz) const {   // in its brick
        return (uint32_t)((ix & mx) | (iy & my) << sy | (iz & mz) << sz);
    }
    GDPM_DEV uint32_t pos(int ix, int iy, int iz) const { return brick(ix, iy, iz) << s | voxel(ix, iy, iz); }
};
template <class J>
GDPM_DEV TallyOrder tally_order(const J& job, int nx, int ny) {
    return TallyOrder(job.brick.mx, job.brick.my, job.brick.mz, nx, ny);
}

// energy leaving the phantom: per-history output (test mode)
template <class R>
GDPM_DEV void history_escape(JobPtr J, double e, const R& r) {
    if (J->hist) {
        const unsigned long long h = ((unsigned long long)r.hhi << 32 | r.hlo) - J->hist0;
        atomic_add_f64(global_ptr(J->hist) + 2 * h + 1, e);
    }
}

// What a workgroup counts, in LDS: the jobs' particle births and deaths and
// escaped energy, and the pass counters of the two particle types.  The
// wavefronts add to it when they leave a job and when they end, and the
// workgroup folds it into global memory once.  With every wavefront adding its
// own counters to global memory, a pass with next to no work took 130 us: 3072
// wavefronts x 14 additions to a few lines.
struct GroupTally {
    uint32_t born[kMaxJobs], died[kMaxJobs];
    double esc[kMaxJobs];
    uint32_t pc[2][kPassCounters];
};
constexpr uint32_t kGroupTallyF4 = (sizeof(GroupTally) + 15u) / 16u;
typedef GDPM_LDS GroupTally* GroupPtr;

template <class T>
GDPM_DEV void lds_add(GDPM_LDS T* p, T v) {
    (void)__hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
GDPM_DEV void group_clear(GroupPtr g) {
    GDPM_LDS uint32_t* w = (GDPM_LDS uint32_t*)g;
    for (uint32_t i = threadIdx.x; i < sizeof(GroupTally) / 4u; i += blockDim.x) w[i] = 0u;
}

// fold the per-job counters of a wavefront into the workgroup's (before a
// switch, at the end)
GDPM_DEV void job_flush(double& e_esc, WaveTally& c, int j, GroupPtr g) {
    const double esc = wave_sum(e_esc);
    if (lane_id() == 0) {
        if (esc != 0.0) lds_add(&g->esc[j], esc);
        if (c.born) lds_add(&g->born[j], c.born);
        if (c.died) lds_add(&g->died[j], c.died);
    }
    e_esc = 0.0;
    c.pushes += c.born;
    c.born = c.died = 0u;
}

// fold the pass counters of a wavefront into the workgroup's
GDPM_DEV void pass_finish(const WaveTally& c, int ri, GroupPtr g) {
    if (lane_id() == 0) {
        GDPM_LDS uint32_t* p = g->pc[ri];
        auto add = [p](int i, uint32_t v) {
            if (v) lds_add(p + i, v);
        };
        add(PC_EVENTS, c.events);
        add(PC_REAL, c.real[0]);
        add(PC_HARD, c.real[1]);
        add(PC_DEPOSITS, c.dep);
        add(PC_PUSHES, c.pushes);
        add(PC_LOADED, c.ld);
        add(PC_REQUEUED, c.rq);
        add(PC_ANOMALIES, c.bad);
        add(PC_TYPE0, c.it[0]);
        add(PC_TYPE1, c.it[1]);
    }
}

// fold the workgroup's counters into the jobs' and the pass's (every thread of
// the workgroup takes part)
GDPM_DEV void group_flush(Args A, GroupPtr g) {
    __syncthreads();
    GDPM_GLOBAL JobCtl* jc = global_ptr(A->R.jc);
    const int n_jobs = A->R.n_jobs;
    for (int j = (int)threadIdx.x; j < n_jobs; j += blockDim.x) {
        if (g->esc[j] != 0.0) atomic_add_f64(&jc->e_esc[j], g->esc[j]);
        if (g->born[j]) atomic_add(&jc->births[j], (unsigned long long)g->born[j]);
        if (g->died[j]) atomic_add(&jc->deaths[j], (unsigned long long)g->died[j]);
    }
    for (int i = (int)threadIdx.x; i < 2 * kPassCounters; i += blockDim.x) {
        const uint32_t v = g->pc[i / kPassCounters][i % kPassCounters];
        if (v)
            atomic_add(&jc->part[i / kPassCounters][blockIdx.x % kParts][i % kPassCounters], (unsigned long long)v);
    }
}

// ---------------------------------------------------------------------------
// samplers (the draw order is part of the contract with the reference)
// ---------------------------------------------------------------------------

// Klein-Nishina: eps = E'/E where the distribution function reaches one
// uniform draw u, from the tabulated inverse (bilinear in log2 E and u, of
// q = ln(eps/eps0)/ln(1/eps0), so that eps = eps0^(1 - q)); then
// t = 1 - cos(theta) and the azimuth (in turns).  No rejection: every lane
// of a wavefront runs the same instructions.
template <class TT, class RNG>
GDPM_DEV void sample_compton(const TT& T, RNG& r, uint32_t k0, uint32_t k1, float e, float& eps,
                             float& t, float& turns) {
    const float k = e * (1.0f / kMec2f);
    const float u = uniform(r, k0, k1);
    float fe = (hlog2(e) - T.kn_lo) * T.kn_inv;
    fe = fminf(fmaxf(fe, 0.0f), (float)(T.kn_ne - 1));
    const int i = min((int)fe, T.kn_ne - 2);
    const float a = fe - (float)i;
    const float fu = u * (float)(T.kn_nu - 1);
    const int j = min((int)fu, T.kn_nu - 2);
    const float b = fu - (float)j;
    const GDPM_GLOBAL float* p = global_ptr(T.kn) + (i * T.kn_nu + j);
    const float q0 = fmaf(b, p[1] - p[0], p[0]);
    const float q1 = fmaf(b, p[T.kn_nu + 1] - p[T.kn_nu], p[T.kn_nu]);
    const float q = fmaf(a, q1 - q0, q0);
    eps = fminf(hexp2(-hlog2(1.0f + 2.0f * k) * (1.0f - q)), 1.0f);
    t = (1.0f - eps) * hrcp(k) * hrcp(eps);
    turns = uniform(r, k0, k1);
}

// Moller: eps = W/T by a 1/eps^2 proposal on [W_cc/T, 1/2] and rejection
// eps^2 B(eps) / 2.25; then the azimuth
template <class RNG>
GDPM_DEV void sample_moller(RNG& r, uint32_t k0, uint32_t k1, float tt, float wcc, float& eps,
                            float& turns) {
    const float g = 1.0f + tt * (1.0f / kMec2f), e0 = fdiv(wcc, tt);
    const float ig = hrcp(g);
    const float c1 = (g - 1.0f) * ig, c2 = (2.0f * g - 1.0f) * ig * ig;
    for (;;) {
        // a trial takes two draws, and the azimuth after the last one a third
        r.ensure(3u, k0, k1);
        const float ua = uniform(r, k0, k1);
        eps = fdiv(e0, 1.0f - ua * (1.0f - 2.0f * e0));
        const float ub = uniform(r, k0, k1);
        const float ie = hrcp(eps), io = hrcp(1.0f - eps);
        const float br = c1 * c1 + ie * (ie - c2) + io * (io - c2);
        if (ub * 2.25f <= eps * eps * br) break;
    }
    turns = uniform(r, k0, k1);
}

// bremsstrahlung photon energy: 1/k proposal on [W_cb, T], rejection by the
// complete-screening spectrum
template <class RNG>
GDPM_DEV float sample_brems(RNG& r, uint32_t k0, uint32_t k1, float tt, float wcb) {
    const float lr = hlog2(tt) - hlog2(wcb);
    const float it = hrcp(tt);
    float kph;
    for (;;) {
        r.ensure(2u, k0, k1);
        const float ua = uniform(r, k0, k1);
        // the hardware log2 and exp2 are within about an ulp each, so near
        // ua = 1 their product could exceed T by a few ulps and leave the
        // electron a negative energy: the photon takes at most T
        kph = fminf(wcb * hexp2(ua * lr), tt);
        const float ub = uniform(r, k0, k1);
        const float yy = kph * it;
        if (ub * (4.0f / 3.0f) <= 4.0f / 3.0f - 4.0f / 3.0f * yy + yy * yy) break;
    }
    return kph;
}

// isotropic direction of the first annihilation photon (cos, then azimuth)
template <class RNG>
GDPM_DEV void sample_iso(RNG& r, uint32_t k0, uint32_t k1, float& du, float& dv, float& dw) {
    const float ct = 2.0f * uniform(r, k0, k1) - 1.0f;
    const float turns = uniform(r, k0, k1);
    const float st = hsqrt((1.0f - ct) * (1.0f + ct));
    du = st * cos_turns(turns);
    dv = st * sin_turns(turns);
    dw = ct;
}

// Compton electron: along the momentum transfer E d0 - E' d of a photon
// turned from d0 to d with E -> E' (no binding: momentum conservation)
GDPM_DEV void compton_electron_dir(float e, float e1, float u0, float v0, float w0, float u, float v,
                                   float w, float& eu, float& ev, float& ew) {
    eu = e * u0 - e1 * u;
    ev = e * v0 - e1 * v;
    ew = e * w0 - e1 * w;
    const float nn = eu * eu + ev * ev + ew * ew;
    if (nn > 0.0f) {
        const float in = hrsq(nn);
        eu *= in; ev *= in; ew *= in;
    } else {
        eu = u0; ev = v0; ew = w0;
    }
}

// pair production: K = E - 2 mc^2 split at the uniform u (T- = u K), the
// larger part computed and the smaller taken as K minus it, so that
// T- + T+ = K exactly; the positron keeps a = E - K
GDPM_DEV void pair_split(float e, float u, float& tm, float& tp, float& aa) {
    const float kk = e - kTwoMec2f;
    aa = e - kk;
    const float tc = u * kk;
    tp = kk - tc;
    tm = 2.0f * tc >= kk ? tc : kk - tp;
}

// ---------------------------------------------------------------------------
// secondaries of one event, pushed with the wave converged
// ---------------------------------------------------------------------------
// charged: up to two; the second (a positron) shares the first one's direction
struct PendCharged {
    int n;
    float e0, du, dv, dw;   // first particle and the common direction
    float a0;               // first particle: annihilation energy if it is a positron
    uint32_t role;          // first particle: role word
    float e1, a1;           // second particle (always the pair positron, role 1)
};
// photons: one (role word wb) or two back to back (roles wb, wb + 1)
struct PendPhoton {
    int n;
    float e, u, v, w;
    uint32_t wb;
};

// a new particle of annihilation energy a (0: an electron or a photon)
template <class R>
GDPM_DEV void write_particle(GDPM_GLOBAL f4* q, float x, float y, float z, float e, float u, float v, float w,
                             const R& r, uint32_t path, uint32_t vox, float a, uint32_t job) {
    q[0] = f4{x, y, z, e};
    q[1] = f4{u, v, w, -1.0f};
    ((GDPM_GLOBAL u4*)q)[2] = u4{r.hlo, r.hhi, path, 0u};
    ((GDPM_GLOBAL u4*)q)[3] = u4{vox, __float_as_uint(a), a > 0.0f ? 1u : 0u, job};
}

// secondaries inherit the job and the batch slot (`jb`) of their history
template <class R>
GDPM_DEV void push_charged(const PendCharged& q, PushState& ps, Args A, JobPtr J, uint32_t jb, float x, float y,
                           float z, uint32_t vox, const R& rng, WaveTally& c) {
    const uint64_t b0 = ballot(q.n >= 1), b1 = ballot(q.n >= 2);
    const uint32_t n0 = (uint32_t)__popcll(b0), n = n0 + (uint32_t)__popcll(b1);
    if (n == 0) return;
    const Reservation res = reserve(ps, A, 1, n);
    if (!res.ok) return;
    if (q.n > 0)
        write_particle(record_ptr(A, 1, slot_of(res, mbcnt(b0))), x, y, z, q.e0, q.du, q.dv, q.dw, rng,
                       spawn_path(rng, J->k0, J->k1, (int)q.role), vox, q.a0, jb);
    if (q.n > 1)
        write_particle(record_ptr(A, 1, slot_of(res, n0 + mbcnt(b1))), x, y, z, q.e1, q.du, q.dv, q.dw, rng,
                       spawn_path(rng, J->k0, J->k1, 1), vox, q.a1, jb);
    c.born += n;
}

template <class R>
GDPM_DEV void push_photons(const PendPhoton& q, PushState& ps, Args A, JobPtr J, uint32_t jb, float x, float y,
                           float z, const R& rng, WaveTally& c) {
    const uint64_t b0 = ballot(q.n >= 1), b1 = ballot(q.n >= 2);
    const uint32_t n0 = (uint32_t)__popcll(b0), n = n0 + (uint32_t)__popcll(b1);
    if (n == 0) return;
    const Reservation res = reserve(ps, A, 0, n);
    if (!res.ok) return;
    if (q.n > 0)
        write_particle(record_ptr(A, 0, slot_of(res, mbcnt(b0))), x, y, z, q.e, q.u, q.v, q.w, rng,
                       spawn_path(rng, J->k0, J->k1, (int)q.wb), 0u, 0.0f, jb);
    if (q.n > 1)
        write_particle(record_ptr(A, 0, slot_of(res, n0 + mbcnt(b1))), x, y, z, q.e, -q.u, -q.v, -q.w, rng,
                       spawn_path(rng, J->k0, J->k1, (int)q.wb + 1), 0u, 0.0f, jb);
    c.born += n;
}

// ---------------------------------------------------------------------------
// pass set-up and completion (one block, between passes): the job segments
// come from the re-binning that precedes every pass
// ---------------------------------------------------------------------------
// rebinned = 0: the queue was not re-binned because only job `lone` holds
// particles: the whole queue, empty slots included, is that job's segment and
// the other jobs' segments are empty (they start at its end, so that a
// wavefront's first job is `lone`)
// In a pass of one job's queue, read as
// it is, wavefront w starts with records [w first, (w + 1) first) of the
// segment, without claiming them, and claims begin after those of the last.
GDPM_DEV uint32_t claim_size(uint32_t left, uint32_t waves, int ri) {
    return min(max(left / (2u * waves), kClaimMin), ri == 0 ? kClaimMaxPhoton : kClaimMaxElectron);
}
GDPM_DEV void setup_pass(Ctl* ctl, const RunDev& R, int ri, int rebinned, int lone, PassGrid grid) {
    JobCtl* jc = R.jc;
    RingCtl& r = ctl->ring[ri];
    // a permuted pass reads positions [0, n_valid) of the permutation; its
    // records stay in [head, tail), which it consumes whole
    const bool perm = rebinned && r.permuted;
    const uint32_t count = ctl->overflow ? 0u : (perm ? ctl->n_valid : r.tail - r.head);
    // of several jobs a wavefront takes one after the other, so it counts what each has
    const uint32_t lanes = 64u * grid.blocks * grid.wide;
    static_assert(kMaxJobs <= 256, "one thread per job");
    const uint32_t jobs =
        rebinned ? (uint32_t)__syncthreads_count((int)threadIdx.x < R.n_jobs && jc->seg_count[ri][threadIdx.x] > 0u) : 1u;
    const uint32_t group_waves = count >= kWideMin * lanes && count >= kWideMinJob * jobs * lanes ? grid.wide : grid.narrow;
    const uint32_t waves = grid.blocks * group_waves;
    if (!rebinned)
        for (int j = threadIdx.x; j < R.n_jobs; j += blockDim.x) {
            jc->seg_begin[ri][j] = j <= lone ? 0u : count;
            jc->seg_count[ri][j] = j == lone ? count : 0u;
        }
    __syncthreads();
    for (int j = threadIdx.x; j < R.n_jobs; j += blockDim.x)
        jc->claim[ri][j] = rebinned ? 0u : waves * claim_size(count, waves, ri);
    const int nw = (R.n_jobs + 63) >> 6;
    for (int k = threadIdx.x; k < kMaxJobs / 64; k += blockDim.x) {
        unsigned long long m = 0ull;
        if (k < nw && !ctl->overflow)
            for (int b = 0; b < 64 && k * 64 + b < R.n_jobs; ++b)
                if (jc->seg_count[ri][k * 64 + b] > 0u) m |= 1ull << b;
        jc->left[ri][k] = m;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        r.begin = perm ? 0u : r.head;
        r.count = count;
        r.group_waves = group_waves;
        const uint32_t claim = claim_size(count, waves, ri);
        r.first = rebinned ? 0u : claim;
        // (the slots that all wavefronts leave unused are no more with `wide` of them)
        r.push = min(max(claim, kPushMin), kPushMax * grid.narrow / group_waves);
        r.next_head = r.tail;
        if (!perm) r.permuted = 0u;
    }
}
__global__ void __launch_bounds__(256) k_setup(Ctl* ctl, RunDev R, int ri, int rebinned, int lone, PassGrid grid) {
    setup_pass(ctl, R, ri, rebinned, lone, grid);
}

// completion of a pass, by the first wavefront of a workgroup; clock: the slot of
// Ctl::ticks that its time goes to (-1: none)
GDPM_DEV void finish_pass(Ctl* ctl, JobCtl* jc, int ri, int clock) {
    if (threadIdx.x >= 64) return;
    if (threadIdx.x == 0) {
        RingCtl& r = ctl->ring[ri];
        r.head = r.permuted ? r.next_head : r.begin + r.count;
        r.count = 0u;
        r.permuted = 0u;
        if (clock >= 0) ctl->ticks[clock] += wall_clock64() - ctl->t_start;
    }
    // the pass counters of the workgroups: lane i folds counter i
    unsigned long long v = 0ull;
    if (threadIdx.x < (unsigned)kPassCounters)
        for (int k = 0; k < kParts; ++k) {
            v += jc->part[ri][k][threadIdx.x];
            jc->part[ri][k][threadIdx.x] = 0ull;
        }
    switch (threadIdx.x) {
        case PC_EVENTS: ctl->ev[ri == 0 ? EV_FLIGHTS : EV_ESTEPS] += v; break;
        case PC_REAL: ctl->ev[ri == 0 ? EV_REAL : EV_HARD_CAND] += v; break;
        case PC_HARD: ctl->ev[EV_HARD] += v; break;
        case PC_DEPOSITS:
            ctl->ev[EV_DEPOSITS] += v;
            ctl->pass_ev[ri][2] += v;
            break;
        case PC_LOADED: ctl->pass_ev[ri][0] += v; break;
        case PC_ANOMALIES: ctl->anomalies += v; break;
        case PC_TYPE0: ctl->itype[ri == 0 ? 1 : 3] += v; break;
        case PC_TYPE1: ctl->itype[2] += v; break;
        default: break;
    }
    const unsigned long long rq = __shfl(v, PC_REQUEUED), pushes = __shfl(v, PC_PUSHES);
    if (threadIdx.x == 0) {
        ctl->ev[EV_PUSHES] += pushes;
        ctl->pass_ev[ri][1] += pushes + rq;
        ctl->pass_ev[ri][3] += rq;
    }
}

// ---------------------------------------------------------------------------
// The ends of a scheduler iteration.  An iteration is a chain of small kernels
// around the passes, and most of a small job's time went into the gaps between
// them: copies to and from the host, timing events (6 us on either side of a
// pass), set-up and completion apart.  The first kernel reads the iteration's
// source segments from pinned host memory, the last writes the counters there
// and then the iteration's number, which the host waits for.
// ---------------------------------------------------------------------------
// what is written here is read by the passes' kernels, or by the host
GDPM_DEV void host_store(unsigned long long* p, unsigned long long v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}
// a value this kernel may have just changed
GDPM_DEV unsigned long long fresh(const unsigned long long* p) {
    return __hip_atomic_load(const_cast<unsigned long long*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// setup: bit ri set: also set up pass ri (a pass that is not re-binned first)
__global__ void __launch_bounds__(256) k_begin(Ctl* ctl, RunDev R, const StepHost* h, SrcHdr* hdr, SrcSeg* segs,
                                               int setup, int lone, PassGrid grid0, PassGrid grid1) {
    __shared__ uint32_t n[2];
    if (threadIdx.x < 2) {
        const int ri = threadIdx.x;
        SrcHdr d = h->hdr[ri];
        n[ri] = d.nseg;
        RingCtl& r = ctl->ring[ri];
        // the records are part of the queue from here on; the source kernels
        // write them at [base, base + total)
        d.base = r.tail;
        if (d.total) {
            if (r.tail + d.total - r.head > R.hard[ri]) atomicOr(&ctl->overflow, 1u);
            else r.tail += d.total;
        }
        hdr[ri] = d;
    }
    __syncthreads();
    constexpr int kCap = kMaxSegs / 2, kWords = sizeof(SrcSeg) / 8;
    static_assert(sizeof(SrcSeg) % 8 == 0, "copied in 8-byte words");
    for (int ri = 0; ri < 2; ++ri) {
        const unsigned long long* q = reinterpret_cast<const unsigned long long*>(h->segs + ri * kCap);
        unsigned long long* d = reinterpret_cast<unsigned long long*>(segs + ri * kCap);
        for (uint32_t i = threadIdx.x; i < n[ri] * kWords; i += blockDim.x) d[i] = q[i];
    }
    if (setup & 1) setup_pass(ctl, R, 0, 0, lone, grid0);
    if (setup & 2) setup_pass(ctl, R, 1, 0, lone, grid1);
}

// between the passes: completion of the photon pass, set-up of the electron pass
__global__ void __launch_bounds__(256) k_mid(Ctl* ctl, RunDev R, int setup, int lone, PassGrid grid) {
    finish_pass(ctl, R.jc, 0, 0);
    if (setup) setup_pass(ctl, R, 1, 0, lone, grid);
}

// the end of an iteration; fused: one launch ran both passes
__global__ void __launch_bounds__(256) k_end(Ctl* ctl, RunDev R, const StepHost* h, StepMirror* out, int fused) {
    if (fused) finish_pass(ctl, R.jc, 0, 2);
    finish_pass(ctl, R.jc, 1, fused ? -1 : 1);
    __threadfence();
    __syncthreads();
    static_assert(sizeof(Ctl) % 8 == 0, "copied in 8-byte words");
    const unsigned long long* c = reinterpret_cast<const unsigned long long*>(ctl);
    unsigned long long* o = reinterpret_cast<unsigned long long*>(&out->ctl);
    for (uint32_t i = threadIdx.x; i < sizeof(Ctl) / 8; i += blockDim.x) host_store(o + i, fresh(c + i));
    const JobCtl* jc = R.jc;
    for (int j = threadIdx.x; j < R.n_jobs; j += blockDim.x) {
        host_store(&out->births[j], jc->births[j]);
        host_store(&out->deaths[j], jc->deaths[j]);
        host_store(reinterpret_cast<unsigned long long*>(&out->e_in[j]), __double_as_longlong(jc->e_in[j]));
        host_store(reinterpret_cast<unsigned long long*>(&out->e_esc[j]), __double_as_longlong(jc->e_esc[j]));
    }
    __threadfence_system();
    __syncthreads();
    if (threadIdx.x == 0)
        __hip_atomic_store(&out->seq, h->seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// the control blocks at the start of a run (queues empty, at position `start`)
__global__ void __launch_bounds__(1024) k_init(Ctl* ctl, JobCtl* jc, StatsDev* stats, uint32_t start) {
    uint32_t* c = reinterpret_cast<uint32_t*>(ctl);
    for (uint32_t i = threadIdx.x; i < sizeof(Ctl) / 4; i += blockDim.x) c[i] = 0u;
    uint32_t* q = reinterpret_cast<uint32_t*>(jc);
    for (uint32_t i = threadIdx.x; i < sizeof(JobCtl) / 4; i += blockDim.x) q[i] = 0u;
    uint32_t* t = reinterpret_cast<uint32_t*>(stats);
    for (uint32_t i = threadIdx.x; i < offsetof(StatsDev, inv_n) / 4; i += blockDim.x) t[i] = 0u;
    __syncthreads();
    if (threadIdx.x < 2) {
        RingCtl& r = ctl->ring[threadIdx.x];
        r.head = r.tail = r.begin = start;
    }
}

// a job enters slot `slot`: its description, its majorant (from pinned host
// memory), zero counters and tallies
struct AdmitArgs {
    JobDev job;
    JobDev* jobs;
    JobCtl* jc;
    const float* majorant;   // pinned host memory, n_grid values
    float* mumax;
    size_t n_tally, n_hist;  // doubles
    int slot, n_grid;
};
__global__ void __launch_bounds__(256) k_admit(AdmitArgs a) {
    const size_t t = blockIdx.x * (size_t)blockDim.x + threadIdx.x, n = (size_t)gridDim.x * blockDim.x;
    for (size_t i = t; i < (size_t)a.n_grid; i += n) a.mumax[i] = a.majorant[i];
    double2* q = reinterpret_cast<double2*>(a.job.tally);   // (at least 256-byte aligned)
    for (size_t i = t; i < a.n_tally / 2; i += n) q[i] = make_double2(0.0, 0.0);
    if (t == 0 && (a.n_tally & 1)) a.job.tally[a.n_tally - 1] = 0.0;
    for (size_t i = t; i < a.n_hist; i += n) a.job.hist[i] = 0.0;
    if (t == 0) {
        a.jobs[a.slot] = a.job;
        a.jc->births[a.slot] = a.jc->deaths[a.slot] = 0ull;
        a.jc->e_in[a.slot] = a.jc->e_esc[a.slot] = 0.0;
    }
}

// ---------------------------------------------------------------------------
// claiming input: positions [0, seg_count) of the job's segment
// ---------------------------------------------------------------------------
// (kPerm: other jobs may have records in the pass, and look for them in the
// masks of unclaimed jobs)
template <bool kPerm>
GDPM_DEV void claim_refill(ClaimState& cs, Args A, const WJob& W, int ri) {
    if (cs.done || cs.next != cs.end) return;
    // the wave has used up its items: claim a new chunk if the job has more.
    // Chunks shrink as the segment drains (guided self-scheduling), so that the
    // last items spread over many wavefronts.  The shared counters are touched
    // once per claim, never per iteration.
    GDPM_GLOBAL Ctl* ctl = global_ptr(A->ctl);
    GDPM_GLOBAL JobCtl* jc = global_ptr(A->R.jc);
    const uint32_t count = W.seg_count;
    const uint32_t waves = pass_waves(A, ri);
    const uint32_t left = count - min(cs.seen, count);
    const uint32_t chunk = claim_size(left, waves, ri);
    if (load_agent(&ctl->overflow)) {   // a queue overflowed: the run is void
        cs.done = true;
        return;
    }
    const uint32_t leader = first_lane(ballot(true));
    uint32_t base = 0;
    if (lane_id() == leader) base = atomic_add(&jc->claim[ri][W.j], chunk);
    base = bcast(base, leader);
    cs.seen = base + chunk;
    if (base >= count) {
        if (kPerm && lane_id() == leader)
            (void)__hip_atomic_fetch_and(&jc->left[ri][W.j >> 6], ~(1ull << (W.j & 63)), __ATOMIC_RELAXED,
                                         __HIP_MEMORY_SCOPE_AGENT);
        cs.done = true;
        return;
    }
    cs.next = base;
    cs.end = min(base + chunk, count);
}

// the claims of a wavefront that starts on a job; `first`: what it takes
// without claiming (see k_setup).  The wavefronts of a workgroup start far apart
// in the segment, so that a small pass spreads over the CUs.
GDPM_DEV ClaimState claim_start(const WJob& W, uint32_t first, uint32_t waves) {
    ClaimState cs{0u, 0u, 0u, false};
    if (first) {
        const uint32_t w = __builtin_amdgcn_readfirstlane((threadIdx.x >> 6) * gridDim.x + blockIdx.x);
        cs.next = min(w * first, W.seg_count);
        cs.end = min(cs.next + first, W.seg_count);
        cs.seen = waves * first;
        cs.done = cs.next == cs.end;
    }
    return cs;
}

// the queue position of input position `pos` of a pass: itself, or through the
// permutation of a pass re-binned by job (`perm` non-null); both masked, so
// that any value reads inside the queue
GDPM_DEV uint32_t input_slot(const GDPM_GLOBAL uint32_t* perm, uint32_t mask, uint32_t pos) {
    return (perm ? perm[pos & mask] : pos) & mask;
}

// refill the lanes without a particle from the wave's claimed items; returns
// true in the lanes that loaded a record.  Lanes wait until kRefillMin of them
// are empty (or no lane is busy): a refill stalls the wavefront on record
// loads, so it pays to do it for several lanes at once.  kSolo (a
// measurement form): one particle per wavefront at a time, so the wavefront
// executes exactly the instructions of that particle's path.
template <bool kSolo, bool kPerm>
GDPM_DEV bool refill(bool active, ClaimState& cs, Args A, const WJob& W, int ri, uint32_t begin,
                     const GDPM_GLOBAL uint32_t* perm, Rec& p, WaveTally& c) {
    if (cs.done) return false;
    const uint64_t need = ballot(!active);
    if (!need) return false;
    if constexpr (kSolo) {
        if (ballot(active)) return false;
    } else {
        if ((uint32_t)__popcll(need) < kRefillMin && ballot(active)) return false;
    }
    claim_refill<kPerm>(cs, A, W, ri);
    const uint32_t have = cs.end - cs.next;
    const uint32_t rank = mbcnt(need);
    const uint32_t take = kSolo ? min(have, 1u) : min(have, (uint32_t)__popcll(need));
    const uint32_t first = begin + W.seg_begin;
    bool got = false;
    if (!active && rank < take) {
        const GDPM_GLOBAL f4* q = record_ptr(A, ri, input_slot(perm, A->R.mask[ri], first + cs.next + rank));
        p.a = q[0];
        p.b = q[1];
        p.c = ((const GDPM_GLOBAL u4*)q)[2];
        p.d = ((const GDPM_GLOBAL u4*)q)[3];
        got = !record_empty(p.a.w);
        if (got && (p.d.w & 0xFFFFu) != W.tag) {
            // a record of another job (or of an earlier job in this slot) in
            // this job's segment: only a broken bookkeeping puts it there; it
            // is dropped and counted
            atomic_add(&global_ptr(A->ctl)->anomalies, 1ull);
            got = false;
        }
    }
    cs.next += take;
    c.ld += take;
    return got;
}

// ---------------------------------------------------------------------------
// source pass: segments of new histories (job, first id, count, batch slot) ->
// primaries in the queue of the source particle type (section 2.3); a primary
// whose ray misses the phantom leaves an empty slot and counts as escaped
// ---------------------------------------------------------------------------
// The segments are cut into units, and each wavefront takes a run of consecutive
// units: 64 histories of a segment, or, for a Metropolis source, a group of chains
// through all of the job's segments.  With all workgroups on one segment after the
// other, each added its sums to the job's counters after every segment: 24 us a
// segment, and a round of ten batches has ten.  What bounds it now is the
// writing of the records (64 B each), so these go through LDS to be
// written as whole lines.
struct SourceArgs {
    Ctl* ctl;
    RunDev R;
    const SrcSeg* segs;
    const SrcHdr* hdr;
    int ri;
};
struct SourceTally {   // of a workgroup, per job
    double e_in[kMaxJobs], e_esc[kMaxJobs];
    uint32_t born[kMaxJobs];
};

// the records of a history: its 2^split copies, copy c on stream path c (copy 0
// is the unsplit primary)
GDPM_DEV Rec primary_record(const Primary& p, unsigned long long h, uint32_t copy, uint32_t vox, uint32_t jb) {
    Rec r;
    // the stream continues at the draw after the source's draws
    r.a = f4{p.x, p.y, p.z, p.in ? p.e : kEmptyEnergy};
    r.b = f4{p.u, p.v, p.w, -1.0f};
    r.c = u4{(uint32_t)h, (uint32_t)(h >> 32), copy, p.draws};
    r.d = u4{vox, 0u, 0u, jb};
    return r;
}

__global__ void __launch_bounds__(256) k_source(SourceArgs) {
    const GDPM_CONST SourceArgs* A = (const GDPM_CONST SourceArgs*)__builtin_amdgcn_kernarg_segment_ptr();
    __shared__ SourceTally tally;
    __shared__ f4 line[4][4 * 64];
    if (((const GDPM_CONST Ctl*)A->ctl)->overflow) return;
    const GDPM_CONST SrcHdr* hdr = (const GDPM_CONST SrcHdr*)A->hdr;
    const GDPM_CONST SrcSeg* segs = (const GDPM_CONST SrcSeg*)A->segs;
    const int nseg = (int)hdr->nseg, ri = A->ri;
    const uint32_t base = hdr->base, units = hdr->units;
    for (uint32_t i = threadIdx.x; i < sizeof(SourceTally) / 4u; i += blockDim.x)
        reinterpret_cast<uint32_t*>(&tally)[i] = 0u;
    __syncthreads();
    GDPM_LDS f4* lds = (GDPM_LDS f4*)line[threadIdx.x >> 6];
    const uint32_t lane = lane_id();
    const uint32_t waves = gridDim.x * (blockDim.x >> 6);
    const uint32_t w = __builtin_amdgcn_readfirstlane(blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6));
    const uint32_t per = (units + waves - 1u) / waves;
    const uint32_t c1 = min((w + 1u) * per, units);
    uint32_t c = min(w * per, units);
    int s = 0;   // the last segment that starts at or before unit c
    for (int hi = nseg - 1; s < hi;) {
        const int mid = (s + hi + 1) >> 1;
        if (segs[mid].unit0 <= c) s = mid;
        else hi = mid - 1;
    }
    double e_in = 0.0, e_esc = 0.0;
    uint32_t born = 0u;
    int job = -1;
    // a wavefront's sums of one job
    auto flush = [&]() {
        if (job < 0) return;
        const double in = wave_sum(e_in), out = wave_sum(e_esc);
        if (lane == 0) {
            lds_add((GDPM_LDS double*)&tally.e_in[job], in);
            if (out != 0.0) lds_add((GDPM_LDS double*)&tally.e_esc[job], out);
            lds_add((GDPM_LDS uint32_t*)&tally.born[job], born);
        }
        e_in = e_esc = 0.0;
        born = 0u;
    };
    for (; c < c1; ++c) {
        while (s + 1 < nseg && segs[s + 1].unit0 <= c) ++s;
        const GDPM_CONST SrcSeg* sg = segs + s;
        if ((int)sg->job != job) {
            flush();
            job = (int)sg->job;
        }
        const JobPtr J = (JobPtr)A->R.jobs + job;
        const uint32_t k0 = J->k0, k1 = J->k1;
        const uint32_t copies = 1u << J->split;
        const uint32_t tag = (uint32_t)job | ((J->gen & 0xFFu) << 8);
        // counts and, if its records are not written together, writes a primary
        auto account = [&](const Primary& p, unsigned long long h, bool live) {
            if (!live) return;
            e_in += (double)p.e;
            if (!p.in) {
                // all copies escape: weight 1 each, like the tallies
                const double out = (double)p.e * (double)copies;
                e_esc += out;
                if (J->hist) atomic_add_f64(global_ptr(J->hist) + 2 * (h - J->hist0) + 1, out);
            }
        };
        auto voxel = [&](const Primary& p) {
            if (ri == 0 || !p.in) return 0u;
            int ix, iy, iz;
            voxel_of(J->G, p.x, p.y, p.z, ix, iy, iz);
            return pack_vox(ix, iy, iz);
        };
        auto write = [&](const Primary& p, unsigned long long h, uint32_t first, uint32_t jb) {
            const uint32_t vox = voxel(p);
            for (uint32_t k = 0; k < copies; ++k)
                write_record((GDPM_GLOBAL f4*)(global_ptr(A->R.buf[ri]) + ((base + first + k) & A->R.mask[ri])),
                             primary_record(p, h, k, vox, jb));
        };
        if (!J->S.metro) {
            const uint32_t i0 = (c - sg->unit0) * 64u, i = i0 + lane;
            const uint32_t n = min(64u, sg->n - i0);   // histories of this unit
            const bool live = lane < n;
            const unsigned long long h = sg->h0 + (live ? i : i0);
            Primary p;
            if (J->S.n_phsp) p = phase_space_primary(J->S, J->G, h);
            else p = make_primary(J->S, J->G, h, source_draws(h, k0, k1), k0, k1, -1, sg->rpos + i, sg->rsize);
            account(p, h, live);
            born += copies * count(live && p.in);
            const uint32_t jb = tag | (sg->batch << 16);
            if (copies > 1u) {
                if (live) write(p, h, sg->off + i * copies, jb);
                continue;
            }
            // 64 records of 64 B are consecutive in the queue: lane L writes piece
            // L % 4 of record 16 k + L / 4.  In LDS the pieces of a record are
            // rotated by its number, so that neither side has a bank conflict.
            const Rec r = primary_record(p, h, 0u, voxel(p), jb);
            const uint32_t rot = (lane >> 2) & 3u;
            lds[4u * lane + (0u ^ rot)] = r.a;
            lds[4u * lane + (1u ^ rot)] = r.b;
            ((GDPM_LDS u4*)lds)[4u * lane + (2u ^ rot)] = r.c;
            ((GDPM_LDS u4*)lds)[4u * lane + (3u ^ rot)] = r.d;
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            const uint32_t slot0 = base + sg->off + i0;
#pragma unroll
            for (uint32_t k = 0; k < 4u; ++k) {
                const uint32_t rec = 16u * k + (lane >> 2), piece = lane & 3u;
                const f4 v = lds[4u * rec + (piece ^ ((rec >> 2) & 3u))];
                if (rec < n)
                    ((GDPM_GLOBAL f4*)(global_ptr(A->R.buf[ri]) + ((slot0 + rec) & A->R.mask[ri])))[piece] = v;
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            continue;
        }
        // Metropolis: 64 / g chains, g lanes each, through the job's segments in
        // order.  A chain's g next steps are resolved together: which of them move
        // depends on the state before each, the last move or the state the
        // chain came with, so the moves are found from the states that the moves
        // of the last turn imply, until they no longer change (after turn t the
        // first t steps are right; a few turns do).
        const uint32_t g = sg->lanes;
        const uint32_t sub = lane & (g - 1u), lead = lane - sub;
        const uint32_t chain = (c - sg->unit0) * (64u / g) + lead / g;
        GDPM_GLOBAL uint32_t* chains = global_ptr(J->chains);
        const GDPM_GLOBAL float* f = global_ptr(J->S.f);
        uint32_t state = chains[chain];
        float f_state = f[state];
        const uint64_t mine = (g == 64u ? ~0ull : ((1ull << g) - 1ull)) << lead;
        for (uint32_t q = 0; q < sg->group; ++q) {
            const GDPM_CONST SrcSeg* t = sg + q;
            const uint32_t first = (uint32_t)((chain + kMetroChains - t->h0 % kMetroChains) % kMetroChains);
            const uint32_t jb = tag | (t->batch << 16);
            for (uint32_t b = first; ballot(b < t->n); b += g * kMetroChains) {
                const uint32_t i = b + sub * kMetroChains;
                const bool live = b < t->n && i < t->n && i >= b;
                const unsigned long long h = t->h0 + (live ? i : 0u);
                const f4 d = source_draws(h, k0, k1);
                const uint32_t trial = metropolis_trial(J->S, d.y);
                const float f_j = f[trial];
                uint64_t moves = 0ull;
                uint32_t from = 64u;   // the lane whose trial the step starts from (64: the chain's state)
                for (uint32_t turn = 0; turn <= g; ++turn) {
                    const uint64_t before = moves & mine & ((1ull << lane) - 1ull);
                    from = before ? 63u - (uint32_t)__clzll(before) : 64u;
                    const float f_from = __shfl(f_j, (int)(from & 63u));
                    const uint64_t now =
                        ballot(live && metropolis_moves(d.z, from == 64u ? f_state : f_from, f_j));
                    const bool same = now == moves;
                    moves = now;
                    if (same) break;
                }
                // the beamlet of this step: its trial if it moved, else the state before it
                const uint32_t held = __shfl(trial, (int)(from & 63u));
                const uint32_t beamlet = (moves >> lane) & 1ull ? trial : (from == 64u ? state : held);
                // the chain's state after its last move here
                const uint64_t all = moves & mine;
                const uint32_t last = all ? 63u - (uint32_t)__clzll(all) : 0u;
                const uint32_t end_state = __shfl(trial, (int)last);
                const float end_f = __shfl(f_j, (int)last);
                state = all ? end_state : state;
                f_state = all ? end_f : f_state;
                const Primary p =
                    make_primary(J->S, J->G, h, d, k0, k1, (int)beamlet, t->rpos + i, t->rsize);
                account(p, h, live);
                born += copies * count(live && p.in);
                if (live) write(p, h, t->off + i * copies, jb);
            }
        }
        if (sub == 0u) chains[chain] = state;
    }
    flush();
    __syncthreads();
    GDPM_GLOBAL JobCtl* jc = global_ptr(A->R.jc);
    const int n_jobs = A->R.n_jobs;
    for (int j = (int)threadIdx.x; j < n_jobs; j += blockDim.x) {
        if (tally.e_in[j] != 0.0) atomic_add_f64(&jc->e_in[j], tally.e_in[j]);
        if (tally.e_esc[j] != 0.0) atomic_add_f64(&jc->e_esc[j], tally.e_esc[j]);
        if (tally.born[j]) atomic_add(&jc->births[j], (unsigned long long)tally.born[j]);
    }
}

// ---------------------------------------------------------------------------
// LDS of a transport workgroup
// ---------------------------------------------------------------------------
// Interpolation tables are staged in LDS (kLds) when they fit; one workgroup
// per CU shares them.
extern __shared__ f4 lds_tables[];

// Layout (float4 units): the workgroup's counters; the tables, if staged (photons:
// the total cross sections, then the majorant of the pass's job; electrons: range and
// mu_hard, 1/lambda_1, the inverse range and its scales, the screening); then per
// wavefront one slice: its lanes' generator words, then the photons' pool or the
// electrons' brick sums (if there is room)
constexpr uint32_t kRingF4 = kRngWords * 64u / 4u;   // generator words of a wavefront
template <class TT>
GDPM_HD uint32_t tables_f4(int ri, const TT& T) {
    const uint32_t floats = ri == 0 ? (uint32_t)((T.n_mat + 1) * T.pg_n)
                                    : (uint32_t)(T.n_mat * (3 * T.eg_n + T.nr) + T.n_mat + T.aw_n);
    return (floats + 3u) / 4u;
}
// an electron wavefront's brick sums, [voxel of the brick][lane] (FP64), and its list
// of lanes that leave their bricks
constexpr uint32_t kBrickF4 = kBrickVoxels * 64u / 2u + 64u * 2u / 16u;
// a photon wavefront's pool of photons, [piece][slot], 48 bytes each, the slots'
// columns, and generator words of as many columns more (see photon_pass)
constexpr uint32_t kPool = 64u, kPhotonCols = 64u + kPool;
constexpr uint32_t kPoolF4 = 3u * kPool + kPool / 4u;
// ri: 0 photons, 1 electrons, 2 both (k_transport), 3 both without the photons' pool: with
// one for each wavefront, 12 of them and the electron tables of 4 materials would take
// 175,248 of the CU's 163,840 bytes, and without 136,848.  The pool is kept where it fits:
// with 10 wavefronts, 3e7 photons took 16.7 and 13.9 ms (CTs of 0.2 and 0.4 cm) with it
// and 17.7 and 14.9 without.
GDPM_HD uint32_t slice_f4(int ri, bool bricks) {
    const uint32_t photons = kRngWords * kPhotonCols / 4u + kPoolF4, electrons = kRingF4 + (bricks ? kBrickF4 : 0u);
    return ri == 0 || (ri == 2 && photons > electrons) ? photons : electrons;
}

// the device clock at the start of a pass (its completion takes the difference)
GDPM_DEV void start_clock(Args A) {
    if (blockIdx.x == 0 && threadIdx.x == 0) global_ptr(A->ctl)->t_start = wall_clock64();
}

// a workgroup none of whose wavefronts has a record to start with: it ends
// before it stages the tables (nothing is left to claim either)
GDPM_DEV bool group_idle(Args A, int ri) {
    const GDPM_CONST RingCtl* rc = ring_const(A, ri);
    return rc->count == 0u || (rc->first && blockIdx.x * rc->first >= rc->count);
}

// ---------------------------------------------------------------------------
// photon pass: Woodcock tracking (section 2.1), one flight per iteration
// ---------------------------------------------------------------------------
// One wavefront's share of a photon pass.  ptab: the total cross sections (in
// LDS or global memory); lmaj: the job's majorant in LDS (kMajLds: a pass of one job; else it
// is read from global memory); ring: the wavefront's generator words and its pool (kPark; without it a
// lane waits in passes of any length).
//
// Without the pool, vector instructions were issued in two thirds of the cycles, half of
// them to sample interactions, which come in one of four flights: sampled as soon as 22
// lanes had one, they ran on 26 of 64 lanes and the flights on 50, since the lanes of those
// waited.
// In a pass with several photons per lane they are parked instead, in a pool of 64
// photons in LDS, and the lane goes on with another photon, until there is one for each
// lane; then the wavefront exchanges the photons in its lanes for parked ones, samples
// them and flies on, and the exchanged ones are the first that empty lanes take.
// Interactions run on 60 lanes and flights too: 8.10 instead of 8.49 ms for 5e7
// photons on a CT of 0.4 cm voxels, 9.25 instead of 9.54 on 0.2 cm, 4.09 instead of 4.21 for
// 2e7 on slabs.  A photon keeps its buffered draws when it changes places (the column
// of the generator words goes with it): generated again, they took what the fuller
// lanes gave.  In a pass with few photons a lane waits: they end before the pool fills,
// and the exchange cost 8% of it (1e5 photons).
// What bounds the pass now are the latencies of the voxel reads and, on fine grids, the
// lines that they fetch (6.5 TB/s on the CT of 0.2 cm): vector instructions are issued in
// 43% of the cycles there, 52% on 0.4 cm, 42% on slabs, on 70 to 74% of the lanes.
template <bool kSolo, bool kPerm, bool kMajLds, bool kPark, class PT>
GDPM_DEV void photon_pass(Args A0, const PT ptab, const GDPM_LDS float* lmaj, GDPM_LDS float* ring, GroupPtr group) {
    const GDPM_CONST RingCtl* rc = ring_const(A0, 0);
    const uint32_t begin = rc->begin, total = rc->count;
    // a re-binned pass reads its input through the permutation (only the kPerm
    // form has that code: the passes of a lone job keep the plain reads)
    const GDPM_GLOBAL uint32_t* perm_in =
        kPerm && rc->permuted ? global_ptr(bin_perm(A0->R.bin[0], A0->R.mask[0])) : nullptr;
    const uint32_t waves = pass_waves(A0, 0);
    const bool big = !kSolo && total >= kTailMinPerLane * 64u * waves;
    const bool park = kPark && big;

    constexpr uint32_t kCols = kPark ? kPhotonCols : 64u;
    GDPM_LDS f4* const pool = (GDPM_LDS f4*)(ring + kRngWords * kCols);
    GDPM_LDS uint32_t* const cols = (GDPM_LDS uint32_t*)(pool + 3u * kPool);
    int j = first_job(A0, total, 0);
    uint32_t first = rc->first;
    PushState pg{0u, 0u, rc->push}, pe{0u, 0u, rc->push};
    double e_esc = 0.0;   // escaped energy of the current job
    WaveTally wt{};
    uint32_t iters = 0u;
    bool last_job = !kPerm;   // no other job has records left in this pass
    const float pg_lo = pin(A0->T.pg_lo), pg_inv = pin(A0->T.pg_inv);
    const int pg_n = pin(A0->T.pg_n);
    // one job at a time: a wavefront switches jobs with all its lanes empty
    while (j >= 0) {
        WJob W;
        load_job(W, A0, j, 0);
        // what a flight needs of the job, in scalar registers: read again in each
        // iteration, every use waited for a scalar load of its own
        const float idx = pin(W.p->G.idx), idy = pin(W.p->G.idy), idz = pin(W.p->G.idz);
        const uint32_t lx = pin(__float_as_uint(W.p->G.lx)), ly = pin(__float_as_uint(W.p->G.ly)),
                       lz = pin(__float_as_uint(W.p->G.lz));
        const int nx = pin(W.p->G.nx), ny = pin(W.p->G.ny), nz = pin(W.p->G.nz);
        const GDPM_GLOBAL uint32_t* vox = pin(global_ptr(W.p->G.vox));
        const uint32_t k0 = pin(W.p->k0), k1 = pin(W.p->k1);
        const GDPM_GLOBAL float* gmaj = pin(global_ptr(W.p->mumax));
        const bool hist = W.p->hist != nullptr;
        ClaimState cs = claim_start(W, first, waves);
        first = 0u;
        bool active = false;
        float x = 0, y = 0, z = 0, u = 0, v = 0, w = 0, e = 0;
        uint32_t pb = 0u;   // batch slot of the lane's history
        int pm = -1;        // >= 0: a real interaction waits, in a voxel of this material
        Rng<kCols> rng;
        rng.buf = ring + lane_id();
        if (kPark) cols[lane_id()] = kPool + lane_id();
        rng_start(rng, 0u, 0u, 0u, 0u);
        int next = -1;
        // the pool: photons with an interaction in slots [0, parked), then `ready` ones
        // without
        uint32_t parked = 0u, ready = 0u;
        for (;;) {
            const Args A = reread(A0);
            const JobPtr J = reread(W.p);
            Rec p;
            if (ready == 0u && refill<kSolo, kPerm>(active, cs, A, W, 0, begin, perm_in, p, wt)) {
                // + 0: a position of -0 becomes +0 (see inside)
                x = p.a.x + 0.0f; y = p.a.y + 0.0f; z = p.a.z + 0.0f; e = p.a.w;
                u = p.b.x; v = p.b.y; w = p.b.z;
                pb = p.d.w >> 16;
                rng_start(rng, p.c.x, p.c.y, p.c.z, p.c.w);
                active = true;
                // an energy that ends the photon where it is: below the
                // absorption energy, or non-finite (only from a damaged record)
                pm = e < A->R.ecut_g || !(e <= kMaxEnergy) ? kAbsorb : -1;
            }
            if (!ballot(active) && parked + ready == 0u) {
                if (cs.done && last_job) break;
                if (!cs.done) continue;
            } else {
                const bool fly = active && pm < 0;
                rng_topup(rng, fly, active, 2u, k0, k1);
                wt.events += count(fly);
                const float ul = rng.peek(0u), ua = rng.peek(1u);
                int gi;
                float gt;
                grid(hlog2(e), pg_lo, pg_inv, pg_n, gi, gt);
                float mumax;
                if constexpr (kMajLds) mumax = lerp1(lmaj, gi, gt);
                else mumax = lerp1(gmaj, gi, gt);
                // The flight is computed on every lane, without branches: a lane
                // that waits or is empty flies a distance of 0, which leaves it
                // where it is, and only the loads and the tallies are masked.
                const float s = fly ? neg_ln(ul) * hrcp(mumax) : 0.0f;
                rng.ctr += fly ? 2u : 0u;
                x = fmaf(s, u, x);
                y = fmaf(s, v, y);
                z = fmaf(s, w, z);
                const bool in = fly && inside(lx, ly, lz, x, y, z);
                int ix, iy, iz;
                const int vv = voxel_of(idx, idy, idz, nx, ny, nz, x, y, z, ix, iy, iz);
                uint32_t vx = 0u;
                if (in) vx = vox[vv];
                if (fly && !in) {
                    e_esc += (double)e;
                    if (hist) history_escape(J, (double)e, rng);
                    active = false;
                }
                wt.died += count(fly && !in);
                {
                    const int m = voxel_material(vx);
                    const float mu = ptab.total(m * pg_n + gi, gt);
                    const bool real = in && ua * mumax < voxel_density(vx) * mu;
                    pm = real ? m : pm;   // the interaction waits (see below)
                    wt.real[0] += count(real);
                }
                const uint64_t br = ballot(active && pm >= 0), bf = ballot(active && pm < 0), be = ballot(!active);
                const uint32_t nr = (uint32_t)__popcll(br), nf = (uint32_t)__popcll(bf), ne = (uint32_t)__popcll(be);
                const bool sample =
                    parked + nr > 0u && (cs.done || nf == 0u || (park ? parked + nr > kPool : nr >= kRealBatch));
                // Exchange photons with the pool: a lane gives its own to the slot,
                // gets the slot's, or both.  A lane waits where it is without drawing,
                // and in the pool, so each particle's draws keep their order; the cross
                // sections are recomputed from the same inputs.
                bool give = false, get = false;
                uint32_t slot = 0u;
                if (!park) {
                    // (photons wait for their interactions in their lanes)
                } else if (sample) {
                    // the lanes without an interaction get parked photons, and their
                    // own become ready; empty lanes get the last ready ones, or
                    // without any the last parked ones
                    const uint32_t kr = min(ready, ne), ke = ready ? 0u : min(parked, ne);
                    const uint32_t ks = min(parked - ke, nf);
                    const uint32_t r = active ? mbcnt(bf) : mbcnt(be);
                    give = active && pm < 0 && r < ks;
                    get = active ? give : r < kr + ke;
                    slot = active ? parked - ke - ks + r : parked + ready - 1u - r;
                    parked -= ke + ks;
                    ready += ks - kr;
                } else {
                    // lanes with an interaction park their photon, in the place of a
                    // ready one if there is one; empty lanes get the last ready ones
                    const uint32_t ks = min(ready, nr), ke = min(ready - ks, ne);
                    const uint32_t r = active ? mbcnt(br) : mbcnt(be);
                    give = active && pm >= 0;
                    get = active ? give && r < ks : r < ke;
                    slot = active ? parked + r : parked + ready - 1u - r;
                    parked += nr;
                    ready -= ks + ke;
                }
                if (park) {
                    wave_fence();
                    if (give || get) {
                        const f4 a = pool[slot], b = pool[kPool + slot];
                        const u4 c = ((const GDPM_LDS u4*)pool)[2u * kPool + slot];
                        const uint32_t col = cols[slot];
                        if (give) {
                            const uint32_t blocks = rng.nb - (rng.ctr >> 2);   // buffered, 0..2
                            pool[slot] = f4{x, y, z, e};
                            pool[kPool + slot] = f4{u, v, w, __uint_as_float(pb << 16 | blocks << 14 | (uint32_t)(pm + 1))};
                            ((GDPM_LDS u4*)pool)[2u * kPool + slot] = u4{rng.hlo, rng.hhi, rng.path, rng.ctr};
                        }
                        cols[slot] = (uint32_t)(rng.buf - ring);   // a photon keeps the column of its draws
                        rng.buf = ring + col;
                        if (get) {
                            const uint32_t bits = __float_as_uint(b.w);
                            x = a.x; y = a.y; z = a.z; e = a.w;
                            u = b.x; v = b.y; w = b.z;
                            pb = bits >> 16;
                            pm = (int)(bits & 0x3FFFu) - 1;
                            rng.hlo = c.x; rng.hhi = c.y; rng.path = c.z; rng.ctr = c.w;
                            rng.nb = (c.w >> 2) + (bits >> 14 & 3u);
                        } else {
                            pm = -1;
                        }
                        active = get;
                    }
                }
                if (sample) {
                    const uint64_t act0 = ballot(active);
                    if (ballot(get)) {   // other photons
                        voxel_of(idx, idy, idz, nx, ny, nz, x, y, z, ix, iy, iz);
                        grid(hlog2(e), pg_lo, pg_inv, pg_n, gi, gt);
                    }
                    const bool kerma = (J->flags & 64u) != 0u;
                    const float ecut_e = A->R.ecut_e;
                    PendCharged qe;
                    PendPhoton qg;
                    qe.n = 0;
                    qg.n = 0;
                    int itype = -1;    // the interaction sampled by this lane
                    double dep = 0.0;  // its deposit, in the lane's voxel
                    rng_topup(rng, pm >= 0, active, 4u, k0, k1);
                    if (pm == kAbsorb) {
                        if (e <= kMaxEnergy) dep = (double)e;
                        else atomic_add(&global_ptr(A->ctl)->anomalies, 1ull);
                        active = false;
                        pm = -1;
                    }
                    if (pm >= 0) {
                        const f4 mu = lerp4(global_f4(A->T.phot) + pm * pg_n, gi, gt);
                        const float r = uniform(rng, k0, k1) * mu.w;
                        itype = r < mu.x ? 0 : (r < mu.x + mu.y ? 1 : 2);
                        if (itype == 0) {
                            float eps, t, turns;
                            sample_compton(A->T, rng, k0, k1, e, eps, t, turns);
                            const float u0 = u, v0 = v, w0 = w;
                            rotate(u, v, w, 1.0f - t, hsqrt(fmaxf(0.0f, t * (2.0f - t))), turns);
                            // exact split of E into E' and T (the unit is built without
                            // contraction, so the product is rounded on its own)
                            const float ec = eps * e;
                            float e1, te;
                            if (2.0f * ec >= e) {
                                e1 = ec;
                                te = e - ec;
                            } else {
                                te = e - ec;
                                e1 = e - te;
                            }
                            if (kerma || te <= ecut_e) {
                                dep = (double)te;
                            } else {
                                float eu, ev, ew;
                                compton_electron_dir(e, e1, u0, v0, w0, u, v, w, eu, ev, ew);
                                qe.n = 1; qe.e0 = te; qe.du = eu; qe.dv = ev; qe.dw = ew;
                                qe.a0 = 0.0f; qe.role = 0u;
                            }
                            e = e1;
                            if (e < A->R.ecut_g) {   // absorbed where it is
                                dep += (double)e;
                                active = false;
                            }
                        } else if (itype == 1) {
                            // photoelectric: the electron takes E along the photon
                            if (kerma || e <= ecut_e) {
                                dep = (double)e;
                            } else {
                                qe.n = 1; qe.e0 = e; qe.du = u; qe.dv = v; qe.dw = w;
                                qe.a0 = 0.0f; qe.role = 0u;
                            }
                            active = false;
                        } else {
                            // pair: uniform split of E - 2 mc^2; the positron keeps a = E - K
                            float tm, tp, aa;
                            pair_split(e, uniform(rng, k0, k1), tm, tp, aa);
                            const bool e_local = kerma || tm <= ecut_e;
                            const bool p_local = kerma || tp <= ecut_e;
                            if (p_local) {
                                float du, dv, dw;
                                sample_iso(rng, k0, k1, du, dv, dw);
                                dep = (double)tp;
                                qg.n = 2; qg.e = 0.5f * aa; qg.u = du; qg.v = dv; qg.w = dw; qg.wb = 2u;
                            }
                            if (e_local) dep += (double)tm;
                            qe.du = u; qe.dv = v; qe.dw = w;
                            if (!e_local) {
                                qe.n = 1; qe.e0 = tm; qe.a0 = 0.0f; qe.role = 0u;
                                if (!p_local) {
                                    qe.n = 2; qe.e1 = tp; qe.a1 = aa;
                                }
                            } else if (!p_local) {
                                qe.n = 1; qe.e0 = tp; qe.a0 = aa; qe.role = 1u;
                            }
                            active = false;
                        }
                        pm = -1;
                    }
                    if (dep != 0.0) add_dose(J, pb, tally_order(*J, J->G.nx, J->G.ny).pos(ix, iy, iz), dep, rng);
                    wt.dep += count(dep != 0.0);
                    wt.it[0] += count(itype == 1);
                    wt.it[1] += count(itype == 2);
                    // secondaries: electrons/positrons to queue 1, annihilation photons to queue 0
                    const uint32_t jb = W.tag | (pb << 16);
                    push_charged(qe, pe, A, J, jb, x, y, z, pack_vox(ix, iy, iz), rng, wt);
                    push_photons(qg, pg, A, J, jb, x, y, z, rng, wt);
                    wt.died += (uint32_t)__popcll(act0 & ~ballot(active));
                }
            }
            if (++iters > kMaxWaveIterations) {
                // safety net, never reached in a sound run: end the particles
                // still held (counted as anomalies) so the grid always drains
                const uint32_t n = count(active) + parked + ready;
                wt.died += n;
                wt.bad += n;
                active = false;
                break;
            }
            if (cs.done) {
                // this job has nothing left to claim in the pass: move to a job
                // that has records left, or at the tail of a large pass stop
                // early; the particles still held go to the next pass
                int nj = -1;
                if (!last_job) {
                    nj = next_job(global_ptr(A->R.jc), W.j, A->R.n_jobs, 0);
                    last_job = nj < 0;
                }
                // (the interactions of the parked ones come first)
                if (parked == 0u && (nj >= 0 || (big && count(active) + ready < kTailLanes))) {
                    Rec q;
                    q.a = f4{x, y, z, e};
                    q.b = f4{u, v, w, -1.0f};
                    q.c = u4{rng.hlo, rng.hhi, rng.path, rng_ctr(rng)};
                    q.d = u4{0u, 0u, 0u, W.tag | (pb << 16)};
                    requeue(active, pg, A, 0, q, wt);
                    if (ready) {   // their turn is the next iteration
                        active = false;
                        continue;
                    }
                    next = nj;
                    break;
                }
            }
        }
        job_flush(e_esc, wt, W.j, group);
        j = next;
    }
    release(pe, A0, 1);
    release(pg, A0, 0);
    pass_finish(wt, 0, group);
}

// The kernel's arguments are read through pass_args(); the parameter only
// declares their layout.
template <bool kLds, bool kSolo, bool kPerm>
__global__ void __launch_bounds__(1024) k_photon(PassArgs) {
    const Args A = pass_args();
    start_clock(A);
    if (!kPerm && group_idle(A, 0)) return;
    const GroupPtr group = (GroupPtr)lds_tables;
    GDPM_LDS f4* lds = (GDPM_LDS f4*)lds_tables + kGroupTallyF4;
    group_clear(group);
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if constexpr (kLds) {
        const GDPM_CONST Tables& T = A->T;
        const int np = T.n_mat * T.pg_n;
        GDPM_LDS float* tot = (GDPM_LDS float*)lds;
        for (int i = threadIdx.x; i < np; i += blockDim.x) tot[i] = global_f4(T.phot)[i].w;
        GDPM_LDS float* lmaj = tot + np;
        if constexpr (!kPerm) {
            // a pass of one job: its majorant too
            const int j = first_job(A, ring_const(A, 0)->count, 0);
            if (j >= 0) {
                const GDPM_GLOBAL float* mj = global_ptr(((JobPtr)A->R.jobs)[j].mumax);
                for (int i = threadIdx.x; i < T.pg_n; i += blockDim.x) lmaj[i] = mj[i];
            }
        }
        __syncthreads();
        if (wave < ring_const(A, 0)->group_waves)
            photon_pass<kSolo, kPerm, !kPerm, true>(
                A, PhotLds{tot}, lmaj, (GDPM_LDS float*)(lds + tables_f4(0, T) + wave * slice_f4(0, false)), group);
    } else {
        __syncthreads();
        if (wave < ring_const(A, 0)->group_waves)
            photon_pass<kSolo, kPerm, false, true>(A, PhotGlobal{global_f4(A->T.phot)}, nullptr,
                                             (GDPM_LDS float*)(lds + wave * slice_f4(0, false)), group);
    }
    group_flush(A, group);
}

// ---------------------------------------------------------------------------
// electron pass: class-II condensed history with a random hinge, one step per
// iteration (section 2.1)
// ---------------------------------------------------------------------------
// One wavefront's share of an electron pass.  E: the stopping and scattering
// data and the inverse range (in LDS or global memory); ring: the wavefront's
// generator words, and behind them its brick sums (if A0->bricks).
//
// A deposit added to the tally as the particle left its voxel made the pass wait
// for the additions: 307 M of them took 13.1 of 15.9 ms on a CT of 0.2 cm voxels,
// where the rest of the pass takes 10.8.  Now a particle's deposits are summed per
// voxel in LDS while it stays in a brick of the tally (see Brick), and when it
// leaves, as many lanes as the brick has voxels add the sums in one instruction, one
// line of memory.  A particle that leaves with one deposit adds it itself.  Bricks of
// 2x2x2 voxels leave room for 14 wavefronts and not for the screening table (a
// lookup of it in global memory waits for the additions before it), those of 4 voxels
// for 16 with it: what took 15.9, 10.2, 4.6 and 18.4 ms (5e7 photons on CTs of 0.2 and
// 0.4 cm, 2e7 photons and 5e6 electrons on 0.3 cm slabs) took 13.1, 9.9, 4.4 and 12.5
// with the former and takes 12.5, 8.9, 4.0 and 13.8 with the latter.  What bounds it now is
// vector instructions (78, 83, 95 and 69% of the cycles in the four) with half of their
// lanes at work, and the latencies between them.
template <bool kSolo, bool kPerm, class EL>
GDPM_DEV void electron_pass(Args A0, const EL E, GDPM_LDS float* ring, GroupPtr group) {
    GDPM_LDS double* const sums = (GDPM_LDS double*)(ring + 4u * kRingF4);
    GDPM_LDS uint16_t* const leavers = (GDPM_LDS uint16_t*)(sums + kBrickVoxels * 64u);
    if (A0->bricks)
        for (int i = 0; i < kBrickVoxels; ++i) sums[64u * i + lane_id()] = 0.0;
    const GDPM_CONST RingCtl* rc = ring_const(A0, 1);
    const uint32_t begin = rc->begin, total = rc->count;
    const GDPM_GLOBAL uint32_t* perm_in =
        kPerm && rc->permuted ? global_ptr(bin_perm(A0->R.bin[1], A0->R.mask[1])) : nullptr;
    const uint32_t waves = pass_waves(A0, 1);
    const bool big = !kSolo && total >= kTailMinPerLane * 64u * waves;

    int j = first_job(A0, total, 1);
    uint32_t first = rc->first;
    PushState pg{0u, 0u, rc->push}, pe{0u, 0u, rc->push};
    double e_esc = 0.0;   // escaped energy of the current job
    WaveTally wt{};
    uint32_t iters = 0u;
    bool last_job = !kPerm;   // no other job has records left in this pass
    const ElecGrid eg(A0->T);
    const int n_mat = pin(A0->T.n_mat);
    const float ecut = pin(A0->R.ecut_e);
    // one job at a time: a wavefront switches jobs with all its lanes empty
    while (j >= 0) {
        WJob W;
        load_job(W, A0, j, 1);
        // what a step needs of the job, in scalar registers (see the photon pass)
        const Spacing G{pin(W.p->G.dx), pin(W.p->G.dy), pin(W.p->G.dz)};
        const int nx = pin(W.p->G.nx), ny = pin(W.p->G.ny), nz = pin(W.p->G.nz);
        const GDPM_GLOBAL uint32_t* vox = pin(global_ptr(W.p->G.vox));
        const uint32_t k0 = pin(W.p->k0), k1 = pin(W.p->k1);
        const bool no_ms = (W.p->flags & 8u) != 0u;
        const TallyOrder O = tally_order(*W.p, nx, ny);
        GDPM_GLOBAL double* const tally = pin(global_ptr(W.p->tally));
        const uint32_t nv = pin((uint32_t)W.p->nv);   // (positions fit 31 bits)
        const bool hist = W.p->hist != nullptr;
        const bool sum_bricks = A0->bricks && O.s > 0;
        ClaimState cs = claim_start(W, first, waves);
        first = 0u;
        bool active = false;
        float x = 0, y = 0, z = 0, u = 0, v = 0, w = 0, e = 0, nh = -1.0f;
        float aa = 0.0f;    // > 0: a positron, and its annihilation energy
        int ix = 0, iy = 0, iz = 0;
        uint32_t vx = 0u;   // the current voxel, reloaded when the particle enters one
        double de = 0.0;    // deposit in it, not yet tallied
        float hq = -1.0f;   // >= 0: a hard event waits; the step-start mu_h per g/cm^2
        uint32_t pb = 0u;   // batch slot of the lane's history
        Rng<64u> rng;
        rng.buf = ring + lane_id();
        rng_start(rng, 0u, 0u, 0u, 0u);
        int next = -1;
        bool summed = false;    // the lane's brick has sums in LDS
        // Add the sums of the lanes of `leave` (their brick: b) to the tally, one lane
        // per voxel, and clear them; the wavefront is converged.
        auto flush_bricks = [&](bool leave, uint32_t b) {
            const uint64_t m = ballot(leave);
            const uint32_t n = (uint32_t)__popcll(m);
            if (leave) leavers[mbcnt(m)] = (uint16_t)(lane_id() | pb << 6);
            wave_fence();
            for (uint32_t k = 0; k < n; k += 64 / kBrickVoxels) {
                const uint32_t g = k + lane_id() / kBrickVoxels, v = lane_id() % kBrickVoxels;
                const uint32_t l = leavers[min(g, n - 1u)];
                const uint32_t lb = (uint32_t)__builtin_amdgcn_ds_bpermute((int)(l << 2), (int)b);
                GDPM_LDS double* q = sums + 64u * v + (l & 63u);
                const double d = *q;
                if (g < n && d != 0.0) {
                    *q = 0.0;
                    atomic_add_f64(tally + ((unsigned long long)(l >> 6) * nv + (lb << O.s | v)), d);
                }
            }
            wave_fence();
        };
        for (;;) {
            const Args A = reread(A0);
            const JobPtr J = reread(W.p);
            Rec p;
            if (refill<kSolo, kPerm>(active, cs, A, W, 1, begin, perm_in, p, wt)) {
                x = p.a.x; y = p.a.y; z = p.a.z; e = p.a.w;
                u = p.b.x; v = p.b.y; w = p.b.z; nh = p.b.w;
                ix = (int)(p.d.x & 2047u);
                iy = (int)((p.d.x >> 11) & 2047u);
                iz = (int)(p.d.x >> 22);
                aa = (p.d.z & 1u) ? __uint_as_float(p.d.y) : 0.0f;
                pb = p.d.w >> 16;
                rng_start(rng, p.c.x, p.c.y, p.c.z, p.c.w);
                vx = vox[ix + nx * (iy + ny * iz)];
                active = true;
            }
            if (!ballot(active)) {
                if (cs.done && last_job) break;
                if (!cs.done) continue;
            } else {
                const uint64_t act0 = ballot(active);
                if (active && !(e <= kMaxEnergy)) {
                    // a non-finite energy can only come from a damaged record: end the
                    // particle (counted as an anomaly) rather than feed it to a
                    // rejection sampler that would never accept
                    atomic_add(&global_ptr(A->ctl)->anomalies, 1ull);
                    active = false;
                    hq = -1.0f;
                }
                const bool step = active && hq < 0.0f && e > ecut;
                wt.events += count(step);
                // a step draws at most 4 numbers, the first for a fresh hard-event distance
                rng_topup(rng, step, active, 4u, k0, k1);
                const uint32_t brick = O.brick(ix, iy, iz), vin = O.voxel(ix, iy, iz);   // voxel of the step
                bool crossed = false;
                bool left = false;   // the brick
                if (step) {
                    const float rho = voxel_density(vx);
                    const int m = voxel_material(vx);
                    const float irho = hrcp(rho);
                    if (nh < 0.0f) nh = neg_ln(rng.draw());
                    const float xi = rng.draw();
                    const float t0 = e;
                    int ci;
                    float ct;
                    eg.cell(m, t0, ci, ct);
                    const f2 q0 = E.range_hard(ci, ct);
                    const float rsc = rinv_scale(E, eg, n_mat, m);
                    const float mus = rho * q0.y;
                    const float sh = mus > 0.0f ? nh * hrcp(mus) : 3.0e38f;
                    const float tfl = fmaxf(0.75f * t0, ecut);
                    eg.cell(m, tfl, ci, ct);
                    const float rtf = E.range(ci, ct);
                    const float rfl = tfl > ecut ? rtf : 0.0f;
                    const float se = (q0.x - rfl) * irho;
                    const bool hard = sh < se;
                    const float s = hard ? sh : se;
                    const float s1 = xi * s, s2 = s - s1;
                    float tend = tfl;
                    if (hard) tend = fminf(fmaxf(range_inv(E.rinv, rsc, eg.nr, m, q0.x - rho * s), tfl), t0);
                    // first half: to the hinge, or to the voxel face if that comes
                    // first.  Lanes that cross and lanes that reach the hinge share
                    // one move, one range lookup and one deposit.
                    int ax;
                    float db = face_dist(G, x, y, z, u, v, w, ix, iy, iz, ax);
                    crossed = db < s1;
                    float travelled = db;
                    {
                        const float d1 = crossed ? db : s1;
                        x = fmaf(d1, u, x); y = fmaf(d1, v, y); z = fmaf(d1, w, z);
                        const float t1 =
                            fminf(fmaxf(range_inv(E.rinv, rsc, eg.nr, m, q0.x - rho * d1), tend), e);
                        de += (double)(e - t1);
                        e = t1;
                    }
                    if (!crossed) {
                        // hinge: modified-Wentzel deflection for the whole step
                        if (!no_ms) {
                            const float tmid = 0.5f * (t0 + tend);
                            eg.cell(m, tmid, ci, ct);
                            const float tt = s * rho * E.inv_lambda(ci, ct);
                            const float mu = mw_mu(eg, E.aw, tt, rng.draw());
                            const float turns = rng.draw();
                            rotate(u, v, w, 1.0f - 2.0f * mu, 2.0f * hsqrt(mu * (1.0f - mu)), turns);
                        }
                        // second half: to the step end or the face; a lane that
                        // reaches the end loses exactly the energy left above tend
                        db = face_dist(G, x, y, z, u, v, w, ix, iy, iz, ax);
                        crossed = db < s2;
                        travelled = s1 + db;
                        const float d2 = crossed ? db : s2;
                        x = fmaf(d2, u, x); y = fmaf(d2, v, y); z = fmaf(d2, w, z);
                        float t2 = tend;
                        if (crossed)
                            t2 = fminf(fmaxf(range_inv(E.rinv, rsc, eg.nr, m, q0.x - rho * travelled), tend), e);
                        de += (double)(e - t2);
                        e = t2;
                    }
                    if (crossed) {
                        nh -= mus * travelled;
                        // move onto the face and into the next voxel
                        const bool a0 = ax == 0, a1 = ax == 1;
                        const float da = a0 ? u : (a1 ? v : w);
                        const int ia = a0 ? ix : (a1 ? iy : iz);
                        const int na = a0 ? nx : (a1 ? ny : nz);
                        const float ha = a0 ? G.dx : (a1 ? G.dy : G.dz);
                        const int in = da > 0.0f ? ia + 1 : ia - 1;
                        const float pa = (float)(da > 0.0f ? in : ia) * ha;
                        left = ((in ^ ia) & ~(a0 ? O.mx : (a1 ? O.my : O.mz))) != 0;
                        x = a0 ? pa : x;
                        y = a1 ? pa : y;
                        z = a0 || a1 ? z : pa;
                        ix = a0 ? in : ix;
                        iy = a1 ? in : iy;
                        iz = a0 || a1 ? iz : in;
                        if ((unsigned)in >= (unsigned)na) {
                            // a positron takes its annihilation energy along (summed in FP64)
                            const double out = (double)e + (double)aa;
                            e_esc += out;
                            history_escape(J, out, rng);
                            active = false;
                        } else {
                            // the next voxel's density and material, needed by the next step
                            vx = vox[ix + nx * (iy + ny * iz)];
                        }
                    } else if (hard) {
                        hq = q0.y;   // the hard event waits (see below)
                    } else {
                        nh -= mus * s;
                    }
                }
                // Hard events are rare (a few per hundred steps): run as they come,
                // their sampling would occupy the whole wavefront for one or two
                // lanes in most iterations.  A lane with one waits, where it is and
                // without drawing, until kHardBatch lanes wait, the wavefront has no
                // other live lane, or the pass has nothing left to claim; then they
                // are sampled together.  Each particle's draws keep their order.
                PendCharged qe;
                PendPhoton qg;
                qe.n = 0;
                qg.n = 0;
                const uint64_t bh = ballot(hq >= 0.0f);
                if (bh && (cs.done || (uint32_t)__popcll(bh) >= kHardBatch || bh == ballot(active))) {
                    int htype = -1;   // the hard event sampled by this lane
                    wt.real[0] += (uint32_t)__popcll(bh);
                    rng_topup(rng, hq >= 0.0f, active, 4u, k0, k1);
                    if (hq >= 0.0f) {
                        // delta scattering against the step-start majorant
                        // (mu_h grows with T; the step ended at e)
                        int ci;
                        float ct;
                        eg.cell(voxel_material(vx), e, ci, ct);
                        const f4 q1 = lerp4(global_f4(A->T.elec), ci, ct);
                        if (uniform(rng, k0, k1) * hq < q1.y) {
                            htype = uniform(rng, k0, k1) * q1.y < q1.z ? 0 : 1;
                            if (htype == 0) {
                                float eps, turns;
                                const float tt = e;
                                sample_moller(rng, k0, k1, tt, ecut, eps, turns);
                                const float tp = tt - eps * tt;   // >= T/2
                                const float wd = tt - tp;         // exact
                                const float tm2 = tt + kTwoMec2f;
                                const float itt = hrcp(tt);
                                const float cd = hsqrt(wd * tm2 * itt * hrcp(wd + kTwoMec2f));
                                const float cpr = hsqrt(tp * tm2 * itt * hrcp(tp + kTwoMec2f));
                                float du = u, dv = v, dw = w;
                                rotate(du, dv, dw, cd, hsqrt(fmaxf(0.0f, 1.0f - cd * cd)), turns);
                                rotate(u, v, w, cpr, hsqrt(fmaxf(0.0f, 1.0f - cpr * cpr)), turns + 0.5f);
                                if (wd <= ecut) {
                                    de += (double)wd;
                                } else {
                                    qe.n = 1; qe.e0 = wd; qe.du = du; qe.dv = dv; qe.dw = dw;
                                    qe.a0 = 0.0f; qe.role = 0u;
                                }
                                e = tp;
                            } else {
                                const float tt = e;
                                const float kph = sample_brems(rng, k0, k1, tt, A->R.ecut_g);
                                float kp, el;
                                if (2.0f * kph >= tt) {
                                    kp = kph;
                                    el = tt - kph;
                                } else {
                                    el = tt - kph;
                                    kp = tt - el;
                                }
                                qg.n = 1; qg.e = kp; qg.u = u; qg.v = v; qg.w = w; qg.wb = 0u;
                                e = el;
                            }
                        }
                        nh = -1.0f;
                        hq = -1.0f;
                    }
                    wt.real[1] += count(htype >= 0);
                    wt.it[0] += count(htype == 0);
                }
                // Absorption, in the iteration that brings the particle below its
                // absorption energy (a particle that has just entered a voxel, or a
                // positron with a secondary to push, is absorbed in the next one); a
                // positron annihilates at rest into two photons.
                const bool absorb =
                    active && hq < 0.0f && e <= ecut && !crossed && !(aa > 0.0f && qe.n + qg.n > 0);
                if (absorb) {
                    de += (double)e;
                    if (aa > 0.0f) {
                        float du, dv, dw;
                        rng.ensure(2u, k0, k1);
                        sample_iso(rng, k0, k1, du, dv, dw);
                        qg.n = 2; qg.e = 0.5f * aa; qg.u = du; qg.v = dv; qg.w = dw; qg.wb = 0u;
                    }
                    active = false;
                }
                // the deposit of a voxel goes to the tally when the particle leaves
                // the voxel or ends
                const bool flush = (crossed || absorb) && de != 0.0;
                const bool leave = left || !active;
                if (flush) {
                    if (!sum_bricks || (leave && !summed)) {
                        atomic_add_f64(tally + ((unsigned long long)pb * nv + (brick << O.s | vin)), de);
                    } else {
                        lds_add(sums + 64u * vin + lane_id(), de);
                        summed = true;
                    }
                    if (hist) add_history(J, de, rng);
                    de = 0.0;
                }
                if (ballot(leave && summed)) {
                    wave_fence();
                    flush_bricks(leave && summed, brick);
                    summed = summed && !leave;
                }
                wt.dep += count(flush);
                wt.died += (uint32_t)__popcll(act0 & ~ballot(active));
                const uint32_t jb = W.tag | (pb << 16);
                push_charged(qe, pe, A, J, jb, x, y, z, pack_vox(ix, iy, iz), rng, wt);
                push_photons(qg, pg, A, J, jb, x, y, z, rng, wt);
            }
            if (++iters > kMaxWaveIterations) {
                // safety net, never reached in a sound run: end the particles
                // still held (counted as anomalies) so the grid always drains
                const uint32_t n = count(active);
                wt.died += n;
                wt.bad += n;
                active = false;
                break;
            }
            if (cs.done) {
                // this job has nothing left to claim in the pass: move to a job
                // that has records left, or at the tail of a large pass stop
                // early; the particles still held go to the next pass
                int nj = -1;
                if (!last_job) {
                    nj = next_job(global_ptr(A->R.jc), W.j, A->R.n_jobs, 1);
                    last_job = nj < 0;
                }
                if (nj >= 0 || (big && count(active) < kTailLanes)) {
                    Rec q;
                    q.a = f4{x, y, z, e};
                    q.b = f4{u, v, w, nh};
                    q.c = u4{rng.hlo, rng.hhi, rng.path, rng_ctr(rng)};
                    q.d = u4{pack_vox(ix, iy, iz), __float_as_uint(aa), aa > 0.0f ? 1u : 0u, W.tag | (pb << 16)};
                    requeue(active, pe, A, 1, q, wt);
                    next = nj;
                    break;
                }
            }
        }
        // deposits of the particles handed on (or ended by the bound), in their voxels
        if (de != 0.0) add_dose(W.p, pb, O.pos(ix, iy, iz), de, rng);
        wt.dep += count(de != 0.0);
        if (ballot(summed)) flush_bricks(summed, O.brick(ix, iy, iz));
        job_flush(e_esc, wt, W.j, group);
        j = next;
    }
    release(pe, A0, 1);
    release(pg, A0, 0);
    pass_finish(wt, 1, group);
}

// stage the electron tables; every thread of the workgroup takes part
GDPM_DEV ElecLds stage_electron_tables(const GDPM_CONST Tables& T, GDPM_LDS f4* lds) {
    const int ne = T.n_mat * T.eg_n, nr = T.n_mat * T.nr;
    GDPM_LDS f2* rh = (GDPM_LDS f2*)lds;
    GDPM_LDS float* lam = (GDPM_LDS float*)(rh + ne);
    GDPM_LDS float* lr = lam + ne;
    for (int i = threadIdx.x; i < ne; i += blockDim.x) {
        const f4 q = global_f4(T.elec)[i];
        rh[i] = f2{q.x, q.y};
        lam[i] = q.w;
    }
    for (int i = threadIdx.x; i < nr; i += blockDim.x) lr[i] = global_ptr(T.rinv)[i];
    for (int i = threadIdx.x; i < T.n_mat; i += blockDim.x) lr[nr + i] = global_ptr(T.rinv_scale)[i];
    GDPM_LDS float* aw = lr + nr + T.n_mat;
    for (int i = threadIdx.x; i < T.aw_n; i += blockDim.x) aw[i] = global_ptr(T.aw)[i];
    __syncthreads();
    return ElecLds{rh, lam, lr, aw};
}

template <bool kLds, bool kSolo, bool kPerm>
__global__ void __launch_bounds__(1024) k_electron(PassArgs) {
    const Args A = pass_args();
    start_clock(A);
    if (!kPerm && group_idle(A, 1)) return;
    const GroupPtr group = (GroupPtr)lds_tables;
    GDPM_LDS f4* lds = (GDPM_LDS f4*)lds_tables + kGroupTallyF4;
    group_clear(group);
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if constexpr (kLds) {
        const ElecLds E = stage_electron_tables(A->T, lds);
        if (wave < ring_const(A, 1)->group_waves)
            electron_pass<kSolo, kPerm>(
                A, E, (GDPM_LDS float*)(lds + tables_f4(1, A->T) + wave * slice_f4(1, A->bricks)), group);
    } else {
        __syncthreads();
        const ElecGlobal E{global_f4(A->T.elec), global_ptr(A->T.rinv), global_ptr(A->T.rinv_scale),
                           global_ptr(A->T.aw)};
        if (wave < ring_const(A, 1)->group_waves)
            electron_pass<kSolo, kPerm>(A, E, (GDPM_LDS float*)(lds + wave * slice_f4(1, A->bricks)), group);
    }
    group_flush(A, group);
}

// ---------------------------------------------------------------------------
// both passes of an iteration in one launch: the first `photon_waves`
// wavefronts of each workgroup start with the photon pass, the others with the
// electron pass, and a wavefront that has finished its first pass helps with
// the other.  The photon pass mostly waits on its random voxel reads and the
// electron pass mostly issues vector instructions, so a CU runs one while the
// other waits.  The electron tables are in
// LDS; the photon cross sections and majorants are read through the caches; the photons
// have their pool where it fits (kPark, see slice_f4).  Measured slower than the passes
// apart: 16.5, 13.7, 1.13 and 10.7 ms instead of 13.7, 10.6, 1.11 and 10.4 (3e7 photons on
// CTs of 0.2 and 0.4 cm, 3e5 on the latter, 3e6 electrons on slabs).
// Each pass reads what its queue held at the set-up: what either pass pushes
// is transported in the next iteration.
// ---------------------------------------------------------------------------
template <bool kPerm, bool kPark>
__global__ void __launch_bounds__(768) k_transport(PassArgs) {
    const Args A = pass_args();
    start_clock(A);
    const GroupPtr group = (GroupPtr)lds_tables;
    GDPM_LDS f4* lds = (GDPM_LDS f4*)lds_tables + kGroupTallyF4;
    group_clear(group);
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const ElecLds E = stage_electron_tables(A->T, lds);
    GDPM_LDS float* ring = (GDPM_LDS float*)(lds + tables_f4(1, A->T) + wave * slice_f4(kPark ? 2 : 3, A->bricks));
    for (int k = 0; k < 2; ++k) {
        const bool photons = ((int)wave < A->photon_waves) == (k == 0);
        if (photons)
            photon_pass<false, kPerm, false, kPark>(A, PhotGlobal{global_f4(A->T.phot)}, nullptr, ring, group);
        else
            electron_pass<false, kPerm>(A, E, ring, group);
    }
    group_flush(A, group);
}

// ---------------------------------------------------------------------------
// queue re-binning: counting sort of the positions [head, tail) by the key job x
// bin (bins: log2-energy intervals, or boxes of the phantom with `space` > 0).
// The records stay where they are: the count pass keeps each position's key,
// the scatter writes the permutation, in key order, of the positions that hold
// a running job's record (empty ones are dropped), and the pass reads its input
// through it.  Each job's records form one segment of the permutation.
// ---------------------------------------------------------------------------
GDPM_DEV int energy_bin(float e, float lo, float inv, int nb) {
    const int b = (int)((hlog2(e) - lo) * inv);
    return min(max(b, 0), nb - 1);
}

// the box of a position when the phantom is cut into space^3 equal boxes
// (x fastest); positions on or past the far faces fall in the last box
GDPM_DEV int space_bin(const Geom& G, float x, float y, float z, int space) {
    const float sc = (float)space;
    const int bx = min(max((int)(x * G.idx * sc / (float)G.nx), 0), space - 1);
    const int by = min(max((int)(y * G.idy * sc / (float)G.ny), 0), space - 1);
    const int bz = min(max((int)(z * G.idz * sc / (float)G.nz), 0), space - 1);
    return bx + space * (by + space * bz);
}

// the slot of a record's job if that job is running in it (slot below n_jobs,
// same generation), else -1
GDPM_DEV int record_job(const RunDev& R, uint32_t job_word) {
    const int slot = (int)(job_word & 0xFFu);
    if (slot >= R.n_jobs) return -1;
    const uint32_t gen = R.jobs[slot].gen & 0xFFu;
    return ((job_word >> 8) & 0xFFu) == gen ? slot : -1;
}

// re-binning key word of the record in `slot`: job x nb + bin, kEmptyKey for an
// empty position, kOrphanKey for a record of no running job
GDPM_DEV uint32_t record_key(const RunDev& R, const Particle* buf, uint32_t mask, uint32_t slot, int nb,
                             float lo, float inv, int space) {
    const float4 w0 = reinterpret_cast<const float4*>(buf + (slot & mask))[0];
    const float4 w3 = reinterpret_cast<const float4*>(buf + (slot & mask))[3];
    if (record_empty(w0.w)) return kEmptyKey;
    const int j = record_job(R, __float_as_uint(w3.w));
    if (j < 0) return kOrphanKey;
    const int b = space > 0 ? space_bin(R.jobs[j].G, w0.x, w0.y, w0.z, space) : energy_bin(w0.w, lo, inv, nb);
    return (uint32_t)(j * nb + b);
}

__global__ void __launch_bounds__(256) k_bin_count(Ctl* ctl, RunDev R, int ri, int nb, float lo,
                                                   float inv, int space) {
    if (ctl->overflow) return;
    extern __shared__ uint32_t hist[];
    const int nk = R.n_jobs * nb;
    for (int i = threadIdx.x; i < nk; i += blockDim.x) hist[i] = 0u;
    __syncthreads();
    const RingCtl& r = ctl->ring[ri];
    const uint32_t n = r.tail - r.head;
    const Particle* buf = R.buf[ri];
    // each position's key is kept (4 B), so that the scatter does not read
    // the records again
    uint32_t* kw = bin_keys(R.bin[ri]);
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
        const uint32_t k = record_key(R, buf, R.mask[ri], r.head + i, nb, lo, inv, space);
        if (k < kOrphanKey) atomicAdd(&hist[k], 1u);
        kw[i] = k;
    }
    __syncthreads();
    for (int i = threadIdx.x; i < nk; i += blockDim.x)
        if (hist[i]) atomicAdd(&R.jc->bin_count[i], hist[i]);
}

// exclusive scan of the key counts (one block of 1024 threads, <= 4 keys each);
// also the jobs' segments and the number of records kept
__global__ void __launch_bounds__(1024) k_bin_scan(Ctl* ctl, RunDev R, int nb, int ri) {
    if (ctl->overflow) return;
    __shared__ uint32_t part[1024];
    JobCtl* jc = R.jc;
    const int nk = R.n_jobs * nb;
    const int per = (nk + 1023) / 1024;
    const int k0 = threadIdx.x * per;
    uint32_t s = 0u;
    for (int k = k0; k < k0 + per && k < nk; ++k) s += jc->bin_count[k];
    part[threadIdx.x] = s;
    __syncthreads();
    for (int off = 1; off < 1024; off <<= 1) {   // inclusive Hillis-Steele scan
        const uint32_t a = threadIdx.x >= (unsigned)off ? part[threadIdx.x - off] : 0u;
        __syncthreads();
        part[threadIdx.x] += a;
        __syncthreads();
    }
    uint32_t acc = part[threadIdx.x] - s;
    for (int k = k0; k < k0 + per && k < nk; ++k) {
        jc->bin_cursor[k] = acc;
        acc += jc->bin_count[k];
        jc->bin_count[k] = 0u;
    }
    __syncthreads();
    const uint32_t total = part[1023];
    for (int j = threadIdx.x; j < R.n_jobs; j += blockDim.x) {
        const uint32_t b0 = jc->bin_cursor[j * nb];
        const uint32_t b1 = j + 1 < R.n_jobs ? jc->bin_cursor[(j + 1) * nb] : total;
        jc->seg_begin[ri][j] = b0;
        jc->seg_count[ri][j] = b1 - b0;
    }
    if (threadIdx.x == 0) ctl->n_valid = total;
}

__global__ void __launch_bounds__(256) k_bin_scatter(Ctl* ctl, RunDev R, int ri, int nb) {
    if (ctl->overflow) return;
    extern __shared__ uint32_t cnt[];   // [nk] this block's counts, then ranks; [nk] its bases
    const int nk = R.n_jobs * nb;
    uint32_t* base = cnt + nk;
    const RingCtl& r = ctl->ring[ri];
    const uint32_t n = r.tail - r.head;
    const uint32_t mask = R.mask[ri];
    const uint32_t* kw = bin_keys(R.bin[ri]);
    uint32_t* perm = bin_perm(R.bin[ri], mask);
    // each block takes one contiguous share of the positions: it counts its
    // keys, takes its place in every key's run with one atomic per key, then
    // writes its positions (one global atomic per key and block, not per tile)
    const uint32_t per = (n + gridDim.x - 1) / gridDim.x;
    const uint32_t i0 = min(n, blockIdx.x * per), i1 = min(n, i0 + per);
    for (int q = threadIdx.x; q < nk; q += blockDim.x) cnt[q] = 0u;
    __syncthreads();
    for (uint32_t i = i0 + threadIdx.x; i < i1; i += blockDim.x) {
        const uint32_t k = kw[i];
        if (k < kOrphanKey) atomicAdd(&cnt[k], 1u);
    }
    __syncthreads();
    for (int q = threadIdx.x; q < nk; q += blockDim.x) {
        base[q] = cnt[q] ? atomicAdd(&R.jc->bin_cursor[q], cnt[q]) : 0u;
        cnt[q] = 0u;
    }
    __syncthreads();
    for (uint32_t i = i0 + threadIdx.x; i < i1; i += blockDim.x) {
        const uint32_t k = kw[i];
        if (k < kOrphanKey) {
            perm[(base[k] + atomicAdd(&cnt[k], 1u)) & mask] = r.head + i;
        } else if (k == kOrphanKey) {
            // a record of a job no longer running: only a broken bookkeeping
            // leaves one; it is dropped (the count pass skipped it) and counted
            atomicAdd(&ctl->anomalies, 1ull);
        }
    }
}

// live records per job in both queues (a consistency check of the host's
// particle accounting; counts[j] += records of job j)
__global__ void __launch_bounds__(256) k_count_records(const Ctl* ctl, RunDev R,
                                                       unsigned long long* counts) {
    for (int ri = 0; ri < 2; ++ri) {
        const RingCtl& r = ctl->ring[ri];
        const uint32_t n = r.tail - r.head;
        const Particle* buf = R.buf[ri];
        for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
            const float4* q = reinterpret_cast<const float4*>(buf + ((r.head + i) & R.mask[ri]));
            const int j = !record_empty(q[0].w) ? record_job(R, __float_as_uint(q[3].w)) : -1;
            if (j >= 0) atomicAdd(&counts[j], 1ull);
        }
    }
}

// after the re-binning the pass reads the queue through the permutation
__global__ void k_bin_swap(Ctl* ctl, int ri) {
    if (ctl->overflow) return;
    ctl->ring[ri].permuted = 1u;
}


// ---------------------------------------------------------------------------
// batch statistics (section 2.2.1, section 3.1): per voxel the mean over the
// batches of D_b = E_b / (rho V n_b) and its standard error
// ---------------------------------------------------------------------------
// Both kernels are bound by HBM once their grid is small: two workgroups per CU.
// With a workgroup per 256 voxels the reductions at the end, one addition of
// every workgroup to the same address (85 million a second), were all of their
// time: 70 and 96 us on a million voxels, where the data take 20 and 5 us.
constexpr int kStatThreads = 512;

// sums of a and b and maximum of c over the workgroup, in thread 0
GDPM_DEV void block_reduce(double& a, double& b, double& c) {
    __shared__ double sh[3][kStatThreads / 64];
    a = wave_sum(a);
    b = wave_sum(b);
    for (int o = 32; o > 0; o >>= 1) c = fmax(c, __shfl_xor(c, o));
    const int w = threadIdx.x >> 6;
    if (lane_id() == 0) {
        sh[0][w] = a;
        sh[1][w] = b;
        sh[2][w] = c;
    }
    __syncthreads();
    if (threadIdx.x == 0)
        for (int i = 1; i < kStatThreads / 64; ++i) {
            a += sh[0][i];
            b += sh[1][i];
            c = fmax(c, sh[2][i]);
        }
}

// mean and sum of squared deviations of a voxel's batch doses d(0) .. d(nb - 1)
template <class F>
GDPM_DEV void voxel_stats(int nb, F d, double& mean, double& s2) {
    double s = 0.0;
    for (int b = 0; b < nb; ++b) s += d(b);
    mean = s / nb;
    s2 = 0.0;
    for (int b = 0; b < nb; ++b) {
        const double x = d(b) - mean;
        s2 += x * x;
    }
}

typedef const GDPM_CONST StatsArgs* StatsPtr;

// The arguments are read through the kernel-argument segment (the batches'
// normalisation is indexed there).
__global__ void __launch_bounds__(kStatThreads) k_dose_stats(StatsArgs) {
    const StatsPtr A = (StatsPtr)__builtin_amdgcn_kernarg_segment_ptr();
    constexpr int kHeld = 10;   // batches whose energies stay in registers between the two sums
    const GDPM_GLOBAL double* slots = global_ptr(A->slots);
    const GDPM_GLOBAL uint32_t* vox = global_ptr(A->vox);
    GDPM_GLOBAL double* dose = global_ptr(A->dose);
    GDPM_GLOBAL double* sigma = global_ptr(A->sigma);
    const size_t nvox = A->nvox;
    const TallyOrder O = tally_order(*A, A->nx, A->ny);
    const int nb = A->nb;
    const double min_rho = (double)A->min_rho;
    double emax = 0.0, edep = 0.0, none = 0.0;
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < nvox;
         i += (size_t)gridDim.x * blockDim.x) {
        // the voxel whose energies are at position i of the tallies
        size_t o = i;
        if (O.s > 0) {
            const uint32_t b = (uint32_t)(i >> O.s), v = (uint32_t)i;
            const uint32_t row = b / (uint32_t)O.nbx, bz = row / (uint32_t)O.nby;
            const uint32_t bx = b - row * (uint32_t)O.nbx, by = row - bz * (uint32_t)O.nby;
            const uint32_t x = bx << O.mx | (v & O.mx), y = by << O.my | (v >> O.sy & O.my),
                           z = bz << O.mz | (v >> O.sz & O.mz);
            o = x + (size_t)A->nx * (y + (size_t)A->ny * z);
        }
        const double rho = (double)voxel_density(vox[o]);
        const double im = 1.0 / (rho * A->vvox);
        double mean, s2;
        if (nb == kHeld) {
            double eb[kHeld];
#pragma unroll
            for (int b = 0; b < kHeld; ++b) eb[b] = slots[(size_t)b * nvox + i];
#pragma unroll
            for (int b = 0; b < kHeld; ++b) edep += eb[b];
            double s = 0.0;
#pragma unroll
            for (int b = 0; b < kHeld; ++b) s += eb[b] * im * A->inv_n[b];
            mean = s / kHeld;
            s2 = 0.0;
#pragma unroll
            for (int b = 0; b < kHeld; ++b) {
                const double x = eb[b] * im * A->inv_n[b] - mean;
                s2 += x * x;
            }
        } else {
            for (int b = 0; b < nb; ++b) edep += slots[(size_t)b * nvox + i];
            if (nb <= kArgBatches) {
                voxel_stats(nb, [&](int b) { return slots[(size_t)b * nvox + i] * im * A->inv_n[b]; }, mean, s2);
            } else {
                const GDPM_GLOBAL double* inv = (const GDPM_GLOBAL double*)A->red->inv_n;
                voxel_stats(nb, [&](int b) { return slots[(size_t)b * nvox + i] * im * inv[b]; }, mean, s2);
            }
        }
        if (dose) dose[o] = mean;
        if (sigma) sigma[o] = nb > 1 ? sqrt(s2 / ((double)nb * (nb - 1))) : 0.0;
        if (rho >= min_rho) emax = fmax(emax, mean);
    }
    block_reduce(edep, none, emax);
    if (threadIdx.x == 0) {
        StatsDev* red = A->red;
        unsafeAtomicAdd(&red->e_dep, edep);
        atomicMax(&red->dmax_bits, (unsigned long long)__double_as_longlong(emax));
    }
}

// mean of sigma / D_max over voxels with D > D_max / 2
__global__ void __launch_bounds__(kStatThreads) k_unc(StatsDev* red, const double* dose, const double* sigma,
                                                      const uint32_t* vox, float min_rho, size_t nvox) {
    const double dmax = __longlong_as_double((long long)red->dmax_bits);
    double s = 0.0, c = 0.0, none = 0.0;
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < nvox;
         i += (size_t)gridDim.x * blockDim.x) {
        if (dose[i] > 0.5 * dmax && voxel_density(vox[i]) >= min_rho) {
            s += sigma[i];
            c += 1.0;
        }
    }
    block_reduce(s, c, none);
    if (threadIdx.x == 0 && c != 0.0) {
        unsafeAtomicAdd(&red->sigma_sum, s);
        unsafeAtomicAdd(&red->count, c);
    }
}

// the reductions to the host (pinned memory, `seq` last), and zero again
__global__ void k_stats_end(StatsDev* red, StatsDev* out, uint32_t seq) {
    static_assert(offsetof(StatsDev, seq) == 32, "four 8-byte reductions");
    unsigned long long* r = reinterpret_cast<unsigned long long*>(red);
    unsigned long long* o = reinterpret_cast<unsigned long long*>(out);
    for (int i = 0; i < 4; ++i) {
        host_store(o + i, r[i]);
        r[i] = 0ull;
    }
    __hip_atomic_store(&out->seq, seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// ---------------------------------------------------------------------------
// test kernels
// ---------------------------------------------------------------------------
__global__ void k_test_philox(uint32_t k0, uint32_t k1, const uint4* ctr, uint4* out, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    uint4 c = ctr[i];
    philox(k0, k1, c.x, c.y, c.z, c.w);
    out[i] = c;
}

__global__ void k_test_sample(Tables T, int which, float e, float p1, float p2, uint32_t k0,
                              uint32_t k1, int n, float* out1, float* out2) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    RegRng r((uint32_t)i, 0u, 0u);
    float a = 0.0f, b = 0.0f;
    if (which == 0) {
        float eps, t, turns;
        sample_compton(T, r, k0, k1, e, eps, t, turns);
        a = eps;
        b = 1.0f - t;
    } else if (which == 1) {
        float eps, turns;
        sample_moller(r, k0, k1, e, p1, eps, turns);
        const float tt = e, tp = tt - eps * tt, wd = tt - tp;
        a = wd / tt;
        b = hsqrt(tp * (tt + kTwoMec2f) / (tt * (tp + kTwoMec2f)));
    } else if (which == 2) {
        a = sample_brems(r, k0, k1, e, p1);
    } else if (which == 3) {
        a = mw_mu(ElecGrid(T), global_ptr(T.aw), e, uniform(r, k0, k1));
    } else if (which == 4) {
        float u = 0.0f, v = 0.0f, w = 1.0f;
        const int nh = (int)p2;
        for (int k = 0; k < nh; ++k) {
            const float mu = mw_mu(ElecGrid(T), global_ptr(T.aw), e, uniform(r, k0, k1));
            const float turns = uniform(r, k0, k1);
            rotate(u, v, w, 1.0f - 2.0f * mu, 2.0f * hsqrt(mu * (1.0f - mu)), turns);
        }
        a = w;
        b = u * u + v * v + w * w;
    } else if (which == 5) {
        float du, dv, dw;
        sample_iso(r, k0, k1, du, dv, dw);
        a = dw;
        b = -(du * du + dv * dv + dw * dw);
    } else if (which == 6) {
        float tm, tp, aa;
        pair_split(e, uniform(r, k0, k1), tm, tp, aa);
        a = tm / (e - kTwoMec2f);
        b = (tm + tp) - (e - kTwoMec2f);   // 0: the split is exact
    } else if (which == 7) {
        // the photon interaction's kinematics on a photon along +z
        float eps, t, turns;
        sample_compton(T, r, k0, k1, e, eps, t, turns);
        float u = 0.0f, v = 0.0f, w = 1.0f;
        rotate(u, v, w, 1.0f - t, hsqrt(fmaxf(0.0f, t * (2.0f - t))), turns);
        const float e1 = eps * e;
        float eu, ev, ew;
        compton_electron_dir(e, e1, 0.0f, 0.0f, 1.0f, u, v, w, eu, ev, ew);
        a = ew;
        b = w;
    }
    out1[i] = a;
    if (out2) out2[i] = b;
}

GDPM_DEV void test_source_one(const SourceDev& S, const Geom& G, uint32_t k0, uint32_t k1,
                              unsigned long long hist0, int i, int n, float* out, uint32_t* chain) {
    const unsigned long long h = hist0 + i;
    Primary p;
    if (S.n_phsp) {
        p = phase_space_primary(S, G, h);
    } else {
        const f4 d = source_draws(h, k0, k1);
        if (chain) {
            const uint32_t trial = metropolis_trial(S, d.y);
            if (metropolis_moves(d.z, S.f[*chain], S.f[trial])) *chain = trial;
        }
        p = make_primary(S, G, h, d, k0, k1, chain ? (int)*chain : -1, (uint32_t)i, (uint32_t)n);
    }
    float* o = out + 8 * (size_t)i;
    o[0] = p.e;
    o[1] = p.in ? (float)p.beamlet : -1.0f;
    o[2] = p.x; o[3] = p.y; o[4] = p.z;
    o[5] = p.u; o[6] = p.v; o[7] = p.w;
}

// histories hist0 .. hist0+n-1 as a job starting at hist0 samples them; with
// Metropolis chains one thread per chain, the chains freshly started
__global__ void k_test_source(SourceDev S, Geom G, uint32_t k0, uint32_t k1,
                              unsigned long long hist0, int n, float* out) {
    const uint32_t t = blockIdx.x * blockDim.x + threadIdx.x;
    if (S.metro) {
        if (t >= kMetroChains) return;
        uint32_t state = metropolis_start(S, t, k0, k1);
        const uint32_t first = (uint32_t)((t + kMetroChains - hist0 % kMetroChains) % kMetroChains);
        for (uint32_t i = first; i < (uint32_t)n; i += kMetroChains)
            test_source_one(S, G, k0, k1, hist0, (int)i, n, out, &state);
        return;
    }
    if ((int)t >= n) return;
    test_source_one(S, G, k0, k1, hist0, (int)t, n, out, nullptr);
}

// the start of every Metropolis chain of a job
__global__ void k_metro_init(SourceDev S, uint32_t k0, uint32_t k1, uint32_t* chains) {
    const uint32_t c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c < kMetroChains) chains[c] = metropolis_start(S, c, k0, k1);
}

__global__ void k_test_lookup(Tables T, int which, int m, const float* in, float* out, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float x = in[i];
    float r = 0.0f;
    if (which == 0) {
        int gi;
        float gt;
        grid(hlog2(x), T.pg_lo, T.pg_inv, T.pg_n, gi, gt);
        r = lerp4(global_f4(T.phot) + m * T.pg_n, gi, gt).w;
    } else if (which >= 1 && which <= 4) {
        int i;
        float t;
        ElecGrid(T).cell(m, x, i, t);
        const f4 q = lerp4(global_f4(T.elec), i, t);
        r = which == 1 ? q.x : (which == 2 ? q.y : (which == 3 ? q.z : q.w));
    } else if (which == 5) {
        r = range_inv(global_ptr(T.rinv), T.rinv_scale[m], T.nr, m, x);
    } else if (which == 6) {
        r = mw_screening(ElecGrid(T), global_ptr(T.aw), x);
    }
    out[i] = r;
}

// ---------------------------------------------------------------------------
// host launchers (the host runtime calls these; kernels stay in this unit)
// ---------------------------------------------------------------------------
hipError_t launch_setup(hipStream_t st, Ctl* ctl, const RunDev& R, int ri, int rebinned, int lone, const PassGrid& grid) {
    hipLaunchKernelGGL(k_setup, dim3(1), dim3(256), 0, st, ctl, R, ri, rebinned, lone, grid);
    return hipGetLastError();
}
hipError_t launch_source(hipStream_t st, int blocks, Ctl* ctl, const RunDev& R, const SrcSeg* segs,
                         const SrcHdr* hdr, int ri) {
    const SourceArgs a{ctl, R, segs, hdr, ri};
    hipLaunchKernelGGL(k_source, dim3(blocks), dim3(256), 0, st, a);
    return hipGetLastError();
}
hipError_t launch_begin(hipStream_t st, Ctl* ctl, const RunDev& R, const StepHost* h, SrcHdr* hdr, SrcSeg* segs,
                        int setup, int lone, const PassGrid& grid0, const PassGrid& grid1) {
    hipLaunchKernelGGL(k_begin, dim3(1), dim3(256), 0, st, ctl, R, h, hdr, segs, setup, lone, grid0,
                       grid1);
    return hipGetLastError();
}
hipError_t launch_mid(hipStream_t st, Ctl* ctl, const RunDev& R, int setup, int lone, const PassGrid& grid) {
    hipLaunchKernelGGL(k_mid, dim3(1), dim3(256), 0, st, ctl, R, setup, lone, grid);
    return hipGetLastError();
}
hipError_t launch_end(hipStream_t st, Ctl* ctl, const RunDev& R, const StepHost* h, StepMirror* out, int fused) {
    hipLaunchKernelGGL(k_end, dim3(1), dim3(256), 0, st, ctl, R, h, out, fused);
    return hipGetLastError();
}
hipError_t launch_init(hipStream_t st, Ctl* ctl, JobCtl* jc, StatsDev* stats, uint32_t start) {
    hipLaunchKernelGGL(k_init, dim3(1), dim3(1024), 0, st, ctl, jc, stats, start);
    return hipGetLastError();
}
hipError_t launch_admit(hipStream_t st, int cus, const JobDev& job, JobDev* jobs, JobCtl* jc, const float* majorant,
                        float* mumax, size_t n_tally, size_t n_hist, int slot, int n_grid) {
    const AdmitArgs a{job, jobs, jc, majorant, mumax, n_tally, n_hist, slot, n_grid};
    const size_t need = (n_tally + n_hist + 2047) / 2048 + 1;
    hipLaunchKernelGGL(k_admit, dim3((unsigned)(need < (size_t)(8 * cus) ? need : (size_t)(8 * cus))), dim3(256), 0, st, a);
    return hipGetLastError();
}
// LDS bytes of a pass (ri = 2, 3: both in one launch) with `waves` wavefronts per block
// (lds: its tables staged; bricks: the electrons' brick sums)
size_t transport_lds_bytes(int ri, const Tables& T, int waves, bool lds, bool bricks) {
    const size_t per_wave = slice_f4(ri, bricks);
    return (kGroupTallyF4 + (lds ? (size_t)tables_f4(ri, T) : 0) + (size_t)waves * per_wave) * sizeof(float4);
}

// allow the kernels to use `bytes` of dynamic LDS
hipError_t transport_lds_optin(size_t bytes) {
    const void* kernels[] = {(const void*)k_photon<false, false, false>, (const void*)k_electron<false, false, false>,
                             (const void*)k_photon<false, false, true>, (const void*)k_electron<false, false, true>,
                             (const void*)k_photon<true, false, false>, (const void*)k_electron<true, false, false>,
                             (const void*)k_photon<true, false, true>,  (const void*)k_electron<true, false, true>,
                             (const void*)k_photon<true, true, false>,  (const void*)k_electron<true, true, false>,
                             (const void*)k_photon<true, true, true>,   (const void*)k_electron<true, true, true>,
                             (const void*)k_transport<false, false>,    (const void*)k_transport<true, false>,
                             (const void*)k_transport<false, true>,     (const void*)k_transport<true, true>};
    for (const void* k : kernels) {
        const hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

namespace {
template <bool kPerm>
void launch_transport_form(hipStream_t st, int ri, int blocks, int threads, bool lds, bool solo, size_t bytes,
                           const PassArgs& a) {
    if (ri == 0) {
        if (solo)
            hipLaunchKernelGGL((k_photon<true, true, kPerm>), dim3(blocks), dim3(threads), bytes, st, a);
        else if (lds)
            hipLaunchKernelGGL((k_photon<true, false, kPerm>), dim3(blocks), dim3(threads), bytes, st, a);
        else
            hipLaunchKernelGGL((k_photon<false, false, kPerm>), dim3(blocks), dim3(threads), bytes, st, a);
    } else {
        if (solo)
            hipLaunchKernelGGL((k_electron<true, true, kPerm>), dim3(blocks), dim3(threads), bytes, st, a);
        else if (lds)
            hipLaunchKernelGGL((k_electron<true, false, kPerm>), dim3(blocks), dim3(threads), bytes, st, a);
        else
            hipLaunchKernelGGL((k_electron<false, false, kPerm>), dim3(blocks), dim3(threads), bytes, st, a);
    }
}
}  // namespace

// `solo`: the one-particle-per-wavefront measurement form (staged tables only);
// `permuted`: the pass follows a re-binning by job alone (its input is read
// through the permutation)
hipError_t launch_transport(hipStream_t st, int ri, int blocks, int threads, bool lds, bool bricks, bool solo,
                            bool permuted, Ctl* ctl, const Tables& T, const RunDev& R) {
    const size_t bytes = transport_lds_bytes(ri, T, threads / 64, lds, bricks);
    if (solo && !lds) return hipErrorInvalidValue;
    const PassArgs a{ctl, T, R, 0, bricks};
    if (permuted)
        launch_transport_form<true>(st, ri, blocks, threads, lds, solo, bytes, a);
    else
        launch_transport_form<false>(st, ri, blocks, threads, lds, solo, bytes, a);
    return hipGetLastError();
}
// both passes in one launch (k_transport); ri: 2 or 3, see slice_f4
hipError_t launch_fused(hipStream_t st, int ri, int blocks, int threads, int photon_waves, bool bricks, bool permuted,
                        Ctl* ctl, const Tables& T, const RunDev& R) {
    const size_t bytes = transport_lds_bytes(ri, T, threads / 64, true, bricks);
    const PassArgs a{ctl, T, R, photon_waves, bricks};
    void (*const k)(PassArgs) = ri == 2 ? (permuted ? k_transport<true, true> : k_transport<false, true>)
                                        : (permuted ? k_transport<true, false> : k_transport<false, false>);
    hipLaunchKernelGGL(k, dim3(blocks), dim3(threads), bytes, st, a);
    return hipGetLastError();
}

// nb bins per job (energy intervals, or space^3 boxes with space > 0);
// R.n_jobs * nb <= kMaxKeys
hipError_t launch_rebin(hipStream_t st, int blocks, Ctl* ctl, const RunDev& R, int ri, int nb,
                        float lo, float inv, int space) {
    const size_t nk = (size_t)R.n_jobs * nb;
    hipLaunchKernelGGL(k_bin_count, dim3(blocks), dim3(256), nk * sizeof(uint32_t), st, ctl, R, ri,
                       nb, lo, inv, space);
    hipLaunchKernelGGL(k_bin_scan, dim3(1), dim3(1024), 0, st, ctl, R, nb, ri);
    hipLaunchKernelGGL(k_bin_scatter, dim3(blocks), dim3(256), 2 * nk * sizeof(uint32_t), st, ctl, R,
                       ri, nb);
    hipLaunchKernelGGL(k_bin_swap, dim3(1), dim3(1), 0, st, ctl, ri);
    return hipGetLastError();
}
hipError_t launch_count_records(hipStream_t st, int blocks, const Ctl* ctl, const RunDev& R,
                                unsigned long long* counts) {
    hipLaunchKernelGGL(k_count_records, dim3(blocks), dim3(256), 0, st, ctl, R, counts);
    return hipGetLastError();
}
hipError_t launch_stats(hipStream_t st, int cus, const StatsArgs& a, StatsDev* out, uint32_t seq) {
    const size_t need = (a.nvox + kStatThreads - 1) / kStatThreads;
    const int blocks = (int)(need < (size_t)(2 * cus) ? need : (size_t)(2 * cus));
    hipLaunchKernelGGL(k_dose_stats, dim3(blocks), dim3(kStatThreads), 0, st, a);
    hipLaunchKernelGGL(k_unc, dim3(blocks), dim3(kStatThreads), 0, st, a.red, (const double*)a.dose,
                       (const double*)a.sigma, a.vox, a.min_rho, a.nvox);
    hipLaunchKernelGGL(k_stats_end, dim3(1), dim3(1), 0, st, a.red, out, seq);
    return hipGetLastError();
}
hipError_t launch_test_philox(hipStream_t st, uint32_t k0, uint32_t k1, const uint4* ctr, uint4* out,
                              int n) {
    hipLaunchKernelGGL(k_test_philox, dim3((n + 255) / 256), dim3(256), 0, st, k0, k1, ctr, out, n);
    return hipGetLastError();
}
hipError_t launch_test_sample(hipStream_t st, const Tables& T, int which, float e, float p1, float p2,
                              uint32_t k0, uint32_t k1, int n, float* out1, float* out2) {
    hipLaunchKernelGGL(k_test_sample, dim3((n + 255) / 256), dim3(256), 0, st, T, which, e, p1, p2,
                       k0, k1, n, out1, out2);
    return hipGetLastError();
}
hipError_t launch_test_source(hipStream_t st, const SourceDev& S, const Geom& G, uint32_t k0,
                              uint32_t k1, unsigned long long hist0, int n, float* out) {
    const int blocks = S.metro ? (int)(kMetroChains / 256) : (n + 255) / 256;
    hipLaunchKernelGGL(k_test_source, dim3(blocks), dim3(256), 0, st, S, G, k0, k1, hist0, n, out);
    return hipGetLastError();
}
hipError_t launch_metro_init(hipStream_t st, const SourceDev& S, uint32_t k0, uint32_t k1, uint32_t* chains) {
    hipLaunchKernelGGL(k_metro_init, dim3(kMetroChains / 256), dim3(256), 0, st, S, k0, k1, chains);
    return hipGetLastError();
}
// scattered FP64 atomic additions: `iters` per thread at hashed addresses of
// an array of n words (the dose tally's access pattern without the transport)
__global__ void __launch_bounds__(256) k_atomic_rate(double* buf, uint32_t n, uint32_t iters) {
    const uint32_t t = blockIdx.x * blockDim.x + threadIdx.x;
    for (uint32_t k = 0; k < iters; ++k) {
        uint32_t h = t * 0x9E3779B9u + k * 0x85EBCA6Bu;
        h ^= h >> 16;
        h *= 0x7FEB352Du;
        h ^= h >> 15;
        h *= 0x846CA68Bu;
        h ^= h >> 16;
        unsafeAtomicAdd(&buf[h % n], 1.0);
    }
}

hipError_t launch_atomic_rate(hipStream_t st, int blocks, double* buf, uint32_t n, uint32_t iters) {
    hipLaunchKernelGGL(k_atomic_rate, dim3(blocks), dim3(256), 0, st, buf, n, iters);
    return hipGetLastError();
}

hipError_t launch_test_lookup(hipStream_t st, const Tables& T, int which, int m, const float* in,
                              float* out, int n) {
    hipLaunchKernelGGL(k_test_lookup, dim3((n + 255) / 256), dim3(256), 0, st, T, which, m, in, out, n);
    return hipGetLastError();
}

}  // namespace gdpm
