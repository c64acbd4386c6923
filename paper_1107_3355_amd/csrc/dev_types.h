// Plain data shared by the host runtime and the HIP kernels of libgdpm.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <string.h>

namespace gdpm {

constexpr int kMaxMaterials = 8;
constexpr uint32_t kPushMin = 32;       // ring slots a wavefront reserves at a time: its
constexpr uint32_t kPushMax = 256;      // first claim of the pass, within these bounds (the upper
                                        // one for narrow passes, see setup_pass)
constexpr uint32_t kClaimMin = 32;      // smallest number of queue items a wavefront claims
                                        // with one atomic, and the largest, per particle type:
constexpr uint32_t kClaimMaxPhoton = 2048;   // a photon record lasts a few short iterations, so
constexpr uint32_t kClaimMaxElectron = 256;  // photon wavefronts claim often: larger chunks keep
                                             // them off the shared claim counter
constexpr uint32_t kWideMin = 16;       // a pass with this many records per lane uses all
                                        // wavefronts of its workgroups (see PassGrid),
constexpr uint32_t kWideMinJob = 8;     // if each job has this many on average
constexpr int kMaxBins = 64;            // energy bins of the queue re-binning
constexpr int kMaxJobs = 256;           // dose jobs transported together
constexpr int kMaxKeys = 4096;          // re-binning keys (job x energy bin)
constexpr uint32_t kTailLanes = 16;     // a drained wavefront with fewer particles
                                        // than this hands them to the next pass ...
constexpr uint32_t kTailMinPerLane = 4; // ... if the pass had this many per lane
#ifndef GDPM_HARD_BATCH
#define GDPM_HARD_BATCH 12
#endif
constexpr uint32_t kHardBatch = GDPM_HARD_BATCH;  // electron hard events sampled together
#ifndef GDPM_REAL_BATCH
#define GDPM_REAL_BATCH 22
#endif
constexpr uint32_t kRealBatch = GDPM_REAL_BATCH;  // photon interactions sampled together
constexpr int kAbsorb = 1 << 8;         // a photon to be absorbed where it is (in place of the
                                        // material of a waiting interaction)
constexpr uint32_t kRefillMin = 12;     // empty lanes a wavefront refills at once
constexpr float kMaxEnergy = 1.0e6f;    // MeV; a larger or non-finite energy marks a
                                        // damaged record
constexpr uint32_t kMaxWaveIterations = 1u << 21;  // bound of a wavefront's loop in one
                                        // pass (about 1e3 in practice)

// event counters (same order as the GDPM_EV_* enumeration of the C ABI)
enum { EV_FLIGHTS = 0, EV_REAL, EV_ESTEPS, EV_HARD_CAND, EV_HARD, EV_DEPOSITS, EV_PUSHES,
       EV_HISTORIES };

// An empty queue position carries exactly this energy.  A particle's own
// energy never does: it is >= 0, or a rounding below 0 by a few ulps that the
// transport ends as an absorption, so such a record must still be read as a
// particle (an empty-slot test of e < 0 would lose it: born, never ended).
constexpr float kEmptyEnergy = -1.0f;
__host__ __device__ inline bool record_empty(float e) { return e == kEmptyEnergy; }

// A particle record: 64 bytes, four 16-byte vectors.
struct alignas(16) Particle {
    float x, y, z, e;        // position (cm), kinetic energy (MeV); kEmptyEnergy marks an empty slot
    float u, v, w, nh;       // direction; hard-event mean free paths left (< 0: unset)
    uint32_t hlo, hhi;       // history id
    uint32_t path, ctr;      // Philox stream path id and draw counter
    uint32_t vox;            // charged particles: ix | iy << 11 | iz << 22
    float a;                 // positron: energy of its two annihilation photons together
    uint32_t flags;          // bit 0: positron
    uint32_t job;            // bits 0-7: job slot; 8-15: the slot's generation; 16-31: batch slot
};
static_assert(sizeof(Particle) == 64, "particle record is 64 bytes");

// The wavefronts of a pass: `wide` per workgroup are launched, and if the pass has
// fewer than kWideMin records for each of their lanes, or kWideMinJob in each job,
// only the first `narrow` of them work.  16 wavefronts per CU instead of 12 hide more of
// the latencies, of the electrons' dependent table lookups and the photons' random
// voxel reads: on passes of 5e6 histories (CT, 0.4 cm) the electrons took 19.9
// instead of 22.0 ms and the photons 19.1 instead of 20.7.  With few records the
// wavefronts only share them: the electrons of 1e5 histories took 372 and 343 us.  The
// line: with 4, 8, 16 and 32 records the electrons of 3e6 split histories took 1.97, 1.87,
// 1.87 and 1.99 ms, those of 1e7 histories on slabs 2.33, 2.28, 2.22 and 2.22.  Of
// several jobs: 24 of 1e5 to 3e6 histories took 6.0 ms (photons) and 8.8 (electrons)
// with 16 and 5.3 and 7.9 with 12; four of 5e6 237 ms with 16 and 245 with 12.
struct PassGrid {
    uint32_t blocks, wide, narrow;
};

// One queue (ring buffer of 2^k records, indices wrap modulo 2^32).  Counters
// that many wavefronts add to have a cache line of their own each: additions to
// one line are served one after the other (85 million a second, whatever the
// address in it), and readers of its other words wait with them.
struct alignas(128) RingCtl {
    uint32_t tail;                   // records in [head, tail); wavefronts reserve slots here
    uint32_t pad0[31];
    uint32_t head;
    uint32_t begin, count;   // input of the running pass: [begin, begin + count)
    uint32_t first;          // records a wavefront takes without claiming them (0: it claims)
    uint32_t push;           // slots a wavefront of the running pass reserves at a time
    uint32_t permuted;       // 1: the pass reads its input through the permutation
    uint32_t next_head;      // head after a permuted pass (the tail before it)
    uint32_t group_waves;    // the wavefronts of a workgroup that work in the running pass
    uint32_t pad1[24];
};
static_assert(sizeof(RingCtl) == 256, "two cache lines");

// Device-resident control block of the transport (the host reads it back
// after every scheduler iteration).
struct Ctl {
    RingCtl ring[2];                  // 0 photons, 1 electrons/positrons
    uint32_t overflow;                // (read before every claim)
    uint32_t pad0[31];
    uint32_t n_valid;                 // records kept by the last compaction
    uint32_t pad1;
    unsigned long long t_start;       // device clock when the running pass started
    unsigned long long ticks[3];      // clock ticks in photon, electron and fused passes
    unsigned long long ev[8];
    unsigned long long pass_ev[2][4];  // per pass type: records loaded, records
                                       // stored, tally deposits, records handed
                                       // to the next pass of the same type
    unsigned long long itype[5];      // real interactions: Compton, photoelectric,
                                       // pair, Moller, bremsstrahlung
    unsigned long long anomalies;     // particles ended by a loop bound (0 in a sound run)
};

// a job's statistics: the reductions, and the batches' normalisation if there
// are more than kArgBatches (else it goes with the kernel's arguments)
constexpr int kMaxBatches = 1000;       // N_b of a job
constexpr int kArgBatches = 32;
struct StatsDev {
    double e_dep, sigma_sum, count;     // energy in the tallies; sum of sigma and number of
                                        // voxels above half the maximum dose
    unsigned long long dmax_bits;       // the maximum dose
    uint32_t seq, pad[7];               // (in the host's copy: number of the calculation)
    double inv_n[kMaxBatches];          // 1 / histories of each batch
};

// The order of a job's energy tally: bricks of up to kBrickVoxels voxels, x fastest,
// with the voxels of a brick together (x fastest too).  The electron pass sums a
// particle's deposits in a brick and adds them to the tally together: the tally is
// bound by the number of 64-byte lines that the additions touch (23.5 G a second on the
// whole device, wherever they lie), not by their bytes.  A brick is two voxels wide
// along the two axes with the smallest spacing, whose faces particles cross most
// often (z, then y if equal: the fixed beams run along z), of those with an even
// number of voxels, so that bricks need no padding.
struct Brick {
    int mx, my, mz;   // 1: bricks are two voxels wide along the axis, else 0
};
constexpr int kBrickVoxels = 4;
inline Brick brick_of(const int n[3], const double d[3], bool plain) {
    Brick b{0, 0, 0};
    int* m[3] = {&b.mx, &b.my, &b.mz};
    for (int k = 1; k < kBrickVoxels && !plain; k *= 2) {
        int best = -1;
        for (int a = 2; a >= 0; --a)
            if (!*m[a] && n[a] % 2 == 0 && (best < 0 || d[a] < d[best])) best = a;
        if (best >= 0) *m[best] = 1;
    }
    return b;
}

struct StatsArgs {
    StatsDev* red;           // zero at the start
    const double* slots;     // [nb][nvox] energy tallies, in `brick` order
    size_t nvox;
    Brick brick;
    int nx, ny;              // voxels along x and y
    const uint32_t* vox;
    double vvox;
    double* dose;
    double* sigma;
    int nb;
    float min_rho;
    double inv_n[kArgBatches];
};

// counters of a transport pass, per particle type
enum PassCounters { PC_EVENTS = 0,    // flights or steps
                    PC_REAL,          // real interactions; hard-event candidates
                    PC_HARD,          // electrons: hard events
                    PC_DEPOSITS, PC_PUSHES, PC_LOADED, PC_REQUEUED, PC_ANOMALIES,
                    PC_TYPE0,         // photoelectric; Moller
                    PC_TYPE1,         // pair
                    kPassCounters = 16 };
constexpr int kParts = 8;

// Per-job counters and the job segments of the running pass.  The first four
// arrays are read back by the host after every iteration: a job whose births
// equal its deaths has no particle left in the queues.
struct JobCtl {
    unsigned long long births[kMaxJobs];   // queue records created (primaries, secondaries)
    unsigned long long deaths[kMaxJobs];   // particles ended (absorbed, escaped)
    double e_in[kMaxJobs];                 // source kinetic energy (MeV)
    double e_esc[kMaxJobs];                // energy leaving the phantom (MeV)
    // per particle type [ri] (the two passes of an iteration may run at once):
    uint32_t seg_begin[2][kMaxJobs];       // the job's records in the pass input:
    uint32_t seg_count[2][kMaxJobs];       //   [seg_begin, seg_begin + seg_count)
    uint32_t claim[2][kMaxJobs];           // claim counter of the job's segment
    unsigned long long left[2][kMaxJobs / 64];  // jobs with unclaimed records
    uint32_t bin_count[kMaxKeys];
    uint32_t bin_cursor[kMaxKeys];
    // what the workgroups of a running pass counted (see PassCounters), in
    // kParts parts that lie on different cache lines; folded into the control
    // block by the pass's completion
    unsigned long long part[2][kParts][kPassCounters];
};

// Interpolation tables (single precision, linear in log2 E).
struct Tables {
    const float4* phot;    // [mat][pg_n] {muC, muPE, muPair, muTot} cm^2/g
    const float* mumax;    // [pg_n] Woodcock majorant of the phantom, 1/cm
    float pg_lo, pg_inv;   // node i at log2 E = pg_lo + i / pg_inv
    int pg_n;
    const float4* elec;    // [mat][eg_n] {R g/cm^2, muHard, muMoller, 1/lambda1 cm^2/g}
    float eg_lo, eg_inv;
    int eg_n;
    const float* rinv;     // [mat][nr] E at w = sqrt(R), w uniform from 0
    const float* rinv_scale;  // [mat] (nr - 1) / w_max
    int nr;
    const float* aw;       // [aw_n] log2 A at log2 t = aw_lo + i / aw_inv
    float aw_lo, aw_inv;
    int aw_n;
    int n_mat;
    const float* kn;       // [kn_ne][kn_nu] Klein-Nishina inverse: ln(eps/eps0)/ln(1/eps0)
    float kn_lo, kn_inv;   // at log2 E = kn_lo + i / kn_inv and u = j / (kn_nu - 1)
    int kn_ne, kn_nu;
};

// A voxel of the phantom in 4 bytes: the density's single-precision mantissa
// (bits 0-22), its exponent less kVoxExpBias (bits 23-27: densities in
// [2^-16, 2^16) g/cm^3, every single-precision value there exactly) and the
// material id (bits 28-31).  Half the bytes of a {density, material} pair, so
// the random voxel gathers of the transport touch half the cache lines.
constexpr uint32_t kVoxExpBias = 111u;   // single-precision exponent field of 2^-16
static_assert(kMaxMaterials <= 16, "material ids take 4 bits of a packed voxel");
__host__ __device__ inline bool voxel_density_ok(float rho) {
    const float lo = 1.0f / 65536.0f, hi = 65536.0f;
    return rho >= lo && rho < hi;
}
__host__ __device__ inline uint32_t pack_voxel(float rho, uint32_t mat) {
    uint32_t bits;
    memcpy(&bits, &rho, 4);
    return (bits - (kVoxExpBias << 23)) | (mat << 28);
}
__host__ __device__ inline float voxel_density(uint32_t w) {
    const uint32_t bits = (w & 0x0FFFFFFFu) + (kVoxExpBias << 23);
    float r;
    memcpy(&r, &bits, 4);
    return r;
}
__host__ __device__ inline int voxel_material(uint32_t w) { return (int)(w >> 28); }

struct Geom {
    const uint32_t* vox;   // packed voxels (pack_voxel)
    int nx, ny, nz;
    float dx, dy, dz;
    float idx, idy, idz;   // 1 / voxel size
    float lx, ly, lz;      // extent
};

struct BeamDev {
    float iso[3], dir[3], e1[3], e2[3];
    float sad, bw, bh, hx, hy;   // hx = nbx * bw / 2, hy = nby * bh / 2
    int nbx, nby, off;
};

struct SourceDev {
    int particle, spec_kind, spec_n;
    float e_mono;
    const float* spec_e;
    const float* spec_p;
    const float* spec_c;       // cumulative area at spec_e
    const double* cdf;         // nf + 1 beamlet probabilities P(I)
    int nf;
    const uint32_t* guide;     // guide[k]: I with P(I) <= k / n_guide (start of the search)
    int n_guide;
    const BeamDev* beams;
    const uint16_t* beam_of;   // beamlet -> beam
    int n_beams;
    int metro;                 // 1: Metropolis beamlet chains (Algorithm A1)
    int n_nz;                  // beamlets of nonzero intensity ...
    const uint32_t* nz;        // ... their indices
    const float* f;            // [nf] intensities (negative ones as 0)
    int strata;                // K > 0: energy intervals of a round (section 2.3.2)
    const double* strata_F;    // [K + 1] spectrum CDF at the interval edges
    int strata_shape;          // inside an interval: 0 uniform energy, 1 the spectrum's shape
    float strata_lo, strata_w; // lower edge of the first interval, interval width (MeV)
    const float* phsp;         // [n_phsp][7] phase-space records, or null (section 2.3.3)
    unsigned long long n_phsp;
};

// One dose job: its phantom, source, random key and tallies.
struct JobDev {
    Geom G;
    SourceDev S;
    const float* mumax;        // [pg_n] Woodcock majorant of the job's phantom, 1/cm
    double* tally;             // [n_batches][nv] energy tallies (MeV per voxel), in `brick` order
    unsigned long long nv;     // voxels of the phantom
    Brick brick;
    double* hist;              // per-history (deposited, escaped) or null
    unsigned long long hist0;  // history id of hist[0]
    uint32_t k0, k1;           // Philox key
    uint32_t flags;            // GDPM_* run flags
    uint32_t gen;              // generation of the slot (8 bits): records of an earlier
                               // job in the same slot carry another one
    uint32_t* chains;          // [kMetroChains] Metropolis chain states, or null
    uint32_t split;            // primary splitting: 2^split copies of each history's primary
                               // (tallied at weight 1; the host scales the job's sums by 2^-split)
};

// A run of new histories for the source pass: ids [h0, h0 + n) of job `job`,
// batch slot `batch`, written to queue slots tail + off + i.
struct SrcSeg {
    unsigned long long h0;
    uint32_t n, off;
    uint32_t job, batch;
    uint32_t rpos, rsize;      // position of h0 in its round, and the round's size
    uint32_t unit0;            // its first unit of work in the source pass (see source_units)
    uint32_t lanes, group;     // Metropolis sources: lanes per chain, and the number of
    uint32_t pad;              // segments, this one first, that the job's chains run through
};

// Units of the source pass, one wavefront's work at a time: 64 histories of a
// segment; or 64 / lanes of a Metropolis source's chains through all segments of
// the job (the units are the first segment's).  A chain of n / kMetroChains
// steps per segment gets as many lanes as it has steps, a power of two up to 64.
constexpr uint32_t kMetroChains = 16384;   // Metropolis chains of a job
inline uint32_t metro_lanes(uint64_t n) {
    uint32_t g = 1;
    while (g < 64u && 2u * g <= n / kMetroChains) g *= 2u;
    return g;
}
inline uint32_t source_units(uint64_t n, bool metro, uint32_t lanes) {
    return metro ? kMetroChains / (64u / lanes) : (uint32_t)((n + 63) / 64);
}


// The source passes of one scheduler iteration, per particle type: the host
// writes the numbers of segments and records (pinned memory), the iteration's
// first kernel copies the segments to the device and notes where the records go.
// The kernels read all of it from memory, so that a recorded launch sequence
// stays valid while it changes.
struct SrcHdr {
    uint32_t nseg, total;    // segments, records
    uint32_t base;           // queue position of the first record
    uint32_t units;          // units of work
};
constexpr int kMaxSegs = 4096;          // source segments per iteration (both types)
struct StepHost {
    SrcHdr hdr[2];
    uint32_t seq;            // number of the iteration, echoed when it has ended
    uint32_t pad[7];
    SrcSeg segs[kMaxSegs];   // photon sources' segments, then from kMaxSegs / 2 electron sources'
};

// what the host reads after an iteration (pinned memory, written by the
// iteration's last kernel, `seq` last)
struct StepMirror {
    Ctl ctl;
    unsigned long long births[kMaxJobs], deaths[kMaxJobs];
    double e_in[kMaxJobs], e_esc[kMaxJobs];
    uint32_t seq, pad[31];
};

// The re-binning leaves the records where they are.  Each queue has a
// re-binning buffer of 2C 32-bit words, C the queue capacity: each input
// position's key (kEmptyKey for an empty position, kOrphanKey for a record of a
// job no longer running), then the permutation, the queue positions of the
// pass's input in key order, which the pass reads its input through.
constexpr uint32_t kEmptyKey = 0xFFFFFFFFu, kOrphanKey = 0xFFFFFFFEu;
constexpr size_t kBinWordsPerSlot = 2;
__host__ __device__ inline uint32_t* bin_keys(uint32_t* bin) { return bin; }
__host__ __device__ inline uint32_t* bin_perm(uint32_t* bin, uint32_t mask) { return bin + ((size_t)mask + 1u); }

struct RunDev {
    float ecut_g, ecut_e;      // shared by every job (the tables depend on them)
    const JobDev* jobs;
    JobCtl* jc;
    int n_jobs;                // job slots in use
    int nb;                    // energy bins per job of the re-binning
    Particle* buf[2];          // the queues' records [ring]
    uint32_t* bin[2];          // their re-binning buffers (2 words per queue slot), or null
    uint32_t mask[2];          // capacity - 1
    uint32_t hard[2];          // fill above which a reservation fails
};

// arguments of the transport kernels
struct PassArgs {
    Ctl* ctl;
    Tables T;
    RunDev R;
    int photon_waves;   // fused form: wavefronts of a workgroup that start with photons
    int bricks;         // the workgroup's LDS holds the brick sums of the electrons
};

}  // namespace gdpm
