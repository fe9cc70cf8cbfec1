// sa_internal.h -- contract between the host packer (sa_host.cpp), the C ABI (sa_api.cpp) and the
// HIP kernels (sa_kernels.hip).  Not installed; include/sa.h is the public interface.
#pragma once

#include <cstddef>
#include <cstdint>
#include <string>
#include <vector>

#include "../../include/sa.h"

namespace sa {

// Largest exponent of one variable inside one term that the heat-bath and optimal-transition
// kernels accept (their per-variable polynomial dE(v) = sum_m a_m (v^m - z^m) keeps m <= this).
constexpr int kMaxExpPoly = 16;
// Largest exponent stored at all (8-bit field of the incidence record).
constexpr int kMaxExpStored = 255;
// Heat-bath weights kept in registers when ceil(W/64) <= this; wider ranges recompute them.
constexpr int kHeatBathRegChunk = 32;
// Optimal transition: ranges up to this width take the argmin by enumeration, wider ones from the
// sign changes of the energy difference's forward differences (the same value).
constexpr int kOtmEnumMax = 2048;

// Canonical polynomial: merged terms, nonzero coefficients, factors sorted (a power is a
// repeated index).
struct Canonical {
    int32_t n = 0;
    std::vector<int64_t> t_off;   // n_terms + 1 offsets into t_var
    std::vector<int32_t> t_var;   // factor indices, ascending inside a term
    std::vector<int64_t> t_coef;  // nonzero coefficients
    std::vector<int32_t> lo, hi;  // integer box
    int64_t n_terms() const { return (int64_t)t_coef.size(); }
};

// Validates and canonicalises; returns an SA_* status and fills err on failure.
int canonicalize(const sa_instance *inst, const sa_bounds *bounds, Canonical &out, std::string &err);
// SA_ERANGE when sum_t |J_t| prod zmax^e >= 2^62.  Also reports the largest |dE| bound.
int check_int64_bound(const Canonical &c, std::string &err, double *bound_out);
// True when max_k sum_{t containing k} |J_t| prod_{factors} zmax^e < 2^29, so every energy
// difference |dE| < 2^30 and the difference of two of them fit 32-bit signed arithmetic.
bool dE_fits_32(const Canonical &c);
// every coefficient a_k^(m) (and each incidence record's product) below 2^31 in magnitude
bool coefs_fit_32(const Canonical &c);
// Sec. 3.4 temperature range (T_init, T_final); SA_EINVAL if the problem has no energy scale.
int auto_temperatures(const Canonical &c, double *t_init, double *t_final, std::string &err);
// Geometric cooling of Sec. 3.1 between the two temperatures, as inverse temperatures.
void geometric_betas(double t_init, double t_final, int32_t n_sweeps, double *beta_out);

// Variable record: {lower bound, width W = u - l + 1, first incidence, number of incidences}.
struct VarRec {
    int32_t lo, width, row, deg;
};
// Incidence record of variable k in term t: meta = e_k(t) | (n_other << 8); the other factors
// (indices repeated by exponent) inline in o[0..2] when n_other <= 3, else o[0] is the offset of
// n_other indices in the overflow array (a multiple of four; the list is padded with -1 to a
// multiple of four entries).
struct IncRec {
    uint32_t meta;
    int32_t o[3];
};

// Compact incidence record of a pair term J z_k z_j (index of the other factor j, coefficient J).
struct PairRec {
    int32_t j;
    int32_t J;
};
// a variable's pair records are padded with zero records to a multiple of this many
constexpr int32_t kPairBlock = 16;

// Host-side packed image of a plan (uploaded as one device allocation).
struct Packed {
    int32_t n = 0;
    int32_t n_terms = 0;
    std::vector<VarRec> var;
    std::vector<uint32_t> emask;    // bit m set: some term holds z_k^m (m = 1..31; 31 = ">= 31")
    std::vector<IncRec> inc;
    std::vector<int64_t> inc_coef;
    std::vector<int32_t> overflow;  // other-factor indices of incidences with > 3 others
    int32_t max_other = 0;          // most other factors of any incidence (1: pair terms only)
    std::vector<int32_t> t_off;     // term-major copy for energies
    std::vector<int32_t> t_var;
    std::vector<int64_t> t_coef;
    int32_t max_exp = 0;
    int32_t max_width = 1;
    // dense QUIO form (no incidence records): E = sum_k h_k z_k + d_k z_k^2 + sum_{j<k} J_kj z_j z_k
    // with J stored as a symmetric n x row_stride matrix (zero diagonal and padding)
    bool dense = false;
    int32_t jbytes = 0;             // 1 (int8) or 4 (int32)
    int32_t row_stride = 0;         // elements per matrix row (multiple of 16)
    std::vector<int8_t> jd8;
    std::vector<int32_t> jd32;
    std::vector<int64_t> h, d;
    int64_t n_pairs = 0;
    // compact form of a multilinear QUIO whose coefficients fit int32 (empty otherwise): per
    // variable its pair records (row pair_row[k], pair_deg[k] of them, followed by zero records
    // {0, 0} up to a multiple of kPairBlock) and its linear coefficient
    std::vector<PairRec> pair;
    std::vector<int32_t> pair_row, pair_deg, pair_h;
    bool pair16 = false;   // they have 16-bit indices and couplings
    // settled sweeps (sa_settled.h): 1 for a variable that keeps its coefficients cached (every term holds
    // it to the first or second power, and no variable of the term has more than three other factors there)
    std::vector<uint8_t> cached;
    bool any_cached = false, any_square = false;   // of one that is not fixed / and has a square
    bool z30 = false, z23 = false;  // every bound below 2^30, 2^23 in magnitude
    double energy_bound = 0.0;      // sum_t |J_t| prod zmax^e (check_int64_bound; set by the caller of pack)
};
int pack(const Canonical &c, Packed &out, std::string &err);
int maxe_class_of(int32_t max_exp);

// One slot of the sweep schedule: in window w, wave g of a replica updates variable k (k = -1:
// the wave idles in that window).  Variables of one window share no term, so their updates
// commute and may run at the same time; windows follow the index order of the sweep (Sec. 3.1)
// and fixed variables (l = u) are left out.
struct SchedRec {
    int32_t k;
    int32_t lo, width, row, deg;
    uint32_t emask;
    int32_t pad[2];   // pad[1]: 1 for a variable whose coefficients settled sweeps keep cached
};
// Greedy windows of at most G mutually non-interacting variables, stored wave-major
// (slot g * n_win + w).  Returns the number of windows.
int32_t build_schedule(const Packed &p, int G, std::vector<SchedRec> &out);

// Every variable in index order, k = -1 for a fixed one; returns the number that are not fixed.
int32_t build_order(const Packed &p, std::vector<SchedRec> &out);

// Dependency levels of one sweep: a level holds, in index order, variables (not fixed) none of
// which shares a term with another, each placed after all of its lower-index neighbours' levels.
// Updating the levels one after another, the variables of a level in any order or at once, reads
// every neighbour exactly as the sequential index-order sweep does: a lower-index neighbour
// already updated in this sweep, a higher-index one not yet.  The number of levels is the
// longest chain of neighbours in index order; each variable goes to a level between its earliest
// and its latest, and levels are filled up to whole rounds of `quads` updates where the slack
// allows.  Returns the number of levels; slots are level-major, level_start has one more entry.
// graph: the neighbours, made here if it is empty; for a caller that builds levels for more than one kernel.
struct LevelGraph {
    std::vector<int64_t> lower_at, upper_at;   // n + 1 each: where a variable's neighbours start
    std::vector<int32_t> lower, upper;         // neighbours of lower and of higher index that are not fixed, rising
};
int32_t build_levels(const Packed &p, int32_t quads, std::vector<int32_t> &level_start,
                     std::vector<SchedRec> &slots, LevelGraph *graph = nullptr);
// Rounds of the one-wave quad kernel: the levels of 16 (one wavefront of quads), each cut into
// rounds of 16 slots and padded to whole rounds with idle slots (k = -1, no records), and the sweep
// padded with idle rounds to a multiple of kRoundBatch rounds.  Every slot points at its
// variable's incidence records.  Returns the number of levels; n_real counts the variables placed.
constexpr int32_t kRoundQuads = 16;
constexpr int32_t kRoundBatch = 4;
int32_t build_rounds(const Packed &p, std::vector<SchedRec> &rounds, int32_t &n_real);
// Records per lane that the Metropolis / OTM quad kernel reads for one round (a row of up to
// 4 kMoAhead incidences; longer rows take the rest from the incidence records).
constexpr int32_t kMoAhead = 16;
// A round's record as that kernel reads it: meta as in IncRec, and the LDS byte offsets of the
// other factors' values -- 4 n (the state's element n, which holds 1) for an unused place.
struct MoRec {
    uint32_t meta;
    uint32_t zoff[3];
};
// Round-major copy of the rounds' records: record u of lane L (quad L / 4, its record 4 u + L % 4)
// of round r at ((r kMoAhead + u) 64 + L), with zero coefficients past a row and for records with
// more than three other factors (coefficients as int32 when coef32, else int64).  Marks in
// pad[0] of a round's slot whether its row needs the rest read from the incidence records (more
// than 4 kMoAhead records, or a long record).
void build_mo_records(const Packed &p, std::vector<SchedRec> &rounds, bool coef32, std::vector<MoRec> &rec,
                      std::vector<uint8_t> &coef);

// Device view of a packed plan.
struct DevProblem {
    int32_t n;
    int32_t n_terms;
    const VarRec *var;
    const uint32_t *emask;
    const IncRec *inc;       // incidence records, then one zero record at index inc_pad
    const int64_t *inc_coef;
    const int32_t *overflow;
    const int32_t *t_off;
    const int32_t *t_var;
    const int64_t *t_coef;
    int32_t max_other;       // most other factors of any incidence
    int32_t inc_pad;         // index of the zero record (coefficient 0, no factors)
    int32_t coef32;          // every coefficient a_k^(m) fits int32 (coefs_fit_32)
    // dense QUIO form (dense != 0)
    int32_t dense;
    int32_t jbytes;
    int32_t row_stride;
    const void *jd;
    const int64_t *h;
    const int64_t *d;
    const PairRec *pair;     // compact pair records (nullptr when the problem has none)
};

// A run is one launch, or three: the first runs each replica to its end, or hands it over once the replicas
// change few variables, the next sweep's index in e_out (hand_over); the settled kernel (sa_settled.h) takes it
// from there, and the last writes its energy and finishes it where it came unsettled (a schedule that warms up).
// States pass through z_out.
//
// The launches follow one another, so a replica that left the first while another stays there gains nothing
// and may cost its settled sweeps on top: at a constant temperature, where each settles by chance at a sweep of
// its own, runs took up to 2.4 times as long.  So a replica of a plain run leaves only when all that have
// started are settled (two counters in device memory: started, settled; a replica that ends counts in both, and one
// too near its end to leave is not settled until then: pairs, N = 3000, 200 sweeps x 512 reads, optimal transition
// 28.0 ms where some left beside some that stayed, 24.5 now, 24.8 where none leaves).
constexpr int32_t kPhaseWhole = 0, kPhaseFirst = 1, kPhaseLast = 2;
// A replica becomes settled when at most one update in settled_share changed its variable, over settled_every
// sweeps on end, and is no longer with over twice as many; it leaves the settled kernel after three such stretches.
// A settled sweep serves its changes and visits one after another (about 1.1 us each), where the ordinary
// kernel's G waves share the updates.  Share of changes at which the two take the same time, one replica at a
// constant temperature (dense, HUIO, multilinear and pair problems of 26 to 4000 variables): G = 1 0.35 to 0.9,
// but 0.16 to 0.3 where most ask for a visit (the heat bath's draws about two per change, variables without
// cached coefficients); G = 2 0.2 to 0.34; G = 4 0.08 to 0.15; G = 8 0.03 to 0.05.  In the
// dense form (G = 1, no visits), whose ordinary kernel adds every change to the cached sums as well, a settled sweep
// takes at most 1.24 times an ordinary one however much changes, and less up to 0.65 to 0.95: one in two, and no
// replica comes unsettled, as runs some of whose replicas did took both launches' time.  (64 reads at one temperature,
// one in four against one in two: N = 60 binary, 0.37 changes per update, 13.0 and 7.8 ms; N = 100, W = 16, 0.34, 15.0 and
// 10.6.  Cold, then warmer: N = 60, optimal transition, 20.1 and 7.1 ms.)
// The Metropolis / OTM quad kernel (16 updates per round): 0.02 to 0.055, 0.01 for pair problems. (N = 2000 HUIO,
// 300 sweeps x 1024 reads, one in 96, 48 and 40: optimal transition 27.4, 26.5 and 26.0 ms, Metropolis 31.7,
// 29.3 and 28.7.)
constexpr int32_t settled_share_quad(bool pairs) { return pairs ? 112 : 40; }
// Sweeps left that repay forming the caches (N = 2000 HUIO: 1 ms, 7 sweeps of the quad kernel, of whose time a
// settled one saves a third).
constexpr int32_t kSettledRest = 16, kSettledRestQuad = 48;
// Sweeps of some 30 us together: a check takes about 0.5 us, and over few updates the count of changes is
// mostly chance.
constexpr int32_t settled_every(int32_t n_order, int32_t G) {
    int32_t every = 1;
    while (every < 16 && (int64_t)every * n_order < 48 * G) every *= 2;
    return every;
}
constexpr int32_t kSettledEveryQuad = 4;
// Changes in settled_every sweeps up to which a replica becomes settled.
constexpr int32_t settled_limit(int32_t n_order, int32_t every, int32_t share) {
    const int64_t m = ((int64_t)n_order * every + 1) / share;   // (one in two: up, so that twice as many are all)
    return m > 1 ? (int32_t)m : 1;
}
// A sweep's index as it stands in e_out: energies lie within 2^62 of 0 (check_int64_bound).
constexpr int64_t hand_over(int32_t s) { return INT64_MIN + s; }
constexpr bool handed_over(int64_t e) { return e < -((int64_t)1 << 62); }
constexpr int32_t handed_sweep(int64_t e) { return (int32_t)(e - INT64_MIN); }

// Kernel arguments of one annealing launch.
struct AnnealArgs {
    DevProblem P;
    const double *beta;      // S inverse temperatures (device)
    int32_t n_sweeps;        // S
    int32_t s_begin, s_end;  // sweeps to run
    int32_t n_reads;
    int32_t waves_per_group;
    uint32_t key0, key1;     // Philox key (seed)
    uint32_t instance_id;
    double otm_r;            // < 0: r = s/(S-1)
    int32_t otm_enum_max;    // widest range whose optimal transition is found by enumeration
    const SchedRec *sched;   // G * n_win schedule slots (device)
    int32_t n_win;           // windows per sweep
    int32_t win_waves;       // G: waves per replica (1: each wave is an independent replica)
    const int32_t *z_init;   // device, n_reads * n, or nullptr
    int32_t *z_out;          // device, n_reads * n (also the working state when not in LDS)
    int64_t *e_out;          // device, n_reads
    int32_t dense_cache;     // 1: dense form with one wave per replica and the state in LDS keeps the
                             // coefficient cache c1 (int64 per variable) in LDS after the states
    uint64_t *trace;         // device, n_reads * (s_end - s_begin) zeroed words, or nullptr: each
                             // wave adds its share of the state hash's change per sweep (and of the
                             // initial state's hash into the first sweep); a prefix pass then turns
                             // them into the hash after every sweep
    int32_t phase;           // kPhaseWhole, kPhaseFirst or kPhaseLast
    // the settled kernel (order also where phase is kPhaseFirst)
    const SchedRec *order;   // every variable in index order (build_order)
    int32_t n_order;         // those that are not fixed
    int32_t off_c, off_c2, off_m;   // LDS byte offsets of the caches (dense: c1, else ca; cb; margins; the
                                    // dense team's: c1, -, the state); -1: none
    int32_t closed;          // heat bath: closed-form draws
    int32_t exact53;         // energy differences are below 2^52 in magnitude
    int32_t z30;             // every bound of the problem is below 2^30 in magnitude
    int32_t every;           // sweeps between the checks whether a replica has settled, or is no longer
    int32_t limit;           // changes in as many sweeps up to which it becomes settled; past twice as many it is not
    uint32_t *all;           // replicas started and settled (two counters)
};

// Kernel arguments of one launch of the quad kernel (one update per four lanes, dependency levels).
struct QuadArgs {
    DevProblem P;
    const double *beta;          // S inverse temperatures (device)
    int32_t n_sweeps;
    int32_t s_begin, s_end;
    int32_t n_reads;
    uint32_t key0, key1;
    uint32_t instance_id;
    const int32_t *level_start;  // n_levels + 1 offsets into slots (device)
    const SchedRec *slots;       // level-major variables, or n_rounds rounds of kRoundQuads (device)
    int32_t n_levels;
    int32_t n_rounds;            // Metropolis / optimal transition: rounds per sweep (build_rounds)
    const MoRec *mrec;           // Metropolis / optimal transition: the rounds' records (build_mo_records)
    const void *mcoef;           // and their coefficients (int32 when P.coef32, else int64)
    int32_t uniform_width;       // the common width W of every slot, or 0 when widths differ
    double otm_r;                // < 0: r = s/(S-1); else a fixed r (optimal transition)
    const int32_t *z_init;
    int32_t *z_out;
    int64_t *e_out;
    uint64_t *trace;             // as AnnealArgs::trace
    int32_t phase;               // as AnnealArgs::phase
    int32_t limit;               // (over kSettledEveryQuad sweeps)
    uint32_t *all;
};
// Waves of the quad kernel's workgroup (one replica): heat bath, 8 or 16 (below), and Metropolis /
// optimal transition, one (a HUIO level holds about 16 variables, and a single wave needs no
// barrier between levels); the most values per lane it keeps in registers.
constexpr int kQuadWaves = 8;
constexpr int kQuadWavesHigh = 16;
constexpr int kQuadWavesMO = 1;
constexpr int kQuadMaxR = 32;
// Values per lane of the quad heat bath: the smallest class of 8, 16, 26, 32 holding ceil(W / 4)
// (W = 101 takes 26: 104 places).
constexpr int32_t quad_r_class(int32_t max_width) {
    const int32_t c = (max_width + 3) / 4;
    return c <= 8 ? 8 : c <= 16 ? 16 : c <= 26 ? 26 : kQuadMaxR;
}
// The factored weights of linear variables (sa_quad.h): heat bath, one width W for every variable,
// r >= 16 values per lane and at most r / 4 of the quad's 4 r places past the range.
constexpr bool quad_factored(int rule, int32_t r, int32_t uniform_width) {
    return rule == SA_HEAT_BATH && r >= 16 && uniform_width > 0 && 4 * r - uniform_width >= 0 &&
           4 * r - uniform_width <= r / 4;
}
// The heat-bath variants that hold at most 128 VGPRs, so that a workgroup of 16 waves (four per
// SIMD, rounds of 256 updates) fits without spilling: they run 16 waves, the others 8.
constexpr bool quad_high(int rule, int32_t r, int32_t max_exp, bool fact) {
    return rule == SA_HEAT_BATH_CLOSED ? (max_exp <= 1 || r == 8)
                                       : (r == 8 || (fact && (max_exp <= 1 ? r <= 26 : r == 16)));
}
// Waves per replica of the quad kernel for a problem whose widest range is max_width, whose
// exponents are at most max_exp and whose variables all have width uniform_width (0: not one width).
constexpr int quad_waves(int rule, int32_t max_width, int32_t max_exp, int32_t uniform_width) {
    if (rule == SA_METROPOLIS || rule == SA_OPT_METROPOLIS) return kQuadWavesMO;
    const int32_t r = quad_r_class(max_width);
    return quad_high(rule, r, max_exp, quad_factored(rule, r, uniform_width)) ? kQuadWavesHigh : kQuadWaves;
}
// The common width of the variables that are not fixed, or 0 when they differ (or there are none).
int32_t quad_uniform_width(const Packed &p);
// Launches the quad kernel for rule (SA_HEAT_BATH or SA_HEAT_BATH_CLOSED), a problem whose widest
// range is max_width <= 4 * kQuadMaxR and whose exponents are <= max_exp <= 2 (defined in
// sa_kernels_quad.hip).
int launch_quad(int rule, const QuadArgs &a, int32_t max_width, int32_t max_exp, bool narrow, void *stream,
                std::string &err);
// The same for SA_METROPOLIS and SA_OPT_METROPOLIS, exponents <= max_exp <= 4, kQuadWavesMO waves
// (defined in sa_kernels_quad_mo.hip).
int launch_quad_mo(int rule, const QuadArgs &a, int32_t max_width, int32_t max_exp, bool narrow, void *stream,
                   std::string &err);

// One lane's slot of a chunk of the lane kernel (k = -1: idle; h: the linear coefficient), and where a
// chunk's records are: its first row of 64, and its rows (whole fours).
struct LaneSlot {
    int32_t k, lo, width, h;
};
struct LaneRows {
    int32_t first, rows;
};

// Kernel arguments of one launch of the lane kernel (sa_lane.h: heat bath of multilinear pair problems,
// one update per lane over dependency levels).
struct LaneArgs {
    DevProblem P;
    const double *beta;
    int32_t n_sweeps, s_begin, s_end, n_reads;
    uint32_t key0, key1, instance_id;
    int32_t closed;              // closed-form draws of SA_HEAT_BATH_CLOSED
    int32_t n_rounds;
    int32_t off_places;          // LDS byte offset of the waves' places in every round
    const LaneRows *rounds;      // per round: its first chunk and its level's end (~end in a level's last round)
    const LaneRows *chunks;
    const LaneSlot *slots;       // per chunk and lane
    const void *recs;            // rows of 64 records: 16-bit index and coupling, or 32-bit ones
    const int32_t *z_init;
    int32_t *z_out;
    int64_t *e_out;
    uint64_t *trace;             // as AnnealArgs::trace
};
// The same on the host.
struct LaneImage {
    std::vector<int32_t> level_chunk, level_slots;   // per level: its first chunk; its variables
    std::vector<LaneRows> chunks;
    std::vector<LaneSlot> slots;
    std::vector<uint8_t> recs;
    int64_t n_rows = 0;
    int32_t n_levels = 0, n_slots = 0;   // (n_levels 0: none)
    int32_t n_win8 = 0;                  // windows of eight waves (build_schedule)
    bool compact = false;
};
constexpr int kLaneMaxWaves = 8;
constexpr int32_t kLaneReach = 12;   // rows loaded ahead (sa_lane.h, kLaneAhead)
// The rounds of a sweep for `waves` waves per replica (LaneArgs::rounds).
void build_lane_rounds(const LaneImage &im, int waves, std::vector<LaneRows> &rounds);
// Levels and chunks of a problem with compact pair records, and then their records; compact: 16-bit ones.
void build_lane_chunks(const Packed &p, LaneImage &out, LevelGraph *graph = nullptr);
void build_lane_records(const Packed &p, bool compact, LaneImage &im);
// Whether the lane kernel can run `rule` on this packed problem, and whether with 16-bit records.
bool lane_eligible(int rule, const Packed &p, bool coef32, int max_lds, bool &compact);
// Waves per replica from a problem's chunks (0: the automatic choice goes to another kernel); quads: those of
// the quad kernel's workgroup, 0 where it cannot run the problem.
int lane_waves(const LaneImage &im, const Packed &p, bool compact, int32_t n_reads, int32_t quads, int cus, int max_lds);
// LDS bytes of one replica: state, energy parts and the waves' places in n_rounds rounds.
int64_t lane_lds_bytes(int32_t n, int waves, int32_t n_rounds);
int32_t lane_off_places(int32_t n, int waves);
// The lane kernel for a run, or none (waves = 0).
struct LaneChoice {
    int waves = 0;
    bool compact = false;
    int lds_bytes = 0;
};
// A run of fewer sweeps does not repay building and uploading the lane kernel's image.
constexpr int32_t kLaneMinSweeps = 16;
int launch_lane(LaneArgs a, bool compact, int waves, void *stream, std::string &err);

struct LaunchChoice {
    int win_waves = 1;         // waves per replica (window width)
    int waves_per_group = 1;
    int groups = 1;
    int lds_bytes = 0;
    bool state_in_lds = true;
    int reg_chunk = 0;         // heat bath: weights per lane kept in registers (0: recomputed)
    int maxe_class = 1;        // kernel's largest exponent (1, 2, 4 or 16)
    bool narrow = false;       // energy differences in 32-bit arithmetic
    bool dense_cache = false;  // dense form: coefficient cache in LDS (one wave per replica)
    int variant = 0;
};

// The counters of AnnealArgs::all: in the 256 bytes after the order list's, rounded up to 256.
inline uint32_t *settled_counters(const SchedRec *order, int32_t n) {
    return (uint32_t *)((char *)const_cast<SchedRec *>(order) + (((size_t)n * sizeof(SchedRec) + 255) & ~(size_t)255));
}
// The settled kernel's launch for a problem and a run, or none (lds_bytes = 0).
struct SettledChoice {
    int lds_bytes = 0;     // state and caches of one replica
    int off_c = -1, off_c2 = -1, off_m = -1;
};
SettledChoice choose_settled(const Packed &p, bool coef32, int32_t n_reads, int32_t n_order, int32_t n_sweeps, int device);
// Launches it: `a` as for launch_anneal, with order, n_order and leave set.
int launch_settled(int rule, AnnealArgs a, const SettledChoice &sc, int32_t max_width, int32_t max_exp, bool narrow,
                   void *stream, std::string &err);
// Whether a run of the windows with G waves per replica is long enough for two more launches, which cost one of
// 0.5 ms a tenth (N = 24 pairs, G = 4, 90 sweeps 0.47 to 0.52 ms).
constexpr bool settled_pays(int32_t n_sweeps, int32_t n_order, int32_t G) {
    return (int64_t)n_sweeps * n_order >= 1200 * (int64_t)G;
}
inline int32_t settled_share(int32_t G, int rule, const Packed &p) {
    // whether settled sweeps visit most of what may change
    const bool visits = rule == SA_HEAT_BATH || rule == SA_HEAT_BATH_CLOSED || (!p.dense && !p.any_cached);
    return G > 2 ? 6 * G : visits ? 14 : G == 2 ? 10 : p.dense ? 2 : 4;
}
// A run of the one-wavefront-per-update kernels: one launch, or with sc three (a: order, n_order and all set;
// share: settled_share).
int launch_windows(int rule, AnnealArgs a, const LaunchChoice &lc, const SettledChoice &sc, int32_t share, int32_t max_width,
                   int32_t max_exp, bool narrow, void *stream, std::string &err);

// The same for the Metropolis / OTM quad kernel: q as for launch_quad_mo, a as for launch_settled.
int launch_rounds(int rule, QuadArgs q, AnnealArgs a, const SettledChoice &sc, int32_t max_width, int32_t max_exp,
                  bool narrow, void *stream, std::string &err);

// The dense team kernel (sa_dense_team.h) for a run, or none (waves = 0): several waves per replica where
// the row or the range gives each thread two columns or values, with all waves resident at once.  The
// fewest waves (4, 8 or 16) that hold four values and eight columns per thread: every wave repeats a
// draw's scalar part, about a quarter of its instructions, so more of them are slower.
constexpr int kTeamExchangeBytes = 272;
struct TeamChoice {
    int waves = 0;
    bool small = false;    // c1 as int32
    bool exact53 = false;  // energy differences below 2^52
    int off_c = 0, off_z = 0;
    int lds_bytes = 0;
};
struct BatchInst;
struct BatchTask;
TeamChoice choose_team(int rule, const Packed &p, bool coef32, int32_t n_reads, int device);
int launch_dense_team(int rule, AnnealArgs a, const TeamChoice &tc, void *stream, std::string &err);

// Byte layout of a packed instance in one device area, each part 256-byte aligned (the records
// and their coefficients are followed by one zero record).
struct PackedLayout {
    static constexpr int kParts = 12;
    size_t off[kParts];
    size_t total;
};
PackedLayout packed_layout(const Packed &pk);
// Writes the packed instance into a host image of L.total bytes (padding zeroed).
void stage_packed(const Packed &pk, const PackedLayout &L, char *image);
// Points d at the parts of an image copied to device address base.
void bind_packed(const Packed &pk, const PackedLayout &L, char *base, DevProblem &d);

// Launches one annealing pass (defined in sa_kernels.hip).  Returns an SA_* status.
int launch_anneal(int rule, const AnnealArgs &a, const LaunchChoice &lc, void *stream,
                  std::string &err);
// Picks the launch geometry for n_reads replicas of an n-variable problem on `device`.
LaunchChoice choose_launch(int rule, int32_t n, int32_t n_reads, int32_t max_width, int32_t max_exp,
                           int device, int win_waves, bool narrow_ok, int32_t otm_enum_max, bool dense);
// LDS bytes of one replica's state when its G waves share it (state + per-wave energy slots).
int64_t shared_state_bytes(int32_t n, int G);
// Waves of one batch workgroup; a task runs kBatchWaves / G_p reads of problem p.
constexpr int kBatchWaves = 8;

// One problem of a batch as the persistent kernel sees it.
struct BatchInst {
    DevProblem P;
    const double *beta;      // S inverse temperatures (device)
    const SchedRec *sched;   // schedule for `team` waves per replica
    int32_t n_win;
    int32_t team;            // G_p: waves per replica (1, 2, 4 or 8)
    int32_t slot_stride;     // state elements between the teams' LDS slots
    int32_t n_reads;
    int32_t n_sweeps;
    int32_t s_begin, s_end;  // sweeps of this launch (a server chunk, or the whole schedule)
    int32_t resume;          // 1: start from the states in z_out and energies in e_out (an earlier chunk's)
    int32_t rule;
    uint32_t key0, key1, instance_id;
    int32_t *z_out;          // n_reads x n (device)
    int64_t *e_out;          // n_reads (device)
    // settled sweeps (as AnnealArgs); next == nullptr: none
    int32_t *next;           // n_reads: the next sweep s, or ~s of a settled replica (device)
    const SchedRec *order;
    int32_t n_order, off_c, off_c2, off_m, z30, every, limit;
    int32_t team_waves;      // > 0: run by the dense team kernel (off_c: c1, off_m: the state; exact53 as AnnealArgs)
    int32_t exact53;
};
struct BatchTask {
    int32_t inst;
    int32_t read;            // first read of the task (kBatchWaves / G_p reads)
};
struct BatchArgs {
    const BatchInst *insts;
    const BatchTask *tasks;  // ordered longest first
    int32_t n_tasks;
    uint32_t *counter;       // next task (device)
    int32_t lds_words;       // dynamic LDS of a workgroup, 32-bit words
    int32_t parts_words;     // offset of the waves' energy parts (kBatchWaves int64)
    int32_t phase;           // as AnnealArgs::phase; a problem with next == nullptr is run whole by the first
    int32_t sweep_limit;     // > 0: only the first sweep_limit sweeps (autotuning trials)
};
// One launch of the settled kernel over tasks first .. first + n - 1 of a list, each with lds_bytes of
// LDS: the replicas of a batch in three groups by what their caches take (up to 10, 40 and 160 KB, that
// is 16, 4 and 1 replicas per compute unit), the widest first, each longest first.
struct SettledGroup {
    int32_t first = 0, n = 0;
    int lds_bytes = 0;
};
constexpr int kSettledGroups = 3;
// One launch of the dense team kernel over tasks of the same list: problems of one rule and team size.
struct TeamGroup {
    int32_t first = 0, n = 0;
    int rule = 0, waves = 0, lds_bytes = 0;
    bool small = false;
};
// The groups and their task list, for problems whose replicas take lds[i] bytes (0: not settled) and cost[i].
void settle_batch(const std::vector<BatchInst> &insts, const std::vector<int> &lds, const std::vector<double> &cost,
                  std::vector<BatchTask> &tasks, SettledGroup (&groups)[kSettledGroups]);
int launch_settled_batch(const BatchInst *insts, const BatchTask *tasks, int32_t n_tasks, int lds_bytes, int maxe_class,
                         void *stream, std::string &err);
// Fills a problem's settled fields (next is the caller's) for teams of `team` waves; returns its LDS bytes, or 0.
int settle_inst(const Packed &p, bool coef32, const SchedRec *order, int32_t n_order, int32_t n_sweeps, int device,
                BatchInst &d);
// Gives a dense problem of a batch to the team kernel if choose_team does; returns the choice.
TeamChoice team_inst(int rule, const Packed &p, bool coef32, const SchedRec *order, int32_t n_reads, int device, BatchInst &d);
// Appends the tasks of the problems run by the team kernel (choices[i].waves > 0) and returns their groups.
void group_teams(const std::vector<BatchInst> &insts, const std::vector<TeamChoice> &choices, std::vector<BatchTask> &tasks,
                 std::vector<TeamGroup> &groups);
int launch_team_group(const BatchInst *insts, const BatchTask *tasks, const TeamGroup &g, void *stream, std::string &err);
// One launch of the lane kernel over tasks of the same list: problems of one width of records and team.
struct LaneGroup {
    int32_t first = 0, n = 0;
    int waves = 0, lds_bytes = 0;
    bool compact = false;
};
void group_lanes(const std::vector<LaneChoice> &choices, const std::vector<int32_t> &n_reads, std::vector<BatchTask> &tasks,
                 std::vector<LaneGroup> &groups);
int launch_lane_group(const LaneArgs *list, const BatchTask *tasks, const LaneGroup &g, void *stream, std::string &err);
// A stream beside a batch's, with the events that fork it from there and join it again (hipStream_t,
// hipEvent_t; nullptr: none, its work runs on the batch's stream).
struct SideStream {
    void *stream = nullptr, *fork = nullptr, *join = nullptr;
    int create();                       // hipError_t
    void destroy();
    int fork_from(void *main) const;    // the side stream's next work waits for main's so far
    int mark() const;                   // the end of the side stream's work so far ...
    int join_to(void *main) const;      // ... which main's next work waits for
};
struct BatchLaunch {
    std::vector<LaneGroup> lanes;
    const LaneArgs *lane_args = nullptr;        // device: per problem
    SettledGroup settled[kSettledGroups];
    std::vector<TeamGroup> teams;
    const BatchTask *settled_tasks = nullptr;   // device: the groups' tasks
    // the dense team and lane kernels run beside the persistent kernel (without a side stream: first);
    // their problems get no task of the persistent kernel
    SideStream beside;
    // the settled groups run beside each other: the first on the batch's stream, the others here
    SideStream settled_side;
    int waves_per_group = kBatchWaves;
    int groups = 1;
    int maxe_class = 1;
    bool narrow = false;
    bool z16 = false;        // states held as int16 in LDS (every bound within int16)
};
// Queues the counter reset and the persistent kernel, and with settled groups their kernels and the
// persistent kernel again (all plain kernel launches).
int launch_batch(const BatchArgs &b, const BatchLaunch &bl, void *stream, std::string &err);

// Zeroes n words of device memory with a kernel (no memset node, so the work may be captured).
int launch_zero_u64(uint64_t *p, int64_t n, void *stream, std::string &err);
// Turns per-sweep hash changes into the hash after each sweep: row r of `trace` (n_reads rows of
// n_cols) becomes its own inclusive prefix sum.
int launch_trace_prefix(uint64_t *trace, int32_t n_reads, int32_t n_cols, void *stream, std::string &err);

// Energies of n_states device-resident states (one wavefront per state).
int launch_energy(const DevProblem &P, const int32_t *states, int32_t n_states, int64_t *out,
                  void *stream, std::string &err);

}  // namespace sa
