// gfx950 kernels of parallel flatPERM (Campbell & Janse van Rensburg,
// "Parallel PERM"): Rosenbluth growth with a_+ occupancy scans (Sec. 1,
// eqns (1)-(2)), flatPERM prune/enrich against the running averages (Sec. 2,
// eqn (6)), accumulation of the sample sums (eqn (4)), and the merge of the
// per-sequence sums into the pooled sums of Algorithm 2 (Sec. 3, Fig. 1).
//
// Execution model.  The default growth kernel (batch_kernel) is persistent:
// one 64-lane wavefront takes one (problem, sequence) item at a time from a
// device queue and runs that sequence's tours; every walk quantity is uniform
// over the wave, and the lanes split the parallel parts of a step:
//   - the occupancy scan: lane (dir, o) reads the slot that neighbour dir has in
//     subtable o of the walk's table, so all neighbours are looked up in all
//     their places in one LDS instruction and resolved with two wave ballots;
//   - the random numbers: lane i computes the Philox4x32-10 block of event
//     k0+i-1, so one pass of the multiplies serves 63 events;
//   - the LIFO deletion of abandoned sites after a backtrack.
// The walk's occupancy table (one key per site, restored exactly by LIFO
// deletion through remembered slot ids), the slot ids and the sequence's own
// per-length sums live in LDS (the sums in global memory for long walks); the
// 64 most recent pending copies live in the lanes of a few vector registers.  A
// second kernel (run_kernel) packs 64/TS walks into a wave as teams of TS lanes.
//
// Determinism.  Every floating-point decision uses the same IEEE operations
// in the same order as the reading of the method these kernels implement
// (no contraction: the library is built with -ffp-contract=off), and the
// random numbers are a pure function of (seed, sequence, tour, event).  The
// launch shape therefore never changes a result.
#include <mutex>

#include "pperm_internal.h"

namespace pperm {
namespace {

// ---------------------------------------------------------------------------
// Philox4x32-10 (Salmon et al., SC'11): 10 rounds, Weyl key schedule.
// ---------------------------------------------------------------------------
constexpr uint32_t PHX_M0 = 0xD2511F53u;
constexpr uint32_t PHX_M1 = 0xCD9E8D57u;
constexpr uint32_t PHX_W0 = 0x9E3779B9u;
constexpr uint32_t PHX_W1 = 0xBB67AE85u;

__device__ __forceinline__ uint4 philox10(uint4 c, uint32_t k0, uint32_t k1) {
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const uint32_t lo0 = PHX_M0 * c.x, hi0 = __umulhi(PHX_M0, c.x);
        const uint32_t lo1 = PHX_M1 * c.z, hi1 = __umulhi(PHX_M1, c.z);
        c = make_uint4(hi1 ^ c.y ^ k0, lo1, hi0 ^ c.w ^ k1, lo0);
        k0 += PHX_W0;
        k1 += PHX_W1;
    }
    return c;
}

// ---------------------------------------------------------------------------
// Extended-range weights: x = m * 2^e, m in [0.5, 1) (m = 0, e = 0 for zero).
// Every operation is the correctly rounded result of the exact operation on
// the represented values (frexp and ldexp by at most 63 binades are exact),
// so weights of any size are carried without underflow or overflow.
// ---------------------------------------------------------------------------
struct XF {
    double m;
    int e;
};

__device__ __forceinline__ XF xf_norm(double x, int e) {
    const double m = __builtin_amdgcn_frexp_mant(x);
    const int k = __builtin_amdgcn_frexp_exp(x);
    XF r;
    r.m = m;
    r.e = (m == 0.0) ? 0 : e + k;
    return r;
}

// Written with selects only (no branches): the operand with the larger
// exponent keeps its scale, the other is shifted onto it.  The shift is exact
// while the shifted mantissa stays normal; once it has moved 54 or more
// binades it is below half an ulp of the kept mantissa (which lies in
// [0.5, 1)), so the rounded sum is the kept mantissa whatever it became --
// the same as dropping it, which is how the exact operation is usually
// written (a shift beyond 63 binades is dropped).
__device__ __forceinline__ XF xf_add(XF a, XF b) {
    const bool sw = a.e < b.e;
    const double hm = sw ? b.m : a.m;
    const int he = sw ? b.e : a.e;
    const double lm = sw ? a.m : b.m;
    const int le = sw ? a.e : b.e;
    const int d = he - le;
    const double ls = ldexp(lm, -d);
    XF r = xf_norm(hm + ls, he);
    // zero operands (field by field, so that no struct is selected by address)
    const bool az = (a.m == 0.0), bz = (b.m == 0.0);
    r.m = az ? b.m : (bz ? a.m : r.m);
    r.e = az ? b.e : (bz ? a.e : r.e);
    return r;
}

__device__ __forceinline__ XF xf_mul(XF a, double k) { return xf_norm(a.m * k, a.e); }
__device__ __forceinline__ XF xf_div(XF a, double k) { return xf_norm(a.m / k, a.e); }

// a / b as an ordinary double, exponent gap clamped to [-1000, 1000].
__device__ __forceinline__ double xf_ratio(XF a, XF b) {
    const int d = a.e - b.e;
    const int dc = d < -1000 ? -1000 : (d > 1000 ? 1000 : d);
    double r = ldexp(a.m / b.m, dc);
    r = (d > 1000) ? 0x1p1000 : r;
    r = (d < -1000 || a.m == 0.0) ? 0.0 : r;
    return r;
}

// The same operations where an operand is known to be nonzero (every walk
// weight and every sum that includes one): they give the same result as the
// general ones on such operands, with the zero cases left out.
__device__ __forceinline__ XF xf_norm_nz(double x, int e) {
    XF r;
    r.m = __builtin_amdgcn_frexp_mant(x);
    r.e = e + __builtin_amdgcn_frexp_exp(x);
    return r;
}

// a + b for b != 0: both mantissas are brought to the larger exponent (the
// larger operand's by an exact shift of 0, the other's as in xf_add) and
// added, so no operand swap is needed.  A zero a counts as having the
// smallest exponent: shifted away, its mantissa 0 leaves exactly b.
__device__ __forceinline__ XF xf_add_nz(XF a, XF b) {
    const int ae = (a.m == 0.0) ? -0x40000000 : a.e;
    const int he = ae > b.e ? ae : b.e;
    return xf_norm_nz(ldexp(a.m, ae - he) + ldexp(b.m, b.e - he), he);
}

// x / y, correctly rounded, for operands whose quotient and reciprocal are
// far from the ends of the FP64 range.  Markstein's method: the hardware
// reciprocal refined by two Newton-Raphson steps with fused multiply-adds, the
// quotient x * y, and one correction with the exact residual x - y q.  It is
// the general IEEE division sequence without its operand scaling and
// special-case fix-up, which leave such operands and their quotient unchanged.
__device__ __forceinline__ double recip_normal(double y) {
    double r = __builtin_amdgcn_rcp(y);
    double e = __builtin_fma(-y, r, 1.0);
    r = __builtin_fma(r, e, r);
    e = __builtin_fma(-y, r, 1.0);
    return __builtin_fma(r, e, r);
}
// x / y given r = recip_normal(y)
__device__ __forceinline__ double div_by(double x, double y, double r) {
    const double q = x * r;
    const double res = __builtin_fma(-y, q, x);
    return __builtin_fma(res, r, q);
}
__device__ __forceinline__ double div_normal(double x, double y) { return div_by(x, y, recip_normal(y)); }

__device__ __forceinline__ XF xf_mul_nz(XF a, double k) { return xf_norm_nz(a.m * k, a.e); }
// a / k for an integer 2 <= k < 2^34
__device__ __forceinline__ XF xf_div_nz(XF a, double k) { return xf_norm_nz(div_normal(a.m, k), a.e); }

// a / b for a, b != 0 whose ratio is below 2^34 (a decision's W * seen over a
// sum that includes N copies of W, see walk_sequence): the exponent gap is at
// most 35, so of the general clamp to [-1000, 1000] only the lower end can act.
__device__ __forceinline__ double xf_ratio_nz(XF a, XF b) {
    const int d = a.e - b.e;
    const double r = ldexp(div_normal(a.m, b.m), d < -1000 ? -1000 : d);
    return (d < -1000) ? 0.0 : r;
}

__device__ __forceinline__ XF xf_of(const SumRec& r) { return XF{r.m, r.e}; }

// ---------------------------------------------------------------------------
// Lattice: packed int16 coordinates (offset by 2^15 so that key 0 never
// occurs and marks an empty slot), direction order +x,-x,+y,-y,+z,-z.
// ---------------------------------------------------------------------------
template <int D> struct Lat;
template <> struct Lat<2> {
    using Key = uint32_t;
    static constexpr int DP = 4;  // direction lanes per probe window
    __device__ static Key pack(int x, int y, int) {
        return (uint32_t)(x + 32768) | ((uint32_t)(y + 32768) << 16);
    }
    __device__ static void unpack(Key k, int& x, int& y, int& z) {
        x = (int)(k & 0xFFFFu) - 32768;
        y = (int)(k >> 16) - 32768;
        z = 0;
    }
    __device__ static uint32_t hash(Key k) { return k * 0x9E3779B1u; }
};
template <> struct Lat<3> {
    using Key = uint64_t;
    static constexpr int DP = 8;
    __device__ static Key pack(int x, int y, int z) {
        return (uint64_t)(uint32_t)(x + 32768) | ((uint64_t)(uint32_t)(y + 32768) << 16) |
               ((uint64_t)(uint32_t)(z + 32768) << 32);
    }
    __device__ static void unpack(Key k, int& x, int& y, int& z) {
        x = (int)(k & 0xFFFFu) - 32768;
        y = (int)((k >> 16) & 0xFFFFu) - 32768;
        z = (int)((k >> 32) & 0xFFFFu) - 32768;
    }
    __device__ static uint32_t hash(Key k) {
        return (uint32_t)k * 0x9E3779B1u + (uint32_t)(k >> 32) * 0x85EBCA77u;
    }
};

__device__ __forceinline__ int dir_dx(int d) { return (d == 0) - (d == 1); }
__device__ __forceinline__ int dir_dy(int d) { return (d == 2) - (d == 3); }
__device__ __forceinline__ int dir_dz(int d) { return (d == 4) - (d == 5); }

__device__ __forceinline__ void wave_fence() {
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Every lambda of the walker belongs in its caller: one left as a call would
// keep what it captures in memory.
#define INLINE __attribute__((always_inline))

// Compile-time switches of a generic lambda.
struct yes { static constexpr bool value = true; };
struct no { static constexpr bool value = false; };

// Team phases.
enum : int { PH_NEED_SEQ = 0, PH_NEED_TOUR = 1, PH_NEED_BT = 2, PH_AT_NODE = 3, PH_DONE = 4,
             PH_ABORT = 5 };

// Trajectory digest of a sequence (instrumentation, not part of the method):
// FNV-1a 32 over one byte per growth step, dir | a_+ << 3, kept zero-extended
// in a 64-bit statistics word.
constexpr uint32_t FNV_OFFSET = 2166136261u;
constexpr uint32_t FNV_PRIME = 16777619u;

// Bits 0, DP, 2*DP, ... (W of them): the lanes of one direction in a team.
template <int DP, int W>
__device__ __forceinline__ uint64_t dir_rep() {
    uint64_t r = 0;
#pragma unroll
    for (int j = 0; j < W; ++j) r |= 1ull << (j * DP);
    return r;
}

// Fold a team-local lane mask (TS bits) onto direction bits (DP bits).
template <int TS, int DP>
__device__ __forceinline__ uint32_t fold_dirs(uint64_t x) {
#pragma unroll
    for (int s = TS / 2; s >= DP; s /= 2) x |= x >> s;
    return (uint32_t)(x & ((1u << DP) - 1u));
}

template <int D, int TS>
__global__ void __launch_bounds__(64) run_kernel(RunArgs A) {
    using L_ = Lat<D>;
    using Key = typename L_::Key;
    constexpr int DP = L_::DP;
    static_assert(TS >= DP && TS <= 64 && (TS & (TS - 1)) == 0, "team size");
    constexpr int W = TS / DP;          // probe positions per direction per round
    constexpr int TPW = 64 / TS;        // teams per wave

    extern __shared__ __align__(16) unsigned char lds[];
    const int lane = (int)threadIdx.x;
    const int lt = lane & (TS - 1);
    const int tbase = lane & ~(TS - 1);
    const int tiw = lane / TS;
    const uint32_t team_slot = blockIdx.x * TPW + tiw;

    Key* table = reinterpret_cast<Key*>(lds + (size_t)tiw * A.lds_team_bytes);
    uint16_t* sid = reinterpret_cast<uint16_t*>(lds + (size_t)tiw * A.lds_team_bytes +
                                                (sizeof(Key) << A.slots_log2));
    const uint32_t S = 1u << A.slots_log2;
    const uint32_t smask = S - 1u;
    const uint32_t hshift = 32u - A.slots_log2;

    // probe-lane role
    const int pdir = lt % DP;
    const int poff = lt / DP;
    const bool pvalid = pdir < 2 * D;
    const int pdx = dir_dx(pdir), pdy = dir_dy(pdir), pdz = dir_dz(pdir);
    const uint64_t same_dir = dir_rep<DP, W>() << (tbase + pdir);
    const uint64_t below = (lane == 0) ? 0ull : ((~0ull) >> (64 - lane));
    const uint64_t same_dir_below = same_dir & below;

    const uint32_t n_max = A.n_max;
    const uint32_t row = A.row;
    const bool shared_mode = (A.mode == MODE_SHARED);
    const bool control_mode = (A.mode != MODE_ROSENBLUTH);
    // in Algorithm 2 a sequence's own epoch data stands for the pool's: weight N
    const double pool = shared_mode ? (double)A.N : 1.0;
    const uint64_t pool_u = shared_mode ? (uint64_t)A.N : 1ull;
    const uint32_t cap = A.step_cap;

    // empty table with the origin in it; slot id of site 0
    for (uint32_t i = (uint32_t)lt; i < S; i += TS) table[i] = (Key)0;
    wave_fence();
    const Key origin_key = L_::pack(0, 0, 0);
    if (lt == 0) {
        const uint32_t h = L_::hash(origin_key) >> hshift;
        table[h] = origin_key;
        sid[0] = (uint16_t)h;
    }
    wave_fence();

    StackEntry* stk = A.stack + (size_t)team_slot * n_max;

    // ---- team state (identical in every lane of a team) ----
    int phase = PH_NEED_SEQ;
    uint32_t s = 0, tours_left = 0, m = 0;
    uint64_t t = 0, tt = 0;
    SumRec rec0 = {0.0, 0, 0u};           // L[s][0]: one record per tour
    const SumRec* Grow = A.G;
    uint64_t MGs = 0;
    uint64_t st_steps = 0, st_events = 0, st_enrich = 0, st_copies = 0, st_prunes = 0,
             st_traps = 0, st_tours = 0, st_maxd = 0, st_digest = 0, st_capped = 0;
    uint32_t steps_call = 0;

    uint32_t n = 0;
    XF w = {0.5, 1};
    int ex = 0, ey = 0, ez = 0;
    bool control = false;
    uint64_t k = 0, kb = 0;
    bool stale = true;
    uint4 rb = make_uint4(0, 0, 0, 0);

    uint32_t sp = 0, top_n = 0, top_rem = 0;
    XF top_w = {0.0, 0};

    SumRec Lp = {0.0, 0, 0u}, Gp = {0.0, 0, 0u};   // records of length n + 1 (prefetched)
    XF Lc = {0.0, 0}, Gc = {0.0, 0};               // sums at length n after its record

    for (;;) {
        // ---------------- (1) acquire a sequence ----------------
        const bool need_seq = (phase == PH_NEED_SEQ);
        uint32_t got = 0xFFFFFFFFu;
        if (need_seq && lt == 0) got = atomicAdd(&A.ctrl[CTRL_QUEUE], 1u);
        got = __shfl(got, tbase, 64);
        if (need_seq) {
            if (got < A.N) {
                s = got;
                const size_t rb0 = (size_t)s * row;
                t = A.t[s];
                m = A.m[s];
                rec0 = A.L[rb0];
                const uint64_t* sr = A.stats + (size_t)s * STATS_WORDS;
                st_steps = sr[ST_STEPS]; st_events = sr[ST_EVENTS]; st_enrich = sr[ST_ENRICH];
                st_copies = sr[ST_COPIES]; st_prunes = sr[ST_PRUNES]; st_traps = sr[ST_TRAPS];
                st_tours = sr[ST_TOURS]; st_maxd = sr[ST_MAXDEPTH]; st_digest = sr[ST_DIGEST];
                st_capped = sr[ST_CAPPED];
                Grow = A.G + (size_t)pooled_row(A.mode, s) * row;
                MGs = A.MG[pooled_row(A.mode, s)];
                tours_left = A.tours;
                steps_call = 0;
                phase = PH_NEED_TOUR;
            } else {
                phase = PH_DONE;
            }
        }
        if (__ballot(phase != PH_DONE) == 0ull) break;

        SumRec* Lrow = A.L + (size_t)s * row;

        // ---------------- (2) backtrack / end of tour ----------------
        if (phase == PH_NEED_BT || phase == PH_ABORT) {
            const bool abort = (phase == PH_ABORT);
            const bool tour_end = abort || sp == 0;
            uint32_t rn = 0;
            if (!tour_end) {
                rn = top_n;
                w = top_w;
                top_rem -= 1;
                if (top_rem == 0) {
                    sp -= 1;
                    if (sp > 0) {
                        const StackEntry e = stk[sp - 1];
                        top_n = e.n;
                        top_rem = e.remaining;
                        top_w = XF{e.m, e.e};
                    }
                }
            }
            // LIFO deletion of sites rn+1..n restores the table exactly
            for (uint32_t i = rn + 1 + (uint32_t)lt; i <= n; i += TS) table[sid[i]] = (Key)0;
            if (!tour_end) {
                const Key ek = table[sid[rn]];
                L_::unpack(ek, ex, ey, ez);
                n = rn;
                control = false;
                phase = PH_AT_NODE;
                Lp = Lrow[n + 1];
                Gp = Grow[n + 1];
            } else {
                n = 0;
                ex = ey = ez = 0;
                sp = 0;
                if (abort) {
                    st_capped = 1;
                    tours_left = 0;
                    if (lt == 0) atomicOr(&A.ctrl[CTRL_ERR], ERR_CAP);
                } else {
                    tours_left -= 1;
                }
                if (tours_left > 0) {
                    phase = PH_NEED_TOUR;
                } else {
                    if (lt == 0) {
                        const size_t rb0 = (size_t)s * row;
                        A.L[rb0] = rec0;
                        A.t[s] = t;
                        A.m[s] = m;
                        uint64_t* sr = A.stats + (size_t)s * STATS_WORDS;
                        sr[ST_STEPS] = st_steps; sr[ST_EVENTS] = st_events; sr[ST_ENRICH] = st_enrich;
                        sr[ST_COPIES] = st_copies; sr[ST_PRUNES] = st_prunes; sr[ST_TRAPS] = st_traps;
                        sr[ST_TOURS] = st_tours; sr[ST_MAXDEPTH] = st_maxd; sr[ST_DIGEST] = st_digest;
                        sr[ST_CAPPED] = st_capped;
                    }
                    phase = PH_NEED_SEQ;
                }
            }
        }

        // ---------------- (3) start of a tour ----------------
        if (phase == PH_NEED_TOUR) {
            tt = t;
            t += 1;
            m += 1;
            st_tours += 1;
            w = XF{0.5, 1};                       // W_0 = 1
            {
                const XF r0 = xf_add(xf_of(rec0), w);
                rec0.m = r0.m;
                rec0.e = r0.e;
                rec0.h += 1u;
            }
            k = 0;
            stale = true;
            n = 0;
            ex = ey = ez = 0;
            control = false;
            phase = PH_AT_NODE;
            Lp = Lrow[1];
            Gp = Grow[1];
        }
        wave_fence();

        // ---------------- (4) occupancy scan at the endpoint ----------------
        const bool probing = (phase == PH_AT_NODE);
        const Key nk = L_::pack(ex + pdx, ey + pdy, ez + pdz);
        const uint32_t home = L_::hash(nk) >> hshift;
        bool open = probing && pvalid;
        uint32_t freem = 0;
        int my_ins = -1;
        uint32_t pos = home + (uint32_t)poff;
        for (;;) {
            if (__ballot(open) == 0ull) break;
            bool hit = false, emp = false;
            uint32_t slot = 0;
            if (open) {
                slot = pos & smask;
                const Key v = table[slot];
                hit = (v == nk);
                emp = (v == (Key)0);
            }
            const bool res = hit || emp;
            const uint64_t bres = __ballot(res);
            const bool first = res && ((bres & same_dir_below) == 0ull);
            const uint64_t bfe = __ballot(first && emp);
            const uint64_t bfr = __ballot(first);
            const uint64_t tmaskl = (TS == 64) ? ~0ull : ((1ull << TS) - 1ull);
            freem |= fold_dirs<TS, DP>((bfe >> tbase) & tmaskl);
            const uint32_t done_dirs = fold_dirs<TS, DP>((bfr >> tbase) & tmaskl);
            if (first && emp) my_ins = (int)slot;
            if ((done_dirs >> pdir) & 1u) open = false;
            pos += W;
        }
        const uint32_t a = (uint32_t)__popc(freem);
        if (probing && a == 0) {
            st_traps += 1;
            phase = PH_NEED_BT;
        }

        // ---------------- (5) random blocks ----------------
        const bool growing = (phase == PH_AT_NODE);
        if (__ballot(growing && (stale || (k - kb) >= (uint64_t)TS)) != 0ull) {
            kb = k;
            stale = false;
            const uint64_t kk = kb + (uint64_t)lt;
            rb = philox10(make_uint4((uint32_t)kk, (uint32_t)(kk >> 32), (uint32_t)tt, s), A.key0,
                          A.key1);
        }
        const int src = tbase + (int)((uint32_t)(k - kb) & (uint32_t)(TS - 1));
        const uint32_t B0 = __shfl(rb.x, src, 64);
        const uint32_t B1 = __shfl(rb.y, src, 64);
        const uint32_t B2 = __shfl(rb.z, src, 64);

        // ---------------- (6) decision, growth, record ----------------
        if (growing) {
            k += 1;
            st_events += 1;
            bool pruned = false;
            if (control) {
                // eqn (6): r = W / [W_n], [W_n] = sum / seen with the sequence's
                // own epoch data weighted N; evaluated as (W * seen) / sum
                const XF sum = xf_add(Gc, xf_mul(Lc, pool));
                const double seen = (double)(MGs + pool_u * (uint64_t)m);
                const double r = xf_ratio(xf_mul(w, seen), sum);
                const double u = ((double)(B1 >> 5) * 67108864.0 + (double)(B2 >> 6)) *
                                 (1.0 / 9007199254740992.0);
                if (r >= 1.0) {
                    const double f = floor(r);
                    double c;
                    if (r != f && u < (f + 1.0) - r) c = f;
                    else c = (r == f) ? f : f + 1.0;
                    w = xf_div(w, c);
                    if (c > 1.0) {
                        const uint32_t ci = (uint32_t)c;
                        if (sp > 0) {
                            // every lane of the team stores (and later reloads) the
                            // entry, so each lane only ever reads its own writes
                            StackEntry e;
                            e.n = top_n;
                            e.remaining = top_rem;
                            e.e = top_w.e;
                            e.pad0 = 0u;
                            e.m = top_w.m;
                            e.key = 0ull;
                            stk[sp - 1] = e;
                        }
                        top_n = n;
                        top_rem = ci - 1u;
                        top_w = w;
                        sp += 1;
                        if ((uint64_t)sp > st_maxd) st_maxd = sp;
                        st_enrich += 1;
                        st_copies += (uint64_t)(ci - 1u);
                    }
                } else {
                    // a survivor takes W / r, the running average itself
                    if (u < r) w = xf_div(sum, seen);
                    else pruned = true;
                }
            }
            if (pruned) {
                st_prunes += 1;
                phase = PH_NEED_BT;
            } else {
                const uint32_t j = __umulhi(B0, a);
                uint32_t mm = freem;
                for (uint32_t i = 0; i < j; ++i) mm &= mm - 1u;
                const int dir = __ffs(mm) - 1;
                st_digest = (uint64_t)(((uint32_t)st_digest ^ ((uint32_t)dir | (a << 3))) * FNV_PRIME);
                if (my_ins >= 0 && pdir == dir) {
                    table[my_ins] = nk;
                    sid[n + 1] = (uint16_t)my_ins;
                }
                ex += dir_dx(dir);
                ey += dir_dy(dir);
                ez += dir_dz(dir);
                w = xf_mul(w, (double)a);      // W *= a_+, eqn (2)
                if (w.e > EXP_LIMIT || w.e < -EXP_LIMIT) {
                    if (lt == 0) atomicOr(&A.ctrl[CTRL_ERR], ERR_RANGE);
                }
                n += 1;
                st_steps += 1;
                steps_call += 1;
                // arrival: record into the running sums (eqn (4))
                const XF Lnew = xf_add(xf_of(Lp), w);
                SumRec nr;
                nr.m = Lnew.m;
                nr.e = Lnew.e;
                nr.h = Lp.h + 1u;
                Lrow[n] = nr;
                Lc = Lnew;
                Gc = xf_of(Gp);
                if (cap != 0u && steps_call >= cap) {
                    phase = PH_ABORT;
                } else if (n == n_max) {
                    phase = PH_NEED_BT;
                } else {
                    control = control_mode;
                    Lp = Lrow[n + 1];
                    Gp = Grow[n + 1];
                }
            }
        }
        wave_fence();
    }
}

// ---------------------------------------------------------------------------
// Wave-per-walk growth kernel.  One 64-lane wavefront owns one walk, so every
// quantity of the walk is uniform across the wave and every branch is a
// scalar branch; the lanes only split the occupancy scan (lane = dir * W + o
// reads neighbour dir's slot in subtable o), the Philox blocks (lane i holds
// the block of event kb + i - 1, fetched with readlane) and the LIFO deletions.
// The sequence's own per-length sums live in LDS while its tours run (no
// global round trip on the record / decision path), the pooled sums are loaded
// a step ahead, and each pending-copy entry carries its endpoint site, so a
// backtrack needs no table lookup to restore the walk's end.
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint32_t ufirst(uint32_t v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ uint64_t ufirst64(uint64_t v) {
    return ((uint64_t)ufirst((uint32_t)(v >> 32)) << 32) | (uint64_t)ufirst((uint32_t)v);
}
__device__ __forceinline__ bool ubool(bool b) { return ufirst(b ? 1u : 0u) != 0u; }
// v of lane l (the builtin returns a signed int: convert through uint32_t so
// that the low word of a 64-bit value is never sign-extended)
__device__ __forceinline__ uint32_t lane_value(uint32_t v, uint32_t l) {
    return (uint32_t)__builtin_amdgcn_readlane((int)v, l);
}
__device__ __forceinline__ uint64_t lane_value(uint64_t v, uint32_t l) {
    return ((uint64_t)lane_value((uint32_t)(v >> 32), l) << 32) | (uint64_t)lane_value((uint32_t)v, l);
}
__device__ __forceinline__ double lane_value(double v, uint32_t l) {
    return __builtin_bit_cast(double, lane_value(__builtin_bit_cast(uint64_t, v), l));
}

// Address-space views.  A problem's descriptor is never written while a growth
// launch runs, so it is read through the constant space (scalar loads, whose
// values the compiler knows to be the same in all lanes); sums and the copy
// stack are ordinary global memory.
template <typename T>
__device__ __forceinline__ const __attribute__((address_space(4))) T* as_const(const T* p) {
    return (const __attribute__((address_space(4))) T*)p;
}
template <typename T>
__device__ __forceinline__ __attribute__((address_space(1))) T* as_global(T* p) {
    return (__attribute__((address_space(1))) T*)p;
}

// Whole-record moves through those spaces, one 32-bit word at a time (the
// compiler merges them into wide loads and stores).
template <typename T>
__device__ __forceinline__ T load_const(const T* p) {
    static_assert(sizeof(T) % 4 == 0, "word-sized record");
    T r;
    const __attribute__((address_space(4))) uint32_t* q = (const __attribute__((address_space(4))) uint32_t*)p;
    uint32_t* d = reinterpret_cast<uint32_t*>(&r);
#pragma unroll
    for (size_t i = 0; i < sizeof(T) / 4; ++i) d[i] = q[i];
    return r;
}
template <typename T>
__device__ __forceinline__ T load_global(const T* p) {
    static_assert(sizeof(T) % 4 == 0, "word-sized record");
    T r;
    const __attribute__((address_space(1))) uint32_t* q = (const __attribute__((address_space(1))) uint32_t*)p;
    uint32_t* d = reinterpret_cast<uint32_t*>(&r);
#pragma unroll
    for (size_t i = 0; i < sizeof(T) / 4; ++i) d[i] = q[i];
    return r;
}
template <typename T>
__device__ __forceinline__ void store_global(T* p, const T& v) {
    static_assert(sizeof(T) % 4 == 0, "word-sized record");
    __attribute__((address_space(1))) uint32_t* q = (__attribute__((address_space(1))) uint32_t*)p;
    const uint32_t* d = reinterpret_cast<const uint32_t*>(&v);
#pragma unroll
    for (size_t i = 0; i < sizeof(T) / 4; ++i) q[i] = d[i];
}

// ---------------------------------------------------------------------------
// Memory that waves of one launch hand to each other (the chained launch).  The
// eight XCDs have an L2 each, and a fence at agent scope writes back or
// invalidates all of one, so what is handed over is written and read past the
// L2 instead (relaxed atomics at agent scope, which need no fence), and a wave
// announces its writes once they have arrived.
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint64_t shared_load(const uint64_t* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint32_t shared_load(const uint32_t* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void shared_store(uint64_t* p, uint64_t v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void shared_store(uint32_t* p, uint32_t v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Records and stack entries, 64 bits at a time.
template <typename T>
__device__ __forceinline__ T shared_load_as(const T* p) {
    static_assert(sizeof(T) % 8 == 0, "whole 64-bit words");
    uint64_t w[sizeof(T) / 8];
#pragma unroll
    for (size_t i = 0; i < sizeof(T) / 8; ++i) w[i] = shared_load(reinterpret_cast<const uint64_t*>(p) + i);
    return __builtin_bit_cast(T, w);
}
template <typename T>
__device__ __forceinline__ void shared_store_as(T* p, const T& v) {
    struct Words { uint64_t w[sizeof(T) / 8]; };
    const Words w = __builtin_bit_cast(Words, v);
#pragma unroll
    for (size_t i = 0; i < sizeof(T) / 8; ++i) shared_store(reinterpret_cast<uint64_t*>(p) + i, w.w[i]);
}
// Waits until this wave's writes have arrived.
__device__ __forceinline__ void writes_arrived() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// ---------------------------------------------------------------------------
// Sites of the wave walker.  A site's key is a linear function of its
// coordinates (modulo 2^32 per word), so a neighbour's key is the end's key
// plus a per-direction offset, and no key a walk can meet is 0 (an empty slot).
// word(): the 32-bit word that is hashed.
// ---------------------------------------------------------------------------
struct Site2 {
    using Key = uint32_t;               // x + 2^16 y + origin; coordinates stay below 2^15
    __device__ static Key origin() { return 0x80008000u; }
    __device__ static Key delta(int dir) {
        if (dir >= 4) return 0u;
        const Key mag = (dir >> 1) ? 0x10000u : 1u;
        return (dir & 1) ? 0u - mag : mag;
    }
    __device__ static Key next(Key k, Key d) { return k + d; }
    __device__ static uint32_t word(Key k) { return k; }
    __device__ static bool empty(Key k) { return k == 0u; }
    __device__ static uint32_t mark(Key k) { return k; }      // nonzero iff a site
    __device__ static void unpack(Key k, int& x, int& y, int& z) {
        x = (int)(k & 0xFFFFu) - 32768;
        y = (int)(k >> 16) - 32768;
        z = 0;
    }
};

// Cubic walks of at most COMPACT3_MAX_N steps: x + SITE3_Y y + SITE3_Z z +
// SITE3_0 modulo 2^32.  The shortest nonzero step (in the sum of |coordinate|)
// with the same key as no step at all is 2293 long and the shortest that takes
// the origin's key to 0 is 2065 long (both checked exhaustively by
// tests/test_walker_keys.py), while two sites of one walk, or a site and a neighbour of
// its end, are at most n_max + 1 <= 2064 apart.
struct Site3c {
    using Key = uint32_t;
    __device__ static Key origin() { return SITE3_0; }
    __device__ static Key delta(int dir) {
        if (dir >= 6) return 0u;
        const int axis = dir >> 1;
        const Key mag = axis == 0 ? 1u : axis == 1 ? SITE3_Y : SITE3_Z;
        return (dir & 1) ? 0u - mag : mag;
    }
    __device__ static Key next(Key k, Key d) { return k + d; }
    __device__ static uint32_t word(Key k) { return k; }
    __device__ static bool empty(Key k) { return k == 0u; }
    __device__ static uint32_t mark(Key k) { return k; }
};

// Every other cubic walk: that key in the low word and the square-lattice key
// of (x, y) in the high word, which is never 0.  Equal keys have equal x and y,
// and SITE3_Z is odd, so z is equal too.
struct Site3 {
    using Key = uint64_t;
    __device__ static Key join(uint32_t lo, uint32_t hi) { return ((uint64_t)hi << 32) | lo; }
    __device__ static Key origin() { return join(SITE3_0, 0x80008000u); }
    __device__ static Key delta(int dir) { return join(Site3c::delta(dir), Site2::delta(dir)); }
    __device__ static Key next(Key k, Key d) {
        return join((uint32_t)k + (uint32_t)d, (uint32_t)(k >> 32) + (uint32_t)(d >> 32));
    }
    __device__ static uint32_t word(Key k) { return (uint32_t)k; }
    __device__ static bool empty(Key k) { return (uint32_t)(k >> 32) == 0u; }
    __device__ static uint32_t mark(Key k) { return (uint32_t)(k >> 32); }
    __device__ static void unpack(Key k, int& x, int& y, int& z) {
        Site2::unpack((uint32_t)(k >> 32), x, y, z);
        // SITE3_Z * z, divided by SITE3_Z modulo 2^32
        z = (int)(((uint32_t)k - SITE3_0 - (uint32_t)x - SITE3_Y * (uint32_t)y) * SITE3_Z_INV);
    }
};

template <int D, bool CK> struct SiteOf { using T = Site2; };
template <> struct SiteOf<3, false> { using T = Site3; };
template <> struct SiteOf<3, true> { using T = Site3c; };

// Set bits of m, counted on the vector side (a lane mask that a vector compare
// wrote costs the scalar unit a wait of some 16 cycles before it can read it),
// and x * 2^e beside it: the two instructions between the compare and the counts
// are the wait states the hardware wants between a vector instruction that
// writes a scalar register and one that reads it.
__device__ __forceinline__ uint32_t mask_count(uint64_t m, double x, int e, int scale, double& scaled) {
    uint32_t r;
    int d;
    double y;
    asm("v_sub_u32 %1, %6, %7\n\t"
        "v_ldexp_f64 %2, %5, %1\n\t"
        "v_bcnt_u32_b32 %0, %3, 0\n\t"
        "v_bcnt_u32_b32 %0, %4, %0"
        : "=&v"(r), "=&v"(d), "=&v"(y)
        : "s"((uint32_t)m), "s"((uint32_t)(m >> 32)), "v"(x), "v"(e), "v"(scale));
    scaled = y;
    return r;
}

template <typename T>
__device__ __forceinline__ uint32_t lds_address(T* p) {
    return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)p;
}
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

template <typename T>
__device__ __forceinline__ T lds_load(uint32_t address) {
    return *(const __attribute__((address_space(3))) T*)(uintptr_t)address;
}
template <typename T>
__device__ __forceinline__ void lds_store(uint32_t address, T v) {
    *(__attribute__((address_space(3))) T*)(uintptr_t)address = v;
}
// A record read whole through a word vector.
__device__ __forceinline__ SumRec record_of(u32x4 w) {
    SumRec r;
    r.m = __builtin_bit_cast(double, ((uint64_t)w.y << 32) | w.x);
    r.e = (int32_t)w.z;
    r.h = w.w;
    return r;
}
__device__ __forceinline__ u32x4 words_of(double m, int32_t e, uint32_t h) {
    const uint64_t b = __builtin_bit_cast(uint64_t, m);
    u32x4 r;
    r.x = (uint32_t)b;
    r.y = (uint32_t)(b >> 32);
    r.z = (uint32_t)e;
    r.w = h;
    return r;
}

// One arrival's writes to LDS, by lane `il` alone: the site's key into its table
// slot, its slot id, and the record of its length (for long walks the record goes
// to global memory, see there).  taddr: the slot's LDS address in lane il; saddr,
// raddr: the addresses of the length's slot id and record.  One lane selected
// with a scalar shift takes two instructions; a compare and a saved mask would
// take six and a wait.
__device__ __forceinline__ void write_arrival(uint32_t il, uint32_t taddr, uint32_t key, uint32_t saddr,
                                              uint32_t slot, uint32_t raddr, u32x4 rec) {
    asm volatile("s_lshl_b64 exec, 1, %0\n\t"
                 "ds_write_b32 %1, %2\n\t"
                 "ds_write_b16 %3, %4\n\t"
                 "ds_write_b128 %5, %6\n\t"
                 "s_mov_b64 exec, -1"
                 :: "s"(il), "v"(taddr), "v"(key), "v"(saddr), "v"(slot), "v"(raddr), "v"(rec) : "memory", "scc");
}
__device__ __forceinline__ void write_arrival(uint32_t il, uint32_t taddr, uint64_t key, uint32_t saddr,
                                              uint32_t slot, uint32_t raddr, u32x4 rec) {
    asm volatile("s_lshl_b64 exec, 1, %0\n\t"
                 "ds_write_b64 %1, %2\n\t"
                 "ds_write_b16 %3, %4\n\t"
                 "ds_write_b128 %5, %6\n\t"
                 "s_mov_b64 exec, -1"
                 :: "s"(il), "v"(taddr), "v"(key), "v"(saddr), "v"(slot), "v"(raddr), "v"(rec) : "memory", "scc");
}
__device__ __forceinline__ void write_site(uint32_t il, uint32_t taddr, uint32_t key, uint32_t saddr, uint32_t slot) {
    asm volatile("s_lshl_b64 exec, 1, %0\n\t"
                 "ds_write_b32 %1, %2\n\t"
                 "ds_write_b16 %3, %4\n\t"
                 "s_mov_b64 exec, -1"
                 :: "s"(il), "v"(taddr), "v"(key), "v"(saddr), "v"(slot) : "memory", "scc");
}
__device__ __forceinline__ void write_site(uint32_t il, uint32_t taddr, uint64_t key, uint32_t saddr, uint32_t slot) {
    asm volatile("s_lshl_b64 exec, 1, %0\n\t"
                 "ds_write_b64 %1, %2\n\t"
                 "ds_write_b16 %3, %4\n\t"
                 "s_mov_b64 exec, -1"
                 :: "s"(il), "v"(taddr), "v"(key), "v"(saddr), "v"(slot) : "memory", "scc");
}

// The lanes where |x| < y, and where |x| > y, for the scalar unit (the compiler
// would form |x| in registers for two compares).
__device__ __forceinline__ uint64_t lanes_below(double x, double y) {
    uint64_t m;
    asm("v_cmp_lt_f64_e64 %0, |%1|, %2" : "=s"(m) : "v"(x), "s"(y));
    return m;
}
__device__ __forceinline__ uint64_t lanes_above(double x, double y) {
    uint64_t m;
    asm("v_cmp_gt_f64_e64 %0, |%1|, %2" : "=s"(m) : "v"(x), "v"(y));
    return m;
}

// The lowest bit set in m, or all ones for none.
__device__ __forceinline__ uint32_t first_bit(uint64_t m) {
    uint32_t r;
    asm("s_ff1_i32_b64 %0, %1" : "=s"(r) : "s"(m));
    return r;
}

// Empties the slots at LDS addresses `at` of the lanes whose `index` is below
// `depth` (a vector compare that selects the lanes itself: through a saved mask
// the scalar unit would wait for it).  A lane read must be four wait states behind
// a vector instruction that writes the lane mask, which the compiler does not see
// in here; this form waits for them.
template <typename Key>
__device__ __forceinline__ void clear_sites(uint32_t index, uint32_t depth, uint32_t at) {
    const Key zero = 0;
    if constexpr (sizeof(Key) == 8)
        asm volatile("v_cmpx_lt_u32_e32 %0, %1\n\t"
                     "ds_write_b64 %2, %3\n\t"
                     "s_mov_b64 exec, -1\n\t"
                     "s_nop 1"
                     :: "v"(index), "v"(depth), "v"(at), "v"(zero) : "memory", "vcc");
    else
        asm volatile("v_cmpx_lt_u32_e32 %0, %1\n\t"
                     "ds_write_b32 %2, %3\n\t"
                     "s_mov_b64 exec, -1\n\t"
                     "s_nop 1"
                     :: "v"(index), "v"(depth), "v"(at), "v"(zero) : "memory", "vcc");
}

// The same, and one copy less to resume in lane p mod 64 of `rem` (which fills the
// wait states).
template <typename Key>
__device__ __forceinline__ void clear_sites_take_copy(uint32_t index, uint32_t depth, uint32_t at, uint32_t& rem,
                                                      uint32_t p) {
    const Key zero = 0;
    if constexpr (sizeof(Key) == 8)
        asm volatile("v_cmpx_lt_u32_e32 %1, %2\n\t"
                     "ds_write_b64 %3, %4\n\t"
                     "s_lshl_b64 exec, 1, %5\n\t"
                     "v_add_u32 %0, -1, %0\n\t"
                     "s_mov_b64 exec, -1"
                     : "+v"(rem) : "v"(index), "v"(depth), "v"(at), "v"(zero), "s"(p) : "memory", "vcc", "scc");
    else
        asm volatile("v_cmpx_lt_u32_e32 %1, %2\n\t"
                     "ds_write_b32 %3, %4\n\t"
                     "s_lshl_b64 exec, 1, %5\n\t"
                     "v_add_u32 %0, -1, %0\n\t"
                     "s_mov_b64 exec, -1"
                     : "+v"(rem) : "v"(index), "v"(depth), "v"(at), "v"(zero), "s"(p) : "memory", "vcc", "scc");
}

// The copy stack's registers: one pending entry per lane.
template <typename Key>
struct CopyLanes {
    uint32_t ra, rem;      // the length (its record's address) and the copies to resume
    int32_t e;             // their weight m * 2^e
    double m;
    Key key;               // the walk's end
};

// Writes lane p mod 64 of the entries, selected with a scalar shift.
template <typename Key>
__device__ __forceinline__ void put_entry(CopyLanes<Key>& c, uint32_t p, uint32_t ra, uint32_t rem, int32_t e,
                                          double m, Key key) {
    const uint64_t mb = __builtin_bit_cast(uint64_t, m);
    uint64_t cm = __builtin_bit_cast(uint64_t, c.m);
    uint32_t mlo = (uint32_t)cm, mhi = (uint32_t)(cm >> 32);
    if constexpr (sizeof(Key) == 8) {
        uint32_t klo = (uint32_t)c.key, khi = (uint32_t)(c.key >> 32);
        asm volatile("s_lshl_b64 exec, 1, %7\n\t"
                     "v_mov_b32 %0, %8\n\t"
                     "v_mov_b32 %1, %9\n\t"
                     "v_mov_b32 %2, %10\n\t"
                     "v_mov_b32 %3, %11\n\t"
                     "v_mov_b32 %4, %12\n\t"
                     "v_mov_b32 %5, %13\n\t"
                     "v_mov_b32 %6, %14\n\t"
                     "s_mov_b64 exec, -1"
                     : "+v"(c.ra), "+v"(c.rem), "+v"(c.e), "+v"(mlo), "+v"(mhi), "+v"(klo), "+v"(khi)
                     : "s"(p), "v"(ra), "v"(rem), "v"(e), "v"((uint32_t)mb), "v"((uint32_t)(mb >> 32)),
                       "v"((uint32_t)key), "v"((uint32_t)(key >> 32))
                     : "scc");
        c.key = ((uint64_t)khi << 32) | klo;
    } else {
        asm volatile("s_lshl_b64 exec, 1, %6\n\t"
                     "v_mov_b32 %0, %7\n\t"
                     "v_mov_b32 %1, %8\n\t"
                     "v_mov_b32 %2, %9\n\t"
                     "v_mov_b32 %3, %10\n\t"
                     "v_mov_b32 %4, %11\n\t"
                     "v_mov_b32 %5, %12\n\t"
                     "s_mov_b64 exec, -1"
                     : "+v"(c.ra), "+v"(c.rem), "+v"(c.e), "+v"(mlo), "+v"(mhi), "+v"(c.key)
                     : "s"(p), "v"(ra), "v"(rem), "v"(e), "v"((uint32_t)mb), "v"((uint32_t)(mb >> 32)), "v"(key)
                     : "scc");
    }
    c.m = __builtin_bit_cast(double, ((uint64_t)mhi << 32) | mlo);
}

// One sequence's `tours` tours against frozen pooled sums (the whole hot path
// of one walk); run by one wavefront.  Gsrc: the pooled sums to read (the
// problem's own, or an epoch's copy in a chained launch).  Returns the tours
// run, with bit 31 set if the step cap stopped the sequence (WALK_ABORTED).
// JOB: a chained launch, where the epoch starts here (the sequence's sums and
// tour count start from zero), its sums stay where they are (in LDS, or with
// LONG in the global row) and another wave may have run its last epoch.
// OBS: also record W * R^2 (squared end-to-end distance) at every arrival
// beside the weight, the numerator of the ratio estimator of eqn (5).
// PART: some of a sequence's tours, with its state handed on past the L2 (wave_row:
// with LONG, a row of this wave's own for the sums; left: the rest of the step cap).
// LONG: walks too long for the per-length sums to share LDS with the
// occupancy table; the sums stay in the sequence's global row (read and
// written in place) and LDS holds the table and the slot ids.
//
// What bounds it.  Every step depends on the one before, and a lone wave issues
// an instruction every 4.3 cycles whatever it is (dependent FP64 included), so
// a walk-step costs its instruction count, plus what crosses units: 12 cycles
// for a branch not taken, 20 for one taken, 16 where the scalar unit reads what
// the vector unit wrote.  So the common event -- a walk with a free neighbour,
// a decision that keeps one copy (or a survivor), a growth that ends neither
// the walk, the random block nor the step budget -- is one straight block of 61
// instructions, mostly vector code, with a single branch, its own loop's
// (run_ahead); enrichment to two copies, pruning and trapping (a quarter of the
// square lattice's events) are short blocks beside it; and everything else is
// handled outside, in the extended-range form (the event loop).
// Measured with every case decided in line (255 instructions and 17 branches a
// step) / now, ms, means of three seeds:
//   one square sequence of 20-step walks, 1000 tours      12.4 / 5.05
//   4096 square sequences of 500 steps, 64 tours          77.1 / 29.0
//   16384 cubic sequences of 1000 steps, 32 tours          164 / 68.9
//   256 Rosenbluth walks of up to 6000 cubic steps, twice 6.41 / 1.93
// A lone wave's step (us): square 0.625 / 0.222, cubic 0.610 / 0.205.
constexpr uint32_t WALK_ABORTED = 0x80000000u;
// run_ahead's distance from a decision that the rounding of r could change: the
// hardware's reciprocal has a stated error of 2^29 units in the last place (2^-23),
// and a uniform's high word is within 2^-20.
constexpr double DECISION_MARGIN = 0x1p-16;
// Sites outside their places that are listed, one per lane (a walk has a few at most).
constexpr uint32_t FAR_LIST = 64;

template <int D, bool OBS = false, bool LONG = false, bool CK = false, bool JOB = false, bool PART = false>
__device__ __forceinline__ uint32_t walk_sequence(const ProblemDesc* desc, uint32_t tours, uint32_t cap,
                                                  uint32_t s, unsigned char* lds, const SumRec* Gsrc,
                                                  SumRec* wave_row = nullptr, uint32_t* left = nullptr) {
    static_assert(!(OBS && (JOB || PART)) && !(JOB && PART), "not built");
    constexpr bool HANDED = JOB || PART;       // another wave may have run the sequence before
    // (loads through a generic pointer pass for lane values)
    tours = ufirst(tours);
    cap = ufirst(cap);
    const ProblemDesc P = load_const(desc);
    static_assert(!(OBS && CK), "observables need coordinates, which compact keys do not keep");
    using S_ = typename SiteOf<D, CK>::T;
    using Key = typename S_::Key;
    constexpr int W = (D == 2) ? 16 : 8;       // lanes per direction
    constexpr int LW = (D == 2) ? 4 : 3;
    constexpr uint64_t FIELD = (1ull << W) - 1ull;

    // LDS: the occupancy table, the slot id of every site of the walk and the
    // sequence's own per-length sums (moved in at the start of the sequence's
    // tours and back out at their end)
    Key* table = reinterpret_cast<Key*>(lds);
    uint16_t* sid = reinterpret_cast<uint16_t*>(lds + sizeof(Key) * P.slots);
    const uint32_t row_lds = LONG ? 0u : P.row * (uint32_t)sizeof(SumRec);
    SumRec* Ls = !LONG ? reinterpret_cast<SumRec*>(lds + P.lds_team_bytes)
                       : PART ? wave_row : P.L + (size_t)s * P.row;
    // (observables) the sequence's per-length sums of W * R^2, after its sums
    SumRec* LRs = LONG ? P.LR + (size_t)s * P.row
                       : reinterpret_cast<SumRec*>(lds + P.lds_team_bytes + row_lds);
    // record access: LDS, or the global row of a long walk
    auto rec_ld = [&](const SumRec* p) INLINE -> SumRec {
        if constexpr (LONG) return load_global(p);
        else return *p;
    };
    auto rec_st = [&](SumRec* p, const SumRec& v) INLINE {
        if constexpr (LONG) store_global(p, v);
        else *p = v;
    };
    const int lane = (int)threadIdx.x;
    const uint32_t S = P.slots;

    // The occupancy table is W - 1 subtables of `sub` slots.  A site may sit in
    // one slot of each, found by a hash of its own per subtable, and takes the
    // first that is empty: lane dir * W + o reads the slot of neighbour dir in
    // subtable o, so one LDS read looks a step's neighbours up in all their
    // places, a neighbour is occupied iff one of its lanes reads its key, and
    // lanes below a hit are always occupied (deletion is last in, first out).
    // At load 0.5 a walk of 1000 cubic steps finds its places all taken about
    // once in 10^4 walks (linear probing over the same lanes: ten times per
    // walk), and 0.65 still costs under 0.3% of its steps; such a site goes into
    // any empty slot, and a list of them tells the events to look there (below).  The
    // last lane of a direction, and the lanes past the directions, read slot
    // S - 1, which no subtable holds (S is 2^b or 3 * 2^b, never a multiple of
    // W - 1) and which stays empty: a free direction has a lane that reads an
    // empty slot even when its places are taken.
    // (lanes past the directions: never chosen, whatever is occupied)
    const int pdir = lane / W < 2 * D ? lane / W : 64;
    const int poff = lane % W;
    const uint32_t sub = S / (uint32_t)(W - 1);
    const bool blank = poff == W - 1 || pdir >= 2 * D;
    const uint32_t lane_sub = blank ? 0u : sub;
    const uint32_t lane_base = blank ? S - 1u : (uint32_t)poff * sub;
    const uint32_t lane_mul = ((0x9E3779B1u * (uint32_t)(poff + 1)) ^ (0x85EBCA77u * (uint32_t)(poff + 3))) | 1u;
    const Key pdelta = S_::delta(pdir);
    // (as an LDS address)
    uint32_t lane_at = lane_base * (uint32_t)sizeof(Key) + lds_address(table);
    asm volatile("" : "+v"(lane_at));          // (one addend)
    auto place_of = [&](Key k) INLINE {
        uint32_t h = __umulhi(S_::word(k) * lane_mul, lane_sub);
        asm("" : "+v"(h));                     // (or the shift is merged into the 64-bit product)
        return h * (uint32_t)sizeof(Key) + lane_at;
    };
    // a site's slot id: its LDS address in keys (16 bits: LDS has 160 KB)
    auto id_of = [&](uint32_t place) INLINE { return place / (uint32_t)sizeof(Key); };
    auto clear_id = [&](uint32_t i) INLINE { lds_store<Key>(i * (uint32_t)sizeof(Key), (Key)0); };

    // A zero the compiler cannot see through: addresses and sums formed with it
    // stay in vector registers.
    uint32_t vz;
    asm volatile("v_mov_b32 %0, 0" : "=v"(vz));

    const uint32_t n_max = P.n_max;
    const uint32_t row = P.row;
    const bool shared_mode = (P.mode == MODE_SHARED);
    const bool control_mode = (P.mode != MODE_ROSENBLUTH);
    const double pool = shared_mode ? (double)P.N : 1.0;
    const uint64_t pool_u = shared_mode ? (uint64_t)P.N : 1ull;

    // the empty table with the origin in it, slot id of site 0
    for (uint32_t i = (uint32_t)lane; i < S; i += 64) table[i] = (Key)0;
    wave_fence();
    const Key origin_key = S_::origin();
    if (lane == 0) {                           // (lane 0: subtable 0)
        const uint32_t o = place_of(origin_key);
        lds_store<Key>(o, origin_key);
        sid[0] = (uint16_t)id_of(o);
    }
    wave_fence();

    // the copy stack of sequence s
    StackEntry* stk = P.stack + (size_t)(PART ? blockIdx.x : s) * n_max;
    const size_t rb0 = (size_t)s * row;
    const uint32_t grow = pooled_row(P.mode, s);
    const SumRec* Grow = Gsrc + (size_t)grow * row;
    const uint64_t MGs = ufirst64(JOB ? shared_load(P.MG) : P.MG[grow]);
    uint32_t tlo = ufirst((uint32_t)(HANDED ? shared_load(P.t + s) : P.t[s]));   // tour index: its low word keys the random numbers
    uint32_t m = JOB ? 0u : ufirst(PART ? shared_load(P.m + s) : P.m[s]);
    if constexpr (JOB) {
        for (uint32_t i = (uint32_t)lane; i <= n_max; i += 64u) rec_st(Ls + i, SumRec{0.0, 0, 0u});
    } else if constexpr (PART) {
#pragma unroll 4
        for (uint32_t i = (uint32_t)lane; i <= n_max; i += 64u) rec_st(Ls + i, shared_load_as(P.L + rb0 + i));
    } else if constexpr (!LONG) {
        for (uint32_t i = (uint32_t)lane; i <= n_max; i += 64u) Ls[i] = load_global(P.L + rb0 + i);
        if constexpr (OBS) {
            for (uint32_t i = (uint32_t)lane; i <= n_max; i += 64u) LRs[i] = load_global(P.LR + rb0 + i);
        }
    }
    // In LDS, a row padded to 16 records has a record past the last length's. No
    // number there makes every test of run_ahead fail at n_max: the walk stops
    // there without having been watched.
    const bool guarded = !LONG && row > n_max + 1u;
    if constexpr (!LONG) {
        if (guarded && lane == 0) Ls[n_max + 1u] = SumRec{__builtin_nan(""), 0, 0u};
    }
    wave_fence();
    SumRec rec0 = rec_ld(Ls);
    // counters of this call, added to the sequence's totals at its end
    // (every event grows the walk or prunes a copy, so the steps are the events
    // less the prunings)
    uint32_t c_tours = 0, c_maxd = 0, c_enrich = 0, c_prunes = 0, c_traps = 0;
    uint64_t c_copies = 0, c_events = 0;
    const uint32_t capv = cap ? cap : 0xFFFFFFFFu;   // step cap of this call (0: none)
    const uint64_t* old_digest = P.stats + (size_t)s * STATS_WORDS + ST_DIGEST;
    uint32_t digest = (uint32_t)(HANDED ? shared_load(old_digest) : *old_digest) + vz;
    bool abort = false;
    // the registers of the copy stack (see the tour loop)
    CopyLanes<Key> cs = {0u, 0u, 0, 0.0, (Key)0};

    // byte addresses of length 0: its record (in LDS, or with LONG as an offset
    // from the row) and its slot id; gsums + a record's address is the pooled
    // sum of the same length
    const uint32_t rec_base = LONG ? 0u : lds_address(Ls);
    const uint32_t sid_base = lds_address(sid);
    const unsigned char* gsums = reinterpret_cast<const unsigned char*>(Grow) - rec_base;
    auto pooled = [&](uint32_t address, uint32_t ahead) INLINE {
        return load_global(reinterpret_cast<const SumRec*>(gsums + ahead * 16u + address));
    };

    // (LONG) the row as a buffer: lane 0 stores a record, the other lanes' offsets
    // are past its end and dropped.  (A store among inline assembly would not be
    // counted by the compiler, which then waits for it where it waits for the
    // loads before it: 0.35 us a step instead of 0.28.)
    const __amdgpu_buffer_rsrc_t row_out =
        __builtin_amdgcn_make_buffer_rsrc(Ls, 0, (int)(row * (uint32_t)sizeof(SumRec)), 0x00020000);
    const uint32_t lane_out = lane == 0 ? 0u : 0x80000000u;
    // -2^-501 in a register (see run_ahead), and twice the lane
    double small = -0x1p-501;
    asm volatile("" : "+v"(small));
    const uint32_t lane2 = 2u * (uint32_t)lane;
    // (LONG) the longest walk so far, as the address of its slot id: a row's records
    // past it are as they were
    uint32_t longest = sid_base + vz;

    for (uint32_t tour = 0; tour < tours && !abort; ++tour) {
        // ---- a pass through the empty walk (eqn (4), M) ----
        const uint32_t tt = tlo;
        tlo += 1u;
        m += 1;
        c_tours += 1;
        {
            const XF r0 = xf_add(xf_of(rec0), XF{0.5, 1});   // W_0 = 1
            rec0.m = r0.m;
            rec0.e = r0.e;
            rec0.h += 1u;
        }
        // Events of this tour: kb + li - 1 so far (fewer than 2^32 because the
        // step cap is at most 2^31 and every event either grows the walk or
        // prunes a grown copy).  Lane i of 1 .. 63 holds the random block of
        // event kb + i - 1: its first word b0 and its 53-bit uniform u (exact:
        // integers below 2^53 and power-of-two scalings).  Event 64 of a block
        // reads lane 0, which stops run_ahead.
        uint32_t kb = 0, li = 1, b0 = 0;
        double u = 0.0;
        auto draw = [&]() INLINE {
            // (the key schedule is formed here each time: hoisted, it would take
            // twenty scalar registers)
            uint32_t k0 = P.key0, k1 = P.key1;
            asm volatile("" : "+s"(k0), "+s"(k1));
            const uint4 rb = philox10(make_uint4(kb + (uint32_t)lane - 1u, 0u, tt, s), k0, k1);
            b0 = rb.x;
            u = ((double)(rb.y >> 5) * 67108864.0 + (double)(rb.z >> 6)) * (1.0 / 9007199254740992.0);
        };
        draw();
        // the walk's length, as the addresses of its record and of its slot id
        uint32_t ra = rec_base + vz, sa = sid_base + vz;
        auto length = [&]() INLINE { return (ufirst(ra) - rec_base) >> 4; };
        Key ekey = origin_key;                 // the walk's end
        // sites of the walk outside their places: the first one, and the first
        // FAR_LIST of them, one per lane, in order (all ones: none)
        uint32_t far_lo = ~0u, far_at = ~0u;
        // pending copies: sp entries, the one at position p in lane p mod 64
        // of cs for p >= lo, in global memory for p < lo (at
        // most 64 in registers; the most recent ones, which are resumed first)
        uint32_t sp = 0, lo = 0;
        // tours seen by the running average of eqn (6) (reading of Algorithm 2)
        // and its reciprocal, once per tour and kept in registers
        double seen = (double)(MGs + pool_u * (uint64_t)m);
        asm volatile("" : "+v"(seen));
        const double seen_r = recip_normal(seen);

        // The walk's weight wm * 2^we, its sum at this length Lm * 2^we and the
        // pooled sum G (the next length's once scan has used it).  Inside run_ahead mantissas are left as they
        // come (a power-of-two scale commutes with every rounding as long as
        // nothing leaves the FP64 range) and we is constant, so a sum costs one
        // exact shift of the other operand and the ratio none.  wm is in
        // [0.5, 1) when a block of events begins or a copy resumes; one event
        // at most halves it or makes it 2^6.6 times larger.
        double wm, Lm;
        int we;
        SumRec G;
        uint32_t uf = 0u;                      // what run_ahead compares (see arm)
        SumRec nxt = {0.0, 0, 0u}, nxr = {0.0, 0, 0u};   // records of the next length
        auto steps = [&]() INLINE { return (uint32_t)c_events + kb + li - 1u - c_prunes; };
        // Makes the next events ready for run_ahead: lane i of uf holds the high
        // word of 1 - u - MARGIN, u the uniform of its event, but at least 1/16
        // (survival at a ratio below that, which could scale wm without limit,
        // is decided outside, as is a uniform of 0), and no number (which fails
        // every test) from the event on that could end the step budget or, with no
        // guard, the walk, or at once while some site is outside its places.
        // (After a resume the walk's end is further off than this says, which only
        // stops run_ahead for nothing.)
        auto arm = [&](uint32_t n) INLINE {
            const uint32_t left = min(guarded ? ~0u : n_max - n, capv - steps());
            const uint32_t last = far_lo != ~0u ? li : li + min(left, 64u) - 1u;
            const double uc = (1.0 - DECISION_MARGIN) - (u < 0.0625 ? 0.0625 : u);
            uf = ((uint32_t)lane >= last || lane == 0) ? 0x7FF80000u : (uint32_t)__double2hiint(uc);
        };
        // the next length's records
        auto load_next = [&]() INLINE {
            if constexpr (!LONG) {
                nxt = record_of(lds_load<u32x4>(ra + 16u));
                if constexpr (OBS) nxr = record_of(lds_load<u32x4>(ra + 16u + row_lds));
            } else {
                nxt = load_global(reinterpret_cast<const SumRec*>(reinterpret_cast<const unsigned char*>(Ls) + ra) + 1);
                if constexpr (OBS)
                    nxr = load_global(
                        reinterpret_cast<const SumRec*>(reinterpret_cast<const unsigned char*>(LRs) + ra) + 1);
            }
        };
        // A walk that starts or resumes decides nothing at its length: a pooled
        // sum of exactly W * seen and no sum of its own make the ratio exactly
        // 1, which keeps one copy (and no sum, Lm = 0, marks the case).
        auto no_decision = [&]() INLINE {
            Lm = 0.0;
            G.m = wm * seen;
            G.e = we;
        };
        auto weigh = [&](XF w) INLINE {
            wm = w.m;
            we = w.e + (int)vz;
            asm volatile("" : "+v"(wm));
        };
        weigh(XF{0.5, 1});
        no_decision();
        load_next();
        arm(0u);

        // what scan leaves: the neighbours' keys, slots and contents, the hits,
        // a_+, the choice, and the decision
        Key nk, v;
        uint32_t place, a, il, a8, id, hn;
        uint64_t hits, pick, choice, below1 = 0ull;
        double t, ut, uu, r1 = 0.0, w1, af;
        SumRec nx2 = {0.0, 0, 0u}, nr2 = {0.0, 0, 0u};
        auto fold = [&]() INLINE { digest = (digest ^ ((il >> LW) | a8)) * FNV_PRIME; };
        // (grown: right after commit, whose digest is left for where the look-up
        // takes its time)
        auto scan = [&](auto decide, auto grown) INLINE {
            // occupancy reads, the next length's pooled sum
            nk = S_::next(ekey, pdelta);
            place = place_of(nk);
            v = lds_load<Key>(place);
            if constexpr (LONG) {
                // (one length further: it has a whole step to arrive.  At
                // n_max - 1 that is past the last record: row is padded to
                // 16 records or the next array follows; never used)
                nx2 = load_global(reinterpret_cast<const SumRec*>(reinterpret_cast<const unsigned char*>(Ls) + ra) + 2);
                if constexpr (OBS)
                    nr2 = load_global(
                        reinterpret_cast<const SumRec*>(reinterpret_cast<const unsigned char*>(LRs) + ra) + 2);
            }
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (decltype(grown)::value) fold();
            uu = __hiloint2double((int)lane_value(uf, li), 0);
            const uint32_t bl = lane_value(b0, li);
            w1 = wm;
            if constexpr (decltype(decide)::value) {
                // eqn (6): r = W / [W_n], [W_n] = sum / seen (own epoch
                // data weighted N in Algorithm 2), as (W * seen) / sum.
                // One copy goes on iff u < r < 1 (a survivor, which takes
                // sum / seen) or 1 <= r < 2 and u < 2 - r: iff |r - 1| < 1 - u.
                // The hardware's reciprocal gives r - 1 well within the margin
                // that uf holds back; what falls between is decided outside, as
                // is r < 1 here, from the quotient as IEEE rounds it (which is
                // below 1 iff W * seen < sum).
                const double sum = ldexp(G.m, G.e - we) + Lm * pool;
                const double ww = wm * seen;
                r1 = __builtin_fma(ww, __builtin_amdgcn_rcp(sum), -1.0);
                const double ws = div_by(sum, seen, seen_r);
                below1 = __ballot(ww < sum);
                w1 = ww < sum ? ws : wm;
                G = pooled(ra, 1u);
            }
            __builtin_amdgcn_sched_barrier(0);
            hits = __ballot(v == nk);
            // (and the next length's sum at this scale)
            a = (uint32_t)(2 * D) - mask_count(hits, nxt.m, nxt.e, we, t);
            // The j-th free neighbour, j = floor(B0 a / 2^32): j and the
            // hits in lanes below a lane's own make its direction in the
            // chosen direction's lanes (and in lanes of occupied neighbours
            // of it: those up to the hit, which are not empty, before it,
            // those past the hit after it).  Its first empty place is the
            // lowest such lane that read an empty slot.
            const uint32_t j = __umulhi(bl, a);
            const uint32_t x = __builtin_amdgcn_mbcnt_hi((uint32_t)(hits >> 32),
                                                         __builtin_amdgcn_mbcnt_lo((uint32_t)hits, j));
            pick = __ballot(((x ^ (uint32_t)pdir) | S_::mark(v)) == 0u);
            // (the term that takes the next sum from 1 - u leaves it as it is
            // while it is below a quarter of its last place: for 1 - u of 2^-7
            // or more, sums up to 2^440 * 2^we.  Beyond, the event is decided
            // outside, with the same result)
            ut = __builtin_fma(t, small, uu);
            const uint64_t ok = __ballot(__builtin_fabs(r1) < ut);
            __builtin_amdgcn_sched_barrier(0);
            // what growth needs whoever is chosen, while the scalar unit waits
            af = (double)a;
            a8 = a << 3;
            id = id_of(place);
            hn = nxt.h + 1u;
            asm volatile("" : "+v"(af), "+v"(a8), "+v"(id), "+v"(hn));
            __builtin_amdgcn_sched_barrier(0);
            choice = pick & ok;
            il = first_bit(choice);
        };
        // (il is all ones where nothing was chosen, and a last lane where all
        // places of the chosen neighbour are taken)
        auto chosen = [&]() INLINE { return (~il & (uint32_t)(W - 1)) != 0u; };
        // growth by the lane `il`: W *= a_+, eqn (2), and the record, eqn (4)
        auto commit = [&](double w) INLINE {
            wm = w * af;
            Lm = t + wm;
            ra += 16u;
            asm volatile("" : "+v"(ra));       // (in place, not beside the old value)
            sa += 2u;
            li += 1u;
            const u32x4 rec = words_of(Lm, we, hn);
            if constexpr (!LONG) nxt = record_of(lds_load<u32x4>(ra + 16u));
            if constexpr (LONG) {
                write_site(il, place, nk, sa, id);
                __builtin_amdgcn_raw_buffer_store_b128(rec, row_out, ra | lane_out, 0, 0);
            } else {
                write_arrival(il, place, nk, sa, id, ra, rec);
            }
            ekey = lane_value(nk, il);
            if constexpr (OBS) {
                // R^2 of the new end, exact in FP64 (|coordinates| < 2^15)
                int cx, cy, cz;
                S_::unpack(ekey, cx, cy, cz);
                const double r2 = (double)cx * (double)cx + (double)cy * (double)cy + (double)cz * (double)cz;
                SumRec rr;
                rr.m = ldexp(nxr.m, nxr.e - we) + wm * r2;
                rr.e = we;
                rr.h = 0u;
                if (lane == 0) {
                    if constexpr (LONG)
                        store_global(reinterpret_cast<SumRec*>(reinterpret_cast<unsigned char*>(LRs) + ra), rr);
                    else
                        *reinterpret_cast<SumRec*>(lds + P.lds_team_bytes + row_lds + (ra - rec_base)) = rr;
                }
            }
            if constexpr (LONG) {
                nxt = nx2;
                if constexpr (OBS) nxr = nr2;
            } else {
                if constexpr (OBS) nxr = record_of(lds_load<u32x4>(ra + 16u + row_lds));
            }
        };
        // a copy stack entry: `copies` still to resume here with weight w
        auto push = [&](double w, uint32_t copies) INLINE {
            put_entry(cs, sp, ra, copies + vz, we, w, ekey);
            sp += 1u;
            c_maxd = max(c_maxd, sp);
            c_enrich += 1u;
            c_copies += (uint64_t)copies;
        };
        // back to the most recent pending copy, which the registers hold
        // (at: the slot ids of the last 64 sites; a short walk's reach into the
        // table before them and are not used)
        auto last_ids = [&]() INLINE { return (uint32_t)lds_load<uint16_t>(sa - lane2); };
        auto resume = [&](uint32_t at) INLINE {
            const uint32_t tl = (sp - 1u) & 63u;
            const double wv = lane_value(cs.m, tl);
            wm = __builtin_amdgcn_frexp_mant(wv);
            we = (int)lane_value((uint32_t)cs.e, tl) + __builtin_amdgcn_frexp_exp(wv) + (int)vz;
            asm volatile("" : "+v"(wm));
            ekey = lane_value(cs.key, tl);
            ra = lane_value(cs.ra, tl) + vz;
            const uint32_t rem = lane_value(cs.rem, tl);
            // LIFO deletion of the sites after it restores the table exactly
            const uint32_t end = sa;
            if constexpr (LONG) longest = max(longest, end);
            sa = (ra >> 3) + (sid_base - rec_base / 8u);
            clear_sites_take_copy<Key>(lane2, end - sa, at * (uint32_t)sizeof(Key), cs.rem, tl);
            if (__builtin_expect(__ballot(end - sa > 128u) != 0ull, 0)) {
                uint32_t d = 128u;
                do {
                    at = lds_load<uint16_t>(end - d - lane2);
                    clear_sites<Key>(lane2 + d, end - sa, at * (uint32_t)sizeof(Key));
                    d += 128u;
                } while (__ballot(end - sa > d) != 0ull);
            }
            // (its last copy: the entry is done)
            asm("s_cmp_eq_u32 %1, 1\n\ts_subb_u32 %0, %0, 0" : "+s"(sp) : "s"(rem) : "scc");
            no_decision();
            load_next();
        };
        // Runs common events, and with decisions also the enrichments that make
        // two copies and the prunings and traps that a pending copy in registers
        // follows, until an event needs more.  (The compiler lays loops out with
        // their exit at the end and if-else as two ifs, and copies what a branch
        // changes where that is not how they are written; hence the form.  No
        // variable is declared inside, for the same reason.)
        uint64_t trap, sure = 0ull;
        uint32_t at = 0u, il2 = 0u, ends, two, back;
        auto run_ahead = [&](auto decide) INLINE {
            two = back = 0u;
            do {
                if (two != 0u) {
                    // 1 <= r < 2 and u >= 2 - r
                    il = il2;
                    push(0.5 * wm, 1u);
                    commit(0.5 * wm);
                    fold();
                }
                if (back != 0u) {
                    // u >= r, pruned with probability 1 - r, or a trap (masks of
                    // all lanes: -1 or 0)
                    c_traps -= (uint32_t)trap;
                    c_prunes -= ~(uint32_t)trap;
                    li -= ~(uint32_t)trap;
                    resume(at);
                }
                // (or the product of weight and tours, which a resume forms too, is
                // formed in both branches before here, and the state copied around)
                if constexpr (decltype(decide)::value) asm volatile("" : "+v"(wm));
                scan(decide, no{});
                while (chosen()) {
                    commit(w1);
                    scan(decide, yes{});
                }
                // no free neighbour: a trap, and no event (at n_max no number is
                // equal to itself)
                const uint64_t plain = __ballot(ut == uu);
                trap = __ballot(a == 0u) & plain;
                if constexpr (decltype(decide)::value) {
                    at = last_ids();           // (for resume, while the tests wait)
                    // (a ratio out of range or too near the uniform, a uniform that
                    // is not the event's or a sum out of range: no number passes;
                    // nor does a common decision, all places taken)
                    sure = (lanes_below(r1, 0.9375) & lanes_above(r1, uu + 4.0 * DECISION_MARGIN) & plain) | trap;
                    il2 = first_bit(pick);
                    ends = (uint32_t)(below1 | trap);
                    // two copies need a place for the grown one and one in the
                    // stack's registers, everything else a copy there to go back to
                    two = min(64u - (sp - lo), ~il2 & (uint32_t)(W - 1)) & (uint32_t)sure & ~ends;
                    back = (sp - lo) & (uint32_t)sure & ends;
                    asm volatile("" : "+s"(two), "+s"(back));
                }
            } while ((two | back) != 0u);
        };

        for (;;) {
            if (control_mode) run_ahead(yes{});
            else run_ahead(no{});
            // the walk has ended here: trapped, or certainly pruned
            bool bt = trap != 0ull;
            c_traps += bt ? 1u : 0u;
            if (!bt && sure != 0ull && below1 != 0ull) {
                c_prunes += 1u;
                li += 1u;
                bt = true;
            }
            uint32_t n = length();
            bt = bt || n == n_max;
            if (!bt && li == 64u) {
                // ---- the next random blocks ----
                kb += 63u;
                li = 1u;
                draw();
                const XF w = xf_norm_nz(wm, we);
                Lm = ldexp(Lm, we - w.e);
                weigh(w);
                // (scan has moved on to the next length's sum)
                if (control_mode && __ballot(Lm != 0.0) != 0ull) G = pooled(ra, 0u);
                else no_decision();
                arm(n);
                continue;
            }
            if (!bt) {
                // ---- one event with every case ----
                uint64_t outside = 0ull;       // directions found outside their places (last lanes)
                if (far_lo != ~0u) {
                    // (a cubic walk of 10921 steps in 16384 slots has up to three of
                    // them in its last 1500 steps: 512 Rosenbluth walks of up to that
                    // length took 7.6 ms with the sites from the first one on searched
                    // at each event, 3.6 with the list)
                    auto look = [&](uint32_t i, bool valid) INLINE {
                        const Key k = valid ? lds_load<Key>(sid[valid ? i : 0u] * (uint32_t)sizeof(Key)) : (Key)0;
                        for (int d = 0; d < 2 * D; ++d)
                            if (__ballot(k == lane_value(nk, (uint32_t)(d * W))) != 0ull &&
                                ((hits >> (d * W)) & FIELD) == 0ull)
                                outside |= 1ull << (d * W + W - 1);
                    };
                    look(far_at, far_at <= n);
                    // (past a full list the sites themselves are searched)
                    for (uint32_t b = lane_value(far_at, FAR_LIST - 1u); b < n; b += 64u)
                        look(b + 1u + (uint32_t)lane, b + 1u + (uint32_t)lane <= n);
                }
                const uint32_t au = (uint32_t)(2 * D) - (uint32_t)__popcll(hits | outside);
                XF w = xf_norm_nz(wm, we);
                if (au == 0u) {
                    // (a site outside its places closes the trap)
                    c_traps += 1u;
                    bt = true;
                } else if (control_mode && __ballot(Lm != 0.0) != 0ull) {
                    const SumRec here = rec_ld(Ls + (n + vz));
                    const XF sum = xf_add_nz(xf_of(pooled(ra, 0u)), xf_mul_nz(xf_norm_nz(here.m, here.e), pool));
                    const double rr = xf_ratio_nz(xf_mul_nz(w, seen), sum);
                    const double ul = lane_value(u, li);
                    const double f = floor(rr);
                    // floor(r) as an integer: r > 0, and r <= seen / N < 2^32 because
                    // the sum includes N times the walk's own weight (the clamp
                    // only keeps the conversion defined); r >= 1 iff fi >= 1
                    const uint32_t fi = ufirst((uint32_t)__builtin_fmin(f, 4294967295.0));
                    if (fi >= 1u) {
                        // r >= 1: c = floor(r) with probability ceil(r) - r, else
                        // ceil(r) (r integral: u < 1)
                        const uint32_t ci = ubool(ul < (f + 1.0) - rr) ? fi : fi + 1u;
                        if (ci > 1u) {
                            w = xf_div_nz(w, (double)ci);
                            weigh(w);
                            if (sp - lo == 64u) {
                                // every lane holds an entry: the oldest one moves
                                // to its place in global memory
                                if (lane == (int)(lo & 63u)) {
                                    StackEntry e;
                                    e.n = cs.ra;
                                    e.remaining = cs.rem;
                                    e.e = cs.e;
                                    e.pad0 = 0u;
                                    e.m = cs.m;
                                    e.key = (uint64_t)cs.key;
                                    if constexpr (JOB) shared_store_as(stk + lo, e);
                                    else store_global(stk + lo, e);
                                }
                                lo += 1u;
                            }
                            push(wm, ci - 1u);
                        }
                    } else if (ubool(ul < rr)) {
                        w = xf_div_nz(sum, seen);  // r < 1, survives: W / r
                    } else {
                        c_prunes += 1u;            // r < 1, pruned with probability 1 - r
                        li += 1u;
                        bt = true;
                    }
                }
                if (!bt) {
                    // the chosen direction, by its last lane (every hit of the
                    // directions before it is in a lane below)
                    const uint64_t occ = hits | outside;
                    const uint32_t j = __umulhi(lane_value(b0, li), au);
                    const uint32_t x = __builtin_amdgcn_mbcnt_hi((uint32_t)(occ >> 32),
                                                                 __builtin_amdgcn_mbcnt_lo((uint32_t)occ, j));
                    const uint64_t last =
                        __ballot(x == (uint32_t)(lane / W) && poff == W - 1) & ~outside;
                    const uint32_t first = (uint32_t)__builtin_ctzll(last) & ~(uint32_t)(W - 1);
                    ekey = lane_value(nk, first);
                    const uint64_t places = __ballot(S_::mark(v) == 0u) & ((FIELD >> 1) << first);
                    uint32_t ins = 0u;
                    if (places != 0ull) {
                        ins = lane_value(place, (uint32_t)__builtin_ctzll(places));
                    } else {
                        // all places taken: the first empty slot of the table
                        // (slots outnumber the sites of the longest walk)
                        for (uint32_t b = 0;; b += 64u) {
                            const uint32_t i = b + (uint32_t)lane;
                            const uint64_t em =
                                __ballot(i < sub * (uint32_t)(W - 1) && S_::empty(table[min(i, S - 1u)]));
                            if (em != 0ull) {
                                ins = lds_address(table + b + (uint32_t)__builtin_ctzll(em));
                                break;
                            }
                        }
                        far_lo = min(far_lo, n + 1u);
                        const uint32_t listed = (uint32_t)__popcll(__ballot(far_at != ~0u));
                        if ((uint32_t)lane == listed && listed < FAR_LIST) far_at = n + 1u;
                    }
                    digest = (digest ^ ((first >> LW) | (au << 3))) * FNV_PRIME;
                    w = xf_mul_nz(w, (double)au);
                    n += 1u;
                    ra += 16u;
                    sa += 2u;
                    li += 1u;
                    const XF Lnew = xf_add_nz(xf_of(nxt), w);
                    SumRec nr;
                    nr.m = Lnew.m;
                    nr.e = Lnew.e;
                    nr.h = nxt.h + 1u;
                    if (lane == 0) {
                        lds_store<Key>(ins, ekey);
                        sid[n] = (uint16_t)id_of(ins);
                        rec_st(Ls + n, nr);
                    }
                    if constexpr (OBS) {
                        int cx, cy, cz;
                        S_::unpack(ekey, cx, cy, cz);
                        const double r2 =
                            (double)cx * (double)cx + (double)cy * (double)cy + (double)cz * (double)cz;
                        const XF R = xf_add_nz(xf_of(nxr), xf_mul_nz(w, r2));
                        SumRec ro;
                        ro.m = R.m;
                        ro.e = R.e;
                        ro.h = 0u;
                        if (lane == 0) rec_st(LRs + n, ro);
                    }
                    wave_fence();
                    if (steps() >= capv) {
                        abort = true;
                        break;
                    }
                    // (a sum out of this weight's range makes the ratio 0 or no
                    // number, and the decision comes here)
                    weigh(w);
                    Lm = ldexp(Lnew.m, Lnew.e - we);
                    bt = n == n_max;
                    if (!bt) load_next();
                }
            }
            if (bt) {
                // ---- resume the most recent pending copy, or end the tour ----
                if (sp == 0u) break;
                if (sp == lo) {
                    // no pending entry in registers: bring back the most recent
                    // ones (up to 64) from global memory
                    const uint32_t base = sp > 64u ? sp - 64u : 0u;
                    // (lanes past the top read the top entry: a branch here
                    // would make the compiler take lo, and with it the stack's
                    // height and all that follows from it, for lane values)
                    const uint32_t q = min(base + (((uint32_t)lane - base) & 63u), sp - 1u);
                    StackEntry e;
                    if constexpr (JOB) e = shared_load_as(stk + q);
                    else e = load_global(stk + q);
                    cs.ra = e.n;
                    cs.rem = e.remaining;
                    cs.e = e.e;
                    cs.m = e.m;
                    cs.key = (Key)e.key;
                    lo = base;
                }
                resume(last_ids());
                n = length();
                if (far_lo != ~0u) {
                    if (far_at > n) far_at = ~0u;
                    if (far_lo > n) far_lo = ~0u;
                }
            }
            arm(n);
        }
        // end of the tour (or abort): back to the empty walk
        c_events += kb + li - 1u;
        if constexpr (LONG) longest = max(longest, sa);
        const uint32_t n = length();
        for (uint32_t i = 1u + (uint32_t)lane; i <= n; i += 64u) clear_id(sid[i]);
        wave_fence();
    }
    // (read again, so that the steps need not keep what only the end uses)
    asm volatile("" : "+s"(desc));
    const ProblemDesc Q = load_const(desc);
    // the sums leave normalised (m in [0.5, 1), or 0 with e = 0); with LONG those of
    // the lengths that were reached (4096 square Rosenbluth walks of up to 16383 steps,
    // trapped after 71 on average: 2.41 ms a tour with whole rows, 0.49 with this)
    const uint32_t reached = LONG ? (ufirst(longest) - sid_base) / 2u : Q.n_max;
    auto leave = [&](SumRec* p, SumRec* out) INLINE {
        SumRec r = rec_ld(p);
        const XF v = xf_norm(r.m, r.e);
        r.m = v.m;
        r.e = v.e;
        if constexpr (JOB) rec_st(p, r);
        else if constexpr (PART) shared_store_as(out, r);
        else store_global(out, r);
    };
    if (lane == 0) rec_st(Ls, rec0);
    wave_fence();
#pragma unroll 1
    for (uint32_t i = (uint32_t)lane; i <= reached; i += 64u) {
        leave(Ls + i, Q.L + (size_t)s * Q.row + i);
        if constexpr (OBS) leave(LRs + i, Q.LR + (size_t)s * Q.row + i);
    }
    wave_fence();
    if (lane == 0) {
        if (abort) atomicOr(&Q.ctrl[CTRL_ERR], ERR_CAP);
        if constexpr (HANDED) {
            shared_store(Q.t + s, shared_load(Q.t + s) + c_tours);
            if constexpr (PART) shared_store(Q.m + s, m);
        } else {
            Q.t[s] += c_tours;
            Q.m[s] = m;
        }
    }
    if (lane < STATS_WORDS) {
        // lane i: word i of the sequence's counters
        uint64_t* w = Q.stats + (size_t)s * STATS_WORDS + lane;
        const uint64_t old = HANDED ? shared_load(w) : *w;
        uint64_t c = old;
        c += lane == ST_STEPS ? (uint32_t)c_events - c_prunes : 0u;
        c += lane == ST_EVENTS ? c_events : 0ull;
        c += lane == ST_ENRICH ? c_enrich : 0u;
        c += lane == ST_COPIES ? c_copies : 0ull;
        c += lane == ST_PRUNES ? c_prunes : 0u;
        c += lane == ST_TRAPS ? c_traps : 0u;
        c += lane == ST_TOURS ? c_tours : 0u;
        if (lane == ST_MAXDEPTH && c < c_maxd) c = c_maxd;
        if (lane == ST_DIGEST) c = digest;
        if (lane == ST_CAPPED && abort) c = 1;
        if constexpr (HANDED) shared_store(w, c);
        else *w = c;
    }
    if constexpr (PART) *left = abort ? 0u : cap - ((uint32_t)c_events - c_prunes);
    return c_tours | (abort ? WALK_ABORTED : 0u);
}

// Persistent launch over (problem, sequence) items of one or many problems:
// each wavefront takes the next item from a device queue until none is left.
// A problem alone is a batch of one, so a problem's bits do not depend on what
// else shares the launch.
// (at most 128 VGPRs: four waves per SIMD)
#define WAVES4 __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(4)))

template <bool OBS, bool LONG>
__device__ __forceinline__ void batch_body(const BatchArgs& B) {
    extern __shared__ __align__(16) unsigned char lds[];
    const int lane = (int)threadIdx.x;
    for (;;) {
        uint32_t got = 0u;
        if (lane == 0) got = atomicAdd(B.queue, 1u);
        const uint32_t item = ufirst(__shfl(got, 0, 64));
        if (item >= B.total_items) {
            // each wave comes here once, so the last to come knows it and leaves
            // the queue at 0 for the next launch (which needs no launch to clear it)
            if (item - B.total_items == gridDim.x - 1u && lane == 0) *B.queue = 0u;
            break;
        }
        // the problem owning the item: entries are sorted by their first item
        LaunchEntry E = B.single;
        if (B.count > 1) {
            uint32_t lo = 0, hi = B.count - 1;
            while (lo < hi) {
                const uint32_t mid = (lo + hi + 1) >> 1;
                if (B.entries[mid].first_item <= item) lo = mid;
                else hi = mid - 1;
            }
            E = B.entries[lo];
        }
        // the descriptor is read through the constant space: a flat load would
        // make every field (and so the whole walk's control flow) non-uniform
        const ProblemDesc P = load_const(E.desc);
        const uint32_t s = item - E.first_item;
        if (P.dim == 2) walk_sequence<2, OBS, LONG>(E.desc, E.tours, E.step_cap, s, lds, P.G);
        else if (!OBS && P.ckey) walk_sequence<3, false, LONG, true>(E.desc, E.tours, E.step_cap, s, lds, P.G);
        else walk_sequence<3, OBS, LONG>(E.desc, E.tours, E.step_cap, s, lds, P.G);
    }
}

__global__ void WAVES4 batch_kernel(BatchArgs B) { batch_body<false, false>(B); }

// The same for one problem whose walks also record W * R^2, whose walks are
// long (sums in global memory), or both.
__global__ void WAVES4 batch_obs_kernel(BatchArgs B) { batch_body<true, false>(B); }
__global__ void WAVES4 batch_long_kernel(BatchArgs B) { batch_body<false, true>(B); }
__global__ void WAVES4 batch_long_obs_kernel(BatchArgs B) { batch_body<true, true>(B); }

// One problem whose sequences are more than the waves that run at once.  Their
// steps differ several times over (a tour can be a thousand times longer than
// most), so with whole sequences as work items the last long ones run on a chip
// that has gone idle.  Here an item is a part of a sequence's tours: a wave takes
// the sequences in turn for their first part, and puts a sequence back at the end
// of a list for its next one.  All advance at the same pace, a slow one is never
// left waiting for a start, and only single long tours are left at the end.
// Every sequence enters the list parts - 1 times (also when its step cap has
// stopped it), so each ticket past the first N gets an entry from a wave that is
// running, and every wave ends at a ticket past the last.
// Mean of six epochs, ms, whole sequences / in 2 / 4 / 8 / 16 parts:
//   16384 cubic sequences of 1000 steps, 32 tours, 4096 waves  82.5 / 80.3 / 78.7 / 79.5 / 80.4
//   4096 square sequences of 500 steps, 64 tours, 3072 waves   34.4 / 34.5 / 33.4 / 33.4 / 33.6
// (the cubic steps alone at full rate: 45; the longest sequence alone: 38).
template <bool LONG>
__device__ __forceinline__ void part_body(const PartArgs& A) {
    extern __shared__ __align__(16) unsigned char lds[];
    const int lane = (int)threadIdx.x;
    const ProblemDesc P = load_const(A.desc);
    SumRec* row = LONG ? A.wave_rows + (size_t)blockIdx.x * P.row : nullptr;
    const uint32_t items = P.N * A.parts;
    for (;;) {
        uint32_t got = 0u;
        if (lane == 0) got = atomicAdd(A.queue, 1u);
        const uint32_t item = ufirst(__shfl(got, 0, 64));
        if (item >= items) {
            // (as in batch_body)
            if (item - items == gridDim.x - 1u && lane == 0) *A.queue = 0u;
            break;
        }
        uint32_t s = item, part = 0u, left = A.step_cap;
        if (item >= P.N) {
            uint64_t entry;
            for (uint32_t naps = 1u;; naps = min(2u * naps, 4u)) {
                entry = ufirst64(shared_load(A.list + 1 + (item - P.N)));
                if (entry != 0ull) break;
                for (uint32_t k = 0; k < naps; ++k) __builtin_amdgcn_s_sleep(127);
            }
            s = ((uint32_t)entry & (PART_MAX_N - 1u)) - 1u;
            part = (uint32_t)entry / PART_MAX_N;
            left = (uint32_t)(entry >> 32);
        }
        asm volatile("" ::: "memory");         // (nothing of the sequence is read before it is taken)
        const uint32_t tours = min(A.part_tours, A.tours - part * A.part_tours);
        if (left != 0u) {
            if (P.dim == 2)
                walk_sequence<2, false, LONG, false, false, true>(A.desc, tours, left, s, lds, P.G, row, &left);
            else if (P.ckey)
                walk_sequence<3, false, LONG, true, false, true>(A.desc, tours, left, s, lds, P.G, row, &left);
            else
                walk_sequence<3, false, LONG, false, false, true>(A.desc, tours, left, s, lds, P.G, row, &left);
        }
        if (part + 1u < A.parts) {
            writes_arrived();
            if (lane == 0) {
                const uint64_t at = atomicAdd(reinterpret_cast<unsigned long long*>(A.list), 1ull);
                shared_store(A.list + 1 + at, ((uint64_t)left << 32) | ((part + 1u) * PART_MAX_N + s + 1u));
            }
        }
    }
}

__global__ void WAVES4 part_kernel(PartArgs A) { part_body<false>(A); }
__global__ void WAVES4 part_long_kernel(PartArgs A) { part_body<true>(A); }

// ---------------------------------------------------------------------------
// Device-side epoch chaining.  Every problem runs its whole epoch schedule in
// one persistent launch: a wave claims (problem, epoch, sequence) items, runs
// the sequence's tours of that epoch, and then takes its sequence up the
// problem's merge tree -- the aligned pairwise tree over sequences, padded
// with zeros to p2 leaves -- as far as it is the second of two children to
// arrive, adding its partner's partial row into the left child's row.  The
// wave that completes the root adds the tree into the pooled sums (into a
// fresh per-epoch copy, so that no load of a later epoch ever meets a
// line cached before it was written), adds the epoch's tours to M and
// publishes the next epoch.  The result is the same as run + merge per epoch.
// ---------------------------------------------------------------------------
constexpr uint64_t JOB_IDLE_TICKS = 100000000ull * 120ull;   // 120 s at the 100 MHz clock

__device__ __forceinline__ uint32_t job_finished(const JobArgs& A) {
    uint32_t done = 0;
    for (uint32_t c = 0; c <= A.cls; ++c)
        done += __hip_atomic_load(&A.counters[JOB_FINISHED0 + c], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return done;
}

// Lane 0 tries to claim the next sequence of problem pi's open epoch.  An add
// gives every wave that comes at once its own sequence in one round trip (with
// a compare-and-swap one of them would succeed per round trip); it may run past
// N, which the next epoch's word replaces.  Past the slice's end the claim must
// not open an epoch, which only the compare-and-swap can refuse.
__device__ __forceinline__ bool job_claim(const JobArgs& A, uint32_t pi, uint32_t epochs, uint32_t N,
                                          bool closed, uint32_t& e, uint32_t& s) {
    unsigned long long w;
    if (!closed) {
        w = __hip_atomic_fetch_add(&A.state[pi].word, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        e = (uint32_t)(w >> 32);
        s = (uint32_t)w;
        asm volatile("" ::: "memory");       // (nothing of the epoch is read before it is claimed)
        return e < epochs && s < N;
    }
    w = __hip_atomic_load(&A.state[pi].word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    for (int attempt = 0; attempt < 8; ++attempt) {
        const uint32_t ee = (uint32_t)(w >> 32), cc = (uint32_t)w;
        if (ee >= epochs || cc >= N || (cc == 0u && ee > 0u)) return false;
        if (__hip_atomic_compare_exchange_strong(&A.state[pi].word, &w, w + 1ull, __ATOMIC_RELAXED,
                                                 __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
            asm volatile("" ::: "memory");
            e = ee;
            s = cc;
            return true;
        }
    }
    return false;
}

// The sequence's part of its epoch's merge, after its tours: sample counts,
// tour count, and the climb up the merge tree.  A wave's partial sums stay in
// its LDS row (a long walk's in its global row) and are written out, to the row
// of its node's first leaf, only where the partner is not there yet; the second
// to arrive adds the partner's.  12 problems of 256 sequences and 8 epochs,
// whose longest chain of steps takes 21 ms: 207 ms with agent fences at every
// node, claims by compare-and-swap and all waiting waves polling every 3 us,
// 29.6 ms without.
__device__ void job_merge(const JobArgs& A, const JobProblem& J, const ProblemDesc& P, uint32_t pi,
                          uint32_t e, uint32_t s, uint32_t tours_run, unsigned char* lds) {
    const int lane = (int)threadIdx.x;
    const uint32_t row = P.row, n1 = P.n_max + 1u;
    SumRec* Ls = reinterpret_cast<SumRec*>(lds + P.lds_team_bytes);
    uint32_t l = 0, i = s;
    // the partial sums of node (l, i)
    auto node = [&](uint32_t ll, uint32_t ii) INLINE { return P.L + (size_t)(ii << ll) * row; };
    auto own = [&](uint32_t n) INLINE -> SumRec { return J.lng ? shared_load_as(node(l, i) + n) : Ls[n]; };
    if (J.lng) __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
    for (uint32_t n = (uint32_t)lane; n < n1; n += 64u)
        __hip_atomic_fetch_add(&P.HG[n], (uint64_t)own(n).h, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (lane == 0) {
        __hip_atomic_fetch_add(&A.state[pi].msum, tours_run, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (J.stage != nullptr) {
            // what the group sums of the stop rule need
            SumRec r = own(P.n_max);
            r.h = tours_run;
            shared_store_as(J.stage + s, r);
        }
    }
    for (;;) {
        if (l == J.levels) break;                         // at the root
        if (((i ^ 1u) << l) < J.N) {
            // the partner subtree has leaves: the second of the two goes on
            uint32_t* flag = &J.flags[(J.p2 >> (l + 1u)) + (i >> 1)];
            writes_arrived();
            uint32_t old = 0u;
            if (!J.lng) {
                if (lane == 0) old = shared_load(flag);
                old = ufirst(__shfl(old, 0, 64));
                if (old == 0u) {
                    SumRec* mine = node(l, i);
#pragma unroll 4
                    for (uint32_t n = (uint32_t)lane; n < n1; n += 64u) shared_store_as(mine + n, Ls[n]);
                    writes_arrived();
                }
            }
            if (old == 0u) {
                if (lane == 0)
                    old = __hip_atomic_fetch_add(flag, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                old = ufirst(__shfl(old, 0, 64));
                if (old == 0u) return;                    // the partner will continue
            }
            asm volatile("" ::: "memory");
            if (lane == 0) shared_store(flag, 0u);
            const SumRec* other = node(l, i ^ 1u);
            SumRec* both = node(l + 1u, i >> 1);
#pragma unroll 4
            for (uint32_t n = (uint32_t)lane; n < n1; n += 64u) {
                const XF v = xf_add(xf_of(own(n)), xf_of(shared_load_as(other + n)));
                SumRec r;
                r.m = v.m;
                r.e = v.e;
                r.h = 0u;
                if (J.lng) shared_store_as(both + n, r);
                else Ls[n] = r;
            }
        }
        // (no partner: the padded subtree adds +0, the node is this subtree)
        l += 1u;
        i >>= 1;
    }
    // root: pooled sums of the next epoch, then M, then publish.  (The last
    // epoch's copy was written past the L2 to a fresh place, as this one's is.)
    if (J.lng) writes_arrived();
    const SumRec* Gprev = (e == 0u) ? P.G : J.gver + (size_t)(e - 1u) * (row + JOB_GAP);
    SumRec* Gnext = J.gver + (size_t)e * (row + JOB_GAP);
    SumRec* Gctx = const_cast<SumRec*>(P.G);
#pragma unroll 4
    for (uint32_t n = (uint32_t)lane; n < n1; n += 64u) {
        const SumRec a = load_global(Gprev + n);
        const XF v = xf_add(xf_of(a), xf_of(own(n)));
        SumRec r;
        r.m = v.m;
        r.e = v.e;
        r.h = 0u;
        shared_store_as(Gnext + n, r);
        shared_store_as(Gctx + n, r);
    }
    // the stop rule's group sums: lane k < 16 folds group k (sequences k, k + 16,
    // ... in order) into the context's running group sum and tour count
    double rel = __builtin_inf();
    if (J.stage != nullptr) {
        double gm = 0.0;
        int ge = 0;
        uint64_t gt = 0;
        if ((uint32_t)lane < GROUPS) {
            XF acc = {0.0, 0};
            uint64_t t = 0;
#pragma unroll 4
            for (uint32_t q = (uint32_t)lane; q < J.N; q += GROUPS) {
                const SumRec r = shared_load_as(J.stage + q);
                acc = xf_add(acc, xf_of(r));
                t += r.h;
            }
            const XF g = xf_add(xf_of(shared_load_as(J.gsum + lane)), acc);
            uint64_t* gtours = reinterpret_cast<uint64_t*>(J.gsum + GROUPS);
            gt = shared_load(gtours + lane) + t;
            SumRec r;
            r.m = g.m;
            r.e = g.e;
            r.h = 0u;
            shared_store_as(J.gsum + lane, r);
            shared_store(gtours + lane, gt);
            gm = g.m;
            ge = g.e;
        }
        // the same fixed sequence of operations as the host's group_rel_err
        bool defined = true;
        int e_top = -2147483647 - 1;
        for (uint32_t k = 0; k < GROUPS; ++k) {
            const double mk = __hiloint2double((int)lane_value((uint32_t)__double2hiint(gm), k),
                                               (int)lane_value((uint32_t)__double2loint(gm), k));
            const int ek = (int)lane_value((uint32_t)ge, k);
            const uint64_t tk = lane_value(gt, k);
            if (tk == 0 || mk == 0.0) defined = false;
            else if (ek > e_top) e_top = ek;
        }
        if (defined) {
            double g[GROUPS];
            double total = 0.0;
            for (uint32_t k = 0; k < GROUPS; ++k) {
                const double mk = __hiloint2double((int)lane_value((uint32_t)__double2hiint(gm), k),
                                                   (int)lane_value((uint32_t)__double2loint(gm), k));
                const int ek = (int)lane_value((uint32_t)ge, k);
                const uint64_t tk = lane_value(gt, k);
                g[k] = ldexp(mk / (double)tk, ek - e_top);
                total += g[k];
            }
            const double mean = total / GROUPS;
            double ss = 0.0;
            for (uint32_t k = 0; k < GROUPS; ++k) ss += (g[k] - mean) * (g[k] - mean);
            rel = __builtin_sqrt(ss / (GROUPS - 1)) / (4.0 * mean);
        }
    }
    if (lane == 0) {
        const uint32_t msum = __hip_atomic_exchange(&A.state[pi].msum, 0u, __ATOMIC_RELAXED,
                                                    __HIP_MEMORY_SCOPE_AGENT);
        uint64_t* MG = const_cast<uint64_t*>(P.MG);
        const uint64_t M = shared_load(MG) + msum;
        shared_store(MG, M);
        // a problem one of whose sequences hit its step cap stops after this
        // epoch (its context reports the overflow); the others run on
        const bool failed =
            __hip_atomic_load(&A.state[pi].failed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0u;
        uint32_t stop = 0u;
        if (failed) stop = STOP_FAILED;
        else if (J.stage != nullptr && J.target > 0.0 && rel <= J.target) stop = STOP_TARGET;
        else if (J.cap != 0u && M >= J.cap) stop = STOP_CAP;
        if (failed) __hip_atomic_fetch_add(&A.counters[JOB_FAILED], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (J.result != nullptr) {
            shared_store(J.result + 0, e + 1u);
            shared_store(J.result + 1, stop);
            shared_store(J.result + 2, (uint32_t)__double2loint(rel));
            shared_store(J.result + 3, (uint32_t)__double2hiint(rel));
        }
        const bool last = stop != 0u || e + 1u == J.epochs;
        writes_arrived();
        __hip_atomic_store(&A.state[pi].word, (unsigned long long)(last ? J.epochs : e + 1u) << 32,
                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (last)
            __hip_atomic_fetch_add(&A.counters[JOB_FINISHED0 + J.cls], 1u, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
    }
}

// (at most 128 VGPRs: four waves per SIMD; the register pressure this adds
// costs two spills in a chained item's merge part, none in the step loop)
__global__ void WAVES4 job_kernel(JobArgs A) {
    extern __shared__ __align__(16) unsigned char lds[];
    const int lane = (int)threadIdx.x;
    uint64_t idle_since = __builtin_amdgcn_s_memrealtime();
    uint32_t seen_progress = 0u;
    uint32_t naps = 1u;
    // the slice's clock starts with the first wave to look at it
    unsigned long long* clock0 = reinterpret_cast<unsigned long long*>(A.counters + JOB_CLOCK);
    uint64_t start = 0;
    if (lane == 0) {
        unsigned long long zero = 0ull;
        const unsigned long long now0 = __builtin_amdgcn_s_memrealtime();
        __hip_atomic_compare_exchange_strong(clock0, &zero, now0, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_AGENT);
        start = __hip_atomic_load(clock0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    start = lane_value(start, 0u);
    for (;;) {
        // past the slice's end, no epoch after a problem's first starts (the
        // started ones are finished)
        const bool closed = A.slice_ticks != 0u && __builtin_amdgcn_s_memrealtime() - start >= A.slice_ticks;
        // ---- claim: the first problem (in priority order) with an open item ----
        bool got = false;
        uint32_t pi = 0u, e = 0u, s = 0u;
        for (uint32_t b = A.start; b < A.count && !got; b += 64u) {
            const uint32_t idx = b + (uint32_t)lane;
            uint32_t mine = 0u;
            bool open = false;
            if (idx < A.count) {
                mine = A.order[idx];
                const JobProblem& J = A.probs[mine];
                const unsigned long long w =
                    __hip_atomic_load(&A.state[mine].word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                // (a launch always runs each problem's first epoch, so every
                // call makes progress however short its slice)
                open = (uint32_t)(w >> 32) < J.epochs && (uint32_t)w < J.N &&
                       (!closed || (uint32_t)w > 0u || (uint32_t)(w >> 32) == 0u);
            }
            uint64_t cand = __ballot(open);
            while (cand != 0u && !got) {
                const uint32_t f = (uint32_t)__ffsll((unsigned long long)cand) - 1u;
                cand &= cand - 1u;
                const uint32_t p = lane_value(mine, f);
                uint32_t ok = 0u, ce = 0u, cs = 0u;
                if (lane == 0) {
                    const JobProblem& J = A.probs[p];
                    ok = job_claim(A, p, J.epochs, J.N, closed, ce, cs) ? 1u : 0u;
                }
                ok = ufirst(__shfl(ok, 0, 64));
                if (ok) {
                    got = true;
                    pi = p;
                    e = ufirst(__shfl(ce, 0, 64));
                    s = ufirst(__shfl(cs, 0, 64));
                }
            }
        }
        if (!got) {
            // past the slice's end nothing new becomes claimable (items are only
            // used up), so a wave that finds nothing may leave
            if (closed) break;
            if (job_finished(A) >= A.need) break;
            const uint32_t prog =
                __hip_atomic_load(&A.counters[JOB_PROGRESS], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const uint64_t now = __builtin_amdgcn_s_memrealtime();
            if (prog != seen_progress) {
                seen_progress = prog;
                idle_since = now;
            } else if (now - idle_since > JOB_IDLE_TICKS) {
                // backstop: leave the rest to others (counted, pperm_job_report)
                if (lane == 0)
                    __hip_atomic_fetch_add(&A.counters[JOB_BACKSTOP], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                break;
            }
            // (thousands of waves may be waiting, each poll reads a line per
            // problem past the L2, and the working waves' claims and merges
            // queue behind them: a wave that keeps finding nothing looks again
            // after 3, 7, 14, 27 and at most 54 us)
            for (uint32_t i = 0; i < naps; ++i) __builtin_amdgcn_s_sleep(127);
            naps = min(2u * naps, 16u);
            continue;
        }
        naps = 1u;
        // ---- the item: the sequence's tours of this epoch, then its merge part ----
        const JobProblem J = load_const(A.probs + pi);
        const ProblemDesc P = load_const(J.desc);
        const uint32_t tours = J.sched[e];
        // the job ends with its longest chain of epochs: its waves issue first
        if (J.prio == 3u) __builtin_amdgcn_s_setprio(3);
        else if (J.prio == 2u) __builtin_amdgcn_s_setprio(2);
        else if (J.prio == 1u) __builtin_amdgcn_s_setprio(1);
        // the context's step cap, or the watchdog default of pperm_run_tours
        uint64_t cap64 = P.step_cap ? (uint64_t)P.step_cap : 4096ull * tours * (P.n_max + 1ull);
        const uint32_t cap = cap64 > (1ull << 31) ? (1u << 31) : (uint32_t)cap64;
        const SumRec* Gsrc = (e == 0u) ? P.G : J.gver + (size_t)(e - 1u) * (P.row + JOB_GAP);
        uint32_t rv;
        if (J.lng) {
            // (a long walk's row is read and written in place through the L2 of
            // its XCD: what another one wrote there last must not be met)
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
            rv = (P.dim == 2) ? walk_sequence<2, false, true, false, true>(J.desc, tours, cap, s, lds, Gsrc)
                 : P.ckey     ? walk_sequence<3, false, true, true, true>(J.desc, tours, cap, s, lds, Gsrc)
                              : walk_sequence<3, false, true, false, true>(J.desc, tours, cap, s, lds, Gsrc);
        } else {
            rv = (P.dim == 2) ? walk_sequence<2, false, false, false, true>(J.desc, tours, cap, s, lds, Gsrc)
                 : P.ckey     ? walk_sequence<3, false, false, true, true>(J.desc, tours, cap, s, lds, Gsrc)
                              : walk_sequence<3, false, false, false, true>(J.desc, tours, cap, s, lds, Gsrc);
        }
        if ((rv & WALK_ABORTED) && lane == 0)
            __hip_atomic_fetch_or(&A.state[pi].failed, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        job_merge(A, J, P, pi, e, s, rv & ~WALK_ABORTED, lds);
        __builtin_amdgcn_s_setprio(0);
        if (lane == 0)
            __hip_atomic_fetch_add(&A.counters[JOB_PROGRESS], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        idle_since = __builtin_amdgcn_s_memrealtime();
    }
}

// After a whole-schedule launch: every problem must have merged all of its
// epochs, or have stopped on a step cap (reported through its context
// already).  Anything else -- the launch ended early -- is flagged on the
// problem's context and counted.
__global__ void __launch_bounds__(256) job_check_kernel(JobArgs A) {
    for (uint32_t i = blockIdx.x * 256u + threadIdx.x; i < A.count; i += gridDim.x * 256u) {
        const JobProblem& J = A.probs[A.order[i]];
        const uint32_t done = J.result[0], stop = J.result[1];
        if (done != J.epochs && stop != STOP_FAILED) {
            atomicOr(&J.desc->ctrl[CTRL_ERR], ERR_INCOMPLETE);
            atomicAdd(&A.counters[JOB_INCOMPLETE], 1u);
        }
    }
}

__global__ void __launch_bounds__(256) fill_zero_kernel(uint32_t* p, size_t words) {
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < words; i += (size_t)gridDim.x * 256) p[i] = 0u;
}

// ---------------------------------------------------------------------------
// Merge: aligned pairwise tree over sequences.  A block of up to 16 waves takes
// 64 consecutive rows (sequences) per wave and a strip of 8 columns (lengths);
// lane i of a wave holds row i and the tree over the 64 lanes is a butterfly of
// lane shuffles (xor 1, 2, .., 32): after level l every lane holds the sum of
// its aligned block of 2^(l+1) rows, added as (left block) + (right block) up to
// commutativity, which IEEE addition has.  The waves' sums go through LDS into
// one more butterfly, over 16 lanes per column.  Partial trees of aligned blocks
// are the tree's own nodes, so repeated passes give the whole tree; missing rows
// are +0.0.  The first pass also adds up the tour counts (whole numbers, so in
// any order) and clears what it read.
//
// A small epoch is bound by its launches: 40 sequences take 15.9 us with the
// counts in a launch of their own, 9.8 us without, and up to 512 sequences are
// one pass (64 before; merge_block has the figures).
// ---------------------------------------------------------------------------
constexpr int MERGE_COLS = 8;
constexpr int MERGE_WAVES = 16;
static_assert(MERGE_ROWS == 64 * MERGE_WAVES, "rows of a merge block");

__global__ void __launch_bounds__(MERGE_ROWS) merge_pass_kernel(MergeArgs A) {
    __shared__ SumRec part[MERGE_WAVES * MERGE_COLS];
    __shared__ uint64_t parth[MERGE_WAVES * MERGE_COLS];
    __shared__ uint64_t tours[MERGE_WAVES];
    const int lane = (int)threadIdx.x & 63;
    const int wave = (int)threadIdx.x >> 6;
    const int waves = (int)blockDim.x >> 6;
    const uint32_t r = blockIdx.y * blockDim.x + threadIdx.x;
    const uint32_t c0 = blockIdx.x * MERGE_COLS;
    XF v[MERGE_COLS];
    uint64_t h[MERGE_COLS];
    const bool rv = r < A.rows;
#pragma unroll
    for (int j = 0; j < MERGE_COLS; ++j) {
        const uint32_t c = c0 + (uint32_t)j;
        const bool ok = rv && c < A.ncols;
        const size_t idx = (size_t)r * A.row + c;
        SumRec rec = {0.0, 0, 0u};
        if (ok) rec = A.in[idx];
        v[j] = xf_of(rec);
        h[j] = ok ? (A.hin ? A.hin[idx] : (uint64_t)rec.h) : 0ull;
    }
    const bool counts = A.m != nullptr && blockIdx.x == 0u;
    uint64_t t = counts && rv ? (uint64_t)A.m[r] : 0ull;
    if (A.zero && rv) {
        const SumRec z = {0.0, 0, 0u};
#pragma unroll
        for (int j = 0; j < MERGE_COLS; ++j) {
            const uint32_t c = c0 + (uint32_t)j;
            if (c < A.ncols) A.zero[(size_t)r * A.row + c] = z;
        }
    }
    if (counts) {
        if (rv) A.m[r] = 0u;
#pragma unroll
        for (int lvl = 1; lvl < 64; lvl <<= 1) t += __shfl_xor(t, lvl, 64);
        if (lane == 0) tours[wave] = t;
    }
    // butterfly: after step lvl every lane holds the sum of its aligned block of
    // 2*lvl rows; the extended-range sum is commutative, so both lanes of a pair
    // compute the same (left block) + (right block)
#pragma unroll
    for (int lvl = 1; lvl < 64; lvl <<= 1) {
#pragma unroll
        for (int j = 0; j < MERGE_COLS; ++j) {
            XF o;
            o.m = __shfl_xor(v[j].m, lvl, 64);
            o.e = __shfl_xor(v[j].e, lvl, 64);
            v[j] = xf_add(v[j], o);
            h[j] += __shfl_xor(h[j], lvl, 64);
        }
    }
    // a column's sum of this block's rows, to its place
    auto leave = [&](uint32_t c, XF vv, uint64_t hh) INLINE {
        const size_t o = (size_t)blockIdx.y * A.row + c;
        if (A.accumulate) {
            vv = xf_add(xf_of(A.out[o]), vv);
            if (A.hout) hh += A.hout[o];
        }
        SumRec rec;
        rec.m = vv.m;
        rec.e = vv.e;
        rec.h = 0u;
        A.out[o] = rec;
        if (A.hout) A.hout[o] = hh;
    };
    if (lane < MERGE_COLS) {
        // select column `lane` without dynamic register indexing
        XF vv = {0.0, 0};
        uint64_t hh = 0;
#pragma unroll
        for (int j = 0; j < MERGE_COLS; ++j) {
            if (j == lane) { vv = v[j]; hh = h[j]; }
        }
        if (waves == 1) {
            // (a block of one wave has nothing to add up)
            if (c0 + (uint32_t)lane < A.ncols) leave(c0 + (uint32_t)lane, vv, hh);
        } else {
            SumRec rec;
            rec.m = vv.m;
            rec.e = vv.e;
            rec.h = 0u;
            part[lane * MERGE_WAVES + wave] = rec;
            parth[lane * MERGE_WAVES + wave] = hh;
        }
    }
    if (waves == 1) {
        if (counts && lane == 0)
            atomicAdd(reinterpret_cast<unsigned long long*>(A.MG), (unsigned long long)t);
        return;
    }
    __syncthreads();
    if (wave != 0) return;
    // the waves' sums: lane = 16 * (column & 3) + wave, four columns at a time
    const int w = lane & (MERGE_WAVES - 1);
#pragma unroll
    for (int j0 = 0; j0 < MERGE_COLS; j0 += 64 / MERGE_WAVES) {
        const int j = j0 + lane / MERGE_WAVES;
        XF vv = {0.0, 0};
        uint64_t hh = 0;
        if (w < waves) {
            vv = xf_of(part[j * MERGE_WAVES + w]);
            hh = parth[j * MERGE_WAVES + w];
        }
#pragma unroll
        for (int lvl = 1; lvl < MERGE_WAVES; lvl <<= 1) {
            XF o;
            o.m = __shfl_xor(vv.m, lvl, 64);
            o.e = __shfl_xor(vv.e, lvl, 64);
            vv = xf_add(vv, o);
            hh += __shfl_xor(hh, lvl, 64);
        }
        const uint32_t c = c0 + (uint32_t)j;
        if (w == 0 && c < A.ncols) leave(c, vv, hh);
    }
    if (counts && lane == 0) {
        uint64_t all = 0;
        for (int k = 0; k < waves; ++k) all += tours[k];
        atomicAdd(reinterpret_cast<unsigned long long*>(A.MG), (unsigned long long)all);
    }
}

__global__ void __launch_bounds__(256) merge_independent_kernel(SumRec* L, uint32_t* m, SumRec* G,
                                                                uint64_t* HG, uint64_t* MG,
                                                                uint32_t N, uint32_t row) {
    const size_t total = (size_t)N * row;
    const SumRec z = {0.0, 0, 0u};
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < total;
         i += (size_t)gridDim.x * 256) {
        const SumRec l = L[i];
        const XF g = xf_add(xf_of(G[i]), xf_of(l));
        SumRec rec;
        rec.m = g.m;
        rec.e = g.e;
        rec.h = 0u;
        G[i] = rec;
        HG[i] += l.h;
        L[i] = z;
    }
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < N; i += (size_t)gridDim.x * 256) {
        MG[i] += m[i];
        m[i] = 0u;
    }
}

// Group sums for the error estimate: lane k < 16 folds the records at n_max of
// sequences k, k + 16, k + 32, ... (in that order, from zero) and adds the
// result to the group's running total; tours likewise.  Runs before the merge
// that zeroes the records.
__global__ void __launch_bounds__(64) group_sums_kernel(const SumRec* L, const uint32_t* m,
                                                        uint32_t N, uint32_t row, uint32_t n_max,
                                                        SumRec* gsum, uint64_t* gtours) {
    const uint32_t k = threadIdx.x;
    if (k >= GROUPS) return;
    XF acc = {0.0, 0};
    uint64_t tours = 0;
    for (uint32_t s = k; s < N; s += GROUPS) {
        acc = xf_add(acc, xf_of(L[(size_t)s * row + n_max]));
        tours += m[s];
    }
    const XF g = xf_add(xf_of(gsum[k]), acc);
    SumRec r;
    r.m = g.m;
    r.e = g.e;
    r.h = 0u;
    gsum[k] = r;
    gtours[k] += tours;
}

__global__ void reset_ctrl_kernel(uint32_t* ctrl) {
    if (threadIdx.x == CTRL_QUEUE) ctrl[CTRL_QUEUE] = 0u;
}

// A new context's state in one launch: zeros from `zero` on, the digests among
// them (low word of statistics word ST_DIGEST) at the FNV-1a 32 offset basis, and
// the descriptor, which comes as an argument.  Two launches and a copy took 21.8 us
// of a small call's create, this 14.8 us.
__global__ void __launch_bounds__(256) init_state_kernel(uint32_t* zero, size_t words, size_t stats0,
                                                         size_t stats_words, ProblemDesc d,
                                                         ProblemDesc* desc) {
    const size_t desc0 = (size_t)((const uint32_t*)desc - zero);
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < words;
         i += (size_t)gridDim.x * 256) {
        if (i - desc0 < sizeof(ProblemDesc) / 4) continue;      // (inside the range)
        const size_t k = i - stats0;
        const bool digest = k < stats_words && is_digest_word(k);
        zero[i] = digest ? FNV_OFFSET : 0u;
    }
    if (blockIdx.x == 0u && threadIdx.x == 0u) *desc = d;
}

template <int D, int TS>
hipError_t launch_run_t(const RunArgs& a, uint32_t wgs, uint32_t lds, hipStream_t s) {
    hipLaunchKernelGGL((run_kernel<D, TS>), dim3(wgs), dim3(64), lds, s, a);
    return hipGetLastError();
}

template <int D, int TS>
hipError_t occupancy_t(uint32_t lds, int* blocks) {
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks, run_kernel<D, TS>, 64, lds);
}

}  // namespace

hipError_t launch_reset_ctrl(uint32_t* ctrl, hipStream_t s) {
    hipLaunchKernelGGL(reset_ctrl_kernel, dim3(1), dim3(64), 0, s, ctrl);
    return hipGetLastError();
}

hipError_t launch_init_state(void* zero_base, size_t zero_bytes, const uint64_t* stats, uint32_t N,
                             const ProblemDesc& d, ProblemDesc* desc, hipStream_t s) {
    const size_t words = zero_bytes / 4;
    uint32_t blocks = (uint32_t)((words + 255) / 256);
    if (blocks > 4096) blocks = 4096;
    if (blocks == 0) blocks = 1;
    const size_t stats0 = (size_t)((const uint32_t*)stats - (const uint32_t*)zero_base);
    hipLaunchKernelGGL(init_state_kernel, dim3(blocks), dim3(256), 0, s, (uint32_t*)zero_base, words,
                       stats0, (size_t)N * STATS_WORDS * 2u, d, desc);
    return hipGetLastError();
}

#define PPERM_TS_SWITCH(D, FN, ...)                                     \
    switch (team_lanes) {                                               \
        case 4: if (D == 2) return FN<2, 4>(__VA_ARGS__); break;        \
        case 8: return FN<D, 8>(__VA_ARGS__);                           \
        case 16: return FN<D, 16>(__VA_ARGS__);                         \
        case 32: return FN<D, 32>(__VA_ARGS__);                         \
        case 64: return FN<D, 64>(__VA_ARGS__);                         \
        default: break;                                                 \
    }

hipError_t launch_batch(const BatchArgs& b, uint32_t workgroups, uint32_t lds_bytes, hipStream_t s,
                        bool observables, bool long_walk) {
    const dim3 g(workgroups), t(64);
    if (long_walk && observables) hipLaunchKernelGGL(batch_long_obs_kernel, g, t, lds_bytes, s, b);
    else if (long_walk) hipLaunchKernelGGL(batch_long_kernel, g, t, lds_bytes, s, b);
    else if (observables) hipLaunchKernelGGL(batch_obs_kernel, g, t, lds_bytes, s, b);
    else hipLaunchKernelGGL(batch_kernel, g, t, lds_bytes, s, b);
    return hipGetLastError();
}

hipError_t launch_parts(const PartArgs& a, uint32_t workgroups, uint32_t lds_bytes, hipStream_t s, bool long_walk) {
    if (long_walk) hipLaunchKernelGGL(part_long_kernel, dim3(workgroups), dim3(64), lds_bytes, s, a);
    else hipLaunchKernelGGL(part_kernel, dim3(workgroups), dim3(64), lds_bytes, s, a);
    return hipGetLastError();
}

hipError_t launch_job(const JobArgs& a, uint32_t workgroups, uint32_t lds_bytes, hipStream_t s) {
    hipLaunchKernelGGL(job_kernel, dim3(workgroups), dim3(64), lds_bytes, s, a);
    return hipGetLastError();
}

hipError_t launch_job_check(const JobArgs& a, hipStream_t s) {
    const uint32_t blocks = (a.count + 255u) / 256u;
    hipLaunchKernelGGL(job_check_kernel, dim3(blocks ? blocks : 1u), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t job_occupancy(uint32_t lds_bytes, int* blocks_per_cu) {
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, job_kernel, 64, lds_bytes);
}

hipError_t launch_fill_zero(void* p, size_t bytes, hipStream_t s) {
    const size_t words = bytes / 4;
    if (words == 0) return hipSuccess;
    uint32_t blocks = (uint32_t)((words + 255) / 256);
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(fill_zero_kernel, dim3(blocks), dim3(256), 0, s, (uint32_t*)p, words);
    return hipGetLastError();
}

hipError_t batch_occupancy(uint32_t lds_bytes, int* blocks_per_cu, bool long_walk) {
    if (long_walk) return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, batch_long_kernel, 64, lds_bytes);
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, batch_kernel, 64, lds_bytes);
}

hipError_t launch_run(const RunArgs& a, uint32_t dim, uint32_t team_lanes, uint32_t workgroups,
                      uint32_t lds_bytes, hipStream_t s) {
    if (dim == 2) {
        PPERM_TS_SWITCH(2, launch_run_t, a, workgroups, lds_bytes, s)
    } else if (dim == 3) {
        PPERM_TS_SWITCH(3, launch_run_t, a, workgroups, lds_bytes, s)
    }
    return hipErrorInvalidValue;
}

hipError_t run_kernel_lds_ok(uint32_t dim, uint32_t team_lanes, uint32_t lds_bytes,
                             int* blocks_per_cu) {
    if (team_lanes == 64) return batch_occupancy(lds_bytes, blocks_per_cu);
    if (dim == 2) {
        PPERM_TS_SWITCH(2, occupancy_t, lds_bytes, blocks_per_cu)
    } else if (dim == 3) {
        PPERM_TS_SWITCH(3, occupancy_t, lds_bytes, blocks_per_cu)
    }
    return hipErrorInvalidValue;
}

hipError_t launch_merge_pass(const MergeArgs& a, hipStream_t s) {
    const uint32_t waves = (a.rows < a.block ? a.rows + 63u : a.block) / 64u;
    dim3 grid((a.ncols + MERGE_COLS - 1) / MERGE_COLS, (a.rows + a.block - 1) / a.block);
    hipLaunchKernelGGL(merge_pass_kernel, grid, dim3(64u * waves), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_group_sums(const SumRec* L, const uint32_t* m, uint32_t N, uint32_t row,
                             uint32_t n_max, SumRec* gsum, uint64_t* gtours, hipStream_t s) {
    hipLaunchKernelGGL(group_sums_kernel, dim3(1), dim3(64), 0, s, L, m, N, row, n_max, gsum, gtours);
    return hipGetLastError();
}

hipError_t launch_merge_independent(SumRec* L, uint32_t* m, SumRec* G, uint64_t* HG, uint64_t* MG,
                                    uint32_t N, uint32_t row, hipStream_t s) {
    size_t total = (size_t)N * row;
    uint32_t blocks = (uint32_t)((total + 255) / 256);
    if (blocks > 8192) blocks = 8192;
    hipLaunchKernelGGL(merge_independent_kernel, dim3(blocks), dim3(256), 0, s, L, m, G, HG, MG,
                       N, row);
    return hipGetLastError();
}

}  // namespace pperm

// Scratch of the allocation-free batched launch (pperm_run_batch_noalloc): the
// queue words of its launches, then one launch entry per problem.  Each device
// the library runs on holds its own copy for the life of the process; calls on
// one device share it.
static __device__ __align__(256) unsigned char
    scratch[pperm::NOALLOC_QUEUE_BYTES + pperm::NOALLOC_MAX_PROBLEMS * sizeof(pperm::LaunchEntry)];

// The device address of `scratch` on the current device, looked up once per
// device with that device current (the host-side name of the array is not a
// device address and must never reach a kernel or a copy).
hipError_t pperm::noalloc_scratch(void** ptr, size_t* bytes) {
    constexpr int kMaxDevices = 64;
    static std::mutex mu;
    static void* addr[kMaxDevices] = {};
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(mu);
    if (addr[dev] == nullptr) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        addr[dev] = p;
    }
    *ptr = addr[dev];
    *bytes = sizeof(scratch);
    return hipSuccess;
}
