// The reduced problem ("core") of one candidate, solved by one workgroup.  Included by
// spdy_dp.hip, inside its namespace.
//
// Eq. 1 is a multiple-choice knapsack problem.  For any multiplier lambda >= 0 the relaxed problem
// (pick in every layer the level with the least err + lambda * tau, subtract lambda * B) bounds
// every feasible profile from below, and a level whose excess over its layer's minimum is larger
// than the distance from that bound to the cost of a known profile lies on no optimal one
// (reduction by Lagrangian bounds: Dyer 1984, Zemel 1984; Pisinger 1995 for the core of a
// multiple-choice problem).  The same test on a partial profile discards cells of the table.
// On the tables this solver is for, one to three levels per layer and one to three hundred
// buckets of a row are left, out of some thirty levels and thousands of buckets, so Eq. 2 over
// what is left takes 10^4 updates where the whole table takes 10^7, in a few KB of LDS.
//
// Results are Alg. 1's, bit for bit, because only what can lie on NO profile of least fp32 cost is
// left out.  With errors >= 0 every partial sum of a profile P of least cost V is at most
// V <= U (U: the fp32 cost of a known profile), so each of its L - 1 rounded adds is off by at
// most hu = 2^-24 * 2^floor(log2 U), and in real numbers c(P) <= U + (L - 1) hu.  Levels and cells
// whose bound exceeds that are dropped, the bounds being formed in fp64 with a margin for its own
// rounding; every profile that ties for the least cost survives, so the smallest t of the
// argmin and the smallest level of each step of the walk back are found among the same
// candidates as in the whole table.
//
// What it does not take is left to the full table (profile[0] = kGivenUp): a negative or NaN error,
// a negative time, sums near the end of the fp32 range, more surviving levels, rows wider than both LDS
// and memory hold, or more work than the limits of the launch.
//
// What bounds it: latency; one wave per SIMD issues an instruction every seven or eight clocks whatever it
// is, so fewer instructions per pass and fewer passes are what counts, not bytes.  Thousands of clocks of a
// candidate by its own stamps, mean of 250 of L = 52, S = 42 (in all 62, the slowest 89): tables 5, the
// two ends 2, multiplier 15 (five passes over the table in LDS, each with four multipliers), known profile
// 13 (single exchanges, then pairs of them), survivors 7, then dependent steps for the reduced table 15
// (nine of them, 20 to 45 for the slowest candidates), walk back 5.
// us a call, mean of eight sets of inputs; with one multiplier a pass, exchanges one at a time and only rows of
// one chunk in a register, and now: K = 250 from an incumbent 75 and 47; K = 100, L = 52, S = 42, B = 10^4 93
// and 85; 384 solves under six budgets 74 and 52; K = 4096, L = 72, S = 40, B = 16384 291 and 236; K = 333,
// S = 127 109 and 68; K = 256, L = 200, S = 64, B = 65536 389 and 214.  The whole table takes 239 (resumed), 213,
// 184, 3130, 903 and 3830.  (The stamps are from before whole values were compared in the multiplier's
// passes, which takes as long.)

constexpr int16_t kGivenUp = -3;         // profile[0] of a candidate the full table has to solve
constexpr int kCoreThreads = 256;
constexpr int kCoreWaves = kCoreThreads / kWave;
constexpr int kCoreMaxLayers = kCoreThreads;
constexpr int kCoreMaxBudget = 1 << 22;  // times stay exact in fp32, a level and a shift in 32 bits
constexpr int kCoreShiftBits = 23;       // a shift is at most the budget
static_assert(kCoreMaxBudget < 1 << kCoreShiftBits && 255ull << kCoreShiftBits <= UINT32_MAX,
              "a level and a shift share a word");
constexpr int kCoreExtra = 128;          // levels beyond one per layer that are not worth halving
constexpr int kCorePairs = 128;          // exchanges of which all pairs are tried, and none
constexpr int kCoreNarrow = 2;           // chunks of a row that one wave does alone
constexpr int kCoreTrips = 5;            // attempts, counting a halving before the first (one is usual)
constexpr int kCoreBudgets = 64;         // budgets per launch
constexpr float kCoreFar = kCoreMaxBudget + 1;   // "time" of a level that may not be chosen
static_assert(kCoreMaxLayers * (long long)kCoreFar <= INT32_MAX, "times are summed in int");

struct CoreStep {        // a layer of the reduced problem with more than one level left
    int layer;
    int first, count;    // its entries in the list
    int span;            // largest shift among them
};
struct CoreEntry {       // a surviving level
    float err;
    uint32_t word;       // level << kCoreShiftBits | shift
};

struct CoreParams {
    int parts, parts_log2;       // threads per layer (a power of two <= 64)
    int per_part;        // levels per thread, a multiple of four (<= 128)
    int share_log2;      // the same of a wave that has all layers to itself
    int pad;             // levels per layer past the last one that are scanned with it
    int step_layers;     // kCoreThreads / S
    int pitch;           // levels per layer in LDS (odd, so that a column of levels is conflict-free)
    int window;          // buckets a row may span in LDS
    int record;          // bytes of LDS for the recorded entries
    int entries;         // room in the list
    int table_bytes;     // LDS of the staged tables; the rows and the record reuse it
    int work;            // sweeps of 64 buckets by one entry before a candidate is given up
    unsigned char *spill;        // rows that do not fit the LDS record, per candidate and budget
    long long spill_bytes;
    int far;                     // kFar: buckets of the two rows in memory, before each record there
    int budgets;                 // J
    int32_t budget[kCoreBudgets];
};

// Non-negative floats (or -0) order like their bits without the sign.
__device__ __forceinline__ unsigned magnitude(float x)
{
    return __builtin_bit_cast(unsigned, x) & 0x7FFFFFFFu;
}
__device__ __forceinline__ unsigned long long pair_key(unsigned high, unsigned low)
{
    return (unsigned long long)high << 32 | low;
}

// A row and a record in memory.  (A pointer that might also be one to LDS would be used by flat
// instructions, and the waits for LDS would wait for memory, too.)
using FarRow = __attribute__((address_space(1))) float *;
using FarBytes = __attribute__((address_space(1))) unsigned char *;

// Loads for the next trip of a loop, above this, are asked for in this trip.  (Where nothing is in the way the
// compiler makes one load of the first trip's and the later ones', at the head of the loop, and waits for it.)
__device__ __forceinline__ void stay_ahead() { asm volatile("" ::: "memory"); }

// a * b + c in a register of its own.  (In the one that c was read to, as the compiler does it, c's neighbours of the
// same read are moved out of the way as soon as they arrive, and waited for.)
__device__ __forceinline__ float fma_apart(float a, float b, float c)
{
    float sum;
    asm("v_fma_f32 %0, %1, %2, %3" : "=v"(sum) : "v"(a), "v"(b), "v"(c));
    return sum;
}

struct CoreBooks {       // where the steps of the reduced table have got to
    int m, a, b, used, spilled, first_spilled, work, prev, failed, wide;
};

struct CoreShared {      // static LDS of the kernel
    float2 sum[2][kCoreWaves];               // (err, tau) of a path, by wave; times as int bits
    float2 ends[2][kCoreWaves];              // the same of the least-time and the least-error path
    unsigned long long key[2][kCoreWaves];
    int2 change[2][kCoreWaves];              // of the wave's best exchange: error (bits), time
    int2 place[2][kCoreWaves];               // sums of the entries (and steps), of the times
    int2 live[2][kCoreWaves];                // first and last bucket of a row that matters
    double least[kCoreWaves];
    CoreBooks books;
};

// One candidate (error source `src` seen from candidate k) under budget B.  Returns through
// profile / cost; profile[0] = kGivenUp if the full table has to do it.  kFar: a row that spans more
// buckets than the window lies in memory, before the record that `spill` is for (wide steps end
// with a barrier, which makes them visible); otherwise it is too wide.
template <bool kFar>
__device__ __forceinline__ void solve_core(const int32_t *__restrict__ tau, const ErrSource src,
                                           int L, int S, int B, const CoreParams &cp,
                                           unsigned char *spill, unsigned char *lds,
                                           CoreShared &sh, int16_t *__restrict__ profile,
                                           float *__restrict__ cost)
{
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    float2 *const table = reinterpret_cast<float2 *>(lds);           // [L][pitch] (err, tau)
    CoreEntry *const list = reinterpret_cast<CoreEntry *>(lds + cp.table_bytes);
    double *const limit = reinterpret_cast<double *>(list + cp.entries);   // [L], see below
    CoreStep *const steps = reinterpret_cast<CoreStep *>(limit + ((L + 1) & ~1));  // [L]
    float *const single = reinterpret_cast<float *>(steps + L);      // [L]
    int *const row_at = reinterpret_cast<int *>(single + L);         // [L]

    // ---- the tables, coalesced, twelve loads in flight
    auto stage = [&]() __attribute__((always_inline)) {
        int bad = 0;
        constexpr int kLoads = 12;
        const int n = L * S;
        const int step_l = cp.step_layers, step_s = kCoreThreads - step_l * S;
        int l = tid / S, s = tid - l * S;
        for (int i0 = tid; i0 < n; i0 += kLoads * kCoreThreads) {
            float e[kLoads];
            int t[kLoads], at[kLoads];
#pragma unroll
            for (int j = 0; j < kLoads; ++j) {
                const int i = i0 + j * kCoreThreads;
                const bool in = i < n;
                at[j] = in ? l * cp.pitch + s : -1;
                e[j] = src.err ? src.err[in ? i : 0]
                               : __fmul_rn(src.c[in ? l : 0], src.w[in ? s : 0]);
                t[j] = tau[in ? i : 0];
                l += step_l;
                s += step_s;
                l += s >= S ? 1 : 0;
                s -= s >= S ? S : 0;
            }
#pragma unroll
            for (int j = 0; j < kLoads; ++j) {
                if (at[j] >= 0) {                 // (else past the end of the tables)
                    bad |= !(e[j] >= 0.0f) || t[j] < 0;
                    const bool out = t[j] > B || e[j] == __builtin_inff();
                    table[at[j]] = out ? make_float2(__builtin_inff(), kCoreFar)
                                       : make_float2(e[j], (float)t[j]);
                }
            }
        }
        for (int i = tid; i < L * cp.pad; i += kCoreThreads) {
            const int pl = i / cp.pad;
            table[pl * cp.pitch + S + (i - pl * cp.pad)] = make_float2(__builtin_inff(), kCoreFar);
        }
        return bad;
    };
    if (__syncthreads_or(stage())) {
        if (tid == 0)
            profile[0] = kGivenUp;
        return;
    }

    // Thread (layer, part) scans levels [s_begin, s_end) of its layer.
    const int parts = cp.parts;
    const int layer = tid >> cp.parts_log2, part = tid & (parts - 1);
    const bool in_layer = layer < L;
    const bool lead = in_layer && part == 0;
    const int s_begin = in_layer ? part * cp.per_part : 0;
    const float2 *const mine = table + (in_layer ? layer : 0) * cp.pitch;
    // f(err and tau, i) for this thread's levels s_begin + i, four at a time and the next four already on
    // their way (the last four once more at the end; per_part is a multiple of four).
    auto scan = [&](auto f) __attribute__((always_inline)) {
        const float2 *from = mine + s_begin;
        float2 v[4], next_v[4];
#pragma unroll
        for (int q = 0; q < 4; ++q)
            next_v[q] = from[q];
        for (int i = 0; i < cp.per_part; i += 4) {
#pragma unroll
            for (int q = 0; q < 4; ++q)
                v[q] = next_v[q];
            from += i + 4 < cp.per_part ? 4 : 0;
#pragma unroll
            for (int q = 0; q < 4; ++q)
                next_v[q] = from[q];
            stay_ahead();
#pragma unroll
            for (int q = 0; q < 4; ++q)
                f(v[q], i + q);
        }
    };
    int turn = 0;                                 // which half of the double-buffered words
    // ---- the two ends of the multiplier's range: least error (lambda = 0), least time
    float lo_e, lo_t, hi_e, hi_t;                 // (err, tau) of this layer on either path
    float c_lo, c_hi;
    int t_lo, t_hi;
    {
        unsigned long long by_err = ~0ull, by_time = ~0ull;
        scan([&](float2 v, int) {
            by_err = Smaller{}(by_err, pair_key(magnitude(v.x), magnitude(v.y)));
            by_time = Smaller{}(by_time, pair_key(magnitude(v.y), magnitude(v.x)));
        });
        by_err = group_join(by_err, parts, Smaller{});
        by_time = group_join(by_time, parts, Smaller{});
        lo_e = __builtin_bit_cast(float, (unsigned)(by_err >> 32));
        lo_t = __builtin_bit_cast(float, (unsigned)by_err);
        hi_e = __builtin_bit_cast(float, (unsigned)by_time);
        hi_t = __builtin_bit_cast(float, (unsigned)(by_time >> 32));
        // both sums through one barrier
        const float he = from_lane(wave_scan(lead ? hi_e : 0.0f, 0.0f, Add{}), kWave - 1);
        const float le = from_lane(wave_scan(lead ? lo_e : 0.0f, 0.0f, Add{}), kWave - 1);
        const int ht = from_lane(wave_scan(lead ? (int)hi_t : 0, 0, Add{}), kWave - 1);
        const int lt = from_lane(wave_scan(lead ? (int)lo_t : 0, 0, Add{}), kWave - 1);
        if (lane == 0) {
            sh.ends[0][wave] = make_float2(he, __builtin_bit_cast(float, ht));
            sh.ends[1][wave] = make_float2(le, __builtin_bit_cast(float, lt));
        }
        __syncthreads();
        c_hi = c_lo = 0.0f;
        t_hi = t_lo = 0;
#pragma unroll
        for (int w = 0; w < kCoreWaves; ++w) {
            c_hi += sh.ends[0][w].x;
            t_hi += __builtin_bit_cast(int, sh.ends[0][w].y);
            c_lo += sh.ends[1][w].x;
            t_lo += __builtin_bit_cast(int, sh.ends[1][w].y);
        }
        c_hi = uniform(c_hi);
        c_lo = uniform(c_lo);
        t_hi = uniform(t_hi);
        t_lo = uniform(t_lo);
    }
    if (t_hi > B) {                               // also where a layer has no level to choose
        if (tid < L)
            profile[tid] = -1;
        if (tid == 0)
            *cost = __builtin_inff();
        return;
    }

    // ---- the best multiplier: the chord between the two paths, until no path lies below it
    float lambda_f = 0.0f;
    const bool fits = t_lo <= B;                  // the least-error profile meets the budget
    if (!fits) {
        // Four multipliers a pass, one a wave, a lane (or `share` lanes, where layers are few) per layer:
        // five passes, seven for deep networks, where one multiplier a pass took ten to fourteen.  The first
        // wave takes the chord, which decides when to stop; the others where the logarithm of the multiplier,
        // interpolated over the time, meets the budget, and on either side of that.  What a pass costs
        // is instructions: the least of all levels takes two a level, and only the four that it is among are
        // compared with it.  (Two multipliers per thread, layers split over all threads: six
        // passes, each longer by as much.)
        int2 *const picks = reinterpret_cast<int2 *>(steps);         // of the path above the budget, below it
        if (lead)
            picks[layer] = make_int2(-1, -1);
        const int share = 1 << cp.share_log2, of_wave = lane & (share - 1);
        const int levels = ((S + share - 1) / share + 3) & ~3;       // of a lane
        const unsigned long long before = ((1ull << of_wave) - 1ull) << (lane - of_wave);   // lanes of the same layer
        float lam_lo = 0.0f, lam_hi = __builtin_inff();
        for (int trip = 0; trip < 40; ++trip) {
            lambda_f = fmaxf(c_hi - c_lo, 0.0f) * __builtin_amdgcn_rcpf((float)(t_lo - t_hi));
            float lam = lambda_f;
            if (wave > 0) {
                if (lam_lo > 0.0f && lam_hi < __builtin_inff()) {
                    const float f = (float)(t_lo - B) * __builtin_amdgcn_rcpf((float)(t_lo - t_hi));
                    const float x = wave == 1 ? f : (wave == 2 ? 0.8f * f : 0.2f + 0.8f * f);
                    lam = lam_lo * __builtin_amdgcn_exp2f(
                                       x * __builtin_amdgcn_logf(lam_hi * __builtin_amdgcn_rcpf(lam_lo)));
                } else {
                    lam *= wave == 1 ? 0.4f : (wave == 2 ? 0.15f : 2.0f);
                }
                lam = fminf(fmaxf(lam, lam_lo), lam_hi);
            }
            float ce = 0.0f;
            int ct = 0, pick[kCoreMaxLayers / kWave];
#pragma unroll
            for (int b = 0; b < kCoreMaxLayers / kWave; ++b) {
                if (b * kWave >= L)
                    break;
                const int layer_b = b * kWave + (lane >> cp.share_log2);
                const float2 *const row = table + min(layer_b, L - 1) * cp.pitch;
                const int start = of_wave * levels;
                // Eight levels a trip (the last four may be the ones before once more); the next
                // trip's are asked for as soon as this trip's have been used, into the same registers.
                const float2 *const from = row + start;
                auto cost_of = [&](float2 v) __attribute__((always_inline)) {
                    return fma_apart(lam, v.y, v.x);
                };
                float2 v[8];
                auto eight = [&](int i) __attribute__((always_inline)) {
#pragma unroll
                    for (int q = 0; q < 8; ++q)
                        v[q] = from[(q < 4 ? i : min(i + 4, levels - 4)) + (q & 3)];
                };
                float least_b = __builtin_inff();
                int at = 0;                       // the first of the four that it is among
                eight(0);
                int i = 0;
                do {
                    float r[8];
#pragma unroll
                    for (int q = 0; q < 8; ++q)
                        r[q] = cost_of(v[q]);
                    eight(min(i + 8, levels - 4));
                    stay_ahead();
                    const float low = min3(min3(r[0], r[1], r[2]), r[3], least_b);
                    at = low < least_b ? i : at;
                    least_b = min3(min3(r[4], r[5], r[6]), r[7], low);
                    at = least_b < low ? min(i + 4, levels - 4) : at;
                    i += 8;
                } while (i < levels);
                float2 found = from[at + 3];
                int place = start + at + 3;       // of the first level that is the least
#pragma unroll
                for (int q = 2; q >= 0; --q) {
                    const float2 one = from[at + q];
                    const bool is = cost_of(one) == least_b;
                    place = is ? start + at + q : place;
                    found.x = is ? one.x : found.x;
                    found.y = is ? one.y : found.y;
                }
                pick[b] = layer_b < L ? place : -1;
                if (__builtin_amdgcn_readfirstlane(share) > 1) {    // (see group_join)
                    const unsigned own = magnitude(least_b);
                    const bool is = own == group_join(own, share, Smaller{});
                    pick[b] = is && !(__ballot(is) & before) ? pick[b] : -1;
                }
                const bool counts = pick[b] >= 0;
                ce += counts ? found.x : 0.0f;
                ct += counts ? (int)found.y : 0;
            }
            ce = wave_scan(ce, 0.0f, Add{});
            ct = wave_scan(ct, 0, Add{});
            if (lane == kWave - 1) {
                sh.sum[turn][wave] = make_float2(ce, __builtin_bit_cast(float, ct));
                sh.change[turn][wave].x = __builtin_bit_cast(int, lam);
            }
            __syncthreads();
            // lane w holds what wave w found: of the paths that meet the budget the slowest, of the others the
            // fastest, where these are nearer than the ones known
            static_assert(kCoreWaves == 4, "a quad of lanes");
            const float2 sum_w = sh.sum[turn][lane & 3];
            const float lam_w = __builtin_bit_cast(float, sh.change[turn][lane & 3].x);
            const int t_w = __builtin_bit_cast(int, sum_w.y);
            const int t_chord = __builtin_amdgcn_readfirstlane(t_w);
            if (!(t_chord > t_hi && t_chord < t_lo))
                break;
            static_assert(kCoreMaxLayers * (long long)kCoreMaxBudget <= 1 << 30, "a time and a wave share a word");
            const unsigned time_wave = min((unsigned)t_w, (1u << 30) - 1) << 2 | (lane & 3);
            const unsigned under = t_w <= B ? time_wave : 0u, over = t_w <= B ? ~0u : time_wave;
            const unsigned best_hi = uniform(group_join(under, 4, Larger{}));
            const unsigned best_lo = uniform(group_join(over, 4, Smaller{}));
            int hi_wave = -1, lo_wave = -1;
            if (best_hi >> 2 > (unsigned)t_hi) {
                hi_wave = best_hi & 3;
                t_hi = __builtin_amdgcn_readlane(t_w, hi_wave);
                c_hi = lane_value(sum_w.x, hi_wave);
                lam_hi = lane_value(lam_w, hi_wave);
            }
            if ((best_lo >> 2) < (unsigned)t_lo) {
                lo_wave = best_lo & 3;
                t_lo = __builtin_amdgcn_readlane(t_w, lo_wave);
                c_lo = lane_value(sum_w.x, lo_wave);
                lam_lo = lane_value(lam_w, lo_wave);
            }
            turn ^= 1;
#pragma unroll
            for (int b = 0; b < kCoreMaxLayers / kWave; ++b) {
                const int layer_b = b * kWave + (lane >> cp.share_log2);
                if (b * kWave < L && pick[b] >= 0) {
                    if (wave == lo_wave)
                        picks[layer_b].x = min(pick[b], S - 1);
                    if (wave == hi_wave)
                        picks[layer_b].y = min(pick[b], S - 1);
                }
            }
        }
        __syncthreads();                          // the paths are written, the words are read
        const int2 path = picks[in_layer ? layer : 0];
        const float2 lo = mine[max(path.x, 0)], hi = mine[max(path.y, 0)];
        lo_e = path.x >= 0 ? lo.x : lo_e;
        lo_t = path.x >= 0 ? lo.y : lo_t;
        hi_e = path.y >= 0 ? hi.x : hi_e;
        hi_t = path.y >= 0 ? hi.y : hi_t;
    }
    const double lambda = lambda_f;

    // ---- the Lagrangian bound at lambda, in fp64, and the best that one exchange makes of either path:
    // of the one below the budget, the level that saves most error and still meets it; of the one
    // above, the level that costs least and brings it there
    double least = __builtin_inf();               // min over the layer of err + lambda tau
    unsigned long long one_hi = ~0ull, one_lo = ~0ull;        // error and time
    {
        const float top_hi = hi_t + (float)(B - t_hi), top_lo = lo_t + (float)(B - t_lo);
        scan([&](float2 v, int) {
            least = Smaller{}(least, __builtin_fma(lambda, (double)v.y, (double)v.x));
            const unsigned long long o = pair_key(magnitude(v.x), magnitude(v.y));
            one_hi = v.y <= top_hi ? Smaller{}(one_hi, o) : one_hi;
            one_lo = v.y <= top_lo ? Smaller{}(one_lo, o) : one_lo;
        });
    }
    least = group_join(least, parts, Smaller{});
    one_hi = group_join(one_hi, parts, Smaller{});
    one_lo = group_join(one_lo, parts, Smaller{});
    auto error_of = [](unsigned long long key) { return __builtin_bit_cast(float, (unsigned)(key >> 32)); };
    auto time_of = [](unsigned long long key) { return __builtin_bit_cast(float, (unsigned)key); };
    const float with_hi = c_hi + (error_of(one_hi) - hi_e);
    const float with_lo = one_lo == ~0ull ? __builtin_inff() : c_lo + (error_of(one_lo) - lo_e);
    const bool from_lo = with_lo < with_hi;
    const unsigned long long one_key =            // about its cost, the layer's thread, the path
        lead ? pair_key(magnitude(fmaxf(from_lo ? with_lo : with_hi, 0.0f)), tid << 1 | (from_lo ? 1 : 0))
             : ~0ull;
    const double run_least = wave_scan(lead ? least : 0.0, 0.0, Add{});
    const unsigned long long run_one = wave_scan(one_key, ~0ull, Smaller{});
    if (lane == kWave - 1) {
        sh.least[wave] = run_least;
        sh.key[turn][wave] = run_one;
    }
    __syncthreads();
    double sum_least = 0.0, upto_least = run_least;
    unsigned long long known_key = ~0ull;
#pragma unroll
    for (int w = 0; w < kCoreWaves; ++w) {
        const double o = sh.least[w];
        upto_least += w < wave ? o : 0.0;
        sum_least += o;
        known_key = Smaller{}(known_key, sh.key[turn][w]);
    }
    sum_least = uniform(sum_least);
    known_key = uniform(known_key);
    const float known = __builtin_bit_cast(float, (unsigned)(known_key >> 32));
    turn ^= 1;
    const double relaxed = sum_least - lambda * B;

    // ---- a profile that meets the budget: from either path by the best exchange, or the best two
    // of levels whose excess a profile of the cost known so far can afford, all pairs of up to kCorePairs
    // of them; where there are more, of the nearest, and then once more from the profile found instead of
    // the path below the budget.  Its cost is the least there is for more than half of the candidates here,
    // and its distance from the bound a third of what the best exchanges one after the other leave (five
    // passes of 2900 clocks), so the table that is left has half the steps and a third of the rows at the
    // worst (searches of L = 52 - 54, S = 40 - 42: 88 - 300 row sweeps of 64 buckets before, 36 - 94 now).
    // A second time for all with many levels made the slowest of searches up to 5 % slower, none at all
    // up to 1.5 times.
    if (!fits) {
        struct Exchange {                         // against the path below the budget, and the one above
            float hi;
            uint32_t word_hi;                     // layer << 24 | time + kMiddle
            float lo;
            uint32_t word_lo;
        };
        constexpr int kMiddle = 1 << 23;
        static_assert(kCoreMaxBudget < kMiddle && kCoreMaxLayers <= 256, "a layer and a time share a word");
        Exchange *const exchange = reinterpret_cast<Exchange *>(list);
        const int room = min(kCorePairs, cp.entries / 2);     // (an entry of the list is half as large)
        float *const time_in = reinterpret_cast<float *>(row_at);        // beside `single`
        float cost_known = known;
        for (int round = 0; round < 2; ++round) {
            double affords = fmax((double)cost_known - relaxed, 0.0) * 1.0001;
            unsigned long long kept[2];
            int listed = 0, first_place = 0, all = 0;
            int trip = 0;
            for (;; ++trip) {
                const double keep_to = least + affords;
                int count = 0;
                kept[0] = kept[1] = 0;
                scan([&](float2 v, int i) {
                    const bool keep = __builtin_fma(lambda, (double)v.y, (double)v.x) <= keep_to;
                    const unsigned long long bit = keep ? 1ull << (i & 63) : 0ull;
                    kept[0] |= i < 64 ? bit : 0ull;
                    kept[1] |= i < 64 ? 0ull : bit;
                    count += keep ? 1 : 0;
                });
                const int of_layer = group_join(count, parts, Add{});
                listed = of_layer > 1 && in_layer ? count : 0;
                const int run = wave_scan(listed, 0, Add{});
                const int run_t = wave_scan(lead ? (int)hi_t : 0, 0, Add{});
                if (lane == kWave - 1)
                    sh.place[turn][wave] = make_int2(run, run_t);
                __syncthreads();
                first_place = run - listed;
                all = t_hi = 0;
#pragma unroll
                for (int w = 0; w < kCoreWaves; ++w) {
                    const int2 o = sh.place[turn][w];
                    first_place += w < wave ? o.x : 0;
                    all += o.x;
                    t_hi += o.y;
                }
                all = uniform(all);
                t_hi = uniform(t_hi);
                turn ^= 1;
                if (all < room || trip == 2)
                    break;
                affords *= fmin(0.5, 0.8 * room / all);
            }
            all = min(all, room - 1);             // (what there is no room for is left out)
            // calls f(level, place) for what this thread has listed
            auto for_listed = [&](auto f) __attribute__((always_inline)) {
                int place = first_place;
#pragma unroll
                for (int half = 0; half < 2; ++half) {
                    unsigned long long left = listed ? kept[half] : 0;
                    while (left) {
                        f(s_begin + 64 * half + __builtin_ctzll(left), place++);
                        left &= left - 1;
                    }
                }
            };
            for_listed([&](int level, int place) {
                const float2 v = mine[level];
                const uint32_t word = (uint32_t)layer << 24;
                if (place < all)
                    exchange[place] = Exchange{v.x - hi_e, word | (uint32_t)(kMiddle + (int)(v.y - hi_t)),
                                               v.x - lo_e, word | (uint32_t)(kMiddle + (int)(v.y - lo_t))};
            });
            if (tid == 0)                         // none: a pair with it is a single exchange
                exchange[all] = Exchange{0.0f, 0xFF000000u | kMiddle, 0.0f, 0xFF000000u | kMiddle};
            __syncthreads();
            // Lane j holds exchanges j and 64 + j; every wave pairs a fourth of all with them.
            Exchange own[2];
#pragma unroll
            for (int c = 0; c < 2; ++c)
                own[c] = exchange[min(c * kWave + lane, all)];
            constexpr int kOne = 1 << 17;         // the best exchange by itself
            float best = cost_known;
            int which = kOne;                     // or the two of a pair and (bit 16) the path
            auto pair_with = [&](auto ci, auto cj) __attribute__((always_inline)) {
                constexpr int kI = decltype(ci)::value, kJ = decltype(cj)::value;
                const unsigned layer_j = own[kJ].word_hi >> 24;
                const int hi_j = (int)(own[kJ].word_hi & 0xFFFFFF);
                const int lo_j = (int)(own[kJ].word_lo & 0xFFFFFF);
                const float with_hi_j = c_hi + own[kJ].hi, with_lo_j = c_lo + own[kJ].lo;
                for (int i = wave; i < min(kWave, all - kI * kWave); i += kCoreWaves) {
                    const unsigned word_hi = (unsigned)__builtin_amdgcn_readlane((int)own[kI].word_hi, i);
                    const unsigned word_lo = (unsigned)__builtin_amdgcn_readlane((int)own[kI].word_lo, i);
                    const int room_hi = B - t_hi + 2 * kMiddle - (int)(word_hi & 0xFFFFFF);
                    const int room_lo = B - t_lo + 2 * kMiddle - (int)(word_lo & 0xFFFFFF);
                    const bool two = layer_j != word_hi >> 24;    // (not twice the same layer)
                    const float cost_hi = with_hi_j + lane_value(own[kI].hi, i);
                    const float cost_lo = with_lo_j + lane_value(own[kI].lo, i);
                    const int pair = (kI * kWave + i) | kJ * kWave << 8;
                    const bool take_hi = two && hi_j <= room_hi && cost_hi < best;
                    best = take_hi ? cost_hi : best;
                    which = take_hi ? pair : which;
                    const bool take_lo = two && lo_j <= room_lo && cost_lo < best;
                    best = take_lo ? cost_lo : best;
                    which = take_lo ? pair | 1 << 16 : which;
                }
            };
            pair_with(Many<0>{}, Many<0>{});
            if (all >= kWave) {
                pair_with(Many<0>{}, Many<1>{});
                pair_with(Many<1>{}, Many<1>{});
            }
            const unsigned long long key =
                from_lane(wave_scan(pair_key(magnitude(fmaxf(best, 0.0f)),
                                             (unsigned)(which & kOne ? which : which + (lane << 8))),
                                    ~0ull, Smaller{}),
                          kWave - 1);
            if (lane == 0)
                sh.key[turn][wave] = key;
            __syncthreads();
            unsigned long long win = ~0ull;
#pragma unroll
            for (int w = 0; w < kCoreWaves; ++w)
                win = Smaller{}(win, sh.key[turn][w]);
            which = (int)uniform((unsigned)win);
            turn ^= 1;
            if (round == 0 || !(which & kOne)) {
                const bool lo_path = (which & kOne ? (int)known_key & 1 : which >> 16 & 1) != 0;
                // (what is no exchange is nobody's and in no layer)
                const int first = which & kOne ? all : which & 0xFF;
                const int second = which & kOne ? all : which >> 8 & 0xFF;
                const int first_layer = first < all ? (int)(exchange[first].word_hi >> 24) : -1;
                const int second_layer = second < all ? (int)(exchange[second].word_hi >> 24) : -1;
                if (lead && layer != first_layer && layer != second_layer) {
                    const bool changed = which & kOne && (int)((unsigned)known_key >> 1) == tid;
                    const unsigned long long one = lo_path ? one_lo : one_hi;
                    single[layer] = changed ? error_of(one) : (lo_path ? lo_e : hi_e);
                    time_in[layer] = changed ? time_of(one) : (lo_path ? lo_t : hi_t);
                }
                if (layer == first_layer || layer == second_layer)
                    for_listed([&](int level, int place) {
                        if (place < all && (place == first || place == second)) {
                            single[layer] = mine[level].x;
                            time_in[layer] = mine[level].y;
                        }
                    });
            }
            if (trip == 0 || round > 0)
                break;
            cost_known = __builtin_bit_cast(float, (unsigned)(uniform(win) >> 32));
            __syncthreads();                      // the profile is written, the exchanges are read
            c_hi = cost_known;
            hi_e = single[in_layer ? layer : 0];
            hi_t = time_in[in_layer ? layer : 0];
        }
    } else if (lead) {
        single[layer] = lo_e;
    }
    __syncthreads();                              // `single` is written, the exchanges are read
    // U: the profile's cost, summed as Alg. 1 does.  (A bound on that from `best` needs no sum over the layers,
    // 3000 clocks, but the distance from the relaxed problem is 10^-5 of the cost: twice the levels survived.)
    float upper = -0.0f;
    for (int base = 0; base < L; base += kWave) {
        const float e = base + lane < L ? single[base + lane] : -0.0f;   // (x + -0 is x)
        for (int i = 0; i < min(kWave, L - base); i += 8)
#pragma unroll
            for (int q = 0; q < 8; ++q)
                upper += lane_value(e, i + q);
    }
    const double hu = 0x1p-24 * (double)__builtin_bit_cast(
                                    float, __builtin_bit_cast(unsigned, upper) & 0x7F800000u);
    const double margin = 1e-11 * (sum_least + lambda * B + (double)upper);

    // ---- survivors: count, place, write
    // `target`: the cost a profile must not exceed to be looked for.  U is safe, and mostly the least cost or
    // near it.  Where it leaves very many levels it is not, and half the way from the bound to it is tried
    // first, which is as good as U if a profile of at most that cost turns up; if not, U comes next, or the
    // cost that did turn up.  (From 64 levels on, or where U's distance from the bound is mostly rounding, as
    // in deep networks, that finds one too seldom.)  What exceeds the limits of the launch is halved, too, and
    // then what lies between the half and that.
    double target = (double)upper, beyond = __builtin_inf();   // (beyond: exceeded the limits)
    bool first_try = target - relaxed > 8.0 * (L - 1) * hu;
    int work = 0;                                 // of all attempts
    auto halved = [&](double x) { return relaxed + 0.5 * (x - relaxed); };
    const bool in_range = upper < 1e38f && lambda_f < 1e30f;   // (false for a NaN, too)
    for (int trip = 0; trip < kCoreTrips && in_range; ++trip) {
        const double keep_to = least + (target + (L - 1) * hu - relaxed + margin);
        int count = 0, first_t = INT32_MAX, last_t = -1;
        unsigned long long kept[2] = {0, 0};      // bit i: level s_begin + i (per_part <= 128)
        scan([&](float2 v, int i) {
            const bool keep = __builtin_fma(lambda, (double)v.y, (double)v.x) <= keep_to;
            const unsigned long long bit = keep ? 1ull << (i & 63) : 0ull;
            kept[0] |= i < 64 ? bit : 0ull;
            kept[1] |= i < 64 ? 0ull : bit;
            count += keep ? 1 : 0;
            first_t = keep ? min(first_t, (int)v.y) : first_t;
            last_t = keep ? max(last_t, (int)v.y) : last_t;
        });
        const int of_layer = group_join(count, parts, Add{});
        first_t = group_join(first_t, parts, Smaller{});
        last_t = group_join(last_t, parts, Larger{});
        // sums over the threads up to this one: entries of the layers that have more than one, with
        // these layers above bit 16; smallest times
        const bool is_step = lead && of_layer > 1;
        const int listed = (of_layer > 1 && in_layer ? count : 0) + (is_step ? 1 << 16 : 0);
        const int run = wave_scan(listed, 0, Add{});
        const int run_t = wave_scan(lead ? first_t : 0, 0, Add{});
        if (lane == kWave - 1)
            sh.place[turn][wave] = make_int2(run, run_t);
        __syncthreads();
        int before = run - listed, all = 0, upto_t = run_t, base_t = 0;
#pragma unroll
        for (int w = 0; w < kCoreWaves; ++w) {
            const int2 o = sh.place[turn][w];
            before += w < wave ? o.x : 0;
            upto_t += w < wave ? o.y : 0;
            all += o.x;
            base_t += o.y;
        }
        all = uniform(all);
        base_t = uniform(base_t);
        turn ^= 1;
        const int total = all & 0xFFFF, nsteps = all >> 16;
        if (first_try && total - nsteps > kCoreExtra) {
            first_try = false;
            target = halved(target);
            continue;
        }
        first_try = false;
        bool wide = total > cp.entries;           // exceeds the limits
        bool failed = wide || base_t > B;
        int place = before & 0xFFFF;
        if (!failed) {
            if (lead) {
                // a partial profile of layers 0..l with fp32 cost D at time t can only be completed
                // to a cost of at most `target` if D + lambda t <= target + (L - 1 - l) hu +
                // lambda B - (least values above); times count from the sum of the smallest ones
                limit[layer] = target + (L - 1 - layer) * hu + lambda * B -
                               (sum_least - upto_least) + margin - lambda * upto_t;
                if (is_step)
                    steps[before >> 16] = CoreStep{layer, place, of_layer, last_t - first_t};
            }
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                unsigned long long left = in_layer ? kept[half] : 0;
                while (left) {
                    const int s = s_begin + 64 * half + __builtin_ctzll(left);
                    const float2 v = mine[s];
                    left &= left - 1;
                    if (of_layer == 1) {          // this level it is
                        single[layer] = v.x;
                        profile[layer] = (int16_t)s;
                    } else {
                        list[place++] = CoreEntry{v.x, (uint32_t)s << kCoreShiftBits |
                                                           (uint32_t)((int)v.y - first_t)};
                    }
                }
            }
        }
        __syncthreads();

        // ---- Eq. 2 on what is left: two alternating rows over the staged tables' LDS
        // A layer with one level left adds its error to every bucket and shifts nothing: the layers
        // between two steps are added to the row of the step before them, in order.  A step's
        // chunks of 64 buckets are divided among the waves; every wave keeps the same books.
        float *const row0 = reinterpret_cast<float *>(lds), *const row1 = row0 + cp.window;
        unsigned char *const rec = lds + 2 * cp.window * sizeof(float);
        const int budget = B - base_t;            // buckets are counted from the smallest times
        int held_at = 0;                          // lane i holds `single` of layer held_at + i
        float held = lane < L ? single[lane] : 0.0f;
        auto single_of = [&](int l) __attribute__((always_inline)) {
            if ((l & ~(kWave - 1)) != held_at) {
                held_at = l & ~(kWave - 1);
                held = held_at + lane < L ? single[held_at + lane] : 0.0f;
            }
            return lane_value(held, l & (kWave - 1));
        };
        auto add_singles = [&](float v, int from, int to) __attribute__((always_inline)) {
            for (int l = from; l < to; ++l)
                v += single_of(l);
            return v;
        };
        auto none = []() __attribute__((always_inline)) { return CoreEntry{__builtin_inff(), 0}; };
        // lane i holds step base_step + i
        int base_step = 0;
        CoreStep held_step{L, 0, 0, 0};
        double held_limit = 0.0;
        auto load_steps = [&](int base) __attribute__((always_inline)) {
            base_step = base;
            const int i = base + lane;
            held_step = i < nsteps ? steps[i] : CoreStep{L, 0, 0, 0};
            // the layers up to the next step are added to this step's row before it is judged
            const int until = i + 1 < nsteps ? steps[i + 1].layer : L;
            held_step.layer |= until << 16;
            held_limit = limit[until - 1];
        };
        float *prev = row0;
        int far_prev = -1;                        // where the previous row is, if it lies in memory
        auto far_row = [&](int at) __attribute__((always_inline)) {
            return (FarRow) reinterpret_cast<float *>(spill) - 2 * cp.far + at;
        };
        int a = 0, b = 0;                         // buckets of the previous row that still matter
        int used = 0, spilled = 0, first_spilled = nsteps;
        CoreEntry next = none();
        if (!failed) {
            load_steps(0);
            const float v = add_singles(-0.0f, 0, nsteps ? __builtin_amdgcn_readlane(
                                                               held_step.layer, 0) & 0xFFFF
                                                         : L);
            if (tid == 0)
                prev[0] = v;
            next = lane < total ? list[lane] : none();
        }
        __syncthreads();
        // The best of n entries, in order, for bucket a + x; `en`: lane i holds entry i.
        auto visit = [&](auto row, CoreEntry en, int i, int x, unsigned reach, int index, float &best,
                         int &arg, auto width) __attribute__((always_inline)) {
            constexpr int kMany = decltype(width)::value;
            const int shift = (int)(en.word & ((1u << kCoreShiftBits) - 1u));
            float p[kMany];
#pragma unroll
            for (int q = 0; q < kMany; ++q) {
                const int u = x - __builtin_amdgcn_readlane(shift, i + q);
                const bool ok = (unsigned)u <= reach;
                const float d = row[ok ? u : 0];
                p[q] = (ok ? d : __builtin_inff()) + lane_value(en.err, i + q);
            }
#pragma unroll
            for (int q = 0; q < kMany; ++q) {
                const bool take = p[q] < best;
                best = take ? p[q] : best;
                arg = take ? index + q : arg;
            }
        };
        int m = 0;
        // Steps whose rows fit one chunk, most of them, by one wave: the row stays in a register, lane
        // `off` + x holding bucket a + x, and entries fetch their cells from other lanes.  What bounds a
        // step is the number of instructions one wave issues one after the other; here there is no row to
        // write and read again, no choice of where it lies, and half the branches.  Takes at least
        // the step that the caller has looked at; the row is left in LDS.  us a call, with the walk back
        // in registers, before and after: K = 64 under six budgets, L = 54, S = 40: 79.2 and 76.4;
        // K = 4096, L = 72: 302 and 290; K = 100, L = 52 (wide rows): 74.0 and 73.1.
        auto one_chunk = [&]() __attribute__((always_inline)) {
            float row = prev[min(lane, b - a)];
            int off = 0;
            for (;;) {
                if (m - base_step >= kWave)
                    load_steps(m);
                const int i_m = m - base_step;
                const int n = __builtin_amdgcn_readlane(held_step.count, i_m);
                const int top = min(b + __builtin_amdgcn_readlane(held_step.span, i_m), budget);
                const int width = top - a + 1;
                if (width > kWave || n > kWave || used + width > cp.record || work + n > cp.work)
                    break;
                const int first = __builtin_amdgcn_readlane(held_step.first, i_m);
                const int layers_m = __builtin_amdgcn_readlane(held_step.layer, i_m);
                const double lim = from_lane(held_limit, i_m);
                const CoreEntry en = lane < n ? next : none();
                const int follow = first + n + lane;
                next = follow < total ? list[follow] : none();
                work += n;
                row_at[m] = used - a;             // (every lane, the same)
                const int shift = (int)(en.word & ((1u << kCoreShiftBits) - 1u));
                const unsigned reach = (unsigned)(b - a);
                float best = __builtin_inff();
                int arg = 0;
                auto some = [&](int i, auto many) __attribute__((always_inline)) {
                    constexpr int kMany = decltype(many)::value;
                    float v[kMany];
#pragma unroll
                    for (int q = 0; q < kMany; ++q) {
                        const int u = lane - __builtin_amdgcn_readlane(shift, i + q);
                        const float d = __builtin_bit_cast(
                            float, __builtin_amdgcn_ds_bpermute((u + off) * 4,
                                                                __builtin_bit_cast(int, row)));
                        v[q] = ((unsigned)u <= reach ? d : __builtin_inff()) +
                               lane_value(en.err, i + q);
                    }
#pragma unroll
                    for (int q = 0; q < kMany; ++q) {
                        const bool take = v[q] < best;
                        best = take ? v[q] : best;
                        arg = take ? i + q : arg;
                    }
                };
                if (n <= 2)
                    some(0, Many<2>{});
                else
                    for (int i = 0; i < n; i += 4)
                        some(i, Many<4>{});
                best = add_singles(best, (layers_m & 0xFFFF) + 1, layers_m >> 16);
                const bool in = lane < width;
                if (in)
                    rec[used + lane] = (unsigned char)arg;
                const unsigned long long set = __ballot(
                    in && __builtin_fma(lambda, (double)(a + lane), (double)best) <= lim);
                used += width;
                row = best;
                ++m;
                if (set == 0) {                   // no profile costs as little as `target`
                    failed = true;
                    break;
                }
                off = __builtin_ctzll(set);
                b = a + 63 - __builtin_clzll(set);
                a += off;
                if (m == nsteps)
                    break;
            }
            float *const to = prev >= row1 ? row0 : row1;
            to[lane] = row;
            prev = to + off;
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
        };
        // The same for rows of two chunks, in two registers: `off` + x is the place of bucket a + x in both. A
        // cell and the one 64 buckets above lie in the same lane, so an entry takes two exchanges.  Thousands of
        // clocks of the slowest candidate, mean of eight seeds, through LDS and so: K = 256, L = 200, S = 64
        // (the mean candidate's 109 steps: 239 and 156) 607 and 536; K = 250, L = 52, S = 42 115 and 100; 384
        // solves under six budgets 119 and 106; K = 4096, L = 72 206 and 184; K = 100 204 and 199.
        auto two_chunks = [&]() __attribute__((always_inline)) {
            float row0_v = prev[min(lane, b - a)], row1_v = prev[min(kWave + lane, b - a)];
            int off = 0;
            for (;;) {
                if (m - base_step >= kWave)
                    load_steps(m);
                const int i_m = m - base_step;
                const int n = __builtin_amdgcn_readlane(held_step.count, i_m);
                const int top = min(b + __builtin_amdgcn_readlane(held_step.span, i_m), budget);
                const int width = top - a + 1;
                if (width <= kWave || width > 2 * kWave || n > kWave || used + width > cp.record ||
                    work + 2 * n > cp.work)
                    break;
                const int first = __builtin_amdgcn_readlane(held_step.first, i_m);
                const int layers_m = __builtin_amdgcn_readlane(held_step.layer, i_m);
                const double lim = from_lane(held_limit, i_m);
                const CoreEntry en = lane < n ? next : none();
                const int follow = first + n + lane;
                next = follow < total ? list[follow] : none();
                work += 2 * n;
                row_at[m] = used - a;             // (every lane, the same)
                const int shift = (int)(en.word & ((1u << kCoreShiftBits) - 1u));
                const int reach = b - a;
                float best0 = __builtin_inff(), best1 = __builtin_inff();
                int arg0 = 0, arg1 = 0;
                const int at = lane + off;
                auto some = [&](int i, auto many) __attribute__((always_inline)) {
                    constexpr int kMany = decltype(many)::value;
                    float v0[kMany], v1[kMany];
#pragma unroll
                    for (int q = 0; q < kMany; ++q) {
                        const int by = __builtin_amdgcn_readlane(shift, i + q);
                        const int u = lane - by, place = at - by;
                        const float x0 = __builtin_bit_cast(
                            float, __builtin_amdgcn_ds_bpermute(place * 4, __builtin_bit_cast(int, row0_v)));
                        const float x1 = __builtin_bit_cast(
                            float, __builtin_amdgcn_ds_bpermute(place * 4, __builtin_bit_cast(int, row1_v)));
                        const float err = lane_value(en.err, i + q);
                        const float d0 = place < kWave ? x0 : x1, d1 = place < 0 ? x0 : x1;
                        v0[q] = ((unsigned)u <= (unsigned)reach ? d0 : __builtin_inff()) + err;
                        v1[q] = ((unsigned)(u + kWave) <= (unsigned)reach ? d1 : __builtin_inff()) + err;
                    }
#pragma unroll
                    for (int q = 0; q < kMany; ++q) {
                        const bool take0 = v0[q] < best0, take1 = v1[q] < best1;
                        best0 = take0 ? v0[q] : best0;
                        arg0 = take0 ? i + q : arg0;
                        best1 = take1 ? v1[q] : best1;
                        arg1 = take1 ? i + q : arg1;
                    }
                };
                for (int i = 0; i < n; i += 2)
                    some(i, Many<2>{});
                for (int l = (layers_m & 0xFFFF) + 1; l < layers_m >> 16; ++l) {
                    const float single_l = single_of(l);
                    best0 += single_l;
                    best1 += single_l;
                }
                const bool in1 = kWave + lane < width;
                rec[used + lane] = (unsigned char)arg0;
                if (in1)
                    rec[used + kWave + lane] = (unsigned char)arg1;
                const unsigned long long set0 = __ballot(
                    __builtin_fma(lambda, (double)(a + lane), (double)best0) <= lim);
                const unsigned long long set1 = __ballot(
                    in1 && __builtin_fma(lambda, (double)(a + kWave + lane), (double)best1) <= lim);
                used += width;
                row0_v = best0;
                row1_v = best1;
                ++m;
                if ((set0 | set1) == 0) {         // no profile costs as little as `target`
                    failed = true;
                    break;
                }
                off = set0 ? __builtin_ctzll(set0) : kWave + __builtin_ctzll(set1);
                b = a + (set1 ? 2 * kWave - 1 - __builtin_clzll(set1) : kWave - 1 - __builtin_clzll(set0));
                a += off;
                if (m == nsteps)
                    break;
            }
            float *const to = prev >= row1 ? row0 : row1;
            to[lane] = row0_v;
            to[kWave + lane] = row1_v;
            prev = to + off;
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
        };
        while (m < nsteps && !failed) {
            // One step.  A row of one or two chunks is done by wave 0 alone, as are the narrow ones
            // after it, without a barrier: the others wait for where it has got to.
            bool alone = false;
            for (;;) {
                if (m - base_step >= kWave)
                    load_steps(m);
                const int i_m = m - base_step;
                const int n = __builtin_amdgcn_readlane(held_step.count, i_m);
                const int first = __builtin_amdgcn_readlane(held_step.first, i_m);
                const int span = __builtin_amdgcn_readlane(held_step.span, i_m);
                const int layers_m = __builtin_amdgcn_readlane(held_step.layer, i_m);
                const double lim = from_lane(held_limit, i_m);
                const int top = min(b + span, budget);
                const int width = top - a + 1;
                const int chunks = (width + kWave - 1) / kWave;
                const bool narrow = chunks <= kCoreNarrow;
                if (alone && !narrow)
                    break;
                if (narrow && wave != 0) {
                    alone = true;
                    break;
                }
                alone = narrow;
                if ((!kFar || far_prev < 0) && narrow && n <= kWave && first_spilled == nsteps &&
                    used + width <= cp.record && work + n * chunks <= cp.work &&
                    chunks * kWave <= cp.window) {
                    if (chunks == 1)
                        one_chunk();
                    else
                        two_chunks();
                    if (failed || m == nsteps)
                        break;
                    continue;
                }
                const CoreEntry held_entry = lane < n ? next : none();
                const int follow = first + n + lane;   // the next step's entries
                next = follow < total ? list[follow] : none();
                work += n * chunks;
                const bool spills = first_spilled < nsteps || used + width > cp.record;
                const bool to_far = kFar && width > cp.window;
                if (width > (to_far ? cp.far : cp.window) || work > cp.work ||
                    (spills && spilled + width > cp.spill_bytes)) {
                    failed = wide = true;
                    break;
                }
                const int out = spills ? spilled : used;
                first_spilled = spills ? min(first_spilled, m) : first_spilled;
                if (tid == 0)
                    row_at[m] = out - a;
                spilled += spills ? width : 0;
                used += spills ? 0 : width;
                float *const cur = prev >= row1 ? row0 : row1;
                const int far_cur = far_prev >= 0 && far_prev < cp.far ? cp.far : 0;
                const unsigned reach = (unsigned)(b - a);
                int low = INT32_MAX, high = -1;   // live buckets of the new row, from a
                for (int c = narrow ? 0 : wave; c < chunks; c += narrow ? 1 : kCoreWaves) {
                    const int x = c * kWave + lane;
                    float best = __builtin_inff();
                    int arg = 0;
                    auto visit_all = [&](auto row) __attribute__((always_inline)) {
                        for (int blk = 0; blk < n; blk += kWave) {
                            CoreEntry en = held_entry;
                            if (blk > 0)
                                en = blk + lane < n ? list[first + blk + lane] : none();
                            for (int i = 0; i < min(kWave, n - blk); i += 4)
                                visit(row, en, i, x, reach, blk + i, best, arg, Many<4>{});
                        }
                    };
                    if (kFar && far_prev >= 0) {
                        visit_all(far_row(far_prev));
                    } else if (n <= 2) {
                        visit(prev, held_entry, 0, x, reach, 0, best, arg, Many<2>{});
                    } else if constexpr (kFar) {
                        visit_all(prev);
                    } else {                      // (as visit_all; through it 2 - 3 % slower at L = 10)
                        for (int blk = 0; blk < n; blk += kWave) {
                            CoreEntry en = held_entry;
                            if (blk > 0)
                                en = blk + lane < n ? list[first + blk + lane] : none();
                            for (int i = 0; i < min(kWave, n - blk); i += 4)
                                visit(prev, en, i, x, reach, blk + i, best, arg, Many<4>{});
                        }
                    }
                    best = add_singles(best, (layers_m & 0xFFFF) + 1, layers_m >> 16);
                    const bool in = x < width;
                    if (in) {
                        if (kFar && to_far)
                            far_row(far_cur)[x] = best;
                        else
                            cur[x] = best;
                        if (spills)
                            ((FarBytes)spill)[out + x] = (unsigned char)arg;
                        else
                            rec[out + x] = (unsigned char)arg;
                    }
                    const bool live =
                        in && __builtin_fma(lambda, (double)(a + x), (double)best) <= lim;
                    const unsigned long long set = __ballot(live);
                    if (set) {
                        low = min(low, c * kWave + __builtin_ctzll(set));
                        high = c * kWave + 63 - __builtin_clzll(set);
                    }
                }
                if (!narrow) {
                    if (lane == 0)
                        sh.live[turn][wave] = make_int2(low, high);
                    __syncthreads();
#pragma unroll
                    for (int w = 0; w < kCoreWaves; ++w) {
                        const int2 o = sh.live[turn][w];
                        low = min(low, o.x);
                        high = max(high, o.y);
                    }
                    turn ^= 1;
                    low = __builtin_amdgcn_readfirstlane(low);
                    high = __builtin_amdgcn_readfirstlane(high);
                }
                ++m;
                if (high < 0) {                   // no profile costs as little as `target`
                    failed = true;
                    break;
                }
                b = a + high;
                a = a + low;
                if constexpr (kFar)
                    far_prev = to_far ? far_cur + low : -1;
                if (!kFar || !to_far)
                    prev = cur + low;
                if (!narrow || m == nsteps)
                    break;
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                __builtin_amdgcn_wave_barrier();
            }
            if (alone) {                          // the same in every wave
                if (tid == 0)
                    sh.books = CoreBooks{m, a, b, used, spilled, first_spilled, work,
                                         (int)(prev - row0), failed ? 1 : 0, wide ? 1 : 0};
                __syncthreads();
                const CoreBooks books = sh.books;
                m = uniform(books.m);
                a = uniform(books.a);
                b = uniform(books.b);
                used = uniform(books.used);
                spilled = uniform(books.spilled);
                first_spilled = uniform(books.first_spilled);
                work = uniform(books.work);
                prev = row0 + uniform(books.prev);
                far_prev = -1;                    // (narrow rows fit the window)
                failed = uniform(books.failed) != 0;
                wide = uniform(books.wide) != 0;
                if (m < nsteps && !failed) {
                    if (m - base_step >= kWave)
                        load_steps(m);
                    const int at = __builtin_amdgcn_readlane(held_step.first, m - base_step) + lane;
                    next = at < total ? list[at] : none();
                }
                __syncthreads();                  // the books may be written again
            }
        }

        // ---- least cost, smallest time among equals, then the walk back
        unsigned long long key = ~0ull;
        if (!failed) {
            for (int x = lane; x <= b - a; x += kWave)
                key = Smaller{}(key, pair_key(magnitude(kFar && far_prev >= 0 ? far_row(far_prev)[x] : prev[x]), x));
            key = from_lane(wave_scan(key, ~0ull, Smaller{}), kWave - 1);
            const unsigned at = (unsigned)key;
            // the sum over the profile in layer order
            const float value = uniform(kFar && far_prev >= 0 ? far_row(far_prev)[at] : prev[at]);
            failed = !((double)value <= target);
            if (!failed) {
                if (wave != 0)
                    return;
                if (lane == 0)
                    *cost = value;
            } else {
                upper = fminf(upper, value);
            }
        }
        if (failed) {
            beyond = wide ? target : beyond;
            const double missed = target;
            target = wide ? halved(target) : fmin((double)upper, relaxed + 2.0 * (target - relaxed));
            if (!(target < beyond))               // between the one that found none and what is too much
                target = 0.5 * (missed + beyond);
            if (work > cp.work)
                break;
            __syncthreads();                      // every wave is through with the rows
            stage();
            __syncthreads();
            continue;
        }
        if (first_spilled < nsteps)
            __threadfence_block();
        int t = a + (int)(unsigned)key;
        for (int base = (nsteps - 1) & ~(kWave - 1); nsteps > 0 && base >= 0; base -= kWave) {
            // lane i holds step base + i, and what it chose
            const int n = min(kWave, nsteps - base);
            const CoreStep st = steps[min(base + lane, nsteps - 1)];
            const int at = row_at[min(base + lane, nsteps - 1)];
            auto words_of = [&](int i) __attribute__((always_inline)) {
                return list[min(__builtin_amdgcn_readlane(st.first, i) + lane, total - 1)].word;
            };
            uint32_t next_words = words_of(n - 1), chosen = 0;
            for (int i = n - 1; i >= 0; --i) {
                const uint32_t words = next_words;
                const int here = __builtin_amdgcn_readlane(at, i) + t;
                int e;
                if (base + i >= first_spilled)
                    e = __builtin_amdgcn_readfirstlane(((FarBytes)spill)[here]);
                else
                    e = __builtin_amdgcn_readfirstlane(rec[here]);
                if (i > 0)
                    next_words = words_of(i - 1);
                const uint32_t word =
                    e < kWave ? (uint32_t)__builtin_amdgcn_readlane((int)words, e)
                              : uniform(list[__builtin_amdgcn_readlane(st.first, i) + e].word);
                chosen = lane == i ? word : chosen;
                t -= (int)(word & ((1u << kCoreShiftBits) - 1u));
            }
            if (lane < n)
                profile[st.layer] = (int16_t)(chosen >> kCoreShiftBits);
        }
        return;
    }
    if (tid == 0)                                 // the same in every thread
        profile[0] = kGivenUp;
}
