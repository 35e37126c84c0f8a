// A few toy tables, solved in one launch.  Included by spdy_dp.hip, inside its namespace.
//
// What bounds the smallest calls is launches: reducing the tables, the fill and the walk back take 5, 8 and
// 6 us for L = S = 8, B = 256, nearly all of it latency between and within three kernels.  Here a workgroup
// has a candidate to itself, with its tables, two rows and the level of every cell in LDS, and does the
// whole of Alg. 1 as it stands: nothing is subtracted from the times, a thread takes every so many-th
// bucket, levels in index order with a strict "<", one barrier a layer, then the argmin and the walk.
// Shift and error of a level are the same for all lanes: lane s of a wave holds those of level s.

constexpr int kSmallThreads = 1024;
constexpr int kSmallLds = 60 * 1024;  // (no attribute to set before the launch)

struct SmallShared {
    float best[kSmallThreads / kWave];
    int time[kSmallThreads / kWave];
    int end;
};

// Buckets of a row, whole waves; LDS of a workgroup.
__host__ __device__ constexpr int small_row(int B) { return (B + kWave) / kWave * kWave; }
constexpr size_t small_lds(int L, int S, int B)
{
    return (size_t)L * S * sizeof(int2) + (size_t)small_row(B) * (2 * sizeof(float) + (size_t)L);
}

__global__ __launch_bounds__(kSmallThreads) void dp_small(const int32_t *__restrict__ tau, ErrSource src,
                                                          int L, int S, int B,
                                                          int16_t *__restrict__ profile,
                                                          float *__restrict__ cost,
                                                          int32_t *__restrict__ has_table)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char small_bytes[];
    __shared__ SmallShared sh;
    const int k = blockIdx.x, tid = threadIdx.x, threads = blockDim.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave), waves = threads / kWave;
    const int cells = small_row(B);
    int2 *const table = reinterpret_cast<int2 *>(small_bytes);       // [L][S] time, error
    float *prev = reinterpret_cast<float *>(table + L * S), *cur = prev + cells;
    unsigned char *const rec = reinterpret_cast<unsigned char *>(cur + cells);       // [L][cells]
    const ErrSource mine = src.of_candidate(k, L, S);
    if (k == 0 && tid == 0)
        *has_table = 0;                           // the workspace holds none
    for (int i = tid; i < L * S; i += threads) {
        const int l = i / S;
        table[i] = make_int2(tau[i], __float_as_int(mine.layer(l, S).at(i - l * S)));
    }
    for (int t = tid; t < cells; t += threads)
        prev[t] = t == 0 ? -0.0f : __builtin_inff();
    __syncthreads();

    int2 level = lane < S ? table[lane] : make_int2(INT32_MAX, 0);
    for (int l = 0; l < L; ++l) {
        const int2 now = level;
        if (l + 1 < L && lane < S)
            level = table[(l + 1) * S + lane];
        for (int t = tid; t < cells; t += threads) {
            float best = __builtin_inff();
            int arg = 0;
            for (int s = 0; s < S; s += 4) {      // (lanes past the last level hold a time that never fits)
                float v[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const unsigned u = (unsigned)t - (unsigned)__builtin_amdgcn_readlane(now.x, s + q);
                    const bool fits = u <= (unsigned)t;
                    const float d = prev[fits ? u : 0];
                    v[q] = (fits ? d : __builtin_inff()) +
                           __int_as_float(__builtin_amdgcn_readlane(now.y, s + q));
                }
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const bool take = v[q] < best;
                    best = take ? v[q] : best;
                    arg = take ? s + q : arg;
                }
            }
            cur[t] = best;
            rec[l * cells + t] = (unsigned char)arg;
        }
        float *const swap = cur;
        cur = prev;
        prev = swap;
        __syncthreads();
    }

    // least cost, smallest time among equals
    float bv = __builtin_inff();
    int bt = INT32_MAX;
    for (int t = tid; t <= B; t += threads)
        argmin_merge(bv, bt, prev[t], t);
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) {
        const float ov = __shfl_down(bv, off, kWave);
        const int ot = __shfl_down(bt, off, kWave);
        argmin_merge(bv, bt, ov, ot);
    }
    if (lane == 0) {
        sh.best[wave] = bv;
        sh.time[wave] = bt;
    }
    __syncthreads();
    if (wave > 0)
        return;
    bv = sh.best[0];
    bt = sh.time[0];
    for (int w = 1; w < waves; ++w)
        argmin_merge(bv, bt, sh.best[w], sh.time[w]);
    const bool feasible = bv < __builtin_inff();
    if (lane == 0)
        cost[k] = bv;
    int16_t *const prof = profile + (size_t)k * L;
    int t = feasible ? bt : 0;
    for (int base = (L - 1) & ~(kWave - 1); base >= 0; base -= kWave) {
        int chosen = -1;                          // lane i: of layer base + i
        for (int l = min(base + kWave, L) - 1; feasible && l >= base; --l) {
            const int s = __builtin_amdgcn_readfirstlane(rec[l * cells + t]);
            chosen = lane == l - base ? s : chosen;
            t -= __builtin_amdgcn_readfirstlane(table[l * S + s].x);
        }
        if (base + lane < L)
            prof[base + lane] = (int16_t)chosen;
    }
}
