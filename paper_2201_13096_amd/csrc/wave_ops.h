// Scans and reductions over the lanes of a wavefront, by DPP.  Included by spdy_dp.hip, inside its
// namespace.

// A number that a generic lambda takes as a constant.
template <int N> struct Many {
    static constexpr int value = N;
};

template <int kCtrl, int kRows, class T> __device__ __forceinline__ T dpp_from(T none, T x)
{
    static_assert(sizeof(T) == 4 || sizeof(T) == 8, "words");
    if constexpr (sizeof(T) == 4) {
        return __builtin_bit_cast(T, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, none),
                                                                 __builtin_bit_cast(int, x), kCtrl,
                                                                 kRows, 0xf, false));
    } else {
        const unsigned long long n = __builtin_bit_cast(unsigned long long, none);
        const unsigned long long b = __builtin_bit_cast(unsigned long long, x);
        const unsigned lo = dpp_from<kCtrl, kRows>((unsigned)n, (unsigned)b);
        const unsigned hi = dpp_from<kCtrl, kRows>((unsigned)(n >> 32), (unsigned)(b >> 32));
        return __builtin_bit_cast(T, (unsigned long long)hi << 32 | lo);
    }
}
template <class T> __device__ __forceinline__ T from_lane(T x, int lane)
{
    if constexpr (sizeof(T) == 4) {
        return __builtin_bit_cast(T,
                                  __builtin_amdgcn_readlane(__builtin_bit_cast(int, x), lane));
    } else {
        const unsigned long long b = __builtin_bit_cast(unsigned long long, x);
        const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)b, lane);
        const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(b >> 32), lane);
        return __builtin_bit_cast(T, (unsigned long long)hi << 32 | lo);
    }
}

// A value that is the same in every lane, in scalar registers: what is read from LDS is divergent to
// the compiler, and loops and branches on it would run under an execution mask.
template <class T> __device__ __forceinline__ T uniform(T x)
{
    if constexpr (sizeof(T) == 4) {
        return __builtin_bit_cast(T, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, x)));
    } else {
        const unsigned long long b = __builtin_bit_cast(unsigned long long, x);
        const unsigned lo = (unsigned)__builtin_amdgcn_readfirstlane((int)b);
        const unsigned hi = (unsigned)__builtin_amdgcn_readfirstlane((int)(b >> 32));
        return __builtin_bit_cast(T, (unsigned long long)hi << 32 | lo);
    }
}

// Inclusive scan over the 64 lanes (lane 63 holds the total): row_shr 1, 2, 4, 8, then the last
// lane of a row is broadcast into the rows after it.
template <class T, class Op> __device__ __forceinline__ T wave_scan(T v, T none, Op op)
{
    v = op(v, dpp_from<0x111, 0xf>(none, v));
    v = op(v, dpp_from<0x112, 0xf>(none, v));
    v = op(v, dpp_from<0x114, 0xf>(none, v));
    v = op(v, dpp_from<0x118, 0xf>(none, v));
    v = op(v, dpp_from<0x142, 0xa>(none, v));
    v = op(v, dpp_from<0x143, 0xc>(none, v));
    return v;
}
struct Add {
    template <class T> __device__ __forceinline__ T operator()(T a, T b) const { return a + b; }
};
struct Larger {
    template <class T> __device__ __forceinline__ T operator()(T a, T b) const
    {
        return a > b ? a : b;
    }
};
struct Smaller {
    template <class T> __device__ __forceinline__ T operator()(T a, T b) const
    {
        return a < b ? a : b;
    }
};

// Combines v over aligned groups of `parts` lanes, the result in every lane of the group.  A
// step pairs each lane with one of the other half of its (twice as large) group; the halves
// are uniform by then, so mirrors serve where no exchange of lanes at that distance exists.
template <class T, class Op> __device__ __forceinline__ T group_join(T v, int parts, Op op)
{
    // (read here, or the compiler keeps the conditions as lane masks and turns them into branches again at
    // every call, four instructions each)
    const int p = __builtin_amdgcn_readfirstlane(parts);
    if (p == 1)
        return v;
    v = op(v, dpp_from<0xB1, 0xf>(v, v));         // quad_perm 1 0 3 2
    if (p == 2)
        return v;
    v = op(v, dpp_from<0x4E, 0xf>(v, v));         // quad_perm 2 3 0 1
    if (p == 4)
        return v;
    v = op(v, dpp_from<0x141, 0xf>(v, v));        // row_half_mirror
    if (p == 8)
        return v;
    v = op(v, dpp_from<0x140, 0xf>(v, v));        // row_mirror
    if (p == 16)
        return v;
    v = op(v, __shfl_xor(v, 16, kWave));
    if (p == 32)
        return v;
    return op(v, __shfl_xor(v, 32, kWave));
}
