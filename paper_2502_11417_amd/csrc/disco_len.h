// Prompt tokens by length, as the threshold searches and the policy solves read them: A(L) = prompt tokens of the requests
// of length >= L.  The table in device memory holds, for every length, the tokens from it to the end of its block of
// LEN_BLOCK lengths (k_len_reduce); behind its nbins entries lie the tokens of longer prompts, an entry per slice
// (k_len_hist).  A workgroup that reads sums adds up the blocks in LDS first, so A(L) is one read of device memory.
// (One workgroup that turned the whole table into suffix sums, and the searches behind it, took 34 us with 32 772
// lengths and 13 us with 4098.)
#pragma once
#include "disco_device.h"

namespace {

// Lengths 0 .. LEN_MAX_BINS - 1 of the largest table (128 KB of LDS counts where it is made, and where a small trace's lies).
constexpr int LEN_MAX_BINS = 32772;
constexpr int LEN_BLOCK = 64;
constexpr int LEN_MAX_BLOCKS = 1024;                    // of a table (threads of the workgroup that adds them up)

struct LenScratch { u64 above[LEN_MAX_BLOCKS]; u64 wave[16], beyond[16]; };

struct LenSums {
    const u64* table;
    const u64* above;                                   // LDS: tokens of the blocks above a block and of longer prompts
    u64 beyond;                                         // tokens of the prompts longer than the table holds
    int nbins;
    __device__ __forceinline__ u64 operator()(int L) const
    {
        if (L < 0) L = 0;
        return L < nbins ? table[L] + above[L / LEN_BLOCK] : beyond;
    }
};

__device__ __forceinline__ u64 wave_suffix_u64(u64 x)
{
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const unsigned lo = (unsigned)__shfl_down((int)(unsigned)x, d, 64), hi = (unsigned)__shfl_down((int)(unsigned)(x >> 32), d, 64);
        if (lane + d < 64) x += ((u64)hi << 32) | lo;
    }
    return x;
}

// All 1024 threads of a workgroup; nslices <= 1024.
__device__ __forceinline__ LenSums len_sums(const u64* table, int nbins, int nslices, LenScratch& s)
{
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int nblk = (nbins + LEN_BLOCK - 1) / LEN_BLOCK;
    const u64 mine = t < nblk ? table[(size_t)t * LEN_BLOCK] : 0ull;      // the whole block
    const u64 longer = wave_sum_u64(t < nslices ? table[nbins + t] : 0ull);
    u64 incl = wave_suffix_u64(mine);
    if (lane == 0) { s.wave[wave] = incl; s.beyond[wave] = longer; }
    __syncthreads();
    u64 beyond = 0ull;
    for (int w = 0; w < 16; ++w) { beyond += s.beyond[w]; incl += w > wave ? s.wave[w] : 0ull; }
    s.above[t] = incl - mine + beyond;
    __syncthreads();
    return LenSums{table, s.above, beyond, nbins};
}

}  // namespace
