// Which tiles of the crowded experts a workgroup of k_grouped_stream takes: arithmetic alone, for the kernel and for the host's tests.
#pragma once
#include <hip/hip_runtime.h>

// The workgroups of a die are two teams, 18 that begin with the whole tiles and 14 that begin with the rests.  A team takes the tiles of its share of a list in turn, and
// those of the rests' last round, which is cut short, in reverse: not to who has a whole tile more.  Blocks of 4 row tiles x 4 feature tiles of the whole ones are neighbours
// (what they share comes from one L2), all features of a row tile of the rests.
// leave: where the rests are a stream of 12 rounds and 0.3 ms (256 features x 1024 channels a round) and more, the last four of a die (one for each of its four shader engines, to which a
// launch's workgroups go in turn) take whole tiles only, and go: other streams' launches find CUs, instead of waiting for this one's end.  A pass of 37 tokens, 256 experts, 512 x 1024,
// median and longest us, beside layers of 16384 tokens, 4 uses, with all CUs held / so (with k_grouped_gemm in that place), and these layers alone: 1024 experts of 1024 x 2048
// 867, 1700 / 118, 403 (259, 613), 1855 / 1877 (2010), loaded evenly 1876 / 1945 (2017); 512 529, 1062 / 132, 602 (185, 511), 1190 / 1201 (1350); 1024 of 512 x 2048 503, 990 / 113, 558 (187,
// 559), 1069 / 1079 (1169).  On the other side of the line, leaving from 1 GB of weights on, whatever the rounds, alone: 256 experts, 2048 x 2048, 64 uses each 869 / 950; 64, 1024 x 8192 475 / 584
// (nine rounds instead of eight, two instead of one); 512, 1024 x 1024 489 / 526.  (28 workgroups a die from the start: 1907, 120 us beside it; 31 or 30: no better beside it than 32)
struct StreamDeal {
    static constexpr int WORKGROUPS = 256;
    struct Place { int row, column; };                         // row tile of its kind, feature tile

    int half;                                                  // 0: whole tiles first
    bool leave;

    // n_whole, n_rest row tiles of nt feature tiles each, whose sums have K channels
    __host__ __device__ StreamDeal(int workgroup, int n_whole, int n_rest, int nt, int K) : n_whole(n_whole), nt(nt)
    {
        const int die = workgroup & 7, slot = workgroup >> 3;
        leave = (long long)n_rest * nt >= 12 * WORKGROUPS && (long long)n_rest * nt * K >= 12ll * WORKGROUPS * 1024;
        half = slot < 28 ? slot & 1 : 0;
        turn = slot < 28 ? slot >> 1 : slot - 14;
        team = half ? 14 : 18;
        rest_team = leave ? 14 : team;
        const int at = die * 32 + half * 18, rest_at = leave ? die * 28 + half * 14 : at, rest_of = leave ? 224 : 256;
        whole0 = share(n_whole, at, 256);
        wholes = share(n_whole, at + team, 256) - whole0;
        rest0 = share(n_rest, rest_at, rest_of);
        const int rests = share(n_rest, rest_at + rest_team, rest_of) - rest0;
        const int more = wholes % team, ahead = (more < rest_team ? more : rest_team) % rest_team;   // the first round of rests begins behind who has a whole tile more
        const int rounds = (ahead + rests) / rest_team * rest_team, full = rests < rounds - ahead ? rests : rounds - ahead;
        first = turn < ahead ? turn - ahead + rest_team : turn - ahead;
        regular = full > first ? (full - first + rest_team - 1) / rest_team : 0;
        last = rounds + rest_team - 1 - turn - ahead;          // this workgroup's of the last round, if it has one
        rest_all = turn < rest_team ? regular + (last >= 0 && last < rests) : 0;
    }
    __host__ __device__ int whole_count() const { return (wholes - turn + team - 1) / team; }
    __host__ __device__ int rest_count() const { return rest_all; }
    __host__ __device__ Place whole(int s) const
    {
        const int i = whole0 + turn + team * s;
        const int strip = i / (4 * nt), i1 = i - strip * 4 * nt, rows4 = n_whole - strip * 4 < 4 ? n_whole - strip * 4 : 4;   // 4 row tiles, all features
        const int col = i1 / (rows4 * 4), i2 = i1 - col * rows4 * 4, cols4 = nt - col * 4 < 4 ? nt - col * 4 : 4;
        return {strip * 4 + i2 / cols4, col * 4 + i2 % cols4};
    }
    __host__ __device__ Place rest(int s) const
    {
        const int i = rest0 + (s < regular ? first + rest_team * s : last), m = i / nt;
        return {m, i - m * nt};
    }

private:
    int n_whole, nt, turn, team, rest_team, whole0, wholes, rest0, first, regular, last, rest_all;
    __host__ __device__ int share(int n, int i, int of) const { return int((long long)n * nt * i / of); }
};
