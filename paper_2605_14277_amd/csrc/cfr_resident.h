// Games whose iteration state fits the LDS of the workgroups that own them
// iterate inside one launch (k_resident): declarations shared by the host
// planner (cfr_resident_plan.hip) and the kernel (cfr_resident.hip).  Not
// part of the public ABI.
//
// A game is owned by a team of `blocks` workgroups.  Each player's treeplex
// is cut at a level c: the decision points of level c and everything below
// them are dealt to the workgroups in contiguous runs of level-c decision
// points (whole subtrees), the levels above c (the shallow part) are held by
// every workgroup, which all compute the same values for them.  A workgroup
// keeps its sequences' utilities, strategies, regrets and averages in LDS
// for as many iterations as the launch runs, and computes the payoff rows of
// exactly its own sequences, so only two things pass between workgroups: the
// values of the level-c decision points (with the utilities of the shallow
// sequences) and the sequence-form strategies that the products gather.
// They pass through device memory with agent-scope accesses, ordered by a
// barrier over the team.  A team of one workgroup has no shallow part and
// passes nothing.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <memory>
#include <vector>

#include "cfr_internal.h"

namespace cfr {

constexpr int kResThreadsMax = 1024;
constexpr int kResWavesMax = kResThreadsMax / 64;
// A game alone in a workgroup of 256 threads up to this many sequences (both
// players'): a barrier over 16 waves costs more than they bring.
constexpr int32_t kResFewSeq = 512;
constexpr int kResXcds = 8;
constexpr int kResCus = 256;              // workgroups of a team at most (fewer on a smaller device)
constexpr int kResXcdCus = 32;            // a team up to this size stays on one XCD
constexpr uint32_t kResLds = 156 * 1024;  // LDS one workgroup may take
constexpr int kResBarWords = 1024;        // counters of one team (u32)
constexpr int kResTeamsMax = 32767;       // games in one launch
constexpr int64_t kResSeqMax = 1200000;   // sequences of a game at most (its state's bytes decide)
// Setting a game up (us), measured for n sequences of both players: 0.2 to 0.3
// ms for 92, 0.4 for 458 and 1,500, 0.9 for 2,300, 1.7 for 6,200, 2.6 to 4.7
// for 17,000, 3.2 to 6.8 for 24,000, 3.0 for 62,000, 2.1 to 5.7 for 113,000, 3.5
// to 4.8 for 187,000, 5.2 for 315,000 and 11 for 597,000: larger games have
// fewer team sizes to choose from.  It is done once the iterations asked for
// since the last set-up would have saved as much; an iteration saves 15 to 70 us
// over one launch a step (17,000 sequences 38 to 23, 92 26 to 8, 6,300 43 to 18,
// 118,000 106 to 33).
constexpr double kResSaveUs = 20;
inline double res_setup_us(int64_t n)
{
    return 250.0 + 0.25 * (double)(n < 16000 ? n : 16000) + 0.012 * (double)n;
}
// The loop and the launches that it replaces are timed against each other over
// this many iterations, unless the loop's estimate is below this share of the
// launches': measured times were at most 2.8 times the loop's estimate and at
// least 1.2 times the launches'.
constexpr int64_t kResTrial = 32;
constexpr double kResSure = 0.45;
// A set of games whose teams were not used after all costs twice as much the
// next time, up to this many times over.
constexpr int kResBackoff = 10;
// A batch's last game saves 2 to 12 us an iteration in a team of all units
// (27 instead of 39, 38 instead of 41, 50 instead of 53).
constexpr double kResWiderUs = 5;
constexpr int64_t kResMinIterations = 4;  // a shorter run's set-up and copies cost what it saves
constexpr int64_t kResLaunchIterations = 1024;  // bounds the time of one launch

// A wave's worth of payoff rows: `rows` whole rows of n stream elements in
// all (at most res_chunk, or one longer row), each summed by 1 << lr lanes.
struct ResChunk {
    int32_t off, n;   // first element in the team's streams, elements
    int32_t rows_lr;  // rows | lr << 16
    int32_t meta;     // first row's entry in the row table (rows + 1 of them)
};

// One workgroup's share of one player, at and below the cut level.  Its
// decision points are numbered level by level, children of one sequence one
// after another, and its sequences follow; local sequence 0 stands for the
// empty sequence.  A group is a run of at most 64 sequences of one level,
// whole decision points: what a wave takes at a time on the way up.  Offsets
// are into the team's pools of 32-bit and 16-bit integers.
struct ResPart {
    int32_t nq, ni, nlev;
    int32_t lev;         // i32 [nlev + 1]: first group of each level (of those at grp)
    int32_t grp;         // i32 [groups + 1]: first local sequence of each group
    int32_t gs;          // i32 [nq]: global sequence of each local one
    int32_t cut;         // i32: which of the cut level's each of its first level's is
    int32_t kn, in;      // u16 [nq]: place among its decision point's actions | actions << 8,
                         // and the local decision point
    int32_t cp, pq;      // u16: first child [nq + 1], parent sequence [nq] (of the shallow
                         // part for the first level, when there is one)
    int32_t first_q;     // sequences before this one belong to the first level
    int32_t c0, nc;      // its chunks
};

// The shallow part of one player, levels 0 .. c-1, numbered the same way;
// children continue into the cut level's decision points, [ni, ni + ncut).
struct ResShallow {
    int32_t c, nq, ni, ncut;
    int32_t lev, grp, gs;
    int32_t kn, in, cp, pq;
};

struct ResTeam {
    int32_t slot, blocks;
    int32_t seq0[2];          // the game's empty sequences (global)
    int32_t quads[2];         // product w reads quads (summed in registers) instead of elements
    int32_t pub[2];           // player p's strategy is published: 0 no (one workgroup gathers
                              // from LDS), 1 in x, 2 in xp at pos
    int32_t lean;             // averages and own strategies are kept in device memory, not in LDS
    ResShallow sh[2];
    const ResPart *part;      // [blocks][2]
    const int32_t *i32;
    const uint16_t *u16;
    const ResChunk *chunk;
    const uint32_t *row;      // destination | first element in its chunk << 16 of each row
    const int32_t *idx[2];
    const void *val[2];
    void *cutv[2];            // compute type [ncut]
    void *gx[2];              // value type [shallow sequences]
    uint32_t *bar;
};

// Stream elements of a chunk a lane takes: as many as keep the kernel within
// 128 vector registers (16 waves a compute unit) and 2 KB of staging a wave.
__host__ __device__ constexpr int res_rounds(int value_bytes, bool quads)
{
    return value_bytes == 8 ? (quads ? 2 : 4) : (quads ? 4 : 8);
}
__host__ __device__ constexpr int res_chunk(int value_bytes, bool quads)
{
    return 64 * res_rounds(value_bytes, quads);
}
// Staging of one wave: a chunk's products, or a group's values in the compute
// type.
constexpr uint32_t kResStage = 2048;
static_assert(res_chunk(8, false) * 8 <= kResStage && res_chunk(4, false) * 4 <= kResStage &&
                  res_chunk(4, true) * 4 <= kResStage && 64 * 8 <= kResStage,
              "a chunk's products and a group's values fit");

// LDS offsets (bytes) of one player's arrays: the workgroup's own sequences
// first, then the shallow ones (sequences from nq, decision points from ni,
// values of the cut level after the shallow ones').
struct ResOff {
    uint32_t r, s, v, g, b, x, pub, kn, in, cp, pq;
};
constexpr uint32_t kResLdsHead = 128;  // scalars and flags at the start of LDS

// The layout for the host's size check and the kernel (which reads the
// records through pointers of its own kind).
template <typename Shallow, typename Share>
__host__ __device__ inline uint32_t res_layout(Shallow sh, Share part, uint32_t V, uint32_t R,
                                               uint32_t C, int lean, ResOff &o0, ResOff &o1)
{
    const auto player = [&](uint32_t at, const auto &h, const auto &q, ResOff &o) {
        const auto take = [&at](uint32_t bytes) {
            const uint32_t a = at;
            at += (bytes + 15u) & ~15u;
            return a;
        };
        const uint32_t nq = (uint32_t)(q.nq + h.nq), ni = (uint32_t)(q.ni + h.ni);
        o.r = take(R * nq);
        o.s = take(lean ? 0 : R * nq);
        o.v = take(C * (ni + (uint32_t)h.ncut));
        o.g = take(V * nq);
        o.b = take(V * nq);
        o.x = take(lean ? 0 : V * nq);
        o.pub = take(4 * nq);
        o.kn = take(2 * nq);
        o.in = take(2 * nq);
        o.cp = take(2 * (nq + 1));
        o.pq = take(2 * nq);
        return at;
    };
    return player(player(kResLdsHead, sh[0], part[0], o0), sh[1], part[1], o1);
}

// ---- host ----------------------------------------------------------------

// The treeplexes of a game in level order, kept on the host for planning.
struct ResSource {
    int32_t n_inf[2] = {0, 0};
    std::vector<int32_t> inf_first[2], seq_par[2], child_ptr[2], child_idx[2];
    std::vector<int32_t> lvl_inf[2], lvl_seq[2];
};

// Rows of one product as the planner takes them: stream elements of each row
// (row pointers) and log2 of the lanes that share a row.
struct ResRows {
    const std::vector<int32_t> *ptr = nullptr;
    std::vector<uint8_t> lr;  // [n_seq]
};

struct ResidentPlan {
    int most = 0;       // workgroups it was allowed
    int blocks = 0;
    uint32_t lds = 0;   // bytes of the largest workgroup's arrays (without the waves' staging)
    int32_t n_seq = 0;  // of both players
    double cost_us = 0;  // estimate of one iteration
    ResShallow sh[2];
    std::vector<ResPart> part;
    std::vector<int32_t> i32;
    std::vector<uint16_t> u16;
    std::vector<ResChunk> chunk;
    std::vector<uint32_t> row;
    std::vector<int32_t> src;  // first stream element of each row (game-local)
    int32_t chunk0[2] = {0, 0}, n_chunk[2] = {0, 0};  // chunks of each product
    int64_t elements[2] = {0, 0};
    std::vector<int32_t> local[2];  // one workgroup: local sequence of each of the game's
    // device memory: everything above, the streams and the exchange arrays
    std::shared_ptr<char> dev;
    size_t dev_bytes = 0;
    ResTeam team;
};

// Workgroups that a game of n sequences needs at least (what every one keeps of
// its sequences fills its LDS).
inline int64_t res_least_blocks(int64_t n, int prec)
{
    const int64_t bytes = n * (int64_t)(accum_bytes(prec) + 2 * value_bytes(prec) + 10);
    return (bytes + kResLds - 1) / kResLds;
}

// Chooses a team size (at most max_blocks) and cuts for a game, or returns
// false when its state fits no team's LDS.  seq_base: the game's first
// sequences in the engine.  Host only.
bool plan_resident(const ResSource &src, const ResRows rows[2], const int64_t seq_base[2], int prec,
                   int max_blocks, ResidentPlan &plan);

hipError_t launch_res_fill(int prec, bool quads, int n_chunk, const ResChunk *chunk,
                           const uint32_t *row, const int32_t *src, const int32_t *idx,
                           const void *val, int64_t base, const int32_t *unperm,
                           const int32_t *local, int32_t col0, int32_t *out_idx, void *out_val,
                           hipStream_t st);
// n iterations of every team.  map: [grid] team | rank << 16 of each
// workgroup, or -1.  cooperative: the teams have barriers, so every
// workgroup has to be resident.
hipError_t launch_resident(int prec, const ResTeam *teams, const int32_t *map, int grid,
                           uint32_t lds, int threads, bool cooperative, int n, int mode, Scalars *sc,
                           const DevPlayer &p0, const DevPlayer &p1, hipStream_t st);

}  // namespace cfr
