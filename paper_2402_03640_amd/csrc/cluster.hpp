// Cluster solver: the whole Algorithm 1 loop of one (instance, restart) runs
// in C workgroups on the CUs of one XCD, with the relaxed values of every
// variable (in the wide form: their roundings) in each workgroup's LDS.  Used
// where the state of an instance fits LDS but one workgroup is too slow and the
// tiled kernels are bound by launch latency or by the fabric traffic of their
// gathers.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "cluster_shape.hpp"
#include "kernels.hpp"
#include "plan.hpp"

namespace hms {

constexpr int kClusterMaxK = 5;       // longest clause
constexpr int32_t kClusterMaxT = 1 << 20;
constexpr int32_t kClusterMaxR = 1 << 20;  // restarts: the host holds a record of each

// One instance of a cluster launch (device-visible).
struct ClusterDesc {
    const TileDesc* c_tile;
    const uint32_t* c_ent;
    const TileDesc* v_tile;
    const uint32_t* v_ent;
    const int32_t* var_old;
    const int64_t* c_w;   // weight of each clause row, or null
    // built by launch_cluster_build
    uint32_t* counts;     // [n_act] occurrences per variable: positive | negative << 16
    int32_t* bins;        // [kClusterBins] variables per list length, then the first rank of each
    int32_t* slot;        // [n_act] LDS slot of a variable
    int32_t* var;         // [C * slice] variable of an LDS slot, -1: none
    int2* tile;           // [v_tiles] first record block, list length
    uint32_t* rec;        // occurrence records
    float* wrec;          // weighted: clause weight per record
    uint32_t* cslot;      // [c_ent] clause entries with LDS slots in place of variables
    float2* scal;         // Adam scalars of each step of this launch
    int32_t n, n_act, c_tiles, v_tiles, C, log2C, NO, slice;
    int64_t c_ent_n;
    int32_t R, T, K, opt;
    int64_t w_empty, best0;
    float two_over_m, lr, b1, b2, eps, omb1, omb2;
    double inv_m;
    uint64_t seed;
    const float* x0;      // caller order [n][R] or null
    const float* m0;
    const float* v0;
    int32_t step0, resume;
    uint8_t* best_a;      // [R][n] caller order
    int64_t* best;        // [R]
    int32_t* best_step;   // [R]
    double* final_loss;   // [R]
    float* x_final;       // caller order [n][R] or null
    float* m_final;
    float* v_final;
    TracePoint* trace;    // [trace_cap][R] or null
    int32_t trace_cap, wide;
};

// One cluster of a launch: restart r of desc, its exchange buffers, and the
// control words of its registration (arrived count; 0 undecided, 1 go, 2 void).
struct ClusterGroup {
    const ClusterDesc* desc;
    float* tbuf;       // [2][C * slice] signed tanh, by LDS slot (kClusterOneWords: 64-bit words
                       // {t, step}, zero before the launch; kClusterWide: [2][C * slice + 64] by
                       // position, then [2][C * slice / 64] words of roundings)
    uint64_t* flags;   // [C] 128-byte lines, by step parity: step number | partial count << 32
                       // (kClusterOneWords: [4][up to 15 C], by step, one word per counting wavefront);
                       // zero before the launch
    double* losses;    // [2][C] partial losses, by step parity (kClusterOneWords: [4][C])
    int32_t* ctl;      // [0] arrived, [1] decision, [2] a bounded wait ran out
    int32_t r, C;
};

struct ClusterLaunch {
    const ClusterGroup* groups;  // device; clusters of XCD x are [off[x], off[x + 1])
    int32_t* tickets;            // device [kXcds], zero
    int32_t off[kXcds + 1];
    uint64_t wait_ticks;         // wall-clock ticks (100 MHz) that a cluster waits to fill
    int32_t shared_off;          // LDS offset of the workgroup variables (set by launch_cluster)
};

// How long the clusters of a launch of T steps wait to fill beside other work: as
// long as the solve takes, about, and no longer than 20 ms (a solve of 300 steps
// beside work that keeps CUs for longer took 24 ms, 20 of them this wait).
inline uint64_t cluster_wait_ticks(int32_t T) {
    return (uint64_t)std::min<int64_t>(std::max<int64_t>((int64_t)T * 500, 200000), 2000000);
}
// Whether the instance can run as a cluster solve at all, and the sizes that its
// shape depends on; then the shape for R restarts.
bool cluster_size(const HostPlan& P, ClusterSize& Z);
bool cluster_shape(const HostPlan& P, int32_t R, size_t lds_cap, ClusterShape& sh);
constexpr int kClusterBins = 512;  // list lengths (rows kept whole have at most kSplitDense entries)
// Words of a record block (8 records of each list for 64 rows: column bits,
// then the records) and the most blocks of an instance with `cols`
// variable-side columns in `tiles` tiles.
constexpr int cluster_record_words(int NO) { return NO <= 2 ? 1 : 2; }
constexpr int cluster_head_words(bool wide) { return wide ? 256 : 128; }
constexpr int cluster_block_words(int NO, bool wide) { return cluster_head_words(wide) + 1024 * cluster_record_words(NO); }
inline size_t cluster_blocks(size_t cols, int32_t tiles) { return cols / 8 + (size_t)tiles; }

// Variable order, records and clause slots of `count` instances (Ds on the
// device, hostDs the same on the host) from their device plans, and the Adam
// scalars of steps step0 .. step0 + T - 1.  D.bins is zero.
hipError_t launch_cluster_build(const ClusterDesc* Ds, const ClusterDesc* hostDs, int32_t count, hipStream_t s);
// Bytes of one cluster's exchange buffer and flags.
inline size_t cluster_tbuf_bytes(const ClusterShape& sh) {
    const size_t P = (size_t)sh.C * sh.slice;
    if (sh.mode == kClusterWide) return 2 * (P + 64) * 4 + 2 * (P / 64) * 8;
    return 2 * P * (sh.mode == kClusterOneWords ? 8 : 4);
}
inline size_t cluster_flag_bytes(const ClusterShape& sh) { return (size_t)sh.C * 512; }
hipError_t launch_cluster(const ClusterLaunch& L, const ClusterShape& sh, bool weighted, size_t lds_cap,
                          hipStream_t s);

}  // namespace hms
