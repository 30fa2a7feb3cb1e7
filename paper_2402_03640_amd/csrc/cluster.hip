// Cluster solver (see cluster.hpp).
//
// A restart's variables are spread over the C workgroups of a cluster, tile by
// tile of the variable side (tile i to workgroup i % C, so every workgroup gets
// its share of each degree).  Every workgroup holds t = signed tanh(x) of all
// variables in LDS.  An iteration is one pass over the workgroup's own
// occurrences: for occurrence (variable, clause) a record names the clause's
// other literals, so the clause's score is taken again at each of its
// occurrences from LDS and neither an adjoint array nor a second pass is
// needed.  The optimizer step follows in place, the new t goes to the other
// workgroups through the XCD's L2, and one flag per workgroup ends the
// iteration.
//
// The arithmetic is the tiled kernels', operation for operation.  In an
// unsatisfied clause every signed term is -|tanh|, so its score is minus the
// sum of magnitudes taken in the clause's own order, and an occurrence of
// variable i enters i's sum with the sign of "x_i rounds to true" alone; the
// sum runs over i's occurrences in plan order in FP64, and occurrences of
// satisfied clauses add zero.
//
// Exchange.  All workgroups of a cluster run on one XCD (each reads the XCC_ID
// register and takes a ticket there), so its L2 is the point they share:
// stores write through the vector L1 into it, loads of exchanged data carry
// the device scope, which the vector L1 never serves.  No cache is written back
// or invalidated.  Measured: a step of 32 workgroups that exchange 80 KB this
// way costs 0.65 us for the flags and 2.0 us for the copies; an agent-scope
// release costs over 100 us, since it writes back the whole L2.
//
// Forward progress.  A workgroup waits for others only after its whole cluster
// has registered: the last to arrive decides "go"; a workgroup that has waited
// too long decides "void" with a compare-and-swap, and then none starts and the
// host takes the tiled kernels.  After "go" all C workgroups are resident and
// running.  Every later wait is bounded as well.
#include "cluster.hpp"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <mutex>

#include "device_common.hpp"

namespace hms {

namespace {

constexpr int kWaves = kClusterThreads / 64;
constexpr int kFlagStride = 16;          // u64 per flag: one 128-byte line
constexpr uint64_t kRegisterTicks = 2000000;  // wall-clock ticks (100 MHz) a cluster waits to fill: 20 ms
constexpr int kSpinLimit = 1 << 21;      // polls of one flag, about a second

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// Pointers that come out of memory, in the global address space: a generic
// load counts as an LDS access as well, and every wait for a gather would then
// wait for the record loads in flight.
#define HMS_GLOBAL __attribute__((address_space(1)))

__host__ __device__ __forceinline__ size_t up16(size_t b) { return (b + 15) & ~size_t(15); }

// Workgroup variables, after the arrays (no static LDS: the records' byte
// offsets are then LDS addresses as they stand).
struct Shared {
    const ClusterGroup* group;
    int member, dead;
    unsigned long long cnt[2], tot[2];
    double los[kWaves];
};

// LDS of a workgroup: t of all variables and two constants, own x, m, v, own
// rounded bits (current and best).
__host__ __device__ __forceinline__ size_t t_bytes(int32_t C, int32_t slice) { return up16(((size_t)C * slice + 2) * 4); }
size_t lds_bytes(int32_t C, int32_t slice) {
    return up16(t_bytes(C, slice) + (size_t)slice * 12 + (size_t)(slice / 64) * 16) + sizeof(Shared);
}

// ---- build ------------------------------------------------------------------
// A variable's occurrences are kept as two lists, the positive and the negative
// literals, each in plan order.  A clause is in the loss only if all its
// literals are false, so at any time one of the two lists adds nothing (the
// positive one when x rounds to true) and a step walks the other alone.  Rows
// are ordered by their longer list, so the 64 rows of a tile end together
// (3-CNF, 12.9 occurrences per variable: 8.5 records walked instead of 13.3).

__device__ __forceinline__ int list_len(uint32_t counts) { return max((int)(counts & 0xffffu), (int)(counts >> 16)); }

// Occurrences of each variable and the histogram of list lengths (summed in
// LDS first: lengths repeat, and device atomics on one word go one by one).
__global__ __launch_bounds__(1024) void k_cluster_count(ClusterDesc D) {
    __shared__ int h[kClusterBins];
    const int v = blockIdx.x * 1024 + threadIdx.x;
    if (threadIdx.x < kClusterBins) h[threadIdx.x] = 0;
    __syncthreads();
    if (v < D.n_act) {
        const TileDesc d = D.v_tile[v / kTile];
        const uint32_t pad = (uint32_t)D.c_tiles * kTile;
        uint32_t cnt = 0;
#pragma unroll 8
        for (uint32_t c = 0; c < d.len; ++c) {
            const uint32_t e = D.v_ent[(size_t)d.base + (size_t)c * kTile + v % kTile];
            if ((e & kIdx) != pad) cnt += (e & kSign) ? 1u << 16 : 1u;
        }
        D.counts[v] = cnt;
        atomicAdd(h + list_len(cnt), 1);
    }
    __syncthreads();
    if (threadIdx.x < kClusterBins && h[threadIdx.x] != 0) atomicAdd(D.bins + threadIdx.x, h[threadIdx.x]);
}

// First rank of each list length (longest first), and every tile's length and
// first record block.  One workgroup.
__global__ __launch_bounds__(kClusterBins) void k_cluster_scan(ClusterDesc D) {
    __shared__ int first[kClusterBins + 1];
    __shared__ int blocks[kClusterMaxPos / kTile];
    const int tid = threadIdx.x;
    first[tid] = D.bins[kClusterBins - 1 - tid];  // by descending length
    __syncthreads();
    if (tid == 0) {
        int sum = 0;
        for (int i = 0; i < kClusterBins; ++i) {
            const int c = first[i];
            first[i] = sum;
            sum += c;
        }
        first[kClusterBins] = sum;
    }
    __syncthreads();
    for (int t = tid; t < D.v_tiles; t += kClusterBins) {
        // the length whose ranks hold the tile's first row: the last bin
        // that starts at or before it
        int lo = 0, hi = kClusterBins;
        while (hi - lo > 1) {
            const int mid = (lo + hi) / 2;
            if (first[mid] <= t * kTile) lo = mid;
            else hi = mid;
        }
        const int len = kClusterBins - 1 - lo;
        D.tile[t].y = len;
        blocks[t] = (len + 7) / 8;
    }
    __syncthreads();
    if (tid == 0) {
        int sum = 0;
        for (int t = 0; t < D.v_tiles; ++t) {
            D.tile[t].x = sum;
            sum += blocks[t];
        }
    }
    D.bins[kClusterBins - 1 - tid] = first[tid];
}

// Rank, and with it tile, workgroup and LDS slot of each variable.  Equal
// lengths take ranks in any order: nothing but the placement depends on it.
__global__ __launch_bounds__(1024) void k_cluster_rank(ClusterDesc D) {
    __shared__ int h[kClusterBins];
    const int i = blockIdx.x * 1024 + threadIdx.x;
    const int P = D.C * D.slice;
    if (threadIdx.x < kClusterBins) h[threadIdx.x] = 0;
    __syncthreads();
    const int len = i < D.n_act ? list_len(D.counts[i]) : 0;
    int rank = i < D.n_act ? atomicAdd(h + len, 1) : i;  // within the workgroup's share of its length
    __syncthreads();
    if (threadIdx.x < kClusterBins && h[threadIdx.x] != 0)
        h[threadIdx.x] = atomicAdd(D.bins + threadIdx.x, h[threadIdx.x]);
    __syncthreads();
    if (i >= P) return;
    if (i < D.n_act) rank += h[len];
    // ranks past the last variable (the rest of the last tile, unused tiles) hold none
    const int tile = rank / kTile;
    const int s = (tile & (D.C - 1)) * D.slice + (tile >> D.log2C) * kTile + rank % kTile;
    D.var[s] = i < D.n_act ? i : -1;
    if (i < D.n_act) D.slot[i] = s;
}

// Records, one workgroup per variable tile, lane = row.  A record names the LDS
// byte offsets of the clause's other literals (two 15-bit slots per word, bits
// 2..16 and 17..31) and their signs (bits 0 and 1); clauses shorter than NO + 1
// are filled with the "false" slot P, places past a list's end (and
// tautologies, which are never unsatisfied) with the "true" slot P + 1.  A
// record block holds 8 records of both lists: one word of bits per row and
// list (own literal comes after other literal j in the clause, j = 2 .. NO, 8
// bits each; the first two terms of a sum commute), then the records in quads
// of 16 bytes per row, so every load of a wavefront covers whole lines.
__global__ __launch_bounds__(1024) void k_cluster_records(ClusterDesc D) {
    __shared__ uint8_t at[2][kSplitDense][64];         // column of each list's k-th entry
    __shared__ uint32_t bits[2][kSplitDense / 8][64];
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int NO = D.NO;
    const int W = NO <= 2 ? 1 : 2;
    const uint32_t P = (uint32_t)D.C * (uint32_t)D.slice;
    const uint32_t pad = (uint32_t)D.c_tiles * kTile;
    if ((int)blockIdx.x >= D.v_tiles) {
        // the rest of the grid: clause entries by slot
        const int64_t stride = (int64_t)(gridDim.x - D.v_tiles) * 1024;
        for (int64_t i = (int64_t)(blockIdx.x - D.v_tiles) * 1024 + threadIdx.x; i < D.c_ent_n; i += stride) {
            const uint32_t l = D.c_ent[i];
            const uint32_t u = l & kIdx;
            D.cslot[i] = (u == (uint32_t)D.n ? P : (uint32_t)D.slot[u]) | (l & kSign);
        }
        return;
    }
    const int tile = blockIdx.x;
    const int2 ti = D.tile[tile];
    const int v = D.var[(tile & (D.C - 1)) * D.slice + (tile >> D.log2C) * kTile + lane];
    const TileDesc d = v >= 0 ? D.v_tile[v / kTile] : TileDesc{0, 0, 0, 0};
    const uint32_t* ent = D.v_ent + d.base + (v >= 0 ? v % kTile : 0);
    const uint32_t cnt = v >= 0 ? D.counts[v] : 0u;
    const int blocks = (ti.y + 7) / 8;
    uint32_t* rp = D.rec + (size_t)ti.x * cluster_block_words(NO);
    for (int i = wave; i < 2 * blocks; i += 16) bits[i & 1][i >> 1][lane] = 0;
    if (wave == 0) {
        int kp = 0, kn = 0;
#pragma unroll 8
        for (uint32_t c = 0; c < d.len; ++c) {
            const uint32_t e = ent[(size_t)c * kTile];
            if ((e & kIdx) == pad) continue;
            if (e & kSign) at[1][kn++][lane] = (uint8_t)c;
            else at[0][kp++][lane] = (uint8_t)c;
        }
    }
    __syncthreads();
    for (int item = wave; item < blocks * 16; item += 16) {
        const int k = item >> 1, neg = item & 1;  // the k-th record of a list
        uint32_t o[4] = {P, P, P, P};
        uint32_t sg = 0;
        int own = 0;
        float wf = 1.0f;
        bool live = k < (neg ? (int)(cnt >> 16) : (int)(cnt & 0xffffu));
        if (live) {
            const uint32_t row = ent[(size_t)at[neg][k][lane] * kTile] & kIdx;
            const TileDesc cd = D.c_tile[row / kTile];
            live = (cd.flags & 1u) == 0;
            if (live) {
                int j = 0;
                for (uint32_t cc = 0; cc < cd.len; ++cc) {
                    const uint32_t l = D.c_ent[(size_t)cd.base + (size_t)cc * kTile + row % kTile];
                    const uint32_t u = l & kIdx;
                    if (u == (uint32_t)D.n) break;  // the clause's padding
                    if (u == (uint32_t)v) {
                        own = (int)cc;
                    } else if (j < NO) {
                        o[j] = (uint32_t)D.slot[u];
                        sg |= (l >> 31) << j;
                        ++j;
                    }
                }
                if (D.wrec != nullptr) wf = (float)D.c_w[row];
            }
        }
        if (!live) o[0] = P + 1u;
        const int blk = k >> 3, i = k & 7;
        uint32_t* qp = rp + (size_t)blk * cluster_block_words(NO) + 128 + neg * 512 * W;
        for (int w = 0; w < W; ++w) {
            const int q = i * W + w;  // word of the row's 8 W
            qp[(q >> 2) * 256 + lane * 4 + (q & 3)] = (o[2 * w] << 2) | (o[2 * w + 1] << 17) | ((sg >> (2 * w)) & 3u);
        }
        uint32_t b = 0;
        for (int j = 2; j <= NO; ++j) b |= (own >= j ? 1u : 0u) << (i + 8 * (j - 2));
        if (b != 0) atomicOr(&bits[neg][blk][lane], b);
        if (D.wrec != nullptr)
            D.wrec[((size_t)(ti.x + blk) * 16 + neg * 8 + (i & 4)) * 64 + lane * 4 + (i & 3)] = wf;
    }
    __syncthreads();
    for (int i = wave; i < 2 * blocks; i += 16)
        rp[(size_t)(i >> 1) * cluster_block_words(NO) + (i & 1) * 64 + lane] = bits[i & 1][i >> 1][lane];
}

__global__ __launch_bounds__(256) void k_cluster_scalars(float2* scal, int32_t step0, int32_t T, double lr, double b1,
                                                         double b2) {
    const int32_t k = (int32_t)(blockIdx.x * 256 + threadIdx.x);
    if (k >= T) return;
    float ss, ib2;
    adam_scalars((double)(step0 + k) + 1.0, lr, b1, b2, ss, ib2);
    scal[k] = make_float2(ss, ib2);
}

template <int N>
struct Cols {
    static constexpr int value = N;
};

// A wave-uniform pointer, and a structure behind one, in scalar registers.
template <typename T>
__device__ __forceinline__ T* uniform(T* p) {
    const uint64_t a = (uint64_t)p;
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)a);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(a >> 32));
    return (T*)(((uint64_t)hi << 32) | lo);
}
template <typename T>
__device__ __forceinline__ T load_uniform(const T* p) {
    static_assert(sizeof(T) % 4 == 0, "whole words");
    const uint32_t* w = reinterpret_cast<const uint32_t*>(p);
    uint32_t u[sizeof(T) / 4];
#pragma unroll
    for (size_t i = 0; i < sizeof(T) / 4; ++i) u[i] = ldc(w + i);
    T out;
    __builtin_memcpy(&out, u, sizeof(T));
    return out;
}

// Out of line: the branch inside tanhf would make the compiler treat the whole
// tile loop around it as divergent (vector branches and masks for its trip
// counts).
__device__ __attribute__((noinline)) float signed_tanh_call(float x) { return signed_tanh(x); }

template <int NO, bool WT>
__global__ __launch_bounds__(kClusterThreads) void k_cluster(ClusterLaunch A) {
    constexpr int W = NO <= 2 ? 1 : 2;
    constexpr int BW = cluster_block_words(NO);
    extern __shared__ __align__(16) unsigned char smem[];
    Shared& sh = *reinterpret_cast<Shared*>(smem + A.shared_off);

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    // ---- registration ---------------------------------------------------------
    if (tid == 0) {
        const int x = __builtin_amdgcn_s_getreg((3 << 11) | 20) & (kXcds - 1);  // XCC_ID
        int tk = __hip_atomic_fetch_add(A.tickets + x, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const ClusterGroup* g = nullptr;
        for (int i = A.off[x]; i < A.off[x + 1]; ++i) {
            if (tk < A.groups[i].C) {
                g = A.groups + i;
                break;
            }
            tk -= A.groups[i].C;
        }
        if (g != nullptr) {
            int32_t* ctl = g->ctl;
            const int before = __hip_atomic_fetch_add(ctl, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            int expect = 0;
            if (before == g->C - 1)
                __hip_atomic_compare_exchange_strong(ctl + 1, &expect, 1, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                     __HIP_MEMORY_SCOPE_AGENT);
            const uint64_t t0 = wall_clock64();
            int go = 0;
            while ((go = __hip_atomic_load(ctl + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) == 0) {
                if (wall_clock64() - t0 > kRegisterTicks) {
                    expect = 0;
                    __hip_atomic_compare_exchange_strong(ctl + 1, &expect, 2, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                         __HIP_MEMORY_SCOPE_AGENT);
                }
            }
            if (go != 1) g = nullptr;
        }
        sh.group = g;
        sh.member = tk;
        sh.dead = 0;
        sh.cnt[0] = sh.cnt[1] = sh.tot[0] = sh.tot[1] = 0;
    }
    __syncthreads();
    const ClusterGroup* gp = uniform(sh.group);
    if (gp == nullptr) return;
    const ClusterGroup G = load_uniform(gp);
    const ClusterDesc D = load_uniform(G.desc);
    const int member = __builtin_amdgcn_readfirstlane(sh.member);
    const int C = G.C;
    const int log2C = D.log2C;
    const int slice = D.slice;
    const int r = G.r;
    const int n = D.n;
    const int n_act = D.n_act;  // variables past these are in no clause
    const int P = C * slice;
    const int ntl = (D.v_tiles - member + C - 1) >> log2C;  // own variable tiles
    float* lt = reinterpret_cast<float*>(smem);
    float* lx = reinterpret_cast<float*>(smem + t_bytes(C, slice));
    float* lm = lx + slice;
    float* lv = lm + slice;
    uint64_t* pbits = reinterpret_cast<uint64_t*>(lv + slice);
    uint64_t* bbits = pbits + slice / 64;
    uint8_t* best_a = D.best_a + (size_t)r * n;

    // ---- initial point ----------------------------------------------------------
    auto initial = [&](int v, int& o) {
        o = D.var_old[v];
        if (D.x0 != nullptr) return D.x0[(size_t)o * D.R + r];
        const uint64_t z = splitmix64(D.seed + (uint64_t)r, (uint64_t)o + 1);
        return 2.0f * ((float)(z >> 40) * (1.0f / 16777216.0f)) - 1.0f;
    };
    for (int i = tid; i < P; i += kClusterThreads) {
        const int v = D.var[i];
        int o = 0;
        const float x = v >= 0 ? initial(v, o) : 0.0f;
        lt[i] = signed_tanh(x);
        const int l = i - member * slice;
        if (l >= 0 && l < slice) {
            lx[l] = x;
            lm[l] = v >= 0 && D.m0 != nullptr ? D.m0[(size_t)o * D.R + r] : 0.0f;
            lv[l] = v >= 0 && D.v0 != nullptr ? D.v0[(size_t)o * D.R + r] : 0.0f;
        }
    }
    if (tid == 0) {
        lt[P] = -0.0f;     // a literal that is false
        lt[P + 1] = 0.0f;  // a literal that is true
    }
    // inactive variables keep their start
    if (member == 0)
        for (int v = n_act + tid; v < n; v += kClusterThreads) {
            int o;
            const float x = initial(v, o);
            const size_t e = (size_t)o * D.R + r;
            if (!D.resume) best_a[o] = x > 0.0f ? 1 : 0;
            if (D.x_final != nullptr) D.x_final[e] = x;
            if (D.m_final != nullptr) {
                D.m_final[e] = D.m0 != nullptr ? D.m0[e] : 0.0f;
                D.v_final[e] = D.v0 != nullptr ? D.v0[e] : 0.0f;
            }
        }
    __syncthreads();
    const int32_t* my_var = D.var + member * slice;  // own variables, by own slot
    for (int q = wave; q < ntl; q += kWaves) {
        const int v = my_var[q * 64 + lane];
        bool bit = false;
        if (v >= 0) bit = D.resume ? best_a[D.var_old[v]] != 0 : lx[q * 64 + lane] > 0.0f;
        const uint64_t b = __ballot(bit);
        if (lane == 0) bbits[q] = b;
    }
    int64_t best = D.resume ? D.best[r] : D.best0;
    int best_step = D.resume ? D.best_step[r] : -1;

    const AdamCoef co{D.b1, D.b2, D.eps, D.omb1, D.omb2};
    const float tom = D.two_over_m;
    const float lr = D.lr;
    const int T = D.T, K = D.K, opt = D.opt, step0 = D.step0;
    const int c_tiles = D.c_tiles;
    const int2* tiles = D.tile;
    const TileDesc* c_tile = D.c_tile;
    const HMS_GLOBAL uint32_t* cslot = (const HMS_GLOBAL uint32_t*)D.cslot;
    const HMS_GLOBAL int64_t* c_w = (const HMS_GLOBAL int64_t*)D.c_w;
    const HMS_GLOBAL uint32_t* rec = (const HMS_GLOBAL uint32_t*)D.rec;
    const HMS_GLOBAL float* wrec = (const HMS_GLOBAL float*)D.wrec;
    const uint32_t* scal = reinterpret_cast<const uint32_t*>(D.scal);
    const int64_t w_empty = D.w_empty;

    // copies: wavefront w takes part `part` of `parts` of a peer's slice
    // (two whole slices with 32 workgroups)
    const int parts = C <= kWaves ? kWaves >> log2C : 1;
    const int rounds = C <= kWaves ? 1 : C / kWaves;

    // own tiles of this wavefront
    const int my_tiles = ntl > wave ? (ntl - 1 - wave) / kWaves + 1 : 0;
    auto own_tile = [&](int i) { return i * kWaves + wave; };
    // one record block of the list that counts (neg: x rounds to true), loaded
    // one block ahead
    struct Block {
        uint32_t w[8 * W];
        float wf[WT ? 8 : 1];
        uint32_t bits;
    };
    auto fetch = [&](Block& b, int block, bool neg) {
        const HMS_GLOBAL uint32_t* bp = rec + (size_t)block * BW;
        b.bits = bp[(neg ? 64 : 0) + lane];
        const HMS_GLOBAL u32x4* qp = (const HMS_GLOBAL u32x4*)(bp + 128) + ((neg ? 128 * W : 0) + lane);
#pragma unroll
        for (int k = 0; k < 2 * W; ++k) {
            const u32x4 v = qp[k * 64];
            b.w[4 * k] = v.x;
            b.w[4 * k + 1] = v.y;
            b.w[4 * k + 2] = v.z;
            b.w[4 * k + 3] = v.w;
        }
        if constexpr (WT) {
            const HMS_GLOBAL f32x4* fp = (const HMS_GLOBAL f32x4*)(wrec + (size_t)block * 1024) + ((neg ? 128 : 0) + lane);
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const f32x4 v = fp[k * 64];
                b.wf[4 * k] = v.x;
                b.wf[4 * k + 1] = v.y;
                b.wf[4 * k + 2] = v.z;
                b.wf[4 * k + 3] = v.w;
            }
        }
    };
    // records OFF .. OFF + N - 1 of a block
    auto sum_records = [&](auto nc, auto oc, const Block& b, const float to, double& Gm) {
        constexpr int N = decltype(nc)::value, OFF = decltype(oc)::value;
        float t[N][NO];
#pragma unroll
        for (int c = 0; c < N; ++c)
#pragma unroll
            for (int j = 0; j < NO; ++j) {
                const uint32_t w = b.w[(OFF + c) * W + (j >> 1)];
                t[c][j] = *reinterpret_cast<const float*>(smem + ((j & 1 ? w >> 15 : w) & 0x1fffcu));
            }
#pragma unroll
        for (int c = 0; c < N; ++c) {
            // sign bit set in lanes whose clause is unsatisfied: the own literal
            // is false on this list, and so is every other
            uint32_t fl = ~0u;
#pragma unroll
            for (int j = 0; j < NO; ++j)
                fl &= __float_as_uint(t[c][j]) ^ (b.w[(OFF + c) * W + (j >> 1)] << (j & 1 ? 30 : 31));
            // magnitudes in clause order: z is the own term until its place is reached
            uint32_t z = __float_as_uint(to);
            float f = fabsf(t[c][0]);
#pragma unroll
            for (int j = 2; j <= NO; ++j) {
                uint32_t after;  // all ones where the own literal comes after literal j
                asm("v_bfe_i32 %0, %1, %2, 1" : "=v"(after) : "v"(b.bits), "n"(OFF + c + 8 * (j - 2)));
                const uint32_t oj = __float_as_uint(t[c][j - 1]);
                uint32_t take;
                asm("v_bfi_b32 %0, %1, %2, %3" : "=v"(take) : "v"(after), "v"(oj), "v"(z));
                asm("v_bfi_b32 %0, %1, %2, %3" : "=v"(z) : "v"(after), "v"(z), "v"(oj));
                f = f + fabsf(__uint_as_float(take));
            }
            f = f + fabsf(__uint_as_float(z));
            if constexpr (WT) f = f * b.wf[OFF + c];
            uint32_t a = __float_as_uint(f * tom) & (uint32_t)((int)fl >> 31);
            asm("" : "+v"(a));  // the mask stays on the 32-bit value
            Gm = Gm + (double)__uint_as_float(a);
        }
    };
    auto tile_info = [&](int i) {
        const uint32_t* p = reinterpret_cast<const uint32_t*>(tiles + (own_tile(i) * C + member));
        return make_int2((int)ldc(p), (int)ldc(p + 1));
    };
    int2 tn = make_int2(0, 0);
    Block nx;
    if (my_tiles > 0) {
        tn = tile_info(0);
        fetch(nx, __builtin_amdgcn_readfirstlane(tn.x), lx[own_tile(0) * 64 + lane] > 0.0f);
    }

    int kc = step0 % K;
    for (int step = 0; step <= T; ++step) {
        const bool last = step == T;
        const bool eval = kc == 0 || last;
        if (++kc == K) kc = 0;
        const bool want_loss = last || (eval && D.trace != nullptr);
        const int par = step & 1;
        HMS_GLOBAL float* tb = (HMS_GLOBAL float*)G.tbuf + (size_t)par * P;
        // ---- count and loss of this iterate: the clause tiles, dealt out over
        // the cluster's wavefronts from the last one on (the variable tiles
        // start at the first)
        if (eval) {
            unsigned long long cnt = 0;
            double los = 0.0;
            for (int ct = (kWaves - 1 - wave) * C + member; ct < c_tiles; ct += kWaves * C) {
                const TileDesc d = ldtile(c_tile + ct);
                if (d.flags & 1u) continue;  // tautologies are never unsatisfied
                float f = 0.0f;
                uint32_t all = ~0u;
                for (uint32_t c = 0; c < d.len; ++c) {
                    const uint32_t en = cslot[(size_t)d.base + (size_t)c * kTile + lane];
                    const uint32_t b = __float_as_uint(lt[en & kIdx]) ^ (en & kSign);
                    f = f + __uint_as_float(b);
                    all &= b;
                }
                const bool unsat = lane < (int)d.nreal && (all >> 31) != 0;
                if constexpr (WT) {
                    const int64_t w = unsat ? c_w[(size_t)ct * kTile + lane] : 0;
                    cnt += (unsigned long long)w;
                    if (want_loss && unsat) los += ((double)f * (double)f) * (double)w;
                } else {
                    cnt += (unsigned long long)__popcll(__ballot(unsat));
                    if (want_loss && unsat) los += (double)f * (double)f;
                }
            }
            if constexpr (WT)
                for (int o = 32; o >= 1; o >>= 1) cnt += __shfl_xor(cnt, o);
            if (lane == 0 && cnt != 0) atomicAdd(&sh.cnt[par], cnt);
            if (want_loss) {
                for (int o = 32; o >= 1; o >>= 1) los += __shfl_xor(los, o);
                if (lane == 0) sh.los[wave] = los;
            }
        }
        // ---- transposed sums and optimizer step of the own variables --------
        float2 sc = make_float2(0.0f, 1.0f);
        if (!last && opt != kSgd)
            sc = make_float2(__uint_as_float(ldc(scal + 2 * step)), __uint_as_float(ldc(scal + 2 * step + 1)));
        if (eval)
            for (int q = wave; q < ntl; q += kWaves) {
                const uint64_t b = __ballot(lx[q * 64 + lane] > 0.0f);
                if (lane == 0) pbits[q] = b;
            }
        if (!last) {
            for (int i = 0; i < my_tiles; ++i) {
                const int q = own_tile(i);
                const int tb0 = __builtin_amdgcn_readfirstlane(tn.x), len = __builtin_amdgcn_readfirstlane(tn.y);
                const int l = q * 64 + lane;
                const float xo = lx[l];
                const float to = lt[member * slice + l];
                double Gm = 0.0;
                // the next tile; the last one's next is fetched once its x is known
                const bool more = i + 1 < my_tiles;
                if (more) tn = tile_info(i + 1);
                const float xn = lx[own_tile(more ? i + 1 : i) * 64 + lane];
                for (int k = 0; k < len; k += 8) {
                    Block b = nx;
#pragma unroll
                    for (int j = 0; j < 8 * W; ++j) asm volatile("" : "+v"(b.w[j]));
                    asm volatile("" : "+v"(b.bits));
                    const int left = len - k;
                    if (left > 8) fetch(nx, tb0 + (k >> 3) + 1, xo > 0.0f);
                    else if (more) fetch(nx, __builtin_amdgcn_readfirstlane(tn.x), xn > 0.0f);
                    // up to 16 gathers go out together
                    if constexpr (NO == 2) {
                        if (left > 6) sum_records(Cols<8>{}, Cols<0>{}, b, to, Gm);
                        else if (left > 4) sum_records(Cols<6>{}, Cols<0>{}, b, to, Gm);
                        else if (left > 2) sum_records(Cols<4>{}, Cols<0>{}, b, to, Gm);
                        else sum_records(Cols<2>{}, Cols<0>{}, b, to, Gm);
                    } else {
                        if (left > 2) sum_records(Cols<4>{}, Cols<0>{}, b, to, Gm);
                        else sum_records(Cols<2>{}, Cols<0>{}, b, to, Gm);
                        if (left > 6) sum_records(Cols<4>{}, Cols<4>{}, b, to, Gm);
                        else if (left > 4) sum_records(Cols<2>{}, Cols<4>{}, b, to, Gm);
                    }
                }
                // a positive literal in the loss adds -a, a negative one +a (0.0 - 0.0 keeps an empty sum +0)
                const double Gs = xo > 0.0f ? Gm : 0.0 - Gm;
                const float g = grad_of(xo, Gs);
                float x = xo;
                if (opt == kSgd) {
                    x = x - lr * g;
                } else {
                    float mm = lm[l], vv = lv[l];
                    adam_update(x, mm, vv, g, sc.x, sc.y, co);
                    lm[l] = mm;
                    lv[l] = vv;
                }
                lx[l] = x;
                __hip_atomic_store(tb + member * slice + l, signed_tanh_call(x), __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_WORKGROUP);
            }
            // the next step's first block, in flight over the exchange
            if (my_tiles > 0) {
                tn = tile_info(0);
                fetch(nx, __builtin_amdgcn_readfirstlane(tn.x), lx[own_tile(0) * 64 + lane] > 0.0f);
            }
        }
        // ---- the step's flag: own stores have reached the L2 ------------------
        // flags and losses alternate between two places: a workgroup that is
        // done may publish the next step while another still reads this one,
        // but not the one after, which needs the other's next flag
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        if (tid == 0) {
            if (want_loss) {
                double ls = 0.0;
                for (int w = 0; w < kWaves; ++w) ls = ls + sh.los[w];
                __hip_atomic_store(G.losses + par * C + member, ls, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                __builtin_amdgcn_s_waitcnt(0);
            }
            const uint64_t f = (uint64_t)(uint32_t)(step + 1) | ((uint64_t)sh.cnt[par] << 32);
            __hip_atomic_store((HMS_GLOBAL uint64_t*)G.flags + (size_t)member * kFlagStride + par, f, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            sh.cnt[par ^ 1] = 0;
            sh.tot[par ^ 1] = 0;
        }
        // ---- every workgroup's new t (and count) ------------------------------
        // a wavefront waits for its one or two peers (one per lane), then
        // copies its part of their slices
        {
            const int pw = rounds == 1 ? wave / parts : wave;
            const int part = rounds == 1 ? wave % parts : 0;
            const int peer0 = (pw + member) & (C - 1);
            const int peer1 = rounds == 1 ? peer0 : (pw + kWaves + member) & (C - 1);
            const HMS_GLOBAL uint64_t* fl =
                (const HMS_GLOBAL uint64_t*)G.flags + (size_t)(lane & 1 ? peer1 : peer0) * kFlagStride + par;
            uint64_t f = 0;
            bool ok = lane >= 2;
            for (int spins = 0; spins <= kSpinLimit; ++spins) {
                if (!ok) {
                    f = __hip_atomic_load(fl, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    ok = (uint32_t)f == (uint32_t)(step + 1);
                }
                if (__ballot(!ok) == 0) break;
            }
            if (__ballot(!ok) != 0) sh.dead = 1;
            if (eval && part == 0 && lane < rounds) atomicAdd(&sh.tot[par], (unsigned long long)(f >> 32));
            if (!last) {
                // device-scope loads: from the L2, never from this CU's L1
                const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void*)tb, 0, P * 4, 0x00020000);
                const int s4 = slice / 4;
                u32x4* dst = reinterpret_cast<u32x4*>(lt);
                const int stride = parts * 64;
                const int n4 = rounds * s4;  // 16-byte pieces of both slices
                for (int i0 = part * 64; i0 < n4; i0 += 6 * stride) {
                    u32x4 v[6];
                    int at[6];
#pragma unroll
                    for (int j = 0; j < 6; ++j) {
                        const int i = i0 + j * stride + lane;
                        at[j] = i < s4 ? peer0 * s4 + i : peer1 * s4 + (i - s4);
                        if (i < n4) v[j] = __builtin_amdgcn_raw_buffer_load_b128(rs, at[j] * 16, 0, 16);
                    }
#pragma unroll
                    for (int j = 0; j < 6; ++j)
                        if (i0 + j * stride + lane < n4) dst[at[j]] = v[j];
                }
            }
        }
        __syncthreads();
        if (__builtin_amdgcn_readfirstlane(sh.dead)) break;
        if (eval) {
            const int64_t c = w_empty + (int64_t)sh.tot[par];
            const bool improved = c < best;
            if (improved) {
                best = c;
                best_step = step0 + step;
                for (int q = wave; q < ntl; q += kWaves)
                    if (lane == 0) bbits[q] = pbits[q];
            }
            if (want_loss && member == 0 && tid == 0) {
                double ls = 0.0;
                for (int p = 0; p < C; ++p)
                    ls = ls + __hip_atomic_load(G.losses + par * C + p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (last) D.final_loss[r] = ls * D.inv_m;
                if (D.trace != nullptr) {
                    const int64_t gs = (int64_t)step0 + step;
                    const int64_t row = ((gs + K - 1) / K - ((int64_t)step0 + K - 1) / K) % D.trace_cap;
                    D.trace[(size_t)row * D.R + r] = TracePoint{(int32_t)gs, 0, c, ls * D.inv_m};
                }
            }
        }
    }
    if (__builtin_amdgcn_readfirstlane(sh.dead)) {
        if (tid == 0) __hip_atomic_store(G.ctl + 2, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return;
    }
    for (int q = wave; q < ntl; q += kWaves) {
        const int v = my_var[q * 64 + lane];
        const uint64_t b = bbits[q];
        if (v >= 0) {
            const int o = D.var_old[v];
            const size_t e = (size_t)o * D.R + r;
            const int l = q * 64 + lane;
            best_a[o] = (uint8_t)((b >> lane) & 1u);
            if (D.x_final != nullptr) D.x_final[e] = lx[l];
            if (D.m_final != nullptr) {
                D.m_final[e] = lm[l];
                D.v_final[e] = lv[l];
            }
        }
    }
    if (member == 0 && tid == 0) {
        D.best[r] = best;
        D.best_step[r] = best_step;
    }
}

std::mutex g_cluster_attr_mu;

template <int NO, bool WT>
hipError_t launch_as(ClusterLaunch L, size_t lds, size_t lds_cap, hipStream_t s) {
    L.shared_off = (int32_t)(lds - sizeof(Shared));
    static std::atomic<uint64_t> set_on{0};  // bit d: attribute set on device d
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const uint64_t bit = dev >= 0 && dev < 64 ? uint64_t(1) << dev : 0;
    if (!bit || !(set_on.load(std::memory_order_acquire) & bit)) {
        std::lock_guard<std::mutex> lk(g_cluster_attr_mu);
        e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_cluster<NO, WT>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_cap);
        if (e != hipSuccess) return e;
        set_on.fetch_or(bit, std::memory_order_release);
    }
    // one workgroup per CU: they are dealt round-robin over the XCDs, so every
    // XCD gets kXcdCus tickets; the surplus exits at once
    hipLaunchKernelGGL((k_cluster<NO, WT>), dim3(kXcds * kXcdCus), dim3(kClusterThreads), lds, s, L);
    return hipGetLastError();
}

}  // namespace

bool cluster_shape(const HostPlan& P, int32_t R, size_t lds_cap, ClusterShape& sh) {
    if (P.n_heavy != 0 || P.v_tiles < 2 || P.w_total >= (int64_t(1) << 32)) return false;
    uint32_t k = 0;
    for (const TileDesc& d : P.c_tile)
        if (!(d.flags & 1u)) k = std::max(k, d.len);
    if (k > (uint32_t)kClusterMaxK) return false;
    sh.NO = std::max(2, (int32_t)k - 1);
    // as many workgroups per restart as leave every restart its own at once
    int32_t C = kXcdCus;
    while (C > 2 && (int64_t)kXcds * (kXcdCus / C) < R) C /= 2;
    while (C > 2 && C > P.v_tiles) C /= 2;
    for (;; C *= 2) {
        if (C > kXcdCus) return false;
        sh.slice = (P.v_tiles + C - 1) / C * kTile;
        sh.lds = lds_bytes(C, sh.slice);
        if (sh.lds <= lds_cap && (int64_t)C * sh.slice + 2 <= kClusterMaxPos) break;
    }
    sh.C = C;
    sh.per_launch = kXcds * (kXcdCus / C);
    return true;
}

hipError_t launch_cluster_build(const ClusterDesc& D, double lr, double b1, double b2, hipStream_t s) {
    const int P = D.C * D.slice;
    hipLaunchKernelGGL(k_cluster_count, dim3((D.n_act + 1023) / 1024), dim3(1024), 0, s, D);
    hipLaunchKernelGGL(k_cluster_scan, dim3(1), dim3(kClusterBins), 0, s, D);
    hipLaunchKernelGGL(k_cluster_rank, dim3((P + 1023) / 1024), dim3(1024), 0, s, D);
    const int extra = (int)std::min<int64_t>((D.c_ent_n + 4095) / 4096, 1024);
    hipLaunchKernelGGL(k_cluster_records, dim3(D.v_tiles + extra), dim3(1024), 0, s, D);
    if (D.T > 0)
        hipLaunchKernelGGL(k_cluster_scalars, dim3((D.T + 255) / 256), dim3(256), 0, s, D.scal, D.step0, D.T, lr, b1, b2);
    return hipGetLastError();
}

hipError_t launch_cluster(const ClusterLaunch& L, int32_t NO, bool weighted, size_t lds, size_t lds_cap,
                          hipStream_t s) {
    if (lds > lds_cap) return hipErrorInvalidValue;
    switch (NO) {
        case 2: return weighted ? launch_as<2, true>(L, lds, lds_cap, s) : launch_as<2, false>(L, lds, lds_cap, s);
        case 3: return weighted ? launch_as<3, true>(L, lds, lds_cap, s) : launch_as<3, false>(L, lds, lds_cap, s);
        case 4: return weighted ? launch_as<4, true>(L, lds, lds_cap, s) : launch_as<4, false>(L, lds, lds_cap, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace hms
