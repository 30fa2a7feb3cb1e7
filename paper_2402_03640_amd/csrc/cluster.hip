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

constexpr int kWaves = kClusterWaves;
constexpr int kFlagStride = 16;          // u64 per flag: one 128-byte line
constexpr int kSpinLimit = 1 << 21;      // polls of one flag, about a second

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// Pointers that come out of memory, in the global address space: a generic
// load counts as an LDS access as well, and every wait for a gather would then
// wait for the record loads in flight.
#define HMS_GLOBAL __attribute__((address_space(1)))

// Workgroup variables, after the arrays (no static LDS: the records' byte
// offsets are then LDS addresses as they stand).
struct Shared {
    const ClusterGroup* group;
    int member, dead;
    unsigned long long cnt[2], tot[4];
    double los[kWaves];
    unsigned long long wcnt[kWaves];
};
static_assert(sizeof(Shared) == kClusterSharedBytes, "the LDS sizes count these");

// A wave-uniform pointer, and a structure behind one, in scalar registers.
template <typename T>
__device__ __forceinline__ T* uniform(T* p) {
    const uint64_t a = (uint64_t)p;
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)a);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(a >> 32));
    return (T*)(((uint64_t)hi << 32) | lo);
}
// The same pointer, opaque to the compiler: what is loaded through it is loaded
// there and then, not ahead of a loop.
template <typename T>
__device__ __forceinline__ const T* launder(const T* p) {
    asm volatile("" : "+s"(p));
    return p;
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

// ---- build ------------------------------------------------------------------
// A variable's occurrences are kept as two lists, the positive and the negative
// literals, each in plan order.  A clause is in the loss only if all its
// literals are false, so at any time one of the two lists adds nothing (the
// positive one when x rounds to true) and a step walks the other alone.  Rows
// are ordered by their longer list, so the 64 rows of a tile end together
// (3-CNF, 12.9 occurrences per variable: 8.5 records walked instead of 13.3).
// Every kernel builds one instance per row of its grid: Ds[blockIdx.y].

// Wide form: where slot s is named and its t kept.  The low five bits are the
// rotation that brings the slot's bit of its 32-bit word to the top.
__device__ __forceinline__ uint32_t wide_pos(uint32_t s) { return (s & ~31u) | ((s + 1u) & 31u); }

__device__ __forceinline__ int list_len(uint32_t counts) { return max((int)(counts & 0xffffu), (int)(counts >> 16)); }

// Occurrences of each variable and the histogram of list lengths (summed in
// LDS first: lengths repeat, and device atomics on one word go one by one).
__global__ __launch_bounds__(1024) void k_cluster_count(const ClusterDesc* Ds) {
    const ClusterDesc D = load_uniform(Ds + blockIdx.y);
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
__global__ __launch_bounds__(kClusterBins) void k_cluster_scan(const ClusterDesc* Ds) {
    const ClusterDesc D = load_uniform(Ds + blockIdx.y);
    __shared__ int first[kClusterBins + 1];
    __shared__ int sums[kClusterBins];
    __shared__ uint8_t blocks[kClusterMaxWide / kTile];
    const int tid = threadIdx.x;
    // running sum over the workgroup of one value per thread, own value included
    auto running = [&](int own) {
        sums[tid] = own;
        __syncthreads();
        for (int o = 1; o < kClusterBins; o <<= 1) {
            const int left = tid >= o ? sums[tid - o] : 0;
            __syncthreads();
            sums[tid] += left;
            __syncthreads();
        }
        return sums[tid];
    };
    const int here = D.bins[kClusterBins - 1 - tid];  // by descending length
    const int upto = running(here);
    first[tid] = upto - here;
    if (tid == kClusterBins - 1) first[kClusterBins] = upto;
    __syncthreads();
    // a run of tiles per thread
    const int run = (D.v_tiles + kClusterBins - 1) / kClusterBins;
    int mine = 0;
    for (int t = tid * run; t < (tid + 1) * run && t < D.v_tiles; ++t) {
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
        blocks[t] = (uint8_t)((len + 7) / 8);
        mine += blocks[t];
    }
    int sum = running(mine) - mine;
    for (int t = tid * run; t < (tid + 1) * run && t < D.v_tiles; ++t) {
        D.tile[t].x = sum;
        sum += blocks[t];
    }
    D.bins[kClusterBins - 1 - tid] = first[tid];
}

// Rank, and with it tile, workgroup and LDS slot of each variable.  Equal
// lengths take ranks in any order: nothing but the placement depends on it.
__global__ __launch_bounds__(1024) void k_cluster_rank(const ClusterDesc* Ds) {
    const ClusterDesc D = load_uniform(Ds + blockIdx.y);
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
// of 16 bytes per row, so every load of a wavefront covers whole lines.  In the
// wide form a literal is a 16-bit position, and a second word of bits per row
// and list holds the signs (bit NO i + j for other literal j of record i).
__global__ __launch_bounds__(1024) void k_cluster_records(const ClusterDesc* Ds) {
    const ClusterDesc D = load_uniform(Ds + blockIdx.y);
    __shared__ uint8_t at[2][kSplitDense][64];         // column of each list's k-th entry
    __shared__ uint32_t bits[2][kSplitDense / 8][64];
    __shared__ uint32_t sign[2][kSplitDense / 8][64];  // wide form
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int NO = D.NO;
    const bool wide = D.wide != 0;
    const int W = cluster_record_words(NO);
    const int block_words = cluster_block_words(NO, wide);
    const uint32_t P = (uint32_t)D.C * (uint32_t)D.slice;
    const uint32_t pad = (uint32_t)D.c_tiles * kTile;
    if ((int)blockIdx.x >= D.v_tiles) {
        // the rest of the grid: clause entries by slot
        const int64_t stride = (int64_t)(gridDim.x - D.v_tiles) * 1024;
        for (int64_t i = (int64_t)(blockIdx.x - D.v_tiles) * 1024 + threadIdx.x; i < D.c_ent_n; i += stride) {
            const uint32_t l = D.c_ent[i];
            const uint32_t u = l & kIdx;
            const uint32_t at = u == (uint32_t)D.n ? P : (uint32_t)D.slot[u];
            D.cslot[i] = (wide ? wide_pos(at) : at) | (l & kSign);
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
    uint32_t* rp = D.rec + (size_t)ti.x * block_words;
    for (int i = wave; i < 2 * blocks; i += 16) bits[i & 1][i >> 1][lane] = sign[i & 1][i >> 1][lane] = 0;
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
        uint32_t* qp = rp + (size_t)blk * block_words + cluster_head_words(wide) + neg * 512 * W;
        for (int w = 0; w < W; ++w) {
            const int q = i * W + w;  // word of the row's 8 W
            qp[(q >> 2) * 256 + lane * 4 + (q & 3)] =
                wide ? wide_pos(o[2 * w]) | (wide_pos(o[2 * w + 1]) << 16)
                     : (o[2 * w] << 2) | (o[2 * w + 1] << 17) | ((sg >> (2 * w)) & 3u);
        }
        uint32_t b = 0;
        for (int j = 2; j <= NO; ++j) b |= (own >= j ? 1u : 0u) << (i + 8 * (j - 2));
        if (b != 0) atomicOr(&bits[neg][blk][lane], b);
        if (wide && sg != 0) atomicOr(&sign[neg][blk][lane], sg << (i * NO));
        if (D.wrec != nullptr)
            D.wrec[((size_t)(ti.x + blk) * 16 + neg * 8 + (i & 4)) * 64 + lane * 4 + (i & 3)] = wf;
    }
    __syncthreads();
    for (int i = wave; i < 2 * blocks; i += 16) {
        uint32_t* hp = rp + (size_t)(i >> 1) * block_words + (i & 1) * 64 + lane;
        hp[0] = bits[i & 1][i >> 1][lane];
        if (wide) hp[128] = sign[i & 1][i >> 1][lane];
    }
}

__global__ __launch_bounds__(256) void k_cluster_scalars(const ClusterDesc* Ds) {
    const ClusterDesc D = load_uniform(Ds + blockIdx.y);
    const int32_t k = (int32_t)(blockIdx.x * 256 + threadIdx.x);
    if (k >= D.T) return;
    float ss, ib2;
    adam_scalars((double)(D.step0 + k) + 1.0, (double)D.lr, (double)D.b1, (double)D.b2, ss, ib2);
    D.scal[k] = make_float2(ss, ib2);
}

// The word at a byte of the dynamic LDS array: by LDS address, or by index.
// The kernels declare no other LDS, so the array starts at 0 (enroll checks
// that), and an index costs an addition of that 0 per access: n = 20000, 64
// restarts 12.0 us a step by index, 11.6 by address (with the record blocks in
// two buffers in turn instead of copied).  Where one tile's latency counts, not
// the instructions, the index is the faster one (n = 1000: 2.78 against 2.85).
struct LdsAddress {
    __device__ __forceinline__ uint32_t operator()(uint32_t at) const {
        return *(const __attribute__((address_space(3))) uint32_t*)at;
    }
};
struct LdsIndex {
    const unsigned char* smem;
    __device__ __forceinline__ uint32_t operator()(uint32_t at) const {
        return *reinterpret_cast<const uint32_t*>(smem + at);
    }
};
// Before LdsAddress is used the array's address has to have escaped, or the
// compiler may hold stores to it to be no concern of those loads.
__device__ __forceinline__ void escape_lds(const unsigned char* smem) {
    asm volatile("" : : "v"((const __attribute__((address_space(3))) unsigned char*)smem) : "memory");
}

// Out of line: the branch inside tanhf would make the compiler treat the whole
// tile loop around it as divergent (vector branches and masks for its trip
// counts).
__device__ __attribute__((noinline)) float signed_tanh_call(float x) { return signed_tanh(x); }

// Waits until this wavefront's stores have reached the L2.  As an instruction
// with a memory effect: the builtin has none, and would let the compiler move a
// relaxed store across it.
__device__ __forceinline__ void stores_done() { asm volatile("s_waitcnt vmcnt(0)" : : : "memory"); }
// What others published before the flag just read is loaded after it.
__device__ __forceinline__ void flag_seen() { asm volatile("" : : : "memory"); }

// One record block of the list that counts (neg: x rounds to true).
template <int NO, bool WT, bool WIDE = false>
struct RecordBlock {
    static constexpr int W = cluster_record_words(NO);
    uint32_t w[8 * W];
    float wf[WT ? 8 : 1];
    uint32_t bits, sign;
    // the block's first `left` records, all or the first half
    __device__ __forceinline__ void load(const HMS_GLOBAL uint32_t* rec, const HMS_GLOBAL float* wrec, int block,
                                         int left, bool neg, int lane) {
        const HMS_GLOBAL uint32_t* bp = rec + (size_t)block * cluster_block_words(NO, WIDE);
        bits = bp[(neg ? 64 : 0) + lane];
        if constexpr (WIDE) sign = bp[(neg ? 192 : 128) + lane];
        const HMS_GLOBAL u32x4* qp =
            (const HMS_GLOBAL u32x4*)(bp + cluster_head_words(WIDE)) + ((neg ? 128 * W : 0) + lane);
#pragma unroll
        for (int k = 0; k < 2 * W; ++k) {
            if (WIDE && k == W && left <= 4) break;
            const u32x4 v = qp[k * 64];
            w[4 * k] = v.x;
            w[4 * k + 1] = v.y;
            w[4 * k + 2] = v.z;
            w[4 * k + 3] = v.w;
        }
        if constexpr (WT) {
            const HMS_GLOBAL f32x4* fp = (const HMS_GLOBAL f32x4*)(wrec + (size_t)block * 1024) + ((neg ? 128 : 0) + lane);
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                if (WIDE && k == 1 && left <= 4) break;
                const f32x4 v = fp[k * 64];
                wf[4 * k] = v.x;
                wf[4 * k + 1] = v.y;
                wf[4 * k + 2] = v.z;
                wf[4 * k + 3] = v.w;
            }
        }
    }
};

// Adds records OFF .. OFF + N - 1 of a block to the row's sum of magnitudes.
// t sits at LDS byte `at` (a power of two past every offset, or 0).
template <int N, int OFF, class Lds, int NO, bool WT>
__device__ __forceinline__ void sum_records(const Lds lds, const uint32_t at, const RecordBlock<NO, WT>& b,
                                            const float to, const float tom, double& Gm) {
    constexpr int W = RecordBlock<NO, WT>::W;
    float t[N][NO];
#pragma unroll
    for (int c = 0; c < N; ++c)
#pragma unroll
        for (int j = 0; j < NO; ++j) {
            const uint32_t w = b.w[(OFF + c) * W + (j >> 1)];
            t[c][j] = __uint_as_float(lds(((j & 1 ? w >> 15 : w) & 0x1fffcu) | at));
        }
#pragma unroll
    for (int c = 0; c < N; ++c) {
        // sign bit set in lanes whose clause is unsatisfied: the own literal is
        // false on this list, and so is every other
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
}

// The first `left` records of a block (1 to 8; whole pairs, the rest is inert),
// up to 16 gathers together.
template <class Lds, int NO, bool WT>
__device__ __forceinline__ void sum_block(const Lds lds, const uint32_t at, const RecordBlock<NO, WT>& b,
                                          const int left, const float to, const float tom, double& Gm) {
    if constexpr (NO == 2) {
        if (left > 6) sum_records<8, 0>(lds, at, b, to, tom, Gm);
        else if (left > 4) sum_records<6, 0>(lds, at, b, to, tom, Gm);
        else if (left > 2) sum_records<4, 0>(lds, at, b, to, tom, Gm);
        else sum_records<2, 0>(lds, at, b, to, tom, Gm);
    } else {
        if (left > 2) sum_records<4, 0>(lds, at, b, to, tom, Gm);
        else sum_records<2, 0>(lds, at, b, to, tom, Gm);
        if (left > 6) sum_records<4, 4>(lds, at, b, to, tom, Gm);
        else if (left > 4) sum_records<2, 4>(lds, at, b, to, tom, Gm);
    }
}

// The same in the wide form.  The roundings of the other literals (a bit each,
// in LDS) say which lanes' clauses are unsatisfied; those alone read the values
// of t, from the L2.
template <int N, int OFF, int NO, bool WT>
__device__ __forceinline__ void sum_records(const __amdgpu_buffer_rsrc_t rs,
                                            const RecordBlock<NO, WT, true>& b, const float to, const float tom,
                                            double& Gm) {
    constexpr int W = cluster_record_words(NO);
    uint32_t t[N][NO], sat[N];
#pragma unroll
    for (int c = 0; c < N; ++c)
#pragma unroll
        for (int j = 0; j < NO; ++j)
            t[c][j] = LdsAddress{}((b.w[(OFF + c) * W + (j >> 1)] >> (j & 1 ? 19 : 3)) & 0x1ffcu);
#pragma unroll
    for (int c = 0; c < N; ++c) {
        uint32_t any = 0;  // top bit: some other literal is true
#pragma unroll
        for (int j = 0; j < NO; ++j) {
            const uint32_t w = b.w[(OFF + c) * W + (j >> 1)];
            any |= __builtin_amdgcn_alignbit(t[c][j], t[c][j], j & 1 ? w >> 16 : w) ^
                   (b.sign << (31 - ((OFF + c) * NO + j)));
        }
        sat[c] = (uint32_t)((int)any >> 31);
    }
#pragma unroll
    for (int c = 0; c < N; ++c)
        if (sat[c] == 0) {
#pragma unroll
            for (int j = 0; j < NO; ++j) {
                const uint32_t w = b.w[(OFF + c) * W + (j >> 1)];
                t[c][j] = __builtin_amdgcn_raw_buffer_load_b32(rs, (int)((j & 1 ? w >> 14 : w << 2) & 0x3fffcu), 0, 16);
            }
        }
#pragma unroll
    for (int c = 0; c < N; ++c) {
        uint32_t z = __float_as_uint(to);
        float f = fabsf(__uint_as_float(t[c][0]));
#pragma unroll
        for (int j = 2; j <= NO; ++j) {
            uint32_t after;  // all ones where the own literal comes after literal j
            asm("v_bfe_i32 %0, %1, %2, 1" : "=v"(after) : "v"(b.bits), "n"(OFF + c + 8 * (j - 2)));
            uint32_t take;
            asm("v_bfi_b32 %0, %1, %2, %3" : "=v"(take) : "v"(after), "v"(t[c][j - 1]), "v"(z));
            asm("v_bfi_b32 %0, %1, %2, %3" : "=v"(z) : "v"(after), "v"(z), "v"(t[c][j - 1]));
            f = f + fabsf(__uint_as_float(take));
        }
        f = f + fabsf(__uint_as_float(z));
        if constexpr (WT) f = f * b.wf[OFF + c];
        uint32_t a = __float_as_uint(f * tom) & ~sat[c];
        asm("" : "+v"(a));  // the mask stays on the 32-bit value
        Gm = Gm + (double)__uint_as_float(a);
    }
}
template <int NO, bool WT>
__device__ __forceinline__ void sum_block(const __amdgpu_buffer_rsrc_t rs,
                                          const RecordBlock<NO, WT, true>& b, const int left, const float to,
                                          const float tom, double& Gm) {
    if constexpr (NO == 2) {
        if (left > 4) sum_records<8, 0>(rs, b, to, tom, Gm);
        else sum_records<4, 0>(rs, b, to, tom, Gm);
    } else {
        sum_records<4, 0>(rs, b, to, tom, Gm);
        if (left > 4) sum_records<4, 4>(rs, b, to, tom, Gm);
    }
}

// The sum over the wavefront, in every lane.
__device__ __forceinline__ uint32_t wave_sum(uint32_t v) {
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, true);   // row_shr:1
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, true);   // row_shr:2
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, true);   // row_shr:4
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, true);   // row_shr:8
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false);  // row_bcast:15
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false);  // row_bcast:31
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// One row's part in the count and the loss.
template <bool WT>
__device__ __forceinline__ void count_row(const bool unsat, const float f, const HMS_GLOBAL int64_t* c_w,
                                          const size_t row, const bool want_loss, unsigned long long& cnt, double& los) {
    if constexpr (WT) {
        const int64_t w = unsat ? c_w[row] : 0;
        cnt += (unsigned long long)w;
        if (want_loss && unsat) los += ((double)f * (double)f) * (double)w;
    } else {
        cnt += (unsigned long long)__popcll(__ballot(unsat));
        if (want_loss && unsat) los += (double)f * (double)f;
    }
}

// Unsatisfied weight of clause tiles ct0, ct0 + stride, ...; the loss terms are
// added to los.  Both are the wavefront's sums.
template <bool WT, class Lds>
__device__ __forceinline__ unsigned long long count_clauses(const Lds lds, const uint32_t at,
                                                            const TileDesc* c_tile, const HMS_GLOBAL uint32_t* cslot,
                                                            const HMS_GLOBAL int64_t* c_w, const int c_tiles,
                                                            const int ct0, const int stride, const int lane,
                                                            const bool want_loss, double& los) {
    unsigned long long cnt = 0;
    double l = 0.0;
    for (int ct = ct0; ct < c_tiles; ct += stride) {
        const TileDesc d = ldtile(c_tile + ct);
        if (d.flags & 1u) continue;  // tautologies are never unsatisfied
        float f = 0.0f;
        uint32_t all = ~0u;
#pragma unroll 5
        for (uint32_t c = 0; c < d.len; ++c) {
            const uint32_t en = cslot[(size_t)d.base + (size_t)c * kTile + lane];
            const uint32_t b = lds(((en & kIdx) << 2) | at) ^ (en & kSign);
            f = f + __uint_as_float(b);
            all &= b;
        }
        count_row<WT>(lane < (int)d.nreal && (all >> 31) != 0, f, c_w, (size_t)ct * kTile + lane, want_loss, cnt, l);
    }
    if constexpr (WT)
        for (int o = 32; o >= 1; o >>= 1) cnt += __shfl_xor(cnt, o);
    if (want_loss) {
        for (int o = 32; o >= 1; o >>= 1) l += __shfl_xor(l, o);
        los += l;
    }
    return cnt;
}

// The same in the wide form (t only where the loss is wanted).
template <bool WT>
__device__ __forceinline__ unsigned long long count_clauses_wide(const __amdgpu_buffer_rsrc_t rs,
                                                                 const TileDesc* c_tile,
                                                                 const HMS_GLOBAL uint32_t* cslot,
                                                                 const HMS_GLOBAL int64_t* c_w, const int c_tiles,
                                                                 const int ct0, const int stride, const int lane,
                                                                 const bool want_loss, double& los) {
    unsigned long long cnt = 0;
    double l = 0.0;
    for (int ct = ct0; ct < c_tiles; ct += stride) {
        const TileDesc d = ldtile(c_tile + ct);
        if (d.flags & 1u) continue;  // tautologies are never unsatisfied
        uint32_t any = 0;
#pragma unroll 5
        for (uint32_t c = 0; c < d.len; ++c) {
            const uint32_t en = cslot[(size_t)d.base + (size_t)c * kTile + lane];
            const uint32_t b = LdsAddress{}((en >> 3) & 0x0ffffffcu);
            any |= __builtin_amdgcn_alignbit(b, b, en) ^ en;
        }
        float f = 0.0f;
        if (want_loss)
            for (uint32_t c = 0; c < d.len; ++c) {
                const uint32_t en = cslot[(size_t)d.base + (size_t)c * kTile + lane];
                const uint32_t t = __builtin_amdgcn_raw_buffer_load_b32(rs, (int)((en << 2) | (uint32_t)((int)any >> 31)), 0, 16);
                f = f + __uint_as_float(t ^ (en & kSign));
            }
        count_row<WT>(lane < (int)d.nreal && (any >> 31) == 0, f, c_w, (size_t)ct * kTile + lane, want_loss, cnt, l);
    }
    if constexpr (WT)
        for (int o = 32; o >= 1; o >>= 1) cnt += __shfl_xor(cnt, o);
    if (want_loss) {
        for (int o = 32; o >= 1; o >>= 1) l += __shfl_xor(l, o);
        los += l;
    }
    return cnt;
}

// One clause tile's entries in registers (clauses of at most kClusterMaxK
// literals), for a wavefront that counts it every time.
struct ClauseCache {
    uint32_t en[kClusterMaxK];
    int len = 0, tile = 0;
    bool real = false;
    __device__ __forceinline__ void load(const TileDesc* c_tile, const HMS_GLOBAL uint32_t* cslot, const int ct,
                                         const int c_tiles, const int lane) {
        if (ct >= c_tiles) return;
        const TileDesc d = ldtile(c_tile + ct);
        if (d.flags & 1u) return;
        tile = ct;
        len = (int)d.len;
        real = lane < (int)d.nreal;
#pragma unroll
        for (int c = 0; c < kClusterMaxK; ++c)
            if (c < len) en[c] = cslot[(size_t)d.base + (size_t)c * kTile + lane];
    }
    template <bool WT>
    __device__ __forceinline__ unsigned long long count(const LdsIndex lds, const uint32_t at,
                                                        const HMS_GLOBAL int64_t* c_w, const bool want_loss, double& los,
                                                        const int lane) const {
        los = 0.0;
        unsigned long long cnt = 0;
        if (len == 0) return 0;
        float f = 0.0f;
        uint32_t all = ~0u, b[kClusterMaxK];
#pragma unroll
        for (int c = 0; c < kClusterMaxK; ++c)
            if (c < len)
                b[c] = lds(((en[c] & kIdx) << 2) | at) ^ (en[c] & kSign);
#pragma unroll
        for (int c = 0; c < kClusterMaxK; ++c)
            if (c < len) {
                f = f + __uint_as_float(b[c]);
                all &= b[c];
            }
        count_row<WT>(real && (all >> 31) != 0, f, c_w, (size_t)tile * kTile + lane, want_loss, cnt, los);
        if constexpr (WT)
            for (int o = 32; o >= 1; o >>= 1) cnt += __shfl_xor(cnt, o);
        if (want_loss)
            for (int o = 32; o >= 1; o >>= 1) los += __shfl_xor(los, o);
        return cnt;
    }
};

// The flag exchange, after the workgroup's flag is out: a wavefront waits for
// its one or two peers (one per lane), then copies its part of their slices
// into LDS (16 / C wavefronts per peer, two whole slices each with 32
// workgroups).
template <bool WIDE = false>
__device__ __forceinline__ void collect(const ClusterGroup& G, Shared& sh, unsigned char* smem, HMS_GLOBAL float* tb,
                                        const int member, const int C, const int log2C, const int slice,
                                        const int wave, const int lane, const int step, const bool eval,
                                        const bool last) {
    const int par = step & 1;
    const int parts = C <= kWaves ? kWaves >> log2C : 1;
    const int rounds = C <= kWaves ? 1 : C / kWaves;
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
    flag_seen();
    if (__ballot(!ok) != 0) sh.dead = 1;
    if (eval && part == 0 && lane < rounds) atomicAdd(&sh.tot[par], (unsigned long long)(f >> 32));
    if (last) return;
    // device-scope loads: from the L2, never from this CU's L1
    const int P = C * slice;
    if constexpr (WIDE) {
        // a word of roundings per tile (tb: where they are kept)
        const HMS_GLOBAL uint64_t* from = (const HMS_GLOBAL uint64_t*)tb;
        uint64_t* to = reinterpret_cast<uint64_t*>(smem);
        const int st = slice / 64, nt = rounds * st;
        for (int i = part * 64 + lane; i < nt; i += parts * 64) {
            const int w = i < st ? peer0 * st + i : peer1 * st + (i - st);
            to[w] = __hip_atomic_load(from + w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        return;
    }
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void*)tb, 0, P * 4, 0x00020000);
    const int s4 = slice / 4;
    u32x4* dst = reinterpret_cast<u32x4*>(smem);
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

// Initial value of variable v (o: its place in the caller's order).
__device__ __forceinline__ float start_x(const ClusterDesc& D, const int r, const int v, int& o) {
    o = D.var_old[v];
    if (D.x0 != nullptr) return D.x0[(size_t)o * D.R + r];
    const uint64_t z = splitmix64(D.seed + (uint64_t)r, (uint64_t)o + 1);
    return 2.0f * ((float)(z >> 40) * (1.0f / 16777216.0f)) - 1.0f;
}

// Variables in no clause keep their start (all threads of one workgroup).
__device__ __forceinline__ void keep_inactive(const ClusterDesc& D, const int r, const int tid, uint8_t* best_a) {
    for (int v = D.n_act + tid; v < D.n; v += kClusterThreads) {
        int o;
        const float x = start_x(D, r, v, o);
        const size_t e = (size_t)o * D.R + r;
        if (!D.resume) best_a[o] = x > 0.0f ? 1 : 0;
        if (D.x_final != nullptr) D.x_final[e] = x;
        if (D.m_final != nullptr) {
            D.m_final[e] = D.m0 != nullptr ? D.m0[e] : 0.0f;
            D.v_final[e] = D.v0 != nullptr ? D.v0[e] : 0.0f;
        }
    }
}

// Registration of a workgroup (one thread): its place on its XCD, then the
// wait until the whole cluster has arrived.  sh.group is null when there is
// nothing to do: no cluster left for this ticket, or one that did not fill.
__device__ void enroll(const ClusterLaunch& A, const unsigned char* smem, Shared& sh) {
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
    if ((uint32_t)(uintptr_t)(const __attribute__((address_space(3))) unsigned char*)smem != 0) g = nullptr;
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
            if (wall_clock64() - t0 > A.wait_ticks) {
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
    sh.cnt[0] = sh.cnt[1] = sh.tot[0] = sh.tot[1] = sh.tot[2] = sh.tot[3] = 0;
}

// Several variable tiles per wavefront, state in LDS.  3-CNF n = 20000, 64
// restarts: 11.7 us a step, bound by vector instructions (24460 in a CU's 27600
// cycles a step; without the optimizer's 130 per tile 9.2 us, without copying
// t 11.4, with the records always the same 11.8 where all takes 11.9).  A record
// costs 17 of them.  Taking 16-bit slots out with one instruction each
// (sub-dword addressing) saves one and gains nothing: it issues at half rate.
//
// WIDE: for more variables than t fits LDS for (past 30720 with 32 workgroups,
// 31744 with 16).  LDS holds the roundings, a bit each, which decide for every
// record whether its clause is unsatisfied; t itself is gathered from the L2
// only in the lanes (a tenth or so) where it is.  An iteration exchanges the
// bits, not t.  Bound by the latency of those gathers and the stream of records
// (with neither: 4.3 of 7.9 us a step at n = 33000, 5.4 of 11.4 at n = 55566).
// A literal takes 16 bits (with 32 the records no longer stay in the L2: 10.8
// and 13.6), and the second half of a row's last block is loaded only where it
// is used (which does not pay with t in LDS: 12.5 against 11.9 us at n = 20000,
// 64 restarts).
template <int NO, bool WT, bool WIDE>
__global__ __launch_bounds__(kClusterThreads) void k_cluster(ClusterLaunch A) {
    constexpr int W = cluster_record_words(NO);
    extern __shared__ __align__(16) unsigned char smem[];
    Shared& sh = *reinterpret_cast<Shared*>(smem + A.shared_off);

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    escape_lds(smem);
    if (tid == 0) enroll(A, smem, sh);
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
    const int P = C * slice;
    const int ntl = (D.v_tiles - member + C - 1) >> log2C;  // own variable tiles
    // t of all variables, or (WIDE) their roundings; own t is kept in lo then
    float* lt = reinterpret_cast<float*>(smem);
    uint64_t* lround = reinterpret_cast<uint64_t*>(smem);
    float* lx = reinterpret_cast<float*>(smem + (WIDE ? cluster_bits_bytes(C, slice) : cluster_t_bytes(C, slice)));
    float* lm = lx + slice;
    float* lv = lm + slice;
    float* lo = lv + slice;
    uint64_t* pbits = reinterpret_cast<uint64_t*>(WIDE ? lo + slice : lo);
    const int TP = WIDE ? P + 64 : P;  // places of one copy of t in the exchange buffer
    HMS_GLOBAL uint64_t* rbuf = (HMS_GLOBAL uint64_t*)(G.tbuf + 2 * (size_t)TP);  // WIDE: [2][P / 64]
    uint64_t* bbits = pbits + slice / 64;
    uint8_t* best_a = D.best_a + (size_t)r * n;

    // ---- initial point ----------------------------------------------------------
    for (int i = tid; i < P; i += kClusterThreads) {
        const int v = D.var[i];
        int o = 0;
        const float x = v >= 0 ? start_x(D, r, v, o) : 0.0f;
        const float t = signed_tanh(x);
        const int l = i - member * slice;
        if constexpr (WIDE) {
            // every workgroup writes the start of all variables, the same
            // values: what it reads in step 0 is there once its own stores are
            __hip_atomic_store((HMS_GLOBAL float*)G.tbuf + TP + wide_pos((uint32_t)i), t, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_WORKGROUP);
            const uint64_t bits = __ballot(x > 0.0f);
            if (lane == 0) lround[i / 64] = bits;
            if (l >= 0 && l < slice) lo[l] = t;
        } else {
            lt[i] = t;
        }
        if (l >= 0 && l < slice) {
            lx[l] = x;
            lm[l] = v >= 0 && D.m0 != nullptr ? D.m0[(size_t)o * D.R + r] : 0.0f;
            lv[l] = v >= 0 && D.v0 != nullptr ? D.v0[(size_t)o * D.R + r] : 0.0f;
        }
    }
    if (tid == 0) {
        if constexpr (WIDE) {
            lround[P / 64] = 2;  // slot P: a literal that is false, P + 1: one that is true
            for (int c = 0; c < 2; ++c)
                __hip_atomic_store((HMS_GLOBAL float*)G.tbuf + c * (size_t)TP + wide_pos((uint32_t)P), -0.0f,
                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        } else {
            lt[P] = -0.0f;     // a literal that is false
            lt[P + 1] = 0.0f;  // a literal that is true
        }
    }
    if constexpr (WIDE) stores_done();
    if (member == 0) keep_inactive(D, r, tid, best_a);
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

    // own tiles of this wavefront
    const int my_tiles = ntl > wave ? (ntl - 1 - wave) / kWaves + 1 : 0;
    auto own_tile = [&](int i) { return i * kWaves + wave; };
    RecordBlock<NO, WT, WIDE> ra, rb;  // record blocks in turn: one in use, the next one loading
    bool turn = false;                 // rb is the one in use
    auto fetch = [&](RecordBlock<NO, WT, WIDE>& b, int block, int left, bool neg) { b.load(rec, wrec, block, left, neg, lane); };
    auto tile_info = [&](int i) {
        const uint32_t* p = reinterpret_cast<const uint32_t*>(tiles + (own_tile(i) * C + member));
        return make_int2((int)ldc(p), (int)ldc(p + 1));
    };
    int2 tn = make_int2(0, 0);
    if (my_tiles > 0) {
        tn = tile_info(0);
        fetch(ra, __builtin_amdgcn_readfirstlane(tn.x), __builtin_amdgcn_readfirstlane(tn.y), lx[own_tile(0) * 64 + lane] > 0.0f);
    }

    int kc = step0 % K;
    for (int step = 0; step <= T; ++step) {
        const bool last = step == T;
        const bool eval = kc == 0 || last;
        if (++kc == K) kc = 0;
        const bool want_loss = last || (eval && D.trace != nullptr);
        const int par = step & 1;
        HMS_GLOBAL float* tb = (HMS_GLOBAL float*)G.tbuf + (size_t)par * TP;
        // this iterate's t (WIDE): written in the step before
        const __amdgpu_buffer_rsrc_t rs =
            __builtin_amdgcn_make_buffer_rsrc((void*)(G.tbuf + (size_t)(par ^ 1) * TP), 0, TP * 4, 0x00020000);
        // ---- count and loss of this iterate ------------------------------------
        if (eval) {
            // the clause tiles are dealt out from the last wavefront on (the
            // variable tiles start at the first)
            double los = 0.0;
            unsigned long long cnt;
            if constexpr (WIDE)
                cnt = count_clauses_wide<WT>(rs, c_tile, cslot, c_w, c_tiles, (kWaves - 1 - wave) * C + member,
                                             kWaves * C, lane, want_loss, los);
            else
                cnt = count_clauses<WT>(LdsAddress{}, 0u, c_tile, cslot, c_w, c_tiles, (kWaves - 1 - wave) * C + member,
                                        kWaves * C, lane, want_loss, los);
            if (lane == 0 && cnt != 0) atomicAdd(&sh.cnt[par], cnt);
            if (want_loss && lane == 0) sh.los[wave] = los;
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
                const float to = WIDE ? lo[l] : lt[member * slice + l];
                double Gm = 0.0;
                // the next tile; the last one's next is fetched once its x is known
                const bool more = i + 1 < my_tiles;
                if (more) tn = tile_info(i + 1);
                const float xn = lx[own_tile(more ? i + 1 : i) * 64 + lane];
                for (int k = 0; k < len; k += 8) {
                    const int left = len - k;
                    auto block = [&](RecordBlock<NO, WT, WIDE>& b, RecordBlock<NO, WT, WIDE>& nx) {
                        // the block in use has arrived before the next one's loads go out: its wait
                        // would be for both
#pragma unroll
                        for (int j = 0; j < 8 * W; ++j) asm volatile("" : "+v"(b.w[j]));
                        asm volatile("" : "+v"(b.bits));
                        if (left > 8) fetch(nx, tb0 + (k >> 3) + 1, left - 8, xo > 0.0f);
                        else if (more) fetch(nx, __builtin_amdgcn_readfirstlane(tn.x), __builtin_amdgcn_readfirstlane(tn.y), xn > 0.0f);
                        if constexpr (WIDE) sum_block(rs, b, left, to, tom, Gm);
                        else sum_block(LdsAddress{}, 0u, b, left, to, tom, Gm);
                    };
                    if (turn) block(rb, ra);
                    else block(ra, rb);
                    turn = !turn;
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
                const float t = signed_tanh_call(x);
                const uint32_t at = (uint32_t)(member * slice + l);
                __hip_atomic_store(tb + (WIDE ? wide_pos(at) : at), t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                if constexpr (WIDE) {
                    lo[l] = t;
                    const uint64_t up = __ballot(x > 0.0f);
                    if (lane == 0)
                        __hip_atomic_store(rbuf + (size_t)par * (P / 64) + member * (slice / 64) + q, up,
                                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                }
            }
            // the next step's first block, in flight over the exchange
            if (my_tiles > 0) {
                tn = tile_info(0);
                fetch(ra, __builtin_amdgcn_readfirstlane(tn.x), __builtin_amdgcn_readfirstlane(tn.y), lx[own_tile(0) * 64 + lane] > 0.0f);
                turn = false;
            }
        }
        // ---- the step's flag: own stores have reached the L2 ------------------
        // flags and losses alternate between two places: a workgroup that is
        // done may publish the next step while another still reads this one,
        // but not the one after, which needs the other's next flag
        stores_done();
        __syncthreads();
        if (tid == 0) {
            if (want_loss) {
                double ls = 0.0;
                for (int w = 0; w < kWaves; ++w) ls = ls + sh.los[w];
                __hip_atomic_store(G.losses + par * C + member, ls, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                stores_done();
            }
            const uint64_t f = (uint64_t)(uint32_t)(step + 1) | ((uint64_t)sh.cnt[par] << 32);
            __hip_atomic_store((HMS_GLOBAL uint64_t*)G.flags + (size_t)member * kFlagStride + par, f, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            sh.cnt[par ^ 1] = 0;
            sh.tot[par ^ 1] = 0;
        }
        // ---- every workgroup's new t (and count) ------------------------------
        if constexpr (WIDE)
            collect<true>(G, sh, smem, (HMS_GLOBAL float*)(rbuf + (size_t)par * (P / 64)), member, C, log2C, slice, wave,
                          lane, step, eval, last);
        else
            collect(G, sh, smem, tb, member, C, log2C, slice, wave, lane, step, eval, last);
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

// At most one variable tile per wavefront: x, m, v and the records of the list
// in use stay in registers (the records are loaded again when a variable's
// rounding turns), and what the next step needs of x alone (sech^2) is taken
// while the exchange is under way.  A step is one chain of latencies, so every
// link counts.
//
// EX (up to kOneSlots LDS slots): t goes out as 64-bit words {t, step} and every
// thread polls the slots it copies, so there is no flag to wait for: the
// workgroup barrier before it, the wait for the stores' acknowledgement and one
// round trip through the L2 go.  t is held twice in LDS (a slow wavefront still
// gathers the old values while others fill in the new), the second copy at byte
// kAltByte.  The lower half of the wavefronts holds the variable tiles and
// copies t; those without a tile count, their clause tiles' entries in
// registers, and publish {step, count} per wavefront, which the upper half
// collects one step later, when it has long arrived; the best is brought up to
// date then.  Collected counts are summed over lanes before they go to LDS (64
// atomics on one address held the barrier for 1.1 us).  Counts and losses are
// kept for four steps: a workgroup may be one step ahead of another that still
// collects the step before.
//
// us a step, against the flag exchange, the form for many tiles and the
// resident solver: mixed n = 1000, 16 restarts 2.74 counting every step and 2.65
// every 50 (3.49 and 2.87; 3.68 and 3.44; 3.63 and 3.09); 3-CNF n = 4000, one
// restart 2.56 (2.79; 3.40; -).  More wavefronts for t and fewer for the count
// lose with a count every step (4.7 with half of the wavefronts counting).
template <int NO, bool WT, bool EX>
__global__ __launch_bounds__(kClusterThreads) void k_cluster_one(ClusterLaunch A) {
    extern __shared__ __align__(16) unsigned char smem[];
    Shared& sh = *reinterpret_cast<Shared*>(smem + A.shared_off);
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (tid == 0) enroll(A, smem, sh);
    __syncthreads();
    const ClusterGroup* gp = uniform(sh.group);
    if (gp == nullptr) return;
    const ClusterGroup G = load_uniform(gp);
    const ClusterDesc* dp = G.desc;
    const int member = __builtin_amdgcn_readfirstlane(sh.member);
    const int C = G.C;
    const int r = G.r;
    int P, slice;
    bool mine, own_bit = false;
    int var = -1, o = 0, best_step;
    float x = 0.0f, m = 0.0f, v = 0.0f;
    int64_t best;
    RecordBlock<NO, WT> b0, b1;
    int len = 0, block0 = 0;
    ClauseCache cache;
    float tom, lr;
    AdamCoef co;
    int T, K, opt, kc;
    const uint32_t* scal;
    const HMS_GLOBAL int64_t* c_w;
    // EX: the slots this thread copies (bit j: slot tid + 512 j is a real
    // tile's) and whether it collects a count word
    constexpr int kHalf = kClusterThreads / 2;
    constexpr int NP = kOneSlots / kHalf;
    int CW;  // counting wavefronts, those without a tile (the last CW)
    uint32_t todo_t = 0;
    bool todo_c = false, counting;
    {
    const ClusterDesc D = load_uniform(launder(dp));
    slice = D.slice;
    P = C * slice;
    CW = kWaves - slice / 64;
    mine = wave * C + member < D.v_tiles;  // this wavefront's tile
    float* lt = reinterpret_cast<float*>(smem);
    uint8_t* best_a = D.best_a + (size_t)r * D.n;

    // ---- initial point ----------------------------------------------------------
    for (int i = tid; i < P; i += kClusterThreads) {
        const int v = D.var[i];
        int o;
        lt[i] = v >= 0 ? signed_tanh(start_x(D, r, v, o)) : 0.0f;
    }
    if (tid == 0)
        for (int k = 0; k < (EX ? 2 : 1); ++k) {
            float* p = reinterpret_cast<float*>(smem + (k ? kAltByte : 0u));
            p[P] = -0.0f;     // a literal that is false
            p[P + 1] = 0.0f;  // a literal that is true
        }
    if (member == 0) keep_inactive(D, r, tid, best_a);
    if (mine) var = D.var[member * slice + wave * 64 + lane];
    if (var >= 0) {
        x = start_x(D, r, var, o);
        const size_t e = (size_t)o * D.R + r;
        if (D.m0 != nullptr) m = D.m0[e];
        if (D.v0 != nullptr) v = D.v0[e];
        own_bit = D.resume ? best_a[o] != 0 : x > 0.0f;
    }
    best = D.resume ? D.best[r] : D.best0;
    best_step = D.resume ? D.best_step[r] : -1;
    co = AdamCoef{D.b1, D.b2, D.eps, D.omb1, D.omb2};
    tom = D.two_over_m;
    lr = D.lr;
    T = D.T;
    K = D.K;
    opt = D.opt;
    kc = D.step0 % K;
    scal = reinterpret_cast<const uint32_t*>(D.scal);
    c_w = (const HMS_GLOBAL int64_t*)D.c_w;
    if (mine) {
        const uint32_t* p = reinterpret_cast<const uint32_t*>(D.tile + (wave * C + member));
        block0 = __builtin_amdgcn_readfirstlane((int)ldc(p));
        len = __builtin_amdgcn_readfirstlane((int)ldc(p + 1));
        const HMS_GLOBAL uint32_t* rec = (const HMS_GLOBAL uint32_t*)D.rec;
        const HMS_GLOBAL float* wrec = (const HMS_GLOBAL float*)D.wrec;
        b0.load(rec, wrec, block0, 8, x > 0.0f, lane);
        if (len > 8) b1.load(rec, wrec, block0 + 1, 8, x > 0.0f, lane);
    }
    if constexpr (EX) {
        if (tid < kHalf) {
#pragma unroll
            for (int j = 0; j < NP; ++j) {
                const int i = tid + j * kHalf;
                if (i < P && (i % slice) / 64 * C + i / slice < D.v_tiles) todo_t |= 1u << j;
            }
        }
        // word i: workgroup i / CW, its wavefront kWaves - 1 - i % CW.  Published
        // as far as there are clause tiles, the last wavefront's always (the
        // loss goes before it)
        const int i = tid - kHalf;
        todo_c = i >= 0 && i < CW * C && (i % CW == 0 || i % CW * C + i / CW < D.c_tiles);
    }
    counting = !EX || (wave >= kWaves - CW && (wave == kWaves - 1 || (kWaves - 1 - wave) * C + member < D.c_tiles));
    if (EX && counting)
        cache.load(D.c_tile, (const HMS_GLOBAL uint32_t*)D.cslot, (kWaves - 1 - wave) * C + member, D.c_tiles, lane);
    }
    // from here on what only some steps need is read again where it is needed:
    // kept, it would fill the scalar registers and spill
    const int np = (P + kHalf - 1) / kHalf;
    HMS_GLOBAL uint64_t* words = (HMS_GLOBAL uint64_t*)G.tbuf;   // [2][P]
    HMS_GLOBAL uint64_t* counts = (HMS_GLOBAL uint64_t*)G.flags; // [4][CW C]
    float to = signed_tanh(x);
    float s2 = sech2f(x);
    bool neg = x > 0.0f;
    bool pend = false, pend_was = false;  // the step before was counted; the rounding it had
    // this thread's count word of iterate `it`, when it has arrived
    auto count_of = [&](int it, uint32_t& got, bool& left) {
        if (!left) return;
        const uint64_t c = __hip_atomic_load(counts + (it & 3) * CW * C + tid - kHalf, __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_AGENT);
        if ((uint32_t)c != (uint32_t)(it + 1)) return;
        got = (uint32_t)(c >> 32);
        left = false;
    };
    auto add_counts = [&](uint32_t got, unsigned long long* tot) {
        const unsigned long long sum =
            WT ? ((unsigned long long)wave_sum(got >> 16) << 16) + wave_sum(got & 0xffffu) : wave_sum(got);
        if (lane == 0 && sum != 0) atomicAdd(tot, sum);
    };
    // the outcome of iterate `it`, counted in full
    auto outcome = [&](int it, bool bit, unsigned long long total, int lpar) {
        const ClusterDesc* d = launder(dp);
        const int64_t c = load_uniform(&d->w_empty) + (int64_t)total;
        if (c < best) {
            best = c;
            best_step = load_uniform(&d->step0) + it;
            own_bit = bit;
        }
        if (member != 0) return;
        TracePoint* trace = load_uniform(&d->trace);
        if ((it == T || trace != nullptr) && tid == 0) {
            double* losses = load_uniform(&launder(gp)->losses);
            double ls = 0.0;
            for (int p = 0; p < C; ++p)
                ls = ls + __hip_atomic_load(losses + lpar * C + p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            ls = ls * load_uniform(&d->inv_m);
            if (it == T) load_uniform(&d->final_loss)[r] = ls;
            if (trace != nullptr) {
                const int64_t s0 = load_uniform(&d->step0);
                const int64_t gs = s0 + it;
                const int64_t row = ((gs + K - 1) / K - (s0 + K - 1) / K) % load_uniform(&d->trace_cap);
                trace[(size_t)row * load_uniform(&d->R) + r] = TracePoint{(int32_t)gs, 0, c, ls};
            }
        }
    };
    const bool traced = load_uniform(&launder(dp)->trace) != nullptr;
    __syncthreads();

    for (int step = 0; step <= T; ++step) {
        const bool last = step == T;
        const bool eval = kc == 0 || last;
        if (++kc == K) kc = 0;
        const bool want_loss = last || (eval && traced);
        const int par = step & 1;
        const uint32_t at = EX && par ? kAltByte : 0u;
        const uint32_t epoch = (uint32_t)(step + 1);
        HMS_GLOBAL float* tb = (HMS_GLOBAL float*)G.tbuf + (size_t)par * P;
        if (eval && counting) {
            double los = 0.0;
            unsigned long long cnt = 0;
            const int first = (kWaves - 1 - wave) * C + member;
            if constexpr (EX) cnt = cache.count<WT>(LdsIndex{smem}, at, c_w, want_loss, los, lane);
            const ClusterDesc* d = launder(dp);
            const int c_tiles = load_uniform(&d->c_tiles);
            if (!EX || first + CW * C < c_tiles)
                cnt += count_clauses<WT>(LdsIndex{smem}, at, load_uniform(&d->c_tile),
                                         (const HMS_GLOBAL uint32_t*)load_uniform(&d->cslot), c_w, c_tiles,
                                         EX ? first + CW * C : first, (EX ? CW : kWaves) * C, lane, want_loss, los);
            if (lane == 0) {
                if constexpr (EX) {
                    if (want_loss) {
                        sh.los[wave] = los;
                        sh.wcnt[wave] = cnt;
                    } else {
                        __hip_atomic_store(counts + ((step & 3) * C + member) * CW + (kWaves - 1 - wave),
                                           (uint64_t)epoch | ((uint64_t)cnt << 32), __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_WORKGROUP);
                    }
                } else {
                    if (cnt != 0) atomicAdd(&sh.cnt[par], cnt);
                    if (want_loss) sh.los[wave] = los;
                }
            }
        }
        const bool was = x > 0.0f;
        if (mine && !last) {
            float2 sc = make_float2(0.0f, 1.0f);
            if (opt != kSgd)
                sc = make_float2(__uint_as_float(ldc(scal + 2 * step)), __uint_as_float(ldc(scal + 2 * step + 1)));
            double Gm = 0.0;
            sum_block(LdsIndex{smem}, at, b0, len, to, tom, Gm);
            if (len > 8) sum_block(LdsIndex{smem}, at, b1, len - 8, to, tom, Gm);
            for (int k = 16; k < len; k += 8) {
                RecordBlock<NO, WT> b;
                const ClusterDesc* d = launder(dp);
                b.load((const HMS_GLOBAL uint32_t*)load_uniform(&d->rec), (const HMS_GLOBAL float*)load_uniform(&d->wrec),
                       block0 + (k >> 3), 8, neg, lane);
                sum_block(LdsIndex{smem}, at, b, len - k, to, tom, Gm);
            }
            // a positive literal in the loss adds -a, a negative one +a (0.0 - 0.0 keeps an empty sum +0)
            const double Gs = was ? Gm : 0.0 - Gm;
            const float g = (float)((double)s2 * Gs);
            if (opt == kSgd) x = x - lr * g;
            else adam_update(x, m, v, g, sc.x, sc.y, co);
            to = signed_tanh_call(x);
            const int slot = member * slice + wave * 64 + lane;
            if constexpr (EX)
                __hip_atomic_store(words + (size_t)par * P + slot, (uint64_t)__float_as_uint(to) | ((uint64_t)epoch << 32),
                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            else
                __hip_atomic_store(tb + slot, to, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            // the next step's share that needs x alone
            neg = x > 0.0f;
            if (__ballot(neg != was) != 0) {
                const ClusterDesc* d = launder(dp);
                const HMS_GLOBAL uint32_t* rec = (const HMS_GLOBAL uint32_t*)load_uniform(&d->rec);
                const HMS_GLOBAL float* wrec = (const HMS_GLOBAL float*)load_uniform(&d->wrec);
                b0.load(rec, wrec, block0, 8, neg, lane);
                if (len > 8) b1.load(rec, wrec, block0 + 1, 8, neg, lane);
            }
            s2 = sech2f(x);
        }
        if constexpr (EX) {
            if (want_loss) {
                // all partial losses before the counts that stand for them
                __syncthreads();
                if (wave == kWaves - 1 && lane == 0) {
                    const int c_tiles = load_uniform(&launder(dp)->c_tiles);
                    double* losses = load_uniform(&launder(gp)->losses);
                    double ls = 0.0;
                    for (int w = 0; w < CW; ++w)
                        if (w == 0 || w * C + member < c_tiles) ls = ls + sh.los[kWaves - 1 - w];
                    __hip_atomic_store(losses + (step & 3) * C + member, ls, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_WORKGROUP);
                    stores_done();
                    for (int w = 0; w < CW; ++w)
                        if (w == 0 || w * C + member < c_tiles)
                            __hip_atomic_store(counts + ((step & 3) * C + member) * CW + w,
                                               (uint64_t)epoch | ((uint64_t)sh.wcnt[kWaves - 1 - w] << 32),
                                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                }
            }
            int spins = 0;
            if (wave < kWaves / 2) {
                // the new t of every slot, into the next step's copy
                uint32_t left = last ? 0u : todo_t;
                unsigned char* next = smem + (par ? 0u : kAltByte) + 4 * tid;
                const HMS_GLOBAL uint64_t* from = words + (size_t)par * P + tid;
                while (__ballot(left != 0) != 0) {
                    uint64_t w[NP];
#pragma unroll
                    for (int j = 0; j < NP; ++j)
                        if (j < np) {
                            if (left & (1u << j))
                                w[j] = __hip_atomic_load(from + j * kHalf, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        }
#pragma unroll
                    for (int j = 0; j < NP; ++j)
                        if (j < np) {
                            if ((left & (1u << j)) && (uint32_t)(w[j] >> 32) == epoch) {
                                *reinterpret_cast<uint32_t*>(next + 4 * j * kHalf) = (uint32_t)w[j];
                                left &= ~(1u << j);
                            }
                        }
                    if (++spins > kSpinLimit) {
                        sh.dead = 1;
                        break;
                    }
                }
            } else {
                // the counts of the step before (and, at the end, of this one)
                bool left_p = pend && todo_c, left_c = last && todo_c;
                uint32_t got_p = 0, got_c = 0;
                while (__ballot(left_p || left_c) != 0) {
                    count_of(step - 1, got_p, left_p);
                    count_of(step, got_c, left_c);
                    if (++spins > kSpinLimit) {
                        sh.dead = 1;
                        break;
                    }
                }
                if (tid - kHalf < (CW * C + 63 & ~63)) {
                    if (pend) add_counts(got_p, &sh.tot[step % 3]);
                    if (last) add_counts(got_c, &sh.tot[3]);
                }
            }
        } else {
            // own stores have reached the L2, then the flag
            stores_done();
            __syncthreads();
            if (tid == 0) {
                if (want_loss) {
                    double ls = 0.0;
                    for (int w = 0; w < kWaves; ++w) ls = ls + sh.los[w];
                    __hip_atomic_store(load_uniform(&launder(gp)->losses) + par * C + member, ls, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                    stores_done();
                }
                __hip_atomic_store((HMS_GLOBAL uint64_t*)G.flags + (size_t)member * kFlagStride + par,
                                   (uint64_t)epoch | ((uint64_t)sh.cnt[par] << 32), __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_WORKGROUP);
                sh.cnt[par ^ 1] = 0;
                sh.tot[par ^ 1] = 0;
            }
            collect(G, sh, smem, tb, member, C, __builtin_ctz(C), slice, wave, lane, step, eval, last);
        }
        __syncthreads();
        if (__builtin_amdgcn_readfirstlane(sh.dead)) break;
        if constexpr (EX) {
            // three totals in turn; the one cleared here was last read before
            // this barrier and is next added to after the next one
            if (tid == 0) sh.tot[(step + 2) % 3] = 0;
            if (pend) outcome(step - 1, pend_was, sh.tot[step % 3], (step - 1) & 3);
            if (last) outcome(step, was, sh.tot[3], step & 3);
            pend = eval;
            pend_was = was;
        } else if (eval) {
            outcome(step, was, sh.tot[par], par);
        }
    }
    if (__builtin_amdgcn_readfirstlane(sh.dead)) {
        if (tid == 0) __hip_atomic_store(load_uniform(&launder(gp)->ctl) + 2, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return;
    }
    const ClusterDesc D = load_uniform(launder(dp));
    if (var >= 0) {
        const size_t e = (size_t)o * D.R + r;
        D.best_a[(size_t)r * D.n + o] = own_bit ? 1 : 0;
        if (D.x_final != nullptr) D.x_final[e] = x;
        if (D.m_final != nullptr) {
            D.m_final[e] = m;
            D.v_final[e] = v;
        }
    }
    if (member == 0 && tid == 0) {
        D.best[r] = best;
        D.best_step[r] = best_step;
    }
}

std::mutex g_cluster_attr_mu;

template <typename Kernel>
hipError_t launch_as(Kernel kernel, ClusterLaunch L, size_t lds, size_t lds_cap, hipStream_t s,
                     std::atomic<uint64_t>& set_on) {
    L.shared_off = (int32_t)(lds - sizeof(Shared));
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const uint64_t bit = dev >= 0 && dev < 64 ? uint64_t(1) << dev : 0;
    if (!bit || !(set_on.load(std::memory_order_acquire) & bit)) {
        std::lock_guard<std::mutex> lk(g_cluster_attr_mu);
        e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)lds_cap);
        if (e != hipSuccess) return e;
        set_on.fetch_or(bit, std::memory_order_release);
    }
    // one workgroup per CU: they are dealt round-robin over the XCDs, so every
    // XCD gets kXcdCus tickets; the surplus exits at once
    hipLaunchKernelGGL(kernel, dim3(kXcds * kXcdCus), dim3(kClusterThreads), lds, s, L);
    return hipGetLastError();
}

template <int NO, bool WT>
hipError_t launch_mode(const ClusterLaunch& L, const ClusterShape& sh, size_t lds_cap, hipStream_t s) {
    static std::atomic<uint64_t> set_on[4];  // bit d: the kernel's attribute is set on device d
    switch (sh.mode) {
        case kClusterMany: return launch_as(k_cluster<NO, WT, false>, L, sh.lds, lds_cap, s, set_on[0]);
        case kClusterWide: return launch_as(k_cluster<NO, WT, true>, L, sh.lds, lds_cap, s, set_on[3]);
        case kClusterOne: return launch_as(k_cluster_one<NO, WT, false>, L, sh.lds, lds_cap, s, set_on[1]);
        default: return launch_as(k_cluster_one<NO, WT, true>, L, sh.lds, lds_cap, s, set_on[2]);
    }
}

}  // namespace

bool cluster_size(const HostPlan& P, ClusterSize& Z) {
    if (P.n_heavy != 0 || P.v_tiles < 2 || P.w_total >= (int64_t(1) << 32)) return false;
    uint32_t k = 0;
    for (const TileDesc& d : P.c_tile)
        if (!(d.flags & 1u)) k = std::max(k, d.len);
    if (k > (uint32_t)kClusterMaxK) return false;
    Z.v_tiles = P.v_tiles;
    Z.NO = std::max(2, (int32_t)k - 1);
    return true;
}

bool cluster_shape(const HostPlan& P, int32_t R, size_t lds_cap, ClusterShape& sh) {
    ClusterSize Z;
    return cluster_size(P, Z) && cluster_shape_of(Z, R, lds_cap, sh);
}

hipError_t launch_cluster_build(const ClusterDesc* Ds, const ClusterDesc* hostDs, int32_t count, hipStream_t s) {
    int32_t vars = 0, slots = 0, tiles = 0, T = 0;
    int64_t entries = 0;
    for (int32_t i = 0; i < count; ++i) {
        const ClusterDesc& D = hostDs[i];
        vars = std::max(vars, D.n_act);
        slots = std::max(slots, D.C * D.slice);
        tiles = std::max(tiles, D.v_tiles);
        entries = std::max(entries, D.c_ent_n);
        T = std::max(T, D.T);
    }
    hipLaunchKernelGGL(k_cluster_count, dim3((vars + 1023) / 1024, count), dim3(1024), 0, s, Ds);
    hipLaunchKernelGGL(k_cluster_scan, dim3(1, count), dim3(kClusterBins), 0, s, Ds);
    hipLaunchKernelGGL(k_cluster_rank, dim3((slots + 1023) / 1024, count), dim3(1024), 0, s, Ds);
    const int extra = (int)std::max<int64_t>(std::min<int64_t>((entries + 4095) / 4096, 1024), 1);
    hipLaunchKernelGGL(k_cluster_records, dim3(tiles + extra, count), dim3(1024), 0, s, Ds);
    if (T > 0) hipLaunchKernelGGL(k_cluster_scalars, dim3((T + 255) / 256, count), dim3(256), 0, s, Ds);
    return hipGetLastError();
}

hipError_t launch_cluster(const ClusterLaunch& L, const ClusterShape& sh, bool weighted, size_t lds_cap,
                          hipStream_t s) {
    if (sh.lds > lds_cap) return hipErrorInvalidValue;
    switch (sh.NO) {
        case 2: return weighted ? launch_mode<2, true>(L, sh, lds_cap, s) : launch_mode<2, false>(L, sh, lds_cap, s);
        case 3: return weighted ? launch_mode<3, true>(L, sh, lds_cap, s) : launch_mode<3, false>(L, sh, lds_cap, s);
        case 4: return weighted ? launch_mode<4, true>(L, sh, lds_cap, s) : launch_mode<4, false>(L, sh, lds_cap, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace hms
