// Grouped execution of a recorded program: independent products of one dependency level run as one
// launch over a table of work items.
#pragma once
#include "common.hpp"

namespace lrcc {

// One output tile of one product: rows m0.., columns n0.. of op `op`, reduction steps [t0, t1) of its
// (segment, k) range starting at segment sb, added to (beta) or stored at the block at C.
struct GroupItem {
    void *C;
    int op, m0, n0, sb, t0, t1;
    float js;          // the job's multiplier of alpha
    int beta;
    int tile;          // index into kGroupTiles
};

// out[e] = sum over nsrc arrays, `n` elements; src indexes the table of source pointers
struct SumSeg {
    void *dst;
    i64 n;
    int src0, nsrc;
};

constexpr int kGroupTK = 16;          // reduction elements per step of a grouped product
// rows, columns, reduction elements per step, and a step's matrix instructions of one wave in units of
// those of one 16x16x16 complex product on the matrix cores of its type
struct GroupTile { int m, n, k, frags; };
constexpr GroupTile kGroupTiles[5] = {{32, 32, 16, 1}, {64, 64, 16, 4}, {16, 64, 16, 1}, {64, 16, 16, 1}, {128, 64, 32, 8}};
constexpr int kSplitTile = 4;            // on the bf16 matrix cores, complex64 (split.hip)
// Index of the tile for M x N outputs of each of `jobs` blocks with reductions of K; fill: the launch has
// to fill the device.
int best_tile(int M, int N, int K, i64 jobs, bool fp64, bool fill);
constexpr int kSumChunk = 1024;       // elements of a SumSeg per workgroup
constexpr int kMaxSlabs = 16;         // arrays an output kernel can sum

// Arrays whose elementwise sum is the value of a tensor.
struct SlabList {
    const void *p[kMaxSlabs];
    int n;
};
inline SlabList one_slab(const void *p) {
    SlabList s{};
    s.p[0] = p;
    s.n = 1;
    return s;
}

// items [0, n) of the device table, all of one launch class: 0 the tiles of one fragment per wave, 1 64x64,
// 2 the bf16 tiles
inline int tile_class(int tile) { return tile == kSplitTile ? 2 : tile == 1 ? 1 : 0; }
template <typename T>
hipError_t launch_gemm_group(int cls, const GemmArgs *ops, const GroupItem *items, int n, hipStream_t s);
hipError_t launch_split_group(const GemmArgs *ops, const GroupItem *items, int n, hipStream_t s);
// work: one (segment, first element / kSumChunk) pair per workgroup
template <typename T>
hipError_t launch_sums(const SumSeg *segs, const void *const *src, const int2 *work, int n, hipStream_t s);

}  // namespace lrcc
