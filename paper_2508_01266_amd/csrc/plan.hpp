// Host-side planner: k-blocked tensors and their contractions as GEMM job lists.
#pragma once
#include <array>
#include <complex>
#include <functional>
#include <map>
#include <memory>
#include <stdexcept>
#include <string>
#include <vector>

#include "common.hpp"
#include "group.hpp"

namespace lrcc {

// A momentum-conserving tensor stored as dense blocks (Sec. II.A, Eq. momentum).
// Indices have class 'o' or 'v'.  Four-index tensors obey
// sg[0] k0 + sg[1] k1 + sg[2] k2 + sg[3] k3 = 0 on the k mesh km and are stored as
// [k0][k1][k2] blocks (k3 implied); two-index tensors are k-diagonal, [k0]
// blocks.  An optional right-hand-side axis of extent nR sits at the start of
// every block: block = [R][d0][d1]...  Elements are interleaved complex.
struct KT {
    void *p = nullptr;
    std::string cls;
    int sg[4] = {1, 1, -1, -1};
    int nR = 0;
    int nk = 0, no = 0, nv = 0;   // nk = km.size()
    KMesh km;
    int nidx() const { return (int)cls.size(); }
    int ext(int d) const { return cls[d] == 'o' ? no : nv; }
    i64 inner() const {
        i64 e = nR > 0 ? nR : 1;
        for (int d = 0; d < nidx(); ++d) e *= ext(d);
        return e;
    }
    i64 nblocks() const {
        i64 b = 1;
        for (int d = 0; d < nidx() - 1; ++d) b *= nk;
        return b;
    }
    i64 count() const { return inner() * nblocks(); }
};

struct LrccError : std::runtime_error {
    int code;
    LrccError(int c, const std::string &m) : std::runtime_error(m), code(c) {}
};

// Event timing of recorded launches: pairs of events recorded on the launch
// stream around every op with a given tag (and around whole program runs).
enum { TAG_NONE = 0, TAG_LADDER = 1, TAG_PROGRAM = 2, TAG_BUILD = 3, NTAGS = 4 };
struct Profiler {
    bool on = false;
    std::vector<std::pair<int, std::pair<hipEvent_t, hipEvent_t>>> marks;
    std::vector<hipEvent_t> pool;
    hipEvent_t ev();
    void record(int tag, hipEvent_t a, hipEvent_t b) { marks.push_back({tag, {a, b}}); }
    // sums (ms, count) per tag, recycles the events
    void read(double *ms, long long *cnt);
    ~Profiler();
};

// A tunable launch of a recorded program: the op index and a setter for its
// variant (candidate 0 or 1).
struct Tunable {
    size_t op;
    int ncand;                           // number of valid candidates
    std::function<void(int)> set;
};

// Data flow of one recorded op of a program that may run grouped (see Program::group).  Tensors are
// identified by their base pointers; `acc`: adds to the tensor it writes; `full`: writes every element.
struct Node {
    enum Kind { GEMM, ZERO, COPY, ADD, WRITE, OUT } kind = GEMM;
    size_t op = 0;                    // index into Program::ops
    std::vector<const void *> reads;
    void *write = nullptr;            // tensor written (null for OUT)
    i64 count = 0;                    // its elements
    bool acc = false, full = true;
    bool real = false;                // real numbers, half the size: one WRITE, in their own buffer only
    // WRITE: the op writing to dst, or adding to it.  OUT: the op reading, for each of its reads, the sum of
    // the arrays that make it up
    std::function<hipError_t(hipStream_t, void *dst, bool acc)> write_to;
    std::function<hipError_t(hipStream_t, const std::vector<SlabList> &)> from;
    // further tensors the op of a WRITE node stores in full, always in their own buffers
    std::vector<std::pair<void *, i64>> also;
};

// Most bytes of the extra arrays of one grouped form, by the free device memory: 1 GiB (six doubles arrays of
// 64 MB, the largest that are split over several, with room for the smaller tensors), and an eighth of what is
// free, as for the ladder's scratch arrays, so that programs never take the last of it.
constexpr size_t group_budget_of(size_t free_bytes) {
    return free_bytes / 8 < ((size_t)1 << 30) ? free_bytes / 8 : (size_t)1 << 30;
}

// A recorded sequence of device launches plus the device memory it owns.
struct Program {
    std::vector<std::function<hipError_t(hipStream_t)>> ops;
    std::vector<int> tags;  // per op (TAG_NONE unless set by tag_last)
    std::vector<std::string> names;  // per op, for the per-op timing report
    void name_last(const std::string &n) {
        names.resize(ops.size());
        names.back() = n;
    }
    // Grouped form: the ops' data flow (one node per op where every op has one) and the launches made
    // from it by group(): the products of one dependency level as one launch over a table of work
    // items, with separate arrays for contributions to one tensor that would have to wait for each
    // other.  Empty: the program runs op by op.
    std::vector<Node> nodes;
    struct Launch {
        std::function<hipError_t(hipStream_t)> fn;
        int tag;
        std::string name;
    };
    std::vector<Launch> grouped;
    std::map<size_t, int> group_tiles;   // tiles of the products that share launches in it, by op
    bool use_grouped = true;             // run the grouped form where there is one
    bool runs_grouped() const { return use_grouped && !grouped.empty(); }
    // node of the op recorded last
    Node &node(Node::Kind k, std::vector<const void *> reads, void *write, i64 count, bool acc = false) {
        Node n;
        n.kind = k;
        n.op = ops.size() - 1;
        n.reads = std::move(reads);
        n.write = write;
        n.count = count;
        n.acc = acc;
        nodes.push_back(std::move(n));
        return nodes.back();
    }
    // make the grouped form if the data flow allows it and its extra arrays take at most `budget`
    // bytes; returns whether it was made.  keep: every tensor the program writes is read by others (else
    // only through OUT nodes)
    template <typename T>
    bool group(size_t budget, bool keep = false);
    template <typename T>
    bool make_grouped(size_t budget, bool keep);
    std::vector<Tunable> tunables;
    // numbers of a tuning choice: one per tunable launch and, where there is a grouped form, 0 grouped or 1 op by op
    size_t choices() const { return tunables.size() + (grouped.empty() ? 0 : 1); }
    bool tuned = false;
    std::string tune_key;
    // Time every tunable op under each candidate (full program runs, so the
    // recomputed outputs stay valid) and keep the fastest per op.
    hipError_t autotune(hipStream_t s, std::vector<int> &choice);
    void apply(const std::vector<int> &choice);
    std::vector<void *> owned;
    i64 flops = 0;       // executed real flops of the recorded GEMMs and ladder
    i64 last_flops = 0;  // executed flops of the op recorded last
    i64 tag_flops[NTAGS] = {0, 0, 0, 0};
    void tag_last(int t) {
        tags.resize(ops.size(), TAG_NONE);
        tags.back() = t;
        tag_flops[t] += last_flops;
    }
    hipError_t run(hipStream_t s, Profiler *prof = nullptr);
    hipError_t run_range(hipStream_t s, size_t begin, size_t end);
    // the recorded GEMM launches (op index -> arguments as tuned, precision, executed flops)
    struct GemmOp {
        std::shared_ptr<GemmArgs> args;
        bool fp64;
        i64 flops;
        std::vector<i64> offC;          // host copies of the job lists
        std::vector<int> segBeg;
        std::vector<float> jscale;
        i64 sizeC;
    };
    std::map<size_t, GemmOp> gemm_ops;
    // real flops of the matrix-core instructions of the GEMM launches with tag t: 8 per complex
    // multiply-add formed, 48 for the tiles that form a real product from six bf16 ones
    double tag_mfma_flops(int t) const;
    // ladder path of a sigma program: 1 integrals rebuilt in LDS, 2 stored blocks, 3 blocks built
    // one momentum class at a time (0: no ladder term)
    int ladder_path = 0;
    // the rebuild-in-LDS ladder launch of a sigma program (for multi-chain launches)
    std::shared_ptr<LadderArgs> ladder_args;
    size_t ladder_op = (size_t)-1;
    // Replay through a HIP graph captured on first use for this key (the
    // pointers the recorded launches read); `s` must not be the null stream.
    typedef std::array<const void *, 5> GraphKey;
    std::map<GraphKey, hipGraphExec_t> graphs;
    hipError_t run_graph(hipStream_t s, const GraphKey &key);
    void drop_graphs();
    void *alloc(size_t bytes);
    ~Program();
};

// C[cl] (+)= alpha * sum A[al] B[bl]; labels are one character per index, 'R'
// for the right-hand-side axis (first in a label string when present).
// pack: label pairs ("pq" per pair, at most one pair per GEMM index group) over which
// the launches run on unique pairs only: momentum blocks k_p <= k_q, and p < q inside the
// diagonal blocks k_p = k_q (triangle splits).  A summed pair must be antisymmetric in both
// operands (factor 2).  An output pair leaves C defined only on those unique pairs (the
// others are not written; with accumulate false C is zeroed first): with factor 2 for a
// consumer that antisymmetrises C in the pair, or with its true values when the pair's first
// label is in `exact`, for a consumer that reads C through the same packing.
template <typename T>
void contract(Program &P, const KT &C, const std::string &cl, const KT &A, const std::string &al, const KT &B,
              const std::string &bl, std::complex<double> alpha, bool accumulate = true,
              const std::string &pack = "", const std::string &exact = "");

// Raw strided GEMM with explicit job/segment lists (host vectors are uploaded).
// sizeA/B/C are the element counts of the operands: every address the GEMM can
// form is checked against them before the launch is recorded.
// jscale (optional, one per job) multiplies alpha job by job.
template <typename T>
void raw_gemm(Program &P, GemmArgs g, const std::vector<i64> &offC, const std::vector<int> &segBeg,
              const std::vector<i64> &segA, const std::vector<i64> &segB, i64 sizeA, i64 sizeB, i64 sizeC,
              const std::vector<float> &jscale = {});

// Placeholder-or-real device allocation honouring g_dry_run.
void *dev_alloc(size_t bytes);
void dev_free(void *p);
// starts (ends) a dry run; bytes of the placeholder at p in it (SIZE_MAX: not the start of one)
void dry_run(bool on);
size_t dry_bytes(const void *p);

}  // namespace lrcc
