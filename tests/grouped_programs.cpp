// Small recorded programs for the grouped form (Program::group): their layout in a dry run, and on a device their
// values when the same program runs grouped, op by op and grouped again; and single products with long reductions.
// grouped_programs NAME [run]
#include <hip/hip_runtime.h>

#include <complex>
#include <cstdio>
#include <cstring>
#include <string>

#include "elem.hpp"
#include "plan.hpp"

using namespace lrcc;
typedef std::complex<double> cd;

namespace {

constexpr int kM = 8, kN = 8, kK = 8, kBlocks = 4;
constexpr i64 kBlock = (i64)kM * kN;
bool g_run = false;

struct Array {
    void *p = nullptr;
    std::vector<cd> h;
    explicit Array(i64 n, int seed = 0) : h(n) {
        for (i64 i = 0; i < n; ++i) h[i] = seed ? cd((i * seed) % 7 - 3, (i * (seed + 4)) % 5 - 2) : cd(1e30, 1e30);
        p = dev_alloc(n * 16);
        if (g_run && hipMemcpy(p, h.data(), n * 16, hipMemcpyHostToDevice) != hipSuccess) std::exit(3);
    }
};

std::vector<cd> read(const void *p, i64 n) {
    std::vector<cd> v(n);
    if (hipMemcpy(v.data(), p, n * 16, hipMemcpyDeviceToHost) != hipSuccess) std::exit(3);
    return v;
}

void zero(Program &P, void *p, i64 n) {
    P.ops.push_back([=](hipStream_t s) { return zero_fill<double>(p, n, s); });
    P.node(Node::ZERO, {}, p, n);
}

// C += A B for the given blocks (A, B: one kM x kK and one kK x kN matrix, C: kBlocks blocks)
void product(Program &P, const Array &A, const Array &B, void *C, std::vector<i64> blocks) {
    GemmArgs g{};
    g.shape = -1;
    g.A = A.p; g.B = B.p; g.C = C;
    g.M = kM; g.N = kN; g.K = kK;
    g.sm = Split{1, kM}; g.sn = Split{1, kN}; g.sk = Split{1, kK};
    g.Am = Strides{{0, 0, kK}}; g.Ak = Strides{{0, 0, 1}};
    g.Bk = Strides{{0, 0, kN}}; g.Bn = Strides{{0, 0, 1}};
    g.Cm = Strides{{0, 0, kN}}; g.Cn = Strides{{0, 0, 1}};
    g.bNfast = 1;
    g.alpha_re = 1;
    g.beta = 1;
    std::vector<i64> off, zeros(blocks.size(), 0);
    std::vector<int> beg{0};
    for (i64 b : blocks) { off.push_back(b * kBlock); beg.push_back((int)off.size()); }
    raw_gemm<double>(P, g, off, beg, zeros, zeros, (i64)kM * kK, (i64)kK * kN, kBlocks * kBlock);
}

std::vector<SlabList> g_lists;       // what the output step of the last run read
std::vector<cd> g_out;

void output(Program &P, void *Z, i64 n) {
    auto sum = [n](const SlabList &l) {
        g_lists.push_back(l);
        if (!g_run) return hipSuccess;
        if (hipDeviceSynchronize() != hipSuccess) return hipErrorUnknown;
        g_out.assign(n, cd(0, 0));
        for (int q = 0; q < l.n; ++q) {
            const std::vector<cd> v = read(l.p[q], n);
            for (i64 i = 0; i < n; ++i) g_out[i] += v[i];
        }
        return hipSuccess;
    };
    P.ops.push_back([=](hipStream_t) { return sum(one_slab(Z)); });
    P.node(Node::OUT, {Z}, nullptr, n).from = [=](hipStream_t, const std::vector<SlabList> &l) { return sum(l[0]); };
}

// Z from a product over half of its blocks and two over all: three arrays, the first stored in part
int partial() {
    const Array A(kM * kK, 3), B(kK * kN, 5), C(kM * kK, 2), Z(kBlocks * kBlock);
    Program P;
    zero(P, Z.p, kBlocks * kBlock);
    product(P, A, B, Z.p, {0, 1});
    product(P, C, B, Z.p, {0, 1, 2, 3});
    product(P, A, B, Z.p, {0, 1, 2, 3});
    output(P, Z.p, kBlocks * kBlock);
    if (!P.group<double>((size_t)1 << 20)) { std::printf("not grouped\n"); return 1; }
    g_lists.clear();
    if (!g_run) {
        (void)P.grouped.back().fn(nullptr);
        const SlabList &l = g_lists.at(0);
        std::printf("arrays %d\n", l.n);
        for (int q = 0; q < l.n; ++q)
            if (l.n > 1 && l.p[q] == Z.p) { std::printf("an array stored in part is the tensor's own buffer\n"); return 1; }
        return 0;
    }
    std::vector<cd> ref(kBlocks * kBlock);
    for (i64 b = 0; b < kBlocks; ++b)
        for (int m = 0; m < kM; ++m)
            for (int n = 0; n < kN; ++n) {
                cd s = 0;
                for (int k = 0; k < kK; ++k)
                    s += (C.h[m * kK + k] + A.h[m * kK + k] * (b < 2 ? 2.0 : 1.0)) * B.h[k * kN + n];
                ref[b * kBlock + m * kN + n] = s;
            }
    int bad = 0;
    for (int form = 0; form < 4; ++form) {
        P.use_grouped = form % 2 == 0;
        if (P.run(nullptr, nullptr) != hipSuccess) return 3;
        const bool same = g_out == ref;          // small whole numbers: every sum is exact
        std::printf("%s: %s\n", P.use_grouped ? "grouped" : "op by op", same ? "ok" : "wrong");
        bad += !same;
    }
    return bad ? 1 : 0;
}

void copy(Program &P, void *d, const void *src, i64 n) {
    P.ops.push_back([=](hipStream_t s) { return hipMemcpyAsync(d, src, n * 16, hipMemcpyDeviceToDevice, s); });
    P.node(Node::COPY, {src}, d, n);
}
void add(Program &P, void *d, const void *src, i64 n) {
    P.ops.push_back([=](hipStream_t s) { return add_inplace<double>(d, src, n, s); });
    P.node(Node::ADD, {src}, d, n);
}

// T = C1 + C2, arrays that no op writes, read by a product
int constants() {
    const i64 n = kBlocks * kBlock;
    const Array A(kM * kK, 3), C1(kK * kN, 2), C2(kK * kN, 5), T(kK * kN), Z(n);
    Program P;
    copy(P, T.p, C1.p, kK * kN);
    add(P, T.p, C2.p, kK * kN);
    zero(P, Z.p, n);
    product(P, A, T, Z.p, {0, 1, 2, 3});
    output(P, Z.p, n);
    const bool made = P.group<double>((size_t)1 << 20);
    bool sums = false;
    for (const auto &l : P.grouped) sums = sums || l.name.find("sums") != std::string::npos;
    std::printf("%s\n", !made ? "not grouped" : sums ? "summed" : "grouped, the operand is never formed");
    return made && !sums ? 1 : 0;
}

// T is cleared and nothing is added to it (a product without jobs); other programs read it
int cleared() {
    const i64 n = kBlocks * kBlock;
    const Array A(kM * kK, 3), B(kK * kN, 5), T(n), Z(n);
    Program P;
    zero(P, T.p, n);
    zero(P, Z.p, n);
    product(P, A, B, Z.p, {0, 1, 2, 3});
    const bool made = P.group<double>((size_t)1 << 20, true);
    bool clears = false;
    for (const auto &l : P.grouped) clears = clears || l.name == "clear";
    std::printf("%s\n", !made ? "not grouped" : clears ? "cleared" : "grouped, the tensor is never cleared");
    return made && !clears ? 1 : 0;
}

// the extra arrays take at most 1 GiB and an eighth of the free memory: a program that needs more runs op by op
int budget() {
    const size_t gib = (size_t)1 << 30;
    if (group_budget_of(288 * gib) != gib || group_budget_of(8 * gib) != gib || group_budget_of(4 * gib) != gib / 2 ||
        group_budget_of(0) != 0) { std::printf("budget\n"); return 1; }
    const i64 n = kBlocks * kBlock;
    const Array A(kM * kK, 3), B(kK * kN, 5), Z(n);
    Program P;
    zero(P, Z.p, n);
    product(P, A, B, Z.p, {0, 1});
    product(P, A, B, Z.p, {0, 1, 2, 3});
    output(P, Z.p, n);
    const size_t need = 2 * n * 16;
    const bool less = P.group<double>(group_budget_of(8 * need - 8)), enough = P.group<double>(group_budget_of(8 * need));
    std::printf("%d %d\n", less, enough);
    return !less && enough ? 0 : 1;
}

// Relative error of one complex64 product of kM x n and n x kN random matrices on the fp32 (64x64) and bf16 tiles
// in one piece each, against 64 bits
int reduction(int n) {
    constexpr int M = 64, N = 32;
    typedef std::complex<float> cf;
    unsigned long long state = 12345;
    auto rnd = [&] {                     // uniform in [-1, 1), mean zero
        state = state * 6364136223846793005ull + 1442695040888963407ull;
        return (float)((double)(state >> 40) / (1 << 23) - 1.0);
    };
    std::vector<cf> A((size_t)M * n), B((size_t)n * N), C(M * N);
    for (cf &x : A) x = cf(rnd(), rnd());
    for (cf &x : B) x = cf(rnd(), rnd());
    std::vector<cd> ref(M * N, 0);
    for (int k = 0; k < n; ++k)
        for (int m = 0; m < M; ++m) {
            const cd a = A[(size_t)m * n + k];
            for (int j = 0; j < N; ++j) {
                const cd b = B[(size_t)k * N + j];
                ref[m * N + j] += cd(a.real() * b.real() - a.imag() * b.imag(), a.real() * b.imag() + a.imag() * b.real());
            }
        }
    auto up = [](const void *p, size_t bytes) {
        void *d = nullptr;
        if (hipMalloc(&d, bytes) != hipSuccess || hipMemcpy(d, p, bytes, hipMemcpyHostToDevice) != hipSuccess) std::exit(3);
        return d;
    };
    const i64 zero64 = 0;
    const int beg[2] = {0, 1};
    GemmArgs g{};
    g.A = up(A.data(), A.size() * sizeof(cf));
    g.B = up(B.data(), B.size() * sizeof(cf));
    g.C = up(C.data(), C.size() * sizeof(cf));
    g.M = M; g.N = N; g.K = n;
    g.sm = split_magic(Split{1, M}); g.sn = split_magic(Split{1, N}); g.sk = split_magic(Split{1, n});
    g.Am = Strides{{0, 0, n}}; g.Ak = Strides{{0, 0, 1}};
    g.Bk = Strides{{0, 0, N}}; g.Bn = Strides{{0, 0, 1}};
    g.Cm = Strides{{0, 0, N}}; g.Cn = Strides{{0, 0, 1}};
    g.bNfast = 1;
    g.alpha_re = 1;
    g.offC = g.segA = g.segB = (const i64 *)up(&zero64, sizeof zero64);
    g.segBeg = (const int *)up(beg, sizeof beg);
    g.njobs = g.njobs_all = g.ksplit = 1;
    double err[2], norm = 0;
    for (const cd &r : ref) norm += std::norm(r);
    for (int q = 0; q < 2; ++q) {
        g.shape = q ? kSplitTile : 1;
        if (launch_gemm<float>(g, nullptr) != hipSuccess || hipDeviceSynchronize() != hipSuccess ||
            hipMemcpy(C.data(), g.C, C.size() * sizeof(cf), hipMemcpyDeviceToHost) != hipSuccess) return 3;
        double e = 0;
        for (int i = 0; i < M * N; ++i) e += std::norm(cd(C[i]) - ref[i]);
        err[q] = std::sqrt(e / norm);
    }
    std::printf("%d %.3e %.3e\n", n, err[0], err[1]);
    return 0;
}

}  // namespace

int main(int argc, char **argv) {
    if (argc < 2) return 2;
    const std::string name = argv[1];
    g_run = argc > 2 && !std::strcmp(argv[2], "run");
    g_dry_run = !g_run;
    if (name == "partial") return partial();
    if (name == "reduction") {
        for (int n : {40, 320, 1600, 12800, 98304})
            if (reduction(n)) return 3;
        return 0;
    }
    if (name == "constants") return constants();
    if (name == "budget") return budget();
    if (name == "cleared") return cleared();
    return 2;
}
